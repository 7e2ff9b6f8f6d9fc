// Which neighbours of the schedule go out in one launch, without a GPU.
//   merge_host independent          updates of one launch share no memory, neighbours or not; exit status 0: passed
//   merge_host launches <config>    the launches of more than one kernel under the uncapped plan, a line each: op of the first, kernels,
//                                   and for the two gradients of a linear layer the rows of their output tiles
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../paper_2506_06472_amd/csrc/kernels.h"
#include "../paper_2506_06472_amd/csrc/merge.h"

using namespace tio;

namespace {

// three updates whose gradients, weights and moments lie one after the other; then the third one's weights in the place of the gradient
// of the first, second and third
int independent() {
    Program p;
    Plan plan;
    std::vector<std::vector<uint64_t>> at;
    for (int i = 0; i < 3; ++i) {
        KernelRec r{OP_ADAMW, {}, {}, {64}, 0};
        std::vector<uint64_t> where(kMaxRoles, UINT64_MAX);
        for (int role = 0; role < kMaxRoles; ++role) r.t[role] = -1;
        for (int role : {0, 1, 3, 4}) {
            r.t[role] = (int)p.tensors.size();
            r.fl[role] = role == 0 ? 1 : 3;
            where[role] = 256 * p.tensors.size();
            p.tensors.push_back({256, KIND_ACT, ""});
        }
        p.kernels.push_back(r);
        at.push_back(where);
    }
    plan.entries_at.resize(3); plan.kernel_wait_pre.resize(3); plan.kernel_wait_off.resize(3); plan.kernel_needs_event.resize(3);
    if (merged_launches(p, plan, at) != std::vector<int>{3, 1, 1}) { std::printf("three independent updates\n"); return 1; }
    const std::vector<int> want[] = {{2, 1, 1}, {1, 2, 1}};      // the third on its own; the first on its own
    const int moved[] = {2, 1}, over[] = {0, 0};
    for (int i = 0; i < 2; ++i) {
        auto a = at;
        a[moved[i]][1] = at[over[i]][0];
        if (merged_launches(p, plan, a) != want[i]) { std::printf("update %d over the gradient of update %d\n", moved[i], over[i]); return 1; }
    }
    return 0;
}

int launches(char **argv) {
    tio_model_cfg c{};
    int32_t *const field[] = {&c.arch, &c.n_layers, &c.d_model, &c.n_heads, &c.d_ff, &c.vocab, &c.seq_len, &c.batch, &c.precision, &c.micro_batches};
    for (size_t i = 0; i < sizeof field / sizeof *field; ++i) *field[i] = std::atoi(argv[i]);
    c.norm_eps = 1e-5f; c.rope_theta = 1e4f;
    const Program p = build_program(c);
    const Trace t = trace_from_program(p);
    const Plan plan = build_plan(t, analyze(t), (uint64_t)1 << 62, 0, tio_plan_opts{1, 24, 0, 0, 0, 0, 0, 0});
    std::vector<std::vector<uint64_t>> at(p.kernels.size(), std::vector<uint64_t>(kMaxRoles, UINT64_MAX));
    for (size_t k = 0; k < at.size(); ++k)
        for (int r = 0; r < kMaxRoles; ++r)
            if (p.kernels[k].t[r] >= 0) at[k][r] = address_at(plan, p.kernels[k].t[r], (int)k);
    const std::vector<int> count = merged_launches(p, plan, at);
    for (size_t k = 0; k < count.size(); k += count[k]) {
        if (count[k] < 2) continue;
        std::printf("%d %d", p.kernels[k].op, count[k]);
        if (p.kernels[k].op == OP_GEMM_DX)
            for (size_t j : {k, k + 1}) {
                int rows = 0, cols = 0;
                k::gemm_f32_tile(p.kernels[j].p[0], p.kernels[j].p[1], &rows, &cols);
                std::printf(" %d", rows);
            }
        std::printf("\n");
    }
    return 0;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc == 2 && !std::strcmp(argv[1], "independent")) return independent();
    if (argc == 12 && !std::strcmp(argv[1], "launches")) return launches(argv + 2);
    return 2;
}
