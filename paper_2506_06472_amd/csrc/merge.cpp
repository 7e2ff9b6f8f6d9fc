#include "merge.h"

#include <hip/hip_runtime_api.h>

#include "kernels.h"

namespace tio {

namespace {

// Between kernels j - 1 and j nothing is issued, waited for or recorded.
bool nothing_between(const Plan &p, int j) {
    return p.entries_at[j].empty() && p.kernel_wait_pre[j].empty() && p.kernel_wait_off[j].empty() && !p.kernel_needs_event[j - 1];
}

struct Schedule {
    const Program &prog;
    const Plan &plan;
    const std::vector<std::vector<uint64_t>> &at;

    // The two kernels share no memory that one of them writes (a range may be taken over from a tensor that dies at one by one that
    // another gives birth to); shared: a tensor that the merged launch hands from one to the other itself, or -1.
    bool independent(int k0, int k1, int shared) const {
        const KernelRec &x = prog.kernels[k0], &y = prog.kernels[k1];
        for (int i = 0; i < kMaxRoles; ++i)
            for (int j = 0; j < kMaxRoles; ++j) {
                if (x.t[i] < 0 || y.t[j] < 0 || !((x.fl[i] | y.fl[j]) & 2) || (x.t[i] == shared && y.t[j] == shared)) continue;
                const uint64_t a = at[k0][i], b = at[k1][j];
                if (a < b + prog.tensors[y.t[j]].bytes && b < a + prog.tensors[x.t[i]].bytes) return false;
            }
        return true;
    }

    // updates in a row; the two gradients of a linear layer where both products are small; the row products of attention's backward pass
    // with that pass where its kernel computes them
    int merged_from(int k) const {
        const int N = (int)prog.kernels.size();
        const KernelRec &r = prog.kernels[k];
        const tio_model_cfg &c = prog.cfg;
        auto next = [&](int j, int op) { return j < N && prog.kernels[j].op == op && nothing_between(plan, j); };
        if (r.op == OP_ADAMW) {
            auto fits = [&](int j) {               // an update joins a launch if it is independent of every one in it
                for (int i = k; i < j; ++i)
                    if (!independent(i, j, -1)) return false;
                return true;
            };
            int n = 1;
            while (n < k::kAdamwMax && next(k + n, OP_ADAMW) && fits(k + n)) ++n;
            return n;
        }
        if (r.op == OP_GEMM_DX && next(k + 1, OP_GEMM_DW) && c.precision == TIO_PREC_FP32) {
            const KernelRec &w = prog.kernels[k + 1];
            return k::gemm_f32_pairs(r.p[0], r.p[1], w.p[0], w.p[1]) && independent(k, k + 1, -1) ? 2 : 1;
        }
        if (r.op == OP_ATTN_BWD_PRE && next(k + 1, OP_ATTN_BWD))
            return k::attn_bwd_has_delta(c.precision, c.seq_len, c.n_heads, c.d_model / c.n_heads) && independent(k, k + 1, r.t[2]) ? 2 : 1;
        return 1;
    }
};

}  // namespace

std::vector<int> merged_launches(const Program &prog, const Plan &plan, const std::vector<std::vector<uint64_t>> &at) {
    const Schedule s{prog, plan, at};
    std::vector<int> count(prog.kernels.size(), 1);
    for (size_t k = 0; k < count.size(); k += count[k]) count[k] = s.merged_from((int)k);
    return count;
}

}  // namespace tio
