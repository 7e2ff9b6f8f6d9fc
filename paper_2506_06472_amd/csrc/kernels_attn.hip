// Causal self-attention, forward and backward, on the packed [S, 3d] q|k|v layout (no head transposes ever touch HBM), in
// fp32 arithmetic on the fp32 matrix instruction: the fp32 workloads, and bf16 tensors with head dimension 32 (the
// probabilities stay fp32).  bf16 with head dimension 64 or 128 runs on the bf16 matrix cores (kernels_attn_mfma.hip).
//
// A wavefront owns 32 query rows (forward, dQ) or 32 key rows (dK/dV) and takes the other side in tiles of 32 rows straight
// from global memory into operand registers: no LDS tiles and no barriers in the loop.  Scores are produced transposed
// (other side x own rows), so an own row is a lane index: the softmax statistics live in one lane (plus one exchange with
// lane + 32), and register r of the score accumulator is, as it is, the second product's operand for the two rows
// 8 (r/4) + r%4 and that + 4 (the matrix instruction takes one contraction row from each lane half).
// v_mfma_f32_32x32x2_f32 multiplies and adds in fp32.
//
// Bound: the matrix cores (157 TFLOP/s) for long sequences, memory latency and idle compute units for the short ones the
// fp32 workloads have.  So the four (or eight) wavefronts of a workgroup share 32 own rows, take every fourth tile each and merge at
// the end, in wavefront order.  Giving every wavefront 32 rows of its own instead lost at every size, also where the rows fill the
// chip many times over (fp32, forward and backward, microseconds, shared / own rows: 4 x 333 x 4 x 32 43 / 117, 8 x 512 x 8 x 64
// 218 / 257, 4 x 2048 x 12 x 64 1580 / 2155): the shared form has four times the workgroups of a quarter the length, and the
// last rows of a causal mask end sooner.  With a row per lane on the vector ALU the first of these took 446.
// Since then, with delta, dQ and dK/dV in one launch, tiles behind buffer descriptors, row statistics handed round the lanes, and a
// merge that four wavefronts share: 4 x 333 x 4 x 32 43.1 -> 25.0, 2 x 64 x 4 x 32 21.7 -> 10.7, 8 x 512 x 8 x 64 218 -> 165.
// Statistics are fp32 (log-sum-exp saved for the backward pass, which recomputes the probabilities from it); every sum has a
// fixed order; the blocks of dQ and those of dK/dV are workgroups of their own, so that no atomics are needed.
#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

constexpr int TPB = 256;
constexpr int ROWS = 32;         // own rows of a wavefront, and rows of a tile of the other side

// Up to 32 rows of one head from a row r0 on, behind a buffer descriptor: rows past the sequence read as zeros.  An element's address is
// one register that the lane keeps for the whole kernel, a uniform offset and a constant; with 64-bit addresses per row and the clamp
// to the last row the address arithmetic was most of the instructions of a kernel whose code runs once or twice, and reading
// the code took longer than running it.
template <typename T> struct Rows {
    static constexpr bool WIDE = false;
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t pitch;
    __device__ __forceinline__ Rows(const T *head, int64_t ld, int r0, int Tn, int dh) {
        const int n = Tn - r0 < ROWS ? Tn - r0 : ROWS;
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(head + r0 * ld), 0, (int)(uint32_t)(((n - 1) * ld + dh) * (int64_t)sizeof(T)), 0x00020000);
        pitch = (uint32_t)(ld * (int64_t)sizeof(T));
    }
};
// The same where 32 rows span 4 GiB and more, which 32-bit offsets do not reach: 64-bit addresses, rows past the sequence read its last.
template <typename T> struct WideRows {
    static constexpr bool WIDE = true;
    const T *head;
    int64_t ld;
    int n;
    __device__ __forceinline__ WideRows(const T *head, int64_t ld, int r0, int Tn, int) : head(head + r0 * ld), ld(ld), n(Tn - r0) {}
    __device__ __forceinline__ const T *row(int r) const { return head + (r < n ? r : n - 1) * ld; }
};
__device__ __forceinline__ void load4(float *f, const float *p) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
__device__ __forceinline__ void load4(float *f, const bf16_t *p) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
}
__device__ __forceinline__ void load4(float *f, const Rows<float> &x, uint32_t off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(x.rsrc, (int)off, 0, 0);
    f[0] = __uint_as_float(v[0]); f[1] = __uint_as_float(v[1]); f[2] = __uint_as_float(v[2]); f[3] = __uint_as_float(v[3]);
}
__device__ __forceinline__ void load4(float *f, const Rows<bf16_t> &x, uint32_t off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(x.rsrc, (int)off, 0, 0);
    f[0] = __uint_as_float(v[0] << 16); f[1] = __uint_as_float(v[0] & 0xffff0000u);
    f[2] = __uint_as_float(v[1] << 16); f[3] = __uint_as_float(v[1] & 0xffff0000u);
}
__device__ __forceinline__ float load1(const Rows<float> &x, uint32_t off, uint32_t uniform) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x.rsrc, (int)off, (int)uniform, 0));
}
__device__ __forceinline__ float load1(const Rows<bf16_t> &x, uint32_t off, uint32_t uniform) {
    return __uint_as_float((uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(x.rsrc, (int)off, (int)uniform, 0) << 16);
}
__device__ __forceinline__ void store4(float *p, const float *f) { *reinterpret_cast<float4 *>(p) = make_float4(f[0], f[1], f[2], f[3]); }
__device__ __forceinline__ void store4(bf16_t *p, const float *f) {
    *reinterpret_cast<uint2 *>(p) = make_uint2(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]));
}
__device__ __forceinline__ float max_halves(float x) { return fmaxf(x, __shfl_xor(x, 32, 64)); }
__device__ __forceinline__ float sum_halves(float x) { return x + __shfl_xor(x, 32, 64); }
// row of a 32-row tile that register r of an accumulator holds in lane half lhi
__device__ __forceinline__ int acc_row(int r, int lhi) { return 8 * (r >> 2) + 4 * lhi + (r & 3); }
__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}
__device__ __forceinline__ floatx16 mfma(float a, float b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// One row per lane pair, all of the head dimension: the operand whose contraction index is the head dimension.  A lane half
// holds elements 8 c + 4 half .. + 3 of chunk c, on both operands of a product alike.
template <int DH> struct RowFrag {
    float f[DH / 2];
    template <typename T> __device__ __forceinline__ void load(const WideRows<T> &x, int lane) {
        const T *row = x.row(lane & 31) + 4 * (lane >> 5);
#pragma unroll
        for (int c = 0; c < DH / 8; ++c) load4(f + 4 * c, row + 8 * c);
    }
    template <typename T> __device__ __forceinline__ void load(const Rows<T> &x, int lane) {
        const uint32_t off = (uint32_t)(lane & 31) * x.pitch + (uint32_t)(lane >> 5) * (4 * sizeof(T));
#pragma unroll
        for (int c = 0; c < DH / 8; ++c) load4(f + 4 * c, x, off + c * 8 * (uint32_t)sizeof(T));
    }
};
template <int DH> __device__ __forceinline__ floatx16 dot_rows(const RowFrag<DH> &a, const RowFrag<DH> &b) {
    floatx16 s = zero16();
#pragma unroll
    for (int i = 0; i < DH / 2; ++i) s = mfma(a.f[i], b.f[i], s);
    return s;
}
// A 32-row tile whose rows are the contraction index: register (i, r) is column 32 i + lane % 32 of row acc_row(r).
template <int DH> struct ColFrag {
    float f[DH / 32][16];
    template <typename T> __device__ __forceinline__ void load(const WideRows<T> &x, int lane) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const T *row = x.row(acc_row(r, lane >> 5)) + (lane & 31);
#pragma unroll
            for (int i = 0; i < DH / 32; ++i) f[i][r] = to_f32(row[32 * i]);
        }
    }
    template <typename T> __device__ __forceinline__ void load(const Rows<T> &x, int lane) {
        const uint32_t off = (uint32_t)(4 * (lane >> 5)) * x.pitch + (uint32_t)(lane & 31) * (uint32_t)sizeof(T);
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int i = 0; i < DH / 32; ++i) f[i][r] = load1(x, off + 32 * i * (uint32_t)sizeof(T), (uint32_t)acc_row(r, 0) * x.pitch);
    }
    // acc[i] += (columns 32 i ..)^T . p
    __device__ __forceinline__ void add_to(floatx16 (&acc)[DH / 32], const floatx16 &p) const {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int i = 0; i < DH / 32; ++i) acc[i] = mfma(f[i][r], p[r], acc[i]);
    }
};

// Workgroup -> head and first own row; all row blocks of a head go to one XCD (its L2 then holds the head's other side).
// false: no such head.
__device__ __forceinline__ bool place(int64_t heads, int Tn, bool long_last, unsigned block, int64_t &bh, int &r0) {
    const int nblk = (Tn + ROWS - 1) / ROWS;
    const int slot = (int)(block >> 3);
    bh = (int64_t)(slot / nblk) * 8 + (int)(block & 7);
    const int blk = slot % nblk;
    r0 = (long_last ? nblk - 1 - blk : blk) * ROWS;           // longest rows first
    return bh < heads;
}
// LDS of the merge: the wavefronts' accumulators of one 32-column block
template <int NW> constexpr int merge_floats() { return NW * 16 * 64; }
// Sums of the wavefronts' accumulators, in wavefront order, stored to the rows the lanes hold (nullptr: no such row).  Wavefronts 0 to 3
// sum and store one of the four groups of four consecutive columns each: with all of it in wavefront 0 the others stood idle for the
// longest serial part of a short sequence.  weight[w] is applied to wavefront w's accumulators, scale to the sum.
template <typename T, int DH, int NW>
__device__ __forceinline__ void merge_store(const floatx16 (&acc)[DH / 32], float *lds, int wave, int lane, const float (&weight)[NW], float scale,
                                            T *row) {
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) {
        __syncthreads();                                      // the block before has been read
#pragma unroll
        for (int r = 0; r < 16; ++r) lds[(wave * 16 + r) * 64 + lane] = acc[i][r];
        __syncthreads();
        if (wave < 4) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = lds[(4 * wave + e) * 64 + lane] * weight[0];
#pragma unroll
                for (int w = 1; w < NW; ++w) v[e] += lds[(w * 16 + 4 * wave + e) * 64 + lane] * weight[w];
                v[e] *= scale;
            }
            if (row) store4(row + 32 * i + 8 * wave + 4 * (lane >> 5), v);
        }
    }
}

// ---------------------------------------------------------------- forward
template <template <typename> class R, typename T, int DH, int NW>
__global__ void __launch_bounds__(NW * 64) attn_fwd_k(const T *__restrict__ qkv, T *__restrict__ o, float *__restrict__ lse,
                                                  int64_t heads, int Tn, int64_t H, float scale) {
    __shared__ float part[merge_floats<NW>()];
    __shared__ float stat[2][NW][ROWS];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    int64_t bh;
    int q0;
    if (!place(heads, Tn, true, blockIdx.x, bh, q0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q = q0 + l32;
    const T *base = qkv + b * Tn * ld + h * DH;
    RowFrag<DH> qf;
    qf.load(R<T>(base, ld, q0, Tn, DH), lane);
    floatx16 acc[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) acc[i] = zero16();
    float m = -INFINITY, l = 0.f;
    const int ntiles = q0 / ROWS + 1;                         // every tile holds a key that each of the rows sees
    for (int t = wave; t < ntiles; t += NW) {
        const int j0 = t * ROWS;
        RowFrag<DH> kf;
        ColFrag<DH> vf;
        kf.load(R<T>(base + d, ld, j0, Tn, DH), lane);
        vf.load(R<T>(base + 2 * d, ld, j0, Tn, DH), lane);
        floatx16 s = dot_rows(kf, qf);
        const float m_old = m;
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = j0 + acc_row(r, lhi) <= q ? s[r] * scale : -INFINITY;
            tmax = fmaxf(tmax, s[r]);
        }
        m = fmaxf(m, max_halves(tmax));
        const float ref = m == -INFINITY ? 0.f : m;           // scores of -inf so far: probabilities 0, not NaN
        const float corr = expf(m_old - ref);
        l *= corr;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[r] = expf(s[r] - ref); l += s[r]; }
#pragma unroll
        for (int i = 0; i < DH / 32; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] *= corr;
        vf.add_to(acc, s);
    }
    l = sum_halves(l);
    if (lhi == 0) { stat[0][wave][l32] = m; stat[1][wave][l32] = l; }
    __syncthreads();
    float f[NW], M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, stat[0][w][l32]);
    l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {                 // a wavefront without a tile has maximum -inf and sum 0
        f[w] = expf(stat[0][w][l32] - (M == -INFINITY ? 0.f : M));
        l += stat[1][w][l32] * f[w];
    }
    m = M;
    merge_store<T, DH, NW>(acc, part, wave, lane, f, 1.0f / l, q < Tn ? o + (b * Tn + q) * d + h * DH : nullptr);
    if (wave == 0 && lhi == 0 && q < Tn) lse[bh * Tn + q] = m + logf(l);
}

// ---------------------------------------------------------------- backward
// delta[b,h,t] = sum_e dO[s,h,e] * O[s,h,e].  dh / (elements per 16 bytes) consecutive lanes share one (s, h):
// the wavefront reads consecutive 16-byte chunks, and the partial sums meet in a fixed xor-shuffle order, that of row_dot.
template <typename T>
__global__ void __launch_bounds__(TPB) attn_bwd_pre_k(const T *__restrict__ dO, const T *__restrict__ O,
                                                      float *__restrict__ delta, int64_t Bn, int64_t Tn, int64_t H, int64_t dh) {
    constexpr int V = Vec16<T>::N;
    const int G = (int)(dh / V);                                     // lanes per (s, h): a power of two, at most 64
    const int64_t idx = (int64_t)blockIdx.x * TPB + threadIdx.x;    // chunk index = ((s * H + h) * G + g)
    const bool ok = idx < Bn * Tn * H * G;
    float sum = 0.f;
    if (ok) {
        Vec16<T> x, y; x.load(dO + idx * V); y.load(O + idx * V);
        float fx[V], fy[V]; x.get(fx); y.get(fy);
#pragma unroll
        for (int i = 0; i < V; ++i) sum = fmaf(fx[i], fy[i], sum);
    }
    for (int o = 1; o < G; o <<= 1) sum += __shfl_xor(sum, o, 64);
    if (ok && idx % G == 0) {
        const int64_t sh = idx / G, s = sh / H, h = sh % H;
        const int64_t b = s / Tn, t = s % Tn;
        delta[(b * H + h) * Tn + t] = sum;
    }
}

// Operands of the backward pass.  O: nullptr, or the forward pass's output, from which delta is then computed here and written.
template <typename T> struct BwdArgs {
    const T *dO, *qkv, *O;
    const float *lse;
    float *delta;
    T *dqkv;
    int64_t heads, H;
    int Tn;
    float scale;
};
// sum over the head dimension of g * x, for the row a lane pair holds; the same in both lanes, and the bits of attn_bwd_pre_k, so that a
// step does not depend on whether delta has a launch of its own
template <typename T, int DH> __device__ __forceinline__ float row_dot(const RowFrag<DH> &g, const RowFrag<DH> &x, int lane) {
    static_assert(DH == 32, "the order of the sum");
    float p[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        auto four = [&](float sum) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sum = fmaf(g.f[4 * c + i], x.f[4 * c + i], sum);
            return sum;
        };
        const float first = four(0.f);
        // 16 bytes of the row, one chain of that kernel, are four elements, or eight: this half's behind the other half's
        p[c] = sizeof(T) == 4 ? sum_halves(first) : __shfl(four(__shfl(first, lane & 31, 64)), lane | 32, 64);
    }
    return (p[0] + p[1]) + (p[2] + p[3]);
}

// dQ: own query rows, keys and values stream
template <template <typename> class R, typename T, int DH, int NW, bool OWN_DELTA>
__device__ __forceinline__ void dq_rows(const BwdArgs<T> &a, unsigned block, float *part) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t H = a.H, d = H * DH, ld = 3 * d, Tn = a.Tn;
    int64_t bh;
    int q0;
    if (!place(a.heads, a.Tn, true, block, bh, q0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q = q0 + l32, qc = min(q, a.Tn - 1);
    const T *base = a.qkv + b * Tn * ld + h * DH;
    RowFrag<DH> qf, gf;
    qf.load(R<T>(base, ld, q0, a.Tn, DH), lane);
    gf.load(R<T>(a.dO + b * Tn * d + h * DH, d, q0, a.Tn, DH), lane);
    const float li = a.lse[bh * Tn + qc];
    float di;
    if constexpr (OWN_DELTA) {
        RowFrag<DH> of;
        of.load(R<T>(a.O + b * Tn * d + h * DH, d, q0, a.Tn, DH), lane);
        di = row_dot<T>(gf, of, lane);
        if (wave == 0 && lhi == 0 && q < a.Tn) a.delta[bh * Tn + q] = di;
    } else {
        di = a.delta[bh * Tn + qc];
    }
    floatx16 dq[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) dq[i] = zero16();
    const int ntiles = q0 / ROWS + 1;
    for (int t = wave; t < ntiles; t += NW) {
        const int j0 = t * ROWS;
        const R<T> k(base + d, ld, j0, a.Tn, DH), v(base + 2 * d, ld, j0, a.Tn, DH);
        RowFrag<DH> kf, vf;
        ColFrag<DH> kc;
        kf.load(k, lane);
        vf.load(v, lane);
        kc.load(k, lane);
        floatx16 s = dot_rows(kf, qf);
        const floatx16 dp = dot_rows(vf, gf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = j0 + acc_row(r, lhi) <= q ? expf(s[r] * a.scale - li) : 0.f;
            s[r] = p * (dp[r] - di);                          // the 1/sqrt(dh) factor is applied once, to the sums
        }
        kc.add_to(dq, s);
    }
    float one[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) one[w] = 1.f;
    merge_store<T, DH, NW>(dq, part, wave, lane, one, a.scale, q < a.Tn ? a.dqkv + (b * Tn + q) * ld + h * DH : nullptr);
}

// dK, dV: own key rows, queries and output gradients stream
template <template <typename> class R, typename T, int DH, int NW, bool OWN_DELTA>
__device__ __forceinline__ void dkv_rows(const BwdArgs<T> &a, unsigned block, float *part) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t H = a.H, d = H * DH, ld = 3 * d, Tn = a.Tn;
    int64_t bh;
    int kv0;
    if (!place(a.heads, a.Tn, false, block, bh, kv0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int kv = kv0 + l32;
    const T *base = a.qkv + b * Tn * ld + h * DH, *gbase = a.dO + b * Tn * d + h * DH;
    const float *ls = a.lse + bh * Tn, *dl = a.delta + bh * Tn;
    RowFrag<DH> kf, vf;
    kf.load(R<T>(base + d, ld, kv0, a.Tn, DH), lane);
    vf.load(R<T>(base + 2 * d, ld, kv0, a.Tn, DH), lane);
    floatx16 dk[DH / 32], dv[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) { dk[i] = zero16(); dv[i] = zero16(); }
    for (int i0 = kv0 + wave * ROWS; i0 < a.Tn; i0 += NW * ROWS) {
        const R<T> qr(base, ld, i0, a.Tn, DH), gr(gbase, d, i0, a.Tn, DH);
        const int row = min(i0 + l32, a.Tn - 1);
        RowFrag<DH> qf, gf;
        ColFrag<DH> qc, gc;
        qf.load(qr, lane);
        gf.load(gr, lane);
        // log-sum-exp and delta of row l32 of the tile: handed to the lanes that need them through the LDS crossbar, in place of 32
        // loads of one value each (8 x 512 tokens, 8 heads of 64, this and the shared launch: 175 -> 151 us)
        const float lse_row = ls[row];
        float delta_row;
        if constexpr (OWN_DELTA) {
            RowFrag<DH> of;
            of.load(R<T>(a.O + b * Tn * d + h * DH, d, i0, a.Tn, DH), lane);
            delta_row = row_dot<T>(gf, of, lane);
        } else {
            delta_row = dl[row];
        }
        gc.load(gr, lane);
        qc.load(qr, lane);
        floatx16 s = dot_rows(qf, kf), dp = dot_rows(gf, vf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = i0 + acc_row(r, lhi);
            const float li = __shfl(lse_row, acc_row(r, lhi), 64), di = __shfl(delta_row, acc_row(r, lhi), 64);
            const float p = (q >= kv && q < a.Tn) ? expf(s[r] * a.scale - li) : 0.f;
            dp[r] = p * (dp[r] - di);
            s[r] = p;
        }
        gc.add_to(dv, s);
        qc.add_to(dk, dp);
    }
    float one[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) one[w] = 1.f;
    T *krow = kv < a.Tn ? a.dqkv + (b * Tn + kv) * ld + d + h * DH : nullptr;
    merge_store<T, DH, NW>(dk, part, wave, lane, one, a.scale, krow);
    merge_store<T, DH, NW>(dv, part, wave, lane, one, 1.0f, krow ? krow + d : nullptr);
}

// The blocks of key rows come first, they are the longer ones; then the blocks of query rows.  One launch for both: the sequences that
// this path is for fill neither the chip with one of them, nor the time of a launch.  Two wavefronts per SIMD at head size 64 (235
// registers; left to itself the compiler takes 288 and there is one), three at 32; one with 64-bit addresses.
template <bool WIDE, int DH, int NW> constexpr int waves_per_simd() { return DH == 128 || WIDE ? 1 : DH == 64 || NW == 8 ? 2 : 3; }
template <template <typename> class R, typename T, int DH, int NW, bool OWN_DELTA>
__global__ void __launch_bounds__(NW * 64, (waves_per_simd<R<T>::WIDE, DH, NW>())) attn_bwd_k(const BwdArgs<T> a, unsigned blocks, unsigned first) {
    __shared__ float part[merge_floats<NW>()];
    const unsigned block = first + blockIdx.x;
    if (block < blocks) dkv_rows<R, T, DH, NW, OWN_DELTA>(a, block, part);
    else dq_rows<R, T, DH, NW, OWN_DELTA>(a, block - blocks, part);
}

unsigned grid_for(int64_t heads, int64_t Tn) { return (unsigned)((Tn + ROWS - 1) / ROWS * ((heads + 7) / 8) * 8); }

// Eight wavefronts share a block's rows where that shortens the longest chain of tiles and the chip has room for them: at head size 32,
// from five tiles on, up to two workgroups per compute unit.  fp32, whole backward pass, four / eight wavefronts, us: 1 x 512 tokens,
// 3 heads of 32 19.1 / 16.5; 4 x 333, 4 heads 18.8 / 16.7; 8 x 512, 12 heads 88 / 128; 2 x 64, 4 heads 6.0 / 6.9; heads of 64: 2 x
// 200, 8 heads 18.5 / 18.2, 8 x 512, 8 heads 121 / 161.  The forward kernel gains less (4 x 333: 8.9 / 8.3; 1 x 512: 10.5 / 9.8).
bool eight_wavefronts(int64_t blocks, int64_t Tn, int64_t dh) { return dh == 32 && Tn > 4 * ROWS && blocks <= 512; }

template <int DH> constexpr bool own_delta() { return DH == 32; }    // at 64 it does not fit the registers, and delta has a launch of its own
// whether 32 rows of q, k and v are too wide for Rows
bool wide(int dtype, int64_t H, int64_t dh) { return ROWS * 3 * H * dh * (dtype == TIO_PREC_BF16 ? 2 : 4) >= ((int64_t)1 << 32); }
template <template <typename> class R, typename T, int DH, int NW, bool OWN_DELTA> void launch_both(hipStream_t s, const BwdArgs<T> &a, unsigned blocks) {
    if ((uint64_t)2 * blocks * NW * 64 < ((uint64_t)1 << 32)) {
        attn_bwd_k<R, T, DH, NW, OWN_DELTA><<<2 * blocks, NW * 64, 0, s>>>(a, blocks, 0);
    } else {                     // a grid has fewer than 2^32 threads
        attn_bwd_k<R, T, DH, NW, OWN_DELTA><<<blocks, NW * 64, 0, s>>>(a, blocks, 0);
        attn_bwd_k<R, T, DH, NW, OWN_DELTA><<<blocks, NW * 64, 0, s>>>(a, blocks, blocks);
    }
}
template <typename T, int DH> void launch_bwd(hipStream_t s, const BwdArgs<T> &a, bool wide) {
    const unsigned blocks = grid_for(a.heads, a.Tn);
    if (wide) {
        launch_both<WideRows, T, DH, 4, false>(s, a, blocks);
    } else if constexpr (own_delta<DH>()) {
        const bool eight = eight_wavefronts(2 * (int64_t)blocks, a.Tn, DH);
        if (a.O && eight) launch_both<Rows, T, DH, 8, true>(s, a, blocks);
        else if (a.O) launch_both<Rows, T, DH, 4, true>(s, a, blocks);
        else if (eight) launch_both<Rows, T, DH, 8, false>(s, a, blocks);
        else launch_both<Rows, T, DH, 4, false>(s, a, blocks);
    } else {
        launch_both<Rows, T, DH, 4, false>(s, a, blocks);
    }
}

}  // namespace

#define TIO_ATTN_DISPATCH(dtype, dh, ...)                                                         \
    do {                                                                                          \
        if ((dtype) == TIO_PREC_BF16) {                                                           \
            using T = bf16_t;                                                                     \
            if ((dh) == 32) { constexpr int DH = 32; __VA_ARGS__; }                               \
            else if ((dh) == 64) { constexpr int DH = 64; __VA_ARGS__; }                          \
            else { constexpr int DH = 128; __VA_ARGS__; }                                         \
        } else {                                                                                  \
            using T = float;                                                                      \
            if ((dh) == 32) { constexpr int DH = 32; __VA_ARGS__; }                               \
            else if ((dh) == 64) { constexpr int DH = 64; __VA_ARGS__; }                          \
            else { constexpr int DH = 128; __VA_ARGS__; }                                         \
        }                                                                                         \
    } while (0)

void attn_fwd(hipStream_t s, int dtype, const void *qkv, void *o, float *lse, int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    if (attn_mfma_supported(dtype, Tn, H, dh)) { attn_fwd_mfma(s, qkv, o, lse, B, Tn, H, dh); return; }
    const float scale = 1.0f / sqrtf((float)dh);
    TIO_ATTN_DISPATCH(dtype, dh, {
        const unsigned grid = grid_for(B * H, Tn);
        constexpr int MANY = DH == 32 ? 8 : 4;
        if (wide(dtype, H, dh)) attn_fwd_k<WideRows, T, DH, 4><<<grid, 256, 0, s>>>((const T *)qkv, (T *)o, lse, B * H, (int)Tn, H, scale);
        else if (eight_wavefronts(grid, Tn, DH)) attn_fwd_k<Rows, T, DH, MANY><<<grid, MANY * 64, 0, s>>>((const T *)qkv, (T *)o, lse, B * H, (int)Tn, H, scale);
        else attn_fwd_k<Rows, T, DH, 4><<<grid, 256, 0, s>>>((const T *)qkv, (T *)o, lse, B * H, (int)Tn, H, scale);
    });
}

void attn_bwd_pre(hipStream_t s, int dtype, const void *dO, const void *O, float *delta, int64_t B, int64_t Tn, int64_t H,
                  int64_t dh) {
    const int64_t n = B * Tn * H * (dh / (dtype == TIO_PREC_BF16 ? 8 : 4));
    if (dtype == TIO_PREC_BF16)
        attn_bwd_pre_k<bf16_t><<<(unsigned)((n + TPB - 1) / TPB), TPB, 0, s>>>((const bf16_t *)dO, (const bf16_t *)O, delta, B, Tn, H, dh);
    else
        attn_bwd_pre_k<float><<<(unsigned)((n + TPB - 1) / TPB), TPB, 0, s>>>((const float *)dO, (const float *)O, delta, B, Tn, H, dh);
}

bool attn_bwd_has_delta(int dtype, int64_t Tn, int64_t H, int64_t dh) {
    return (dh == 32 && !wide(dtype, H, dh)) || attn_mfma_supported(dtype, Tn, H, dh);
}

void attn_bwd(hipStream_t s, int dtype, const void *dO, const void *qkv, const void *O, const float *lse, float *delta, void *dqkv,
              int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    if (O && !attn_bwd_has_delta(dtype, Tn, H, dh)) attn_bwd_pre(s, dtype, dO, O, delta, B, Tn, H, dh);
    if (attn_mfma_supported(dtype, Tn, H, dh)) { attn_bwd_mfma(s, dO, qkv, O, lse, delta, dqkv, B, Tn, H, dh); return; }
    const float scale = 1.0f / sqrtf((float)dh);
    TIO_ATTN_DISPATCH(dtype, dh, {
        const BwdArgs<T> a{(const T *)dO, (const T *)qkv, (const T *)O, lse, delta, (T *)dqkv, B * H, H, (int)Tn, scale};
        launch_bwd<T, DH>(s, a, wide(dtype, H, dh));
    });
}

}  // namespace k
}  // namespace tio
