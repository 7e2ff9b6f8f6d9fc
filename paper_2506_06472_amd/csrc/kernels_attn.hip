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
// fp32 workloads have.  So the four wavefronts of a workgroup share 32 own rows, take every fourth tile each and merge at the
// end, in wavefront order.  Giving every wavefront 32 rows of its own instead lost at every size, also where the rows fill the
// chip many times over (fp32, forward and backward, microseconds, shared / own rows: 4 x 333 x 4 x 32 43 / 117, 8 x 512 x 8 x 64
// 218 / 257, 4 x 2048 x 12 x 64 1580 / 2155): the shared form has four times the workgroups of a quarter the length, and the
// last rows of a causal mask end sooner.  With a row per lane on the vector ALU the first of these took 446.
// Statistics are fp32 (log-sum-exp saved for the backward pass, which recomputes the probabilities from it); every sum has a
// fixed order; dQ and dK/dV are separate launches, so that no atomics are needed.
#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

constexpr int TPB = 256;
constexpr int ROWS = 32;         // own rows of a wavefront, and rows of a tile of the other side

__device__ __forceinline__ void load4(float *f, const float *p) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
__device__ __forceinline__ void load4(float *f, const bf16_t *p) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
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
    template <typename T> __device__ __forceinline__ void load(const T *row, int lhi) {
#pragma unroll
        for (int c = 0; c < DH / 8; ++c) load4(f + 4 * c, row + 8 * c + 4 * lhi);
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
    template <typename T> __device__ __forceinline__ void load(const T *base, int64_t ld, int r0, int last, int lane) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = min(r0 + acc_row(r, lane >> 5), last);
#pragma unroll
            for (int i = 0; i < DH / 32; ++i) f[i][r] = to_f32(base[(int64_t)row * ld + 32 * i + (lane & 31)]);
        }
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
__device__ __forceinline__ bool place(int64_t heads, int Tn, bool long_last, int64_t &bh, int &r0) {
    const int nblk = (Tn + ROWS - 1) / ROWS;
    const int slot = (int)blockIdx.x >> 3;
    bh = (int64_t)(slot / nblk) * 8 + ((int)blockIdx.x & 7);
    const int blk = slot % nblk;
    r0 = (long_last ? nblk - 1 - blk : blk) * ROWS;           // longest rows first
    return bh < heads;
}
// Sums of the four wavefronts' accumulators in wavefront order, in wavefront 0; scale[w] is applied to wavefront w's.
template <int N> __device__ __forceinline__ void merge(floatx16 (&acc)[N], float *lds, int wave, int lane, const float (&scale)[TPB / 64]) {
    __syncthreads();
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) lds[((wave - 1) * N * 16 + i * 16 + r) * 64 + lane] = acc[i][r];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float x = acc[i][r] * scale[0];
#pragma unroll
                for (int w = 1; w < TPB / 64; ++w) x += lds[((w - 1) * N * 16 + i * 16 + r) * 64 + lane] * scale[w];
                acc[i][r] = x;
            }
    }
}
template <int DH> constexpr int merge_floats() { return (TPB / 64 - 1) * (DH / 32) * 16 * 64; }
// the row of the output this lane holds, four consecutive columns at a time
template <typename T, int DH> __device__ __forceinline__ void store_rows(T *row, const floatx16 (&acc)[DH / 32], float scale, int lhi) {
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float v[4] = {acc[i][4 * g] * scale, acc[i][4 * g + 1] * scale, acc[i][4 * g + 2] * scale, acc[i][4 * g + 3] * scale};
            store4(row + 32 * i + 8 * g + 4 * lhi, v);
        }
}

// ---------------------------------------------------------------- forward
template <typename T, int DH>
__global__ void __launch_bounds__(TPB) attn_fwd_k(const T *__restrict__ qkv, T *__restrict__ o, float *__restrict__ lse,
                                                  int64_t heads, int Tn, int64_t H, float scale) {
    __shared__ float part[merge_floats<DH>()];
    __shared__ float stat[2][TPB / 64][ROWS];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    int64_t bh;
    int q0;
    if (!place(heads, Tn, true, bh, q0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q = q0 + l32, last = Tn - 1;
    const T *base = qkv + b * Tn * ld + h * DH;
    RowFrag<DH> qf;
    qf.load(base + (int64_t)min(q, last) * ld, lhi);
    floatx16 acc[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) acc[i] = zero16();
    float m = -INFINITY, l = 0.f;
    const int ntiles = q0 / ROWS + 1;                         // every tile holds a key that each of the rows sees
    for (int t = wave; t < ntiles; t += TPB / 64) {
        const int j0 = t * ROWS;
        RowFrag<DH> kf;
        ColFrag<DH> vf;
        kf.load(base + d + (int64_t)min(j0 + l32, last) * ld, lhi);
        vf.load(base + 2 * d, ld, j0, last, lane);
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
    float f[TPB / 64], M = -INFINITY;
#pragma unroll
    for (int w = 0; w < TPB / 64; ++w) M = fmaxf(M, stat[0][w][l32]);
    l = 0.f;
#pragma unroll
    for (int w = 0; w < TPB / 64; ++w) {                 // a wavefront without a tile has maximum -inf and sum 0
        f[w] = expf(stat[0][w][l32] - (M == -INFINITY ? 0.f : M));
        l += stat[1][w][l32] * f[w];
    }
    m = M;
    merge<DH / 32>(acc, part, wave, lane, f);
    if (wave > 0) return;
    if (q < Tn) {
        store_rows<T, DH>(o + (b * Tn + q) * d + h * DH, acc, 1.0f / l, lhi);
        if (lhi == 0) lse[bh * Tn + q] = m + logf(l);
    }
}

// ---------------------------------------------------------------- backward
// delta[b,h,t] = sum_e dO[s,h,e] * O[s,h,e].  dh / (elements per 16 bytes) consecutive lanes share one (s, h):
// the wavefront reads consecutive 16-byte chunks, and the partial sums meet in a fixed xor-shuffle order.
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

// dQ: own query rows, keys and values stream
template <typename T, int DH>
__global__ void __launch_bounds__(TPB) attn_bwd_dq_k(const T *__restrict__ dO, const T *__restrict__ qkv,
                                                     const float *__restrict__ lse, const float *__restrict__ delta,
                                                     T *__restrict__ dqkv, int64_t heads, int Tn, int64_t H, float scale) {
    __shared__ float part[merge_floats<DH>()];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    int64_t bh;
    int q0;
    if (!place(heads, Tn, true, bh, q0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q = q0 + l32, last = Tn - 1, qc = min(q, last);
    const T *base = qkv + b * Tn * ld + h * DH;
    RowFrag<DH> qf, gf;
    qf.load(base + (int64_t)qc * ld, lhi);
    gf.load(dO + (b * Tn + qc) * d + h * DH, lhi);
    const float li = lse[bh * Tn + qc], di = delta[bh * Tn + qc];
    floatx16 dq[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) dq[i] = zero16();
    const int ntiles = q0 / ROWS + 1;
    for (int t = wave; t < ntiles; t += TPB / 64) {
        const int j0 = t * ROWS;
        const T *krow = base + d + (int64_t)min(j0 + l32, last) * ld;
        RowFrag<DH> kf, vf;
        ColFrag<DH> kc;
        kf.load(krow, lhi);
        vf.load(krow + d, lhi);
        kc.load(base + d, ld, j0, last, lane);
        floatx16 s = dot_rows(kf, qf);
        const floatx16 dp = dot_rows(vf, gf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = j0 + acc_row(r, lhi) <= q ? expf(s[r] * scale - li) : 0.f;
            s[r] = p * (dp[r] - di);                          // the 1/sqrt(dh) factor is applied once, to the sums
        }
        kc.add_to(dq, s);
    }
    const float one[TPB / 64] = {1.f, 1.f, 1.f, 1.f};
    merge<DH / 32>(dq, part, wave, lane, one);
    if (wave > 0) return;
    if (q < Tn) store_rows<T, DH>(dqkv + (b * Tn + q) * ld + h * DH, dq, scale, lhi);
}

// dK, dV: own key rows, queries and output gradients stream
template <typename T, int DH>
__global__ void __launch_bounds__(TPB) attn_bwd_dkv_k(const T *__restrict__ dO, const T *__restrict__ qkv,
                                                      const float *__restrict__ lse, const float *__restrict__ delta,
                                                      T *__restrict__ dqkv, int64_t heads, int Tn, int64_t H, float scale) {
    __shared__ float part[merge_floats<DH>()];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    int64_t bh;
    int kv0;
    if (!place(heads, Tn, false, bh, kv0)) return;
    const int64_t b = bh / H, h = bh % H;
    const int kv = kv0 + l32, last = Tn - 1;
    const T *base = qkv + b * Tn * ld + h * DH, *gbase = dO + b * Tn * d + h * DH;
    const float *ls = lse + bh * Tn, *dl = delta + bh * Tn;
    RowFrag<DH> kf, vf;
    kf.load(base + d + (int64_t)min(kv, last) * ld, lhi);
    vf.load(base + 2 * d + (int64_t)min(kv, last) * ld, lhi);
    floatx16 dk[DH / 32], dv[DH / 32];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i) { dk[i] = zero16(); dv[i] = zero16(); }
    for (int i0 = kv0 + wave * ROWS; i0 < Tn; i0 += TPB / 64 * ROWS) {
        RowFrag<DH> qf, gf;
        ColFrag<DH> qc, gc;
        const int row = min(i0 + l32, last);
        qf.load(base + (int64_t)row * ld, lhi);
        gf.load(gbase + (int64_t)row * d, lhi);
        gc.load(gbase, d, i0, last, lane);
        qc.load(base, ld, i0, last, lane);
        floatx16 s = dot_rows(qf, kf), dp = dot_rows(gf, vf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = i0 + acc_row(r, lhi), c = min(q, last);
            const float p = (q >= kv && q < Tn) ? expf(s[r] * scale - ls[c]) : 0.f;
            dp[r] = p * (dp[r] - dl[c]);
            s[r] = p;
        }
        gc.add_to(dv, s);
        qc.add_to(dk, dp);
    }
    const float one[TPB / 64] = {1.f, 1.f, 1.f, 1.f};
    merge<DH / 32>(dk, part, wave, lane, one);
    merge<DH / 32>(dv, part, wave, lane, one);
    if (wave > 0) return;
    if (kv < Tn) {
        T *krow = dqkv + (b * Tn + kv) * ld + d + h * DH;
        store_rows<T, DH>(krow, dk, scale, lhi);
        store_rows<T, DH>(krow + d, dv, 1.0f, lhi);
    }
}

unsigned grid_for(int64_t heads, int64_t Tn) { return (unsigned)((Tn + ROWS - 1) / ROWS * ((heads + 7) / 8) * 8); }

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
        attn_fwd_k<T, DH><<<grid_for(B * H, Tn), TPB, 0, s>>>((const T *)qkv, (T *)o, lse, B * H, (int)Tn, H, scale);
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

void attn_bwd(hipStream_t s, int dtype, const void *dO, const void *qkv, const float *lse, const float *delta, void *dqkv,
              int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    if (attn_mfma_supported(dtype, Tn, H, dh)) { attn_bwd_mfma(s, dO, qkv, lse, delta, dqkv, B, Tn, H, dh); return; }
    const float scale = 1.0f / sqrtf((float)dh);
    const unsigned grid = grid_for(B * H, Tn);
#define TIO_ATTN_ARGS (const T *)dO, (const T *)qkv, lse, delta, (T *)dqkv, B * H, (int)Tn, H, scale
    TIO_ATTN_DISPATCH(dtype, dh, {
        attn_bwd_dq_k<T, DH><<<grid, TPB, 0, s>>>(TIO_ATTN_ARGS);
        attn_bwd_dkv_k<T, DH><<<grid, TPB, 0, s>>>(TIO_ATTN_ARGS);
    });
#undef TIO_ATTN_ARGS
}

}  // namespace k
}  // namespace tio
