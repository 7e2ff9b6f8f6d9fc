// Dense contractions of the training step: C[M,N] = A . B^T (+bias) (+residual).
//
// bf16: the MFMA kernel of kernels_gemm_dl.hip (operand tiles loaded straight into LDS) does the work; this file holds the
// dispatch, the split-K reduction and a plain MFMA kernel with 64-bit addressing that takes over when an operand is
// too large for the first one's 32-bit buffer offsets.  In the plain kernel a workgroup owns a
// BM x BN tile of C; both operand tiles are staged through LDS in [row][k] order with a 16-byte row
// pad, so that every MFMA operand is one 16-byte LDS read.  Operands that are stored with the
// contraction index as the slow dimension ("k-major": the weight in dX = dY.W, both operands in
// dW = dY^T.X) are transposed in registers in 8x8 blocks on their way into LDS, so no transposed
// copy of any tensor ever exists in HBM.  The accumulator layout is chosen so that each lane owns
// 4 consecutive columns of a row of C: the epilogue (bias, residual, rounding to bf16) writes 8 bytes
// per store.
//
// fp32: kernels_gemm_f32.hip.
#include <stdexcept>

#include <mutex>

#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

template <int BM, int BN, int BK, int WGM, int WGN, int NBUF, bool AKM, bool BKM>
__global__ void __launch_bounds__(WGM *WGN * 64)
    gemm_bf16_k(const uint16_t *__restrict__ A, int64_t lda, const uint16_t *__restrict__ B, int64_t ldb,
                const uint16_t *__restrict__ bias, const uint16_t *__restrict__ resid, int64_t ldr,
                uint16_t *__restrict__ C, int64_t ldc, int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n,
                uint16_t *__restrict__ rowsum, float *__restrict__ ws, int64_t k_chunk, int rowsum_acc) {
    constexpr int NT = WGM * WGN * 64;
    constexpr int TPR = NT / BM;           // threads that share one row of the A tile for the row sums
    static_assert(NT % BM == 0 && (TPR & (TPR - 1)) == 0 && TPR <= 64 && BK % (8 * TPR) == 0, "row-sum mapping");
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int LS = BK + LDS_PAD;
    // NBUF operand tile pairs in LDS: with two, the stores of tile k+1 overlap the MFMAs of tile k and
    // one barrier per tile suffices
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    constexpr int TILE = (BM + BN) * LS;
    uint16_t *As = smem, *Bs = smem + BM * LS;

    // Tile order.  Workgroups are dealt to the 8 XCDs round-robin and every XCD has its own L2, so the
    // launch index is first turned into (xcd, index within the xcd) and each XCD gets one contiguous
    // eighth of the tile sequence; within the sequence groups of 8 tile rows walk the columns together.
    // The workgroups that share an L2 then work on neighbouring tiles: the 8 A tiles of the group stay in
    // that L2 and every B tile is fetched into it once per group, instead of once per XCD per group.
    const int tid = threadIdx.x;
    const int total_tiles = tiles_m * tiles_n;
    const int xcd_chunk = (total_tiles + 7) / 8;
    const int bid = (int)(blockIdx.x % 8) * xcd_chunk + (int)(blockIdx.x / 8);
    if (bid >= total_tiles) return;          // padding workgroups of the last chunk (whole workgroup, before any barrier)
    constexpr int GROUP = 8;
    const int per_group = GROUP * tiles_n;
    const int g = bid / per_group;
    const int gm0 = g * GROUP;
    const int gsz = tiles_m - gm0 < GROUP ? tiles_m - gm0 : GROUP;
    const int tm = gm0 + (bid % per_group) % gsz;
    const int tn = (bid % per_group) / gsz;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int l32 = lane & 31, lhi = lane >> 5;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    Stage<BM, BK, NT, AKM> sa;
    Stage<BN, BK, NT, BKM> sb;
    // split-K: workgroup row blockIdx.y owns the contraction range [kbeg, kend) and writes an fp32
    // partial tile to the workspace; a second launch adds the partials in split order
    const int64_t kbeg = (int64_t)blockIdx.y * k_chunk;
    const int64_t kend = (ws != nullptr && kbeg + k_chunk < K) ? kbeg + k_chunk : K;
    const int nk = (int)((kend - kbeg + BK - 1) / BK);
    sa.load(A, lda, m0, M, kbeg, kend, tid);
    sb.load(B, ldb, n0, N, kbeg, kend, tid);
    sa.store(As, tid);
    sb.store(Bs, tid);
    __syncthreads();
    // optional fused row sums of A over the whole contraction (the bias gradient when A = dY^T):
    // done by the workgroups of the first tile column, TPR threads per row, in k order
    const bool do_rowsum = rowsum != nullptr && tn == 0;
    float rsum = 0.f;
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) {
            sa.load(A, lda, m0, M, kbeg + (int64_t)(kt + 1) * BK, kend, tid);
            sb.load(B, ldb, n0, N, kbeg + (int64_t)(kt + 1) * BK, kend, tid);
        }
        if (NBUF == 2) { As = smem + (kt & 1) * TILE; Bs = As + BM * LS; }
        if (do_rowsum) {
            const uint16_t *row = As + (tid / TPR) * LS + (tid % TPR) * (BK / TPR);
#pragma unroll
            for (int c = 0; c < BK / TPR; c += 8) {
                const uint4 v = *reinterpret_cast<const uint4 *>(row + c);
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) rsum += __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            Frag fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i].u = *reinterpret_cast<const uint4 *>(As + (wm * WM + i * 32 + l32) * LS + ks * 16 + lhi * 8);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[j].u = *reinterpret_cast<const uint4 *>(Bs + (wn * WN + j * 32 + l32) * LS + ks * 16 + lhi * 8);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    // first operand indexes the accumulator's register dimension (n), second its lane dimension (m)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j].v, fa[i].v, acc[i][j], 0, 0, 0);
        }
        if (NBUF == 2) {
            if (kt + 1 < nk) {
                sa.store(smem + ((kt + 1) & 1) * TILE, tid);
                sb.store(smem + ((kt + 1) & 1) * TILE + BM * LS, tid);
            }
            __syncthreads();
        } else {
            __syncthreads();
            if (kt + 1 < nk) {
                sa.store(As, tid);
                sb.store(Bs, tid);
                __syncthreads();
            }
        }
    }

    if (do_rowsum) {
#pragma unroll
        for (int o = 1; o < TPR; o <<= 1) rsum += __shfl_xor(rsum, o, 64);
        const int64_t m = m0 + tid / TPR;
        if (tid % TPR == 0 && m < M) {
            if (ws) ws[(int64_t)gridDim.y * M * N + (int64_t)blockIdx.y * M + m] = rsum;
            else rowsum[m] = (uint16_t)f32_to_bf16_bits(rsum + (rowsum_acc ? bf16_bits_to_f32(rowsum[m]) : 0.f));
        }
    }
    // epilogue: lane holds C[m][n .. n+3] for 4 groups of columns per 32x32 tile
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int64_t m = m0 + wm * WM + i * 32 + l32;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t n = n0 + wn * WN + j * 32 + q * 8 + lhi * 4;
                if (n >= N) continue;
                float v[4] = {acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
                if (ws) {          // N is a multiple of 4 in split mode
                    *reinterpret_cast<float4 *>(ws + ((int64_t)blockIdx.y * M + m) * N + n) = make_float4(v[0], v[1], v[2], v[3]);
                    continue;
                }
                if (n + 4 <= N) {
                    if (bias) {
                        const uint2 t = *reinterpret_cast<const uint2 *>(bias + n);
                        v[0] += __uint_as_float(t.x << 16); v[1] += __uint_as_float(t.x & 0xffff0000u);
                        v[2] += __uint_as_float(t.y << 16); v[3] += __uint_as_float(t.y & 0xffff0000u);
                    }
                    if (resid) {
                        const uint2 t = *reinterpret_cast<const uint2 *>(resid + m * ldr + n);
                        v[0] += __uint_as_float(t.x << 16); v[1] += __uint_as_float(t.x & 0xffff0000u);
                        v[2] += __uint_as_float(t.y << 16); v[3] += __uint_as_float(t.y & 0xffff0000u);
                    }
                    uint2 o;
                    o.x = pack_bf16x2(v[0], v[1]);
                    o.y = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<uint2 *>(C + m * ldc + n) = o;
                } else {
                    for (int e = 0; e < 4 && n + e < N; ++e) {
                        float x = v[e];
                        if (bias) x += bf16_bits_to_f32(bias[n + e]);
                        if (resid) x += bf16_bits_to_f32(resid[m * ldr + n + e]);
                        C[m * ldc + n + e] = (uint16_t)f32_to_bf16_bits(x);
                    }
                }
            }
        }
    }
}

// Adds the split-K partials in split order, then bias and residual, and rounds once; also finishes the fused row sums.  A thread has four
// columns of a row (the last ones of a row: up to four), and the partials of eight ranges on their way at a time.
__global__ void __launch_bounds__(256) splitk_reduce_k(const float *__restrict__ ws, const uint16_t *__restrict__ bias, const uint16_t *resid,
                                                       int64_t ldr, uint16_t *C, int64_t ldc, uint16_t *__restrict__ rowsum, int64_t M, int64_t N,
                                                       int splits, int accumulate) {
    constexpr int AHEAD = 8;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t ld = partial_ld(N), nq = ld / 4, total = M * nq;
    if (idx < total) {
        const int64_t m = idx / nq, n = (idx % nq) * 4;
        const float *at = ws + m * ld + n;
        const int cols = N - n < 4 ? (int)(N - n) : 4;
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        for (int sp = 0; sp < splits; sp += AHEAD) {
            float4 part[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
                if (sp + i < splits) part[i] = *reinterpret_cast<const float4 *>(at + (int64_t)(sp + i) * M * ld);
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
                if (sp + i < splits) { a[0] += part[i].x; a[1] += part[i].y; a[2] += part[i].z; a[3] += part[i].w; }
        }
        uint16_t *c = C + m * ldc + n;
        const uint16_t *extra[2] = {bias ? bias + n : nullptr, accumulate ? c : resid ? resid + m * ldr + n : nullptr};   // accumulate: earlier micro-batches' sum is in C
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (!extra[k]) continue;
            if (cols == 4) {
                const uint2 t = *reinterpret_cast<const uint2 *>(extra[k]);
                a[0] += __uint_as_float(t.x << 16); a[1] += __uint_as_float(t.x & 0xffff0000u);
                a[2] += __uint_as_float(t.y << 16); a[3] += __uint_as_float(t.y & 0xffff0000u);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < cols) a[e] += bf16_bits_to_f32(extra[k][e]);
            }
        }
        if (cols == 4) {
            *reinterpret_cast<uint2 *>(c) = make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < cols) c[e] = (uint16_t)f32_to_bf16_bits(a[e]);
        }
    } else if (rowsum != nullptr && idx - total < M) {
        const int64_t m = idx - total;
        const float *r = ws + (int64_t)splits * M * ld;
        float a = r[m];
        for (int sp = 1; sp < splits; ++sp) a += r[(int64_t)sp * M + m];
        if (accumulate) a += bf16_bits_to_f32(rowsum[m]);
        rowsum[m] = (uint16_t)f32_to_bf16_bits(a);
    }
}
void splitk_reduce(hipStream_t s, const void *ws, const void *bias, const void *resid, int64_t ldr, void *C, int64_t ldc, void *rowsum, int64_t M,
                   int64_t N, int splits, bool accumulate) {
    const int64_t n = M * (partial_ld(N) / 4) + (rowsum ? M : 0);
    splitk_reduce_k<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const float *)ws, (const uint16_t *)bias, (const uint16_t *)resid, ldr, (uint16_t *)C,
                                                                 ldc, (uint16_t *)rowsum, M, N, splits, (int)accumulate);
}

// ---- scratch space of products that are split without a workspace from their caller
// A fixed array on every device, in SLOTS parts.  A product takes a part for its two launches: the stream first waits for the event
// that the part's last user recorded behind its own, and the lock is held from the choice of the part to the recording, so that two
// threads' launches on one stream do not mix.  A stream gets the part it had before, if it is still the last one there, so that
// up to SLOTS streams do not wait for each other; with more, a product waits until another stream has come as far as its last cut product
// (HIP's four hardware queues are shared by then anyway).  A product has one part, whatever its size: with four parts of 32 MiB, of
// which a large product took two or all, 200 x 304 x 15000 behind 20 of 4096 x 1024 x 32000 on another stream took 4150 us; now 209, and 38 with
// those in one range, where they take 365 us instead of 252.  72 MiB hold every cut that pays: of 24 contractions of 20000 to 50257 with
// 18 to 112 MiB of partials in two ranges, none that needs more than 64 is cut, or quicker with parts of 128 MiB.  The array costs 0.4 ms of
// host time per MiB once, when the first cut product loads it (52 ms with 128 MiB, 115 now).  No allocation, and no
// waiting on the host.  (An allocation from a stream-ordered pool for each product took 18 us of host time.)
constexpr int SLOTS = 4, DEVICES = 64;
constexpr int64_t SLOT_BYTES = (int64_t)72 << 20;
__device__ __align__(256) unsigned char split_partials[SLOTS * SLOT_BYTES];

struct Slot {
    hipEvent_t free = nullptr;
    hipStream_t user = nullptr;
    uint64_t used = 0;           // number of its last use; 0: never
};
struct SlotsOfDevice {
    unsigned char *base = nullptr;
    bool failed = false;
    uint64_t uses = 0;
    Slot slot[SLOTS];
};
std::mutex slots_mu;
SlotsOfDevice slots_of[DEVICES];

class SplitScratch {
    std::unique_lock<std::mutex> lock;
    hipStream_t s;
    SlotsOfDevice *owner = nullptr;
    Slot *mine = nullptr;
    unsigned char *at = nullptr;

public:
    // partials() is nullptr where there is no part to be had: a stream under capture (a replay would not wait for the part's other
    // users), one of another device than the current one (the array's address and the events are the current one's), or a device that
    // refuses the array or an event, or has refused to record one: nobody could wait for the part's user then
    explicit SplitScratch(hipStream_t stream) : s(stream) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &capture) != hipSuccess) { (void)hipGetLastError(); return; }
        int dev = -1;
        if (capture != hipStreamCaptureStatusNone || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= DEVICES) return;
        hipDevice_t of_stream = dev;
        if (s && hipStreamGetDevice(s, &of_stream) != hipSuccess) { (void)hipGetLastError(); return; }
        if (of_stream != dev) return;
        lock = std::unique_lock<std::mutex>(slots_mu);
        SlotsOfDevice &d = slots_of[dev];
        if (!d.base && !d.failed) prepare(d);
        if (d.failed) { lock.unlock(); return; }
        Slot *best = &d.slot[0];
        for (Slot &x : d.slot) {
            if (x.used && x.user == s) { best = &x; break; }
            if (x.used < best->used) best = &x;
        }
        if (best->used && hipStreamWaitEvent(s, best->free, 0) != hipSuccess) { (void)hipGetLastError(); lock.unlock(); return; }
        owner = &d;
        mine = best;
        mine->user = s;
        mine->used = ++d.uses;
        at = d.base + (mine - d.slot) * SLOT_BYTES;
    }
    ~SplitScratch() {
        if (mine && hipEventRecord(mine->free, s) != hipSuccess) owner->failed = true;      // the caller reports the error
    }
    float *partials() const { return reinterpret_cast<float *>(at); }

private:
    // once per device; another thread's capture in global mode must not see these calls as its own
    static void prepare(SlotsOfDevice &d) {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        void *p = nullptr;
        bool ok = hipGetSymbolAddress(&p, HIP_SYMBOL(split_partials)) == hipSuccess && p;
        for (Slot &x : d.slot) ok = ok && hipEventCreateWithFlags(&x.free, hipEventDisableTiming) == hipSuccess;
        if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (ok) d.base = (unsigned char *)p;
        else { (void)hipGetLastError(); d.failed = true; }
    }
};

}  // namespace

template <int BM, int BN, int BK, int WGM, int WGN, int NBUF>
static void launch_bf16(hipStream_t s, bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
                        const void *B, int64_t ldb, const void *bias, const void *resid, int64_t ldr, void *C, int64_t ldc,
                        void *rowsum, void *workspace, int splits, bool accumulate) {
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + BN - 1) / BN);
    float *ws = splits > 1 ? (float *)workspace : nullptr;
    const int64_t k_chunk = splits > 1 ? ((K + splits - 1) / splits + BK - 1) / BK * BK : K;
    const dim3 grid((unsigned)(8 * ((tiles_m * tiles_n + 7) / 8)), (unsigned)(splits > 1 ? splits : 1));
    const dim3 block(WGM * WGN * 64);
    constexpr size_t lds = (size_t)NBUF * (BM + BN) * (BK + LDS_PAD) * 2;
    static bool attr_done = false;           // tiles above 64 KiB of LDS need the limit raised once per kernel
    if (!attr_done) {
        (void)hipFuncSetAttribute((const void *)gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipFuncSetAttribute((const void *)gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipFuncSetAttribute((const void *)gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipFuncSetAttribute((const void *)gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_done = true;
    }
#define TIO_GEMM_ARGS (const uint16_t *)A, lda, (const uint16_t *)B, ldb, (const uint16_t *)bias, (const uint16_t *)resid, ldr, \
                      (uint16_t *)C, ldc, M, N, K, tiles_m, tiles_n, (uint16_t *)rowsum, ws, k_chunk, (int)accumulate
    if (!a_km && !b_km) gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, false, false><<<grid, block, lds, s>>>(TIO_GEMM_ARGS);
    else if (!a_km && b_km) gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, false, true><<<grid, block, lds, s>>>(TIO_GEMM_ARGS);
    else if (a_km && b_km) gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, true, true><<<grid, block, lds, s>>>(TIO_GEMM_ARGS);
    else gemm_bf16_k<BM, BN, BK, WGM, WGN, NBUF, true, false><<<grid, block, lds, s>>>(TIO_GEMM_ARGS);
#undef TIO_GEMM_ARGS
    if (ws) splitk_reduce(s, ws, nullptr, nullptr, 0, C, ldc, rowsum, M, N, splits, accumulate);
}

void gemm(hipStream_t s, int dtype, bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
          const void *B, int64_t ldb, const void *bias, const void *resid, int64_t ldr, void *C, int64_t ldc,
          void *rowsum, void *workspace, int splits, bool accumulate) {
    if (M <= 0 || N <= 0 || K <= 0) return;
    // split-K needs the fp32 workspace, no epilogue operands and whole float4 rows
    if (dtype != TIO_PREC_BF16 || !workspace || bias || resid || (N % 4) || splits < 2) splits = 1;
    // accumulate: C += A.B^T and rowsum += row sums (gradient accumulation over micro-batches).  In a single
    // pass the old C is the residual operand (every element is read and then written by the same lane); with
    // split-K, the caller's or the cut made here, the reduction launch adds it.
    if (accumulate && splits == 1) {
        if (resid) throw std::invalid_argument("gemm: accumulate cannot be combined with a residual operand");
        resid = C;
        ldr = ldc;
    }
    if (dtype == TIO_PREC_BF16 && splits == 1) {
        const int own = gemm_bf16_splits(a_km, b_km, M, N, K, lda, ldb, rowsum != nullptr, SLOT_BYTES);
        if (own > 1) {
            const SplitScratch scratch(s);
            float *const ws = scratch.partials();
            if (ws && gemm_bf16_direct(s, a_km, b_km, M, N, K, A, lda, B, ldb, nullptr, nullptr, 0, C, ldc, rowsum, ws, own, accumulate)) {
                splitk_reduce(s, ws, bias, resid, ldr, C, ldc, rowsum, M, N, own, accumulate);
                return;
            }
        }
    }
    if (dtype == TIO_PREC_BF16) {
        float *const wsp = splits > 1 ? (float *)workspace : nullptr;
        if (gemm_bf16_direct(s, a_km, b_km, M, N, K, A, lda, B, ldb, bias, resid, ldr, C, ldc, rowsum, wsp, splits, accumulate)) {
            if (splits > 1) splitk_reduce(s, workspace, nullptr, nullptr, 0, C, ldc, rowsum, M, N, splits, accumulate);
            return;
        }
        // operands too large for 32-bit buffer offsets: plain kernel with 64-bit addressing
        launch_bf16<128, 128, 64, 2, 2, 1>(s, a_km, b_km, M, N, K, A, lda, B, ldb, bias, resid, ldr, C, ldc, rowsum, workspace, splits, accumulate);
    } else {
        gemm_f32(s, a_km, b_km, F32Product{M, N, K, A, lda, B, ldb, bias, resid, ldr, C, ldc, rowsum, accumulate});
    }
}

void gemm_bf16_route(bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool rowsum, int *ranges, int64_t *rows,
                     int64_t *cols) {
    *ranges = gemm_bf16_splits(a_km, b_km, M, N, K, lda, ldb, rowsum, SLOT_BYTES);
    *rows = *cols = 0;
    if (*ranges == 1) gemm_bf16_first_launch(a_km, b_km, M, N, K, lda, ldb, rowsum, rows, cols);
}

}  // namespace k
}  // namespace tio
