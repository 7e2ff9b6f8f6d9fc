// fp32 GEMM for gfx950 on the fp32 matrix instruction: C[M,N] = A . B^T (+bias) (+residual), for every combination of
// operand layouts, with the row sums of A from the same launch.
//
// v_mfma_f32_32x32x2_f32 multiplies and adds in fp32 like a chain of fused multiply-adds, at 256 flops per clock and
// compute unit: twice what scalar (not packed) vector instructions reach, from one register per operand instead of
// an LDS read per multiply-add.  Bound: the matrix cores (157 TFLOP/s) for products that fill the chip, launch and memory
// latency for the tiny ones.
//
//  * a contraction tile of BK elements goes global -> registers (two tiles ahead) -> one of two LDS stages; one barrier a tile;
//  * contraction index contiguous: LDS [row][BK + 4], read 16 bytes at a time (rows 4 banks apart modulo 64: no conflicts);
//    contraction index slow: LDS [k][rows + 8], read 4 bytes at a time (the two lane halves are 4 k-rows = 32 banks apart);
//  * a lane half takes k = 8c + 4 half + j in product j of chunk c, on both operands alike;
//  * small outputs have too few tiles to fill 256 compute units and too short a contraction to hide a memory latency, so
//    their tile is 32x32 and the four wavefronts of a workgroup split every contraction tile between them; the four
//    partial tiles are added in wavefront order.
// Measured figures stand at the choice of the tile, tile_of.
#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

template <int ROWS, int BK, int NT, bool KM> struct F32Operand {
    static constexpr int PITCH = KM ? ROWS + 8 : BK + 4;
    static constexpr int FLOATS = KM ? BK * PITCH : ROWS * PITCH;
    static constexpr int PER = ROWS * BK / 4 / NT;                // 16-byte chunks per thread and tile
    static constexpr int CPR = KM ? ROWS / 4 : BK / 4;            // chunks per LDS row
    static_assert(PER >= 1 && PER * NT * 4 == ROWS * BK, "chunks divide over the threads");
    const float *p[PER];
    int64_t step;                                                // floats from one contraction tile to the next
    int rows, part_rows;                                          // rows of the operand in this tile; some chunk holds both valid and other rows
    __device__ __forceinline__ void init(const float *base, int64_t ld, int rows_valid, int tid) {
        rows = rows_valid;
        part_rows = KM && rows_valid < ROWS && (rows_valid & 3);
        step = KM ? (int64_t)BK * ld : BK;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = i * NT + tid, o = c / CPR, q = c % CPR;
            // rows past the end read a valid row, or with KM the padding up to the leading dimension: what comes out of them is never stored
            if (KM) p[i] = base + (int64_t)o * ld + (q * 4 < rows_valid ? q * 4 : 0);
            else p[i] = base + (int64_t)(o < rows_valid ? o : rows_valid - 1) * ld + q * 4;
        }
    }
    __device__ __forceinline__ void load(float4 (&r)[PER], int kt) const {
#pragma unroll
        for (int i = 0; i < PER; ++i) r[i] = *reinterpret_cast<const float4 *>(p[i] + kt * step);
    }
    // the last tile of a contraction, where it is no multiple of BK or has partly valid chunks: whole chunks as such, a partly valid one
    // element by element, nothing at or past the end is read (all of them element by element: 128 x 2496 x 50 6.9 us, now 6.0; 128 x
    // 2496 x 16 6.1, now 5.8).  In the tiles before, what follows a partly valid chunk of a k-row is that row's padding (every tile this
    // way: 768 x 1307 x 717 with both operands k-major 33 us, now 22; 167 x 429 x 1920 23, now 15.4)
    __device__ void load_edge(float4 (&r)[PER], const float *base, int64_t ld, int kt, int kvalid, int tid) const {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = i * NT + tid, o = c / CPR, q = c % CPR;
            const float *at = base + kt * step + (int64_t)o * ld + q * 4;         // o: operand row, or k if KM; q * 4: the other one
            const int there = (o < (KM ? kvalid : rows)) ? (KM ? rows : kvalid) - q * 4 : 0;       // elements of the chunk that are there
            float v[4] = {0.f, 0.f, 0.f, 0.f};
            if (there >= 4) {
                r[i] = *reinterpret_cast<const float4 *>(at);
                continue;
            }
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < there) v[e] = at[e];
            r[i] = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
    static __device__ __forceinline__ void store(float *lds, const float4 (&r)[PER], int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = i * NT + tid;
            *reinterpret_cast<float4 *>(lds + (c / CPR) * PITCH + (c % CPR) * 4) = r[i];
        }
    }
    // the four values of chunk c for row `row`: k = 8c + 4 lhi + 0..3
    static __device__ __forceinline__ void frag(float (&f)[4], const float *lds, int row, int c, int lhi) {
        if (KM) {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = lds[(c * 8 + lhi * 4 + j) * PITCH + row];
        } else {
            const float4 v = *reinterpret_cast<const float4 *>(lds + row * PITCH + c * 8 + lhi * 4);
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        }
    }
    static __device__ __forceinline__ float at(const float *lds, int row, int k) { return KM ? lds[k * PITCH + row] : lds[row * PITCH + k]; }
};

// operands of one product
struct F32Args {
    const float *A, *B, *bias, *resid;
    float *C, *rowsum;
    int64_t lda, ldb, ldr, ldc, M, N, K;
    int tiles_m, tiles_n, rowsum_acc;
};

template <int BM, int BN, int BK, int WGM, int WGN, int KG, bool AKM, bool BKM> struct F32Tile {
    static constexpr int NT = WGM * WGN * KG * 64;
    using OpA = F32Operand<BM, BK, NT, AKM>;
    using OpB = F32Operand<BN, BK, NT, BKM>;
    static constexpr int STAGE = OpA::FLOATS + OpB::FLOATS, RED = (KG - 1) * BM * BN;
    static constexpr int FLOATS = 2 * STAGE > RED ? 2 * STAGE : RED;      // of LDS
    static unsigned blocks(int tiles_m, int tiles_n) { return 8 * (((unsigned)tiles_m * tiles_n + 7) / 8); }
    static __device__ __forceinline__ void run(const F32Args &a, unsigned block, float *smem);
};

template <int BM, int BN, int BK, int WGM, int WGN, int KG, bool AKM, bool BKM>
__device__ __forceinline__ void F32Tile<BM, BN, BK, WGM, WGN, KG, AKM, BKM>::run(const F32Args &a, unsigned block, float *smem) {
    const float *__restrict__ A = a.A, *__restrict__ B = a.B, *__restrict__ bias = a.bias, *resid = a.resid;
    float *C = a.C, *__restrict__ rowsum = a.rowsum;
    const int64_t lda = a.lda, ldb = a.ldb, ldr = a.ldr, ldc = a.ldc, M = a.M, N = a.N, K = a.K;
    const int tiles_m = a.tiles_m, tiles_n = a.tiles_n, rowsum_acc = a.rowsum_acc;
    constexpr int TPR = NT / BM;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int CH = BK / 8 / KG;                               // chunks of eight k per wavefront and tile
    static_assert(TPR <= 64 && (TPR & (TPR - 1)) == 0 && BK % TPR == 0 && CH >= 1, "row-sum mapping, chunks per wavefront");
    const int total = tiles_m * tiles_n;
    const int bid = (int)(block % 8) * ((total + 7) / 8) + (int)(block / 8);      // neighbouring tiles on one XCD
    if (bid >= total) return;
    const int tm = bid % tiles_m, tn = bid / tiles_m;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int kg = wave % KG, wt = wave / KG, wm = wt / WGN, wn = wt % WGN;

    const float *baseA = AKM ? A + m0 : A + m0 * lda, *baseB = BKM ? B + n0 : B + n0 * ldb;
    OpA oa;
    OpB ob;
    oa.init(baseA, lda, (int)(M - m0 < BM ? M - m0 : BM), tid);
    ob.init(baseB, ldb, (int)(N - n0 < BN ? N - n0 : BN), tid);
    const int nk = (int)((K + BK - 1) / BK), nkf = (int)(K / BK), rem = (int)(K - (int64_t)nkf * BK);
    const int fast = nk - nkf || !(oa.part_rows || ob.part_rows) ? nkf : nkf - 1;      // tiles without edges

    float4 ra[2][OpA::PER], rb[2][OpB::PER];
    auto load = [&](int set, int kt) {
        if (kt < fast) {
            oa.load(ra[set], kt);
            ob.load(rb[set], kt);
        } else {
            const int kv = kt < nkf ? BK : rem;
            oa.load_edge(ra[set], baseA, lda, kt, kv, tid);
            ob.load_edge(rb[set], baseB, ldb, kt, kv, tid);
        }
    };
    auto store = [&](int set) {
        OpA::store(smem + set * STAGE, ra[set], tid);
        OpB::store(smem + set * STAGE + OpA::FLOATS, rb[set], tid);
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const bool do_rowsum = rowsum != nullptr && tn == 0;
    float rsum = 0.f;

    load(0, 0);
    if (nk > 1) load(1, 1);
    store(0);
    __syncthreads();
    auto tile = [&](int set, int kt) {                // stage `set` holds tile kt, the other register set tile kt + 1
        if (kt + 2 < nk) load(set, kt + 2);
        const float *As = smem + set * STAGE, *Bs = As + OpA::FLOATS;
        if (do_rowsum) {
#pragma unroll 4
            for (int j = 0; j < BK / TPR; ++j) rsum += OpA::at(As, tid / TPR, (tid % TPR) * (BK / TPR) + j);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float fa[TM][4], fb[TN][4];
#pragma unroll
            for (int i = 0; i < TM; ++i) OpA::frag(fa[i], As, wm * WM + i * 32 + l32, kg * CH + c, lhi);
#pragma unroll
            for (int j = 0; j < TN; ++j) OpB::frag(fb[j], Bs, wn * WN + j * 32 + l32, kg * CH + c, lhi);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store(set ^ 1);
        __syncthreads();
    };
    for (int kt = 0; kt < nk; kt += 2) {
        tile(0, kt);
        if (kt + 1 < nk) tile(1, kt + 1);
    }

    if (do_rowsum) {
#pragma unroll
        for (int o = 1; o < TPR; o <<= 1) rsum += __shfl_xor(rsum, o, 64);
        const int64_t m = m0 + tid / TPR;
        if (tid % TPR == 0 && m < M) rowsum[m] = rsum + (rowsum_acc ? rowsum[m] : 0.f);
    }
    if (KG > 1) {                                     // the last barrier came after every read of the stages
        if (kg > 0) {
            float *dst = smem + ((kg - 1) * (WGM * WGN) + wt) * (WM * WN) + lane;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) dst[((i * TN + j) * 16 + r) * 64] = acc[i][j][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 1; g < KG; ++g) {
            const float *src = smem + ((g - 1) * (WGM * WGN) + wt) * (WM * WN) + lane;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] += src[((i * TN + j) * 16 + r) * 64];
        }
    }
    // lane l holds column l % 32: every store instruction writes two full 128-byte row pieces
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int64_t n = n0 + wn * WN + j * 32 + l32;
        if (n >= N) continue;
        const float bn = bias ? bias[n] : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = m0 + wm * WM + i * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
                if (m < M) C[m * ldc + n] = acc[i][j][r] + bn + (resid ? resid[m * ldr + n] : 0.f);
            }
    }
}

// 16x16 tiles on v_mfma_f32_16x16x4_f32 for outputs of a few thousand elements: four times the workgroups, and a quarter of the
// chain of dependent products per contraction element (8 clocks against 32).  Four wavefronts split every contraction tile; lane
// quarter q takes k = 16c + 4q + j in product j of chunk c.
template <bool AKM, bool BKM> struct F32Tiny {
    static constexpr int T = 16, BK = 128, NT = 256, KG = 4;
    using OpA = F32Operand<T, BK, NT, AKM>;
    using OpB = F32Operand<T, BK, NT, BKM>;
    static constexpr int STAGE = OpA::FLOATS + OpB::FLOATS, FLOATS = 2 * STAGE;
    static_assert(FLOATS >= (KG - 1) * 4 * 64, "the partial tiles fit the stages");
    static unsigned blocks(int tiles_m, int tiles_n) { return (unsigned)(tiles_m * tiles_n); }
    static __device__ __forceinline__ void run(const F32Args &a, unsigned block, float *smem);
};
template <bool AKM, bool BKM> __device__ __forceinline__ void F32Tiny<AKM, BKM>::run(const F32Args &a, unsigned block, float *smem) {
    const float *__restrict__ A = a.A, *__restrict__ B = a.B, *__restrict__ bias = a.bias, *resid = a.resid;
    float *C = a.C, *__restrict__ rowsum = a.rowsum;
    const int64_t lda = a.lda, ldb = a.ldb, ldr = a.ldr, ldc = a.ldc, M = a.M, N = a.N, K = a.K;
    const int tiles_m = a.tiles_m, rowsum_acc = a.rowsum_acc;
    constexpr int CH = BK / 16 / KG, TPR = NT / T;
    typedef float floatx4 __attribute__((ext_vector_type(4)));

    const int tm = (int)block % tiles_m, tn = (int)block / tiles_m;
    const int64_t m0 = (int64_t)tm * T, n0 = (int64_t)tn * T;
    const int tid = threadIdx.x, kg = tid >> 6, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const float *baseA = AKM ? A + m0 : A + m0 * lda, *baseB = BKM ? B + n0 : B + n0 * ldb;
    OpA oa;
    OpB ob;
    oa.init(baseA, lda, (int)(M - m0 < T ? M - m0 : T), tid);
    ob.init(baseB, ldb, (int)(N - n0 < T ? N - n0 : T), tid);
    const int nk = (int)((K + BK - 1) / BK), nkf = (int)(K / BK), rem = (int)(K - (int64_t)nkf * BK);
    const int fast = nk - nkf || !(oa.part_rows || ob.part_rows) ? nkf : nkf - 1;      // tiles without edges
    float4 ra[2][OpA::PER], rb[2][OpB::PER];
    auto load = [&](int set, int kt) {
        if (kt < fast) {
            oa.load(ra[set], kt);
            ob.load(rb[set], kt);
        } else {
            const int kv = kt < nkf ? BK : rem;
            oa.load_edge(ra[set], baseA, lda, kt, kv, tid);
            ob.load_edge(rb[set], baseB, ldb, kt, kv, tid);
        }
    };
    auto store = [&](int set) {
        OpA::store(smem + set * STAGE, ra[set], tid);
        OpB::store(smem + set * STAGE + OpA::FLOATS, rb[set], tid);
    };
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    const bool do_rowsum = rowsum != nullptr && tn == 0;
    float rsum = 0.f;
    load(0, 0);
    if (nk > 1) load(1, 1);
    store(0);
    __syncthreads();
    auto tile = [&](int set, int kt) {                // stage `set` holds tile kt, the other register set tile kt + 1
        if (kt + 2 < nk) load(set, kt + 2);
        const float *As = smem + set * STAGE, *Bs = As + OpA::FLOATS;
        if (do_rowsum) {
#pragma unroll
            for (int j = 0; j < BK / TPR; ++j) rsum += OpA::at(As, tid / TPR, (tid % TPR) * (BK / TPR) + j);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float fa[4], fb[4];
            OpA::frag(fa, As, l16, 2 * (kg * CH + c), lq);
            OpB::frag(fb, Bs, l16, 2 * (kg * CH + c), lq);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[e], acc, 0, 0, 0);
        }
        if (kt + 1 < nk) store(set ^ 1);
        __syncthreads();
    };
    for (int kt = 0; kt < nk; kt += 2) {
        tile(0, kt);
        if (kt + 1 < nk) tile(1, kt + 1);
    }
    if (do_rowsum) {
#pragma unroll
        for (int o = 1; o < TPR; o <<= 1) rsum += __shfl_xor(rsum, o, 64);
        const int64_t m = m0 + tid / TPR;
        if (tid % TPR == 0 && m < M) rowsum[m] = rsum + (rowsum_acc ? rowsum[m] : 0.f);
    }
    float *red = smem;                                // the last barrier came after every read of the stages
    if (kg > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((kg - 1) * 4 + r) * 64 + lane] = acc[r];
    }
    __syncthreads();
    if (kg > 0) return;
    const int64_t n = n0 + l16;
    if (n >= N) return;
    const float bn = bias ? bias[n] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + 4 * lq + r;
        float x = acc[r];
#pragma unroll
        for (int g = 0; g < KG - 1; ++g) x += red[(g * 4 + r) * 64 + lane];
        if (m < M) C[m * ldc + n] = x + bn + (resid ? resid[m * ldr + n] : 0.f);
    }
}

template <typename Tile> __global__ void __launch_bounds__(Tile::NT) gemm_f32_mfma_k(const F32Args a) {
    __shared__ __attribute__((aligned(16))) float smem[Tile::FLOATS];
    Tile::run(a, blockIdx.x, smem);
}
// two independent products in one launch
template <typename T0, typename T1> __global__ void __launch_bounds__(T0::NT) gemm_f32_pair_k(const F32Args a0, unsigned blocks0, const F32Args a1) {
    static_assert(T0::NT == T1::NT, "one workgroup size");
    __shared__ __attribute__((aligned(16))) float smem[T0::FLOATS > T1::FLOATS ? T0::FLOATS : T1::FLOATS];
    if (blockIdx.x < blocks0) T0::run(a0, blockIdx.x, smem);
    else T1::run(a1, blockIdx.x - blocks0, smem);
}

template <bool AKM, bool BKM> using Tile64 = F32Tile<64, 64, 32, 2, 2, 1, AKM, BKM>;
template <bool AKM, bool BKM> using Tile64x32 = F32Tile<64, 32, 32, 2, 1, 2, AKM, BKM>;
template <bool AKM, bool BKM> using Tile32 = F32Tile<32, 32, 64, 1, 1, 4, AKM, BKM>;

template <template <bool, bool> class Tile> void launch(hipStream_t s, bool a_km, bool b_km, const F32Args &a) {
#define TIO_F32(AKM, BKM) gemm_f32_mfma_k<Tile<AKM, BKM>><<<Tile<AKM, BKM>::blocks(a.tiles_m, a.tiles_n), Tile<AKM, BKM>::NT, 0, s>>>(a)
    if (!a_km && !b_km) TIO_F32(false, false);
    else if (!a_km && b_km) TIO_F32(false, true);
    else if (a_km && b_km) TIO_F32(true, true);
    else TIO_F32(true, false);
#undef TIO_F32
}

// The output tile.  A unit holds three or four workgroups at a time, and these products have few more for it, so that the time is taken
// as that of the compute unit with the most tiles: us per 64 x 64 x 768 of work (cost's last arguments: one tile on that unit, two, more),
// which fall with the number of tiles there are to cover each other's latencies.  us, 64x64 / 64x32 / 32x32, tiles on that unit in brackets:
//   1024 x 3072 x  768  47 ( 3) / 57 ( 6) /  63 (12)      1024 x  768 x 3072  75 ( 1) / 71 ( 2) /  53 ( 3)
//   3072 x  768 x 1024  58 ( 3) / 56 ( 5) /  62 ( 9)      2048 x  768 x 3072 114 ( 2) / 96 ( 3) / 113 ( 6)
//   1500 x  900 x 2000  79 ( 2) / 65 ( 3) /  73 ( 6)       512 x 1024 x 1024  28 ( 1) / 22 ( 1) /  17 ( 2)
//   1024 x 1024 x 1024  28 ( 1) / 27 ( 2) /  28 ( 4)       300 x 2000 x 2500  63 ( 1) / 62 ( 2) /  45 ( 3)
// 128x128 tiles leave one wavefront per SIMD where the others leave three, and lose everywhere (2048^3: 174, 160 with 64x64).
// 16x16 tiles up to 160 tiles of 32x32: 128 x 128 x 1024 (16 tiles) 12.5 -> 6.0 us, 256 x 512 x 512 (128) 8.5 -> 5.6,
// 300 x 500 x 1000 (160) 13.2 -> 11.5, but 64 x 3000 x 512 (188) 8.7 -> 10.2 with a k-major operand.
struct TileShape {
    int rows, cols;
};
constexpr TileShape T16{16, 16}, T32{32, 32}, T64x32{64, 32}, T64{64, 64};
TileShape tile_of(int64_t M, int64_t N) {
    auto tiles = [&](TileShape t) { return ((M + t.rows - 1) / t.rows) * ((N + t.cols - 1) / t.cols); };
    if (tiles(T32) <= 160) return T16;
    auto cost = [&](TileShape t, double one, double two, double more) {
        if (t.rows * t.cols < 4096 && tiles(t) > ((int64_t)1 << 24) - 8) return 1e300;     // a grid has fewer than 2^32 threads
        const int64_t n = (tiles(t) + 255) / 256;
        return (double)n * (t.rows * t.cols / 4096.0) * (n == 1 ? one : n == 2 ? two : more);
    };
    const double c64 = cost(T64, 18, 14.3, 14.3), c64x32 = cost(T64x32, 27.5, 17, 15.5), c32 = cost(T32, 33, 20.7, 18);
    return c64 <= c64x32 && c64 <= c32 ? T64 : c64x32 <= c32 ? T64x32 : T32;
}
bool small(TileShape t) { return t.rows <= 32; }
F32Args args_of(const F32Product &p, TileShape t) {
    return F32Args{(const float *)p.A, (const float *)p.B, (const float *)p.bias, (const float *)p.resid, (float *)p.C, (float *)p.rowsum,
                   p.lda, p.ldb, p.ldr, p.ldc, p.M, p.N, p.K, (int)((p.M + t.rows - 1) / t.rows), (int)((p.N + t.cols - 1) / t.cols),
                   (int)p.accumulate};
}

}  // namespace

void gemm_f32(hipStream_t s, bool a_km, bool b_km, const F32Product &p) {
    const TileShape tile = tile_of(p.M, p.N);
    const F32Args a = args_of(p, tile);
    if (tile.rows == 16) launch<F32Tiny>(s, a_km, b_km, a);
    else if (tile.rows == 32) launch<Tile32>(s, a_km, b_km, a);
    else if (tile.cols == 32) launch<Tile64x32>(s, a_km, b_km, a);
    else launch<Tile64>(s, a_km, b_km, a);
}

void gemm_f32_tile(int64_t M, int64_t N, int *rows, int *cols) {
    const TileShape t = tile_of(M, N);
    *rows = t.rows;
    *cols = t.cols;
}

// Both gradients of a linear layer in one launch, where the tiles of both are small (16 or 32 square): such products last
// about as long as a launch, and neither fills the chip (4.2 + 4.5 us in the tiny GPT step, nine times: that step, with merged updates
// and delta in the launch of attention backward as well, 344 -> 268 us).
bool gemm_f32_pairs(int64_t M0, int64_t N0, int64_t M1, int64_t N1) { return small(tile_of(M0, N0)) && small(tile_of(M1, N1)); }

void gemm_f32_pair(hipStream_t s, const F32Product &dx, const F32Product &dw) {
    const TileShape t0 = tile_of(dx.M, dx.N), t1 = tile_of(dw.M, dw.N);
    const F32Args a0 = args_of(dx, t0), a1 = args_of(dw, t1);
    using X16 = F32Tiny<false, true>;
    using X32 = Tile32<false, true>;
    using W16 = F32Tiny<true, true>;
    using W32 = Tile32<true, true>;
#define TIO_F32_PAIR(X, W)                                                                                          \
    {                                                                                                               \
        const unsigned n0 = X::blocks(a0.tiles_m, a0.tiles_n), n1 = W::blocks(a1.tiles_m, a1.tiles_n);              \
        gemm_f32_pair_k<X, W><<<n0 + n1, X::NT, 0, s>>>(a0, n0, a1);                                                \
    }
    if (t0.rows == 16 && t1.rows == 16) TIO_F32_PAIR(X16, W16)
    else if (t0.rows == 16) TIO_F32_PAIR(X16, W32)
    else if (t1.rows == 16) TIO_F32_PAIR(X32, W16)
    else TIO_F32_PAIR(X32, W32)
#undef TIO_F32_PAIR
}

}  // namespace k
}  // namespace tio
