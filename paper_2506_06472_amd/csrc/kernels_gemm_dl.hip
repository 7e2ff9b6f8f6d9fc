// bf16 MFMA GEMM for gfx950 whose operand tiles go from global memory straight into LDS
// (buffer loads with the LDS bit): C[M,N] = A . B^T (+bias) (+residual), fp32 accumulate.
//
//  * no staging registers and no LDS store instructions: a wavefront-wide load instruction fills 1 KiB of
//    consecutive LDS bytes (lane i writes bytes 16 i .. 16 i + 15); which 16-byte chunk of the operand a lane
//    fetches is chosen so that the LDS image is the bank-swizzled tile the fragment reads expect;
//  * an operand tile is ROWS x 64 bf16 = ROWS * 128 bytes without padding.
//      contraction index contiguous ("k-contig"): LDS row r holds the eight chunks of operand row r, chunk c at
//      slot c ^ ((r >> 1) & 7): the sixteen rows read together by a quarter wavefront fall into sixteen
//      different 16-byte bank groups;
//      contraction index slow ("k-major"): LDS row k holds ROWS elements, chunk c at slot c ^ swz(k): the eight
//      k-rows half a wavefront's transposing read touches fall into different 32-byte bank groups, and the 32 consecutive
//      bytes four lanes read stay consecutive;
//  * four wavefronts, one per SIMD, with a quarter of the output tile each (128x128 of 256x256): a third less LDS traffic
//    per flop than eight.  One wavefront per SIMD hides nothing by switching, so the order of every product, fragment read and
//    tile load is pinned: a tile of 64 is two contraction steps, fragments double-buffered in registers across steps and across
//    the one barrier a tile has;
//  * LDS holds D and a half contraction tiles (a ring per operand, 2.5 of 256x256), so that the loads are spread evenly over a tile
//    and are issued D - 1 to D - 0.5 tiles before they are waited for.
// Bound: the power limit on operands with many set bits (the clock follows it), the matrix cores otherwise.  Measured, 4096 x
// 4096 x 8192, contraction-contiguous operands, TFLOP/s on normal values / on zeros: eight wavefronts of 128x64 with 32x32x16
// products and two stages 1333 / 1775; four wavefronts with 16x16x32 products 1435 / 1795; with the loads spread over the tile
// 1492 / 2049 (without any loads 2146 on zeros: issued in a burst they fill the queue and stall the wavefront's products).
// Prefetching lines into the L2 four tiles ahead as well: 1406 / 1795, the extra traffic costs more clock than it saves.
#include <type_traits>

#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;                                          // contraction tile

// c += a . b with the accumulator held in an accumulation register, where it stays: left to itself the compiler moves
// accumulators between the two register files around almost every product of a kernel that uses most of both.  It does not
// know the instruction's hazards from here: settle() stands wherever an accumulator is written or read by something else.
__device__ __forceinline__ void mfma_acc(floatx4 &c, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// c += a . b0 or a . b1 as `which` says (uniform; anything but 0 and 1: nothing).  One block, so that c stays in one place: the
// compiler would move it from branch to branch without the wait a product's result needs.
__device__ __forceinline__ void mfma_pick(floatx4 &c, const bf16x8 &a, const bf16x8 &b0, const bf16x8 &b1, int which) {
    asm volatile("s_cmp_eq_u32 %4, 0\n\ts_cbranch_scc1 .Lpick0_%=\n\ts_cmp_eq_u32 %4, 1\n\ts_cbranch_scc0 .Lpick_end_%=\n\t"
                 "v_mfma_f32_16x16x32_bf16 %0, %1, %3, %0\n\ts_branch .Lpick_end_%=\n"
                 ".Lpick0_%=:\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n.Lpick_end_%=:"
                 : "+v"(c)
                 : "v"(a), "v"(b0), "v"(b1), "s"(which)
                 : "scc");
}
// The first with a tile load (see load_to_lds_b128) behind it: the product fills the wait state that M0 needs.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void mfma_acc_load(floatx4 &c, const bf16x8 &a, const bf16x8 &b, i32x4 rsrc, uint32_t lds_addr, uint32_t voff,
                                              uint32_t soff) {
    asm volatile("s_mov_b32 m0, %3\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tbuffer_load_dwordx4 %4, %5, %6 offen lds"
                 : "+a"(c)
                 : "v"(a), "v"(b), "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

template <int ROWS, int NT, bool KM> struct DlOperand;

// ---- contraction index contiguous
template <int ROWS, int NT> struct DlOperand<ROWS, NT, false> {
    static constexpr int BYTES = ROWS * BK * 2;
    static constexpr int BLOCKS = BYTES / 1024, NW = NT / 64, PER = BLOCKS / NW;     // 1 KiB blocks per wavefront
    static constexpr int READS = 1;                             // LDS read instructions per fragment
    static_assert(BLOCKS % NW == 0, "blocks divide over the wavefronts");
    uint32_t voff[PER];
    __device__ __forceinline__ void init(int64_t ld, int rows_valid, int kvalid, int wave, int lane) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int b = i * NW + wave, r = b * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            voff[i] = (r < rows_valid && c * 8 < kvalid) ? (uint32_t)(((int64_t)r * ld + c * 8) * 2) : DL_OOB;
        }
    }
    static __device__ __forceinline__ uint32_t tile_step(int64_t) { return BK * 2; }
    __device__ __forceinline__ void load_one(int i, i32x4 rsrc, uint32_t kb, uint32_t stage, int wave) const {
        load_to_lds_b128(rsrc, stage + (i * NW + wave) * 1024, voff[i], kb);
    }
    // fragment: lane l reads chunk 4 ks + l/16 of row row0 + sub*16 + l%16 (row0 a multiple of 16)
    uint32_t foff[BK / 32];
    __device__ __forceinline__ void init_frag(int row0, int lane) {
        const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
        for (int ks = 0; ks < BK / 32; ++ks) foff[ks] = (uint32_t)((row0 + l16) * 128 + (((ks * 4 + lq) ^ (l16 >> 1)) << 4));
    }
    __device__ __forceinline__ bf16x8 frag(const unsigned char *stage, int sub, int ks) const {
        Frag f;
        f.u = *reinterpret_cast<const uint4 *>(stage + foff[ks] + sub * 2048);
        return f.v;
    }
    __device__ __forceinline__ void second_step() { foff[0] = foff[1]; }
    // zeroes elements kvalid .. of a landed tile (kvalid not a multiple of eight: a load brings whole chunks)
    static __device__ __forceinline__ void clear_tail(unsigned char *stage, int kvalid, int tid) {
        for (int r = tid; r < ROWS; r += NT) {
            unsigned char *chunk = stage + r * 128 + (((kvalid >> 3) ^ ((r >> 1) & 7)) << 4);
            for (int e = kvalid & 7; e < 8; ++e) reinterpret_cast<uint16_t *>(chunk)[e] = 0;
        }
    }
};

// ---- contraction index slow: LDS row k = ROWS elements
template <int ROWS, int NT> struct DlOperand<ROWS, NT, true> {
    static constexpr int BYTES = ROWS * BK * 2;
    static constexpr int CPK = ROWS / 8;                        // chunks per k-row
    static constexpr int BLOCKS = BYTES / 1024, NW = NT / 64, PER = BLOCKS / NW;
    static constexpr int READS = 2;
    static_assert(BLOCKS % NW == 0 && ROWS % 64 == 0, "blocks divide over the wavefronts; rows of an even number of 128 bytes");
    // what the chunk index of k-row k is XORed with: k-rows 0..3 and 8..11 are read together, 32 bytes of each, and have to
    // fall into eight different 32-byte bank groups; where a row is an odd number of 128 bytes odd rows are 128 bytes off already
    static __device__ __forceinline__ int swz(int k) {
        return (ROWS % 128 == 0 ? (k & 3) << 2 : ((k >> 1) & 1) << 2) ^ (((k >> 3) & 1) << 1);
    }
    uint32_t voff[PER];
    __device__ __forceinline__ void init(int64_t ld, int rows_valid, int kvalid, int wave, int lane) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = (i * NW + wave) * 64 + lane, kk = at / CPK, c = (at % CPK) ^ swz(kk);
            voff[i] = (c * 8 < rows_valid && kk < kvalid) ? (uint32_t)(((int64_t)kk * ld + c * 8) * 2) : DL_OOB;
        }
    }
    static __device__ __forceinline__ uint32_t tile_step(int64_t ld) { return (uint32_t)(BK * ld * 2); }
    __device__ __forceinline__ void load_one(int i, i32x4 rsrc, uint32_t kb, uint32_t stage, int wave) const {
        load_to_lds_b128(rsrc, stage + (i * NW + wave) * 1024, voff[i], kb);
    }
    // transposing read: within 16 lanes, lanes 4j..4j+3 address k-row j (32 consecutive bytes); lane i receives
    // column i of four consecutive k
    uint32_t foff[8];                                           // per 16-row group of the wavefront's tile
    __device__ __forceinline__ void init_frag(int row0, int lane) {
        const int kk = (lane >> 4) * 8 + ((lane & 15) >> 2);
#pragma unroll
        for (int sub = 0; sub < 8; ++sub) {
            const int col = row0 + sub * 16 + (lane & 3) * 4;
            foff[sub] = (uint32_t)(kk * (ROWS * 2) + (((col >> 3) ^ swz(kk)) << 4) + (col & 7) * 2);
        }
    }
    __device__ __forceinline__ bf16x8 frag(const unsigned char *stage, int sub, int ks) const {
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const unsigned char *p = stage + foff[sub] + ks * 32 * (ROWS * 2);
        union { s16x4 h[2]; bf16x8 v; } f;
        f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
        f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * (ROWS * 2)));
        return f.v;
    }
    __device__ __forceinline__ void second_step() {
#pragma unroll
        for (int sub = 0; sub < 8; ++sub) foff[sub] += 32 * ROWS * 2;
    }
    static __device__ __forceinline__ void clear_tail(unsigned char *, int, int) {}       // whole k-rows: masked on their way in
};

// Workgroup -> output tile and contraction range; each XCD's L2 sees one contiguous part of the tile sequence (and, where the
// number of ranges allows it, one range).  false: a padding workgroup.
__device__ __forceinline__ bool place(int tiles_m, int tiles_n, int xsplits, int &split, int &nsplit, int &tm, int &tn) {
    const int total_tiles = tiles_m * tiles_n;
    int bid;
    if (xsplits) {
        const int x = (int)(blockIdx.x % 8), i = (int)(blockIdx.x / 8);
        const int parts = 8 / xsplits, chunk = (total_tiles + parts - 1) / parts;
        nsplit = xsplits;
        split = x % xsplits;
        if (i >= chunk) return false;
        bid = (x / xsplits) * chunk + i;
    } else {
        nsplit = (int)gridDim.y;
        split = (int)blockIdx.y;
        bid = (int)(blockIdx.x % 8) * ((total_tiles + 7) / 8) + (int)(blockIdx.x / 8);
    }
    if (bid >= total_tiles) return false;
    // consecutive workgroups walk down GROUP tile rows before moving to the next tile column; products with very many tile
    // rows (weight gradients of the wide layers) do better with the narrower band (measured: +3..5 % there, -2 % elsewhere)
    const int GROUP = tiles_m > 64 ? 4 : 8;
    const int per_group = GROUP * tiles_n;
    const int g = bid / per_group;
    const int gm0 = g * GROUP;
    const int gsz = tiles_m - gm0 < GROUP ? tiles_m - gm0 : GROUP;
    tm = gm0 + (bid % per_group) % gsz;
    tn = (bid % per_group) / gsz;
    return true;
}

// Row sums of A as products with a vector of ones: rs[u] belongs to the 16-row group 2u + wn of the wavefront (the two
// wavefronts that share A's rows take every other group), lane l holds the sum of its row l%16.
__device__ __forceinline__ bf16x8 ones8() {
    Frag f;
    f.u = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    return f.v;
}
template <int TM>
__device__ __forceinline__ void store_rowsum(const floatx4 (&rs)[TM / 2], int lane, int wn, int64_t mw, int64_t M, int64_t N, uint16_t *rowsum,
                                             int accumulate, float *ws, int split, int nsplit) {
#pragma unroll
    for (int u = 0; u < TM / 2; ++u) {
        const int64_t m = mw + (2 * u + wn) * 16 + lane;
        if (lane < 16 && m < M) {
            if (ws) ws[(int64_t)nsplit * M * partial_ld(N) + (int64_t)split * M + m] = rs[u][0];
            else rowsum[m] = (uint16_t)f32_to_bf16_bits(rs[u][0] + (accumulate ? bf16_bits_to_f32(rowsum[m]) : 0.f));
        }
    }
}

// What a lane has of eight columns of a row of which the first n are there (rows start on 8-byte boundaries): whole groups of four,
// and up to three elements behind them, which are put together only where they are used: doing so behind their loads would wait for
// them.  Missing elements are zero.
struct Piece {
    uint2 lo, hi;
    uint32_t t[3];
    __device__ __forceinline__ void load(const uint16_t *p, int n) {
        lo = hi = make_uint2(0, 0);
        t[0] = t[1] = t[2] = 0;
        if (n >= 4) lo = *reinterpret_cast<const uint2 *>(p);
        if (n >= 8) hi = *reinterpret_cast<const uint2 *>(p + 4);
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < (n & 3)) t[e] = p[(n & 4) + e];
    }
    __device__ __forceinline__ uint4 get(int n) const {
        const uint2 w = make_uint2(t[0] | (t[1] << 16), t[2]);
        const uint2 a = n >= 4 ? lo : w, b = n >= 8 ? hi : n > 4 ? w : make_uint2(0, 0);
        return make_uint4(a.x, a.y, b.x, b.y);
    }
    static __device__ __forceinline__ void store(uint16_t *p, const uint4 &v, int n) {
        if (n >= 4) *reinterpret_cast<uint2 *>(p) = make_uint2(v.x, v.y);
        if (n >= 8) *reinterpret_cast<uint2 *>(p + 4) = make_uint2(v.z, v.w);
        const uint32_t w0 = n & 4 ? v.z : v.x, w1 = n & 4 ? v.w : v.y, u[3] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu};
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < (n & 3)) p[(n & 4) + e] = (uint16_t)u[e];
    }
};
__device__ __forceinline__ void add8(float (&v)[8], const uint4 &t) {
    const uint32_t u[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[2 * e] += __uint_as_float(u[e] << 16); v[2 * e + 1] += __uint_as_float(u[e] & 0xffff0000u); }
}

// ---- epilogue: a wavefront's part of the output tile through LDS as fp32, 16 rows at a time, so that a lane ends up with eight
// consecutive columns of one row: bias, residual and output (or the fp32 partial tile of a split product) move as whole 16-byte chunks.
//
// A part that lies wholly inside the output is straight-line code for the operands it has: tests of them between the blocks keep
// the compiler from having one block's LDS reads and another's stores under way together, and with one wavefront per SIMD nothing
// else hides them.  With a residual the next blocks' reads of it and of LDS are issued ahead as well.  Measured with 256x256 tiles and
// operands in the caches, us, tests inside / straight-line: 8192 x 4096 x 64 24.1 / 21.9, with bias 27.4 / 21.8, with residual 39.0 /
// 33.2; 8192 x 12288 x 768 149 / 142, with bias 164 / 146, with residual 211 / 193.
template <int TM, int TN> struct Part {
    static constexpr int WN = TN * 16, SPF = WN + 4, CPR = WN / 8, PASSES = 16 * CPR / 64;
    static_assert((16 * CPR) % 64 == 0, "a 16-row block is a whole number of wavefront passes");
    int row[PASSES], col[PASSES];                    // this lane's chunks of a block
    __device__ __forceinline__ explicit Part(int lane) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            row[p] = (p * 64 + lane) / CPR;
            col[p] = (p * 64 + lane) % CPR * 8;
        }
    }
    static __device__ __forceinline__ void to_lds(float *at, const floatx4 (&acc)[TN], int lane) {
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<floatx4 *>(at + (lane & 15) * SPF + j * 16 + (lane >> 4) * 4) = acc[j];
    }
    __device__ __forceinline__ void from_lds(float (&v)[PASSES][8], const float *at) const {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 t = *reinterpret_cast<const float4 *>(at + row[p] * SPF + col[p] + 4 * h);
                v[p][4 * h] = t.x; v[p][4 * h + 1] = t.y; v[p][4 * h + 2] = t.z; v[p][4 * h + 3] = t.w;
            }
    }
};
template <int TM> constexpr int stage_rows() { return TM * 16 < 64 ? TM * 16 : 64; }
template <int TM, int TN> constexpr int stage_floats() { return stage_rows<TM>() * Part<TM, TN>::SPF; }       // a wavefront's staging area
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
    return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}
__device__ __forceinline__ void store8(float *dst, const float (&v)[8], int n) {       // whole groups of four
    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    if (n > 4) *reinterpret_cast<float4 *>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

template <int TM, int TN, bool BIAS, bool RESID, bool WS, bool STREAM>
__device__ __forceinline__ void store_inside(const floatx4 (&acc)[TM][TN], float *stage, int lane, int64_t mw, int64_t nw, int64_t M, int64_t N,
                                             const uint16_t *__restrict__ bias, const uint16_t *resid, int64_t ldr, uint16_t *C, int64_t ldc,
                                             float *__restrict__ ws, int split) {
    using P = Part<TM, TN>;
    constexpr int PASSES = P::PASSES, AHEAD = RESID ? 1 : 0;         // blocks that pass through LDS ahead of the one being stored
    const P part(lane);
    const int64_t ldo = WS ? partial_ld(N) : ldc;
    int64_t out[PASSES], res[PASSES];
    uint4 b[PASSES], r[PASSES];
    float v[2][PASSES][8];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        out[p] = ((WS ? (int64_t)split * M : 0) + mw + part.row[p]) * ldo + nw + part.col[p];
        if (RESID) res[p] = (mw + part.row[p]) * ldr + nw + part.col[p];
        if (BIAS) b[p] = *reinterpret_cast<const uint4 *>(bias + nw + part.col[p]);
        if (RESID) r[p] = *reinterpret_cast<const uint4 *>(resid + res[p]);
    }
    auto through_lds = [&](int i) __attribute__((always_inline)) {
        float *at = stage + (i & AHEAD) * 16 * P::SPF;
        P::to_lds(at, acc[i], lane);
        __builtin_amdgcn_wave_barrier();
        part.from_lds(v[i & AHEAD], at);
        __builtin_amdgcn_wave_barrier();
    };
    if (AHEAD) through_lds(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        uint4 now[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (!RESID) continue;
            now[p] = r[p];
            if (i + 1 < TM) r[p] = *reinterpret_cast<const uint4 *>(resid + res[p] + (int64_t)(i + 1) * 16 * ldr);
        }
        if (i + AHEAD < TM) through_lds(i + AHEAD);
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            float (&x)[8] = v[i & AHEAD][p];
            if (WS) { store8(ws + out[p] + (int64_t)i * 16 * ldo, x, 8); continue; }
            if (BIAS) add8(x, b[p]);
            if (RESID) add8(x, now[p]);
            const uint4 w = pack8(x);
            uint16_t *to = C + out[p] + (int64_t)i * 16 * ldo;
            if (STREAM) __builtin_nontemporal_store((tio_u32x4){w.x, w.y, w.z, w.w}, reinterpret_cast<tio_u32x4 *>(to));
            else *reinterpret_cast<uint4 *>(to) = w;
        }
    }
}

// A part that reaches past the output's last row or column, or whose rows start on 8-byte boundaries (leading dimensions of 8k + 4):
// up to eight columns of a row at a time, of which `cols` says how many there are; nothing at or past column N or row M is touched.
// It is on the critical path of the last tiles of every row, so the residual is a block ahead here too, and a loop, since straight-line
// code for what few wavefronts run has to be fetched by them alone.  One chunk after the other, each waiting for its residual, took
// 101 us for 8192 x 4093 x 768 with residual, this 71 (256x256 tiles; operands in the caches).
template <int TM, int TN>
__device__ __forceinline__ void store_edge(const floatx4 (&acc)[TM][TN], float *stage, int lane, int64_t mw, int64_t nw, int64_t M, int64_t N,
                                           const uint16_t *__restrict__ bias, const uint16_t *resid, int64_t ldr, uint16_t *C, int64_t ldc,
                                           float *__restrict__ ws, int split) {
    using P = Part<TM, TN>;
    constexpr int PASSES = P::PASSES, BATCH = stage_rows<TM>() / 16;         // blocks in LDS at a time
    static_assert(BATCH % 2 == 0 && (TM == BATCH || TM == 2 * BATCH), "blocks in pairs, one batch or two");
    const P part(lane);
    const int rows = M - mw < TM * 16 ? (int)(M - mw) : TM * 16;
    const int64_t ldo = ws ? partial_ld(N) : ldc;
    int cols[PASSES];
    int64_t out[PASSES], res[PASSES];
    uint4 b[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int64_t left = N - nw - part.col[p];
        cols[p] = left >= 8 ? 8 : left > 0 ? (int)left : 0;
        out[p] = ((ws ? (int64_t)split * M : 0) + mw + part.row[p]) * ldo + nw + part.col[p];
        res[p] = (mw + part.row[p]) * ldr + nw + part.col[p];
        if (bias) {
            Piece t;
            t.load(bias + nw + part.col[p], cols[p]);
            b[p] = t.get(cols[p]);
        }
    }
    auto load_resid = [&](int g, Piece (&r)[PASSES]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) r[p].load(resid + res[p] + (int64_t)g * 16 * ldr, g * 16 + part.row[p] < rows ? cols[p] : 0);
    };
    auto block = [&](int g, const Piece (&r)[PASSES], Piece (&ahead)[PASSES]) __attribute__((always_inline)) {
        if (resid && g + 1 < TM) load_resid(g + 1, ahead);
        float v[PASSES][8];
        part.from_lds(v, stage + (g % BATCH) * 16 * P::SPF);
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (g * 16 + part.row[p] >= rows || cols[p] == 0) continue;
            if (ws) { store8(ws + out[p] + (int64_t)g * 16 * ldo, v[p], cols[p]); continue; }
            if (bias) add8(v[p], b[p]);
            if (resid) add8(v[p], r[p].get(cols[p]));
            Piece::store(C + out[p] + (int64_t)g * 16 * ldo, pack8(v[p]), cols[p]);
        }
    };
    Piece r0[PASSES], r1[PASSES];
    if (resid) load_resid(0, r0);
    auto batch = [&](auto FIRST) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < BATCH; ++i) P::to_lds(stage + i * 16 * P::SPF, acc[FIRST() + i], lane);
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int g = FIRST(); g < FIRST() + BATCH; g += 2) {
            block(g, r0, r1);
            block(g + 1, r1, r0);
        }
        __builtin_amdgcn_wave_barrier();
    };
    batch(std::integral_constant<int, 0>{});
    if constexpr (TM > BATCH) batch(std::integral_constant<int, BATCH>{});
}
// An output larger than the memory-side cache (256 MiB) is stored past the caches: nothing of it would be found there, and dirty lines
// take the operands' place.  That is decided by the size of the product, for both of its launches where it has two, and holds for the parts
// inside plain outputs; those with bias or residual, the ragged ends and the sums of cut contractions are stored as ever.
// us: 8192 x 50176 x 768 608 -> 557, 8192 x 50257 x 768 667 -> 588, 8192 x 22016 x 4096 1011 -> 996, 8192 x 32000 x
// 4096 1482 both; with 100 MB (1021 x 50257 x 768) it would be 101 -> 104; in two launches 8176 x 16470 x 3143 747 -> 665, whose first has
// just under 256 MiB.
constexpr int64_t STREAMED = (int64_t)1 << 27;          // elements
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const floatx4 (&acc)[TM][TN], float *stage, int lane, int64_t mw, int64_t nw, int64_t M, int64_t N,
                                           const uint16_t *__restrict__ bias, const uint16_t *resid, int64_t ldr, uint16_t *C, int64_t ldc,
                                           float *__restrict__ ws, int split, int streamed) {
    const bool inside = mw + TM * 16 <= M && nw + TN * 16 <= N;
    const bool wide = ldc % 8 == 0 && (resid == nullptr || ldr % 8 == 0);
#define TIO_STORE(BIAS, RESID, WS, STREAM) store_inside<TM, TN, BIAS, RESID, WS, STREAM>(acc, stage, lane, mw, nw, M, N, bias, resid, ldr, C, ldc, ws, split)
    if (inside && ws) TIO_STORE(false, false, true, false);
    else if (inside && wide) {
        if (bias && resid) TIO_STORE(true, true, false, false);
        else if (bias) TIO_STORE(true, false, false, false);
        else if (resid) TIO_STORE(false, true, false, false);
        else if (streamed) TIO_STORE(false, false, false, true);
        else TIO_STORE(false, false, false, false);
    } else if (mw < M && nw < N) store_edge<TM, TN>(acc, stage, lane, mw, nw, M, N, bias, resid, ldr, C, ldc, ws, split);
#undef TIO_STORE
}

template <int BM, int BN, int WGM, int WGN, int D, bool AKM, bool BKM, bool ROWSUM>
__global__ void __launch_bounds__(WGM *WGN * 64)
    gemm_bf16_dl_k(const uint16_t *__restrict__ A, int64_t lda, const uint16_t *__restrict__ B, int64_t ldb,
                   const uint16_t *__restrict__ bias, const uint16_t *__restrict__ resid, int64_t ldr,
                   uint16_t *__restrict__ C, int64_t ldc, int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n,
                   uint16_t *__restrict__ rowsum, float *__restrict__ ws, int64_t k_chunk, int rowsum_acc, int xsplits, int streamed) {
    constexpr int NT = WGM * WGN * 64;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
    static_assert(TM <= 8 && TN <= 8 && BK == 64, "two contraction steps of 32 per tile");
    using OpA = DlOperand<BM, NT, AKM>;
    using OpB = DlOperand<BN, NT, BKM>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_dl[];

    const int tid = threadIdx.x;
    int split, nsplit, tm, tn;
    if (!place(tiles_m, tiles_n, xsplits, split, nsplit, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave / WGN, wn = wave % WGN;

    const int64_t kbeg = (int64_t)split * k_chunk;
    const int64_t kend = (ws != nullptr && kbeg + k_chunk < K) ? kbeg + k_chunk : K;
    const int kspan = kend > kbeg ? (int)(kend - kbeg) : 0;
    const int nkf = kspan / BK, rem = kspan % BK, nk = nkf + (rem ? 1 : 0);

    const int rows_a = (int)(M - m0 < BM ? M - m0 : BM), rows_b = (int)(N - n0 < BN ? N - n0 : BN);
    const uint16_t *baseA = AKM ? A + kbeg * lda + m0 : A + m0 * lda + kbeg;
    const uint16_t *baseB = BKM ? B + kbeg * ldb + n0 : B + n0 * ldb + kbeg;
    const int k8 = (kspan + 7) / 8 * 8;
    const int64_t recA = kspan == 0 ? 0 : AKM ? ((int64_t)(kspan - 1) * lda + (rows_a + 7) / 8 * 8) * 2 : ((int64_t)(rows_a - 1) * lda + k8) * 2;
    const int64_t recB = kspan == 0 ? 0 : BKM ? ((int64_t)(kspan - 1) * ldb + (rows_b + 7) / 8 * 8) * 2 : ((int64_t)(rows_b - 1) * ldb + k8) * 2;
    const i32x4 rsA = make_rsrc(baseA, (uint32_t)recA), rsB = make_rsrc(baseB, (uint32_t)recB);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem_dl));
    const uint32_t stepA = OpA::tile_step(lda), stepB = OpB::tile_step(ldb);

    OpA oa;
    OpB ob;
    oa.init(lda, rows_a, BK, wave, lane);
    ob.init(ldb, rows_b, BK, wave, lane);
    oa.init_frag(wm * WM, lane);
    ob.init_frag(wn * WN, lane);

    // acc[i][j]: lane l holds C row 16 i + l%16, columns 16 j + 4 (l/16) + 0..3
    floatx4 acc[TM][TN], rs[TM / 2];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        rs[i / 2] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    }
    static_assert(WGN == 2 && TM % 2 == 0, "row sums: two wavefronts share A's rows");
    const bool do_rowsum = ROWSUM && tn == 0;
    const int rs_group = do_rowsum ? wn : 2;
    bf16x8 ones = ones8();
    if (ROWSUM) asm volatile("" : "+v"(ones));       // written once, here: not right before a product that reads it

    // LDS: a ring of D + 1 A tiles, then one of D B tiles.  While tile t is multiplied, the tiles up to t + D - 1 sit there or
    // are landing; A's spare slot takes A of tile t + D in the first half of the tile, and B's slot of tile t itself takes B of
    // tile t + D in the second half, when its last fragments are in registers.
    constexpr uint32_t RINGA = (D + 1) * OpA::BYTES, RINGB = D * OpB::BYTES;
    auto next_a = [&](uint32_t at) __attribute__((always_inline)) { return at + OpA::BYTES >= RINGA ? 0u : at + OpA::BYTES; };
    auto next_b = [&](uint32_t at) __attribute__((always_inline)) { return at + OpB::BYTES >= RINGA + RINGB ? RINGA : at + OpB::BYTES; };
    auto load_tile = [&](int kt, uint32_t at, auto OP) __attribute__((always_inline)) {      // kt < nk; OP 0: A, 1: B
        constexpr bool isA = OP() == 0;
        if (kt < nkf) {
#pragma unroll
            for (int l = 0; l < (isA ? OpA::PER : OpB::PER); ++l) {
                if (isA) oa.load_one(l, rsA, (uint32_t)kt * stepA, lds0 + at, wave);
                else ob.load_one(l, rsB, (uint32_t)kt * stepB, lds0 + at, wave);
            }
        } else if (isA) {                            // the last, partial tile: chunks beyond the contraction read as zero
            OpA t;
            t.init(lda, rows_a, rem, wave, lane);
#pragma unroll
            for (int l = 0; l < OpA::PER; ++l) t.load_one(l, rsA, (uint32_t)kt * stepA, lds0 + at, wave);
        } else {
            OpB t;
            t.init(ldb, rows_b, rem, wave, lane);
#pragma unroll
            for (int l = 0; l < OpB::PER; ++l) t.load_one(l, rsB, (uint32_t)kt * stepB, lds0 + at, wave);
        }
    };
    // tile kt has landed for every wavefront: what a partial chunk brought from behind the contraction's end goes to zero
    auto clear_tail = [&](int kt, uint32_t atA, uint32_t atB) __attribute__((always_inline)) {
        if (kt == nkf && (rem & 7)) {
            OpA::clear_tail(smem_dl + atA, rem, tid);
            OpB::clear_tail(smem_dl + atB, rem, tid);
            __syncthreads();
        }
    };

    bf16x8 fa[2][TM], fb[2][TN];
    // fragment r of a step in the order the products need them: A row group 0, every B column group, the other A row groups
    auto read_one = [&](int set, uint32_t atA, uint32_t atB, int ks, int r) __attribute__((always_inline)) {
        if (r == 0) fa[set][0] = oa.frag(smem_dl + atA, 0, ks);
        else if (r <= TN) fb[set][r - 1] = ob.frag(smem_dl + atB, r - 1, ks);
        else fa[set][r - TN] = oa.frag(smem_dl + atA, r - TN, ks);
    };
    constexpr int NQ = TM * TN, NR = TM + TN;
    // The products of one contraction step from register set S, with the next step's fragment reads and the loads of one
    // operand tile between them in a pinned order: the reads over the first three quarters, so that the last one has landed
    // when the step ends; the loads evenly over the whole step (LOADS 0: none, 1: A, 2: B): a compute unit takes sixteen
    // clocks for each, and a wavefront whose load finds the queue full stalls with its products.
    // Column groups are taken back and forth, so that consecutive products always share an operand, which draws less power: 8192 x 22016
    // x 4096 976 -> 969 us, 22016 x 4096 x 8192 with both operands k-major 1040 -> 1031 (a loop of products alone 2040 -> 2085 TFLOP/s).
    // The row sums' product follows the first one of an odd row group, not the last, where the next step's reads are already done:
    // 768 x 3072 x 8192 77.6 -> 76.6 us, 3072 x 768 x 8192 51.1 -> 50.4.
    auto step = [&](auto S, uint32_t rA, uint32_t rB, auto RKS, auto LOADS, int lkt, uint32_t at) __attribute__((always_inline)) {
        constexpr int NL = LOADS() == 1 ? OpA::PER : LOADS() == 2 ? OpB::PER : 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int i = q / TN, j = i % 2 ? TN - 1 - q % TN : q % TN, l = q * NL / NQ;
            if (NL > 0 && (q == 0 || (q - 1) * NL / NQ != l)) {
                if (LOADS() == 1) mfma_acc_load(acc[i][j], fb[S()][j], fa[S()][i], rsA, lds0 + at + (l * OpA::NW + wave) * 1024, oa.voff[l % OpA::PER], (uint32_t)lkt * stepA);
                else mfma_acc_load(acc[i][j], fb[S()][j], fa[S()][i], rsB, lds0 + at + (l * OpB::NW + wave) * 1024, ob.voff[l % OpB::PER], (uint32_t)lkt * stepB);
            } else {
                mfma_acc(acc[i][j], fb[S()][j], fa[S()][i]);
            }
            if (ROWSUM && q % TN == 0 && i % 2 == 1) mfma_pick(rs[i / 2], ones, fa[S()][i - 1], fa[S()][i], rs_group);
#pragma unroll
            for (int r = q * NR * 4 / (NQ * 3); r < (q + 1) * NR * 4 / (NQ * 3) && r < NR; ++r) read_one(S() ^ 1, rA, rB, RKS(), r);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr auto wait_vm = [](int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); };      // s_waitcnt vmcnt(n)
    constexpr int PA = OpA::PER, PB = OpB::PER;
    static_assert((D - 1) * (PA + PB) < 64, "loads in flight fit the counter");

    // prologue: tiles 0 .. D - 1 on their way, tile 0 landed, fragments of its step 0 in registers
#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < nk) {
            load_tile(t, t * OpA::BYTES, c0);
            load_tile(t, RINGA + t * OpB::BYTES, c1);
        }
    if (nk >= D) __builtin_amdgcn_s_waitcnt(wait_vm((D - 1) * (PA + PB)));       // the later tiles' loads may be outstanding
    else __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
    clear_tail(0, 0, RINGA);
    if (nk > 0) {
#pragma unroll
        for (int r = 0; r < NR; ++r) read_one(0, 0, RINGA, 0, r);
    }
    auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
        if (ROWSUM) {
#pragma unroll
            for (int u = 0; u < TM / 2; ++u) asm volatile("" : "+v"(rs[u]));
        }
    };
    pin();
    settle();

    uint32_t atA = 0, atB = RINGA, spareA = D * OpA::BYTES;      // ring offsets: tile kt's operands, A's spare slot
    auto tile = [&](int kt, auto FULL) __attribute__((always_inline)) {      // FULL: tile kt + D is a full tile
        const uint32_t nxA = next_a(atA), nxB = next_b(atB);
        if (FULL()) {
            step(c0, atA, atB, c1, c1, kt + D, spareA);
        } else {
            if (kt + D < nk) load_tile(kt + D, spareA, c0);
            step(c0, atA, atB, c1, c0, 0, 0);
        }
        // tile kt+1 has landed for this wavefront (later tiles' loads may be outstanding); after the barrier it has landed for
        // all, and nobody reads tile kt's slots any more
        if (FULL()) __builtin_amdgcn_s_waitcnt(wait_vm((D - 1) * PA + (D - 2) * PB) & 0xC0FF);     // and lgkmcnt(0)
        else __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (FULL()) {
            step(c1, nxA, nxB, c0, c2, kt + D, atB);
        } else {
            if (kt + 1 < nk) clear_tail(kt + 1, nxA, nxB);
            if (kt + D < nk) load_tile(kt + D, atB, c1);
            step(c1, nxA, nxB, c0, c0, 0, 0);        // after the last tile these reads fetch nothing that is used
        }
        spareA = atA;
        atA = nxA;
        atB = nxB;
    };
    int kt = 0;
    for (; kt + D < nkf; ++kt) tile(kt, c1);
    for (; kt < nk; ++kt) tile(kt, c0);
    settle();
    pin();

    if (do_rowsum) store_rowsum<TM>(rs, lane, wn, m0 + wm * WM, M, N, rowsum, rowsum_acc, ws, split, nsplit);
    store_tile<TM, TN>(acc, reinterpret_cast<float *>(smem_dl) + wave * stage_floats<TM, TN>(), lane, m0 + wm * WM, n0 + wn * WN, M, N, bias, resid,
                       ldr, C, ldc, ws, split, streamed);      // the rings are free: the last barrier came after every fragment read
    static_assert((size_t)RINGA + RINGB >= (size_t)WGM * WGN * stage_floats<TM, TN>() * 4, "the staging blocks fit the rings");
}

// 64x64 tiles for products with too few larger ones: eight wavefronts in two groups, each with one of the two contraction steps
// of every tile, so that two wavefronts per SIMD cover each other's LDS latency; the groups' sums are added in order.  A tile
// is 256 clocks of loads and 128 of products, so the ring is D tiles deep.
template <int D, bool AKM, bool BKM, bool ROWSUM>
__global__ void __launch_bounds__(512)
    gemm_bf16_small_k(const uint16_t *__restrict__ A, int64_t lda, const uint16_t *__restrict__ B, int64_t ldb,
                      const uint16_t *__restrict__ bias, const uint16_t *__restrict__ resid, int64_t ldr,
                      uint16_t *__restrict__ C, int64_t ldc, int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n,
                      uint16_t *__restrict__ rowsum, float *__restrict__ ws, int64_t k_chunk, int rowsum_acc, int xsplits, int streamed) {
    constexpr int BM = 64, BN = 64, NT = 512, TM = 2, TN = 2;
    using OpA = DlOperand<BM, NT, AKM>;
    using OpB = DlOperand<BN, NT, BKM>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_dl[];

    const int tid = threadIdx.x;
    int split, nsplit, tm, tn;
    if (!place(tiles_m, tiles_n, xsplits, split, nsplit, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

    const int64_t kbeg = (int64_t)split * k_chunk;
    const int64_t kend = (ws != nullptr && kbeg + k_chunk < K) ? kbeg + k_chunk : K;
    const int kspan = kend > kbeg ? (int)(kend - kbeg) : 0;
    const int nkf = kspan / BK, rem = kspan % BK, nk = nkf + (rem ? 1 : 0);

    const int rows_a = (int)(M - m0 < BM ? M - m0 : BM), rows_b = (int)(N - n0 < BN ? N - n0 : BN);
    const uint16_t *baseA = AKM ? A + kbeg * lda + m0 : A + m0 * lda + kbeg;
    const uint16_t *baseB = BKM ? B + kbeg * ldb + n0 : B + n0 * ldb + kbeg;
    const int k8 = (kspan + 7) / 8 * 8;
    const int64_t recA = kspan == 0 ? 0 : AKM ? ((int64_t)(kspan - 1) * lda + (rows_a + 7) / 8 * 8) * 2 : ((int64_t)(rows_a - 1) * lda + k8) * 2;
    const int64_t recB = kspan == 0 ? 0 : BKM ? ((int64_t)(kspan - 1) * ldb + (rows_b + 7) / 8 * 8) * 2 : ((int64_t)(rows_b - 1) * ldb + k8) * 2;
    const i32x4 rsA = make_rsrc(baseA, (uint32_t)recA), rsB = make_rsrc(baseB, (uint32_t)recB);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem_dl));
    const uint32_t stepA = OpA::tile_step(lda), stepB = OpB::tile_step(ldb);

    OpA oa;
    OpB ob;
    oa.init(lda, rows_a, BK, wave, lane);
    ob.init(ldb, rows_b, BK, wave, lane);
    oa.init_frag(wm * 32, lane);
    ob.init_frag(wn * 32, lane);
    if (kg) {                                        // this wavefront's contraction step is the second one
        oa.second_step();
        ob.second_step();
    }

    floatx4 acc[TM][TN], rs[1] = {(floatx4){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    const bool do_rowsum = ROWSUM && tn == 0;
    const bf16x8 ones = ones8();

    constexpr uint32_t TILE = OpA::BYTES + OpB::BYTES;
    constexpr int PL = OpA::PER + OpB::PER;
    auto load_tile = [&](int kt, uint32_t at) __attribute__((always_inline)) {      // kt < nk
        if (kt < nkf) {
#pragma unroll
            for (int l = 0; l < OpA::PER; ++l) oa.load_one(l, rsA, (uint32_t)kt * stepA, lds0 + at, wave);
#pragma unroll
            for (int l = 0; l < OpB::PER; ++l) ob.load_one(l, rsB, (uint32_t)kt * stepB, lds0 + at + OpA::BYTES, wave);
        } else {                                     // the last, partial tile: chunks beyond the contraction read as zero
            OpA ta;
            OpB tb;
            ta.init(lda, rows_a, rem, wave, lane);
            tb.init(ldb, rows_b, rem, wave, lane);
#pragma unroll
            for (int l = 0; l < OpA::PER; ++l) ta.load_one(l, rsA, (uint32_t)kt * stepA, lds0 + at, wave);
#pragma unroll
            for (int l = 0; l < OpB::PER; ++l) tb.load_one(l, rsB, (uint32_t)kt * stepB, lds0 + at + OpA::BYTES, wave);
        }
    };
    auto clear_tail = [&](int kt, uint32_t at) __attribute__((always_inline)) {
        if (kt == nkf && (rem & 7)) {
            OpA::clear_tail(smem_dl + at, rem, tid);
            OpB::clear_tail(smem_dl + at + OpA::BYTES, rem, tid);
            __syncthreads();
        }
    };
    bf16x8 fa[2][TM], fb[2][TN];
    auto read_frags = [&](auto S, uint32_t at) __attribute__((always_inline)) {
        const unsigned char *As = smem_dl + at, *Bs = As + OpA::BYTES;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[S()][i] = oa.frag(As, i, 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[S()][j] = ob.frag(Bs, j, 0);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr auto wait_vm = [](int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); };      // s_waitcnt vmcnt(n)
    static_assert(D * PL < 64, "loads in flight fit the counter");

#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < nk) load_tile(t, t * TILE);
    if (nk >= D) __builtin_amdgcn_s_waitcnt(wait_vm((D - 1) * PL));
    else __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
    clear_tail(0, 0);
    if (nk > 0) read_frags(c0, 0);

    uint32_t at = 0;                                 // ring offset of tile kt, whose fragments are in set S or on their way there
    auto tile = [&](int kt, auto S, auto FULL) __attribute__((always_inline)) {
        constexpr std::integral_constant<int, (S() ^ 1)> other{};
        const uint32_t nx = at + TILE >= D * TILE ? 0u : at + TILE;
        // tile kt+1 has landed; tile kt's fragments are in everybody's registers, its slot is free
        if (FULL()) __builtin_amdgcn_s_waitcnt(wait_vm((D - 2) * PL) & 0xC0FF);
        else __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (!FULL() && kt + 1 < nk) clear_tail(kt + 1, nx);
        read_frags(other, nx);                       // after the last tile these reads fetch nothing that is used
        if (FULL() || kt + D < nk) load_tile(kt + D, at);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[S()][j], fa[S()][i], acc[i][j], 0, 0, 0);
        if (ROWSUM && do_rowsum) rs[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, wn ? fa[S()][1] : fa[S()][0], rs[0], 0, 0, 0);
        at = nx;
    };
    int kt = 0;
    for (; kt + 1 + D < nkf; kt += 2) {
        tile(kt, c0, c1);
        tile(kt + 1, c1, c1);
    }
    for (; kt < nk; kt += 2) {
        tile(kt, c0, c0);
        if (kt + 1 < nk) tile(kt + 1, c1, c0);
    }

    // the second group's sums join the first's
    float *red = reinterpret_cast<float *>(smem_dl) + (wave & 3) * (TM * TN * 4 + 1) * 64 + lane;
    __syncthreads();
    if (kg) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[((i * TN + j) * 4 + e) * 64] = acc[i][j][e];
        }
        red[TM * TN * 4 * 64] = rs[0][0];
    }
    __syncthreads();
    if (kg) return;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] += red[((i * TN + j) * 4 + e) * 64];
    }
    rs[0][0] += red[TM * TN * 4 * 64];
    if (do_rowsum) store_rowsum<TM>(rs, lane, wn, m0 + wm * 32, M, N, rowsum, rowsum_acc, ws, split, nsplit);
    constexpr size_t RED = 4 * (TM * TN * 4 + 1) * 64 * 4;
    static_assert(D * TILE >= RED + 4 * stage_floats<TM, TN>() * 4, "reduction and staging blocks fit the ring");
    store_tile<TM, TN>(acc, reinterpret_cast<float *>(smem_dl + RED) + wave * stage_floats<TM, TN>(), lane, m0 + wm * 32, n0 + wn * 32, M, N, bias, resid, ldr,
                       C, ldc, ws, split, streamed);
}
struct Product {
    hipStream_t s;
    bool a_km, b_km;
    int64_t M, N, K;
    const uint16_t *A;
    int64_t lda;
    const uint16_t *B;
    int64_t ldb;
    const uint16_t *bias, *resid;
    int64_t ldr;
    uint16_t *C;
    int64_t ldc;
    uint16_t *rowsum;
    float *ws;
    int splits, rowsum_acc, streamed;
};

template <auto *KERNEL> void launch(const Product &p, int BM, int BN, int threads, size_t lds) {
    static const hipError_t raised = hipFuncSetAttribute((const void *)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)raised;
    const int64_t k_chunk = p.splits > 1 ? ((p.K + p.splits - 1) / p.splits + BK - 1) / BK * BK : p.K;
    const int tiles_m = (int)((p.M + BM - 1) / BM), tiles_n = (int)((p.N + BN - 1) / BN), tiles = tiles_m * tiles_n;
    const int xsplits = (p.splits == 2 || p.splits == 4 || p.splits == 8) ? p.splits : 0;
    const dim3 grid = xsplits ? dim3((unsigned)(8 * ((tiles + 8 / xsplits - 1) / (8 / xsplits))))
                              : dim3((unsigned)(8 * ((tiles + 7) / 8)), (unsigned)(p.splits > 1 ? p.splits : 1));
    KERNEL<<<grid, threads, lds, p.s>>>(p.A, p.lda, p.B, p.ldb, p.bias, p.resid, p.ldr, p.C, p.ldc, p.M, p.N, p.K, tiles_m, tiles_n,
                                        p.rowsum, p.ws, k_chunk, p.rowsum_acc, xsplits, p.streamed);
}

// With row sums the layout of a weight gradient (both operands k-major) has every tile, the others the two square ones above 64:
// the large one for outputs that fill the chip with it (8192 x 22016 x 4096, A and B contraction-contiguous: 1050 us, 1385 with 128x128
// alone; the kernel with eight wavefronts before took 1182).
constexpr bool row_sums_in_every_layout(int bm, int bn) { return bm == bn && bm >= 128; }
template <int BM, int BN, int D> void launch_dl(const Product &p) {
    constexpr size_t lds = (size_t)((D + 1) * BM + D * BN) * BK * 2;
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
#define TIO_DL(AKM, BKM, RS) launch<gemm_bf16_dl_k<BM, BN, 2, 2, D, AKM, BKM, RS>>(p, BM, BN, 256, lds)
    if (p.rowsum) {
        if (p.a_km && p.b_km) TIO_DL(true, true, true);
        else if constexpr (row_sums_in_every_layout(BM, BN)) {
            if (p.a_km) TIO_DL(true, false, true);
            else if (p.b_km) TIO_DL(false, true, true);
            else TIO_DL(false, false, true);
        }
    } else if (!p.a_km && !p.b_km) TIO_DL(false, false, false);
    else if (!p.a_km && p.b_km) TIO_DL(false, true, false);
    else if (p.a_km && p.b_km) TIO_DL(true, true, false);
    else TIO_DL(true, false, false);
#undef TIO_DL
}
template <int D> void launch_small(const Product &p) {
    constexpr size_t lds = (size_t)D * 128 * BK * 2;
#define TIO_SMALL(AKM, BKM, RS) launch<gemm_bf16_small_k<D, AKM, BKM, RS>>(p, 64, 64, 512, lds)
    if (p.rowsum) TIO_SMALL(true, true, true);
    else if (!p.a_km && !p.b_km) TIO_SMALL(false, false, false);
    else if (!p.a_km && p.b_km) TIO_SMALL(false, true, false);
    else if (p.a_km && p.b_km) TIO_SMALL(true, true, false);
    else TIO_SMALL(true, false, false);
#undef TIO_SMALL
}

// The tiles and what they take, in microseconds: `tile` per contraction tile of 64 with the chip full (the clock follows the
// power drawn: 0.6 of it with few compute units busy), `fixed` per output tile (first loads, epilogue).  per_cu = 2: two
// workgroups share a compute unit, so a round is 512 of them; `solo` / `solo_fixed` where there are no more workgroups than units.
// Checked on 137 products (the GPT-2-small, Llama-7B and ragged shapes, contractions from 64, random sizes, layouts and epilogues;
// operands in no cache): the choice is the fastest tile or one within 4 % of it on 131 of them, 17 % slower on the worst.  A ragged
// output costs a quarter of `fixed` once, because the parts that end inside the output are stored piece by piece and, in the last round,
// behind nothing: without that term 3328 x 3904 x 128 with cached operands took 256x256 (15 us; 128x128 12).
// Some of them, 256x256 / 256x192 / 128x192 / 128x128 / 64x64, us (before, choosing between eight wavefronts on the first and the fourth by
// the fill of the last round: 8192 x 768 x 3072 53, head 1021 x 768 x 50257 528 and 1021 x 50257 x 768 110, 1024^3 15, 8192 x 4096 x 128 30):
//    8192 x  768 x  3072   62 /  55 /  41 /  49 /  72      1021 x   768 x 50257  1095 / 1008 / 642 /  543 / 262
//    8192 x 3072 x   768   47 /  40 /  59 /  50 /  78      1021 x 50257 x   768   101 /  104 / 130 /  113 / 183
//     768 x  768 x  8192  137 / 119 /  83 /  89 /  39      8192 x 22016 x  4096   984 / 1060 / 1360 / 1356
//    8192 x 4096 x   128   26 /  32 /  42 /  31 /  56      1000 x  5120 x  5120   101 /   83 /  63 /   82 / 100
//     256 x 12055 x 11884 284 / 242 / 205 / 151 / 217     10624 x   832 x   101    16 /   14 /  15 /   11 /  18
// The costs know neither where an operand's rows start in a cache line nor what the caches hold: for 1021 x 768 x 50257 they give the
// 64x64 tile 161 us, which it takes (158) with warm operands in rows of whole 128-byte lines; rows of 100528 bytes make that 199, and
// operands in no cache 264 (with whole lines 222).
struct TileChoice {
    int bm, bn, per_cu;
    double tile, fixed, solo, solo_fixed;
    void (*launch)(const Product &);
    double cost(int64_t M, int64_t N, int64_t nk, int splits) const {
        const int64_t groups = ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * splits;
        const double rounds = (double)((groups + 256 * per_cu - 1) / (256 * per_cu));
        const double edge = M % (bm / 2) || N % (bn / 2) ? 0.25 * fixed / rounds : 0;      // less the more rounds: few end with one
        if (per_cu == 2 && groups <= 256) return (double)nk * solo + solo_fixed + edge;
        const double clock = per_cu == 1 && groups < 256 ? 0.6 + 0.4 * (double)groups / 256 : 1.0;
        return rounds * ((double)nk * tile * clock + fixed) + edge;
    }
};
const TileChoice TILES[] = {
    {256, 256, 1, 1.33, 10, 0, 0, launch_dl<256, 256, 2>}, {256, 192, 1, 1.03, 10, 0, 0, launch_dl<256, 192, 2>},
    {128, 192, 1, 0.60, 8, 0, 0, launch_dl<128, 192, 3>},  {128, 128, 2, 0.88, 5, 0.49, 4, launch_dl<128, 128, 2>},
    {64, 64, 2, 0.42, 3, 0.2, 3.5, launch_small<4>},
};

// The tiles that can address the operands and have the layout, and what they cost.
struct Choice {
    bool a_km, b_km, rowsum;
    int64_t K, lda, ldb;
    int splits;
    int64_t kspan, nk;
    Choice(bool a_km, bool b_km, int64_t K, int64_t lda, int64_t ldb, bool rowsum, int splits)
        : a_km(a_km), b_km(b_km), rowsum(rowsum), K(K), lda(lda), ldb(ldb), splits(splits > 1 ? splits : 1),
          kspan(splits > 1 ? ((K + splits - 1) / splits + BK - 1) / BK * BK : K), nk((kspan + BK - 1) / BK) {}
    bool can(const TileChoice &t) const {
        // 32-bit buffer offsets: what one workgroup addresses of an operand has to lie within 1 GiB
        auto span = [&](bool km, int64_t rows, int64_t ld) { return (km ? (kspan + 3 * BK) * ld : rows * ld + kspan + 3 * BK) * 2; };
        constexpr int64_t LIMIT = (int64_t)1 << 30;
        return (!rowsum || (a_km && b_km) || row_sums_in_every_layout(t.bm, t.bn)) && span(a_km, t.bm, lda) < LIMIT && span(b_km, t.bn, ldb) < LIMIT;
    }
    // the tile with the lowest cost; nullptr: none can
    const TileChoice *best(int64_t M, int64_t N, double *its_cost = nullptr) const {
        const TileChoice *best = nullptr;
        double best_cost = 0;
        for (const TileChoice &t : TILES) {
            if (!can(t)) continue;
            const double cost = t.cost(M, N, nk, splits);
            if (!best || cost < best_cost) { best = &t; best_cost = cost; }
        }
        if (its_cost) *its_cost = best_cost;
        return best;
    }
};

// A product in one launch, or in two: `rows` of its rows or `cols` of its columns (the other is 0) with `first`, which are whole rounds of
// workgroups, and what is left with another tile, where the last round of one launch would be nearly empty.  That has to promise a
// fifteenth, and 3 us for the second launch: the costs are good to 4 %.  Products under 40 us are left alone (and not kept waiting for
// the comparison).  Of 40 products of random sizes that are cut, the slowest against one launch takes 1 % more, the quickest 17 % less, 6.6 %
// less on average.  us, one launch / two, each product repeated by itself: 1021 x 50257 x 768 103 / 90 (among the other products of its
// layer, with nothing of its operands in the caches, 106 / 104, and 50257 x 768 x 1021 93 / 87), 50257 x 768 x 8192 524 / 489 (both operands
// k-major), 4224 x 12277 x 4778 463 / 394, 6208 x 2880 x 19392 650 / 536, 16000 x 3136 x 2319 216 / 184, 1792 x 9664 x 704 34.8 / 30.4; 4340 x
// 9232 x 1970 148.7 / 150.0.
struct Plan {
    const TileChoice *first, *rest = nullptr;
    int64_t rows = 0, cols = 0;
    double cost = 0;                                 // us
    Plan(const Choice &c, int64_t M, int64_t N) {
        first = c.best(M, N, &cost);
        if (!first || c.splits > 1 || cost < 40) return;
        double best_cost = cost * (14.0 / 15);
        for (const TileChoice &t : TILES) {
            if (!c.can(t)) continue;
            const int64_t tm = (M + t.bm - 1) / t.bm, tn = (N + t.bn - 1) / t.bn, full = tm * tn / (256 * t.per_cu) * (256 * t.per_cu);
            if (full == 0 || full == tm * tn) continue;
            for (const bool by_rows : {false, true}) {
                const int64_t n = by_rows ? full / tn * t.bm : full / tm * t.bn;
                if (n == 0) continue;
                const int64_t m1 = by_rows ? n : M, n1 = by_rows ? N : n, m2 = by_rows ? M - n : M, n2 = by_rows ? N : N - n;
                double both = 0;
                const TileChoice *other = m2 > 0 && n2 > 0 ? c.best(m2, n2, &both) : nullptr;
                if (!other) continue;
                both += t.cost(m1, n1, c.nk, 1) + 3;
                if (both < best_cost) {
                    cost = best_cost = both;
                    first = &t;
                    rest = other;
                    rows = by_rows ? n : 0;
                    cols = by_rows ? 0 : n;
                }
            }
        }
    }
};

}  // namespace

bool gemm_bf16_direct(hipStream_t s, bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B,
                      int64_t ldb, const void *bias, const void *resid, int64_t ldr, void *C, int64_t ldc, void *rowsum, float *ws,
                      int splits, bool rowsum_accumulate) {
    const Plan plan(Choice(a_km, b_km, K, lda, ldb, rowsum != nullptr, splits), M, N);
    if (!plan.first) return false;
    Product p{s, a_km, b_km, M, N, K, (const uint16_t *)A, lda, (const uint16_t *)B, ldb, (const uint16_t *)bias, (const uint16_t *)resid,
              ldr, (uint16_t *)C, ldc, (uint16_t *)rowsum, ws, splits, (int)rowsum_accumulate, (int)(M * N >= STREAMED)};
    if (!plan.rest) {
        plan.first->launch(p);
        return true;
    }
    if (plan.rows) p.M = plan.rows;
    else p.N = plan.cols;
    plan.first->launch(p);
    if (plan.rows) {
        p.M = M - plan.rows;
        p.A += a_km ? plan.rows : plan.rows * lda;
        p.C += plan.rows * ldc;
        if (resid) p.resid += plan.rows * ldr;
        if (rowsum) p.rowsum += plan.rows;
    } else {
        p.N = N - plan.cols;
        p.B += b_km ? plan.cols : plan.cols * ldb;
        p.C += plan.cols;
        if (bias) p.bias += plan.cols;
        if (resid) p.resid += plan.cols;
        p.rowsum = nullptr;                          // the first launch has them
    }
    plan.rest->launch(p);
    return true;
}

// A long contraction with a small output leaves most compute units without a tile, and the small tiles that keep more of them busy fetch
// more than a unit can load.  Cut into ranges it costs the partials' way to memory and back, a launch and the events around the
// scratch space, and has to promise a seventh for that (the launch and the events take host time too), or a twentieth of a product of
// 100 us and more: there the costs above, made from shorter ones, promise too little (they know 480 us of the first one's 653).  us, in
// one range / cut:
//   1021 x 768 x 50257 264 / 107 (eight)    64 x 1024 x 22016 99 / 25     200 x 300 x 15000 68 / 17     300 x 300 x 8000 36 / 15
//   8192 x 768 x 50257 653 / 562 (two)      8192 x 1024 x 32000 503 / 379 (two)    4096 x 1024 x 32000 343 / 206 (four)    8192 x 512 x 20000 202 / 146
//   4096 x 2048 x 32000 494 / 374 (two)     4096 x 1792 x 12940 187 / 150 (two); left alone 8192 x 1280 x 16000 260 / 301, 8192 x 768 x 8192 85 / 89
// and left alone, though a cut with a workspace at hand gains something: 128 x 2000 x 4000 19.0 / 12.6 + 3, 1024 x 2048 x 8192 54 / 44 + 3,
// 1000 x 1000 x 10000 45 / 37 + 3; 768 x 768 x 1900 10.8 / 14.3 + 3.
int gemm_bf16_splits(bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool rowsum, int64_t bytes) {
    if (K < 2048) return 1;              // 32 tiles of the smallest kind take less than the cut costs; the small products that are quick to
                                         // run are not kept waiting for the comparison
    const Plan one(Choice(a_km, b_km, K, lda, ldb, rowsum, 1), M, N);
    if (!one.first) return 1;
    const double whole = one.cost;
    int best = 1;
    double best_cost = (whole < 100 ? 0.85 : 0.95) * whole;
    for (int s = 2; s <= 8 && K >= 256 * s; s *= 2) {
        const int64_t partials = s * (M * partial_ld(N) + M) * 4;
        double cost = 0;
        if (partials > bytes || !Choice(a_km, b_km, K, lda, ldb, rowsum, s).best(M, N, &cost)) break;
        cost += 7.5 + 2e-6 * (double)partials / 6;                // us; the partials go through the caches at 6 TB/s
        if (cost < best_cost) { best = s; best_cost = cost; }
    }
    return best;
}

void gemm_bf16_tile(bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool rowsum, int splits, int *rows,
                    int *cols) {
    const TileChoice *t = Plan(Choice(a_km, b_km, K, lda, ldb, rowsum, splits), M, N).first;
    *rows = t ? t->bm : 0;
    *cols = t ? t->bn : 0;
}

void gemm_bf16_first_launch(bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool rowsum, int64_t *rows,
                            int64_t *cols) {
    const Plan plan(Choice(a_km, b_km, K, lda, ldb, rowsum, 1), M, N);
    *rows = plan.rest ? plan.rows : 0;
    *cols = plan.rest ? plan.cols : 0;
}

}  // namespace k
}  // namespace tio
