// Causal self-attention on the matrix cores (bf16, head dimension 64 or 128), forward and backward,
// on the packed [S, 3d] q|k|v layout.
//
// Each wavefront owns 32 query rows (forward, dQ) or 32 key rows (dK/dV), or 16 where the chip has room for twice as many
// workgroups, and keeps their operand fragments in registers for the whole kernel; the other side streams through LDS in row-major
// tiles.  Scores are produced transposed (keys x queries in the forward and dQ kernels, queries x keys in the dK/dV kernel) so that in
// the accumulator layout the row owned by the wavefront is the lane index: the softmax statistics of a row live in one lane of each of
// the four groups of sixteen, and the probabilities can be fed to the second product straight from registers as its B operand.  The
// operand whose contraction index is the sequence position (V in P.V, K in dS.K, Q and dO in the dK/dV products) is read from the same
// row-major tile with the transposing LDS read (ds_read_b64_tr_b16), in the slot order the accumulator registers dictate: no
// transposed copies.
//
// All products are v_mfma_f32_16x16x32_bf16, D[16x16] += A[16x32] . B[32x16]: lane l supplies row (A) or column (B) l%16 and eight
// contraction slots of lane group l/16; of D it holds column l%16 and rows 4 (l/16) + 0..3.  At head size 128 these kernels run into
// the power limit (the clock stands at 1.5 to 1.8 GHz of 2.4 in the forward kernel, by card; on zeros, which draw less, it takes a fifth to a
// quarter less; at head size 64 2.2 GHz and 6 %), and at that limit a loop of nothing but products on normal values does 2000 to 2060 TFLOP/s with
// this instruction and 1750 to 1800 with v_mfma_f32_32x32x16_bf16, on zeros both 2440.  Of a SIMD's time the matrix cores work 51 to 57 % at head
// size 128 and 35 to 43 at 64, the vector ALU 37 to 60 and 57 to 68.  Consecutive products share one operand (the order of
// the second index turns round with every step of the first), 2 % of the same loop.  With 32x32x16 products, two wavefronts per SIMD
// in the forward kernel and no fragments of the transposed operand ahead, forward / forward and backward, us, before and now:
//   4 x 2048, 32 heads of 128 158 / 685 -> 143 / 600    2 x 4096, 52 of 128 457 / 1935 -> 412 / 1745    8 x 1024, 12 of 64 22.9 / 95 -> 21 / 86
// Tiles go from global memory straight into LDS (buffer loads with the LDS bit; rows past the end of the sequence arrive as zeros), so
// a tile costs one barrier and neither staging registers nor LDS store instructions.  The tiles are unpadded; a permutation of the
// 16-byte chunks of every row, applied through the choice of the chunk each lane fetches, keeps both kinds of fragment reads free of
// bank conflicts.  All fragments run through small rings of registers a few fragments ahead of the products that use them.
// Statistics are fp32, exp2 with the 1/sqrt(dh) scale folded into the exponent; the causal mask is
// applied only on tiles that cross the diagonal; the backward pass recomputes P from the saved
// log-sum-exp; dQ and dK/dV come from workgroups of their own, so every sum has a fixed order and no atomics; no result depends on
// how many rows a wavefront owns.
#include <type_traits>

#include "../../include/teraio.h"
#include "device_common.h"
#include "kernels.h"
#include "mfma_tiles.h"

namespace tio {
namespace k {

namespace {

constexpr int NT = 256;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    union { bf16x2 h; uint32_t u; } c;
    c.h = __builtin_convertvector((f32x2){a, b}, bf16x2);
    return c.u;
}

// c += a . b, 16x16x32 (lane layouts: see the top of the file)
__device__ __forceinline__ void mma(floatx4 &c, const bf16x8 &a, const bf16x8 &b) { c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// B operand of a product over 32 rows from the accumulators of their two groups of 16 (slots 0..3 of lane group g: rows 4 g + 0..3, slots
// 4..7: rows 16 + 4 g + 0..3)
__device__ __forceinline__ bf16x8 pack8(const floatx4 &a, const floatx4 &b) {
    Frag f;
    f.u = make_uint4(pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3]));
    return f.v;
}
__device__ __forceinline__ floatx4 zero4() { return (floatx4){0.f, 0.f, 0.f, 0.f}; }
// a value combined over the four lane groups (lanes i, i + 16, i + 32, i + 48), the same in all of them: the swaps hand every lane the
// values of two groups without a trip through the LDS queue, behind which a cross-lane read would wait
__device__ __forceinline__ float sum_neighbours(float x) {         // lanes i and i ^ 16
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_halves(float x) {             // lanes i and i ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_groups(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
// Accumulators of columns 16 i .. + 15 (a) and 16 i + 16 .. + 31 (b) of a row to bf16 at p = row start + 16 i: a lane holds four columns
// of either and ends up with eight consecutive ones, so that a row's 32 columns are four stores of 16 bytes.
__device__ __forceinline__ void store32(uint16_t *p, const floatx4 &a, const floatx4 &b, float f, int group) {
    const auto lo = __builtin_amdgcn_permlane32_swap(pack2(a[0] * f, a[1] * f), pack2(b[0] * f, b[1] * f), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(pack2(a[2] * f, a[3] * f), pack2(b[2] * f, b[3] * f), false, false);
    const auto l2 = __builtin_amdgcn_permlane16_swap(lo[0], lo[1], false, false);
    const auto h2 = __builtin_amdgcn_permlane16_swap(hi[0], hi[1], false, false);
    *reinterpret_cast<uint4 *>(p + 8 * group) = make_uint4(l2[0], h2[0], l2[1], h2[1]);
}
// the lane index, computed where it stands: not kept in a register over a loop
__device__ __forceinline__ int lane_here() {
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}
__device__ __forceinline__ u32x4 buf_load(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
}
// an offset behind every descriptor here (fits() below keeps them under 2 GiB)
constexpr uint32_t PAST_ALL = 0x80000000u;
// descriptor over rows [0, Tn) of one head's slice: rows at or past Tn read as zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t head_rsrc(const uint16_t *base, int64_t Tn, int64_t ld, int dh) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)(((Tn - 1) * ld + dh) * 2), 0x00020000);
}
__device__ __forceinline__ bf16x8 buf_frag(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    union { u32x4 u; bf16x8 v; } f;
    f.u = buf_load(rsrc, off);
    return f.v;
}

// Workgroup -> (batch*head, block of rows).  Workgroups are dealt to the 8 XCDs round-robin and each XCD has its own L2, so all row
// blocks of one head are given to one XCD (head = 8*i + xcd): the K and V rows of a head are then fetched into one L2 only, and reused
// there by the head's other row blocks.  Under the causal mask a head's blocks differ in length by up to their number (block 0 is the
// longest), and consecutive workgroups of an XCD go to its 32 compute units in turn.  In the order (head, block) a unit therefore gets
// blocks of one length wherever the number of blocks divides 32: of 8 x 1024 tokens, 12 heads of 64, three of the longest (48 tiles; 27
// on average) or three of the shortest.  So an XCD's heads are taken `heads` at a time, and within them all blocks 0 come first, then
// all blocks 1: the longest first, the shorter ones where units become free.  Where all workgroups are resident from the start and none
// becomes free, every other row of 32 is turned round (`turn`), which pairs long with short.  Forward / backward us, order (head,
// block) / this: 8 x 1024, 12 heads of 64 31 / 23.5, 101 / 82; 4 x 2048, 32 of 128 181 / 170, 654 / 553; 1 x 4096, 32 of 64 125 / 82.5,
// 344 / 274; 2 x 4096, 52 of 128 484 / 473, 1649 / 1570.
struct Order {
    int heads;
    bool turn;
};
// Returns false for the padding workgroups when the head count is not a multiple of 8.
__device__ __forceinline__ bool head_and_block(unsigned block, int64_t n_heads, int n_blocks, Order order, int64_t &bh, int &blk) {
    const int xcd = (int)(block & 7), slot = (int)(block >> 3);
    const int of_xcd = (int)((n_heads + 7) / 8), first = slot / (order.heads * n_blocks) * order.heads;
    const int here = of_xcd - first < order.heads ? of_xcd - first : order.heads;
    int w = slot - first * n_blocks;
    if (order.turn && (w & 32) && (w | 31) < here * n_blocks) w ^= 31;
    bh = (int64_t)(first + w % here) * 8 + xcd;
    blk = w / here;
    return bh < n_heads;
}

// ------------------------------------------------------------------------------------------ tiles
// LDS tiles: [rows][DH] bf16 without padding, filled straight from global memory (no staging registers, no LDS store instructions); the
// 16-byte chunk c of row r sits at chunk c ^ swz(r).  A tile is read row-wise (lane group g takes chunk 4 ks + g of sixteen rows) and
// through transposing reads (two lane groups at a time take 32 bytes, an aligned pair of chunks, of each of eight consecutive rows); the
// permutation keeps both free of bank conflicts (the banks span 256 bytes).  Of a row-wise read sixteen lanes are served at a time, but
// not of one group: rows 0..3 and 12..15 of one with rows 4..11 of the next, whose chunk differs in its last bit.  So swz takes
// 16 different values over the sixteen rows (DH 64: eight, two rows per 256 bytes) and values that differ in the last bit stay within
// either set of rows ((r>>2) ^ (r>>3) beside r>>3), and the pairs of eight consecutive rows land on different pairs.  With the bits of
// r>>2 alone the row-wise reads took twice their time (SQ_LDS_BANK_CONFLICT; now 0).
template <int DH> __device__ __forceinline__ int swz(int r) {
    return (DH == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2) | ((((r >> 2) ^ (r >> 3)) & 1) << 1) | ((r >> 3) & 1);
}
// per-lane parts of the fragment addresses (element offsets into a tile), computed once per kernel: the XOR makes
// them non-additive in the contraction step, so each step has its own; with LEAN only the first step's is kept and a step's
// is one more XOR away (for the kernel that has no registers to spare)
template <int DH, bool LEAN = false> struct TileLanes {
    static constexpr int CPR = DH / 8, KS = DH / 32, DT = DH / 16;
    int roff[LEAN ? 1 : KS];          // row-wise fragment of contraction step ks: row lane%16, chunk 4 ks + lane/16
    int troff[LEAN ? 1 : DT];         // transposing fragment of column block i: rows 4 (lane/16) + (lane%16)/4 (and + 16), columns by lane
    __device__ __forceinline__ TileLanes(int lane) {
        const int l16 = lane & 15, g = lane >> 4, rl = 4 * g + (l16 >> 2);
#pragma unroll
        for (int ks = 0; ks < (LEAN ? 1 : KS); ++ks) roff[ks] = (l16 * CPR + ((ks * 4 + g) ^ swz<DH>(l16))) * 8;
#pragma unroll
        for (int i = 0; i < (LEAN ? 1 : DT); ++i) troff[i] = (rl * CPR + ((2 * i + ((lane & 3) >> 1)) ^ swz<DH>(rl))) * 8 + 4 * (lane & 1);
    }
    // rows row0 + lane%16 (row0 a multiple of 16), contraction step ks
    __device__ __forceinline__ bf16x8 row(const uint16_t *lds, int row0, int ks) const {
        Frag f;
        f.u = *reinterpret_cast<const uint4 *>(lds + row0 * DH + (LEAN ? roff[0] ^ (ks * 32) : roff[LEAN ? 0 : ks]));
        return f.v;
    }
    // "column 16 i + lane%16, contraction over rows r0 .. r0+31 in the slot order of pack8" (r0 a multiple of 16)
    __device__ __forceinline__ bf16x8 tr(const uint16_t *lds, int r0, int i) const {
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        union { s16x4 h[2]; bf16x8 v; } f;
        const uint16_t *p = lds + r0 * DH + (LEAN ? troff[0] ^ (16 * i) : troff[LEAN ? 0 : i]);
        f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
        f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 16 * DH));
        return f.v;
    }
};
// A [ROWS][DH] tile on its way from global memory into LDS: a wavefront-wide load fills 1 KiB of consecutive LDS bytes
// (lane i writes bytes 16 i ..), so which chunk a lane fetches decides where it lands: lane i of block b fetches, for
// row b*RPB + i/CPR, the logical chunk (i%CPR) ^ swz(row).  Rows past the sequence lie outside the descriptor and
// arrive as zeros.
template <int DH, int NW, int ROWS> struct DmaTile {
    static constexpr int CPR = DH / 8, RPB = 64 / CPR, BLOCKS = ROWS * DH * 2 / 1024, PER = BLOCKS / NW;
    static_assert(BLOCKS % NW == 0, "blocks divide over the wavefronts");
    static_assert((NW * RPB) % 16 == 0, "the permutation repeats from one load of a wavefront to its next");
    uint32_t voff, step;           // byte offset of this lane's chunk in the wavefront's first block; bytes between its blocks (uniform)
    __device__ __forceinline__ DmaTile(uint32_t ld_bytes, int wave, int lane) {
        const int row = wave * RPB + lane / CPR;
        voff = (uint32_t)row * ld_bytes + (uint32_t)(((lane % CPR) ^ swz<DH>(row & 15)) * 16);
        step = __builtin_amdgcn_readfirstlane((uint32_t)(NW * RPB) * ld_bytes);
    }
    // load i of the PER that make up this wavefront's share of a tile (soff = row0 * ld_bytes, uniform): rows
    // i * NW * RPB further down, which only moves the uniform part of the address (the scalar offset takes part
    // in the descriptor's range check like the per-lane one: checked on the hardware)
    __device__ __forceinline__ void load_one(int i, i32x4 rsrc, uint32_t soff, uint32_t lds_addr, int wave) const {
        load_to_lds_b128(rsrc, lds_addr + (uint32_t)(i * NW + wave) * 1024u, voff, soff + (uint32_t)i * step);
    }
    // rows row0 .. row0+ROWS-1 of the head behind rsrc to the tile at LDS address lds_addr
    __device__ __forceinline__ void load(i32x4 rsrc, uint32_t row0, uint32_t ld_bytes, uint32_t lds_addr, int wave) const {
        const uint32_t soff = __builtin_amdgcn_readfirstlane(row0 * ld_bytes);
#pragma unroll
        for (int i = 0; i < PER; ++i) load_one(i, rsrc, soff, lds_addr, wave);
    }
};

// ------------------------------------------------------------------------------------------ forward
// Tiles of 32 keys in a ring of three: loads are issued two tiles ahead, and a workgroup's 48 KiB (head size 128) and its registers
// leave room for three wavefronts per SIMD, where two tiles of 64 keys and a second set of scores allowed two.  A wavefront runs its own
// number of tiles in front of the diagonal, without mask and branch, so that no branch around a tile keeps a second copy of its
// accumulators alive.  4 x 2048 tokens, 32 heads of 128: 158 -> 151 us, 2 x 4096, 52 heads 470 -> 440 (before the change of the product).
// NG: groups of 16 query rows of a wavefront.
template <int DH, int NG>
__global__ void __launch_bounds__(NT, DH == 64 || NG == 1 ? 4 : 3) attn_fwd_mfma_k(const uint16_t *__restrict__ qkv, uint16_t *__restrict__ o,
                                                      float *__restrict__ lse, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    constexpr int KS = DH / 32, DT = DH / 16, TE = 32 * DH, RING = 4, ROWS = NT / 64 * 16 * NG;
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];    // ring of three pairs of tiles: 32 rows of K | 32 rows of V
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2);
    const int nblk = (int)((Tn + ROWS - 1) / ROWS);
    int64_t bh;
    int blk;
    if (!head_and_block(blockIdx.x, Bn * H, nblk, order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q0 = (nblk - 1 - blk) * ROWS;                               // longest rows first
    const int q0w = q0 + wave * 16 * NG;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const __amdgpu_buffer_rsrc_t rsQ = head_rsrc(qb, Tn, ld, DH);
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const i32x4 rsK = make_rsrc(qb + d, head_bytes), rsV = make_rsrc(qb + 2 * d, head_bytes);
    const float c = scale * LOG2E;
    const TileLanes<DH> L(lane);
    using Dma = DmaTile<DH, NT / 64, 32>;
    const Dma dma(ldb, wave, lane);
    constexpr int PER = Dma::PER;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    bf16x8 qf[NG][KS];                                  // of rows q0w + 16 u + lane%16
#pragma unroll
    for (int u = 0; u < NG; ++u)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[u][ks] = buf_frag(rsQ, (uint32_t)(q0w + 16 * u + l16) * ldb + (ks * 32 + grp * 8) * 2);
    floatx4 oacc[DT][NG];
    float m[NG], l[NG];                                 // reference exponent (log2 domain, scaled) and sum
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        m[u] = -INFINITY;
        l[u] = 0.f;
#pragma unroll
        for (int i = 0; i < DT; ++i) oacc[i][u] = zero4();
    }
    const int kv_end = q0 + ROWS < (int)Tn ? q0 + ROWS : (int)Tn;
    const int ntiles = (kv_end + 31) / 32;

    dma.load(rsK, 0, ldb, lds0, wave);
    dma.load(rsV, 0, ldb, lds0 + TE * 2, wave);
    dma.load(rsK, 32, ldb, lds0 + 2 * TE * 2, wave);
    dma.load(rsV, 32, ldb, lds0 + 3 * TE * 2, wave);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): this wavefront's part of tile 0 has landed (and Q, which the compiler knows of)
    __builtin_amdgcn_s_barrier();
    int slot = 0;                                       // of tile t in the ring
    // Tile t + 2 goes to the slot of tile t - 1, free since the barrier that ended it; past the last tile the loads lie outside the
    // descriptor and bring zeros that nobody reads.  They are issued one at a time between the score products: issued together
    // right after the barrier, the loads of all wavefronts of a compute unit queue up behind one another and every wavefront stalls.
    struct Next { uint32_t soff, to; };
    auto next_of = [&](int t) __attribute__((always_inline)) {
        return Next{(uint32_t)__builtin_amdgcn_readfirstlane(t + 2 < ntiles ? (uint32_t)(t + 2) * 32 * ldb : PAST_ALL),
                    lds0 + (uint32_t)(slot == 0 ? 2 : slot - 1) * 2 * TE * 2};
    };
    auto next_load = [&](int i, const Next &n) __attribute__((always_inline)) {         // PER loads of K, then as many of V
        if (i < PER) dma.load_one(i, rsK, n.soff, n.to, wave);
        else dma.load_one(i - PER, rsV, n.soff, n.to + TE * 2, wave);
    };
    auto end_of_tile = [&]() __attribute__((always_inline)) {
        slot = slot == 2 ? 0 : slot + 1;
        __builtin_amdgcn_s_waitcnt(0x0070 | 2 * PER);   // tile t+1 has landed, tile t+2 may be on its way; lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
    };
    // DIAG: the tile on the diagonal, which has key q0w
    auto tile = [&](int t, auto DIAG) __attribute__((always_inline)) {
        const uint16_t *Ks = smem + slot * 2 * TE, *Vs = Ks + TE;
        const Next next = next_of(t);
        floatx4 s[2][NG];                               // [keys 16 k ..][queries 16 u ..]
        {
            constexpr int N = 2 * KS;
            bf16x8 ring[RING];
            auto frag = [&](int f) { return L.row(Ks, (f & 1) * 16, f / 2); };
#pragma unroll
            for (int f = 0; f < RING; ++f) ring[f] = frag(f);
#pragma unroll
            for (int u = 0; u < NG; ++u) s[0][u] = s[1][u] = zero4();
#pragma unroll
            for (int f = 0; f < N; ++f) {
#pragma unroll
                for (int v = 0; v < NG; ++v) mma(s[f & 1][(f + v) % NG], ring[f % RING], qf[(f + v) % NG][f / 2]);
                if (f + RING < N) ring[f % RING] = frag(f + RING);
#pragma unroll
                for (int i = f * 2 * PER / N; i < (f + 1) * 2 * PER / N; ++i) next_load(i, next);
            }
            // pin the order: RING reads, then the products of a fragment and one read in turn, then the last products
            __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
            for (int f = 0; f < N - RING; ++f) {
                __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, NG * RING, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (DIAG()) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int u = 0; u < NG; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (16 * (k - u) + r > (NG == 1 ? q0w % 32 : 0) + l16 - 4 * grp) s[k][u][r] = -INFINITY;
        }
        // The reference exponent m only has to keep exp2(x - m) in range, it need not be the running maximum.  The
        // probabilities are first taken with the m at hand, and their sum tells whether that was good enough: only
        // when the sum of some lane of a group of 16 rows reaches 2^16 (or is not a number: m is still -inf in the first tile of a row,
        // where key 0 is visible to every row) is the row maximum of the tile computed, m raised to it, everything
        // accumulated so far rescaled and the tile redone.  After the first keys that is rare, and the common
        // path has no maximum, no exchange between the lane groups and no rescale in it.
        floatx4 p[2][NG];
        float psum[NG];
        auto probabilities = [&](int u) __attribute__((always_inline)) {
            psum[u] = 0.f;
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[k][u][r] = __builtin_amdgcn_exp2f(fmaf(s[k][u][r], c, -m[u]));
                    psum[u] += p[k][u][r];
                }
        };
#pragma unroll
        for (int u = 0; u < NG; ++u) probabilities(u);
        if (__any(!(psum[0] < 65536.0f) || !(psum[NG - 1] < 65536.0f))) {
#pragma unroll
            for (int u = 0; u < NG; ++u) {
                if (!__any(!(psum[u] < 65536.0f))) continue;       // by itself: the bits do not depend on the rows of a wavefront
                float tmax = -INFINITY;
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) tmax = fmaxf(tmax, s[k][u][r]);
                const float mn = fmaxf(m[u], max_groups(tmax) * c), corr = __builtin_amdgcn_exp2f(m[u] - mn);
                l[u] *= corr;
                m[u] = mn;
#pragma unroll
                for (int i = 0; i < DT; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) oacc[i][u][r] *= corr;
                probabilities(u);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 pk[NG];
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            l[u] += psum[u];
            pk[u] = pack8(p[0][u], p[1][u]);
        }
        // V fragment i: columns 16 i .. + 15 of the 32 keys; like the K fragments they run through a ring of register sets
        constexpr int VR = 4;
        bf16x8 vf[VR];
#pragma unroll
        for (int i = 0; i < VR; ++i) vf[i] = L.tr(Vs, 0, i);
#pragma unroll
        for (int i = 0; i < DT; ++i) {
#pragma unroll
            for (int v = 0; v < NG; ++v) mma(oacc[i][(i + v) % NG], vf[i % VR], pk[(i + v) % NG]);
            if (i + VR < DT) vf[i % VR] = L.tr(Vs, 0, i + VR);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * VR, 0);
#pragma unroll
        for (int i = 0; i < DT - VR; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NG * VR, 0);
        end_of_tile();
    };
    // A wavefront's tiles: those in front of its diagonal, without mask and branch, the one on it, and those that only later
    // wavefronts of the workgroup need, of which it loads its share.
    int t = 0;
    if (q0w < (int)Tn) {
        for (; t < q0w / 32; ++t) tile(t, std::false_type{});
        tile(t++, std::true_type{});
    }
    for (; t < ntiles; ++t) {
        const Next next = next_of(t);
#pragma unroll
        for (int i = 0; i < 2 * PER; ++i) next_load(i, next);
        end_of_tile();
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // no load may be on its way to LDS that this workgroup gives back
#pragma unroll
    for (int u = 0; u < NG; ++u) l[u] = sum_halves(sum_neighbours(l[u]));
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int q = q0w + 16 * u + l16;
        const float inv = 1.0f / l[u];
        uint16_t *orow = o + (b * Tn + q) * d + h * DH;
        // the lane groups exchange columns of a row, so they take part or not together
        if (q < Tn) {
#pragma unroll
            for (int i = 0; i < DT; i += 2) store32(orow + 16 * i, oacc[i][u], oacc[i + 1][u], inv, grp);
            if (grp == 0) lse[bh * Tn + q] = (m[u] + log2f(l[u])) * LN2;
        }
    }
}

// ------------------------------------------------------------------------------------------ dQ
// Sum of the products of eight elements, in order.
__device__ __forceinline__ float chunk_dot(const bf16x8 &g, const bf16x8 &o) {
    Frag a, b;
    a.v = g;
    b.v = o;
    const uint32_t x[4] = {a.u.x, a.u.y, a.u.z, a.u.w}, y[4] = {b.u.x, b.u.y, b.u.z, b.u.w};
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sum = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), sum);
        sum = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), sum);
    }
    return sum;
}
// Sum over the head dimension of two rows of which the four lane groups have the fragments, the same in all of them: in the order of
// attn_bwd_pre_k, whose bits these are (chains of eight elements, then pairs).
template <int KS> __device__ __forceinline__ float row_dot(const bf16x8 (&g)[KS], const bf16x8 (&o)[KS]) {
    float p[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) p[ks] = sum_halves(sum_neighbours(chunk_dot(g[ks], o[ks])));
#pragma unroll
    for (int o2 = 1; o2 < KS; o2 *= 2)
#pragma unroll
        for (int ks = 0; ks < KS; ks += 2 * o2) p[ks] += p[ks + o2];
    return p[0];
}

// Bound: the matrix cores and the vector ALU, which work for 57 and 48 % of the time at head size 128 (39 and 57 at 64) and for a fifth to a third
// of the products' time together, and power; the tiles in front of the diagonal run through a loop of their own, without mask and
// branch.  Three wavefronts per SIMD at head size 64, two at 128.  With fragments of the transposed K tile four ahead in registers, where
// the compiler read each right before its products, 4 x 2048 tokens, 32 heads of 128, forward and backward 634 -> 614 us (dK/dV too).
// O: nullptr, or the forward pass's output: delta is then computed here, from the rows of dO that are in registers anyway, and
// written for the dK/dV kernel, in place of a launch that reads both tensors (forward and backward 100.8 -> 97.2 us and 708 -> 687).
template <int DH, int NW, int NG>
__device__ __forceinline__ void dq_rows(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const uint16_t *__restrict__ O,
                                        const float *__restrict__ lse, float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn,
                                        int64_t Tn, int64_t H, float scale, Order order, unsigned block) {
    constexpr int KS = DH / 32, DT = DH / 16, TE = 64 * DH, RING = 4, TR = 4, ROWS = NW * 16 * NG;
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];    // [2 buffers][K tile | V tile] of 64 rows
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2);
    const int nblk = (int)((Tn + ROWS - 1) / ROWS);
    int64_t bh;
    int blk;
    if (!head_and_block(block, Bn * H, nblk, order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q0 = (nblk - 1 - blk) * ROWS;
    const int q0w = q0 + wave * 16 * NG;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const __amdgpu_buffer_rsrc_t rsQ = head_rsrc(qb, Tn, ld, DH);
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const i32x4 rsK = make_rsrc(qb + d, head_bytes), rsV = make_rsrc(qb + 2 * d, head_bytes);
    const __amdgpu_buffer_rsrc_t rsG = head_rsrc(dO + b * Tn * d + h * DH, Tn, d, DH);
    const float c = scale * LOG2E;
    const TileLanes<DH> L(lane);
    const DmaTile<DH, NW, 64> dma(ldb, wave, lane);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    bf16x8 qf[NG][KS], gf[NG][KS];                       // of rows q0w + 16 u + lane%16
    float lse2[NG], dl[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int q = q0w + 16 * u + l16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[u][ks] = buf_frag(rsQ, (uint32_t)q * ldb + (ks * 32 + grp * 8) * 2);
            gf[u][ks] = buf_frag(rsG, (uint32_t)q * (uint32_t)(d * 2) + (ks * 32 + grp * 8) * 2);
        }
        lse2[u] = q < Tn ? lse[bh * Tn + q] * LOG2E : 0.f;
        if (O) {
            const __amdgpu_buffer_rsrc_t rsO = head_rsrc(O + b * Tn * d + h * DH, Tn, d, DH);
            bf16x8 of[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) of[ks] = buf_frag(rsO, (uint32_t)q * (uint32_t)(d * 2) + (ks * 32 + grp * 8) * 2);
            dl[u] = row_dot<KS>(gf[u], of);
            if (q < Tn && grp == 0) delta[bh * Tn + q] = dl[u];
        } else {
            dl[u] = q < Tn ? delta[bh * Tn + q] : 0.f;
        }
    }
    floatx4 dq[DT][NG];
#pragma unroll
    for (int i = 0; i < DT; ++i) dq[i][0] = dq[i][NG - 1] = zero4();
    const int kv_end = q0 + ROWS < (int)Tn ? q0 + ROWS : (int)Tn;
    const int ntiles = (kv_end + 63) / 64;

    dma.load(rsK, 0, ldb, lds0, wave);
    dma.load(rsV, 0, ldb, lds0 + TE * 2, wave);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): this wavefront's part of tile 0 has landed
    __syncthreads();
    // DIAG: tiles that cross the diagonal of some row of this workgroup, the last ones; the others have no mask and no branch in them
    auto tile = [&](int t, auto DIAG) __attribute__((always_inline)) {
        const int j0 = t * 64;
        const uint16_t *Ks = smem + (t & 1) * 2 * TE, *Vs = Ks + TE;
        if (t + 1 < ntiles) {                           // the other buffer is free since the barrier that ended tile t-1
            const uint32_t nx = lds0 + (uint32_t)((t + 1) & 1) * 2 * TE * 2;
            dma.load(rsK, (uint32_t)j0 + 64, ldb, nx, wave);
            dma.load(rsV, (uint32_t)j0 + 64, ldb, nx + TE * 2, wave);
        }
        if (!DIAG() || j0 <= q0w + 16 * NG - 1) {
#pragma unroll
            for (int kb = 0; kb < 64; kb += 32) {           // 32 keys at a time: a second set of scores would take the registers of a wavefront
                floatx4 s[2][NG], dp[2][NG];                // [keys kb + 16 k ..][queries 16 u ..]
                {
                    // S = K.Q^T and dP = V.dO^T; the K and V fragments run RING ahead of their products
                    constexpr int N = 4 * KS;
                    bf16x8 ring[RING];
                    auto frag = [&](int f) { return L.row((f & 1) ? Vs : Ks, kb + ((f >> 1) & 1) * 16, f >> 2); };
#pragma unroll
                    for (int f = 0; f < RING; ++f) ring[f] = frag(f);
#pragma unroll
                    for (int u = 0; u < NG; ++u) s[0][u] = s[1][u] = dp[0][u] = dp[1][u] = zero4();
#pragma unroll
                    for (int f = 0; f < N; ++f) {
                        const int k = (f >> 1) & 1, ks = f >> 2;
#pragma unroll
                        for (int v = 0; v < NG; ++v) {
                            const int u = ((f >> 1) + v) % NG;
                            if (f & 1) mma(dp[k][u], ring[f % RING], gf[u][ks]);
                            else mma(s[k][u], ring[f % RING], qf[u][ks]);
                        }
                        if (f + RING < N) ring[f % RING] = frag(f + RING);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                    for (int f = 0; f < N - RING; ++f) {
                        __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, NG * RING, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int u = 0; u < NG; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float p = __builtin_amdgcn_exp2f(fmaf(s[k][u][r], c, -lse2[u]));
                            if (DIAG() && kb + 16 * k - 16 * u + r > q0w - j0 + l16 - 4 * grp) p = 0.0f;
                            s[k][u][r] = p * (dp[k][u][r] - dl[u]);          // the 1/sqrt(dh) factor is applied once, to the sums
                        }
                __builtin_amdgcn_sched_barrier(0);
                bf16x8 ds[NG], kf[TR];
#pragma unroll
                for (int u = 0; u < NG; ++u) ds[u] = pack8(s[0][u], s[1][u]);
                // the transposed K fragments run TR ahead of their products
#pragma unroll
                for (int i = 0; i < TR; ++i) kf[i] = L.tr(Ks, kb, i);
#pragma unroll
                for (int i = 0; i < DT; ++i) {
#pragma unroll
                    for (int v = 0; v < NG; ++v) mma(dq[i][(i + v) % NG], kf[i % TR], ds[(i + v) % NG]);
                    if (i + TR < DT) kf[i % TR] = L.tr(Ks, kb, i + TR);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, 2 * TR, 0);
#pragma unroll
                for (int i = 0; i < DT - TR; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, NG * TR, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): this wavefront's part of tile t+1 has landed
        __syncthreads();
    };
    int t = 0;
    for (; t < q0 / 64; ++t) tile(t, std::false_type{});
    for (; t < ntiles; ++t) tile(t, std::true_type{});
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int q = q0w + 16 * u + l16;
        if (q < Tn) {                                   // lane groups together: they exchange columns
            uint16_t *orow = dqkv + (b * Tn + q) * ld + h * DH;
#pragma unroll
            for (int i = 0; i < DT; i += 2) store32(orow + 16 * i, dq[i][u], dq[i + 1][u], scale, grp);
        }
    }
}

template <int DH>
__global__ void __launch_bounds__(NT, DH == 64 ? 3 : 2) attn_bwd_dq_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv,
                                                         const uint16_t *__restrict__ O, const float *__restrict__ lse, float *__restrict__ delta,
                                                         uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    dq_rows<DH, NT / 64, 2>(dO, qkv, O, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
}

// ------------------------------------------------------------------------------------------ dK, dV
// Both gradients in one launch: S and dP are computed once for the two of them, and the Q and dO tiles are loaded once.  The
// accumulators and K fragments of 32 key rows take 160 of the 256 registers that two wavefronts per SIMD allow at head size 128,
// so the V fragments are not kept in registers there but read from LDS (the workgroup's V rows, loaded once); to have room for
// them, and half the tile loads per product, a workgroup is eight wavefronts with 256 key rows.  Bound: latency between the
// products of two wavefronts per SIMD (three at head size 64), a third of their cycles, and power.  Nothing may spill: a reload from
// scratch in the loop waits for the tile loads in flight, and the wavefront with it keeps the others at the barrier.  So the offsets of the reads are one register and an
// exclusive or each at head size 128, each of two wavefronts fetches one of the statistics, and the lane index is computed where it is used.
// The tiles behind the diagonal run through a loop of their own, without mask and branch; at head size 64 a second loop gains nothing
// over a mask of two instructions.
// The same sum with a row spread over four neighbouring lanes, CH chunks of eight elements each, the same in all of them.
template <int CH> __device__ __forceinline__ float quad_dot(const bf16x8 (&g)[CH], const bf16x8 (&o)[CH]) {
    float p[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) p[c] = chunk_dot(g[c], o[c]);
#pragma unroll
    for (int o2 = 1; o2 < CH; o2 *= 2)
#pragma unroll
        for (int c = 0; c < CH; c += 2 * o2) p[c] += p[c + o2];
    auto add_from = [](float x, auto LANES) {
        return x + __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), LANES(), 0xf, 0xf, true));
    };
    const float pair = add_from(p[0], std::integral_constant<int, 0xB1>{});         // lanes 1 0 3 2
    return add_from(pair, std::integral_constant<int, 0x4E>{});                    // lanes 2 3 0 1
}
// V rows in LDS instead of registers (NG: groups of 16 key rows of a wavefront)
template <int DH, int NG> constexpr bool dkv_v_in_lds() { return DH == 128 && NG == 2; }
template <int DH> constexpr int dkv_waves() { return DH == 128 ? 8 : 4; }
template <int DH, int NW, int NG, bool DELTA>
__device__ __forceinline__ void dkv_rows(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const uint16_t *__restrict__ O,
                                         const float *__restrict__ lse, const float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H,
                                         float scale, Order order, unsigned block) {
    constexpr int KS = DH / 32, DT = DH / 16, TE = 64 * DH, RING = 4, TR = 4, KEYS = NW * 16 * NG;
    constexpr bool VLDS = dkv_v_in_lds<DH, NG>(), ONE_LOOP = DH == 64;
    constexpr int BUF = 2 * TE;                                          // Q tile | dO tile, filled as in the forward kernel
    // [2 buffers][Q | dO], [KEYS][DH] V rows if VLDS, then [2][64 lse | 64 delta] floats
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2), ldg = (uint32_t)(d * 2);
    int64_t bh;
    int blk;
    if (!head_and_block(block, Bn * H, (int)((Tn + KEYS - 1) / KEYS), order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int kv0 = blk * KEYS;                                           // earliest keys see the most queries: first
    const int kv0w = kv0 + wave * 16 * NG;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const __amdgpu_buffer_rsrc_t rsK = head_rsrc(qb + d, Tn, ld, DH), rsV = head_rsrc(qb + 2 * d, Tn, ld, DH);
    const i32x4 rsQ = make_rsrc(qb, head_bytes);
    const i32x4 rsG = make_rsrc(dO + b * Tn * d + h * DH, (uint32_t)(((Tn - 1) * d + DH) * 2));
    const float c = scale * LOG2E;
    const TileLanes<DH, VLDS> L(lane);
    const DmaTile<DH, NW, 64> dmaQ(ldb, wave, lane), dmaG(ldg, wave, lane);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    const uint16_t *Vs = smem + 2 * BUF;

    bf16x8 kf[NG][KS], vf[NG][VLDS ? 1 : KS];             // of keys kv0w + 16 k + lane%16
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t at = (uint32_t)(kv0w + 16 * k + l16) * ldb + (ks * 32 + grp * 8) * 2;
            kf[k][ks] = buf_frag(rsK, at);
            if (!VLDS) vf[k][VLDS ? 0 : ks] = buf_frag(rsV, at);
        }
    if (VLDS) {
        const i32x4 rs = make_rsrc(qb + 2 * d, head_bytes);
#pragma unroll
        for (int i = 0; i < KEYS / 64; ++i) dmaQ.load(rs, (uint32_t)(kv0 + 64 * i), ldb, lds0 + (2 * BUF + i * TE) * 2, wave);
    }
    floatx4 dk[DT][NG], dv[DT][NG];
#pragma unroll
    for (int i = 0; i < DT; ++i) dk[i][0] = dk[i][NG - 1] = dv[i][0] = dv[i][NG - 1] = zero4();
    const int ntiles = ((int)Tn - kv0 + 63) / 64;

    // Statistics of row i0 + lane, one tile ahead, log-sum-exp in wavefront 0 and delta in wavefront 1: through descriptors of the head's
    // rows (rows past the sequence read zero; no addresses to keep in registers), used only where they go to LDS, a tile after their fetch.
    // DELTA: four lanes to a row fetch its dO and O instead and multiply them.
    const __amdgpu_buffer_rsrc_t rsS = buffer_over((DELTA || wave == 0 ? lse : delta) + bh * Tn, (uint32_t)Tn * 4);
    const float to_lds = DELTA || wave == 0 ? LOG2E : 1.f;
    constexpr int STATS = DELTA ? 1 : 2, CH = DH / 32;                    // wavefronts that fetch statistics; chunks of a row to a lane
    static_assert(!DELTA || NW == 4, "four lanes to each of 64 rows");
    float st = 0.f;
    bf16x8 go[DELTA ? CH : 1], oo[DELTA ? CH : 1];
    const __amdgpu_buffer_rsrc_t rsD = head_rsrc(dO + b * Tn * d + h * DH, Tn, d, DH), rsO = head_rsrc((DELTA ? O : dO) + b * Tn * d + h * DH, Tn, d, DH);
    float *stats = reinterpret_cast<float *>(smem + 2 * BUF + (VLDS ? KEYS * DH : 0));
    auto load_stats = [&](int i0) {
        if (wave < STATS) st = buffer_load4(rsS, (uint32_t)(i0 + lane_here()) * 4);
        if (DELTA) {
            const int ln = lane_here();
            const uint32_t at = (uint32_t)(i0 + wave * 16 + (ln >> 2)) * ldg + (ln & 3) * CH * 16;
#pragma unroll
            for (int c = 0; c < (DELTA ? CH : 0); ++c) {
                go[c] = buf_frag(rsD, at + c * 16);
                oo[c] = buf_frag(rsO, at + c * 16);
            }
        }
    };
    auto store_stats = [&](int buf) {
        if (wave < STATS) stats[buf * 128 + wave * 64 + lane_here()] = st * to_lds;
        if (DELTA) {
            const float sum = quad_dot<DELTA ? CH : 1>(go, oo);
            const int ln = lane_here();
            if ((ln & 3) == 0) stats[buf * 128 + 64 + wave * 16 + (ln >> 2)] = sum;
        }
    };
    auto load_tile = [&](int i0, int buf) {
        const uint32_t at = lds0 + (uint32_t)buf * BUF * 2;
        dmaQ.load(rsQ, (uint32_t)i0, ldb, at, wave);
        dmaG.load(rsG, (uint32_t)i0, ldg, at + TE * 2, wave);
    };
    load_tile(kv0, 0);
    load_stats(kv0);
    store_stats(0);
    if (ntiles > 1) load_stats(kv0 + 64);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): this wavefront's part of tile 0 (and of V) has landed
    __syncthreads();
    // DIAG: tiles that cross the diagonal of some key of this workgroup, the first ones; the others have no mask and no branch in them
    // (ONE_LOOP: every tile is taken for one).  END: the last tile where the sequence ends inside it, in code of its own.  Its rows past the
    // sequence are masked too: their Q, dO and statistics are zero, which adds nothing while K is finite, but with an infinite component
    // of a key their scores are not numbers.
    using Plain = std::integral_constant<int, 0>;
    using Diag = std::integral_constant<int, 1>;
    using End = std::integral_constant<int, 2>;
    auto key_less_4group = []() __attribute__((always_inline)) { const int ln = lane_here(); return (ln & 15) - 4 * (ln >> 4); };
    auto tile = [&](int t, auto KIND) __attribute__((always_inline)) {
        constexpr bool DIAG = KIND() == Diag(), END = KIND() == End();
        const int i0 = kv0 + t * 64;
        const uint16_t *Qs = smem + (t & 1) * BUF, *Gs = Qs + TE;
        const float *L2s = stats + (t & 1) * 128, *Ds = L2s + 64;
        if (!END && t + 1 < ntiles) {                           // the other buffer is free since the barrier that ended tile t-1
            // The statistics fetched a tile ago go to LDS before the tile loads are issued: the write waits for every
            // outstanding vector memory operation of the wavefront, and behind the tile loads that would be their
            // whole latency, at the start of every tile.
            store_stats((t + 1) & 1);
            load_tile(i0 + 64, (t + 1) & 1);
            if (t + 2 < ntiles) load_stats(i0 + 128);
        }
        if (KIND() == Plain() || i0 + 63 >= kv0w) {
            const int masked = DIAG ? kv0w - i0 + key_less_4group() : 0;       // rows of the tile before this lane's first key, less 4 grp
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                floatx4 s[2][NG], dp[2][NG];             // [rows 16 u ..][keys 16 k ..]
                {
                    // S^T = Q.K^T, then dP^T = dO.V^T; the Q and dO fragments run RING ahead of their products, V's two ahead
                    constexpr int N = 4 * KS;
                    bf16x8 ring[RING], vr[2];
                    auto frag = [&](int f) { return L.row(f < 2 * KS ? Qs : Gs, qt * 32 + (f & 1) * 16, (f >> 1) % KS); };
                    auto vfrag = [&](int f) { return L.row(Vs, wave * 16 * NG + (f & 1) * 16, (f >> 1) % KS); };
#pragma unroll
                    for (int f = 0; f < RING; ++f) ring[f] = frag(f);
#pragma unroll
                    for (int u = 0; u < 2; ++u) s[u][0] = s[u][NG - 1] = dp[u][0] = dp[u][NG - 1] = zero4();
#pragma unroll
                    for (int f = 0; f < N; ++f) {
                        const int u = f & 1, ks = (f >> 1) % KS;
#pragma unroll
                        for (int v = 0; v < NG; ++v) {
                            const int k = (f + v) % NG;
                            if (f < 2 * KS) mma(s[u][k], ring[f % RING], kf[k][ks]);
                            else mma(dp[u][k], ring[f % RING], VLDS ? vr[k] : vf[k][VLDS ? 0 : ks]);
                        }
                        if (f + RING < N) ring[f % RING] = frag(f + RING);
                        // V's fragments of the next contraction step, each behind the product that used the last of its predecessor
                        if (VLDS && f + 2 >= 2 * KS && f + 2 < N) {
                            if (f < 2 * KS) vr[f & 1] = vfrag(f + 2);
                            else if (f & 1) { vr[0] = vfrag(f + 1); vr[1] = vfrag(f + 2); }
                        }
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                    for (int f = 0; f < N; ++f) {
                        __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
                        const int reads = (f + RING < N ? 1 : 0) + (VLDS && f + 2 >= 2 * KS && f + 2 < N ? f < 2 * KS ? 1 : 2 * (f & 1) : 0);
                        if (reads == 3) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                        else if (reads == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        else if (reads == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    // rows 16 u + 4 grp + 0..3 of this 32-row group: their statistics are 16 contiguous bytes
                    const int group4 = 4 * (END ? lane_here() >> 4 : grp), ql = qt * 32 + 16 * u + group4;
                    const float4 l4 = *reinterpret_cast<const float4 *>(L2s + ql), d4 = *reinterpret_cast<const float4 *>(Ds + ql);
                    const int first = END ? kv0w - i0 + key_less_4group() : 0, end = (int)Tn - i0 - group4;
                    const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dvv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int k = 0; k < NG; ++k)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int row = qt * 32 + 16 * u + r;
                            float p = __builtin_amdgcn_exp2f(fmaf(s[u][k][r], c, -lv[r]));
                            if (DIAG && row - 16 * k < masked) p = 0.0f;
                            if (END && (row - 16 * k < first || row >= end)) p = 0.0f;
                            dp[u][k][r] = p * (dp[u][k][r] - dvv[r]);        // the 1/sqrt(dh) factor is applied once, to the sums
                            s[u][k][r] = p;
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
                const bf16x8 pf[2] = {pack8(s[0][0], s[1][0]), pack8(s[0][NG - 1], s[1][NG - 1])};
                const bf16x8 ds[2] = {pack8(dp[0][0], dp[1][0]), pack8(dp[0][NG - 1], dp[1][NG - 1])};
                // dV += dO^T.P, then dK += Q^T.dS; the transposed fragments run TR ahead of their products
                auto trf = [&](int f) { return L.tr(f < DT ? Gs : Qs, qt * 32, f % DT); };
                bf16x8 fr[TR];
#pragma unroll
                for (int f = 0; f < TR; ++f) fr[f] = trf(f);
#pragma unroll
                for (int f = 0; f < 2 * DT; ++f) {
#pragma unroll
                    for (int v = 0; v < NG; ++v) {
                        const int k = (f + v) % NG;
                        if (f < DT) mma(dv[f][k], fr[f % TR], pf[k]);
                        else mma(dk[f - DT][k], fr[f % TR], ds[k]);
                    }
                    if (f + TR < 2 * DT) fr[f % TR] = trf(f + TR);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, 2 * TR, 0);
#pragma unroll
                for (int f = 0; f < 2 * DT - TR; ++f) {
                    __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, NG * TR, 0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): this wavefront's part of tile t+1 has landed
        __syncthreads();
    };
    const int whole = ((int)Tn - kv0) / 64, diag = ONE_LOOP || whole < KEYS / 64 ? whole : KEYS / 64;
    int t = 0;
    for (; t < diag; ++t) tile(t, Diag());
    if constexpr (!ONE_LOOP)
        for (; t < whole; ++t) tile(t, Plain());
    if (t < ntiles) tile(t, End());
    const int last = lane_here();
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const int key = kv0w + 16 * k + (last & 15);
        if (key < (int)Tn) {                            // lane groups together: they exchange columns
            uint16_t *krow = dqkv + (b * Tn + key) * ld + d + h * DH;
#pragma unroll
            for (int i = 0; i < DT; i += 2) {
                store32(krow + 16 * i, dk[i][k], dk[i + 1][k], scale, last >> 4);
                store32(krow + d + 16 * i, dv[i][k], dv[i + 1][k], 1.0f, last >> 4);
            }
        }
    }
}

template <int DH>
__global__ void __launch_bounds__(dkv_waves<DH>() * 64, DH == 64 ? 3 : 2)
    attn_bwd_dkv_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const float *__restrict__ lse,
                        const float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    dkv_rows<DH, dkv_waves<DH>(), 2, false>(dO, qkv, nullptr, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
}

// Both kernels' blocks in one launch, those of key rows first: for sequences whose blocks leave the chip room, where each of the two
// kernels lasts as long as its longest chain of tiles.  The same rows to a block on either side; every output has the bits of the two
// launches.  Delta comes from a launch of its own, or (DELTA) both kinds of blocks multiply dO and O themselves: the blocks of query rows
// theirs, which they write, and those of key rows all that they meet, a tile ahead.
template <int DH, int NW, int NG, bool DELTA>
__global__ void __launch_bounds__(NW * 64, NG == 1 ? 2 : DH == 64 ? 3 : 2)
    attn_bwd_both_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const uint16_t *__restrict__ O, const float *__restrict__ lse,
                         float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order,
                         unsigned blocks) {
    if (blockIdx.x < blocks) dkv_rows<DH, NW, NG, DELTA>(dO, qkv, O, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
    else dq_rows<DH, NW, NG>(dO, qkv, DELTA ? O : nullptr, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x - blocks);
}

template <int DH> constexpr size_t fwd_smem() { return (size_t)3 * 2 * 32 * DH * 2; }      // three pairs of tiles
template <int DH> constexpr size_t kv_smem() { return (size_t)2 * 2 * 64 * DH * 2; }       // two buffers of two tiles
template <int DH, int NW, int NG> constexpr size_t dkv_smem() {         // tiles, V rows, then statistics
    return (size_t)2 * 2 * 64 * DH * 2 + (dkv_v_in_lds<DH, NG>() ? (size_t)NW * 16 * NG * DH * 2 : 0) + 2 * 128 * 4;
}

// Unsigned 32-bit buffer offsets: one head's rows, and PAST more, span less than 2 GiB.  A block's rows past the sequence (up to
// its size less one) are addressed too and refused by the descriptor, so their offsets must not wrap around 4 GiB: as many rows as
// twice PAST keep Tn + rows below twice Tn + PAST.
constexpr int64_t PAST = 192;
static_assert(dkv_waves<64>() * 32 <= 2 * PAST && dkv_waves<128>() * 32 <= 2 * PAST && 128 <= 2 * PAST, "offsets past the sequence do not wrap");
bool fits(int64_t Tn, int64_t H, int64_t dh) { return (Tn + PAST) * 3 * H * dh * 2 < ((int64_t)1 << 31); }

// The order and the grid of a kernel whose workgroups take `rows` rows each and of which a compute unit holds per_cu.  Heads taken
// together: all of them where that leaves nothing to wait for a free unit, otherwise as many as have 16 MiB of K and V (or Q and dO), so
// that an XCD's 4 MiB L2 sees most of a tile's reuse by the other blocks (4 x 2048, 32 heads of 128, 2 / 4 / 8 / 16 heads, forward: 176 /
// 169 / 167 / 171 us; 2 x 4096, 52 heads 486 / 487 / 473 / 483).
struct Launch {
    dim3 grid;
    Order order;
    Launch(int64_t n_heads, int64_t Tn, int64_t dh, int rows, int per_cu) {
        const int64_t of_xcd = (n_heads + 7) / 8, blocks = (Tn + rows - 1) / rows, by_bytes = ((int64_t)16 << 20) / (Tn * dh * 4);
        grid = dim3((unsigned)(blocks * of_xcd * 8));
        order.turn = of_xcd * blocks <= 32 * per_cu;
        order.heads = (int)(order.turn || by_bytes >= of_xcd ? of_xcd : by_bytes > 1 ? by_bytes : 1);
    }
};

}  // namespace

bool attn_mfma_supported(int dtype, int64_t Tn, int64_t H, int64_t dh) {
    return dtype == TIO_PREC_BF16 && (dh == 64 || dh == 128) && fits(Tn, H, dh);
}

void attn_fwd_mfma(hipStream_t s, const void *qkv, void *o, float *lse, int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    const float scale = 1.0f / sqrtf((float)dh);
#define TIO_ATTN_FWD(DH, NG)                                                                                                                   \
    {                                                                                                                                          \
        const Launch l(B * H, Tn, DH, NT / 64 * 16 * NG, DH == 64 ? 4 : 3);                                                                    \
        attn_fwd_mfma_k<DH, NG><<<l.grid, NT, fwd_smem<DH>(), s>>>((const uint16_t *)qkv, (uint16_t *)o, lse, B, Tn, H, scale, l.order);       \
    }
    // Sixteen rows to a wavefront while the chip holds about all workgroups of 64 rows at once: half the work in a tile, where the chain
    // of a wavefront's tiles is what counts; more of them would load K and V twice as often.  us, 32 / 16 rows (workgroups of 64, the heads
    // rounded up to the XCDs: one with a head more than the others decides).  At head size 128 the line is where all of them are resident, four to
    // a unit, for long sequences: with as many workgroups of fewer heads, the longest chain of tiles is more of the launch, and half the work in
    // its tiles counts for more than twice the loads; for short ones it is lower.
    //   heads of 64:  8 x  192,  7  5.6 /  5.0 (168)    1 x 4096,  9 54.5 / 44.1 (1024)   3 x 2000, 13 29.9 / 29.7 (1280)
    //                 2 x 2048, 20 34.4 / 33.0 (1280)   4 x 3904,  5 57.8 / 59.3 (1464)   8 x 1024, 12 21.2 / 22.2 (1536)
    //   of 128:       4 x  333,  6 10.3 /  7.8 (144)    1 x 2048,  8 39.8 / 28.5 (256)    7 x  868,  8 23.3 / 19.6 (784)
    //                 8 x  256, 26 13.5 / 15.1 (832)    4 x 1024, 16 27.2 / 29.0 (1024)   1 x 4000,  9 72.7 / 65.1 (1008)
    const bool one = Launch(B * H, Tn, dh, 64, 1).grid.x <= (dh == 64 ? 1280 : Tn < 2048 ? 800 : 1024);
    if (dh == 64) {
        if (one) TIO_ATTN_FWD(64, 1) else TIO_ATTN_FWD(64, 2)
    } else {
        if (one) TIO_ATTN_FWD(128, 1) else TIO_ATTN_FWD(128, 2)
    }
#undef TIO_ATTN_FWD
}

void attn_bwd_mfma(hipStream_t s, const void *dO, const void *qkv, const void *O, const float *lse, float *delta, void *dqkv,
                   int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    const float scale = 1.0f / sqrtf((float)dh);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)attn_bwd_dq_mfma_k<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kv_smem<128>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_dkv_mfma_k<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, dkv_waves<128>(), 2>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_both_mfma_k<128, 8, 2, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, 8, 2>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_both_mfma_k<128, 4, 1, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, 4, 1>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_both_mfma_k<128, 4, 1, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, 4, 1>());
        attr_set = true;
    }
    // One launch for both gradients while its workgroups are at most a little more than the chip holds at once, with 16 rows to a
    // wavefront as in the forward pass while it holds about twice the workgroups of 64 rows (and up to 256 rows of a sequence nearly twice as
    // many of them: a block of 128 or 256 rows is a whole sequence or half of one there, most of whose products the mask throws away).
    // Forward and backward, us (workgroups of 64 rows on either side):
    //   32 rows, as in the launches below them / 16 rows
    //     heads of 64:  5 x 145, 22 19.1 / 16.1 (330)    8 x 512, 12 38.9 / 34.2 (768)    1 x 4096, 8 150 / 120 (512)    8 x 300, 20 34.4 / 30.7 (800)
    //                   8 x 256, 52 59.0 / 56.0 (1664)   6 x 512, 24 52.1 / 53.0 (1152)   8 x 1024, 8 64.1 / 66.1 (1024)
    //     of 128:       4 x 333,  6 32.9 / 24.6 (144)    1 x 2048, 8 112 / 83 (256)       3 x 700, 25 80.6 / 77.6 (880)    4 x 512, 16 53.1 / 44.5 (512)
    //                   8 x 256, 40 87.2 / 85.7 (1280)   8 x 512, 16 78.4 / 84.0 (1024)   1 x 4096, 16 311 / 335 (1024)
    //   32 rows, two launches / one
    //     heads of 64:  1 x 4096, 16 203 / 182           8 x 1024, 8 62.4 / 57.9          4 x 500, 31 41.1 / 39.5
    //     of 128:       4 x 1024, 16 112 / 104           1 x 4096, 16 362 / 304           2 x 2000, 15 191 / 165
    // Delta inside that launch while the tiles are few: the products are done over by every block of keys, the launch they replace
    // takes 3 us and two more between launches.  us, a launch of its own / inside: 5 x 145, 22 heads of 64 16.3 / 13.6, 8 x 512, 12 37.9 / 35.0,
    // 1 x 1024, 12 35.8 / 35.1, 1 x 4096, 8 123 / 131; 4 x 100, 6 heads of 128 14.9 / 12.8, 4 x 512, 16 47.5 / 44.8, 1 x 1024, 5 42.5 / 45.9.
    constexpr int64_t OWN_DELTA = 65536;                  // sequence length times head size
#define TIO_ATTN_BOTH_AS(DH, NW, NG, DELTA)                                                                                                    \
    attn_bwd_both_mfma_k<DH, NW, NG, DELTA><<<2 * l.grid.x, NW * 64, dkv_smem<DH, NW, NG>(), s>>>(                                             \
        (const uint16_t *)dO, (const uint16_t *)qkv, (const uint16_t *)O, lse, delta, (uint16_t *)dqkv, B, Tn, H, scale, l.order, l.grid.x)
#define TIO_ATTN_BOTH(DH, NW, NG, WORKGROUPS)                                                                                                  \
    {                                                                                                                                          \
        const Launch l(B * H, Tn, DH, NW * 16 * NG, NG == 1 ? 2 : DH == 64 ? 3 : 1);                                                           \
        if (2 * (int64_t)l.grid.x <= WORKGROUPS) {                                                                                             \
            if (NG == 1 && O && Tn * DH <= OWN_DELTA) {                                                                                        \
                TIO_ATTN_BOTH_AS(DH, NW, NG, (NG == 1));                                                                                       \
                return;                                                                                                                        \
            }                                                                                                                                  \
            if (O) attn_bwd_pre(s, TIO_PREC_BF16, dO, O, delta, B, Tn, H, DH);                                                                 \
            TIO_ATTN_BOTH_AS(DH, NW, NG, false);                                                                                               \
            return;                                                                                                                            \
        }                                                                                                                                      \
    }
#define TIO_ATTN_BWD(DH, DQ_PER_CU, DKV_PER_CU)                                                                                                \
    {                                                                                                                                          \
        const Launch q(B * H, Tn, DH, 128, DQ_PER_CU), kv(B * H, Tn, DH, dkv_waves<DH>() * 32, DKV_PER_CU);                                    \
        attn_bwd_dq_mfma_k<DH><<<q.grid, NT, kv_smem<DH>(), s>>>((const uint16_t *)dO, (const uint16_t *)qkv, (const uint16_t *)O, lse, delta, \
                                                                 (uint16_t *)dqkv, B, Tn, H, scale, q.order);                                  \
        attn_bwd_dkv_mfma_k<DH><<<kv.grid, dkv_waves<DH>() * 64, dkv_smem<DH, dkv_waves<DH>(), 2>(), s>>>(                                        \
            (const uint16_t *)dO, (const uint16_t *)qkv, lse, delta, (uint16_t *)dqkv, B, Tn, H, scale, kv.order);                             \
    }
    if (dh == 64) {
        TIO_ATTN_BOTH(64, 4, 1, 2 * (Tn <= 256 ? 1664 : 896))
        TIO_ATTN_BOTH(64, 4, 2, 1024)
        TIO_ATTN_BWD(64, 3, 3)
    } else {
        TIO_ATTN_BOTH(128, 4, 1, 2 * (Tn <= 256 ? 1664 : 896))
        TIO_ATTN_BOTH(128, 8, 2, 512)
        TIO_ATTN_BWD(128, 2, 1)
    }
#undef TIO_ATTN_BOTH
#undef TIO_ATTN_BOTH_AS
#undef TIO_ATTN_BWD
}

}  // namespace k
}  // namespace tio
