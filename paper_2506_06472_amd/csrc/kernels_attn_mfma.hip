// Causal self-attention on the matrix cores (bf16, head dimension 64 or 128), forward and backward,
// on the packed [S, 3d] q|k|v layout.
//
// Each wavefront owns 32 query rows (forward, dQ) or 32 key rows (dK/dV) and keeps their operand
// fragments in registers for the whole kernel; the other side streams through LDS in row-major tiles of
// 64 rows.  Scores are produced transposed (keys x queries in the forward and dQ kernels, queries x keys
// in the dK/dV kernel) so that in the accumulator layout of v_mfma_f32_32x32x16_bf16 the row owned by the
// wavefront is the lane index: the softmax statistics of a row live in one lane (plus one exchange with
// lane+32), and the probabilities can be fed to the second product straight from registers as its B
// operand.  The operand whose contraction index is the sequence position (V in P.V, K in dS.K, Q and dO
// in the dK/dV products) is read from the same row-major tile with the transposing LDS read
// (ds_read_b64_tr_b16), in the slot order the accumulator registers dictate: no transposed copies.
// Tiles go from global memory straight into the other half of a double LDS buffer one tile ahead (buffer
// loads with the LDS bit; rows past the end of the sequence arrive as zeros), so a tile costs one barrier and
// neither staging registers nor LDS store instructions.  The tiles are unpadded; a permutation of the 16-byte
// chunks of every row, applied through the choice of the chunk each lane fetches, keeps both kinds of
// fragment reads free of bank conflicts.  The fragments of the first products of a tile run through a small
// ring of registers a few fragments ahead of the products that use them.
// Statistics are fp32, exp2 with the 1/sqrt(dh) scale folded into the exponent; the causal mask is
// applied only on tiles that cross the diagonal; the backward pass recomputes P from the saved
// log-sum-exp; dQ and dK/dV come from workgroups of their own, so every sum has a fixed order and no atomics.
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
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    union { bf16x2 h; uint32_t u; } c;
    c.h = __builtin_convertvector((f32x2){a, b}, bf16x2);
    return c.u;
}

// B operand of a 16-deep product from accumulator registers R0..R0+7 (the contraction index is the
// accumulator's row index: slots 0..3 = rows base+4*lhi+0..3, slots 4..7 = rows base+8+4*lhi+0..3)
template <int R0> __device__ __forceinline__ bf16x8 pack8(const floatx16 &v) {
    Frag f;
    f.u = make_uint4(pack2(v[R0], v[R0 + 1]), pack2(v[R0 + 2], v[R0 + 3]), pack2(v[R0 + 4], v[R0 + 5]), pack2(v[R0 + 6], v[R0 + 7]));
    return f.v;
}
__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}
// a value combined over the two halves of the wavefront (lanes i and i + 32), the same in both: v_permlane32_swap hands
// every lane the value of both halves without a trip through the LDS queue, behind which a cross-lane read would wait
__device__ __forceinline__ float max_halves(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// the lane index, computed where it stands: not kept in a register over a loop
__device__ __forceinline__ int lane_here() {
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}
// row index inside a 32x32 accumulator tile of register r for lane half lhi
__device__ __forceinline__ int acc_row(int r, int lhi) { return 8 * (r >> 2) + 4 * lhi + (r & 3); }

__device__ __forceinline__ u32x4 buf_load(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
}
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

// ------------------------------------------------------------------------------------------ forward
// LDS tiles of the forward kernel: [64 rows][DH] bf16 without padding, filled straight from global memory (no
// staging registers, no LDS store instructions); the 16-byte chunk c of row r sits at chunk c ^ swz(r).  K is read
// row-wise (16-byte fragments of 16 consecutive rows at one logical chunk) and V through transposing reads (32 lanes
// take 64 bytes, an aligned quad of chunks, of each of four consecutive rows); the permutation keeps both free of bank
// conflicts (the banks span 256 bytes): over the rows that share banks swz takes 16 (DH 128) or 8 (DH 64, two rows per
// 256 bytes) different values, and the quads of four consecutive rows land on different quads (DH 128:
// swz = (r%4)*4 + (r/4)%4) or on two quads in each half of the banks (DH 64: swz = ((r/2)%2)*4 + (r/4)%4).
template <int DH> __device__ __forceinline__ int swz(int r) {
    return DH == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
}
// per-lane parts of the fragment addresses (element offsets into a tile), computed once per kernel: the XOR makes
// them non-additive in the contraction step, so each step has its own; with LEAN only the first step's is kept and a step's
// is one more XOR away (for the kernel that has no registers to spare)
template <int DH, bool LEAN = false> struct TileLanes {
    static constexpr int CPR = DH / 8, KS = DH / 16, DT = DH / 32;
    int roff[LEAN ? 1 : KS];          // row-wise fragment of contraction step ks: row lane%32, chunk 2 ks + lane/32
    int troff[LEAN ? 1 : DT][LEAN ? 1 : 2];      // transposing fragment of column block i: rows 4 (lane/32) + (lane%16)/4 (+ 8), columns by lane
    __device__ __forceinline__ TileLanes(int lane) {
        const int l32 = lane & 31, lhi = lane >> 5;
#pragma unroll
        for (int ks = 0; ks < (LEAN ? 1 : KS); ++ks) roff[ks] = (l32 * CPR + ((ks * 2 + lhi) ^ swz<DH>(l32 & 15))) * 8;
#pragma unroll
        for (int i = 0; i < (LEAN ? 1 : DT); ++i)
#pragma unroll
            for (int h = 0; h < (LEAN ? 1 : 2); ++h) {
                const int rl = 4 * lhi + ((lane & 15) >> 2) + 8 * h;
                const int chunk = 4 * i + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
                troff[i][h] = (rl * CPR + (chunk ^ swz<DH>(rl))) * 8 + 4 * (lane & 1);
            }
    }
    // A operand, rows row0 + lane%32 (row0 a multiple of 16), contraction step ks
    __device__ __forceinline__ bf16x8 row(const uint16_t *lds, int row0, int ks) const {
        Frag f;
        f.u = *reinterpret_cast<const uint4 *>(lds + row0 * DH + (LEAN ? roff[0] ^ (ks * 16) : roff[LEAN ? 0 : ks]));
        return f.v;
    }
    // A operand "column 32 i + lane%32, contraction over rows r0 .. r0+15 in the slot order of pack8" (r0 a multiple of 16)
    __device__ __forceinline__ bf16x8 tr(const uint16_t *lds, int r0, int i) const {
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        union { s16x4 h[2]; bf16x8 v; } f;
        // LEAN (head size 128): column block i moves bits 2 and 3 of the chunk index, eight rows further down bit 1
        f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lds + r0 * DH + (LEAN ? troff[0][0] ^ (32 * i) : troff[LEAN ? 0 : i][0])));
        f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4 *)(lds + r0 * DH + (LEAN ? (troff[0][0] ^ (32 * i + 16)) + 8 * DH : troff[LEAN ? 0 : i][LEAN ? 0 : 1])));
        return f.v;
    }
};
// A [64][DH] tile on its way from global memory into LDS: a wavefront-wide load fills 1 KiB of consecutive LDS bytes
// (lane i writes bytes 16 i ..), so which chunk a lane fetches decides where it lands: lane i of block b fetches, for
// row b*RPB + i/CPR, the logical chunk (i%CPR) ^ swz(row).  Rows past the sequence lie outside the descriptor and
// arrive as zeros.
template <int DH, int NW = NT / 64> struct DmaTile {
    static constexpr int CPR = DH / 8, RPB = 64 / CPR, BLOCKS = 64 * DH * 2 / 1024, PER = BLOCKS / NW;
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
    // rows row0 .. row0+63 of the head behind rsrc to the tile at LDS address lds_addr
    __device__ __forceinline__ void load(i32x4 rsrc, uint32_t row0, uint32_t ld_bytes, uint32_t lds_addr, int wave) const {
        const uint32_t soff = __builtin_amdgcn_readfirstlane(row0 * ld_bytes);
#pragma unroll
        for (int i = 0; i < PER; ++i) load_one(i, rsrc, soff, lds_addr, wave);
    }
};

// Scores are produced transposed (keys x queries); a 64-key tile is handled as two groups of 32 keys.  The K
// fragments run through a ring of registers RING fragments ahead of their products: left to itself the compiler reads
// every fragment into the same registers right before its product and waits for it, sixteen exposed LDS latencies per
// tile.  Both score products are issued first; the softmax arithmetic of the first group then runs on the vector ALU
// while the matrix cores are still busy with the second group's scores, and that of the second group while they
// accumulate the first group's P.V.
template <int DH>
__global__ void __launch_bounds__(NT, 2) attn_fwd_mfma_k(const uint16_t *__restrict__ qkv, uint16_t *__restrict__ o,
                                                      float *__restrict__ lse, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    constexpr int KS = DH / 16, DT = DH / 32, TE = 64 * DH, RING = 4;
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];    // [2 buffers][K tile | V tile]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2);
    const int nblk = (int)((Tn + 127) / 128);
    int64_t bh;
    int blk;
    if (!head_and_block(blockIdx.x, Bn * H, nblk, order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q0 = (nblk - 1 - blk) * 128;                               // longest rows first
    const int q0w = q0 + wave * 32, q = q0w + l32;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const __amdgpu_buffer_rsrc_t rsQ = head_rsrc(qb, Tn, ld, DH);
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const i32x4 rsK = make_rsrc(qb + d, head_bytes), rsV = make_rsrc(qb + 2 * d, head_bytes);
    const float c = scale * LOG2E;
    const TileLanes<DH> L(lane);
    const DmaTile<DH> dma(ldb, wave, lane);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = buf_frag(rsQ, (uint32_t)q * ldb + (ks * 16 + lhi * 8) * 2);
    floatx16 oacc[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) oacc[i] = zero16();
    float m = -INFINITY, l = 0.f;                       // reference exponent (log2 domain, scaled) and sum
    const int kv_end = q0 + 128 < (int)Tn ? q0 + 128 : (int)Tn;
    const int ntiles = (kv_end + 63) / 64;

    dma.load(rsK, 0, ldb, lds0, wave);
    dma.load(rsV, 0, ldb, lds0 + TE * 2, wave);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): this wavefront's part of tile 0 has landed
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
        const int j0 = t * 64;
        const uint16_t *Ks = smem + (t & 1) * 2 * TE, *Vs = Ks + TE;
        // Tile t+1 goes to the other buffer, free since the barrier that ended tile t-1.  Its loads are issued one at a
        // time between the score products: issued together right after the barrier, the loads of all eight wavefronts
        // of a compute unit queue up behind one another and every wavefront stalls in the issue.
        const bool more = t + 1 < ntiles;
        const uint32_t nx = lds0 + (uint32_t)((t + 1) & 1) * 2 * TE * 2;
        const uint32_t nsoff = __builtin_amdgcn_readfirstlane(((uint32_t)j0 + 64) * ldb);
        constexpr int NL = 2 * DmaTile<DH>::PER;           // K loads, then V loads
        auto next_load = [&](int i) {
            if (i < DmaTile<DH>::PER) dma.load_one(i, rsK, nsoff, nx, wave);
            else dma.load_one(i - DmaTile<DH>::PER, rsV, nsoff, nx + TE * 2, wave);
        };
        if (more && j0 > q0w + 31) {                    // this wavefront has no products here: it still loads its share
#pragma unroll
            for (int i = 0; i < NL; ++i) next_load(i);
        }
        if (j0 <= q0w + 31) {
            floatx16 s[2];
            {
                constexpr int N = 2 * KS;
                bf16x8 ring[RING];
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = L.row(Ks, (i / KS) * 32, i % KS);
                s[0] = zero16();
                s[1] = zero16();
#pragma unroll
                for (int idx = 0; idx < N; ++idx) {
                    s[idx / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[idx % RING], qf[idx % KS], s[idx / KS], 0, 0, 0);
                    if (idx + RING < N) ring[idx % RING] = L.row(Ks, ((idx + RING) / KS) * 32, (idx + RING) % KS);
                    if (more) {
#pragma unroll
                        for (int i = idx * NL / N; i < (idx + 1) * NL / N; ++i) next_load(i);
                    }
                }
                // pin the order: RING reads, then one product and one read in turn, then the last products
                __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                for (int idx = 0; idx < N - RING; ++idx) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, RING, 0);
            }
            const bool diag = j0 + 63 > q0w;           // the tile crosses the diagonal of some row of this wavefront
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                if (diag) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (j0 + kt * 32 + acc_row(r, lhi) > q) s[kt][r] = -INFINITY;
                }
                // The reference exponent m only has to keep exp2(x - m) in range, it need not be the running maximum.  The
                // probabilities are first taken with the m at hand, and their sum tells whether that was good enough: only
                // when some lane's sum reaches 2^16 (or is not a number: m is still -inf in the first group of a row,
                // where key 0 is visible to every row) is the row maximum of the group computed, m raised to it, everything
                // accumulated so far rescaled and the group redone.  After the first keys that is rare, and the common
                // path has no maximum, no exchange between the lane halves and no rescale in it.
                float pr[16], psum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    pr[r] = __builtin_amdgcn_exp2f(fmaf(s[kt][r], c, -m));
                    psum += pr[r];
                }
                if (__any(!(psum < 65536.0f))) {
                    float tmax = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kt][r]);
                    tmax = max_halves(tmax) * c;
                    const float mn = fmaxf(m, tmax);
                    const float corr = __builtin_amdgcn_exp2f(m - mn);
                    l *= corr;
                    m = mn;
#pragma unroll
                    for (int i = 0; i < DT; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[i][r] *= corr;
                    psum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        pr[r] = __builtin_amdgcn_exp2f(fmaf(s[kt][r], c, -m));
                        psum += pr[r];
                    }
                }
                l += psum;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = pr[r];
                const bf16x8 pk[2] = {pack8<0>(s[kt]), pack8<8>(s[kt])};
                // V fragment f of the group: keys 16 (f / DT) .. + 15, columns 32 (f % DT) .. + 31; like the K fragments
                // they run through a ring of register sets, VR products ahead
                constexpr int NPV = 2 * DT, VR = 4;
                bf16x8 vf[VR];
#pragma unroll
                for (int f = 0; f < VR; ++f) vf[f] = L.tr(Vs, kt * 32 + 16 * (f / DT), f % DT);
#pragma unroll
                for (int f = 0; f < NPV; ++f) {
                    oacc[f % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f % VR], pk[f / DT], oacc[f % DT], 0, 0, 0);
                    if (f + VR < NPV) vf[f % VR] = L.tr(Vs, kt * 32 + 16 * ((f + VR) / DT), (f + VR) % DT);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, 2 * VR, 0);
#pragma unroll
                for (int f = 0; f < NPV - VR; ++f) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, VR, 0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): this wavefront's part of tile t+1 has landed
        __syncthreads();
    }
    l = sum_halves(l);
    if (q < Tn) {
        const float inv = 1.0f / l;
        uint16_t *orow = o + (b * Tn + q) * d + h * DH;
#pragma unroll
        for (int i = 0; i < DT; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint2 w;
                w.x = pack2(oacc[i][4 * g] * inv, oacc[i][4 * g + 1] * inv);
                w.y = pack2(oacc[i][4 * g + 2] * inv, oacc[i][4 * g + 3] * inv);
                *reinterpret_cast<uint2 *>(orow + i * 32 + 8 * g + 4 * lhi) = w;
            }
        if (lhi == 0) lse[bh * Tn + q] = (m + log2f(l)) * LN2;
    }
}

// ------------------------------------------------------------------------------------------ dQ
// Sum over the head dimension of two rows of which a lane pair has the fragments, the same in both lanes: in the order of
// attn_bwd_pre_k, whose bits these are (chains of eight elements, then pairs).
template <int KS> __device__ __forceinline__ float row_dot(const bf16x8 (&g)[KS], const bf16x8 (&o)[KS]) {
    float p[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        Frag a, b;
        a.v = g[ks];
        b.v = o[ks];
        const uint32_t x[4] = {a.u.x, a.u.y, a.u.z, a.u.w}, y[4] = {b.u.x, b.u.y, b.u.z, b.u.w};
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sum = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), sum);
            sum = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), sum);
        }
        p[ks] = sum_halves(sum);
    }
#pragma unroll
    for (int o2 = 1; o2 < KS; o2 *= 2)
#pragma unroll
        for (int ks = 0; ks < KS; ks += 2 * o2) p[ks] += p[ks + o2];
    return p[0];
}

// Bound: vector work (exponentials, masks) and latency between the products; the tiles in front of the diagonal run through a loop of
// their own, without mask and branch.  Three wavefronts per SIMD at head size 64, which a ring of three fragments leaves registers for.
// 8 x 1024 tokens, 12 heads of 64: 45.9 -> 39.4 us (two wavefronts per SIMD 43.1); 4 x 2048, 32 heads of 128: 272 -> 252.
// O: nullptr, or the forward pass's output: delta is then computed here, from the rows of dO that are in registers anyway, and
// written for the dK/dV kernel, in place of a launch that reads both tensors (forward and backward 100.8 -> 97.2 us and 708 -> 687).
template <int DH, int NW>
__device__ __forceinline__ void dq_rows(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const uint16_t *__restrict__ O,
                                        const float *__restrict__ lse, float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn,
                                        int64_t Tn, int64_t H, float scale, Order order, unsigned block) {
    constexpr int KS = DH / 16, DT = DH / 32, TE = 64 * DH, RING = DH == 64 ? 3 : 4, ROWS = NW * 32;
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];    // [2 buffers][K tile | V tile], filled as in the forward kernel
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2);
    const int nblk = (int)((Tn + ROWS - 1) / ROWS);
    int64_t bh;
    int blk;
    if (!head_and_block(block, Bn * H, nblk, order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int q0 = (nblk - 1 - blk) * ROWS;
    const int q0w = q0 + wave * 32, q = q0w + l32;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const __amdgpu_buffer_rsrc_t rsQ = head_rsrc(qb, Tn, ld, DH);
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const i32x4 rsK = make_rsrc(qb + d, head_bytes), rsV = make_rsrc(qb + 2 * d, head_bytes);
    const __amdgpu_buffer_rsrc_t rsG = head_rsrc(dO + b * Tn * d + h * DH, Tn, d, DH);
    const float c = scale * LOG2E;
    const bool live = q < Tn;
    const TileLanes<DH> L(lane);
    const DmaTile<DH, NW> dma(ldb, wave, lane);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    bf16x8 qf[KS], gf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        qf[ks] = buf_frag(rsQ, (uint32_t)q * ldb + (ks * 16 + lhi * 8) * 2);
        gf[ks] = buf_frag(rsG, (uint32_t)q * (uint32_t)(d * 2) + (ks * 16 + lhi * 8) * 2);
    }
    const float lse2 = live ? lse[bh * Tn + q] * LOG2E : 0.f;
    float dl;
    if (O) {
        const __amdgpu_buffer_rsrc_t rsO = head_rsrc(O + b * Tn * d + h * DH, Tn, d, DH);
        bf16x8 of[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) of[ks] = buf_frag(rsO, (uint32_t)q * (uint32_t)(d * 2) + (ks * 16 + lhi * 8) * 2);
        dl = row_dot<KS>(gf, of);
        if (live && lhi == 0) delta[bh * Tn + q] = dl;
    } else {
        dl = live ? delta[bh * Tn + q] : 0.f;
    }
    floatx16 dq[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) dq[i] = zero16();
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
        if (!DIAG() || j0 <= q0w + 31) {
            floatx16 s[2], dp[2];
            {
                // S = K.Q^T and dP = V.dO^T for both key groups; the K and V fragments run RING ahead of their products
                constexpr int N = 4 * KS;
                bf16x8 ring[RING];
                auto frag = [&](int idx) { return L.row((idx & 1) ? Vs : Ks, (idx / (2 * KS)) * 32, (idx / 2) % KS); };
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = frag(i);
                s[0] = zero16(); s[1] = zero16(); dp[0] = zero16(); dp[1] = zero16();
#pragma unroll
                for (int idx = 0; idx < N; ++idx) {
                    const int kt = idx / (2 * KS), ks = (idx / 2) % KS;
                    if (idx & 1) dp[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[idx % RING], gf[ks], dp[kt], 0, 0, 0);
                    else s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[idx % RING], qf[ks], s[kt], 0, 0, 0);
                    if (idx + RING < N) ring[idx % RING] = frag(idx + RING);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                for (int idx = 0; idx < N - RING; ++idx) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, RING, 0);
            }
            // per group of 32 keys: the element-wise part of one group overlaps the other group's products
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float p = __builtin_amdgcn_exp2f(fmaf(s[kt][r], c, -lse2));
                    if (DIAG() && kt * 32 + acc_row(r, 0) > q - j0 - 4 * lhi) p = 0.0f;
                    s[kt][r] = p * (dp[kt][r] - dl);          // the 1/sqrt(dh) factor is applied once, to the sums
                }
                const bf16x8 d0 = pack8<0>(s[kt]), d1 = pack8<8>(s[kt]);
#pragma unroll
                for (int i = 0; i < DT; ++i) {
                    dq[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Ks, kt * 32, i), d0, dq[i], 0, 0, 0);
                    dq[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Ks, kt * 32 + 16, i), d1, dq[i], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): this wavefront's part of tile t+1 has landed
        __syncthreads();
    };
    int t = 0;
    for (; t < q0 / 64; ++t) tile(t, std::false_type{});
    for (; t < ntiles; ++t) tile(t, std::true_type{});
    if (live) {
        uint16_t *orow = dqkv + (b * Tn + q) * ld + h * DH;
#pragma unroll
        for (int i = 0; i < DT; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint2 w;
                w.x = pack2(dq[i][4 * g] * scale, dq[i][4 * g + 1] * scale);
                w.y = pack2(dq[i][4 * g + 2] * scale, dq[i][4 * g + 3] * scale);
                *reinterpret_cast<uint2 *>(orow + i * 32 + 8 * g + 4 * lhi) = w;
            }
    }
}

template <int DH>
__global__ void __launch_bounds__(NT, DH == 64 ? 3 : 2) attn_bwd_dq_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv,
                                                         const uint16_t *__restrict__ O, const float *__restrict__ lse, float *__restrict__ delta,
                                                         uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    dq_rows<DH, NT / 64>(dO, qkv, O, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
}

// ------------------------------------------------------------------------------------------ dK, dV
// Both gradients in one launch: S and dP are computed once for the two of them, and the Q and dO tiles are loaded once.  A
// wavefront's accumulators and K fragments take 160 of the 256 registers that two wavefronts per SIMD allow at head size 128,
// so its V fragments are not kept in registers there but read from LDS (the workgroup's V rows, loaded once); to have room for
// them, and half the tile loads per product, a workgroup is eight wavefronts with 256 key rows.  Bound: latency between the
// products of two wavefronts per SIMD.  Measured at 4 x 2048 tokens, 32 heads of 128 (kernel trace): 393 us, where two launches with
// four wavefronts each (dV, then dK) took 227 + 302; whole backward pass faster at every size tried, from 1 x 64 x 2 heads (forward and
// backward 25.4 -> 21.5 us) to 1 x 4096 x 52 (1457 -> 1233).  Head size 64, 8 x 1024 tokens, 12 heads: 60 us.
// The tiles behind the diagonal run through a loop of their own, without mask and branch: 4 x 2048, 32 heads of 128 444 -> 413 us.  At
// head size 64 a second loop takes the registers of the third wavefront per SIMD and gains nothing over a mask of two instructions
// (8 x 1024, 12 heads: 62 -> 56.3 us, 57.0 with two loops).
// Every one of the 256 registers is in use at head size 128, and nothing may spill: a reload from scratch in the loop waits for the
// tile loads in flight, and the wavefront with it keeps the others at the barrier (six spilled registers, and the statistics multiplied
// where they are loaded: 8 % of the kernel).  So the offsets of the transposing reads are one register and an exclusive or each, each of
// two wavefronts fetches one of the statistics, and the lane index is computed where it is used.  Transposed fragments four ahead in
// registers: slower by 9 %, for want of the registers.
template <int DH> constexpr int dkv_waves() { return DH == 128 ? 8 : 4; }
template <int DH, int NW>
__device__ __forceinline__ void dkv_rows(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const float *__restrict__ lse,
                                         const float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H,
                                         float scale, Order order, unsigned block) {
    constexpr int KS = DH / 16, DT = DH / 32, TE = 64 * DH, RING = 4, KEYS = NW * 32;
    constexpr bool VLDS = DH == 128, ONE_LOOP = DH == 64;
    constexpr int BUF = 2 * TE;                                          // Q tile | dO tile, filled as in the forward kernel
    // [2 buffers][Q | dO], [KEYS][DH] V rows if VLDS, then [2][64 lse | 64 delta] floats
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int64_t d = H * DH, ld = 3 * d;
    const uint32_t ldb = (uint32_t)(ld * 2), ldg = (uint32_t)(d * 2);
    int64_t bh;
    int blk;
    if (!head_and_block(block, Bn * H, (int)((Tn + KEYS - 1) / KEYS), order, bh, blk)) return;
    const int64_t b = bh / H, h = bh % H;
    const int kv0 = blk * KEYS;                                           // earliest keys see the most queries: first
    const int kv0w = kv0 + wave * 32, kv = kv0w + l32;
    const uint16_t *qb = qkv + b * Tn * ld + h * DH;
    const uint32_t head_bytes = (uint32_t)(((Tn - 1) * ld + DH) * 2);
    const __amdgpu_buffer_rsrc_t rsK = head_rsrc(qb + d, Tn, ld, DH), rsV = head_rsrc(qb + 2 * d, Tn, ld, DH);
    const i32x4 rsQ = make_rsrc(qb, head_bytes);
    const i32x4 rsG = make_rsrc(dO + b * Tn * d + h * DH, (uint32_t)(((Tn - 1) * d + DH) * 2));
    const float c = scale * LOG2E;
    const TileLanes<DH, VLDS> L(lane);
    const DmaTile<DH, NW> dmaQ(ldb, wave, lane), dmaG(ldg, wave, lane);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    const uint16_t *Vs = smem + 2 * BUF;

    bf16x8 kf[KS], vf[VLDS ? 1 : KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        kf[ks] = buf_frag(rsK, (uint32_t)kv * ldb + (ks * 16 + lhi * 8) * 2);
        if (!VLDS) vf[VLDS ? 0 : ks] = buf_frag(rsV, (uint32_t)kv * ldb + (ks * 16 + lhi * 8) * 2);
    }
    if (VLDS) {
        const i32x4 rs = make_rsrc(qb + 2 * d, head_bytes);
#pragma unroll
        for (int i = 0; i < KEYS / 64; ++i) dmaQ.load(rs, (uint32_t)(kv0 + 64 * i), ldb, lds0 + (2 * BUF + i * TE) * 2, wave);
    }
    floatx16 dk[DT], dv[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) { dk[i] = zero16(); dv[i] = zero16(); }
    const int ntiles = ((int)Tn - kv0 + 63) / 64;

    // Statistics of row i0 + lane, one tile ahead, log-sum-exp in wavefront 0 and delta in wavefront 1: through descriptors of the head's
    // rows (rows past the sequence read zero; no addresses to keep in registers), used only where they go to LDS, a tile after their fetch.
    const __amdgpu_buffer_rsrc_t rsS = buffer_over((wave == 0 ? lse : delta) + bh * Tn, (uint32_t)Tn * 4);
    const float to_lds = wave == 0 ? LOG2E : 1.f;
    float st = 0.f;
    float *stats = reinterpret_cast<float *>(smem + 2 * BUF + (VLDS ? KEYS * DH : 0));
    auto load_stats = [&](int i0) {
        if (wave < 2) st = buffer_load4(rsS, (uint32_t)(i0 + lane_here()) * 4);
    };
    auto store_stats = [&](int buf) {
        if (wave < 2) stats[buf * 128 + wave * 64 + lane_here()] = st * to_lds;
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
    auto key_less_4half = []() __attribute__((always_inline)) { const int ln = lane_here(); return (ln & 31) - 4 * (ln >> 5); };
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
            const int masked = DIAG ? kv0w - i0 + key_less_4half() : 0;        // rows of the tile before this lane's key, less 4 lhi
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                floatx16 s = zero16(), dp = zero16();
                {
                    // S^T = Q.K^T, then dP^T = dO.V^T; the Q and dO fragments run RING ahead of their products, V's VR ahead
                    constexpr int N = 2 * KS, VR = 2;
                    bf16x8 ring[RING], vr[VLDS ? VR : 1];
                    auto frag = [&](int idx) { return L.row(idx < KS ? Qs : Gs, qt * 32, idx % KS); };
#pragma unroll
                    for (int i = 0; i < RING; ++i) ring[i] = frag(i);
#pragma unroll
                    for (int idx = 0; idx < N; ++idx) {
                        if (idx < KS) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[idx % RING], kf[idx % KS], s, 0, 0, 0);
                        else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[idx % RING], VLDS ? vr[VLDS ? idx % VR : 0] : vf[VLDS ? 0 : idx % KS], dp, 0, 0, 0);
                        if (idx + RING < N) ring[idx % RING] = frag(idx + RING);
                        if (VLDS && idx + VR >= KS && idx + VR < N) vr[VLDS ? idx % VR : 0] = L.row(Vs, wave * 32, (idx + VR) % KS);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                    for (int idx = 0; idx < N; ++idx) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        const int reads = (idx + RING < N ? 1 : 0) + (VLDS && idx + VR >= KS && idx + VR < N ? 1 : 0);
                        if (reads == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        else if (reads == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                }
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    // rows 8*r4 + 4*lhi + 0..3 of this 32-row group: their statistics are 16 contiguous bytes
                    const int half4 = 4 * (END ? lane_here() >> 5 : lhi), ql = qt * 32 + 8 * r4 + half4;
                    const float4 l4 = *reinterpret_cast<const float4 *>(L2s + ql), d4 = *reinterpret_cast<const float4 *>(Ds + ql);
                    const int first = END ? kv0w - i0 + key_less_4half() : 0, end = (int)Tn - i0 - half4;
                    const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dvv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = 4 * r4 + e;
                        float p = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lv[e]));
                        if (DIAG && qt * 32 + 8 * r4 + e < masked) p = 0.0f;
                        if (END && (qt * 32 + 8 * r4 + e < first || qt * 32 + 8 * r4 + e >= end)) p = 0.0f;
                        dp[r] = p * (dp[r] - dvv[e]);        // the 1/sqrt(dh) factor is applied once, to the sums
                        s[r] = p;
                    }
                }
                const bf16x8 p0 = pack8<0>(s), p1 = pack8<8>(s), d0 = pack8<0>(dp), d1 = pack8<8>(dp);
#pragma unroll
                for (int i = 0; i < DT; ++i) {
                    dv[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Gs, qt * 32, i), p0, dv[i], 0, 0, 0);
                    dv[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Gs, qt * 32 + 16, i), p1, dv[i], 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < DT; ++i) {
                    dk[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Qs, qt * 32, i), d0, dk[i], 0, 0, 0);
                    dk[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.tr(Qs, qt * 32 + 16, i), d1, dk[i], 0, 0, 0);
                }
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
    const int last = lane_here(), half = last >> 5, key = kv0w + (last & 31);
    if (key < (int)Tn) {
        uint16_t *krow = dqkv + (b * Tn + key) * ld + d + h * DH, *vrow = krow + d;
#pragma unroll
        for (int i = 0; i < DT; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint2 w;
                w.x = pack2(dk[i][4 * g] * scale, dk[i][4 * g + 1] * scale);
                w.y = pack2(dk[i][4 * g + 2] * scale, dk[i][4 * g + 3] * scale);
                *reinterpret_cast<uint2 *>(krow + i * 32 + 8 * g + 4 * half) = w;
                w.x = pack2(dv[i][4 * g], dv[i][4 * g + 1]);
                w.y = pack2(dv[i][4 * g + 2], dv[i][4 * g + 3]);
                *reinterpret_cast<uint2 *>(vrow + i * 32 + 8 * g + 4 * half) = w;
            }
    }
}

template <int DH>
__global__ void __launch_bounds__(dkv_waves<DH>() * 64, DH == 64 ? 3 : 2)
    attn_bwd_dkv_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const float *__restrict__ lse,
                        const float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order) {
    dkv_rows<DH, dkv_waves<DH>()>(dO, qkv, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
}

// Both kernels' blocks in one launch, those of key rows first: for sequences whose blocks leave the chip room, where each of the two
// kernels lasts as long as its longest chain of tiles.  The same rows to a block on either side; delta comes from a launch of its own, and
// every output has the bits of the two launches.  At head size 128 with four wavefronts a workgroup has a compute unit to itself (its
// V rows in LDS), and its wavefronts all registers of their SIMD.
template <int DH, int NW>
__global__ void __launch_bounds__(NW * 64, DH == 64 ? 3 : NW == 4 ? 1 : 2)
    attn_bwd_both_mfma_k(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ qkv, const float *__restrict__ lse,
                         float *__restrict__ delta, uint16_t *__restrict__ dqkv, int64_t Bn, int64_t Tn, int64_t H, float scale, Order order,
                         unsigned blocks) {
    if (blockIdx.x < blocks) dkv_rows<DH, NW>(dO, qkv, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x);
    else dq_rows<DH, NW>(dO, qkv, nullptr, lse, delta, dqkv, Bn, Tn, H, scale, order, blockIdx.x - blocks);
}

template <int DH> constexpr size_t kv_smem() { return (size_t)2 * 2 * 64 * DH * 2; }       // two buffers of two tiles
template <int DH, int NW> constexpr size_t dkv_smem() {         // tiles, V rows, then statistics
    return (size_t)2 * 2 * 64 * DH * 2 + (DH == 128 ? (size_t)NW * 32 * DH * 2 : 0) + 2 * 128 * 4;
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
    const Launch l(B * H, Tn, dh, 128, dh == 64 ? 4 : 2);
    const float scale = 1.0f / sqrtf((float)dh);
    static bool attr_set = false;
    if (!attr_set) {       // head dimension 128 needs more than the default 64 KiB of LDS
        (void)hipFuncSetAttribute((const void *)attn_fwd_mfma_k<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kv_smem<128>());
        attr_set = true;
    }
    if (dh == 64) attn_fwd_mfma_k<64><<<l.grid, NT, kv_smem<64>(), s>>>((const uint16_t *)qkv, (uint16_t *)o, lse, B, Tn, H, scale, l.order);
    else attn_fwd_mfma_k<128><<<l.grid, NT, kv_smem<128>(), s>>>((const uint16_t *)qkv, (uint16_t *)o, lse, B, Tn, H, scale, l.order);
}

void attn_bwd_mfma(hipStream_t s, const void *dO, const void *qkv, const void *O, const float *lse, float *delta, void *dqkv,
                   int64_t B, int64_t Tn, int64_t H, int64_t dh) {
    const float scale = 1.0f / sqrtf((float)dh);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)attn_bwd_dq_mfma_k<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kv_smem<128>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_dkv_mfma_k<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, dkv_waves<128>()>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_both_mfma_k<128, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, 4>());
        (void)hipFuncSetAttribute((const void *)attn_bwd_both_mfma_k<128, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_smem<128, 8>());
        attr_set = true;
    }
    // One launch for both gradients while its workgroups, which a unit holds three of at head size 64 and one of at 128, are at most a
    // little more than the chip holds at once.  Forward and backward, us, two launches / one (workgroups):
    //   heads of 64:  1 x 1024, 12 heads  65 /  50 (256)     8 x 512, 12 47 / 41 (768)       8 x 300, 20 37.4 / 35.4 (960)
    //                 1 x 4096,  8       213 / 169 (512)     8 x 192,  7 22.7 / 19.6 (224)   8 x 1024, 12 90.8 / 91.5 (1536)
    //   of 128, four wavefronts, eight in brackets:  1 x 2048, 8 178 / 126 [137] (256 [128])   4 x 512, 16 68 / 58 [56] (512 [256])
    //                 (two rounds of four wavefronts are better with long chains: 1 x 4096, 4 heads 330 / 230 [255], 2 x 1024, 16 105 / 81
    //                 [84], but 8 x 256, 16 49 / 46 [43])
    //                 4 x 333, 6 52 / 37 [42] (144 [96])     3 x 700, 25 90 / - [87] (960 [480])   8 x 1024, 16 217 / - [225] (- [1024])
#define TIO_ATTN_BOTH(DH, NW, WORKGROUPS)                                                                                                      \
    {                                                                                                                                          \
        const Launch l(B * H, Tn, DH, NW * 32, DH == 64 ? 3 : 1);                                                                              \
        if (2 * (int64_t)l.grid.x <= WORKGROUPS) {                                                                                             \
            if (O) attn_bwd_pre(s, TIO_PREC_BF16, dO, O, delta, B, Tn, H, DH);                                                                 \
            attn_bwd_both_mfma_k<DH, NW><<<2 * l.grid.x, NW * 64, dkv_smem<DH, NW>(), s>>>(                                                    \
                (const uint16_t *)dO, (const uint16_t *)qkv, lse, delta, (uint16_t *)dqkv, B, Tn, H, scale, l.order, l.grid.x);                \
            return;                                                                                                                            \
        }                                                                                                                                      \
    }
#define TIO_ATTN_BWD(DH, DQ_PER_CU, DKV_PER_CU)                                                                                                \
    {                                                                                                                                          \
        const Launch q(B * H, Tn, DH, 128, DQ_PER_CU), kv(B * H, Tn, DH, dkv_waves<DH>() * 32, DKV_PER_CU);                                    \
        attn_bwd_dq_mfma_k<DH><<<q.grid, NT, kv_smem<DH>(), s>>>((const uint16_t *)dO, (const uint16_t *)qkv, (const uint16_t *)O, lse, delta, \
                                                                 (uint16_t *)dqkv, B, Tn, H, scale, q.order);                                  \
        attn_bwd_dkv_mfma_k<DH><<<kv.grid, dkv_waves<DH>() * 64, dkv_smem<DH, dkv_waves<DH>()>(), s>>>(                                        \
            (const uint16_t *)dO, (const uint16_t *)qkv, lse, delta, (uint16_t *)dqkv, B, Tn, H, scale, kv.order);                             \
    }
    if (dh == 64) {
        TIO_ATTN_BOTH(64, 4, 1024)
        TIO_ATTN_BWD(64, 3, 3)
    } else {
        TIO_ATTN_BOTH(128, 4, (Tn < 1024 ? 256 : 512))
        TIO_ATTN_BOTH(128, 8, 512)
        TIO_ATTN_BWD(128, 2, 1)
    }
#undef TIO_ATTN_BOTH
#undef TIO_ATTN_BWD
}

}  // namespace k
}  // namespace tio
