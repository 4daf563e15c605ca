// FlexAttention backward kernels for gfx950 (backward template of paper section 4.1, walking the
// BlockMask in both orientations, section 4.2).  The paper gives no formulas; with P recomputed
// from the saved LSE this is the usual softmax-attention calculus:
//     dV = P^T dO,  dP = dO V^T,  dS' = P * (dP - delta),  delta = rowsum(dO * O),
//     dS = dS' * d score_mod / d s,  dQ = scale * dS K,  dK = scale * dS^T Q.
// Three kernels, no floating-point atomics (results are deterministic):
//   bwd_delta_kernel   -delta and the row constant of P = exp2(f(score) + rc) per query row (where the dQ kernel, which
//                      can make them, does not run first).
//   bwd_dkdv_kernel    one workgroup per 64 keys of one (b, hkv); walks the q-blocks listed for
//                      that column of blocks (transposed BlockMask) for every query head of the
//                      group; score tile in S = Q K^T orientation so that P and dS are the B
//                      operands of dV^T += dO^T P and dK^T += Q^T dS; the two waves that share
//                      keys split the outputs (one dV, one dK) and exchange P / dS through LDS.
//   bwd_dq_kernel      one workgroup per row of blocks of one (b, hq); walks the kv-blocks listed
//                      for it; score tile transposed (S^T = K Q^T) so that dS^T is the B operand of
//                      dQ^T += K^T dS^T and LSE / delta are per-lane scalars.
// Tiles (Q, dO in the first kernel; K, V in the second) go from global memory straight into
// XOR-swizzled LDS tiles, double buffered; the transposed operands (dO^T, Q^T, K^T) come out of
// the same row-major tiles through transposing LDS reads.  dP accumulates on top of -delta.
#pragma once

#include <type_traits>

#include "flex_common.h"
#include "lds_tiles.h"

namespace flexattn {

struct BwdArgs {
    const bf16* Q;
    const bf16* K;
    const bf16* V;
    const bf16* O;
    const bf16* dO;
    const float* LSE;
    bf16* dQ;
    bf16* dK;
    bf16* dV;
    float* delta;   // [B, Hq, q_len]  MINUS rowsum(dO * O): the dP accumulators start from it
    float* lse2;    // [B, Hq, q_len]  row constant rc of ScoreMod::p_with_grad (from LSE); -inf for dead rows
    // gradients of captured tensors: per-workgroup partial sums, [B, Hq, NR] and [B, Hq, NR, rel_len]
    float* cap_alibi;
    float* cap_rel;
    int64_t q_sb, q_sh, q_ss, k_sb, k_sh, k_ss, v_sb, v_sh, v_ss, o_sb, o_sh, o_ss, do_sb, do_sh, do_ss;
    int64_t dq_sb, dq_sh, dq_ss, dk_sb, dk_sh, dk_ss, dv_sb, dv_sh, dv_ss;
    int B, Hq, Hkv, G, q_len, kv_len;
    int NR, NC, Bq, Bk;
    int bm_Bm, bm_Hm;
    UnitSets abreast;      // of the launch (unit_of_workgroup)
    int head_parts;        // dK/dV: workgroups among which the query heads of a group are divided (kv_head_parts),
    int least_steps;       //        kPartsIfLong: if the longest column has as many steps
    int halved;            // MIXED: how many of the rows of blocks, in work order, are taken in halves
    int turns_above;       // dS in memory: heads take turns where the longest row has more tiles (documents; 0: always)
    const int32_t* kv_num;
    const int32_t* kv_idx;
    const int32_t* full_kv_num;
    const int32_t* full_kv_idx;
    const int32_t* q_num;
    const int32_t* q_idx;
    const int32_t* full_q_num;
    const int32_t* full_q_idx;
    const int32_t* kv_order;   // nullable work orders (rows / columns of blocks, longest first)
    const int32_t* q_order;
    // dS kept in memory (bwd_stored.h): the dK/dV kernel writes the dS of every block it visits, a lean
    // kernel contracts it with K.  Null ds_store: nothing is written.
    bf16* ds_store;            // [heads that share no dS, ds_blocks, Bk / 64, Bq / 64, 4096] (see ds_chunk)
    const int32_t* ds_colbase; // [planes * NC] first block slot of every column of blocks
    const int32_t* ds_grid;    // [planes, NR, NC] slot of block (row, column)
    int64_t ds_blocks;         // slots per head (capacity)
    float scale;
    flexattn_mod_params p;
    bool make_delta;           // the dQ kernel works the row scalars out itself (and writes them)
    bool dq_last;              // (host) dQ is written over what dK/dV or the row scalars are made of: it runs last, after a pass for the latter
    float* kv_part;        // dK/dV, head_parts > 1: their sums, [head_parts][dV, dK][B, Hkv, kv_len, D] (host: where there is room for them, or null)
};

// Among how many workgroups the query heads of a group are divided.  One that takes them all walks G times the steps of a column: few KV heads
// leave most of the chip idle, and end with the longest column alone.  A part costs its sums in fp32, 128 bytes a key and D / 16 each way, and all a launch that
// adds them up (3 us).  So: up to 768 workgroups (D = 64: all that run at once), as many parts as spare the longest column's workgroup 48 steps of 64 rows (D = 128: 32, whose steps
// are longer) or more for each beyond the first, or 12 (6) while they are no more than half of the CUs.  worth(parts): what else speaks against it (parts_pay).
// us, dK/dV, whole groups -> this, S x query / KV heads, causal: D = 64, 4096 x 8 / 1 137 -> 55, 1500 x 16 / 2
// 60 -> 33, 3000 x 32 / 4 112 -> 105, 700 x 8 / 1 35 -> 16; D = 128, 1500 x 8 / 1 126 -> 41, 3000 x 16 / 2 242 -> 95,
// 3000 x 4 / 1 124 -> 42, 6000 x 8 / 4 220 -> 162; no mask, D = 128, 6000 x 16 / 2 825 -> 574; window of
// 1000, D = 64, 6000 x 32 / 4 151 -> 124.  More parts: 1500 x 32 x 8 / 1, D = 128, two 375, whole 342; window of 1024, 4 x 5000 x 16 / 2, D = 64, two 208, whole 198, no mask, 12653 x 8 / 2, two 843, whole 797;
// shorter ones: 300 x 2 / 1, D = 64 14.4, whole 11.2.
// Over 7695 launches (one to sixteen KV heads, groups of 2 to 16, S = 300 to 12000; no mask, causal with and without a soft-cap, a window, a window or a prefix, documents of 16 to 200 and of 256 to
// 4096, canvases) three were slower than whole, by 3 to 5 %; all together, divided or not, they were 1.21 (D = 64) and 1.38 times as fast.
// That sweep was made before parts_pay's lines for parts of unlike size were last moved, and not again since.
template <class Worth>
int kv_head_parts(int64_t units, int G, int kv_len, int D, int64_t longest_column, Worth&& worth) {
    const int64_t tiles = units * ((kv_len + 63) / 64), steps = (longest_column + 63) / 64;
    int parts = 1;
    for (int p = 2; p <= G && p <= 8 && tiles * p <= 768; p *= 2) {
        const int64_t groups = tiles * p, spared = G - (G + p - 1) / p;     // heads
        if (steps * spared >= (int64_t)(p - 1) * (groups <= 128 ? (D == 64 ? 12 : 6) : (D == 64 ? 48 : 32)) && worth(p)) parts = p;
    }
    return parts;
}
// The query heads of a group that a dK/dV workgroup takes, and where their sums go.  Kernels of their own: what this keeps over the walk and the second way
// to write the sums spill up to 6 registers in those that take whole groups, whose launches of one round last up to 4 % longer (one kernel for both -> two, us: D = 64,
// window of 300 and soft-cap, S = 1000, 32 heads 17.6 -> 17.2, documents with ALiBi, S = 800, 24 heads 18.0 -> 17.6; D = 128, causal, S = 1000, 4 heads 18.5 -> 17.7, no mask,
// S = 500, 8 heads 13.5 -> 13.0).
enum class Groups { kWhole, kParts, kPartsIfLong };
template <Groups GROUPS>
struct KvHeads {
    int part, first, end;
    bool apart;         // the sums are those of a part
    // unit: (b, hkv, part) -> (b, hkv).  (`parts` is asked here and `apart` at the sums even where they are known: else the parts' addresses are made ahead of the walk and
    // spill 50 scalar registers: relative bias, window of 200 or prefix of 64, S = 8192, 16 / 2 heads, D = 128, 389 -> 405 us, D = 64 159 -> 169)
    __device__ __forceinline__ KvHeads(const BwdArgs& a, int parts, int& unit) : part(0), first(0), end(a.G), apart(false) {
        if (GROUPS != Groups::kWhole && parts > 1) {
            part = unit % parts;
            unit /= parts;
            first = part * a.G / parts;
            end = (part + 1) * a.G / parts;
            apart = true;
        }
    }
    __device__ __forceinline__ float* sums(const BwdArgs& a, int unit, int is_k, int D) const {
        return a.kv_part + (((int64_t)(2 * part + is_k) * a.B * a.Hkv + unit) * a.kv_len) * D;
    }
};
// kPartsIfLong: among how many workgroups the heads are divided in the end, by the steps of a head in the longest column of blocks (the first in work order) of the first plane.
__device__ __forceinline__ int parts_if_long(const BwdArgs& a) {
    const int col = min(max(ldc(a.q_order), 0), a.NC - 1);
    return (ldc(a.full_q_num + col) + ldc(a.q_num + col)) * (a.Bq / 64) < a.least_steps ? 1 : a.head_parts;
}
// Workgroup -> (b, hkv, part) and its piece of a column's, of a launch for a.head_parts; parts: of how many.  False: nothing to do.
template <Groups GROUPS>
__device__ __forceinline__ bool kv_unit_of_workgroup(const BwdArgs& a, int per_unit, UnitSets abreast, int& parts, int& unit, int& rank) {
    parts = GROUPS == Groups::kWhole ? 1 : GROUPS == Groups::kParts ? a.head_parts : parts_if_long(a);
    const int units = a.B * a.Hkv * parts;
    if (GROUPS == Groups::kPartsIfLong && blockIdx.x >= unit_grid(units, per_unit)) return false;
    return unit_of_workgroup(units, per_unit, abreast, unit, rank);
}

constexpr uint32_t kBwdStageCaptured = 8u;   // internal: the captured-tensor sums instead of dQ

// dS in memory.  The non-empty blocks of all BlockMask planes are numbered column by column of blocks,
// in the order of the merged (FULL, then PARTIAL) column lists: that number is the block's slot.
// Heads that share a plane share the numbering and differ in `rep`.  A block is cut into Bk / 64 tiles
// of 64 keys, a tile into Bq / 64 steps of 64 query rows, and a step is the 8 KiB the four waves of
// the dK/dV workgroup hold in registers after the step: wave (kb, x) two chunks of 1 KiB, lane
// (key 32 kb + l32, half h) 16 bytes of each -- chunk c holds rows 32 x + 16 c + 8 jj + 4 h + i at
// position 4 jj + i.  Slots are clamped to the capacity: a caller that passes too small a capacity
// gets wrong gradients, never an access outside the workspace.
__device__ __forceinline__ int64_t ds_rep(const BwdArgs& a, int b, int hq) {
    return (int64_t)(a.bm_Bm > 1 ? 0 : b) * (a.bm_Hm > 1 ? 1 : a.Hq) + (a.bm_Hm > 1 ? 0 : hq);
}
// index of the 8 KiB step (in units of 4096 bf16) of block `slot`, key tile `st`, row step `sidx`
__device__ __forceinline__ int64_t ds_chunk(const BwdArgs& a, int64_t rep, int slot, int st, int sidx) {
    const int64_t sl = min(max((int64_t)slot, (int64_t)0), a.ds_blocks - 1);
    return ((rep * a.ds_blocks + sl) * (a.Bk / 64) + st) * (a.Bq / 64) + sidx;
}

// ------------------------------------------------------------------------------------------
// -delta = -rowsum(dO * O) and the per-row constant rc of ScoreMod::p_with_grad (so that the main
// kernels get P = exp2(f(score) + rc) with no further per-row arithmetic); rc = -inf for rows
// without a visible key (LSE = -inf), which makes their P vanish.
template <int D, uint32_t SCORE>
__global__ __launch_bounds__(256) void bwd_delta_kernel(const BwdArgs a) {
    // 8 lanes per row (D = 64) or 16 lanes per row (D = 128): each lane owns 8 consecutive dims.
    constexpr int LPR = D / 8;
    constexpr int RPB = 256 / LPR;
    const int64_t rows = (int64_t)a.B * a.Hq * a.q_len;
    const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
    const int c = threadIdx.x % LPR;
    if (row >= rows) return;
    const int q = (int)(row % a.q_len);
    const int h = (int)((row / a.q_len) % a.Hq);
    const int b = (int)(row / ((int64_t)a.q_len * a.Hq));
    const bf16x8 o = *(const bf16x8*)(a.O + b * a.o_sb + h * a.o_sh + (int64_t)q * a.o_ss + c * 8);
    const bf16x8 g = *(const bf16x8*)(a.dO + b * a.do_sb + h * a.do_sh + (int64_t)q * a.do_ss + c * 8);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s = __builtin_fmaf((float)o[i], (float)g[i], s);
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (c == 0) {
        a.delta[row] = -s;
        const float l = a.LSE[row];
        const ScoreMod<SCORE> smod(a.p, h, a.scale);
        a.lse2[row] = smod.row_const((l == -INFINITY) ? INFINITY : l * kLog2e);
    }
}

// -delta and the row constant of a lane's row from its dO (in the layout of an MFMA operand), as bwd_delta_kernel
// makes them, to the bit: dO is in the dQ kernels' registers anyway, and the pass over O and dO is spared.  (us of the
// whole backward, with the pass -> this: causal, S = 1024, 64 x 16 heads 774 -> 741 at D = 64, 1501 -> 1442 at D = 128; window of
// 1024, S = 5000, 4 x 16 / 2 heads 340 -> 328, 685 -> 666; packed documents with ALiBi, S = 16384 410 -> 399; of the captured
// sums of a relative bias, S = 8192, window of 1024, D = 128 240 -> 224.)
template <int D, uint32_t SCORE>
__device__ __forceinline__ void row_scalars(const BwdArgs& a, int b, int hq, int q, int half, const bf16x8 (&g)[D / 16], float& rc, float& neg_delta) {
    const bf16* op = a.O + b * a.o_sb + hq * a.o_sh + (int64_t)q * a.o_ss + half * 8;
    float s[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const bf16x8 o = *(const bf16x8*)(op + ks * 16);
        s[ks] = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) s[ks] = __builtin_fmaf((float)o[i], (float)g[ks][i], s[ks]);
    }
    // (added up in the order of bwd_delta_kernel: the same bits)
#pragma unroll
    for (int n = D / 32; n > 0; n >>= 1)
#pragma unroll
        for (int i = 0; i < n; ++i) s[i] += s[i + n];
    neg_delta = -(s[0] + swap_halves(s[0]));
    const float l = a.LSE[((int64_t)b * a.Hq + hq) * a.q_len + q];
    rc = ScoreMod<SCORE>(a.p, hq, a.scale).row_const(l == -INFINITY ? INFINITY : l * kLog2e);
}

// Neighborhood masks: bit kb + 2 x is set if the mask hides the block of the 32 query rows q0 + 32 x .. and the 32
// keys kv0 + 32 kb .. .  The dQ kernel that reads dS back takes the same answer for the same block
// (CanvasBlocks::hidden_bits), so the dS of such a block is neither written nor read.
__device__ __forceinline__ int canvas_step_bits(const flexattn_mod_params& p, int q0, int kv0) {
    const CanvasBlocks cb(p);
    const CanvasBlocks::Box qw[2] = {cb.windows(q0), cb.windows(q0 + 32)};
    const uint32_t b = cb.hidden_bits(qw, kv0);     // bit 2 x + kb
    return (int)b;
}

// ------------------------------------------------------------------------------------------
// dK, dV.  256 threads = 4 waves, one workgroup per 64 keys of one (b, hkv), two workgroups per CU
// (two waves per SIMD, from different workgroups, so that one wave's exp / dS arithmetic runs
// beside the other's MFMAs).  The listed q-blocks are walked in steps of 64 query rows.  Wave
// w = (kb, x), kb = w & 1, x = w >> 1:
//   scores     S and dP - delta of the 32 x 32 block (rows 32 x .. +32 of the step, keys 32 kb .. +32),
//              turned into P and dS (bf16, B-operand layout);
//   exchange   the x = 0 wave hands its dS to the x = 1 wave of the same keys through LDS and gets
//              that wave's P;
//   outputs    the x = 0 wave accumulates dV^T += dO^T P over all 64 rows (its own P, then its
//              partner's), the x = 1 wave dK^T += Q^T dS.  Each output row belongs to one wave: no
//              reduction at the end, and 64 accumulator registers per lane instead of 128, which
//              is what lets two workgroups share a CU.
// Q / dO tiles and the per-row scalars are double buffered in LDS; the loads of step v+1 are
// issued at the top of step v.  Two barriers per step: after the exchange writes, and at the end
// (exchange buffer and ring slot free again, next tiles landed).
//
// OWN (D = 64): there both accumulators fit a wave, so every wave keeps dV^T and dK^T of its own 32 rows x
// 32 keys per step: no exchange, no selects between P and dS, one barrier a step, and the two waves of the
// same keys add their halves up once at the end.  V waits in LDS instead of registers (16 of them), which
// is what keeps three workgroups on a CU: with V in registers the kernel spills, and two workgroups are 20 %
// slower.  Blocks of a PARTIAL step that the mask hides from all 32 rows skip everything but S and dP.
// Step by step it is bound by the sum of its MFMAs and its vector work, short columns by the turnover of
// workgroups.  us, exchange -> own rows (one MI355X): causal, 64 x 16 heads, S = 1024: 491 -> 472; window of
// 1024, S = 5000, Hq 16, Hkv 2, B = 4: 222 -> 210; packed documents with ALiBi, S = 16384, 16 heads: 262 -> 252;
// soft-cap, S = 4096, 64 heads: 532 -> 502; relative bias, window 1024, S = 8192: 598 -> 548.
//
// Which form: own rows at D = 64, but for launches that are too uneven for it (own_rows_pay).  A soft-cap on top of a bias, and the rectangles of a canvas, leave too
// few registers at three waves per SIMD (6 to 24 spills: 431 -> 447 us with ALiBi, 350 -> 370 with documents
// and a relative bias; canvas 684 -> 763) and keep the exchange, as does D = 128, whose two accumulators
// are 128 registers.
//
// CUT, neighborhood masks: the walk leaves out the steps that are hidden from all four waves, and a
// wave the vector work and the outputs of its hidden blocks (D = 128, 128 x 128 pixels, tiles of 8 x 8, K = 13, 64 heads:
// 1047 -> 907 us; 100 x 90 row-major, K = 9: 802 -> 771; D = 64 where canvas_cut_pays, 128 x 128, K = 13 548 -> 481, 64 x 64 in Morton order, K = 21,
// 234 -> 204).
//
// LEAVE (kernels of their own; no own rows, other masks; a relative bias with a soft-cap would spill more): the walk leaves out the steps at its front, where the PARTIAL blocks are, that the indices alone hide
// from all four waves: every other column of 64 keys has one at its diagonal if Bq = 128 or Bk = 128, one at the window's far edge, and all have
// one behind a q_len in the first half of its block.  us, B x H = 256, D = 128: causal, S = 1024 214 -> 207,
// S = 300 (512) 79.6 -> 72; window of 512, S = 4096 (64) 218 -> 209; window of 195, soft-cap, Bq = 64, Bk = 128, S = 2427 (512) 673 -> 608;
// causal, ALiBi and soft-cap, 128 x 128, S = 947, Hkv = 2 (48) 261 -> 237; long causal columns 1.00x to 1.02x;
// D = 64, ALiBi and soft-cap, S = 1000 (256) 124 -> 120, 300 (1024) 92.9 -> 80.9, 128 x 128, S = 947, Hkv = 2 (48) 170 -> 161.
// (With own rows such a step has no more than S and dP, and short columns lose by the walk's layout what that is: 16 x 16 heads, S = 1024,
// Bq = 64 99 -> 101, B = 8, S = 500 24.3 -> 25.2.)
template <int D, uint32_t MASK, uint32_t SCORE>
constexpr bool dkdv_own_rows() {
    constexpr bool biased_cap = (SCORE & FLEXATTN_SCORE_SOFTCAP) && (SCORE & (FLEXATTN_SCORE_ALIBI | FLEXATTN_SCORE_REL_BIAS));
    return D == 64 && !PartialMask<MASK>::kCanvas && !biased_cap;
}
// Whether there are kernels that LEAVE (leaving_out_pays: which launches take them).
template <int D, uint32_t MASK, uint32_t SCORE>
constexpr bool dkdv_can_leave() {
    return !dkdv_own_rows<D, MASK, SCORE>() && !PartialMask<MASK>::kCanvas && !((SCORE & FLEXATTN_SCORE_REL_BIAS) && (SCORE & FLEXATTN_SCORE_SOFTCAP));
}
// M0 RULE: this kernel fills LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the
// compiler's back.  Keep every register array in it indexed by compile-time constants (no movrel /
// s_set_gpr_idx code, which would also use M0) and add no other LDS-DMA or M0-based construct.
template <int D, uint32_t MASK, uint32_t SCORE, bool OWN = dkdv_own_rows<D, MASK, SCORE>(), bool CUT = PartialMask<MASK>::kCanvas, Groups GROUPS = Groups::kWhole,
          bool LEAVE = false>
__global__ __launch_bounds__(256, bwd_waves_per_simd<D>()) void bwd_dkdv_kernel(const BwdArgs a) {
    constexpr int TQ = 64;                         // query rows per step
    constexpr int TILE = TQ * D;                   // elements per LDS tile
    constexpr int NKS = D / 16, NDB = D / 32;
    using Loader = WaveTileLoader<D, 4>;
    __shared__ __attribute__((aligned(1024))) bf16 smem[(OWN ? 5 : 4) * TILE];   // 2 x (Q tile, dO tile); OWN: V tile
    __shared__ __attribute__((aligned(1024))) u32x4 s_xchg[OWN ? 1 : 4][2][64];   // [wave][16-row slice][lane]
    __shared__ __attribute__((aligned(256))) float s_row[2][2][TQ];           // [slot][rc | -delta][row]
    constexpr int kListMax = 512;
    __shared__ int s_steps[kListMax + 2];          // the walk of the current head, see below
    __shared__ int s_pos[CUT ? kListMax + 2 : 1], s_count;
    static_assert(!LEAVE || dkdv_can_leave<D, MASK, SCORE>(), "of the waves that exchange P and dS, and of masks that the indices decide");
    __shared__ uint64_t s_left_out;
    using Score = ScoreMod<SCORE, true>;
    __shared__ float s_rel[Score::kRel ? kRelTableMax : 1];   // relative-bias row of the current head
    using Mask = PartialMask<MASK>;
    __shared__ __attribute__((aligned(256))) uint32_t s_tag[2][Mask::kTags ? TQ : 4];   // [slot] tags of a PARTIAL step's queries
    __shared__ u32x2 s_corners[Mask::kCanvas && !Mask::kCells ? 64 : 1];        // key_corners() of the keys
    __shared__ u32x4 s_rect[Mask::kCells ? 64 : 1];                             // cells: the queries that see them

    // workgroup -> (b, hkv, 64-key tile).  The columns of
    // blocks are taken in the BlockMask's work order (longest first; that of the group's first query
    // head where the mask has a plane per head), the 64-key tiles of a column side by side.
    const int sub_k = a.Bk / 64;                   // tiles per column of blocks
    int unit, slot;                                // NC * sub_k slots >= tiles: the last column may be cut short
    int parts;
    if (!kv_unit_of_workgroup<GROUPS>(a, a.NC * sub_k, a.abreast, parts, unit, slot)) return;
    if (a.ds_store) unit = last_unit_first(unit, a.B * a.Hkv * parts);
    const KvHeads<GROUPS> heads(a, parts, unit);
    const int b = unit / a.Hkv, hkv = unit % a.Hkv;
    int col = slot / sub_k;
    if (a.q_order) {
        const int64_t plane0 = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hkv * a.G : 0);
        col = min(max(a.q_order[plane0 * a.NC + col], 0), a.NC - 1);   // clamped: a bad order array stays inside the lists
    }
    const int key_tile = slot % sub_k;             // which 64 keys of the column of blocks
    const int tile = col * sub_k + key_tile;
    const int kv0 = tile * 64;
    if (kv0 >= a.kv_len) return;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = w & 1, x = w >> 1;
    const int kv_lane = kv0 + 32 * kb + l32;

    // K, V fragments of this wave's 32 keys: B operands (column = key, k-slots = dims)
    bf16x8 kf[NKS], vf[OWN ? 1 : NKS];
    {
        // keys past kv_len (last tile of a length that is no multiple of 64) take a copy of the last
        // real key; the mask hides them and they are never stored
        const int kv_ld = min(kv_lane, a.kv_len - 1);
        const bf16* kp = a.K + b * a.k_sb + hkv * a.k_sh + (int64_t)kv_ld * a.k_ss + half * 8;
        const bf16* vp = a.V + b * a.v_sb + hkv * a.v_sh + (int64_t)kv_ld * a.v_ss + half * 8;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            kf[ks] = *(const bf16x8*)(kp + ks * 16);
            if constexpr (!OWN) vf[ks] = *(const bf16x8*)(vp + ks * 16);
        }
    }

    // x = 0: dV^T, x = 1: dK^T (row = dim, column = key); OWN: dV^T here, dK^T in acc_k
    f32x16 acc[NDB], acc_k[OWN ? NDB : 1];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[db][r] = 0.0f;
            if constexpr (OWN) acc_k[db][r] = 0.0f;
        }

    const int sub = a.Bq / TQ;          // steps per BlockMask row block (1 or 2)
    const int sub_shift = sub >> 1;
    const Loader q_loader(a.q_ss, w, lane), do_loader(a.do_ss, w, lane);
    const uint32_t ring = lds_addr(smem);
    const uint32_t wave_row = lds_addr(&s_row[0][w & 1][0]);
    const uint32_t q_bytes = (uint32_t)((a.q_len - 1) * a.q_ss + D) * 2u;
    const uint32_t do_bytes = (uint32_t)((a.q_len - 1) * a.do_ss + D) * 2u;
    const int q_row_bytes = (int)a.q_ss * 2, do_row_bytes = (int)a.do_ss * 2;
    // scores: this wave's 32 rows of the Q tile (the dO tile is one tile further)
    const RowReader<D> row_reader(l32, half, ring + x * 32 * D * 2);
    // OWN: V's 64 rows wait in LDS (rows past kv_len as zeros), this wave's keys at v_lds beside row_reader's offsets
    const uint32_t v_lds = (uint32_t)(4 * TILE + (kb - x) * 32 * D) * 2u;
    if constexpr (OWN) {
        const Loader v_loader(a.v_ss, w, lane);
        v_loader.start(make_rsrc(a.V + b * a.v_sb + hkv * a.v_sh, (uint32_t)((a.kv_len - 1) * a.v_ss + D) * 2u),
                       ring + 4 * TILE * 2, kv0 * (int)a.v_ss * 2);     // (awaited with the first step's tiles)
    }
    // outputs: the tile this wave contracts with (x = 0: dO, x = 1: Q), its own rows first, then
    // its partner's
    // (OWN: its own rows of both tiles, dO one tile behind Q)
    const uint32_t out_tile = ring + (x || OWN ? 0 : TILE * 2);
    const TrReader<D> tr_own(lane, out_tile + x * 32 * D * 2), tr_other(lane, out_tile + (1 - x) * 32 * D * 2);
    const uint32_t row_lds = lds_addr(&s_row[0][0][0]) + (32 * x + 4 * half) * 4;
    const uint32_t xchg_mine = lds_addr(&s_xchg[OWN ? 0 : w][0][lane]), xchg_theirs = lds_addr(&s_xchg[OWN ? 0 : w ^ 2][0][lane]);
    const int q_off = q_offset_of(a.p, b);
    const Mask mask(a.p, b, a.kv_len);
    uint32_t k_tag = 0;
    i32x4 doc_rsrc = {};
    if constexpr (Mask::kDoc) {
        const int32_t* docs = a.p.doc_ids + (int64_t)b * a.p.doc_stride_b;
        k_tag = (uint32_t)docs[min(kv_lane, a.kv_len - 1)];
        doc_rsrc = make_rsrc(docs, (uint32_t)(q_off + a.q_len) * 4u);
    }
    typename Mask::CellBase cell_base = {};
    if constexpr (Mask::kCells) {
        cell_base = mask.base_of_keys(a.p, kv0 + 32 * kb);
        if (x == 0) s_rect[32 * kb + l32] = mask.key_rectangle(kv_lane, cell_base);     // (visible as below)
    } else if constexpr (Mask::kCanvas) {
        if (tid < 64) s_corners[tid] = mask.key_corners(kv0 + tid);     // (visible after the barriers before the first step)
    }
    // Tags of the 64 queries of the step whose first row is q0, into s_tag[slot] (visible after the
    // barrier that makes the step's tiles visible)
    auto make_tags = [&](int slot, int q0) __attribute__((always_inline)) {
        if constexpr (Mask::kDoc) {
            if (w == 0) dma_dword(doc_rsrc, lds_addr(&s_tag[slot][0]), lane * 4, (q_off + q0) * 4);
        }
        if constexpr (Mask::kCanvas) {
            if (w == 2 * slot) s_tag[slot][lane] = mask.query_block_tag(q_off + min(q0 + lane, a.q_len - 1));
        }
    };
    const uint32_t ds_lane = (uint32_t)(w * 1024 + lane * 8);     // this lane's place inside a step of dS in memory (bf16 elements)

    for (int g = heads.first; g < heads.end; ++g) {
        const int hq = hkv * a.G + g;
        const int64_t line = ((int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0)) * a.NC + col;
        const int n_full = a.full_q_num[line], n_part = a.q_num[line];
        const int32_t* full_idx = a.full_q_idx + line * a.NR;
        const int32_t* part_idx = a.q_idx + line * a.NR;
        const int H_all = (n_full + n_part) * sub;  // steps
        if (H_all == 0) continue;
        // dS to memory: where step u of this column's walk goes is ds_col + (pos * sub_k * sub + sidx) * 4096
        // for u = pos * sub + sidx (everything that does not change with u folded into ds_col, so that a
        // step pays a handful of scalar instructions); pos is clamped to the capacity
        bf16* ds_col = nullptr;
        int ds_pos_max = 0;
        if (a.ds_store) {
            const int slot0 = min(max(ldc(a.ds_colbase + line), 0), (int)a.ds_blocks - 1);
            ds_col = a.ds_store + ds_chunk(a, ds_rep(a, b, hq), slot0, key_tile, 0) * 4096;
            ds_pos_max = (int)a.ds_blocks - 1 - slot0;
        }
        const i32x4 q_rsrc = make_rsrc(a.Q + b * a.q_sb + hq * a.q_sh, q_bytes);
        const i32x4 do_rsrc = make_rsrc(a.dO + b * a.do_sb + hq * a.do_sh, do_bytes);
        // waves 0, 2 fetch the rc row, waves 1, 3 the -delta row (the duplicates write the same values)
        const i32x4 row_rsrc =
            make_rsrc(((w & 1) ? a.delta : a.lse2) + ((int64_t)b * a.Hq + hq) * a.q_len, (uint32_t)a.q_len * 4u);
        const Score smod(a.p, hq, a.scale, lds_addr(s_rel));
        // (the previous head's last step ended with a barrier: nobody reads its row any more; the
        // barrier behind the first segment's walk makes this one visible)
        smod.fill_table(tid, 256);

        // The merged list (FULL blocks, then PARTIAL ones) is walked from its END: every workgroup of
        // a head then spends most of its time descending from the last row block, so the workgroups
        // that run side by side on an XCD ask its L2 for the same Q / dO tiles at about the same
        // time.  The walk is laid out in LDS first, kListMax steps at a time -- one entry per step:
        // first query row | 1 if the block is PARTIAL -- so that the main loop finds the next row
        // offset with one LDS read issued a step ahead.  (CUT: bit 1 + w says that the mask
        // hides wave w's block, see canvas_step_bits, and s_pos holds the step's position in the column's walk.)
        for (int seg0 = 0; seg0 < H_all; seg0 += kListMax) {
            int H = min(kListMax, H_all - seg0);
            if constexpr (CUT) {
                // one wave lays the walk out and leaves out the steps that are hidden from all four waves (but
                // for the very first: no segment is empty)
                if (w == 0) {
                    int n = 0;
                    for (int i0 = 0; i0 < H; i0 += 64) {
                        const int i = i0 + lane, u = max(H_all - 1 - (seg0 + i), 0), pos = u / sub, sidx = u - pos * sub;
                        const int blk = pos < n_full ? full_idx[pos] : part_idx[pos - n_full];
                        const int q0 = blk * a.Bq + sidx * TQ;
                        const int bits = pos < n_full ? 0 : canvas_step_bits(a.p, q0, kv0);
                        const bool keep = i < H && (bits != 15 || i == 0);
                        const uint64_t kept = __ballot(keep);
                        if (keep) {
                            const int at = n + __popcll(kept & ((1ull << lane) - 1));
                            s_steps[at] = q0 | (pos >= n_full ? 1 : 0) | (bits << 1);
                            s_pos[at] = u;
                            if (kept >> lane == 1ull) s_steps[at + 1] = s_steps[at];     // (see below; the next 64 overwrite it)
                        }
                        n += __popcll(kept);
                    }
                    if (lane == 0) s_count = n;
                }
                __syncthreads();
                H = __builtin_amdgcn_readfirstlane(s_count);
            }
            // (LEAVE: the steps that are kept of the first 64 move up to the 65th, and the walk starts behind the gap.  Bits 1 .. 5 say by how
            // many places, for that of their dS in memory.)
            for (int i = CUT ? H : tid; i < H; i += 256) {
                const int u = H_all - 1 - (seg0 + i), pos = u / sub, sidx = u - pos * sub;
                const int blk = pos < n_full ? full_idx[pos] : part_idx[pos - n_full];
                const int q0 = blk * a.Bq + sidx * TQ;
                int up = 0;
                if constexpr (LEAVE) {
                    if (i < 64) {
                        const bool hid = seg0 == 0 && pos >= n_full && (q0 >= a.q_len || mask.hidden(q_off + q0, q_off + q0 + TQ - 1, kv0, kv0 + 63));
                        uint64_t out = __ballot(hid);
                        if (__popcll(out) == H) out &= ~1ull;                       // (no segment is empty)
                        if (a.ds_store && __popcll(out) > 31) out = 0;              // (no room in an entry)
                        if (i == 0) s_left_out = out;
                        if ((out >> i) & 1) continue;
                        up = __popcll(out >> i);
                    }
                }
                const int e = (blk * a.Bq + sidx * TQ) | ((up & 31) << 1) | (pos >= n_full ? 1 : 0);
                s_steps[i + up] = e;
                // loads are issued for one step past the end as well (into the free ring slot,
                // never read): it repeats the last step's rows
                if (i + up == H - 1) s_steps[H] = e;
            }
            __syncthreads();
            uint64_t left_out = 0;
            if constexpr (LEAVE)
                left_out = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(s_left_out >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)s_left_out);
            const int first = __popcll(left_out);
            int ld_v = first;                       // step whose loads are issued next
            int u_step = H_all - 1 - seg0 - first;          // position of the current step in the column's walk (counts down)
            int e_next = s_steps[first];
            int q0_of[2];                           // first query row of the step in each ring slot,
            bool part_of[2];                        // and whether its block is PARTIAL
            // (CUT) whether the mask hides this wave's 32 x 32 block, and that of the other wave of its keys
            bool hid_of[2] = {false, false}, hid_other_of[2] = {false, false};
            int up_of[2] = {0, 0};                  // (LEAVE) by how many places it moved

            int ld_q0 = 0;                          // first row of the step being loaded
            constexpr int kLoads = 2 * Loader::NI + 1;      // load instructions per wave and step
            auto load_begin = [&](auto slot_tag) {
                constexpr int SLOT = decltype(slot_tag)::value;
                const int e = __builtin_amdgcn_readfirstlane(e_next);
                ld_q0 = e & ~63;
                q0_of[SLOT] = ld_q0;
                part_of[SLOT] = e & 1;
                if constexpr (CUT) {
                    hid_of[SLOT] = (e >> (1 + w)) & 1;
                    hid_other_of[SLOT] = (e >> (1 + (w ^ 2))) & 1;
                }
                if constexpr (LEAVE) up_of[SLOT] = (e >> 1) & 31;
                e_next = s_steps[++ld_v];
            };
            // piece P of the loads of a step: NI for the Q tile, NI for the dO tile, one row of scalars
            auto load_piece = [&](auto slot_tag, auto piece_tag) {
                constexpr int SLOT = decltype(slot_tag)::value, P = decltype(piece_tag)::value;
                if constexpr (P < Loader::NI)
                    q_loader.template start_one<P>(q_rsrc, ring + SLOT * 2 * (TILE * 2), ld_q0 * q_row_bytes);
                else if constexpr (P < 2 * Loader::NI)
                    do_loader.template start_one<P - Loader::NI>(do_rsrc, ring + (SLOT * 2 + 1) * (TILE * 2),
                                                                 ld_q0 * do_row_bytes);
                else
                    dma_dword(row_rsrc, wave_row + SLOT * 2 * TQ * 4, lane * 4, ld_q0 * 4);
            };
            auto load_step = [&](auto slot_tag) {   // all at once (prologue)
                load_begin(slot_tag);
                static_for<0, kLoads>([&](auto piece_tag) { load_piece(slot_tag, piece_tag); });
            };
            // this lane's 16 row scalars of a step: rows 8 rg + 4 half + {0..3} of the wave's 32
            auto read_row4 = [&](int slot, int which, int rg) {
                return *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)(
                    row_lds + (uint32_t)((slot * 2 + which) * TQ + 8 * rg) * 4);
            };
            auto read_rows = [&](int slot, int which, f32x4 (&out)[4]) {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) out[rg] = read_row4(slot, which, rg);
            };

            // this wave's dS of the step to memory, as it sits in the registers
            auto store_ds = [&](int u_at, u32x4 c0, u32x4 c1) {
                const int u = CUT ? __builtin_amdgcn_readfirstlane(u_at) : u_at, pos = u >> sub_shift;
                bf16* dst = ds_col + (int64_t)(min(pos, ds_pos_max) * (sub_k * sub) + (u - (pos << sub_shift))) * 4096;
                // (written once, read once by another kernel much later: no reason to keep it in a cache)
                __builtin_nontemporal_store(c0, (u32x4*)(dst + ds_lane));
                __builtin_nontemporal_store(c1, (u32x4*)(dst + ds_lane + 512));
            };
            if (LEAVE && a.ds_store)                // dS of the steps left out
                for (uint64_t rest = left_out; rest; rest &= rest - 1) store_ds(H_all - 1 - __builtin_ctzll(rest), u32x4{}, u32x4{});
            load_step(std::integral_constant<int, 0>{});
            if (part_of[0]) make_tags(0, q0_of[0]);
            wait_vmem();
            __syncthreads();

            // the next step's tiles must have landed; the two dS stores, the youngest vector-memory
            // operations of the step (the counter retires in issue order), may still be under way
            auto end_step = [&](bool stored) {
                if (stored) wait_vmem_but<2>();
                else wait_vmem();
                __syncthreads();
            };

            // ---- one step; SLOT = v & 1 is compile-time so that every LDS access is "VGPR + immediate"
            auto step = [&](auto slot_tag) {
                constexpr int SLOT = decltype(slot_tag)::value;
                constexpr uint32_t q_cur = SLOT * 2 * (TILE * 2), do_cur = q_cur + TILE * 2;
                // step v+1 (or the dummy past the end); its loads are issued between the MFMAs below: a
                // wave waits on every load instruction until the memory pipe has taken it
                constexpr std::integral_constant<int, SLOT ^ 1> ld_slot{};
                load_begin(ld_slot);
                if (part_of[SLOT ^ 1]) make_tags(SLOT ^ 1, q0_of[SLOT ^ 1]);
                const int q_first = q0_of[SLOT] + 32 * x;
                // (wave-uniform) does the mask touch this wave's 32 x 32 block at all?
                const bool partial = part_of[SLOT] && !mask.full(q_off + q_first, q_off + q_first + 31, kv0 + 32 * kb,
                                                                 kv0 + 32 * kb + 31);

                // a block that the mask hides from all of its rows adds nothing (zeros in the stored dS)
                bool hid = false;
                if constexpr (CUT) hid = hid_of[SLOT];
                else if constexpr (OWN) hid = part_of[SLOT] && mask.hidden(q_off + q_first, q_off + q_first + 31, kv0 + 32 * kb, kv0 + 32 * kb + 31);
                // (a canvas' here, while the score accumulators do not take registers yet)
                typename Mask::Bits bits = {};
                typename Mask::CellMasks cells = {{~0u, ~0u}, ~0u};
                if constexpr (Mask::kCanvas && !Mask::kCells) {
                    if (partial && !hid) bits = mask.match_queries(&s_tag[SLOT][32 * x], s_corners[32 * kb + l32], half);
                }
                // scores
                f32x4 nd[4], rcv4[4];
                read_rows(SLOT, 1, nd);
                f32x16 sacc, dpacc;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sacc[r] = 0.0f;
                    dpacc[r] = nd[r >> 2][r & 3];    // dP - delta comes out of the accumulation
                }
                {   // operand fragments are read PF MFMAs ahead of their use
                    constexpr int NM = 2 * NKS, PF = OWN ? 2 : 4;
                    auto frag = [&](int m) { return row_reader.read((m & 1) ? do_cur : q_cur, 0, m >> 1); };
                    bf16x8 fr[NM], vr[NKS];
#pragma unroll
                    for (int m = 0; m < PF; ++m) fr[m] = frag(m);
                    static_for<0, NM>([&](auto m_tag) {
                        constexpr int m = decltype(m_tag)::value;
                        if constexpr (m + PF < NM) fr[m + PF] = frag(m + PF);
                        if constexpr (OWN && !(m & 1)) vr[m >> 1] = row_reader.read(v_lds, 0, m >> 1);
                        if (m & 1) dpacc = mfma32(fr[m], OWN ? vr[m >> 1] : vf[OWN ? 0 : m >> 1], dpacc);
                        else sacc = mfma32(fr[m], kf[m >> 1], sacc);
                        static_for<0, kLoads>([&](auto piece_tag) {
                            if constexpr (decltype(piece_tag)::value * NM / kLoads == m) load_piece(ld_slot, piece_tag);
                        });
                        __builtin_amdgcn_sched_barrier(0);
                    });
                }
                if constexpr (!OWN) read_rows(SLOT, 0, rcv4);
                // relative bias: one value for the whole 32 x 32 block unless it lies near the diagonal
                float rel_uni;
                const bool rel_is_uni = smod.rel_uniform(q_off + q_first - (kv0 + 32 * kb + 31),
                                                         q_off + q_first + 31 - (kv0 + 32 * kb), rel_uni);
                if (partial && !Mask::kCanvas) {
                    bits = mask.key_bits(kv_lane, q_off + q_first + 4 * half);
                    if constexpr (Mask::kDoc) Mask::match_documents(bits, &s_tag[SLOT][32 * x], k_tag, l32, half, false);
                }
                u32x4 pk[2] = {}, dsk[2] = {};
                if (!hid) {
                    if constexpr (Mask::kCells) {
                        // (the lane's number is asked for again: what is held of it over the loop spills, and a reload waits for the next tiles)
                        const int again = lane_again();
                        if (partial) cells = mask.cell_masks(s_rect[32 * kb + (again & 31)], &s_tag[SLOT][32 * x], cell_base, again >> 5, true);
                    }
                    constexpr int kAhead = Score::kRel || Score::kCap ? 0 : 2;
                    if constexpr (OWN) {
#pragma unroll
                        for (int c4 = 0; c4 < kAhead; ++c4) rcv4[c4] = read_row4(SLOT, 0, c4);
                    }
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4) {
                        float sv[4], rcv[4], gr[4], pe[4], ds[4];
                        // alibi / rel-bias need q - kv = dq0 + 8 (r >> 2) + (r & 3); the soft-cap and the plain score do not
                        using RelPos = typename decltype(smod)::RelPos;
                        constexpr bool kNeedsPos = Score::kAlibi || Score::kRel;
                        const int dq0 = kNeedsPos ? q_off + q_first + 4 * half - kv_lane : 0;
                        const float abase = smod.alibi_base(dq0);
                        auto rel = [&](int r) __attribute__((always_inline)) {
                            return kNeedsPos ? RelPos(dq0, abase, 8 * (r >> 2) + (r & 3)) : RelPos(0);
                        };
                        // (OWN: a quad of row constants, two ahead of its use; for four there are no registers, nor with a relative bias or a
                        // soft-cap for any.  us, dK/dV, where they are used -> two ahead: no mask, S = 1600, 36 heads 67 -> 65, causal, S = 2000,
                        // 30 heads 52 -> 51, ALiBi, S = 2048, 128 heads 180 -> 177 (2 spills); soft-cap, 5 and 6 spills, causal, S = 600, 256 heads 59 ->
                        // 61, S = 8192, 32 heads 683 -> 678, window of 300, S = 4096, 32 heads 52 -> 54)
                        if constexpr (OWN) {
                            if (c4 + kAhead < 4) rcv4[c4 + kAhead] = read_row4(SLOT, 0, c4 + kAhead);
                        }
                        const RelPos dqk[4] = {rel(4 * c4), rel(4 * c4 + 1), rel(4 * c4 + 2), rel(4 * c4 + 3)};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = 4 * c4 + i;
                            sv[i] = sacc[r];
                            rcv[i] = rcv4[r >> 2][r & 3];
                        }
                        if (rel_is_uni) smod.template p_with_grad4<true>(sv, dqk, rcv, gr, pe, rel_uni);
                        else smod.template p_with_grad4<false>(sv, dqk, rcv, gr, pe);
                        if (partial && !Mask::kCells) {
                            asm volatile("" ::: "memory");   // keep this a (scalar, rarely taken) branch
                            // (a masked P makes dS vanish with it.  Rows past q_len hold zeros in Q and dO: whatever
                            // the mask says there adds nothing)
                            if constexpr (Mask::kCanvas) {
                                mask.keep_queries(bits, &s_tag[SLOT][32 * x], c4, half, pe);
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; ++i) pe[i] = keep_or_zero(Mask::keep(bits, 4 * c4 + i), pe[i]);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) ds[i] = pe[i] * gr[i] * dpacc[4 * c4 + i];
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const int e = 2 * c4 + i;
                            pk[e >> 2][e & 3] = pack_bf16(pe[2 * i], pe[2 * i + 1]);
                            dsk[e >> 2][e & 3] = pack_bf16(ds[2 * i], ds[2 * i + 1]);
                            if constexpr (Mask::kCells) {
                                pk[e >> 2][e & 3] = cells.pair(pk[e >> 2][e & 3], e);
                                dsk[e >> 2][e & 3] = cells.pair(dsk[e >> 2][e & 3], e);
                            }
                        }
                    }
                }
                // (wave-uniform; the blocks a canvas hides are not read back, see CANVAS in bwd_stored.h)
                const bool stored = a.ds_store && !(CUT && hid);
                if (stored) store_ds(CUT ? s_pos[ld_v - 2] : u_step + up_of[SLOT], dsk[0], dsk[1]);
                --u_step;
                if constexpr (OWN) {
                    // outputs: dV^T += dO^T P and dK^T += Q^T dS over this wave's own 32 rows
                    if (!hid) {
                        constexpr int NM = 4 * NDB, PF = 2;       // MFMAs: [slice c][block db][dV, dK]
                        auto frag = [&](int m) {
                            return tr_own.read((m & 1) ? q_cur : do_cur, 16 * ((m >> 1) / NDB), (m >> 1) % NDB);
                        };
                        bf16x8 fr[NM];
#pragma unroll
                        for (int m = 0; m < PF; ++m) fr[m] = frag(m);
#pragma unroll
                        for (int m = 0; m < NM; ++m) {
                            if (m + PF < NM) fr[m + PF] = frag(m + PF);
                            const int c = (m >> 1) / NDB, db = (m >> 1) % NDB;
                            if (m & 1) acc_k[db] = mfma32(fr[m], __builtin_bit_cast(bf16x8, dsk[c]), acc_k[db]);
                            else acc[db] = mfma32(fr[m], __builtin_bit_cast(bf16x8, pk[c]), acc[db]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    end_step(stored);
                    return;
                }
                // exchange: keep what this wave's output needs, hand over the other
                u32x4 own[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    own[c] = x ? dsk[c] : pk[c];
                    *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(xchg_mine + c * 1024) = x ? pk[c] : dsk[c];
                }
                // outputs: contraction over this wave's own 32 rows (while the exchange settles), then,
                // after the barrier, over its partner's
                constexpr uint32_t slot_off = SLOT * 2 * (TILE * 2);
                constexpr int NMH = 2 * NDB, PF = 4;          // MFMAs per half: [slice c][block db]
                u32x4 theirs[2];
                auto out_half = [&](const TrReader<D>& reader, uint32_t further, const u32x4 (&bop)[2]) {
                    auto frag = [&](int m) { return reader.read(slot_off + further, 16 * (m / NDB), m % NDB); };
                    bf16x8 fr[NMH];
#pragma unroll
                    for (int m = 0; m < PF; ++m) fr[m] = frag(m);
#pragma unroll
                    for (int m = 0; m < NMH; ++m) {
                        if (m + PF < NMH) fr[m + PF] = frag(m + PF);
                        acc[m % NDB] = mfma32(fr[m], __builtin_bit_cast(bf16x8, bop[m / NDB]), acc[m % NDB]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (!hid) out_half(tr_own, 0u, own);
                __syncthreads();
                if (!hid_other_of[SLOT]) {
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        theirs[c] = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(xchg_theirs + c * 1024);
                    // (CUT: tr_other's addresses are made here, it has no registers to keep them)
                    uint32_t further = 0;
                    if constexpr (CUT) {
                        further = (uint32_t)((1 - 2 * x) * 32 * D * 2);
                        asm volatile("" : "+s"(further));
                    }
                    out_half(CUT ? tr_own : tr_other, further, theirs);
                }
                end_step(stored);
            };

            int v = first;
            for (; v + 1 < H; v += 2) {
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
            }
            if (v < H) step(std::integral_constant<int, 0>{});
        }
    }

    // ---- OWN: the two waves of the same keys add up, the x = 0 wave dV^T, the x = 1 wave dK^T (the ring is
    // free: the last step ended with a barrier)
    if constexpr (OWN) {
        wait_vmem();        // (a column without a step has V's load still under way, and must not end before it)
        f32x4* give = (f32x4*)smem + w * (NDB * 4 * 64) + lane;
        const f32x4* take = (const f32x4*)smem + (w ^ 2) * (NDB * 4 * 64) + lane;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = x ? acc[db][4 * rg + i] : acc_k[db][4 * rg + i];
                give[(db * 4 + rg) * 64] = v;
            }
        __syncthreads();
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const f32x4 v = take[(db * 4 + rg) * 64];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[db][4 * rg + i] = (x ? acc_k[db][4 * rg + i] : acc[db][4 * rg + i]) + v[i];
            }
    }
    // ---- dV (x = 0) or dK (x = 1, with the scale and the score_mod's gradient factor), bf16
    {
        if (GROUPS != Groups::kWhole && heads.apart) {      // (kv_parts_sum_kernel scales)
            if (kv_lane >= a.kv_len) return;
            float* out = heads.sums(a, unit, x, D) + (int64_t)kv_lane * D;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    *(f32x4*)(out + db * 32 + 8 * rg + 4 * half) = f32x4{acc[db][4 * rg], acc[db][4 * rg + 1], acc[db][4 * rg + 2], acc[db][4 * rg + 3]};
            return;
        }
        // (asked once the addresses are there: us, D = 64, asked here / there, window of 300, S = 1000, 16 heads 12.6 / 12.0, 16 x 200 x 16 20.6 / 20.3, documents, 8 x 500 x 16 24.6 / 23.6;
        // ALiBi would spill up to 4 registers more)
        if (Score::kAlibi && kv_lane >= a.kv_len) return;
        const float oscale = x ? a.scale * ScoreMod<SCORE>::grad_scale() : 1.0f;
        bf16* op = x ? a.dK + b * a.dk_sb + hkv * a.dk_sh + (int64_t)kv_lane * a.dk_ss
                     : a.dV + b * a.dv_sb + hkv * a.dv_sh + (int64_t)kv_lane * a.dv_ss;
        if (!Score::kAlibi && kv_lane >= a.kv_len) return;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                u32x2 o;
                o[0] = pack_bf16(acc[db][4 * rg] * oscale, acc[db][4 * rg + 1] * oscale);
                o[1] = pack_bf16(acc[db][4 * rg + 2] * oscale, acc[db][4 * rg + 3] * oscale);
                *(u32x2*)(op + db * 32 + 8 * rg + 4 * half) = o;
            }
    }
}

// ------------------------------------------------------------------------------------------
// Sums along the diagonals q - k of a 32 x 32 block whose lane (q, half) holds v[r] at k = elem_pos(r) + 4 half:
// lane 31 + q - k receives the sum of that diagonal.  Each half adds its keys up from one end to the
// other, moving what it has by as many lanes as the key moves, so that a diagonal stays in one lane: the
// first half towards the upper lanes, the second towards the lower ones.
// Bound by its chain of dependent adds, about 500 clocks a block.  (An LDS atomic per element, as the captured
// sums did, took 139 clocks of the CU each, 2200 a block.  us of the captured kernel, before -> after: relative
// bias of 256, S = 8192, window 1024, D = 64: 482 -> 146; S = 32768, window 4096, D = 128: 7610 -> 5120.)
template <int N, bool UP>
__device__ __forceinline__ float move_lanes(float v) {
    if constexpr (N == 0) return v;
    // wave_shr:1 / wave_shl:1, zeros move in
    else return move_lanes<N - 1, UP>(__builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), UP ? 0x138 : 0x130, 0xf, 0xf, true)));
}
__device__ __forceinline__ float diagonal_sums(const f32x16& v, int half) {
    float up = half ? 0.0f : v[0], down = half ? v[15] : 0.0f;
    static_for<1, 16>([&](auto r_tag) {
        constexpr int r = decltype(r_tag)::value;
        up = move_lanes<elem_pos(r) - elem_pos(r - 1), true>(up) + (half ? 0.0f : v[r]);
        down = move_lanes<elem_pos(16 - r) - elem_pos(15 - r), false>(down) + (half ? v[15 - r] : 0.0f);
    });
    return move_lanes<4, true>(up) + move_lanes<5, false>(down);     // q - k is at lane 27 + q - k, 36 + q - k
}

// dQ.  NW waves, each owning 32 query rows of the row of blocks; structure of the forward kernel.
// CAPTURED: the same walk and the same dS, but instead of dQ the kernel sums what the score_mod's
// captured tensors receive: dS * (q_idx - kv_idx) for the ALiBi bias of the head, dS per table entry
// for the relative bias (the factor ScoreMod::grad_scale() is applied by the reduction that follows).
// One partial result per workgroup; the blocks whose every pair falls on the table's last (or first)
// entry are summed in registers, the others along their diagonals, one LDS atomic per block and diagonal.
// M0 RULE: this kernel fills LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the
// compiler's back.  Keep every register array in it indexed by compile-time constants (no movrel /
// s_set_gpr_idx code, which would also use M0) and add no other LDS-DMA or M0-based construct.
//
// SKIP: hidden blocks are left out, which means not to spread the loads of the next tile over the MFMAs of this one.
// Four waves at D = 64 (window of 1024, S = 5000: 130 -> 124 us; canvas 100 x 90, K = 9, row-major: 349 -> 290; masks that hide a diagonal or nothing
// too: causal, S = 520, 96 heads 18.1 -> 16.9, no mask, S = 100, 256 heads 12.2 -> 11.2, S = 1300, 42 heads 38.8 -> 37.2, but with a soft-cap, S = 1000,
// 48 heads 41.2 -> 42.1), not with two (tiles of 8 x 8, K = 13: 348 -> 374) nor at D = 128.
template <int D, int NW>
constexpr bool dq_skips_hidden() {
    return D == 64 && NW == 4;
}
// PAIRS: a workgroup takes 64 rows; the four waves are two slices of 32 rows times the two key halves of every tile, and the two waves
// of the same rows add up at the end.  Two waves, one per slice, leave LDS for one (D = 128) or 2.5 (D = 64) waves per SIMD;
// four that share the tiles make it two and three (dq_pairs_pay has the times, and where the halves of rows of blocks of 128 take this form).
// MIXED: some rows of blocks whole (dq_halved_rows).
template <int D, int NW, uint32_t MASK, uint32_t SCORE, bool CAPTURED = false, bool SKIP = dq_skips_hidden<D, NW>(), bool PAIRS = false, bool MIXED = false>
__global__ __launch_bounds__(NW * 64, bwd_waves_per_simd<D>()) void bwd_dq_kernel(const BwdArgs a) {
    static_assert(!PAIRS || (NW == 4 && SKIP), "two row slices times two key halves");
    static_assert(!MIXED || (PAIRS && !CAPTURED), "halves and whole rows");
    constexpr int kShortTiles = 10;                                  // MIXED: longest rows of no more stay whole
    constexpr int kSlices = PAIRS ? NW / 2 : NW;
    const int Bq = MIXED ? 128 : PAIRS ? a.Bq : kSlices * 32;
    constexpr int TILE = 64 * D;
    __shared__ __attribute__((aligned(1024))) bf16 smem[4 * TILE];   // K(even), K(odd), V(even), V(odd)
    constexpr int kTabAlibi = 1024;                                  // the table has at most 1024 entries
    __shared__ float s_tab[CAPTURED ? kTabAlibi + 1 : 1];            // relative-bias entries, then the ALiBi sum
    __shared__ float s_rel[ScoreMod<SCORE>::kRel ? kRelTableMax : 1]; // relative-bias row of the head (values)
    using Mask = PartialMask<MASK>;
    __shared__ __attribute__((aligned(256))) uint32_t s_tag[2][Mask::kTags ? 64 : 4];   // tags of a PARTIAL tile's keys (even, odd)
    __shared__ uint8_t s_hidden[Mask::kCanvas && SKIP ? kHiddenTiles : 1];           // CanvasBlocks::hidden_bits of the first tiles

    int unit, rem;
    UnitSets abreast = a.abreast;
    if constexpr (Mask::kDoc) abreast = abreast_if_long(abreast, a.B * a.Hkv, longest_row(a.kv_order, a.full_kv_num, a.kv_num, 0, a.NR, a.Bk / 64));
    if (!unit_of_workgroup(a.B * a.Hkv, a.G * (MIXED ? a.NR + a.halved : a.NR * (PAIRS ? Bq / 64 : 1)), abreast, unit, rem)) return;
    unit = last_unit_first(unit, a.B * a.Hkv);
    int slice = 0;                                                   // PAIRS: which 64 rows of the block
    bool whole = false;                                              // MIXED: 32 rows and all keys to a wave
    if constexpr (MIXED) {
        const int64_t rows = ((int64_t)(a.bm_Bm > 1 ? unit / a.Hkv : 0) * a.bm_Hm + (a.bm_Hm > 1 ? unit % a.Hkv * a.G : 0)) * a.NR;
        if (!half_or_row(a.kv_order, a.full_kv_num, a.kv_num, rows, a.NR, a.G, a.Bk / 64, a.halved, kShortTiles, rem, slice, whole)) return;
    } else if constexpr (PAIRS) {
        slice = rem & (Bq / 64 - 1);
        rem >>= Bq == 128 ? 1 : 0;
    }
    const int g = rem % a.G;
    const int b = unit / a.Hkv, hkv = unit % a.Hkv, hq = hkv * a.G + g;
    const int64_t plane = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0);
    const int row = a.kv_order ? min(max(ldc(a.kv_order + plane * a.NR + rem / a.G), 0), a.NR - 1) : a.NR - 1 - rem / a.G;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int my_slice = PAIRS && !whole ? w & 1 : w, my_keys = PAIRS && !whole ? w >> 1 : 0;
    const int first_row = row * Bq + 64 * slice, wave_rows = first_row + my_slice * 32;
    if (PAIRS && !CAPTURED && first_row >= a.q_len) return;
    const int q_row = wave_rows + l32;

    const int64_t line = ((int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0)) * a.NR + row;
    const int n_full = ldc(a.full_kv_num + line), n_part = ldc(a.kv_num + line);
    const int sub = a.Bk / 64;
    const int T = (n_full + n_part) * sub;

    bf16* dq_ptr = a.dQ + b * a.dq_sb + hq * a.dq_sh + (int64_t)q_row * a.dq_ss;
    // rows past q_len are computed on a copy of the last real row and never stored
    const bool real_row = q_row < a.q_len;
    const int q_ld = min(q_row, a.q_len - 1);
    const int64_t cap_slot = ((int64_t)b * a.Hq + hq) * a.NR + row;
    if (T == 0) {
        if constexpr (CAPTURED) {
            if constexpr (ScoreMod<SCORE>::kRel)
                for (int i = tid; i < a.p.rel_len; i += NW * 64) a.cap_rel[cap_slot * a.p.rel_len + i] = 0.0f;
            if constexpr (ScoreMod<SCORE>::kAlibi)
                if (tid == 0) a.cap_alibi[cap_slot] = 0.0f;
        } else if (real_row) {
            for (int d0 = half * 8; d0 < D; d0 += 16) *(u32x4*)(dq_ptr + d0) = u32x4{0, 0, 0, 0};
            if (a.make_delta && half == 0) {            // (no column of blocks lists these rows)
                const int64_t rowi = ((int64_t)b * a.Hq + hq) * a.q_len + q_row;
                a.delta[rowi] = 0.0f;
                a.lse2[rowi] = -INFINITY;
            }
        }
        return;
    }
    if constexpr (CAPTURED)
        for (int i = tid; i <= kTabAlibi; i += NW * 64) s_tab[i] = 0.0f;   // before the first barrier below

    bf16x8 qf[D / 16], dof[D / 16];
    {
        const bf16* qp = a.Q + b * a.q_sb + hq * a.q_sh + (int64_t)q_ld * a.q_ss + half * 8;
        const bf16* dp = a.dO + b * a.do_sb + hq * a.do_sh + (int64_t)q_ld * a.do_ss + half * 8;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            qf[ks] = *(const bf16x8*)(qp + ks * 16);
            dof[ks] = *(const bf16x8*)(dp + ks * 16);
        }
    }
    const int64_t rowi = ((int64_t)b * a.Hq + hq) * a.q_len + q_ld;
    float lse2, neg_delta;
    if (CAPTURED || a.make_delta) {
        row_scalars<D, SCORE>(a, b, hq, q_ld, half, dof, lse2, neg_delta);
        if (!CAPTURED && real_row && half == 0 && my_keys == 0) {
            a.delta[rowi] = neg_delta;
            a.lse2[rowi] = lse2;
        }
    } else {
        lse2 = a.lse2[rowi];
        neg_delta = a.delta[rowi];
    }
    const i32x4 k_rsrc = make_rsrc(a.K + b * a.k_sb + hkv * a.k_sh, (uint32_t)((a.kv_len - 1) * a.k_ss + D) * 2u);
    const i32x4 v_rsrc = make_rsrc(a.V + b * a.v_sb + hkv * a.v_sh, (uint32_t)((a.kv_len - 1) * a.v_ss + D) * 2u);
    const int k_row_bytes = (int)a.k_ss * 2, v_row_bytes = (int)a.v_ss * 2;
    const ScoreMod<SCORE, true> smod(a.p, hq, a.scale, lds_addr(s_rel));
    smod.fill_table(tid, NW * 64);                  // visible after the prologue's barrier
    const int q_pos = q_ld + q_offset_of(a.p, b);   // as the mods see it
    const Mask mask(a.p, b, a.kv_len);
    uint32_t q_tag = 0;
    bool scattered = false;
    i32x4 doc_rsrc = {};
    if constexpr (Mask::kDoc) {
        const int32_t* docs = a.p.doc_ids + (int64_t)b * a.p.doc_stride_b;
        q_tag = (uint32_t)docs[q_pos];
        doc_rsrc = make_rsrc(docs, (uint32_t)a.kv_len * 4u);
    }
    typename Mask::CellBase cell_base = {};
    u32x4 q_rect = {};
    if constexpr (Mask::kCells) {
        cell_base = mask.base_of_queries(a.p, wave_rows);
        q_rect = mask.query_rectangle(q_pos, cell_base);
    } else if constexpr (Mask::kCanvas) {
        q_tag = mask.query_pixel(q_pos);
    }
    auto make_tags = [&](int buf, int kv0, int turn) __attribute__((always_inline)) {   // as in the forward
        if constexpr (Mask::kDoc) {
            if (w == 0) dma_dword(doc_rsrc, lds_addr(&s_tag[buf][0]), lane * 4, kv0 * 4);
        }
        if constexpr (Mask::kCanvas) {
            if (w == (turn & (NW - 1))) s_tag[buf][lane] = mask.key_pixel(min(kv0 + lane, a.kv_len - 1));
        }
    };

    TileWalk<> walk(a.full_kv_idx + line * a.NC, a.kv_idx + line * a.NC, n_full, n_part, sub, a.Bk);
    const WaveTileLoader<D, NW> k_loader(a.k_ss, w, lane), v_loader(a.v_ss, w, lane);
    auto load_tiles = [&](int buf, int kv0) {
        k_loader.start(k_rsrc, lds_addr(smem) + buf * (TILE * 2), kv0 * k_row_bytes);
        v_loader.start(v_rsrc, lds_addr(smem) + (2 + buf) * (TILE * 2), kv0 * v_row_bytes);
    };
    const RowReader<D> row_reader(l32, half, lds_addr(smem) + my_keys * 32 * D * 2);
    const TrReader<D> tr_reader(lane, lds_addr(smem) + my_keys * 32 * D * 2);
    // a row past q_len must add nothing to the sums
    const float rc = (CAPTURED && !real_row) ? -INFINITY : lse2;
    const int q_wave_min = wave_rows + q_offset_of(a.p, b);   // smallest q_idx of this wave's rows
    float g_alibi = 0.0f, g_hi = 0.0f, g_lo = 0.0f;

    f32x16 dq[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[db][r] = 0.0f;

    // a wave leaves out the blocks of 32 keys that the mask hides from all of its rows, and all if it has no row
    const bool no_row = wave_rows >= a.q_len;
    if constexpr (SKIP && Mask::kCanvas) fill_hidden_tiles<kSlices, NW * 64>(s_hidden, a.p, a.kv_idx + line * a.NC, n_full, T, sub, a.Bk, first_row, tid);
    auto hidden_block = [&](int t, bool partial, int kv, int kvb) __attribute__((always_inline)) {
        if constexpr (Mask::kCanvas) return no_row || (t < kHiddenTiles && ((__builtin_amdgcn_readfirstlane((int)s_hidden[t]) >> (2 * my_slice + kvb)) & 1));
        else return no_row || (partial && mask.hidden(q_wave_min, q_wave_min + 31, kv, kv + 31));
    };
    bool part_next = false;
    int kv0 = walk.next(part_next);
    load_tiles(0, kv0);
    if (part_next) make_tags(0, kv0, 0);
    wait_vmem();
    __syncthreads();
    if constexpr (Mask::kDoc) scattered = Mask::scattered_ids(q_tag);               // (not earlier: q_tag would be waited for)

    // One tile on buffer BUF (compile-time, so that every LDS read is "VGPR + immediate"); half_tag: the wave's half of it alone.
    auto step = [&](int t, auto buf_tag, auto half_tag) __attribute__((always_inline)) {
        constexpr int BUF = decltype(buf_tag)::value;
        const int kv0_cur = kv0;
        const bool partial = part_next;
        // K(t+1), V(t+1) go to buffer BUF ^ 1, last read in step t-1.  Their loads are issued piece by
        // piece between the first MFMAs below: a wave waits on every load instruction until the
        // memory pipe has taken it.
        const bool ld = t + 1 < T;
        if (ld) {
            kv0 = walk.next(part_next);
            if (part_next) make_tags(BUF ^ 1, kv0, t + 1);
        }
        constexpr uint32_t kt = BUF * (TILE * 2), vt = (2 + BUF) * (TILE * 2);
        using L = WaveTileLoader<D, NW>;
        // (MIXED at D = 64: with four read ahead 7 registers spill, ALiBi, S = 16384, 16 heads 158 -> 176 us)
        constexpr int NKS = D / 16, NDB = D / 32, PF = MIXED && D == 64 ? 3 : 4;

        if constexpr (SKIP) {
            if (ld) load_tiles(BUF ^ 1, kv0);
        }
        static_for<0, decltype(half_tag)::value ? 1 : 2>([&](auto kvb_tag) __attribute__((always_inline)) {
            constexpr int kvb = decltype(kvb_tag)::value;
            const int block = decltype(half_tag)::value ? my_keys : kvb;        // (the readers know my_keys)
            if constexpr (SKIP) {
                if (hidden_block(t, partial, kv0_cur + 32 * block, block)) return;
            }
            // S^T = K Q^T and dP^T = V dO^T for 32 keys; operand fragments read PF MFMAs ahead
            f32x16 sacc, dpacc;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sacc[r] = 0.0f;
                dpacc[r] = neg_delta;        // dP - delta comes out of the accumulation
            }
            {
                constexpr int NM = 2 * NKS, NP = 2 * L::NI;
                auto frag = [&](int m) { return row_reader.read((m & 1) ? vt : kt, kvb * 32, m >> 1); };
                bf16x8 fr[NM];
#pragma unroll
                for (int m = 0; m < PF; ++m) fr[m] = frag(m);
                static_for<0, NM>([&](auto m_tag) {
                    constexpr int m = decltype(m_tag)::value;
                    if constexpr (m + PF < NM) fr[m + PF] = frag(m + PF);
                    if (m & 1) dpacc = mfma32(fr[m], dof[m >> 1], dpacc);
                    else sacc = mfma32(fr[m], qf[m >> 1], sacc);
                    if constexpr (kvb == 0 && !SKIP) {
                        static_for<0, NP>([&](auto p_tag) {
                            constexpr int p = decltype(p_tag)::value;
                            if constexpr (p * NM / NP == m) {
                                if (ld) {
                                    if constexpr (p < L::NI)
                                        k_loader.template start_one<p>(k_rsrc, lds_addr(smem) + (BUF ^ 1) * (TILE * 2),
                                                                       kv0 * k_row_bytes);
                                    else
                                        v_loader.template start_one<p - L::NI>(
                                            v_rsrc, lds_addr(smem) + (2 + (BUF ^ 1)) * (TILE * 2), kv0 * v_row_bytes);
                                }
                            }
                        });
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            // q_idx - kv_idx of element r is dq0 - 8 (r >> 2) - (r & 3)
            const int dq0 = q_pos - (kv0_cur + block * 32 + 4 * half);
            const float abase = smod.alibi_base(dq0);
            float rel_uni;
            const int kvs_blk = kv0_cur + block * 32;
            const bool rel_is_uni = smod.rel_uniform(q_wave_min - (kvs_blk + 31), q_wave_min + 31 - kvs_blk, rel_uni);
            auto rel = [&](int r) __attribute__((always_inline)) {
                return typename decltype(smod)::RelPos(dq0, abase, -(8 * (r >> 2) + (r & 3)));
            };
            if (rel_is_uni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float gr;
                    const float pe = smod.template p_with_grad<true>(sacc[r], rel(r), rc, gr, rel_uni);
                    dpacc[r] = pe * gr * dpacc[r];
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float gr;
                    const float pe = smod.template p_with_grad<false>(sacc[r], rel(r), rc, gr);
                    dpacc[r] = pe * gr * dpacc[r];
                }
            }
            typename Mask::CellMasks cells = {{~0u, ~0u}, ~0u};
            if constexpr (Mask::kCells) {
                if (partial) cells = mask.cell_masks(q_rect, &s_tag[BUF][block * 32], cell_base, half, kvs_blk <= mask.kv_last);
            } else if (partial && !mask.full(q_wave_min, q_wave_min + 31, kvs_blk, kvs_blk + 31)) {
                asm volatile("" ::: "memory");   // keep this a branch
                typename Mask::Bits bits = mask.row_bits(q_pos, kvs_blk + 4 * half);
                if constexpr (Mask::kDoc) Mask::match_documents(bits, &s_tag[BUF][block * 32], q_tag, l32, half, scattered);
                if constexpr (Mask::kCanvas) {
                    mask.template mask_keys<false>(bits, &s_tag[BUF][block * 32], q_tag, half, [&](int r, uint32_t m) __attribute__((always_inline)) { dpacc[r] = keep_or_zero(m, dpacc[r]); });
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) dpacc[r] = keep_or_zero(Mask::keep(bits, r), dpacc[r]);
                }
            }
            if constexpr (CAPTURED) {
                const int kvs = kvs_blk;
                if constexpr (ScoreMod<SCORE>::kAlibi) {
                    // (integers below 2^24: the differences are exact, in one instruction instead of a subtraction and a conversion.  us: causal,
                    // S = 4096, 32 heads, D = 64 / 128 104 -> 99 / 167 -> 158, packed documents, S = 16384, D = 64 177 -> 168)
                    const float first = (float)dq0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) g_alibi = __builtin_fmaf(dpacc[r], first - (float)elem_pos(r), g_alibi);
                }
                if constexpr (ScoreMod<SCORE>::kRel) {
                    if (q_wave_min - (kvs + 31) >= smod.rel_max) {          // every pair on the last entry
#pragma unroll
                        for (int r = 0; r < 16; ++r) g_hi += dpacc[r];
                    } else if (q_wave_min + 31 <= kvs) {                     // every pair on the first entry
#pragma unroll
                        for (int r = 0; r < 16; ++r) g_lo += dpacc[r];
                    } else {
                        const int dqk = q_wave_min - kvs + lane - 31;
                        atomicAdd(&s_tab[min(max(dqk, 0), smod.rel_max)], diagonal_sums(dpacc, half));
                    }
                }
                return;
            }
            // dQ^T += K^T dS^T
            u32x4 dsk[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    dsk[c][jj] = pack_bf16(dpacc[8 * c + 2 * jj], dpacc[8 * c + 2 * jj + 1]);
                    if constexpr (Mask::kCells) dsk[c][jj] = cells.pair(dsk[c][jj], 4 * c + jj);
                }
            {
                constexpr int NM = 2 * NDB;              // [slice c][block db]
                auto frag = [&](int m) { return tr_reader.read(kt, kvb * 32 + 16 * (m / NDB), m % NDB); };
                bf16x8 fr[NM];
#pragma unroll
                for (int m = 0; m < PF; ++m) fr[m] = frag(m);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    if (m + PF < NM) fr[m + PF] = frag(m + PF);
                    dq[m % NDB] = mfma32(fr[m], __builtin_bit_cast(bf16x8, dsk[m / NDB]), dq[m % NDB]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        });
        wait_vmem();
        __syncthreads();
    };
    auto all_tiles = [&](auto half_tag) __attribute__((always_inline)) {
        int t = 0;
        for (; t + 1 < T; t += 2) {
            step(t, std::integral_constant<int, 0>{}, half_tag);
            step(t + 1, std::integral_constant<int, 1>{}, half_tag);
        }
        if (t < T) step(t, std::integral_constant<int, 0>{}, half_tag);
    };
    // (two loops: in one for both, which moves the readers, long rows took 3 to 9 % more)
    if constexpr (MIXED) {
        if (whole) all_tiles(std::false_type{});
        else all_tiles(std::true_type{});
    } else {
        all_tiles(std::bool_constant<PAIRS>{});
    }

    if constexpr (CAPTURED) {
        auto wave_sum = [](float v) {
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            return v;
        };
        if constexpr (ScoreMod<SCORE>::kAlibi) {
            const float g = wave_sum(g_alibi);
            if (lane == 0) atomicAdd(&s_tab[kTabAlibi], g);
        }
        if constexpr (ScoreMod<SCORE>::kRel) {
            const float hi = wave_sum(g_hi), lo = wave_sum(g_lo);
            if (lane == 0) {
                atomicAdd(&s_tab[smod.rel_max], hi);
                atomicAdd(&s_tab[0], lo);
            }
        }
        __syncthreads();
        if constexpr (ScoreMod<SCORE>::kRel)
            for (int i = tid; i < a.p.rel_len; i += NW * 64) a.cap_rel[cap_slot * a.p.rel_len + i] = s_tab[i];
        if constexpr (ScoreMod<SCORE>::kAlibi)
            if (tid == 0) a.cap_alibi[cap_slot] = s_tab[kTabAlibi];
        return;
    }
    const float qscale = a.scale * ScoreMod<SCORE>::grad_scale();
    if (PAIRS && !whole) {
        // each of the two waves of the same rows finishes half of the dims and hands over the other half (the last step ended
        // with a barrier: the tiles are free)
        constexpr int HDB = D / 64;
        f32x4* give = (f32x4*)smem + w * (HDB * 4 * 64) + lane;
        const f32x4* take = (const f32x4*)smem + (w ^ 2) * (HDB * 4 * 64) + lane;
#pragma unroll
        for (int q = 0; q < HDB * 4; ++q) {
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = my_keys ? dq[q >> 2][4 * (q & 3) + i] : dq[HDB + (q >> 2)][4 * (q & 3) + i];
            give[q * 64] = v;
        }
        __syncthreads();
        if (!real_row) return;
#pragma unroll
        for (int q = 0; q < HDB * 4; ++q) {
            f32x4 v = take[q * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (v[i] + (my_keys ? dq[HDB + (q >> 2)][4 * (q & 3) + i] : dq[q >> 2][4 * (q & 3) + i])) * qscale;
            u32x2 pk;
            pk[0] = pack_bf16(v[0], v[1]);
            pk[1] = pack_bf16(v[2], v[3]);
            *(u32x2*)(dq_ptr + (my_keys * HDB + (q >> 2)) * 32 + 8 * (q & 3) + 4 * half) = pk;
        }
        return;
    }
    if (!real_row) return;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            u32x2 pk;
            pk[0] = pack_bf16(dq[db][4 * rg] * qscale, dq[db][4 * rg + 1] * qscale);
            pk[1] = pack_bf16(dq[db][4 * rg + 2] * qscale, dq[db][4 * rg + 3] * qscale);
            *(u32x2*)(dq_ptr + db * 32 + 8 * rg + 4 * half) = pk;
        }
}

}  // namespace flexattn
