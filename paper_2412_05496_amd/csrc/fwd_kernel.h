// FlexAttention forward kernel for gfx950 (paper Eq. 1; forward template of section 4.1; block
// skipping, full/partial split and indirect KV-block access of section 4.2; the KV prefetch of
// the "Data Prefetching Pipeline" paragraph is the two-deep asynchronous LDS pipeline below).
//
// One workgroup owns one row of BlockMask blocks (Bq = NW * 32 query rows of one (b, hq)); each
// wave owns 32 of those rows.  The score tile is computed TRANSPOSED, S^T = K Q^T, so that in the
// MFMA result layout every lane holds scores of ONE query (column l % 32) and 16 keys per 32-key
// block in its registers: the row max / row sum of the online softmax are in-register reductions
// plus one exchange between the two halves of the wave, and P^T is already laid out as the B
// operand of O^T += V^T P^T.  K and V tiles go from global memory straight into LDS (LDS-DMA buffer
// loads, issued one at a time between the MFMAs of the next score tile); K rows are
// the A operand of K Q^T as they are, V^T fragments come out of the row-major V tile through the
// transposing LDS read.  Q lives in registers for the whole kernel.
//
// Five forms of the loop over the tiles, the first four with one barrier per tile:
//   pipelined  while the VALU works on the softmax of tile t, the MFMA unit computes S^T of tile t + 1; K(t + 2) and
//              V(t + 1) are in flight from HBM / L2 meanwhile;
//   PLAIN      (D = 64) a 32-key block after the other, K and V one 64-key tile ahead: four waves per SIMD instead of
//              three (fwd_plain, plain_pays);
//   UNITS      (D = 128) the same with 32-key tiles in a ring of three, two tiles ahead: three instead of two
//              (fwd_units, units_pay);
//   PAIRS      four waves on 64 rows, each with its half of a tile's keys: rows of blocks of 64, and halves of 128 (pairs_pay);
//   SPLIT      for launches that leave the chip idle: the waves of a workgroup share 32 rows and take their keys in turn,
//              each through LDS of its own, and merge (m, l, O) at the end (split_waves).
#pragma once

#include <type_traits>

#include "flex_common.h"
#include "lds_tiles.h"

namespace flexattn {

struct FwdArgs {
    const bf16* Q;
    const bf16* K;
    const bf16* V;
    bf16* O;
    float* LSE;
    int64_t q_sb, q_sh, q_ss, k_sb, k_sh, k_ss, v_sb, v_sh, v_ss, o_sb, o_sh, o_ss;
    int B, Hq, Hkv, G, q_len, kv_len;
    int NR, NC, Bk, sub;   // BlockMask geometry; sub = Bk / 64 kernel tiles per block
    int bm_Bm, bm_Hm;
    UnitSets abreast;      // of the launch (unit_of_workgroup)
    const int32_t* kv_num;
    const int32_t* kv_idx;
    const int32_t* full_num;
    const int32_t* full_idx;
    const int32_t* kv_order;   // nullable: rows of blocks, longest first
    float scale;
    flexattn_mod_params p;
    // paged K/V (section 5.1): K, V point at the pools, k_sb = v_sb = 0, k_sh = v_sh = page_size * D,
    // k_ss = v_ss = D; page p starts page_stride elements after page p - 1; the physical block of
    // every BlockMask entry stands at the same place in phys_kv_idx / phys_full_idx
    const int32_t* phys_kv_idx;
    const int32_t* phys_full_idx;
    int64_t page_stride;
    int n_pool_pages;
    int Bq;                // rows of a BlockMask block
    unsigned first_id;     // PAIRS: of the launch's workgroups, where there are several launches (kMaxLaunch)
    int halved;            // MIXED: how many of the rows of blocks, in work order, are taken in halves
};

constexpr int kTileKV = 64;   // keys per kernel tile

// Which form of the tile loop.  The pipelined one keeps the scores of two tiles, which at D = 64 allows three
// waves per SIMD; the plain one needs 112 to 128 registers: four waves, whose turns hide more than the pipeline
// does, and hidden blocks of PARTIAL tiles cost nothing.  us, pipelined -> plain (one MI355X, Bq = 128, D = 64):
// causal, S = 1024, 64 x 16 heads: 277 -> 250; window of 1024, S = 5000: 114 -> 105; relative bias, S = 8192,
// 64 heads: 158 -> 127; no mask, S = 2048: 89.5 -> 86.5; packed documents with ALiBi: 218 -> 216.
// The pipelined one stays where it is the better one: a bounded soft-cap, whose softmax needs no running
// maximum (287 -> 299); and, where neither a window, documents nor a canvas ends rows early, long rows on a chip that is not full and
// soft-caps whose maximum has to be tracked (plain_pays; plain / pipelined, S x heads: causal, 4096 x 36 126 / 120, 4096 x 48 136 / 151, 8192 x 20 238 /
// 211, 16384 x 10 408 / 390, 4096 x 64 178 / 192, ALiBi, 4096 x 40 145 / 127; cap of 100, 2048 x 72 104 / 92, 8192 x 32 485 / 461, 1024 x 256 89.5 / 91.9), but
// rows of one length whose workgroups are the four per CU that run at once (no mask, 4096 x 32 152 / 155, 16384 x 8 585 / 597, but 4096 x 40 193 / 190, 8192 x
// 10 215 / 210).  Neighborhood masks gain most: 37 % of the 32 x 32 blocks of 8 x 8 tiles with K = 13 are hidden (490 ->
// 340 at 128 x 128 pixels).
template <int D, int NW, bool BOUNDED>
constexpr bool fwd_plain() {
    return D == 64 && NW == 4 && !BOUNDED;
}

template <uint32_t SCORE>
bool plain_pays(int kv_len, unsigned grid, bool uneven) {
    if (SCORE & FLEXATTN_SCORE_SOFTCAP) return kv_len < 2048;
    return kv_len < 4096 || grid >= 6 * 256 || (!uneven && grid > 3 * 256 && grid <= 4 * 256);
}

// The same at D = 128, where 64-key tiles of K and V leave LDS for two workgroups: units of 32 keys in a ring of
// three take 48 KiB, three workgroups of 168 registers.  The chip's power limit eats most of the gain on long
// dense rows, so the rule is by what was measured (us, pipelined -> units; D = 128, Bq = 128):
//   documents, canvases and biases always: documents, S = 2048 200 -> 184, one of S = 8192 1092 -> 1063; ALiBi,
//   S = 1000 254 -> 246, S = 8192 1325 -> 1313; relative bias, S = 32768 5166 -> 4876; neighborhood, 128 x 128, K = 13
//   582 -> 502, 64 x 64, K = 63 1360 -> 1349;
//   otherwise by length: causal S = 1024 233 -> 224, no mask 317 -> 319, S = 1536 331 -> 329, S = 2048 561 -> 570, causal
//   S = 8192 592 -> 626 (four sequences of 16 heads: 1099 -> 1105);
//   never with a relative bias under a soft-cap: its table no longer lets three in (325 -> 345);
//   and only where the workgroups are three rounds of the chip: with fewer there is nothing to put beside a
//   workgroup, and each is slower by itself (one sequence, S = 4096, ALiBi, 24 heads 172 -> 215).
// Windows of at most half the keys have rows of one length, and the workgroups go in rounds, of 768 with units and of 512 without: units where that is one round less, or where
// there are many rounds (S = 4096, window of 1024; heads 16: 43.9 -> 45.3, 24: 71.1 -> 62.8, 32: 82.5 -> 95.2, 40: 105 -> 102,
// 64: 154.4 -> 153.6; the same with a relative bias and a prefix, window of 512: 41.2 -> 45.9, 67.3 -> 57.4, 76.6 -> 90.3,
// 100 -> 97, 147 -> 147; S = 5000, four sequences of 16 / 2 heads: 186 -> 171).  Longer windows go by length (window = S = 4096,
// heads 24: 133 -> 159, 40: 203 -> 210; S = 8192, 40 heads: 710 -> 731).
enum class FwdUnits { kNever, kAlways, kShort, kWindow };
constexpr int kUnitsMaxKeys = 1536, kUnitsMinGroups = 9 * 256;
template <int D, int NW, uint32_t MASK, uint32_t SCORE>
constexpr FwdUnits fwd_units() {
    constexpr bool cap = SCORE & FLEXATTN_SCORE_SOFTCAP, bias = SCORE & (FLEXATTN_SCORE_ALIBI | FLEXATTN_SCORE_REL_BIAS);
    if (D != 128 || NW != 4 || (cap && (SCORE & FLEXATTN_SCORE_REL_BIAS))) return FwdUnits::kNever;
    if (mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW)) return FwdUnits::kWindow;
    if (mask_uses(MASK, FLEXATTN_M_DOCUMENT | FLEXATTN_M_NEIGHBORHOOD) || (bias && !cap)) return FwdUnits::kAlways;
    return FwdUnits::kShort;
}
// grid: the workgroups that are launched
template <uint32_t MASK, uint32_t SCORE>
bool units_pay(const FwdArgs& a, int64_t grid) {
    constexpr FwdUnits rule = fwd_units<128, 4, MASK, SCORE>();
    if constexpr (rule == FwdUnits::kNever) return false;
    if constexpr (rule == FwdUnits::kWindow) {
        const int64_t reach = (int64_t)a.p.window + (mask_uses(MASK, FLEXATTN_M_PREFIX) ? a.p.prefix_len : 0);
        if (2 * reach <= a.kv_len) return (grid > 2 * 256 && grid <= 3 * 256) || grid >= 5 * 256;
    }
    return (rule == FwdUnits::kAlways || a.kv_len <= kUnitsMaxKeys) && (int64_t)a.B * a.Hq * a.NR >= kUnitsMinGroups;
}
// The split form: a workgroup takes 32 rows instead of a row of blocks, and its waves the 32-key units of those rows in
// turn.  A small launch ends with its longest chain of tiles on a wave, which this makes 4 or 8 times shorter, on up to four
// times as many CUs; it costs each wave its own loads of K and V and a merge of the waves' results, which a full chip has no
// room for.  us, a row of blocks -> 4 waves / 8 waves: causal, S = 4096, D = 64, 1 head 54 -> 23.5 / 15.8, 4 heads 55 -> 24.8 / 20.1, 8 54 ->
// 33.5 / 34.0, 16 77 -> 59 / 64, 24 105 -> 90 / 96, 32 113 -> 117; D = 128, 1 head 78 -> 33.6 / 22.8, 4 78 -> 38.6 / 32.3, 8 77 -> 55.6 /
// 62.4, 16 114 -> 109 / 124, 24 138 -> 162; S = 16384, 1 head 271 -> 105 / 69, D = 128 465 -> 146 / 105, 4 heads 362 -> 385; S = 1000, D = 64,
// 8 / 32 / 64 heads 17.9 -> 8.8 / 7.3, 18.3 -> 15.5, 23.6 -> 24.4, D = 128, 8 / 16 / 32 heads 22.8 -> 11.9 / 10.5, 23.1 -> 15.1, 23.8 -> 24.5;
// S = 300, D = 64, 8 / 64 / 128 heads 7.5 -> 5.4 / 5.2, 7.8 -> 7.1, 9.5 -> 11.9, D = 128, 8 / 32 / 64 heads 9.7 -> 7.0, 10.0 -> 9.0, 10.3 ->
// 13.8; no mask, S = 2048, D = 64, 4 / 16 / 24 heads 32.6 -> 13.7 / 10.3, 32.7 -> 30.1, 43.6 -> 44.4, D = 128, 4 / 8 / 16 heads 41.3 -> 19.7
// / 16.4, 40.6 -> 28.2, 44.5 -> 55.1; window of 512, S = 4096, D = 64, 8 / 16 heads 13.1 -> 12.2, 17.9 -> 22.0, D = 128, 4 / 8 heads 19.4 ->
// 12.0 / 16.5, 19.2 -> 22.4; chunks of 518 on 9000 cached keys, 2 heads 126 -> 56 / 35, D = 128 178 -> 86 / 51; of 500, 64 heads, 130 -> 129,
// D = 128 203 -> 256.
// Short rows lose first (a row of blocks -> 4 waves): D = 64, causal, S = 130, 128 heads 6.7 -> 8.6, S = 256, 128 heads 8.3 -> 9.7, window of 64, S = 800,
// 40 heads 8.7 -> 9.6, documents of 16 to 100, S = 8192, 8 heads 13.6 -> 18.3, of 100 to 400, 12 heads 23.9 -> 26.8 (but of 256 to 4096, 8 heads 87 ->
// 46: the host cannot tell them apart); D = 128, no mask, S = 800, 20 heads 21.2 -> 22.3, S = 1100, 21 heads 27.3 -> 30.7, documents of 16 to 100,
// S = 4160, 7 heads 15.1 -> 18.6 (of 256 to 4096 84 -> 39).
// So: while the workgroups, of 32 rows each, are no more than 2 per CU, or 4 at D = 64 (where a wave's loads weigh less) with rows of 448 keys or
// more (no mask, S = 800, 35 heads 16.5 -> 15.2; documents of 16 to 100, S = 8192, 4 heads 11.1 -> 10.6; with a relative bias, whose units cost more, rows of
// any length, S = 256, 112 heads 14.3 -> 12.1); and long rows of uneven length, whose longest a full row of blocks leaves alone at the end, up to 12
// and 4.  One head's window alone at D = 128 no more than 1 per CU: neighbouring slices, dealt to all XCDs, no longer share an L2 (S = 16384, window of 1000
// 29 -> 39, of 300 16.3 -> 17.4).
// Returns the waves, 0: a workgroup per row of blocks.
template <uint32_t MASK, uint32_t SCORE>
int split_waves(const FwdArgs& a, int D) {
    const int64_t groups = unit_grid(a.B * a.Hkv, a.G * a.NR * (a.Bq / 32));
    const LineShape rows = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const int64_t keys = rows.sure;
    int64_t most = 2 * 256;
    if (D == 64) {
        constexpr bool rel = (SCORE & FLEXATTN_SCORE_REL_BIAS) != 0, doc = PartialMask<MASK>::kDoc;
        if (keys >= 448 || (doc && a.kv_len >= 448) || (rel && a.kv_len >= 256)) most = 4 * 256;
        if (rows.sure_uneven && keys >= 2048) most = keys < 4096 ? 8 * 256 : keys < 12000 ? 12 * 256 : 10 * 256;
    } else {
        if (rows.sure_uneven && keys >= 1024) most = keys >= 2048 ? 4 * 256 : 3 * 256;
        if (mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW) && a.B * a.Hkv == 1 && 8 * keys < a.kv_len) most = 256;
    }
    if (groups > most) return 0;
    const bool eight = groups <= 256 ? rows.longest > (D == 64 ? 256 : 512) : groups <= 512 && (D == 64 ? keys >= 2048 : rows.sure_uneven && keys >= 4096);
    return eight ? 8 : 4;
}
// The pairs form: a workgroup takes 64 rows, and its four waves are two slices of 32 rows times the two 32-key halves of every
// tile; the two waves of the same rows merge (m, l, O) at the end.  Rows of blocks of 64 always: two waves, one per slice, leave
// LDS for one (D = 128) or 2.5 (D = 64) waves per SIMD, four that share the tiles make it two and four (us, two waves -> pairs, Bq
// = 64: causal, S = 8192, 16 heads, D = 128 / 64 381 -> 302 / 225 -> 178; S = 1024, 256 heads 153 -> 117 / 72 -> 62; S = 300, 1024 heads 98 -> 91 /
// 40 -> 39; no mask, S = 2048, 64 heads 192 -> 155 / 105 -> 85; window of 1024, S = 8192, 2 x 16 / 4 heads 225 -> 169 / 108 -> 88; soft-cap, S = 835, 45 x
// 32 heads 641 -> 529 / 347 -> 296).  Rows of blocks of 128 where their halves end the launch sooner: rows of uneven length on a chip
// that they do not fill for long, by the workgroups of 128 rows (us, a row of blocks -> pairs, S x heads: causal, D = 64, 8192 x 16
// 189 -> 170, 4096 x 32 106 -> 98, 2048 x 64 65 -> 58, 16384 x 6 259 -> 257, but 16384 x 16 614 -> 627, 8192 x 64 622 -> 654, 1024 x 256 60 -> 62;
// D = 128, 8192 x 8 173 -> 153, 4096 x 16 110 -> 83, 2048 x 32 60 -> 58, but 8192 x 16 279 -> 299, 16384 x 6 399 -> 446; soft-cap, D = 64, 4096
// x 32 142 -> 123, but 8192 x 16 246 -> 252; documents of 256 to 4096 with ALiBi, their longest rows in halves (halved_rows), D = 64, 8192 x 16 92 -> 63, 16384 x
// 6 96 -> 67, 16384 x 16 146 -> 132, 8192 x 32 165 -> 141, 2048 x 128 111 -> 103, but 8192 x 64 279 -> 272 and of 100 to 400 77 -> 81; D = 128, 4096 x 16
// 95 -> 64, 8192 x 8 75 -> 58, 16384 x 6 117 -> 97, but 8192 x 16 100 -> 102, 16384 x 9 126 -> 135, without ALiBi 16384 x 16 214 -> 228).
// Rows of one length, or shorter than 2048: long ones at D = 64 while there are at most two workgroups per CU (no mask, 1500 x 32 33 -> 29, 4000 x 12 75 -> 63,
// even from one and a half on, 1500 x 36 35.6 -> 34.1, 1500 x 40 33.6 -> 34.8, but 3000 x 32 88 -> 95; chunks of 640 on 2000 to 3000 cached keys, 2 x 32 heads
// 69 -> 58, 2 x 48 78 -> 75, of 1500 on 8000, 32 heads 189 -> 168; windows, 2048 x 28, of 1024 25.8 -> 24.3, 4096 x 16, of 2048 45 -> 45, but 4096 x 32, of 500
// 31 -> 36; window of 1500 or prefix of 200 with a relative bias, 4096 x 16 50 -> 43; canvases, 32 x 32, K = 21, 48 heads 28.7 -> 23.6, 64 x 64, K = 27, 13 heads
// 50 -> 36, Morton order, K = 21, 16 heads 51 -> 40; causal, 1050 x 52 20.6 -> 20.4, 1600 x 36 29 -> 26, ALiBi, 2000 x 30 45 -> 37, soft-cap, 1600 x 36 40 -> 32;
// D = 128, no mask, 1500 x 32 51 -> 53).
// Documents of a few tokens, which the host cannot tell from long ones, pay a little (8192 x 16, of 16 to 100 19.7 -> 20.8).
template <uint32_t MASK, bool BOUNDED>
bool pairs_pay(const FwdArgs& a, int D, unsigned grid) {
    if (a.Bq == 64) return true;
    const LineShape rows = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    if (D == 64 && rows.sure >= 1024 && grid <= 2 * 256) return true;
    if (!rows.uneven || a.kv_len < 2048) return false;
    constexpr bool doc = PartialMask<MASK>::kDoc;
    if (D == 128) return grid <= (doc ? 3 * 256 : 2 * 256);
    return grid <= (doc ? 8 * 256 : 4 * 256) && !(BOUNDED && !doc && a.kv_len >= 8192);
}
// Documents with Bq = 128: a third of the rows of blocks, the longest, goes in halves, and of a batch whose longest row is short (tiles of 64
// keys) none; the host cannot tell.  A workgroup of the same kernel takes a row as a whole, two passes over every tile's halves.
// (us, D = 64, a workgroup per row of blocks / all in halves / this: documents of 16 to 100, 8192 x 16 19.8 / 23.2 / 20.4, ALiBi, 16384 x 16 34.7 / 39.0 /
// 36.9, of 100 to 400, 4096 x 16 20.2 / 17.0 / 16.1, of 256 to 4096, 4096 x 16 74 / 51 / 45, 8192 x 16 88 / 60 / 59, ALiBi, 16384 x 16 178 / 127 / 129; D = 128, of
// 16 to 100, 8192 x 8 20.5 / 22.3 / 18.7, of 100 to 400, 16384 x 6 35.7 / 37.4 / 33.0, of 256 to 4096, 2048 x 48 58 / 59 / 51, ALiBi, 4096 x 16 111 / 62 / 63,
// 8192 x 12 115 / 77 / 80.  A quarter or a half in halves: 1 to 8 % less on one side each.  Empty workgroups between full ones
// instead of whole rows: 28 for the first.)  A relative bias under a soft-cap whose maximum is tracked keeps all in halves at D = 64: the whole rows
// cost it 18 spills (of 16 to 100, 8192 x 16 30.3 -> 33.9).
template <int D, uint32_t MASK, uint32_t SCORE, bool BOUNDED>
constexpr bool mixed_pays() {
    return PartialMask<MASK>::kDoc && !(D == 64 && (SCORE & FLEXATTN_SCORE_REL_BIAS) && (SCORE & FLEXATTN_SCORE_SOFTCAP) && !BOUNDED);
}
template <int D>
constexpr int kShortTiles = D == 64 ? 6 : 10;
// Waves per SIMD to compile for: what registers (512 per SIMD lane) and LDS admit.  The pipelined variants
// with a relative-bias table would spill at three.
template <int D, uint32_t SCORE, bool UNITS, bool PLAIN, bool SPLIT, bool PAIRS>
constexpr int fwd_waves_per_simd() {
    if (SPLIT) return 2;
    if (PAIRS) return D == 64 ? 4 : 2;
    if (D != 64) return UNITS ? 3 : 2;
    if (PLAIN) return 4;
    return (SCORE & FLEXATTN_SCORE_REL_BIAS) ? 2 : 3;
}

// BOUNDED: the score_mod ends in a soft-cap small enough that the cap itself serves as the fixed
// softmax maximum (see ScoreMod::bounded); chosen by the host from the cap value.
// UNITS: 32-key units in a ring of three (fwd_units).  PLAIN: no tile pipeline (fwd_plain).  PAIRS: see pairs_pay.  MIXED: PAIRS with Bq = 128
// where only some rows of blocks go in halves (halved_rows).  SPLIT: the NW waves share 32 rows and take the keys in turn (split_waves).
// PAGED: the tiles of K and V are fetched from a paged pool through the converted block lists;
// the mods keep seeing the logical key index.
// M0 RULE: this kernel fills LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the
// compiler's back.  Keep every register array in it indexed by compile-time constants (no movrel /
// s_set_gpr_idx code, which would also use M0) and add no other LDS-DMA or M0-based construct.
template <int D, int NW, uint32_t MASK, uint32_t SCORE, bool BOUNDED, bool PAGED, bool UNITS = false,
          bool PLAIN = fwd_plain<D, NW, BOUNDED>(), bool SPLIT = false, bool PAIRS = false, bool MIXED = false>
__global__ __launch_bounds__(NW * 64, (fwd_waves_per_simd<D, SCORE, UNITS, PLAIN, SPLIT, PAIRS>())) void fwd_kernel(const FwdArgs a) {
    static_assert(!PAIRS || (NW == 4 && !UNITS && !PLAIN && !SPLIT), "two row slices times two key halves");
    static_assert(!MIXED || PAIRS, "halves and whole rows");
    constexpr int kSlices = PAIRS ? NW / 2 : NW;    // of 32 rows
    const int Bq = MIXED ? 128 : SPLIT || PAIRS ? a.Bq : kSlices * 32;
    constexpr int TILE = kTileKV * D;              // elements per LDS tile

    // K(even), K(odd), V(even), V(odd); UNITS: three slots of 32 keys, K then V; SPLIT: 32 keys of K, then V, for each wave
    __shared__ __attribute__((aligned(1024))) bf16 smem[(SPLIT ? NW : UNITS ? 3 : 4) * TILE];
    using Score = ScoreMod<SCORE, true>;
    __shared__ float s_rel[Score::kRel ? kRelTableMax : 1];           // relative-bias row of the head
    using Mask = PartialMask<MASK>;
    constexpr bool CELLS = Mask::kCells;
    static_assert(!(CELLS && BOUNDED), "cells: the running maximum's branch sets their masks");
    __shared__ __attribute__((aligned(256))) uint32_t s_tag[SPLIT ? NW : UNITS ? 3 : 2][Mask::kTags ? kTileKV : 4];   // tags of a PARTIAL tile's keys, per buffer (SPLIT: wave)

    constexpr bool kHiddenTable = Mask::kCanvas && (UNITS || PLAIN || SPLIT || PAIRS);
    __shared__ uint32_t s_qtag[Mask::kTags && !CELLS ? NW * 64 : 1];            // each lane's own tag (its query's)
    __shared__ u32x4 s_rect[CELLS ? NW * 32 : 1];              // cells: its window, for both halves
    __shared__ uint8_t s_hidden[kHiddenTable ? kHiddenTiles : 1];    // CanvasBlocks::hidden_bits of the first tiles

    // ---- workgroup -> (b, hkv, g, row of blocks).  Rows are taken longest first (the BlockMask's work order), or
    // last-first without one (causal-like masks: longest first).
    int unit, rem, slice = 0;
    const int per_unit = a.G * (MIXED ? a.NR + a.halved : a.NR * (SPLIT ? Bq / 32 : PAIRS ? Bq / 64 : 1));
    UnitSets abreast = SPLIT ? one_by_one(a.B * a.Hkv) : a.abreast;
    if constexpr (Mask::kDoc && !SPLIT) abreast = abreast_if_long(abreast, a.B * a.Hkv, longest_row(a.kv_order, a.full_num, a.kv_num, 0, a.NR, a.sub));
    if (!unit_of_workgroup(blockIdx.x + (PAIRS ? a.first_id : 0u), a.B * a.Hkv, per_unit, abreast, unit, rem)) return;
    if constexpr (SPLIT) {
        slice = rem & (Bq / 32 - 1);                // which 32 rows of the block
        rem >>= Bq == 128 ? 2 : 1;
    }
    bool whole = false;                             // MIXED: 32 rows and all keys to a wave
    if constexpr (MIXED) {
        const int64_t rows = ((int64_t)(a.bm_Bm > 1 ? unit / a.Hkv : 0) * a.bm_Hm + (a.bm_Hm > 1 ? unit % a.Hkv * a.G : 0)) * a.NR;
        if (!half_or_row(a.kv_order, a.full_num, a.kv_num, rows, a.NR, a.G, a.sub, a.halved, kShortTiles<D>, rem, slice, whole)) return;
    } else if constexpr (PAIRS) {
        slice = rem & (Bq / 64 - 1);                // which 64 rows of the block
        rem >>= Bq == 128 ? 1 : 0;
    }
    const int g = rem % a.G;
    const int b = unit / a.Hkv, hkv = unit % a.Hkv, hq = hkv * a.G + g;
    const int64_t plane = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0);
    // (an order array that is no permutation gives wrong rows; clamped so that it cannot leave the arrays)
    const int row = a.kv_order ? min(max(ldc(a.kv_order + plane * a.NR + rem / a.G), 0), a.NR - 1) : a.NR - 1 - rem / a.G;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int my_slice = PAIRS && !whole ? w & 1 : w, my_keys = PAIRS && !whole ? w >> 1 : 0;  // PAIRS: which 32 rows, which 32 keys of every tile
    const int first_row = row * Bq + (SPLIT ? 32 : 64) * slice;            // of the workgroup
    const int wave_rows = first_row + (SPLIT ? 0 : my_slice) * 32;         // first of the wave's 32 rows
    const int q_row = wave_rows + l32;
    if ((SPLIT || PAIRS) && first_row >= a.q_len) return;

    const int64_t line = plane * a.NR + row;
    const int n_full = ldc(a.full_num + line), n_part = ldc(a.kv_num + line);
    const int T = (n_full + n_part) * a.sub;

    bf16* o_ptr = a.O + b * a.o_sb + hq * a.o_sh + (int64_t)q_row * a.o_ss;
    float* lse_ptr = a.LSE + ((int64_t)b * a.Hq + hq) * a.q_len + q_row;
    // rows past q_len (last block of a length that is no multiple of Bq) are computed on a copy of
    // the last real row and never stored
    const bool real_row = q_row < a.q_len;
    const int q_ld = min(q_row, a.q_len - 1);
    if (T == 0) {   // every key of these rows is masked
        if (real_row) {
            for (int d0 = half * 8; d0 < D; d0 += 16) *(u32x4*)(o_ptr + d0) = u32x4{0, 0, 0, 0};
            if (half == 0) *lse_ptr = -INFINITY;
        }
        return;
    }

    // Q fragments: B operand of K Q^T, column q_row, k-slots d = 16 ks + 8 half + [0, 8)
    bf16x8 qf[D / 16];
    {
        const bf16* qp = a.Q + b * a.q_sb + hq * a.q_sh + (int64_t)q_ld * a.q_ss + half * 8;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *(const bf16x8*)(qp + ks * 16);
    }
    const bf16* k_head = a.K + b * a.k_sb + hkv * a.k_sh;
    const bf16* v_head = a.V + b * a.v_sb + hkv * a.v_sh;
    const i32x4 k_rsrc = make_rsrc(k_head, (uint32_t)((a.kv_len - 1) * a.k_ss + D) * 2u);
    const i32x4 v_rsrc = make_rsrc(v_head, (uint32_t)((a.kv_len - 1) * a.v_ss + D) * 2u);
    const int k_row_bytes = (int)a.k_ss * 2, v_row_bytes = (int)a.v_ss * 2;
    // Where the 64 rows of a tile come from: a buffer descriptor and the byte offset of the first
    // row in it.  Contiguous K/V: one descriptor per head, the tile chosen by the offset.  PAGED: a
    // descriptor of exactly the tile, based at row `row` of pool page `page` (clamped to the pool,
    // so that a wrong page table reads wrong rows and never faults).
    auto tile_src = [&](const bf16* head, i32x4 whole, int row_bytes, int kv0, int page, int row, i32x4& rsrc,
                        int& soff) __attribute__((always_inline)) {
        if constexpr (PAGED) {
            const int pg = min(max(page, 0), a.n_pool_pages - 1);
            rsrc = make_rsrc(head + (int64_t)pg * a.page_stride + row * D, (uint32_t)((UNITS || SPLIT ? 32 : kTileKV) * D * 2));
            soff = 0;
        } else {
            rsrc = whole;
            soff = kv0 * row_bytes;
        }
    };

    const Score smod(a.p, hq, a.scale, lds_addr(s_rel));
    smod.fill_table(tid, NW * 64);                  // visible after the prologue's barrier
    const int q_pos = q_ld + q_offset_of(a.p, b);   // as the mods see it
    const int q_wave_min = wave_rows + q_offset_of(a.p, b);   // the wave's rows: q_wave_min .. +31
    const Mask mask(a.p, b, a.kv_len);
    // the lane's own tag waits in LDS as well: a register held for it over the whole kernel ends in spills
    // whose reloads wait for the tile loads
    bool scattered = false;
    if constexpr (Mask::kDoc) {
        const uint32_t id = (uint32_t)(a.p.doc_ids + (int64_t)b * a.p.doc_stride_b)[q_pos];
        s_qtag[tid] = id;
        scattered = Mask::scattered_ids(id);
    }
    typename Mask::CellBase cell_base = {};
    if constexpr (CELLS) {
        cell_base = mask.base_of_queries(a.p, wave_rows);
        s_rect[w * 32 + l32] = mask.query_rectangle(q_pos, cell_base);
    } else if constexpr (Mask::kCanvas) {
        s_qtag[tid] = mask.query_pixel(q_pos);
    }
    // Tags of the keys of the tile at kv0, into s_tag[buf] (visible after the next barrier): document ids
    // come by LDS-DMA (keys past the end read as 0), pixels are worked out by one of the waves.
    auto make_tags = [&](int buf, int kv0, int turn) __attribute__((always_inline)) {
        if constexpr (Mask::kDoc) {
            if (SPLIT || w == 0)
                dma_global_dword(lds_addr(&s_tag[buf][0]), a.p.doc_ids + (int64_t)b * a.p.doc_stride_b,
                                 min(kv0 + lane, a.kv_len - 1) * 4);
        }
        if constexpr (Mask::kCanvas) {
            if (SPLIT || w == (turn & (NW - 1))) s_tag[buf][lane] = mask.key_pixel(min(kv0 + lane, a.kv_len - 1));
        }
    };
    if constexpr (kHiddenTable) fill_hidden_tiles<SPLIT ? 1 : kSlices, NW * 64>(s_hidden, a.p, a.kv_idx + line * a.NC, n_full, T, a.sub, a.Bk, first_row, tid);
    // 32-key blocks of tile t that are hidden from this wave (bit 0, bit 1); visible after the prologue's barrier
    auto hidden_of = [&](int t) __attribute__((always_inline)) -> uint32_t {
        if constexpr (!kHiddenTable) return 0u;
        else return t < min(T, kHiddenTiles) ? ((uint32_t)__builtin_amdgcn_readfirstlane((int)s_hidden[t]) >> (SPLIT ? 0 : 2 * my_slice)) & 3u : 0u;
    };
    const float inv_neg2c = smod.capl2 > 0.0f ? -0.5f / smod.capl2 : 0.0f;   // 1 / (-2 cap log2 e)

    // ALiBi: from the end where the largest scores are (the bias falls with the distance: from the diagonal), so that the first
    // block of a row sets a maximum that stays; the other way round a steep head moves it in every block.
    // (us, forwards -> this: a step on packed documents, S = 16384, 16 heads, D = 64 658 -> 612; chunks of 1811 on about 2000 cached keys,
    // four sequences of 8 heads, D = 128, 146 -> 125; of 902 on about 6000, two of 8, D = 64, 72 -> 64)
    static_assert(!(Mask::kCanvas && Score::kAlibi), "s_hidden goes by the walk's forward order");
    const bool backwards = Score::kAlibi && smod.k_bias < 0.0f;
    // first key and PARTIAL flag of tiles t, t+1, t+2 (the walk is always two tiles ahead)
    TileWalk<PAGED> walk(a.full_idx + line * a.NC, a.kv_idx + line * a.NC, n_full, n_part, a.sub, a.Bk,
                         PAGED ? a.phys_full_idx + line * a.NC : nullptr, PAGED ? a.phys_kv_idx + line * a.NC : nullptr, backwards);
    int kv_t = 0, kv_t1 = 0, kv_t2 = 0;
    bool part_t = false, part_t1 = false, part_t2 = false;
    int pg_t = 0, pg_t1 = 0, pg_t2 = 0, pr_t = 0, pr_t1 = 0, pr_t2 = 0;   // PAGED: page, row in page
    const uint32_t smem_bytes = lds_addr(smem);
    const WaveTileLoader<D, SPLIT ? 4 : NW> k_loader(a.k_ss, w, lane), v_loader(a.v_ss, w, lane);   // (SPLIT has its own)
    // buf = tile index & 1
    auto load_k = [&](int buf, int kv0, int page, int row) {
        i32x4 rsrc;
        int soff;
        tile_src(k_head, k_rsrc, k_row_bytes, kv0, page, row, rsrc, soff);
        k_loader.start(rsrc, smem_bytes + buf * (TILE * 2), soff);
    };
    auto load_v = [&](int buf, int kv0, int page, int row) {
        i32x4 rsrc;
        int soff;
        tile_src(v_head, v_rsrc, v_row_bytes, kv0, page, row, rsrc, soff);
        v_loader.start(rsrc, smem_bytes + (2 + buf) * (TILE * 2), soff);
    };
    RowReader<D> k_reader(l32, half, my_keys * 32 * D * 2);
    TrReader<D> v_reader(lane, my_keys * 32 * D * 2);

    // S^T = K Q^T for the two 32-key blocks of the K tile in buffer BUF (compile-time);
    // between(m) runs after the m-th of the 2 D / 16 MFMAs (used to spread out tile loads)
    auto qk = [&](auto buf_tag, f32x16 (&s)[2], auto&& between) {
        constexpr int BUF = decltype(buf_tag)::value;
        constexpr int NKS = D / 16;
        static_for<0, 2 * NKS>([&](auto m_tag) {
            constexpr int m = decltype(m_tag)::value, kvb = m / NKS, ks = m % NKS;
            if constexpr (ks == 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kvb][r] = 0.0f;
            }
            s[kvb] = mfma32(k_reader.read(smem_bytes + BUF * (TILE * 2), kvb * 32, ks), qf[ks], s[kvb]);
            between(m_tag);
        });
    };

    f32x16 oacc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.0f;
    // base-2 running max and this lane's part of the running sum; with a bounded soft-cap the
    // maximum is fixed at the cap from the start
    float m_run = BOUNDED ? smod.capl2 : -INFINITY, l_run = 0.0f;
    float m_use = 0.0f;     // the maximum the exponentials subtract: m_run, or 0 while the row has seen no key
    float m_thr = -INFINITY; // what a block's largest shifted score must exceed for the maximum to move
    bool seeded = false;     // (wave-uniform) every row has seen a key

    // score_mod, mask_mod (partial blocks only) and softmax of one 32-key block whose first key is
    // kvs: s -> P^T as two bf16 fragments.  The mask is a separate, rarely taken pass (kept a real
    // branch) so that the common path is one straight run of VALU work next to the MFMAs around it.
    // mask_mod of the 32-key block kvb of the tile in buffer buf: put(all-ones or 0, s) for every element
    auto masked = [&](f32x16& s, int kvs, int buf, int kvb, auto&& put) __attribute__((always_inline)) {
        typename Mask::Bits bits = mask.row_bits(q_pos, kvs + 4 * half);
        const uint32_t q_tag = Mask::kTags && !CELLS ? s_qtag[tid] : 0u;
        if constexpr (Mask::kDoc) Mask::match_documents(bits, &s_tag[buf][kvb * 32], q_tag, l32, half, scattered);
        if constexpr (Mask::kCanvas && !CELLS) {
            mask.template mask_keys<true>(bits, &s_tag[buf][kvb * 32], q_tag, half, [&](int r, uint32_t m) __attribute__((always_inline)) { s[r] = put(m, s[r]); });
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = put(Mask::keep(bits, r), s[r]);
        }
    };
    // The probabilities of a block as two bf16 fragments, and this lane's part of the row sum: over the bf16-rounded
    // probabilities, the values P V is computed from, two at a time (dot product of a packed pair with (1, 1), fp32 accumulation).
    typename Mask::CellMasks cells = {{~0u, ~0u}, ~0u};      // of the block that is worked on
    auto weigh = [&](const f32x16& s, bf16x8 (&pf)[2], auto&& prob) __attribute__((always_inline)) {
        float psum[2] = {0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            u32x4 pk;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                pk[jj] = pack_bf16(prob(s[8 * c + 2 * jj]), prob(s[8 * c + 2 * jj + 1]));
                if constexpr (CELLS) pk[jj] = cells.pair(pk[jj], 4 * c + jj);
                psum[jj & 1] = pair_sum_bf16(pk[jj], psum[jj & 1]);
            }
            pf[c] = __builtin_bit_cast(bf16x8, pk);
        }
        return psum[0] + psum[1];
    };
    auto softmax = [&](f32x16& s, int kvs, bool tile_partial, int buf, int kvb, bf16x8 (&pf)[2]) {
        const bool partial = tile_partial && !mask.full(q_wave_min, q_wave_min + 31, kvs, kvs + 31);   // (wave-uniform)
        // q_idx - kv_idx of element r is dq0 - 8 (r >> 2) - (r & 3)
        const int dq0 = q_pos - kvs - 4 * half;
        const float abase = smod.alibi_base(dq0);
        auto rel = [&](int r) __attribute__((always_inline)) {
            return typename Score::RelPos(dq0, abase, -(8 * (r >> 2) + (r & 3)));
        };
        // relative bias: one value for the whole block unless it lies near the diagonal
        float rel_uni;
        const bool rel_is_uni = smod.rel_uniform(q_wave_min - (kvs + 31), q_wave_min + 31 - kvs, rel_uni);
        if constexpr (BOUNDED) {
            // p = 2^(x - cap log2 e) = 2^(-2 cap log2 e * r), r = 1 / (1 + e): no maximum to track
            auto prob = [&](float e) __attribute__((always_inline)) {
                // -2 cap log2e / (1 + e) as ONE reciprocal: rcp((1 + e) / (-2 cap log2e))
                return fast_exp2(fast_rcp(__builtin_fmaf(e, inv_neg2c, inv_neg2c)));
            };
            if (rel_is_uni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = prob(fast_exp2(smod.template pre<true>(s[r], rel(r), rel_uni)));
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = prob(fast_exp2(smod.template pre<false>(s[r], rel(r))));
            }
            if (partial) {
                // Keep this a branch, not 16 selects on every tile.  Windows: by holding on to the scores, or the last
                // tile's copy of this spills 184 registers at D = 128 (8 heads, S = 200 to 1024: 10.3 -> 10.0,
                // 14.0 -> 13.7 us); causal masks are 1 to 3 % faster with the fence on memory.
                if constexpr (mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW)) asm volatile("" : "+v"(s));
                else asm volatile("" ::: "memory");
                masked(s, kvs, buf, kvb, keep_or_zero);
            }
            l_run += weigh(s, pf, [](float x) __attribute__((always_inline)) { return x; });
        } else {
            // Online softmax.  The running maximum only has to keep exp2(s - m) in range, so it follows
            // the scores lazily: the score_mod subtracts the CURRENT maximum on its way (folded into its
            // multiply-adds), and the maximum moves only when the block's probabilities under it add up to more
            // than kLazySum in some lane, or while some row has seen no key (O / l and LSE = m + log2 l come out
            // the same).  The sum is there anyway, so that a block whose maximum stays costs no maximum at all: 12 of
            // 66 vector instructions at D = 64 (us, a maximum per block -> this: no mask, S = 777, 128 heads, D = 64 35.8 -> 34.3; chunks
            // of 2048 on 4096 to 14336 cached keys, 4 sequences of 32 heads, D = 128 1382 -> 1353).
            constexpr float kLazyMax = 8.0f, kLazySum = 4096.0f;    // 16 of 2^kLazyMax: above the sum, the largest is above the maximum
            const float shift = -m_use;
            if (rel_is_uni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = smod.template apply_shifted<true>(s[r], rel(r), rel_uni, shift);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = smod.template apply_shifted<false>(s[r], rel(r), 0.0f, shift);
            }
            if constexpr (CELLS) {
                cells = {{~0u, ~0u}, ~0u};
                if (partial) cells = mask.cell_masks(s_rect[w * 32 + l32], &s_tag[buf][kvb * 32], cell_base, half, kvs <= mask.kv_last);
            } else if (partial) {
                if constexpr (Mask::kTags) asm volatile("" : "+v"(s));
                else asm volatile("" ::: "memory");
                masked(s, kvs, buf, kvb, keep_or_neg_inf);
            }
            auto track = [&]() __attribute__((always_inline)) {
                if constexpr (CELLS) {       // (the weights need no more than their pairs' masks)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[r] = keep_or_neg_inf(cells.element(r), s[r]);
                }
                float mx = s[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
                mx = max_halves(mx);
                if (__any(mx > m_thr)) {                 // some row of the wave moves its maximum (by mx)
                    const float up = mx > m_thr ? mx : 0.0f;
                    // (a row's first keys: nothing to rescale yet, and 2^-mx could overflow)
                    const float alpha = m_thr == -INFINITY ? 0.0f : fast_exp2(-up);
                    m_use += up;                         // (0 before the row's first key)
                    m_run = mx > m_thr ? m_use : m_run;
                    m_thr = mx > m_thr ? kLazyMax : m_thr;
                    seeded = !__any(m_thr == -INFINITY);
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[r] -= up;
                    l_run *= alpha;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
                }
            };
            auto weighed = [&]() __attribute__((always_inline)) { return weigh(s, pf, [](float x) __attribute__((always_inline)) { return fast_exp2(x); }); };
            float sum = 0.0f;
            constexpr bool kOnePlace = D == 128 ? !SPLIT && (Score::kAlibi || Mask::kTags) : PLAIN && Score::kAlibi;
            if constexpr (kOnePlace) {
                // (the weights in one place: in two, registers spill, which short rows pay for most; us, two -> one: D = 64, causal with ALiBi, S = 100,
                // 2048 heads 27.8 -> 24.2, S = 300, 1024 heads 44.1 -> 39.6, S = 1500, 256 heads 123 -> 118; D = 128, documents of 16 to 100 with ALiBi,
                // S = 16384, 16 heads 70 -> 66.  Elsewhere within 1 to 2 % either way.)
                bool moves = !seeded;
                for (;;) {
                    if (moves) track();
                    sum = weighed();
                    if (moves || !__any(sum > kLazySum)) break;
                    moves = true;
                }
            } else {
                // SPLIT: a maximum per block, since a wave's few blocks are mostly a row's first (us, the sum -> this: causal, S = 256, 2 heads 5.29 ->
                // 5.26, S = 4096, 4 heads 21.5 -> 21.3, documents, S = 4096, 4 heads 23.4 -> 23.0, chunks of 518 on 9000 cached keys, 2 heads 63.7 -> 62.6).
                bool moves = true;
                if (!SPLIT && seeded) {
                    sum = weighed();
                    moves = __any(sum > kLazySum);
                }
                if (moves) {
                    track();
                    sum = weighed();
                }
            }
            l_run += sum;
        }
    };

    // O^T += V^T P^T for the 32-key block kvb (compile-time) of the V tile in buffer BUF
    auto pv = [&](auto buf_tag, int kvb, const bf16x8 (&pf)[2]) {
        constexpr int BUF = decltype(buf_tag)::value;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                oacc[db] = mfma32(v_reader.read(smem_bytes + (2 + BUF) * (TILE * 2), kvb * 32 + 16 * c, db), pf[c], oacc[db]);
    };

    // ---- prologue: K(0), V(0) (and K(1), S^T(0) below) in flight
    auto first_tile = [&]() {
        kv_t = walk.next(part_t, pg_t, pr_t);
        load_k(0, kv_t, pg_t, pr_t);
        load_v(0, kv_t, pg_t, pr_t);
        if (part_t) make_tags(0, kv_t, 0);
    };
    // (a wave of the last block whose rows lie past q_len hides all: D = 64, 128 heads of 777 rows, no mask 37.2 -> 36.6 us, of 660,
    // causal 20.8 -> 19.1)
    const bool no_row = wave_rows >= a.q_len;
    auto hidden_block = [&](uint32_t bits, bool partial, int kv, int kvb) __attribute__((always_inline)) {
        if constexpr (Mask::kCanvas) return no_row || (bits & (1u << kvb)) != 0;
        else return no_row || (partial && mask.hidden(q_wave_min, q_wave_min + 31, kv, kv + 31));
    };
    if constexpr (SPLIT) {
        // Wave w takes the 32-key units w, w + NW, ... that are not hidden from its rows, through LDS of its own and
        // without a barrier.  K(next) is asked for when S^T has been computed, V(next) after P V: each has the other half of the
        // turn to arrive.
        constexpr uint32_t UT = 32 * D * 2;
        using L = WaveTileLoader<D, 1, 32>;
        const L k_load(a.k_ss, 0, lane), v_load(a.v_ss, 0, lane);
        const uint32_t k_lds = smem_bytes + (uint32_t)w * 2 * UT, v_lds = k_lds + UT;
        const int TU = 2 * T, per_block = 2 * a.sub, shift = a.sub == 1 ? 1 : 2, n_blocks = n_full + n_part;
        auto place = [&](int p) __attribute__((always_inline)) { return backwards ? n_blocks - 1 - p : p; };
        auto at = [&](const int32_t* full, const int32_t* part, int u) __attribute__((always_inline)) {
            const int p = place(min(u >> shift, n_blocks - 1));
            return ldc(p < n_full ? full + line * a.NC + p : part + line * a.NC + (p - n_full));
        };
        int u_next = w, blk_next = at(a.full_idx, a.kv_idx, w), pg_next = PAGED ? at(a.phys_full_idx, a.phys_kv_idx, w) : 0;
        int kv = 0, page = 0, prow = 0;                 // the unit that is loaded next
        bool partial = false;
        auto advance = [&]() __attribute__((always_inline)) {
            while (u_next < TU) {
                const int u = u_next, in_block = u & (per_block - 1), s0 = (backwards ? per_block - 1 - in_block : in_block) * 32;
                kv = blk_next * a.Bk + s0;
                page = pg_next;
                prow = s0;
                partial = place(u >> shift) >= n_full;
                u_next += NW;
                blk_next = at(a.full_idx, a.kv_idx, u_next);
                if constexpr (PAGED) pg_next = at(a.phys_full_idx, a.phys_kv_idx, u_next);
                if (!hidden_block(hidden_of(u >> 1) >> (u & 1), partial, kv, 0)) return true;
            }
            return false;
        };
        auto load = [&](const L& loader, const bf16* head, i32x4 whole, int row_bytes, uint32_t lds) __attribute__((always_inline)) {
            i32x4 rsrc;
            int soff;
            tile_src(head, whole, row_bytes, kv, page, prow, rsrc, soff);
            loader.start(rsrc, lds, soff);
        };
        if constexpr (kHiddenTable || Score::kRel) __syncthreads();
        bool more = advance();
        if (more) {
            if (partial) make_tags(w, kv, 0);
            load(k_load, k_head, k_rsrc, k_row_bytes, k_lds);
            load(v_load, v_head, v_rsrc, v_row_bytes, v_lds);
        }
        while (more) {
            wait_vmem_but<L::NI>();                     // K and the tags are here
            asm volatile("" ::: "memory");
            const int kv_now = kv;
            const bool partial_now = partial;
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
            read_ahead<D / 16>([&](auto m) { return k_reader.read(k_lds, 0, decltype(m)::value); },
                                    [&](auto m, bf16x8 f) { s = mfma32(f, qf[decltype(m)::value], s); });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // (K has left LDS)
            more = advance();
            if (more) load(k_load, k_head, k_rsrc, k_row_bytes, k_lds);
            bf16x8 pf[2];
            softmax(s, kv_now, partial_now, w, 0, pf);
            if (more && partial) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // (the tags have been read)
                make_tags(w, kv, 0);
            }
            // V is here; K(next) and its tags may be under way
            if (!more) wait_vmem();
            else if (Mask::kDoc && partial) wait_vmem_but<L::NI + 1>();
            else wait_vmem_but<L::NI>();
            asm volatile("" ::: "memory");
            constexpr int NDB = D / 32;
            read_ahead<2 * NDB>([&](auto m) { return v_reader.read(v_lds, 16 * (decltype(m)::value / NDB), decltype(m)::value % NDB); },
                                     [&](auto m, bf16x8 f) {
                                         constexpr int db = decltype(m)::value % NDB, c = decltype(m)::value / NDB;
                                         oacc[db] = mfma32(f, pf[c], oacc[db]);
                                     });
            if (more) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // (V has left LDS)
                load(v_load, v_head, v_rsrc, v_row_bytes, v_lds);
            }
        }
        // ---- the waves' (m, l, O) become one: every wave leaves its O in its own tiles, quad by quad, and adds up every
        // NW-th quad of all waves
        __shared__ float s_ml[NW][2][32];
        const float l_wave = l_run + swap_halves(l_run);
        if (half == 0) {
            s_ml[w][0][l32] = m_run;
            s_ml[w][1][l32] = l_wave;
        }
        f32x4* mine = (f32x4*)(smem + w * TILE) + lane;
#pragma unroll
        for (int q = 0; q < D / 8; ++q)
            mine[q * 64] = f32x4{oacc[q >> 2][4 * (q & 3)], oacc[q >> 2][4 * (q & 3) + 1], oacc[q >> 2][4 * (q & 3) + 2], oacc[q >> 2][4 * (q & 3) + 3]};
        __syncthreads();
        float m = -INFINITY, l = 0.0f, wgt[NW];
#pragma unroll
        for (int v = 0; v < NW; ++v) m = fmaxf(m, s_ml[v][0][l32]);
        const float m_from = m == -INFINITY ? 0.0f : m;     // (no key at all: every weight 0)
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            wgt[v] = fast_exp2(s_ml[v][0][l32] - m_from);
            l += wgt[v] * s_ml[v][1][l32];
        }
        if (!real_row) return;
        const float inv = l > 0.0f ? 1.0f / l : 0.0f;
        for (int q = w; q < D / 8; q += NW) {
            f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int v = 0; v < NW; ++v) o += wgt[v] * *((const f32x4*)(smem + v * TILE) + q * 64 + lane);
            u32x2 pk;
            pk[0] = pack_bf16(o[0] * inv, o[1] * inv);
            pk[1] = pack_bf16(o[2] * inv, o[3] * inv);
            *(u32x2*)(o_ptr + 8 * q + 4 * half) = pk;
        }
        if (w == 0 && half == 0) *lse_ptr = l > 0.0f ? (m + fast_log2(l)) * kLn2 : -INFINITY;
        return;
    } else if constexpr (UNITS) {
        // 32 keys at a time through a ring of three slots, two units ahead: unit u + 2 is asked for when every
        // wave is done with u - 1, whose slot it takes.
        constexpr uint32_t UT = 32 * D * 2;
        using UnitLoader = WaveTileLoader<D, NW, 32>;
        const UnitLoader ku_loader(a.k_ss, w, lane), vu_loader(a.v_ss, w, lane);
        TileWalk<PAGED, 32> uwalk(a.full_idx + line * a.NC, a.kv_idx + line * a.NC, n_full, n_part, 2 * a.sub, a.Bk,
                                  PAGED ? a.phys_full_idx + line * a.NC : nullptr, PAGED ? a.phys_kv_idx + line * a.NC : nullptr, backwards);
        const int TU = 2 * T;
        int kv_of[3];
        bool part_of[3];
        auto fetch = [&](int u, auto slot_tag) {
            constexpr int SLOT = decltype(slot_tag)::value;
            int pg = 0, pr = 0, soff;
            i32x4 rsrc;
            const int kv = uwalk.next(part_of[SLOT], pg, pr);
            kv_of[SLOT] = kv;
            if (part_of[SLOT]) make_tags(SLOT, kv, u);
            tile_src(k_head, k_rsrc, k_row_bytes, kv, pg, pr, rsrc, soff);
            ku_loader.start(rsrc, smem_bytes + SLOT * 2 * UT, soff);
            tile_src(v_head, v_rsrc, v_row_bytes, kv, pg, pr, rsrc, soff);
            vu_loader.start(rsrc, smem_bytes + SLOT * 2 * UT + UT, soff);
        };
        auto unit_step = [&](int u, auto slot_tag) {
            constexpr int SLOT = decltype(slot_tag)::value;
            if (u + 1 < TU) wait_vmem_but<2 * UnitLoader::NI>();     // (unit u + 1 may still be under way)
            else wait_vmem();
            __syncthreads();
            const int kv = kv_of[SLOT];
            const bool partial = part_of[SLOT];
            if (u + 2 < TU) fetch(u + 2, std::integral_constant<int, (SLOT + 2) % 3>{});
            if (!hidden_block(hidden_of(u >> 1) >> (u & 1), partial, kv, 0)) {
                f32x16 s;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < D / 16; ++ks) s = mfma32(k_reader.read(smem_bytes + SLOT * 2 * UT, 0, ks), qf[ks], s);
                bf16x8 pf[2];
                softmax(s, kv, partial, SLOT, 0, pf);
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        oacc[db] = mfma32(v_reader.read(smem_bytes + SLOT * 2 * UT + UT, 16 * c, db), pf[c], oacc[db]);
            }
        };
        const std::integral_constant<int, 0> s0;
        const std::integral_constant<int, 1> s1;
        const std::integral_constant<int, 2> s2;
        fetch(0, s0);
        fetch(1, s1);
        int u = 0;
        for (; u + 2 < TU; u += 3) {
            unit_step(u, s0);
            unit_step(u + 1, s1);
            unit_step(u + 2, s2);
        }
        if (u < TU) unit_step(u, s0);
        if (u + 1 < TU) unit_step(u + 1, s1);
    } else if constexpr (PAIRS) {
        // Every wave takes its 32 keys of every tile (whole: all 64, one half after the other), K and V one tile ahead.
        first_tile();
        auto pair_step = [&](int t, auto buf_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            wait_vmem();
            __syncthreads();        // tile t has landed, and nobody still reads tile t - 1
            const uint32_t hid = hidden_of(t) >> my_keys;
            const int kv0 = kv_t;
            const bool partial = part_t;
            if (t + 1 < T) {
                kv_t = walk.next(part_t, pg_t, pr_t);
                load_k(BUF ^ 1, kv_t, pg_t, pr_t);
                load_v(BUF ^ 1, kv_t, pg_t, pr_t);
                if (part_t) make_tags(BUF ^ 1, kv_t, t + 1);
            }
            int keys = my_keys;
            do {
                const int kv = kv0 + 32 * keys;
                if (!hidden_block(hid, partial, kv, 0)) {
                    f32x16 s;
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
                    read_ahead<D / 16>([&](auto m) { return k_reader.read(smem_bytes + BUF * (TILE * 2), 0, decltype(m)::value); },
                                       [&](auto m, bf16x8 f) { s = mfma32(f, qf[decltype(m)::value], s); });
                    bf16x8 pf[2];
                    softmax(s, kv, partial, BUF, keys, pf);
                    constexpr int NDB = D / 32;
                    read_ahead<2 * NDB>([&](auto m) { return v_reader.read(smem_bytes + (2 + BUF) * (TILE * 2), 16 * (decltype(m)::value / NDB), decltype(m)::value % NDB); },
                                        [&](auto m, bf16x8 f) {
                                            constexpr int db = decltype(m)::value % NDB, c = decltype(m)::value / NDB;
                                            oacc[db] = mfma32(f, pf[c], oacc[db]);
                                        });
                }
                if (!MIXED || !whole) break;
                keys ^= 1;
                k_reader.move(keys ? 64 * D : -64 * D);
                v_reader.move(keys ? 64 * D : -64 * D);
            } while (keys);
        };
        int t = 0;
        for (; t + 1 < T; t += 2) {
            pair_step(t, std::integral_constant<int, 0>{});
            pair_step(t + 1, std::integral_constant<int, 1>{});
        }
        if (t < T) pair_step(t, std::integral_constant<int, 0>{});
        if (!MIXED || !whole) {
            // ---- the two waves of the same rows become one: each finishes half of the dims and hands over the other half
            __shared__ float s_ml[NW][2][32];
            const float l_wave = l_run + swap_halves(l_run);
            if (half == 0) {
                s_ml[w][0][l32] = m_run;
                s_ml[w][1][l32] = l_wave;
            }
            constexpr int HDB = D / 64;
            __syncthreads();            // (the last tile has been read)
            f32x4* give = (f32x4*)smem + w * (HDB * 4 * 64) + lane;
#pragma unroll
            for (int q = 0; q < HDB * 4; ++q) {
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = my_keys ? oacc[q >> 2][4 * (q & 3) + i] : oacc[HDB + (q >> 2)][4 * (q & 3) + i];
                give[q * 64] = v;
            }
            __syncthreads();
            const float m_other = s_ml[w ^ 2][0][l32], m = fmaxf(m_run, m_other), m_from = m == -INFINITY ? 0.0f : m;
            const float mine = fast_exp2(m_run - m_from), theirs = fast_exp2(m_other - m_from);
            const float l = mine * l_wave + theirs * s_ml[w ^ 2][1][l32];
            const float inv = l > 0.0f ? 1.0f / l : 0.0f;
            if (!real_row) return;
            const f32x4* take = (const f32x4*)smem + (w ^ 2) * (HDB * 4 * 64) + lane;
#pragma unroll
            for (int q = 0; q < HDB * 4; ++q) {
                f32x4 o = theirs * take[q * 64];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(mine, my_keys ? oacc[HDB + (q >> 2)][4 * (q & 3) + i] : oacc[q >> 2][4 * (q & 3) + i], o[i]) * inv;
                u32x2 pk;
                pk[0] = pack_bf16(o[0], o[1]);
                pk[1] = pack_bf16(o[2], o[3]);
                *(u32x2*)(o_ptr + (my_keys * HDB + (q >> 2)) * 32 + 8 * (q & 3) + 4 * half) = pk;
            }
            if (my_keys == 0 && half == 0) *lse_ptr = l > 0.0f ? (m + fast_log2(l)) * kLn2 : -INFINITY;
            return;
        }
    } else if constexpr (PLAIN) {
        // One block of 32 keys after the other, K and V one tile ahead.  A wave leaves out the blocks that
        // the mask hides from all of its rows.
        first_tile();
        auto plain_step = [&](int t, auto buf_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            wait_vmem();
            __syncthreads();        // tile t has landed, and nobody still reads tile t - 1
            const uint32_t hid = hidden_of(t);
            const int kv0 = kv_t;
            const bool partial = part_t;
            if (t + 1 < T) {
                kv_t = walk.next(part_t, pg_t, pr_t);
                load_k(BUF ^ 1, kv_t, pg_t, pr_t);
                load_v(BUF ^ 1, kv_t, pg_t, pr_t);
                if (part_t) make_tags(BUF ^ 1, kv_t, t + 1);
            }
            static_for<0, 2>([&](auto kvb_tag) {
                constexpr int kvb = decltype(kvb_tag)::value;
                if (!hidden_block(hid, partial, kv0 + 32 * kvb, kvb)) {
                    f32x16 s;
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
                    for (int ks = 0; ks < D / 16; ++ks)
                        s = mfma32(k_reader.read(smem_bytes + BUF * (TILE * 2), kvb * 32, ks), qf[ks], s);
                    bf16x8 pf[2];
                    softmax(s, kv0 + 32 * kvb, partial, BUF, kvb, pf);
                    pv(buf_tag, kvb, pf);
                }
            });
        };
        int t = 0;
        for (; t + 1 < T; t += 2) {
            plain_step(t, std::integral_constant<int, 0>{});
            plain_step(t + 1, std::integral_constant<int, 1>{});
        }
        if (t < T) plain_step(t, std::integral_constant<int, 0>{});
    } else {
        first_tile();
        if (T > 1) {
            kv_t1 = walk.next(part_t1, pg_t1, pr_t1);
            load_k(1, kv_t1, pg_t1, pr_t1);
        }
        wait_vmem();
        __syncthreads();
        f32x16 s_cur[2], s_next[2];
        qk(std::integral_constant<int, 0>{}, s_cur, [](auto) {});

        // One tile (t & 1 == BUF).  S^T of tile t+1 (MFMA) is issued next to the softmax of tile t (VALU),
        // P V of the first 32 keys next to the softmax of the second 32.
        auto tile_step = [&](int t, auto buf_tag, auto has_next_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            constexpr bool HAS_NEXT = decltype(has_next_tag)::value;
            // Everything this wave asked for has landed; after the barrier so has everyone else's, and
            // nobody still reads K(t) [buffer BUF] or V(t-1) [buffer BUF ^ 1], which are refilled next.
            wait_vmem();
            __syncthreads();
            // K(t+2) and V(t+1) are loaded piece by piece between the MFMAs of S^T(t+1): a wave waits on
            // every load instruction until the memory pipe has taken it, and a burst of them from all
            // waves at once keeps everybody waiting
            const bool ld_k = t + 2 < T;
            if (ld_k) kv_t2 = walk.next(part_t2, pg_t2, pr_t2);
            i32x4 k_src, v_src;
            int k_soff, v_soff;
            tile_src(k_head, k_rsrc, k_row_bytes, kv_t2, pg_t2, pr_t2, k_src, k_soff);
            tile_src(v_head, v_rsrc, v_row_bytes, kv_t1, pg_t1, pr_t1, v_src, v_soff);
            const int kv0 = kv_t;
            const bool partial = part_t;
            if constexpr (HAS_NEXT) {
                if (part_t1) make_tags(BUF ^ 1, kv_t1, t + 1);
            }
            bf16x8 pf[2];
            if constexpr (HAS_NEXT) {
                using L = decltype(k_loader);
                constexpr int NP = 2 * L::NI, NMQ = 2 * (D / 16);
                qk(std::integral_constant<int, BUF ^ 1>{}, s_next, [&](auto m_tag) {
                    static_for<0, NP>([&](auto p_tag) {
                        constexpr int p = decltype(p_tag)::value;
                        if constexpr (p * NMQ / NP == decltype(m_tag)::value) {
                            if constexpr (p < L::NI) {
                                if (ld_k) k_loader.template start_one<p>(k_src, smem_bytes + BUF * (TILE * 2), k_soff);
                            } else {
                                v_loader.template start_one<p - L::NI>(v_src, smem_bytes + (2 + (BUF ^ 1)) * (TILE * 2), v_soff);
                            }
                        }
                    });
                });
            }
            softmax(s_cur[0], kv0, partial, BUF, 0, pf);
            pv(buf_tag, 0, pf);
            softmax(s_cur[1], kv0 + 32, partial, BUF, 1, pf);
            pv(buf_tag, 1, pf);
            if constexpr (HAS_NEXT) {
#pragma unroll
                for (int kvb = 0; kvb < 2; ++kvb) s_cur[kvb] = s_next[kvb];
            }
            kv_t = kv_t1, part_t = part_t1;
            kv_t1 = kv_t2, part_t1 = part_t2;
            if constexpr (PAGED) pg_t1 = pg_t2, pr_t1 = pr_t2;
        };
        {
            const std::integral_constant<int, 0> b0;
            const std::integral_constant<int, 1> b1;
            int t = 0;
            for (; t + 2 < T; t += 2) {
                tile_step(t, b0, std::true_type{});
                tile_step(t + 1, b1, std::true_type{});
            }
            if (T - t == 2) {
                tile_step(t, b0, std::true_type{});
                tile_step(t + 1, b1, std::false_type{});
            } else {
                tile_step(t, b0, std::false_type{});
            }
        }
    }

    // ---- epilogue: O = O^T / l, LSE = ln 2 * (m + log2 l)
    const float l_tot = l_run + swap_halves(l_run);
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    if (!real_row) return;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            u32x2 pk;
            pk[0] = pack_bf16(oacc[db][4 * rg] * inv, oacc[db][4 * rg + 1] * inv);
            pk[1] = pack_bf16(oacc[db][4 * rg + 2] * inv, oacc[db][4 * rg + 3] * inv);
            *(u32x2*)(o_ptr + db * 32 + 8 * rg + 4 * half) = pk;
        }
    if (half == 0) *lse_ptr = l_tot > 0.0f ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
}

template <int D, uint32_t MASK, uint32_t SCORE, bool BOUNDED, bool PAGED>
int launch_fwd_shape(const FwdArgs& args, int Bq, hipStream_t st) {
    FwdArgs a = args;
    const unsigned grid = unit_grid(a.B * a.Hkv, a.G * a.NR);
    const LineShape rows_shape = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    auto order_units = [&](int rows, int per_cu) { a.abreast = units_abreast(a.B * a.Hkv, a.G * rows, per_cu, rows_abreast<MASK>(rows_shape, a.kv_len, D)); };
    if (const int waves = split_waves<MASK, SCORE>(a, D)) {
        const dim3 slices(unit_grid(a.B * a.Hkv, a.G * a.NR * (Bq / 32)));
        if (waves == 8) hipLaunchKernelGGL((fwd_kernel<D, 8, MASK, SCORE, BOUNDED, PAGED, false, false, true>), slices, dim3(512), 0, st, a);
        else hipLaunchKernelGGL((fwd_kernel<D, 4, MASK, SCORE, BOUNDED, PAGED, false, false, true>), slices, dim3(256), 0, st, a);
        return FLEXATTN_OK;
    }
    if (pairs_pay<MASK, BOUNDED>(a, D, grid)) {
        constexpr bool can_mix = mixed_pays<D, MASK, SCORE, BOUNDED>();
        const bool mixed = Bq == 128 && can_mix;
        a.halved = Bq == 64 ? 0 : mixed ? halved_rows(a.NR) : a.NR;
        order_units(a.NR + a.halved, D == 64 ? 4 : 2);
        const unsigned pieces = unit_grid(a.B * a.Hkv, a.G * (a.NR + a.halved));
        for (a.first_id = 0; a.first_id < pieces; a.first_id += kMaxLaunch) {
            const dim3 ids(min(pieces - a.first_id, kMaxLaunch));
            if (mixed) hipLaunchKernelGGL((fwd_kernel<D, 4, MASK, SCORE, BOUNDED, PAGED, false, false, false, true, can_mix>), ids, dim3(256), 0, st, a);
            else hipLaunchKernelGGL((fwd_kernel<D, 4, MASK, SCORE, BOUNDED, PAGED, false, false, false, true>), ids, dim3(256), 0, st, a);
        }
        return FLEXATTN_OK;
    }
    if (Bq != 128) return FLEXATTN_ERR_UNSUPPORTED;
    if constexpr (D == 128) {
        if constexpr (fwd_units<128, 4, MASK, SCORE>() != FwdUnits::kNever) {
            if (units_pay<MASK, SCORE>(a, grid)) {
                order_units(a.NR, 3);
                hipLaunchKernelGGL((fwd_kernel<128, 4, MASK, SCORE, BOUNDED, PAGED, true>), dim3(grid), dim3(256), 0, st, a);
                return FLEXATTN_OK;
            }
        }
        order_units(a.NR, 2);
    } else {
        constexpr bool dense = !mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW | FLEXATTN_M_DOCUMENT | FLEXATTN_M_NEIGHBORHOOD);
        if constexpr (fwd_plain<64, 4, BOUNDED>() && dense) {
            if (!plain_pays<SCORE>(a.kv_len, grid, rows_shape.uneven)) {
                order_units(a.NR, 3);
                hipLaunchKernelGGL((fwd_kernel<64, 4, MASK, SCORE, BOUNDED, PAGED, false, false>), dim3(grid), dim3(256), 0, st, a);
                return FLEXATTN_OK;
            }
        }
        order_units(a.NR, 4);
    }
    hipLaunchKernelGGL((fwd_kernel<D, 4, MASK, SCORE, BOUNDED, PAGED>), dim3(grid), dim3(256), 0, st, a);
    return FLEXATTN_OK;
}

template <uint32_t MASK, uint32_t SCORE, bool PAGED = false>
int launch_fwd_variant(const FwdArgs& a, int D, int Bq, hipStream_t st) {
    auto of = [&](auto head_dim) {
        constexpr int DD = decltype(head_dim)::value;
        if constexpr (SCORE & FLEXATTN_SCORE_SOFTCAP) {
            if (2.0f * a.p.softcap * kLog2e <= 100.0f) return launch_fwd_shape<DD, MASK, SCORE, true, PAGED>(a, Bq, st);
        }
        return launch_fwd_shape<DD, MASK, SCORE, false, PAGED>(a, Bq, st);
    };
    if (D == 64) return of(std::integral_constant<int, 64>{});
    if constexpr (PartialMask<MASK>::kCells) return FLEXATTN_ERR_UNSUPPORTED;        // (variant_of: the general kernels)
    else return of(std::integral_constant<int, 128>{});
}

}  // namespace flexattn
