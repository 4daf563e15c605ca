// Shared device/host pieces of libflexattn (gfx950 only): vector types, MFMA wrappers,
// the mask_mod / score_mod functors (paper sections 3.1 and 3.2) and host-side status helpers.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flexattn.h"

namespace flexattn {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// D[32x32] += A[32x16] * B[16x32], bf16 inputs, fp32 accumulate.
// Operand layout (wave64): lane l supplies A[row = l % 32][k-slots of half l / 32] and
// B[k-slots of half l / 32][col = l % 32], eight bf16 each; the k-slot <-> k mapping is the same
// for A and B, so any consistent choice contracts correctly.
// Result layout: register r of lane l holds D[row = 8 * (r / 4) + 4 * (l / 32) + r % 4][col = l % 32].
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Row of the 32x32 result tile held in register r by a lane of half `half` (= lane / 32).
__device__ __forceinline__ constexpr int crow(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// f(integral_constant<int, B>), ..., f(integral_constant<int, E - 1>)
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// acc + lo(pair) + hi(pair) for a packed pair of bf16 values (v_dot2c_f32_bf16).
__device__ __forceinline__ float pair_sum_bf16(uint32_t pair, float acc) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair), __builtin_bit_cast(bf16x2_t, 0x3f803f80u),
                                           acc, false);
}

// Load of read-only data at a wave-uniform address: constant address space, so the compiler may
// use the scalar cache and keep the load off the vector memory counter.
__device__ __forceinline__ int32_t ldc(const int32_t* p) {
    return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Exchange a value with the lane 32 away (the other half of the wave).
__device__ __forceinline__ float swap_halves(float v) { return __shfl_xor(v, 32, 64); }

// The values of the two lanes l, l ^ 16 (SWAP16) or l, l ^ 32 in one order or the other, so that a commutative
// operation on the pair is a reduction over it: one exchange in the vector unit (a shuffle goes through LDS, and
// takes six instructions to address).
struct LanePair {
    float a, b;
};
template <bool SWAP16>
__device__ __forceinline__ LanePair lane_pair(float v) {
    const unsigned u = __builtin_bit_cast(unsigned, v);
    if constexpr (SWAP16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
    }
}
// max(a, b) as one instruction (fmaxf first puts both through a max of their own to quieten NaNs)
__device__ __forceinline__ float raw_max(float a, float b) {
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
    return m;
}
// The larger of this lane's value and that of the lane 32 away.
__device__ __forceinline__ float max_halves(float v) {
    const LanePair p = lane_pair<false>(v);
    return raw_max(p.a, p.b);
}

// This lane's number in its wave, worked out here and now.
__device__ __forceinline__ int lane_again() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
    return lane;
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    bf16x2 v;
    v[0] = (bf16)lo;
    v[1] = (bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// ---------------------------------------------------------------------------------------
// mask_mod: OR of up to two AND-terms over the primitive predicates.
// ---------------------------------------------------------------------------------------
// Token index -> pixel of the canvas, for the neighborhood mask (appendix, Neighborhood Attention).
struct CanvasOrder {
    int width, layout, tile_log2, tiles_x;
    float inv_width, inv_tiles_x;
    __device__ __forceinline__ explicit CanvasOrder(const flexattn_mod_params& p) {
        width = p.na_width;
        layout = p.na_layout;
        tile_log2 = p.na_tile > 0 ? 31 - __builtin_clz((unsigned)p.na_tile) : 0;
        tiles_x = width >> tile_log2;
        inv_width = fast_rcp((float)width);
        inv_tiles_x = fast_rcp((float)tiles_x);
    }
    // n = quot * d + rem for 0 <= n < 2^24: a float estimate of the quotient (off by one at most),
    // then one exact correction step
    __device__ __forceinline__ static void divmod(int n, int d, float inv_d, int& quot, int& rem) {
        int qq = (int)(((float)n + 0.5f) * inv_d);
        int rr = n - qq * d;
        const bool lo = rr < 0, hi = rr >= d;
        quot = qq + (hi ? 1 : 0) - (lo ? 1 : 0);
        rem = rr + (lo ? d : 0) - (hi ? d : 0);
    }
    // every second bit of v, packed (the inverse of interleaving with zeros)
    __device__ __forceinline__ static int even_bits(uint32_t v) {
        v &= 0x55555555u;
        v = (v | (v >> 1)) & 0x33333333u;
        v = (v | (v >> 2)) & 0x0f0f0f0fu;
        v = (v | (v >> 4)) & 0x00ff00ffu;
        v = (v | (v >> 8)) & 0x0000ffffu;
        return (int)v;
    }
    __device__ __forceinline__ void pixel(int n, int& x, int& y) const {
        if (layout == FLEXATTN_NA_MORTON) {
            x = even_bits((uint32_t)n);
            y = even_bits((uint32_t)n >> 1);
        } else if (layout == FLEXATTN_NA_TILED) {
            const int in_tile = n & ((1 << (2 * tile_log2)) - 1);
            int ty, tx;
            divmod(n >> (2 * tile_log2), tiles_x, inv_tiles_x, ty, tx);
            y = (ty << tile_log2) + (in_tile >> tile_log2);
            x = (tx << tile_log2) + (in_tile & ((1 << tile_log2) - 1));
        } else {
            divmod(n, width, inv_width, y, x);
        }
    }
};

// Which 32 x 32 blocks of a neighborhood mask hide every pair, found from boxes around the pixels of 32
// consecutive tokens.  Of the tiles a BlockMask of 128 x 64 blocks lists, a wave's 32 queries meet only some:
// 15 of 24 32-key blocks with 8 x 8 tiles and K = 13.
struct CanvasBlocks {
    CanvasOrder order;
    int t, tiles_x, w, h, r;    // tiles of 2^t x 2^t pixels (row-major: of one pixel), tiles_x side by side
    float inv_tiles_x;
    bool morton, known;         // known: the queries are the pixels (no offsets)
    struct Box {
        int x0, x1, y0, y1;
    };
    __device__ __forceinline__ explicit CanvasBlocks(const flexattn_mod_params& p) : order(p) {
        t = p.na_layout == FLEXATTN_NA_TILED ? order.tile_log2 : 0;
        w = p.na_width;
        h = p.na_height;
        tiles_x = w >> t;
        inv_tiles_x = fast_rcp((float)tiles_x);
        r = p.na_kernel >> 1;
        morton = p.na_layout == FLEXATTN_NA_MORTON;
        known = p.q_offsets == nullptr;
    }
    // around the pixels of the tokens n .. n + 31, n a multiple of 32
    __device__ __forceinline__ Box tokens(int n) const {
        if (morton) {               // 8 x 4 pixels
            const int x = CanvasOrder::even_bits((uint32_t)n), y = CanvasOrder::even_bits((uint32_t)n >> 1);
            return {x, x + 7, y, y + 3};
        }
        int tx, ty;
        CanvasOrder::divmod(n >> (2 * t), tiles_x, inv_tiles_x, ty, tx);
        if (2 * t >= 5) {           // inside one tile: whole lines of it, or a part of one
            const int in = n & ((1 << (2 * t)) - 1), lines = t >= 5 ? 1 : 32 >> t, len = t >= 5 ? 32 : 1 << t;
            const int x = (tx << t) + (in & ((1 << t) - 1)), y = (ty << t) + (in >> t);
            return {x, x + len - 1, y, y + lines - 1};
        }
        // tiles side by side, which may go on at the start of the next line of tiles
        const int end = tx + (32 >> (2 * t)) - 1;
        if (end < tiles_x) return {tx << t, (end << t) + (1 << t) - 1, ty << t, (ty << t) + (1 << t) - 1};
        int lines, rest;
        CanvasOrder::divmod(end, tiles_x, inv_tiles_x, lines, rest);
        return {0, w - 1, ty << t, ((ty + lines) << t) + (1 << t) - 1};
    }
    // around the windows of the queries n .. n + 31
    __device__ __forceinline__ Box windows(int n) const {
        Box b = tokens(n);
        b.x0 = min(max(b.x0, r), w - 1 - r) - r;
        b.x1 = min(max(b.x1, r), w - 1 - r) + r;
        b.y0 = min(max(b.y0, r), h - 1 - r) - r;
        b.y1 = min(max(b.y1, r), h - 1 - r) + r;
        return b;
    }
    __device__ __forceinline__ bool hidden(const Box& query_windows, const Box& keys) const {
        return known && (keys.x1 < query_windows.x0 || keys.x0 > query_windows.x1 || keys.y1 < query_windows.y0 ||
                         keys.y0 > query_windows.y1);
    }
    // bit 2 w + j: the 32 keys from kv0 + 32 j on are hidden from the 32 queries from q0 + 32 w on
    template <int NW>
    __device__ __forceinline__ uint32_t hidden_bits(const Box (&query_windows)[NW], int kv0) const {
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const Box keys = tokens(kv0 + 32 * j);
#pragma unroll
            for (int w = 0; w < NW; ++w) bits |= hidden(query_windows[w], keys) ? 1u << (2 * w + j) : 0u;
        }
        return bits;
    }
};

struct NoCanvas {
    __device__ __forceinline__ explicit NoCanvas(const flexattn_mod_params&) {}
    __device__ __forceinline__ void pixel(int, int&, int&) const {}
};

// Of the eighth of a launch's units that an XCD takes (whole ones): `sets` sets, one after the other, of 2^side units whose
// pieces take turns (the last set: and what is left over).
struct UnitSets {
    int side, sets;
};
// Workgroup -> (unit, rank): which KV head of which batch entry, and which of its per_unit pieces (longest first).
// Workgroup ids go to the 8 XCDs in turn.  Eight units at a time, a unit's pieces all go to one XCD, so that its K and V
// stay in that XCD's L2.  The 1 .. 7 units beyond a multiple of eight come first and are cut into eighths, every eighth
// piece each; an XCD takes as many eighths side by side as there are such units: all XCDs have the same work, with
// the pieces of at most two units in an L2.  (First, because what comes last ends the launch, and the long pieces of a whole
// unit then start earlier.)  False: nothing to do (the last round of eighths).  (A whole unit on one XCD leaves others idle:
// us, that -> this, causal: S = 16384, D = 128, 1 head, forward 472 -> 289, dK/dV 832 -> 269, dQ 574 -> 326; 3 heads, D = 64,
// 309 -> 213, 537 -> 262, 371 -> 238; S = 8192, D = 128, 16 query and 2 KV heads 874 -> 285, 1855 -> 1074, 1064 -> 369; S = 4096, 9
// heads, D = 64, 76 -> 54, 82 -> 61, 83 -> 61, D = 128, 105 -> 80, 130 -> 93, 130 -> 92; 8 and 16 heads the same within 2 %.)
// The units of a set take turns piece by piece, so that the long pieces of all start before the short ones (units_abreast).  (A launch that all runs at once
// lasts as long as its workgroups' way to their first load: kernels whose units always come one by one say so themselves, and the others' arguments lie
// beside those that are read here anyway, where a line of their own cost 0.5 us: dK/dV, D = 128, causal, S = 1024, 16 heads.)
__device__ __forceinline__ bool unit_of_workgroup(unsigned id, int units, int per_unit, UnitSets abreast, int& unit, int& rank) {
    const int xcd = id & 7, rest = units & 7, rest_pieces = rest * ((per_unit + 7) >> 3);
    const int k = id >> 3;
    if (k >= rest_pieces) {
        const int p = k - rest_pieces, u = p / per_unit;
        if (abreast.side == 0) {
            unit = u * 8 + xcd;
            rank = p - u * per_unit;
            return true;
        }
        const int set = min(u >> abreast.side, abreast.sets - 1);
        const int first = set << abreast.side, in = p - first * per_unit;
        int of = in >> abreast.side, turn = in & ((1 << abreast.side) - 1);
        if (const int last = (units >> 3) - first; set + 1 == abreast.sets && last != 1 << abreast.side) {
            of = in / last;
            turn = in - of * last;
        }
        unit = (first + turn) * 8 + xcd;
        rank = of;
        return true;
    }
    const int round = k / rest, eighth = xcd * rest + k - round * rest;
    unit = (units & ~7) + (eighth >> 3);
    rank = 8 * round + (eighth & 7);
    return rank < per_unit;
}
__device__ __forceinline__ bool unit_of_workgroup(int units, int per_unit, UnitSets abreast, int& unit, int& rank) {
    return unit_of_workgroup(blockIdx.x, units, per_unit, abreast, unit, rank);
}
// The unit in its place where an XCD takes its whole units the other way round.  Kernels that follow one another on the same
// tensors do so in turn -- forward up, dQ down, dK/dV up; where dS is kept in memory the row scalars up, dK/dV down, dQ up -- so that
// the second starts on what the first has touched last, of which the memory's cache of 256 MB still holds as much.  (Bound by nothing but what misses
// that cache: smaller tensors take the same time, and an XCD keeps its units, else those that fit its L2 lose 3 %.)  us, dQ and dK/dV together,
// both up -> this: causal, D = 64, S = 1024 x 1024 heads 726 -> 703, 512 x 1024 251 -> 241, 2048 x 256 557 -> 545; D = 128, 1024 x 256
// 362 -> 350, 200 x 1024 182 -> 173; no mask, D = 64, 1000 x 512 527 -> 516; canvas 64 x 64, K = 9, 128 heads 334 -> 324; a step with
// dS in memory, soft-cap, D = 128, 1024 x 256 489 -> 479, 2048 x 128 762 -> 754.
__host__ __device__ inline int last_unit_first(int unit, int units) {
    const int whole = units & ~7;
    return unit < whole ? whole - 8 - (unit & ~7) + (unit & 7) : unit;
}
__host__ __device__ inline UnitSets one_by_one(int units) { return {0, units >= 8 ? units >> 3 : 1}; }
// How many units take turns.  Pieces of uneven length end a launch sooner if the short ones of many units come last, and units that
// a set's workgroups hold at once share the XCD's L2 all the same.  So: as many as make two rounds of the XCD's workgroups (per_cu of them on each of 32 CUs),
// at most 8 (rows), 4 (columns: dK/dV, S = 1024, 1024 heads, 436 one by one, 417 four, 429 eight, 468 all): with more, a unit's K and V
// have left L2 before its next piece.  Rows of one length gain nothing, and a unit that fills the XCD by itself loses the lockstep in which its
// workgroups stream K and V (chunks of 2048 on 4096 .. 14336 cached keys, 4 x 32 / 8 heads, 1277 -> 1571 with four): one by one.
// us, one by one -> so (one MI355X), causal: forward / dQ / dK/dV, D = 64, S = 1024 x 1024 heads 219 -> 202 / 284 -> 263 / 436 -> 417, 1024 x 256 60 -> 51 / 78 -> 64 /
// 109 -> 102, 2048 x 256 178 -> 165 / 238 -> 217 / 344 -> 336, 4096 x 64 181 -> 153 / 231 -> 219 / 317 -> 298, 8192 x 64 635 -> 577 / 821 -> 764 / 1145 -> 1122, 1500 x 40
// 27 -> 22 / 32 -> 27 / 42 -> 35, 200 x 2048 43 -> 43 / 57 -> 54 / 128 -> 112, soft-cap, 1024 x 256 86 -> 68 / 113 -> 89 / 125 -> 117, 16 / 4 heads, 2048 x 128
// 92 -> 83 / 122 -> 121 / 189 -> 156; D = 128, 1024 x 256 113 -> 98 / 150 -> 135 / 224 -> 215, 2048 x 128 174 -> 157 / 230 -> 210 / 337 -> 328, 8192 x 32 552 -> 532 /
// 741 -> 710 (its columns one by one); the captured sums of ALiBi, D = 64, 2048 x 64 82 -> 60; documents of 256 to 4096, D = 64, 8192 x 64 244 -> 218 / 302 -> 273 (columns gain
// nothing: 407), D = 128, 4096 x 64 224 -> 189 / 286 -> 252; windows of 512, D = 64, 4096 x 64 54 -> 53 / 69 -> 67.
constexpr int kRowsAbreast = 8, kColumnsAbreast = 4;
inline UnitSets units_abreast(int units, int per_unit, int per_cu, int most) {
    const int mine = units >> 3, round = 32 * per_cu;
    const int limit = per_unit < 4 && most > 4 ? 4 : most;      // (24 workgroups to a set: 32 CUs are dealt them unevenly, dQ, 300 x 512 26 -> 27)
    int side = 0;
    while (2 << side <= limit && 2 << side <= mine && (int64_t)per_unit << side < 2 * round) ++side;
    return {side, mine > 0 ? mine >> side : 1};
}
__host__ __device__ inline unsigned unit_grid(int units, int per_unit) {
    return 8u * ((unsigned)(units >> 3) * (unsigned)per_unit + (unsigned)(units & 7) * (unsigned)((per_unit + 7) / 8));
}
// A launch counts its work items in 32 bits: 2^24 workgroups of 256 are too many (some are then left out, without an error).
// What may need more takes several launches of at most this many.
constexpr unsigned kMaxLaunch = 1u << 23;

// Tiles of the longest row of blocks (the first in work order) of a plane whose rows start at plane_rows.
__device__ __forceinline__ int longest_row(const int32_t* order, const int32_t* full_num, const int32_t* part_num, int64_t plane_rows, int NR, int sub) {
    const int64_t longest = plane_rows + (order ? min(max(ldc(order + plane_rows), 0), NR - 1) : NR - 1);
    return (ldc(full_num + longest) + ldc(part_num + longest)) * sub;
}
// Documents of a few hundred tokens, which the host cannot tell from longer ones, head by head: their rows are bound by K and V, which then stay
// in L2 (D = 64, 8192 x 64, us, head by head / abreast: of 30 to 300 tokens, forward 61 / 67, dQ 85 / 91, of 100 to 1000 95 / 95, 130 / 133, of 256 to 4096
// 249 / 223, 304 / 278).  By the longest row of the launch's first plane, which all workgroups ask alike, and also where no head takes turns (dQ, D = 64, 12 heads of
// 3000, documents of 16 to 100: 13.3, asked only where some do 14.0, D = 128 21.1 and 21.8: the lines are needed next anyway).
constexpr int kAbreastTiles = 24;
__device__ __forceinline__ UnitSets abreast_if_long(UnitSets abreast, int units, int longest) {
    return longest > kAbreastTiles ? abreast : one_by_one(units);
}
// Workgroups that take either a row of blocks of 128 rows as a whole or one of its halves (MIXED in the forward and dQ): the first `halved` ranks in
// halves, but where the longest row of the unit's first plane (the first in work order) is short, none; the ids that are left over then are the
// last.  rem: the piece of a unit (G query heads) of G * (NR + halved) -> the piece of G * NR rows.  False: nothing to do.
__device__ __forceinline__ bool half_or_row(const int32_t* order, const int32_t* full_num, const int32_t* part_num, int64_t plane_rows, int NR, int G,
                                            int sub, int halved, int short_tiles, int& rem, int& slice, bool& whole) {
    const int halves = longest_row(order, full_num, part_num, plane_rows, NR, sub) > short_tiles ? 2 * halved * G : 0;
    if (rem - (halves >> 1) >= NR * G) return false;
    whole = rem >= halves;
    slice = whole ? 0 : rem & 1;
    rem = whole ? rem - (halves >> 1) : rem >> 1;
    return true;
}
constexpr int halved_rows(int NR) { return (NR + 2) / 3; }

// Offset conversion for inference (section 5.2): the position the mods see for query row 0 of
// batch entry b.
__device__ __forceinline__ int q_offset_of(const flexattn_mod_params& p, int b) {
    return p.q_offsets ? ldc(p.q_offsets + b) : 0;
}

// ---------------------------------------------------------------------------------------
// mask_mod of a PARTIAL block inside the MFMA kernels.
//
// A lane holds 16 elements of a 32 x 32 block that share its query (forward, dQ) or its key (dK/dV) and
// run along the other index at the compile-time positions crow(r, 0) behind a base.  Everything in the
// mask that compares indices is an interval of those positions per term, so it is worked out once per
// block as a bit mask (about ten instructions) and costs an element one bit-field extract and one
// select by bits, whatever the composition.  What is looked up per token -- the document id, the pixel of
// the canvas -- is a 32-bit tag, the other side's in an LDS table of the tile.  Equal document ids become
// bits as well, by one ballot per distinct id of the 32 tokens (one or two in packed documents).  The pixels that
// match a lane's are a rectangle, of which 32 consecutive tokens hold a piece that is worked out line by line
// (tokens_inside; the tags of the block's first token say where it lies), or, in kernels of their own for canvases that cut 32
// tokens into many pieces (canvas_by_tags), compared per element, and for those whose 32 tokens are always a cell of 8 x 4 pixels
// (canvas_in_cells) kept by pairs (CellMasks).
// (Evaluating the mask element by element instead -- the canvas decode of every key, a lane exchange or a
// table read per document id -- made PARTIAL blocks several times as expensive as FULL ones: neighborhood
// attention on 128 x 128 pixels, K = 13, D = 64, B = 4, H = 16: forward 0.98 ms, dK/dV 1.60 ms before, 0.42
// and 0.67 since; the forward 0.34 where it also leaves out the blocks CanvasBlocks finds hidden.  Pixels as rectangles instead
// of six instructions a score, B = 4, H = 16, us forward / backward: 128 x 128, K = 13, tiles of 8 x 8 282 -> 252 / 841 -> 807, row-major, 64 x 64,
// K = 9 78 -> 68 / 223 -> 215; 64 x 64, K = 9, Morton order 57 -> 53 / 181 -> 175, tiles of 16 x 16 72 -> 63 / 200 -> 189.)
// ---------------------------------------------------------------------------------------

// Position of element r of a lane's 16 (without the 4 * half that goes into the base).
__device__ __forceinline__ constexpr int elem_pos(int r) { return 8 * (r >> 2) + (r & 3); }

// bits p of lo <= p <= hi, for the positions 0 .. 27 that elem_pos() takes
__device__ __forceinline__ uint32_t interval_bits(int lo, int hi) {
    const int h = min(max(hi, -1), 27) + 1, l = min(max(lo, 0), 28);
    return ((1u << h) - 1u) & ~((1u << l) - 1u);
}

// All-ones if bit `pos` of `bits` is set, else 0 (the intrinsic, because the compiler turns the shifts it
// stands for, and the `and` that follows, into a test and a select: three instructions for two)
__device__ __forceinline__ uint32_t bit_mask(uint32_t bits, int pos) {
    return (uint32_t)__builtin_amdgcn_sbfe((int)bits, (uint32_t)pos, 1u);
}

// v where m is all-ones, 0 (or -inf) where it is 0
__device__ __forceinline__ float keep_or_zero(uint32_t m, float v) {
    return __builtin_bit_cast(float, m & __builtin_bit_cast(uint32_t, v));
}
__device__ __forceinline__ float keep_or_neg_inf(uint32_t m, float v) {
    return __builtin_bit_cast(float, (m & __builtin_bit_cast(uint32_t, v)) | (~m & 0xff800000u));
}

// A canvas whose matching pixels are compared token by token (canvas_by_tags); not accepted from callers.
constexpr uint32_t kCanvasByTags = 0x40u;
// A canvas whose 32 consecutive tokens are cells of 8 x 4 pixels (canvas_in_cells), line by line, or (both bits) in Z order.
constexpr uint32_t kCanvasCells = 0x80u, kCanvasCellsZ = 0xc0u;

template <uint32_t MASK>
struct PartialMask {
    static constexpr uint32_t T0 = MASK & 0xffu, T1 = (MASK >> 8) & 0xffu, PRIMS = T0 | T1;
    static constexpr uint32_t kTagged = FLEXATTN_M_DOCUMENT | FLEXATTN_M_NEIGHBORHOOD;
    static constexpr bool kDoc = (PRIMS & FLEXATTN_M_DOCUMENT) != 0, kCanvas = (PRIMS & FLEXATTN_M_NEIGHBORHOOD) != 0;
    static constexpr bool kTags = kDoc || kCanvas, kCells = kCanvas && (PRIMS & kCanvasCells) != 0,
                          kCellsZ = kCells && (PRIMS & kCanvasByTags) != 0, kByTags = kCanvas && !kCells && (PRIMS & kCanvasByTags) != 0;
    static constexpr int kMaxIds = 9;
    static_assert(!(kDoc && kCanvas), "one tag per token: documents or pixels");

    int window, prefix_len, ctx, kv_last;
    // pixels (x, y) as x | y << y_shift with one guard bit above each coordinate (guard): with the tag of
    // a query the top left corner of its window minus the guard bits, a = key tag - query tag has both
    // guard bits set iff x >= x0 and y >= y0, and span + 2 guard - a iff x <= x0 + span and y <= y0 + span.
    uint32_t guard, far;
    int y_shift;
    // How 32 consecutive tokens, the first at a multiple of 32, lie on the canvas: each line of it a run of its own (kLines, row-major),
    // lines of 2^line_log2 pixels below each other (kRows, tiles of 8 x 8 and more), or 8 x 4 in Z order (kZ).
    enum Way { kLines, kRows, kZ };
    int way, line_log2;
    std::conditional_t<kCanvas, CanvasOrder, NoCanvas> canvas;
    int na_r, na_w, na_h;

    __device__ __forceinline__ PartialMask(const flexattn_mod_params& p, int b, int kv_len) : canvas(p) {
        window = p.window;
        prefix_len = p.prefix_len;
        ctx = (PRIMS & FLEXATTN_M_CTX_LEN) ? ldc(p.ctx_lens + b) : 0;
        kv_last = kv_len - 1;
        guard = far = 0;
        y_shift = na_r = na_w = na_h = line_log2 = 0;
        way = kLines;
        if constexpr (kCanvas) {
            na_w = p.na_width;
            na_h = p.na_height;
            na_r = p.na_kernel >> 1;
            const int xb = 32 - __builtin_clz((unsigned)na_w), yb = 32 - __builtin_clz((unsigned)na_h);   // xb + yb <= 22
            y_shift = xb + 1;
            guard = (1u << xb) | (1u << (y_shift + yb));
            far = (uint32_t)(2 * na_r) * (1u | (1u << y_shift)) + 2u * guard;
            line_log2 = min(canvas.tile_log2, 5);
            way = p.na_layout == FLEXATTN_NA_MORTON ? kZ : p.na_layout == FLEXATTN_NA_TILED && line_log2 > 0 ? kRows : kLines;
        }
    }
    // Tags of a key and of a query (indices as the mods see them, in range).
    __device__ __forceinline__ uint32_t key_pixel(int kv) const {
        int x, y;
        canvas.pixel(kv, x, y);
        return (uint32_t)x | ((uint32_t)y << y_shift);
    }
    // top left corner of the window of a query: centred on its pixel, moved inside the canvas
    __device__ __forceinline__ void window_corner(int q, int& x, int& y) const {
        canvas.pixel(q, x, y);
        x = min(max(x, na_r), na_w - 1 - na_r) - na_r;
        y = min(max(y, na_r), na_h - 1 - na_r) - na_r;
    }
    __device__ __forceinline__ uint32_t query_pixel(int q) const {
        int x, y;
        window_corner(q, x, y);
        return ((uint32_t)x | ((uint32_t)y << y_shift)) - guard;
    }
    // what the table of a step's 32-query blocks holds (match_queries, keep_queries)
    __device__ __forceinline__ uint32_t query_block_tag(int q) const { return kByTags ? query_pixel(q) : key_pixel(q); }
    __device__ __forceinline__ bool pixels_match(uint32_t key_tag, uint32_t query_tag) const {
        const uint32_t a = key_tag - query_tag;
        return (a & (far - a) & guard) == guard;
    }

    // Bits of the elements whose index comparisons hold: `plain` for the terms that end there, `tagged` for
    // those that also want the tags to match.
    struct Bits {
        uint32_t plain, tagged;
        __device__ __forceinline__ void add(uint32_t term, uint32_t b) {
            if (term & kTagged) tagged |= b;
            else plain |= b;
        }
    };
    template <uint32_t TERM>
    __device__ __forceinline__ uint32_t row_term(int q, int kv_base) const {
        int hi = kv_last;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) hi = min(hi, q);
        if constexpr (TERM & FLEXATTN_M_PREFIX) hi = min(hi, prefix_len - 1);
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) hi = min(hi, ctx - 1);
        int lo = 0;
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) lo = __builtin_elementwise_sub_sat(q - kv_base, window);
        return interval_bits(lo, hi - kv_base);
    }
    // the lane holds query q and the keys kv_base + elem_pos(r)
    __device__ __forceinline__ Bits row_bits(int q, int kv_base) const {
        Bits out = {0u, 0u};
        out.add(T0, row_term<T0>(q, kv_base));
        if constexpr (T1 != 0) out.add(T1, row_term<T1>(q, kv_base));
        return out;
    }
    template <uint32_t TERM>
    __device__ __forceinline__ uint32_t key_term(int kv, int q_base) const {
        bool there = kv <= kv_last;
        if constexpr (TERM & FLEXATTN_M_PREFIX) there = there && kv < prefix_len;
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) there = there && kv < ctx;
        int lo = 0, hi = 27;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) lo = kv - q_base;
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) hi = __builtin_elementwise_add_sat(kv - q_base, window);
        return there ? interval_bits(lo, hi) : 0u;
    }
    // the lane holds key kv and the queries q_base + elem_pos(r)
    __device__ __forceinline__ Bits key_bits(int kv, int q_base) const {
        Bits out = {0u, 0u};
        out.add(T0, key_term<T0>(kv, q_base));
        if constexpr (T1 != 0) out.add(T1, key_term<T1>(kv, q_base));
        return out;
    }
    // Document masks: whether the 32 tokens of a wave (the id of token l % 32 in lane l; all lanes take part) belong to
    // more documents than packed ones do.
    __device__ __forceinline__ static bool scattered_ids(uint32_t id) {
        uint32_t left = 0xffffffffu;
#pragma unroll 1
        for (int n = 0; n < kMaxIds && left != 0; ++n)
            left &= ~(uint32_t)__ballot(id == (uint32_t)__builtin_amdgcn_readlane((int)id, __builtin_ctz(left)));
        return left != 0;
    }
    // `tags` (in LDS) holds the ids of the block's 32 tokens of the other index, `mine` is this lane's.  Packed documents
    // are matched by one ballot per id (all lanes of the wave take part); a wave whose own ids are scattered compares its
    // lanes' 16 elements one by one, which takes the time of about seven ids.  (64 ids at random, S = 4096, 32 heads, us, a
    // ballot per id throughout -> this: forward 349 -> 210 at D = 64, 386 -> 225 at D = 128, dQ 296 -> 175, 425 -> 277.  dK/dV
    // stays with the ballots: 272 -> 182, but packed documents 1 to 3 % slower.)
    __device__ __forceinline__ static void match_documents(Bits& bits, const uint32_t* tags, uint32_t mine, int l32, int half, bool scattered) {
        uint32_t same = 0;
        if (scattered) {
#pragma unroll 1
            for (int rg = 0; rg < 4; ++rg) {
                const u32x4 t = *(const u32x4*)&tags[8 * rg + 4 * half];
                const uint32_t four = (t[0] == mine ? 1u : 0u) | (t[1] == mine ? 2u : 0u) | (t[2] == mine ? 4u : 0u) | (t[3] == mine ? 8u : 0u);
                same |= four << (8 * rg);
            }
        } else {
            const uint32_t theirs = tags[l32];
            for (uint32_t left = 0xffffffffu; left != 0;) {
                const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)theirs, __builtin_ctz(left));
                const uint32_t equal = (uint32_t)__ballot(theirs == id);
                left &= ~equal;
                same |= mine == id ? equal : 0u;
            }
            same >>= 4 * half;
        }
        bits.plain |= bits.tagged & same;
    }
    // bits lo .. end - 1 of 32
    __device__ __forceinline__ static uint32_t span(int lo, int end) {
        const int l = min(max(lo, 0), 32), e = min(max(end, 0), 32);
        return (uint32_t)((1ull << e) - 1ull) & ~(uint32_t)((1ull << l) - 1ull);
    }
    // Which of 32 consecutive tokens, whose pixels are in `tags` (LDS; the first is asked), lie inside a lane's rectangle (corners
    // included).
    __device__ __forceinline__ uint32_t tokens_inside(const uint32_t* tags, int x0, int y0, int x1, int y1) const {
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)tags[0]), xm = (1u << (y_shift - 1)) - 1u;
        const int fx = (int)(first & xm), fy = (int)(first >> y_shift);
        if (way == kLines) {
            uint32_t bits = 0;
            if (na_w < 32) {                // several lines: the line's bits once, moved to each
                const uint32_t line = span(x0, x1 + 1), tall = (uint32_t)(y1 - y0);
                for (int y = fy, at = 32 - fx; at < 64; ++y, at += na_w)
                    bits |= (uint32_t)(y - y0) <= tall ? (uint32_t)(((uint64_t)line << at) >> 32) : 0u;
            } else {
                for (int y = fy, at = -fx; at < 32; ++y, at += na_w) bits |= y >= y0 && y <= y1 ? span(at + x0, at + x1 + 1) : 0u;
            }
            return bits;
        }
        uint32_t xs = span(x0 - fx, x1 + 1 - fx);
        if (way == kRows) {
            // (the line's bits, again for every line)
            xs = __builtin_amdgcn_perm(xs, xs, line_log2 == 3 ? 0x00000000u : line_log2 == 4 ? 0x01000100u : 0x03020100u);
            return xs & span((y0 - fy) << line_log2, (y1 + 1 - fy) << line_log2);
        }
        // token 16 x2 + 8 y1 + 4 x1 + 2 y0 + x0 of the pixel (x, y), bit by bit
        xs = (xs & 0x0fu) | ((xs & 0xf0u) << 12);
        xs = (xs & 0x00030003u) | ((xs & 0x000c000cu) << 2);
        xs |= xs << 2;
        xs |= xs << 8;
        uint32_t ys = span(y0 - fy, y1 + 1 - fy);
        ys = (ys & 0x3u) | ((ys & 0xcu) << 6);
        ys = (ys & 0x101u) | ((ys & 0x202u) << 1);
        ys |= ys << 1;
        ys |= ys << 4;
        ys |= ys << 16;
        return xs & ys;
    }
    // put(r, all-ones or 0) for each of a lane's elements: its query has the window at `query_tag`, they are the keys whose pixels
    // are in `tags` (LDS).  ONE_READ: there are no registers for four reads of them at a time.
    template <bool ONE_READ, typename F>
    __device__ __forceinline__ void mask_keys(Bits bits, const uint32_t* tags, uint32_t query_tag, int half, F&& put) const {
        if constexpr (kByTags) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const u32x4 t = *(const u32x4*)&tags[8 * rg + 4 * half];
                if constexpr (ONE_READ) asm volatile("" ::: "memory");
#pragma unroll
                for (int i = 0; i < 4; ++i) put(4 * rg + i, keep(bits, 4 * rg + i) | (pixels_match(t[i], query_tag) ? bit_mask(bits.tagged, elem_pos(4 * rg + i)) : 0u));
            }
        } else {
            const uint32_t corner = query_tag + guard;
            const int x0 = (int)(corner & ((1u << (y_shift - 1)) - 1u)), y0 = (int)(corner >> y_shift);
            bits.plain |= bits.tagged & (tokens_inside(tags, x0, y0, x0 + 2 * na_r, y0 + 2 * na_r) >> (4 * half));
#pragma unroll
            for (int r = 0; r < 16; ++r) put(r, keep(bits, r));
        }
    }
    // The queries that see a key are a rectangle too: those around it, and up to the border where the windows there reach
    // it.  Its corners (the key's own pixel twice where keep_queries compares tags); empty past the last key.
    __device__ __forceinline__ u32x2 key_corners(int kv) const {
        if (kv > kv_last) return u32x2{(1u << (y_shift - 1)) - 1u, 0u};      // (a column past any query's)
        const uint32_t tag = key_pixel(kv);
        if constexpr (kByTags) return u32x2{tag, tag};
        const int x = (int)(tag & ((1u << (y_shift - 1)) - 1u)), y = (int)(tag >> y_shift), d = 2 * na_r;
        const int x0 = x <= d ? 0 : x - na_r, x1 = x >= na_w - 1 - d ? na_w - 1 : x + na_r;
        const int y0 = y <= d ? 0 : y - na_r, y1 = y >= na_h - 1 - d ? na_h - 1 : y + na_r;
        return u32x2{(uint32_t)x0 | ((uint32_t)y0 << y_shift), (uint32_t)x1 | ((uint32_t)y1 << y_shift)};
    }
    // The lane's key has these key_corners(), its elements are the queries whose query_block_tag() is in `tags`: what keep_queries
    // wants to know of them (their bits, or the key's pixel).
    __device__ __forceinline__ Bits match_queries(const uint32_t* tags, u32x2 corners, int half) const {
        static_assert((T0 & ~(kCanvasByTags | kCanvasCells)) == FLEXATTN_M_NEIGHBORHOOD && T1 == 0, "a canvas with another predicate: dK/dV asks the pixels alone");
        if constexpr (kByTags) return Bits{corners[0], 0u};
        const uint32_t xm = (1u << (y_shift - 1)) - 1u;
        return Bits{tokens_inside(tags, (int)(corners[0] & xm), (int)(corners[0] >> y_shift), (int)(corners[1] & xm), (int)(corners[1] >> y_shift)) >> (4 * half), 0u};
    }
    // Cells: what a lane's rectangle of pixels leaves of a cell's elements.  Elements 2 p and 2 p + 1 are two pixels side by side, eight of them on a
    // line: line by line p = 2 y + x / 2 (for the half's four columns), in Z order the bits of p are y0, y1, x2.  So a pair of packed bf16 is kept by two of six
    // masks, one operation a pair where a mask per element takes two an element and its place in the block another 20.
    struct CellMasks {
        uint32_t x[2], lines;       // (all-ones or 0 for either pixel of a pair; a bit for each of four lines)
        __device__ __forceinline__ uint32_t of(int p) const { return x[kCellsZ ? p >> 2 : p & 1] & bit_mask(lines, kCellsZ ? p & 3 : p >> 1); }
        __device__ __forceinline__ uint32_t pair(uint32_t v, int p) const { return v & of(p); }
        // all-ones or 0
        __device__ __forceinline__ uint32_t element(int r) const {
            const int m = (int)of(r >> 1);
            return (uint32_t)(r & 1 ? m >> 16 : (int)((uint32_t)m << 16) >> 16);
        }
    };
    // The corner that the columns and lines of a wave's rectangles count from: its 32 queries' windows, or the queries around its 32 keys.
    struct CellBase {
        int col, line;
    };
    __device__ __forceinline__ static CellBase base_at(int x0, int y0) {
        return {__builtin_amdgcn_readfirstlane(x0 >> 3), __builtin_amdgcn_readfirstlane(y0 & ~3)};
    }
    __device__ __forceinline__ CellBase base_of_queries(const flexattn_mod_params& p, int q) const {
        const CanvasBlocks::Box w = CanvasBlocks(p).windows(q);
        return base_at(w.x0, w.y0);
    }
    __device__ __forceinline__ CellBase base_of_keys(const flexattn_mod_params& p, int kv) const {
        const CanvasBlocks::Box k = CanvasBlocks(p).tokens(kv);
        return base_at(k.x0 <= 2 * na_r ? 0 : k.x0 - na_r, k.y0 <= 2 * na_r ? 0 : k.y0 - na_r);
    }
    // A lane's rectangle (corners included) as 64 columns and 64 lines.
    __device__ __forceinline__ static u32x4 rectangle(int x0, int y0, int x1, int y1, CellBase base) {
        auto bits = [](int lo, int hi) { return (~0ull >> (63 - hi)) & (~0ull << lo); };
        const uint64_t xs = bits(x0 - 8 * base.col, x1 - 8 * base.col), ys = bits(y0 - base.line, y1 - base.line);
        return u32x4{(uint32_t)xs, (uint32_t)(xs >> 32), (uint32_t)ys, (uint32_t)(ys >> 32)};
    }
    __device__ __forceinline__ u32x4 query_rectangle(int q, CellBase base) const {
        int x, y;
        window_corner(q, x, y);
        return rectangle(x, y, x + 2 * na_r, y + 2 * na_r, base);
    }
    __device__ __forceinline__ u32x4 key_rectangle(int kv, CellBase base) const {
        int x, y;
        canvas.pixel(min(kv, kv_last), x, y);
        const int d = 2 * na_r;
        return rectangle(x <= d ? 0 : x - na_r, y <= d ? 0 : y - na_r, x >= na_w - 1 - d ? na_w - 1 : x + na_r, y >= na_h - 1 - d ? na_h - 1 : y + na_r, base);
    }
    // tags: of the cell's tokens (key_pixel, in LDS; the first is asked); there: whether it has any
    __device__ __forceinline__ CellMasks cell_masks(u32x4 rect, const uint32_t* tags, CellBase base, int half, bool there) const {
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)tags[0]);
        const int col = (int)((first & ((1u << (y_shift - 1)) - 1u)) >> 3) - base.col, line = (int)(first >> y_shift) - base.line;
        if (!there || (unsigned)col > 7u || (unsigned)line > 63u) return CellMasks{};
        typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
        typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
        // the column's bits in bytes 1 and 3 (the half's first pixel first), two of them moved up to the signs of both 16-bit halves
        const u16x2 t = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(rect[1], rect[0], 0x000c000cu | (uint32_t)col << 8 | (uint32_t)col << 24) >> ((kCellsZ ? 2 : 4) * half));
        auto mask = [&](int bit) __attribute__((always_inline)) {
            const u16x2 up = {(uint16_t)(7 - bit), (uint16_t)(6 - bit)};
            return __builtin_bit_cast(uint32_t, (i16x2)(__builtin_bit_cast(i16x2, (u16x2)(t << up)) >> (int16_t)15));
        };
        CellMasks m;
        m.x[0] = mask(0);
        m.x[1] = mask(kCellsZ ? 4 : 2);
        m.lines = (uint32_t)(((uint64_t)rect[3] << 32 | rect[2]) >> line);
        return m;
    }
    // Elements 4 c4 .. of the lane, kept or 0.
    __device__ __forceinline__ void keep_queries(const Bits& bits, const uint32_t* tags, int c4, int half, float (&pe)[4]) const {
        u32x4 t = {};
        if constexpr (kByTags) t = *(const u32x4*)&tags[8 * c4 + 4 * half];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kByTags) pe[i] = keep_or_zero(pixels_match(bits.plain, t[i]) ? ~0u : 0u, pe[i]);
            else pe[i] = keep_or_zero(keep(bits, 4 * c4 + i), pe[i]);
        }
    }
    // All-ones if element r is kept, else 0.
    __device__ __forceinline__ static uint32_t keep(const Bits& bits, int r) { return bit_mask(bits.plain, elem_pos(r)); }
    // Wave-uniform shortcut: no pair of the rectangle is masked (decided by index comparisons alone).
    template <uint32_t TERM>
    __device__ __forceinline__ bool term_full(int q_lo, int q_hi, int kv_lo, int kv_hi) const {
        if constexpr ((TERM & kTagged) != 0) return false;
        bool f = true;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) f = f && q_lo >= kv_hi;
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) f = f && q_hi - kv_lo <= window;
        if constexpr (TERM & FLEXATTN_M_PREFIX) f = f && kv_hi < prefix_len;
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) f = f && kv_hi < ctx;
        return f;
    }
    __device__ __forceinline__ bool full(int q_lo, int q_hi, int kv_lo, int kv_hi) const {
        bool f = term_full<T0>(q_lo, q_hi, kv_lo, kv_hi);
        if constexpr (T1 != 0) f = f || term_full<T1>(q_lo, q_hi, kv_lo, kv_hi);
        return f && kv_hi <= kv_last;
    }
    // The opposite: every pair of the rectangle is masked (decided by index comparisons alone).
    template <uint32_t TERM>
    __device__ __forceinline__ bool term_hidden(int q_lo, int q_hi, int kv_lo, int kv_hi) const {
        bool h = false;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) h = h || q_hi < kv_lo;
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) h = h || q_lo - kv_hi > window;
        if constexpr (TERM & FLEXATTN_M_PREFIX) h = h || kv_lo >= prefix_len;
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) h = h || kv_lo >= ctx;
        return h;
    }
    __device__ __forceinline__ bool hidden(int q_lo, int q_hi, int kv_lo, int kv_hi) const {
        bool h = term_hidden<T0>(q_lo, q_hi, kv_lo, kv_hi);
        if constexpr (T1 != 0) h = h && term_hidden<T1>(q_lo, q_hi, kv_lo, kv_hi);
        return h || kv_lo > kv_last;
    }
};

// ---------------------------------------------------------------------------------------
// score_mod in the base-2 domain.  apply(acc, q - kv) returns log2(e) * score_mod(acc * scale),
// so that exp(score') = exp2(apply(...)).  Order: ALiBi, relative bias, soft-cap.
// dscore(x) is d score_mod / d s given x = apply(...), used by the backward pass.
// ---------------------------------------------------------------------------------------
// Compiler-only fence on four values: everything that produces them is ordered before everything
// that uses them afterwards (no instruction is emitted).
__device__ __forceinline__ void pin4(float (&v)[4]) {
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}

// LDSTAB: the relative-bias row of the head has been copied to LDS (fill_table), pre-multiplied, and
// is looked up there: one 32-bit address per score instead of a 64-bit global address, which is
// what keeps the table variant of the MFMA kernels inside their register budget.
constexpr int kRelTableMax = 1024;         // flexattn_mod_params::rel_len is at most this

template <uint32_t SCORE, bool LDSTAB = false>
struct ScoreMod {
    static constexpr bool kAlibi = SCORE & FLEXATTN_SCORE_ALIBI;
    static constexpr bool kRel = SCORE & FLEXATTN_SCORE_REL_BIAS;
    static constexpr bool kCap = SCORE & FLEXATTN_SCORE_SOFTCAP;
    float k_acc;      // multiplies the raw dot product
    float k_bias;     // alibi_bias[h], pre-multiplied like k_acc
    float k_tab;      // factor applied to table entries
    float capl2;      // softcap * log2(e)
    const float* tab; // rel_bias row of head h
    int rel_max;
    float rel_first, rel_last;   // first and last table entry, times k_tab
    uint32_t tab_lds; // LDSTAB: LDS byte address of the pre-multiplied row

    __device__ __forceinline__ ScoreMod(const flexattn_mod_params& p, int h, float scale, uint32_t tab_lds_ = 0)
        : tab_lds(tab_lds_) {
        float mul = kCap ? (2.0f * kLog2e / p.softcap) : kLog2e;   // soft-cap needs exp(2 s / cap)
        k_acc = scale * mul;
        k_bias = kAlibi ? p.alibi_bias[h] * mul : 0.0f;
        k_tab = mul;
        tab = kRel ? p.rel_bias + (int64_t)h * p.rel_len : nullptr;
        rel_max = kRel ? p.rel_len - 1 : 0;
        capl2 = kCap ? p.softcap * kLog2e : 0.0f;
        rel_first = kRel ? __builtin_bit_cast(float, ldc((const int32_t*)tab)) * k_tab : 0.0f;
        rel_last = kRel ? __builtin_bit_cast(float, ldc((const int32_t*)tab + rel_max)) * k_tab : 0.0f;
    }

    // LDSTAB: every thread of the workgroup copies its share of the head's row (a barrier must follow
    // before the first lookup, and precede the next fill)
    __device__ __forceinline__ void fill_table(int tid, int nthreads) const {
        if constexpr (kRel && LDSTAB) {
            for (int i = tid; i <= rel_max; i += nthreads)
                *(__attribute__((address_space(3))) float*)(uintptr_t)(tab_lds + 4u * (uint32_t)i) = tab[i] * k_tab;
        }
    }

    // Relative bias of a whole block of scores whose q_idx - kv_idx spans [dq_min, dq_max]
    // (wave-uniform bounds): the index is clamped to the table, so a block that lies at or beyond the
    // last entry, or at or before the first, adds ONE value to all its scores -- almost every block
    // of a long sequence -- and only the blocks near the diagonal look the table up per element.
    // The functions below take UNI = true and that value (pre-multiplied like k_tab) for such blocks.
    __device__ __forceinline__ bool rel_uniform(int dq_min, int dq_max, float& value) const {
        value = 0.0f;
        if constexpr (!kRel) return true;
        if (dq_min >= rel_max) {
            value = rel_last;
            return true;
        }
        if (dq_max <= 0) {
            value = rel_first;
            return true;
        }
        return false;
    }

    // q_idx - kv_idx of one score element.  The kernels know it as dq0 + c with dq0 shared by the 16
    // elements a lane holds of a 32 x 32 block and c a compile-time constant, so the ALiBi term
    // bias * (dq0 + c) costs one addition of abase = alibi_base(dq0), computed once per block, and
    // one fma with a literal instead of a subtraction, a conversion and an fma per element.
    struct RelPos {
        int dq;
        float abase, c;
        __device__ __forceinline__ RelPos(int dq_) : dq(dq_), abase(0.0f), c((float)dq_) {}
        __device__ __forceinline__ RelPos(int dq0, float abase_, int c_) : dq(dq0 + c_), abase(abase_), c((float)c_) {}
    };
    __device__ __forceinline__ float alibi_base(int dq0) const { return kAlibi ? k_bias * (float)dq0 : 0.0f; }

    // Scaled score plus the additive biases, times the factor the following exp2 needs.
    template <bool UNI = false>
    __device__ __forceinline__ float pre(float acc, RelPos rp, float uni = 0.0f) const {
        float y;
        if constexpr (kRel && UNI) y = __builtin_fmaf(acc, k_acc, uni);
        else y = acc * k_acc;
        if constexpr (kAlibi) y = __builtin_fmaf(k_bias, rp.c, y + rp.abase);
        if constexpr (kRel && !UNI) {
            int r = rp.dq < 0 ? 0 : (rp.dq > rel_max ? rel_max : rp.dq);
            if constexpr (LDSTAB) y += *(const __attribute__((address_space(3))) float*)(uintptr_t)(tab_lds + 4u * (uint32_t)r);
            else y = __builtin_fmaf(tab[r], k_tab, y);
        }
        return y;
    }

    // Soft-cap only: r = 1 / (1 + exp(2 s / cap)), so that cap * tanh(s / cap) = cap * (1 - 2 r).
    template <bool UNI = false>
    __device__ __forceinline__ float cap_r(float acc, RelPos dq, float uni = 0.0f) const {
        return fast_rcp(1.0f + fast_exp2(pre<UNI>(acc, dq, uni)));
    }

    template <bool UNI = false>
    __device__ __forceinline__ float apply(float acc, RelPos dq, float uni = 0.0f) const {
        if constexpr (kCap) {
            return __builtin_fmaf(-2.0f * capl2, cap_r<UNI>(acc, dq, uni), capl2);
        } else {
            return pre<UNI>(acc, dq, uni);
        }
    }

    // apply() + shift with the addition folded into the multiply-adds that are there anyway (the
    // online softmax passes minus its running maximum: the score arrives ready for exp2).
    template <bool UNI = false>
    __device__ __forceinline__ float apply_shifted(float acc, RelPos rp, float uni, float shift) const {
        if constexpr (kCap) {
            return __builtin_fmaf(-2.0f * capl2, cap_r<UNI>(acc, rp, uni), capl2 + shift);
        } else if constexpr (kAlibi) {
            float y = __builtin_fmaf(acc, k_acc, __builtin_fmaf(k_bias, rp.c, rp.abase + ((kRel && UNI) ? uni + shift : shift)));
            if constexpr (kRel && !UNI) y += rel_entry(rp.dq);
            return y;
        } else {
            float y = __builtin_fmaf(acc, k_acc, (kRel && UNI) ? uni + shift : shift);
            if constexpr (kRel && !UNI) y += rel_entry(rp.dq);
            return y;
        }
    }
    // the relative-bias entry of q_idx - kv_idx = dq, times k_tab
    __device__ __forceinline__ float rel_entry(int dq) const {
        const int r = dq < 0 ? 0 : (dq > rel_max ? rel_max : dq);
        if constexpr (LDSTAB) return *(const __attribute__((address_space(3))) float*)(uintptr_t)(tab_lds + 4u * (uint32_t)r);
        else return tab[r] * k_tab;
    }

    // A soft-capped score never exceeds the cap, so softmax can use the cap itself as its
    // (fixed) maximum when 2^(-2 cap log2 e) is still far from fp32 underflow: no running max,
    // no rescaling, and p = exp2(-2 capl2 r) directly.
    __device__ __forceinline__ bool bounded() const { return kCap && 2.0f * capl2 <= 100.0f; }

    // The backward needs d score_mod / d s up to the constant factor grad_scale(): for the soft-cap,
    // 1 - tanh^2 = 4 r (1 - r) with r from cap_r(), so g = r - r^2 and the 4 is folded into the
    // final scaling of dQ / dK (see p_with_grad).
    static constexpr float grad_scale() { return kCap ? 4.0f : 1.0f; }

    // Backward: P = exp(score' - LSE) from the raw dot product, with the row's constant folded in.
    // row_const() maps LSE * log2(e) (+inf for a row without visible keys) to that constant.
    __device__ __forceinline__ float row_const(float lse2) const { return kCap ? capl2 - lse2 : -lse2; }
    // The same for four independent elements, written stage by stage (pin4 keeps the stages apart):
    // a wave that is alone on its SIMD loses several cycles on every vector instruction that
    // consumes the result of the one before it.
    template <bool UNI = false>
    __device__ __forceinline__ void p_with_grad4(const float (&acc)[4], const RelPos (&dq)[4], const float (&rc)[4],
                                                 float (&g)[4], float (&p)[4], float uni = 0.0f) const {
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)   // (without a soft-cap the row constant rides on the score_mod's multiply-adds)
            x[i] = kCap ? pre<UNI>(acc[i], dq[i], uni) : apply_shifted<UNI>(acc[i], dq[i], uni, rc[i]);
        pin4(x);
        if constexpr (kCap) {
            float r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = fast_exp2(x[i]);
            pin4(x);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = 1.0f + x[i];
            pin4(x);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = fast_rcp(x[i]);
            pin4(r);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __builtin_fmaf(-2.0f * capl2, r[i], rc[i]);
            pin4(x);
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] = __builtin_fmaf(-r[i], r[i], r[i]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] = 1.0f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = fast_exp2(x[i]);
        pin4(p);
    }
    template <bool UNI = false>
    __device__ __forceinline__ float p_with_grad(float acc, RelPos dq, float rc, float& g, float uni = 0.0f) const {
        if constexpr (kCap) {
            const float r = cap_r<UNI>(acc, dq, uni);
            g = __builtin_fmaf(-r, r, r);
            return fast_exp2(__builtin_fmaf(-2.0f * capl2, r, rc));
        } else {
            g = 1.0f;
            return fast_exp2(apply_shifted<UNI>(acc, dq, uni, rc));
        }
    }
};

// Waves per SIMD the backward kernels are compiled for: at D = 64 they fit 168 registers, so three workgroups
// share a CU (more latency hiding, more chances for one wave's MFMAs to run beside another's VALU work).
constexpr int bwd_waves_per_simd_of(int D) { return D == 64 ? 3 : 2; }
template <int D>
constexpr int bwd_waves_per_simd() {
    return bwd_waves_per_simd_of(D);
}

// ---------------------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------------------
void set_last_hip_error(int e);

#define FLEXATTN_HIP_TRY(expr)                          \
    do {                                                \
        hipError_t _e = (expr);                         \
        if (_e != hipSuccess) {                         \
            ::flexattn::set_last_hip_error((int)_e);    \
            return FLEXATTN_ERR_HIP;                    \
        }                                               \
    } while (0)

inline bool mask_id_valid(uint32_t m) {
    return (m & ~0x3f3fu) == 0 && !((m & 0xffu) == 0 && (m >> 8) != 0);
}
constexpr bool mask_uses(uint32_t m, uint32_t prim) { return ((m | (m >> 8)) & prim) != 0; }
// What the host can tell of the rows of a mask: how many keys the longest see, and whether others see far fewer (so that
// a launch of few rows ends with the longest alone); and how many they see at least, for rules that must not make short rows slower.
// A row of packed documents may see a tile or two whatever the batch's length, a row of a canvas about the pixels around 64.
struct LineShape {
    int64_t longest;
    bool uneven;
    int64_t sure;
    bool sure_uneven;
};
inline LineShape line_shape(uint32_t mask, const flexattn_mod_params& p, int q_len, int kv_len) {
    const uint32_t prims = mask | (mask >> 8);
    LineShape s = {kv_len, (prims & FLEXATTN_M_DOCUMENT) || ((prims & FLEXATTN_M_CAUSAL) && 2 * (int64_t)q_len > kv_len), kv_len, false};
    if (prims & FLEXATTN_M_SLIDING_WINDOW) {
        const int64_t reach = (int64_t)p.window + 1 + ((prims & FLEXATTN_M_PREFIX) ? p.prefix_len : 0);
        s.uneven = s.uneven && 2 * reach > kv_len;
        if (reach < s.longest) s.longest = reach;
    }
    s.sure = s.longest;
    s.sure_uneven = s.uneven && !(prims & FLEXATTN_M_DOCUMENT);
    if ((prims & FLEXATTN_M_DOCUMENT) && s.sure > 64) s.sure = 64;
    if (prims & FLEXATTN_M_NEIGHBORHOOD) {
        const int64_t around = (int64_t)(p.na_kernel + 16) * (p.na_kernel + 8);
        if (around < s.sure) s.sure = around;
    }
    return s;
}
template <uint32_t MASK>
LineShape line_shape(const flexattn_mod_params& p, int q_len, int kv_len) {
    return line_shape(MASK, p, q_len, kv_len);
}
// units_abreast's limit for the rows of a mask: of uneven length, or, at D = 64, windows of an eighth of the keys or more, whose first rows are shorter than the others (us, forward / dQ, one by one -> in turns,
// Bq = 128, 4 x 2048 x 16, window of 600 31 -> 29 / 48 -> 41, of 300 23.0 -> 23.1 / 37 -> 33, of 100 18.6 -> 19.0 / 27.2 -> 26.6, 8192 x 64, of 600 110 -> 111 / 162 -> 162, of 100 57 -> 59 / 94 -> 99, 2 x 3000 x 24, of 600
// 39 -> 34 / 49 -> 46, of 300, 64 x 128 28 -> 30 / 41 -> 44; at D = 128 window of 512, 4096 x 64: dQ 141 -> 146).
template <uint32_t MASK>
int rows_abreast(const LineShape& rows, int kv_len, int D) {
    const bool window = mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW) && !mask_uses(MASK, FLEXATTN_M_PREFIX);
    return rows.uneven || (D == 64 && window && 8 * rows.longest > kv_len) ? kRowsAbreast : 1;
}
inline bool score_id_valid(uint32_t s) { return (s & ~7u) == 0; }

// Pointers the selected mods will dereference must be present.
inline int check_mod_params(uint32_t mask_id, uint32_t score_id, const flexattn_mod_params* p) {
    if (!mask_id_valid(mask_id) || !score_id_valid(score_id)) return FLEXATTN_ERR_INVALID_ARG;
    bool need = mask_id != 0 || score_id != 0;
    if (need && !p) return FLEXATTN_ERR_INVALID_ARG;
    if (!p) return FLEXATTN_OK;
    if (mask_uses(mask_id, FLEXATTN_M_DOCUMENT) && !p->doc_ids) return FLEXATTN_ERR_INVALID_ARG;
    if (mask_uses(mask_id, FLEXATTN_M_CTX_LEN) && !p->ctx_lens) return FLEXATTN_ERR_INVALID_ARG;
    if ((score_id & FLEXATTN_SCORE_ALIBI) && !p->alibi_bias) return FLEXATTN_ERR_INVALID_ARG;
    if ((score_id & FLEXATTN_SCORE_REL_BIAS) && (!p->rel_bias || p->rel_len <= 0 || p->rel_len > 1024))
        return FLEXATTN_ERR_INVALID_ARG;
    if ((score_id & FLEXATTN_SCORE_SOFTCAP) && !(p->softcap > 0.0f)) return FLEXATTN_ERR_INVALID_ARG;
    if (mask_uses(mask_id, FLEXATTN_M_NEIGHBORHOOD)) {
        const int w = p->na_width, h = p->na_height, k = p->na_kernel, t = p->na_tile;
        if (w <= 0 || h <= 0 || (int64_t)w * h > (1 << 20)) return FLEXATTN_ERR_INVALID_ARG;
        if (k < 1 || !(k & 1) || k > w || k > h) return FLEXATTN_ERR_INVALID_ARG;
        if (p->na_layout == FLEXATTN_NA_TILED) {
            if (t <= 0 || (t & (t - 1)) || w % t || h % t) return FLEXATTN_ERR_INVALID_ARG;
        } else if (p->na_layout == FLEXATTN_NA_MORTON) {
            if (w != h || (w & (w - 1))) return FLEXATTN_ERR_INVALID_ARG;
        } else if (p->na_layout != FLEXATTN_NA_ROW_MAJOR) {
            return FLEXATTN_ERR_INVALID_ARG;
        }
    }
    return FLEXATTN_OK;
}

// The neighborhood mask is defined on a canvas of exactly q_len == kv_len tokens.
inline int check_canvas(uint32_t mask_id, const flexattn_mod_params* p, int q_len, int kv_len) {
    if (!mask_uses(mask_id, FLEXATTN_M_NEIGHBORHOOD)) return FLEXATTN_OK;
    const int64_t n = (int64_t)p->na_width * p->na_height;
    return (q_len == n && kv_len == n) ? FLEXATTN_OK : FLEXATTN_ERR_INVALID_ARG;
}

// Whether the kernels compare the pixels of a canvas token by token, and not as the rectangle that a lane's window is: where 32
// tokens are many short pieces, or (queries, in dK/dV) do not start at a known multiple of 32.
// (us, compared -> as a rectangle, 64 heads, K = 9 at 64 x 64, K = 7 and 3 for the narrow ones, forward / dK/dV / dQ: tiles of 2 x 2 68 -> 74 / 127 -> 139 /
// 87 -> 105, of 4 x 4 62 -> 61 / 110 -> 114 / 74 -> 77, row-major 4 x 1024 38 -> 40 / 75 -> 79 / 51 -> 55, 8 x 512 38 -> 39 / 75 -> 76 / 51 -> 53, but 16 x 256 42 ->
// 40 / 75 -> 73 / 56 -> 55, 31 x 132 50 -> 46 / 92 -> 88 / 66 -> 64.  Both in one kernel cost the rectangles' side up to 15 % of dQ: spills, and code that
// leaves the instruction cache.)
inline bool canvas_by_tags(const flexattn_mod_params& p, bool backward) {
    if (backward && p.q_offsets) return true;
    if (p.na_layout == FLEXATTN_NA_MORTON) return p.na_width < 8;
    if (p.na_layout == FLEXATTN_NA_TILED && p.na_tile > 1) return p.na_tile < 8;
    return p.na_width < 16;
}

// Whether 32 consecutive tokens, the first at a multiple of 32, are cells of 8 x 4 pixels whose rectangles fit the 64 columns and lines of
// PartialMask::rectangle.  Those of a cell's keys are the widest: 2 r + 8 columns, 3 r + 8 where they reach a border (and up to 7 before
// the first, a multiple of 8, but for the left border's), so r <= 16; on a canvas both of whose borders they reach, all of its 4 r + 8.
// (Positions that start elsewhere, other tiles, which cut 32 tokens otherwise, and wider windows are compared as before.)  Cells against
// that, us, B = 4, H = 16, D = 64, forward / dQ / dK/dV: 128 x 128, K = 13, tiles of 8 241 -> 232 / 296 -> 276 / 450 -> 450; 64 x 64, K = 27,
// tiles of 8 128 -> 115 / 158 -> 142 / 224 -> 219, K = 3 51.7 -> 51.4 / 64.1 -> 59.5 / 101.7 -> 100; K = 9, Morton 51.7 -> 49.6 / 65.6 -> 59.7 /
// 102.3 -> 99.4.  At D = 128 dQ 1.04x to 1.12x, dK/dV 1.00x to 1.03x; the forward compares as before.
inline bool canvas_in_cells(const flexattn_mod_params& p) {
    if (p.q_offsets || !(p.na_layout == FLEXATTN_NA_MORTON ? p.na_width >= 8 : p.na_layout == FLEXATTN_NA_TILED && p.na_tile == 8)) return false;
    const int r = p.na_kernel / 2, side = p.na_width < p.na_height ? p.na_width : p.na_height;
    return r <= (side > 4 * r + 8 ? 16 : 14);
}

// The (mask, score) pairs that forward/backward kernels are instantiated for: the paper's examples
// and benchmark variants, and three compositions of them (sliding window with a soft-cap; nested
// score_mods: ALiBi then soft-cap, relative bias then soft-cap under a document mask).  The functors
// compose freely -- another pair is one more line here (and in the launcher lists that
// FLEXATTN_VARIANT_INDICES drives), nothing else -- but for a canvas with another predicate, for which dK/dV would have to
// ask key_bits again (PartialMask::match_queries does not compile for it).
// X(mask_id, score_id)
#define FLEXATTN_FOR_EACH_VARIANT(X)                                                    \
    X(FLEXATTN_MASK_NONE, FLEXATTN_SCORE_IDENTITY)                                      \
    X(FLEXATTN_MASK_CAUSAL, FLEXATTN_SCORE_IDENTITY)                                    \
    X(FLEXATTN_MASK_CAUSAL, FLEXATTN_SCORE_ALIBI)                                       \
    X(FLEXATTN_MASK_CAUSAL, FLEXATTN_SCORE_SOFTCAP)                                     \
    X(FLEXATTN_MASK_SWA_CAUSAL, FLEXATTN_SCORE_IDENTITY)                                \
    X(FLEXATTN_MASK_PREFIX_LM, FLEXATTN_SCORE_IDENTITY)                                 \
    X(FLEXATTN_MASK_DOCUMENT_CAUSAL, FLEXATTN_SCORE_IDENTITY)                           \
    X(FLEXATTN_MASK_DOCUMENT_CAUSAL, FLEXATTN_SCORE_ALIBI)                              \
    X(FLEXATTN_MASK_SWA_CAUSAL_OR_PREFIX, FLEXATTN_SCORE_REL_BIAS)                      \
    X(FLEXATTN_MASK_NEIGHBORHOOD, FLEXATTN_SCORE_IDENTITY)                              \
    X(FLEXATTN_MASK_SWA_CAUSAL, FLEXATTN_SCORE_SOFTCAP)                                 \
    X(FLEXATTN_MASK_CAUSAL, (FLEXATTN_SCORE_ALIBI | FLEXATTN_SCORE_SOFTCAP))            \
    X(FLEXATTN_MASK_DOCUMENT_CAUSAL, (FLEXATTN_SCORE_REL_BIAS | FLEXATTN_SCORE_SOFTCAP))  \
    X((FLEXATTN_MASK_NEIGHBORHOOD | kCanvasByTags), FLEXATTN_SCORE_IDENTITY)            \
    X((FLEXATTN_MASK_NEIGHBORHOOD | kCanvasCells), FLEXATTN_SCORE_IDENTITY)             \
    X((FLEXATTN_MASK_NEIGHBORHOOD | kCanvasCellsZ), FLEXATTN_SCORE_IDENTITY)

// One entry per line of FLEXATTN_FOR_EACH_VARIANT: X(index)
#define FLEXATTN_VARIANT_INDICES(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)

}  // namespace flexattn
