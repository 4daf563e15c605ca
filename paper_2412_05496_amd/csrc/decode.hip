// Paged split-KV decode (decoding template of paper section 4.1; page-table indirection fused
// into the KV-block walk as in section 5.1) and the partial-softmax combine.
//
// The path is bound by reading K and V once from HBM; a small batch is bound by latency: launches, the
// chain arguments -> context length and page ids -> K / V rows, and the per-tile arithmetic that nothing else hides.  One
// WORKGROUP of four (or eight, waves_of) waves owns one (sequence, KV head, KV split); the waves take its 32-key tiles in turn
// and do not synchronise until the end: each walks the logical pages of its keys, looks every key's page
// up in the page table and pulls the K and V rows straight from the pool into its private, XOR-swizzled
// LDS tiles (global_load_lds_dwordx4: every wave instruction moves 1 KiB of whole 256-byte rows, so the
// page gather is fully coalesced; non-temporal, since a decode step reads every K / V row exactly once);
// the gather of its next tile is started as soon as the current tile's operand fragments sit in registers.
// S^T = K Q^T takes K rows from LDS as the A operand with the G <= 16 query heads of the group as the
// columns of the B operand (16x16x32 MFMAs), so K and V are read once per KV head, never once per query
// head; V^T comes out of the row-major V tile through the transposing LDS read.  The waves' (m, l, O) are
// merged in LDS into one result of the split; the combine kernel merges the splits of a (sequence, head)
// with log-sum-exp weights, and is not needed where a sequence has a single split.
// Measured on MI355X, 32 query / 8 KV heads, D = 128, 16-token pages (before: one wave per split, 32-column
// MFMAs, one wave per head walking the splits in the combine): one sequence of 8k tokens 33 -> 14 us (9.5 since the page
// ids do not wait for the context length, nor the combine's loads, and the arguments come in one go: 10.7 before), of 32k
// 69 -> 27, four of 8k 40 -> 26, sixteen of 8k 102 -> 86 (6.2 TB/s), 64 of 1k to 32k 783 -> 718 (at the rate of a plain
// streaming read).
#include <mutex>

#include "flex_common.h"
#include "lds_tiles.h"

// Workspace of flexattn_paged_decode_static(): lives in the library's device image, one copy per
// GPU, for callers that cannot allocate.  In host code this name is only a handle for
// hipGetSymbolAddress(); kernels receive the device address it returns, like any other workspace.
constexpr size_t kStaticScratchBytes = (size_t)40 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace flexattn {

constexpr int kDecWaves = 4;       // waves per workgroup, all on one split
constexpr int kDecTile = 32;       // keys per inner tile
constexpr int kDecSplitMax = 2048; // keys per split: a power of two in [kDecSplitMin, kDecSplitMax],
constexpr int kDecSplitMin = 128;

struct DecodeArgs {
    const bf16* Q;
    int64_t q_stride_seq;
    const bf16* K_pool;
    const bf16* V_pool;
    const int32_t* page_table;
    int64_t pt_stride;
    const int32_t* ctx_lens;
    int nseq, Hq, Hkv, G, page_size, page_shift, max_splits;
    int split_len;       // keys per split
    int max_ctx;         // max_pages * page_size: context lengths are clamped to what the page table can address
    int n_pool_pages;    // page ids are clamped to [0, n_pool_pages)
    int window;          // sliding window (q_idx - kv <= window), -1 if none
    float scale;
    flexattn_mod_params p;
    float* part_O;    // [nseq, Hq, max_splits, D]
    float* part_ml;   // [nseq, Hq, max_splits, 2]  (running max in base 2, sum)
    bf16* O;
    float* LSE;
};

// Reads the kernel's arguments in one go: each of their cache lines is a round trip to memory, which the compiler puts
// where the first of its values is used.
__device__ __forceinline__ void want_arguments(const DecodeArgs& a) {
    asm volatile("" :: "s"(a.Q), "s"(a.q_stride_seq), "s"(a.K_pool), "s"(a.V_pool), "s"(a.page_table), "s"(a.pt_stride), "s"(a.ctx_lens),
                 "s"(a.nseq), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.page_size), "s"(a.page_shift), "s"(a.max_splits), "s"(a.split_len),
                 "s"(a.max_ctx), "s"(a.n_pool_pages), "s"(a.window), "s"(a.scale), "s"(a.part_O), "s"(a.part_ml), "s"(a.O), "s"(a.LSE));
}

// 2 N consecutive elements of O.  O needs no more than the alignment of its elements (ANY); it is written in one store
// where it is aligned for it.
template <bool ANY, int N>
__device__ __forceinline__ void store_o(const DecodeArgs& a, int64_t at, const uint32_t (&v)[N]) {
    typedef uint32_t vec __attribute__((ext_vector_type(N)));
    bf16* p = a.O + at;
    if (!ANY || ((uintptr_t)a.O & 15) == 0) {
        vec x;
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = v[i];
        *(vec*)p = x;
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            ((uint16_t*)p)[2 * i] = (uint16_t)v[i];
            ((uint16_t*)p)[2 * i + 1] = (uint16_t)(v[i] >> 16);
        }
    }
}

// reductions over the four lanes that hold the same query column (lanes l, l ^ 16, l ^ 32, l ^ 48)
__device__ __forceinline__ float column_max(float v) {
    const LanePair p = lane_pair<true>(v);
    return max_halves(raw_max(p.a, p.b));
}
__device__ __forceinline__ float column_sum(float v) {
    const LanePair p = lane_pair<true>(v);
    const LanePair q = lane_pair<false>(p.a + p.b);
    return q.a + q.b;
}

__device__ __forceinline__ float wave_max(float v) {
    // lanes l ^ 1, l ^ 2, then (with those already equal) the mirror images within 8 and 16 lanes
    auto moved = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = raw_max(v, moved(v, std::integral_constant<int, 0xb1>{}));      // quad_perm 1 0 3 2
    v = raw_max(v, moved(v, std::integral_constant<int, 0x4e>{}));      // quad_perm 2 3 0 1
    v = raw_max(v, moved(v, std::integral_constant<int, 0x141>{}));     // row_half_mirror
    v = raw_max(v, moved(v, std::integral_constant<int, 0x140>{}));     // row_mirror
    return column_max(v);
}

// Where a running maximum starts.  Not at -inf, which would turn a row into NaN whose scores are all -inf in some
// tile, wave or split (keys that a bias masks; a wave sees every fourth tile only).
constexpr float kNoScore = -3.4028234663852886e38f;

// D[16x16] += A[16x32] * B[32x16]: lane l supplies A[row = l % 16][k-slots of group l / 16] and
// B[k-slots of group l / 16][col = l % 16]; register i of lane l holds D[row = 4 * (l / 16) + i][col = l % 16].
// The G <= 16 query heads of a KV head are the columns: half the multiplications, softmax
// instructions and accumulators of a 32-column tile whose upper columns no head would use.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// M0 RULE: this kernel fills LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the
// compiler's back.  Keep every register array in it indexed by compile-time constants (no movrel /
// s_set_gpr_idx code, which would also use M0) and add no other LDS-DMA or M0-based construct.
template <int D, uint32_t SCORE, bool ANY_O, int W>
__device__ __forceinline__ void decode_split(const DecodeArgs& a, int tid, int unit, int split) {
    constexpr int DC = D / 8;                  // 16-byte chunks per row
    constexpr int RPI = 64 / DC;               // rows per wave instruction
    constexpr int NI = kDecTile / RPI;         // instructions per tile and tensor
    constexpr int TILE = kDecTile * D;         // elements
    constexpr int NKC = D / 32, NDB = D / 16;  // 32-dim slices of the score product, 16-dim blocks of O
    constexpr int OROW = D + 4;                // floats per query row of a wave's O in LDS (padded: 16 rows, no conflicts)
    __shared__ __attribute__((aligned(1024))) bf16 smem[W * 2 * TILE];   // per wave: K tile, V tile
    __shared__ float s_ml[W][2][16];   // per wave: running max, sum of the 16 query columns
    static_assert(16 * OROW * 4 <= 2 * TILE * 2, "a wave's O must fit its own K and V tiles");

    if constexpr (!ANY_O) want_arguments(a);            // (the general kernel, which loops, has no registers for them all)
    const int lane = tid & 63, grp = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = unit / a.Hkv, hkv = unit % a.Hkv;
    const int ctx_len = ldc(a.ctx_lens + b);
    __builtin_amdgcn_sched_barrier(0);                  // (asked for before everything else)
    const int32_t* pt = a.page_table + (int64_t)b * a.pt_stride;
    const int page_mask = a.page_size - 1;
    const int64_t slab = (int64_t)a.page_size * D;      // elements per (page, head)
    // Page ids of the rows this lane fetches for one tile (NI wave instructions, RPI rows each), of rows past the
    // context as well: they do not wait for its length.
    auto lookup = [&](int tok0, int (&pg)[NI]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int tok = min(tok0 + i * RPI + lane / DC, a.max_ctx - 1);
            pg[i] = min(max(pt[tok >> a.page_shift], 0), a.n_pool_pages - 1);
        }
    };
    // The page ids of the tile a wave starts with are asked for beside the context length: one round trip to memory
    // instead of two.
    const int tok_begin = split * a.split_len, tok_guess = tok_begin + wave * kDecTile;
    int pg_next[NI];
    lookup(tok_guess, pg_next);
    const bool g_ok = l16 < a.G;                        // query head of the group held by this lane: l16
    const int hq = hkv * a.G + (g_ok ? l16 : 0);
    u32x4 q_raw[NKC];                                   // column l16, dims 32 kc + 8 grp ..
    {
        const bf16* qp = a.Q + (int64_t)b * a.q_stride_seq + (int64_t)hq * D + grp * 8;
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) q_raw[kc] = *(const u32x4*)(qp + kc * 32);
    }
    asm volatile("" ::: "memory");                      // (or the compiler sinks these loads below the test of the length)
    // A context length beyond what the page table addresses (or a negative one) is clamped, and so is
    // every page id below: wrong device-side tables give wrong rows, never an access outside the
    // table, the pools or the workspace.
    const int ctx = min(max(ctx_len, 0), a.max_ctx);
    // The query sits at q_idx = ctx - 1 (the offset of the decode step), so "causal" is kv < ctx and a
    // sliding window adds the lower bound kv >= q_idx - window.
    const int kv_lo = a.window >= 0 ? max(ctx - 1 - a.window, 0) : 0;
    if (tok_begin >= ctx || tok_begin + a.split_len <= kv_lo) {         // (uniform over the workgroup)
        if (ctx == 0 && split == 0) {
            for (int i = tid; i < a.G * D / 8; i += W * 64)
                store_o<ANY_O, 4>(a, ((int64_t)b * a.Hq + hkv * a.G) * D + i * 8, {0u, 0u, 0u, 0u});
            if (a.LSE && tid < a.G) a.LSE[(int64_t)b * a.Hq + hkv * a.G + tid] = -INFINITY;
        }
        return;
    }
    const int tok_end = min(ctx, tok_begin + a.split_len);
    // the waves take the 32-key tiles of the split in turn, from the first tile that holds a visible key
    const int tok_first = max(tok_begin, kv_lo & ~(kDecTile - 1)) + wave * kDecTile;
    constexpr int kStep = W * kDecTile;
    bf16* k_tile = smem + wave * 2 * TILE;
    bf16* v_tile = k_tile + TILE;

    // Gather of the 32 K rows and 32 V rows of a tile through the page table, straight into LDS.  The
    // LDS-DMA loads are inline assembly so that the compiler does not make later LDS reads wait for
    // them (see lds_tiles.h); completion is awaited with wait_vmem() at the top of the next iteration.
    // Rows past the context re-read the tile's first key, which exists: a masked V row must be a real one.
    auto gather = [&](int tok0, const int (&pg)[NI]) __attribute__((always_inline)) {
        const int pg_first = __builtin_amdgcn_readfirstlane(pg[0]);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = i * RPI + lane / DC;
            const bool there = tok0 + row < ctx;
            const int tok = there ? tok0 + row : tok0, page = there ? pg[i] : pg_first;
            const int64_t off = ((int64_t)page * a.Hkv + hkv) * slab + (int64_t)(tok & page_mask) * D +
                                (((lane % DC) ^ swz<D>(row)) * 8);
            dma_global_nt(lds_addr(k_tile + i * 512), a.K_pool + off);
            dma_global_nt(lds_addr(v_tile + i * 512), a.V_pool + off);
        }
    };
    if (tok_first < tok_end) {
        if (tok_first != tok_guess) lookup(tok_first, pg_next);     // (a window begins inside the split)
        gather(tok_first, pg_next);
        if (tok_first + kStep < tok_end) lookup(tok_first + kStep, pg_next);
    }

    bf16x8 qf[NKC];
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) qf[kc] = __builtin_bit_cast(bf16x8, g_ok ? q_raw[kc] : u32x4{0, 0, 0, 0});
    const ScoreMod<SCORE> smod(a.p, hq, a.scale);
    const int q_idx = ctx - 1;

    // LDS byte addresses of the operand reads for the first 16 keys (rows r + 16 have the swizzle of r).
    // K: row l16, 16-byte chunk 4 kc + grp.  V^T: transposing reads; group grp covers rows 4 grp .. +3 and
    // 16 + 4 grp .. +3 -- the keys whose scores the lanes of the group hold.
    uint32_t k_off[NKC], v_off[NDB];
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) k_off[kc] = lds_addr(k_tile) + 2u * (uint32_t)tile_off<D>(l16, 4 * kc + grp);
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
        const int row = 4 * grp + (l16 >> 2), col = 16 * db + 4 * (l16 & 3);
        v_off[db] = lds_addr(v_tile) + 2u * (uint32_t)(tile_off<D>(row, col >> 3) + (col & 7));
    }

    f32x4 oacc[NDB];                                    // O^T: dims 16 db + 4 grp + i of query l16
#pragma unroll
    for (int db = 0; db < NDB; ++db) oacc[db] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float m_run = kNoScore, l_run = 0.0f;

    for (int tok0 = tok_first; tok0 < tok_end; tok0 += kStep) {
        // ---- tile tok0 has landed; take every operand fragment out of LDS, then start the gather of
        // the next tile into the same (wave-private) buffers so that it runs beside this tile's compute
        wait_vmem();
        bf16x8 kfr[2][NKC], vfr[NDB];
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                kfr[kb][kc] = *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)(k_off[kc] + kb * 16 * D * 2);
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            const u32x2 lo = lds_read_tr4(v_off[db]), hi = lds_read_tr4(v_off[db] + 16 * D * 2);
            vfr[db] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
        }
        if (tok0 + kStep < tok_end) {
            __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0): the fragments are in registers
            gather(tok0 + kStep, pg_next);
            if (tok0 + 2 * kStep < tok_end) lookup(tok0 + 2 * kStep, pg_next);
        }

        // ---- S^T = K Q^T for the two 16-key blocks
        f32x4 sacc[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) sacc[kb] = mfma16(kfr[kb][kc], qf[kc], sacc[kb]);

        // ---- score_mod, mask kv_lo <= kv < ctx_len (only the first and the last tile can hold masked
        // keys), softmax
        const bool ragged = tok0 + kDecTile > tok_end || tok0 < kv_lo;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = smod.apply(sacc[e >> 2][e & 3], q_idx - (tok0 + 16 * (e >> 2) + 4 * grp + (e & 3)));
        if (ragged) {
            asm volatile("" ::: "memory");              // keep this a branch, not eight tests on every tile
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int kv = tok0 + 16 * (e >> 2) + 4 * grp + (e & 3);
                x[e] = kv >= tok_end || kv < kv_lo ? -INFINITY : x[e];
            }
        }
        float mx = x[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = raw_max(mx, x[e]);
        mx = column_max(mx);
        const float m_new = fmaxf(m_run, mx);
        const float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        float psum = 0.0f;
        u32x4 pk;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const float p0 = fast_exp2(x[2 * jj] - m_new), p1 = fast_exp2(x[2 * jj + 1] - m_new);
            psum += p0 + p1;
            pk[jj] = pack_bf16(p0, p1);
        }
        const bf16x8 pf = __builtin_bit_cast(bf16x8, pk);
        l_run = l_run * alpha + psum;
        if (__any(alpha != 1.0f)) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) oacc[db][i] *= alpha;
        }

        // ---- O^T += V^T P^T
#pragma unroll
        for (int db = 0; db < NDB; ++db) oacc[db] = mfma16(vfr[db], pf, oacc[db]);
    }

    // ---- the waves' (m, l, O) become one result of the split.  Every wave leaves its part in its own
    // tiles (all of whose reads and loads are done); a wave without a tile contributes weight 0.
    const float l_tot = column_sum(l_run);
    float* o_wave = (float*)k_tile;
    if (g_ok) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) *(f32x4*)(o_wave + l16 * OROW + 16 * db + 4 * grp) = oacc[db];
        if (grp == 0) {
            s_ml[wave][0][l16] = m_run;
            s_ml[wave][1][l16] = l_tot;
        }
    }
    __syncthreads();
    // The only non-empty split of a sequence writes the final O and LSE; the combine kernel leaves such
    // sequences alone.
    const bool only = (ctx - 1) / a.split_len == kv_lo / a.split_len;
    for (int it = tid; it < a.G * (D / 4); it += W * 64) {
        const int g = it / (D / 4), d = (it % (D / 4)) * 4;
        float m = s_ml[0][0][g];
#pragma unroll
        for (int w = 1; w < W; ++w) m = fmaxf(m, s_ml[w][0][g]);
        float L = 0.0f;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float wgt = fast_exp2(s_ml[w][0][g] - m);
            L += wgt * s_ml[w][1][g];
            o += wgt * *(const f32x4*)((const float*)(smem + w * 2 * TILE) + g * OROW + d);
        }
        const int64_t head = (int64_t)b * a.Hq + hkv * a.G + g;
        if (only) {
            const float inv = L > 0.0f ? 1.0f / L : 0.0f;
            store_o<ANY_O, 2>(a, head * D + d, {pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv)});
            if (d == 0 && a.LSE) a.LSE[head] = (m + fast_log2(L)) * kLn2;
        } else {
            const int64_t item = head * a.max_splits + split;
            *(f32x4*)(a.part_O + item * D + d) = o;
            if (d == 0) *(float2*)(a.part_ml + item * 2) = make_float2(m, L);
        }
    }
}

// One workgroup per (sequence, KV head) and split.  GENERAL: per (sequence, KV head) and every gridDim.y-th split, and O
// at any element address (a kernel of its own, of four waves, because either costs a small call one to ten percent).
template <int D, uint32_t SCORE, bool GENERAL, int W>
__global__ __launch_bounds__(W * 64, (D == 64 ? 4 : 2)) void decode_split_kernel(const DecodeArgs a) {
    if constexpr (!GENERAL) {
        decode_split<D, SCORE, false, W>(a, threadIdx.x, blockIdx.x, blockIdx.y);
    } else {
        for (int split = blockIdx.y; split < a.max_splits; split += gridDim.y) {
            int tid = threadIdx.x, unit = blockIdx.x;
            asm volatile("" : "+v"(tid), "+s"(unit));       // (or all that depends on them is worked out ahead of the first split's end)
            decode_split<D, SCORE, true, W>(a, tid, unit, split);
            if ((split + (int)gridDim.y) * (int64_t)a.split_len >= ldc(a.ctx_lens + unit / a.Hkv)) break;
            __syncthreads();                                // the merge has read LDS
        }
    }
}

// One workgroup per (sequence, query head): O = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^(m_s - max m).
// What bounds it is latency: a launch, and one round trip to memory.  Everything the first 64 splits left is asked
// for at once, without a window before the context length says how many there are (the workspace has room for every
// split, and what a split did not write gets no weight), and the rows of the splits are read side by side by 256 threads.
template <int D, bool ANY_O>
__global__ __launch_bounds__(kDecWaves * 64) void decode_combine_kernel(const DecodeArgs a) {
    constexpr int LPR = D / 4, ROWS = kDecWaves * 64 / LPR, PRE = 64 / ROWS;   // lanes per row, rows side by side
    __shared__ float s_o[ROWS][D + 4];
    __shared__ float s_l[ROWS];
    want_arguments(a);
    const int tid = threadIdx.x, lane = tid & 63, r0 = tid / LPR, d = (tid % LPR) * 4;
    const int b = blockIdx.x / a.Hq, hq = blockIdx.x % a.Hq;
    const int ctx_len = ldc(a.ctx_lens + b);
    __builtin_amdgcn_sched_barrier(0);
    const int64_t head = (int64_t)b * a.Hq + hq, base = head * a.max_splits;
    f32x4 pre[PRE];
    float2 pre_ml[PRE];
    float m_pre;
    auto ask = [&](int from) __attribute__((always_inline)) {
        const int last = a.max_splits - 1;
        m_pre = a.part_ml[(base + min(from + lane, last)) * 2];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            if (from + i * ROWS > last) break;                                      // (the same for all)
            const int64_t item = base + min(from + r0 + i * ROWS, last);
            pre[i] = *(const f32x4*)(a.part_O + item * D + d);
            pre_ml[i] = *(const float2*)(a.part_ml + item * 2);
        }
    };
    if (a.window < 0) ask(0);
    asm volatile("" ::: "memory");                                                  // (or these loads sink below the test of the length)
    const int ctx = min(max(ctx_len, 0), a.max_ctx);                                // as in the split kernel
    const int ns = (ctx + a.split_len - 1) / a.split_len;                           // <= max_splits
    const int s0 = a.window >= 0 ? max(ctx - 1 - a.window, 0) / a.split_len : 0;    // splits below the window are empty
    if (ns - s0 <= 1) return;                                                       // written by the split kernel
    if (a.window >= 0) ask(s0);
    float m = s0 + lane < ns ? m_pre : -INFINITY;
    for (int s = s0 + 64 + lane; s < ns; s += 64) m = fmaxf(m, a.part_ml[(base + s) * 2]);
    m = wave_max(m);
    float L = 0.0f;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    auto add = [&](const f32x4& row, float2 ml) {
        const float wgt = fast_exp2(ml.x - m);
        L += wgt * ml.y;
        acc += wgt * row;
    };
#pragma unroll
    for (int i = 0; i < PRE; ++i)
        if (s0 + r0 + i * ROWS < ns) add(pre[i], pre_ml[i]);
#pragma unroll 4
    for (int s = s0 + r0 + PRE * ROWS; s < ns; s += ROWS)
        add(*(const f32x4*)(a.part_O + (base + s) * D + d), *(const float2*)(a.part_ml + (base + s) * 2));
    *(f32x4*)&s_o[r0][d] = acc;
    if (d == 0) s_l[r0] = L;
    __syncthreads();
    if (tid < D / 2) {
        float o0 = 0.0f, o1 = 0.0f, lt = 0.0f;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            o0 += s_o[r][2 * tid];
            o1 += s_o[r][2 * tid + 1];
            lt += s_l[r];
        }
        const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
        store_o<ANY_O, 1>(a, head * D + 2 * tid, {pack_bf16(o0 * inv, o1 * inv)});
        if (tid == 0 && a.LSE) a.LSE[head] = (m + fast_log2(lt)) * kLn2;
    }
}

// Keys per split: the largest power of two in [kDecSplitMin, longest] that still cuts the longest context
// the page table addresses (the host cannot see the context lengths) into `want` pieces over all
// (sequence, KV head) units.
static int cut(const flexattn_decode_dims* d, long long want, int longest) {
    const long long per_piece = (long long)d->max_pages * d->page_size * d->nseq * d->Hkv / want;
    int len = kDecSplitMin;
    while (len < longest && 2 * len <= per_piece) len *= 2;
    return len;
}
// A workgroup works on one (sequence, KV head, split).  512 workgroups are two per CU, all that run at
// once: a small batch is cut until it offers them (measured, D = 128, 8 KV heads, us at 256 / 512 / 1024 /
// 2048 keys per split: one sequence of 32k tokens 29.3 / 27.1 / 29.2 / 41.1, four of 8k 27.9 / 26.4 / 28.8 /
// 41.0, one of 128k 102 / 92 / 88 / 86).  A large batch takes the longest splits, which pay a workgroup's
// start and its partial result least often (64 sequences of 1k to 32k: 908 / 797 / 753 / 719, and 715
// at 4096, where a batch whose contexts stay far below the table's reach would no longer fill the chip).  At D = 64 four
// workgroups fit a CU, but the same aim is the better one where contexts come near the table's reach (us at 512 / 1024
// workgroups, 8 KV heads: one of 32k 13.6 / 14.6, 64 of 1k 20.5 / 25.3, 16 of 4k 23.5 / 23.9; 16 of 2k in a table of 4k, 4 KV
// heads 10.7 / 9.0).
//
// A table that reaches no further than kDecOneSplit keys is not cut where few workgroups would run: the combine kernel,
// and a launch that waits for another, cost more than a wave's second tile.  (us, cut -> one split, 4 KV heads and 1 or 32
// sequences, a context of 250: D = 64 6.2 -> 3.7, 6.4 -> 4.0, D = 128 6.8 -> 4.8, 7.2 -> 5.3; of 500, D = 64 6.1 -> 4.6, 6.9 -> 5.4, D = 128, 8 / 128 /
// 256 units 6.7 -> 6.2, 9.0 -> 8.4, 14.3 -> 11.1; not with 4 units, whose rows few CUs must pull: 6.7 -> 8.6.)
constexpr int kDecOneSplit = 512;
static int split_len_of(const flexattn_decode_dims* d) {
    const long long reach = (long long)d->max_pages * d->page_size, units = (long long)d->nseq * d->Hkv;
    const int len = cut(d, 512, kDecSplitMax);
    if (len >= reach || reach > kDecOneSplit) return len;
    if (d->D == 128 && (units > 256 || (reach > 256 && units < 8))) return len;
    return reach > 256 ? 512 : 256;
}
// Waves per workgroup.  Eight hide each other's waits better where all workgroups run at once with two tiles or more to a
// wave of four: D = 64 (512 workgroups fill LDS), and single splits at D = 128 (256 do; us, four waves -> eight: 16 sequences of
// 100 to 4096 tokens, 4 KV heads, D = 64 11.6 -> 9.9; 32 of 500, 8 KV heads, D = 128 14.4 -> 11.1; cut contexts at D = 128 the other way:
// one of 7600 9.7 -> 12.3).
static int waves_of(const flexattn_decode_dims* d, int split_len, int max_splits) {
    const long long groups = (long long)d->nseq * d->Hkv * max_splits;
    return split_len >= 256 && (d->D == 64 ? groups <= 512 : max_splits == 1 && groups <= 256) ? 8 : 4;
}

static int splits(const flexattn_decode_dims* d, int len) {
    return (int)(((long long)d->max_pages * d->page_size + len - 1) / len);
}
// Room in the workspace: for the splits of 128 to 1024 keys of 1024 pieces, never fewer than are made.
static int max_splits_of(const flexattn_decode_dims* d) { return splits(d, cut(d, 1024, 1024)); }

template <int D>
static int launch_decode(const DecodeArgs& a, uint32_t score_id, int waves, hipStream_t st) {
    // The host sees how far the page table reaches, not how long the contexts are: a workgroup beyond their end
    // returns at once, but holds its LDS until then.  More than kMaxGroups (32 rounds of the chip) are not launched; a
    // workgroup then takes several splits, if the context has them (us without -> with, a table of 1M tokens: 64
    // sequences of 512 tokens, 8 KV heads, D = 64 / 128: 95.9 / 143.8 -> 17.6 / 37.5).
    constexpr int kMaxGroups = 16384;
    const int units = a.nseq * a.Hkv, room = (kMaxGroups + units - 1) / units;
    const bool aligned = ((uintptr_t)a.O & 15) == 0, general = a.max_splits > room || !aligned;
    const dim3 grid((unsigned)units, (unsigned)(a.max_splits < room ? a.max_splits : room));
    switch (score_id) {
#define CASE(S)                                                                                           \
    case S:                                                                                               \
        if (general) hipLaunchKernelGGL((decode_split_kernel<D, S, true, 4>), grid, dim3(256), 0, st, a);  \
        else if (waves == 8) hipLaunchKernelGGL((decode_split_kernel<D, S, false, 8>), grid, dim3(512), 0, st, a);  \
        else hipLaunchKernelGGL((decode_split_kernel<D, S, false, 4>), grid, dim3(256), 0, st, a);      \
        break;
        CASE(FLEXATTN_SCORE_IDENTITY)
        CASE(FLEXATTN_SCORE_ALIBI)
        CASE(FLEXATTN_SCORE_SOFTCAP)
        CASE(FLEXATTN_SCORE_REL_BIAS)
#undef CASE
        default: return FLEXATTN_ERR_UNSUPPORTED;
    }
    const dim3 heads((unsigned)(a.nseq * a.Hq));
    if (a.max_splits > 1 && aligned) hipLaunchKernelGGL((decode_combine_kernel<D, false>), heads, dim3(kDecWaves * 64), 0, st, a);
    else if (a.max_splits > 1) hipLaunchKernelGGL((decode_combine_kernel<D, true>), heads, dim3(kDecWaves * 64), 0, st, a);
    return FLEXATTN_OK;
}

}  // namespace flexattn

using namespace flexattn;

static int check_decode_dims(const flexattn_decode_dims* d) {
    if (!d) return FLEXATTN_ERR_INVALID_ARG;
    if (d->nseq <= 0 || d->Hq <= 0 || d->Hkv <= 0 || d->max_pages <= 0 || d->n_pool_pages <= 0)
        return FLEXATTN_ERR_INVALID_ARG;
    if (d->Hq % d->Hkv != 0) return FLEXATTN_ERR_INVALID_ARG;
    if (d->D != 64 && d->D != 128) return FLEXATTN_ERR_UNSUPPORTED;
    if (d->Hq / d->Hkv > 16) return FLEXATTN_ERR_UNSUPPORTED;
    if (d->page_size < 16 || d->page_size > 1024 || (d->page_size & (d->page_size - 1)))
        return FLEXATTN_ERR_UNSUPPORTED;
    if ((long long)d->max_pages * d->page_size > (1ll << 30)) return FLEXATTN_ERR_UNSUPPORTED;
    return FLEXATTN_OK;
}

extern "C" size_t flexattn_paged_decode_workspace_bytes(const flexattn_decode_dims* d) {
    if (check_decode_dims(d) != FLEXATTN_OK) return 0;
    const size_t items = (size_t)d->nseq * d->Hq * max_splits_of(d);
    return items * ((size_t)d->D + 2) * sizeof(float);
}

// Device address of `scratch` on the current device, looked up once per device.
static int static_scratch(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    FLEXATTN_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return FLEXATTN_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        FLEXATTN_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return FLEXATTN_ERR_HIP;
        addr[dev] = p;
    }
    *out = addr[dev];
    return FLEXATTN_OK;
}

extern "C" size_t flexattn_paged_decode_static_capacity(void) { return kStaticScratchBytes; }

extern "C" int flexattn_paged_decode_static(const flexattn_decode_dims* d, const void* Q, int64_t stride_q_seq,
                                            const void* K_pool, const void* V_pool, const int32_t* page_table,
                                            int64_t pt_stride, const int32_t* ctx_lens, uint32_t score_id,
                                            uint32_t mask_id, const flexattn_mod_params* params, float scale, void* O,
                                            float* LSE, void* stream) {
    int rc = check_decode_dims(d);
    if (rc != FLEXATTN_OK) return rc;
    // Every partial that counts in the combine kernel was written by the split kernel of the same call, so
    // nothing in the array has to start at zero.
    if (flexattn_paged_decode_workspace_bytes(d) > kStaticScratchBytes) return FLEXATTN_ERR_WORKSPACE;
    void* ws = nullptr;
    if ((rc = static_scratch(&ws)) != FLEXATTN_OK) return rc;
    return flexattn_paged_decode(d, Q, stride_q_seq, K_pool, V_pool, page_table, pt_stride, ctx_lens, score_id,
                                 mask_id, params, scale, O, LSE, ws, kStaticScratchBytes, stream);
}

extern "C" int flexattn_paged_decode(const flexattn_decode_dims* d, const void* Q, int64_t stride_q_seq,
                                     const void* K_pool, const void* V_pool, const int32_t* page_table,
                                     int64_t pt_stride, const int32_t* ctx_lens, uint32_t score_id, uint32_t mask_id,
                                     const flexattn_mod_params* params, float scale, void* O, float* LSE, void* ws,
                                     size_t ws_bytes, void* stream) {
    int rc = check_decode_dims(d);
    if (rc != FLEXATTN_OK) return rc;
    if (!Q || !K_pool || !V_pool || !page_table || !ctx_lens || !O || !ws) return FLEXATTN_ERR_INVALID_ARG;
    if (pt_stride < d->max_pages || stride_q_seq < (int64_t)d->Hq * d->D || (stride_q_seq % 8) != 0)
        return FLEXATTN_ERR_INVALID_ARG;
    if (((uintptr_t)Q & 15) || ((uintptr_t)K_pool & 15) || ((uintptr_t)V_pool & 15) || ((uintptr_t)ws & 15))
        return FLEXATTN_ERR_INVALID_ARG;
    if (!(scale > 0.0f)) return FLEXATTN_ERR_INVALID_ARG;
    const uint32_t kCtxWindow = FLEXATTN_M_CTX_LEN | FLEXATTN_M_SLIDING_WINDOW;   // one AND-term
    if (mask_id != FLEXATTN_MASK_CTX_LEN && mask_id != kCtxWindow) return FLEXATTN_ERR_UNSUPPORTED;
    flexattn_mod_params p = {};
    if (params) p = *params;
    p.ctx_lens = ctx_lens;
    if ((rc = check_mod_params(mask_id, score_id, &p)) != FLEXATTN_OK) return rc;
    if (ws_bytes < flexattn_paged_decode_workspace_bytes(d)) return FLEXATTN_ERR_WORKSPACE;

    DecodeArgs a = {};
    a.Q = (const bf16*)Q; a.q_stride_seq = stride_q_seq;
    a.K_pool = (const bf16*)K_pool; a.V_pool = (const bf16*)V_pool;
    a.page_table = page_table; a.pt_stride = pt_stride; a.ctx_lens = ctx_lens;
    a.nseq = d->nseq; a.Hq = d->Hq; a.Hkv = d->Hkv; a.G = d->Hq / d->Hkv;
    a.page_size = d->page_size;
    a.page_shift = __builtin_ctz((unsigned)d->page_size);
    a.split_len = split_len_of(d);
    a.max_splits = splits(d, a.split_len);
    a.max_ctx = d->max_pages * d->page_size;
    a.n_pool_pages = d->n_pool_pages;
    a.window = mask_id == kCtxWindow ? p.window : -1;
    a.scale = scale; a.p = p;
    const size_t items = (size_t)d->nseq * d->Hq * a.max_splits;
    a.part_O = (float*)ws;
    a.part_ml = (float*)ws + items * d->D;
    a.O = (bf16*)O; a.LSE = LSE;
    const int waves = waves_of(d, a.split_len, a.max_splits);
    rc = d->D == 128 ? launch_decode<128>(a, score_id, waves, (hipStream_t)stream)
                     : launch_decode<64>(a, score_id, waves, (hipStream_t)stream);
    if (rc != FLEXATTN_OK) return rc;
    FLEXATTN_HIP_TRY(hipGetLastError());
    return FLEXATTN_OK;
}
