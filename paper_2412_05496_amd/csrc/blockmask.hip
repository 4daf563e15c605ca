// BlockMask construction (paper section 4.2) and the paged BlockMask conversion (section 5.1).
//
// One workgroup makes the lists of one line: of a row of blocks, or of a column of blocks (both
// orientations in one launch; a column classifies its blocks again instead of waiting for the rows).  A
// thread classifies a block from the index ranges and, for documents and canvas pixels, from the range of
// ids or coordinates its tokens take: that settles the blocks that are hidden or visible as a whole.  The
// others are counted exactly by one wave each, a lane per query row: the keys that row sees are a 64-bit
// mask per term (an interval, and the keys whose document id equals the row's, by one ballot for each of the first
// ids, or whose pixels match), whose population is the count.  Pixels are all different, and ids in any order may be:
// those keys are compared one by one (a ballot for each, us -> this: 64 x 64 pixels, K = 41 102 -> 51, row-major 107 -> 51,
// 128 x 128, K = 101 268 -> 136; 64 ids at random, S = 4096 89 -> 57).
// What bounds it is latency, not arithmetic: two short kernels (us on packed documents, S = 16384, before the ids were read 16
// bytes at a time, the next block's asked for ahead, and the statistics summed without atomics: 38 -> 22; 16 x 4096 46 -> 26).  (A wave per block that evaluated
// mask_mod scalar by scalar, 8192 to a block, and then one wave per line to compact: 0.18 ms on packed
// documents of 16384 tokens, 0.11 ms for four causal chunks of 2048 queries on 16384 keys, 0.49 ms for
// 128 x 128 pixels.)
#include "flex_common.h"

namespace flexattn {

// What the tokens of one side of a block have in common.  Documents: ids in [a0, a1].  Canvas: keys with
// x in [a0, a1] and y in [b0, b1]; queries whose windows start at x0 in [a0, a1], y0 in [b0, b1].
struct TokenRange {
    int a0, a1, b0, b1;
};
constexpr TokenRange kNoTokens = {INT32_MAX, INT32_MIN, INT32_MAX, INT32_MIN};
constexpr TokenRange kAnyTokens = {INT32_MIN / 2, INT32_MAX / 2, INT32_MIN / 2, INT32_MAX / 2};

// The mask on whole blocks and, exactly, on the scalars of a block.
template <uint32_t MASK>
struct BlockEval {
    using Partial = PartialMask<MASK>;
    static constexpr uint32_t T0 = MASK & 0xffu, T1 = (MASK >> 8) & 0xffu;
    Partial mask;
    const int32_t* docs;
    int q_off, q_len, kv_len, Bq, Bk;
    __device__ __forceinline__ BlockEval(const flexattn_mod_params& p, int b, int q_len_, int kv_len_, int Bq_, int Bk_)
        : mask(p, b, kv_len_), docs(Partial::kDoc ? p.doc_ids + (int64_t)b * p.doc_stride_b : nullptr),
          q_off(q_offset_of(p, b)), q_len(q_len_), kv_len(kv_len_), Bq(Bq_), Bk(Bk_) {}

    // n tokens more of the key (query) side of a block
    __device__ __forceinline__ void take_keys(TokenRange& r, int kv, int n) const {
        if constexpr (Partial::kDoc) take_ids(r, docs + kv, n);
        if constexpr (Partial::kCanvas) {
            for (int t = 0; t < n; ++t) {
                int x, y;
                mask.canvas.pixel(kv + t, x, y);
                take(r.a0, r.a1, x);
                take(r.b0, r.b1, y);
            }
        }
    }
    __device__ __forceinline__ void take_queries(TokenRange& r, int q, int n) const {
        if constexpr (Partial::kDoc) take_ids(r, docs + q_off + q, n);
        if constexpr (Partial::kCanvas) {
            for (int t = 0; t < n; ++t) {
                int x, y;
                mask.window_corner(q_off + q + t, x, y);
                take(r.a0, r.a1, x);
                take(r.b0, r.b1, y);
            }
        }
    }
    // A thread reads the ids of its block 16 bytes at a time (at any element address), eight loads under way: a load per id
    // touches 64 cache lines a wave as well and is waited for four times as often.
    __device__ __forceinline__ static void take_ids(TokenRange& r, const int32_t* ids, int n) {
        typedef int32_t quad __attribute__((ext_vector_type(4), aligned(4)));
        int t = 0;
        for (; t + 32 <= n; t += 32) {
            quad v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = *(const quad*)(ids + t + 4 * i);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) take(r.a0, r.a1, v[i][e]);
        }
        for (; t < n; ++t) take(r.a0, r.a1, ids[t]);
    }
    __device__ __forceinline__ static void take(int& lo, int& hi, int v) {
        lo = min(lo, v);
        hi = max(hi, v);
    }
    // Rows and keys of block (i, j) that exist.
    __device__ __forceinline__ int rows_of(int i) const { return min(Bq, q_len - i * Bq); }
    __device__ __forceinline__ int keys_of(int j) const { return min(Bk, kv_len - j * Bk); }

    // 0: every pair of the rectangle is hidden, 2: none is, 1: undecided.  (kind() also: 3, see there.)
    template <uint32_t TERM>
    __device__ __forceinline__ int term_kind(int q_lo, int q_hi, int kv_lo, int kv_hi, const TokenRange& rq,
                                             const TokenRange& rk) const {
        bool e = false, f = true;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) e = e || q_hi < kv_lo, f = f && q_lo >= kv_hi;
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) e = e || q_lo - kv_hi > mask.window, f = f && q_hi - kv_lo <= mask.window;
        if constexpr (TERM & FLEXATTN_M_PREFIX) e = e || kv_lo >= mask.prefix_len, f = f && kv_hi < mask.prefix_len;
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) e = e || kv_lo >= mask.ctx, f = f && kv_hi < mask.ctx;
        if constexpr (TERM & FLEXATTN_M_DOCUMENT) {
            e = e || rq.a1 < rk.a0 || rk.a1 < rq.a0;
            f = f && rq.a0 == rq.a1 && rk.a0 == rk.a1 && rq.a0 == rk.a0;
        }
        if constexpr (TERM & FLEXATTN_M_NEIGHBORHOOD) {
            const int span = 2 * mask.na_r;
            e = e || rk.a1 < rq.a0 || rk.a0 > rq.a1 + span || rk.b1 < rq.b0 || rk.b0 > rq.b1 + span;
            f = f && rk.a0 >= rq.a1 && rk.a1 <= rq.a0 + span && rk.b0 >= rq.b1 && rk.b1 <= rq.b0 + span;
        }
        return e ? 0 : (f ? 2 : 1);
    }
    __device__ __forceinline__ int kind(int i, int j, const TokenRange& rq, const TokenRange& rk) const {
        const int q_lo = q_off + i * Bq, q_hi = q_lo + rows_of(i) - 1, kv_lo = j * Bk, kv_hi = kv_lo + keys_of(j) - 1;
        int k = term_kind<T0>(q_lo, q_hi, kv_lo, kv_hi, rq, rk);
        if constexpr (T1 != 0) {
            const int k1 = term_kind<T1>(q_lo, q_hi, kv_lo, kv_hi, rq, rk);
            k = k == 2 || k1 == 2 ? 2 : max(k, k1);
        }
        // what lies outside the score matrix counts as masked: a block that is cut short is never FULL, but 3 if nothing else is hidden
        return k == 2 && (rows_of(i) < Bq || keys_of(j) < Bk) ? 3 : k;
    }

    // bits of [lo, hi] among the keys kv0 .. kv0 + 63
    __device__ __forceinline__ static uint64_t span_bits(int lo, int hi, int kv0) {
        const int h = min(max(hi - kv0, -1), 63) + 1, l = min(max(lo - kv0, 0), 64);
        const uint64_t below_h = h == 0 ? 0ull : ~0ull >> (64 - h), below_l = l == 0 ? 0ull : ~0ull >> (64 - l);
        return below_h & ~below_l;
    }
    template <uint32_t TERM>
    __device__ __forceinline__ uint64_t term_bits(int q, int kv0, uint64_t match) const {
        int hi = kv_len - 1, lo = 0;
        if constexpr (TERM & FLEXATTN_M_CAUSAL) hi = min(hi, q);
        if constexpr (TERM & FLEXATTN_M_PREFIX) hi = min(hi, mask.prefix_len - 1);
        if constexpr (TERM & FLEXATTN_M_CTX_LEN) hi = min(hi, mask.ctx - 1);
        if constexpr (TERM & FLEXATTN_M_SLIDING_WINDOW) lo = max(__builtin_elementwise_sub_sat(q, mask.window), 0);
        return span_bits(lo, hi, kv0) & ((TERM & Partial::kTagged) ? match : ~0ull);
    }
    // The document ids of up to 128 rows and 128 keys of a block, two of each to a lane.  (Pixels are worked out where they are used.)
    struct Tags {
        uint32_t q[2], k[2];
    };
    __device__ __forceinline__ Tags tags(int i, int j, int r0, int k0, int lane) const {
        Tags t = {};
        if constexpr (Partial::kDoc) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                t.q[c] = (uint32_t)docs[q_off + i * Bq + min(r0 + 64 * c + lane, rows_of(i) - 1)];
                t.k[c] = (uint32_t)docs[j * Bk + min(k0 + 64 * c + lane, keys_of(j) - 1)];
            }
        }
        return t;
    }
    // Unmasked scalars of block (i, j) in the rows of this lane, by the whole wave.  first: its tags(i, j, 0, 0, lane);
    // all: whether every pair of a whole block is visible.
    static constexpr int kBallots = 6, kUnroll = Partial::kCanvas ? 1 : 4;      // (a canvas' keys are long unrolled code as it is)
    __device__ __forceinline__ int count(int i, int j, int lane, const Tags& first, bool& all) const {
        const int rows = rows_of(i), keys = keys_of(j);
        int sum = 0;
        bool seen = rows == Bq && keys == Bk;
        for (int r0 = 0; r0 < rows; r0 += 128) {
            for (int k0 = 0; k0 < keys; k0 += 128) {
                const Tags t = r0 == 0 && k0 == 0 ? first : tags(i, j, r0, k0, lane);
#pragma unroll kUnroll
                for (int c = 0; c < 4; ++c) {
                    const int rc = r0 + 64 * (c >> 1), kc = k0 + 64 * (c & 1);
                    if (rc >= rows || kc >= keys) continue;
                    const int q = q_off + i * Bq + min(rc + lane, rows - 1), kv0 = j * Bk + kc, n = min(64, keys - kc);
                    uint32_t q_tag = c & 2 ? t.q[1] : t.q[0], k_tag = c & 1 ? t.k[1] : t.k[0];
                    if constexpr (Partial::kCanvas) {
                        q_tag = mask.query_pixel(q);
                        k_tag = mask.key_pixel(min(kv0 + lane, kv_len - 1));
                    }
                    const uint64_t match = tag_bits(q_tag, k_tag, ~0ull >> (64 - n));
                    uint64_t bits = term_bits<T0>(q, kv0, match);
                    if constexpr (T1 != 0) bits |= term_bits<T1>(q, kv0, match);
                    const int mine = __popcll(bits & (~0ull >> (64 - n)));
                    sum += rc + lane < rows ? mine : 0;
                    seen = seen && mine == n;
                }
            }
        }
        all = __all(seen);
        return sum;
    }
    // the keys among `there` (a bit per lane) whose tag matches the lane's query
    __device__ __forceinline__ uint64_t tag_bits(uint32_t q_tag, uint32_t k_tag, uint64_t there) const {
        if constexpr (!Partial::kTags) return ~0ull;
        uint64_t match = 0;
        if constexpr (Partial::kDoc) {      // the first ids by one ballot each
            for (int i = 0; i < kBallots && there != 0; ++i) {
                const uint32_t tag = (uint32_t)__builtin_amdgcn_readlane((int)k_tag, __builtin_ctzll(there));
                const uint64_t same = __ballot(k_tag == tag);
                there &= ~same;
                match |= tag == q_tag ? same : 0ull;
            }
        }
        if (there != 0) {                   // key by key
            uint32_t part[2] = {0u, 0u};
#pragma unroll
            for (int at = 0; at < 64; ++at) {
                const uint32_t tag = (uint32_t)__builtin_amdgcn_readlane((int)k_tag, at);
                const bool same = Partial::kDoc ? tag == q_tag : mask.pixels_match(tag, q_tag);
                part[at >> 5] |= same ? 1u << (at & 31) : 0u;
            }
            match |= (uint64_t)part[1] << 32 | part[0];
        }
        return match;
    }
};

struct LineArgs {
    flexattn_mod_params p;
    int Bm, Hm, NR, NC, Bq, Bk, q_len, kv_len;
    int32_t *kv_num, *kv_idx, *full_kv_num, *full_kv_idx, *q_num, *q_idx, *full_q_num, *full_q_idx;
    unsigned long long* stats;          // nullable
    unsigned long long* row_scalars;    // unmasked scalars of every row of blocks (null: added to stats by atomics)
};

template <uint32_t MASK, int kLineThreads>
__global__ __launch_bounds__(kLineThreads) void build_lines_kernel(const LineArgs a) {
    using Eval = BlockEval<MASK>;
    constexpr int kLineWaves = kLineThreads / 64;
    constexpr bool kTags = Eval::Partial::kTags;
    __shared__ TokenRange s_fixed;                 // the tokens of the line itself
    __shared__ uint8_t s_kind[kLineThreads];
    __shared__ uint16_t s_todo[kLineThreads];
    __shared__ int s_ntodo, s_part[kLineWaves], s_full[kLineWaves];
    __shared__ unsigned long long s_scalars;       // unmasked scalars of the line's PARTIAL blocks
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long planes = (long long)a.Bm * a.Hm, row_lines = planes * a.NR, lines = row_lines + planes * a.NC;

    for (long long id = blockIdx.x; id < lines; id += gridDim.x) {
        const bool is_row = id < row_lines;
        const long long line = is_row ? id : id - row_lines;
        const int n_lines = is_row ? a.NR : a.NC, len = is_row ? a.NC : a.NR;
        const int self = (int)(line % n_lines);
        const int b = (int)(line / n_lines / a.Hm);
        const Eval ev(a.p, b, a.q_len, a.kv_len, a.Bq, a.Bk);
        int32_t* out_p = (is_row ? a.kv_idx : a.q_idx) + line * len;
        int32_t* out_f = (is_row ? a.full_kv_idx : a.full_q_idx) + line * len;

        if (tid == 0) s_scalars = 0;
        if constexpr (kTags) {
            if (tid == 0) s_fixed = kNoTokens;
            __syncthreads();
            TokenRange r = kNoTokens;
            if (is_row) for (int t = tid; t < ev.rows_of(self); t += kLineThreads) ev.take_queries(r, self * a.Bq + t, 1);
            else for (int t = tid; t < ev.keys_of(self); t += kLineThreads) ev.take_keys(r, self * a.Bk + t, 1);
            atomicMin(&s_fixed.a0, r.a0);
            atomicMax(&s_fixed.a1, r.a1);
            if constexpr (Eval::Partial::kCanvas) {
                atomicMin(&s_fixed.b0, r.b0);
                atomicMax(&s_fixed.b1, r.b1);
            }
        }
        int np = 0, nf = 0;
        for (int c0 = 0; c0 < len; c0 += kLineThreads) {
            if (tid == 0) s_ntodo = 0;
            __syncthreads();
            const int k = c0 + tid;
            int kind = 0;
            if (k < len) {
                const int i = is_row ? self : k, j = is_row ? k : self;
                kind = ev.kind(i, j, kAnyTokens, kAnyTokens);       // what the index comparisons alone decide
                if constexpr (kTags) {
                    if (kind == 1) {
                        TokenRange r = kNoTokens;
                        if (is_row) ev.take_keys(r, k * a.Bk, ev.keys_of(k));
                        else ev.take_queries(r, k * a.Bq, ev.rows_of(k));
                        kind = is_row ? ev.kind(i, j, s_fixed, r) : ev.kind(i, j, r, s_fixed);
                    }
                }
                if (kind == 1) s_todo[atomicAdd(&s_ntodo, 1)] = (uint16_t)tid;
                // (PARTIAL, with nothing to count: every block of a last row of blocks that is cut short.  us of the build, counted -> not: chunks of 202 on
                // 1051 to 6408 cached keys, 3 sequences 11.4 -> 5.6, of 223 on 1529 to 6538, 6 sequences 14.5 -> 6.2, no mask, S = 12653 22.8 -> 6.2)
                if (kind == 3) {
                    if (is_row && a.stats) atomicAdd(&s_scalars, (unsigned long long)ev.rows_of(i) * (unsigned)ev.keys_of(j));
                    kind = 1;
                }
            }
            s_kind[tid] = (uint8_t)kind;
            __syncthreads();
            const int n_todo = s_ntodo;
            // (the tags of the wave's next block are asked for before this one's are used)
            auto tags_of = [&](int t) __attribute__((always_inline)) {
                const int kk = __builtin_amdgcn_readfirstlane((int)s_todo[min(t, n_todo - 1)]) + c0;
                return is_row ? ev.tags(self, kk, 0, 0, lane) : ev.tags(kk, self, 0, 0, lane);
            };
            if (wave < n_todo) {
                unsigned long long scalars = 0;
                typename Eval::Tags next = tags_of(wave);
                for (int t = wave; t < n_todo; t += kLineWaves) {
                    const typename Eval::Tags now = next;
                    next = tags_of(t + kLineWaves);
                    const int kk = __builtin_amdgcn_readfirstlane((int)s_todo[t]);
                    bool full;
                    const int mine = is_row ? ev.count(self, c0 + kk, lane, now, full) : ev.count(c0 + kk, self, lane, now, full);
                    const bool any = __any(mine != 0);
                    if (lane == 0) s_kind[kk] = (uint8_t)(any ? (full ? 2 : 1) : 0);
                    scalars += full ? 0 : mine;
                }
                if (is_row && a.stats) {                // (only the rows' are reported)
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) scalars += __shfl_xor(scalars, off, 64);
                    if (lane == 0) atomicAdd(&s_scalars, scalars);
                }
            }
            __syncthreads();
            kind = s_kind[tid];
            const unsigned long long mp = __ballot(kind == 1), mf = __ballot(kind == 2);
            if (lane == 0) {
                s_part[wave] = __popcll(mp);
                s_full[wave] = __popcll(mf);
            }
            __syncthreads();
            int p0 = np, f0 = nf;
#pragma unroll
            for (int w = 0; w < kLineWaves; ++w) {
                p0 += w < wave ? s_part[w] : 0;
                f0 += w < wave ? s_full[w] : 0;
                np += s_part[w];
                nf += s_full[w];
            }
            const unsigned long long below = (1ull << lane) - 1;
            if (kind == 1) out_p[p0 + __popcll(mp & below)] = k;
            if (kind == 2) out_f[f0 + __popcll(mf & below)] = k;
        }
        for (int k = np + tid; k < len; k += kLineThreads) out_p[k] = 0;
        for (int k = nf + tid; k < len; k += kLineThreads) out_f[k] = 0;
        if (tid == 0) {
            (is_row ? a.kv_num : a.q_num)[line] = np;
            (is_row ? a.full_kv_num : a.full_q_num)[line] = nf;
            const unsigned long long scalars = s_scalars + (unsigned long long)nf * (unsigned)(a.Bq * a.Bk);
            if (is_row && a.row_scalars) {
                a.row_scalars[line] = scalars;
            } else if (is_row && a.stats) {
                if (np) atomicAdd(&a.stats[0], (unsigned long long)np);
                if (nf) atomicAdd(&a.stats[1], (unsigned long long)nf);
                if (scalars) atomicAdd(&a.stats[3], scalars);
                if (id == 0) atomicAdd(&a.stats[2], (unsigned long long)(row_lines * a.NC));
            }
        }
        __syncthreads();
    }
}

// Work order of both orientations: per plane, the lines sorted by descending num + full_num (ties by
// ascending index).  A line's place is the number of keys (kOrderCountMax - count, index) below its own,
// counted by one thread over a copy of all keys in LDS: no passes and no barriers in between, which is
// what a sort of a few hundred lines consists of otherwise (bitonic: 7.6 us for 256 lines).  More than
// kOrderMax lines are left in the fixed order: descending index for rows, ascending for columns.
//
// One workgroup beside them adds up the statistics of the rows.
__device__ __forceinline__ void sum_stats(const LineArgs& a) {
    __shared__ unsigned long long s_sum[4][3];
    const long long rows = (long long)a.Bm * a.Hm * a.NR;
    unsigned long long sum[3] = {0, 0, 0};
#pragma unroll 4
    for (long long r = threadIdx.x; r < rows; r += 256) {
        sum[0] += (unsigned)a.kv_num[r];
        sum[1] += (unsigned)a.full_kv_num[r];
        sum[2] += a.row_scalars[r];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum[i] += __shfl_xor(sum[i], off, 64);
        if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6][i] = sum[i];
    }
    __syncthreads();
    if (threadIdx.x < 3) a.stats[threadIdx.x < 2 ? threadIdx.x : 3] = s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x] + s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x];
    if (threadIdx.x == 3) a.stats[2] = (unsigned long long)(rows * a.NC);
}
constexpr int kOrderMax = 8192, kOrderIdxBits = 13, kOrderCountMax = (1 << 18) - 1;
__global__ __launch_bounds__(256) void order_lines_kernel(const LineArgs a, int32_t* __restrict__ kv_order,
                                                          int32_t* __restrict__ q_order) {
    __shared__ __attribute__((aligned(16))) uint32_t keys[kOrderMax];
    if (blockIdx.y == 2) {
        if (blockIdx.x == 0 && blockIdx.z == 0) sum_stats(a);
        return;
    }
    const bool rows = blockIdx.y == 0;
    int32_t* order = rows ? kv_order : q_order;
    const int n = rows ? a.NR : a.NC;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (!order || (int)(blockIdx.x * 256) >= n) return;
    for (int plane = blockIdx.z; plane < a.Bm * a.Hm; plane += gridDim.z) {
        const int64_t base = (int64_t)plane * n;
        if (n > kOrderMax) {
            if (i < n) order[base + i] = rows ? n - 1 - i : i;
            continue;
        }
        const int32_t* num = (rows ? a.kv_num : a.q_num) + base;
        const int32_t* full = (rows ? a.full_kv_num : a.full_q_num) + base;
        const int n4 = (n + 3) & ~3;
        for (int t = threadIdx.x; t < n4; t += 256)
            keys[t] = t < n ? ((uint32_t)(kOrderCountMax - min(num[t] + full[t], kOrderCountMax)) << kOrderIdxBits) | (uint32_t)t
                            : 0xffffffffu;
        __syncthreads();
        if (i < n) {
            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
            const uint32_t own = keys[i];
            int place = 0;
#pragma unroll 4
            for (int t = 0; t < n4; t += 4) {
                const u32x4_t v = *(const u32x4_t*)&keys[t];
                place += (v[0] < own) + (v[1] < own) + (v[2] < own) + (v[3] < own);
            }
            order[base + place] = i;
        }
        __syncthreads();
    }
}

__global__ void zero_stats_kernel(unsigned long long* stats) {
    if (threadIdx.x < 4) stats[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void paged_convert_kernel(
    const int32_t* __restrict__ num_blocks, const int32_t* __restrict__ indices, int Hm, int NR, int NC,
    const int32_t* __restrict__ page_table, long long pt_stride, int32_t* __restrict__ phys_indices,
    int32_t* __restrict__ phys2log, int n_pool_pages, long long total) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long long line = e / NC;
    const int k = (int)(e % NC);
    const long long b = line / ((long long)Hm * NR);
    int32_t out = 0;
    if (k < num_blocks[line]) {
        const int32_t logical = indices[e];
        out = page_table[b * pt_stride + logical];
        if (phys2log && out >= 0 && out < n_pool_pages) phys2log[out] = logical;
    }
    phys_indices[e] = out;
}

template <uint32_t MASK>
static void launch_lines(const LineArgs& a, hipStream_t st) {
    const long long lines = (long long)a.Bm * a.Hm * (a.NR + a.NC);
    const unsigned grid = (unsigned)(lines < (1 << 20) ? lines : (1 << 20));    // (the kernel strides over the rest)
    // Documents of a few long sequences: eight waves share the count of a line's undecided blocks (us of the build, 256 -> 512
    // threads: S = 16384, documents of 256 to 4096 27.5 -> 21.9, of 8000 39.8 -> 28.7, of 16 to 100 15.9 -> 18.5; S = 32768, 768 lines 34.2 -> 33.4;
    // 16 x 4096, 1536 lines 25.8 -> 40.8, whose waves no longer run all at once; 128 x 128 pixels 48 -> 53).
    if constexpr (PartialMask<MASK>::kDoc) {
        if (lines <= 512) {
            hipLaunchKernelGGL((build_lines_kernel<MASK, 512>), dim3(grid), dim3(512), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((build_lines_kernel<MASK, 256>), dim3(grid), dim3(256), 0, st, a);
}

}  // namespace flexattn

using namespace flexattn;

extern "C" int flexattn_blockmask_sizes(int32_t Bm, int32_t Hm, int32_t q_len, int32_t kv_len, int32_t Bq,
                                           int32_t Bk, flexattn_blockmask_counts* sizes) {
    if (!sizes || Bm <= 0 || Hm <= 0 || q_len <= 0 || kv_len <= 0 || Bq <= 0 || Bk <= 0)
        return FLEXATTN_ERR_INVALID_ARG;
    const int64_t NR = ((int64_t)q_len + Bq - 1) / Bq, NC = ((int64_t)kv_len + Bk - 1) / Bk;
    const int64_t planes = (int64_t)Bm * Hm;
    if (planes * NR * NC > (1ll << 31)) return FLEXATTN_ERR_UNSUPPORTED;
    sizes->NR = (int32_t)NR;
    sizes->NC = (int32_t)NC;
    sizes->kv_num_blocks = sizes->full_kv_num_blocks = planes * NR;
    sizes->kv_indices = sizes->full_kv_indices = planes * NR * NC;
    sizes->q_num_blocks = sizes->full_q_num_blocks = planes * NC;
    sizes->q_indices = sizes->full_q_indices = planes * NC * NR;
    sizes->kv_order = planes * NR;
    sizes->q_order = planes * NC;
    return FLEXATTN_OK;
}

extern "C" size_t flexattn_blockmask_workspace_bytes(int32_t Bm, int32_t Hm, int32_t q_len, int32_t kv_len,
                                                     int32_t Bq, int32_t Bk) {
    if (Bm <= 0 || Hm <= 0 || q_len <= 0 || kv_len <= 0 || Bq <= 0 || Bk <= 0) return 0;
    const size_t NR = ((size_t)q_len + Bq - 1) / Bq, NC = ((size_t)kv_len + Bk - 1) / Bk;
    return ((size_t)Bm * Hm * NR * NC + 255) & ~(size_t)255;
}

extern "C" int flexattn_blockmask_build(uint32_t mask_id, const flexattn_mod_params* params,
                                        const flexattn_blockmask* bm, int64_t* stats, void* ws, size_t ws_bytes,
                                        void* stream) {
    if (!bm || !ws) return FLEXATTN_ERR_INVALID_ARG;
    if (bm->Bm <= 0 || bm->Hm <= 0 || bm->q_len <= 0 || bm->kv_len <= 0 || bm->Bq <= 0 || bm->Bk <= 0)
        return FLEXATTN_ERR_INVALID_ARG;
    if (!bm->kv_num_blocks || !bm->kv_indices || !bm->full_kv_num_blocks || !bm->full_kv_indices ||
        !bm->q_num_blocks || !bm->q_indices || !bm->full_q_num_blocks || !bm->full_q_indices)
        return FLEXATTN_ERR_INVALID_ARG;
    int rc = check_mod_params(mask_id, 0, params);
    if (rc != FLEXATTN_OK) return rc;
    if ((rc = check_canvas(mask_id, params, bm->q_len, bm->kv_len)) != FLEXATTN_OK) return rc;
    const int NR = (bm->q_len + bm->Bq - 1) / bm->Bq, NC = (bm->kv_len + bm->Bk - 1) / bm->Bk;
    const long long nblocks = (long long)bm->Bm * bm->Hm * NR * NC;
    if (nblocks > (1ll << 31) || (long long)bm->Bq * bm->Bk > (1ll << 24)) return FLEXATTN_ERR_UNSUPPORTED;
    if (ws_bytes < flexattn_blockmask_workspace_bytes(bm->Bm, bm->Hm, bm->q_len, bm->kv_len, bm->Bq, bm->Bk))
        return FLEXATTN_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    LineArgs a = {};
    if (params) a.p = *params;
    a.Bm = bm->Bm; a.Hm = bm->Hm; a.NR = NR; a.NC = NC; a.Bq = bm->Bq; a.Bk = bm->Bk;
    a.q_len = bm->q_len; a.kv_len = bm->kv_len;
    a.kv_num = bm->kv_num_blocks; a.kv_idx = bm->kv_indices;
    a.full_kv_num = bm->full_kv_num_blocks; a.full_kv_idx = bm->full_kv_indices;
    a.q_num = bm->q_num_blocks; a.q_idx = bm->q_indices;
    a.full_q_num = bm->full_q_num_blocks; a.full_q_idx = bm->full_q_indices;
    a.stats = (unsigned long long*)stats;
    // The rows leave their scalars in the workspace, where a row has the eight blocks that make it large enough: atomics of
    // all rows on one cache line, which go one after the other, bounded the build of many (us, 16 sequences of 4096 38.7 -> 25.8, 64 of 1000
    // 37.3 -> 25.1, one of 16384 29.8 -> 27.5).
    if (a.stats && NC >= 8 && ((uintptr_t)ws & 7) == 0) a.row_scalars = (unsigned long long*)ws;
    else if (a.stats) hipLaunchKernelGGL(zero_stats_kernel, dim3(1), dim3(64), 0, st, a.stats);

    // The builder is instantiated for every mask the two-term encoding can express with
    // the primitives below; unknown combinations are rejected rather than approximated.
    switch (mask_id) {
#define CASE(M) case M: launch_lines<M>(a, st); break;
        CASE(FLEXATTN_MASK_NONE)
        CASE(FLEXATTN_MASK_CAUSAL)
        CASE(FLEXATTN_MASK_SLIDING_WINDOW)
        CASE(FLEXATTN_MASK_SWA_CAUSAL)
        CASE(FLEXATTN_MASK_DOCUMENT)
        CASE(FLEXATTN_MASK_DOCUMENT_CAUSAL)
        CASE(FLEXATTN_MASK_PREFIX_LM)
        CASE(FLEXATTN_MASK_SWA_CAUSAL_OR_PREFIX)
        CASE(FLEXATTN_MASK_CTX_LEN)
        CASE(FLEXATTN_MASK_NEIGHBORHOOD)
        CASE((FLEXATTN_M_CTX_LEN | FLEXATTN_M_CAUSAL))
        CASE((FLEXATTN_MASK_SWA_CAUSAL | FLEXATTN_M_DOCUMENT))
#undef CASE
        default: return FLEXATTN_ERR_UNSUPPORTED;
    }
    FLEXATTN_HIP_TRY(hipGetLastError());
    if (bm->kv_order || bm->q_order || a.row_scalars) {
        const int planes = bm->Bm * bm->Hm, longest = NR > NC ? NR : NC;
        hipLaunchKernelGGL(order_lines_kernel, dim3((unsigned)((longest + 255) / 256), a.row_scalars ? 3 : 2, (unsigned)(planes < 4096 ? planes : 4096)),
                           dim3(256), 0, st, a, bm->kv_order, bm->q_order);
        FLEXATTN_HIP_TRY(hipGetLastError());
    }
    return FLEXATTN_OK;
}

extern "C" int flexattn_paged_convert_blockmask(const int32_t* num_blocks, const int32_t* indices, int32_t Bm,
                                                int32_t Hm, int32_t NR, int32_t NC, const int32_t* page_table,
                                                int64_t pt_stride, int32_t* phys_indices, int32_t* phys2log,
                                                int32_t n_pool_pages, void* stream) {
    if (!num_blocks || !indices || !page_table || !phys_indices) return FLEXATTN_ERR_INVALID_ARG;
    if (Bm <= 0 || Hm <= 0 || NR <= 0 || NC <= 0 || pt_stride < NC || n_pool_pages <= 0)
        return FLEXATTN_ERR_INVALID_ARG;
    const long long total = (long long)Bm * Hm * NR * NC;
    hipLaunchKernelGGL(paged_convert_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, num_blocks, indices, Hm, NR, NC, page_table, (long long)pt_stride,
                       phys_indices, phys2log, n_pool_pages, total);
    FLEXATTN_HIP_TRY(hipGetLastError());
    return FLEXATTN_OK;
}
