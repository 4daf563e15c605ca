// The backward with dS kept in memory (an alternative to recomputing S and dP in a dQ kernel).
//
// The dK/dV kernel computes dS for every block it visits anyway; with ds_store set it also writes it
// out, and dQ = scale * dS K (section 4.1's backward, written out at the top of bwd_kernel.h) becomes
// one block-sparse GEMM over what was written: 1 GEMM and no softmax arithmetic instead of 3 GEMMs
// and all of it -- the backward executes 5 GEMMs, its algorithmic count, instead of 7.  The price is
// HBM: 2 bytes per unmasked score written once and read once, and a workspace of that size -- which
// this GPU has (288 GB; 4.4 GB for 64 heads of dense-causal S = 8192).  Still no floating-point
// atomics: every dQ row is summed by one wave in the order of its BlockMask row.
//
//   bwd_slots_scan_kernel / bwd_slots_fill_kernel   number the non-empty blocks (see ds_chunk in
//                      bwd_kernel.h) and lay the numbers out as a [planes, NR, NC] grid, so that the
//                      row-walking kernel finds the block the column-walking kernel wrote;
//   bwd_dq_stored_kernel   one workgroup per row of blocks of one (b, hq): K and dS tiles stream
//                      through LDS, dQ^T += K^T dS^T with both operands from transposing LDS
//                      reads.  Bound by the HBM read of dS.
#pragma once

#include "bwd_kernel.h"

namespace flexattn {

// Exclusive prefix sum of the merged column-list lengths over all `lines` = planes * NC columns of
// blocks; colbase[lines] = total.  One workgroup.
__global__ __launch_bounds__(1024) void bwd_slots_scan_kernel(const int32_t* __restrict__ q_num,
                                                              const int32_t* __restrict__ full_q_num, int lines, int NR,
                                                              int32_t* __restrict__ colbase) {
    __shared__ int s_sum[1024];
    const int tid = threadIdx.x;
    const int per = (lines + 1023) / 1024;
    const int lo = min(tid * per, lines), hi = min(lo + per, lines);
    auto count = [&](int l) { return min(max(full_q_num[l], 0), NR) + min(max(q_num[l], 0), NR); };
    int sum = 0;
    for (int l = lo; l < hi; ++l) sum += count(l);
    s_sum[tid] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {      // inclusive scan of the per-thread sums
        const int v = tid >= off ? s_sum[tid - off] : 0;
        __syncthreads();
        s_sum[tid] += v;
        __syncthreads();
    }
    int base = s_sum[tid] - sum;
    for (int l = lo; l < hi; ++l) {
        colbase[l] = base;
        base += count(l);
    }
    if (tid == 1023) colbase[lines] = s_sum[1023];
}

// grid[plane, r, c] = colbase[plane * NC + c] + j for the j-th entry r of the merged list of column c.
// One workgroup per column of blocks.
__global__ __launch_bounds__(256) void bwd_slots_fill_kernel(const int32_t* __restrict__ q_num,
                                                             const int32_t* __restrict__ q_idx,
                                                             const int32_t* __restrict__ full_q_num,
                                                             const int32_t* __restrict__ full_q_idx, int NR, int NC,
                                                             const int32_t* __restrict__ colbase,
                                                             int32_t* __restrict__ grid) {
    const int l = blockIdx.x, plane = l / NC, c = l - plane * NC;
    const int n_full = min(max(full_q_num[l], 0), NR), n_part = min(max(q_num[l], 0), NR);
    const int base = colbase[l];
    for (int j = threadIdx.x; j < n_full + n_part; j += 256) {
        const int r = j < n_full ? full_q_idx[(int64_t)l * NR + j] : q_idx[(int64_t)l * NR + j - n_full];
        if (r >= 0 && r < NR) grid[((int64_t)plane * NR + r) * NC + c] = base + j;
    }
}

// Transposing reads of a wave's own slice of a dS tile: 64 keys x 32 query columns, row-major and
// unpadded in LDS (a transposing read of 64 lanes covers 8 rows x 64 bytes = 512 contiguous bytes:
// no bank conflicts without any swizzle).  Fragment: column lane % 32, k-slots = rows
// r0 + 4 h + {0..3} and r0 + 8 + 4 h + {0..3}, like TrReader.
struct SliceTrReader {
    uint32_t off;
    __device__ __forceinline__ SliceTrReader(int lane, uint32_t base) {
        const int j = lane & 15, grp = lane >> 4;
        const int row = 4 * (grp >> 1) + (j >> 2), col = 16 * (grp & 1) + 4 * (j & 3);
        off = base + 2u * (uint32_t)(row * 32 + col);
    }
    __device__ __forceinline__ bf16x8 read(uint32_t slot_bytes, int r0) const {
        const u32x2 lo = lds_read_tr4(slot_bytes + off + 2u * r0 * 32);
        const u32x2 hi = lds_read_tr4(slot_bytes + off + 2u * (r0 + 8) * 32);
        u32x4 f = {lo[0], lo[1], hi[0], hi[1]};
        return __builtin_bit_cast(bf16x8, f);
    }
};

// M0 RULE: this kernel fills LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the
// compiler's back.  Keep every register array in it indexed by compile-time constants (no movrel /
// s_set_gpr_idx code, which would also use M0) and add no other LDS-DMA or M0-based construct.
//
// Pipeline.  K tiles are shared by the workgroup: double buffered, one barrier per tile.  A wave
// needs only ITS 32 query columns of a dS tile -- 4 KiB that the dK/dV kernel wrote contiguously --
// so every wave keeps a private ring of two slices and no barrier guards it.  Per tile t a wave
// issues K(t+1) and then dS(t+2); the vector-memory counter retires in issue order, so
// "all but the last four" at the top of a tile means K(t) and dS(t) have landed while dS(t+1) is
// still under way: the HBM read of dS runs two tiles ahead of its use, the L2 read of K one.
//
// CANVAS (neighborhood masks): the blocks of 32 keys that the mask hides from a wave's 32 rows are neither
// loaded (an empty descriptor fills the slice with zeros) nor multiplied; the dK/dV kernel may not have written
// them.  (8 x 8 tiles, K = 13, D = 64, 64 heads of 128 x 128 pixels: 336 -> 330 us, Morton order, K = 21: 710 ->
// 559, where K tiles weigh less against dS.)
//
// HEADS: a workgroup takes the same row of blocks of HEADS query heads that share a KV head and a BlockMask plane, NW waves each:
// the K tiles, which come from L2 but cost as many loads as dS, serve all of them (relative bias, S =
// 32768, 2 x 32 / 8 heads: 4680 -> 4080 us, 5 TB/s of dS).
// ROWS: the same with ROWS neighbouring rows of blocks of one head, whose lists are merged column by column; a tile that one of the
// rows does not list is left out by its waves (a zero times a K that is not finite would be NaN).
template <int D, int NW, bool CANVAS, int HEADS = 1, int ROWS = 1>
__global__ __launch_bounds__(NW * 64 * HEADS * ROWS, 2) void bwd_dq_stored_kernel(const BwdArgs a, const float qscale) {
    constexpr int Bq = NW * 32, THREADS = NW * 64 * HEADS * ROWS;
    static_assert(ROWS == 1 || (ROWS == 2 && HEADS == 1 && !CANVAS), "one thing at a time");
    constexpr int TILE_K = 64 * D, TILE_S = 64 * Bq, SLICE = 64 * 32;   // bf16 elements
    constexpr int kList = 512;
    static_assert(ROWS == 1 || THREADS == kList, "a thread per column");
    __shared__ __attribute__((aligned(1024))) bf16 smem[2 * TILE_K + HEADS * ROWS * NW * 2 * SLICE];   // K(even), K(odd); per wave dS(even), dS(odd)
    __shared__ int s_kv0[kList + 2];                                 // first key of a tile, -1: nothing to add
    __shared__ int s_chunk[kList + 2];                               // where its dS starts (ds_chunk without the rep)
    __shared__ int s_slot[ROWS > 1 ? ROWS : 1][ROWS > 1 ? kList : 1], s_listed[ROWS > 1 ? ROWS : 1][ROWS > 1 ? kList : 1], s_count[16];   // ROWS: see below
    __shared__ uint8_t s_hid[CANVAS ? kList + 2 : 1];                // CanvasBlocks::hidden_bits of the tile

    int unit, rem;
    const int groups = a.G / HEADS;
    const int row_sets = (a.NR + ROWS - 1) / ROWS;
    UnitSets abreast = a.abreast;
    if (a.turns_above && abreast.side && longest_row(a.kv_order, a.full_kv_num, a.kv_num, 0, a.NR, a.Bk / 64) <= a.turns_above) abreast = one_by_one(a.B * a.Hkv);
    if (!unit_of_workgroup(a.B * a.Hkv, groups * row_sets, abreast, unit, rem)) return;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), w = wave & (NW - 1);
    const int g = (rem % groups) * HEADS + (ROWS > 1 ? 0 : wave / NW);
    const int b = unit / a.Hkv, hkv = unit % a.Hkv, hq = hkv * a.G + g;
    const int64_t plane = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0);
    // (ROWS: the last rows first; the last set may have only one)
    const int first_row = (row_sets - 1 - rem / groups) * ROWS;
    const int row = ROWS > 1 ? first_row + wave / NW
                    : a.kv_order ? min(max(ldc(a.kv_order + plane * a.NR + rem / groups), 0), a.NR - 1) : a.NR - 1 - rem / groups;

    // the dS tile's columns are the block's query rows with bits 2 and 3 of the index exchanged (the
    // order in which the dK/dV kernel's registers hold them): lane l32 of wave w owns this row
    const int q_in_block = 32 * w + (l32 & 19) + ((l32 & 4) << 1) + ((l32 & 8) >> 1);
    const int q_row = row * Bq + q_in_block;
    const bool real_row = q_row < a.q_len;
    bf16* dq_ptr = a.dQ + b * a.dq_sb + hq * a.dq_sh + (int64_t)q_row * a.dq_ss;

    const int64_t line = plane * a.NR + (ROWS > 1 ? min(row, a.NR - 1) : row);
    const int n_full = ldc(a.full_kv_num + line), n_part = ldc(a.kv_num + line);
    const int sub_k = a.Bk / 64;
    const int T_all = (n_full + n_part) * sub_k;
    if (ROWS == 1 && T_all == 0) {
        if (real_row)
            for (int d0 = half * 8; d0 < D; d0 += 16) *(u32x4*)(dq_ptr + d0) = u32x4{0, 0, 0, 0};
        return;
    }
    const int32_t* full_idx = a.full_kv_idx + line * a.NC;
    const int32_t* part_idx = a.kv_idx + line * a.NC;
    const int32_t* grid_row = a.ds_grid + line * a.NC;
    // this wave's slice of the head's tiles: columns 32 w .. of a tile are the 4 KiB at w * 4096
    const bf16* ds_head = a.ds_store + ds_rep(a, b, hq) * a.ds_blocks * ((int64_t)a.Bk * Bq) + w * SLICE;

    const i32x4 k_rsrc = make_rsrc(a.K + b * a.k_sb + hkv * a.k_sh, (uint32_t)((a.kv_len - 1) * a.k_ss + D) * 2u);
    const int k_row_bytes = (int)a.k_ss * 2;
    const WaveTileLoader<D, NW * HEADS * ROWS> k_loader(a.k_ss, wave, lane);
    // slice position (key, 8 columns) <- where the dK/dV kernel put those 8 values: chunk c = columns
    // 16 c .., lane 32 h + key % 32 of the wave that had keys 32 kb ..
    int32_t s_voff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int pos = i * 64 + lane, key = pos >> 2, pc = pos & 3;
        s_voff[i] = (key >> 5) * 2048 + (pc >> 1) * 1024 + (32 * (pc & 1) + (key & 31)) * 16;
    }
    const uint32_t k_lds = lds_addr(smem), s_lds = k_lds + 2 * TILE_K * 2 + wave * (2 * SLICE * 2);
    const TrReader<D> tr_k(lane, k_lds);
    const SliceTrReader tr_s(lane, s_lds);

    f32x16 dq[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[db][r] = 0.0f;

    const int seg_end = ROWS > 1 ? a.NC : T_all;        // ROWS: a segment is kList columns
    for (int seg0 = 0; seg0 < seg_end; seg0 += kList) {
        int T = min(kList, T_all - seg0);
        if constexpr (ROWS > 1) {
            // every row enters the slots of its blocks under their columns; the columns that any row lists move together
#pragma unroll
            for (int r = 0; r < ROWS; ++r) s_slot[r][tid] = -1;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                if (first_row + r >= a.NR) break;
                const int64_t l = plane * a.NR + first_row + r;
                const int nf = ldc(a.full_kv_num + l), n = nf + ldc(a.kv_num + l);
                for (int i = tid; i < n; i += THREADS) {
                    const int c = min(max(i < nf ? a.full_kv_idx[l * a.NC + i] : a.kv_idx[l * a.NC + i - nf], 0), a.NC - 1);
                    if ((unsigned)(c - seg0) < (unsigned)kList)
                        s_slot[r][c - seg0] = (int)min(max((int64_t)a.ds_grid[l * a.NC + c], (int64_t)0), a.ds_blocks - 1);
                }
            }
            __syncthreads();
            bool listed = false;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) listed = listed || s_slot[r][tid] >= 0;
            const uint64_t mine = __ballot(listed);
            if (lane == 0) s_count[wave] = __popcll(mine);
            __syncthreads();
            int at = __popcll(mine & ((1ull << lane) - 1)), total = 0;
#pragma unroll
            for (int v = 0; v < THREADS / 64; ++v) {
                const int n = s_count[v];
                at += v < wave ? n : 0;
                total += n;
            }
            if (listed) {
                s_kv0[at] = (seg0 + tid) * a.Bk;
#pragma unroll
                for (int r = 0; r < ROWS; ++r) s_listed[r][at] = s_slot[r][tid];
            }
            T = __builtin_amdgcn_readfirstlane(total) * sub_k;
        }
        for (int i = ROWS > 1 ? T : tid; i < T; i += THREADS) {
            const int t = seg0 + i, pos = t / sub_k, st = t - pos * sub_k;
            const int c = min(max(pos < n_full ? full_idx[pos] : part_idx[pos - n_full], 0), a.NC - 1);
            const int kv0 = c * a.Bk + st * 64;
            const int slot = (int)min(max((int64_t)grid_row[c], (int64_t)0), a.ds_blocks - 1);
            s_kv0[i] = kv0 < a.kv_len ? kv0 : -1;      // the dK/dV kernel has no workgroup for keys past kv_len
            s_chunk[i] = slot * sub_k + st;
            if constexpr (CANVAS) {
                const CanvasBlocks cb(a.p);
                CanvasBlocks::Box qw[NW];
#pragma unroll
                for (int v = 0; v < NW; ++v) qw[v] = cb.windows(row * Bq + 32 * v);
                s_hid[i] = pos < n_full ? 0 : (uint8_t)cb.hidden_bits(qw, kv0);
            }
        }
        __syncthreads();

        if (ROWS > 1 && T == 0) continue;               // (the same for all; the next segment's first barrier is behind s_slot's writes)
        // first key of tile i, or -1; and where its dS starts, or -1
        auto kv0_of = [&](int i) __attribute__((always_inline)) {
            if constexpr (ROWS == 1) return __builtin_amdgcn_readfirstlane(s_kv0[i]);
            const int st = sub_k == 2 ? i & 1 : 0, kv0 = __builtin_amdgcn_readfirstlane(s_kv0[sub_k == 2 ? i >> 1 : i]) + 64 * st;
            return kv0 < a.kv_len ? kv0 : -1;
        };
        auto chunk_of = [&](int i) __attribute__((always_inline)) {
            if constexpr (ROWS == 1) return __builtin_amdgcn_readfirstlane(s_chunk[i]);
            const int slot = __builtin_amdgcn_readfirstlane(s_listed[wave / NW & (ROWS - 1)][sub_k == 2 ? i >> 1 : i]);
            return slot < 0 ? -1 : slot * sub_k + (sub_k == 2 ? i & 1 : 0);
        };
        auto load_k = [&](int i, auto buf_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            const int kv0 = max(kv0_of(i), 0);
            k_loader.start(k_rsrc, k_lds + BUF * (TILE_K * 2), kv0 * k_row_bytes);
        };
        auto hidden_of = [&](int i) -> uint32_t {
            if constexpr (!CANVAS) return 0u;
            else return ((uint32_t)__builtin_amdgcn_readfirstlane((int)s_hid[i]) >> (2 * w)) & 3u;
        };
        bool listed_of[2] = {true, true};       // ROWS: whether this wave's row lists the tile of the slot
        // a tile with nothing to add is loaded through an empty descriptor, which fills the slice with zeros
        auto load_s = [&](int i, auto buf_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            const int kv0 = kv0_of(i), chunk = chunk_of(i);
            const uint32_t hid = hidden_of(i);
            if constexpr (ROWS > 1) listed_of[BUF] = chunk >= 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {       // (j >> 1: which 32 keys)
                const bool there = kv0 >= 0 && (ROWS == 1 || chunk >= 0) && !(hid & (1u << (j >> 1)));
                const i32x4 rsrc = make_rsrc(ds_head + (int64_t)(ROWS == 1 ? chunk : max(chunk, 0)) * TILE_S, there ? (uint32_t)SLICE * 2u : 0u);
                dma_x1_nt(rsrc, s_lds + BUF * (SLICE * 2) + j * 1024, s_voff[j], 0);
            }
        };
        const std::integral_constant<int, 0> b0;
        const std::integral_constant<int, 1> b1;
        load_k(0, b0);
        load_s(0, b0);
        if (T > 1) load_s(1, b1);

        auto step = [&](int t, auto buf_tag) {
            constexpr int BUF = decltype(buf_tag)::value;
            constexpr std::integral_constant<int, BUF ^ 1> nxt{};
            // K(t) and dS(t) have landed; dS(t+1), if there is one, may still be under way
            if (t + 1 < T) wait_vmem_but<4>();
            else wait_vmem();
            __syncthreads();
            constexpr uint32_t kt = BUF * (TILE_K * 2), stl = BUF * (SLICE * 2);
            if (ROWS > 1 && !listed_of[BUF]) {          // (wave-uniform; the barriers and the other tiles' loads stay)
                if (t + 1 < T) load_k(t + 1, nxt);
                if (t + 2 < T) load_s(t + 2, buf_tag);
                return;
            }
            bf16x8 bfr[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) bfr[ks] = tr_s.read(stl, 16 * ks);
            // (the slot is refilled below: the reads above must have left LDS first)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[0]), "+v"(bfr[1]), "+v"(bfr[2]), "+v"(bfr[3]) :: "memory");
            const uint32_t hid = hidden_of(t);
            if (t + 1 < T) load_k(t + 1, nxt);
            if (t + 2 < T) load_s(t + 2, buf_tag);
            constexpr int NDB = D / 32, NM = 4 * NDB, PF = 4;       // [16-key slice][block db]
            if constexpr (CANVAS) {
                static_for<0, 2>([&](auto j_tag) {
                    constexpr int j = decltype(j_tag)::value;
                    if (!(hid & (1u << j))) {
#pragma unroll
                        for (int m = j * NM / 2; m < (j + 1) * NM / 2; ++m)
                            dq[m % NDB] = mfma32(tr_k.read(kt, 16 * (m / NDB), m % NDB), bfr[m / NDB], dq[m % NDB]);
                    }
                });
                return;
            }
            auto frag = [&](int m) { return tr_k.read(kt, 16 * (m / NDB), m % NDB); };
            bf16x8 fr[NM];
#pragma unroll
            for (int m = 0; m < PF; ++m) fr[m] = frag(m);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                if (m + PF < NM) fr[m + PF] = frag(m + PF);
                dq[m % NDB] = mfma32(fr[m], bfr[m / NDB], dq[m % NDB]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int t = 0;
        for (; t + 1 < T; t += 2) {
            step(t, b0);
            step(t + 1, b1);
        }
        if (t < T) step(t, b0);
        __syncthreads();        // everybody has read the last K tile and the lists
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

enum class StoredShare { kNone, kHeads, kRows };     // (stored_share; D = 128, Bq = 128)
template <bool CANVAS>
int launch_bwd_stored_dq(const BwdArgs& args, int D, float qscale, StoredShare share, bool uneven, bool documents, hipStream_t st) {
    BwdArgs a = args;
    const unsigned grid_q = unit_grid(a.B * a.Hkv, a.G * a.NR);
    a.abreast = units_abreast(a.B * a.Hkv, share == StoredShare::kNone ? a.G * a.NR : a.G * ((a.NR + 1) / 2), share != StoredShare::kNone ? 1 : bwd_waves_per_simd_of(D), uneven ? kRowsAbreast : 1);
    // Short documents one head after the other, as in abreast_if_long.  us of dQ, B x S x heads, one by one / in turns, documents of 16 to 100, 30 to 300, 100 to 1000 and 256 to 4096: D = 64,
    // 8192 x 64 61 / 64, 68 / 71, 125 / 124, 329 / 285, 4 x 4096 x 16 35.7 / 37.0, 39.5 / 40.3, 68 / 60, 203 / 161; D = 128, 8 x 2048 x 64 189 / 206, 207 / 234, 314 / 328, 604 / 582, 4 x 4096 x 16 50 / 51,
    // 53 / 58, 83 / 78, 228 / 198, 16 x 1024 x 32 91 / 94, 104 / 103, 154 / 138, 191 / 168.
    if (documents) a.turns_above = 8;
    if constexpr (!CANVAS) {
        if (share == StoredShare::kHeads) {         // (an even number of heads to a group, one plane for all)
            hipLaunchKernelGGL((bwd_dq_stored_kernel<128, 4, false, 2>), dim3(unit_grid(a.B * a.Hkv, a.G / 2 * a.NR)), dim3(512), 0, st, a, qscale);
            return FLEXATTN_OK;
        }
        if (share == StoredShare::kRows) {
            hipLaunchKernelGGL((bwd_dq_stored_kernel<128, 4, false, 1, 2>), dim3(unit_grid(a.B * a.Hkv, a.G * ((a.NR + 1) / 2))), dim3(512), 0, st, a, qscale);
            return FLEXATTN_OK;
        }
    }
    if (D == 128 && a.Bq == 128) hipLaunchKernelGGL((bwd_dq_stored_kernel<128, 4, CANVAS>), dim3(grid_q), dim3(256), 0, st, a, qscale);
    else if (D == 128) hipLaunchKernelGGL((bwd_dq_stored_kernel<128, 2, CANVAS>), dim3(grid_q), dim3(128), 0, st, a, qscale);
    else if (a.Bq == 128) hipLaunchKernelGGL((bwd_dq_stored_kernel<64, 4, CANVAS>), dim3(grid_q), dim3(256), 0, st, a, qscale);
    else hipLaunchKernelGGL((bwd_dq_stored_kernel<64, 2, CANVAS>), dim3(grid_q), dim3(128), 0, st, a, qscale);
    return FLEXATTN_OK;
}

}  // namespace flexattn
