// dQ and dK/dV for launches that leave the chip idle: the waves of a workgroup share 32 query rows (dQ) or 32 keys (dK/dV)
// and take the 32-wide units of the other index in turn, each through LDS of its own and without a barrier; their sums
// are added up at the end.  What ends a small launch is a wave's chain of units, which this makes as many times shorter as
// there are waves, on two to four times as many CUs.  The arithmetic is that of bwd_dq_kernel and bwd_dkdv_kernel
// (bwd_kernel.h), in the same precision.
#pragma once

#include "bwd_kernel.h"

namespace flexattn {

// Adds up what NW waves hold in QUADS register quads each: a wave leaves its quads in `mine` (QUADS KiB of LDS, 64 lanes x 16
// bytes a quad), and after the barrier takes every NW-th quad of all waves (`all`: the regions side by side).
template <int NW, int QUADS, typename F>
__device__ __forceinline__ void add_quads(f32x4* all, int w, int lane, const f32x4 (&quads)[QUADS], F&& out) {
    f32x4* mine = all + w * (QUADS * 64) + lane;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) mine[q * 64] = quads[q];
    __syncthreads();
    for (int q = w; q < QUADS; q += NW) {
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < NW; ++v) o += all[v * (QUADS * 64) + q * 64 + lane];
        out(q, o);
    }
}

// M0 RULE: these kernels fill LDS through the LDS-DMA helpers of lds_tiles.h, which write M0 behind the compiler's back.  Keep
// every register array in them indexed by compile-time constants (no movrel / s_set_gpr_idx code, which would also use M0)
// and add no other LDS-DMA or M0-based construct.
//
// dQ.  A unit's K and V are asked for when the one before has left LDS: K's rows for S^T, K^T's fragments for dQ (kept in
// registers meanwhile) and V's rows for dP^T.
template <int D, int NW, uint32_t MASK, uint32_t SCORE>
__global__ __launch_bounds__(NW * 64, D == 64 ? 2 : 1) void bwd_dq_split_kernel(const BwdArgs a) {
    constexpr uint32_t UT = 32 * D * 2;
    using Score = ScoreMod<SCORE, true>;
    using Mask = PartialMask<MASK>;
    using L = WaveTileLoader<D, 1, 32>;
    __shared__ __attribute__((aligned(1024))) bf16 smem[NW * 64 * D];       // per wave: K, V
    __shared__ float s_rel[Score::kRel ? kRelTableMax : 1];
    __shared__ __attribute__((aligned(256))) uint32_t s_tag[NW][Mask::kTags ? 64 : 4];
    __shared__ uint8_t s_hidden[Mask::kCanvas ? kHiddenTiles : 1];

    int unit, rem;
    if (!unit_of_workgroup(a.B * a.Hkv, a.G * a.NR * (a.Bq / 32), one_by_one(a.B * a.Hkv), unit, rem)) return;
    const int slice = rem & (a.Bq / 32 - 1);
    rem >>= a.Bq == 128 ? 2 : 1;
    const int g = rem % a.G;
    const int b = unit / a.Hkv, hkv = unit % a.Hkv, hq = hkv * a.G + g;
    const int64_t plane = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0);
    const int row = a.kv_order ? min(max(ldc(a.kv_order + plane * a.NR + rem / a.G), 0), a.NR - 1) : a.NR - 1 - rem / a.G;
    const int q0 = row * a.Bq + slice * 32;
    if (q0 >= a.q_len) return;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q_row = q0 + l32;
    const bool real_row = q_row < a.q_len;
    const int q_ld = min(q_row, a.q_len - 1);
    const int64_t line = plane * a.NR + row;
    const int n_full = ldc(a.full_kv_num + line), n_part = ldc(a.kv_num + line);
    const int sub = a.Bk / 64, T = (n_full + n_part) * sub;
    bf16* dq_ptr = a.dQ + b * a.dq_sb + hq * a.dq_sh + (int64_t)q_row * a.dq_ss;
    const int64_t rowi = ((int64_t)b * a.Hq + hq) * a.q_len + q_ld;
    if (T == 0) {
        if (real_row && w == 0) {
            for (int d0 = half * 8; d0 < D; d0 += 16) *(u32x4*)(dq_ptr + d0) = u32x4{0, 0, 0, 0};
            if (a.make_delta && half == 0) {
                a.delta[rowi] = 0.0f;
                a.lse2[rowi] = -INFINITY;
            }
        }
        return;
    }

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
    float rc, neg_delta;
    if (a.make_delta) {
        row_scalars<D, SCORE>(a, b, hq, q_ld, half, dof, rc, neg_delta);
        if (w == 0 && real_row && half == 0) {
            a.delta[rowi] = neg_delta;
            a.lse2[rowi] = rc;
        }
    } else {
        rc = a.lse2[rowi];
        neg_delta = a.delta[rowi];
    }
    const i32x4 k_rsrc = make_rsrc(a.K + b * a.k_sb + hkv * a.k_sh, (uint32_t)((a.kv_len - 1) * a.k_ss + D) * 2u);
    const i32x4 v_rsrc = make_rsrc(a.V + b * a.v_sb + hkv * a.v_sh, (uint32_t)((a.kv_len - 1) * a.v_ss + D) * 2u);
    const Score smod(a.p, hq, a.scale, lds_addr(s_rel));
    smod.fill_table(tid, NW * 64);
    const int q_off = q_offset_of(a.p, b), q_pos = q_ld + q_off, q_wave_min = q0 + q_off;
    const Mask mask(a.p, b, a.kv_len);
    uint32_t q_tag = 0;
    bool scattered = false;
    if constexpr (Mask::kDoc) {
        q_tag = (uint32_t)(a.p.doc_ids + (int64_t)b * a.p.doc_stride_b)[q_pos];
        scattered = Mask::scattered_ids(q_tag);
    }
    typename Mask::CellBase cell_base = {};
    u32x4 q_rect = {};
    if constexpr (Mask::kCells) {
        cell_base = mask.base_of_queries(a.p, q0);
        q_rect = mask.query_rectangle(q_pos, cell_base);
    }
    if constexpr (Mask::kCanvas) {
        if constexpr (!Mask::kCells) q_tag = mask.query_pixel(q_pos);
        fill_hidden_tiles<1, NW * 64>(s_hidden, a.p, a.kv_idx + line * a.NC, n_full, T, sub, a.Bk, q0, tid);
    }
    auto make_tags = [&](int kv0) __attribute__((always_inline)) {
        if constexpr (Mask::kDoc)
            dma_global_dword(lds_addr(&s_tag[w][0]), a.p.doc_ids + (int64_t)b * a.p.doc_stride_b, min(kv0 + lane, a.kv_len - 1) * 4);
        if constexpr (Mask::kCanvas) s_tag[w][lane] = mask.key_pixel(min(kv0 + lane, a.kv_len - 1));
    };

    const L k_load(a.k_ss, 0, lane), v_load(a.v_ss, 0, lane);
    const uint32_t k_lds = lds_addr(smem) + (uint32_t)w * 2 * UT, v_lds = k_lds + UT;
    const RowReader<D> rows(l32, half);
    const TrReader<D> cols(lane);
    const int TU = 2 * T, per_block = 2 * sub, shift = sub == 1 ? 1 : 2, n_blocks = n_full + n_part;
    auto block_at = [&](int u) __attribute__((always_inline)) {
        const int p = min(u >> shift, n_blocks - 1);
        return ldc(p < n_full ? a.full_kv_idx + line * a.NC + p : a.kv_idx + line * a.NC + (p - n_full));
    };
    int u_next = w, blk_next = block_at(w), kv = 0;
    bool partial = false;
    auto advance = [&]() __attribute__((always_inline)) {       // the wave's next unit that is not hidden from all rows
        while (u_next < TU) {
            const int u = u_next;
            kv = blk_next * a.Bk + (u & (per_block - 1)) * 32;
            partial = (u >> shift) >= n_full;
            u_next += NW;
            blk_next = block_at(u_next);
            bool hid = false;
            if constexpr (Mask::kCanvas) hid = (u >> 1) < kHiddenTiles && ((__builtin_amdgcn_readfirstlane((int)s_hidden[u >> 1]) >> (u & 1)) & 1);
            else hid = partial && mask.hidden(q_wave_min, q_wave_min + 31, kv, kv + 31);
            if (!hid) return true;
        }
        return false;
    };
    auto load = [&]() __attribute__((always_inline)) {
        k_load.start(k_rsrc, k_lds, kv * (int)a.k_ss * 2);
        v_load.start(v_rsrc, v_lds, kv * (int)a.v_ss * 2);
    };

    f32x16 dq[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[db][r] = 0.0f;
    if constexpr (Mask::kCanvas || Score::kRel) __syncthreads();
    bool more = advance();
    if (more) {
        if (partial) make_tags(kv);
        load();
    }
    while (more) {
        wait_vmem();
        asm volatile("" ::: "memory");
        const int kv_now = kv;
        const bool masked = partial && !mask.full(q_wave_min, q_wave_min + 31, kv, kv + 31);
        f32x16 sacc, dpacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sacc[r] = 0.0f;
            dpacc[r] = neg_delta;                   // dP - delta comes out of the accumulation
        }
        if constexpr (D == 64) {
            read_ahead<D / 8>([&](auto m) { return rows.read((decltype(m)::value & 1) ? v_lds : k_lds, 0, decltype(m)::value >> 1); },
                              [&](auto m, bf16x8 f) {
                                  constexpr int ks = decltype(m)::value >> 1;
                                  if constexpr (decltype(m)::value & 1) dpacc = mfma32(f, dof[ks], dpacc);
                                  else sacc = mfma32(f, qf[ks], sacc);
                              });
        } else {            // (there the compiler's order is 3 % the better one)
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) {
                sacc = mfma32(rows.read(k_lds, 0, ks), qf[ks], sacc);
                dpacc = mfma32(rows.read(v_lds, 0, ks), dof[ks], dpacc);
            }
        }
        bf16x8 kt[2][D / 32];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int db = 0; db < D / 32; ++db) kt[c][db] = cols.read(k_lds, 16 * c, db);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (K and V have left LDS)
        more = advance();
        if (more) load();

        const int dq0 = q_pos - (kv_now + 4 * half);            // q_idx - kv_idx of element r is dq0 - elem_pos(r)
        const float abase = smod.alibi_base(dq0);
        float rel_uni;
        const bool rel_is_uni = smod.rel_uniform(q_wave_min - (kv_now + 31), q_wave_min + 31 - kv_now, rel_uni);
        auto rel = [&](int r) __attribute__((always_inline)) { return typename Score::RelPos(dq0, abase, -elem_pos(r)); };
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
            if (masked) cells = mask.cell_masks(q_rect, &s_tag[w][0], cell_base, half, kv_now <= mask.kv_last);
        } else if (masked) {
            asm volatile("" ::: "memory");          // keep this a branch
            typename Mask::Bits bits = mask.row_bits(q_pos, kv_now + 4 * half);
            if constexpr (Mask::kDoc) Mask::match_documents(bits, &s_tag[w][0], q_tag, l32, half, scattered);
            if constexpr (Mask::kCanvas) {
                mask.template mask_keys<false>(bits, &s_tag[w][0], q_tag, half, [&](int r, uint32_t m) __attribute__((always_inline)) { dpacc[r] = keep_or_zero(m, dpacc[r]); });
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) dpacc[r] = keep_or_zero(Mask::keep(bits, r), dpacc[r]);
            }
        }
        if (more && partial) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the tags have been read)
            make_tags(kv);
        }
        // dQ^T += K^T dS^T
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            u32x4 ds;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                ds[jj] = pack_bf16(dpacc[8 * c + 2 * jj], dpacc[8 * c + 2 * jj + 1]);
                if constexpr (Mask::kCells) ds[jj] = cells.pair(ds[jj], 4 * c + jj);
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db) dq[db] = mfma32(kt[c][db], __builtin_bit_cast(bf16x8, ds), dq[db]);
        }
    }
    f32x4 quads[D / 8];
#pragma unroll
    for (int q = 0; q < D / 8; ++q)
        quads[q] = f32x4{dq[q >> 2][4 * (q & 3)], dq[q >> 2][4 * (q & 3) + 1], dq[q >> 2][4 * (q & 3) + 2], dq[q >> 2][4 * (q & 3) + 3]};
    const float qscale = a.scale * Score::grad_scale();
    add_quads<NW, D / 8>((f32x4*)smem, w, lane, quads, [&](int q, const f32x4& o) __attribute__((always_inline)) {
        u32x2 pk;
        pk[0] = pack_bf16(o[0] * qscale, o[1] * qscale);
        pk[1] = pack_bf16(o[2] * qscale, o[3] * qscale);
        if (real_row) *(u32x2*)(dq_ptr + 8 * q + 4 * half) = pk;
    });
}

// dK, dV.  Q and dO of 32 rows in two slots a wave, one unit ahead; K and V of the 32 keys in registers, dV^T and dK^T of the
// wave's rows as well.  With dS kept in memory (ds_store) a unit writes its part of a step: that of wave (kb, x) in
// bwd_dkdv_kernel; hidden units of index masks write zeros, those of a canvas are not read back.
template <int D, int NW, uint32_t MASK, uint32_t SCORE, Groups GROUPS>
__global__ __launch_bounds__(NW * 64, D == 64 ? 2 : 1) void bwd_dkdv_split_kernel(const BwdArgs a) {
    constexpr uint32_t UT = 32 * D * 2;
    constexpr int NKS = D / 16, NDB = D / 32;
    using Score = ScoreMod<SCORE, true>;
    using Mask = PartialMask<MASK>;
    using L = WaveTileLoader<D, 1, 32>;
    __shared__ __attribute__((aligned(1024))) bf16 smem[NW * 128 * D];      // per wave: two slots of Q, dO
    __shared__ __attribute__((aligned(256))) float s_row[NW][2][2][64];     // [wave][slot][rc | -delta][row, 32 of 64]
    __shared__ float s_rel[Score::kRel ? kRelTableMax : 1];
    __shared__ __attribute__((aligned(256))) uint32_t s_tag[NW][2][Mask::kTags ? 64 : 4];

    const int slices = a.Bk / 32;
    int unit, slot_rank, parts;
    if (!kv_unit_of_workgroup<GROUPS>(a, a.NC * slices, UnitSets{}, parts, unit, slot_rank)) return;
    const KvHeads<GROUPS> heads(a, parts, unit);
    const int b = unit / a.Hkv, hkv = unit % a.Hkv;
    int col = slot_rank / slices;
    if (a.q_order) {
        const int64_t plane0 = (int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hkv * a.G : 0);
        col = min(max(ldc(a.q_order + plane0 * a.NC + col), 0), a.NC - 1);
    }
    const int part = slot_rank & (slices - 1), kv0 = col * a.Bk + part * 32;
    // (the dQ kernel reads dS in tiles of 64 keys whose first key exists)
    if ((a.ds_store ? kv0 & ~63 : kv0) >= a.kv_len) return;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kv_lane = kv0 + l32, kv_ld = min(kv_lane, a.kv_len - 1);
    bf16x8 kf[NKS], vf[NKS];
    {
        const bf16* kp = a.K + b * a.k_sb + hkv * a.k_sh + (int64_t)kv_ld * a.k_ss + half * 8;
        const bf16* vp = a.V + b * a.v_sb + hkv * a.v_sh + (int64_t)kv_ld * a.v_ss + half * 8;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            kf[ks] = *(const bf16x8*)(kp + ks * 16);
            vf[ks] = *(const bf16x8*)(vp + ks * 16);
        }
    }
    f32x16 dv[NDB], dk[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dv[db][r] = dk[db][r] = 0.0f;

    const int q_off = q_offset_of(a.p, b);
    const Mask mask(a.p, b, a.kv_len);
    const int32_t* docs = Mask::kDoc ? a.p.doc_ids + (int64_t)b * a.p.doc_stride_b : nullptr;
    uint32_t k_tag = 0;
    if constexpr (Mask::kDoc) k_tag = (uint32_t)docs[kv_ld];
    u32x2 corners = {};
    typename Mask::CellBase cell_base = {};
    u32x4 k_rect = {};
    if constexpr (Mask::kCells) {
        cell_base = mask.base_of_keys(a.p, kv0);
        k_rect = mask.key_rectangle(kv_lane, cell_base);
    } else if constexpr (Mask::kCanvas) {
        corners = mask.key_corners(kv_lane);
    }
    const L q_load(a.q_ss, 0, lane), do_load(a.do_ss, 0, lane);
    const uint32_t base = lds_addr(smem) + (uint32_t)w * 4 * UT;
    const RowReader<D> rows(l32, half, base);
    const TrReader<D> cols(lane, base);
    const uint32_t q_bytes = (uint32_t)((a.q_len - 1) * a.q_ss + D) * 2u, do_bytes = (uint32_t)((a.q_len - 1) * a.do_ss + D) * 2u;
    const int per_block = a.Bq / 32, shift = a.Bq == 128 ? 2 : 1;
    int first = w;                                  // the wave's first unit of the next head's walk

    for (int g = heads.first; g < heads.end; ++g) {
        const int hq = hkv * a.G + g;
        const int64_t line = ((int64_t)(a.bm_Bm > 1 ? b : 0) * a.bm_Hm + (a.bm_Hm > 1 ? hq : 0)) * a.NC + col;
        const int n_full = ldc(a.full_q_num + line), n_part = ldc(a.q_num + line), H = (n_full + n_part) * per_block;
        const i32x4 q_rsrc = make_rsrc(a.Q + b * a.q_sb + hq * a.q_sh, q_bytes);
        const i32x4 do_rsrc = make_rsrc(a.dO + b * a.do_sb + hq * a.do_sh, do_bytes);
        const int64_t row0 = ((int64_t)b * a.Hq + hq) * a.q_len;
        const i32x4 rc_rsrc = make_rsrc(a.lse2 + row0, (uint32_t)a.q_len * 4u), nd_rsrc = make_rsrc(a.delta + row0, (uint32_t)a.q_len * 4u);
        const Score smod(a.p, hq, a.scale, lds_addr(s_rel));
        if constexpr (Score::kRel) {
            __syncthreads();                        // (everybody is done with the previous head's row)
            smod.fill_table(tid, NW * 64);
            __syncthreads();
        }
        int ds_slot0 = 0;
        int64_t ds_of_rep = 0;
        if (a.ds_store) {
            ds_slot0 = ldc(a.ds_colbase + line);
            ds_of_rep = ds_rep(a, b, hq);
        }
        // this wave's part of the dS of walk position (pos, sidx)
        auto store_ds = [&](int pos, int sidx, u32x4 c0, u32x4 c1) __attribute__((always_inline)) {
            bf16* dst = a.ds_store + ds_chunk(a, ds_of_rep, ds_slot0 + pos, part >> 1, sidx >> 1) * 4096 +
                        ((part & 1) + 2 * (sidx & 1)) * 1024 + lane * 8;
            __builtin_nontemporal_store(c0, (u32x4*)dst);
            __builtin_nontemporal_store(c1, (u32x4*)(dst + 512));
        };
        // The walk, from its end as in bwd_dkdv_kernel: unit u of the wave is row slice H - 1 - u of the column's merged list.
        auto block_at = [&](int u) __attribute__((always_inline)) {
            const int p = max(H - 1 - u, 0) >> shift;
            return H == 0 ? 0 : ldc(p < n_full ? a.full_q_idx + line * a.NR + p : a.q_idx + line * a.NR + (p - n_full));
        };
        int u_next = first, blk_next = block_at(first);
        int q0 = 0, pos = 0, sidx = 0;              // the unit that is loaded next
        bool partial = false;
        auto advance = [&]() __attribute__((always_inline)) {
            while (u_next < H) {
                const int u = H - 1 - u_next;
                pos = u >> shift;
                sidx = u & (per_block - 1);
                q0 = blk_next * a.Bq + sidx * 32;
                partial = pos >= n_full;
                u_next += NW;
                blk_next = block_at(u_next);
                if (q0 >= a.q_len) continue;        // (rows that do not exist)
                bool hid = false;
                if constexpr (Mask::kCanvas) {
                    if (partial) {
                        const CanvasBlocks cb(a.p);
                        hid = __builtin_amdgcn_readfirstlane(cb.hidden(cb.windows(q0), cb.tokens(kv0)) ? 1 : 0);
                    }
                } else {
                    hid = partial && mask.hidden(q_off + q0, q_off + q0 + 31, kv0, kv0 + 31);
                    if (hid && a.ds_store) store_ds(pos, sidx, u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0});
                }
                if (!hid) return true;
            }
            return false;
        };
        constexpr int kLoads = 2 * L::NI + 2;
        // (a dword load brings 64 rows of scalars; the second 32 are those of the next unit and not used)
        auto load = [&](auto slot_tag) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_tag)::value;
            if (partial) {
                if constexpr (Mask::kDoc) dma_global_dword(lds_addr(&s_tag[w][SLOT][0]), docs, (q_off + min(q0 + lane, a.q_len - 1)) * 4);
                if constexpr (Mask::kCanvas) s_tag[w][SLOT][lane] = mask.query_block_tag(q_off + min(q0 + lane, a.q_len - 1));
            }
            q_load.start(q_rsrc, base + SLOT * 2 * UT, q0 * (int)a.q_ss * 2);
            do_load.start(do_rsrc, base + SLOT * 2 * UT + UT, q0 * (int)a.do_ss * 2);
            dma_dword(rc_rsrc, lds_addr(&s_row[w][SLOT][0][0]), lane * 4, q0 * 4);
            dma_dword(nd_rsrc, lds_addr(&s_row[w][SLOT][1][0]), lane * 4, q0 * 4);
        };
        bool more = advance();
        if (more) load(std::integral_constant<int, 0>{});
        // one unit; false after the last
        auto step = [&](auto slot_tag) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_tag)::value;
            const int q_now = q_off + q0, pos_now = pos, sidx_now = sidx;
            const bool partial_now = partial;
            more = advance();
            if (more) load(std::integral_constant<int, SLOT ^ 1>{});
            if (!more) wait_vmem();
            else if (Mask::kDoc && partial) wait_vmem_but<kLoads + 1>();
            else wait_vmem_but<kLoads>();
            asm volatile("" ::: "memory");
            constexpr uint32_t q_t = SLOT * 2 * UT, do_t = q_t + UT;
            f32x16 sacc, dpacc;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const f32x4 nd = *(const f32x4*)&s_row[w][SLOT][1][8 * rg + 4 * half];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sacc[4 * rg + i] = 0.0f;
                    dpacc[4 * rg + i] = nd[i];
                }
            }
            read_ahead<2 * NKS>([&](auto m) { return rows.read((decltype(m)::value & 1) ? do_t : q_t, 0, decltype(m)::value >> 1); },
                                   [&](auto m, bf16x8 f) {
                                       constexpr int ks = decltype(m)::value >> 1;
                                       if constexpr (decltype(m)::value & 1) dpacc = mfma32(f, vf[ks], dpacc);
                                       else sacc = mfma32(f, kf[ks], sacc);
                                   });
            float rel_uni;
            const bool rel_is_uni = smod.rel_uniform(q_now - (kv0 + 31), q_now + 31 - kv0, rel_uni);
            const bool masked = partial_now && !mask.full(q_now, q_now + 31, kv0, kv0 + 31);
            typename Mask::Bits bits = {};
            typename Mask::CellMasks cells = {{~0u, ~0u}, ~0u};
            if (masked) {
                if constexpr (Mask::kCells) {
                    cells = mask.cell_masks(k_rect, &s_tag[w][SLOT][0], cell_base, half, true);
                } else if constexpr (Mask::kCanvas) {
                    bits = mask.match_queries(&s_tag[w][SLOT][0], corners, half);
                } else {
                    bits = mask.key_bits(kv_lane, q_now + 4 * half);
                    if constexpr (Mask::kDoc) Mask::match_documents(bits, &s_tag[w][SLOT][0], k_tag, l32, half, false);
                }
            }
            u32x4 pk[2], dsk[2];
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) {
                float sv[4], rcv[4], gr[4], pe[4], ds[4];
                using RelPos = typename Score::RelPos;
                constexpr bool kNeedsPos = Score::kAlibi || Score::kRel;
                const int dq0 = kNeedsPos ? q_now + 4 * half - kv_lane : 0;
                const float abase = smod.alibi_base(dq0);
                auto rel = [&](int r) __attribute__((always_inline)) { return kNeedsPos ? RelPos(dq0, abase, elem_pos(r)) : RelPos(0); };
                const RelPos dqk[4] = {rel(4 * c4), rel(4 * c4 + 1), rel(4 * c4 + 2), rel(4 * c4 + 3)};
                const f32x4 rc4 = *(const f32x4*)&s_row[w][SLOT][0][8 * c4 + 4 * half];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sv[i] = sacc[4 * c4 + i];
                    rcv[i] = rc4[i];
                }
                if (rel_is_uni) smod.template p_with_grad4<true>(sv, dqk, rcv, gr, pe, rel_uni);
                else smod.template p_with_grad4<false>(sv, dqk, rcv, gr, pe);
                if (masked && !Mask::kCells) {
                    asm volatile("" ::: "memory");   // keep this a branch
                    if constexpr (Mask::kCanvas) {
                        mask.keep_queries(bits, &s_tag[w][SLOT][0], c4, half, pe);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) pe[i] = keep_or_zero(Mask::keep(bits, 4 * c4 + i), pe[i]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) ds[i] = pe[i] * gr[i] * dpacc[4 * c4 + i];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    pk[c4 >> 1][2 * (c4 & 1) + i] = pack_bf16(pe[2 * i], pe[2 * i + 1]);
                    dsk[c4 >> 1][2 * (c4 & 1) + i] = pack_bf16(ds[2 * i], ds[2 * i + 1]);
                    if constexpr (Mask::kCells) {
                        pk[c4 >> 1][2 * (c4 & 1) + i] = cells.pair(pk[c4 >> 1][2 * (c4 & 1) + i], 2 * c4 + i);
                        dsk[c4 >> 1][2 * (c4 & 1) + i] = cells.pair(dsk[c4 >> 1][2 * (c4 & 1) + i], 2 * c4 + i);
                    }
                }
            }
            if (a.ds_store) store_ds(pos_now, sidx_now, dsk[0], dsk[1]);
            // dV^T += dO^T P, dK^T += Q^T dS
            // (MFMAs: [slice c][block db][dV, dK])
            read_ahead<4 * NDB>([&](auto m) {
                                       constexpr int i = decltype(m)::value >> 1;
                                       return cols.read((decltype(m)::value & 1) ? q_t : do_t, 16 * (i / NDB), i % NDB);
                                   },
                                   [&](auto m, bf16x8 f) {
                                       constexpr int c = (decltype(m)::value >> 1) / NDB, db = (decltype(m)::value >> 1) % NDB;
                                       if constexpr (decltype(m)::value & 1) dk[db] = mfma32(f, __builtin_bit_cast(bf16x8, dsk[c]), dk[db]);
                                       else dv[db] = mfma32(f, __builtin_bit_cast(bf16x8, pk[c]), dv[db]);
                                   });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the slot has been read)
            return more;
        };
        if (more)
            while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
            }
        first = u_next - H;                         // (the heads' walks are dealt to the waves as one)
    }

    f32x4 quads[D / 4];
#pragma unroll
    for (int q = 0; q < D / 4; ++q) {
        const f32x16& acc = q < D / 8 ? dv[(q % (D / 8)) >> 2] : dk[(q % (D / 8)) >> 2];
        quads[q] = f32x4{acc[4 * (q & 3)], acc[4 * (q & 3) + 1], acc[4 * (q & 3) + 2], acc[4 * (q & 3) + 3]};
    }
    const float kscale = a.scale * Score::grad_scale();
    add_quads<NW, D / 4>((f32x4*)smem, w, lane, quads, [&](int q, const f32x4& o) __attribute__((always_inline)) {
        const bool is_k = q >= D / 8;
        if (GROUPS != Groups::kWhole && heads.apart) {
            if (kv_lane < a.kv_len) *(f32x4*)(heads.sums(a, unit, is_k, D) + (int64_t)kv_lane * D + 8 * (q % (D / 8)) + 4 * half) = o;
            return;
        }
        const float s = is_k ? kscale : 1.0f;
        bf16* out = is_k ? a.dK + b * a.dk_sb + hkv * a.dk_sh + (int64_t)kv_lane * a.dk_ss
                         : a.dV + b * a.dv_sb + hkv * a.dv_sh + (int64_t)kv_lane * a.dv_ss;
        u32x2 pk;
        pk[0] = pack_bf16(o[0] * s, o[1] * s);
        pk[1] = pack_bf16(o[2] * s, o[3] * s);
        if (kv_lane < a.kv_len) *(u32x2*)(out + 8 * (q % (D / 8)) + 4 * half) = pk;
    });
}

// Where the split kernels take over (waves, 0: they do not), by the slices of 32 rows or keys of the launch and their length.
// us, bwd_dq_kernel -> 4 waves / 8 waves: causal, S = 4096, D = 64, 1 head 58 -> 23 / 16, 4 59 -> 25 / 22, 8 59 -> 36 / 41, 16 86 -> 70 / 82, 32
// 127 -> 136; D = 128 (4 waves), 1 head 86 -> 36, 4 87 -> 44, 8 88 -> 85, 16 139 -> 168; S = 1000, D = 64, 8 / 32 / 64 heads 18.8 -> 8.8 / 7.8, 19.3
// -> 17.3, 27 -> 32, D = 128, 8 / 16 / 32 heads 27 -> 14, 27 -> 19, 29 -> 38; S = 300, D = 64, 32 / 64 heads 8.2 -> 7.0, 8.4 -> 11.0, D = 128, 8 / 32
// heads 11.6 -> 8.2, 11.8 -> 13.4; no mask, S = 2048, D = 64, 4 / 8 / 16 heads 32 -> 14 / 11, 33 -> 18 / 21, 33 -> 34, D = 128, 4 / 8 / 16
// heads 46 -> 22, 46 -> 42, 52 -> 83; window of 512, S = 4096, D = 64, 4 / 8 heads 14.8 -> 8.9 / 12.3, 15.1 -> 16.6, D = 128, 4 heads 20.5 -> 21.6.
// Short rows lose first (bwd_dq_kernel -> 4 waves): D = 64, no mask, S = 520, 37 heads 14.7 -> 17.9, S = 800, 30 heads 18.3 -> 21.1, causal, S = 130, 102 heads
// 8.8 -> 12.3, S = 520, 45 heads 13.9 -> 16.2, documents of 16 to 100, S = 8192, 4 heads 12.9 -> 17.6, 8 heads 17.3 -> 32.0 (of 256 to 4096 77 ->
// 34, 83 -> 60: the host cannot tell them apart, line_shape); D = 128, no mask, S = 520, 15 heads 20.3 -> 22.4, S = 800, 20 heads 25.8 -> 39.7, documents of
// 16 to 100, S = 8192, 2 heads 16.5 -> 21.3 (of 256 to 4096 97 -> 46), one head's window of 1000, S = 16384 34.5 -> 41.3 (split_waves has why).
template <uint32_t MASK>
int dq_split_waves(const BwdArgs& a, int D) {
    const int64_t groups = unit_grid(a.B * a.Hkv, a.G * a.NR * (a.Bq / 32));
    const LineShape rows = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const int64_t keys = rows.sure;
    if (D == 128) {
        int64_t most = keys >= 2048 ? 512 : 256;
        if (rows.sure_uneven) most = keys >= 4096 ? 1024 : keys >= 768 ? 512 : keys >= 448 ? 384 : 256;
        if (a.B * a.Hkv == 1 && 8 * keys < a.kv_len) most = 256;
        return groups <= most ? 4 : 0;
    }
    int64_t most = keys >= 2048 ? 768 : 512;
    if (rows.sure_uneven) most = keys >= 4096 ? 2048 : keys >= 1000 ? 1024 : keys >= 640 ? 640 : 512;
    if (groups > most) return 0;
    return (groups <= 256 ? rows.longest >= 512 : groups <= 512 && rows.sure_uneven && keys >= 2048) ? 8 : 4;
}
// The pairs form of dQ (bwd_dq_kernel), by the length of the longest rows with Bq = 64, and with Bq = 128 by the workgroups of 128
// uneven rows, whose halves end a launch sooner.  us of the whole backward, without -> with: Bq = 64, D = 128, causal, S = 8192, 16
// heads 950 -> 892, S = 512, 128 heads 85 -> 81, S = 300, 1024 heads 280 -> 284, window of 1024 546 -> 493, D = 64, S = 8192 527 -> 488, S = 835, 45 x
// 32 heads 931 -> 885, S = 512 45 -> 48, documents, S = 16384, 16 heads 414 -> 373; Bq = 128, S x heads, D = 64, causal, 8192 x 16 532 -> 506, 2048 x 32
// 104 -> 99, 16384 x 16 1952 -> 1905, 8192 x 32 1010 -> 1013, but 1024 x 256 188 -> 193, D = 128, causal, 4096 x 16 294 -> 262, but 8192 x 16 909 -> 918.
// us of dQ, Bq = 128: documents of 256 to 4096, their longest rows in halves, 8192 x 16 99 -> 76, ALiBi, 16384 x 6 110 -> 74, 16384 x 16 180 -> 162, 2048 x 128
// 132 -> 128, but 8192 x 64 345 -> 348, 16384 x 32 337 -> 348, D = 128, 4096 x 16 119 -> 78, 8192 x 12 127 -> 99, 16384 x 6 150 -> 121, but 16384 x 9 162 -> 168,
// 16384 x 16 286 -> 304; of 16 to 100, which the host cannot tell from longer ones, 16384 x 6 21.9 -> 23.0, 2048 x 128 46.1 -> 47.2, D = 128, 8192 x 8 26.3 ->
// 25.8; shorter or even rows at D = 64, causal, 1050 x 52 27.8 -> 26.9, 1600 x 36 39 -> 34, no mask, 1500 x 32 41 -> 38, 2000 x 20 49 -> 43, canvases, 64 x 64,
// K = 21, 12 heads 50 -> 43, 32 x 32, K = 21, 48 heads 34 -> 29, but no mask, 1300 x 40 38 -> 45, 4000 x 14 97 -> 111,
// row-major, K = 27, 16 heads 68 -> 80 (in tiles of 8 x 8 70 -> 60).
template <uint32_t MASK>
bool dq_pairs_pay(const BwdArgs& a, int D) {
    const LineShape rows = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const unsigned grid = unit_grid(a.B * a.Hkv, a.G * a.NR);
    if (a.Bq == 64) return rows.longest >= (D == 64 ? 768 : 448) && grid <= kMaxLaunch;
    if (D == 64 && rows.sure >= 1024 && 2 * grid <= (rows.uneven ? 4 : 3) * 256) return true;
    if (!rows.uneven || a.kv_len < 2048) return false;
    return grid <= (D == 64 ? 8 * 256 : PartialMask<MASK>::kDoc ? 4 * 256 : 2 * 256);
}
// Documents with Bq = 128 in the pairs form: how many of the rows of blocks, the longest, go in halves while the others stay whole, unless even the
// longest is short (half_or_row).  us of dQ, a workgroup per row of blocks / all in halves / this: D = 64, documents of 16 to 100, 8192 x 16 28.7 / 33.8 / 28.7,
// ALiBi, 16384 x 16 46.4 / 56.7 / 46.8, of 100 to 400, 8192 x 16 31.7 / 38.2 / 32.0, 4096 x 16 25.2 / 23.1 / 25.0, of 256 to 4096, 8192 x 16 98 / 74 / 76, ALiBi,
// 16384 x 16 175 / 166 / 158; D = 128, of 16 to 100, 8192 x 8 26.1 / 30.4 / 25.5, 2048 x 48 39.4 / 44.1 / 38.2, of 100 to 400, 8192 x 12 43.8 / 50.4 / 44.9, of 256 to
// 4096, 8192 x 8 94 / 70 / 70, ALiBi, 4096 x 16 118 / 79 / 76, 2048 x 48 74 / 75 / 66, 16384 x 6 145 / 121 / 124.  All of them at D = 64 while the whole rows are
// about a round (a quarter of long ones, with a loop that is slower: 8192 x 16 79 and 77), a quarter then (a third, ALiBi, 16384 x 16 167 and 164).
// A relative bias under a soft-cap keeps all in halves: 12 and 19 spills.
template <uint32_t MASK, uint32_t SCORE>
constexpr bool dq_can_mix() {
    return PartialMask<MASK>::kDoc && !((SCORE & FLEXATTN_SCORE_REL_BIAS) && (SCORE & FLEXATTN_SCORE_SOFTCAP));
}
inline int dq_halved_rows(int D, int NR, unsigned grid) { return D == 128 ? halved_rows(NR) : grid <= 4 * 256 ? NR : (NR + 3) / 4; }
// us, bwd_dkdv_kernel -> 4 waves / 8 waves: causal, S = 4096, D = 64, 1 head 51 -> 39 / 21, 4 52 -> 41 / 29, 8 58 -> 50 / 54, 16 92 -> 98; D = 128 (4
// waves), 1 head 72 -> 45, 4 74 -> 58, 8 90 -> 111; 8 query and 1 KV heads, S = 2048 199 -> 145 / 74, D = 128 280 -> 166; 32 / 8, S = 2048 101 -> 77 /
// 53; S = 1000, D = 64, 8 / 16 / 32 heads 16.8 -> 13.7 / 10.1, 17.1 -> 15.9 / 15.3, 23.2 -> 25.1, D = 128, 8 / 16 heads 23.8 -> 16.8, 24.2 -> 23.9; S =
// 300, D = 64, 32 / 64 heads 9.4 -> 8.8, 12.0 -> 14.1, D = 128, 8 / 32 heads 12.9 -> 10.3, 13.4 -> 16.3; no mask, S = 2048, D = 64, 4 / 8 / 16 heads 29
// -> 22 / 15, 29 -> 26 / 28, 41 -> 48, D = 128, 4 / 8 heads 40 -> 26, 42 -> 51; window of 512 or prefix of 256, S = 8192, D = 64, 2 x 16 / 4 heads,
// whose first columns are as long as the sequence times the group 557 -> 324 / 311.
// Short columns lose first (bwd_dkdv_kernel -> 4 waves): D = 64, no mask, S = 130, 51 heads, 8 waves 9.0 -> 12.2, S = 800, 30 heads 21.1 -> 24.8,
// documents of 16 to 100, S = 8192, 4 heads 14.3 -> 17.2 (of 256 to 4096 63 -> 40: the host cannot tell them apart), a window of 200 or prefix of 100, S =
// 800, 81 heads, 8 waves 41 -> 63; D = 128, no mask, S = 800, 10 heads 22.4 -> 29.1 (causal 22.5 -> 16.7), documents of 16 to 100, S = 8192, 2 heads 15.3 -> 21.5
// (of 256 to 4096 74 -> 54), a window of 200 or prefix of 100, S = 800, 40 heads 36 -> 48 (S = 2080, 15 heads 72 -> 53).
// The lines go by the workgroups launched, not by the keys' slices, some of which lie past the last key.  Few long columns (a prefix with a window): as many
// workgroups as the columns have rows, whose chain is what ends the launch.
template <uint32_t MASK>
int dkdv_split_waves(const BwdArgs& a, int D) {
    const int64_t groups = unit_grid(a.B * a.Hkv * a.head_parts, a.NC * (a.Bk / 32));
    // (the columns of a mask that is its own transpose's mirror image are shaped like its rows; a prefix is seen by all rows)
    LineShape cols = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const bool few_long = mask_uses(MASK, FLEXATTN_M_PREFIX) && !cols.uneven;
    if (mask_uses(MASK, FLEXATTN_M_PREFIX)) cols = {a.q_len, true, a.q_len, true};
    const int64_t rows = cols.sure < a.q_len ? cols.sure : a.q_len;
    auto between = [](int64_t lo, int64_t v, int64_t hi) { return v < lo ? lo : v > hi ? hi : v; };
    if (D == 128) {
        int64_t most = 256;
        if (cols.sure_uneven) most = rows >= 2048 ? 512 : rows >= 1000 ? 448 : rows >= 448 ? 320 : 256;
        if (few_long) most = between(256, 5 * rows / 8, 2048);
        return groups <= most ? 4 : 0;
    }
    if (few_long) return groups <= between(256, rows / 2, 2048) ? 8 : groups <= between(256, rows, 2048) ? 4 : 0;
    int64_t most = PartialMask<MASK>::kDoc && a.q_len >= 1000 ? 512 : 448;
    if (cols.sure_uneven) most = rows >= 2048 ? 1024 : 512;
    if (groups > most) return 0;
    return groups <= 256 || (groups <= 512 && cols.sure_uneven && rows >= 2048) ? 8 : 4;
}

// dK/dV at D = 64: own rows, but for launches that are as long as their longest column of blocks, where a workgroup is
// alone on its CU most of the time: there the exchange is faster, whose operands are read further ahead.  They are
// told by what the columns' steps make of 768 workgroups (three per CU) beside the longest column: a third of it (270 of
// 768 for a mask whose columns are as long as the longest).  Windows and documents have columns of about one length and
// hidden blocks to leave out, a soft-cap more vector work than the operands' reads take.
// us, exchange -> own rows: causal, S = 1024, 8 heads 16.8 -> 18.7; S = 4096, 8 heads 57.7 -> 59.8; S = 2048, 16 heads 38.7 -> 38.1, 32 heads 56.5 -> 54.3; no mask, S = 1024, 8 heads 16.9 -> 17.9, S = 4096, 8 heads
// 78.2 -> 76.7; window 512 or prefix 128, S = 8192, 16 heads 163 -> 170, S = 2048, 32 heads 55.5 -> 53.8.
template <uint32_t MASK>
bool own_rows_pay(const BwdArgs& a, unsigned grid) {
    const float longest = a.q_len / 64.0f;          // steps
    float mean = MASK == FLEXATTN_MASK_NONE ? longest : 0.5f * longest;
    if (mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW))
        mean = fminf(longest, a.p.window / 64.0f + 2.0f + longest * a.p.prefix_len / a.kv_len);
    return grid * mean > 270.0f * longest;
}
// dK/dV of canvases at D = 64: whether leaving hidden steps and blocks out pays.  64 tokens in a row reach over a canvas of up to
// 100 pixels, and a window over most of a small one: nothing is hidden, and looking for it costs up to 9 % (us, computed whole -> left out, 262144
// tokens in all: row-major 24 x 24, K = 21 119 -> 127, 40 x 200, K = 7 89 -> 94, 64 x 64, K = 7 106 -> 111, 100 x 100, K = 3 84 -> 89, 128 x 128, K = 3 90 -> 94, K = 7
// 160 -> 157, K = 27 537 -> 484, 200 x 40, K = 3 120 -> 114, K = 13 399 -> 319; tiles of 8 x 8, 16 x 16, K = 7 74 -> 79, 24 x 24, K = 13 103 -> 99, K = 21 122 -> 131, 32 x
// 32, K = 7 109 -> 98, K = 27 180 -> 186, 64 x 64, K = 27 246 -> 242; Morton order alike).
inline bool canvas_cut_pays(const flexattn_mod_params& p) {
    if (p.na_layout == FLEXATTN_NA_ROW_MAJOR) return p.na_width >= 160 || (p.na_width > 100 && p.na_kernel >= 7);
    const int side = p.na_width < p.na_height ? p.na_width : p.na_height;
    return side >= 24 && 5 * p.na_kernel <= 3 * side;
}
// Whether dK/dV looks for steps to leave out (LEAVE).  Lists of 64 x 64 blocks have none.  Workgroups that all run at once end with the longest
// column, which seldom has any, and later by the look: D = 128, 11 x 2 heads, S = 465, prefix, 128 x 128 16.1 -> 16.4 us.  A relative bias spills 5 registers with
// the walk's gap, and looks only where most columns have hidden steps, those of 128 keys, or behind a q_len in the first half of its block: us, D = 128, 16 heads, no look -> look,
// B x S, window of 300 (S = 300: of 100), 16 x 300 49.1 -> 46.3, 128 x 128 50.7 -> 46.9, 16 x 947 / 4 KV heads 177 -> 172, 128 x 128 206 -> 193, but 8 x 1000 109.7 -> 111.3
// (128 x 128 114.6 -> 111.5), with dS in memory 111.7 -> 115.4.
template <uint32_t MASK, uint32_t SCORE>
bool leaving_out_pays(const BwdArgs& a, int D, unsigned grid) {
    if ((SCORE & FLEXATTN_SCORE_REL_BIAS) && a.Bk == 64 && (a.q_len - 1) % 128 >= 64) return false;
    return a.Bq + a.Bk > 128 && grid > 256u * (unsigned)bwd_waves_per_simd_of(D);
}
template <uint32_t MASK, uint32_t SCORE, Groups GROUPS>
void launch_dkdv64(const BwdArgs& a, unsigned grid, bool leave_out, hipStream_t st) {
    constexpr bool own = dkdv_own_rows<64, MASK, SCORE>(), canvas = PartialMask<MASK>::kCanvas;
    constexpr bool even = mask_uses(MASK, FLEXATTN_M_DOCUMENT) ||
                          (mask_uses(MASK, FLEXATTN_M_SLIDING_WINDOW) && !mask_uses(MASK, FLEXATTN_M_PREFIX));
    if constexpr (own && !even && !(SCORE & FLEXATTN_SCORE_SOFTCAP)) {
        if (!own_rows_pay<MASK>(a, grid)) {
            hipLaunchKernelGGL((bwd_dkdv_kernel<64, MASK, SCORE, false, canvas, GROUPS>), dim3(grid), dim3(256), 0, st, a);
            return;
        }
    }
    if constexpr (canvas) {
        if (!canvas_cut_pays(a.p)) {
            hipLaunchKernelGGL((bwd_dkdv_kernel<64, MASK, SCORE, false, false, GROUPS>), dim3(grid), dim3(256), 0, st, a);
            return;
        }
    }
    if constexpr (dkdv_can_leave<64, MASK, SCORE>() && GROUPS == Groups::kWhole) {          // (launches for parts are no larger than a round)
        if (leave_out) {
            hipLaunchKernelGGL((bwd_dkdv_kernel<64, MASK, SCORE, own, canvas, GROUPS, true>), dim3(grid), dim3(256), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((bwd_dkdv_kernel<64, MASK, SCORE, own, canvas, GROUPS>), dim3(grid), dim3(256), 0, st, a);
}

// Rows that the longest column of blocks sees (of a canvas: those around its pixels).
template <uint32_t MASK>
int64_t longest_column(const BwdArgs& a) {
    if (mask_uses(MASK, FLEXATTN_M_PREFIX)) return a.q_len;
    const LineShape cols = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const int64_t rows = PartialMask<MASK>::kCanvas ? cols.sure : cols.longest;
    return rows < a.q_len ? rows : a.q_len;
}
// What speaks against parts beside the steps they spare (kv_head_parts).  Whole groups that are split among the waves of their workgroups
// use the chip already: two parts that would be split among fewer, parts of a single head that would not be split, small groups of more workgroups than two to a CU and parts of unlike size of more than one lose.  Parts of unlike size, whose larger ones end the launch, only
// while the CUs are hardly shared, or, of a large group, where sharing them costs less than a head, or where the few long columns of a prefix are what a launch is made of (us, dK/dV, whole / two / four,
// S x query / KV heads: D = 64, no mask, 4000 x 4 / 2 45 / 64, 1500 x 20 / 5 37 / 51 / 41, 1000 x 56 / 8 45 / 65 / 49, causal, 4000 x 8 / 4 48 / 54, 4000 x 12 / 3 75 / 75 / 82; a window of 200 or a prefix of 64, 4000 x 12 / 6
// 45 / 60, of 300 or 50, 2048 x 40 / 8 66 / 79, but 7000 x 6 / 3 70 / 53, 12000 x 4 / 2 114 / 67, D = 128 284 / 155; unlike parts: no mask,
// 6000 x 5 / 1, D = 64 137 / - / 195, causal, 4000 x 9 / 3, D = 128 125 / 160, 1500 x 18 / 6 53 / 68, but no mask, 1500 x 7 / 1, D = 64 56 / 38 / 25, causal with a soft-cap, 3888 x 35 / 5, D = 128 580 / 393).
// Documents, many of which the host cannot tell to be short, spare a workgroup little and pay the sums of all keys.  So few sums for each head that is spared that documents of 16 to 200 tokens do not lose by
// more than 3 % (D = 128, 1500 x 4 / 2, of 16 to 100, 8 %: 14.7 / 15.7, of 256 to 4096 40 / 28), or else they ask (kPartsIfLong).  Whole groups that are split do not ask, bwd_dkdv_kernel is no match for them: 3000 x 2 x 8 / 2,
// D = 64, documents of 16 to 100, split 17, in two 23, whole after the question 27, of 256 to 4096 97 / 86; 9000 x 4 / 1 18 / - / 21 and 122 / - / 63.
inline bool short_documents_pay(const BwdArgs& a, int D, int parts) {
    const int64_t sums = a.B * a.Hkv * ((a.kv_len + 63) / 64) * (int64_t)parts * 64 * D, spared = a.G - (a.G + parts - 1) / parts;      // of dK; heads
    return sums <= (a.G >= 4 ? 1200000 : D == 128 ? 800000 : 0) * spared;
}
template <uint32_t MASK>
bool parts_pay(const BwdArgs& a, int D, int parts) {
    auto waves = [&](int p) {
        BwdArgs of = a;
        of.head_parts = p;
        return dkdv_split_waves<MASK>(of, D);
    };
    const int whole = waves(1), then = waves(parts);
    const int64_t groups = a.B * a.Hkv * ((a.kv_len + 63) / 64) * (int64_t)parts;
    const LineShape rows = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const bool prefix = mask_uses(MASK, FLEXATTN_M_PREFIX), few_long = prefix && !rows.uneven && (groups <= 384 || a.B * a.Hkv <= (D == 64 ? 3 : 6));
    if (a.G % parts) {
        if (groups > (D == 64 ? 128 : 256) && !(a.G > 2 * parts && (D == 64 || prefix || rows.sure_uneven)) && !(a.G >= 3 * parts && groups <= 512) && !few_long) return false;
        if (whole && groups > 256 && !few_long) return false;
    }
    if (whole && ((parts == 2 && then < whole) || (a.G < 4 && groups > 512 && !few_long) || (D == 64 && !then && a.G < 2 * parts))) return false;
    return !PartialMask<MASK>::kDoc || short_documents_pay(a, D, parts) || (!whole && a.q_order);
}
// dV (blockIdx.y = 0) and dK from what the parts of every group left: eight dims a thread, in the order of the parts.
template <bool IF_LONG>
__global__ __launch_bounds__(256) void kv_parts_sum_kernel(const BwdArgs a, int D, float kscale) {
    const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x, rows = (int64_t)a.B * a.Hkv * a.kv_len;
    const int shift = D == 128 ? 4 : 3, d = ((int)at & ((1 << shift) - 1)) * 8;
    const int64_t row = at >> shift;
    if (row >= rows) return;
    if (IF_LONG && parts_if_long(a) == 1) return;       // (the columns' workgroups have written)
    const bool is_k = blockIdx.y != 0;
    const float* src = a.kv_part + ((int64_t)is_k * rows + row) * D + d;
    f32x4 lo = *(const f32x4*)src, hi = *(const f32x4*)(src + 4);
    for (int part = 1; part < a.head_parts; ++part) {
        src += 2 * rows * D;
        lo += *(const f32x4*)src;
        hi += *(const f32x4*)(src + 4);
    }
    const float s = is_k ? kscale : 1.0f;
    const int kv = (int)(row % a.kv_len), unit = (int)(row / a.kv_len), b = unit / a.Hkv, hkv = unit - b * a.Hkv;
    bf16* out = is_k ? a.dK + b * a.dk_sb + hkv * a.dk_sh + (int64_t)kv * a.dk_ss : a.dV + b * a.dv_sb + hkv * a.dv_sh + (int64_t)kv * a.dv_ss;
    *(u32x4*)(out + d) = u32x4{pack_bf16(lo[0] * s, lo[1] * s), pack_bf16(lo[2] * s, lo[3] * s), pack_bf16(hi[0] * s, hi[1] * s), pack_bf16(hi[2] * s, hi[3] * s)};
}

// dK/dV, and what adds the parts of groups up.  kPartsIfLong, whose launch has workgroups enough for whole groups as well: us, whole / in parts / this, S x query / KV heads, documents of 16 to 100, 30 to 300
// and 256 to 4096: D = 64, 6000 x 8 / 4 15.3 / 23.5 / 18.2, 18.9 / 24.9 / 21.7, 75 / 55 / 56, 8000 x 6 / 3 15.8 / 23.9 / 18.5, 19.3 / 25.2 / 21.9, 101 / 69 / 70; D = 128, 6000 x 8 / 4 23.6 / 39.4 / 25.9,
// 28.7 / 41.7 / 30.3, 108 / 81 / 81, 6000 x 32 / 4 64 / 73 / 67, 83 / 80 / 81, 408 / 267 / 267, 3000 x 2 x 8 / 2 31.7 / 38.2 / 34.0, 40.3 / 40.6 / 41.4, 212 / 97 / 97.  (What is left of short ones' loss is
// the launch that adds nothing up, and the question, 1 us.)
template <uint32_t MASK, uint32_t SCORE, Groups GROUPS>
void launch_dkdv(const BwdArgs& args, int D, bool uneven, hipStream_t st) {
    BwdArgs a = args;
    const int units = a.B * a.Hkv * a.head_parts;
    const int waves = GROUPS == Groups::kPartsIfLong ? 0 : dkdv_split_waves<MASK>(a, D), per_unit = a.NC * (a.Bk / (waves ? 32 : 64));
    const unsigned grid = std::max(unit_grid(units, per_unit), GROUPS == Groups::kPartsIfLong ? unit_grid(a.B * a.Hkv, per_unit) : 0u);
    constexpr bool canvas = PartialMask<MASK>::kCanvas;
    a.least_steps = a.G < 4 ? 12 : 5;
    if constexpr (GROUPS != Groups::kPartsIfLong) {
        if (D == 128 && waves) hipLaunchKernelGGL((bwd_dkdv_split_kernel<128, 4, MASK, SCORE, GROUPS>), dim3(grid), dim3(256), 0, st, a);
        else if (waves == 8) hipLaunchKernelGGL((bwd_dkdv_split_kernel<64, 8, MASK, SCORE, GROUPS>), dim3(grid), dim3(512), 0, st, a);
        else if (waves) hipLaunchKernelGGL((bwd_dkdv_split_kernel<64, 4, MASK, SCORE, GROUPS>), dim3(grid), dim3(256), 0, st, a);
    }
    if (!waves) {
        a.abreast = units_abreast(units, per_unit, bwd_waves_per_simd_of(D), uneven && !mask_uses(MASK, FLEXATTN_M_DOCUMENT) ? kColumnsAbreast : 1);
        const bool leave_out = leaving_out_pays<MASK, SCORE>(a, D, grid);
        if (D == 64) launch_dkdv64<MASK, SCORE, GROUPS>(a, grid, leave_out, st);
        else if constexpr (dkdv_can_leave<128, MASK, SCORE>()) {
            if (leave_out) hipLaunchKernelGGL((bwd_dkdv_kernel<128, MASK, SCORE, false, canvas, GROUPS, true>), dim3(grid), dim3(256), 0, st, a);
            else hipLaunchKernelGGL((bwd_dkdv_kernel<128, MASK, SCORE, false, canvas, GROUPS>), dim3(grid), dim3(256), 0, st, a);
        } else {
            hipLaunchKernelGGL((bwd_dkdv_kernel<128, MASK, SCORE, false, canvas, GROUPS>), dim3(grid), dim3(256), 0, st, a);
        }
    }
    if constexpr (GROUPS != Groups::kWhole) {
        const float kscale = a.scale * ScoreMod<SCORE>::grad_scale();
        const int64_t eights = (int64_t)a.B * a.Hkv * a.kv_len * (D / 8);
        hipLaunchKernelGGL(kv_parts_sum_kernel<GROUPS == Groups::kPartsIfLong>, dim3((unsigned)((eights + 255) / 256), 2), dim3(256), 0, st, a, D, kscale);
    }
}

template <uint32_t MASK, uint32_t SCORE>
int launch_bwd_variant(const BwdArgs& args, int D, uint32_t stages, hipStream_t st) {
    BwdArgs a = args;
    const int units = a.B * a.Hkv;
    a.head_parts = a.kv_part ? kv_head_parts(units, a.G, a.kv_len, D, longest_column<MASK>(a), [&](int p) { return parts_pay<MASK>(a, D, p); }) : 1;
    if (a.head_parts == 1) a.kv_part = nullptr;
    const LineShape rows_shape = line_shape<MASK>(a.p, a.q_len, a.kv_len);
    const bool uneven = rows_shape.uneven;
    auto rows_by = [&](int rows) { return units_abreast(units, a.G * rows, bwd_waves_per_simd_of(D), rows_abreast<MASK>(rows_shape, a.kv_len, D)); };
    const unsigned grid_q = unit_grid(a.B * a.Hkv, a.G * a.NR);
    const bool kv = stages & FLEXATTN_BWD_DKDV, q = stages & FLEXATTN_BWD_DQ;
    // dQ first, where it makes the row scalars that dK/dV reads; last, after a pass that makes them, where it is written over
    // what either reads
    if ((stages & FLEXATTN_BWD_DELTA) && (!q || a.dq_last)) {
        const size_t rows = (size_t)a.B * a.Hq * a.q_len;
        if (D == 128) hipLaunchKernelGGL((bwd_delta_kernel<128, SCORE>), dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((bwd_delta_kernel<64, SCORE>), dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, st, a);
    }
    auto run_dq = [&] {
        BwdArgs aq = a;
        aq.make_delta = (stages & FLEXATTN_BWD_DELTA) && !a.dq_last;
        const int waves = dq_split_waves<MASK>(a, D);
        if (waves) {
            const dim3 slices(unit_grid(a.B * a.Hkv, a.G * a.NR * (a.Bq / 32)));
            if (D == 128) hipLaunchKernelGGL((bwd_dq_split_kernel<128, 4, MASK, SCORE>), slices, dim3(256), 0, st, aq);
            else if (waves == 8) hipLaunchKernelGGL((bwd_dq_split_kernel<64, 8, MASK, SCORE>), slices, dim3(512), 0, st, aq);
            else hipLaunchKernelGGL((bwd_dq_split_kernel<64, 4, MASK, SCORE>), slices, dim3(256), 0, st, aq);
        } else if (dq_pairs_pay<MASK>(a, D)) {
            constexpr bool can_mix = dq_can_mix<MASK, SCORE>();
            const bool mixed = can_mix && a.Bq == 128;
            BwdArgs part = aq;
            part.halved = a.Bq == 64 ? 0 : mixed ? dq_halved_rows(D, a.NR, grid_q) : a.NR;
            part.abreast = rows_by(a.NR + part.halved);
            const dim3 pieces(unit_grid(a.B * a.Hkv, a.G * (a.NR + part.halved)));
            if (D == 128 && mixed) hipLaunchKernelGGL((bwd_dq_kernel<128, 4, MASK, SCORE, false, true, true, can_mix>), pieces, dim3(256), 0, st, part);
            else if (D == 128) hipLaunchKernelGGL((bwd_dq_kernel<128, 4, MASK, SCORE, false, true, true>), pieces, dim3(256), 0, st, part);
            else if (mixed) hipLaunchKernelGGL((bwd_dq_kernel<64, 4, MASK, SCORE, false, true, true, can_mix>), pieces, dim3(256), 0, st, part);
            else hipLaunchKernelGGL((bwd_dq_kernel<64, 4, MASK, SCORE, false, true, true>), pieces, dim3(256), 0, st, part);
        } else {
            aq.abreast = rows_by(a.NR);
            if (D == 128 && a.Bq == 128) hipLaunchKernelGGL((bwd_dq_kernel<128, 4, MASK, SCORE>), dim3(grid_q), dim3(256), 0, st, aq);
            else if (D == 128) hipLaunchKernelGGL((bwd_dq_kernel<128, 2, MASK, SCORE>), dim3(grid_q), dim3(128), 0, st, aq);
            else if (a.Bq == 128) hipLaunchKernelGGL((bwd_dq_kernel<64, 4, MASK, SCORE>), dim3(grid_q), dim3(256), 0, st, aq);
            else hipLaunchKernelGGL((bwd_dq_kernel<64, 2, MASK, SCORE>), dim3(grid_q), dim3(128), 0, st, aq);
        }
    };
    if (q && !a.dq_last) run_dq();
    if (kv) {
        if (!a.kv_part) launch_dkdv<MASK, SCORE, Groups::kWhole>(a, D, uneven, st);
        else if (!PartialMask<MASK>::kDoc || short_documents_pay(a, D, a.head_parts)) launch_dkdv<MASK, SCORE, Groups::kParts>(a, D, uneven, st);
        else if constexpr (PartialMask<MASK>::kDoc) launch_dkdv<MASK, SCORE, Groups::kPartsIfLong>(a, D, uneven, st);
    }
    if (q && a.dq_last) run_dq();
    if (stages & kBwdStageCaptured) {
        a.abreast = rows_by(a.NR);
        if constexpr ((SCORE & (FLEXATTN_SCORE_ALIBI | FLEXATTN_SCORE_REL_BIAS)) != 0) {
            if (D == 128 && a.Bq == 128) hipLaunchKernelGGL((bwd_dq_kernel<128, 4, MASK, SCORE, true>), dim3(grid_q), dim3(256), 0, st, a);
            else if (a.Bq == 128) hipLaunchKernelGGL((bwd_dq_kernel<64, 4, MASK, SCORE, true>), dim3(grid_q), dim3(256), 0, st, a);
            // (us, two waves -> pairs, ALiBi, causal: D = 64 / 128, S = 8192, 16 heads 276 -> 237 / 435 -> 321, S = 700, 256 heads 59 -> 52 / 100
            // -> 85, S = 1000, 4 heads 26 -> 17 / 32 -> 21, but S = 300, 1024 heads 71 -> 76 / 141 -> 143; documents, S = 8192, 16 heads 121 -> 85 / 178 -> 121)
            else if (const bool pairs = line_shape<MASK>(a.p, a.q_len, a.kv_len).longest >= 448 && grid_q <= kMaxLaunch; D == 128) {
                if (pairs) hipLaunchKernelGGL((bwd_dq_kernel<128, 4, MASK, SCORE, true, true, true>), dim3(grid_q), dim3(256), 0, st, a);
                else hipLaunchKernelGGL((bwd_dq_kernel<128, 2, MASK, SCORE, true>), dim3(grid_q), dim3(128), 0, st, a);
            } else if (pairs) hipLaunchKernelGGL((bwd_dq_kernel<64, 4, MASK, SCORE, true, true, true>), dim3(grid_q), dim3(256), 0, st, a);
            else hipLaunchKernelGGL((bwd_dq_kernel<64, 2, MASK, SCORE, true>), dim3(grid_q), dim3(128), 0, st, a);
        } else {
            return FLEXATTN_ERR_UNSUPPORTED;     // this score_mod captures no tensor
        }
    }
    return FLEXATTN_OK;
}

}  // namespace flexattn
