// flexattn_backward: argument validation, the delta pre-pass and dispatch to the compiled variant.
#include "bwd_stored.h"
#include "variants.h"

namespace flexattn {

#define DECL(i) int bwd_launch_##i(const BwdArgs&, int, uint32_t, hipStream_t);
FLEXATTN_VARIANT_INDICES(DECL)
#undef DECL
typedef int (*BwdLauncher)(const BwdArgs&, int, uint32_t, hipStream_t);
#define ENTRY(i) bwd_launch_##i,
static const BwdLauncher kBwdLaunchers[kNumVariants] = {FLEXATTN_VARIANT_INDICES(ENTRY)};
#undef ENTRY
int check_tensor(const flexattn_tensor* t);
int check_extent(const flexattn_tensor* t, int len, int D);
int check_problem(const flexattn_dims* d, const flexattn_blockmask* bm);

}  // namespace flexattn

using namespace flexattn;

namespace {
size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }
size_t row_scalar_bytes(const flexattn_dims* d) { return (size_t)2 * d->B * d->Hq * d->q_len * sizeof(float); }
// Room, behind what a workspace must hold, for the sums of divided groups: as many parts as columns that all rows list would be given.
size_t kv_part_bytes(const flexattn_dims* d) {
    if (d->Hkv <= 0 || d->kv_len <= 0 || d->Hq % d->Hkv || (d->D != 64 && d->D != 128)) return 0;
    const size_t parts = (size_t)kv_head_parts((int64_t)d->B * d->Hkv, d->Hq / d->Hkv, d->kv_len, d->D, d->q_len, [](int) { return true; });
    return parts < 2 ? 0 : parts * 2 * d->B * d->Hkv * d->kv_len * d->D * sizeof(float);
}
}  // namespace

extern "C" size_t flexattn_backward_workspace_bytes(const flexattn_dims* d) {
    if (!d || d->B <= 0 || d->Hq <= 0 || d->q_len <= 0) return 0;
    const size_t parts = kv_part_bytes(d);
    return parts ? align256(row_scalar_bytes(d)) + parts : row_scalar_bytes(d);
}

namespace {
// Workspace of the backward that keeps dS in memory: the row scalars of the recomputing backward,
// then the slot numbering (column bases, grid), then the dS blocks, which end at `end`.  (What is optional, the sums of divided groups, comes
// behind them: stages that are called with workspaces of different sizes find one another's blocks.)
struct StoredLayout {
    size_t colbase_off, grid_off, store_off, end;
    int64_t cap;        // slots per head
    int lines, planes;
};
bool stored_layout(const flexattn_dims* d, const flexattn_blockmask* bm, int64_t n_blocks, StoredLayout* out) {
    if (!d || !bm || d->B <= 0 || d->Hq <= 0 || d->q_len <= 0 || d->kv_len <= 0 || n_blocks < 0) return false;
    if (bm->Bq <= 0 || bm->Bk <= 0 || bm->Bm <= 0 || bm->Hm <= 0) return false;
    const int64_t NR = (d->q_len + bm->Bq - 1) / bm->Bq, NC = (d->kv_len + bm->Bk - 1) / bm->Bk;
    const int64_t planes = (int64_t)bm->Bm * bm->Hm, lines = planes * NC;
    const int64_t cap = n_blocks > 0 ? n_blocks : 1;    // (times Bk / 64 tiles and Bq / 64 steps it must fit an int)
    if (lines >= (1ll << 30) || planes * NR * NC >= (1ll << 40) || cap * 4 >= (1ll << 31)) return false;
    const int64_t reps = (int64_t)(bm->Bm > 1 ? 1 : d->B) * (bm->Hm > 1 ? 1 : d->Hq);
    out->cap = cap;
    out->lines = (int)lines;
    out->planes = (int)planes;
    out->colbase_off = align256(row_scalar_bytes(d));
    out->grid_off = out->colbase_off + align256((size_t)(lines + 1) * sizeof(int32_t));
    out->store_off = out->grid_off + align256((size_t)(planes * NR * NC) * sizeof(int32_t));
    out->end = out->store_off + (size_t)reps * (size_t)cap * (size_t)bm->Bq * (size_t)bm->Bk * sizeof(bf16);
    return true;
}

// Whether two tensors may share memory (the spans of their rows meet).
struct Span {
    uintptr_t lo, hi;
    Span(const flexattn_tensor* t, int B, int H, int len, int D)
        : lo((uintptr_t)t->ptr), hi(lo + 2 * (uintptr_t)((B - 1) * t->stride_b + (H - 1) * t->stride_h + (len - 1) * t->stride_s + D)) {}
    Span(const float* p, size_t n) : lo((uintptr_t)p), hi(lo + 4 * n) {}
    bool meets(const Span& o) const { return lo < o.hi && o.lo < hi; }
};

bool same_rows(const flexattn_tensor* a, const flexattn_tensor* b) {
    return a->ptr == b->ptr && a->stride_b == b->stride_b && a->stride_h == b->stride_h && a->stride_s == b->stride_s;
}

// How the dQ kernel that reads dS back shares its K tiles (bwd_stored.h), D = 128, Bq = 128: among two heads of a group, else among two rows
// of blocks; on long rows, with enough workgroups left.  us of the whole backward, a head's row of blocks by itself -> shared: two heads, S x
// query / KV heads, causal with soft-cap, 8192 x 64 / 32 3572 -> 3502, 8192 x 16 / 8 919 -> 897, no mask, 16384 x 4 / 2 1565 -> 1518, but 2048 x 32 / 8
// 185 -> 195, 1000 x 16 / 4 83 -> 93; two rows, causal with soft-cap, 8192 x 64 3685 -> 3602, 4096 x 32 527 -> 518, prefix, 4000 x 32 491 -> 484, but 2048
// x 128 608 -> 619, no mask, 1500 x 96 412 -> 415, causal, 8192 x 8 466 -> 479, window of 1024, 8192 x 32 550 -> 561.
StoredShare stored_share(const flexattn_dims* d, const flexattn_blockmask* bm, uint32_t mask_id, const flexattn_mod_params& p) {
    if (d->D != 128 || bm->Bq != 128 || mask_uses(mask_id, FLEXATTN_M_NEIGHBORHOOD)) return StoredShare::kNone;
    if (line_shape(mask_id, p, d->q_len, d->kv_len).sure < 4000) return StoredShare::kNone;
    const int64_t sets = (int64_t)d->B * d->Hq * ((d->q_len + 127) / 128) / 2;
    if (d->Hq / d->Hkv % 2 == 0 && bm->Hm == 1) return sets >= 256 ? StoredShare::kHeads : StoredShare::kNone;
    return sets >= 512 && !mask_uses(mask_id, FLEXATTN_M_SLIDING_WINDOW) ? StoredShare::kRows : StoredShare::kNone;
}

// Whether dS through memory is faster than recomputing it for dQ.  Memory costs 4 bytes a score and three more small launches
// (about 8 us); recomputing costs two matrix products and the score_mod, which at D = 64 is the less, but for a soft-cap on
// long rows.  us of the whole backward, dS in memory -> recomputed:
//   D = 64     causal, S = 1024, 64 x 16 heads 916 -> 736; S = 4096, 64 heads 630 -> 539; S = 256, 2 heads 22.5 -> 14.1; no mask, S = 2048,
//              8 x 16 593 -> 477; window of 1024, S = 5000, 4 x 16 / 2 388 -> 321; documents with ALiBi, S = 16384 461 -> 394;
//   soft-cap   8 heads, S = 1024 33.0 -> 22.9, 2048 55.8 -> 44.0; 32 x 16, S = 512 175 -> 160; 4 heads, S = 8192 207 -> 198; but 32, S = 2048 124 ->
//              142, 32, S = 8192 1244 -> 1281; window of 1024, S = 5000, 4 x 16 / 4 430 -> 414;
//   canvases   (whose blocks are mostly hidden parts, which dS in memory leaves out at the granularity of a wave's 32 x 32)
//              64 x 64 pixels, K = 13, 4 heads 40.7 -> 32.5; 128 x 128, 2 heads 49.7 -> 51.0, row-major 87 -> 102, 8 heads 119 -> 115,
//              row-major 223 -> 240, 64 heads 990 -> 881 (812 since dK/dV leaves hidden steps out); 100 x 100, row-major, K = 9, 2 x 16 / 4 386
//              -> 370;
//   D = 128    only small launches: causal, 16 heads, S = 512 32.7 -> 25.0, 8 x 16 84.7 -> 77.7; 2 heads, S = 4096 109 -> 90; 8 heads, S = 2048
//              75.5 -> 66.8; window of 512, 32 heads, S = 2048 99.4 -> 95.8; 4 heads, S = 8192 290 -> 338; soft-cap, 8 heads, S = 1024 43.8 -> 38.1,
//              32 / 8 heads 87.5 -> 92.6; 32 x 32 pixels, 8 heads 43.3 -> 35.1, 64 x 64, 4 heads 51.9 -> 54.9.
// and through memory where dQ recomputed is not split among the waves of a workgroup (dq_split_waves): D = 64, documents with a relative bias and a soft-cap, S = 1100,
// 16 heads 39.3 -> 48.5, 64 x 64 pixels, K = 27, 16 heads 129 -> 148 (4 heads 86 -> 75); D = 128, documents, S = 1100, 8 heads 36.0 -> 39.5, no mask 54.6 -> 58.1
// (4 heads 46 -> 37), a window of 300 or prefix of 100 with a relative bias, S = 1100, 8 heads 44 -> 50, 64 heads 118 -> 123.
// The lines go by slices of 32 query rows and by the longest row (line_shape).
bool stored_pays(const flexattn_dims* d, uint32_t mask_id, uint32_t score_id, const flexattn_mod_params& p) {
    const int64_t slices = (int64_t)d->B * d->Hq * ((d->q_len + 31) / 32);
    const LineShape rows = line_shape(mask_id, p, d->q_len, d->kv_len);
    const bool cap = score_id & FLEXATTN_SCORE_SOFTCAP, rel = score_id & FLEXATTN_SCORE_REL_BIAS;
    if (mask_uses(mask_id, FLEXATTN_M_NEIGHBORHOOD)) {
        if (d->D == 128) return slices > 256;
        return (d->q_len > 4096 && slices < 8192) || (p.na_kernel >= 21 && slices > 1024);
    }
    if (d->D == 64) return cap && (rel ? slices > 512 : slices > 1024 && rows.longest >= (rows.uneven ? 1024 : 1536));
    if (cap || rel) return slices > 256;
    if (slices <= 512) return slices > 256 && !rows.sure_uneven && !mask_uses(mask_id, FLEXATTN_M_SLIDING_WINDOW);
    return rows.longest > 1024 || slices >= 4096;
}

// ds_blocks < 0: dQ recomputes S and dP; otherwise dS goes through memory, but in whole calls for which stored_pays says no.
int backward_impl(const flexattn_dims* dims, const flexattn_tensor* Q,
                                        const flexattn_tensor* K, const flexattn_tensor* V, const flexattn_tensor* O,
                                        const flexattn_tensor* dO, const float* LSE, uint32_t score_id,
                                        uint32_t mask_id, const flexattn_mod_params* params,
                                        const flexattn_blockmask* bm, float scale, const flexattn_tensor* dQ,
                                        const flexattn_tensor* dK, const flexattn_tensor* dV, void* ws,
                                        size_t ws_bytes, void* stream, uint32_t stages, int64_t ds_blocks) {
    int rc = check_problem(dims, bm);
    if (rc != FLEXATTN_OK) return rc;
    if (stages == 0 || (stages & ~FLEXATTN_BWD_ALL)) return FLEXATTN_ERR_INVALID_ARG;
    const flexattn_tensor* ts[] = {Q, K, V, O, dO};
    for (const flexattn_tensor* t : ts)
        if ((rc = check_tensor(t)) != FLEXATTN_OK) return rc;
    if ((stages & FLEXATTN_BWD_DQ) && (rc = check_tensor(dQ)) != FLEXATTN_OK) return rc;
    if ((stages & FLEXATTN_BWD_DKDV) && ((rc = check_tensor(dK)) != FLEXATTN_OK || (rc = check_tensor(dV)) != FLEXATTN_OK))
        return rc;
    if ((rc = check_extent(Q, dims->q_len, dims->D)) != FLEXATTN_OK) return rc;
    if ((rc = check_extent(dO, dims->q_len, dims->D)) != FLEXATTN_OK) return rc;
    if ((rc = check_extent(K, dims->kv_len, dims->D)) != FLEXATTN_OK) return rc;
    if ((rc = check_extent(V, dims->kv_len, dims->D)) != FLEXATTN_OK) return rc;
    static const flexattn_tensor kNoTensor = {nullptr, 0, 0, 0};
    if (!(stages & FLEXATTN_BWD_DQ)) dQ = &kNoTensor;
    if (!(stages & FLEXATTN_BWD_DKDV)) dK = dV = &kNoTensor;
    if (!LSE || !ws || !(scale > 0.0f) || ((uintptr_t)ws & 15)) return FLEXATTN_ERR_INVALID_ARG;
    if (!bm->q_num_blocks || !bm->q_indices || !bm->full_q_num_blocks || !bm->full_q_indices)
        return FLEXATTN_ERR_INVALID_ARG;
    if ((rc = check_mod_params(mask_id, score_id, params)) != FLEXATTN_OK) return rc;
    if ((rc = check_canvas(mask_id, params, dims->q_len, dims->kv_len)) != FLEXATTN_OK) return rc;
    const int vi = variant_of(mask_id, score_id, params, true, dims->D);
    if (vi < 0) return FLEXATTN_ERR_UNSUPPORTED;
    bool stored = ds_blocks >= 0;
    StoredLayout lay = {};
    if (stored) {
        if (!stored_layout(dims, bm, ds_blocks, &lay)) return FLEXATTN_ERR_INVALID_ARG;
        if (((uintptr_t)ws & 255)) return FLEXATTN_ERR_INVALID_ARG;
    }
    const size_t needed = stored ? lay.end : row_scalar_bytes(dims), part_off = align256(needed), part_bytes = kv_part_bytes(dims);
    if (ws_bytes < needed) return FLEXATTN_ERR_WORKSPACE;

    BwdArgs a = {};
    a.Q = (const bf16*)Q->ptr; a.K = (const bf16*)K->ptr; a.V = (const bf16*)V->ptr;
    a.O = (const bf16*)O->ptr; a.dO = (const bf16*)dO->ptr; a.LSE = LSE;
    a.dQ = (bf16*)dQ->ptr; a.dK = (bf16*)dK->ptr; a.dV = (bf16*)dV->ptr;
    const size_t rows = (size_t)dims->B * dims->Hq * dims->q_len;
    a.delta = (float*)ws; a.lse2 = (float*)ws + rows;
    a.q_sb = Q->stride_b; a.q_sh = Q->stride_h; a.q_ss = Q->stride_s;
    a.k_sb = K->stride_b; a.k_sh = K->stride_h; a.k_ss = K->stride_s;
    a.v_sb = V->stride_b; a.v_sh = V->stride_h; a.v_ss = V->stride_s;
    a.o_sb = O->stride_b; a.o_sh = O->stride_h; a.o_ss = O->stride_s;
    a.do_sb = dO->stride_b; a.do_sh = dO->stride_h; a.do_ss = dO->stride_s;
    a.dq_sb = dQ->stride_b; a.dq_sh = dQ->stride_h; a.dq_ss = dQ->stride_s;
    a.dk_sb = dK->stride_b; a.dk_sh = dK->stride_h; a.dk_ss = dK->stride_s;
    a.dv_sb = dV->stride_b; a.dv_sh = dV->stride_h; a.dv_ss = dV->stride_s;
    a.B = dims->B; a.Hq = dims->Hq; a.Hkv = dims->Hkv; a.G = dims->Hq / dims->Hkv;
    a.q_len = dims->q_len; a.kv_len = dims->kv_len;
    a.NR = (dims->q_len + bm->Bq - 1) / bm->Bq; a.NC = (dims->kv_len + bm->Bk - 1) / bm->Bk;
    a.Bq = bm->Bq; a.Bk = bm->Bk;
    a.bm_Bm = bm->Bm; a.bm_Hm = bm->Hm;
    a.kv_num = bm->kv_num_blocks; a.kv_idx = bm->kv_indices;
    a.full_kv_num = bm->full_kv_num_blocks; a.full_kv_idx = bm->full_kv_indices;
    a.q_num = bm->q_num_blocks; a.q_idx = bm->q_indices;
    a.full_q_num = bm->full_q_num_blocks; a.full_q_idx = bm->full_q_indices;
    a.kv_order = bm->kv_order; a.q_order = bm->q_order;
    a.scale = scale;
    if (params) a.p = *params;
    if (part_bytes && ws_bytes >= part_off + part_bytes) a.kv_part = (float*)((char*)ws + part_off);     // (a workspace without room for them will do)
    if (stages & FLEXATTN_BWD_DQ) {
        // outputs written over inputs: dQ over Q or dO waits for dK/dV, over O or LSE for the pass that makes the row scalars of
        // them (but over O row for row: a wave reads its rows of O before it writes them); with dS in memory it may also take V's place
        const Span dq(dQ, dims->B, dims->Hq, dims->q_len, dims->D), lse(LSE, rows);
        auto other_rows = [&](const flexattn_tensor* t) {
            return dq.meets(Span(t, dims->B, dims->Hq, dims->q_len, dims->D)) && !same_rows(t, dQ);
        };
        a.dq_last = dq.meets(Span(Q, dims->B, dims->Hq, dims->q_len, dims->D)) || dq.meets(Span(dO, dims->B, dims->Hq, dims->q_len, dims->D)) ||
                    other_rows(O) || dq.meets(lse);
        // A whole call may recompute dS, from Q, dO and V, unless dQ or what comes before it may have taken their place: a row
        // of Q or dO may be dQ's own, which its wave has read, but no other, and V must be there.  (A DQ stage by itself finds
        // dS written, and the tensors perhaps gone.)
        const Span v(V, dims->B, dims->Hkv, dims->kv_len, dims->D);
        auto over_v = [&](const flexattn_tensor* t) { return v.meets(Span(t, dims->B, dims->Hkv, dims->kv_len, dims->D)); };
        if (stored && stages == FLEXATTN_BWD_ALL && !dq.meets(v) && !other_rows(Q) && !other_rows(dO) && !(a.dq_last && (over_v(dK) || over_v(dV))))
            stored = stored_pays(dims, mask_id, score_id, a.p);
    }

    hipStream_t st = (hipStream_t)stream;
    if (stored) {
        int32_t* colbase = (int32_t*)((char*)ws + lay.colbase_off);
        int32_t* grid = (int32_t*)((char*)ws + lay.grid_off);
        a.ds_colbase = colbase;
        a.ds_grid = grid;
        a.ds_store = (bf16*)((char*)ws + lay.store_off);
        a.ds_blocks = lay.cap;
        if (stages & FLEXATTN_BWD_DELTA) {      // the block numbering belongs to the pre-pass
            hipLaunchKernelGGL(bwd_slots_scan_kernel, dim3(1), dim3(1024), 0, st, a.q_num, a.full_q_num, lay.lines,
                               a.NR, colbase);
            hipLaunchKernelGGL(bwd_slots_fill_kernel, dim3((unsigned)lay.lines), dim3(256), 0, st, a.q_num, a.q_idx,
                               a.full_q_num, a.full_q_idx, a.NR, a.NC, colbase, grid);
        }
        // delta and dK/dV (which writes dS) from the compiled variant; dQ from what it wrote
        if (stages & (FLEXATTN_BWD_DELTA | FLEXATTN_BWD_DKDV)) {
            rc = kBwdLaunchers[vi](a, dims->D, stages & (FLEXATTN_BWD_DELTA | FLEXATTN_BWD_DKDV), st);
            if (rc != FLEXATTN_OK) return rc;
        }
        if (stages & FLEXATTN_BWD_DQ) {
            const float qscale = scale * ((score_id & FLEXATTN_SCORE_SOFTCAP) ? 4.0f : 1.0f);   // ScoreMod::grad_scale()
            if (mask_uses(mask_id, FLEXATTN_M_NEIGHBORHOOD)) launch_bwd_stored_dq<true>(a, dims->D, qscale, StoredShare::kNone, false, false, st);
            else launch_bwd_stored_dq<false>(a, dims->D, qscale, stored_share(dims, bm, mask_id, a.p), line_shape(mask_id, a.p, dims->q_len, dims->kv_len).uneven,
                                             mask_uses(mask_id, FLEXATTN_M_DOCUMENT), st);
        }
    } else {
        rc = kBwdLaunchers[vi](a, dims->D, stages, st);     // the delta pre-pass depends on the score_mod too
        if (rc != FLEXATTN_OK) return rc;
    }
    FLEXATTN_HIP_TRY(hipGetLastError());
    return FLEXATTN_OK;
}
}  // namespace

extern "C" int flexattn_backward_stages(const flexattn_dims* dims, const flexattn_tensor* Q,
                                        const flexattn_tensor* K, const flexattn_tensor* V, const flexattn_tensor* O,
                                        const flexattn_tensor* dO, const float* LSE, uint32_t score_id,
                                        uint32_t mask_id, const flexattn_mod_params* params,
                                        const flexattn_blockmask* bm, float scale, const flexattn_tensor* dQ,
                                        const flexattn_tensor* dK, const flexattn_tensor* dV, void* ws,
                                        size_t ws_bytes, void* stream, uint32_t stages) {
    return backward_impl(dims, Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV, ws, ws_bytes,
                         stream, stages, -1);
}

extern "C" int flexattn_backward(const flexattn_dims* dims, const flexattn_tensor* Q, const flexattn_tensor* K,
                                 const flexattn_tensor* V, const flexattn_tensor* O, const flexattn_tensor* dO,
                                 const float* LSE, uint32_t score_id, uint32_t mask_id,
                                 const flexattn_mod_params* params, const flexattn_blockmask* bm, float scale,
                                 const flexattn_tensor* dQ, const flexattn_tensor* dK, const flexattn_tensor* dV,
                                 void* ws, size_t ws_bytes, void* stream) {
    return flexattn_backward_stages(dims, Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV, ws,
                                    ws_bytes, stream, FLEXATTN_BWD_ALL);
}

extern "C" size_t flexattn_backward_stored_workspace_bytes(const flexattn_dims* dims, const flexattn_blockmask* bm,
                                                           int64_t n_blocks) {
    StoredLayout lay;
    if (!stored_layout(dims, bm, n_blocks, &lay)) return 0;
    const size_t parts = kv_part_bytes(dims);
    return parts ? align256(lay.end) + parts : lay.end;
}

extern "C" int flexattn_backward_stored(const flexattn_dims* dims, const flexattn_tensor* Q, const flexattn_tensor* K,
                                        const flexattn_tensor* V, const flexattn_tensor* O, const flexattn_tensor* dO,
                                        const float* LSE, uint32_t score_id, uint32_t mask_id,
                                        const flexattn_mod_params* params, const flexattn_blockmask* bm, float scale,
                                        const flexattn_tensor* dQ, const flexattn_tensor* dK, const flexattn_tensor* dV,
                                        int64_t n_blocks, void* ws, size_t ws_bytes, void* stream, uint32_t stages) {
    if (n_blocks < 0) return FLEXATTN_ERR_INVALID_ARG;
    return backward_impl(dims, Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV, ws, ws_bytes,
                         stream, stages, n_blocks);
}

// ---- gradients of captured tensors -----------------------------------------------------------
namespace {
// Sum of the per-workgroup partials over batch and rows of blocks, in a fixed order, times `factor`:
// out[hq, i] = factor * sum_{b, row} part[((b * Hq + hq) * NR + row) * width + i].
// 32 entries side by side, the rows of blocks of an entry dealt to 32 threads whose sums are added in order; a thread
// takes its rows of every batch entry, so with fewer than 32 rows some have none.  Bound by the latency of one thread's
// loads.  (One thread per entry walked all
// partials: 196 us for 8192 entries of 512 partials, a fifth of the kernel that makes them on short
// sequences; 10 us since.)
__global__ __launch_bounds__(1024) void captured_reduce_kernel(const float* __restrict__ part, int B, int Hq, int NR,
                                                               int width, float factor, float* __restrict__ out) {
    __shared__ double s_sum[32][32];
    const int e = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int idx = blockIdx.x * 32 + e;
    double sum = 0.0;
    if (idx < Hq * width) {
        const int hq = idx / width, i = idx - hq * width;
        for (int b = 0; b < B; ++b) {
            const float* src = part + ((int64_t)b * Hq + hq) * NR * width + i;
            for (int row = g; row < NR; row += 32) sum += (double)src[(int64_t)row * width];
        }
    }
    s_sum[g][e] = sum;
    __syncthreads();
    if (g != 0 || idx >= Hq * width) return;
    for (int k = 1; k < 32; ++k) sum += s_sum[k][e];
    out[idx] = (float)(sum * (double)factor);
}

size_t captured_slots(const flexattn_dims* d, const flexattn_blockmask* bm) {
    return (size_t)d->B * d->Hq * ((d->q_len + bm->Bq - 1) / bm->Bq);
}
}  // namespace

extern "C" size_t flexattn_backward_captured_workspace_bytes(const flexattn_dims* d, const flexattn_blockmask* bm,
                                                             uint32_t score_id, const flexattn_mod_params* params) {
    if (!d || !bm || d->B <= 0 || d->Hq <= 0 || d->q_len <= 0 || bm->Bq <= 0) return 0;
    size_t n = 0;
    if (score_id & FLEXATTN_SCORE_ALIBI) n += captured_slots(d, bm);
    if ((score_id & FLEXATTN_SCORE_REL_BIAS) && params && params->rel_len > 0)
        n += captured_slots(d, bm) * (size_t)params->rel_len;
    return n * sizeof(float);
}

extern "C" int flexattn_backward_captured(const flexattn_dims* dims, const flexattn_tensor* Q,
                                          const flexattn_tensor* K, const flexattn_tensor* V, const flexattn_tensor* O,
                                          const flexattn_tensor* dO, const float* LSE, uint32_t score_id,
                                          uint32_t mask_id, const flexattn_mod_params* params,
                                          const flexattn_blockmask* bm, float scale, float* d_alibi_bias,
                                          float* d_rel_bias, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_problem(dims, bm);
    if (rc != FLEXATTN_OK) return rc;
    const flexattn_tensor* ts[] = {Q, K, V, O, dO};
    for (const flexattn_tensor* t : ts)
        if ((rc = check_tensor(t)) != FLEXATTN_OK) return rc;
    if ((rc = check_extent(K, dims->kv_len, dims->D)) != FLEXATTN_OK) return rc;
    if ((rc = check_extent(V, dims->kv_len, dims->D)) != FLEXATTN_OK) return rc;
    if (!LSE || !ws || !(scale > 0.0f) || ((uintptr_t)ws & 15)) return FLEXATTN_ERR_INVALID_ARG;
    if ((rc = check_mod_params(mask_id, score_id, params)) != FLEXATTN_OK) return rc;
    if ((rc = check_canvas(mask_id, params, dims->q_len, dims->kv_len)) != FLEXATTN_OK) return rc;
    const bool alibi = score_id & FLEXATTN_SCORE_ALIBI, rel = score_id & FLEXATTN_SCORE_REL_BIAS;
    if (!alibi && !rel) return FLEXATTN_ERR_UNSUPPORTED;               // nothing is captured
    if ((alibi && !d_alibi_bias) || (rel && !d_rel_bias)) return FLEXATTN_ERR_INVALID_ARG;
    const int vi = variant_of(mask_id, score_id, params, true, dims->D);
    if (vi < 0) return FLEXATTN_ERR_UNSUPPORTED;
    if (ws_bytes < flexattn_backward_captured_workspace_bytes(dims, bm, score_id, params)) return FLEXATTN_ERR_WORKSPACE;

    BwdArgs a = {};
    a.Q = (const bf16*)Q->ptr; a.K = (const bf16*)K->ptr; a.V = (const bf16*)V->ptr;
    a.O = (const bf16*)O->ptr; a.dO = (const bf16*)dO->ptr; a.LSE = LSE;
    const size_t slots = captured_slots(dims, bm);
    a.cap_alibi = (float*)ws;
    a.cap_rel = a.cap_alibi + (alibi ? slots : 0);
    a.q_sb = Q->stride_b; a.q_sh = Q->stride_h; a.q_ss = Q->stride_s;
    a.k_sb = K->stride_b; a.k_sh = K->stride_h; a.k_ss = K->stride_s;
    a.v_sb = V->stride_b; a.v_sh = V->stride_h; a.v_ss = V->stride_s;
    a.o_sb = O->stride_b; a.o_sh = O->stride_h; a.o_ss = O->stride_s;
    a.do_sb = dO->stride_b; a.do_sh = dO->stride_h; a.do_ss = dO->stride_s;
    a.B = dims->B; a.Hq = dims->Hq; a.Hkv = dims->Hkv; a.G = dims->Hq / dims->Hkv;
    a.q_len = dims->q_len; a.kv_len = dims->kv_len;
    a.NR = (dims->q_len + bm->Bq - 1) / bm->Bq; a.NC = (dims->kv_len + bm->Bk - 1) / bm->Bk;
    a.Bq = bm->Bq; a.Bk = bm->Bk;
    a.bm_Bm = bm->Bm; a.bm_Hm = bm->Hm;
    a.kv_num = bm->kv_num_blocks; a.kv_idx = bm->kv_indices;
    a.full_kv_num = bm->full_kv_num_blocks; a.full_kv_idx = bm->full_kv_indices;
    a.scale = scale;
    a.p = *params;

    hipStream_t st = (hipStream_t)stream;
    rc = kBwdLaunchers[vi](a, dims->D, kBwdStageCaptured, st);
    if (rc != FLEXATTN_OK) return rc;
    // the kernels' dS lacks the constant factor of the score_mod's derivative
    const float factor = (score_id & FLEXATTN_SCORE_SOFTCAP) ? 4.0f : 1.0f;
    if (alibi)
        hipLaunchKernelGGL(captured_reduce_kernel, dim3((unsigned)((a.Hq + 31) / 32)), dim3(1024), 0, st, a.cap_alibi,
                           a.B, a.Hq, a.NR, 1, factor, d_alibi_bias);
    if (rel)
        hipLaunchKernelGGL(captured_reduce_kernel, dim3((unsigned)((a.Hq * a.p.rel_len + 31) / 32)), dim3(1024), 0, st,
                           a.cap_rel, a.B, a.Hq, a.NR, a.p.rel_len, factor, d_rel_bias);
    FLEXATTN_HIP_TRY(hipGetLastError());
    return FLEXATTN_OK;
}
