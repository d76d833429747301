// C ABI of the hybrid delta attention library: argument checks, workspace carving, launches.
#include <math.h>
#include <mutex>
#include <new>
#include <stdlib.h>
#include <string.h>

#include "../../include/delta_attn.h"
#include "cache.hpp"
#include "common.hpp"
#include "kernels.hpp"

using namespace da;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline size_t elt_size(int dtype) { return dtype == DA_F32 ? 4 : 2; }

struct WsLayout {
    size_t khat, scan, scan_total, queue, copies, counts, total;
};

// what prefill_mfma_supported reads, for a prefill of p's rows behind `cached` rows
PrefillArgs shape_args(const da_prefill_params *p, int64_t cached) {
    PrefillArgs a = {};
    a.dtype = p->dtype;
    a.B = p->batch;
    a.Hq = p->n_q_heads;
    a.Hkv = p->n_kv_heads;
    a.d = p->head_dim;
    a.n = (int)cached + p->seq_len;
    return a;
}

da_status check_params(const da_prefill_params *p) {
    if (!p) return DA_ERR_INVALID_ARG;
    if (p->batch < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1 || p->head_dim < 1 || p->seq_len < 1)
        return DA_ERR_INVALID_ARG;
    if (p->n_q_heads % p->n_kv_heads != 0) return DA_ERR_INVALID_ARG;
    if (p->window < 1) return DA_ERR_INVALID_ARG;
    if (!(p->theta >= 0.f)) return DA_ERR_INVALID_ARG;          // also rejects NaN
    if (!(p->scale >= 0.f) || isinf(p->scale)) return DA_ERR_INVALID_ARG;
    if (p->head_dim % 32 != 0 || p->head_dim > 256) return DA_ERR_UNSUPPORTED;
    if (p->dtype != DA_F32 && p->dtype != DA_BF16) return DA_ERR_UNSUPPORTED;
    if (p->score_mode != DA_SCORE_GATHER && p->score_mode != DA_SCORE_REBASE) return DA_ERR_UNSUPPORTED;
    if (p->window_mode != DA_WINDOW_BLOCK && p->window_mode != DA_WINDOW_SLIDING) return DA_ERR_UNSUPPORTED;
    if ((int64_t)p->batch * p->n_q_heads > 65535 * 64) return DA_ERR_UNSUPPORTED;
    return DA_OK;
}

WsLayout layout(const da_prefill_params *p) {
    const size_t units = (size_t)p->batch * p->n_kv_heads;
    const size_t rows = units * (size_t)p->seq_len;
    WsLayout w;
    size_t off = 0;
    w.khat = off;
    off += align_up(rows * p->head_dim * elt_size(p->dtype));
    w.scan = off;
    off += align_up(delta_scan_scratch_bytes(p->dtype, (int)units, p->seq_len, p->head_dim));
    w.scan_total = off;
    // The attention launch's counters, then room for aligned copies of K and V (4 bytes per key element, launch_copy_aligned).
    // The size is the 8 bytes per key element and 4 per row that it has been since surviving entries were written out here:
    // callers size their buffers by it, and what the built-in scratch is too small for does not change.
    w.queue = off;
    w.copies = off + kPrefillQueueBytes;
    static_assert(kPrefillQueueBytes + 64 * 4 <= 64 * 8 + kAlign && kPrefillQueueBytes % 16 == 0, "one row of head_dim 64 makes room for them");
    off += align_up(rows * p->head_dim * 8) + align_up(rows * sizeof(uint32_t));
    w.total = off;
    w.counts = p->seq_len >= 64 ? off - align_up(units * (p->head_dim / 8) * sizeof(uint32_t)) : 0;   // (0: no room)
    // (64 rows leave 256 bytes per unit and channel behind the copies, less the counters)
    return w;
}

inline float score_scale(float scale, int d) { return resolved_scale(scale, d); }

da_status prefill_checked(const da_prefill_params *p, const WsLayout &w, const void *Q, const void *K, const void *V,
                          void *O, uint32_t *mask_bits, uint64_t *nnz, da_cache *cache, void *workspace, hipStream_t s);

// ---- built-in scratch of delta_attn_prefill_noalloc.  One copy per GPU, held from the time the library is loaded
// on that GPU until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress, not a
// device address: its address on a device is looked up once per device, with that device current, and only that
// pointer is ever handed to kernels.
constexpr size_t kScratchBytes = DA_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

void *scratch_of_current_device() {
    static std::mutex mu;
    static void *ptr_of[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        set_last_error("delta_attn_prefill_noalloc: no current device, or a device ordinal above 63");
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            set_last_error("delta_attn_prefill_noalloc: hipGetSymbolAddress: %s", hipGetErrorName(e));
            (void)hipGetLastError();
            return nullptr;
        }
        ptr_of[dev] = ptr;
    }
    return ptr_of[dev];
}

// the kernels read the workspace with 16-byte loads; regions are carved at multiples of 256
inline bool ws_aligned(const void *ws) { return ((uintptr_t)ws & (kAlign - 1)) == 0; }

}  // namespace

extern "C" {

const char *delta_attn_last_error(void) { return last_error_text(); }

void delta_attn_stage_timing_enable(int32_t on) { timing_enable(on != 0); }

int32_t delta_attn_stage_timing_read(double *ms_per_stage, int32_t *calls_per_stage) {
    if (!ms_per_stage || !calls_per_stage) return -1;
    return timing_collect(ms_per_stage, calls_per_stage);
}

const char *delta_attn_version(void) { return "delta_attn 0.1 (gfx950)"; }

const char *delta_attn_status_string(da_status s) {
    switch (s) {
        case DA_OK: return "ok";
        case DA_ERR_INVALID_ARG: return "invalid argument";
        case DA_ERR_UNSUPPORTED: return "unsupported configuration";
        case DA_ERR_WORKSPACE: return "workspace missing or too small";
        case DA_ERR_STATE: return "cache state does not allow this call";
        case DA_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

int32_t delta_attn_window_from_gamma(int32_t n, double gamma, int32_t w_max) {
    if (n < 1 || w_max < 1 || !(gamma > 0.0)) return 1;
    double w = floor(gamma * (double)n);
    if (w > (double)w_max) w = (double)w_max;
    if (w < 1.0) w = 1.0;
    return (int32_t)w;
}

size_t delta_attn_prefill_workspace_bytes(const da_prefill_params *p) {
    if (check_params(p) != DA_OK) return 0;
    return layout(p).total;
}

size_t delta_attn_delta_scan_workspace_bytes(const da_prefill_params *p) {
    if (check_params(p) != DA_OK) return 0;
    const WsLayout w = layout(p);
    return w.scan_total;   // reference keys + per-chunk states: the first two regions of the prefill layout
}

da_status delta_attn_delta_scan(const da_prefill_params *p, const void *K, uint32_t *mask_bits, uint64_t *nnz,
                                void *k_hat, void *workspace, size_t workspace_bytes, void *hip_stream) {
    da_status st = check_params(p);
    if (st != DA_OK) return st;
    if (!K || !mask_bits || !nnz) return DA_ERR_INVALID_ARG;
    const WsLayout w = layout(p);
    if (!workspace || workspace_bytes < w.scan_total || !ws_aligned(workspace)) return DA_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;
    (void)hipGetLastError();
    // (where one work group per unit does all of it, that is faster than one launch here and another to add up)
    const int units = p->batch * p->n_kv_heads;
    uint32_t *const counts = delta_scan_settles(p->dtype, units, p->seq_len, p->head_dim) ? (uint32_t *)(ws + w.scan) : nullptr;
    launch_nnz_sum(launch_delta_scan(p->dtype, K, k_hat ? k_hat : ws + w.khat, mask_bits, ws + w.scan, counts, nnz, units, p->seq_len,
                                     p->head_dim, p->theta, s, nullptr, nullptr), s);
    return launch_ok("delta_scan") ? DA_OK : DA_ERR_HIP;
}

da_status delta_attn_prefill(const da_prefill_params *p, const void *Q, const void *K, const void *V, void *O,
                             uint32_t *mask_bits, uint64_t *nnz, da_cache *cache, void *workspace,
                             size_t workspace_bytes, void *hip_stream) {
    da_status st = check_params(p);
    if (st != DA_OK) return st;
    if (!Q || !K || !V || !O || !mask_bits || !nnz) return DA_ERR_INVALID_ARG;
    const WsLayout w = layout(p);
    if (!workspace || workspace_bytes < w.total || !ws_aligned(workspace)) return DA_ERR_WORKSPACE;
    if (cache) {
        st = cache_check_for_prefill(cache, p);
        if (st != DA_OK) return st;
    }
    return prefill_checked(p, w, Q, K, V, O, mask_bits, nnz, cache, workspace, (hipStream_t)hip_stream);
}

da_status delta_attn_prefill_noalloc(const da_prefill_params *p, const void *Q, const void *K, const void *V, void *O,
                                     uint32_t *mask_bits, uint64_t *nnz, void *hip_stream) {
    da_status st = check_params(p);
    if (st != DA_OK) return st;
    if (!Q || !K || !V || !O || !mask_bits || !nnz) return DA_ERR_INVALID_ARG;
    const WsLayout w = layout(p);
    if (w.total > kScratchBytes) {
        set_last_error("delta_attn_prefill_noalloc: these params need %zu bytes of scratch, the built-in buffer holds %zu",
                       w.total, kScratchBytes);
        return DA_ERR_WORKSPACE;
    }
    void *ws = scratch_of_current_device();
    if (!ws) return DA_ERR_HIP;
    // Nothing in the buffer has to start at zero: every region is written by the scan before the attention
    // kernel reads it.
    return prefill_checked(p, w, Q, K, V, O, mask_bits, nnz, nullptr, ws, (hipStream_t)hip_stream);
}

}  // extern "C"

namespace {
// the body shared by the two prefill entry points; arguments, workspace and cache have been checked
da_status prefill_checked(const da_prefill_params *p, const WsLayout &w, const void *Q, const void *K, const void *V,
                          void *O, uint32_t *mask_bits, uint64_t *nnz, da_cache *cache, void *workspace,
                          hipStream_t s) {
    char *ws = (char *)workspace;
    void *khat = ws + w.khat;
    const int units = p->batch * p->n_kv_heads;

    (void)hipGetLastError();   // do not inherit an earlier, unrelated error
    PrefillArgs a;
    a.dtype = p->dtype;
    a.d = p->head_dim;
    a.B = p->batch;
    a.Hkv = p->n_kv_heads;
    a.Hq = p->n_q_heads;
    a.n = p->seq_len;
    a.q_off = 0;
    a.nq = p->seq_len;
    a.W = p->window;
    a.scale_log2 = score_scale(p->scale, p->head_dim) * 1.4426950408889634f;
    a.sliding = p->window_mode == DA_WINDOW_SLIDING;
    a.Q = Q;
    a.K = K;
    a.V = V;
    a.Khat = khat;
    a.O = O;
    const bool in_one = prefill_short_supported(a), scans = !in_one && !cache && prefill_generic_scans(a);   // (a cache wants the reference keys)
    if (!in_one && !scans) {
        stage_begin(kStageScan, s);
        a.queue = p->head_dim >= 64 ? (uint32_t *)(ws + w.queue) : nullptr;  // (32: another kernel, and less room)
        a.sum = launch_delta_scan(p->dtype, K, khat, mask_bits, ws + w.scan, w.counts ? (uint32_t *)(ws + w.counts) : nullptr, nnz, units,
                                  p->seq_len, p->head_dim, p->theta, s, nullptr, a.queue);
        stage_end(kStageScan, s);
        if (!launch_ok("delta_scan")) return DA_ERR_HIP;
    }
    stage_begin(kStageAttn, s);
    bool launched = true, filled = false;                        // filled: the attention launch takes the cache's part along
    if (in_one || prefill_mfma_supported(a)) {
        const size_t bytes = (size_t)units * p->seq_len * p->head_dim * 2;
        launch_copy_aligned(a, ws + w.copies, ws + w.copies + bytes, bytes, s);
        if (in_one) {
            launch_prefill_short(a, p->theta, cache ? khat : nullptr, mask_bits, nnz, s);
        } else {
            CacheFill fill = {};
            if (cache && cache->fast) fill = cache_fill(cache, 0, p->seq_len, p->seq_len, a.K, a.V, khat, mask_bits, nullptr, nnz, a.sum);
            filled = fill.items > 0 && prefill_takes_fill(a, fill);
            if (filled) a.sum = NnzSum{};                            // (the hand-off adds up)
            launch_prefill_mfma(a, filled ? &fill : nullptr, s);
        }
    } else {
        const PrefillScan scan = {mask_bits, nnz, p->theta};
        launched = launch_prefill_generic(a, scans ? &scan : nullptr, s);
    }
    stage_end(kStageAttn, s);
    if (!launched) return DA_ERR_UNSUPPORTED;
    if (!launch_ok("prefill attention")) return DA_ERR_HIP;
    if (filled) {
        cache->len = p->seq_len;
    } else if (cache) {
        stage_begin(kStageCacheFill, s);
        cache_fill_from_prefill(cache, p, a.K, a.V, khat, mask_bits, nnz, s);   // (K and V, or their aligned copies)
        stage_end(kStageCacheFill, s);
        if (!launch_ok("cache_fill")) return DA_ERR_HIP;
    }
    return DA_OK;
}

// workspace of delta_attn_prefill_append: what the scan of the new rows needs (the whole-sequence arrays live in the
// cache, see da_prefix)
struct AppendLayout {
    size_t scan, queue, total;
};

AppendLayout append_layout(const da_prefill_params *p) {
    AppendLayout w;
    size_t off = 0;
    w.scan = off;
    off += align_up(delta_scan_scratch_bytes(p->dtype, p->batch * p->n_kv_heads, p->seq_len, p->head_dim));
    w.queue = off;
    off += align_up(kPrefillQueueBytes);
    w.total = off;
    return w;
}

// The cache's whole-sequence arrays (da_prefix), allocated on first use and zero-filled (rows nothing has written yet
// must hold finite numbers: the kernels load whole tiles and discard what lies past the sequence).
da_status ensure_prefix(da_cache *c) {
    if (!c->pf) {
        c->pf = new (std::nothrow) da_prefix();
        if (!c->pf) return DA_ERR_HIP;
        memset(c->pf, 0, sizeof(*c->pf));
    }
    da_prefix *f = c->pf;
    const size_t units = (size_t)c->B * c->Hkv, d = c->d, ld = c->max_seq;
    bool ok = true, fresh = false;
    auto room = [&](void **ptr, size_t bytes) {
        if (!ok || *ptr) return;
        ok = hipMalloc(ptr, bytes) == hipSuccess && hipMemset(*ptr, 0, bytes) == hipSuccess;
        fresh = true;
    };
    room(&f->k, units * ld * d * 2);
    room(&f->h, units * ld * d * 2);
    room(&f->v, units * ld * d * 2);
    room((void **)&f->m, units * ld * (d / 32) * 4);
    // (hipMemset returns before the memory is cleared, on the null stream, which the caller's stream need not wait for)
    if (fresh && ok) ok = hipStreamSynchronize(nullptr) == hipSuccess;
    if (!ok) {
        (void)launch_ok("prefill_append: room for the cached sequence as plain arrays");   // records the error text
        return DA_ERR_HIP;
    }
    return DA_OK;
}

da_status check_append(const da_prefill_params *p, const da_cache *c) {
    da_status st = check_params(p);
    if (st != DA_OK) return st;
    if (!c) return DA_ERR_INVALID_ARG;
    if (!c->fast) return DA_ERR_UNSUPPORTED;                 // only the column-run cache layout can be continued
    if (c->B != p->batch || c->Hq != p->n_q_heads || c->Hkv != p->n_kv_heads || c->d != p->head_dim ||
        c->dtype != p->dtype || c->theta != p->theta)
        return DA_ERR_STATE;
    if (!cache_scale_matches(c, p->scale)) return DA_ERR_STATE;   // one score scale for prefill and decode (Eq. 1)
    if (c->len + p->seq_len > c->max_seq) return DA_ERR_STATE;
    // raw keys of a window come from the ring of the decode_window newest rows; no window reaches back further
    // than the sequence is long
    const int64_t reach = p->window < c->len + p->seq_len ? p->window : c->len + p->seq_len;
    if (c->len > 0 && reach > c->Wd) return DA_ERR_UNSUPPORTED;
    if (!prefill_mfma_supported(shape_args(p, c->len))) return DA_ERR_UNSUPPORTED;   // (more tiles than a grid holds)
    return DA_OK;
}
}  // namespace

extern "C" {

size_t delta_attn_prefill_append_workspace_bytes(const da_prefill_params *p, const da_cache *cache) {
    if (check_append(p, cache) != DA_OK) return 0;
    return append_layout(p).total;
}

da_status delta_attn_prefill_append(const da_prefill_params *p, const void *Q, const void *K, const void *V, void *O,
                                    uint32_t *mask_bits, uint64_t *nnz, da_cache *cache, void *workspace,
                                    size_t workspace_bytes, void *hip_stream) {
    da_status st = check_append(p, cache);
    if (st != DA_OK) return st;
    if (!Q || !K || !V || !O || !mask_bits || !nnz) return DA_ERR_INVALID_ARG;
    const int t0 = (int)cache->len, m = p->seq_len, nk = t0 + m, d = p->head_dim;
    const AppendLayout w = append_layout(p);
    if (!workspace || workspace_bytes < w.total || !ws_aligned(workspace)) return DA_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;
    const int units = p->batch * p->n_kv_heads;
    (void)hipGetLastError();
    st = ensure_prefix(cache);
    if (st != DA_OK) return st;
    da_prefix *f = cache->pf;
    const int ld = cache->max_seq;

    // 1. the cached rows as plain arrays: kept from the previous piece, or (after decode steps or a one-shot prefill
    //    into this cache) unpacked from the cache; the new rows behind them
    const bool kept = f->rows == t0;
    f->rows = -1;                                   // in flux until this call has gone through
    if (!kept) expand_cache_runs(cache, t0, ld, f->k, f->h, f->v, f->m, s);
    // 2. Eq. 2-3 over the new rows, continuing from the cache's reference key (row 0 of an empty cache is the basis); keys, values and
    //    reference keys join the plain arrays
    stage_begin(kStageScan, s);
    auto row_of = [&](void *array) { return (char *)array + (size_t)t0 * d * 2; };
    const RowCopy copy = {{K, V}, {row_of(f->k), row_of(f->v)}, units, m, ld, d / 8};
    // (the scan's counts lie where decode steps leave their partial rows: d + 4 floats per query head at the least)
    const NnzSum sum = launch_delta_scan(p->dtype, K, row_of(f->h), mask_bits, ws + w.scan, (uint32_t *)cache->part, nnz, units, m, d,
                                         p->theta, s, t0 > 0 ? cache->khat : nullptr, (uint32_t *)(ws + w.queue), &copy);
    stage_end(kStageScan, s);
    if (!launch_ok("delta_scan")) return DA_ERR_HIP;
    // 3. attention of the new rows over all nk keys; the new rows join the cache
    PrefillArgs a;
    a.dtype = p->dtype;
    a.B = p->batch;
    a.Hq = p->n_q_heads;
    a.Hkv = p->n_kv_heads;
    a.d = d;
    a.n = nk;
    a.q_off = t0;
    a.nq = m;
    a.ld = ld;
    a.W = p->window;
    a.scale_log2 = score_scale(p->scale, d) * 1.4426950408889634f;
    a.sliding = p->window_mode == DA_WINDOW_SLIDING;
    a.Q = Q;
    a.K = f->k;
    a.V = f->v;
    a.Khat = f->h;
    a.O = O;
    a.queue = (uint32_t *)(ws + w.queue);
    const CacheFill fill = cache_fill(cache, t0, nk, ld, f->k, f->v, f->h, mask_bits, f->m, nnz, sum);
    const bool filled = prefill_takes_fill(a, fill);
    stage_begin(kStageAttn, s);
    launch_prefill_mfma(a, filled ? &fill : nullptr, s);   // (supported: check_append has asked)
    stage_end(kStageAttn, s);
    if (!launch_ok("prefill_append attention")) return DA_ERR_HIP;
    if (!filled) {
        stage_begin(kStageCacheFill, s);
        launch_cache_fill(fill, s);
        stage_end(kStageCacheFill, s);
        if (!launch_ok("cache_fill")) return DA_ERR_HIP;
    }
    cache->len = nk;
    f->rows = nk;
    return DA_OK;
}

da_status delta_attn_sparsity(const uint64_t *nnz_dev, int32_t batch, int32_t n_kv_heads, int64_t rows,
                              int32_t head_dim, int32_t window, void *hip_stream, double *s_m, double *s_c) {
    if (!nnz_dev || !s_m || !s_c || batch < 1 || n_kv_heads < 1 || rows < 1 || head_dim < 1 || window < 1)
        return DA_ERR_INVALID_ARG;
    const size_t units = (size_t)batch * n_kv_heads;
    uint64_t *host = new (std::nothrow) uint64_t[units];
    if (!host) return DA_ERR_HIP;
    hipStream_t s = (hipStream_t)hip_stream;
    hipError_t e = hipMemcpyAsync(host, nnz_dev, units * sizeof(uint64_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        delete[] host;
        return DA_ERR_HIP;
    }
    uint64_t total = 0;
    for (size_t u = 0; u < units; ++u) total += host[u];
    delete[] host;
    const double all = (double)units * (double)rows * (double)head_dim;
    *s_m = 1.0 - (double)total / all;
    const double w = (double)(window < rows ? window : rows);
    *s_c = *s_m * (1.0 - w / (double)rows);
    return DA_OK;
}

}  // extern "C"
