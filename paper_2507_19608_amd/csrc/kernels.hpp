// Host-side launch functions of the kernels (one .hip file each).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace da {

// Raises the dynamic-LDS limit of kernel `fn` to `bytes` on the current device, once per device (`done` holds one bit
// per device ordinal; safe to call from several threads).  On failure the error is left for launch_ok() to report
// and the next call tries again.
void ensure_dynamic_lds(const void *fn, int bytes, std::atomic<uint64_t> &done);

// Checks hipGetLastError(); on failure records "<stage>: <hip error>" for delta_attn_last_error()
// and returns false.
bool launch_ok(const char *stage);
const char *last_error_text();
// records a printf-style message as the calling thread's last error text
void set_last_error(const char *fmt, ...) __attribute__((format(printf, 1, 2)));

// Optional per-stage timing with HIP events recorded on the caller's stream (off by default).
// Numbered as in the header, whose stage 1 no kernel has any more.
enum Stage { kStageScan = 0, kStageAttn = 2, kStageCacheFill, kStageAppend, kStageChunk, kStageCombine, kNumStages };
void stage_begin(int stage, hipStream_t s);   // no-ops unless timing is enabled
void stage_end(int stage, hipStream_t s);
void timing_enable(bool on);
int timing_collect(double *ms_per_stage, int *calls_per_stage);

// Fired entries that a scan has left per unit and group of channels, [units][groups] (at most 64 groups), for the launch that follows
// it to add up into nnz [units].  groups == 0: nnz has been written.
struct NnzSum {
    const uint32_t *counts = nullptr;
    uint64_t *nnz = nullptr;
    int groups = 0, units = 0;
};

struct PrefillArgs {
    int dtype;            // 0 f32, 1 bf16
    int B, Hq, Hkv, d, n, W;   // n = number of key rows
    int q_off, nq;             // the query rows are positions q_off .. q_off + nq - 1 (q_off + nq == n)
    int ld = 0;                // > 0 (matrix-core path only): K, V, Khat have ld >= n rows of room per unit; 0: exactly n
    float scale_log2;     // score scale * log2(e)
    int sliding;          // 1: exact region is the band i - j < W instead of squares of side W
    const void *Q, *K, *V, *Khat;
    void *O;
    uint32_t *queue;      // (matrix-core path) kPrefillQueueBytes, zeroed
    NnzSum sum;           // to be added up on the way
};
struct CacheFill;         // (cache.hpp)
constexpr int kPrefillQueueBytes = 512;

// Rows of a piece of a longer sequence that join arrays with `ld` rows of room per unit: src[k] [units][rows][..] to dst[k], which points at the first
// unit's first new row.  In pieces of 16 bytes, `pieces` a row; sources may start anywhere.
struct RowCopy {
    const void *src[2];
    void *dst[2];
    int units, rows, ld, pieces;
};

void launch_fill_u64(uint64_t *p, uint64_t v, int n, hipStream_t s);

// scratch: delta_scan_scratch_bytes(); counts: NULL, or room for units * d / 8 words, which may then be left for the caller to
// add up (NnzSum; launch_nnz_sum, where no other launch takes it along); init: NULL (row 0 is the basis row), or [units][d], the
// reference key the rows continue from; zeroed: NULL, or kPrefillQueueBytes to clear for the attention launch that follows
size_t delta_scan_scratch_bytes(int dtype, int units, int n, int d);
// copy: rows that the launch copies beside the scan, and Khat's room (NULL: none, n rows)
NnzSum launch_delta_scan(int dtype, const void *K, void *Khat, uint32_t *mask_bits, void *scratch, uint32_t *counts, uint64_t *nnz,
                         int units, int n, int d, float theta, hipStream_t s, const void *init, uint32_t *zeroed, const RowCopy *copy = nullptr);
void launch_nnz_sum(const NnzSum &sum, hipStream_t s);
bool delta_scan_settles(int dtype, int units, int n, int d);   // without `counts` a second launch follows
// Generic path: any head_dim in {32, 64, ..., 256}, both dtypes, binary32 products.  Returns false if the head_dim has
// no instantiation.  q_off and ld are not for it.
// scan: NULL, or what the scan of the keys is to write, which the launch then does itself (a.Khat and a.sum are not for it); only where
// prefill_generic_scans says so.
struct PrefillScan {
    uint32_t *mask_bits;
    uint64_t *nnz;
    float theta;
};
bool prefill_generic_scans(const PrefillArgs &a);
bool launch_prefill_generic(const PrefillArgs &a, const PrefillScan *scan, hipStream_t s);
// Matrix-core path: bf16, head_dim 64 or 128.  K and V have to be aligned to 16 bytes when it is launched.
bool prefill_mfma_supported(const PrefillArgs &a);
// K and V that are not are copied to room_k, room_v (`bytes` each, aligned), which take their place in `a`.
void launch_copy_aligned(PrefillArgs &a, void *room_k, void *room_v, size_t bytes, hipStream_t s);
// fill: NULL, or a hand-off whose items the launch takes along; not where prefill_takes_fill says that a launch of its own is faster.
void launch_prefill_mfma(const PrefillArgs &a, const CacheFill *fill, hipStream_t s);
bool prefill_takes_fill(const PrefillArgs &a, const CacheFill &fill);
// Scan and attention in one launch, of prompts whose rows fit into LDS: bf16, head_dim 64 or 128.  K and V have to be aligned to 16
// bytes when it is launched.  khat: NULL, or [units][n][d] for the reference keys; a.Khat, a.queue and a.sum are not for it.
bool prefill_short_supported(const PrefillArgs &a);
void launch_prefill_short(const PrefillArgs &a, float theta, void *khat, uint32_t *mask_bits, uint64_t *nnz, hipStream_t s);
// compute units of the current device (256 if it cannot be asked)
int device_cu_count();

}  // namespace da
