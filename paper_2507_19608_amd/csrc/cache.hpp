// Decode-time cache object (Sec. III-A last paragraph, Sec. III-C).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/delta_attn.h"
#include "kernels.hpp"

constexpr int kChunk = 64;   // rows per decode chunk; one reference-key checkpoint per chunk

// What delta_attn_prefill_append keeps between its calls on one cache (Sec. III-C, a prompt processed in pieces):
// the sequence so far as the plain arrays the prefill kernels read, so that a piece only adds its own rows instead
// of unpacking the whole prefix again.  Device memory with max_seq rows of room per unit (row stride
// max_seq), allocated by the first such call, freed with the
// cache.  Host-side bookkeeping: kernels never see it.
struct da_prefix {
    void *k, *h, *v;      // [units][max_seq][d]     keys (raw where a window may need them, see expand_cache_kernel),
                          //                         reference keys, values
    uint32_t *m;          // [units][max_seq][d/32]  mask rows
    int64_t rows;         // k, h, v, m describe rows 0 .. rows - 1 of the cached sequence; only trusted while
                          // rows == the cache's length (decode steps and one-shot prefills do not maintain them)
};

struct da_cache {
    int B, Hq, Hkv, d, max_seq, Wd, dtype;
    float theta, scale;
    int64_t len;          // rows held (all sequences of the batch advance together)
    int device;
    int cus;              // compute units of `device` (0 until the first decode step has asked)
    int nck;              // checkpoints per unit: max_seq / kChunk + 1, or 1 in the column-run layout
    int max_chunks;       // (max_seq + kChunk - 1) / kChunk
    int max_parts;        // partial rows per query head that one decode step can leave
    int vrows;            // max_seq rounded up to a whole chunk (row capacity of V)
    int plan_merge;       // launch plan of the column-run layout: -1 auto, 0 spread over work groups, 1 one per unit
    int plan_slots;       // wave slots a launch is sized for, 0 = from the device
    int fast;             // 1: bf16, head_dim 64 or 128, decode window >= kChunk or >= max_seq, <= 32 query heads per KV
                          //    head: the column-run layout below
    // per (batch, KV head) unit, all device memory:
    uint32_t *mask;       // [units][max_seq][d/32]   delta mask bits
    // Surviving key values (the new reference values at the positions the mask marks).
    //   row layout (fast == 0): row after row, channels ascending inside a row, appended one row per step; kChunk * d
    //     elements of room per chunk.
    //   column-run layout (fast == 1): written once per chunk, when its last row has arrived ("sealed"):
    //     for every channel in ascending order one run = the reference value held when the chunk starts,
    //     then the channel's surviving values in row order.  Rows of an unsealed chunk are always inside
    //     the decode window (window >= kChunk, or the whole cache), where raw keys are used, so they need no run.  Every
    //     64 channels have their own part of the room, kRunHalfRoom elements, with their column masks and starts in front.
    void *surv;           // [units][max_chunks][kChunk * d], or [run_room_stride(d)]
    uint32_t *ccnt;       // [units][max_chunks]      row layout: elements stored in the chunk's room; column-run
                          //                          layout: those of channels 0..63 in the low half, those of
                          //                          channels 64.. in the high half
    void *ck;             // fast == 0: [units][nck][d], ck[m] = reference key after row m*kChunk - 1 (m >= 1);
                          // fast == 1: [units][d], reference key in front of the chunk that is not sealed yet (the sealed
                          //            ones have theirs in their runs)
    void *khat;           // [units][d]               current reference key
    void *ring;           // [units][Wd][d]           raw key of position p at slot p % Wd
    void *V;              // fast == 0: [units][vrows / 8][d][8], 8 rows interleaved per channel;
                          // fast == 1: [units][vrows / 16][d][16], 16 rows per channel in matrix-core
                          //            accumulator order (slot 8 k + i holds row 8 (i / 4) + 4 k + i % 4)
    uint64_t *nnz;        // [units]
    float *part;          // [B*Hq][max_parts][d + 4] partial (o[d], m, l, 2 unused) rows of one decode step
    uint32_t *arrived;    // [units] work groups of a unit that have left their partial rows (column-run layout); 0 between steps
    da_prefix *pf;        // host pointer, NULL until delta_attn_prefill_append has run on this cache
};

// Column-run layout: elements of room per chunk - one per key element, one carried-in value per channel and, per 64 channels, their
// column masks and where their runs start (768 bytes, see decode_runs.hip).  Those are what makes a step's k_hat look-up one
// matrix product; a cache with few query heads per KV head is larger for them, since the partial rows and checkpoints that this
// layout does not need weigh less there: 273 -> 279 bytes a row and KV head with one (head_dim 64, 32 K rows), 286 -> 280 with
// four; 546 -> 558 and 570 -> 559 at head_dim 128.
constexpr int kRunHalfRoom = 384 + (kChunk + 1) * 64;
__host__ __device__ inline size_t run_room_stride(int d) { return (size_t)(d / 64) * kRunHalfRoom; }
// work groups that share a unit in a decode step, at most: what the last of them can merge in a few round trips
constexpr int kMaxParts = 32;
// ... and the walkers of each, at least
inline int run_walkers(int d) { return d == 64 ? 4 : 1; }

// floats per partial row: o[d], running maximum, running sum, padded to a 16-byte multiple
__host__ __device__ inline int part_stride(int d) { return d + 4; }

namespace da {
// the scale a params value stands for: 0 selects 1 / sqrt(head_dim) (Eq. 1)
inline float resolved_scale(float scale, int d) { return scale > 0.f ? scale : 1.0f / sqrtf((float)d); }
inline bool cache_scale_matches(const da_cache *c, float scale) {
    return resolved_scale(scale, c->d) == resolved_scale(c->scale, c->d);
}
da_status cache_check_for_prefill(const da_cache *c, const da_prefill_params *p);
void cache_fill_from_prefill(da_cache *c, const da_prefill_params *p, const void *K, const void *V,
                             const void *Khat, const uint32_t *mask_bits,
                             const uint64_t *nnz, hipStream_t s);
// column-run layout (fast == 1)
// Rows t0 .. n_k - 1 of a sequence on their way into a cache that holds rows 0 .. t0 - 1 (kernels: cache_fill.hpp).
struct CacheFill {
    const unsigned short *K, *V, *H;     // [units][ld][d] keys, values, reference keys, from row 0 on
    const uint32_t *Mnew;                // [units][n_k - t0][d/32] mask rows from t0 on
    uint32_t *Mall;                      // [units][ld][d/32] mask rows from row 0 on, to which the new ones are added; NULL where t0 == 0 and nobody wants them
    const uint64_t *nnz_new;             // [units], or, where sum.groups > 0, to be added up
    NnzSum sum;
    da_cache cache;
    int ld, t0, n_k;
    int units, items;                    // chunks with new rows of all units
};
CacheFill cache_fill(const da_cache *c, int t0, int n_k, int ld, const void *K, const void *V, const void *H, const uint32_t *Mnew, uint32_t *Mall,
                     const uint64_t *nnz_new, const NnzSum &sum);
void launch_cache_fill(const CacheFill &f, hipStream_t s);
// writes the cached rows 0 .. t0 - 1 out as whole-sequence arrays with ld >= t0 rows of room per unit
void expand_cache_runs(da_cache *c, int t0, int ld, void *Kfull, void *Hfull, void *Vfull, uint32_t *Mfull,
                       hipStream_t s);
void decode_step_runs(da_cache *c, const void *q, const void *k, const void *v, void *o, uint32_t *mask_row, int t,
                     float scale_log2, hipStream_t s);
void seal_chunk_runs(da_cache *c, int chunk, hipStream_t s);
}  // namespace da
