// Rows on their way into a cache in the column-run layout: what a chunk looks like once it is sealed, and the hand-off of prefilled rows
// (Sec. III-C), which runs in an attention launch beside its tiles or in a launch of its own.
#pragma once
#include "cache.hpp"
#include "common.hpp"
#include "mfma.hpp"

namespace da {

// V cache, column-run layout: 16 rows per channel, [unit][t / 16][channel][16].  Inside a group of 16 the
// slot of row p is 8 k + i with k = (p / 4) % 2 and i = 4 (p / 8) + p % 4: the order in which the 32x32
// matrix-core accumulator hands 8 consecutive registers of lane half k to the next contraction.
__device__ __forceinline__ size_t v16_index(int unit, int vrows, int d, int t, int ch) {
    const int p = t & 15;
    const int slot = 8 * ((p >> 2) & 1) + 4 * (p >> 3) + (p & 3);
    return (((size_t)unit * (vrows >> 4) + (t >> 4)) * d + ch) * 16 + slot;
}

template <typename Cache>                                     // (da_cache, in whichever address space)
__device__ __forceinline__ bf16_t *run_room(const Cache &c, int unit, int chunk) {
    return (bf16_t *)c.surv + ((size_t)unit * c.max_chunks + chunk) * run_room_stride(c.d);
}

// A sealed chunk's room holds, per 64 channels (kHalfRoom elements apart): the column masks (64 x 8 bytes: bit r = the
// channel's mask bit of row r), where each channel's run starts (64 x 4 bytes: byte offset from the head), then the runs.
constexpr int kHead = 256 + 128;                             // elements of masks and starts
constexpr int kHalfRoom = kRunHalfRoom;
static_assert(kHalfRoom == kHead + (kChunk + 1) * 64 && kHalfRoom % 8 == 0, "16-byte pieces");

// Seals 64 channels of one chunk, by one wave (lane = channel): head and runs - for every channel in ascending order
// {reference value held before the chunk, then its surviving values in row order}.  From the chunk's keys (row stride d) and
// mask rows in LDS into LDS; returns the number of elements.
__device__ __forceinline__ uint32_t build_runs(const bf16_t *keys, int d, const uint32_t *mask, int wpr, bf16_t held, bf16_t *room) {
    const int lane = lane_id();
    uint32_t lo = 0, hi = 0;                                     // the channel's mask bits of rows 0..31, 32..63
#pragma unroll 16
    for (int r = 0; r < 32; ++r) {
        lo |= ((mask[r * wpr + (lane >> 5)] >> (lane & 31)) & 1u) << r;
        hi |= ((mask[(r + 32) * wpr + (lane >> 5)] >> (lane & 31)) & 1u) << r;
    }
    uint32_t total;
    uint32_t p = kHead + wave_exclusive_scan((uint32_t)__popc(lo) + (uint32_t)__popc(hi) + 1u, &total);
    ((uint32_t *)room)[2 * lane] = lo;
    ((uint32_t *)room)[2 * lane + 1] = hi;
    ((uint32_t *)room)[128 + lane] = 2u * p;
    room[p++] = held;
    for (int rb = 0; rb < kChunk; rb += 16) {                    // 16 keys at a time: reads first
        bf16_t kv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) kv[u] = keys[(rb + u) * d + lane];
        const uint32_t bits = (rb < 32 ? lo : hi) >> (rb & 31);
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if ((bits >> u) & 1u) room[p++] = kv[u];
    }
    return kHead + total;
}

// sealed channels in LDS [D / 64][kHalfRoom] -> the chunk's room, 16-byte pieces (the last one may carry a few elements nobody
// reads)
template <int D, int NT, typename Cache>
__device__ __forceinline__ void store_runs(const Cache &c, int unit, int chunk, const bf16_t *runs, const uint32_t *len, int tid) {
    for (int h = 0; h < D / 64; ++h) {
        u32x4 *dst = (u32x4 *)(run_room(c, unit, chunk) + h * kHalfRoom);
        const u32x4 *src = (const u32x4 *)(runs + h * kHalfRoom);
        for (int i = tid; i < (int)(len[h] + 7) / 8; i += NT) dst[i] = src[i];
    }
    if (tid == 0) c.ccnt[(size_t)unit * c.max_chunks + chunk] = len[0] | (D > 64 ? len[1] << 16 : 0u);
}

// One chunk of one unit of a hand-off, by NT threads: rows t0 .. n_k - 1 (t0 = rows the cache already holds) are appended, item by item those
// of a chunk that contains such a row.  What lies in the chunk and its predecessor before t0 is read from the same arrays.
// The chunk's rows pass through LDS, whole lines in and out.  (A wave per chunk with a lane per channel that loaded and stored
// two bytes at a time took 26 us on 1024 rows of 10 units of 128; a launch of 256 threads a chunk 8.7 us.)
template <int D>
constexpr int kFillLds = 2 * kChunk * D * 2 + D / 64 * kRunHalfRoom * 2 + kChunk * (D / 32) * 4 + 16;
template <int D, int NT, typename Fill>                       // (CacheFill, in whichever address space)
__device__ __forceinline__ void fill_chunk(const Fill &f, int item, char *lds, int tid) {
    constexpr int WPR = D / 32, P = D / 8, kIn = kChunk * P / NT;
    bf16_t *const keys = (bf16_t *)lds, *const vals = keys + kChunk * D, *const runs = vals + kChunk * D;
    uint32_t *const mask = (uint32_t *)(runs + D / 64 * kHalfRoom), *const len = mask + kChunk * WPR;
    static_assert((kChunk * D * 2) % 16 == 0 && (D / 64 * kHalfRoom * 2) % 16 == 0, "16-byte pieces");
    const auto &c = f.cache;
    const int t0 = f.t0, n_k = f.n_k, m = n_k - t0;
    const int at = item / f.units, unit = item - at * f.units, chunk = at + t0 / kChunk, r0 = chunk * kChunk;
    const int wave = tid >> 6, lane = tid & 63;
    const int ra = max(r0, t0), rb = min(r0 + kChunk, n_k);      // new rows of this chunk
    const size_t row0 = (size_t)unit * f.ld, new0 = (size_t)unit * m, cache0 = (size_t)unit * c.max_seq;
    auto held_of = [&](int row, int ch) { return f.H[(row0 + row) * D + ch]; };
    // 1. keys (the chunk's old rows included), values and mask rows into LDS
    {
        u32x4 kk[kIn], vv[kIn];
#pragma unroll
        for (int i = 0; i < kIn; ++i) {                          // (rows past the end are the last one again)
            const int idx = tid + i * NT, row = min(r0 + idx / P, rb - 1), p = idx % P;
            kk[i] = ((const u32x4 *)f.K)[(row0 + row) * P + p];
            vv[i] = ((const u32x4 *)f.V)[(row0 + row) * P + p];
        }
        uint32_t mw = 0;
        const int mrow = min(r0 + tid / WPR, rb - 1);
        if (tid < kChunk * WPR)
            mw = mrow >= t0 ? f.Mnew[(new0 + mrow - t0) * WPR + tid % WPR] : f.Mall[(row0 + mrow) * WPR + tid % WPR];
#pragma unroll
        for (int i = 0; i < kIn; ++i) {
            const int idx = tid + i * NT, row = r0 + idx / P, p = idx % P;
            ((u32x4 *)keys)[idx] = kk[i];
            ((u32x4 *)vals)[idx] = vv[i];
            if (row >= ra && row < rb && row >= n_k - c.Wd) ((u32x4 *)c.ring)[((size_t)unit * c.Wd + row % c.Wd) * P + p] = kk[i];
        }
        if (tid < kChunk * WPR) {
            const int row = r0 + tid / WPR;
            mask[tid] = mw;
            if (row >= ra && row < rb) {
                c.mask[(cache0 + row) * WPR + tid % WPR] = mw;
                if (f.Mall) f.Mall[(row0 + row) * WPR + tid % WPR] = mw;
            }
        }
    }
    if (at == 0 && wave == 3) {
        const NnzSum sum = {f.sum.counts, f.sum.nnz, f.sum.groups, f.sum.units};
        const uint64_t fresh = sum.groups > 0 ? add_up_nnz(sum, lane < 8 ? unit : sum.units) : f.nnz_new[unit];
        if (lane == 0) c.nnz[unit] = (t0 == 0 ? 0ull : c.nnz[unit]) + fresh;
    }
    if (tid < D) {
        if (chunk > 0 && r0 >= t0 && rb - r0 < kChunk) ((bf16_t *)c.ck)[(size_t)unit * D + tid] = held_of(r0 - 1, tid);   // (the last chunk)
        if (rb == n_k) ((bf16_t *)c.khat)[(size_t)unit * D + tid] = held_of(n_k - 1, tid);
    }
    __syncthreads();
    // 2. a chunk completed by these rows is sealed, by the first wave of every 64 channels; the others start on the values
    const bool seals = rb - r0 == kChunk;
    if (seals && wave < D / 64) {
        const bf16_t held = chunk > 0 ? held_of(r0 - 1, 64 * wave + lane) : (bf16_t)0;
        const uint32_t n = build_runs(keys + 64 * wave, D, mask + 2 * wave, WPR, held, runs + wave * kHalfRoom);
        if (lane == 0) len[wave] = n;
    }
    // 3. values: 16 rows of one channel are contiguous, in slot order (v16_index).  A group that starts with a new row is
    //    written whole (rows past the end as zeros), one that starts with old rows only gets its new slots
    const int first = seals ? D / 64 : 0, threads = NT - 64 * first;
    for (int i = tid - 64 * first; i >= 0 && i < (kChunk / 16) * D; i += threads) {
        const int g0 = r0 + i / D * 16, ch = i % D;
        if (g0 >= rb || g0 + 16 <= ra) continue;
        if (g0 >= ra) {
            uint32_t w[8];
#pragma unroll
            for (int slot = 0; slot < 16; ++slot) {
                const int row = g0 + 8 * ((slot & 7) >> 2) + 4 * (slot >> 3) + (slot & 3);
                const uint32_t v = row < rb ? vals[(row - r0) * D + ch] : 0u;
                w[slot >> 1] = (slot & 1) ? w[slot >> 1] | (v << 16) : v;
            }
            u32x4 *dst = (u32x4 *)((bf16_t *)c.V + (((size_t)unit * (c.vrows >> 4) + (g0 >> 4)) * D + ch) * 16);
            dst[0] = u32x4{w[0], w[1], w[2], w[3]};
            dst[1] = u32x4{w[4], w[5], w[6], w[7]};
        } else {
            for (int row = ra; row < min(g0 + 16, rb); ++row)
                ((bf16_t *)c.V)[v16_index(unit, c.vrows, D, row, ch)] = vals[(row - r0) * D + ch];
        }
    }
    __syncthreads();
    if (seals) store_runs<D, NT>(c, unit, chunk, runs, len, tid);
}

}  // namespace da
