// Delta matrix construction on the key matrix (Sec. II-C Eq. 2-3; Sec. III-A strategy 3).
#include "common.hpp"
#include "kernels.hpp"

#include <stdarg.h>
#include <stdio.h>

#include <mutex>
#include <type_traits>
#include <utility>

namespace da {

static thread_local char g_last_error[256] = "";

bool launch_ok(const char *stage) {
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return true;
    snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%s)", stage, hipGetErrorName(e), hipGetErrorString(e));
    return false;
}

const char *last_error_text() { return g_last_error; }

void set_last_error(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
}

void ensure_dynamic_lds(const void *fn, int bytes, std::atomic<uint64_t> &done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 63;   // ordinals past 62 share a bit: set every time
    const uint64_t bit = (uint64_t)1 << dev;
    if (dev < 63 && (done.load(std::memory_order_acquire) & bit)) return;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess)
        done.fetch_or(bit, std::memory_order_release);
}

// ---- stage timing: a pool of event pairs, filled in call order, summed and recycled by the reader
namespace {
constexpr int kMaxPairs = 8192;
struct Pair {
    hipEvent_t a, b;
    int stage;
};
std::mutex g_timing_mutex;   // the pool is process-wide: a benchmarking aid, serialised rather than per call
std::atomic<bool> g_timing{false};
Pair g_pairs[kMaxPairs];
int g_created = 0, g_used = 0, g_open[kNumStages];
}  // namespace

void stage_begin(int stage, hipStream_t s) {
    if (!g_timing.load(std::memory_order_relaxed)) return;
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    if (g_used >= kMaxPairs) return;
    if (g_used >= g_created) {
        if (hipEventCreate(&g_pairs[g_created].a) != hipSuccess) return;
        if (hipEventCreate(&g_pairs[g_created].b) != hipSuccess) return;
        ++g_created;
    }
    g_pairs[g_used].stage = stage;
    g_open[stage] = g_used;
    (void)hipEventRecord(g_pairs[g_used].a, s);
    ++g_used;
}

void stage_end(int stage, hipStream_t s) {
    if (!g_timing.load(std::memory_order_relaxed)) return;
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    if (g_open[stage] < 0) return;
    (void)hipEventRecord(g_pairs[g_open[stage]].b, s);
    g_open[stage] = -1;
}

void timing_enable(bool on) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    g_timing.store(on);
    g_used = 0;
    for (int i = 0; i < kNumStages; ++i) g_open[i] = -1;
}

// Sums elapsed ms per stage over everything recorded since the last read; the caller has
// synchronised the streams involved.  Returns the number of event pairs read.
int timing_collect(double *ms_per_stage, int *calls_per_stage) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    for (int i = 0; i < kNumStages; ++i) {
        ms_per_stage[i] = 0.0;
        calls_per_stage[i] = 0;
    }
    int n = 0;
    for (int i = 0; i < g_used; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, g_pairs[i].a, g_pairs[i].b) == hipSuccess) {
            ms_per_stage[g_pairs[i].stage] += ms;
            calls_per_stage[g_pairs[i].stage] += 1;
            ++n;
        }
    }
    g_used = 0;
    return n;
}

// The recurrence of Eq. 2-3 is sequential in t and is not an associative scan, but it forgets its past every time a
// channel fires: from then on the held value is k(t) whatever it was before.  So time is cut into pieces that are walked in
// parallel from a guessed incoming state, and pieces whose guess was wrong are walked again from the right one:
//
//   scan_whole_kernel     prompts of up to some thousand rows (whole_plan): one work group per unit and few channels, all rows in LDS,
//       so that nothing is left for a second launch; the counts are added up by the launch that follows anyway.
//   scan_segments_kernel  one work group per (unit, segment of S rows, group of channels); lane = channel, and the waves of
//       64 channels cut the segment into runs of rows.  The segment's rows and up to `warm` rows before it are copied to LDS
//       once (16-byte loads, every one in flight together: row by row from global memory the walk paid a memory round
//       trip per batch of rows).  Every run first walks the rows before it from the guess "held = an earlier row", then its
//       own rows, replacing each key in LDS by its reference key.  Runs then compare the value they started from with
//       the value the run before ended on and walk again, in parallel, until all agree: after round i the first i + 1 runs
//       are exact, and a run usually meets its old chain (both fire at the same row) after a few rows, so a round or
//       two does it.  Reference keys leave LDS in 16-byte pieces.
//   scan_settle_kernel    prompts of several segments: one work group per unit and 16 channels takes every segment's start from its predecessor's
//       end, in order, walks what differs again, in parallel, and adds up nnz.  Where units are many, scan_settle_rounds_kernel: one of 64 channels, which walks
//       what differs in rounds as long as that settles it, else in order.
//
// Exact for any input.  The wave ballot of the threshold decision is the mask word itself.
// Against two passes and an ordered repair with row-by-row loads: 20 x 8192 rows of 128 in bf16 (86 MB in and out, 5 % jumps) 62 ->
// 38 us a call.
constexpr int kScanLdsMax = 144 * 1024;    // a one-segment prompt: 128 KB of rows, their mask words, the runs' end values

// lane L of (lo, hi) takes the two halves of a wave mask: two instructions, where comparing the lane number and selecting
// twice takes five.  (s_nop: a mask that a vector compare has just written may be read two wait states later, which the
// compiler does not look after inside asm.)
template <int L>
__device__ __forceinline__ void mask_to_lane(uint32_t &lo, uint32_t &hi, uint64_t mask) {
    asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
        : "+v"(lo), "+v"(hi)
        : "s"((uint32_t)mask), "s"((uint32_t)(mask >> 32)), "n"(L));
}

constexpr int U = 16;      // rows in a batch

// f(0), f(1), ... f(U - 1) with the index a constant
template <typename F, int... I>
__device__ __forceinline__ void for_batch_impl(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <typename F>
__device__ __forceinline__ void for_batch(F f) {
    for_batch_impl(f, std::make_integer_sequence<int, U>{});
}

// rows a .. b - 1 (LDS, this lane's channel, row stride d elements) in order: batch(t, k) for U rows from t on, then
// single(t, k) for each of the rest.  Batches of U rows, the
// next one's LDS reads issued before this one is worked on; keys are kept as stored until then (a conversion at the
// read would wait for it), and a batch past the end re-reads the last U rows, so that no read hangs on a condition.
template <typename T, typename Batch, typename Single>
__device__ __forceinline__ void each_row(const T *rows, int d, int a, int b, Batch batch, Single single) {
    auto fetch = [&](T (&k)[U], int t) {
        const T *r = rows + min(t, b - U) * d;
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = r[u * d];
    };
    int t = a;
    if (t + U <= b) {
        T ka[U], kb[U];
        fetch(ka, t);
        while (true) {
            fetch(kb, t + U);
            batch(t, ka);
            t += U;
            if (t + U > b) break;
            fetch(ka, t + U);
            batch(t, kb);
            t += U;
            if (t + U > b) break;
        }
    }
    for (; t < b; ++t) single(t, rows[t * d]);
}

// the value held after rows a .. b - 1, from `held`; nothing is written
template <typename T>
__device__ __forceinline__ float walk(const T *rows, int d, int a, int b, float held, float theta) {
    auto step = [&](T raw) {
        const float k = to_f32(raw);
        held = fabsf(k - held) > theta ? k : held;
    };
    each_row(
        rows, d, a, b,
        [&](int, const T (&k)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) step(k[u]);
        },
        [&](int, T k) { step(k); });
    return held;
}

// Walks rows t0 .. t1 - 1 again, from `held` instead of `spec` (where the recorded chain started), until the two chains meet
// in every lane (one that has met its old chain writes what stands there already).  Kp: the keys, Hp: the reference keys
// (this lane's channel, row strides d and dh elements), Mp: the two mask words of the wave's channels (row stride dm; `two`:
// both exist).  Returns the value the rows end on (`end` is the recorded one); *adjust receives the change of the number of
// fired entries.
template <typename T>
__device__ __forceinline__ float rewalk(const T *Kp, int d, T *Hp, int dh, uint32_t *Mp, int dm, bool two, int t0, int t1,
                                        float spec, float held, float end, bool active, float theta, long long *adjust) {
    const int lane = threadIdx.x & 63;
    bool synced = !active || __float_as_uint(spec) == __float_as_uint(held);
    auto fetch = [&](T (&k)[U], int tb) {                        // rows past the end are clamped and not worked on
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = Kp[(size_t)min(tb + u, t1 - 1) * d];
    };
    auto work = [&](const T (&kk)[U], int tb) {
        uint32_t wlo = 0, whi = 0;
        T *h = Hp + (size_t)tb * dh;
        for_batch([&](auto u) {
            const bool here = active && tb + u < t1;
            const float k = to_f32(kk[u]);
            const bool fs = here && fabsf(k - spec) > theta, ft = here && fabsf(k - held) > theta;
            spec = fs ? k : spec;
            held = ft ? k : held;
            const uint64_t bt = __ballot(ft);
            mask_to_lane<u>(wlo, whi, bt);
            *adjust += (long long)__popcll(bt) - (long long)__popcll(__ballot(fs));
            if (here) store_exact(h, (size_t)u * dh, held);
        });
        synced = synced || __float_as_uint(spec) == __float_as_uint(held);   // (chains that have met stay together)
        if (lane < U && tb + lane < t1) {
            uint32_t *m = Mp + (size_t)(tb + lane) * dm;
            m[0] = wlo;
            if (two) m[1] = whi;
        }
        return tb + U < t1 && __any(!synced);
    };
    T ka[U], kb[U];
    fetch(ka, t0);
    for (int tb = t0;; tb += 2 * U) {
        fetch(kb, tb + U);
        if (!work(ka, tb)) break;
        fetch(ka, tb + 2 * U);
        if (!work(kb, tb + U)) break;
    }
    return synced ? end : held;
}

// Work group `at` of `groups` copies its share of the rows, 64 at a time of one unit.  (A prompt fed in pieces: the launch that scans a piece
// leaves compute units idle, and its attention reads keys and values from arrays that hold the whole sequence.)
typedef unsigned __attribute__((ext_vector_type(4), aligned(2))) u32x4_any;
__device__ __forceinline__ void copy_rows(const RowCopy &c, int at, int groups) {
    constexpr int kRows = 64, N = 8;
    const int blocks = (c.rows + kRows - 1) / kRows, threads = (int)blockDim.x;
    for (int i = at; i < c.units * blocks; i += groups) {
        const int unit = i / blocks, r0 = (i - unit * blocks) * kRows, count = min(kRows, c.rows - r0) * c.pieces;
        for (int k = 0; k < 2; ++k) {
            const u32x4_any *src = (const u32x4_any *)c.src[k] + ((size_t)unit * c.rows + r0) * c.pieces;
            uint4 *dst = (uint4 *)c.dst[k] + ((size_t)unit * c.ld + r0) * c.pieces;
            for (int p0 = threadIdx.x; p0 < count; p0 += N * threads) {
                u32x4_any v[N];
#pragma unroll
                for (int u = 0; u < N; ++u) v[u] = src[min(p0 + u * threads, count - 1)];
#pragma unroll
                for (int u = 0; u < N; ++u)
                    if (p0 + u * threads < count) dst[p0 + u * threads] = uint4{v[u][0], v[u][1], v[u][2], v[u][3]};
            }
        }
    }
}

// What a scan launch looks like.  `dl` channels per work group (all of them, or 64), `waves` waves.
struct ScanPlan {
    int S, nseg, warm;      // rows per segment, segments, rows walked before a segment
    int dl, waves;
    size_t lds;             // dynamic LDS bytes of scan_segments_kernel
};

template <typename T>
struct ScanArgs {
    const T *__restrict__ K;
    T *__restrict__ Khat;
    uint32_t *__restrict__ mask_bits;
    T *starts, *ends;                    // [units][nseg][d] value every segment started from / ended on
    uint32_t *counts;                    // [units][nseg][groups of 64 channels] fired entries
    unsigned long long *nnz;
    const T *init;
    uint32_t *zeroed;                    // kPrefillQueueBytes, or NULL
    int n, d, S, nseg, warm, dl;
    float theta;
    int ld;                              // rows of room per unit in Khat
};

// DL: channels per work group where known when compiling (LDS offsets become immediates), or 0.  Copy: RowCopy, for whose rows the last blockIdx.z
// is there, or nothing (with a look at them in every launch 20 x 8192 rows of 128 took 36.2 instead of 35.4 us).
template <typename T, int DL, typename... Copy>
__global__ __launch_bounds__(512) void scan_segments_kernel(ScanArgs<T> g, Copy... copy) {
    extern __shared__ __attribute__((aligned(16))) char lds_s[];
    const int groups = (int)gridDim.z - (int)sizeof...(Copy);
    if (sizeof...(Copy) > 0 && (int)blockIdx.z == groups) {
        (copy_rows(copy, (int)(blockIdx.y * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.y)), ...);
        return;
    }
    const int seg = blockIdx.x, unit = blockIdx.y, tid = threadIdx.x, lane = tid & 63, threads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = g.n, d = g.d, ch0 = blockIdx.z * g.dl;
    const int dl = DL ? DL : min(g.dl, d - ch0);                 // this work group's channels
    const int wpr = d >> 5, wl = dl >> 5, CW = (dl + kWave - 1) / kWave, TW = (threads >> 6) / CW;
    const int t0 = seg * g.S, t1 = min(n, t0 + g.S), lo = max(0, t0 - g.warm), rows = t1 - lo;
    const float theta = g.theta;
    T *R = (T *)lds_s;                                           // [rows][dl]: keys, then reference keys from row t0 on
    uint32_t *M = (uint32_t *)(R + rows * dl);                   // [t1 - t0][wl] mask words
    float *E = (float *)(M + (t1 - t0) * wl);                    // [TW][dl] value every run ended on
    uint32_t *cnt = (uint32_t *)(E + TW * dl);                   // fired entries
    const T *Kp = g.K + (size_t)unit * n * d + ch0;
    const int ppr = dl * (int)sizeof(T) / 16, gpr = d * (int)sizeof(T) / 16;   // 16-byte pieces per row here / in memory
    // 1. the rows into LDS
    {
        const uint4 *src = (const uint4 *)(Kp + (size_t)lo * d);
        uint4 *dst = (uint4 *)R;
        const int pieces = rows * ppr;
        constexpr int kIn = 8;
        for (int i0 = tid; i0 < pieces; i0 += kIn * threads) {
            // (pieces past the end are the last one again, loaded and stored: under a condition the compiler would
            // pull each load down to its store and wait for it there)
            uint4 v[kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                const int i = min(i0 + k * threads, pieces - 1);
                v[k] = src[(size_t)(i / ppr) * gpr + i % ppr];
            }
#pragma unroll
            for (int k = 0; k < kIn; ++k) dst[min(i0 + k * threads, pieces - 1)] = v[k];
        }
        if (tid == 0) *cnt = 0;
        if (g.zeroed && seg == 0 && unit == 0 && blockIdx.z == 0 && tid < kPrefillQueueBytes / 4) g.zeroed[tid] = 0;
        if (g.nseg > 1 && seg == 0 && blockIdx.z == 0 && tid == 0) g.nnz[unit] = 0;   // (scan_settle_kernel adds to it)
    }
    __syncthreads();
    // 2. this wave's run of rows a .. b - 1 (LDS rows) and the guess it starts from
    const int run = wave / CW, c = (wave % CW) * kWave + lane;
    constexpr bool kFull = DL > 0;                               // every wave has a run of 64 channels
    const bool works = kFull || run < TW, active = kFull || (works && c < dl);
    const int cs = kFull ? c : min(c, dl - 1), word = (wave % CW) * 2;
    const int L = (t1 - t0 + TW - 1) / TW;
    const int a = works ? min(t0 + run * L, t1) - lo : 0, b = works ? min(t0 + (run + 1) * L, t1) - lo : 0;
    T *Rc = R + cs;
    float start = 0.f;
    if (a < b) {
        // a run after the first warms up on half the rows: what it gets wrong is put right inside the work group
        const int w = max(0, a - (run == 0 ? g.warm : g.warm / 2));
        if (w == 0 && lo == 0 && g.init)
            start = walk(Rc, dl, 0, a, load_f32(g.init, (size_t)unit * d + ch0 + cs), theta);
        else if (a > 0)
            start = walk(Rc, dl, w + 1, a, load_f32(Rc, (size_t)(w * dl)), theta);   // (row 0: the basis row, exact)
    }
    const bool basis = a == 0 && lo == 0 && !g.init;             // the run's first row is kept whole
    __syncthreads();                                             // nobody needs the keys of another run any more
    // 3. the run itself
    float held = start;
    uint32_t fired = 0;
    auto row = [&](int t, T raw, bool first) -> uint64_t {       // returns the row's mask
        const float k = to_f32(raw);
        const bool fire = (kFull || active) && (first || fabsf(k - held) > theta);   // Eq. 2 in binary32
        held = fire ? k : held;                                                      // Eq. 3
        const uint64_t bal = __ballot(fire);
        fired += __popcll(bal);
        if (active) store_exact(Rc, (size_t)(t * dl), held);
        return bal;
    };
    auto put_mask = [&](int t, uint32_t wlo, uint32_t whi) {
        uint32_t *m = M + (lo + t - t0) * wl + word;
        m[0] = wlo;
        if (word + 1 < wl) m[1] = whi;
    };
    auto single = [&](int t, T raw, bool first) {
        const uint64_t bal = row(t, raw, first);
        if (lane == 0) put_mask(t, (uint32_t)bal, (uint32_t)(bal >> 32));
    };
    int from = a;
    if (basis && a < b) single(from++, Rc[0], true);
    each_row(
        Rc, dl, from, b,
        [&](int t, const T (&k)[U]) {
            uint32_t wlo = 0, whi = 0;                           // lane u keeps the mask of row t + u
            for_batch([&](auto u) { mask_to_lane<u>(wlo, whi, row(t + u, k[u], false)); });
            if (lane < U) put_mask(t + lane, wlo, whi);
        },
        [&](int t, T k) { single(t, k, false); });
    if (active) E[run * dl + c] = held;
    __syncthreads();
    // 4. runs whose guess was wrong, again
    long long adjust = 0;
    for (int round = 1; round < TW; ++round) {
        float prev = start;
        const bool follows = active && run > 0 && a < b;
        if (follows) prev = E[(run - 1) * dl + c];
        const bool wrong = follows && __float_as_uint(prev) != __float_as_uint(start);
        if (!__syncthreads_or(wrong)) break;                     // (also: every run has read its predecessor's end)
        if (__any(wrong)) {
            held = rewalk(Kp + (size_t)lo * d + cs, d, Rc, dl, M + (lo - t0) * wl + word, wl, word + 1 < wl, a, b, start, prev,
                          held, active, theta, &adjust);
            start = prev;
            if (active) E[run * dl + c] = held;
        }
        __syncthreads();
    }
    if (lane == 0 && a < b) atomicAdd(cnt, (uint32_t)((long long)fired + adjust));
    // 5. out: reference keys, mask words, the segment's boundary values, nnz
    if (g.nseg > 1 && active) {
        const size_t at = ((size_t)unit * g.nseg + seg) * d + ch0 + c;
        if (run == 0) store_exact(g.starts, at, start);
        if (run == (t1 - t0 - 1) / L) store_exact(g.ends, at, held);     // the run that holds the segment's last row
    }
    __syncthreads();
    {
        uint4 *dst = (uint4 *)(g.Khat + ((size_t)unit * g.ld + t0) * d + ch0);
        const uint4 *src = (const uint4 *)(R + (t0 - lo) * dl);
        for (int i = tid; i < (t1 - t0) * ppr; i += threads) dst[(size_t)(i / ppr) * gpr + i % ppr] = src[i];
        uint32_t *mo = g.mask_bits + ((size_t)unit * n + t0) * wpr + (ch0 >> 5);
        for (int i = tid; i < (t1 - t0) * wl; i += threads) mo[(size_t)(i / wl) * wpr + i % wl] = M[i];
    }
    if (tid == 0) {
        if (g.nseg > 1)
            g.counts[((size_t)unit * g.nseg + seg) * groups + blockIdx.z] = *cnt;
        else
            g.nnz[unit] = *cnt;
    }
}

// The value that a lane's row per lane - `rows` of them, at most 64 - ends on from `held`, bits of a float: the lanes vote on which fire.
__device__ __forceinline__ int fired_in(float k, int rows, int held, float theta) {
    const int lane = threadIdx.x & 63;
    uint64_t fires = __ballot(lane < rows && fabsf(k - __int_as_float(held)) > theta);   // Eq. 2 in binary32
    while (fires) {
        const int t = __builtin_ctzll(fires);
        held = __builtin_amdgcn_readlane(__float_as_int(k), t);                          // Eq. 3
        fires = __ballot(lane < rows && fabsf(k - __int_as_float(held)) > theta) & (~1ull << t);
    }
    return held;
}

// One channel's runs (or segments) 1 .. count - 1 by one wave: those whose start is not what the one before ends on are walked from that, in order.
// walk(run, start's bits): what it ends on, in every lane.  Returns whether there was one.
template <typename End, typename Start, typename Put, typename Walk>
__device__ __forceinline__ bool runs_in_order(int count, End end_of, Start start_of, Put put_end, Walk walk) {
    const int lane = threadIdx.x & 63;
    bool found = false;
    int held = 0, last = 0;                                      // (what the run `last` ends on now)
    for (int r0 = 1; r0 < count; r0 += 64) {
        const int mine = min(r0 + lane, count - 1);              // a lane per run: what it should start from, and did
        int from = __float_as_int(end_of(mine - 1));
        const int start = __float_as_int(start_of(mine));
        if (lane == 0 && last == r0 - 1 && last > 0) from = held;
        uint64_t wrong = __ballot(r0 + lane < count && from != start);
        found = found || wrong;
        while (wrong) {
            const int i = __builtin_ctzll(wrong), r = r0 + i;
            wrong &= wrong - 1;
            held = walk(r, __builtin_amdgcn_readlane(from, i));
            last = r;
            if (lane == 0) put_end(r, __int_as_float(held));
            if (i < 63 && r + 1 < count) {
                from = lane == i + 1 ? held : from;
                wrong = (wrong & ~(2ull << i)) | (held != __builtin_amdgcn_readlane(start, i + 1) ? 2ull << i : 0ull);
            }
        }
    }
    return found;
}

// ---- One launch for a prompt of up to some thousand rows: a work group takes a few channels (DL = 8, 16 or 32) of every row of
// a unit, so that all of a prompt's rows lie in one LDS and nothing has to be settled between work groups, and the channels of
// one unit still spread over many compute units.  A thread walks one run of L rows in two neighbouring channels (two
// chains: one alone leaves every other issue slot empty); runs start from the guess "held = the row before".  The ends travel from run to run,
// at first in rounds as above, but nothing is written in a round: a wrong run of L rows is walked again whole.  A round moves a chain on by one run and lasts as long as
// 32 rows' walk, also where few chains are wrong, so that after one round or none a wave per channel takes them in order.  One last walk puts the reference keys in
// the place of the keys.  The mask is what the reference keys say: an entry has fired
// where a row differs from the one before (it fires only if |k - held| > theta >= 0, and then holds k).
// A thread then has a row in registers: it goes out with its mask bits.  What bounds it: 50 clocks per row and two channels in the chain,
// 48 rows of it and a run's own, the rest is latency; 8 x 1024 rows of 64: rows in LDS after 1.2 us, walked after 3.2, settled 3.5, replaced
// 4.2, out 5.4.  Rounds alone / this, the scan's launches of 8 x 2048 rows of 64 back to back: 5 % jumps 13.3 / 12.0, threshold 0.2 17.8 / 13.9, 1 % 15.4 / 12.6,
// 1 % and 0.2 31.2 / 17.8, 20 % 11.2 / 11.1; 5 x 4096 of 128 17.8 / 17.4, 21.2 / 19.2, 19.1 / 17.9, 30.7 / 23.8, 16.7 / 16.7.
template <typename T>
struct WholeArgs {
    const T *__restrict__ K;
    T *__restrict__ Khat;
    uint32_t *__restrict__ mask_bits;
    uint32_t *counts;                    // [units][groups of DL channels] fired entries
    const T *init;
    uint32_t *zeroed;                    // kPrefillQueueBytes, or NULL
    int units, n, d, L, warm;            // L rows a run, a multiple of 8
    uint32_t by_l_mul, by_l_shift;       // n / L
    float theta;
    int ld;                              // rows of room per unit in Khat
    int blocks;                          // work groups that scan
    int rounds;                          // before the rest settles in order
};

template <typename T> struct TwoRaw;
template <> struct TwoRaw<bf16_t> { using type = uint32_t; };
template <> struct TwoRaw<float> { using type = uint2; };
__device__ __forceinline__ float first_of(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float second_of(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ float first_of(uint2 v) { return __uint_as_float(v.x); }
__device__ __forceinline__ float second_of(uint2 v) { return __uint_as_float(v.y); }
__device__ __forceinline__ void both(uint32_t &v, float a, float b) { v = (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u); }
__device__ __forceinline__ void both(uint2 &v, float a, float b) { v = uint2{__float_as_uint(a), __float_as_uint(b)}; }

// which of 16 (bf16) or 4 (fp32) channels differ between two rows' 16-byte pieces, one bit each
template <typename T>
__device__ __forceinline__ uint32_t piece_bits(uint4 x, uint4 y);
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
template <>
__device__ __forceinline__ uint32_t piece_bits<bf16_t>(uint4 x, uint4 y) {   // 8 channels: even ones in the low half's bits 0, 2, 4, 6
    const uint32_t w[4] = {x.x ^ y.x, x.y ^ y.y, x.z ^ y.z, x.w ^ y.w};
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const u16x2_t one = __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, w[j]), u16x2_t{1, 1});
        m |= __builtin_bit_cast(uint32_t, one) << (2 * j);
    }
    return (m & 0xffffu) | (m >> 15);                            // odd channels: from bit 16 + 2 j to bit 2 j + 1
}
template <>
__device__ __forceinline__ uint32_t piece_bits<float>(uint4 x, uint4 y) {
    return min(x.x ^ y.x, 1u) | min(x.y ^ y.y, 1u) << 1 | min(x.z ^ y.z, 1u) << 2 | min(x.w ^ y.w, 1u) << 3;
}

// 32 channels a work group: rounds alone (whole_plan)
template <int DL> constexpr bool kInOrder = DL < 32;

template <typename T, int DL, typename... Copy>                  // Copy: RowCopy, for the work groups behind those that scan, or nothing
__global__ __launch_bounds__(512) void scan_whole_kernel(WholeArgs<T> g, Copy... copy) {
    using Raw = typename TwoRaw<T>::type;
    constexpr int PR = DL / 2;                                   // threads of a run
    constexpr int P = DL * (int)sizeof(T) / 16;                  // 16-byte pieces of a row
    constexpr int kPer = 16 / (int)sizeof(T);                    // channels of a piece
    extern __shared__ __attribute__((aligned(16))) char lds_w[];
    // LDS: a row for what the first row continues from, then the runs of L rows with one to spare after each (so that the runs of a
    // wave, read at the same step, lie in different banks), then the runs' ends
    if (sizeof...(Copy) > 0 && (int)blockIdx.x >= g.blocks) {
        (copy_rows(copy, (int)blockIdx.x - g.blocks, (int)gridDim.x - g.blocks), ...);
        return;
    }
    const int groups = g.d / DL, n = g.n, L = g.L;
    const int unit = (int)(blockIdx.x & 7) + 8 * (int)(blockIdx.x / (8 * groups)), group = (int)(blockIdx.x >> 3) % groups;   // (a unit keeps to one XCD)
    if (unit >= g.units) return;
    const int tid = threadIdx.x, threads = blockDim.x, ch0 = group * DL;
    const int runs = (n + L - 1) / L, run = tid / PR, p = tid % PR;
    const bool works = run < runs;
    auto run_of = [&](int t) { return (int)(__umulhi(2u * (uint32_t)t, g.by_l_mul) >> g.by_l_shift); };
    uint4 *const rows = (uint4 *)lds_w + P;                      // piece q of row t: rows[(t + run_of(t)) * P + q]
    float2 *const E = (float2 *)(rows + (size_t)runs * (L + 1) * P);   // [runs][PR]
    float2 *const S = E + runs * PR;                             // [runs][PR] what the runs have been walked from, where they settle in order
    uint32_t *const flags = (uint32_t *)(kInOrder<DL> ? S + runs * PR : S);   // [2] some run was wrong in an even, odd round
    uint32_t *const total = flags + 2;
    const T *Kp = g.K + (size_t)unit * n * g.d + ch0;
    const int gpr = g.d / kPer;                                  // pieces of a row in memory
    const uint4 *const src = (const uint4 *)Kp;
    {
        const int pieces = n * P;
        constexpr int kIn = 8;
        for (int i0 = tid; i0 < pieces; i0 += kIn * threads) {
            uint4 v[kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) {                      // (pieces past the end are the last one again)
                const int i = min(i0 + k * threads, pieces - 1);
                v[k] = src[(size_t)(i / P) * gpr + i % P];
            }
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                const int i = min(i0 + k * threads, pieces - 1), t = i / P;
                rows[(t + run_of(t)) * P + i % P] = v[k];
            }
        }
        // the last run is filled up with its last row again: walked once more it changes nothing
        for (int i = pieces + tid; i < runs * L * P; i += threads) {
            const int t = i / P;
            rows[(t + runs - 1) * P + i % P] = src[(size_t)(n - 1) * gpr + i % P];
        }
        if (tid < P) rows[tid - P] = g.init ? ((const uint4 *)(g.init + (size_t)unit * g.d + ch0))[tid] : src[tid];
        if (tid < 3) flags[tid] = 0;
        if (g.zeroed && blockIdx.x == 0)
            for (int i = tid; i < kPrefillQueueBytes / 4; i += threads) g.zeroed[i] = 0;
    }
    __syncthreads();
    const float theta = g.theta;
    const int a = run * L;
    constexpr int N = 8;                                         // rows in a batch
    auto fetch = [&](Raw (&k)[N], int t) {                       // rows t .. t + 7, of one run (t is a multiple of 8)
        const Raw *r = (const Raw *)(rows + (t + run_of(t)) * P) + p;
#pragma unroll
        for (int u = 0; u < N; ++u) k[u] = r[u * PR];
    };
    auto step = [&](float2 &held, Raw k) {                       // Eq. 2 in binary32, Eq. 3
        const float x = first_of(k), y = second_of(k);
        held.x = fabsf(x - held.x) > theta ? x : held.x;
        held.y = fabsf(y - held.y) > theta ? y : held.y;
    };
    // the rows t .. end - 1 in order from `held`, the next batch's reads issued before this one is worked on
    auto walk_rows = [&](int t, int end, float2 held) __attribute__((always_inline)) {
        Raw ka[N], kb[N];
        if (t < end) fetch(ka, t);
        for (; t < end; t += 2 * N) {
            fetch(kb, min(t + N, end - N));
#pragma unroll
            for (int u = 0; u < N; ++u) step(held, ka[u]);
            if (t + N >= end) break;
            fetch(ka, min(t + 2 * N, end - N));
#pragma unroll
            for (int u = 0; u < N; ++u) step(held, kb[u]);
        }
        return held;
    };
    float2 start = {0.f, 0.f};
    if (works) {
        // the row before the first of the warm ones, or, exact, what the first row continues from (basis row or init)
        const int w = max(a - g.warm, 0);
        const Raw before = w == 0 ? ((Raw *)(rows - P))[p] : ((Raw *)(rows + (w - 1 + run_of(w - 1)) * P))[p];
        start = walk_rows(w, a, float2{first_of(before), second_of(before)});
        E[tid] = walk_rows(a, a + L, start);
    }
    __syncthreads();
    bool settled;                                                // (DL == 32: in as many rounds as there are runs it always is)
    for (int round = 0;; ++round) {
        float2 from = start;
        if (works && run > 0) from = E[tid - PR];
        const bool wrong = __float_as_uint(from.x) != __float_as_uint(start.x) || __float_as_uint(from.y) != __float_as_uint(start.y);
        if (__any(wrong) && (tid & 63) == 0) flags[round & 1] = 1;
        __syncthreads();                                         // (also: every run has read the end of the one before)
        settled = !flags[round & 1];
        if (settled || round == g.rounds) break;
        if (tid == 0) flags[(round + 1) & 1] = 0;
        if (wrong) {
            start = from;
            E[tid] = walk_rows(a, a + L, start);
        }
        __syncthreads();
    }
    // What is left, in order, a wave per channel: its lanes hold the rows of a run and say which of them fire, so that a row that does not fire costs
    // nothing (60 clocks a row that does, 60 a run; in a round 50 a row of the longest chain's run, and two barriers).
    if constexpr (kInOrder<DL>) {
        if (!settled) {
            if (works) S[tid] = start;
            __syncthreads();
            float *const ends = (float *)E;                      // [runs][DL]
            const float *const starts = (const float *)S;
            const int lane = tid & 63;
            for (int c = __builtin_amdgcn_readfirstlane(tid >> 6); c < DL; c += threads >> 6)
                runs_in_order(
                    runs, [&](int r) { return ends[r * DL + c]; }, [&](int r) { return starts[r * DL + c]; },
                    [&](int r, float end) { ends[r * DL + c] = end; },
                    [&](int r, int held) {
                        return fired_in(load_f32((const T *)(rows + (size_t)r * (L + 1) * P), (size_t)(min(lane, L - 1) * DL + c)), L, held, theta);
                    });
            __syncthreads();
            if (works && run > 0) start = E[tid - PR];
        }
    }
    if (works) {
        Raw *r = (Raw *)(rows + (size_t)run * (L + 1) * P) + p;
        Raw k[N];
        fetch(k, a);
        for (int t = a; t < a + L; t += N, r += N * PR) {
            Raw next[N];
            fetch(next, min(t + N, a + L - N));
#pragma unroll
            for (int u = 0; u < N; ++u) {
                step(start, k[u]);
                both(r[u * PR], start.x, start.y);
            }
#pragma unroll
            for (int u = 0; u < N; ++u) k[u] = next[u];
        }
    }
    __syncthreads();
    // a thread per row: reference keys and mask bits out
    uint32_t fired = 0;
    T *const Hp = g.Khat + (size_t)unit * g.ld * g.d + ch0;
    char *const Mp = (char *)g.mask_bits + (size_t)unit * n * (g.d / 8) + ch0 / 8;
    for (int t = tid; t < n; t += threads) {
        const int at = t + run_of(t), prev = t == 0 ? -1 : t - 1 + run_of(t - 1);
        uint32_t bits = 0;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const uint4 x = rows[at * P + q], y = rows[prev * P + q];
            ((uint4 *)Hp)[(size_t)t * gpr + q] = x;
            bits |= piece_bits<T>(x, y) << (kPer * q);
        }
        if (t == 0 && !g.init) bits = ~0u >> (32 - DL);          // the basis row is kept whole
        fired += (uint32_t)__popc(bits);
        char *const m = Mp + (size_t)t * (g.d / 8);
        if constexpr (DL == 8)
            *(uint8_t *)m = (uint8_t)bits;
        else if constexpr (DL == 16)
            *(uint16_t *)m = (uint16_t)bits;
        else
            *(uint32_t *)m = bits;
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) fired += __shfl_xor(fired, s);
    if ((tid & 63) == 0) atomicAdd(total, fired);
    __syncthreads();
    if (tid == 0) g.counts[(size_t)unit * groups + group] = *total;
}

__global__ __launch_bounds__(256) void nnz_sum_kernel(NnzSum sum) {
    add_up_nnz(sum, (int)(blockIdx.x * 32 + (threadIdx.x >> 3)));
}

constexpr int kSettleWaves = 16;                                 // a channel each
constexpr int kMostSegment = 384;                                // rows of a segment, where there are several, at most (scan_plan)
static_assert(kMostSegment % 64 == 0, "whole blocks of a wave's lanes");

// The reference keys, masks and counts of up to four segments of 16 channels again, one segment to 16 lanes: rows from t0 on (t1 - t0 are a segment's, `most` any one's) from `held`, where those
// there are from `spec`; `mine`: this lane's segment is one of them.  Until the two chains have met in every lane.
template <typename T>
__device__ __forceinline__ void rewalk_four(const T *Kp, T *Hp, uint16_t *Mp, int d, int t0, int t1, int most, float spec, float held, bool mine, float theta,
                                            long long *adjust) {
    const int lane = threadIdx.x & 63, sub = lane >> 4, at = lane & 15;
    bool synced = !mine || __float_as_uint(spec) == __float_as_uint(held);
    auto fetch = [&](T (&k)[U], int tb) {                        // rows past the end are clamped and not worked on
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = Kp[(size_t)min(t0 + tb + u, t1 - 1) * d];
    };
    auto work = [&](const T (&kk)[U], int tb) {
        uint32_t bits = 0;                                       // lane u of a segment's keeps the mask of its row tb + u
        for_batch([&](auto u) {
            const bool here = mine && t0 + tb + u < t1;
            const float k = to_f32(kk[u]);
            const bool fs = here && fabsf(k - spec) > theta, ft = here && fabsf(k - held) > theta;
            spec = fs ? k : spec;
            held = ft ? k : held;
            const uint64_t bt = __ballot(ft);
            *adjust += (long long)__popcll(bt) - (long long)__popcll(__ballot(fs));
            bits = at == u ? (sub & 2 ? (uint32_t)(bt >> 32) : (uint32_t)bt) >> (16 * (sub & 1)) : bits;
            if (here) store_exact(Hp, (size_t)(t0 + tb + u) * d, held);
        });
        synced = synced || __float_as_uint(spec) == __float_as_uint(held);   // (chains that have met stay together)
        if (mine && at < U && t0 + tb + at < t1) Mp[(size_t)(t0 + tb + at) * (d >> 4)] = (uint16_t)bits;
        return tb + U < most && __any(!synced);
    };
    T ka[U], kb[U];
    fetch(ka, 0);
    for (int tb = 0;; tb += 2 * U) {
        fetch(kb, tb + U);
        if (!work(ka, tb)) break;
        fetch(ka, tb + 2 * U);
        if (!work(kb, tb + U)) break;
    }
}

// What segments end on travels in order, a wave per channel (runs_in_order), 16 channels to a work group; then every segment whose start was another is
// walked again once, until it meets what stands there.  What bounds it is that walk's rows in a chain and, where most segments are wrong, the lines that the waves
// read one channel of.  Against rounds of walking 64 channels of a segment again, each up to 384 rows with their stores, and one wave that chased the ends where rounds
// did not help, scans back to back, us: 20 x 8192 rows of 128 34.3 / 33.7, at threshold 0.2 51.7 / 49.2, 1 % jumps 41.4 / 39.6, and 0.2 142.5 / 141.5, drift
// 451 / 230, nothing fires 637 / 251; 10 x 5003 21.7 / 21.2, 35.8 / 33.4, 30.9 / 29.0, 141 / 67, 382 / 101, 379 / 84; 5 x 65536, nothing fires, 5396 / 1528.
template <typename T>
__global__ __launch_bounds__(64 * kSettleWaves) void scan_settle_kernel(ScanArgs<T> g) {
    __shared__ unsigned long long total;
    const int group = blockIdx.x, unit = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = g.n, d = g.d, nseg = g.nseg, columns = (d + 63) / 64;
    const T *const Ku = g.K + (size_t)unit * n * d + group * 16;
    const T *const Hu = g.Khat + (size_t)unit * g.ld * d + group * 16;
    T *const su = g.starts + (size_t)unit * nseg * d + group * 16, *const eu = g.ends + (size_t)unit * nseg * d + group * 16;
    if (tid == 0) total = 0;
    unsigned long long sum = 0;
    if (group < columns)
        for (int s = tid; s < nseg; s += 64 * kSettleWaves) sum += g.counts[((size_t)unit * nseg + s) * columns + group];
    const bool found = runs_in_order(
        nseg, [&](int s) { return load_f32(eu, (size_t)s * d + wave); }, [&](int s) { return load_f32(su, (size_t)s * d + wave); },
        [&](int s, float end) { store_exact(eu, (size_t)s * d + wave, end); },
        [&](int s, int held) {
            // (two blocks of 64 rows first: most chains meet what stands there, which every round here pays for with 64 lines a block)
            const int t0 = s * g.S, rows = min(n - t0, g.S);
            const float stands = load_f32(Hu, (size_t)(t0 + min(127, rows - 1)) * d + wave), end = load_f32(eu, (size_t)s * d + wave);
            auto blocks = [&](auto from, auto to) __attribute__((always_inline)) {
                float k[to - from];
#pragma unroll
                for (int b = from; b < to; ++b) k[b - from] = load_f32(Ku, (size_t)(t0 + min(64 * b + lane, rows - 1)) * d + wave);
#pragma unroll
                for (int b = from; b < to; ++b) held = fired_in(k[b - from], rows - 64 * b, held, g.theta);
            };
            blocks(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
            if (held == __float_as_int(stands)) return __float_as_int(end);
            if (rows > 128) blocks(std::integral_constant<int, 2>{}, std::integral_constant<int, kMostSegment / 64>{});
            return held;
        });
    long long adjust = 0;
    if (__syncthreads_or(found)) {
        const int sub = lane >> 4, c = lane & 15;
        T *const Hp = g.Khat + (size_t)unit * g.ld * d + group * 16 + c;
        uint16_t *const Mp = (uint16_t *)(g.mask_bits + (size_t)unit * n * (d >> 5)) + group;
        for (int s0 = 1 + wave; s0 < nseg; s0 += 4 * kSettleWaves) {
            const int s = min(s0 + sub * kSettleWaves, nseg - 1);
            const float st = load_f32(su, (size_t)s * d + c), from = load_f32(eu, (size_t)(s - 1) * d + c);
            const uint64_t wrong = __ballot(s0 + sub * kSettleWaves < nseg && __float_as_uint(st) != __float_as_uint(from));
            if (wrong)
                rewalk_four(Ku + c, Hp, Mp, d, s * g.S, min(n, s * g.S + g.S), g.S, st, from, (wrong >> (16 * sub) & 0xffff) != 0, g.theta, &adjust);
        }
    }
    if (lane == 0) sum += (unsigned long long)adjust;
    if (sum) atomicAdd(&total, sum);
    __syncthreads();
    if (tid == 0) atomicAdd(g.nnz + unit, total);
}

// The value a segment's rows t0 .. t1 - 1 end on from `held`, without writing anything: once the chain meets the recorded one
// in every lane (Hp: its reference keys) it ends on the recorded end.  Only the compare and the select of Eq. 2-3 per row, 32
// rows in flight behind the 32 being walked.
template <typename T>
__device__ __forceinline__ float chase(const T *Kp, const T *Hp, int d, int t0, int t1, float held, float end, bool active,
                                       float theta) {
    constexpr int N = 32;
    auto fetch = [&](T (&k)[N + 1], int tb) {                    // (the last row again past the end: it fires once at most)
#pragma unroll
        for (int u = 0; u < N; ++u) k[u] = Kp[(size_t)min(tb + u, t1 - 1) * d];
        k[N] = Hp[(size_t)min(tb + N - 1, t1 - 1) * d];
    };
    auto work = [&](const T (&kk)[N + 1], int tb) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float k = to_f32(kk[u]);
            held = fabsf(k - held) > theta ? k : held;
        }
        if (!__any(active && __float_as_uint(held) != __float_as_uint(to_f32(kk[N])))) {
            held = end;
            return false;
        }
        return tb + N < t1;
    };
    T ka[N + 1], kb[N + 1];
    fetch(ka, t0);
    for (int tb = t0;; tb += 2 * N) {
        fetch(kb, tb + N);
        if (!work(ka, tb)) break;
        fetch(ka, tb + 2 * N);
        if (!work(kb, tb + N)) break;
    }
    return held;
}

// Where units are many and work groups of 16 channels would not all be resident: one of 64 channels per unit.
// Rounds of walking wrong segments again, in parallel, as long as every round leaves at most three quarters of them (which
// together is four rounds' work: a steady drift in 63 segments takes 47, 31, 15).  Where channels stay quiet over whole segments a round
// does not: an end value then travels one segment a round, and rounds until it arrives would make the time
// quadratic in the number of segments.  So the first wave settles what is left in order - it only chases the end values, each
// segment once - and one more round, which now has the right starts, writes.
// Scans, us, 5 % jumps / keys that drift steadily / nothing fires: 33 units x 8192 rows of 128 in bf16 44 .. 48 / 488 / 692 .. 716, 96 x 5304 of 64 47 / 461 / 450 .. 465, 300 x 2100 of 64
// 55 / 462 / 450 .. 462.  (Against rounds alone, on units so few that they settle in order now: where nothing fires, 20 x 8192 of 128, 64 segments, 2440 -> 677.)
template <typename T>
__global__ __launch_bounds__(64 * kSettleWaves) void scan_settle_rounds_kernel(ScanArgs<T> g) {
    __shared__ unsigned long long total;
    const int group = blockIdx.x, unit = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = g.n, d = g.d, nseg = g.nseg, wpr = d >> 5;
    const int c = group * kWave + lane, cs = min(c, d - 1), word = group * 2;
    const bool active = c < d;
    const T *Kp = g.K + (size_t)unit * n * d + cs;
    T *Hp = g.Khat + (size_t)unit * g.ld * d + cs;
    uint32_t *Mp = g.mask_bits + (size_t)unit * n * wpr + word;
    T *sp = g.starts + (size_t)unit * nseg * d + cs, *ep = g.ends + (size_t)unit * nseg * d + cs;
    if (tid == 0) total = 0;
    unsigned long long sum = 0;
    for (int s = tid; s < nseg; s += 64 * kSettleWaves) sum += g.counts[((size_t)unit * nseg + s) * gridDim.x + group];
    long long adjust = 0;
    constexpr int G = 4;                                         // segments whose boundary values are fetched together
    bool ordered = false;
    for (int before = 0x7fffffff;;) {
        int walked = 0;
        for (int sb = 1 + wave; sb < nseg; sb += G * kSettleWaves) {
            uint32_t wrong = 0;                                  // bit u: segment sb + u * kSettleWaves
            float st[G], pe[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const size_t s = min(sb + u * kSettleWaves, nseg - 1);
                st[u] = load_f32(sp, s * d);
                pe[u] = load_f32(ep, (s - 1) * d);
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                wrong |= (uint32_t)(sb + u * kSettleWaves < nseg && __any(active && __float_as_uint(st[u]) != __float_as_uint(pe[u]))) << u;
            walked += __popc(wrong);
            for (; wrong; wrong &= wrong - 1) {
                const int s = sb + __builtin_ctz(wrong) * kSettleWaves;
                const float from = load_f32(ep, (size_t)(s - 1) * d);
                const float e = rewalk(Kp, d, Hp, d, Mp, wpr, word + 1 < wpr, s * g.S, min(n, s * g.S + g.S),
                                       load_f32(sp, (size_t)s * d), from, load_f32(ep, (size_t)s * d), active, g.theta, &adjust);
                if (active) {
                    store_exact(sp, (size_t)s * d, from);
                    store_exact(ep, (size_t)s * d, e);
                }
            }
        }
        const int all = __syncthreads_count(lane < walked);      // (at most 64 a wave: a lower bound where segments are many)
        if (all == 0 || ordered) break;
        if (4ll * all > 3ll * before) {
            if (wave == 0) {
                float held = load_f32(ep, 0);                    // (the first segment is exact)
                for (int sb = 1; sb < nseg; sb += G) {
                    float st[G], en[G];
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        const size_t s = min(sb + u, nseg - 1);
                        st[u] = load_f32(sp, s * d);
                        en[u] = load_f32(ep, s * d);
                    }
#pragma unroll 1
                    for (int u = 0; u < G && sb + u < nseg; ++u) {
                        const float start = u == 0 ? st[0] : u == 1 ? st[1] : u == 2 ? st[2] : st[3];
                        const float end = u == 0 ? en[0] : u == 1 ? en[1] : u == 2 ? en[2] : en[3];
                        const size_t t0 = (size_t)(sb + u) * g.S;
                        if (__any(active && __float_as_uint(held) != __float_as_uint(start)))
                            held = chase(Kp, Hp, d, (int)t0, min(n, (int)t0 + g.S), held, end, active, g.theta);
                        else
                            held = end;
                        if (active) store_exact(ep, (size_t)(sb + u) * d, held);
                    }
                }
            }
            ordered = true;
            __syncthreads();
        }
        before = all;
    }
    if (lane == 0) sum += (unsigned long long)adjust;
    if (sum) atomicAdd(&total, sum);
    __syncthreads();
    if (tid == 0) atomicAdd(g.nnz + unit, total);
}

__global__ void fill_u64_kernel(unsigned long long *p, unsigned long long v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

int device_cu_count() {
    static std::atomic<int> cached[64];                          // per device ordinal; 0 = not asked yet
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return 256;
    }
    cus = cached[dev].load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
        (void)hipGetLastError();
        return 256;
    }
    cached[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

void launch_fill_u64(uint64_t *p, uint64_t v, int n, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(fill_u64_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (unsigned long long *)p,
                       (unsigned long long)v, n);
}

// A prompt whose rows fit into LDS is one segment: one work group of 8 waves per unit, one launch (one segment / cut, us a call: 8 x 256
// rows of 64 12.1 / 14.8, 8 x 512 12.6 / 14.6, 64 x 8 x 1024 43.4 / 50.2; at the line few units would rather be cut: 8 x 1024 16.5 /
// 15.1).  Longer ones are cut into segments of 128 rows, 64 channels and 4 waves per work group: with the 128 rows before them 35 KB
// of LDS (bf16), so that four work groups share a compute unit and cover each other's load, walk and store - or of 256 rows,
// which halves the rows walked twice, where that still leaves every compute unit three work groups (128 / 256 rows, bf16: 8 x 2048
// rows of 64 15.6 / 18.8, 5 x 4096 of 128 20.2 / 20.7, 20 x 4096 29.5 / 25.6 - below the line already -, 20 x 8192 41.7 / 39.0, 40 x 8192
// 62.9 / 57.6), or of 384 rows and 8 waves where that still holds and the settling waves have a segment each.  256 / 384, two builds in
// turn, medians of 12, each within 1 %: 20 x 8192 36.6 / 34.6, 20 x 16384 56.2 / 52.3, 40 x 8192 of 64 37.4 / 34.7, 24 x 6144 33.9 / 32.4, 5 x 65536
// 59.6 / 55.8; over 144 launches (12 shapes, 1 / 5 / 20 % jumps, thresholds 0.06 to 0.23) 5.5 % faster on the geometric mean.  Where nearly all
// guesses hold that is 3 to 9 %; where many segments are walked again the time hangs on which ones happen to be wrong, -17 to +39 %; keys that never
// fire -13 (64 x 6144) to +4 %.  Shorter prompts lose what settling then takes longer, 128 x 3000 of 64 127 / 143.  In fp32 a work group of 256 + 128 rows is alone on its compute unit, and 128 rows are as good or better from 16
// units up (32 x 4000 rows of 128: 52.7 / 56.8), unless most guesses are wrong (32 x 8000 rows of 64 that drift slowly: 328 / 248).
static ScanPlan scan_plan(int dtype, int units, int n, int d) {
    const int es = dtype == 0 ? 4 : 2;
    ScanPlan p;
    const bool one = (int64_t)n * d * es <= 128 * 1024;
    p.warm = 128;
    const int64_t columns = (int64_t)units * ((d + 63) / 64), cus = device_cu_count();
    const bool longest = !one && es == 2 && columns * (n / kMostSegment) >= 3 * cus && n >= kMostSegment * kSettleWaves;
    p.S = one ? n : longest ? kMostSegment : columns * (n / 256) >= 3 * cus ? 256 : 128;
    p.nseg = (n + p.S - 1) / p.S;
    p.dl = one ? d : 64;
    p.waves = one || longest ? 8 : 4;
    const int dl = p.dl < d ? p.dl : d, TW = p.waves / ((dl + kWave - 1) / kWave);
    const size_t rows = one ? n : p.S + p.warm;
    p.lds = rows * dl * es + (size_t)p.S * (dl / 32) * 4 + (size_t)TW * dl * 4 + 16;
    return p;
}

size_t delta_scan_scratch_bytes(int dtype, int units, int n, int d) {
    const ScanPlan p = scan_plan(dtype, units, n, d);
    // (room as for segments of 256 rows where they are longer: callers size their buffers by it, and it has been that)
    const int S = p.S > 256 ? 256 : p.S;
    const size_t segs = (size_t)units * ((n + S - 1) / S);
    return p.nseg == 1 ? 0 : 2 * segs * d * (dtype == 0 ? 4 : 2) + segs * ((d + 63) / 64) * 4;
}

template <typename T>
static void scan_typed(const ScanPlan &p, const void *K, void *Khat, uint32_t *mask_bits, void *scratch, uint64_t *nnz,
                       int units, int n, int d, float theta, const void *init, uint32_t *zeroed, const RowCopy *copy, hipStream_t s) {
    const size_t segs = (size_t)units * p.nseg;
    T *starts = (T *)scratch;
    const ScanArgs<T> a = {(const T *)K, (T *)Khat, mask_bits, starts, starts + segs * d, (uint32_t *)(starts + 2 * segs * d),
                           (unsigned long long *)nnz, (const T *)init, zeroed, n, d, p.S, p.nseg, p.warm, p.dl, theta,
                           copy ? copy->ld : n};
    const int groups = (d + p.dl - 1) / p.dl;
    const int which = p.dl == 128 ? 2 : p.dl == 64 && d % 64 == 0 ? 1 : 0;
    static std::atomic<uint64_t> lds_set[6];                     // per instantiation, one bit per device
    const dim3 block(64 * p.waves);
    if constexpr (sizeof(T) == 2) {
        if (copy) {                                              // (what is fed in pieces is bf16, of 64 or 128 channels)
            const auto kernel = which == 2 ? scan_segments_kernel<T, 128, RowCopy> : scan_segments_kernel<T, 64, RowCopy>;
            ensure_dynamic_lds((const void *)kernel, kScanLdsMax, lds_set[3 + which]);
            hipLaunchKernelGGL(kernel, dim3(p.nseg, units, groups + 1), block, p.lds, s, a, *copy);
        }
    }
    if (!copy) {
        const auto kernel = which == 2 ? scan_segments_kernel<T, 128> : which == 1 ? scan_segments_kernel<T, 64> : scan_segments_kernel<T, 0>;
        ensure_dynamic_lds((const void *)kernel, kScanLdsMax, lds_set[which]);
        hipLaunchKernelGGL(kernel, dim3(p.nseg, units, groups), block, p.lds, s, a);
    }
    // In order with 16 channels a work group while each has a compute unit / in rounds with 64 beyond, scans back to back, us: 64 x 6144 rows of 64 37.6 / 38.4, at
    // threshold 0.2 67.9 / 73.0; 33 x 8192 of 128 (264 work groups) 49.6 / 48.2 and 72.4 / 75.4, 96 x 5304 of 64 48.7 / 47.6 and 69.5 / 71.6, 300 x 2100 59.1 / 55.4 and
    // 91.6 / 89.9.  (In order with 64 a work group 57.0 and 114.9 there.)
    if (p.nseg > 1 && (int64_t)units * (d / 16) <= device_cu_count())
        hipLaunchKernelGGL(scan_settle_kernel<T>, dim3(d / 16, units), dim3(64 * kSettleWaves), 0, s, a);
    else if (p.nseg > 1)
        hipLaunchKernelGGL(scan_settle_rounds_kernel<T>, dim3((d + 63) / 64, units), dim3(64 * kSettleWaves), 0, s, a);
}

// What a launch of scan_whole_kernel looks like; L == 0: the prompt is none for it.
struct WholePlan {
    int dl, threads, L, warm, rounds;
    size_t lds;
};
// Few channels per work group where there are few units, more where the work groups would not all be resident (every work group reads
// whole cache lines); rows of at most 64 KB in LDS, so that two share a compute unit; runs of at most kMostRun rows, in
// twice the threads where 256 would have longer ones.
// The rows a run warms up on save rounds where every work group has a compute unit to itself and are only work where it has not.
// One launch here / segments, and their settling where there are several, us, without the 1.5 us between these two (5 % jumps): 8 x 333 rows of 64 6.5 / 9.1,
// 80 x 200 of 128 9.4 / 10.3, 8 x 1024 of 64 9.2 / 13 - 16, 8 x 2048 of 64 11.5 / 14 + 3.9, 10 x 1024 of 128 8.5 / 10 + 3.8, 5 x 4096 of 128
// 15.7 / 12.5 + 4.8, 20 x 4096 24.5 / 22 + 4.9, 160 x 700 20.9 / 25.6 + 5.4, 256 x 2048 of 64 39.9 / 43.8 + 4.8; fp32, 1 x 256 rows of 64 5.0 / 7.5, 4 x
// 1000 7.1 / 9.3 + 3.8, 16 x 2000 of 128 15.8 / 13.7 + 4.3.  Beyond, 10 x 5003 rows of 128 (80 KB a work group) 23.5 / 14.6 + 4.8.  Where more guesses are wrong, calls with scans in rounds
// alone / settling in order, us: 1 % jumps and threshold 0.2, 8 x 2048 of 64 68.0 / 44.0, 10 x 1024 of 128 49.5 / 37.3, 20 x 4096 145 / 135, 160 x 700 98 / 88, 256 x 2048 of
// 64 274 / 254; where nothing fires for the whole prompt 143 / 44, 77 / 38, 311 / 130, 101 / 74, 391 / 244; keys that drift 113 / 49, 80 / 49, 354 / 179,
// 122 / 119, 424 / 293.
// Where there are about as many units as compute units (three quarters and more), and one's rows are 64 to 128 KB, a work group per unit reads whole rows and
// needs no second wave of work groups: 256 x 700 rows of 64 18.7 here / 17.2 there, 256 x 400 of 128 19.9 / 17.2, 200 x 900 of 64 18.4 / 16.7, 256 x 1000 22.5 /
// 23.4; but 256 x 400 of 64 13.3 / 19.0, 160 x 500 of 128 16.5 / 17.4.
constexpr int kMostRun = 32;
static_assert(kMostRun <= kWave, "where runs settle in order the lanes of a wave hold one's rows (fired_in)");
static WholePlan whole_plan(int dtype, int units, int n, int d) {
    const int es = dtype == 0 ? 4 : 2;
    const int64_t cus = device_cu_count();
    WholePlan p = {8, 256, 0, 0, 0, 0};
    if (n < 64 || (int64_t)n * p.dl * es > 64 * 1024) return p;
    if (4 * (int64_t)units >= 3 * cus && (int64_t)n * d * es > 64 * 1024 && (int64_t)n * d * es <= 128 * 1024) return p;
    const auto groups = [&](int dl) { return (int64_t)units * (d / dl); };
    if (groups(8) > 2 * cus) p.dl = 16;
    if ((int64_t)n * p.dl * es > 64 * 1024) return p;            // (8 channels at a time read lines too often there: 88 x 2958 of 128 55 / 46)
    if (p.dl == 16 && groups(16) > 2 * cus && n <= 512) p.dl = 32;
    p.threads = n > kMostRun * (256 / (p.dl / 2)) ? 512 : 256;      // (64 KB are 4096 rows of 8 channels at most: 128 runs)
    const int runs = p.threads / (p.dl / 2);
    p.L = ((n + runs - 1) / runs + 7) / 8 * 8;
    p.warm = groups(p.dl) <= cus ? 48 : 32;
    // (A wave per channel settles, where it takes no other work group's time: a batch of 150 x 700 rows of 128 74.5 us a call with 4 waves, 77 with 8.)
    if (p.dl == 8 && n > 64 && groups(8) <= cus) p.threads = 512;
    // One round first / none: 8 x 2048 rows of 64 12.5 / 12.0 (1 % jumps 13.0 / 12.6, and threshold 0.2 17.0 / 17.8), 10 x 1024 of 128 30.4 / 30.5 a call; where a wave has
    // many runs or channels, 5 x 4096 of 128 17.5 / 17.3 (17.9 / 17.8, 23.8 / 27.1), 150 x 700 of 128 74.5 / 77.4 a call.  Rounds alone where they are short
    // and a wave would have 4 or 8 channels (appends, rounds / one and in order: 162 x 64 rows of 64 20.3 / 21.9, 72 x 80 of 128 41.8 / 45.3, 80 x 119 of 64 54.0 / 54.7; but 55 x 226 of 128 120.5 / 115.8).
    p.rounds = p.dl == 32 || n <= (p.dl == 16 ? 128 : 64) ? runs : groups(p.dl) > cus || n > 2048;
    const int used = (n + p.L - 1) / p.L;
    p.lds = (size_t)(used * (p.L + 1) + 1) * p.dl * es + (size_t)used * p.dl * (p.dl == 32 ? 4 : 8) + 16;   // (kInOrder)
    return p;
}

template <typename T, int DL>
static void whole_typed(const WholeArgs<T> &a, const WholePlan &p, const RowCopy *copy, hipStream_t s) {
    static std::atomic<uint64_t> lds_set[2];                     // per instantiation, one bit per device
    if constexpr (sizeof(T) == 2) {
        if (copy) {
            ensure_dynamic_lds((const void *)scan_whole_kernel<T, DL, RowCopy>, kScanLdsMax, lds_set[1]);
            const unsigned blocks = (unsigned)a.blocks + (unsigned)copy->units * (unsigned)((copy->rows + 63) / 64);
            hipLaunchKernelGGL((scan_whole_kernel<T, DL, RowCopy>), dim3(blocks), dim3(p.threads), p.lds, s, a, *copy);
            return;
        }
    }
    ensure_dynamic_lds((const void *)scan_whole_kernel<T, DL>, kScanLdsMax, lds_set[0]);
    hipLaunchKernelGGL((scan_whole_kernel<T, DL>), dim3((unsigned)a.blocks), dim3(p.threads), p.lds, s, a);
}
template <typename T>
static void whole_scan(const WholePlan &p, const void *K, void *Khat, uint32_t *mask_bits, uint32_t *counts, int units, int n, int d,
                       float theta, const void *init, uint32_t *zeroed, const RowCopy *copy, hipStream_t s) {
    uint32_t l = 0;
    while ((1u << l) < (uint32_t)p.L) ++l;
    const WholeArgs<T> a = {(const T *)K, (T *)Khat, mask_bits, counts, (const T *)init, zeroed, units, n, d, p.L, p.warm,
                            (uint32_t)((((uint64_t)1 << (31 + l)) / (uint64_t)p.L) + 1u), l, theta,
                            copy ? copy->ld : n, 8 * (d / p.dl) * ((units + 7) / 8), p.rounds};
    if (p.dl == 8)
        whole_typed<T, 8>(a, p, copy, s);
    else if (p.dl == 16)
        whole_typed<T, 16>(a, p, copy, s);
    else
        whole_typed<T, 32>(a, p, copy, s);
}

// Khat [units][n][d] and scratch (delta_scan_scratch_bytes) are required scratch/outputs.
NnzSum launch_delta_scan(int dtype, const void *K, void *Khat, uint32_t *mask_bits, void *scratch, uint32_t *counts, uint64_t *nnz,
                         int units, int n, int d, float theta, hipStream_t s, const void *init, uint32_t *zeroed, const RowCopy *copy) {
    const WholePlan w = whole_plan(dtype, units, n, d);
    if (counts && w.L > 0) {
        if (dtype == 0)
            whole_scan<float>(w, K, Khat, mask_bits, counts, units, n, d, theta, init, zeroed, copy, s);
        else
            whole_scan<bf16_t>(w, K, Khat, mask_bits, counts, units, n, d, theta, init, zeroed, copy, s);
        return NnzSum{counts, nnz, d / w.dl, units};
    }
    const ScanPlan p = scan_plan(dtype, units, n, d);
    if (dtype == 0)
        scan_typed<float>(p, K, Khat, mask_bits, scratch, nnz, units, n, d, theta, init, zeroed, copy, s);
    else
        scan_typed<bf16_t>(p, K, Khat, mask_bits, scratch, nnz, units, n, d, theta, init, zeroed, copy, s);
    return NnzSum{};
}

void launch_nnz_sum(const NnzSum &sum, hipStream_t s) {
    if (sum.groups > 0) hipLaunchKernelGGL(nnz_sum_kernel, dim3((sum.units + 31) / 32), dim3(256), 0, s, sum);
}

bool delta_scan_settles(int dtype, int units, int n, int d) { return scan_plan(dtype, units, n, d).nseg > 1; }

}  // namespace da
