// Device code of the delta matrix construction (Sec. II-C Eq. 2-3; Sec. III-A strategy 3), shared by the stand-alone
// kernels and by the fused short-prompt prefill kernel.
#pragma once
#include "common.hpp"

namespace da {

// Eq. 2-3 over rows t0 .. t1 - 1 of one unit for the 64 channels c = 64 * channel_wave + lane, by one wave.
//   first   : the rows start a sequence or continue one: row t0 is then the basis row (kept whole), or, with `init`
//             given, the first row after the reference key init[c]
//   !first  : the scan starts from `start` (the held value before row t0)
// kFinal: mask words, reference keys (Hp) are written and surviving entries counted into *count; otherwise only the
// held value at the end is returned (a speculative pass).
template <typename T, bool kFinal>
__device__ __forceinline__ float scan_rows(const T *__restrict__ Kp, T *__restrict__ Hp, uint32_t *__restrict__ Mp,
                                           int d, int c, int lane, int t0, int t1, bool first, const T *init_row,
                                           float start, float theta, unsigned long long *count) {
    const bool active = c < d;
    const int wpr = d >> 5;
    const bool writer = active && ((lane & 31) == 0);
    const int word = c >> 5;
    const int cs = active ? c : 0;
    // The held value is always a verbatim copy of a key element (or of the incoming state): its stored form is
    // carried along beside the binary32 value the comparison uses, so that storing a reference key converts nothing.
    float held = start;
    T held_raw = from_f32<T>(start);
    unsigned long long cnt = 0;
    int t = t0;
    if (first && init_row) {   // the rows continue a sequence: its reference key is the incoming state
        held_raw = init_row[cs];
        held = to_f32(held_raw);
    } else if (first) {        // row t0 is the basis: kept whole
        held_raw = Kp[(size_t)t0 * d + cs];
        held = to_f32(held_raw);
        if (kFinal) {
            if (active) Hp[(size_t)t0 * d + c] = held_raw;
            if (writer) Mp[(size_t)t0 * wpr + word] = 0xffffffffu;
            cnt = __popcll(__ballot(active));
        }
        t = t0 + 1;
    }
    // Rows in batches of U; two register sets alternate, the next batch is requested before the current one is
    // worked on (loads past the end are clamped to the last row and never used), so that a batch's memory
    // latency is hidden behind the previous batch's arithmetic instead of being paid once per batch.  The mask
    // words of a batch are collected in registers (lane u of each half keeps the word of row u) and stored once.
    constexpr int U = 16;
    auto load_batch = [&](T (&k)[U], int tb) {
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = Kp[(size_t)min(tb + u, t1 - 1) * d + cs];
    };
    auto work_batch = [&](const T (&k)[U], int tb) {
        uint32_t my_word = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float kf = to_f32(k[u]);
            const float diff = kf - held;                    // Eq. 2 condition in binary32
            const bool fire = active && (fabsf(diff) > theta);
            held = fire ? kf : held;                          // Eq. 3
            held_raw = fire ? k[u] : held_raw;
            if (kFinal) {
                const uint64_t b = __ballot(fire);
                my_word = ((lane & 31) == u) ? (uint32_t)(b >> (lane & 32)) : my_word;
                if (active) Hp[(size_t)(tb + u) * d + c] = held_raw;
                cnt += __popcll(b);
            }
        }
        if (kFinal && active && (lane & 31) < U) Mp[(size_t)(tb + (lane & 31)) * wpr + word] = my_word;
    };
    if (t + U <= t1) {
        T ka[U], kb[U];
        load_batch(ka, t);
        while (t + U <= t1) {
            load_batch(kb, t + U);
            work_batch(ka, t);
            t += U;
            if (t + U > t1) break;
            load_batch(ka, t + U);
            work_batch(kb, t);
            t += U;
        }
    }
    for (; t < t1; ++t) {
        const T kr = Kp[(size_t)t * d + cs];
        const float k = to_f32(kr);
        const bool fire = active && (fabsf(k - held) > theta);
        held = fire ? k : held;
        held_raw = fire ? kr : held_raw;
        if (kFinal) {
            const uint64_t b = __ballot(fire);
            if (writer) Mp[(size_t)t * wpr + word] = (uint32_t)(b >> (lane & 32));
            if (active) Hp[(size_t)t * d + c] = held_raw;
            cnt += __popcll(b);
        }
    }
    if (kFinal) *count = cnt;
    return held;
}

}  // namespace da
