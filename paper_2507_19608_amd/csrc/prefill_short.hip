// Short prompts in bf16, head_dim 64 or 128: delta scan and hybrid attention (Eq. 2-4, Eq. 1) in one launch.
//
// All of a unit's keys, reference keys and values fit into one LDS (up to 416 rows of 64, 200 of 128), so a work group takes them in
// once, builds the reference keys there and walks its share of the score rows with no barrier and no load between: neither K_hat
// nor a second launch goes through memory.  Several work groups share a unit's score rows; each scans the unit's keys for itself.
//
// What bounds it is latency.  16 x 200 tokens, 20 / 5 heads of 128, us after the first work group's start: all have their keys at 2.3, have walked their runs at
// 6.4, have their reference keys at 7.1, the first items end at 9.7 to 14.5 (4.0 to 7.8 each: the two waves of a SIMD share its matrix cores), second ones
// at 13.4, masks and the launch at 15.3.  Times here and below: calls in a graph, 5 % jumps, theta 0.1113, mean of six inputs.  Two launches (delta_scan.hip,
// prefill_mfma.hip) / this one: 32 / 8 heads of 64, 1 x 64 tokens 12.0 / 6.6, 1 x 333 16.0 / 9.7, 64 x 200 68.8 / 41.2, 32 x 400 70.9 / 47.5; 20 / 5 heads of 128, 1 x
// 200 18.2 / 11.3, 16 x 200 31.5 / 17.2, 256 x 200 301 / 173; over 76 shapes of 1 to 416 tokens, 1 to 256 prompts and six kinds of heads (an earlier
// build, one input each) 1.04 to 2.4 times as fast, 1.75 on the geometric mean: there is no line inside the range.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace da {

namespace {

typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef __attribute__((address_space(3))) uint32_t *lds_word;
typedef __attribute__((address_space(3))) uint16_t *lds_half;

constexpr int NW = 8;                    // waves of a work group
constexpr int kScanWaves = 4;            // of these walk keys, one a SIMD (eight waves and shorter runs took as long at 16 x 200 tokens, within 1 %)
template <int D> constexpr int kMostRows = D == 64 ? 416 : 200;              // so that three arrays fit (short_lds)

struct ShortArgs {
    const bf16_t *__restrict__ Q;
    const bf16_t *__restrict__ K;
    const bf16_t *__restrict__ V;
    bf16_t *__restrict__ O;
    bf16_t *__restrict__ Khat;           // NULL, or where reference keys go too
    uint32_t *__restrict__ mask_bits;
    uint64_t *__restrict__ nnz;
    int Hq, n, W, sliding;
    int units, g;                        // batch x KV heads; query heads per KV head
    int rt_log2;                         // an item is this many rows of 32 >> rt_log2 heads
    int row_groups, items;               // of a unit
    int parts, mask_part;                // work groups that share a unit's items; the one that writes its mask
    int L0, L, warm;                     // rows of the scan's first run, of a later one, and before that: multiples of 8
    Divisor by_units, by_hkv, by_hgroups, by_w;
    float scale_log2, theta;
};

// wait_loads<n>() for n known at run time, at most 7
__device__ __forceinline__ void wait_loads_but(int n) {
    switch (n) {
        case 7: return wait_loads<7>();
        case 6: return wait_loads<6>();
        case 5: return wait_loads<5>();
        case 4: return wait_loads<4>();
        case 3: return wait_loads<3>();
        case 2: return wait_loads<2>();
        case 1: return wait_loads<1>();
        default: return wait_loads<0>();
    }
}

// kSplit: waves that share an item's keys, alternate blocks of 64 each, and meet at the end
template <int D, int kSplit>
__global__ __launch_bounds__(64 * NW, 2) void prefill_short_kernel(ShortArgs a) {
    constexpr int kRowB = 2 * D, kSeg = D / 8, kRpl = 64 / kSeg;    // bytes and 16-byte segments of a row; rows of a 1 KiB load
    constexpr int KS = D / 16, MT = D / 32;
    constexpr int kRuns = kScanWaves * 64 / D;                   // runs of the scan
    constexpr uint32_t kDist = kMostRows<D> * kRowB;             // from a key to its reference key (an instruction's own offset)
    constexpr int kGroups = NW / kSplit;                         // of waves that take an item
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    typedef __attribute__((address_space(3))) u32x4 *lds_vec;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, li = lane & 31;
    const int n = a.n;
    const int part = quotient((int)blockIdx.x, a.by_units), unit = (int)blockIdx.x - part * a.units;
    const int b = quotient(unit, a.by_hkv), hk = unit - b * a.by_hkv.d;
    // LDS: keys, reference keys (kDist behind), values (the last row again up to a multiple of 8, of 32 for values), what runs of the scan
    // end on, words.
    // A row's segments are permuted by its number so that the reads are free of bank conflicts.
    const int nk = (n + 7) & ~7, nv = (n + 31) & ~31;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)lds_raw;
    const uint32_t k_at = lds0, h_at = k_at + kDist, v_at = h_at + nk * kRowB, e_at = v_at + nv * kRowB;
    uint32_t *const words = (uint32_t *)(lds_raw + (e_at - lds0) + kScanWaves * 256);   // [2] some run was wrong, [2] next item, [3] fired entries
    auto keys_perm = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
    auto vals_perm = [](int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };

    // ---- requests: keys and values
    const char *const Kp = (const char *)(a.K + (size_t)unit * n * D);
    const char *const Vp = (const char *)(a.V + (size_t)unit * n * D);
    int v_loads = 0;
    for (int j = wave; j < (nk + kRpl - 1) / kRpl; j += NW) {
        const int row = j * kRpl + lane / kSeg;
        load_to_lds<0>(Kp, (uint32_t)(min(row, n - 1) * kRowB + (((lane % kSeg) ^ keys_perm(row)) << 4)), k_at + j * 1024);
    }
    for (int j = wave; j < nv / kRpl; j += NW, ++v_loads) {
        const int row = j * kRpl + lane / kSeg;
        load_to_lds<0>(Vp, (uint32_t)(min(row, n - 1) * kRowB + (((lane % kSeg) ^ vals_perm(row)) << 4)), v_at + j * 1024);
    }
    // an item: RT consecutive rows of GH heads, 32 score rows; the last rows come first
    const int count = part < a.parts ? (a.items - part + a.parts - 1) / a.parts : 0;
    const int RT = 1 << a.rt_log2;
    const size_t q_at = ((size_t)b * a.Hq + hk * a.g) * n * D;
    const char *const Qp = (const char *)(a.Q + q_at);
    char *const Op = (char *)(a.O + q_at);
    u32x4 q[KS];
    int row0 = 0, my_row = 0;                                    // of the item: its first row, this lane's
    uint32_t my_at = 0;                                          // this lane's row in Qp and Op, bytes
    auto open = [&](int i) __attribute__((always_inline)) {
        const int it = part + i * a.parts;
        const int down = quotient(it, a.by_hgroups), hg = it - down * a.by_hgroups.d;
        row0 = (a.row_groups - 1 - down) << a.rt_log2;
        my_row = min(row0 + (li & (RT - 1)), n - 1);
        my_at = (uint32_t)(((hg << (5 - a.rt_log2)) + (li >> a.rt_log2)) * n + my_row) * kRowB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q[ks] = *(const u32x4_any *)(Qp + my_at + half * 16 + ks * 32);
    };
    const int at_first = wave / kSplit;
    if (tid < 4) words[tid] = tid == 2 ? kGroups : 0;

    // ---- Eq. 2-3.  A thread walks one run of rows in one channel.  Runs after the first start from the guess "held =
    //      the row before" some rows earlier; one whose guess was wrong walks again, until it meets what it has written.  (Two neighbouring channels a thread and
    //      twice the runs, of equal length, walk more warm rows than others: 16 x 200 tokens of 20 / 5 heads of 128 17.9 / 17.2 us, 1 x 333 of 32 / 8 of 64
    //      10.7 / 10.1, 14 shapes and five kinds of keys 1.066 on the geometric mean, the least at 416 rows that fire often, 10.76 / 10.87.)
    {
        wait_loads_but(v_loads);
        lds_barrier();
        if (at_first < count) open(at_first);                    // (these have the scan's time to come)
        const float theta = a.theta;
        const int run = tid / D, ch = tid % D;
        const int r0 = run == 0 ? 0 : a.L0 + (run - 1) * a.L, r1 = min(run == 0 ? a.L0 : r0 + a.L, nk);
        const bool works = run < kRuns && r0 < n;
        const lds_word ends = (lds_word)(uintptr_t)e_at;
        auto at_row = [&](int t) { return k_at + (uint32_t)(t * kRowB + (((ch >> 3) ^ keys_perm(t)) << 4) + (ch & 7) * 2); };
        auto load = [](uint32_t at) { return (uint32_t)*(lds_half)(uintptr_t)at << 16; };
        constexpr int B = 8;                                     // rows in a batch (the permutation of rows repeats after two)
        float x;
        auto walk = [&](auto writes, auto meets, int t, int end) __attribute__((always_inline)) {
            uint32_t at[2][B], key[2][B], base = at_row(t);
            // row u of a batch: the segment's permutation is the batch's and, exclusive, u's
            auto read = [&](int h) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    at[h][u] = base ^ (keys_perm(u) << 4);
                    key[h][u] = *(lds_half)(uintptr_t)(at[h][u] + u * kRowB);
                }
                base = (base ^ (keys_perm(B) << 4)) + B * kRowB;
                asm volatile("" ::: "memory");                   // (here, and not where they are used)
                __builtin_amdgcn_sched_barrier(0);
            };
            auto work = [&](int h) __attribute__((always_inline)) {
                uint32_t old = 0;
                if (meets) old = load(at[h][B - 1] + (B - 1) * kRowB + kDist);
                auto put = [&](int u) __attribute__((always_inline)) { *(lds_half)(uintptr_t)(at[h][u] + u * kRowB + kDist) = (uint16_t)(__float_as_uint(x) >> 16); };
                float kx = __uint_as_float(key[h][0] << 16), kn = 0.f;
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    // Eq. 2 in binary32, Eq. 3 (the select waits two states for its mask: what else there is to do comes between, 1.02)
                    const bool f = fabsf(kx - x) > theta;
                    __builtin_amdgcn_sched_barrier(0);
                    if (u + 1 < B) kn = __uint_as_float(key[h][u + 1] << 16);
                    if (writes && u > 0) put(u - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    x = f ? kx : x;
                    kx = kn;
                }
                if (writes) put(B - 1);
                t += B;
                return t < end && !(meets && !__any(__float_as_uint(x) != old));
            };
            read(0);
            while (true) {
                read(1);
                if (!work(0)) break;
                read(0);
                if (!work(1)) break;
            }
            return t;
        };
        constexpr std::true_type yes;
        constexpr std::false_type no;
        float start = 0.f;
        if (works) {
            const int w = max(r0 - a.warm, 0);
            start = x = __uint_as_float(load(at_row(max(w - 1, 0))));
            if (w < r0) {
                walk(no, no, w, r0);
                start = x;
            }
            walk(yes, no, r0, r1);
            ends[tid] = __float_as_uint(x);
        }
        lds_barrier();
        for (int round = 0; round < kRuns; ++round) {
            float from = start;
            if (works && run > 0) from = __uint_as_float(ends[tid - D]);
            const bool wrong = __float_as_uint(from) != __float_as_uint(start);
            if (__any(wrong) && lane == 0) words[round & 1] = 1;
            lds_barrier();
            if (!words[round & 1]) break;
            if (tid == 0) words[(round + 1) & 1] = 0;
            if (__any(wrong) && works) {
                start = x = from;
                if (walk(yes, yes, r0, r1) >= r1) ends[tid] = __float_as_uint(x);
            }
            lds_barrier();
        }
    }
    wait_loads<0>();                                             // the values
    lds_barrier();

    // ---- score rows
    // per-lane addresses inside an array of rows: every read below is one of these, an exclusive-or of a few bits, a constant
    const uint32_t k_lane = li * kRowB + ((half ^ keys_perm(li)) << 4);
    const int lq = lane & 15, lg = (lane >> 4) & 1;
    const uint32_t v_lane = v_at + (4 * half + (lq >> 2)) * kRowB + (vals_perm(lq >> 2) << 4) + lg * 32 + (lq & 3) * 8;
    auto win_start = [&](int r) { return a.sliding ? max(r - a.W + 1, 0) : quotient(r, a.by_w) * a.W; };
    constexpr int kAhead = D == 64 ? 4 : 5;
    f32x16 o[MT];
    float m_run, l_run[4];
    auto attend = [&](auto next_item) __attribute__((always_inline)) {
        const int split = kSplit == 1 ? 0 : wave % kSplit;
        const int first = row0, last = min(row0 + RT - 1, n - 1);
        const int row = my_row, my_win = win_start(row), win_first = win_start(first), win_last = win_start(last);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[mt][r] = 0.f;
        m_run = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) l_run[k] = 0.f;
        // 32 NT keys from column c0 on
        auto block = [&](auto tiles, int c0, bool ends) __attribute__((always_inline)) {
            constexpr int NT = tiles;
            f32x16 s[NT];
            auto product = [&](f32x16 &acc, bf16x8 op, int ks) {
                if (ks == 0) {
                    f32x16 zero;
#pragma unroll
                    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, __builtin_bit_cast(bf16x8, q[ks]), zero, 0, 0, 0);
                } else
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, __builtin_bit_cast(bf16x8, q[ks]), acc, 0, 0, 0);
            };
            // K_hat where some row has the tile's columns left of its window, else K
            uint32_t from[NT];
#pragma unroll
            for (int T = 0; T < NT; ++T) from[T] = (c0 + 32 * T < win_last ? h_at : k_at) + (c0 + 32 * T) * kRowB + k_lane;
            {
                bf16x8 op[NT * KS];
                for_each_index<NT * KS + kAhead>([&](auto j) {
                    if constexpr (j >= kAhead) product(s[(j - kAhead) % NT], op[j - kAhead], (j - kAhead) / NT);
                    if constexpr (j < NT * KS) op[j] = *(const __attribute__((address_space(3))) bf16x8 *)(uintptr_t)(from[j % NT] ^ ((j / NT) << 5));
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            if constexpr (NT == 1) {
                if (c0 < win_last && c0 + 32 > win_first) {      // some row has part of the tile inside its window, some left of it
                    f32x16 x;
                    const uint32_t keys = k_at + c0 * kRowB + k_lane;
                    bf16x8 op[KS];
                    for_each_index<KS + kAhead>([&](auto j) {
                        if constexpr (j >= kAhead) product(x, op[j - kAhead], j - kAhead);
                        if constexpr (j < KS) op[j] = *(const __attribute__((address_space(3))) bf16x8 *)(uintptr_t)(keys ^ (j << 5));
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    // (a bit spread over the word chooses, see the other prefill kernel's masks)
                    const int skip = min(max(my_win - c0, 0), 32);
                    const uint32_t inside = (skip < 32 ? ~0u << skip : 0u) >> (4 * half);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const uint32_t take = (uint32_t)__builtin_amdgcn_sbfe((int)inside, 8 * (r >> 2) + (r & 3), 1);
                        s[0][r] = __uint_as_float((__float_as_uint(x[r]) & take) | (__float_as_uint(s[0][r]) & ~take));
                    }
                }
            }
            if (ends) next_item();                               // (the queries are done with)
            if (c0 + 32 * NT > first + 1) {                      // some row does not see all of it
                const int to = min(max(row + 1 - c0, 0), 32 * NT);
                const uint64_t seen = (to > 0 ? ~(uint64_t)0 >> (64 - to) : 0) >> (4 * half);
#pragma unroll
                for (int T = 0; T < NT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const uint32_t take = (uint32_t)__builtin_amdgcn_sbfe((int)(uint32_t)(seen >> (32 * T)), 8 * (r >> 2) + (r & 3), 1);
                        s[T][r] = __uint_as_float((__float_as_uint(s[T][r]) & take) | (0xff800000u & ~take));
                    }
            }
            // online softmax, as in the other prefill kernel
            auto max3 = [](float x, float y, float z) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z); };
            float mx[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                mx[k] = max3(s[0][k], s[0][k + 4], s[0][k + 8]);
                mx[k] = NT == 1 ? __builtin_elementwise_maximum(mx[k], s[0][k + 12]) : max3(mx[k], s[0][k + 12], s[NT - 1][k]);
                if (NT == 2) mx[k] = __builtin_elementwise_maximum(max3(mx[k], s[NT - 1][k + 4], s[NT - 1][k + 8]), s[NT - 1][k + 12]);
            }
            float bm = __builtin_elementwise_maximum(max3(mx[0], mx[1], mx[2]), mx[3]);
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
            bm = __builtin_elementwise_maximum(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * a.scale_log2;
            if (__any(bm > m_run + 8.f)) {
                const float m_new = fmaxf(m_run, bm);
                const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
                m_run = m_new;
#pragma unroll
                for (int k = 0; k < 4; ++k) l_run[k] *= alpha;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] *= alpha;
            }
            const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
            u32x4 pb[2 * NT];
#pragma unroll
            for (int T = 0; T < NT; ++T)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    f32x2 p;
                    p[0] = __builtin_amdgcn_exp2f(fmaf(s[T][r], a.scale_log2, neg_m));
                    p[1] = __builtin_amdgcn_exp2f(fmaf(s[T][r + 1], a.scale_log2, neg_m));
                    const bf16x2 pk = __builtin_convertvector(p, bf16x2);
                    pb[2 * T + (r >> 3)][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
                    l_run[(r >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pk, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run[(r >> 1) & 3], false);
                }
            const uint32_t vbase = v_lane + c0 * kRowB;
            bf16x8 op[2 * NT * MT];
            for_each_index<2 * NT * MT + kAhead>([&](auto j) {
                if constexpr (j >= kAhead) {
                    constexpr int kk = (j - kAhead) / MT, mt = (j - kAhead) % MT;
                    o[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[j - kAhead], __builtin_bit_cast(bf16x8, pb[kk]), o[mt], 0, 0, 0);
                }
                if constexpr (j < 2 * NT * MT) {
                    constexpr int kk = j / MT, mt = j % MT;
                    const uint32_t at = (vbase ^ (mt << 6)) + 16 * kk * kRowB;
                    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)at);
                    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)(at + 8 * kRowB));
                    op[j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        constexpr std::integral_constant<int, 1> one;
        constexpr std::integral_constant<int, 2> two;
        for (int c0 = 64 * split; c0 <= last;) {
            // (a tile of 32 columns of which both kinds of scores are taken, or the last one, goes alone)
            const bool pair = c0 % 64 == 0 && c0 + 32 <= last && (c0 + 64 <= win_first || c0 >= win_last);
            const int next = c0 + (pair ? 64 : 32), to = next % 64 == 0 || next > last ? next + (63 & -next) + 64 * (kSplit - 1) : next;
            if (pair)
                block(two, c0, to > last);
            else
                block(one, c0, to > last);
            c0 = to;
        }
    };
    auto row_sum = [&]() {
        const float l = (l_run[0] + l_run[1]) + (l_run[2] + l_run[3]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    };
    // 8 output channels' words of two lane halves change places so that each lane stores 16 bytes: channels 8 (2 k + half) .. + 7 of tile mt
    auto store = [&](uint32_t at, int mt, int k, const float *v, float inv) __attribute__((always_inline)) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = pack_bf16x2(v[2 * j] * inv, v[2 * j + 1] * inv);
        const auto lo = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        *(u32x4_any *)(Op + at + mt * 64 + k * 32 + half * 16) = u32x4{lo[0], hi[0], lo[1], hi[1]};
    };
    // 64 rows of the mask, a lane each: an entry has fired where its row differs from the one before (it fires only if |k - held| > theta >=
    // 0, and then holds k)
    auto mask_rows = [&](int t0) __attribute__((always_inline)) {
        const int t = min(t0 + lane, n - 1), tp = max(t - 1, 0);
        uint32_t bits[D / 32];
#pragma unroll
        for (int w = 0; w < D / 32; ++w) {
            bits[w] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int s = 4 * w + j;
                const u32x4 x = *(lds_vec)(uintptr_t)(h_at + t * kRowB + ((s ^ keys_perm(t)) << 4));
                const u32x4 y = *(lds_vec)(uintptr_t)(h_at + tp * kRowB + ((s ^ keys_perm(tp)) << 4));
                uint32_t m = 0;                                  // even channels in bits 0, 2, 4, 6, odd ones in 16, 18, ...
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
                    m |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, x[i] ^ y[i]), u16x2_t{1, 1})) << (2 * i);
                }
                bits[w] |= ((m & 0xffffu) | (m >> 15)) << (8 * j);
            }
            if (t == 0) bits[w] = ~0u;                           // the basis row is kept whole
        }
        uint32_t fired = 0;
        if (t0 + lane < n) {
            uint32_t *const to = a.mask_bits + ((size_t)unit * n + t) * (D / 32);
#pragma unroll
            for (int w = 0; w < D / 32; ++w) {
                to[w] = bits[w];
                fired += (uint32_t)__popc(bits[w]);
            }
        }
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) fired += __shfl_xor(fired, s);
        if (lane == 0) atomicAdd(&words[3], fired);
        if (a.Khat) {
            char *const Hp = (char *)(a.Khat + (size_t)unit * n * D);
            for (int j = t0 / kRpl; j < min(t0 + 64, nk) / kRpl; ++j) {
                const int r = j * kRpl + lane / kSeg;
                if (r < n) *(u32x4 *)(Hp + (size_t)r * kRowB + (lane % kSeg) * 16) = *(lds_vec)(uintptr_t)(h_at + r * kRowB + (((lane % kSeg) ^ keys_perm(r)) << 4));
            }
        }
    };
    const int mask_items = part == a.mask_part ? (n + 63) / 64 : 0;
    if constexpr (kSplit == 1) {
        int i = wave;
        while (i < count) {
            int next = 0;
            const int row = row0;
            const uint32_t at = my_at;
            const bool mine = row + (li & (RT - 1)) < n;
            attend([&]() __attribute__((always_inline)) {
                if (lane == 0) next = (int)atomicAdd(&words[2], 1u);
                next = __builtin_amdgcn_readfirstlane(next);
                if (next < count) open(next);
            });
            const float inv = 1.f / row_sum();
            if (mine)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        float v[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) v[j] = o[mt][8 * k + j];
                        store(at, mt, k, v, inv);
                    }
            i = next;
        }
        while (i < count + mask_items) {
            mask_rows((i - count) * 64);
            int next = 0;
            if (lane == 0) next = (int)atomicAdd(&words[2], 1u);
            i = __builtin_amdgcn_readfirstlane(next);
        }
    } else {
        // the waves of a group have taken every kSplit-th block; they meet in LDS, each finishes part of the channels
        const bool works = at_first < count;
        constexpr int kMine = 16 * MT / kSplit;                  // registers of the output that a wave finishes
        float l_tot = 0.f;
        if (works) {
            attend([]() {});
            l_tot = row_sum();
        }
        for (int i = wave; i < mask_items; i += NW) mask_rows(i * 64);
        __syncthreads();                                         // keys, reference keys and values are done with
        float *const xo = (float *)lds_raw;                      // [wave][16 MT][64]
        float *const xm = xo + NW * 16 * MT * 64;                // [wave][64][2] maximum, sum
        if (works) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) xo[(wave * 16 * MT + mt * 16 + r) * 64 + lane] = o[mt][r];
            xm[(wave * 64 + lane) * 2] = m_run;
            xm[(wave * 64 + lane) * 2 + 1] = l_tot;
        }
        if (mask_items > 0 && tid == 0) a.nnz[unit] = words[3];  // (this work group exchanges nothing)
        __syncthreads();
        if (works) {
            const int w0 = wave / kSplit * kSplit, mine = wave % kSplit * kMine;
            float f[kSplit], M = -INFINITY, l = 0.f;
#pragma unroll
            for (int w = 0; w < kSplit; ++w) M = fmaxf(M, xm[((w0 + w) * 64 + lane) * 2]);   // (the first wave has seen key 0)
#pragma unroll
            for (int w = 0; w < kSplit; ++w) {
                f[w] = __builtin_amdgcn_exp2f(xm[((w0 + w) * 64 + lane) * 2] - M);
                l += xm[((w0 + w) * 64 + lane) * 2 + 1] * f[w];
            }
            const float inv = 1.f / l;
            const bool stores = row0 + (li & (RT - 1)) < n;
#pragma unroll
            for (int k = 0; k < kMine / 8; ++k) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    v[j] = 0.f;
#pragma unroll
                    for (int w = 0; w < kSplit; ++w) v[j] += xo[((w0 + w) * 16 * MT + mine + 8 * k + j) * 64 + lane] * f[w];
                }
                const int at = (mine + 8 * k) / 8;               // 16 channels from 16 `at` on
                if (stores) store(my_at, at >> 1, at & 1, v, inv);
            }
        }
        return;
    }
    if (mask_items > 0) {
        __syncthreads();
        if (tid == 0) a.nnz[unit] = words[3];
    }
}

// what a launch looks like; L == 0: the prompt is none for it
struct ShortPlan {
    int split, parts, L, L0, warm;
    size_t lds;
};

size_t short_lds(int n, int d) {
    const int nk = (n + 7) & ~7, nv = (n + 31) & ~31;
    return (size_t)((d == 64 ? kMostRows<64> : kMostRows<128>) + nk + nv) * d * 2 + kScanWaves * 256 + 16;
}

// One work group to a compute unit (its LDS).  A wave takes an item of 32 score rows, kSplit of them one together where compute units
// are idle and the longest item has that many blocks (1 / 2 / 4, us: 32 / 8 heads of 64, 1 x 64 tokens 6.6 / 7.3 / 7.2, 1 x 200
// 9.9 / 9.2 / 8.6, 1 x 333 11.8 / 10.6 / 9.7; 20 / 5 of 128, 1 x 200 13.7 / 12.5 / 11.4).  Else a unit is cut so that every wave has one item and one
// wave is left for the mask, or into as many work groups as are resident: more would each scan the unit again (16 x 200 tokens of 20 / 5
// heads of 128, cut in 1 / 2 / 3 / 4: 27.2 / 19.3 / 17.3 / 25.8 us).
// Rows that runs warm up on save rounds, where the rows that the keys' guesses need are not there anyway.  Geometric mean over 14 shapes and five kinds of keys (jumps of 1 to 20 %, theta
// 0.11 to 0.2), four inputs each, times as fast as 64 of them and runs of equal length: 48 / 56 / 64 / 72 rows 1.060 / 1.066 / 1.067 / 1.067; the worst, 1 x 416 rows of 64 that fire often
// (20 %, 0.15), 10.66 / 10.87 / 11.04 / 11.07 us for 10.76.
ShortPlan short_plan(const PrefillArgs &p) {
    ShortPlan s = {};
    if (p.dtype != 1 || (p.d != 64 && p.d != 128)) return s;
    const int g = p.Hq / p.Hkv, runs = kScanWaves * 64 / p.d;
    if (p.n > (p.d == 64 ? kMostRows<64> : kMostRows<128>)) return s;
    const int GH = g % 4 == 0 ? 4 : g % 2 == 0 ? 2 : 1, rt = 32 / GH;
    const int64_t units = (int64_t)p.B * p.Hkv, items = (int64_t)((p.n + rt - 1) / rt) * (g / GH), slots = device_cu_count();
    // (a unit's queries are addressed by 32 bits, work groups and items are counted by 31)
    if ((int64_t)g * p.n * p.d * 2 >= (int64_t)1 << 31 || units * 32 >= (int64_t)1 << 31 || items >= (int64_t)1 << 28) return s;
    s.warm = 56;
    const int later = (p.n - s.warm + runs - 1) / runs;          // the first run has no rows to warm up on and takes as many more
    s.L = later > 8 ? (later + 7) & ~7 : 8;
    s.L0 = ((p.n + 7) & ~7) - (runs - 1) * s.L;
    if (s.L0 < 8) s.L0 = 8;
    s.lds = short_lds(p.n, p.d);
    s.split = 1;
    for (int k = 4; k > 1; k /= 2)
        if (p.n > 32 * k && units * ((items * k + NW - 1) / NW + 1) <= slots) {
            s.split = k;
            break;
        }
    if (s.split > 1) {
        s.parts = (int)((items * s.split + NW - 1) / NW);
        const size_t meet = (size_t)NW * (p.d / 2 + 2) * 64 * 4; // (they meet where the rows were)
        if (s.lds < meet) s.lds = meet;
    } else {
        const int64_t most = slots / units > 0 ? slots / units : 1, wanted = (items + NW - 2) / (NW - 1);
        s.parts = (int)(wanted < most ? wanted : most);
    }
    return s;
}

template <int D, int kSplit>
void launch_short(const ShortArgs &a, const ShortPlan &s, hipStream_t stream) {
    const auto kernel = prefill_short_kernel<D, kSplit>;
    static std::atomic<uint64_t> lds_set;                        // per instantiation, one bit per device
    ensure_dynamic_lds((const void *)kernel, 160 * 1024, lds_set);
    const int blocks = a.units * (a.mask_part >= a.parts ? a.parts + 1 : a.parts);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(512), s.lds, stream, a);
}

}  // namespace

bool prefill_short_supported(const PrefillArgs &p) { return short_plan(p).L > 0; }

void launch_prefill_short(const PrefillArgs &p, float theta, void *khat, uint32_t *mask_bits, uint64_t *nnz, hipStream_t stream) {
    const ShortPlan s = short_plan(p);
    ShortArgs a = {};
    a.Q = (const bf16_t *)p.Q;
    a.K = (const bf16_t *)p.K;
    a.V = (const bf16_t *)p.V;
    a.O = (bf16_t *)p.O;
    a.Khat = (bf16_t *)khat;
    a.mask_bits = mask_bits;
    a.nnz = nnz;
    a.Hq = p.Hq;
    a.n = p.n;
    a.W = p.W;
    a.sliding = p.sliding;
    a.units = p.B * p.Hkv;
    a.g = p.Hq / p.Hkv;
    const int GH = a.g % 4 == 0 ? 4 : a.g % 2 == 0 ? 2 : 1, rt = 32 / GH, hgroups = a.g / GH;
    a.rt_log2 = __builtin_ctz(rt);
    a.row_groups = (p.n + rt - 1) / rt;
    a.items = a.row_groups * hgroups;
    a.parts = s.parts;
    a.mask_part = s.split > 1 ? s.parts : s.parts - 1;
    a.L = s.L;
    a.L0 = s.L0;
    a.warm = s.warm;
    a.by_units = divisor(a.units);
    a.by_hkv = divisor(p.Hkv);
    a.by_hgroups = divisor(hgroups);
    a.by_w = divisor(p.W);
    a.scale_log2 = p.scale_log2;
    a.theta = theta;
    if (p.d == 64)
        s.split == 4 ? launch_short<64, 4>(a, s, stream) : s.split == 2 ? launch_short<64, 2>(a, s, stream) : launch_short<64, 1>(a, s, stream);
    else
        s.split == 4 ? launch_short<128, 4>(a, s, stream) : s.split == 2 ? launch_short<128, 2>(a, s, stream) : launch_short<128, 1>(a, s, stream);
}

}  // namespace da
