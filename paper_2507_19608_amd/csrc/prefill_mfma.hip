// Hybrid-attention prefill for bf16 inputs, head_dim 64 or 128 (Sec. III-B prefill stage; Eq. 4; Eq. 1).
//
// Work group = 8 waves on one tile of score rows: RT consecutive query rows x GH query heads of one KV head (they
// share K, V and the delta matrix); a wave owns 32 score rows.  A row's window is its square of side W on the diagonal, or
// the band of the W newest keys.
//
//   left of the window   the running score of Eq. 4 is, by the telescoped sum of the delta rows up to column j, the
//                        product of the query with the held key, q . k_hat(j): K_hat Q^T on the matrix cores.
//                        DA_SCORE_GATHER takes this form too: adding up the surviving entries one by one on the
//                        vector ALU was bound by instruction issue and LDS at 8.1 ms on 4 x 8192 tokens, 20 / 5 heads
//                        of 128, 60 % sparsity - the survivors of a block cost about 16 times its dense product.
//   inside the window    exact scores K Q^T.
//
// The keys of a tile are walked as one list of blocks: first the blocks with columns left of some row's window (scores
// from K_hat), then the blocks with columns inside some row's window (scores from K).  A block in which rows disagree is in
// the list twice, each time with the other part masked: there is one loop and one kind of block, and what a block
// reads is two tiles, keys and values.
//
// What bounds it: matrix cores and vector ALU take turns.  A block of 64 keys costs a wave 1024 cycles of matrix work at
// head_dim 128 (512 at 64) and about 1000 of softmax, so a SIMD is only busy if one of its two waves multiplies while the
// other takes exponentials.  The waves therefore run in two groups half a block apart (waves 0-3 and 4-7, one of each per
// SIMD), handed from phase to phase by barriers:
//     A: | PV(b-1) S(b) | softmax(b)   | PV(b) S(b+1) | ...
//     B:                | PV(b-1) S(b) | softmax(b)   | ...
// Built like this the card's power limit is what is left on long prompts: products fed from LDS with nothing else going on draw
// the clock down to 1.7 GHz, and orders of the reads, priorities or row sums that take fewer cycles take as long.
// 4 x 8192 tokens, 20 / 5 heads of 128: 1340 -> 1215 us (all waves in step, a barrier per 32 keys, tiles by way of registers
// and V re-ordered by a launch of its own before); 1 x 4096: 190 -> 115 us, most of it from the order of the tiles below.
//
// kSplit = 2: a tile has 128 score rows and the two groups walk alternate blocks of 32 keys, with their own running
// (maximum, sum, output), and meet in LDS at the end.  Twice the tiles, each done in 0.8 of the time: for launches that would
// otherwise wait for their longest tile (see launch_d).
//
// Tiles go from global memory to LDS directly (global_load_lds, 16 bytes per lane, no registers), row-major, two blocks ahead
// in three buffers.  The 16-byte segments of a row are permuted by the row number so that the reads are free of bank
// conflicts: keys by 128-bit reads down a column of rows, values by transposing reads (ds_read_b64_tr_b16: lane j of 16
// receives channel j of four key rows whose 8-byte pieces the 16 lanes address), which is why V needs no re-ordering launch.
//
// Matrix-core layouts (v_mfma_f32_32x32x16_bf16, wave64): A lane l holds row l%32, k = 8*(l/32)..+7; B lane l holds column
// l%32, same k; D lane l holds column l%32, rows 8*(r/4) + 4*(l/32) + r%4 for register r.  Scores are produced transposed
// (keys x score rows) so that a lane owns one score row, and D registers 8a..8a+7 are exactly the B operand of the a-th
// k-step of P V once V^T is fetched in the matching key order.
#include <math.h>

#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"

namespace da {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kSpan = 64;       // keys of one turn of the loop (both groups together where they walk different ones)

struct MfmaArgs {
    const bf16_t *__restrict__ Q;
    const bf16_t *__restrict__ K;
    const bf16_t *__restrict__ Khat;
    const bf16_t *__restrict__ V;
    bf16_t *__restrict__ O;
    int Hq, Hkv, n, W, sliding;
    int ld;                             // rows of room per unit in K, Khat, V (>= n)
    int q_off, nq;                      // query rows are positions q_off .. q_off + nq - 1 of the n keys
    int units, GH, RT, tiles, hgroups;  // batch x KV heads, heads per tile, rows per head and tile, row tiles, head chunks per unit
    int xsplit;                         // > 0: XCD-aware order, every unit split this many ways (see the kernel)
    float scale_log2;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// 64 x 16 bytes from base + the lanes' offsets to LDS bytes lds .. lds + 1023 (wave-uniform), lane after lane.  In asm, so
// that the compiler does not order later LDS reads behind it: whoever reads the tile waits for the count (wait_loads) and
// then passes a barrier.  (s_nop: m0 may be used by an LDS load one wait state after it was written.)
__device__ __forceinline__ void load_to_lds(const char *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {                   // until at most N of this wave's loads are in flight
    static_assert(N < 16, "one field of the count");
    __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}
// The border between two phases: nothing moves across it, in the compiler either.
__device__ __forceinline__ void phase_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// f(0), f(1), ... f(N - 1) with the index a constant
template <typename F, int... I>
__device__ __forceinline__ void for_each_index_impl(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_each_index(F f) {
    for_each_index_impl(f, std::make_integer_sequence<int, N>{});
}

template <int D, int kSplit>
__global__ __launch_bounds__(512) void prefill_mfma_kernel(MfmaArgs a) {
    constexpr int kRowB = D * 2;                // bytes of a row
    constexpr int kSeg = D / 8;                 // 16-byte segments of a row
    constexpr int kTile = kSpan * kRowB;        // bytes of a tile (keys or values of one turn)
    constexpr int kIpw = kTile / 1024 / 8;      // 1 KiB loads per wave that fill a tile
    constexpr int kLoads = 2 * kIpw;            // loads per wave and turn
    constexpr int KB = kSpan / kSplit;          // keys per block
    constexpr int NT = KB / 32;                 // score tiles per block
    constexpr int KS = D / 16;                  // k-steps of Q K^T
    constexpr int MT = D / 32;                  // channel tiles of the output
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];   // [3] key tiles, [3] value tiles

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = wave >> 2;
    const int half = lane >> 5, li = lane & 31;

    // ---- which tile.  Work groups go to the 8 XCDs round-robin by index, and within an XCD they start in order, each on a
    //      compute unit of the shader engine whose turn it is: a long tile late in the order waits while compute units
    //      elsewhere are idle, and then runs alone.  So the longest (last) tiles of every unit come first, the
    //      shortest last.  Every XCD has its own L2, and all tiles of a unit stream the same K, K_hat and V: where the units -
    //      or, with xsplit, units cut by tile index modulo xsplit - deal out evenly, an XCD keeps to its own.
    int unit, bid;
    if (a.xsplit > 0) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int parts = a.units * a.xsplit / 8;                // of this XCD: xcd, xcd + 8, ...
        const int part = xcd + 8 * (slot % parts);
        unit = part / a.xsplit;
        bid = slot / parts * a.xsplit + part % a.xsplit;
    } else {
        unit = blockIdx.x % a.units;
        bid = blockIdx.x / a.units;
    }
    const int hchunk = bid % a.hgroups;
    const int tile = a.tiles - 1 - bid / a.hgroups;
    const int b = unit / a.Hkv, hk = unit % a.Hkv;
    const int g = a.Hq / a.Hkv;
    const int head0 = hk * g + hchunk * a.GH;
    const int n = a.n, W = a.W, RT = a.RT;
    const int i0 = a.q_off + tile * RT, i_last = min(i0 + RT - 1, n - 1);   // first and last query position

    const char *Kp = (const char *)(a.K + (size_t)unit * a.ld * D);
    const char *Hp = (const char *)(a.Khat + (size_t)unit * a.ld * D);
    const char *Vp = (const char *)(a.V + (size_t)unit * a.ld * D);

    // ---- this lane's score row: sr = 32 * (wave, or wave of its group) + li (both lane halves) -> query row i0 + r of head
    //      head0 + hh.  A wave's 32 rows are consecutive rows of one head (RT is a multiple of 32).
    const int my_sr = 32 * (kSplit == 1 ? wave : wave & 3) + li;
    const int my_hh = my_sr / RT, my_r = my_sr - my_hh * RT;
    const int my_i = i0 + my_r;
    const bool my_valid = my_i < n;
    // first exact column of row r: start of its square, or of its band (monotone in r either way)
    auto win_start = [&](int r) { return a.sliding ? max(r - W + 1, 0) : (r / W) * W; };
    const int my_win = win_start(min(my_i, n - 1));
    const int wave_first = __builtin_amdgcn_readfirstlane(my_i);         // rows of this wave: wave_first .. + 31
    const int wave_win_first = win_start(min(wave_first, n - 1)), wave_win_last = win_start(min(wave_first + 31, n - 1));

    // ---- the list of blocks: n_hat blocks from key 0 on for K_hat, then blocks kb0 .. i_last / KB for K
    const int win_first = win_start(i0), win_last = win_start(i_last);
    const int n_hat = (win_last + KB - 1) / KB, kb0 = win_first / KB;
    const int nv = n_hat + i_last / KB - kb0 + 1;
    const int turns = (nv + kSplit - 1) / kSplit;
    auto block_of = [&](int v) { return v < n_hat ? v : kb0 + v - n_hat; };

    u32x4 qreg[KS];
    {
        const bf16_t *my_q =
            a.Q + (((size_t)b * a.Hq + head0 + my_hh) * a.nq + (min(my_i, n - 1) - a.q_off)) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = *(const u32x4 *)(my_q + ks * 16);
    }

    // ---- tile loads: a wave fills 8 rows of the tile (of its own group's block), 1 KiB load i the rows r .. r + 64 / kSeg - 1
    //      of these, lane = (row, segment as stored); the segment it fetches is the stored one permuted by the row number.
    //      A lane's offset from the load's first row never changes, except where the keys end inside a load.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)lds_raw;
    auto keys_perm = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
    auto vals_perm = [](int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };
    constexpr int kRpl = 64 / kSeg;                              // rows per load
    static_assert(kIpw * kRpl == 8, "a wave fills 8 rows");
    const int lrow = lane / kSeg, lseg = lane % kSeg;
    auto lane_off = [&](int i, bool keys, int row) -> uint32_t { // row: of the load's rows, clamped to the keys there are
        const int r = wave * 8 + i * kRpl + lrow;
        return row * kRowB + ((lseg ^ (keys ? keys_perm(r) : vals_perm(r))) << 4);
    };
    uint32_t k_off[kIpw], v_off[kIpw];
#pragma unroll
    for (int i = 0; i < kIpw; ++i) {
        k_off[i] = lane_off(i, true, lrow);
        v_off[i] = lane_off(i, false, lrow);
    }
    // first key row that this wave loads of its group's block in a turn, and which rows the scores of that block are taken from
    struct Source {
        const char *keys;
        int row;
    };
    auto source_of = [&](int turn) -> Source {
        const int v = min(kSplit == 1 ? turn : turn * kSplit + grp, nv - 1);   // (past the end: the last block again, unread)
        return {v < n_hat ? Hp : Kp, block_of(v) * KB + (wave * 8) % KB};
    };
    auto load_tile = [&](const char *src, int row, int buf, bool keys) {
        const uint32_t to = lds0 + (keys ? 0 : 3 * kTile) + buf * kTile + wave * (8 * kRowB);
#pragma unroll
        for (int i = 0; i < kIpw; ++i) {
            if (row + 8 <= n) {
                load_to_lds(src + (size_t)(uint32_t)row * kRowB + i * (kRpl * kRowB), keys ? k_off[i] : v_off[i], to + i * 1024);
            } else {
                const int first = min(row + i * kRpl, n - 1);
                load_to_lds(src + (size_t)(uint32_t)first * kRowB, lane_off(i, keys, min(lrow, n - 1 - first)), to + i * 1024);
            }
        }
    };

    f32x16 oacc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[mt][r] = 0.f;
    float m_run = -INFINITY;
    float l_run[4] = {0.f, 0.f, 0.f, 0.f};      // four chains of the running sum, this lane half's share
    f32x16 s[NT];                               // raw scores of the current block
    u32x4 pb[2 * NT];                           // its probabilities, bf16, as P V operands

    const int row_base = kSplit == 1 ? 0 : grp * KB;             // this group's rows in a tile
    // per-lane addresses inside a tile: every read below is one of these, an exclusive-or of a few bits, a constant
    const uint32_t k_lane = lds0 + (row_base + li) * kRowB + ((half ^ keys_perm(li)) << 4);
    const int L = lane & 15, lg = (lane >> 4) & 1;
    const uint32_t v_lane = lds0 + 3 * kTile + (row_base + 4 * half + (L >> 2)) * kRowB + (vals_perm(L >> 2) << 4) + lg * 32 + (L & 3) * 8;

    // A matrix phase: P V of the turn before (value buffer vb), then the scores of this turn (key buffer kb).  Every matrix
    // instruction takes its first operand fresh from LDS; the reads run kAhead instructions in front, from one product
    // into the next.  (The order is nailed down instruction by instruction: left alone the compiler issues a read, waits
    // for it and multiplies.)
    auto matrix_phase = [&](auto with_values, auto with_scores, int vb, int kb) {
        constexpr int nv = with_values ? 2 * NT * MT : 0, nk = with_scores ? NT * KS : 0;
        const uint32_t vbase = v_lane + vb * kTile, kbase = k_lane + kb * kTile;
        bf16x8 op[nv + nk];
        auto read = [&](auto i) {
            if constexpr (i < nv) {
                // lane l: channel 32 mt + l % 32, keys 16 kk + 4 (l / 32) + {0..3} and 8 more
                constexpr int kk = i / MT, mt = i % MT;
                const uint32_t at = (vbase ^ (mt << 6)) + 16 * kk * kRowB;
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)at);
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)(at + 8 * kRowB));
                op[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
            } else {
                constexpr int ks = (i - nv) / NT, T = (i - nv) % NT;
                op[i] = *(const __attribute__((address_space(3))) bf16x8 *)(uintptr_t)((kbase ^ (ks << 5)) + T * 32 * kRowB);
            }
        };
        auto multiply = [&](auto i) {
            if constexpr (i < nv) {
                constexpr int kk = i / MT, mt = i % MT;
                oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[i], __builtin_bit_cast(bf16x8, pb[kk]), oacc[mt], 0, 0, 0);
            } else {
                constexpr int ks = (i - nv) / NT, T = (i - nv) % NT;
                if constexpr (ks == 0) {
                    f32x16 zero;
#pragma unroll
                    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                    s[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[i], __builtin_bit_cast(bf16x8, qreg[ks]), zero, 0, 0, 0);
                } else {
                    s[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[i], __builtin_bit_cast(bf16x8, qreg[ks]), s[T], 0, 0, 0);
                }
            }
        };
        constexpr int kAhead = 5;
        for_each_index<nv + nk + kAhead>([&](auto i) {
            if constexpr (i >= kAhead) multiply(std::integral_constant<int, i - kAhead>{});
            if constexpr (i < nv + nk) read(i);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Masks where some row of the tile does not see all of block v, then online softmax: s -> pb.  The running maximum is
    // only raised when the block maximum exceeds it by more than 2^8 in the exponent, so probabilities stay <= 256
    // and the accumulator is rarely rescaled.
    auto softmax = [&](int v) {
        const int jb = block_of(v) * KB;
        const bool hat = v < n_hat, none = kSplit > 1 && v >= nv;        // (none: a turn in which this group has no block)
        if (none || (hat ? jb + KB > wave_win_first : jb < wave_win_last || jb + KB > wave_first + 1)) {
            const int lo = hat ? 0 : my_win, cnt = none ? 0 : hat ? my_win : my_i - my_win + 1;   // columns lo .. lo + cnt - 1
            const int j0 = jb + 4 * half - lo;
#pragma unroll
            for (int T = 0; T < NT; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    s[T][r] = (uint32_t)(j0 + 32 * T + 8 * (r >> 2) + (r & 3)) < (uint32_t)cnt ? s[T][r] : -INFINITY;
        }
        float bm;
        {
            float mx[4];                                         // four chains: one would wait for itself
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                mx[k] = fmaxf(fmaxf(s[0][4 * k], s[0][4 * k + 1]), fmaxf(s[0][4 * k + 2], s[0][4 * k + 3]));
                if (NT == 2) mx[k] = fmaxf(mx[k], fmaxf(fmaxf(s[NT - 1][4 * k], s[NT - 1][4 * k + 1]), fmaxf(s[NT - 1][4 * k + 2], s[NT - 1][4 * k + 3])));
            }
            bm = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
            bm = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * a.scale_log2;
        }
        if (__any(bm > m_run + 8.f)) {
            const float m_new = fmaxf(m_run, bm);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
            m_run = m_new;
#pragma unroll
            for (int k = 0; k < 4; ++k) l_run[k] *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) oacc[mt] *= alpha;
        }
        const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
        // The row sum is taken over the probabilities as rounded to bf16, i.e. over the very weights that P V uses:
        // the output is then an exact weighted mean of the value rows, and the rounding of the weights cannot bias it
        // (summing the unrounded ones does, by up to 2^-9 relative when many weights are equal).
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                f32x2 p;                                         // bare v_exp_f32: tiny results may flush to 0
                p[0] = __builtin_amdgcn_exp2f(fmaf(s[T][r], a.scale_log2, neg_m));
                p[1] = __builtin_amdgcn_exp2f(fmaf(s[T][r + 1], a.scale_log2, neg_m));
                const bf16x2 pk = __builtin_convertvector(p, bf16x2);
                pb[2 * T + (r >> 3)][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
                l_run[(r >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pk, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run[(r >> 1) & 3], false);
            }
    };

    // ---- the walk.  Key tile t lies in buffer t % 3, value tile t too; key tile t + 2 and value tile t + 1 are requested
    //      in turn t's matrix phase, when no wave reads what those buffers held any more (the other group is at most one
    //      phase behind), and are waited for two phases later.
    Source s0 = source_of(0), s1 = source_of(1);                 // sources of turns t and t + 1
    load_tile(s0.keys, s0.row, 0, true);
    load_tile(s1.keys, s1.row, 1, true);
    load_tile(Vp, s0.row, 0, false);
    wait_loads<kLoads>();                                        // key tile 0
    // (the queries are waited for here: left to the compiler, the wait would stand at their first use inside the loop and there
    // drain the tile loads, every turn)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
    phase_barrier();
    if (grp == 1) phase_barrier();                               // group B starts one phase later
    constexpr std::true_type yes;
    constexpr std::false_type no;
    int buf = 0;                                                 // turn % 3
    auto vector_phase = [&](int turn, int next, int prev) {
        if (grp == 1) wait_loads<0>();                           // key tile turn + 1, value tile turn
        phase_barrier();
        __builtin_amdgcn_s_setprio(1);
        const Source s2 = source_of(turn + 2);
        load_tile(s2.keys, s2.row, prev, true);
        load_tile(Vp, s1.row, next, false);
        s1 = s2;
        softmax(kSplit == 1 ? turn : turn * kSplit + grp);
        __builtin_amdgcn_s_setprio(0);
        if (grp == 0) wait_loads<kLoads>();
        phase_barrier();
    };
    matrix_phase(no, yes, 0, 0);
    vector_phase(0, 1, 2);
    for (int turn = 1; turn < turns; ++turn) {
        const int prev = buf;
        buf = buf == 2 ? 0 : buf + 1;
        const int next = buf == 2 ? 0 : buf + 1;
        matrix_phase(yes, yes, prev, buf);
        vector_phase(turn, next, prev);
    }
    matrix_phase(yes, no, buf, 0);
    if (grp == 0) phase_barrier();                               // (group B's last softmax phase)
    wait_loads<0>();                                             // no load into LDS outlives its wave

    // ---------------------------------------------------------------- epilogue
    float l_tot = (l_run[0] + l_run[1]) + (l_run[2] + l_run[3]);
    l_tot += __shfl_xor(l_tot, 32);
    bf16_t *orow = a.O + (((size_t)b * a.Hq + head0 + my_hh) * a.nq + (my_i - a.q_off)) * D;
    auto store = [&](int mt, float inv) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            u32x2 w;
            w[0] = pack_bf16x2(oacc[mt][4 * q4 + 0] * inv, oacc[mt][4 * q4 + 1] * inv);
            w[1] = pack_bf16x2(oacc[mt][4 * q4 + 2] * inv, oacc[mt][4 * q4 + 3] * inv);
            *(u32x2 *)(orow + mt * 32 + 8 * q4 + 4 * half) = w;
        }
    };
    if constexpr (kSplit == 1) {
        if (my_valid) {
            const float inv = 1.f / l_tot;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) store(mt, inv);
        }
    } else {
        // wave w of group A and wave w of group B hold the same rows: each hands the other half of its channels over and
        // finishes its own half
        constexpr int MH = MT / 2;
        float *xo = (float *)lds_raw;                            // [group][wave of the group][MH][16][64]
        float *xm = xo + 2 * 4 * MH * 16 * 64;                   // [group][wave of the group][64][2] maximum, sum
        const int w4 = wave & 3;
        __syncthreads();                                         // the tiles are done with
#pragma unroll
        for (int mh = 0; mh < MH; ++mh)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                xo[(((grp * 4 + w4) * MH + mh) * 16 + r) * 64 + lane] = grp == 0 ? oacc[MH + mh][r] : oacc[mh][r];
        xm[((grp * 4 + w4) * 64 + lane) * 2] = m_run;
        xm[((grp * 4 + w4) * 64 + lane) * 2 + 1] = l_tot;
        __syncthreads();
        const int other = 1 - grp;
        const float m2 = xm[((other * 4 + w4) * 64 + lane) * 2], l2 = xm[((other * 4 + w4) * 64 + lane) * 2 + 1];
        const float M = fmaxf(m_run, m2);                        // (a row sees its own key: one of the two is finite)
        const float f1 = __builtin_amdgcn_exp2f(m_run - M), f2 = __builtin_amdgcn_exp2f(m2 - M);
        const float inv = 1.f / (l_tot * f1 + l2 * f2);
#pragma unroll
        for (int mh = 0; mh < MH; ++mh)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float x = xo[(((other * 4 + w4) * MH + mh) * 16 + r) * 64 + lane];
                if (grp == 0)
                    oacc[mh][r] = oacc[mh][r] * f1 + x * f2;
                else
                    oacc[MH + mh][r] = oacc[MH + mh][r] * f1 + x * f2;
            }
        if (my_valid) {
#pragma unroll
            for (int mh = 0; mh < MH; ++mh) {
                if (grp == 0)
                    store(mh, inv);
                else
                    store(MH + mh, inv);
            }
        }
    }
}

template <int D, int kSplit>
void launch_tiles(const PrefillArgs &p, MfmaArgs &a, hipStream_t s) {
    const int units = p.B * p.Hkv, g = p.Hq / p.Hkv;
    a.GH = (g % 4 == 0) ? 4 : (g % 2 == 0) ? 2 : 1;
    a.RT = 256 / kSplit / a.GH;
    a.tiles = (p.nq + a.RT - 1) / a.RT;
    a.hgroups = g / a.GH;
    a.units = units;
    // XCD-aware order needs units * xsplit parts to deal out evenly over 8 XCDs and a unit to split evenly
    a.xsplit = 0;
    for (int sp = 1; sp <= 8; sp *= 2)
        if ((units * sp) % 8 == 0) {
            if ((a.tiles * a.hgroups) % sp == 0 && sp < 8) a.xsplit = sp;
            break;
        }
    constexpr int lds = 6 * kSpan * D * 2;
    static_assert(kSplit == 1 || lds >= 2 * 4 * (D / 64) * 16 * 64 * 4 + 2 * 4 * 64 * 2 * 4, "the merge reuses the tiles' room");
    static std::atomic<uint64_t> lds_set;                        // per instantiation, one bit per device
    ensure_dynamic_lds((const void *)prefill_mfma_kernel<D, kSplit>, lds, lds_set);
    const size_t blocks = (size_t)units * a.tiles * a.hgroups;
    hipLaunchKernelGGL((prefill_mfma_kernel<D, kSplit>), dim3((unsigned)blocks), dim3(512), lds, s, a);
}

template <int D>
void launch_d(const PrefillArgs &p, hipStream_t s) {
    MfmaArgs a;
    a.Q = (const bf16_t *)p.Q;
    a.K = (const bf16_t *)p.K;
    a.Khat = (const bf16_t *)p.Khat;
    a.V = (const bf16_t *)p.V;
    a.O = (bf16_t *)p.O;
    a.Hq = p.Hq;
    a.Hkv = p.Hkv;
    a.n = p.n;
    a.W = p.W;
    a.sliding = p.sliding;
    a.ld = p.ld > 0 ? p.ld : p.n;
    a.q_off = p.q_off;
    a.nq = p.nq;
    a.scale_log2 = p.scale_log2;
    // Whole or split tiles: a split one has half the rows and takes 0.8 of the time, so splitting shortens the longest tile and
    // costs 1.6 times the work.  A launch lasts at least as long as its longest tile, as the work per compute unit, and,
    // with more tiles than compute units, as two of the longest that have to share one (which the pieces of a chunked
    // prefill, all of about one length, come up against); lengths run evenly from the first row's to the last row's.
    // Splitting has to promise a tenth.  In units of one whole tile over 64 keys.
    const int g = p.Hq / p.Hkv, heads = (g % 4 == 0) ? 4 : (g % 2 == 0) ? 2 : 1;
    const double cus = device_cu_count(), shortest = p.q_off / 64.0, longest = p.n / 64.0;
    auto lasts = [&](int rows, double per_tile) {
        const double tiles = (double)p.B * p.Hkv * (g / heads) * ((p.nq + rows - 1) / rows);
        const double shared = tiles > cus ? 2.0 * (longest - (longest - shortest) * cus / tiles) : 0.0;
        return per_tile * fmax(fmax(longest, shared), tiles * 0.5 * (shortest + longest) / cus);
    };
    if (lasts(128 / heads, 0.8) < 0.9 * lasts(256 / heads, 1.0))
        launch_tiles<D, 2>(p, a, s);
    else
        launch_tiles<D, 1>(p, a, s);
}

}  // namespace

bool prefill_mfma_supported(const PrefillArgs &p) {
    return p.dtype == 1 && (p.d == 64 || p.d == 128) &&
           (size_t)p.B * p.Hkv * ((p.n + 31) / 32) * (p.Hq / p.Hkv) < ((size_t)1 << 31) &&
           (((uintptr_t)p.K | (uintptr_t)p.V) & 15) == 0;        // (loads straight into LDS want aligned rows)
}

void launch_prefill_mfma(const PrefillArgs &p, hipStream_t s) {
    if (p.d == 64)
        launch_d<64>(p, s);
    else
        launch_d<128>(p, s);
}

}  // namespace da
