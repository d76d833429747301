// Hybrid-attention prefill for bf16 inputs, head_dim 64 or 128 (Sec. III-B prefill stage; Eq. 4; Eq. 1).
//
// Work group = 8 waves on one tile of score rows: RT consecutive query rows x GH query heads of one KV head (they
// share K, V and the delta matrix); a wave owns 32 score rows.  A row's window is its square of side W on the diagonal, or
// the band of the W newest keys.
//
//   left of the window   the running score of Eq. 4 is, by the telescoped sum of the delta rows up to column j, the
//                        product of the query with the held key, q . k_hat(j): K_hat Q^T on the matrix cores.
//                        DA_SCORE_GATHER takes this form too: adding up the surviving entries one by one on the
//                        vector ALU was bound by instruction issue and LDS, at 8.04 ms on 4 x 8192 tokens, 20 / 5 heads
//                        of 128, 60 % sparsity, which take 1.10 to 1.20 ms here (the clock differs from card to card).
//   inside the window    exact scores K Q^T.
//
// The keys of a tile are walked as one list of blocks: first the blocks with columns left of some row's window (scores
// from K_hat), then the blocks with columns inside some row's window (scores from K).  A block in which rows disagree is in
// the list twice, each time with the other part masked: there is one loop and one kind of block, and what a block
// reads is two tiles, keys and values.
//
// What bounds it: matrix cores and vector ALU take turns.  A block of 64 keys costs a wave 1088 cycles of matrix work at
// head_dim 128 (512 at 64) and about 590 of issue for softmax and addresses, so a SIMD is only busy if one of its two waves multiplies while the
// other takes exponentials.  The waves therefore run in two groups half a block apart (waves 0-3 and 4-7, one of each per
// SIMD), with one barrier for every block (|), group A's before its matrix phase and group B's before its vector phase:
//     A: | PV(b-1) S(b)   softmax(b)    | PV(b) S(b+1) softmax(b+1) |
//     B: | softmax(b-1)   PV(b-1) S(b)  | softmax(b)   PV(b) S(b+1) |
// Between two barriers a wave goes from phase to phase by itself: a block takes the sum of its two phases, not twice the longer one, as it did with
// a barrier between them (4 x 8192 tokens, 20 / 5 heads of 128, by the counters: 2960 to 3040 -> 2840 to 2870 clocks a block and pair of waves; 38 shapes 1.00 to 1.07 times as
// fast, 1.03 on the geometric mean, with the shorter read-ahead of the operands and, at head_dim 64, kLate).  What the tiles need for that: three of each kind, requested up to two turns ahead.  Where every group has its own
// there is room for two, and the next ones can only be requested behind the barrier, by all waves at once; see kLate.
// A wave in its matrix phase goes first (s_setprio): it issues one instruction in 32 clocks, and every one that has to wait for
// the other wave's arithmetic lengthens the phase (without it 5 % more clocks).  What is added to a matrix phase - addresses, loads, the look at the masks -
// comes out at more than it saves in the vector phase: its instructions wait in order for whatever is issued between them.
// Counters on 4 x 8192 tokens, 20 / 5 heads of 128, with the barrier between the phases: 1.96 M clocks a launch (without it 1.85), 1520 a phase, of which one wave's matrix instructions
// fill 1088 and the other wave's vector instructions 586; with row sums by dot products on the vector ALU and the maximum of every block 2.08 M and 1610
// (692 of issue).  Before that, with the priority the other way round, a branch and an address for every
// load, fmaxf, a wait where the next tile is asked for, a pause between tiles and queries and outputs in pieces it was 2.43 M; of 15 %
// fewer clocks 7 % are left in time (1344 -> 1256 us a call, in turn on one card): the clock goes down under this load, to 1.6 of 2.4 GHz.
//
// kStream: where many whole tiles, or long ones, follow each other on a compute unit, the next one's first keys and queries are
// requested, and its first scores taken, while the last one's values are still added up and its outputs stored.  Pausing / not: 1 x 4096
// tokens 104 / 102 us, 4 x 8192 1224 / 1214, 26 x 512 77.8 / 73.5.  At head_dim 64 a second work group on the compute unit works in the
// pause (see launch_d).
//
// kSplit = 2: a tile has 128 score rows and the two groups walk alternate blocks of 64 keys, with their own running
// (maximum, sum, output), and meet in LDS at the end.  Twice the tiles, each done in 0.64 of the time (1.13 instead of 1.76 us for 64
// keys at head_dim 128, 0.81 instead of 1.31 at 64: the same work per wave, twice the loads): for the last, longest rows of a
// launch that would otherwise wait for them.  A launch cuts its rows into whole and split tiles where that promises to end first
// (see launch_d) and hands them out longest first from a counter.  Attention alone, all whole / all split / as cut: 2048 tokens, 32
// / 8 heads of 64: 41.5 / 30.8 / 30.3 us; 1 x 1024, 20 / 5 heads of 128: 32.2 / 23.0 / 22.9; 16 x 200: 25.8 / 28.6 / 25.5; 4 x 2048: 104 / 110 /
// 103; 1 x 4096: 99.7 / 93.4 / 92.7.
//
// Figures here and below for up to 416 rows of 64 or 200 of 128 (16 x 200, 14 x 200, 64 x 64, 133 x 64, 512 x 64, 55 x 130, 1 x 333 tokens) were taken when
// prompts of such lengths still came here in one call.  These have a kernel of their own now (prefill_short.hip); pieces of a prompt of such lengths come here.
//
// Tiles go from global memory to LDS directly (global_load_lds, 16 bytes per lane, no registers), row-major, up to two blocks ahead
// in three buffers, or two where every group has its own.  The 16-byte segments of a row are permuted by the row number so that the reads are free of bank
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

#include "cache_fill.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace da {

namespace {

constexpr int KB = 64;          // keys of a block
constexpr int kQueueStride = kPrefillQueueBytes / 8 / 4;

struct MfmaArgs {
    const bf16_t *__restrict__ Q;
    const bf16_t *__restrict__ K;
    const bf16_t *__restrict__ Khat;
    const bf16_t *__restrict__ V;
    bf16_t *__restrict__ O;
    int Hq, n, W, sliding;
    int ld;                             // rows of room per unit in K, Khat, V (>= n)
    int q_off, nq;                      // query rows are positions q_off .. q_off + nq - 1 of the n keys
    int GH;                             // heads per tile
    struct Kind {
        int rt_log2, tiles, row0;       // log2 of rows per head and tile, row tiles, first query row
        int first, end;                 // positions of these tiles in the launch's order
    } kinds[2];                         // whole tiles, split tiles
    int g;                              // query heads per KV head
    Divisor by_hkv, by_hgroups, by_w;   // KV heads, head chunks per unit, window
    Divisor by_units, by_parts;         // batch x KV heads; what an XCD has of them, or of their parts (see the kernel)
    int xsplit_log2;                    // >= 0: XCD-aware order, every unit split 2^this many ways
    int blocks, turn_at;                // tiles of the launch; where their order turns (see prefill_mfma_kernel)
    int total;                          // tiles and, behind them, items of a hand-off to a cache
    uint32_t *queue;                    // [8] counters, kQueueStride apart, zero at the start: tiles handed out beyond the first of each work group
    float scale_log2;
    NnzSum sum;
};

// The tiles of one kind: those at `pos` and the positions the queue hands out after it; returns the first of these past the
// kind's end.  a: the kernel's argument, of which the walk keeps a few words in registers.  None of these kernels
// may spill: a ticket of the queue is on its way into its register while other things are done, and a copy of that would be one of the old value
// (a build in which one does fails).
template <int D, int kSplit, bool kStream, bool kLate, bool kQueue>   // kQueue: there may be tiles beyond those of the grid
__device__ __forceinline__ int tiles_of_kind(const MfmaArgs &a, int pos, char *lds_raw) {
    constexpr int kRowB = D * 2;                // bytes of a row
    constexpr int kSeg = D / 8;                 // 16-byte segments of a row
    constexpr int kTile = KB * kSplit * kRowB;  // bytes of a tile (keys or values of one turn, of both groups)
    constexpr int kBufs = kSplit == 1 ? 3 : 2;  // tiles of each kind in LDS
    constexpr int kRows = KB * kSplit / 8;      // rows of a tile that a wave fills
    constexpr int kIpw = kTile / 1024 / 8;      // by this many 1 KiB loads
    constexpr int kLoads = 2 * kIpw;            // loads per wave and turn
    constexpr int NT = KB / 32;                 // score tiles per block
    static_assert(NT == 2, "the block's maximum");
    constexpr int KS = D / 16;                  // k-steps of Q K^T
    constexpr int MT = D / 32;                  // channel tiles of the output
    // LDS: [kBufs] key tiles, [kBufs] value tiles, at the end the next tile; where a tile begins, its queries lie behind the first value
    // tile
    constexpr int kRoom = 4 * KB * 2 * kRowB;   // of everything but the next tile's number
    int *const next_tile = (int *)(lds_raw + kRoom);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = wave >> 2;
    const int half = lane >> 5, li = lane & 31;

    const int n = a.n;
    const int my_sr = 32 * (kSplit == 1 ? wave : wave & 3);     // the wave's first score row

    // ---- the tile whose keys and values are being requested
    const char *Kp, *Hp, *Vp;
    const bf16_t *q_rows;                       // where position 0 of the wave's head would be in Q
    bf16_t *o_rows;                             // ... in O
    int first;                                  // rows of this wave: first .. + 31, some or all of which may lie past the end
    int n_hat, kb0, nv, turns;                  // the list of blocks: n_hat from key 0 on for K_hat, then kb0 .. for K
    // first exact column of row r: start of its square, or of its band (monotone in r either way)
    auto win_start = [](const auto &a, int r) { return a.sliding ? max(r - a.W + 1, 0) : quotient(r, a.by_w) * a.W; };
    // (what a tile needs of the arguments is read for every tile: kept in registers across the walk, it would not fit)
    auto arguments = []() __attribute__((always_inline)) {
        auto *ap = (const __attribute__((address_space(4))) MfmaArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ap));
        return ap;
    };
    // ---- the tile whose scores are taken: with kStream a tile is opened while the one before is still worked on
    int my_win;                                 // this lane's row's first exact column (both lane halves; past the end: the last row again)
    int wave_first, wave_win_first, wave_win_last;              // first row of the wave, first exact columns of its first and last
    int at_hat, at_kb0, at_nv, at_turns;        // n_hat .. turns
    int at_steady;                              // (kStream) turns up to here, in which the wave masks nothing and requests K_hat two turns ahead
    bf16_t *out_rows;
    auto my_row = [&]() { return min(wave_first + (lane_here() & 31), n - 1); };
    auto take_rows = [&](const auto &a) __attribute__((always_inline)) {
        const int last = a.n - 1;
        wave_first = min(first, last);
        my_win = win_start(a, min(first + (lane_here() & 31), last));
        wave_win_first = win_start(a, wave_first);
        wave_win_last = win_start(a, min(wave_first + 31, last));
        at_hat = n_hat, at_kb0 = kb0, at_nv = nv, at_turns = turns;
        at_steady = min(min(wave_win_first / KB, turns - 4), min(n_hat, a.n / KB) - 2);
        out_rows = o_rows;
    };
    auto take_tile = [&]() __attribute__((always_inline)) { take_rows(*arguments()); };
    auto open_tile = [&](int pos) __attribute__((always_inline)) {
        const auto &a = *arguments();
        const auto &kind = a.kinds[kSplit - 1];
        const int n = a.n, RT = 1 << kind.rt_log2;
        const int at = pos - kind.first;
        int unit, bid;
        if (a.xsplit_log2 >= 0) {
            const int xcd = at & 7, slot = at >> 3;
            const int turn = quotient(slot, a.by_parts);
            const int part = xcd + 8 * (slot - turn * a.by_parts.d); // of this XCD's: xcd, xcd + 8, ...
            unit = part >> a.xsplit_log2;
            bid = (turn << a.xsplit_log2) + (part & ((1 << a.xsplit_log2) - 1));
        } else {
            bid = quotient(at, a.by_units);
            unit = at - bid * a.by_units.d;
        }
        const int row_tile = quotient(bid, a.by_hgroups), hchunk = bid - row_tile * a.by_hgroups.d;
        const int tile = kind.tiles - 1 - row_tile;
        const int b = quotient(unit, a.by_hkv), hk = unit - b * a.by_hkv.d;
        const int i0 = a.q_off + kind.row0 + (tile << kind.rt_log2), i_last = min(i0 + RT - 1, n - 1);   // first and last query position
        Kp = (const char *)(a.K + (size_t)unit * a.ld * D);
        Hp = (const char *)(a.Khat + (size_t)unit * a.ld * D);
        Vp = (const char *)(a.V + (size_t)unit * a.ld * D);
        // a wave's 32 score rows are consecutive rows of one head (RT is a multiple of 32)
        const int head = hk * a.g + hchunk * a.GH + (my_sr >> kind.rt_log2);
        first = i0 + (my_sr & (RT - 1));
        const size_t row0 = ((size_t)b * a.Hq + head) * a.nq - a.q_off;
        q_rows = a.Q + row0 * D;
        o_rows = a.O + row0 * D;
        const int win_first = win_start(a, i0), win_last = win_start(a, i_last);
        n_hat = (win_last + KB - 1) / KB;
        kb0 = win_first / KB;
        nv = n_hat + i_last / KB - kb0 + 1;
        turns = kStream ? max(nv, 2) : (nv + kSplit - 1) / kSplit;
        if constexpr (!kStream) take_rows(a);
    };
    u32x4 qreg[KS];
    // (the addresses are those of the opened tile; in asm, since the compiler, where it counts these loads, waits for
    // them at their first use inside the loop and there drains the tile loads, every turn: wait_loads, then have_queries)
    auto load_queries = [&]() __attribute__((always_inline)) {
        const uint32_t off = min(first + (lane_here() & 31), n - 1) * kRowB + (lane_here() >> 5) * 16;
        for_each_index<KS>([&](auto ks) { load_in_flight<ks * 32>(qreg[ks], (const char *)q_rows, off); });
    };
    auto have_queries = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
    };

    // ---- tile loads: a wave fills kRows rows of the tile (of its own group's block), 1 KiB load i the rows r .. r + 64 / kSeg - 1
    //      of these, lane = (row, segment as stored); the segment it fetches is the stored one permuted by the row number.
    //      A lane's offset from the load's first row never changes, except where the keys end inside a load.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)lds_raw;
    auto keys_perm = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
    auto vals_perm = [](int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };
    constexpr int kRpl = 64 / kSeg;                              // rows per load
    static_assert(kIpw * kRpl == kRows && kRpl * kRowB == 1024, "a wave's loads fill its rows");
    auto lane_off = [&](int i, bool keys, int rows) -> uint32_t { // rows: of the load, those that there are
        const int l = lane_here(), lrow = l / kSeg, r = wave * kRows + i * kRpl + lrow;
        return min(lrow, rows - 1) * kRowB + (((l % kSeg) ^ (keys ? keys_perm(r) : vals_perm(r))) << 4);
    };
    uint32_t k_off[kIpw], v_off[kIpw];
#pragma unroll
    for (int i = 0; i < kIpw; ++i) {
        k_off[i] = lane_off(i, true, kRpl);
        v_off[i] = lane_off(i, false, kRpl);
    }
    // The queries of a tile before which the matrix cores have nothing to do come through LDS, in whole rows: as operands, 32 rows by 32 bytes
    // an instruction, the eight waves' 64 KB went through an L1 of 32 in pieces of its lines (16 x 200 tokens of 20 / 5 heads of 128: 2.3 us until
    // all was asked for, of 16 that a tile took).  Both groups hold the same rows of a split tile: each loads half.  Operands / rows: 16 x 200
    // 28.3 / 27.2 us, 4 x 512 22.4 / 21.5, 1 x 1024 23.9 / 22.8, 4 x 1024 43.7 / 42.8; 32 / 8 heads of 64, 333 tokens 11.8 / 11.5, 2048 32.6 / 32.0.
    constexpr int kQWave = 32 * kRowB, kQLoads = kQWave / 1024 / kSplit;
    const uint32_t lds_q = lds0 + (kBufs + 1) * kTile + my_sr * kRowB;
    static_assert((kBufs + 1) * kTile + (kSplit == 1 ? 8 : 4) * kQWave <= kRoom, "queries");
    auto stage_queries = [&]() __attribute__((always_inline)) {
        const int l = lane_here();
#pragma unroll
        for (int i = 0; i < kQLoads; ++i) {
            const int at = (kSplit == 1 ? 0 : grp * kQLoads) + i, r = at * kRpl + l / kSeg;
            load_to_lds<0>((const char *)q_rows, min(first + r, n - 1) * kRowB + (((l % kSeg) ^ keys_perm(r)) << 4), lds_q + at * 1024);
        }
    };
    auto staged_queries = [&]() __attribute__((always_inline)) {   // behind a barrier; the area is free behind the next one
        const int l = lane_here(), r = l & 31;
        typedef const __attribute__((address_space(3))) u32x4 *lds_vec;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = *(lds_vec)(uintptr_t)(lds_q + r * kRowB + (((2 * ks + (l >> 5)) ^ keys_perm(r)) << 4));
    };
    // first key row that this wave loads of its group's block in a turn, and which rows the scores of that block are taken from
    struct Source {
        const char *keys;
        int row;
    };
    auto source_of = [&](int turn) -> Source {
        const int v = min(kSplit == 1 ? turn : turn * kSplit + grp, nv - 1);   // (past the end: the last block again, unread)
        return {v < n_hat ? Hp : Kp, (v < n_hat ? v : kb0 + v - n_hat) * KB + (wave * kRows) % KB};
    };
    auto lds_of = [&](int buf, bool keys) { return lds0 + (keys ? 0 : kBufs * kTile) + buf * kTile + wave * (kRows * kRowB); };
    auto load_tile = [&](const char *src, int row, uint32_t to, bool keys) __attribute__((always_inline)) {
        if (__builtin_expect(row + kRows <= n, true)) {
            const char *from = src + (size_t)(uint32_t)row * kRowB;
            for_each_index<kIpw>([&](auto i) { load_to_lds<i * 1024>(from, keys ? k_off[i] : v_off[i], to); });
        } else {
#pragma unroll
            for (int i = 0; i < kIpw; ++i) {
                const int first = min(row + i * kRpl, n - 1);
                load_to_lds<0>(src + (size_t)(uint32_t)first * kRowB, lane_off(i, keys, n - first), to + i * 1024);
            }
        }
    };

    f32x16 oacc[MT];
    constexpr bool kMatrixSums = D == 128;      // row sums on the matrix cores
    constexpr float kRaise = 8.f;               // in log2 units: by what a block's maximum has to exceed the running one for that to be raised
    constexpr int kSums = kMatrixSums ? 1 : 4;
    float m_run, l_run[kSums];                  // kMatrixSums: maximum + kRaise - 1, sum; else maximum, this lane half's share of the sum in four chains
    f32x16 s[NT];                               // raw scores of the current block
    u32x4 pb[2 * NT];                           // its probabilities, bf16, as P V operands

    const int row_base = kSplit == 1 ? 0 : grp * KB;             // this group's rows in a tile
    // per-lane addresses inside a tile: every read below is one of these, an exclusive-or of a few bits, a constant
    const uint32_t k_lane = lds0 + (row_base + li) * kRowB + ((half ^ keys_perm(li)) << 4);
    const int L = lane & 15, lg = (lane >> 4) & 1;
    const uint32_t v_lane = lds0 + kBufs * kTile + (row_base + 4 * half + (L >> 2)) * kRowB + (vals_perm(L >> 2) << 4) + lg * 32 + (L & 3) * 8;

    // The row sum is taken over the probabilities as rounded to bf16, i.e. over the very weights that P V uses: the output is then an exact
    // weighted mean of the value rows, and the rounding of the weights cannot bias it (summing the unrounded ones does, by up to 2^-9
    // relative when many weights are equal).  At head_dim 128 on the matrix cores, while a phase's first operands are on their way from LDS: as a
    // 16 x 16 x 32 operand the probabilities of score rows c and c + 16 lie in the same column, of which these ones and zeros take the lanes of
    // one.  A v_dot2c_f32_bf16 waits for a turn of the matrix cores behind the other wave's products: with 16 of them a block a vector phase
    // took 1360 clocks, and no instruction less in it made it shorter; now 1060, the matrix phase 1200.  (4 x 4 x 4 products, of which every lane has its own
    // column, 4 x 8192 tokens 1125 / 1136 us.  At head_dim 64, where the vector ALU is what there is least of and other waves fill such waits, 32 x 2048
    // tokens took 672 / 682 us in this way.)
    const uint32_t one = ((lane >> 2) ^ (lane >> 4)) & 1 ? 0u : 0x3f803f80u;

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
        constexpr int kAhead = D == 64 ? 3 : 4;
        const u32x4 ones = {one, one, one, one};
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};                        // (the lane's row, in every register)
        for_each_index<nv + nk + kAhead>([&](auto i) {
            if constexpr (i >= kAhead) multiply(std::integral_constant<int, i - kAhead>{});
            if constexpr (i < nv + nk) read(i);
            if constexpr (kMatrixSums && nv > 0 && i < 2 * NT)
                sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, pb[i]), sum, 0, 0, 0);
            if constexpr (kMatrixSums && nv > 0 && i == 2 * NT + 2) l_run[0] += sum[0];
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Masks where some row of the wave does not see all of the block, then online softmax: s -> pb.
    auto softmax = [&](int v, auto masks) __attribute__((always_inline)) {   // masks: some row may not see all of the block
        const bool hat = v < at_hat, none = v >= at_nv;          // (none: a turn in which this group has no block)
        const int jb = (hat ? v : at_kb0 + v - at_hat) * KB;
        if (masks && (none || (hat ? jb + KB > wave_win_first : jb < wave_win_last || jb + KB > wave_first + 1))) {
            // the row's columns of the block, [from, to), as bits; two instructions a score: a bit spread over the word chooses (a
            // compare, a select and the wait for the condition between them took 600 clocks a block, half of the softmax itself)
            const int row = my_row();
            const int from = min(max((hat ? 0 : my_win) - jb, 0), KB), to = none ? 0 : min(max((hat ? my_win : row + 1) - jb, 0), KB);
            uint64_t seen = to > 0 ? ~(uint64_t)0 >> (64 - to) : 0;
            seen = from < 64 ? seen >> from << from : 0;
            seen >>= 4 * (lane_here() >> 5);                 // (the lane half's first row is column 4)
#pragma unroll
            for (int T = 0; T < NT; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t take = (uint32_t)__builtin_amdgcn_sbfe((int)(uint32_t)(seen >> (32 * T)), 8 * (r >> 2) + (r & 3), 1);
                    s[T][r] = __uint_as_float((__float_as_uint(s[T][r]) & take) | (0xff800000u & ~take));
                }
        }
        // s -> pb, against m.  kMatrixSums: returns the words of pb or-ed together; else adds them up.
        auto exponentials = [&](float m) __attribute__((always_inline)) {
            uint32_t any = 0;
#pragma unroll
            for (int T = 0; T < NT; ++T)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    f32x2 p;                                     // bare v_exp_f32: tiny results may flush to 0
                    p[0] = __builtin_amdgcn_exp2f(fmaf(s[T][r], a.scale_log2, -m));
                    p[1] = __builtin_amdgcn_exp2f(fmaf(s[T][r + 1], a.scale_log2, -m));
                    const bf16x2 pk = __builtin_convertvector(p, bf16x2);
                    any |= pb[2 * T + (r >> 3)][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
                    if constexpr (!kMatrixSums)                  // (four chains: one would wait for itself)
                        l_run[(r >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pk, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run[(r >> 1) & 3], false);
                }
            return any;
        };
        // the block's maximum, in log2 units
        auto block_max = [&]() __attribute__((always_inline)) {
            // (three operands to an instruction, and not fmaxf, which quiets every operand with an instruction of its own:
            // where a score is NaN its row is NaN either way)
            auto max3 = [](float x, float y, float z) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z); };
            float mx[4];                                         // four chains: one would wait for itself
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                mx[k] = max3(s[0][k], s[0][k + 4], s[0][k + 8]);
                mx[k] = max3(mx[k], s[0][k + 12], s[1][k]);
                mx[k] = __builtin_elementwise_maximum(max3(mx[k], s[1][k + 4], s[1][k + 8]), s[1][k + 12]);
            }
            const float bm = __builtin_elementwise_maximum(max3(mx[0], mx[1], mx[2]), mx[3]);
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
            return __builtin_elementwise_maximum(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * a.scale_log2;
        };
        auto raise = [&](float bm) __attribute__((always_inline)) {
            // (the maximum of a row with a NaN score is NaN at head_dim 128)
            const float m_new = kMatrixSums ? __builtin_elementwise_maximum(m_run, bm + (kRaise - 1.f)) : fmaxf(m_run, bm);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
            m_run = m_new;
#pragma unroll
            for (int k = 0; k < kSums; ++k) l_run[k] *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) oacc[mt] *= alpha;
        };
        // The running maximum is only raised where a block's exceeds it by 2^kRaise: the accumulator is rarely rescaled, and a row's largest
        // weight mostly stays the power of two that bf16 holds exactly.  (Raised beyond 2^60 only, errors against 64 bits are up to 0.5 % larger.)
        if constexpr (kMatrixSums) {
            // The exponentials say themselves whether there is one: they are taken against the maximum as it stands, with m_run so far above it
            // that then, and only then, one is 2 or more and has a bit of its exponent that no smaller one has.  A block's maximum is only looked for
            // where that is so, or some row has none yet, and they are taken again.  With the sums on the matrix cores, and no masks and addresses in
            // most turns, us a call, before / now: 20 / 5 heads of 128, 4 x 8192 tokens 1171 / 1128, 1 x 4096 107.1 / 103.9, 2 x 5003 in a band 263 /
            // 256, 2 x 4096 in pieces of 1024 257 / 251 (the sums alone).
            uint32_t large = 0x40004000u;
            if (!__any(m_run == -INFINITY)) large &= exponentials(m_run);
            if (__builtin_expect(__any(large != 0), false)) {
                const float bm = block_max();
                raise(bm);
                const float m = m_run == -INFINITY ? 0.f : m_run;
                exponentials(m);
                // An infinity or a NaN among them must not meet the zeros of the row whose column it shares: its own row's sum is NaN from here on.  (A NaN
                // score makes the maximum one.)  Finite scores give an infinity too: from 2^31 on half a step of the maximum is 128 or more, by which
                // the exponent, rounded once, can exceed it; below 2^30 an exponent stays below 64.
                if (__builtin_expect(__any(!(fabsf(m) < 0x1p30f)), false)) {
                    uint32_t full = 0;                           // bit 15, 31: an exponent of all ones
#pragma unroll
                    for (int k = 0; k < 2 * NT; ++k)
#pragma unroll
                        for (int j = 0; j < 4; ++j) full |= (pb[k][j] & 0x7f807f80u) + 0x00800080u;
                    const auto both = __builtin_amdgcn_permlane32_swap(full, full, false, false);
                    const bool none = ((both[0] | both[1]) & 0x80008000u) == 0;
                    const uint32_t take = none ? ~0u : 0u;
#pragma unroll
                    for (int k = 0; k < 2 * NT; ++k)
#pragma unroll
                        for (int j = 0; j < 4; ++j) pb[k][j] &= take;
                    l_run[0] = none ? l_run[0] : __builtin_nanf("");
                }
            }
        } else {
            // (at head_dim 64 the scores, kept until that is known, would not fit into the registers)
            const float bm = block_max();
            if (__any(bm > m_run + kRaise)) raise(bm);
            exponentials(m_run == -INFINITY ? 0.f : m_run);
        }
    };

    // ---- the walk.  The tiles of turn t lie in buffers t % kBufs.  The key tile of turn t + 2 and the value tile of turn t + 1 are
    //      requested in turn t's vector phase.  With three buffers nobody reads what those held any more: it was last read in turn t - 1's matrix
    //      phase, and a barrier lies between.  They have landed before the barrier in front of turn t + 2: group A waits for them at the end of turn t + 1's vector phase, group B
    //      at its beginning, in front of the same barrier.  (A fourth buffer, and requests a turn earlier, changed nothing.)
    //      With kSplit = 2 a group reads rows of its own, in two buffers: a barrier more, between matrix and vector phase, frees them, or (kLate) the
    //      requests wait for the turn's one.
    const char *values;                                          // whose value rows are requested next
    int values_row;
    constexpr std::true_type yes;
    constexpr std::false_type no;
    int buf = 0;                                                 // turn % kBufs
    auto after = [](int b) { return b == kBufs - 1 ? 0 : b + 1; };
    auto request = [&](int turn, int key_buf, int value_buf) __attribute__((always_inline)) {   // turn: of the opened tile
        const Source far = source_of(turn);
        load_tile(far.keys, far.row, lds_of(key_buf, true), true);
        load_tile(values, values_row, lds_of(value_buf, false), false);
        values = Vp;
        values_row = far.row;
    };
    auto first_loads = [&]() __attribute__((always_inline)) {
        const Source s0 = source_of(0);
        load_tile(s0.keys, s0.row, lds_of(0, true), true);
        values = Vp;
        values_row = s0.row;
        request(1, 1, 0);
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[mt][r] = 0.f;
        m_run = -INFINITY;
#pragma unroll
        for (int k = 0; k < kSums; ++k) l_run[k] = 0.f;
    };
    auto row_sum = [&]() {
        if constexpr (kMatrixSums) return l_run[0];
        const float l = (l_run[0] + l_run[kSums / 4]) + (l_run[kSums / 2] + l_run[kSums - 1]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    };
    auto packed = [](const f32x16 &o, int q4, float inv) {
        return u32x2{pack_bf16x2(o[4 * q4 + 0] * inv, o[4 * q4 + 1] * inv), pack_bf16x2(o[4 * q4 + 2] * inv, o[4 * q4 + 3] * inv)};
    };
    const int queues = a.xsplit_log2 >= 0 ? 8 : 1, total = a.total, end = a.kinds[kSplit - 1].end;
    uint32_t *const queue = a.queue + (pos & (queues - 1)) * kQueueStride;
    const int handed_out = (int)gridDim.x + (pos & (queues - 1));
    // the counts that the scan has left, by a wave that waits for its first loads meanwhile (positions from the queue are larger), and
    // first by the last work groups, which have the least to do where all of them are there at once
    auto add_up = [&]() __attribute__((always_inline)) {
        if (wave != 7 || pos >= (int)gridDim.x) return;
        const auto &a = *arguments();
        const NnzSum sum = {a.sum.counts, a.sum.nnz, a.sum.groups, a.sum.units};
        if (sum.groups == 0) return;
        for (int u = (int)(gridDim.x - 1 - blockIdx.x); u < sum.units; u += 8 * (int)gridDim.x)
            add_up_nnz(sum, u + (lane >> 3) * (int)gridDim.x);
    };
    const bool asks = kQueue && total > (int)gridDim.x;
    uint32_t ticket = 0;
    // Wave 0 asks for the next tile; in asm, so that nobody waits for the answer (2 us) before it is needed.
    auto ask = [&]() __attribute__((always_inline)) {
        if (asks && wave == 0 && lane_here() == 0)
            asm volatile("s_nop 4\n\tglobal_atomic_add %0, %1, %2, %3 sc0" : "+v"(ticket) : "v"(0), "v"(1), "s"(queue) : "memory");
    };
    int flip = 0;                               // (kStream) two words in turn: wave 0 may be about to write one while group B still reads the other
    // ... and tells the others, once it has waited for the answer; `total`: there is none
    auto tell = [&]() __attribute__((always_inline)) {
        if (wave == 0 && lane_here() == 0) next_tile[flip] = asks ? handed_out + queues * (int)ticket : total;
    };
    auto told = [&]() __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(next_tile[flip]); };

    if constexpr (kStream) {
        // A finished tile's outputs, from row `from` on, turned in LDS behind the tiles into whole rows, each wave its own, half of the
        // channels at a time (that is the room).  As 8 bytes of 32 rows a store they kept a vector phase waiting: 20 / 5 heads of 128, 64 x
        // 512 tokens 212 / 192 us, 256 x 64 58.4 / 49.1, 4 x 2048 110.6 / 106.0.
        constexpr int kHSeg = D / 16, kHStores = 32 * kHSeg * 16 / 1024;
        auto store_rows = [&](bf16_t *to, int from, float inv) __attribute__((always_inline)) {
            typedef __attribute__((address_space(3))) u32x2 *lds_pair;
            typedef const __attribute__((address_space(3))) u32x4 *lds_vec;
            const int l = lane_here(), row = l & 31, seg = l % kHSeg;
            const uint32_t at = lds0 + 2 * kBufs * kTile + wave * (32 * kHSeg * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int c = 0; c < kHSeg; ++c)
                    *(lds_pair)(uintptr_t)(at + row * (kHSeg * 16) + ((c ^ (row & (kHSeg - 1))) << 4) + 8 * (l >> 5)) =
                        packed(oacc[h * (MT / 2) + (c >> 2)], c & 3, inv);
#pragma unroll
                for (int k = 0; k < kHStores; ++k) {
                    const int r = k * (64 / kHSeg) + l / kHSeg;
                    *(u32x4 *)(to + (ptrdiff_t)min(from + r, n - 1) * D + h * (D / 2) + seg * 8) =
                        *(lds_vec)(uintptr_t)(at + r * (kHSeg * 16) + ((seg ^ (r & (kHSeg - 1))) << 4));
                }
            }
        };
        static_assert(2 * kBufs * kTile + 8 * 32 * kHSeg * 16 <= kRoom, "outputs");
        // Tile follows tile without a pause: the requests run two turns ahead of the scores, across the end of a tile into the
        // next one, and the phase that adds up a tile's last values takes the scores of the next one's first keys.  Its
        // outputs are stored in the vector phase after that.  (Drained and filled again, and with queries and outputs in
        // pieces, a tile cost 16 to 19 K clocks beside its turns of 3.2 K.)  The next tile is asked for so early that its number is there when it is opened, two
        // turns before the end; hence at least two turns a tile (the second one sees nothing where there is one block).
        open_tile(pos);
        stage_queries();
        first_loads();
        bool early = turns < 4;                                  // (too short to ask on the way)
        if (early) ask();
        add_up();
        take_tile();
        clear();
        int turn = 0, opened = 2;                                // of the tile that is worked on; requested turns of the opened one
        bool ahead = false, full = false;                        // the opened tile is the next one; the accumulators hold a finished tile
        bf16_t *full_rows = nullptr;                             // its rows
        int full_first = 0, taken = first;
        bool stored = false;                                     // in the vector phase before
        wait_loads<0>();
        if (early) tell();
        phase_barrier();
        staged_queries();
        phase_barrier();                                         // (their area is free)
        matrix_phase(no, yes, 0, 0);
        while (true) {
            // the key tile of turn + 1 and the value tile of turn (loads and stores end in order)
            if (grp == 1) {
                if (stored)
                    wait_loads<2 * kHStores>();
                else
                    wait_loads<0>();
                phase_barrier();
            }
            __builtin_amdgcn_s_setprio(0);
            const bool last = turn == at_turns - 1;
            if (last && ahead) load_queries();                   // (nobody multiplies by the old ones any more)
            if (opened == turns && !ahead) {
                const int next = told();
                if (next < end) {
                    open_tile(next);
                    ahead = true;
                    opened = 0;
                    flip ^= 1;
                }
            }
            request(opened, after(after(buf)), after(buf));
            const bool asking = opened == turns - 2, telling = opened == turns - 1;
            if (opened < turns) ++opened;
            const bool stores = full && full_first < n;
            if (full) {
                const float inv = 1.f / row_sum();
                if (stores) store_rows(full_rows, full_first, inv);
                clear();
            }
            softmax(turn, yes);
            __builtin_amdgcn_s_setprio(1);                       // (for the matrix phase that follows)
            if (grp == 0 || (last && ahead)) {                   // what was asked for in earlier turns, the queries
                if (stores)
                    wait_loads<kLoads + 2 * kHStores>();
                else
                    wait_loads<kLoads>();
            }
            have_queries();
            if (telling) tell();
            if (asking) ask();
            if (grp == 0) phase_barrier();
            const int prev = buf;
            buf = after(buf);
            if (last && !ahead) break;
            matrix_phase(yes, yes, prev, buf);
            stored = stores;
            full = last;
            if (last) {
                full_rows = out_rows;
                full_first = taken;
                taken = first;
                take_tile();
                ahead = false;
                turn = 0;
            } else {
                ++turn;
            }
            // most turns of a long tile: the blocks left of all windows, one array after the other, nothing masked, nothing past the end, and
            // nothing else to be done - not the first one, which stores, nor the last four
            if (turn > 0 && turn < at_steady) {
                const char *keys = Hp + (size_t)(uint32_t)(opened * KB + wave * kRows) * kRowB;
                const char *vals = Vp + (size_t)(uint32_t)values_row * kRowB;
                const int from = turn;
                for (; turn < at_steady; ++turn) {
                    if (grp == 1) {
                        wait_loads<0>();
                        phase_barrier();
                    }
                    __builtin_amdgcn_s_setprio(0);
                    const int prev = buf, far = after(after(buf));
                    buf = after(buf);
                    loads_to_lds(keys, k_off, lds_of(far, true));
                    loads_to_lds(vals, v_off, lds_of(buf, false));
                    keys += KB * kRowB;
                    vals += KB * kRowB;
                    softmax(turn, no);
                    __builtin_amdgcn_s_setprio(1);
                    if (grp == 0) {
                        wait_loads<kLoads>();
                        phase_barrier();
                    }
                    matrix_phase(yes, yes, prev, buf);
                }
                opened += turn - from;
                values_row += (turn - from) * KB;
                values = Vp;
                stored = false;
            }
        }
        matrix_phase(yes, no, buf == 0 ? kBufs - 1 : buf - 1, 0);
        wait_loads<0>();                                         // no load into LDS outlives the work group
        const float inv = 1.f / row_sum();
        if (taken < n) store_rows(out_rows, wave_first, inv);
        return told();
    } else {
        // kLate: one barrier a turn with two tiles of each kind, the next ones requested behind it.  A work group that has its compute unit for itself is done
        // sooner (32 / 8 heads of 64, 2048 tokens: 2711 -> 2567 clocks a turn); of two that share one the first is not so far ahead of the second any
        // more (1.53 and 2.9 us a turn -> 1.75 and 2.7), see launch_d.  At head_dim 128 64 KB at once take the address path longer than is saved (3046 -> 3430).
        static_assert(!kLate || kSplit > 1, "whole tiles have the room");
        int asks_at = -1;                                        // (kLate) the turn, for the wave that does: two instructions in front of a matrix phase
        auto vector_phase = [&](int turn) __attribute__((always_inline)) {
            auto ends_turn = [&]() __attribute__((always_inline)) {
                wait_loads<0>();                                 // key tile turn + 1, value tile turn
                phase_barrier();
            };
            auto requests = [&]() __attribute__((always_inline)) { request(turn + 2, after(after(buf)), after(buf)); };
            if (kSplit == 1 || kLate) {
                if (grp == 1) ends_turn();
            } else {
                phase_barrier();
            }
            __builtin_amdgcn_s_setprio(0);
            if (!kLate || grp == 1) requests();
            softmax(kSplit == 1 ? turn : turn * kSplit + grp, yes);
            // asked for three turns before the tile ends: whoever asks first gets the longest tile left.  Behind the turn's loads, where a wait for
            // older ones does not wait for it, and kLate behind the turn's barrier, where none comes before the next turn's.
            if (!kLate && turn == max(turns - 3, 0)) ask();
            __builtin_amdgcn_s_setprio(1);                       // (for the matrix phase that follows)
            if constexpr (kLate) {
                if (grp == 0) {
                    ends_turn();
                    requests();
                    if (turn == asks_at) ask();                  // (wave 0 is one of these)
                }
            } else if (kSplit > 1 || grp == 0) {
                wait_loads<kLoads>();
                phase_barrier();
            }
        };
        open_tile(pos);
        stage_queries();
        first_loads();
        add_up();
        wait_loads<kLoads>();                                    // the queries and the first keys; the rest like any turn's
        while (true) {
            clear();
            buf = 0;
            if constexpr (kLate) asks_at = asks && wave == 0 ? max(turns - 3, 0) : -1;
            phase_barrier();
            staged_queries();
            if (kSplit == 1 || (!kLate && grp == 1)) phase_barrier();   // (the area is free; group B starts one phase later)
            matrix_phase(no, yes, 0, 0);
            vector_phase(0);
            for (int turn = 1; turn < turns; ++turn) {
                const int prev = buf;
                buf = after(buf);
                matrix_phase(yes, yes, prev, buf);
                vector_phase(turn);
            }
            matrix_phase(yes, no, buf, 0);
            if (kSplit > 1 && !kLate && grp == 0) phase_barrier();   // (group B's last vector phase)
            wait_loads<0>();                                     // no load into LDS outlives its tile
            const float l_tot = row_sum();
            tell();
            constexpr int MO = MT / kSplit;                      // channel tiles that this wave stores
            u32x2 words[MO][4];
            __syncthreads();                                     // the tiles are done with
            pos = told();
            const int lane = lane_here();
            if constexpr (kSplit == 1) {
                const float inv = 1.f / l_tot;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) words[mt][q4] = packed(oacc[mt], q4, inv);
            } else {
                // wave w of group A and wave w of group B hold the same rows: each hands the other half of its channels over and
                // finishes its own half
                float *xo = (float *)lds_raw;                    // [group][wave of the group][MO][16][64]
                float *xm = xo + 2 * 4 * MO * 16 * 64;           // [group][wave of the group][64][2] maximum, sum
                const int w4 = wave & 3, other = 1 - grp;
#pragma unroll
                for (int mo = 0; mo < MO; ++mo)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        xo[(((grp * 4 + w4) * MO + mo) * 16 + r) * 64 + lane] = grp == 0 ? oacc[MO + mo][r] : oacc[mo][r];
                xm[((grp * 4 + w4) * 64 + lane) * 2] = m_run;
                xm[((grp * 4 + w4) * 64 + lane) * 2 + 1] = l_tot;
                __syncthreads();
                const float m2 = xm[((other * 4 + w4) * 64 + lane) * 2], l2 = xm[((other * 4 + w4) * 64 + lane) * 2 + 1];
                const float M = fmaxf(m_run, m2);                // (a row sees its own key: one of the two is finite)
                const float f1 = __builtin_amdgcn_exp2f(m_run - M), f2 = __builtin_amdgcn_exp2f(m2 - M);
                const float inv = 1.f / (l_tot * f1 + l2 * f2);
#pragma unroll
                for (int mo = 0; mo < MO; ++mo) {
                    f32x16 o;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float x = xo[(((other * 4 + w4) * MO + mo) * 16 + r) * 64 + lane];
                        o[r] = (grp == 0 ? oacc[mo][r] : oacc[MO + mo][r]) * f1 + x * f2;
                    }
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) words[mo][q4] = packed(o, q4, inv);
                }
                __syncthreads();                                 // the exchange is done with
            }
            // The outputs turn in LDS, each wave its own, from 8 bytes of 32 rows a store to whole rows: 16 pieces of 16 bytes a row were 4096
            // writes of partial lines from a work group at head_dim 128, 1.8 us at the end of its tile (8 bytes / rows: 20 / 5 heads of 128, 16 x
            // 200 tokens 27.1 / 25.1 us, 4 x 512 21.6 / 19.4, 4 x 1024 42.2 / 38.5, 64 x 64 26.1 / 22.1; 32 / 8 heads of 64, 2048 tokens 31.8 / 31.0).
            constexpr int kOSeg = D / kSplit / 8, kORow = kOSeg * 16, kOStores = 32 * kORow / 1024;   // 16-byte segments of a row here
            typedef __attribute__((address_space(3))) u32x2 *lds_pair;
            typedef const __attribute__((address_space(3))) u32x4 *lds_vec;
            const uint32_t o_lds = lds0 + wave * (32 * kORow);
            const int o_row = lane & 31, o_seg = lane % kOSeg;
#pragma unroll
            for (int mo = 0; mo < MO; ++mo)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *(lds_pair)(uintptr_t)(o_lds + o_row * kORow + (((4 * mo + q4) ^ (o_row & (kOSeg - 1))) << 4) + 8 * (lane >> 5)) = words[mo][q4];
            u32x4 rows[kOStores];
#pragma unroll
            for (int k = 0; k < kOStores; ++k) {
                const int r = k * (64 / kOSeg) + lane / kOSeg;
                rows[k] = *(lds_vec)(uintptr_t)(o_lds + r * kORow + ((o_seg ^ (r & (kOSeg - 1))) << 4));
            }
            lds_barrier();                                       // all have turned theirs: the next tile's loads may come, of either kind
            bf16_t *const o_to = out_rows + (kSplit > 1 ? grp * (D / 2) : 0) + o_seg * 8;
            const int o_first = wave_first + lane / kOSeg;
            const bool more = pos < end, stores = first < n;     // (first: still this tile's)
            // the next tile's loads go out, then the outputs: its first keys are on their way while these are stored
            if (more) {
                open_tile(pos);
                stage_queries();
                first_loads();
            }
            if (stores) {
#pragma unroll
                for (int k = 0; k < kOStores; ++k) *(u32x4 *)(o_to + (ptrdiff_t)min(o_first + k * (64 / kOSeg), n - 1) * D) = rows[k];
            }
            if (stores)
                wait_loads<kOStores + kLoads>();                 // the queries and the first keys
            else
                wait_loads<kLoads>();
            if (!more) return pos;
        }
    }
}

// Work groups go to the 8 XCDs round-robin by index, and every work group takes further tiles from a counter, in order, so no
// compute unit is idle while there are tiles: the longest (last) tiles of every unit come first, the shortest last.  (One work
// group per tile instead is started in order, each on a compute unit of the shader engine whose turn it is, and waits for
// that one.)  Every XCD has its own L2, and all tiles of a unit stream the same K, K_hat and V: where the units - or
// units cut by tile index modulo 2^xsplit_log2 - deal out evenly, an XCD keeps to its own, with a counter of its own.
// Where all tiles are resident at once, two to a compute unit, the second ones come in ascending order, so that short ones share
// with long ones.
// Behind the tiles come the chunks that a cache is handed (fill_chunk), for whoever is done with the tiles or has none: a piece of a
// prompt, or a short one, leaves compute units idle, and the hand-off's own launch took 9 us of each.
// (kernels of their own: with the look for such a chunk at its end every other launch took 0.5 to 1 us longer.)
// kForm 1: kStream at head_dim 128, kLate at 64; 2: kLate where every work group has one tile and none asks for another.  Fill: CacheFill, or nothing
template <int D, int kForm, typename... Fill>
__global__ __launch_bounds__(512, D == 64 ? 4 : 2) void prefill_mfma_kernel(MfmaArgs a, Fill...) {
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    int pos = blockIdx.x;
    if (pos >= a.turn_at && pos < a.blocks) pos = a.blocks - 8 - ((pos - a.turn_at) & ~7) + (pos & 7);
    if (pos < a.kinds[1].end) pos = tiles_of_kind<D, 2, false, kForm != 0 && D == 64, kForm != 2>(a, pos, lds_raw);
    if (pos < a.kinds[0].end) pos = tiles_of_kind<D, 1, kForm != 0 && D == 128, false, kForm != 2>(a, pos, lds_raw);
    if constexpr (sizeof...(Fill) == 0) return;
    // (the arguments of what follows are read here: in registers from the start on they would push others out across the walk)
    typedef const __attribute__((address_space(4))) char arg_char;
    auto *args = (arg_char *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const auto &b = *(const __attribute__((address_space(4))) MfmaArgs *)args;
    static_assert(sizeof(MfmaArgs) % alignof(CacheFill) == 0, "the second argument follows the first");
    const auto &fill = *(const __attribute__((address_space(4))) CacheFill *)(args + sizeof(MfmaArgs));
    static_assert(kFillLds<D> <= 4 * KB * 2 * D * 2, "the room of the tiles");
    int *const next = (int *)(lds_raw + 4 * KB * 2 * D * 2);
    const int tid = (int)threadIdx.x;
    while (pos < b.total) {
        __syncthreads();                                         // the LDS is free
        if (tid == 0) {
            const int queues = b.xsplit_log2 >= 0 ? 8 : 1, mine = pos & (queues - 1);
            *next = b.total > (int)gridDim.x ? (int)gridDim.x + mine + queues * (int)atomicAdd(b.queue + mine * kQueueStride, 1u) : b.total;
        }
        fill_chunk<D, 512>(fill, pos - b.blocks, lds_raw, tid);
        pos = *next;
    }
}

// Loads straight into LDS want aligned rows; a tensor that does not start on 16 bytes (a slice of a larger one) is laid out
// anew in front of the launch.  (The kernel of binary32 products needs no alignment, but took 1148 instead of 154 us on 1 x 4096
// tokens, 20 / 5 heads of 128, 14.7 instead of 1.30 ms on 4 x 8192; with the copies 160 us and 1.25 ms.  Queries and outputs, which move once, start
// anywhere: 16 bytes of global memory a lane at any address, bit for bit the same.)
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
struct CopyPair {
    const u32x4_any *src[2];
    u32x4 *dst[2];
};
__global__ __launch_bounds__(256) void copy_aligned_kernel(CopyPair c, size_t pieces) {
    constexpr int N = 4;
    const u32x4_any *src = c.src[blockIdx.y];
    u32x4 *dst = c.dst[blockIdx.y];
    const size_t i0 = (size_t)blockIdx.x * (256 * N) + threadIdx.x;
    u32x4 v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = src[min(i0 + k * 256, pieces - 1)];
#pragma unroll
    for (int k = 0; k < N; ++k)
        if (i0 + k * 256 < pieces) dst[i0 + k * 256] = v[k];
}

// as many work groups as are resident at once: one per compute unit, at head_dim 64 two (64 KB of LDS, 128 registers)
int resident(int d) {
    const int cus = device_cu_count() >= 8 ? device_cu_count() & ~7 : 8;
    return d == 64 ? 2 * cus : cus;
}

template <int D>
void launch_d(const PrefillArgs &p, const CacheFill *fill, hipStream_t s) {
    MfmaArgs a;
    a.Q = (const bf16_t *)p.Q;
    a.K = (const bf16_t *)p.K;
    a.Khat = (const bf16_t *)p.Khat;
    a.V = (const bf16_t *)p.V;
    a.O = (bf16_t *)p.O;
    a.Hq = p.Hq;
    a.n = p.n;
    a.W = p.W;
    a.sliding = p.sliding;
    a.ld = p.ld > 0 ? p.ld : p.n;
    a.q_off = p.q_off;
    a.nq = p.nq;
    a.scale_log2 = p.scale_log2;
    a.queue = p.queue;
    a.sum = p.sum;
    const int units = p.B * p.Hkv, g = p.Hq / p.Hkv;
    a.GH = (g % 4 == 0) ? 4 : (g % 2 == 0) ? 2 : 1;
    const int rt = 256 / a.GH, hgroups = g / a.GH;               // rows of a whole tile
    a.g = g;
    a.by_hkv = divisor(p.Hkv);
    a.by_hgroups = divisor(hgroups);
    a.by_w = divisor(p.W);
    a.by_units = divisor(units);
    const int slots = resident(D), cus = D == 64 ? slots / 2 : slots;
    // XCD-aware order needs units * 2^xsplit parts to deal out evenly over 8 XCDs and a unit's tiles, of either kind, to split
    // evenly
    int xsplit = 0;
    while ((units << xsplit) % 8 != 0) ++xsplit;
    auto even = [&](int tiles) { return (tiles * hgroups) % (1 << xsplit) == 0; };
    // Whole tiles for the first rows, split ones for the rest.  Of some ways to cut, the one that promises to be done first: with
    // the tiles in order of length, longest first, a launch on C compute units lasts at least as long as its work / C, and as
    // the k + 1 shortest of its kC + 1 longest tiles, which some compute unit has to take; the estimate is the largest of these.
    // In units of a whole tile's turn a tile costs kWhole or kHalf beside its turns, and a split one's turn kHalfTurn (fitted to 250
    // timed launches of 42 shapes, 8 % off on the average; head_dim 64: work of the two that share a compute unit, where one
    // alone takes kAlone times as long).  That was with two barriers a turn in all tiles, and a whole tile's turn is shorter since; with the present
    // kernels, 26 shapes, the chosen cut is 0.7 % slower on the average than the best of up to 11 at head_dim 128 (the worst 3 x 1436 tokens of 32 / 8 heads, 81.8 / 78.8 us) and
    // 0.6 % at 64 (3 x 2500 of 16 / 2 in a sliding window, 68.5 / 66.8); before, of up to 13, 1.0 and 1.1 %, where looking at k = 1 alone was 6.0 and 3.9 %: 1 x 4096 tokens, 20 / 5 heads
    // of 128, 103 -> 93 us, 2 x 5003 in a sliding window 276 -> 247, 4 x 512 26.7 -> 22.4, 4 x 1024 48.1 -> 43.1.
    constexpr float kWhole = D == 128 ? 6.5f : 4.2f, kHalf = D == 128 ? 6.5f : 4.4f, kHalfTurn = D == 128 ? 1.22f : 0.93f, kAlone = D == 128 ? 1.f : 1.19f;
    const int all = (p.nq + rt - 1) / rt, columns = units * hgroups;
    // turns of a tile of R rows from row i0 on (see open_tile)
    auto turns = [&](int i0, int R) {
        auto win_start = [&](int r) {
            return p.sliding ? (r - p.W + 1 > 0 ? r - p.W + 1 : 0) : (int)(((uint64_t)(2u * (uint32_t)r) * a.by_w.mul >> 32) >> a.by_w.shift) * p.W;
        };
        i0 += p.q_off;
        const int last = (i0 + R < p.n ? i0 + R : p.n) - 1;
        return (win_start(last) + KB - 1) / KB + last / KB - win_start(i0) / KB + 1;
    };
    auto cut = [&](int whole, bool ordered) {
        const int rows = whole * rt < p.nq ? whole * rt : p.nq, split = (p.nq - rows + rt / 2 - 1) / (rt / 2);
        a.kinds[1] = {__builtin_ctz(rt / 2), split, rows, 0, columns * split};
        a.kinds[0] = {__builtin_ctz(rt), whole, 0, columns * split, columns * (whole + split)};
        a.xsplit_log2 = ordered ? xsplit : -1;
    };
    constexpr int kMost = 1024;                                  // row tiles that are looked at: with more, all stay whole
    if (all > kMost) {
        cut(all, xsplit < 3 && even(all));
    } else {
        float whole_cost[kMost], half_cost[2 * kMost];           // of a row tile, and of every half of one
        const int halves = (p.nq + rt / 2 - 1) / (rt / 2);
        for (int t = 0; t < all; ++t) whole_cost[t] = kWhole + (float)turns(t * rt, rt);
        for (int t = 0; t < halves; ++t) half_cost[t] = kHalf + kHalfTurn * (float)((turns(t * (rt / 2), rt / 2) + 1) / 2);
        // (few ways where there are many tiles to a compute unit: less is at stake)
        const bool many = (int64_t)all * columns > 8 * (int64_t)cus;
        const int ways = many ? 32 : 10, step = (all + ways - 1) / ways, fewest = many ? all - 4 * step : 0;
        float best = INFINITY;
        for (int whole = all;; whole = whole > step ? (whole - 1) / step * step : 0) {   // row tiles that stay whole
            const int split = halves > 2 * whole ? halves - 2 * whole : 0;
            // on `some` compute units, of which those of a row tile's columns that `of` says come
            auto estimate = [&](int some, auto of) {
                float work = 0.f, lasts = 0.f;
                int64_t tiles = 0, level = 0;                    // tiles so far; the next k
                for (int w = whole - 1, h = halves - 1; w >= 0 || h >= 2 * whole;) {
                    const bool takes_half = w < 0 || (h >= 2 * whole && half_cost[h] > whole_cost[w]);
                    const int n = of(takes_half ? halves - 1 - h : whole - 1 - w);
                    const float cost = takes_half ? half_cost[h--] : whole_cost[w--];
                    tiles += n;
                    work += cost * (float)n;
                    for (; tiles > level * some; ++level) lasts = fmaxf(lasts, (float)(level + 1) * cost * (level == 0 ? kAlone : 1.f));
                }
                return fmaxf(lasts, work / (float)some);
            };
            // In XCD-aware order the XCDs that take tiles 0, 2^xsplit, ... of their units, the longest, are done last; in the other one
            // every XCD streams every unit, which costs 2 % (timed, -4 to 4).  20 / 5 heads of 128, in XCD-aware order wherever the parts deal out /
            // as chosen: 14 x 200 tokens 36 / 27, 10 x 1000 93 / 84, 2 x 2500 85 / 78, 6 x 2500 220 / 208; 32 / 8 of 64 stay as they are.
            const int64_t tiles = (int64_t)columns * (whole + split);
            const bool paired = D == 64 && tiles > cus && tiles <= slots, orders = xsplit < 3 && even(whole) && even(split);
            float lasts = 1.02f * estimate(cus, [&](int) { return columns; });
            bool ordered = false;
            if (orders) {
                const int mine = (units << xsplit) / 8, part = (1 << xsplit) - 1;
                const float as = estimate(cus / 8, [&](int tile) {
                    return mine * ((tile * hgroups + hgroups + part) / (part + 1) - (tile * hgroups + part) / (part + 1));
                });
                ordered = paired || as <= lasts;
                if (ordered) lasts = as;
            }
            if (paired) {                                        // tile j shares with the j-th last one (turn_at)
                auto cost_at = [&](int at) { return at < split ? half_cost[halves - 1 - at] : whole_cost[whole - 1 - (at - split)]; };
                for (int j = 0; j < (int)tiles - cus; j += columns > 8 ? columns : 8)
                    lasts = fmaxf(lasts, cost_at(j / columns) + cost_at(((int)tiles - 1 - j) / columns));
                lasts = fmaxf(lasts, cost_at(((int)tiles - cus - 1) / columns) + cost_at(cus / columns));
            }
            if (lasts <= best) {                                 // (of equals the one with more split tiles: the rest are done earlier)
                best = lasts;
                cut(whole, ordered);
            }
            if (whole <= fewest || whole == 0) break;
        }
    }
    a.blocks = a.kinds[0].end;
    a.total = a.blocks + (fill ? fill->items : 0);
    const bool ordered = a.xsplit_log2 >= 0;
    if (ordered) a.by_parts = divisor((units << xsplit) / 8);
    a.turn_at = D == 64 && a.blocks > cus && a.blocks <= slots && ordered ? cus : a.blocks;
    constexpr int lds = 4 * KB * 2 * D * 2 + 16;                 // split tiles take more
    static_assert(lds >= 6 * KB * D * 2 + 16 && lds >= 2 * 4 * (D / 64) * 16 * 64 * 4 + 2 * 4 * 64 * 2 * 4, "whole tiles, the merge");
    // Tile after tile without a pause where that many follow each other, or long ones do (head_dim 128, 20 / 5 heads, pausing / not:
    // 1 x 4096 tokens 104 / 102 us, 26 x 512 77.8 / 73.5, 133 x 64 34.8 / 32.1, though 27 x 900 173 / 179); for a second tile of few turns
    // what is done beside two groups' turns in turn takes longer than a pause (7 x 598 34.7 / 35.4, 4 x 512 18.3 / 18.7).  (Those with two barriers a turn.  With one,
    // calls of 25 shapes, pausing / not: taken 1 x 5390 of 20 / 5 heads 160.5 / 157.3, 1 x 5487 of 32 / 8 254.6 / 250.2, 4 x 8319 of 8 / 8 575 / 565, the least 4 x 3718 of 8 / 8 158.2 / 159.9; not
    // taken 6 x 527 of 32 / 8 44.9 / 45.8, 3 x 1409 of 16 / 2 47.7 / 49.0, the most 1 x 2138 of 32 / 8 61.0 / 60.2.)  At head_dim
    // 64 the other work group of the compute unit fills the pause, and over 27 launches of 64 to 1400 tokens pausing was faster by 0.9 % on the
    // average, -4 to 12 (32 / 8 heads: 512 x 64 83.6 / 80.5, 55 x 130 32.9 / 36.9, 16 x 700 61.8 / 64.1, 12 x 1024 82.4 / 86.0, 8 x 1500 106 / 107,
    // 4 x 4096 306 / 306).
    const int64_t whole_tiles = (int64_t)columns * a.kinds[0].tiles;
    // At head_dim 64 instead: one barrier a turn for split tiles, too (kLate), where most tiles are split and about all of them are resident at once, or so many follow
    // that it does not matter which of the two work groups of a compute unit is done first; between that the longest tiles, which came first, would end
    // last.  Times as fast with it over 190 launches of 440 to 3024 tiles: up to 537 tiles, three quarters of them split or more 1.037 on the geometric
    // mean (0.943 to 1.085), fewer 0.984 (0.949 to 1.007; 70 to 75 % of an earlier build 0.997); 538 to 997 tiles 1.00 (0.85 to 1.09, gains where nearly all of at most 560 are split); more, a
    // third or more split 1.033 (1.003 to 1.066), fewer 1.005 (0.985 to 1.023; whole tiles alone 1.000).  Two barriers / one, us a call, of 16 / 2 heads: 1 x 4672 tokens, 456
    // of 520 tiles split, 83.2 / 77.2, 2 x 3099, 296 of 536, 72.8 / 74.3, 1 x 8201, 508 of 768, 177 / 209, 3 x 6923, 1020 of 1812, 338 / 330.
    const int64_t tiles64 = a.blocks;
    const bool late = 20 * tiles64 <= 21 * slots ? 4 * (int64_t)a.kinds[1].end >= 3 * tiles64 : 20 * tiles64 >= 39 * slots;
    const bool stream = D == 64 ? late : (2 * whole_tiles >= 5 * slots || (whole_tiles > slots && p.q_off + a.kinds[0].tiles * rt / 2 >= 24 * KB));
    const dim3 grid(a.total < slots ? a.total : slots), block(512);
    // (kLate with / without the look for the turn to ask in, launches that need none: 1 x 2048 tokens of 32 / 8 heads 36.4 / 36.0 us, 1 x 3000 of 16 / 2 46.3 / 45.7, 4 x 2048 of 8 / 8 42.3 / 42.1)
    constexpr int kResident = D == 64 ? 2 : 1;
    const int form = stream ? (a.total <= slots ? kResident : 1) : 0;
    static std::atomic<uint64_t> lds_set[6];                     // per instantiation, one bit per device
    if (fill) {
        const auto kernel = form == 0 ? prefill_mfma_kernel<D, 0, CacheFill> : form == 1 ? prefill_mfma_kernel<D, 1, CacheFill> : prefill_mfma_kernel<D, kResident, CacheFill>;
        ensure_dynamic_lds((const void *)kernel, lds, lds_set[3 + form]);
        hipLaunchKernelGGL(kernel, grid, block, lds, s, a, *fill);
        return;
    }
    const auto kernel = form == 0 ? prefill_mfma_kernel<D, 0> : form == 1 ? prefill_mfma_kernel<D, 1> : prefill_mfma_kernel<D, kResident>;
    ensure_dynamic_lds((const void *)kernel, lds, lds_set[form]);
    hipLaunchKernelGGL(kernel, grid, block, lds, s, a);
}

}  // namespace

bool prefill_mfma_supported(const PrefillArgs &p) {
    return p.dtype == 1 && (p.d == 64 || p.d == 128) &&
           (size_t)p.B * p.Hkv * ((p.n + 31) / 32) * (p.Hq / p.Hkv) < ((size_t)1 << 31);
}

void launch_copy_aligned(PrefillArgs &a, void *room_k, void *room_v, size_t bytes, hipStream_t s) {
    CopyPair c = {};
    int count = 0;
    auto take = [&](const void *&tensor, void *room) {
        if (((uintptr_t)tensor & 15) == 0) return;
        c.src[count] = (const u32x4_any *)tensor;
        c.dst[count++] = (u32x4 *)room;
        tensor = room;
    };
    take(a.K, room_k);
    take(a.V, room_v);
    if (!count) return;
    const size_t pieces = bytes / 16;
    hipLaunchKernelGGL(copy_aligned_kernel, dim3((unsigned)((pieces + 1023) / 1024), count), dim3(256), 0, s, c, pieces);
}

void launch_prefill_mfma(const PrefillArgs &p, const CacheFill *fill, hipStream_t s) {
    if (p.d == 64)
        launch_d<64>(p, fill, s);
    else
        launch_d<128>(p, fill, s);
}

// A chunk by an attention launch's work groups, two of which at most share a compute unit, takes longer than by six small ones of a launch of its own; what
// that launch costs is its start and end.  In that launch / this one, us a call (prompt, hand-off, one decode step) at items per resident work group:
// 32 / 8 heads of 64, 1 x 512 tokens 0.1 31.3 / 25.9, 4 x 512 0.5 39.0 / 36.7, 2 x 8192 of 16 / 2 1 338 / 326, 16 x 600 2.5 77.3 / 76.1, 32 x 1024 8 242 / 254; 20 / 5 heads
// of 128, 1 x 512 0.2 36.7 / 30.1, 8 x 500 1.3 55.5 / 49.8, 4 x 2048 2.5 135 / 129, 1 x 8192 2.5 352 / 340, 32 x 300 of 8 / 8 heads 3.1 89.9 / 95.3, 16 x 1024 5 168 / 170, 4 x
// 6000 7.3 676 / 682.
bool prefill_takes_fill(const PrefillArgs &p, const CacheFill &fill) { return 2 * (int64_t)fill.items <= 5 * (int64_t)resident(p.d); }

}  // namespace da
