// Hybrid-attention prefill for bf16 inputs, head_dim 64 or 128 (Sec. III-B prefill stage; Eq. 4; Eq. 1).
//
// Work group = 512 threads (8 waves) on 256 "score rows": RT consecutive query rows x GH query heads of
// one KV head (they share K, V and the delta matrix).  Key columns are walked left to right in blocks
// of 32.  A row's window is its square of side W on the diagonal, or the band of the W newest keys.
//
//   left of the window   the running score of Eq. 4 is, by the telescoped sum of the delta rows up to column j, the
//                        product of the query with the held key, q . k_hat(j): K_hat Q^T on the matrix cores.
//                        DA_SCORE_GATHER takes this form here too.  Adding up the surviving entries one by one on the
//                        vector ALU (fp16 q from LDS, v_fma_mix_f32, 4 cycles for 64 products) was bound by
//                        instruction issue and LDS at 8.1 ms on 4 x 8192 tokens, 20 / 5 heads of 128, 60 % sparsity,
//                        where the matrix cores take 1.45 ms for all products: a dense product of 32 x 32 x 16 costs
//                        32 cycles, the survivors of the same block about 16 times that, and even a block without
//                        any survivor cost more in the exchange of its column updates than its dense product.
//                        The product sums head_dim terms in binary32 instead of every delta so far.
//   inside the window    exact scores K Q^T; where a tile straddles windows, both products and a select per element
//   every block          online softmax with lane-local row state, P V on the matrix cores with V pre-transposed.
//
// Matrix-core layouts (v_mfma_f32_32x32x16_bf16, wave64): A lane l holds row l%32, k = 8*(l/32)..+7;
// B lane l holds column l%32, same k; D lane l holds column l%32, rows 8*(r/4) + 4*(l/32) + r%4 for
// register r.  Scores are produced transposed (keys x score rows) so that a lane owns one score row,
// and D registers 8a..8a+7 are exactly the B operand of the a-th k-step of P V once V^T is fetched in
// the matching key order.
#include "common.hpp"
#include "kernels.hpp"
#include "scan_device.hpp"
#include "vt_device.hpp"

namespace da {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kRows = 256;      // score rows per work group
constexpr int kWaves = 8;

struct MfmaArgs {
    const bf16_t *__restrict__ Q;
    const bf16_t *__restrict__ K;
    const bf16_t *__restrict__ Khat;
    const bf16_t *__restrict__ Vt;      // per unit: V in matrix-core operand order, D * n_pad elements
    bf16_t *__restrict__ O;
    int Hq, Hkv, n, n_pad, W, sliding;
    int ld, ld_pad;                     // rows of room per unit in K, Khat, V (>= n), and the padded stride of Vt that
                                        // goes with it (>= n_pad)
    int q_off, nq;                      // query rows are positions q_off .. q_off + nq - 1 of the n keys
    int GH, RT, tiles, hgroups;         // heads per group chunk, rows per tile, row tiles, head chunks per unit
    int xsplit;                         // > 0: XCD-aware order, every unit split this many ways (see the kernel)
    float scale_log2;
    // fused short-prompt launch only: what the stand-alone scan, compaction and V re-order kernels take
    const bf16_t *__restrict__ V;       // [unit][n][D] as the caller passed it
    uint32_t *__restrict__ mask_bits;   // out
    unsigned long long *__restrict__ nnz;   // out
    float theta;
};

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

template <int D>
__global__ __launch_bounds__(256) void transpose_v_kernel(const bf16_t *__restrict__ V, bf16_t *__restrict__ Vt,
                                                          int n, int ld, int ld_pad, int blk0) {
    __shared__ bf16_t tile[kTB][D + 2];
    constexpr int MT = D / 32;
    const int unit = blockIdx.y, blk = blk0 + blockIdx.x;
    transpose_v_block<D, 256>(V + (size_t)unit * ld * D,
                              (u32x4 *)(Vt + (size_t)unit * D * ld_pad) + (size_t)blk * (2 * MT * 64), blk * kTB, n, tile,
                              (int)threadIdx.x, [] { __syncthreads(); });
}

// What the stand-alone scan and V re-order launches do for a unit, done by one work group of the fused
// short-prompt kernel for the key rows 0 .. need - 1 that its own query rows see (512 threads; `lds` is scratch of
// fused_lds_bytes(D, need) bytes that nothing else uses yet).  The key rows are copied into LDS once; Eq. 2-3 run
// there row by row (wave ballot = mask word), leaving the reference keys and mask words beside them in LDS, from where
// they go out to the workspace and the caller's mask array.
// Every work group of a unit does this on its own and writes the same workspace arrays with the same values (only
// final values are ever stored, and only for rows and blocks all of whose inputs the work group holds): a work group
// reads only what it has itself written, whatever the others are doing.
// `writer` (one work group per unit, one that needs every row) also stores the unit's nnz.
__host__ __device__ constexpr size_t fused_lds_bytes(int d, int need) {
    return 64 + (size_t)2 * need * d * 2 + (size_t)need * (d / 32) * 4;
}

template <int D>
__device__ __forceinline__ void fused_prepare(const MfmaArgs &a, int unit, int need, bool writer, char *lds) {
    constexpr int CW = D / kWave;                               // waves that scan (64 channels each)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.n;
    const bf16_t *Kp = a.K + (size_t)unit * a.ld * D;
    bf16_t *Hp = const_cast<bf16_t *>(a.Khat) + (size_t)unit * a.ld * D;
    uint32_t *Mp = a.mask_bits + (size_t)unit * n * (D / 32);
    unsigned long long *cnt = (unsigned long long *)lds;        // [CW] surviving entries per scanning wave
    bf16_t *Kl = (bf16_t *)(lds + 64);                          // [need][D] keys
    bf16_t *Hl = Kl + (size_t)need * D;                         // [need][D] reference keys
    uint32_t *Ml = (uint32_t *)(Hl + (size_t)need * D);         // [need][D / 32] mask words
    // 1. the key rows into LDS
    {
        constexpr int kPer = kFusedMaxElems / 8 / 512;           // 16-byte pieces per thread at the largest prompt
        u32x4 piece[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {                         // every load issued before the first is parked
            const int idx = tid + i * 512;
            piece[i] = ((const u32x4 *)Kp)[min(idx, need * (D / 8) - 1)];
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int idx = tid + i * 512;
            if (idx < need * (D / 8)) ((u32x4 *)Kl)[idx] = piece[i];
        }
    }
    __syncthreads();
    // 2. Eq. 2-3 over the rows, in order, by CW waves (64 channels each)
    if (wave < CW) {
        unsigned long long c = 0;
        scan_rows<bf16_t, true>(Kl, Hl, Ml, D, wave * kWave + lane, lane, 0, need, true, (const bf16_t *)nullptr, 0.f,
                                a.theta, &c);
        if (lane == 0) cnt[wave] = c;
    }
    __syncthreads();
    // 3. reference keys and mask words out to the workspace / the caller's mask array; nnz
    for (int idx = tid; idx < need * (D / 8); idx += 512) ((u32x4 *)Hp)[idx] = ((const u32x4 *)Hl)[idx];
    for (int idx = tid; idx < need * (D / 32); idx += 512) Mp[idx] = Ml[idx];
    if (writer && tid == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < CW; ++w) t += cnt[w];
        a.nnz[unit] = t;
    }
    __syncthreads();
    // 4. V into matrix-core operand order, a block of 32 keys per wave at a time (the LDS copies above are done with)
    {
        typedef bf16_t (*tile_t)[D + 2];
        tile_t tile = (tile_t)(lds + 64 + (size_t)wave * kTB * (D + 2) * sizeof(bf16_t));
        const bf16_t *Vp = a.V + (size_t)unit * a.ld * D;
        u32x4 *Op = (u32x4 *)(const_cast<bf16_t *>(a.Vt) + (size_t)unit * D * a.ld_pad);
        for (int blk = wave; blk * kTB < need; blk += kWaves)
            transpose_v_block<D, kWave>(Vp, Op + (size_t)blk * (2 * (D / 32) * 64), blk * kTB, n, tile, lane, [] {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            });
    }
    __threadfence();
    __syncthreads();
}

// kAligned: the launcher has checked that every tile's rows share one window whose start is a multiple of the block
// size; the K_hat tile of the near blocks, its loads and its branches then do not exist in the instantiation.
// kFused: the work group first runs the delta scan and the V re-order for its unit itself (short prompts: one launch
// instead of four; see fused_prepare).
template <int D, bool kAligned, bool kFused = false>
__global__ __launch_bounds__(512) void prefill_mfma_kernel(MfmaArgs a) {
    // (aligned explicitly: the dynamic region starts where the static variables below end, and every tile in
    // it is accessed with 16-byte instructions)
    extern __shared__ __attribute__((aligned(256))) char lds_raw[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction; tell the compiler
    const int half = lane >> 5, li = lane & 31;

    // ---- which tile.  Work groups go to the 8 XCDs round-robin by index, and every XCD has its own L2; all
    //      tiles of a unit stream the same K, K_hat and V.  So the index is first turned into
    //      (XCD, slot on that XCD), and each XCD is given whole units - or, when the unit count does not
    //      divide by 8, units split `xsplit` ways by tile index modulo xsplit - one after the other: a unit's
    //      streams are then fetched into xsplit L2s instead of all 8.  Within a part, heavy (late) tiles first.
    int bid = blockIdx.x;
    const int per_unit = a.tiles * a.hgroups;
    if (a.xsplit > 0) {
        const int xcd = bid & 7, slot = bid >> 3;
        const int per_part = per_unit / a.xsplit;            // work groups of one part
        const int part = xcd + 8 * (slot / per_part);        // parts xcd, xcd + 8, ... belong to this XCD
        const int within = slot % per_part;
        bid = (part / a.xsplit) * per_unit + within * a.xsplit + part % a.xsplit;
    }
    const int unit = bid / per_unit;
    bid -= unit * per_unit;
    const int hchunk = bid % a.hgroups;
    const int tile = a.tiles - 1 - bid / a.hgroups;
    const int b = unit / a.Hkv, hk = unit % a.Hkv;
    const int g = a.Hq / a.Hkv;
    const int head0 = hk * g + hchunk * a.GH;
    const int n = a.n, W = a.W, RT = a.RT;
    const int i0 = a.q_off + tile * RT, i_last = min(i0 + RT - 1, n - 1);   // first and last query position

    const bf16_t *Kp = a.K + (size_t)unit * a.ld * D;
    const bf16_t *Hp = a.Khat + (size_t)unit * a.ld * D;
    const bf16_t *Vtp = a.Vt + (size_t)unit * D * a.ld_pad;

    // score row sr = hh * RT + r  ->  query row i0 + r of head head0 + hh
    auto q_row_ptr = [&](int sr) -> const bf16_t * {
        const int hh = sr / RT, r = sr - hh * RT;
        const int i = min(i0 + r, n - 1);
        return a.Q + (((size_t)b * a.Hq + head0 + hh) * a.nq + (i - a.q_off)) * D;
    };

    if constexpr (kFused) {
        fused_prepare<D>(a, unit, min(n, i_last + 1), tile == a.tiles - 1 && hchunk == 0, lds_raw);
    }

    // ---- this wave's score rows for softmax / PV: sr = 32 * wave + li (both lane halves)
    const int my_sr = 32 * wave + li;
    const int my_hh = my_sr / RT, my_r = my_sr - my_hh * RT;
    const int my_i = i0 + my_r;
    const bool my_valid = my_i < n;
    // first exact column of row r: start of its square, or of its band (monotone in r either way)
    auto win_start = [&](int r) { return a.sliding ? max(r - W + 1, 0) : (r / W) * W; };
    const int my_win = win_start(min(my_i, n - 1));
    const bf16_t *my_q = q_row_ptr(my_sr);

    constexpr int KS = D / 16;     // k-steps of Q K^T
    constexpr int MT = D / 32;     // channel tiles of the output

    f32x16 oacc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[mt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    const int win_first = win_start(i0);         // smallest window start of the tile's rows
    const int win_last = win_start(i_last);      // largest
    const bool aligned = kAligned || ((win_first % kTB == 0) && (win_first == win_last));
    const int nblocks = i_last / kTB + 1;

    // Online softmax + PV for one block; s[16] are this lane's raw scores (-inf where masked), sc the
    // positive factor that turns them into log2 units.  The running maximum is only raised when the
    // block maximum exceeds it by more than 2^8 in the exponent, so probabilities stay <= 256 and the
    // accumulator is rarely rescaled.
    auto softmax_pv = [&](float (&s)[16], float sc, const u32x4 (&vreg)[2 * MT]) {
        float bm = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) bm = fmaxf(bm, s[r]);
        bm = fmaxf(bm, __shfl_xor(bm, 32)) * sc;
        if (__any(bm > m_run + 8.f)) {
            const float m_new = fmaxf(m_run, bm);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[mt][r] *= alpha;
        }
        const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
            p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], sc, neg_m));   // bare v_exp_f32: tiny results may flush to 0
        // The row sum is taken over the probabilities as rounded to bf16, i.e. over the very weights that P V uses:
        // the output is then an exact weighted mean of the value rows, and the rounding of the weights cannot bias it
        // (summing the unrounded ones does, by up to 2^-9 relative when many weights are equal).
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        float psum = 0.f;
#pragma unroll
        for (int ka = 0; ka < 2; ++ka) {
            u32x4 pb;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                f32x2 pr;
                pr[0] = p[8 * ka + 2 * k];
                pr[1] = p[8 * ka + 2 * k + 1];
                const bf16x2 pk = __builtin_convertvector(pr, bf16x2);
                psum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, psum, false);
                pb[k] = __builtin_bit_cast(uint32_t, pk);
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vreg[ka * MT + mt]), as_bf16x8(pb),
                                                                  oacc[mt], 0, 0, 0);
        }
        l_run += psum;
    };

    // ---------------------------------------------------------------- key blocks
    // Exact scores K Q^T, or K_hat Q^T left of the window, on the matrix cores.  The K / K_hat / V tiles of a
    // block are fetched once per work group, one 16-byte piece per thread, a block ahead into registers,
    // then parked in LDS in operand order (lane-contiguous 16-byte slots, conflict free) where all 8 waves
    // read them.  Three LDS buffers rotate (tiles are requested two blocks ahead); one barrier per block.
    {
        u32x4 qreg[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = *(const u32x4 *)(my_q + ks * 16 + half * 8);
        constexpr int kTileBytes = D * 64;                       // 32 keys x D channels, bf16
        constexpr int kPieces = kTileBytes / 16;                 // 16-byte pieces per tile (256 or 512)
        char *tiles = lds_raw;                        // [3 buffers][K, K_hat, V]
        // Every thread loads a piece - at head_dim 64, where a tile has only 256, the upper half of the work group
        // loads the lower half's pieces again and does not store them: loads that sit under a condition make the
        // compiler wait for every load in flight before a piece is parked, the younger set's included.
        const bool has_piece = kPieces == 512 || tid < kPieces;
        const int ptid = tid & (kPieces - 1);
        // K piece of thread ptid: key row ptid % 32, 8-channel segment ptid / 32.  Its operand-order slot is then
        // ptid itself, so a wave's 64 LDS stores are contiguous (a row-major thread-to-piece map made 16 lanes
        // hit the same banks)
        const int pr = ptid & 31, pseg = ptid >> 5;
        const int kslot = ((pseg >> 1) * 64 + (pseg & 1) * 32 + pr) * 16;
        // operand X of a block: K_hat while every row has the block outside its window else K
        auto first_src = [&](int jb) -> const bf16_t * { return (jb + kTB <= win_first) ? Hp : Kp; };
        struct Pieces {
            u32x4 k, h, v;
        };
        auto load_tiles = [&](Pieces &pc, int blk) {
            const int jb = blk * kTB;
            const size_t roff = (size_t)min(jb + pr, n - 1) * D + pseg * 8;
            pc.k = *(const u32x4 *)(first_src(jb) + roff);
            if (!kAligned) pc.h = *(const u32x4 *)(Hp + roff);   // unconditional unless the tile cannot exist
            pc.v = *((const u32x4 *)Vtp + (size_t)blk * kPieces + ptid);
        };
        auto store_tiles = [&](const Pieces &pc, int buf) {
            char *base = tiles + buf * (3 * kTileBytes);
            if (has_piece) {
                *(u32x4 *)(base + kslot) = pc.k;
                if (!aligned) *(u32x4 *)(base + kTileBytes + kslot) = pc.h;
                *(u32x4 *)(base + 2 * kTileBytes + ptid * 16) = pc.v;
            }
        };
        // transposed score tile S^T[key][score row] = X[jb + key] . q, X tile in operand order at xt (a per-lane
        // address: tile base + 16 * lane, so that every read below is that address plus a constant)
        auto score_tile = [&](const char *xt) -> f32x16 {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const u32x4 xa = *(const u32x4 *)(xt + ks * 1024);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(xa), as_bf16x8(qreg[ks]), acc, 0, 0, 0);
            }
            return acc;
        };
        // raw score registers of a block: exact / K_hat scores picked per element, causal mask applied
        auto block_scores = [&](float (&s)[16], const char *base, int jb) {
            {
                const f32x16 sk = score_tile(base);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = sk[r];
            }
            if (!aligned && first_src(jb) == Kp && jb < win_last) {
                // some row has part of the block left of its window: exact score inside the row's own
                // window, K_hat score (telescoped Eq. 4) left of it
                const f32x16 sh = score_tile(base + kTileBytes);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = jb + 8 * (r >> 2) + 4 * half + (r & 3);
                    s[r] = (j >= my_win) ? s[r] : sh[r];
                }
            }
            if (jb + kTB > i0 + 1) {   // some entry is masked for some row of the tile
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = jb + 8 * (r >> 2) + 4 * half + (r & 3);
                    s[r] = (j <= my_i) ? s[r] : -INFINITY;
                }
            }
        };
        // Software pipeline over blocks: the score MFMAs of block b+1 are issued before the softmax of
        // block b, so matrix-core and vector-ALU work of one wave overlap.  Buffer b % 3 holds the tiles of
        // block b; its K tile is read one iteration before its V tile.
        // Two register sets of pieces alternate: a set is parked in LDS and at once re-used for the block two
        // further on, so no set is ever copied (a copy of registers that a load is still filling waits for it).
        // Loads and stores are issued every iteration, past the last block too (clamped to it: a dead buffer gets
        // a copy nobody reads), so that the number of loads in flight is the same on every path and the wait
        // before a set is parked lets the younger set's loads stay in flight.
        Pieces pa, pb;
        load_tiles(pa, 0);
        load_tiles(pb, min(1, nblocks - 1));
        lds_barrier();                                           // the fused preparation's LDS use is over
        store_tiles(pa, 0);
        load_tiles(pa, min(2, nblocks - 1));
        lds_barrier();
        float s_a[16], s_b[16];                                  // raw scores of the current / the next block, in turn
        const char *lane_tiles = tiles + lane * 16;              // per-lane view of the tile buffers
        block_scores(s_a, lane_tiles, 0);
        int buf = 0;
        // one block: `next` holds the pieces of block blk + 1, s_cur this block's scores, s_next receives the next one's
        auto do_block = [&](int blk, Pieces &next, float (&s_cur)[16], float (&s_next)[16]) {
            const char *base = lane_tiles + buf * (3 * kTileBytes);
            const int nbuf = buf == 2 ? 0 : buf + 1;
            store_tiles(next, nbuf);
            load_tiles(next, min(blk + 3, nblocks - 1));            // in flight for two iterations
            lds_barrier();                                       // LDS only: the tile loads stay in flight
            if (blk + 1 < nblocks) block_scores(s_next, lane_tiles + nbuf * (3 * kTileBytes), (blk + 1) * kTB);
            u32x4 vreg[2 * MT];
#pragma unroll
            for (int k = 0; k < 2 * MT; ++k) vreg[k] = *(const u32x4 *)(base + 2 * kTileBytes + k * 1024);
            softmax_pv(s_cur, a.scale_log2, vreg);
            buf = nbuf;
        };
        // everything requested so far has landed before the loop is entered: the wait at its head then only has to
        // cover what the previous trip left in flight (the compiler sizes it for the worse of both ways in)
        __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
        for (int blk = 0; blk < nblocks; blk += 2) {
            do_block(blk, pb, s_a, s_b);
            if (blk + 1 < nblocks) do_block(blk + 1, pa, s_b, s_a);
        }
    }

    // ---------------------------------------------------------------- epilogue
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (my_valid) {
        const float inv = 1.f / l_tot;
        bf16_t *orow = a.O + (((size_t)b * a.Hq + head0 + my_hh) * a.nq + (my_i - a.q_off)) * D;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                u32x2 w;
                w[0] = pack_bf16x2(oacc[mt][4 * q4 + 0] * inv, oacc[mt][4 * q4 + 1] * inv);
                w[1] = pack_bf16x2(oacc[mt][4 * q4 + 2] * inv, oacc[mt][4 * q4 + 3] * inv);
                *(u32x2 *)(orow + mt * 32 + 8 * q4 + 4 * half) = w;
            }
    }
}

// tiles of a launch: row tiles x head chunks x units; GH heads of RT rows make a tile's kRows score rows
static void tile_counts(const PrefillArgs &p, int &GH, int &RT, int &tiles, int &hgroups) {
    const int g = p.Hq / p.Hkv;
    GH = (g % 4 == 0) ? 4 : (g % 2 == 0) ? 2 : 1;
    RT = kRows / GH;
    tiles = (p.nq + RT - 1) / RT;
    hgroups = g / GH;
}

template <int D>
static void launch_d(const PrefillArgs &p, void *vt, int n_pad, hipStream_t s) {
    const int units = p.B * p.Hkv;
    const int ld = p.ld > 0 ? p.ld : p.n, ld_pad = p.ld > 0 ? prefill_mfma_n_pad(p.ld) : n_pad;
    if (!p.fused && p.vt_from < n_pad / kTB)
        hipLaunchKernelGGL((transpose_v_kernel<D>), dim3(n_pad / kTB - p.vt_from, units), dim3(256), 0, s,
                           (const bf16_t *)p.V, (bf16_t *)vt, p.n, ld, ld_pad, p.vt_from);
    MfmaArgs a;
    a.ld = ld;
    a.ld_pad = ld_pad;
    a.V = (const bf16_t *)p.V;
    a.mask_bits = p.mask_bits;
    a.nnz = (unsigned long long *)p.nnz;
    a.theta = p.theta;
    a.Q = (const bf16_t *)p.Q;
    a.K = (const bf16_t *)p.K;
    a.Khat = (const bf16_t *)p.Khat;
    a.Vt = (const bf16_t *)vt;
    a.O = (bf16_t *)p.O;
    a.Hq = p.Hq;
    a.Hkv = p.Hkv;
    a.n = p.n;
    a.n_pad = n_pad;
    a.W = p.W;
    a.sliding = p.sliding;
    tile_counts(p, a.GH, a.RT, a.tiles, a.hgroups);
    a.q_off = p.q_off;
    a.nq = p.nq;
    a.scale_log2 = p.scale_log2;
    const size_t lds_near = (size_t)9 * D * 64;
    // fused_prepare's scratch: LDS copies of up to kFusedMaxElems key elements, or the per-wave V tiles
    const size_t lds_prep = fused_lds_bytes(D, kFusedMaxElems / D) > (size_t)64 + kWaves * kTB * (D + 2) * 2
                                ? fused_lds_bytes(D, kFusedMaxElems / D) : (size_t)64 + kWaves * kTB * (D + 2) * 2;
    const size_t lds_fused = lds_near > lds_prep ? lds_near : lds_prep;
    static std::atomic<uint64_t> lds_set[3];                     // per instantiation of launch_d, one bit per device
    ensure_dynamic_lds((const void *)prefill_mfma_kernel<D, false>, (int)lds_near, lds_set[0]);
    ensure_dynamic_lds((const void *)prefill_mfma_kernel<D, true>, (int)lds_near, lds_set[1]);
    ensure_dynamic_lds((const void *)prefill_mfma_kernel<D, false, true>, (int)lds_fused, lds_set[2]);
    const size_t blocks = (size_t)units * a.tiles * a.hgroups;
    // XCD-aware order needs units * xsplit parts to deal out evenly over 8 XCDs and a unit to split evenly
    a.xsplit = 0;
    for (int sp = 1; sp <= 8; sp *= 2)
        if ((units * sp) % 8 == 0) {
            if ((a.tiles * a.hgroups) % sp == 0 && sp < 8) a.xsplit = sp;
            break;
        }
    // every tile's rows (RT consecutive positions from q_off on) lie in one window square whose start is a multiple
    // of the block size
    const bool all_aligned = !p.sliding && p.W % kTB == 0 && p.W % a.RT == 0 && p.q_off % a.RT == 0;
    const dim3 grid((unsigned)blocks), block(512);
    if (p.fused)
        hipLaunchKernelGGL((prefill_mfma_kernel<D, false, true>), grid, block, lds_fused, s, a);
    else if (all_aligned)
        hipLaunchKernelGGL((prefill_mfma_kernel<D, true>), grid, block, lds_near, s, a);
    else
        hipLaunchKernelGGL((prefill_mfma_kernel<D, false>), grid, block, lds_near, s, a);
}

int prefill_mfma_n_pad(int n) { return (n + 63) / 64 * 64; }

bool prefill_mfma_supported(const PrefillArgs &p) {
    return p.dtype == 1 && (p.d == 64 || p.d == 128) &&
           (size_t)p.B * p.Hkv * ((p.n + 63) / 64) * (p.Hq / p.Hkv) < ((size_t)1 << 31);
}

void launch_prefill_mfma(const PrefillArgs &p, void *vt, hipStream_t s) {
    const int n_pad = prefill_mfma_n_pad(p.n);
    if (p.d == 64)
        launch_d<64>(p, vt, n_pad, s);
    else
        launch_d<128>(p, vt, n_pad, s);
}

}  // namespace da
