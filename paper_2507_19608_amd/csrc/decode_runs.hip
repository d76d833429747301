// Decode stage for bf16 caches in the column-run layout (Sec. III-B decode stage, Sec. III-C): head_dim 64
// or 128, decode window of at least one chunk (or of the whole cache).  The compact delta cache keeps, per chunk of kChunk rows
// and per channel, the run of surviving key values; a chunk is sealed into that form once, when its last
// row has arrived, while its rows are still inside the decode window.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "cache.hpp"
#include "cache_fill.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

using namespace da;

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;

// Seal from the raw-key ring: runs right after the step that appended the chunk's last row.
template <int D>
__global__ __launch_bounds__(256) void seal_from_ring_kernel(da_cache c, int chunk) {
    constexpr int WPR = D / 32, P = D / 8;                       // mask words, 16-byte pieces per row
    __shared__ __attribute__((aligned(16))) bf16_t keys[kChunk * D];
    __shared__ __attribute__((aligned(16))) bf16_t runs[(D / 64) * kHalfRoom];
    __shared__ uint32_t mask[kChunk * WPR], len[2];
    const int unit = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, r0 = chunk * kChunk;
    const u32x4 *ring = (const u32x4 *)c.ring + (size_t)unit * c.Wd * P;
    u32x4 kk[kChunk * P / 256];
#pragma unroll
    for (int i = 0; i < kChunk * P / 256; ++i) {
        const int idx = tid + i * 256;
        kk[i] = ring[(size_t)((r0 + idx / P) % c.Wd) * P + idx % P];
    }
    const uint32_t mw = tid < kChunk * WPR ? c.mask[((size_t)unit * c.max_seq + r0) * WPR + tid] : 0u;
#pragma unroll
    for (int i = 0; i < kChunk * P / 256; ++i) ((u32x4 *)keys)[tid + i * 256] = kk[i];
    if (tid < kChunk * WPR) mask[tid] = mw;
    __syncthreads();
    if (wave < D / 64) {
        const bf16_t held = chunk > 0 ? ((const bf16_t *)c.ck)[(size_t)unit * D + tid] : (bf16_t)0;
        const uint32_t n = build_runs(keys + 64 * wave, D, mask + 2 * wave, WPR, held, runs + wave * kHalfRoom);
        if ((tid & 63) == 0) len[wave] = n;
    }
    __syncthreads();
    store_runs<D, 256>(c, unit, chunk, runs, len, tid);
}

// Hand-off of prefilled rows to the cache where no attention launch takes it along (cache_fill.hpp).
template <int D>
__global__ __launch_bounds__(256) void cache_fill_runs_kernel(CacheFill f) {
    __shared__ __attribute__((aligned(16))) char lds[kFillLds<D>];
    fill_chunk<D, 256>(f, (int)blockIdx.x, lds, (int)threadIdx.x);
}

// The inverse of the hand-off, for a prefill that continues a cached sequence: rows 0 .. t0 - 1 of the cache
// are written out as plain arrays [units][ld][...] (ld >= t0 rows of room per unit): reference keys (from
// the sealed runs, or for the unsealed last chunk from the ring), keys (raw for the rows the ring still
// holds, the reference key otherwise), values, mask rows.  One wave per (chunk, unit), lane = channel.
__global__ __launch_bounds__(64) void expand_cache_kernel(da_cache c, int t0, int ld, bf16_t *__restrict__ Kfull,
                                                          bf16_t *__restrict__ Hfull, bf16_t *__restrict__ Vfull,
                                                          uint32_t *__restrict__ Mfull) {
    const int chunk = blockIdx.x, unit = blockIdx.y, lane = threadIdx.x;
    const int d = c.d, wpr = d >> 5;
    const int r0 = chunk * kChunk, rows = min(kChunk, t0 - r0);
    const bool sealed = rows == kChunk;
    const uint32_t *Mp = c.mask + ((size_t)unit * c.max_seq + r0) * wpr;
    for (int i = lane; i < rows * wpr; i += kWave) Mfull[((size_t)unit * ld + r0) * wpr + i] = Mp[i];
    const bf16_t *room = run_room(c, unit, chunk);
    const bf16_t *ring = (const bf16_t *)c.ring + (size_t)unit * c.Wd * d;
    uint32_t base = 0;
    for (int c0 = 0; c0 < d; c0 += kWave) {
        const int ch = c0 + lane;
        // rows in batches of 16 (one group of the V layout): all loads of a batch are issued before anything is
        // stored, so that their latency is paid once per batch, not once per row
        uint64_t cm = 0;
        for (int rb = 0; rb < rows; rb += 16) {
            uint32_t w[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) w[u] = Mp[(size_t)min(rb + u, rows - 1) * wpr + (ch >> 5)];   // clamped: branch-free
#pragma unroll
            for (int u = 0; u < 16; ++u) cm |= (uint64_t)(rb + u < rows ? (w[u] >> (ch & 31)) & 1u : 0u) << (rb + u);
        }
        uint32_t total = 0, p = 0;
        bf16_t held = 0;
        if (sealed) {
            p = base + kHead + wave_exclusive_scan((uint32_t)__popcll(cm) + 1u, &total);
            held = room[p];
        } else if (chunk > 0) {
            held = ((const bf16_t *)c.ck)[(size_t)unit * d + ch];
        }
        for (int rb = 0; rb < rows; rb += 16) {
            bf16_t kraw[16], sv[16];
            // the 16 values of this channel and row group are contiguous in the V cache, in slot order
            const u32x4 *vp = (const u32x4 *)((const bf16_t *)c.V + (((size_t)unit * (c.vrows >> 4) + ((r0 + rb) >> 4)) * d + ch) * 16);
            const u32x4 v0 = vp[0], v1 = vp[1];
            const uint32_t bits = (uint32_t)(cm >> rb) & 0xffffu;      // the batch's mask bits of this channel
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int r = rb + u, row = r0 + r;
                // every load is in bounds whatever the row (ring slot of any position; p stays inside the room), so
                // none of them is conditional and all of a batch are in flight together
                kraw[u] = ring[(size_t)(row % c.Wd) * d + ch];
                p += sealed ? (bits >> u) & 1u : 0u;                        // p: position of the newest survivor
                sv[u] = room[p];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int r = rb + u, row = r0 + r;
                const bool raw_here = row >= t0 - c.Wd;                     // always true for an unsealed chunk
                if ((bits >> u) & 1u) held = sealed ? sv[u] : kraw[u];
                const int slot = 8 * ((u >> 2) & 1) + 4 * (u >> 3) + (u & 3);
                const uint32_t vw = slot < 8 ? v0[slot >> 1] : v1[(slot - 8) >> 1];
                const size_t o = ((size_t)unit * ld + row) * d + ch;
                if (r < rows) {
                    Hfull[o] = held;
                    Kfull[o] = raw_here ? kraw[u] : held;
                    Vfull[o] = (bf16_t)((slot & 1) ? vw >> 16 : vw & 0xffffu);
                }
            }
        }
        base = kHalfRoom;
    }
}

// D1: delta of the new key against the carried reference key (Eq. 2-3), by one wave per unit.  The
// surviving values themselves are already in the raw-key ring; the run is built when the chunk is sealed.
// What it reads is asked for when the step begins and stored from at its end: nothing of the step waits for it.
template <int D>
struct NewRow {
    bf16_t k[D / kWave], h[D / kWave], v[D / kWave];
    uint64_t nnz;
    __device__ __forceinline__ void load(const da_cache &c, int unit, int lane, const bf16_t *__restrict__ k_new,
                                         const bf16_t *__restrict__ v_new) {
#pragma unroll
        for (int i = 0; i < D / kWave; ++i) {
            const size_t at = (size_t)unit * D + kWave * i + lane;
            k[i] = k_new[at];
            h[i] = ((const bf16_t *)c.khat)[at];
            v[i] = v_new[at];
        }
        nnz = c.nnz[unit];
    }
    __device__ __forceinline__ void append(const da_cache &c, int unit, int lane, uint32_t *__restrict__ mask_row, int t, int slot) const {
        uint32_t fired = 0;
#pragma unroll
        for (int i = 0; i < D / kWave; ++i) {
            const int ch = kWave * i + lane;
            const bool fire = t == 0 || fabsf(bf16_to_f32(k[i]) - bf16_to_f32(h[i])) > c.theta;   // (t == 0: basis row)
            if (t > 0 && t % kChunk == 0) ((bf16_t *)c.ck)[(size_t)unit * D + ch] = h[i];
            if (fire) ((bf16_t *)c.khat)[(size_t)unit * D + ch] = k[i];
            ((bf16_t *)c.ring)[((size_t)unit * c.Wd + slot) * D + ch] = k[i];
            ((bf16_t *)c.V)[v16_index(unit, c.vrows, D, t, ch)] = v[i];
            const uint64_t b = __ballot(fire);
            if ((lane & 31) == 0) {
                const uint32_t w = (uint32_t)(b >> (lane & 32));
                c.mask[((size_t)unit * c.max_seq + t) * (D / 32) + (ch >> 5)] = w;
                if (mask_row) mask_row[(size_t)unit * (D / 32) + (ch >> 5)] = w;
            }
            fired += __popcll(b);
        }
        if (lane == 0) c.nnz[unit] = (t == 0 ? 0ull : nnz) + fired;
    }
};

// One decode step, one launch: gridDim.x work groups per unit of NW walkers each; a walker is one wave at head_dim 64, two
// waves at head_dim 128 that each take 64 of the channels (all query heads of the unit's group either way).  Walker w of all
// the unit's walkers takes chunks w, w + walkers, ... with flash-style running (max, sum, output) in registers, and asks for
// the next chunk's mask rows and runs while it works on the current one; a launch is sized so that all of its waves are
// resident at once.
// Per chunk:
//   1. history chunks (rows left of the decode window): head and runs of the wave's 64 channels are copied to LDS; the
//      reference value k_hat(j)[c] (Eq. 3) is element {start of c's run} + #{marked rows <= j of channel c} - by telescoping
//      Eq. 4 the history score of row j is q . k_hat(j).  The counts come from the matrix cores: column masks as bytes
//      (64 channels x 64 rows) times a triangle of twos, plus the starts, is the table of byte addresses, exact in int32,
//      and comes out in the layout that the next product takes its keys in: lane l holds row l % 32 of a half chunk,
//      channels 8 q + 4 (l / 32)..+3.  That leaves one LDS read per element.  (Counting on the vector ALU - ballot, two
//      mbcnt, two adds per channel of 64 rows - made 702 vector instructions a chunk of the 384 that it takes now.)
//      Window rows are 64-bit loads from the raw-key ring, the newest from k_new, asked for before the history rows of a chunk
//      that has both are worked on;
//   2. two neighbouring channels to a register: the 32x32x16 operand, with the queries fetched in the same channel order;
//   3. scores S[row][head] on the matrix cores (heads padded to 32 columns); at head_dim 128 the two waves
//      exchange their halves of the contraction through LDS and both hold the full scores (they wait for each other alone, by a
//      word of LDS each: barriers made all walkers of a work group wait for the slowest copy in every turn); softmax update in
//      the accumulator registers (lane = head, 32 rows per lane, the other 32 in lane + 32);
//   4. the accumulator registers, rounded to bf16, are the B operand of O^T += V^T P^T as they stand, because
//      the V cache stores each group of 16 rows in exactly that order; O^T (the wave's 64 channels) keeps
//      lane = head, so the running rescale needs no cross-lane traffic.
// The walkers of a work group merge their (o, m, l) in LDS.  A unit's only work group writes the normalised output; of
// several, each leaves its partial row in scratch, and the one that finds the others' there merges and writes (with a second
// launch for it a step took 14.1 instead of 12.3 us at 20 units of 2048 rows of 128, and its own time on the host).  On this chip every
// XCD has its own L2, and fences that write it back or drop it cost more than the second launch did; so the partial rows,
// and nothing else, are stored past it (relaxed device-scope stores), waited for, counted with a device-scope add, and read
// past it.
// What bounds a step of few chunks is the chain launch - counts and runs - keys - scores - merge - meeting; 8 units of 512 rows of 64, before what
// follows: 1.2 us until all is asked for, 0.7 until it is there, 0.9 keys, 0.5 softmax, 0.4 P V, 1.2 merge, 2.2 meeting.  Requests in one go and
// before anything else, no division and no constant worked out in their way or after their wait, the append at the end, work groups
// of 4 walkers: 7.95 -> 6.65 us a step together; 8 units of 200 rows 6.5 -> 5.6; 20 of 6000 rows of 128 17.1 -> 15.5, 40 of 3000 17.4 -> 16.2; 256 of 2048 rows of
// 64, which the memory bounds, 21.6 -> 20.7.  (V a chunk ahead took longer in every one of them; one copy of a turn's code
// instead of two changed nothing.)
template <int D, int NW>
__global__ __launch_bounds__(64 * NW * (D / 64), 2) void decode_step_runs_kernel(da_cache c, const bf16_t *__restrict__ q_new,
                                                                              const bf16_t *__restrict__ k_new,
                                                                              const bf16_t *__restrict__ v_new,
                                                                              bf16_t *__restrict__ o_out,
                                                                              uint32_t *__restrict__ mask_row, int t, int g, int nparts,
                                                                              int slot, float scale_log2) {
    constexpr int H = D / 64;                                // waves that share a chunk, 64 channels each
    constexpr int KS = 4, CT = 2;                            // per wave: contraction steps, output tiles
    constexpr int kPieces = (kHalfRoom + 511) / 512;         // 1 KiB copies (16 bytes per lane) that cover 64 channels
    // two staging areas for the runs of a chunk, used in turn: separate arrays, so that reads of one are known
    // not to touch the other while its copy is still in flight
    __shared__ __attribute__((aligned(16))) bf16_t stage_a_all[NW * H][kPieces * 512];
    __shared__ __attribute__((aligned(16))) bf16_t stage_b_all[NW * H][kPieces * 512];
    __shared__ float ml_all[NW][32][2];                      // [walker][head] maximum, sum
    __shared__ int done_by[NW * H];
    __shared__ uint32_t before;                              // work groups of the unit that were done before this one
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = wv / H, half = wv % H, coff = 64 * half;   // part inside the work group; channel half
    bf16_t *stage_a = stage_a_all[wv], *stage_b = stage_b_all[wv];
    const int unit = blockIdx.y, lane = threadIdx.x & 63;
    // (all arguments that the first requests need are read together: one after the other, each is a wait before them)
    asm volatile("" ::"s"(q_new), "s"(k_new), "s"(v_new), "s"(c.khat), "s"(c.nnz), "s"(c.surv), "s"(c.ccnt), "s"(c.max_chunks), "s"(c.Wd), "s"(t), "s"(g),
                 "s"(nparts));
    const int nchunks = t / kChunk + 1;
    // (taking every walkers-th chunk spreads an uneven count, and the cheaper window chunks at the end, evenly)
    const int c_step = NW * nparts, c_begin = (int)blockIdx.x * NW + wave, c_end = nchunks;
    const int first_head = unit * g;                         // of the batch's; g = Hq / Hkv <= 32 in this layout; slot = t % Wd
    const int n32 = lane & 31, kap = lane >> 5;
    const int win_begin = t + 1 - c.Wd;
    // rows of chunk ch left of the decode window (> 0 only for sealed chunks, because Wd >= kChunk)
    auto hist_of = [&](int ch) { return min(max(win_begin - ch * kChunk, 0), min(kChunk, t + 1 - ch * kChunk)); };

    // History chunk ch: the runs of this wave's channels go straight from global memory to the LDS staging area
    // (128-bit LDS-direct loads: lane i of a copy lands at base + 16 i); its mask rows, lane = row.
    // cnt: the chunk's element counts (channels 0..63, channels 64.. << 16); pieces `from` .. of the copy.
    const bf16_t *const rooms = (const bf16_t *)c.surv + (size_t)unit * c.max_chunks * run_room_stride(D);
    const uint32_t *const counts = c.ccnt + (size_t)unit * c.max_chunks;
    auto copy_runs = [&](int ch, uint32_t cnt, bf16_t *sv, int from) {
        const uint32_t first = half * kHalfRoom, len = half ? cnt >> 16 : cnt & 0xffffu;   // this wave's runs
        const bf16_t *runs = rooms + (size_t)ch * run_room_stride(D) + first;
#pragma unroll
        for (int p = 0; p < kPieces; ++p)
            if (p >= from && (uint32_t)p * 512u < len && first + p * 512 + lane * 8 + 8 <= (uint32_t)run_room_stride(D))
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(runs + p * 512 + lane * 8),
                                                 (__attribute__((address_space(3))) void *)(sv + p * 512), 16, 0, 0);
    };
    // Everything a walker begins with is asked for before anything is waited for.  The first chunk's copy does not wait for its element
    // counts: the pieces that a chunk with two fifths of its entries fills are copied anyway, the rest when the counts are there.
    constexpr int kSure = 4;
    const bool begins_with_runs = c_begin < c_end && hist_of(c_begin) > 0;
    uint32_t first_count = 0, tot_v = 0;                     // tot_v: element counts of the chunk after the next one's copy
    if (begins_with_runs) {
        int none = 0;                                        // (as a vector load: a scalar one would be waited for with the next arguments)
        asm("" : "+v"(none));
        first_count = counts[c_begin + none];
        copy_runs(c_begin, kSure * 512u | (kSure * 512u << 16), stage_a, 0);
    }
    if (c_begin + c_step < c_end && hist_of(c_begin + c_step) > 0)
        tot_v = counts[c_begin + c_step];
    const bool appends = half == 0 && (nchunks - 1) % c_step == c_begin;   // this wave owns row t
    NewRow<D> row_t;
    if (appends) row_t.load(c, unit, lane, k_new, v_new);
    // q operands (B operand of the score contraction): lane l = head l % 32, channels coff + 16 s + 4 (l / 32)..+3 and 8 more
    // (columns past the last head repeat it: their results go nowhere)
    u32x4 qop[KS];
    {
        const bf16_t *qrow = q_new + (size_t)(first_head + min(n32, g - 1)) * D + coff + 4 * kap;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const u32x2 q0 = *(const u32x2 *)(qrow + 16 * s), q1 = *(const u32x2 *)(qrow + 16 * s + 8);
            qop[s] = u32x4{q0[0], q0[1], q1[0], q1[1]};
        }
    }
    // the triangle of twos (B operand, int8): lane l = row l % 32 of a half chunk, byte i of register k = row 16 (l / 32) + 4 k + i
    i32x4 tri;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) w |= (16 * kap + 4 * k + i <= n32 ? 2u : 0u) << (8 * i);
        tri[k] = (int)w;
    }
    f32x16 o[CT];                                            // O^T: lane = head, register r of tile ct =
#pragma unroll                                               // channel coff + 32 ct + 8 (r / 4) + 4 (l / 32) + r % 4
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;
    // (worked out here, while the first loads are on their way: the compiler would do it when they have landed)
    asm volatile("" : "+v"(tri), "+v"(o[0]), "+v"(o[1]));
    if (begins_with_runs) copy_runs(c_begin, __builtin_amdgcn_readfirstlane(first_count), stage_a, kSure);

    float m_run = -INFINITY, l_run = 0.f;                    // l_run: this lane half's share of the sum

    // The two waves of a walker at head_dim 128 wait for each other, and for nobody else: what each has done, in steps of two a turn.
    // (They are of one work group, so both are there, and take the same chunks; LDS accesses of a wave are carried out in order.  In asm:
    // as ordinary accesses they would wait for the copies into LDS that are on their way.)
    int turn = 0;
    const uint32_t done_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int *)done_by;
    auto tell = [&](int done) __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\tds_write_b32 %0, %1" ::"v"(done_at + 4 * wv), "v"(done) : "memory");
    };
    auto await = [&](int done) __attribute__((always_inline)) {
        while (true) {
            int by;
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(by) : "v"(done_at + 4 * (wv ^ (H - 1))) : "memory");
            if (__builtin_amdgcn_readfirstlane(by) >= done) break;
            __builtin_amdgcn_s_sleep(1);
        }
    };
    if (H == 2) {
        tell(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    }

    auto do_chunk = [&](int chunk, bf16_t *sv, bf16_t *sv_next, const bf16_t *sv_partner) __attribute__((always_inline)) {
        const bool newest = chunk == nchunks - 1;            // this wave owns row t
        const int r0 = chunk * kChunk;
        const int nrows = min(kChunk, t + 1 - r0);
        const int hist_rows = hist_of(chunk);
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this chunk's runs have landed in LDS
        // the next chunk's runs, and the element count of the one after it, fly in meanwhile
        if (chunk + c_step < c_end) {
            if (H == 2) await(2 * turn);                     // (the partner is done with the scores that lie where they go)
            copy_runs(chunk + c_step, __builtin_amdgcn_readfirstlane(tot_v), sv_next, 0);
            tot_v = 0;
            if (chunk + 2 * c_step < c_end && hist_of(chunk + 2 * c_step) > 0)
                tot_v = counts[chunk + 2 * c_step];
        }
        // V operands of the chunk (needed last, requested first): lane l = channel coff + 32 ct + l % 32, rows of
        // lane half l / 32 of each 16-row group; the newest row is patched in from v_new
        u32x4 vop[CT][2][2];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    const int row16 = r0 + 32 * T + 16 * s2, ch = coff + 32 * ct + n32;
                    vop[ct][T][s2] = *(const u32x4 *)((const bf16_t *)c.V +
                                                      (((size_t)unit * (c.vrows >> 4) + (row16 >> 4)) * D + ch) * 16 + 8 * kap);
                }
        // 1., 2. the keys as operands: kop[T][s] = row 32 T + l % 32, channels coff + 16 s + 4 (l / 32)..+3 and 8 more
        u32x4 kop[2][KS], raw[2][KS];
        uint32_t v_last[CT];
        if (hist_rows < kChunk) {                            // window rows, asked for before the history rows are worked on
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                const int row = r0 + 32 * T + n32;
#pragma unroll
                for (int s = 0; s < KS; ++s) raw[T][s] = u32x4{0u, 0u, 0u, 0u};
                if (32 * T + n32 >= hist_rows && row <= t) {
                    const int back = slot - (t - row);           // (of the last Wd rows: one turn of the ring at most)
                    const bf16_t *src = (row == t ? k_new + (size_t)unit * D
                                                  : (const bf16_t *)c.ring + ((size_t)unit * c.Wd + (back < 0 ? back + c.Wd : back)) * D) + coff + 4 * kap;
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        const u32x2 x0 = *(const u32x2 *)(src + 16 * s), x1 = *(const u32x2 *)(src + 16 * s + 8);
                        raw[T][s] = u32x4{x0[0], x0[1], x1[0], x1[1]};
                    }
                }
            }
            if (newest)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) v_last[ct] = v_new[(size_t)unit * D + coff + 32 * ct + n32];
        }
        if (hist_rows > 0) {
            const __attribute__((address_space(3))) char *room = (const __attribute__((address_space(3))) char *)sv;
            const int lds_base = (int)(uintptr_t)room;
            // starts of the runs, in the layout of the product: register 4 q + e = channel 8 q + 4 (l / 32) + e; column masks
            i32x4 st[2][4];
            u32x2 cm[2];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                cm[ct] = *(const __attribute__((address_space(3))) u32x2 *)(room + (32 * ct + n32) * 8);
#pragma unroll
                for (int qd = 0; qd < 4; ++qd)
                    st[ct][qd] = *(const __attribute__((address_space(3))) i32x4 *)(room + 512 + (32 * ct + 8 * qd + 4 * kap) * 4);
            }
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                i32x16 start;                                // as LDS addresses
#pragma unroll
                for (int r = 0; r < 16; ++r) start[r] = st[ct][r >> 2][r & 3] + lds_base;
                // column masks, a byte per row: lane l = channel l % 32, rows 32 u + 16 (l / 32) .. + 15
                i32x4 bytes[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t bits = cm[ct][u] >> (16 * kap);
#pragma unroll
                    for (int k = 0; k < 4; ++k)              // four bits to four bytes
                        bytes[u][k] = (int)(__umul24((bits >> (4 * k)) & 15u, 0x204081u) & 0x01010101u);
                }
                const i32x4 twos = {0x02020202, 0x02020202, 0x02020202, 0x02020202};
                i32x16 at[2];
                at[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bytes[0], tri, start, 0, 0, 0);
                at[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bytes[0], twos, start, 0, 0, 0);
                at[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bytes[1], tri, at[1], 0, 0, 0);
                // (the reads are written out: through a pointer made of an integer they could alias the copy in flight for the
                // next chunk, and the compiler would wait for that first; so the wait states between a matrix result and
                // its use as an address - 19 at most - are written out too)
                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(at[0]), "+v"(at[1]));
                uint32_t val_of[2][16];
#pragma unroll
                for (int T = 0; T < 2; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) asm volatile("ds_read_u16 %0, %1" : "=v"(val_of[T][r]) : "v"(at[T][r]));
#pragma unroll
                for (int T = 0; T < 2; ++T) {
                    uint32_t *val = val_of[T];
                    if (T == 0)
                        asm volatile("s_waitcnt lgkmcnt(15)"
                                     : "+v"(val[0]), "+v"(val[1]), "+v"(val[2]), "+v"(val[3]), "+v"(val[4]), "+v"(val[5]), "+v"(val[6]),
                                       "+v"(val[7]), "+v"(val[8]), "+v"(val[9]), "+v"(val[10]), "+v"(val[11]), "+v"(val[12]),
                                       "+v"(val[13]), "+v"(val[14]), "+v"(val[15]));
                    else
                        asm volatile("s_waitcnt lgkmcnt(0)"
                                     : "+v"(val[0]), "+v"(val[1]), "+v"(val[2]), "+v"(val[3]), "+v"(val[4]), "+v"(val[5]), "+v"(val[6]),
                                       "+v"(val[7]), "+v"(val[8]), "+v"(val[9]), "+v"(val[10]), "+v"(val[11]), "+v"(val[12]),
                                       "+v"(val[13]), "+v"(val[14]), "+v"(val[15]));
#pragma unroll
                    for (int r = 0; r < 16; r += 2)          // channel 32 ct + 8 (r / 4) + 4 (l / 32) + r % 4 and the next
                        kop[T][2 * ct + (r >> 3)][(r & 7) >> 1] = val[r] | (val[r + 1] << 16);
                }
            }
        }
        if (hist_rows < kChunk) {
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int k = 0; k < 4; ++k) kop[T][s][k] = 32 * T + n32 >= hist_rows ? raw[T][s][k] : kop[T][s][k];
            // the raw rows are awaited here, inside the branch only window chunks take: left to the compiler the
            // wait lands after the join and history chunks would drain their in-flight V and run copies there
            __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
        }
        // 3. scores: lane l holds head l % 32 at rows 32 T + 8 (r / 4) + 4 (l / 32) + r % 4
        f32x16 acc[2];
#pragma unroll
        for (int T = 0; T < 2; ++T) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[T][r] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s)
                acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[T][s]),
                                                                 __builtin_bit_cast(bf16x8, qop[s]), acc[T], 0, 0, 0);
        }
        if (H == 2) {
            // the other wave contracted the other 64 channels: the halves meet in the staging areas each wave has
            // just finished reading its own of (registers 4 q .. 4 q + 3 of lane l at four floats 64 q + l: conflict free), and are added in
            // the same order by both, so both hold the same scores
            f32x4 *mine = (f32x4 *)sv;
            const f32x4 *theirs = (const f32x4 *)sv_partner;
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    mine[(4 * T + q) * 64 + lane] = f32x4{acc[T][4 * q], acc[T][4 * q + 1], acc[T][4 * q + 2], acc[T][4 * q + 3]};
            tell(2 * turn + 1);
            await(2 * turn + 1);
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 x = theirs[(4 * T + q) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[T][4 * q + e] = half ? x[e] + acc[T][4 * q + e] : acc[T][4 * q + e] + x[e];
                }
            tell(2 * turn + 2);                              // (what was read of the partner's area has arrived)
            ++turn;
        }
        if (nrows < kChunk) {                                // only the newest chunk has rows that do not exist yet
            const int lim = nrows - 4 * kap;                     // compared with constants: nothing to keep in registers
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * T + 8 * (r >> 2) + (r & 3) >= lim) acc[T][r] = -INFINITY;
        }
        float mx = acc[0][0];
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[T][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));                  // row r0 of a chunk is always valid, so mx is finite
        const float m = fmaxf(m_run, mx * scale_log2);       // running maximum in log2 units (the scale is positive)
        if (__any(m > m_run)) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m);   // first chunk: exp2(-inf) = 0 on zeros
            l_run *= alpha;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) o[ct] *= alpha;
            m_run = m;
        }
        u32x4 pa[2][2];
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(acc[T][r], scale_log2, -m));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(acc[T][r + 1], scale_log2, -m));
                // the sum runs over the probabilities as rounded to bf16, the weights P V uses: their rounding
                // then cannot bias the weighted mean
                const bf16x2 pk = __builtin_convertvector(f32x2{p0, p1}, bf16x2);
                l_run = __builtin_amdgcn_fdot2_f32_bf16(pk, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run, false);
                pa[T][r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
            }
        if (newest) {
            // the position is made opaque here so that the select conditions are worked out inside this branch, once per step,
            // instead of being kept in registers across the whole chunk loop
            int tt = t;
            asm volatile("" : "+s"(tt));
            const int pt = tt & 15;
            const int kap_t = (pt >> 2) & 1, i_t = 4 * (pt >> 3) + (pt & 3);
            const int Tn = (tt >> 5) & 1, sn = (tt >> 4) & 1;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const uint32_t vn = v_last[ct];
#pragma unroll
                for (int TT = 0; TT < 2; ++TT)
#pragma unroll
                    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            const bool hit = TT == Tn && ss == sn && w == (i_t >> 1) && kap == kap_t;
                            const uint32_t old = vop[ct][TT][ss][w];
                            const uint32_t pat = (i_t & 1) ? ((old & 0xffffu) | (vn << 16)) : ((old & 0xffff0000u) | vn);
                            vop[ct][TT][ss][w] = hit ? pat : old;
                        }
            }
        }
        // 4. O^T += V^T P^T: channels x heads, contraction over the chunk's 64 rows in accumulator order
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
                    o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vop[ct][T][s2]),
                                                                    __builtin_bit_cast(bf16x8, pa[T][s2]), o[ct], 0, 0, 0);
    };
    const bf16_t *partner_a = stage_a_all[wv ^ (H - 1)], *partner_b = stage_b_all[wv ^ (H - 1)];
    auto take = [&](int chunk, bf16_t *sv, bf16_t *sv_next, const bf16_t *sv_partner) __attribute__((always_inline)) {
        if (chunk < c_end) do_chunk(chunk, sv, sv_next, sv_partner);
    };
    for (int first = (int)blockIdx.x * NW; first < c_end; first += 2 * c_step) {     // (walker 0's chunk of the turn)
        take(first + wave, stage_a, stage_b, partner_a);
        if (first + c_step < c_end) take(first + c_step + wave, stage_b, stage_a, partner_b);
    }
    // the new row goes into the cache (other waves of this launch never read what is written here)
    if (appends) row_t.append(c, unit, lane, mask_row, t, slot);
    const float l_all = l_run + __shfl_xor(l_run, 32);
    // the walkers' (o, m, l) meet in LDS (a walker without chunks contributes m = -inf, l = 0)
    if (H > 1) __syncthreads();                              // (the partner may still read this wave's staging area)
    float *obuf = (float *)stage_a;                          // [g][64] of this wave; its staging areas are idle now
    if (n32 < g) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                *(f32x4 *)(obuf + n32 * 64 + 32 * ct + 8 * rq + 4 * kap) =
                    f32x4{o[ct][4 * rq], o[ct][4 * rq + 1], o[ct][4 * rq + 2], o[ct][4 * rq + 3]};
        if (kap == 0 && half == 0) {
            ml_all[wave][n32][0] = m_run;
            ml_all[wave][n32][1] = l_all;
        }
    }
    __syncthreads();
    constexpr int kThreads = 64 * NW * H;
    float *part = c.part + (size_t)first_head * c.max_parts * part_stride(D);   // [head][max_parts][part_stride]
    // two channels of a head per thread at a time; a row's last pair is its maximum and sum
    auto put = [&](int h, int ch, float x, float y) {
        const uint64_t v = (uint64_t)__float_as_uint(x) | ((uint64_t)__float_as_uint(y) << 32);
        __hip_atomic_store((uint64_t *)(part + ((size_t)h * c.max_parts + blockIdx.x) * part_stride(D) + ch), v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    };
    auto get = [&](int h, int p, int ch) -> f32x2 {
        const uint64_t v = __hip_atomic_load((const uint64_t *)(part + ((size_t)h * c.max_parts + p) * part_stride(D) + ch),
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return f32x2{__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32))};
    };
    for (int e = threadIdx.x; e < g * (D / 2); e += kThreads) {
        const int h = e / (D / 2), ch = e % (D / 2) * 2;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, ml_all[w][h][0]);
        const float M0 = M == -INFINITY ? 0.f : M;           // (a work group without chunks)
        float L = 0.f, x = 0.f, y = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = __builtin_amdgcn_exp2f(ml_all[w][h][0] - M0);
            const f32x2 v = *(const f32x2 *)((const float *)stage_a_all[w * H + (ch >> 6)] + h * 64 + (ch & 63));
            L = fmaf(f, ml_all[w][h][1], L);
            x = fmaf(f, v[0], x);
            y = fmaf(f, v[1], y);
        }
        if (nparts == 1) {
            const float inv = 1.f / L;
            *(uint32_t *)(o_out + (size_t)(first_head + h) * D + ch) =
                (uint32_t)f32_to_bf16(x * inv) | ((uint32_t)f32_to_bf16(y * inv) << 16);
        } else {
            put(h, ch, x, y);
            if (ch == 0) put(h, D, M, L);
        }
    }
    if (nparts == 1) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's stores have reached memory
    __syncthreads();
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(c.arrived + unit, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (before != (uint32_t)nparts - 1u) return;
    if (threadIdx.x == 0) __hip_atomic_store(c.arrived + unit, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next step
    auto finish = [&](int h, int ch, float x, float y, float L) __attribute__((always_inline)) {
        const float inv = 1.f / L;
        *(uint32_t *)(o_out + (size_t)(first_head + h) * D + ch) = (uint32_t)f32_to_bf16(x * inv) | ((uint32_t)f32_to_bf16(y * inv) << 16);
    };
    // Few parts: every thread asks for their maxima and sums itself.
    auto merge_few = [&](auto batch) __attribute__((always_inline)) {
        constexpr int kB = batch;                            // partial rows fetched together
        for (int e = threadIdx.x; e < g * (D / 2); e += kThreads) {
            const int h = e / (D / 2), ch = e % (D / 2) * 2;
            float M = -INFINITY, L = 0.f, x = 0.f, y = 0.f;
            for (int p0 = 0; p0 < nparts; p0 += kB) {
                f32x2 v[kB], ml[kB];
#pragma unroll
                for (int k = 0; k < kB; ++k) {               // (past the end: the last one again, not used)
                    v[k] = get(h, min(p0 + k, nparts - 1), ch);
                    ml[k] = get(h, min(p0 + k, nparts - 1), D);
                }
                float mb = M;
#pragma unroll
                for (int k = 0; k < kB; ++k) mb = fmaxf(mb, ml[k][0]);   // (part 0 has rows: finite)
                const float f = __builtin_amdgcn_exp2f(M - mb);
                L *= f;
                x *= f;
                y *= f;
#pragma unroll
                for (int k = 0; k < kB; ++k) {
                    const float w = p0 + k < nparts ? __builtin_amdgcn_exp2f(ml[k][0] - mb) : 0.f;
                    L = fmaf(w, ml[k][1], L);
                    x = fmaf(w, v[k][0], x);
                    y = fmaf(w, v[k][1], y);
                }
                M = mb;
            }
            finish(h, ch, x, y, L);
        }
    };
    // More, at head_dim 128: a lane asks for the maximum and sum of one part of its head (a head is 64 lanes, a unit has at most 32 parts) and works out
    // its weight while the rows, up to 16, are on their way.  Every batch is a trip past the L2s: of 8 rows and 8 maxima / this, us a step: 5 units of
    // 8000 rows 11.6 / 11.3, of 1500 9.6 / 9.2, 10 of 1800 9.1 / 8.7, 20 of 6000 15.7 / 15.3
    // (20 of 2000, 8 parts, whose batch is as it was: 10.2 / 10.3).
    auto merge_many = [&]() __attribute__((always_inline)) {
        constexpr int kB = 16;                               // rows fetched together
        static_assert(kMaxParts <= 32 && D / 2 >= 32 && (D / 2) % 32 == 0, "a lane for each part");
        for (int e = threadIdx.x; e < g * (D / 2); e += kThreads) {
            const int h = e / (D / 2), ch = e % (D / 2) * 2, p = lane & 31;
            const f32x2 ml = get(h, min(p, nparts - 1), D);
            f32x2 v[kB];
#pragma unroll
            for (int k = 0; k < kB; ++k) v[k] = get(h, min(k, nparts - 1), ch);   // (past the end: the last one again, not used)
            float M = ml[0];                                 // (part 0 has rows: the maximum is finite)
#pragma unroll
            for (int s = 16; s > 0; s >>= 1) M = fmaxf(M, __shfl_xor(M, s));
            const float w = p < nparts ? __builtin_amdgcn_exp2f(ml[0] - M) : 0.f;
            float L = w * ml[1], x = 0.f, y = 0.f;
#pragma unroll
            for (int s = 16; s > 0; s >>= 1) L += __shfl_xor(L, s);
            for (int p0 = 0;;) {
#pragma unroll
                for (int k = 0; k < kB; ++k) {
                    const float wk = p0 + k < nparts ? __shfl(w, p0 + k, 32) : 0.f;
                    x = fmaf(wk, v[k][0], x);
                    y = fmaf(wk, v[k][1], y);
                }
                p0 += kB;
                if (p0 >= nparts) break;
#pragma unroll
                for (int k = 0; k < kB; ++k) v[k] = get(h, min(p0 + k, nparts - 1), ch);
            }
            finish(h, ch, x, y, L);
        }
    };
    // Batches of 8 / of 4 for up to 4 parts: 8 units of 1000 rows of 64 7.24 / 7.13 us a step, 5 of 300 rows of 128 8.2 / 8.0.  At head_dim 64 more than 8 parts
    // in one batch would gain (8 units of 8000 rows 9.05 / 8.85, 4 of 4000 7.9 / 7.65), but that code in the kernel costs the rest 1 % (8 of 2000 6.95 / 7.0).
    if (nparts <= 4) {
        merge_few(std::integral_constant<int, 4>{});
        return;
    }
    if constexpr (D == 128)
        if (nparts > 8) {
            merge_many();
            return;
        }
    merge_few(std::integral_constant<int, 8>{});
}

}  // namespace

namespace da {

CacheFill cache_fill(const da_cache *c, int t0, int n_k, int ld, const void *K, const void *V, const void *H, const uint32_t *Mnew, uint32_t *Mall,
                     const uint64_t *nnz_new, const NnzSum &sum) {
    CacheFill f = {(const bf16_t *)K, (const bf16_t *)V, (const bf16_t *)H, Mnew, Mall, nnz_new, sum, *c, ld, t0, n_k, 0, 0};
    f.units = c->B * c->Hkv;
    f.items = ((n_k + kChunk - 1) / kChunk - t0 / kChunk) * f.units;
    return f;
}

void launch_cache_fill(const CacheFill &f, hipStream_t s) {
    if (f.cache.d == 64)
        hipLaunchKernelGGL(cache_fill_runs_kernel<64>, dim3(f.items), dim3(256), 0, s, f);
    else
        hipLaunchKernelGGL(cache_fill_runs_kernel<128>, dim3(f.items), dim3(256), 0, s, f);
}

void expand_cache_runs(da_cache *c, int t0, int ld, void *Kfull, void *Hfull, void *Vfull, uint32_t *Mfull,
                       hipStream_t s) {
    if (t0 <= 0) return;
    hipLaunchKernelGGL(expand_cache_kernel, dim3((t0 + kChunk - 1) / kChunk, c->B * c->Hkv), dim3(64), 0, s, *c, t0,
                       ld, (bf16_t *)Kfull, (bf16_t *)Hfull, (bf16_t *)Vfull, Mfull);
}

void decode_step_runs(da_cache *c, const void *q, const void *k, const void *v, void *o, uint32_t *mask_row, int t,
                      float scale_log2, hipStream_t s) {
    const int units = c->B * c->Hkv, nchunks = t / kChunk + 1;
    if (c->cus < 1 &&
        (hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess || c->cus < 1))
        c->cus = 256;
    // Work groups of 8 waves - 8 walkers at head_dim 64, 4 at head_dim 128 -, one per compute unit by LDS and registers: as many
    // per unit as keep the whole launch resident, no more than the last one can merge in a few round trips, or just one where
    // that has as few turns (a turn saved is worth the meeting: 20 .. 80 units of 300 rows, head_dim 128, 9.9 .. 10.1 us in two
    // turns of one work group, 9.5 .. 9.9 in one of two; 16 units of 500 rows, head_dim 64, 7.4 and 7.7).
    // Smaller ones, us a step:
    //  - half the walkers, where all work groups still have a compute unit each and a unit no more than 16: a SIMD then has one wave to
    //    serve.  head_dim 64, 8 / 4 walkers: 8 units of 512 rows 7.7 / 7.1, of 2000 9.0 / 7.9, 16 of 1000 8.4 / 7.5, 60 of 876 9.9 / 8.5 (but 32 work
    //    groups a unit, 8 units of 8000 rows: 9.5 / 10.6); head_dim 128, 4 / 2 walkers: 20 units of 300 rows 9.5 / 8.8, of 500 9.8 / 8.9, 5 of 2000
    //    10.1 / 9.5.  Likewise where there are only so many chunks (head_dim 64, 4 of them: 6.0 / 5.8).
    //  - more units than compute units: two work groups of 4 walkers of head_dim 64 fit one.  300 units of 200 rows 10.2 / 7.3, of 800 18.9 / 15.3,
    //    512 of 2000 37.8 / 36.0.
    //    (256 units of 2048 rows, 8 / 4 walkers: 20.3 / 20.8, and 24.0 / 25.9 where other caches are stepped in between.)
    //  - head_dim 128, whole work groups of 4 deal out badly to a number of units that does not divide the compute units: 2 or 1 are
    //    taken where the launch then has fewer turns, and 2 also where it has as many, but four or more; not where one work group of 4 per unit
    //    uses three quarters of the compute units, or half of them for few turns (2048 rows, other caches in between, 192 units 41.9 -> 37.0,
    //    256 units 50.9 -> 46.8).  4 / 2 / 1: 2000 rows, 20 units 10.8 / 11.8 / 13.8, 60 units 15.2 / 16.0
    //    / 17.1, 96 units 20.1 / 20.0 / 18.9, 140 units 29.2 / 26.2 / 25.5, 192 units 30.2 / 32.0 / 30.7, 256 units 37.4 / 38.3 / 38.2; 300 rows, 160 units 10.4 / 11.5 / 11.9,
    //    192 units 10.3 / 12.0 / 12.6; 1000 rows, 160 units 19.2 / 18.9 / 19.2, 320 units 37.6 / 32.8 / 30.5, 512 units 42.6 / 38.0 / 40.1.
    const int H = c->d / 64, slots = c->plan_slots > 0 ? c->plan_slots : c->cus * 8, cus = std::max(1, slots / 8);
    struct Plan {
        int nw, most, turns, cost;                           // walkers per work group, work groups per unit, turns of each, in all
    };
    auto turns = [&](int nw, int parts) { return (nchunks + nw * parts - 1) / (nw * parts); };
    auto plan = [&](int nw) {
        const int resident = std::max(1, slots / (nw * H)), most = std::max(1, std::min(resident / units, kMaxParts));
        const int t_each = turns(nw, most);
        return Plan{nw, most, t_each, (int)std::min<int64_t>((int64_t)t_each * (((int64_t)units * most + resident - 1) / resident), 1 << 30)};
    };
    auto parts_of = [&](const Plan &p) { return (nchunks + p.nw * p.turns - 1) / (p.nw * p.turns); };
    Plan p = plan(8 / H);
    bool one_each = c->plan_merge == 1;                      // one work group per unit
    if (!one_each) {
        const bool free = c->plan_merge < 0;
        const Plan half = plan(4 / H);
        if (c->d == 64 && (nchunks <= 4 || (units > cus && half.cost <= p.cost))) {
            p = half;
        } else if (c->d == 128 && free && units <= cus && (4 * (int64_t)units >= 3 * (int64_t)cus || (2 * (int64_t)units > cus && turns(4, 1) <= 4))) {
            one_each = true;
        } else if (free && p.turns < turns(p.nw, 1) && half.turns == p.turns && parts_of(half) <= 16 && (int64_t)units * parts_of(half) <= cus) {
            p = half;
        } else if (c->d == 128) {
            const Plan one = plan(1);
            if (half.cost < p.cost || (half.cost == p.cost && half.cost >= 4)) p = half;
            if (one.cost < p.cost) p = one;
        }
    }
    int parts = 1;
    if (!one_each && (p.turns < turns(p.nw, 1) || c->plan_merge == 0)) parts = parts_of(p);
    const auto kernel = c->d == 64 ? (p.nw == 8 ? decode_step_runs_kernel<64, 8> : decode_step_runs_kernel<64, 4>)
                        : p.nw == 4 ? decode_step_runs_kernel<128, 4> : p.nw == 2 ? decode_step_runs_kernel<128, 2> : decode_step_runs_kernel<128, 1>;
    hipLaunchKernelGGL(kernel, dim3(parts, units), dim3(64 * p.nw * H), 0, s, *c, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,
                       (bf16_t *)o, mask_row, t, c->Hq / c->Hkv, parts, t % c->Wd, scale_log2);
}

void seal_chunk_runs(da_cache *c, int chunk, hipStream_t s) {
    const dim3 grid(c->B * c->Hkv);
    if (c->d == 64)
        hipLaunchKernelGGL(seal_from_ring_kernel<64>, grid, dim3(256), 0, s, *c, chunk);
    else
        hipLaunchKernelGGL(seal_from_ring_kernel<128>, grid, dim3(256), 0, s, *c, chunk);
}

}  // namespace da
