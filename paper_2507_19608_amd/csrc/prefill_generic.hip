// Hybrid-attention prefill (Sec. III-B prefill stage; Eq. 4; Eq. 1) in binary32 on the matrix cores
// (v_mfma_f32_16x16x4): fp32 inputs, and bf16 inputs of head dims that prefill_mfma.hip has no kernel for.  Any head_dim
// that is a multiple of 32 up to 256.
//
// Scores left of the window are Eq. 4's running sum in telescoped form, q . k_hat(j); a block of keys that straddles
// a window takes both products and a select per element.
//
// Work group = 16 consecutive query rows of one query head; its 8 waves take the blocks of 32 keys in turn, each
// with its own running (maximum, sum, output), and meet in LDS once at the end.  The calls this kernel sees are small
// (a numerics user's single head of a few hundred rows), so what bounds it is how many waves there are and how long the
// longest one walks: a wave per 64 rows that walked every key took 725 us on 256 rows of one head of 64 (4 waves on the
// chip, operands by scalar loads); rows by 16 and keys by 8 give 128 waves of one or two blocks each: 6.8 us, 12.6 for the whole
// call with a scan in front and 9.8 where it is part of the launch.
//
// kScans: the keys left of a work group's windows fit into its LDS, so it takes them in and makes them reference keys there for itself
// (Eq. 2-3), and no launch and no pass through memory comes in front; one more work group per unit writes the mask.  (A block's values
// and window keys asked for in front of the scan, when that took 2 us more: 11.6 / 11.6 us at 256 rows of 64, 13.4 / 15.0 at 128 of 128, which then spills.)
//
// Matrix-core layout (16x16x4, wave64): A lane l holds row l % 16, k = l / 16; B lane l column l % 16, same k; D lane l
// column l % 16, rows 4 (l / 16) + r.  Scores are taken transposed (keys x query rows): a lane owns one query row, and
// register r of a score tile is the B operand of a P V step whose k-th key is 4 k + r.  The contraction over channels runs
// in the order that lets every operand be a 16-byte load of a row (step e of group s: channel 16 s + 4 (l / 16) + e), and
// output tile e of a channel group covers the channels VW m + e, so that a lane loads and stores VW consecutive ones.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace da {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned short u16x4;
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kWavesG = 8;       // waves of a work group, one block of keys each in turn
constexpr int kKeys = 32;        // keys per block: two score tiles

template <typename T>
struct KArgs {
    const T *__restrict__ Q;
    const T *__restrict__ K;
    const T *__restrict__ V;
    const T *__restrict__ Khat;
    T *__restrict__ O;
    int Hq, Hkv, n, W, sliding;
    float scale_log2;
    NnzSum sum;
    uint32_t *__restrict__ mask_bits;            // from here on: kScans
    uint64_t *__restrict__ nnz;
    float theta;
};

__device__ __forceinline__ f32x4 load4(const float *p) { return *(const f32x4 *)p; }
__device__ __forceinline__ f32x4 load4(const bf16_t *p) {
    const u16x4 v = *(const u16x4 *)p;
    return f32x4{bf16_to_f32(v[0]), bf16_to_f32(v[1]), bf16_to_f32(v[2]), bf16_to_f32(v[3])};
}
__device__ __forceinline__ f32x2 load2(const float *p) { return *(const f32x2 *)p; }
__device__ __forceinline__ f32x2 load2(const bf16_t *p) {
    const u16x2 v = *(const u16x2 *)p;
    return f32x2{bf16_to_f32(v[0]), bf16_to_f32(v[1])};
}

// A scan of n rows: 2 * 64 * kWavesG / d runs of so many rows each (a multiple of a batch), and the rows of all of them, which end with the last row again
constexpr int kBatch = 8;
__host__ __device__ constexpr int run_rows(int n, int d) {
    const int runs = 2 * 64 * kWavesG / d;
    return ((n + runs - 1) / runs + kBatch - 1) / kBatch * kBatch;
}
__host__ __device__ constexpr int scan_room(int n, int d) { return (n + run_rows(n, d) - 1) / run_rows(n, d) * run_rows(n, d); }
// LDS of a work group that scans n rows, or fewer: these, four floats apart so that 16 rows' reads of one segment lie in different banks; what the runs end
// on; three words
constexpr size_t scan_lds(int n, int d) { return ((size_t)scan_room(n, d) * (d + 4) + 2 * 64 * kWavesG + 4) * sizeof(float); }

// The reference keys of a unit's rows 0 .. n - 1, in LDS [scan_room][D + 4].  A thread walks a run of rows in two neighbouring channels, from the guess "held
// = the row before" kWarm rows earlier; runs whose start is not what the run before has ended on walk again, in rounds, and one last walk puts reference
// keys in the place of keys (as scan_whole_kernel does).  Runs are whole batches, so that a row costs its read and the three operations of each channel: with the last
// run's end looked for in every row, 1 head of 64, 256 rows took 11.6 us a call, now 9.8.
template <int D>
__device__ __forceinline__ void scan_rows(const float *__restrict__ K, int n, float theta, float *rows) {
    constexpr int S = D + 4, PR = D / 2, kRuns = 64 * kWavesG / PR, kWarm = 48, N = kBatch;
    const int L = run_rows(n, D), room = scan_room(n, D);
    float2 *const E = (float2 *)(rows + (size_t)room * S);
    int *const flags = (int *)(E + 64 * kWavesG);                // [2] some run was wrong in an even, odd round
    const int tid = threadIdx.x;
    {
        const int pieces = n * (D / 4), all = room * (D / 4);
        for (int i0 = tid; i0 < all; i0 += N * 64 * kWavesG) {
            f32x4 v[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {                        // (rows past the end are the last one again: walked once more it changes nothing)
                const int i = min(i0 + k * 64 * kWavesG, all - 1);
                v[k] = load4(K + 4 * (size_t)(i < pieces ? i : pieces - D / 4 + i % (D / 4)));
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int i = min(i0 + k * 64 * kWavesG, all - 1);
                *(f32x4 *)(rows + i / (D / 4) * S + i % (D / 4) * 4) = v[k];
            }
        }
        if (tid < 2) flags[tid] = 0;
    }
    __syncthreads();
    const int run = tid / PR, p = tid % PR, a = run * L;
    const bool works = a < n;
    float *const mine = rows + 2 * p;
    // rows t .. end - 1 (whole batches) in order from `held`, the next batch's reads issued before this one is worked on; with `write` they become what is held
    auto walk = [&](int t, int end, float2 held, auto write) __attribute__((always_inline)) {
        float2 k[2][N];
        auto fetch = [&](float2 (&x)[N], int from) {
            const float *const r = mine + from * S;
#pragma unroll
            for (int u = 0; u < N; ++u) x[u] = *(const float2 *)(r + u * S);
        };
        auto work = [&](const float2 (&x)[N]) {
            float *const r = mine + t * S;
#pragma unroll
            for (int u = 0; u < N; ++u) {
                held.x = fabsf(x[u].x - held.x) > theta ? x[u].x : held.x;                  // Eq. 2 in binary32, Eq. 3
                held.y = fabsf(x[u].y - held.y) > theta ? x[u].y : held.y;
                if (write) *(float2 *)(r + u * S) = held;
            }
            t += N;
        };
        if (t < end) fetch(k[0], t);
        while (t < end) {
            fetch(k[1], min(t + N, end - N));
            work(k[0]);
            if (t >= end) break;
            fetch(k[0], min(t + N, end - N));
            work(k[1]);
        }
        return held;
    };
    float2 start = {0.f, 0.f};
    if (works) {
        const int w = max(a - kWarm, 0);                         // (row 0 is the basis row: exact)
        start = walk(w, a, *(const float2 *)(mine + max(w - 1, 0) * S), std::false_type{});
        E[tid] = walk(a, a + L, start, std::false_type{});
    }
    __syncthreads();
    for (int round = 0; round < kRuns; ++round) {
        float2 from = start;
        if (works && run > 0) from = E[tid - PR];
        const bool wrong = __float_as_uint(from.x) != __float_as_uint(start.x) || __float_as_uint(from.y) != __float_as_uint(start.y);
        if (__any(wrong) && (tid & 63) == 0) flags[round & 1] = 1;
        __syncthreads();                                         // (also: every run has read the end of the one before)
        if (!flags[round & 1]) break;
        if (tid == 0) flags[(round + 1) & 1] = 0;
        if (wrong) {
            start = from;
            E[tid] = walk(a, a + L, start, std::false_type{});
        }
        __syncthreads();
    }
    if (works) walk(a, a + L, start, std::true_type{});
    __syncthreads();
}

// Mask words and count of a unit whose reference keys lie in LDS: an entry has fired where a row differs from the one before (it fires only if |k -
// held| > theta >= 0, and then holds k).
template <int D>
__device__ __forceinline__ void write_mask(const float *rows, int n, uint32_t *__restrict__ mask, uint64_t *__restrict__ nnz) {
    constexpr int S = D + 4, WPR = D / 32;
    uint32_t *const total = (uint32_t *)(rows + (size_t)scan_room(n, D) * S + 2 * 64 * kWavesG) + 2;
    if (threadIdx.x == 0) *total = 0;
    __syncthreads();
    uint32_t fired = 0;
    for (int i = threadIdx.x; i < n * WPR; i += 64 * kWavesG) {
        const int t = i / WPR, w = i % WPR;
        const float *x = rows + t * S + 32 * w, *y = x - (t > 0 ? S : 0);
        uint32_t bits = 0;
#pragma unroll
        for (int c = 0; c < 32; c += 4) {
            const f32x4 u = *(const f32x4 *)(x + c), v = *(const f32x4 *)(y + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) bits |= (uint32_t)(__float_as_uint(u[e]) != __float_as_uint(v[e])) << (c + e);
        }
        if (t == 0) bits = ~0u;                                  // the basis row is kept whole
        mask[i] = bits;
        fired += (uint32_t)__popc(bits);
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) fired += __shfl_xor(fired, s);
    if ((threadIdx.x & 63) == 0) atomicAdd(total, fired);
    __syncthreads();
    if (threadIdx.x == 0) *nnz = *total;
}

template <typename T, int D, bool kScans>
__global__ __launch_bounds__(64 * kWavesG) void prefill_generic_kernel(KArgs<T> a) {
    constexpr int VW = D % 64 == 0 ? 4 : 2;      // channels a lane loads and stores at a time
    constexpr int CG = D / (16 * VW);            // channel groups of the output
    constexpr int KS = D / 16;                   // 16-channel groups of the contraction
    constexpr int kRowsG = 16;
    extern __shared__ __attribute__((aligned(16))) float lds_g[];
    float *ml = lds_g;                           // [wave][kRowsG][2] running maximum, sum
    float *obuf = lds_g + kWavesG * kRowsG * 2;  // [wave][kRowsG][D + 4] outputs before the merge

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int n = a.n, W = a.W;
    const int tile = (int)gridDim.x - 1 - (int)blockIdx.x;       // longest rows first; kScans: in front of them the mask
    const int i0 = tile * kRowsG, i_last = min(n - 1, i0 + kRowsG - 1);
    const int h = blockIdx.y, b = blockIdx.z;
    const int unit = b * a.Hkv + h / (a.Hq / a.Hkv);
    if constexpr (kScans) {
        if (i0 >= n) {
            if (h % (a.Hq / a.Hkv) != 0) return;
            scan_rows<D>(a.K + (size_t)unit * n * D, n, a.theta, lds_g);
            write_mask<D>(lds_g, n, a.mask_bits + (size_t)unit * n * (D / 32), a.nnz + unit);
            return;
        }
    }
    if (!kScans && wave == kWavesG - 1 && tile == 0 && h % (a.Hq / a.Hkv) == 0 && a.sum.groups > 0)      // (the shortest rows)
        add_up_nnz(a.sum, lane < 8 ? unit : a.sum.units);
    const T *Qp = a.Q + (size_t)(b * a.Hq + h) * n * D;
    const T *Kp = a.K + (size_t)unit * n * D;
    const T *Vp = a.V + (size_t)unit * n * D;
    const T *Hp = a.Khat + (size_t)unit * n * D;

    // first exact column of row r: start of its square, or of its band (monotone in r either way)
    auto win_start = [&](int r) { return a.sliding ? max(r - W + 1, 0) : (r / W) * W; };
    const int win_first = win_start(i0), win_last = win_start(i_last);
    const int my_i = i0 + l16, my_row = min(my_i, n - 1), my_win = win_start(my_row);
    f32x4 q[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) q[s] = load4(Qp + (size_t)my_row * D + 16 * s + 4 * lg);

    if constexpr (kScans)
        if (win_last > 0) scan_rows<D>(Kp, win_last, a.theta, lds_g);
    const int hat_rows = kScans ? win_last : n, hat_stride = kScans ? D + 4 : D;
    const T *const hats = kScans ? (const T *)lds_g : Hp;

    f32x4 o[CG][VW];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e) o[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int jb = wave * kKeys; jb <= i_last; jb += kWavesG * kKeys) {
        // scores of the block: X = K, or K_hat where every row has the block left of its window
        f32x4 s[2];
        auto scores = [&](const T *X, int rows, int stride, f32x4 (&acc)[2]) __attribute__((always_inline)) {
            const T *x0 = X + (size_t)min(jb + l16, rows - 1) * stride + 4 * lg;
            const T *x1 = X + (size_t)min(jb + 16 + l16, rows - 1) * stride + 4 * lg;
            acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g = 0; g < KS; ++g) {
                const f32x4 k0 = load4(x0 + 16 * g), k1 = load4(x1 + 16 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(k0[e], q[g][e], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(k1[e], q[g][e], acc[1], 0, 0, 0);
                }
            }
        };
        const bool far = jb + kKeys <= win_first;
        if constexpr (kScans) {                  // (from different memories)
            if (far)
                scores((const T *)lds_g, hat_rows, hat_stride, s);
            else
                scores(Kp, n, D, s);
        } else {
            scores(far ? Hp : Kp, n, D, s);
        }
        if (!far && jb < win_last) {             // some row has part of the block left of its window
            f32x4 sh[2];
            scores(hats, hat_rows, hat_stride, sh);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[kt][r] = jb + 16 * kt + 4 * lg + r >= my_win ? s[kt][r] : sh[kt][r];
        }
        float bm = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool seen = jb + 16 * kt + 4 * lg + r <= my_i;
                s[kt][r] = seen ? s[kt][r] * a.scale_log2 : -INFINITY;
                bm = fmaxf(bm, s[kt][r]);
            }
        bm = fmaxf(bm, __shfl_xor(bm, 16));
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const float m_new = fmaxf(m, bm);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;    // (a row that sees nothing of this wave's keys yet)
        const float alpha = exp2f(m - m_use);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int g = 0; g < CG; ++g)
#pragma unroll
            for (int e = 0; e < VW; ++e) o[g][e] *= alpha;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[kt][r] = exp2f(s[kt][r] - m_use);
                l += s[kt][r];
            }
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T *v = Vp + (size_t)min(jb + 16 * kt + 4 * lg + r, n - 1) * D + VW * l16;   // (p is 0 past the row)
#pragma unroll
                for (int g = 0; g < CG; ++g) {
                    float vv[VW];
                    if constexpr (VW == 4) {
                        const f32x4 x = load4(v + 64 * g);
                        for (int e = 0; e < 4; ++e) vv[e] = x[e];
                    } else {
                        const f32x2 x = load2(v + 32 * g);
                        for (int e = 0; e < 2; ++e) vv[e] = x[e];
                    }
#pragma unroll
                    for (int e = 0; e < VW; ++e) o[g][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[e], s[kt][r], o[g][e], 0, 0, 0);
                }
            }
    }

    // the waves' partial results meet: row maxima and sums first, then the outputs at the common maximum
    if constexpr (kScans) __syncthreads();       // (the reference keys lay there)
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (lg == 0) {
        ml[(wave * kRowsG + l16) * 2] = m;
        ml[(wave * kRowsG + l16) * 2 + 1] = l;
    }
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float *dst = obuf + (size_t)(wave * kRowsG + l16) * (D + 4) + 16 * VW * g + VW * (4 * lg + r);
#pragma unroll
            for (int e = 0; e < VW; ++e) dst[e] = o[g][e][r];
        }
    __syncthreads();
    for (int idx = threadIdx.x; idx < kRowsG * (D / 4); idx += 64 * kWavesG) {
        const int row = idx / (D / 4), c = (idx % (D / 4)) * 4;
        if (i0 + row >= n) continue;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWavesG; ++w) M = fmaxf(M, ml[(w * kRowsG + row) * 2]);   // wave 0 has key 0: M is finite
        float L = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWavesG; ++w) {
            const float f = exp2f(ml[(w * kRowsG + row) * 2] - M);
            L = fmaf(f, ml[(w * kRowsG + row) * 2 + 1], L);
            acc += f * *(const f32x4 *)(obuf + (size_t)(w * kRowsG + row) * (D + 4) + c);
        }
        const float inv = 1.f / L;
        T *dst = a.O + ((size_t)(b * a.Hq + h) * n + i0 + row) * D + c;
#pragma unroll
        for (int e = 0; e < 4; ++e) store_from_f32(dst, e, acc[e] * inv);
    }
}

template <typename T, int D>
constexpr size_t merge_lds = (size_t)kWavesG * 16 * (D + 6) * sizeof(float);

template <typename T, int D>
void launch_one(const PrefillArgs &p, const PrefillScan *scan, hipStream_t s) {
    KArgs<T> a = {};
    a.Q = (const T *)p.Q;
    a.K = (const T *)p.K;
    a.V = (const T *)p.V;
    a.Khat = (const T *)p.Khat;
    a.O = (T *)p.O;
    a.Hq = p.Hq;
    a.Hkv = p.Hkv;
    a.n = p.n;
    a.W = p.W;
    a.sliding = p.sliding;
    a.scale_log2 = p.scale_log2;
    a.sum = p.sum;
    if constexpr (sizeof(T) == 4 && (D == 64 || D == 128)) {
        if (scan) {
            a.mask_bits = scan->mask_bits;
            a.nnz = scan->nnz;
            a.theta = scan->theta;
            const size_t rows = scan_lds(p.n, D), lds = rows > merge_lds<T, D> ? rows : merge_lds<T, D>;
            static std::atomic<uint64_t> set;   // one bit per device
            ensure_dynamic_lds((const void *)prefill_generic_kernel<T, D, true>, 160 * 1024, set);
            static_assert(scan_lds(32768 / D, D) <= 160 * 1024, "prefill_generic_scans");
            hipLaunchKernelGGL((prefill_generic_kernel<T, D, true>), dim3((p.n + 15) / 16 + 1, p.Hq, p.B), dim3(64 * kWavesG), lds, s, a);
            return;
        }
    }
    // (32 rows per work group, which halve the reads of K and V per row, took longer: fp32, 8 heads of 64, 2048 tokens 97.6 us
    // against 85.3, 8 heads of 128 182 against 152; bf16, 4 x 1000 tokens, 20 / 5 heads of 96 344 against 226.)
    static std::atomic<uint64_t> lds_set;   // per instantiation, one bit per device
    ensure_dynamic_lds((const void *)prefill_generic_kernel<T, D, false>, (int)merge_lds<T, D>, lds_set);
    hipLaunchKernelGGL((prefill_generic_kernel<T, D, false>), dim3((p.n + 15) / 16, p.Hq, p.B), dim3(64 * kWavesG), (merge_lds<T, D>), s, a);
}

template <typename T>
bool launch_by_dim(const PrefillArgs &p, const PrefillScan *scan, hipStream_t s) {
    switch (p.d) {
        case 32: launch_one<T, 32>(p, scan, s); return true;
        case 64: launch_one<T, 64>(p, scan, s); return true;
        case 96: launch_one<T, 96>(p, scan, s); return true;
        case 128: launch_one<T, 128>(p, scan, s); return true;
        case 160: launch_one<T, 160>(p, scan, s); return true;
        case 192: launch_one<T, 192>(p, scan, s); return true;
        case 224: launch_one<T, 224>(p, scan, s); return true;
        case 256: launch_one<T, 256>(p, scan, s); return true;
        default: return false;
    }
}

}  // namespace

// Every work group then scans the keys of its unit anew, beside the others as long as each has a compute unit; the scan's own launch spreads over more of them.
// fp32, a scan in front / in the same launch, us a call: 1 head of 64, 64 tokens 9.4 / 7.5, 256 12.6 / 9.8, 400 15.2 / 13.1, 512 16.4 / 14.2 (more rows are not tried: at 588
// of 64 the LDS is full); 2 x 200, 4 heads 12.3 / 9.9; 1 head of 128, 128 tokens 12.6 / 10.6, 256 16.4 / 14.3; up to 256 work groups: 4 x 64, 8 heads 10.0 / 7.8, 480, 8 heads 17.3 / 14.4, 2 x 200, 8 heads
// of 128 17.8 / 14.3.  Not taken: 264, 512, 8 / 1 heads 16.5 / 14.5; 272, 2 x 256, 8 heads 13.7 / 14.9 and 1 x 256, 16 / 4 heads 12.8 / 14.9; 288, 128, 32 / 8 heads 10.7 / 11.1; 896, 8 x 200, 8
// heads 23.3 / 25.1.
bool prefill_generic_scans(const PrefillArgs &p) {
    return p.dtype == 0 && (p.d == 64 || p.d == 128) && (int64_t)p.n * p.d <= 32768 &&
           (int64_t)p.B * p.Hq * ((p.n + 15) / 16 + 1) <= device_cu_count();
}

bool launch_prefill_generic(const PrefillArgs &p, const PrefillScan *scan, hipStream_t s) {
    return p.dtype == 0 ? launch_by_dim<float>(p, scan, s) : launch_by_dim<bf16_t>(p, scan, s);
}

}  // namespace da
