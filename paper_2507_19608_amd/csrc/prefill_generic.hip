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
// chip, operands by scalar loads); rows by 16 and keys by 8 give 128 waves of one or two blocks each: 6.8 us, 16.0 for the whole
// call with the scan.
//
// Matrix-core layout (16x16x4, wave64): A lane l holds row l % 16, k = l / 16; B lane l column l % 16, same k; D lane l
// column l % 16, rows 4 (l / 16) + r.  Scores are taken transposed (keys x query rows): a lane owns one query row, and
// register r of a score tile is the B operand of a P V step whose k-th key is 4 k + r.  The contraction over channels runs
// in the order that lets every operand be a 16-byte load of a row (step e of group s: channel 16 s + 4 (l / 16) + e), and
// output tile e of a channel group covers the channels VW m + e, so that a lane loads and stores VW consecutive ones.
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

template <typename T, int D>
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
    const int tile = (int)gridDim.x - 1 - (int)blockIdx.x;       // longest rows first
    const int i0 = tile * kRowsG, i_last = min(n - 1, i0 + kRowsG - 1);
    const int h = blockIdx.y, b = blockIdx.z;
    const int unit = b * a.Hkv + h / (a.Hq / a.Hkv);
    if (wave == kWavesG - 1 && tile == 0 && h % (a.Hq / a.Hkv) == 0 && a.sum.groups > 0)      // (the shortest rows)
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

    f32x4 o[CG][VW];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e) o[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int jb = wave * kKeys; jb <= i_last; jb += kWavesG * kKeys) {
        // scores of the block: X = K, or K_hat where every row has the block left of its window
        f32x4 s[2];
        auto scores = [&](const T *X, f32x4 (&acc)[2]) {
            const T *x0 = X + (size_t)min(jb + l16, n - 1) * D + 4 * lg;
            const T *x1 = X + (size_t)min(jb + 16 + l16, n - 1) * D + 4 * lg;
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
        scores(far ? Hp : Kp, s);
        if (!far && jb < win_last) {             // some row has part of the block left of its window
            f32x4 sh[2];
            scores(Hp, sh);
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
void launch_one(const PrefillArgs &p, hipStream_t s) {
    KArgs<T> a;
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
    // (32 rows per work group, which halve the reads of K and V per row, took longer: fp32, 8 heads of 64, 2048 tokens 97.6 us
    // against 85.3, 8 heads of 128 182 against 152; bf16, 4 x 1000 tokens, 20 / 5 heads of 96 344 against 226.)
    constexpr size_t lds = (size_t)kWavesG * 16 * (D + 6) * sizeof(float);
    static std::atomic<uint64_t> lds_set;   // per instantiation, one bit per device
    ensure_dynamic_lds((const void *)prefill_generic_kernel<T, D>, (int)lds, lds_set);
    hipLaunchKernelGGL((prefill_generic_kernel<T, D>), dim3((p.n + 15) / 16, p.Hq, p.B), dim3(64 * kWavesG), lds, s, a);
}

template <typename T>
bool launch_by_dim(const PrefillArgs &p, hipStream_t s) {
    switch (p.d) {
        case 32: launch_one<T, 32>(p, s); return true;
        case 64: launch_one<T, 64>(p, s); return true;
        case 96: launch_one<T, 96>(p, s); return true;
        case 128: launch_one<T, 128>(p, s); return true;
        case 160: launch_one<T, 160>(p, s); return true;
        case 192: launch_one<T, 192>(p, s); return true;
        case 224: launch_one<T, 224>(p, s); return true;
        case 256: launch_one<T, 256>(p, s); return true;
        default: return false;
    }
}

}  // namespace

bool launch_prefill_generic(const PrefillArgs &p, hipStream_t s) {
    return p.dtype == 0 ? launch_by_dim<float>(p, s) : launch_by_dim<bf16_t>(p, s);
}

}  // namespace da
