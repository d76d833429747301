// What the bf16 prefill kernels share: operand types, loads straight into LDS, the phases' border, divisions by what the host knows.
#pragma once
#include <utility>

#include "common.hpp"

namespace da {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) char lds_char;

// n / d for 0 <= n < 2^31 by a divisor known to the host: three scalar instructions, where the division's own two dozen
// (times nine, one after the other, before the first load can go out) took 0.5 us of every work group
struct Divisor {
    uint32_t mul, shift;
    int d;
};
inline Divisor divisor(int d) {
    uint32_t l = 0;
    while (((uint64_t)1 << l) < (uint64_t)d) ++l;
    return Divisor{(uint32_t)((((uint64_t)1 << (31 + l)) / (uint64_t)d) + 1u), l, d};
}
template <typename Div>          // (Divisor, in whichever address space)
__device__ __forceinline__ int quotient(int n, const Div &d) { return (int)(__umulhi(2u * (uint32_t)n, d.mul) >> d.shift); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// 64 x 16 bytes from base + at + the lanes' offsets to LDS bytes lds + at .. + 1023 (wave-uniform; `at` is the instruction's own
// offset, which moves both ends), lane after lane.  In asm, so that the compiler does not order later LDS reads behind it: whoever
// reads the tile waits for the count (wait_loads) and then passes a barrier.  m0 is declared as written: uses of its own that the compiler makes of it must not lie across this (the
// warning, that it will not restore a reserved register, is what is wanted; as an operand that the compiler writes it
// cost 0.6 % on 4 x 8192 tokens).  (s_nop: m0 may be used by an LDS load one wait state after it was written.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int At>
__device__ __forceinline__ void load_to_lds(const char *base, uint32_t off, uint32_t lds) {
    static_assert(At >= 0 && At < 4096, "13 bits, signed");
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)), "n"(At)
                 : "memory", "m0");
}
// two of them, 1 KiB apart
__device__ __forceinline__ void loads_to_lds(const char *base, const uint32_t (&off)[2], uint32_t lds) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %2\n\t"
                 "global_load_lds_dwordx4 %1, %2 offset:1024" ::"v"(off[0]), "v"(off[1]), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds))
                 : "memory", "m0");
}
#pragma clang diagnostic pop
// 16 bytes a lane that the caller waits for.  (s_nop: a scalar register that a vector instruction has just written - a readlane, or a
// spilled one read back - may be used as an address five wait states later, which the compiler does not look after inside asm.  The
// tile loads above do without: their rows are scalar arithmetic, and nothing in these kernels is spilled.)
template <int At>
__device__ __forceinline__ void load_in_flight(u32x4 &to, const char *base, uint32_t off) {
    asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2 offset:%3" : "+v"(to) : "v"(off), "s"(base), "n"(At) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {                   // until at most N of this wave's loads are in flight
    static_assert(N < 64, "six bits of the count");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
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

// the lane's number, worked out where it is needed once per tile instead of held in a register through the walk
__device__ __forceinline__ int lane_here() {
    uint32_t none = 0;
    asm volatile("" : "+s"(none));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
}

}  // namespace da
