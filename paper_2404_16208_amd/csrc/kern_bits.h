// kern_bits.h -- bit-matrix helpers shared by the sample-tiled kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ranc {

// Sample (within its 32-sample group) of bit b of a history word. The order
// is the row order of the 32x32 MFMA result (lane l, element r is row
// 8*(r/4) + 4*(l/32) + r%4), so a lane's 16 results and its partner lane's
// form one word without reordering.
__device__ inline int sigma32(int b) { return 8 * ((b & 15) >> 2) + 4 * (b >> 4) + (b & 3); }

// Bit of sample i (within its 32-sample group) in a history word: the
// inverse of sigma32.
__device__ inline int sigma32_inv(int i) { return 16 * ((i & 7) >> 2) + 4 * (i >> 3) + (i & 3); }

// x of lane ^ K within each row of 16 lanes, as a data-parallel primitive
// (vector pipe only: no LDS round trip, whose latency the five dependent
// stages of a transpose would each pay).
template <int K> __device__ inline uint32_t lane_xor(uint32_t x)
{
    static_assert(K == 1 || K == 2 || K == 4 || K == 8, "within a row of 16 lanes");
    constexpr int QUAD_XOR1 = 0xB1, QUAD_XOR2 = 0x4E, QUAD_XOR3 = 0x1B, HALF_MIRROR = 0x141, ROR8 = 0x128;
    if constexpr (K == 4) {   // lane ^ 7, then lane ^ 3
        x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, HALF_MIRROR, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, QUAD_XOR3, 0xF, 0xF, true);
    } else {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, K == 1 ? QUAD_XOR1 : K == 2 ? QUAD_XOR2 : ROR8, 0xF, 0xF,
                                                     true);
    }
}

// Sum of a 32-bit value over the 64 lanes of a wavefront (every lane gets it).
__device__ inline uint32_t wave_sum_dpp(uint32_t v)
{
    v += lane_xor<1>(v);
    v += lane_xor<2>(v);
    v += lane_xor<4>(v);
    v += lane_xor<8>(v);
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = (uint32_t)a[0] + (uint32_t)a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (uint32_t)b[0] + (uint32_t)b[1];
}

// One stage of a recursive bit-matrix transpose: lanes whose index has bit K
// clear exchange the bits with index bit K set for their partner's (lane ^ K)
// bits with index bit K clear.
template <int K>
__device__ inline uint32_t transpose_stage(uint32_t x, int lane)
{
    const bool up = (lane & K) != 0;
    if constexpr (K == 16) {
        // even[l], odd[l]: x of the even and the odd row of 16 lanes of l's half
        const auto sw = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        const uint32_t even = (uint32_t)sw[0], odd = (uint32_t)sw[1];
        return __builtin_amdgcn_perm(odd, even, up ? 0x07060302u : 0x05040100u);
    } else if constexpr (K == 8) {
        return __builtin_amdgcn_perm(lane_xor<8>(x), x, up ? 0x03070105u : 0x06020400u);
    } else {
        constexpr uint32_t M = K == 4 ? 0x0F0F0F0Fu : K == 2 ? 0x33333333u : 0x55555555u;
        const uint32_t r = __builtin_rotateright32(lane_xor<K>(x), up ? K : 32 - K);
        const uint32_t keep = up ? ~M : M;
        return (x & keep) | (r & ~keep);
    }
}

// 32 x 32 bit transpose within each half-wave: lane i of a half receives, as
// bit j, bit i of lane j of the same half. Every lane must be active.
__device__ inline uint32_t transpose32(uint32_t x, int lane)
{
    x = transpose_stage<16>(x, lane);
    x = transpose_stage<8>(x, lane);
    x = transpose_stage<4>(x, lane);
    x = transpose_stage<2>(x, lane);
    return transpose_stage<1>(x, lane);
}

// Four rows' compare, select and spike bit: v[i] = u[i] >= th ? r[i] : v[i],
// f = 2 f + fire for i = 3 down to 0. Written out because the compiler turns
// the spike bit into a select and a shift (two instructions); the compare's
// lane mask is the carry of one add. Four compares come first, so each mask is
// read at least three instructions after it was written (two are required).
__device__ __forceinline__ void fire_rows(uint32_t &f, int32_t &v0, int32_t &v1, int32_t &v2, int32_t &v3, int32_t u0,
                                          int32_t u1, int32_t u2, int32_t u3, int32_t r0, int32_t r1, int32_t r2,
                                          int32_t r3, int32_t th)
{
    uint64_t m1, m2, m3;
    asm volatile("v_cmp_ge_i32_e64 %7, %11, %16\n\t"
        "v_cmp_ge_i32_e64 %6, %10, %16\n\t"
        "v_cmp_ge_i32_e64 %5, %9, %16\n\t"
        "v_cmp_ge_i32_e32 vcc, %8, %16\n\t"
        "v_cndmask_b32_e64 %4, %4, %15, %7\n\t"
        "v_cndmask_b32_e64 %3, %3, %14, %6\n\t"
        "v_cndmask_b32_e64 %2, %2, %13, %5\n\t"
        "v_cndmask_b32_e32 %1, %1, %12, vcc\n\t"
        "v_addc_co_u32_e64 %0, %7, %0, %0, %7\n\t"
        "v_addc_co_u32_e64 %0, %6, %0, %0, %6\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %5\n\t"
        "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+v"(f), "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(u0), "v"(u1), "v"(u2), "v"(u3), "v"(r0), "v"(r1), "v"(r2), "v"(r3), "v"(th)
        : "vcc");
}
// (the same with u = v and one reset value)
__device__ __forceinline__ void fire_rows(uint32_t &f, int32_t &v0, int32_t &v1, int32_t &v2, int32_t &v3, int32_t rs,
                                          int32_t th)
{
    uint64_t m1, m2, m3;
    asm volatile("v_cmp_ge_i32_e64 %7, %4, %9\n\t"
        "v_cmp_ge_i32_e64 %6, %3, %9\n\t"
        "v_cmp_ge_i32_e64 %5, %2, %9\n\t"
        "v_cmp_ge_i32_e32 vcc, %1, %9\n\t"
        "v_cndmask_b32_e64 %4, %4, %8, %7\n\t"
        "v_cndmask_b32_e64 %3, %3, %8, %6\n\t"
        "v_cndmask_b32_e64 %2, %2, %8, %5\n\t"
        "v_cndmask_b32_e32 %1, %1, %8, vcc\n\t"
        "v_addc_co_u32_e64 %0, %7, %0, %0, %7\n\t"
        "v_addc_co_u32_e64 %0, %6, %0, %0, %6\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %5\n\t"
        "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+v"(f), "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(rs), "v"(th)
        : "vcc");
}

// fire_rows' spike bits before a lane swap takes them as they are: the swap needs
// two wait states after a vector instruction wrote its register, and the compiler
// keeps them only after instructions of its own.
__device__ __forceinline__ void rows_settled(uint32_t &f)
{
    asm volatile("s_nop 1" : "+v"(f));
}

}  // namespace ranc
