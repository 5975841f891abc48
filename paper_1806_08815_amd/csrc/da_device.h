// da_device.h -- device helpers shared by the step kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "da_internal.h"

namespace dapt {
namespace {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

enum : uint32_t { kTagMetropolis = 0, kTagSelect = 1, kTagExchange = 2, kTagInit = 3 };

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 products
// with the key advanced by the Weyl constants between rounds.
__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += kPhiloxW0;
            k1 += kPhiloxW1;
        }
        const uint64_t p0 = (uint64_t)kPhiloxM0 * (uint64_t)c0;   // v_mad_u64_u32
        const uint64_t p1 = (uint64_t)kPhiloxM1 * (uint64_t)c2;
        c0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        c1 = (uint32_t)p1;
        c2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c3 = (uint32_t)p0;
    }
    return make_uint4(c0, c1, c2, c3);
}

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int w) {
    return w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
}

// Number of set bits of `mask` in lanes below this one.
__device__ __forceinline__ int mbcnt64(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ int readlane(int v, int lane) {
    return __builtin_amdgcn_readlane(v, lane);
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
// a wave-uniform 64-bit value kept in scalar registers (the 64-bit division
// of the level arithmetic leaves its results in vector registers)
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint64_t u = (uint64_t)v;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Exclusive prefix sum over the wave of c and the wave total from a DPP scan:
// inclusive sums within rows of 16 lanes (shifts 1,
// 2, 4, 8), then each row's predecessors added by the row broadcasts of lanes
// 15 and 31; six dependent adds instead of a ballot and two mbcnt per bit.
__device__ __forceinline__ void wave_scan(int c, int &excl, int &total) {
    int v = c;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    excl = v - c;
    total = __builtin_amdgcn_readlane(v, 63);
}

// h[bit] for a wave-uniform bit: a select tree on the bits of `bit` (F - 1
// selects, log2 F uniform conditions)
// (explicit selects: written as plain conditionals the compiler turns the
// tree back into an indexed read, a compare chain per level)
template <int F>
__device__ __forceinline__ int pick_field(const int (&h)[F], int bit) {
    const int ub = __builtin_amdgcn_readfirstlane(bit);
    int v[F];
#pragma unroll
    for (int f = 0; f < F; ++f) v[f] = h[f];
#pragma unroll
    for (int w = 1; w < F; w <<= 1) {
        const uint64_t up = (ub & w) ? ~0ull : 0ull;   // wave-uniform lane mask
#pragma unroll
        for (int q = 0; q < F; q += 2 * w)
            asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(v[q]) : "v"(v[q]), "v"(v[q + w]), "s"(up));
    }
    return v[0];
}

template <typename T, int F>
struct VecOf {
    typedef T type __attribute__((ext_vector_type(F)));
};

// h[f] += raw[f] * dw for 16-bit couplings and |dw| < 2^15: one 16 x 16 -> 32
// bit multiply-add per field, which takes the coupling in place from its half
// of the loaded dword (op_sel selects the high half).
template <typename WT, int F>
__device__ __forceinline__ void update_i16(const typename VecOf<WT, F>::type &raw, int dw,
                                           int (&h)[F]) {
    if constexpr (sizeof(WT) == 2 && F == 2) {
        const int pr = __builtin_bit_cast(int, raw);
        asm("v_mad_i32_i16 %0, %1, %2, %0" : "+v"(h[0]) : "v"(pr), "s"(dw));
        asm("v_mad_i32_i16 %0, %1, %2, %0 op_sel:[1,0,0,0]" : "+v"(h[1]) : "v"(pr), "s"(dw));
    } else if constexpr (sizeof(WT) == 2) {
        typedef typename VecOf<int, F / 2>::type PairV;
        const PairV pr = __builtin_bit_cast(PairV, raw);
#pragma unroll
        for (int q = 0; q < F / 2; ++q) {
            asm("v_mad_i32_i16 %0, %1, %2, %0" : "+v"(h[2 * q]) : "v"(pr[q]), "s"(dw));
            asm("v_mad_i32_i16 %0, %1, %2, %0 op_sel:[1,0,0,0]" : "+v"(h[2 * q + 1]) : "v"(pr[q]), "s"(dw));
        }
    }
}

// Level in force at step s of an S-step, L-level schedule: floor(s L / S),
// clamped to the last level (the host never launches steps s >= S; the clamp
// keeps a level-table read in range whatever it is given).
__device__ __forceinline__ int level_of(int64_t s, int32_t L, int64_t S) {
    return S > 0 ? min((int)((s * (int64_t)L) / S), L - 1) : 0;
}

// First step whose level exceeds `lvl`.
__device__ __forceinline__ int64_t next_level_step(int lvl, int32_t L, int64_t S) {
    if (lvl + 1 >= L) return INT64_MAX;
    return ((int64_t)(lvl + 1) * S + L - 1) / L;
}

}  // namespace
}  // namespace dapt
