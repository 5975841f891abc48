// da_wave.hip -- the Digital Annealer step with every replica in one wavefront or
// in a team of wavefronts that draw and bound for themselves.
//
// Method: Algorithm 2 (Sec. II.B) of Aramon et al., arXiv:1806.08815, and its
// parallel-tempering rounds (Sec. II.D).
//
// One wave holds a replica of up to 1024 variables: lane g owns the F variables
// g*F .. g*F+F-1 (F = 1, 2, 4, 8, 16).  Then nothing of a step leaves the wave: no
// barrier, no exchange through LDS, no random-number waves.  What bounds such a
// step is its instruction count (a wave issues one instruction of any kind every
// four cycles), so the work is laid out to issue little and to wait for nothing:
//   * The Metropolis test is the sign of one sum per flip.  The threshold
//     of a draw is bracketed by one fp32 log2 and multiply-add of the draw (see
//     wave_level), and a cost inside the bracket is decided by the definition
//     d < T (-ln U_u) in double.  No threshold table, bracket table or direct
//     table is built, staged or read.
//   * Costs are held as fixed point d 2^q, q chosen per level so that T 2^q is
//     about 2^16: the bracket is then a few parts in 10^5 of T for couplings of
//     any scale, +-1 instances included.
//   * Step s+1's draws (Philox) and brackets are computed while row k of W is
//     in flight.  With F < 8 a Philox block serves 8/F lanes; the wave then
//     draws 8/F steps at once, one block per lane, and hands them out through LDS.
//   * The first rounds of Philox are constant over the steps but for two xors;
//     the xors of the later ones are three-input.
//   * Energy, offset and counts are wave-uniform scalars.
// ns per step, before (compute and random-number waves on tables, da_kernels.hip)
// and now: N = 64, 16 replicas 668 -> 200; N = 512 Gaussian, 64 replicas ~600 -> 430;
// N = 1024 Gaussian, 1024 replicas 690 -> 660 (VALU instructions per replica-step
// 359 -> 230; two such anneals at once 690 -> 465 each), 2048 replicas 1440 -> 1016,
// +-1 2190 -> 1108.
//
// Beyond 512 variables with few replicas the chain of one wave is too long, and a
// team shares it (wave_run, team_draws): one barrier a step, the lanes' records and
// the bounds of random-number waves through LDS.  What bounds it then is the chain
// row fetch (231 ns from L2), test, scan, exchange, search: N = 1024, 128 replicas
// 543 (direct tables, +-1), 533 (Gaussian), 718 (+-1, short levels) -> 492 .. 529;
// dense int32 N = 999 890 -> 552; a new temperature every step 1030 -> 570; N = 8192,
// 64 replicas 2700 -> 1120.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "da_device.h"
#include "da_internal.h"

#ifndef DAPT_PART
#error "compile with -DDAPT_PART=0 .. 9"
#endif

namespace dapt {

namespace {

constexpr double kLn2 = 0.69314718055994530942;

// Round keys of the draws and the xor that takes them, a ^ b ^ key.
//   From scalar registers by the builtin, not inline asm: keys that were spilled come
// back by v_readlane, after which a vector instruction may read the scalar only two
// wait states later.  The compiler keeps these for its own instructions and cannot
// for text.
//   In vector registers (VEC) inline asm has no such rule to break, and the compiler
// then spreads the field update among the draws: one wave of 16 flips per lane,
// 16-bit couplings, 1024 replicas of N = 1024: 67.9 ms an anneal with the builtin, 66.4
// so, for 14 registers.  Where those spill (32-bit couplings) or the waves share the
// update's wait (teams, batches: 8.4 against 9.3 ms) it is the slower.
template <bool VEC>
struct DrawKeys {
    uint32_t k0, k1;
    __device__ __forceinline__ DrawKeys(uint32_t a, uint32_t b) : k0(a), k1(b) {}
    __device__ __forceinline__ uint32_t xor_k0(uint32_t a, uint32_t b, int r) const {
        return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b,
                                                     (int)(k0 + (uint32_t)r * kPhiloxW0), 0x96);
    }
    __device__ __forceinline__ uint32_t xor_k1(uint32_t a, uint32_t b, int r) const {
        return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b,
                                                     (int)(k1 + (uint32_t)r * kPhiloxW1), 0x96);
    }
};
template <>
struct DrawKeys<true> {
    uint32_t a[10], b[10];   // of rounds 3 .. 9
    __device__ __forceinline__ DrawKeys(uint32_t k0, uint32_t k1) {
#pragma unroll
        for (int r = 3; r < 10; ++r) {
            a[r] = k0 + (uint32_t)r * kPhiloxW0;
            b[r] = k1 + (uint32_t)r * kPhiloxW1;
            asm("" : "+v"(a[r]), "+v"(b[r]));   // (held, not made again at each use)
        }
    }
    static __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t k) {
        uint32_t r;
        asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "v"(k));
        return r;
    }
    __device__ __forceinline__ uint32_t xor_k0(uint32_t x, uint32_t y, int r) const {
        return xor3(x, y, a[r]);
    }
    __device__ __forceinline__ uint32_t xor_k1(uint32_t x, uint32_t y, int r) const {
        return xor3(x, y, b[r]);
    }
};

// The Metropolis draws of one Philox block (counter (block, step, rid, 0)) over
// many steps.  Of the ten rounds, what does not depend on the step is kept: the
// first product of rounds 0 and 2, the second of rounds 0 and 1.
struct DrawBlock {
    uint32_t b1, d2, e2, f3;   // with the round keys they are xored with folded in
    __device__ __forceinline__ void init(uint32_t block, uint32_t rid, uint32_t k0, uint32_t k1) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * block, p1 = (uint64_t)kPhiloxM1 * rid;
        const uint32_t c2 = (uint32_t)(p0 >> 32) ^ kTagMetropolis ^ k1;
        b1 = (uint32_t)p0 ^ (k1 + kPhiloxW1);
        const uint64_t q1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t c0 = (uint32_t)(q1 >> 32) ^ (uint32_t)p1 ^ (k0 + kPhiloxW0);
        d2 = (uint32_t)q1 ^ (k0 + 2u * kPhiloxW0);
        const uint64_t q0 = (uint64_t)kPhiloxM0 * c0;
        e2 = (uint32_t)(q0 >> 32) ^ (k1 + 2u * kPhiloxW1);
        f3 = (uint32_t)q0 ^ (k1 + 3u * kPhiloxW1);
    }
    // r0: hi(M1 rid) ^ k0, wave-uniform
    template <bool VEC>
    __device__ __forceinline__ uint4 draw(uint32_t step, uint32_t r0,
                                          const DrawKeys<VEC> &keys) const {
        const uint64_t s1 = (uint64_t)kPhiloxM0 * (r0 ^ step);      // round 1
        uint32_t c2 = (uint32_t)(s1 >> 32) ^ b1;
        uint64_t p1 = (uint64_t)kPhiloxM1 * c2;                     // round 2
        uint32_t c0 = (uint32_t)(p1 >> 32) ^ d2;
        uint32_t c1 = (uint32_t)p1;
        c2 = (uint32_t)s1 ^ e2;
        uint64_t p0 = (uint64_t)kPhiloxM0 * c0;                     // round 3
        p1 = (uint64_t)kPhiloxM1 * c2;
        c0 = keys.xor_k0((uint32_t)(p1 >> 32), c1, 3);
        c1 = (uint32_t)p1;
        c2 = (uint32_t)(p0 >> 32) ^ f3;
        uint32_t c3 = (uint32_t)p0;
#pragma unroll
        for (int r = 4; r < 10; ++r) {
            p0 = (uint64_t)kPhiloxM0 * c0;
            p1 = (uint64_t)kPhiloxM1 * c2;
            c0 = keys.xor_k0((uint32_t)(p1 >> 32), c1, r);
            c1 = (uint32_t)p1;
            c2 = keys.xor_k1((uint32_t)(p0 >> 32), c3, r);
            c3 = (uint32_t)p0;
        }
        return make_uint4(c0, c1, c2, c3);
    }
};

// One temperature of the wave kernel.  With T' = T 2^q and y = T' (-ln U_u), a
// flip of fixed-point cost d' = d 2^q is accepted iff d' < y.  Per draw
//   L(u) = round(log2(u + 1/2) ga + gb), ga = -T' ln 2, gb = 16 T' ln 2 - margin,
// where the margin covers the rounding and m, a bound on the error (gerr per
// unit of T': the fp32 roundings and ln 2 times the device's log2 error, which
// is measured over all 65536 arguments).  Then d' <= L + c0 implies d' < y, and
// d' >= L + c0 + wt implies d' >= y; a cost in between takes the definition.
//   Without CLAMP the sum carries 1.5 2^23, so that its bits are that constant's
// plus L (T' < 2^18 keeps it in [2^23, 2^24)); c0 = 0, wt = 2 m + 3.
//   With CLAMP, L = max(0, trunc(..)) by a conversion: any T', and costs of zero
// never fall in between, which T' of a few units (couplings too large for more
// fraction bits) would make common: where q >= 1, c0 = 1 is allowed, as d' <= 1
// means d' <= 0 < y.  wt = 2 m + 2.
// T = 0 accepts d' < 0 only: ga = 0 and L + c0 = -1 state it exactly.
// The test uses z = L + c0 + E_off' - s' less one where x = 0 (s' = (1 - 2x) h',
// its negative taken as a one's complement): z >= 0 accepts, z < -wt rejects.
struct WaveLevel {
    float ga, gb;
    uint32_t zamb;   // z is undecided iff (uint32_t)z > zamb
    int c0;          // with the constant of the sum's bits taken off
    int q;
};

template <bool CLAMP>
__device__ __forceinline__ WaveLevel wave_level(double T, int qcap, float gerr) {
    WaveLevel w;
    const bool pos = __double_as_longlong(T) != 0;   // (T >= 0)
    // (T = f 2^e with f in [1/2, 1), e = 0 for T = 0: T 2^q < 2^17 where q > 0)
    const int q = min(max(17 - __builtin_amdgcn_frexp_exp(T), 0), qcap);
    const double Tq = __builtin_ldexp(T, q);
    const float m = (float)Tq * gerr + 0.01f;
    const int c0 = !CLAMP ? 0 : (pos ? min(q, 1) : -1);
    const int wt = pos ? (int)(2.0f * m) + (CLAMP ? 2 : 3) : 1 - min(q, 1);
    const double mid = Tq * (16.0 * kLn2);
    w.ga = (float)(-Tq * kLn2);
    // (T = 0: L = 0 with c0 = -1, L = -1 with c0 = 0)
    if constexpr (CLAMP) w.gb = (float)(mid - (double)m - (double)c0);
    else w.gb = (float)(12582912.0 + __builtin_floor(mid - (double)m - 0.5));
    w.zamb = 0xFFFFFFFFu - (uint32_t)wt;
    w.c0 = CLAMP ? c0 : (int)((uint32_t)c0 - kGenMagic);
    w.q = q;
    return w;
}

// The level that lane `l` holds, in scalar registers (ga, gb: for the bounds'
// multiply-add, which takes one scalar, as they are).
__device__ __forceinline__ WaveLevel level_at(const WaveLevel &w, int l) {
    WaveLevel r;
    r.ga = __int_as_float(readlane(__float_as_int(w.ga), l));
    r.gb = __int_as_float(readlane(__float_as_int(w.gb), l));
    r.zamb = (uint32_t)readlane((int)w.zamb, l);
    r.c0 = readlane(w.c0, l);
    r.q = readlane(w.q, l);
    return r;
}

template <bool CLAMP>
__device__ __forceinline__ int draw_bound(uint32_t u, float ga, float gb) {
    const float lg = __builtin_amdgcn_logf((float)u + 0.5f);
    const float t = __builtin_fmaf(lg, ga, gb);
    if constexpr (!CLAMP) return __float_as_int(t);
    int L;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(L) : "v"(t));   // negative -> 0
    return L;
}

// Inclusive prefix sum over the wave (rows of 16 by shifts, then the rows'
// predecessors by the broadcasts of lanes 15 and 31).
__device__ __forceinline__ int incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// h[bit], bit wave-uniform (negative: some field).  Of 16 fields by an indexed
// register read, which the compiler makes of a vector: 15 selects cost more
// (1024 replicas of N = 1024: 683 -> 672 ns a step); of 8 the selects are faster (482 -> 436 ns a step), switching the index
// mode on and off stalls the wave.
template <int F>
__device__ __forceinline__ int field_at(const int (&h)[F], int bit) {
    if constexpr (F == 1) {
        return h[0];
    } else if constexpr (F < 16) {
        return pick_field<F>(h, bit);
    } else {
        typedef int V __attribute__((ext_vector_type(F)));
        V v;
#pragma unroll
        for (int f = 0; f < F; ++f) v[f] = h[f];
        return v[bit & (F - 1)];
    }
}

// First set bit of a wave-uniform mask; -1 when there is none.
__device__ __forceinline__ int first_bit(uint64_t m) {
    int r;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(m));
    return r;
}
__device__ __forceinline__ int first_bit(uint32_t m) {
    int r;
    asm("s_ff1_i32_b32 %0, %1" : "=s"(r) : "s"(m));
    return r;
}

// Lane records of a replica of several waves: accepted mask, x bits, and the
// inclusive prefix of the accepted counts within the wave.
template <int F>
struct LaneRec {   // F <= 8: one word
    typedef uint32_t type;
    static __device__ __forceinline__ type make(uint32_t acc, uint32_t xb, int incl) {
        return acc | (xb << 8) | ((uint32_t)incl << 16);
    }
    static __device__ __forceinline__ uint32_t acc(type r) { return r & 0xFFu; }
    static __device__ __forceinline__ uint32_t x(type r) { return r >> 8; }   // (low F bits)
    static __device__ __forceinline__ int incl(type r) { return (int)(r >> 16); }
    static __device__ __forceinline__ type lane(type r, int l) { return (type)readlane((int)r, l); }
};
template <>
struct LaneRec<16> {
    typedef uint2 type;
    static __device__ __forceinline__ type make(uint32_t acc, uint32_t xb, int incl) {
        return make_uint2(acc | ((uint32_t)incl << 16), xb);
    }
    static __device__ __forceinline__ uint32_t acc(type r) { return r.x & 0xFFFFu; }
    static __device__ __forceinline__ uint32_t x(type r) { return r.y; }
    static __device__ __forceinline__ int incl(type r) { return (int)(r.x >> 16); }
    static __device__ __forceinline__ type lane(type r, int l) {
        return make_uint2((uint32_t)readlane((int)r.x, l), (uint32_t)readlane((int)r.y, l));
    }
};

// LDS of a team of waves, by step parity: the lanes' records and the energy
// change, then the bounds that the random-number waves hand over.
template <int F>
__host__ __device__ constexpr int team_rec_bytes(int NW) {
    return (NW < 4 ? 4 : NW) * 64 * (F > 8 ? 8 : 4) + 16;
}
// Bounds of one step: of every Philox block the first four draws' and, in the other
// half, the last four's, so that neighbouring lanes read neighbouring 16 bytes.
__host__ __device__ constexpr int team_half_bytes(int N) { return (N + 1023) / 1024 * 128 * 16 + 128; }

// The random-number waves of a team: during step s they write the bounds of step
// s + 1, at its temperature, for the barrier of step s to hand over.  They fill
// issue slots the other waves leave while they wait on each other and on W.
// Each lane draws HB Philox blocks.
template <int HB, bool CLAMP, bool FEAT>
__device__ __forceinline__ void team_draws(const JobDesc &J, int rr, uint8_t *ring, int hw) {
    const int lane = threadIdx.x & 63;
    const int half = team_half_bytes(J.N);
    const uint32_t rid = (uint32_t)__builtin_amdgcn_readfirstlane((int)(J.rid_base + (uint32_t)rr));
    const uint32_t k0 = (uint32_t)J.seed, k1 = (uint32_t)(J.seed >> 32);
    const uint32_t r0 = __umulhi(kPhiloxM1, rid) ^ k0;
    const bool perstep = FEAT && J.stepT != nullptr;
    int64_t a = J.s0, b = J.s1;
    if (J.round_ptr) {
        a = (int64_t)*J.round_ptr * J.K;
        b = a + J.K;
    }
    const uint32_t s0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
    const uint32_t s1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    int lvl = 0;
    uint32_t t_next = 0xFFFFFFFFu;
    auto next_of = [&](int l) -> uint32_t {
        const int64_t n = next_level_step(l, J.L, J.S);
        return (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(n > (int64_t)0x7FFFFFFF ? 0xFFFFFFFFu : (uint32_t)n));
    };
    if (J.lvl_of_rep) {
        lvl = __builtin_amdgcn_readfirstlane(J.lvl_of_rep[rr]);
    } else if (!perstep) {
        lvl = __builtin_amdgcn_readfirstlane(level_of(a, J.L, J.S));
        t_next = next_of(lvl);
    }
    WaveLevel ls;
    float ga, gb;
    auto level_of_step = [&](uint32_t t) {
        if (perstep) {
            ls = wave_level<CLAMP>(
                J.stepT[min((int64_t)((t & ~63u) + (uint32_t)lane), J.S - 1)].T, J.qcap, J.gerr);
        } else {
            ls = wave_level<CLAMP>(J.temps[lvl], J.qcap, J.gerr);
            ga = ls.ga;
            gb = ls.gb;
        }
    };
    level_of_step(s0);
    const DrawKeys<false> keys(k0, k1);
    DrawBlock db[HB];
#pragma unroll
    for (int q = 0; q < HB; ++q)
        db[q].init((uint32_t)((hw * HB + q) * 64 + lane), rid, k0, k1);
    auto produce = [&](uint32_t t) {
        if (perstep) {
            ga = __int_as_float(readlane(__float_as_int(ls.ga), (int)(t & 63u)));
            gb = __int_as_float(readlane(__float_as_int(ls.gb), (int)(t & 63u)));
        }
        uint8_t *slot = ring + (t & 1u) * (2 * half) + (hw * HB * 64 + lane) * 16;
#pragma unroll
        for (int q = 0; q < HB; ++q) {
            const uint4 r = db[q].draw(t, r0, keys);
            int4 e0, e1;
            e0.x = draw_bound<CLAMP>(r.x & 0xFFFFu, ga, gb);
            e0.y = draw_bound<CLAMP>(r.x >> 16, ga, gb);
            e0.z = draw_bound<CLAMP>(r.y & 0xFFFFu, ga, gb);
            e0.w = draw_bound<CLAMP>(r.y >> 16, ga, gb);
            e1.x = draw_bound<CLAMP>(r.z & 0xFFFFu, ga, gb);
            e1.y = draw_bound<CLAMP>(r.z >> 16, ga, gb);
            e1.z = draw_bound<CLAMP>(r.w & 0xFFFFu, ga, gb);
            e1.w = draw_bound<CLAMP>(r.w >> 16, ga, gb);
            *reinterpret_cast<int4 *>(slot + q * 1024) = e0;
            *reinterpret_cast<int4 *>(slot + half + q * 1024) = e1;
        }
    };
    if (s0 != s1) produce(s0);
    __syncthreads();
    for (uint32_t t = s0 + 1; t < s1; ++t) {
        if (t == t_next) {
            lvl = (int64_t)J.L > J.S
                      ? __builtin_amdgcn_readfirstlane(level_of((int64_t)t, J.L, J.S))
                      : lvl + 1;
            t_next = next_of(lvl);
            level_of_step(t);
        } else if (perstep && (t & 63u) == 0u) {
            level_of_step(t);
        }
        produce(t);
        __syncthreads();
    }
    if (s0 != s1) __syncthreads();   // the last step's
    __syncthreads();                 // after the last step
}

// value of lane l
__device__ __forceinline__ double lane_double(double v, int l) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)readlane((int)(u >> 32), l) << 32) |
                                            (uint32_t)readlane((int)(uint32_t)u, l)));
}

// End of a parallel-tempering round for replica rr (one wave of it; its energy is
// stored): the last replica of the chain does the chain's exchange sweep
// (Algorithm 3's move; k_pt_exchange is the same for more than 64 temperatures),
// the last chain opens the next round.  Nothing waits: the others just count
// themselves.  A kernel of its own took 6 us a round.  Lane p holds slot p; the
// pairs are walked in order, each decision after the swaps before it.
__device__ __forceinline__ void pt_sweep(const JobDesc &J, int rr, uint32_t t) {
    const PtDesc &P = J.pt;
    const int lane = threadIdx.x & 63;
    const int M = P.M, c = rr / M;
    uint32_t n = 0;
    // (energies go to and come from the device's coherence point, so a wait for
    // the store before the count is all the order this needs: a device-wide fence
    // would write back a whole L2 for every replica)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0)
        n = __hip_atomic_fetch_add(&P.done[c], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)n) != (uint32_t)M - 1u) return;
    asm volatile("" ::: "memory");
    const bool on = lane < M;
    int rep = 0;
    int64_t E = 0;
    double lnu = 0.0, db = 0.0;
    if (on) {
        rep = P.slot2rep[(size_t)c * M + lane];
        E = __hip_atomic_load(&J.E[(size_t)c * M + rep], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t u = philox((uint32_t)lane, t, (uint32_t)c, kTagExchange, (uint32_t)J.seed,
                                  (uint32_t)(J.seed >> 32)).x & 0xFFFFu;
        lnu = -J.G[u];
        db = P.dbeta[lane];
    }
    int a = readlane(rep, 0);   // the replica that stands in slot p
    int64_t Ea = uniform64(E);
    int slot = rep;             // this lane's slot after the sweep
    bool swapped = false;
    for (int p = 0; p + 1 < M; ++p) {
        const int b = readlane(rep, p + 1);
        const int64_t Eb = (int64_t)(((uint64_t)(uint32_t)readlane((int)(E >> 32), p + 1) << 32) |
                                     (uint32_t)readlane((int)(uint32_t)(uint64_t)E, p + 1));
        const double delta = __dmul_rn(lane_double(db, p), (double)(Ea - Eb));
        const bool sw = lane_double(lnu, p) < delta;
        if (lane == p) {
            slot = sw ? b : a;
            swapped = sw;
        }
        a = sw ? a : b;
        Ea = sw ? Ea : Eb;
    }
    if (lane == M - 1) slot = a;
    if (on) {
        P.slot2rep[(size_t)c * M + lane] = slot;
        P.lvl_of_rep[(size_t)c * M + slot] = lane;
        if (swapped) P.pair_swaps[(size_t)c * (M - 1) + lane] += 1;
    }
    const int sw = (int)__popcll(ballot(swapped));
    if (lane == 0) {
        P.n_swaps[c] += sw;
        P.done[c] = 0u;
        // (every replica of every chain has read the round index before the
        // last chain gets here)
        if (__hip_atomic_fetch_add(&P.round[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
            (uint32_t)P.chains - 1u) {
            P.round[1] = 0u;
            P.round[0] = t + 1u;
        }
    }
}

// Runs steps [s0, s1) of replica rr by the J.NW <= NWC waves of a team (NWC = 1:
// this wave alone; NWC = 16: any number).  wl: W in LDS (WLDS); lds: this wave's
// Philox blocks [2][64] (alone, F < 8), or a team's records and bounds (HELP: from
// its random-number waves; else every wave draws its own, F >= 8).  FEAT: per-step
// schedules and single-trial proposals; without it neither leaves code in the loop.
// VK: round keys in vector registers (DrawKeys).
//
// A team meets at one barrier a step.  Before it every wave leaves its lanes'
// records in LDS; after it every wave finds the chosen flip from them (up to
// four waves: from all records of its own lane number, read at once), reads row
// k of W for its own fields, and the wave that holds the flip leaves its energy
// change for the others to add a step later.
template <typename WT, int F, int NWC, bool HELP, bool WLDS, bool CLAMP, bool FEAT, bool VK = false>
__device__ __forceinline__ void wave_run(const JobDesc &J, int rr, const uint8_t *wl, uint8_t *lds,
                                         int wr) {
    constexpr bool TEAM = NWC > 1;
    typedef LaneRec<F> Rec;
    typedef typename Rec::type RecT;
    const int NW = TEAM ? J.NW : 1;
    static_assert(!HELP || TEAM, "random-number waves serve teams");
    // this step's half of the records, and the other; its energy change at the end
    const int RB = team_rec_bytes<F>(NW);
    int rec_o = 0;
    auto recs = [&](int o) { return reinterpret_cast<RecT *>(lds + o); };
    auto denergy = [&](int o) { return reinterpret_cast<int *>(lds + o + RB - 16); };
    uint4 *ring = reinterpret_cast<uint4 *>(lds);
    constexpr int NB = F >= 8 ? F / 8 : 1;   // Philox blocks per lane and step (F >= 8)
    constexpr int P = F >= 8 ? 1 : 8 / F;   // steps drawn at once
    static_assert(!TEAM || F >= 8, "a team's lanes draw whole blocks");
    constexpr int RW = F >= 2 ? F / 2 : 1;   // 32-bit words of a lane's draws
    constexpr int NX = (F + 3) / 4;
    typedef typename VecOf<WT, F>::type RowV;
    const int lane = threadIdx.x & 63;
    const int i0 = (wr * 64 + lane) * F;
    const int ld = J.ld;
    const bool lane_has = i0 < ld;
    const int col0 = lane_has ? i0 : 0;   // lanes past the row hold ghost flips only
    const uint32_t rid = (uint32_t)__builtin_amdgcn_readfirstlane((int)(J.rid_base + (uint32_t)rr));
    const uint32_t k0 = (uint32_t)J.seed, k1 = (uint32_t)(J.seed >> 32);
    const uint32_t r0 = __umulhi(kPhiloxM1, rid) ^ k0;
    const bool perstep = FEAT && J.stepT != nullptr;
    const bool single = FEAT && J.single != 0;
    const uint32_t ge_mask = lane < F ? ((0xFFFFu << lane) & ((1u << F) - 1u)) : 0u;
    // int32 couplings below 2^23 take the 24-bit multiply-add
    const bool w24 = sizeof(WT) < 4 || J.w24 != 0;

    // --- replica state -----------------------------------------------------
    int h[F];
    uint32_t xb = 0, bxb = 0, vmask = 0;
#pragma unroll
    for (int f = 0; f < F; ++f) h[f] = 0;
    const size_t base = (size_t)rr * ld + i0;
    typedef typename VecOf<int, F>::type IV;
    typedef typename VecOf<uint8_t, F>::type BV;
    if (lane_has) {
        const IV hv = *reinterpret_cast<const IV *>(J.h + base);
        const BV xv = *reinterpret_cast<const BV *>(J.x + base);
        const BV bv = *reinterpret_cast<const BV *>(J.bx + base);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            h[f] = hv[f];
            xb |= (uint32_t)(xv[f] & 1) << f;
            bxb |= (uint32_t)(bv[f] & 1) << f;
            if (i0 + f < J.N) vmask |= 1u << f;
        }
    }
    // the complement of x as bytes 0x00 / 0xFF, four flips per word: a flip's
    // sign mask is then one sign-extended byte operand
    uint32_t nx[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) nx[q] = 0u;
#pragma unroll
    for (int f = 0; f < F; ++f) nx[f >> 2] |= ((xb >> f) & 1u) ? 0u : (0xFFu << (8 * (f & 3)));
    // energies as the best one and what the current one lies above it
    int64_t bE = uniform64(J.bE[rr]);
    int64_t gap = uniform64(J.E[rr]) - bE;
    int eoff = __builtin_amdgcn_readfirstlane(J.eoff[rr]);
    uint32_t nacc = 0;
    const int inc = J.eoff_inc, inc_cap = kEoffMax - J.eoff_inc;
    // past max |h| the offset changes no decision: every flip is accepted
    const int ecap = J.ecap;

    // --- steps and level in force --------------------------------------------
    int64_t a = J.s0, b = J.s1;
    uint32_t pt_round = 0;
    if (J.round_ptr) {
        pt_round = (uint32_t)__builtin_amdgcn_readfirstlane((int)*J.round_ptr);
        a = (int64_t)pt_round * J.K;
        b = a + J.K;
    }
    uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
    const uint32_t s1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    int lvl = 0;
    uint32_t s_next = 0xFFFFFFFFu;   // first step of the next level
    auto next_of = [&](int l) -> uint32_t {
        const int64_t n = next_level_step(l, J.L, J.S);
        return (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(n > (int64_t)0x7FFFFFFF ? 0xFFFFFFFFu : (uint32_t)n));
    };
    auto step_T = [&](uint32_t t) -> double {   // per-step schedules; past the end: the last
        return J.stepT[min((int64_t)t, J.S - 1)].T;
    };
    if (J.lvl_of_rep) {
        lvl = __builtin_amdgcn_readfirstlane(J.lvl_of_rep[rr]);
    } else if (!perstep) {
        lvl = __builtin_amdgcn_readfirstlane(level_of(a, J.L, J.S));
        s_next = next_of(lvl);
    }
    // the level of step t; per-step schedules: those of its 64 steps, lane by lane
    WaveLevel ls, lv;
    auto level_of_step = [&](uint32_t t) {
        if (perstep) {
            ls = wave_level<CLAMP>(step_T((t & ~63u) + (uint32_t)lane), J.qcap, J.gerr);
            lv = level_at(ls, (int)(t & 63u));
        } else {
            const WaveLevel w = wave_level<CLAMP>(J.temps[lvl], J.qcap, J.gerr);
            lv = level_at(w, 0);
            lv.ga = w.ga;
            lv.gb = w.gb;
        }
    };
    level_of_step(s);
#pragma unroll
    for (int f = 0; f < F; ++f) h[f] = (int)((uint32_t)h[f] << lv.q);
    int ec = 0, dwp = 0, dwn = 0;
    auto level_consts = [&]() {
        ec = (int)(((uint32_t)min(eoff, ecap) << lv.q) + (uint32_t)lv.c0);
        dwp = (int)((uint32_t)J.wscale << lv.q);
        dwn = -dwp;
    };
    auto rescale = [&](int dq) {   // to dq more fraction bits
#pragma unroll
        for (int f = 0; f < F; ++f) h[f] = dq > 0 ? (int)((uint32_t)h[f] << dq) : h[f] >> -dq;
    };
    level_consts();

    // --- draws ---------------------------------------------------------------
    const DrawKeys<VK> keys(k0, k1);
    DrawBlock db[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q)
        db[q].init(P == 1 ? (uint32_t)(i0 >> 3) + q : (uint32_t)(lane & (8 * F - 1)), rid, k0, k1);
    // F < 8: the blocks of the P steps from t (a multiple of P), one per lane,
    // into the half of the ring that the group before it does not hold
    auto produce = [&](uint32_t t) {
        const uint32_t sub = (uint32_t)lane / (8u * F);
        ring[(t & P) / P * 64 + lane] = db[0].draw(t + sub, r0, keys);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // this lane's draws of step t: flip f is half f & 1 of word f >> 1
    auto fetch = [&](uint32_t t, uint32_t (&r)[RW]) {
        if constexpr (F >= 8) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const uint4 v = db[q].draw(t, r0, keys);
                r[4 * q] = v.x;
                r[4 * q + 1] = v.y;
                r[4 * q + 2] = v.z;
                r[4 * q + 3] = v.w;
            }
        } else {
            const uint8_t *p = reinterpret_cast<const uint8_t *>(ring) +
                               (t & (2 * P - 1)) * (128 * F) + lane * (2 * F);
            if constexpr (F == 4) {
                const uint2 v = *reinterpret_cast<const uint2 *>(p);
                r[0] = v.x;
                r[RW - 1] = v.y;
            } else if constexpr (F == 2) {
                r[0] = *reinterpret_cast<const uint32_t *>(p);
            } else {
                r[0] = *reinterpret_cast<const uint16_t *>(p);
            }
        }
    };
    auto draw16 = [&](const uint32_t (&r)[RW], int f) -> uint32_t {
        return (f & 1) ? (r[f >> 1] >> 16) : (F == 1 ? r[0] : (r[f >> 1] & 0xFFFFu));
    };
    int tv[F];
    auto bounds = [&](const uint32_t (&r)[RW]) {
#pragma unroll
        for (int f = 0; f < F; ++f) tv[f] = draw_bound<CLAMP>(draw16(r, f), lv.ga, lv.gb);
    };
    // selection draws: lane l holds that of step (s & ~63) + l
    int vsel = 0;
    // rn: the draws of this step (F >= 8), or of the next one, read ahead from
    // the ring, which holds this step's and the next one's group (F < 8)
    uint32_t rn[RW];
    if constexpr (!HELP) {
        if (P > 1) produce(s & ~(uint32_t)(P - 1));
        fetch(s, rn);
        bounds(rn);
        if (P > 1) {
            if (((s + 1) & (P - 1)) == 0) produce(s + 1);
            fetch(s + 1, rn);
        }
    }
    // HELP: this lane's bounds of step t from the ring (lanes past the last
    // block: some block's)
    const int half = HELP ? team_half_bytes(J.N) : 0;
    const uint8_t *hring = lds + 2 * RB + min(i0 >> 3, (J.N - 1) >> 3) * 16;
    auto handed = [&](uint32_t t, int (&o)[F]) {
        const uint8_t *p = hring + (t & 1u) * (2 * half);
#pragma unroll
        for (int q = 0; q < F / 4; ++q) {
            const int4 e = *reinterpret_cast<const int4 *>(p + (q & 1) * half + (q >> 1) * 16);
            o[(4 * q) % F] = e.x;
            o[(4 * q + 1) % F] = e.y;
            o[(4 * q + 2) % F] = e.z;
            o[(4 * q + 3) % F] = e.w;
        }
    };
    int prop = single ? (int)(s % (uint32_t)J.N) : 0;
    if constexpr (TEAM) {
        // records of waves the team does not have: none accepted, ever
        for (int q = NW * 64 + wr * 64 + lane; q < (NW < 4 ? 256 : 0); q += NW * 64)
            recs(0)[q] = recs(RB)[q] = Rec::make(0u, 0u, 0);
        if (wr == 0 && lane == 0) *denergy(0) = *denergy(RB) = 0;
        if (HELP) __builtin_amdgcn_s_setprio(2);
        __syncthreads();
        if constexpr (HELP) handed(s, tv);
    }

    // segments in which neither the level nor the selection draws change
    for (bool first = true; s != s1; first = false) {
        if (first || (s & 63u) == 0u)
            vsel = (int)philox(0u, (s & ~63u) + (uint32_t)lane, rid, kTagSelect, k0, k1).x;
        if (s == s_next || (perstep && (s & 63u) == 0u)) {
            // the level that opens here: its fixed point, and this step's
            // bounds once more
            const int q = lv.q;
            if (!perstep) {
                lvl = (int64_t)J.L > J.S
                          ? __builtin_amdgcn_readfirstlane(level_of((int64_t)s, J.L, J.S))
                          : lvl + 1;
                s_next = next_of(lvl);
            }
            level_of_step(s);
            if (lv.q != q) rescale(lv.q - q);
            level_consts();
            if constexpr (!HELP) {
                uint32_t rc[RW];
                if constexpr (P > 1) {
                    fetch(s, rc);
                    bounds(rc);
                } else {
                    bounds(rn);
                }
            }
        }
        const uint32_t seg = min(min(s1, s_next), (s & ~63u) + 64u);
        for (; s != seg; ++s) {
            // 1. the tests.  sgn collects the sign bits of z; undecided costs
            // are the largest z as unsigned numbers
            uint32_t sgn = 0, zmax = 0;
            int z[F];
#pragma unroll
            for (int f = F - 1; f >= 0; --f) {
                const int mx = (int)(int8_t)(nx[f >> 2] >> (8 * (f & 3)));
                uint32_t zs;
                asm("v_add3_u32 %0, %1, %2, %3" : "=v"(zs) : "v"(h[f] ^ mx), "v"(tv[f]), "s"(ec));
                z[f] = (int)zs;
                sgn = F == 1 ? zs >> 31 : __builtin_amdgcn_alignbit(sgn, zs, 31);
                zmax = max(zmax, zs);
            }
            uint32_t acc;
            asm("v_bfi_b32 %0, %1, 0, %2" : "=v"(acc) : "v"(sgn), "v"(vmask));   // ~sgn & vmask
            if (__builtin_expect(ballot(zmax > lv.zamb) != 0, 0)) {
                // rare: the definition, in double
                uint32_t rc[RW];
                if constexpr (P > 1 || HELP) {
                    fetch(s, rc);
                } else {
#pragma unroll
                    for (int q = 0; q < RW; ++q) rc[q] = rn[q];
                }
                const int eo = ec - lv.c0;
                const double T = __builtin_ldexp(perstep ? step_T(s) : J.temps[lvl], lv.q);
                double g[F];
#pragma unroll
                for (int f = 0; f < F; ++f)
                    g[f] = J.G[(uint32_t)z[f] > lv.zamb ? draw16(rc, f) : 0u];
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const int mx = (int)(int8_t)(nx[f >> 2] >> (8 * (f & 3)));
                    const int d = mx - (h[f] ^ mx) - eo;   // (1 - 2x) h - E_off
                    const bool in = (uint32_t)z[f] > lv.zamb && ((vmask >> f) & 1u);
                    acc |= (uint32_t)(in && (double)d < T * g[f]) << f;
                }
            }
            if (single) acc &= wr * 64 + lane == prop / F ? 1u << (prop % F) : 0u;

            // 2. the chosen flip: the j-th accepted one in index order.  A step
            // that accepts none runs the same instructions with ts = -1 (no
            // lane), row 0 and factor 0: the branch around them costs more
            const uint32_t v = (uint32_t)readlane(vsel, (int)(s & 63u));
            int m, ts, bit = 0, ws = 0;
            uint32_t xk = 0;
            int dEp = 0;
            int tn[F];   // HELP: the next step's bounds
            if constexpr (TEAM) {
                const int incl = incl_scan(__popc(acc));
                RecT *rec = recs(rec_o);
                rec[wr * 64 + lane] = Rec::make(acc, xb, incl);
                __syncthreads();
                // everything the step reads from LDS at once
                dEp = *denergy(RB - rec_o);
                int j;
                RecT r2;
                if constexpr (NWC <= 4) {
                    RecT r[NWC];
                    int to[NWC];   // accepted in waves 0 .. q
#pragma unroll
                    for (int q = 0; q < NWC; ++q) r[q] = rec[q * 64 + lane];
                    if constexpr (HELP) handed(s + 1, tn);
                    m = 0;
#pragma unroll
                    for (int q = 0; q < NWC; ++q) to[q] = m += Rec::incl(Rec::lane(r[q], 63));
                    j = (int)__umulhi(v, (uint32_t)m);
                    r2 = r[0];
                    int base = 0;
#pragma unroll
                    for (int q = 1; q < NWC; ++q) {
                        // (numbers: as conditions these would go through lane masks)
                        const int past = (to[q - 1] - 1 - j) >> 31;   // j >= to[q - 1]: -1
                        ws -= past;
                        base += (to[q - 1] - (q > 1 ? to[q > 1 ? q - 2 : 0] : 0)) & past;
                        r2 = past ? r[q] : r2;
                    }
                    j -= base;
                } else {
                    const int t = Rec::incl(rec[min(lane, NW - 1) * 64 + 63]);
                    if constexpr (HELP) handed(s + 1, tn);
                    const int scan = incl_scan(lane < NW ? t : 0);
                    m = readlane(scan, 63);
                    j = (int)__umulhi(v, (uint32_t)m);
                    ws = max(first_bit(ballot(scan > j)), 0);
                    j -= readlane(scan, ws) - readlane(t, ws);
                    r2 = rec[ws * 64 + lane];
                }
                ts = first_bit(ballot(Rec::incl(r2) > j));
                const RecT rs = Rec::lane(r2, ts);
                const uint32_t need = (uint32_t)(Rec::incl(rs) - j);
                bit = first_bit((uint32_t)ballot((uint32_t)__popc(Rec::acc(rs) & ge_mask) == need) &
                                Rec::acc(rs));
                xk = Rec::x(rs);
            } else if constexpr (F == 1) {
                const uint64_t mk = ballot(acc != 0);
                m = (int)__popcll(mk);
                const int j = (int)__umulhi(v, (uint32_t)m);
                ts = first_bit(ballot(mbcnt64(mk) == j) & mk);
            } else if constexpr (F == 2) {
                const uint64_t m0 = ballot((acc & 1u) != 0), m1 = ballot((acc & 2u) != 0);
                m = (int)(__popcll(m0) + __popcll(m1));
                const int j = (int)__umulhi(v, (uint32_t)m);
                const int excl = mbcnt64(m0) + mbcnt64(m1);
                // of the j-th flip's lane either flip 0 has rank j, or flip 1 has
                const uint64_t e0 = ballot(excl == j) & m0;
                const uint64_t e1 = ballot(excl + (int)(acc & 1u) == j) & m1;
                const int t0 = first_bit(e0), t1 = first_bit(e1);   // one of them is -1
                ts = max(t0, t1);
                asm("s_not_b32 %0, %1\n\ts_lshr_b32 %0, %0, 31" : "=s"(bit) : "s"(t1) : "scc");
            } else {
                const int incl = incl_scan(__popc(acc));
                m = readlane(incl, 63);
                const int j = (int)__umulhi(v, (uint32_t)m);
                ts = first_bit(ballot(incl > j));
                const uint32_t rs = (uint32_t)readlane((int)acc, ts);
                // the set bit with incl - j set bits at or above it
                const uint32_t need = (uint32_t)(readlane(incl, ts) - j);
                bit = first_bit((uint32_t)ballot((uint32_t)__popc(rs & ge_mask) == need) & rs);
            }
            // (a team without an accepted flip has some ws)
            const int k = TEAM ? (m > 0 ? (ws * 64 + ts) * F + bit : 0) : max(ts * F + bit, 0);
            // 3. row k of W, the step's only bulk traffic
            typedef __attribute__((address_space(3))) const RowV LdsRowV;
            typedef __attribute__((address_space(1))) const RowV GlobalRowV;
            RowV raw;
            if constexpr (WLDS)
                raw = *(LdsRowV *)(reinterpret_cast<const WT *>(wl) + k * ld + col0);
            else
                raw = *(GlobalRowV *)(reinterpret_cast<const WT *>(J.W) +
                                      (size_t)(uint32_t)(k * ld) + col0);
            int dE = 0, dw, hk = 0;
            if constexpr (!TEAM) {
                xk = (uint32_t)readlane((int)xb, ts);
                hk = readlane(field_at<F>(h, bit), ts) >> lv.q;
            }
            // (1 - 2 x_k) h_k, the rows' factor and the count, none of them when
            // m = 0 (written out: the compiler carries conditions of scalars
            // through 64-bit masks)
#define DAPT_FLIP(BIT, ...)                                                            \
    asm("s_sub_i32 %0, 0, %3\n\t"                                                      \
        "s_bitcmp1_b32 %4, " BIT "\n\t"                                                \
        "s_cselect_b32 %0, %0, %3\n\t"                                                 \
        "s_cselect_b32 %1, %6, %5\n\t"                                                 \
        "s_cmp_gt_i32 %7, 0\n\t"                                                       \
        "s_cselect_b32 %0, %0, 0\n\t"                                                  \
        "s_cselect_b32 %1, %1, 0\n\t"                                                  \
        "s_addc_u32 %2, %2, 0"                                                         \
        : "=&s"(dE), "=&s"(dw), "+s"(nacc)                                             \
        : "s"(hk), "s"(xk), "s"(dwp), "s"(dwn), "s"(m) __VA_ARGS__                     \
        : "scc")
            if constexpr (F == 1) DAPT_FLIP("0", );
            else DAPT_FLIP("%8", , "s"(bit));
#undef DAPT_FLIP
            auto flip = [&]() __attribute__((always_inline)) {
                const uint64_t mb = 0xFFull << (8 * (bit & 7));
                xb ^= 1u << bit;
                if constexpr (NX <= 2) {
                    nx[0] ^= (uint32_t)mb;
                    if (NX > 1) nx[NX - 1] ^= (uint32_t)(mb >> 32);
                } else {
                    const uint64_t lo = bit < 8 ? mb : 0ull, hi = bit < 8 ? 0ull : mb;
                    nx[0] ^= (uint32_t)lo;
                    nx[1] ^= (uint32_t)(lo >> 32);
                    nx[NX - 2] ^= (uint32_t)hi;
                    nx[NX - 1] ^= (uint32_t)(hi >> 32);
                }
            };
            auto add_energy = [&](int d) __attribute__((always_inline)) {
                gap += (int64_t)d;
                int gap_hi = (int)(gap >> 32);
                asm("" : "+s"(gap_hi));   // (tested as a scalar)
                if (__builtin_expect(gap_hi < 0, 0)) {
                    bE += gap;
                    gap = 0;
                    bxb = xb;
                }
            };
            if constexpr (TEAM) {
                // the last step's energy change, its state not yet flipped
                add_energy(__builtin_amdgcn_readfirstlane(dEp));
                int *dEw = denergy(rec_o);
                if (ws == wr) {
                    hk = readlane(field_at<F>(h, bit), ts) >> lv.q;
                    if (lane == ts) {
                        *dEw = ((xk >> (bit & 31)) & 1u) ? -hk : hk;
                        flip();
                    }
                }
                rec_o = RB - rec_o;
            } else {
                if (lane == ts) flip();
                add_energy(dE);
            }
            const int eo = eoff;
            eoff = 0;
            ec = lv.c0;
            if (__builtin_expect(m == 0, 0)) {
                asm volatile("");   // (a branch: the selects cost more)
                if constexpr (TEAM) {
                    if (wr == 0 && lane == 0) *denergy(RB - rec_o) = 0;
                }
                // min(E_off + inc, 2^30) without leaving int32 (both in [0, 2^30])
                eoff = min(eo, inc_cap) + inc;
                ec = (int)(((uint32_t)min(eoff, ecap) << lv.q) + (uint32_t)lv.c0);
            }

            // 4. while the row is in flight: the draws and bounds of step s + 1
            int dq = 0;
            if constexpr (FEAT) {
                if (perstep) {
                    // its temperature; the fields follow after this step's
                    // update (past the 64 steps at hand: done again above)
                    const int q = lv.q;
                    lv = level_at(ls, (int)((s + 1) & 63u));
                    dq = lv.q - q;
                }
                if (single) prop = prop + 1 == J.N ? 0 : prop + 1;
            }
            if constexpr (HELP) {
#pragma unroll
                for (int f = 0; f < F; ++f) tv[f] = tn[f];
            } else if constexpr (P == 1) {
                fetch(s + 1, rn);
                bounds(rn);
            } else {
                bounds(rn);
                if (((s + 2) & (P - 1)) == 0) produce(s + 2);
                fetch(s + 2, rn);
            }

            // 5. every field moves by +-W row k
            if constexpr (sizeof(WT) == 2 && F >= 2) {
                update_i16<WT, F>(raw, dw, h);
            } else if constexpr (sizeof(WT) == 2) {
                asm("v_mad_i32_i16 %0, %1, %2, %0" : "+v"(h[0]) : "v"((int)raw[0]), "s"(dw));
            } else if (w24) {
#pragma unroll
                for (int f = 0; f < F; ++f)
                    asm("v_mad_i32_i24 %0, %1, %2, %0" : "+v"(h[f]) : "v"((int)raw[f]), "s"(dw));
            } else {
#pragma unroll
                for (int f = 0; f < F; ++f)
                    h[f] = (int)((uint32_t)h[f] + (uint32_t)raw[f] * (uint32_t)dw);
            }
            if constexpr (FEAT) {
                if (perstep) {
                    if (dq) rescale(dq);
                    level_consts();
                }
            }
        }
    }

    if constexpr (TEAM) {
        // the last step's energy change
        __syncthreads();
        const int d = __builtin_amdgcn_readfirstlane(*denergy(RB - rec_o));
        gap += (int64_t)d;
        if (gap < 0) {
            bE += gap;
            gap = 0;
            bxb = xb;
        }
    }

    // --- state back to HBM -----------------------------------------------------
    if (lane_has) {
        IV hv;
        BV xv, bv;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            hv[f] = h[f] >> lv.q;
            xv[f] = (uint8_t)((xb >> f) & 1u);
            bv[f] = (uint8_t)((bxb >> f) & 1u);
        }
        *reinterpret_cast<IV *>(J.h + base) = hv;
        *reinterpret_cast<BV *>(J.x + base) = xv;
        *reinterpret_cast<BV *>(J.bx + base) = bv;
    }
    if (wr == 0 && lane == 0) {
        // (where another wave's sweep reads it: pt_sweep)
        __hip_atomic_store(&J.E[rr], bE + gap, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        J.bE[rr] = bE;
        J.eoff[rr] = eoff;
        J.nacc[rr] += nacc;
    }
    if constexpr (!FEAT) {
        if (J.pt.M > 0 && wr == 0) pt_sweep(J, rr, pt_round);
    }
}

// One wave per replica, the J.RPW replicas from rr0 per workgroup (they share W in
// LDS and nothing else).  LDS: [W][2][64] Philox blocks per wave (F < 8).
template <typename WT, int F, bool WLDS, bool CLAMP, bool FEAT, bool VK = false>
__device__ __forceinline__ void wave_block(const JobDesc &J, int rr0, uint8_t *smem) {
    int w_bytes = 0;
    if constexpr (WLDS) {
        const int n16 = J.N * J.ld * (int)sizeof(WT) / 16;
        const uint4 *src = reinterpret_cast<const uint4 *>(J.W);
        uint4 *dst = reinterpret_cast<uint4 *>(smem);
        for (int q = threadIdx.x; q < n16; q += blockDim.x) dst[q] = src[q];
        __syncthreads();
        w_bytes = n16 * 16;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave >= J.RPW || rr0 + wave >= J.R) return;
    wave_run<WT, F, 1, false, WLDS, CLAMP, FEAT, VK>(J, rr0 + wave, smem,
                                                     smem + w_bytes + (F < 8 ? wave * 2048 : 0), 0);
}

// A team of J.NW waves and J.NH random-number waves for replica rr; HB: Philox
// blocks per lane of the latter (0: none of them).
template <typename WT, int F, int NWC, int HB, bool CLAMP, bool FEAT>
__device__ __forceinline__ void team_block(const JobDesc &J, int rr, uint8_t *smem) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave < J.NW) {
        wave_run<WT, F, NWC, (HB > 0), false, CLAMP, FEAT>(J, rr, smem, smem, wave);
    } else if constexpr (HB > 0) {
        // (its lanes' blocks past N land in the padding of the ring)
        if (wave < J.NW + J.NH)
            team_draws<HB, CLAMP, FEAT>(J, rr, smem + 2 * team_rec_bytes<F>(J.NW), wave - J.NW);
    }
}

template <typename WT, int F, bool WLDS, bool CLAMP, bool FEAT>
__global__ __launch_bounds__(1024) void k_wave(JobDesc J) {
    extern __shared__ __align__(16) uint8_t smem[];
    wave_block<WT, F, WLDS, CLAMP, FEAT, F == 16 && sizeof(WT) == 2>(J, blockIdx.x * J.RPW, smem);
}

template <typename WT, int F, int NWC, int HB, bool CLAMP, bool FEAT>
__global__ __launch_bounds__(NWC > 4 ? 1024 : 512) void k_team(JobDesc J) {
    extern __shared__ __align__(16) uint8_t smem[];
    team_block<WT, F, NWC, HB, CLAMP, FEAT>(J, blockIdx.x, smem);
}

// Replicas of many jobs of one coupling type in one launch: every workgroup runs
// the item of its index in its job's shape (mix_shape: at most 8 waves, the
// waves past a shape's end at once).  The items come longest first, so the
// launch's tail is short.
template <typename WT, bool CLAMP, bool FEAT>
__global__ __launch_bounds__(512) void k_mix(const JobDesc *__restrict__ jobs,
                                             const BatchItem *__restrict__ items) {
    extern __shared__ __align__(16) uint8_t smem[];
    const BatchItem it = items[blockIdx.x];
    const JobDesc J = jobs[__builtin_amdgcn_readfirstlane(it.job)];
    const int r0 = __builtin_amdgcn_readfirstlane(it.r0);
    if (J.NW == 1) {
        switch (J.F) {
            case 1:
                if (J.w_lds) wave_block<WT, 1, true, CLAMP, FEAT>(J, r0, smem);
                else wave_block<WT, 1, false, CLAMP, FEAT>(J, r0, smem);
                break;
            case 2:
                if (J.w_lds) wave_block<WT, 2, true, CLAMP, FEAT>(J, r0, smem);
                else wave_block<WT, 2, false, CLAMP, FEAT>(J, r0, smem);
                break;
            case 4: wave_block<WT, 4, false, CLAMP, FEAT>(J, r0, smem); break;
            case 8: wave_block<WT, 8, false, CLAMP, FEAT>(J, r0, smem); break;
            default: wave_block<WT, 16, false, CLAMP, FEAT>(J, r0, smem); break;
        }
    } else if (J.F == 8) {
        if (J.NW <= 2) team_block<WT, 8, 2, 2, CLAMP, FEAT>(J, r0, smem);
        else team_block<WT, 8, 4, 2, CLAMP, FEAT>(J, r0, smem);
    } else if (J.NW <= 2) {
        team_block<WT, 16, 2, 0, CLAMP, FEAT>(J, r0, smem);
    } else if (J.NH > 0) {
        team_block<WT, 16, 4, 2, CLAMP, FEAT>(J, r0, smem);
    } else {
        team_block<WT, 16, 16, 0, CLAMP, FEAT>(J, r0, smem);
    }
}

// Launches KERNEL<.., CLAMP, FEAT> as the job needs.
#define DAPT_LAUNCH(KERNEL, ...)                                                                 \
    do {                                                                                         \
        const hipStream_t st = reinterpret_cast<hipStream_t>(stream);                            \
        if (J.stepT || J.single)                                                                 \
            hipLaunchKernelGGL((KERNEL<__VA_ARGS__, true, true>), dim3(blocks), dim3(threads),   \
                               lds, st, J);                                                      \
        else if (J.wclamp)                                                                       \
            hipLaunchKernelGGL((KERNEL<__VA_ARGS__, true, false>), dim3(blocks), dim3(threads),  \
                               lds, st, J);                                                      \
        else                                                                                     \
            hipLaunchKernelGGL((KERNEL<__VA_ARGS__, false, false>), dim3(blocks), dim3(threads), \
                               lds, st, J);                                                      \
        return (int)hipGetLastError();                                                           \
    } while (0)

}  // namespace

// (defined here, compiled for one coupling type and team size per part of this file)
template <typename WT>
int launch_wave_w(const JobDesc &J, int F, int blocks, int threads, size_t lds, void *stream) {
    // (the forms that wave_shape chooses: W in LDS wherever it fits there, which it
    // does up to 128 variables, and past 256 for int8 alone)
    if (J.w_lds) {
        if constexpr (sizeof(WT) == 1)
            if (F == 8) DAPT_LAUNCH(k_wave, WT, 8, true);
        switch (F) {
            case 1: DAPT_LAUNCH(k_wave, WT, 1, true);
            case 2: DAPT_LAUNCH(k_wave, WT, 2, true);
            case 4: DAPT_LAUNCH(k_wave, WT, 4, true);
            default: return (int)hipErrorInvalidValue;
        }
    }
    if constexpr (sizeof(WT) == 4)
        if (F == 4) DAPT_LAUNCH(k_wave, WT, 4, false);
    switch (F) {
        case 8: DAPT_LAUNCH(k_wave, WT, 8, false);
        case 16: DAPT_LAUNCH(k_wave, WT, 16, false);
        default: return (int)hipErrorInvalidValue;
    }
}

template <typename WT>
int launch_team_w(const JobDesc &J, int F, int blocks, int threads, size_t lds, void *stream) {
    const int key = F * 1000 + (J.NW <= 2 ? 2 : J.NW <= 4 ? 4 : 16) * 10 +
                    (J.NH == 0 ? 0 : J.NH * 512 >= J.N ? 1 : 2);
    switch (key) {   // (those that wave_shape chooses)
        case 8021: DAPT_LAUNCH(k_team, WT, 8, 2, 1);
        case 8022: DAPT_LAUNCH(k_team, WT, 8, 2, 2);
        case 8041: DAPT_LAUNCH(k_team, WT, 8, 4, 1);
        case 8042: DAPT_LAUNCH(k_team, WT, 8, 4, 2);
        case 8162: DAPT_LAUNCH(k_team, WT, 8, 16, 2);
        case 16040: DAPT_LAUNCH(k_team, WT, 16, 4, 0);
        case 16042: DAPT_LAUNCH(k_team, WT, 16, 4, 2);
        case 16160: DAPT_LAUNCH(k_team, WT, 16, 16, 0);
        case 16162: DAPT_LAUNCH(k_team, WT, 16, 16, 2);
        case 16020: DAPT_LAUNCH(k_team, WT, 16, 2, 0);
        default: return (int)hipErrorInvalidValue;
    }
}
#undef DAPT_LAUNCH

template <typename WT>
int launch_mix_w(const JobDesc *jobs, const BatchItem *items, int mode, int blocks, size_t lds,
                 void *stream) {
    const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    switch (mode) {
        case 0:
            hipLaunchKernelGGL((k_mix<WT, false, false>), dim3(blocks), dim3(512), lds, st, jobs, items);
            break;
        case 1:
            hipLaunchKernelGGL((k_mix<WT, true, false>), dim3(blocks), dim3(512), lds, st, jobs, items);
            break;
        default:
            hipLaunchKernelGGL((k_mix<WT, true, true>), dim3(blocks), dim3(512), lds, st, jobs, items);
            break;
    }
    return (int)hipGetLastError();
}

#if DAPT_PART == 1
template int launch_wave_w<int8_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 2
template int launch_wave_w<int16_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 3
template int launch_wave_w<int32_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 4
template int launch_team_w<int8_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 5
template int launch_team_w<int16_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 6
template int launch_team_w<int32_t>(const JobDesc &, int, int, int, size_t, void *);
#elif DAPT_PART == 7
template int launch_mix_w<int8_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);
#elif DAPT_PART == 8
template int launch_mix_w<int16_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);
#elif DAPT_PART == 9
template int launch_mix_w<int32_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);
#endif

#if DAPT_PART == 0
extern template int launch_wave_w<int8_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_wave_w<int16_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_wave_w<int32_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_team_w<int8_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_team_w<int16_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_team_w<int32_t>(const JobDesc &, int, int, int, size_t, void *);
extern template int launch_mix_w<int8_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);
extern template int launch_mix_w<int16_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);
extern template int launch_mix_w<int32_t>(const JobDesc *, const BatchItem *, int, int, size_t, void *);

int launch_mix(const JobDesc *jobs, const BatchItem *items, int dtype, int mode, int blocks,
               size_t lds, void *stream) {
    if (blocks < 1 || mode < 0 || mode > 2) return (int)hipErrorInvalidValue;
    switch (dtype) {
        case 1: return launch_mix_w<int8_t>(jobs, items, mode, blocks, lds, stream);
        case 2: return launch_mix_w<int16_t>(jobs, items, mode, blocks, lds, stream);
        case 4: return launch_mix_w<int32_t>(jobs, items, mode, blocks, lds, stream);
        default: return (int)hipErrorInvalidValue;
    }
}

size_t wave_lds_bytes(int F, int N, int NW, int NH, int RPW, int64_t w_lds_bytes) {
    if (NW > 1)
        return 2 * (size_t)(F > 8 ? team_rec_bytes<16>(NW) : team_rec_bytes<8>(NW)) +
               (NH > 0 ? 4 * (size_t)team_half_bytes(N) : 0);
    return (size_t)w_lds_bytes + (F < 8 ? (size_t)RPW * 2048 : 0);
}

int launch_wave(const JobDesc &J, int F, int blocks, int threads, size_t lds, void *stream) {
    // a replica's waves hold 64 F variables each; everything the kernel indexes
    // is sized by these
    const bool team = J.NW > 1;
    if (job_range_error(J) != nullptr || J.N > 64 * F * J.NW || !J.G || (!J.temps && !J.stepT) ||
        threads != 64 * (J.NW + J.NH) * J.RPW || (int64_t)blocks * J.RPW < J.R ||
        lds < wave_lds_bytes(F, J.N, J.NW, J.NH, J.RPW, J.w_lds ? (int64_t)J.N * J.ld * J.dtype : 0))
        return (int)hipErrorInvalidValue;
    if (team ? J.RPW != 1 || J.w_lds || blocks != J.R || threads > (J.NW > 4 ? 1024 : 512) ||
                   (J.NH > 0 && J.N > 1024 * J.NH)
             : J.NH != 0)
        return (int)hipErrorInvalidValue;
    switch (J.dtype) {
        case 1:
            return team ? launch_team_w<int8_t>(J, F, blocks, threads, lds, stream)
                        : launch_wave_w<int8_t>(J, F, blocks, threads, lds, stream);
        case 2:
            return team ? launch_team_w<int16_t>(J, F, blocks, threads, lds, stream)
                        : launch_wave_w<int16_t>(J, F, blocks, threads, lds, stream);
        case 4:
            return team ? launch_team_w<int32_t>(J, F, blocks, threads, lds, stream)
                        : launch_wave_w<int32_t>(J, F, blocks, threads, lds, stream);
        default: return (int)hipErrorInvalidValue;
    }
}

// Largest |log2 as the device evaluates it - log2| over the arguments u + 1/2
// of all draws: G[u] = -ln U_u gives the latter as 16 - G[u] / ln 2.
__global__ __launch_bounds__(256) void k_log_error(const double *__restrict__ G, float *out) {
    __shared__ float part[256];
    float e = 0.0f;
    for (int u = threadIdx.x; u < 65536; u += 256) {
        const float lg = __builtin_amdgcn_logf((float)u + 0.5f);
        e = fmaxf(e, (float)fabs((double)lg - (16.0 - G[u] / kLn2)));
    }
    part[threadIdx.x] = e;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) part[threadIdx.x] = fmaxf(part[threadIdx.x], part[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = part[0];
}

int launch_log_error(const double *G, float *out, void *stream) {
    hipLaunchKernelGGL(k_log_error, dim3(1), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), G,
                       out);
    return (int)hipGetLastError();
}
#endif  // DAPT_PART == 0

}  // namespace dapt
