// da_fields.hip -- local fields H = X W^T + b and energies E = x^T Q x of many
// states on the matrix cores, for every coupling type.
//
// X holds 0/1 bytes, so the product is exact on v_mfma_i32_32x32x32_i8 for any
// integer couplings once these are cut into byte planes:
//   w = sum_p 256^p d_p,   d_top signed, the lower digits unsigned.
// The unsigned digits enter the matrix cores as d - 128 (one xor), and 128
// times the number of set bits of the state is added back per plane.  Every
// plane's sum stays below 2^20 (N <= 8192); the planes are put together
// modulo 2^32, which is exact because the field itself fits int32.
// int8 couplings have one plane, int16 two, int32 four, or three where every
// coupling is known to lie below 2^23.
//
// Two forms: one wave per 32 x 32 tile reading its operands straight from
// memory (small products, where latency and the number of waves count), and
// 128-row workgroup tiles staged through LDS (large ones).  Both end either by
// storing the fields or, for energies, by adding
//   2 E = sum_i x_i ((W x)_i + 2 b_i)
// over the tile's columns while the fields are still in registers, so energies
// never write or read the [R][ld] fields.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "da_internal.h"

namespace dapt {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int perm(int hi, int lo, uint32_t sel) {
    return (int)__builtin_amdgcn_perm((uint32_t)hi, (uint32_t)lo, sel);
}

constexpr int kUnsign = (int)0x80808080u;   // unsigned digit -> digit - 128, bytewise

// 16 consecutive couplings as P planes of 16 bytes.
template <int P>
__device__ __forceinline__ void load_planes(const int8_t *p, v4i (&out)[P]) {
    out[0] = *reinterpret_cast<const v4i *>(p);
}

template <int P>
__device__ __forceinline__ void load_planes(const int16_t *p, v4i (&out)[P]) {
    const v4i a = reinterpret_cast<const v4i *>(p)[0], c = reinterpret_cast<const v4i *>(p)[1];
    const int d[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        out[0][q] = perm(d[2 * q + 1], d[2 * q], 0x06040200u) ^ kUnsign;
        out[1][q] = perm(d[2 * q + 1], d[2 * q], 0x07050301u);
    }
}

template <int P>
__device__ __forceinline__ void load_planes(const int32_t *p, v4i (&out)[P]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4i d = reinterpret_cast<const v4i *>(p)[q];
        const int a0 = perm(d.y, d.x, 0x05010400u), a2 = perm(d.y, d.x, 0x07030602u);
        const int c0 = perm(d.w, d.z, 0x05010400u), c2 = perm(d.w, d.z, 0x07030602u);
        out[0][q] = perm(c0, a0, 0x05040100u) ^ kUnsign;
        out[1][q] = perm(c0, a0, 0x07060302u) ^ kUnsign;
        out[2][q] = perm(c2, a2, 0x05040100u) ^ (P > 3 ? kUnsign : 0);
        if constexpr (P > 3) out[3][q] = perm(c2, a2, 0x07060302u);
    }
}

// What the - 128 of the lower planes takes away per set bit of the state.
template <int P>
constexpr int plane_fix() {
    int c = 0;
    for (int p = 0; p + 1 < P; ++p) c += 128 << (8 * p);
    return c;
}

// Bytes nonzero -> 1.
__device__ __forceinline__ int nonzero_bytes(int v) {
    const uint32_t x = (uint32_t)v;
    return (int)(((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) >> 7) & 0x01010101u);
}

// 16 states' bytes of row r from column k on.  RAW: caller's rows, N bytes
// apart at any alignment, any nonzero byte a one; bytes past column N belong to
// the next row and meet zero couplings, and nothing is read past the last
// state.  Else: rows of 0/1 bytes, ld apart.
template <bool RAW>
__device__ __forceinline__ v4i load_x(const uint8_t *X, int64_t total, int r, int k, int N,
                                      int ld) {
    if constexpr (!RAW) {
        return *reinterpret_cast<const v4i *>(X + (size_t)r * ld + k);
    } else {
        const int64_t off = (int64_t)r * N + k;
        v4i v = {0, 0, 0, 0};
        if (off + 16 <= total) {
            __builtin_memcpy(&v, X + off, 16);
        } else {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const uint32_t byte = off + q < total ? X[off + q] : 0u;
                v[q >> 2] |= (int)(byte << (8 * (q & 3)));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = nonzero_bytes(v[q]);
        return v;
    }
}

__device__ __forceinline__ int count_bits(v4i a, int c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_sdot4(a[q], 0x01010101, c, false);
    return c;
}

// Sum of s over the 32 lanes of each half wave, valid in lanes 31 and 63.
// |s| < 2^44: added as its low 24 bits and the rest, each of which stays in
// int32 over 32 lanes (row shifts within 16 lanes, then the broadcast of lane 15).
__device__ __forceinline__ int64_t half_wave_sum(int64_t s) {
    int lo = (int)(s & 0xFFFFFF), hi = (int)(s >> 24);
#define DAPT_DPP_ADD(ctrl, rows)                                                     \
    lo += __builtin_amdgcn_update_dpp(0, lo, ctrl, rows, 0xf, false);                \
    hi += __builtin_amdgcn_update_dpp(0, hi, ctrl, rows, 0xf, false);
    DAPT_DPP_ADD(0x111, 0xf)   // row_shr:1
    DAPT_DPP_ADD(0x112, 0xf)   // row_shr:2
    DAPT_DPP_ADD(0x114, 0xf)   // row_shr:4
    DAPT_DPP_ADD(0x118, 0xf)   // row_shr:8
    DAPT_DPP_ADD(0x142, 0xa)   // row_bcast:15 into rows 1 and 3
#undef DAPT_DPP_ADD
    return ((int64_t)hi << 24) + (int64_t)lo;
}

struct FieldArgs {
    const uint8_t *X;
    int64_t x_total;       // bytes of X (RAW)
    const void *W;
    const int32_t *b;
    int32_t *H;            // fields [R][ld], or null
    int64_t *E;            // energies [R] (one column split), or
    int64_t *part;         // [splits][R] partial sums of 2 E
    int32_t R, N, ld, wscale;
    int32_t kstep;         // columns of the reduction per split (a multiple of 64)
};

// One wave per 32 (states) x 32 (variables) tile; a workgroup's four waves
// take neighbouring column tiles of one row tile, and step on by the grid.
// The operands of the next 64 columns of the reduction are on their way while
// this 64 are multiplied.  Energies may split the reduction too (grid z): 2 E is
// additive over it.
template <typename WT, int P, bool ENERGY>
__global__ __launch_bounds__(256) void k_fields_wave(FieldArgs A) {
    __shared__ int64_t red[4][32];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r0 = blockIdx.x * 32;
    const int row = lane & 31, kh = (lane >> 5) * 16;
    const int ra = min(r0 + row, A.R - 1);
    const int ld = A.ld;
    const int kb = blockIdx.z * A.kstep, ke = min(kb + A.kstep, ld);
    int64_t es[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) es[v] = 0;
    for (int ti = blockIdx.y * 4 + wave; ti < ld / 32; ti += gridDim.y * 4) {
        const int c0 = ti * 32;
        const WT *pb = reinterpret_cast<const WT *>(A.W) + (size_t)(c0 + row) * ld + kh;
        v16i acc[P];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[p][v] = 0;
        int cnt = 0;
        v4i a[2], bb[2][P];
        auto fetch = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                a[q] = load_x<ENERGY>(A.X, A.x_total, ra, kk + 32 * q + kh, A.N, ld);
                load_planes<P>(pb + kk + 32 * q, bb[q]);
            }
        };
        fetch(kb);
        for (int kk = kb; kk < ke; kk += 64) {
            v4i ac[2], bc[2][P];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                ac[q] = a[q];
#pragma unroll
                for (int p = 0; p < P; ++p) bc[q][p] = bb[q][p];
            }
            if (kk + 64 < ke) fetch(kk + 64);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (P > 1) cnt = count_bits(ac[q], cnt);
#pragma unroll
                for (int p = 0; p < P; ++p)
                    acc[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ac[q], bc[q][p], acc[p], 0, 0,
                                                                   0);
            }
        }
        if (P > 1) cnt += __shfl_xor(cnt, 32);   // the two k halves of a row
        const int col = c0 + (lane & 31);
        const int bcol = blockIdx.z == 0 ? A.b[col] : 0;
        // this column's bits of the states, all loads in flight at once (read
        // in bounds whatever the tile, then masked)
        uint8_t xv[16] = {};
        if constexpr (ENERGY) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = min(r0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), A.R - 1);
                xv[v] = A.X[(int64_t)r * A.N + min(col, A.N - 1)];
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rl = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            const int r = r0 + rl;
            uint32_t h = (uint32_t)acc[P - 1][v];
#pragma unroll
            for (int p = P - 2; p >= 0; --p) h = h * 256u + (uint32_t)acc[p][v];
            if (P > 1) h += (uint32_t)(plane_fix<P>()) * (uint32_t)__shfl(cnt, rl);
            h *= (uint32_t)A.wscale;
            if constexpr (ENERGY) {
                const bool on = xv[v] != 0 && r < A.R && col < A.N;
                es[v] += on ? (int64_t)(int32_t)h + 2 * (int64_t)bcol : 0;
            } else {
                if (r < A.R) A.H[(size_t)r * ld + col] = (int32_t)(h + (uint32_t)bcol);
            }
        }
    }
    if constexpr (ENERGY) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t s = half_wave_sum(es[v]);
            if ((lane & 31) == 31) red[wave][8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)] = s;
        }
        __syncthreads();
        const int r = r0 + (int)threadIdx.x;
        if (threadIdx.x < 32 && r < A.R) {
            const int64_t s = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] +
                              red[3][threadIdx.x];
            if (gridDim.y * gridDim.z == 1) A.E[r] = s / 2;
            else A.part[(size_t)(blockIdx.z * gridDim.y + blockIdx.y) * A.R + r] = s;
        }
    }
}

// 2000 states, N = 3000, int16: 70 us (1.0 int8 POP/s), with the padding pass and
// the sums 82 us; one row of W added per set bit (the first form for 16- and
// 32-bit couplings) took 6860 us, a reduction tile of 64 columns 96 us, and the
// states' bits read one by one in the sums 85 us.
//
// 128 states x BN variables per workgroup, four waves of 64 x BN/2 (MFMA tiles
// of 32 x 32, one accumulator per plane); the reduction advances 128 at a time
// through LDS, the next tile's operands fetched into registers meanwhile: the
// loads' latency (operands beyond one XCD's L2) bounds a tile, so a tile is as
// deep as registers and two workgroups per CU allow.  Eight lanes read 128
// consecutive bytes of a row, couplings are cut into planes on the way into
// LDS, and LDS rows are padded by 16 bytes, which spreads the 16-byte fragment
// reads of consecutive rows over all banks.  BN = 128 for one or two planes, 64
// for more: 64 to 128 accumulator registers.
constexpr int kFM = 128, kFK = 128, kFRow = kFK + 16;


template <typename WT, int P, bool ENERGY>
__global__ __launch_bounds__(256, 2) void k_fields_tiled(FieldArgs A) {
    constexpr int BN = P <= 2 ? 128 : 64;
    constexpr int TN = BN / 64;                    // column tiles per wave
    constexpr int QA = kFM / 32, QB = BN / 32;     // 16-byte pieces per thread
    __shared__ __align__(16) int8_t As[kFM * kFRow];
    __shared__ __align__(16) int8_t Bs[P][BN * kFRow];
    __shared__ int cnt_s[kFM];
    __shared__ int64_t red[2][kFM];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int ld = A.ld;
    // workgroups go to the 8 XCDs in turn: each XCD takes a contiguous run of
    // tiles, rows fastest, so that its L2 holds a few columns' couplings
    const int gx = (A.R + kFM - 1) / kFM;
    const int n = gridDim.x, xcd = blockIdx.x & 7;
    const int id = xcd * (n >> 3) + min(xcd, n & 7) + (int)(blockIdx.x >> 3);
    const int r0 = (id % gx) * kFM, c0 = (id / gx) * BN;
    // staging: thread t copies bytes 16 (t & 7) .. of state rows t/8 + 32 q and
    // the couplings of the same columns of coupling rows t/8 + 32 q
    const int srow = t >> 3, sk = (t & 7) * 16;
    const WT *gb[QB];
    int ar[QA];
#pragma unroll
    for (int q = 0; q < QA; ++q) ar[q] = min(r0 + srow + 32 * q, A.R - 1);
#pragma unroll
    for (int q = 0; q < QB; ++q)
        gb[q] = reinterpret_cast<const WT *>(A.W) + (size_t)min(c0 + srow + 32 * q, ld - 1) * ld +
                sk;
    v16i acc[P][2][TN];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[p][i][j][v] = 0;
    const int frow = lane & 31, fk = (lane >> 5) * 16;
    int cnt[QA] = {};
    const v4i zero = {0, 0, 0, 0};
    v4i a[QA], bp[QB][P];
    const int kb = blockIdx.z * A.kstep, ke = min(kb + A.kstep, ld);
    // (the last tile may be half a tile: nothing is read past column ke)
    auto fetch = [&](int k0) __attribute__((always_inline)) {
        const bool in = k0 + sk < ke;
#pragma unroll
        for (int q = 0; q < QA; ++q)
            a[q] = in ? load_x<false>(A.X, 0, ar[q], k0 + sk, A.N, ld) : zero;
        if (in) {
#pragma unroll
            for (int q = 0; q < QB; ++q) load_planes<P>(gb[q] + k0, bp[q]);
        }
    };
    fetch(kb);
    for (int k0 = kb; k0 < ke; k0 += kFK) {
        __syncthreads();   // the previous tile is no longer read
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            *reinterpret_cast<v4i *>(As + (srow + 32 * q) * kFRow + sk) = a[q];
            if (P > 1) cnt[q] = count_bits(a[q], cnt[q]);
        }
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int p = 0; p < P; ++p)
                *reinterpret_cast<v4i *>(&Bs[p][(srow + 32 * q) * kFRow + sk]) = bp[q][p];
        __syncthreads();
        if (k0 + kFK < ke) fetch(k0 + kFK);
        const int kn = min(kFK, ke - k0);
        for (int kc = 0; kc < kn; kc += 64) {
#pragma unroll
            for (int ks = 0; ks < 64; ks += 32) {
                v4i fa[2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    fa[i] = *reinterpret_cast<const v4i *>(
                        As + (wm * 64 + i * 32 + frow) * kFRow + kc + ks + fk);
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const v4i fb = *reinterpret_cast<const v4i *>(
                            &Bs[p][(wn * (BN / 2) + j * 32 + frow) * kFRow + kc + ks + fk]);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            acc[p][i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                                fa[i], fb, acc[p][i][j], 0, 0, 0);
                    }
            }
        }
    }
    if (P > 1) {
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            int c = cnt[q];
#pragma unroll
            for (int w = 1; w < 8; w <<= 1) c += __shfl_xor(c, w);
            if ((t & 7) == 0) cnt_s[srow + 32 * q] = c;
        }
        __syncthreads();
    }
    int bcol[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
        bcol[j] = blockIdx.z == 0 ? A.b[min(c0 + wn * (BN / 2) + j * 32 + (lane & 31), ld - 1)] : 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // these columns' bits of the states, all loads in flight at once (read
        // in bounds whatever the tile, then masked)
        uint8_t xv[TN][16] = {};
        if constexpr (ENERGY) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = r0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    const int col = c0 + wn * (BN / 2) + j * 32 + (lane & 31);
                    xv[j][v] = A.X[(size_t)min(r, A.R - 1) * ld + min(col, ld - 1)];
                }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rl = wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            const int r = r0 + rl;
            const uint32_t fix = P > 1 ? (uint32_t)plane_fix<P>() * (uint32_t)cnt_s[rl] : 0u;
            int64_t es = 0;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = c0 + wn * (BN / 2) + j * 32 + (lane & 31);
                uint32_t h = (uint32_t)acc[P - 1][i][j][v];
#pragma unroll
                for (int p = P - 2; p >= 0; --p) h = h * 256u + (uint32_t)acc[p][i][j][v];
                h = (h + fix) * (uint32_t)A.wscale;
                if constexpr (ENERGY) {
                    const bool on = xv[j][v] != 0 && r < A.R && col < ld;
                    es += on ? (int64_t)(int32_t)h + 2 * (int64_t)bcol[j] : 0;
                } else {
                    if (r < A.R && col < ld)
                        A.H[(size_t)r * ld + col] = (int32_t)(h + (uint32_t)bcol[j]);
                }
            }
            if constexpr (ENERGY) {
                es = half_wave_sum(es);
                if ((lane & 31) == 31) red[wn][rl] = es;
            }
        }
    }
    if constexpr (ENERGY) {
        __syncthreads();
        if (t < kFM && r0 + t < A.R) {
            const int64_t s = red[0][t] + red[1][t];
            const int gy = n / gx;
            if (gy * gridDim.z == 1) A.E[r0 + t] = s / 2;
            else A.part[(size_t)(blockIdx.z * gy + id / gx) * A.R + r0 + t] = s;
        }
    }
}

// Caller's states [R][N] as rows of 0/1 bytes [R][ld], zero past column N, for
// the tiled form, whose column tiles read each state many times.
__global__ __launch_bounds__(256) void k_pad_states(FieldArgs A, uint8_t *__restrict__ out) {
    const int per = A.ld / 16;
    const int64_t n = (int64_t)A.R * per;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(q / per), k = (int)(q - (int64_t)r * per) * 16;
        v4i v = {0, 0, 0, 0};
        if (k < A.N) v = load_x<true>(A.X, A.x_total, r, k, A.N, A.ld);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int left = A.N - (k + 4 * w);   // bytes of this word inside the row
            if (left < 4) v[w] &= left <= 0 ? 0 : (1 << (8 * left)) - 1;
        }
        *reinterpret_cast<v4i *>(out + q * 16) = v;
    }
}

// Adds up the partial sums: 16 states per workgroup, 16 threads each, so that
// the loads of a state's splits are in flight together.
__global__ __launch_bounds__(256) void k_energy_sum(const int64_t *__restrict__ part,
                                                    int64_t *__restrict__ E, int32_t R,
                                                    int32_t splits) {
    __shared__ int64_t red[16][16];
    const int c = threadIdx.x & 15, q0 = threadIdx.x >> 4;
    const int r = blockIdx.x * 16 + c;
    int64_t s = 0;
    if (r < R)
        for (int q = q0; q < splits; q += 16) s += part[(size_t)q * R + r];
    red[q0][c] = s;
    __syncthreads();
    if (threadIdx.x < 16 && r < R) {
        s = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) s += red[q][threadIdx.x];
        E[r] = s / 2;
    }
}

struct FieldPlan {
    bool tiled;
    int gx, gy, gz;   // row tiles, column splits, splits of the reduction
    int kstep;
};

// Which form, and how the work is split.
//
// The tiled form from 1.1 M output elements on.  Energies, us a call, wave form
// and tiled form: 1500 x 2048 int8 55 and 29, int16 103 and 47; 1000 x 1024
// int8 13 and 17, int16 18 and 19 (one 128-row tile more or less per CU does
// not pay for the padding pass there); 512 x 4096 int16 100 and 48.
//
// Fields: every column tile its own wave, the reduction whole.  Energies: the
// sums of all splits are added up by a second kernel, unless a small product
// (ld <= 256) runs unsplit in one launch; the reduction is split (at least 256
// columns each) until there is about a workgroup per CU: 16 states of N = 4096,
// int16, 60 us unsplit, 17 us split 8 ways; splitting on to three workgroups per
// CU costs 23 us, the partial sums' own work.
constexpr int64_t kTiledFrom = 1100000;

FieldPlan field_plan(int32_t R, int32_t ld, int planes, bool energy) {
    FieldPlan p;
    // enough 128-row tiles to fill the chip: the LDS-tiled form
    p.tiled = (int64_t)R * ld >= kTiledFrom;
    if (p.tiled) {
        const int bn = planes <= 2 ? 128 : 64;
        p.gx = (R + kFM - 1) / kFM;
        p.gy = (ld + bn - 1) / bn;
    } else {
        p.gx = (R + 31) / 32;
        p.gy = (ld / 32 + 3) / 4;
    }
    p.gz = 1;
    if (energy && !p.tiled && ld <= 256) p.gy = 1;
    else if (energy) {
        p.gz = std::max(1, std::min(ld / 256, 256 / (p.gx * p.gy)));
    }
    p.kstep = ((ld + p.gz - 1) / p.gz + 63) / 64 * 64;
    p.gz = (ld + p.kstep - 1) / p.kstep;
    return p;
}

// Elements of the partial sums in the energy scratch (rounded up to 256 bytes).
int64_t pad_offset(const FieldPlan &p, int32_t R) {
    const int64_t splits = (int64_t)p.gy * p.gz;
    return splits > 1 ? (splits * R + 31) / 32 * 32 : 0;
}

template <typename WT, int P, bool ENERGY>
int launch_fields_t(FieldArgs A, hipStream_t s) {
    const FieldPlan p = field_plan(A.R, A.ld, P, ENERGY);
    A.kstep = p.kstep;
    if (ENERGY && p.tiled) {
        // scratch: the partial sums, then the padded states
        uint8_t *xp = reinterpret_cast<uint8_t *>(A.part + pad_offset(p, A.R));
        const int64_t n = (int64_t)A.R * (A.ld / 16);
        hipLaunchKernelGGL(k_pad_states, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65535)),
                           dim3(256), 0, s, A, xp);
        A.X = xp;
    }
    if (p.tiled)
        hipLaunchKernelGGL((k_fields_tiled<WT, P, ENERGY>), dim3(p.gx * p.gy, 1, p.gz), dim3(256),
                           0, s, A);
    else
        hipLaunchKernelGGL((k_fields_wave<WT, P, ENERGY>), dim3(p.gx, p.gy, p.gz), dim3(256), 0, s,
                           A);
    if (ENERGY && p.gy * p.gz > 1)
        hipLaunchKernelGGL(k_energy_sum, dim3((A.R + 15) / 16), dim3(256), 0, s, A.part, A.E,
                           A.R, p.gy * p.gz);
    return (int)hipGetLastError();
}

template <bool ENERGY>
int launch_fields_any(const FieldArgs &A, int dtype, int planes, hipStream_t s) {
    if (A.R < 1 || A.N < 1 || A.N > kMaxN || A.ld < A.N || (A.ld & 63) != 0)
        return (int)hipErrorInvalidValue;
    switch (dtype) {
        case 1: return launch_fields_t<int8_t, 1, ENERGY>(A, s);
        case 2: return launch_fields_t<int16_t, 2, ENERGY>(A, s);
        case 4:
            return planes == 3 ? launch_fields_t<int32_t, 3, ENERGY>(A, s)
                               : launch_fields_t<int32_t, 4, ENERGY>(A, s);
        default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace

int coupling_planes(int dtype, int64_t hbound, int32_t wscale) {
    if (dtype < 4) return dtype;
    const int64_t g = wscale < 0 ? -(int64_t)wscale : (int64_t)wscale;
    return g > 0 && hbound / g < (int64_t(1) << 23) - 1 ? 3 : 4;
}

int launch_fields(const JobDesc &J, int planes, const uint8_t *X, int32_t R, int32_t *H,
                  void *stream) {
    const FieldArgs A{X, 0, J.W, J.b, H, nullptr, nullptr, R, J.N, J.ld, J.wscale, J.ld};
    return launch_fields_any<false>(A, J.dtype, planes, reinterpret_cast<hipStream_t>(stream));
}

int64_t energy_scratch_elems(const JobDesc &J, int planes, int32_t count) {
    const FieldPlan p = field_plan(count, J.ld, planes, true);
    return pad_offset(p, count) + (p.tiled ? ((int64_t)count * J.ld + 7) / 8 : 0);
}

int launch_energy(const JobDesc &J, int planes, const uint8_t *x, int32_t count, int64_t *E,
                  int64_t *scratch, void *stream) {
    const FieldArgs A{x, (int64_t)count * J.N, J.W, J.b, nullptr, E, scratch,
                      count, J.N, J.ld, J.wscale, J.ld};
    return launch_fields_any<true>(A, J.dtype, planes, reinterpret_cast<hipStream_t>(stream));
}

}  // namespace dapt
