// da_prepare.hip -- an instance's device image from its QUBO matrix.
//
// W_ij = Q_ij + Q_ji off the diagonal and b_i = Q_ii (Sec. V of
// arXiv:1806.08815), W divided by the common factor of all couplings and padded
// to rows of ld (da_internal.h).  Both passes read each pair of tiles (I, J) and
// (J, I) of Q once, the second through LDS for its transpose: bound by reading Q,
// N = 2048 (16 MB) takes 25 us where the host took 21 ms; what is left of
// da_create is the upload of Q.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "da_internal.h"

namespace dapt {

namespace {

constexpr int kTile = 64;

// |w| of a pair is at most 2^32: remainders in 32 bits wherever both fit
__device__ uint64_t gcd_step(uint64_t g, uint64_t w) {
    while (w) {
        const uint64_t r = ((g | w) >> 32) ? g % w : (uint64_t)((uint32_t)g % (uint32_t)w);
        g = w;
        w = r;
    }
    return g;
}

// t[i][j] = Q[J + i][I + j]^T, that is Q[(J + j'), (I + i')] read along rows
__device__ void load_transposed(const int32_t *__restrict__ Q, int N, int I, int J,
                                int32_t (&t)[kTile][kTile + 1]) {
    for (int q = threadIdx.x; q < kTile * kTile; q += blockDim.x) {
        const int r = q >> 6, c = q & 63;
        t[c][r] = J + r < N && I + c < N ? Q[(size_t)(J + r) * N + I + c] : 0;
    }
    __syncthreads();
}

// Row sums of |W| into row[N], the largest |W| into *maxw and every workgroup's
// common factor into gcds (0: no coupling in its tile).  One workgroup per tile
// pair I <= J.
__global__ __launch_bounds__(256) void k_derive(const int32_t *__restrict__ Q, int N,
                                                unsigned long long *row,
                                                unsigned long long *maxw,
                                                unsigned long long *gcds) {
    __shared__ int32_t t[kTile][kTile + 1];
    __shared__ unsigned long long cs[kTile], red[256], redg[256];
    const int tiles = gridDim.x;
    const int bi = blockIdx.y, bj = blockIdx.x;
    if (bi > bj) {
        if (threadIdx.x == 0) gcds[(size_t)bi * tiles + bj] = 0ull;
        return;
    }
    const int I = bi * kTile, J = bj * kTile;
    if (threadIdx.x < kTile) cs[threadIdx.x] = 0ull;
    load_transposed(Q, N, I, J, t);
    const int c = threadIdx.x & 63;
    uint64_t g = 0, mw = 0, col = 0;
    for (int r = threadIdx.x >> 6; r < kTile; r += 4) {
        const int i = I + r, j = J + c;
        uint64_t aw = 0;
        if (i < N && j < N && i < j) {
            const int64_t w = (int64_t)Q[(size_t)i * N + j] + (int64_t)t[r][c];
            aw = (uint64_t)(w < 0 ? -w : w);
        }
        col += aw;
        mw = aw > mw ? aw : mw;
        if (aw && g != 1) g = gcd_step(g, aw);
        // the wave holds row r of the tile
        uint64_t s = aw;
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor((unsigned long long)s, o);
        if (c == 0 && s) atomicAdd(&row[i], (unsigned long long)s);
    }
    if (col) atomicAdd(&cs[c], (unsigned long long)col);
    red[threadIdx.x] = mw;
    redg[threadIdx.x] = g;
    __syncthreads();
    if (threadIdx.x < kTile && cs[threadIdx.x]) atomicAdd(&row[J + threadIdx.x], cs[threadIdx.x]);
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + o]);
            redg[threadIdx.x] = gcd_step(redg[threadIdx.x], redg[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (red[0]) atomicMax(maxw, red[0]);
        gcds[(size_t)bi * tiles + bj] = redg[0];
    }
}

// out: the largest |b_i| + sum_j |W_ij|, the largest |W_ij|, the common factor.
__global__ __launch_bounds__(1024) void k_derive_sum(const int32_t *__restrict__ Q, int N,
                                                     const unsigned long long *row,
                                                     const unsigned long long *maxw,
                                                     const unsigned long long *gcds, int n_gcds,
                                                     unsigned long long *out) {
    __shared__ unsigned long long red[1024], redg[1024];
    uint64_t m = 0, g = 0;
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        const int64_t b = Q[(size_t)i * N + i];
        const uint64_t v = row[i] + (uint64_t)(b < 0 ? -b : b);
        m = v > m ? v : m;
    }
    for (int q = threadIdx.x; q < n_gcds; q += blockDim.x)
        if (g != 1 && gcds[q]) g = gcd_step(g, gcds[q]);
    red[threadIdx.x] = m;
    redg[threadIdx.x] = g;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + o]);
            redg[threadIdx.x] = gcd_step(redg[threadIdx.x], redg[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = red[0];
        out[1] = *maxw;
        out[2] = redg[0];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_image(const int32_t *__restrict__ Q, int N, int ld,
                                               double g, T *__restrict__ W,
                                               int32_t *__restrict__ b) {
    __shared__ int32_t t[kTile][kTile + 1];
    const int I = blockIdx.y * kTile, J = blockIdx.x * kTile;
    load_transposed(Q, N, I, J, t);
    for (int q = threadIdx.x; q < kTile * kTile; q += blockDim.x) {
        const int r = q >> 6, c = q & 63, i = I + r, j = J + c;
        int64_t w = 0;
        if (i < N && j < N && i != j) w = (int64_t)Q[(size_t)i * N + j] + (int64_t)t[r][c];
        // (a multiple of g below 2^33: the quotient is exact in double)
        W[(size_t)i * ld + j] = (T)(int64_t)((double)w / g);
        if (i == j) b[i] = i < N ? Q[(size_t)i * N + i] : 0;
    }
}

__global__ void k_zero_u64(unsigned long long *p, int n) {
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x)
        p[q] = 0ull;
}

}  // namespace

size_t derive_scratch_bytes(int N) {
    const size_t tiles = (size_t)(N + kTile - 1) / kTile;
    return ((size_t)N + 1 + tiles * tiles + 3) * 8;
}

int launch_derive(const int32_t *Q, int N, uint64_t *scratch, uint64_t **out, void *stream) {
    const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int tiles = (N + kTile - 1) / kTile;
    auto *row = reinterpret_cast<unsigned long long *>(scratch);
    unsigned long long *maxw = row + N, *gcds = maxw + 1, *res = gcds + (size_t)tiles * tiles;
    hipLaunchKernelGGL(k_zero_u64, dim3((N + 256) / 256), dim3(256), 0, st, row, N + 1);
    hipLaunchKernelGGL(k_derive, dim3(tiles, tiles), dim3(256), 0, st, Q, N, row, maxw, gcds);
    hipLaunchKernelGGL(k_derive_sum, dim3(1), dim3(1024), 0, st, Q, N, row, maxw, gcds,
                       tiles * tiles, res);
    *out = reinterpret_cast<uint64_t *>(res);
    return (int)hipGetLastError();
}

int launch_image(const int32_t *Q, int N, int ld, int dtype, int64_t g, void *W, int32_t *b,
                 void *stream) {
    const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const dim3 grid(ld / kTile, ld / kTile);
    if (dtype == 1)
        hipLaunchKernelGGL(k_image<int8_t>, grid, dim3(256), 0, st, Q, N, ld, (double)g,
                           static_cast<int8_t *>(W), b);
    else if (dtype == 2)
        hipLaunchKernelGGL(k_image<int16_t>, grid, dim3(256), 0, st, Q, N, ld, (double)g,
                           static_cast<int16_t *>(W), b);
    else if (dtype == 4)
        hipLaunchKernelGGL(k_image<int32_t>, grid, dim3(256), 0, st, Q, N, ld, (double)g,
                           static_cast<int32_t *>(W), b);
    else
        return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

}  // namespace dapt
