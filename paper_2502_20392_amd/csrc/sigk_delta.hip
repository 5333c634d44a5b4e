// sigk_delta.hip -- the cell-coefficient field for many channels.
//
// For d > 32 the coefficients c_kl = <dx_k, dy_l> are no longer cheap next to
// the cell map (2d flops against about 6P^2), and they form a dense matrix
// product of the two increment sequences, dY dX^T.  This kernel computes it on
// the FP64 matrix cores (v_mfma_f64_16x16x4f64) for every pair of a Gram call
// and stores it in the order the strip sweep reads it: per 64-row strip s,
// step t and lane j, the coefficient of cell (t - j, 64 s + j), so that each
// step of the sweep reads 64 consecutive doubles.  Entries of cells outside
// the grid are never written (the sweep masks them).
//
// Block: 64 rows (one strip) x 64 columns of one pair, four waves of
// 32 x 32, each a 2 x 2 set of 16 x 16 MFMA tiles; channels are staged in LDS
// 16 at a time, the increments formed on the way in.  The result tile goes
// through LDS so that each step's run of lanes is written contiguously.
//
// A stage is 16 MFMAs per wave (about 1100 cycles) against a global load's
// latency of one to two thousand, so the next stage's points are loaded into
// registers while this one's products run, and two LDS buffers leave one
// barrier per stage; the result tile reuses their space, which lets four
// blocks share a CU.  4096 x 4096 cells, d 512: 0.86 ms with a load, a barrier
// and the products in turn, 0.45 ms now.
#include "sigk_device.h"

namespace sigk {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kKT = 16;  // channels per LDS stage

// Lane layout of v_mfma_f64_16x16x4f64 (checked on the device): A[i][k] in
// lane i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane j + 16 (i % 4),
// element i / 4.
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(4))) delta_gemm_kernel(FwdArgs a) {
    // two stages of increments [buffer][y, x][row][channel]; later the result
    constexpr int kLd = kKT + 1, kStage = 64 * kLd;
    __shared__ double lds[64 * 65 > 4 * kStage ? 64 * 65 : 4 * kStage];
    const int pair = (int)blockIdx.z;
    const Geo g = resolve(a, pair, 1, 0);
    const int m = g.m, n = g.n, d = a.d;
    const int s = (int)blockIdx.y;
    const int k0 = (int)blockIdx.x * 64, l0 = s * 64;
    if (k0 >= m || l0 >= n) return;  // uniform over the block
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int rb = (w >> 1) * 32, cb = (w & 1) * 32;
    d4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    // thread: channel cc of rows r0 + 16 i
    const int cc = tid % kKT, r0 = tid / kKT;
    double ylo[4], yhi[4], xlo[4], xhi[4];
    auto load = [&](int kc) {
        const int ch = min(kc + cc, d - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = r0 + 16 * i;
            const double* yp = g.y + (int64_t)min(l0 + r, n - 1) * d + ch;
            const double* xp = g.x + (int64_t)min(k0 + r, m - 1) * d + ch;
            ylo[i] = yp[0];
            yhi[i] = yp[d];
            xlo[i] = xp[0];
            xhi[i] = xp[d];
        }
    };
    load(0);
    for (int kc = 0, buf = 0; kc < d; kc += kKT, buf ^= 1) {
        double* sy = lds + buf * 2 * kStage;
        double* sx = sy + kStage;
        const bool in = kc + cc < d;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = r0 + 16 * i;
            sy[r * kLd + cc] = in && l0 + r < n ? yhi[i] - ylo[i] : 0.0;
            sx[r * kLd + cc] = in && k0 + r < m ? xhi[i] - xlo[i] : 0.0;
        }
        __syncthreads();
        if (kc + kKT < d) load(kc + kKT);
#pragma unroll
        for (int kk = 0; kk < kKT; kk += 4) {
            double av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                av[i] = sy[(rb + 16 * i + (lane & 15)) * kLd + kk + (lane >> 4)];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                bv[j] = sx[(cb + 16 * j + (lane & 15)) * kLd + kk + (lane >> 4)];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
    __syncthreads();
    double(*so)[65] = (double(*)[65])lds;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                so[rb + 16 * i + (lane >> 4) + 4 * r][cb + 16 * j + (lane & 15)] = acc[i][j][r];
    __syncthreads();
    // step t = k0 + u: lane j of the strip holds column t - j
    double* dst = a.delta + g.delta + (int64_t)s * delta_steps(m) * kWave;
    for (int u = w; u < 127; u += 4) {
        const int kt = u - lane;  // column within the tile
        if (kt >= 0 && kt < 64 && l0 + lane < n && k0 + kt < m)
            dst[(int64_t)(k0 + u) * kWave + lane] = so[lane][kt];
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0)
        atomicAdd(&a.hdr->flops, 2ull * (unsigned long long)d * (unsigned long long)m *
                                     (unsigned long long)n);
}

}  // namespace

hipError_t launch_delta_gemm(const FwdArgs& a, hipStream_t s) {
    const int64_t m = a.lx - 1, n = a.ly - 1;
    const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((n + 63) / 64), (unsigned)a.npairs);
    hipLaunchKernelGGL(delta_gemm_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace sigk
