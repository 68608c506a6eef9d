// Fourier factors of the three-dimensional spectral series (the paper's
// duplicated-mode use, Sec. 3 footnote) and the mixing of coefficients
// between the full mode list (n, m, l) and its distinct (n, m) pairs.
//
// F_l(phi) = cos(l phi) for l >= 0 and sin(|l| phi) for l < 0, the same
// convention as the angular factor of Eq. zernike-poly.
//
// The three kernels evaluate J Q angles each and read or write O(J B + U Q B)
// values: bound by the angles (about 45 vector instructions, angle.hpp) and,
// with few modes per lane, by load latency.  Planes go to the lanes of a wave
// where rows of T are read along them, modes to the waves.  18 513 modes x 64
// planes, 1 set, mix / unmix / phi gradient: 8 / 6 / 17 us, from 18 / 24 / 75 with a
// general sincos and the phi gradient on one workgroup per plane.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "angle.hpp"
#include "series3d.hpp"

namespace zp {
namespace {

constexpr int kThreads = 256;
constexpr int kWave = 64, kSub = kThreads / kWave;

// F_l(phi) and dF_l/dphi (|l| is at most 2^20, so the angle is exact to
// rounding, angle.hpp).
__device__ __forceinline__ void fourier(int l, const Turn &phi, double &F, double &dF)
{
    const double fa = (double)(l < 0 ? -l : l);
    double cs, sn;
    phi.angle(fa, cs, sn);
    F = l >= 0 ? cs : sn;
    dF = l >= 0 ? -fa * sn : fa * cs;
}

// One workgroup per 64 elements (q, b) of T's rows and per pair u (striding in
// y): its four waves share the pair's modes and add up through LDS.
__global__ __launch_bounds__(kThreads) void mix_kernel(const int32_t *__restrict__ uptr,
                                                       const int32_t *__restrict__ jl, const int32_t *__restrict__ l,
                                                       const double *__restrict__ c, int64_t B,
                                                       const double *__restrict__ phi, int64_t QB, int64_t U,
                                                       int64_t e0, double *__restrict__ T)
{
    __shared__ double red[kSub][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t e = e0 + (int64_t)blockIdx.x * kWave + lane, el = e < QB ? e : QB - 1;
    const int64_t q = el / B, b = el - q * B;
    const Turn ph(phi[q]);
    for (int64_t u = blockIdx.y; u < U; u += gridDim.y) {
        double acc = 0.0;
        const int t1 = uptr[u + 1];
#pragma unroll 4
        for (int t = uptr[u] + wave; t < t1; t += kSub) {
            const int j = jl[t];
            double F, dF;
            fourier(l[j], ph, F, dF);
            acc = __builtin_fma(c[(int64_t)j * B + b], F, acc);
        }
        red[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && e < QB) T[u * QB + e] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
        __syncthreads();
    }
}

// 64 elements (j, b) per workgroup, whose four waves share the planes (their
// angles in quarter turns through LDS, a tile of planes at a time).
__global__ __launch_bounds__(kThreads) void unmix_kernel(const int32_t *__restrict__ owner,
                                                         const int32_t *__restrict__ l,
                                                         const double *__restrict__ gT, int64_t B,
                                                         const double *__restrict__ phi, int64_t Q, int64_t J,
                                                         int64_t t0, double *__restrict__ grad_c)
{
    __shared__ Turn ph[kThreads];
    __shared__ double red[kSub][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = (int)threadIdx.x / kWave;
    const int64_t t = t0 + (int64_t)blockIdx.x * kWave + lane;
    const bool live = t < J * B;
    const int64_t j = live ? t / B : 0, b = live ? t - j * B : 0;
    const int lj = l[j];
    const double *row = gT + (int64_t)owner[j] * Q * B + b;
    double acc = 0.0;
    for (int64_t q0 = 0; q0 < Q; q0 += kThreads) {
        const int n = (int)(Q - q0 < kThreads ? Q - q0 : kThreads);
        __syncthreads();
        if ((int)threadIdx.x < n) ph[threadIdx.x] = Turn(phi[q0 + threadIdx.x]);
        __syncthreads();
#pragma unroll 4
        for (int q = wave; q < n; q += kSub) {
            double F, dF;
            fourier(lj, ph[q], F, dF);
            acc = __builtin_fma(F, row[(q0 + q) * B], acc);
        }
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && live) grad_c[t] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Partial sums of grad_phi: workgroup (x, y) takes a wave of planes q (one per
// lane, so that rows of gT are read along q) and the modes dealt to y's four
// waves, which add up through LDS.  part: [ny][Q].
__global__ __launch_bounds__(kThreads) void phi_grad_kernel(const int32_t *__restrict__ owner,
                                                            const int32_t *__restrict__ l,
                                                            const double *__restrict__ gT,
                                                            const double *__restrict__ c, int64_t B,
                                                            const double *__restrict__ phi, int64_t Q, int64_t J,
                                                            double *__restrict__ part)
{
    __shared__ double red[kSub][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t q = (int64_t)blockIdx.x * kWave + lane, ql = q < Q ? q : Q - 1;
    const Turn ph(phi[ql]);
    double acc = 0.0;
#pragma unroll 4
    for (int64_t j = (int64_t)blockIdx.y * kSub + wave; j < J; j += (int64_t)gridDim.y * kSub) {
        const double *g = gT + ((int64_t)owner[j] * Q + ql) * B;
        const double *cj = c + j * B;
        double s = 0.0;
        for (int64_t b = 0; b < B; ++b) s = __builtin_fma(cj[b], g[b], s);
        double F, dF;
        fourier(l[j], ph, F, dF);
        acc = __builtin_fma(dF, s, acc);
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && q < Q)
        part[(int64_t)blockIdx.y * Q + q] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// grad_phi[q] = sum of the ny partial sums, in a fixed order.
__global__ __launch_bounds__(kThreads) void phi_reduce_kernel(const double *__restrict__ part, int64_t ny, int64_t Q,
                                                              double *__restrict__ grad_phi)
{
    __shared__ double red[kSub][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = (int)threadIdx.x / kWave;
    const int64_t q = (int64_t)blockIdx.x * kWave + lane, ql = q < Q ? q : Q - 1;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t y = wave; y < ny; y += kSub) acc += part[y * Q + ql];
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && q < Q) grad_phi[q] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

} // namespace

zp_status launch_fourier_mix(const Plan3 &p, const double *c, int64_t B, const double *phi, int64_t Q, double *T,
                             hipStream_t s)
{
    const int64_t U = (int64_t)p.un.size(), QB = Q * B;
    if (U == 0 || QB == 0) return ZP_OK;
    constexpr int64_t kMost = max_workgroups(kThreads) * kWave; // elements of one launch
    for (int64_t e0 = 0; e0 < QB; e0 += kMost) {
        const dim3 grid((unsigned)((std::min(kMost, QB - e0) + kWave - 1) / kWave), (unsigned)std::min<int64_t>(U, 65535));
        hipLaunchKernelGGL(mix_kernel, grid, dim3(kThreads), 0, s, p.d_uptr, p.d_jl, p.d_l, c, B, phi, QB, U, e0, T);
        const zp_status st = hip_check(hipGetLastError(), "fourier mix launch");
        if (st != ZP_OK) return st;
    }
    return ZP_OK;
}

zp_status launch_fourier_unmix(const Plan3 &p, const double *gT, int64_t B, const double *phi, int64_t Q,
                               double *grad_c, hipStream_t s)
{
    const int64_t J = (int64_t)p.n.size();
    if (J == 0 || B == 0) return ZP_OK;
    constexpr int64_t kMost = max_workgroups(kThreads) * kWave;
    for (int64_t t0 = 0; t0 < J * B; t0 += kMost) {
        const dim3 grid((unsigned)((std::min(kMost, J * B - t0) + kWave - 1) / kWave));
        hipLaunchKernelGGL(unmix_kernel, grid, dim3(kThreads), 0, s, p.d_owner, p.d_l, gT, B, phi, Q, J, t0, grad_c);
        const zp_status st = hip_check(hipGetLastError(), "fourier unmix launch");
        if (st != ZP_OK) return st;
    }
    return ZP_OK;
}

zp_status launch_fourier_phi_grad(const Plan3 &p, const double *gT, const double *c, int64_t B, const double *phi,
                                  int64_t Q, double *part, int64_t part_rows, double *grad_phi, hipStream_t s)
{
    const int64_t J = (int64_t)p.n.size();
    if (Q == 0) return ZP_OK;
    const int64_t bx = (Q + kWave - 1) / kWave;
    if (bx > max_workgroups(kThreads)) return set_error(ZP_ERR_ARG, "Q too large for one launch");
    // enough workgroups to fill the chip, each with some modes per wave
    const int64_t want = std::max<int64_t>(1, std::min((J + 8 * kSub - 1) / (8 * kSub), (512 + bx - 1) / bx));
    const int64_t ny = std::max<int64_t>(1, std::min(want, part_rows));
    double *to = ny == 1 ? grad_phi : part;
    hipLaunchKernelGGL(phi_grad_kernel, dim3((unsigned)bx, (unsigned)ny), dim3(kThreads), 0, s, p.d_owner, p.d_l, gT, c,
                       B, phi, Q, J, to);
    if (ny > 1)
        hipLaunchKernelGGL(phi_reduce_kernel, dim3((unsigned)bx), dim3(kThreads), 0, s, part, ny, Q, grad_phi);
    return hip_check(hipGetLastError(), "fourier phi-gradient launch");
}

} // namespace zp
