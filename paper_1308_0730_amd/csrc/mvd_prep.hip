// FP64 preparation of kernels on the device: correlations of small windows
// (the compound kernels of eq. 222 and 230 and their adjoint) and the x and y
// stages of kernel spectra.  The same sums as the host code of mvd_host.cpp
// (which stays for kernels too large for the limits here): that code took
// 1 to 165 ms of a handle's first iteration, more than the iterations.
#include <hip/hip_runtime.h>

#include "mvd_gmem.h"
#include "mvd_kernels.h"

using namespace mvdk;

namespace {

constexpr int kCorrWaves = 16, kCorrX = 8;

// out[d] = sum_e A[e] B[d + s e] for every d of the centred out window, e over
// A's centred window, B zero outside its own.  Small windows are bound by the
// latency of B's loads, few workgroups (17^3: 10 per correlation) walking
// A's rows; large ones by FP64 FMAs.  Eight outputs along x per thread take
// 15 loads of B for 64 FMAs, A is the same for a whole wave, and sixteen waves
// of a workgroup share out A's rows.  Fixed summation order.  31x31x41, six
// views, Optimization I (30 pairs, 4.7e10 FMAs): 165 ms of host transforms
// before, 11 ms now with the planes; 17^3, two views, EFF: 7.3 and 0.5 ms.
__global__ void __launch_bounds__(64 * kCorrWaves) k_corr(const CorrJob* __restrict__ jobs) {
  __shared__ double red[kCorrWaves / 2][64][kCorrX + 1];
  const CorrJob& J = jobs[blockIdx.y];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = (J.o[0] + kCorrX - 1) / kCorrX, total = gx * J.o[1] * J.o[2];
  if ((int)blockIdx.x * 64 >= total) return;
  const int t = min((int)blockIdx.x * 64 + lane, total - 1);
  const int x0 = t % gx * kCorrX, y0 = t / gx % J.o[1], z0 = t / gx / J.o[1];
  // position in B of (d - r_o) + s (e - r_a) + r_b with e counted from 0 in
  // the direction of B
  const int bx = x0 - J.o[0] / 2 - J.a[0] / 2 + J.b[0] / 2;
  const int by = y0 - J.o[1] / 2 - J.a[1] / 2 + J.b[1] / 2;
  const int bz = z0 - J.o[2] / 2 - J.a[2] / 2 + J.b[2] / 2;
  const int na = J.a[0] * J.a[1] * J.a[2];
  double acc[kCorrX] = {};
  for (int row = wave; row < J.a[1] * J.a[2]; row += kCorrWaves) {
    const int ez = row / J.a[1], ey = row - ez * J.a[1];
    const int z = bz + ez, y = by + ey;
    const bool in = (unsigned)z < (unsigned)J.b[2] && (unsigned)y < (unsigned)J.b[1];
    const double* B = J.B + ((int64_t)(in ? z : 0) * J.b[1] + (in ? y : 0)) * J.b[0];
    for (int e0 = 0; e0 < J.a[0]; e0 += 8) {
      double b[kCorrX + 7];
#pragma unroll
      for (int i = 0; i < kCorrX + 7; ++i) {
        const int x = bx + e0 + i;
        b[i] = in && (unsigned)x < (unsigned)J.b[0] ? ldg(B + x) : 0.0;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (e0 + k >= J.a[0]) break;
        const int i = row * J.a[0] + e0 + k;
        const double a = J.A[J.s > 0 ? i : na - 1 - i];
#pragma unroll
        for (int j = 0; j < kCorrX; ++j) acc[j] += a * b[k + j];
      }
    }
  }
  // the upper half of the waves hands its sums to the lower, which hands on
  if (wave >= kCorrWaves / 2)
#pragma unroll
    for (int j = 0; j < kCorrX; ++j) red[wave - kCorrWaves / 2][lane][j] = acc[j];
  __syncthreads();
  if (wave < kCorrWaves / 2)
#pragma unroll
    for (int j = 0; j < kCorrX; ++j) red[wave][lane][j] += acc[j];
  __syncthreads();
  for (int i = threadIdx.x; i < 64 * kCorrX; i += 64 * kCorrWaves) {
    const int l = i / kCorrX, j = i % kCorrX, tt = (int)blockIdx.x * 64 + l;
    if (tt >= total) continue;
    const int x = tt % gx * kCorrX + j;
    if (x >= J.o[0]) continue;
    double s = 0;
    for (int w = 0; w < kCorrWaves / 2; ++w) s += red[w][l][j];
    stg(J.out + (int64_t)(tt / gx) * J.o[0] + x, s);
  }
}

__device__ double block_sum(double x, double* red) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  return s;
}

// One workgroup per view: K_v = U / sum U with U = mirror(P_v) prod_w f_vw
// (or mirror(P_v)^n), and, when kbar is given, the adjoint of that product:
// dL/dU, T_vw = dL/df_vw and the direct term dL/dmirror(P_v).
__global__ void __launch_bounds__(1024) k_compound(const CompoundJob* __restrict__ jobs, int n, int power,
                                                   double* __restrict__ sums) {
  __shared__ double red[16];
  const int v = blockIdx.x;
  const CompoundJob& J = jobs[v];
  const int nk = J.nk;
  auto u_of = [&](int i) {
    const double m = J.P[nk - 1 - i];
    if (power) return pow(m, (double)n);
    double u = m;
    for (int w = 0; w < n; ++w)
      if (w != v) u *= J.f[(int64_t)w * nk + i];
    return u;
  };
  double s = 0, kk = 0;
  for (int i = threadIdx.x; i < nk; i += blockDim.x) {
    const double u = u_of(i);
    s += u;
    if (J.kbar) kk += J.kbar[i] * u;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) sums[v] = s;
  if (!J.kbar) {
    for (int i = threadIdx.x; i < nk; i += blockDim.x) J.K[i] = u_of(i) / s;
    return;
  }
  kk = block_sum(kk, red) / s;
  for (int i = threadIdx.x; i < nk; i += blockDim.x) {
    const double ub = (J.kbar[i] - kk) / s, m = J.P[nk - 1 - i];
    double d = ub;
    for (int w = 0; w < n; ++w)
      if (w != v) d *= J.f[(int64_t)w * nk + i];
    J.direct[i] = d;
    for (int w = 0; w < n; ++w) {
      if (w == v) continue;
      double p = ub * m;
      for (int u = 0; u < n; ++u)
        if (u != v && u != w) p *= J.f[(int64_t)u * nk + i];
      J.T[(int64_t)w * nk + i] = p;
    }
  }
}

// dL/dP_w: its parts over every view, in view order.
__global__ void __launch_bounds__(256) k_vjp_sum(const VjpJob* __restrict__ jobs, int n) {
  const int w = blockIdx.y;
  const VjpJob& J = jobs[w];
  const int i = (int)blockIdx.x * 256 + threadIdx.x, nk = J.nk;
  if (i >= nk) return;
  double g = J.direct[nk - 1 - i];
  for (int v = 0; v < n; ++v) {
    if (v == w) continue;
    g += J.mv[(int64_t)v * nk + i];
    g += J.pw[(int64_t)v * nk + i];
    if (J.mw) g += J.mw[(int64_t)v * nk + i];
  }
  J.g[i] = g;
}

// x and y stages of the spectra of centred kernels: plane d of the common z
// window, 16 kx, every ky.  The x stage of the plane's rows goes through LDS;
// FP64 throughout, scaled and rounded once to FP32.  tx and ty are the host's
// tables and no product is contracted: the planes have the host code's bits
// (PSF gradients are ill-conditioned enough to show a changed rounding).
// Six views of 31x31x41 on 512x512: 91 ms on the host, 1.2 ms here.
__global__ void __launch_bounds__(256) k_kernel_planes(const PlaneJob* __restrict__ jobs, int nx, int ny, int Mp,
                                                       int kzw, int64_t h_main, double scale,
                                                       const double2* __restrict__ gtx,
                                                       const double2* __restrict__ gty) {
#pragma clang fp contract(off)
  extern __shared__ double2 sh[];
  const PlaneJob& J = jobs[blockIdx.z];
  const int M = nx / 2, d = blockIdx.y, k0 = (int)blockIdx.x * 16, tid = threadIdx.x;
  float2* out = reinterpret_cast<float2*>(J.out);
  const int z = d - (kzw - J.kz) / 2;
  const bool in = z >= 0 && z < J.kz;
  double2 *tx = sh, *ty = tx + nx, *rows = ty + ny;
  if (in) {
    for (int m = tid; m < nx; m += 256) tx[m] = ldg(gtx + m);
    for (int m = tid; m < ny; m += 256) ty[m] = ldg(gty + m);
    __syncthreads();
    for (int i = tid; i < J.ky * 16; i += 256) {
      const int y = i >> 4, k = k0 + (i & 15);
      double re = 0, im = 0;
      if (k <= M) {
        // phase index k (x - cx) mod nx, stepped by k along x
        int idx = (int)((int64_t)k * ((J.kx - 1) / 2) % nx);
        idx = idx ? nx - idx : 0;
        const double* row = J.K + ((int64_t)z * J.ky + y) * J.kx;
        for (int x = 0; x < J.kx; ++x) {
          const double a = ldg(row + x);
          re += a * tx[idx].x;
          im += a * tx[idx].y;
          idx += k;
          if (idx >= nx) idx -= nx;
        }
      }
      rows[i] = make_double2(re, im);
    }
    __syncthreads();
  }
  const int k = k0 + (tid & 15);
  if (k > M) return;
  for (int ky = tid >> 4; ky < ny; ky += 16) {
    double re = 0, im = 0;
    if (in) {
      int idx = (int)((int64_t)ky * ((J.ky - 1) / 2) % ny);
      idx = idx ? ny - idx : 0;
      for (int y = 0; y < J.ky; ++y) {
        const double2 a = rows[y * 16 + (tid & 15)], w = ty[idx];
        re += a.x * w.x - a.y * w.y;
        im += a.x * w.y + a.y * w.x;
        idx += ky;
        if (idx >= ny) idx -= ny;
      }
    }
    const int64_t o = k < M ? ((int64_t)d * ny + ky) * Mp + k : h_main + (int64_t)d * ny + ky;
    stg(out + o, make_float2((float)(re * scale), (float)(im * scale)));
  }
}

}  // namespace

hipError_t mvd_launch_corr(const CorrJob* jobs, int n, int max_groups, hipStream_t s) {
  if (n < 1) return hipSuccess;
  k_corr<<<dim3((unsigned)((max_groups + 63) / 64), (unsigned)n), 64 * kCorrWaves, 0, s>>>(jobs);
  return hipGetLastError();
}

int mvd_corr_groups(const int* o) { return (o[0] + kCorrX - 1) / kCorrX * o[1] * o[2]; }

hipError_t mvd_launch_compound(const CompoundJob* jobs, int n, int power, double* sums, hipStream_t s) {
  k_compound<<<n, 1024, 0, s>>>(jobs, n, power, sums);
  return hipGetLastError();
}

hipError_t mvd_launch_vjp_sum(const VjpJob* jobs, int n, int max_nk, hipStream_t s) {
  k_vjp_sum<<<dim3((unsigned)((max_nk + 255) / 256), (unsigned)n), 256, 0, s>>>(jobs, n);
  return hipGetLastError();
}

size_t mvd_kernel_planes_lds(int nx, int ny, int ky) { return (size_t)(nx + ny + 16 * ky) * sizeof(double2); }

hipError_t mvd_launch_kernel_planes(const PlaneJob* jobs, int n, int nx, int ny, int Mp, int kzw, int64_t h_main,
                                    double scale, int max_ky, const double2* tx, const double2* ty, hipStream_t s) {
  k_kernel_planes<<<dim3((unsigned)(nx / 2 / 16 + 1), (unsigned)kzw, (unsigned)n), 256,
                    mvd_kernel_planes_lds(nx, ny, max_ky), s>>>(jobs, nx, ny, Mp, kzw, h_main, scale, tx, ty);
  return hipGetLastError();
}
