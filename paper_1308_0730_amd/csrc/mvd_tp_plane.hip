// Plane pass of the two-pass convolution and the builder of its kernel
// spectra (see mvd_two_pass.h).
#include "mvd_two_pass.h"

using namespace mvdk;

namespace {

// Largest workgroup of the plane pass.
constexpr int kPlaneThreads = 1024;

__global__ void __launch_bounds__(kPlaneThreads)
    k_plane(const TpJob* __restrict__ jobs, int njobs, const float2* __restrict__ twp, int v, int role, int conj,
            int src_saved) {
  extern __shared__ float2 dyn[];
  int local;
  const int jid = find_tp(jobs, njobs, false, local);
  if (jid < 0) return;
  const TpJob& J = jobs[jid];
  if (v >= J.nviews) return;
  const int T = blockDim.x, nz = J.nz, n1 = J.n1, P = J.pl;
  float2* s_z = dyn + nz * P;
  float2* s_y = s_z + nz;
  const int64_t off = (int64_t)local * nz * n1;
  const float2* src = reinterpret_cast<const float2*>(src_saved ? J.saved : J.spec) + off;
  float2* dst = reinterpret_cast<float2*>(J.spec) + off;
  const float2* k = reinterpret_cast<const float2*>(J.K2[role]) + (int64_t)v * J.k2_elems + off;
  const tp::Axis Z{n1, 1, P, nz, J.mg_n1}, Y{nz, P, 1, n1, J.mg_nz};
  // the thread's first table entries: loaded now, stored once the first data
  // loads are out
  const int tid = threadIdx.x;
  const float2 *tz = twp + J.tw_z, *ty = twp + J.tw_y;
  const int R = J.R;
  const float2 r_z = ldg(tz + (tid < nz ? tid : 0)), r_y = ldg(ty + (tid < n1 ? tid * R : 0));
  auto st_tables = [&] {
    if (tid < nz) s_z[tid] = r_z;
    if (tid < n1) s_y[tid] = r_y;
    for (int i = tid + T; i < nz; i += T) s_z[i] = ldg(tz + i);
    for (int i = tid + T; i < n1; i += T) s_y[i] = ldg(ty + i * R);
  };
  switch (J.sz[0].radix) {
#define X(r) \
  case r: tp::st_load<r>(dyn, src, Z, J.sz[0], s_z, T, st_tables); break;
    TP_RADICES(X)
#undef X
  }
  for (int s = 1; s < J.nsz; ++s) {
    __syncthreads();
    tp::lds_stage<false>(dyn, Z, J.sz[s], s_z, T);
  }
  for (int s = 0; s < J.nsy - 1; ++s) {
    __syncthreads();
    tp::lds_stage<false>(dyn, Y, J.sy[s], s_y, T);
  }
  __syncthreads();
  switch (J.sy[J.nsy - 1].radix) {
#define X(r) \
  case r: tp::st_mul<r>(dyn, k, Y, conj, T); break;
    TP_RADICES(X)
#undef X
  }
  for (int s = J.nsy - 2; s >= 0; --s) {
    __syncthreads();
    tp::lds_stage<true>(dyn, Y, J.sy[s], s_y, T);
  }
  for (int s = J.nsz - 1; s >= 1; --s) {
    __syncthreads();
    tp::lds_stage<true>(dyn, Z, J.sz[s], s_z, T);
  }
  __syncthreads();
  switch (J.sz[0].radix) {
#define X(r) \
  case r: tp::st_store<r>(dyn, dst, Z, J.sz[0], s_z, T); break;
    TP_RADICES(X)
#undef X
  }
}

// Kernel spectrum of one (view, kx, j) plane from the kernel planes (their x
// and y stages): place the taps of every ky = R k1 + j on its z line, in the
// position order the plane pass leaves k1 in, transform along z and store
// [y1 position][z position], halved (the x passes leave twice the spectrum).
__global__ void __launch_bounds__(kPlaneThreads)
    k_plane_kernel(const TpJob* __restrict__ jobs, const float2* __restrict__ twp, int role,
                   float2* __restrict__ out) {
  extern __shared__ float2 dyn[];
  const TpJob& J = jobs[0];
  const int T = blockDim.x, nz = J.nz, n1 = J.n1, P = J.pl, R = J.R;
  const int local = (int)(blockIdx.x % (unsigned)J.yz_tiles), v = (int)(blockIdx.x / (unsigned)J.yz_tiles);
  if (v >= J.nviews) return;
  const int kx = local / R, j = local - kx * R;
  float2* s_z = dyn + nz * P;
  for (int i = threadIdx.x; i < nz; i += T) s_z[i] = ldg(twp + J.tw_z + i);
  const float2* H = reinterpret_cast<const float2*>(J.H[role]) + (int64_t)v * J.h_elems;
  for (int it = threadIdx.x; it < nz * n1; it += T) {
    const int z = it / n1, p = it - z * n1;
    int rest = p, len = n1, mul = 1, k1 = 0;
    for (int s = 0; s < J.nsy; ++s) {
      const int r = J.sy[s].radix;
      len /= r;
      const int d = rest / len;
      rest -= d * len;
      k1 += d * mul;
      mul *= r;
    }
    const int ky = R * k1 + j;
    int d = z + J.cz;
    if (d >= nz) d -= nz;
    float2 x = make_float2(0.f, 0.f);
    if (d < J.kz)
      x = kx < J.M ? ldg(H + ((int64_t)d * J.ny + ky) * J.Mp + kx) : ldg(H + J.h_main + (int64_t)d * J.ny + ky);
    dyn[z * P + p] = x;
  }
  const tp::Axis Z{n1, 1, P, nz, J.mg_n1};
  for (int s = 0; s < J.nsz; ++s) {
    __syncthreads();
    tp::lds_stage<false>(dyn, Z, J.sz[s], s_z, T);
  }
  __syncthreads();
  float2* o = out + (int64_t)v * J.k2_elems + (int64_t)local * nz * n1;
  for (int it = threadIdx.x; it < nz * n1; it += T) {
    const int p = it / nz, z = it - p * nz;
    const float2 x = dyn[z * P + p];
    stg(o + it, make_float2(0.5f * x.x, 0.5f * x.y));
  }
}

}  // namespace

hipError_t mvd_launch_plane(const TpArgs& a, int threads, size_t lds, int v, int role, int conj, int src_saved) {
  k_plane<<<a.grid, threads, lds, a.stream>>>(a.jobs, a.njobs, a.tw, v, role, conj, src_saved);
  return hipGetLastError();
}

hipError_t mvd_launch_plane_kernel(const TpArgs& a, size_t lds, int role, float* out) {
  k_plane_kernel<<<a.grid, 256, lds, a.stream>>>(a.jobs, a.tw, role, reinterpret_cast<float2*>(out));
  return hipGetLastError();
}
