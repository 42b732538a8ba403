// Two passes over HBM per convolution instead of four (see TpJob).
//
// What bounds the four-pass form on volumes whose (y, z) planes are small is
// not HBM: at 64^3 and 128^3 each of its launches is latency (4 to 13 us for
// 2 to 17 MB), and on larger blocks the three column passes move the
// spectrum six times.  A kx plane of such a volume (after the x passes took
// an R-point factor of the y transform) is at most 64 KB, so one workgroup
// can hold it in LDS and do the whole rest of the convolution on it.
//
// The plane's transforms work in place: decimation in frequency forwards, no
// reordering, product in that order, decimation in time backwards.  A
// butterfly reads and writes the same LDS words, so a stage needs one
// barrier and no second buffer, any length runs with runtime strides and
// compile-time radices, and the last forward stage, the product and the
// first inverse stage share one trip through registers.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_ct.h"
#include "mvd_device.h"
#include "mvd_kernels.h"

namespace mvdk {
namespace tp {

// float2 at a 32-bit byte offset from a uniform base: one address register
// and no 64-bit arithmetic per access (spectra of this form stay below 4 GB)
__device__ __forceinline__ float2 ldo(const float2* base, unsigned off) {
  return *reinterpret_cast<const gmem<float2>*>(reinterpret_cast<const gmem<char>*>(gp(base)) + off);
}
__device__ __forceinline__ void sto(float2* base, unsigned off, float2 v) {
  *reinterpret_cast<gmem<float2>*>(reinterpret_cast<gmem<char>*>(gp(base)) + off) = v;
}

// Keep a running offset out of the compiler's hands: it would rewrite the
// sums as products, and 32-bit integer products issue at a quarter of the
// rate of the adds (they took half of the stages' issue time).
__device__ __forceinline__ int hide(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ int qdiv(int j, unsigned magic, int d) { return d == 1 ? j : udiv(j, magic); }

// ---------------------------------------------------------------------------
// Stages of the plane pass.  Butterfly (line, block b, j) holds the elements
// at positions b nb R + j + i nb, i < R, of one line.

// forward: R-point DFT, then the twiddles of the remaining length
template <int R>
__device__ __forceinline__ void dif_regs(float2* v, const float2* tw, int jt, bool last) {
  Dft<R, false>::run(v);
  if (!last) {
    int ti = jt;
#pragma unroll
    for (int i = 1; i < R; ++i) {
      v[i] = cmul(v[i], tw[ti]);
      ti = hide(ti + jt);
    }
  }
}
// inverse: conjugate twiddles, then the inverse DFT
template <int R>
__device__ __forceinline__ void dit_regs(float2* v, const float2* tw, int jt, bool last) {
  if (!last) {
    int ti = jt;
#pragma unroll
    for (int i = 1; i < R; ++i) {
      v[i] = cmul(v[i], cconj(tw[ti]));
      ti = hide(ti + jt);
    }
  }
  Dft<R, true>::run(v);
}

struct Axis {
  int nl, ls, ps;    // lines, LDS stride between lines and between positions
  int L;
  unsigned mg_nl;
};

// One stage in LDS.
template <int R, bool INV>
__device__ __forceinline__ void st_lds(float2* lds, const Axis& A, const TpStage& S, const float2* tw, int T) {
  const int nb = uni(S.nb), total = uni(A.nl * (A.L / R)), st = uni(nb * A.ps);
  const bool last = nb == 1;
  for (int it = threadIdx.x; it < total; it += T) {
    const int q = qdiv(it, A.mg_nl, A.nl), line = it - (int)__umul24(q, A.nl);
    const int b = qdiv(q, S.mg_nb, nb), j = q - (int)__umul24(b, nb);
    float2* e = lds + __umul24(line, A.ls) + __umul24(__umul24(b, nb * R) + j, A.ps);
    float2 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = e[i * st];
    if (INV)
      dit_regs<R>(v, tw, __umul24(j, S.tws), last);
    else
      dif_regs<R>(v, tw, __umul24(j, S.tws), last);
#pragma unroll
    for (int i = 0; i < R; ++i) e[i * st] = v[i];
  }
}

// First forward z stage: global plane (z lines of n1, y1 contiguous) -> LDS.
// The first round of loads is issued before the workgroup's tables are
// stored (and the barrier after that).
template <int R, class F>
__device__ __forceinline__ void st_load(float2* lds, const float2* g, const Axis& A, const TpStage& S,
                                        const float2* tw, int T, F&& st_tables) {
  const int nb = uni(S.nb), total = uni(A.nl * (A.L / R)), st = uni(nb * A.ps);
  const unsigned gs = 8u * (unsigned)uni(nb * A.nl);
  const bool last = nb == 1;
  float2 v[R];
  auto load = [&](int it) {  // it = j nl + line
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = ldo(g, 8u * (unsigned)it + i * gs);
  };
  if ((int)threadIdx.x < total) load(threadIdx.x);
  st_tables();
  __syncthreads();
  for (int it = threadIdx.x; it < total; it += T) {
    const int j = qdiv(it, A.mg_nl, A.nl), line = it - (int)__umul24(j, A.nl);
    float2* e = lds + line + __umul24(j, A.ps);
    dif_regs<R>(v, tw, __umul24(j, S.tws), last);
#pragma unroll
    for (int i = 0; i < R; ++i) e[i * st] = v[i];
    if (it + T < total) load(it + T);
  }
}

// Last inverse z stage: LDS -> global plane.
template <int R>
__device__ __forceinline__ void st_store(float2* lds, float2* g, const Axis& A, const TpStage& S, const float2* tw,
                                         int T) {
  const int nb = uni(S.nb), total = uni(A.nl * (A.L / R)), st = uni(nb * A.ps);
  const unsigned gs = 8u * (unsigned)uni(nb * A.nl);
  const bool last = nb == 1;
  for (int it = threadIdx.x; it < total; it += T) {
    const int j = qdiv(it, A.mg_nl, A.nl), line = it - (int)__umul24(j, A.nl);
    const float2* e = lds + line + __umul24(j, A.ps);
    float2 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = e[i * st];
    dit_regs<R>(v, tw, __umul24(j, S.tws), last);
#pragma unroll
    for (int i = 0; i < R; ++i) sto(g, 8u * (unsigned)it + i * gs, v[i]);
  }
}

// Last forward y stage, product, first inverse y stage (lines are z
// positions: consecutive lanes read consecutive kernel values).
template <int R>
__device__ __forceinline__ void st_mul(float2* lds, const float2* k, const Axis& A, int conj, int T) {
  const int total = uni(A.nl * (A.L / R));
  const unsigned ks = 8u * (unsigned)uni(A.nl);
  for (int it = threadIdx.x; it < total; it += T) {
    const int b = qdiv(it, A.mg_nl, A.nl), line = it - (int)__umul24(b, A.nl);
    const unsigned ko = 8u * (line + __umul24(b * R, A.nl));
    float2* e = lds + __umul24(line, A.ls) + b * R;
    float2 v[R], h[R];
#pragma unroll
    for (int i = 0; i < R; ++i) h[i] = ldo(k, ko + i * ks);
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = e[i];
    Dft<R, false>::run(v);
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = cmul(v[i], conj ? cconj(h[i]) : h[i]);
    Dft<R, true>::run(v);
#pragma unroll
    for (int i = 0; i < R; ++i) e[i] = v[i];
  }
}

#define TP_RADICES(X) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16)

template <bool INV>
__device__ __forceinline__ void lds_stage(float2* lds, const Axis& A, const TpStage& S, const float2* tw, int T) {
  switch (S.radix) {
#define X(r) \
  case r: st_lds<r, INV>(lds, A, S, tw, T); break;
    TP_RADICES(X)
#undef X
  }
}

}  // namespace tp

// Workgroup -> (job, tile).  Workgroups go round robin over the eight XCDs,
// each with its own L2; tiles are dealt so that each XCD takes a contiguous
// run of them, in order: neighbouring x tiles write neighbouring parts of
// the same lines, which then meet in one L2.
__device__ __forceinline__ int find_tp(const TpJob* __restrict__ jobs, int njobs, bool x, int& local) {
  const int n = (int)gridDim.x, c8 = (n + 7) >> 3, r8 = n & 7;
  const int xcd = (int)blockIdx.x & 7, i8 = (int)blockIdx.x >> 3;
  // XCDs 0 .. r8 - 1 get c8 workgroups, the others one less (all c8 when r8 = 0)
  int t = r8 == 0 || xcd < r8 ? xcd * c8 + i8 : r8 * c8 + (xcd - r8) * (c8 - 1) + i8;
  if (njobs == 1) {
    local = t;
    return 0;
  }
  for (int j = 0; j < njobs; ++j) {
    const int c = x ? jobs[j].nz * jobs[j].atiles : jobs[j].yz_tiles;
    if (t < c) {
      local = t;
      return j;
    }
    t -= c;
  }
  local = 0;
  return -1;
}

// ---------------------------------------------------------------------------
// x pass of the two-pass form: MODE 0 R2C of psi, 1 blur -> ratio -> R2C, 2
// back-projection -> update -> R2C, 3 fold into the combined factor, 4 last
// fold and combined update -> R2C.  A workgroup holds the a R rows
// y1 + m n1 (a consecutive y1, m < R) at one z; each wave transforms RPW of
// them; the R-point y transforms and the half-spectrum arithmetic run on the
// workgroup's rows between two barriers.  Rows in LDS have an odd pitch, and
// the lanes of the spectrum phases take k in steps of ks (a where the range
// of k divides well), so neither the row stages nor those phases pile up on
// a bank.
// LDS pitch of a row: odd
constexpr int tp_row_pitch(int M) { return M | 1; }

// Item `it` of the spectrum phases: y1 offset yi and kx k of a pair (k, M - k);
// false outside the tile.
template <int M>
__device__ __forceinline__ bool tp_item(const TpJob& J, int it, int n, int t, int& yi, int& k) {
  const int c = tp::qdiv(it, J.mg_a, J.a), h = tp::qdiv(c, J.mg_kg, J.kg);
  yi = it - (int)__umul24(c, J.a);
  k = (int)__umul24(c - (int)__umul24(h, J.kg), J.ks) + h;
  return it < n && k < M / 2 + 1 && t * J.a + yi < J.n1;
}

// Spectrum of the tile's rows -> the packed rows' M-point spectra in LDS.
// The first round of loads is issued before the barrier that completes the
// workgroup's tables.
template <int M, int R>
__device__ __forceinline__ void tp_gather(const TpJob& J, float2* rows, const float2* s_pp, const float2* s_wr,
                                          const float2* spec, int z, int t, int T) {
  constexpr int U = R >= 4 ? 1 : R >= 2 ? 2 : 4;  // items in flight
  constexpr int PM = tp_row_pitch(M);
  const int a = J.a, n = a * J.kg * J.ks, rs = tp::uni(a * PM);
  const unsigned ps = 8u * (unsigned)(J.nz * J.n1), o0 = 8u * (unsigned)(z * J.n1 + t * a);
  float2 xa[U][R], xb[U][R];
  int yi[U], kk[U];
  auto load = [&](int it0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int k;
      kk[u] = tp_item<M>(J, it0 + u * T, n, t, yi[u], k) ? k : -1;
      if (kk[u] >= 0) {
        const unsigned o = o0 + 8u * (unsigned)yi[u], ko = (unsigned)k * (R * ps);
        const unsigned oa = o + ko, ob = o + (M * R * ps - ko);
#pragma unroll
        for (int j = 0; j < R; ++j) {
          xa[u][j] = tp::ldo(spec, oa + j * ps);
          xb[u][j] = tp::ldo(spec, ob + j * ps);
        }
      }
    }
  };
  load(threadIdx.x);
  __syncthreads();
  for (int it0 = threadIdx.x; it0 < n; it0 += U * T) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = kk[u];
      if (k < 0) continue;
#pragma unroll
      for (int j = 1; j < R; ++j) {
        const float2 w = cconj(s_wr[yi[u] * R + j]);
        xa[u][j] = cmul(xa[u][j], w);
        xb[u][j] = cmul(xb[u][j], w);
      }
      if constexpr (R > 1) {
        Dft<R, true>::run(xa[u]);
        Dft<R, true>::run(xb[u]);
      }
      const float2 tw = cconj(s_pp[k]);
      float2* r0 = rows + __umul24(yi[u], PM);
#pragma unroll
      for (int m = 0; m < R; ++m) {
        float2* row = r0 + m * rs;
        const float2 p = xa[u][m], q = xb[u][m];
        // Z[k] = (p + conj q) + i e, e = conj(t) (p - conj q); the mirrored
        // product t (q - conj p) is -conj e, so Z[M-k] needs no second one
        const float2 s = make_float2(p.x + q.x, p.y - q.y);
        const float2 e = cmul(tw, make_float2(p.x - q.x, p.y + q.y));
        row[k] = make_float2(s.x - e.y, s.y + e.x);
        if (k != 0 && 2 * k != M) row[M - k] = make_float2(s.x + e.y, e.x - s.y);
      }
    }
    if (it0 + U * T < n) load(it0 + U * T);
  }
}

// The packed rows' M-point spectra in LDS -> the tile's part of the spectrum.
template <int M, int R>
__device__ __forceinline__ void tp_scatter(const TpJob& J, const float2* rows, const float2* s_pp, const float2* s_wr,
                                           float2* spec, int z, int t, int T) {
  constexpr int PM = tp_row_pitch(M);
  const int a = J.a, n = a * J.kg * J.ks, rs = tp::uni(a * PM);
  const unsigned ps = 8u * (unsigned)(J.nz * J.n1), o0 = 8u * (unsigned)(z * J.n1 + t * a);
  for (int it = threadIdx.x; it < n; it += T) {
    int yi, k;
    if (!tp_item<M>(J, it, n, t, yi, k)) continue;
    float2 xa[R], xb[R];
    const float2 tw = s_pp[k];
    const float2* r0 = rows + __umul24(yi, PM);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const float2* row = r0 + m * rs;
      const float2 zk = row[k];
      if (k == 0) {
        xa[m] = make_float2(2.f * (zk.x + zk.y), 0.f);
        xb[m] = make_float2(2.f * (zk.x - zk.y), 0.f);
      } else {
        // 2 X[k] = s - i e, e = t (z_k - conj z_(M-k)) (the kernel spectra
        // hold the 1/2); the mirrored product is -conj e
        const float2 zm = row[M - k];
        const float2 s = make_float2(zk.x + zm.x, zk.y - zm.y);
        const float2 e = cmul(tw, make_float2(zk.x - zm.x, zk.y + zm.y));
        xa[m] = make_float2(s.x + e.y, s.y - e.x);
        xb[m] = make_float2(s.x - e.y, -(s.y + e.x));
      }
    }
    if constexpr (R > 1) {
      Dft<R, false>::run(xa);
      Dft<R, false>::run(xb);
    }
    const unsigned o = o0 + 8u * (unsigned)yi;
    const unsigned ko = (unsigned)k * (R * ps), oa = o + ko, ob = o + (M * R * ps - ko);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j > 0) {
        const float2 w = s_wr[yi * R + j];
        xa[j] = cmul(xa[j], w);
        xb[j] = cmul(xb[j], w);
      }
      tp::sto(spec, oa + j * ps, xa[j]);
      if (2 * k != M) tp::sto(spec, ob + j * ps, xb[j]);
    }
  }
}

// Pointwise step on the last inverse x stage's registers (see RowOp in
// mvd_ct_passes.h); ro[i] is the volume offset of the row of butterfly slot
// i, negative for rows outside the tile.
template <int MODE, int PITCH, int MAXB, int R>
struct TpOp {
  float2* buf;
  const float2 (&pa)[MAXB][R];
  const float2 (&pb)[MAXB][R];
  const int (&ro)[MAXB];
  float* psi;
  float* acc;
  bool weighted, first, geo;
  float eps, lamp, inv_n;
  double flux;
  unsigned ncr, ncn;
  bool bad;
  static constexpr bool lds = true;
  __device__ __forceinline__ void st(int line, int pos, float2 z, int i, int r) {
    const bool ok = ro[i] >= 0;
    const unsigned g = 4u * (unsigned)(ro[i] + 2 * pos);
    float2 o;
    if (MODE == 1) {
      unsigned n = 0;
      o = ratio2(pa[i][r], z, eps, n);
      ncr += ok ? n : 0u;
    } else {
      ncn += ok ? (z.x < 0.f) + (z.y < 0.f) : 0;
      const float cx = z.x > 0.f ? z.x : 0.f, cy = z.y > 0.f ? z.y : 0.f;
      if (MODE == 2) {
        const float2 p = pa[i][r];
        const float tx = tikhonov(p.x * cx, lamp), ty = tikhonov(p.y * cy, lamp);
        o = weighted ? make_float2(p.x + pb[i][r].x * (tx - p.x), p.y + pb[i][r].y * (ty - p.y))
                     : make_float2(tx, ty);
      } else {
        float mx = cx, my = cy;
        if (!first) {
          mx = geo ? pa[i][r].x * cx : pa[i][r].x + cx;
          my = geo ? pa[i][r].y * cy : pa[i][r].y + cy;
        }
        if (MODE == 3) {
          o = make_float2(mx, my);
          if (ok) tp::sto(reinterpret_cast<float2*>(acc), g, o);
        } else {
          const float gx = geo ? powf(mx, inv_n) : mx * inv_n;
          const float gy = geo ? powf(my, inv_n) : my * inv_n;
          o = make_float2(tikhonov(pb[i][r].x * gx, lamp), tikhonov(pb[i][r].y * gy, lamp));
        }
      }
      if ((MODE == 2 || MODE == 4) && ok) {
        tp::sto(reinterpret_cast<float2*>(psi), g, o);
        flux += (double)o.x + (double)o.y;
        bad |= !(isfinite(o.x) && isfinite(o.y));
      }
    }
    buf[__umul24((unsigned)line, PITCH) + pos] = o;
  }
};

// A wave's rows in LDS.
template <int PITCH>
struct TpRow {
  float2* p;
  static constexpr bool lds = true;
  __device__ __forceinline__ float2 ld(int line, int pos) const { return p[__umul24((unsigned)line, PITCH) + pos]; }
  __device__ __forceinline__ void st(int line, int pos, float2 v) const {
    p[__umul24((unsigned)line, PITCH) + pos] = v;
  }
};

#define TP_SPLITS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9)

template <int MODE, int RPW, int M, int... Rs>
__global__ void __launch_bounds__(64 * TP_MAX_WAVES)
    k_xpass_tp(const TpJob* __restrict__ jobs, int njobs, const float2* __restrict__ twp, int v,
               Partial* __restrict__ parts, int* __restrict__ flags, int opt) {
  constexpr int PM = tp_row_pitch(M);
  constexpr int RL = LastRadix<Rs...>::value;
  using LM = LastMap<M, RL, 64, RPW, false, true>;
  extern __shared__ float2 dyn[];
  __shared__ double rf[TP_MAX_WAVES];
  __shared__ unsigned rc[TP_MAX_WAVES];
  int local;
  const int jid = find_tp(jobs, njobs, true, local);
  if (jid < 0) return;
  const TpJob& J = jobs[jid];
  const int T = blockDim.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (MODE != 0 && v >= J.nviews) {
    if (tid == 0 && parts) {
      if (MODE == 1)
        parts[blockIdx.x].ratio_clamps = 0;
      else
        parts[blockIdx.x].flux = 0.0, parts[blockIdx.x].neg_clamps = 0;
    }
    return;
  }
  const int RW = (T >> 6) * RPW;
  float2* s_tw = dyn + RW * PM;
  float2* s_pp = s_tw + M;
  float2* s_wr = s_pp + M;
  const int z = local / J.atiles, t = local - z * J.atiles;
  const int a = J.a, R = J.R, n1 = J.n1;
  for (int i = tid; i < M; i += T) {
    s_tw[i] = ldg(twp + J.tw_x + i);
    s_pp[i] = ldg(twp + J.pp + i);
  }
  for (int i = tid; i < a * R; i += T) {  // W_ny^(y1 j), i = yi R + j
    const int yi = tp::qdiv(i, J.mg_R, R), j = i - (int)__umul24(yi, R);
    const int e = (int)__umul24(t * a + yi, j);  // < ny where the row is valid
    s_wr[i] = ldg(twp + J.tw_y + (e < J.ny ? e : 0));
  }
  float2* spec = reinterpret_cast<float2*>(J.spec);
  const TpRow<PM> L{dyn + wave * RPW * PM};
  const bool first = opt & XOPT_FIRST, geo = opt & XOPT_GEO;
  double flux = 0.0;
  unsigned ncr = 0, ncn = 0;
  bool bad = false;
  // volume offset of row `line` of this wave, -1 outside the tile
  auto row_of = [&](int line) {
    const int rho = wave * RPW + line, m = tp::qdiv(rho, J.mg_a, a), y1 = t * a + rho - (int)__umul24(m, a);
    return (m < R && y1 < n1) ? (z * J.ny + y1 + m * n1) * J.nx : -1;
  };

  if constexpr (MODE == 0) {
    constexpr int R1 = FirstRadix<Rs...>::value;
    constexpr int MB = FirstMap<M, R1, 64, RPW>::MAXB;
    constexpr int NB = M / R1;
    float2 in[MB][R1];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int it = lane + i * 64, line = it / NB, j = it % NB;
      const int o = it < NB * RPW ? row_of(line) : -1;
#pragma unroll
      for (int r = 0; r < R1; ++r) in[i][r] = o >= 0 ? ld2(J.psi + o + 2 * (j + r * NB)) : make_float2(0.f, 0.f);
    }
    __syncthreads();  // tables
    Plain<TpRow<PM>> out{L};
    CtRun<false, M, 64, RPW, false, SYNC_WAVE24, 1, true, Rs...>::run(lane, s_tw, RegSrc<MB, R1>{in}, L, out);
  } else {
    // operands of the pointwise step, in the order the last inverse stage
    // produces its outputs
    float2 pa[LM::MAXB][RL], pb[LM::MAXB][RL];
    int ro[LM::MAXB];
    const float* opa = MODE == 1 ? J.phi + (int64_t)v * J.V : MODE == 2 ? J.psi : (first ? nullptr : J.acc);
    const float* opb = MODE == 2 ? (J.w ? J.w + (int64_t)v * J.V : nullptr) : MODE == 4 ? J.psi : nullptr;
#pragma unroll
    for (int i = 0; i < LM::MAXB; ++i) {
      int line, j;
      const bool ok = LM::at(lane, i, line, j);
      ro[i] = ok ? row_of(line) : -1;
      // rows outside the tile read row 0 and are ignored
      const unsigned g = 4u * (unsigned)(max(ro[i], 0) + 2 * j);
      if (opa)
#pragma unroll
        for (int r = 0; r < RL; ++r) pa[i][r] = tp::ldo(reinterpret_cast<const float2*>(opa), g + 8 * r * LM::NB);
      if ((MODE == 2 || MODE == 4) && opb)
#pragma unroll
        for (int r = 0; r < RL; ++r) pb[i][r] = tp::ldo(reinterpret_cast<const float2*>(opb), g + 8 * r * LM::NB);
    }
    switch (R) {
#define X(r) \
  case r: tp_gather<M, r>(J, dyn, s_pp, s_wr, spec, z, t, T); break;
      TP_SPLITS(X)
#undef X
    }
    __syncthreads();
    TpOp<MODE, PM, LM::MAXB, RL> op{L.p,  pa,    pb,  ro,    J.psi,  J.acc, opb != nullptr, first, geo,
                                    J.eps, J.lamp, 1.f / (float)J.nviews, 0.0, 0u, 0u, false};
    CtRun<true, M, 64, RPW, false, SYNC_WAVE24, 1, true, Rs...>::run(lane, s_tw, L, L, op);
    flux = op.flux;
    ncr = op.ncr;
    ncn = op.ncn;
    bad = op.bad;
    if (MODE != 3) {
      Plain<TpRow<PM>> out{L};
      CtRun<false, M, 64, RPW, false, SYNC_WAVE24, 1, true, Rs...>::run(lane, s_tw, L, L, out);
    }
  }
  if (MODE != 3) {
    __syncthreads();
    switch (R) {
#define X(r) \
  case r: tp_scatter<M, r>(J, dyn, s_pp, s_wr, spec, z, t, T); break;
      TP_SPLITS(X)
#undef X
    }
  }
  if (MODE != 0) {
    if ((MODE == 2 || MODE == 4) && bad) atomicOr(flags, 1);
    if (parts) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        if (MODE == 1) {
          ncr += __shfl_xor(ncr, o);
        } else {
          flux += __shfl_xor(flux, o);
          ncn += __shfl_xor(ncn, o);
        }
      }
      if (lane == 0) {
        if (MODE == 1)
          rc[wave] = ncr;
        else
          rf[wave] = flux, rc[wave] = ncn;
      }
      __syncthreads();
      if (tid == 0) {
        flux = 0.0;
        ncr = ncn = 0;
        for (int i = 0; i < (T >> 6); ++i) {
          if (MODE == 1)
            ncr += rc[i];
          else
            flux += rf[i], ncn += rc[i];
        }
        if (MODE == 1)
          parts[blockIdx.x].ratio_clamps = ncr;
        else
          parts[blockIdx.x].flux = flux, parts[blockIdx.x].neg_clamps = ncn;
      }
    }
  }
}

}  // namespace mvdk
