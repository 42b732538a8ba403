// x passes of the two-pass convolution that write no volume (modes 0 and 1)
// for every 5-smooth half-row length of the range; the update is in
// mvd_tp_x_update.hip, the combined modes are in mvd_tp_x_comb.hip.
#include "mvd_exact_lengths.h"
#include "mvd_two_pass.h"

using namespace mvdk;

// Half-row lengths with two-pass kernels: the row plans of up to TP_MAX_M
// points.
int mvd_tp_row(int M, int* rows, size_t* lds_row) {
  switch (M) {
#define X(m, rpw, ...)                                      \
  case m:                                                   \
    *rows = rpw;                                            \
    *lds_row = (size_t)tp_row_pitch(m) * sizeof(float2);    \
    return 1;
    MVD_TP_ROW(X)
#undef X
    default:
      return 0;
  }
}

hipError_t mvd_launch_x_tp(const TpArgs& a, int M, int waves, size_t lds, int mode, int v, Partial* parts, int* flags,
                           int opt) {
  if (mode >= 3) return mvd_launch_x_tp_comb(a, M, waves, lds, mode, v, parts, flags, opt);
  if (mode == 2) return mvd_launch_x_tp_update(a, M, waves, lds, v, parts, flags, opt);
  switch (M) {
#define XM(md, m, rpw, ...)                                                                                   \
  case md:                                                                                                    \
      k_xpass_tp<md, rpw, m, __VA_ARGS__><<<a.grid, 64 * waves, lds, a.stream>>>(a.jobs, a.njobs, a.tw, v,    \
                                                                                 parts, flags, opt);          \
    break;
#define X(m, rpw, ...)                  \
  case m:                               \
    switch (mode) {                     \
      XM(0, m, rpw, __VA_ARGS__)        \
      XM(1, m, rpw, __VA_ARGS__)        \
      default:                          \
        return hipErrorInvalidValue;    \
    }                                   \
    break;
    MVD_TP_ROW(X)
#undef X
#undef XM
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
