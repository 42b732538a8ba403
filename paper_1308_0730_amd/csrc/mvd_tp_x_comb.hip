// x passes of the two-pass convolution in the combined updates (modes 3, 4).
#include "mvd_exact_lengths.h"
#include "mvd_two_pass.h"

using namespace mvdk;

hipError_t mvd_launch_x_tp_comb(const TpArgs& a, int M, int waves, size_t lds, int mode, int v, Partial* parts,
                                int* flags, int opt) {
  switch (M) {
#define XM(md, m, rpw, ...)                                                                                   \
  case md:                                                                                                    \
      k_xpass_tp<md, rpw, m, __VA_ARGS__><<<a.grid, 64 * waves, lds, a.stream>>>(a.jobs, a.njobs, a.tw, v,    \
                                                                                 parts, flags, opt);          \
    break;
#define X(m, rpw, ...)                  \
  case m:                               \
    switch (mode) {                     \
      XM(3, m, rpw, __VA_ARGS__)        \
      XM(4, m, rpw, __VA_ARGS__)        \
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
