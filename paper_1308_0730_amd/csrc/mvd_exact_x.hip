// x passes of the sequential scheme (modes 0-2) with compile-time plans for
// every 5-smooth half-row length (lists in mvd_exact_lengths.h); the modes
// of the combined updates are in mvd_exact_x_comb.hip.  A launch covers jobs
// whose nx / 2 is the plan's length.
#include "mvd_ct_passes.h"
#include "mvd_exact_lengths.h"

using namespace mvdk;

int mvd_exact_row_shape(int M, int* waves, int* rows) {
  switch (M) {
#define X(m, wpb, rpw, ...) \
  case m:                   \
    *waves = wpb;           \
    *rows = rpw;            \
    return 1;
    MVD_EXACT_ROW(X)
#undef X
    default:
      return 0;
  }
}

// The ratio pass may take other radices than the update, at the same rows per
// wave (gen_exact_lengths.py): 360 points 73 -> 60 us, 432 points 401 -> 340 us,
// 480 and 500 points 10 % faster; with them the update pass is up to 45 %
// slower (more than 128 registers).  The forward pass (mode 0) keeps the
// update's: a run continued from a saved estimate then starts from the bits
// of the spectrum that the update would have left.
#define XK(md, m, wpb, rpw, ...)                                                                               \
  k_xpass_ct<md, wpb, rpw, m, __VA_ARGS__><<<a.grid, 64 * wpb, 0, a.stream>>>(a.jobs, a.njobs, a.plans, a.tw, \
                                                                             v, parts, flags, opt)

static hipError_t launch_ratio(const LaunchArgs& a, int M, int v, Partial* parts, int* flags, int opt) {
  switch (M) {
#define X(m, wpb, rpw, ...)          \
  case m:                            \
    XK(1, m, wpb, rpw, __VA_ARGS__); \
    break;
    MVD_EXACT_ROW_FWD(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t mvd_launch_x_exact(const LaunchArgs& a, int M, int mode, int v, Partial* parts, int* flags, int opt) {
  if (mode == 3 || mode == 4) return mvd_launch_x_exact_comb(a, M, mode, v, parts, flags, opt);
  if (mode & XMODE_WIN) return mvd_launch_x_exact_win(a, M, mode, v, parts, flags, opt);
  if (mode == 1) return launch_ratio(a, M, v, parts, flags, opt);
  if (mode != 0 && mode != 2) return hipErrorInvalidValue;
  switch (M) {
#define X(m, wpb, rpw, ...)            \
  case m:                              \
    if (mode == 0)                     \
      XK(0, m, wpb, rpw, __VA_ARGS__); \
    else                               \
      XK(2, m, wpb, rpw, __VA_ARGS__); \
    break;
    MVD_EXACT_ROW(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
