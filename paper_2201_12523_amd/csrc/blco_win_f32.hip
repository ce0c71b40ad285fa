// Instantiations of the window MTTKRP kernel (blco_win.h): fp32 factors.
#include "blco_win.h"

KernelFn blco::select_win_f32(int N, int R, bool stash, int wpt) {
  return select_win_t<float, false>(N, R, false, stash, wpt);
}
