// Instantiations of the window MTTKRP kernel (blco_win.h): bf16 factors.
#include "blco_win.h"

KernelFn blco::select_win_bf16(int N, int R, bool even, bool stash, int wpt) {
  return select_win_t<uint16_t, false>(N, R, even, stash, wpt);
}
