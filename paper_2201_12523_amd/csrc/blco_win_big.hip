// Instantiations of the window MTTKRP kernel (blco_win.h): 64-bit gather addresses.
#include "blco_win.h"

KernelFn blco::select_win_big(int N, int R, int fdt, bool stash, int wpt) {
  return fdt == BLCO_F32 ? select_win_t<float, true>(N, R, false, stash, wpt)
                         : select_win_t<uint16_t, true>(N, R, R % 2 == 0, stash, wpt);
}
