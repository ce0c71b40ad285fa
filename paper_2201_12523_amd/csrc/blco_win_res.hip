// Instantiations of the window MTTKRP kernel (blco_win.h): the fused CP-gradient walk.
#include "blco_win.h"

KernelFn blco::select_res(int N, int R, bool even, int fdt, bool stash, int wpt) {
  return fdt == BLCO_F32 ? select_res_t<float>(N, R, false, stash, wpt)
                         : select_res_t<uint16_t>(N, R, even, stash, wpt);
}
