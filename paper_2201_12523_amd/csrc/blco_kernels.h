// Launch parameters and kernel selection shared by the device translation units of the
// BLCO library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace blco {

constexpr int kWaves = 4;             // waves per workgroup
constexpr int kBlock = kWaves * 64;   // threads per workgroup

// Everything a launch over one contiguous range of non-zeros needs.
struct KParams {
  const uint64_t* keys;   // keys[0] is global non-zero `base`
  const float* vals;
  int64_t base;           // global index of keys[0]; a multiple of 64
  int64_t n;              // non-zeros in this launch
  const int64_t* run_start;   // runs of equal block key (global indices)
  const uint32_t* run_base;   // nruns x N: high bits of each mode, in place
  const int32_t* tile_run;    // global tile -> run of its first non-zero
  int multi;                  // more than one run (else every base is 0)
  const void* A[8];           // factor matrices (A[mode] unused by MTTKRP)
  float* out;                 // MTTKRP: I_mode x R; loss: residual (nnz)
  float* resid;               // fused residual walk: residual of each non-zero (n)
  double* partials;           // loss: one fp64 partial sum per workgroup
  int R;                      // MTTKRP: elements between output rows; loss: ranks
  int RV;                     // window kernel: ranks to flush (R, or fewer: output padding)
  int RG;                     // window kernel: ranks to gather (RV, or more: zeros)
  int mode;
  uint32_t shift[8];
  uint32_t mask[8];
  const uint32_t* hot;        // window kernel: frequent rows of the target mode
  int nhot;                   // window kernel: frequent rows held in the LDS stash
  const uint32_t* tab;        // window kernel, hot copies: the target mode's row table
  int64_t copy_off;           // ... bytes from out to the copies: copies x copy_stride floats per row
  int copies;                 // ... copies of a row (a power of two)
  int copy_stride;            // ... floats of one copy
  int out_copies;             // window kernel: copies of the output (a power of two)
  int64_t out_step;           // ... elements from one to the next
  uint32_t short_rows;        // hierarchical kernel: target mode length
  int short_width;            // hierarchical kernel: ranks per slice
  uint32_t rowbytes;          // bytes between factor rows
  uint32_t abytes[8];         // bytes of each factor matrix (clamped to 2^32 - 1)
  float scale;                // host-side scale of every term
  const double* scale_dev;    // optional device-side scale (one double)
};

typedef void (*KernelFn)(KParams);

// The window kernel for N modes and R ranks to gather: fp32 factors, bf16 factors, 64-bit
// gather addresses (factor type fdt), and the fused CP-gradient walk.  even: factor rows lie
// an even number of elements apart (vector gathers of bf16 ranks); stash: frequent rows
// apart; wpt: window size (non-zeros per thread, or minus the threads per non-zero).
KernelFn select_win_f32(int N, int R, bool stash, int wpt);
KernelFn select_win_bf16(int N, int R, bool even, bool stash, int wpt);
KernelFn select_win_big(int N, int R, int fdt, bool stash, int wpt);
KernelFn select_res(int N, int R, bool even, int fdt, bool stash, int wpt);

}  // namespace blco
