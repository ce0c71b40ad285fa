// The window MTTKRP kernel (register-based conflict resolution) and the device helpers it
// shares with the other kernels of the BLCO library (gfx950, wave64).  Included by
// blco_device.hip (helpers) and by the translation units that instantiate the window
// kernel (blco_win_*.hip), compiled in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "blco_internal.h"
#include "blco_kernels.h"

using namespace blco;

template <typename FT>
__device__ __forceinline__ float ld_factor(const void* A, size_t i);

template <>
__device__ __forceinline__ float ld_factor<float>(const void* A, size_t i) {
  return static_cast<const float*>(A)[i];
}

template <>
__device__ __forceinline__ float ld_factor<uint16_t>(const void* A, size_t i) {
  return __uint_as_float((uint32_t)static_cast<const uint16_t*>(A)[i] << 16);
}

// Coordinates of one non-zero: kept bits by shift and mask, the rest from
// the block key of the run that holds it (Figure 6b).
template <int N>
__device__ __forceinline__ void decode(const KParams& p, uint64_t key, int64_t gidx,
                                       uint32_t (&c)[N]) {
  uint32_t base[N];
#pragma unroll
  for (int m = 0; m < N; ++m) base[m] = 0;
  if (p.multi) {
    int run = p.tile_run[gidx >> 6];
    while (gidx >= p.run_start[run + 1]) ++run;
#pragma unroll
    for (int m = 0; m < N; ++m) base[m] = p.run_base[(size_t)run * N + m];
  }
#pragma unroll
  for (int m = 0; m < N; ++m) c[m] = ((uint32_t)(key >> p.shift[m]) & p.mask[m]) | base[m];
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float term_scale(const KParams& p) {
  return p.scale_dev ? (float)((double)p.scale * p.scale_dev[0]) : p.scale;
}

constexpr int kWin = 1024;     // threads of the window kernel
constexpr int kWinRounds = 4;  // dispatch rounds of the persistent window kernel
constexpr int kWinBits = 10;
#ifndef BLCO_WIN_U
#define BLCO_WIN_U 8
#endif
// minimum waves per SIMD requested from the compiler: 8 lets two 1024-thread
// workgroups share a CU (measured about 1.7x faster than one)
#ifndef BLCO_WIN_OCC
#define BLCO_WIN_OCC 8
#endif

constexpr int kBucketBits = 12;
constexpr int kBuckets = 1 << kBucketBits;   // hash buckets per 1024-non-zero window

// In-place exclusive prefix sum of NB counters in LDS by a workgroup of NT
// threads (NB a multiple of NT): per-thread serial sums, a wave scan by
// cross-lane shifts, and one LDS pass over the per-wave totals.
template <int NB, int NT>
__device__ __forceinline__ void block_exclusive_scan(uint32_t* a, int tid, uint32_t* wsum) {
  constexpr int PER = NB / NT;
  uint32_t v[PER];
  uint32_t tot = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v[i] = a[tid * PER + i];
    tot += v[i];
  }
  const int lane = tid & 63;
  uint32_t inc = tot;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == 63) wsum[tid >> 6] = inc;
  __syncthreads();
  // the earlier waves' totals: one per lane of a 16-lane row, summed across the row (a
  // loop over them is a chain of up to 15 LDS reads)
  static_assert(NT <= 1024, "at most 16 waves");
  uint32_t wbase = (lane & 15) < (tid >> 6) ? wsum[lane & 15] : 0u;
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) wbase += (uint32_t)__shfl_xor((int)wbase, off);
  uint32_t run = wbase + inc - tot;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    a[tid * PER + i] = run;
    run += v[i];
  }
  __syncthreads();
}

// Lane q of this lane's 16-lane row (DPP row_newbcast), and the value of the
// lane q places further along the row (DPP row_shl).  q must fold to a
// constant where they are called (unrolled loops).
__device__ __forceinline__ uint32_t row_bcast(uint32_t v, int q) {
  switch (q) {
    case 0: return __builtin_amdgcn_update_dpp(0u, v, 0x150, 0xF, 0xF, false);
    case 1: return __builtin_amdgcn_update_dpp(0u, v, 0x151, 0xF, 0xF, false);
    case 2: return __builtin_amdgcn_update_dpp(0u, v, 0x152, 0xF, 0xF, false);
    case 3: return __builtin_amdgcn_update_dpp(0u, v, 0x153, 0xF, 0xF, false);
    case 4: return __builtin_amdgcn_update_dpp(0u, v, 0x154, 0xF, 0xF, false);
    case 5: return __builtin_amdgcn_update_dpp(0u, v, 0x155, 0xF, 0xF, false);
    case 6: return __builtin_amdgcn_update_dpp(0u, v, 0x156, 0xF, 0xF, false);
    case 7: return __builtin_amdgcn_update_dpp(0u, v, 0x157, 0xF, 0xF, false);
    case 8: return __builtin_amdgcn_update_dpp(0u, v, 0x158, 0xF, 0xF, false);
    case 9: return __builtin_amdgcn_update_dpp(0u, v, 0x159, 0xF, 0xF, false);
    case 10: return __builtin_amdgcn_update_dpp(0u, v, 0x15A, 0xF, 0xF, false);
    case 11: return __builtin_amdgcn_update_dpp(0u, v, 0x15B, 0xF, 0xF, false);
    case 12: return __builtin_amdgcn_update_dpp(0u, v, 0x15C, 0xF, 0xF, false);
    case 13: return __builtin_amdgcn_update_dpp(0u, v, 0x15D, 0xF, 0xF, false);
    case 14: return __builtin_amdgcn_update_dpp(0u, v, 0x15E, 0xF, 0xF, false);
    default: return __builtin_amdgcn_update_dpp(0u, v, 0x15F, 0xF, 0xF, false);
  }
}
__device__ __forceinline__ uint32_t row_shl(uint32_t v, int q) {
  switch (q) {
    case 1: return __builtin_amdgcn_update_dpp(0u, v, 0x101, 0xF, 0xF, false);
    case 2: return __builtin_amdgcn_update_dpp(0u, v, 0x102, 0xF, 0xF, false);
    case 3: return __builtin_amdgcn_update_dpp(0u, v, 0x103, 0xF, 0xF, false);
    case 4: return __builtin_amdgcn_update_dpp(0u, v, 0x104, 0xF, 0xF, false);
    case 5: return __builtin_amdgcn_update_dpp(0u, v, 0x105, 0xF, 0xF, false);
    case 6: return __builtin_amdgcn_update_dpp(0u, v, 0x106, 0xF, 0xF, false);
    case 7: return __builtin_amdgcn_update_dpp(0u, v, 0x107, 0xF, 0xF, false);
    case 8: return __builtin_amdgcn_update_dpp(0u, v, 0x108, 0xF, 0xF, false);
    case 9: return __builtin_amdgcn_update_dpp(0u, v, 0x109, 0xF, 0xF, false);
    case 10: return __builtin_amdgcn_update_dpp(0u, v, 0x10A, 0xF, 0xF, false);
    case 11: return __builtin_amdgcn_update_dpp(0u, v, 0x10B, 0xF, 0xF, false);
    case 12: return __builtin_amdgcn_update_dpp(0u, v, 0x10C, 0xF, 0xF, false);
    case 13: return __builtin_amdgcn_update_dpp(0u, v, 0x10D, 0xF, 0xF, false);
    case 14: return __builtin_amdgcn_update_dpp(0u, v, 0x10E, 0xF, 0xF, false);
    default: return __builtin_amdgcn_update_dpp(0u, v, 0x10F, 0xF, 0xF, false);
  }
}

// target row of a record (field N - 1 of the record at LDS offset `at`)
__device__ __forceinline__ uint32_t seg_target(const uint32_t* rec, int at, int mode, int N) {
  (void)mode;
  return rec[at + N - 1];
}
constexpr uint32_t kBufFlags = 0x00020000u;  // raw buffer resource word 3 (gfx9 family)

// Factor-row gathers.  Raw buffer loads with a 32-bit byte offset (row * row
// bytes + rank offset) when every factor is below 4 GiB: no 64-bit address
// arithmetic, and the descriptor's size bound drops stray offsets.  Larger
// factors take 64-bit global addresses (BIG).  (Structured, index-scaled
// buffer loads would cover both but measured 1.5-2x slower on gfx950.)
template <typename FT>
__device__ __forceinline__ float ld_buf(__amdgpu_buffer_rsrc_t r, uint32_t off, int more = 0);
template <>
__device__ __forceinline__ float ld_buf<float>(__amdgpu_buffer_rsrc_t r, uint32_t off, int more) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, more, 0));
}
template <>
__device__ __forceinline__ float ld_buf<uint16_t>(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                  int more) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, more, 0)
                         << 16);
}

// fp32 gathers of the window kernel at four ranks per lane (33-64 ranks): a global load
// from the factor's base (uniform, in scalar registers) plus the zero-extended 32-bit
// byte offset.  That reaches all of 4 GiB, so a factor of exactly 4 GiB (2^24 rows of 64
// ranks) keeps 32-bit offsets, where a buffer descriptor's 32-bit size stops one byte
// short.  Measured on the 4-mode 200M-non-zero workload at R = 64: 17.5 -> 15.1 ms on the
// mode that gathers such a factor (it took 64-bit addresses before), 15.7 -> 15.2 ms on
// its other frequent-row mode; at two ranks per lane the same loads were 5% slower on the
// frequent-row modes, so R <= 32 keeps buffer loads.
__device__ __forceinline__ float ld_base(const void* A, uint32_t off) {
  return *reinterpret_cast<const float*>(static_cast<const char*>(A) + off);
}

// RPL consecutive bf16 factor elements from byte offset off, widened to fp32: one
// 4- or 8-byte buffer load when VEC (every run starts 4-byte aligned: R is even), else
// RPL 2-byte loads.  Element k sits at the lower address, in the low half of its word.
template <int RPL, bool VEC>
__device__ __forceinline__ void ld_bf16_run(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                            float (&t)[RPL]) {
  if constexpr (RPL == 2 && VEC) {
    {
      const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
      t[0] = __uint_as_float(v << 16);
      t[1] = __uint_as_float(v & 0xFFFF0000u);
      return;
    }
  } else if constexpr (RPL == 4 && VEC) {
    {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
      t[0] = __uint_as_float(v[0] << 16);
      t[1] = __uint_as_float(v[0] & 0xFFFF0000u);
      t[2] = __uint_as_float(v[1] << 16);
      t[3] = __uint_as_float(v[1] & 0xFFFF0000u);
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < RPL; ++k) t[k] = ld_buf<uint16_t>(r, off + 2u * (uint32_t)k);
}

// The same run through a 64-bit address (a factor of 4 GiB or more), which has no
// bounds check: only elements with act[k] set (ranks below R) are read, so a run that
// ends past the last row stays inside the factor.  VEC reads RPL / 2 four-byte words
// (runs start 4-byte aligned and R is even, so a word is read whole or not at all).
template <int RPL, bool VEC>
__device__ __forceinline__ void ld_bf16_run_ptr(const uint16_t* src, const bool (&act)[RPL],
                                                float (&t)[RPL]) {
  if constexpr (VEC && RPL % 2 == 0) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(src);
#pragma unroll
    for (int q = 0; q < RPL / 2; ++q) {
      const uint32_t v = act[2 * q] ? w[q] : 0u;
      t[2 * q] = __uint_as_float(v << 16);
      t[2 * q + 1] = __uint_as_float(v & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int k = 0; k < RPL; ++k) t[k] = act[k] ? ld_factor<uint16_t>(src, (size_t)k) : 0.f;
  }
}

// Adds a lane group's segment sums to one output row.  base + e is the slice's first
// rank of that row (E: uint32_t where element indices fit it, which saves 64-bit
// additions); ranks from nvalid on are not written.  Lane rl of the group holds
// ranks rl, rl + LPN, ... (fp32 factors), or with PACKED the RPL consecutive ranks
// RPL * rl, ... (bf16 factors).
//
// MI355X performs these atomics at the memory side, one request per aligned 64 bytes an
// instruction touches, so what counts is that each instruction covers one aligned
// segment.  ALIGNED (16-lane groups, R a multiple of 16 and a 64-byte-aligned output):
// the j-th instruction adds ranks 16 j .. 16 j + 15 where they lie.  Else the sums are
// first moved along the group by the row's misalignment s, so that the j-th instruction
// covers the j-th aligned segment the row touches: a row of R = 31 takes 2.9 requests
// instead of 3.9, one of 33 ranks 3.1 instead of 5 (measured on 5M non-zeros of a 3-mode
// power-law tensor, unmoved: R = 31 0.36 ms per mode, R = 33 0.48 ms, where R = 32 took
// 0.19 ms and R = 64 0.36 ms).  Groups of 64 lanes cover 256 bytes at a time and stay as
// they lie.
template <int RPL, int LPN, bool PACKED, bool ALIGNED, typename E>
__device__ __forceinline__ void flush_row(float* base, E e, const float (&a)[RPL], float scale,
                                          int rl, int nvalid) {
  if constexpr (!PACKED && (ALIGNED || LPN != 16)) {
    float* dst = base + (E)(e + (E)rl);
#pragma unroll
    for (int k = 0; k < RPL; ++k)
      if (ALIGNED || rl + k * LPN < nvalid) unsafeAtomicAdd(dst + k * LPN, a[k] * scale);
  } else {
    const int s = (ALIGNED || LPN != 16)
                      ? 0
                      : (int)(((uint32_t)(reinterpret_cast<uintptr_t>(base) >> 2) + (uint32_t)e) & 15);
    float* dst = base + (E)(e + (E)rl);   // rank rl; the segments begin s ranks before
    constexpr int SEG = (ALIGNED || LPN != 16) ? RPL : RPL + 1;
    if constexpr (PACKED) {
#pragma unroll
      for (int j = 0; j < SEG; ++j) {
        const int q = rl + j * LPN - s;
        const int src = q < 0 ? 0 : q / RPL;
        float v = 0.f;
#pragma unroll
        for (int s2 = 0; s2 < RPL; ++s2) {
          const float t2 = __shfl(a[s2], src & (LPN - 1), LPN);
          if (s2 == q - src * RPL) v = t2;
        }
        if (q >= 0 && q < nvalid) unsafeAtomicAdd(dst + (j * LPN - s), v * scale);
      }
    } else {
      float rot[RPL];
#pragma unroll
      for (int k = 0; k < RPL; ++k) rot[k] = __shfl(a[k], (rl - s) & 15, 16);
#pragma unroll
      for (int j = 0; j < SEG; ++j) {
        const int q = rl + j * 16 - s;
        const float v = rl >= s ? rot[j < RPL ? j : 0] : rot[j > 0 ? j - 1 : 0];
        if (q >= 0 && q < nvalid) unsafeAtomicAdd(dst + (j * 16 - s), v * scale);
      }
    }
  }
}

// Frequent-row lookup of the window kernel: open addressing over kHotSlots
// LDS slots holding (row, stash index); at most half full.
constexpr int kHotSlots = 2 * blco::kHotMax;
constexpr uint32_t kNoRow = 0xFFFFFFFFu;
constexpr uint32_t kHotFlag = 0x80000000u;   // record target field: stash index follows

__device__ __forceinline__ uint32_t hot_hash(uint32_t row) {
  return (row * 0x9E3779B1u) >> (32 - 9);   // 9 bits: kHotSlots = 512
}

__device__ __forceinline__ int hot_lookup(const uint32_t* keys, const uint32_t* idx, uint32_t row) {
  uint32_t h = hot_hash(row);
  for (int probe = 0; probe < kHotSlots; ++probe) {
    const uint32_t k = keys[h];
    if (k == row) return (int)idx[h];
    if (k == kNoRow) return -1;
    h = (h + 1) & (kHotSlots - 1);
  }
  return -1;
}

// Frequent rows of the larger windows (hot copies, below): a direct-mapped table of
// kTabSlots entries, so a look-up is one LDS read.
__device__ __forceinline__ uint32_t tab_slot(uint32_t row, uint32_t mult) {
  return (row * mult) >> (32 - blco::kTabBits);
}

// BLCO MTTKRP with register-based conflict resolution (Sections 5.1-5.2) over
// windows of 1024 * WPT consecutive non-zeros; persistent workgroups take windows
// in turn (see below)
//   processing: WPT non-zeros per thread are loaded (the next window's load is
//     issued before the current walk) and decoded by shift and mask; the
//     window is grouped by target with a counting sort (LDS histogram with
//     atomic ranks, exclusive scan, scatter) on a hash of the target, so each
//     target's terms form one contiguous segment, and each grouped position
//     gets a record: byte offsets of the other modes' factor rows, target,
//     value;
//   computing: groups of LPN lanes (RPL ranks per lane) walk LPN consecutive
//     grouped positions each (records read from LDS, or for N = 3 held one
//     per lane and passed along the group by DPP row broadcasts),
//     gathering factor rows with buffer loads and
//     summing the scaled Hadamard products in registers; a segment that ends
//     inside the group is flushed once per rank; a segment that crosses into
//     later groups is completed by the group it started in, from partial sums
//     the later groups leave in LDS.
// A flush is a device-scope atomic into the output, which MI355X performs at
// the memory side (same-address updates serialise at about 32 ns), except for
// the mode's frequent rows (found at build time): those get buckets of their
// own, so each has exactly one segment per window, and its flush is a plain
// add into the workgroup's LDS stash row; the stash goes to the output with
// one atomic per (row, rank) when the workgroup ends.
//
// RES (the fused CP-gradient walk, one rank slice): the values are the data x_k,
// and each position also gathers its target row, so the walk forms the model
// xhat_k = sum_r prod_m A^(m)[i_m^k, r] (a sum over the 16 lanes of the group),
// the residual e_k = x_k - xhat_k, which it writes to p.resid in BLCO order, and
// sums e_k * prod_{m != mode} A^(m) instead of x_k * prod_{m != mode} A^(m).
//
// WPT: non-zeros per thread, so a window holds kWin * WPT non-zeros; -1, -2 and -4: windows
// of kWin, kWin / 2 and kWin / 4 non-zeros; the walk of the last two has only 8 or 4
// positions per lane group, all gathered at once.  win_wpt (blco_device.hip) chooses.
//
// Windows of 2048 at three or four ranks per lane, without a stash, add to p.out_copies copies of
// the whole output by window number, which k_unpad adds up (out_copies, blco_device.hip).
//
// STASH with another WPT than 1: hot copies.  A frequent row (one LDS read per non-zero
// finds it; the full stash probes its table) is flushed to one of p.copies copies of
// it in a workspace, by window number, which k_hot_sum adds to the output afterwards.
// That is there for the sums' accuracy, and shortens the chains of same-row atomics:
// straight to the output each of the hottest rows is one fp32 addition per window, 10^5
// of them on 200M non-zeros, whose roundings put 5.5e-6 of the output's norm on that
// tensor's first mode (64-bit reference) against 0.9e-6 with the full stash.  Sums made in
// LDS first need workgroups that stay for many windows, which costs more than the
// atomics they save (that mode: 8.6 ms with the full stash, 6.9 ms with none).
template <int LPN, int RPL, typename FT, int N, bool BIG, bool STASH, bool RES = false,
          bool VEC = false, int WPT = 1>
__global__ __launch_bounds__(kWin, (WPT >= 4 || WPT < -1) ? 4 : BLCO_WIN_OCC) void k_mttkrp_win(
    KParams p) {
  constexpr bool SMALL = WPT < -1;              // fewer non-zeros than threads
  constexpr bool COPIES = STASH && WPT != 1;    // hot copies
  constexpr int W = WPT < 0 ? kWin / -WPT : kWin * WPT;   // non-zeros per window
  constexpr int PER = WPT < 0 ? 1 : WPT;        // non-zeros per thread
  constexpr int G = kWin / LPN;                 // groups of LPN lanes
  constexpr int PPG = W / G;                    // grouped positions per group (= LPN * WPT)
  static_assert(PPG <= 64, "a group's segment ends must fit one 64-bit word");
  static_assert(!COPIES || (!SMALL && !BIG), "hot copies: 32-bit offsets, whole windows");
  // hash buckets: four per non-zero up to 1024, 6144 per 2048 (two workgroups per CU keep
  // fitting in LDS), 12288 per 4096
  constexpr int NB = W <= kWin ? 4 * W : WPT == 2 ? kBuckets * 3 / 2 : kBuckets * 3;
  static_assert(NB % kWin == 0, "the scan takes NB / kWin buckets per thread");
  // positions whose gathers are issued together: BLCO_WIN_U / RPL, except for
  // 3-mode tensors at one or four ranks per lane, where 4 and 1 positions keep
  // the registers from spilling and measured 8% and 3% faster; the fused
  // residual walk also gathers the target row and keeps the value, the
  // residual and the position of each, so it takes half as many (at four it
  // spilled about 45 registers per lane; 4-mode 80M-non-zero CP gradient step
  // 13.1 -> 12.0 ms)
  constexpr int UW0 = (N == 3 && RPL == 1) ? 4 : (N == 3 && RPL == 4) ? 1 : BLCO_WIN_U / RPL;
  // small windows: every position of a group at once up to 8 (one workgroup per CU, so
  // registers allow it)
  constexpr int UW = SMALL ? (RPL >= 3 ? 4 : 8) : RES ? (UW0 > 1 ? UW0 / 2 : 1) : UW0;
  constexpr int U = PPG < UW ? PPG : UW;
  // record fields: the other modes' row offsets, target, value; with RES also the
  // position in the window and, where the target field cannot give it (full stash), the
  // target row's offset
  constexpr bool TOFF = RES && STASH && !COPIES;
  constexpr int NF = TOFF ? N + 3 : RES ? N + 2 : N + 1;
  constexpr int NP = NF <= 4 ? 4 : ((NF + 1) / 2) * 2;
  static_assert(!RES || (LPN == 16 && !BIG), "fused residual walk: 16-lane groups, 32-bit offsets");
  // bf16 factors: each lane holds RPL consecutive ranks, so one 4- or 8-byte load
  // gathers them when R is even (VEC; measured 14% faster per mode on 200M
  // non-zeros), 2-byte loads otherwise; fp32 keeps ranks LPN apart, whose 4-byte
  // loads measured faster than 8- and 16-byte ones
  constexpr bool PACKED = sizeof(FT) == 2 && RPL > 1;
  static_assert(!VEC || PACKED, "vector gathers are for packed bf16 ranks");
  // fp32 gathers at three or four ranks per lane: ld_base instead of buffer loads
  constexpr bool BASE32 = sizeof(FT) == 4 && LPN == 16 && RPL >= 3 && !RES && !BIG;
  // the record's target field holds the row's first element (row * R, below 2^32) where
  // that is all the flush needs: one 32-bit add and a shifted 64-bit add instead of two
  // quarter-rate 64-bit multiplies per flush.  With hot copies a frequent row has the top
  // bit set (kHotFlag) over the first element of its copy; with RES, which also needs the
  // row's offset, the field holds the row (and kHotFlag).  The full stash's field holds
  // the row, or kHotFlag and its stash index.
  constexpr bool IDX = !BIG && !RES && (!STASH || COPIES);
  __shared__ __align__(16) uint32_t s_rec[W * NP];  // records by grouped position
  __shared__ uint64_t s_end[W / 64];
  // the histogram (processing) and the carry partial sums (computing) are never
  // live at once: they share one array
  constexpr int NHH = NB > kWin * RPL ? NB : kWin * RPL;
  __shared__ __align__(16) uint32_t s_hist[NHH];
  float* s_head = reinterpret_cast<float*>(s_hist);
  __shared__ uint32_t s_wsum[kWin / 64];
  extern __shared__ __align__(16) unsigned char s_dyn_win[];
  // frequent rows in the full stash; without it one window per workgroup
  constexpr bool FULLSTASH = STASH && !COPIES;
  const int K = FULLSTASH ? p.nhot : 0;
  // hot copies: the row table, and this window's copy
  __shared__ uint32_t s_tkey[COPIES ? kTabSlots : 1];
  __shared__ __align__(4) uint8_t s_tidx[COPIES ? kTabSlots : 4];
  uint32_t tmult = 0;
  if constexpr (COPIES) {
    tmult = p.tab[0];
    for (int i = threadIdx.x; i < kTabSlots; i += kWin) s_tkey[i] = p.tab[1 + i];
    if (threadIdx.x < kTabSlots / 4)
      reinterpret_cast<uint32_t*>(s_tidx)[threadIdx.x] = p.tab[1 + kTabSlots + threadIdx.x];
  }
  // first element of this window's copy of frequent row i
  auto copy_elem = [&](uint32_t i) {
    return (i * (uint32_t)p.copies + (uint32_t)(blockIdx.x & (uint32_t)(p.copies - 1))) *
           (uint32_t)p.copy_stride;
  };
  // the copy of the output that this window adds to
  constexpr bool OUTS = !BIG && !RES && !STASH && LPN == 16 && RPL >= 3 && WPT == 2;
  float* const out =
      OUTS ? p.out + (int64_t)(blockIdx.x & (uint32_t)(p.out_copies - 1)) * p.out_step : p.out;
  const int R = p.R;
  const int RV = p.RV, RG = p.RG;
  float* s_stash = reinterpret_cast<float*>(s_dyn_win);   // K x R
  uint32_t* s_hkey = reinterpret_cast<uint32_t*>(s_stash + (size_t)K * R);
  uint32_t* s_hidx = s_hkey + kHotSlots;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int64_t nwin = (p.n + W - 1) / W;
  if (K > 0) {
    for (int i = tid; i < K * R; i += kWin) s_stash[i] = 0.f;
    for (int i = tid; i < kHotSlots; i += kWin) s_hkey[i] = kNoRow;
    __syncthreads();
    if (tid < K) {
      const uint32_t row = p.hot[tid];
      uint32_t h = hot_hash(row);
      for (int probe = 0; probe < kHotSlots; ++probe) {
        if (atomicCAS(&s_hkey[h], kNoRow, row) == kNoRow) {
          s_hidx[h] = (uint32_t)tid;
          break;
        }
        h = (h + 1) & (kHotSlots - 1);
      }
    }
  }
  // windows of this workgroup: blockIdx.x, blockIdx.x + gridDim.x, ...
  const int64_t wstep = gridDim.x;
  // the first window's non-zeros of this thread: window positions tid + i * kWin
  uint64_t nkey[PER];
  float nx[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    nkey[i] = 0;
    nx[i] = 0.f;
    const int64_t k = (int64_t)blockIdx.x * W + tid + i * kWin;
    if ((!SMALL || tid < W) && (int64_t)blockIdx.x < nwin && k < p.n) {
      nkey[i] = p.keys[k];
      nx[i] = p.vals[k];
    }
  }
  constexpr int NO = N > 1 ? N - 1 : 1;          // other modes
  __amdgpu_buffer_rsrc_t rs[NO];
  const void* ap[NO];
#pragma unroll
  for (int j = 0; j + 1 < N; ++j) {
    const int m = (j < p.mode) ? j : j + 1;
    ap[j] = p.A[m];
    rs[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.A[m]), 0, (int)p.abytes[m],
                                              (int)kBufFlags);
  }
  // the target mode's factor (read by the fused residual walk only)
  const __amdgpu_buffer_rsrc_t rs_t = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.A[RES ? p.mode : 0]), 0, RES ? (int)p.abytes[p.mode] : 0,
      (int)kBufFlags);
  const float scale = term_scale(p);
  const int g = tid / LPN;
  const int rl = tid % LPN;
  const int p0 = g * PPG;
  const uint64_t gmask = PPG >= 64 ? ~0ULL : ((1ULL << PPG) - 1);

  for (int64_t win = blockIdx.x; win < nwin; win += wstep) {
    const int64_t k0 = win * W;
    const int nvalid = (int)min((int64_t)W, p.n - k0);

    // ---- processing: decode, group by target
    uint32_t c[PER][N], tgt[PER], tfield[PER], bkt[PER], rank[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int wp = tid + i * kWin;   // position in the window
      if (wp < nvalid) {
        decode<N>(p, nkey[i], p.base + k0 + wp, c[i]);
      } else {
#pragma unroll
        for (int m = 0; m < N; ++m) c[i][m] = 0;
      }
      tgt[i] = 0;
#pragma unroll
      for (int m = 0; m < N; ++m)
        if (m == p.mode) tgt[i] = c[i][m];
    }
    for (int i = tid; i < NB; i += kWin) s_hist[i] = 0;
    __syncthreads();   // also: the stash lookup is built, the previous window is done
    // counting sort on a hash of the target; a frequent row has bucket = its
    // stash index, the other targets share the remaining buckets (two targets
    // sharing a bucket may interleave, which only splits a segment)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const bool valid = tid + i * kWin < nvalid;
      tfield[i] = IDX ? tgt[i] * (uint32_t)R : tgt[i];
      const int hs = (FULLSTASH && K > 0 && valid) ? hot_lookup(s_hkey, s_hidx, tgt[i]) : -1;
      if constexpr (COPIES) {
        const uint32_t slot = tab_slot(tgt[i], tmult);
        if (s_tkey[slot] == tgt[i]) tfield[i] = kHotFlag | (RES ? tgt[i] : copy_elem(s_tidx[slot]));
      }
      if (hs >= 0) {
        bkt[i] = (uint32_t)hs;
        tfield[i] = kHotFlag | (uint32_t)hs;
      } else {
        const uint32_t h = tgt[i] * 0x9E3779B1u;
        bkt[i] = (uint32_t)K + (uint32_t)(((uint64_t)h * (uint32_t)(NB - K)) >> 32);
      }
      rank[i] = valid ? atomicAdd(&s_hist[bkt[i]], 1u) : 0u;
    }
    __syncthreads();
    block_exclusive_scan<NB, kWin>(s_hist, tid, s_wsum);
    // record at the grouped position: fields 0..N-2 the byte offsets (row
    // indices when BIG) of the other modes' factor rows in ascending mode
    // order, field N-1 the target field, field N the value; padding positions
    // (nvalid and above) stay where they are
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int wp = tid + i * kWin;
      if (SMALL && wp >= W) continue;
      const int pos = wp < nvalid ? (int)(s_hist[bkt[i]] + rank[i]) : wp;
#pragma unroll
      for (int j = 0; j + 1 < N; ++j) {
        const uint32_t cj = (j < p.mode) ? c[i][j] : c[i][j + 1];
        s_rec[pos * NP + j] = BIG ? cj : cj * p.rowbytes;
      }
      s_rec[pos * NP + N - 1] = tfield[i];
      s_rec[pos * NP + N] = __float_as_uint(wp < nvalid ? nx[i] : 0.f);
      if constexpr (RES) {
        s_rec[pos * NP + NF - 1] = (uint32_t)wp;
        if constexpr (TOFF) s_rec[pos * NP + N + 1] = tgt[i] * p.rowbytes;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int wp = tid + i * kWin;
      if (SMALL && wp >= W) continue;   // whole waves: W is a multiple of 64
      const uint32_t t0 = s_rec[wp * NP + N - 1];
      const bool end = (wp < nvalid) && (wp == nvalid - 1 || s_rec[(wp + 1) * NP + N - 1] != t0);
      const uint64_t em = __ballot(end);
      if (lane == 0) s_end[wp >> 6] = em;
    }
    // the next window's non-zeros, in flight during this walk
    if constexpr (FULLSTASH) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int64_t k = (win + wstep) * W + tid + i * kWin;
        if (win + wstep < nwin && k < p.n) {
          nkey[i] = p.keys[k];
          nx[i] = p.vals[k];
        }
      }
    }
    __syncthreads();

    // ---- computing: LPN lanes per group, RPL ranks per lane (lane j holds
    // ranks j, j + LPN, ... for fp32 factors, ranks RPL*j .. RPL*j + RPL - 1 for
    // bf16), each group walking LPN consecutive positions
    using EndT = std::conditional_t<(PPG <= 32), uint32_t, uint64_t>;
    const EndT endw = (EndT)(s_end[p0 >> 6] >> (p0 & 63));
    const bool starts_before =
        p0 > 0 && p0 < nvalid && !((s_end[(p0 - 1) >> 6] >> ((p0 - 1) & 63)) & 1);
    const bool can_carry = p0 + PPG <= nvalid;
    // 3-mode tensors with 16-lane groups (one DPP row per group): the walk
    // takes record fields from registers.  Lane rl of a group starts with the
    // record of the group's position rl; each step of U positions broadcasts
    // lanes 0..U-1 of the row and then shifts the row down by U lanes.  (For
    // other mode counts the extra registers cost more than the LDS reads save.)
    constexpr bool kRowB = (LPN == 16) && (N == 3) && !SMALL;
    // a frequent row's segment sums into its stash row (one owner per window)
    auto stash_add = [&](uint32_t tf, const float (&a)[RPL], int r0) {
      float* srow = s_stash + (size_t)(tf & ~kHotFlag) * R + r0 + (PACKED ? rl * RPL : rl);
#pragma unroll
      for (int k = 0; k < RPL; ++k)
        if (r0 + (PACKED ? rl * RPL + k : rl + k * LPN) < RV) srow[PACKED ? k : k * LPN] += a[k];
    };
    // adds a segment of target field tf to its row
    auto flush = [&](uint32_t tf, const float (&a)[RPL], auto whole_c, int r0) {
      constexpr bool WHOLE = decltype(whole_c)::value;
      const int nv = min(RV - r0, LPN * RPL);
      if constexpr (COPIES) {
        const bool hot = tf & kHotFlag;
        uint32_t e = tf & ~kHotFlag;
        if constexpr (RES) e = hot ? copy_elem(s_tidx[tab_slot(e, tmult)]) : e * (uint32_t)R;
        // out plus a selected distance: of a choice between two pointers the compiler makes a
        // load of the chosen parameter at every flush, behind which the gathers wait
        float* base =
            reinterpret_cast<float*>(reinterpret_cast<char*>(p.out) + (hot ? p.copy_off : 0));
        flush_row<RPL, LPN, PACKED, WHOLE>(base, e + (uint32_t)r0, a, scale, rl, nv);
      } else if constexpr (IDX) {
        flush_row<RPL, LPN, PACKED, WHOLE>(out, tf + (uint32_t)r0, a, scale, rl, nv);
      } else {
        flush_row<RPL, LPN, PACKED, WHOLE>(p.out, (size_t)tf * R + r0, a, scale, rl, nv);
      }
    };
    // one slice of LPN * RPL ranks from r0 on.  FULL: every rank of the slice can be
    // gathered, by immediate offsets from one address per row and without masks.  WHOLE: also
    // every one of them is an output rank, and output rows are 64-byte aligned.
    auto walk = [&](auto full_c, auto whole_c, auto r0_c) {
      constexpr bool FULL = decltype(full_c)::value;
      const int r0 = r0_c;
      EndT ew = endw;
      uint32_t myrec[kRowB ? NF : 1];
      bool ract[RPL];
      uint32_t loff[RPL];
      float acc[RPL], carry[RPL];
#pragma unroll
      for (int k = 0; k < RPL; ++k) {
        const int r = PACKED ? r0 + rl * RPL + k : r0 + rl + k * LPN;
        ract[k] = r < RG;
        loff[k] = (uint32_t)(FULL || ract[k] ? r : 0) * (uint32_t)sizeof(FT);
        acc[k] = 0.f;
        carry[k] = 0.f;
      }
      bool first = true, has_carry = false;
      for (int q0 = 0; q0 < PPG; q0 += U) {
        if constexpr (kRowB) {
          // the records of the next LPN positions, one per lane
          if (q0 % LPN == 0) {
#pragma unroll
            for (int f = 0; f < NF; ++f) myrec[f] = s_rec[(p0 + q0 + rl) * NP + f];
          }
        }
        float pr[U][RPL];
        float ta[RES ? U : 1][RPL];
        float xs[RES ? U : 1];
        uint32_t wpos[RES ? U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // the record of position q0 + u: from the row, or from LDS
          uint32_t e[NF];
#pragma unroll
          for (int f = 0; f < NF; ++f)
            if (f != N - 1 || (RES && !TOFF)) {
              if constexpr (kRowB) e[f] = row_bcast(myrec[f], u);
            }
          const uint32_t* er = &s_rec[(p0 + q0 + u) * NP];
          const float xv = __uint_as_float(kRowB ? e[N] : er[N]);
#pragma unroll
          for (int k = 0; k < RPL; ++k) pr[u][k] = RES ? 1.f : xv;
          if constexpr (RES) {
            xs[u] = xv;
            constexpr int TF = TOFF ? N + 1 : N - 1;
            uint32_t toff = kRowB ? e[TF] : er[TF];
            if constexpr (!TOFF) toff = (toff & (COPIES ? ~kHotFlag : ~0u)) * p.rowbytes;
            wpos[u] = kRowB ? e[NF - 1] : er[NF - 1];
            if constexpr (PACKED) {
              ld_bf16_run<RPL, VEC>(rs_t, toff + loff[0], ta[u]);
            } else {
#pragma unroll
              for (int k = 0; k < RPL; ++k)
                ta[u][k] = FULL ? ld_buf<FT>(rs_t, toff + loff[0], k * LPN * (int)sizeof(FT))
                                : ld_buf<FT>(rs_t, toff + loff[k]);
            }
          }
#pragma unroll
          for (int j = 0; j + 1 < N; ++j) {
            const uint32_t f = kRowB ? e[j] : er[j];
            if constexpr (BIG && PACKED) {
              const FT* rowp = static_cast<const FT*>(ap[j]) + (size_t)f * R;
              float t3[RPL];
              ld_bf16_run_ptr<RPL, VEC>(rowp + loff[0] / sizeof(FT), ract, t3);
#pragma unroll
              for (int k = 0; k < RPL; ++k) pr[u][k] *= t3[k];
            } else if constexpr (BIG) {
              const FT* rowp = static_cast<const FT*>(ap[j]) + (size_t)f * R;
#pragma unroll
              for (int k = 0; k < RPL; ++k)
                pr[u][k] *= ld_factor<FT>(rowp, (size_t)(loff[k] / sizeof(FT)));
            } else if constexpr (PACKED) {
              float t3[RPL];
              ld_bf16_run<RPL, VEC>(rs[j], f + loff[0], t3);
#pragma unroll
              for (int k = 0; k < RPL; ++k) pr[u][k] *= t3[k];
            } else if constexpr (BASE32) {
#pragma unroll
              for (int k = 0; k < RPL; ++k)
                pr[u][k] *= FULL ? ld_base(static_cast<const float*>(ap[j]) + k * LPN, f + loff[0])
                                 : ld_base(ap[j], f + loff[k]);
            } else {
#pragma unroll
              for (int k = 0; k < RPL; ++k)
                pr[u][k] *= FULL ? ld_buf<FT>(rs[j], f + loff[0], k * LPN * (int)sizeof(FT))
                                 : ld_buf<FT>(rs[j], f + loff[k]);
            }
          }
        }
        if constexpr (RES) {
          // model at each position (sum over the group's 16 lanes), residual, and
          // the residual-scaled product of the other modes' rows
#pragma unroll
          for (int u = 0; u < U; ++u) {
            float part = 0.f;
#pragma unroll
            for (int k = 0; k < RPL; ++k)
              if (FULL || ract[k]) part += pr[u][k] * ta[u][k];
#pragma unroll
            for (int off = LPN / 2; off > 0; off >>= 1) part += __shfl_xor(part, off);
            const float ev = xs[u] - part;
#pragma unroll
            for (int k = 0; k < RPL; ++k) pr[u][k] *= ev;
            if (rl == 0 && (int)wpos[u] < nvalid) p.resid[k0 + wpos[u]] = ev;
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = q0 + u;
#pragma unroll
          for (int k = 0; k < RPL; ++k) acc[k] += pr[u][k];
          // shifted along instead of tested at bit q: the compiler hoists tests at constant
          // bits into scalar registers, one pair per position, and spills them
          const bool seg_end = ew & 1;
          ew >>= 1;
          if (seg_end || (q == PPG - 1 && can_carry)) {
            if (first && starts_before) {
#pragma unroll
              for (int k = 0; k < RPL; ++k) s_head[tid * RPL + k] = acc[k];
            } else if (seg_end) {
              const uint32_t tf = kRowB ? row_bcast(myrec[kRowB ? N - 1 : 0], u)
                                        : seg_target(s_rec, (p0 + q) * NP, p.mode, N);
              if (FULLSTASH && K > 0 && (tf & kHotFlag)) {
                stash_add(tf, acc, r0);
              } else {
                flush(tf, acc, whole_c, r0);
              }
            } else {
#pragma unroll
              for (int k = 0; k < RPL; ++k) carry[k] = acc[k];
              has_carry = true;
            }
#pragma unroll
            for (int k = 0; k < RPL; ++k) acc[k] = 0.f;
            first = false;
          }
        }
        if constexpr (kRowB) {
#pragma unroll
          for (int f = 0; f < NF; ++f) myrec[f] = row_shl(myrec[f], U);
        }
      }
      __syncthreads();
      if (has_carry) {
        // this group owns a segment that continues into the next groups
        for (int g2 = g + 1; g2 < G; ++g2) {
          const int q2 = g2 * PPG;
#pragma unroll
          for (int k = 0; k < RPL; ++k) carry[k] += s_head[(g2 * LPN + rl) * RPL + k];
          if ((s_end[q2 >> 6] >> (q2 & 63)) & gmask) break;
        }
        const uint32_t tf = seg_target(s_rec, (p0 + PPG - 1) * NP, p.mode, N);
        if (FULLSTASH && K > 0 && (tf & kHotFlag)) {
          stash_add(tf, carry, r0);
        } else {
          flush(tf, carry, whole_c, r0);
        }
      }
      __syncthreads();
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if constexpr (LPN == 16) {
      // one slice (RG <= 16 RPL): its first rank folds to 0
      using Zero = std::integral_constant<int, 0>;
      if constexpr (!BIG && !FULLSTASH) {
        if (RG != 16 * RPL)
          walk(No{}, No{}, Zero{});
        else if (RV == RG && R % 16 == 0 && (reinterpret_cast<uintptr_t>(p.out) & 63) == 0)
          walk(Yes{}, Yes{}, Zero{});
        else
          walk(Yes{}, No{}, Zero{});
      } else {
        walk(No{}, No{}, Zero{});
      }
    } else {
      for (int r0 = 0; r0 < R; r0 += LPN * RPL) walk(No{}, No{}, r0);
    }
    if constexpr (!FULLSTASH) break;
  }
  // ---- the stash of frequent rows: one atomic per (row, rank) that received a term
  if (K > 0) {
    __syncthreads();
    for (int i = tid; i < K * R; i += kWin) {
      const float v = s_stash[i];
      const int hr = i / R;
      if (v != 0.f) unsafeAtomicAdd(p.out + (size_t)p.hot[hr] * R + (i - hr * R), v * scale);
    }
  }
}

// ====================================================================== selection

// modes up to which windows of other than 1024 non-zeros are built
constexpr int kWideMaxN = 5;

template <int LPN, int RPL, typename FT, bool BIG, bool STASH, bool RES, bool VEC>
static KernelFn pick_many_n(int N) {
  switch (N) {
    case 6: return k_mttkrp_win<LPN, RPL, FT, 6, BIG, STASH, RES, VEC>;
    case 7: return k_mttkrp_win<LPN, RPL, FT, 7, BIG, STASH, RES, VEC>;
    default: return k_mttkrp_win<LPN, RPL, FT, 8, BIG, STASH, RES, VEC>;
  }
}

template <int LPN, int RPL, typename FT, bool BIG, bool STASH, bool RES, bool VEC>
static KernelFn pick_any_n(int N) {
  switch (N) {
    case 1: return k_mttkrp_win<LPN, RPL, FT, 1, BIG, STASH, RES, VEC>;
    case 2: return k_mttkrp_win<LPN, RPL, FT, 2, BIG, STASH, RES, VEC>;
    case 3: return k_mttkrp_win<LPN, RPL, FT, 3, BIG, STASH, RES, VEC>;
    case 4: return k_mttkrp_win<LPN, RPL, FT, 4, BIG, STASH, RES, VEC>;
    case 5: return k_mttkrp_win<LPN, RPL, FT, 5, BIG, STASH, RES, VEC>;
    default: return pick_many_n<LPN, RPL, FT, BIG, STASH, RES, VEC>(N);
  }
}

template <int RPL, typename FT, bool BIG, bool RES, bool VEC, int WPT, bool STASH = false>
static KernelFn pick_wide_n(int N) {
  switch (N) {
    case 1: return k_mttkrp_win<16, RPL, FT, 1, BIG, STASH, RES, VEC, WPT>;
    case 2: return k_mttkrp_win<16, RPL, FT, 2, BIG, STASH, RES, VEC, WPT>;
    case 3: return k_mttkrp_win<16, RPL, FT, 3, BIG, STASH, RES, VEC, WPT>;
    case 4: return k_mttkrp_win<16, RPL, FT, 4, BIG, STASH, RES, VEC, WPT>;
    default: break;
  }
  // the residual walk's windows of 2048 end at four modes (win_wpt)
  if constexpr (!(RES && WPT == 2))
    return k_mttkrp_win<16, RPL, FT, 5, BIG, STASH, RES, VEC, WPT>;
  return nullptr;
}

// 16-lane groups of RPL ranks per lane; wpt as win_wpt gives it.  Three ranks per lane have no
// full stash and no windows of 1024 (select_win_t); 64-bit addresses no small windows and, up to
// kWideMaxN modes, none of 1024 without a stash (win_wpt); copies have windows of 2048 (wide_pays).
template <int RPL, typename FT, bool BIG, bool VEC>
static KernelFn pick_win16(int N, bool stash, int wpt) {
  if constexpr (!BIG) {
    if (stash && wpt == 2) return pick_wide_n<RPL, FT, BIG, false, VEC, 2, true>(N);
  }
  if constexpr (RPL != 3)
    if (stash) return pick_any_n<16, RPL, FT, BIG, true, false, VEC>(N);
  if constexpr (!BIG) {
    if (wpt == -4) return pick_wide_n<RPL, FT, BIG, false, VEC, -4>(N);
    if (wpt == -2) return pick_wide_n<RPL, FT, BIG, false, VEC, -2>(N);
  }
  if (wpt == 2) return pick_wide_n<RPL, FT, BIG, false, VEC, 2>(N);
  if constexpr (RPL >= 3)
    if (wpt == 4) return pick_wide_n<RPL, FT, BIG, false, VEC, 4>(N);
  if constexpr (RPL == 3)
    return nullptr;
  else if constexpr (BIG)
    return pick_many_n<16, RPL, FT, BIG, false, false, VEC>(N);
  else
    return pick_any_n<16, RPL, FT, BIG, false, false, VEC>(N);
}

// Window kernel shape (lanes per non-zero x ranks per lane), chosen by measurement on
// the power-law workloads: R <= 16: 16 x 1; R <= 32: 16 x 2 (8 x 4 was 1.8x slower);
// fp32 up to 48 without a stash: 16 x 3; R <= 64: 16 x 4 (10% faster than 32 x 2);
// larger: 64 x 2 per pass over the rank.  A stash with wpt 1 is the full one.  VEC (vector gathers of packed bf16 ranks) only
// where the ranks are packed: bf16 factors, two or more ranks per lane, and rows an even
// number of elements apart.
template <typename FT, bool BIG>
static KernelFn select_win_t(int N, int R, bool even, bool stash, int wpt) {
  constexpr bool H = sizeof(FT) == 2;
  const bool vec = H && even;
  if (R <= 16) return pick_win16<1, FT, BIG, false>(N, stash, wpt);
  if (R <= 32)
    return vec ? pick_win16<2, FT, BIG, H>(N, stash, wpt) : pick_win16<2, FT, BIG, false>(N, stash, wpt);
  if constexpr (!H && !BIG)
    if (R <= 48 && wpt != 1) return pick_win16<3, FT, BIG, false>(N, stash, wpt);
  if (R <= 64)
    return vec ? pick_win16<4, FT, BIG, H>(N, stash, wpt) : pick_win16<4, FT, BIG, false>(N, stash, wpt);
  if (stash)
    return vec ? pick_any_n<64, 2, FT, BIG, true, false, H>(N)
               : pick_any_n<64, 2, FT, BIG, true, false, false>(N);
  return vec ? pick_any_n<64, 2, FT, BIG, false, false, H>(N)
             : pick_any_n<64, 2, FT, BIG, false, false, false>(N);
}

// the fused residual walk (16-lane groups, one rank slice of at most 64, 32-bit offsets)
template <int RPL, typename FT, bool VEC>
static KernelFn pick_res(int N, bool stash, int wpt) {
  if (stash && wpt == 2) return pick_wide_n<RPL, FT, false, true, VEC, 2, true>(N);
  // one non-zero per thread with copies: the walk's only long window at five modes (win_wpt)
  if (stash && wpt == -1) return k_mttkrp_win<16, RPL, FT, 5, false, true, true, VEC, -1>;
  if (stash) return pick_any_n<16, RPL, FT, false, true, true, VEC>(N);
  if (wpt == 2) return pick_wide_n<RPL, FT, false, true, VEC, 2>(N);
  if (wpt == -4) return pick_wide_n<RPL, FT, false, true, VEC, -4>(N);
  if (wpt == -2) return pick_wide_n<RPL, FT, false, true, VEC, -2>(N);
  return pick_any_n<16, RPL, FT, false, false, true, VEC>(N);
}

template <typename FT>
static KernelFn select_res_t(int N, int R, bool even, bool stash, int wpt) {
  constexpr bool H = sizeof(FT) == 2;
  const bool vec = H && even;
  if (R <= 16) return pick_res<1, FT, false>(N, stash, wpt);
  if (R <= 32) return vec ? pick_res<2, FT, H>(N, stash, wpt) : pick_res<2, FT, false>(N, stash, wpt);
  return vec ? pick_res<4, FT, H>(N, stash, wpt) : pick_res<4, FT, false>(N, stash, wpt);
}
