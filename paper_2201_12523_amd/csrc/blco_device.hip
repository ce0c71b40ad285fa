// Device runtime and gfx950 kernels of the BLCO sparse MTTKRP library.
//
// Method: Nguyen et al., "Efficient, Out-of-Memory Sparse MTTKRP on Massively
// Parallel Architectures", ICS '22.  Two MTTKRP kernels follow the processing /
// computing split of Section 5.1 (Figure 7), re-designed for wave64 and the
// memory-side atomics of MI355X:
//   k_mttkrp_win (register-based resolution, Section 5.2): one 1024-thread
//     workgroup per window of 256 to 4096 consecutive non-zeros (blco_win.h,
//     win_wpt).  Processing: each thread loads up to four (key, value) pairs
//     (coalesced), decodes the coordinates
//     by shift and mask (Figure 6b), and the window is grouped by target row
//     with a counting sort on a hash of the target (LDS histogram, workgroup
//     scan, scatter), so each target forms one segment; every grouped position
//     gets a record (byte offsets of the other modes' rows, target, value).
//     Computing: groups of 16 lanes (1-4 ranks per lane) walk the records,
//     gather the factor rows with raw buffer loads, sum the scaled Hadamard
//     products in registers while the target repeats, and add each finished
//     segment to the output with one atomic per rank.  A mode's frequent rows
//     (found at build time) go to copies in the call's workspace instead, or,
//     without one, to an LDS stash flushed once per persistent workgroup.
//     The workspace also holds padded factors and output rows, copies of the
//     output, and the non-zeros of a flat mode moved to buckets of target rows
//     (plan_call).
//   k_mttkrp_short (hierarchical resolution, Section 5.1), which the Section
//     5.3 heuristic picks for modes shorter than the compute-unit count: each
//     workgroup keeps a private LDS copy of all target rows (a rank slice) and
//     adds it to the output once at its end.
// Also here: the sampled CP model / residual / fp64 loss kernels, the bf16
// cast, the out-of-memory streaming runtime and the C ABI of include/blco.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "blco_internal.h"
#include "blco_kernels.h"
#include "blco_win.h"

using namespace blco;

#define HIPCHK(expr)                                                                         \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return set_error(BLCO_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));         \
  } while (0)

// ====================================================================== device code

// Zero-fill of an output and of a second array (a kernel rather than a memset so the call
// can be captured).
__device__ __forceinline__ void zero_range(float* __restrict__ p, int64_t n, int64_t i,
                                           int64_t stride) {
  if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
    float4* q = reinterpret_cast<float4*>(p);
    int64_t n4 = n >> 2;
    for (int64_t j = i; j < n4; j += stride) q[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t j = (n4 << 2) + i; j < n; j += stride) p[j] = 0.f;
  } else {
    for (int64_t j = i; j < n; j += stride) p[j] = 0.f;
  }
}

// What a call does before its main kernel, in one launch: clears the output and the hot
// copies, copies factors into rows of Rp elements (zeros from R on), and sets the cursors
// of the grouping to the buckets' starts.
struct PrepParams {
  float* zero[2];
  int64_t nzero[2];
  int npad;                // factors to copy
  const void* src[8];
  void* dst[8];
  int64_t rows[8];
  int R, Rp;
  const uint32_t* starts;  // kGroupBuckets, or NULL
  uint32_t* cursor;
};

template <typename E>
__device__ __forceinline__ void pad_rows(const E* __restrict__ src, E* __restrict__ dst,
                                         int64_t rows, int R, int Rp, int64_t i, int64_t stride) {
  struct alignas(4 * sizeof(E)) Four { E v[4]; };
  const int q4 = Rp / 4;
  for (int64_t j = i; j < rows * q4; j += stride) {
    const int64_t row = j / q4;
    const int c = (int)(j - row * q4) * 4;
    Four f;
#pragma unroll
    for (int k = 0; k < 4; ++k) f.v[k] = c + k < R ? src[row * R + c + k] : E(0);
    reinterpret_cast<Four*>(dst)[j] = f;
  }
}

__global__ __launch_bounds__(256) void k_prep(PrepParams p, int bf16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int z = 0; z < 2; ++z)
    if (p.nzero[z] > 0) zero_range(p.zero[z], p.nzero[z], i, stride);
  for (int m = 0; m < p.npad; ++m) {
    if (bf16)
      pad_rows(static_cast<const uint16_t*>(p.src[m]), static_cast<uint16_t*>(p.dst[m]), p.rows[m],
               p.R, p.Rp, i, stride);
    else
      pad_rows(static_cast<const float*>(p.src[m]), static_cast<float*>(p.dst[m]), p.rows[m], p.R,
               p.Rp, i, stride);
  }
  if (p.starts && i < kGroupBuckets) p.cursor[i] = p.starts[i];
}

// out (+)= the first R elements of every row of a padded output, or the sum of its copies (in fp64).
// Added with atomics: calls on several streams may add to one output.
__global__ __launch_bounds__(256) void k_unpad(const float* __restrict__ src, int64_t rows, int R,
                                               int Rp, int copies, int64_t step, int add,
                                               float* __restrict__ out) {
  const int64_t n = rows * R, stride = (int64_t)gridDim.x * 256;
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += stride) {
    const int64_t row = j / R;
    const float* at = src + row * Rp + (j - row * R);
    float v = at[0];
    if (copies > 1) {
      double a = (double)v;
      for (int c = 1; c < copies; ++c) a += (double)at[c * step];
      v = (float)a;
    }
    if (add)
      unsafeAtomicAdd(out + j, v);
    else
      out[j] = v;
  }
}

// Distinct rows of mode blockIdx.y in sampled window blockIdx.x (flush_start), into counts[m][0] (the
// window's first half) and counts[m][1]: a set of rows in LDS, at most half full.
__global__ __launch_bounds__(1024) void k_flushes(KParams p, uint32_t* __restrict__ counts) {
  constexpr uint32_t kSlots = 2 * kFlushWindow;
  __shared__ uint32_t s_slot[kSlots];
  __shared__ uint32_t s_n[2];
  const int m = (int)blockIdx.y, N = (int)gridDim.y;
  const int64_t k0 = flush_start(p.n, (int)blockIdx.x);
  for (uint32_t i = threadIdx.x; i < kSlots; i += 1024) s_slot[i] = 0xFFFFFFFFu;
  if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    for (int i = threadIdx.x; i < kFlushWindow / 2; i += 1024) {
      const int64_t k = k0 + half * (kFlushWindow / 2) + i;
      uint32_t row = (uint32_t)(p.keys[k] >> p.shift[m]) & p.mask[m];
      if (p.multi) {
        int run = p.tile_run[k >> 6];
        while (k >= p.run_start[run + 1]) ++run;
        row |= p.run_base[(size_t)run * N + m];
      }
      if (row == 0xFFFFFFFFu) row = 0xFFFFFFFEu;   // the empty slot's mark
      uint32_t h = (row * 0x9E3779B1u) >> 19;      // 13 bits: kSlots
      for (uint32_t probe = 0; probe < kSlots; ++probe) {
        const uint32_t was = atomicCAS(&s_slot[h], 0xFFFFFFFFu, row);
        if (was == 0xFFFFFFFFu) {
          if (half == 0) atomicAdd(&s_n[0], 1u);
          atomicAdd(&s_n[1], 1u);
        }
        if (was == 0xFFFFFFFFu || was == row) break;
        h = (h + 1) & (kSlots - 1);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 2) atomicAdd(&counts[2 * m + threadIdx.x], s_n[threadIdx.x]);
}

// Bucket of a target row: equal ranges of rows.
__device__ __forceinline__ uint32_t group_bucket(uint32_t row, uint32_t mul) {
  return (uint32_t)(((uint64_t)row * mul) >> 32);
}

// Non-zeros of each bucket of one mode (a tensor of one run without block bits).
__global__ __launch_bounds__(256) void k_group_count(const uint64_t* __restrict__ keys, int64_t n,
                                                     int shift, uint32_t mask, uint32_t mul,
                                                     uint32_t* __restrict__ counts) {
  __shared__ uint32_t s_c[kGroupBuckets];
  for (int i = threadIdx.x; i < kGroupBuckets; i += 256) s_c[i] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride)
    atomicAdd(&s_c[group_bucket((uint32_t)(keys[i] >> shift) & mask, mul)], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kGroupBuckets; i += 256)
    if (s_c[i]) atomicAdd(&counts[i], s_c[i]);
}

// counts -> starts, in place (one workgroup).
__global__ __launch_bounds__(kGroupBuckets) void k_group_starts(uint32_t* __restrict__ c) {
  __shared__ uint32_t s_c[kGroupBuckets];
  __shared__ uint32_t s_wsum[kGroupBuckets / 64];
  const int tid = threadIdx.x;
  s_c[tid] = c[tid];
  __syncthreads();
  block_exclusive_scan<kGroupBuckets, kGroupBuckets>(s_c, tid, s_wsum);
  c[tid] = s_c[tid];
}

// Moves keys and values to their target row's bucket.  Without it a mode whose rows hardly
// repeat inside a window makes one memory-side atomic row-update per non-zero (4M non-zeros
// of 300007 x 200003 x 100003, R = 100: 1.53 ms per mode, all of it atomics); in bucket
// order a window holds few rows, each many times.  A workgroup takes kGroupPer keys per
// thread, ranks them inside each bucket with LDS counters, reserves its places with one
// atomic per bucket, and writes them where they go: runs of a bucket are short, but the
// workgroups' runs adjoin, so the L2 completes the lines.
constexpr int kGroupPer = 16;
__global__ __launch_bounds__(1024) void k_group(const uint64_t* __restrict__ keys,
                                                const float* __restrict__ vals, int64_t n,
                                                int shift, uint32_t mask, uint32_t mul,
                                                uint32_t* __restrict__ cursor,
                                                uint64_t* __restrict__ gkeys,
                                                float* __restrict__ gvals) {
  __shared__ uint32_t s_c[kGroupBuckets];
  const int tid = threadIdx.x;
  static_assert(kGroupBuckets == 1024, "one bucket per thread");
  s_c[tid] = 0;
  const int64_t k0 = (int64_t)blockIdx.x * (1024 * kGroupPer) + tid;
  uint64_t key[kGroupPer];
  uint32_t at[kGroupPer];
#pragma unroll
  for (int i = 0; i < kGroupPer; ++i) {
    const int64_t k = k0 + (int64_t)i * 1024;
    key[i] = k < n ? keys[k] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGroupPer; ++i) {
    const uint32_t b = group_bucket((uint32_t)(key[i] >> shift) & mask, mul);
    at[i] = k0 + (int64_t)i * 1024 < n ? atomicAdd(&s_c[b], 1u) : 0u;
  }
  __syncthreads();
  const uint32_t c = s_c[tid];
  const uint32_t base = c ? atomicAdd(&cursor[tid], c) : 0u;
  __syncthreads();
  s_c[tid] = base;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGroupPer; ++i) {
    const int64_t k = k0 + (int64_t)i * 1024;
    if (k < n) {
      const uint32_t q = s_c[group_bucket((uint32_t)(key[i] >> shift) & mask, mul)] + at[i];
      gkeys[q] = key[i];
      gvals[q] = vals[k];
    }
  }
}

// Adds the copies of frequent row hot[blockIdx.x] to the output (see k_mttkrp_win): each
// thread sums every fourth copy of one rank in order, then the four partial sums meet.
__global__ __launch_bounds__(kBlock) void k_hot_sum(const float* __restrict__ copy,
                                                    const uint32_t* __restrict__ hot, int copies,
                                                    int stride, int RV, int R,
                                                    float* __restrict__ out) {
  __shared__ float s_part[kBlock];
  const int r = threadIdx.x & 63, q = threadIdx.x >> 6;   // RV <= 64
  const float* c = copy + (size_t)blockIdx.x * copies * stride;
  float a = 0.f;
  if (r < RV)
    for (int i = q; i < copies; i += 4) a += c[(size_t)i * stride + r];
  s_part[threadIdx.x] = a;
  __syncthreads();
  if (q == 0 && r < RV) {
    const float v = (s_part[r] + s_part[64 + r]) + (s_part[128 + r] + s_part[192 + r]);
    // atomic: calls on several streams may add to one output
    if (v != 0.f) unsafeAtomicAdd(out + (size_t)hot[blockIdx.x] * R + r, v);
  }
}

// ---------------------------------------------------------------------------
// BLCO MTTKRP with hierarchical conflict resolution (Section 5.1, steps 1-6),
// the mechanism the heuristic of Section 5.3 picks for short target modes.
//
// Each workgroup owns a contiguous range of the ALTO-ordered non-zeros and a
// slice of at most 64 ranks (blockIdx.y), and keeps a private copy of that
// slice of all I_n output rows in LDS (the stash; it covers every target row,
// so no lookup is needed).  Per batch of kShortB non-zeros:
//   processing: one non-zero per thread is loaded (coalesced) and decoded by
//     shift and mask; the batch is grouped by target row with a counting sort
//     (LDS histogram with atomic ranks, exclusive scan, scatter), and each
//     grouped position gets a record: byte offsets of the other modes' factor
//     rows, target row, value;
//   computing: each group of LPN lanes (RPL ranks per lane) walks LPN
//     consecutive grouped positions, kShortLoads / RPL at a time, gathering
//     the other modes' rows and summing the scaled Hadamard products in
//     registers while the target stays the same;
//   stash update: a target's positions form one run, so each run has one
//     owner, the group holding its first position.  A group whose first
//     segment continues a run from an earlier group leaves that partial sum
//     in a per-group carry slot; after a barrier the owner of a run that
//     crosses into later groups adds their carries.  Every owner then adds its
//     run's sum into the stash row with a plain LDS read-modify-write: no two
//     lanes touch one stash entry in a batch, so no LDS atomics are needed
//     (fp32 LDS atomics measured several times slower than this on gfx950).
// When the range is done the stash is added to the output with one global
// atomic per (row, rank) that received any term, so an output row sees one
// update per workgroup instead of one per window.
constexpr int kShortB = 1024;               // threads = non-zeros per batch
constexpr int kShortLPN = 16;               // lanes per position
constexpr int kShortNG = kShortB / kShortLPN;   // lane groups = positions per group
constexpr int kShortHist = 1024;            // histogram bins (>= I_n)
constexpr int kShortLds = 64 * 1024;        // records + histogram + carries + stash
constexpr int kShortLoads = 8;              // positions x ranks in flight per lane

// LDS bytes besides the stash: records, histogram, scan totals, carry slots
// (one per group, cls = 16, 32 or 64 floats: the ranks one group covers)
__host__ __device__ constexpr size_t short_fixed_lds(int N, int cls) {
  return (size_t)kShortB * (N + 1) * 4 + (size_t)kShortHist * 4 + (kShortB / 64) * 4 +
         (size_t)kShortNG * cls * 4;
}

//
// Rank layout as in the window kernel: with bf16 factors each lane holds RPL
// consecutive ranks of the slice (VEC: one 4- or 8-byte gather when R is even).
template <int RPL, typename FT, int N, bool BIG, bool VEC = false>
__global__ __launch_bounds__(kShortB, 8) void k_mttkrp_short(KParams p, int64_t per) {
  extern __shared__ __align__(16) unsigned char smem_short[];
  constexpr int LPN = kShortLPN;
  constexpr bool PACKED = sizeof(FT) == 2 && RPL > 1;
  static_assert(!VEC || PACKED, "vector gathers are for packed bf16 ranks");
  constexpr int NF = N + 1;
  constexpr int NG = kShortNG;
  constexpr int C = kShortB / NG;            // positions per group and batch
  constexpr int U = kShortLoads / RPL;       // positions in flight per group
  constexpr int CW = LPN * RPL;              // ranks one group covers (carry slot)
  const int I = (int)p.short_rows;
  const int SW = p.short_width;              // <= CW
  const int rlo = (int)blockIdx.y * SW;
  const int W = min(SW, p.R - rlo);
  uint32_t* s_rec = reinterpret_cast<uint32_t*>(smem_short);    // kShortB x NF
  uint32_t* s_hist = s_rec + kShortB * NF;                      // kShortHist
  uint32_t* s_wsum = s_hist + kShortHist;                       // kShortB / 64
  float* s_carry = reinterpret_cast<float*>(s_wsum + kShortB / 64);   // NG x CW
  float* s_out = s_carry + NG * CW;                             // I x SW
  const int tid = threadIdx.x;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = min(p.n, lo + per);
  if (lo >= hi || W <= 0) return;
  for (int i = tid; i < I * SW; i += kShortB) s_out[i] = 0.f;
  for (int i = tid; i < kShortHist; i += kShortB) s_hist[i] = 0;
  const int gi = tid / LPN, rl = tid % LPN;
  constexpr int NO = N > 1 ? N - 1 : 1;
  __amdgpu_buffer_rsrc_t rs[NO];
  const void* ap[NO];
#pragma unroll
  for (int j = 0; j + 1 < N; ++j) {
    const int m = (j < p.mode) ? j : j + 1;
    ap[j] = p.A[m];
    rs[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.A[m]), 0, (int)p.abytes[m],
                                              (int)kBufFlags);
  }
  uint32_t loff[RPL];
  bool ract[RPL];
  int rix[RPL];   // slice-relative rank of each of this lane's RPL values
#pragma unroll
  for (int q = 0; q < RPL; ++q) {
    const int r = PACKED ? rl * RPL + q : rl + q * LPN;
    rix[q] = r;
    ract[q] = r < W;
    loff[q] = (uint32_t)(rlo + (ract[q] ? r : 0)) * (uint32_t)sizeof(FT);
  }
  for (int64_t b0 = lo; b0 < hi; b0 += kShortB) {
    // ---- processing: load, decode, group by target
    __syncthreads();   // histogram cleared; the previous batch's records and carries consumed
    const int64_t k = b0 + tid;
    const bool valid = k < hi;
    uint32_t c[N];
    float x = 0.f;
    uint32_t tgt = 0, rank = 0;
    if (valid) {
      decode<N>(p, p.keys[k], p.base + k, c);
      x = p.vals[k];
#pragma unroll
      for (int m = 0; m < N; ++m)
        if (m == p.mode) tgt = c[m];
      rank = atomicAdd(&s_hist[tgt], 1u);
    }
    __syncthreads();
    block_exclusive_scan<kShortHist, kShortB>(s_hist, tid, s_wsum);
    if (valid) {
      const int pos = (int)(s_hist[tgt] + rank);
#pragma unroll
      for (int j = 0; j + 1 < N; ++j)
        s_rec[pos * NF + j] = ((j < p.mode) ? c[j] : c[j + 1]) * (BIG ? 1u : p.rowbytes);
      s_rec[pos * NF + N - 1] = tgt;
      s_rec[pos * NF + N] = __float_as_uint(x);
    }
    __syncthreads();
    // ---- computing: segment sums of this group's positions
    const int nb = (int)min<int64_t>(kShortB, hi - b0);
    const int q0 = gi * C;
    const int qe = min(q0 + C, nb);
    float acc[RPL];
    uint32_t cur = 0;
    bool pending = false;   // owner of a run that continues into later groups
    int run_end = 0;        // end of that run (grouped position)
    if (q0 < qe) {
      cur = s_rec[q0 * NF + N - 1];
      const bool first_shared = q0 > 0 && s_rec[(q0 - 1) * NF + N - 1] == cur;
      const bool last_cont = qe < nb && s_rec[qe * NF + N - 1] == s_rec[(qe - 1) * NF + N - 1];
      bool first = true;
#pragma unroll
      for (int q = 0; q < RPL; ++q) acc[q] = 0.f;
      for (int j0 = q0; j0 < qe; j0 += U) {
        float pr[U][RPL];
        uint32_t tg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int j = j0 + u;
          const uint32_t* e = &s_rec[(j < qe ? j : j0) * NF];
          const float xv = __uint_as_float(e[N]);
          tg[u] = e[N - 1];
#pragma unroll
          for (int q = 0; q < RPL; ++q) pr[u][q] = xv;
#pragma unroll
          for (int jj = 0; jj + 1 < N; ++jj) {
            if constexpr (BIG && PACKED) {
              const FT* rowp = static_cast<const FT*>(ap[jj]) + (size_t)e[jj] * p.R;
              float t3[RPL];
              ld_bf16_run_ptr<RPL, VEC>(rowp + loff[0] / sizeof(FT), ract, t3);
#pragma unroll
              for (int q = 0; q < RPL; ++q) pr[u][q] *= t3[q];
            } else if constexpr (BIG) {
              const FT* rowp = static_cast<const FT*>(ap[jj]) + (size_t)e[jj] * p.R;
#pragma unroll
              for (int q = 0; q < RPL; ++q)
                pr[u][q] *= ld_factor<FT>(rowp, (size_t)(loff[q] / sizeof(FT)));
            } else if constexpr (PACKED) {
              float t3[RPL];
              ld_bf16_run<RPL, VEC>(rs[jj], e[jj] + loff[0], t3);
#pragma unroll
              for (int q = 0; q < RPL; ++q) pr[u][q] *= t3[q];
            } else {
#pragma unroll
              for (int q = 0; q < RPL; ++q) pr[u][q] *= ld_buf<FT>(rs[jj], e[jj] + loff[q]);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (j0 + u >= qe) break;
          if (tg[u] != cur) {
            // a finished segment that does not reach the end of this group
            if (first && first_shared) {
#pragma unroll
              for (int q = 0; q < RPL; ++q) s_carry[gi * CW + rix[q]] = acc[q];
            } else {
#pragma unroll
              for (int q = 0; q < RPL; ++q)
                if (ract[q]) s_out[cur * SW + rix[q]] += acc[q];
            }
            first = false;
            cur = tg[u];
#pragma unroll
            for (int q = 0; q < RPL; ++q) acc[q] = 0.f;
          }
#pragma unroll
          for (int q = 0; q < RPL; ++q) acc[q] += pr[u][q];
        }
      }
      // the segment that reaches the end of this group
      if (first && first_shared) {
#pragma unroll
        for (int q = 0; q < RPL; ++q) s_carry[gi * CW + rix[q]] = acc[q];
      } else if (last_cont) {
        pending = true;
        // the scanned histogram holds each target's first position, so the
        // run of `cur` ends where the next target's begins
        run_end = cur + 1 < (uint32_t)kShortHist ? (int)s_hist[cur + 1] : nb;
      } else {
#pragma unroll
        for (int q = 0; q < RPL; ++q)
          if (ract[q]) s_out[cur * SW + rix[q]] += acc[q];
      }
    }
    __syncthreads();
    // ---- owners of runs that cross groups add the later groups' carries
    if (pending) {
#pragma unroll 4
      for (int g2 = gi + 1; g2 * C < run_end; ++g2) {
#pragma unroll
        for (int q = 0; q < RPL; ++q) acc[q] += s_carry[g2 * CW + rix[q]];
      }
#pragma unroll
      for (int q = 0; q < RPL; ++q)
        if (ract[q]) s_out[cur * SW + rix[q]] += acc[q];
    }
    for (int i = tid; i < kShortHist; i += kShortB) s_hist[i] = 0;
  }
  __syncthreads();
  // ---- one global atomic per stash entry that received a term
  const float scale = term_scale(p);
  for (int i = tid; i < I * W; i += kShortB) {
    const int row = i / W, r = i - row * W;
    const float v = s_out[row * SW + r];
    if (v != 0.f) unsafeAtomicAdd(p.out + (size_t)row * p.R + rlo + r, v * scale);
  }
}

// Sampled CP model, residual and squared residual sums (Section 2.2 model):
// one wave per 64 consecutive non-zeros.  Each non-zero's record (byte offsets,
// or row indices when BIG, of its N factor rows, and its value) goes to LDS;
// groups of 16 lanes (RPL ranks per lane) then walk 16 records each,
// 8 / RPL at a time, issuing every gather of those records before the first
// use, and reduce the rank sum across the group.  The residual x - xhat is
// written in BLCO order; the squared residuals are summed in fp64 per
// workgroup (k_reduce_loss adds the partials in a fixed order).  bf16 factors take
// the packed rank layout of the MTTKRP kernels (VEC: one 4- or 8-byte gather).
template <int RPL, typename FT, int N, bool BIG, bool VEC = false>
__global__ __launch_bounds__(kBlock) void k_loss_tile(KParams p) {
  constexpr int LPN = 16;
  constexpr bool PACKED = sizeof(FT) == 2 && RPL > 1;
  static_assert(!VEC || PACKED, "vector gathers are for packed bf16 ranks");
  constexpr int G = 64 / LPN;                  // groups per wave
  constexpr int PPG = 64 / G;                  // records per group
  constexpr int NF = N + 1;
  constexpr int U = (8 / RPL) < PPG ? (8 / RPL) : PPG;
  __shared__ uint32_t s[kWaves][64][NF];
  __shared__ float s_e[kWaves][64];
  __shared__ double s_part[kWaves];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int64_t tile = (int64_t)blockIdx.x * kWaves + wv;
  const int64_t k = tile * 64 + lane;
  const bool valid = k < p.n;
  uint32_t c[N];
  float x = 0.f;
  if (valid) {
    uint64_t key = p.keys[k];
    x = p.vals[k];
    decode<N>(p, key, p.base + k, c);
  } else {
#pragma unroll
    for (int m = 0; m < N; ++m) c[m] = 0;
  }
#pragma unroll
  for (int m = 0; m < N; ++m) s[wv][lane][m] = BIG ? c[m] : c[m] * p.rowbytes;
  s[wv][lane][N] = __float_as_uint(x);
  s_e[wv][lane] = x;
  __amdgpu_buffer_rsrc_t rs[N];
#pragma unroll
  for (int m = 0; m < N; ++m)
    rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.A[m]), 0, (int)p.abytes[m],
                                              (int)kBufFlags);
  wave_sync_lds();
  const int g = lane / LPN;
  const int rl = lane % LPN;
  const int R = p.R;
  for (int r0 = 0; r0 < R; r0 += LPN * RPL) {
    uint32_t loff[RPL];
    bool ract[RPL];
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int r = PACKED ? r0 + rl * RPL + q : r0 + rl + q * LPN;
      ract[q] = r < R;
      loff[q] = (uint32_t)(ract[q] ? r : 0) * (uint32_t)sizeof(FT);
    }
    for (int q0 = 0; q0 < PPG; q0 += U) {
      float v[U][RPL];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t* e = s[wv][g * PPG + q0 + u];
#pragma unroll
        for (int q = 0; q < RPL; ++q) v[u][q] = 1.f;
#pragma unroll
        for (int m = 0; m < N; ++m) {
          const uint32_t f = e[m];
          if constexpr (BIG && PACKED) {
            const FT* rowp = static_cast<const FT*>(p.A[m]) + (size_t)f * R;
            float t3[RPL];
            ld_bf16_run_ptr<RPL, VEC>(rowp + loff[0] / sizeof(FT), ract, t3);
#pragma unroll
            for (int q = 0; q < RPL; ++q) v[u][q] *= t3[q];
          } else if constexpr (BIG) {
            const FT* rowp = static_cast<const FT*>(p.A[m]) + (size_t)f * R;
#pragma unroll
            for (int q = 0; q < RPL; ++q)
              v[u][q] *= ld_factor<FT>(rowp, (size_t)(loff[q] / sizeof(FT)));
          } else if constexpr (PACKED) {
            float t3[RPL];
            ld_bf16_run<RPL, VEC>(rs[m], f + loff[0], t3);
#pragma unroll
            for (int q = 0; q < RPL; ++q) v[u][q] *= t3[q];
          } else {
#pragma unroll
            for (int q = 0; q < RPL; ++q) v[u][q] *= ld_buf<FT>(rs[m], f + loff[q]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float part = 0.f;
#pragma unroll
        for (int q = 0; q < RPL; ++q)
          if (ract[q]) part += v[u][q];
#pragma unroll
        for (int off = LPN / 2; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (rl == 0) s_e[wv][g * PPG + q0 + u] -= part;
      }
    }
  }
  wave_sync_lds();
  const float e = s_e[wv][lane];
  if (valid && p.out) p.out[k] = e;
  double e2 = valid ? (double)e * (double)e : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) e2 += __shfl_xor(e2, off);
  if (lane == 0) s_part[wv] = e2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += s_part[w];
    p.partials[blockIdx.x] = t;
  }
}

// Sum of squares of a residual in fp64: workgroup b sums entries
// [b * kSqPer, (b + 1) * kSqPer) in a fixed order into part[b].
constexpr int kSqPer = 4096;
__global__ __launch_bounds__(256) void k_sumsq(const float* __restrict__ r, int64_t n,
                                               double* __restrict__ part) {
  __shared__ double sh[256];
  const int64_t lo = (int64_t)blockIdx.x * kSqPer;
  const int64_t hi = min(n, lo + (int64_t)kSqPer);
  double a = 0.0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const double e = (double)r[i];
    a += e * e;
  }
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// loss = 1/2 * sum of the partials, in a fixed order (one workgroup).
__global__ __launch_bounds__(1024) void k_reduce_loss(const double* __restrict__ part, int64_t n,
                                                      double* __restrict__ loss) {
  __shared__ double sh[1024];
  double a = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 1024) a += part[i];
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = 0.5 * sh[0];
}

// Arrays of one launch of an element-wise kernel: row blockIdx.y of the grid takes one.  A
// training step casts and scales one array per mode; a launch of its own for each took 4 us
// of host time and 2-5 us of an otherwise idle device.
struct Arrays {
  const float* src[BLCO_MAX_MODES];
  void* dst[BLCO_MAX_MODES];
  int64_t n[BLCO_MAX_MODES];
};

// fp32 -> bf16, round to nearest even; NaN stays a (quiet) NaN.
__global__ __launch_bounds__(256) void k_cast_bf16(Arrays a) {
  const float* __restrict__ src = a.src[blockIdx.y];
  uint16_t* __restrict__ dst = static_cast<uint16_t*>(a.dst[blockIdx.y]);
  const int64_t n = a.n[blockIdx.y], stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    uint32_t u = __float_as_uint(src[i]);
    uint16_t b;
    if ((u & 0x7fffffffu) > 0x7f800000u) {
      b = (uint16_t)((u >> 16) | 0x40u);
    } else {
      u += 0x7fffu + ((u >> 16) & 1u);
      b = (uint16_t)(u >> 16);
    }
    dst[i] = b;
  }
}

// Calibration of the memory-side atomic rate: for each k < n, one row-op on
// out row rows[k]: 16 lanes add 1.0f to the row's R entries, lane l holding
// ranks l, l + 16, ..., as the window kernel flushes a finished segment.  Row
// ids at or past nrows are skipped.
__global__ __launch_bounds__(256) void k_atomic_probe(float* __restrict__ out, int64_t nrows,
                                                      const uint32_t* __restrict__ rows,
                                                      int64_t n, int R) {
  const int64_t g = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const int rl = threadIdx.x & 15;
  if (g >= n) return;
  const uint32_t row = rows[g];
  if ((int64_t)row >= nrows) return;
  float* dst = out + (size_t)row * R;
  for (int r = rl; r < R; r += 16) unsafeAtomicAdd(dst + r, 1.0f);
}

// Measurement kernel: groups of 16 lanes read kGatherRows rows of table each (ranks
// l, l + 16, ... per lane, all loads of a group in flight together), as the MTTKRP
// kernels gather factor rows; lane 0 of a group stores its partial sum in sink[group].
constexpr int kGatherRows = 6;
__global__ __launch_bounds__(256) void k_gather_probe(const float* __restrict__ table,
                                                      int64_t nrows,
                                                      const uint32_t* __restrict__ rows,
                                                      int64_t n, int R, float* __restrict__ sink) {
  const int64_t g = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const int rl = threadIdx.x & 15;
  const int64_t k0 = g * kGatherRows;
  if (k0 >= n) return;
  uint32_t rr[kGatherRows];
#pragma unroll
  for (int j = 0; j < kGatherRows; ++j) {
    rr[j] = k0 + j < n ? rows[k0 + j] : 0xFFFFFFFFu;
    if ((int64_t)rr[j] >= nrows) rr[j] = 0xFFFFFFFFu;
  }
  float s = 0.f;
#pragma unroll 4
  for (int r = rl; r < R; r += 16) {
    float v[kGatherRows];
#pragma unroll
    for (int j = 0; j < kGatherRows; ++j)
      v[j] = rr[j] != 0xFFFFFFFFu ? table[(size_t)rr[j] * R + r] : 0.f;
#pragma unroll
    for (int j = 0; j < kGatherRows; ++j) s += v[j];
  }
  if (rl == 0) sink[g] = s;
}

// x[i] *= (float)(alpha * scale[0]) (the chain-rule factor of an autograd backward).
__global__ __launch_bounds__(256) void k_scale(Arrays a, const double* __restrict__ scale,
                                               double alpha) {
  float* __restrict__ x = static_cast<float*>(a.dst[blockIdx.y]);
  const float f = (float)(alpha * (scale ? scale[0] : 1.0));
  const int64_t n = a.n[blockIdx.y], stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) x[i] *= f;
}

// ====================================================================== dispatch

typedef void (*ShortFn)(KParams, int64_t);

template <int RPL, typename FT, bool BIG, bool VEC>
static ShortFn pick_short_v(int N) {
  switch (N) {
    case 1: return k_mttkrp_short<RPL, FT, 1, BIG, VEC>;
    case 2: return k_mttkrp_short<RPL, FT, 2, BIG, VEC>;
    case 3: return k_mttkrp_short<RPL, FT, 3, BIG, VEC>;
    case 4: return k_mttkrp_short<RPL, FT, 4, BIG, VEC>;
    case 5: return k_mttkrp_short<RPL, FT, 5, BIG, VEC>;
    case 6: return k_mttkrp_short<RPL, FT, 6, BIG, VEC>;
    case 7: return k_mttkrp_short<RPL, FT, 7, BIG, VEC>;
    default: return k_mttkrp_short<RPL, FT, 8, BIG, VEC>;
  }
}

// VEC where the bf16 ranks are packed (two or more per lane) and R is even
template <int RPL, typename FT, bool BIG>
static ShortFn pick_short(int N, int R) {
  if constexpr (sizeof(FT) == 2 && RPL > 1) {
    if (R % 2 == 0) return pick_short_v<RPL, FT, BIG, true>(N);
  }
  return pick_short_v<RPL, FT, BIG, false>(N);
}

// ranks per lane of the hierarchical kernel for a slice width (<= 64)
static int short_rpl(int SW) { return SW <= 16 ? 1 : SW <= 32 ? 2 : 4; }

template <typename FT, bool BIG>
static ShortFn select_short_t(int N, int SW, int R) {
  const int rpl = short_rpl(SW);
  if (rpl == 1) return pick_short<1, FT, BIG>(N, R);
  if (rpl == 2) return pick_short<2, FT, BIG>(N, R);
  return pick_short<4, FT, BIG>(N, R);
}

static ShortFn select_short(int N, int SW, int R, int fdt, bool big) {
  if (fdt == BLCO_F32)
    return big ? select_short_t<float, true>(N, SW, R) : select_short_t<float, false>(N, SW, R);
  return big ? select_short_t<uint16_t, true>(N, SW, R)
             : select_short_t<uint16_t, false>(N, SW, R);
}

static size_t short_lds(int N, uint64_t rows, int SW) {
  return short_fixed_lds(N, kShortLPN * short_rpl(SW)) + (size_t)rows * SW * sizeof(float);
}

// Rank-slice width of the hierarchical kernel: slices of at most 64 ranks, as
// even as possible, in multiples of 16 when there are several, such that the
// stash (I_n x SW fp32), the records, the histogram and the carry slots fit in
// kShortLds bytes.  0 when even a 16-rank slice does not fit.
static int short_slice_width(int N, uint64_t rows, int R) {
  if (rows > (uint64_t)kShortHist) return 0;
  for (int slices = (R + 63) / 64; slices <= (R + 15) / 16; ++slices) {
    const int w = slices == 1 ? R : ((R + slices - 1) / slices + 15) / 16 * 16;
    if (short_lds(N, rows, w) <= (size_t)kShortLds) return w;
  }
  return 0;
}

// Compute units of the current device (the Section 5.3 threshold), read once per device.
static int device_cus() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    cached[dev] = v;
  }
  return cached[dev];
}

template <int RPL, typename FT, bool BIG, bool VEC>
static KernelFn pick_loss_v(int N) {
  switch (N) {
    case 1: return k_loss_tile<RPL, FT, 1, BIG, VEC>;
    case 2: return k_loss_tile<RPL, FT, 2, BIG, VEC>;
    case 3: return k_loss_tile<RPL, FT, 3, BIG, VEC>;
    case 4: return k_loss_tile<RPL, FT, 4, BIG, VEC>;
    case 5: return k_loss_tile<RPL, FT, 5, BIG, VEC>;
    case 6: return k_loss_tile<RPL, FT, 6, BIG, VEC>;
    case 7: return k_loss_tile<RPL, FT, 7, BIG, VEC>;
    default: return k_loss_tile<RPL, FT, 8, BIG, VEC>;
  }
}

// VEC where the bf16 ranks are packed (two or more per lane) and R is even
template <int RPL, typename FT, bool BIG>
static KernelFn pick_loss(int N, int R) {
  if constexpr (sizeof(FT) == 2 && RPL > 1) {
    if (R % 2 == 0) return pick_loss_v<RPL, FT, BIG, true>(N);
  }
  return pick_loss_v<RPL, FT, BIG, false>(N);
}

template <typename FT, bool BIG>
static KernelFn select_loss_t(int N, int R) {
  if (R <= 16) return pick_loss<1, FT, BIG>(N, R);
  if (R <= 32) return pick_loss<2, FT, BIG>(N, R);
  return pick_loss<4, FT, BIG>(N, R);
}

static KernelFn select_loss(int N, int R, int fdt, bool big) {
  if (fdt == BLCO_F32)
    return big ? select_loss_t<float, true>(N, R) : select_loss_t<float, false>(N, R);
  return big ? select_loss_t<uint16_t, true>(N, R) : select_loss_t<uint16_t, false>(N, R);
}

// Conflict-resolution mechanism of a mode-`mode` MTTKRP at rank R (Section
// 5.3): the tensor's setting, where AUTO takes the hierarchical mechanism when
// the target mode is shorter than the device's compute units.  *sw receives
// the hierarchical kernel's rank-slice width.
static int resolve(const blco_tensor* t, int mode, int rank, int* sw) {
  const uint64_t rows = t->lay.dims[mode];
  const int w = short_slice_width(t->lay.N, rows, rank);
  *sw = w;
  if (t->resolution == BLCO_RES_REGISTER) return BLCO_RES_REGISTER;
  if (t->resolution == BLCO_RES_HIERARCHICAL) {
    if (!w)
      return set_error(BLCO_EUNSUPPORTED,
                       "hierarchical resolution: mode %d (%llu rows) does not fit the LDS stash",
                       mode, (unsigned long long)rows);
    return BLCO_RES_HIERARCHICAL;
  }
  return (w && rows < (uint64_t)device_cus()) ? BLCO_RES_HIERARCHICAL : BLCO_RES_REGISTER;
}

// Static LDS bytes of a kernel, read once per kernel.
static size_t kernel_static_lds(const void* f) {
  static std::mutex mu;
  static std::vector<std::pair<const void*, size_t>> cache;
  std::lock_guard<std::mutex> lock(mu);
  for (auto& e : cache)
    if (e.first == f) return e.second;
  hipFuncAttributes a;
  size_t v = 64 * 1024;   // unknown: assume no room
  if (hipFuncGetAttributes(&a, f) == hipSuccess) v = a.sharedSizeBytes;
  cache.push_back({f, v});
  return v;
}

// LDS a workgroup may use on the current device: a CU's, at most the per-workgroup limit;
// read once per device.
static size_t cu_lds() {
  static size_t cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 64 * 1024;
  if (!cached[dev]) {
    int cu = 0, blk = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
            hipSuccess || cu <= 0)
      cu = 64 * 1024;
    if (hipDeviceGetAttribute(&blk, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
        blk <= 0)
      blk = 64 * 1024;
    cached[dev] = std::min<size_t>((size_t)cu, (size_t)blk);
  }
  return cached[dev];
}

// LDS per window-kernel workgroup where two share a CU.
static size_t win_lds_budget() {
  static size_t cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 64 * 1024;
  if (!cached[dev]) {
    int cu = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
            hipSuccess || cu <= 0)
      cu = 64 * 1024;
    cached[dev] = std::min<size_t>((size_t)cu / 2, cu_lds());
  }
  return cached[dev];
}

// ====================================================================== host runtime

static size_t factor_elem_bytes(int fdt) { return fdt == BLCO_BF16 ? 2 : 4; }

static void fill_params(const blco_tensor* t, KParams* p) {
  memset(p, 0, sizeof(*p));
  const Layout& L = t->lay;
  for (int m = 0; m < L.N; ++m) {
    p->shift[m] = L.w[m] ? (uint32_t)L.s[m] : 0u;
    p->mask[m] = L.w[m] >= 32 ? 0xFFFFFFFFu : ((1u << L.w[m]) - 1u);
  }
  p->run_start = t->d_run_start;
  p->run_base = t->d_run_base;
  p->tile_run = t->d_tile_run;
  p->multi = (t->run_start.size() > 2) ? 1 : 0;
  if (t->run_start.size() == 2) {
    for (int m = 0; m < L.N; ++m)
      if (t->run_base[m]) p->multi = 1;
  }
  p->scale = 1.0f;
}

// One launch of k_prep, or none where there is nothing to do.
static int prepare(const PrepParams& p, int fdt, hipStream_t s) {
  int64_t most = p.starts ? kGroupBuckets * 4 : 0;
  for (int z = 0; z < 2; ++z) most = std::max(most, p.nzero[z]);
  for (int m = 0; m < p.npad; ++m) most = std::max(most, p.rows[m] * p.Rp);
  if (most <= 0) return BLCO_OK;
  const int64_t blocks = std::min<int64_t>((most / 4 + 255) / 256 + 1, 8192);
  hipLaunchKernelGGL(k_prep, dim3((unsigned)blocks), dim3(256), 0, s, p, fdt == BLCO_BF16 ? 1 : 0);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

static int fill_zero(float* out, int64_t n, hipStream_t s) {
  PrepParams p = {};
  p.zero[0] = out;
  p.nzero[0] = n;
  return prepare(p, BLCO_F32, s);
}

static int check_factor_args(const blco_tensor* t, int mode, const void* const* factors, int fdt,
                             int rank, const float* out, bool need_mode_factor) {
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  const int N = t->lay.N;
  if (mode < 0 || mode >= N) return set_error(BLCO_EINVAL, "mode %d outside 0..%d", mode, N - 1);
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (fdt != BLCO_F32 && fdt != BLCO_BF16) return set_error(BLCO_EINVAL, "factor dtype %d", fdt);
  if (!factors) return set_error(BLCO_EINVAL, "factors is NULL");
  for (int m = 0; m < N; ++m)
    if ((m != mode || need_mode_factor) && !factors[m] && t->nnz > 0)
      return set_error(BLCO_EINVAL, "factors[%d] is NULL", m);
  if (!out) return set_error(BLCO_EINVAL, "out is NULL");
  int sw = 0;
  const int res = resolve(t, mode, rank, &sw);
  return res < 0 ? res : BLCO_OK;
}

// Row flushes per non-zero that windows of 4096 have to save over windows of 2048 (win_wpt).
static double wide_saves(int N) { return N <= 4 ? 0.05 : 0.095; }

// Window of the window kernel over n non-zeros without a stash, as k_mttkrp_win's WPT:
// the smallest window that needs no more windows than the device has compute units, up
// to the largest that pays in a long launch (2048 non-zeros; 4096 at R > 32, where four
// ranks per lane cover the gathers of the one workgroup per CU it allows).  A short
// launch is bound by the latency of one window: with 1000 x 500 x 300 uniform indices,
// 30k non-zeros took 16.1 us in windows of 2048 (43 us in windows of 4096 at R = 64) and
// take 6 us (9 us) in windows of 256.  More windows than compute units cost more than they
// save, in row flushes and in the chain of same-row flushes of a skewed mode: 250k power-law
// non-zeros at R = 16 take 23, 17, 13 and 18 us in windows of 256, 512, 1024 and 2048.  Windows of
// 256 end at three quarters as many windows: 60k non-zeros take 11.5 us in 235 of them and 10.8 in
// 118 of 512 (uniform indices: 8.3 and 8.9; R = 64: 16.1 and 14.9), and the longer chains put a
// skewed mode 1.46 times as far from 64 bits as in windows of 2048 (1.8e-7 and 1.25e-7; 1.45e-7 in
// windows of 512).  38k at R = 64 take 14 us in 148 of them and 15 in 74.
//
// At R > 32 a window of 2048 leaves two workgroups per CU; one of 4096 merges more.  It pays on a
// mode without frequent rows where it saves wide_saves(N) row flushes per non-zero (counted at
// construction: the rows a window holds follow from how the non-zeros lie, and an estimate from
// the mode lengths was several times off on skewed tensors).  Windows of 2048 and 4096, us per mode,
// by the flushes saved.  8M non-zeros of 21007 x 9001 x 1501 x 367, R = 64: 0.079: 575 and 509;
// 0.096: 517 and 455; 0.105: 473 and 429; 0.075: 383 and 379; 50M of 2^24 x 2^22 x 2^20 x 2^10, R =
// 64 bf16: 0.073: 4370 and 3830; 0.101: 2800 and 2480; 2000 x 1000 x 500: 0.024: 188 and 258; 0.012:
// 164 and 233.  Five modes, whose records are half as long again, 8M, R = 64: 0.091: 447 and 449;
// 0.068: 374 and 401; 0.059: 360 and 388; 2M: 0.100: 159 and 144.  Grouped non-zeros repeat their
// rows in 2048 already (20M of 200003 x 100003 x 50021, R = 64 bf16: 2.64 and 3.15 ms).
//
// careful: CP-ALS multiplies the sums by V^+ (condition number about 1e3 on a planted model),
// which turns their last bits into its factors' fifth digit, so its updates keep one order of
// summation at every size: the full stash on a mode with frequent rows, else windows of 2048 (4096
// at R > 32).  1M power-law non-zeros, R = 16, 5 iterations, over 48 inputs: two runs of this
// route leave the third factor 7e-5 apart in norm, the routes below move it by 1.4e-4; time 1.24
// against 1.15 ms.
//
// wide: whether windows of 4096 pay, or are wanted for their shorter chains (out_copies).
static int win_wpt(int N, int R, bool resid, bool big, bool wide, int64_t n, bool careful) {
  if (R > 64 || N > kWideMaxN) return 1;
  if (careful) return R > 32 ? 4 : 2;
  // the fused residual walk's records hold one field more: at N = 5 two windows of 2048 no
  // longer share a CU, and at R > 32 its walk has no registers for four per thread
  const int most = resid ? (N <= 4 ? 2 : 1) : R > 32 && wide ? 4 : 2;
  if (big) return most;
  const int64_t cus = device_cus();
  if (n <= kWin / 4 * cus * 3 / 4) return -4;
  for (int w : {-2, 1, 2})
    if (w == most || n <= (w < 0 ? kWin / -w : kWin * w) * cus) return w;
  return most;
}

static KernelFn select_win(int N, int R, bool even, int fdt, bool big, bool stash, int wpt) {
  if (big) return select_win_big(N, R, fdt, stash, wpt);
  return fdt == BLCO_F32 ? select_win_f32(N, R, stash, wpt)
                         : select_win_bf16(N, R, even, stash, wpt);
}

// Frequent rows of the target mode that the window kernel `f` keeps in its
// LDS stash: as many as fit beside the kernel's own LDS in one workgroup's
// share of a CU, or none when the rows left out would not be much less
// frequent than the most frequent one (a stash shortens the longest atomic
// chains only then: measured slower on a 1024-row uniform mode, where a fifth
// of the rows fit).  An explicit threshold at build time keeps the stash
// regardless.  The kernel's static LDS does not depend on the factor type.
static int stash_rows(const blco_tensor* t, int mode, int rank, KernelFn f) {
  if (t->nhot[mode] <= 0) return 0;
  int K = 0;
  const size_t fixed = kernel_static_lds((const void*)f) + 2 * (size_t)kHotSlots * 4;
  const size_t budget = win_lds_budget();
  if (budget > fixed)
    K = (int)std::min<size_t>((size_t)t->nhot[mode], (budget - fixed) / ((size_t)rank * 4));
  if (K > 0 && !t->hot_forced) {
    const uint64_t* cnt = t->hot_cnt.data() + (size_t)mode * (kHotMax + 1);
    if (cnt[K] * 4 > cnt[0]) K = 0;
  }
  return K;
}

// Whether mode `mode` at rank `rank` may take hot copies (see k_mttkrp_win) instead of the
// full stash, which is tied to windows of 1024 non-zeros: 2048 merge about as much without
// its look-up and its resident workgroups.  An explicit threshold at build time keeps the
// full stash.
static bool copies_ok(const blco_tensor* t, int mode, int rank, int ranks, bool big) {
  return !t->hot_forced && !big && t->lay.N <= kWideMaxN && ranks <= 64 &&
         t->lay.dims[mode] * (uint64_t)rank <= (1ULL << 31);
}

// Whether a mode has rows worth keeping apart: not where the rows beyond the recorded ones
// are about as frequent as they are (every row then has equally long chains of atomics).
static bool has_frequent_rows(const blco_tensor* t, int mode) {
  if (t->nhot[mode] <= 0) return false;
  const uint64_t* cnt = t->hot_cnt.data() + (size_t)mode * (kHotMax + 1);
  return t->hot_forced || cnt[t->nhot[mode]] * 4 <= cnt[0];
}

// A launch of at most this many windows needs no copies: its hottest rows see no more
// atomics than the full stash's own flushes would make.
constexpr int64_t kCopyMinWindows = 2048;
constexpr int kCopyMax = 64;   // most copies of a row

// Copies of each frequent row: at most about kChain additions to one, up to kCopyMax copies (launches
// of 67M non-zeros; 200M put 1526 additions on a copy).  The full stash made a chain of 512 to
// 2048 additions of a row, one per workgroup.  Error from 64 bits of a mode's output (norm), 3-mode
// power-law non-zeros, R = 16, with the stash, at most 4096 additions and at most 512: 8M: 6.2e-7,
// 6.6e-7, 3.1e-7; 16M: 6.1e-7, 6.6e-7, 3.3e-7; 50M, the last two: 6.1e-7, 4.2e-7; and 8M take 141
// us per mode instead of 157, as same-row atomics wait for each other.
constexpr int64_t kChain = 512;
static int copy_count(int64_t nwin) {
  int c = 1;
  while (c < kCopyMax && c * kChain < nwin) c *= 2;
  return c;
}

static int copy_stride(int rank) { return (rank + 15) / 16 * 16; }   // whole 64-byte lines

static bool big_gathers(const blco_tensor* t, int mode, int rank, int fdt, bool window,
                        bool resid);

// Most elements of an output that the window kernel addresses in 32 bits: its records hold a
// row's first element, and a flush adds a lane number of up to 15 to it before it takes the row's
// distance from a 64-byte line off (flush_row), so the last row has to end 16 before 2^32.
constexpr uint64_t kIndexMax = (1ULL << 32) - 16;

// Expected row flushes per non-zero of mode `mode` in windows of W of n non-zeros, taken as
// spread evenly over the index space: the window covers the index's lowest
// log2(W * cells / n) bits, so mode m moves over 2^(its bits among them) rows.
static double window_flushes(const blco_tensor* t, int mode, double W, double n) {
  const Layout& L = t->lay;
  double k = log2(W / n);
  for (int m = 0; m < L.N; ++m) k += log2((double)L.dims[m]);
  double bits = 0;
  for (int j = 0; j < L.b[mode]; ++j)
    bits += std::min(1.0, std::max(0.0, k - (double)L.pos[mode][j]));
  const double rows = std::min((double)L.dims[mode], exp2(bits));
  return rows * -expm1(-W / rows) / W;
}

// Row flushes per non-zero of mode `mode` in windows of kFlushWindow / 2 (half 0) and kFlushWindow
// (half 1) non-zeros, as counted at construction (0 below kFlushMin non-zeros).
static double flushes(const blco_tensor* t, int mode, int half) {
  return (double)t->flush_rows[mode][half] / (kFlushSamples * (kFlushWindow / (2 - half)));
}

// Whether windows of 4096 pay on mode `mode` (win_wpt).
static bool wide_pays(const blco_tensor* t, int mode, int gather, bool grouped) {
  return !grouped && gather % 16 == 0 && !has_frequent_rows(t, mode) &&
         flushes(t, mode, 0) - flushes(t, mode, 1) >= wide_saves(t->lay.N);
}

// Copies of the output that a launch in windows of 2048 at R > 32 adds to in turn (1: the output
// itself).  A row's sum is a chain of fp32 additions, one per window that holds it, and twice as
// many as in windows of 4096, the only ones there were at R > 32: 1.35 times their error on a mode
// that every window holds whole.  Copies shorten the chains; they are taken where clearing and
// adding them up is nothing against the launch (dims x copies x 128 <= n: under 2% of it), which
// is where chains are long.  8M non-zeros of 21007 x 9001 x 1501 x 367 x 301, R = 35, the mode of
// 367 rows: 1.01e-6 from 64 bits without copies, 7.6e-7 in windows of 4096, 2.6e-7 with 16 copies;
// all five modes 1693 us without and 1680 with, as same-row atomics wait for each other less.
// Without room for them such a launch takes windows of 4096.
static int out_copies(const blco_tensor* t, int mode, int rank, int gather, bool grouped, int64_t n) {
  if (rank <= 32 || rank > 64 || t->lay.N > kWideMaxN || n < (1 << 20) || grouped ||
      has_frequent_rows(t, mode) || wide_pays(t, mode, gather, grouped))
    return 1;
  int c = 1;
  while (c < 16 && t->lay.dims[mode] * 128 * 2 * (uint64_t)c <= (uint64_t)n) c *= 2;
  return c;
}

// The window kernel a launch over n non-zeros takes: its instantiation, windows, frequent
// rows in LDS and the slots of their look-up table.
struct WinPlan {
  KernelFn f;
  int wpt;
  int64_t nwin;
  int stash;     // rows in the full stash
  int copies;    // copies of each row in the row table (0: none)
  size_t bytes;  // workspace of the copies
};

// rank: elements between output rows; ranks, gather: ranks and ranks to gather (more
// where factors are padded); even: factor rows an even number of elements
// apart.  room: bytes of workspace there are; copies that do not fit it are not taken, and
// the mode falls back to the full stash where that applies.
// wide: windows of 4096 where they are built, whatever they save.
static WinPlan plan_win(const blco_tensor* t, int mode, int rank, int ranks, int gather, bool even,
                        int fdt, bool big, bool resid, int64_t n, size_t room, bool careful,
                        bool grouped, bool wide) {
  const int N = t->lay.N;
  auto pick = [&](bool stash, int w) {
    return resid ? select_res(N, gather, even, fdt, stash, w)
                 : select_win(N, gather, even, fdt, big, stash, w);
  };
  auto windows = [&](int w) {
    const int64_t W = w < 0 ? kWin / -w : (int64_t)kWin * w;
    return (n + W - 1) / W;
  };
  const bool frequent = has_frequent_rows(t, mode);
  WinPlan w = {nullptr,
               win_wpt(N, gather, resid, big, wide || wide_pays(t, mode, gather, grouped), n, careful),
               0, 0, 0, 0};
  // one non-zero per thread (the residual walk at N = 5): -1 is the form with copies
  const int lw = w.wpt == 1 ? -1 : w.wpt;
  const bool few = windows(lw) <= kCopyMinWindows;
  if (!careful && frequent && copies_ok(t, mode, rank, ranks, big) && (few || (lw != -1 || resid))) {
    if (few) {
      w.f = pick(false, w.wpt);
      w.nwin = windows(w.wpt);
      return w;
    }
    const int c = copy_count(windows(lw));
    const size_t bytes = sizeof(float) * (size_t)t->nhot[mode] * c * copy_stride(ranks);
    if (bytes <= room) {
      w.f = pick(true, lw);
      w.wpt = lw;
      w.nwin = windows(lw);
      w.copies = c;
      w.bytes = bytes;
      return w;
    }
  }
  if (frequent) {
    w.f = pick(true, 1);
    w.stash = stash_rows(t, mode, rank, w.f);
    if (w.stash > 0) w.wpt = 1;
  }
  if (w.stash == 0) w.f = pick(false, w.wpt);
  w.nwin = windows(w.wpt);
  return w;
}

// Workspace of a call: device memory the caller lends it (may be empty).
struct Work {
  char* p = nullptr;
  size_t bytes = 0;
  bool careful = false;   // a CP-ALS update: the full stash, and no copies or grouping (win_wpt)
};

static size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// Elements between factor rows of a launch: the rank, or more where the factors are copied
// into padded rows first, whose padding is gathered and multiplied like ranks.  Ranks that
// do not fill the 16-lane groups mask lanes at every gather, rows that start inside 16 bytes
// gather at half rate, and bf16 rows an odd number of elements apart take 2-byte loads.
// Rows are padded to whole groups where they are few against the non-zeros; up to 32 ranks
// also where they are not that few; and above, bf16 rows to 16 bytes only (longer rows are
// more lines, and rows enough to miss the caches are bound by those).  4M non-zeros, all
// modes, unpadded and padded, with the outputs padded as below: 2000 x 1000 x 500, fp32,
// R = 10: 265 and 157 us; R = 28: 213 and 193; R = 35: 382 and 255; R = 97: 737 and 582;
// bf16 R = 17: 416 and 188; R = 35: 756 and 351; 21007 x 9001 x 1501 x 367 x 31, R = 35: 1293
// and 1060; R = 60: 1282 and 1127; 200000 x 100000 x 20000, R = 17: 553 and 482; R = 31: 635
// and 490; bf16 R = 35: 952, to 40 712 and to 48 780; fp32 R = 50: 842, to 52 869 and to 64
// 898.  The copy reads and writes every row once (about 0.06 us per thousand rows at R = 32).
constexpr size_t kPadMax = (size_t)1 << 30;   // bytes of padded factors, and of a padded output
static int padded_rank(const blco_tensor* t, int mode, int rank, int fdt, bool all, int64_t n) {
  uint64_t rows = 0;
  for (int m = 0; m < t->lay.N; ++m)
    if (all || m != mode) rows += t->lay.dims[m];
  if (n < (1 << 18) || rows * 8 > (uint64_t)n) return rank;
  int Rp = (rank + 15) / 16 * 16;
  if (rank > 32 && rows * 32 > (uint64_t)n)
    Rp = fdt == BLCO_BF16 && rank % 2 != 0 ? (rank + 7) / 8 * 8 : rank;
  return rows * Rp * factor_elem_bytes(fdt) > kPadMax ? rank : Rp;
}

// Elements between the rows the window kernel flushes to: the rank, or whole 64-byte lines in
// a workspace whose rows are then copied to the output (k_unpad).  Unpadded rows cross into
// more lines and share them, and a line's atomics are performed one after another: 4M
// non-zeros of 200000 x 100000 x 20000, all modes: R = 10: 502 and 371 us; R = 31: 635 and
// 532; R = 97: 1594 and 1530.  Clearing and copying pay where the rows are few against the
// non-zeros: R = 50 on the same tensor took 841 us, with all modes padded 870.
//
// The kernel's 32-bit element indices address the padded rows, so these are bounded, as the padded
// factors are: kPadMax bytes (16M rows of 16 elements) of workspace.
static int padded_out(const blco_tensor* t, int mode, int rank, int64_t n) {
  const uint64_t rows = t->lay.dims[mode];
  if (n < (1 << 18) || rows * (rank > 32 ? 32 : 8) > (uint64_t)n) return rank;
  const int Ro = (rank + 15) / 16 * 16;
  return rows * Ro * sizeof(float) > kPadMax ? rank : Ro;
}
static_assert(kPadMax / sizeof(float) <= kIndexMax, "padded outputs keep 32-bit indices");

// Whether a launch over n non-zeros moves them to buckets of target rows first (k_group):
// where the row flushes that saves, at the memory side's rate (about 52 ps per 64-byte line),
// are worth twice the move (about 20 us and 18 ps per non-zero).  Only flat modes of
// tensors of one run, whose buckets were counted at build time.  4M non-zeros of 300007 x
// 200003 x 100003, all modes, as they lie and moved: R = 32: 1164 and 575 us; R = 48: 1747 and
// 990; R = 100: 4459 and 2106, bf16 4396 and 1561; R = 16 is left as it is (flushes of one
// line: 0.19 ms per mode).  20M of 200003 x 100003 x 50021, bf16 R = 64: 9144 and 2638.
//
// That is asked of the flushes non-zeros spread evenly would make; those counted at construction
// have to be worth the move too (1.2 times), since skewed modes beside a flat one keep its windows
// on few rows: 30M of 50000 x 30000 x 20000, the uniform mode beside two power-law ones, make 0.16
// flushes per non-zero, not 0.5: R = 32: 610 us as they lie and 650 moved; R = 64: 1205 and 918;
// R = 128: 2648 and 1492.
static bool group_pays(const blco_tensor* t, int mode, int rank, int64_t n) {
  if (!t->d_group || !t->grouped[mode] || n != t->nnz) return false;
  const double W = rank > 64 ? 1024 : 2048, N = (double)n;
  const double lines = ceil(rank / 16.0) + (rank % 16 ? 0.5 : 0.0);
  const double even = window_flushes(t, mode, rank > 32 && rank <= 64 ? 4096 : W, N);
  const double half = flushes(t, mode, 0), whole = flushes(t, mode, 1);
  const double now = rank > 32 && rank <= 64 && half - whole >= wide_saves(t->lay.N) ? whole : half;
  // in bucket order: W non-zeros of the rows of W / (n / buckets) buckets, at least one
  const double per = N / kGroupBuckets, I = (double)t->lay.dims[mode];
  const double rows = std::max(1.0, I / kGroupBuckets * std::max(1.0, W / per));
  const double then = rows * -expm1(-W / rows) / W + 1.0 / per;
  const double move = 20e-6 + N * 18e-12;
  return N * (even - std::min(even, then)) * lines * 52e-12 > 2 * move &&
         N * (now - std::min(now, then)) * lines * 52e-12 > 1.2 * move;
}

// How a call runs: padded factors (their row stride, 0: as they are) and output rows,
// grouping, and the workspace that takes.
struct CallPlan {
  int pad;
  int out;       // elements between flushed rows (the rank: the output itself)
  bool group;
  size_t copy_bytes;
  size_t bytes;
  int outs;      // copies of the output
  bool wide;     // windows of 4096 for want of room for those
};

// careful: only padded factors, which change no sum.
static CallPlan plan_call(const blco_tensor* t, int mode, int rank, int fdt, int res, bool resid,
                          int64_t n, size_t room, bool careful) {
  const int N = t->lay.N;
  const size_t fsz = factor_elem_bytes(fdt);
  CallPlan c = {0, rank, false, 0, 0, 1, false};
  const bool reg = res == BLCO_RES_REGISTER;
  auto left = [&] { return room > c.bytes ? room - c.bytes : 0; };
  const bool big = big_gathers(t, mode, rank, fdt, false, false) ||
                   big_gathers(t, mode, rank, fdt, true, resid);
  if (reg && !careful) {
    c.copy_bytes = up256(plan_win(t, mode, rank, rank, rank, rank % 2 == 0, fdt,
                                  big_gathers(t, mode, rank, fdt, true, resid), resid, n, room,
                                  false, false, false)
                             .bytes);
    c.bytes = c.copy_bytes;
  }
  if (!big) {
    const int Rp = padded_rank(t, mode, rank, fdt, resid, n);
    size_t bytes = 0;
    for (int m = 0; m < N; ++m)
      if (m != mode || resid) bytes += up256((size_t)t->lay.dims[m] * Rp * fsz);
    if (Rp != rank && bytes <= left()) {
      c.pad = Rp;
      c.bytes += bytes;
    }
  }
  if (reg && !big && !careful) {
    const int Ro = padded_out(t, mode, rank, n);
    const size_t bytes = up256((size_t)t->lay.dims[mode] * Ro * sizeof(float));
    if (Ro != rank && bytes <= left()) {
      c.out = Ro;
      c.bytes += bytes;
    }
  }
  if (reg && !resid && !big && !careful && group_pays(t, mode, rank, n)) {
    const size_t bytes =
        up256(8 * (size_t)n) + up256(4 * (size_t)n) + up256(4 * (size_t)kGroupBuckets);
    if (bytes <= left()) {
      c.group = true;
      c.bytes += bytes;
    }
  }
  if (reg && !resid && !careful) {
    const int outs = out_copies(t, mode, rank, c.pad ? c.pad : rank, c.group, n);
    if (outs > 1) {
      const int Ro = (rank + 15) / 16 * 16;
      const size_t one = up256((size_t)t->lay.dims[mode] * Ro * sizeof(float));
      const size_t bytes = one * (size_t)(c.out != rank ? outs - 1 : outs);
      if (!big && one * (size_t)outs <= kPadMax && bytes <= left()) {
        c.out = Ro;
        c.outs = outs;
        c.bytes += bytes;
      } else {
        c.wide = true;
      }
    }
  }
  return c;
}

// Everything a launch over n non-zeros decides: resolution, addressing, CallPlan and, where the
// window kernel runs, WinPlan.
struct LaunchPlan {
  int res;
  int sw;               // hierarchical kernel: ranks per slice
  bool big, big_win;    // 64-bit addresses in the hierarchical / the window kernel
  CallPlan cp;
  int stride;           // elements between factor rows
  WinPlan w;
  int64_t grid;         // workgroups of the window kernel
};

static int plan_launch(const blco_tensor* t, int mode, int rank, int fdt, bool resid, int64_t n,
                       size_t room, bool careful, LaunchPlan* L) {
  L->res = resolve(t, mode, rank, &L->sw);
  if (L->res < 0) return L->res;
  L->big = big_gathers(t, mode, rank, fdt, false, false);
  L->big_win = big_gathers(t, mode, rank, fdt, true, resid);
  L->cp = plan_call(t, mode, rank, fdt, L->res, resid, n, room, careful);
  L->stride = L->cp.pad ? L->cp.pad : rank;
  if (L->res != BLCO_RES_REGISTER) return BLCO_OK;
  L->w = plan_win(t, mode, L->cp.out, rank, L->stride, L->stride % 2 == 0, fdt, L->big_win, resid,
                  n, L->cp.copy_bytes, careful, L->cp.group, L->cp.wide);
  // with a stash: persistent workgroups, kWinRounds times the resident count
  // (two per CU) in a long launch, which balances its end (1-2% faster than one round
  // on 50M non-zeros); once the resident count in a shorter one, where the stash
  // flushes count more (2M non-zeros, R = 16: 68 us and 58 us); without one: a
  // workgroup per window (about 1% faster than persistent ones)
  const int rounds = careful || L->w.nwin >= 16 * 1024 ? kWinRounds : 1;
  L->grid = L->w.stash > 0 ? std::min<int64_t>(L->w.nwin, (int64_t)device_cus() * 2 * rounds)
                           : L->w.nwin;
  return BLCO_OK;
}

// Launch the MTTKRP kernel over [lo, lo + n) of the tensor given by keys/vals, clearing the
// output first if `clear`.
// With resid != nullptr the fused residual walk runs instead (the caller has
// checked fused_mode_ok): resid[0, n) receives the residual of each non-zero.
static int launch_mttkrp(const blco_tensor* t, const uint64_t* keys, const float* vals,
                         int64_t lo, int64_t n, int mode, const void* const* factors, int fdt,
                         int rank, float scale, const double* scale_dev, float* out,
                         hipStream_t s, const Work& ws, bool clear, float* resid = nullptr) {
  const int64_t clear_n = clear ? (int64_t)t->lay.dims[mode] * rank : 0;
  if (n <= 0) return fill_zero(out, clear_n, s);
  const int N = t->lay.N;
  KParams p;
  fill_params(t, &p);
  p.keys = keys;
  p.vals = vals;
  p.base = lo;
  p.n = n;
  for (int m = 0; m < N; ++m) p.A[m] = factors[m];
  p.out = out;
  p.R = rank;
  p.mode = mode;
  p.scale = scale;
  p.scale_dev = scale_dev;
  p.resid = resid;
  const size_t fsz = factor_elem_bytes(fdt);
  LaunchPlan L;
  int rc = plan_launch(t, mode, rank, fdt, resid != nullptr, n, ws.bytes, ws.careful, &L);
  if (rc) return rc;
  const CallPlan& cp = L.cp;
  const int stride = L.stride;
  if (resid && (L.res != BLCO_RES_REGISTER || L.big || rank > 64 ||
                (size_t)t->lay.dims[mode] * rank * fsz > 0xFFFFFFFFull))
    return set_error(BLCO_EUNSUPPORTED, "fused residual walk on mode %d", mode);
  // the workspace: hot copies, padded factors, grouped non-zeros and their cursors
  PrepParams pre = {};
  pre.zero[0] = out;
  pre.nzero[0] = clear_n;
  char* at = ws.p + cp.copy_bytes;
  if (cp.pad) {
    pre.R = rank;
    pre.Rp = stride;
    for (int m = 0; m < N; ++m) {
      if (m == mode && !resid) continue;
      pre.src[pre.npad] = factors[m];
      pre.dst[pre.npad] = at;
      pre.rows[pre.npad++] = (int64_t)t->lay.dims[m];
      p.A[m] = at;
      at += up256((size_t)t->lay.dims[m] * stride * fsz);
    }
  }
  p.rowbytes = (uint32_t)((size_t)stride * fsz);
  for (int m = 0; m < N; ++m) {
    const size_t bytes = (size_t)t->lay.dims[m] * stride * fsz;
    p.abytes[m] = (uint32_t)std::min<size_t>(bytes, 0xFFFFFFFFull);
  }
  if (L.res == BLCO_RES_HIERARCHICAL) {
    if ((rc = prepare(pre, fdt, s))) return rc;
    const int sw = L.sw;
    p.short_rows = (uint32_t)t->lay.dims[mode];
    p.short_width = sw;
    const int slices = (rank + sw - 1) / sw;
    // two resident workgroups per CU over all slices; each takes an equal range of at
    // least one batch (four batches left a short launch on a few CUs: 100k non-zeros,
    // R = 32, 200 rows: 26 us with four, 10 us with one; a CP-ALS update keeps four)
    const int64_t want = std::max<int64_t>(device_cus() * 2 / slices, 1);
    int64_t per = std::max<int64_t>((n + want - 1) / want, (int64_t)kShortB * (ws.careful ? 4 : 1));
    per = (per + kShortB - 1) / kShortB * kShortB;
    const int64_t nwg = (n + per - 1) / per;
    const size_t lds = short_lds(N, t->lay.dims[mode], sw);
    ShortFn f = select_short(N, sw, stride, fdt, L.big);
    hipLaunchKernelGGL(f, dim3((unsigned)nwg, (unsigned)slices), dim3(kShortB), lds, s, p, per);
    HIPCHK(hipGetLastError());
    return BLCO_OK;
  }
  // flushed rows in the workspace: their padding takes the sums of padded gathers (zeros)
  float* rows = out;
  const int ro = cp.out;
  const bool apart = ro != rank || cp.outs > 1;
  p.out_copies = cp.outs;
  if (apart) {
    rows = reinterpret_cast<float*>(at);
    const size_t one = up256((size_t)t->lay.dims[mode] * ro * sizeof(float));
    at += one * (size_t)cp.outs;
    p.out_step = (int64_t)(one / sizeof(float));
    pre.zero[0] = rows;
    pre.nzero[0] = p.out_step * cp.outs;
    p.R = ro;
  }
  if (cp.group) {
    uint64_t* gk = reinterpret_cast<uint64_t*>(at);
    at += up256(8 * (size_t)n);
    float* gv = reinterpret_cast<float*>(at);
    at += up256(4 * (size_t)n);
    pre.starts = t->d_group + (size_t)mode * kGroupBuckets;
    pre.cursor = reinterpret_cast<uint32_t*>(at);
    p.keys = gk;
    p.vals = gv;
  }
  p.RG = stride;
  p.RV = std::max(rank, std::min(stride, ro));
  p.out = rows;
  const WinPlan& w = L.w;
  p.hot = t->d_hot + (size_t)mode * kHotMax;
  p.nhot = w.stash;
  if (w.copies) {
    float* copy = reinterpret_cast<float*>(ws.p);
    p.tab = t->d_tab + (size_t)mode * kTabWords;
    p.copy_off = reinterpret_cast<char*>(copy) - reinterpret_cast<char*>(rows);
    p.copies = w.copies;
    p.copy_stride = copy_stride(rank);
    pre.zero[1] = copy;
    pre.nzero[1] = (int64_t)(w.bytes / sizeof(float));
  }
  if ((rc = prepare(pre, fdt, s))) return rc;
  if (cp.group) {
    const int64_t per = 1024 * kGroupPer;
    hipLaunchKernelGGL(k_group, dim3((unsigned)((n + per - 1) / per)), dim3(1024), 0, s, keys,
                       vals, n, (int)p.shift[mode], p.mask[mode], t->group_mul[mode], pre.cursor,
                       const_cast<uint64_t*>(p.keys), const_cast<float*>(p.vals));
    HIPCHK(hipGetLastError());
  }
  const size_t dyn = w.stash > 0 ? (size_t)w.stash * ro * 4 + 2 * (size_t)kHotSlots * 4 : 0;
  hipLaunchKernelGGL(w.f, dim3((unsigned)L.grid), dim3(kWin), dyn, s, p);
  HIPCHK(hipGetLastError());
  if (w.copies) {
    hipLaunchKernelGGL(k_hot_sum, dim3((unsigned)t->nhot[mode]), dim3(kBlock), 0, s,
                       (const float*)ws.p, p.hot, p.copies, p.copy_stride, rank, ro, rows);
    HIPCHK(hipGetLastError());
  }
  if (apart) {
    const int64_t I = (int64_t)t->lay.dims[mode];
    const int64_t blocks = std::min<int64_t>((I * rank + 255) / 256, 8192);
    hipLaunchKernelGGL(k_unpad, dim3((unsigned)blocks), dim3(256), 0, s, (const float*)rows, I, rank,
                       ro, cp.outs, p.out_step, clear ? 0 : 1, out);
    HIPCHK(hipGetLastError());
  }
  return BLCO_OK;
}

int blco::device_alloc(void** p, size_t bytes) {
  *p = nullptr;
  const hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) return BLCO_OK;
  *p = nullptr;
  (void)hipGetLastError();
  return set_error(e == hipErrorOutOfMemory ? BLCO_ENOMEM : BLCO_EDEVICE,
                   "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
}

static void* pinned_alloc(size_t n) {
  void* p = nullptr;
  if (hipHostMalloc(&p, n, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return p;
}
static void pinned_free(void* p) { (void)hipHostFree(p); }


template <class T>
static int upload(T** dst, const T* src, size_t count, size_t* acc) {
  size_t bytes = sizeof(T) * std::max<size_t>(count, 1);
  int rc = device_alloc((void**)dst, bytes);
  if (rc) return rc;
  if (count) HIPCHK(hipMemcpy(*dst, src, sizeof(T) * count, hipMemcpyHostToDevice));
  *acc += bytes;
  return BLCO_OK;
}

// The copies of streamed calls queued on one stream follow one another: a call's copies start
// when kCopyLead bytes are left of those of the call queued there before it.  Its kernels come
// after that call's anyway, so nothing completes later for the wait; but where tensors are
// streamed in turn, each through its own copy stream, their copies otherwise share the host link,
// which then moves less, and the first call's kernels start late.  The lead covers what a wait
// between streams costs.  Three tensors in turn, us per call without waiting, waiting for all, and
// for all but 64 MiB: 20M non-zeros (240 MB) 4570, 4385 and 4340; 10.6M in two chunks 2295, 2357 and
// 2288; 7.7M (R = 64) 2207, 2082 and 2101; 3.7M 812, 843 and 811; 2.1M 470, 508 and 470.  The
// streams most recently used, kept while any tensor has been streamed.
constexpr int64_t kCopyLead = (int64_t)64 << 20;
struct LastCopies {
  struct Entry {
    int dev;
    hipStream_t s;
    hipEvent_t done;
    uint64_t used;
  };
  static constexpr size_t kMost = 16;
  std::mutex mu;
  std::vector<Entry> e;
  uint64_t calls = 0;
  int tensors = 0;

  Entry* find(int dev, hipStream_t s) {
    for (Entry& x : e)
      if (x.dev == dev && x.s == s) return &x;
    return nullptr;
  }
  // copies queued on cs from now on wait for the last ones of calls on s
  hipError_t follow(int dev, hipStream_t s, hipStream_t cs) {
    std::lock_guard<std::mutex> lock(mu);
    const Entry* x = find(dev, s);
    return x ? hipStreamWaitEvent(cs, x->done, 0) : hipSuccess;
  }
  // the next call on s starts its copies behind what has been queued on cs
  hipError_t mark(int dev, hipStream_t s, hipStream_t cs) {
    std::lock_guard<std::mutex> lock(mu);
    Entry* x = find(dev, s);
    if (!x) {
      if (e.size() >= kMost) {
        auto old = std::min_element(e.begin(), e.end(), [](const Entry& a, const Entry& b) {
          return a.used < b.used;
        });
        (void)hipEventDestroy(old->done);
        e.erase(old);
      }
      hipEvent_t ev;
      hipError_t rc = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
      if (rc != hipSuccess) return rc;
      e.push_back({dev, s, ev, 0});
      x = &e.back();
    }
    x->used = ++calls;
    return hipEventRecord(x->done, cs);
  }
  void add() {
    std::lock_guard<std::mutex> lock(mu);
    ++tensors;
  }
  void drop() {
    std::lock_guard<std::mutex> lock(mu);
    if (--tensors > 0) return;
    for (Entry& x : e) (void)hipEventDestroy(x.done);
    e.clear();
  }
};
static LastCopies& last_copies() {
  static LastCopies* l = new LastCopies;   // outlives every tensor freed at exit
  return *l;
}

static void release_device(blco_tensor* t) {
  StreamState& st = t->st;
  if (st.copy_stream) {
    (void)hipStreamSynchronize((hipStream_t)st.copy_stream);
    for (int i = 0; i < 2; ++i) {
      if (st.ev_free[i]) (void)hipEventSynchronize((hipEvent_t)st.ev_free[i]);
    }
  }
  for (void* e : st.ev_t) {
    (void)hipEventSynchronize((hipEvent_t)e);
    (void)hipEventDestroy((hipEvent_t)e);
  }
  for (int i = 0; i < 2; ++i) {
    if (st.d_keys[i]) (void)hipFree(st.d_keys[i]);
    if (st.d_vals[i]) (void)hipFree(st.d_vals[i]);
    if (st.d_res[i]) (void)hipFree(st.d_res[i]);
    if (st.ev_ready[i]) (void)hipEventDestroy((hipEvent_t)st.ev_ready[i]);
    if (st.ev_free[i]) (void)hipEventDestroy((hipEvent_t)st.ev_free[i]);
  }
  if (st.copy_stream) {
    (void)hipStreamDestroy((hipStream_t)st.copy_stream);
    last_copies().drop();
  }
  st = StreamState();
  for (void* q : {(void*)t->d_keys, (void*)t->d_vals, (void*)t->d_run_start, (void*)t->d_run_base,
                  (void*)t->d_tile_run, (void*)t->d_partials, (void*)t->d_hot, (void*)t->d_tab,
                  (void*)t->d_group})
    if (t->owned(q)) (void)hipFree(q);
  t->d_group = nullptr;
  t->d_hot = nullptr;
  t->d_tab = nullptr;
  t->d_keys = nullptr;
  t->d_vals = nullptr;
  t->d_run_start = nullptr;
  t->d_run_base = nullptr;
  t->d_tile_run = nullptr;
  t->d_partials = nullptr;
}

int blco::count_flushes_device(blco_tensor* t, uint32_t* counts, void* stream) {
  if (t->nnz < kFlushMin) return BLCO_OK;
  hipStream_t s = (hipStream_t)stream;
  KParams p;
  fill_params(t, &p);
  p.keys = t->d_keys;
  p.n = t->nnz;
  hipLaunchKernelGGL(k_flushes, dim3((unsigned)kFlushSamples, (unsigned)t->lay.N), dim3(1024), 0, s, p,
                     counts);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

// Counts the buckets of the modes k_group may serve: flat modes of a device tensor of one run
// without block-key bits, long enough to have several rows per bucket, whose windows hardly
// repeat a row.
int blco::make_groups(blco_tensor* t, void* stream) {
  const Layout& L = t->lay;
  if (!t->d_keys || t->nnz < kGroupMinNnz || t->nnz >= ((int64_t)1 << 32) ||
      t->run_start.size() != 2 || L.S > 0)
    return BLCO_OK;
  auto flat = [&](int m) {
    return L.dims[m] >= 4 * (uint64_t)kGroupBuckets && !has_frequent_rows(t, m) &&
           window_flushes(t, m, 2048.0, (double)t->nnz) >= 0.4;
  };
  bool any = false;
  for (int m = 0; m < L.N; ++m) any = any || flat(m);
  if (!any) return BLCO_OK;
  hipStream_t s = (hipStream_t)stream;
  HIPCHK(hipStreamSynchronize(s));   // the counted flushes
  any = false;
  for (int m = 0; m < L.N; ++m) {
    t->grouped[m] = flat(m) && flushes(t, m, 0) >= 0.1;   // fewer never pay (group_pays)
    any = any || t->grouped[m];
  }
  if (!any) return BLCO_OK;
  if (!t->d_group) {
    const size_t bytes = sizeof(uint32_t) * (size_t)L.N * kGroupBuckets;
    int rc = device_alloc((void**)&t->d_group, bytes);
    if (rc) return rc;
    t->device_bytes += bytes;
  }
  int rc = fill_zero(reinterpret_cast<float*>(t->d_group), (int64_t)L.N * kGroupBuckets, s);
  if (rc) return rc;
  KParams p;
  fill_params(t, &p);
  for (int m = 0; m < L.N; ++m) {
    if (!t->grouped[m]) continue;
    t->group_mul[m] = (uint32_t)(((uint64_t)kGroupBuckets << 32) / L.dims[m]);
    uint32_t* c = t->d_group + (size_t)m * kGroupBuckets;
    hipLaunchKernelGGL(k_group_count, dim3(256), dim3(256), 0, s, (const uint64_t*)t->d_keys,
                       t->nnz, (int)p.shift[m], p.mask[m], t->group_mul[m], c);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(k_group_starts, dim3(1), dim3(kGroupBuckets), 0, s, c);
    HIPCHK(hipGetLastError());
  }
  return BLCO_OK;
}

// ====================================================================== C ABI

extern "C" int blco_build(int nmodes, const uint64_t* dims, int64_t nnz,
                          const uint32_t* const* coords, const float* values,
                          const blco_build_opts* opts, blco_tensor** out) {
  clear_error();
  if (!out) return set_error(BLCO_EINVAL, "out is NULL");
  *out = nullptr;
  int key_bits = 64;
  int64_t cap = (int64_t)1 << 27;
  int placement = BLCO_PLACE_DEVICE;
  int64_t hot_min = kHotMinCount;
  if (opts) {
    key_bits = opts->key_bits;
    cap = opts->max_block_nnz;
    placement = opts->placement;
    if (opts->hot_min_count != 0) hot_min = opts->hot_min_count;
  }
  const bool hot_forced = opts && opts->hot_min_count > 0;
  if (placement != BLCO_PLACE_DEVICE && placement != BLCO_PLACE_PINNED &&
      placement != BLCO_PLACE_HOST)
    return set_error(BLCO_EINVAL, "placement %d", placement);
  blco_tensor* t = new (std::nothrow) blco_tensor();
  if (!t) return set_error(BLCO_ENOMEM, "host allocation failed");
  t->placement = placement;
  HostAlloc ha = nullptr;
  HostFree hf = nullptr;
  if (placement == BLCO_PLACE_PINNED) {
    ha = pinned_alloc;
    hf = pinned_free;
  }
  int rc = host_build(nmodes, dims, nnz, coords, values, key_bits, cap, ha, hf, t);
  if (rc) {
    delete t;
    return rc;
  }
  find_hot_rows(coords, nnz, hot_min, t);
  make_row_tables(t);
  count_flushes(t);
  t->hot_forced = hot_forced;
  if (placement == BLCO_PLACE_HOST) {
    *out = t;
    return BLCO_OK;
  }
  auto fail = [&](int code) {
    release_device(t);
    free_host_arrays(t);
    delete t;
    return code;
  };
  if (hipGetDevice(&t->device) != hipSuccess) {
    set_error(BLCO_EDEVICE, "hipGetDevice failed");
    return fail(BLCO_EDEVICE);
  }
  size_t acc = 0;
  if ((rc = upload(&t->d_run_start, t->run_start.data(), t->run_start.size(), &acc))) return fail(rc);
  if ((rc = upload(&t->d_run_base, t->run_base.data(), t->run_base.size(), &acc))) return fail(rc);
  if ((rc = upload(&t->d_tile_run, t->tile_run.data(), t->tile_run.size(), &acc))) return fail(rc);
  if ((rc = upload(&t->d_hot, t->hot.data(), t->hot.size(), &acc))) return fail(rc);
  if ((rc = upload(&t->d_tab, t->tab.data(), t->tab.size(), &acc))) return fail(rc);
  if (placement == BLCO_PLACE_DEVICE) {
    if ((rc = upload(&t->d_keys, t->h_keys, (size_t)nnz, &acc))) return fail(rc);
    if ((rc = upload(&t->d_vals, t->h_vals, (size_t)nnz, &acc))) return fail(rc);
    free_host_arrays(t);
  }
  t->device_bytes = acc;
  if (placement == BLCO_PLACE_DEVICE) {
    if ((rc = make_groups(t, nullptr))) return fail(rc);
    if (hipStreamSynchronize(nullptr) != hipSuccess) {
      set_error(BLCO_EDEVICE, "bucket counts failed");
      return fail(BLCO_EDEVICE);
    }
  }
  *out = t;
  return BLCO_OK;
}

// Whether a mode's launch gathers with 64-bit addresses in the window kernel / elsewhere:
// factors below 4 GiB are gathered with 32-bit byte offsets, larger ones with 64-bit
// addresses; the window kernel's fp32 gathers at 33-64 ranks (ld_base; not the fused
// residual walk) also take a factor of exactly 4 GiB with 32-bit offsets.  An output of more
// than kIndexMax elements takes the window kernel's 64-bit form too.
static bool big_gathers(const blco_tensor* t, int mode, int rank, int fdt, bool window,
                        bool resid) {
  const size_t fsz = factor_elem_bytes(fdt);
  if ((size_t)rank * fsz >= (1ULL << 31)) return true;
  const bool base32 = window && fdt == BLCO_F32 && rank > 32 && rank <= 64 && !resid;
  for (int m = 0; m < t->lay.N; ++m)
    if (m != mode &&
        (size_t)t->lay.dims[m] * rank * fsz > (base32 ? (1ULL << 32) : 0xFFFFFFFFull))
      return true;
  return window && (uint64_t)t->lay.dims[mode] * (uint64_t)rank > kIndexMax;
}

// Workspace the MTTKRP of mode `mode` over n non-zeros can use (0: none).
static size_t mode_workspace(const blco_tensor* t, int mode, int rank, int fdt, bool resid,
                             int64_t n, bool careful = false) {
  int sw = 0;
  const int res = n > 0 ? resolve(t, mode, rank, &sw) : BLCO_EINVAL;
  if (res < 0) {
    clear_error();
    return 0;
  }
  return plan_call(t, mode, rank, fdt, res, resid, n, ~(size_t)0 / 2, careful).bytes;
}

// The in-memory MTTKRP calls, with an optional workspace.
static int mttkrp_impl(blco_tensor* t, int mode, const float* values, const void* const* factors,
                       int factor_dtype, int rank, const double* scale, double alpha,
                       bool accumulate, float* out, const Work& ws, hipStream_t s) {
  int rc = check_factor_args(t, mode, factors, factor_dtype, rank, out, false);
  if (rc) return rc;
  if (t->placement != BLCO_PLACE_DEVICE)
    return set_error(BLCO_EINVAL, "in-memory MTTKRP needs a tensor placed on the device; "
                                  "use blco_mttkrp_stream for a pinned tensor");
  if (!values && t->nnz > 0) return set_error(BLCO_EINVAL, "values is NULL");
  return launch_mttkrp(t, t->d_keys, values, 0, t->nnz, mode, factors, factor_dtype, rank,
                       (float)alpha, scale, out, s, ws, !accumulate);
}

size_t blco::mttkrp_workspace(const blco_tensor* t, int mode, int rank, int factor_dtype) {
  return mode_workspace(t, mode, rank, factor_dtype, false, t->nnz, true);
}

int blco::mttkrp_careful(blco_tensor* t, int mode, const void* const* factors, int factor_dtype,
                         int rank, float* out, void* ws, size_t ws_bytes, void* stream) {
  return mttkrp_impl(t, mode, t->d_vals, factors, factor_dtype, rank, nullptr, 1.0, false, out,
                     Work{static_cast<char*>(ws), ws_bytes, true}, (hipStream_t)stream);
}

static int make_work(void* ws, size_t bytes, Work* w) {
  if (!ws && bytes > 0) return set_error(BLCO_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) & 255)
    return set_error(BLCO_EINVAL, "workspace must be 256-byte aligned");
  *w = Work{static_cast<char*>(ws), ws ? bytes : 0, false};
  return BLCO_OK;
}

extern "C" int blco_mttkrp_v(blco_tensor* t, int mode, const float* values,
                             const void* const* factors, int factor_dtype, int rank,
                             const double* scale, double alpha, float* out, void* stream) {
  clear_error();
  return mttkrp_impl(t, mode, values, factors, factor_dtype, rank, scale, alpha, false, out,
                     Work(), (hipStream_t)stream);
}

extern "C" int blco_mttkrp(blco_tensor* t, int mode, const void* const* factors, int factor_dtype,
                           int rank, float* out, void* stream) {
  clear_error();
  return mttkrp_impl(t, mode, t ? t->d_vals : nullptr, factors, factor_dtype, rank, nullptr, 1.0,
                     false, out, Work(), (hipStream_t)stream);
}

extern "C" int blco_mttkrp_acc(blco_tensor* t, int mode, const void* const* factors,
                               int factor_dtype, int rank, float* out, void* stream) {
  clear_error();
  return mttkrp_impl(t, mode, t ? t->d_vals : nullptr, factors, factor_dtype, rank, nullptr, 1.0,
                     true, out, Work(), (hipStream_t)stream);
}

extern "C" int blco_mttkrp_ws(blco_tensor* t, int mode, const float* values,
                              const void* const* factors, int factor_dtype, int rank,
                              const double* scale, double alpha, int accumulate, float* out,
                              void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  Work ws;
  int rc = make_work(workspace, workspace_bytes, &ws);
  if (rc) return rc;
  return mttkrp_impl(t, mode, values ? values : (t ? t->d_vals : nullptr), factors, factor_dtype,
                     rank, scale, alpha, accumulate != 0, out, ws, (hipStream_t)stream);
}

// Whether the fused residual walk can serve mode m: register-based resolution,
// one rank slice of 16-lane groups (R <= 64) and 32-bit gather offsets.
static bool fused_mode_ok(const blco_tensor* t, int m, int rank, int fdt) {
  int sw = 0;
  if (resolve(t, m, rank, &sw) != BLCO_RES_REGISTER) {
    clear_error();
    return false;
  }
  const size_t fsz = factor_elem_bytes(fdt);
  if (rank > 64 || (size_t)rank * fsz >= (1ULL << 31)) return false;
  for (int j = 0; j < t->lay.N; ++j)
    if ((size_t)t->lay.dims[j] * rank * fsz > 0xFFFFFFFFull) return false;
  return true;
}

// Partial sums the loss needs per launch of the sampled-loss kernel over n non-zeros.
static int64_t loss_blocks(int64_t n) { return ((n + 63) / 64 + kWaves - 1) / kWaves; }

// The sampled-loss kernel over [lo, lo + n) of the tensor given by keys/vals: the
// residual of each non-zero into resid (may be NULL) and one fp64 partial sum of
// squared residuals per workgroup into partials[0, loss_blocks(n)).
static int launch_loss(const blco_tensor* t, const uint64_t* keys, const float* vals, int64_t lo,
                       int64_t n, const void* const* factors, int fdt, int rank, float* resid,
                       double* partials, hipStream_t s) {
  if (n <= 0) return BLCO_OK;
  KParams p;
  fill_params(t, &p);
  p.keys = keys;
  p.vals = vals;
  p.base = lo;
  p.n = n;
  for (int m = 0; m < t->lay.N; ++m) p.A[m] = factors[m];
  p.out = resid;
  p.partials = partials;
  p.R = rank;
  p.mode = -1;
  // factors below 4 GiB are gathered with 32-bit byte offsets, larger ones
  // with 64-bit addresses
  const size_t fsz = factor_elem_bytes(fdt);
  p.rowbytes = (uint32_t)((size_t)rank * fsz);
  bool big = (size_t)rank * fsz >= (1ULL << 31);
  for (int m = 0; m < t->lay.N; ++m) {
    const size_t bytes = (size_t)t->lay.dims[m] * rank * fsz;
    p.abytes[m] = (uint32_t)std::min<size_t>(bytes, 0xFFFFFFFFull);
    if (bytes > 0xFFFFFFFFull) big = true;
  }
  KernelFn f = select_loss(t->lay.N, rank, fdt, big);
  hipLaunchKernelGGL(f, dim3((unsigned)loss_blocks(n)), dim3(kBlock), 0, s, p);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

// Device array of at least `count` fp64 partial sums held by the tensor.
static int ensure_partials(blco_tensor* t, int64_t count, hipStream_t s) {
  count = std::max<int64_t>(count, 1);
  if (t->partials_cap >= count) return BLCO_OK;
  if (t->d_partials) {
    HIPCHK(hipStreamSynchronize(s));
    HIPCHK(hipFree(t->d_partials));
    t->d_partials = nullptr;
    t->partials_cap = 0;
  }
  int rc = device_alloc((void**)&t->d_partials, sizeof(double) * (size_t)count);
  if (rc) return rc;
  t->partials_cap = count;
  return BLCO_OK;
}

// The CP gradient of blco_cp_grad inside stream_modes: the residual comes from the
// fused walk of mode m0 (or, when no mode allows it, from the sampled-loss kernel)
// and feeds the other modes' MTTKRPs.
struct GradArgs {
  int m0;                   // mode of the fused residual walk, -1: sampled-loss kernel first
  float scale;              // host-side scale of every gradient term (-alpha)
  const double* scale_dev;  // optional device-side scale
  float* resid;             // DEVICE placement: the caller's residual (nnz)
  double* loss;             // device: 1/2 sum of squared residuals
  double* partials;         // DEVICE placement: workspace of partial sums, NULL: the tensor's
};

// Residual and gradients of one range [lo, lo + n) whose keys/vals are given;
// partial sums of squared residuals go to part[0, ...) and their count to *nparts.
static int grad_range(blco_tensor* t, const GradArgs& g, const uint64_t* keys, const float* vals,
                      int64_t lo, int64_t n, const void* const* factors, int fdt, int rank,
                      float* const* outs, float* resid, double* part, int64_t* nparts,
                      hipStream_t s, const Work& ws, bool clear) {
  int rc;
  *nparts = 0;
  if (n <= 0) return BLCO_OK;
  if (g.m0 >= 0) {
    if ((rc = launch_mttkrp(t, keys, vals, lo, n, g.m0, factors, fdt, rank, g.scale, g.scale_dev,
                            outs[g.m0], s, ws, clear, resid)))
      return rc;
    *nparts = (n + kSqPer - 1) / kSqPer;
    hipLaunchKernelGGL(k_sumsq, dim3((unsigned)*nparts), dim3(256), 0, s, (const float*)resid, n,
                       part);
    HIPCHK(hipGetLastError());
  } else {
    if ((rc = launch_loss(t, keys, vals, lo, n, factors, fdt, rank, resid, part, s))) return rc;
    *nparts = loss_blocks(n);
  }
  for (int m = 0; m < t->lay.N; ++m) {
    if (m == g.m0) continue;
    if ((rc = launch_mttkrp(t, keys, resid, lo, n, m, factors, fdt, rank, g.scale, g.scale_dev,
                            outs[m], s, ws, clear)))
      return rc;
  }
  return BLCO_OK;
}

// Partial sums per range of n non-zeros (the larger of the two kernels' counts).
static int64_t grad_parts(int64_t n) {
  return std::max<int64_t>((n + kSqPer - 1) / kSqPer, loss_blocks(n));
}

// First mode whose MTTKRP can carry the gradient's fused residual walk, or -1.
static int fused_mode(const blco_tensor* t, int rank, int fdt) {
  for (int m = 0; m < t->lay.N; ++m)
    if (fused_mode_ok(t, m, rank, fdt)) return m;
  return -1;
}

// Device memory of a call over the selected modes (one bit each) under a budget: what it cannot do
// without, the non-zeros per staging buffer and the bytes of workspace it uses of those lent.
struct StreamPlan {
  size_t fixed;     // factors read + selected outputs + the tensor's own arrays
  size_t per_nnz;   // staging: key and value, and the chunk's residual for the gradient
  int64_t cap;      // non-zeros per staging buffer
  size_t ws;
};

// The staging comes first: the workspace has what the staging leaves over (the staging ends at
// the tensor's size or its blocks'), or takes at most an eighth of the memory for both, and only
// as much as launches over a chunk of that size use.  Streaming is bound by the host link, so
// larger chunks cost nothing that a workspace could give back, while chunks of 64 non-zeros
// cost four events and every mode's launches each.
static int plan_stream(const blco_tensor* t, unsigned modes, bool grad, int rank, int fdt,
                       size_t budget, size_t lent, StreamPlan* p) {
  const Layout& L = t->lay;
  bool need[BLCO_MAX_MODES] = {};
  p->fixed = t->device_bytes;
  for (int m = 0; m < L.N; ++m) {
    if (!(modes >> m & 1)) continue;
    p->fixed += (size_t)L.dims[m] * rank * sizeof(float);
    for (int j = 0; j < L.N; ++j)
      if (j != m || grad) need[j] = true;   // the residual reads every factor
  }
  for (int m = 0; m < L.N; ++m)
    if (need[m]) p->fixed += (size_t)L.dims[m] * rank * factor_elem_bytes(fdt);
  const int m0 = grad ? fused_mode(t, rank, fdt) : -1;
  auto used = [&](int64_t n) {
    size_t most = 0;
    if (lent > 0)
      for (int m = 0; m < L.N; ++m)
        if (modes >> m & 1) most = std::max(most, mode_workspace(t, m, rank, fdt, m == m0, n));
    return std::min(most, lent);
  };
  p->cap = 0;
  p->per_nnz = 0;
  if (t->placement == BLCO_PLACE_DEVICE) {
    if (p->fixed > budget)
      return set_error(BLCO_ENOMEM, "budget %zu below factors + outputs + tensor = %zu", budget,
                       p->fixed);
    const size_t ws = used(t->nnz);
    p->ws = ws <= budget - p->fixed ? ws : 0;
    return BLCO_OK;
  }
  p->per_nnz = sizeof(uint64_t) + sizeof(float) + (grad ? sizeof(float) : 0);
  if (budget < p->fixed + 2 * 64 * p->per_nnz)
    return set_error(BLCO_ENOMEM, "budget %zu cannot hold factors + outputs + tables (%zu) and "
                                  "two staging buffers", budget, p->fixed);
  auto staged = [&](size_t room) {
    int64_t cap = (int64_t)(room / 2 / p->per_nnz);
    cap = std::min(cap, ((t->max_block_nnz + 63) / 64) * 64);
    cap = std::min(cap, ((t->nnz + 63) / 64) * 64);
    return std::max<int64_t>(cap / 64 * 64, 64);
  };
  const size_t room = budget - p->fixed;
  p->cap = staged(room);
  p->ws = used(p->cap);
  if (p->ws <= room - 2 * (size_t)p->cap * p->per_nnz) return BLCO_OK;
  const int64_t less = p->ws <= room / 8 ? staged(room - p->ws) : 0;
  p->ws = less ? std::min(p->ws, used(less)) : 0;
  if (p->ws) p->cap = less;
  return BLCO_OK;
}

// Stream the pinned non-zeros once through two reused staging buffers and,
// for every chunk, run the MTTKRP of each selected mode (outs[m] != NULL) while
// the chunk is resident.  Device bytes: factors read + selected outputs +
// tensor tables + two staging buffers + workspace used <= budget.
static int stream_modes(blco_tensor* t, const void* const* factors, int factor_dtype, int rank,
                        float* const* outs, size_t device_budget_bytes, hipStream_t s,
                        Work ws, const GradArgs* grad = nullptr) {
  const Layout& L = t->lay;
  unsigned modes = 0;
  for (int m = 0; m < L.N; ++m)
    if (outs[m]) modes |= 1u << m;
  if (!modes) return set_error(BLCO_EINVAL, "no output given");
  int rc;
  if (t->placement == BLCO_PLACE_DEVICE && grad) {
    double* part = grad->partials;
    if (!part) {
      if ((rc = ensure_partials(t, grad_parts(t->nnz), s))) return rc;
      part = t->d_partials;
    }
    int64_t np = 0;
    if ((rc = grad_range(t, *grad, t->d_keys, t->d_vals, 0, t->nnz, factors, factor_dtype, rank,
                         outs, grad->resid, part, &np, s, ws, true)))
      return rc;
    hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(1024), 0, s, (const double*)part, np,
                       grad->loss);
    HIPCHK(hipGetLastError());
    t->stream_peak_bytes = t->device_bytes + ws.bytes;
    for (int m = 0; m < L.N; ++m)
      t->stream_peak_bytes +=
          (size_t)L.dims[m] * rank * (sizeof(float) + factor_elem_bytes(factor_dtype));
    t->stream_chunks = 0;
    t->st.timed_chunks = 0;
    return BLCO_OK;
  }
  if (t->placement != BLCO_PLACE_DEVICE && t->placement != BLCO_PLACE_PINNED)
    return set_error(BLCO_EINVAL, "streaming needs a tensor in pinned host memory");
  StreamPlan sp;
  if ((rc = plan_stream(t, modes, grad != nullptr, rank, factor_dtype, device_budget_bytes,
                        ws.bytes, &sp)))
    return rc;
  ws.bytes = sp.ws;
  if (t->placement == BLCO_PLACE_DEVICE) {
    for (int m = 0; m < L.N; ++m) {
      if (!outs[m]) continue;
      if ((rc = launch_mttkrp(t, t->d_keys, t->d_vals, 0, t->nnz, m, factors, factor_dtype, rank,
                              1.0f, nullptr, outs[m], s, ws, true)))
        return rc;
    }
    t->stream_peak_bytes = sp.fixed + ws.bytes;
    t->stream_chunks = 0;
    t->st.timed_chunks = 0;
    return BLCO_OK;
  }
  const int64_t cap = sp.cap;
  StreamState& st = t->st;
  if (!st.copy_stream) {
    hipStream_t cs;
    HIPCHK(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    st.copy_stream = cs;
    last_copies().add();
    for (int i = 0; i < 2; ++i) {
      hipEvent_t e1, e2;
      HIPCHK(hipEventCreateWithFlags(&e1, hipEventDisableTiming));
      HIPCHK(hipEventCreateWithFlags(&e2, hipEventDisableTiming));
      st.ev_ready[i] = e1;
      st.ev_free[i] = e2;
    }
  }
  if (st.cap_nnz != cap) {
    // buffers of another size: wait until no kernel reads the old ones, then replace them
    for (int i = 0; i < 2; ++i) {
      HIPCHK(hipEventSynchronize((hipEvent_t)st.ev_free[i]));
      if (st.d_keys[i]) HIPCHK(hipFree(st.d_keys[i]));
      if (st.d_vals[i]) HIPCHK(hipFree(st.d_vals[i]));
      st.d_keys[i] = nullptr;
      st.d_vals[i] = nullptr;
    }
    st.cap_nnz = 0;
    for (int i = 0; i < 2; ++i)
      if ((rc = device_alloc((void**)&st.d_keys[i], sizeof(uint64_t) * (size_t)cap)) ||
          (rc = device_alloc((void**)&st.d_vals[i], sizeof(float) * (size_t)cap)))
        return rc;
    st.cap_nnz = cap;
  }
  if (grad && st.res_cap != cap) {
    for (int i = 0; i < 2; ++i) {
      HIPCHK(hipEventSynchronize((hipEvent_t)st.ev_free[i]));
      if (st.d_res[i]) HIPCHK(hipFree(st.d_res[i]));
      st.d_res[i] = nullptr;
    }
    st.res_cap = 0;
    for (int i = 0; i < 2; ++i)
      if ((rc = device_alloc((void**)&st.d_res[i], sizeof(float) * (size_t)cap))) return rc;
    st.res_cap = cap;
  }
  for (int m = 0; m < L.N; ++m)
    if (outs[m] && (rc = fill_zero(outs[m], (int64_t)L.dims[m] * rank, s))) return rc;
  const int64_t nchunks = (t->nnz + cap - 1) / cap;
  if (grad && (rc = ensure_partials(t, nchunks * grad_parts(cap), s))) return rc;
  int64_t poff = 0;   // partial sums written so far (CP gradient)
  // the previous call's timing events must have fired before they are reused
  for (size_t i = 0; i < st.ev_t.size(); ++i) HIPCHK(hipEventSynchronize((hipEvent_t)st.ev_t[i]));
  while ((int64_t)st.ev_t.size() < 4 * nchunks) {
    hipEvent_t e;
    HIPCHK(hipEventCreate(&e));
    st.ev_t.push_back(e);
  }
  st.timed_chunks = 0;
  HIPCHK(last_copies().follow(t->device, s, (hipStream_t)st.copy_stream));
  int64_t chunks = 0;
  hipStream_t cs = (hipStream_t)st.copy_stream;
  bool marked = false;
  // before a copy with `left` bytes of the call still to be queued
  auto lead = [&](int64_t left) {
    if (marked || left > kCopyLead) return hipSuccess;
    marked = true;
    return last_copies().mark(t->device, s, cs);
  };
  for (int64_t lo = 0; lo < t->nnz; lo += cap, ++chunks) {
    const int b = (int)(chunks & 1);
    const int64_t cnt = std::min(cap, t->nnz - lo);
    const int64_t key = sizeof(uint64_t), val = sizeof(float);
    const int64_t after = (t->nnz - lo - cnt) * (key + val);   // bytes of later chunks
    hipEvent_t* ev = reinterpret_cast<hipEvent_t*>(&st.ev_t[4 * chunks]);
    HIPCHK(hipStreamWaitEvent(cs, (hipEvent_t)st.ev_free[b], 0));
    HIPCHK(hipEventRecord(ev[0], cs));
    HIPCHK(lead(after + cnt * (key + val)));
    HIPCHK(hipMemcpyAsync(st.d_keys[b], t->h_keys + lo, (size_t)(cnt * key), hipMemcpyHostToDevice, cs));
    HIPCHK(lead(after + cnt * val));
    // (the last values in two pieces where they are more than the lead)
    const int64_t head = marked || after ? cnt : cnt - kCopyLead / val;
    HIPCHK(hipMemcpyAsync(st.d_vals[b], t->h_vals + lo, (size_t)(head * val), hipMemcpyHostToDevice, cs));
    if (head < cnt) {
      HIPCHK(lead((cnt - head) * val));
      HIPCHK(hipMemcpyAsync(st.d_vals[b] + head, t->h_vals + lo + head, (size_t)((cnt - head) * val),
                            hipMemcpyHostToDevice, cs));
    }
    HIPCHK(hipEventRecord(ev[1], cs));
    HIPCHK(hipEventRecord((hipEvent_t)st.ev_ready[b], cs));
    HIPCHK(hipStreamWaitEvent(s, (hipEvent_t)st.ev_ready[b], 0));
    HIPCHK(hipEventRecord(ev[2], s));
    if (grad) {
      int64_t np = 0;
      if ((rc = grad_range(t, *grad, st.d_keys[b], st.d_vals[b], lo, cnt, factors, factor_dtype,
                           rank, outs, st.d_res[b], t->d_partials + poff, &np, s, ws, false)))
        return rc;
      poff += np;
    } else {
      for (int m = 0; m < L.N; ++m) {
        if (!outs[m]) continue;
        if ((rc = launch_mttkrp(t, st.d_keys[b], st.d_vals[b], lo, cnt, m, factors, factor_dtype,
                                rank, 1.0f, nullptr, outs[m], s, ws, false)))
          return rc;
      }
    }
    HIPCHK(hipEventRecord(ev[3], s));
    HIPCHK(hipEventRecord((hipEvent_t)st.ev_free[b], s));
  }
  if (grad) {
    hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(1024), 0, s, (const double*)t->d_partials,
                       poff, grad->loss);
    HIPCHK(hipGetLastError());
  }
  st.timed_chunks = chunks;
  t->stream_peak_bytes = sp.fixed + ws.bytes + 2 * (size_t)cap * sp.per_nnz;
  t->stream_chunks = chunks;
  return BLCO_OK;
}

extern "C" int blco_mttkrp_stream(blco_tensor* t, int mode, const void* const* factors,
                                  int factor_dtype, int rank, float* out,
                                  size_t device_budget_bytes, void* stream) {
  clear_error();
  int rc = check_factor_args(t, mode, factors, factor_dtype, rank, out, false);
  if (rc) return rc;
  float* outs[BLCO_MAX_MODES] = {};
  outs[mode] = out;
  return stream_modes(t, factors, factor_dtype, rank, outs, device_budget_bytes,
                      (hipStream_t)stream, Work());
}

static int stream_all_impl(blco_tensor* t, const void* const* factors, int factor_dtype, int rank,
                           float* const* outs, size_t device_budget_bytes, const Work& ws,
                           hipStream_t stream) {
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  if (!outs) return set_error(BLCO_EINVAL, "outs is NULL");
  float* o[BLCO_MAX_MODES] = {};
  int first = -1;
  for (int m = 0; m < t->lay.N; ++m) {
    o[m] = outs[m];
    if (o[m] && first < 0) first = m;
  }
  if (first < 0) return set_error(BLCO_EINVAL, "no output given");
  for (int m = 0; m < t->lay.N; ++m) {
    if (!o[m]) continue;
    int rc = check_factor_args(t, m, factors, factor_dtype, rank, o[m], false);
    if (rc) return rc;
    for (int j = 0; j < t->lay.N; ++j) {
      if (j == m || !o[j]) continue;
      const float* a = o[m];
      const float* b = o[j];
      const size_t na = (size_t)t->lay.dims[m] * rank, nb = (size_t)t->lay.dims[j] * rank;
      if (a < b + nb && b < a + na) return set_error(BLCO_EINVAL, "outs[%d] overlaps outs[%d]", m, j);
    }
  }
  return stream_modes(t, factors, factor_dtype, rank, o, device_budget_bytes, stream, ws);
}

extern "C" int blco_mttkrp_stream_all(blco_tensor* t, const void* const* factors,
                                      int factor_dtype, int rank, float* const* outs,
                                      size_t device_budget_bytes, void* stream) {
  clear_error();
  return stream_all_impl(t, factors, factor_dtype, rank, outs, device_budget_bytes, Work(),
                         (hipStream_t)stream);
}

extern "C" int blco_mttkrp_stream_all_ws(blco_tensor* t, const void* const* factors,
                                         int factor_dtype, int rank, float* const* outs,
                                         size_t device_budget_bytes, void* workspace,
                                         size_t workspace_bytes, void* stream) {
  clear_error();
  Work ws;
  int rc = make_work(workspace, workspace_bytes, &ws);
  if (rc) return rc;
  return stream_all_impl(t, factors, factor_dtype, rank, outs, device_budget_bytes, ws,
                         (hipStream_t)stream);
}

// ---- workspace of blco_cp_grad_noalloc: the fp64 partial sums of the loss live in
// a static device array instead of memory the tensor allocates.  Each device holds
// its own copy; host code reaches it only through the address hipGetSymbolAddress
// returns for the current device (the array's name is not a device address there).
constexpr int64_t kScratchParts = 1 << 19;   // 4 MiB of fp64 partial sums per device
static __device__ __align__(256) double scratch[kScratchParts];
constexpr int kScratchDevs = 64;

// Device address of `scratch` on the current device, looked up once per device.
static int scratch_ptr(double** out) {
  static std::mutex mu;
  static double* addr[kScratchDevs] = {};
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kScratchDevs)
    return set_error(BLCO_EDEVICE, "device %d outside 0..%d", dev, kScratchDevs - 1);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return set_error(BLCO_EDEVICE, "no device address for the workspace on device %d", dev);
    addr[dev] = static_cast<double*>(p);
  }
  *out = addr[dev];
  return BLCO_OK;
}

// blco_cp_grad and blco_cp_grad_noalloc; with noalloc the tensor must be on the
// device and the partial sums go to the static workspace.
static int cp_grad_impl(blco_tensor* t, const void* const* factors, int factor_dtype, int rank,
                        const double* scale, double alpha, float* residual, double* loss,
                        float* const* grads, size_t device_budget_bytes, void* stream,
                        bool noalloc, const Work& work) {
  clear_error();
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  if (!loss) return set_error(BLCO_EINVAL, "loss is NULL");
  if (!grads) return set_error(BLCO_EINVAL, "grads is NULL");
  if (!factors) return set_error(BLCO_EINVAL, "factors is NULL");
  if (noalloc && t->placement != BLCO_PLACE_DEVICE)
    return set_error(BLCO_EINVAL, "the allocation-free CP gradient needs a tensor on the device");
  const int N = t->lay.N;
  float* o[BLCO_MAX_MODES] = {};
  for (int m = 0; m < N; ++m) {
    o[m] = grads[m];
    if (!o[m]) return set_error(BLCO_EINVAL, "grads[%d] is NULL", m);
    if (!factors[m]) return set_error(BLCO_EINVAL, "factors[%d] is NULL", m);
    int rc = check_factor_args(t, m, factors, factor_dtype, rank, o[m], true);
    if (rc) return rc;
  }
  for (int m = 0; m < N; ++m)
    for (int j = 0; j < N; ++j) {
      if (j == m) continue;
      const size_t na = (size_t)t->lay.dims[m] * rank, nb = (size_t)t->lay.dims[j] * rank;
      if (o[m] < o[j] + nb && o[j] < o[m] + na)
        return set_error(BLCO_EINVAL, "grads[%d] overlaps grads[%d]", m, j);
    }
  if (t->placement == BLCO_PLACE_DEVICE) {
    if (!residual && t->nnz > 0) return set_error(BLCO_EINVAL, "residual is NULL");
  } else if (t->placement == BLCO_PLACE_PINNED) {
    if (residual)
      return set_error(BLCO_EINVAL, "residual must be NULL for a tensor in pinned host memory");
  } else {
    return set_error(BLCO_EINVAL, "the CP gradient needs a tensor on the device or in pinned "
                                  "host memory");
  }
  if (noalloc && grad_parts(t->nnz) > kScratchParts)
    return set_error(BLCO_EUNSUPPORTED, "%lld non-zeros need %lld partial sums; the static workspace "
                                  "holds %lld (at most %lld non-zeros are always accepted)",
                     (long long)t->nnz, (long long)grad_parts(t->nnz), (long long)kScratchParts,
                     (long long)kScratchParts * kBlock);
  hipStream_t s = (hipStream_t)stream;
  int rc;
  double* ws = nullptr;
  if (noalloc && (rc = scratch_ptr(&ws))) return rc;
  if (t->nnz == 0) {
    for (int m = 0; m < N; ++m)
      if ((rc = fill_zero(o[m], (int64_t)t->lay.dims[m] * rank, s))) return rc;
    hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(1024), 0, s, (const double*)nullptr,
                       (int64_t)0, loss);
    HIPCHK(hipGetLastError());
    return BLCO_OK;
  }
  GradArgs g;
  g.m0 = fused_mode(t, rank, factor_dtype);
  g.scale = (float)(-alpha);
  g.scale_dev = scale;
  g.resid = residual;
  g.loss = loss;
  g.partials = ws;
  return stream_modes(t, factors, factor_dtype, rank, o, device_budget_bytes, s, work, &g);
}

extern "C" int blco_cp_grad(blco_tensor* t, const void* const* factors, int factor_dtype,
                            int rank, const double* scale, double alpha, float* residual,
                            double* loss, float* const* grads, size_t device_budget_bytes,
                            void* stream) {
  return cp_grad_impl(t, factors, factor_dtype, rank, scale, alpha, residual, loss, grads,
                      device_budget_bytes, stream, false, Work());
}

extern "C" int blco_cp_grad_ws(blco_tensor* t, const void* const* factors, int factor_dtype,
                               int rank, const double* scale, double alpha, float* residual,
                               double* loss, float* const* grads, size_t device_budget_bytes,
                               void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  Work ws;
  int rc = make_work(workspace, workspace_bytes, &ws);
  if (rc) return rc;
  return cp_grad_impl(t, factors, factor_dtype, rank, scale, alpha, residual, loss, grads,
                      device_budget_bytes, stream, false, ws);
}

extern "C" int blco_cp_grad_noalloc(blco_tensor* t, const void* const* factors, int factor_dtype,
                                    int rank, const double* scale, double alpha, float* residual,
                                    double* loss, float* const* grads, void* stream) {
  return cp_grad_impl(t, factors, factor_dtype, rank, scale, alpha, residual, loss, grads, 0,
                      stream, true, Work());
}

extern "C" int blco_sampled_loss(blco_tensor* t, const void* const* factors, int factor_dtype,
                                 int rank, float* residual, double* loss, void* stream) {
  clear_error();
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  if (!loss) return set_error(BLCO_EINVAL, "loss is NULL");
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (factor_dtype != BLCO_F32 && factor_dtype != BLCO_BF16)
    return set_error(BLCO_EINVAL, "factor dtype %d", factor_dtype);
  if (!factors) return set_error(BLCO_EINVAL, "factors is NULL");
  for (int m = 0; m < t->lay.N; ++m)
    if (!factors[m]) return set_error(BLCO_EINVAL, "factors[%d] is NULL", m);
  if (t->placement != BLCO_PLACE_DEVICE)
    return set_error(BLCO_EINVAL, "the sampled loss needs a tensor placed on the device");
  hipStream_t s = (hipStream_t)stream;
  if (t->nnz == 0) {
    // no non-zeros: the loss is 0 (the reduction over zero partials writes it),
    // and no factor row is gathered
    hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(1024), 0, s, (const double*)nullptr,
                       (int64_t)0, loss);
    HIPCHK(hipGetLastError());
    return BLCO_OK;
  }
  const int64_t blocks = loss_blocks(t->nnz);
  int rc;
  if ((rc = ensure_partials(t, blocks, s))) return rc;
  if ((rc = launch_loss(t, t->d_keys, t->d_vals, 0, t->nnz, factors, factor_dtype, rank, residual,
                        t->d_partials, s)))
    return rc;
  hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(1024), 0, s, (const double*)t->d_partials,
                     blocks, loss);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

extern "C" int blco_atomic_probe(float* out, int64_t nrows, int rank, const uint32_t* rows,
                                 int64_t n, void* stream) {
  clear_error();
  if (n < 0 || nrows < 0) return set_error(BLCO_EINVAL, "negative size");
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (n == 0) return BLCO_OK;
  if (!out || !rows) return set_error(BLCO_EINVAL, "out or rows is NULL");
  const int64_t blocks = (n * 16 + 255) / 256;
  if (blocks > 0x7FFFFFFF) return set_error(BLCO_EINVAL, "n = %lld too large", (long long)n);
  hipLaunchKernelGGL(k_atomic_probe, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                     out, nrows, rows, n, rank);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

extern "C" int blco_gather_probe(const float* table, int64_t nrows, int rank,
                                 const uint32_t* rows, int64_t n, float* sink, void* stream) {
  clear_error();
  if (n < 0 || nrows < 0) return set_error(BLCO_EINVAL, "negative size");
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (n == 0) return BLCO_OK;
  if (!table || !rows || !sink) return set_error(BLCO_EINVAL, "table, rows or sink is NULL");
  const int64_t groups = (n + kGatherRows - 1) / kGatherRows;
  const int64_t blocks = (groups * 16 + 255) / 256;
  if (blocks > 0x7FFFFFFF) return set_error(BLCO_EINVAL, "n = %lld too large", (long long)n);
  hipLaunchKernelGGL(k_gather_probe, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                     table, nrows, rows, n, rank, sink);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

// Grid of an element-wise launch over `count` arrays.
static dim3 array_grid(const int64_t* n, int count) {
  int64_t most = 1;
  for (int i = 0; i < count; ++i) most = std::max(most, n[i]);
  return dim3((unsigned)std::min<int64_t>((most + 255) / 256, 16384), (unsigned)count);
}

extern "C" int blco_scale_all(int count, float* const* x, const int64_t* n, const double* scale,
                              double alpha, void* stream) {
  clear_error();
  if (count < 0 || count > BLCO_MAX_MODES)
    return set_error(BLCO_EINVAL, "%d arrays outside 0..%d", count, BLCO_MAX_MODES);
  if (count > 0 && (!x || !n)) return set_error(BLCO_EINVAL, "x or n is NULL");
  Arrays a = {};
  int k = 0;
  for (int i = 0; i < count; ++i) {
    if (n[i] < 0) return set_error(BLCO_EINVAL, "n = %lld < 0", (long long)n[i]);
    if (n[i] == 0) continue;
    if (!x[i]) return set_error(BLCO_EINVAL, "x is NULL");
    a.dst[k] = x[i];
    a.n[k++] = n[i];
  }
  if (k == 0) return BLCO_OK;
  hipLaunchKernelGGL(k_scale, array_grid(a.n, k), dim3(256), 0, (hipStream_t)stream, a, scale,
                     alpha);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

extern "C" int blco_scale(float* x, int64_t n, const double* scale, double alpha,
                          void* stream) {
  return blco_scale_all(1, &x, &n, scale, alpha, stream);
}

extern "C" int blco_set_resolution(blco_tensor* t, int resolution) {
  clear_error();
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  if (resolution != BLCO_RES_AUTO && resolution != BLCO_RES_REGISTER &&
      resolution != BLCO_RES_HIERARCHICAL)
    return set_error(BLCO_EINVAL, "resolution %d", resolution);
  t->resolution = resolution;
  return BLCO_OK;
}

extern "C" int blco_resolution(const blco_tensor* t, int mode, int rank, int* chosen) {
  clear_error();
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  if (mode < 0 || mode >= t->lay.N)
    return set_error(BLCO_EINVAL, "mode %d outside 0..%d", mode, t->lay.N - 1);
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (!chosen) return set_error(BLCO_EINVAL, "chosen is NULL");
  int sw = 0;
  const int res = resolve(t, mode, rank, &sw);
  if (res < 0) return res;
  *chosen = res;
  return BLCO_OK;
}

extern "C" int blco_frequent_rows(const blco_tensor* t, int mode, int rank, int* rows) {
  clear_error();
  if (!t || !rows) return set_error(BLCO_EINVAL, "tensor or rows is NULL");
  if (mode < 0 || mode >= t->lay.N)
    return set_error(BLCO_EINVAL, "mode %d outside 0..%d", mode, t->lay.N - 1);
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  const WinPlan w = plan_win(t, mode, rank, rank, rank, rank % 2 == 0, BLCO_F32, false, false,
                             std::max<int64_t>(t->nnz, 1), 0, false, false, false);
  *rows = w.stash;
  return BLCO_OK;
}

// Lanes per non-zero and ranks per lane of the window kernel (select_win_t, select_res_t).
static void win_shape(int gather, int fdt, bool big, bool resid, int wpt, int* lanes, int* rpl) {
  *lanes = gather <= 64 ? 16 : 64;
  if (gather > 64) *rpl = 2;
  else if (gather <= 32) *rpl = gather <= 16 ? 1 : 2;
  else *rpl = fdt == BLCO_F32 && !big && !resid && gather <= 48 && wpt != 1 ? 3 : 4;
}

extern "C" int blco_plan(const blco_tensor* t, int mode, int rank, int factor_dtype, int use,
                         int64_t nnz, size_t workspace_bytes, blco_plan_t* plan) {
  clear_error();
  if (!t || !plan) return set_error(BLCO_EINVAL, "tensor or plan is NULL");
  if (mode < 0 || mode >= t->lay.N)
    return set_error(BLCO_EINVAL, "mode %d outside 0..%d", mode, t->lay.N - 1);
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (factor_dtype != BLCO_F32 && factor_dtype != BLCO_BF16)
    return set_error(BLCO_EINVAL, "factor dtype %d", factor_dtype);
  if (use < BLCO_USE_MTTKRP || use > BLCO_USE_ALS) return set_error(BLCO_EINVAL, "use %d", use);
  if (nnz < 0) return set_error(BLCO_EINVAL, "nnz %lld < 0", (long long)nnz);
  const bool resid = use == BLCO_USE_RESIDUAL;
  if (resid && !fused_mode_ok(t, mode, rank, factor_dtype))
    return set_error(BLCO_EUNSUPPORTED, "fused residual walk on mode %d", mode);
  const int64_t n = nnz ? nnz : std::max<int64_t>(t->nnz, 1);
  LaunchPlan L;
  int rc = plan_launch(t, mode, rank, factor_dtype, resid, n, workspace_bytes, use == BLCO_USE_ALS,
                       &L);
  if (rc) return rc;
  memset(plan, 0, sizeof(*plan));
  plan->resolution = L.res;
  plan->factor_stride = L.stride;
  plan->out_stride = L.cp.out;
  plan->grouped = L.cp.group;
  plan->out_copies = L.cp.outs;
  plan->workspace_bytes = L.cp.bytes;
  for (int h = 0; h < 2; ++h) plan->flushes[h] = flushes(t, mode, h);
  plan->vector_gathers = factor_dtype == BLCO_BF16 && L.stride % 2 == 0;
  if (L.res != BLCO_RES_REGISTER) {
    plan->wide = L.big;
    plan->window = kShortB;
    plan->lanes = kShortLPN;
    plan->ranks_per_lane = short_rpl(L.sw);
    return BLCO_OK;
  }
  plan->wide = L.big_win;
  plan->wpt = L.w.wpt;
  plan->window = L.w.wpt < 0 ? kWin / -L.w.wpt : kWin * L.w.wpt;
  plan->stash_rows = L.w.stash;
  plan->copies = L.w.copies;
  plan->workgroups = L.grid;
  win_shape(L.stride, factor_dtype, L.big_win, resid, L.w.wpt, &plan->lanes, &plan->ranks_per_lane);
  return BLCO_OK;
}

extern "C" int blco_workspace(const blco_tensor* t, int mode, int rank, int factor_dtype,
                              size_t* bytes) {
  clear_error();
  if (!t || !bytes) return set_error(BLCO_EINVAL, "tensor or bytes is NULL");
  if (mode < -1 || mode >= t->lay.N)
    return set_error(BLCO_EINVAL, "mode %d outside -1..%d", mode, t->lay.N - 1);
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (factor_dtype != BLCO_F32 && factor_dtype != BLCO_BF16)
    return set_error(BLCO_EINVAL, "factor dtype %d", factor_dtype);
  size_t most = 0;
  for (int m = 0; m < t->lay.N; ++m) {
    if (mode >= 0 && m != mode) continue;
    most = std::max(most, mode_workspace(t, m, rank, factor_dtype, false, t->nnz));
    if (mode < 0 && fused_mode_ok(t, m, rank, factor_dtype))
      most = std::max(most, mode_workspace(t, m, rank, factor_dtype, true, t->nnz));
  }
  *bytes = (most + 255) / 256 * 256;
  return BLCO_OK;
}

extern "C" int blco_stream_plan(const blco_tensor* t, unsigned modes, int gradient, int rank,
                                int factor_dtype, size_t device_budget_bytes,
                                size_t workspace_bytes, size_t* used, int64_t* chunk_nnz) {
  clear_error();
  if (!t || !used || !chunk_nnz) return set_error(BLCO_EINVAL, "tensor, used or chunk_nnz is NULL");
  if (rank < 1) return set_error(BLCO_EINVAL, "rank %d < 1", rank);
  if (factor_dtype != BLCO_F32 && factor_dtype != BLCO_BF16)
    return set_error(BLCO_EINVAL, "factor dtype %d", factor_dtype);
  const unsigned all = (1u << t->lay.N) - 1;
  if (gradient) modes = all;
  if (!modes || (modes & ~all)) return set_error(BLCO_EINVAL, "modes 0x%x", modes);
  StreamPlan p;
  int rc = plan_stream(t, modes, gradient != 0, rank, factor_dtype, device_budget_bytes,
                       workspace_bytes, &p);
  if (rc) return rc;
  *used = p.ws;
  *chunk_nnz = p.cap;
  return BLCO_OK;
}

extern "C" int blco_cast_bf16_all(int count, const float* const* src, uint16_t* const* dst,
                                  const int64_t* n, void* stream) {
  clear_error();
  if (count < 0 || count > BLCO_MAX_MODES)
    return set_error(BLCO_EINVAL, "%d arrays outside 0..%d", count, BLCO_MAX_MODES);
  if (count > 0 && (!src || !dst || !n)) return set_error(BLCO_EINVAL, "src, dst or n is NULL");
  Arrays a = {};
  int k = 0;
  for (int i = 0; i < count; ++i) {
    if (n[i] < 0) return set_error(BLCO_EINVAL, "n < 0");
    if (n[i] == 0) continue;
    if (!src[i] || !dst[i]) return set_error(BLCO_EINVAL, "src or dst is NULL");
    a.src[k] = src[i];
    a.dst[k] = dst[i];
    a.n[k++] = n[i];
  }
  if (k == 0) return BLCO_OK;
  hipLaunchKernelGGL(k_cast_bf16, array_grid(a.n, k), dim3(256), 0, (hipStream_t)stream, a);
  HIPCHK(hipGetLastError());
  return BLCO_OK;
}

extern "C" int blco_cast_bf16(const float* src, uint16_t* dst, int64_t n, void* stream) {
  return blco_cast_bf16_all(1, &src, &dst, &n, stream);
}

extern "C" int blco_info(const blco_tensor* t, blco_info_t* info) {
  clear_error();
  if (!t || !info) return set_error(BLCO_EINVAL, "tensor or info is NULL");
  memset(info, 0, sizeof(*info));
  const Layout& L = t->lay;
  info->nmodes = L.N;
  info->nnz = t->nnz;
  info->total_bits = L.T;
  info->key_bits = L.K;
  info->block_bits = L.S;
  for (int m = 0; m < L.N; ++m) {
    info->bits[m] = L.b[m];
    info->kept[m] = L.w[m];
    info->shift[m] = L.s[m];
    info->high[m] = L.h[m];
    info->dims[m] = L.dims[m];
    info->hot_rows[m] = t->nhot[m];
  }
  for (int k = 0; k < 5; ++k) info->build_stage_ms[k] = t->build_stage_ms[k];
  info->nblocks = (int64_t)t->block_id.size();
  info->nruns = (int64_t)t->run_start.size() - 1;
  info->placement = t->placement;
  info->device_bytes = t->device_bytes;
  info->host_bytes = (t->h_keys ? (size_t)t->nnz * (sizeof(uint64_t) + sizeof(float)) : 0);
  info->stream_peak_bytes = t->stream_peak_bytes;
  info->stream_chunks = t->stream_chunks;
  info->stream_chunk_nnz = t->st.cap_nnz;
  const StreamState& st = t->st;
  if (st.timed_chunks > 0) {
    hipEvent_t* ev = reinterpret_cast<hipEvent_t*>(const_cast<void**>(st.ev_t.data()));
    const int64_t n = st.timed_chunks;
    HIPCHK(hipEventSynchronize(ev[4 * (n - 1) + 3]));
    double copy = 0.0, kern = 0.0;
    for (int64_t c = 0; c < n; ++c) {
      float a = 0.f, b = 0.f;
      HIPCHK(hipEventElapsedTime(&a, ev[4 * c], ev[4 * c + 1]));
      HIPCHK(hipEventElapsedTime(&b, ev[4 * c + 2], ev[4 * c + 3]));
      copy += a;
      kern += b;
    }
    float tot = 0.f;
    HIPCHK(hipEventElapsedTime(&tot, ev[0], ev[4 * (n - 1) + 3]));
    info->stream_copy_ms = copy;
    info->stream_kernel_ms = kern;
    info->stream_total_ms = tot;
  }
  return BLCO_OK;
}

extern "C" int blco_export(const blco_tensor* t, uint64_t* keys, float* values,
                           uint64_t* block_ids, int64_t* block_starts) {
  clear_error();
  if (!t) return set_error(BLCO_EINVAL, "tensor is NULL");
  const size_t n = (size_t)t->nnz;
  if (keys && n) {
    if (t->h_keys) memcpy(keys, t->h_keys, n * sizeof(uint64_t));
    else HIPCHK(hipMemcpy(keys, t->d_keys, n * sizeof(uint64_t), hipMemcpyDeviceToHost));
  }
  if (values && n) {
    if (t->h_vals) memcpy(values, t->h_vals, n * sizeof(float));
    else HIPCHK(hipMemcpy(values, t->d_vals, n * sizeof(float), hipMemcpyDeviceToHost));
  }
  if (block_ids && !t->block_id.empty())
    memcpy(block_ids, t->block_id.data(), t->block_id.size() * sizeof(uint64_t));
  if (block_starts) memcpy(block_starts, t->block_start.data(), t->block_start.size() * sizeof(int64_t));
  return BLCO_OK;
}

extern "C" void blco_free(blco_tensor* t) {
  if (!t) return;
  if (t->placement != BLCO_PLACE_HOST) release_device(t);
  free_host_arrays(t);
  delete t;
}
