// BLCO construction on the GPU (Sections 4.1-4.2), from coordinates and values
// already in device memory.
//
// Steps, each a kernel or a device-wide primitive on the caller's stream:
//   1. ALTO linearization of every coordinate (Section 4.1): bit j of mode n
//      goes to position pos[n][j] of a 64- or 128-bit index (per-byte deposit
//      tables); out-of-range coordinates are flagged;
//   2. a stable radix sort along the encoding line (blco_sort.hip), least
//      significant digits first, the values moved along: one sort over the low
//      64 bits, then, for indices over 64 bits, one over the high bits.  The first
//      also moves the high bits (32-bit words for indices of at most 96 bits), the
//      second the low bits, so no array follows a permutation by gathers;
//   3. re-encoding in sorted order (Figure 6b) from the sorted index: every
//      index bit below K moves to its mode's field (a byte table), the block
//      key is the index above bit K;
//   4. runs of equal block key (flags and a stream compaction), copied to the host, where
//      the block list, per-run high bits and tile table are finished by the
//      same code as the host builder;
//   5. the frequent rows of each mode (sampled rows sorted and run-length
//      counted, then a stable descending radix sort of the counts).
// The result equals blco_build's bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "blco_internal.h"

using namespace blco;

#define HIPCHK(expr)                                                                         \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return set_error(BLCO_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));         \
  } while (0)

namespace {

struct LinParams {
  const uint32_t* coords[BLCO_MAX_MODES];
  uint64_t dims[BLCO_MAX_MODES];
  uint8_t pos[BLCO_MAX_MODES][32];
  int b[BLCO_MAX_MODES];
  int w[BLCO_MAX_MODES];
  int s[BLCO_MAX_MODES];
  int N;
  int K;
  int T;
};

// First bad non-zero, and the AND and OR of the low and high index words: what the host
// reads once the non-zeros are linearized.
struct LinResult {
  unsigned long long bad, lo_and, lo_or, hi_and, hi_or;
};

constexpr int kEncBytes = 8;   // K <= 64

// Byte tables of the bit map, the cleared LinResult and the cleared flush counts.  dep[((m * 4 + k) * 256 + v) * 2 +
// {0, 1}]: the (lo, hi) index bits of byte k of a mode-m coordinate holding v;
// enc[k * 256 + v]: key bits of byte k of an index holding v.
__global__ __launch_bounds__(256) void k_tables(LinParams p, uint64_t* __restrict__ dep,
                                                uint64_t* __restrict__ enc,
                                                LinResult* __restrict__ res,
                                                uint32_t* __restrict__ counts) {
  const int v = threadIdx.x;
  if (blockIdx.x == 0 && v < 2 * BLCO_MAX_MODES) counts[v] = 0;
  if (blockIdx.x == 0 && v == 0) *res = LinResult{~0ull, ~0ull, 0ull, ~0ull, 0ull};
  const int nd = p.N * 4;
  if ((int)blockIdx.x < nd) {
    const int m = blockIdx.x / 4, k = blockIdx.x % 4;
    uint64_t xl = 0, xh = 0;
    for (int j = 0; j < 8; ++j) {
      const int bj = 8 * k + j;
      if (!((v >> j) & 1) || bj >= p.b[m]) continue;
      const int q = p.pos[m][bj];
      if (q < 64)
        xl |= 1ull << q;
      else
        xh |= 1ull << (q - 64);
    }
    dep[((size_t)blockIdx.x * 256 + v) * 2] = xl;
    dep[((size_t)blockIdx.x * 256 + v) * 2 + 1] = xh;
    return;
  }
  const int k = blockIdx.x - nd;
  uint64_t x = 0;
  for (int m = 0; m < p.N; ++m)
    for (int j = 0; j < p.b[m]; ++j) {
      const int q = (int)p.pos[m][j] - 8 * k;   // bit j of mode m is bit q of this byte
      if (q >= 0 && q < 8 && 8 * k + q < p.K && ((v >> q) & 1)) x |= 1ull << (p.s[m] + j);
    }
  enc[(size_t)k * 256 + v] = x;
}

// ALTO index of every non-zero (lo: bits 0..63; hi: bits 64..127, or hi32: bits
// 64..95 of an index of at most 96 bits; or neither); res: the smallest non-zero number
// with a coordinate out of range, and the AND and OR of the index words (the sorts skip
// digits they show to be constant).  Without a high part the lo halves of the deposit table
// are staged in LDS (N * 8 KiB of dynamic LDS), once per workgroup of a grid that
// strides over the non-zeros.
__global__ __launch_bounds__(256) void k_linearize(LinParams p, int64_t n,
                                                   const uint64_t* __restrict__ dep,
                                                   uint64_t* __restrict__ lo,
                                                   uint64_t* __restrict__ hi,
                                                   uint32_t* __restrict__ hi32,
                                                   LinResult* __restrict__ res) {
  extern __shared__ uint64_t s_dep[];   // [(m * 4 + k) * 256 + v], lo halves (no high part)
  __shared__ unsigned long long s_red[4][4];
  const bool wide = hi || hi32;
  if (!wide) {
    for (int j = threadIdx.x; j < p.N * 4 * 256; j += 256) s_dep[j] = dep[2 * j];
    __syncthreads();
  }
  unsigned long long red[4] = {~0ull, 0ull, ~0ull, 0ull};
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    uint64_t l = 0, h = 0;
    for (int m = 0; m < p.N; ++m) {
      uint32_t c = p.coords[m][i];
      if ((uint64_t)c >= p.dims[m]) {
        atomicMin(&res->bad, (unsigned long long)i);
        c = 0;
      }
      if (!wide) {
        const uint64_t* d = s_dep + (size_t)m * 4 * 256;
#pragma unroll
        for (int k = 0; k < 4; ++k) l |= d[k * 256 + ((c >> (8 * k)) & 255u)];
      } else {
        const uint64_t* d = dep + (size_t)m * 4 * 256 * 2;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t v = (c >> (8 * k)) & 255u;
          l |= d[(k * 256 + v) * 2];
          h |= d[(k * 256 + v) * 2 + 1];
        }
      }
    }
    lo[i] = l;
    if (hi) hi[i] = h;
    if (hi32) hi32[i] = (uint32_t)h;
    red[0] &= l;
    red[1] |= l;
    red[2] &= h;
    red[3] |= h;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned long long o = __shfl_xor(red[q], off, 64);
      red[q] = q & 1 ? (red[q] | o) : (red[q] & o);
    }
  }
  if ((threadIdx.x & 63) == 0)
    for (int q = 0; q < 4; ++q) s_red[threadIdx.x >> 6][q] = red[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    const int q = threadIdx.x;
    unsigned long long x = s_red[0][q];
    for (int w = 1; w < 4; ++w) x = q & 1 ? (x | s_red[w][q]) : (x & s_red[w][q]);
    unsigned long long* dst = q == 0 ? &res->lo_and : q == 1 ? &res->lo_or
                                                  : q == 2 ? &res->hi_and : &res->hi_or;
    if (q & 1)
      atomicOr(dst, x);
    else
      atomicAnd(dst, x);
  }
}

// Run that holds the first non-zero of each 64-non-zero tile: the last run starting at or
// before it.
__global__ __launch_bounds__(256) void k_tile_run(const int64_t* __restrict__ run_start,
                                                  int64_t nruns, int64_t ntiles,
                                                  int32_t* __restrict__ tile_run) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= ntiles) return;
  const int64_t e = i * kTile;
  int64_t a = 0, b = nruns;   // run_start[a] <= e < run_start[b]
  while (b - a > 1) {
    const int64_t m = (a + b) / 2;
    if (run_start[m] <= e)
      a = m;
    else
      b = m;
  }
  tile_run[i] = (int32_t)a;
}

// Keys and block keys in sorted order, from the sorted index (slo: bits 0..63;
// shi: bits 64..127, or shi32: bits 64..95; or neither): the key gathers every index
// bit below K into its mode's field through a byte table (enc[k][v]: key bits of
// byte k holding v); the block key is the index above bit K.  The values are
// already in place: the sorts moved them.
__global__ __launch_bounds__(256) void k_encode(int64_t n, int K, const uint64_t* __restrict__ enc,
                                                const uint64_t* __restrict__ slo,
                                                const uint64_t* __restrict__ shi,
                                                const uint32_t* __restrict__ shi32,
                                                uint64_t* __restrict__ keys,
                                                uint64_t* __restrict__ bkey) {
  __shared__ uint64_t s_enc[kEncBytes * 256];
  for (int i = threadIdx.x; i < kEncBytes * 256; i += 256) s_enc[i] = enc[i];
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint64_t l = slo[i], h = shi ? shi[i] : shi32 ? (uint64_t)shi32[i] : 0;
  const uint64_t low = K >= 64 ? l : (l & ((1ULL << K) - 1));
  uint64_t key = 0;
#pragma unroll
  for (int k = 0; k < kEncBytes; ++k) key |= s_enc[k * 256 + ((low >> (8 * k)) & 255)];
  keys[i] = key;
  if (!bkey) return;
  uint64_t B;
  if (K >= 64)
    B = h >> (K - 64);
  else if (K == 0)
    B = l;
  else
    B = (l >> K) | (h << (64 - K));
  bkey[i] = B;
}

__global__ __launch_bounds__(256) void k_run_flags(const uint64_t* __restrict__ bkey, int64_t n,
                                                   uint8_t* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) flag[i] = (i == 0 || bkey[i] != bkey[i - 1]) ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_gather_keys(const uint64_t* __restrict__ bkey,
                                                     const int64_t* __restrict__ starts,
                                                     int64_t nruns, uint64_t* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < nruns) out[r] = bkey[starts[r]];
}

__global__ __launch_bounds__(256) void k_sample(const uint32_t* __restrict__ c, int64_t samples,
                                                int64_t step, uint32_t* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s < samples) out[s] = c[s * step];
}

__global__ __launch_bounds__(256) void k_row_flags(const uint32_t* __restrict__ sorted, int64_t n,
                                                   uint8_t* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) flag[i] = (i == 0 || sorted[i] != sorted[i - 1]) ? 1 : 0;
}

// Run-length encoding from the run starts of a sorted array: the value and the
// length of every run.
__global__ __launch_bounds__(256) void k_runs(const uint32_t* __restrict__ sorted,
                                              const int64_t* __restrict__ starts, int64_t nruns,
                                              int64_t n, uint32_t* __restrict__ uniq,
                                              uint32_t* __restrict__ cnt) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= nruns) return;
  const int64_t a = starts[r], e = r + 1 < nruns ? starts[r + 1] : n;
  uniq[r] = sorted[a];
  cnt[r] = (uint32_t)(e - a);
}

unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>((n + 255) / 256, 1); }

constexpr unsigned kStrideGrid = 2048;   // workgroups of grid-stride kernels (8 per CU)

// Events at the stage boundaries of one build on its stream (released on return).
struct StageEvents {
  static constexpr int kN = 6;
  hipEvent_t ev[kN] = {};
  bool ok = true;
  StageEvents() {
    for (auto& e : ev)
      if (hipEventCreate(&e) != hipSuccess) ok = false;
  }
  ~StageEvents() {
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
  }
  void mark(int k, hipStream_t s) {
    if (ok) (void)hipEventRecord(ev[k], s);
  }
  // elapsed ms between consecutive marks, once the last has completed
  void read(double* ms) {
    if (!ok || hipEventSynchronize(ev[kN - 1]) != hipSuccess) return;
    for (int k = 0; k + 1 < kN; ++k) {
      float x = 0.f;
      if (hipEventElapsedTime(&x, ev[k], ev[k + 1]) == hipSuccess) ms[k] = x;
    }
  }
};

// Device memory of one build: taken in turn from the block the caller lends, and
// allocated where that has no room (released on every return path).  reuse() starts over
// in the block: what was taken since keep() is dead for work queued from then on.
struct Pool {
  std::vector<void*> ptrs;
  char* block = nullptr;
  size_t bytes = 0, at = 0, kept = 0;
  ~Pool() {
    for (void* p : ptrs) (void)hipFree(p);
  }
  void keep() { kept = at; }
  void reuse() { at = kept; }
  template <typename T>
  int get(T** out, size_t count) {
    const size_t need = std::max<size_t>(count, 1) * sizeof(T);
    if (at <= bytes && need <= bytes - at) {
      *out = reinterpret_cast<T*>(block + at);
      at += (need + 255) / 256 * 256;
      return BLCO_OK;
    }
    void* p = nullptr;
    int rc = device_alloc(&p, need);
    if (rc) return rc;
    ptrs.push_back(p);
    *out = static_cast<T*>(p);
    return BLCO_OK;
  }
};

// The tensor's own arrays: from the caller's storage while it has room, else allocated.
struct Home {
  blco_tensor* t;
  size_t at = 0;
  template <typename T>
  int get(T** dst, size_t count, size_t* acc) {
    const size_t need = sizeof(T) * std::max<size_t>(count, 1);
    if (t->storage && at <= t->storage_bytes && need <= t->storage_bytes - at) {
      *dst = reinterpret_cast<T*>(t->storage + at);
      at += (need + 255) / 256 * 256;
    } else {
      int rc = device_alloc((void**)dst, need);
      if (rc) return rc;
    }
    *acc += need;
    return BLCO_OK;
  }
};

template <typename T>
int upload_to(Home& home, T** dst, const T* src, size_t count, hipStream_t s, size_t* acc) {
  int rc = home.get(dst, count, acc);
  if (rc) return rc;
  if (count) HIPCHK(hipMemcpyAsync(*dst, src, sizeof(T) * count, hipMemcpyHostToDevice, s));
  return BLCO_OK;
}

void release_tensor_arrays(blco_tensor* t) {
  for (void* p : {(void*)t->d_keys, (void*)t->d_vals, (void*)t->d_run_start,
                  (void*)t->d_run_base, (void*)t->d_tile_run, (void*)t->d_hot, (void*)t->d_tab,
                  (void*)t->d_group})
    if (t->owned(p)) (void)hipFree(p);
  t->d_keys = nullptr;
  t->d_vals = nullptr;
  t->d_run_start = nullptr;
  t->d_run_base = nullptr;
  t->d_tile_run = nullptr;
  t->d_hot = nullptr;
  t->d_tab = nullptr;
  t->d_group = nullptr;
  free_host_arrays(t);
}

void pinned_release(void* p) { (void)hipHostFree(p); }

// Frequent rows of every mode, as find_hot_rows: the rows of every step-th
// non-zero are sorted and run-length counted (no atomics: hot rows would
// serialise), then the kHotMax + 1 most frequent (ties by row, as the stable
// sort keeps ascending rows) are kept and those reaching the threshold marked.
int gpu_hot_rows(const LinParams& lp, int64_t nnz, int64_t min_count, Pool& pool, hipStream_t s,
                 blco_tensor* t) {
  const int N = lp.N;
  t->hot.assign((size_t)N * kHotMax, 0xFFFFFFFFu);
  t->hot_cnt.assign((size_t)N * (kHotMax + 1), 0);
  for (int n = 0; n < N; ++n) t->nhot[n] = 0;
  if (nnz <= 0 || min_count < 0) return BLCO_OK;
  const int64_t step = std::max<int64_t>(1, nnz / ((int64_t)1 << 22));
  const int64_t samples = (nnz + step - 1) / step;
  const uint64_t need = (uint64_t)std::max<int64_t>(1, (min_count + step - 1) / step);
  int rc;
  uint32_t *smp, *sorted, *uniq, *cnt, *cnt2, *row2, *tk, *tv;
  uint8_t* flag;
  int64_t* starts;
  unsigned int* ws;
  if ((rc = pool.get(&smp, samples)) || (rc = pool.get(&sorted, samples)) ||
      (rc = pool.get(&uniq, samples)) || (rc = pool.get(&cnt, samples)) ||
      (rc = pool.get(&cnt2, samples)) || (rc = pool.get(&row2, samples)) ||
      (rc = pool.get(&tk, samples)) || (rc = pool.get(&tv, samples)) ||
      (rc = pool.get(&flag, samples)) || (rc = pool.get(&starts, samples)) ||
      (rc = pool.get(&ws, std::max(sort_workspace_words(samples), select_workspace_words(samples)))))
    return rc;
  for (int n = 0; n < N; ++n) {
    const uint64_t I = lp.dims[n];
    if (I > ((uint64_t)1 << 26)) continue;
    const int bits = std::max(1, lp.b[n]);
    hipLaunchKernelGGL(k_sample, dim3(grid_of(samples)), dim3(256), 0, s, lp.coords[n], samples,
                       step, smp);
    HIPCHK(hipGetLastError());
    // the sampled rows in order, their runs (row, count), the runs by count,
    // most frequent first (equal counts keep ascending rows: the sort is stable)
    if ((rc = radix_sort_u32(smp, nullptr, sorted, nullptr, tk, nullptr, samples, bits, false, ws,
                             s)))
      return rc;
    hipLaunchKernelGGL(k_row_flags, dim3(grid_of(samples)), dim3(256), 0, s, sorted, samples,
                       flag);
    HIPCHK(hipGetLastError());
    int64_t nu = 0;
    if ((rc = select_flagged(flag, samples, starts, &nu, ws, s))) return rc;
    hipLaunchKernelGGL(k_runs, dim3(grid_of(nu)), dim3(256), 0, s, sorted, starts, nu, samples,
                       uniq, cnt);
    HIPCHK(hipGetLastError());
    if ((rc = radix_sort_u32(cnt, uniq, cnt2, row2, tk, tv, nu, 32, true, ws, s))) return rc;
    const size_t k = std::min<size_t>((size_t)nu, kHotMax + 1);
    std::vector<uint32_t> hc(k), hr(k);
    if (k) {
      HIPCHK(hipMemcpyAsync(hc.data(), cnt2, k * 4, hipMemcpyDeviceToHost, s));
      HIPCHK(hipMemcpyAsync(hr.data(), row2, k * 4, hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
    }
    int nh = 0;
    for (size_t j = 0; j < k; ++j) {
      t->hot_cnt[(size_t)n * (kHotMax + 1) + j] = (uint64_t)hc[j] * (uint64_t)step;
      if (j < (size_t)kHotMax && hc[j] >= need) t->hot[(size_t)n * kHotMax + nh++] = hr[j];
    }
    t->nhot[n] = nh;
  }
  return BLCO_OK;
}

int build_on_device(int nmodes, const uint64_t* dims, int64_t nnz, const uint32_t* const* coords,
                    const float* values, int key_bits, int64_t cap, int64_t hot_min,
                    hipStream_t s, void* ws_block, size_t ws_bytes, blco_tensor* t) {
  int rc;
  const Layout& L = t->lay;
  t->nnz = nnz;
  t->max_block_nnz = cap;
  LinParams lp;
  memset(&lp, 0, sizeof(lp));
  lp.N = L.N;
  lp.K = L.K;
  lp.T = L.T;
  for (int m = 0; m < L.N; ++m) {
    lp.coords[m] = coords[m];
    lp.dims[m] = L.dims[m];
    lp.b[m] = L.b[m];
    lp.w[m] = L.w[m];
    lp.s[m] = L.s[m];
    for (int j = 0; j < L.b[m]; ++j) lp.pos[m][j] = (uint8_t)L.pos[m][j];
  }
  Pool pool;
  pool.block = static_cast<char*>(ws_block);
  pool.bytes = ws_bytes;
  Home home{t};
  StageEvents stage;
  stage.mark(0, s);
  const bool wide = L.T > 64;
  // an index over 64 bits is sorted in two parts: the sort over the low 64 bits moves
  // the values and the high bits (32-bit words up to 96 bits, else 64-bit), the sort
  // over the high bits moves the values and the low bits; one of at most 64 bits
  // carries the values through its one sort
  const bool mid = wide && L.T <= 96;
  const bool blocked = L.S > 0;   // without block bits every block key is 0: none are written
  uint64_t *lo, *lo2, *hi = nullptr, *his = nullptr, *hif = nullptr, *bkey = nullptr;
  uint32_t *h32 = nullptr, *h32s = nullptr, *h32f = nullptr, *vs = nullptr, *tv2 = nullptr;
  LinResult* res;
  uint64_t *d_dep, *d_enc;
  uint32_t* counts;
  if ((rc = pool.get(&counts, 2 * BLCO_MAX_MODES))) return rc;
  pool.keep();
  if ((rc = pool.get(&res, 1)) || (rc = pool.get(&d_dep, (size_t)L.N * 4 * 256 * 2)) ||
      (rc = pool.get(&d_enc, (size_t)kEncBytes * 256)) || (rc = pool.get(&lo, nnz)) ||
      (rc = pool.get(&lo2, nnz)) || (blocked && (rc = pool.get(&bkey, nnz))))
    return rc;
  if (wide && ((rc = pool.get(&vs, nnz)) || (rc = pool.get(&tv2, nnz))))
    return rc;
  if (mid && ((rc = pool.get(&h32, nnz)) || (rc = pool.get(&h32s, nnz)) ||
              (rc = pool.get(&h32f, nnz))))
    return rc;
  if (wide && !mid && ((rc = pool.get(&hi, nnz)) || (rc = pool.get(&his, nnz)) ||
                       (rc = pool.get(&hif, nnz))))
    return rc;
  // 1. linearize, through per-byte deposit tables
  hipLaunchKernelGGL(k_tables, dim3(L.N * 4 + kEncBytes), dim3(256), 0, s, lp, d_dep, d_enc, res,
                     counts);
  HIPCHK(hipGetLastError());
  if (nnz > 0)
    hipLaunchKernelGGL(k_linearize, dim3(std::min<unsigned>(grid_of(nnz), kStrideGrid)), dim3(256),
                       wide ? 0 : (size_t)L.N * 4 * 256 * sizeof(uint64_t), s, lp, nnz, d_dep, lo,
                       mid ? nullptr : hi, h32, res);
  HIPCHK(hipGetLastError());
  LinResult lin;
  HIPCHK(hipMemcpyAsync(&lin, res, sizeof(lin), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  const unsigned long long first_bad = lin.bad;
  const uint64_t lo_bits[2] = {lin.lo_and, lin.lo_or}, hi_bits[2] = {lin.hi_and, lin.hi_or};
  if (first_bad != ~0ULL) {
    const int64_t i = (int64_t)first_bad;
    for (int m = 0; m < L.N; ++m) {
      uint32_t c = 0;
      HIPCHK(hipMemcpy(&c, coords[m] + i, 4, hipMemcpyDeviceToHost));
      if ((uint64_t)c >= L.dims[m])
        return set_error(BLCO_ERANGE, "coordinate %u of mode %d at non-zero %lld is >= %llu", c, m,
                         (long long)i, (unsigned long long)L.dims[m]);
    }
    return set_error(BLCO_ERANGE, "coordinate out of range at non-zero %lld", (long long)i);
  }
  // 2. stable sort along the encoding line
  stage.mark(1, s);
  size_t acc = 0;
  if ((rc = home.get(&t->d_keys, (size_t)nnz, &acc)) ||
      (rc = home.get(&t->d_vals, (size_t)nnz, &acc)))
    return rc;
  if (nnz > 0) {
    const int nb0 = std::max(1, std::min(L.T, 64));
    uint64_t* tk;
    uint32_t* tv;
    unsigned int* ws;
    if ((rc = pool.get(&tk, nnz)) || (rc = pool.get(&tv, nnz)) ||
        (rc = pool.get(&ws, sort_workspace_words(nnz))))
      return rc;
    const uint32_t* v_in = reinterpret_cast<const uint32_t*>(values);
    uint32_t* v_out = reinterpret_cast<uint32_t*>(t->d_vals);
    if (!wide) {
      // at most 64 index bits: the values travel with the keys into the tensor
      if ((rc = radix_sort_u64(lo, v_in, lo2, v_out, tk, tv, nnz, nb0, ws, s, lo_bits))) return rc;
    } else {
      // the low 64 bits, moving the values and the high bits; then the high bits,
      // moving the values (into the tensor) and the low bits
      uint64_t* tk2;
      if (!mid && (rc = pool.get(&tk2, nnz))) return rc;
      SortVals v1 = {};
      v1.in32[0] = v_in;
      v1.out32[0] = vs;
      v1.tmp32[0] = tv;
      if (mid) {
        v1.in32[1] = h32;
        v1.out32[1] = h32s;
        v1.tmp32[1] = tv2;
      } else {
        v1.in64 = hi;
        v1.out64 = his;
        v1.tmp64 = tk2;
      }
      if ((rc = radix_sort_u64_vals(lo, lo2, tk, v1, nnz, nb0, ws, s, lo_bits))) return rc;
      SortVals v2 = {};
      v2.in32[0] = vs;
      v2.out32[0] = v_out;
      v2.tmp32[0] = tv2;
      v2.in64 = lo2;
      v2.out64 = lo;   // the unsorted low bits are no longer needed
      v2.tmp64 = tk;
      if (mid) {
        if ((rc = radix_sort_u32_vals(h32s, h32f, tv, v2, nnz, L.T - 64, ws, s, hi_bits)))
          return rc;
      } else {
        if ((rc = radix_sort_u64_vals(his, hif, tk2, v2, nnz, L.T - 64, ws, s, hi_bits)))
          return rc;
      }
      std::swap(lo, lo2);   // lo2: the low bits in the final order
    }
  }
  // 3. re-encode in sorted order; keys and values go straight into the tensor
  stage.mark(2, s);
  if (nnz > 0) {
    hipLaunchKernelGGL(k_encode, dim3(grid_of(nnz)), dim3(256), 0, s, nnz, L.K, d_enc, lo2,
                       wide && !mid ? hif : nullptr, mid ? h32f : nullptr, t->d_keys,
                       blocked ? bkey : nullptr);
    HIPCHK(hipGetLastError());
  }
  // 4. runs of equal block key
  stage.mark(3, s);
  std::vector<int64_t> run_start;
  std::vector<uint64_t> run_key;
  if (nnz > 0 && !blocked) {
    run_start.assign(1, 0);
    run_key.assign(1, 0);
  } else if (nnz > 0) {
    uint8_t* flag;
    int64_t* starts;
    uint64_t* keys_at;
    if ((rc = pool.get(&flag, nnz)) || (rc = pool.get(&starts, nnz))) return rc;
    hipLaunchKernelGGL(k_run_flags, dim3(grid_of(nnz)), dim3(256), 0, s, bkey, nnz, flag);
    HIPCHK(hipGetLastError());
    unsigned int* ws;
    if ((rc = pool.get(&ws, select_workspace_words(nnz)))) return rc;
    int64_t nruns = 0;
    if ((rc = select_flagged(flag, nnz, starts, &nruns, ws, s))) return rc;
    if ((rc = pool.get(&keys_at, nruns))) return rc;
    hipLaunchKernelGGL(k_gather_keys, dim3(grid_of(nruns)), dim3(256), 0, s, bkey, starts, nruns,
                       keys_at);
    HIPCHK(hipGetLastError());
    run_start.resize((size_t)nruns);
    run_key.resize((size_t)nruns);
    HIPCHK(hipMemcpyAsync(run_start.data(), starts, 8 * nruns, hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(run_key.data(), keys_at, 8 * nruns, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
  }
  finish_runs(L, nnz, run_start, run_key, cap, t, false);
  // the row flushes of sampled windows, where they need no run tables (a copy between pageable
  // memory and the device waits for the stream: the tables go up, and the counts come back, after
  // the frequent rows)
  if (!blocked && (rc = count_flushes_device(t, counts, s))) return rc;
  // 5. frequent rows
  stage.mark(4, s);
  pool.reuse();
  if ((rc = gpu_hot_rows(lp, nnz, hot_min, pool, s, t))) return rc;
  make_row_tables(t);
  stage.mark(5, s);
  if ((rc = upload_to(home, &t->d_hot, t->hot.data(), t->hot.size(), s, &acc)) ||
      (rc = upload_to(home, &t->d_tab, t->tab.data(), t->tab.size(), s, &acc)) ||
      (rc = upload_to(home, &t->d_run_start, t->run_start.data(), t->run_start.size(), s, &acc)) ||
      (rc = upload_to(home, &t->d_run_base, t->run_base.data(), t->run_base.size(), s, &acc)))
    return rc;
  if (blocked && nnz > 0) {
    const int64_t ntiles = (nnz + kTile - 1) / kTile;
    if ((rc = home.get(&t->d_tile_run, (size_t)ntiles, &acc))) return rc;
    hipLaunchKernelGGL(k_tile_run, dim3(grid_of(ntiles)), dim3(256), 0, s,
                       (const int64_t*)t->d_run_start, (int64_t)t->run_start.size() - 1, ntiles,
                       t->d_tile_run);
    HIPCHK(hipGetLastError());
  }
  if (blocked && (rc = count_flushes_device(t, counts, s))) return rc;
  if (t->placement == BLCO_PLACE_DEVICE &&
      (rc = home.get(&t->d_group, (size_t)L.N * kGroupBuckets, &acc)))
    return rc;
  t->device_bytes = acc;
  if (nnz >= kFlushMin)
    HIPCHK(hipMemcpyAsync(t->flush_rows, counts, sizeof(t->flush_rows), hipMemcpyDeviceToHost, s));
  if (t->placement == BLCO_PLACE_DEVICE && (rc = make_groups(t, s))) return rc;
  HIPCHK(hipStreamSynchronize(s));
  stage.read(t->build_stage_ms);
  return BLCO_OK;
}

size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// Workspace of a build: the larger of what linearizing, sorting and run detection hold
// together and what the frequent-row counts hold.
size_t build_workspace(const Layout& L, int64_t nnz) {
  const size_t n = (size_t)std::max<int64_t>(nnz, 1);
  const bool wide = L.T > 64, mid = wide && L.T <= 96;
  size_t a = 2048 + up256((size_t)L.N * 4 * 256 * 16) + up256((size_t)kEncBytes * 256 * 8);
  a += 2 * up256(8 * n);                                     // lo, lo2
  a += up256(8 * n) + up256(4 * n) + up256(4 * sort_workspace_words(nnz));   // spares
  if (wide) a += 2 * up256(4 * n);
  if (mid) a += 3 * up256(4 * n);
  if (wide && !mid) a += 4 * up256(8 * n);
  if (L.S > 0)   // block keys, flags, run starts
    a += 2 * up256(8 * n) + up256(n) + up256(4 * select_workspace_words(nnz)) + (1 << 20);
  const size_t smp = std::min<size_t>(n, (size_t)2 << 22);
  const size_t b = 8 * up256(4 * smp) + up256(smp) + up256(8 * smp) +
                   up256(4 * std::max(sort_workspace_words((int64_t)smp),
                                      select_workspace_words((int64_t)smp)));
  return std::max(a, b + 256);   // the flush counts are kept through both
}

// Storage of a tensor's arrays (the run tables of a blocked tensor, whose size the data
// decide, are allocated apart where they do not fit the slack).
size_t build_storage(const Layout& L, int64_t nnz) {
  const size_t n = (size_t)std::max<int64_t>(nnz, 1);
  return up256(8 * n) + up256(4 * n) + up256((n + kTile - 1) / kTile * 4) +
         up256((size_t)L.N * kHotMax * 4) + up256((size_t)L.N * kTabWords * 4) +
         up256((size_t)L.N * kGroupBuckets * 4) + 4096;
}

}  // namespace

static int build_device_impl(int nmodes, const uint64_t* dims, int64_t nnz,
                             const uint32_t* const* coords, const float* values,
                             const blco_build_opts* opts, void* storage, size_t storage_bytes,
                             void* workspace, size_t workspace_bytes, void* stream,
                             blco_tensor** out) {
  if (!out) return set_error(BLCO_EINVAL, "out is NULL");
  *out = nullptr;
  if (nmodes < 1 || nmodes > BLCO_MAX_MODES)
    return set_error(BLCO_EUNSUPPORTED, "nmodes %d outside 1..%d", nmodes, BLCO_MAX_MODES);
  if (!dims) return set_error(BLCO_EINVAL, "dims is NULL");
  if (nnz < 0) return set_error(BLCO_EINVAL, "nnz %lld < 0", (long long)nnz);
  if (nnz >= ((int64_t)1 << 31) - 1)
    return set_error(BLCO_EUNSUPPORTED, "the GPU builder takes fewer than 2^31 - 1 non-zeros");
  if (nnz > 0 && (!coords || !values)) return set_error(BLCO_EINVAL, "coords or values is NULL");
  for (int n = 0; n < nmodes; ++n) {
    if (dims[n] < 1) return set_error(BLCO_EINVAL, "dims[%d] = 0", n);
    if (dims[n] > (1ULL << 32))
      return set_error(BLCO_EUNSUPPORTED, "dims[%d] = %llu > 2^32", n, (unsigned long long)dims[n]);
    if (nnz > 0 && !coords[n]) return set_error(BLCO_EINVAL, "coords[%d] is NULL", n);
  }
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
  if (key_bits < 1 || key_bits > 64) return set_error(BLCO_EINVAL, "key_bits %d outside 1..64", key_bits);
  if (cap < 1) return set_error(BLCO_EINVAL, "max_block_nnz < 1");
  if (placement != BLCO_PLACE_DEVICE && placement != BLCO_PLACE_PINNED)
    return set_error(BLCO_EINVAL, "the GPU builder places the tensor on the device or in pinned memory");
  blco_tensor* t = new (std::nothrow) blco_tensor();
  if (!t) return set_error(BLCO_ENOMEM, "host allocation failed");
  t->placement = placement;
  t->hot_forced = opts && opts->hot_min_count > 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipGetDevice(&t->device) != hipSuccess) {
    delete t;
    return set_error(BLCO_EDEVICE, "hipGetDevice failed");
  }
  int rc = make_layout(nmodes, dims, key_bits, &t->lay);
  if (rc == BLCO_OK && storage && placement == BLCO_PLACE_DEVICE) {
    t->storage = static_cast<char*>(storage);
    t->storage_bytes = storage_bytes;
  }
  if (rc == BLCO_OK)
    rc = build_on_device(nmodes, dims, nnz, coords, values, key_bits, cap, hot_min, s, workspace,
                         workspace_bytes, t);
  if (rc == BLCO_OK && placement == BLCO_PLACE_PINNED) {
    // the non-zeros move to pinned host memory for streaming
    const size_t n1 = (size_t)std::max<int64_t>(nnz, 1);
    if (hipHostMalloc((void**)&t->h_keys, n1 * 8, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&t->h_vals, n1 * 4, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      rc = set_error(BLCO_ENOMEM, "pinned allocation of %lld non-zeros failed", (long long)nnz);
    } else {
      t->host_free = pinned_release;
      if (hipMemcpy(t->h_keys, t->d_keys, (size_t)nnz * 8, hipMemcpyDeviceToHost) != hipSuccess ||
          hipMemcpy(t->h_vals, t->d_vals, (size_t)nnz * 4, hipMemcpyDeviceToHost) != hipSuccess) {
        rc = set_error(BLCO_EDEVICE, "copy of the non-zeros to pinned memory failed");
      } else {
        (void)hipFree(t->d_keys);
        (void)hipFree(t->d_vals);
        t->d_keys = nullptr;
        t->d_vals = nullptr;
        t->device_bytes -= n1 * 12;
      }
    }
  }
  if (rc != BLCO_OK) {
    (void)hipStreamSynchronize(s);   // copies into the tensor may be under way
    release_tensor_arrays(t);
    delete t;
    return rc;
  }
  *out = t;
  return BLCO_OK;
}

extern "C" int blco_build_device(int nmodes, const uint64_t* dims, int64_t nnz,
                                 const uint32_t* const* coords, const float* values,
                                 const blco_build_opts* opts, void* stream, blco_tensor** out) {
  clear_error();
  return build_device_impl(nmodes, dims, nnz, coords, values, opts, nullptr, 0, nullptr, 0, stream,
                           out);
}

extern "C" int blco_build_device_in(int nmodes, const uint64_t* dims, int64_t nnz,
                                    const uint32_t* const* coords, const float* values,
                                    const blco_build_opts* opts, void* storage,
                                    size_t storage_bytes, void* workspace, size_t workspace_bytes,
                                    void* stream, blco_tensor** out) {
  clear_error();
  if ((!storage && storage_bytes) || (!workspace && workspace_bytes))
    return set_error(BLCO_EINVAL, "storage or workspace is NULL");
  if ((reinterpret_cast<uintptr_t>(storage) | reinterpret_cast<uintptr_t>(workspace)) & 255)
    return set_error(BLCO_EINVAL, "storage and workspace must be 256-byte aligned");
  return build_device_impl(nmodes, dims, nnz, coords, values, opts, storage, storage_bytes,
                           workspace, workspace_bytes, stream, out);
}

extern "C" int blco_build_device_sizes(int nmodes, const uint64_t* dims, int64_t nnz,
                                       const blco_build_opts* opts, size_t* storage_bytes,
                                       size_t* workspace_bytes) {
  clear_error();
  if (!storage_bytes || !workspace_bytes) return set_error(BLCO_EINVAL, "a size is NULL");
  if (nmodes < 1 || nmodes > BLCO_MAX_MODES)
    return set_error(BLCO_EUNSUPPORTED, "nmodes %d outside 1..%d", nmodes, BLCO_MAX_MODES);
  if (!dims) return set_error(BLCO_EINVAL, "dims is NULL");
  if (nnz < 0) return set_error(BLCO_EINVAL, "nnz %lld < 0", (long long)nnz);
  if (nnz >= ((int64_t)1 << 31) - 1)
    return set_error(BLCO_EUNSUPPORTED, "the GPU builder takes fewer than 2^31 - 1 non-zeros");
  for (int n = 0; n < nmodes; ++n) {
    if (dims[n] < 1) return set_error(BLCO_EINVAL, "dims[%d] = 0", n);
    if (dims[n] > (1ULL << 32))
      return set_error(BLCO_EUNSUPPORTED, "dims[%d] = %llu > 2^32", n, (unsigned long long)dims[n]);
  }
  const int key_bits = opts ? opts->key_bits : 64;
  if (key_bits < 1 || key_bits > 64) return set_error(BLCO_EINVAL, "key_bits %d outside 1..64", key_bits);
  Layout L;
  int rc = make_layout(nmodes, dims, key_bits, &L);
  if (rc) return rc;
  *storage_bytes = opts && opts->placement != BLCO_PLACE_DEVICE ? 0 : build_storage(L, nnz);
  *workspace_bytes = build_workspace(L, nnz);
  return BLCO_OK;
}
