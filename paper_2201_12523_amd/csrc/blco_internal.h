// Internal definitions shared by the host builder and the device runtime of
// the BLCO library.  Not installed; the public interface is include/blco.h.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/blco.h"

namespace blco {

constexpr int kTile = 64;  // non-zeros per wave tile (one per lane of a wave64)
constexpr int kHotMax = 256;  // frequent rows kept per mode
constexpr int kGroupBuckets = 1024;            // target-row buckets of a grouped MTTKRP
constexpr int64_t kGroupMinNnz = 1 << 20;      // fewer non-zeros are never grouped
// Table of a mode's frequent rows, as the window kernel's hot copies look them up: a
// multiplier, kTabSlots rows (0xFFFFFFFF: empty; the row r is at slot
// (r * multiplier) >> (32 - kTabBits)), and kTabSlots one-byte places in `hot`.
constexpr int kTabBits = 9;
constexpr int kTabSlots = 1 << kTabBits;
constexpr int kTabWords = 1 + kTabSlots + kTabSlots / 4;
// Windows sampled for a mode's row flushes: at most this many, evenly spaced, of kFlushWindow
// non-zeros each; their first halves give the flushes of windows half as long.
// Nothing asks for them in a launch of fewer than kFlushMin (win_wpt, group_pays), so a smaller
// tensor has none counted: a build of 100k took 30 us longer for them.
constexpr int kFlushSamples = 64;
constexpr int kFlushWindow = 4096;
constexpr int64_t kFlushMin = 1 << 19;
constexpr int64_t kHotMinCount = 2048;  // default: a frequent row holds at least this many non-zeros

// The bit map of a tensor (Sections 4.1-4.2).
struct Layout {
  int N = 0;
  uint64_t dims[BLCO_MAX_MODES] = {};
  int b[BLCO_MAX_MODES] = {};        // bits per mode
  int pos[BLCO_MAX_MODES][32] = {};  // ALTO position of bit j of mode n
  int T = 0, K = 0, S = 0;           // total bits, kept bits, block-key bits
  int w[BLCO_MAX_MODES] = {};        // kept bits of mode n
  int s[BLCO_MAX_MODES] = {};        // field shift of mode n in the key
  int h[BLCO_MAX_MODES] = {};        // bits of mode n in the block key
};

// Device-side state used only by blco_mttkrp_stream (owned by the tensor).
struct StreamState {
  void* copy_stream = nullptr;     // hipStream_t, library-owned, default priority
  void* ev_ready[2] = {nullptr, nullptr};
  void* ev_free[2] = {nullptr, nullptr};
  uint64_t* d_keys[2] = {nullptr, nullptr};
  float* d_vals[2] = {nullptr, nullptr};
  float* d_res[2] = {nullptr, nullptr};   // residual of each staged chunk (CP gradient)
  int64_t cap_nnz = 0;             // non-zeros per staging buffer
  int64_t res_cap = 0;             // non-zeros per residual buffer
  // timing events of the last call: per chunk copy start/end (copy stream)
  // and kernel start/end (caller's stream)
  std::vector<void*> ev_t;         // 4 per chunk
  int64_t timed_chunks = 0;
};

}  // namespace blco

struct blco_tensor {
  blco::Layout lay;
  int64_t nnz = 0;
  int placement = BLCO_PLACE_DEVICE;
  int64_t max_block_nnz = 0;
  // blocks after splitting (export / info), and runs of equal block key (kernels)
  std::vector<uint64_t> block_id;
  std::vector<int64_t> block_start;  // nblocks + 1
  std::vector<int64_t> run_start;    // nruns + 1
  std::vector<uint32_t> run_base;    // nruns * N: high bits of mode n of the run, already shifted by w_n
  std::vector<int32_t> tile_run;     // per 64-non-zero tile: run holding its first non-zero
  // host arrays (HOST: malloc, PINNED: hipHostMalloc; DEVICE: released after upload)
  uint64_t* h_keys = nullptr;
  float* h_vals = nullptr;
  void (*host_free)(void*) = nullptr;
  // device arrays
  uint64_t* d_keys = nullptr;
  float* d_vals = nullptr;
  int64_t* d_run_start = nullptr;
  uint32_t* d_run_base = nullptr;
  int32_t* d_tile_run = nullptr;
  double* d_partials = nullptr;  // sampled-loss partial sums (one per tile group)
  int64_t partials_cap = 0;
  // device arrays inside [storage, storage + storage_bytes) belong to the caller
  char* storage = nullptr;
  size_t storage_bytes = 0;
  bool owned(const void* q) const {
    return q && !(storage && (const char*)q >= storage && (const char*)q < storage + storage_bytes);
  }
  size_t device_bytes = 0;
  blco::StreamState st;
  size_t stream_peak_bytes = 0;
  int64_t stream_chunks = 0;
  int device = -1;
  int resolution = BLCO_RES_AUTO;   // conflict resolution (blco_set_resolution)
  // frequent rows of each mode (kHotMax per mode, most frequent first, padded
  // with 0xFFFFFFFF): the register-based kernel sums them per workgroup in LDS
  std::vector<uint32_t> hot;         // N * kHotMax
  std::vector<uint64_t> hot_cnt;     // N * (kHotMax + 1): estimated counts of the most frequent rows
  int nhot[BLCO_MAX_MODES] = {};
  bool hot_forced = false;           // an explicit threshold: stash whatever fits
  double build_stage_ms[5] = {};     // blco_build_device stage times (blco_info_t)
  uint32_t* d_hot = nullptr;
  std::vector<uint32_t> tab;         // N * kTabWords: row tables of the frequent rows
  uint32_t* d_tab = nullptr;
  // distinct rows of each mode over the sampled windows of kFlushWindow / 2 and kFlushWindow
  // non-zeros
  uint32_t flush_rows[BLCO_MAX_MODES][2] = {};
  // grouped MTTKRP: first non-zero of each bucket of a mode (N * kGroupBuckets), and the
  // multiplier that gives a row's bucket
  uint32_t* d_group = nullptr;
  bool grouped[BLCO_MAX_MODES] = {};
  uint32_t group_mul[BLCO_MAX_MODES] = {};
};

namespace blco {

int set_error(int code, const char* fmt, ...);
void clear_error();

// Device memory: ENOMEM where there is none (the HIP error is taken back, so that the caller may free
// some and try again), EDEVICE for other failures.  Defined in blco_device.hip.
int device_alloc(void** p, size_t bytes);

typedef void* (*HostAlloc)(size_t);
typedef void (*HostFree)(void*);

// Host half of blco_build: validates, linearizes, sorts, re-encodes, blocks.
// Fills everything but the device arrays.  h_keys/h_vals come from `alloc`
// and are released with `release` (NULL: malloc/free).
int host_build(int nmodes, const uint64_t* dims, int64_t nnz, const uint32_t* const* coords,
               const float* values, int key_bits, int64_t max_block_nnz, HostAlloc alloc,
               HostFree release, blco_tensor* t);

// Frequent rows of every mode (t->hot, t->nhot): rows counted over at most
// 2^22 evenly spaced non-zeros, the kHotMax most frequent whose estimated count
// reaches min_count (< 0: none).  Modes longer than 2^26 get none.
void find_hot_rows(const uint32_t* const* coords, int64_t nnz, int64_t min_count, blco_tensor* t);

// The row tables of the frequent rows (t->tab from t->hot and t->nhot).
void make_row_tables(blco_tensor* t);

void free_host_arrays(blco_tensor* t);

// Bit map of a tensor (Sections 4.1-4.2); EUNSUPPORTED when the block key
// would need more than 64 bits.
int make_layout(int N, const uint64_t* dims, int key_bits, Layout* L);

// Blocks, per-run high bits and tile -> run table from the runs of equal
// block key (run_start without the final nnz; run_key their block keys; tiles: whether the
// tile table is wanted).
void finish_runs(const Layout& L, int64_t nnz, const std::vector<int64_t>& run_start,
                 const std::vector<uint64_t>& run_key, int64_t max_block_nnz, blco_tensor* t,
                 bool tiles = true);

// blco_mttkrp with a workspace of ws_bytes (256-byte aligned; may be empty) for a caller that
// amplifies the sums' rounding, and the most workspace the call can use.  Defined in
// blco_device.hip.
int mttkrp_careful(blco_tensor* t, int mode, const void* const* factors, int factor_dtype,
                   int rank, float* out, void* ws, size_t ws_bytes, void* stream);
size_t mttkrp_workspace(const blco_tensor* t, int mode, int rank, int factor_dtype);

// First non-zero of the i-th sampled window of n >= kFlushMin non-zeros.
constexpr int64_t flush_start(int64_t n, int i) {
  return (n / kFlushWindow - 1) * i / (kFlushSamples - 1) * kFlushWindow;
}

// Counts the distinct rows of the sampled windows (t->flush_rows): on the host from the host
// arrays, or on the device from d_keys and the run tables there, into `counts` (device, cleared,
// sizeof(flush_rows) bytes), queued on `stream`.
void count_flushes(blco_tensor* t);
int count_flushes_device(blco_tensor* t, uint32_t* counts, void* stream);

// Bucket counts for the grouped MTTKRP, queued on `stream` (a hipStream_t), which it waits for
// first where the counted flushes decide.
int make_groups(blco_tensor* t, void* stream);

// Device sorting and compaction of the GPU builder (blco_sort.hip), ordered on
// stream s (a hipStream_t, void* here so the host builder needs no HIP header).
// The sort waits for s once (to read its digit counts) and returns with its
// passes queued; the selection waits for s to return the count.
//
// Stable ascending radix sort of n < 2^31 keys over bits [0, bits) (bits beyond
// them must be zero), with u32 values when vin != NULL: (kin, vin) -> (kout, vout),
// the input is only read, (ktmp, vtmp) are spares of n entries, ws holds
// sort_workspace_words(n) words.  The u32 form can sort descending (on the
// complemented key, still stable).  andor: the bitwise AND and OR of all keys where the
// caller has them (host; the sort then waits for nothing).
size_t sort_workspace_words(int64_t n);
int radix_sort_u64(const uint64_t* kin, const uint32_t* vin, uint64_t* kout, uint32_t* vout,
                   uint64_t* ktmp, uint32_t* vtmp, int64_t n, int bits, unsigned int* ws,
                   void* s, const uint64_t* andor = nullptr);
int radix_sort_u32(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout,
                   uint32_t* ktmp, uint32_t* vtmp, int64_t n, int bits, bool descending,
                   unsigned int* ws, void* s);

// The same sort with more values moved along: up to two u32 arrays (in32[0], then
// in32[1]) and one u64 array, at most three words per key (two u32 arrays exclude the
// u64 one); each output and spare array holds n entries, unused entries are NULL.
struct SortVals {
  const uint32_t* in32[2];
  uint32_t* out32[2];
  uint32_t* tmp32[2];
  const uint64_t* in64;
  uint64_t* out64;
  uint64_t* tmp64;
};
int radix_sort_u64_vals(const uint64_t* kin, uint64_t* kout, uint64_t* ktmp, const SortVals& v,
                        int64_t n, int bits, unsigned int* ws, void* s,
                        const uint64_t* andor = nullptr);
int radix_sort_u32_vals(const uint32_t* kin, uint32_t* kout, uint32_t* ktmp, const SortVals& v,
                        int64_t n, int bits, unsigned int* ws, void* s,
                        const uint64_t* andor = nullptr);

// The indices i < n with flag[i] != 0, ascending, into out; their number into
// *count (host).  ws holds select_workspace_words(n) words.
size_t select_workspace_words(int64_t n);
int select_flagged(const uint8_t* flag, int64_t n, int64_t* out, int64_t* count,
                   unsigned int* ws, void* s);

}  // namespace blco
