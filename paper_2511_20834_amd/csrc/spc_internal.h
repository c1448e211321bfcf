// Internal declarations shared by the translation units of libspc (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <memory>
#include <mutex>
#include <optional>
#include <tuple>
#include <vector>

#include "spc.h"

namespace spc {

// ---------------------------------------------------------------- errors
int set_error(int code, const char* fmt, ...);
#define SPC_HIP_CHECK(expr)                                                                       \
  do {                                                                                            \
    hipError_t e__ = (expr);                                                                      \
    if (e__ != hipSuccess)                                                                        \
      return ::spc::set_error(SPC_ERR_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__), \
                              __FILE__, __LINE__);                                                \
  } while (0)
#define SPC_RETURN_IF(expr)     \
  do {                          \
    int rc__ = (expr);          \
    if (rc__ != SPC_OK) return rc__; \
  } while (0)

// ---------------------------------------------------------------- streams
// What a stream handle stands for.  The handle alone does not say: the default stream's is the same on every device, and
// hipStreamPerThread in every thread.  An entry point makes one of these from the handle it was given; what is remembered
// (caches, levels, maps) remembers this.
struct StreamId {
  hipStream_t s = nullptr;
  int device = 0;
  uint32_t thread = 0;  // hipStreamPerThread: the number of its thread; else 0
  StreamId() = default;
  explicit StreamId(hipStream_t handle);  // on the current device, for the calling thread
  operator hipStream_t() const { return s; }
  bool here() const;  // whether the handle means this stream in the calling thread
  bool operator==(const StreamId& o) const { return s == o.s && device == o.device && thread == o.thread; }
  bool operator!=(const StreamId& o) const { return !(*this == o); }
  bool operator<(const StreamId& o) const { return std::tie(s, device, thread) < std::tie(o.s, o.device, o.thread); }
};
// Makes a device the current one for a scope (releases may come from a thread that works on another).
class DeviceScope {
  int before_ = -1;

 public:
  explicit DeviceScope(int device) {
    int now = device;
    if (hipGetDevice(&now) == hipSuccess && now != device && hipSetDevice(device) == hipSuccess) before_ = now;
  }
  ~DeviceScope() {
    if (before_ >= 0) (void)hipSetDevice(before_);
  }
  DeviceScope(const DeviceScope&) = delete;
  DeviceScope& operator=(const DeviceScope&) = delete;
};

// ---------------------------------------------------------------- device block cache
// hipMalloc costs tens of microseconds and synchronises; kernel maps are built per
// frame, so freed blocks are kept and handed out again — only to work on the stream
// that last used them, which makes stream order the only synchronisation needed.
void* pool_alloc(size_t bytes, const StreamId& stream);  // nullptr on failure (error set)
void pool_free(void* p, const StreamId& stream);
int pool_release_all();
// Blocks that hold zeros between their uses: whoever takes one leaves it cleared by the last kernel it enqueues on the
// stream (clean = false: it may not be).  As above, a block goes back to work on the same stream only; one that is taken is in nobody
// else's hands until it is given back.  NULL while the stream is being captured (replays of the graph would share the block with
// later calls), for hipStreamPerThread (such blocks would pile up with the threads), or when there is no memory.
// Small blocks come from memory that is part of the library's image; may_alloc: others, and what does not fit there, from the cache.
// Without it the call asks the runtime for no memory (a request would be refused, and end the recording, while another thread
// records a graph in the global mode).
void* zeroed_alloc(size_t bytes, const StreamId& stream, bool may_alloc);
void zeroed_free(void* p, size_t bytes, const StreamId& stream, bool clean);
// Makes everything enqueued on `waiter` from now on run after what `producer` holds at this moment
// (an event recorded on `producer`; nothing happens when the two are the same stream, or when `waiter` has been
// ordered behind `producer` before and the library has enqueued nothing on `producer` since and has never been recorded
// into a graph there).  Where one of them is another thread's hipStreamPerThread, which cannot be reached from here, the device is
// drained instead.  Used before a block goes back to the cache of a stream other than the one whose kernels last read it;
// the streams' device is the current one.
void order_stream_after(const StreamId& waiter, const StreamId& producer);
// Every library call that enqueues kernels reading pooled blocks on `s` says so once they are enqueued, or recorded (an
// order that another thread makes meanwhile is then made again): order_stream_after relies on it.
void note_stream_work(const StreamId& s);
struct StreamWorkNote {
  StreamId s;
  ~StreamWorkNote() { note_stream_work(s); }
};

// ---------------------------------------------------------------- counts the host waits for
// A level's count goes to device memory, and from there to a slot in pinned host memory, tagged with a number of this
// build's own, so that the host can poll for exactly this value.  A host that waited for an event and copied four bytes paid
// 21 us from the kernel's end to the number; the poll sees it about 2 us after the store.  The slot is written by the first
// search on the level, as it starts: by then the kernels that make the level have ended, so whoever has the count may read
// the keys, on any stream.
struct CountNote {
  unsigned long long* slot = nullptr;  // device address of the pinned slot, or NULL
  uint32_t tag = 0;
#ifdef __HIPCC__
  __device__ void publish(int v) const {
    if (slot)
      __hip_atomic_store(slot, (static_cast<unsigned long long>(tag) << 32) | static_cast<uint32_t>(v), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
#endif
};
// A slot is handed out again only to work on the stream that wrote it last (stream order keeps an earlier owner's late
// store in front of the new owner's, and the tag tells them apart).
struct CountSlot {
  unsigned long long* host = nullptr;
  unsigned long long* dev = nullptr;
  uint32_t tag = 0;
};
CountSlot count_slot_alloc(const StreamId& s);  // host == nullptr when no pinned memory is to be had
void count_slot_free(const CountSlot& c, const StreamId& s);

// ---------------------------------------------------------------- packing
struct PackInfo {
  int key_bits;
  int sh_b, sh_x, sh_y;  // left shifts of the batch/x/y fields (z has shift 0)
  int bits_b, bits_x, bits_y, bits_z;
  int used_bits;
};
int check_desc(const spc_pack_desc* d, PackInfo* pi);
// Mask that clears the low m bits of every spatial field (Section 5.3).
uint64_t level_mask(const PackInfo& pi, int m);

// ---------------------------------------------------------------- offset subsets
// Subset of the K^3 weight offsets (bit k of word k/32): all of them for a single dataflow, the dense or the
// sparse ones of the hybrid dual dataflow (Section 5.4).
constexpr int KMASK_WORDS = 11;  // 7^3 = 343 bits
struct KMask {
  uint32_t w[KMASK_WORDS];
#ifdef __HIPCC__
  __host__ __device__
#endif
  bool has(int k) const { return (w[k >> 5] >> (k & 31)) & 1u; }
};
// L1 norm of weight offset k in units of the input stride (Section 5.4: offsets below the threshold are the
// dense ones).  Even kernel sizes have offsets {0, 1} per axis.
inline int offset_l1(int K, int k) {
  const int iz = k % K, iy = (k / K) % K, ix = k / (K * K);
  if (K % 2 == 0) return ix + iy + iz;
  const int c = (K - 1) / 2;
  return (ix > c ? ix - c : c - ix) + (iy > c ? iy - c : c - iy) + (iz > c ? iz - c : c - iz);
}

// ---------------------------------------------------------------- coordinate levels
// One sorted packed-key array (a stride level).  n is known on the host for the
// caller's own array; for derived levels it lives on the device until the host asks.
struct Level {
  std::atomic<int> refs{1};
  void* keys = nullptr;   // device
  bool owns_keys = false;
  int64_t cap = 0;        // rows allocated / upper bound of n
  int64_t n_host = -1;    // -1: not yet fetched
  int64_t presumed = 0;   // rows it presumably holds: settled when it is made, whatever the host learns of the count later
  int64_t n_fetched = -1; // last value read back from n_dev (equals n_host unless the level was built under capture)
  bool captured = false;  // produced while its stream was being captured into a graph: every replay rewrites it
  int* n_dev = nullptr;   // device int (nullptr when n_host is authoritative from the start)
  CountSlot slot;         // where the host polls for the count (not for levels built under capture)
  bool announced = false; // a search that fills the slot has been enqueued
  int stride = 1;
  StreamId stream;               // stream the level was produced on
  std::vector<StreamId> readers; // other streams whose kernels read the keys (map searches)
  void add_reader(const StreamId& s) {
    if (s == stream) return;
    for (const StreamId& r : readers)
      if (r == s) return;
    readers.push_back(s);
  }
};
void level_unref(Level* l);
bool stream_is_capturing(hipStream_t s);

// Derive the levels with strides 2^m[i] of `src_keys` (mask, sort, unique), whose own stride is src_stride; out[i] for
// i < count.  Enqueues only.
int downsample_levels(const void* src_keys, int64_t n_src, int src_stride, const PackInfo& pi, const int* m, int count, Level** out,
                      const StreamId& stream);

// ---------------------------------------------------------------- packing (Section 5.3)
struct PackParams {
  int sh_b, sh_x, sh_y;
  int bits_b, bits_x, bits_y, bits_z;
  int ox, oy, oz, pad;
  uint32_t lim_x, lim_y, lim_z;  // a field holds v - origin below 2^bits - 2 pad
};

#ifdef __HIPCC__
// Key of one (b,x,y,z) row.  A field that does not fit (guard band on both sides included)
// gives the all-ones key and sets `bad`.
template <typename KeyT>
__device__ inline KeyT pack_key_flag(const int4 c, const PackParams& p, bool& bad) {
  // (in 32 bits: where v >= origin, the difference is the wrapped one; a limit of 2^bits - 2 pad below zero admits nothing)
  const uint32_t fx = uint32_t(c.y) - uint32_t(p.ox), fy = uint32_t(c.z) - uint32_t(p.oy), fz = uint32_t(c.w) - uint32_t(p.oz);
  const bool ok = uint32_t(c.x) < (1u << p.bits_b) && c.y >= p.ox && c.z >= p.oy && c.w >= p.oz && fx < p.lim_x && fy < p.lim_y && fz < p.lim_z;
  bad |= !ok;
  return ok ? (KeyT(c.x) << p.sh_b) | (KeyT(fx + p.pad) << p.sh_x) | (KeyT(fy + p.pad) << p.sh_y) | KeyT(fz + p.pad)
            : ~KeyT(0);
}
// Same, raising bit 0 of *status (when status is not NULL) for a rejected row.
template <typename KeyT>
__device__ inline KeyT pack_key(const int4 c, const PackParams& p, int32_t* status) {
  bool bad = false;
  const KeyT k = pack_key_flag<KeyT>(c, p, bad);
  if (bad && status) atomicOr(status, 1);
  return k;
}
// (a pointer that is not a kernel argument itself is a generic one to the compiler, and reads through it flat loads)
#define SPC_GLOBAL __attribute__((address_space(1)))
// Pins a loaded value in a vector register at this point of the program (used after a whole
// batch of loads has been issued): the compiler can then neither sink the loads into later
// branches nor spread them between other memory operations.  Loads and stores share one completion counter on this target, so a load
// that is waited for between stores also waits for every store issued before it.
#define SPC_PIN_LOADED(x) asm volatile("" : "+v"(x))
#endif

// ---------------------------------------------------------------- bucket sort (own kernels)
constexpr int BS_MAX_WG = 128;      // workgroups of the count / scatter passes of recorded sorts with a column scan
constexpr int BS_MAX_BIN_BITS = 14;
constexpr int BS_MAX_BIN = 1 << BS_MAX_BIN_BITS;  // fine bins (top used key bits)
// Sizes of the partitioning sort; below: one workgroup in LDS; above: rocPRIM (the split's regions and bins are sized for no more).
// 3 * 10^6 keys: pack + sort 66 us against 177 us with rocPRIM.
constexpr int64_t BS_MIN_N = 4096, BS_MAX_N = 8192 * 1024;
constexpr int64_t BS_LARGE_N = 600000;  // recorded sorts of fewer keys: in launches that count, scatter and rank (measured where these are)
inline bool use_bucket_sort(int64_t n) { return n >= BS_MIN_N && n <= BS_MAX_N; }
// Keys up to which the first pass adds its counts to the bins' totals, and how many a workgroup takes then.  Beyond, the additions
// (some 35 per ns, and hardly two keys of a workgroup share a bin) would take longer than a launch that sums the table's columns
// (pack + sort of 500 k random voxels with them 24.3 us, without 21.8; below the line eager sorts keep to two launches).
constexpr int64_t BS_ADD_N = 524288, BS_MID_N = 200000, BS_SHORT_N = 65536;
constexpr int BS_ADD_SHARE = 2048, BS_SHORT_SHARE = 1024, BS_LONG_SHARE = 4096;
// Up to so many workgroups their counts are summed where they are read, where totals would have to be cleared first: a launch
// less, but every workgroup reads the whole table.  Replayed pack + sort, us, cleared / summed: 4.2 k 20.8 / 17.2, 14 k 21.1 / 18.3, 33 k
// (32 workgroups) 22.4 / 20.5, 40 k 23.6 / 24.1, 60 k 24.0 / 27.8.
constexpr int BS_SUM_WG = 32;
constexpr int BS_PART = 64;         // keys per rank workgroup (recorded sorts)
constexpr int BS_PAD_KEYS = 32;     // all-ones keys kept behind the scattered keys
struct BucketPlan {
  int n_wg, per, shift, n_bin;
  bool add;  // the count pass adds the counts up itself (no column scan)
};
BucketPlan bucket_plan(int64_t n, int used_bits, bool unique);
size_t bucket_sort_ws_bytes(int key_bits, int64_t n);
// coords -> sorted keys (+ permutation); enqueues two kernels (split, merge), three above BS_ADD_N keys (bins' starts) or where
// there is no cleared block for the totals of more than BS_SUM_WG workgroups (their clearing), and one more where they are recorded
// (below BS_LARGE_N keys: count, scatter and rank).  Asks for no device memory.
int bucket_pack_sort(int key_bits, const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status,
                     void* keys_out, int32_t* perm_out, void* ws, const StreamId& s);
// One level to produce: the sorted distinct values of keys_in & mask, and their count.
constexpr int BS_MAX_LEVELS = 8;  // levels of one batch (the block rows of its launches)
struct LevelJob {
  uint64_t mask;
  void* keys_out;
  int32_t* count;
};
// n_levels <= BS_MAX_LEVELS levels of the same keys by the same three or four launches; level y works in ws + y * ws_pitch
int bucket_mask_unique(int key_bits, const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, void* ws,
                       size_t ws_pitch, const StreamId& s);

// fewer than BS_MIN_N keys: one workgroup sorts them in LDS, one launch
int small_pack_sort(int key_bits, const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status, void* keys_out,
                    int32_t* perm_out, hipStream_t s);
int small_mask_unique(int key_bits, const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, hipStream_t s);

// ---------------------------------------------------------------- sort (rocPRIM radix sort)
size_t sort_pairs_temp_bytes(int key_bits, int64_t n);
int sort_pairs(int key_bits, const void* keys_in, void* keys_out, const int32_t* vals_in, int32_t* vals_out,
               int64_t n, int end_bit, void* temp, size_t temp_bytes, hipStream_t s);
size_t sort_keys_temp_bytes(int key_bits, int64_t n);
int sort_keys(int key_bits, const void* keys_in, void* keys_out, int64_t n, int end_bit, void* temp,
              size_t temp_bytes, hipStream_t s);

}  // namespace spc

namespace spc {
// Event behind the last kernel of a network build, and the consumer stream that has waited for it most recently (stream
// order covers the maps' later uses there).
struct MapsReady {
  hipEvent_t e = nullptr;
  std::optional<StreamId> last_waiter;  // (none at first: the default stream is one like any other)
  ~MapsReady() {
    if (e) (void)hipEventDestroy(e);
  }
};
}  // namespace spc

// The 27 offsets of a 3x3x3 kernel leave mask bits free: the search marks the blocks of few pairs, from which the feature
// kernel tells a level whose neighbourhoods are nearly empty.  32 pairs are the voxels themselves, a cell that is multiplied on its
// own; with 18 more on average the product rows of the pooled way no longer fit its LDS at once (indoor scans, 64->64: 240 k voxels,
// 14 more, 40 us pooled and 46 by phases; 300 k, 17 more, 73 and 66).  Where a level's voxels are not their own neighbours (strided and
// transposed layers) all pairs are product rows and none is marked: random voxels, stride 2, 64->128, 110 k 84 us pooled and 42 by
// phases, 430 k 319 and 140.
constexpr uint32_t POOL_MARK = 1u << 31;
constexpr int POOL_BLOCK_PAIRS = 50;
constexpr int SHARED_TILES = 1024;  // tiles of a feature kernel that may be shared by several workgroups

// ---------------------------------------------------------------- kernel map object
struct spc_kmap {
  std::atomic<int> refs{1};
  spc::PackInfo pi{};
  spc_layer_desc desc{};
  int K3 = 0;
  bool sym = false;                 // WS lists hold offsets k < (K^3-1)/2 only (symmetric half-map)
  int k_lim = 0;                    // offsets that have a WS list of their own
  int hybrid_t = 0;                 // > 0: built for the hybrid dual dataflow with this threshold
  spc::KMask os_k{}, ws_k{};        // offsets whose matrix column / whose list the build wrote
  spc::Level* in_level = nullptr;   // the layer's input voxels
  spc::Level* out_level = nullptr;  // the layer's output voxels
  const int32_t* in_perm = nullptr; // caller's row number of every input voxel (borrowed), or NULL
  int64_t out_cap = 0;              // rows allocated in os_map / ws lists
  int64_t n_out_hint = -1;          // caller's estimate of n_out for kernel selection while n_host is unknown
  bool captured = false;            // built while its stream was being captured into a graph
  int64_t n_blocks_cap = 0;         // 32-row blocks allocated
  int mask_words = 0;               // ceil(K3/32)
  int32_t* os_map = nullptr;        // blocked OS layout [n_blocks][K3][32]: entry (i,k) at ((i/32)*K3+k)*32 + i%32
  uint32_t* block_masks = nullptr;  // [n_blocks][mask_words]: bit k set iff some row of the block has offset k
  int32_t* ws_in = nullptr;         // [K3][out_cap]
  int32_t* ws_out = nullptr;        // [K3][out_cap]
  int32_t* nnz_dev = nullptr;       // [K3]
  int32_t* tile_counts = nullptr;   // [K3][n_tiles] scratch of the two-pass compaction
  int32_t* list_base = nullptr;     // [n_blocks+1][K3]: first entry of every list whose output row is >= 32 * block
  int32_t* list_base_in = nullptr;  // symmetric half-map: the same by input row
  uint8_t* tile_sub = nullptr;      // [n_tiles][K3][tile/32]: pairs of the tile before every 32-row block (scratch of the list build)
  int2* tile_pairs = nullptr;       // per search tile a slab of compacted pairs (in, offset << 8 | row of the tile) (scratch of the list build)
  int64_t ws_stride = 0;            // entries between consecutive lists in ws_in / ws_out
  int32_t* arrived = nullptr;       // [SHARED_TILES] counters of feature kernels whose workgroups share tiles: zeroed by the build, left zero
  int32_t* inv_parent = nullptr;    // strided maps, on request: for every INPUT voxel p its pair (out q, offset k) as q*K^3+k
  spc_kmap* twin = nullptr;         // transposed map derived from its strided twin (a reference is held): WS lists alias the twin's
  int tile = 0, n_tiles = 0;
  std::vector<int64_t> nnz_host;    // filled lazily
  std::shared_ptr<spc::MapsReady> ready;  // set when nobody has joined the build stream: consumers on other streams wait for it
  std::vector<spc::StreamId> consumers;  // streams other than `stream` whose feature kernels have read the map
  spc::StreamId stream;             // stream the map was built on
};
