// Host-side runtime of libspc: error reporting, the device block cache, packing
// descriptors and coordinate-level bookkeeping.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <map>
#include <set>
#include <unordered_map>
#include <utility>
#include <vector>

#include "spc_internal.h"

namespace spc {

static thread_local char g_err[512] = "";

int set_error(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

// ---------------------------------------------------------------- streams
namespace {
void thread_ended(uint32_t thread);
// A number for every thread that has used hipStreamPerThread (never given twice); what the caches hold for the thread's
// stream goes to the others when it ends.
struct ThreadNumber {
  uint32_t n;
  ThreadNumber() {
    static std::atomic<uint32_t> next{0};
    n = ++next;
  }
  ~ThreadNumber() { thread_ended(n); }
};
uint32_t this_thread() {
  static thread_local ThreadNumber t;
  return t.n;
}
}  // namespace

StreamId::StreamId(hipStream_t handle) : s(handle), thread(handle == hipStreamPerThread ? this_thread() : 0) {
  if (hipGetDevice(&device) != hipSuccess) (void)hipGetLastError();
}
bool StreamId::here() const { return thread == 0 || thread == this_thread(); }

// ---------------------------------------------------------------- block cache
// Freed blocks are kept for reuse, binned by rounded size AND by the stream whose work
// last touched them: a block is handed out again only to work enqueued on that same
// stream, so stream order alone guarantees that the previous user has finished (blocks
// are returned right after the kernels that use them were enqueued, not after they ran).
namespace {
// Part of the library's image, on every device: blocks for zeroed_alloc that need no allocation.  A sort of up to half a million
// coordinates takes 4 to 32 KB per stream.
constexpr size_t IMAGE_BYTES = size_t(2) << 20, IMAGE_MOST = size_t(32) << 10;
__device__ __align__(256) unsigned char image_zeros[IMAGE_BYTES];
struct Image {
  char* base = nullptr;
  size_t used = 0;  // from the start
  int taken = 0;    // blocks in somebody's hands
  bool holds(const void* p) const { return base && p >= base && p < base + IMAGE_BYTES; }
};
struct Pool {
  std::mutex mu;
  std::map<std::pair<size_t, StreamId>, std::vector<void*>> free_blocks;
  std::unordered_map<void*, size_t> live;  // block -> rounded size
  std::map<std::pair<size_t, StreamId>, std::vector<void*>> zeroed;  // (live as far as the above is concerned)
  size_t n_zeroed = 0;  // of them from the cache
  std::map<int, Image> images;  // by device
  std::map<int, std::vector<std::pair<size_t, void*>>> ended;  // by device: free blocks of threads that are no more, with their sizes
  bool take(size_t r, const StreamId& stream, void** p) {
    auto it = free_blocks.find({r, stream});
    if (it == free_blocks.end() || it->second.empty()) return false;
    *p = it->second.back();
    it->second.pop_back();
    live[*p] = r;
    return true;
  }
};
Pool& pool() {
  static Pool* p = new Pool;  // never destroyed: device memory is reclaimed by the driver at exit
  return *p;
}
size_t round_size(size_t b) {
  if (b < 4096) return 4096;
  if (b < (size_t(1) << 20)) {  // next power of two below 1 MiB
    size_t r = 4096;
    while (r < b) r <<= 1;
    return r;
  }
  const size_t g = size_t(1) << 20;  // 1 MiB granules above
  return (b + g - 1) / g * g;
}
}  // namespace

void* pool_alloc(size_t bytes, const StreamId& stream) {
  const size_t r = round_size(bytes);
  Pool& P = pool();
  void* p = nullptr;
  bool adopt = false;
  {
    std::lock_guard<std::mutex> lk(P.mu);
    if (P.take(r, stream, &p)) return p;
    auto it = P.ended.find(stream.device);
    adopt = it != P.ended.end() && !it->second.empty();
  }
  // What an ended thread's stream has used is anybody's once the device has been drained.
  if (adopt && !stream_is_capturing(stream)) {
    std::vector<std::pair<size_t, void*>> blocks;
    {
      std::lock_guard<std::mutex> lk(P.mu);
      blocks.swap(P.ended[stream.device]);
    }
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    if (!idle) (void)hipGetLastError();
    std::lock_guard<std::mutex> lk(P.mu);
    for (const auto& b : blocks) {
      if (idle) P.free_blocks[{b.first, stream}].push_back(b.second);
      else P.ended[stream.device].push_back(b);
    }
    if (P.take(r, stream, &p)) return p;
  }
  hipError_t e = hipMalloc(&p, r);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    pool_release_all();
    e = hipMalloc(&p, r);
  }
  if (e != hipSuccess) {
    set_error(SPC_ERR_NOMEM, "hipMalloc(%zu) failed: %s", r, hipGetErrorString(e));
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(P.mu);
  P.live[p] = r;
  return p;
}

void pool_free(void* p, const StreamId& stream) {
  if (!p) return;
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  auto it = P.live.find(p);
  if (it == P.live.end()) return;
  P.free_blocks[{it->second, stream}].push_back(p);
  P.live.erase(it);
}

namespace {
constexpr size_t MAX_ZEROED = 256;  // kept blocks; further ones go back to the ordinary cache
__global__ __launch_bounds__(256) void clear_kernel(uint4* p, size_t n) {
  const size_t i = blockIdx.x * size_t(256) + threadIdx.x;
  if (i < n) p[i] = make_uint4(0, 0, 0, 0);
}
}  // namespace

void* zeroed_alloc(size_t bytes, const StreamId& stream, bool may_alloc) {
  if (stream.thread != 0 || stream_is_capturing(stream)) return nullptr;
  const size_t r = round_size(bytes);
  Pool& P = pool();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    Image& image = P.images[stream.device];
    auto it = P.zeroed.find({r, stream});
    if (it != P.zeroed.end() && !it->second.empty()) {
      void* p = it->second.back();
      it->second.pop_back();
      if (image.holds(p)) ++image.taken;
      else --P.n_zeroed;
      return p;
    }
    if (!image.base && r <= IMAGE_MOST) {
      void* p = nullptr;
      if (hipGetSymbolAddress(&p, HIP_SYMBOL(image_zeros)) == hipSuccess) image.base = static_cast<char*>(p);
      else (void)hipGetLastError();
    }
    if (image.base && r <= IMAGE_MOST && image.used + r <= IMAGE_BYTES) {
      void* p = image.base + image.used;
      image.used += r;
      ++image.taken;
      return p;
    }
  }
  if (!may_alloc) return nullptr;
  void* p = pool_alloc(r, stream);
  if (!p) return nullptr;
  hipLaunchKernelGGL(clear_kernel, dim3(static_cast<unsigned>((r / 16 + 255) / 256)), dim3(256), 0, stream, static_cast<uint4*>(p), r / 16);
  if (hipGetLastError() == hipSuccess) return p;
  pool_free(p, stream);
  return nullptr;
}

void zeroed_free(void* p, size_t bytes, const StreamId& stream, bool clean) {
  Pool& P = pool();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    Image& image = P.images[stream.device];
    const bool in_image = image.holds(p);
    if (in_image && !clean) return;  // (counts as taken for good)
    if (clean && (in_image || P.n_zeroed < MAX_ZEROED)) {
      P.zeroed[{round_size(bytes), stream}].push_back(p);
      if (in_image) --image.taken;
      else ++P.n_zeroed;
      return;
    }
  }
  pool_free(p, stream);
}

namespace {
// How much the library has enqueued on every stream, and how much of it each (waiter, producer) pair has been ordered
// behind: releasing the maps of a network asks for the same pair dozens of times with nothing new in between (a
// release of 25 layers' maps on three streams took the host 230 us in event records and cross-stream waits, now 94).
// A stream the library has been recorded on may also hold replays of that graph, which nobody counts: it is asked for an
// event every time.
struct StreamOrder {
  std::mutex mu;
  std::map<StreamId, uint64_t> work;
  std::map<std::pair<StreamId, StreamId>, uint64_t> ordered;
  std::set<StreamId> recorded;
  bool all_recorded = false;  // more recorded streams than are worth remembering: every stream counts as one
};
StreamOrder& stream_order() {
  static StreamOrder* o = new StreamOrder;
  return *o;
}
constexpr size_t MAX_TRACKED_STREAMS = 1024;
}  // namespace

void note_stream_work(const StreamId& s) {
  const bool recording = stream_is_capturing(s);
  StreamOrder& O = stream_order();
  std::lock_guard<std::mutex> lk(O.mu);
  if (recording && O.recorded.size() < MAX_TRACKED_STREAMS) O.recorded.insert(s);
  else if (recording && !O.recorded.count(s)) O.all_recorded = true;
  if (O.work.size() > MAX_TRACKED_STREAMS || O.ordered.size() > MAX_TRACKED_STREAMS) {  // forgetting only means ordering once more
    O.work.clear();
    O.ordered.clear();
  }
  ++O.work[s];
}

void order_stream_after(const StreamId& waiter, const StreamId& producer) {
  if (waiter == producer) return;
  if (!waiter.here() || !producer.here()) {
    if (hipDeviceSynchronize() != hipSuccess) (void)hipGetLastError();
    return;
  }
  // (an order recorded into a graph says nothing about eager work, and the other way round)
  StreamOrder& O = stream_order();
  std::lock_guard<std::mutex> lk(O.mu);  // held until the wait is enqueued: whoever finds the entry may rely on it
  if (!stream_is_capturing(waiter) && !stream_is_capturing(producer) && !O.all_recorded && !O.recorded.count(producer)) {
    const uint64_t now = O.work[producer];
    auto it = O.ordered.find({waiter, producer});
    if (it != O.ordered.end() && it->second == now) return;
    O.ordered[{waiter, producer}] = now;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipStreamSynchronize(producer);  // no event to be had: wait on the host instead
    return;
  }
  if (hipEventRecord(e, producer) != hipSuccess || hipStreamWaitEvent(waiter, e, 0) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipStreamSynchronize(producer);
  }
  (void)hipEventDestroy(e);  // released once the record has completed
}

// ---------------------------------------------------------------- pinned count slots
namespace {
constexpr size_t SLOT_PITCH = 64, SLOTS_PER_PAGE = 64;
struct Slots {
  std::mutex mu;
  uint32_t next_tag = 0;
  std::map<StreamId, std::vector<CountSlot>> free_slots;
  std::vector<CountSlot> ended;  // of threads that are no more (a late store of theirs carries another tag: the host then copies the count)
};
Slots& slots() {
  static Slots* p = new Slots;
  return *p;
}
}  // namespace

CountSlot count_slot_alloc(const StreamId& s) {
  Slots& S = slots();
  std::lock_guard<std::mutex> lk(S.mu);
  std::vector<CountSlot>& v = S.free_slots[s];
  if (v.empty() && !S.ended.empty()) {
    v.push_back(S.ended.back());
    S.ended.pop_back();
  }
  if (v.empty()) {
    void *h = nullptr, *d = nullptr;
    if (hipHostMalloc(&h, SLOT_PITCH * SLOTS_PER_PAGE, hipHostMallocMapped | hipHostMallocCoherent | hipHostMallocPortable) != hipSuccess ||
        hipHostGetDevicePointer(&d, h, 0) != hipSuccess) {
      (void)hipGetLastError();
      if (h) (void)hipHostFree(h);
      return CountSlot{};
    }
    memset(h, 0, SLOT_PITCH * SLOTS_PER_PAGE);
    for (size_t i = 0; i < SLOTS_PER_PAGE; ++i) {
      CountSlot c;
      c.host = reinterpret_cast<unsigned long long*>(static_cast<char*>(h) + i * SLOT_PITCH);
      c.dev = reinterpret_cast<unsigned long long*>(static_cast<char*>(d) + i * SLOT_PITCH);
      v.push_back(c);
    }
  }
  CountSlot c = v.back();
  v.pop_back();
  if (++S.next_tag == 0) ++S.next_tag;
  c.tag = S.next_tag;
  return c;
}

void count_slot_free(const CountSlot& c, const StreamId& s) {
  if (!c.host) return;
  Slots& S = slots();
  std::lock_guard<std::mutex> lk(S.mu);
  S.free_slots[s].push_back(c);
}

namespace {
void thread_ended(uint32_t thread) {
  {
    Pool& P = pool();
    std::lock_guard<std::mutex> lk(P.mu);
    for (auto it = P.free_blocks.begin(); it != P.free_blocks.end();) {
      const StreamId& id = it->first.second;
      if (id.thread != thread) {
        ++it;
        continue;
      }
      for (void* b : it->second) P.ended[id.device].push_back({it->first.first, b});
      it = P.free_blocks.erase(it);
    }
  }
  Slots& S = slots();
  std::lock_guard<std::mutex> lk(S.mu);
  for (auto it = S.free_slots.begin(); it != S.free_slots.end();) {
    if (it->first.thread != thread) {
      ++it;
      continue;
    }
    S.ended.insert(S.ended.end(), it->second.begin(), it->second.end());
    it = S.free_slots.erase(it);
  }
}
}  // namespace

int pool_release_all() {
  Pool& P = pool();
  std::map<int, std::vector<void*>> blocks;  // by device
  std::set<int> images;                      // whose blocks go back to the image
  {
    std::lock_guard<std::mutex> lk(P.mu);
    for (auto& kv : P.free_blocks)
      for (void* b : kv.second) blocks[kv.first.second.device].push_back(b);
    P.free_blocks.clear();
    for (auto& kv : P.images)
      if (kv.second.used > 0 && kv.second.taken == 0) {
        images.insert(kv.first);
        blocks[kv.first];
        kv.second.used = IMAGE_BYTES;  // (nobody takes any before the device has been drained)
      }
    for (auto it = P.zeroed.begin(); it != P.zeroed.end();) {
      const int device = it->first.second.device;
      std::vector<void*> kept;
      for (void* b : it->second) {
        if (!P.images[device].holds(b)) {
          blocks[device].push_back(b);
          P.live.erase(b);
        } else if (!images.count(device)) {
          kept.push_back(b);
        }
      }
      it->second.swap(kept);
      it = it->second.empty() ? P.zeroed.erase(it) : std::next(it);
    }
    P.n_zeroed = 0;
    for (auto& kv : P.ended)
      for (const auto& b : kv.second) blocks[kv.first].push_back(b.second);
    P.ended.clear();
  }
  for (auto& kv : blocks) {
    const DeviceScope scope(kv.first);
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    for (void* b : kv.second) (void)hipFree(b);
    if (!images.count(kv.first) || !idle) continue;
    std::lock_guard<std::mutex> lk(P.mu);
    P.images[kv.first].used = 0;
  }
  return SPC_OK;
}

// ---------------------------------------------------------------- descriptors
int check_desc(const spc_pack_desc* d, PackInfo* pi) {
  if (!d) return set_error(SPC_ERR_ARG, "pack descriptor is NULL");
  if (d->key_bits != 32 && d->key_bits != 64) return set_error(SPC_ERR_ARG, "key_bits must be 32 or 64");
  const int b[4] = {d->bits_b, d->bits_x, d->bits_y, d->bits_z};
  int sum = 0;
  for (int i = 0; i < 4; ++i) {
    if (b[i] < 0 || b[i] > 31) return set_error(SPC_ERR_ARG, "field width %d out of [0,31]", b[i]);
    sum += b[i];
  }
  if (d->bits_x < 1 || d->bits_y < 1 || d->bits_z < 1) return set_error(SPC_ERR_ARG, "spatial fields need >= 1 bit");
  if (sum > d->key_bits) return set_error(SPC_ERR_ARG, "fields need %d bits, key has %d", sum, d->key_bits);
  if (d->pad < 0) return set_error(SPC_ERR_ARG, "pad must be >= 0");
  pi->key_bits = d->key_bits;
  pi->bits_b = d->bits_b;
  pi->bits_x = d->bits_x;
  pi->bits_y = d->bits_y;
  pi->bits_z = d->bits_z;
  pi->sh_y = d->bits_z;
  pi->sh_x = d->bits_z + d->bits_y;
  pi->sh_b = d->bits_z + d->bits_y + d->bits_x;
  pi->used_bits = sum;
  return SPC_OK;
}

uint64_t level_mask(const PackInfo& pi, int m) {
  auto field = [&](int bits) -> uint64_t {
    uint64_t all = (bits >= 64) ? ~uint64_t(0) : ((uint64_t(1) << bits) - 1);
    uint64_t low = (m >= bits) ? all : ((uint64_t(1) << m) - 1);
    return all & ~low;
  };
  uint64_t mask = 0;
  mask |= ((pi.bits_b ? ((uint64_t(1) << pi.bits_b) - 1) : 0) << pi.sh_b);
  mask |= field(pi.bits_x) << pi.sh_x;
  mask |= field(pi.bits_y) << pi.sh_y;
  mask |= field(pi.bits_z);
  return mask;
}

bool stream_is_capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return st != hipStreamCaptureStatusNone;
}

void level_unref(Level* l) {
  if (!l) return;
  if (l->refs.fetch_sub(1) == 1) {
    // the blocks go back to the producing stream's cache: that stream must not reuse them before the
    // searches that read the keys on other streams have finished
    if (!l->readers.empty() && (l->owns_keys || l->n_dev)) {
      const DeviceScope scope(l->stream.device);
      for (const StreamId& r : l->readers) order_stream_after(l->stream, r);
    }
    if (l->owns_keys) pool_free(l->keys, l->stream);
    pool_free(l->n_dev, l->stream);
    count_slot_free(l->slot, l->stream);
    delete l;
  }
}

}  // namespace spc

extern "C" {

const char* spc_last_error(void) { return spc::g_err; }
const char* spc_version(void) { return "spc-gfx950 0.1"; }
int spc_release_cache(void) { return spc::pool_release_all(); }

static int ceil_log2(int64_t v) {  // smallest b with 2^b >= v
  int b = 0;
  while ((int64_t(1) << b) < v) ++b;
  return b;
}

int spc_pack_desc_fit(const int32_t lo[3], const int32_t hi[3], int32_t n_batch, int32_t max_stride,
                      int32_t max_reach, int32_t key_bits, spc_pack_desc* out) {
  if (!lo || !hi || !out) return spc::set_error(SPC_ERR_ARG, "NULL argument");
  if (n_batch < 1 || max_stride < 1 || (max_stride & (max_stride - 1)) || max_reach < 0)
    return spc::set_error(SPC_ERR_ARG, "n_batch >= 1, max_stride a power of two, max_reach >= 0 required");
  if (key_bits != 0 && key_bits != 32 && key_bits != 64) return spc::set_error(SPC_ERR_ARG, "key_bits must be 0, 32 or 64");
  const int64_t S = max_stride;
  const int64_t pad = (int64_t(max_reach) + S - 1) / S * S;
  int bits[3];
  for (int a = 0; a < 3; ++a) {
    if (hi[a] < lo[a]) return spc::set_error(SPC_ERR_ARG, "hi < lo on axis %d", a);
    int64_t l = lo[a];
    int64_t org = (l >= 0 ? l / S : -((-l + S - 1) / S)) * S;  // floor to a multiple of S
    out->origin[a] = static_cast<int32_t>(org);
    bits[a] = std::max(1, ceil_log2(int64_t(hi[a]) - org + 2 * pad + 1));
    if (bits[a] > 31) return spc::set_error(SPC_ERR_RANGE, "axis %d needs %d bits", a, bits[a]);
  }
  out->bits_b = ceil_log2(n_batch);
  out->bits_x = bits[0];
  out->bits_y = bits[1];
  out->bits_z = bits[2];
  out->pad = static_cast<int32_t>(pad);
  const int sum = out->bits_b + bits[0] + bits[1] + bits[2];
  if (sum > 64 || (key_bits == 32 && sum > 32)) return spc::set_error(SPC_ERR_RANGE, "coordinates need %d key bits", sum);
  out->key_bits = key_bits ? key_bits : (sum <= 32 ? 32 : 64);
  return SPC_OK;
}

}  // extern "C"
