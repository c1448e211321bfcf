// C entries to the emulated sort, for ctypes.  `bucket_sort.inc` is csrc/bucket_sort.hip with the names of the emulator in it.
#include "bucket_sort.inc"

#include <sys/mman.h>

#include <random>
#include <string>

namespace {
bool keep_totals, recording;
std::vector<int32_t> totals;  // the library's cleared block
int disturb_how = -1;
uint16_t* disturb_ws;
size_t disturb_words;
std::mt19937 disturb_rng;
int launches;
}  // namespace

namespace spc {
int set_error(int code, const char*, ...) { return code; }
StreamId::StreamId(hipStream_t h) : s(h) {}
bool StreamId::here() const { return true; }
bool stream_is_capturing(hipStream_t) { return recording; }
void* zeroed_alloc(size_t bytes, const StreamId&, bool) {
  if (!keep_totals || recording) return nullptr;
  totals.assign(bytes / 4, 0);
  return totals.data();
}
void zeroed_free(void*, size_t, const StreamId&, bool) {
  if (disturb_how >= 0) return;
  for (int32_t t : totals)
    if (t != 0) fprintf(stderr, "the totals were not left cleared\n"), abort();
}
}  // namespace spc

void emu::before_launch(const char* kernel) {
  ++launches;
  if (disturb_how < 0 || !strstr(kernel, "merge")) return;
  for (size_t i = 0; i < disturb_words; ++i)
    if (disturb_rng() % 97 == 0) disturb_ws[i] = static_cast<uint16_t>(disturb_rng());
  if (disturb_words > 0 || totals.empty()) return;
  for (int i = 0; i < 256; ++i) {
    int32_t& t = totals[disturb_rng() % totals.size()];
    t = disturb_how == 0 ? 2 * t : disturb_how == 1 ? 0 : disturb_how == 2 ? t + 3000 : t / 2;
  }
}

extern "C" {
// Memory that ends (up to its alignment) where nothing may be touched.
void* emu_guarded(size_t bytes, size_t align) {
  const size_t page = 4096, used = (bytes + page - 1) / page * page;
  char* m = static_cast<char*>(mmap(nullptr, used + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  mprotect(m, page, PROT_NONE);
  mprotect(m + page + used, page, PROT_NONE);
  char* p = m + page + (used - bytes) / align * align;
  memset(p, 0xee, bytes);
  return p;
}
// disturb: -1, how the totals are changed before they are read (0 to 3), or that the workspace is, if one is given
void emu_mode(int keep, int record, int disturb, int seed, void* ws, size_t ws_bytes) {
  disturb_ws = static_cast<uint16_t*>(ws);
  disturb_words = ws_bytes / 2;
  keep_totals = keep != 0;
  recording = record != 0;
  disturb_how = disturb;
  disturb_rng.seed(seed);
  launches = 0;
}
int emu_launches() { return launches; }
size_t emu_ws_bytes(int key_bits, int64_t n) { return spc::bucket_sort_ws_bytes(key_bits, n); }
int emu_pack_sort(int key_bits, const int32_t* coords, int64_t n, const int* bits, int pad, void* keys, int32_t* perm, void* ws) {
  auto limit = [&](int b) { return static_cast<uint32_t>((int64_t(1) << b) - 2 * pad); };
  const spc::PackParams p{bits[0] + bits[1] + bits[2], bits[1] + bits[2], bits[2], 0, bits[0], bits[1], bits[2], 0, 0, 0, pad,
                          limit(bits[0]), limit(bits[1]), limit(bits[2])};
  return spc::bucket_pack_sort(key_bits, reinterpret_cast<const int4*>(coords), n, p, bits[0] + bits[1] + bits[2], nullptr, keys, perm, ws,
                               spc::StreamId(nullptr));
}
int emu_levels(int key_bits, const void* keys, int64_t n, int used_bits, int count, const uint64_t* masks, void** out, int32_t* counts, void* ws,
               size_t pitch) {
  spc::LevelJob jobs[spc::BS_MAX_LEVELS];
  for (int y = 0; y < count; ++y) jobs[y] = {masks[y], out[y], counts + y};
  return spc::bucket_mask_unique(key_bits, keys, n, jobs, count, used_bits, ws, pitch, spc::StreamId(nullptr));
}
}
