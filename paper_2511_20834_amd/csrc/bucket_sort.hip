// Sort of packed voxel keys for the cloud sizes of this workload (thousands to a few million
// keys), without look-back spinning: every workgroup orders its share of the keys by the top `fb` used key bits ("bins") in LDS, and
// further workgroups take whole bins from all shares and put them in order (two launches, see split + merge; crowded bins are shared).
// Fewer keys than BS_MIN_N are sorted by one workgroup.  Recorded sorts (stream capture) of up to BS_LARGE_N keys go another
// way, in three launches or four:
//
//   count    each workgroup produces its share of the keys, histograms their bins in LDS, adds its counts to the bins' totals in
//            memory and keeps what it found there, its place inside the bins, in its row of a table (or writes the counts);
//   colscan  (above BS_ADD_N) exclusive prefixes down the table's columns, and the bins' totals;
//   scatter  each workgroup scans the bin totals (where every bin starts) and moves its keys,
//            with their source index, to their bin's range; the workgroups also write, for every
//            64 scattered positions, the window of whole bins that covers them;
//   rank     64 keys per workgroup; a key's final position is the start of its window plus the
//            number of window keys that sort before it, counted by comparing against every
//            window key (see bs_rank_kernel).
//
// Equal keys (not a valid cloud, but not rejected unless validation was asked for) get distinct positions, so the permutation is
// complete whatever the input.  32-bit keys that are split and merged are ordered as (key, source) pairs; among equal 64-bit keys, and in
// recorded sorts that scatter, the order is that of LDS atomics and not the same from run to run.  Downsampling sorts the masked keys
// alone and drops the repeated ones.
#include <algorithm>
#include <type_traits>

#include "spc_internal.h"

namespace spc {

constexpr int BS_THREADS = 256;   // sort / gather workgroups
constexpr int BS_WIDE = 1024;     // count / scan / scatter workgroups

__device__ inline int bs_bin(uint64_t key, int shift, int n_bin) {
  const uint64_t b = key >> shift;
  return b < uint64_t(n_bin) ? static_cast<int>(b) : n_bin - 1;  // all-ones keys of rejected rows go last
}

// ---------------------------------------------------------------- key sources
// A source splits "fetch" from "make the key": the kernels below fetch a batch of rows first and
// only then compute, so that the batch's loads are in flight together.
template <typename KeyT>
struct SrcPack {
  const int4* coords;
  PackParams p;
  int32_t* status;
  struct Raw {
    int4 c;
  };
  __device__ Raw load(int64_t i) const { return Raw{coords[i]}; }
  __device__ static void pin(Raw& r) { SPC_PIN_LOADED(r.c.x); }
  __device__ KeyT key(const Raw& r, bool& bad) const { return pack_key_flag<KeyT>(r.c, p, bad); }
  __device__ bool skip(const Raw&, KeyT) const { return false; }
  __device__ SrcPack level(int) const { return *this; }
  __device__ void report(bool bad) const {
    if (bad && status) atomicOr(status, 1);
  }
};
template <typename KeyT>
struct SrcMask {
  const KeyT* keys;
  KeyT mask;
  struct Raw {
    KeyT cur, prev;
    bool has_prev;
  };
  __device__ Raw load(int64_t i) const { return Raw{keys[i], keys[i > 0 ? i - 1 : 0], i > 0}; }
  __device__ static void pin(Raw& r) {
    SPC_PIN_LOADED(r.cur);
    SPC_PIN_LOADED(r.prev);
  }
  __device__ KeyT key(const Raw& r, bool&) const { return r.cur & mask; }
  // The finer level is sorted, so runs along z collapse to runs of equal masked keys: only the
  // first key of a run takes part (the result is the set of distinct keys either way).
  __device__ bool skip(const Raw& r, KeyT key) const { return r.has_prev && (r.prev & mask) == key; }
  __device__ void report(bool) const {}
};
// A batch of levels of one network is produced by the same launches: block row y makes level y.
template <typename KeyT>
struct SrcMasks {
  const KeyT* keys;
  KeyT masks[BS_MAX_LEVELS];
  __device__ SrcMask<KeyT> level(int y) const { return SrcMask<KeyT>{keys, masks[y]}; }
};

// This block row's copy of a workspace array: the workspaces of a batch of levels lie ws_pitch bytes apart.
template <typename T>
__device__ inline T* level_ws(T* p, size_t ws_pitch) {
  using Byte = std::conditional_t<std::is_const<T>::value, const char, char>;
  return reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + blockIdx.y * ws_pitch);
}

// ---------------------------------------------------------------- split + merge
// The sort in two launches (three with the bins' starts of large inputs, one more for levels):
//
//   split   (bs_count_kernel, SPLIT) a workgroup makes its share of the keys, orders them by bin in LDS and stores them, bin after
//           bin, to a region of its own, with a row of the table `off` that says where every bin starts in there (16 bits each; the
//           last entry is the region's number of keys).  Nothing is scattered in memory.  Up to BS_ADD_N keys it also adds its counts
//           to the bins' totals;
//   starts  (bs_starts_kernel, above BS_ADD_N keys, where that would be too many additions, and for recorded levels) sums the
//           table's columns, which gives every bin's place in the sorted sequence, and from these every merging workgroup's bins;
//   merge   workgroup p takes the whole bins that start among sorted positions p * q .. p * q + q - 1: one contiguous piece of every
//           region.  It fetches them, orders them in LDS (a second split by their next key bits, then counting inside that split's
//           bins) and stores them, lane next to lane.  A bin of more keys than fit the LDS beside others is shared by the workgroups
//           whose positions it covers: each reads all of it, but takes only the second bins that start among its positions (crowd);
//   compact (levels) equal keys are all in one workgroup, which drops them; this kernel closes the gaps between the workgroups.
//
// No windows overlap and nothing is compared twice, and no key is a memory transaction of its own on its
// way.  What bounds it up to half a million keys: two launches, three dependent round trips of the merge (totals, pieces, keys) and
// fetching its instructions, which run once: unrolled eight and sixteen times the same merge took 17 us where this one takes 8.6,
// so loops over bins and regions stay rolled and a thread has two keys.  From 10^6 keys on: the coordinates (split 30 us at 3 * 10^6),
// whose workgroups fill a CU's LDS, and the short pieces (merge 30 us).  us, kernels of count / scatter / rank (and column scan, windows that did
// not fit, from 600 k) against split / starts / merge: 6 k 4.0 / 4.4 / 4.3 against 4.0 / - / 6.6; LiDAR 120 k 4.9 / 6.5 / 9.4 against 5.0 / - / 8.6;
// indoor 240 k 7.4 / 11.2 / 13.2 against 9.0 / - / 9.4; random 3 * 10^6 19.6 / 9.9 / 44.1 / 26.6 / 4.8 against 29.7 / 6.0 / 29.4; a level of
// 120 k (with its compaction) 4.5 / 6.7 / 10.2 / 4.2 against 4.7 / - / 9.9 / 4.1.
// Recorded sorts of up to BS_LARGE_N keys still count, scatter and rank.  That is not the faster way: replayed, us, against split and
// merge, 33 k 23.0 / 20.0, 120 k 27.8 / 22.2, 240 k 36.6 / 27.3, 524 k 45.8 / 43.6, 599 k 57 / 33; 64-bit keys 120 k 30.2 / 23.3, 400 k
// 46.6 / 47.9 (up to 14 k the same).
constexpr int BS_MT = 1024;        // merge threads
constexpr int BS_SPLIT_KPT = 12;   // keys per split thread at most
constexpr int BS_RANK_SOLO_N = 400000;
constexpr int BS_NSUB = 4096;      // second split's bins
constexpr int BS_CROWDED = 128;    // keys of a second bin beyond which all are split once more (see order_crowded)
constexpr int BS_ARRIVE = 16, BS_ARRIVE_PITCH = 32;  // counters of the workgroups that have read the totals, on lines of their own, and one more
constexpr int BS_MAX_SPLIT = 1024; // split workgroups
static_assert(BS_MAX_BIN / 2 <= 8 * BS_MT, "two rounds of bins where there are totals (up to 8192)");
static_assert(BS_NSUB == 4 * BS_MT && BS_MAX_SPLIT == BS_MT, "bins and regions per thread");

// Inclusive sum over the lanes of a wave.
__device__ inline int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // lane 15 of rows 0 and 2 to the row behind
  return x + __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // lane 31 to rows 2 and 3
}
// Exclusive sum over a workgroup of WAVES waves; *total is that of all.  `sums` is free again after the workgroup's next barrier.
template <int WAVES>
__device__ inline int block_scan(int v, int* sums, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = wave_scan(v);
  if (lane == 63) sums[wave] = x;
  __syncthreads();
  const int s = wave_scan(lane < WAVES ? sums[lane] : 0);
  *total = __builtin_amdgcn_readlane(s, WAVES - 1);
  const int before = __shfl(s, max(wave - 1, 0), 64);
  return x - v + (wave > 0 ? before : 0);
}

// A region's elements: 64-bit records (key, source index) for 32-bit keys of coordinates; keys, with the source indices in an
// array of their own, for 64-bit ones; keys alone for levels.
template <typename KeyT, bool DEDUP>
struct BsForm {
  static constexpr bool REC = !DEDUP && sizeof(KeyT) == 4, ROWS = !DEDUP && sizeof(KeyT) == 8;
  using Elem = std::conditional_t<REC, uint64_t, KeyT>;
  __device__ static KeyT key(Elem e) { return static_cast<KeyT>(REC ? static_cast<uint64_t>(e) >> 32 : e); }
};
constexpr int bs_off_pitch(int n_bin) { return n_bin + 8; }
// LDS of the split kernel: two bins' counts to a word, the region, and (ROWS) its keys' places in the share.
template <typename KeyT, bool DEDUP>
size_t bs_split_lds(int n_bin, int per) {
  using F = BsForm<KeyT, DEDUP>;
  return size_t(std::max(n_bin / 2, 4) + 4) * 4 + size_t(per) * (sizeof(typename F::Elem) + (F::ROWS ? 2 : 0));
}

template <typename KeyT, bool DEDUP, int KPT, bool ADD, typename Level>
__device__ inline void bs_split(const Level& src, int64_t n, int per, int shift, int n_bin,
                                typename BsForm<KeyT, DEDUP>::Elem* __restrict__ recs, int32_t* __restrict__ rows, uint16_t* __restrict__ off,
                                int32_t* __restrict__ tot) {
  using F = BsForm<KeyT, DEDUP>;
  using Elem = typename F::Elem;
  extern __shared__ __align__(16) unsigned bs_lds[];
  __shared__ int sums[BS_WIDE / 64];
  unsigned* hist = bs_lds;
  const int n_words = n_bin / 2;
  Elem* stage = reinterpret_cast<Elem*>(bs_lds + max(n_words, 4) + 4);  // (one more start behind the last bin's)
  uint16_t* place = reinterpret_cast<uint16_t*>(stage + per);
  const int t = threadIdx.x;
  const int64_t lo = int64_t(blockIdx.x) * per, hi = min<int64_t>(n, lo + per);
  typename Level::Raw raw[KPT];
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * BS_WIDE < per) raw[u] = src.load(min<int64_t>(lo + u * BS_WIDE + t, hi - 1));
  for (int b = t; b < n_words; b += BS_WIDE) hist[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * BS_WIDE < per) Level::pin(raw[u]);
  bool bad = false;
  KeyT key[KPT];
  int at[KPT];  // bin << 16 | place among the share's keys of the bin, or -1
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * BS_WIDE < per) {
      bool bad_u = false;
      key[u] = src.key(raw[u], bad_u);
      at[u] = -1;
      if (lo + u * BS_WIDE + t < hi) {
        bad |= bad_u;
        if (!src.skip(raw[u], key[u])) {
          const int bin = bs_bin(key[u], shift, n_bin), half = 16 * (bin & 1);
          at[u] = (bin << 16) | static_cast<int>((atomicAdd(&hist[bin >> 1], 1u << half) >> half) & 0xffffu);
        }
      }
    }
  src.report(bad);
  __syncthreads();
  // starts of the bins inside the region
  off += int64_t(blockIdx.x) * bs_off_pitch(n_bin);
  constexpr int WPT = BS_MAX_BIN / 2 / BS_WIDE;
  const int wpt = max(n_words / BS_WIDE, 1), w0 = t * wpt;
  unsigned c[WPT];
  int sum = 0;
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    c[j] = j < wpt && w0 < n_words ? hist[w0 + j] : 0u;
    sum += static_cast<int>((c[j] & 0xffffu) + (c[j] >> 16));
  }
  int total;
  unsigned run = block_scan<BS_WIDE / 64>(sum, sums, &total);
#pragma unroll
  for (int j = 0; j < WPT; ++j)
    if (j < wpt && w0 < n_words) {
      const unsigned a = c[j] & 0xffffu, b = c[j] >> 16;
      const unsigned starts = run | ((run + a) << 16);
      hist[w0 + j] = starts;
      reinterpret_cast<unsigned*>(off)[w0 + j] = starts;
      run += a + b;
    }
  if (t == 0) {
    off[n_bin] = static_cast<uint16_t>(total);
    hist[n_words] = static_cast<unsigned>(total);
  }
  __syncthreads();
  if constexpr (ADD) {  // (lane next to lane: an instruction's additions then meet in few lines of memory)
    for (int w = t; w < n_words; w += BS_WIDE) {
      const unsigned here = hist[w], next = hist[w + 1];
      const int a = static_cast<int>((here >> 16) - (here & 0xffffu)), b = static_cast<int>((next & 0xffffu) - (here >> 16));
      if (a) __hip_atomic_fetch_add(tot + 2 * w, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (b) __hip_atomic_fetch_add(tot + 2 * w + 1, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * BS_WIDE < per && at[u] >= 0) {
      const int bin = at[u] >> 16, to = static_cast<int>((hist[bin >> 1] >> (16 * (bin & 1))) & 0xffffu) + (at[u] & 0xffff);
      if constexpr (F::REC) stage[to] = (uint64_t(key[u]) << 32) | static_cast<uint32_t>(lo + u * BS_WIDE + t);
      else stage[to] = key[u];
      if constexpr (F::ROWS) place[to] = static_cast<uint16_t>(u * BS_WIDE + t);
    }
  __syncthreads();
  for (int i = t; i < total; i += BS_WIDE) {
    recs[lo + i] = stage[i];
    if constexpr (F::ROWS) rows[lo + i] = static_cast<int32_t>(lo) + place[i];
  }
}

// (recorded sorts)
template <typename KeyT, bool ADD, typename Level>
__device__ inline void bs_count(const Level& src, int64_t n, int per, int shift, int n_bin, KeyT* __restrict__ keys0,
                                int32_t* __restrict__ table, int32_t* __restrict__ tot) {
  extern __shared__ __align__(16) unsigned bs_lds[];
  int* hist = reinterpret_cast<int*>(bs_lds);  // [n_bin]
  for (int b = threadIdx.x; b < n_bin; b += BS_WIDE) hist[b] = 0;
  __syncthreads();
  const int64_t lo = int64_t(blockIdx.x) * per, hi = min<int64_t>(n, lo + per);
  bool bad = false;
  // four rows per thread and pass, fetched before any of them is turned into a key
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += 4 * BS_WIDE) {
    typename Level::Raw raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[u] = src.load(min<int64_t>(i0 + u * BS_WIDE, hi - 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) Level::pin(raw[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      bool bad_u = false;
      const KeyT key = src.key(raw[u], bad_u);
      if (i0 + u * BS_WIDE < hi) {
        bad |= bad_u;
        keys0[i0 + u * BS_WIDE] = key;
        if (!src.skip(raw[u], key)) atomicAdd(&hist[bs_bin(key, shift, n_bin)], 1);
      }
    }
  }
  src.report(bad);
  __syncthreads();
  table += int64_t(blockIdx.x) * n_bin;
  if constexpr (ADD) {
    for (int b0 = threadIdx.x; b0 < n_bin; b0 += 4 * BS_WIDE) {
      int c[4], at[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) c[u] = b0 + u * BS_WIDE < n_bin ? hist[b0 + u * BS_WIDE] : 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c[u]) at[u] = __hip_atomic_fetch_add(tot + b0 + u * BS_WIDE, c[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c[u]) table[b0 + u * BS_WIDE] = at[u];  // (the scatter pass uses the others as little)
    }
  } else {
    for (int b = threadIdx.x; b < n_bin; b += BS_WIDE) table[b] = hist[b];
  }
}
// ---------------------------------------------------------------- count
// First launch of a sort.  KPT > 0: split (KPT keys per thread at most); `out` is the regions, `table` their rows of bin starts, `rows`
// the source indices where they are apart, and `arrived` is cleared for the merge.  KPT = 0 (recorded sorts): `out` is the keys as
// they come and `table` rows of counts, or with ADD of what their addition to the totals returned.
// ADD: the counts go to the bins' totals (zero before), in whatever order the workgroups come; 4096 bins and 30 workgroups with
// keys in all of them take 1.7 us, fewer bins are hit the shorter a workgroup's share is.
template <typename KeyT, typename Src, bool DEDUP, int KPT, bool ADD>
__global__ __launch_bounds__(BS_WIDE) void bs_count_kernel(const Src srcs, int64_t n, int per, int shift, int n_bin, void* out,
                                                           void* table, size_t ws_pitch, int32_t* tot, size_t tot_pitch, int32_t* rows,
                                                           int32_t* arrived) {
  const auto src = srcs.level(blockIdx.y);
  if constexpr (KPT > 0) {
    if (arrived && blockIdx.x == 0 && threadIdx.x <= BS_ARRIVE) arrived[threadIdx.x * BS_ARRIVE_PITCH] = 0;
    bs_split<KeyT, DEDUP, KPT, ADD>(src, n, per, shift, n_bin, level_ws(static_cast<typename BsForm<KeyT, DEDUP>::Elem*>(out), ws_pitch), rows,
                                    level_ws(static_cast<uint16_t*>(table), ws_pitch), ADD ? level_ws(tot, tot_pitch) : nullptr);
  } else {
    bs_count<KeyT, ADD>(src, n, per, shift, n_bin, static_cast<KeyT*>(out), static_cast<int32_t*>(table), tot);
  }
}
// Clears the totals where they are not kept cleared.
__global__ __launch_bounds__(BS_THREADS) void bs_clear_kernel(int32_t* __restrict__ tot, int n_bin) {
  const int b = blockIdx.x * BS_THREADS + threadIdx.x;
  if (b < n_bin) tot[b] = 0;
}

// The bins of merging workgroup p: from bin `first` on, which starts at sorted position `start`, to bin `last`, which ends at `end` and is
// not empty.  A workgroup whose `start` lies behind its positions, in a bin of an earlier one, has none.  `lead` is where the bin starts that
// ends at `start` (if that is not the workgroup's first position), `tail` where `last` does.
struct BsShare {
  int32_t first, start, lead, last, end, tail;
};

// 128 bins per workgroup; a wave sums a sixteenth of the table's rows, 256 bytes at a time.
constexpr int BS_START_BINS = 128;
__global__ __launch_bounds__(BS_WIDE) void bs_starts_kernel(const uint16_t* __restrict__ off, int n_wg, int n_bin, int q, int n_share,
                                                            BsShare* __restrict__ share, int32_t* __restrict__ n_kept, size_t ws_pitch) {
  off = level_ws(off, ws_pitch);
  share = level_ws(share, ws_pitch);
  n_kept = level_ws(n_kept, ws_pitch);
  constexpr int WAVES = BS_WIDE / 64;
  __shared__ int part[WAVES][BS_START_BINS + 2];
  __shared__ int tail[WAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, f0 = blockIdx.x * BS_START_BINS, f1 = min(f0 + BS_START_BINS, n_bin);
  const int pitch = bs_off_pitch(n_bin), col = min(f0 + 2 * lane, n_bin);
  int a = 0, b = 0, e = 0, all = 0;  // where bins f0 + 2 lane, the next one and f1 start, and the number of keys
#pragma unroll 8
  for (int w = wave; w < n_wg; w += WAVES) {
    const uint16_t* row = off + int64_t(w) * pitch;
    const unsigned v = *reinterpret_cast<const unsigned*>(row + col);
    a += static_cast<int>(v & 0xffffu);
    b += static_cast<int>(v >> 16);
    e += row[f1];
    all += row[n_bin];
  }
  part[wave][2 * lane] = a;
  part[wave][2 * lane + 1] = b;
  if (lane == 0) part[wave][BS_START_BINS] = e, tail[wave] = all;
  __syncthreads();
  const int j = threadIdx.x, f = f0 + j;
  if (j > BS_START_BINS) return;  // (two waves and a lane stay)
  int s = 0, total = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    s += part[w][j];
    total += tail[w];
  }
  if (f < f1) {
    int end = 0;
    const int behind = f + 1 < f1 ? j + 1 : BS_START_BINS;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) end += part[w][behind];
    if (f == 0) share[0].first = 0, share[0].start = 0, share[0].lead = 0, *n_kept = total;
    if (s < end) {  // not empty
      const int p = s / q;
      if (end >= (p + 1) * q || end == total) share[p].last = f, share[p].end = end, share[p].tail = s;
      for (int p1 = p + 1; p1 < n_share && p1 * q <= end; ++p1) share[p1].first = f + 1, share[p1].start = end, share[p1].lead = s;
    }
  }
}

// ---------------------------------------------------------------- merge
// Where a workgroup's bins start: from the bins' totals, from the sums of the table's columns (few regions, where there are no
// totals), or as bs_starts_kernel has left them.
enum { BS_TOTALS = 0, BS_TABLE = 1, BS_STARTS = 2 };
template <typename KeyT, bool DEDUP>
struct MergeArgs {
  const typename BsForm<KeyT, DEDUP>::Elem* recs;
  const int32_t* rows;
  const uint16_t* off;
  int n_wg, per, shift, n_bin, q, n, used_bits;
  int32_t* tot;  // BS_TOTALS
  size_t tot_pitch;
  int clear;          // whether the totals are to be cleared (pack; levels: by the last kernel)
  int32_t* arrived;   // zeros (from the split kernel)
  const BsShare* share;  // BS_STARTS
  int32_t* n_kept;
  KeyT* out_k;        // pack: the sorted keys; levels: the distinct ones, those of workgroup p from out_at[p] on
  int32_t* out_v;
  int32_t *out_at, *out_n;
  size_t ws_pitch;
};

// A kernel's only argument, to be loaded anew where this stands.
template <typename Args>
__device__ inline const Args& bs_args_anew(const Args&) {
  using P = const Args __attribute__((address_space(4)))*;
  P p = (P)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Args*)p;
}

// The part of a workgroup's LDS work that does not depend on where the keys come from: `count` keys (element u * BS_MT + t in
// k[u], source indices in v[u] where they are apart) are put in order in L.key (L.row).  Their second bins are (key - base) >> ss,
// below BS_NSUB; a key above lim (of a rejected row) has lim's, one below base (see bs_merge_kernel) base's.  L.hist is zero before.
template <typename KeyT, bool DEDUP, int KPT>
struct BsOrder {
  using F = BsForm<KeyT, DEDUP>;
  using Elem = typename F::Elem;
  static constexpr int CAP = KPT * BS_MT, WAVES = BS_MT / 64;
  static_assert(CAP <= BS_NSUB && BS_NSUB <= 1 << 12, "a place for every key, and their numbers in 12 bits");
  static constexpr int VEC = 16 / sizeof(Elem);  // keys of a 16-byte read
  using Vec = Elem __attribute__((ext_vector_type(VEC)));
  struct Lds {
    __align__(16) Elem key[CAP + 8];
    int32_t row[F::ROWS ? CAP : 1];
    __align__(16) int hist[BS_NSUB + 4];
    int sums[WAVES];
    int seg[64];
    int32_t pre[BS_MAX_SPLIT];
    int32_t src[BS_MAX_SPLIT];
    int first, start, lead, last, end, tail, wave_last[WAVES];
    int taken, done, crowded;
  };
  // A value that all lanes have, to a scalar register: 32-bit keys leave room there, and by them two workgroups share a CU.
  __device__ static int uniform(int v) { return sizeof(KeyT) == 4 ? __builtin_amdgcn_readfirstlane(v) : v; }
  __device__ static void clear(Lds& L) {
    reinterpret_cast<int4*>(L.hist)[threadIdx.x] = make_int4(0, 0, 0, 0);
    if (threadIdx.x == 0) L.crowded = 0;
  }
  // exclusive sums of the second bins' counts in place
  __device__ static void scan(Lds& L) {
    int4* h = reinterpret_cast<int4*>(L.hist) + threadIdx.x;
    const int4 c = *h;
    if (max(max(c.x, c.y), max(c.z, c.w)) > BS_CROWDED) L.crowded = 1;
    int total;
    const int x = block_scan<WAVES>(c.x + c.y + c.z + c.w, L.sums, &total);
    *h = make_int4(x, x + c.x, x + c.x + c.y, x + c.x + c.y + c.z);
    if (threadIdx.x == 0) L.hist[BS_NSUB] = total;
  }
  template <bool AGAIN>
  __device__ static void order(Lds& L, Elem (&k)[KPT], int32_t (&v)[KPT], int count, KeyT base, KeyT lim, int ss, const int t) {
    auto second = [&](Elem e) { return static_cast<int>((min(max(F::key(e), base), lim) - base) >> ss); };
    int r[KPT];
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) r[u] = atomicAdd(&L.hist[second(k[u])], 1);
    __syncthreads();
    scan(L);
    __syncthreads();
    if constexpr (AGAIN) {
      if (__builtin_expect(L.crowded, 0)) {
        order_crowded(L, k, v, r, count, base, lim, ss, t);
        return;
      }
    }
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) {
        const int at = L.hist[second(k[u])] + r[u];
        L.key[at] = k[u];
        if constexpr (F::ROWS) L.row[at] = v[u];
      }
    if (t < 8) L.key[count + t] = ~Elem(0);
    __syncthreads();
    // From here on a thread has the keys of its places: the lanes of a wave then look at the same few second bins, of which
    // every lane reads the same keys.  Those in front of its bin are smaller and those behind it larger, so whole vectors are counted.
    int d[KPT];
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
      const int at = u * BS_MT + t;
      if (at < count) {
        k[u] = L.key[at];
        if constexpr (F::ROWS) v[u] = L.row[at];
        const int b = second(k[u]), lo = L.hist[b] & -VEC, hi = L.hist[b + 1];
        int c = lo;
#pragma unroll 1
        for (int s = lo; s < hi; s += 8) {
          Vec e[8 / VEC];
#pragma unroll
          for (int x = 0; x < 8 / VEC; ++x) e[x] = reinterpret_cast<const Vec*>(L.key + s)[x];
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const Elem o = e[x / VEC][x % VEC];
            c += o < k[u] || (!F::REC && o == k[u] && s + x < at) ? 1 : 0;
          }
        }
        d[u] = c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) {
        L.key[d[u]] = k[u];
        if constexpr (F::ROWS) L.row[d[u]] = v[u];
      }
    __syncthreads();
  }
  // The rest of order() where a second bin has many keys: every one is split once more, into as many places as it has keys, by where a
  // key lies between its bounds.  A key is compared with all of its second bin, and these cover the workgroup's whole range of bins:
  // where that is long and mostly empty (in front of a voxel that lies far away, between a LiDAR cloud's rings), a few of them hold
  // what there is, up to a thousand keys, and one workgroup took longer than all others.  us of pack + sort without / with: 300 k in a box beside one far
  // voxel 34.1 / 18.5, with 64-bit keys 51.3 / 20.4, LiDAR 200 k (shares of 512 positions) 17.9 / 16.5, 260 k 30.8 / 21.3, 310 k 45.7 / 23.0, with 64-bit
  // keys 71.7 / 27.0; a level with its map, LiDAR 310 k 45.6 / 36.3, 350 k 52.3 / 36.9; clouds without such bins the same (random 500 k 24.7 / 24.6).
  // Not for the bins that several workgroups share (crowd): with it there the kernel would not keep its registers.
  __device__ static void order_crowded(Lds& L, Elem (&k)[KPT], int32_t (&v)[KPT], int (&r)[KPT], int count, KeyT base, KeyT lim, int ss, int t) {
    asm volatile("" : "+v"(t));  // (what is derived from it is not to be kept in registers from before)
    const int cut = max(ss - 20, 0);  // (20 bits of the key and 12 of the count)
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) {
        const KeyT d = min(max(F::key(k[u]), base), lim) - base;
        const int b = static_cast<int>(d >> ss), lo = L.hist[b];
        const uint32_t low = static_cast<uint32_t>((d & ((KeyT(1) << ss) - 1)) >> cut), n = L.hist[b + 1] - lo;
        r[u] = lo + static_cast<int>((low * n) >> (ss - cut));
      }
    __syncthreads();
    clear(L);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) r[u] |= atomicAdd(&L.hist[r[u]], 1) << 16;  // (place | which of its keys)
    __syncthreads();
    scan(L);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) L.key[L.hist[r[u] & 0xffff] + (r[u] >> 16)] = k[u];
    if (t < 8) L.key[count + t] = ~Elem(0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) {
        const int first = L.hist[r[u] & 0xffff], at = first + (r[u] >> 16), lo = first & -VEC, hi = L.hist[(r[u] & 0xffff) + 1];
        int c = lo;
#pragma unroll 1
        for (int s = lo; s < hi; s += 8) {
          Vec e[8 / VEC];
#pragma unroll
          for (int x = 0; x < 8 / VEC; ++x) e[x] = reinterpret_cast<const Vec*>(L.key + s)[x];
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const Elem o = e[x / VEC][x % VEC];
            c += o < k[u] || (!F::REC && o == k[u] && s + x < at) ? 1 : 0;
          }
        }
        r[u] = c;
      }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < count) {
        L.key[r[u]] = k[u];
        if constexpr (F::ROWS) L.row[r[u]] = v[u];
      }
    __syncthreads();
  }
  // The ordered keys leave: to `at` on; returns how many (levels: the distinct ones).
  __device__ static int store(Lds& L, const MergeArgs<KeyT, DEDUP>& a, KeyT* out_k, int count, int at, const int t) {
    if constexpr (!DEDUP) {
#pragma unroll
      for (int u = 0; u < KPT; ++u) {
        const int i = u * BS_MT + t;
        if (i < count) {
          const Elem e = L.key[i];
          out_k[at + i] = F::key(e);
          if (a.out_v) a.out_v[at + i] = F::ROWS ? L.row[i] : static_cast<int32_t>(e);
        }
      }
      return count;
    } else {
      const int lane = t & 63, wave = t >> 6;
      unsigned long long head[KPT];
#pragma unroll
      for (int u = 0; u < KPT; ++u) {
        const int i = u * BS_MT + t;
        head[u] = __ballot(i < count && (i == 0 || L.key[i] != L.key[max(i, 1) - 1]));
        if (lane == 0) L.seg[u * WAVES + wave] = __popcll(head[u]);
      }
      static_assert(KPT * WAVES <= 64, "a wave sums the segments");
      __syncthreads();
      const int c = lane < KPT * WAVES ? L.seg[lane] : 0, x = wave_scan(c);
      const int distinct = __builtin_amdgcn_readlane(x, 63);
#pragma unroll
      for (int u = 0; u < KPT; ++u) {
        const int before = __shfl(x - c, u * WAVES + wave, 64);
        if ((head[u] >> lane) & 1ull) out_k[at + before + __popcll(head[u] & ((1ull << lane) - 1ull))] = L.key[u * BS_MT + t];
      }
      return distinct;
    }
  }
  // Bins f0 .. f1, which start at sorted position s: one shared between workgroups, or others of a workgroup whose keys do not fit the LDS
  // together (see bs_merge_kernel).  This workgroup puts those of their second bins in order that start among positions x .. stop - 1 (x is s or its
  // first position).  A second bin of more than `most` keys is split again, by the next twelve bits; where nothing
  // is left to split its keys are equal, and are taken by their source indices, or (levels) all but one dropped by the workgroup they start at.
  // Every level reads the bins once to count, and what is taken is picked out in one more pass: no workgroup waits for another, but keys in
  // one bin are read as often as it has workgroups.  us of pack + sort, and of a level with its map, in brackets where the bin's owner
  // sorted it alone, reading it again for each 2048 keys (64-bit keys; spread over the bins 120 k voxels take 15 and 25):
  // a wall of 3 k in 20 k voxels, one plane of 12/12/8 bits in 32-bit keys, 20, 30 (34, 50); of 20 k in 120 k 28, 41 (338, 389);
  // 20 k voxels and an outlier, all in one bin, 34, 38 (355, 441); 120 k 80, 128 (10 983, 12 490); 3 * 10^6 1660, 2680; in two bins by x
  // 120 k 82, 89 (12 890, 10 370); 600 k 650, 275; 3 * 10^6 8100, 12 300.
  // Returns the number of keys that left; the first went to *at.
  __device__ __attribute__((always_inline)) static int crowd(Lds& L, const MergeArgs<KeyT, DEDUP>& args, int f0, int f1, int s, int x, int stop,
                                                             int kept, int* at) {
    int t = threadIdx.x;  // (what is derived from it is not to be kept in registers for other trips)
    asm volatile("" : "+v"(t));
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    __syncthreads();
    if (t < args.n_wg) {
      const uint16_t* row = (DEDUP ? level_ws(args.off, args.ws_pitch) : args.off) + int64_t(t) * bs_off_pitch(args.n_bin);
      const int from = min<int>(row[f0], args.per);  // (as in bs_merge_kernel)
      L.src[t] = t * args.per + from;
      L.pre[t] = min(row[f1 + 1] - from, args.per - from);
    }
    auto log2_up = [](unsigned n) { return n > 1 ? 32 - __clz(n - 1) : 0; };
#pragma unroll 1
    while (x < stop) {
      const auto& a = bs_args_anew(args);  // (kept in scalar registers over all of this, the arguments would not fit)
      const int most = CAP - a.q;
      const bool over = f1 == a.n_bin - 1 && a.used_bits < int(8 * sizeof(KeyT));  // all-ones keys as in bs_merge_kernel
      const KeyT base = KeyT(f0) << a.shift, lim = over ? KeyT(f1 + 1) << a.shift : ~KeyT(0);
      // all keys of the bins, a wave to a piece, four loads in flight: fn(key, its place in the regions, whether there is one)
      auto each = [&](auto fn) __attribute__((always_inline)) {
#pragma unroll 1
        for (int w = wave; w < a.n_wg; w += WAVES) {
          const int len = __builtin_amdgcn_readfirstlane(L.pre[w]), src = __builtin_amdgcn_readfirstlane(L.src[w]);
#pragma unroll 1
          for (int i0 = 0; i0 < len; i0 += 256) {
            Elem e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = (DEDUP ? level_ws(a.recs, a.ws_pitch) : a.recs)[src + min(i0 + 64 * u + lane, len - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) fn(e[u], src + i0 + 64 * u + lane, i0 + 64 * u + lane < len);
          }
        }
      };
      KeyT low = base;   // the second bins are [low, low + 4096 << sh), from position ns on, or with `by_row` the rows of key `low`
      uint32_t row0 = 0;
      bool by_row = false;
      int sh = max(0, a.shift + log2_up(f1 + 1 - f0 + (over ? 1 : 0)) - 12), ns = s;
#pragma unroll 1
      for (;;) {
        auto second = [&](Elem e, int place, bool ok) __attribute__((always_inline)) {  // second bin, or -1
          const KeyT key = min(F::key(e), lim);
          if (!ok || key < low) return -1;
          KeyT d = key - low;
          if (!DEDUP && by_row) {
            uint32_t row;
            if constexpr (F::ROWS) row = static_cast<uint32_t>(a.rows[place]);
            else row = static_cast<uint32_t>(e);
            if (d != 0 || row < row0) return -1;
            d = row - row0;
          }
          d >>= sh;
          return d < KeyT(BS_NSUB) ? static_cast<int>(d) : -1;
        };
        __syncthreads();
        clear(L);
        __syncthreads();
        each([&](Elem e, int place, bool ok) __attribute__((always_inline)) {
          const int b = second(e, place, ok);
          const unsigned long long some = __ballot(b >= 0);
          if (some == 0ull) return;
          const int head = __builtin_ctzll(some);
          if (__ballot(b == __builtin_amdgcn_readlane(b, head)) == some) {  // (crowded keys: additions to one place come one by one)
            if (lane == head) atomicAdd(&L.hist[b], __popcll(some));
          } else if (b >= 0) {
            atomicAdd(&L.hist[b], 1);
          }
        });
        __syncthreads();
        scan(L);
        if (t == 0) L.taken = 0;
        __syncthreads();
        auto starts = [&](int b) __attribute__((always_inline)) { return ns + uniform(L.hist[b]); };
        const int ne = min(starts(BS_NSUB), a.n);
        if (x >= ne) return kept;  // (totals that are not the regions': no trip but gets further, or ends here)
        static_assert(BS_NSUB == 64 * 64, "two steps of a wave");
        auto holder = [&](int pos) __attribute__((always_inline)) {  // the second bin that holds position pos
          const int b = 64 * (63 - __builtin_clzll(__ballot(ns + L.hist[64 * lane] <= pos)));
          return b + 63 - __builtin_clzll(__ballot(ns + L.hist[b + lane] <= pos));
        };
        int b = holder(x), bs = starts(b), be = starts(b + 1);
        if (bs < x && be - bs <= most) {  // an earlier workgroup's
          x = be;
          if (x >= min(stop, ne)) break;
          b = holder(x), bs = x, be = starts(b + 1);
        }
        if (be - bs > most) {
          ns = bs;
          if (by_row) row0 += static_cast<uint32_t>(b) << sh;
          else low += KeyT(b) << sh;
          if (sh > 0) {
            sh = max(0, sh - 12);
            continue;
          }
          if constexpr (!DEDUP) {  // equal keys
            if (by_row) return kept;  // (as above: no row occurs twice)
            by_row = true;
            sh = max(0, log2_up(a.n_wg * a.per) - 12);
            continue;
          } else {
            if (bs == x) {
              if (kept == 0) *at = x;
              each([&](Elem e, int place, bool ok) __attribute__((always_inline)) {
                if (ok && min(F::key(e), lim) == low) level_ws(a.out_k, a.ws_pitch)[*at + kept] = F::key(e);  // (one value)
              });
              ++kept;
            }
            x = be;
            break;
          }
        }
        int b1 = holder(min(stop, ne) - 1);  // (not empty)
        if (starts(b1 + 1) - starts(b1) <= most) ++b1;
        const int x1 = min(starts(b1), ne), count = x1 - x;
        each([&](Elem e, int place, bool ok) __attribute__((always_inline)) {
          const int to_bin = second(e, place, ok);
          const bool mine = to_bin >= b && to_bin < b1;
          const unsigned long long some = __ballot(mine);
          if (some == 0ull) return;
          const int head = __builtin_ctzll(some);
          int to = 0;
          if (lane == head) to = atomicAdd(&L.taken, __popcll(some));
          to = __builtin_amdgcn_readlane(to, head) + __popcll(some & ((1ull << lane) - 1ull));
          if (mine && to < CAP) {
            L.key[to] = e;
            if constexpr (F::ROWS) L.row[to] = a.rows[place];
          }
        });
        __syncthreads();
        Elem k[KPT] = {};
        int32_t v[KPT] = {};
        int tt = t;  // (as t)
        asm volatile("" : "+v"(tt));
#pragma unroll
        for (int u = 0; u < KPT; ++u)
          if (u * BS_MT + tt < count) {
            k[u] = L.key[u * BS_MT + tt];
            if constexpr (F::ROWS) v[u] = L.row[u * BS_MT + tt];
          }
        clear(L);
        __syncthreads();
        order<false>(L, k, v, count, by_row ? low : low + (KeyT(b) << sh), lim, by_row ? 0 : max(0, sh + log2_up(b1 - b) - 12), tt);
        if (kept == 0) *at = x;
        kept += store(L, a, DEDUP ? level_ws(a.out_k, a.ws_pitch) : a.out_k, count, DEDUP ? *at + kept : x, tt);
        x = x1;
        break;
      }
    }
    return kept;
  }
};

// (32-bit keys: two workgroups to a CU, for which a wave may have 64 vector and 80 scalar registers; with one, 3 * 10^6 keys 28 -> 39 us,
// 150 k 16 -> 20 in all)
template <typename KeyT, bool DEDUP, int KPT, int FROM>
__global__ __launch_bounds__(BS_MT, sizeof(KeyT) == 4 ? 8 : 4) void bs_merge_kernel(const MergeArgs<KeyT, DEDUP> a) {
  using O = BsOrder<KeyT, DEDUP, KPT>;
  using F = typename O::F;
  using Elem = typename F::Elem;
  __shared__ typename O::Lds L;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, p = blockIdx.x;
  const auto* recs = DEDUP ? level_ws(a.recs, a.ws_pitch) : a.recs;
  const uint16_t* off = DEDUP ? level_ws(a.off, a.ws_pitch) : a.off;
  KeyT* out_k = DEDUP ? level_ws(a.out_k, a.ws_pitch) : a.out_k;
  const int pitch = bs_off_pitch(a.n_bin), lo = p * a.q, hi = lo + a.q;
  int first, start, lead, last, end, tail, total;  // as in BsShare
  int32_t* tot = nullptr;
  int came = 0;
  if constexpr (FROM == BS_STARTS) {
    const BsShare* share = DEDUP ? level_ws(a.share, a.ws_pitch) : a.share;
    total = *(DEDUP ? level_ws(a.n_kept, a.ws_pitch) : a.n_kept);
    const BsShare s = share[p];
    first = s.first, start = s.start, lead = s.lead, last = s.last, end = s.end, tail = s.tail;
    O::clear(L);
  } else {
    if constexpr (FROM == BS_TOTALS) tot = DEDUP ? level_ws(a.tot, a.tot_pitch) : a.tot;
    // four bins per thread and round, of which there are two at most
    auto fetch = [&](int f0) {
      int4 c = make_int4(0, 0, 0, 0);
      if (f0 < a.n_bin) {
        if constexpr (FROM == BS_TOTALS) {
          c = *reinterpret_cast<const int4*>(tot + f0);
        } else {
          for (int w = 0; w < a.n_wg; ++w) {
            const uint16_t* row = off + int64_t(w) * pitch + f0;
            const int s0 = row[0], s1 = row[1], s2 = row[2], s3 = row[3];
            c.x += s1 - s0, c.y += s2 - s1, c.z += s3 - s2, c.w += row[4] - s3;
          }
        }
      }
      return c;
    };
    int4 c = fetch(4 * t), later = fetch(4 * (BS_MT + t));
    O::clear(L);
    if (t == 0) L.first = 0, L.start = 0, L.lead = 0, L.end = -1;
    total = 0;
#pragma unroll 1
    for (int r0 = 0; r0 < a.n_bin; r0 += 4 * BS_MT) {
      const int f0 = r0 + 4 * t;
      if (r0 > 0) __syncthreads();  // (the sums of the round before have been read)
      const int sum = c.x + c.y + c.z + c.w;
      int here;
      int s = total + block_scan<O::WAVES>(sum, L.sums, &here);
      total += here;
      if ((s < lo && lo <= s + sum) || (s < hi && hi <= s + sum)) {
        const int n4[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int e = s + n4[j];
          if (s < lo && lo <= e) L.first = f0 + j + 1, L.start = e, L.lead = s;
          if (s < hi && hi <= e) L.last = f0 + j, L.end = e, L.tail = s;
          s = e;
        }
      }
      const unsigned long long some = __ballot(sum != 0);
      const int mine = f0 + (c.w ? 3 : c.z ? 2 : c.y ? 1 : 0);
      const int top = __builtin_amdgcn_readlane(mine, some ? 63 - __builtin_clzll(some) : 0);
      if (lane == 0 && (some || r0 == 0)) L.wave_last[wave] = some ? top : 0;
      c = later;
    }
    __syncthreads();
    first = L.first, start = L.start, lead = L.lead, last = L.last, end = L.end, tail = L.tail;
    if (end < 0) {  // the last bins (uniform), not behind this workgroup's positions
      last = 0, end = tail = total;
      for (int w = 0; w < O::WAVES; ++w) last = max(last, L.wave_last[w]);
    }
    // (the totals have been read)
    if (!DEDUP && a.clear && t == 0)
      came = __hip_atomic_fetch_add(a.arrived + (p % BS_ARRIVE) * BS_ARRIVE_PITCH, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  first = O::uniform(first), start = O::uniform(start), lead = O::uniform(lead);
  last = O::uniform(last), end = O::uniform(end), tail = O::uniform(tail), total = O::uniform(total);
  // (Calls that overlap on one workspace leave totals, shares and rows of the table that are not the regions': nothing outside outputs and
  // workspace is touched then, and all loops end.)
  if constexpr (FROM == BS_STARTS && !DEDUP) {
    first = min(max(first, 0), a.n_bin), last = min(max(last, 0), a.n_bin - 1);
    start = max(start, lo), tail = max(tail, start);
  }
  total = min(total, FROM == BS_STARTS ? bs_args_anew(a).n : a.n), end = min(end, total);  // (anew: else the frame of 64-bit levels is not empty)
  // A bin of more keys than the LDS holds is shared: of its second bins a workgroup takes those that start among its positions, lo .. hi - 1.
  // (LiDAR clouds of 120 k voxels have bins of up to 1700 or so: shared from 1536 on, the pass of such a cloud took 56 us in place of 51.)
  // Where the last bin does not fit beside the others it is taken on its own.
  const bool shared_lead = lo < total && start > lo && start - lead > O::CAP;
  const bool none = lo >= total || start >= min(hi, total) || (FROM == BS_STARTS && first > last);
  const bool apart = !none && end - start > O::CAP;
  int W = none ? 0 : end - start;
  int kept = 0, at0 = start;
  if (__builtin_expect(shared_lead || apart, 0)) {
#pragma unroll 1
    for (int part = 0; part < 3; ++part) {
      int f0 = first, f1 = apart ? last - 1 : last, s = start, x = start, stop = none ? start : apart ? tail : end;
      if (part == 0) f0 = f1 = first - 1, s = lead, x = lo, stop = shared_lead ? min(hi, min(start, total)) : lo;
      if (part == 2) f0 = f1 = last, s = x = tail, stop = !apart ? tail : end - tail > O::CAP ? min(hi, total) : end;
      if (x < stop) kept = O::crowd(L, a, f0, f1, s, x, stop, kept, &at0);
    }
  } else if (W > 0) {
    // ---- the pieces of the regions, one per thread
    int from = 0, len = 0;
    if (t < a.n_wg) {
      const uint16_t* row = off + int64_t(t) * pitch;
      from = min<int>(row[first], a.per);
      len = min(max(row[last + 1] - from, 0), a.per - from);
    }
    int all;
    const int pre = block_scan<O::WAVES>(len, L.sums, &all);
    W = min(W, all);
    if (t < a.n_wg) {
      L.pre[t] = pre;
      L.src[t] = t * a.per + from - pre;
    }
    __syncthreads();
    int top = 1;
    while (2 * top < a.n_wg) top *= 2;
    auto place = [&](int i) {  // of element i in the regions: of the last piece that starts at or before it
      int w = 0;
      for (int s = top; s > 0; s >>= 1)
        if (w + s < a.n_wg && L.pre[w + s] <= i) w += s;
      return L.src[w] + i;
    };
    // (the all-ones keys of rejected rows, in the last bin, count as the first key behind it where there is one)
    const bool over = last == a.n_bin - 1 && a.used_bits < int(8 * sizeof(KeyT));
    const KeyT base = KeyT(first) << a.shift, lim = (KeyT(last + 1) << a.shift) - (over ? 0 : 1);
    const unsigned bins = last + 1 - first + (over ? 1 : 0);
    const int ss = max(0, a.shift + (bins > 1 ? 32 - __clz(bins - 1) : 0) - 12);
    Elem k[KPT];
    int32_t v[KPT];
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * BS_MT + t < W) {
        const int at = place(u * BS_MT + t);
        k[u] = recs[at];
        if constexpr (F::ROWS) v[u] = a.rows[at];
      }
    O::template order<true>(L, k, v, W, base, lim, ss, t);
    kept = O::store(L, a, out_k, W, start, t);
  }
  if constexpr (DEDUP) {
    if (t == 0) {
      level_ws(a.out_at, a.ws_pitch)[p] = at0;
      level_ws(a.out_n, a.ws_pitch)[p] = kept;
    }
  }
  if constexpr (FROM == BS_TOTALS && !DEDUP) {
    // Whoever comes last clears the totals for the next sort.  Workgroups are counted in two steps: additions to one place take
    // some 40 ns each (235 workgroups: 9 us).
    if (a.clear) {
      if (t == 0) {
        const int g = p % BS_ARRIVE, n_share = gridDim.x, groups = min(n_share, BS_ARRIVE);
        L.done = came == (n_share - g + BS_ARRIVE - 1) / BS_ARRIVE - 1 &&
                 __hip_atomic_fetch_add(a.arrived + BS_ARRIVE * BS_ARRIVE_PITCH, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == groups - 1;
      }
      __syncthreads();
      if (L.done)
        for (int b = t; b < a.n_bin; b += BS_MT) tot[b] = 0;
    }
  }
}

// Where the levels of a batch go.
template <typename KeyT>
struct LevelOut {
  KeyT* keys[BS_MAX_LEVELS];
  int32_t* count[BS_MAX_LEVELS];
};

// The merging workgroups' distinct keys, one behind the other, and their number.
template <typename KeyT>
__global__ __launch_bounds__(BS_THREADS) void bs_compact_kernel(const KeyT* __restrict__ part, const int32_t* __restrict__ at,
                                                                const int32_t* __restrict__ num, const LevelOut<KeyT> lo, size_t ws_pitch,
                                                                int32_t* tot, size_t tot_pitch, int n_bin) {
  if (tot)  // (kept cleared between sorts)
    for (int b = blockIdx.x * BS_THREADS + threadIdx.x; b < n_bin; b += gridDim.x * BS_THREADS) level_ws(tot, tot_pitch)[b] = 0;
  part = level_ws(part, ws_pitch);
  at = level_ws(at, ws_pitch);
  num = level_ws(num, ws_pitch);
  __shared__ int sums[BS_THREADS / 64];
  const int t = threadIdx.x, p = blockIdx.x, mine = num[p];
  const KeyT* from = part + at[p];
  int before = 0;
  for (int i = t; i < p; i += BS_THREADS) before += num[i];
  block_scan<BS_THREADS / 64>(before, sums, &before);
  KeyT* out = lo.keys[blockIdx.y] + before;
  for (int i = t; i < mine; i += BS_THREADS) out[i] = from[i];
  if (p == int(gridDim.x) - 1 && t == 0) *lo.count[blockIdx.y] = before + mine;
}

// ---------------------------------------------------------------- small levels: one workgroup, one launch
// Fewer than BS_MIN_N keys (the tiny cloud of a unit test, the coarsest levels of a network): the partitioning
// scheme of the large path inside one workgroup and LDS.  The keys are produced (packed or masked) straight into
// LDS and counted into 4096 bins of their top used bits; a scan gives the bin starts; the keys move, with their source
// index, to their bin's range; and every key's final place is its bin's start plus the number of (key, index)
// pairs of the bin that sort before it (the index breaks ties, so equal keys of an invalid cloud still get distinct
// places).  The downsampling form writes the sorted keys back to LDS and keeps the first key of every run of equal
// keys (a scan over the head flags).  One launch of a few microseconds where the large path has three or four and a
// library sort more; nothing but kernels is enqueued, so it can be recorded into a graph.  Work is quadratic in the
// bin sizes: a cloud whose keys all share their top 12 used bits costs n^2 = 16 M comparisons at most.  (1024 bins: 4000 voxels
// of surfaces 15 us, their stride-2 level with its map 29; 4096 bins: 11 and 20.)
constexpr int BS_SMALL_THREADS = 1024;
constexpr int BS_SMALL_BIN_BITS = 12;
constexpr int BS_SMALL_BINS = 1 << BS_SMALL_BIN_BITS;
static_assert(BS_SMALL_BINS == 4 * BS_SMALL_THREADS, "four bins per thread");
constexpr int BS_SMALL_MAX = 4096;  // >= BS_MIN_N - 1
template <typename KeyT, typename Src, bool DEDUP>
__global__ __launch_bounds__(BS_SMALL_THREADS) void bs_small_sort_kernel(const Src srcs, int n, int shift, const LevelOut<KeyT> lo,
                                                                        int32_t* __restrict__ out_v) {
  const auto src = srcs.level(blockIdx.y);
  KeyT* __restrict__ out_k = lo.keys[blockIdx.y];
  __shared__ KeyT sk0[BS_SMALL_MAX], sk1[BS_SMALL_MAX];
  __shared__ int16_t sv1[BS_SMALL_MAX];
  __shared__ __align__(16) int s_cur[BS_SMALL_BINS];  // counts, then every bin's cursor, in the end where the bin ends
  __shared__ int wave_tot[BS_SMALL_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int4* cur4 = reinterpret_cast<int4*>(s_cur) + tid;
  *cur4 = make_int4(0, 0, 0, 0);
  __syncthreads();
  bool bad = false;
  for (int i = tid; i < n; i += BS_SMALL_THREADS) {
    bool bad_i = false;
    const KeyT key = src.key(src.load(i), bad_i);
    bad |= bad_i;
    sk0[i] = key;
    atomicAdd(&s_cur[bs_bin(key, shift, BS_SMALL_BINS)], 1);
  }
  src.report(bad);
  __syncthreads();
  {  // exclusive scan of the bin counts, four bins per thread
    const int4 c = *cur4;
    const int sum = c.x + c.y + c.z + c.w;
    int x = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    int run = x - sum;
    for (int w = 0; w < wave; ++w) run += wave_tot[w];
    *cur4 = make_int4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
  }
  __syncthreads();
  for (int i = tid; i < n; i += BS_SMALL_THREADS) {
    const KeyT key = sk0[i];
    const int p = atomicAdd(&s_cur[bs_bin(key, shift, BS_SMALL_BINS)], 1);
    sk1[p] = key;
    sv1[p] = static_cast<int16_t>(i);
  }
  __syncthreads();
  for (int x = tid; x < n; x += BS_SMALL_THREADS) {
    const KeyT key = sk1[x];
    const int vi = sv1[x];
    const int b = bs_bin(key, shift, BS_SMALL_BINS);
    const int a = b > 0 ? s_cur[b - 1] : 0, e = s_cur[b];
    int r = a;
    int y = a;
    // eight candidates per trip, read before any is compared: one LDS round trip per trip instead of one per key
    // (a bin of the tiny test cloud holds a few hundred keys, and the loop was nine tenths of the kernel)
    for (; y + 8 <= e; y += 8) {
      KeyT ky[8];
      int16_t vy[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        ky[u] = sk1[y + u];
        vy[u] = sv1[y + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) r += (ky[u] < key || (ky[u] == key && vy[u] < vi)) ? 1 : 0;
    }
    for (; y < e; ++y) {
      const KeyT ky = sk1[y];
      r += (ky < key || (ky == key && sv1[y] < vi)) ? 1 : 0;
    }
    if (DEDUP) {
      sk0[r] = key;  // sorted sequence, kept in LDS for the pass below
    } else {
      out_k[r] = key;
      if (out_v) out_v[r] = vi;
    }
  }
  if (!DEDUP) return;
  __syncthreads();
  // distinct keys: thread t owns the run of positions [t * per, (t + 1) * per)
  const int per = (n + BS_SMALL_THREADS - 1) / BS_SMALL_THREADS;
  int cnt = 0;
  for (int u = 0; u < per; ++u) {
    const int i = tid * per + u;
    cnt += (i < n && (i == 0 || sk0[i] != sk0[i - 1])) ? 1 : 0;
  }
  int x = cnt;
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) wave_tot[wave] = x;
  __syncthreads();
  int base = x - cnt, total = 0;
  for (int w = 0; w < BS_SMALL_THREADS / 64; ++w) {
    if (w < wave) base += wave_tot[w];
    total += wave_tot[w];
  }
  for (int u = 0; u < per; ++u) {
    const int i = tid * per + u;
    if (i < n && (i == 0 || sk0[i] != sk0[i - 1])) out_k[base++] = sk0[i];
  }
  if (tid == 0) *lo.count[blockIdx.y] = total;
}

template <typename KeyT, typename Src, bool DEDUP>
static void launch_small_sort(const Src& src, int64_t n, int used_bits, const LevelOut<KeyT>& lo, int n_levels, int32_t* out_v,
                              hipStream_t s) {
  static_assert(BS_SMALL_MAX >= BS_MIN_N - 1, "the small path covers every size below the partitioning sort's");
  const int shift = std::max(0, used_bits - BS_SMALL_BIN_BITS);  // bins = the top used key bits
  hipLaunchKernelGGL((bs_small_sort_kernel<KeyT, Src, DEDUP>), dim3(1, n_levels), dim3(BS_SMALL_THREADS), 0, s, src,
                     static_cast<int>(n), shift, lo, out_v);
}

template <typename KeyT>
static void small_pack_sort_t(const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status, void* keys_out,
                              int32_t* perm_out, hipStream_t s) {
  LevelOut<KeyT> lo{};
  lo.keys[0] = static_cast<KeyT*>(keys_out);
  launch_small_sort<KeyT, SrcPack<KeyT>, false>(SrcPack<KeyT>{coords, pp, status}, n, used_bits, lo, 1, perm_out, s);
}

int small_pack_sort(int key_bits, const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status, void* keys_out,
                    int32_t* perm_out, hipStream_t s) {
  if (key_bits == 32) small_pack_sort_t<uint32_t>(coords, n, pp, used_bits, status, keys_out, perm_out, s);
  else small_pack_sort_t<uint64_t>(coords, n, pp, used_bits, status, keys_out, perm_out, s);
  if (hipGetLastError() != hipSuccess) return set_error(SPC_ERR_HIP, "sort launch failed");
  return SPC_OK;
}

template <typename KeyT>
static void batch_args(const void* keys_in, const LevelJob* jobs, int n_levels, SrcMasks<KeyT>* src, LevelOut<KeyT>* lo) {
  *src = SrcMasks<KeyT>{static_cast<const KeyT*>(keys_in), {}};
  *lo = LevelOut<KeyT>{};
  for (int y = 0; y < n_levels; ++y) {
    src->masks[y] = static_cast<KeyT>(jobs[y].mask);
    lo->keys[y] = static_cast<KeyT*>(jobs[y].keys_out);
    lo->count[y] = jobs[y].count;
  }
}

template <typename KeyT>
static void small_mask_unique_t(const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, hipStream_t s) {
  SrcMasks<KeyT> src;
  LevelOut<KeyT> lo;
  batch_args(keys_in, jobs, n_levels, &src, &lo);
  launch_small_sort<KeyT, SrcMasks<KeyT>, true>(src, n, used_bits, lo, n_levels, nullptr, s);
}

int small_mask_unique(int key_bits, const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, hipStream_t s) {
  if (key_bits == 32) small_mask_unique_t<uint32_t>(keys_in, n, jobs, n_levels, used_bits, s);
  else small_mask_unique_t<uint64_t>(keys_in, n, jobs, n_levels, used_bits, s);
  if (hipGetLastError() != hipSuccess) return set_error(SPC_ERR_HIP, "downsample launch failed");
  return SPC_OK;
}

// ---------------------------------------------------------------- recorded sorts: column scan (above BS_ADD_N keys)
// One thread per four bins: before[w][f] receives the number of keys of bin f held by workgroups
// < w, tot[f] the bin's total.  The loads of 32 table rows are in flight together (16: 1 us more from 500 k keys on).
constexpr int BS_COL_THREADS = 64;
__global__ __launch_bounds__(BS_COL_THREADS) void bs_colscan_kernel(const int32_t* __restrict__ table,
                                                                    int32_t* __restrict__ before, int n_wg, int n_bin,
                                                                    int32_t* __restrict__ tot) {
  constexpr int ROWS = 32;
  const int f0 = (blockIdx.x * BS_COL_THREADS + threadIdx.x) * 4;
  if (f0 >= n_bin) return;  // n_bin is a multiple of 4
  int4 run = make_int4(0, 0, 0, 0);
  for (int w0 = 0; w0 < n_wg; w0 += ROWS) {
    int4 c[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) c[r] = *reinterpret_cast<const int4*>(table + int64_t(min(w0 + r, n_wg - 1)) * n_bin + f0);
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (w0 + r < n_wg) {
        *reinterpret_cast<int4*>(before + int64_t(w0 + r) * n_bin + f0) = run;
        run.x += c[r].x;
        run.y += c[r].y;
        run.z += c[r].z;
        run.w += c[r].w;
      }
  }
  *reinterpret_cast<int4*>(tot + f0) = run;
}

// ---------------------------------------------------------------- recorded sorts: scatter
// Every workgroup scans the bin totals on its own (16 KB; cheaper than one more launch): start
// of bin f, then the workgroup's first position in the bin, and moves its keys, with their source
// index, to their bin's range.
// It also prepares the rank pass: for every BS_PART scattered
// positions the window of whole bins that covers them, and BS_PAD_KEYS all-ones keys behind the last key.
// What bounds it: the scattered stores, of which a CU issues one lane per cycle, so the shares of the workgroups are short
// (see bucket_plan).
// SUM (few workgroups): `before` is the table of counts as the count pass leaves it
// without ADD, and its rows are summed here, which saves the launch that would clear the totals.
template <typename KeyT, bool SUM>
__global__ __launch_bounds__(BS_WIDE) void bs_scatter_kernel(const KeyT* __restrict__ keys0, int64_t n, int per, int shift,
                                                             int n_bin, const int32_t* __restrict__ before,
                                                             const int32_t* __restrict__ tot, KeyT* __restrict__ keys1,
                                                             int32_t* __restrict__ vals1, int2* __restrict__ win) {
  extern __shared__ int lds_bins[];
  int* pos = lds_bins;                    // [n_bin + 1] this workgroup's running position in every bin
  int* bin_start = lds_bins + n_bin + 1;  // [n_bin + 1] where every bin starts
  __shared__ int wave_tot[BS_WIDE / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // a pass takes four keys per thread; the first pass's are requested before the scan, so that they arrive under it
  const int64_t lo = int64_t(blockIdx.x) * per, hi = min<int64_t>(n, lo + per);
  KeyT key[4];
  auto fetch = [&](int64_t i0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = min<int64_t>(i0 + u * BS_WIDE, hi - 1);
      key[u] = keys0[i];
    }
  };
  fetch(lo + threadIdx.x);
  // exclusive scan of the bin totals, four bins per thread and round (one round up to 4096 bins)
  int total = 0;
  for (int r0 = 0; r0 < n_bin; r0 += 4 * BS_WIDE) {
    const int f0 = r0 + t * 4;
    int4 c = make_int4(0, 0, 0, 0), bef = c;
    if (f0 < n_bin) {
      if constexpr (SUM) {
        constexpr int ROWS = 8;  // loads in flight
        const int n_wg = gridDim.x, me = blockIdx.x;
        for (int w = 0; w < n_wg; w += ROWS) {
          int4 row[ROWS];
#pragma unroll
          for (int r = 0; r < ROWS; ++r) row[r] = *reinterpret_cast<const int4*>(before + int64_t(min(w + r, n_wg - 1)) * n_bin + f0);
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const int all = w + r < n_wg ? -1 : 0, mine = w + r < me ? -1 : 0;
            c.x += row[r].x & all, c.y += row[r].y & all, c.z += row[r].z & all, c.w += row[r].w & all;
            bef.x += row[r].x & mine, bef.y += row[r].y & mine, bef.z += row[r].z & mine, bef.w += row[r].w & mine;
          }
        }
      } else {
        c = *reinterpret_cast<const int4*>(tot + f0);
        bef = *reinterpret_cast<const int4*>(before + int64_t(blockIdx.x) * n_bin + f0);
      }
    }
    const int sum = c.x + c.y + c.z + c.w;
    int x = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (r0 > 0) __syncthreads();  // the wave totals of the round before have been read
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    int base = total + x - sum;
    for (int w = 0; w < BS_WIDE / 64; ++w) {
      if (w < wave) base += wave_tot[w];
      total += wave_tot[w];
    }
    if (f0 < n_bin) {
      const int s0 = base, s1 = base + c.x, s2 = s1 + c.y, s3 = s2 + c.z;
      pos[f0] = s0 + bef.x;
      pos[f0 + 1] = s1 + bef.y;
      pos[f0 + 2] = s2 + bef.z;
      pos[f0 + 3] = s3 + bef.w;
      bin_start[f0] = s0;
      bin_start[f0 + 1] = s1;
      bin_start[f0 + 2] = s2;
      bin_start[f0 + 3] = s3;
    }
  }
  if (t == 0) bin_start[n_bin] = total;
  __syncthreads();
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += 4 * BS_WIDE) {
    // all keys of the pass are fetched, then all positions drawn, then everything stored
    bool use[4];
    int p[4];
    if (i0 >= lo + 4 * BS_WIDE) fetch(i0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      SPC_PIN_LOADED(key[u]);
      use[u] = i0 + u * BS_WIDE < hi;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) p[u] = use[u] ? atomicAdd(&pos[bs_bin(key[u], shift, n_bin)], 1) : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (use[u]) {
        keys1[p[u]] = key[u];
        vals1[p[u]] = static_cast<int32_t>(i0 + u * BS_WIDE);
      }
  }
  // Rank windows (see bs_rank_kernel): part p = scattered positions [p * BS_PART, ...) is ranked
  // inside the range of whole bins that covers it.  Parts are dealt round-robin to the workgroups,
  // one per thread: two binary searches over the bin starts in LDS, done last, while the scattered
  // stores drain.
  if (blockIdx.x == 0 && t < BS_PAD_KEYS) keys1[total + t] = ~KeyT(0);  // the rank kernel reads whole steps
  const int part = blockIdx.x + t * gridDim.x;
  if (int64_t(part) * BS_PART < total) {
    const int x0 = part * BS_PART, x1 = min(x0 + BS_PART, total) - 1;
    // last bin whose start is <= x: the (non-empty) bin that holds position x; both searches in step
    int fa = 0, fb = 0;
    for (int step = n_bin >> 1; step > 0; step >>= 1) {
      const int sa = bin_start[fa + step], sb = bin_start[fb + step];
      if (sa <= x0) fa += step;
      if (sb <= x1) fb += step;
    }
    win[part] = make_int2(bin_start[fa], bin_start[fb + 1]);
  }
}

// ---------------------------------------------------------------- recorded sorts: rank
// After the scatter the keys are ordered by bin, unordered inside a bin.  Workgroup p takes the
// BS_PART = 64 keys at scattered positions [p * BS_PART, ...), one per lane, each of its four waves
// a quarter of the comparisons, and ranks each of them inside the window of whole bins that covers those positions (widened to multiples of 32
// positions): every key before the window is smaller and every key behind it larger, so
// window start + (number of window keys that sort before mine) is the key's final position.
// "Sorts before" is (key, scattered position) order, which makes the positions of equal keys
// distinct without any atomics; below and above the workgroup's own 64 positions that is a plain
// <= resp. < on the key.  Every lane of a wave compares its key with the same window key at the same
// time, so the window is read with scalar loads (128 bytes per step, the next step's load in
// flight while the current one is compared) and a comparison is two vector instructions with a
// scalar operand; LDS only carries the four partial counts of a key to the wave that stores.  (Reading the window back from LDS at a wave-uniform address
// was measured four times slower: 16-byte LDS reads of one address by all lanes are not broadcast.)
// Work per key grows with the window, i.e. with the size of the bins involved, but a big bin is
// shared by as many workgroups as it has parts: no workgroup sorts a dense region of the scene
// alone, which is what bounded the compare-exchange network this replaces on the pack + sort path.
// The scatter leaves BS_RANK_STEP all-ones keys behind the last key, so that whole steps can be
// read at the end of the array.
constexpr int BS_RANK_STEP = BS_PAD_KEYS;  // positions; a window is a whole number of steps
// 128 bytes of keys at a wave-uniform address in scalar registers.  The load is issued by hand and
// its arrival awaited by hand, one compare step later: left to the compiler, the load of a step
// ends up right in front of its first use and every step pays the scalar-memory latency.
typedef uint32_t bs_u32x16 __attribute__((ext_vector_type(16)));
struct BsChunk {
  bs_u32x16 lo, hi;
  // (the address is in scalar registers: derived from blockIdx and kernel arguments)
  __device__ void issue(const void* q) {
    asm volatile("s_load_dwordx16 %0, %2, 0x0\n\ts_load_dwordx16 %1, %2, 0x40" : "=&s"(lo), "=&s"(hi) : "s"(q) : "memory");
  }
  // the counters are operands only to keep the compare step that runs under the load in front of the wait
  __device__ void arrive(int (&c)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(lo), "+s"(hi), "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]));
  }
  template <typename KeyT>
  __device__ KeyT key(int q) const {  // q-th key of the chunk, q a compile-time constant after unrolling
    if constexpr (sizeof(KeyT) == 4) return q < 16 ? lo[q] : hi[q - 16];
    else return q < 8 ? (uint64_t(lo[2 * q + 1]) << 32) | lo[2 * q] : (uint64_t(hi[2 * q - 15]) << 32) | hi[2 * q - 16];
  }
};

// keys k[a, b) that sort before (key, x): MODE 0 for positions below the workgroup's own 64 (equal
// keys count), 2 for positions above (they do not), 1 for the own positions (full comparison).
// a and b are multiples of BS_RANK_STEP.
template <int MODE, typename KeyT>
__device__ inline int bs_count_before(const KeyT* __restrict__ k, int a, int b, KeyT key, int x) {
  constexpr int C = 128 / sizeof(KeyT);  // keys per chunk
  static_assert(BS_RANK_STEP % C == 0, "a step of positions is a whole number of chunks");
  int c[4] = {0, 0, 0, 0};
  if (a >= b) return 0;
  auto compare = [&](const BsChunk& ch, int j) {
#pragma unroll
    for (int q = 0; q < C; ++q) {
      const KeyT e = ch.template key<KeyT>(q);
      bool before;
      if (MODE == 0) before = e <= key;
      else if (MODE == 2) before = e < key;
      else before = e < key || (e == key && j + q < x);
      c[q & 3] += before ? 1 : 0;
    }
  };
  BsChunk A, B;
  A.issue(k + a);
  A.arrive(c);
  for (int j = a; j < b; j += 2 * C) {  // the last chunk is fetched once more instead of running past b
    B.issue(k + min(j + C, b - C));
    compare(A, j);
    B.arrive(c);
    if (j + C < b) {
      A.issue(k + min(j + 2 * C, b - C));
      compare(B, j + C);
      A.arrive(c);
    }
  }
  return (c[0] + c[1]) + (c[2] + c[3]);
}

template <typename KeyT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void bs_rank_kernel(const KeyT* __restrict__ keys1, const int32_t* __restrict__ vals1,
                                                             const int2* __restrict__ win, int n, KeyT* __restrict__ out_k,
                                                             int32_t* __restrict__ out_v) {
  static_assert(BS_PART == 64, "one key per lane");
  __shared__ int partial[WAVES][BS_PART];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int part = blockIdx.x, own0 = part * BS_PART;
  const int x = own0 + lane;
  const bool act = x < n;
  const int2 w = win[part];
  const KeyT key = act ? keys1[x] : ~KeyT(0);
  const int32_t val = act && out_v && wave == 0 ? vals1[x] : 0;
  const int n_pad = (n + BS_RANK_STEP - 1) & ~(BS_RANK_STEP - 1);  // positions n .. n_pad - 1 hold all-ones keys
  const int g0 = w.x & ~(BS_RANK_STEP - 1);
  const int g1 = min(max((w.y + BS_RANK_STEP - 1) & ~(BS_RANK_STEP - 1), own0 + BS_PART), n_pad);
  // the window is cut into the part below the own positions, the own positions and the part above;
  // each is shared out among the waves in contiguous quarters (rounded to whole steps)
  const int own1 = min(own0 + BS_PART, g1);
  auto quarter = [&](int a, int b, int& qa, int& qb) {
    const int steps = (b - a) / BS_RANK_STEP, per = (steps + WAVES - 1) / WAVES;
    qa = min(a + wave * per * BS_RANK_STEP, b);
    qb = min(qa + per * BS_RANK_STEP, b);
  };
  int qa, qb;
  quarter(g0, own0, qa, qb);
  int c = bs_count_before<0>(keys1, qa, qb, key, x);
  quarter(own0, own1, qa, qb);
  c += bs_count_before<1>(keys1, qa, qb, key, x);
  quarter(own1, g1, qa, qb);
  c += bs_count_before<2>(keys1, qa, qb, key, x);
  int r = g0 + c;
  if constexpr (WAVES > 1) {
    partial[wave][lane] = c;
    __syncthreads();
    r = g0;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) r += partial[v][lane];
  }
  if (wave == 0 && act) {
    out_k[r] = key;
    if (out_v) out_v[r] = val;
  }
}

// ---------------------------------------------------------------- host
BucketPlan bucket_plan(int64_t n, int used_bits, bool unique) {
  BucketPlan p{};
  p.add = n <= BS_ADD_N;
  // keys per workgroup: short shares spread the work over the chip, long ones are fewer rows for the merge to look into and, for
  // coordinates, which have keys in almost all bins, fewer additions.  us of pack + sort with shares of 1024 / 2048 / 4096: 20 k 11.3 / 11.4,
  // 60 k 13.2 / 12.3, 120 k 16.8 / 14.4 / 13.3, 180 k 21.7 / 16.4 / 14.9, 240 k - / 21.8 / 19.0, 500 k - / 39.3 / 32.0; of a level with its map,
  // whose sorted keys add to few bins: 20 k 18.0 / 19.9, 60 k 20.5 / 20.8, 120 k 22.3 / 23.5 / 24.0, 180 k 27.1 / 28.1 / 28.8, 500 k
  // 53.1 / 48.8 / 48.7.  The lines for coordinates were drawn where they are scattered (recorded sorts: 180 k 25.4 / 26.2 with 2048 / 4096).
  const int share = n <= BS_SHORT_N ? BS_SHORT_SHARE : p.add && (unique || n <= BS_MID_N) ? BS_ADD_SHARE : BS_LONG_SHARE;
  int n_wg = static_cast<int>(std::min<int64_t>(std::max<int64_t>((n + share - 1) / share, 1), p.add ? n : BS_MAX_WG));
  p.per = static_cast<int>(((n + n_wg - 1) / n_wg + BS_WIDE - 1) / BS_WIDE * BS_WIDE);
  p.n_wg = static_cast<int>(std::max<int64_t>((n + p.per - 1) / p.per, 1));
  // About 16 keys per bin of the key space up to 4096 bins: packing descriptors round every field up
  // to whole bits and scenes are far from cubic, so typically a quarter of the bins is populated.
  // Beyond that, more bins only pay where the rank pass of a recorded sort is bound by its comparisons: 8192 bins from 200 k keys,
  // 16384 from 512 k (10^6 keys: rank 51 -> 32 us; 300 k keys with 16384 bins: slower by 2 us for the longer scans).  Split and merge would
  // do with fewer: us with 8192 / 16384 bins, 530 k 21.8 / 26.5, 700 k 25.6 / 28.9, 10^6 29.5 / 33.2, 3 * 10^6 51.0 / 56.4; but fewer are crowded
  // earlier (a level of 3 * 10^6 with its map, 4096 / 8192 / 16384 bins, 262 / 116 / 120; 1.5 * 10^6 in a box beside one far voxel 163 / 83, with a wall of 250 k 168 / 126).
  int fb = 8;
  while (fb < 12 && (int64_t(16) << fb) < n) ++fb;
  if (n > 200000) fb = 13;
  if (n > 524288) fb = 14;
  static_assert(BS_MAX_BIN_BITS >= 14, "bin table sizes");
  fb = std::max(2, std::min(fb, used_bits));
  p.shift = used_bits - fb;
  p.n_bin = 1 << fb;
  return p;
}


namespace {
// The workspace of a recorded sort, and of one in split + merge form (which is nowhere larger; see bucket_sort_ws_bytes).
template <typename KeyT>
struct Ws {
  KeyT *keys0, *keys1;
  int32_t *vals1, *table, *before, *fstart;
  int2* win;
};
template <typename KeyT>
Ws<KeyT> carve(void* ws, int64_t n) {
  const size_t nn = static_cast<size_t>(std::max<int64_t>(n, 1));
  const size_t k = ((nn + BS_PAD_KEYS) * sizeof(KeyT) + 255) / 256 * 256, v = ((nn + BS_PAD_KEYS) * 4 + 255) / 256 * 256;
  char* c = static_cast<char*>(ws);
  Ws<KeyT> w;
  w.keys0 = reinterpret_cast<KeyT*>(c);
  w.keys1 = reinterpret_cast<KeyT*>(c + k);
  w.vals1 = reinterpret_cast<int32_t*>(c + 2 * k);
  w.table = reinterpret_cast<int32_t*>(c + 2 * k + v);
  const BucketPlan cap = bucket_plan(n, 64, true);
  const size_t tbl = (size_t(cap.n_wg) * cap.n_bin + 63) / 64 * 64;
  w.before = w.table + tbl;
  w.fstart = w.before + (cap.add ? 0 : tbl);
  w.win = reinterpret_cast<int2*>(w.fstart + cap.n_bin + 64);  // 8-byte aligned: every part above is a multiple of 256 bytes
  return w;
}

// Split + merge: sizes of both kernels' shares.
// Levels of more keys: wide workgroups merge also where the totals are read (coordinates: above BS_MID_N).  There are a quarter as many then, and
// each reads all totals first; below, they are too few for the chip.  us, narrow / wide:
//   pack + sort   LiDAR 160 k 15.9 / 20.5, 199 k 15.7 / 19.9 (measured before order_crowded), 210 k 20.5 / 22.2, 240 k 20.2 / 21.4, 270 k 37.0 / 21.5, 310 k
//                 38.3 / 22.7, 350 k 26.1 / 23.6, indoor 180 k 18.2 / 17.7, 210 k 19.6 / 19.2, 290 k 25.8 / 21.3, 400 k 29.7 / 25.0, random 180 k 15.9 / 16.2, 210 k 18.4 /
//                 17.8, 290 k 24.4 / 19.7, 400 k 29.7 / 22.3; 64-bit keys, LiDAR 210 k 28.4 / 28.5, 310 k 50.5 / 26.7, indoor 210 k 25.4 / 21.2, random 400 k 41.8 / 25.2
//   a level with its map   LiDAR 240 k 31.7 / 33.8, 290 k 33.1 / 35.0, 310 k 33.4 / 36.2, 350 k 33.8 / 37.6, indoor 250 k 36.2 / 38.6, 290 k 43.3 / 41.2, 320 k 45.8 / 43.5, 400 k
//                 54.4 / 50.1, random 250 k 35.7 / 36.8, 290 k 43.6 / 41.1, 400 k 51.7 / 46.8; 64-bit keys, LiDAR 240 k 37.8 / 36.2, 350 k 42.5 / 41.0, indoor 290 k 53.7 / 46.0
// So the line for levels is where indoor and random scenes cross; LiDAR clouds of 32-bit keys, whose levels hold fewer keys, lose two to four us above it
// (64-bit keys would gain below it already).
// (Bins that do not fit a narrow workgroup: 260 k in three planes 171 / 138, 524 k in four 403 / 189, 300 k in a box beside a voxel so far away that its
// bins are of 2900 keys 51.7 / 19.0, 64-bit keys 71.2 / 21.3; of 1500 20.1 / 18.4.)
constexpr int64_t BS_WIDE_LEVEL_N = 300000;
struct SplitPlan {
  BucketPlan b;
  int q, n_share;  // positions per merging workgroup
  bool wide;       // four keys per merge thread instead of two
};
// Positions per merging workgroup: short shares spread a small cloud over the chip; long ones take longer pieces and read the totals less often.  Split shares are those of bucket_plan (half as long, 120 k 4.8 -> 5.7 us and 240 k 9.2 -> 11.2 for the
// additions).  Above BS_ADD_N a CU gets one as long as 12288 keys last (half as long, with 8192 bins, 3 * 10^6: 65 -> 69 us in all), but none is
// shorter than 4096, so that from 524 289 to a million keys 129 to 245 CUs have one: us in all with shares of at least 2048 / 3072 / 4096,
// 530 k 28.1 / 28.2 / 26.6, 700 k 30.7 / 30.7 / 29.1, 10^6 33.2 / 33.1 / 33.1.
SplitPlan split_plan(int64_t n, int used_bits, bool unique) {
  SplitPlan p{};
  p.b = bucket_plan(n, used_bits, unique);
  if (!p.b.add) {
    p.b.per = static_cast<int>(std::min<int64_t>(std::max<int64_t>((n / 256 + BS_WIDE - 1) / BS_WIDE, 4), BS_SPLIT_KPT) * BS_WIDE);
    p.b.n_wg = static_cast<int>((n + p.b.per - 1) / p.b.per);
  }
  p.wide = !p.b.add || n > (unique ? BS_WIDE_LEVEL_N : BS_MID_N);
  p.q = p.wide ? 2048 : 512;
  p.n_share = static_cast<int>((n + p.q - 1) / p.q);
  return p;
}
template <typename KeyT, bool DEDUP>
struct SplitWs {
  typename BsForm<KeyT, DEDUP>::Elem* recs;
  int32_t* rows;
  KeyT* part;
  uint16_t* off;
  int32_t *tot, *out_at, *out_n, *n_kept, *arrived;
  BsShare* share;
  size_t bytes;
};
template <typename KeyT, bool DEDUP>
SplitWs<KeyT, DEDUP> carve_split(void* ws, int64_t n, const SplitPlan& p) {
  using F = BsForm<KeyT, DEDUP>;
  SplitWs<KeyT, DEDUP> w{};
  char* c = static_cast<char*>(ws);
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char* r = c + at;
    at += (bytes + 255) / 256 * 256;
    return r;
  };
  w.n_kept = reinterpret_cast<int32_t*>(take(256));
  w.arrived = reinterpret_cast<int32_t*>(take((BS_ARRIVE + 1) * BS_ARRIVE_PITCH * 4));
  w.recs = reinterpret_cast<typename F::Elem*>(take(size_t(n) * sizeof(typename F::Elem)));
  if (F::ROWS) w.rows = reinterpret_cast<int32_t*>(take(size_t(n) * 4));
  if (DEDUP) {
    w.part = reinterpret_cast<KeyT*>(take(size_t(n) * sizeof(KeyT)));
    w.out_at = reinterpret_cast<int32_t*>(take(size_t(p.n_share) * 4));
    w.out_n = reinterpret_cast<int32_t*>(take(size_t(p.n_share) * 4));
  }
  w.share = reinterpret_cast<BsShare*>(take(size_t(p.n_share) * sizeof(BsShare)));
  w.tot = reinterpret_cast<int32_t*>(take(size_t(p.b.n_bin) * 4));
  w.off = reinterpret_cast<uint16_t*>(take(size_t(p.b.n_wg) * bs_off_pitch(p.b.n_bin) * 2));
  w.bytes = at;
  return w;
}

// The bins' totals of a sort: in a block that the library keeps cleared between its sorts (the last kernel clears it again),
// or, where none is to be had (under capture, whose replays know nothing of other sorts; on hipStreamPerThread; once the blocks of
// the library's image are in use on other streams), in the workspace, cleared by a kernel of its own, or nowhere, where so few
// workgroups have counted that their counts may be summed where they are read (p is NULL then).  Levels, whose launches are
// nobody's contract, have none then either (bs_starts_kernel).
struct Totals {
  int32_t* p = nullptr;
  size_t pitch = 0, bytes = 0;
  bool kept = false;
  StreamId s;
  Totals(const BucketPlan& plan, int32_t* in_ws, int n_levels, bool levels, const StreamId& s_) : s(s_) {
    if (!plan.add) return;
    bytes = size_t(plan.n_bin) * 4 * n_levels;
    pitch = size_t(plan.n_bin) * 4;
    p = static_cast<int32_t*>(zeroed_alloc(bytes, s, levels));
    kept = p != nullptr;
    if (kept || levels || plan.n_wg <= BS_SUM_WG) return;
    p = in_ws;
    hipLaunchKernelGGL(bs_clear_kernel, dim3((plan.n_bin + BS_THREADS - 1) / BS_THREADS), dim3(BS_THREADS), 0, s, p, plan.n_bin);
  }
  // once all kernels of the sort are enqueued
  int done(const char* what) {
    const bool ok = hipGetLastError() == hipSuccess;
    if (kept) zeroed_free(p, bytes, s, ok);
    return ok ? SPC_OK : set_error(SPC_ERR_HIP, "%s launch failed", what);
  }
};

// split, (starts,) merge
template <typename KeyT, bool DEDUP, typename Src>
void split_merge(const Src& src, int64_t n, int used_bits, const SplitPlan& p, const SplitWs<KeyT, DEDUP>& w, int n_levels, size_t ws_pitch,
                 const Totals& t, KeyT* out_k, int32_t* out_v, hipStream_t s) {
  const BucketPlan& b = p.b;
  const size_t lds = bs_split_lds<KeyT, DEDUP>(b.n_bin, b.per);
  auto split = [&](auto KPT_, auto ADD_) {
    constexpr int KPT = decltype(KPT_)::value;
    constexpr bool ADD = decltype(ADD_)::value;
    if constexpr (!ADD) {  // (16384 bins or long shares: more than the default LDS limit)
      static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bs_count_kernel<KeyT, Src, DEDUP, KPT, ADD>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024);
      (void)attr;
    }
    hipLaunchKernelGGL((bs_count_kernel<KeyT, Src, DEDUP, KPT, ADD>), dim3(b.n_wg, n_levels), dim3(BS_WIDE), lds, s, src, n, b.per, b.shift,
                       b.n_bin, static_cast<void*>(w.recs), static_cast<void*>(w.off), ws_pitch, t.p, t.pitch, w.rows, t.kept && !DEDUP ? w.arrived : nullptr);
  };
  auto keys = [&](auto ADD_) {
    if (b.per <= 2 * BS_WIDE) split(std::integral_constant<int, 2>{}, ADD_);
    else if (b.per <= 4 * BS_WIDE) split(std::integral_constant<int, 4>{}, ADD_);
    else if constexpr (!decltype(ADD_)::value) split(std::integral_constant<int, BS_SPLIT_KPT>{}, ADD_);
  };
  if (t.p) keys(std::true_type{});
  else keys(std::false_type{});
  MergeArgs<KeyT, DEDUP> a{};
  a.recs = w.recs;
  a.rows = w.rows;
  a.off = w.off;
  a.n_wg = b.n_wg;
  a.per = b.per;
  a.shift = b.shift;
  a.n_bin = b.n_bin;
  a.q = p.q;
  a.n = static_cast<int>(n);
  a.used_bits = used_bits;
  a.tot = t.p;
  a.tot_pitch = t.pitch;
  a.clear = t.kept ? 1 : 0;
  a.arrived = w.arrived;
  a.share = w.share;
  a.n_kept = w.n_kept;
  a.out_k = out_k;
  a.out_v = out_v;
  a.out_at = w.out_at;
  a.out_n = w.out_n;
  a.ws_pitch = ws_pitch;
  auto merge = [&](auto WIDE_, auto FROM_) {
    constexpr int KPT = decltype(WIDE_)::value ? 4 : 2, FROM = decltype(FROM_)::value;
    hipLaunchKernelGGL((bs_merge_kernel<KeyT, DEDUP, KPT, FROM>), dim3(p.n_share, n_levels), dim3(BS_MT), 0, s, a);
  };
  if (!t.p && !DEDUP && b.add) {  // (few regions)
    static_assert(BS_MID_N / BS_LONG_SHARE >= BS_SUM_WG, "never where workgroups merge wide: this form takes 512 positions");
    if constexpr (!DEDUP) merge(std::false_type{}, std::integral_constant<int, BS_TABLE>{});
    return;
  }
  if (!t.p)
    hipLaunchKernelGGL(bs_starts_kernel, dim3((b.n_bin + BS_START_BINS - 1) / BS_START_BINS, n_levels), dim3(BS_WIDE), 0, s, w.off, b.n_wg, b.n_bin,
                       p.q, p.n_share, w.share, w.n_kept, ws_pitch);
  if (t.p && p.wide) merge(std::true_type{}, std::integral_constant<int, BS_TOTALS>{});
  else if (t.p) merge(std::false_type{}, std::integral_constant<int, BS_TOTALS>{});
  else if (p.wide) merge(std::true_type{}, std::integral_constant<int, BS_STARTS>{});
  else if constexpr (DEDUP) merge(std::false_type{}, std::integral_constant<int, BS_STARTS>{});
}
}  // namespace

// Entries of the tables of a sort of up to n keys: never fewer for more keys, so that a workspace for n keys (of this sort's
// range) serves fewer as well.  Shares of up to BS_ADD_N keys are fixed, so a plan's own workgroups grow with n between the
// steps; beyond, shares are rounded up and the workgroups fall at every step (128 for 655360 keys, 107 for one more).
static size_t table_entries(int64_t n) {
  size_t most = n > BS_ADD_N ? size_t(2) * BS_MAX_WG * BS_MAX_BIN : 0;
  for (int64_t m : {std::min(n, BS_SHORT_N), std::min(n, BS_ADD_N)}) {
    const BucketPlan p = bucket_plan(m, 64, true);  // (the more workgroups of the two)
    most = std::max(most, (size_t(p.n_wg) * p.n_bin + 63) / 64 * 64);
  }
  return most;
}

// (also what split + merge take: 8 or 12 bytes a key, twice a key for levels, and rows of 16-bit entries for no more regions than the
// tables' rows, except that beyond 6 Mi keys there are more regions than these)
size_t bucket_sort_ws_bytes(int key_bits, int64_t n) {
  const size_t nn = static_cast<size_t>(std::max<int64_t>(n, 1));
  const size_t k = ((nn + BS_PAD_KEYS) * (key_bits / 8) + 255) / 256 * 256, v = ((nn + BS_PAD_KEYS) * 4 + 255) / 256 * 256;
  const BucketPlan cap = bucket_plan(n, 64, true);
  const size_t tables = std::max(table_entries(n) * 4, (nn / (BS_SPLIT_KPT * BS_WIDE) + 1) * bs_off_pitch(BS_MAX_BIN) * 2 * size_t(n > BS_ADD_N));
  return 2 * k + v + tables + (cap.n_bin + 64 + 2 * (nn / BS_PART + 2)) * 4 + 2048;
}

template <typename KeyT>
static int recorded_pack_sort(const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status, KeyT* keys_out,
                              int32_t* perm_out, void* ws, const StreamId& s) {
  const BucketPlan p = bucket_plan(n, used_bits, false);
  const Ws<KeyT> w = carve<KeyT>(ws, n);
  Totals tot(p, w.fstart, 1, false, s);
  const SrcPack<KeyT> src{coords, pp, status};
  using Src = SrcPack<KeyT>;
  const bool sum = p.add && !tot.p;
  auto count = [&](auto ADD_) {
    hipLaunchKernelGGL((bs_count_kernel<KeyT, Src, false, 0, decltype(ADD_)::value>), dim3(p.n_wg), dim3(BS_WIDE), size_t(p.n_bin) * 4, s, src, n,
                       p.per, p.shift, p.n_bin, static_cast<void*>(w.keys0), static_cast<void*>(w.table), size_t(0), tot.p, size_t(0),
                       static_cast<int32_t*>(nullptr), static_cast<int32_t*>(nullptr));
  };
  if (tot.p) count(std::true_type{});
  else count(std::false_type{});
  if (!p.add)
    hipLaunchKernelGGL(bs_colscan_kernel, dim3((p.n_bin / 4 + BS_COL_THREADS - 1) / BS_COL_THREADS), dim3(BS_COL_THREADS), 0, s, w.table, w.before,
                       p.n_wg, p.n_bin, w.fstart);
  auto scatter = [&](auto SUM_) {
    constexpr bool SUM = decltype(SUM_)::value;
    // (the scatter pass holds two ints per bin: beyond 8191 bins that is more than the default LDS limit)
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bs_scatter_kernel<KeyT, SUM>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (2 * BS_MAX_BIN + 2) * 4);
    (void)attr;
    hipLaunchKernelGGL((bs_scatter_kernel<KeyT, SUM>), dim3(p.n_wg), dim3(BS_WIDE), size_t(2 * p.n_bin + 2) * 4, s, w.keys0, n, p.per, p.shift,
                       p.n_bin, p.add ? w.table : w.before, p.add ? tot.p : w.fstart, w.keys1, w.vals1, w.win);
  };
  if (sum) scatter(std::true_type{});
  else scatter(std::false_type{});
  // Four waves share a part's window while the launch is latency-bound (its time is that of the part with
  // the largest window); from BS_RANK_SOLO_N keys on the pass is bound by how many parts
  // a CU has in flight, and one wave per part (no LDS, no barrier, four times the parts per CU) is
  // faster: 10^6 keys 32 -> 26 us; at 240 k keys of dense indoor scenes it was slower (37 -> 47 us).
  const int n_part = static_cast<int>((n + BS_PART - 1) / BS_PART);
  if (n >= BS_RANK_SOLO_N)
    hipLaunchKernelGGL((bs_rank_kernel<KeyT, 1>), dim3(n_part), dim3(64), 0, s, w.keys1, w.vals1, w.win, static_cast<int>(n), keys_out, perm_out);
  else
    hipLaunchKernelGGL((bs_rank_kernel<KeyT, BS_THREADS / 64>), dim3(n_part), dim3(BS_THREADS), 0, s, w.keys1, w.vals1, w.win,
                       static_cast<int>(n), keys_out, perm_out);
  return tot.done("sort");
}

template <typename KeyT>
static int pack_sort_t(const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status, void* keys_out,
                       int32_t* perm_out, void* ws, const StreamId& s) {
  if (n < BS_LARGE_N && stream_is_capturing(s))
    return recorded_pack_sort<KeyT>(coords, n, pp, used_bits, status, static_cast<KeyT*>(keys_out), perm_out, ws, s);
  const SplitPlan p = split_plan(n, used_bits, false);
  const SplitWs<KeyT, false> w = carve_split<KeyT, false>(ws, n, p);
  Totals tot(p.b, w.tot, 1, false, s);
  split_merge<KeyT, false>(SrcPack<KeyT>{coords, pp, status}, n, used_bits, p, w, 1, 0, tot, static_cast<KeyT*>(keys_out), perm_out, s);
  return tot.done("sort");
}

int bucket_pack_sort(int key_bits, const int4* coords, int64_t n, const PackParams& pp, int used_bits, int32_t* status,
                     void* keys_out, int32_t* perm_out, void* ws, const StreamId& s) {
  return key_bits == 32 ? pack_sort_t<uint32_t>(coords, n, pp, used_bits, status, keys_out, perm_out, ws, s)
                        : pack_sort_t<uint64_t>(coords, n, pp, used_bits, status, keys_out, perm_out, ws, s);
}

template <typename KeyT>
static int mask_unique_t(const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, void* ws, size_t ws_pitch,
                         const StreamId& s) {
  const SplitPlan p = split_plan(n, used_bits, true);
  const SplitWs<KeyT, true> w = carve_split<KeyT, true>(ws, n, p);
  SrcMasks<KeyT> src;
  LevelOut<KeyT> lo;
  batch_args(keys_in, jobs, n_levels, &src, &lo);
  Totals tot(p.b, nullptr, n_levels, true, s);
  split_merge<KeyT, true>(src, n, used_bits, p, w, n_levels, ws_pitch, tot, w.part, nullptr, s);
  hipLaunchKernelGGL(bs_compact_kernel<KeyT>, dim3(p.n_share, n_levels), dim3(BS_THREADS), 0, s, w.part, w.out_at, w.out_n, lo, ws_pitch,
                     tot.kept ? tot.p : nullptr, tot.pitch, p.b.n_bin);
  return tot.done("downsample");
}

int bucket_mask_unique(int key_bits, const void* keys_in, int64_t n, const LevelJob* jobs, int n_levels, int used_bits, void* ws,
                       size_t ws_pitch, const StreamId& s) {
  return key_bits == 32 ? mask_unique_t<uint32_t>(keys_in, n, jobs, n_levels, used_bits, ws, ws_pitch, s)
                        : mask_unique_t<uint64_t>(keys_in, n, jobs, n_levels, used_bits, ws, ws_pitch, s);
}

}  // namespace spc
