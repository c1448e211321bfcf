// Kernel-map construction: the one-shot search over sorted packed keys
// (Sections 5.2-5.3), the output-stationary |V_q| x K^3 layout, the filtered
// weight-stationary lists (Section 5.4, cases I and II) and the network-wide
// builder (Section 5.5).
//
// What is kept from the paper: no query structure is built; offsets are split into
// K^2 groups that share (dx,dy); only the smallest-z query of a group is searched and
// the other K-1 are resolved on consecutive positions; queries are formed by adding a
// packed offset to a packed key.
// What is different (CDNA4): a workgroup owns a contiguous tile of sorted output
// voxels, and each of its K waves one x offset.  Because adding a constant keeps the order, all
// queries of a tile with one x offset fall into one contiguous window of the input array.  A wave finds
// its window's two ends 32-ary, the first rounds on 256 probes in LDS (one or two dependent loads for 2^18 keys
// instead of 18), copies the window, with the row numbers its hits will store, into LDS with
// coalesced loads, and every lane then searches in LDS with the window state in scalar registers
// (the kernel is bound by instruction issue).
// Of windows that do not fit the LDS budget every step-th key is staged, and the last few
// probes of their searches go to global memory.
#include <algorithm>
#include <chrono>
#include <map>
#include <set>
#include <thread>
#include <tuple>
#include <type_traits>

#include "spc_internal.h"

namespace spc {

constexpr int N_PROBES = 256;  // first-round probes of the window-bound searches
constexpr int MAX_K = 7;
constexpr int WS_MAX_K3_SEARCH = MAX_K * MAX_K * MAX_K;

template <typename KeyT>
struct SearchParams {
  KeyT X0, dX;      // packed x offset of ix = 0 and its step per ix (wrapping arithmetic: the offsets of an axis are
  KeyT Y0, dY;      // an arithmetic sequence); the same for y
  KeyT ymin, ymax;  // packed smallest and largest y offset
  KeyT zmin;        // packed smallest z offset
  KeyT zstep;       // distance between consecutive z offsets (= input stride)
  int zrev;         // 1: z offsets descend with iz (transposed maps)
  unsigned need;    // bit ix: the offsets with this ix include some of one of the two subsets
};

__device__ inline int lanemask_lt_popc(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(m), 0));
}
// OR over the lanes of each half of the wave; lanes 31 and 63 receive it.
__device__ inline unsigned half_wave_or(unsigned x) {
  x |= static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x111, 0xf, 0xf, true));  // row_shr 1, 2, 4, 8
  x |= static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x112, 0xf, 0xf, true));
  x |= static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x114, 0xf, 0xf, true));
  x |= static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x118, 0xf, 0xf, true));
  x |= static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x142, 0xf, 0xf, true));  // lane 15 of a row to the next row
  return x;
}
// The same, summing.
__device__ inline int half_wave_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  return x + __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, true);  // lane 15 of an even row to the next row
}

// Both ends of a window by one wave: the lower half searches the first index with key >= q, the upper half the first
// index with key > q (q per half).  The first rounds need no memory: both searches start from the same N_PROBES probes
// (the last key of every 1/N_PROBES slice, in LDS), searched 32-ary by the half's lanes with a ballot per round.
// From then on lane p of a half probes the last key of the p-th of 32 sub-slices, and the half's bits of the ballot
// give the sub-slice.  The searches stop once both answers are known to within `slack` positions and return
// the outer ends: a window that is a few keys too wide costs less than
// another round of dependent loads.
template <typename KeyT>
__device__ inline int half_wave_bound(const SPC_GLOBAL KeyT* keys, int n, const KeyT* s_probe, KeyT q, int slack) {
  constexpr int P = 32;
  const int lane = threadIdx.x & 63, p = lane % P;
  const bool upper = lane >= P;
  const int chunk0 = (n + N_PROBES - 1) / N_PROBES;
  auto before = [&](KeyT v) { return upper ? (v <= q) : (v < q); };
  auto count = [&](bool pred) {
    const unsigned long long b = __ballot(pred);
    return __popc(upper ? static_cast<unsigned>(b >> 32) : static_cast<unsigned>(b));
  };
  // number of probes before the answer (probe j is the last key of slice j)
  const int n_probes = (n + chunk0 - 1) / max(chunk0, 1);
  constexpr int STEP = N_PROBES / P;
  const int j1 = (p + 1) * STEP - 1;
  const int c1 = min(count(j1 < n_probes && before(s_probe[j1])), P - 1);
  const int j2 = c1 * STEP + p;
  const int c = c1 * STEP + count(p < STEP && j2 < n_probes && before(s_probe[min(j2, N_PROBES - 1)]));
  int lo = n, hi = n;
  if (c < n_probes) {
    lo = c * chunk0;
    hi = min(lo + chunk0 - 1, n - 1);
  }
  while (__ballot(hi - lo > slack) != 0) {  // every round shortens every unfinished search
    const int len = hi - lo, chunk = (len + P - 1) / P;
    const int first = min(lo + p * chunk, hi);
    const KeyT v = keys[max(0, min(first + chunk - 1, hi - 1))];
    const int m = count(len > 0 && first < hi && before(v));
    if (len > 0) {
      const int nlo = lo + m * chunk;
      if (m * chunk >= len) {  // every sub-slice lies before the answer
        lo = hi;
      } else {
        hi = min(nlo + chunk - 1, hi - 1);
        lo = nlo;
      }
    }
  }
  // the answer lies in [lo, hi]: the low end for a window start, the high end for a window end
  return upper ? hi : lo;
}

// Output voxels per search workgroup (a multiple of the wave size).
// Short tiles spread a small level over the chip
// and keep a workgroup's life short; longer ones pay for their windows less often: build of a map, us, 64 / 128 / 256 rows, 3x3x3,
// 30 k voxels 5.4 / 6.3 / 9.0, 120 k 9.6 / 10.9 / 14.9, 150 k 10.6 / 11.7 / 16.0, 190 k 12.5 / 12.4 / 16.2, 300 k 16.7 / 16.1 / 15.8, 500 k 24.3 / 21.4 /
// 19.4, 10^6 42.6 / 36.2 / 32.2, 3 * 10^6 124 / 102 / 92; 64-bit keys 400 k 23.1 / 21.5 / 24.1, 600 k 31.5 / 28.4 / 29.7, 10^6 49.0 / 41.5 / 41.9; with lists, whose
// records of 256 rows leave a CU few workgroups, 400 k 41.8 / 36.4 / 42.2, 10^6 85 / 71 / 79, 2.5 * 10^6 193 / 156 / 169; 5x5x5, 64 / 128 rows: 30 k 10.6 / 13.1, 240 k 44 / 46.
// (1x1x1, whose rows cost next to nothing and whose list's counts are one column: 64 / 128 / 256 rows, 160 k 8.3 / 5.8 / 7.0, 300 k 8.8 / 7.0 / 7.8, 600 k 12.0 / 9.3 / 8.9, 64-bit keys
// 12.9 / 10.6 / 9.1; with lists 160 k 14.7 / 12.9 / 14.0, 600 k 30.1 / 22.3 / 19.2, 2 * 10^6 82.7 / 53.3 / 40.8.)
inline int search_tile(int K, int64_t n_out, int key_bits, bool lists) {
  if (K == 1) return n_out < 150000 ? 64 : n_out < 400000 ? 128 : 256;
  if (K > 3 || n_out < 185000) return 64;
  return lists || n_out < (key_bits == 32 ? 400000 : 1000000) ? 128 : 256;
}
// Input keys (with their row numbers) that the window of one x offset may occupy in LDS.  A window holds what the tile's
// rows can reach: about as many keys as the tile has rows (more where the input level is finer than the output level),
// a few columns of the scene, and the slack of its bounds.
constexpr int search_win_cap(int tile) { return tile == 64 ? 384 : tile == 128 ? 512 : 640; }

// Two outputs, each for its own subset of the K^3 offsets (Section 5.4: all offsets in one of them for a single
// dataflow; the dense offsets in the matrix and the sparse ones in the lists for the hybrid dual dataflow):
//   os_k: columns of the blocked |V_q| x K^3 matrix M and bits of the per-block offset masks (M = NULL: none);
//   ws_k: (PAIRS = true) weight-stationary lists.  They never pass through a matrix: a tile keeps, per (group,
//         row), the place of its lower bound and the hit bits of the group's K queries in LDS (5 bytes where
//         the matrix has 4 K), and once all groups are searched it writes the hits of the ws_k offsets as
//         compacted pairs (input row, offset << 8 | row of the tile), offset-major and row-ascending, into its own
//         slab of `tile_pairs` (slab = tile * K^3 pairs, of which only the first sum-of-hits are touched);
//         tile_counts gets the hits per (offset, tile).
// x offsets none of whose columns is wanted are not searched (the second half of a symmetric map, for example).
//
// One launch searches NB maps of the same kernel size, block row y map y (NB = 1: a map of its own).  The maps of a
// network's coarse levels are far too small to fill the chip, and a launch each costs more than their work: the nine
// searches of a 25-layer UNet on 120 k voxels took nine launches and 79 us one after the other.
template <typename KeyT>
struct SearchArgs {
  const KeyT* in_keys;
  const int* n_in_d;
  const KeyT* out_keys;
  const int* n_out_d;
  int n_in_h, n_out_h;
  SearchParams<KeyT> sp;
  int32_t* M;
  uint32_t* block_masks;
  int32_t* tile_counts;
  const int32_t* in_perm;
  int2* tile_pairs;
  uint8_t* tile_sub;
  int32_t* inv_parent;
  int32_t* arrived;
  KMask os_k, ws_k;
  int n_tiles_cap;
  int mark_pairs;  // (K = 3) blocks of at most so many pairs are marked
  CountNote note_in, note_out;  // where the host polls for the levels' counts
};
constexpr int SEARCH_BATCH = 8;
// A level's voxel count, kept in a scalar register.  (A pointer that comes out of an indexed argument array is a generic
// one to the compiler: loaded as such, the count and everything derived from it would be per-lane values.)
__device__ inline int level_count(const int* n_d, int n_h) {
  int n = n_h;
  if (n_d) n = *(const SPC_GLOBAL int*)n_d;
  return __builtin_amdgcn_readfirstlane(n);
}
template <typename KeyT, int NB>
struct SearchBatch {
  SearchArgs<KeyT> a[NB];
};

template <typename KeyT, int K, int TILE, bool PAIRS>
constexpr size_t search_lds_bytes() {
  return size_t(K) * search_win_cap(TILE) * (sizeof(KeyT) + 4) + N_PROBES * sizeof(KeyT) + (PAIRS ? size_t(K) * K * TILE * 5 : 0);
}

// Wave w of the K waves of a workgroup owns x offset w: it finds the window of the input array that the tile's queries
// with this x offset can hit, stages it in LDS and searches the tile's rows, 64 at a time, for its K y offsets.  The
// waves wait for each other where the probes have come, and before the block masks are put together.
template <typename KeyT, int K, int TILE, bool PAIRS, int NB>
__global__ __launch_bounds__(64 * K) void kmap_search_kernel(const SearchBatch<KeyT, NB> batch) {
  const SearchArgs<KeyT>& args = batch.a[NB == 1 ? 0 : blockIdx.y];
  const SPC_GLOBAL KeyT* in_keys = (const SPC_GLOBAL KeyT*)args.in_keys;
  const SPC_GLOBAL KeyT* out_keys = (const SPC_GLOBAL KeyT*)args.out_keys;
  const SPC_GLOBAL int32_t* in_perm = (const SPC_GLOBAL int32_t*)args.in_perm;
  SPC_GLOBAL char* M = (SPC_GLOBAL char*)args.M;
  SPC_GLOBAL int32_t* inv_parent = (SPC_GLOBAL int32_t*)args.inv_parent;
  const SearchParams<KeyT>& sp = args.sp;
  const KMask &os_k = args.os_k, &ws_k = args.ws_k;
  constexpr int G = K * K, K3 = K * K * K;
  constexpr int MW = (K3 + 31) / 32;  // mask words per 32-row block
  constexpr int CHUNKS = TILE / 64, MAX_BLOCKS = TILE / 32;
  constexpr int NJ = K <= 5 ? K : 4;  // groups (y offsets) whose searches are in flight together
  static_assert(NJ * K <= 32, "the hits of a batch fit one register");
  constexpr int WIN_CAP = search_win_cap(TILE);
  constexpr int PAD = K;  // all-ones keys behind the window: reads behind a lower bound need no bound
  constexpr int BOUND_SLACK = 32;
  constexpr unsigned KB = sizeof(KeyT);
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_off[PAIRS ? K3 + 1 : 1];  // PAIRS: where every offset's pairs start in the tile's slab
  __shared__ int s_cnt[PAIRS ? K3 : 1];
  __shared__ unsigned s_mask[MAX_BLOCKS * MW];
  __shared__ int s_pairs[K == 3 ? MAX_BLOCKS : 1];  // K = 3: hits of every block
  const int tid = threadIdx.x, lane = tid & 63;
  const int ix = __builtin_amdgcn_readfirstlane(tid >> 6);
  int32_t* wval = reinterpret_cast<int32_t*>(smem) + ix * WIN_CAP;                                     // row numbers of the staged keys
  KeyT* win = reinterpret_cast<KeyT*>(smem + size_t(K) * WIN_CAP * 4) + ix * WIN_CAP;                  // staged window
  KeyT* s_probe = reinterpret_cast<KeyT*>(smem + size_t(K) * WIN_CAP * (4 + KB));
  unsigned char* s_rec = smem + size_t(K) * WIN_CAP * (4 + KB) + N_PROBES * KB;
  int32_t* s_pos = reinterpret_cast<int32_t*>(s_rec);             // PAIRS: [G][TILE] place of the group's lower bound among the staged row numbers, or ~position in the input
  uint8_t* s_hit = reinterpret_cast<uint8_t*>(s_pos + G * TILE);  // PAIRS: [G][TILE] bit t: the group's t-th query (ascending z) hit

  const int n_in = level_count(args.n_in_d, args.n_in_h);
  const int n_out = level_count(args.n_out_d, args.n_out_h);
  const int i0 = blockIdx.x * TILE;
  if (i0 >= n_out) return;  // whole workgroup leaves together
  const int rows = min(TILE, n_out - i0);
  if (blockIdx.x == 0) {
    if (tid == 0) {
      args.note_in.publish(n_in);
      args.note_out.publish(n_out);
    }
    for (int j = tid; j < SHARED_TILES; j += 64 * K) ((SPC_GLOBAL int32_t*)args.arrived)[j] = 0;
  }
  if constexpr (PAIRS)
    for (int k = tid; k < K3; k += 64 * K) s_cnt[k] = 0;
  for (int k = tid; k < MAX_BLOCKS * MW; k += 64 * K) s_mask[k] = 0u;
  if (K == 3 && tid < MAX_BLOCKS) s_pairs[tid] = 0;

  KeyT okey[CHUNKS];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) okey[c] = out_keys[i0 + min(c * 64 + lane, rows - 1)];  // lanes past the end repeat the last row
  const KeyT xoff = sp.X0 + KeyT(ix) * sp.dX + sp.zmin;
  const KeyT zspan = KeyT(K - 1) * sp.zstep;

  // ---- window: adding a constant keeps the order, so what the tile's queries with one x offset can hit is one
  // contiguous piece of the input array (y and z offsets only widen it by a few columns of the scene)
  int wlo = 0, wsz = n_in;  // a small level is one window as a whole
  if (n_in + PAD > WIN_CAP) {
    const int chunk0 = (n_in + N_PROBES - 1) / N_PROBES;
    constexpr int PR = (N_PROBES + 64 * K - 1) / (64 * K);  // probes per thread
    // A load of 64 keys far apart keeps the memory path 64 cycles and brings 64 lines: the workgroup asks for them once, not every
    // wave for itself.  Build of a map, us, before / now: 50 k 7.8 / 6.2, 120 k 12.9 / 9.6, 10^6 38.3 / 32.2, 3 * 10^6 98 / 87, 5x5x5 240 k 39.8 / 34.6.
    KeyT pr[PR];
#pragma unroll
    for (int u = 0; u < PR; ++u)  // (slices past the end are never looked at)
      pr[u] = in_keys[min((long long)(u * (64 * K) + tid + 1) * chunk0 - 1, (long long)n_in - 1)];
    const KeyT kfirst = out_keys[i0], klast = out_keys[i0 + rows - 1];
#pragma unroll
    for (int u = 0; u < PR; ++u)
      if (u * (64 * K) + tid < N_PROBES) s_probe[u * (64 * K) + tid] = pr[u];
    __syncthreads();
    const KeyT q = lane >= 32 ? KeyT(klast + xoff + sp.ymax + zspan) : KeyT(kfirst + xoff + sp.ymin);
    const int b = half_wave_bound<KeyT>(in_keys, n_in, s_probe, q, BOUND_SLACK);
    wlo = __builtin_amdgcn_readlane(b, 0);
    wsz = max(0, __builtin_amdgcn_readlane(b, 32) - wlo);
  }
  if (!((sp.need >> ix) & 1u)) wsz = 0;
  // a window that does not fit is sampled: LDS then holds the last key of every `step` keys
  const int step = max(1, (wsz + WIN_CAP - PAD - 1) / (WIN_CAP - PAD));
  const bool sampled = step > 1;

  // ---- staging: keys and row numbers (the caller's, through the sort permutation, or positions)
  const int staged = (wsz + step - 1) / step;
  if (sampled) {
    for (int e = lane; e < staged + PAD; e += 64) win[e] = e < staged ? in_keys[wlo + min((e + 1) * step, wsz) - 1] : ~KeyT(0);
  } else {
    constexpr int U = 4;
    for (int e0 = lane; e0 < wsz + PAD; e0 += 64 * U) {
      KeyT key[U];
      int32_t val[U];
      if (wsz > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = in_keys[wlo + min(e0 + u * 64, wsz - 1)];
        if (in_perm) {
#pragma unroll
          for (int u = 0; u < U; ++u) val[u] = in_perm[wlo + min(e0 + u * 64, wsz - 1)];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * 64;
        if (e < wsz + PAD) {
          win[e] = e < wsz ? key[u] : ~KeyT(0);
          wval[e] = in_perm ? val[u] : wlo + e;
        }
      }
    }
  }
  __syncthreads();  // (counters and masks are cleared; the wave's own window needs no barrier)

  // ---- per-lane searches, 64 output voxels at a time, the K y offsets interleaved (independent LDS chains hide each
  // other's latency).  The phase is bound by the number of instructions, so everything that is the same for the 64
  // lanes lives in scalar registers.
  // A search keeps the LDS byte address `ab` of the key before its lower bound's current base; a round probes the
  // key half = ceil(n/2) further on and moves the base behind it when that key is smaller than the query, which
  // leaves floor(n/2) keys: one addition, one compare and one select per round, no bounds to check (a probe never
  // leaves the window; finished searches probe the key at `ab` again, which changes nothing).
  // (pointers typed as LDS addresses: 32 bits wide, and every access through them is an LDS instruction)
  using LdsBytes = const __attribute__((address_space(3))) unsigned char*;
  using LdsKey = const __attribute__((address_space(3))) KeyT*;
  using LdsInt = const __attribute__((address_space(3))) int32_t*;
  const LdsBytes lwin = (LdsBytes)(const unsigned char*)win, lval = (LdsBytes)(const unsigned char*)wval;
  const unsigned lane_off = (unsigned(lane >> 5) * unsigned(K3 * 32) + unsigned(lane & 31)) * 4u;  // bytes
  const int64_t b0 = int64_t(i0) >> 5;
  // n bits of a subset from bit b on (the words are picked with scalar selects: static indices keep the masks in scalar registers)
  auto subset_bits = [&](const KMask& m, int b) {
    unsigned lo = 0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < MW; ++i) {
      lo = (b >> 5) == i ? m.w[i] : lo;
      hi = (b >> 5) + 1 == i ? m.w[i] : hi;
    }
    return static_cast<unsigned>(((static_cast<unsigned long long>(hi) << 32) | lo) >> (b & 31));
  };
  // every column of this x offset goes to the matrix, in the order of the queries, and nothing else is asked for
  bool plain = M && !inv_parent && !sp.zrev;
#pragma unroll
  for (int i = 0; i < G; i += 32) plain = plain && (~subset_bits(os_k, ix * G + i) & (G - i >= 32 ? ~0u : (1u << ((G - i) & 31)) - 1u)) == 0u;
  auto search_groups = [&](auto N_, auto IY_, int c, KeyT ok) {
    constexpr int N = decltype(N_)::value, IY = decltype(IY_)::value;  // y offsets IY .. IY + N - 1
    const int v = c * 64 + lane;
    const bool act = v < rows;
    LdsBytes ab[N];
    KeyT q0[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      ab[j] = lwin - KB;  // the key before the window
      q0[j] = ok + (xoff + sp.Y0 + KeyT(IY + j) * sp.dY);
    }
    KeyT d[N][K];  // key - smallest query, for the K keys from the lower bound on, and their row numbers: the K
    int32_t val[N][K];  // z-consecutive queries of a group hit consecutive positions (keys are sorted integers whose z components are multiples of the input stride, Section 5.2)
    for (int n = staged; n > 0;) {
      const int rest = n >> 1, half = n - rest;  // half = ceil(n / 2)
      n = rest;
      LdsBytes cand[N];
      KeyT kv[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        cand[j] = ab[j] + unsigned(half) * KB;
        kv[j] = *(LdsKey)cand[j];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) ab[j] = kv[j] < q0[j] ? cand[j] : ab[j];
    }
    if (!sampled) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        LdsBytes vb;
        if constexpr (KB == 4) vb = ab[j] + (lval - lwin) + 4;
        else vb = lval + (unsigned(ab[j] - lwin + KB) >> 1);
#pragma unroll
        for (int i = 0; i < K; ++i) {
          d[j][i] = *(LdsKey)(ab[j] + (i + 1) * KB);
          val[j][i] = *(LdsInt)(vb + i * 4);
        }
        if constexpr (PAIRS) s_pos[((ix * K) + IY + j) * TILE + v] = static_cast<int>(unsigned(ab[j] - lwin + KB) / KB) + ix * WIN_CAP;
      }
    } else {  // the samples say which `step` keys of the array the lower bound is among: the rest of the way in global memory
      // (large kernels: one group after the other, in rolled rounds, so that this rare path does not set the registers)
      const SPC_GLOBAL KeyT* wkeys = in_keys + wlo;
      constexpr int SIDE = K < 5 ? N : 1;
#pragma unroll
      for (int j0 = 0; j0 < N; j0 += SIDE) {
        int pos[SIDE], len[SIDE];
#pragma unroll
        for (int u = 0; u < SIDE; ++u) {
          pos[u] = static_cast<int>(unsigned(ab[j0 + u] - lwin + KB) / KB) * step;
          len[u] = max(0, min(step - 1, wsz - pos[u]));
        }
        for (int left = step; left > 1; left = (left + 1) >> 1) {
          KeyT kv[SIDE];
#pragma unroll
          for (int u = 0; u < SIDE; ++u) kv[u] = wkeys[unsigned(min(pos[u] + (len[u] >> 1), wsz - 1))];
#pragma unroll
          for (int u = 0; u < SIDE; ++u) {
            const int half = len[u] >> 1;
            const bool less = len[u] > 0 && kv[u] < q0[j0 + u];
            pos[u] += less ? half + 1 : 0;
            len[u] = less ? len[u] - half - 1 : half;
          }
        }
#pragma unroll
        for (int u = 0; u < SIDE; ++u) {
          const int j = j0 + u;
#pragma unroll
          for (int i = 0; i < K; ++i) {
            const bool in = pos[u] + i < wsz;
            const unsigned at = min(pos[u] + i, wsz - 1);
            const KeyT key = wkeys[at];
            d[j][i] = in ? key : KeyT(q0[j] - 1);
            val[j][i] = in_perm ? (in_perm + wlo)[at] : wlo + static_cast<int>(at);
          }
          if constexpr (PAIRS) s_pos[((ix * K) + IY + j) * TILE + v] = ~(wlo + pos[u]);
        }
        if constexpr (SIDE < N) asm volatile("" ::: "memory");
      }
    }
    // A query that reaches the all-ones key could take the padding behind its window for a voxel, and a lane past the
    // last row must not hit at all: waves with such lanes look at every key's place.
    KeyT least = KeyT(~q0[0]);
#pragma unroll
    for (int j = 1; j < N; ++j) least = min(least, KeyT(~q0[j]));
    if (__ballot(least <= zspan || !act)) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int rem = static_cast<int>(unsigned(lwin + unsigned(wsz) * KB - KB - ab[j]) / KB);  // keys of the window from the lower bound on
#pragma unroll
        for (int i = 0; i < K; ++i) d[j][i] = act && (sampled || i < rem) ? d[j][i] : KeyT(q0[j] - 1);
      }
    }
    constexpr int BIT0 = IY * K;
    unsigned hb = 0u;  // bit j * K + t: query t of group j hit
    // Every store into the blocked map M[block][k][32] is two full 128-byte segments; rows past the end of the last
    // block hold -1.  Column of query t: offsets of a group ascend with z, queries too unless the z offsets descend with iz.
    const bool in_block = c * 64 + (lane & 32) < rows;
    SPC_GLOBAL char* Mg = M + ((b0 + c * 2) * int64_t(K3) + ix * G + BIT0) * 128;  // uniform
    // (the usual case has a way of its own: what is decided per group below costs as many scalar instructions as the hits vector
    // ones.  Build of one map, us, before / after: 120 k voxels 12.1 / 11.7, 180 k 15.5 / 14.7, 10^6 42.7 / 39.8, 3 * 10^6 98 / 91.5.
    // Groups of five, looked up and stored one after the other, are slower with it: 5x5x5 pass of 240 k voxels 109.9 / 112.3)
    constexpr bool BATCH = K < 5;  // all groups' rows are found before any is stored (large kernels have no registers for that)
    const bool usual = BATCH && !PAIRS && plain;
    const unsigned osb = usual ? ~0u : M ? subset_bits(os_k, ix * G + BIT0) : 0u, wsb = PAIRS ? subset_bits(ws_k, ix * G + BIT0) : 0u;
    struct Rows {
      int32_t t[K];
    };
    [[maybe_unused]] int hits = 0;
    // where the rows of a group go, unless it is the usual case
    auto emit = [&](int j, Rows r) __attribute__((always_inline)) {
      const int gj = ix * K + IY + j;
      // Inverse of a strided map whose offsets partition the inputs (K = layer stride): every input voxel is hit by
      // exactly one (output, offset), which is all its transposed twin needs (such maps are built without a
      // row permutation, so r holds positions)
      if (inv_parent) {
#pragma unroll
        for (int t = 0; t < K; ++t)
          if (r.t[t] >= 0) inv_parent[r.t[t]] = (i0 + v) * K3 + gj * K + (sp.zrev ? K - 1 - t : t);
      }
      if constexpr (PAIRS) {
        // the tile's records stay in LDS; hits are counted per query: lane j * K + t of `hits` holds the count of query t
        // of group j among the wave's 64 rows
        s_hit[gj * TILE + v] = static_cast<uint8_t>((hb >> (j * K)) & ((1u << K) - 1u));
#pragma unroll
        for (int t = 0; t < K; ++t) {
          const int n_hit = __popcll(__ballot(r.t[t] >= 0));
          hits = lane == j * K + t ? n_hit : hits;
        }
      }
      const unsigned osf = (osb >> (j * K)) & ((1u << K) - 1u);
      if (!M || osf == 0u) return;  // no offset goes to the matrix (uniform)
      if (in_block) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
          const int col = sp.zrev ? K - 1 - t : t;
          if ((osf >> col) & 1u) *(SPC_GLOBAL int32_t*)(Mg + (j * K + col) * 128 + lane_off) = r.t[t];
        }
      }
    };
    Rows rows_of[BATCH ? N : 1];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      // query t (ascending z) sits i <= t positions behind the lower bound, i = number of earlier queries that hit:
      // the key looked at moves on by one where a query has hit
      Rows r;
      bool hit[K];
#pragma unroll
      for (int i = 0; i < K; ++i) d[j][i] -= q0[j];
#pragma unroll
      for (int t = 0; t < K; ++t) {
        hit[t] = d[j][0] == KeyT(t) * sp.zstep;
        r.t[t] = hit[t] ? val[j][0] : -1;
#pragma unroll
        for (int i = 0; i + 1 < K - t; ++i) {
          d[j][i] = hit[t] ? d[j][i + 1] : d[j][i];
          val[j][i] = hit[t] ? val[j][i + 1] : val[j][i];
        }
      }
      unsigned hm = 0u;
#pragma unroll
      for (int t = K - 1; t >= 0; --t) hm = hm + hm + (hit[t] ? 1u : 0u);
      hb |= hm << (j * K);
      if constexpr (BATCH) {
        rows_of[j] = r;
      } else {
        emit(j, r);
      }
    }
    if constexpr (BATCH) {
      if (usual) {
        if (in_block) {
#pragma unroll
          for (int j = 0; j < N; ++j)
#pragma unroll
            for (int t = 0; t < K; ++t) *(SPC_GLOBAL int32_t*)(Mg + (j * K + t) * 128 + lane_off) = rows_of[j].t[t];
        }
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) emit(j, rows_of[j]);
      }
    }
    if constexpr (PAIRS) {  // (these offsets' counts belong to this wave alone)
      const int j = lane / K, t = lane - j * K, col = j * K + (sp.zrev ? K - 1 - t : t);
      if (lane < N * K && ((wsb >> col) & 1u)) s_cnt[ix * G + BIT0 + col] += hits;
    }
    if (M) {  // the blocks' masks
      if (sp.zrev) {  // queries of a group to columns
        unsigned x = 0u;
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
          for (int t = 0; t < K; ++t) x |= ((hb >> (j * K + t)) & 1u) << (j * K + K - 1 - t);
        hb = x;
      }
      hb &= osb;
      if constexpr (K == 3) {
        const int sum = half_wave_sum(__popc(hb));
        if ((lane & 31) == 31) atomicAdd(&s_pairs[c * 2 + (lane >> 5)], sum);
      }
      hb = half_wave_or(hb);
      const int bit = ix * G + BIT0;
      if ((lane & 31) == 31 && hb) {
        const unsigned long long f = static_cast<unsigned long long>(hb) << (bit & 31);
        unsigned* m = &s_mask[(c * 2 + (lane >> 5)) * MW + (bit >> 5)];
        if (static_cast<unsigned>(f)) atomicOr(m, static_cast<unsigned>(f));
        if (static_cast<unsigned>(f >> 32)) atomicOr(m + 1, static_cast<unsigned>(f >> 32));
      }
    }
  };
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    if (c * 64 >= rows) break;  // uniform
    search_groups(std::integral_constant<int, NJ>{}, std::integral_constant<int, 0>{}, c, okey[c]);
    if constexpr (K > NJ) search_groups(std::integral_constant<int, K - NJ>{}, std::integral_constant<int, NJ>{}, c, okey[c]);
  }
  __syncthreads();
  if constexpr (PAIRS) {
    // where every offset's pairs start in the slab: exclusive prefix of the counts, by wave 0
    if (ix == 0) {
      int carry = 0;
      for (int k0 = 0; k0 < K3; k0 += 64) {
        const int k = k0 + lane;
        const int c = k < K3 ? s_cnt[k] : 0;
        int x = c;
        for (int s = 1; s < 64; s <<= 1) {
          const int y = __shfl_up(x, s, 64);
          if (lane >= s) x += y;
        }
        if (k < K3) s_off[k] = carry + x - c;
        carry += __shfl(x, 63, 64);
      }
      if (lane == 0) s_off[K3] = carry;
    }
    for (int k = tid; k < K3; k += 64 * K) args.tile_counts[int64_t(k) * args.n_tiles_cap + blockIdx.x] = s_cnt[k];
    __syncthreads();
    // compaction: a wave takes its own offsets, 64 rows at a time.  The hits of a group follow each other from its lower bound
    // on.  A pair goes to the slab as (input row, offset << 8 | row of the tile): with the offset at hand the fill pass need
    // not search it.  (An offset at a time, with its group's records read again for each, and counts added by lane 0 behind two
    // branches per offset: search of 120 k LiDAR voxels 17.4 us, now 16.1; 240 k indoor voxels, 5x5x5, hybrid 66.0, now 59.4;
    // whole builds of other kernels, tiles and keys: 2x2x2 20 k 13.2, 12.0; 3x3x3 200 k, tiles of 128 rows, 38.4, 32.7; 600 k, of 256, 64-bit
    // keys 100, 83; 5x5x5 240 k 64-bit keys 150, 127; 7x7x7 20 k 53.9, 46.9; 240 k 64-bit keys 297, 257)
    static_assert(TILE <= 256, "a row of the tile in eight bits");
    int2* slab = args.tile_pairs + int64_t(blockIdx.x) * TILE * K3;
    uint8_t* sub = args.tile_sub + int64_t(blockIdx.x) * K3 * MAX_BLOCKS;  // (unused for offsets without pairs)
    const int32_t* wval0 = reinterpret_cast<const int32_t*>(smem);
    const int l = ix * G + min(lane, G - 1), off = s_off[l];
    const unsigned long long some = __ballot(lane < G && s_off[l + 1] > off);  // offsets with pairs (none outside ws_k is counted)
    int done[K][K] = {};  // pairs of the offsets in the tile's rows so far
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      if (some == 0ull || c * 64 >= rows) break;  // uniform
      const int v = c * 64 + lane;
      unsigned msk[K];
      int pos[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        msk[j] = s_hit[(ix * K + j) * TILE + v];
        pos[j] = s_pos[(ix * K + j) * TILE + v];
      }
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (((some >> (j * K)) & ((1u << K) - 1u)) == 0u) continue;  // uniform
#pragma unroll
        for (int t = 0; t < K; ++t) {
          const int jk = j * K + (sp.zrev ? K - 1 - t : t), k = ix * G + jk;
          if (!((some >> jk) & 1u)) continue;  // uniform
          const bool hit = v < rows && ((msk[j] >> t) & 1u);
          const unsigned long long bal = __ballot(hit);
          if (hit) {
            const int ahead = __popc(msk[j] & ((1u << t) - 1u));
            int in;
            if (pos[j] >= 0) in = wval0[pos[j] + ahead];
            else in = in_perm ? in_perm[~pos[j] + ahead] : ~pos[j] + ahead;
            slab[__builtin_amdgcn_readlane(off, jk) + done[j][t] + lanemask_lt_popc(bal)] = make_int2(in, k << 8 | v);
          }
          if (lane < 2)  // pairs of the offset in the tile's blocks before this one
            sub[k * MAX_BLOCKS + c * 2 + lane] = static_cast<uint8_t>(done[j][t] + (lane ? __popc(static_cast<unsigned>(bal)) : 0));
          done[j][t] += __popcll(bal);
        }
      }
    }
  }
  if (M) {
    const int n_bl = (rows + 31) >> 5;
    for (int e = tid; e < n_bl * MW; e += 64 * K)
      args.block_masks[b0 * MW + e] = s_mask[e] | (K == 3 && s_pairs[K == 3 ? e : 0] <= args.mark_pairs ? POOL_MARK : 0u);
  }
}

// Weight-stationary lists from the tiles' slabs of compacted pairs (the search kernel in its PAIRS form): one
// workgroup per tile copies its hits, offset by offset, to where the scan of the per-tile counts puts them.  List k
// comes out ordered by output index, without atomics and without a |V_q| x K^3 matrix having existed.  list_base gets
// where the pairs of every 32-row block start in every list, which is how the feature kernel finds a block's pairs.
// SCAN: tile_base holds the per-tile counts themselves, and every workgroup adds up the tiles before its own (a few
// tiles: cheaper than the scan's launch).
template <bool SCAN>
__global__ __launch_bounds__(256) void ws_fill_pairs_kernel(const int2* __restrict__ tile_pairs, int n_out_h,
                                                            const int* __restrict__ n_out_d, int K3, int tile,
                                                            const int32_t* __restrict__ tile_base, int n_tiles_cap,
                                                            int32_t* __restrict__ nnz, const uint8_t* __restrict__ tile_sub,
                                                            int32_t* __restrict__ ws_in, int32_t* __restrict__ ws_out,
                                                            int64_t ws_stride, int k_lim, int32_t* __restrict__ list_base) {
  __shared__ int s_off[WS_MAX_K3_SEARCH + 1], s_dst[WS_MAX_K3_SEARCH];
  const int n_out = n_out_d ? *n_out_d : n_out_h;
  const int i0 = blockIdx.x * tile;
  if (i0 >= n_out) return;
  const int n_tiles = (n_out + tile - 1) / tile;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if constexpr (SCAN) {
    // eight threads per offset, eight tiles' counts of a thread in flight
    for (int k0 = 0; k0 < K3; k0 += 32) {
      const int k = k0 + (tid >> 3);
      int sum = 0;
      if (k < k_lim) {
        const int32_t* col = tile_base + int64_t(k) * n_tiles_cap;
        for (int t0 = tid & 7; t0 < int(blockIdx.x); t0 += 64) {
          int c[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) c[u] = col[min(t0 + u * 8, int(blockIdx.x))];
#pragma unroll
          for (int u = 0; u < 8; ++u) sum += t0 + u * 8 < int(blockIdx.x) ? c[u] : 0;
        }
      }
      for (int d = 4; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
      if ((tid & 7) == 0 && k < K3) s_dst[k] = sum;
    }
    __syncthreads();
  }
  // counts of this tile (difference of consecutive scanned bases) and their exclusive prefix
  if (wave == 0) {
    int carry = 0;
    for (int k0 = 0; k0 < K3; k0 += 64) {
      const int k = k0 + lane;
      int c = 0;
      if (!SCAN && k < K3) s_dst[k] = 0;
      if (k < k_lim) {
        const int32_t* col = tile_base + int64_t(k) * n_tiles_cap;
        const int b = col[blockIdx.x];
        if constexpr (SCAN) {
          c = b;
        } else {
          c = (int(blockIdx.x) + 1 < n_tiles ? col[blockIdx.x + 1] : nnz[k]) - b;
          s_dst[k] = b;
        }
      }
      int x = c;
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
      }
      if (k < K3) s_off[k] = carry + x - c;
      carry += __shfl(x, 63, 64);
    }
    if (lane == 0) s_off[K3] = carry;
  }
  __syncthreads();
  const int total = s_off[K3];
  const int2* slab = tile_pairs + int64_t(blockIdx.x) * tile * K3;
  const int tile_blocks = tile >> 5, n_bl = (min(tile, n_out - i0) + 31) >> 5;
  const uint8_t* sub = tile_sub + int64_t(blockIdx.x) * K3 * tile_blocks;
  int32_t* base = list_base + (int64_t(i0) >> 5) * K3;
  for (int e = tid; e < n_bl * K3; e += 256) {
    const int b = e / K3, k = e - b * K3;
    base[e] = s_dst[k] + (s_off[k + 1] > s_off[k] ? sub[k * tile_blocks + b] : 0);
  }
  if (int(blockIdx.x) + 1 == n_tiles)  // one row more than blocks: the lists' ends
    for (int k = tid; k < K3; k += 256) {
      const int end = s_dst[k] + s_off[k + 1] - s_off[k];
      base[n_bl * K3 + k] = end;
      if (SCAN) nnz[k] = end;
    }
  for (int e = tid; e < total; e += 256) {
    const int2 pr = slab[e];
    const int k = pr.y >> 8;
    const int64_t dst = int64_t(k) * ws_stride + s_dst[k] + (e - s_off[k]);
    ws_in[dst] = pr.x;
    ws_out[dst] = i0 + (pr.y & 255);
  }
}

// Counts up to which the fill pass adds them up itself: build with lists, 4.1 k voxels 13.8 -> 12.0 us, 20 k (8451 counts)
// 15.7 / 15.2, 30 k 16.5 / 16.6, 60 k 19.6 / 21.7.
// Eight threads add a column, so that no column may be long: 1x1x1, added / scanned, 20 k (313 tiles) 9.5 / 11.0, 40 k (625) 12.2 / 10.7, tiles of 128 rows 60 k (469) 11.9 /
// 11.9, 200 k 18.6 / 13.2, 600 k 47.3 / 22.3.
constexpr int64_t WS_SCAN_IN_FILL = 6144, WS_TILES_IN_FILL = 448;
// One workgroup per offset k: exclusive scan of that offset's per-tile counts in place, total into nnz[k].
// A thread owns a run of consecutive tiles; the runs are fetched in batches of WS_SCAN_U loads per thread that are
// all in flight together (a loop of load, scan, store rounds over 256 tiles at a time took 7.6 us for 3750 tiles:
// fifteen dependent round trips; 1024 threads with four counts each instead of 256 with eight: 3750 tiles, 5x5x5, 6.2 -> 5.1 us,
// 1875 tiles, 3x3x3, 4.5 either way).
constexpr int WS_SCAN_U = 4, WS_SCAN_THREADS = 1024, WS_SCAN_WAVES = WS_SCAN_THREADS / 64;
__global__ __launch_bounds__(WS_SCAN_THREADS) void ws_scan_kernel(int32_t* __restrict__ tile_counts, int n_tiles_cap, int tile,
                                                                  int n_out_h, const int* __restrict__ n_out_d,
                                                                  int32_t* __restrict__ nnz, int k_lim) {
  __shared__ int wave_sum[WS_SCAN_WAVES];
  if (int(blockIdx.x) >= k_lim) {  // offsets without a list of their own (second half of a symmetric map)
    if (threadIdx.x == 0) nnz[blockIdx.x] = 0;
    return;
  }
  const int n_out = n_out_d ? *n_out_d : n_out_h;
  const int n_tiles = (n_out + tile - 1) / tile;
  int32_t* c = tile_counts + int64_t(blockIdx.x) * n_tiles_cap;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int carry = 0;
  for (int b0 = 0; b0 < n_tiles; b0 += WS_SCAN_THREADS * WS_SCAN_U) {
    const int first = b0 + threadIdx.x * WS_SCAN_U;  // this thread's run: tiles first .. first + WS_SCAN_U - 1
    int v[WS_SCAN_U];
#pragma unroll
    for (int u = 0; u < WS_SCAN_U; ++u) v[u] = first + u < n_tiles ? c[first + u] : 0;
    int sum = 0;
#pragma unroll
    for (int u = 0; u < WS_SCAN_U; ++u) sum += v[u];
    int x = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (b0 > 0) __syncthreads();  // the wave sums of the round before have been read
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WS_SCAN_WAVES; ++w) {
      const int s = wave_sum[w];
      if (w < wave) base += s;
      tot += s;
    }
    int run = carry + base + x - sum;
#pragma unroll
    for (int u = 0; u < WS_SCAN_U; ++u) {
      if (first + u < n_tiles) c[first + u] = run;
      run += v[u];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) nnz[blockIdx.x] = carry;
}

// list_base of lists that no tile of a search has left behind (the lists of a transposed map, which are its strided twin's;
// a symmetric half-map's by input row): a thread per (block, list) searches the list's ascending rows.
__global__ __launch_bounds__(256) void list_base_kernel(const int32_t* __restrict__ rows, int64_t stride, const int32_t* __restrict__ nnz,
                                                        int K3, int k_lim, int n_h, const int* __restrict__ n_d,
                                                        int32_t* __restrict__ list_base) {
  const int n = n_d ? *n_d : n_h;
  const int64_t gid = blockIdx.x * int64_t(256) + threadIdx.x;
  const int b = static_cast<int>(gid / K3), k = static_cast<int>(gid - int64_t(b) * K3);
  if (b > (n + 31) >> 5 || k >= k_lim) return;
  const int32_t* list = rows + int64_t(k) * stride;
  int lo = 0, len = nnz[k];
  while (len > 0) {
    const int half = len >> 1;
    const bool less = list[lo + half] < b * 32;
    lo = less ? lo + half + 1 : lo;
    len = less ? len - half - 1 : half;
  }
  list_base[gid] = lo;
}

// Output-stationary layout of a transposed layer from the inverse its strided twin's search left behind (pairs
// of a transposed layer are the twin's pairs with the roles swapped, Section 5.5: maps shared between layers).
// Where the twin's offsets partition its inputs (K = layer stride, e.g. 2x2x2 at stride 2), every output voxel p of
// the transposed layer has exactly one pair, (input parent[p] / K^3, offset parent[p] % K^3): a thread per voxel
// writes its row of the blocked matrix (full lines per offset) and the block masks fall out of ballots.
// Block row y does map y of the batch.
struct TransposedArgs {
  const int32_t* parent;
  const int* n_d;
  int n_h, K3;
  int32_t* Mt;
  uint32_t* block_masks;
  int32_t* arrived;
};
struct TransposedBatch {
  TransposedArgs a[SEARCH_BATCH];
};
__global__ __launch_bounds__(256) void transposed_from_parent_kernel(const TransposedBatch batch) {
  const TransposedArgs& args = batch.a[blockIdx.y];
  const int32_t* __restrict__ parent = args.parent;
  int32_t* __restrict__ Mt = args.Mt;
  uint32_t* __restrict__ block_masks = args.block_masks;
  const int K3 = args.K3;
  const int n = level_count(args.n_d, args.n_h);
  if (blockIdx.x == 0 && n > 0)
    for (int j = threadIdx.x; j < SHARED_TILES; j += 256) args.arrived[j] = 0;
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t blk = p >> 5;
  if (blk * 32 >= n) return;  // whole 32-row blocks leave together (the ballots below stay among one wave's lanes)
  const int pr = p < n ? parent[p] : -1;
  const int q = pr < 0 ? -1 : pr / K3, kp = pr < 0 ? -1 : pr - q * K3;
  const int half = (threadIdx.x >> 5) & 1;
  uint32_t mask = 0;  // K3 <= 32 here
  for (int k = 0; k < K3; ++k) {
    Mt[(blk * K3 + k) * 32 + (p & 31)] = k == kp ? q : -1;
    const unsigned long long b = __ballot(k == kp);
    if ((half ? unsigned(b >> 32) : unsigned(b)) != 0u) mask |= 1u << k;
  }
  if ((p & 31) == 0) block_masks[blk] = mask;
}

__global__ void copy_int_kernel(const int* src, int* dst) { *dst = *src; }

// ---------------------------------------------------------------- host side
static int axis_offset(int K, int s, int i) { return (K % 2 == 1) ? (i - (K - 1) / 2) * s : i * s; }


static std::atomic<int64_t> g_search_launches{0};  // searches enqueued by this process (see spc_search_count)

template <typename KeyT, int K>
static SearchArgs<KeyT> search_args(spc_kmap* m) {
  const PackInfo& pi = m->pi;
  const int sp_stride = m->desc.in_stride;
  const int sign = m->desc.transposed ? -1 : 1;
  SearchParams<KeyT> sp{};
  auto packed = [&](int i, int shift) {  // offset of index i along an axis, shifted into its field (wrapping)
    return static_cast<KeyT>(static_cast<uint64_t>(int64_t(sign) * axis_offset(K, sp_stride, i)) << shift);
  };
  sp.X0 = packed(0, pi.sh_x);
  sp.dX = K > 1 ? static_cast<KeyT>(packed(1, pi.sh_x) - sp.X0) : KeyT(0);
  sp.Y0 = packed(0, pi.sh_y);
  sp.dY = K > 1 ? static_cast<KeyT>(packed(1, pi.sh_y) - sp.Y0) : KeyT(0);
  const bool yrev = int64_t(sign) * axis_offset(K, sp_stride, 0) > int64_t(sign) * axis_offset(K, sp_stride, K - 1);
  sp.ymin = packed(yrev ? K - 1 : 0, pi.sh_y);
  sp.ymax = packed(yrev ? 0 : K - 1, pi.sh_y);
  const int64_t z_a = int64_t(sign) * axis_offset(K, sp_stride, 0), z_b = int64_t(sign) * axis_offset(K, sp_stride, K - 1);
  sp.zmin = static_cast<KeyT>(static_cast<uint64_t>(std::min(z_a, z_b)));
  sp.zstep = static_cast<KeyT>(sp_stride);
  sp.zrev = (K > 1 && z_a > z_b) ? 1 : 0;
  for (int k = 0; k < K * K * K; ++k)
    if ((m->os_map && m->os_k.has(k)) || m->ws_k.has(k)) sp.need |= 1u << (k / (K * K));
  Level* in = m->in_level;
  Level* out = m->out_level;
  SearchArgs<KeyT> a{};
  auto announce = [](Level* lv) {  // (a level is made on the stream of its searches)
    if (lv->announced || !lv->slot.dev) return CountNote{};
    lv->announced = true;
    return CountNote{lv->slot.dev, lv->slot.tag};
  };
  a.note_in = announce(in);
  a.note_out = announce(out);
  a.in_keys = static_cast<const KeyT*>(in->keys);
  a.n_in_h = static_cast<int>(in->n_host < 0 ? 0 : in->n_host);
  a.n_in_d = in->n_dev;
  a.out_keys = static_cast<const KeyT*>(out->keys);
  a.n_out_h = static_cast<int>(out->n_host < 0 ? 0 : out->n_host);
  a.n_out_d = out->n_dev;
  a.sp = sp;
  a.M = m->os_map;
  a.block_masks = m->block_masks;
  a.tile_counts = m->tile_counts;
  a.n_tiles_cap = m->n_tiles;
  a.in_perm = m->in_perm;
  a.os_k = m->os_k;
  a.ws_k = m->ws_k;
  a.tile_pairs = m->tile_pairs;
  a.tile_sub = m->tile_sub;
  a.inv_parent = m->inv_parent;
  a.arrived = m->arrived;
  a.mark_pairs = in == out ? POOL_BLOCK_PAIRS : -1;
  return a;
}

// The searches of ms[0..count): one kernel size, tile length and form (with or without lists) for all.
template <typename KeyT, int K, int TILE>
static void launch_search(spc_kmap* const* ms, int count, hipStream_t s) {
  const spc_kmap* m = ms[0];
  const bool pairs = (m->desc.layout & SPC_LAYOUT_WS) != 0;
  auto go = [&](auto PAIRS_, auto NB_, int first, int n, int n_tiles) {
    constexpr bool PAIRS = decltype(PAIRS_)::value;
    constexpr int NB = decltype(NB_)::value;
    constexpr size_t lds = search_lds_bytes<KeyT, K, TILE, PAIRS>();
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&kmap_search_kernel<KeyT, K, TILE, PAIRS, NB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
    (void)attr;
    SearchBatch<KeyT, NB> b{};
    for (int i = 0; i < n; ++i) b.a[i] = search_args<KeyT, K>(ms[first + i]);
    hipLaunchKernelGGL((kmap_search_kernel<KeyT, K, TILE, PAIRS, NB>), dim3(n_tiles, n), dim3(64 * K), lds, s, b);
  };
  // the large kernels are searched one map at a time: their levels' searches are long enough to stand alone
  constexpr int MOST = K <= 3 ? SEARCH_BATCH : 1;
  for (int first = 0; first < count; first += MOST) {
    const int n = std::min(count - first, MOST);
    int n_tiles = 0;
    for (int i = 0; i < n; ++i) n_tiles = std::max(n_tiles, ms[first + i]->n_tiles);
    if (n_tiles == 0) continue;
    using One = std::integral_constant<int, 1>;
    using Most = std::integral_constant<int, MOST>;
    if constexpr (TILE < 256 || K == 1) {  // (longer tiles of others have no lists)
      if (pairs) {
        n == 1 ? go(std::true_type{}, One{}, first, n, n_tiles) : go(std::true_type{}, Most{}, first, n, n_tiles);
        continue;
      }
    }
    n == 1 ? go(std::false_type{}, One{}, first, n, n_tiles) : go(std::false_type{}, Most{}, first, n, n_tiles);
  }
  g_search_launches.fetch_add(count, std::memory_order_relaxed);
}

template <typename KeyT>
static int launch_search_k(spc_kmap* const* ms, int count, hipStream_t s) {
  // (search_tile gives a map with lists no longer ones: their records would not fit)
  if (ms[0]->tile > 128 && ms[0]->desc.K > 1 && (ms[0]->desc.layout & SPC_LAYOUT_WS))
    return set_error(SPC_ERR_UNSUPPORTED, "lists are not built by tiles of %d rows", ms[0]->tile);
  auto by_tile = [&](auto K_) {
    constexpr int K = decltype(K_)::value;
    switch (ms[0]->tile) {
      case 64: launch_search<KeyT, K, 64>(ms, count, s); break;
      case 128: launch_search<KeyT, K, 128>(ms, count, s); break;
      default: launch_search<KeyT, K, 256>(ms, count, s); break;
    }
  };
  switch (ms[0]->desc.K) {
    case 1: by_tile(std::integral_constant<int, 1>{}); break;
    case 2: by_tile(std::integral_constant<int, 2>{}); break;
    case 3: by_tile(std::integral_constant<int, 3>{}); break;
    case 5: launch_search<KeyT, 5, 64>(ms, count, s); break;
    case 7: launch_search<KeyT, 7, 64>(ms, count, s); break;
    default: return set_error(SPC_ERR_UNSUPPORTED, "kernel size %d not built (1,2,3,5,7 are)", ms[0]->desc.K);
  }
  return SPC_OK;
}

static void kmap_free(spc_kmap* m) {
  if (m->twin) {  // a transposed map derived from its strided twin: the lists (if any) are the twin's
    if (m->ws_in) {
      m->ws_in = m->ws_out = nullptr;
      m->nnz_dev = nullptr;
    }
    // whoever read this map may have read the twin's arrays: the twin's release waits for them as well
    for (const StreamId& c : m->consumers) m->twin->consumers.push_back(c);
    m->twin->consumers.push_back(m->stream);
    spc_kmap* t = m->twin;
    m->twin = nullptr;
    if (t->refs.fetch_sub(1) == 1) kmap_free(t);
  }
  // The arrays return to the build stream's cache, where the next build may take them at once: that
  // stream first waits for the feature kernels other streams have enqueued on this map.
  if (!m->consumers.empty()) {
    const DeviceScope scope(m->stream.device);
    for (const StreamId& c : m->consumers) order_stream_after(m->stream, c);
  }
  pool_free(m->os_map, m->stream);
  pool_free(m->block_masks, m->stream);
  pool_free(m->ws_in, m->stream);
  pool_free(m->ws_out, m->stream);
  pool_free(m->nnz_dev, m->stream);
  pool_free(m->tile_counts, m->stream);
  pool_free(m->tile_pairs, m->stream);
  pool_free(m->tile_sub, m->stream);
  pool_free(m->list_base, m->stream);
  pool_free(m->list_base_in, m->stream);
  pool_free(m->inv_parent, m->stream);
  pool_free(m->arrived, m->stream);
  level_unref(m->in_level);
  level_unref(m->out_level);
  delete m;
}

static int check_layer(const spc_layer_desc* l) {
  if (!l) return set_error(SPC_ERR_ARG, "layer descriptor is NULL");
  auto pow2 = [](int v) { return v >= 1 && (v & (v - 1)) == 0; };
  if (l->K != 1 && l->K != 2 && l->K != 3 && l->K != 5 && l->K != 7)
    return set_error(SPC_ERR_UNSUPPORTED, "kernel size %d not built (1,2,3,5,7 are)", l->K);
  if (!pow2(l->in_stride) || !pow2(l->layer_stride)) return set_error(SPC_ERR_ARG, "strides must be powers of two");
  if (l->transposed != 0 && l->transposed != 1) return set_error(SPC_ERR_ARG, "transposed must be 0 or 1");
  if (l->transposed && l->layer_stride == 1) return set_error(SPC_ERR_ARG, "a transposed layer needs layer_stride > 1");
  const int base = l->layout & SPC_LAYOUT_BOTH;
  const int thr = (l->layout >> 8) & 0xff;
  if (l->layout < 1 || (l->layout & ~0xff07) || base == 0)
    return set_error(SPC_ERR_ARG, "layout must be OS, WS or BOTH (| WS_SYM) (| HYBRID_T(t))");
  if (thr && base != SPC_LAYOUT_BOTH) return set_error(SPC_ERR_ARG, "a hybrid threshold needs both layouts");
  if (l->layout & SPC_LAYOUT_WS_SYM) {
    if (!(l->layout & SPC_LAYOUT_WS)) return set_error(SPC_ERR_ARG, "WS_SYM modifies the WS layout");
    if (l->layer_stride != 1 || l->K % 2 == 0 || l->K < 3)
      return set_error(SPC_ERR_ARG, "the symmetric half-map needs a submanifold layer with odd K >= 3");
  }
  return SPC_OK;
}

// The packing descriptor must suit the layer (Section 5.3): packed(q) + packed(delta) = packed(q + delta)
// holds only while no field borrows or carries, i.e. while the guard band covers the layer's largest
// offset component; and masking the low bits of a field equals floor() on the raw coordinate only if
// the field's bias, origin - pad, is a multiple of the layer's output stride.
static int check_desc_layer(const spc_pack_desc* d, const spc_layer_desc* l) {
  const int64_t reach = int64_t(l->K % 2 ? (l->K - 1) / 2 : l->K - 1) * l->in_stride;
  if (d->pad < reach)
    return set_error(SPC_ERR_ARG, "guard band pad = %d is smaller than the layer's reach %lld (K = %d, in_stride = %d)", d->pad,
                     static_cast<long long>(reach), l->K, l->in_stride);
  const int64_t so = int64_t(l->in_stride) * l->layer_stride;
  for (int a = 0; a < 3; ++a)
    if ((int64_t(d->origin[a]) - d->pad) % so != 0)
      return set_error(SPC_ERR_ARG, "origin[%d] - pad = %lld is not a multiple of the layer's output stride %lld", a,
                       static_cast<long long>(int64_t(d->origin[a]) - d->pad), static_cast<long long>(so));
  return SPC_OK;
}

static int ilog2(int v) {
  int b = 0;
  while ((1 << b) < v) ++b;
  return b;
}

// Makes the map object for given input/output levels (references are taken) with its arrays; nothing is searched yet.
static int prepare_map(Level* in, Level* out, const PackInfo& pi, const spc_layer_desc& l, const StreamId& s, spc_kmap** res,
                       const int32_t* in_perm, bool want_inverse) {
  spc_kmap* m = new spc_kmap;
  m->in_perm = in_perm;
  m->pi = pi;
  m->desc = l;
  m->K3 = l.K * l.K * l.K;
  m->sym = (l.layout & SPC_LAYOUT_WS_SYM) != 0;
  m->k_lim = m->sym ? (m->K3 - 1) / 2 : m->K3;
  // Offsets of the matrix and of the lists.  With a threshold (hybrid dual dataflow, Section 5.4) the offsets
  // whose L1 norm is below it go to the matrix only and the others to the lists only; a symmetric map keeps
  // lists for the first half of its offsets.
  m->hybrid_t = (l.layout >> 8) & 0xff;
  for (int k = 0; k < m->K3; ++k) {
    const bool dense = m->hybrid_t == 0 || offset_l1(l.K, k) < m->hybrid_t;
    const bool sparse = m->hybrid_t == 0 || !dense;
    if ((l.layout & SPC_LAYOUT_OS) && dense) m->os_k.w[k >> 5] |= 1u << (k & 31);
    if ((l.layout & SPC_LAYOUT_WS) && sparse && k < m->k_lim) m->ws_k.w[k >> 5] |= 1u << (k & 31);
  }
  m->stream = s;
  m->captured = stream_is_capturing(s);
  m->in_level = in;
  in->refs++;
  in->add_reader(s);
  m->out_level = out;
  out->refs++;
  out->add_reader(s);
  m->out_cap = out->n_host >= 0 ? out->n_host : out->cap;
  m->tile = search_tile(l.K, m->out_cap, pi.key_bits, (l.layout & SPC_LAYOUT_WS) != 0);
  m->n_tiles = static_cast<int>((m->out_cap + m->tile - 1) / m->tile);
  m->n_blocks_cap = (m->out_cap + 31) / 32;
  m->mask_words = (m->K3 + 31) / 32;
  const size_t cells = std::max<size_t>(size_t(m->n_blocks_cap) * 32 * m->K3, 64);
  const bool with_os = (l.layout & SPC_LAYOUT_OS) != 0;
  // the |V_q| x K^3 matrix and its block masks exist only when the output-stationary layout is asked for
  if (with_os) {
    m->os_map = static_cast<int32_t*>(pool_alloc(cells * 4, s));
    m->block_masks = static_cast<uint32_t*>(pool_alloc(std::max<size_t>(size_t(m->n_blocks_cap) * m->mask_words * 4, 256), s));
  }
  m->nnz_dev = static_cast<int32_t*>(pool_alloc(std::max<size_t>(size_t(m->K3) * 4, 256), s));
  m->ws_stride = m->out_cap;
  if (want_inverse && !in_perm)
    m->inv_parent = static_cast<int32_t*>(pool_alloc(std::max<size_t>(size_t(in->n_host >= 0 ? in->n_host : in->cap) * 4, 256), s));
  m->arrived = static_cast<int32_t*>(pool_alloc(SHARED_TILES * 4, s));
  bool ok = m->nnz_dev && m->arrived && (!with_os || (m->os_map && m->block_masks)) && (m->inv_parent || !(want_inverse && !in_perm));
  if (ok && (l.layout & SPC_LAYOUT_WS)) {
    m->ws_in = static_cast<int32_t*>(pool_alloc(cells * 4, s));
    m->ws_out = static_cast<int32_t*>(pool_alloc(cells * 4, s));
    m->tile_counts = static_cast<int32_t*>(pool_alloc(std::max<size_t>(size_t(m->n_tiles) * m->K3 * 4, 256), s));
    // slabs of compacted pairs, one per search tile (bounded by tile * K^3 pairs each; a tile writes its hits only)
    m->tile_pairs = static_cast<int2*>(pool_alloc(std::max<size_t>(size_t(m->n_tiles) * m->tile * m->K3 * 8, 256), s));
    m->tile_sub = static_cast<uint8_t*>(pool_alloc(std::max<size_t>(size_t(m->n_tiles) * (m->tile / 32) * m->K3, 256), s));
    const size_t base_bytes = size_t(m->n_blocks_cap + 1) * m->K3 * 4;
    m->list_base = static_cast<int32_t*>(pool_alloc(base_bytes, s));
    if (m->sym) m->list_base_in = static_cast<int32_t*>(pool_alloc(base_bytes, s));
    ok = m->ws_in && m->ws_out && m->tile_counts && m->tile_pairs && m->tile_sub && m->list_base && (!m->sym || m->list_base_in);
  }
  if (!ok) {
    kmap_free(m);
    return SPC_ERR_NOMEM;
  }
  *res = m;
  return SPC_OK;
}

static void launch_list_base(const spc_kmap* m, const int32_t* rows, int k_lim, const Level* lv, int32_t* base, hipStream_t s) {
  const int64_t total = (m->n_blocks_cap + 1) * m->K3;
  hipLaunchKernelGGL(list_base_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, rows, m->ws_stride, m->nnz_dev,
                     m->K3, k_lim, static_cast<int>(lv->n_host < 0 ? 0 : lv->n_host), lv->n_host < 0 ? lv->n_dev : nullptr, base);
}

// Searches and lists of prepared maps that agree in kernel size, tile length, key width and in whether they have lists.
static int search_maps(spc_kmap* const* ms, int count, const StreamId& s) {
  SPC_RETURN_IF(ms[0]->pi.key_bits == 32 ? launch_search_k<uint32_t>(ms, count, s) : launch_search_k<uint64_t>(ms, count, s));
  for (int i = 0; i < count; ++i) {
    spc_kmap* m = ms[i];
    if (!(m->desc.layout & SPC_LAYOUT_WS)) break;
    const Level* out = m->out_level;
    const int n_out_h = static_cast<int>(out->n_host < 0 ? 0 : out->n_host);
    auto fill = [&](auto SCAN_) {
      hipLaunchKernelGGL(ws_fill_pairs_kernel<decltype(SCAN_)::value>, dim3(m->n_tiles), dim3(256), 0, s, m->tile_pairs, n_out_h,
                         out->n_dev, m->K3, m->tile, m->tile_counts, m->n_tiles, m->nnz_dev, m->tile_sub, m->ws_in, m->ws_out,
                         m->out_cap, m->k_lim, m->list_base);
    };
    // (a level that may turn out empty leaves its list lengths to the scan)
    if (out->n_host > 0 && m->n_tiles <= WS_TILES_IN_FILL && int64_t(m->n_tiles) * m->k_lim <= WS_SCAN_IN_FILL) {
      fill(std::true_type{});
    } else {
      hipLaunchKernelGGL(ws_scan_kernel, dim3(m->K3), dim3(WS_SCAN_THREADS), 0, s, m->tile_counts, m->n_tiles, m->tile, n_out_h,
                         out->n_dev, m->nnz_dev, m->k_lim);
      if (m->n_tiles > 0) fill(std::false_type{});
    }
    if (m->sym) launch_list_base(m, m->ws_in, m->k_lim, out, m->list_base_in, s);
    // the slabs are dead once the lists are filled: back to the cache (reuse is ordered behind this stream's work)
    pool_free(m->tile_pairs, s);
    pool_free(m->tile_sub, s);
    m->tile_pairs = nullptr;
    m->tile_sub = nullptr;
  }
  if (hipGetLastError() != hipSuccess) return set_error(SPC_ERR_HIP, "kernel-map launch failed");
  return SPC_OK;
}

// One map, searched on its own.
static int build_on_levels(Level* in, Level* out, const PackInfo& pi, const spc_layer_desc& l, const StreamId& s, spc_kmap** res,
                           const int32_t* in_perm = nullptr, bool want_inverse = false) {
  const StreamWorkNote note{s};
  spc_kmap* m = nullptr;
  SPC_RETURN_IF(prepare_map(in, out, pi, l, s, &m, in_perm, want_inverse));
  const int rc = search_maps(&m, 1, s);
  if (rc != SPC_OK) {
    kmap_free(m);
    return rc;
  }
  *res = m;
  return SPC_OK;
}

// A strided layer whose offsets partition its inputs (K = layer stride, even K: offsets {0..K-1} * in_stride) can
// hand its pairs to the transposed layer of the same geometry instead of a second search.
static bool twin_can_share(const spc_layer_desc& strided, const spc_layer_desc& transposed) {
  return !strided.transposed && transposed.transposed && strided.K == transposed.K && strided.in_stride == transposed.in_stride &&
         strided.layer_stride == transposed.layer_stride && strided.K == strided.layer_stride && strided.K % 2 == 0 &&
         strided.K * strided.K * strided.K <= 32;
}

// The transposed map from its strided twin, built on the same stream (see transposed_from_parent_kernel): the matrix from the twin's inverse,
// the lists by taking the twin's with inputs and outputs swapped (for a fixed offset both index sequences ascend
// together, so the order by output index is kept).  Returns SPC_ERR_UNSUPPORTED when the twin lacks what is needed.
static int prepare_from_twin(spc_kmap* twin, Level* coarse, Level* fine, const PackInfo& pi, const spc_layer_desc& l,
                             const StreamId& s, spc_kmap** res) {
  const bool with_os = (l.layout & SPC_LAYOUT_OS) != 0, with_ws = (l.layout & SPC_LAYOUT_WS) != 0;
  if (!twin_can_share(twin->desc, l) || (l.layout & ~SPC_LAYOUT_BOTH) || (with_os && !twin->inv_parent) ||
      (with_ws && (!(twin->desc.layout & SPC_LAYOUT_WS) || twin->hybrid_t || twin->sym)))
    return SPC_ERR_UNSUPPORTED;
  spc_kmap* m = new spc_kmap;
  m->pi = pi;
  m->desc = l;
  m->K3 = l.K * l.K * l.K;
  m->k_lim = m->K3;
  for (int k = 0; k < m->K3; ++k) {
    if (with_os) m->os_k.w[k >> 5] |= 1u << (k & 31);
    if (with_ws) m->ws_k.w[k >> 5] |= 1u << (k & 31);
  }
  m->stream = s;
  m->captured = stream_is_capturing(s);
  m->in_level = coarse;
  coarse->refs++;
  m->out_level = fine;
  fine->refs++;
  m->out_cap = fine->n_host >= 0 ? fine->n_host : fine->cap;
  m->tile = search_tile(l.K, m->out_cap, pi.key_bits, (l.layout & SPC_LAYOUT_WS) != 0);
  m->n_tiles = static_cast<int>((m->out_cap + m->tile - 1) / m->tile);
  m->n_blocks_cap = (m->out_cap + 31) / 32;
  m->mask_words = 1;
  m->twin = twin;
  twin->refs++;
  int rc = SPC_OK;
  if (with_os) {
    m->os_map = static_cast<int32_t*>(pool_alloc(std::max<size_t>(size_t(m->n_blocks_cap) * 32 * m->K3 * 4, 256), s));
    m->block_masks = static_cast<uint32_t*>(pool_alloc(std::max<size_t>(size_t(m->n_blocks_cap) * 4, 256), s));
    m->arrived = static_cast<int32_t*>(pool_alloc(SHARED_TILES * 4, s));
    if (!m->os_map || !m->block_masks || !m->arrived) rc = SPC_ERR_NOMEM;
  }
  if (rc == SPC_OK && with_ws) {
    m->ws_in = twin->ws_out;
    m->ws_out = twin->ws_in;
    m->nnz_dev = twin->nnz_dev;
    m->ws_stride = twin->ws_stride;
    m->list_base = static_cast<int32_t*>(pool_alloc(size_t(m->n_blocks_cap + 1) * m->K3 * 4, s));
    if (!m->list_base) rc = SPC_ERR_NOMEM;
  }
  if (rc != SPC_OK) {
    kmap_free(m);
    return rc;
  }
  *res = m;
  return SPC_OK;
}

// The matrices and list tables of prepared transposed maps (their twins have been searched on the same stream before).
static int fill_from_twins(spc_kmap* const* ms, int count, hipStream_t s) {
  for (int first = 0; first < count; first += SEARCH_BATCH) {
    const int n = std::min(count - first, SEARCH_BATCH);
    TransposedBatch b{};
    int64_t rows = 0;
    for (int i = 0; i < n; ++i) {
      const spc_kmap* m = ms[first + i];
      const Level* fine = m->out_level;
      if (m->list_base) launch_list_base(m, m->ws_out, m->K3, fine, m->list_base, s);
      if (!m->os_map) continue;  // lists only: the twin's (its argument entry has no rows)
      b.a[i] = TransposedArgs{m->twin->inv_parent, fine->n_host < 0 ? fine->n_dev : nullptr,
                              static_cast<int>(fine->n_host < 0 ? 0 : fine->n_host), m->K3, m->os_map, m->block_masks, m->arrived};
      rows = std::max(rows, m->out_cap);
    }
    if (rows > 0)
      hipLaunchKernelGGL(transposed_from_parent_kernel, dim3(static_cast<unsigned>((rows + 255) / 256), n), dim3(256), 0, s, b);
  }
  if (hipGetLastError() != hipSuccess) return set_error(SPC_ERR_HIP, "kernel-map launch failed");
  return SPC_OK;
}

static Level* borrowed_level(const void* keys, int64_t n, int stride) {
  Level* lv = new Level;
  lv->keys = const_cast<void*>(keys);
  lv->owns_keys = false;
  lv->cap = n;
  lv->presumed = n;
  lv->n_host = n;
  lv->stride = stride;
  return lv;
}

// Waits for what a build has enqueued on its stream (a stream that is being captured by now cannot be waited for on
// its own, nor another thread's hipStreamPerThread: the device is drained).
static int wait_stream(bool captured, const StreamId& s) {
  const DeviceScope scope(s.device);
  if (captured || !s.here() || stream_is_capturing(s)) SPC_HIP_CHECK(hipDeviceSynchronize());
  else SPC_HIP_CHECK(hipStreamSynchronize(s));
  return SPC_OK;
}

// Waits until the level's count shows up in its pinned slot (see CountNote): spinning for POLL_SPIN, which covers the level of
// a few million voxels on an idle stream, then, behind whatever else the stream has to do, looking again after pauses of a
// sixteenth of the time waited so far (1 ms at most).  False when the stream has nothing left to run, or reports an error, and
// the count is not there: the caller then waits and copies, which reports what happened.
constexpr std::chrono::microseconds POLL_SPIN{1000}, POLL_MOST{1000};
static bool poll_count(Level* lv, int* v) {
  using Clock = std::chrono::steady_clock;
  auto seen = [&]() {
    const unsigned long long x = __atomic_load_n(lv->slot.host, __ATOMIC_ACQUIRE);
    *v = static_cast<int>(static_cast<uint32_t>(x));
    return static_cast<uint32_t>(x >> 32) == lv->slot.tag;
  };
  const Clock::time_point start = Clock::now();
  for (;;) {
    for (int spin = 0; spin < 64; ++spin) {
      if (seen()) return true;
      __builtin_ia32_pause();
    }
    const auto waited = Clock::now() - start;
    if (waited < POLL_SPIN) continue;
    if (!lv->stream.here() || stream_is_capturing(lv->stream)) return false;
    const DeviceScope scope(lv->stream.device);
    const hipError_t e = hipStreamQuery(lv->stream);
    if (e != hipErrorNotReady) {
      (void)hipGetLastError();
      return seen();
    }
    std::this_thread::sleep_for(std::min<Clock::duration>(waited / 16, POLL_MOST));
  }
}

// Host copy of a level's voxel count in lv->n_fetched.  A level built under stream capture is
// rewritten by every replay of the graph: its events cannot be waited for (they belong to the
// capture), so the whole device is drained instead, and the value is never cached.
static int fetch_level_n(Level* lv) {
  if (lv->n_host >= 0) {
    lv->n_fetched = lv->n_host;
    return SPC_OK;
  }
  int v = 0;
  if (lv->announced && poll_count(lv, &v)) {
    lv->n_host = lv->n_fetched = v;
    return SPC_OK;
  }
  SPC_RETURN_IF(wait_stream(lv->captured, lv->stream));
  SPC_HIP_CHECK(hipMemcpy(&v, lv->n_dev, sizeof(int), hipMemcpyDeviceToHost));
  lv->n_fetched = v;
  if (!lv->captured) lv->n_host = v;
  return SPC_OK;
}

// Waits until the map's arrays are complete (see fetch_level_n for captured builds).
static int wait_map(const spc_kmap* m) { return wait_stream(m->captured, m->stream); }

// Layout every distinct map of a network is built with: the union of what its layers ask for; a map
// shared by layers that disagree about the half-map keeps the full lists.
using NetKey = std::tuple<int, int, int, int>;
static NetKey net_key(const spc_layer_desc& l) { return NetKey(l.K, l.in_stride, l.layer_stride, l.transposed); }
static std::map<NetKey, int> net_layouts(const spc_layer_desc* layers, int n_layers) {
  std::map<NetKey, int> want;
  for (int i = 0; i < n_layers; ++i) want[net_key(layers[i])] |= layers[i].layout & 0xff;
  // a hybrid threshold survives only if every layer that shares the map asks for that same threshold
  for (auto& kv : want) {
    int thr = -1;
    for (int i = 0; i < n_layers; ++i)
      if (net_key(layers[i]) == kv.first) {
        const int t = (layers[i].layout >> 8) & 0xff;
        thr = thr < 0 ? t : (thr == t ? t : 0);
      }
    if (thr > 0) kv.second |= thr << 8;
  }
  for (auto& kv : want) {
    bool all_sym = true;
    for (int i = 0; i < n_layers; ++i)
      if (net_key(layers[i]) == kv.first && (layers[i].layout & SPC_LAYOUT_WS) && !(layers[i].layout & SPC_LAYOUT_WS_SYM))
        all_sym = false;
    if (!all_sym) kv.second &= ~SPC_LAYOUT_WS_SYM;
  }
  return want;
}

// ---------------------------------------------------------------- network builds
// All levels of a network come straight from V_0 (closed form, Section 5.5) and therefore from the same launches, and its
// maps are independent of each other given the levels: maps of one kernel size are searched by one launch, transposed
// maps derived from their strided twins by another.  A 25-layer UNet is built by 5 + 3 launches instead of 33, on one
// stream: with a launch per level and map, events tied three streams together and the host spent 206 us on it (120 k
// voxels); the levels took 110 us of GPU time and take 35.
struct NetBuild {
  const PackInfo& pi;
  std::map<NetKey, int> want;       // layout every distinct map is built with
  std::map<int, Level*> levels;     // stride -> level
  std::map<NetKey, spc_kmap*> maps;
  NetBuild(const PackInfo& p, const void* v0_keys, int64_t n0, const spc_layer_desc* layers, int n_layers)
      : pi(p), want(net_layouts(layers, n_layers)) {
    levels[1] = borrowed_level(v0_keys, n0, 1);
  }
  ~NetBuild() {  // drops the builder's own references
    for (auto& kv : maps)
      if (kv.second->refs.fetch_sub(1) == 1) kmap_free(kv.second);
    for (auto& kv : levels) level_unref(kv.second);
  }

  // The levels the layers [0, n) need and nobody has made yet.
  int make_levels(const spc_layer_desc* layers, int n, const StreamId& s) {
    std::vector<int> ms;
    std::set<int> seen;
    for (int i = 0; i < n; ++i)
      for (int stride : {layers[i].in_stride, layers[i].in_stride * layers[i].layer_stride})
        if (!levels.count(stride) && seen.insert(stride).second) ms.push_back(ilog2(stride));
    if (ms.empty()) return SPC_OK;
    std::vector<Level*> made(ms.size());
    SPC_RETURN_IF(downsample_levels(levels[1]->keys, levels[1]->n_host, 1, pi, ms.data(), static_cast<int>(ms.size()), made.data(), s));
    for (Level* lv : made) levels[lv->stride] = lv;
    return SPC_OK;
  }

  // The distinct maps of layers [0, n) that nobody has made yet, in the order of first use, `most` at a launch (1: every
  // map is searched by a launch of its own).
  // A transposed layer whose strided twin has been built on the same stream takes the twin's pairs; a strided
  // layer with such a transposed twin among the wanted maps leaves its inverse behind for it.
  int make_maps(const spc_layer_desc* layers, int n, const StreamId& s, int most) {
    const StreamWorkNote note{s};
    using Group = std::tuple<int, int, bool>;  // kernel size, tile length, lists
    std::vector<std::pair<Group, std::vector<spc_kmap*>>> groups;
    std::vector<std::pair<NetKey, spc_layer_desc>> transposed;
    int rc = SPC_OK;
    auto enter = [&](const NetKey& key, spc_kmap* m) {
      maps[key] = m;
      const Group g(m->desc.K, m->tile, (m->desc.layout & SPC_LAYOUT_WS) != 0);
      for (auto& kv : groups)
        if (kv.first == g && static_cast<int>(kv.second.size()) < most) {
          kv.second.push_back(m);
          return;
        }
      groups.push_back({g, {m}});
    };
    for (int i = 0; i < n && rc == SPC_OK; ++i) {
      const NetKey key = net_key(layers[i]);
      if (maps.count(key)) continue;
      spc_layer_desc l = layers[i];
      l.layout = want.at(key);
      if (l.transposed) {
        bool listed = false;
        for (auto& t : transposed) listed |= t.first == key;
        if (!listed) transposed.push_back({key, l});
        continue;
      }
      spc_layer_desc t = l;
      t.transposed = 1;
      const bool inverse = want.count(net_key(t)) != 0 && twin_can_share(l, t);
      spc_kmap* m = nullptr;
      rc = prepare_map(levels[l.in_stride], levels[l.in_stride * l.layer_stride], pi, l, s, &m, nullptr, inverse);
      if (rc == SPC_OK) enter(key, m);
    }
    std::vector<spc_kmap*> derived;
    for (size_t i = 0; i < transposed.size() && rc == SPC_OK; ++i) {
      const NetKey& key = transposed[i].first;
      const spc_layer_desc& l = transposed[i].second;
      Level* fine = levels[l.in_stride];
      Level* coarse = levels[l.in_stride * l.layer_stride];
      auto it = maps.find(NetKey(l.K, l.in_stride, l.layer_stride, 0));
      spc_kmap* m = nullptr;
      rc = SPC_ERR_UNSUPPORTED;
      if (it != maps.end() && it->second->stream == s) rc = prepare_from_twin(it->second, coarse, fine, pi, l, s, &m);
      if (rc == SPC_OK) {
        maps[key] = m;
        derived.push_back(m);
      } else if (rc == SPC_ERR_UNSUPPORTED) {
        rc = prepare_map(coarse, fine, pi, l, s, &m, nullptr, false);
        if (rc == SPC_OK) enter(key, m);
      }
    }
    for (auto& kv : groups)
      if (rc == SPC_OK) rc = search_maps(kv.second.data(), static_cast<int>(kv.second.size()), s);
    for (size_t i = 0; i < derived.size() && rc == SPC_OK; i += most)
      rc = fill_from_twins(derived.data() + i, static_cast<int>(std::min<size_t>(derived.size() - i, most)), s);
    return rc;
  }

  // Consumers on streams other than s wait for the maps (each stream once).
  int mark_ready(hipStream_t s) {
    auto r = std::make_shared<MapsReady>();
    if (hipEventCreateWithFlags(&r->e, hipEventDisableTiming) != hipSuccess || hipEventRecord(r->e, s) != hipSuccess)
      return set_error(SPC_ERR_HIP, "event record failed");
    for (auto& kv : maps) kv.second->ready = r;
    return SPC_OK;
  }

  void hand_out(const spc_layer_desc* layers, int n_layers, spc_kmap** out) {
    for (int i = 0; i < n_layers; ++i) {
      out[i] = maps[net_key(layers[i])];
      out[i]->refs++;
    }
  }
};

}  // namespace spc

using namespace spc;

extern "C" {

int spc_build_kmap(const void* in_keys, int64_t n_in, const spc_pack_desc* d, const spc_layer_desc* l, spc_kmap** out,
                   void* stream) {
  return spc_build_kmap_perm(in_keys, n_in, nullptr, d, l, out, stream);
}

int spc_build_kmap_perm(const void* in_keys, int64_t n_in, const int32_t* in_perm, const spc_pack_desc* d,
                        const spc_layer_desc* l, spc_kmap** out, void* stream) {
  PackInfo pi;
  SPC_RETURN_IF(check_desc(d, &pi));
  SPC_RETURN_IF(check_layer(l));
  SPC_RETURN_IF(check_desc_layer(d, l));
  if (!out) return set_error(SPC_ERR_ARG, "out is NULL");
  if (n_in < 0 || n_in > 0x7fffffff || (!in_keys && n_in > 0)) return set_error(SPC_ERR_ARG, "bad in_keys / n_in");
  if (int64_t(n_in) * l->K * l->K * l->K > (int64_t(1) << 40)) return set_error(SPC_ERR_ARG, "map too large");
  const StreamId s(static_cast<hipStream_t>(stream));
  Level* given = borrowed_level(in_keys, n_in, l->in_stride);
  Level* derived = nullptr;
  int rc = SPC_OK;
  const int m = ilog2(l->in_stride * l->layer_stride);
  if (l->layer_stride > 1) rc = downsample_levels(in_keys, n_in, l->in_stride, pi, &m, 1, &derived, s);
  if (rc == SPC_OK) {
    if (in_perm && l->transposed) rc = set_error(SPC_ERR_ARG, "in_perm applies to the given level, which a transposed layer writes");
    else if (in_perm && (l->layout & SPC_LAYOUT_WS_SYM))
      rc = set_error(SPC_ERR_ARG, "a symmetric half-map swaps inputs and outputs: both must be numbered alike (no in_perm)");
    else if (l->layer_stride == 1) rc = build_on_levels(given, given, pi, *l, s, out, in_perm);
    else if (!l->transposed) rc = build_on_levels(given, derived, pi, *l, s, out, in_perm);
    else rc = build_on_levels(derived, given, pi, *l, s, out);
  }
  level_unref(given);
  level_unref(derived);
  return rc;
}

int spc_build_kmaps_network(const void* v0_keys, int64_t n0, const spc_pack_desc* d, const spc_layer_desc* layers,
                            int32_t n_layers, spc_kmap** out, void* const* streams, int32_t n_streams, int32_t flags) {
  PackInfo pi;
  SPC_RETURN_IF(check_desc(d, &pi));
  if (!layers || !out || n_layers < 1) return set_error(SPC_ERR_ARG, "layers/out NULL or n_layers < 1");
  if (!streams || n_streams < 1) return set_error(SPC_ERR_ARG, "at least one stream is required");
  if (n0 < 0 || n0 > 0x7fffffff || (!v0_keys && n0 > 0)) return set_error(SPC_ERR_ARG, "bad v0_keys / n0");
  for (int i = 0; i < n_layers; ++i) {
    SPC_RETURN_IF(check_layer(&layers[i]));
    SPC_RETURN_IF(check_desc_layer(d, &layers[i]));
  }
  // Everything runs on streams[0].  Spread over several streams, or pipelined against the feature layers with a stream
  // each for levels and searches, the same launches were slower at every size measured (a replayed 25-layer UNet step,
  // three streams / one: 20 k voxels 378 / 316 us, 120 k 507 / 457, 200 k 610 / 568, 10^6 5339 / 5325): an edge between
  // two streams costs about 14 us, and the batched launches leave little to overlap.
  const StreamId s(static_cast<hipStream_t>(streams[0]));
  NetBuild b(pi, v0_keys, n0, layers, n_layers);
  if (flags & SPC_NET_SEQUENTIAL) {  // a launch per level and per map, in the order of first use
    for (int i = 0; i < n_layers; ++i) {
      SPC_RETURN_IF(b.make_levels(layers + i, 1, s));
      SPC_RETURN_IF(b.make_maps(layers + i, 1, s, 1));
    }
  } else {
    SPC_RETURN_IF(b.make_levels(layers, n_layers, s));
    SPC_RETURN_IF(b.make_maps(layers, n_layers, s, SEARCH_BATCH));
  }
  if (flags & SPC_NET_PIPELINED) SPC_RETURN_IF(b.mark_ready(s));
  b.hand_out(layers, n_layers, out);
  return SPC_OK;
}

int spc_kmap_set_size_hint(spc_kmap* m, int64_t n_out_hint) {
  if (!m || n_out_hint < 0) return set_error(SPC_ERR_ARG, "map is NULL or hint < 0");
  m->n_out_hint = n_out_hint;
  return SPC_OK;
}

void spc_kmap_destroy(spc_kmap* m) {
  if (m && m->refs.fetch_sub(1) == 1) kmap_free(m);
}

int64_t spc_kmap_n_in(spc_kmap* m) {
  if (!m) return set_error(SPC_ERR_ARG, "map is NULL");
  int rc = fetch_level_n(m->in_level);
  return rc != SPC_OK ? rc : m->in_level->n_fetched;
}
int64_t spc_kmap_n_out(spc_kmap* m) {
  if (!m) return set_error(SPC_ERR_ARG, "map is NULL");
  int rc = fetch_level_n(m->out_level);
  return rc != SPC_OK ? rc : m->out_level->n_fetched;
}
int32_t spc_kmap_kvol(const spc_kmap* m) { return m ? m->K3 : SPC_ERR_ARG; }
const void* spc_kmap_out_keys(const spc_kmap* m) { return m ? m->out_level->keys : nullptr; }
const void* spc_kmap_in_keys(const spc_kmap* m) { return m ? m->in_level->keys : nullptr; }
const int32_t* spc_kmap_os_map(const spc_kmap* m) { return (m && (m->desc.layout & SPC_LAYOUT_OS)) ? m->os_map : nullptr; }

int spc_kmap_copy_out_keys(spc_kmap* m, void* keys_host, int64_t cap) {
  if (!m || !keys_host) return set_error(SPC_ERR_ARG, "NULL argument");
  SPC_RETURN_IF(wait_map(m));
  SPC_RETURN_IF(fetch_level_n(m->out_level));
  const int64_t n = m->out_level->n_fetched;
  if (cap < n) return set_error(SPC_ERR_ARG, "room for %lld keys, map has %lld", (long long)cap, (long long)n);
  if (n > 0) SPC_HIP_CHECK(hipMemcpy(keys_host, m->out_level->keys, size_t(n) * (m->pi.key_bits / 8), hipMemcpyDeviceToHost));
  return SPC_OK;
}

int spc_kmap_ws_lists(const spc_kmap* m, const int32_t** in_idx, const int32_t** out_idx, const int32_t** nnz_dev,
                      int64_t* ws_stride) {
  if (!m) return set_error(SPC_ERR_ARG, "map is NULL");
  if (!(m->desc.layout & SPC_LAYOUT_WS)) return set_error(SPC_ERR_ARG, "map was built without the WS layout");
  if (in_idx) *in_idx = m->ws_in;
  if (out_idx) *out_idx = m->ws_out;
  if (nnz_dev) *nnz_dev = m->nnz_dev;
  if (ws_stride) *ws_stride = m->ws_stride;
  return SPC_OK;
}

int spc_kmap_export_triples(spc_kmap* m, int32_t which, int32_t* triples, int64_t cap, int64_t* nnz_out) {
  if (!m || !nnz_out) return set_error(SPC_ERR_ARG, "NULL argument");
  if (which != SPC_LAYOUT_OS && which != SPC_LAYOUT_WS) return set_error(SPC_ERR_ARG, "which must be OS or WS");
  if (which == SPC_LAYOUT_WS && !(m->desc.layout & SPC_LAYOUT_WS)) return set_error(SPC_ERR_ARG, "WS layout was not built");
  if (which == SPC_LAYOUT_OS && !(m->desc.layout & SPC_LAYOUT_OS)) return set_error(SPC_ERR_ARG, "OS layout was not built");
  SPC_RETURN_IF(wait_map(m));
  SPC_RETURN_IF(fetch_level_n(m->out_level));
  const int64_t n_out = m->out_level->n_fetched;
  const int K3 = m->K3;
  int64_t nnz = 0;
  if (which == SPC_LAYOUT_OS) {
    std::vector<int32_t> M(size_t((n_out + 31) / 32) * 32 * K3);
    if (!M.empty()) SPC_HIP_CHECK(hipMemcpy(M.data(), m->os_map, M.size() * 4, hipMemcpyDeviceToHost));
    for (int k = 0; k < K3; ++k)
      for (int64_t i = 0; i < n_out && m->os_k.has(k); ++i) {  // (a hybrid map holds the dense offsets only)
        const int32_t j = M[((i >> 5) * K3 + k) * 32 + (i & 31)];
        if (j < 0) continue;
        if (nnz < cap && triples) {
          triples[3 * nnz] = k;
          triples[3 * nnz + 1] = j;
          triples[3 * nnz + 2] = static_cast<int32_t>(i);
        }
        ++nnz;
      }
  } else {
    std::vector<int32_t> cnt(K3);
    SPC_HIP_CHECK(hipMemcpy(cnt.data(), m->nnz_dev, size_t(K3) * 4, hipMemcpyDeviceToHost));
    std::vector<int32_t> a, b;
    const int kc = (K3 - 1) / 2;
    auto emit = [&](int k, int32_t in, int32_t out) {
      if (nnz < cap && triples) {
        triples[3 * nnz] = k;
        triples[3 * nnz + 1] = in;
        triples[3 * nnz + 2] = out;
      }
      ++nnz;
    };
    for (int k = 0; k < K3; ++k) {
      if (m->hybrid_t && m->os_k.has(k)) continue;  // a hybrid map keeps lists for the sparse offsets only
      // symmetric half-map: offset k > centre is the list of K^3-1-k with the roles swapped (both
      // index sequences of a list ascend, so the order by output index is kept); the centre pairs
      // every voxel with itself
      if (m->sym && k == kc) {
        for (int64_t i = 0; i < n_out; ++i) emit(k, static_cast<int32_t>(i), static_cast<int32_t>(i));
        continue;
      }
      const bool mirror = m->sym && k > kc;
      const int ks = mirror ? K3 - 1 - k : k;
      const int c = cnt[ks];
      if (c < 0 || c > m->ws_stride) return set_error(SPC_ERR_HIP, "corrupt WS count %d at offset %d", c, ks);
      a.resize(c);
      b.resize(c);
      if (c) {
        SPC_HIP_CHECK(hipMemcpy(a.data(), m->ws_in + int64_t(ks) * m->ws_stride, size_t(c) * 4, hipMemcpyDeviceToHost));
        SPC_HIP_CHECK(hipMemcpy(b.data(), m->ws_out + int64_t(ks) * m->ws_stride, size_t(c) * 4, hipMemcpyDeviceToHost));
      }
      for (int e = 0; e < c; ++e) emit(k, mirror ? b[e] : a[e], mirror ? a[e] : b[e]);
    }
  }
  *nnz_out = nnz;
  return SPC_OK;
}

int64_t spc_search_count(void) { return g_search_launches.load(std::memory_order_relaxed); }

int spc_kmap_search_info(const spc_kmap* m, int32_t* tile_rows, int32_t* window_keys) {
  if (!m) return set_error(SPC_ERR_ARG, "map is NULL");
  if (tile_rows) *tile_rows = m->tile;
  if (window_keys) *window_keys = m->desc.K * search_win_cap(m->tile);
  return SPC_OK;
}

int spc_kmap_nnz(spc_kmap* m, int64_t* nnz_host) {
  if (!m || !nnz_host) return set_error(SPC_ERR_ARG, "NULL argument");
  if (m->nnz_host.empty() || m->captured) {
    SPC_RETURN_IF(wait_map(m));
    SPC_RETURN_IF(fetch_level_n(m->out_level));
    std::vector<int64_t> cnt(m->K3, 0);
    if (m->hybrid_t) {  // dense offsets are counted in the matrix below, the others come from the lists' lengths
      std::vector<int32_t> c(m->K3);
      SPC_HIP_CHECK(hipMemcpy(c.data(), m->nnz_dev, size_t(m->K3) * 4, hipMemcpyDeviceToHost));
      const int kc = (m->K3 - 1) / 2;
      for (int k = 0; k < m->K3; ++k)
        if (!m->os_k.has(k)) cnt[k] = (m->sym && k == kc) ? m->out_level->n_fetched : c[(m->sym && k > kc) ? m->K3 - 1 - k : k];
    }
    if ((m->desc.layout & SPC_LAYOUT_WS) && !m->hybrid_t) {
      std::vector<int32_t> c(m->K3);
      SPC_HIP_CHECK(hipMemcpy(c.data(), m->nnz_dev, size_t(m->K3) * 4, hipMemcpyDeviceToHost));
      for (int k = 0; k < m->K3; ++k) cnt[k] = c[k];
      if (m->sym) {  // the second half mirrors the first, the centre pairs every voxel with itself
        const int kc = (m->K3 - 1) / 2;
        cnt[kc] = m->out_level->n_fetched;
        for (int k = kc + 1; k < m->K3; ++k) cnt[k] = cnt[m->K3 - 1 - k];
      }
    } else {
      const int64_t n_out = m->out_level->n_fetched;
      std::vector<int32_t> M(size_t((n_out + 31) / 32) * 32 * m->K3);
      if (!M.empty()) SPC_HIP_CHECK(hipMemcpy(M.data(), m->os_map, M.size() * 4, hipMemcpyDeviceToHost));
      for (int64_t i = 0; i < n_out; ++i)
        for (int k = 0; k < m->K3; ++k)
          if (m->os_k.has(k)) cnt[k] += M[((i >> 5) * m->K3 + k) * 32 + (i & 31)] >= 0;
    }
    m->nnz_host = cnt;
  }
  for (int k = 0; k < m->K3; ++k) nnz_host[k] = m->nnz_host[k];
  return SPC_OK;
}

}  // extern "C"
