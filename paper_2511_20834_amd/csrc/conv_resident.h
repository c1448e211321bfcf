// Feature kernel for 3x3x3 layers of many voxels whose weights fit a CU's LDS: up to 64 input channels (fp32: 32) by slabs of 32 or 64
// output channels, from the matrix, from lists, or either by offset.
//
// One workgroup of sixteen waves per CU stays for the whole launch.  It brings the slab's weights for all offsets into LDS once (54 KB for
// 32x32, 108 KB for 64x32 and 32x64), and from then on its waves go their own ways without a barrier: a wave, or two that share the
// offsets of a tile (a block of 32 output rows), walks (tile, offset) steps one after the other, across the ends of tiles.  A step's row
// numbers are requested four steps before it and its rows two, so that a wave waits for memory at the start of the launch and hardly
// ever again.  Rows are gathered several lanes to a row and swapped between lanes (conv_common.h); weights are read from LDS in
// operand order.  Two waves of a tile meet through a counter in LDS: one leaves its sums there, the other, in turns, adds them and stores.
//
// What it replaces where it is taken reads the weights of every (32-row block, offset) cell from L2 (split-k kernel: 120 k LiDAR voxels
// 64->64, lists, 3.7 M reads of 64 bytes from L2 against 1.8 M here) or through LDS in phases that all waves wait for (phase kernel).
// us, before / this: lists 64->64 120 k LiDAR 37.9 / 30.4, 200 k 57.6 / 43.1, 10^6 random 188 / 148; matrix 32->32 120 k 14.8 / 12.9,
// 10^6 65 / 48; 64->32 120 k 20.8 / 18.8, 10^6 120 / 67; 24->40 (plain weights) 70 k random 16.8 / 13.0, 10^6 136 / 61; 32->64 200 k LiDAR
// 31.2 / 23.3, random 26.3 / 20.2, 10^6 86 / 64; fp32 32->64 120 k 79 / 69, 10^6 507 / 394.
// What bounds it: the steps' chains (400 cycles alone on a SIMD: some 45 vector instructions, of which a third swap rows between
// lanes, LDS latency, two to four dependent matrix instructions) while a few full tiles last; on random scenes of 10^6 voxels the bytes
// (32->32: 166 MB compulsory in 44 us beside the launch).  Tried: four waves to a tile (120 k 32->32 14.6 against 12.9), a step's row numbers for
// two steps by one load (no change: the memory path is not what binds), lines of the map asked for a tile ahead (10^6 58 against 48).
#pragma once
#include "conv_common.h"

namespace spc {

constexpr int RES_WAVES = 16;
constexpr int RES_K3 = 27;
constexpr int RES_CHUNK = 16;  // tiles go to the XCDs in chunks: neighbours gather the same rows, and every XCD gets its share of dense regions
enum { RES_MATRIX = 0, RES_LISTS = 1, RES_BOTH = 2 };  // where the offsets' pairs come from

struct ResidentArgs {
  const int32_t* M;
  const uint32_t* block_masks;
  const int* n_out_d;
  const void *F, *W;
  void* out;
  int64_t ld_in, ld_out;
  const int32_t *l_in, *l_out, *l_base;
  int64_t l_stride;
  int n_out_h, K3, cin, cout, relu, nb_total, log_share, packed, vec_store;
  uint32_t row_bytes;
  uint32_t os_word, ws_word;  // offsets from the matrix, and from the lists
};

__host__ __device__ constexpr int resident_weight_bytes(int K3, int nkk, int NB) { return K3 * nkk * NB * 1024; }
// A group of waves (two, or one) has room for a block of 32 x 32 sums, or a wave on its own for their rows as they are stored.
__host__ __device__ constexpr int resident_slot(int elem, int log_share) { return elem == 2 && log_share == 0 ? 32 * 80 : 32 * 32 * 4; }
__host__ __device__ constexpr int resident_lds(int K3, int nkk, int NB, int elem, int log_share) {
  return resident_weight_bytes(K3, nkk, NB) + (RES_WAVES >> log_share) * resident_slot(elem, log_share) + 2 * RES_WAVES * 4 + 256;
}

// Waits until the counter has come to v.  (Both waves of a tile walk the same tiles, so whoever counts it up gets there.)
__device__ inline void lds_wait_for(const int* p, int v) {
  while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < v) __builtin_amdgcn_s_sleep(1);
  asm volatile("" ::: "memory");
}

template <typename T, int NB, int NKK, int FROM>
__global__ __launch_bounds__(64 * RES_WAVES) void conv_resident_kernel(const ResidentArgs a) {
  using V = typename Mfma<T>::V;
  using Ints = const SPC_GLOBAL int32_t*;
  constexpr int LPC = Mfma<T>::LPC, SLAB = 2 * LPC;
  constexpr bool LISTED = FROM != RES_MATRIX;
  constexpr int AHEAD = 2;  // steps between the request of rows and their use
  extern __shared__ __align__(16) unsigned char smem[];
  V* const sW = reinterpret_cast<V*>(smem);
  const int K3 = a.K3, cin = a.cin, cout = a.cout, log_share = a.log_share, share = 1 << log_share;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave >> log_share, member = wave & (share - 1);
  float* const slot = reinterpret_cast<float*>(smem + resident_weight_bytes(K3, NKK, NB) + group * resident_slot(sizeof(T), log_share));
  int* const counters = reinterpret_cast<int*>(smem + resident_weight_bytes(K3, NKK, NB) + (RES_WAVES >> log_share) * resident_slot(sizeof(T), log_share));
  int *const s_arrived = counters + group, *const s_done = counters + RES_WAVES + group;
  int* const s_junk = counters + 2 * RES_WAVES;
  const int n_out = a.n_out_d ? *a.n_out_d : a.n_out_h;
  const int n_tiles = (n_out + 31) >> 5, slab = blockIdx.y;
  // tiles of this group of waves, in order: j-th
  const int n_groups = (gridDim.x >> 3) * (RES_WAVES >> log_share), xcd = blockIdx.x & 7;
  const int group_in_xcd = group * (gridDim.x >> 3) + (blockIdx.x >> 3);
  auto tile_of = [&](int j) {
    const int t = j * n_groups + group_in_xcd;
    return ((t / RES_CHUNK) * 8 + xcd) * RES_CHUNK + t % RES_CHUNK;
  };
  Ints const M = (Ints)a.M, masks = (Ints)a.block_masks, l_in = (Ints)a.l_in, l_out = (Ints)a.l_out, l_base = (Ints)a.l_base;
  const T* __restrict__ F = static_cast<const T*>(a.F);
  const T* __restrict__ W = static_cast<const T*>(a.W);

  // Asks for a line per lane, so that the loads that follow find it in L2: to LDS, where nobody looks at it (the compiler does not know
  // of these loads).
  auto touch = [&](const int32_t* p) __attribute__((always_inline)) {
    const unsigned at = static_cast<unsigned>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) int*)s_junk));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(__builtin_amdgcn_readfirstlane(at)), "v"(p) : "memory", "m0");
  };
  // ---- steps: (tile, offset), in the order in which this wave takes them
  int mv = 0;            // (matrix) lane i: the mask of tile j with j % 64 == i
  int lf = 0, le = 0;    // (lists) lane k: where the next tile's pairs of offset k start and end
  int cf = 0, cn = 0;    // of the current one: where they start, how many
  auto load_masks = [&](int j0) {
    const int t = tile_of(j0 + lane);
    mv = t < n_tiles ? masks[t] & a.os_word : 0;
  };
  auto load_bounds = [&](int j) {
    const int t = tile_of(j);
    const int64_t at = int64_t(t < n_tiles ? t : 0) * K3 + min(lane, K3 - 1);
    lf = l_base[at];
    le = l_base[at + K3];
  };
  int g_j = -1, g_blk = 0;
  unsigned g_m = 0u;      // this wave's remaining offsets of the tile
  unsigned g_os = 0u;     // (both) offsets of the tile that come from the matrix
  const int32_t* g_rows = a.M;
  bool g_live = true;
  auto next_tile = [&]() __attribute__((always_inline)) {
    ++g_j;
    const int t = tile_of(g_j);
    g_live = t < n_tiles;
    g_m = 0u;
    if (!g_live) return;
    g_blk = t;
    unsigned m = 0u;
    if constexpr (FROM != RES_LISTS) {
      g_rows = a.M + int64_t(t) * (K3 * 32);
      if ((g_j & 63) == 0) load_masks(g_j);
      g_os = m = static_cast<unsigned>(__builtin_amdgcn_readlane(mv, g_j & 63));
    }
    if constexpr (LISTED) {
      cf = lf;
      cn = (a.ws_word >> lr) & 1u ? le - lf : 0;
      m |= static_cast<unsigned>(__ballot(lane < K3 && cn > 0));
      load_bounds(g_j + 1);
      const int64_t at = min(lane, K3 - 1) * a.l_stride + cf;  // (of the last tile at most the lists' end)
      if (cn > 0 && lane < K3) touch(a.l_out + at);
      if (cn > 0 && lane < K3) touch(a.l_in + at);
    }
    // every share-th of the offsets
    const bool mine = ((m >> lr) & 1u) && (__popc(m & ((1u << lr) - 1u)) & (share - 1)) == member;
    g_m = static_cast<unsigned>(__ballot(mine));
  };
  struct Step {
    int at;   // offset | VALID | LAST | LIVE | pairs (lists) << 16
    int blk;
  };
  constexpr int VALID = 256, LAST = 512, LIVE = 1024;
  int jj[AHEAD];                       // matrix: rows
  int prow[AHEAD], pval[AHEAD];        // lists: pairs
  auto request = [&](auto S_, Step& s) __attribute__((always_inline)) {
    constexpr int S = decltype(S_)::value;
    const bool valid = g_m != 0u;
    const int k = valid ? __builtin_ctz(g_m) : 0;
    s.at = k | (valid ? VALID : 0) | (g_live ? LIVE : 0);
    s.blk = g_blk;
    if constexpr (FROM != RES_LISTS) {
      const __amdgpu_buffer_rsrc_t m_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(g_rows), 0, K3 * 128, 0x00020000);
      jj[S] = __builtin_amdgcn_raw_buffer_load_b32(m_rsrc, lr * 4, k * 128, 0);
    }
    if constexpr (LISTED) {
      int64_t at = 0;
      int off = 0;
      if (valid && (FROM == RES_LISTS || !((g_os >> k) & 1u))) {
        const int n = __builtin_amdgcn_readlane(cn, k);
        s.at |= n << 16;
        at = k * a.l_stride + __builtin_amdgcn_readlane(cf, k);
        off = min(lr, n - 1);
      }
      prow[S] = (l_out + at)[off];
      pval[S] = (l_in + at)[off];
    }
    g_m &= g_m - 1u;
    if (g_m == 0u) {
      s.at |= LAST;
      if (g_live) next_tile();
    }
  };
  const __amdgpu_buffer_rsrc_t rows_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(F), 0, MAX_OFFSET, 0x00020000);
  const unsigned piece_off = NKK * 16 * lh + 16 * (lane & (NKK - 1));
  const unsigned past = (NKK * lh + (lane & (NKK - 1))) * LPC >= cin ? MAX_OFFSET : 0u;  // pieces behind the last channel
  V rows[AHEAD][NKK];
  unsigned offs[NKK];
  auto place = [&](auto S_, const Step& s) __attribute__((always_inline)) {
    constexpr int S = decltype(S_)::value;
    int idx;
    if constexpr (LISTED) {
      // (lanes behind the last pair repeat it)
      const int got = __builtin_amdgcn_ds_permute(((prow[S] & 31) | (lane & 32)) * 4, pval[S] + 1) - 1;
      idx = (s.at >> 16) > 0 ? got : -1;
      if (FROM == RES_BOTH && (s.at >> 16) == 0) idx = s.at & VALID ? jj[S] : -1;
    } else {
      idx = s.at & VALID ? jj[S] : -1;
    }
    const unsigned off = static_cast<unsigned>(idx) * a.row_bytes;
    static_for<NKK>([&](auto I_) { offs[decltype(I_)::value] = (group_lane<NKK, decltype(I_)::value>(off) + piece_off) | past; });
  };
  auto fetch = [&](auto S_) __attribute__((always_inline)) {
    constexpr int S = decltype(S_)::value;
#pragma unroll
    for (int i = 0; i < NKK; ++i) rows[S][i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rows_rsrc, offs[i], 0, 0));
  };

  if (FROM != RES_LISTS && tile_of(0) < n_tiles) touch(a.M + (int64_t(tile_of(0)) * K3 + min(lane, K3 - 1)) * 32);  // (before the masks are known)
  if constexpr (LISTED) load_bounds(0);
  next_tile();
  Step st[2 * AHEAD];  // of the step computed now, and those after it
  static_for<AHEAD>([&](auto S_) { request(S_, st[decltype(S_)::value]); });

  // ---- the weights of this slab of columns, for all offsets, in operand order
  {
    const int KK = (cin + SLAB - 1) / SLAB, total = K3 * NKK * NB;  // fragments
    if (a.packed) {
      // (straight to LDS; the compiler does not know of these loads)
      for (int f = wave; f < total; f += RES_WAVES) {
        const int nb = f % NB, kk = f / NB % NKK, k = f / NB / NKK;
        if (kk < KK) {
          const V* src = reinterpret_cast<const V*>(W) + ((int64_t(k) * KK + kk) * a.nb_total + slab * NB + nb) * 64 + lane;
          const unsigned at = static_cast<unsigned>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) V*)(sW + f * 64)));
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(__builtin_amdgcn_readfirstlane(at)), "v"(src) : "memory", "m0");
        } else {
          sW[f * 64 + lane] = V{};
        }
      }
    } else {
      const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(W), 0, static_cast<uint32_t>(K3) * cin * cout * uint32_t(sizeof(T)), 0x00020000);
      constexpr int U = 4;  // fragments in flight
      for (int f0 = wave; f0 < total; f0 += U * RES_WAVES) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int f = min(f0 + u * RES_WAVES, total - 1), nb = f % NB, kk = f / NB % NKK, k = f / NB / NKK;
          const int c0 = kk * SLAB + LPC * lh, col = (slab * NB + nb) * 32 + lr;
          const unsigned at = ((k * cin + c0) * cout + col) * unsigned(sizeof(T));
#pragma unroll
          for (int j = 0; j < LPC; ++j) {
            const unsigned o = c0 + j < cin && col < cout ? at + j * cout * unsigned(sizeof(T)) : MAX_OFFSET;
            if constexpr (sizeof(T) == 2) v[u][j] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(w_rsrc, o, 0, 0));
            else v[u][j] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(w_rsrc, o, 0, 0));
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) sW[min(f0 + u * RES_WAVES, total - 1) * 64 + lane] = v[u];
      }
    }
    if (tid < 2 * RES_WAVES) counters[tid] = 0;
  }
  static_for<AHEAD>([&](auto S_) {
    constexpr int S = decltype(S_)::value;
    place(S_, st[S]);
    request(S_, st[AHEAD + S]);
    __builtin_amdgcn_sched_barrier(0);
    fetch(S_);
    __builtin_amdgcn_sched_barrier(0);
  });
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(AHEAD * NKK) : "memory");  // (the weights are older than the last of these loads)
  __syncthreads();

  floatx16 acc[NB];
  auto clear = [&]() {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;
  };
  clear();
  const float least = a.relu ? 0.f : -__builtin_inff();
  float z = 0.f;  // NaN once this wave has stored NaN or infinity
  int n_done = 0; // tiles this group has finished
  auto finish = [&](int blk) __attribute__((always_inline)) {
    const int owner = n_done & (share - 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int q = n_done * NB + nb;
      float4* part = reinterpret_cast<float4*>(slot) + lane;
      if (member != owner) {
        lds_wait_for(s_done, q);
#pragma unroll
        for (int r = 0; r < 4; ++r) part[r * 64] = make_float4(acc[nb][4 * r], acc[nb][4 * r + 1], acc[nb][4 * r + 2], acc[nb][4 * r + 3]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_store(s_arrived, q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        continue;
      }
      if (log_share > 0) {
        lds_wait_for(s_arrived, q + 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float4 p = part[r * 64];
          acc[nb][4 * r] += p.x;
          acc[nb][4 * r + 1] += p.y;
          acc[nb][4 * r + 2] += p.z;
          acc[nb][4 * r + 3] += p.w;
        }
      }
      // (what depends on the lane and the pitch only is derived here each time: kept across the steps it would cost registers)
      int l4 = lane, pitch = static_cast<int>(a.ld_out);
      asm volatile("" : "+v"(l4), "+s"(pitch));
      const int left = n_out - blk * 32, col0 = (slab * NB + nb) * 32;
      T* o = static_cast<T*>(a.out) + int64_t(blk) * 32 * pitch + col0;
      auto value = [&](int r) __attribute__((always_inline)) {
        const float v = acc[nb][r];
        z = fmaf(v, 0.f, z);
        return from_f32<T>(v < least ? least : v);
      };
      if (a.vec_store) {
        // Through LDS, 16 bytes of a row per lane: a store of whatever width keeps the memory path as long as one of 16 bytes.
        constexpr int PITCH = sizeof(T) == 2 ? 40 : 32, PER_ROW = 32 / LPC, ROWS = 64 / PER_ROW;
        static_assert(32 * PITCH * sizeof(T) <= resident_slot(sizeof(T), 0), "the tile fits a slot");
        T* put = reinterpret_cast<T*>(slot) + 4 * (l4 >> 5) * PITCH + (l4 & 31);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) put[(8 * (r / 4) + r % 4) * PITCH] = value(r);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int row = l4 / PER_ROW, piece = l4 % PER_ROW;
        V v[32 / ROWS];
#pragma unroll
        for (int i = 0; i < 32 / ROWS; ++i) v[i] = *reinterpret_cast<const V*>(reinterpret_cast<const T*>(slot) + (i * ROWS + row) * PITCH + piece * LPC);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < 32 / ROWS; ++i)
          if (i * ROWS + row < left && col0 + piece * LPC < cout) *reinterpret_cast<V*>(o + int64_t(i * ROWS + row) * pitch + piece * LPC) = v[i];
      } else {
        const int rows_here = col0 + (l4 & 31) < cout ? left - 4 * (l4 >> 5) : 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rr = 8 * (r / 4) + r % 4;
          const T v = value(r);
          if (rr < rows_here) o[int64_t(rr + 4 * (l4 >> 5)) * pitch + (l4 & 31)] = v;
        }
      }
      if (log_share > 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_store(s_done, q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    ++n_done;
    clear();
  };
  auto step = [&](auto S_) __attribute__((always_inline)) {
    constexpr int S = decltype(S_)::value;
    const Step now = st[S];
    const V* Bk = sW + (now.at & 255) * (NKK * NB * 64) + (NKK == 1 ? lane : lh * (NKK / 2 * NB * 64) + lr);
    V bw[NKK][NB];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) bw[kk][nb] = Bk[NKK == 1 ? nb * 64 : (kk / 2 * NB + nb) * 64 + kk % 2 * 32];
    __builtin_amdgcn_sched_barrier(0);
    V x[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) x[kk] = rows[S][kk];
    rows_to_lanes(x);
    st[S] = st[AHEAD + S];
    place(S_, st[S]);
    request(S_, st[AHEAD + S]);
    __builtin_amdgcn_sched_barrier(0);
    fetch(S_);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = Mfma<T>::mma(x[kk], bw[kk][nb], acc[nb]);
    if ((now.at & (LAST | LIVE)) == (LAST | LIVE)) finish(now.blk);
  };
  // (no way out between the two: where they met again, the compiler would wait for loads that are under way on one of them only)
  while (st[0].at & LIVE) {
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no load to LDS is under way when the workgroup ends)
  if (__ballot(z != z)) {
    // outputs stored as NaN, from their own pairs (see conv_by_pairs)
#pragma unroll 1
    for (int j = member; j < n_done; j += share) {
      const int blk = tile_of(j);
#pragma unroll 1
      for (int e = 0; e < NB * 16; ++e) {
        const int rr = 8 * (e % 16 / 4) + e % 4, row = rr + 4 * lh, col = (slab * NB + e / 16) * 32 + lr;
        SPC_GLOBAL T* dst = (SPC_GLOBAL T*)a.out + (int64_t(blk) * 32 + row) * a.ld_out + col;
        float was = 0.f;
        if (blk * 32 + row < n_out && col < cout) was = static_cast<float>(*dst);
#pragma unroll 1
        for (unsigned long long todo = __ballot(was != was); todo; todo &= todo - 1) {
          const int l = __builtin_ctzll(todo), row_l = rr + 4 * (l >> 5), col_l = (slab * NB + e / 16) * 32 + (l & 31);
          auto in_row = [&](int k) -> int {
            if ((a.os_word >> k) & 1u) return (masks[blk] >> k) & 1 ? M[(int64_t(blk) * K3 + k) * 32 + row_l] : -1;
            if (!LISTED || !((a.ws_word >> k) & 1u)) return -1;
            const Ints tab = l_base + int64_t(blk) * K3 + k;
            const int64_t at = k * a.l_stride + tab[0] + lane;  // (a block has at most 32 pairs of an offset)
            int from = -1;
            if (lane < tab[K3] - tab[0] && l_out[at] == blk * 32 + row_l) from = l_in[at];
            const unsigned long long hit = __ballot(from >= 0);
            return hit ? __builtin_amdgcn_readlane(from, __builtin_ctzll(hit)) : -1;
          };
          const SPC_GLOBAL T *Fg = (const SPC_GLOBAL T*)F, *Wg = (const SPC_GLOBAL T*)W;
          const float v = a.packed ? conv_by_pairs<T, true>(in_row, K3, Fg, a.ld_in, Wg, cin, cout, a.nb_total, col_l)
                                   : conv_by_pairs<T, false>(in_row, K3, Fg, a.ld_in, Wg, cin, cout, a.nb_total, col_l);
          if (lane == l) *dst = from_f32<T>(a.relu ? fmaxf(v, 0.f) : v);
        }
      }
    }
  }
}

// ---------------------------------------------------------------- dispatch
static std::atomic<int64_t> g_resident_launches{0};  // see spc_resident_count

// Workgroups of a slab: one per CU for all slabs together, in equal numbers per XCD.
static int64_t resident_workgroups(int n_slabs) { return std::max<int64_t>(32 / n_slabs, 1) * 8; }

template <typename T, int NB, int NKK, int FROM>
static void launch_resident(const ConvArgs& a, int log_share) {
  ResidentArgs k{};
  k.M = a.m->os_map;
  k.block_masks = a.m->block_masks;
  k.n_out_d = a.n_out_d;
  k.F = a.F;
  k.W = a.W;
  k.out = a.out;
  k.ld_in = a.ld_in;
  k.ld_out = a.ld_out;
  k.l_in = a.m->ws_in;
  k.l_out = a.m->ws_out;
  k.l_base = a.m->list_base;
  k.l_stride = a.m->ws_stride;
  k.n_out_h = a.n_out_h;
  k.K3 = a.m->K3;
  k.cin = a.cin;
  k.cout = a.cout;
  k.relu = a.relu;
  k.nb_total = (a.cout + 31) / 32;
  k.log_share = log_share;
  k.packed = a.packed;
  k.row_bytes = static_cast<uint32_t>(a.ld_in * sizeof(T));
  k.os_word = a.os_mask.w[0];
  k.ws_word = a.ws_mask.w[0];
  const int lds = resident_lds(k.K3, NKK, NB, sizeof(T), log_share);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_resident_kernel<T, NB, NKK, FROM>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)attr;
  k.vec_store = a.cout % Mfma<T>::LPC == 0 && a.ld_out % Mfma<T>::LPC == 0 && reinterpret_cast<uintptr_t>(a.out) % 16 == 0;
  const int n_slabs = (k.nb_total + NB - 1) / NB;
  const int64_t tiles = (a.rows_cap + 31) / 32;
  const int64_t wgs = std::min<int64_t>((tiles + 7) / 8 * 8, resident_workgroups(n_slabs));
  hipLaunchKernelGGL((conv_resident_kernel<T, NB, NKK, FROM>), dim3(static_cast<unsigned>(wgs), n_slabs), dim3(64 * RES_WAVES), lds, a.s, k);
  g_resident_launches.fetch_add(1, std::memory_order_relaxed);
}

template <typename T, int NB, int NKK>
static void launch_resident_from(const ConvArgs& a, int log_share) {
  if (!a.any_ws) launch_resident<T, NB, NKK, RES_MATRIX>(a, log_share);
  else if (!a.any_os) launch_resident<T, NB, NKK, RES_LISTS>(a, log_share);
  else launch_resident<T, NB, NKK, RES_BOTH>(a, log_share);
}

// Whether a layer's slabs and rows give all CUs work.  Every workgroup brings the weights of its slab, and a slab's tiles go to the XCDs in chunks:
// with few rows some XCDs have a chunk more than others.  us, split-k kernel / this: plain 64->1056 (33 slabs: a second round) 5 k rows half-filled 66 / 83, random
// 32 / 45, packed 41 / 79; 64->544 (17: 136 workgroups) 30 k 123 / 132, random 54 / 61; fp32 32->1024 5 k 114 / 131, 32->2048 2 k 93 / 143, 32->544 30 k 314 / 493,
// random 126 / 204; but 64->800 (25: 200) 30 k 182 / 140, plain 32->2048 5 k 63 / 35, lists 64->1024 5 k 63 / 52, fp32 32->1024 8.2 k 182 / 138.
template <typename T>
static bool resident_fills(int64_t rows, int n_slabs) {
  const int64_t wgs = resident_workgroups(n_slabs) * n_slabs;
  return wgs <= 256 && wgs >= (sizeof(T) == 4 ? 240 : 192) && rows >= (sizeof(T) == 4 ? 8192 : 4096);
}

// Whether a layer is taken (or asked for: os_variant 3), from what it is and from the rows that its level presumably holds: the
// waves that share a tile are the order of the sums, which is to stay when the host learns the count between two calls.  us, other kernel /
// this, next to the lines (tiles of all slabs; L, R, I: LiDAR, random, indoor scenes; prepacked where nothing else is said and the layer takes that):
//   lists, 16 bits, from 2500 tiles  32->32 L 60 k 12.3 / 10.7, 90 k 15.2 / 12.9, R 130 k 17.0 / 13.9, I 100 k 14.3 / 12.5; 8->32 L 90 k 11.3 / 11.7, R 130 k 14.0 / 12.3, I 100 k
//       12.0 / 11.2; 32->64 L 90 k 20.6 / 16.6, R 130 k 22.6 / 16.6, I 100 k 19.3 / 15.9; plain 24->40 L 90 k 24.9 / 18.7, R 130 k 30.3 / 18.7, I 100 k 25.3 / 18.0
//     64 channels, even slabs of columns, from 4200  64->64 L 90 k 29.9 / 25.9, R 70 k 18.8 / 19.0, I 100 k 25.8 / 25.5; 64->128 40 k L 26.0 / 24.5, R 20.1 / 20.0, I 18.1 / 18.7
//   matrix, 16 bits, from 3000  32->32 L 130 k 14.9 / 13.5, R 12.9 / 11.9, I 100 k 11.2 / 10.4; 64->32 L 130 k 21.8 / 20.2, R 17.7 / 17.0, I 100 k 15.6 / 14.7; 48->96 40 k L 21.3 / 18.5,
//       R 16.6 / 16.1, I 14.8 / 14.0
//     whole slabs of 64 columns, from 4097, where one round of the phase kernel would not do  32->64 L 200 k 29.7 / 24.6, R 300 k 35.0 / 24.6, I 160 k 22.1 / 18.8; 16->128 L 90 k
//       24.4 / 18.9, R 70 k 19.5 / 13.8, I 100 k 21.3 / 17.4 (below: L 120 k 32->64 17.6 / 17.6, 40 k 16->128 10.4 / 11.2; never 64->64 or 64->128: L 120 k 24.8 / 27.3)
//     ragged columns, never prepacked, from 1600  24->40 L 60 k 17.3 / 14.4, R 70 k 16.1 / 13.5, I 60 k 14.1 / 12.8 (below: L 30 k 11.5 / 12.3, R 9.2 / 11.6); 8->40 52 k L 11.1 / 9.4,
//       R 10.2 / 8.9, I 9.9 / 8.9; 64->72 25 k L 28.0 / 17.7, I 15.2 / 12.9; 8->16 52 k L 7.6 / 7.8, R 6.9 / 7.2, I 9.5 / 7.0
//   fp32, from 2000  32->64 40 k L 38.4 / 34.2, R 30.2 / 26.9, I 26.2 / 24.4; 16->64 L 90 k 37.7 / 35.4, R 70 k 27.5 / 26.7, I 100 k 39.0 / 35.5; 32->128 L 25 k 48.4 / 41.7, I 27.3 / 25.8
//     odd slabs of columns, from 6000  32->32 L 200 k 61.7 / 61.2, R 300 k 79.7 / 72.6, I 300 k 76.5 / 69.4; 32->96 L 90 k 83.0 / 80.8, R 70 k 59.4 / 61.8, I 100 k 89.3 / 83.6
//       lists, from 3000  32->32 L 130 k 57.5 / 53.6, R 49.9 / 46.2, I 100 k 44.1 / 39.6
// Three slabs of input channels (16 bits 33 to 48, fp32 17 to 24) are gathered, read and multiplied as four, where the split-k kernel takes three.  So not in
//   fp32                  20->128 LiDAR 80 k 75.3 / 93.2, random 66.4 / 76.8, indoor 68.3 / 81.7; 24->64 49.6 / 52.1, 43.7 / 43.3, 44.6 / 45.8
//   lists, prepacked      64 columns at a time  48->64 LiDAR 90 k 25.2 / 25.4, random 70 k 16.9 / 18.9, indoor 100 k 22.9 / 25.3, half as many rows of a level of stride 2 12.4 / 16.4
//     (but plain 48->64 37.7 / 27.8, 26.3 / 21.2, 37.5 / 27.4); 40->32 80 k 17.6 / 17.1, 13.5 / 14.5, 14.1 / 14.3, 200 k as the others
//   matrix, ragged columns, one slab  40->8 52 k 13.4 / 14.7, 10.7 / 12.6, 9.8 / 12.1; 100 k 21.4 / 18.8, 16.6 / 15.8, 17.5 / 16.4
// 2x2x2 layers are over before the weights pay (50 k rows 64->64 9.8 / 12.3).
// A wave to a tile where there are tiles enough for all, two where not: 32->32 lists 45 k 12.3 / 9.5, 250 k 20.4 / 21.3, 10^6 51 / 60; with 64 columns at a time
// two have twice the sums to exchange: 32->64 lists 60 k 15.0 / 13.8, 75 k 16.2 / 16.7, 10^6 71 / 86.
template <typename T>
static bool conv_resident(const ConvArgs& a) {
  constexpr int LPC = Mfma<T>::LPC, ELEM = sizeof(T), LDS = 160 * 1024;
  const int K3 = a.m->K3, nb_total = (a.cout + 31) / 32;
  // (plain weights are read at offsets of 32 bits; packed ones need not be, but the choice is the same for both)
  if (K3 != RES_K3 || a.m->sym || by_channel<T>(a) || wide_weights<T>(a) || a.cin > 8 * LPC) return false;
  if (wide_rows<T>(a, a.m->in_level->cap)) return false;  // (by the level's bound: its count may be known from one call to the next)
  if (a.ld_out > INT32_MAX) return false;  // (the kernel's pitch)
  const int nkk = a.cin <= 2 * LPC ? 1 : a.cin <= 4 * LPC ? 2 : 4;
  const bool two = nb_total % 2 == 0 && nkk < 4;  // 64 columns at a time
  const int n_slabs = two ? nb_total / 2 : nb_total;
  const int64_t tiles = (a.m->out_level->presumed + 31) / 32 * n_slabs;
  const bool even = nb_total % 2 == 0;
  int64_t least;
  if (ELEM == 4) least = even ? 2000 : a.any_ws ? 3000 : 6000;
  else if (a.any_ws) least = even && !two ? 4200 : 2500;
  else if (a.cout % 64 == 0) least = two ? 4097 : INT64_MAX;
  else least = a.cout % 32 != 0 ? 1600 : 3000;
  if ((a.cin + 2 * LPC - 1) / (2 * LPC) == 3) {  // (a slab of four is empty)
    if (ELEM == 4) least = INT64_MAX;
    else if (a.any_ws && a.packed) least = even ? INT64_MAX : 6000;
    else if (!a.any_ws && a.cout % 32 != 0 && !even) least = 3000;
  }
  if (a.os_variant != 3 && (tiles < least || !resident_fills<T>(a.m->out_level->presumed, n_slabs))) return false;
  int log_share = a.splitk_rb ? a.splitk_rb - 1 : (ELEM == 2 && tiles >= 8000) || (two && tiles >= 2000) ? 0 : 1;
  if (resident_lds(K3, nkk, two ? 2 : 1, ELEM, log_share) > LDS) log_share = 1;
  if (resident_lds(K3, nkk, two ? 2 : 1, ELEM, log_share) > LDS) return false;
  if (nkk == 1) two ? launch_resident_from<T, 2, 1>(a, log_share) : launch_resident_from<T, 1, 1>(a, log_share);
  else if (nkk == 2) two ? launch_resident_from<T, 2, 2>(a, log_share) : launch_resident_from<T, 1, 2>(a, log_share);
  else launch_resident_from<T, 1, 4>(a, log_share);
  return true;
}
}  // namespace spc
