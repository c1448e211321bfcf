// What the feature kernels share: matrix instructions by type, row gathers that swap pieces between lanes, and
// outputs computed from their own pairs.
#pragma once
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "spc_internal.h"

namespace spc {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));

// One slab = the input channels of one operand register pair: lane l holds LPC consecutive channels (16 bytes) of row
// (A) or column (B) l%32, starting at LPC * (l/32).
template <typename T>
struct Mfma;
template <>
struct Mfma<_Float16> {
  using V = half8;
  static constexpr int LPC = 8;
  __device__ static inline floatx16 mma(V a, V b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};
template <>
struct Mfma<__bf16> {
  using V = bf16x8;
  static constexpr int LPC = 8;
  __device__ static inline floatx16 mma(V a, V b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
// fp32: the 32x32x2 instruction takes one channel per lane, so a slab of 8 channels is four of them (channels j and
// 4 + j together); products and sums are fp32 as in the vector unit, at the same peak rate, but a gathered row serves
// 32 output columns from one register.
template <>
struct Mfma<float> {
  using V = floatx4;
  static constexpr int LPC = 4;
  __device__ static inline floatx16 mma(V a, V b, floatx16 c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], c, 0, 0, 0);
    return c;
  }
};

template <typename T>
__device__ inline T from_f32(float v) { return static_cast<T>(v); }  // round to nearest even

// f(integral_constant<int,0>) ... f(integral_constant<int,N-1>): loops whose index must be a
// compile-time constant (register arrays that are never indexed dynamically)
template <int... S, typename Fn>
__device__ inline void static_for_impl(std::integer_sequence<int, S...>, Fn&& f) {
  (f(std::integral_constant<int, S>{}), ...);
}
template <int N, typename Fn>
__device__ inline void static_for(Fn&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

__device__ __align__(16) uint32_t g_zero_row[64];  // zero-initialised, never written

// Outputs that come out as NaN.  The matrix cores multiply whole 32-row cells: a row without a pair at an offset adds zero
// times the offset's weights, and the pooled way below adds every product row of a block to all of its rows, times zero or
// one.  Zero times infinity or NaN is NaN, so one such weight or feature would reach rows that have no pair with it.  All
// kernels therefore compute an output that came out as NaN once more, here, from its own pairs alone (whatever came in from
// outside them has made the sum NaN).  The test costs an instruction per output.
// A wave computes one output together (all lanes active, the same arguments in all): in_row(k) is the output row's input row
// at offset k, or a negative number.
template <typename T, bool PACKED, typename InRow>
__device__ inline float conv_by_pairs(const InRow& in_row, int K3, const SPC_GLOBAL T* F, int64_t ld_in, const SPC_GLOBAL T* W, int cin,
                                      int cout, int nb_total, int col) {
  float sum = 0.f;
#pragma unroll 1
  for (int k = 0; k < K3; ++k) {
    const int j = __builtin_amdgcn_readfirstlane(in_row(k));
    if (j < 0) continue;
#pragma unroll 1
    for (int c = threadIdx.x & 63; c < cin; c += 64) {
      const int64_t at = PACKED ? ((int64_t(k) * ((cin + 15) / 16) + c / 16) * nb_total + col / 32) * 512 + ((c & 8) * 4 + col % 32) * 8 + c % 8
                                : (int64_t(k) * cin + c) * cout + col;
      sum = fmaf(static_cast<float>(F[int64_t(j) * ld_in + c]), static_cast<float>(W[at]), sum);
    }
  }
#pragma unroll 1
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  return sum;
}
// The same for a wave's 32 x 32 NB accumulators, whose first `rows` rows have been stored (lane l holds column l%32, and row
// 0 of its registers is row 4*(l/32) at prow): by_pairs(row, column) replaces the NaNs.
template <typename T, int NB, typename ByPairs>
__device__ inline void redo_nan(const floatx16 (&acc)[NB], int rows, int lane, T* prow, int64_t ld_out, int relu, const ByPairs& by_pairs) {
  float z = 0.f;  // NaN if any of them is NaN or infinite
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) z = fmaf(acc[nb][r], 0.f, z);
  if (!__ballot(z != z)) return;
  unsigned nan = 0u;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) nan |= acc[nb][r] != acc[nb][r] ? 1u << (nb * 16 + r) : 0u;
#pragma unroll 1
  for (int b = 0; b < NB * 16; ++b) {
    const int rr = 8 * (b % 16 / 4) + b % 4, nb = b / 16;
#pragma unroll 1
    for (unsigned long long todo = __ballot((nan >> b) & 1u); todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo), row = rr + 4 * (l >> 5);
      if (row >= rows) continue;
      const float v = by_pairs(row, nb * 32 + (l & 31));
      if (lane == l) prow[rr * ld_out + nb * 32] = from_f32<T>(relu ? fmaxf(v, 0.f) : v);
    }
  }
}

// Gathers.  A CU's vector memory path takes a group of four lanes per cycle as long as the four read one 64-byte piece; four
// lanes with a row each take a cycle each.  Loaded in the MFMA's operand order, where neighbouring lanes hold neighbouring
// rows, rows arrive at 16 bytes per cycle and CU; with four lanes to 64 bytes of a row, at 50 (rows of 128 bytes at random
// places, resident in L2).  So four (or two) neighbouring lanes fetch the pieces of their rows one row after the other, and
// exchange them in registers when they are needed.
// Lanes 2i and 2i+1 (PAIR = 1) or 4i+j and 4i+j+2 (2), for both pairs of registers: the first keeps a and takes the second's a
// for its b, the second keeps b and takes the first's b for its a.  (Written by hand: the compiler takes twice the instructions.
// An instruction that reads other lanes' registers, or a matrix instruction, wants two slots between itself and the write.)
template <int PAIR>
__device__ inline void lane_exchange(intx4& a, intx4& b, intx4& c, intx4& d) {
  constexpr unsigned long long first = PAIR == 1 ? 0x5555555555555555ull : 0x3333333333333333ull;
  intx4 t, u;
#define SPC_EXCHANGE(PERM)                                                                                          \
  asm("s_mov_b64 vcc, %24\n\ts_nop 0\n\t"                                                                          \
      "v_cndmask_b32_dpp %0, %8, %16, vcc " PERM "\n\tv_cndmask_b32_dpp %1, %9, %17, vcc " PERM "\n\t"             \
      "v_cndmask_b32_dpp %2, %10, %18, vcc " PERM "\n\tv_cndmask_b32_dpp %3, %11, %19, vcc " PERM "\n\t"           \
      "v_cndmask_b32_dpp %4, %12, %20, vcc " PERM "\n\tv_cndmask_b32_dpp %5, %13, %21, vcc " PERM "\n\t"           \
      "v_cndmask_b32_dpp %6, %14, %22, vcc " PERM "\n\tv_cndmask_b32_dpp %7, %15, %23, vcc " PERM                   \
      : "=&v"(t.x), "=&v"(t.y), "=&v"(t.z), "=&v"(t.w), "=&v"(u.x), "=&v"(u.y), "=&v"(u.z), "=&v"(u.w)              \
      : "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w), "v"(d.x), "v"(d.y), "v"(d.z), "v"(d.w), "v"(a.x), "v"(a.y),         \
        "v"(a.z), "v"(a.w), "v"(c.x), "v"(c.y), "v"(c.z), "v"(c.w), "s"(first)                                      \
      : "vcc");                                                                                                     \
  asm("s_mov_b64 vcc, %16\n\ts_nop 0\n\t"                                                                          \
      "v_cndmask_b32_dpp %0, %8, %0, vcc " PERM "\n\tv_cndmask_b32_dpp %1, %9, %1, vcc " PERM "\n\t"               \
      "v_cndmask_b32_dpp %2, %10, %2, vcc " PERM "\n\tv_cndmask_b32_dpp %3, %11, %3, vcc " PERM "\n\t"             \
      "v_cndmask_b32_dpp %4, %12, %4, vcc " PERM "\n\tv_cndmask_b32_dpp %5, %13, %5, vcc " PERM "\n\t"             \
      "v_cndmask_b32_dpp %6, %14, %6, vcc " PERM "\n\tv_cndmask_b32_dpp %7, %15, %7, vcc " PERM "\n\ts_nop 1"     \
      : "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w), "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w)                      \
      : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(c.x), "v"(c.y), "v"(c.z), "v"(c.w), "s"(~first)                 \
      : "vcc")
  if constexpr (PAIR == 1) {
    SPC_EXCHANGE("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
  } else {
    SPC_EXCHANGE("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
  }
#undef SPC_EXCHANGE
  a = t;
  c = u;
}
// Lanes 2i and 2i+1, for one pair of registers.  (Phase kernel, 32 channels, exchanged as two pairs of which one is thrown away / so: 32->64 120 k LiDAR 18.9 / 18.0 us,
// random 16.6 / 15.5, 32->128 60 k 18.1 / 17.2, 10^6 random 87 / 87.)
__device__ inline void lane_exchange(intx4& a, intx4& b) {
  intx4 t;
  asm("s_mov_b64 vcc, %12\n\ts_nop 0\n\t"
      "v_cndmask_b32_dpp %0, %4, %8, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %1, %5, %9, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %2, %6, %10, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %3, %7, %11, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : "=&v"(t.x), "=&v"(t.y), "=&v"(t.z), "=&v"(t.w)
      : "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w), "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "s"(0x5555555555555555ull)
      : "vcc");
  asm("s_mov_b64 vcc, %8\n\ts_nop 0\n\t"
      "v_cndmask_b32_dpp %0, %4, %0, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %1, %5, %1, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %2, %6, %2, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_dpp %3, %7, %3, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\ts_nop 1"
      : "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w)
      : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "s"(~0x5555555555555555ull)
      : "vcc");
  a = t;
}
// Pieces as fetched (register i: a piece of the group's row i) to pieces as multiplied (register i: the lane's own row, piece i).
template <typename V, int N>
__device__ inline void rows_to_lanes(V (&v)[N]) {
  if constexpr (N == 1) return;
  intx4 x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = __builtin_bit_cast(intx4, v[i]);
  if constexpr (N == 4) {
    lane_exchange<1>(x[0], x[1], x[2], x[3]);
    lane_exchange<2>(x[0], x[2], x[1], x[3]);
  } else if constexpr (N == 2) {
    lane_exchange(x[0], x[1]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(V, x[i]);
}
// x of lane i of the N lanes that fetch together.
template <int N, int I>
__device__ inline unsigned group_lane(unsigned x) {
  constexpr int perm = N == 4 ? I * 0x55 : N == 2 ? I | (I << 2) | ((2 + I) << 4) | ((2 + I) << 6) : 0xe4;
  return static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), perm, 0xf, 0xf, true));
}
// Bytes that the 32-bit offsets of buffer loads may reach; beyond, they answer zeros.
constexpr uint32_t MAX_OFFSET = 0x80000000u;

struct ListArgs {
  const int32_t *in, *out;          // pairs, list k at k * stride
  const int32_t *base;              // [n_blocks + 1][K3]: first entry of list k whose output row is >= 32 * block
  const int32_t *base_in;           // symmetric half-map: the same by input row
  int64_t stride;
  int sym;
  KMask mask;
};

struct ConvArgs {
  int packed;
  spc_kmap* m;
  const void* F;
  int64_t ld_in;
  const void* W;
  void* out;
  int64_t ld_out;
  int cin, cout, relu;
  int os_variant;  // 0: chosen from the layer's size, 1: phase kernel, 2: split-k kernel, 3: resident weights
  int splitk_rb;   // 0: chosen from the layer's size, else row blocks per workgroup (1, 2)
  int n_out_h;
  const int* n_out_d;
  int64_t rows_cap;  // upper bound of the output rows (exact when the host knows the count)
  int64_t rows_sel;  // best host-side estimate of the output rows: kernel selection and launch shape only
  KMask os_mask, ws_mask;  // offsets of the output-stationary / weight-stationary part
  bool any_os, any_ws;
  StreamId s;
};

// Whether the feature rows are more than the 32-bit offsets of buffer loads reach.
template <typename T>
static bool wide_rows(const ConvArgs& a, int64_t rows) {
  return rows * a.ld_in * int64_t(sizeof(T)) > int64_t(MAX_OFFSET);
}
template <typename T>
static bool wide_rows(const ConvArgs& a) {
  const Level* il = a.m->in_level;
  return wide_rows<T>(a, il->n_host < 0 ? il->cap : il->n_host);
}

// Whether the weights are, in operand order (the plain ones are no more).
template <typename T>
static bool wide_weights(const ConvArgs& a) {
  constexpr int SLAB = 2 * Mfma<T>::LPC;
  return int64_t(a.m->K3) * ((a.cin + SLAB - 1) / SLAB) * ((a.cout + 31) / 32) * 1024 > int64_t(MAX_OFFSET);
}

// Whether the feature rows cannot be read in pieces of 16 bytes.
template <typename T>
static bool by_channel(const ConvArgs& a) {
  constexpr int LPC = Mfma<T>::LPC;
  return a.ld_in % LPC != 0 || reinterpret_cast<uintptr_t>(a.F) % 16 != 0 || a.cin % LPC != 0;
}

}  // namespace spc
