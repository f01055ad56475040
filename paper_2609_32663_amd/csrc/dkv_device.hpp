// Device-side helpers shared by the Distance-KV HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dkv {

constexpr int kWave = 64;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// bf16 halves of a 32-bit word, widened exactly to fp32.
__device__ __forceinline__ float bf16_lo(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t x) { return __uint_as_float(x & 0xffff0000u); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ---------------------------------------------------------------------------
// DPP reductions inside each 16-lane row of a wave.  quad_perm [1,0,3,2] and
// [2,3,0,1] combine within a quad, row_half_mirror pairs the two quads of an
// 8-lane half, row_mirror pairs the two halves; afterwards every lane of the
// row holds the row's result.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float row16_max(float x) {
  x = fmaxf(x, dpp_mov<0xB1>(x));
  x = fmaxf(x, dpp_mov<0x4E>(x));
  x = fmaxf(x, dpp_mov<0x141>(x));
  x = fmaxf(x, dpp_mov<0x140>(x));
  return x;
}

__device__ __forceinline__ float row16_sum(float x) {
  x += dpp_mov<0xB1>(x);
  x += dpp_mov<0x4E>(x);
  x += dpp_mov<0x141>(x);
  x += dpp_mov<0x140>(x);
  return x;
}

// Sum over the lanes of a wave that share (lane % FROM), FROM in {8, 16, 32}:
// lanes i and i ^ 8 meet through a rotation by 8 inside each 16-lane row,
// i ^ 16 and i ^ 32 through the permlane swaps (each swap exchanges half of
// one copy with the other half of a second copy, so adding the two copies
// gives every lane its partner's value).  Every lane ends with the sum.
template <int FROM>
__device__ __forceinline__ float lane_xor_sum(float x) {
  static_assert(FROM == 8 || FROM == 16 || FROM == 32, "unsupported stride");
  if constexpr (FROM <= 8) x += dpp_mov<0x128>(x);  // row_ror:8
  if constexpr (FROM <= 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Keeps the compiler from moving LDS accesses of one wave across this point.
// LDS instructions of a single wave execute in issue order, so no wait is
// needed between a lane's write and another lane's later read.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Block-wide exclusive scan of one int64 per thread.  `tmp` holds NT/64 + 1
// int64 in LDS.  Returns the exclusive prefix; *total receives the sum.
// Must be called by every thread of the block.
// ---------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* tmp, int64_t* total) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  int64_t x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    int64_t y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) tmp[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int w = 0; w < NW; ++w) {
      int64_t t = tmp[w];
      tmp[w] = run;
      run += t;
    }
    tmp[NW] = run;
  }
  __syncthreads();
  const int64_t excl = x - v + tmp[wave];
  *total = tmp[NW];
  __syncthreads();
  return excl;
}

// Workgroup that owns flat row x when `total` rows are cut into P slices
// [floor(w*total/P), floor((w+1)*total/P)).
// The quotient comes from an fp64 division (the numerator is below 2^53) and
// is corrected by one where rounding crossed an integer; a 64-bit integer
// division is a long emulated sequence.
__device__ __forceinline__ int64_t owner_of(int64_t x, int64_t total, int64_t P) {
  const int64_t num = (x + 1) * P - 1;
  int64_t w = (int64_t)((double)num / (double)total);
  if (w * total > num) --w;
  else if ((w + 1) * total <= num) ++w;
  return w < P - 1 ? w : P - 1;
}

// Number of nonzero bytes in a 32-bit word.
__device__ __forceinline__ int nonzero_bytes(uint32_t x) {
  uint32_t y = ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x;
  return __popc(y & 0x80808080u);
}

// Bit e set when byte e of the 16 bytes is nonzero: a word's four flags,
// gathered by a dot product of bytes with the bits' values.
__device__ __forceinline__ uint32_t nonzero_byte_bits(u32x4 w) {
  uint32_t f[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = ((((w[q] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w[q]) >> 7) & 0x01010101u;
  const uint32_t lo = __builtin_amdgcn_udot4(f[1], 0x80402010u, __builtin_amdgcn_udot4(f[0], 0x08040201u, 0u, false), false);
  const uint32_t hi = __builtin_amdgcn_udot4(f[3], 0x80402010u, __builtin_amdgcn_udot4(f[2], 0x08040201u, 0u, false), false);
  return hi << 8 | lo;
}

// Inclusive sum over the lanes of a wave: prefixes inside each 16-lane row by
// row shifts, then the last lane of rows 0 and 2 into the rows after them and
// of row 1 into rows 2 and 3.
template <int CTRL, int ROWS, int BANKS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, BANKS, false);
}

__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
  x = dpp_add<0x111, 0xF, 0xF>(x);  // row_shr:1
  x = dpp_add<0x112, 0xF, 0xF>(x);  // row_shr:2
  x = dpp_add<0x114, 0xF, 0xE>(x);  // row_shr:4
  x = dpp_add<0x118, 0xF, 0xC>(x);  // row_shr:8
  x = dpp_add<0x142, 0xA, 0xF>(x);  // row_bcast:15
  x = dpp_add<0x143, 0xC, 0xF>(x);  // row_bcast:31
  return x;
}

// Bit h set when query head h of a group keeps bin k; prow is the group's
// first pattern row (rows of D bytes).  Eight heads' loads are in flight at a
// time (heads past G repeat the last row): one load per memory round trip
// made eight heads cost six microseconds of a map call.  Groups of at most
// four, two and one head load four, two and one row instead of eight: one
// head with 8,192 bins of 16 15.2 us a map call by one row, 19.6 by eight.
template <int ROWS>
__device__ __forceinline__ uint32_t group_bits_of(const uint8_t* prow, int D, int G, int k) {
  uint32_t bits = 0;
  for (int h0 = 0; h0 < G; h0 += ROWS) {
    uint32_t b[ROWS];
#pragma unroll
    for (int e = 0; e < ROWS; ++e) b[e] = prow[(int64_t)(h0 + e < G ? h0 + e : G - 1) * D + k];
#pragma unroll
    for (int e = 0; e < ROWS; ++e) bits |= (h0 + e < G && b[e] != 0 ? 1u : 0u) << (h0 + e);
  }
  return bits;
}

__device__ __forceinline__ uint32_t group_bits(const uint8_t* prow, int D, int G, int k) {
  if (G == 1) return prow[k] != 0 ? 1u : 0u;
  if (G == 2) return group_bits_of<2>(prow, D, G, k);
  if (G <= 4) return group_bits_of<4>(prow, D, G, k);
  return group_bits_of<8>(prow, D, G, k);
}

// The 16 mask bytes of positions [j0, j0 + 16) of mask row `row` (rows of T
// bytes, `rows` of them, the first 16-byte aligned), zero beyond T; j0 is a
// multiple of 16.  Rows of odd lengths take the two aligned 16-byte blocks
// that hold the bytes (16 byte loads took the count and list passes of a
// 32 x 9,001 mask from 3.1 and 4.9 us to 3.9 and 5.7); only where a block
// would reach past the mask are the bytes read one by one.
__device__ __forceinline__ u32x4 load_mask16(const uint8_t* mask, int64_t row, int64_t rows, int64_t j0, int32_t T) {
  u32x4 w = {0u, 0u, 0u, 0u};
  if (j0 >= T) return w;
  const int64_t f = row * T + j0;
  const int sh = (int)(f & 15);  // the same for the whole row
  if (sh == 0 && j0 + 16 <= T) return *reinterpret_cast<const u32x4*>(mask + f);
  if (f - sh + 32 <= rows * T) {
    const u32x4* at = reinterpret_cast<const u32x4*>(mask + (f - sh));
    const u32x4 x = at[0], y = at[1];
    const uint32_t v[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    const int b = sh & 3;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if ((sh >> 2) == d) {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = __builtin_amdgcn_alignbyte(v[q + d + 1 < 8 ? q + d + 1 : 7], v[q + d], b);
      }
    const int64_t left = T - j0;  // bytes of the next row are not this row's
    if (left < 16) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = (int)left - 4 * q;
        if (n <= 0) w[q] = 0u;
        else if (n < 4) w[q] &= (1u << (8 * n)) - 1u;
      }
    }
    return w;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t j = j0 + e;
    const uint32_t c = (j < T && mask[row * T + j] != 0) ? 1u : 0u;
    w[e >> 2] |= c << (8 * (e & 3));
  }
  return w;
}

// ---------------------------------------------------------------------------
// Ranks over a mask row that one workgroup of kSweepThreads walks in sweeps
// of 16 positions per thread, kSweeps of them at a time (all their loads in
// flight together).
// ---------------------------------------------------------------------------
constexpr int kSweepThreads = 1024;
constexpr int kSweeps = 8;
constexpr int kSweepPositions = kSweepThreads * 16;
constexpr int64_t kPanelPositions = (int64_t)kSweeps * kSweepPositions;

// Keep bits of this thread's runs of a panel (bit e: position e of the run is
// kept).  Whole-row-aligned masks (T a multiple of 16) have all loads in
// flight together; others take two blocks per run, two runs at a time.
__device__ __forceinline__ void panel_bits(const uint8_t* mask, int64_t row, int64_t rows, int64_t base, int32_t T,
                                           uint32_t (&keep)[kSweeps]) {
  const int64_t j = base + (int64_t)threadIdx.x * 16;
  if ((T & 15) == 0) {
    u32x4 w[kSweeps];
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int c = 0; c < kSweeps; ++c) {
      const int64_t j0 = j + c * kSweepPositions;
      w[c] = j0 < T ? *reinterpret_cast<const u32x4*>(mask + row * T + j0) : z;
    }
#pragma unroll
    for (int c = 0; c < kSweeps; ++c) keep[c] = nonzero_byte_bits(w[c]);
  } else {
#pragma unroll
    for (int c = 0; c < kSweeps; c += 2) {
      const u32x4 x = load_mask16(mask, row, rows, j + c * kSweepPositions, T);
      const u32x4 y = load_mask16(mask, row, rows, j + (c + 1) * kSweepPositions, T);
      keep[c] = nonzero_byte_bits(x);
      keep[c + 1] = nonzero_byte_bits(y);
      __builtin_amdgcn_sched_barrier(0);  // two runs at a time: 1,024 threads have 128 registers
    }
  }
}

// cnt[c] (at most 16) becomes the number of marks before this thread's in
// sweep c, sweep-major; returns the marks of all sweeps.  `tmp` holds
// kSweeps * kSweepThreads / 64 words of LDS, free again after the caller's
// next barrier.  Called by every thread of the workgroup.
__device__ __forceinline__ int sweep_ranks(int (&cnt)[kSweeps], int32_t* tmp) {
  constexpr int NW = kSweepThreads / kWave;
  static_assert(NW * kSweeps == 2 * kWave, "two wave totals per lane");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
#pragma unroll
  for (int c = 0; c < kSweeps; c += 2) {  // two 16-bit sums per scan
    const uint32_t own = (uint32_t)cnt[c] | (uint32_t)cnt[c + 1] << 16;
    uint32_t x = wave_inclusive_sum(own);
    if (lane == kWave - 1) {
      tmp[c * NW + wave] = (int32_t)(x & 0xFFFFu);
      tmp[(c + 1) * NW + wave] = (int32_t)(x >> 16);
    }
    x -= own;
    cnt[c] = (int)(x & 0xFFFFu);
    cnt[c + 1] = (int)(x >> 16);
  }
  __syncthreads();
  const int a = tmp[2 * lane], b = tmp[2 * lane + 1];
  const int inc = (int)wave_inclusive_sum((uint32_t)(a + b));
  const int ex = inc - a - b;
#pragma unroll
  for (int c = 0; c < kSweeps; ++c) {
    const int at = (c * NW + wave) >> 1;
    cnt[c] += __builtin_amdgcn_readlane(ex, at) + ((wave & 1) ? __builtin_amdgcn_readlane(a, at) : 0);
  }
  return __builtin_amdgcn_readlane(inc, kWave - 1);
}

}  // namespace dkv
