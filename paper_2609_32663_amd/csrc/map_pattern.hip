// Pattern -> per-KV-head keep mask (Distance-KV, Sec. 3.4, Eq. (4)-(5) and the
// GQA union).
//
// One workgroup per (unit, KV head) segment and chunk of kMapChunk positions
// (a 128K context is 8 chunks, so the grid fills the chip).  The group's G
// pattern rows are folded into one G-bit word per bin in LDS (bit h = query
// head g*G+h keeps the bin), so the union over the group is "word != 0" and
// the per-head decision is one bit.  Each thread then owns 16 consecutive
// positions per sweep and walks the regions they cross (sink, a bin, recent
// window, uncovered, past the context; usually one): the first one's bin comes
// from a division for uniform edges, a binary search over the edges in LDS
// otherwise, the next bin is the one below.  Runs lie on the mask's 16-byte
// grid, so 16 mask bytes are one store.  The retained length is not counted
// from the mask: the first chunk of each segment writes it from the closed
// form of Eq. (4)-(5), |sink U recent| plus the width (clipped to the
// compressible span) of every bin some head of the group keeps, with one
// plain store, so the call is one kernel with no atomics or clearing pass.
// In a ragged batch a unit's context is the first unit_len[n] positions of
// its row: distances count from its end and the rest of the row is not
// retained.

#include <type_traits>

#include "dkv_device.hpp"
#include "dkv_launch.hpp"

namespace dkv {

namespace {

constexpr int kMapThreads = 256;
constexpr int kMapPerThread = 16;
constexpr int kMapChunk = 4 * kMapThreads * kMapPerThread;  // positions per workgroup

// Chunks per segment; at least one, whose workgroup writes the length.
__host__ __device__ inline int64_t map_chunks(int32_t T) {
  const int64_t c = ((int64_t)T + kMapChunk - 1) / kMapChunk;
  return c > 0 ? c : 1;
}

__device__ __forceinline__ int find_bin(int32_t u, const int32_t* edges, int D, int uniform_w) {
  if (uniform_w > 0) {
    const int32_t k = u / uniform_w;
    return k < D ? k : -1;
  }
  if (u >= edges[D]) return -1;
  int lo = 0, hi = D;  // edges[lo] <= u < edges[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (edges[mid] <= u) lo = mid; else hi = mid;
  }
  return lo;
}

// The 16 mask bytes of 16 keep bits.
__device__ __forceinline__ u32x4 mask_bytes(uint32_t keep) {
  u32x4 w;
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = (((keep >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
  return w;
}

typedef u32x4 __attribute__((aligned(1))) u32x4_bytes;  // 16 bytes anywhere

// Stores the 16 mask bytes of positions [j0, j0 + 16), those that are the
// row's; GRID: the address is a multiple of 16.
template <bool GRID>
__device__ __forceinline__ void store_run(uint8_t* row, int32_t j0, int32_t T, bool whole, u32x4 w) {
  if (whole) {
    if (GRID) *reinterpret_cast<u32x4*>(row + j0) = w;
    else *reinterpret_cast<u32x4_bytes*>(row + j0) = w;
  } else {
#pragma unroll
    for (int x = 0; x < kMapPerThread; ++x)
      if (j0 + x >= 0 && j0 + x < T) row[j0 + x] = (uint8_t)(w[x >> 2] >> (8 * (x & 3)));
  }
}

// ALIGNED: T is a multiple of 16, so every row starts on the 16-byte grid.
// HEADS: the per-query-head masks are written too.
// WALK kEach: uniform bins of one or two positions.  A run then crosses eight to
// sixteen, and a position's bin is a shift away, so it is walked position by
// position, unrolled: 8 rows of 9,001 positions and one head each, bins of one
// position, 25.8 us by regions, 20.2 by positions; with the per-head masks 33.9
// and 21.6.  (From three positions on the walk by regions is as fast or faster.)
// WALK kStep: other narrow bins (walk_step) with per-head masks, position by
// position too, one bin down at each lower edge passed.
enum Walk { kRegions, kEach, kStep };
template <bool ALIGNED, bool HEADS, Walk WALK>
__global__ __launch_bounds__(kMapThreads) void map_pattern_kernel(MapParams p) {
  constexpr bool PAIRS = WALK != kRegions;
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ int64_t red[kMapThreads / kWave + 1];
  // heads that keep each position of a run of more than two regions
  __shared__ uint16_t hbits[HEADS && !PAIRS ? kMapPerThread : 1][kMapThreads];

  const int chunks = (int)map_chunks(p.T);
  const int seg = (int)(blockIdx.x / chunks);
  const int64_t chunk0 = (int64_t)(blockIdx.x - (int64_t)seg * chunks) * kMapChunk;
  const int64_t chunk1 = chunk0 + kMapChunk < p.T ? chunk0 + kMapChunk : p.T;
  const int unit = seg / p.Hkv;
  const int g = seg - unit * p.Hkv;
  const int tid = threadIdx.x;
  const int D = p.D, T = p.T, G = p.G;

  uint16_t* qbits = reinterpret_cast<uint16_t*>(smem);
  int32_t* edges = reinterpret_cast<int32_t*>(smem + ((D * 2 + 15) & ~15));

  const uint8_t* prow = p.pattern + ((int64_t)unit * p.Hq + (int64_t)g * G) * D;
  for (int k = tid; k < D; k += kMapThreads) qbits[k] = (uint16_t)group_bits(prow, D, G, k);
  if (p.uniform_width == 0)
    for (int k = tid; k <= D; k += kMapThreads) edges[k] = p.edges[k];
  __syncthreads();

  const uint32_t all_heads = (1u << G) - 1u;
  // this unit's context length (clamped into the row)
  int32_t Tn = T;
  if (p.unit_len != nullptr) {
    Tn = p.unit_len[unit];
    Tn = Tn < 0 ? 0 : (Tn > T ? T : Tn);
  }
  uint8_t* kv_row = p.kv_mask + (int64_t)seg * T;

  if (chunk0 == 0) {
    // retained length, closed form: min(Tn, S + R) always-kept positions,
    // then every kept bin's offsets [E[k], E[k+1]) within the compressible
    // span [0, Tn - S - R)
    const int64_t span = (int64_t)Tn - p.S - p.R;
    int64_t part = 0;
    for (int k = tid; k < D && span > 0; k += kMapThreads) {
      if (qbits[k] == 0) continue;
      const int64_t lo = p.uniform_width > 0 ? (int64_t)p.uniform_width * k : edges[k];
      const int64_t hi_e = p.uniform_width > 0 ? (int64_t)p.uniform_width * (k + 1) : edges[k + 1];
      const int64_t hi = hi_e < span ? hi_e : span;
      if (hi > lo) part += hi - lo;
    }
    int64_t binned;
    block_exclusive_scan<kMapThreads>(part, red, &binned);
    const int64_t always = (int64_t)p.S + p.R < Tn ? (int64_t)p.S + p.R : Tn;
    if (tid == 0) p.kv_len[seg] = (int32_t)(always + binned);
  }

  // positions fit 31 bits (T is at most INT32_MAX - 16): the sweep runs in
  // 32-bit arithmetic, from the chunk's start (past the end j0 would overflow)
  // Runs lie on the mask's 16-byte grid: rows that start off it (T not a
  // multiple of 16) have runs that start up to 15 positions early, and only
  // the runs across a row's ends are stored byte by byte (storing whole odd
  // rows by bytes took 32 rows of 9,001 positions from 4.5 to 9.4 us).
  const int32_t early = ALIGNED ? 0 : (int32_t)(((int64_t)seg * T) & 15);
  const int32_t c0 = (int32_t)chunk0 - early, c1 = ALIGNED || chunk1 == T ? (int32_t)chunk1 : (int32_t)chunk1 - early;
  for (int32_t o = tid * kMapPerThread; o < c1 - c0; o += kMapThreads * kMapPerThread) {
    const int32_t j0 = c0 + o;
    const int32_t jl = j0 + kMapPerThread - 1;
    const bool whole = ALIGNED || (j0 >= 0 && jl < T);  // all 16 bytes are this row's
    // The run region by region: past the context, sink, recent window, a bin,
    // or uncovered.  Along the run u = delta - R falls by one per position, so
    // after a bin comes the one below it: one search per run.  Most runs lie
    // in one region; a wave takes as many steps as its most divided run.
    // (Classifying runs across a region boundary position by position took
    // their waves 7 us, most of a small call.)
    uint32_t keep = 0;          // bit e: position j0 + e is kept
    [[maybe_unused]] uint32_t rb = 0, rl = 0;    // heads of the first region and of the second
    [[maybe_unused]] int32_t b = kMapPerThread;  // end of the first region
    [[maybe_unused]] int regions = 0;
    int k = -1;  // bin of the previous region (D: the uncovered part), or none
    [[maybe_unused]] uint32_t pair[kMapPerThread / 2];  // heads that keep positions 2i (low half) and 2i + 1
    if constexpr (PAIRS) {
      [[maybe_unused]] int32_t lower = 0;  // lower edge of bin k
#pragma unroll
      for (int x = 0; x < kMapPerThread; ++x) {
        const int32_t j = j0 + x, delta = Tn - 1 - j, u = delta - p.R;
        uint32_t bits = 0;
        if (j >= 0 && j < Tn) {
          if (j < p.S || u < 0) {
            bits = all_heads;
          } else if constexpr (WALK == kStep) {
            // bins hold a position at least, so u passes one edge at most
            if (k < 0 || u < lower) {
              if (k >= 0) --k;
              else k = find_bin(u, edges, D, p.uniform_width);
              if (k < 0) k = D;
              lower = p.uniform_width > 0 ? p.uniform_width * k : edges[k];
            }
            if (k < D) bits = qbits[k];
          } else if ((u >> (p.uniform_width - 1)) < D) bits = qbits[u >> (p.uniform_width - 1)];
        }
        if (bits != 0u) keep |= 1u << x;
        if (x & 1) pair[x / 2] |= bits << 16;
        else pair[x / 2] = bits;
      }
    }
    int32_t e = PAIRS ? kMapPerThread : (j0 < 0 ? -j0 : 0);
    while (e < kMapPerThread) {
      const int32_t j = j0 + e;
      uint32_t bits = 0;
      int32_t n = kMapPerThread;  // positions left in the region
      if (j < Tn) {
        const int32_t delta = Tn - 1 - j;
        if (j < p.S) {
          bits = all_heads;
          n = (p.S < Tn ? p.S : Tn) - j;
        } else if (delta < p.R) {
          bits = all_heads;
          n = delta + 1;
        } else {
          const int32_t u = delta - p.R;
          if (k >= 0) {
            --k;
          } else {
            k = find_bin(u, edges, D, p.uniform_width);
            if (k < 0) k = D;
          }
          if (k < D) bits = qbits[k];
          // the positions that stay at or above the region's lower edge (edges
          // fit 31 bits, and W * k is one)
          const int32_t lower = p.uniform_width > 0 ? p.uniform_width * k : edges[k];
          n = u - lower + 1;
        }
      }
      const int32_t end = n < kMapPerThread - e ? e + n : kMapPerThread;
      if (bits != 0u) keep |= (1u << end) - (1u << e);
      if constexpr (HEADS) {
        if (regions == 0) {
          rb = rl = bits;
          b = end;
        } else if (regions == 1) {
          rl = bits;
        } else {
          if (regions == 2)
            for (int32_t x = 0; x < e; ++x) hbits[x][tid] = (uint16_t)(x < b ? rb : rl);
          for (int32_t x = e; x < end; ++x) hbits[x][tid] = (uint16_t)bits;
        }
        ++regions;
      }
      e = end;
    }
    store_run<true>(kv_row, j0, T, whole, mask_bytes(keep));
    if constexpr (HEADS) {
      // The heads' masks from the regions.  A wave whose runs are all uniform
      // has one word per head, one whose runs hold at most two regions a
      // 16-bit keep mask; in the others every position's heads are picked
      // apart in pairs.  (Classifying each position anew and building the
      // masks bit by bit: 4 units of 8 groups of 8 heads at 131,072 with 512
      // bins of 1 to 30 positions 72.5 us, now 18.6; at 131,071, whose rows are
      // off the grid, 23.0 now, and 59.0 when every row was stored by bytes.)
      uint8_t* q_row = p.q_mask + ((int64_t)unit * p.Hq + (int64_t)g * G) * T;
      if (!PAIRS && __builtin_amdgcn_ballot_w64(regions > 1) == 0) {
        for (int h = 0; h < G; ++h, q_row += T) {
          const uint32_t x = (rb >> h) & 1u ? 0x01010101u : 0u;
          store_run<ALIGNED>(q_row, j0, T, whole, u32x4{x, x, x, x});
        }
      } else if (!PAIRS && __builtin_amdgcn_ballot_w64(regions > 2) == 0) {
        const uint32_t head = (1u << b) - 1u;
        for (int h = 0; h < G; ++h, q_row += T) {
          const uint32_t qk = ((rb >> h) & 1u ? head : 0u) | ((rl >> h) & 1u ? 0xFFFFu & ~head : 0u);
          store_run<ALIGNED>(q_row, j0, T, whole, mask_bytes(qk));
        }
      } else {
        if constexpr (!PAIRS) {
#pragma unroll
          for (int x = 0; x < kMapPerThread; x += 2) {
            const uint32_t lo = regions > 2 ? hbits[x][tid] : (x < b ? rb : rl);
            const uint32_t hi = regions > 2 ? hbits[x + 1][tid] : (x + 1 < b ? rb : rl);
            pair[x / 2] = lo | hi << 16;
          }
        }
        for (int h = 0; h < G; ++h, q_row += T) {
          u32x4 w;
#pragma unroll
          for (int q = 0; q < 4; ++q)  // bytes 0 and 2 of two pairs
            w[q] = __builtin_amdgcn_perm((pair[2 * q + 1] >> h) & 0x00010001u, (pair[2 * q] >> h) & 0x00010001u,
                                         0x06040200u);
          store_run<ALIGNED>(q_row, j0, T, whole, w);
        }
      }
    }
  }
}

}  // namespace

// Bins so narrow that a run crosses several and their heads are picked apart
// position by position anyway; bins that cover little of the row leave most runs
// uniform.  16 groups of 8 heads, regions / positions, us: 688 positions, bins of
// 3 on average 9.5 / 7.1; 1,500 positions, of 2 15.2 / 11.1 (14.3 before the walk
// by regions); one head, 1,000 positions, of 4 9.8 / 7.1.  Equal bins of three:
// 4,000 rows of 30,000, one head each, 233 / about 200 (198 before the walk), 168
// rows, four heads each, 39.9 / 42.3 (66 before); of four and more: regions.
static bool walk_step(const MapParams& p) {
  if (p.uniform_width > 0) return p.uniform_width == 3;
  return p.edges[p.D] <= 6 * p.D && 2 * (int64_t)p.edges[p.D] >= p.T;
}

int64_t map_blocks(int32_t T, int64_t num_segments) { return map_chunks(T) * num_segments; }

hipError_t launch_map_pattern(const MapParams& p, int num_segments, hipStream_t stream) {
  size_t lds = ((size_t)p.D * 2 + 15) & ~(size_t)15;
  if (p.uniform_width == 0) lds += (size_t)(p.D + 1) * 4;
  const int64_t blocks = map_blocks(p.T, num_segments);
  if (blocks > 0) {
    auto map = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(kMapThreads), lds, stream, p);
    };
    const bool aligned = (p.T & 15) == 0;
    auto bins = [&](auto al, auto hd) {
      constexpr bool A = decltype(al)::value, H = decltype(hd)::value;
      if (p.uniform_width == 1 || p.uniform_width == 2) map(map_pattern_kernel<A, H, kEach>);
      else if (H && walk_step(p)) map(map_pattern_kernel<A, H, H ? kStep : kRegions>);
      else map(map_pattern_kernel<A, H, kRegions>);
    };
    if (p.q_mask != nullptr) aligned ? bins(std::true_type{}, std::true_type{}) : bins(std::false_type{}, std::true_type{});
    else aligned ? bins(std::true_type{}, std::false_type{}) : bins(std::false_type{}, std::false_type{});
  }
  return hipGetLastError();
}

}  // namespace dkv
