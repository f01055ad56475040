// Exact-budget pattern export (Sec. 3.3, Eq. (topk-pattern); Appendix A,
// exact-budget refinement): the K largest of the L x H x D retention
// probabilities become the pattern's ones, all other entries zeros.
//
// A radix select over the whole grid.  Every entry gets a 32-bit key that
// orders like its value (NaN lowest, -0 equal to +0).  Three rounds of
// digits (11, 11 and 10 bits, most significant first) find the K-th largest
// key v and how many entries equal to v must be kept.  In a round every
// workgroup counts the keys of its contiguous chunk that match the prefix
// found so far (one LDS histogram per wave) and adds its counts to the
// round's global histogram.  The digit of a round -- the one whose bucket
// holds the K-th largest key -- is picked at the start of the next launch by
// every workgroup from that histogram (the kernel boundary publishes it; no
// device-scope fence, which costs an L2 write-back per workgroup, and no
// counters); workgroup 0 also stores the grown prefix for the launch after.
// Ties go to the lowest flat indices: in the last round every workgroup also
// stores its own histogram, so the write pass ranks its chunk's ties after
// the earlier chunks' (their count of the final digit), in index order.
// Five launches (clear, three rounds, write); no launch depends on the host.
// State lives in a caller-provided workspace.

#include <type_traits>

#include "dkv_device.hpp"
#include "dkv_launch.hpp"

namespace dkv {

namespace {

constexpr int kTkThreads = 256;
constexpr int kTkWaves = kTkThreads / kWave;
constexpr int kTkStep = kTkThreads * 4;     // entries per workgroup iteration (one quadruple per thread)
constexpr int kTkGroup = 4;                 // iterations whose loads are in flight together
constexpr int kTkMinChunk = kTkGroup * kTkStep;  // entries per workgroup at least
constexpr int kTkMaxBlocks = 1024;
constexpr int kTkRounds = 3;
constexpr int kTkShift[kTkRounds] = {21, 10, 0};
constexpr int kTkBits[kTkRounds] = {11, 11, 10};
constexpr int kTkMaxBins = 2048;
constexpr int kTkLastBins = 1 << 10;
// workspace (uint32): the prefix and the entries still to take within it
// after the digits of rounds 0 and 1 (two slots: a launch reads one and
// stores the next), kTkCopies histograms per round, then the last round's
// histogram of every workgroup.  Workgroup b adds to copy b % copies and the
// digit's pick sums the copies: with few distinct digits (quantised
// probabilities) all workgroups add to the same words, and one copy made a
// round of 254 workgroups 7.5-9.0 us where four make it 5.6-7.1.
constexpr int kTkCopies = 4;
constexpr int kTkSel = 0;  // round r's result: kTkSel + 2r (prefix), + 1 (need)
constexpr int kTkHist = 4;
constexpr int kTkWgHist = kTkHist + kTkRounds * kTkCopies * kTkMaxBins;

__device__ __forceinline__ uint32_t order_key(float x) {
  if (x != x) return 0u;  // NaN below every number
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0u;  // -0 ties with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

typedef u32x4 __attribute__((aligned(4))) u32x4_words;  // the workspace is 4-byte aligned

// A thread's share of one group of kTkGroup iterations from entry i0 on:
// quadruple s is the entries [i0 + 4 tid + s * kTkStep, + 4), those below `end`;
// the rest have valid = 0.
// probs is 16-byte aligned and i0 a multiple of 4, so a whole quadruple is one
// load; all of a group's loads are in flight together.
struct KeyGroup {
  float4 x[kTkGroup];
  uint32_t valid[kTkGroup];

  __device__ __forceinline__ void load(const float* probs, int64_t i0, int64_t end) {
    const int64_t i = i0 + threadIdx.x * 4;
#pragma unroll
    for (int s = 0; s < kTkGroup; ++s) {
      const int64_t at = i + (int64_t)s * kTkStep;
      x[s] = float4{0.f, 0.f, 0.f, 0.f};
      valid[s] = 0u;
      if (at + 3 < end) {
        x[s] = *reinterpret_cast<const float4*>(probs + at);
        valid[s] = 0xFu;
      } else if (at < end) {
        float* e = &x[s].x;
        e[0] = probs[at];
        valid[s] = 1u;
        if (at + 1 < end) {
          e[1] = probs[at + 1];
          valid[s] = 3u;
        }
        if (at + 2 < end) {
          e[2] = probs[at + 2];
          valid[s] = 7u;
        }
      }
    }
  }

  __device__ __forceinline__ void keys(int s, uint32_t (&key)[4]) const {
    key[0] = order_key(x[s].x);
    key[1] = order_key(x[s].y);
    key[2] = order_key(x[s].z);
    key[3] = order_key(x[s].w);
  }
};

__device__ __forceinline__ void chunk_of(const TopkParams& p, int b, int64_t& c0, int64_t& c1) {
  c0 = (int64_t)b * p.chunk;
  c1 = c0 + p.chunk < p.n ? c0 + p.chunk : p.n;
}

// Runs `body` for a group of iterations: told at compile time that the group is
// whole, or left to skip the iterations past the chunk (small exports are one
// part of a group: 64 entries 20.7 us with all four iterations run, 18.3 with
// one; large ones are whole groups, which the skips slow by 3%).
template <class Body>
__device__ __forceinline__ void whole_or_part(int64_t left, Body body) {
  if (left >= kTkGroup * kTkStep) body(std::true_type{});
  else body(std::false_type{});
}

__global__ __launch_bounds__(kTkThreads) void topk_init_kernel(TopkParams p) {
  const int words = kTkHist + kTkRounds * p.copies * kTkMaxBins;
  for (int i = blockIdx.x * kTkThreads + threadIdx.x; i < words; i += gridDim.x * kTkThreads) p.state[i] = 0u;
}

// The digit of round R: with the keys of round R's global histogram that
// match `prefix` counted per digit, the largest digit whose bucket holds the
// need-th largest of them.  Thread t takes the bins NB - 1 - per t down to
// NB - per (t + 1); its exclusive scan is the count above its first bin and
// the one thread whose bins cross `need` finds the digit.  Every thread gets
// the grown prefix and what is still to take within it.
template <int R>
__device__ __forceinline__ void select_digit(const TopkParams& p, uint32_t& prefix, uint32_t& need, int64_t* red,
                                             uint32_t* out) {
  constexpr int NB = 1 << kTkBits[R];
  constexpr int per = NB / kTkThreads;
  static_assert(NB % kTkThreads == 0 && per % 4 == 0, "bins spread evenly over the threads, in whole loads");
  // the copies' sums: a thread's bins are consecutive, so it loads each copy's
  // by 16 bytes, all loads in flight together (handing the bins over through
  // LDS took a round's 32 KiB of histograms past a quarter of the CU's LDS: with
  // 1,024 workgroups, four a CU, round 1 of 82M entries ran 148 us where it is
  // 80 otherwise)
  const uint32_t* g = p.state + kTkHist + R * p.copies * kTkMaxBins + NB - per * (threadIdx.x + 1);
  uint32_t x[per];
  if (p.copies > 1) {
    u32x4 y[kTkCopies][per / 4];
#pragma unroll
    for (int c = 0; c < kTkCopies; ++c)
#pragma unroll
      for (int v = 0; v < per / 4; ++v) y[c][v] = *reinterpret_cast<const u32x4_words*>(g + c * kTkMaxBins + 4 * v);
#pragma unroll
    for (int v = 0; v < per / 4; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[4 * v + e] = 0;
#pragma unroll
        for (int c = 0; c < kTkCopies; ++c) x[4 * v + e] += y[c][v][e];
      }
  } else {
#pragma unroll
    for (int v = 0; v < per / 4; ++v) {
      const u32x4 y = *reinterpret_cast<const u32x4_words*>(g + 4 * v);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * v + e] = y[e];
    }
  }
  uint32_t h[per];
  int64_t mine = 0;
#pragma unroll
  for (int j = 0; j < per; ++j) {
    h[j] = x[per - 1 - j];
    mine += h[j];
  }
  int64_t all;
  int64_t above = block_exclusive_scan<kTkThreads>(mine, red, &all);
#pragma unroll
  for (int j = 0; j < per; ++j) {
    if (above < (int64_t)need && above + h[j] >= (int64_t)need) {
      out[0] = prefix | ((uint32_t)(NB - 1 - (per * threadIdx.x + j)) << kTkShift[R]);
      out[1] = need - (uint32_t)above;
    }
    above += h[j];
  }
  __syncthreads();
  prefix = out[0];
  need = out[1];
}

// Round R: the previous round's digit (R > 0), then this round's counts.
template <int R>
__global__ __launch_bounds__(kTkThreads) void topk_round_kernel(TopkParams p) {
  constexpr int shift = kTkShift[R];
  constexpr int NB = 1 << kTkBits[R];
  __shared__ uint32_t hist[kTkWaves][NB];
  __shared__ int64_t red[kTkWaves + 1];
  __shared__ uint32_t sel[2];
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  // the chunk's first group is on its way while the digit is picked (for up
  // to 4M entries it is the whole chunk): waiting for each iteration's load in
  // turn, after the digit, made the write pass 7.7 us where it is 5.6 now
  int64_t c0, c1;
  chunk_of(p, blockIdx.x, c0, c1);
  KeyGroup grp;
  grp.load(p.probs, c0, c1);
  for (int i = tid; i < kTkWaves * NB; i += kTkThreads) (&hist[0][0])[i] = 0u;
  uint32_t prefix = 0u, need = (uint32_t)p.k;
  if constexpr (R > 0) {
    if constexpr (R > 1) {
      prefix = p.state[kTkSel + 2 * (R - 2)];
      need = p.state[kTkSel + 2 * (R - 2) + 1];
    }
    select_digit<R - 1>(p, prefix, need, red, sel);
    if (blockIdx.x == 0 && tid == 0) {
      p.state[kTkSel + 2 * (R - 1)] = prefix;
      p.state[kTkSel + 2 * (R - 1) + 1] = need;
    }
  }
  __syncthreads();
  const uint32_t mask = R == 0 ? 0u : 0xFFFFFFFFu << ((shift + kTkBits[R]) & 31);
  for (int64_t i0 = c0; i0 < c1; i0 += kTkGroup * kTkStep) {
    if (i0 > c0) grp.load(p.probs, i0, c1);
    whole_or_part(c1 - i0, [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < kTkGroup; ++s) {
        if (!whole && i0 + s * kTkStep >= c1) continue;
        uint32_t key[4];
        grp.keys(s, key);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((whole || ((grp.valid[s] >> e) & 1u)) && (key[e] & mask) == prefix)
            atomicAdd(&hist[wave][(key[e] >> shift) & (NB - 1)], 1u);
      }
    });
  }
  __syncthreads();
  uint32_t* g = p.state + kTkHist + (R * p.copies + blockIdx.x % p.copies) * kTkMaxBins;
  for (int i = tid; i < NB; i += kTkThreads) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kTkWaves; ++w) c += hist[w][i];
    if (R == kTkRounds - 1) p.state[kTkWgHist + (int64_t)blockIdx.x * kTkLastBins + i] = c;
    if (c) atomicAdd(&g[i], c);
  }
}

__global__ __launch_bounds__(kTkThreads) void topk_write_kernel(TopkParams p) {
  __shared__ int64_t red[kTkWaves + 1];
  __shared__ uint32_t sel[2];
  const int tid = threadIdx.x;
  int64_t c0, c1;
  chunk_of(p, blockIdx.x, c0, c1);
  KeyGroup grp;
  grp.load(p.probs, c0, c1);
  // the last digit: thr is the K-th largest key, take the entries equal to
  // it that are kept
  uint32_t thr = 0u, take = 0u;
  if (p.k > 0) {
    thr = p.state[kTkSel + 2 * (kTkRounds - 2)];
    take = p.state[kTkSel + 2 * (kTkRounds - 2) + 1];
    select_digit<kTkRounds - 1>(p, thr, take, red, sel);
  }
  // entries equal to thr in the chunks before this one
  uint32_t before = 0;
  if (p.k > 0)
    for (int j = tid; j < (int)blockIdx.x; j += kTkThreads)
      before += p.state[kTkWgHist + (int64_t)j * kTkLastBins + (thr & (kTkLastBins - 1))];
  int64_t rank;  // the block's total
  block_exclusive_scan<kTkThreads>(before, red, &rank);
  for (int64_t i0 = c0; i0 < c1; i0 += kTkGroup * kTkStep) {
    if (i0 > c0) grp.load(p.probs, i0, c1);
    // ties per iteration, four 16-bit sums in one scan (an iteration holds at
    // most kTkStep of them)
    static_assert(kTkGroup == 4 && kTkStep < 65536, "four sums per scan");
    whole_or_part(c1 - i0, [&](auto whole) __attribute__((always_inline)) {
      uint32_t eq[kTkGroup];
      uint64_t cnt = 0;
#pragma unroll
      for (int s = 0; s < kTkGroup; ++s) {
        eq[s] = 0u;
        if (!whole && i0 + s * kTkStep >= c1) continue;
        uint32_t key[4];
        grp.keys(s, key);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          eq[s] |= ((whole || ((grp.valid[s] >> e) & 1u)) && p.k > 0 && key[e] == thr ? 1u : 0u) << e;
        cnt |= (uint64_t)__popc(eq[s]) << (16 * s);
      }
      int64_t totals;
      const uint64_t ex = (uint64_t)block_exclusive_scan<kTkThreads>((int64_t)cnt, red, &totals);
#pragma unroll
      for (int s = 0; s < kTkGroup; ++s) {
        if (!whole && i0 + s * kTkStep >= c1) continue;
        const int64_t i = i0 + (int64_t)s * kTkStep + tid * 4;
        int64_t r = rank + (int64_t)((ex >> (16 * s)) & 0xFFFFu);
        uint32_t key[4];
        grp.keys(s, key);
        uchar4 out;
        uint8_t* ob = reinterpret_cast<uint8_t*>(&out);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool t = (eq[s] >> e) & 1u;
          ob[e] = (p.k > 0 && (whole || ((grp.valid[s] >> e) & 1u)) &&
                   (key[e] > thr || (t && r < (int64_t)take)))
                      ? 1
                      : 0;
          r += t ? 1 : 0;
        }
        if (whole || grp.valid[s] == 0xFu) {
          *reinterpret_cast<uchar4*>(p.pattern + i) = out;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if ((grp.valid[s] >> e) & 1u) p.pattern[i + e] = ob[e];
        }
        rank += (int64_t)(((uint64_t)totals >> (16 * s)) & 0xFFFFu);
      }
    });
  }
}

}  // namespace

int topk_blocks(int64_t n) {
  const int64_t b = (n + kTkMinChunk - 1) / kTkMinChunk;
  return (int)(b < 1 ? 1 : (b > kTkMaxBlocks ? kTkMaxBlocks : b));
}

size_t topk_workspace_bytes(int64_t n) {
  return ((size_t)kTkWgHist + (size_t)topk_blocks(n) * kTkLastBins) * sizeof(uint32_t);
}

hipError_t launch_topk_pattern(TopkParams p, hipStream_t stream) {
  if (p.n == 0) return hipSuccess;
  const int blocks = topk_blocks(p.n);
  // chunks are whole iterations of the workgroup's quadruples
  p.chunk = ((p.n + blocks - 1) / blocks + kTkStep - 1) / kTkStep * kTkStep;
  p.copies = blocks >= 64 ? kTkCopies : 1;
  if (p.k > 0) {
    hipLaunchKernelGGL(topk_init_kernel, dim3(6 * p.copies), dim3(kTkThreads), 0, stream, p);
    hipLaunchKernelGGL(topk_round_kernel<0>, dim3(blocks), dim3(kTkThreads), 0, stream, p);
    hipLaunchKernelGGL(topk_round_kernel<1>, dim3(blocks), dim3(kTkThreads), 0, stream, p);
    hipLaunchKernelGGL(topk_round_kernel<2>, dim3(blocks), dim3(kTkThreads), 0, stream, p);
  }
  hipLaunchKernelGGL(topk_write_kernel, dim3(blocks), dim3(kTkThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace dkv
