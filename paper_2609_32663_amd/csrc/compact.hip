// One-time prune and pack of the KV cache (Distance-KV, Sec. 3.4 / Fig. 2(b)),
// and the append of new tokens.
//
// The pack is an order-preserving stream compaction in four passes:
//   count   each (segment, 4096-position tile) counts its retained positions
//           (16 mask bytes per lane, nonzero-byte popcount, block scan);
//   scan    one workgroup turns tile counts into each tile's first rank within
//           its segment, the segment lengths, and the segment offsets
//           (running sum of length + append capacity, unit-major);
//   list    each tile with retained positions ranks them again (block scan),
//           orders them in LDS and writes them, coalesced, to a per-segment
//           list at their rank: list[s][r] is the position of packed row r;
//   copy    a K and a V workgroup per (segment, 8 KiB chunk of packed
//           rows; up to two such chunks of 512-byte rows): LPR lanes move one
//           row with 16-byte non-temporal loads and stores (LPR = row bytes /
//           16), the source row being the list's entry.
// Where one workgroup per segment can walk the whole mask row
// (rank_whole_segments), compact_rank_kernel takes the place of count and
// list: the mask is read once (the pack of 32 segments of 9,001 positions of 256
// bytes 28.4 us with count and list, 25.6 with rank).
// The copy works on the output side because short workgroups copy fastest on
// this part and every copy workgroup then has whole rows to move: on the
// Llama-3.1-8B-shaped 128K stack (35% kept) the pack takes 1.91-1.97 ms this
// way, against 2.09-2.15 ms for a gather per 128-position input sub-tile (most
// of them empty, the others up to 32 KiB) and 2.50-2.55 ms for one per
// 4096-position tile.  (One workgroup copying both K and
// V ran 6% slower in the block gather: four interleaved streams per
// workgroup instead of two.)
// All row arithmetic is 64-bit: a whole-stack cache has more than 2^31 elements.

#include "dkv_device.hpp"
#include "dkv_launch.hpp"

namespace dkv {

namespace {

constexpr int kThreads = 256;
static_assert(kThreads == kCopyThreads, "the dispatch limit counts the copy kernel's workgroups");
constexpr int kPerThread = 16;
static_assert(kThreads * kPerThread == kCompactTile, "tile = threads x 16 positions");

__global__ __launch_bounds__(kThreads) void compact_count_kernel(CompactParams p) {
  __shared__ int64_t red[kThreads / kWave + 1];
  const int tile = blockIdx.x;
  const int seg = blockIdx.y;
  const int64_t j0 = (int64_t)tile * kCompactTile + threadIdx.x * kPerThread;
  const u32x4 w = load_mask16(p.mask, seg, p.nseg, j0, p.T);
  const int64_t c = nonzero_bytes(w[0]) + nonzero_bytes(w[1]) + nonzero_bytes(w[2]) + nonzero_bytes(w[3]);
  int64_t total;
  block_exclusive_scan<kThreads>(c, red, &total);
  if (threadIdx.x == 0) p.tile_cnt[(int64_t)seg * p.ntiles + tile] = (int32_t)total;
}

constexpr int kScanThreads = 1024;

template <bool TILES>
__global__ __launch_bounds__(kScanThreads) void compact_scan_kernel(CompactParams p) {
  __shared__ int64_t red[kScanThreads / kWave + 1];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t s0 = 0; s0 < p.nseg; s0 += kScanThreads) {
    const int64_t s = s0 + threadIdx.x;
    int64_t len = 0;
    if (!TILES && s < p.nseg) len = p.tile_cnt[s];
    if (TILES && s < p.nseg) {
      // the segment's tile counts eight at a time, all eight loads in flight
      int32_t run = 0;
      const int64_t base = s * p.ntiles;
      for (int t0 = 0; t0 < p.ntiles; t0 += 8) {
        int32_t c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) c[e] = p.tile_cnt[base + (t0 + e < p.ntiles ? t0 + e : p.ntiles - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (t0 + e < p.ntiles) {
            p.tile_base[base + t0 + e] = run;
            run += c[e];
          }
      }
      len = run;
    }
    const int64_t need = s < p.nseg ? len + p.cap : 0;
    int64_t chunk_total;
    const int64_t excl = block_exclusive_scan<kScanThreads>(need, red, &chunk_total);
    if (s < p.nseg) {
      // A segment whose rows and append room do not fit below out_rows is
      // not packed: its length becomes the marker -1 (every call that reads
      // lengths treats it as a segment with no rows and no room) and its
      // offset is clamped to out_rows, so no offset handed out points past
      // the buffer.
      const int64_t off = carry + excl;
      const bool fits = off + need <= p.out_rows;
      p.seg_off[s] = fits ? off : (off < p.out_rows ? off : p.out_rows);
      p.seg_len[s] = fits ? (int32_t)len : -1;
    }
    __syncthreads();
    if (threadIdx.x == 0) carry += chunk_total;
    __syncthreads();
  }
  if (threadIdx.x == 0 && p.rows_needed != nullptr) *p.rows_needed = carry;
}

__global__ __launch_bounds__(kThreads) void compact_list_kernel(CompactParams p) {
  __shared__ int64_t red[kThreads / kWave + 1];
  __shared__ int32_t pos[kCompactTile];
  const int tile = blockIdx.x;
  const int seg = blockIdx.y;
  const int64_t ti = (int64_t)seg * p.ntiles + tile;
  // not packed (it does not fit below out_rows), or nothing kept in this tile
  if (p.seg_len[seg] < 0 || p.tile_cnt[ti] == 0) return;
  const int64_t j0 = (int64_t)tile * kCompactTile + threadIdx.x * kPerThread;
  const u32x4 w = load_mask16(p.mask, seg, p.nseg, j0, p.T);
  const int64_t c = nonzero_bytes(w[0]) + nonzero_bytes(w[1]) + nonzero_bytes(w[2]) + nonzero_bytes(w[3]);
  int64_t total;
  int r = (int)block_exclusive_scan<kThreads>(c, red, &total);
  const uint32_t bits = nonzero_byte_bits(w);
#pragma unroll
  for (int e = 0; e < kPerThread; ++e)
    if (bits & (1u << e)) pos[r++] = (int32_t)(j0 + e);
  __syncthreads();
  int32_t* dst = p.list + (int64_t)seg * p.T + p.tile_base[ti];
  for (int i = threadIdx.x; i < total; i += kThreads) dst[i] = pos[i];
}

// One workgroup per segment lists the segment's retained positions (a
// position's rank counts from its own segment's start, so no other segment
// is needed) and leaves the segment's count in tile_cnt[seg]: the mask is
// read once and the count pass falls away.  A wave whose positions are all kept
// writes its 1,024 directly; the others order theirs in LDS first, so that
// stores are coalesced.
constexpr int kRankThreads = 1024;
constexpr int kRankPositions = kRankThreads * kPerThread;

__global__ __launch_bounds__(kRankThreads) void compact_rank_kernel(CompactParams p) {
  constexpr int kWaves = kRankThreads / kWave;
  __shared__ int32_t sums[kWaves];
  __shared__ int32_t pos[kWaves][kWave * kPerThread];
  const int seg = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int32_t* list = p.list + (int64_t)seg * p.T;
  int first = 0;  // positions kept in the steps before
  u32x4 w = load_mask16(p.mask, seg, p.nseg, (int64_t)threadIdx.x * kPerThread, p.T);
  for (int64_t base = 0; base < p.T; base += kRankPositions) {
    const uint32_t keep = nonzero_byte_bits(w);
    // the next step's mask is on its way meanwhile
    w = load_mask16(p.mask, seg, p.nseg, base + kRankPositions + (int64_t)threadIdx.x * kPerThread, p.T);
    const int inc = (int)wave_inclusive_sum((uint32_t)__popc(keep));
    const int n = __builtin_amdgcn_readlane(inc, kWave - 1);  // kept positions of the wave
    if (lane == 0) sums[wave] = n;
    __syncthreads();
    const int upto = (int)wave_inclusive_sum(lane < kWaves ? (uint32_t)sums[lane] : 0u);
    int32_t* dst = list + first + __builtin_amdgcn_readlane(upto, wave) - n;
    first += __builtin_amdgcn_readlane(upto, kWaves - 1);
    const int32_t j0 = (int32_t)base + wave * (kWave * kPerThread);
    if (n == kWave * kPerThread) {
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) dst[e * kWave + lane] = j0 + e * kWave + lane;
    } else if (n > 0) {
      int at = inc - __popc(keep);
#pragma unroll
      for (int e = 0; e < kPerThread; ++e)
        if (keep & (1u << e)) pos[wave][at++] = j0 + lane * kPerThread + e;
      wave_lds_fence();
      for (int i = lane; i < n; i += kWave) dst[i] = pos[wave][i];
      wave_lds_fence();
    }
    __syncthreads();  // sums is free again
  }
  if (threadIdx.x == 0) p.tile_cnt[seg] = first;
}

// ROWS: packed rows of a chunk; GRID: positions of a segment per K and V
// workgroup of the grid.  With GRID = 2 ROWS the grid has workgroups for the
// chunks up to rank T / 2, and each moves the chunk T / 2 further on too where the
// segment reaches so far: most are as short as with a workgroup per chunk, but
// segments that keep little leave half as many without work.  The whole pack of
// 512-byte rows, us, 32-row chunks / 16-row chunks / 16-row chunks this way: 256
// segments of 9,000 positions, 1% kept 40 / 70 / 40, 35% 286 / 268 / 273, 60% 474
// / 445 / 466; 4,096 of 2,000, 1% 131 / 237 / 131, 35% 1,009 / 944 / 963.
template <int LPR, int ROWS, int GRID>
__global__ __launch_bounds__(kThreads) void compact_copy_kernel(CompactParams p) {
  constexpr int kRowsPerPass = kThreads / LPR;
  constexpr int kPasses = (ROWS + kRowsPerPass - 1) / kRowsPerPass;  // rows per lane group
  static_assert(kPasses <= 8, "rows in flight per lane group");
  const int chunk = blockIdx.x >> 1;
  const int which = blockIdx.x & 1;  // 0: K rows (and source positions), 1: V rows
  const int seg = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid % LPR;
  // Most workgroups of the grid lie past their segment's rows: they leave
  // after one scalar load.
  const int32_t len = p.seg_len[seg];
  if (len <= 0) return;  // not packed
  static_assert(GRID == ROWS || GRID == 2 * ROWS, "chunks of a workgroup");
  const int chunks = GRID == ROWS ? 0 : (int)(copy_workgroups(p.T, GRID) / 2);  // of the first half
  if (GRID != ROWS && chunk >= chunks) return;
  for (int64_t r_lo = (int64_t)chunk * ROWS; r_lo < len; r_lo += (int64_t)chunks * ROWS) {
    const int64_t r_hi = r_lo + ROWS < len ? r_lo + ROWS : len;
    const int32_t* list = p.list + (int64_t)seg * p.T;
    int32_t pos[kPasses];
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int64_t r = r_lo + tid / LPR + (int64_t)u * kRowsPerPass;
      pos[u] = list[r < r_hi ? r : r_lo];
    }
    // Every list entry is waited for at once, then every row load is issued
    // before any is waited for (rows past the chunk's end load its first
    // row): waiting per row would also wait for the row loads before it.
#pragma unroll
    for (int u = 0; u < kPasses; ++u) asm volatile("" ::"v"(pos[u]));
    const int64_t dst0 = p.seg_off[seg];
    const int64_t src0 = (int64_t)seg * p.T;
    const u32x4* src = reinterpret_cast<const u32x4*>(which ? p.v : p.k);
    u32x4* dst = reinterpret_cast<u32x4*>(which ? p.v_out : p.k_out);
    u32x4 rb[kPasses];
#pragma unroll
    for (int u = 0; u < kPasses; ++u) rb[u] = __builtin_nontemporal_load(&src[(src0 + pos[u]) * LPR + lane]);
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int64_t r = r_lo + tid / LPR + (int64_t)u * kRowsPerPass;
      if (r < r_hi) {
        __builtin_nontemporal_store(rb[u], &dst[(dst0 + r) * LPR + lane]);
        if (which == 0 && lane == 0 && p.src_pos != nullptr) p.src_pos[dst0 + r] = pos[u];
      }
    }
    if (GRID == ROWS) return;
  }
}

__global__ __launch_bounds__(kThreads) void append_kernel(AppendParams p) {
  const int lpr = p.row_bytes / 16;
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t row_id = gid / lpr;
  const int lane = (int)(gid - row_id * lpr);
  if (row_id >= (int64_t)p.nseg * p.n_new) return;
  const int64_t s = row_id / p.n_new;
  const int64_t t = row_id - s * p.n_new;
  if (p.seg_len[s] < 0) return;  // a segment dkv_compact could not pack has no room
  const int64_t drow = p.seg_off[s] + p.seg_len[s] + p.n_tail + t;
  const u32x4* ks = reinterpret_cast<const u32x4*>(p.k_new);
  const u32x4* vs = reinterpret_cast<const u32x4*>(p.v_new);
  reinterpret_cast<u32x4*>(p.k_c)[drow * lpr + lane] = ks[row_id * lpr + lane];
  reinterpret_cast<u32x4*>(p.v_c)[drow * lpr + lane] = vs[row_id * lpr + lane];
}

}  // namespace

// Whether one workgroup per segment ranks its whole mask row, 16,384 positions
// at a step, or the workgroups take 4096-position tiles in two passes.  A round
// of whole rows takes as long for a few positions as for a step, so tiles are
// ahead for thousands of short segments, and for long rows that too few
// workgroups walk step by step.  The whole pack, whole / tiles, us (256-byte
// rows, 35% kept in runs of 64): 1 segment of 256 positions 8.9 / 11.2, of
// 32,768 13.3 / 13.5, of 65,536 19.7 / 16.0; 32 of 32,768 71.0 / 71.5, of
// 131,072 268 / 258; 128 of 131,072, 128-byte rows, 522 / 522; 256 of 16,384
// 254 / 255; 1,024 of 1,024 70.1 / 71.5; 4,096 of 100 49.0 / 48.1, of 1,024
// 270.6 / 268.1, of 4,096, 128-byte rows, 518 / 524; 16,384 of 256 329 / 311.
static bool rank_whole_segments(int32_t T, int64_t nseg) {
  return T <= 8 * kRankPositions && (nseg >= 128 || T <= 2 * kRankPositions) && (nseg <= 1024 || T >= kCompactTile);
}

size_t compact_workspace_bytes(int64_t nseg, int64_t T) {
  const int64_t ntiles = (T + kCompactTile - 1) / kCompactTile;
  const int64_t n = nseg * (ntiles > 0 ? ntiles : 1);
  return (size_t)(2 * n * 4 + nseg * T * 4 + 256);  // tile counts, tile bases, position lists
}

hipError_t launch_compact(const CompactParams& p, hipStream_t stream) {
  const dim3 grid(p.ntiles > 0 ? p.ntiles : 1, p.nseg);
  const bool whole = p.ntiles > 0 && rank_whole_segments(p.T, p.nseg);
  if (whole) {
    hipLaunchKernelGGL(compact_rank_kernel, dim3(p.nseg), dim3(kRankThreads), 0, stream, p);
    hipLaunchKernelGGL(compact_scan_kernel<false>, dim3(1), dim3(kScanThreads), 0, stream, p);
  } else {
    if (p.ntiles > 0) hipLaunchKernelGGL(compact_count_kernel, grid, dim3(kThreads), 0, stream, p);
    hipLaunchKernelGGL(compact_scan_kernel<true>, dim3(1), dim3(kScanThreads), 0, stream, p);
  }
  if (p.ntiles > 0) {
    if (!whole) hipLaunchKernelGGL(compact_list_kernel, grid, dim3(kThreads), 0, stream, p);
    auto copy = [&](auto kernel) {  // K and V workgroups in turn
      const int64_t n = copy_grid(p.T, copy_rows(p.row_bytes), p.nseg);
      hipLaunchKernelGGL(kernel, dim3((uint32_t)n, p.nseg), dim3(kThreads), 0, stream, p);
    };
    switch (p.row_bytes) {
      case 128: copy(compact_copy_kernel<8, 64, 64>); break;
      case 256: copy(compact_copy_kernel<16, 32, 32>); break;
      case 512:
        // a few long segments that keep little have too few chunks among their
        // idle workgroups for the short ones to pay: 4 segments of 400,000
        // positions, 5% kept 45 us with 32-row chunks, 55 with 16, 16 of 200,000
        // 69 and 74 (64 of 131,072 158 and 162, 10% 309 and 299)
        if (p.nseg < 32 && p.T > 131072) copy(compact_copy_kernel<32, 32, 32>);
        else copy(compact_copy_kernel<32, 16, 32>);
        break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

hipError_t launch_append(const AppendParams& p, hipStream_t stream) {
  const int64_t threads = (int64_t)p.nseg * p.n_new * (p.row_bytes / 16);
  const int64_t blocks = (threads + kThreads - 1) / kThreads;
  if (blocks > 0) hipLaunchKernelGGL(append_kernel, dim3((uint32_t)blocks), dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace dkv
