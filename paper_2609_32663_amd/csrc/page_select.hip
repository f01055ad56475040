// Zero-copy alternative to the pack: list each segment's retained rows where
// they already are, in a cache kept in pages of page_rows consecutive
// positions.
//
// The retained set of a segment is the sink, the recent window and a union of
// whole distance bins (Eq. (4), Eq. (5), union of Sec. 3.4), so its positions
// form a few long runs.  Each run is cut at page boundaries and listed as an
// entry (physical page, logical page, lo, hi) naming slots [lo, hi) of one
// page; decode reads those slots in place.  With the paper's 128-token bins
// and 128-row pages every context entry is a whole page.
//
// A run starts at a kept position whose predecessor is not kept or that opens
// a page.  Short contexts, and longer ones with enough segments
// (select_whole_segments), take one workgroup per segment and one pass over the
// mask (page_select_kernel): 256 segments of 131,072 positions, map included,
// took 49.4 us in the two passes below and take 25.0 (13.4 for the selection
// alone, against 39).  With fewer or longer segments one workgroup each would
// leave the chip idle; those take two passes over the (segment, 4096-position
// tile) grid:
//   count  each thread turns 16 mask bytes into a 16-bit keep mask; the tile
//          sums its run starts and kept positions;
//   emit   each workgroup adds up the run counts of its segment's earlier
//          tiles (its first entry), and each thread writes the entries whose
//          runs start in its 16 positions (page, logical page, lo) and the
//          end slot of the runs that end there; a run's entry index is its
//          start's rank.  The segment's last tile also writes the retained
//          length, the append region's entries (appended tokens are always
//          kept) and the entry count.
// Contexts of more than kSumTiles tiles (4M positions) have a scan pass
// between them: there every emit workgroup summing all earlier tiles would
// cost work quadratic in the context length.
// A context of length 0 has no tile: one small kernel writes those segments.
// Page sizes are multiples of 16 that divide the tile, so a page boundary is
// always the boundary of a thread's 16 positions, and every wave's first
// lane starts a page: neighbouring bits come from the adjacent lane.

#include "dkv_device.hpp"
#include "dkv_launch.hpp"

namespace dkv {

namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 16;
constexpr int kSumTiles = 1024;  // longest context (in tiles) whose emit pass sums tile counts itself
static_assert(kThreads * kPerThread == kCompactTile, "tile = threads x 16 positions");

// Keep mask of this thread's 16 positions, and the run starts and ends among
// them.  A run starts where the previous position is not kept or a page
// begins, and ends where the next position is not kept or a page ends.
struct RunBits {
  uint32_t keep, starts, ends;
};

__device__ __forceinline__ RunBits run_bits(const PageSelectParams& p, int seg, int tile) {
  const int tid = threadIdx.x;
  const int64_t j0 = (int64_t)tile * kCompactTile + tid * kPerThread;
  const uint32_t keep = nonzero_byte_bits(load_mask16(p.mask, seg, p.nseg, j0, p.T));
  const uint32_t left = __shfl_up(keep, 1, kWave);
  const uint32_t right = __shfl_down(keep, 1, kWave);
  const bool page_first = (j0 % p.page_rows) == 0;
  const bool page_last = ((j0 + kPerThread) % p.page_rows) == 0;
  const uint32_t prev = page_first ? 0u : (left >> 15) & 1u;
  const uint32_t next = page_last ? 0u : right & 1u;
  RunBits r;
  r.keep = keep;
  r.starts = keep & ~((keep << 1) | prev);
  r.ends = keep & ~((keep >> 1) | (next << 15));
  return r;
}

__global__ __launch_bounds__(kThreads) void page_count_kernel(PageSelectParams p) {
  __shared__ int64_t red[kThreads / kWave + 1];
  const int tile = blockIdx.x;
  const int seg = blockIdx.y;
  const RunBits r = run_bits(p, seg, tile);
  int64_t starts, kept;
  block_exclusive_scan<kThreads>(__popc(r.starts), red, &starts);
  block_exclusive_scan<kThreads>(__popc(r.keep), red, &kept);
  if (threadIdx.x == 0) {
    p.tile_cnt[(int64_t)seg * p.ntiles + tile] = (int32_t)starts;
    p.tile_kept[(int64_t)seg * p.ntiles + tile] = (int32_t)kept;
  }
  // clear the usage flags of this tile's pages; the emit pass sets the used ones
  if (p.page_used != nullptr) {
    const int per_tile = kCompactTile / p.page_rows;
    const int64_t pg0 = (int64_t)tile * per_tile;
    for (int i = threadIdx.x; i < per_tile; i += kThreads)
      if (pg0 + i < p.pages_per_seg) p.page_used[(int64_t)seg * p.pages_per_seg + pg0 + i] = 0;
  }
}

// The append region [T, T + cap) of segment s: one entry per page it touches,
// after the segment's n context entries; returns the segment's entry count.
// Also marks those pages used and clears the flags of pages past the context
// tiles that the region does not use.  One thread.
__device__ int32_t finish_segment(const PageSelectParams& p, int s, int32_t n) {
  const int pr = p.page_rows;
  if (p.cap > 0) {
    const int64_t first = (int64_t)p.T / pr, last = ((int64_t)p.T + p.cap - 1) / pr;
    for (int64_t lp = first; lp <= last; ++lp, ++n) {
      const int32_t page = p.table[(int64_t)s * p.pages_per_seg + lp];
      if (n < p.max_entries) {
        int32_t* e = p.entries + ((int64_t)s * p.max_entries + n) * 4;
        const int64_t lo = (p.T > lp * pr ? p.T : lp * pr) - lp * pr;
        const int64_t end = (int64_t)p.T + p.cap < (lp + 1) * pr ? (int64_t)p.T + p.cap : (lp + 1) * pr;
        e[0] = page;
        e[1] = (int32_t)lp;
        e[2] = (int32_t)lo;
        e[3] = (int32_t)(end - lp * pr);
      }
      if (p.page_used != nullptr) p.page_used[(int64_t)s * p.pages_per_seg + lp] = 1;
    }
  }
  if (p.page_used != nullptr) {
    const int64_t covered = (int64_t)p.ntiles * (kCompactTile / pr);
    const int64_t tail0 = p.cap > 0 ? (int64_t)p.T / pr : p.pages_per_seg;
    const int64_t tail1 = p.cap > 0 ? ((int64_t)p.T + p.cap - 1) / pr : -1;
    for (int64_t lp = covered; lp < p.pages_per_seg; ++lp)
      if (lp < tail0 || lp > tail1) p.page_used[(int64_t)s * p.pages_per_seg + lp] = 0;
  }
  return n;
}

// Long contexts: one thread per segment turns tile counts into each tile's
// first entry, then finishes the segment.
__global__ __launch_bounds__(kThreads) void page_scan_kernel(PageSelectParams p) {
  const int s = blockIdx.x * kThreads + threadIdx.x;
  if (s >= p.nseg) return;
  const int64_t base = (int64_t)s * p.ntiles;
  int32_t run = 0, kept = 0;
  for (int t = 0; t < p.ntiles; ++t) {
    p.tile_base[base + t] = run;
    run += p.tile_cnt[base + t];
    kept += p.tile_kept[base + t];
  }
  p.seg_len[s] = kept;
  p.n_entries[s] = finish_segment(p, s, run);
}

__global__ __launch_bounds__(kThreads) void page_emit_kernel(PageSelectParams p) {
  __shared__ int64_t red[kThreads / kWave + 1];
  const int tile = blockIdx.x;
  const int seg = blockIdx.y;
  // With tile_base (long contexts) the scan pass gave this tile its first
  // entry and finished the segment; otherwise the workgroup adds up the runs
  // that start in the segment's earlier tiles (high 32 bits; low 32 bits:
  // all its tiles' runs, which the last tile needs) and the last tile sums
  // the retained positions.
  const bool summed = p.tile_base == nullptr;
  const bool last_tile = summed && tile == p.ntiles - 1;
  int64_t before = 0, runs = 0, kept_part = 0;
  if (summed) {
    int64_t packed = 0;
    for (int t = threadIdx.x; t < p.ntiles; t += kThreads) {
      const int64_t c = p.tile_cnt[(int64_t)seg * p.ntiles + t];
      packed += (t < tile ? (c << 32) : 0) + c;
      if (last_tile) kept_part += p.tile_kept[(int64_t)seg * p.ntiles + t];
    }
    int64_t sums;
    block_exclusive_scan<kThreads>(packed, red, &sums);
    before = sums >> 32;
    runs = sums & 0xFFFFFFFFLL;
  } else {
    before = p.tile_base[(int64_t)seg * p.ntiles + tile];
  }
  const RunBits r = run_bits(p, seg, tile);
  int64_t total;
  const int64_t rank = block_exclusive_scan<kThreads>(__popc(r.starts), red, &total);
  const int64_t e0 = before + rank;  // entry of this thread's first start
  const int64_t j0 = (int64_t)tile * kCompactTile + threadIdx.x * kPerThread;
  const int pr = p.page_rows;
  int32_t* ent = p.entries + (int64_t)seg * p.max_entries * 4;
  uint32_t st = r.starts, en = r.ends;
  int64_t e = e0;
  while (st != 0u) {
    const int b = __builtin_ctz(st);
    st &= st - 1u;
    const int64_t j = j0 + b;
    const int64_t lp = j / pr;
    if (e < p.max_entries) {
      ent[e * 4 + 0] = p.table[(int64_t)seg * p.pages_per_seg + lp];
      ent[e * 4 + 1] = (int32_t)lp;
      ent[e * 4 + 2] = (int32_t)(j - lp * pr);
    }
    if (p.page_used != nullptr) p.page_used[(int64_t)seg * p.pages_per_seg + lp] = 1;
    ++e;
  }
  // the run ending at bit b is the last one started at or before b
  while (en != 0u) {
    const int b = __builtin_ctz(en);
    en &= en - 1u;
    const int64_t idx = e0 + __popc(r.starts & ((2u << b) - 1u)) - 1;
    const int64_t j = j0 + b;
    if (idx < p.max_entries) ent[idx * 4 + 3] = (int32_t)(j - (j / pr) * pr + 1);
  }
  if (last_tile) {
    int64_t kept;
    block_exclusive_scan<kThreads>(kept_part, red, &kept);
    if (threadIdx.x == 0) {
      p.seg_len[seg] = (int32_t)kept;
      p.n_entries[seg] = finish_segment(p, seg, (int32_t)runs);
    }
  }
}

// One workgroup per segment, the whole selection in one pass over the mask:
// every thread holds the keep bits of kSweeps runs of 16 positions (all their
// loads in flight at once), ranks its run starts over the segment and writes
// the entries; the page flags are gathered in LDS and stored once.  A 16-run
// lies in one page, so a thread needs one page number per run.
constexpr int kUsedPages = (int)(kPanelPositions / 32);  // most pages of a panel

__global__ __launch_bounds__(kSweepThreads) void page_select_kernel(PageSelectParams p) {
  __shared__ int32_t tmp[kSweeps * kSweepThreads / kWave];
  __shared__ int32_t kept_sum[kSweepThreads / kWave];
  __shared__ __align__(16) uint8_t used[kUsedPages];
  const int seg = blockIdx.x;
  const int tid = threadIdx.x;
  const int pr = p.page_rows;
  const int sh = __builtin_ctz(pr);  // page sizes are powers of two
  const int32_t* table = p.table + (int64_t)seg * p.pages_per_seg;
  int32_t* ent = p.entries + (int64_t)seg * p.max_entries * 4;
  int32_t first = 0;  // entries of the panels before
  int32_t kept = 0;
  for (int64_t base = 0; base < p.T; base += kPanelPositions) {
    uint32_t starts[kSweeps], ends[kSweeps];
    int rank[kSweeps];
    uint32_t bits[kSweeps];
    panel_bits(p.mask, seg, p.nseg, base, p.T, bits);
    if (p.page_used != nullptr)
      for (int i = tid; i < kUsedPages / 4; i += kSweepThreads) reinterpret_cast<uint32_t*>(used)[i] = 0u;
    int32_t page[kSweeps];
#pragma unroll
    for (int c = 0; c < kSweeps; ++c) {
      const int64_t j0 = base + c * kSweepPositions + tid * 16;
      const uint32_t keep = bits[c];
      const uint32_t left = __shfl_up(keep, 1, kWave);
      const uint32_t right = __shfl_down(keep, 1, kWave);
      const uint32_t prev = (j0 & (pr - 1)) == 0 ? 0u : (left >> 15) & 1u;
      const uint32_t next = ((j0 + 16) & (pr - 1)) == 0 ? 0u : right & 1u;
      starts[c] = keep & ~((keep << 1) | prev);
      ends[c] = keep & ~((keep >> 1) | (next << 15));
      kept += __popc(keep);
      rank[c] = __popc(starts[c]);
      page[c] = starts[c] != 0u ? table[j0 >> sh] : 0;
    }
    const int runs = sweep_ranks(rank, tmp);  // its barrier also follows the clearing of `used`
#pragma unroll
    for (int c = 0; c < kSweeps; ++c) {
      const int64_t j0 = base + c * kSweepPositions + tid * 16;
      const int32_t lp = (int32_t)(j0 >> sh);
      const int32_t slot0 = (int32_t)(j0 & (pr - 1));
      uint32_t st = starts[c], en = ends[c];
      const int64_t e0 = (int64_t)first + rank[c];
      if (st != 0u && p.page_used != nullptr) used[lp - (int32_t)(base >> sh)] = 1;
      for (int64_t e = e0; st != 0u; st &= st - 1u, ++e)
        if (e < p.max_entries) {
          *reinterpret_cast<int2*>(ent + e * 4) = int2{page[c], lp};
          ent[e * 4 + 2] = slot0 + __builtin_ctz(st);
        }
      // the run ending at bit b is the last one started at or before b
      for (; en != 0u; en &= en - 1u) {
        const int b = __builtin_ctz(en);
        const int64_t e = e0 + __popc(starts[c] & ((2u << b) - 1u)) - 1;
        if (e < p.max_entries) ent[e * 4 + 3] = slot0 + b + 1;
      }
    }
    first += runs;
    __syncthreads();  // flags complete; tmp free
    if (p.page_used != nullptr) {
      const int64_t pg0 = base >> sh;
      int64_t n = (kPanelPositions >> sh) < p.pages_per_seg - pg0 ? (kPanelPositions >> sh) : p.pages_per_seg - pg0;
      uint8_t* out = p.page_used + (int64_t)seg * p.pages_per_seg + pg0;
      for (int64_t i = tid; i < n; i += kSweepThreads) out[i] = used[i];
      __syncthreads();  // the flags are cleared again for the next panel
    }
  }
  // retained length; the append region [T, T + cap), one entry per page it
  // touches; flags of the pages past the panels (the append region's pages
  // are marked last: a panel's flags may cover the first of them)
  const int wave = tid / kWave;
  for (int o = kWave / 2; o > 0; o >>= 1) kept += __shfl_xor(kept, o, kWave);
  if ((tid & (kWave - 1)) == 0) kept_sum[wave] = kept;
  const int64_t a0 = (int64_t)p.T >> sh, a1 = p.cap > 0 ? ((int64_t)p.T + p.cap - 1) >> sh : a0 - 1;
  if (p.page_used != nullptr) {
    const int64_t panels = (p.T + kPanelPositions - 1) / kPanelPositions;
    uint8_t* out = p.page_used + (int64_t)seg * p.pages_per_seg;
    for (int64_t lp = panels * (kPanelPositions >> sh) + tid; lp < p.pages_per_seg; lp += kSweepThreads) out[lp] = 0;
  }
  __syncthreads();
  for (int64_t lp = a0 + tid; lp <= a1; lp += kSweepThreads) {
    const int64_t e = first + (lp - a0);
    if (e < p.max_entries) {
      const int64_t lo = p.T > (lp << sh) ? p.T - (lp << sh) : 0;
      const int64_t end = (int64_t)p.T + p.cap - (lp << sh);
      *reinterpret_cast<int4*>(ent + e * 4) =
          int4{table[lp], (int32_t)lp, (int32_t)lo, (int32_t)(end < pr ? end : pr)};
    }
    if (p.page_used != nullptr) p.page_used[(int64_t)seg * p.pages_per_seg + lp] = 1;
  }
  if (tid == 0) {
    int32_t n = 0;
    for (int i = 0; i < kSweepThreads / kWave; ++i) n += kept_sum[i];
    p.seg_len[seg] = n;
    p.n_entries[seg] = (int32_t)(first + (a1 - a0 + 1));
  }
}

// Segments of a context of length 0: no retained position, only the append
// region.
__global__ __launch_bounds__(kThreads) void page_empty_kernel(PageSelectParams p) {
  const int s = blockIdx.x * kThreads + threadIdx.x;
  if (s >= p.nseg) return;
  p.seg_len[s] = 0;
  p.n_entries[s] = finish_segment(p, s, 0);
}

}  // namespace

// Whether one workgroup per segment walks its whole mask row (in panels one
// after the other), or the workgroups take 4096-position tiles in two passes.
// A workgroup fills its CU, so the segments take rounds of 256: past the first
// round short rows lose (a round costs 6 us), and a few long rows leave the
// chip idle.  Rows of very many runs spend their time writing entries, which
// the tiles spread wider: the caller's bound on the entries tells (a mapped
// mask has one per page and bin, far below T / 4).  The selection alone, whole
// / tiles, us (128-row pages, 35% kept in runs of 64): 16 segments of 65,536
// 10.3 / 9.9; 64 of 131,072 12.0 / 15.1, of 262,144 19.9 / 21.5; 128 of 524,288
// 43 / 64; 256 of 131,072 14.1 / 39; 512 of 1,024 15.6 / 9.8, of 24,576 16.4 /
// 18.2; 1,024 of 16,384 29 / 22, of 32,768 31 / 39; 4,096 of 1,024 100 / 21, of
// 32,768 117 / 130.  Single positions (an entry per 4.4): 16 of 32,768 17.8 /
// 12.0, 256 of 131,072 106 / 87.
bool select_whole_segments(const PageSelectParams& p) {
  const int64_t T = p.T, nseg = p.nseg;
  if (T > 4 * kPanelPositions) return false;
  if (nseg <= 256 && T <= 10240) return true;
  if (p.max_entries > T / 4) return false;
  if (nseg <= 256) return T <= 32768 || (nseg >= 64 && T <= nseg * kCompactTile);
  return T >= (nseg <= 512 ? 24000 : 32768);
}

size_t page_select_workspace_bytes(int64_t nseg, int64_t T) {
  const int64_t ntiles = (T + kCompactTile - 1) / kCompactTile;
  return (size_t)((ntiles > kSumTiles ? 3 : 2) * nseg * ntiles) * sizeof(int32_t);
}

hipError_t launch_page_select(PageSelectParams p, hipStream_t stream) {
  if (p.nseg == 0) return hipSuccess;
  if (p.ntiles > 0 && select_whole_segments(p)) {
    hipLaunchKernelGGL(page_select_kernel, dim3(p.nseg), dim3(kSweepThreads), 0, stream, p);
  } else if (p.ntiles > 0) {
    // workspace: tile counts, kept positions, and for long contexts each tile's first entry
    p.tile_base = p.ntiles > kSumTiles ? p.tile_kept + (int64_t)p.nseg * p.ntiles : nullptr;
    hipLaunchKernelGGL(page_count_kernel, dim3(p.ntiles, p.nseg), dim3(kThreads), 0, stream, p);
    if (p.tile_base != nullptr)
      hipLaunchKernelGGL(page_scan_kernel, dim3((p.nseg + kThreads - 1) / kThreads), dim3(kThreads), 0, stream, p);
    hipLaunchKernelGGL(page_emit_kernel, dim3(p.ntiles, p.nseg), dim3(kThreads), 0, stream, p);
  } else {
    hipLaunchKernelGGL(page_empty_kernel, dim3((p.nseg + kThreads - 1) / kThreads), dim3(kThreads), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace dkv
