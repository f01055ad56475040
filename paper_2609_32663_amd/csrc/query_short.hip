// Query-block attention for short blocks: at most 128 query rows (tokens x
// heads of a group) per segment, or kShortRows (256) over long segments.  What
// the rows compute is what query_attn.hip computes; here the block is so short
// that reading K and V bounds the call, so the kernel is a stream over the
// keys, split like the decode step's, instead of 256-row query tiles.
//
// Work split.  The keys of all segments are laid end to end (plus a fixed
// cost per segment) and cut into P equal slices, one per workgroup; a slice
// that crosses a segment boundary yields one piece per segment.  Every
// workgroup finds its slice from the segment lengths itself, so there is no
// plan kernel.  Piece (w, s) writes its (max, sum, unnormalised output) per
// row to record slot w + s (unique, contiguous per segment) and a combine
// kernel folds a segment's slots in slot order; a segment inside one
// workgroup is written directly.  Without a workspace (keys too few to
// split) workgroup s takes segment s whole.
//
// Inside a workgroup the waves are RW row waves x KW key waves: a row wave
// holds 32 rows (two 16-row groups), the key waves take 32-key tiles in turn.
//   * K and V tiles go from memory straight into LDS, two or three tiles per
//     key wave; the row waves of a key wave share its tiles and meet once per
//     tile (with one row wave nothing meets in the stream);
//   * scores, lazy running max, fp32 probabilities split into two bf16 parts
//     and both products as in query_attn.hip.
// At the end each key wave finishes its share of the output columns: the
// others hand it theirs through LDS (every lane meets the lane that holds the
// same outputs) and it adds them up in key-wave order.
//
// Why a kernel of its own: the 256-row tiles of query_attn.hip do the products
// of all 256 rows whatever the block holds, in two rounds of workgroups after a
// plan kernel.  Reading K and V is the floor here (23 tokens of an 8B layer at
// 32K: 47 MB, 7.4 us); one round of workgroups that stream at 5.9 TB/s, plus
// prologue, first tile, fold and combine took 52.7 -> 27.7 us for append,
// attention and combine together, 4 tokens at 128K 109 -> 43 us, 64 tokens
// (256 rows) 128 -> 92 us.  From 32 rows on the products and the softmax of
// two waves per SIMD (about 3,500 cycles per 64 keys and 128 rows) take longer
// than the stream; more than 256 rows would read K and V more than once.
//
// Compiled like query_attn.hip (no IEEE mode, no NaN semantics).

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dkv_query_device.hpp"

namespace dkv {

namespace {

constexpr int kSKeys = 32;  // keys per tile
constexpr int kSRG = 2;     // 16-row groups per wave
constexpr int kSMergeThreads = 256;
constexpr int kStreamOnce = 2;  // non-temporal: every K and V byte is read once

template <int D>
struct SCfg {
  static constexpr int kRowBytes = D * 2;
  static constexpr int kChunks = D / 32;                 // 16-byte chunks of a row per lane (QK)
  static constexpr int kBlocks = D / 16;                 // 16-column output blocks per lane
  static constexpr int kRowChunks = D / 8;               // 16-byte chunks per row
  static constexpr int kPairs = D / 16;                  // 32-byte column pairs per row
  static constexpr int kDma = kSKeys * kRowChunks / 64;  // direct loads per tile and matrix
};

__device__ __forceinline__ int64_t short_rows(const QueryParams& p, int s) {
  const int32_t len = p.seg_len[s];
  return len < 0 ? 0 : (int64_t)len + p.n_tail + p.n_q;
}

// Tiles in the ring of a key wave: two, or three where a round holds half as
// many keys (one key wave) or the stream is long enough to pay for a third
// tile's longer start (23 tokens, 8B layer: 128K 56.7 us with two, 52.9 with
// three; 32K 27.7 and 29.5; four are slower on both).
template <int RW, int KW, bool NT>
constexpr int short_stages() {
  return KW == 1 || (RW > 1 && NT) ? 3 : 2;
}

template <int D, int RW, int KW, bool NT>
__global__ __launch_bounds__(512)
void query_short_kernel(QueryParams p) {
  using C = SCfg<D>;
  constexpr int RG = kSRG;
  constexpr int kThreads = RW * KW * kWave;
  constexpr int64_t kSegCost = 196608 / (2 * C::kRowBytes);  // as the decode step's
  extern __shared__ __align__(16) int64_t pre[];             // [nseg + 1] unit prefix, [nseg] offsets (split calls)
  // S tiles per key wave and matrix (separate arrays: the compiler then tells
  // the direct loads into one apart from the reads of the others), and what
  // the key waves hand each other at the fold
  constexpr int S = short_stages<RW, KW, NT>();
  constexpr int kTile = KW * kSKeys * D;
  static_assert(S == 2 || S == 3, "the ring's arrays");
  __shared__ __align__(1024) uint16_t k0[kTile], k1[kTile], k2[S > 2 ? kTile : 8];
  __shared__ __align__(1024) uint16_t v0[kTile], v1[kTile], v2[S > 2 ? kTile : 8];
  constexpr int OB = C::kBlocks / KW;  // 16-column output blocks that a key wave finishes
  constexpr int HB = KW == 1 ? 1 : (KW > 2 ? (OB + 1) / 2 : OB);  // handed over at a time
  __shared__ __align__(16) f32x4 fo[KW][RW][KW > 1 ? KW - 1 : 1][HB][kWave];
  __shared__ __align__(16) float fm[KW][RW][RG][16], fl[KW][RW][RG][16];
  __shared__ int64_t red[RW * KW + 1];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave % RW, kw = wave / RW;
  const int n16 = lane & 15;
  const int kg = lane >> 4;
  const int w = blockIdx.x;
  const int nseg = p.nseg;
  const bool split = p.P > 0;

  // ---- this workgroup's slice ------------------------------------------------
  int64_t lo = 0, hi = 0, total = 0, P = 1;
  int s = w;
  if (split) {
    const int per = (nseg + kThreads - 1) / kThreads;
    const int s_lo = tid * per, s_hi = min(nseg, s_lo + per);
    int64_t sum = 0;
    for (int i = s_lo; i < s_hi; ++i) {
      const int64_t rows = short_rows(p, i);
      const int64_t u = rows > 0 ? rows + kSegCost : 0;
      pre[nseg + 1 + i] = p.seg_off[i];
      pre[i] = u;
      sum += u;
    }
    int64_t all;
    int64_t run = block_exclusive_scan<kThreads>(sum, red, &all);
    for (int i = s_lo; i < s_hi; ++i) {
      const int64_t u = pre[i];
      pre[i] = run;
      run += u;
    }
    if (tid == 0) pre[nseg] = all;
    __syncthreads();
    total = q_uniform64(all);
    P = total < p.P ? total : p.P;
  }
  // segments with no rows (not packed) produce zeros
  for (int z = w; z < nseg; z += gridDim.x) {
    if (p.seg_len[z] >= 0) continue;
    const int b = z / p.Hkv, g = z - (z / p.Hkv) * p.Hkv;
    for (int i = tid; i < p.rows * D; i += kThreads) {
      const int r = i / D, tok = r / p.G;
      p.out[(((int64_t)b * p.n_q + tok) * p.Hq + (int64_t)g * p.G + (r - tok * p.G)) * D + i % D] = 0.f;
    }
    if (split && tid == 0) p.seg_meta[2 * z] = p.seg_meta[2 * z + 1] = 0;  // nothing to combine
  }
  if (split) {
    if (w >= P) return;
    lo = (int64_t)w * total / P;
    hi = (int64_t)(w + 1) * total / P;
    int a = 0, b = nseg;  // pre[a] <= lo < pre[b]
    while (b - a > 1) {
      const int mid = (a + b) >> 1;
      if (pre[mid] <= lo) a = mid;
      else b = mid;
    }
    s = a;
  }
  s = __builtin_amdgcn_readfirstlane(s);

  // Scores are taken with |scale|, as in query_attn.hip.
  const bool qneg = p.scale_log2 < 0.f;
  const float cpos = fmaxf(fabsf(p.scale_log2), 1.17549435e-38f);

  // Lane-constant offsets of the direct loads: lane l of instruction i fills
  // 16-byte chunk 64i + l of a tile's LDS layout (chunk c of key row R is
  // bytes 16c .. 16c + 15), as in query_attn.hip:
  //   K: ((R / 16) * kRowChunks + c) * 16 + R % 16
  //   V: ((R / 8) * kPairs + c / 2) * 16 + (R % 8) * 2 + c % 2
  const uint32_t koff = (uint32_t)(n16 * C::kRowBytes + 16 * kg);
  const uint32_t voff = (uint32_t)(((lane >> 1) & 7) * C::kRowBytes + 16 * (2 * kg + (lane & 1)));

  for (; s < nseg; ++s) {
    int64_t seg_lo = 0, seg_hi = 0, a = 0, bnd;
    if (split) {
      if (pre[s] >= hi) break;
      seg_lo = q_uniform64(pre[s]) + kSegCost;
      seg_hi = q_uniform64(pre[s + 1]);
      a = (lo > seg_lo ? lo : seg_lo) - seg_lo;
      bnd = (hi < seg_hi ? hi : seg_hi) - seg_lo;
    } else {
      bnd = q_uniform64(short_rows(p, s));
    }
    if (a >= bnd) {
      if (!split) break;
      continue;
    }
    const int bseq = s / p.Hkv;
    const int g = s - bseq * p.Hkv;
    const int64_t base_len = (split ? seg_hi - seg_lo : bnd) - p.n_q;  // rows every query row sees
    const int64_t row0 = q_uniform64(split ? pre[nseg + 1 + s] : p.seg_off[s]) + a;
    const char* kbase = reinterpret_cast<const char*>(p.k) + row0 * C::kRowBytes;
    const char* vbase = reinterpret_cast<const char*>(p.v) + row0 * C::kRowBytes;
    const int64_t nkeys = q_uniform64(bnd - a);
    // every row sees the piece's keys below this one
    const int64_t all_see = q_uniform64(base_len + 1 - a < nkeys ? base_len + 1 - a : nkeys);

    // Tile t: keys [32t, 32t + 32) of the piece, loaded by its row waves in
    // turn.  Rows past the piece (whole tiles included) read zeros without
    // touching memory; the row displacement is part of the vector offset,
    // which costs these kernels nothing (23 tokens of an 8B layer at 32K 27.7
    // us either way).
    auto load = [&](uint16_t* kt, uint16_t* vt, int64_t t) __attribute__((always_inline)) {
      const int64_t left = nkeys - t * kSKeys;
      const uint32_t nk = (uint32_t)(left <= 0 ? 0 : (left < kSKeys ? left : kSKeys));
      const int64_t from = nk > 0 ? t * kSKeys * C::kRowBytes : 0;
      const __amdgpu_buffer_rsrc_t ks = q_rsrc(kbase + from, nk * C::kRowBytes);
      const __amdgpu_buffer_rsrc_t vs = q_rsrc(vbase + from, nk * C::kRowBytes);
#pragma unroll
      for (int i0 = 0; i0 < C::kDma; i0 += RW) {
        const int i = i0 + rw;
        if (RW > C::kDma && rw >= C::kDma) break;
        const int at = 16 * (4 * i / C::kRowChunks) * C::kRowBytes + 16 * (4 * i % C::kRowChunks);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ks, (__attribute__((address_space(3))) void*)(kt + 512 * i), 16,
                                                 koff + at, 0, 0, NT ? kStreamOnce : 0);
      }
#pragma unroll
      for (int i0 = 0; i0 < C::kDma; i0 += RW) {
        const int i = i0 + rw;
        if (RW > C::kDma && rw >= C::kDma) break;
        const int at = 8 * (4 * i / C::kPairs) * C::kRowBytes + 32 * (4 * i % C::kPairs);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vs, (__attribute__((address_space(3))) void*)(vt + 512 * i), 16,
                                                 voff + at, 0, 0, NT ? kStreamOnce : 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };

    uint16_t* const kb[3] = {k0 + kw * kSKeys * D, k1 + kw * kSKeys * D, S > 2 ? k2 + kw * kSKeys * D : k2};
    uint16_t* const vb[3] = {v0 + kw * kSKeys * D, v1 + kw * kSKeys * D, S > 2 ? v2 + kw * kSKeys * D : v2};
#pragma unroll
    for (int i = 0; i < S - 1; ++i) load(kb[i], vb[i], kw + i * KW);

    // B operand of QK: query row 16 (RG rw + q) + n16, dims 32u + 8kg .. +7;
    // cut: the keys of the piece that the row sees
    u32x4 qb[RG][C::kChunks];
    int64_t cut[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) {
      const int r = 16 * (RG * rw + q) + n16;
      const bool ok = r < p.rows;
      const int tok = ok ? r / p.G : 0;
      const int64_t see = base_len + tok + 1 - a;
      cut[q] = see < nkeys ? see : nkeys;
      const char* qrow = reinterpret_cast<const char*>(p.q) +
                         (((int64_t)bseq * p.n_q + tok) * p.Hq + (int64_t)g * p.G + (ok ? r - tok * p.G : 0)) *
                             C::kRowBytes;
#pragma unroll
      for (int u = 0; u < C::kChunks; ++u) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        qb[q][u] = ok ? *reinterpret_cast<const u32x4*>(qrow + 64 * u + 16 * kg) : z;
        if (qneg) qb[q][u] ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
      }
    }
    float o[RG][C::kBlocks][4];
    float m[RG], l[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) {
#pragma unroll
      for (int b = 0; b < C::kBlocks; ++b) o[q][b][0] = o[q][b][1] = o[q][b][2] = o[q][b][3] = 0.f;
      m[q] = -INFINITY;
      l[q] = 0.f;
    }

    float sc[RG][2][4];
    u32x4 ph[RG], pl[RG];
    // S^T = K Q^T: lane (n16, kg) receives the scores of keys 16j + 4kg + v
    auto qk = [&](const uint16_t* kt) __attribute__((always_inline)) {
      f32x4 acc[RG][2];
#pragma unroll
      for (int q = 0; q < RG; ++q) acc[q][0] = acc[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < C::kChunks; ++u)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const u32x4 ka = *reinterpret_cast<const u32x4*>(&kt[8 * (lane + 16 * (j * C::kRowChunks + 4 * u))]);
#pragma unroll
          for (int q = 0; q < RG; ++q)
            acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka),
                                                                __builtin_bit_cast(bf16x8, qb[q][u]), acc[q][j], 0, 0, 0);
        }
#pragma unroll
      for (int q = 0; q < RG; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) sc[q][j][v] = acc[q][j][v];
    };
    // Scores of tile t to probabilities, as two bf16 parts.
    auto softmax = [&](int64_t t) __attribute__((always_inline)) {
      const int64_t key0 = t * kSKeys;
      if (key0 + kSKeys > all_see) {
        asm volatile("");  // keeps this a branch: the selects would run for every tile
#pragma unroll
        for (int q = 0; q < RG; ++q) {
          const int64_t rel = cut[q] - key0;
          const int lim = (int)(rel < 0 ? 0 : (rel < kSKeys ? rel : kSKeys));  // keys [0, lim) of the tile count
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * j + 4 * kg + v >= lim) sc[q][j][v] = -INFINITY;
        }
      }
      // The reference max moves only when a tile's max passes it by more than
      // kLazy; the wave leaves it and the accumulators alone unless a row's
      // does (one of the row's four lanes sees that by itself).
      float mx[RG];
      bool over = false;
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        mx[q] = sc[q][0][0];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) mx[q] = fmaxf(mx[q], sc[q][j][v]);
        over |= mx[q] * cpos > m[q] + kLazy;
      }
      if (__builtin_amdgcn_ballot_w64(over)) {
#pragma unroll
        for (int q = 0; q < RG; ++q) {
          const float mt = row4_max(mx[q]) * cpos;
          const bool grow = mt > m[q] + kLazy;
          const float alpha = fast_exp2(grow ? m[q] - mt : 0.f);
          m[q] = grow ? mt : m[q];
          l[q] *= alpha;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float av = __shfl(alpha, 4 * kg + v, 64);
#pragma unroll
            for (int b = 0; b < C::kBlocks; ++b) o[q][b][v] *= av;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        const float m_use = m[q] == -INFINITY ? 0.f : m[q];
        float ps = 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            sc[q][j][v] = fast_exp2(__builtin_fmaf(sc[q][j][v], cpos, -m_use));
            ps += sc[q][j][v];
          }
        l[q] += ps;
        asm volatile("" : "+v"(l[q]));  // the sum is formed here, not sunk into a later phase
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t x, y;
          bf16_split(sc[q][e >> 1][2 * (e & 1)], sc[q][e >> 1][2 * (e & 1) + 1], x, y);
          ph[q][e] = x;
          pl[q][e] = y;
        }
      }
    };
    // O += P V; transpose reads as in query_attn.hip: lane 4r + c of group kg
    // reads row 4kg + r (and 16 + 4kg + r), columns 16b + 4c .. + 3
    auto pv = [&](const uint16_t* vt) __attribute__((always_inline)) {
      const uint16_t* vr0 = &vt[8 * ((kg >> 1) * C::kPairs * 16 + (4 * (kg & 1) + (n16 >> 2)) * 2 + ((n16 >> 1) & 1)) +
                                4 * (n16 & 1)];
#pragma unroll
      for (int b0 = 0; b0 < C::kBlocks; b0 += 2) {
        u32x4 vf[2];
#pragma unroll
        for (int bb = 0; bb < 2; ++bb) {
          const int b = b0 + bb;
          const uint2 w0 = __builtin_bit_cast(
              uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vr0 + 8 * 16 * b)));
          const uint2 w1 = __builtin_bit_cast(
              uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vr0 + 8 * 16 * (2 * C::kPairs + b))));
          vf[bb] = u32x4{w0.x, w0.y, w1.x, w1.y};
        }
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int q = 0; q < RG; ++q) {
              const int b = b0 + bb;
              f32x4 c = {o[q][b][0], o[q][b][1], o[q][b][2], o[q][b][3]};
              c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, part ? pl[q] : ph[q]),
                                                          __builtin_bit_cast(bf16x8, vf[bb]), c, 0, 0, 0);
              o[q][b][0] = c[0];
              o[q][b][1] = c[1];
              o[q][b][2] = c[2];
              o[q][b][3] = c[3];
            }
      }
    };

    // Waits until at most the `out` youngest loads of the wave are out;
    // with several row waves all meet then, so that the tiles' rows are
    // visible to each and everybody has left what it read before.
    auto arrive = [&](auto out) __attribute__((always_inline)) {
      constexpr int kOut = decltype(out)::value;
      constexpr int kWait = 0x0F70 | (kOut & 15) | ((kOut >> 4) << 14);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(kWait);
      if (RW > 1) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // rounds of KW tiles, the same number for every wave of the workgroup
    const int64_t nround = q_uniform64((nkeys + kSKeys * KW - 1) / (kSKeys * KW));
    // A single row wave issues tile t + S - 1 before it waits for tile t
    // (only it reads the buffer); with several that must follow the meeting.
    for (int64_t r0 = 0; r0 < nround; r0 += S) {
#pragma unroll
      for (int i = 0; i < S; ++i) {
        const int64_t r = r0 + i;
        if (r < nround) {
          if (RW == 1) load(kb[(i + S - 1) % S], vb[(i + S - 1) % S], kw + (r + S - 1) * KW);
          arrive(std::integral_constant<int, (RW == 1 ? S - 1 : S - 2) * 2 * C::kDma / RW>{});
          if (RW > 1) load(kb[(i + S - 1) % S], vb[(i + S - 1) % S], kw + (r + S - 1) * KW);
          qk(kb[i]);
          softmax(kw + r * KW);
          pv(vb[i]);
        }
      }
    }
    // no direct load may still be writing LDS when the next piece begins or
    // the workgroup ends
    __builtin_amdgcn_s_waitcnt(0x0F70);

    // ---- fold the key waves and write the output or this piece's record --------
    // Key wave k finishes output blocks k OB .. k OB + OB - 1: the others hand
    // it theirs (the lane that holds the same outputs), row group by row
    // group, and it adds them up in key-wave order.
    bool single = true;
    float* rec = p.rec;
    if (split) {
      const int64_t w_first = owner_of(seg_lo, total, P);
      const int64_t w_last = owner_of(seg_hi - 1, total, P);
      single = w_first == w_last;
      if (w == w_first && tid == 0) {
        p.seg_meta[2 * s] = (int32_t)(w_first + s);
        p.seg_meta[2 * s + 1] = (int32_t)(w_last - w_first + 1);
      }
      rec = p.rec + (int64_t)(w + s) * p.rec_rows * (D + 2);
    }
#pragma unroll
    for (int q = 0; q < RG; ++q) {
      l[q] = lane_xor_sum<16>(l[q]);
      if (kg == 0) {
        fm[kw][rw][q][n16] = m[q];
        fl[kw][rw][q][n16] = l[q];
      }
    }
#pragma unroll
    for (int z = 0; z < RG * OB / HB; ++z) {
      const int q = z / (OB / HB), h0 = z % (OB / HB) * HB;  // row group, first of the HB blocks
      if (z > 0) __syncthreads();
#pragma unroll
      for (int k = 0; k < KW; ++k)
        if (kw != k) {
#pragma unroll
          for (int b = 0; b < HB; ++b) {
            const int x = k * OB + h0 + b;
            fo[k][rw][kw < k ? kw : kw - 1][b][lane] = f32x4{o[q][x][0], o[q][x][1], o[q][x][2], o[q][x][3]};
          }
        }
      __syncthreads();
      f32x4 M = *reinterpret_cast<const f32x4*>(&fm[0][rw][q][4 * kg]);
#pragma unroll
      for (int k = 1; k < KW; ++k) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(&fm[k][rw][q][4 * kg]);
#pragma unroll
        for (int v = 0; v < 4; ++v) M[v] = fmaxf(M[v], x[v]);
      }
      f32x4 L = {0.f, 0.f, 0.f, 0.f}, A[HB];
#pragma unroll
      for (int b = 0; b < HB; ++b) A[b] = L;
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(&fm[k][rw][q][4 * kg]);
        const f32x4 y = *reinterpret_cast<const f32x4*>(&fl[k][rw][q][4 * kg]);
        f32x4 f;
#pragma unroll
        for (int v = 0; v < 4; ++v) f[v] = fast_exp2(x[v] - (M[v] == -INFINITY ? 0.f : M[v]));
        L += f * y;
#pragma unroll
        for (int b = 0; b < HB; ++b) {
          const int x2 = k * OB + h0 + b;
          f32x4 c;
          if (kw == k) c = f32x4{o[q][x2][0], o[q][x2][1], o[q][x2][2], o[q][x2][3]};
          else c = fo[kw][rw][k < kw ? k : k - 1][b][lane];
          A[b] += f * c;
        }
      }
      const int r0 = 16 * (RG * rw + q) + 4 * kg;    // this lane's rows: r0 .. r0 + 3
      const int c0 = 16 * (OB * kw + h0) + n16;      // and columns: c0 + 16b
      if (single) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = r0 + v;
          if (r < p.rows) {
            const int tok = r / p.G;
            float* orow = p.out + (((int64_t)bseq * p.n_q + tok) * p.Hq + (int64_t)g * p.G + (r - tok * p.G)) * D;
            const float inv = L[v] > 0.f ? 1.f / L[v] : 0.f;
#pragma unroll
            for (int b = 0; b < HB; ++b) orow[c0 + 16 * b] = A[b][v] * inv;
          }
        }
      } else if (r0 < p.rows) {  // rec_rows covers whole groups of 4 rows
        if (kw == 0 && h0 == 0 && n16 == 0) {
          *reinterpret_cast<f32x4*>(rec + r0) = M;
          *reinterpret_cast<f32x4*>(rec + p.rec_rows + r0) = L;
        }
        float* rrow = rec + 2 * p.rec_rows + (int64_t)r0 * D + c0;
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int b = 0; b < HB; ++b) rrow[v * D + 16 * b] = A[b][v];
      }
    }
    if (!split) break;
    __syncthreads();  // the fold's LDS is reused by the next piece
  }
}

// Combine kernel: one workgroup per (segment, row), as the decode step's:
// thread (ph, cq) folds pieces ph, ph + kPhases, ... of columns 4cq..4cq+3,
// kBatch records per memory round trip, then the phases are folded in order.
template <int D>
__global__ __launch_bounds__(kSMergeThreads) void query_short_merge_kernel(QueryParams p) {
  constexpr int kQuads = D / 4;
  constexpr int kPhases = kSMergeThreads / kQuads;
  constexpr int kBatch = 8;
  __shared__ __align__(16) f32x4 xa[kSMergeThreads];
  __shared__ float xm[kSMergeThreads], xl[kSMergeThreads];
  const int s = blockIdx.x / p.rows;
  const int r = blockIdx.x - s * p.rows;
  const int n = p.seg_meta[2 * s + 1];
  if (n <= 1) return;
  const int64_t stride = (int64_t)p.rec_rows * (D + 2);
  const float* first = p.rec + (int64_t)p.seg_meta[2 * s] * stride;
  const int tid = threadIdx.x;
  const int cq = tid % kQuads, ph = tid / kQuads;
  float M = -INFINITY, L = 0.f;
  f32x4 A = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = ph; k0 < n; k0 += kPhases * kBatch) {
    float m[kBatch], l[kBatch];
    f32x4 a[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int k = k0 + i * kPhases;
      m[i] = -INFINITY;
      l[i] = 0.f;
      a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k < n) {
        const float* rec = first + (int64_t)k * stride;
        m[i] = rec[r];
        l[i] = rec[p.rec_rows + r];
        a[i] = *reinterpret_cast<const f32x4*>(rec + 2 * p.rec_rows + (int64_t)r * D + 4 * cq);
      }
    }
    float mb = M;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) mb = fmaxf(mb, m[i]);
    const float mu = mb == -INFINITY ? 0.f : mb;
    const float rs = fast_exp2(M - mu);
    L *= rs;
    A *= rs;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float f = fast_exp2(m[i] - mu);
      L += f * l[i];
      A += f * a[i];
    }
    M = mb;
  }
  xm[tid] = M;
  xl[tid] = L;
  xa[tid] = A;
  __syncthreads();
  if (tid < kQuads) {
    float Mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < kPhases; ++q) Mx = fmaxf(Mx, xm[tid + q * kQuads]);
    const float mu = Mx == -INFINITY ? 0.f : Mx;
    float Lt = 0.f;
    f32x4 At = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kPhases; ++q) {
      const int t = tid + q * kQuads;
      const float f = fast_exp2(xm[t] - mu);
      Lt += f * xl[t];
      At += f * xa[t];
    }
    const int bseq = s / p.Hkv, g = s - (s / p.Hkv) * p.Hkv;
    const int tok = r / p.G;
    float* o = p.out + (((int64_t)bseq * p.n_q + tok) * p.Hq + (int64_t)g * p.G + (r - tok * p.G)) * D + 4 * cq;
    *reinterpret_cast<f32x4*>(o) = At * (Lt > 0.f ? 1.f / Lt : 0.f);
  }
}

template <int D, int RW, int KW>
hipError_t launch_short_r(const QueryParams& p, hipStream_t stream) {
  const size_t lds = p.P > 0 ? (2 * (size_t)p.nseg + 1) * sizeof(int64_t) : 0;
  const dim3 grid((unsigned)(p.P > 0 ? p.P : p.nseg)), block(RW * KW * kWave);
  if (p.stream_once) hipLaunchKernelGGL((query_short_kernel<D, RW, KW, true>), grid, block, lds, stream, p);
  else hipLaunchKernelGGL((query_short_kernel<D, RW, KW, false>), grid, block, lds, stream, p);
  if (p.P > 1)
    hipLaunchKernelGGL((query_short_merge_kernel<D>), dim3((unsigned)(p.nseg * p.rows)), dim3(kSMergeThreads), 0,
                       stream, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_short_d(const QueryParams& p, hipStream_t stream) {
  if (p.rows <= 32) return launch_short_r<D, 1, 4>(p, stream);
  if (p.rows <= 64) return launch_short_r<D, 2, 2>(p, stream);
  if (p.rows <= 128) return launch_short_r<D, 4, 2>(p, stream);
  return launch_short_r<D, 8, 1>(p, stream);
}

}  // namespace

hipError_t launch_query_short(const QueryParams& p, int head_dim, hipStream_t stream) {
  return head_dim == 64 ? launch_short_d<64>(p, stream) : launch_short_d<128>(p, stream);
}

}  // namespace dkv
