// Contig sizes and GreedyPartitioning (Sections 4.2 and 4.3).
//
//  k_part_zero / k_part_count  per-label counter (4 per read, +1 per read of
//                              degree 1 in L): size q = c >> 2, roots of degree
//                              one = c & 3 (2 for a path, 0 for a cycle)
//  k_part_compact              eligible components in ascending label order
//                              (single-pass look-back scan), label -> index map
//  k_part_wzero / k_part_weight bases weights (lengths of a component's reads)
//  k_part_lpt                  one workgroup: sort by (weight desc, label asc),
//                              exact LPT, sort by (bin, label), read offsets
//  k_part_hist / k_part_place  the (bin, label) order and read offsets over many
//                              workgroups instead, where one-read components
//                              make up a large graph's
#include "cg_device.h"

namespace cg {

constexpr int kPartBlock = 256;

__global__ __launch_bounds__(kPartBlock) void k_part_zero(int32_t n, int32_t *__restrict__ cnt) {
  const int64_t v = (int64_t)blockIdx.x * kPartBlock + threadIdx.x;
  if (v < n) cnt[v] = 0;
}

__global__ __launch_bounds__(kPartBlock) void k_part_count(int32_t n, const uint8_t *__restrict__ flags,
                                                           const int32_t *__restrict__ label,
                                                           int32_t *cnt) {
  const int64_t v = (int64_t)blockIdx.x * kPartBlock + threadIdx.x;
  if (v >= n) return;
  const uint32_t f = flags[v];
  const uint32_t degL = ((f >> 1) & 1) + ((f >> 2) & 1);
  atomicAdd((uint32_t *)cnt + label[v], 4u + (degL == 1 ? 1u : 0u));
}

// kCompactPer consecutive reads per thread, so that every block of a large
// graph is resident at once and the look-back chain is short
constexpr int kCompactPer = 4;
__global__ __launch_bounds__(kScanBlock) void k_part_compact(
    int32_t n, const uint8_t *__restrict__ flags, int32_t *label_comp, int32_t min_reads,
    int32_t *__restrict__ comp_label, int32_t *__restrict__ comp_size,
    uint8_t *__restrict__ comp_kind, int32_t *__restrict__ d_n_comp, ScanCtx sc, int nblocks) {
  const int blk = lookback_ticket(sc);
  const int64_t v0 = ((int64_t)blk * kScanBlock + threadIdx.x) * kCompactPer;
  uint32_t c[kCompactPer];
  bool elig[kCompactPer];
  uint32_t cnt = 0;
#pragma unroll
  for (int k = 0; k < kCompactPer; ++k) {
    const int64_t v = v0 + k;
    c[k] = v < n ? (uint32_t)label_comp[v] : 0u;
    elig[k] = v < n && (c[k] >> 2) >= (uint32_t)min_reads && !(flags[v] & 1);
    cnt += elig[k] ? 1u : 0u;
  }
  unsigned long long incl_end;
  unsigned long long ex = lookback_block_scan(sc, blk, (unsigned long long)cnt, &incl_end);
#pragma unroll
  for (int k = 0; k < kCompactPer; ++k) {
    const int64_t v = v0 + k;
    if (v >= n) continue;
    if (elig[k]) {
      const uint32_t q = c[k] >> 2;
      comp_label[ex] = (int32_t)v;
      comp_size[ex] = (int32_t)q;
      comp_kind[ex] = q == 1 ? CG_KIND_SINGLE : ((c[k] & 3u) ? CG_KIND_PATH : CG_KIND_CYCLE);
      label_comp[v] = (int32_t)ex;
      ++ex;
    } else {
      label_comp[v] = -1;
    }
  }
  if (blk == nblocks - 1 && threadIdx.x == 0) *d_n_comp = (int32_t)incl_end;
  lookback_finish(sc, nblocks);
}

// ---------------------------------------------------------------------------
// Single-workgroup sort + LPT.
// ---------------------------------------------------------------------------
// bases weight of each eligible component: the lengths of its reads
__global__ __launch_bounds__(kPartBlock) void k_part_wzero(int32_t n, uint64_t *__restrict__ w) {
  const int64_t v = (int64_t)blockIdx.x * kPartBlock + threadIdx.x;
  if (v < n) w[v] = 0;
}

__global__ __launch_bounds__(kPartBlock) void k_part_weight(int32_t n, const int32_t *__restrict__ label,
                                                            const int32_t *__restrict__ label_comp,
                                                            const uint32_t *__restrict__ read_len,
                                                            uint64_t *w) {
  const int64_t v = (int64_t)blockIdx.x * kPartBlock + threadIdx.x;
  if (v >= n) return;
  const int32_t c = label_comp[label[v]];
  if (c >= 0) atomicAdd((unsigned long long *)w + c, (unsigned long long)read_len[v]);
}

// later: k_part_place takes the (bin, label) order
__global__ __launch_bounds__(kLptBlock) void k_part_lpt(int32_t P, const int32_t *__restrict__ d_n_comp,
                                                        const int32_t *__restrict__ comp_size,
                                                        const uint64_t *__restrict__ weight,
                                                        unsigned int *status, int32_t *comp_bin,
                                                        int32_t *__restrict__ comp_rank,
                                                        int32_t *__restrict__ comp_start,
                                                        uint64_t *__restrict__ bin_load,
                                                        uint64_t *g_keys, int32_t *g_bin,
                                                        uint64_t *g_bins, int later) {
  __shared__ uint64_t s_keys[kSortCapLds];
  __shared__ int32_t s_bin[kSortCapLds];
  __shared__ uint64_t s_binA[kBinCapLds], s_binB[kBinCapLds];
  __shared__ uint32_t s_cnt[kLptBlock / kWave * 256];
  uint32_t *big_cnt = reinterpret_cast<uint32_t *>(s_keys);  // s_keys is the LDS form's
  const int nc = *d_n_comp;
  int32_t *rank = later ? nullptr : comp_rank;
  int32_t *bin_of = later ? comp_bin : g_bin;
  if (nc <= kSortCapLds && P <= kBinCapLds && !later)
    lpt_body<kLptBlock, false>(nc, P, comp_size, weight, s_keys, s_bin, s_cnt, s_binA, s_binB,
                               comp_bin, comp_rank, comp_start, bin_load, nullptr, status);
  else
    lpt_body<kLptBlock, true>(nc, P, comp_size, weight, g_keys, bin_of, big_cnt,
                              P <= kBinCapLds ? s_binA : g_bins,
                              P <= kBinCapLds ? s_binB : g_bins + P, comp_bin, rank, comp_start,
                              bin_load, nullptr, status);
}

// ---------------------------------------------------------------------------
// The (bin, label) order of many components: a counting sort by bin over
// chunks of consecutive components (they are indexed in label order), a
// workgroup each.  k_part_hist counts the components and reads of every bin
// per chunk; k_part_place adds up the chunks before its own and the bins
// before each bin, splits its chunk among its waves the same way, and writes
// every component's rank and first read.  (components << 32) | reads in one
// word, each below 2^31.  One workgroup sorting 110,000 components in global
// memory took 3 ms, its scattered stores alone 0.1 ms; the two passes take
// about 10 us.
// ---------------------------------------------------------------------------
constexpr int kPlaceBlock = 256;
constexpr int kPlaceWaves = kPlaceBlock / kWave;
constexpr int kPlaceChunk = 2048;  // components per chunk at least
constexpr int kPlaceChunks = 128;  // chunks at most, so that adding them up stays short
static_assert(kBinCapLds <= kPlaceChunk && kPlaceChunk <= kSortCapLds,
              "a chunk's counts take the key scratch of its components (two keys a read)");

__device__ __forceinline__ uint64_t place_word(int32_t reads) {
  return (1ull << 32) | (uint32_t)reads;
}

__global__ __launch_bounds__(kPlaceBlock) void k_part_hist(int32_t P, int32_t chunk,
                                                           const int32_t *__restrict__ d_n_comp,
                                                           const int32_t *__restrict__ comp_size,
                                                           const int32_t *__restrict__ comp_bin,
                                                           uint64_t *__restrict__ hist) {
  __shared__ unsigned long long h[kBinCapLds];
  const int64_t nc = *d_n_comp, c0 = (int64_t)blockIdx.x * chunk;
  if (c0 >= nc) return;
  for (int b = threadIdx.x; b < P; b += kPlaceBlock) h[b] = 0;
  __syncthreads();
  const int64_t c1 = c0 + chunk < nc ? c0 + chunk : nc;
#pragma unroll 4
  for (int64_t c = c0 + threadIdx.x; c < c1; c += kPlaceBlock)
    atomicAdd(h + comp_bin[c], (unsigned long long)place_word(comp_size[c]));
  __syncthreads();
  for (int b = threadIdx.x; b < P; b += kPlaceBlock) hist[(int64_t)blockIdx.x * P + b] = h[b];
}

__global__ __launch_bounds__(kPlaceBlock) void k_part_place(int32_t P, int32_t chunk,
                                                            const int32_t *__restrict__ d_n_comp,
                                                            const int32_t *__restrict__ comp_size,
                                                            const int32_t *__restrict__ comp_bin,
                                                            const uint64_t *__restrict__ hist,
                                                            int32_t *__restrict__ comp_rank,
                                                            int32_t *__restrict__ comp_start) {
  __shared__ unsigned long long pos[kBinCapLds];
  __shared__ unsigned long long wpos[kPlaceWaves][kBinCapLds];
  __shared__ unsigned long long sh[kPlaceWaves + 1];
  const int64_t nc = *d_n_comp, c0 = (int64_t)blockIdx.x * chunk;
  if (c0 >= nc) return;
  const int chunks = (int)((nc + chunk - 1) / chunk);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), l = lane_id();
  // this wave's components
  const int per = (chunk + kPlaceWaves - 1) / kPlaceWaves;
  const int64_t a = c0 + (int64_t)w * per, ce = c0 + chunk < nc ? c0 + chunk : nc;
  const int64_t z = a + per < ce ? a + per : ce;
  unsigned long long *my = wpos[w];
  for (int b = l; b < P; b += kWave) my[b] = 0;
  wave_lds_sync();
#pragma unroll 4
  for (int64_t c = a + l; c < z; c += kWave)
    atomicAdd(my + comp_bin[c], (unsigned long long)place_word(comp_size[c]));
  // where this chunk's part of each bin starts
  unsigned long long carry = 0;
  for (int base = 0; base < P; base += kPlaceBlock) {
    const int b = base + (int)threadIdx.x;
    unsigned long long before = 0, all = 0;
    if (b < P) {
#pragma unroll 8
      for (int k = 0; k < chunks; ++k) {
        const unsigned long long x = hist[(int64_t)k * P + b];
        before += k < (int)blockIdx.x ? x : 0ull;
        all += x;
      }
    }
    unsigned long long tot;
    const unsigned long long ex = block_excl_scan<unsigned long long, kPlaceBlock>(all, sh, &tot);
    if (b < P) pos[b] = carry + ex + before;
    carry += tot;
  }
  __syncthreads();
  for (int b = threadIdx.x; b < P; b += kPlaceBlock) {
    unsigned long long x = pos[b];
    for (int k = 0; k < kPlaceWaves; ++k) {
      const unsigned long long y = wpos[k][b];
      wpos[k][b] = x;
      x += y;
    }
  }
  __syncthreads();
  int kb = 0;
  while ((1 << kb) < P) ++kb;
  const uint64_t below = (1ull << l) - 1ull;
  for (int64_t base = a; base < z; base += kWave) {
    const int64_t c = base + l;
    const bool v = c < z;
    const int32_t b = v ? comp_bin[c] : 0, q = v ? comp_size[c] : 0;
    uint64_t peers = __ballot(v);
    for (int k = 0; k < kb; ++k) {
      const bool bit = (b >> k) & 1;
      const uint64_t m = __ballot(v && bit);
      peers &= bit ? m : ~m;
    }
    const unsigned long long at = my[b];
    // the reads of the lanes of this bin before this one: one each, and
    // what the longer components among them have more
    const int32_t k = __popcll(peers & below);
    int32_t more = 0;
    for (uint64_t big = __ballot(q > 1); big; big &= big - 1) {
      const int t = (int)__builtin_ctzll(big);
      const int32_t bt = __builtin_amdgcn_readlane(b, t), qt = __builtin_amdgcn_readlane(q, t);
      more += bt == b && t < l ? qt - 1 : 0;
    }
    const int32_t rank = (int32_t)(at >> 32) + k, start = (int32_t)(uint32_t)at + k + more;
    wave_lds_sync();
    if (v) {
      comp_rank[c] = rank;
      comp_start[c] = start;
      // the bin's last lane leaves where the next round goes on
      if ((peers & ~below) == 1ull << l)
        my[b] = (unsigned long long)(uint32_t)(rank + 1) << 32 | (uint32_t)(start + q);
    }
    wave_lds_sync();
  }
}

int launch_partition(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const uint8_t *flags,
                     const int32_t *label, int32_t P, int32_t min_reads, int32_t weight,
                     const cg_parts &out, hipStream_t st) {
  const PhaseRange range("cg: GreedyPartitioning");
  const int32_t n = g.n;
  if (min_reads < 1) min_reads = 1;
  const int grid = n > 0 ? (int)((n + kPartBlock - 1) / kPartBlock) : 1;
  if (n > 0) {
    CG_LAUNCH(ctx, k_part_zero, dim3(grid), dim3(kPartBlock), st, n, out.label_comp);
    CG_LAUNCH(ctx, k_part_count, dim3(grid), dim3(kPartBlock), st, n, flags, label,
                       out.label_comp);
  }
  const int nb = scan_blocks(n > 0 ? (n + kCompactPer - 1) / kCompactPer : 1);
  CG_LAUNCH(ctx, k_part_compact, dim3(nb), dim3(kScanBlock), st, n, flags, out.label_comp,
                     min_reads, out.comp_label, out.comp_size, out.comp_kind, out.d_n_comp,
                     scan_ctx(ctx, s), nb);
  const bool bases = weight == CG_WEIGHT_BASES;
  if (bases && n > 0) {
    CG_LAUNCH(ctx, k_part_wzero, dim3(grid), dim3(kPartBlock), st, n, s.comp_w);
    CG_LAUNCH(ctx, k_part_weight, dim3(grid), dim3(kPartBlock), st, n, label, out.label_comp,
                       g.read_len, s.comp_w);
  }
  // one-read components are most of a graph's, so where they are wanted of
  // more reads than the LDS sort holds, the order is left to the passes below
  // (two launches, which the few components of other graphs do not repay)
  const bool place = min_reads <= 1 && n > kSortCapLds && P <= kBinCapLds;
  CG_LAUNCH(ctx, k_part_lpt, dim3(1), dim3(kLptBlock), st, P, out.d_n_comp, out.comp_size,
                     bases ? (const uint64_t *)s.comp_w : nullptr, &ctx->fixed->status,
                     out.comp_bin, out.comp_rank, out.comp_start, out.bin_load, s.keys, s.aux,
                     s.bins, place ? 1 : 0);
  if (place) {
    const int32_t per = (n + kPlaceChunks - 1) / kPlaceChunks;
    const int32_t chunk = per > kPlaceChunk ? per : kPlaceChunk;
    const dim3 chunks((unsigned)((n + chunk - 1) / chunk));
    CG_LAUNCH(ctx, k_part_hist, chunks, dim3(kPlaceBlock), st, P, chunk, out.d_n_comp,
              out.comp_size, out.comp_bin, s.keys);
    CG_LAUNCH(ctx, k_part_place, chunks, dim3(kPlaceBlock), st, P, chunk, out.d_n_comp,
              out.comp_size, out.comp_bin, s.keys, out.comp_rank, out.comp_start);
  }
  return hip_check(hipGetLastError(), "k_part");
}

}  // namespace cg
