// Contig sizes and GreedyPartitioning (Sections 4.2 and 4.3).
//
//  k_part_zero / k_part_count  per-label counter (4 per read, +1 per read of
//                              degree 1 in L): size q = c >> 2, roots of degree
//                              one = c & 3 (2 for a path, 0 for a cycle); in the
//                              whole path the count also finishes the component
//                              labels and gives every read its member slot
//  k_part_chunks               eligible roots per chunk of reads, for a least
//                              size that the flags do not decide
//  k_part_compact              eligible components in ascending label order,
//                              label -> index map: a workgroup per chunk adds up
//                              the chunks before its own
//  k_part_wzero / k_part_weight bases weights (lengths of a component's reads)
//  k_part_lpt                  one workgroup: sort by (weight desc, label asc),
//                              exact LPT, sort by (bin, label), read offsets
//  k_part_hist / k_part_place  the (bin, label) order and read offsets over many
//                              workgroups instead, where one-read components
//                              make up a large graph's
#include "cg_device.h"

namespace cg {

constexpr int kPartBlock = 256;

__global__ __launch_bounds__(kPartBlock) void k_part_zero(int32_t n, const uint8_t *__restrict__ flags,
                                                          int32_t *__restrict__ cnt) {
  const int64_t v = (int64_t)blockIdx.x * kPartBlock + threadIdx.x;
  if (v < n) cnt[v] = (flags[v] & 6) ? 0 : 4;
}

// Chunks of consecutive reads, a workgroup each, for the count and the
// compaction: rounds of kChunkRound reads, and as many rounds as keep the
// chunks at kChunks, so that adding up the chunks before one's own stays a
// load per thread.
constexpr int kChunkBlock = 1024;
constexpr int kChunkPer = 2;
constexpr int kChunkRound = kChunkBlock * kChunkPer;
constexpr int kChunks = 1024;
static int chunk_rounds(int32_t n) {
  const int64_t rounds = ((int64_t)n + kChunkRound - 1) / kChunkRound;
  return (int)((rounds + kChunks - 1) / kChunks);
}
static int chunk_count(int32_t n) {
  const int64_t per = (int64_t)kChunkRound * chunk_rounds(n);
  return n > 0 ? (int)(((int64_t)n + per - 1) / per) : 1;
}

// The workgroup's sum of x, in thread 0.
__device__ __forceinline__ uint32_t chunk_sum(uint32_t x, uint32_t *sh) {
  x = wave_sum(x);
  if (lane_id() == 0) sh[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x < kWave) x = wave_sum(threadIdx.x < kChunkBlock / kWave ? sh[threadIdx.x] : 0u);
  return x;
}

// Reads without kept entries are counted already (first_count).  A
// workgroup's others are counted per component in an LDS hash table first:
// one atomic per read on the component's counter queues on its address
// (about 4.5 ns each: 57 us for the 15,000 reads of 13 components).
// kFind: the labels are a forest still; every read's is set to its root, and
// slot gives its place among its component's reads.  kBases: the lengths are
// added up with the counts (two passes over all reads after the compaction,
// with an atomic per read, took 11.6 us of the 17 Mbp graph's 88).
struct CountExtra {
  int32_t *slot;
  const Fixed *fx;  // branch and entry counts of the mask pass, mask_parts of them
  int mask_parts;
  int32_t *d_counts;
  const uint32_t *read_len;  // kBases: lengths, added up at each root
  uint64_t *root_w;
};
constexpr int kCountSlots = 2 * kChunkRound;  // at most half full
template <bool kFind, bool kBases>
__global__ __launch_bounds__(kChunkBlock) void k_part_count(int32_t n, int rounds,
                                                            const uint8_t *__restrict__ flags,
                                                            int32_t *label, int32_t *cnt,
                                                            int32_t min_reads,
                                                            uint2 *__restrict__ chunks,
                                                            CountExtra ex) {
  __shared__ int32_t s_key[kCountSlots];
  __shared__ uint32_t s_cnt[kCountSlots];
  __shared__ unsigned long long s_w[kBases ? kCountSlots : 1];
  __shared__ uint32_t sh[kChunkBlock / kWave];
  uint32_t elig = 0, multi = 0;
  for (int r = 0; r < rounds; ++r) {
    const int64_t base = ((int64_t)blockIdx.x * rounds + r) * kChunkRound;
    if (base >= n) break;
    uint32_t f[kChunkPer], len[kChunkPer];
    int32_t v[kChunkPer], root[kChunkPer];
#pragma unroll
    for (int k = 0; k < kChunkPer; ++k) {
      const int64_t x = base + k * kChunkBlock + threadIdx.x;
      v[k] = (int32_t)x;
      f[k] = x < n ? flags[x] : 1u;
      root[k] = v[k];
      len[k] = 0;
      if (x < n && (f[k] & 6u)) {
        root[k] = kFind ? ld_relaxed(label + x) : label[x];
        if constexpr (kBases) len[k] = ex.read_len[x];
      }
    }
    for (int i = threadIdx.x; i < kCountSlots; i += kChunkBlock) {
      s_key[i] = -1;
      s_cnt[i] = 0;
      if constexpr (kBases) s_w[i] = 0;
    }
    if constexpr (kFind) {
      // both reads' climbs side by side; a long one leaves where it has got to
      bool more = true;
      int32_t first[kChunkPer];
#pragma unroll
      for (int k = 0; k < kChunkPer; ++k) first[k] = root[k];
      for (int hop = 0; more; ++hop) {
        int32_t p[kChunkPer];
#pragma unroll
        for (int k = 0; k < kChunkPer; ++k) p[k] = (f[k] & 6u) ? ld_relaxed(label + root[k]) : root[k];
        more = false;
#pragma unroll
        for (int k = 0; k < kChunkPer; ++k) {
          if (p[k] != root[k]) {
            more = true;
            if (hop >= kClimbQuiet) st_relaxed(label + v[k], p[k]);
          }
          root[k] = p[k];
        }
      }
#pragma unroll
      for (int k = 0; k < kChunkPer; ++k)
        if (root[k] != first[k]) st_relaxed(label + v[k], root[k]);
    }
    int h[kChunkPer];
    uint32_t at[kChunkPer];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kChunkPer; ++k) {
      h[k] = -1;
      if (root[k] == v[k] && eligible(f[k], 2, min_reads)) {
        ++elig;
        multi += (f[k] & 6u) ? 1u : 0u;
      }
      if (!(f[k] & 6u)) continue;
      uint32_t i = ((uint32_t)root[k] * 2654435761u) >> 16 & (kCountSlots - 1);
      while (true) {  // ends: the table is at most half full
        const int32_t old = atomicCAS(s_key + i, -1, root[k]);
        if (old == -1 || old == root[k]) break;
        i = (i + 1) & (kCountSlots - 1);
      }
      h[k] = (int)i;
      at[k] = atomicAdd(s_cnt + i, (f[k] & 6u) == 6u ? 4u : 5u);
      if constexpr (kBases) atomicAdd(s_w + i, (unsigned long long)len[k]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCountSlots; i += kChunkBlock) {
      const int32_t x = s_key[i];
      if (x < 0) continue;
      if constexpr (kBases) atomicAdd((unsigned long long *)ex.root_w + x, s_w[i]);
      s_cnt[i] = atomicAdd((uint32_t *)cnt + x, s_cnt[i]) >> 2;
    }
    __syncthreads();
    if constexpr (kFind) {
#pragma unroll
      for (int k = 0; k < kChunkPer; ++k)
        if (h[k] >= 0) ex.slot[v[k]] = (int32_t)(s_cnt[h[k]] + (at[k] >> 2));
      __syncthreads();
    }
  }
  elig = chunk_sum(elig, sh);
  __syncthreads();
  multi = chunk_sum(multi, sh);
  if (chunks && threadIdx.x == 0) chunks[blockIdx.x] = make_uint2(elig, multi);
  if constexpr (kFind) {
    // the last workgroup adds up the mask pass's counts
    static_assert(kMaskMaxBlocks <= kChunkBlock, "a part per thread");
    if (blockIdx.x != gridDim.x - 1) return;
    const unsigned long long p =
        (int)threadIdx.x < ex.mask_parts ? ex.fx->mask_part[threadIdx.x] : 0ull;
    __syncthreads();
    const uint32_t nb = chunk_sum((uint32_t)p, sh);
    __syncthreads();
    const uint32_t ml = chunk_sum((uint32_t)(p >> 32), sh);
    if (threadIdx.x == 0) {
      ex.d_counts[0] = (int32_t)nb;
      ex.d_counts[1] = (int32_t)ml;
    }
  }
}

__global__ __launch_bounds__(kChunkBlock) void k_part_chunks(int32_t n, int rounds,
                                                             const uint8_t *__restrict__ flags,
                                                             const int32_t *__restrict__ cnt,
                                                             int32_t min_reads,
                                                             uint2 *__restrict__ chunks) {
  __shared__ uint32_t sh[kChunkBlock / kWave];
  uint32_t elig = 0;
  const int64_t base = (int64_t)blockIdx.x * rounds * kChunkRound;
  for (int r = 0; r < rounds * kChunkPer; ++r) {
    const int64_t v = base + (int64_t)r * kChunkBlock + threadIdx.x;
    if (v >= n) break;
    const uint32_t c = (uint32_t)cnt[v];
    if (c > 0 && eligible(flags[v], c >> 2, min_reads)) ++elig;
  }
  elig = chunk_sum(elig, sh);
  if (threadIdx.x == 0) chunks[blockIdx.x] = make_uint2(elig, elig);
}

// Two consecutive reads per thread and round.  (A single-pass look-back scan
// in this place waited for its tickets, its predecessors and a release per
// workgroup: 29 us on the 1 Gbp graph, 7 us on a graph of one workgroup.)
// Member slots and list places come from cursors, a round's at a time.
__global__ __launch_bounds__(kChunkBlock) void k_part_compact(
    int32_t n, int rounds, const uint2 *__restrict__ chunks, const uint8_t *__restrict__ flags,
    int32_t *label_comp, int32_t min_reads, int32_t *__restrict__ comp_label,
    int32_t *__restrict__ comp_size, uint8_t *__restrict__ comp_kind,
    int32_t *__restrict__ d_n_comp, MemberOut mo) {
  __shared__ unsigned long long sh[kChunkBlock / kWave + 1];
  __shared__ uint32_t s_before, s_before2, s_slot, s_large, s_list;
  __shared__ uint32_t sh32[kChunkBlock / kWave], sh32b[kChunkBlock / kWave + 1];
  const int64_t base0 = (int64_t)blockIdx.x * rounds * kChunkRound;
  static_assert(kChunks <= kChunkBlock, "a chunk per thread");
  const uint2 ch = threadIdx.x < blockIdx.x ? chunks[threadIdx.x] : make_uint2(0, 0);
  uint32_t before = ch.x, before2 = ch.y;
  uint32_t c[kChunkPer], f[kChunkPer];
  auto load = [&](int64_t base) {
#pragma unroll
    for (int k = 0; k < kChunkPer; ++k) {
      const int64_t v = base + (int64_t)threadIdx.x * kChunkPer + k;
      c[k] = v < n ? (uint32_t)label_comp[v] : 0u;
      f[k] = v < n ? flags[v] : 1u;
    }
  };
  load(base0);
  before = chunk_sum(before, sh32);
  if (mo.keys) {
    __syncthreads();
    before2 = chunk_sum(before2, sh32);
  }
  if (threadIdx.x == 0) {
    s_before = before;
    s_before2 = before2;
    s_large = 0;
  }
  __syncthreads();
  before = s_before;
  before2 = s_before2;
  for (int r = 0; r < rounds; ++r) {
    const int64_t base = base0 + (int64_t)r * kChunkRound;
    if (base >= n) break;
    if (r > 0) load(base);
    // (components << 32) | their reads, each below 2^31
    unsigned long long x = 0;
    bool el[kChunkPer];
    uint32_t large[kChunkPer];
#pragma unroll
    for (int k = 0; k < kChunkPer; ++k) {
      large[k] = 0;
      el[k] = c[k] > 0 && eligible(f[k], c[k] >> 2, min_reads);
      x += el[k] ? 1ull << 32 | (c[k] >> 2) : 0ull;
      if (mo.start && el[k] && c[k] >> 2 > (uint32_t)kWalkSmallCap) large[k] = 1 + atomicAdd(&s_large, 1u);
    }
    unsigned long long tot;
    const unsigned long long ex = block_excl_scan<unsigned long long, kChunkBlock>(x, sh, &tot);
    if (mo.start) {
      // (the scan's barriers lie between the counts and these)
      if (threadIdx.x == 0 && (uint32_t)tot) s_slot = atomicAdd(&mo.fx->fill_cursor, (uint32_t)tot);
      if (threadIdx.x == kWave && s_large) s_list = atomicAdd(&mo.fx->n_listed, s_large);
      __syncthreads();
    }
    uint32_t at2 = before2;
    if (mo.keys) {
      uint32_t y = 0, tot2;
#pragma unroll
      for (int k = 0; k < kChunkPer; ++k) y += el[k] && c[k] >> 2 > 1u ? 1u : 0u;
      at2 += block_excl_scan<uint32_t, kChunkBlock>(y, sh32b, &tot2);
      before2 += tot2;
    }
    uint32_t at = before + (uint32_t)(ex >> 32);
    uint32_t slot = mo.start ? s_slot + (uint32_t)ex : 0u;
#pragma unroll
    for (int k = 0; k < kChunkPer; ++k) {
      const int64_t v = base + (int64_t)threadIdx.x * kChunkPer + k;
      if (v >= n) continue;
      if (el[k]) {
        const uint32_t q = c[k] >> 2;
        comp_label[at] = (int32_t)v;
        comp_size[at] = (int32_t)q;
        comp_kind[at] = q == 1 ? CG_KIND_SINGLE : ((c[k] & 3u) ? CG_KIND_PATH : CG_KIND_CYCLE);
        if (mo.start) mo.start[at] = (int32_t)slot;
        if (mo.comp_w) mo.comp_w[at] = (f[k] & 6u) ? mo.root_w[v] : (uint64_t)mo.read_len[v];
        if (large[k]) mo.list[s_list + large[k] - 1] = (int32_t)at;
        label_comp[v] = (int32_t)at;
        if (mo.keys) {
          const uint64_t key = (uint64_t)(0xFFFFFFFFu - q) << 32 | at;
          if (q > 1) mo.keys[at2++] = key;
          else mo.keys[(int64_t)n + (at - at2)] = key;
        }
        ++at;
        slot += q;
      } else {
        label_comp[v] = -1;
      }
    }
    before += (uint32_t)(tot >> 32);
    if (mo.start && rounds > 1) {  // the places are read before the next round's
      __syncthreads();
      if (threadIdx.x == 0) s_large = 0;
      __syncthreads();
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    *d_n_comp = (int32_t)before;
    if (mo.keys) mo.fx->n_multi = before2;
  }
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

// Workgroup 0 of the LPT.  In the whole path the others put every read of a
// component into its slot meanwhile (the partition leaves all but one compute
// unit idle; as a launch of its own after it this took 12 us of the 50 Mbp
// graph's and 33 us of the 1 Gbp graph's).
struct FillArgs {
  int32_t n;
  const uint8_t *flags;
  const int32_t *label, *label_comp, *mstart, *slot;
  int32_t *tmp;
};
__device__ __forceinline__ void fill_members(const FillArgs &fa) {
  const int64_t stride = (int64_t)(gridDim.x - 1) * kLptBlock;
  constexpr int U = 2;
  for (int64_t v0 = (int64_t)(blockIdx.x - 1) * kLptBlock + threadIdx.x; v0 < fa.n;
       v0 += U * stride) {
    int32_t lab[U], c[U], at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = v0 + u * stride;
      lab[u] = v < fa.n && (fa.flags[v] & 6u) ? fa.label[v] : -1;
      at[u] = lab[u] >= 0 ? fa.slot[v] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = lab[u] >= 0 ? fa.label_comp[lab[u]] : -1;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] >= 0) fa.tmp[fa.mstart[c[u]] + at[u]] = (int32_t)(v0 + u * stride);
  }
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
                                                        uint64_t *g_bins, int later,
                                                        const unsigned int *n_multi, int32_t n,
                                                        RankOut ro, FillArgs fa) {
  __shared__ alignas(16) uint64_t s_keys[kSortCapLds];
  __shared__ int32_t s_bin[kSortCapLds];
  __shared__ uint64_t s_binA[kBinCapLds], s_binB[kBinCapLds];
  __shared__ uint32_t s_cnt[kLptBlock / kWave * 256];
  uint32_t *big_cnt = reinterpret_cast<uint32_t *>(s_keys);  // s_keys is the LDS form's
  if (blockIdx.x > 0) {
    fill_members(fa);
    return;
  }
  const int nc = *d_n_comp;
  int32_t *rank = later ? nullptr : comp_rank;
  int32_t *bin_of = later ? comp_bin : g_bin;
  // (the compaction has split the keys: the others' lie from key n on)
  const int multi = n_multi ? (int)*n_multi : -1;
  if (nc <= kSortCapLds && P <= kBinCapLds && !later)
    lpt_body<kLptBlock, false>(nc, P, comp_size, weight, s_keys, s_bin, s_cnt, s_binA, s_binB,
                               comp_bin, comp_rank, comp_start, bin_load, nullptr, status, nullptr, nullptr,
                               ro);
  else
    lpt_body<kLptBlock, true>(nc, P, comp_size, weight, multi < 0 ? g_keys : g_keys + (n - multi),
                              bin_of, big_cnt,
                              P <= kBinCapLds ? s_binA : g_bins,
                              P <= kBinCapLds ? s_binB : g_bins + P, comp_bin, rank, comp_start,
                              bin_load, nullptr, status, nullptr, nullptr, ro, multi, g_keys);
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
                                                            int32_t *__restrict__ comp_start,
                                                            RankOut ro) {
  __shared__ unsigned long long pos[kBinCapLds];
  __shared__ unsigned long long wpos[kPlaceWaves][kBinCapLds];
  __shared__ unsigned long long sh[kPlaceWaves + 1];
  const int64_t nc = *d_n_comp, c0 = (int64_t)blockIdx.x * chunk;
  if (ro.bin_vptr && nc == 0 && blockIdx.x == 0) {
    for (int b = threadIdx.x; b <= P; b += kPlaceBlock) ro.bin_vptr[b] = 0;
    if (threadIdx.x == 0) ro.d_sizes[0] = ro.d_sizes[1] = ro.loc_row_ptr[0] = 0;
  }
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
    if (b < P) {
      pos[b] = carry + ex + before;
      if (ro.bin_vptr && blockIdx.x == 0) ro.bin_vptr[b] = (int32_t)(uint32_t)(carry + ex);
    }
    carry += tot;
  }
  if (ro.bin_vptr && blockIdx.x == 0 && threadIdx.x == 0)
    ro.bin_vptr[P] = ro.d_sizes[0] = (int32_t)(uint32_t)carry;
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
      if (ro.bin_vptr && q > 1 && ro.comp_kind[c] == CG_KIND_CYCLE) mark_cycle(ro.cyc, rank);
      // the bin's last lane leaves where the next round goes on
      if ((peers & ~below) == 1ull << l)
        my[b] = (unsigned long long)(uint32_t)(rank + 1) << 32 | (uint32_t)(start + q);
    }
    wave_lds_sync();
  }
}

// Whether the (bin, label) order is left to k_part_hist and k_part_place
static bool place_later(int32_t n, int32_t P, int32_t min_reads) {
  return min_reads <= 1 && n > kSortCapLds && P <= kBinCapLds;
}

// bases weights (if wanted), the LPT, and the order of many components; fa.n > 0:
// the weights are there, and the members' slots are filled meanwhile
static void launch_lpt(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const int32_t *label,
                       int32_t P, int32_t min_reads, int32_t weight, const cg_parts &out,
                       const RankOut &ro, const FillArgs &fa, hipStream_t st) {
  const int32_t n = g.n;
  const bool bases = weight == CG_WEIGHT_BASES;
  if (bases && n > 0 && fa.n == 0) {
    const dim3 grid((unsigned)((n + kPartBlock - 1) / kPartBlock));
    CG_LAUNCH(ctx, k_part_wzero, grid, dim3(kPartBlock), st, n, s.comp_w);
    CG_LAUNCH(ctx, k_part_weight, grid, dim3(kPartBlock), st, n, label, out.label_comp,
                       g.read_len, s.comp_w);
  }
  // one-read components are most of a graph's, so where they are wanted of
  // more reads than the LDS sort holds, the order is left to the passes below
  // (two launches, which the few components of other graphs do not repay)
  const bool place = place_later(n, P, min_reads);
  // the fill takes a compute unit per workgroup (the LPT's LDS), four reads a
  // thread where that leaves some
  const int64_t fill = ((int64_t)fa.n + 4 * kLptBlock - 1) / (4 * kLptBlock);
  CG_LAUNCH(ctx, k_part_lpt, dim3((unsigned)(1 + (fill < 255 ? fill : 255))), dim3(kLptBlock), st,
            P, out.d_n_comp, out.comp_size, bases ? (const uint64_t *)s.comp_w : nullptr,
            &ctx->fixed->status, out.comp_bin, out.comp_rank, out.comp_start, out.bin_load, s.keys,
            s.aux, s.bins, place ? 1 : 0, place && !bases ? &ctx->fixed->n_multi : nullptr, n,
            place ? RankOut{} : ro, fa);
  if (place) {
    const int32_t per = (n + kPlaceChunks - 1) / kPlaceChunks;
    const int32_t chunk = per > kPlaceChunk ? per : kPlaceChunk;
    const dim3 chunks((unsigned)((n + chunk - 1) / chunk));
    CG_LAUNCH(ctx, k_part_hist, chunks, dim3(kPlaceBlock), st, P, chunk, out.d_n_comp,
              out.comp_size, out.comp_bin, s.keys);
    CG_LAUNCH(ctx, k_part_place, chunks, dim3(kPlaceBlock), st, P, chunk, out.d_n_comp,
              out.comp_size, out.comp_bin, s.keys, out.comp_rank, out.comp_start, ro);
  }
}

// the eligible components (counts in label_comp, chunk sums unless the flags
// decide), with member slots and the large ones' list if wanted
static void launch_compact(cg_ctx *ctx, const cg_graph &g, uint2 *chunks, const uint8_t *flags,
                           int32_t min_reads, const cg_parts &out, const MemberOut &mo,
                           hipStream_t st) {
  const int32_t n = g.n;
  const int rounds = chunk_rounds(n);
  const dim3 grid((unsigned)chunk_count(n));
  if (min_reads > 2 && n > 0)
    CG_LAUNCH(ctx, k_part_chunks, grid, dim3(kChunkBlock), st, n, rounds, flags, out.label_comp,
              min_reads, chunks);
  CG_LAUNCH(ctx, k_part_compact, grid, dim3(kChunkBlock), st, n, rounds, chunks, flags,
            out.label_comp, min_reads, out.comp_label, out.comp_size, out.comp_kind, out.d_n_comp,
            mo);
}

int launch_partition(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const uint8_t *flags,
                     const int32_t *label, int32_t P, int32_t min_reads, int32_t weight,
                     const cg_parts &out, hipStream_t st) {
  const PhaseRange range("cg: GreedyPartitioning");
  const int32_t n = g.n;
  if (min_reads < 1) min_reads = 1;
  static_assert(sizeof(uint2) <= sizeof(uint64_t), "a chunk's counts fit a read's word");
  uint2 *chunks = reinterpret_cast<uint2 *>(s.piece_off);  // until the pieces
  // read counts sort themselves as far as they are one
  uint64_t *keys =
      place_later(n, P, min_reads) && weight == CG_WEIGHT_READS ? s.keys : nullptr;
  if (n > 0) {
    CG_LAUNCH(ctx, k_part_zero, dim3((unsigned)((n + kPartBlock - 1) / kPartBlock)),
              dim3(kPartBlock), st, n, flags, out.label_comp);
    CG_LAUNCH(ctx, (k_part_count<false, false>), dim3((unsigned)chunk_count(n)), dim3(kChunkBlock), st, n,
              chunk_rounds(n), flags, const_cast<int32_t *>(label), out.label_comp, min_reads,
              min_reads <= 2 ? chunks : nullptr, CountExtra{});
  }
  launch_compact(ctx, g, chunks, flags, min_reads, out,
                 MemberOut{nullptr, nullptr, ctx->fixed, keys, nullptr, nullptr, nullptr}, st);
  launch_lpt(ctx, g, s, label, P, min_reads, weight, out, RankOut{}, FillArgs{}, st);
  return hip_check(hipGetLastError(), "k_part");
}

int launch_path_partition(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const PathArgs &a,
                          hipStream_t st) {
  const int32_t n = g.n, min_reads = a.min_reads < 1 ? 1 : a.min_reads;
  uint2 *chunks = reinterpret_cast<uint2 *>(s.piece_off);  // until the pieces
  // read counts sort themselves as far as they are one
  uint64_t *keys =
      place_later(n, a.P, min_reads) && a.weight == CG_WEIGHT_READS ? s.keys : nullptr;
  int32_t *mstart = reinterpret_cast<int32_t *>(s.fill);
  const bool bases = a.weight == CG_WEIGHT_BASES;
  uint64_t *root_w = s.piece_src;  // until the pieces
  const MemberOut mo{mstart, s.memb, ctx->fixed, keys, bases ? s.comp_w : nullptr, root_w,
                     g.read_len};
  if (front_fits(n)) {
    const int rc = launch_front(ctx, g, s, a, mo, st);
    if (rc) return rc;
  } else {
    int mask_parts = 0;
    const int rc = launch_path_mask(ctx, g, s, a, &mask_parts, st);
    if (rc) return rc;
    // (the count finishes the labels, too)
    const PhaseRange range("cg: GreedyPartitioning");
    const CountExtra ex{s.lidx, ctx->fixed, mask_parts, a.d_counts, g.read_len, root_w};
    const dim3 grid((unsigned)chunk_count(n));
    uint2 *sums = min_reads <= 2 ? chunks : nullptr;
    if (bases)
      CG_LAUNCH(ctx, (k_part_count<true, true>), grid, dim3(kChunkBlock), st, n, chunk_rounds(n),
                a.flags, a.label, a.parts.label_comp, min_reads, sums, ex);
    else
      CG_LAUNCH(ctx, (k_part_count<true, false>), grid, dim3(kChunkBlock), st, n, chunk_rounds(n),
                a.flags, a.label, a.parts.label_comp, min_reads, sums, ex);
    launch_compact(ctx, g, chunks, a.flags, min_reads, a.parts, mo, st);
  }
  const PhaseRange range("cg: GreedyPartitioning");
  const RankOut ro{a.local.bin_vptr, a.local.d_sizes, a.local.loc_row_ptr, a.parts.comp_kind,
                   cyc_marks(s.estart, n)};
  const FillArgs fa{n, a.flags, a.label, a.parts.label_comp, mstart, s.lidx, s.tmp};
  launch_lpt(ctx, g, s, a.label, a.P, min_reads, a.weight, a.parts, ro, fa, st);
  return hip_check(hipGetLastError(), "k_part");
}

// The five steps together: eight launches (ten where every read is wanted of
// a large graph, four for a small graph) where the steps one by one take
// fifteen to eighteen.  The mask pass sets up the component forest and the
// counters, the count finishes the labels and gives out the member slots (all
// of it and the compaction one pass in LDS for a small graph, k_front.hip),
// the LPT's launch fills them, and one pass over the components induces and
// walks.
int launch_path(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const PathArgs &a,
                hipStream_t st) {
  int rc;
  if (g.n == 0) {
    rc = launch_mask(ctx, g, a.flags, a.d_counts, st);
    if (!rc) rc = launch_partition(ctx, g, s, a.flags, a.label, a.P, a.min_reads, a.weight, a.parts, st);
    if (!rc) rc = launch_induce(ctx, g, s, a.flags, a.label, a.parts, a.P, a.local, st);
  } else {
    rc = launch_path_partition(ctx, g, s, a, st);
    if (!rc) rc = launch_comp(ctx, g, s, a, reinterpret_cast<int32_t *>(s.fill), st);
    const int32_t max_contigs = g.n / (a.min_reads < 1 ? 1 : a.min_reads);
    if (!rc) {
      const PhaseRange range("cg: LocalAssembly");
      rc = launch_contigs(ctx, g, s, a.parts, a.local, a.P, max_contigs, a.out, st, a.status);
    }
    return rc;
  }
  if (!rc) rc = launch_assemble(ctx, g, s, a.parts, a.local, a.P, a.out, st);
  return rc;
}

}  // namespace cg
