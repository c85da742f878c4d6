// Device code shared by the single-graph kernels and the batched kernels:
// union-find, the sort + LPT body, the per-component walk and the packed
// base access.  Each part names the step of Algorithm 2 it serves.
#pragma once

#include <type_traits>

#include "cg_internal.h"

namespace cg {

// LDS written by the lanes of a wave is seen by all of its lanes after this:
// a wave's LDS accesses are carried out in order, so this only keeps the
// compiler from moving accesses across it
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the first position in the sorted a[0, q), in LDS or not, holding a value >= x
__device__ __forceinline__ int32_t lower_bound_i32(const int32_t *a, int q, int32_t x) {
  int lo = 0, hi = q;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (a[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// The same for N values at once, so that their loads overlap (q >= 1).
template <int N>
__device__ __forceinline__ void lds_lower_bounds(const int32_t *a, int q, const int32_t (&x)[N],
                                                 int (&p)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) p[k] = 0;
  for (int step = 1 << (31 - __clz(q)); step > 0; step >>= 1) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int t = p[k] + step;
      if (t <= q && a[t - 1] < x[k]) p[k] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// BranchRemoval: flags of a vertex whose row starts at b and has `deg`
// entries: bit0 branch (deg >= 3); bit1 / bit2 entry 0 / 1 kept (neither end
// is a branch vertex).
// ---------------------------------------------------------------------------
// u0, u1: the row's first two columns, where it has them and no more.
__device__ __forceinline__ uint32_t vertex_flags(const int32_t *__restrict__ row_ptr,
                                                 const int32_t *__restrict__ col, int32_t b,
                                                 int32_t deg, int32_t &u0, int32_t &u1) {
  u0 = u1 = 0;
  if (deg >= 3) return 1u;
  uint32_t f = 0;
  if (deg > 0) {
    u0 = col[b];
    if (row_ptr[u0 + 1] - row_ptr[u0] < 3) f |= 2;
    if (deg == 2) {
      u1 = col[b + 1];
      if (row_ptr[u1 + 1] - row_ptr[u1] < 3) f |= 4;
    }
  }
  return f;
}

// A read's parent before any union: the smaller of its kept neighbours if it
// is smaller than the read itself.  Every kept edge then joins its larger end
// to its smaller one but for the second edge of a read with two smaller
// neighbours (a third of a chain's reads in random order), and only these
// are left for the unions.
__device__ __forceinline__ int32_t first_parent(int32_t v, uint32_t f, int32_t u0, int32_t u1) {
  int32_t p = v;
  if ((f & 2) && u0 < p) p = u0;
  if ((f & 4) && u1 < p) p = u1;
  return p;
}

// Steps of a read's climb to its root, once the unions are done, before it
// starts to leave where it has got to as its label (its own only, always an
// ancestor), from which the climbs through it go on.  Ids in random order take
// fewer steps (stores from the fourth step on: 100,000 reads of one chain 21
// us instead of 18); where reads are numbered along the genome every parent is
// the read before, and the climbs double their strides so.
constexpr int kClimbQuiet = 16;
// Such a read is told by a neighbour at most this far below it (two reads of a
// graph in random order seldom are).
constexpr int kSortedNear = 64;

// a read's counter before the count: a read without kept entries is counted
__device__ __forceinline__ int32_t first_count(uint32_t f) { return (f & 6) ? 0 : 4; }

// Whether root v (a read that is its component's label) of q reads and flags f
// makes an eligible component.  Up to two reads the flags tell: a component
// of more than one read is one whose root has kept entries.
__device__ __forceinline__ bool eligible(uint32_t f, uint32_t q, int32_t min_reads) {
  if (f & 1) return false;
  return min_reads <= 1 || (min_reads == 2 ? (f & 6) != 0 : q >= (uint32_t)min_reads);
}

// What the compaction gives out besides the components.  start, if given: the
// first member slot of each, and the list of those above kWalkSmallCap reads,
// both in any order.
// keys, if given: the LPT's keys by read count, those of the components of more
// than one read from keys[0] on, the others' from keys[n] on.
// comp_w, if given: the bases weights, a lone read's length or its root's sum.
struct MemberOut {
  int32_t *start, *list;
  Fixed *fx;
  uint64_t *keys;
  uint64_t *comp_w;
  const uint64_t *root_w;
  const uint32_t *read_len;
};
// Cycles by component rank: a bitmap, the cycles of every kCycSuper ranks,
// and whether there is any (most graphs have none, and then nothing else is
// read).  Kept in the scratch's estart array.
constexpr int kCycSuper = 2048;
struct CycMarks {
  uint32_t *bits, *super, *any;
};
__host__ __device__ __forceinline__ CycMarks cyc_marks(int32_t *area, int32_t n) {
  uint32_t *b = reinterpret_cast<uint32_t *>(area);
  const int64_t w = ((int64_t)n + 31) / 32, sp = ((int64_t)n + kCycSuper - 1) / kCycSuper;
  return CycMarks{b, b + w, b + w + sp};
}
// words of the area they take
__host__ __device__ __forceinline__ int32_t cyc_words(int32_t n) {
  return n > 0 ? (int32_t)(((int64_t)n + 31) / 32 + ((int64_t)n + kCycSuper - 1) / kCycSuper + 1) : 0;
}
__device__ __forceinline__ void mark_cycle(const CycMarks &m, int32_t rank) {
  atomicOr(m.bits + (rank >> 5), 1u << (rank & 31));
  atomicAdd(m.super + rank / kCycSuper, 1u);
  *m.any = 1;
}

// What the induce step takes from the components in rank order, written by
// the partition step of the whole path: where the bins start, and the cycles.
struct RankOut {
  int32_t *bin_vptr;  // null: not wanted
  int32_t *d_sizes, *loc_row_ptr;
  const uint8_t *comp_kind;
  CycMarks cyc;
};

// ---------------------------------------------------------------------------
// ConnectedComponent: union-find with min-id roots
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t uf_find(int32_t *P, int32_t x) {
  while (true) {
    int32_t p = ld_relaxed(P + x);
    if (p == x) return x;
    int32_t gp = ld_relaxed(P + p);
    if (gp == p) return p;
    st_relaxed(P + x, gp);  // path halving: gp is an ancestor of x
    x = gp;
  }
}

__device__ __forceinline__ void uf_union(int32_t *P, int32_t a, int32_t b) {
  a = uf_find(P, a);
  b = uf_find(P, b);
  while (a != b) {
    if (a < b) {
      int32_t old = atomicCAS(P + b, b, a);  // link the larger root under the smaller
      if (old == b) return;
      b = old;
    } else {
      int32_t old = atomicCAS(P + a, a, b);
      if (old == a) return;
      a = old;
    }
  }
}

// Tagged forest: each entry holds (tag << 32) | parent, and an entry whose
// tag is not the current run's stands for "no parent".  Bumping the tag
// between runs therefore resets the whole forest without touching it, so
// the hooks can run in the same pass that finds the kept entries.  Parents
// are always smaller than their children, so every root is its tree's
// minimum id.
__device__ __forceinline__ uint64_t ld_relaxed64(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed64(uint64_t *p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t tf_entry(uint32_t tag, int32_t parent) {
  return ((uint64_t)tag << 32) | (uint32_t)parent;
}
__device__ __forceinline__ int32_t tf_parent(const uint64_t *F, uint32_t tag, int32_t x) {
  const uint64_t e = ld_relaxed64(F + x);
  return (uint32_t)(e >> 32) == tag ? (int32_t)(uint32_t)e : x;
}

__device__ __forceinline__ int32_t tf_find(uint64_t *F, uint32_t tag, int32_t x) {
  while (true) {
    const int32_t p = tf_parent(F, tag, x);
    if (p == x) return x;
    const int32_t gp = tf_parent(F, tag, p);
    if (gp == p) return p;
    st_relaxed64(F + x, tf_entry(tag, gp));  // path halving
    x = gp;
  }
}

// ---------------------------------------------------------------------------
// GreedyPartitioning: sort + LPT on one workgroup
// ---------------------------------------------------------------------------
constexpr int kLptBlock = 1024;
constexpr int kSortCapLds = 8192;  // components sorted in LDS
constexpr int kBinCapLds = 2048;   // bins kept in LDS

__device__ __forceinline__ int next_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Exclusive prefix minimum over the lanes of the wave (lane 0 gets
// 0xFFFFFFFF): row shifts 1, 2, 4, 8 within rows of 16 lanes, then the row
// broadcasts of lanes 15 and 31 (lanes without a source take the identity).
// Every lane of the wave must be active.
__device__ __forceinline__ uint32_t wave_excl_min_u32(uint32_t x) {
  const int id = -1;  // 0xFFFFFFFF
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x111, 0xF, 0xF, false));  // row_shr:1
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x112, 0xF, 0xF, false));  // row_shr:2
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x114, 0xF, 0xF, false));  // row_shr:4
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x118, 0xF, 0xF, false));  // row_shr:8
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x142, 0xA, 0xF, false));  // row_bcast:15
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x138, 0xF, 0xF, false);       // wave_shr:1
}

// The largest x of the wave, in every lane.  Every lane must be active.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  x = max(x, wave_dpp<0x111, 0xF>(x));
  x = max(x, wave_dpp<0x112, 0xF>(x));
  x = max(x, wave_dpp<0x114, 0xF>(x));
  x = max(x, wave_dpp<0x118, 0xF>(x));
  x = max(x, wave_dpp<0x142, 0xA>(x));
  x = max(x, wave_dpp<0x143, 0xC>(x));
  return wave_lane(x, kWave - 1);
}

// x of lane l ^ J: quad permutes for J = 1, 2, row shifts by 4 for J = 4, a
// rotation of each 16-lane row by 8 for J = 8, a swap of rows for J = 16 and of
// halves for J = 32.  Every lane of the wave must be active.
template <int J>
__device__ __forceinline__ uint32_t wave_xor_u32(uint32_t x) {
  const int v = (int)x;
  if constexpr (J == 1) {
    return (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  } else if constexpr (J == 2) {
    return (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  } else if constexpr (J == 4) {
    const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0xF, false);  // row_shl:4
    const uint32_t dn = (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    return (lane_id() & 4) ? dn : up;
  } else if constexpr (J == 8) {
    return (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false);  // row_ror:8
  } else if constexpr (J == 16) {
    // odd rows of 16 lanes of one copy with the even ones of the other
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return (lane_id() & 16) ? (uint32_t)r[0] : (uint32_t)r[1];
  } else {
    static_assert(J == 32, "partner distance");
    // the swap of one copy's upper with the other's lower half
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (lane_id() & 32) ? (uint32_t)r[0] : (uint32_t)r[1];
  }
}

// Bitonic sort of one value per lane across the wave, ascending in lane
// order: stage (K, J) for K = 2..64, J = K/2..1; of the first LANES lanes
// where the others hold the largest value.  All lanes active.
template <int LANES = kWave, int K = 2, int J = 1>
__device__ __forceinline__ uint32_t wave_sort_u32(uint32_t x, int l) {
  const uint32_t p = wave_xor_u32<J>(x);
  const bool keep_min = ((l & J) == 0) == ((l & K) == 0);
  x = keep_min ? min(x, p) : max(x, p);
  if constexpr (J > 1) return wave_sort_u32<LANES, K, J / 2>(x, l);
  else if constexpr (K < LANES) return wave_sort_u32<LANES, 2 * K, K>(x, l);
  else return x;
}

// One compare-exchange of a bitonic stage (k, J), J < 64, in registers: x is
// element i of the array, held by lane i % 64, and its partner i ^ J is held
// by lane (i % 64) ^ J of the same wave.  Every lane of the wave takes part.
template <int J, typename K>
__device__ __forceinline__ K bitonic_lane_step(K x, int i, int k) {
  K p;
  if constexpr (sizeof(K) == 8)
    p = ((K)wave_xor_u32<J>((uint32_t)(x >> 32)) << 32) | wave_xor_u32<J>((uint32_t)x);
  else
    p = (K)wave_xor_u32<J>((uint32_t)x);
  const bool keep_min = ((i & J) == 0) == ((i & k) == 0);
  const K mn = x < p ? x : p, mx = x < p ? p : x;
  return keep_min ? mn : mx;
}

// Stages (k, j) for j = min(k/2, 32) down to 1 on two independent elements
// (k wave-uniform, so each test is a scalar branch)
template <typename K>
__device__ __forceinline__ void bitonic_lane_merge(K &x0, K &x1, int i0, int i1, int k) {
  if (k >= 64) {
    x0 = bitonic_lane_step<32>(x0, i0, k);
    x1 = bitonic_lane_step<32>(x1, i1, k);
  }
  if (k >= 32) {
    x0 = bitonic_lane_step<16>(x0, i0, k);
    x1 = bitonic_lane_step<16>(x1, i1, k);
  }
  if (k >= 16) {
    x0 = bitonic_lane_step<8>(x0, i0, k);
    x1 = bitonic_lane_step<8>(x1, i1, k);
  }
  if (k >= 8) {
    x0 = bitonic_lane_step<4>(x0, i0, k);
    x1 = bitonic_lane_step<4>(x1, i1, k);
  }
  if (k >= 4) {
    x0 = bitonic_lane_step<2>(x0, i0, k);
    x1 = bitonic_lane_step<2>(x1, i1, k);
  }
  x0 = bitonic_lane_step<1>(x0, i0, k);
  x1 = bitonic_lane_step<1>(x1, i1, k);
}

// Stages (k, j) of every k in [k0, k1] with j < 64, in registers, two
// 64-element segments per wave at a time (independent chains, so their lane
// shuffles overlap); no barrier: a wave only touches its own segments.
// Elements past N2 (N2 < 64, or a missing second segment) are held as the
// largest key and never meet a real one.
template <typename K>
__device__ __forceinline__ void bitonic_segments(K *a, int N2, int k0, int k1) {
  const int nw = (int)(blockDim.x / kWave);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int l = lane_id();
  const int nseg = (N2 + kWave - 1) / kWave;
  for (int sgm = w; sgm < nseg; sgm += 2 * nw) {
    const int i0 = sgm * kWave + l, i1 = (sgm + nw) * kWave + l;
    K x0 = i0 < N2 ? a[i0] : ~K(0);
    K x1 = i1 < N2 ? a[i1] : ~K(0);
    for (int k = k0; k <= k1; k <<= 1) bitonic_lane_merge(x0, x1, i0, i1, k);
    if (i0 < N2) a[i0] = x0;
    if (i1 < N2) a[i1] = x1;
  }
}

// Sort a[0, N2) ascending (N2 a power of two) with every thread of the
// workgroup.  Only the stages whose pairs lie 64 or more apart go through
// memory, two per pass and barrier; the stages inside 64-element segments
// run in registers (for N2 = 512: 4 passes through memory, 45 stages).
// kLdsOnly: the barriers order LDS only, so the caller's global loads stay
// in flight through the sort.
template <typename K, bool kLdsOnly = false>
__device__ __forceinline__ void bitonic_sort(K *a, int N2) {
  auto bar = [] {
    if constexpr (kLdsOnly) lds_barrier();
    else __syncthreads();
  };
  bitonic_segments(a, N2, 2, N2 < kWave ? N2 : kWave);
  bar();
  for (int k = 2 * kWave; k <= N2; k <<= 1) {
    int j = k >> 1;
    // two stages (j, j/2) per barrier: each thread takes the four elements
    // i, i + j/2, i + j, i + 3j/2 (bits j and j/2 of i clear), all sorted in
    // the same direction since they differ only below k
    for (; j >= 2 * kWave; j >>= 2) {
      const int h = j >> 1;
      for (int t = threadIdx.x; t < N2 / 4; t += blockDim.x) {
        const int i = ((t & ~(h - 1)) << 2) | (t & (h - 1));
        const bool up = (i & k) == 0;
        K x0 = a[i], x1 = a[i + h], x2 = a[i + j], x3 = a[i + j + h];
        if ((x0 > x2) == up) { const K tmp = x0; x0 = x2; x2 = tmp; }
        if ((x1 > x3) == up) { const K tmp = x1; x1 = x3; x3 = tmp; }
        if ((x0 > x1) == up) { const K tmp = x0; x0 = x1; x1 = tmp; }
        if ((x2 > x3) == up) { const K tmp = x2; x2 = x3; x3 = tmp; }
        a[i] = x0;
        a[i + h] = x1;
        a[i + j] = x2;
        a[i + j + h] = x3;
      }
      bar();
    }
    if (j >= kWave) {  // one stage left above the register stages
      for (int t = threadIdx.x; t < N2 / 2; t += blockDim.x) {
        const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));  // pair (i, i + j)
        const K x = a[i], y = a[i + j];
        if ((x > y) == ((i & k) == 0)) {
          a[i] = y;
          a[i + j] = x;
        }
      }
      bar();
    }
    bitonic_segments(a, N2, k, k);
    bar();
  }
}

// Sort a[0, n) (distinct keys, at most one per thread; 16-byte aligned, filled
// up with the largest value to a multiple of four) by counting the smaller
// keys of each: every thread reads every key, 16 bytes at one address for a
// whole wave, and no step waits for another's result.  (A bitonic sort is a
// chain of 36 stages for 190 keys.  Little code, too: what a launch runs once
// it fetches from memory first.)
template <typename K>
__device__ __forceinline__ void rank_sort(K *a, int n) {
  constexpr int V = 16 / sizeof(K);
  struct alignas(16) Quad {
    K k[V];
  };
  const int i = (int)threadIdx.x;
  const K x = i < n ? a[i] : K(0);
  int r = 0;
  if (__builtin_amdgcn_readfirstlane(i) < n) {
#pragma unroll 2
    for (int c = 0; c < n; c += V) {
      const Quad y = *reinterpret_cast<const Quad *>(a + c);
#pragma unroll
      for (int k = 0; k < V; ++k) r += y.k[k] < x ? 1 : 0;
    }
  }
  __syncthreads();
  if (i < n) a[r] = x;
  __syncthreads();
}

// Stable sort of a[0, n) by bits 16 and up of its 32-bit keys, whose low 16
// bits are each key's index (the input is in index order), so the result is
// the order of the whole keys.  LSD radix sort over `passes` 8-bit digits
// from bit 16.  Each wave takes a contiguous run of keys, 64 per round in
// order: the lanes holding the same digit are found by eight ballots, and a
// key's rank is the wave's running count of its digit (in LDS) plus the
// lanes below it with the same digit.  One block scan over the counts in
// (digit, wave) order gives every digit's start for every wave.  tmp holds
// n keys, cnt 256 counters per wave (LDS), sh the block scan's words.
// n <= kRadixRounds * BLOCK.  Returns the array holding the result (a after
// an even number of passes, else tmp).
constexpr int kRadixRounds = 8;
template <int BLOCK>
__device__ __forceinline__ uint32_t *radix_sort_hi16(uint32_t *a, uint32_t *tmp, int n, int passes,
                                                     uint32_t *cnt, uint32_t *sh) {
  constexpr int NW = BLOCK / kWave;
  constexpr int E = 256 * NW / BLOCK;  // (digit, wave) counters per thread in the scan
  static_assert(E * BLOCK == 256 * NW, "whole counters per thread");
  const int w = threadIdx.x / kWave, l = lane_id();
  const int per_w = ((n + NW - 1) / NW + kWave - 1) & ~(kWave - 1);
  const int rounds = per_w / kWave;  // uniform, at most kRadixRounds
  const uint64_t below = (1ull << l) - 1ull;
  uint32_t *my = cnt + w * 256;
  uint32_t *src = a, *dst = tmp;
  for (int p = 0; p < passes; ++p) {
    const int s = 16 + 8 * p;
    for (int d = l; d < 256; d += kWave) my[d] = 0;
    uint32_t x[kRadixRounds];
    int pos[kRadixRounds];
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
      x[r] = 0;
      pos[r] = 0;
      if (r >= rounds) continue;
      const int i = w * per_w + r * kWave + l;
      const bool v = i < n;
      x[r] = v ? src[i] : 0u;
      const uint32_t d = (x[r] >> s) & 255u;
      uint64_t peers = __ballot(v);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = __ballot(v && bit);
        peers &= bit ? m : ~m;
      }
      const uint32_t c = my[d];  // the digit's count before this round
      pos[r] = (int)c + __popcll(peers & below);
      // the lowest lane holding the digit adds the round's keys of it
      if (v && (peers & below) == 0) my[d] = c + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // every (digit, wave) count to its start: exclusive scan in digit-major
    // order
    uint32_t c[E], sum = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = (int)threadIdx.x * E + k;
      c[k] = cnt[(e % NW) * 256 + e / NW];
      sum += c[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan<uint32_t, BLOCK>(sum, sh, &tot);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = (int)threadIdx.x * E + k;
      cnt[(e % NW) * 256 + e / NW] = ex;
      ex += c[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
      if (r >= rounds) continue;
      const int i = w * per_w + r * kWave + l;
      if (i < n) dst[my[(x[r] >> s) & 255u] + pos[r]] = x[r];
    }
    __syncthreads();
    uint32_t *t = src;
    src = dst;
    dst = t;
  }
  return src;
}

// The same sort for more keys than registers and LDS hold: n 64-bit keys
// already in the order of their low words, sorted by the bytes of their high
// words.  Each wave reads its run twice a pass, for the counts and for the
// places; a round of 64 keys that all hold one digit (most of a graph's
// components are one read long) needs no ballots.  For 110,000 keys of one
// byte a pass takes about 20 us of one workgroup where the bitonic sort,
// which this replaces, took 3 ms.
template <int BLOCK>
__device__ __forceinline__ uint64_t *radix_sort_hi32(uint64_t *a, uint64_t *tmp, int n, int passes,
                                                     uint32_t *cnt, uint32_t *sh) {
  constexpr int NW = BLOCK / kWave;
  constexpr int E = 256 * NW / BLOCK;
  constexpr int U = 8;  // rounds whose loads are issued together
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), l = lane_id();
  const int per_w = ((n + NW - 1) / NW + kWave - 1) & ~(kWave - 1);
  const int64_t i0 = (int64_t)w * per_w;
  const int64_t i1 = i0 + per_w < n ? i0 + per_w : n;
  const uint64_t below = (1ull << l) - 1ull;
  uint32_t *my = cnt + w * 256;
  uint64_t *src = a, *dst = tmp;
  for (int p = 0; p < passes; ++p) {
    const int s = 32 + 8 * p;
    for (int d = l; d < 256; d += kWave) my[d] = 0;
    wave_lds_sync();
    for (int64_t i = i0; i < i1; i += U * kWave) {
      uint32_t d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = i + u * kWave + l;
        d[u] = k < i1 ? (uint32_t)(src[k] >> s) & 255u : 256u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint64_t live = __ballot(d[u] < 256u);
        const uint32_t d0 = __builtin_amdgcn_readfirstlane((int)d[u]);
        if (__ballot(d[u] == d0) == live) {
          if (l == 0 && live) my[d0] += (uint32_t)__popcll(live);
        } else if (d[u] < 256u) {
          atomicAdd(my + d[u], 1u);
        }
        wave_lds_sync();
      }
    }
    __syncthreads();
    uint32_t c[E], sum = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = (int)threadIdx.x * E + k;
      c[k] = cnt[(e % NW) * 256 + e / NW];
      sum += c[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan<uint32_t, BLOCK>(sum, sh, &tot);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = (int)threadIdx.x * E + k;
      cnt[(e % NW) * 256 + e / NW] = ex;
      ex += c[k];
    }
    __syncthreads();
    for (int64_t i = i0; i < i1; i += U * kWave) {
      uint64_t x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = i + u * kWave + l;
        x[u] = k < i1 ? src[k] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool v = i + u * kWave + l < i1;
        const uint64_t live = __ballot(v);
        const uint32_t d = (uint32_t)(x[u] >> s) & 255u;
        const uint32_t d0 = __builtin_amdgcn_readfirstlane((int)d);
        uint64_t peers = live;
        if (__ballot(v && d == d0) != live) {
#pragma unroll
          for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(v && bit);
            peers &= bit ? m : ~m;
          }
        }
        const uint32_t at = my[d];
        wave_lds_sync();
        if (v) {
          dst[at + (uint32_t)__popcll(peers & below)] = x[u];
          if ((peers & below) == 0) my[d] = at + (uint32_t)__popcll(peers);
        }
        wave_lds_sync();
      }
    }
    __syncthreads();
    uint64_t *t = src;
    src = dst;
    dst = t;
  }
  return src;
}

// bytes of x that are not all zero from the top
__device__ __forceinline__ int value_bytes(uint32_t x) { return (39 - __clz(x)) >> 3; }

// number of elements of the sorted array a[0..len) that are < x
__device__ __forceinline__ int lower_bound_u64(const uint64_t *a, int len, uint64_t x) {
  int lo = 0, hi = len;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// x of lane l + 1 in lane l, by a DPP wave shift (wave_shl:1), and the largest
// value in lane 63, which has no source
__device__ __forceinline__ uint64_t wave_next_u64(uint64_t x) {
  const int lo = (int)(uint32_t)x, hi = (int)(uint32_t)(x >> 32);
  const uint32_t nlo = (uint32_t)__builtin_amdgcn_update_dpp(-1, lo, 0x130, 0xF, 0xF, false);
  const uint32_t nhi = (uint32_t)__builtin_amdgcn_update_dpp(-1, hi, 0x130, 0xF, 0xF, false);
  return ((uint64_t)nhi << 32) | nlo;
}

// x of lane l - 1 in lane l, by a DPP wave shift (wave_shr:1); lane 0 keeps
// its own x
__device__ __forceinline__ uint32_t wave_prev_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x138, 0xF, 0xF, false);
}
// x of lane l + 1 in lane l (wave_shl:1); lane 63 keeps its own x
__device__ __forceinline__ uint32_t wave_next_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x130, 0xF, 0xF, false);
}

// weight of the t-th item in LPT order, from the sorted keys (32-bit keys
// (2^16-1 - w) << 16 | index, or 64-bit (2^32-1 - w) << 32 | index)
__device__ __forceinline__ uint32_t lpt_item_weight(const uint32_t *srt, const uint64_t *keys,
                                                    bool k32, int t) {
  return 0xFFFFFFFFu - (k32 ? 0xFFFF0000u | (srt[t] >> 16) : (uint32_t)(keys[t] >> 32));
}

// Bin keys are (load << 16) | bin: ascending key order is ascending
// (load, bin), i.e. the least loaded bin with the lowest index first.
constexpr int kBinBits = 16;
constexpr int kLptRoundMin = 4;   // equal items taken as one round from this many
constexpr int kLptPrefixMin = 5;  // prefix rounds (any weights) from this many items
// Up to this many bins item by item without a round's tests, which cost as
// much as several items and place few.  7,000 one-read components, 16 bins: 290
// us either way, 24 bins: 288 us item by item, 215 in rounds; weights of many
// values, 16 bins: 338 and 505 us, 24 bins: 340 and 374; one to three bins,
// where no round comes about: 281 and 1,620.
constexpr int kLptStepBins = 16;
constexpr int kLptSteps = 8;  // items a turn there, a divisor of the wave's lanes
constexpr int kLptWideSteps = 4;  // and with wide keys (2, 4, 8 a turn: 730, 691, 703 us)
constexpr int kLptBlockBins = 256;  // rounds over the whole list from this many bins
constexpr int kLptBlockMin = 96;    // ... where they place this many items
constexpr int kLptBulkMin = 256;  // whole rounds of equal items taken at once from this many

// One past the last item of item a's weight wt, by the whole wave: 64 probes
// a step.  a holds wt; the items' weights do not increase.
__device__ __forceinline__ int lpt_run_end(const uint32_t *srt, const uint64_t *keys, bool k32,
                                           int a, int nc, uint32_t wt) {
  int lo = a, hi = nc;  // lo holds wt, hi does not (or is the end)
  while (hi - lo > 1) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int64_t i = (int64_t)lo + (int64_t)(lane_id() + 1) * step;
    const int k = __popcll(__ballot(i < hi && lpt_item_weight(srt, keys, k32, (int)i) == wt));
    lo += k * step;
    hi = hi < lo + step ? hi : lo + step;
  }
  return hi;
}

// The values of lanes 0..c-1 and those of lanes c..63, each sorted across its
// lanes, merged: the first run turned round makes both a bitonic run, which
// the six stages of a bitonic merge sort (a rank search over the lanes took
// seven lane shuffles one after another, about twice the time).
__device__ __forceinline__ uint32_t lpt_merge_lanes(uint32_t x, int l, int c) {
  x = (uint32_t)__shfl((int)x, l < c ? c - 1 - l : l);
  x = bitonic_lane_step<32>(x, l, kWave);
  x = bitonic_lane_step<16>(x, l, kWave);
  x = bitonic_lane_step<8>(x, l, kWave);
  x = bitonic_lane_step<4>(x, l, kWave);
  x = bitonic_lane_step<2>(x, l, kWave);
  return bitonic_lane_step<1>(x, l, kWave);
}

// With comp_kind and comp_estart given, it also writes each component's
// first local CSR entry (2(q-1) entries for a path, 2q for a cycle, none for
// a single read, in (bin, label) order) and returns their total.  bin_reads,
// if given (global memory, read back with atomic loads), gets the reads of
// each bin.  kBig: keys and bin_of are global memory (2 nc keys), else LDS
// (nc up to 8 BLOCK).
// s_cnt: LDS for the radix sorts, 256 words per wave.
// comp_rank null: the (bin, label) order is left to a later pass, and bin_of
// is comp_bin itself.  multi >= 0 (kBig, weights are read counts): the
// compaction has written the keys of the multi components of more than one
// read from `unsorted` on and those of the others, which come last in LPT
// order, from keys + multi on.
template <int BLOCK, bool kBig>
__device__ __forceinline__ int lpt_body(int nc, int P, const int32_t *__restrict__ comp_size,
                                        const uint64_t *__restrict__ weight,
                                        uint64_t *keys, int32_t *bin_of, uint32_t *s_cnt,
                                        uint64_t *binA,
                                        uint64_t *binB, int32_t *comp_bin,
                                        int32_t *__restrict__ comp_rank,
                                        int32_t *__restrict__ comp_start,
                                        uint64_t *__restrict__ bin_load,
                                        uint64_t *__restrict__ bin_reads,
                                        unsigned int *status,
                                        const uint8_t *__restrict__ comp_kind = nullptr,
                                        int32_t *__restrict__ comp_estart = nullptr,
                                        const RankOut &ro = RankOut{}, int multi = -1,
                                        uint64_t *unsorted = nullptr) {
  static_assert(BLOCK > 2 * kWave, "the pipelined windows' merge needs threads beyond two waves");
  __shared__ uint64_t win[2][kWave];  // a window's raised keys, alternating buffers
  __shared__ uint32_t s_min[BLOCK / kWave];  // rounds over the list: each wave's least raised key
  __shared__ int s_cp, s_unsorted;           // items placed; whether their keys need a sort
  __shared__ int32_t s_opbin[kWave];                 // rounds taken at once: their bins in order,
  __shared__ int32_t s_op_at, s_op_items, s_op_bins;  // first item, items (0: none), bins
  __shared__ int32_t sh_scan[BLOCK / kWave + 1];
  __shared__ int64_t sh_scan64[BLOCK / kWave + 1];
  __shared__ unsigned long long s_total;
  __shared__ unsigned int s_wmax;
  const int tid = threadIdx.x;
  const int N2 = next_pow2(nc > 4 ? nc : 4);
  if (tid == 0) {
    s_total = 0;
    s_wmax = 0;
  }
  __syncthreads();

  // 1. sort by (weight desc, label asc); components are indexed in label
  // order.  The weight is the read count, or the given weights (below 2^32).
  // Keys are ((2^32-1 - w) << 32) | i, or, when every weight and index fits
  // 16 bits, ((2^16-1 - w) << 16) | i in 32 bits (k32: the first half of
  // keys holds them); ~0 pads to N2.
  // Eight components per thread and round, their weights loaded together;
  // the LDS form's are all held in one round.
  constexpr int kPer = 8;
  uint32_t *keys32 = reinterpret_cast<uint32_t *>(keys);
  uint32_t wt8[kPer], wmax = 0;
  if constexpr (kBig) {
    if (multi >= 0) {
      if (multi < nc) wmax = 1;
      for (int i = tid; i < multi; i += BLOCK) {
        const uint32_t w = 0xFFFFFFFFu - (uint32_t)(unsorted[i] >> 32);
        wmax = w > wmax ? w : wmax;
      }
    }
  }
  for (int base = 0; base < nc && (!kBig || multi < 0); base += kPer * BLOCK) {
    if (weight) {
      uint64_t w[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int i = base + k * BLOCK + tid;
        w[k] = base + k * BLOCK < nc && i < nc ? weight[i] : 0;
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        if (w[k] > 0xFFFFFFFFull) {
          atomicOr(status, CG_STATUS_WEIGHT_RANGE);
          w[k] = 0xFFFFFFFFull;
        }
        wt8[k] = (uint32_t)w[k];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int i = base + k * BLOCK + tid;
        wt8[k] = base + k * BLOCK < nc && i < nc ? (uint32_t)comp_size[i] : 0u;
      }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) wmax = wt8[k] > wmax ? wt8[k] : wmax;
    if constexpr (kBig) {
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int i = base + k * BLOCK + tid;
        if (i < nc) keys[i] = ((uint64_t)(0xFFFFFFFFu - wt8[k]) << 32) | (uint32_t)i;
      }
    }
  }
  wmax = wave_max_u32(wmax);
  if (lane_id() == 0 && wmax) atomicMax(&s_wmax, wmax);
  for (int b = tid; b < P; b += blockDim.x) binA[b] = (uint64_t)b;  // load 0, sorted
  __syncthreads();
  const bool k32 = !kBig && nc <= 0xFFFF && s_wmax <= 0xFFFFu;
  if constexpr (!kBig) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (k * BLOCK >= N2) continue;
      const int i = k * BLOCK + tid;
      if (i >= N2) continue;
      if (k32) keys32[i] = i < nc ? ((0xFFFFu - wt8[k]) << 16) | (uint32_t)i : ~0u;
      else keys[i] = i < nc ? ((uint64_t)(0xFFFFFFFFu - wt8[k]) << 32) | (uint32_t)i : ~0ull;
    }
  }
  __syncthreads();
  // the keys in LPT order: in LDS up to 256 keys by ranks, above by radix passes over the weight's bytes (with fewer waves,
  // whose rounds run one after another, only where one pass does), else by a
  // bitonic sort; in global memory by radix passes
  auto radix = [&](int passes) {
    return nc <= kRadixRounds * BLOCK &&
           (BLOCK >= 1024 ? nc > 256 : passes == 1 && nc > 2 * BLOCK);
  };
  auto small_sort = [&](auto *k) {
    if (nc <= 256) rank_sort(k, nc);
    else bitonic_sort(k, N2);
  };
  const uint32_t *srt = keys32;
  if constexpr (kBig) {
    const int passes = value_bytes(s_wmax);
    if (multi < 0) {
      keys = radix_sort_hi32<BLOCK>(keys, keys + nc, nc, passes, s_cnt,
                                    reinterpret_cast<uint32_t *>(sh_scan));
    } else {
      // from and to `unsorted` in turn, so that the last pass ends in keys
      uint64_t *from = unsorted, *to = keys;
      if (passes % 2 == 0) {
        for (int i = tid; i < multi; i += BLOCK) keys[i] = unsorted[i];
        __syncthreads();
        from = keys;
        to = unsorted;
      }
      radix_sort_hi32<BLOCK>(from, to, multi, passes, s_cnt, reinterpret_cast<uint32_t *>(sh_scan));
    }
  } else if (k32 && radix(s_wmax < 256u ? 1 : 2))
    srt = radix_sort_hi16<BLOCK>(keys32, keys32 + N2, nc, s_wmax < 256u ? 1 : 2, s_cnt,
                                 reinterpret_cast<uint32_t *>(sh_scan));
  else if (k32)
    small_sort(keys32);
  else
    small_sort(keys);

  // 2. LPT.  The bins are kept sorted by (load, bin).  A window holds the W
  // least loaded bins in the lanes of wave 0 (sorted across lanes): each
  // component goes to lane 0's bin, whose new key is then re-inserted by
  // ballot + shift.  Within W steps of a window only its W bins can be the
  // minimum (step t picks a bin of initial rank <= t), so after W steps the
  // window is merged back into the sorted bin list.
  const int W = P < kWave ? P : kWave;
  const bool single_window = P <= kWave;
  // Narrow keys: a bin's key (load << kb) | bin with kb bits for the bin index
  // (2^kb >= P), less the least load of the window or batch, in 32 bits below
  // the padding value 0xFFFFFFFF: a step then needs about 12 vector
  // instructions instead of 17.  Same order, same choices.  The loads differ
  // by at most the largest weight wmax (a bin's last item found it the least
  // loaded), the least load rises by at most (64 / W + 1) wmax over a window's
  // or batch's 64 items, and a raised key adds one weight, which bounds the
  // differences.  The bin lists hold whole 64-bit keys.
  int kb = 0;
  while ((1 << kb) < P) ++kb;
  // Where one component outweighs the others by far that bound fails, but all
  // weights together may still be below 2^(32 - kb), and so is then every load
  // and every raised one (an item is added to a load that it is not part of):
  // 7,000 components and one of 18 Mbases, 64 bins: 310 us, 856 with wide keys.
  bool narrow =
      kb <= 16 && (unsigned long long)s_wmax * ((kWave + W - 1) / W + 4) + 1 < (1ull << (32 - kb));
  if (!narrow && kb <= 16) {
    unsigned long long sum = 0;
    for (int i = tid; i < nc; i += BLOCK) {
      const uint64_t w = weight ? weight[i] : (uint64_t)comp_size[i];
      sum += w > 0xFFFFFFFFull ? 0xFFFFFFFFull : w;
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) atomicAdd(&s_total, sum);
    __syncthreads();
    narrow = s_total + 1 < (1ull << (32 - kb));
  }
  const int bb = narrow ? kb : kBinBits;
  int i0 = 0;
  if (!single_window && nc > P) {
    // The first round in one pass.  Every weight is at least 1, so item t
    // (t < P) finds bins 0..t-1 loaded and bin t empty, the least loaded one
    // with the lowest index: items 0..P-1 go to bins 0..P-1.  The weights do
    // not increase along the items, so in the bin list sorted by (load, bin)
    // bin t comes after the bins of smaller load (those past its run of
    // equal weights) and in bin order within its run.
    for (int t = tid; t < P; t += blockDim.x) {
      const uint32_t wt = lpt_item_weight(srt, keys, k32, t);
      int lo = 0, hi = t;  // the run's first item: the first of weight <= wt
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (lpt_item_weight(srt, keys, k32, mid) > wt) lo = mid + 1;
        else hi = mid;
      }
      const int g0 = lo;
      lo = t;
      hi = P;  // one past the run's last item (within the first round)
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (lpt_item_weight(srt, keys, k32, mid) < wt) hi = mid;
        else lo = mid + 1;
      }
      const int pos = (P - lo) + (t - g0);
      binA[pos] = ((uint64_t)wt << bb) | (uint64_t)t;
      bin_of[k32 ? (srt[t] & 0xFFFFu) : (uint32_t)keys[t]] = t;
    }
    i0 = P;
  }
  __syncthreads();  // (outside the branch: inside it, the compiler kept a stack frame)
  // Above 64 bins the windows are pipelined (the workgroup has more than
  // 2 * 64 threads): after a window's steps, wave 0
  // forms the next window in its lanes as the W least of the raised keys and
  // the next W keys of the list (a bitonic merge in registers) and goes on,
  // while the other waves merge the raised keys back into the list.  One
  // barrier per window; the raised keys alternate between two buffers, so a
  // window's keys are written while the other waves still merge the last
  // ones, and the list alternates between binA and binB.
  // Above 64 bins, the items of the least weight (from s_last on, where there
  // are at least 4 P of them, as one-read components are) go in whole rounds
  // of the list as far as its order allows, by all threads.
  int s_last = nc;
  // items at .. at + items - 1 to bins 0 .. m - 1 of a list, over and over
  auto store_rounds = [&](int at, int items, int m, auto bin) {
    int r = m > 0 ? tid % m : 0;
    const int step = m > 0 ? BLOCK % m : 0;
#pragma unroll 8
    for (int k = tid; k < items; k += BLOCK) {
      bin_of[k32 ? (srt[at + k] & 0xFFFFu) : (uint32_t)keys[at + k]] = bin(r);
      r += step;
      r -= r >= m ? m : 0;
    }
  };
  if (kBig && !single_window && nc - i0 >= 8 * P) {
    const uint32_t wl = lpt_item_weight(srt, keys, k32, nc - 1);
    int lo = i0, hi = nc - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (lpt_item_weight(srt, keys, k32, mid) > wl) lo = mid + 1;
      else hi = mid;
    }
    if (nc - lo >= 4 * P && wl > 0) s_last = __builtin_amdgcn_readfirstlane(lo);
  }
  // (wave 0) Whole rounds of equal items from item `at` on, weight q, if there
  // are: the m lanes below lane 0's raised key take an item each in order, J
  // times over, for as long as all of them stay below lane m's key (to the
  // run's end when they are all bins).  The workgroup stores these items' bins.
  uint64_t load0 = 0;  // what narrow keys are relative to
  auto whole_rounds = [&](int at, uint32_t q, uint32_t iw, uint32_t &key) {
    const int l = tid;
    const uint32_t bmask = (1u << kb) - 1u;
    if (at + kLptBulkMin <= nc && q > 0 &&
        q == 0xFFFFFFFFu - (uint32_t)__builtin_amdgcn_readlane((int)iw, kWave - 1)) {
      const uint32_t qe = (uint32_t)__builtin_amdgcn_readfirstlane(
          (int)lpt_item_weight(srt, keys, k32, at + kLptBulkMin - 1));
      if (q == qe) {
        const uint32_t wk = q << kb;
        const int m =
            __popcll(__ballot(key < (uint32_t)__builtin_amdgcn_readlane((int)key, 0) + wk));
        uint32_t J = (uint32_t)((lpt_run_end(srt, keys, k32, at, nc, q) - at) / m);
        if (m < W) {
          const uint32_t jm = ((uint32_t)__builtin_amdgcn_readlane((int)key, m) - 1u -
                               (uint32_t)__builtin_amdgcn_readlane((int)key, m - 1)) / wk + 1u;
          J = J < jm ? J : jm;
        }
        const int items = (int)(J * (uint32_t)m);
        if (items >= kLptBulkMin) {
          if (l < m) s_opbin[l] = (int32_t)(key & bmask);
          if (l == 0) {
            s_op_at = at;
            s_op_items = items;
            s_op_bins = m;
          }
          if (m == W) load0 += (uint64_t)J * wk;  // every key: the order stays
          else key = lpt_merge_lanes(l < m ? key + J * wk : key, l, m);
          return true;
        }
      }
    }
    return false;
  };
  int cur = 0;
  while (i0 < nc) {
    if (kBig && i0 >= s_last) {
      const uint64_t wk = (uint64_t)lpt_item_weight(srt, keys, k32, i0) << bb;
      while (i0 < nc) {
        // the m bins below the least loaded one's raised key take an item
        // each, J times over: as long as they all stay below bin m's key
        const int m = lower_bound_u64(binA, P, binA[0] + wk);
        int64_t J = (nc - i0) / m;
        if (m < P) {
          const uint64_t jm = (binA[m] - 1 - binA[m - 1]) / wk + 1;
          J = (uint64_t)J < jm ? J : (int64_t)jm;
        }
        const int items = __builtin_amdgcn_readfirstlane((int)(J * m));
        if (items < kLptBulkMin) break;
        store_rounds(i0, items, m, [&](int r) { return (int32_t)(binA[r] & ((1ull << bb) - 1)); });
        // the raised bins and the others, two sorted runs, merged by rank
        for (int b = tid; b < P; b += blockDim.x) {
          const uint64_t x = binA[b] + (b < m ? (uint64_t)J * wk : 0ull);
          const int r = b < m ? lower_bound_u64(binA + m, P - m, x)
                              : lower_bound_u64(binA, m, x - (uint64_t)J * wk) - m;
          binB[b + r] = x;
        }
        __syncthreads();
        uint64_t *t = binA;
        binA = binB;
        binB = t;
        i0 += items;
      }
      if (i0 >= nc) break;
    }
    // Rounds over the whole list, by all threads: items i0, i0 + 1, ... go to
    // the list's bins 0, 1, ... for as long as each bin's key is below every
    // key the earlier items of the round raised (as in a wave's prefix round
    // below).  A list of hundreds of bins takes hundreds of items at once, where
    // a window of 64 takes 64: 4,478 components on 1,024 bins took 54 windows,
    // 66 us; the loop takes 36 us so.
    const bool blocks =
        BLOCK >= 1024 && narrow && P >= kLptBlockBins && P <= 2 * BLOCK;
    if (blocks) {
      constexpr int E = 2;  // bins per thread: 2 tid, 2 tid + 1
      uint32_t *srt_bins = reinterpret_cast<uint32_t *>(binB);
      const int Pn = next_pow2(P);  // below 2 P: fits binB
      const int w = tid / kWave;
      while (i0 < nc && i0 < (s_last < nc ? s_last : nc)) {
        const int n_it = nc - i0 < P ? nc - i0 : P;
        const uint64_t least = binA[0] >> bb << bb;
        uint32_t key[E], r[E];
        uint32_t mine = 0xFFFFFFFFu;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int j = tid * E + e;
          key[e] = j < P ? (uint32_t)(binA[j] - least) : 0xFFFFFFFFu;
          r[e] = j < n_it ? key[e] + (lpt_item_weight(srt, keys, k32, i0 + j) << kb) : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) mine = r[e] < mine ? r[e] : mine;
        // the least raised key before this thread's bins
        uint32_t lower = wave_excl_min_u32(mine);
        const uint32_t wmin = lower < mine ? lower : mine;
        if (tid == 0) s_cp = n_it;
        if (lane_id() == kWave - 1) s_min[w] = wmin;
        __syncthreads();
        for (int k = 0; k < w; ++k) lower = s_min[k] < lower ? s_min[k] : lower;
        int fail = n_it;
#pragma unroll
        for (int e = E - 1; e >= 0; --e) {
          const int j = tid * E + e;
          const uint32_t low = e == 0 ? lower : (r[0] < lower ? r[0] : lower);
          if (j < n_it && key[e] >= low) fail = j;
        }
        const uint64_t bad = __ballot(fail < n_it);
        if (bad && lane_id() == (int)__builtin_ctzll(bad)) atomicMin(&s_cp, fail);
        if (tid == 0) s_unsorted = 0;
        __syncthreads();
        const int cp = __builtin_amdgcn_readfirstlane(s_cp);
        if (cp < kLptBlockMin && cp < nc - i0) break;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int j = tid * E + e;
          if (j < cp) {
            const int i = i0 + j;
            bin_of[k32 ? (srt[i] & 0xFFFFu) : (uint32_t)keys[i]] =
                (int32_t)(key[e] & ((1u << kb) - 1u));
            key[e] = r[e];
          }
          if (j < Pn) srt_bins[j] = key[e];
        }
        __syncthreads();
        bool down = false;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int j = tid * E + e;
          down = down || (j > 0 && j < cp && srt_bins[j - 1] > key[e]);
        }
        if (down) s_unsorted = 1;
        __syncthreads();
        if (!s_unsorted) {
          // the raised bins and the others, two sorted runs, merged by rank
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int j = tid * E + e;
            if (j >= P) continue;
            int lo = j < cp ? cp : 0, hi = j < cp ? P : cp;
            while (lo < hi) {
              const int mid = (lo + hi) >> 1;
              if (srt_bins[mid] < key[e]) lo = mid + 1;
              else hi = mid;
            }
            binA[j < cp ? j + lo - cp : j - cp + lo] = least + key[e];
          }
        } else {
          bitonic_sort(srt_bins, Pn);
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int j = tid * E + e;
            if (j < P) binA[j] = least + srt_bins[j];
          }
        }
        __syncthreads();
        i0 += cp;
      }
      if (i0 >= nc) break;
    }
    // (every turn of this loop goes on to place at least one item here)
    // the items up to lim in windows (all of them in one window up to 64 bins)
    int lim = i0 < s_last ? s_last : (nc - i0 < P ? nc : i0 + P);
    if (blocks && lim > i0 + 2 * kWave) lim = i0 + 2 * kWave;
    uint32_t key32 = 0xFFFFFFFFu;  // wave 0: the window's keys (narrow or wide)
    uint64_t key64 = ~0ull;
    if (tid < kWave) {
      load0 = binA[0] >> bb << bb;
      if (narrow) key32 = tid < W ? (uint32_t)(binA[tid] - load0) : 0xFFFFFFFFu;
      else key64 = tid < W ? binA[tid] : ~0ull;
    }
    while (i0 < lim) {
      const int T = single_window ? nc - i0 : (lim - i0 < W ? lim - i0 : W);
      if (kBig && tid == 0) s_op_items = 0;
      if (tid < kWave && narrow && P <= kLptStepBins) {
        // Few bins (one window): no rounds but whole ones.  Item by item, lane
        // 0's bin takes it, and its raised key nk goes among the others, which
        // move down by one: lane l gets the middle one of its own key, lane
        // l + 1's and nk.  (Lanes from W on hold the largest value; lanes past
        // the items raise nothing, so that a step of theirs changes nothing.)
        const int l = tid;
        const uint32_t bmask = (1u << kb) - 1u;
        uint32_t key = key32;
        for (int base = 0; base < T; base += kWave) {
          const uint32_t sub = (uint32_t)__builtin_amdgcn_readlane((int)key, 0) & ~bmask;
          key -= l < W ? sub : 0u;
          load0 += sub;
          const int at = i0 + base, cnt = T - base < kWave ? T - base : kWave;
          uint64_t item = 0;
          if (l < cnt)
            item = k32 ? ((uint64_t)(0xFFFF0000u | (srt[at + l] >> 16)) << 32) | (srt[at + l] & 0xFFFFu)
                       : keys[at + l];
          const uint32_t iw = (uint32_t)(item >> 32);
          const uint32_t q = 0xFFFFFFFFu - (uint32_t)__builtin_amdgcn_readlane((int)iw, 0);
          if (kBig && whole_rounds(at, q, iw, key)) break;
          const uint32_t add = l < cnt ? (0xFFFFFFFFu - iw) << kb : 0u;
          int32_t mine = 0;  // bin of item l
          for (int t0 = 0; t0 < cnt; t0 += kLptSteps) {
#pragma unroll
            for (int t = t0; t < t0 + kLptSteps; ++t) {
              const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)key, 0);
              const uint32_t nk = k0 + (uint32_t)__builtin_amdgcn_readlane((int)add, t);
              mine = l == t ? (int32_t)(k0 & bmask) : mine;
              const uint32_t nxt = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, 0x130, 0xF,
                                                                         0xF, false);  // wave_shl:1
              key = min(nxt, max(nk, key));
            }
          }
          if (l < cnt) bin_of[(uint32_t)item] = mine;
        }
        if (l < W) win[cur][l] = load0 + key;
        key32 = key;
      } else if (tid < kWave && narrow) {
        const int l = tid;
        const uint32_t bmask = (1u << kb) - 1u;
        uint32_t key = key32;
        for (int base = 0, cnt; base < T; base += cnt) {
          cnt = __builtin_amdgcn_readfirstlane(T - base < kWave ? T - base : kWave);
          // keys relative to the least load again
          const uint32_t sub = (uint32_t)__builtin_amdgcn_readlane((int)key, 0) & ~bmask;
          key -= l < W ? sub : 0u;
          load0 += sub;
          uint64_t item = 0;
          if (l < cnt) {
            const int at = i0 + base + l;
            item = k32 ? ((uint64_t)(0xFFFF0000u | (srt[at] >> 16)) << 32) | (srt[at] & 0xFFFFu)
                       : keys[at];
          }
          int32_t mine = 0;  // bin of item l
          const uint32_t iw = (uint32_t)(item >> 32);
          // (no whole rounds in the LDS forms: at 64 bins the few components they
          // hold gain less from it than other graphs lose, 1.5 us of 25)
          const int at = i0 + base;
          const uint32_t q = 0xFFFFFFFFu - (uint32_t)__builtin_amdgcn_readlane((int)iw, 0);
          if (kBig && single_window && whole_rounds(at, q, iw, key)) break;
          for (int t = 0; t < cnt;) {
            const uint32_t wt = (uint32_t)__builtin_amdgcn_readlane((int)iw, t);
            const uint32_t q = 0xFFFFFFFFu - wt;
            const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)key, 0);
            const uint32_t nk = k0 + (q << kb);
            const uint64_t below = __ballot(key < nk);  // lane 0 and the lanes below nk
            // items t, t+1, ... of the same weight (within this batch)
            const uint64_t same = __ballot(l < cnt && iw == wt) >> t;
            const int run = ~same ? (int)__builtin_ctzll(~same) : kWave;
            const int m = __popcll(below);
            const int c = run < m ? run : m;
            // A prefix round: items t, t+1, ... go to lanes 0, 1, ... for as
            // long as each lane's key is below every key the earlier items of
            // the round raised (lane j is then the least loaded bin when item
            // t + j comes), whatever the weights.  Only lanes below nk can
            // qualify, so it is tried when m allows a long enough round and an
            // equal run does not already take all m.
            int cp = 0;
            uint32_t r = 0xFFFFFFFFu;
            if (m >= kLptPrefixMin && c < m) {
              const bool has = l < cnt - t && l < W;
              const uint32_t ql = 0xFFFFFFFFu - (uint32_t)__shfl((int)iw, (l + t) & (kWave - 1));
              r = has ? key + (ql << kb) : 0xFFFFFFFFu;  // lane l's key after item t + l
              const uint32_t lower = wave_excl_min_u32(r);
              const uint64_t ok = __ballot(has && key < lower);
              cp = ~ok ? (int)__builtin_ctzll(~ok) : kWave;
            }
            if (cp >= kLptPrefixMin) {
              const uint32_t src = (uint32_t)__shfl((int)key, (l - t) & (kWave - 1));
              if (l >= t && l < t + cp) mine = (int32_t)(src & bmask);
              // raised keys in lanes 0..cp-1, the rest unchanged: merged where
              // the raised ones are in order, else sorted
              const uint32_t prev = wave_prev_u32(r);  // by every lane, before the test
              const bool down = l > 0 && l < cp && prev > r;
              key = l < cp ? r : key;
              if (__ballot(down)) {
                key = wave_sort_u32<32>(key, l);
                if (W > 32) key = wave_sort_u32<kWave, kWave, 32>(key, l);
              } else {
                key = lpt_merge_lanes(key, l, cp);
              }
              t += cp;
              // the next items at once, so that a round is not cut short by
              // the end of the lanes' items
              if (base + cnt < T) cnt = t;
            } else if (c >= kLptRoundMin) {
              // a round: c equal items go to lanes 0..c-1 in order (each of
              // those bins is below lane 0's raised key, so the steps would pick
              // them one after another); the raised keys of lanes 0..c-1 and
              // the keys of lanes c.. are two sorted runs, merged by rank
              const uint32_t src = (uint32_t)__shfl((int)key, (l - t) & (kWave - 1));
              if (l >= t && l < t + c) mine = (int32_t)(src & bmask);
              const uint32_t x = l < c ? key + (q << kb) : key;
              key = lpt_merge_lanes(x, l, c);
              t += c;
              if (base + cnt < T) cnt = t;
            } else {
              mine = l == t ? (int32_t)(k0 & bmask) : mine;
              const int p = __popcll(below) - 1;  // lanes 1.. below nk
              const uint32_t nxt = wave_next_u32(key);
              key = l < p ? nxt : (l == p ? nk : key);
              t += 1;
            }
          }
          if (l < cnt) bin_of[(uint32_t)item] = mine;
        }
        if (l < W) win[cur][l] = load0 + key;
        key32 = key;
      } else if (tid < kWave) {
        const int l = tid;
        uint64_t key = key64;
        for (int base = 0; base < T; base += kWave) {
          const int cnt = __builtin_amdgcn_readfirstlane(T - base < kWave ? T - base : kWave);
          uint64_t item = 0;
          if (l < cnt) {
            const int at = i0 + base + l;
            item = k32 ? ((uint64_t)(0xFFFF0000u | (srt[at] >> 16)) << 32) | (srt[at] & 0xFFFFu)
                       : keys[at];
          }
          // item by item, as with few bins and narrow keys
          const uint64_t add =
              l < cnt ? (uint64_t)(0xFFFFFFFFu - (uint32_t)(item >> 32)) << kBinBits : 0ull;
          int32_t mine = 0;  // bin of item l, kept in lane l until the batch ends
          for (int t0 = 0; t0 < cnt; t0 += kLptWideSteps) {
#pragma unroll
            for (int t = t0; t < t0 + kLptWideSteps; ++t) {
              const uint64_t k0 = wave_lane(key, 0), nk = k0 + wave_lane(add, t);
              mine = l == t ? (int32_t)(k0 & ((1u << kBinBits) - 1)) : mine;
              const uint64_t nxt = wave_next_u64(key), x = nk > key ? nk : key;
              key = nxt < x ? nxt : x;
            }
          }
          if (l < cnt) bin_of[(uint32_t)item] = mine;
        }
        if (l < W) win[cur][l] = key;
        key64 = key;
      }
      // the window's raised keys are out, and the previous window's merge (by
      // the other waves, during these steps) is done
      __syncthreads();
      if (single_window) {
        if (tid < W) binA[tid] = win[cur][tid];
        int items = 0, at = nc;
        if constexpr (kBig) {
          items = __builtin_amdgcn_readfirstlane(s_op_items);
          if (items) at = __builtin_amdgcn_readfirstlane(s_op_at);
          store_rounds(at, items, s_op_bins, [&](int r) { return s_opbin[r]; });
          __syncthreads();
        }
        i0 = at + items;
      } else {
        if (tid < kWave) {
          if (i0 + T < lim) {
            // the next window: the W (= 64) least of the raised keys and
            // binA[W..2W), as min(raised key l, binA[2W-1-l]) (a bitonic run
            // holding exactly those) sorted by the bitonic merge's stages
            const int l = tid, j = W + (kWave - 1) - l;
            if (narrow) {
              const uint32_t b = j < P ? (uint32_t)(binA[j] - load0) : 0xFFFFFFFFu;
              uint32_t c = key32 < b ? key32 : b;
              c = bitonic_lane_step<32>(c, l, kWave);
              c = bitonic_lane_step<16>(c, l, kWave);
              c = bitonic_lane_step<8>(c, l, kWave);
              c = bitonic_lane_step<4>(c, l, kWave);
              c = bitonic_lane_step<2>(c, l, kWave);
              key32 = bitonic_lane_step<1>(c, l, kWave);
            } else {
              const uint64_t b = j < P ? binA[j] : ~0ull;
              uint64_t c = key64 < b ? key64 : b;
              c = bitonic_lane_step<32>(c, l, kWave);
              c = bitonic_lane_step<16>(c, l, kWave);
              c = bitonic_lane_step<8>(c, l, kWave);
              c = bitonic_lane_step<4>(c, l, kWave);
              c = bitonic_lane_step<2>(c, l, kWave);
              key64 = bitonic_lane_step<1>(c, l, kWave);
            }
          }
        } else {
          // the other waves: the raised keys (sorted) merged with binA[W..P)
          // (sorted) into binB.  Merge thread t < W places raised key t (its
          // rank in binA[W..P) by binary search); the others place the list's
          // keys, two at once (each one's rank among the W = 64 raised keys by
          // six fixed steps, the two searches interleaved)
          const uint64_t *wk = win[cur];
          const int t = tid - kWave, mt = (int)blockDim.x - kWave - W;  // list threads
          if (t < W) {
            const uint64_t x = wk[t];
            binB[t + lower_bound_u64(binA + W, P - W, x)] = x;
          } else {
            for (int j0 = t - W; j0 < P - W; j0 += 2 * mt) {
              const int j1 = j0 + mt;
              const bool two = j1 < P - W;
              const uint64_t x0 = binA[W + j0], x1 = two ? binA[W + j1] : 0ull;
              int r0 = 0, r1 = 0;
  #pragma unroll
              for (int step = kWave / 2; step > 0; step >>= 1) {
                r0 += wk[r0 + step - 1] < x0 ? step : 0;
                r1 += wk[r1 + step - 1] < x1 ? step : 0;
              }
              r0 += wk[r0] < x0 ? 1 : 0;
              r1 += wk[r1] < x1 ? 1 : 0;
              binB[j0 + r0] = x0;
              if (two) binB[j1 + r1] = x1;
            }
          }
        }
        uint64_t *t = binA;
        binA = binB;
        binB = t;
        cur ^= 1;
        i0 += T;
      }
    }
    __syncthreads();  // the last merge is done: binA holds the whole bin list
  }
  // 3. (bin, label) order, read offsets and the reads of each bin; keys
  // (bin << 16) | i in 32 bits when bin and index fit 16 bits
  auto store_loads = [&] {
    for (int b = tid; b < P; b += blockDim.x) {
      const uint64_t k = binA[b];
      bin_load[k & ((1ull << bb) - 1)] = k >> bb;
    }
  };
  if (!comp_rank) {
    store_loads();
    return 0;
  }
  const bool b32 = !kBig && nc <= 0xFFFF && P <= 0x10000;
  if (kBig) keys = reinterpret_cast<uint64_t *>(keys32);  // the start of the key area
  for (int i = tid; i < (kBig ? nc : N2); i += blockDim.x) {
    if (b32)
      keys32[i] = i < nc ? ((uint32_t)bin_of[i] << 16) | (uint32_t)i : ~0u;
    else
      keys[i] = i < nc ? ((uint64_t)(uint32_t)bin_of[i] << 32) | (uint32_t)i : ~0ull;
  }
  // the reads of each bin are summed in binB (free once the loads are out;
  // in LDS when the bins are), then written once per bin
  if (bin_reads) {
    for (int b = tid; b < P; b += blockDim.x) binB[b] = 0;
    __syncthreads();
    for (int i = tid; i < nc; i += blockDim.x)
      atomicAdd((unsigned long long *)binB + bin_of[i], (unsigned long long)comp_size[i]);
  }
  __syncthreads();
  // (bin, label) order: radix passes over the bin's bytes (one up to 256
  // bins) as above, else a bitonic sort
  const uint32_t *srt2 = keys32;
  if constexpr (kBig)
    keys = radix_sort_hi32<BLOCK>(keys, keys + nc, nc, value_bytes((uint32_t)(P - 1)), s_cnt,
                                  reinterpret_cast<uint32_t *>(sh_scan));
  else if (b32 && radix(P <= 256 ? 1 : 2))
    srt2 = radix_sort_hi16<BLOCK>(keys32, keys32 + N2, nc, P <= 256 ? 1 : 2, s_cnt,
                                  reinterpret_cast<uint32_t *>(sh_scan));
  else if (b32)
    small_sort(keys32);
  else
    small_sort(keys);
  // a thread takes up to eight consecutive components of the order per round
  int carry = 0, ecarry = 0;
  for (int base = 0; base < nc; base += kPer * BLOCK) {
    const int E = nc - base < kPer * BLOCK ? (nc - base + BLOCK - 1) / BLOCK : kPer;
    uint32_t c[kPer];
    int32_t sz[kPer], e2[kPer], sum = 0, esum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = base + tid * E + k;
      c[k] = ~0u;
      if (k >= E) continue;
      c[k] = i < nc ? (b32 ? srt2[i] & 0xFFFFu : (uint32_t)keys[i]) : ~0u;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      sz[k] = e2[k] = 0;
      if (k >= E) continue;
      const bool v = c[k] != ~0u;
      sz[k] = v ? comp_size[c[k]] : 0;
      if (comp_estart && v) {
        const uint8_t kd = comp_kind[c[k]];
        e2[k] = kd == CG_KIND_PATH ? 2 * (sz[k] - 1) : (kd == CG_KIND_CYCLE ? 2 * sz[k] : 0);
      }
      sum += sz[k];
      esum += e2[k];
    }
    // reads and local entries in one scan: (reads << 32) | entries, each
    // field's total below 2^32 (entries <= 2 * reads, reads < 2^31)
    int32_t st, est = 0;
    if (comp_estart) {
      int64_t tot;
      const int64_t ex = block_excl_scan<int64_t, BLOCK>(((int64_t)sum << 32) | (uint32_t)esum,
                                                         sh_scan64, &tot);
      st = carry + (int32_t)(ex >> 32);
      est = ecarry + (int32_t)(uint32_t)ex;
      carry += (int32_t)(tot >> 32);
      ecarry += (int32_t)(uint32_t)tot;
    } else {
      int32_t tot;
      st = carry + block_excl_scan<int32_t, BLOCK>(sum, sh_scan, &tot);
      carry += tot;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (k >= E || c[k] == ~0u) continue;
      const int i = base + tid * E + k;
      comp_start[c[k]] = st;
      comp_rank[c[k]] = i;
      if (ro.bin_vptr) {
        // where the bins from the last component's on to this one's start
        const int32_t b = (int32_t)(b32 ? srt2[i] >> 16 : (uint32_t)(keys[i] >> 32));
        const int32_t pb =
            i > 0 ? (int32_t)(b32 ? srt2[i - 1] >> 16 : (uint32_t)(keys[i - 1] >> 32)) : -1;
        for (int32_t x = pb + 1; x <= b; ++x) ro.bin_vptr[x] = st;
        if (ro.comp_kind[c[k]] == CG_KIND_CYCLE) mark_cycle(ro.cyc, i);
      }
      st += sz[k];
      if (comp_estart) {
        comp_estart[c[k]] = est;
        est += e2[k];
      }
    }
  }
  if (ro.bin_vptr) {
    const int32_t last =
        nc > 0 ? (int32_t)(b32 ? srt2[nc - 1] >> 16 : (uint32_t)(keys[nc - 1] >> 32)) : -1;
    for (int b = last + 1 + tid; b <= P; b += blockDim.x) ro.bin_vptr[b] = carry;
    if (tid == 0) {
      ro.d_sizes[0] = carry;
      if (nc == 0) ro.d_sizes[1] = ro.loc_row_ptr[0] = 0;
    }
  }
  // the per-bin and per-component results, stored after the last barrier
  // (a barrier waits for the stores issued before it); binA still holds the
  // final bin list and binB the reads of each bin
  store_loads();
  if (bin_reads)
    for (int b = tid; b < P; b += blockDim.x) bin_reads[b] = binB[b];
  if (comp_bin != bin_of)
    for (int i = tid; i < nc; i += blockDim.x) comp_bin[i] = bin_of[i];
  return ecarry;
}

// ---------------------------------------------------------------------------
// InducedSubgraph: sort one component's block of reads by id (local numbers
// follow (bin, label, id)); one workgroup of kIndBlock threads
// ---------------------------------------------------------------------------
constexpr int kIndBlock = 256;
constexpr int kIndLocalCap = 1024;

// lidx (the local number of each read) is written for components above CAP
// reads only (the ones whose neighbours are then numbered through it instead
// of the sorted block).
// Member i's id is members[MS * i].
template <int BLOCK, int CAP, int MS = 1>
__device__ __forceinline__ void sort_component_block(int q, int st,
                                                     const int32_t *__restrict__ members,
                                                     int32_t *__restrict__ perm,
                                                     int32_t *__restrict__ lidx, int32_t *a) {
  if (q <= CAP) {
    int N2 = 1;
    while (N2 < q) N2 <<= 1;
    for (int i = threadIdx.x; i < N2; i += BLOCK) a[i] = i < q ? members[MS * i] : 0x7FFFFFFF;
    __syncthreads();
    // non-negative ids padded with the largest int32: the same order as uint32
    bitonic_sort(reinterpret_cast<uint32_t *>(a), N2);
    for (int i = threadIdx.x; i < q; i += BLOCK) {
      perm[st + i] = a[i];
    }
  } else {
    // large component: its ids in a bitmap of CAP / 2 words of LDS, one window
    // of ids after another, and the set bits before each word: a read's rank
    // is the bits below its own (every member is loaded twice per window;
    // counting the smaller ids took q loads per read, 1.5 ms for the 3,000
    // reads of one component)
    constexpr int kWords = CAP / 2;
    __shared__ int32_t sh_lo, sh_hi;
    __shared__ int32_t sh_cnt[BLOCK / kWave + 1];
    if (threadIdx.x == 0) {
      sh_lo = 0x7FFFFFFF;
      sh_hi = 0;
    }
    __syncthreads();
    int32_t mn = 0x7FFFFFFF, mx = 0;
    for (int i = threadIdx.x; i < q; i += BLOCK) {
      const int32_t x = members[MS * (int64_t)i];
      mn = x < mn ? x : mn;
      mx = x > mx ? x : mx;
    }
    atomicMin(&sh_lo, mn);
    atomicMax(&sh_hi, mx);
    __syncthreads();
    uint32_t *bits = reinterpret_cast<uint32_t *>(a);
    int32_t *pre = a + kWords;
    int32_t done = 0;  // members below the window
    for (int64_t w0 = sh_lo & ~31; w0 <= sh_hi; w0 += 32 * kWords) {
      for (int i = threadIdx.x; i < kWords; i += BLOCK) bits[i] = 0;
      __syncthreads();
      for (int i = threadIdx.x; i < q; i += BLOCK) {
        const int64_t x = members[MS * (int64_t)i] - w0;
        if (x >= 0 && x < 32 * kWords) atomicOr(bits + (x >> 5), 1u << (x & 31));
      }
      __syncthreads();
      constexpr int E = kWords / BLOCK;  // consecutive words per thread
      static_assert(E * BLOCK == kWords, "whole words per thread");
      int32_t sum = 0;
#pragma unroll
      for (int k = 0; k < E; ++k) sum += __popc(bits[threadIdx.x * E + k]);
      int32_t tot;
      int32_t ex = done + block_excl_scan<int32_t, BLOCK>(sum, sh_cnt, &tot);
#pragma unroll
      for (int k = 0; k < E; ++k) {
        pre[threadIdx.x * E + k] = ex;
        ex += __popc(bits[threadIdx.x * E + k]);
      }
      done += tot;
      __syncthreads();
      for (int i = threadIdx.x; i < q; i += BLOCK) {
        const int32_t v = members[MS * (int64_t)i];
        const int64_t x = v - w0;
        if (x >= 0 && x < 32 * kWords) {
          const int32_t r = pre[x >> 5] + __popc(bits[x >> 5] & ((1u << (x & 31)) - 1u));
          perm[st + r] = v;
          lidx[v] = st + r;
        }
      }
      __syncthreads();
    }
  }
  __syncthreads();
}

// InducedSubgraph for one component, all in one workgroup: sort its reads
// (members, in any order) by id, number them st, st+1, ..., and write their
// local CSR rows (kept entries in row order of S, neighbours renumbered,
// entry index kept)
// starting at entry estart.  Neighbours of a kept entry lie in the same
// component, so their local numbers come from the sorted block itself.
template <int BLOCK, int CAP, int MS = 1>
__device__ __forceinline__ void induce_component(
    int q, int st, int estart, const int32_t *__restrict__ members,
    const uint8_t *__restrict__ flags,
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    int32_t *__restrict__ perm, int32_t *__restrict__ lidx, int32_t *__restrict__ loc_row_ptr,
    int32_t *__restrict__ loc_col, int32_t *__restrict__ loc_eid, int32_t *a,
    int32_t *sh_scan) {
  sort_component_block<BLOCK, CAP, MS>(q, st, members, perm, lidx, a);  // ends with a barrier
  const bool in_lds = q <= CAP;
  int carry = 0;
  for (int base = 0; base < q; base += BLOCK) {
    const int i = base + threadIdx.x;
    int32_t v = -1, b = 0;
    uint32_t f = 0;
    if (i < q) {
      v = in_lds ? a[i] : perm[st + i];
      f = flags[v];
      b = row_ptr[v];  // with the flags, before the scan
    }
    const int32_t deg = (int32_t)(((f >> 1) & 1) + ((f >> 2) & 1));
    int32_t tot;
    const int32_t ex = block_excl_scan<int32_t, BLOCK>(deg, sh_scan, &tot);
    if (i < q) {
      int32_t r = estart + carry + ex;
      loc_row_ptr[st + i] = r;
      for (int j = 0; j < 2; ++j) {
        if (!(f & (2u << j))) continue;
        const int32_t u = col[b + j];
        int32_t li;
        if (in_lds) {
          int lo = 0, hi = q - 1;  // u is in the sorted block
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (a[mid] < u) lo = mid + 1;
            else hi = mid;
          }
          li = st + lo;
        } else {
          li = lidx[u];
        }
        loc_col[r] = li;
        loc_eid[r] = b + j;
        ++r;
      }
    }
    carry += tot;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// LocalAssembly: chain walk of one component, packed base access
// ---------------------------------------------------------------------------
constexpr int kWalkBlock = 256;
constexpr int kWalkRaysCap = 4096;           // reads per component with rays in LDS
// small components: one wave each, so many more are walked at once
constexpr int kWalkSmallCap = 128;

// Where a piece starts in the store, as the copy needs it (Section 4.4: the
// piece is bases [skip, skip + plen) of its read in walking orientation).
// Bits 0-62: forward, the stored base of the piece's first base; reverse,
// one past the stored base of its first base (the piece is read backwards
// from there).  Bit 63: the read is walked reverse-complemented.  A read
// ends inside the store (read_off + read_len <= 16 seq_words), so the base
// offset stays below 2^63.
__device__ __forceinline__ uint64_t piece_anchor(uint64_t roff, uint32_t rlen, uint32_t skip,
                                                 bool rev) {
  return rev ? ((roff + rlen - skip) | (1ull << 63)) : roff + skip;
}

typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

struct WalkArrays {
  int32_t *nb;     // [2q] local neighbour of slot k of read i (-1: none / cut)
  int32_t *eid;    // [2q] entry index in S of that slot (LDS form: the piece lengths
                   // in walk order take its place once the rows are written)
  uint32_t *ray;   // [2q] rays in LDS (see walk_chain)
  uint64_t *gray;  // [2q] rays in global memory, of a component too large for LDS rays
  // the LDS form also keeps what the pieces need, loaded before the doubling:
  int32_t *vid;    // [q] read id of local read i
  uint32_t *rlen;  // [q] its length
  uint64_t *roff;  // [q] its first base in the store
  uint8_t *es;     // [2q] strand bits of the entry of slot k
  uint32_t *eo;    // [2q] its pre (explicit coordinates) or overlap length
  uint32_t *ep;    // [2q] its post (explicit coordinates)
};

// What a walk keeps where: everything in LDS; only the rays in LDS; nothing.
enum WalkMode { kWalkLds, kWalkRaysLds, kWalkGlobal };

// The arrays in global scratch (16 n ints) of the component whose block
// starts at st: the blocks of different components are disjoint, so slices
// never overlap.
__device__ __forceinline__ WalkArrays walk_scratch(int32_t *buf, int64_t n, int64_t st,
                                                   uint32_t *ray) {
  WalkArrays w{};
  w.nb = buf + 2 * st;
  w.eid = buf + 2 * n + 2 * st;
  w.gray = reinterpret_cast<uint64_t *>(buf + 4 * n) + 2 * st;
  w.ray = ray;
  return w;
}

// What a component's contig record takes from the component table: its
// record index (the component's (bin, label) rank), label and bin.  Loaded
// when the component's work starts, so that no load waits at its end.
struct CompRec {
  int32_t rank, label, bin;
};
__device__ __forceinline__ CompRec comp_rec(const cg_parts &parts, int c, int32_t rank) {
  return CompRec{rank, ((const CG_GLOBAL int32_t *)parts.comp_label)[c],
                 ((const CG_GLOBAL int32_t *)parts.comp_bin)[c]};
}
__device__ __forceinline__ CompRec comp_rec(const cg_parts &parts, int c) {
  return comp_rec(parts, c, ((const CG_GLOBAL int32_t *)parts.comp_rank)[c]);
}

// Steps 2-5 of the walk, from the component's rows in w (nb, eid; and in the
// LDS form vid, rlen, roff, es, eo, ep); first: the smallest of the thread's
// reads that has one neighbour (0x7FFFFFFF: none).
template <int BLOCK, int CAP, WalkMode kMode>
__device__ __forceinline__ void walk_chain(const CompRec &cr, int q, int st, int first, WalkArrays w,
                                           const cg_graph &g, const int32_t *__restrict__ perm,
                                           const cg_contigs &out, const Scratch &s,
                                           uint64_t *sh_scan);

// A component of one workgroup of BLOCK threads, or of one wave of a larger
// workgroup (BLOCK = kWave: no workgroup barrier, the arrays are the wave's
// own).
template <int BLOCK, int CAP, WalkMode kMode>
__device__ __forceinline__ void walk_component(
    int c, int q, int st, WalkArrays w, const cg_graph &g, const cg_parts &parts,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ loc_row_ptr,
    const int32_t *__restrict__ loc_col, const int32_t *__restrict__ loc_eid,
    const cg_contigs &out, const Scratch &s, uint64_t *sh_scan) {
  const int tid = BLOCK == kWave ? lane_id() : (int)threadIdx.x;
  const CompRec cr = comp_rec(parts, c);
  int first = 0x7FFFFFFF;
  // 1. local rows of the component's block
  if constexpr (kMode == kWalkLds) {
    // and, in three rounds of loads issued together, the read ids and
    // lengths and the entries' strand bits and overlaps (or coordinates)
    constexpr int R = CAP / BLOCK;
    const CG_GLOBAL int32_t *lrp = (const CG_GLOBAL int32_t *)loc_row_ptr;
    const CG_GLOBAL int32_t *lcol = (const CG_GLOBAL int32_t *)loc_col;
    const CG_GLOBAL int32_t *leid = (const CG_GLOBAL int32_t *)loc_eid;
    const CG_GLOBAL int32_t *gperm = (const CG_GLOBAL int32_t *)perm;
    const CG_GLOBAL uint32_t *glen = (const CG_GLOBAL uint32_t *)g.read_len;
    const CG_GLOBAL uint64_t *goff = (const CG_GLOBAL uint64_t *)g.read_off;
    const CG_GLOBAL uint8_t *gstr = (const CG_GLOBAL uint8_t *)g.strand;
    const CG_GLOBAL uint32_t *gov =
        (const CG_GLOBAL uint32_t *)(g.pre ? g.pre : g.ovl);
    const CG_GLOBAL uint32_t *gpost = (const CG_GLOBAL uint32_t *)g.post;
    int ra[R], rd[R], rv[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = tid + u * BLOCK;
      ra[u] = rd[u] = rv[u] = 0;
      if (i < q) {
        ra[u] = lrp[st + i];
        rd[u] = lrp[st + i + 1];
        rv[u] = gperm[st + i];
      }
    }
    int c0[R], c1[R], e0[R], e1[R];
    uint32_t rl[R];
    uint64_t ro[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = tid + u * BLOCK;
      const int deg = i < q ? rd[u] - ra[u] : 0;
      c0[u] = c1[u] = e0[u] = e1[u] = -1;
      rl[u] = 0;
      ro[u] = 0;
      if (i < q) {
        rl[u] = glen[rv[u]];
        ro[u] = goff[rv[u]];
      }
      if (deg >= 1) {
        c0[u] = lcol[ra[u]];
        e0[u] = leid[ra[u]];
      }
      if (deg >= 2) {
        c1[u] = lcol[ra[u] + 1];
        e1[u] = leid[ra[u] + 1];
      }
    }
    uint32_t s0[R], s1[R], o0[R], o1[R], p0[R], p1[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      s0[u] = s1[u] = o0[u] = o1[u] = p0[u] = p1[u] = 0;
      if (e0[u] >= 0) {
        s0[u] = gstr[e0[u]];
        o0[u] = gov[e0[u]];
        if (gpost) p0[u] = gpost[e0[u]];
      }
      if (e1[u] >= 0) {
        s1[u] = gstr[e1[u]];
        o1[u] = gov[e1[u]];
        if (gpost) p1[u] = gpost[e1[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = tid + u * BLOCK;
      if (i >= q) continue;
      w.nb[2 * i] = c0[u] >= 0 ? c0[u] - st : -1;
      w.nb[2 * i + 1] = c1[u] >= 0 ? c1[u] - st : -1;
      if (c0[u] >= 0 && c1[u] < 0 && i < first) first = i;
      w.vid[i] = rv[u];
      w.rlen[i] = rl[u];
      w.roff[i] = ro[u];
      w.es[2 * i] = (uint8_t)s0[u];
      w.es[2 * i + 1] = (uint8_t)s1[u];
      w.eo[2 * i] = o0[u];
      w.eo[2 * i + 1] = o1[u];
      w.ep[2 * i] = p0[u];
      w.ep[2 * i + 1] = p1[u];
    }
  } else {
    constexpr int U = 4;
    for (int b0 = tid; b0 < q; b0 += U * BLOCK) {
      int a[U], deg[U], c0[U], c1[U], e0[U], e1[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = b0 + u * BLOCK < q ? b0 + u * BLOCK : q - 1;
        a[u] = loc_row_ptr[st + i];
        deg[u] = loc_row_ptr[st + i + 1] - a[u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c0[u] = deg[u] >= 1 ? loc_col[a[u]] - st : -1;
        c1[u] = deg[u] >= 2 ? loc_col[a[u] + 1] - st : -1;
        e0[u] = deg[u] >= 1 ? loc_eid[a[u]] : -1;
        e1[u] = deg[u] >= 2 ? loc_eid[a[u] + 1] : -1;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = b0 + u * BLOCK;
        if (i >= q) continue;
        w.nb[2 * i] = c0[u];
        w.nb[2 * i + 1] = c1[u];
        if (deg[u] == 1 && i < first) first = i;
        w.eid[2 * i] = e0[u];
        w.eid[2 * i + 1] = e1[u];
      }
    }
  }
  walk_chain<BLOCK, CAP, kMode>(cr, q, st, first, w, g, perm, out, s, sh_scan);
}

// Ray (i, k) leaves read i through slot k.  It holds how many steps it has
// gone and the ray it goes on with, or how it ended: at the walk's start or
// at the chain's other end.  Both are in one word, so that a jump
// (ray += the ray it goes on with) replaces them together: a ray's word is
// true whenever it is read, and no barrier is needed between jumps.
struct Ray32 {  // LDS: steps << 16 | next (rays and steps below 0xFFFE)
  typedef uint32_t T;
  static constexpr T kAtStart = 0xFFFEu, kAtEnd = 0xFFFFu;
  static __device__ __forceinline__ T make(uint32_t steps, T next) { return steps << 16 | next; }
  static __device__ __forceinline__ T next(T x) { return x & 0xFFFFu; }
  static __device__ __forceinline__ int steps(T x) { return (int)(x >> 16); }
  static __device__ __forceinline__ T jump(T x, T y) { return (x & 0xFFFF0000u) + y; }
};
struct Ray64 {  // global memory: steps << 32 | next
  typedef uint64_t T;
  static constexpr T kAtStart = 0xFFFFFFFEull, kAtEnd = 0xFFFFFFFFull;
  static __device__ __forceinline__ T make(uint32_t steps, T next) {
    return (uint64_t)steps << 32 | next;
  }
  static __device__ __forceinline__ T next(T x) { return x & 0xFFFFFFFFull; }
  static __device__ __forceinline__ int steps(T x) { return (int)(x >> 32); }
  static __device__ __forceinline__ T jump(T x, T y) { return (x & ~0xFFFFFFFFull) + y; }
};
template <typename T>
__device__ __forceinline__ T ray_ld(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void ray_st(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Jumps the rays to their ends (pointer doubling; U rays of a thread at a
// time, their loads issued together).  Every pass of the loop moves a ray
// that has not ended at least one ray on, so it ends within q passes
// whatever the other waves do, and within about log2 q when they keep up.
// kVisit 0: a thread's U rays are all it has.  Else it goes round its rays,
// kVisit jumps a visit, so that all of them keep up: where the reads are
// numbered along the chain the rays after a thread's first ones are those of
// its later visits, and taking the first ones to their ends went through these
// one by one (one component of 12,000 reads: 36 ms, 0.2 ms so; in random order
// 0.34 and 0.32 ms).
template <typename RAY, int BLOCK, int U, int kVisit>
__device__ __forceinline__ void walk_rays(typename RAY::T *ray, int n_rays, int tid) {
  typedef typename RAY::T T;
  constexpr bool kAll = kVisit == 0;
  // (no more passes than reads, so that no input can keep it here)
  const int visit = kAll ? n_rays / 2 : kVisit;
  uint64_t ended = 0;  // the first 64 visits whose rays have all ended
  bool again = true;
  for (int turn = 0; again && turn <= n_rays / 2; ++turn) {
    again = false;
    uint64_t bit = 1;
    for (int r0 = tid; r0 < n_rays; r0 += U * BLOCK, bit <<= 1) {
      if (!kAll && (ended & bit)) continue;
      T x[U];
      bool more = false;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * BLOCK;
        x[u] = r < n_rays ? ray_ld(ray + r) : RAY::kAtEnd;
        more = more || RAY::next(x[u]) < RAY::kAtStart;
      }
      for (int pass = 0; more && pass < visit; ++pass) {
        T y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const T nx = RAY::next(x[u]);
          y[u] = ray_ld(ray + (nx < RAY::kAtStart ? (int)nx : 0));
        }
        more = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (RAY::next(x[u]) >= RAY::kAtStart) continue;
          x[u] = RAY::jump(x[u], y[u]);
          ray_st(ray + r0 + u * BLOCK, x[u]);
          more = more || RAY::next(x[u]) < RAY::kAtStart;
        }
      }
      again = again || more;
      ended |= more ? 0ull : bit;
    }
    if constexpr (kAll) break;
  }
}

template <int BLOCK, int CAP, WalkMode kMode>
__device__ __forceinline__ void walk_chain(const CompRec &cr, int q, int st, int first, WalkArrays w,
                                           const cg_graph &g, const int32_t *__restrict__ perm,
                                           const cg_contigs &out, const Scratch &s,
                                           uint64_t *sh_scan) {
  constexpr bool kLds = kMode == kWalkLds;
  constexpr bool kOneWave = BLOCK == kWave;
  const int tid = kOneWave ? lane_id() : (int)threadIdx.x;
  // the LDS form orders LDS only at its barriers (its global stores stay in
  // flight; nothing it reads back from global memory was written here); the
  // other forms' arrays are global memory
  auto wbar = [] {
    if constexpr (kOneWave) wave_lds_sync();
    else if constexpr (kLds) lds_barrier();
    else __syncthreads();
  };
  // 2. start: the first read of local degree 1 (the smaller-id root, since
  // the block is in id order); a cycle starts at its first read and loses
  // the edge to the larger-numbered neighbour of it
  __shared__ int s_start, s_sej;  // (a one-wave walk keeps these in registers)
  if constexpr (!kOneWave) {
    if (tid == 0) {
      s_start = 0x7FFFFFFF;
      s_sej = 0;
    }
  }
  wbar();
  if constexpr (kOneWave) {
    // (the largest complement: an index is never negative)
    first = 0x7FFFFFFF - (int)wave_max_u32((uint32_t)(0x7FFFFFFF - first));
  } else {
    if (first != 0x7FFFFFFF) atomicMin(&s_start, first);
    wbar();
    first = s_start;
  }
  const bool cyc = first == 0x7FFFFFFF && q > 1;
  const int s0 = first == 0x7FFFFFFF ? 0 : first;
  if (cyc) {  // uniform
    if (tid == 0) {
      const int x = w.nb[0], y = w.nb[1];
      const int t = x > y ? x : y;  // closing neighbour
      if (x > y) w.nb[0] = -1; else w.nb[1] = -1;
      if (w.nb[2 * t] == 0) w.nb[2 * t] = -1; else w.nb[2 * t + 1] = -1;
    }
    wbar();
  }
  // 3. rays, jumped along the chain to its ends
  typedef typename std::conditional<kMode == kWalkGlobal, Ray64, Ray32>::type RAY;
  typename RAY::T *ray;
  if constexpr (kMode == kWalkGlobal) ray = w.gray;
  else ray = w.ray;
  constexpr int V = kLds ? (CAP > BLOCK ? CAP / BLOCK : 1) : 2;  // reads of a thread at a time
  for (int b0 = tid; b0 < q; b0 += V * BLOCK) {
    int y[V][2], z[V][2][2];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int i = b0 + u * BLOCK;
#pragma unroll
      for (int k = 0; k < 2; ++k) y[u][k] = i < q ? w.nb[2 * i + k] : -1;
    }
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int x = y[u][k] >= 0 ? y[u][k] : 0;
        z[u][k][0] = w.nb[2 * x];
        z[u][k][1] = w.nb[2 * x + 1];
      }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int i = b0 + u * BLOCK;
      if (i >= q) continue;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        typename RAY::T x = RAY::kAtEnd;
        if (y[u][k] >= 0) {
          const int k2 = z[u][k][0] == i ? 1 : 0;  // the neighbour's slot that does not lead back
          x = RAY::make(1, (k2 ? z[u][k][1] : z[u][k][0]) >= 0
                               ? (typename RAY::T)(2 * y[u][k] + k2)
                               : (y[u][k] == s0 ? RAY::kAtStart : RAY::kAtEnd));
        }
        ray_st(ray + 2 * i + k, x);
      }
    }
  }
  wbar();
  // (jumps a visit: 4, 8, 16, 48 on rays in global memory, 20 components of
  // 20,000 reads: 885, 900, 920, 950 us; rays in LDS, eight a thread and 16
  // jumps: the 50 Mbp graph's long contigs 118.0 us, four a thread 119.8)
  if constexpr (kLds) walk_rays<RAY, BLOCK, 2 * CAP / BLOCK, 0>(ray, 2 * q, tid);
  else if constexpr (kMode == kWalkGlobal) walk_rays<RAY, BLOCK, 4, 4>(ray, 2 * q, tid);
  else if (q <= 2 * BLOCK) walk_rays<RAY, BLOCK, 4, 0>(ray, 2 * q, tid);
  else walk_rays<RAY, BLOCK, 8, 16>(ray, 2 * q, tid);
  wbar();
  // 4. rank, predecessor, successor, orientation and piece of every read, U
  // reads of a thread at a time: what a read needs comes in three rounds of
  // loads (its slots and rays; its predecessor's slots, its entries and the
  // read itself; the two entries' fields), each round's issued together.  In
  // LDS the compiler keeps more in flight with one read at a time.
  int32_t *R_vid = out.layout_vid + st;
  uint8_t *R_rev = out.layout_rev + st;
  uint32_t *R_len = s.piece_len + st;
  uint64_t *R_src = s.piece_src + st;
  const int rank_c = cr.rank;
  const bool coords = g.pre != nullptr;
  bool sej = false;
  constexpr int U = kLds ? 1 : 2;
  for (int b0 = tid; b0 < q; b0 += U * BLOCK) {
    int rank[U], pred[U], ss[U], ps[U], pe[U], se[U];
    int32_t v[U];
    uint32_t L[U], ses[U], pes[U], so[U], pp[U];
    uint64_t roff[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b0 + u * BLOCK;
      rank[u] = 0;
      pred[u] = ss[u] = -1;
      v[u] = 0;
      if (i >= q) continue;
      const int n0 = w.nb[2 * i], n1 = w.nb[2 * i + 1];
      const typename RAY::T y0 = ray[2 * i], y1 = ray[2 * i + 1];
      v[u] = kLds ? w.vid[i] : perm[st + i];
      if (i == s0) {
        ss[u] = n0 >= 0 ? 2 * i : (n1 >= 0 ? 2 * i + 1 : -1);
      } else if (n0 >= 0 && RAY::next(y0) == RAY::kAtStart) {
        rank[u] = RAY::steps(y0);
        pred[u] = n0;
        if (n1 >= 0) ss[u] = 2 * i + 1;
      } else if (n1 >= 0 && RAY::next(y1) == RAY::kAtStart) {
        rank[u] = RAY::steps(y1);
        pred[u] = n1;
        if (n0 >= 0) ss[u] = 2 * i;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b0 + u * BLOCK;
      ps[u] = pe[u] = se[u] = -1;  // ps: slot of pred leading to i (its entry pred -> i)
      L[u] = 0;
      roff[u] = 0;
      if (i >= q) continue;
      L[u] = kLds ? w.rlen[i] : g.read_len[v[u]];
      roff[u] = kLds ? w.roff[i] : g.read_off[v[u]];
      if (!kLds && ss[u] >= 0) se[u] = w.eid[ss[u]];
      if (pred[u] >= 0) {
        const bool back0 = w.nb[2 * pred[u]] == i;
        ps[u] = back0 ? 2 * pred[u] : 2 * pred[u] + 1;
        if constexpr (!kLds) {
          // (both in one 8-byte load: a large component is bound by its one
          // compute unit's scattered accesses; with lay_contig stored in the
          // reads' order, 50 Mbp's component pass with long contigs took
          // 84.5 us instead of 88.0)
          const i32x2 ee = *reinterpret_cast<const i32x2 *>(w.eid + 2 * pred[u]);
          pe[u] = back0 ? ee.x : ee.y;
        }
      }
    }
    // strand bits, overlap or coordinates of the two entries
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ses[u] = pes[u] = so[u] = pp[u] = 0;
      if (ss[u] >= 0) {
        ses[u] = kLds ? w.es[ss[u]] : (uint32_t)g.strand[se[u]];
        so[u] = kLds ? w.eo[ss[u]] : (coords ? g.pre[se[u]] : g.ovl[se[u]]);
      }
      if (ps[u] >= 0) {
        pes[u] = kLds ? w.es[ps[u]] : (uint32_t)g.strand[pe[u]];
        if (coords) pp[u] = kLds ? w.ep[ps[u]] : g.post[pe[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b0 + u * BLOCK;
      if (i >= q) continue;
      int orient;
      if (i == s0) orient = ss[u] >= 0 ? (int)(ses[u] & 1) : 0;
      else if (ps[u] >= 0) orient = (int)((pes[u] >> 1) & 1);
      else orient = 0;  // unreachable for a chain: every read but the start has a predecessor
      // the piece: walking offsets [skip, end] of the read (Section 4.4: from
      // post of the entering entry to pre of the leaving one, in stored
      // coordinates; from overlap lengths: the read minus its overlap with the
      // successor)
      uint32_t skip = 0, plen = L[u];
      if (coords) {
        const int64_t first_b =
            ps[u] >= 0 ? (orient ? (int64_t)L[u] - 1 - pp[u] : (int64_t)pp[u]) : 0;
        const int64_t last_b =
            ss[u] >= 0 ? (orient ? (int64_t)L[u] - 1 - so[u] : (int64_t)so[u]) : (int64_t)L[u] - 1;
        skip = (uint32_t)first_b;
        plen = last_b >= first_b ? (uint32_t)(last_b - first_b + 1) : 0u;
      } else if (ss[u] >= 0) {
        plen -= so[u];
      }
      if (ss[u] >= 0 && (int)(ses[u] & 1) != orient) sej = true;
      R_vid[rank[u]] = v[u];
      R_rev[rank[u]] = (uint8_t)orient;
      R_len[rank[u]] = plen;
      if constexpr (kLds) w.eid[rank[u]] = (int32_t)plen;
      R_src[rank[u]] = piece_anchor(roff[u], L[u], skip, orient != 0);
      s.lay_contig[st + i] = rank_c;  // every piece's, so in any order
    }
  }
  uint64_t carry = 0;
  if constexpr (kOneWave) {
    sej = __ballot(sej) != 0ull;
  } else {
    if (sej) s_sej = 1;
  }
  wbar();
  // 5. piece offsets in walk order
  if constexpr (kOneWave) {
    for (int base = 0; base < q; base += BLOCK) {
      const int i = base + tid;
      const uint32_t x = i < q ? (kLds ? (uint32_t)w.eid[i] : R_len[i]) : 0u;
      const uint32_t inc = wave_incl_scan(x);
      if (i < q) s.piece_off[st + i] = carry + (inc - x);
      carry += wave_lane(inc, kWave - 1);
    }
  } else {
    // (above the LDS form's sizes, a run of E pieces per thread)
    constexpr int E = kLds ? 1 : 4;
    for (int base = 0; base < q; base += E * BLOCK) {
      const int i = base + tid * E;
      uint32_t x[E];
      uint64_t sum = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        x[e] = i + e < q ? (kLds ? (uint32_t)w.eid[i + e] : R_len[i + e]) : 0u;
        sum += x[e];
      }
      uint64_t tot;
      uint64_t ex = carry + block_excl_scan<uint64_t, BLOCK, kLds>(sum, sh_scan, &tot);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (i + e < q) s.piece_off[st + i + e] = ex;
        ex += x[e];
      }
      carry += tot;
    }
  }
  if (tid == 0) {
    if constexpr (!kOneWave) sej = s_sej != 0;
    out.label[rank_c] = cr.label;
    out.bin[rank_c] = cr.bin;
    out.start[rank_c] = kLds ? w.vid[s0] : perm[st + s0];
    out.n_reads[rank_c] = q;
    out.len[rank_c] = carry;
    out.cflags[rank_c] = (q == 1 ? CG_CONTIG_SINGLE : 0u) | (cyc ? CG_CONTIG_CIRCULAR : 0u) |
                         (sej ? CG_CONTIG_SAME_END_JOIN : 0u);
    out.layout_off[rank_c] = st;
  }
  wbar();
}

// ---------------------------------------------------------------------------
// InducedSubgraph and LocalAssembly of one component of at most CAP reads in
// one pass, by a workgroup of BLOCK threads or one wave (BLOCK = kWave).  The
// caller has gathered each member's id v, kept bits kb (1: entry 0, 2: entry
// 1), A = (id, first column, second column, first entry), Bq = (length, overlap
// or pre of entry 0, of entry 1, strands of both), Cq = post of both and ro,
// where the read starts in the store.  The local numbers follow the ids; every
// field goes into the walk's LDS arrays at its local number while perm and the
// local CSR rows are written out, so the walk reads nothing back.
// ---------------------------------------------------------------------------
template <int BLOCK, int CAP>
__device__ __forceinline__ void iw_rows(const CompRec &cr, int q, int st, int32_t estart,
                                        const int32_t (&v)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        const uint32_t (&kb)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        const i32x4 (&A)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        const i32x4 (&Bq)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        const i32x2 (&Cq)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        const uint64_t (&ro)[CAP >= BLOCK ? CAP / BLOCK : 1],
                                        WalkArrays w, const cg_graph &g, const cg_local &local,
                                        const cg_contigs &out, const Scratch &s,
                                        uint64_t *sh_scan) {
  constexpr int R = CAP >= BLOCK ? CAP / BLOCK : 1;  // members per thread
  const int tid = BLOCK == kWave ? lane_id() : (int)threadIdx.x;
  auto bar = [] {
    if constexpr (BLOCK == kWave) wave_lds_sync();
    else lds_barrier();
  };
  // 1. local numbers: the ids in order in a (the walk's ray array, unused
  // until its rays), each member's rank among them
  int32_t *a = reinterpret_cast<int32_t *>(w.ray);
  int32_t rk[R];
  if constexpr (BLOCK == kWave) {
    // one wave: a rank is the number of smaller ids, counted over the lanes
#pragma unroll
    for (int u = 0; u < R; ++u) rk[u] = 0;
#pragma unroll
    for (int u2 = 0; u2 < R; ++u2) {
      const int cnt = q - u2 * kWave < kWave ? q - u2 * kWave : kWave;
      for (int l2 = 0; l2 < cnt; ++l2) {
        const int32_t x = __builtin_amdgcn_readlane(v[u2], l2);
#pragma unroll
        for (int u = 0; u < R; ++u) rk[u] += x < v[u] ? 1 : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (tid + u * BLOCK < q) a[rk[u]] = v[u];
    bar();
  } else {
    int N2 = 1;
    while (N2 < q) N2 <<= 1;
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = tid + u * BLOCK;
      if (i < N2) a[i] = i < q ? v[u] : 0x7FFFFFFF;
    }
    bar();
    // ids are non-negative and the padding is the largest int32, so their
    // order as uint32 is the same; the stages within 64 elements run in
    // registers (8 barriers for 512 ids instead of 45), and the barriers
    // order LDS only, so the gathers above stay in flight
    bitonic_sort<uint32_t, true>(reinterpret_cast<uint32_t *>(a), N2);
  }
  // the neighbours' local numbers (and a workgroup's members' own), searched
  // together
  int nr[2 * R];
  if constexpr (BLOCK == kWave) {
    int32_t x[2 * R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      x[2 * u] = (kb[u] & 1u) ? A[u].y : A[u].z;
      x[2 * u + 1] = A[u].z;
    }
    lds_lower_bounds<2 * R>(a, q, x, nr);
  } else {
    int32_t x[3 * R];
    int p[3 * R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      x[3 * u] = (kb[u] & 1u) ? A[u].y : A[u].z;
      x[3 * u + 1] = A[u].z;
      x[3 * u + 2] = v[u];
    }
    lds_lower_bounds<3 * R>(a, q, x, p);
#pragma unroll
    for (int u = 0; u < R; ++u) {
      nr[2 * u] = p[3 * u];
      nr[2 * u + 1] = p[3 * u + 1];
      rk[u] = p[3 * u + 2];
    }
  }
  // 2. every member's fields at its local number: its kept entries in row
  // order (slot 0, then slot 1), neighbours as local numbers
#pragma unroll
  for (int u = 0; u < R; ++u) {
    if (tid + u * BLOCK >= q) continue;
    const int r = rk[u];
    // slot 0: the first kept entry (entry 0, else entry 1); slot 1: entry 1
    // when both are kept (selects, no indexed arrays)
    const bool k0 = kb[u] & 1u, k1 = (kb[u] & 2u) != 0u;
    const bool s0 = k0 || k1, s1 = k0 && k1;
    const uint32_t sw = (uint32_t)Bq[u].w;
    const int32_t e0 = k0 ? A[u].w : A[u].w + 1;
    const uint32_t es0 = k0 ? (sw & 0xFFu) : ((sw >> 8) & 0xFFu);
    const uint32_t eo0 = (uint32_t)(k0 ? Bq[u].y : Bq[u].z);
    const uint32_t ep0 = (uint32_t)(k0 ? Cq[u].x : Cq[u].y);
    w.nb[2 * r] = s0 ? nr[2 * u] : -1;
    w.eid[2 * r] = s0 ? e0 : -1;
    w.es[2 * r] = (uint8_t)(s0 ? es0 : 0u);
    w.eo[2 * r] = s0 ? eo0 : 0u;
    w.ep[2 * r] = s0 ? ep0 : 0u;
    w.nb[2 * r + 1] = s1 ? nr[2 * u + 1] : -1;
    w.eid[2 * r + 1] = s1 ? A[u].w + 1 : -1;
    w.es[2 * r + 1] = (uint8_t)(s1 ? (sw >> 8) & 0xFFu : 0u);
    w.eo[2 * r + 1] = s1 ? (uint32_t)Bq[u].z : 0u;
    w.ep[2 * r + 1] = s1 ? (uint32_t)Cq[u].y : 0u;
    w.vid[r] = v[u];
    w.rlen[r] = (uint32_t)Bq[u].x;
    w.roff[r] = ro[u];
  }
  bar();
  // 3. perm and the local CSR rows, in local order
  CG_GLOBAL int32_t *perm = (CG_GLOBAL int32_t *)local.perm;
  CG_GLOBAL int32_t *lrp = (CG_GLOBAL int32_t *)local.loc_row_ptr;
  CG_GLOBAL int32_t *lcol = (CG_GLOBAL int32_t *)local.loc_col;
  CG_GLOBAL int32_t *leid = (CG_GLOBAL int32_t *)local.loc_eid;
  int32_t carry = 0;
  int first = 0x7FFFFFFF;  // the thread's first read with one neighbour
  for (int base = 0; base < q; base += BLOCK) {
    const int i = base + tid;
    int32_t n0 = -1, n1 = -1;
    if (i < q) {
      n0 = w.nb[2 * i];
      n1 = w.nb[2 * i + 1];
      if (n0 >= 0 && n1 < 0 && i < first) first = i;
    }
    const int32_t deg = (n0 >= 0 ? 1 : 0) + (n1 >= 0 ? 1 : 0);
    int32_t tot;
    const int32_t ex = block_excl_scan<int32_t, BLOCK, true>(deg, (int32_t *)sh_scan, &tot);
    if (i < q) {
      const int32_t r0 = estart + carry + ex;
      perm[st + i] = a[i];
      lrp[st + i] = r0;
      if (n0 >= 0) {
        lcol[r0] = st + n0;
        leid[r0] = w.eid[2 * i];
      }
      if (n1 >= 0) {
        lcol[r0 + 1] = st + n1;
        leid[r0 + 1] = w.eid[2 * i + 1];
      }
    }
    carry += tot;
  }
  walk_chain<BLOCK, CAP, kWalkLds>(cr, q, st, first, w, g, local.perm, out, s, sh_scan);
}

// cycles of rank below r; called by a whole wave with uniform r
__device__ __forceinline__ int32_t cycles_before(const CycMarks &m, int32_t r) {
  if (*m.any == 0) return 0;
  const int32_t sp = r / kCycSuper, w = r >> 5;
  int32_t k = 0;
  for (int32_t i = lane_id(); i < sp; i += kWave) k += (int32_t)m.super[i];
  for (int32_t i = sp * (kCycSuper / 32) + lane_id(); i < w; i += kWave) k += __popc(m.bits[i]);
  if (lane_id() == 0) k += __popc(m.bits[w] & ((1u << (r & 31)) - 1u));
  return wave_sum(k);
}

// One-read components: a lane each.
__device__ __forceinline__ void walk_single(const cg_graph &g, const cg_parts &parts, int c, int st,
                                            const cg_contigs &out, const Scratch &s) {
  const CompRec cr = comp_rec(parts, c);
  const int32_t v = cr.label;
  const uint32_t L = g.read_len[v];
  const uint64_t off = g.read_off[v];
  out.layout_vid[st] = v;
  out.layout_rev[st] = 0;
  s.piece_len[st] = L;
  s.piece_src[st] = piece_anchor(off, L, 0, false);
  s.piece_off[st] = 0;
  s.lay_contig[st] = cr.rank;
  out.label[cr.rank] = v;
  out.bin[cr.rank] = cr.bin;
  out.start[cr.rank] = v;
  out.n_reads[cr.rank] = 1;
  out.len[cr.rank] = L;
  out.cflags[cr.rank] = CG_CONTIG_SINGLE;
  out.layout_off[cr.rank] = st;
}

// ---------------------------------------------------------------------------
// Packed base copy
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t rev_fields32(uint32_t v) {
  const uint32_t y = __builtin_bitreverse32(v);
  return ((y >> 1) & 0x55555555u) | ((y & 0x55555555u) << 1);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One piece as the copy needs it.
struct PieceD {
  uint64_t a;     // piece_anchor without its strand bit
  uint64_t poff;  // first base of the piece in its contig
  uint64_t L;     // contig length
  uint64_t cb;    // first output word of the contig
  uint32_t plen;  // piece length
  int32_t rev;    // read walked reverse-complemented
};

// The per-piece arrays are read in piece order (coalesced across a wave's
// lanes); only the two per-contig arrays are gathered.  CB points to the
// contigs' first bases (global memory, or LDS).
template <typename CB>
struct PieceArraysT {
  const CG_GLOBAL int32_t *lay_contig;
  const CG_GLOBAL uint64_t *piece_off;
  const CG_GLOBAL uint32_t *piece_len;
  const CG_GLOBAL uint64_t *piece_src;
  const CG_GLOBAL uint64_t *clen;
  CB cbase;
};
typedef PieceArraysT<const CG_GLOBAL uint64_t *> PieceArrays;

__device__ __forceinline__ PieceArrays piece_arrays(const int32_t *lay_contig,
                                                    const uint64_t *piece_off,
                                                    const uint32_t *piece_len,
                                                    const uint64_t *piece_src,
                                                    const uint64_t *clen, const uint64_t *cbase) {
  return PieceArrays{(const CG_GLOBAL int32_t *)lay_contig, (const CG_GLOBAL uint64_t *)piece_off,
                     (const CG_GLOBAL uint32_t *)piece_len, (const CG_GLOBAL uint64_t *)piece_src,
                     (const CG_GLOBAL uint64_t *)clen,      (const CG_GLOBAL uint64_t *)cbase};
}

template <typename CB>
__device__ __forceinline__ PieceD load_piece(const PieceArraysT<CB> &A, int32_t p) {
  PieceD d;
  const int32_t k = A.lay_contig[p];
  const uint64_t a = A.piece_src[p];
  d.a = a & ~(1ull << 63);
  d.rev = (int32_t)(a >> 63);
  d.plen = A.piece_len[p];
  d.poff = A.piece_off[p];
  d.L = A.clen[k];
  d.cb = A.cbase[k] >> 4;
  return d;
}

// Store word index clamped into [0, nwords - 1]; a window may start before
// the store (reverse pieces of the first reads) or end after it, and the
// words it then reads are never used.
__device__ __forceinline__ uint64_t clamp_word(int64_t w, uint64_t nwords) {
  return w < 0 ? 0 : ((uint64_t)w >= nwords ? nwords - 1 : (uint64_t)w);
}

// 16 stored bases starting at base b (any alignment, b taken as signed) as
// one word: a 64-bit funnel shift of two store words.
__device__ __forceinline__ uint32_t window16(const CG_GLOBAL uint32_t *__restrict__ seq,
                                             uint64_t nwords, uint64_t b) {
  const int64_t w = (int64_t)b >> 4;
  const uint32_t lo = seq[clamp_word(w, nwords)];
  const uint32_t hi = seq[clamp_word(w + 1, nwords)];
  return __builtin_amdgcn_alignbit(hi, lo, 2u * (uint32_t)(b & 15));
}

// reverse the 16 2-bit fields of a word and complement them
__device__ __forceinline__ uint32_t revcomp16(uint32_t x) { return ~rev_fields32(x); }

__device__ __forceinline__ uint32_t low_fields(int k) {
  return k >= 16 ? 0xFFFFFFFFu : ((1u << (2 * k)) - 1u);
}

// Stored base where the 16-base window holding a piece's first 16 bases (in
// walking orientation) starts: forward at the piece's first base, reverse 15
// bases below it (the window is then read backwards).  a is the piece's
// anchor without its strand bit.
__device__ __forceinline__ uint64_t head_src(uint64_t a, bool rev) { return rev ? a - 16 : a; }

// The first k (<= 16) bases of a piece in walking orientation, in fields 0..k-1
// (fields above k are not cleared).
__device__ __forceinline__ uint32_t piece_head16(const CG_GLOBAL uint32_t *__restrict__ seq,
                                                 uint64_t nwords, const PieceD &f) {
  const uint32_t x = window16(seq, nwords, head_src(f.a, f.rev != 0));
  return f.rev ? revcomp16(x) : x;
}

// Copy descriptor of one piece: output words [w0, w0 + nw) of the bases
// array are the words whose first base lies in the piece.
//   sw0   store word at which the window of the piece's first group (output
//         word w0) starts; the group at word w0 + k starts at sw0 + k
//         (forward) or sw0 - k (reverse).  Signed: a reverse window may start
//         before the store.  Forward, output word w begins at stored base
//         16 sw0 + sh/2 + 16 (w - w0); reverse, the (16 kGroupWords)-base
//         window of the group at word w begins there with w0 - w in place of
//         w - w0.
//   info  bits 0-4: bases of the piece in its last owned word (1..16);
//         bit 5: reverse; bit 6: the piece ends its contig; bits 8-11: the
//         window's first base within its first store word (the funnel shift
//         is twice that)
struct CopyD {
  int64_t sw0;
  uint64_t w0;
  uint32_t nw, info;
};

// words per group: a lane's share of one row of a step
constexpr int kGroupWords = 4;
static_assert(kGroupWords % 4 == 0, "groups are moved in 16-byte units");
// What a word straddling into the next piece needs of it.
struct CopyE {
  uint64_t hsrc;   // head_src of the piece
  uint32_t info;   // plen | reverse << 30 | ends its contig << 31
};

__device__ __forceinline__ CopyD copy_desc(const PieceD &d) {
  CopyD c;
  const uint64_t pend = d.poff + d.plen;
  const uint64_t j0 = (d.poff + 15) >> 4, j1 = (pend + 15) >> 4;
  c.w0 = d.cb + j0;
  c.nw = (uint32_t)(j1 - j0);
  const uint32_t fs = (uint32_t)(pend - 16 * (j1 - 1));
  // stored base where the window of the first group begins (modulo 2^64)
  const uint64_t sb0 = d.rev ? d.a - 16 * kGroupWords + d.poff - 16 * j0 : d.a - d.poff + 16 * j0;
  c.sw0 = (int64_t)sb0 >> 4;
  c.info = fs | (d.rev ? 32u : 0u) | (pend == d.L ? 64u : 0u) | ((uint32_t)(sb0 & 15) << 8);
  return c;
}

__device__ __forceinline__ CopyE copy_next(const PieceD &e) {
  CopyE c;
  c.hsrc = head_src(e.a, e.rev != 0);
  c.info = e.plen | (e.rev ? (1u << 30) : 0u) | (e.poff + e.plen == e.L ? (1u << 31) : 0u);
  return c;
}

constexpr int kCopyUnroll = 2;  // groups per lane per step

// One step of the copy: kCopyUnroll groups per lane (groups g, g + 64, ...),
// their pieces' descriptors and store windows.
struct CopyStage {
  uint32_t win[kCopyUnroll][kGroupWords + 1];  // the last word only where the neighbouring
                                               // lane lacks it (nb)
  uint32_t hlo[kCopyUnroll], hhi[kCopyUnroll];  // store words of the next piece's head
  CopyD d[kCopyUnroll];
  CopyE e[kCopyUnroll];
  uint32_t k[kCopyUnroll];
  int t[kCopyUnroll];
  bool ok[kCopyUnroll];
  bool nb[kCopyUnroll];  // the last word is word 0 of the next group's window, held by
                         // lane l + 1 (forward) or l - 1 (reverse)
};


// Find the pieces of a step's groups and start its loads.
__device__ __forceinline__ void copy_fetch(CopyStage &S, uint32_t gb, uint32_t G, uint32_t gstart,
                                           const CopyD &my, const CopyE &nx,
                                           const CG_GLOBAL uint32_t *__restrict__ seq,
                                           uint64_t nwords, int lane) {
#pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) S.t[u] = 0;
  // piece of group g: the last lane t with gstart[t] <= g (gstart is
  // non-decreasing and equals G from lane cnt on, so t < cnt when g < G).
  // Six fixed steps, every lane shuffling in every step: a shuffle must
  // never run with part of the wave switched off.
#pragma unroll
  for (int step = kWave / 2; step > 0; step >>= 1) {
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
      const uint32_t g = gb + lane + kWave * u;
      const uint32_t sm = __shfl(gstart, S.t[u] + step);
      if (sm <= g) S.t[u] += step;
    }
  }
#pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) {
    const int t = S.t[u];
    S.d[u].sw0 = __shfl(my.sw0, t);
    S.d[u].w0 = __shfl(my.w0, t);
    S.d[u].nw = __shfl(my.nw, t);
    S.d[u].info = __shfl(my.info, t);
    S.e[u].hsrc = __shfl(nx.hsrc, t);
    S.e[u].info = __shfl(nx.info, t);
    const uint32_t gs = __shfl(gstart, t);
    const uint32_t g = gb + lane + kWave * u;
    S.ok[u] = g < G;
    S.k[u] = S.ok[u] ? kGroupWords * (g - gs) : 0;  // first owned word of the group
  }
  // loads only, so that nothing here waits for memory and the step's loads
  // stay in flight while the previous step is finished
#pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) {
    const CopyD &d = S.d[u];
    const bool rev = d.info & 32u;
    // the piece's window: kGroupWords + 1 store words covering the group's
    // bases, as 16-byte loads (dword aligned) and a dword; clamped word by
    // word at the ends of the store, where the words outside it are never used
    const int64_t sw = S.ok[u] ? (rev ? d.sw0 - (int64_t)S.k[u] : d.sw0 + (int64_t)S.k[u]) : 0;
    // the neighbouring lane's group is the next one of the same piece: its
    // window starts at the last word of this one
    // (both shifts by every lane, then the choice: a shift must never run
    // with part of the wave switched off)
    const uint32_t tk = (uint32_t)S.t[u] | (S.ok[u] ? 0x80000000u : 0u);
    const uint32_t tprev = wave_prev_u32(tk), tnext = wave_next_u32(tk);
    const uint32_t tnb = rev ? tprev : tnext;
    const int tn = (int)(tnb & 0x7FFFFFFFu);
    const bool okn = (tnb >> 31) != 0u;
    const bool edge = rev ? lane == 0 : lane == kWave - 1;
    S.nb[u] = false;
    if (sw >= 0 && sw + kGroupWords + 1 <= (int64_t)nwords) {
#pragma unroll
      for (int v = 0; v < kGroupWords / 4; ++v) {
        u32x4 a;
        __builtin_memcpy(&a, seq + sw + 4 * v, 16);
        S.win[u][4 * v] = a.x;
        S.win[u][4 * v + 1] = a.y;
        S.win[u][4 * v + 2] = a.z;
        S.win[u][4 * v + 3] = a.w;
      }
      S.nb[u] = S.ok[u] && okn && !edge && tn == S.t[u];
      S.win[u][kGroupWords] = S.nb[u] ? 0u : seq[sw + kGroupWords];
    } else {
#pragma unroll
      for (int i = 0; i <= kGroupWords; ++i) S.win[u][i] = seq[clamp_word(sw + i, nwords)];
    }
    // the next piece's first 16 bases, for the group holding the piece's
    // last word
    S.hlo[u] = S.hhi[u] = 0;
    if (S.ok[u] && S.k[u] + kGroupWords >= d.nw) {
      const int64_t hw = (int64_t)S.e[u].hsrc >> 4;
      S.hlo[u] = seq[clamp_word(hw, nwords)];
      S.hhi[u] = seq[clamp_word(hw + 1, nwords)];
    }
  }
}

// a 16-byte store, dword aligned
__device__ __forceinline__ void store_dwords4(CG_GLOBAL uint32_t *o, u32x4 x) {
  __builtin_memcpy(o, &x, 16);
}

// Finish a step: words from the windows, the pieces' last words, stores.
template <typename CB>
__device__ __forceinline__ void copy_emit(const CopyStage &S, const PieceArraysT<CB> &A, int32_t c0,
                                          int32_t n_e, const CG_GLOBAL uint32_t *__restrict__ seq,
                                          uint64_t nwords, CG_GLOBAL uint32_t *__restrict__ bases) {
#pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) {
    // the last window word from the neighbouring lane, while every lane is
    // still active
    const uint32_t up = wave_next_u32(S.win[u][0]), dn = wave_prev_u32(S.win[u][0]);
    if (!S.ok[u]) continue;
    const CopyD &d = S.d[u];
    const bool rev = d.info & 32u;
    uint32_t win[kGroupWords + 1];
#pragma unroll
    for (int i = 0; i < kGroupWords; ++i) win[i] = S.win[u][i];
    win[kGroupWords] = S.nb[u] ? (rev ? dn : up) : S.win[u][kGroupWords];
    const uint32_t sh = 2u * ((d.info >> 8) & 15u);
    const uint32_t nw = d.nw - S.k[u] < kGroupWords ? d.nw - S.k[u] : kGroupWords;
    uint32_t out[kGroupWords];
#pragma unroll
    for (int i = 0; i < kGroupWords; ++i)
      out[i] = rev ? revcomp16(__builtin_amdgcn_alignbit(win[kGroupWords - i],
                                                         win[kGroupWords - 1 - i], sh))
                   : __builtin_amdgcn_alignbit(win[i + 1], win[i], sh);
    const int fs = (int)(d.info & 31u);
    if (S.k[u] + nw == d.nw && fs < 16) {
      // the piece's last word: its own fs bases, then the next piece(s) or
      // zero padding at the contig's end
      uint32_t x = out[nw - 1] & low_fields(fs);
      if (!(d.info & 64u)) {
        const CopyE &e = S.e[u];
        const int pl = (int)(e.info & 0x3FFFFFFFu);
        const int k2 = 16 - fs < pl ? 16 - fs : pl;
        const bool erev = e.info & (1u << 30);
        uint32_t head =
            __builtin_amdgcn_alignbit(S.hhi[u], S.hlo[u], 2u * (uint32_t)(e.hsrc & 15));
        if (erev) head = revcomp16(head);
        x |= (head & low_fields(k2)) << (2 * fs);
        int filled = fs + k2;
        // pieces shorter than the rest of the word: take the following ones
        if (filled < 16 && !(e.info & (1u << 31))) {
          for (int32_t pp = c0 + S.t[u] + 2; filled < 16 && pp < n_e; ++pp) {
            const PieceD f = load_piece(A, pp);
            const int k3 = 16 - filled < (int)f.plen ? 16 - filled : (int)f.plen;
            const uint32_t y = piece_head16(seq, nwords, f);
            x |= (y & low_fields(k3)) << (2 * filled);
            filled += k3;
            if (f.poff + f.plen == f.L) break;
          }
        }
      }
      out[nw - 1] = x;
    }
    CG_GLOBAL uint32_t *o = bases + d.w0 + S.k[u];
    if (nw == kGroupWords) {
#pragma unroll
      for (int v = 0; v < kGroupWords / 4; ++v) {
        store_dwords4(o + 4 * v, u32x4{out[4 * v], out[4 * v + 1], out[4 * v + 2], out[4 * v + 3]});
      }
    } else {
#pragma unroll
      for (int i = 0; i < kGroupWords; ++i)
        if (i < (int)nw) o[i] = out[i];
    }
  }
}

// One wave copies the chunk of cnt (<= 64) consecutive pieces starting at
// piece c0 of a graph with n_e pieces.  Lane l gathers piece c0+l's
// descriptor; the chunk's kGroupWords-word groups (each owned by the piece holding
// the first base of its words) are then spread over the lanes, 64 groups per
// row, so lanes of one row work on different pieces.  Every word is a
// funnel shift of two store words, reverse-complemented in registers for a
// reverse piece; only a piece's last word can run into the next piece(s).
// Steps are software-pipelined: the loads of step s + 1 are issued before
// step s is finished, so a wave always has loads in flight.
// c0, cnt and n_e are wave-uniform; every lane runs every step.
template <typename CB>
__device__ __forceinline__ void copy_chunk(const uint32_t *seq_, uint64_t nwords, uint32_t *bases_,
                                           const PieceArraysT<CB> &A, int32_t c0, int cnt,
                                           int32_t n_e, int lane) {
  const CG_GLOBAL uint32_t *seq = (const CG_GLOBAL uint32_t *)seq_;
  CG_GLOBAL uint32_t *bases = (CG_GLOBAL uint32_t *)bases_;
  CopyD my{};
  uint32_t ng = 0;
  PieceD pd{};
  if (lane < cnt) {
    pd = load_piece(A, c0 + lane);
    my = copy_desc(pd);
    ng = (my.nw + kGroupWords - 1) / kGroupWords;
  }
  // the next piece of every lane's piece: from the next lane, or loaded for
  // the chunk's last piece
  CopyE nx;
  {
    const CopyE mine = copy_next(pd);
    nx.hsrc = __shfl_down(mine.hsrc, 1);
    nx.info = __shfl_down(mine.info, 1);
    if (lane == cnt - 1 && c0 + lane + 1 < n_e) nx = copy_next(load_piece(A, c0 + lane + 1));
  }
  const uint32_t gincl = wave_incl_scan(ng);
  const uint32_t gstart = gincl - ng;
  const uint32_t G = wave_lane(gincl, kWave - 1);
  constexpr uint32_t kStep = kWave * kCopyUnroll;
  CopyStage S0, S1;
  if (G > 0) copy_fetch(S0, 0, G, gstart, my, nx, seq, nwords, lane);
  for (uint32_t gb = 0; gb < G; gb += 2 * kStep) {
    if (gb + kStep < G) copy_fetch(S1, gb + kStep, G, gstart, my, nx, seq, nwords, lane);
    copy_emit(S0, A, c0, n_e, seq, nwords, bases);
    if (gb + kStep < G) {
      if (gb + 2 * kStep < G) copy_fetch(S0, gb + 2 * kStep, G, gstart, my, nx, seq, nwords, lane);
      copy_emit(S1, A, c0, n_e, seq, nwords, bases);
    }
  }
}

}  // namespace cg
