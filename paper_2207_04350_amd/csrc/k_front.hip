// The first half of the whole path for a graph of few reads, in one workgroup
// and LDS: BranchRemoval (flags), ConnectedComponent (labels), the components'
// sizes, the reads' member slots and the eligible components in label order.
//
// Over the chip these are four launches whose time is launch and latency: a
// union's device-scope loads take about 1 us each where LDS takes 50 ns, and
// the counters' atomics likewise (2.9 + 7.8 + 7.5 + 4.4 us for 1,000 reads, 3.5
// + 11.9 + 9.7 + 5.0 us for 13,000).
#include "cg_device.h"

namespace cg {

constexpr int kFrontBlock = 1024;
// Reads at most.  One compute unit fetches about 10 GB/s of what it has not
// got, so the time grows by 1.7 us per 1,000 reads from 6 us, the passes over
// the chip by 0.7 us from 21 us: the lines meet at about 15,000 reads, and
// LDS holds the parents, counters, flags and a list of this many.
constexpr int kFrontReads = 12288;
constexpr int kFrontPer = 4;        // reads whose loads are issued together

bool front_fits(int32_t n) { return n > 0 && n <= kFrontReads; }

struct FrontArgs {
  int32_t n, min_reads;
  const int32_t *row_ptr, *col;
  uint8_t *flags;
  int32_t *d_counts, *label, *slot;
  cg_parts parts;
  MemberOut mo;
  int32_t *zero;
  unsigned long long *scan_status;
  int32_t zero_words, n_status;
  int reset;
};

__device__ __forceinline__ int32_t front_ld(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// The climb halves the path behind it: where reads are numbered along the
// genome every read's parent is the one before it, and climbs that leave the
// path as it was take as many steps as the component has reads (a sorted chain
// of 12,000 reads: 40.5 ms).  A halving store only ever puts an ancestor in
// the place of a parent, so it takes nothing from a union beside it.
__device__ __forceinline__ int32_t front_find(int32_t *par, int32_t x) {
  while (true) {
    const int32_t p = front_ld(par + x);
    if (p == x) return x;
    const int32_t gp = front_ld(par + p);
    if (gp == p) return p;
    __hip_atomic_store(par + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    x = gp;
  }
}
// a larger root goes under a smaller one, so every climb ends
__device__ __forceinline__ void front_union(int32_t *par, int32_t a, int32_t b) {
  a = front_find(par, a);
  b = front_find(par, b);
  while (a != b) {
    const int32_t hi = a > b ? a : b, lo = a > b ? b : a;
    const int32_t old = atomicCAS(par + hi, hi, lo);
    if (old == hi) return;
    a = old;
    b = lo;
  }
}

__global__ __launch_bounds__(kFrontBlock) void k_front(FrontArgs a) {
  // (the bases weights take its place: 64-bit sums of the components of more
  // than one read, half as many as reads at most)
  __shared__ alignas(16) int32_t s_par[kFrontReads];
  static_assert(kFrontReads % 2 == 0, "a 64-bit word per two reads");
  __shared__ int32_t s_cnt[kFrontReads];  // the edge a union is left for, then the counters
  __shared__ uint16_t s_list[kFrontReads];  // the reads with kept entries, in any order
  __shared__ uint8_t s_flag[kFrontReads];
  __shared__ int s_n;
  __shared__ unsigned long long sh[kFrontBlock / kWave + 1];
  __shared__ uint32_t s_large;
  const int tid = (int)threadIdx.x, n = a.n;
  if (tid == 0) s_n = 0;
  lds_barrier();
  // 1. flags, first parents and open edges
  uint32_t nb = 0, ml = 0;
  for (int r = 0; r < n; r += kFrontPer * kFrontBlock) {
    int32_t b[kFrontPer], deg[kFrontPer], u0[kFrontPer], u1[kFrontPer], d0[kFrontPer],
        d1[kFrontPer];
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      const int v = r + k * kFrontBlock + tid;
      b[k] = deg[k] = 0;
      if (v - tid >= n) continue;
      b[k] = v < n ? a.row_ptr[v] : 0;
      deg[k] = v < n ? a.row_ptr[v + 1] - b[k] : 0;
    }
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      u0[k] = deg[k] == 1 || deg[k] == 2 ? a.col[b[k]] : 0;
      u1[k] = deg[k] == 2 ? a.col[b[k] + 1] : 0;
    }
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      d0[k] = deg[k] == 1 || deg[k] == 2 ? a.row_ptr[u0[k] + 1] - a.row_ptr[u0[k]] : 3;
      d1[k] = deg[k] == 2 ? a.row_ptr[u1[k] + 1] - a.row_ptr[u1[k]] : 3;
    }
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      const int v = r + k * kFrontBlock + tid;
      if (v - tid >= n) continue;
      const uint32_t f = deg[k] >= 3 ? 1u : (d0[k] < 3 ? 2u : 0u) | (d1[k] < 3 ? 4u : 0u);
      const uint64_t kept = __ballot((f & 6u) != 0);
      int32_t at = 0;
      if (lane_id() == 0 && kept) at = atomicAdd(&s_n, __popcll(kept));
      at = __builtin_amdgcn_readfirstlane(at) + __popcll(kept & ((1ull << lane_id()) - 1ull));
      if (v >= n) continue;
      a.flags[v] = (uint8_t)f;
      s_flag[v] = (uint8_t)f;
      s_par[v] = first_parent(v, f, u0[k], u1[k]);
      if (f & 6u) {
        s_list[at] = (uint16_t)v;
        // both kept neighbours smaller: the larger one is left to a union
        const int32_t hi = u0[k] > u1[k] ? u0[k] : u1[k];
        s_cnt[v] = (f & 6u) == 6u && hi < v ? hi : -1;
      } else {
        s_cnt[v] = first_count(f);
        a.label[v] = v;
      }
      nb += f & 1u;
      ml += (f >> 1 & 1u) + (f >> 2 & 1u);
    }
  }
  // what starts at zero
  for (int i = tid; i < a.zero_words; i += kFrontBlock) a.zero[i] = 0;
  for (int i = tid; i < a.n_status; i += kFrontBlock) a.scan_status[i] = 0;
  if (tid == 0) {
    s_large = 0;
    if (a.reset) {
      a.mo.fx->mask_ticket = 0;
      a.mo.fx->status = 0;
      a.mo.fx->scan_ticket = 0;
      a.mo.fx->scan_done = 0;
    }
  }
  unsigned long long tot;
  (void)block_excl_scan<unsigned long long, kFrontBlock>((unsigned long long)ml << 32 | nb, sh, &tot);
  if (tid == 0) {
    a.d_counts[0] = (int32_t)(uint32_t)tot;
    a.d_counts[1] = (int32_t)(uint32_t)(tot >> 32);
  }
  // 2. unions (the scan's barriers lie between), then the counters
  const int n_list = s_n;
  for (int i = tid; i < n_list; i += kFrontBlock) {
    const int v = s_list[i];
    if (s_cnt[v] >= 0) front_union(s_par, v, s_cnt[v]);
    s_cnt[v] = 0;
  }
  lds_barrier();
  // 3. labels, counts and slots
  for (int i = tid; i < n_list; i += kFrontBlock) {
    const int v = s_list[i];
    const int32_t root = front_find(s_par, v);
    const uint32_t at = atomicAdd(reinterpret_cast<uint32_t *>(s_cnt) + root,
                                  (s_flag[v] & 6u) == 6u ? 4u : 5u);
    a.slot[v] = (int32_t)(at >> 2);
    a.label[v] = root;
  }
  __syncthreads();  // (the labels are read back below)
  // 4. the eligible components: a wave takes consecutive reads, 64 a round in
  // order, so that ballots and wave scans give the places within a wave's
  // reads; first its components, their reads and those of more than one read
  const int E = (n + kFrontBlock - 1) / kFrontBlock;
  const int w0 = __builtin_amdgcn_readfirstlane(tid / kWave) * E * kWave, l = lane_id();
  const uint64_t below = (1ull << l) - 1ull;
  unsigned long long x = 0;
  uint32_t y = 0, y_tot;
  for (int v = w0 + l; v < w0 + E * kWave; v += kWave) {
    const uint32_t c = v < n ? (uint32_t)s_cnt[v] : 0u;
    const bool el = c > 0 && eligible(s_flag[v < n ? v : 0], c >> 2, a.min_reads);
    x += el ? 1ull << 32 | c >> 2 : 0ull;
    y += el && c >> 2 > 1u ? 1u : 0u;
  }
  unsigned long long ex = block_excl_scan<unsigned long long, kFrontBlock>(x, sh, &tot);
  uint32_t multi = block_excl_scan<uint32_t, kFrontBlock>(y, reinterpret_cast<uint32_t *>(sh), &y_tot);
  // (the wave's first lane holds what lies before the wave)
  ex = wave_lane(ex, 0);
  multi = wave_lane(multi, 0);
  // (the parents are not needed any more)
  unsigned long long *w = reinterpret_cast<unsigned long long *>(s_par);  // bases by multi index
  if (a.mo.comp_w) {
    for (int i = tid; i < (int)y_tot; i += kFrontBlock) w[i] = 0;
    lds_barrier();
  }
  uint32_t at0 = (uint32_t)(ex >> 32), slot0 = (uint32_t)ex;
  for (int v = w0 + l; v < w0 + E * kWave; v += kWave) {
    const uint32_t c = v < n ? (uint32_t)s_cnt[v] : 0u;
    const uint32_t q = c >> 2;
    const bool el = c > 0 && eligible(s_flag[v < n ? v : 0], q, a.min_reads);
    const uint64_t em = __ballot(el);
    if (em) {
      const uint64_t mm = __ballot(el && q > 1u);
      const uint32_t reads = wave_incl_scan(el ? q : 0u);
      const uint32_t at = at0 + (uint32_t)__popcll(em & below);
      const uint32_t mu = multi + (uint32_t)__popcll(mm & below);
      if (el) {
        a.parts.comp_label[at] = v;
        a.parts.comp_size[at] = (int32_t)q;
        a.parts.comp_kind[at] = q == 1 ? CG_KIND_SINGLE : ((c & 3u) ? CG_KIND_PATH : CG_KIND_CYCLE);
        a.mo.start[at] = (int32_t)(slot0 + reads - q);
        if (q > (uint32_t)kWalkSmallCap) a.mo.list[atomicAdd(&s_large, 1u)] = (int32_t)at;
        if (a.mo.keys) {
          const uint64_t key = (uint64_t)(0xFFFFFFFFu - q) << 32 | at;
          if (q > 1) a.mo.keys[mu] = key;
          else a.mo.keys[(int64_t)n + (at - mu)] = key;
        }
        if (a.mo.comp_w && q == 1) a.mo.comp_w[at] = a.mo.read_len[v];
      }
      if (v < n) {
        a.parts.label_comp[v] = el ? (int32_t)at : -1;
        // with bases weights: a root's multi index, for its reads below
        s_cnt[v] = el && q > 1 ? (int32_t)mu : -1;
      }
      at0 += (uint32_t)__popcll(em);
      multi += (uint32_t)__popcll(mm);
      slot0 += wave_lane(reads, kWave - 1);
    } else if (v < n) {
      a.parts.label_comp[v] = -1;
      s_cnt[v] = -1;
    }
  }
  if (a.mo.comp_w) {
    lds_barrier();
    for (int i = tid; i < n_list; i += kFrontBlock) {
      const int v = s_list[i];
      const int32_t m = s_cnt[a.label[v]];
      if (m >= 0) atomicAdd(w + m, (unsigned long long)a.mo.read_len[v]);
    }
    lds_barrier();
    for (int v = w0 + l; v < w0 + E * kWave; v += kWave)  // (this thread's own label_comp)
      if (v < n && s_cnt[v] >= 0) a.mo.comp_w[a.parts.label_comp[v]] = w[s_cnt[v]];
  }
  __syncthreads();
  if (tid == 0) {
    *a.parts.d_n_comp = (int32_t)(uint32_t)(tot >> 32);
    a.mo.fx->n_listed = s_large;
    a.mo.fx->n_multi = y_tot;
  }
}

int launch_front(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const PathArgs &a,
                 const MemberOut &mo, hipStream_t st) {
  const PhaseRange range("cg: BranchRemoval + ConnectedComponent");
  const FrontArgs fa{g.n, a.min_reads < 1 ? 1 : a.min_reads, g.row_ptr, g.col, a.flags, a.d_counts,
                     a.label, s.lidx, a.parts, mo, s.estart, s.scan_status, cyc_words(g.n),
                     scan_blocks((int64_t)g.n + 1) + 1, a.reset ? 1 : 0};
  CG_LAUNCH(ctx, k_front, dim3(1), dim3(kFrontBlock), st, fa);
  return hip_check(hipGetLastError(), "k_front");
}

}  // namespace cg
