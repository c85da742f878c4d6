// InducedSubgraph and LocalAssembly of every component in one pass, for the
// whole path on one graph (the steps called one by one keep a pass each,
// k_induce.hip and k_assemble.hip).
//
// A component's work is a chain of dependent loads (its record, its members,
// their rows, the entries) and latency is what bounds it: the rows written by
// one pass were read back by the next, four more loads in a row (induce + walk
// 12.9 + 10.7 us on the 50 Mbp graph, 40 + 28 us on the 1 Gbp graph, 62 + 147
// us where 13 components hold up to 4,000 reads each; 19, 49 and 84 us now).
#include "cg_device.h"

namespace cg {

// Components by size: a lane for one read, a wave up to kWalkSmallCap reads, a
// workgroup above; everything in LDS up to kCompCap reads.  The LDS is what
// the waves of a workgroup need (two workgroups, 16 waves, to a compute unit).
constexpr int kCompBlock = 512;
constexpr int kCompWaves = kCompBlock / kWave;
constexpr int kCompCap = 512;
constexpr int kCompBytes = 58;  // LDS per read of the one-pass walk
constexpr int kCompWords = kCompWaves * kWalkSmallCap * kCompBytes / 4;
static_assert(kCompCap <= kCompWaves * kWalkSmallCap && kCompCap % kCompBlock == 0,
              "the workgroup's arrays fit the waves'");

// the walk's arrays of CAP reads in buf
template <int CAP>
__device__ __forceinline__ WalkArrays comp_arrays(uint32_t *buf) {
  WalkArrays w{};
  w.roff = reinterpret_cast<uint64_t *>(buf);
  w.nb = reinterpret_cast<int32_t *>(buf + 2 * CAP);
  w.eid = reinterpret_cast<int32_t *>(buf + 4 * CAP);
  w.ray = buf + 6 * CAP;
  w.eo = buf + 8 * CAP;
  w.ep = buf + 10 * CAP;
  w.vid = reinterpret_cast<int32_t *>(buf + 12 * CAP);
  w.rlen = buf + 13 * CAP;
  w.es = reinterpret_cast<uint8_t *>(buf + 14 * CAP);
  return w;
}

struct CompArgs {
  cg_graph g;
  const uint8_t *flags;
  cg_parts parts;
  const int32_t *mstart, *tmp;
  CycMarks cyc;
  cg_local local;
  cg_contigs out;
  Scratch s;
  const int32_t *list;  // the components above kWalkSmallCap reads, *n_listed of them
  const unsigned int *n_listed;
  int n_big;
};

// A component of at most CAP reads by a workgroup or (BLOCK = kWave) a wave:
// its members' fields in three rounds of loads issued together.
template <int BLOCK, int CAP>
__device__ __forceinline__ void comp_lds(const CompArgs &a, int c, int q, int st, int32_t es,
                                         int32_t ms, uint32_t *buf, uint64_t *sh_scan) {
  constexpr int R = CAP >= BLOCK ? CAP / BLOCK : 1;
  const int tid = BLOCK == kWave ? lane_id() : (int)threadIdx.x;
  const int32_t *mem = a.tmp + ms;
  const uint32_t *ov = a.g.pre ? a.g.pre : a.g.ovl;
  const bool coords = a.g.post != nullptr;
  int32_t v[R];
  uint32_t kb[R];
  i32x4 A[R], Bq[R];
  i32x2 Cq[R];
  uint64_t ro[R];
#pragma unroll
  for (int u = 0; u < R; ++u) v[u] = mem[tid + u * BLOCK < q ? tid + u * BLOCK : 0];
  const CompRec cr = comp_rec(a.parts, c);
#pragma unroll
  for (int u = 0; u < R; ++u) {
    kb[u] = ((uint32_t)a.flags[v[u]] >> 1) & 3u;
    A[u] = i32x4{v[u], -1, -1, a.g.row_ptr[v[u]]};
    Bq[u] = i32x4{(int32_t)a.g.read_len[v[u]], 0, 0, 0};
    Cq[u] = i32x2{0, 0};
    ro[u] = a.g.read_off[v[u]];
  }
#pragma unroll
  for (int u = 0; u < R; ++u) {
    if (tid + u * BLOCK >= q) {
      v[u] = 0x7FFFFFFF;
      continue;
    }
    const int32_t b = A[u].w;
    if (kb[u] & 1u) {
      A[u].y = a.g.col[b];
      Bq[u].y = (int32_t)ov[b];
      Bq[u].w = a.g.strand[b];
      if (coords) Cq[u].x = (int32_t)a.g.post[b];
    }
    if (kb[u] & 2u) {
      A[u].z = a.g.col[b + 1];
      Bq[u].z = (int32_t)ov[b + 1];
      Bq[u].w |= (int32_t)a.g.strand[b + 1] << 8;
      if (coords) Cq[u].y = (int32_t)a.g.post[b + 1];
    }
  }
  iw_rows<BLOCK, CAP>(cr, q, st, es, v, kb, A, Bq, Cq, ro, comp_arrays<CAP>(buf), a.g, a.local,
                      a.out, a.s, sh_scan);
}

// A component above kCompCap reads, with a bitmap of all read ids in LDS: its
// reads' ranks are the bits set below their own, so nothing is sorted (the
// bitonic sort of 4,096 ids and the scans of the rows took 62 us), and the
// rows need no scan (every read has two entries but for a path's two ends).
// The rays take the bitmap's place; before them, in LDS while there is room,
// the neighbours.
enum CompPlace { kAllLds, kRaysLds, kNoneLds };
__device__ __forceinline__ int64_t comp_bitmap(int32_t n) {
  const int64_t words = ((int64_t)n + 31) / 32;
  return 4 * words + 2 * words + 4;
}
// where a component of q reads keeps what, or -1: the bitmap does not fit
__device__ __forceinline__ int comp_place(int q, int32_t n) {
  const int64_t lds = 4 * (int64_t)kCompWords, bm = comp_bitmap(n), rays = 8 * (int64_t)q;
  if (bm > lds || q > 0xFFFF) return -1;  // (ranks are 16 bits)
  const bool small = q < 0x7FFF;          // and so are the ends of LDS rays
  if (small && rays + (bm > rays ? bm : rays) <= lds) return kAllLds;
  return small && rays <= lds ? kRaysLds : kNoneLds;
}
template <CompPlace kPlace>
__device__ __forceinline__ void comp_big(const CompArgs &a, int c, int q, int st, int32_t es,
                                         int32_t ms, uint32_t *buf, uint64_t *sh_scan) {
  __shared__ int32_t s_end[2];  // a path's ends, by id and then by rank
  __shared__ int s_ends;
  constexpr int U = 4;
  const int tid = (int)threadIdx.x;
  const int words = (a.g.n + 31) / 32;
  uint32_t *bits = kPlace == kAllLds ? buf + 2 * q : buf;
  uint16_t *pre = reinterpret_cast<uint16_t *>(bits + words);
  const int32_t *mem = a.tmp + ms;
  const CompRec cr = comp_rec(a.parts, c);
  if (tid == 0) {
    s_ends = 0;
    s_end[0] = s_end[1] = 0x7FFFFFFF;
  }
  for (int i = tid; i < words; i += kCompBlock) bits[i] = 0;
  __syncthreads();
  for (int b0 = tid; b0 < q; b0 += U * kCompBlock) {
    int32_t v[U];
    uint32_t f[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = b0 + u * kCompBlock < q ? mem[b0 + u * kCompBlock] : -1;
#pragma unroll
    for (int u = 0; u < U; ++u) f[u] = v[u] >= 0 ? a.flags[v[u]] : 6u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v[u] < 0) continue;
      atomicOr(bits + (v[u] >> 5), 1u << (v[u] & 31));
      if ((f[u] & 6u) != 6u) {
        const int k = atomicAdd(&s_ends, 1);
        if (k < 2) s_end[k] = v[u];
      }
    }
  }
  __syncthreads();
  {
    const int per = (words + kCompBlock - 1) / kCompBlock;
    const int w0 = tid * per, w1 = w0 + per < words ? w0 + per : words;
    uint32_t sum = 0, tot;
    for (int i = w0; i < w1; ++i) sum += (uint32_t)__popc(bits[i]);
    uint32_t ex = block_excl_scan<uint32_t, kCompBlock>(sum, reinterpret_cast<uint32_t *>(sh_scan),
                                                        &tot);
    for (int i = w0; i < w1; ++i) {
      pre[i] = (uint16_t)ex;
      ex += (uint32_t)__popc(bits[i]);
    }
  }
  __syncthreads();
  auto rank = [&](int32_t x) {
    return (int32_t)pre[x >> 5] + __popc(bits[x >> 5] & ((1u << (x & 31)) - 1u));
  };
  const int32_t e0 = s_end[0] != 0x7FFFFFFF ? rank(s_end[0]) : 0x7FFFFFFF;
  const int32_t e1 = s_end[1] != 0x7FFFFFFF ? rank(s_end[1]) : 0x7FFFFFFF;
  WalkArrays w = walk_scratch(a.s.walk, a.g.n, st, bits);
  if constexpr (kPlace == kAllLds) w.nb = reinterpret_cast<int32_t *>(buf);
  int first = 0x7FFFFFFF;
  for (int b0 = tid; b0 < q; b0 += U * kCompBlock) {
    int32_t v[U], b[U], c0[U], c1[U];
    uint32_t f[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = b0 + u * kCompBlock < q ? mem[b0 + u * kCompBlock] : -1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      f[u] = v[u] >= 0 ? a.flags[v[u]] : 0u;
      b[u] = v[u] >= 0 ? a.g.row_ptr[v[u]] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c0[u] = (f[u] & 2u) ? a.g.col[b[u]] : -1;
      c1[u] = (f[u] & 4u) ? a.g.col[b[u] + 1] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v[u] < 0) continue;
      const int32_t r = rank(v[u]);
      // slot 0: the first kept entry, slot 1: the second one
      const int32_t n0 = rank(c0[u] >= 0 ? c0[u] : (c1[u] >= 0 ? c1[u] : v[u]));
      const int32_t n1 = c0[u] >= 0 && c1[u] >= 0 ? rank(c1[u]) : -1;
      const int32_t d0 = c0[u] >= 0 ? b[u] : b[u] + 1;
      const bool any = c0[u] >= 0 || c1[u] >= 0;
      const int32_t t = es + 2 * r - (e0 < r ? 1 : 0) - (e1 < r ? 1 : 0);
      a.local.perm[st + r] = v[u];
      a.local.loc_row_ptr[st + r] = t;
      w.nb[2 * r] = any ? n0 : -1;
      w.nb[2 * r + 1] = n1;
      w.eid[2 * r] = any ? d0 : -1;
      w.eid[2 * r + 1] = n1 >= 0 ? b[u] + 1 : -1;
      if (any) {
        a.local.loc_col[t] = st + n0;
        a.local.loc_eid[t] = d0;
        if (n1 < 0 && r < first) first = r;
      }
      if (n1 >= 0) {
        a.local.loc_col[t + 1] = st + n1;
        a.local.loc_eid[t + 1] = b[u] + 1;
      }
    }
  }
  __syncthreads();
  walk_chain<kCompBlock, kCompBlock, kPlace == kNoneLds ? kWalkGlobal : kWalkRaysLds>(
      cr, q, st, first, w, a.g, a.local.perm, a.out, a.s, sh_scan);
}

// The others above kCompCap reads (of graphs above 316,000 reads): sorted in
// LDS or by a bitmap in windows, rows by scans, the walk's arrays in scratch
// (the rays in LDS up to kCompRays reads).
constexpr int kCompSortCap = 8192;
constexpr int kCompRays = 4096;
static_assert(kCompSortCap <= kCompWords && 2 * kCompRays <= kCompWords, "they fit the LDS");
__device__ __forceinline__ void comp_huge(const CompArgs &a, int c, int q, int st, int32_t es,
                                          int32_t ms, uint32_t *buf, uint64_t *sh_scan) {
  induce_component<kCompBlock, kCompSortCap>(
      q, st, es, a.tmp + ms, a.flags, a.g.row_ptr, a.g.col, a.local.perm, a.s.lidx,
      a.local.loc_row_ptr, a.local.loc_col, a.local.loc_eid, reinterpret_cast<int32_t *>(buf),
      reinterpret_cast<int32_t *>(sh_scan));
  // (the walk takes the entries after a component's last from its next row)
  if (threadIdx.x == 0)
    a.local.loc_row_ptr[st + q] = es + 2 * q - (a.parts.comp_kind[c] == CG_KIND_CYCLE ? 0 : 2);
  __syncthreads();
  const WalkArrays w = walk_scratch(a.s.walk, a.g.n, st, buf);
  if (q <= kCompRays)
    walk_component<kCompBlock, kCompRays, kWalkRaysLds>(
        c, q, st, w, a.g, a.parts, a.local.perm, a.local.loc_row_ptr, a.local.loc_col,
        a.local.loc_eid, a.out, a.s, sh_scan);
  else
    walk_component<kCompBlock, kCompRays, kWalkGlobal>(
        c, q, st, w, a.g, a.parts, a.local.perm, a.local.loc_row_ptr, a.local.loc_col,
        a.local.loc_eid, a.out, a.s, sh_scan);
}

// Workgroups 0 .. n_big - 1 take the listed components, those above
// kWalkSmallCap reads, so that the longest ones start first; the waves of the
// others take runs of consecutive components, neighbouring runs in different
// workgroups, so that a few components spread over the compute units.
__global__ __launch_bounds__(kCompBlock, 4) void k_comp(CompArgs a) {
  __shared__ alignas(16) uint32_t buf[kCompWords];
  __shared__ uint64_t sh_scan[kCompWaves + 1];
  const cg_parts &parts = a.parts;
  const int nc = *parts.d_n_comp;
  if ((int)blockIdx.x < a.n_big) {
    const int k = (int)*a.n_listed;
    for (int i = (int)blockIdx.x; i < k; i += a.n_big) {
      const int c = __builtin_amdgcn_readfirstlane(a.list[i]);
      const int q = parts.comp_size[c], st = parts.comp_start[c], r = parts.comp_rank[c];
      const int32_t ms = a.mstart[c];
      const int32_t es = 2 * (st - r + cycles_before(a.cyc, r));
      if (threadIdx.x == 0 && r == nc - 1) {
        const int32_t m_e = es + 2 * q - (parts.comp_kind[c] == CG_KIND_CYCLE ? 0 : 2);
        a.local.loc_row_ptr[st + q] = m_e;
        a.local.d_sizes[1] = m_e;
      }
      const int place = q <= kCompCap ? -1 : comp_place(q, a.g.n);
      if (q <= kCompCap) comp_lds<kCompBlock, kCompCap>(a, c, q, st, es, ms, buf, sh_scan);
      else if (place == kAllLds) comp_big<kAllLds>(a, c, q, st, es, ms, buf, sh_scan);
      else if (place == kRaysLds) comp_big<kRaysLds>(a, c, q, st, es, ms, buf, sh_scan);
      else if (place == kNoneLds) comp_big<kNoneLds>(a, c, q, st, es, ms, buf, sh_scan);
      else comp_huge(a, c, q, st, es, ms, buf, sh_scan);
      __syncthreads();
    }
    return;
  }
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  // workgroups with work: one wave per component, on every compute unit, or all
  int64_t nb = (nc + kCompWaves - 1) / kCompWaves;
  nb = nb < 256 ? 256 : nb;
  nb = nb < (int64_t)gridDim.x - a.n_big ? nb : (int64_t)gridDim.x - a.n_big;
  if ((int)blockIdx.x - a.n_big >= nb) return;
  const int64_t nw = nb * kCompWaves, w = wv * nb + (blockIdx.x - a.n_big);
  // components per wave: at most one each where the waves suffice
  int64_t run = (nc + nw - 1) / nw;
  if (run > kWave) run = kWave;
  for (int64_t c0 = w * run; c0 < nc; c0 += nw * run) {
    const int64_t c = c0 + lane_id();
    const bool live = lane_id() < run && c < nc;
    const int32_t q = live ? parts.comp_size[c] : 0;
    const int32_t st = live ? parts.comp_start[c] : 0, r = live ? parts.comp_rank[c] : 0;
    const int32_t ms = live ? a.mstart[c] : 0;
    int32_t es = 2 * (st - r);
    if (*a.cyc.any != 0)
      for (int t = 0; t < (int)run; ++t) {
        const int32_t k = cycles_before(a.cyc, __builtin_amdgcn_readlane(r, t));
        if (lane_id() == t) es += 2 * k;
      }
    if (live && q == 1) {
      a.local.perm[st] = parts.comp_label[c];
      a.local.loc_row_ptr[st] = es;
      walk_single(a.g, parts, (int)c, st, a.out, a.s);
    }
    if (live && r == nc - 1 && q <= kWalkSmallCap) {
      const int32_t m_e = es + 2 * q - (parts.comp_kind[c] == CG_KIND_CYCLE ? 0 : 2);
      a.local.loc_row_ptr[st + q] = m_e;
      a.local.d_sizes[1] = m_e;
    }
    for (uint64_t todo = __ballot(q > 1 && q <= kWalkSmallCap); todo; todo &= todo - 1) {
      const int t = (int)__builtin_ctzll(todo);
      const int tq = __builtin_amdgcn_readlane(q, t), tst = __builtin_amdgcn_readlane(st, t);
      const int32_t tes = __builtin_amdgcn_readlane(es, t), tms = __builtin_amdgcn_readlane(ms, t);
      uint32_t *mine = buf + wv * (kCompWords / kCompWaves);
      // one member per lane up to kWave reads, two above
      if (tq <= kWave) comp_lds<kWave, kWave>(a, (int)c0 + t, tq, tst, tes, tms, mine, sh_scan);
      else comp_lds<kWave, kWalkSmallCap>(a, (int)c0 + t, tq, tst, tes, tms, mine, sh_scan);
    }
  }
}

int launch_comp(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const PathArgs &a,
                const int32_t *mstart, hipStream_t st) {
  const PhaseRange range("cg: InducedSubgraph + LocalAssembly");
  const int32_t n = g.n;
  // workgroups for as many components above kWalkSmallCap reads as there can
  // be, and waves for components of two reads, up to two rounds of what is
  // resident at once
  const int n_big = n / (kWalkSmallCap + 1) < 512 ? n / (kWalkSmallCap + 1) : 512;
  const int64_t nw = ((int64_t)n / 2 + kCompWaves) / kCompWaves;
  const CompArgs ca{g, a.flags, a.parts, mstart, s.tmp, cyc_marks(s.estart, n), a.local, a.out, s,
                    s.memb, &ctx->fixed->n_listed, n_big};
  CG_LAUNCH(ctx, k_comp, dim3((unsigned)(n_big + (nw < 1024 ? nw : 1024))), dim3(kCompBlock), st,
            ca);
  return hip_check(hipGetLastError(), "k_comp");
}

}  // namespace cg
