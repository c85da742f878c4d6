// InducedSubgraph (Section 4.3): V_i = reads owned by bin i, E_i = entries of
// L with both ends in V_i, renumbered locally with the global ids kept.  All
// bins share one local numbering ordered by (bin, label, id): a component's
// reads form the block [comp_start, comp_start + q), and its local CSR rows
// the entries from comp_estart on, so one component's part of every output is
// independent of the others'.  As a step of its own (the whole path's
// partition step fills the slots, k_partition.hip, and its component pass
// does the rest, k_components.hip):
//
//  k_ind_init   bucket cursors, components by rank, the cycle marks cleared
//  k_ind_fill   each read with kept entries claims a slot in its component's
//               block; bin_vptr and n_e from the components in rank order;
//               cycles marked by rank
//  k_ind_comp   sorts each component's reads by id and writes perm and the
//               local CSR rows: lanes for one-read components, a wave up to
//               128 reads, a workgroup above
//
// The entries before a component need no scan of the rows: a path of q reads
// has 2q - 2 of them and a cycle 2q, so they are 2 (comp_start - comp_rank),
// plus two for every cycle of lower rank.
#include "cg_device.h"

namespace cg {

constexpr int kIndInitBlock = 256;
__global__ __launch_bounds__(kIndInitBlock) void k_ind_init(
    int32_t n, int32_t P, const int32_t *__restrict__ d_n_comp,
    const int32_t *__restrict__ comp_rank, uint32_t *__restrict__ fill,
    int32_t *__restrict__ by_rank, CycMarks cyc, int32_t *__restrict__ bin_vptr,
    int32_t *__restrict__ loc_row_ptr, int32_t *__restrict__ d_sizes) {
  const int32_t nc = *d_n_comp;
  const int64_t t0 = (int64_t)blockIdx.x * kIndInitBlock + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * kIndInitBlock;
  for (int64_t c = t0; c < nc; c += nt) {
    fill[c] = 0;
    by_rank[comp_rank[c]] = (int32_t)c;
  }
  for (int64_t w = t0; w < (nc + 31) / 32; w += nt) cyc.bits[w] = 0;
  for (int64_t w = t0; w < (nc + kCycSuper - 1) / kCycSuper; w += nt) cyc.super[w] = 0;
  if (t0 == 0 && n > 0) *cyc.any = 0;
  if (nc == 0) {
    for (int64_t b = t0; b <= P; b += nt) bin_vptr[b] = 0;
    if (t0 == 0) {
      loc_row_ptr[0] = 0;
      d_sizes[0] = d_sizes[1] = 0;
    }
  }
}

// The slots of a workgroup's reads are counted per component in an LDS hash
// table first, so that the workgroup takes one slot range per component: one
// atomic per read on the component's cursor queues on its address (about
// 4.5 ns each: 69 us for the 15,000 reads of 13 components, 10 us now; 13 to
// 11 us where 556 components share them).
constexpr int kFillBlock = 1024;
constexpr int kFillPer = 2;                           // reads per thread
constexpr int kFillSlots = 2 * kFillBlock * kFillPer;  // at most half full
__global__ __launch_bounds__(kFillBlock) void k_ind_fill(
    int32_t n, int32_t P, const uint8_t *__restrict__ flags, const int32_t *__restrict__ label,
    cg_parts parts, uint32_t *fill, const int32_t *__restrict__ by_rank, CycMarks cyc,
    int32_t *__restrict__ tmp, int32_t *__restrict__ bin_vptr, int32_t *__restrict__ d_sizes) {
  __shared__ int32_t s_key[kFillSlots];
  __shared__ uint32_t s_cnt[kFillSlots];
  const int32_t nc = *parts.d_n_comp;
  const int64_t t0 = (int64_t)blockIdx.x * kFillBlock + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * kFillBlock;
  // the reads' flags and labels, and their components (-1: none, or a read
  // of a one-read component, which needs no slot)
  int32_t v[kFillPer], c[kFillPer], lab[kFillPer];
  bool in[kFillPer];
#pragma unroll
  for (int k = 0; k < kFillPer; ++k) {
    const int64_t x = ((int64_t)blockIdx.x * kFillPer + k) * kFillBlock + threadIdx.x;
    v[k] = (int32_t)x;
    in[k] = x < n && (flags[x] & 6u);
    lab[k] = in[k] ? label[x] : 0;
  }
  for (int i = threadIdx.x; i < kFillSlots; i += kFillBlock) {
    s_key[i] = -1;
    s_cnt[i] = 0;
  }
#pragma unroll
  for (int k = 0; k < kFillPer; ++k) c[k] = in[k] ? parts.label_comp[lab[k]] : -1;
  // components in rank order: where the bins start
  for (int64_t r = t0; r < nc; r += nt) {
    const int32_t x = by_rank[r], prev = r > 0 ? parts.comp_bin[by_rank[r - 1]] : -1;
    const int32_t st = parts.comp_start[x];
    for (int32_t b = prev + 1; b <= parts.comp_bin[x]; ++b) bin_vptr[b] = st;
    if (parts.comp_kind[x] == CG_KIND_CYCLE) mark_cycle(cyc, (int32_t)r);
  }
  if (nc > 0) {
    const int32_t x = by_rank[nc - 1];
    const int32_t n_e = parts.comp_start[x] + parts.comp_size[x];
    for (int64_t b = (int64_t)parts.comp_bin[x] + 1 + t0; b <= P; b += nt) bin_vptr[b] = n_e;
    if (t0 == 0) d_sizes[0] = n_e;
  }
  __syncthreads();
  int slot[kFillPer];
  uint32_t at[kFillPer];
#pragma unroll
  for (int k = 0; k < kFillPer; ++k) {
    slot[k] = -1;
    if (c[k] < 0) continue;
    uint32_t h = ((uint32_t)c[k] * 2654435761u) >> 16 & (kFillSlots - 1);
    while (true) {  // ends: the table is at most half full
      const int32_t old = atomicCAS(s_key + h, -1, c[k]);
      if (old == -1 || old == c[k]) break;
      h = (h + 1) & (kFillSlots - 1);
    }
    slot[k] = (int)h;
    at[k] = atomicAdd(s_cnt + h, 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kFillSlots; i += kFillBlock) {
    const int32_t x = s_key[i];
    if (x >= 0) s_cnt[i] = (uint32_t)parts.comp_start[x] + atomicAdd(fill + x, s_cnt[i]);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kFillPer; ++k)
    if (slot[k] >= 0) tmp[s_cnt[slot[k]] + at[k]] = v[k];
}

// One component of 2 .. kIndWaveCap reads by one wave.  The ranks of the ids
// are counted over the lanes; every member's kept columns go to LDS at its
// rank, then lane i writes local read i.  s points at 4 * kIndWaveCap ints of
// the wave's own.
constexpr int kIndWaveCap = 128;
__device__ __forceinline__ void ind_wave(int q, int st, int estart, const int32_t *members,
                                         const uint8_t *__restrict__ flags,
                                         const int32_t *__restrict__ row_ptr,
                                         const int32_t *__restrict__ col, int32_t *s,
                                         const cg_local &out) {
  constexpr int R = kIndWaveCap / kWave;
  const int l = lane_id();
  int32_t *s_id = s, *s_b = s + kIndWaveCap, *s_c0 = s + 2 * kIndWaveCap,
          *s_c1 = s + 3 * kIndWaveCap;
  int32_t v[R], b[R], c0[R], c1[R], rk[R];
  uint32_t f[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int i = l + u * kWave;
    v[u] = i < q ? members[i] : 0x7FFFFFFF;
  }
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const bool live = l + u * kWave < q;
    f[u] = live ? flags[v[u]] : 0u;
    b[u] = live ? row_ptr[v[u]] : 0;
    rk[u] = 0;
  }
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
  for (int u = 0; u < R; ++u) {
    c0[u] = (f[u] & 2u) ? col[b[u]] : -1;
    c1[u] = (f[u] & 4u) ? col[b[u] + 1] : -1;
  }
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (l + u * kWave < q) {
      s_id[rk[u]] = v[u];
      s_b[rk[u]] = b[u];
      s_c0[rk[u]] = c0[u];
      s_c1[rk[u]] = c1[u];
    }
  wave_lds_sync();
  int32_t r0 = estart;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int i = l + u * kWave;
    const bool live = i < q;
    const int32_t x0 = live ? s_c0[i] : -1, x1 = live ? s_c1[i] : -1;
    const int32_t deg = (x0 >= 0 ? 1 : 0) + (x1 >= 0 ? 1 : 0);
    const int32_t inc = wave_incl_scan(deg);
    int32_t t = r0 + inc - deg;
    if (live) {
      out.perm[st + i] = s_id[i];
      out.loc_row_ptr[st + i] = t;
      const int32_t e = s_b[i];
      if (x0 >= 0) {
        out.loc_col[t] = st + lower_bound_i32(s_id, q, x0);
        out.loc_eid[t] = e;
        ++t;
      }
      if (x1 >= 0) {
        out.loc_col[t] = st + lower_bound_i32(s_id, q, x1);
        out.loc_eid[t] = e + 1;
      }
    }
    r0 += wave_lane(inc, kWave - 1);
  }
  wave_lds_sync();
}

// Workgroups 0 .. n_big - 1 take the components above kIndWaveCap reads (the
// longest ones start first); the waves of the others take runs of consecutive
// components, one-read components a lane each.  1024 threads and at most
// 64 registers: two workgroups, all 32 waves of a compute unit, and LDS for
// the sort of 16,384 reads.
constexpr int kIndCompBlock = 1024;
constexpr int kIndCompCap = 16384;
constexpr int kIndCompWaves = kIndCompBlock / kWave;
static_assert(kIndCompWaves * 4 * kIndWaveCap <= kIndCompCap, "the waves' LDS fits the sort's");
__global__ __launch_bounds__(kIndCompBlock, 8) void k_ind_comp(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const uint8_t *__restrict__ flags, cg_parts parts, const int32_t *__restrict__ tmp,
    int32_t *__restrict__ lidx, CycMarks cyc, cg_local out, int n_big) {
  __shared__ int32_t a[kIndCompCap];
  __shared__ int32_t sh_scan[kIndCompBlock / kWave + 1];
  __shared__ int s_n;
  __shared__ int32_t s_list[kIndCompBlock];
  const int32_t nc = *parts.d_n_comp;
  if ((int)blockIdx.x < n_big) {
    // this workgroup's components: blockIdx.x, + n_big, + 2 n_big, ...
    for (int64_t base = blockIdx.x; base < nc; base += (int64_t)n_big * kIndCompBlock) {
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      const int64_t c = base + (int64_t)n_big * threadIdx.x;
      if (c < nc && parts.comp_size[c] > kIndWaveCap) s_list[atomicAdd(&s_n, 1)] = (int32_t)c;
      __syncthreads();
      const int k = s_n;
      for (int i = 0; i < k; ++i) {
        const int32_t x = s_list[i];
        const int32_t q = parts.comp_size[x], st = parts.comp_start[x], r = parts.comp_rank[x];
        const int32_t es = 2 * (st - r + cycles_before(cyc, r));
        induce_component<kIndCompBlock, kIndCompCap>(q, st, es, tmp + st, flags, row_ptr, col,
                                                     out.perm, lidx, out.loc_row_ptr, out.loc_col,
                                                     out.loc_eid, a, sh_scan);
        if (threadIdx.x == 0 && r == nc - 1) {
          const int32_t m_e = es + 2 * q - (parts.comp_kind[x] == CG_KIND_CYCLE ? 0 : 2);
          out.loc_row_ptr[st + q] = m_e;
          out.d_sizes[1] = m_e;
        }
      }
      __syncthreads();
    }
    return;
  }
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int64_t w = (int64_t)(blockIdx.x - n_big) * kIndCompWaves + wv;
  const int64_t nw = (int64_t)(gridDim.x - n_big) * kIndCompWaves;
  // components per wave: at most one each where the waves suffice
  int64_t run = (nc + nw - 1) / nw;
  if (run > kWave) run = kWave;
  for (int64_t c0 = w * run; c0 < nc; c0 += nw * run) {
    const int64_t c = c0 + lane_id();
    const bool live = lane_id() < run && c < nc;
    const int32_t q = live ? parts.comp_size[c] : 0;
    const int32_t st = live ? parts.comp_start[c] : 0, r = live ? parts.comp_rank[c] : 0;
    const int32_t lab = live ? parts.comp_label[c] : 0;
    const bool cycles = *cyc.any != 0;
    int32_t es = 2 * (st - r);
    if (cycles)
      for (int t = 0; t < (int)run; ++t) {
        const int32_t k = cycles_before(cyc, __builtin_amdgcn_readlane(r, t));
        if (lane_id() == t) es += 2 * k;
      }
    if (live && q == 1) {
      out.perm[st] = lab;
      out.loc_row_ptr[st] = es;
    }
    if (live && r == nc - 1 && q <= kIndWaveCap) {
      const int32_t m_e = es + 2 * q - (parts.comp_kind[c] == CG_KIND_CYCLE ? 0 : 2);
      out.loc_row_ptr[st + q] = m_e;
      out.d_sizes[1] = m_e;
    }
    for (uint64_t todo = __ballot(q > 1 && q <= kIndWaveCap); todo; todo &= todo - 1) {
      const int t = (int)__builtin_ctzll(todo);
      const int tq = __builtin_amdgcn_readlane(q, t), tst = __builtin_amdgcn_readlane(st, t);
      ind_wave(tq, tst, __builtin_amdgcn_readlane(es, t), tmp + tst, flags, row_ptr, col,
               a + wv * 4 * kIndWaveCap, out);
    }
  }
}

int launch_induce(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const uint8_t *flags,
                  const int32_t *label, const cg_parts &parts, int32_t P, const cg_local &out,
                  hipStream_t st) {
  const PhaseRange range("cg: InducedSubgraph");
  const int32_t n = g.n;
  const CycMarks cyc = cyc_marks(s.estart, n);
  const int64_t zg = ((int64_t)n + kIndInitBlock - 1) / kIndInitBlock;
  CG_LAUNCH(ctx, k_ind_init, dim3((unsigned)(zg < 1 ? 1 : (zg > 256 ? 256 : zg))),
            dim3(kIndInitBlock), st, n, P, parts.d_n_comp, parts.comp_rank, s.fill, s.aux, cyc,
            out.bin_vptr, out.loc_row_ptr, out.d_sizes);
  if (n > 0) {
    const int64_t per = (int64_t)kFillBlock * kFillPer;
    CG_LAUNCH(ctx, k_ind_fill, dim3((unsigned)((n + per - 1) / per)), dim3(kFillBlock), st, n, P,
              flags, label, parts, s.fill, s.aux, cyc, s.tmp, out.bin_vptr, out.d_sizes);
    // workgroups: as many as can hold a component above kIndWaveCap reads,
    // up to one per compute unit; waves for components of two reads, up to
    // what is resident at once
    const int n_big = n / (kIndWaveCap + 1) < 256 ? n / (kIndWaveCap + 1) : 256;
    const int64_t nw = ((int64_t)n / 2 + kIndCompWaves) / kIndCompWaves;
    CG_LAUNCH(ctx, k_ind_comp, dim3((unsigned)(n_big + (nw < 512 ? nw : 512))),
              dim3(kIndCompBlock), st, g.row_ptr, g.col, flags, parts, s.tmp, s.lidx, cyc, out,
              n_big);
  }
  return hip_check(hipGetLastError(), "k_ind");
}

}  // namespace cg
