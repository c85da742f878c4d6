// The step before the path (Algorithm 1: Prune(IsContainedRead), then
// TransitiveReduction; Section 2 defines redundant vertices and redundant
// edges) on an overlap graph R given like a string graph:
//
//  k_red_contained  a read is contained when an entry covers all of it
//                   (ovl >= len) from a longer read, or an equally long one
//                   with a smaller id; a contained read's entries are dropped
//  k_red_near       the entries of a row that lead to reads that are not
//                   contained, with overlap, strands, place in the row and the
//                   read's length, side by side (rows up to kRedCap entries,
//                   while the scratch has room; none at all where the rows are
//                   short and most reads stay, see red_crowded)
//  k_red_trans      row u's near neighbours v in LDS with, for each, where v's
//                   near entries start and how many there are; the lanes
//                   then take the (v, v->x) pairs of all neighbours together
//                   and look each x up among u's: entry u->x is marked
//                   transitive when u, v, x is a valid walk with u->x's end
//                   orientations and overhangs that add up to u->x's.  A row
//                   that k_red_near left out is read in full; a longer one is
//                   read in place, one neighbour at a time.
//  k_red_keep       an entry stays when neither read is contained and
//                   neither it nor its twin is marked; entries kept per row
//                   and per block of rows
//  k_red_compact    row pointers of the string graph (each workgroup adds up
//                   the blocks before its own) and the kept entries in R's
//                   column order
//
// Where read lengths spread, most reads are contained (88% at 30x, 12 +- 4
// kbp), and these rows are done after the first pass.  A workgroup of the later
// passes takes a block of up to 64 rows and its waves only those that are not
// contained, a wave each, so that the resident waves all have a row to work on:
// with a wave per row, contained or not, four rows to a workgroup, two thirds of
// a workgroup's waves had left while its LDS stayed taken.  One pass moves a
// row's dependent loads (row, neighbour, neighbour's row, overlap) one after
// another, so resident waves are what bounds it.  At 30x a read that is not
// contained has 70 entries, 11 of them to others like it: the near entries
// leave 1.8 M pairs of 11.5 M (50 Mbp: k_red_near 15 and k_red_trans 26 us;
// 97 us on whole rows, 224 us with a wave per row besides).
//
// kept[e] starts with whether the entry's read is contained in bit 2 (k_red_near
// for the rows with near entries and those above kRedCap, k_red_trans for those
// that it reads in full), carries the mark in bit 0 (k_red_trans), the decision in
// bit 1 (k_red_keep), and ends as 0 / 1 (k_red_compact).
//
// The overhang test: sfx(x->y) = len(y) - ovl(x->y), and
// sfx(u->v) + sfx(v->x) - sfx(u->x) = len(v) - ovl(u->v) - ovl(v->x) + ovl(u->x)
// (len(x) cancels), so x's length is never read.
#include "cg_device.h"

namespace cg {

constexpr int kRedWaves = 4;
constexpr int kRedBlock = kRedWaves * kWave;
constexpr int kRedCap = 256;   // row entries k_red_trans holds in registers
constexpr int kRedPer = kRedCap / kWave;
// Neighbours not contained that k_red_trans holds in LDS: 11 or 22 KB a
// workgroup, which is resident waves (100 Mbp at 15x, rows of 28 entries: 551 us
// with room for 128, 777 for 256).  More than 128 they are where the rows have
// well above 128 entries and most reads stay (reads of one length at 70x to
// 120x: 1.1 to 5.3 ms with room for 256, 2.5 to 14 with the rows read in place).
// From kRedWideRow entries a read on a sample of the rows tells them (red_wide),
// and the instance that is not wanted leaves, 2-3 us (10 Mbp at 60x of 12 +- 4
// kbp 69 us, 72 with the wide one, 66 with the narrow one alone; 1 Mbp at 90x of
// 12 +- 0.3 kbp, 74 near neighbours a row, 399, 530 and 379; 2 Mbp at 60x of one
// length, 110 of them, 768, 765 and 1,058).  (Where the entries are twice kRedCap
// and more, nearly every row is read in place, and the room serves none: 618 us
// with 128, 635 with 256.)
constexpr int kRedNear = 128, kRedNearWide = 256;
constexpr int kRedWideRow = 96;       // entries per read
constexpr uint32_t kRedWideNear = 96;  // near neighbours per row from which it is kRedNearWide
static_assert(kRedNearWide == kRedCap, "no row that fits the registers is read in place");
constexpr int kRedRows = 64;     // rows per workgroup at most: a lane of a wave each
constexpr int kRedShards = 64;   // parts of the near entries' memory at most, a cursor each
// words between the cursors: atomics on one line queue up (about 4.5 ns each:
// 79 us for 15,000 of them on adjacent cursors)
constexpr int kRedCursor = 64;
constexpr int kRedList = 256;    // surviving entries a wave of k_red_keep collects
constexpr int kRedDirect = 4096;  // blocks whose counts each workgroup of k_red_compact adds up itself
// Lanes per row of k_red_contained: 16, or a wave where the rows are long.
constexpr int kRedGroup = 16;
constexpr int kRedWaveRow = 256;  // entries per read from which it is a wave
// A read's near entries from which filling their room does not pay, where the
// rows are short; with longer ones the pairs saved outweigh the pass (10 Mbp at
// 45x, 30 near entries a read: 20 us of it save 34, at 10x, 14 of them: 4 save 2)
constexpr uint32_t kRedCrowd = 8;
constexpr int kRedShortRow = 40;  // entries per read
// the sample's words: rows that stay times this, plus their entries
constexpr uint32_t kRedStay = 1u << 20;
static_assert(2 * kWave * (kWave / kRedGroup) * kRedCap < (int)kRedStay &&
              2 * kWave * (kWave / kRedGroup) < 1 << 12, "the sample's sums fit a word");

// Rows per workgroup: kRedRows, or fewer where that leaves the chip's 256
// compute units short of workgroups, at least one per wave.
static int red_rows(int32_t n, int blocks) {
  int R = kRedRows;
  while (R > kRedWaves && n / R < blocks) R >>= 1;
  return R;
}
constexpr int kRedBlocks = 1024;
// k_red_trans, whose rows take unequal time, wants more of them (8,333 reads of
// about one length at 10x: 26 us instead of 37; 50 Mbp at 30x 38.8 and 40.5,
// with 4,096 39.3, 17 Mbp 24.0 and 27.7; 2 Mbp at 100x of 12 +- 0.3 kbp 803 and
// 1,158), and its wide instance more still (2 Mbp at 100x: 4.00 ms with 1,024 and
// 2,048, 3.01 with 3,072; 10 Mbp at 60x of one length 1.04 and 1.00 ms, 1.05 with
// 4,096); not so where nearly every row is read in place (0.3 Mbp at 600x: 1.87 ms
// with 1,024, 2.00 with 2,048).
constexpr int kRedTransBlocks = 2048, kRedWideBlocks = 3072;

// 16 lanes per row, or 64 for long rows, four entries each in flight: a row has
// 55 entries on average at 30x.  Only an entry that covers the read (ovl >= len) needs its
// column and that read's length.  6.9 M entries: 21 us (28 us with a wave per
// row and every column loaded); rows of 590 and 1,200 entries: 6.9 and 16.9 us
// with a wave each, 12.7 and 29.7 with 16 lanes, rows of 150: 11.3 and 11.9.
template <int kGroup>
__global__ __launch_bounds__(kRedBlock) void k_red_contained(cg_graph g, uint8_t *contained,
                                                             uint8_t *__restrict__ kept,
                                                             int32_t *__restrict__ cursors,
                                                             int32_t shards,
                                                             uint32_t *__restrict__ sample,
                                                             int stride) {
  const int64_t t = (int64_t)blockIdx.x * kRedBlock + threadIdx.x;
  if (t < shards) cursors[t * kRedCursor] = 0;
  const int64_t row = t / kGroup;
  const int gl = (int)(threadIdx.x % kGroup);
  const bool live = row < g.n;
  const int32_t v = live ? (int32_t)row : 0;
  const int32_t a = live ? g.row_ptr[v] : 0, d = live ? g.row_ptr[v + 1] - a : 0;
  const uint32_t lv = live ? g.read_len[v] : 0u;
  const uint64_t group = (kGroup < kWave ? (1ull << (kGroup % kWave)) - 1ull : ~0ull)
                         << (lane_id() / kGroup * kGroup);
  bool found = false;
  for (int32_t base = 0; __ballot(base < d && !found); base += 4 * kGroup) {
    uint32_t o[4];
    bool c = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t i = base + k * kGroup + gl;
      o[k] = i < d && !found ? g.ovl[a + i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t i = base + k * kGroup + gl;
      if (i < d && !found && o[k] >= lv) {
        const int32_t u = g.col[a + i];
        const uint32_t lu = g.read_len[u];
        c = c || lu > lv || (lu == lv && u < v);
      }
    }
    found = found || (__ballot(c) & group) != 0ull;
  }
  if (live && gl == 0) contained[v] = found ? 1 : 0;
  // a sampled wave's rows that stay, and their entries (see red_crowded and
  // red_wide; only the latter counts rows above kRedCap, which have no near ones)
  const int64_t wave = t / kWave;
  if (kGroup < kWave && __builtin_amdgcn_readfirstlane((int)(wave & ((1 << stride) - 1))) == 0) {
    const int32_t over = g.m < (int64_t)kRedWideRow * g.n ? 0 : kRedCap;
    const uint32_t stay =
        wave_sum(live && gl == 0 && !found ? kRedStay + (uint32_t)(d <= kRedCap ? d : over) : 0u);
    if (lane_id() == 0) sample[wave >> stride] = stay;
  }
  if (found)
    for (int32_t i = gl; i < d; i += kGroup) kept[a + i] = 0;
}

// Whether most reads stay, so that the near entries would need far more room
// than there is: then no row has any, and all are read in full.  Told from a
// sample of the rows, the same for every wave that asks: the entries of rows
// that stay times the share of reads that do is within some percent of the near
// entries (reads of one length at 10x: 18.3 a read, of 12 +- 4 kbp at 8x to 30x
// 2.5 to 1.8).  With room for four a read, filling it does not pay above
// kRedCrowd.
// red_sample loads it, ahead of the loads that do not depend on the answer: the
// first pass's waves of 64 / kRedGroup rows, every 2^k-th of them, 64 to 127.
__host__ __device__ __forceinline__ int32_t red_waves(int32_t n) {
  return (int32_t)(((int64_t)n * kRedGroup + kWave - 1) / kWave);
}
__host__ __device__ __forceinline__ int red_stride(int32_t n) {  // k
  int k = 0;
  while (red_waves(n) >> k >= 2 * kWave) ++k;
  return k;
}
struct RedSample {
  uint32_t lane, rows;
};
__device__ __forceinline__ RedSample red_sample(const uint32_t *sample, int32_t n, int k) {
  const int32_t ns = (red_waves(n) + (1 << k) - 1) >> k;
  const int l = lane_id();
  return RedSample{(l < ns ? sample[l] : 0u) + (l + kWave < ns ? sample[l + kWave] : 0u),
                   (uint32_t)ns * (kWave / kRedGroup)};
}
__device__ __forceinline__ bool red_crowded(const RedSample &s) {
  const uint32_t x = wave_sum(s.lane);
  return x / kRedStay * (x % kRedStay) > kRedCrowd * s.rows * s.rows;
}
// Whether rows want kRedNearWide near neighbours in LDS, by the same sample: the
// entries of rows that stay, by all rows, are within some percent of the near
// entries of such a row.
__device__ __forceinline__ bool red_wide(const RedSample &s) {
  return wave_sum(s.lane) % kRedStay >= kRedWideNear * s.rows;
}

// A workgroup's block of R rows: lane r holds row r's first entry and its
// entries; mask: the rows that are not contained.
struct RedRows {
  int32_t first, entries;
  uint64_t mask;
};
__device__ __forceinline__ RedRows red_block(const cg_graph &g, int R, const uint8_t *contained) {
  const int64_t u = (int64_t)blockIdx.x * R + lane_id();
  const bool v = lane_id() < R && u < g.n;
  RedRows x;
  const uint8_t c = v ? contained[u] : 1;
  x.first = v ? g.row_ptr[u] : 0;
  x.entries = v ? g.row_ptr[u + 1] - x.first : 0;
  x.mask = __ballot(v && !c);
  return x;
}

// a valid walk u, v, x with u->x's end orientations (strand bits s = bit 0,
// d = bit 1 of u->v, v->x and u->x)
__device__ __forceinline__ bool same_ends(uint32_t suv, uint32_t svx, uint32_t sux) {
  return (suv & 1u) == (sux & 1u) && ((suv >> 1) & 1u) == (svx & 1u) &&
         ((svx >> 1) & 1u) == ((sux >> 1) & 1u);
}

__device__ __forceinline__ bool within(int64_t d, uint32_t fuzz) {
  return (d < 0 ? -d : d) <= (int64_t)fuzz;
}

// Near entries: {read, overlap, strands | place in the row << 2, read length}.
// A read's are near[first .. first + count) of its table entry; first < 0:
// none kept, its row is read in full.
struct RedNear {
  uint4 *ent;
  int2 *table;
  int32_t *cursors;
  int32_t shards, cap;  // parts of ent and entries in each
  uint32_t *sample;     // rows that stay, for red_crowded, and its stride
  int stride;
};

__global__ __launch_bounds__(kRedBlock) void k_red_near(cg_graph g, int R,
                                                        const uint8_t *__restrict__ contained,
                                                        uint8_t *__restrict__ kept, RedNear near) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
  const RedSample sample = red_sample(near.sample, g.n, near.stride);
  const RedRows blk = red_block(g, R, contained);
  uint64_t rows = blk.mask;
  if (g.m < (int64_t)kRedShortRow * g.n && red_crowded(sample)) {
    if (w == 0 && ((rows >> lane) & 1ull))
      near.table[(int64_t)blockIdx.x * R + lane] = make_int2(-1, 0);
    rows &= __ballot(blk.entries > kRedCap);
  }
  // the part changes from block to block, so that its cursor is not waited for
  const int32_t part = (int32_t)(blockIdx.x % near.shards), base0 = part * near.cap;
  for (int i = 0; rows; rows &= rows - 1, ++i) {
    if (i % kRedWaves != w) continue;
    const int r = (int)__builtin_ctzll(rows);
    const int32_t u = (int32_t)blockIdx.x * R + r;
    const int32_t a = __builtin_amdgcn_readlane(blk.first, r);
    const int32_t du = __builtin_amdgcn_readlane(blk.entries, r);
    if (du > kRedCap) {
      for (int32_t e = lane; e < du; e += kWave) kept[a + e] = contained[g.col[a + e]] ? 4 : 0;
      if (lane == 0) near.table[u] = make_int2(-1, 0);
      continue;
    }
    int32_t x[kRedPer], f[kRedPer];
    uint32_t o[kRedPer], st[kRedPer];
    bool keep[kRedPer];
#pragma unroll
    for (int k = 0; k < kRedPer; ++k) {
      x[k] = -1;
      o[k] = st[k] = 0;
      if (k * kWave >= du) continue;
      const int32_t e = k * kWave + lane;
      if (e < du) {
        x[k] = g.col[a + e];
        o[k] = g.ovl[a + e];
        st[k] = g.strand[a + e];
      }
    }
    int nf = 0;
#pragma unroll
    for (int k = 0; k < kRedPer; ++k) keep[k] = x[k] >= 0 && !contained[x[k]];
#pragma unroll
    for (int k = 0; k < kRedPer; ++k) {
      const uint64_t m = __ballot(keep[k]);
      f[k] = nf + __popcll(m & ((1ull << lane) - 1ull));
      nf += __popcll(m);
    }
    int32_t at = 0;
    if (lane == 0) at = atomicAdd(near.cursors + part * kRedCursor, nf);
    at = __builtin_amdgcn_readfirstlane(at);
    const bool room = at <= near.cap - nf;
    if (lane == 0) near.table[u] = room ? make_int2(base0 + at, nf) : make_int2(-1, 0);
    if (!room) continue;
#pragma unroll
    for (int k = 0; k < kRedPer; ++k)
      if (x[k] >= 0) kept[a + k * kWave + lane] = keep[k] ? 0 : 4;
#pragma unroll
    for (int k = 0; k < kRedPer; ++k)
      if (keep[k])
        near.ent[base0 + at + f[k]] =
            make_uint4((uint32_t)x[k], o[k], (st[k] & 3u) | (uint32_t)(k * kWave + lane) << 2,
                       g.read_len[x[k]]);
  }
}

// Row u longer than kRedCap or with more near neighbours than LDS has room
// for, read in place: one neighbour at a time, marks straight to kept.
__device__ void red_trans_long(const cg_graph &g, uint32_t fuzz, const uint8_t *contained,
                               uint8_t *kept, int32_t u, int32_t a, int32_t du, int lane) {
  const int32_t *rc = g.col + a;
  for (int32_t f = 0; f < du; ++f) {
    const int32_t v = rc[f];
    if (contained[v]) continue;
    const uint32_t suv = g.strand[a + f];
    const int64_t base = (int64_t)g.read_len[v] - g.ovl[a + f];
    const int32_t b = g.row_ptr[v], dv = g.row_ptr[v + 1] - b;
    for (int32_t i = lane; i < dv; i += kWave) {
      const int32_t x = g.col[b + i];
      if (x == u) continue;
      const int p = lower_bound_i32(rc, du, x);
      if (p == du || rc[p] != x) continue;
      if (!same_ends(suv, g.strand[b + i], g.strand[a + p])) continue;
      if (!within(base - (int64_t)g.ovl[b + i] + (int64_t)g.ovl[a + p], fuzz)) continue;
      if (!contained[x]) kept[a + p] = 1;
    }
  }
}

// 8 workgroups to a compute unit where LDS has room for them (at most 64
// registers; seven of them and 100 Mbp at 15x took 169 us instead of 118).
// With kAsk it leaves the rows to the instance of other kNear if red_wide says so.
template <int kNear, bool kAsk>
__global__ __launch_bounds__(kRedBlock, kNear <= kRedNear ? 8 : 1) void k_red_trans(
    cg_graph g, uint32_t fuzz, int R, const uint8_t *__restrict__ contained, uint8_t *kept,
    RedNear near) {
  if (kAsk && red_wide(red_sample(near.sample, g.n, near.stride)) != (kNear > kRedNear)) return;
  // u's near neighbours in column order: their ids, overlaps, first entries
  // (near ones, or of the whole row: bit 2 of the strands), the pairs of those
  // before, lengths, strands and marks
  __shared__ int32_t sh_col[kRedWaves][kNear];
  __shared__ uint32_t sh_ovl[kRedWaves][kNear];
  __shared__ int32_t sh_vb[kRedWaves][kNear];
  __shared__ int32_t sh_pfx[kRedWaves][kNear];
  __shared__ uint32_t sh_vlen[kRedWaves][kNear];
  __shared__ uint8_t sh_str[kRedWaves][kNear], sh_mark[kRedWaves][kNear];
  __shared__ int s_next;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
  if (threadIdx.x == 0) s_next = kRedWaves;
  __syncthreads();
  int32_t *s_col = sh_col[w], *s_vb = sh_vb[w], *s_pfx = sh_pfx[w];
  uint32_t *s_ovl = sh_ovl[w], *s_vlen = sh_vlen[w];
  uint8_t *s_str = sh_str[w], *s_mark = sh_mark[w];
  const RedRows blk = red_block(g, R, contained);
  const bool mine = (blk.mask >> lane) & 1ull;
  const int2 tab = mine ? near.table[(int64_t)blockIdx.x * R + lane] : make_int2(-1, 0);
  uint64_t rows = blk.mask;
  const int n_rows = __popcll(rows);
  // the waves take the rows as they come free; `at` is the row lowest in rows
  for (int at = 0, i = w; i < n_rows;) {
    for (; at < i; ++at) rows &= rows - 1;
    const int r = (int)__builtin_ctzll(rows);
    const int32_t u = (int32_t)blockIdx.x * R + r;
    const int32_t a = __builtin_amdgcn_readlane(blk.first, r);
    const int32_t du = __builtin_amdgcn_readlane(blk.entries, r);
    const int32_t own = __builtin_amdgcn_readlane(tab.x, r);
    int nf = own >= 0 ? __builtin_amdgcn_readlane(tab.y, r) : 0;
    bool longer = own >= 0 ? nf > kNear : du > kRedCap;
    if (!longer) {
      // the near neighbours, a lane each: rounds of 64 near entries, or of the
      // whole row
      int32_t v[kRedPer], f[kRedPer], e[kRedPer];
      uint32_t o[kRedPer], st[kRedPer], lv[kRedPer];
      bool keep[kRedPer];
      const int len = own >= 0 ? nf : du;
#pragma unroll
      for (int k = 0; k < kRedPer; ++k) {
        v[k] = -1;
        e[k] = f[k] = 0;
        o[k] = st[k] = lv[k] = 0;
        if (k * kWave >= len) continue;
        const int32_t p = k * kWave + lane;
        if (own >= 0) {
          if (p < len) {
            const uint4 x = near.ent[own + p];
            v[k] = (int32_t)x.x;
            o[k] = x.y;
            st[k] = x.z & 3u;
            e[k] = (int32_t)(x.z >> 2);
            lv[k] = x.w;
          }
        } else if (p < len) {
          v[k] = g.col[a + p];
          o[k] = g.ovl[a + p];
          st[k] = g.strand[a + p] & 3u;
          e[k] = p;
          lv[k] = g.read_len[v[k]];
        }
      }
#pragma unroll
      for (int k = 0; k < kRedPer; ++k) {
        keep[k] = v[k] >= 0;
        f[k] = k * kWave + lane;
      }
      if (own < 0) {
#pragma unroll
        for (int k = 0; k < kRedPer; ++k) {
          keep[k] = keep[k] && !contained[v[k]];
          const uint64_t m = __ballot(keep[k]);
          f[k] = nf + __popcll(m & ((1ull << lane) - 1ull));
          nf += __popcll(m);
        }
        longer = nf > kNear;
        if (longer) {
          nf = 0;  // read in place below: nothing of it goes to LDS
#pragma unroll
          for (int k = 0; k < kRedPer; ++k) {
            if (k * kWave + lane < du) kept[a + k * kWave + lane] = keep[k] ? 0 : 4;
            keep[k] = false;
          }
          __threadfence_block();  // these land before any mark
        }
      }
      int32_t b[kRedPer], dv[kRedPer];
#pragma unroll
      for (int k = 0; k < kRedPer; ++k) {
        b[k] = dv[k] = 0;
        if (k * kWave >= len || !keep[k]) continue;
        const int2 t = near.table[v[k]];
        b[k] = t.x;
        dv[k] = t.y;
        if (t.x < 0) {
          b[k] = g.row_ptr[v[k]];
          dv[k] = g.row_ptr[v[k] + 1] - b[k];
          st[k] |= 4u;
        }
      }
      int32_t pairs = 0;
#pragma unroll
      for (int k = 0; k < kRedPer; ++k) {
        if (k * kWave >= len) continue;
        const int32_t inc = wave_incl_scan(dv[k]);
        if (keep[k]) {
          s_col[f[k]] = v[k];
          s_ovl[f[k]] = o[k];
          s_str[f[k]] = (uint8_t)st[k];
          s_mark[f[k]] = 0;
          s_vb[f[k]] = b[k];
          s_vlen[f[k]] = lv[k];
          s_pfx[f[k]] = pairs + inc - dv[k];
        }
        pairs += wave_lane(inc, kWave - 1);
      }
      wave_lds_sync();
      // pair t belongs to the last neighbour j with s_pfx[j] <= t (one with
      // entries: t < pairs rules out an empty last neighbour); two pairs per
      // lane, so that their searches and loads overlap
      constexpr int U = 2;
      int top = 1;
      while (2 * top < nf) top *= 2;
      for (int32_t base = 0; base < pairs; base += U * kWave) {
        int j[U], p[U];
        uint32_t x[U], sx[U], ox[U];
        bool hit[U];
#pragma unroll
        for (int k = 0; k < U; ++k) j[k] = p[k] = 0;
        for (int step = top; step > 0; step >>= 1) {
#pragma unroll
          for (int k = 0; k < U; ++k) {
            const int q = j[k] + step;
            if (q < nf && s_pfx[q] <= base + k * kWave + lane) j[k] = q;
          }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const int32_t t = base + k * kWave + lane;
          hit[k] = t < pairs;
          x[k] = sx[k] = ox[k] = 0;
          if (!hit[k]) continue;
          const int32_t y = s_vb[j[k]] + (t - s_pfx[j[k]]);
          if (s_str[j[k]] & 4u) {
            x[k] = (uint32_t)g.col[y];
            ox[k] = g.ovl[y];
            sx[k] = g.strand[y];
          } else {
            const uint4 z = near.ent[y];
            x[k] = z.x;
            ox[k] = z.y;
            sx[k] = z.z;
          }
        }
        for (int step = top; step > 0; step >>= 1) {
#pragma unroll
          for (int k = 0; k < U; ++k) {
            const int q = p[k] + step;
            if (q < nf && s_col[q] <= (int32_t)x[k]) p[k] = q;
          }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
          if (!hit[k] || (int32_t)x[k] == u || s_col[p[k]] != (int32_t)x[k]) continue;
          if (!same_ends(s_str[j[k]], sx[k], s_str[p[k]])) continue;
          const int64_t d =
              (int64_t)s_vlen[j[k]] - (int64_t)s_ovl[j[k]] - (int64_t)ox[k] + (int64_t)s_ovl[p[k]];
          if (within(d, fuzz)) s_mark[p[k]] = 1;
        }
      }
      wave_lds_sync();
      if (own >= 0) {
#pragma unroll
        for (int k = 0; k < kRedPer; ++k)
          if (keep[k] && s_mark[f[k]]) kept[a + e[k]] = 1;
      } else if (!longer) {
#pragma unroll
        for (int k = 0; k < kRedPer; ++k)
          if (k * kWave + lane < du) kept[a + k * kWave + lane] = keep[k] ? s_mark[f[k]] : 4;
      }
      wave_lds_sync();
    }
    if (longer) red_trans_long(g, fuzz, contained, kept, u, a, du, lane);
    if (lane == 0) i = atomicAdd(&s_next, 1);
    i = __builtin_amdgcn_readfirstlane(i);
  }
}

// The entries left over of a wave's rows are collected in LDS first, so that
// the binary searches for their twins (a chain of loads each) run side by
// side: one row at a time the 50 Mbp graph took 25 us.
__global__ __launch_bounds__(kRedBlock) void k_red_keep(cg_graph g, int R,
                                                        const uint8_t *__restrict__ contained,
                                                        uint8_t *kept, uint32_t *__restrict__ counts,
                                                        uint32_t *__restrict__ blocks) {
  __shared__ uint32_t s_cnt[kRedRows];
  __shared__ int32_t sh_ent[kRedWaves][kRedList];
  __shared__ uint8_t sh_row[kRedWaves][kRedList];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
  if (threadIdx.x < kRedRows) s_cnt[threadIdx.x] = 0;
  const RedRows blk = red_block(g, R, contained);
  __syncthreads();
  int32_t *s_ent = sh_ent[w];
  uint8_t *s_row = sh_row[w];
  int n_list = 0;
  auto search = [&] {
    wave_lds_sync();
    for (int i = lane; i < n_list; i += kWave) {
      // the twin x->u: its mark decides as well
      const int32_t e = s_ent[i], r = s_row[i], u = (int32_t)blockIdx.x * R + r;
      const int32_t x = g.col[e];
      const int32_t b = g.row_ptr[x], dx = g.row_ptr[x + 1] - b;
      const int q = lower_bound_i32(g.col + b, dx, u);
      if (q < dx && g.col[b + q] == u && (kept[b + q] & 1u)) continue;
      // bit 0 is left as it was: other rows read it as their twin's mark
      kept[e] = 2;
      atomicAdd(s_cnt + r, 1u);
    }
    n_list = 0;
    wave_lds_sync();
  };
  uint64_t rows = blk.mask;
  for (int i = 0; rows; rows &= rows - 1, ++i) {
    if (i % kRedWaves != w) continue;
    const int r = (int)__builtin_ctzll(rows);
    const int32_t a = __builtin_amdgcn_readlane(blk.first, r);
    const int32_t du = __builtin_amdgcn_readlane(blk.entries, r);
    for (int32_t base = 0; base < du; base += kWave) {
      const int32_t e = base + lane;
      // neither marked nor to a contained read
      const bool left = e < du && !(kept[a + e] & 5u);
      const uint64_t m = __ballot(left);
      if (left) {
        const int at = n_list + __popcll(m & ((1ull << lane) - 1ull));
        s_ent[at] = a + e;
        s_row[at] = (uint8_t)r;
      }
      n_list += __popcll(m);
      if (n_list > kRedList - kWave) search();
    }
  }
  search();
  __syncthreads();
  if (w == 0) {
    const int64_t u = (int64_t)blockIdx.x * R + lane;
    const uint32_t c = s_cnt[lane];
    if (lane < R && u < g.n) counts[u] = c;
    const uint32_t sum = wave_sum(c);
    if (lane == 0) blocks[blockIdx.x] = sum;
  }
}

// one workgroup of the sums over many blocks: blocks[i] becomes the entries of
// the blocks before i (above kRedDirect blocks, 2.6e5 reads, where each
// workgroup of k_red_compact adding them up itself would cost more)
__global__ __launch_bounds__(kScanBlock) void k_red_sums(int nb, uint32_t *__restrict__ blocks) {
  __shared__ uint32_t sh[kScanBlock / kWave + 1];
  const int per = (nb + kScanBlock - 1) / kScanBlock;
  const int i0 = (int)threadIdx.x * per, i1 = i0 + per < nb ? i0 + per : nb;
  uint32_t x = 0, tot;
  for (int i = i0; i < i1; ++i) x += blocks[i];
  uint32_t ex = block_excl_scan<uint32_t, kScanBlock>(x, sh, &tot);
  for (int i = i0; i < i1; ++i) {
    const uint32_t c = blocks[i];
    blocks[i] = ex;
    ex += c;
  }
}

__global__ __launch_bounds__(kRedBlock) void k_red_compact(
    cg_graph g, int R, int summed, const uint8_t *__restrict__ contained,
    const uint32_t *__restrict__ counts, const uint32_t *__restrict__ blocks, uint8_t *kept,
    int32_t *__restrict__ s_row_ptr, int32_t *__restrict__ d_m, int32_t *__restrict__ s_col,
    uint32_t *__restrict__ s_ovl, uint8_t *__restrict__ s_strand) {
  __shared__ uint32_t s_sum[kRedWaves];
  __shared__ int32_t s_off[kRedRows];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
  // the entries of the blocks before this one
  uint32_t x = 0;
  if (summed) {
    if (threadIdx.x == 0) x = blocks[blockIdx.x];
  } else {
#pragma unroll 4
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kRedBlock) x += blocks[i];
  }
  x = wave_sum(x);
  if (lane == 0) s_sum[w] = x;
  const int64_t u0 = (int64_t)blockIdx.x * R;
  const RedRows blk = red_block(g, R, contained);
  __syncthreads();
  if (w == 0) {
    int32_t before = 0;
    for (int k = 0; k < kRedWaves; ++k) before += (int32_t)s_sum[k];
    const bool v = lane < R && u0 + lane < g.n;
    const int32_t c = v ? (int32_t)counts[u0 + lane] : 0;
    const int32_t inc = wave_incl_scan(c);
    s_off[lane] = before + inc - c;
    if (v) s_row_ptr[u0 + lane] = before + inc - c;
    if (blockIdx.x == gridDim.x - 1 && lane == kWave - 1) {
      s_row_ptr[g.n] = before + inc;
      *d_m = before + inc;
    }
  }
  __syncthreads();
  uint64_t rows = blk.mask;
  for (int i = 0; rows; rows &= rows - 1, ++i) {
    if (i % kRedWaves != w) continue;
    const int r = (int)__builtin_ctzll(rows);
    const int32_t a = __builtin_amdgcn_readlane(blk.first, r);
    const int32_t du = __builtin_amdgcn_readlane(blk.entries, r);
    int32_t at = s_off[r];
    for (int32_t base = 0; base < du; base += kWave) {
      const int32_t e = base + lane;
      const bool k = e < du && (kept[a + e] & 2u);
      const uint64_t mask = __ballot(k);
      if (k) {
        const int32_t o = at + __popcll(mask & ((1ull << lane) - 1ull));
        s_col[o] = g.col[a + e];
        s_ovl[o] = g.ovl[a + e];
        s_strand[o] = g.strand[a + e];
      }
      if (e < du) kept[a + e] = k ? 1 : 0;
      at += __popcll(mask);
    }
  }
}

int launch_reduce(cg_ctx *ctx, const cg_graph &g, const Scratch &s, uint32_t fuzz,
                  uint8_t *contained, uint8_t *kept, int32_t *s_row_ptr, int32_t *s_col,
                  uint32_t *s_ovl, uint8_t *s_strand, int32_t *d_m, hipStream_t st) {
  const PhaseRange range("cg: reduce");
  const int32_t n = g.n;
  const int R = red_rows(n, kRedBlocks);
  const int nb = n > 0 ? (int)(((int64_t)n + R - 1) / R) : 1;
  uint32_t *counts = s.piece_len, *blocks = s.fill;
  // room for four near entries per read, in the walk area (12 +- 4 kbp reads
  // have 2.8 at 8x and fewer above, reads of about one length 15 and more, of
  // which the first rows' then fit); a part for every 256 reads (the cursors take 64 words of lidx
  // each)
  const int64_t near_cap = 4 * (int64_t)n < 0x7FFFFFFF ? 4 * (int64_t)n : 0x7FFFFFFF;
  const int32_t shards = n / 256 < 1 ? 1 : (n / 256 < kRedShards ? n / 256 : kRedShards);
  const RedNear near{reinterpret_cast<uint4 *>(s.walk), reinterpret_cast<int2 *>(s.tmp), s.lidx,
                     shards, (int32_t)(near_cap / shards), reinterpret_cast<uint32_t *>(s.keys),
                     red_stride(n)};
  if (n > 0) {
    const bool waves = g.m >= (int64_t)kRedWaveRow * n;
    const int64_t groups = ((int64_t)n * (waves ? kWave : kRedGroup) + kRedBlock - 1) / kRedBlock;
    if (waves)
      CG_LAUNCH(ctx, k_red_contained<kWave>, dim3((unsigned)groups), dim3(kRedBlock), st, g,
                contained, kept, near.cursors, shards, near.sample, near.stride);
    else
      CG_LAUNCH(ctx, k_red_contained<kRedGroup>, dim3((unsigned)groups), dim3(kRedBlock), st, g,
                contained, kept, near.cursors, shards, near.sample, near.stride);
    CG_LAUNCH(ctx, k_red_near, dim3(nb), dim3(kRedBlock), st, g, R, contained, kept, near);
    const bool longer = g.m >= (int64_t)2 * kRedCap * n;
    const bool wide = g.m >= (int64_t)kRedWideRow * n && !longer, ask = wide && !waves;
    const int Rw = red_rows(n, kRedWideBlocks);
    const int Rn = red_rows(n, longer ? kRedBlocks : kRedTransBlocks);
    // both instances from 96 entries a read on, and the sample has one of them
    // leave; the pass with a wave a row takes none, and long rows want the wide one
    const dim3 gw((unsigned)(((int64_t)n + Rw - 1) / Rw));
    const dim3 gn((unsigned)(((int64_t)n + Rn - 1) / Rn));
    if (ask) {
      CG_LAUNCH(ctx, (k_red_trans<kRedNearWide, true>), gw, dim3(kRedBlock), st, g, fuzz, Rw,
                contained, kept, near);
      CG_LAUNCH(ctx, (k_red_trans<kRedNear, true>), gn, dim3(kRedBlock), st, g, fuzz, Rn, contained,
                kept, near);
    } else if (wide) {
      CG_LAUNCH(ctx, (k_red_trans<kRedNearWide, false>), gw, dim3(kRedBlock), st, g, fuzz, Rw,
                contained, kept, near);
    } else {
      CG_LAUNCH(ctx, (k_red_trans<kRedNear, false>), gn, dim3(kRedBlock), st, g, fuzz, Rn,
                contained, kept, near);
    }
    CG_LAUNCH(ctx, k_red_keep, dim3(nb), dim3(kRedBlock), st, g, R, contained, kept, counts,
              blocks);
    if (nb > kRedDirect) CG_LAUNCH(ctx, k_red_sums, dim3(1), dim3(kScanBlock), st, nb, blocks);
  }
  CG_LAUNCH(ctx, k_red_compact, dim3(nb), dim3(kRedBlock), st, g, R, nb > kRedDirect ? 1 : 0,
            contained, counts, blocks, kept, s_row_ptr, d_m, s_col, s_ovl, s_strand);
  return hip_check(hipGetLastError(), "k_red");
}

}  // namespace cg
