// LocalAssembly (Section 4.4).  A contig is the concatenation
//   l_r[alpha:pre(e0)] + l_c1[post(e0):pre(e1)] + ... + l_r'[post(e_{q-2}):beta]
// over the chain r, c1, ..., r' of a component: every read but the last
// contributes the part of its walking orientation that precedes its overlap
// with the next read (len - ovl bases), the last read all its bases.
//
// As a step of its own (the whole path walks in its component pass,
// k_components.hip, and shares the last two):
//
//  k_asm_walk     every component by its size (a lane, a wave, a workgroup):
//                 start read, walk order by pointer jumping over the chain's
//                 arcs (Wyllie list ranking), orientation from the strand
//                 bits, piece lengths and offsets, layout and contig record
//  k_asm_offsets  contig base offsets (16-base aligned) in (bin, label) order
//  k_asm_copy     chunks of consecutive pieces, one wave each: every output
//                 word is written by the piece holding its first base, 2-bit
//                 funnel shifts for unaligned starts, reverse + complement in
//                 registers
#include "cg_device.h"

namespace cg {

// Components by size: a lane for one read, a wave up to kWalkSmallCap reads,
// a workgroup up to kAsmWalkCap reads with everything in LDS, up to
// kAsmRaysCap reads with the rays in LDS, and above with them in global
// memory.  A component's walk is mostly latency (dependent gathers), so as
// many as possible run at once: the LDS of four waves' components is that of
// a workgroup's, 27 KB, five workgroups to a compute unit.
// Workgroups 0 .. n_big - 1 take the components above kWalkSmallCap reads, so
// that the longest ones start first; the waves of the others take runs of
// consecutive components.
constexpr int kAsmWalkBlock = 256;
constexpr int kAsmWalkCap = 512;
constexpr int kAsmWalkWaves = kAsmWalkBlock / kWave;
static_assert(kAsmWalkCap % kAsmWalkBlock == 0, "whole members per thread");
static_assert(kAsmWalkCap == kAsmWalkWaves * kWalkSmallCap, "the waves share the workgroup's LDS");
constexpr int kAsmWalkWords = 13 * kAsmWalkCap + kAsmWalkCap / 2;  // 54 bytes per read
constexpr int kAsmRaysCap = kAsmWalkWords / 2;
// The look-back words that k_asm_offsets scans with start at zero: as a step of
// its own it follows whatever call had the context's scratch last, and a
// smaller graph's arrays lie where a larger one's words do.
__global__ __launch_bounds__(kAsmWalkBlock, 5) void k_asm_walk(
    cg_graph g, cg_parts parts, cg_local local, cg_contigs out, Scratch s, int n_big,
    int n_status) {
  __shared__ alignas(16) uint32_t buf[kAsmWalkWords];
  __shared__ uint64_t sh_scan[kAsmWalkBlock / kWave + 1];
  __shared__ int s_n;
  __shared__ int32_t s_list[kAsmWalkBlock];
  for (int64_t i = (int64_t)blockIdx.x * kAsmWalkBlock + threadIdx.x; i < n_status;
       i += (int64_t)gridDim.x * kAsmWalkBlock)
    s.scan_status[i] = 0;
  const int nc = *parts.d_n_comp;
  // the arrays of cap reads from read slot r0 of kAsmWalkCap on
  auto arrays = [&](int r0) {
    constexpr int C = kAsmWalkCap;
    WalkArrays w{};
    w.roff = reinterpret_cast<uint64_t *>(buf) + r0;
    w.nb = reinterpret_cast<int32_t *>(buf + 2 * C) + 2 * r0;
    w.ray = buf + 4 * C + 2 * r0;
    w.eo = buf + 6 * C + 2 * r0;
    w.ep = buf + 8 * C + 2 * r0;
    w.vid = reinterpret_cast<int32_t *>(buf + 10 * C) + r0;
    w.rlen = buf + 11 * C + r0;
    w.eid = reinterpret_cast<int32_t *>(buf + 12 * C) + r0;  // the piece lengths only
    w.es = reinterpret_cast<uint8_t *>(buf + 13 * C) + 2 * r0;
    return w;
  };
  if ((int)blockIdx.x < n_big) {
    for (int64_t base = blockIdx.x; base < nc; base += (int64_t)n_big * kAsmWalkBlock) {
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      const int64_t x = base + (int64_t)n_big * threadIdx.x;
      if (x < nc && parts.comp_size[x] > kWalkSmallCap) s_list[atomicAdd(&s_n, 1)] = (int32_t)x;
      __syncthreads();
      const int k = s_n;
      for (int i = 0; i < k; ++i) {
        const int c = __builtin_amdgcn_readfirstlane(s_list[i]);
        const int q = parts.comp_size[c], st = parts.comp_start[c];
        if (q <= kAsmWalkCap) {
          walk_component<kAsmWalkBlock, kAsmWalkCap, kWalkLds>(
              c, q, st, arrays(0), g, parts, local.perm, local.loc_row_ptr, local.loc_col,
              local.loc_eid, out, s, sh_scan);
        } else if (q <= kAsmRaysCap) {
          walk_component<kAsmWalkBlock, kAsmRaysCap, kWalkRaysLds>(
              c, q, st, walk_scratch(s.walk, g.n, st, buf), g, parts, local.perm,
              local.loc_row_ptr, local.loc_col, local.loc_eid, out, s, sh_scan);
        } else {
          walk_component<kAsmWalkBlock, kAsmRaysCap, kWalkGlobal>(
              c, q, st, walk_scratch(s.walk, g.n, st, buf), g, parts, local.perm,
              local.loc_row_ptr, local.loc_col, local.loc_eid, out, s, sh_scan);
        }
      }
      __syncthreads();
    }
    return;
  }
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int64_t w = (int64_t)(blockIdx.x - n_big) * kAsmWalkWaves + wv;
  const int64_t nw = (int64_t)(gridDim.x - n_big) * kAsmWalkWaves;
  int64_t run = (nc + nw - 1) / nw;
  if (run > kWave) run = kWave;
  for (int64_t c0 = w * run; c0 < nc; c0 += nw * run) {
    const int64_t c = c0 + lane_id();
    const bool live = lane_id() < run && c < nc;
    const int32_t q = live ? parts.comp_size[c] : 0;
    const int32_t st = live ? parts.comp_start[c] : 0;
    if (q == 1) walk_single(g, parts, (int)c, st, out, s);
    for (uint64_t todo = __ballot(q > 1 && q <= kWalkSmallCap); todo; todo &= todo - 1) {
      const int t = (int)__builtin_ctzll(todo);
      const int tq = __builtin_amdgcn_readlane(q, t), tst = __builtin_amdgcn_readlane(st, t);
      walk_component<kWave, kWalkSmallCap, kWalkLds>(
          (int)c0 + t, tq, tst, arrays(wv * kWalkSmallCap), g, parts, local.perm,
          local.loc_row_ptr, local.loc_col, local.loc_eid, out, s, sh_scan);
    }
  }
}

// contig word offsets: scan of ceil(len/16) in record order.  One workgroup
// up to kOffItems contigs, what its threads hold in registers (5 us); above,
// the workgroups of a look-back scan over kOffItems contigs each, the others
// leave at once (110,000 contigs: 15 us, 146 us in one workgroup's rounds).
constexpr int kOffRun = 8;  // contigs per thread, in registers
constexpr int kOffItems = kOffRun * kScanBlock;
static int offsets_blocks(int32_t n) { return (int)(((int64_t)n + kOffItems - 1) / kOffItems); }
__global__ __launch_bounds__(kScanBlock) void k_asm_offsets(const int32_t *__restrict__ d_n_comp,
                                                            const uint64_t *__restrict__ len,
                                                            uint64_t *__restrict__ base_off,
                                                            uint64_t cap_words,
                                                            uint64_t *__restrict__ d_total_words,
                                                            Fixed *fx, ScanCtx sc) {
  __shared__ unsigned long long sh[kScanBlock / kWave + 1];
  const int nc = *d_n_comp;
  const int nblocks = nc > kOffItems ? (int)(((int64_t)nc + kOffItems - 1) / kOffItems) : 1;
  if ((int)blockIdx.x >= nblocks) return;
  const int blk = nblocks > 1 ? lookback_ticket(sc) : 0;
  // thread t takes E consecutive contigs, their lengths loaded at once: one
  // block scan of the thread sums (a loop over blocks of contigs waited for a
  // load and a scan per block)
  const int cnt = nc - blk * kOffItems < kOffItems ? nc - blk * kOffItems : kOffItems;
  const int E = (cnt + kScanBlock - 1) / kScanBlock;
  const int k0 = blk * kOffItems + (int)threadIdx.x * E;
  const int k1 = blk * kOffItems + cnt;
  unsigned long long w[kOffRun], x = 0;
#pragma unroll
  for (int r = 0; r < kOffRun; ++r) {
    w[r] = r < E && k0 + r < k1 ? (len[k0 + r] + 15) / 16 : 0;
    x += w[r];
  }
  unsigned long long ex, total;
  if (nblocks > 1) ex = lookback_block_scan(sc, blk, x, &total);
  else ex = block_excl_scan<unsigned long long, kScanBlock>(x, sh, &total);
#pragma unroll
  for (int r = 0; r < kOffRun; ++r) {
    if (r < E && k0 + r < k1) base_off[k0 + r] = 16 * ex;
    ex += w[r];
  }
  if (threadIdx.x == 0 && blk == nblocks - 1) {
    *d_total_words = total;
    if (total > cap_words) atomicOr(&fx->status, CG_STATUS_BASES_OVERFLOW);
  }
  if (nblocks > 1) lookback_finish(sc, nblocks);
}

constexpr int kCopyBlock = 256;
constexpr int kCopyWavesPerCU = 16;  // resident copy waves per compute unit (4 per SIMD)
constexpr int kCopyRounds = 4;       // copy chunks per resident wave slot
constexpr int kCopyMinPieces = 2;    // pieces per copy chunk at least

// a wave's share of the pieces' chunks
template <typename CB>
__device__ __forceinline__ void copy_share(const uint32_t *seq, uint64_t seq_words, uint32_t *bases,
                                           const PieceArraysT<CB> &A, int32_t n_e,
                                           int32_t chunk_target) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t gw = blockIdx.x * (blockDim.x / kWave) + wave;
  const int32_t nwv = gridDim.x * (blockDim.x / kWave);
  // pieces per chunk: about chunk_target chunks (a few per wave slot of the
  // device, so the slots drain evenly while each chunk's setup, a chain of
  // dependent descriptor loads, is paid for enough pieces), at least
  // kCopyMinPieces, at most one piece per lane
  int32_t C = (n_e + chunk_target - 1) / chunk_target;
  C = C < kCopyMinPieces ? kCopyMinPieces : (C > kWave ? kWave : C);
  const int32_t n_chunks = (n_e + C - 1) / C;
  for (int32_t ch = gw; ch < n_chunks; ch += nwv) {
    const int32_t c0 = ch * C;
    const int cnt = n_e - c0 < C ? n_e - c0 : C;
    copy_chunk(seq, seq_words, bases, A, c0, cnt, n_e, lane_id());
  }
}

__global__ __launch_bounds__(kCopyBlock) void k_asm_copy(const uint32_t *__restrict__ seq,
                                                         uint64_t seq_words,
                                                         const int32_t *__restrict__ bin_vptr,
                                                         int32_t P,
                                                         const uint64_t *__restrict__ piece_off,
                                                         const uint32_t *__restrict__ piece_len,
                                                         const uint64_t *__restrict__ piece_src,
                                                         const int32_t *__restrict__ lay_contig,
                                                         const uint64_t *__restrict__ clen,
                                                         const uint64_t *__restrict__ cbase,
                                                         const uint64_t *__restrict__ d_total_words,
                                                         uint64_t cap_words,
                                                         uint32_t *__restrict__ bases,
                                                         int32_t chunk_target,
                                                         const Fixed *fx, StatusOut so) {
  // the last kernel of the path: no earlier one can still raise a bit
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (so.set) *so.set = fx->status;
    if (so.add && fx->status) atomicOr(so.add, fx->status);
  }
  if (*d_total_words > cap_words) return;
  const int32_t n_e = bin_vptr[P];
  const PieceArrays A = piece_arrays(lay_contig, piece_off, piece_len, piece_src, clen, cbase);
  copy_share(seq, seq_words, bases, A, n_e, chunk_target);
}

// Offsets and copy of a small graph in one launch: every workgroup scans all
// contigs' lengths for itself, in LDS (a few per thread), and copies from
// there; the first one stores the offsets.  A launch of k_asm_offsets is 4 us
// of latency, a workgroup's own scan a fraction of that (1,000 reads: 3.8 + 8.5
// us as two launches, 8.4 as one; a path of 1,000 reads 41.4 -> 39.0 us, of
// 13,000 72.4 -> 71.1).  Up to kOwnContigs contigs and as many reads as give no
// more workgroups (32 reads each) than are resident with that much LDS: a
// second round of them would scan again.
constexpr int kOwnContigs = 8192;
constexpr int kOwnReads = 16384;
__global__ __launch_bounds__(kCopyBlock) void k_asm_bases(cg_graph g, const int32_t *bin_vptr,
                                                          int32_t P, const int32_t *d_n_comp,
                                                          Scratch s, cg_contigs out,
                                                          int32_t chunk_target, Fixed *fx,
                                                          StatusOut so) {
  __shared__ uint64_t base[kOwnContigs];
  __shared__ unsigned long long sh[kCopyBlock / kWave + 1];
  const int nc = *d_n_comp;
  const int32_t n_e = bin_vptr[P];
  for (int k = threadIdx.x; k < nc; k += kCopyBlock) base[k] = (out.len[k] + 15) / 16;
  __syncthreads();
  const int E = (nc + kCopyBlock - 1) / kCopyBlock;
  const int k0 = (int)threadIdx.x * E, k1 = k0 + E < nc ? k0 + E : nc;
  unsigned long long x = 0, total;
  for (int k = k0; k < k1; ++k) x += base[k];
  unsigned long long ex = block_excl_scan<unsigned long long, kCopyBlock>(x, sh, &total);
  for (int k = k0; k < k1; ++k) {
    const unsigned long long w = base[k];
    base[k] = 16 * ex;
    ex += w;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int k = threadIdx.x; k < nc; k += kCopyBlock) out.base_off[k] = base[k];
    if (threadIdx.x == 0) {
      *out.d_total_words = total;
      // the last kernel of the path: no earlier one can still raise a bit
      unsigned int bits = fx->status;
      if (total > out.cap_words) {
        atomicOr(&fx->status, CG_STATUS_BASES_OVERFLOW);
        bits |= CG_STATUS_BASES_OVERFLOW;
      }
      if (so.set) *so.set = bits;
      if (so.add && bits) atomicOr(so.add, bits);
    }
  }
  if (total > out.cap_words) return;
  typedef const __attribute__((address_space(3))) uint64_t *LdsBase;
  const PieceArrays p = piece_arrays(s.lay_contig, s.piece_off, s.piece_len, s.piece_src, out.len,
                                     nullptr);
  const PieceArraysT<LdsBase> A{p.lay_contig, p.piece_off, p.piece_len, p.piece_src, p.clen,
                                (LdsBase)base};
  copy_share(g.seq, g.seq_words, out.bases, A, n_e, chunk_target);
}

// offsets and bases of the walked contigs, at most max_contigs of them
int launch_contigs(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const cg_parts &parts,
                   const cg_local &local, int32_t P, int32_t max_contigs, const cg_contigs &out,
                   hipStream_t st, const StatusOut &so) {
  const int32_t n = g.n;
  // about eight pieces per wave, so a small graph still spreads over the chip
  const int cgrid = (n + 31) / 32 < 8192 ? (n + 31) / 32 : 8192;
  // chunks: kCopyRounds per resident wave slot (kCopyWavesPerCU per compute
  // unit at the copy's register use), and never fewer than the grid's waves
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess ||
      cus < 1)
    cus = 1;
  const int64_t tgt = (int64_t)kCopyRounds * kCopyWavesPerCU * cus;
  const int64_t gw = (int64_t)cgrid * (kCopyBlock / kWave);
  const int32_t chunk_target = (int32_t)(tgt > gw ? gw : tgt);
  if (max_contigs <= kOwnContigs && n <= kOwnReads) {
    CG_LAUNCH(ctx, k_asm_bases, dim3(cgrid), dim3(kCopyBlock), st, g, local.bin_vptr, P,
              parts.d_n_comp, s, out, chunk_target, ctx->fixed, so);
    return hip_check(hipGetLastError(), "k_asm");
  }
  CG_LAUNCH(ctx, k_asm_offsets, dim3((unsigned)offsets_blocks(n)), dim3(kScanBlock), st,
            parts.d_n_comp, out.len, out.base_off, out.cap_words,
            out.d_total_words, ctx->fixed, scan_ctx(ctx, s));
  CG_LAUNCH(ctx, k_asm_copy, dim3(cgrid), dim3(kCopyBlock), st, g.seq, g.seq_words,
                     local.bin_vptr, P, s.piece_off, s.piece_len, s.piece_src, s.lay_contig,
                     out.len, out.base_off, out.d_total_words, out.cap_words, out.bases,
                     chunk_target, ctx->fixed, so);
  return hip_check(hipGetLastError(), "k_asm");
}

int launch_assemble(cg_ctx *ctx, const cg_graph &g, const Scratch &s, const cg_parts &parts,
                    const cg_local &local, int32_t P, const cg_contigs &out, hipStream_t st) {
  const PhaseRange range("cg: LocalAssembly");
  const int32_t n = g.n;
  if (n == 0) {
    CG_LAUNCH(ctx, k_asm_offsets, dim3(1), dim3(kScanBlock), st, parts.d_n_comp, out.len,
                       out.base_off, out.cap_words, out.d_total_words, ctx->fixed,
                       scan_ctx(ctx, s));
    return hip_check(hipGetLastError(), "k_asm");
  }
  // workgroups for as many components above kWalkSmallCap reads as there can
  // be, and waves for components of two reads, up to a few rounds of what is
  // resident at once
  const int n_big = n / (kWalkSmallCap + 1) < 2048 ? n / (kWalkSmallCap + 1) : 2048;
  const int64_t nw = ((int64_t)n / 2 + kAsmWalkWaves) / kAsmWalkWaves;
  CG_LAUNCH(ctx, k_asm_walk, dim3((unsigned)(n_big + (nw < 2048 ? nw : 2048))),
            dim3(kAsmWalkBlock), st, g, parts, local, out, s, n_big, offsets_blocks(n));
  return launch_contigs(ctx, g, s, parts, local, P, n, out, st, StatusOut{});
}

}  // namespace cg
