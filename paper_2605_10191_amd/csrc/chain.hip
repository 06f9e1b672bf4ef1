// Fused Clenshaw step for the chain models (XXZ, t-V) in a particle-number
// sector, laid out for wave64 execution.
//
// A state is split as s = hi << Lb | lo.  States in ascending order are
// grouped by hi, and the rows of one hi form a contiguous block of
// binom(Lb, N - popcount(hi)) rows (at most 252 for Lb = 10) whose low parts
// run through the Lb-bit strings of that popcount in ascending order, so
//     rank(s) = hi_off[hi] + lo_rank[lo]
// and the position of a row inside its block is lo_rank[lo].
//
// Each wavefront processes a segment of one block (up to 128 rows, lanes on
// consecutive rows; a block of more rows is split into two segments, which
// both stage it: one segment per block, processed in two passes, measured
// slower since the second pass waits for the first).  Within a wavefront hi is uniform, hence:
//   - a hop inside the low part stays in the block.  The wavefront stages
//     the block's b_{i+1} entries in LDS once (coalesced) and reads those
//     neighbours from LDS at position lo_rank[lo'];
//   - a hop across a bond inside the high part moves to row r + d with a
//     wave-uniform d = hi_off[hi'] - hi_off[hi]: fully coalesced gathers;
//   - the bond joining the two parts and the periodic bond land in another
//     block at r + d + lo_rank[lo'] - lo_rank[lo] (d uniform);
//   - the diagonal is DLO[lo] (LDS) + a uniform high part + two cross terms.
// All wave-uniform data of a segment (offsets, flags, diagonal part) is
// precomputed into a 128-byte record read with scalar loads.  A high-part
// bond whose two bits are equal in the segment's high part cannot hop: its
// gather is skipped by a wave-uniform branch; the joining and periodic
// gathers are masked per lane.  All gathers of a lane's rows are issued
// before any is consumed, so they are in flight together.
//
// Locality: the eight XCDs each sweep a contiguous eighth of the segments
// (workgroups are dispatched to the XCDs round robin), so most high-part
// gathers of an XCD stay in its own L2; the streamed vectors v and b2 are
// read past the caches while they are small (see stream_nt).
#include <algorithm>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <tuple>
#include <utility>

#include "chain_dev.hpp"
#include "internal.hpp"

namespace polfed {

void build_chain_split(polfed_op* op) {
  const int L = op->L, N = op->N;
  const int Lb = std::min(kChainLoBits, L / 2), Lh = L - Lb;
  REQUIRE(Lh - 1 <= kChainMaxHighBonds, "chain: too many high bonds");
  const int nlo = 1 << Lb;
  // low parts: ranks within their popcount class, list grouped by popcount
  std::vector<int32_t> lo_rank(nlo), cnt(Lb + 1, 0), lo_base(Lb + 2, 0);
  for (int lo = 0; lo < nlo; ++lo) lo_rank[lo] = cnt[__builtin_popcount(lo)]++;
  for (int p = 0; p <= Lb; ++p) lo_base[p + 1] = lo_base[p] + cnt[p];
  std::vector<uint16_t> lolist(nlo);
  for (int lo = 0; lo < nlo; ++lo)
    lolist[lo_base[__builtin_popcount(lo)] + lo_rank[lo]] = (uint16_t)lo;
  // block positions of the low-bond neighbours (own position if no hop), then
  // the ranks of lo with its top bit and with bit 0 flipped (all < 256)
  std::vector<uint8_t> npos((size_t)nlo * 16, 0);
  for (int lo = 0; lo < nlo; ++lo) {
    uint8_t* q = &npos[(size_t)lo * 16];
    for (int b = 0; b + 1 < Lb; ++b) {
      const bool act = ((lo >> b) & 1) != ((lo >> (b + 1)) & 1);
      q[b] = (uint8_t)(act ? lo_rank[lo ^ (3 << b)] : lo_rank[lo]);
    }
    q[9] = (uint8_t)lo_rank[lo ^ (1 << (Lb - 1))];
    q[10] = (uint8_t)lo_rank[lo ^ 1];
    // the number of low bonds without a hop, and lo itself
    q[11] = (uint8_t)(Lb - 1 - __builtin_popcount((lo ^ (lo >> 1)) & ((1 << (Lb - 1)) - 1)));
    q[12] = (uint8_t)(lo & 255);
    q[13] = (uint8_t)(lo >> 8);
  }
  std::vector<double> dlo(nlo);
  for (int lo = 0; lo < nlo; ++lo) {
    double f = op->vzz * __builtin_popcount(lo & (lo >> 1));
    for (int i = 0; i < Lb; ++i)
      if ((lo >> i) & 1) f += op->site_f[i];
    dlo[lo] = f;
  }
  // high parts: first row of each block
  const int64_t nhi = (int64_t)1 << Lh;
  std::vector<int32_t> hi_off(nhi + 1, 0);
  int64_t acc = 0, nseg = 0;
  for (int64_t hi = 0; hi < nhi; ++hi) {
    hi_off[hi] = (int32_t)acc;
    const int need = N - __builtin_popcountll(hi);
    if (need < 0 || need > Lb) continue;
    acc += cnt[need];
    nseg += (cnt[need] + kChainSegRows - 1) / kChainSegRows;
  }
  hi_off[nhi] = (int32_t)acc;
  // one record per segment (room for all at once: while they grew, an operator
  // at L = 24 took 2.8 ms instead of 1.6)
  std::vector<int32_t> rec;
  rec.reserve((size_t)nseg * kChainRecWords);
  op->split_dseg.clear();
  op->split_dseg.reserve((size_t)nseg);
  for (int64_t hi = 0; hi < nhi; ++hi) {
    const int need = N - __builtin_popcountll(hi);
    if (need < 0 || need > Lb) continue;
    const int bs = cnt[need];
    const int hoff = hi_off[hi];
    double dhi = op->vzz * __builtin_popcountll(hi & (hi >> 1)) + op->c0;
    for (int i = 0; i < Lh; ++i)
      if ((hi >> i) & 1) dhi += op->site_f[Lb + i];
    int32_t w[kChainRecWords] = {0};
    int idle = 0;
    for (int b = 0; b + 1 < Lh; ++b) {
      const bool act = ((hi >> b) & 1) != ((hi >> (b + 1)) & 1);
      w[10 + b] = act ? hi_off[hi ^ (3LL << b)] - hoff : 0;
      idle += act ? 0 : 1;
    }
    w[4] = idle;
    for (int b = 0; b + 1 < Lh; ++b) w[4] |= (w[10 + b] != 0) << (8 + b);
    w[5] = hi_off[hi ^ 1] - hoff;
    // the joining hop of a row moves the particle between the bits Lb - 1 and
    // Lb past no other one, so it changes the rank by +-binom(Lb - 1, m) with
    // m the particles below: the same for every row of the block that can hop
    if (hi & 1)
      w[7] = need < Lb ? -(int32_t)host_binom()[(Lb - 1) * kBinomN + need] : 0;
    else
      w[7] = need > 0 ? (int32_t)host_binom()[(Lb - 1) * kBinomN + need - 1] : 0;
    w[6] = hi_off[hi ^ (1LL << (Lh - 1))] - hoff;
    std::memcpy(&w[8], &dhi, sizeof(double));
    const int nseg_hi = (bs + kChainSegRows - 1) / kChainSegRows;
    op->split_dseg.insert(op->split_dseg.end(), nseg_hi, dhi);
    for (int st = 0; st < bs; st += kChainSegRows) {
      w[0] = hoff + st;
      w[1] = std::min(kChainSegRows, bs - st);
      w[2] = lo_base[need] + st;
      w[3] = (int32_t)((hi & 1) | (((hi >> (Lh - 1)) & 1) << 1) | (bs << 2) | (st << 12));
      rec.insert(rec.end(), w, w + kChainRecWords);
    }
  }
  // field sums over low bits 0-4 and 5-9 (per-column diagonals of a batch)
  op->split_fab.assign(64, 0.0);
  for (int e = 0; e < 32; ++e)
    for (int k = 0; k < 5; ++k)
      if ((e >> k) & 1) {
        if (k < Lb) op->split_fab[e] += op->site_f[k];
        if (5 + k < Lb) op->split_fab[32 + e] += op->site_f[5 + k];
      }
  hipStream_t s = op->ctx->stream;
  op->split_Lb = Lb;
  op->split_nseg = (int64_t)(rec.size() / kChainRecWords);
  // packed LDS images: [neighbour positions | diagonal of the low part (T) |
  // low-part list], indexed by the low part; then the same three tables
  // indexed by position p in the low-part list (entry p describes lolist[p]),
  // so that a row's tables are one lookup away from its list position
  for (int w = 0; w < 2; ++w) {
    const int tb = w == 0 ? 8 : 4;
    std::vector<unsigned char> blob(chain_blob_bytes(nlo, tb), 0);
    unsigned char* p = blob.data();
    for (int q = 0; q < nlo; ++q) std::memcpy(p + 16 * q, &npos[(size_t)lolist[q] * 16], 16);
    p += 16 * (size_t)nlo;
    for (int q = 0; q < nlo; ++q) {
      if (tb == 8) {
        std::memcpy(p + 8 * q, &dlo[lolist[q]], 8);
      } else {
        const float f = (float)dlo[lolist[q]];
        std::memcpy(p + 4 * q, &f, 4);
      }
    }
    std::memcpy(p + (size_t)tb * nlo, lolist.data(), 2 * (size_t)nlo);
    upload(w == 0 ? op->d_blobl64 : op->d_blobl32, blob.data(), blob.size(), s);
  }
  for (int w = 0; w < 2; ++w) {
    const int tb = w == 0 ? 8 : 4;
    std::vector<unsigned char> blob(chain_blob_bytes(nlo, tb), 0);
    unsigned char* p = blob.data();
    std::memcpy(p, npos.data(), npos.size());
    p += npos.size();
    for (int lo = 0; lo < nlo; ++lo) {
      if (tb == 8) {
        std::memcpy(p + 8 * lo, &dlo[lo], 8);
      } else {
        const float f = (float)dlo[lo];
        std::memcpy(p + 4 * lo, &f, 4);
      }
    }
    std::memcpy(p + (size_t)tb * nlo, lolist.data(), 2 * (size_t)nlo);
    upload(w == 0 ? op->d_blob64 : op->d_blob32, blob.data(), blob.size(), s);
  }
  upload(op->d_rec, rec.data(), rec.size(), s);
  // tiles of 2^KT consecutive high parts (segments are in ascending hi), for
  // the largest KT with at least 512 tiles and for KT - 1
  std::vector<int32_t> seg_of_hi(nhi + 1, 0);
  {
    int32_t sidx = 0;
    for (int64_t hi = 0; hi < nhi; ++hi) {
      seg_of_hi[hi] = sidx;
      const int need = N - __builtin_popcountll(hi);
      if (need >= 0 && need <= Lb) sidx += (cnt[need] + kChainSegRows - 1) / kChainSegRows;
    }
    seg_of_hi[nhi] = sidx;
  }
  op->split_hi_off = hi_off;
  op->split_seg_of_hi = seg_of_hi;
  op->wtiles.clear();
  const int KT = chain_tile_bits(L);
  for (int v = 0; v < 3; ++v) {
    auto& T = op->tiles[v];
    T = polfed_op::Tiles{};
    const int kt = KT - v;
    if (KT == 0 || kt < 2) continue;
    const int64_t nt = (int64_t)1 << (Lh - kt);
    std::vector<int32_t> tiles((size_t)nt * 4, 0);
    for (int64_t t = 0; t < nt; ++t) {
      const int64_t h0 = t << kt, h1 = (t + 1) << kt;
      tiles[4 * t] = hi_off[h0];
      tiles[4 * t + 1] = hi_off[h1] - hi_off[h0];
      tiles[4 * t + 2] = seg_of_hi[h0];
      tiles[4 * t + 3] = seg_of_hi[h1] - seg_of_hi[h0];
      T.max_rows = std::max(T.max_rows, tiles[4 * t + 1]);
    }
    T.bits = kt;
    T.n = (int)nt;
    upload(T.d, tiles.data(), tiles.size(), s);
  }
  op->tuned[0] = op->tuned[1] = -1;
  HIPC(hipStreamSynchronize(s));
}

// HALVES = 2 splits every segment between two wavefronts (64 rows each, one
// row per lane): twice the independent wavefronts, each with half the
// dependent work, for chains too short to fill the chip.
template <typename T, int L, int HALVES = 1>
__global__ __launch_bounds__(256) void k_chain_split(
    ChainSplitDev c, T sigma, T tau, T a, const T* __restrict__ v,
    const T* __restrict__ b1, const T* b2, T* out, int nxcd,
    const int32_t* __restrict__ recs) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int Lh = L - Lb;
  constexpr int NLO = 1 << Lb;
  constexpr int NH = Lh - 1;  // bonds inside the high part
  constexpr int NL = Lb - 1;  // bonds inside the low part
  constexpr int RPL = 2 / HALVES;               // rows per lane and pass
  constexpr int kPasses = kChainSegRows / 128;  // passes per segment
  constexpr int SPL = kChainStageRows / 64;  // staged rows per lane
  constexpr int BLOB = chain_blob_bytes(NLO, (int)sizeof(T));
  constexpr int CHUNKS = BLOB / 16;
  constexpr uint32_t TB = sizeof(T);
  using u4 = __attribute__((ext_vector_type(4))) uint32_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  {  // one vectorized, unrolled copy of the packed tables into LDS
    const u4* src = reinterpret_cast<const u4*>(sizeof(T) == 8 ? c.blob64 : c.blob32);
    u4* dst = reinterpret_cast<u4*>(smem);
    constexpr int PER = (CHUNKS + 255) / 256;
    u4 tmp[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < CHUNKS) tmp[k] = src[i];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < CHUNKS) dst[i] = tmp[k];
    }
  }
  const u4* s_np = reinterpret_cast<const u4*>(smem);
  const T* s_dlo = reinterpret_cast<const T*>(smem + 16 * NLO);
  const uint16_t* s_lo = reinterpret_cast<const uint16_t*>(s_dlo + NLO);
  T* stage = reinterpret_cast<T*>(smem + BLOB) + (threadIdx.x >> 6) * kChainStageRows;
  __syncthreads();

  // this XCD's contiguous share of the segments
  const int xcd = blockIdx.x % nxcd;
  const int blocks_x = gridDim.x / nxcd;
  const int64_t nvirt = c.nseg * HALVES;  // (segment, half) work items
  const int64_t s_begin = nvirt * xcd / nxcd, s_end = nvirt * (xcd + 1) / nxcd;
  const int wpb = blockDim.x >> 6;
  const int64_t wstride = (int64_t)blocks_x * wpb;
  const int lane = threadIdx.x & 63;
  const T vzz = (T)c.vzz, t_in = (T)c.t_in, t_pb = (T)c.t_pb;
  const bool nt = stream_nt<T>(c.D);
  const uint32_t vbytes = (uint32_t)(c.D * TB);
  const rsrc_t rb1 = make_rsrc(b1, vbytes), rv = make_rsrc(v, v ? vbytes : 0),
               rb2 = make_rsrc(b2, b2 ? vbytes : 0), rout = make_rsrc(out, vbytes);
  int64_t vi = s_begin + (int64_t)(blockIdx.x / nxcd) * wpb + uniform(threadIdx.x >> 6);
  if (vi >= s_end) return;
  for (; vi < s_end; vi += wstride) {
    const int64_t si = vi / HALVES;
    const int half = (int)(vi % HALVES);
    const SegRec<NH> cur = load_rec<NH>(recs + (int64_t)uniform((int)si) * kChainRecWords);
    if (half * 64 >= cur.len) continue;
    const int hi0 = cur.flags & 1, hitop = (cur.flags >> 1) & 1;
    const int bs = (cur.flags >> 2) & 1023, st = (cur.flags >> 12) & 1023;
    const int blk0 = cur.row0 - st;
    const uint32_t so_blk = (uint32_t)blk0 * TB, so_row = (uint32_t)cur.row0 * TB;
    // the block of b_{i+1} for the low-part hops: loads now, LDS later
    T stg[SPL];
#pragma unroll
    for (int m = 0; m < SPL; ++m)
      stg[m] = 64 * m < bs ? bload<T>(rb1, (uint32_t)min(lane + 64 * m, bs - 1) * TB, so_blk)
                           : T(0);
    // the segment's rows in passes of 128 (two rows per lane); the block is
    // staged in LDS by the first pass
    for (int pass = 0; pass < kPasses; ++pass) {
      const int p0 = pass * 128 + half * 64;
      if (p0 >= cur.len) break;
      // rows of this lane, clamped into the segment (a clamped lane repeats
      // the last row and stores the same value)
      int jj[RPL], lo[RPL];
      u4 np[RPL];
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        jj[i] = min(p0 + lane + 64 * i, cur.len - 1);
        lo[i] = s_lo[cur.lidx + jj[i]];
        np[i] = s_np[lo[i]];
      }
      // global gathers: high-part hops at uniform offsets, joining and
      // periodic bonds, and the streamed v and b_{i+2}
      T g_hi[RPL][NH > 0 ? NH : 1], g_j[RPL], g_p[RPL], vv[RPL], bt[RPL];
      bool act_j[RPL], act_p[RPL];
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const uint32_t off = (uint32_t)jj[i] * TB;
#pragma unroll
        for (int b = 0; b < NH; ++b)
          g_hi[i][b] = cur.dh[b] != 0
                           ? bload<T>(rb1, off, (uint32_t)(cur.row0 + cur.dh[b]) * TB)
                           : T(0);
        const int l = lo[i];
        act_j[i] = ((l >> (Lb - 1)) & 1) != hi0;
        act_p[i] = c.periodic && ((l & 1) != hitop);
        const int rj = (int)((np[i][2] >> 8) & 255u);   // byte 9
        const int rp = (int)((np[i][2] >> 16) & 255u);  // byte 10
        g_j[i] = act_j[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_join + rj) * TB, 0) : T(0);
        g_p[i] = act_p[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_pbc + rp) * TB, 0) : T(0);
        vv[i] = bt[i] = T(0);
        if (v) bload_stream<T>(rv, off, so_row, nt, &vv[i]);
        if (b2) bload_stream<T>(rb2, off, so_row, nt, &bt[i]);
      }
      if (pass == 0) {
        wave_sync();  // the previous segment's LDS reads are done
#pragma unroll
        for (int m = 0; m < SPL; ++m)
          if (64 * m < bs) stage[min(lane + 64 * m, bs - 1)] = stg[m];
        wave_sync();
      }
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int l = lo[i];
        const T bo = stage[st + jj[i]];
        T hop = 0;
#pragma unroll
        for (int b = 0; b < NL; ++b) hop += stage[(np[i][b >> 2] >> (8 * (b & 3))) & 255u];
#pragma unroll
        for (int b = 0; b < NH; ++b) hop += g_hi[i][b];
        const int xlo = (l ^ (l >> 1)) & ((1 << NL) - 1);
        const int n_idle = NL - __popc(xlo);
        hop -= (T)n_idle * bo;
        hop += act_j[i] ? g_j[i] : T(0);
        const int lo_top = (l >> (Lb - 1)) & 1, lo0 = l & 1;
        const int n11x = (lo_top & hi0) + (c.periodic ? (hitop & lo0) : 0);
        const T dg = s_dlo[l] + (T)cur.dhi + vzz * (T)n11x;
        const T acc = dg * bo + t_in * hop + (act_p[i] ? t_pb * g_p[i] : T(0));
        T o = sigma * acc + tau * bo - bt[i];
        if (v) o += a * vv[i];
        bstore<kAuxNT>(o, rout, (uint32_t)jj[i] * TB, so_row);
      }
    }
  }
}

// Direct kernel: a wavefront takes one segment, lane l the adjacent rows 2l
// and 2l + 1, so that every coalesced access moves both rows in one 16-byte
// instruction.  Made for chains where a wavefront runs one or two segments a
// launch (up to L = 21: a step is then a chain of round trips, not bytes):
//   - a row's low-part tables are read from global memory in list order (26
//     bytes a row, coalesced) with the rest, instead of a 27 KB copy into LDS
//     per workgroup that everything else waits for;
//   - the joining bond is one more gather at a wave-uniform row offset (see
//     build_chain_split), so only the periodic bond waits for the tables.
// With MULTI the columns of a column-major block are spread over the XCDs
// (8, 4, 2 or 1 of them a column), so a column's gathers stay in its XCDs'
// L2; each column has its operator's records and tables, or all have one
// operator's (cols null: H on the columns of a block).
//
// A bond without a hop in the segment is passed by with a branch both where it
// is loaded and where it is added; the empty asm keeps the compiler from
// adding zeros instead.
//
// Measured (FP64, L = 20, us a step): 4 columns 13.5 (interleaved) -> 9.6, one
// column launched one by one 6.8 (segment kernel) -> 5.9.
//
// Loads past the segment's end read other rows (unused) or fall outside the
// buffer (read as 0); stores are guarded per row.
template <typename T, int L, bool MULTI>
__global__ __launch_bounds__(256) void k_chain_direct(
    ChainSplitDev c, T sigma, T tau, T a, const ChainCol* __restrict__ cols, int ncol, int nb,
    const T* __restrict__ sc, const T* __restrict__ acoef, T half, const T* __restrict__ v,
    const T* __restrict__ b1, const T* b2, T* out, int nxcd, int xpc) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int Lh = L - Lb;
  constexpr int NLO = 1 << Lb;
  constexpr int NH = Lh - 1;
  constexpr int NL = Lb - 1;
  constexpr int SPL = kChainStageRows / 128;  // staged row pairs per lane
  constexpr uint32_t TB = sizeof(T);
  using u4 = __attribute__((ext_vector_type(4))) uint32_t;
  __shared__ __attribute__((aligned(16))) T s_stage[4 * kChainStageRows];
  T* stage = s_stage + (threadIdx.x >> 6) * kChainStageRows;
  const int xcd = blockIdx.x % nxcd;
  const int lane = threadIdx.x & 63;
  const T vzz = (T)c.vzz, t_in = (T)c.t_in, t_pb = (T)c.t_pb;
  const bool nt = stream_nt<T>(MULTI ? c.D * ncol : c.D);
  const uint32_t vbytes = (uint32_t)(c.D * TB);
  // this XCD's share: segments [s_begin, s_begin + nsx) of the columns
  // first, first + step, ...
  const int part = MULTI ? xcd % xpc : xcd, parts = MULTI ? xpc : nxcd;
  const int s_begin = (int)(c.nseg * part / parts);
  const int nsx = (int)(c.nseg * (part + 1) / parts) - s_begin;
  const int first = MULTI ? xcd / xpc : 0, step = MULTI ? nxcd / xpc : 1;
  const int ncx = MULTI ? (ncol - first + step - 1) / step : 1;
  const int64_t items = (int64_t)nsx * max(ncx, 0);
  const int64_t stride = (int64_t)(gridDim.x / nxcd) * 4;
  for (int64_t it = (int64_t)(blockIdx.x / nxcd) * 4 + uniform(threadIdx.x >> 6); it < items;
       it += stride) {
    const int k = MULTI ? (int)(it / nsx) : 0;
    const int si = uniform(s_begin + (int)(it - (int64_t)k * nsx));
    const int col = uniform(first + k * step);
    const int64_t coff = MULTI ? (int64_t)col * c.D : 0;
    const bool own = MULTI && cols;  // the columns' own operators, or one for all
    const int32_t* recs = own ? cols[col].rec : c.rec;
    const unsigned char* blob = reinterpret_cast<const unsigned char*>(
        sizeof(T) == 8 ? (own ? cols[col].blobl64 : c.blobl64)
                       : (own ? cols[col].blobl32 : c.blobl32));
    const rsrc_t rb1 = make_rsrc(b1 + coff, vbytes), rv = make_rsrc(v ? v + coff : b1, v ? vbytes : 0),
                 rb2 = make_rsrc(b2 ? b2 + coff : b1, b2 ? vbytes : 0),
                 rout = make_rsrc(out + coff, vbytes);
    const rsrc_t rnp = make_rsrc(blob, 16 * NLO), rdl = make_rsrc(blob + 16 * NLO, TB * NLO);
    const int32_t* rec = recs + (int64_t)si * kChainRecWords;
    const SegRec<NH> cur = load_rec<NH>(rec);
    const int d_near = uniform(rec[7]);
    uint32_t act = (uint32_t)uniform(rec[4]) >> 8;  // high bonds with a hop
    const int hi0 = cur.flags & 1, hitop = (cur.flags >> 1) & 1;
    const int bs = (cur.flags >> 2) & 1023, st = (cur.flags >> 12) & 1023;
    const int blk0 = cur.row0 - st;
    const uint32_t so_blk = (uint32_t)blk0 * TB, so_row = (uint32_t)cur.row0 * TB;
    const uint32_t pair_off = (uint32_t)(2 * lane) * TB;
    // the lane's two rows, clamped into the segment, and their tables
    int jj[2];
    u4 np[2];
    T dl[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      jj[i] = min(2 * lane + i, cur.len - 1);
      const uint32_t q = (uint32_t)(cur.lidx + jj[i]);
      np[i] = __builtin_amdgcn_raw_buffer_load_b128(rnp, 16 * q, 0, 0);
      dl[i] = bload<T>(rdl, TB * q, 0);
    }
    T sg[SPL][2], g_hi[NH > 0 ? NH : 1][2], g_j[2], vv[2], bt[2];
#pragma unroll
    for (int m = 0; m < SPL; ++m) {
      if (128 * m < bs)
        bload2<T>(rb1, pair_off + (uint32_t)(128 * m) * TB, so_blk, sg[m][0], sg[m][1]);
      else
        sg[m][0] = sg[m][1] = T(0);
    }
#pragma unroll
    for (int b = 0; b < NH; ++b) {
      if ((act >> b) & 1u) {
        asm volatile("");
        bload2<T>(rb1, pair_off, (uint32_t)(cur.row0 + cur.dh[b]) * TB, g_hi[b][0], g_hi[b][1]);
      }
    }
    if (d_near != 0)
      bload2<T>(rb1, pair_off + (uint32_t)((cur.row0 + d_near) * (int)TB), 0, g_j[0], g_j[1]);
    else
      g_j[0] = g_j[1] = T(0);
    if (v)
      bload_stream<T, 2>(rv, pair_off, so_row, nt, vv);
    else
      vv[0] = vv[1] = T(0);
    if (b2)
      bload_stream<T, 2>(rb2, pair_off, so_row, nt, bt);
    else
      bt[0] = bt[1] = T(0);
    bool act_j[2], act_p[2];
    T g_p[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      act_j[i] = (int)((np[i][3] >> (Lb - 1)) & 1u) != hi0;
      act_p[i] = c.periodic && (int)(np[i][3] & 1u) != hitop;
      const int rp = (int)((np[i][2] >> 16) & 255u);
      g_p[i] = act_p[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_pbc + rp) * TB, 0) : T(0);
    }
    wave_sync();  // the previous segment's LDS reads are done
#pragma unroll
    for (int m = 0; m < SPL; ++m) {
      const int r = 128 * m + 2 * lane;
      if (r < bs) {
        stage[r] = sg[m][0];
        if (r + 1 < bs) stage[r + 1] = sg[m][1];
      }
    }
    wave_sync();
    const T sig = own ? half * sc[col] : sigma, ta = own ? half * sc[nb + col] : tau;
    const T ac = own ? (acoef ? acoef[col] : T(0)) : a;
    T o[2], bo[2], hop[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      bo[i] = stage[st + jj[i]];
      T h = 0;
#pragma unroll
      for (int b = 0; b < NL; ++b) h += stage[(np[i][b >> 2] >> (8 * (b & 3))) & 255u];
      hop[i] = h - (T)(int)(np[i][2] >> 24) * bo[i];  // idle low bonds read the row itself
    }
    // (reread, or the first tests' results are held in registers)
    asm volatile("" : "+s"(act));
#pragma unroll
    for (int b = 0; b < NH; ++b) {
      if ((act >> b) & 1u) {
        asm volatile("");
        hop[0] += g_hi[b][0];
        hop[1] += g_hi[b][1];
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      hop[i] += act_j[i] ? g_j[i] : T(0);
      const int lo_top = (int)((np[i][3] >> (Lb - 1)) & 1u), lo0 = (int)(np[i][3] & 1u);
      const int n11x = (lo_top & hi0) + (c.periodic ? (hitop & lo0) : 0);
      const T dg = dl[i] + (T)cur.dhi + vzz * (T)n11x;
      const T acc = dg * bo[i] + t_in * hop[i] + (act_p[i] ? t_pb * g_p[i] : T(0));
      o[i] = sig * acc + ta * bo[i] - bt[i];
      if (v) o[i] += ac * vv[i];
    }
    const int r0 = 2 * lane;
    if (r0 + 1 < cur.len)
      bstore2<kAuxNT>(o[0], o[1], rout, pair_off, so_row);
    else if (r0 < cur.len)
      bstore<kAuxNT>(o[0], rout, pair_off, so_row);
  }
}

template <typename T, int L>
static void launch_direct(hipStream_t s, const polfed_op* op, T sigma, T tau, T a, const T* v,
                          const T* b1, const T* b2, T* out) {
  ChainSplitDev c = op->chain_split();
  int64_t grid = std::min<int64_t>((c.nseg + 3) / 4, (int64_t)op->ctx->n_cu * kChainBlocksPerCU);
  int nxcd = 1;
  if (grid >= 64) {
    grid = (grid + 7) / 8 * 8;
    nxcd = 8;
  }
  grid = std::max<int64_t>(grid, 1);
  hipLaunchKernelGGL((k_chain_direct<T, L, false>), dim3((unsigned)grid), dim3(256), 0, s, c, sigma, tau, a, (const ChainCol*)nullptr, 1, 1, (const T*)nullptr,
                     (const T*)nullptr, T(1), v, b1, b2, out, nxcd, 1);
  HIPC(hipGetLastError());
}

// Columns [col0, col0 + ncol) of a batch, one step (see k_chain_direct).
template <typename T, int L>
static void launch_direct_cols(hipStream_t s, const ChainBatch& bt, int col0, int ncol, T half,
                               const T* acoef, const T* v, const T* b1, const T* b2, T* out) {
  const polfed_op* op0 = bt.ops[0];
  ChainSplitDev c = op0->chain_split();
  int xpc = 8;
  while (xpc > 1 && xpc * ncol > 8) xpc /= 2;
  const int64_t per = (c.nseg / xpc + 1) * ((ncol + 8 / xpc - 1) / (8 / xpc));  // items of an XCD
  int64_t grid = 8 * std::min<int64_t>((per + 3) / 4, (int64_t)op0->ctx->n_cu * kChainBlocksPerCU / 8);
  const bool f64 = sizeof(T) == 8;
  const T* sc = (const T*)(f64 ? bt.sc64.get() : bt.sc32.get());
  const size_t o = (size_t)col0 * op0->D;
  hipLaunchKernelGGL((k_chain_direct<T, L, true>), dim3((unsigned)std::max<int64_t>(grid, 8)),
                     dim3(256), 0, s, c, T(0), T(0), T(0), bt.cols.as<ChainCol>() + col0, ncol,
                     bt.nb, sc + col0, acoef ? acoef + col0 : nullptr, half, v ? v + o : nullptr,
                     b1 + o, b2 ? b2 + o : nullptr, out + o, 8, xpc);
  HIPC(hipGetLastError());
}

// out = H x for n vectors of one operator, column-major.
template <int L>
static void launch_direct_block(hipStream_t s, const polfed_op* op, int n, const double* x,
                                double* out) {
  ChainSplitDev c = op->chain_split();
  int xpc = 8;
  while (xpc > 1 && xpc * n > 8) xpc /= 2;
  const int64_t per = (c.nseg / xpc + 1) * ((n + 8 / xpc - 1) / (8 / xpc));  // items of an XCD
  const int64_t grid =
      8 * std::min<int64_t>((per + 3) / 4, (int64_t)op->ctx->n_cu * kChainBlocksPerCU / 8);
  hipLaunchKernelGGL((k_chain_direct<double, L, true>), dim3((unsigned)std::max<int64_t>(grid, 8)),
                     dim3(256), 0, s, c, 1.0, 0.0, 0.0, (const ChainCol*)nullptr, n, n,
                     (const double*)nullptr, (const double*)nullptr, 1.0, (const double*)nullptr,
                     x, (const double*)nullptr, out, 8, xpc);
  HIPC(hipGetLastError());
}

// H on the columns of a block in one launch, where a launch a column is mostly
// its own latency: below the paired kernel's chains (L = 20, 120 columns:
// 180 us, a launch a column 590).  False: not done.
bool chain_apply_block(hipStream_t s, const polfed_op* op, int n, const double* x, double* out) {
  if (n < 2 || op->model != Model::Chain || op->storage != POLFED_MATRIX_FREE ||
      op->split_nseg <= 0 || op->forced[0])
    return false;
  switch (op->L) {
#define POLFED_CASE(LL)                           \
  case LL:                                        \
    launch_direct_block<LL>(s, op, n, x, out);    \
    return true;
    POLFED_CASE(4) POLFED_CASE(5) POLFED_CASE(6) POLFED_CASE(7) POLFED_CASE(8)
    POLFED_CASE(9) POLFED_CASE(10) POLFED_CASE(11) POLFED_CASE(12) POLFED_CASE(13)
    POLFED_CASE(14) POLFED_CASE(15) POLFED_CASE(16) POLFED_CASE(17) POLFED_CASE(18)
    POLFED_CASE(19) POLFED_CASE(20) POLFED_CASE(21)
#undef POLFED_CASE
    default: return false;
  }
}

template <typename T>
void chain_direct_cols(hipStream_t s, const ChainBatch& bt, int col0, int ncol, T half,
                       const T* acoef, const T* v, const T* b1, const T* b2, T* out) {
  switch (bt.ops[0]->L) {
#define POLFED_CASE(LL)                                                                     \
  case LL:                                                                                  \
    launch_direct_cols<T, LL>(s, bt, col0, ncol, half, acoef, v, b1, b2, out);              \
    break;
    POLFED_CASE(4) POLFED_CASE(5) POLFED_CASE(6) POLFED_CASE(7) POLFED_CASE(8)
    POLFED_CASE(9) POLFED_CASE(10) POLFED_CASE(11) POLFED_CASE(12) POLFED_CASE(13)
    POLFED_CASE(14) POLFED_CASE(15) POLFED_CASE(16) POLFED_CASE(17) POLFED_CASE(18)
    POLFED_CASE(19) POLFED_CASE(20) POLFED_CASE(21) POLFED_CASE(22) POLFED_CASE(23)
    POLFED_CASE(24) POLFED_CASE(25) POLFED_CASE(26) POLFED_CASE(27) POLFED_CASE(28)
#undef POLFED_CASE
    default: fail(POLFED_ERR_INVALID, "batch: chain length outside 4..28");
  }
}
template void chain_direct_cols<double>(hipStream_t, const ChainBatch&, int, int, double,
                                        const double*, const double*, const double*,
                                        const double*, double*);
template void chain_direct_cols<float>(hipStream_t, const ChainBatch&, int, int, float,
                                       const float*, const float*, const float*, const float*,
                                       float*);

constexpr int kPairedFirst = 22;  // variant 3 is the paired kernel from here on

// Paired variant: the direct kernel for chains where a wavefront runs many
// segments, so that the low-part tables are worth a copy into LDS, and what
// counts is the traffic of the gathers: the joining bond is gathered by the
// rows that hop only (us a step, direct / paired: FP32 L = 22 9.5 / 8.6,
// L = 24 22.1 / 17.4, FP64 L = 23 16.0 / 15.7; FP64 L = 20 5.9 / 6.4, L = 21
// 7.9 / 8.0).  The tables are in list order and carry the low part and the
// number of idle low bonds, so a row's LDS reads are one round trip (FP32
// L = 23, 10 up, open: 10.55 -> 10.2).  Four workgroups a CU: six take 28.4
// instead of 25.3 (FP64 L = 24, open), three 11.3 instead of 10.2 (FP32).
template <typename T, int L>
__global__ __launch_bounds__(256) void k_chain_pair(
    ChainSplitDev c, T sigma, T tau, T a, const T* __restrict__ v,
    const T* __restrict__ b1, const T* b2, T* out, int nxcd,
    const int32_t* __restrict__ recs) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int Lh = L - Lb;
  constexpr int NLO = 1 << Lb;
  constexpr int NH = Lh - 1;
  constexpr int NL = Lb - 1;
  constexpr int SPL = kChainStageRows / 128;  // staged row pairs per lane
  constexpr int BLOB = wt_blob_bytes(NLO, (int)sizeof(T));
  constexpr int CHUNKS = BLOB / 16;
  constexpr uint32_t TB = sizeof(T);
  using u4 = __attribute__((ext_vector_type(4))) uint32_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  {
    const u4* src = reinterpret_cast<const u4*>(sizeof(T) == 8 ? c.blobl64 : c.blobl32);
    u4* dst = reinterpret_cast<u4*>(smem);
    constexpr int PER = (CHUNKS + 255) / 256;
    u4 tmp[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < CHUNKS) tmp[k] = src[i];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < CHUNKS) dst[i] = tmp[k];
    }
  }
  const u4* s_np = reinterpret_cast<const u4*>(smem);
  const T* s_dlo = reinterpret_cast<const T*>(smem + 16 * NLO);
  T* stage = reinterpret_cast<T*>(smem + BLOB) + (threadIdx.x >> 6) * kChainStageRows;
  __syncthreads();

  const int xcd = blockIdx.x % nxcd;
  const int blocks_x = gridDim.x / nxcd;
  const int64_t s_begin = c.nseg * xcd / nxcd, s_end = c.nseg * (xcd + 1) / nxcd;
  const int wpb = blockDim.x >> 6;
  const int64_t wstride = (int64_t)blocks_x * wpb;
  const int lane = threadIdx.x & 63;
  const T vzz = (T)c.vzz, t_in = (T)c.t_in, t_pb = (T)c.t_pb;
  const bool nt = stream_nt<T>(c.D);
  const uint32_t vbytes = (uint32_t)(c.D * TB);
  const rsrc_t rb1 = make_rsrc(b1, vbytes), rv = make_rsrc(v, v ? vbytes : 0),
               rb2 = make_rsrc(b2, b2 ? vbytes : 0), rout = make_rsrc(out, vbytes);
  int64_t si = s_begin + (int64_t)(blockIdx.x / nxcd) * wpb + uniform(threadIdx.x >> 6);
  if (si >= s_end) return;
  for (; si < s_end; si += wstride) {
    const SegRec<NH> cur = load_rec<NH>(recs + (int64_t)uniform((int)si) * kChainRecWords);
    const int hi0 = cur.flags & 1, hitop = (cur.flags >> 1) & 1;
    const int bs = (cur.flags >> 2) & 1023, st = (cur.flags >> 12) & 1023;
    const int blk0 = cur.row0 - st;
    const uint32_t so_blk = (uint32_t)blk0 * TB, so_row = (uint32_t)cur.row0 * TB;
    const uint32_t pair_off = (uint32_t)(2 * lane) * TB;
    // stage the block: pairs of rows
    T sg[SPL][2];
#pragma unroll
    for (int m = 0; m < SPL; ++m) {
      if (128 * m < bs)
        bload2<T>(rb1, pair_off + (uint32_t)(128 * m) * TB, so_blk, sg[m][0], sg[m][1]);
      else
        sg[m][0] = sg[m][1] = T(0);
    }
    // the lane's two rows, clamped into the segment
    int jj[2];
    u4 np[2];
    bool act_j[2], act_p[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      jj[i] = min(2 * lane + i, cur.len - 1);
      np[i] = s_np[cur.lidx + jj[i]];
      act_j[i] = (int)((np[i][3] >> (Lb - 1)) & 1u) != hi0;
      act_p[i] = c.periodic && (int)(np[i][3] & 1u) != hitop;
    }
    T g_hi[NH > 0 ? NH : 1][2], g_j[2], g_p[2], vv[2], bt[2];
#pragma unroll
    for (int b = 0; b < NH; ++b) {
      if (cur.dh[b] != 0)
        bload2<T>(rb1, pair_off, (uint32_t)(cur.row0 + cur.dh[b]) * TB, g_hi[b][0], g_hi[b][1]);
      else
        g_hi[b][0] = g_hi[b][1] = T(0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int rj = (int)((np[i][2] >> 8) & 255u);
      const int rp = (int)((np[i][2] >> 16) & 255u);
      g_j[i] = act_j[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_join + rj) * TB, 0) : T(0);
      g_p[i] = act_p[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_pbc + rp) * TB, 0) : T(0);
    }
    if (v)
      bload_stream<T, 2>(rv, pair_off, so_row, nt, vv);
    else
      vv[0] = vv[1] = T(0);
    if (b2)
      bload_stream<T, 2>(rb2, pair_off, so_row, nt, bt);
    else
      bt[0] = bt[1] = T(0);
    wave_sync();  // the previous segment's LDS reads are done
#pragma unroll
    for (int m = 0; m < SPL; ++m) {
      const int r = 128 * m + 2 * lane;
      if (r < bs) {
        stage[r] = sg[m][0];
        if (r + 1 < bs) stage[r + 1] = sg[m][1];
      }
    }
    wave_sync();
    T o[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int l = (int)np[i][3];
      const T bo = stage[st + jj[i]];
      T hop = 0;
#pragma unroll
      for (int b = 0; b < NL; ++b) hop += stage[(np[i][b >> 2] >> (8 * (b & 3))) & 255u];
#pragma unroll
      for (int b = 0; b < NH; ++b) hop += g_hi[b][i];
      hop -= (T)(int)(np[i][2] >> 24) * bo;  // idle low bonds read the row itself
      hop += act_j[i] ? g_j[i] : T(0);
      const int lo_top = (l >> (Lb - 1)) & 1, lo0 = l & 1;
      const int n11x = (lo_top & hi0) + (c.periodic ? (hitop & lo0) : 0);
      const T dg = s_dlo[cur.lidx + jj[i]] + (T)cur.dhi + vzz * (T)n11x;
      const T acc = dg * bo + t_in * hop + (act_p[i] ? t_pb * g_p[i] : T(0));
      o[i] = sigma * acc + tau * bo - bt[i];
      if (v) o[i] += a * vv[i];
    }
    const int r0 = 2 * lane;
    if (r0 + 1 < cur.len)
      bstore2<kAuxNT>(o[0], o[1], rout, pair_off, so_row);
    else if (r0 < cur.len)
      bstore<kAuxNT>(o[0], rout, pair_off, so_row);
  }
}

template <typename T, int L>
static void launch_pair(hipStream_t s, const polfed_op* op, T sigma, T tau, T a, const T* v,
                        const T* b1, const T* b2, T* out) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int NLO = 1 << Lb;
  const size_t shm = wt_blob_bytes(NLO, (int)sizeof(T)) + 4 * kChainStageRows * sizeof(T);
  const int bpc = std::max(1, std::min(kChainBlocksPerCU, (int)(kLdsPerCU / shm)));
  ChainSplitDev c = op->chain_split();
  const int64_t blocks_needed = (c.nseg + 3) / 4;
  int64_t grid = std::min<int64_t>(blocks_needed, (int64_t)op->ctx->n_cu * bpc);
  int nxcd = 1;
  if (grid >= 64) {
    grid -= grid % 8;
    nxcd = 8;
  }
  grid = std::max<int64_t>(grid, 1);
  hipLaunchKernelGGL((k_chain_pair<T, L>), dim3((unsigned)grid), dim3(256), shm, s, c, sigma,
                     tau, a, v, b1, b2, out, nxcd, c.rec);
  HIPC(hipGetLastError());
}

// Tile variant for long chains: a workgroup stages a whole tile of 2^KT
// consecutive high parts of b_{i+1} in LDS (one coalesced read of its rows),
// so the low-part hops, the joining bond (high bit 0) and the KT - 1 bonds
// inside the tile's high bits are LDS reads; only the bonds among the
// remaining high bits and the periodic bond gather from global memory.  The
// tile's segments are shared among the workgroup's wavefronts; each lane
// holds two adjacent rows, as in the paired kernel.
template <typename T, int L, int KT>
__global__ __launch_bounds__(kTileThreads) void k_chain_tile(
    ChainSplitDev c, T sigma, T tau, T a, const T* __restrict__ v,
    const T* __restrict__ b1, const T* b2, T* out, int nxcd, int ntiles,
    const int32_t* __restrict__ recs, const int32_t* __restrict__ tiles) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int Lh = L - Lb;
  constexpr int NLO = 1 << Lb;
  constexpr int NH = Lh - 1;   // bonds inside the high part
  constexpr int NHL = KT - 1;  // of which inside the tile: b < NHL
  constexpr int NL = Lb - 1;
  constexpr int BLOB = chain_blob_bytes(NLO, (int)sizeof(T));
  constexpr int CHUNKS = BLOB / 16;
  constexpr uint32_t TB = sizeof(T);
  using u4 = __attribute__((ext_vector_type(4))) uint32_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  {
    const u4* src = reinterpret_cast<const u4*>(sizeof(T) == 8 ? c.blob64 : c.blob32);
    u4* dst = reinterpret_cast<u4*>(smem);
    for (int i = threadIdx.x; i < CHUNKS; i += kTileThreads) dst[i] = src[i];
  }
  const u4* s_np = reinterpret_cast<const u4*>(smem);
  const T* s_dlo = reinterpret_cast<const T*>(smem + 16 * NLO);
  const uint16_t* s_lo = reinterpret_cast<const uint16_t*>(s_dlo + NLO);
  T* s_tile = reinterpret_cast<T*>(smem + BLOB);

  const int xcd = blockIdx.x % nxcd;
  const int wg = blockIdx.x / nxcd, nwg = gridDim.x / nxcd;
  const int t_begin = (int)((int64_t)ntiles * xcd / nxcd);
  const int t_end = (int)((int64_t)ntiles * (xcd + 1) / nxcd);
  const int wave = uniform(threadIdx.x >> 6);
  constexpr int NW = kTileThreads / 64;
  const int lane = threadIdx.x & 63;
  const T vzz = (T)c.vzz, t_in = (T)c.t_in, t_pb = (T)c.t_pb;
  const bool nt = stream_nt<T>(c.D);
  const uint32_t vbytes = (uint32_t)(c.D * TB);
  const rsrc_t rb1 = make_rsrc(b1, vbytes), rv = make_rsrc(v, v ? vbytes : 0),
               rb2 = make_rsrc(b2, b2 ? vbytes : 0), rout = make_rsrc(out, vbytes);
  for (int t = t_begin + wg; t < t_end; t += nwg) {
    const int trow0 = tiles[4 * t], trows = tiles[4 * t + 1];
    const int tseg0 = tiles[4 * t + 2], tnseg = tiles[4 * t + 3];
    __syncthreads();  // the previous tile's LDS reads are done (and the tables)
    {  // two rows per thread and access; rows past the tile are not stored
      constexpr int U = 4;
      const uint32_t so = (uint32_t)trow0 * TB;
      for (int i0 = 0; i0 < trows; i0 += 2 * U * kTileThreads) {
        T x[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + 2 * (u * kTileThreads + (int)threadIdx.x);
          if (i < trows)
            bload2<T>(rb1, (uint32_t)i * TB, so, x[u][0], x[u][1]);
          else
            x[u][0] = x[u][1] = T(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + 2 * (u * kTileThreads + (int)threadIdx.x);
          if (i < trows) s_tile[i] = x[u][0];
          if (i + 1 < trows) s_tile[i + 1] = x[u][1];
        }
      }
    }
    __syncthreads();
    for (int si = tseg0 + wave; si < tseg0 + tnseg; si += NW) {
      const SegRec<NH> cur = load_rec<NH>(recs + (int64_t)uniform(si) * kChainRecWords);
      const int hi0 = cur.flags & 1, hitop = (cur.flags >> 1) & 1;
      const int st = (cur.flags >> 12) & 1023;
      const int blk0 = cur.row0 - st;
      const int lrow0 = cur.row0 - trow0, lblk0 = blk0 - trow0;
      const uint32_t so_row = (uint32_t)cur.row0 * TB;
      const uint32_t pair_off = (uint32_t)(2 * lane) * TB;
      // lane l holds the adjacent rows 2l and 2l + 1 (clamped into the segment)
      int jj[2], lo[2];
      u4 np[2];
      bool act_j[2], act_p[2];
      T g_hi[NH - NHL > 0 ? NH - NHL : 1][2], g_p[2], vv[2], bt[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        jj[i] = min(2 * lane + i, cur.len - 1);
        const int l = s_lo[cur.lidx + jj[i]];
        lo[i] = l;
        np[i] = s_np[l];
        act_j[i] = ((l >> (Lb - 1)) & 1) != hi0;
        act_p[i] = c.periodic && ((l & 1) != hitop);
      }
#pragma unroll
      for (int b = NHL; b < NH; ++b) {
        if (cur.dh[b] != 0)
          bload2<T>(rb1, pair_off, (uint32_t)(cur.row0 + cur.dh[b]) * TB, g_hi[b - NHL][0],
                    g_hi[b - NHL][1]);
        else
          g_hi[b - NHL][0] = g_hi[b - NHL][1] = T(0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int rp = (int)((np[i][2] >> 16) & 255u);
        g_p[i] = act_p[i] ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_pbc + rp) * TB, 0) : T(0);
      }
      if (v)
        bload_stream<T, 2>(rv, pair_off, so_row, nt, vv);
      else
        vv[0] = vv[1] = T(0);
      if (b2)
        bload_stream<T, 2>(rb2, pair_off, so_row, nt, bt);
      else
        bt[0] = bt[1] = T(0);
      T o[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int l = lo[i];
        const int lr = lrow0 + jj[i];
        const T bo = s_tile[lr];
        T hop = 0;
#pragma unroll
        for (int b = 0; b < NL; ++b)
          hop += s_tile[lblk0 + (int)((np[i][b >> 2] >> (8 * (b & 3))) & 255u)];
        const int xlo = (l ^ (l >> 1)) & ((1 << NL) - 1);
        hop -= (T)(NL - __popc(xlo)) * bo;
#pragma unroll
        for (int b = 0; b < NHL; ++b)
          if (cur.dh[b] != 0) hop += s_tile[lr + cur.dh[b]];
#pragma unroll
        for (int b = NHL; b < NH; ++b) hop += g_hi[b - NHL][i];
        const int rj = (int)((np[i][2] >> 8) & 255u);
        if (act_j[i]) hop += s_tile[lblk0 + cur.d_join + rj];
        const int lo_top = (l >> (Lb - 1)) & 1, lo0 = l & 1;
        const int n11x = (lo_top & hi0) + (c.periodic ? (hitop & lo0) : 0);
        const T dg = s_dlo[l] + (T)cur.dhi + vzz * (T)n11x;
        const T acc = dg * bo + t_in * hop + (act_p[i] ? t_pb * g_p[i] : T(0));
        o[i] = sigma * acc + tau * bo - bt[i];
        if (v) o[i] += a * vv[i];
      }
      const int r0 = 2 * lane;
      if (r0 + 1 < cur.len)
        bstore2<kAuxNT>(o[0], o[1], rout, pair_off, so_row);
      else if (r0 < cur.len)
        bstore<kAuxNT>(o[0], rout, pair_off, so_row);
    }
  }
}

// XCDs of the device: the staged-tile table carries this many ranges.
constexpr int kWtXcds = 8;

// Staged-tile kernel.  A tile is the set of rows whose state bits outside
// [0, Lb + KT) (and, for a wrapped tile, outside the top bit L - 1) are
// fixed: 2^WR runs of 2^KT consecutive high parts, each run a contiguous
// range of rows.  The workgroup copies the tile's rows of b_{i+1} into LDS
// with direct-to-LDS buffer loads (one 16-byte load per lane fills 1 KB of
// LDS, no registers involved), so that
//   - the low-part hops, the joining bond and the KT - 1 bonds among the
//     tile's high bits read LDS;
//   - in a wrapped tile the periodic bond (L - 1, 0) reads LDS too: its
//     target differs in the top bit, so it lies in the tile's other run;
//   - only the bonds between the tile's high bits and the fixed middle
//     bits gather from global memory, at wave-uniform row offsets;
//   - a row's low-part tables (in list order) are LDS reads.
// With DB the next tile is staged into a second LDS buffer while the current
// one is processed.
//
// What bounds it at L = 24 to 26 is what the L2s fetch and write (counters):
// at L = 24 154 MB a step with two buffers (137 with one, which is slower), 86
// of them the vectors themselves; at the 7.5 TB/s of a plain pass over the same
// vectors that is 20 us of 25.5.  At L = 26 637 MB (333 the vectors), 85 us of
// 100.  Below that it is the work of a segment: a bond without a hop is passed by with a branch where it is loaded
// and where it is added, the low part and the number of its idle bonds come
// with the neighbour positions, a hop that a row does not have reads a zero,
// and FP32 is held to 64 registers, for two workgroups a CU.
//
// us a step of a filter, before and after (with the streamed vectors read
// through the caches and the shares below): FP64 L = 23 18.1 -> 14.4, 24 28.8
// -> 26.5, 25 58.5 -> 50.0, 26 108 -> 99; FP32 L = 24 20.1 -> 17.2, 25 39.6 ->
// 30.3, 26 70.9 -> 55.5.  One row a lane in FP64 (64 registers, twice the
// wavefronts) was slower, 33 at L = 24: the L1 takes 16 lookups for a 64-lane
// load whether a lane reads 8 bytes or 16.
template <typename T, int L, int KT, int WR, int DB, int NT>
__global__ __launch_bounds__(NT, sizeof(T) == 4 ? 8 : 4) void k_chain_wt(
    ChainSplitDev c, T sigma, T tau, T a, const T* __restrict__ v,
    const T* __restrict__ b1, const T* b2, T* out, int nxcd, int rounds, int buf_rows,
    const int32_t* __restrict__ recs, const int32_t* __restrict__ tiles,
    const int32_t* __restrict__ shares) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int NLO = 1 << Lb;
  constexpr int NH = L - Lb - 1;  // bonds inside the high part
  constexpr int NHL = KT - 1;     // of which inside the tile: b < NHL
  constexpr int NFAR = NH - NHL;
  constexpr int NL = Lb - 1;
  constexpr int R = 2;  // rows per lane
  constexpr int UNITS = kChainSegRows / (64 * R);
  constexpr int BLOB = wt_blob_bytes(NLO, (int)sizeof(T));
  constexpr int CHUNKS = BLOB / 16;
  constexpr int CH = 1024 / (int)sizeof(T);  // rows per staging load of a wave
  constexpr int NW = NT / 64;
  constexpr uint32_t TB = sizeof(T);
  using u4 = __attribute__((ext_vector_type(4))) uint32_t;
  using lds_ptr = __attribute__((address_space(3))) void*;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  {
    const u4* src = reinterpret_cast<const u4*>(sizeof(T) == 8 ? c.blobl64 : c.blobl32);
    u4* dst = reinterpret_cast<u4*>(smem);
    for (int i = threadIdx.x; i < CHUNKS; i += NT) dst[i] = src[i];
    if (threadIdx.x < 4) reinterpret_cast<uint32_t*>(smem + BLOB)[threadIdx.x] = 0;
  }
  // list-ordered tables: entry p describes the p-th low part of the list
  const u4* s_np = reinterpret_cast<const u4*>(smem);
  const T* s_dlo = reinterpret_cast<const T*>(smem + 16 * NLO);
  // a zero behind the tables (what a hop that does not exist reads), then
  // the tile buffers of buf_rows rows of b_{i+1}
  constexpr uint32_t ZERO = BLOB;
  constexpr uint32_t BUF0 = BLOB + 16;
  const uint32_t buf_bytes = DB ? (uint32_t)buf_rows * TB : 0u;

  const int xcd = blockIdx.x % nxcd;
  const int wg = blockIdx.x / nxcd, nwg = gridDim.x / nxcd;
  // the tiles of this workgroup: one share a round, a share going from
  // segment s0 of tile t0 up to segment s1 of tile t1
  struct Pos {
    int r, t, s0, t1, s1, t_end;
  };
  auto share = [&](Pos& p) {
    const int32_t* q = shares + 2 * ((xcd * rounds + p.r) * nwg + wg);
    p.t = uniform(q[0]);
    p.s0 = uniform(q[1]);
    p.t1 = uniform(q[2]);
    p.s1 = uniform(q[3]);
    p.t_end = p.s1 > 0 ? p.t1 + 1 : p.t1;
  };
  auto settle = [&](Pos& p) {  // on to the next share that has a tile left
    while (p.t >= p.t_end && p.r < rounds) {
      if (++p.r < rounds) share(p);
    }
  };
  Pos at{};
  share(at);
  settle(at);
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const T vzz = (T)c.vzz, t_in = (T)c.t_in, t_pb = (T)c.t_pb;
  const bool nt = stream_nt<T>(c.D);
  const uint32_t vbytes = (uint32_t)(c.D * TB);
  const rsrc_t rb1 = make_rsrc(b1, vbytes), rv = make_rsrc(v, v ? vbytes : 0),
               rb2 = make_rsrc(b2, b2 ? vbytes : 0), rout = make_rsrc(out, vbytes);
  // the tile's runs of rows into a buffer, in chunks of 1 KB dealt round
  // robin to the waves; a run's last chunk spills into the run's padding
  auto stage = [&](int t, uint32_t buf) {
    const int32_t* tt = tiles + 8 * t;
    int rbase = 0;
#pragma unroll
    for (int r = 0; r < (1 << WR); ++r) {
      const int row0 = tt[4 * r], rows = tt[4 * r + 1];
      const int nch = (rows + CH - 1) / CH;
      for (int ch = wave; ch < nch; ch += NW)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rb1, (lds_ptr)(smem + buf + (size_t)(rbase + ch * CH) * TB), 16,
            (uint32_t)(ch * CH) * TB + 16u * lane, (uint32_t)row0 * TB, 0, 0);
      rbase += nch * CH;
    }
  };
  if (DB && at.r < rounds) stage(at.t, BUF0);
  for (int it = 0; at.r < rounds; ++it) {
    const int t = at.t;
    const bool last = t == at.t1;
    const int u_first = at.s0, u_last = at.s1;
    ++at.t;
    at.s0 = 0;
    settle(at);
    const uint32_t cb = BUF0 + ((it & 1) ? buf_bytes : 0u);
    if (DB) {
      // this tile was requested one iteration ago; once every wave has it
      // (and is done with the other buffer), stage the next tile
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (at.r < rounds) stage(at.t, BUF0 + ((it & 1) ? 0u : buf_bytes));
    } else {
      __syncthreads();  // the previous tile's LDS reads are done
      stage(t, cb);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
    const int32_t* tt = tiles + 8 * t;
    const int r0row = tt[0], r0seg = tt[2], r0nseg = tt[3];
    const int r1row = WR ? tt[4] : 0, r1seg = WR ? tt[6] - r0nseg : 0, r1nseg = WR ? tt[7] : 0;
    const int base1 = WR ? ((tt[1] + CH - 1) / CH) * CH : 0;
    const int u_end = (last ? u_last : r0nseg + r1nseg) * UNITS;
    int u = u_first * UNITS + wave;
    auto record = [&](int uu) {
      const int j = uu / UNITS;
      return recs + (int64_t)(j + (WR && j >= r0nseg ? r1seg : r0seg)) * kChainRecWords;
    };
    for (; u < u_end; u += NW) {
      const int32_t* rec = record(u);
      const SegRec<NH> cur = load_rec<NH>(rec);
      const int d_near = uniform(rec[7]);
      uint32_t act = (uint32_t)uniform(rec[4]) >> 8;  // bonds with a hop
      const int j = u / UNITS;
      const int p0 = (u % UNITS) * 64 * R;  // first row of the unit in its segment
      if (UNITS > 1 && p0 >= cur.len) continue;
      const bool in1 = WR && j >= r0nseg;
      // LDS byte address = TB * global row + shift (own run), + pshift (the
      // other run)
      const uint32_t shift = cb + (uint32_t)(in1 ? base1 - r1row : -r0row) * TB;
      const uint32_t pshift = cb + (uint32_t)(in1 ? -r0row : base1 - r1row) * TB;
      const int hi0 = cur.flags & 1, hitop = (cur.flags >> 1) & 1;
      const int blk0 = cur.row0 - ((cur.flags >> 12) & 1023);
      const uint32_t row = (uint32_t)(cur.row0 + p0);
      const uint32_t blk = (uint32_t)blk0 * TB + shift;
      const uint32_t so_row = row * TB;
      const int r0 = R * lane, left = cur.len - p0;
      const uint32_t off = (uint32_t)r0 * TB;
      // global loads first: the streamed v and b_{i+2}, then the high bonds
      // at uniform offsets.  The empty asm keeps a bond's branch a branch:
      // half of the bonds are idle in a segment, and a branch costs less
      // than the zeros and additions of a select.
      T vv[R], bt[R], g_hi[NFAR > 0 ? NFAR : 1][R], g_p[R];
      if (v) bload_stream<T, R>(rv, off, so_row, nt, vv);
      if (b2) bload_stream<T, R>(rb2, off, so_row, nt, bt);
#pragma unroll
      for (int b = NHL; b < NH; ++b)
        if ((act >> b) & 1u) {
          asm volatile("");
          bload_rows<T, R>(rb1, off, so_row + (uint32_t)cur.dh[b] * TB, g_hi[b - NHL]);
        }
      T o[R], bo[R], hop[R];
      u4 np[R];
#pragma unroll
      for (int i = 0; i < R; ++i) np[i] = s_np[cur.lidx + p0 + min(r0 + i, left - 1)];
      if (!WR) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const uint32_t lo = np[i][3];
          const bool act_p = c.periodic && (int)(lo & 1u) != hitop;
          g_p[i] = act_p ? bload<T>(rb1, (uint32_t)(blk0 + cur.d_pbc +
                                                    (int)((np[i][2] >> 16) & 255u)) * TB, 0)
                         : T(0);
        }
      }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int rr = min(r0 + i, left - 1);
        const uint32_t lo = np[i][3];
        const uint32_t own = (row + (uint32_t)rr) * TB + shift;
        const bool act_j = (int)((lo >> (Lb - 1)) & 1u) != hi0;
        const bool act_p = c.periodic && (int)(lo & 1u) != hitop;
        bo[i] = lds_at<T>(smem, own);
        T h = lds_at<T>(smem, act_j ? own + (uint32_t)d_near * TB : ZERO);
#pragma unroll
        for (int b = 0; b < NL; ++b)
          h += lds_at<T>(smem, blk + ((np[i][b >> 2] >> (8 * (b & 3))) & 255u) * TB);
        // idle low bonds read the row itself
        h -= (T)(int)(np[i][2] >> 24) * bo[i];
#pragma unroll
        for (int b = 0; b < NHL; ++b)
          if ((act >> b) & 1u) {
            asm volatile("");
            h += lds_at<T>(smem, own + (uint32_t)cur.dh[b] * TB);
          }
        hop[i] = h;
        if (WR)
          g_p[i] = lds_at<T>(smem, act_p ? (uint32_t)(blk0 + cur.d_pbc +
                                                      (int)((np[i][2] >> 16) & 255u)) * TB +
                                               pshift
                                         : ZERO);
        const int lo_top = (int)((lo >> (Lb - 1)) & 1u);
        const int n11x = (lo_top & hi0) + (c.periodic ? (hitop & (int)(lo & 1u)) : 0);
        o[i] = s_dlo[cur.lidx + p0 + rr] + (T)cur.dhi + vzz * (T)n11x;
      }
      // (reread, or the first tests' results are held in 24 registers)
      asm volatile("" : "+s"(act));
#pragma unroll
      for (int b = NHL; b < NH; ++b)
        if ((act >> b) & 1u) {
          asm volatile("");
#pragma unroll
          for (int i = 0; i < R; ++i) hop[i] += g_hi[b - NHL][i];
        }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const T acc = o[i] * bo[i] + t_in * hop[i] + t_pb * g_p[i];
        o[i] = sigma * acc + tau * bo[i];
      }
      if (b2) {
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] -= bt[i];
      }
      if (v) {
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] += a * vv[i];
      }
      if (r0 + R <= left)
        bstore_rows<T, R, kAuxNT>(o, rout, off, so_row);
      else if (r0 < left)
        bstore<kAuxNT>(o[0], rout, off, so_row);
    }
  }
}

// Staged-tile configurations: tile bits (chain_wt_bits minus this), wrap, double
// buffer, threads per workgroup.
struct WtConf {
  int dkt, wrap, db, nt;
};
constexpr WtConf kWtConf[] = {
    {0, 1, 0, 1024},   // 6: wrapped tile, one buffer
    {-1, 0, 1, 512},   // 7: twice the run, not wrapped, two buffers
    {-1, 0, 0, 1024},  // 8: twice the run, not wrapped, one buffer
    {0, 1, 1, 1024},   // 9: wrapped tile, two buffers
};
constexpr int kWtFirst = 6, kWtCount = (int)(sizeof(kWtConf) / sizeof(kWtConf[0]));

// Tile bits of the staged-tile kernel's wrapped tile at chain length L.
constexpr int chain_wt_bits(int L) {
  const int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  const int Lh = L - Lb;
  const int kt = Lh - 10 < 4 ? Lh - 10 : 4;
  return (L >= 20 && kt >= 2) ? kt : 0;
}

static const polfed_op::WTiles* wt_tables(const polfed_op* op, int kt, int wrap) {
  const int key = kt * 2 + wrap;
  auto it = op->wtiles.find(key);
  if (it != op->wtiles.end()) return it->second.n > 0 ? &it->second : nullptr;
  polfed_op::WTiles& W = op->wtiles[key];
  const int Lh = op->L - op->split_Lb;
  if (kt < 1 || Lh - kt - wrap < 3 || op->split_hi_off.empty()) return nullptr;
  const auto& ho = op->split_hi_off;
  const auto& so = op->split_seg_of_hi;
  const int64_t nt = (int64_t)1 << (Lh - kt - wrap);
  TallyScope untallied(nullptr);  // the table lives as long as the operator
  std::vector<int32_t> tab;
  std::vector<int64_t> tid;   // the tile index t of each entry
  for (int64_t t = 0; t < nt; ++t) {
    int32_t e[8] = {0};
    int rows_tot = 0, bufr[2] = {0, 0};
    for (int r = 0; r <= wrap; ++r) {
      const int64_t h0 = ((int64_t)r << (Lh - 1)) | (t << kt), h1 = h0 + ((int64_t)1 << kt);
      e[4 * r] = ho[h0];
      e[4 * r + 1] = ho[h1] - ho[h0];
      e[4 * r + 2] = so[h0];
      e[4 * r + 3] = so[h1] - so[h0];
      rows_tot += e[4 * r + 1];
      for (int p = 0; p < 2; ++p) {
        const int ch = p == 0 ? 128 : 256;
        bufr[p] += ((e[4 * r + 1] + ch - 1) / ch) * ch;
      }
    }
    if (rows_tot == 0) continue;
    tab.insert(tab.end(), e, e + 8);
    tid.push_back(t);
    for (int p = 0; p < 2; ++p) W.buf_rows[p] = std::max(W.buf_rows[p], bufr[p]);
  }
  W.kt = kt;
  W.wrap = wrap;
  W.n = (int)(tab.size() / 8);
  // Order of the tiles and their split over the XCDs.  A hop across a bond
  // between two fixed bits of a tile swaps them, which keeps the popcount of
  // the fixed bits t; only the bonds at the ends of the fixed range change
  // it.  Tiles sorted by popcount(t), then by the popcount of the upper half
  // of t (swaps inside either half keep it), then by t, therefore keep most
  // of their global gathers inside a contiguous range of the table, and each
  // XCD takes such a range, cut where the rows (not the tiles) are balanced.
  // Hopping gathers sent to another XCD's range, counted over the sector:
  // 26.6% instead of 39.9% in plain t order at L = 24, 22.1% instead of
  // 33.2% at L = 26, 38.8% instead of 50.3% at L = 22.
  const int tbits = Lh - kt - wrap, thalf = (tbits + 1) / 2;
  std::vector<int> ord(W.n);
  std::iota(ord.begin(), ord.end(), 0);
  auto order_key = [&](int x) {
    const unsigned long long t = (unsigned long long)tid[x];
    return std::make_tuple(__builtin_popcountll(t), __builtin_popcountll(t >> (tbits - thalf)),
                           tid[x]);
  };
  std::stable_sort(ord.begin(), ord.end(),
                   [&](int x, int y) { return order_key(x) < order_key(y); });
  std::vector<int32_t> sorted;
  sorted.reserve(tab.size());
  for (int i : ord) {
    sorted.insert(sorted.end(), tab.begin() + 8 * (size_t)i, tab.begin() + 8 * (size_t)i + 8);
    W.nseg.push_back(tab[8 * (size_t)i + 3] + tab[8 * (size_t)i + 7]);
  }
  tab.swap(sorted);
  upload(W.d, tab.data(), tab.size(), op->ctx->stream);
  HIPC(hipStreamSynchronize(op->ctx->stream));
  return W.n > 0 ? &W : nullptr;
}

// Rounds in which the workgroups go through an XCD's range of the tile table.
// In one round each has one contiguous share and at most one tile's remainder
// to wait for; but tiles that are processed at the same time are then far from
// each other in the table, and so are their gathers.  That costs nothing while
// an XCD's part of b_{i+1} fits its 4 MB L2 (FP64 L = 23 in one round 14.4 us a
// step, in two 15.9), and from there on a round takes one tile of every
// workgroup, neighbours in the table (FP64 L = 25, one round / as many as
// tiles: 57.8 / 50.0; L = 26 124 / 101, which also is the order that the
// gathers were counted in).
static int wt_rounds(const polfed_op* op, const polfed_op::WTiles* W, int n, bool fp32) {
  if (op->D * (fp32 ? 4 : 8) <= kWtXcds * (int64_t)(4 << 20)) return 1;
  return std::max(1, (W->n + n / 2) / n);
}
// Shares of n workgroups of the table's segments: workgroup k starts at
// entry k (tile, segment in it) and ends where k + 1 starts.  A segment takes
// a wavefront about the same time whatever its rows, so segments, not rows
// or tiles, are what is dealt out evenly: with whole tiles per workgroup the
// XCDs of the largest tiles at L = 24 had 98 tiles for 64 workgroups, two
// rounds for 1.5 rounds' work.  A tile that two workgroups share is staged by
// both.
static const int32_t* wt_shares(const polfed_op* op, const polfed_op::WTiles* W, int n) {
  DevBuf& d = W->shares[n];
  if (!d.get()) {
    TallyScope untallied(nullptr);
    int64_t all = 0;
    for (int x : W->nseg) all += x;
    std::vector<int32_t> tab;
    int64_t before = 0;  // segments of the tiles before t
    int t = 0;
    for (int k = 0; k <= n; ++k) {
      const int64_t g = all * k / n;
      while (t < W->n && before + W->nseg[t] <= g) before += W->nseg[t++];
      tab.push_back(t);
      tab.push_back((int32_t)(g - before));
    }
    upload(d, tab.data(), tab.size(), op->ctx->stream);
    HIPC(hipStreamSynchronize(op->ctx->stream));
  }
  return d.as<int32_t>();
}

// LDS of a workgroup: tables, the zero, one or two tile buffers.
static size_t wt_shm(const polfed_op* op, const polfed_op::WTiles* W, bool fp32, int db) {
  const int tb = fp32 ? 4 : 8;
  return wt_blob_bytes(1 << op->split_Lb, tb) + 16 +
         (size_t)(db ? 2 : 1) * W->buf_rows[fp32 ? 1 : 0] * tb;
}

// Workgroups of a launch: as many as are resident at once, in whole XCDs.
static int wt_grid(const polfed_op* op, const polfed_op::WTiles* W, size_t shm, int nt) {
  const int per_cu = std::max(1, std::min((int)(kLdsPerCU / shm), 2048 / nt));
  int64_t grid = std::min<int64_t>(W->n, (int64_t)op->ctx->n_cu * per_cu);
  if (grid >= 64) grid -= grid % kWtXcds;
  return (int)std::max<int64_t>(grid, 1);
}

// The variant's tables, built if they are not there yet (a later launch may
// be under capture).
bool chain_wt_exists(const polfed_op* op, int var, bool fp32) {
  if (op->model != Model::Chain || op->split_nseg <= 0) return false;
  if (var < kWtFirst || var >= kWtFirst + kWtCount) return false;
  const WtConf C = kWtConf[var - kWtFirst];
  const int KT = chain_wt_bits(op->L) - C.dkt;
  if (chain_wt_bits(op->L) == 0 || KT < 1) return false;
  const polfed_op::WTiles* W = wt_tables(op, KT, C.wrap);
  if (!W) return false;
  const size_t shm = wt_shm(op, W, fp32, C.db);
  if (shm > kLdsPerCU) return false;
  const int grid = wt_grid(op, W, shm, C.nt);
  wt_shares(op, W, grid * wt_rounds(op, W, grid, fp32));
  return true;
}

template <typename T, int L, int KT, int WR, int DB, int NT>
static bool launch_wt(hipStream_t s, const polfed_op* op, T sigma, T tau, T a, const T* v,
                      const T* b1, const T* b2, T* out) {
  const polfed_op::WTiles* W = wt_tables(op, KT, WR);
  if (!W) return false;
  const bool fp32 = sizeof(T) == 4;
  const size_t shm = wt_shm(op, W, fp32, DB);
  if (shm > kLdsPerCU) return false;
  const int grid = wt_grid(op, W, shm, NT);
  const int nxcd = grid >= 64 ? kWtXcds : 1;
  const int rounds = wt_rounds(op, W, grid, fp32);
  const ChainSplitDev c = op->chain_split();
  hipLaunchKernelGGL((k_chain_wt<T, L, KT, WR, DB, NT>), dim3((unsigned)grid), dim3(NT), shm, s,
                     c, sigma, tau, a, v, b1, b2, out, nxcd, rounds, W->buf_rows[fp32 ? 1 : 0],
                     c.rec, W->d.as<int32_t>(), wt_shares(op, W, grid * rounds));
  HIPC(hipGetLastError());
  return true;
}

template <typename T, int L, int I>
static bool launch_wt_conf(hipStream_t s, const polfed_op* op, T sigma, T tau, T a, const T* v,
                           const T* b1, const T* b2, T* out) {
  constexpr WtConf C = kWtConf[I];
  constexpr int KT = chain_wt_bits(L) - C.dkt;
  if constexpr (chain_wt_bits(L) == 0 || KT < 1) {
    return false;
  } else {
    return launch_wt<T, L, KT, C.wrap, C.db, C.nt>(s, op, sigma, tau, a, v, b1, b2, out);
  }
}

template <typename T, int L, int... I>
static bool launch_wt_any(hipStream_t s, const polfed_op* op, int i, T sigma, T tau, T a,
                          const T* v, const T* b1, const T* b2, T* out,
                          std::integer_sequence<int, I...>) {
  bool ok = false;
  ((i == I ? (ok = launch_wt_conf<T, L, I>(s, op, sigma, tau, a, v, b1, b2, out), 0) : 0), ...);
  return ok;
}

// Launch shape: kChainBlocksPerCU persistent blocks per CU, the blocks of a
// launch mapped XCD-contiguously once there are enough of them.

template <typename T, int L, int HALVES = 1>
static void launch_split(hipStream_t s, const polfed_op* op, T sigma, T tau, T a,
                         const T* v, const T* b1, const T* b2, T* out) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int NLO = 1 << Lb;
  constexpr int bpc = kChainBlocksPerCU;
  const size_t shm = chain_blob_bytes(NLO, (int)sizeof(T)) + 4 * kChainStageRows * sizeof(T);
  ChainSplitDev c = op->chain_split();
  const int64_t blocks_needed = (c.nseg * HALVES + 3) / 4;
  int64_t grid = std::min<int64_t>(blocks_needed, (int64_t)op->ctx->n_cu * bpc);
  int nxcd = 1;
  if (grid >= 64) {
    grid -= grid % 8;
    nxcd = 8;
  }
  grid = std::max<int64_t>(grid, 1);
  hipLaunchKernelGGL((k_chain_split<T, L, HALVES>), dim3((unsigned)grid), dim3(256), shm, s, c,
                     sigma, tau, a, v, b1, b2, out, nxcd, c.rec);
  HIPC(hipGetLastError());
}

template <typename T, int L, int KT>
static void launch_tile(hipStream_t s, const polfed_op* op, const polfed_op::Tiles& tl, T sigma,
                        T tau, T a, const T* v, const T* b1, const T* b2, T* out) {
  constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
  constexpr int NLO = 1 << Lb;
  const size_t shm = chain_blob_bytes(NLO, (int)sizeof(T)) + (size_t)tl.max_rows * sizeof(T);
  const int per_cu = std::max(1, (int)(kLdsPerCU / shm));
  ChainSplitDev c = op->chain_split();
  int64_t grid = std::min<int64_t>(tl.n, (int64_t)op->ctx->n_cu * per_cu);
  int nxcd = 1;
  if (grid >= 64) {
    grid -= grid % 8;
    nxcd = 8;
  }
  grid = std::max<int64_t>(grid, 1);
  hipLaunchKernelGGL((k_chain_tile<T, L, KT>), dim3((unsigned)grid), dim3(kTileThreads), shm, s, c,
                     sigma, tau, a, v, b1, b2, out, nxcd, tl.n, c.rec, tl.d.as<int32_t>());
  HIPC(hipGetLastError());
}

// Step-kernel variants of a chain: 0 = segment kernel, 1 + i = tile kernel
// with tiles[i].  Returns false for a variant that does not exist.
template <typename T, int L>
static bool launch_variant(hipStream_t s, const polfed_op* op, int var, T sigma, T tau, T a,
                           const T* v, const T* b1, const T* b2, T* out) {
  constexpr int KT = chain_tile_bits(L);
  if (var == 0) {
    launch_split<T, L>(s, op, sigma, tau, a, v, b1, b2, out);
    return true;
  }
  if (var == 3) {
    if constexpr (L >= kPairedFirst)
      launch_pair<T, L>(s, op, sigma, tau, a, v, b1, b2, out);
    else
      launch_direct<T, L>(s, op, sigma, tau, a, v, b1, b2, out);
    return true;
  }
  if (var == 4) {
    launch_split<T, L, 2>(s, op, sigma, tau, a, v, b1, b2, out);
    return true;
  }
  if (var >= kWtFirst && var < kWtFirst + kWtCount)
    return launch_wt_any<T, L>(s, op, var - kWtFirst, sigma, tau, a, v, b1, b2, out,
                               std::make_integer_sequence<int, kWtCount>{});
  if constexpr (KT >= 2) {
    constexpr int Lb = (L / 2 < kChainLoBits) ? L / 2 : kChainLoBits;
    if (var != 1 && var != 2 && var != 5) return false;
    const auto& tl = op->tiles[var == 5 ? 2 : var - 1];
    if (tl.n <= 0) return false;
    if (chain_blob_bytes(1 << Lb, (int)sizeof(T)) + (size_t)tl.max_rows * sizeof(T) > kLdsPerCU)
      return false;
    if (var == 1 && tl.bits == KT) {
      launch_tile<T, L, KT>(s, op, tl, sigma, tau, a, v, b1, b2, out);
      return true;
    }
    if constexpr (KT - 1 >= 2) {
      if (var == 2 && tl.bits == KT - 1) {
        launch_tile<T, L, KT - 1>(s, op, tl, sigma, tau, a, v, b1, b2, out);
        return true;
      }
    }
    if constexpr (KT - 2 >= 2) {
      if (var == 5 && tl.bits == KT - 2) {
        launch_tile<T, L, KT - 2>(s, op, tl, sigma, tau, a, v, b1, b2, out);
        return true;
      }
    }
  }
  return false;
}

// Picks the fastest variant for (op, precision) by replaying 20 launches of
// each on scratch vectors; not while the stream is being captured.  The
// choice is shared by the context's operators of the same chain pattern
// (same kernels and tables, other diagonals).
template <typename T, int L>
static int tuned_variant(hipStream_t s, const polfed_op* op) {
  const int pi = sizeof(T) == 8 ? 0 : 1;
  if (op->tuned[pi] >= 0) return op->tuned[pi];
  const std::string pkey = std::string(sizeof(T) == 8 ? "step64" : "step32");
  {
    const int v = pattern_choice(op, pkey);
    if (v >= 0) {
      chain_res_prepare(s, op, pi == 1);
      return op->tuned[pi] = v;
    }
  }
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIPC(hipStreamIsCapturing(s, &cs));
  if (cs != hipStreamCaptureStatusNone) return 0;
  chain_res_prepare(s, op, pi == 1);  // the tables of the resident filter
  const size_t n = (size_t)op->D;
  DevBuf bv(n * sizeof(T)), bb1(n * sizeof(T)), bb2(n * sizeof(T));
  HIPC(hipMemsetAsync(bv.get(), 0, n * sizeof(T), s));
  HIPC(hipMemsetAsync(bb1.get(), 0, n * sizeof(T), s));
  HIPC(hipMemsetAsync(bb2.get(), 0, n * sizeof(T), s));
  HIPC(hipStreamSynchronize(s));  // the operator's tables and the scratch vectors
  int best = 0;
  float best_us = 1e30f;
  for (int var = 0; var < kWtFirst + kWtCount; ++var) {
    const bool ok = launch_variant<T, L>(s, op, var, T(0.1), T(0), T(0), bv.as<T>(),
                                         bb1.as<T>(), bb2.as<T>(), bb2.as<T>());
    if (!ok) continue;
    HIPC(hipStreamSynchronize(s));
    const float us = replay_time_us(
        [&](hipStream_t ts) {
          launch_variant<T, L>(ts, op, var, T(0.1), T(0), T(0), bv.as<T>(), bb1.as<T>(),
                               bb2.as<T>(), bb2.as<T>());
        },
        20);
    if (verbose())
      std::fprintf(stderr, "[polfed] chain step L=%d %s variant %d: %.2f us\n", L,
                   sizeof(T) == 8 ? "fp64" : "fp32", var, us);
    if (us < best_us) {
      best_us = us;
      best = var;
    }
  }
  HIPC(hipStreamSynchronize(s));
  pattern_choice_set(op, pkey, best);
  return op->tuned[pi] = best;
}

template <typename T>
bool chain_split_step(hipStream_t s, const polfed_op* op, T sigma, T tau, T a,
                      const T* v, const T* b1, const T* b2, T* out) {
  if (op->split_nseg <= 0) return false;
  switch (op->L) {
#define POLFED_CASE(LL)                                                                     \
  case LL:                                                                                  \
    if (!launch_variant<T, LL>(s, op, tuned_variant<T, LL>(s, op), sigma, tau, a, v, b1, b2, \
                               out))                                                        \
      launch_split<T, LL>(s, op, sigma, tau, a, v, b1, b2, out);                            \
    return true;
    POLFED_CASE(4) POLFED_CASE(5) POLFED_CASE(6) POLFED_CASE(7) POLFED_CASE(8)
    POLFED_CASE(9) POLFED_CASE(10) POLFED_CASE(11) POLFED_CASE(12) POLFED_CASE(13)
    POLFED_CASE(14) POLFED_CASE(15) POLFED_CASE(16) POLFED_CASE(17) POLFED_CASE(18)
    POLFED_CASE(19) POLFED_CASE(20) POLFED_CASE(21) POLFED_CASE(22) POLFED_CASE(23)
    POLFED_CASE(24) POLFED_CASE(25) POLFED_CASE(26) POLFED_CASE(27) POLFED_CASE(28)
#undef POLFED_CASE
    default: return false;
  }
}

template bool chain_split_step<double>(hipStream_t, const polfed_op*, double, double, double,
                                       const double*, const double*, const double*, double*);
template bool chain_split_step<float>(hipStream_t, const polfed_op*, float, float, float,
                                      const float*, const float*, const float*, float*);

}  // namespace polfed

polfed::ChainSplitDev polfed_op::chain_split() const {
  polfed::ChainSplitDev c{};
  c.D = D;
  c.N = N;
  c.periodic = periodic;
  c.t_in = t_in;
  c.t_pb = t_pb;
  c.vzz = vzz;
  c.blob64 = d_blob64.get();
  c.blob32 = d_blob32.get();
  c.blobl64 = d_blobl64.get();
  c.blobl32 = d_blobl32.get();
  c.rec = d_rec.as<int32_t>();
  c.nseg = split_nseg;
  return c;
}
