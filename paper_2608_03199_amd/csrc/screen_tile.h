// screen_tile.h -- the screened partition scan: every (query, row) pair of a
// tile is bounded with 8-bit integer products, and only the pairs whose bound
// reaches tau are scored exactly, so the result is the exact scan's.
//
// Why it is exact.  A row x of list l is stored, beside its exact values, as
// x^ = s_l xi (xi: 8-bit integers), a query as q^ = s_q qi, and
//   q.x = q^.x^ + q^.(x - x^) + (q - q^).x
//       <= s_q s_l (qi.xi) + |q^| e_l + |q - q^| n_l,
// with e_l the largest |x - x^| and n_l the largest |x| of the list (both
// rounded up, as are |q^| and |q - q^|).  The integer product is exact.  The
// scan's score is the fp32 sum of the products, at most
//   2 (d + 2) 2^-24 |q| |x| + u,  u = 2^-126 d (2 + |q| + |x|),
// above q.x.  The first term is the rounding of d products and sums; u is
// what underflow adds to it, which no relative term covers: a product or a
// sum below 2^-126 may lose all of itself (2 d 2^-126), and so may a stored
// value below it (|q_t| or |x_t| times 2^-126 each; the matrix units were
// measured to keep denormal values, the bound does not need them to).  So a
// pair whose score reaches tau has
//   qi.xi >= T(q, l) = floor((tau - slack) / (s_q s_l)),
// slack = |q^| e_l + |q - q^| n_l + 2 (d + 2) 2^-24 |q| n_l + u: no such pair
// is screened out (T is kept in a few bits, rounded down; see BItem).  Pairs that pass are scored with the exact scan's MFMA
// sequence on the stored values (the same bits) and compared with tau.  Where
// the bound is not finite (a list or a query with inf or NaN, an overflowing
// norm) T is below every product: all its pairs are scored.
//
// Why it pays.  The 8-bit rows are half (fp16) or a quarter (fp32) of the
// bytes, and v_mfma_i32_16x16x64_i8 multiplies at twice the fp16 rate and 32
// times the fp32 rate.  The threshold costs nothing: each accumulator starts
// at -T of its query, so a pair passes when its sum is not negative.
#pragma once

#include "mfma_tile.h"
#include "tile_end.h"

namespace sieve {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Accumulator start of a padding query: no product can bring it to zero.
constexpr int32_t kInitNever = -(1 << 30);

__device__ __forceinline__ i32x4 mma_i8(u32x4 a, u32x4 b, i32x4 acc) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a),
                                               __builtin_bit_cast(i32x4, b), acc, 0, 0, 0);
}

// One wave's row blocks of a tile: blocks b0, b0 + nw, ... of the nblk
// 16-row blocks that start at `frag` in the 8-bit fragment-order copy (whole
// blocks: the rows past the tile's last one are the partition's zero
// padding).  NC: 64-byte chunks per row.  Blocks past the end re-read the
// last one, so that every load is issued unconditionally and the compiler's
// wait counts stay exact.
template <int NC>
__device__ __forceinline__ const char* block_ptr(const char* frag, int nblk, int blk) {
  const int b = min(blk, nblk - 1);  // uniform
  return frag + (size_t)b * (NC * 1024);
}

// Whether some pair of the row block passes (uniform); mq: the largest sum of
// each query block, for cand to skip the blocks without a pair.
template <int QB>
__device__ __forceinline__ bool vote_blocks(const i32x4 (&acc)[QB], int (&mq)[QB]) {
  int mx = -1;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    mq[qb] = max(max(acc[qb][0], acc[qb][1]), max(acc[qb][2], acc[qb][3]));
    mx = max(mx, mq[qb]);
  }
  return __ballot(mx >= 0) != 0ull;
}

// Ring depth (row blocks) of the register-held stream: the fragments of the
// queries take 4 NC QB registers, the accumulator starts and the accumulators
// 4 QB each.
template <int NC, int QB, int kRegs>
constexpr int screen_ring() {
  const int nb = (kRegs - 4 * NC * QB - 8 * QB - (kRegs > 128 ? 96 : 48)) / (4 * NC);
  return nb < 3 ? 3 : (nb > 8 ? 8 : nb);
}

// Query fragments in registers (rows of at most two chunks).  Per step: the
// MFMAs of one row block, then its vote; the vote's latency is hidden by the
// other waves of the SIMD.  cand(acc, mq, blk) runs for blocks that
// hold a passing pair; when it cannot take a block it sets resume >= 0 and the
// stream ends.
template <int NC, int QB, int kRegs, typename Cand>
__device__ __forceinline__ void stream_screen_reg(const u32x4* __restrict__ lds, int segs,
                                                  const int32_t* s_init,
                                                  const char* __restrict__ frag, int nblk, int b0,
                                                  int nw, const int& resume, Cand& cand) {
  constexpr int NB = screen_ring<NC, QB, kRegs>();
  const int lane = threadIdx.x & 63;
  const int h = lane >> 4;
  if (b0 >= nblk) return;
  u32x4 qf[NC][QB];
  i32x4 init[QB];
  {
    const u32x4* arow = lds + (lane & 15) * segs + h;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      init[qb] = *(const i32x4*)(s_init + qb * 16 + 4 * h);
#pragma unroll
      for (int c = 0; c < NC; ++c) qf[c][qb] = arow[qb * 16 * segs + 4 * c];
    }
  }
  const uint32_t lo = (uint32_t)lane * 16u;
  auto load = [&](int blk, u32x4(&dst)[NC]) {
    const char* p = block_ptr<NC>(frag, nblk, blk);
#pragma unroll
    for (int c = 0; c < NC; ++c) dst[c] = *(const u32x4*)(p + c * 1024 + lo);
  };
  u32x4 buf[NB][NC];
#pragma unroll
  for (int j = 0; j < NB - 1; ++j) load(b0 + j * nw, buf[j]);
  // nothing issued before stays in flight inside the loop (see
  // stream_rows_sliced)
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_sched_barrier(0);
  int blk = b0;
  auto step = [&](auto jc) {
    constexpr int j = decltype(jc)::value;
    load(blk + (NB - 1) * nw, buf[(j + NB - 1) % NB]);
    __builtin_amdgcn_sched_barrier(0);  // the prefetch stays above the MFMAs
    i32x4 acc[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) acc[qb] = mma_i8(qf[0][qb], buf[j][0], init[qb]);
#pragma unroll
    for (int c = 1; c < NC; ++c) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) acc[qb] = mma_i8(qf[c][qb], buf[j][c], acc[qb]);
    }
    int mq[QB];
    if (vote_blocks(acc, mq)) cand(acc, mq, blk);
    blk += nw;
  };
  // whole trips of NB steps (blocks past the last are not taken by cand)
  const int nsteps = (nblk - b0 + nw - 1) / nw;
  for (int t = (nsteps + NB - 1) / NB; t > 0 && resume < 0; --t)
    unroll_steps(step, std::make_integer_sequence<int, NB>{});
}

// Longer rows: the query fragments are read from LDS for every row block,
// the rows come in slices of up to kSliceChunks chunks, NB - 1 slices ahead.
template <int NC, int QB, typename Cand>
__device__ __forceinline__ void stream_screen_lds(const u32x4* __restrict__ lds, int segs,
                                                  const int32_t* s_init,
                                                  const char* __restrict__ frag, int nblk, int b0,
                                                  int nw, const int& resume, Cand& cand) {
  constexpr int S = NC < kSliceChunks ? NC : kSliceChunks;
  constexpr int NS = (NC + S - 1) / S;
  constexpr int NB = QB <= 2 ? 4 : (QB <= 4 || S <= 6 ? 3 : 2);
  const int lane = threadIdx.x & 63;
  const int h = lane >> 4;
  if (b0 >= nblk) return;
  const uint32_t lo = (uint32_t)lane * 16u;
  auto load = [&](int blk, int s, u32x4(&dst)[S]) {
    const char* p = block_ptr<NC>(frag, nblk, blk);
#pragma unroll
    for (int c = 0; c < S; ++c)
      if (s * S + c < NC) dst[c] = *(const u32x4*)(p + (s * S + c) * 1024 + lo);
  };
  u32x4 buf[NB][S];
  int rb = b0;
#pragma unroll
  for (int u = 0; u < NB - 1; ++u) load(rb + (u / NS) * nw, u % NS, buf[u]);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_sched_barrier(0);
  i32x4 acc[QB];
  for (; resume < 0;) {
#pragma unroll
    for (int u = 0; u < NB * NS; ++u) {
      const int s = u % NS;
      const int blk = rb + (u / NS) * nw;
      if (blk >= nblk) return;
      if (s == 0) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) acc[qb] = *(const i32x4*)(s_init + qb * 16 + 4 * h);
      }
      const int un = u + NB - 1;
      load(rb + (un / NS) * nw, un % NS, buf[un % NB]);
      __builtin_amdgcn_sched_barrier(0);  // the prefetch stays above the MFMAs
      const u32x4* arow = lane_arow(lds, segs);
      u32x4 a0[QB], a1[QB];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) a0[qb] = arow[qb * 16 * segs + 4 * s * S];
#pragma unroll
      for (int c = 0; c < S; ++c) {
        if (s * S + c < NC) {
          u32x4(&cur)[QB] = (c & 1) ? a1 : a0;
          u32x4(&nxt)[QB] = (c & 1) ? a0 : a1;
          if (c + 1 < S && s * S + c + 1 < NC) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) nxt[qb] = arow[qb * 16 * segs + 4 * (s * S + c + 1)];
          }
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) acc[qb] = mma_i8(cur[qb], buf[u % NB][c], acc[qb]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (s == NS - 1) {
        int mq[QB];
        if (vote_blocks(acc, mq)) cand(acc, mq, blk);
      }
    }
    rb += NB * nw;
  }
}

// Exact scores of the wave's arena entries [0, n): 16 pairs at a time, pair i
// as row i of the A operand (its query) and column i of the B operand (its
// row), so that the products' diagonal holds the pairs' scores, summed by the
// exact scan's MFMA sequence in its chunk order.  Entries whose score reaches
// tau stay, compacted in order; returns their number.  Bound by the latency
// of the gathered row and query reads: two groups of pairs are in flight.
template <int DT>
__device__ __forceinline__ int rescore_pairs(TileSpill* ent, int n, const ScreenArgs& a, int64_t r0,
                                             const int32_t* sq) {
  const int lane = threadIdx.x & 63;
  const int h = lane >> 4, r16 = lane & 15;
  const int dsegs = a.d / DTraits<DT>::kSegDims;
  const size_t row_bytes = (size_t)a.d * DTraits<DT>::kElem;
  const char* vbase = (const char*)a.vectors + (size_t)r0 * row_bytes;
  const char* qbase = (const char*)a.queries;
  const int full = dsegs >> 2;  // whole chunks
  const int rem = dsegs & 3;    // segments of a last, partial one
  int out = 0;
  __builtin_amdgcn_wave_barrier();  // entries written by other lanes of the wave
  for (int base = 0; base < n; base += 32) {
    TileSpill e[2];
    const u32x4 *qp[2], *vp[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      e[g] = ent[min(base + 16 * g + r16, n - 1)];
      qp[g] = (const u32x4*)(qbase + (size_t)sq[e[g].rowq >> kSpillRowBits] * row_bytes);
      vp[g] = (const u32x4*)(vbase +
                             (size_t)(e[g].rowq & ((1u << kSpillRowBits) - 1u)) * row_bytes);
    }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    int c = 0;
    // U chunks of both groups are in flight at once: each step is one trip to
    // memory, so long rows take eight chunks a step
    auto chunks = [&](auto uc) {
      constexpr int U = decltype(uc)::value;
      u32x4 qv[U][2], rv[U][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          qv[u][g] = qp[g][4 * (c + u) + h];
          rv[u][g] = vp[g][4 * (c + u) + h];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[g] = mma_chunk<DT>(qv[u][g], rv[u][g], acc[g]);
      }
      c += U;
    };
    while (c + 8 <= full) chunks(std::integral_constant<int, 8>{});
    while (c + 4 <= full) chunks(std::integral_constant<int, 4>{});
    for (; c < full + (rem ? 1 : 0); ++c) {
      const bool ok = 4 * c + h < dsegs;
      const int sc = ok ? 4 * c + h : 0;
      const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        u32x4 qv = qp[g][sc], rv = vp[g][sc];
        if (!ok) qv = rv = zero;
        acc[g] = mma_chunk<DT>(qv, rv, acc[g]);
      }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      // pair r16's score: element r16 % 4 of the lane with h = r16 / 4
      float v = acc[g][0];
#pragma unroll
      for (int r = 1; r < 4; ++r) v = (r16 & 3) == r ? acc[g][r] : v;
      const bool keep = h == (r16 >> 2) && base + 16 * g + r16 < n && v >= a.tau;
      const unsigned long long m = __ballot(keep);
      if (keep)
        ent[out + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            TileSpill{v, e[g].rowq};
      out += __popcll(m);
    }
    __builtin_amdgcn_wave_barrier();
  }
  return out;
}

// LDS-DMA copy of the tile's 8-bit query rows (row_u4 16-byte segments each,
// padded to whole chunks) into the staging buffer: 64 consecutive 16-byte
// slots per wave instruction; padding rows repeat row 0 and the pad segment
// repeats segment 0 (never multiplied into a result that is used).
__device__ __forceinline__ void stage_screen(u32x4* buf, int segs, const u32x4* __restrict__ q8,
                                             const int32_t* sq, int nq) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const int row_u4 = segs - 1;
  const int total = ((nq + 15) >> 4) * 16 * segs;
  const int nchunk = (total + 63) >> 6;
  for (int c = wave; c < nchunk; c += nwaves) {
    const int sidx = c * 64 + lane;
    const int row = sidx / segs, seg = sidx - row * segs;
    const int qrow = sq[row < nq ? row : 0];
    const int segc = (seg < row_u4 && sidx < total) ? seg : 0;
    const u32x4* src = q8 + (size_t)qrow * row_u4 + segc;
    __builtin_amdgcn_global_load_lds((const void*)src,
                                     (__attribute__((address_space(3))) void*)(buf + c * 64), 16,
                                     0, 0);
  }
}

template <int QB, int kMax, typename F>
__device__ __forceinline__ void with_blocks(int qb_n, F&& f) {
  if constexpr (QB >= kMax) {
    f(std::integral_constant<int, kMax>{});
  } else {
    if (qb_n <= QB)
      f(std::integral_constant<int, QB>{});
    else
      with_blocks<QB + 1, kMax>(qb_n, f);
  }
}

// The screened scan.  NC: 64-byte chunks per 8-bit row; kReg: query
// fragments in registers; kMaxQB: 16-query blocks per tile at most; kNT
// threads, kOcc work-groups per CU.  The tile schedule is the exact scan's:
// the round's tiles in 8 contiguous ranges, one per XCD, taken in a fixed
// stride (static) or from per-XCD cursors with stealing (dynamic).  While tile
// t runs, the items of t + 1, the record of t + 2 and the claim of t + 3 load;
// the queries of t + 1 stage under t's end.
template <int NC, bool kReg, int kMaxQB, int kNT, int kOcc>
__global__ __launch_bounds__(kNT, kOcc) void screen_scan_kernel(ScreenArgs a) {
  constexpr int kTQ = 16 * kMaxQB;
  constexpr int kSegs = 4 * NC + 1;
  extern __shared__ u32x4 lds[];
  __shared__ int32_t s_q[2][kTQ];
  __shared__ int32_t s_rank[2][kTQ];
  __shared__ int64_t s_ex[2][kTQ];
  __shared__ __align__(16) int32_t s_init[2][kTQ];  // accumulator start: -T of the query
  __shared__ TileShared<kTQ, kNT> S;
  __shared__ int s_first[3], s_next;
  __shared__ unsigned long long s_passed[kNT / 64];
  TileSpill* const arena_g = a.spill + (size_t)blockIdx.x * arena_block_entries(a.spill_cap);
  SrtEnt* const arena_srt = (SrtEnt*)(arena_g + a.spill_cap);
  TileSpill* const s_arena = (TileSpill*)(lds + a.cand_u4);
  const int arena_lds = a.arena_lds;
  constexpr int nwv = kNT / 64;
  const int wv = wave_id();
  const int lane = threadIdx.x & 63;
  const int h = lane >> 4, r16 = lane & 15;
  const int wcap = arena_lds / nwv, gcap = a.spill_cap / nwv;
  TileSpill* const mine = s_arena + wv * wcap;
  const int ntiles = a.rc->ntiles;
  const u32x4* q8 = (const u32x4*)a.q8;

  const int home = blockIdx.x & 7;
  int xq = 0, kseq = 0;
  auto claim = [&]() -> int {
    if (!a.dynamic) {
      const int b = (int)(((int64_t)ntiles * home) / 8);
      const int e = (int)(((int64_t)ntiles * (home + 1)) / 8);
      const int tt = b + (blockIdx.x >> 3) + kseq * (int)(gridDim.x >> 3);
      ++kseq;
      return tt < e ? tt : -1;
    }
    while (xq < 8) {
      const int x = (home + xq) & 7;
      const int b = (int)(((int64_t)ntiles * x) / 8), e = (int)(((int64_t)ntiles * (x + 1)) / 8);
      const int i = atomicAdd(&a.rc->queue[x], 1);
      if (b + i < e) return b + i;
      ++xq;
    }
    return -1;
  };
  auto load_rec = [&](int tt) -> Tile {
    Tile r = {0, 0, 0, 0, 0};
    tt = __builtin_amdgcn_readfirstlane(tt);
    if (tt >= 0) r = a.tiles[tt];
    return r;
  };
  auto load_items = [&](const Tile& r) -> BItem {
    const int64_t idx = r.nq > 0 ? r.item_begin + min((int)threadIdx.x, r.nq - 1) : 0;
    return a.bucket[idx];
  };
  auto put_items = [&](int set, const Tile& r, const BItem& it) {
    if ((int)threadIdx.x < kTQ) {
      const bool real = (int)threadIdx.x < r.nq;
      s_init[set][threadIdx.x] =
          real ? -((it.rank >> kThrShift) * (1 << thr_unit(NC))) : kInitNever;
      if (real) {
        s_q[set][threadIdx.x] = it.q;
        s_rank[set][threadIdx.x] = it.rank & (kMaxRanks - 1);
        s_ex[set][threadIdx.x] = it.ex;
      }
    }
  };

  if (threadIdx.x == 0) {
    s_first[0] = claim();
    s_first[1] = claim();
    s_first[2] = claim();
    S.pool_n = 0;
    S.over_n = 0;
    S.sel_n = 0;
  }
  if (threadIdx.x < kTQ) {
    S.hits[threadIdx.x] = 0;
    S.lost[threadIdx.x] = 0;
  }
  __syncthreads();
  int t = s_first[0], tn = s_first[1], ta = s_first[2];
  Tile rec = load_rec(t), recN = load_rec(tn);
  put_items(0, rec, load_items(rec));
  int set = 0;
  __syncthreads();
  if (t >= 0) stage_screen(lds, kSegs, q8, s_q[0], rec.nq);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  unsigned long long passed = 0;  // pairs scored exactly (this wave)
  while (t >= 0) {
    const int nset = set ^ 1;
    // loads for the tiles ahead, in flight with the row ring's first loads:
    // the next tile's items, the record of the one after, the claim of a third
    const BItem itN = load_items(recN);
    const Tile recA = load_rec(ta);
    int tb = -1;
    if (threadIdx.x == 0) tb = claim();
    const int32_t* sq = s_q[set];
    const int nq = rec.nq;
    const int64_t r0 = rec.r0;
    const int nrows = rec.nrows;
    const int nblk = (nrows + 15) >> 4;
    // the tile's first row starts a 16-row block of the copy
    const int64_t fr0 = r0 + a.frag_offsets[rec.list] - a.list_offsets[rec.list];
    const char* frag = (const char*)a.v8 + (size_t)(fr0 >> 4) * (NC * 1024);

    int wcnt = 0, gcnt = 0;            // this wave's pairs: LDS part, global part
    int first = wv, first_qb = 0;      // where the stream starts or resumes
    for (;;) {
      int resume = -1;                 // (block << 5 | query block) that did not fit
      // Half of a near-duplicate tile's blocks come here: one compare per
      // query block, then one per element of the blocks with a pair; the
      // lanes of an element's mask take consecutive slots.
      auto cand = [&](const auto& acc, const auto& mq, int blk) {
        constexpr int QB = sizeof(acc) / sizeof(acc[0]);
        if (blk >= nblk || blk < first || resume >= 0) return;
        const unsigned long long rows =
            blk * 16 + 16 <= nrows ? ~0ull : __ballot(blk * 16 + r16 < nrows);
        const int qmin = blk == first ? first_qb : 0;
        const uint32_t roff = (uint32_t)(blk * 16 + r16) | (uint32_t)(4 * h) << kSpillRowBits;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          if ((__ballot(mq[qb] >= 0) & rows) == 0ull || qb < qmin || resume >= 0) continue;
          unsigned long long m[4];
          int tot = 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            m[r] = __ballot(acc[qb][r] >= 0) & rows;
            tot += __popcll(m[r]);
          }
          if (wcnt + tot > wcap) {
            resume = blk << 5 | qb;
            continue;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (m[r] == 0ull) continue;
            if ((m[r] >> lane) & 1ull)
              mine[wcnt + (int)__builtin_amdgcn_mbcnt_hi(
                              (uint32_t)(m[r] >> 32),
                              __builtin_amdgcn_mbcnt_lo((uint32_t)m[r], 0u))] =
                  TileSpill{0.f, roff + ((uint32_t)(qb * 16 + r) << kSpillRowBits)};
            wcnt += __popcll(m[r]);
          }
        }
      };
      with_blocks<1, kMaxQB>((nq + 15) >> 4, [&](auto qbc) {
        constexpr int QB = decltype(qbc)::value;
        if constexpr (kReg)
          stream_screen_reg<NC, QB, 512 / (kNT / 256 * kOcc)>(
              lds, kSegs, s_init[set], frag, nblk, first, nwv, resume, cand);
        else
          stream_screen_lds<NC, QB>(lds, kSegs, s_init[set], frag, nblk, first, nwv, resume, cand);
      });
      passed += (unsigned)wcnt;
      wcnt = a.dtype == SIEVE_F32 ? rescore_pairs<SIEVE_F32>(mine, wcnt, a, r0, sq)
                                  : rescore_pairs<SIEVE_F16>(mine, wcnt, a, r0, sq);
      if (resume < 0) break;
      // the LDS part is full of passing pairs: its qualifying ones move to the
      // global part (past that they are counted for the exact top-k pass), and
      // the stream resumes at the block that did not fit
      for (int i = lane; i < wcnt; i += 64) {
        const TileSpill e = mine[i];
        const int qs = (int)(e.rowq >> kSpillRowBits);
        if (gcnt + i < gcap)
          arena_g[wv * gcap + gcnt + i] = e;
        else if (a.ids[r0 + (e.rowq & ((1u << kSpillRowBits) - 1u))] != s_ex[set][qs])
          atomicAdd(&S.lost[qs], 1);
      }
      gcnt = min(gcnt + wcnt, gcap);
      wcnt = 0;
      first = resume >> 5;
      first_qb = resume & 31;
    }
    if (lane == 0) {
      S.wcnt[wv] = wcnt;
      S.gcnt[wv] = gcnt;
    }
    put_items(nset, recN, itN);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's arena stores are complete (in L2)
    __syncthreads();                // every wave is done with the tile's queries
    if (tn >= 0) stage_screen(lds, kSegs, q8, s_q[nset], recN.nq);
    finish_tile<kTQ, kNT>(a, S, s_arena, arena_lds, wcap, arena_g, gcap, arena_srt, sq,
                          s_rank[set], s_ex[set], nq, r0, r0 + nrows, fr0 - r0);
    __syncthreads();  // the counts and the arena are read; reset them for the next tile
    if ((int)threadIdx.x < nq) {
      S.hits[threadIdx.x] = 0;
      S.lost[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) {
      s_next = tb;
      S.pool_n = 0;
      S.over_n = 0;
      S.sel_n = 0;
    }
    __builtin_amdgcn_s_waitcnt(0);  // the next tile's staging
    __syncthreads();
    t = tn;
    tn = ta;
    ta = s_next;
    rec = recN;
    recN = recA;
    set = nset;
  }
  // one add per work-group, spread over the XCDs
  if (lane == 0) s_passed[wv] = passed;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long sum = 0;
    for (int w = 0; w < nwv; ++w) sum += s_passed[w];
    if (sum) atomicAdd(&a.rc->screened[home], sum);
  }
}

// Dynamic LDS: the staged queries, then the arena (at least kArenaWaveMin
// entries per wave: a wave's pairs of one query block always fit an empty
// part).
constexpr int kScreenDynLds = 150 * 1024;
constexpr int kArenaWaveMin = 256;

template <int NC, bool kReg, int kMaxQB, int kNT, int kOcc>
hipError_t launch_screen_k(ScreenArgs a, int32_t grid, hipStream_t s) {
  static const size_t dyn_max = [] {
    hipFuncAttributes fa{};
    int dev = 0, per_block = 0;
    if (hipFuncGetAttributes(&fa, (const void*)screen_scan_kernel<NC, kReg, kMaxQB, kNT, kOcc>) !=
            hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
            hipSuccess)
      return (size_t)0;
    // kOcc work-groups share a CU's 160 KB
    const size_t most = std::min((size_t)per_block, (size_t)(160 * 1024 / kOcc));
    const size_t left = most > fa.sharedSizeBytes ? most - fa.sharedSizeBytes : 0;
    return std::min(left, (size_t)kScreenDynLds) & ~(size_t)1023;
  }();
  if (dyn_max == 0) return hipErrorInvalidValue;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)screen_scan_kernel<NC, kReg, kMaxQB, kNT, kOcc>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_max);
  if (attr != hipSuccess) return attr;
  if (a.tile_q > 16 * kMaxQB || a.tile_q < 1 || a.k < 1 || a.k > 64) return hipErrorInvalidValue;
  const size_t rows = (size_t)(a.tile_q + 15) / 16 * 16;
  const size_t stage = (rows * (4 * NC + 1) * 16 + 1023) & ~(size_t)1023;
  const size_t room = dyn_max > stage ? dyn_max - stage : 0;
  a.arena_lds = (int32_t)std::min<size_t>(room / sizeof(TileSpill), kArenaLdsMax);
  if (a.arena_lds < kArenaWaveMin * (kNT / 64)) return hipErrorInvalidValue;
  a.cand_u4 = (int32_t)(stage / 16);
  const size_t lds = stage + (size_t)a.arena_lds * sizeof(TileSpill);
  hipLaunchKernelGGL((screen_scan_kernel<NC, kReg, kMaxQB, kNT, kOcc>), dim3(grid), dim3(kNT), lds,
                     s, a);
  return hipGetLastError();
}

}  // namespace
}  // namespace sieve
