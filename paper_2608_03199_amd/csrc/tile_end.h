// tile_end.h -- the end of a scan tile: from the qualifying pairs in the
// work-group's candidate arena to the round's hit flags and the candidate
// pool (Algorithm 1's filtered top-k per partition, kept for the final
// MergeTopK).  Shared by the exact scan and the screened scan: both leave the
// same pairs in the arena (exact score >= tau, own row included), so both
// write the same hits and pool entries.
#pragma once

#include "sieve_internal.h"
#include "wave_sort.h"

namespace sieve {
namespace {

// Unsigned key whose order is the float order of finite and infinite scores
// (sign flipped for positive values, all bits flipped for negative ones; -0
// takes +0's key, as the two compare equal).
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x == 0.0f ? 0.0f : x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Top-k selection at the end of a tile: score keys per lane held in
// registers, and the LDS arena entries (8 bytes) each wave borrows to compact
// 64 segment positions.
constexpr int kSelR = 8;
constexpr int kSelSlots = 64 * (int)sizeof(int32_t) / (int)sizeof(TileSpill);

// Per-tile LDS state (kTQ: staged queries at most).  hits, lost and the
// counters are zero when a tile starts; the arena holds wave w's pairs as
// wcnt[w] entries of its LDS part, then gcnt[w] of its global part.
template <int kTQ, int kNT>
struct TileShared {
  int32_t hits[kTQ];  // qualifying rows per staged query in this tile
  int32_t over[kTQ];  // staged queries whose candidates overflowed
  int32_t lost[kTQ];  // their qualifying rows the full arena did not take
  int32_t sel[kTQ];   // staged queries with more than k pairs
  int32_t soff[kTQ];  // their segment in the grouped arena
  int32_t scur[kTQ];
  int32_t poff[kTQ];  // their first pool entry (after the tile's base)
  int32_t wcnt[kNT / 64], gcnt[kNT / 64];
  int32_t pool_n, over_n, sel_n, rbase;
  unsigned long long pbase;
};

// After the barrier that ends the tile's stream (every wave's arena stores
// done, wcnt / gcnt written).  sq, srank, sex: the tile's items; [r0, r1) its
// rows; fd: copy row minus store row of its partition.  The caller resets S
// after the next barrier.
template <int kTQ, int kNT>
__device__ __forceinline__ void finish_tile(const ScanArgs& a, TileShared<kTQ, kNT>& S,
                                            TileSpill* s_arena, int arena_lds, int wcap,
                                            const TileSpill* arena_g, int gcap,
                                            SrtEnt* arena_srt, const int32_t* sq,
                                            const int32_t* srank, const int64_t* sex, int nq,
                                            int64_t r0, int64_t r1, int64_t fd) {
  constexpr int nwv = kNT / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // the arena's parts: pairs held per wave, their prefix; any global part?
  int wpre[kNT / 64 + 1];
  bool ext = false;
  wpre[0] = 0;
#pragma unroll
  for (int w = 0; w < kNT / 64; ++w) {
    const int gw = S.gcnt[w];
    ext |= gw > 0;
    wpre[w + 1] = wpre[w] + S.wcnt[w] + gw;
  }
  // Candidates in the arena's global extension were stored by other waves of
  // the work-group: an acquire at agent scope invalidates the CU's vector L1,
  // whose lines of that area may be stale (read in an earlier tile).
  if (ext) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

  // The arena's pairs are counted per staged query, each query's own row
  // excluded (a pair whose row id is the query's excluded id); four pairs
  // per thread are in flight at once.
  const int na = wpre[kNT / 64];  // pairs the arena holds
  auto arena_at = [&](int e) -> TileSpill {
    int w = 0;
#pragma unroll
    for (int u = 1; u < kNT / 64; ++u) w += e >= wpre[u] ? 1 : 0;
    int ew = e;
#pragma unroll
    for (int u = 1; u < kNT / 64; ++u) ew = w == u ? e - wpre[u] : ew;
    const int nl = S.wcnt[w];
    return ew < nl ? s_arena[w * wcap + ew] : arena_g[w * gcap + ew - nl];
  };
  auto excluded = [&](const TileSpill& ts, int64_t id) {
    return id == sex[ts.rowq >> kSpillRowBits];
  };
  auto row_id = [&](const TileSpill& ts) -> int64_t {
    return a.ids[r0 + (ts.rowq & ((1u << kSpillRowBits) - 1u))];
  };
  for (int e0 = threadIdx.x; e0 < na; e0 += 4 * (int)blockDim.x) {
    TileSpill ts[4];
    int64_t id[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * (int)blockDim.x;
      ts[u] = arena_at(e < na ? e : e0);
      id[u] = row_id(ts[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * (int)blockDim.x < na && !excluded(ts[u], id[u]))
        atomicAdd(&S.hits[ts[u].rowq >> kSpillRowBits], 1);
  }
  __syncthreads();

  // Per staged query: the hit flag; then its candidates to the pool (all of
  // them, or its exact top k when it has more), or, when the arena could not
  // take all of them, a heavy record for the exact top-k pass.
  int c = 0, keep = 0;
  if ((int)threadIdx.x < nq) {
    const int lost = S.lost[threadIdx.x];
    c = S.hits[threadIdx.x];
    if (c + lost > 0) {
      const int q = sq[threadIdx.x];
      const int rk = srank[threadIdx.x];
      atomicMax(&a.lmax[q], rk + 1);
      if (a.hitbits)
        atomicOr(&a.hitbits[(int64_t)q * a.hit_words + (rk >> 5)], 1u << (rk & 31));
      if (lost == 0) {
        keep = min(c, a.k);
        S.poff[threadIdx.x] = atomicAdd(&S.pool_n, keep);
        atomicAdd(&a.hcount[q], keep);
        if (c > a.k) S.sel[atomicAdd(&S.sel_n, 1)] = threadIdx.x;
      } else {
        S.over[atomicAdd(&S.over_n, 1)] = threadIdx.x;
      }
    }
    c += lost;
  }
  if (a.stats) {
    // qualifying pairs of the tile, for the statistics: one add per wave.
    // Not counted where none are asked for: adds on one address serialise
    // (30,000 items over 1,024 lists: 11 of 78 us a round).
    unsigned long long cs = (unsigned long long)c;
    for (int o = 32; o > 0; o >>= 1) cs += __shfl_xor(cs, o);
    if (lane == 0 && cs) atomicAdd(&a.rc->cands, cs);
  }
  __syncthreads();
  const int pool_n = S.pool_n, over_n = S.over_n, sel_n = S.sel_n;  // block-uniform
  if (pool_n + over_n > 0) {
    if (threadIdx.x == 0) {
      S.pbase = pool_n ? atomicAdd(a.pool_count, (unsigned long long)pool_n) : 0ull;
      S.rbase = over_n ? atomicAdd(&a.rc->heavy, (over_n + kHeavyQ - 1) / kHeavyQ) : 0;
    }
    if ((int)threadIdx.x < nq) S.scur[threadIdx.x] = 0;
    // segments of the sorted area, for the queries with more than k pairs
    // only (wave 0: an exclusive prefix over S.sel, kPer consecutive
    // entries per lane)
    if (sel_n > 0 && threadIdx.x < 64) {
      constexpr int kPer = (kTQ + 63) / 64;
      int v[kPer];
      int tot = 0;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int j = kPer * lane + u;
        v[u] = j < sel_n ? S.hits[S.sel[j]] : 0;
        tot += v[u];
      }
      int inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      int ex = inc - tot;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int j = kPer * lane + u;
        if (j < sel_n) S.soff[S.sel[j]] = ex;
        ex += v[u];
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < over_n) {
      const int gi = threadIdx.x / kHeavyQ, m = threadIdx.x % kHeavyQ;
      const int64_t rec = (int64_t)S.rbase + gi;
      if (rec < a.heavy_cap) {
        HeavyRec* hr = a.heavy + rec;
        const int i = S.over[threadIdx.x];
        hr->q[m] = sq[i];
        hr->rank[m] = srank[i];
        hr->ex[m] = sex[i];
        if (m == 0) {
          hr->r0 = r0;
          hr->fd = fd;
          hr->nrows = (int32_t)(r1 - r0);
          hr->nq = min(kHeavyQ, over_n - gi * kHeavyQ);
        }
      }
    }
    if (pool_n > 0) {
      // The arena's pairs, own rows and heavy queries left out: a query
      // with at most k of them writes them to its pool segment directly;
      // one with more groups them in the sorted area (counting sort) for
      // the exact top-k merge below.  Four pairs per thread in flight.
      const int k = a.k;
      for (int e0 = threadIdx.x; e0 < na; e0 += 4 * (int)blockDim.x) {
        TileSpill ts[4];
        int64_t id[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = e0 + u * (int)blockDim.x;
          ts[u] = arena_at(e < na ? e : e0);
          id[u] = row_id(ts[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int qs = (int)(ts[u].rowq >> kSpillRowBits);
          if (e0 + u * (int)blockDim.x >= na || id[u] == sex[qs] || S.lost[qs] > 0) continue;
          const int ci = S.hits[qs];
          const int slot = atomicAdd(&S.scur[qs], 1);
          if (ci <= k) {
            const unsigned long long pi = S.pbase + (unsigned long long)(S.poff[qs] + slot);
            if ((int64_t)pi < a.pool_cap) {
              Hit hv;
              hv.score = ts[u].score;
              hv.q = a.hitbits ? (sq[qs] | (srank[qs] << kRankShift)) : sq[qs];
              hv.id = id[u];
              a.pool[pi] = hv;
            }
          } else {
            arena_srt[S.soff[qs] + slot] = SrtEnt{ts[u].score, 0, id[u]};
          }
        }
      }
      if (sel_n > 0) {
        // the grouped area is read by other waves: stores complete,
        // barrier, L1 invalidated (as above)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        // queries with more than k: one wave selects the query's top k from
        // its segment.  Up to kSelR * 64 pairs: their score keys sit in
        // registers, kSelR per lane; the k-th largest of the 64 lane maxima (a radix
        // select over order-preserving score keys, ballots only) is a lower
        // bound L on the k-th score, since k lanes hold a pair >= L.  When at
        // most 64 pairs reach L, their positions are compacted through the
        // wave's slice of the (now idle) LDS arena, and the pairs are loaded
        // and sorted once: every pair of the top k is among them, ties at L
        // included.  Otherwise (and for longer
        // segments) the segment is merged 64 pairs at a time: the next batch
        // loads under this one's sort, and a batch none of whose pairs
        // reaches the k-th score kept so far is not sorted.
        const Cand none = {-INFINITY, 0x7fffffffffffffffll, -1};
        const bool slots_ok = arena_lds >= nwv * kSelSlots;  // uniform
        int32_t* const wslot = (int32_t*)(s_arena + wv * kSelSlots);
        for (int j = threadIdx.x >> 6; j < sel_n; j += blockDim.x >> 6) {
          const int i = S.sel[j];
          const int ci = S.hits[i];
          const SrtEnt* seg = arena_srt + S.soff[i];
          auto fetch = [&](int b0) -> Cand {
            if (b0 + lane >= ci) return none;
            const SrtEnt se = seg[b0 + lane];
            return Cand{se.score, (long long)se.id, 0};
          };
          Cand top = none;
          bool picked = false;
          if (slots_ok && ci > 64 && ci <= kSelR * 64) {
            uint32_t key[kSelR];
            uint32_t kmax = 0;
#pragma unroll
            for (int r = 0; r < kSelR; ++r) {
              const int e = r * 64 + lane;
              key[r] = e < ci ? order_key(seg[e].score) : 0u;
              kmax = max(kmax, key[r]);
            }
            // k-th largest lane maximum (every lane holds a pair: ci > 64)
            uint32_t pre = 0, msk = 0;
            int need = k;
            for (int b = 31; b >= 0; --b) {
              const uint32_t bit = 1u << b;
              const int nhi = __popcll(__ballot((kmax & msk) == pre && (kmax & bit) != 0u));
              if (nhi >= need)
                pre |= bit;
              else
                need -= nhi;
              msk |= bit;
            }
            int cnt = 0;
#pragma unroll
            for (int r = 0; r < kSelR; ++r) cnt += __popcll(__ballot(key[r] >= pre));
            if (cnt <= 64) {
              // segment positions of the pairs that reach L, then one load each
              int pos = 0;
#pragma unroll
              for (int r = 0; r < kSelR; ++r) {
                const bool take = key[r] >= pre;
                const unsigned long long m = __ballot(take);
                if (take)
                  wslot[pos + (int)__builtin_amdgcn_mbcnt_hi(
                                  (uint32_t)(m >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = r * 64 + lane;
                pos += __popcll(m);
              }
              __builtin_amdgcn_wave_barrier();
              Cand c = none;
              if (lane < cnt) {
                const SrtEnt se = seg[wslot[lane]];
                c = Cand{se.score, (long long)se.id, 0};
              }
              __builtin_amdgcn_wave_barrier();  // slots read before the next query's
              top = wave_sort_desc<false>(c, lane);
              picked = true;
            }
          }
          if (!picked) {
            top = wave_sort_desc<false>(fetch(0), lane);
            Cand nxt = fetch(64);
            for (int b0 = 64; b0 < ci; b0 += 64) {
              Cand cnd = nxt;
              nxt = fetch(b0 + 64);
              const Cand kth = shfl_cand<false>(top, k - 1);
              if (__ballot(!better(kth, cnd)) == 0ull) continue;
              cnd = wave_sort_desc<false>(cnd, lane);
              const Cand rv = shfl_cand<false>(cnd, 63 - lane);  // top ++ reverse(cnd): bitonic
              top = better(top, rv) ? top : rv;
              top = wave_merge_desc<false>(top, lane);
            }
          }
          const int kk = min(ci, k);
          const unsigned long long base = S.pbase + (unsigned long long)S.poff[i];
          if (lane < kk && (int64_t)(base + lane) < a.pool_cap) {
            Hit hv;
            hv.score = top.s;
            hv.q = a.hitbits ? (sq[i] | (srank[i] << kRankShift)) : sq[i];
            hv.id = top.id;
            a.pool[base + lane] = hv;
          }
        }
      }
    }
  }
}

}  // namespace
}  // namespace sieve
