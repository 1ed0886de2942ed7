// screen.hip -- the 8-bit copies that the screened scan reads (the bound they
// serve is derived in screen_tile.h): of the stored vectors once, when the
// index is loaded, and of a search's queries once per search.
#include "mfma_tile.h"

namespace sieve {
namespace {

// A 64-byte chunk count the screened kernels are built for.
constexpr int kChunkCounts[] = {1, 2, 3, 4, 6, 8, 12, 16};

// 16 consecutive dimensions at p, the first ndims of them real (a multiple
// of 8; none where ndims <= 0).
template <int DT>
__device__ __forceinline__ void load16(const char* p, int ndims, float (&v)[16]) {
  u32x4 w[16 / DTraits<DT>::kSegDims];
#pragma unroll
  for (int s = 0; s < 16 / DTraits<DT>::kSegDims; ++s) {
    w[s] = u32x4{0u, 0u, 0u, 0u};
    if (DTraits<DT>::kSegDims * s < ndims) w[s] = ((const u32x4*)p)[s];
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if constexpr (DT == SIEVE_F32)
      v[e] = __builtin_bit_cast(f32x4, w[e / 4])[e % 4];
    else
      v[e] = (float)__builtin_bit_cast(f16x8, w[e / 8])[e % 8];
  }
}

// Sums over quantised values in units of the scale: tt = (x / s)^2,
// hh = q^2, rr = (x / s - q)^2.
struct QuantSums {
  float tt = 0.f, hh = 0.f, rr = 0.f;
};

// 16 values to 8-bit integers of scale 1 / inv.  NaN becomes 0 (the
// parameters of its list or query are infinite then).
__device__ __forceinline__ u32x4 quant16(const float (&v)[16], float inv, QuantSums& z) {
  u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float t = v[e] * inv;
    const float c = fminf(fmaxf(rintf(t), -127.f), 127.f);
    const float q = c == c ? c : 0.f;
    z.tt = fmaf(t, t, z.tt);
    z.hh = fmaf(q, q, z.hh);
    z.rr = fmaf(t - q, t - q, z.rr);
    w[e >> 2] |= ((uint32_t)(int32_t)q & 255u) << (8 * (e & 3));
  }
  return w;
}

// Upper bounds of the norms that belong to sums over nseg 16-value segments.
// t = x inv has a relative error of 2^-22 (the reciprocal's and the
// product's), at most 127 2^-22 < 4e-5 absolute, and t - q is exact; the fp32
// sums of at most 1,024 non-negative terms lose less than 1e-4 of their
// value.  fmaxf: a norm below 1e-30 keeps its products out of the underflow.
__device__ __forceinline__ float norm_up(float s, float sum) {
  return fmaxf(s * sqrtf(sum) * 1.0002f, 1e-30f);
}
__device__ __forceinline__ float err_up(float s, float sum, int nseg) {
  return fmaxf(s * (sqrtf(sum) + 4e-5f * sqrtf(16.f * (float)nseg)) * 1.0002f, 1e-30f);
}
__device__ __forceinline__ float scale_of(float mx) { return fmaxf(mx * (1.f / 127.f), 1e-36f); }

// The partition of copy row p: the last L with foff[L] <= p.
__device__ __forceinline__ int list_of(const int64_t* __restrict__ foff, int nlist, int64_t p) {
  int lo = 0, hi = nlist;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (foff[mid] <= p) lo = mid; else hi = mid;
  }
  return lo;
}

// Both load-time passes give a wave kRunBlocks consecutive 16-row blocks of
// the fragment-order copies; a block lies in one partition, so the partition
// is searched once per wave and then followed, and a list's maxima take one
// atomic per wave and list.  Lane l handles row l % 16 of its block.
constexpr int kRunBlocks = 8;

template <typename Body, typename Flush>
__device__ __forceinline__ void for_blocks(const int64_t* __restrict__ off,
                                           const int64_t* __restrict__ foff, int32_t nlist,
                                           int64_t nblk, Body&& body, Flush&& flush) {
  const int lane = threadIdx.x & 63;
  const int64_t b0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kRunBlocks;
  if (b0 >= nblk) return;
  const int64_t b1 = b0 + kRunBlocks < nblk ? b0 + kRunBlocks : nblk;
  int L = list_of(foff, nlist, b0 * 16);
  for (int64_t b = b0; b < b1; ++b) {
    while (foff[L + 1] <= b * 16) {
      flush(L);
      ++L;
    }
    const int64_t k = b * 16 - foff[L] + (lane & 15);
    const bool real = k < off[L + 1] - off[L];
    body(b, L, off[L] + (real ? k : 0), real);
  }
  flush(L);
}

// First pass: the exact fragment-order copy (frag, where the dimension has
// one) and the largest |value| of each list (lpar[L].pad, as integer bits:
// NaN above inf).
template <int DT>
__global__ __launch_bounds__(256) void index_rows_kernel(
    const char* __restrict__ vectors, const int64_t* __restrict__ off,
    const int64_t* __restrict__ foff, int32_t nlist, int32_t d, int64_t nblk,
    u32x4* __restrict__ frag, ScreenParam* __restrict__ lpar) {
  const int lane = threadIdx.x & 63, h = lane >> 4;
  const int dsegs = d / DTraits<DT>::kSegDims;
  const int nch = (dsegs + 3) / 4;
  uint32_t mx = 0;  // fp16: the lane's even and odd elements in two halves
  for_blocks(
      off, foff, nlist, nblk,
      [&](int64_t b, int, int64_t row, bool real) {
        const u32x4* src = (const u32x4*)(vectors + row * (int64_t)d * DTraits<DT>::kElem);
#pragma unroll 4
        for (int c = 0; c < nch; ++c) {
          u32x4 w = {0u, 0u, 0u, 0u};
          if (real && 4 * c + h < dsegs) w = src[4 * c + h];
          if (frag) frag[(b * nch + c) * 64 + lane] = w;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (DT == SIEVE_F32) {
              mx = max(mx, w[e] & 0x7fffffffu);
            } else {
              const uint32_t x = w[e] & 0x7fff7fffu;
              mx = max(mx >> 16, x >> 16) << 16 | max(mx & 0xffffu, x & 0xffffu);
            }
          }
        }
      },
      [&](int L) {
        if (!lpar) return;
        uint32_t m = mx;
        mx = 0;
        if constexpr (DT == SIEVE_F16) {
          const uint16_t hb = (uint16_t)max(m >> 16, m & 0xffffu);
          m = __float_as_uint((float)__builtin_bit_cast(_Float16, hb));
        }
        for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
        if (lane == 0 && m) atomicMax((uint32_t*)&lpar[L].pad, m);
      });
}

// Second pass: the 8-bit rows and the lists' scale, err and norm.
template <int DT>
__global__ __launch_bounds__(256) void screen_rows_kernel(
    const char* __restrict__ vectors, const int64_t* __restrict__ off,
    const int64_t* __restrict__ foff, int32_t nlist, int32_t d, int32_t nc, int64_t nblk,
    u32x4* __restrict__ v8, ScreenParam* __restrict__ lpar) {
  const int lane = threadIdx.x & 63, h = lane >> 4;
  float mt = 0.f, mr = 0.f;  // the largest sums of this lane's rows of the list
  for_blocks(
      off, foff, nlist, nblk,
      [&](int64_t b, int L, int64_t row, bool real) {
        const uint32_t mb = __float_as_uint(lpar[L].pad);
        const float inv = mb < 0x7f800000u ? 1.f / scale_of(__uint_as_float(mb)) : 1.f;
        const char* src = vectors + row * (int64_t)d * DTraits<DT>::kElem;
        QuantSums z;
#pragma unroll 2
        for (int c = 0; c < nc; ++c) {
          const int dim = c * 64 + h * 16;
          float v[16];
          load16<DT>(src + (int64_t)dim * DTraits<DT>::kElem, real ? d - dim : 0, v);
          v8[(b * nc + c) * 64 + lane] = quant16(v, inv, z);
        }
        z.tt += __shfl_xor(z.tt, 16);
        z.tt += __shfl_xor(z.tt, 32);
        z.rr += __shfl_xor(z.rr, 16);
        z.rr += __shfl_xor(z.rr, 32);
        mt = fmaxf(mt, z.tt);
        mr = fmaxf(mr, z.rr);
      },
      [&](int L) {
        for (int o = 8; o > 0; o >>= 1) {
          mt = fmaxf(mt, __shfl_xor(mt, o));
          mr = fmaxf(mr, __shfl_xor(mr, o));
        }
        const uint32_t mb = __float_as_uint(lpar[L].pad);
        const bool finite = mb < 0x7f800000u;
        const float s = finite ? scale_of(__uint_as_float(mb)) : 1.f;
        if (lane == 0) {
          lpar[L].s = s;
          const float err = finite ? err_up(s, mr, 4 * nc) : INFINITY;
          const float norm = finite ? norm_up(s, mt) : INFINITY;
          atomicMax((uint32_t*)&lpar[L].err, __float_as_uint(err));
          atomicMax((uint32_t*)&lpar[L].norm, __float_as_uint(norm));
        }
        mt = mr = 0.f;
      });
}

// Scores of row pairs of sampled lists, for the estimate of how many pairs a
// threshold lets pass: work-group i (one wave) takes the middle full 16-row
// block of list i nlist / nsamp and writes the 8-bit scores of its rows
// against each other (-inf on and below the diagonal, or for lists of fewer
// than 16 rows).
__global__ __launch_bounds__(64) void screen_sample_kernel(
    const u32x4* __restrict__ v8, const int64_t* __restrict__ off,
    const int64_t* __restrict__ foff, int32_t nlist, int32_t nc,
    const ScreenParam* __restrict__ lpar, float* __restrict__ out) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x, h = lane >> 4, r16 = lane & 15;
  const int L = (int)((int64_t)blockIdx.x * nlist / gridDim.x);
  const int64_t len = off[L + 1] - off[L];
  i32x4 acc = {0, 0, 0, 0};
  if (len >= 16) {
    const u32x4* blk = v8 + ((foff[L] >> 4) + ((len >> 4) - 1) / 2) * (int64_t)nc * 64;
    for (int c = 0; c < nc; ++c) {
      const i32x4 x = __builtin_bit_cast(i32x4, blk[c * 64 + lane]);
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, x, acc, 0, 0, 0);
    }
  }
  const float ss = lpar[L].s * lpar[L].s;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 4 * h + r;
    out[(size_t)blockIdx.x * 256 + i * 16 + r16] =
        len >= 16 && i < r16 ? ss * (float)acc[r] : -INFINITY;
  }
}

// 16 lanes per query, 16 dimensions per lane and step.  The search's resets
// (f) ride along, which saves their launch.
template <int DT>
__global__ __launch_bounds__(256) void screen_queries_kernel(const char* __restrict__ queries,
                                                             int64_t nq, int32_t d, int32_t nc,
                                                             u32x4* __restrict__ q8,
                                                             ScreenParam* __restrict__ qpar,
                                                             FillSegs f) {
#pragma unroll
  for (int k = 0; k < kFillSegs; ++k) {
    int32_t* __restrict__ p = f.seg[k].p;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < f.seg[k].n;
         i += (int64_t)gridDim.x * blockDim.x)
      p[i] = f.seg[k].v;
  }
  const int l16 = threadIdx.x & 15;
  const int64_t q = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const bool real = q < nq;
  const char* row = queries + (real ? q : 0) * (int64_t)d * DTraits<DT>::kElem;
  const int nseg = 4 * nc;  // 16-dimension segments
  uint32_t mx = 0;
  for (int s = l16; s < nseg; s += 16) {
    float v[16];
    load16<DT>(row + (int64_t)s * 16 * DTraits<DT>::kElem, d - s * 16, v);
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = max(mx, __float_as_uint(v[e]) & 0x7fffffffu);
  }
  for (int o = 8; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
  const bool finite = mx < 0x7f800000u;
  const float sc = finite ? scale_of(__uint_as_float(mx)) : 1.f;
  const float inv = 1.f / sc;
  QuantSums z;
  for (int s = l16; s < nseg; s += 16) {
    float v[16];
    load16<DT>(row + (int64_t)s * 16 * DTraits<DT>::kElem, d - s * 16, v);
    const u32x4 w = quant16(v, inv, z);
    if (real) q8[q * nseg + s] = w;
  }
  for (int o = 8; o > 0; o >>= 1) {
    z.hh += __shfl_xor(z.hh, o);
    z.rr += __shfl_xor(z.rr, o);
  }
  if (real && l16 == 0)
    qpar[q] = ScreenParam{sc, finite ? err_up(sc, z.rr, nseg) : INFINITY,
                          finite ? norm_up(sc, z.hh) : INFINITY, 0.f};
}

}  // namespace

int screen_chunks(int d) {
  const int nc = (d + 63) / 64;
  for (int c : kChunkCounts)
    if (nc <= c) return c;
  return 0;
}

size_t screen_rows_bytes(int d, int64_t frag_rows) {
  return (size_t)((frag_rows + 15) / 16) * (size_t)screen_chunks(d) * 1024;
}

// The exact fragment-order copy's dimensions (those the exact scan is
// compiled for; the others read the row-major store).
size_t vector_frag_bytes(int dtype, int d, int64_t frag_rows) {
  const bool fixed = dtype == SIEVE_F32 ? (d == 64 || d == 128)
                                        : (d == 64 || d == 128 || d == 768);
  if (!fixed || frag_rows <= 0) return 0;
  const int64_t row_bytes = (int64_t)d * (dtype == SIEVE_F32 ? 4 : 2);
  return (size_t)((frag_rows + 15) / 16) * (size_t)((row_bytes + 63) / 64) * 1024;
}

hipError_t launch_index_rows(int dtype, int d, const void* vectors, const int64_t* offsets,
                             const int64_t* frag_offsets, int32_t nlist, int64_t frag_rows,
                             void* frag, void* v8, ScreenParam* lpar, hipStream_t s) {
  const int nc = screen_chunks(d);
  if (nlist < 1 || (v8 && (nc == 0 || !lpar))) return hipErrorInvalidValue;
  if (v8) {
    const hipError_t e = launch_zero_bytes(lpar, (int64_t)nlist * sizeof(ScreenParam), s);
    if (e != hipSuccess) return e;
  }
  if (frag_rows <= 0 || (!frag && !v8)) return hipSuccess;
  const int64_t nblk = frag_rows / 16;
  const int64_t want = (nblk + 4 * kRunBlocks - 1) / (4 * kRunBlocks);
  if (want > INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)want);
  auto pass1 = [&](auto k) {
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, (const char*)vectors, offsets, frag_offsets,
                       nlist, d, nblk, (u32x4*)frag, v8 ? lpar : nullptr);
    return hipGetLastError();
  };
  auto pass2 = [&](auto k) {
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, (const char*)vectors, offsets, frag_offsets,
                       nlist, d, nc, nblk, (u32x4*)v8, lpar);
    return hipGetLastError();
  };
  const hipError_t e = dtype == SIEVE_F32 ? pass1(index_rows_kernel<SIEVE_F32>)
                                          : pass1(index_rows_kernel<SIEVE_F16>);
  if (e != hipSuccess || !v8) return e;
  return dtype == SIEVE_F32 ? pass2(screen_rows_kernel<SIEVE_F32>)
                            : pass2(screen_rows_kernel<SIEVE_F16>);
}

hipError_t launch_screen_sample(int d, const void* v8, const int64_t* offsets,
                                const int64_t* frag_offsets, int32_t nlist,
                                const ScreenParam* lpar, float* out, hipStream_t s) {
  const int nc = screen_chunks(d);
  if (nc == 0 || nlist < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(screen_sample_kernel, dim3(kScreenSample), dim3(64), 0, s, (const u32x4*)v8,
                     offsets, frag_offsets, nlist, nc, lpar, out);
  return hipGetLastError();
}

hipError_t launch_screen_queries(int dtype, int d, const void* queries, int64_t nq, void* q8,
                                 ScreenParam* qpar, const FillSegs& f, hipStream_t s) {
  const int nc = screen_chunks(d);
  if (nc == 0) return hipErrorInvalidValue;
  if (nq <= 0) return hipErrorInvalidValue;
  int64_t most = 0;
  for (int k = 0; k < kFillSegs; ++k) {
    if (f.seg[k].n < 0 || (f.seg[k].n > 0 && !f.seg[k].p)) return hipErrorInvalidValue;
    most = std::max(most, f.seg[k].n);
  }
  // work-groups past the queries only fill
  const int64_t fill = std::min<int64_t>((most + 255) / 256, 4096);
  const dim3 grid((unsigned)std::max<int64_t>((nq + 15) / 16, fill));
  if (dtype == SIEVE_F32)
    hipLaunchKernelGGL(screen_queries_kernel<SIEVE_F32>, grid, dim3(256), 0, s,
                       (const char*)queries, nq, d, nc, (u32x4*)q8, qpar, f);
  else
    hipLaunchKernelGGL(screen_queries_kernel<SIEVE_F16>, grid, dim3(256), 0, s,
                       (const char*)queries, nq, d, nc, (u32x4*)q8, qpar, f);
  return hipGetLastError();
}

// 112 queries where two work-groups of 128 would pass a CU's LDS.
int screen_tile_q(int d, bool dense) {
  return !dense ? 64 : (screen_chunks(d) == 8 ? 112 : 128);
}

int screen_grid_per_cu(int d, bool dense) {
  const int nc = screen_chunks(d);
  return dense && nc > 8 ? 1 : 2;
}

hipError_t launch_screen_scan(const ScreenArgs& a, int32_t grid, hipStream_t s) {
  const int nc = screen_chunks(a.d);
  if (nc == 0 || !a.v8 || !a.q8 || !a.frag_offsets || !a.arena_on) return hipErrorInvalidValue;
  return nc <= 2 ? launch_screen_scan_reg(nc, a, grid, s) : launch_screen_scan_lds(nc, a, grid, s);
}

}  // namespace sieve
