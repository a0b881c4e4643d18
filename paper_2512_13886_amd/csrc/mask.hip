// Wanda mask selection on the device: the mask that the weight update starts
// from (Algorithm 1 takes M from a selector; the configurations use Wanda's
// saliency, cited in Section 2, with the 2:4 pattern of Section 4).
//
// score[j][i] = W0[j][i]^2 * c[i] in fp64 (the square of |W0| sqrt(c): same
// order; the square of an fp32 weight is exact in fp64 and the product is
// rounded once, so every IEEE implementation gets the same bits). Scores are
// compared through an order-preserving 64-bit key: NaN lowest, -0 == +0.
//
// Unstructured: a workgroup finds a row's keep-th largest key T, then keeps
// every key > T and, in index order, as many keys == T as are still needed.
// Rows of up to 16384 columns live in registers (k_mask_select), longer ones
// are read again for each digit of an 8-pass radix select (k_mask_topk).
// 2:4: one thread per group of 4 ranks its scores.
#include "common.h"

namespace optima {
namespace {

constexpr int kMaskThreads = 256;

__device__ inline double col_value(const void* c, int dtype, int64_t stride, int64_t i) {
  return dtype == OPTIMA_DTYPE_F64 ? static_cast<const double*>(c)[i * stride]
                                   : double(static_cast<const float*>(c)[i * stride]);
}

__device__ inline uint64_t mask_key(float w, double c) {
  const double wd = double(w);
  double s = (wd * wd) * c;
  if (s != s) return 0;       // NaN ranks below everything
  if (s == 0.0) s = 0.0;      // -0 ranks with +0
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(s));
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ void __launch_bounds__(kMaskThreads) k_mask_topk(const float* W0, int64_t d,
                                                            const void* c, int c_dtype,
                                                            int64_t c_stride, int64_t keep,
                                                            uint8_t* mask) {
  __shared__ unsigned hist[256];
  __shared__ uint64_t s_prefix;
  __shared__ int64_t s_need;
  __shared__ int64_t scan[kMaskThreads];
  const int64_t j = blockIdx.x;
  const float* w = W0 + j * d;
  uint8_t* m = mask + j * d;
  const int tid = threadIdx.x;
  if (keep <= 0 || keep >= d) {
    const uint8_t v = keep > 0 ? 1 : 0;
    for (int64_t i = tid; i < d; i += kMaskThreads) m[i] = v;
    return;
  }
  uint64_t prefix = 0, pmask = 0;
  int64_t need = keep;  // keys still to take at or below the current prefix
  for (int pass = 7; pass >= 0; --pass) {
    const int shift = 8 * pass;
    hist[tid] = 0;
    __syncthreads();
    for (int64_t i = tid; i < d; i += kMaskThreads) {
      const uint64_t k = mask_key(w[i], col_value(c, c_dtype, c_stride, i));
      if ((k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & 255], 1u);
    }
    __syncthreads();
    if (tid == 0) {
      int64_t above = 0;
      int b = 255;
      for (; b > 0; --b) {
        if (above + hist[b] >= need) break;
        above += hist[b];
      }
      s_prefix = prefix | (uint64_t(b) << shift);
      s_need = need - above;
    }
    __syncthreads();
    prefix = s_prefix;
    need = s_need;
    pmask |= uint64_t(255) << shift;
  }
  // prefix is now the keep-th largest key T; `need` keys equal to T are kept,
  // the ones with the lowest indices. Each thread takes a contiguous range.
  const int64_t chunk = (d + kMaskThreads - 1) / kMaskThreads;
  const int64_t lo = tid * chunk < d ? tid * chunk : d;
  const int64_t hi = lo + chunk < d ? lo + chunk : d;
  int64_t eq = 0;
  for (int64_t i = lo; i < hi; ++i)
    eq += mask_key(w[i], col_value(c, c_dtype, c_stride, i)) == prefix;
  scan[tid] = eq;
  __syncthreads();
  if (tid == 0) {  // exclusive scan in thread order
    int64_t run = 0;
    for (int t = 0; t < kMaskThreads; ++t) {
      const int64_t v = scan[t];
      scan[t] = run;
      run += v;
    }
  }
  __syncthreads();
  int64_t rank = scan[tid];
  for (int64_t i = lo; i < hi; ++i) {
    const uint64_t k = mask_key(w[i], col_value(c, c_dtype, c_stride, i));
    uint8_t v = k > prefix ? 1 : 0;
    if (k == prefix) v = rank++ < need ? 1 : 0;
    m[i] = v;
  }
}

// Reductions and scans over a wave on the DPP network (no LDS): row shifts
// within 16 lanes, then the two row broadcasts. Lane 63 ends with the result.
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp(uint32_t old, uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(old), int(v), CTRL, ROWS, 0xf, false));
}
__device__ inline uint32_t wave_scan_add(uint32_t v) {  // inclusive, in lane order
  v += dpp<0x111, 0xf>(0u, v);  // row_shr:1, 2, 4, 8
  v += dpp<0x112, 0xf>(0u, v);
  v += dpp<0x114, 0xf>(0u, v);
  v += dpp<0x118, 0xf>(0u, v);
  v += dpp<0x142, 0xa>(0u, v);  // row_bcast:15 into rows 1 and 3
  v += dpp<0x143, 0xc>(0u, v);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ inline uint32_t wave_min(uint32_t v) {
  v = min(v, dpp<0x111, 0xf>(v, v));
  v = min(v, dpp<0x112, 0xf>(v, v));
  v = min(v, dpp<0x114, 0xf>(v, v));
  v = min(v, dpp<0x118, 0xf>(v, v));
  v = min(v, dpp<0x142, 0xa>(v, v));
  v = min(v, dpp<0x143, 0xc>(v, v));
  return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}

// Unstructured masks of rows that fit the registers of one workgroup
// (d <= T NK): thread t holds the columns (q T + t) 4 + e, e < 4, of the row,
// and their column values for all rows that its workgroup takes, so that W0 is
// read once and the column values (a cache line each when they are a Hessian's
// diagonal) once per workgroup.
//
// The keep-th largest key is found on the keys' high words, and on the low
// words of those that share the one found, by histograms over the words'
// range: the range [lo, hi] of the candidates is cut into up to kBins equal
// bins, and the bin that holds the wanted word becomes the range. It ends when
// all words of the range are kept (the usual end, after two or three passes on
// the high words: the bins follow the words' own range, where radix digits of
// a double's exponent put nearly every key into one bin) or when the range is
// a single value. Keys equal to the last one kept go by their index.
//
// Bound by each row's chain of passes and barriers rather than by HBM (5 bytes
// an element). 14336 x 4096 from a Hessian's diagonal: 124 us, 2.4 TB/s, against
// 2605 us of the radix select over global memory (k_mask_topk), which gathered
// the diagonal again in all ten of its passes over a row and met at one or two
// histogram bins. 64-bit words throughout took 188 us (130 registers, three
// workgroups a CU).
constexpr int kBinBits = 10, kBins = 1 << kBinBits;

template <int T>
struct SelectShared {
  unsigned hist[kBins];
  unsigned wave_sum[T / 64], wave_lo[T / 64], wave_hi[T / 64];
  unsigned bin, above, count;
};

struct Range {
  uint32_t lo, hi;  // inclusive
  uint32_t need;    // words of the range still to keep (>= 1)
  uint32_t count;   // words in the range
};

// Narrows r to the end described above over the words v[q] with active(q).
// The histogram is zero on entry and on return.
template <int T, int NK, typename Active>
__device__ inline void narrow(Range& r, const uint32_t (&v)[NK], Active active,
                              SelectShared<T>& sh) {
  constexpr int kPer = kBins / T, kWaves = T / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t lo = ~0u, inv_hi = ~0u;
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (active(q)) {
      lo = min(lo, v[q]);
      inv_hi = min(inv_hi, ~v[q]);
    }
  lo = wave_min(lo);
  inv_hi = wave_min(inv_hi);
  if (lane == 0) {
    sh.wave_lo[wave] = lo;
    sh.wave_hi[wave] = ~inv_hi;
  }
  __syncthreads();
  uint32_t hi = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    lo = min(lo, sh.wave_lo[w]);
    hi = max(hi, sh.wave_hi[w]);
  }
  r.lo = lo;
  r.hi = hi;
  while (r.need != r.count && r.lo != r.hi) {
    const int bits = 32 - __clz(int(r.hi - r.lo));
    const int shift = bits > kBinBits ? bits - kBinBits : 0;
#pragma unroll
    for (int q = 0; q < NK; ++q)
      if (active(q) && v[q] - r.lo <= r.hi - r.lo) atomicAdd(&sh.hist[(v[q] - r.lo) >> shift], 1u);
    __syncthreads();
    // Thread t sums and clears kPer bins; thread 0 has the highest.
    unsigned own[kPer], sum = 0;
#pragma unroll
    for (int b = 0; b < kPer; ++b) {
      const int bin = kBins - 1 - (tid * kPer + b);
      own[b] = sh.hist[bin];
      sh.hist[bin] = 0;
      sum += own[b];
    }
    unsigned upto = wave_scan_add(sum);
    if (lane == 63) sh.wave_sum[wave] = upto;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) upto += w < wave ? sh.wave_sum[w] : 0u;
    unsigned above = upto - sum;
    if (above < r.need && upto >= r.need) {  // exactly one thread
#pragma unroll
      for (int b = 0; b < kPer; ++b) {
        if (above < r.need && above + own[b] >= r.need) {
          sh.bin = unsigned(kBins - 1 - (tid * kPer + b));
          sh.above = above;
          sh.count = own[b];
        }
        above += own[b];
      }
    }
    __syncthreads();
    const uint32_t first = r.lo + (sh.bin << shift), width = (1u << shift) - 1u;
    r.need -= sh.above;
    r.count = sh.count;
    r.hi = r.hi - first > width ? first + width : r.hi;  // first + width may wrap
    r.lo = first;
  }
}

template <int T, int NK, int WAVES, bool VEC, typename C>
__global__ void __launch_bounds__(T, WAVES) k_mask_select(const float* W0, int64_t n_cols,
                                                          int64_t d, const C* c, int64_t c_stride,
                                                          int64_t keep, uint8_t* mask) {
  static_assert(NK % 4 == 0 && kBins % T == 0, "whole groups of 4 and bins per thread");
  constexpr int kWaves = T / 64;
  __shared__ SelectShared<T> sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int dd = int(d);
  auto in_row = [&](int q) { return ((q >> 2) * T + tid) * 4 + (q & 3) < dd; };
  C cv[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q)
    cv[q] = in_row(q) ? c[int64_t(((q >> 2) * T + tid) * 4 + (q & 3)) * c_stride] : C(0);
  for (int b = tid; b < kBins; b += T) sh.hist[b] = 0;

  for (int64_t j = blockIdx.x; j < n_cols; j += gridDim.x) {
    const float* w = W0 + j * d;
    uint32_t kh[NK], kl[NK];
#pragma unroll
    for (int q = 0; q < NK; q += 4) {
      const int i = ((q >> 2) * T + tid) * 4;
      float v[4] = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {  // d % 4 == 0: groups are all in or all out
        if (i < dd) {
          const float4 x = *reinterpret_cast<const float4*>(w + i);
          v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = i + e < dd ? w[i + e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t k = mask_key(v[e], double(cv[q + e]));
        kh[q + e] = uint32_t(k >> 32);
        kl[q + e] = uint32_t(k);
      }
    }
    Range r{0u, 0u, uint32_t(keep), uint32_t(dd)};
    narrow<T, NK>(r, kh, in_row, sh);
    // The last key kept is (top, r.lo) or above; below it none is.
    uint32_t top = r.lo;
    if (r.need != r.count) {
      // Rows of one high word end the first call before any barrier that follows
      // its reads of the waves' ranges, which the second call writes again.
      __syncthreads();
      narrow<T, NK>(r, kl, [&](int q) { return in_row(q) && kh[q] == top; }, sh);
    } else {
      r.lo = 0u;
    }

    uint8_t* m = mask + j * d;
    unsigned base = 0;  // equal keys at lower indices than this group's
#pragma unroll
    for (int q = 0; q < NK; q += 4) {
      const int i = ((q >> 2) * T + tid) * 4;
      uint32_t out = 0;
      if (r.need == r.count) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          out |= uint32_t(kh[q + e] > top || (kh[q + e] == top && kl[q + e] >= r.lo)) << (8 * e);
      } else {  // of the keys equal to (top, r.lo), the `need` lowest indices
        bool equal[4];
        unsigned eq = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          equal[e] = in_row(q + e) && kh[q + e] == top && kl[q + e] == r.lo;
          eq += equal[e];
        }
        const unsigned upto = wave_scan_add(eq);
        __syncthreads();
        if (lane == 63) sh.wave_sum[wave] = upto;
        __syncthreads();
        unsigned rank = base + upto - eq;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) {
          rank += v < wave ? sh.wave_sum[v] : 0u;
          base += sh.wave_sum[v];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool kept = kh[q + e] > top || (kh[q + e] == top && kl[q + e] > r.lo) ||
                            (equal[e] && rank++ < r.need);
          out |= uint32_t(kept) << (8 * e);
        }
      }
      if (VEC) {
        if (i < dd) *reinterpret_cast<uint32_t*>(m + i) = out;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + e < dd) m[i + e] = uint8_t(out >> (8 * e));
      }
    }
  }
}

// 2:4: one thread per group column; blocks of rows share its four column
// values, which stay in registers. Bound by HBM (5 bytes an element): with the
// values of a Hessian's diagonal (stride d + 1, a cache line each) read again
// for every row, their lines set the time instead. VEC: 16-byte loads of W0
// (its address is 16-byte aligned; rows are, since d % 4 == 0).
template <bool VEC>
__global__ void __launch_bounds__(kMaskThreads) k_mask_2to4(const float* W0, int64_t n_cols,
                                                            int64_t d, const void* c, int c_dtype,
                                                            int64_t c_stride, uint8_t* mask) {
  const int64_t g = int64_t(blockIdx.x) * kMaskThreads + threadIdx.x;
  if (4 * g >= d) return;
  double cv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) cv[q] = col_value(c, c_dtype, c_stride, 4 * g + q);
  for (int64_t j = blockIdx.y; j < n_cols; j += gridDim.y) {
    const int64_t e0 = j * d + 4 * g;
    float w[4];
    if (VEC) {
      const float4 v = *reinterpret_cast<const float4*>(W0 + e0);
      w[0] = v.x, w[1] = v.y, w[2] = v.z, w[3] = v.w;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = W0[e0 + q];
    }
    uint64_t k[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = mask_key(w[q], cv[q]);
    uint32_t out = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int beaten = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) beaten += (k[r] > k[q]) || (k[r] == k[q] && r < q);
      out |= uint32_t(beaten < 2) << (8 * q);
    }
    *reinterpret_cast<uint32_t*>(mask + e0) = out;
  }
}

}  // namespace

namespace {

// Launches k_mask_select for rows of at most T NK columns, at WAVES waves a
// SIMD: as many workgroups as are resident at once, so that each reads the
// column values once for all of its rows.
template <int T, int NK, int WAVES>
void launch_select(const float* W0, int64_t n_cols, int64_t d, const void* c, int c_dtype,
                   int64_t c_stride, int64_t keep, uint8_t* mask, hipStream_t s) {
  const dim3 grid(unsigned(std::min<int64_t>(n_cols, 256 * (WAVES * 256 / T)))), block(T);
  const bool vec = d % 4 == 0 && aligned16(W0);
  const float* cf = static_cast<const float*>(c);
  const double* cd = static_cast<const double*>(c);
  if (c_dtype == OPTIMA_DTYPE_F64) {
    if (vec)
      hipLaunchKernelGGL((k_mask_select<T, NK, WAVES, true, double>), grid, block, 0, s, W0,
                         n_cols, d, cd, c_stride, keep, mask);
    else
      hipLaunchKernelGGL((k_mask_select<T, NK, WAVES, false, double>), grid, block, 0, s, W0,
                         n_cols, d, cd, c_stride, keep, mask);
  } else if (vec) {
    hipLaunchKernelGGL((k_mask_select<T, NK, WAVES, true, float>), grid, block, 0, s, W0, n_cols,
                       d, cf, c_stride, keep, mask);
  } else {
    hipLaunchKernelGGL((k_mask_select<T, NK, WAVES, false, float>), grid, block, 0, s, W0, n_cols,
                       d, cf, c_stride, keep, mask);
  }
}

}  // namespace

optima_status wanda_mask(const float* W0, int64_t n_cols, int64_t d, const void* col_sq,
                         int col_dtype, int64_t col_stride, int pattern, double sparsity,
                         uint8_t* mask, hipStream_t s) {
  if (n_cols == 0) return OPTIMA_OK;
  if (pattern == OPTIMA_MASK_2TO4) {
    // About 16 workgroups of 256 threads a CU over (group columns, rows).
    const int64_t gx = ceil_div(d / 4, kMaskThreads);
    const int64_t gy = std::min<int64_t>({n_cols, std::max<int64_t>(1, 4096 / gx), 65535});
    const dim3 grid{unsigned(gx), unsigned(gy)};
    if (aligned16(W0))
      hipLaunchKernelGGL(k_mask_2to4<true>, grid, dim3(kMaskThreads), 0, s, W0, n_cols, d, col_sq,
                         col_dtype, col_stride, mask);
    else
      hipLaunchKernelGGL(k_mask_2to4<false>, grid, dim3(kMaskThreads), 0, s, W0, n_cols, d, col_sq,
                         col_dtype, col_stride, mask);
  } else {
    const int64_t keep = d - int64_t(floor(sparsity * double(d)));
    // The smallest workgroup whose registers hold a row at 16 columns a thread
    // (4096 columns: 124 us; two waves more a SIMD at 8 a thread 128 us, 1024
    // threads at 4 a thread 156 us); longer rows are read again in every pass
    // (k_mask_topk).
    if (keep <= 0 || keep >= d || d > 16384)
      hipLaunchKernelGGL(k_mask_topk, dim3(unsigned(n_cols)), dim3(kMaskThreads), 0, s, W0, d,
                         col_sq, col_dtype, col_stride, keep, mask);
    else if (d <= 1024)
      launch_select<256, 4, 8>(W0, n_cols, d, col_sq, col_dtype, col_stride, keep, mask, s);
    else if (d <= 4096)
      launch_select<256, 16, 4>(W0, n_cols, d, col_sq, col_dtype, col_stride, keep, mask, s);
    else if (d <= 8192)
      launch_select<512, 16, 4>(W0, n_cols, d, col_sq, col_dtype, col_stride, keep, mask, s);
    else
      launch_select<1024, 16, 4>(W0, n_cols, d, col_sq, col_dtype, col_stride, keep, mask, s);
  }
  OPTIMA_LAUNCH_CHECK();
  return OPTIMA_OK;
}

}  // namespace optima
