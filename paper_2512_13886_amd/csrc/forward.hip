// Forward pass of a linear layer on the calibration tokens, for the layer
// loop of Algorithm 1: its outputs y = L(x) feed the next layer's Hessian and
// the update X <- L(X) that follows the pruning of L. It also forms the
// squared output error between two weight sets. The relative layer-wise
// error of Section 4 is a ratio of such errors, each against the dense
// layer's outputs.
//
// Z = X W^T with X [n_tok][d_in] bf16 (calibration activations) and W fp32
// rounded to bf16 (round to nearest even, the weights a bf16 model stores),
// on v_mfma_f32_16x16x32_bf16 with fp32 accumulation: the 128 x 128 tile of
// the GEMM core with token rows as A and weight rows as B (both contiguous in
// d_in). Epilogue per 4 consecutive outputs: the squared difference to a
// reference Z (fp64 partial sums), the activation and the store.
#include "common.h"
#include "readback.h"
#include "gemm256.h"
#include "gemm_core.h"

namespace optima {
namespace {

// bf16 copy of W with rows padded by zeros to a multiple of the tile; flags[0]
// = 1 if W holds a NaN or Inf. One thread per 8 values (d_in % 64 == 0); VEC:
// W is 16-byte aligned. Bound by HBM: 6 bytes a value.
template <bool VEC>
__global__ void __launch_bounds__(kThreads) k_weights_bf16(const float* W, int64_t d_out,
                                                           int64_t d_in, int64_t rows_pad,
                                                           uint16_t* Wb, int* flags) {
  const int64_t i = 8 * (int64_t(blockIdx.x) * kThreads + threadIdx.x);
  if (i >= rows_pad * d_in) return;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (i < d_out * d_in) {
    if (VEC) {
      const float4 a = *reinterpret_cast<const float4*>(W + i);
      const float4 b = *reinterpret_cast<const float4*>(W + i + 4);
      v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w;
      v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = W[i + k];
    }
  }
  bool bad = false;
  uint32_t h[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    bad |= !isfinite(v[k]);
    h[k] = bf16_rne_bits(v[k]);
  }
  *reinterpret_cast<uint4*>(Wb + i) = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16),
                                                 h[4] | (h[5] << 16), h[6] | (h[7] << 16));
  if (bad) atomicOr(flags, 1);
}

__device__ inline float act_apply(int act, float z) {
  return act == OPTIMA_ACT_SILU ? z / (1.f + expf(-z)) : z;
}

// Four consecutive outputs z of token t from output n on: adds their squared
// difference to the reference y to e (with_ref) and stores the activation (Y
// and y_dtype as in k_forward).
__device__ inline void forward_chunk(float4 z, float4 y, bool with_ref, size_t o, int act, void* Y,
                                     int y_dtype, double& e) {
  if (with_ref) {
    const double a = double(z.x) - y.x, b = double(z.y) - y.y, cc = double(z.z) - y.z,
                 d = double(z.w) - y.w;
    e += a * a + b * b + cc * cc + d * d;
  }
  if (y_dtype == OPTIMA_DTYPE_F32) {
    *reinterpret_cast<float4*>(static_cast<float*>(Y) + o) =
        make_float4(act_apply(act, z.x), act_apply(act, z.y), act_apply(act, z.z),
                    act_apply(act, z.w));
  } else if (y_dtype == OPTIMA_DTYPE_BF16) {
    const uint32_t b0 = bf16_rne_bits(act_apply(act, z.x)), b1 = bf16_rne_bits(act_apply(act, z.y));
    const uint32_t b2 = bf16_rne_bits(act_apply(act, z.z)), b3 = bf16_rne_bits(act_apply(act, z.w));
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(Y) + o) =
        make_uint2(b0 | (b1 << 16), b2 | (b3 << 16));
  }
}

// The rows x 32 staged 16-byte chunks of a tile by THREADS threads, kBatch at a
// time: the batch's reference loads go out together, before any of them is
// used. staged(r, ch) is chunk ch of row r, token m0 + r, outputs n0 + 4 ch on.
template <int ROWS, int THREADS, typename Staged>
__device__ inline void forward_epilogue(Staged staged, int64_t m0, int64_t n0, int64_t n_tok,
                                        int64_t d_out, int act, void* Y, int y_dtype,
                                        const float* Y_ref, double& e) {
  constexpr int kBatch = 8;
  static_assert(ROWS * 32 % (THREADS * kBatch) == 0, "whole batches");
  const int ch = threadIdx.x & 31;
  const int64_t n = n0 + 4 * ch;
  if (n >= d_out) return;  // d_out % 4 == 0: chunks are all in or all out
#pragma unroll 1
  for (int q = 0; q < ROWS * 32 / THREADS; q += kBatch) {
    float4 y[kBatch];
    if (Y_ref) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int r = (threadIdx.x + THREADS * (q + u)) >> 5;
        const int64_t t = m0 + r < n_tok ? m0 + r : n_tok - 1;
        y[u] = *reinterpret_cast<const float4*>(Y_ref + size_t(t) * size_t(d_out) + size_t(n));
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int r = (threadIdx.x + THREADS * (q + u)) >> 5;
      if (m0 + r >= n_tok) continue;
      forward_chunk(staged(r, ch), y[u], Y_ref != nullptr,
                    size_t(m0 + r) * size_t(d_out) + size_t(n), act, Y, y_dtype, e);
    }
  }
}

// One 128 x 128 tile of Z per workgroup (tokens x outputs). A y_dtype other
// than BF16 or F32 stores nothing; err_part[blockIdx.x] receives the tile's sum of
// (Z - Y_ref)^2. Nothing is written if *flags is set (W is not finite).
__global__ void __launch_bounds__(Tile128::kThreads) k_forward(const char* X, int64_t n_tok,
                                                               int64_t d_in, const uint16_t* Wb,
                                                               int64_t d_out, int act,
                                                               void* Y, int y_dtype,
                                                               const float* Y_ref,
                                                               double* err_part,
                                                               const int* flags) {
  if (*flags) return;
  using Cfg = Tile128;
  __shared__ __attribute__((aligned(1024))) char lds0[Cfg::kBufBytes];
  __shared__ __attribute__((aligned(1024))) char lds1[Cfg::kBufBytes];
  __shared__ double red[Cfg::kThreads / 64];
  const int tiles_m = int((n_tok + kTile - 1) / kTile);
  const int tiles_n = int((d_out + kTile - 1) / kTile);
  int tm, tn;
  tile_of_block(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, &tm, &tn);
  const int64_t m0 = int64_t(tm) * kTile, n0 = int64_t(tn) * kTile;
  const int64_t pitch = d_in * 2;  // bytes per row of X and of Wb
  Operands<Cfg> src;
#pragma unroll
  for (int i = 0; i < Cfg::kLoadsA; ++i) {
    int64_t t = m0 + load_row<Cfg>(i);
    t = t < n_tok ? t : n_tok - 1;
    src.a[i] = X + t * pitch + load_seg_bytes<Cfg>(i);
  }
  const char* wb = reinterpret_cast<const char*>(Wb);
#pragma unroll
  for (int i = 0; i < Cfg::kLoadsB; ++i)
    src.b[i] = wb + (n0 + load_row<Cfg>(i)) * pitch + load_seg_bytes<Cfg>(i);
  f4 acc[Cfg::MB][Cfg::NB];
  gemm_tile_mainloop<Cfg, Bf16Tag>(acc, src, int(pitch / Cfg::SRB), lds0, lds1);
  stage_tile<Cfg>(acc, lds0, lds1);
  __syncthreads();

  double e = 0.0;
  forward_epilogue<kTile, Cfg::kThreads>(
      [&](int r, int ch) { return staged_chunk(lds0, lds1, r, ch); }, m0, n0, n_tok, d_out, act, Y,
      y_dtype, Y_ref, e);
  if (err_part) {
    e = block_sum(e, red);
    if (threadIdx.x == 0) err_part[blockIdx.x] = e;
  }
}

// The same on 256 x 256 tiles (gemm256.h), for products that fill the chip with
// them. The accumulators are staged through the stage buffers in two halves of
// 128 columns: row t of a half takes 512 bytes, rows 32 h .. 32 h + 31 in
// buffer h, 16-byte chunk c of row r at physical chunk c ^ (r & 31).
__global__ void __launch_bounds__(Tile256::kThreads) k_forward256(const char* X, int64_t n_tok,
                                                                  int64_t d_in, const uint16_t* Wb,
                                                                  int64_t d_out, int64_t w_rows,
                                                                  int act, void* Y, int y_dtype,
                                                                  const float* Y_ref,
                                                                  double* err_part,
                                                                  const int* flags) {
  if (*flags) return;
  __shared__ __attribute__((aligned(1024))) char l0[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l1[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l2[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l3[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l4[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l5[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l6[Tile256::kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char l7[Tile256::kHalfBytes];
  __shared__ double red[Tile256::kWaves];
  const int tiles_m = int((n_tok + Tile256::BM - 1) / Tile256::BM);
  const int tiles_n = int((d_out + Tile256::BN - 1) / Tile256::BN);
  int tm, tn;
  tile_of_block(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, &tm, &tn);
  const int64_t m0 = int64_t(tm) * Tile256::BM, n0 = int64_t(tn) * Tile256::BN;
  const int64_t pitch = d_in * 2;  // bytes per row of X and of Wb
  Operands256 src;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < Tile256::kHalfLoads; ++i) {
      const int64_t r = 128 * h + t256_load_row(i);
      src.a[h][i] = X + std::min(m0 + r, n_tok - 1) * pitch + t256_seg_bytes(i);
      src.b[h][i] = reinterpret_cast<const char*>(Wb) + std::min(n0 + r, w_rows - 1) * pitch +
                    t256_seg_bytes(i);
    }
  Acc256 acc;
  gemm256_mainloop<Bf16Tag>(acc, src, int(pitch / Tile256::kSRB), l0, l1, l2, l3, l4, l5, l6, l7,
                            [] {});

  double e = 0.0;
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    if (qb) __syncthreads();
#pragma unroll
    for (int qa = 0; qa < 2; ++qa)
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = t256_row(qa, mi, k);
#pragma unroll
          for (int ni = 0; ni < 2; ++ni) {
            const int c = t256_col(0, ni);
            *reinterpret_cast<float*>(t256_stage_row(l0, l1, l2, l3, l4, l5, l6, l7, r) +
                                      ((c >> 2) ^ (r & 31)) * 16 + (c & 3) * 4) =
                acc.q[qa][qb][mi][ni][k];
          }
        }
    __syncthreads();
    forward_epilogue<Tile256::BM, Tile256::kThreads>(
        [&](int r, int ch) {
          return *reinterpret_cast<const float4*>(
              t256_stage_row(l0, l1, l2, l3, l4, l5, l6, l7, r) + ((ch ^ (r & 31)) * 16));
        },
        m0, n0 + 128 * qb, n_tok, d_out, act, Y, y_dtype, Y_ref, e);
  }
  if (err_part) {
    for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (int w = 0; w < Tile256::kWaves; ++w) sum += red[w];
      err_part[blockIdx.x] = sum;
    }
  }
}

// err_out = sum of the n per-tile partials, in a fixed order.
__global__ void __launch_bounds__(kThreads) k_err_reduce(const double* part, int n,
                                                         double* err_out, const int* flags) {
  if (*flags) return;
  __shared__ double red[kThreads / 64];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += kThreads) s += part[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) *err_out = s;
}

// Whether the 256 x 256 tile takes a product: it fills a CU with one workgroup,
// the 128 x 128 tile with two. In units of the former's round over 256 CUs, a
// round of the latter (half the outputs, at 0.62 of the rate) takes 0.8.
// Measured at d_in = 4096, fp32 outputs: 4096 x 4096 (1 round against 2) 138
// against 168 us, 32768 x 4096 878 against 1126 us; 6000 x 1024 (1 against 1)
// stays at the small tile, 88 us.
bool forward_wide(int64_t n_tok, int64_t d_out) {
  constexpr int64_t kCus = 256;
  const int64_t wide = ceil_div(ceil_div(n_tok, Tile256::BM) * ceil_div(d_out, Tile256::BN), kCus);
  const int64_t small = ceil_div(ceil_div(n_tok, kTile) * ceil_div(d_out, kTile), 2 * kCus);
  return 5 * wide <= 4 * small;
}

struct FwdLayout {
  uint16_t* Wb;
  double* part;
  int* flags;
};

FwdLayout carve_forward(void* ws, int64_t n_tok, int64_t d_in, int64_t d_out, size_t* bytes) {
  Carver c(ws);
  FwdLayout l{};
  const int64_t rows_pad = round_up(d_out, kTile);
  l.Wb = c.take<uint16_t>(size_t(rows_pad) * size_t(d_in));
  l.part = c.take<double>(size_t(ceil_div(n_tok, kTile) * ceil_div(d_out, kTile)));
  l.flags = c.take<int>(4);
  if (bytes) *bytes = c.bytes();
  return l;
}

}  // namespace

size_t linear_forward_workspace_bytes(int64_t n_tok, int64_t d_in, int64_t d_out) {
  size_t b = 0;
  carve_forward(nullptr, n_tok, d_in, d_out, &b);
  return b;
}

optima_status linear_forward(const void* X, int64_t n_tok, int64_t d_in, const float* W,
                             int64_t d_out, int act, void* Y, int y_dtype, const float* Y_ref,
                             double* err_out, void* ws, hipStream_t s) {
  FwdLayout l = carve_forward(ws, n_tok, d_in, d_out, nullptr);
  const int64_t rows_pad = round_up(d_out, kTile);
  OPTIMA_HIP_TRY(hipMemsetAsync(l.flags, 0, sizeof(int), s));
  const dim3 wg(unsigned(ceil_div(rows_pad * d_in, int64_t(8) * kThreads)));
  if (aligned16(W))
    hipLaunchKernelGGL(k_weights_bf16<true>, wg, dim3(kThreads), 0, s, W, d_out, d_in, rows_pad,
                       l.Wb, l.flags);
  else
    hipLaunchKernelGGL(k_weights_bf16<false>, wg, dim3(kThreads), 0, s, W, d_out, d_in, rows_pad,
                       l.Wb, l.flags);
  OPTIMA_LAUNCH_CHECK();
  // The products are queued behind the flag's copy and check the flag
  // themselves, so that the GPU does not wait for the host in between.
  PendingReadBack finite;
  OPTIMA_HIP_TRY(finite.begin(l.flags, sizeof(int), s));
  if (n_tok > 0) {
    int64_t tiles = ceil_div(n_tok, Tile256::BM) * ceil_div(d_out, Tile256::BN);
    if (forward_wide(n_tok, d_out)) {
      hipLaunchKernelGGL(k_forward256, dim3(unsigned(tiles)), dim3(Tile256::kThreads), 0, s,
                         static_cast<const char*>(X), n_tok, d_in, l.Wb, d_out, rows_pad, act, Y,
                         Y ? y_dtype : -1, err_out ? Y_ref : nullptr, err_out ? l.part : nullptr,
                         l.flags);
    } else {
      tiles = ceil_div(n_tok, kTile) * ceil_div(d_out, kTile);
      hipLaunchKernelGGL(k_forward, dim3(unsigned(tiles)), dim3(Tile128::kThreads), 0, s,
                         static_cast<const char*>(X), n_tok, d_in, l.Wb, d_out, act, Y,
                         Y ? y_dtype : -1, err_out ? Y_ref : nullptr, err_out ? l.part : nullptr,
                         l.flags);
    }
    OPTIMA_LAUNCH_CHECK();
    if (err_out) {
      hipLaunchKernelGGL(k_err_reduce, dim3(1), dim3(kThreads), 0, s, l.part, int(tiles), err_out,
                         l.flags);
      OPTIMA_LAUNCH_CHECK();
    }
  }
  int flag = 0;
  OPTIMA_HIP_TRY(finite.end(&flag));
  if (flag) return OPTIMA_E_NONFINITE;
  if (n_tok == 0 && err_out) OPTIMA_HIP_TRY(hipMemsetAsync(err_out, 0, sizeof(double), s));
  return OPTIMA_OK;
}

}  // namespace optima
