// Layer Hessian H = X^T X (Section 3.4 "Hessian calculation") and damping.
//
// The tokens arrive row-major, X[t][i]. Both MFMA operands of X^T X need the
// token index contiguous, so each slab of up to kMaxSlab tokens is first
// transposed into XT[i][t] (features padded to the 128-wide tile, tokens
// padded with zeros to a whole 128-byte stage). The product then runs on the
// lower-triangular 128x128 tiles only, each tile's slab of tokens split into
// `splits` contiguous ranges so that small layers still fill the GPU. Every
// (tile, split) workgroup adds its partial sum into a private fp32 buffer, so
// no atomics are involved and the result is deterministic. A final pass sums
// the partials in split order, adds the incoming H when accumulating, and
// writes each lower-triangle value to both (i, j) and (j, i): H comes out
// exactly symmetric.
//
// bf16 tokens use v_mfma_f32_16x16x32_bf16 (the bf16 x bf16 products are exact
// in fp32); fp32 tokens use v_mfma_f32_16x16x4_f32.
//
// bf16 tokens with d a multiple of 256 (every transformer width here) take a
// direct path instead: no transpose. Token rows go from X straight into LDS
// and the MFMA operands are gathered from there with gfx950's transposing LDS
// read, on 256 x 256 lower-triangular tiles; the whole token range is one
// launch, split along the tokens so that the tiles fill all CUs evenly.
#include "common.h"
#include "gemm_core.h"

namespace optima {
namespace {

constexpr int64_t kMaxSlab = 65536;

struct HessPlan {
  int64_t dp, esz, kse, slab, tiles;
  int splits;
  size_t xt_elems, part_elems;
};

HessPlan plan(int64_t n_tok, int64_t d, int dtype) {
  HessPlan p{};
  p.dp = round_up(d, kTile);
  p.esz = dtype == OPTIMA_DTYPE_BF16 ? 2 : 4;
  p.kse = kStageRowBytes / p.esz;  // tokens per 128-byte stage
  p.slab = std::min<int64_t>(round_up(std::max<int64_t>(n_tok, 1), p.kse), kMaxSlab);
  const int64_t T = p.dp / kTile;
  p.tiles = T * (T + 1) / 2;
  const int64_t stages = p.slab / p.kse;
  p.splits = int(std::max<int64_t>(1, std::min<int64_t>({ceil_div(2048, p.tiles), 64, stages})));
  p.xt_elems = size_t(p.dp) * size_t(p.slab);
  p.part_elems = size_t(p.splits) * size_t(p.dp) * size_t(p.dp);
  return p;
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_transpose(const T* X, int64_t d, int64_t t0,
                                                        int64_t rows, int64_t cols_pad, int64_t dp,
                                                        T* XT) {
  __shared__ T tile[64][65];
  const int64_t tt0 = int64_t(blockIdx.x) * 64;  // token within the slab
  const int64_t f0 = int64_t(blockIdx.y) * 64;   // feature
  for (int e = threadIdx.x; e < 64 * 64; e += kThreads) {
    const int r = e >> 6, c = e & 63;
    const int64_t tt = tt0 + r, f = f0 + c;
    T v{};
    if (tt < rows && f < d) v = X[(t0 + tt) * d + f];
    tile[r][c] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += kThreads) {
    const int r = e >> 6, c = e & 63;  // r: feature, c: token
    const int64_t f = f0 + r, tt = tt0 + c;
    if (f < dp && tt < cols_pad) XT[f * cols_pad + tt] = tile[c][r];
  }
}

// Lower-triangular tile index -> (ti, tj), ti >= tj.
__device__ inline void tri_tile(int idx, int* ti, int* tj) {
  int i = int((sqrtf(8.f * float(idx) + 1.f) - 1.f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= idx) ++i;
  while (i * (i + 1) / 2 > idx) --i;
  *ti = i;
  *tj = idx - i * (i + 1) / 2;
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_syrk(const char* XT, int64_t pitch_bytes,
                                                   int stages, int splits, int64_t dp,
                                                   float* part, int first) {
  __shared__ __attribute__((aligned(1024))) char lds0[Tile128::kBufBytes];
  __shared__ __attribute__((aligned(1024))) char lds1[Tile128::kBufBytes];
  const int tile = blockIdx.x / splits;
  const int sp = blockIdx.x - tile * splits;
  int ti, tj;
  tri_tile(tile, &ti, &tj);
  const int s0 = int(int64_t(stages) * sp / splits);
  const int s1 = int(int64_t(stages) * (sp + 1) / splits);
  using Cfg = Tile128;
  Operands<Cfg> src;
  const int64_t k_off = int64_t(s0) * Cfg::SRB;
#pragma unroll
  for (int i = 0; i < Cfg::kLoadsA; ++i)
    src.a[i] = XT + (int64_t(ti) * kTile + load_row<Cfg>(i)) * pitch_bytes + k_off +
               load_seg_bytes<Cfg>(i);
#pragma unroll
  for (int i = 0; i < Cfg::kLoadsB; ++i)
    src.b[i] = XT + (int64_t(tj) * kTile + load_row<Cfg>(i)) * pitch_bytes + k_off +
               load_seg_bytes<Cfg>(i);
  f4 acc[Cfg::MB][Cfg::NB];
  gemm_tile_mainloop<Cfg, T>(acc, src, s1 - s0, lds0, lds1);
  float* P = part + size_t(sp) * size_t(dp) * size_t(dp);
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t i = int64_t(ti) * kTile + acc_row<Cfg>(mi, e);
#pragma unroll
      for (int ni = 0; ni < 4; ++ni) {
        const int64_t j = int64_t(tj) * kTile + acc_col<Cfg>(ni);
        float* q = P + i * dp + j;
        *q = first ? acc[mi][ni][e] : *q + acc[mi][ni][e];
      }
    }
}

// Sums the split partials of the 64x64 block (bi, bj), bi >= bj, into H and
// mirrors it to the upper triangle.
__global__ void __launch_bounds__(kThreads) k_hess_reduce(const float* part, int splits, int64_t dp,
                                                          int64_t d, float* H, int accumulate) {
  __shared__ float tile[64][65];
  int bi, bj;
  tri_tile(blockIdx.x, &bi, &bj);
  for (int e = threadIdx.x; e < 64 * 64; e += kThreads) {
    const int r = e >> 6, c = e & 63;
    const int64_t i = int64_t(bi) * 64 + r, j = int64_t(bj) * 64 + c;
    float v = 0.f;
    if (i < d && j < d && (bi > bj || r >= c)) {
      for (int s = 0; s < splits; ++s) v += part[size_t(s) * dp * dp + i * dp + j];
      if (accumulate) v = H[i * d + j] + v;
      H[i * d + j] = v;
    }
    tile[r][c] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += kThreads) {
    const int r = e >> 6, c = e & 63;  // output row bj*64 + r, column bi*64 + c
    const int64_t i = int64_t(bj) * 64 + r, j = int64_t(bi) * 64 + c;
    if (i < d && j < d && (bi > bj || c > r)) H[i * d + j] = tile[c][r];
  }
}

// The same for d % 4 == 0 with 16-byte chunks of 4 columns: thread t takes
// chunks t, t + 256, t + 512 and t + 768 of the block and adds the splits
// of all four in split order, so 16 loads are in flight per step. The sums
// are those of k_hess_reduce, bit for bit.
__global__ void __launch_bounds__(kThreads) k_hess_reduce4(const float* part, int splits, int64_t dp,
                                                           int64_t d, float* H, int accumulate) {
  static_assert(kThreads == 256, "four chunks per thread cover the 64 x 64 block");
  __shared__ float tile[64][65];
  int bi, bj;
  tri_tile(blockIdx.x, &bi, &bj);
  float4 v[4];
  int64_t off[4];
  bool in[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int ch = threadIdx.x + kThreads * q, r = ch >> 4, c = 4 * (ch & 15);
    const int64_t i = int64_t(bi) * 64 + r, j = int64_t(bj) * 64 + c;
    in[q] = i < d && j < d;  // d % 4 == 0: chunks are all in or all out
    off[q] = in[q] ? i * dp + j : 0;
    v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const size_t plane = size_t(dp) * size_t(dp);
#pragma unroll 2
  for (int sp = 0; sp < splits; ++sp) {
    const float* P = part + size_t(sp) * plane;
    float4 t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) t[q] = *reinterpret_cast<const float4*>(P + off[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q].x += t[q].x;
      v[q].y += t[q].y;
      v[q].z += t[q].z;
      v[q].w += t[q].w;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int ch = threadIdx.x + kThreads * q, r = ch >> 4, c = 4 * (ch & 15);
    const int64_t i = int64_t(bi) * 64 + r, j = int64_t(bj) * 64 + c;
    float e[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
    if (in[q]) {
      float* h = H + i * d + j;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool lower = bi > bj || r >= c + k;
        if (!lower) e[k] = 0.f;
        else if (accumulate) e[k] = h[k] + e[k];
      }
      if (bi > bj) {
        *reinterpret_cast<float4*>(h) = make_float4(e[0], e[1], e[2], e[3]);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (r >= c + k) h[k] = e[k];
      }
    } else {
      e[0] = e[1] = e[2] = e[3] = 0.f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) tile[r][c + k] = e[k];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += kThreads) {
    const int r = e >> 6, c = e & 63;  // output row bj*64 + r, column bi*64 + c
    const int64_t i = int64_t(bj) * 64 + r, j = int64_t(bi) * 64 + c;
    if (i < d && j < d && (bi > bj || c > r)) H[i * d + j] = tile[c][r];
  }
}

// Shared diagonal preconditioning: D_i = diag(H)_i^(-1/2) (computed in fp64,
// 1 where the diagonal is not positive and finite).
__global__ void __launch_bounds__(kThreads) k_jacobi_d(const float* H, int64_t d, float* D) {
  const int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= d) return;
  const double h = H[i * d + i];
  D[i] = (h > 0.0 && isfinite(h)) ? float(1.0 / sqrt(h)) : 1.f;
}

// H_ij <- H_ij (D_i D_j): the factor is the same product for (i, j) and
// (j, i), so an exactly symmetric H stays exactly symmetric.
__global__ void __launch_bounds__(kThreads) k_jacobi_scale(float* H, int64_t d, const float* D) {
  const int64_t total = d * d;
  for (int64_t e = int64_t(blockIdx.x) * kThreads + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * kThreads) {
    const int64_t i = e / d, j = e - i * d;
    H[e] = H[e] * (D[i] * D[j]);
  }
}

__global__ void __launch_bounds__(1024) k_damp(float* H, int64_t d, float rel, float* lambda_out) {
  __shared__ double red[16];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < d; i += 1024) s += double(H[i * d + i]);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  double tr = 0.0;
  for (int w = 0; w < 16; ++w) tr += red[w];
  const double lam = double(rel) * tr / double(d);
  if (threadIdx.x == 0) *lambda_out = isfinite(lam) ? float(lam) : __builtin_nanf("");
  if (!isfinite(lam)) return;
  for (int64_t i = threadIdx.x; i < d; i += 1024) H[i * d + i] = float(double(H[i * d + i]) + lam);
}

// ---------------------------------------------------------------------------
// Direct path (bf16, d % 256 == 0)
// ---------------------------------------------------------------------------
//
// Workgroup: one 256 x 256 output tile (ti, tj), ti >= tj, over a contiguous
// range of 64-token stages; 8 waves in a 4 x 2 grid, each wave owning 64 x
// 128 outputs (4 x 8 blocks of 16 x 16). The stages stream through a ring of
// four LDS buffers of 32 tokens each, so that while one buffer is read the
// loads of the next three are in flight. Buffer: block A holds
// X[t][256 ti + 0..255] and block B X[t][256 tj + 0..255] for its 32 tokens,
// one 512-byte row per token, written by direct loads (one wave load = 1 KiB
// = 2 token rows). Within a row the 16-byte segment g sits at physical
// segment g ^ swz(row), which keeps both the loads' writes and the
// transposing reads free of bank conflicts.
//
// Operands: ds_read_b64_tr_b16 treats the eight-byte reads of each 16-lane
// group as a 4 x 16 matrix of 16-bit values (lane j supplies row j / 4,
// columns 4 (j % 4) .. 4 (j % 4) + 3) and returns column i to lane i. Lanes
// j of group g address token row 8 g + 4 h + j / 4 and features
// f + 4 (j % 4): lane i then holds tokens 8 g + 4 h + 0..3 of feature f + i,
// and the reads for h = 0 and h = 1 together give the 8 consecutive tokens
// that a 16x16x32 bf16 MFMA takes from lane (g, i), for both operands. The
// output block (lane, e) is then H[f_a + 4 g + e][f_b + i] as in the NT core.
namespace dt {
constexpr int kRows = 64;                   // tokens per stage (unit of the token splits)
constexpr int kBufRows = 32;                // tokens per ring buffer (one MFMA K step)
constexpr int kRing = 4;                    // ring buffers
constexpr int kBlock = 256;                 // features per operand block (tile side)
constexpr int kRowBytes = 2 * kBlock;       // 512
constexpr int kBlockBytes = kBufRows * kRowBytes;
constexpr int kBufBytes = 2 * kBlockBytes;  // 32 KiB per ring buffer
constexpr int kMaxSplits = 64;
constexpr int kCus = 256;                   // MI355X compute units (sizing only)

// Wave layout of the 256 x 256 tile: WAVES / 2 x 2 waves; with 8 waves each
// owns 64 x 128 outputs and two waves share each SIMD. (Four waves of
// 128 x 128 read a third fewer LDS bytes per MFMA, but with one wave per SIMD
// nothing hides the LDS and load latency: measured 1.5 times slower.)
template <int WAVES>
struct Cfg {
  static constexpr int kWaves = WAVES;
  static constexpr int kThreads = 64 * WAVES;
  static constexpr int WGN = 2, WGM = WAVES / WGN;
  static constexpr int kMB = kBlock / WGM / 16, kNB = kBlock / WGN / 16;
  static constexpr int kLoads = kBlockBytes / 1024 / WAVES;  // wave loads per block per thread
  static constexpr int kBufLoads = 2 * kLoads;                // per buffer (blocks A and B)
};

// Physical XOR of the 16-byte segment index for token row r of a stage:
// flips segment bits 1-3 by (r & 3) and bit 3 of r.
__device__ inline int swz(int r) { return 2 * ((r & 3) | (((r >> 3) & 1) << 2)); }

typedef short v4s __attribute__((ext_vector_type(4)));

__device__ inline uint2 tr_read(const char* p) {
  const v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4s*)(p));
  return __builtin_bit_cast(uint2, v);
}

// Direct loads of one ring buffer. Round i of this thread fetches token row
// row0 + 2 WAVES i (row0 = 2 wave + lane / 32) at physical segment lane % 32;
// `a` / `b` point at that row's A / B block for round 0 without the segment
// offset, seg[i & 1] is the logical segment's byte offset for the round.
template <typename C>
__device__ inline void issue(const char* a, const char* b, int64_t round_bytes, const int (&seg)[2],
                             char* buf) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < C::kLoads; ++i)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(a + i * round_bytes + seg[i & 1]),
        (__attribute__((address_space(3))) void*)(buf + (i * C::kWaves + wave) * 1024), 16, 0, 0);
#pragma unroll
  for (int i = 0; i < C::kLoads; ++i)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(b + i * round_bytes + seg[i & 1]),
        (__attribute__((address_space(3))) void*)(buf + kBlockBytes + (i * C::kWaves + wave) * 1024),
        16, 0, 0);
}

// Operand fragments of the 32 tokens in ring buffer `buf`.
template <typename C>
__device__ inline void read_frags(const char* buf, uint4 (&a)[C::kMB], uint4 (&b)[C::kNB]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WGN, wn = wave % C::WGN;
  const int g = lane >> 4, j = lane & 15;
  // Token row 8 g + 4 h + j / 4 has (row & 3) = j / 4 and bit 3 of the row
  // equal to g & 1, so its swizzle depends on the lane only.
  const int sw = 2 * ((j >> 2) | ((g & 1) << 2));
  const int intra = 8 * (j & 1);
  const int seg_lane = (j & 3) >> 1;
  const char* A0 = buf + (8 * g + (j >> 2)) * kRowBytes;
  const char* A1 = A0 + 4 * kRowBytes;
#pragma unroll
  for (int mi = 0; mi < C::kMB; ++mi) {
    const int o = (((((wm * C::kMB + mi) * 16) >> 3) + seg_lane) ^ sw) * 16 + intra;
    const uint2 lo = tr_read(A0 + o), hi = tr_read(A1 + o);
    a[mi] = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
#pragma unroll
  for (int ni = 0; ni < C::kNB; ++ni) {
    const int o = (((((wn * C::kNB + ni) * 16) >> 3) + seg_lane) ^ sw) * 16 + intra;
    const uint2 lo = tr_read(A0 + kBlockBytes + o), hi = tr_read(A1 + kBlockBytes + o);
    b[ni] = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
}

template <typename C>
__device__ inline void mfma_step(f4 (&acc)[C::kMB][C::kNB], const uint4 (&a)[C::kMB],
                                 const uint4 (&b)[C::kNB]) {
#pragma unroll
  for (int mi = 0; mi < C::kMB; ++mi)
#pragma unroll
    for (int ni = 0; ni < C::kNB; ++ni)
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, a[mi]), __builtin_bit_cast(bf16x8, b[ni]), acc[mi][ni], 0, 0,
          0);
}

template <typename C>
__device__ inline void compute(f4 (&acc)[C::kMB][C::kNB], const char* buf) {
  constexpr int kReads = 2 * (C::kMB + C::kNB), kMfma = C::kMB * C::kNB;
  uint4 a[C::kMB], b[C::kNB];
  read_frags<C>(buf, a, b);
  mfma_step<C>(acc, a, b);
  __builtin_amdgcn_sched_group_barrier(0x020, C::kBufLoads, 0);
  __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
  __builtin_amdgcn_sched_group_barrier(0x008, kMfma, 0);
}

// One step of the ring: buffer `cur` holds the next 32 tokens once this
// wave's loads other than the two most recent buffers' have landed and every
// wave has arrived (so every wave is also done reading `nxt`, read one step
// earlier); then the loads of the buffer three ahead go to `nxt` and `cur` is
// consumed.
template <typename C>
__device__ inline void ring_step(f4 (&acc)[C::kMB][C::kNB], const char* a, const char* b,
                                 int64_t round_bytes, const int (&seg)[2], char* cur, char* nxt) {
  ring_barrier<2 * C::kBufLoads>();
  issue<C>(a, b, round_bytes, seg, nxt);
  compute<C>(acc, cur);
}

}  // namespace dt

// Lower-triangle tile (ti >= tj) of position idx in an order that keeps
// nearby positions on few feature blocks: the triangle of nt blocks is cut
// into super-tiles of 4 x 4 blocks, taken row by row (SI >= SJ), and each
// super-tile's tiles row by row. 32 consecutive positions touch 8 to 12
// blocks instead of nearly all of them.
__device__ inline void grouped_tri_tile(int idx, int nt, int* ti, int* tj) {
  constexpr int G = 4;
  const int ns = (nt + G - 1) / G;
  *ti = 0;
  *tj = 0;
  for (int SI = 0; SI < ns; ++SI)
    for (int SJ = 0; SJ <= SI; ++SJ) {
      const int i0 = G * SI, i1 = min(i0 + G, nt), j0 = G * SJ, j1 = min(j0 + G, nt);
      const int w = j1 - j0, m = i1 - i0;
      const int cnt = SI != SJ ? m * w : m * (m + 1) / 2;
      if (idx < cnt) {
        if (SI != SJ) {
          *ti = i0 + idx / w;
          *tj = j0 + idx % w;
        } else {
          int r = 0;
          while (idx > r) idx -= ++r;
          *ti = i0 + r;
          *tj = j0 + idx;
        }
        return;
      }
      idx -= cnt;
    }
}

// X: [full * 64][d] bf16 (full >= 1), followed, if not NULL, by the 64 rows of
// `tail`. The work units are the (split, tile) pairs of the triangle of d / 256
// blocks; split sp covers stages [full sp / splits, full (sp + 1) / splits), and
// the tail is one split more. The dispatcher
// sends workgroup b to XCD b % 8, so XCD x runs workgroups x, x + 8, ... in
// that order. XCD x owns the x-th eighth of the tiles in grouped_tri_tile
// order (a few feature blocks) for every split, and runs them split by
// split. Its 32 resident workgroups then share one or two token ranges and
// few blocks, which its L2 fetches once for all of them; and all eight XCDs
// move through the tokens together, so the device-wide cache serves one
// XCD's misses to the others. The grid is 8 times the largest XCD share;
// workgroups beyond their XCD's share exit at once. With `spread` (few tiles,
// whose eighths would leave XCDs idle) workgroup b takes unit b instead.
// The partial sums are part[0] for split 0, part[1] for the tail, then the other
// splits ([d][d] fp32 each): sums in that order, few rows to few rows first.
// FUSED: one workgroup runs all ranges of a tile, the tail's first, and does
// H (+)= their sum, both triangles. Registers hold one 256 x 256 fp32 tile, so
// the running sum waits in part[tile] (256 KiB, thread by thread, 16 bytes a
// lane) while a range is summed; only its own thread reads an entry back. The
// sums are added in the order of k_hess_reduce: H is the same bit for bit.
template <int WAVES, bool FUSED>
__global__ void __launch_bounds__(64 * WAVES) k_syrk_direct(const uint16_t* X,
                                                            const uint16_t* tail, int64_t d,
                                                            int full, int splits, int spread,
                                                            float* part, float* H,
                                                            int accumulate) {
  using namespace dt;
  using C = Cfg<WAVES>;
  __shared__ __attribute__((aligned(1024))) char lds0[kBufBytes];
  __shared__ __attribute__((aligned(1024))) char lds1[kBufBytes];
  __shared__ __attribute__((aligned(1024))) char lds2[kBufBytes];
  __shared__ __attribute__((aligned(1024))) char lds3[kBufBytes];
  static_assert(kRing == 4 && kRows == 2 * kBufRows, "the loop below is written for this ring");
  const int nt = int(d / kBlock);
  const int n_tiles = nt * (nt + 1) / 2;
  int t0 = 0, tx = n_tiles, l = blockIdx.x;
  if (!spread) {
    const int x = blockIdx.x & 7;
    t0 = int(int64_t(n_tiles) * x / 8);
    tx = int(int64_t(n_tiles) * (x + 1) / 8) - t0;
    l = blockIdx.x >> 3;
  }
  const int tails = tail != nullptr;
  if (int64_t(l) >= int64_t(tx) * (FUSED ? 1 : splits + tails)) return;
  const int tile = t0 + l % tx;
  int sp = l / tx;
  int ti, tj;
  grouped_tri_tile(tile, nt, &ti, &tj);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = 2 * wave + (lane >> 5);
  const int seg[2] = {((lane & 31) ^ swz(row)) * 16, ((lane & 31) ^ swz(row + 2 * WAVES)) * 16};
  const int64_t row_bytes = d * 2;
  const int64_t round_bytes = 2 * WAVES * row_bytes;
  const int64_t buf_bytes = kBufRows * row_bytes;
  // The workgroup's nb buffers of 32 tokens (at least one stage of two).
  const bool rest = !FUSED && sp == splits;  // the tail's unit
  const int s0 = FUSED || rest ? 0 : int(int64_t(full) * sp / splits);
  const int s1 = FUSED ? full + tails : rest ? 1 : int(int64_t(full) * (sp + 1) / splits);
  const int nb = 2 * (s1 - s0);
  // This thread's first rows of blocks ti and tj in buffer 0, and the offset of
  // buffer q: in X, or (FUSED) first in the tail's two buffers (a scalar, so that
  // a step adds it with the rest of the addresses). Loads past the last buffer
  // repeat it (into buffers nobody reads again) so that every step waits for the
  // same count; they are drained after the loop.
  const char* x0 = reinterpret_cast<const char*>(rest ? tail : X) + int64_t(s0) * kRows * row_bytes;
  const char* xa = x0 + row * row_bytes + int64_t(ti) * kBlock * 2;
  const char* xb = x0 + row * row_bytes + int64_t(tj) * kBlock * 2;
  const int q_x = FUSED ? 2 * tails : 0;
  const int64_t to_tail = int64_t(reinterpret_cast<uintptr_t>(tail)) -
                          int64_t(reinterpret_cast<uintptr_t>(x0)) + q_x * buf_bytes;
  auto at = [&](int q) {
    q = q < nb ? q : nb - 1;
    if (!FUSED) return int64_t(uint32_t(q)) * buf_bytes;
    return (q - q_x) * buf_bytes + (q < q_x ? to_tail : int64_t(0));
  };
  f4 acc[C::kMB][C::kNB];
#pragma unroll
  for (int mi = 0; mi < C::kMB; ++mi)
#pragma unroll
    for (int ni = 0; ni < C::kNB; ++ni) acc[mi][ni] = f4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int q, char* cur, char* nxt) {
    const int64_t off = at(q);
    ring_step<C>(acc, xa + off, xb + off, round_bytes, seg, cur, nxt);
  };
  // FUSED: after buffer q - 1, if a range but the last ends there, its sum joins
  // the running sum. The ring goes on across ranges; the stores are drained, so
  // the counts that its steps wait for stay those of its loads. (The opaque base
  // and the barriers keep the compiler from holding 32 addresses, or all loads,
  // in registers that it would have to spill for them.)
  f4* const sums = reinterpret_cast<f4*>(part) + size_t(tile) * (kBlock * kBlock / 4);
  int cut = FUSED ? (tails ? 2 : 2 * int(int64_t(full) / splits)) : 0;
  auto range_end = [&](int q) {
    if (!FUSED || q != cut || q == nb) return;
    f4* Q = sums;
    asm volatile("" : "+s"(Q));
#pragma unroll
    for (int mi = 0; mi < C::kMB; ++mi) {
      f4* const q4 = Q + mi * C::kNB * 64 * WAVES;
      if (sp > 0) {
        f4 sum[C::kNB];
#pragma unroll
        for (int ni = 0; ni < C::kNB; ++ni) sum[ni] = q4[ni * 64 * WAVES + threadIdx.x];
#pragma unroll
        for (int ni = 0; ni < C::kNB; ++ni) acc[mi][ni] = sum[ni] + acc[mi][ni];
      }
#pragma unroll
      for (int ni = 0; ni < C::kNB; ++ni) {
        q4[ni * 64 * WAVES + threadIdx.x] = acc[mi][ni];
        acc[mi][ni] = f4{0.f, 0.f, 0.f, 0.f};
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmcnt<0>();
    ++sp;
    cut = q_x + 2 * int(int64_t(full) * (sp + 1 - tails) / splits);
  };

  issue<C>(xa + at(0), xb + at(0), round_bytes, seg, lds0);
  issue<C>(xa + at(1), xb + at(1), round_bytes, seg, lds1);
  issue<C>(xa + at(2), xb + at(2), round_bytes, seg, lds2);
  int q = 0;
  for (; q + 4 <= nb; q += 4) {
    step(q + 3, lds0, lds3);
    step(q + 4, lds1, lds0);
    range_end(q + 2);
    step(q + 5, lds2, lds1);
    step(q + 6, lds3, lds2);
    range_end(q + 4);
  }
  if (q < nb) {
    step(q + 3, lds0, lds3);
    step(q + 4, lds1, lds0);
  }
  wait_vmcnt<0>();
  __syncthreads();
  if (FUSED && sp > 0) {
#pragma unroll
    for (int mi = 0; mi < C::kMB; ++mi) {
      const f4* q4 = sums + mi * C::kNB * 64 * WAVES;
#pragma unroll
      for (int ni = 0; ni < C::kNB; ++ni) acc[mi][ni] = q4[ni * 64 * WAVES + threadIdx.x] + acc[mi][ni];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int slot = rest ? 1 : sp + (sp > 0 ? tails : 0);
  float* P = FUSED ? H : part + size_t(slot) * size_t(d) * size_t(d);
  const int wm = wave / C::WGN, wn = wave % C::WGN;
#pragma unroll
  for (int mi = 0; mi < C::kMB; ++mi) {
    const int64_t i0 = int64_t(ti) * kBlock + (wm * C::kMB + mi) * 16 + 4 * (lane >> 4);
    const int64_t j0 = int64_t(tj) * kBlock + wn * C::kNB * 16 + (lane & 15);
    if (FUSED && accumulate) {  // 32 loads in flight before the first store
      float h[C::kNB][4];
#pragma unroll
      for (int ni = 0; ni < C::kNB; ++ni)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          h[ni][e] = i0 + e >= j0 + 16 * ni ? P[(i0 + e) * d + j0 + 16 * ni] : 0.f;
#pragma unroll
      for (int ni = 0; ni < C::kNB; ++ni)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mi][ni][e] = h[ni][e] + acc[mi][ni][e];
    }
#pragma unroll
    for (int ni = 0; ni < C::kNB; ++ni) {
      const int64_t jj = j0 + 16 * ni;
      const f4 v = acc[mi][ni];
      if (!FUSED || ti != tj) {
#pragma unroll
        for (int e = 0; e < 4; ++e) P[(i0 + e) * d + jj] = v[e];
        // The mirror entries of a lane's four rows are consecutive.
        if (FUSED) *reinterpret_cast<float4*>(P + jj * d + i0) = make_float4(v[0], v[1], v[2], v[3]);
      } else {  // the diagonal tile's lower triangle and its mirror
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i0 + e >= jj) {
            P[(i0 + e) * d + jj] = v[e];
            P[jj * d + i0 + e] = v[e];
          }
      }
    }
  }
}

// Copies `rows` (< 64) token rows starting at t0 into a zero-padded 64-row
// buffer so that the direct path never loads past the end of X.
__global__ void __launch_bounds__(kThreads) k_tail_rows(const uint16_t* X, int64_t d, int64_t t0,
                                                        int rows, uint16_t* out) {
  const int64_t total = int64_t(dt::kRows) * d;
  for (int64_t e = int64_t(blockIdx.x) * kThreads + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * kThreads) {
    const int64_t r = e / d;
    out[e] = r < rows ? X[(t0 + r) * d + (e - r * d)] : uint16_t(0);
  }
}

constexpr int kDirectWaves = 8;  // the layout of k_syrk_direct that the library launches

struct DirectPlan {
  int64_t tiles;
  int full_stages, tail_rows;
  int splits;  // of the whole stages
  bool spread, fused;
  size_t part_elems;
};

// Grid of k_syrk_direct over `tiles` tiles and `splits` splits: every unit, or
// 8 times the largest XCD share (ceil(tiles / 8) tiles, every split).
unsigned direct_grid(int64_t tiles, int splits, bool spread) {
  return unsigned((spread ? tiles : 8 * ceil_div(tiles, int64_t(8))) * splits);
}

bool direct_ok(int64_t d, int dtype) {
  return dtype == OPTIMA_DTYPE_BF16 && d % dt::kBlock == 0;
}

DirectPlan direct_plan(int64_t n_tok, int64_t d) {
  DirectPlan p{};
  const int64_t nt = d / dt::kBlock;
  p.tiles = nt * (nt + 1) / 2;
  p.full_stages = int(n_tok / dt::kRows);
  p.tail_rows = int(n_tok % dt::kRows);
  const int stages = std::max(1, p.full_stages);
  // Eighths of the tiles per XCD, unless they would leave more than a seventh
  // of the chip idle (1, 3, 6 or 10 tiles: d up to 1024).
  p.spread = 7 * 8 * ceil_div(p.tiles, int64_t(8)) > 8 * p.tiles;
  // Splits along the tokens: the rounds of workgroups per CU relative to the
  // work, 1% a split for starts and ends, at most 4 GiB of partials. This is a
  // lower bound for precision too: each split is a chain of fp32 sums of its
  // own, and a 2048-token sequence at d = 4096 in one chain instead of 11 had a
  // relative error of 1.5e-7 against 64 bits instead of 3.8e-8.
  const int64_t share = ceil_div(p.tiles, int64_t(8));
  const auto affordable = [d](int S) {
    return S == 1 || double(S) * double(d) * double(d) * 4.0 <= double(int64_t(1) << 32);
  };
  const int max_s = std::min(dt::kMaxSplits, stages);
  // More than that only where tiles spread over all CUs gain from it, and from
  // 32 stages a split on: d = 256 with 32768 tokens in 64 splits instead of 32
  // gained nothing and was off by 1.17e-7 instead of 1.06e-7; d = 1024 in 25
  // instead of 16 took 64 us instead of 72, 1.08e-7 instead of 1.15e-7. The
  // rounds relative to the work (1.6 us a 64-token stage), and for each split
  // the larger of 1% of a full chip's work and the partial sums' bytes, written
  // and read at 5.2 TB/s. With rounds(S) / S against a price of a split that grows
  // no faster than the work, a split that pays off pays off for more tokens too.
  const double tri_bytes = double(p.tiles) * dt::kBlock * dt::kBlock * 4.0;
  const int64_t units = p.spread ? p.tiles : 8 * share;  // a split
  const double stage_us = double(stages) * 1.6;
  const double split_us =
      std::max(0.01 * double(units) / dt::kCus * stage_us, tri_bytes * 2.0 / 5.2e6);
  struct Splits {
    int least, best;
    double best_us;
  };
  const auto splits_from = [&](int first) {  // at least `first`
    Splits s{first, first, 1e30};
    double least_cost = 1e30;
    for (int S = first; S <= max_s && affordable(S); ++S) {
      const double c = double(ceil_div(share * S, int64_t(dt::kCus / 8))) / S * (1.0 + 0.01 * S);
      if (c < least_cost - 1e-12) {
        s.least = S;
        least_cost = c;
      }
    }
    const int most = stages >= 32 * s.least ? max_s : s.least;
    for (int S = s.least; S <= most && affordable(S); ++S) {
      const double rounds = double(ceil_div(units * S, int64_t(dt::kCus)));
      const double c = rounds / S * stage_us + S * split_us + 5.0;
      if (c < s.best_us * (1.0 - 1e-12)) {
        s.best = S;
        s.best_us = c;
      }
    }
    return s;
  };
  // A range with last rows takes two splits at least: the widths that fill the chip
  // with one (5632, 7936 and others) are then off by 1.6e-7 of fp64 instead of
  // 2.5e-7 at 2000 tokens, which take 118 us instead of 104. Whole stages keep their
  // one chain: 2048 tokens 85 us.
  const int tails = p.full_stages > 0 && p.tail_rows > 0;
  const Splits two = splits_from(max_s > 1 && affordable(2) ? 2 : 1);
  const Splits plan = tails ? two : splits_from(1);
  p.splits = plan.best;
  // FUSED: every tile's ranges in one workgroup, kRangeUs between two of them
  // and kEndUs for the stores to H. Short ranges of many tiles, where the
  // partial sums outweigh the idle CUs: d = 4096 with 512 tokens 83 us instead
  // of 105, 2048 tokens 145 instead of 206.
  constexpr double kRangeUs = 8.0, kEndUs = 13.0;
  const double rounds = double(ceil_div(8 * share, int64_t(dt::kCus)));
  const double fused_cost =
      rounds * (double(stages + tails) * 1.6 + (plan.least - 1 + tails) * kRangeUs + kEndUs);
  const double split_cost = plan.best_us + tails * (tri_bytes * 2.0 / 5.2e6 + 3.0);
  p.fused = p.tiles >= 32 && fused_cost < 0.9 * split_cost;
  // One [d][d] partial per split and one for the last rows, which are no stage:
  // a chain of sums of their own, as a longer one would be less precise (3000
  // tokens of d = 3072 off by 1.54e-7 instead of 1.51e-7). The running sums of
  // FUSED (d (d + 256) / 2 entries) fit one partial. The size stays that of the
  // split plan with last rows, which never takes fewer splits for more stages, from
  // the first token beyond a stage on: a workspace for more tokens always holds
  // fewer.
  p.part_elems = size_t(std::max(two.best, p.splits) + (n_tok > dt::kRows)) * size_t(d) * size_t(d);
  if (p.fused) p.splits = plan.least;
  return p;
}

// Sums the split partials (pitch dp) into H (pitch d), both triangles.
optima_status reduce_partials(const float* part, int splits, int64_t dp, int64_t d, float* H,
                              int accumulate, hipStream_t s) {
  const int64_t B = ceil_div(d, 64);
  const dim3 grid(unsigned(B * (B + 1) / 2));
  if (d % 4 == 0)
    hipLaunchKernelGGL(k_hess_reduce4, grid, dim3(kThreads), 0, s, part, splits, dp, d, H,
                       accumulate);
  else
    hipLaunchKernelGGL(k_hess_reduce, grid, dim3(kThreads), 0, s, part, splits, dp, d, H,
                       accumulate);
  OPTIMA_LAUNCH_CHECK();
  return OPTIMA_OK;
}

}  // namespace

size_t hessian_workspace_bytes(int64_t n_tok, int64_t d, int dtype) {
  Carver c(nullptr);
  if (direct_ok(d, dtype)) {
    const DirectPlan p = direct_plan(n_tok, d);
    c.take<float>(p.part_elems);
    c.take<uint16_t>(size_t(dt::kRows) * size_t(d));
    return c.bytes();
  }
  const HessPlan p = plan(n_tok, d, dtype);
  c.take<char>(p.xt_elems * p.esz);
  c.take<float>(p.part_elems);
  return c.bytes();
}

optima_status hessian_accumulate(const void* X, int dtype, int64_t n_tok, int64_t d, float* H,
                                 int accumulate, void* ws, hipStream_t s) {
  if (n_tok == 0) {
    if (!accumulate) OPTIMA_HIP_TRY(hipMemsetAsync(H, 0, size_t(d) * size_t(d) * sizeof(float), s));
    return OPTIMA_OK;
  }
  if (direct_ok(d, dtype) && aligned16(X)) {
    const DirectPlan p = direct_plan(n_tok, d);
    Carver c(ws);
    float* part = c.take<float>(p.part_elems);
    uint16_t* tail = c.take<uint16_t>(size_t(dt::kRows) * size_t(d));
    const uint16_t* Xb = static_cast<const uint16_t*>(X);
    if (p.tail_rows > 0) {
      hipLaunchKernelGGL(k_tail_rows, dim3(256), dim3(kThreads), 0, s, Xb, d,
                         int64_t(p.full_stages) * dt::kRows, p.tail_rows, tail);
      OPTIMA_LAUNCH_CHECK();
    }
    const uint16_t* rest = p.full_stages > 0 && p.tail_rows > 0 ? tail : nullptr;
    if (p.full_stages == 0) Xb = tail;  // the padded copy is the only stage
    const int full = std::max(1, p.full_stages), splits = p.splits + (rest != nullptr);
    const dim3 threads(64 * kDirectWaves);
    if (p.fused)
      hipLaunchKernelGGL((k_syrk_direct<kDirectWaves, true>), dim3(direct_grid(p.tiles, 1, p.spread)),
                         threads, 0, s, Xb, rest, d, full, p.splits, int(p.spread), part, H,
                         accumulate);
    else
      hipLaunchKernelGGL((k_syrk_direct<kDirectWaves, false>),
                         dim3(direct_grid(p.tiles, splits, p.spread)), threads, 0, s, Xb, rest, d,
                         full, p.splits, int(p.spread), part, H, 0);
    OPTIMA_LAUNCH_CHECK();
    return p.fused ? OPTIMA_OK : reduce_partials(part, splits, d, d, H, accumulate, s);
  }
  const HessPlan p = plan(n_tok, d, dtype);
  Carver c(ws);
  char* XT = c.take<char>(p.xt_elems * p.esz);
  float* part = c.take<float>(p.part_elems);
  int first = 1;
  for (int64_t t0 = 0; t0 < n_tok; t0 += p.slab) {
    const int64_t rows = std::min<int64_t>(p.slab, n_tok - t0);
    const int stages = int(ceil_div(rows, p.kse));
    const int64_t cols = int64_t(stages) * p.kse;
    const dim3 tg(unsigned(ceil_div(cols, 64)), unsigned(ceil_div(p.dp, 64)));
    if (dtype == OPTIMA_DTYPE_BF16) {
      hipLaunchKernelGGL(k_transpose<uint16_t>, tg, dim3(kThreads), 0, s,
                         static_cast<const uint16_t*>(X), d, t0, rows, p.slab, p.dp,
                         reinterpret_cast<uint16_t*>(XT));
    } else {
      hipLaunchKernelGGL(k_transpose<float>, tg, dim3(kThreads), 0, s,
                         static_cast<const float*>(X), d, t0, rows, p.slab, p.dp,
                         reinterpret_cast<float*>(XT));
    }
    OPTIMA_LAUNCH_CHECK();
    const dim3 sg(unsigned(p.tiles * p.splits));
    const int64_t pitch = p.slab * p.esz;
    if (dtype == OPTIMA_DTYPE_BF16) {
      hipLaunchKernelGGL(k_syrk<Bf16Tag>, sg, dim3(kThreads), 0, s, XT, pitch, stages, p.splits,
                         p.dp, part, first);
    } else {
      hipLaunchKernelGGL(k_syrk<float>, sg, dim3(kThreads), 0, s, XT, pitch, stages, p.splits,
                         p.dp, part, first);
    }
    OPTIMA_LAUNCH_CHECK();
    first = 0;
  }
  return reduce_partials(part, p.splits, p.dp, d, H, accumulate, s);
}

optima_status hessian_jacobi(float* H, int64_t d, float* D, hipStream_t s) {
  hipLaunchKernelGGL(k_jacobi_d, dim3(unsigned(ceil_div(d, kThreads))), dim3(kThreads), 0, s, H, d,
                     D);
  OPTIMA_LAUNCH_CHECK();
  const int64_t blocks = std::min<int64_t>(8192, ceil_div(d * d, kThreads));
  hipLaunchKernelGGL(k_jacobi_scale, dim3(unsigned(blocks)), dim3(kThreads), 0, s, H, d, D);
  OPTIMA_LAUNCH_CHECK();
  return OPTIMA_OK;
}

optima_status hessian_damp(float* H, int64_t d, float rel, float* lambda_out, hipStream_t s) {
  hipLaunchKernelGGL(k_damp, dim3(1), dim3(1024), 0, s, H, d, rel, lambda_out);
  OPTIMA_LAUNCH_CHECK();
  return OPTIMA_OK;
}

}  // namespace optima
