// MFMA main loop of a 256x128 output tile of C = A B^T with A 2:4-sparse, on
// v_smfmac_f32_16x16x64_bf16.
//
// When every group of 4 consecutive K values of every A row has at most 2
// nonzeros (a 2:4 pruning mask applied to the multiplied vectors), A is kept
// compressed: per group 2 stored values, the entries at 2 positions p0 < p1
// that cover the group's nonzeros (padded with the lowest free positions),
// and per stored value its 2-bit position. One sparse MFMA multiplies a
// 16 x 64 block of A (16 x 32 stored values) by a dense 64 x 16 block of B,
// in the time of a dense 16 x 16 x 32 one, so it skips the products with
// the zeros.
//
// Operand layout of the instruction (checked on gfx950 against a reference
// product for every lane and value slot): lane l supplies A row l % 16 and
// the 8 stored values of logical K [16 g, 16 g + 16), g = l / 16, two per
// group of 4 in group order; bits 2 i..2 i + 1 of its 16-bit index give the
// position of stored value i within its group. Lane l supplies B column
// l % 16 at K [8 g, 8 g + 8) (values 0-7) and [32 + 8 g, 32 + 8 g + 8)
// (values 8-15). The result has the layout of the dense 16 x 16 MFMA.
//
// Storage of A: per row and 64-column block of K, 128 bytes: the 32 stored
// hi values (64 B), then the 32 stored lo values; lane group g's 16 bytes
// sit at byte 16 g of each plane. Indices: per row and block four 16-bit
// words (8 bytes), word g for lane group g; the tile reads them stage-major
// (one stage's words of consecutive tile rows are contiguous): with 8 bytes per
// row in a row-major array each stage's 2 KiB would touch 256 cache lines, as
// many as the A rows. B: split planes, 256 bytes a row and stage.
//
// Work split: 8 waves, one workgroup per CU. The operand loads from L2, not the
// MFMAs, bound these products, so the tile is the largest whose double-buffered
// stages fit the LDS: two half tiles of 128 A rows (16 KiB each), the B tile
// (32 KiB) and the index words (2 KiB). Wave (wm, wn) of a 2 x 4 grid owns
// 64 x 32 outputs of each A half, and a stage is two phases in the manner of
// gemm256.h (memory part and MFMA part, waves 4-7 one part behind):
//   1: read A0, B, indices   A0 B   fetch A1 of the next stage
//   2: read A1               A1 B   fetch A0, B, indices of the stage after it
// Each piece is fetched again as soon as both groups have read it, and each part
// waits for the loads of the phase after its own (all but the newest nine of
// the wave), so that 64 to 80 KiB stay in flight throughout. Waiting once per
// stage for all of it, with one barrier between whole stages, took (us an
// iteration, then this loop): d = 8192, 4096 columns 947, 828; d = 14336, 1024
// columns 781, 654; d = 4096, 4096 columns 253, 231 (596 TFLOP/s counted dense).
// Launches with few stages per workgroup gain nothing or lose up to 1 us (d =
// 2048, 128 columns: 18.6, 19.4; gemm_sparse_short). All eight waves in step: 5 to
// 10 % slower.
#pragma once

#include "gemm128.h"

namespace optima {

struct SpTile {
  static constexpr int BM = 256, BN = 128, kWaves = 8, kThreads = 512;
  static constexpr int kKPerStage = 64;
  static constexpr int kARowBytes = 128;  // stored A bytes per row and stage
  static constexpr int kBRowBytes = 256;  // B bytes per row and stage (both planes)
  static constexpr int kABytes = 128 * kARowBytes, kBBytes = BN * kBRowBytes, kIdxBytes = BM * 8;
  static constexpr int kLoadsB = kBBytes / 1024 / kWaves;
  // Loads a wave issues per stage beside A1's: A0, B and the indices.
  static constexpr int kInFlight = 2 * Tile256::kHalfLoads + kLoadsB + 1;
};

// Source addresses of this thread's loads at the first stage: load i of A half h
// fetches tile row 128 h + t256_load_row(i), byte t256_seg_bytes(i) of its
// stage; load i of B tile row sp_b_row(i), byte sp_b_seg_bytes(i); ai its 4
// bytes of index words.
struct SpOperands {
  const char* a[2][Tile256::kHalfLoads];
  const char* b[SpTile::kLoadsB];
  const char* ai;
  int64_t ai_stage;  // bytes from one stage's index words to the next
};

// B rows take 256 bytes (16 segments, segment g at physical g ^ (r % 16));
// index row r takes 8 bytes, 2 lanes per row.
__device__ inline int sp_b_row(int i) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (i * SpTile::kWaves + wave) * 4 + (lane >> 4);
}
__device__ inline int sp_b_seg_bytes(int i) {
  return (int(threadIdx.x & 15) ^ (sp_b_row(i) & 15)) * 16;
}
__device__ inline int sp_idx_row() { return (threadIdx.x >> 6) * 32 + (threadIdx.x & 63) / 2; }
__device__ inline int sp_idx_bytes() { return (threadIdx.x & 1) * 4; }

__device__ inline bf16x16 sp_b_pair(bf16x8 k0, bf16x8 k1) {
  return __builtin_shufflevector(k0, k1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
}

template <bool RANGES>
struct SpAcc {
  f4 q[2][4][2];                  // [A half][16-row block][16-column block]
  f4 sum[RANGES ? 2 : 0][4][2];  // of the ranges that have ended
};

namespace sp {

__device__ inline void fetch_b(const SpOperands& src, int64_t s, char* b, char* ix) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < SpTile::kLoadsB; ++i)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src.b[i] + s * SpTile::kBRowBytes),
        (__attribute__((address_space(3))) void*)(b + (i * SpTile::kWaves + wave) * 1024), 16, 0, 0);
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)(src.ai + s * src.ai_stage),
      (__attribute__((address_space(3))) void*)(ix + wave * 256), 4, 0, 0);
}

// Fragments of this wave's 32 B rows: [block][plane], K [0, 32) and [32, 64).
__device__ inline void read_b(bf16x16 (&f)[2][2], const char* b) {
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) & 3, g = lane >> 4;
  const int r = wn * 32 + (lane & 15), sw = r & 15;
  const char* p = b + r * SpTile::kBRowBytes;
  auto at = [&](int n, int seg) {
    return *reinterpret_cast<const bf16x8*>(p + n * 16 * SpTile::kBRowBytes + ((seg ^ sw) * 16));
  };
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    f[n][0] = sp_b_pair(at(n, g), at(n, 8 + g));
    f[n][1] = sp_b_pair(at(n, 4 + g), at(n, 12 + g));
  }
}

__device__ inline void read_idx(int (&x)[4], const char* ix, int r0) {
  const int lane = threadIdx.x & 63;
  const char* p = ix + (r0 + (lane & 15)) * 8 + 2 * (lane >> 4);
#pragma unroll
  for (int m = 0; m < 4; ++m) x[m] = *reinterpret_cast<const uint16_t*>(p + m * 16 * 8);
}

__device__ inline void half(f4 (&c)[4][2], const bf16x8 (&a)[4][2], const bf16x16 (&b)[2][2],
                            const int (&x)[4]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {  // hi hi, hi lo, lo hi
    const int pa = p >> 1, pb = p & 1;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
        c[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a[mi][pa], b[ni][pb], c[mi][ni], x[mi],
                                                              0, 0);
  }
}

// After a stage: if its range ends, the range's sum joins those before it.
template <bool RANGES>
__device__ inline void end_range(SpAcc<RANGES>& acc, SumRanges& ranges) {
  if (!ranges.step()) return;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    f4& q = acc.q[i >> 3][(i >> 1) & 3][i & 1];
    acc.sum[i >> 3][(i >> 1) & 3][i & 1] += q;
    q = f4{0.f, 0.f, 0.f, 0.f};
  }
}

template <bool RANGES>
__device__ inline void add_ranges(SpAcc<RANGES>& acc) {
  if constexpr (RANGES)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      f4& q = acc.q[i >> 3][(i >> 1) & 3][i & 1];
      q = acc.sum[i >> 3][(i >> 1) & 3][i & 1] + q;
    }
}

// One stage from buffers a0, a1, b, ix; na1 is the other A1 buffer, s1 and s2
// the next two stages.
template <bool RANGES>
__device__ inline void stage(SpAcc<RANGES>& acc, const SpOperands& src, SumRanges& ranges,
                             int64_t s1, int64_t s2, char* a0, char* a1, char* b, char* ix,
                             char* na1) {
  constexpr int kLeave = SpTile::kInFlight;
  const int wm = threadIdx.x >> 8;
  bf16x8 fa[4][2];
  bf16x16 fb[2][2];
  int x0[4], x1[4];
  t256::read<4>(fa, a0, wm * 64);
  read_b(fb, b);
  read_idx(x0, ix, wm * 64);
  read_idx(x1, ix, 128 + wm * 64);
  t256::fetch(src.a[1], s1 * SpTile::kARowBytes, na1);
  t256::end_memory<kLeave>();
  half(acc.q[0], fa, fb, x0);
  t256::barrier();
  t256::read<4>(fa, a1, wm * 64);
  t256::fetch(src.a[0], s2 * SpTile::kARowBytes, a0);
  fetch_b(src, s2, b, ix);
  t256::end_memory<kLeave>();
  half(acc.q[1], fa, fb, x1);
  if constexpr (RANGES) end_range(acc, ranges);
  t256::barrier();
}

}  // namespace sp

// n stages (n >= 0) of the sparse product. The LDS arguments are distinct
// __shared__ arrays of SpTile::kABytes, kBBytes and kIdxBytes; fetches past the
// last stage repeat it, into buffers that nobody reads again. (Peeling the last
// two stages without them cost the loop 2 % and gained nothing on short
// contractions.) `aside` runs once the first fetches are out.
template <bool RANGES, typename Aside>
__device__ inline void gemm_sparse_mainloop(SpAcc<RANGES>& acc, const SpOperands& src,
                                            SumShape shape, int n, char* a00,
                                            char* a01, char* b0, char* ix0, char* a10, char* a11,
                                            char* b1, char* ix1, Aside aside) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    acc.q[i >> 3][(i >> 1) & 3][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (RANGES) acc.sum[i >> 3][(i >> 1) & 3][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
  }
  if (n <= 0) return;
  auto at = [n](int s) { return int64_t(s < n ? s : n - 1); };
  t256::fetch(src.a[0], 0, a00);
  sp::fetch_b(src, 0, b0, ix0);
  t256::fetch(src.a[1], 0, a01);
  t256::fetch(src.a[0], at(1) * SpTile::kARowBytes, a10);
  sp::fetch_b(src, at(1), b1, ix1);
  aside();
  SumRanges ranges(shape);
  t256::end_memory<SpTile::kInFlight>();
  const bool behind = threadIdx.x >= 256;  // waves 4-7
  if (behind) t256::barrier();
  int s = 0;
  for (; s + 1 < n; s += 2) {
    sp::stage(acc, src, ranges, at(s + 1), at(s + 2), a00, a01, b0, ix0, a11);
    sp::stage(acc, src, ranges, at(s + 2), at(s + 3), a10, a11, b1, ix1, a01);
  }
  if (s < n) sp::stage(acc, src, ranges, at(s + 1), at(s + 2), a00, a01, b0, ix0, a11);
  if (!behind) t256::barrier();
  sp::add_ranges(acc);
  // No load may still be writing LDS when the workgroup moves on.
  wait_vmcnt<0>();
  __syncthreads();
}

// The same with all eight waves in step, for few stages: whole stages with one
// barrier each, the first two fetched at once, none fetched twice. Without ranges
// both halves of A have registers, so that a stage's LDS reads all go out before
// its first MFMA. d = 512 with 64 columns (a stage a workgroup) 11.0 us an
// iteration, 11.5 by the loop above.
template <bool RANGES, typename Aside>
__device__ inline void gemm_sparse_short(SpAcc<RANGES>& acc, const SpOperands& src, SumShape shape,
                                         int n, char* a00, char* a01, char* b0, char* ix0,
                                         char* a10, char* a11, char* b1, char* ix1, Aside aside) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    acc.q[i >> 3][(i >> 1) & 3][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (RANGES) acc.sum[i >> 3][(i >> 1) & 3][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
  }
  if (n <= 0) return;
  constexpr int kStage = SpTile::kInFlight;  // a wave's loads
  SumRanges ranges(SumShape{0, 0, 0});
  const int wm = threadIdx.x >> 8;
  auto fetch = [&](int s, char* a0, char* a1, char* b, char* ix) {
    t256::fetch(src.a[0], int64_t(s) * SpTile::kARowBytes, a0);
    sp::fetch_b(src, s, b, ix);
    t256::fetch(src.a[1], int64_t(s) * SpTile::kARowBytes, a1);
  };
  // Waits for stage s; every wave has then read the stage before it.
  auto landed = [&](int s) {
    if (s == 0 && n > 1)
      t256::end_memory<kStage>();
    else
      t256::end_memory<0>();
  };
  auto compute = [&](const char* a0, const char* a1, const char* b, const char* ix) {
    bf16x8 fa[4][2], fa1[4][2];
    bf16x16 fb[2][2];
    int x0[4], x1[4];
    t256::read<4>(fa, a0, wm * 64);
    sp::read_b(fb, b);
    sp::read_idx(x0, ix, wm * 64);
    sp::read_idx(x1, ix, 128 + wm * 64);
    if (!RANGES) t256::read<4>(fa1, a1, wm * 64);  // registers for both halves
    sp::half(acc.q[0], fa, fb, x0);
    if (RANGES) t256::read<4>(fa1, a1, wm * 64);
    sp::half(acc.q[1], fa1, fb, x1);
    if constexpr (RANGES) sp::end_range(acc, ranges);
  };
  fetch(0, a00, a01, b0, ix0);
  if (n > 1) fetch(1, a10, a11, b1, ix1);
  aside();
  if (RANGES) ranges = SumRanges(shape);
  for (int s = 0; s < n; s += 2) {
    landed(s);
    if (s > 0 && s + 1 < n) fetch(s + 1, a10, a11, b1, ix1);
    compute(a00, a01, b0, ix0);
    if (s + 1 == n) break;
    landed(s + 1);
    if (s + 2 < n) fetch(s + 2, a00, a01, b0, ix0);
    compute(a10, a11, b1, ix1);
  }
  sp::add_ranges(acc);
  __syncthreads();
}

// Epilogue staging of the 256 x 128 accumulators: 512 bytes a row, 32 rows in
// each 16 KiB (the four A buffers, then the halves of the B buffers); 16-byte
// column chunk c of row r at physical chunk c ^ (r & 31).
__device__ inline char* sp_stage_row(char* a00, char* a01, char* a10, char* a11, char* b0, char* b1,
                                     int r) {
  const int h = r >> 5;
  char* lo = h & 2 ? (h & 1 ? a11 : a10) : (h & 1 ? a01 : a00);
  char* hi = (h & 2 ? b1 : b0) + (h & 1) * 16384;
  return (h & 4 ? hi : lo) + (r & 31) * 512;
}

}  // namespace optima
