// MFMA main loop of a 128x128 output tile of C = A B^T by 8 waves, one
// workgroup per CU, for products with too few outputs for the 256x256 tile of
// gemm256.h: the same two wave groups half a phase apart, on whole stages.
//
// Stages of 128 bytes a row (64 bf16 values, or 32 columns of split planes) go
// through a ring of four 32-KiB LDS buffers. Wave (wm, wn) of a 2 x 4 grid owns
// 64 x 32 outputs. A stage is a memory part (twelve 16-byte LDS reads a lane,
// the fetch of the stage three ahead) and an MFMA part, each ended by a barrier;
// waves 4-7 run one part behind waves 0-3, so that of the two waves of a SIMD
// one reads while the other multiplies. A buffer is fetched again one stage
// after it was read, by when both groups' reads have returned (each wave waits
// for them before the barrier that ends its memory part); and each wave waits in
// the memory part of stage s for its fetches of stage s + 1, which the group
// behind does in the part before the group ahead first reads them.
//
// Bound by the loads: 32 KiB a stage, 0.56 us on a full chip (15 TB/s out of the
// L2s), where the stage's MFMAs take 0.35. d = 4096 with 1024 columns (256 tiles
// of 128 stages): 80 us plus 12 us of fused update, against 111 us for the
// 4-wave tile split in two.
//
// What bounds the error of a sum is the number of MFMA additions to one chain. It
// is kept down in one of two ways. Without RANGES the small products of split planes
// have accumulators of their own, and a stage rounds the sum once instead of three
// times. With RANGES the workgroup ends the ranges of its sum (SumRanges) in
// registers, where they join a running sum by plain fp32 additions. d = 768 with
// 3072 columns, 8 CG iterations: W is off by 9.7e-7 of fp64 in one range, 9.1e-7 in
// five, which take 2.1 instead of 2.0 ms of 64 rAPDHG iterations. Both at once need
// more registers than there are: half as long again.
#pragma once

#include "gemm256.h"

namespace optima {

struct Ring128 {
  static constexpr int BM = 128, BN = 128, kWaves = 8, kThreads = 512;
  static constexpr int kSRB = 128;              // bytes per row and stage
  static constexpr int kBufBytes = 256 * kSRB;  // A rows, then B rows
  static constexpr int kLoads = 2;              // wave loads per stage of A, and of B
};

// Source addresses of this thread's loads at the first stage: load i of A or B
// fetches tile row t256_load_row(i), byte t256_seg_bytes(i) of its stage.
struct OperandsR128 {
  const char* a[Ring128::kLoads];
  const char* b[Ring128::kLoads];
};

template <bool RANGES>
struct AccR128 {
  f4 q[4][2];      // [16-row block][16-column block]
  f4 other[4][2];  // the ranges that have ended, or the hi lo and lo hi products
};
// Where the ranges of a sum end, as a workgroup meets them: `count` ranges of
// `stages` stages, range r ending before stage stages (r + 1) / count; the
// workgroup starts at stage s0. count 0: it has one range.
struct SumShape {
  int stages, count, s0;
};
struct SumRanges {
  int until;  // stages to the end of the present range
  int len, rem, count, part;

  // Divisions, for after the first loads. (32 bits: stages count stays below 2^31.)
  __device__ inline explicit SumRanges(const SumShape& s)
      : until(0x7fffffff), len(0), rem(0), count(s.count), part(0) {
    if (!count) return;
    const unsigned n = s.stages, c = count;
    unsigned r = s.s0 * c / n;
    while (n * r / c <= unsigned(s.s0)) ++r;
    len = n / c;
    rem = n % c;
    until = n * r / c - s.s0;
    part = n * r % c;
  }
  // A stage has been added; whether its range ends.
  __device__ inline bool step() {
    if (--until > 0) return false;
    part += rem;
    until = len + (part >= count);
    part -= part >= count ? count : 0;
    return true;
  }
};
__device__ inline int r128_row(int mi, int e) { return t256_row(0, mi, e); }
__device__ inline int r128_col(int ni) { return t256_col(0, ni); }

// LEFT: stages left, this one included (4: or more); the last three fetch
// nothing, and wait for what is in flight.
template <typename T, int LEFT, bool RANGES>
__device__ inline void r128_stage(AccR128<RANGES>& acc, const OperandsR128& src, SumRanges& ranges,
                                  int s, char* cur, char* nxt) {
  constexpr int kStage = 2 * Ring128::kLoads;
  const int wm = threadIdx.x >> 8, wn = (threadIdx.x >> 6) & 3;
  bf16x8 fa[4][2], fb[2][2];
  t256::read<4>(fa, cur, wm * 64);
  t256::read<2>(fb, cur + 128 * Ring128::kSRB, wn * 32);
  if constexpr (LEFT >= 4) {
    const int64_t off = int64_t(s + 3) * Ring128::kSRB;
    t256::fetch(src.a, off, nxt);
    t256::fetch(src.b, off, nxt + 128 * Ring128::kSRB);
  }
  t256::end_memory<LEFT >= 4 ? 2 * kStage : LEFT == 3 ? kStage : LEFT == 2 ? 0 : -1>();
  t256::quadrant<T>(acc.q, RANGES ? acc.q : acc.other, fa, fb);
  if (RANGES && LEFT > 1 && ranges.step()) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc.other[i >> 1][i & 1] += acc.q[i >> 1][i & 1];
      acc.q[i >> 1][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
    }
  }
  t256::barrier();
}

// The last three stages, from buffers c0, c1, c2.
template <typename T, bool RANGES>
__device__ inline void r128_last3(AccR128<RANGES>& acc, const OperandsR128& src, SumRanges& ranges,
                                  char* c0, char* c1, char* c2) {
  r128_stage<T, 3>(acc, src, ranges, 0, c0, nullptr);
  r128_stage<T, 2>(acc, src, ranges, 0, c1, nullptr);
  r128_stage<T, 1>(acc, src, ranges, 0, c2, nullptr);
}

// n stages (n >= 0) of a sum, with RANGES its ranges as `shape` has them. b0..b3 are
// distinct __shared__ arrays of Ring128::kBufBytes. `aside` runs once the first
// fetches are out.
template <typename T, bool RANGES, typename Aside>
__device__ inline void r128_mainloop(AccR128<RANGES>& acc, const OperandsR128& src, SumShape shape,
                                     int n, char* b0, char* b1, char* b2, char* b3, Aside aside) {
  constexpr int kStage = 2 * Ring128::kLoads;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    acc.q[i >> 1][i & 1] = acc.other[i >> 1][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
  if (n <= 0) return;
  auto fetch = [&](int s, char* buf) {
    t256::fetch(src.a, int64_t(s) * Ring128::kSRB, buf);
    t256::fetch(src.b, int64_t(s) * Ring128::kSRB, buf + 128 * Ring128::kSRB);
  };
  const bool behind = threadIdx.x >= 256;  // waves 4-7
  fetch(0, b0);
  if (n < 3) {
    aside();
    SumRanges ranges(shape);
    if (n == 2) {
      fetch(1, b1);
      t256::end_memory<kStage>();
    } else {
      t256::end_memory<0>();
    }
    if (behind) t256::barrier();
    if (n == 2) {
      r128_stage<T, 2>(acc, src, ranges, 0, b0, nullptr);
      r128_stage<T, 1>(acc, src, ranges, 0, b1, nullptr);
    } else {
      r128_stage<T, 1>(acc, src, ranges, 0, b0, nullptr);
    }
  } else {
    fetch(1, b1);
    fetch(2, b2);
    aside();
    SumRanges ranges(shape);
    t256::end_memory<2 * kStage>();
    if (behind) t256::barrier();
    int s = 0;
    for (; s + 7 <= n; s += 4) {
      r128_stage<T, 4>(acc, src, ranges, s, b0, b3);
      r128_stage<T, 4>(acc, src, ranges, s + 1, b1, b0);
      r128_stage<T, 4>(acc, src, ranges, s + 2, b2, b1);
      r128_stage<T, 4>(acc, src, ranges, s + 3, b3, b2);
    }
    // 3 to 6 stages are left.
    if (n - s == 3) {
      r128_last3<T>(acc, src, ranges, b0, b1, b2);
    } else if (n - s == 4) {
      r128_stage<T, 4>(acc, src, ranges, s, b0, b3);
      r128_last3<T>(acc, src, ranges, b1, b2, b3);
    } else if (n - s == 5) {
      r128_stage<T, 4>(acc, src, ranges, s, b0, b3);
      r128_stage<T, 4>(acc, src, ranges, s + 1, b1, b0);
      r128_last3<T>(acc, src, ranges, b2, b3, b0);
    } else {
      r128_stage<T, 4>(acc, src, ranges, s, b0, b3);
      r128_stage<T, 4>(acc, src, ranges, s + 1, b1, b0);
      r128_stage<T, 4>(acc, src, ranges, s + 2, b2, b1);
      r128_last3<T>(acc, src, ranges, b3, b0, b1);
    }
  }
  if (!behind) t256::barrier();
#pragma unroll
  for (int i = 0; i < 8; ++i)
    acc.q[i >> 1][i & 1] = acc.other[i >> 1][i & 1] + acc.q[i >> 1][i & 1];
  // No load may still be writing LDS when the workgroup moves on.
  wait_vmcnt<0>();
  __syncthreads();
}

// Epilogue staging of the tile through buffers b0 and b1: 512 bytes a row, rows
// 0-63 in b0; 16-byte column chunk c of row r at physical chunk c ^ (r & 31).
__device__ inline char* r128_stage_row(char* b0, char* b1, int r) {
  return (r < 64 ? b0 : b1) + (r & 63) * 512;
}

}  // namespace optima
