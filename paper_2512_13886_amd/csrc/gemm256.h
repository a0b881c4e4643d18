// MFMA main loop of a 256x256 output tile of C = A B^T (both operands row-major
// with the contraction contiguous, as in gemm_core.h) by 8 waves, one workgroup
// per CU.
//
// Stages of 128 bytes a row: 64 bf16 values, or 32 columns of split planes (64
// bytes of hi, 64 of lo). A stage is four half tiles of 128 rows, A0, A1, B0
// and B1, 16 KiB each, in LDS arrays of their own (two of each, 128 KiB). Wave
// (wm, wn) of a 2 x 4 grid owns 64 x 32 outputs of each of the four quadrants
// (A half, B half), and multiplies a stage in four phases, one quadrant each:
//   1: read A0, B0   A0 B0      fetch A1 of the next stage
//   2: read B1       A0 B1      fetch A0 of the stage after it
//   3: read A1       A1 B1      fetch B0 of the stage after it
//   4:               A1 B0      fetch B1 of the stage after it
// so every half tile is fetched again as soon as all waves have read it, and
// six to eight 1-KiB loads a wave stay in flight across each stage's end.
//
// A phase is a memory part (LDS reads, the fetch) and an MFMA part, each ended
// by a barrier, and waves 4-7 run one part behind waves 0-3. Waves w and w + 4
// share a SIMD, so in every interval one of them multiplies while the other
// reads. What makes it safe, with parts numbered along the barriers:
//   - a wave's LDS reads have returned before the barrier that ends its memory
//     part, and a half tile is refilled in a later part of either group;
//   - a wave waits for its fetches of the next stage (all but the newest three
//     half tiles) in the memory part of phase 4. The group behind does so in
//     the part before the one in which the group ahead first reads them.
//
// Bound by the MFMAs and, in phase 1, the LDS reads (24 KiB a wave and stage).
// bf16, 32768 x 4096 outputs: each further 4096 of the contraction takes 715 us
// (1.54 PFLOP/s; the 4-wave 128 x 128 loop runs at 0.96). Without the half-phase
// offset between the groups the whole product takes 10 % longer; raising the
// wave's priority around its MFMAs changes nothing.
#pragma once

#include "gemm_core.h"

namespace optima {

struct Tile256 {
  static constexpr int BM = 256, BN = 256, kWaves = 8, kThreads = 512;
  static constexpr int kSRB = 128;                  // bytes per row and stage
  static constexpr int kHalfBytes = 128 * kSRB;     // one half tile
  static constexpr int kHalfLoads = kHalfBytes / 1024 / kWaves;  // wave loads per half tile
};

// Source addresses of this thread's loads at the first stage: half tile h of A
// or B, load i, fetches tile row 128 h + t256_load_row(i), at byte
// t256_seg_bytes(i) of the row's stage. 16-byte aligned.
struct Operands256 {
  const char* a[2][Tile256::kHalfLoads];
  const char* b[2][Tile256::kHalfLoads];
};

__device__ inline int t256_load_row(int i) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (i * Tile256::kWaves + wave) * 8 + (lane >> 3);
}
// 16-byte segment g of row r sits at physical segment g ^ (r % 8).
__device__ inline int t256_seg_bytes(int i) {
  return (int(threadIdx.x & 7) ^ (t256_load_row(i) & 7)) * 16;
}

struct Acc256 {
  f4 q[2][2][4][2];  // [A half][B half][16-row block][16-column block]
};

// Row and column, within the tile, of element e of block (mi, ni) of quadrant
// (qa, qb) of this thread.
__device__ inline int t256_row(int qa, int mi, int e) {
  const int lane = threadIdx.x & 63, wm = threadIdx.x >> 8;
  return qa * 128 + wm * 64 + mi * 16 + 4 * (lane >> 4) + e;
}
__device__ inline int t256_col(int qb, int ni) {
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) & 3;
  return qb * 128 + wn * 32 + ni * 16 + (lane & 15);
}

namespace t256 {

__device__ inline void fetch(const char* const (&src)[Tile256::kHalfLoads], int64_t off, char* half) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < Tile256::kHalfLoads; ++i)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src[i] + off),
        (__attribute__((address_space(3))) void*)(half + (i * Tile256::kWaves + wave) * 1024), 16, 0,
        0);
}

// Fragments of NBLK 16-row blocks from row r0 of a half tile: segments g and
// 4 + g of the rows (the two 32-value K steps of bf16, or the hi and lo planes).
template <int NBLK>
__device__ inline void read(bf16x8 (&f)[NBLK][2], const char* half, int r0) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int r = r0 + (lane & 15);
  const char* p0 = half + r * Tile256::kSRB + ((g ^ (r & 7)) * 16);
  const char* p1 = half + r * Tile256::kSRB + (((4 + g) ^ (r & 7)) * 16);
#pragma unroll
  for (int m = 0; m < NBLK; ++m) {
    f[m][0] = *reinterpret_cast<const bf16x8*>(p0 + m * 16 * Tile256::kSRB);
    f[m][1] = *reinterpret_cast<const bf16x8*>(p1 + m * 16 * Tile256::kSRB);
  }
}

// The second and third products of split planes go to `cross`, which may be c.
template <typename T>
__device__ inline void quadrant(f4 (&c)[4][2], f4 (&cross)[4][2], const bf16x8 (&a)[4][2],
                                const bf16x8 (&b)[2][2]) {
  constexpr bool kSplit = std::is_same<T, Bf16x3Tag>::value;
#pragma unroll
  for (int p = 0; p < (kSplit ? 3 : 2); ++p) {
    // bf16: both K steps; split planes: hi hi, hi lo, lo hi.
    const int pa = kSplit ? p >> 1 : p, pb = kSplit ? p & 1 : p;
    f4 (&to)[4][2] = kSplit && p > 0 ? cross : c;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        to[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mi][pa], b[ni][pb], to[mi][ni], 0, 0, 0);
  }
}

__device__ inline void barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// End of a memory part: LDS reads back, and all but N loads landed (N < 0: no
// wait for loads).
template <int N>
__device__ inline void end_memory() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  if constexpr (N >= 0)
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x70);  // vmcnt(N) lgkmcnt(0)
  else
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  barrier();
}

// One stage from buffers a0, a1, b0, b1; na1 is the other A1 buffer.
template <typename T>
__device__ inline void stage(Acc256& acc, const Operands256& src, int64_t off1, int64_t off2,
                             char* a0, char* a1, char* b0, char* b1, char* na1) {
  const int wm = threadIdx.x >> 8, wn = (threadIdx.x >> 6) & 3;
  bf16x8 fa[4][2], fb0[2][2], fb1[2][2];
  read<4>(fa, a0, wm * 64);
  read<2>(fb0, b0, wn * 32);
  fetch(src.a[1], off1, na1);
  end_memory<-1>();
  quadrant<T>(acc.q[0][0], acc.q[0][0], fa, fb0);
  barrier();
  read<2>(fb1, b1, wn * 32);
  fetch(src.a[0], off2, a0);
  end_memory<-1>();
  quadrant<T>(acc.q[0][1], acc.q[0][1], fa, fb1);
  barrier();
  read<4>(fa, a1, wm * 64);
  fetch(src.b[0], off2, b0);
  end_memory<-1>();
  quadrant<T>(acc.q[1][1], acc.q[1][1], fa, fb1);
  barrier();
  fetch(src.b[1], off2, b1);
  end_memory<3 * Tile256::kHalfLoads>();
  quadrant<T>(acc.q[1][0], acc.q[1][0], fa, fb0);
  barrier();
}

}  // namespace t256

// n stages (n >= 0) of tile products. The LDS arguments are distinct
// __shared__ arrays of Tile256::kHalfBytes; fetches past the last stage repeat
// it, into buffers that nobody reads again. `aside` runs once the first fetches
// are out.
template <typename T, typename Aside>
__device__ inline void gemm256_mainloop(Acc256& acc, const Operands256& src, int n, char* a00,
                                        char* a01, char* b00, char* b01, char* a10, char* a11,
                                        char* b10, char* b11, Aside aside) {
#pragma unroll
  for (int i = 0; i < 32; ++i) acc.q[i >> 4][(i >> 3) & 1][(i >> 1) & 3][i & 1] = f4{0.f, 0.f, 0.f, 0.f};
  if (n <= 0) return;
  auto at = [n](int s) { return int64_t(s < n ? s : n - 1) * Tile256::kSRB; };
  t256::fetch(src.a[0], 0, a00);
  t256::fetch(src.b[0], 0, b00);
  t256::fetch(src.b[1], 0, b01);
  t256::fetch(src.a[1], 0, a01);
  t256::fetch(src.a[0], at(1), a10);
  t256::fetch(src.b[0], at(1), b10);
  t256::fetch(src.b[1], at(1), b11);
  aside();
  t256::end_memory<3 * Tile256::kHalfLoads>();
  const bool behind = threadIdx.x >= 256;  // waves 4-7
  if (behind) t256::barrier();
  int s = 0;
  for (; s + 1 < n; s += 2) {
    t256::stage<T>(acc, src, at(s + 1), at(s + 2), a00, a01, b00, b01, a11);
    t256::stage<T>(acc, src, at(s + 2), at(s + 3), a10, a11, b10, b11, a01);
  }
  if (s < n) t256::stage<T>(acc, src, at(s + 1), at(s + 2), a00, a01, b00, b01, a11);
  if (!behind) t256::barrier();
  // No load may still be writing LDS when the workgroup moves on.
  wait_vmcnt<0>();
  __syncthreads();
}

// Epilogue staging of 256 rows x 128 columns of fp32 through the eight buffers:
// 512 bytes a row, rows 32 h .. 32 h + 31 in buffer h; 16-byte column chunk c
// of row r at physical chunk c ^ (r & 31), free of bank conflicts for the
// MFMA-layout writes and the row-chunk reads.
__device__ inline char* t256_stage_row(char* l0, char* l1, char* l2, char* l3, char* l4, char* l5,
                                       char* l6, char* l7, int r) {
  const int h = r >> 5;
  char* lo = h & 2 ? (h & 1 ? l3 : l2) : (h & 1 ? l1 : l0);
  char* hi = h & 2 ? (h & 1 ? l7 : l6) : (h & 1 ? l5 : l4);
  return (h & 4 ? hi : lo) + (r & 31) * 512;
}

}  // namespace optima
