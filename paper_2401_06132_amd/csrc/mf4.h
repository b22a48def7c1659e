// Small operators on the matrix cores, one column per lane (gfx950).
//
// v_mfma_f32_4x4x1_16b computes, for each of 16 blocks of four lanes,
// D[i][j] = C[i][j] + A[i] B[j]: lane l = 4 b + j supplies A[l mod 4] and
// B[j] of its block b and holds the four values D[0..3][j].  With the block
// broadcast (cbsz = 4: all 16 blocks take the A of block abid; cbsz = 3: the
// eight blocks of each half wave take the A of their half's block abid) the
// lane's four accumulators gain op[0..3] times its own value: four rows of a
// wave-uniform operator applied to 64 columns, one per lane, with nothing
// exchanged between lanes.  One VGPR holds 16 such operator columns
// ("chunks": four rows at one k), so an operator of R rows and K columns
// needs ceil(R/4) K / 16 registers and no scalar or LDS operand traffic.
// The products are fused multiply-adds in single precision in the order of
// k, the same bits as a loop of fmaf (checked over the lane layout, the
// broadcasts and random operands).  Measured on the MI355X: 8.9 cycles for
// 4 x 64 multiply-adds against 4 x 4.8 for vector FMAs.  The two do not
// overlap (a SIMD with one wave of each kind takes the sum of their times:
// single-precision matrix and vector instructions share the ALUs), so the gain
// is this rate and the operands that no longer come through LDS.
//
// The instruction ignores EXEC: every call below sits in wave-uniform
// control flow, with out-of-range items clamped to a valid one and dropped
// at the store.
#pragma once

#include <hip/hip_runtime.h>

namespace fr {

typedef float mf4v __attribute__((ext_vector_type(4)));

// never defined: a call that is left after constant folding ends the compilation
__device__ __attribute__((error("mf4: the chunk must be a constant below 16 (CBSZ = 3: 8)"))) void mf4_bad_chunk();

// one chunk: c + (chunk abid of a) * b; abid must fold to a constant below 16
// (CBSZ = 3: 8), any other does not compile
template <int CBSZ = 4>
__device__ __forceinline__ mf4v mf4(float a, float b, mf4v c, int abid) {
#define FR_MF4(i) \
  case i: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CBSZ, i, 0);
  switch (abid) {
    FR_MF4(0) FR_MF4(1) FR_MF4(2) FR_MF4(3) FR_MF4(4) FR_MF4(5) FR_MF4(6) FR_MF4(7)
  }
  if constexpr (CBSZ == 4) {
    switch (abid) { FR_MF4(8) FR_MF4(9) FR_MF4(10) FR_MF4(11) FR_MF4(12) FR_MF4(13) FR_MF4(14) FR_MF4(15) }
  }
#undef FR_MF4
  mf4_bad_chunk();
  return c;
}

// An operator of T row tiles (4 T rows) and K columns as chunks in the order
// c = k T + t; chunk c of the device table is at [c / 16][4 (c mod 16) + row].
template <int T, int K>
struct Mf4Op {
  static constexpr int NREG = (T * K + 15) / 16, FLOATS = NREG * 64;
  float a[NREG];
  __device__ __forceinline__ void load(const float* __restrict__ tab, int lane) {
#pragma unroll
    for (int i = 0; i < NREG; ++i) a[i] = tab[i * 64 + lane];
  }
  // acc[t] += rows of column k < K times x
  __device__ __forceinline__ void col(int k, float x, mf4v (&acc)[T]) const {
    if (k < 0 || k >= K) mf4_bad_chunk();
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = mf4(a[(k * T + t) / 16], x, acc[t], (k * T + t) % 16);
  }
};

// host: pack rows r < R of op(r, k) into dst (FLOATS zeroed entries)
template <int T, int K, typename F>
void mf4_pack(float* dst, int R, const F& op) {
  for (int i = 0; i < Mf4Op<T, K>::FLOATS; ++i) dst[i] = 0.0f;
  for (int k = 0; k < K; ++k)
    for (int t = 0; t < T; ++t)
      for (int r = 0; r < 4 && 4 * t + r < R; ++r) {
        const int c = k * T + t;
        dst[(c / 16) * 64 + 4 * (c % 16) + r] = float(op(4 * t + r, k));
      }
}

// a(lane) + a(lane ^ 32) in the lower half wave, b(lane) + b(lane ^ 32) in
// the upper one
__device__ __forceinline__ float half_sums(float a, float b) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const u2 s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s.x) + __uint_as_float(s.y);
}

}  // namespace fr
