// Arithmetic that more than one kernel must give the same bits of: the RIA scores (Section 3, Eq. 1), written by one kernel
// and computed where they are needed by the pruning of a mask refresh, and the LoRA merge (Section 4.3, Eq. 10), with and
// without the sums of the scores.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace vnm {

// a / b rounded to nearest, from y = 1 / b rounded to nearest: q0 = a y is within 1.5 ulp, one correction
// makes q1 a faithful quotient, and for a faithful quotient the second one gives the correctly rounded result
// (Markstein's theorem).  It needs exact residuals, so nothing may overflow or underflow: a is 0 or k 2^-136 with an
// integer k < 2^41, b an integer-valued double up to 2^63, so quotients are at least 2^-199 and residuals, multiples of
// 2^-136 or of half an ulp of the quotient, above 2^-252.  (a comes from an fp32 conversion that keeps subnormals: fp32
// denormals must not be flushed in this file.)
// Five operations per element; the division by itself takes about fifteen, two of them per element
// (53 us on 4096 x 4096, of which the memory traffic needs a third).
__device__ __forceinline__ double sc_div(double a, double b, double y) {
  const double q0 = a * y;
  const double q1 = fma(fma(-b, q0, a), y, q0);
  return fma(fma(-b, q1, a), y, q1);
}

// The 15 magnitude bits of an fp16 pattern read as fp32 are the magnitude times 2^-112 (subnormals and the top exponent
// included): units of 2^-24 times 2^-136, a scale that the activation factor takes back exactly.
__device__ __forceinline__ double sc_scaled(unsigned h) { return (double)__uint_as_float((h & 0x7FFFu) << 13); }

// One correction instead of two, for b up to 2^48: the same bits.  a is a multiple of ulp(q), and so is b q0 (b is an
// integer); |a - b q0| < 1.5 b ulp(q) < 2^53 ulp(q), so the residual is exact and q1 is the rounding of a value that misses
// a / b by less than 1.5 ulp(q) 2^-53 (twice that where q0 and q lie in different binades).  And a / b keeps further away
// than that from every midpoint M 2^-k (M odd, ulp(q) = 2^(1-k)): a 2^k - M b, a nonzero integer in units of the last place
// of a (M would have to divide a 2^k and has 54 bits, a 11), is at least 1, so the distance is at least ulp(q) / (2 b),
// 2^-49 ulp(q).
constexpr double kScSmall = 0x1p48;
__device__ __forceinline__ double sc_div_small(double a, double b, double y) {
  const double q0 = a * y;
  return fma(fma(-b, q0, a), y, q0);
}

// One score: cd, cy the column's sum and its reciprocal, rd, ry the row's, ad = act * 2^136.  SMALL: both sums are at most
// kScSmall (weights that add up to 2^24).
template <bool SMALL = false>
__device__ __forceinline__ float sc_ria(unsigned h, double cd, double cy, double ad, double rd, double ry) {
  const double a = sc_scaled(h);
  const double sum = SMALL ? sc_div_small(a, cd, cy) + sc_div_small(a, rd, ry) : sc_div(a, cd, cy) + sc_div(a, rd, ry);
  return (float)(sum * ad);
}

// ---- LoRA merge of 8 rows x 8 columns: fp16(W + scale * B A), every product and sum rounded on its own (no contraction
// into fused multiply-adds), k ascending.  The pointers are those of the tile's first row and column; W and A are 16-byte
// aligned there.  CLAMP: rows beyond `last` repeat row `last`.
constexpr int kMergeRows = 8;   // rows per thread: A is fetched once per 8 rows instead of once per row

template <int K, bool CLAMP>
__device__ __forceinline__ void merge_steps(const float* B, int64_t ldb, const float* A, int64_t lda, int k, int last,
                                            float (&acc)[kMergeRows][8]) {
#pragma clang fp contract(off)
  float4 a0[K], a1[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    a0[u] = *(const float4*)(A + (int64_t)(k + u) * lda);
    a1[u] = *(const float4*)(A + (int64_t)(k + u) * lda + 4);
  }
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const float a[8] = {a0[u].x, a0[u].y, a0[u].z, a0[u].w, a1[u].x, a1[u].y, a1[u].z, a1[u].w};
#pragma unroll
    for (int v = 0; v < kMergeRows; ++v) {
      const float b = B[(int64_t)(CLAMP && v > last ? last : v) * ldb + k + u];
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float p = b * a[e]; acc[v][e] = acc[v][e] + p; }
    }
  }
}

template <bool CLAMP>
__device__ __forceinline__ void merge_load(const unsigned short* W, int64_t ldw, int last, uint4 (&w4)[kMergeRows]) {
#pragma unroll
  for (int v = 0; v < kMergeRows; ++v) w4[v] = *(const uint4*)(W + (int64_t)(CLAMP && v > last ? last : v) * ldw);
}

template <bool CLAMP>
__device__ __forceinline__ void merge_tile(const uint4 (&w4)[kMergeRows], const float* B, int64_t ldb, const float* A,
                                           int64_t lda, int r, float scale, int last, uint4 (&out)[kMergeRows]) {
#pragma clang fp contract(off)
  float acc[kMergeRows][8];
#pragma unroll
  for (int v = 0; v < kMergeRows; ++v)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[v][e] = 0.f;
  // four rows of A at a time are requested before the first use (one row per trip left a memory round trip exposed per k:
  // 28 us on 4096 x 4096 at r = 16)
  int k = 0;
  for (; k + 4 <= r; k += 4) merge_steps<4, CLAMP>(B, ldb, A, lda, k, last, acc);
  for (; k < r; ++k) merge_steps<1, CLAMP>(B, ldb, A, lda, k, last, acc);
#pragma unroll
  for (int v = 0; v < kMergeRows; ++v) {
    const unsigned d[4] = {w4[v].x, w4[v].y, w4[v].z, w4[v].w};
    unsigned m[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const unsigned short hb = (unsigned short)(d[e / 2] >> (16 * (e & 1)));
      _Float16 h;
      __builtin_memcpy(&h, &hb, 2);
      const float sp = scale * acc[v][e];
      const _Float16 res = (_Float16)(sp + (float)h);
      unsigned short rb;
      __builtin_memcpy(&rb, &res, 2);
      m[e / 2] = (e & 1) ? (m[e / 2] | ((unsigned)rb << 16)) : rb;
    }
    out[v] = make_uint4(m[0], m[1], m[2], m[3]);
  }
}

}  // namespace vnm
