// Mask refresh of LoRA training with dynamic masks (Section 4.3, Eq. 10) in three kernels: the merge, which also takes the
// row and column sums of the RIA scores (Section 3, Eq. 1) while it holds the merged weights in registers; a small one that
// adds the sums up; and the pruning, which computes the scores where it needs them (vnm_prune_fast.hip).
// Same bits as vnm_lora_merge, vnm_ria_scores and vnm_prune_compress_scored in a row, which read the merged weight three
// more times and write and read an fp32 score matrix in between.  That chain is what runs for shapes and alignments
// these kernels do not take.
#include "vnm_internal.h"
#include "vnm_score.h"

namespace vnm {
namespace {

constexpr int kRfWaves = 4;
constexpr int kRfRows = kRfWaves * kMergeRows;      // rows of a workgroup
constexpr int kRfCols = 512;                        // columns of a workgroup, 8 adjacent ones per lane

// Merge of a tile of 32 rows x 512 columns, a wave per 8 rows, and the tile's sums of magnitudes: one per column (32 rows)
// and one per row (512 columns), in doubles scaled by 2^-136 (sc_scaled).  All are exact: a sum of up to 512 magnitudes of
// at most 2^41 units.  No atomics, every partial sum is written by one thread.
// Column sums are stored lane by lane (position 64 e + lane of the tile holds column 8 lane + e), so that the store is
// contiguous; ria_prepare_kernel knows.
// Bound by the merge's arithmetic: separate products and sums are 14 us of vector issue at r = 16 on 4096 x 4096, the sums
// another 4; 27 us.  Longer-lived waves lose (two tiles of 8 rows per wave, the next one's weights requested ahead: 29 us, and
// 33.5 us against 26.5 for the whole refresh of 1000 x 1000), and so do A and B in LDS (34 us).
__global__ void __launch_bounds__(64 * kRfWaves)
merge_sums_kernel(const unsigned short* __restrict__ W, int64_t ldw, const float* __restrict__ B, int64_t ldb,
                  const float* __restrict__ A, int64_t lda, int r, float scale, int64_t out, int64_t in,
                  unsigned short* __restrict__ Wm, int64_t ldm, double* __restrict__ colpart, double* __restrict__ rowpart) {
  __shared__ double part[kRfWaves][8][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t o0 = (int64_t)blockIdx.y * kRfRows + wave * kMergeRows;
  const int64_t i0 = (int64_t)blockIdx.x * kRfCols + lane * 8;
  const bool col_ok = i0 < in;                        // in % 8 == 0: all 8 columns or none
  const int64_t ic = col_ok ? i0 : 0;
  const int rows = out - o0 >= kMergeRows ? kMergeRows : (out > o0 ? (int)(out - o0) : 0);
  double cs[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) cs[e] = 0.0;
  if (rows > 0) {
    uint4 w[kMergeRows], m[kMergeRows];
    if (rows == kMergeRows) {
      merge_load<false>(W + o0 * ldw + ic, ldw, 0, w);
      merge_tile<false>(w, B + o0 * ldb, ldb, A + ic, lda, r, scale, 0, m);
    } else {
      merge_load<true>(W + o0 * ldw + ic, ldw, rows - 1, w);
      merge_tile<true>(w, B + o0 * ldb, ldb, A + ic, lda, r, scale, rows - 1, m);
    }
    double rs[8];
#pragma unroll
    for (int v = 0; v < kMergeRows; ++v) {
      rs[v] = 0.0;
      const bool ok = col_ok && v < rows;
      if (ok) *(uint4*)(Wm + (o0 + v) * ldm + i0) = m[v];
      const unsigned d[4] = {ok ? m[v].x : 0u, ok ? m[v].y : 0u, ok ? m[v].z : 0u, ok ? m[v].w : 0u};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double lo = sc_scaled(d[e]), hi = sc_scaled(d[e] >> 16);
        cs[2 * e] += lo;
        cs[2 * e + 1] += hi;
        rs[v] += lo + hi;
      }
    }
    // row sums over the wave: in each of three steps a lane passes on half of its rows and keeps the other half, so that
    // lane l holds one row, then three plain steps
    auto half = [&](bool upper, int o, auto count) {
      constexpr int n = decltype(count)::value;
#pragma unroll
      for (int e = 0; e < n; ++e) {
        const double send = upper ? rs[e] : rs[e + n], keep = upper ? rs[e + n] : rs[e];
        rs[e] = keep + __shfl_xor(send, o);
      }
    };
    half(lane & 1, 1, std::integral_constant<int, 4>{});
    half(lane & 2, 2, std::integral_constant<int, 2>{});
    half(lane & 4, 4, std::integral_constant<int, 1>{});
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) rs[0] += __shfl_xor(rs[0], o);
    const int row = (lane & 1) * 4 + ((lane >> 1) & 1) * 2 + ((lane >> 2) & 1);
    if (lane < 8 && row < rows) rowpart[(o0 + row) * gridDim.x + blockIdx.x] = rs[0];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[wave][e][lane] = cs[e];
  __syncthreads();
  double* cp = colpart + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kRfCols;
#pragma unroll
  for (int p = threadIdx.x; p < kRfCols; p += 64 * kRfWaves) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kRfWaves; ++k) t += part[k][p >> 6][p & 63];
    cp[p] = t;
  }
}

__device__ __forceinline__ unsigned long long rf_units(double scaled) { return (unsigned long long)(scaled * 0x1p136); }

// prep f64 [3][in] and [2][out], what a score needs of its column -- the sum (in units), its reciprocal and act * 2^136 --
// and of its row.  The first col_tiles * 8 workgroups take 64 positions of a tile each, the row tiles over their four
// waves; the others 256 rows.  Totals are taken in integers (they may not fit 53 bits).
__global__ void __launch_bounds__(256)
ria_prepare_kernel(const double* __restrict__ colpart, int64_t row_tiles, int64_t col_tiles, int64_t in,
                   const float* __restrict__ act, const double* __restrict__ rowpart, int64_t out, double* __restrict__ prep) {
  if (blockIdx.x >= col_tiles * 8) {
    const int64_t row = ((int64_t)blockIdx.x - col_tiles * 8) * 256 + threadIdx.x;
    if (row >= out) return;
    const double* p = rowpart + row * col_tiles;
    unsigned long long t = 0;
    int64_t k = 0;
    for (; k + 8 <= col_tiles; k += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[k + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) t += rf_units(v[u]);
    }
    for (; k < col_tiles; ++k) t += rf_units(p[k]);
    const double c = (double)t;
    prep[3 * in + row] = c;
    prep[3 * in + out + row] = c > 0.0 ? 1.0 / c : 0.0;
    return;
  }
  __shared__ unsigned long long part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tile = blockIdx.x >> 3;
  const int e = blockIdx.x & 7;
  const double* p = colpart + tile * kRfCols + e * 64 + lane;
  const int64_t pitch = col_tiles * kRfCols;
  unsigned long long t = 0;
  int64_t k = wave;
  for (; k + 28 < row_tiles; k += 32) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(k + 4 * u) * pitch];
#pragma unroll
    for (int u = 0; u < 8; ++u) t += rf_units(v[u]);
  }
  for (; k < row_tiles; k += 4) t += rf_units(p[k * pitch]);
  part[wave][lane] = t;
  __syncthreads();
  const int64_t col = tile * kRfCols + lane * 8 + e;
  if (wave == 0 && col < in) {
    const double c = (double)(part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane]);
    prep[col] = c;
    prep[in + col] = c > 0.0 ? 1.0 / c : 0.0;          // a zero sum: every quotient of its terms is 0
    prep[2 * in + col] = (double)act[col] * 0x1p136;
  }
}

// Workspace of the fused form: [column partial sums | row partial sums | prep]
struct RefreshLayout { int64_t rt, ct, rowpart, prep, bytes; };
RefreshLayout refresh_layout(int64_t out, int64_t in) {
  RefreshLayout l;
  l.rt = (out + kRfRows - 1) / kRfRows;
  l.ct = (in + kRfCols - 1) / kRfCols;
  l.rowpart = l.rt * l.ct * kRfCols * 8;
  l.prep = l.rowpart + out * l.ct * 8;
  l.bytes = l.prep + (3 * in + 2 * out) * 8;
  return l;
}

}  // namespace
}  // namespace vnm

using namespace vnm;

extern "C" int vnm_refresh_mask_workspace_bytes(int64_t out, int64_t in, int V, int N, int M, int64_t* bytes) {
  if (!bytes) return VNM_ERR_NULL;
  if (int rc = check_pattern(out, in, V, N, M)) return rc;
  *bytes = prune_fast_ria_applicable(nullptr, in, make_dims(out, in, V, M)) ? refresh_layout(out, in).bytes : 0;
  return VNM_OK;
}

extern "C" int vnm_refresh_mask(const void* W, int64_t out, int64_t in, int64_t ldw, const void* B, int64_t ldb, const void* A,
                                int64_t lda, int r, float scale, const void* act, int V, int N, int M, void* W_merged, int64_t ldm,
                                void* values, void* meta, void* colidx, void* mask, void* packed, void* workspace,
                                int64_t workspace_bytes, void* stream) {
  if (!W || !W_merged || !act || !values || !meta || !colidx || !workspace || (r > 0 && (!B || !A))) return VNM_ERR_NULL;
  if (int rc = check_pattern(out, in, V, N, M)) return rc;
  if (r < 0 || ldw < in || ldm < in || (r > 0 && (ldb < r || lda < in))) return VNM_ERR_SHAPE;
  if (((uintptr_t)W & 1) || ((uintptr_t)W_merged & 1) || ((uintptr_t)B & 3) || ((uintptr_t)A & 3) || ((uintptr_t)act & 3) ||
      ((uintptr_t)values & 3) || ((uintptr_t)colidx & 3) || ((uintptr_t)packed & 255) || ((uintptr_t)workspace & 7))
    return VNM_ERR_ALIGN;
  const Dims d = make_dims(out, in, V, M);
  const RefreshLayout l = refresh_layout(out, in);
  if (packed && !has_packed(V, M)) return VNM_ERR_UNSUPPORTED;
  // 16-byte accesses to rows of W, A and the merged weight; grids
  if (ldw % 8 != 0 || lda % 4 != 0 || (((uintptr_t)W | (uintptr_t)A) & 15) || !prune_fast_ria_applicable(W_merged, ldm, d) ||
      l.rt > 65535 || l.ct * 8 + out > 0x7FFFFFFF)
    return VNM_ERR_UNSUPPORTED;
  if (workspace_bytes < l.bytes) return VNM_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  double* colpart = (double*)workspace;
  double* rowpart = (double*)((char*)workspace + l.rowpart);
  double* prep = (double*)((char*)workspace + l.prep);
  hipLaunchKernelGGL(merge_sums_kernel, dim3((unsigned)l.ct, (unsigned)l.rt), dim3(64 * kRfWaves), 0, st,
                     (const unsigned short*)W, ldw, (const float*)B, ldb, (const float*)A, lda, r, scale, out, in,
                     (unsigned short*)W_merged, ldm, colpart, rowpart);
  hipLaunchKernelGGL(ria_prepare_kernel, dim3((unsigned)(l.ct * 8 + (out + 255) / 256)), dim3(256), 0, st, colpart,
                     l.rt, l.ct, in, (const float*)act, rowpart, out, prep);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_hip_error(e, "merge_sums_kernel"); return VNM_ERR_HIP; }
  return launch_prune_fast_ria(W_merged, ldm, prep, d, values, meta, colidx, mask, packed, st);
}
