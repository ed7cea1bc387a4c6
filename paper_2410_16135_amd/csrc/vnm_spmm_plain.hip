// vnm_spmm on the canonical triple for the layers the matrix-core kernels do not take: V = 16 or
// M > 16 (no packed copy), rows of X that are not 16-byte aligned, no packed copy handed in.
//
// Both kernels multiply exactly the kept weights with the columns they select (no dense expansion:
// an infinity in a column that a row does not select must not reach it) and accumulate in fp32.
// spmm_generic_kernel, one thread per output walking all of K with uncoalesced 2-byte loads of the
// triple, is the cross-check behind VNM_PATH_GENERIC and the faster one where there are few column blocks
// (plain_scalar_faster).
#include <type_traits>
#include "vnm_internal.h"
#include "vnm_rules.h"

namespace vnm {
namespace {

struct PlainArgs {
  const unsigned short* X; int64_t T, ldx;
  const unsigned* values;            // one dword per (row, block): the two kept weights
  const unsigned char* meta;
  const unsigned* colidx;            // one dword per (row block, block): the four kept columns
  int64_t out, in, B;
  int V, M;
  void* Y; int64_t ldy; int y_fp32;
  Fused f;
};

__device__ __forceinline__ float plain_f(unsigned short bits) {
  _Float16 h;
  __builtin_memcpy(&h, &bits, 2);
  return (float)h;
}

__device__ __forceinline__ void plain_store(const PlainArgs& a, int64_t t, int64_t o, float v) {
  if (a.f.bias) v += (float)a.f.bias[o];
  const int64_t dst = a.f.perm_out ? (int64_t)a.f.perm_out[o] : o;          // Eq. 6, P_o^T
  if (dst < 0 || dst >= a.out) return;
  if (a.y_fp32) ((float*)a.Y)[t * a.ldy + dst] = v;
  else ((_Float16*)a.Y)[t * a.ldy + dst] = (_Float16)v;
}

// column of X that column c of the weight multiplies, -1 for none (Eq. 6, P_i^T)
__device__ __forceinline__ int64_t plain_src(const PlainArgs& a, int64_t c) {
  if (c >= a.in) return -1;
  if (!a.f.perm_in) return c;
  const int64_t s = a.f.perm_in[c];
  return s >= 0 && s < a.in ? s : -1;
}

// ---- many tokens: lane = two adjacent tokens, wave = RW adjacent rows of one row block.
// A workgroup (16 waves) owns 16 RW rows x 128 tokens and walks K in chunks of NB column blocks.  The
// chunk of X sits in LDS as [column][128 tokens] (pitch 260 bytes: the stores of a wave, which run
// along the columns, fall into different banks), so a wave reads the column a weight selects with one
// conflict-free 4-byte read per lane.  Weights are decoded one block per lane (coalesced loads) and
// handed to the whole wave with v_readlane: per (row, block) 8 vector instructions serve 128 tokens.
// Bound by that instruction stream: 10 vector and LDS instructions per (row, block), 4 of them multiply-adds, are half of
// the time, the rest is moving X.  X reaches LDS two tokens at a time (4-byte stores; 2-byte ones, and offsets scaled by
// the scalar unit per block, 25.4 -> 23.5 us on 1000 x 1030 at V = 16, M = 7, 333 tokens, fp32 result, where
// spmm_generic_kernel takes 219; 4096 x 4096, M = 5, 200 tokens 217 -> 202).  Sums run over the blocks in
// ascending order like that kernel's: the results are the same bits.
constexpr int kPlainPitch = kPlainTok * 2 + 4;
static_assert((kPlainCols + 255) * (kPlainPitch / 4) < 65536, "two offsets in a dword");

// A chunk is at most kPlainCols columns: its 128 tokens then fit 16 (PAIR) or 32 registers per lane, which are
// filled for the next chunk while the present one is multiplied.  PAIR: X moves two columns at a time.

template <int RW, bool PAIR>
__global__ void __launch_bounds__(1024)
spmm_plain_tokens_kernel(const PlainArgs a, int NB) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int TU = kPlainTok / 16, CW = PAIR ? 2 : 1, NX = kPlainCols / 64 / CW;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t0 = (int64_t)blockIdx.x * kPlainTok;
  const int64_t wg_row = (int64_t)blockIdx.y * (16 * RW);
  const int64_t row0 = wg_row + wave * RW;
  const int64_t r = row0 / a.V;                       // RW divides V: one row block per wave
  const bool active = row0 < a.out;
  const int64_t mrow = (a.B + 1) / 2;
  float acc[RW][2];
#pragma unroll
  for (int q = 0; q < RW; ++q) acc[q][0] = acc[q][1] = 0.f;
  unsigned pair[RW], byte[RW], k4 = 0, xr[NX][TU];
  bool live[NX];
  int64_t row_off[TU];                                // byte offsets of the wave's token rows, uniform
#pragma unroll
  for (int u = 0; u < TU; ++u) {
    const int64_t t = t0 + 2 * (wave + 16 * (u >> 1)) + (u & 1);     // pairs of adjacent tokens
    row_off[u] = (t < a.T ? t : a.T - 1) * a.ldx * 2;
  }
  // chunk b0: this wave's weights, one block per lane, and 8 token rows of X, lanes along the columns
  auto fetch = [&](int64_t b0) {
    const int nb = (int)(a.B - b0 < NB ? a.B - b0 : NB);
    if (active) {
      const int64_t b = b0 + (lane < nb ? lane : nb - 1);
      k4 = a.colidx[r * a.B + b];
#pragma unroll
      for (int q = 0; q < RW; ++q) {                  // rows of the padding (< R V) hold zeros
        pair[q] = a.values[(row0 + q) * a.B + b];
        byte[q] = a.meta[(row0 + q) * mrow + (b >> 1)];
      }
    }
    // the loads carry no predicate (a branch around each would keep them from being in flight together): a
    // token beyond the last repeats the last one and is never stored, a column that does not exist reads
    // column 0 and is zeroed on its way to LDS
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int c = (lane + 64 * k) * CW;
      const int64_t s = c < nb * a.M ? plain_src(a, b0 * a.M + c) : -1;
      const unsigned off = s >= 0 ? (unsigned)s * 2u : 0u;
      live[k] = s >= 0;
#pragma unroll
      for (int u = 0; u < TU; ++u) {
        const char* row = (const char*)a.X + row_off[u];
        if constexpr (PAIR) xr[k][u] = *(const unsigned*)(row + off);
        else xr[k][u] = *(const unsigned short*)(row + off);
      }
    }
  };
  fetch(0);
  for (int64_t b0 = 0; b0 < a.B; b0 += NB) {
    const int nb = (int)(a.B - b0 < NB ? a.B - b0 : NB);
    const int ncol = nb * a.M;
    unsigned val[RW], offs[RW];                       // the two kept weights; the two columns of the chunk they select
    const unsigned base = (unsigned)lane * a.M, odd = (unsigned)(b0 + lane) & 1;
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      const unsigned nib = odd ? byte[q] >> 4 : byte[q] & 15u;
      const unsigned c0 = base + ((k4 >> (8 * (nib & 3))) & 0xFFu), c1 = base + ((k4 >> (8 * (nib >> 2))) & 0xFFu);
      val[q] = pair[q];
      offs[q] = (c0 | (c1 << 16)) * (kPlainPitch / 4);      // in dwords: below 2^16 each
    }
    __syncthreads();                                  // the previous chunk has been read
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int c = (lane + 64 * k) * CW;
      if (c < ncol) {
#pragma unroll
        for (int u = 0; u < TU; u += 2) {
          // two tokens of a column per store
          unsigned char* d = smem + c * kPlainPitch + (wave + 8 * u) * 4;
          const unsigned x0 = live[k] ? xr[k][u] : 0u, x1 = live[k] ? xr[k][u + 1] : 0u;
          *(unsigned*)d = __builtin_amdgcn_perm(x1, x0, 0x05040100u);
          if constexpr (PAIR) *(unsigned*)(d + kPlainPitch) = __builtin_amdgcn_perm(x1, x0, 0x07060302u);
        }
      }
    }
    __syncthreads();
    if (b0 + NB < a.B) fetch(b0 + NB);
    if (active) {
      const unsigned char* xl = smem + lane * 4;
      // eight reads in flight per row, then their products; a loop with v_readlane is not unrolled by itself
      auto blocks = [&](int b, auto count) {
        constexpr int N = decltype(count)::value;
        unsigned w[RW][N], x0[RW][N], x1[RW][N];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
          for (int q = 0; q < RW; ++q) {
            const unsigned o = __builtin_amdgcn_readlane(offs[q], b + n);
            w[q][n] = __builtin_amdgcn_readlane(val[q], b + n);
            x0[q][n] = *(const unsigned*)(xl + (o & 0xFFFFu) * 4);
            x1[q][n] = *(const unsigned*)(xl + (o >> 16) * 4);
          }
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
          for (int q = 0; q < RW; ++q) {
            const float w0 = plain_f((unsigned short)w[q][n]), w1 = plain_f((unsigned short)(w[q][n] >> 16));
            acc[q][0] = fmaf(w0, plain_f((unsigned short)x0[q][n]), acc[q][0]);
            acc[q][1] = fmaf(w0, plain_f((unsigned short)(x0[q][n] >> 16)), acc[q][1]);
            acc[q][0] = fmaf(w1, plain_f((unsigned short)x1[q][n]), acc[q][0]);
            acc[q][1] = fmaf(w1, plain_f((unsigned short)(x1[q][n] >> 16)), acc[q][1]);
          }
      };
      constexpr int N = RW >= 4 ? 2 : 4;
      int b = 0;
      for (; b + N <= nb; b += N) blocks(b, std::integral_constant<int, N>{});
      for (; b < nb; ++b) blocks(b, std::integral_constant<int, 1>{});
    }
  }
  // results through LDS, so that a store covers the adjacent channels of a token
  constexpr int P = 16 * RW + 1;
  float* ep = (float*)smem;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RW; ++q) {
    ep[(2 * lane) * P + wave * RW + q] = acc[q][0];
    ep[(2 * lane + 1) * P + wave * RW + q] = acc[q][1];
  }
  __syncthreads();
  for (int e = tid; e < kPlainTok * 16 * RW; e += 1024) {
    const int tok = e / (16 * RW), q = e % (16 * RW);
    const int64_t t = t0 + tok, o = wg_row + q;
    if (t < a.T && o < a.out) plain_store(a, t, o, ep[tok * P + q]);
  }
}

// ---- few tokens: lane = one column block, wave = 8 rows of one row block x TT tokens.
// The four columns of a block that its rows choose from are loaded once per 8 rows; a row picks its
// two with one byte permute.  No LDS: neighbouring lanes read neighbouring blocks, so the 2-byte loads of a
// wave cover a few cache lines.  The 64 partial sums of an output meet in a butterfly at the end.
constexpr int kPlainRows = 8;

template <int TT>
__global__ void __launch_bounds__(256)
spmm_plain_blocks_kernel(const PlainArgs a) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * kPlainRows;
  if (row0 >= a.out) return;                          // uniform over the wave; no barrier below
  const int64_t t0 = (int64_t)blockIdx.y * TT;
  const int64_t r = row0 / a.V;
  const int64_t mrow = (a.B + 1) / 2;
  float acc[kPlainRows][TT];
#pragma unroll
  for (int q = 0; q < kPlainRows; ++q)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[q][t] = 0.f;
  for (int64_t b = lane; b < a.B; b += 64) {
    const unsigned k4 = a.colidx[r * a.B + b];
    unsigned pair[kPlainRows], byte[kPlainRows];
#pragma unroll
    for (int q = 0; q < kPlainRows; ++q) {
      pair[q] = a.values[(row0 + q) * a.B + b];
      byte[q] = a.meta[(row0 + q) * mrow + (b >> 1)];
    }
    unsigned xlo[TT], xhi[TT];                        // columns 0, 1 and 2, 3 of the block's kept four
    unsigned short x[4][TT];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t s = plain_src(a, b * a.M + ((k4 >> (8 * k)) & 0xFFu));
#pragma unroll
      for (int t = 0; t < TT; ++t) x[k][t] = s >= 0 && t0 + t < a.T ? a.X[(t0 + t) * a.ldx + s] : (unsigned short)0;
    }
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      xlo[t] = x[0][t] | ((unsigned)x[1][t] << 16);
      xhi[t] = x[2][t] | ((unsigned)x[3][t] << 16);
    }
#pragma unroll
    for (int q = 0; q < kPlainRows; ++q) {
      const unsigned nib = (b & 1) ? byte[q] >> 4 : byte[q] & 15u;
      // byte selector of (position p0, position p1): bytes 2 p, 2 p + 1 of the 8
      const unsigned sel = ((nib & 3) * 0x0202u + 0x0100u) | (((nib >> 2) * 0x0202u + 0x0100u) << 16);
      const float w0 = plain_f((unsigned short)pair[q]), w1 = plain_f((unsigned short)(pair[q] >> 16));
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        const unsigned xs = __builtin_amdgcn_perm(xhi[t], xlo[t], sel);
        acc[q][t] = fmaf(w0, plain_f((unsigned short)xs), acc[q][t]);
        acc[q][t] = fmaf(w1, plain_f((unsigned short)(xs >> 16)), acc[q][t]);
      }
    }
  }
  float mine = 0.f;
#pragma unroll
  for (int q = 0; q < kPlainRows; ++q)
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      float v = acc[q][t];
#pragma unroll
      for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
      mine = lane == q * TT + t ? v : mine;           // lane q TT + t keeps output (row q, token t)
    }
  if (lane < kPlainRows * TT) {
    const int64_t o = row0 + lane / TT, t = t0 + lane % TT;
    if (o < a.out && t < a.T) plain_store(a, t, o, mine);
  }
}

template <int RW, bool PAIR>
int launch_plain_tokens2(const PlainArgs& a, int NB, hipStream_t st) {
  size_t lds = (size_t)(NB * a.M + 1) * kPlainPitch;          // (a pair may end one column past the chunk)
  const size_t ep = (size_t)kPlainTok * (16 * RW + 1) * 4;
  if (ep > lds) lds = ep;
  auto kern = spmm_plain_tokens_kernel<RW, PAIR>;
  if (int rc = allow_big_lds((const void*)kern, "hipFuncSetAttribute(spmm_plain)")) return rc;
  const dim3 grid((unsigned)((a.T + kPlainTok - 1) / kPlainTok), (unsigned)((a.out + 16 * RW - 1) / (16 * RW)));
  hipLaunchKernelGGL(kern, grid, dim3(1024), lds, st, a, NB);
  return VNM_OK;
}

template <int RW>
int launch_plain_tokens(const PlainArgs& a, int NB, hipStream_t st) {
  // two columns per load where every pair of a row is 4-byte aligned and inside the row
  const bool pair = !a.f.perm_in && a.in % 2 == 0 && a.ldx % 2 == 0 && ((uintptr_t)a.X & 3) == 0 && (NB * a.M) % 2 == 0;
  return pair ? launch_plain_tokens2<RW, true>(a, NB, st) : launch_plain_tokens2<RW, false>(a, NB, st);
}

}  // namespace

bool spmm_plain_applicable(int64_t T, const void* colidx, const Dims& d) {
  // the four kept columns of a block are read as one dword
  return ((uintptr_t)colidx & 3) == 0 && plain_sizes_fit(T, d.out, d.in, d.M) && !plain_scalar_faster(T, d.out, d.B, d.M);
}

int launch_spmm_plain(const void* X, int64_t T, int64_t ldx, const void* values, const void* meta, const void* colidx,
                      const Dims& d, void* Y, int64_t ldy, int y_dtype, const Fused& f, hipStream_t st) {
  PlainArgs a;
  a.X = (const unsigned short*)X; a.T = T; a.ldx = ldx;
  a.values = (const unsigned*)values; a.meta = (const unsigned char*)meta; a.colidx = (const unsigned*)colidx;
  a.out = d.out; a.in = d.in; a.B = d.B; a.V = d.V; a.M = d.M;
  a.Y = Y; a.ldy = ldy; a.y_fp32 = y_dtype; a.f = f;
  int rc = VNM_OK;
  if (T >= kPlainManyTokens) {
    const PlainPlan p = plain_plan(T, d.out, d.M);
    if (p.rows_per_wave == 4) rc = launch_plain_tokens<4>(a, p.blocks, st);
    else if (p.rows_per_wave == 2) rc = launch_plain_tokens<2>(a, p.blocks, st);
    else rc = launch_plain_tokens<1>(a, p.blocks, st);
  } else {
    const unsigned gx = (unsigned)((d.out + 4 * kPlainRows - 1) / (4 * kPlainRows));
    if (T == 1) hipLaunchKernelGGL(spmm_plain_blocks_kernel<1>, dim3(gx, 1), dim3(256), 0, st, a);
    else if (T == 2) hipLaunchKernelGGL(spmm_plain_blocks_kernel<2>, dim3(gx, 1), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(spmm_plain_blocks_kernel<4>, dim3(gx, (unsigned)((T + 3) / 4)), dim3(256), 0, st, a);
  }
  if (rc != VNM_OK) return rc;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_hip_error(e, "spmm_plain kernels"); return VNM_ERR_HIP; }
  return VNM_OK;
}

}  // namespace vnm
