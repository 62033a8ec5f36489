// float32 GEMM over ragged active-row sets: Y[M][N] = A[M][K] . W[N][K]^T with
// fused epilogues (rc_internal.h).  The QKV epilogue writes fresh active keys
// and values straight to their token positions in the cache slot (the fusion of
// Sec. 3.4, "Kernel Fusing"), and the residual epilogue can scatter the
// merged hidden state into the cached H (Sec. 3.3 merge).
//
// 32-row tiles whose four waves each hold the whole tile and take a quarter
// of every K stage: LDS reads are two per eight MFMAs of 64 clocks, small
// grids get many workgroups, and the float32 matrix rate (157 TFLOP/s) or, at
// a few hundred rows, the first weights' latency is what is left.  64-wide
// stages stream through a ring of direct copies, two workgroups per CU.
// Against register-staged 64x64 to 128x128 tiles of 2x2 waves: at 154 rows
// 59.6 -> 9.3 us (1152 x 1152) and 230 -> 31 (MLP-down); at 4096 rows MLP-up
// 457 -> 414, QKV 409 -> 315, MLP-down 779 -> 404.
//
// Ring rows are 256 bytes, their sixteen 16-byte chunks XOR-swizzled by row &
// 15 (16 rows of a fragment read touch every bank once).  A lane's 16 bytes
// are four k of its operand row, used one per 32x32x2 MFMA: instruction e
// multiplies k = e of the lower half-wave and k = 4 + e of the upper one, the
// same pairs in A and W.  The waves' partial tiles are summed in wave order.
#include "rc_common.h"
#include "rc_launch.h"
#include "rc_internal.h"

namespace rc {

constexpr int GF_S = 3, GF_BM = 32, GF_K = 64;

template <int BN, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  constexpr int FN = BN / 32, ROWS = GF_BM + BN, STAGE = ROWS * GF_K * 4;
  constexpr int AC = GF_BM * 256 / 4096, NL = ROWS * 256 / 4096;  // copies per wave: A rows', all
  constexpr int CLD = BN + 4;
  static_assert(4 * GF_BM * CLD * 4 <= GF_S * STAGE, "the partial tiles fit the ring");
  __shared__ __attribute__((aligned(1024))) char lds[GF_S * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g32 = lane >> 5, r32 = lane & 31;
  // column panels share an XCD's L2: the row tiles of a panel are consecutive
  const int T = gridDim.x * gridDim.y, L = xcd_logical_id(blockIdx.x + gridDim.x * blockIdx.y, T);
  const int m0 = (L % gridDim.x) * GF_BM, n0 = (L / gridDim.x) * BN;
  const float *A = (const float *)g.A, *W = (const float *)g.W;
  const int nk = g.K / GF_K;
  const float *src[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int row = (i * 4 + wave) * 4 + (lane >> 4), c = (lane & 15) ^ (row & 15);
    src[i] = (i < AC ? A + (size_t)min(m0 + row, g.M - 1) * g.lda : W + (size_t)(n0 + row - GF_BM) * g.K) + c * 4;
  }
  auto issue = [&](int slot, int kt) {
#pragma unroll
    for (int i = 0; i < NL; ++i) lds_dma16(src[i] + kt * GF_K, lds + slot * STAGE + (i * 4 + wave) * 1024);
  };
  f32x16 acc[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
#pragma unroll
  for (int s = 0; s < GF_S - 1; ++s)
    if (s < nk) issue(s, s);
  for (int kt = 0, slot = 0; kt < nk; ++kt, slot = slot == GF_S - 1 ? 0 : slot + 1) {
    if (kt + 1 < nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // (the last stage's fragments have been multiplied: its slot is free past the barrier)
    asm volatile("s_barrier" ::: "memory");
    if (kt + GF_S - 1 < nk) issue(slot == 0 ? GF_S - 1 : slot - 1, kt + GF_S - 1);
    const char *st = lds + slot * STAGE;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = ((wave * 4 + q * 2 + g32) ^ (r32 & 15)) << 4;
      const f32x4 a = *(const f32x4 *)(st + r32 * 256 + c);
      f32x4 b[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = *(const f32x4 *)(st + (GF_BM + j * 32 + r32) * 256 + c);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[j][e], acc[j], 0, 0, 0);
    }
  }
  __syncthreads();
  float *ct = (float *)lds + wave * GF_BM * CLD;
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) ct[((e >> 2) * 8 + g32 * 4 + (e & 3)) * CLD + j * 32 + r32] = acc[j][e];
  __syncthreads();

  constexpr int IT = GF_BM * BN / 4 / 256;
  const int col = (tid % (BN / 4)) * 4, n = n0 + col, row0 = tid / (BN / 4);
  constexpr int RSTEP = 1024 / BN;
  f32x4 bb = f32x4{0.0f, 0.0f, 0.0f, 0.0f}, gt = f32x4{1.0f, 1.0f, 1.0f, 1.0f};
  if (g.bias) bb = *(const f32x4 *)(g.bias + n);
  if (EPI == EPI_RESID && g.gate) gt = *(const f32x4 *)(g.gate + n);
  if (EPI == EPI_RESID && g.gate && g.gate2) gt += *(const f32x4 *)(g.gate2 + n);
  int part = 0, hh = 0, dd = 0;
  if (EPI == EPI_QKV || EPI == EPI_TEXTKV) {
    part = n / g.hidden;
    const int c = n - part * g.hidden;
    hh = c / kHeadDim;
    dd = c - hh * kHeadDim;
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int row = row0 + it * RSTEP, m = m0 + row;
    if (m >= g.M) continue;
    f32x4 v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < 4; ++w) v += *(const f32x4 *)((const float *)lds + (w * GF_BM + row) * CLD + col);
    v += bb;
    if (EPI == EPI_STORE) {
      *(f32x4 *)((float *)g.out + (size_t)m * g.ldo + n) = v;
    } else if (EPI == EPI_GELU) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = gelu_tanh(v[q]);
      *(f32x4 *)((float *)g.out + (size_t)m * g.ldo + n) = v;
    } else if (EPI == EPI_RESID) {
      f32x4 *xp = (f32x4 *)(g.X + (size_t)m * g.ldx + n);
      v = *xp + gt * v;
      *xp = v;
      if (g.xt) *(f32x4 *)((float *)g.xt + (size_t)m * g.ldx + n) = v;
      if (g.hrows) *(f32x4 *)((float *)g.hrows + (size_t)m * g.N + n) = v;
      if (g.hslot) {
        const int pk = g.rows[m];
        *(f32x4 *)((float *)g.hslot + row_chain(pk) * g.chain_stride + (size_t)row_token(pk) * g.hidden + n) = v;
      }
    } else if (EPI == EPI_QKV) {
      if (part == 0) {
        *(f32x4 *)((float *)g.out + (size_t)m * g.ldo + n) = v;
      } else {
        const int pk = g.rows[m];
        *(f32x4 *)((float *)(part == 1 ? g.kslot : g.vslot) + (size_t)row_chain(pk) * g.chain_stride +
                   ((size_t)hh * g.tokens + row_token(pk)) * kHeadDim + dd) = v;
      }
    } else if (EPI == EPI_TEXTKV) {
      const int b = m / g.text_len, t = m - b * g.text_len;
      float *base = (float *)g.tkv + (size_t)b * g.tkv_chain_stride;
      const size_t half = (size_t)(g.hidden / kHeadDim) * g.text_pad * kHeadDim;
      if (part == 0) {
        *(f32x4 *)(base + ((size_t)hh * g.text_pad + t) * kHeadDim + dd) = v;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) base[half + ((size_t)hh * kHeadDim + dd + q) * g.text_pad + t] = v[q];
      }
    }
  }
}

// Row tiles along x: y ends at 65536, which 32-row tiles pass at two million
// rows (128 chains of 2048 px).
dim3 gemm_f32_grid(int M, int N, int bn) { return dim3((M + GF_BM - 1) / GF_BM, N / bn); }

template <int BN> static hipError_t launch_f32(const GemmArgs &a, int epi, hipStream_t s) {
  const dim3 grid = gemm_f32_grid(a.M, a.N, BN), block(256);
  switch (epi) {
    case EPI_STORE: rc_launch(gemm_f32_kernel<BN, EPI_STORE>, grid, block, 0, s, a); break;
    case EPI_GELU: rc_launch(gemm_f32_kernel<BN, EPI_GELU>, grid, block, 0, s, a); break;
    case EPI_RESID: rc_launch(gemm_f32_kernel<BN, EPI_RESID>, grid, block, 0, s, a); break;
    case EPI_QKV: rc_launch(gemm_f32_kernel<BN, EPI_QKV>, grid, block, 0, s, a); break;
    case EPI_TEXTKV: rc_launch(gemm_f32_kernel<BN, EPI_TEXTKV>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Tile choice: the tile whose fullest CU has the least to do (a 32x64 tile
// is two 32x32 ones), 32x64 where they are equal (half the A traffic).  At 154
// rows QKV is 270 of the 32x64 tiles, two on some CUs and one on most: 26.5 us,
// 22 with 540 of 32x32.
hipError_t launch_gemm_f32(const GemmArgs &a, int epi, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N % 64 != 0 || a.K % GF_K != 0) return hipErrorInvalidValue;
  const long w64 = (long)((a.M + GF_BM - 1) / GF_BM) * (a.N / 64);
  return (w64 + 255) / 256 * 2 <= (2 * w64 + 255) / 256 ? launch_f32<64>(a, epi, s) : launch_f32<32>(a, epi, s);
}

}  // namespace rc
