// bf16 matrix-core GEMM with large wave tiles: Y[M][N] = A[M][K] . W[N][K]^T,
// N a multiple of 144 (two heads), with the epilogues of the step
// (rc_internal.h); chosen by plan_gemm (rc_gemm2.hip) where it is faster.
//
// What bounds a GEMM of 32x64 or 64x32 wave tiles is LDS: it reads 1.5 KB of
// fragments per 32x32x16 MFMA, 192 bytes per clock and CU where LDS gives 128.
// A wave tile of 64x144 (FM = 4) reads 13 fragments for 36 16x16x32 MFMAs, 90
// bytes per clock; 32x144 (FM = 2), for fewer rows, 11 for 18.
// * Workgroup tiles: 256x288 (4x2 waves), 256x144 and 128x144 (4x1 waves in
//   two K groups), one workgroup per CU; 128x288 (2x2 waves), two per CU, for
//   grids of several rounds, whose epilogues overlap the other's K loop.
// * The W fragments are operand A of the MFMA, so a lane's accumulators are
//   four consecutive columns of one row.
// * Operands move global -> LDS by direct copies of 1 KB per wave into a ring
//   of S stages (32 k per K group), 16-byte chunks swizzled so that a fragment
//   read of 16 rows touches every bank once.
// * A stage's fragments are read while the stage before is multiplied, in the
//   registers that its fragments leave; one barrier per stage.
//
// Measured at 4096 x 4608 x 1152 (256x288 tiles): 0.9 us per stage of 32 k,
// 1.33 PFLOP/s in the loop (a large library GEMM reaches 1.42 here; the power
// limit holds the clock near 1.9 GHz), 3 us to the first stage and 16 us of
// epilogue (GELU: vector issue): 54 us, 68 with the smaller tiles.
#include "rc_common.h"
#include "rc_launch.h"
#include "rc_internal.h"

#include <algorithm>
#include <cmath>

namespace rc {

constexpr int G3_WN = 144;   // columns of a wave tile: 9 blocks of 16
constexpr int G3_NB = 9;

template <int N> __device__ __forceinline__ void wait_vm_g3() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// 16-byte chunk swizzle of a ring row of 64 KG bytes: the 16 rows of a
// fragment read touch all 64 banks once.
template <int KG> __device__ __forceinline__ int swz3(int row) {
  static_assert(KG == 1 || KG == 2, "ring rows of 64 or 128 bytes");
  return KG == 1 ? (row >> 2) & 3 : (row >> 1) & 7;
}

template <int FM, int WGM, int WGN, int KG, int S, int EPI, bool SPLIT>
__global__ __launch_bounds__(64 * WGM * WGN * KG, 2) void gemm3_kernel(GemmArgs g, float *partial, int k_per_split) {
  constexpr int NW = WGM * WGN * KG;
  static_assert(NW == 8 || NW == 4, "eight or four waves");
  constexpr int BM = 16 * FM * WGM, BN = G3_WN * WGN, RB = 64 * KG, CPR = 4 * KG, RPC = 64 / CPR;
  constexpr int STAGE = (BM + BN) * RB;
  constexpr int AC = BM * RB / 1024, TC = STAGE / 1024;  // wave copies of a stage: the A rows', all
  static_assert(AC % NW == 0, "the A rows' copies split over the waves");
  constexpr int NL = (TC + NW - 1) / NW, NFULL = TC % NW ? TC % NW : NW;  // copies per wave: NL on the first NFULL, else NL - 1
  constexpr bool FOLD = EPI == EPI_GELU_FOLD;
  // the output goes through the ring in bands of HB rows, one fp32 tile per
  // K group; rows padded so that 16 rows' 16-byte writes touch all banks
  constexpr int WM = 16 * FM, CLD = BN + 4;
  constexpr int HB = WGM % 2 == 0 && KG * 2 * WM * CLD * 4 <= S * STAGE ? 2 * WM : WM, PASSES = BM / HB;
  static_assert(KG * HB * CLD * 4 <= S * STAGE && BM % HB == 0, "a band fits the ring");
  // column vectors of the epilogue, [NCOL][BN] floats: bias; then gate, gate2
  // and the fold's two scale parts, or u and v.  Eight waves: behind the
  // ring, copied first.  Four waves (two workgroups per CU share its LDS):
  // behind the band, in the ring's end, copied after the K loop.
  constexpr int NCOL = SPLIT ? 0 : EPI == EPI_RESID ? 5 : FOLD ? 3 : 1;
  constexpr bool COL_LATE = NW == 4;
  constexpr int COL_OFF = COL_LATE ? KG * HB * CLD * 4 : S * STAGE;
  constexpr int COL_END = COL_OFF + NCOL * BN * 4, WARM_OFF = COL_END > S * STAGE ? COL_END : S * STAGE;
  static_assert(WARM_OFF + 256 <= kLdsBytes / (8 / NW), "LDS of one CU");
  __shared__ __attribute__((aligned(1024))) char lds[WARM_OFF + 256];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = wave / (WGM * WGN), w4 = wave % (WGM * WGN), wm = w4 / WGN, wn = w4 % WGN;
  const int l16 = lane & 15, lq = lane >> 4;

  const int tiles_m = gridDim.y, tiles_n = gridDim.x, TT = tiles_m * tiles_n, T = TT * gridDim.z;
  const int p = blockIdx.x + tiles_n * (blockIdx.y + tiles_m * blockIdx.z);
  const int L = xcd_logical_id(p, T);
  const int kz = L / TT, r = L - kz * TT;
  constexpr int GM = 2048 / BM;
  const int grp = r / (GM * tiles_n), gm = min(GM, tiles_m - grp * GM), idx = r - grp * GM * tiles_n;
  const int tm = grp * GM + idx % gm, tn = idx / gm;
  const int m0 = tm * BM, n0 = tn * BN;
  if (wave == 0) warm_lines(g.warm, g.warm_lines, p, T, lds + WARM_OFF);

  auto copy_columns = [&]() {  // (missing vectors are skipped, and not read)
    for (int w = wave; w < NCOL; w += NW) {
      const float *cv = w == 0 ? g.bias : FOLD ? (w == 1 ? g.fold_u : g.fold_v)
                        : w == 1 ? g.gate : w == 2 ? g.gate2 : g.fold_scale[w == 4];
      if (cv) {
#pragma unroll
        for (int c = 0; c < (BN * 4 + 1023) / 1024; ++c)
          if (c * 64 + lane < BN / 4) lds_dma16s(cv + n0 + c * 256, lane * 16, lds + COL_OFF + w * BN * 4 + c * 1024);
      }
    }
  };
  if (!COL_LATE) copy_columns();

  const int nk = k_per_split / (32 * KG);
  const char *Ab = (const char *)((const bf16 *)g.A + (size_t)m0 * g.lda + (size_t)kz * k_per_split);
  const char *Wb = (const char *)((const bf16 *)g.W + (size_t)n0 * g.K + (size_t)kz * k_per_split);
  // byte offset of the 16 bytes this lane copies: its A row in each of the
  // wave's copies (rows past the last are clamped to it and never stored),
  // its W row in the first (the others are a uniform distance further)
  constexpr int NA = AC / NW;
  const int row0 = wave * RPC + lane / CPR;
  const unsigned chunk = ((lane % CPR) ^ swz3<KG>(row0)) * 16u;  // (copies are multiples of 16 rows apart)
  unsigned off_a[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) off_a[i] = (unsigned)(min(m0 + row0 + i * NW * RPC, g.M - 1) - m0) * (unsigned)g.lda * 2u + chunk;
  const unsigned off_w = (unsigned)row0 * (unsigned)g.K * 2u + chunk;
  const size_t w_step = (size_t)NW * RPC * g.K * 2;
  auto issue = [&](int slot, int kt) {
    char *s = lds + slot * STAGE + wave * 1024;
    const size_t kb = (size_t)kt * RB;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (i < NL - 1 || wave < NFULL) {
        if (i < NA) lds_dma16s(Ab + kb, off_a[i], s + i * NW * 1024);
        else lds_dma16s(Wb + kb + (i - NA) * w_step, off_w, s + i * NW * 1024);
      }
  };
  // wait until at most `later` stages' copies (issued last) are in flight
  auto wait_stages = [&](int later) {
    if (later >= 2) {
      if (wave < NFULL) wait_vm_g3<2 * NL>();
      else wait_vm_g3<2 * (NL - 1)>();
    } else if (later == 1) {
      if (wave < NFULL) wait_vm_g3<NL>();
      else wait_vm_g3<NL - 1>();
    } else {
      wait_vm_g3<0>();
    }
  };

  // fragment addresses: row l16 of a 16-row block, k chunk kgrp * 4 + lq
  // (16-row blocks start at multiples of 16: the swizzle sees l16 only)
  const int fr = l16 * RB + (((kgrp * 4 + lq) ^ swz3<KG>(l16)) << 4);
  const int a_off = wm * FM * 16 * RB + fr, b_off = (BM + wn * G3_WN) * RB + fr;

  f32x4 acc[FM][G3_NB];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < G3_NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  constexpr int AHEAD = S == 3 ? S : S - 1;  // stages issued before a step needs them
#pragma unroll
  for (int s = 0; s < AHEAD; ++s)
    if (s < nk) issue(s, s);
  wait_stages(min(nk - 1, AHEAD - 1));
  asm volatile("s_barrier" ::: "memory");
  bf16x8 a[FM], b[G3_NB];
#pragma unroll
  for (int i = 0; i < FM; ++i) a[i] = *(const bf16x8 *)(lds + a_off + i * 16 * RB);
#pragma unroll
  for (int j = 0; j < G3_NB; ++j) b[j] = *(const bf16x8 *)(lds + b_off + j * 16 * RB);

  // Step kt multiplies the fragments of stage kt, already in registers, and
  // reads those of stage kt + 1 in their place: a W fragment after its last
  // use, the A fragments behind the last JT column blocks, which run row by
  // row.  Its start waits for stage kt + 1; past the barrier the slot of stage
  // kt - 1, whose fragments every wave has multiplied, takes stage kt + S - 1.
  // With three slots the wave also waits for its reads of stage kt, and that
  // slot takes stage kt + S (two workgroups per CU, or two K groups, cover
  // the wait; with four slots it would be 300 of 1450 clocks of a step).
  constexpr int JT = 3;
  int slot = 0;
#pragma nounroll
  for (int kt = 0; kt < nk; ++kt) {
    const int ns = slot == S - 1 ? 0 : slot + 1;
    if (kt + 1 < nk) {
      wait_stages(min(nk - 2 - kt, AHEAD - 2));
      if (S == 3) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else asm volatile("s_barrier" ::: "memory");
      if (kt + AHEAD < nk) issue(S == 3 ? slot : slot == 0 ? S - 1 : slot - 1, kt + AHEAD);
    }
    const char *st = lds + ns * STAGE;  // (the last step's reads of a stale slot are never used)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < G3_NB - JT; ++j) {
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
      b[j] = *(const bf16x8 *)(st + b_off + j * 16 * RB);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int j = G3_NB - JT; j < G3_NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
      a[i] = *(const bf16x8 *)(st + a_off + i * 16 * RB);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = G3_NB - JT; j < G3_NB; ++j) b[j] = *(const bf16x8 *)(st + b_off + j * 16 * RB);
    __builtin_amdgcn_sched_barrier(0);
    slot = ns;
  }

  // ---------------------------------------------------------------- epilogue
  // Bands of HB rows pass through LDS.  Sixteen lanes then take a row's 144
  // columns of one wave tile: columns 4 l16 + 64 k, k = 0, 1, and on the first
  // four lanes 128 + 4 l16.  The code is kept short (each band runs the same
  // instructions): instructions run once are fetched at about 1 us per
  // kilobyte, which an epilogue straight from the accumulators (20 KB) paid
  // with 20 to 40 us per workgroup.
  // Addresses are a uniform base of the tile plus 32-bit offsets, and the
  // column vectors stay in registers: the vector ALU's issue bounds this part.
  constexpr bool RESID = EPI == EPI_RESID && !SPLIT;
  constexpr int UNITS = HB * WGN / (4 * NW);  // (row, wave tile) units per 16-lane group and band
  constexpr int UC = UNITS < 4 ? UNITS : RESID ? 2 : 4;  // units whose loads are in flight together
  constexpr int RSTEP = 4 / WGN;                         // rows between a lane group's units
  const int part = EPI == EPI_QKV ? n0 / g.hidden : 0;
  const bool need_rows = RESID ? g.hslot != nullptr : part > 0;
  auto st4 = [](void *q, f32x4 v) {
    bf16x4 o;
    o[0] = (bf16)v[0]; o[1] = (bf16)v[1]; o[2] = (bf16)v[2]; o[3] = (bf16)v[3];
    *(bf16x4 *)q = o;
  };
  if (COL_LATE && NCOL) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    copy_columns();
  }
  const bool tail = l16 < 4;                       // lanes with a third group of columns
  const int uc = WGN == 1 ? 0 : (lq & 1) * G3_WN;  // WGN = 2: lane groups alternate between the wave tiles
  const int c0 = uc + l16 * 4, c2 = c0 + (tail ? 128 : 0);  // (the others repeat their first group, unused)
  const int rlane = WGN == 1 ? lq : lq >> 1;
  const int mlast = g.M - 1 - m0;
  f32x4 cb[3], cg[3], cs[3];  // bias (and v); gate or -u; 1 + scale of the fold
  unsigned hoff[3];           // key/value byte offset of the columns
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int c = n0 + (k < 2 ? c0 + 64 * k : c2) - part * g.hidden, hh = c / kHeadDim;
    hoff[k] = EPI == EPI_QKV ? (unsigned)(hh * g.tokens * kHeadDim + c - hh * kHeadDim) * 2u : 0u;
  }
#pragma nounroll
  for (int chunk = 0; chunk < PASSES * (UNITS / UC); ++chunk) {
    const int pass = chunk / (UNITS / UC), q0 = (chunk % (UNITS / UC)) * UC;
    const int band0 = (wave * UNITS + q0) * RSTEP + rlane, row0 = pass * HB + band0;  // unit q: row0 + q RSTEP
    // everything the chunk reads from memory, before the barriers
    f32x4 x[RESID ? UC : 1][3];
    int pk[UC];
    float2 f0[FOLD ? UC : 1], f1[FOLD ? UC : 1];
#pragma unroll
    for (int q = 0; q < UC; ++q) {
      const int rc = min(row0 + q * RSTEP, mlast);
      pk[q] = need_rows ? (g.rows + m0)[rc] : 0;
      if (RESID) {
        const char *X = (const char *)(g.X + (size_t)m0 * g.ldx + n0);
        const unsigned o = (unsigned)(rc * g.ldx + c0) * 4u;
        x[q][0] = *(const f32x4 *)(X + o);
        x[q][1] = *(const f32x4 *)(X + o + 256);
        x[q][2] = *(const f32x4 *)(X + (unsigned)(rc * g.ldx + c2) * 4u);
      }
      if (FOLD) {
        const float2 *st = g.fold_stats + (size_t)m0 * g.fold_nt + rc * g.fold_nt;
        f0[q] = st[min(l16, g.fold_nt - 1)];
        f1[q] = st[min(l16 + 16, g.fold_nt - 1)];
      }
    }
    if (q0 == 0) {
      // barriers on LDS accesses only: the last band's stores stay in flight
      if (chunk == 0) wait_vm_g3<0>();  // (column vectors)
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the ring (or the last band) is consumed
      if ((wm * WM) / HB == pass) {
        float *ct = (float *)lds + ((size_t)kgrp * HB + wm * WM - pass * HB) * CLD + wn * G3_WN;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < G3_NB; ++j) *(f32x4 *)(ct + (i * 16 + l16) * CLD + j * 16 + lq * 4) = acc[i][j];
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (chunk == 0) {
        auto col = [&](int w, int k) {
          return *(const f32x4 *)(lds + COL_OFF + (w * BN + (k < 2 ? c0 + 64 * k : c2)) * 4);
        };
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          cb[k] = cs[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          cg[k] = f32x4{1.0f, 1.0f, 1.0f, 1.0f};
          if (NCOL && g.bias) cb[k] = col(0, k);
          if (RESID && g.gate) cg[k] = g.gate2 ? col(1, k) + col(2, k) : col(1, k);
          if (RESID) cs[k] = g.fold_stats ? 1.0f + col(3, k) + col(4, k) : f32x4{1.0f, 1.0f, 1.0f, 1.0f};
          if (FOLD) {
            cg[k] = -col(1, k);
            cb[k] += col(2, k);
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < UC; ++q) {
      const int row = row0 + q * RSTEP;
      const bool ok = row <= mlast;
      f32x4 v[3];
      const float *ct = (const float *)lds + (band0 + q * RSTEP) * CLD;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float *cp = ct + (k < 2 ? c0 + 64 * k : c2);
        v[k] = *(const f32x4 *)cp;
        if (KG == 2) v[k] += *(const f32x4 *)(cp + HB * CLD);
      }
      if (SPLIT) {
        char *P = (char *)(partial + ((size_t)kz * g.M + m0) * g.N + n0);
        const unsigned o = (unsigned)(row * g.N + c0) * 4u;
        if (ok) {
          *(f32x4 *)(P + o) = v[0];
          *(f32x4 *)(P + o + 256) = v[1];
          if (tail) *(f32x4 *)(P + o + 512) = v[2];
        }
      } else if (RESID) {
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = x[q][k] + cg[k] * (v[k] + cb[k]);
        if (g.fold_stats) {
          // statistics of the row over these 144 columns (a tile of the fold)
          float sm = (v[0][0] + v[0][1]) + (v[0][2] + v[0][3]) + ((v[1][0] + v[1][1]) + (v[1][2] + v[1][3]));
          sm += tail ? (v[2][0] + v[2][1]) + (v[2][2] + v[2][3]) : 0.0f;
          const float mean = row16_sum(sm) / G3_WN;
          float d2 = 0.0f, d2t = 0.0f;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            d2 += (v[0][e] - mean) * (v[0][e] - mean) + (v[1][e] - mean) * (v[1][e] - mean);
            d2t += (v[2][e] - mean) * (v[2][e] - mean);
          }
          d2 = row16_sum(d2 + (tail ? d2t : 0.0f));
          if (ok && l16 == 0)
            (g.fold_stats + (size_t)m0 * g.fold_nt)[row * g.fold_nt + (n0 + uc) / G3_WN] = make_float2(mean, d2);
        }
        if (ok) {
          const unsigned o = (unsigned)(row * g.ldx + c0) * 4u;
          char *X = (char *)(g.X + (size_t)m0 * g.ldx + n0);
          *(f32x4 *)(X + o) = v[0];
          *(f32x4 *)(X + o + 256) = v[1];
          if (tail) *(f32x4 *)(X + o + 512) = v[2];
          if (g.hslot || g.hrows) {
            char *h = g.hslot ? (char *)((bf16 *)g.hslot + row_chain(pk[q]) * g.chain_stride +
                                         (size_t)row_token(pk[q]) * g.hidden + n0 + c0)
                              : (char *)((bf16 *)g.hrows + (size_t)(m0 + row) * g.N + n0 + c0);
            st4(h, v[0]);
            st4(h + 128, v[1]);
            if (tail) st4(h + 256, v[2]);
          }
          if (g.xt) {
            char *xt = (char *)((bf16 *)g.xt + (size_t)m0 * g.ldx + n0);
            st4(xt + (o >> 1), v[0] * cs[0]);
            st4(xt + (o >> 1) + 128, v[1] * cs[1]);
            if (tail) st4(xt + (o >> 1) + 256, v[2] * cs[2]);
          }
        }
      } else {
        if (FOLD) {
          // mean and 1/std of the row from the producer's partials (equal
          // column counts), then h W^T = r (x~ W^T - mean u) + v
          const int nt = g.fold_nt;
          const bool o0 = l16 < nt, o1 = l16 + 16 < nt;
          const float cnt = (float)(g.K / nt);
          const float mu = row16_sum((o0 ? f0[q].x : 0.0f) + (o1 ? f1[q].x : 0.0f)) / (float)nt;
          const float e0 = f0[q].x - mu, e1 = f1[q].x - mu;
          const float m2 = row16_sum((o0 ? f0[q].y + cnt * e0 * e0 : 0.0f) + (o1 ? f1[q].y + cnt * e1 * e1 : 0.0f));
          const float rstd = rsqrtf(m2 / (float)g.K + g.fold_eps);
#pragma unroll
          for (int k = 0; k < 3; ++k) v[k] = rstd * (v[k] + mu * cg[k]) + cb[k];
        } else {
#pragma unroll
          for (int k = 0; k < 3; ++k) v[k] += cb[k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (EPI == EPI_GELU || FOLD)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][e] = gelu_tanh(v[k][e]);
          if (EPI == EPI_QKV && part == 0) v[k] *= g.q_scale;
        }
        if (ok) {
          if (EPI == EPI_QKV && part > 0) {
            char *s = (char *)((bf16 *)(part == 1 ? g.kslot : g.vslot) + (size_t)row_chain(pk[q]) * g.chain_stride +
                               (size_t)row_token(pk[q]) * kHeadDim);
            st4(s + hoff[0], v[0]);
            st4(s + hoff[1], v[1]);
            if (tail) st4(s + hoff[2], v[2]);
          } else {
            char *o = (char *)((bf16 *)g.out + (size_t)m0 * g.ldo + n0);
            const unsigned off = (unsigned)(row * g.ldo + c0) * 2u;
            st4(o + off, v[0]);
            st4(o + off + 128, v[1]);
            if (tail) st4(o + off + 256, v[2]);
          }
        }
      }
    }
  }
  if (RESID && g.fold_stats && g.fold_extra && tm == 0 && tid < BN / 4) {
    // the four rows of a consumer that takes u and v from its own tiles:
    // 1 + scale and shift, each as its bf16 rounding and the remainder's
    const int n = n0 + tid * 4;
    const f32x4 sc = 1.0f + *(const f32x4 *)(g.fold_scale[0] + n) + *(const f32x4 *)(g.fold_scale[1] + n);
    const f32x4 sh = *(const f32x4 *)(g.fold_shift[0] + n) + *(const f32x4 *)(g.fold_shift[1] + n);
    f32x4 hi, hi2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      hi[q] = (float)(bf16)sc[q];
      hi2[q] = (float)(bf16)sh[q];
    }
    bf16 *e = (bf16 *)g.fold_extra + n;
    st4(e, hi);
    st4(e + g.N, sc - hi);
    st4(e + 2 * (size_t)g.N, hi2);
    st4(e + 3 * (size_t)g.N, sh - hi2);
  }
}

// u = W (1 + scale) and v = W shift of a folded LayerNorm, for every block of
// a step (fp32 sums over the bf16 weights).  A workgroup holds 1 + scale and
// shift in LDS and takes 32 rows of W, eight per wave, all loaded before the
// first is used: bound by the weights' bytes (14 us for four blocks' 42 MB;
// 22.9 with a row per wave, which reads the two vectors again for each row).
constexpr int UV_ROWS = 32;
__global__ __launch_bounds__(256) void fold_uv_kernel(FoldUvArgs a) {
  constexpr int RW = UV_ROWS / 4, MAXC = 3;  // rows per wave; C <= 512 MAXC
  __shared__ float sc[512 * MAXC], sh[512 * MAXC];
  const int l = blockIdx.y, tid = threadIdx.x, lane = tid & 63, n0 = blockIdx.x * UV_ROWS + (tid >> 6) * RW;
  bf16x8 w[RW][MAXC];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const bf16 *row = (const bf16 *)a.w[l] + (size_t)(n0 + r) * a.C;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int k = (lane + 64 * i) * 8;
      w[r][i] = Mfma<bf16>::zero();
      if (k < a.C) w[r][i] = *(const bf16x8 *)(row + k);
    }
  }
  const float *sst = a.sst[l] + (size_t)a.shift_row * a.C, *t0 = a.t0 + (size_t)a.shift_row * a.C;
  for (int k = tid; k < 512 * MAXC; k += 256) {
    sh[k] = k < a.C ? sst[k] + t0[k] : 0.0f;
    sc[k] = k < a.C ? 1.0f + sst[a.C + k] + t0[a.C + k] : 0.0f;
  }
  __syncthreads();
  float u[RW], v[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) u[r] = v[r] = 0.0f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = (lane + 64 * i) * 8 + q;
      const float s = sc[k], t = sh[k];
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        u[r] += (float)w[r][i][q] * s;
        v[r] += (float)w[r][i][q] * t;
      }
    }
  float *out = a.uv + (size_t)(a.l0 + l) * 2 * a.F;
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    u[r] = wave_sum(u[r]);
    v[r] = wave_sum(v[r]);
    if (lane == 0) {
      out[n0 + r] = u[r];
      out[a.F + n0 + r] = v[r];
    }
  }
}

hipError_t launch_fold_uv(const FoldUvArgs &a, int layers, hipStream_t s) {
  if (layers <= 0) return hipSuccess;
  if (layers > FoldUvArgs::kLayers || a.F % UV_ROWS || a.C % 8 || a.C > 1536) return hipErrorInvalidValue;
  rc_launch(fold_uv_kernel, dim3(a.F / UV_ROWS, layers), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int FM, int WGM, int WGN, int KG, int S, bool SPLIT>
static void launch_g3(const GemmArgs &a, int epi, int splits, float *partial, hipStream_t s) {
  constexpr int BM = 16 * FM * WGM, BN = G3_WN * WGN;
  dim3 grid(a.N / BN, (a.M + BM - 1) / BM, splits);
  const int kps = a.K / splits;
#define RC_G3(E) rc_launch(gemm3_kernel<FM, WGM, WGN, KG, S, E, SPLIT>, grid, dim3(64 * WGM * WGN * KG), 0, s, a, partial, kps)
  if constexpr (SPLIT) {
    RC_G3(EPI_RESID);
  } else {
    switch (epi) {
      case EPI_STORE: RC_G3(EPI_STORE); break;
      case EPI_GELU: RC_G3(EPI_GELU); break;
      case EPI_GELU_FOLD: RC_G3(EPI_GELU_FOLD); break;
      case EPI_RESID: RC_G3(EPI_RESID); break;
      case EPI_QKV: RC_G3(EPI_QKV); break;
    }
  }
#undef RC_G3
}

hipError_t launch_gemm3(const GemmArgs &a, int epi, const GemmPlan &pl, float *partial, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N % pl.bn || a.K % (32 * pl.kg * pl.splits) || epi == EPI_TEXTKV ||
      (pl.splits > 1 && (epi != EPI_RESID || pl.bm != 128 || pl.bn != 144)))
    return hipErrorInvalidValue;
  if (epi == EPI_QKV && a.hidden % pl.bn) return hipErrorInvalidValue;
  if (epi == EPI_GELU_FOLD &&
      (a.fold_nt <= 0 || a.fold_nt > kFoldMaxTiles || a.K % a.fold_nt || !a.fold_stats || !a.fold_u || !a.fold_v))
    return hipErrorInvalidValue;
  if (epi == EPI_RESID && a.fold_stats && (pl.splits > 1 || a.fold_nt != a.N / G3_WN || !a.xt)) return hipErrorInvalidValue;
  switch (pl.bm * 1000 + pl.bn) {
    case 256288: launch_g3<4, 4, 2, 1, 4, false>(a, epi, 1, nullptr, s); break;
    case 256144: launch_g3<4, 4, 1, 2, 3, false>(a, epi, 1, nullptr, s); break;
    case 128144:
      if (pl.splits > 1) launch_g3<2, 4, 1, 2, 4, true>(a, epi, pl.splits, partial, s);
      else launch_g3<2, 4, 1, 2, 4, false>(a, epi, 1, nullptr, s);
      break;
    case 128288: launch_g3<4, 2, 2, 1, 3, false>(a, epi, 1, nullptr, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rc
