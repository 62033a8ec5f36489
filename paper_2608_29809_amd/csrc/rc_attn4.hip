// bf16 self-attention over a cache slot (head dim 72): active queries of one
// (chain, head, key range) against all its keys, key splits combined by a
// second kernel.
//
// Scores are formed transposed (S^T = K Q^T), so a lane owns one query and
// its probabilities are in registers the B operand of O^T = V^T P^T:
// * key order inside a 32-key sub-tile: the K row that lane m supplies is
//   key pi(m) = ((m>>4)&1)*16 + ((m>>2)&1)*8 + ((m>>3)&1)*4 + (m&3), so that
//   accumulator e = c*8 + k of lane group g is key c*16 + g*8 + k;
// * dims 0..63 of O^T are two 32x32x16 blocks; dims 64..71 and the softmax
//   denominator (a row of ones behind the values, so that it sums the same
//   rounded probabilities) are one block of 16 rows by 16x16x32, whose two
//   query halves take their operand from v_permlane16_swap of the two 16-key
//   operands.  (A third 32-row block would spend 64 instead of 32 matrix
//   clocks per 32 queries x 32 keys on nine useful rows: 1112 against 1050 us
//   per launch for 16384 queries of 16384 keys.)
// * V^T operands are assembled from the token-major value tile by LDS
//   transpose reads (ds_read_b64_tr_b16).
//
// Softmax without a running maximum.  The queries arrive multiplied by
// log2(e)/sqrt(72), so a score is a base-2 logit and its probability is one
// v_exp_f32 of the accumulator, relative to the fixed reference 0: bf16
// probabilities and fp32 sums keep their relative precision over the whole
// exponent range, so any reference serves as long as nothing leaves the
// range.  A workgroup one of whose denominators is not inside [2^-40, 2^80]
// (or is NaN), or one of whose sums of values is not finite (values above
// 2^48 beside a large denominator), starts again relative to each query's
// maximum over the key range: a pass over the keys finds it, and its negative
// goes as three bf16 parts (24 bits: exactly) into the query dims 72..74,
// which meet ones in the padded key dims.  Probabilities below 2^-126 are
// lost, at most 2^-72 of an accepted denominator for 16384 keys, and values
// above 2^-86 keep their precision.  The restart costs what it repeats: with
// every workgroup in it, 723 queries of 4096 keys and their combine take 53.6
// us instead of 30.2, 4096 of 4096 190 instead of 85, 16384 of 16384 2.5 ms
// instead of 1.14 (logits beyond 55, or all of a query's below -28).
//
// A wave holds QH = 2 or 1 halves of 32 queries.  What bounds the kernel: for
// many queries the matrix core at the clock that the power limit leaves (63 %
// of the matrix cycles at 1.84 GHz for 16384 x 16384: 1.3 PFLOP/s with the
// padding, the rate of a large library GEMM here).  A unit of 32 queries and
// 32 keys takes 320 matrix clocks of its SIMD and, for QH = 1, 10 KB of key and
// value fragments: the four SIMDs of a CU read 40 KB in that time, all that LDS
// gives (128 bytes per clock).  QH = 2 reads each fragment once for 64 queries,
// half of that.  For a few hundred queries the fixed time bounds it (about 4 us
// to the first tile, 1.2 us of stores), and QH = 1 gives it more workgroups
// with shorter ends.  The work is written as pairs of 32x32 units so that the
// exponentials of one run under the matrix instructions of the other; the
// groups are kept apart by scheduling barriers, and a wave has issue priority
// over the other wave of its SIMD in its PV half (23.3 against 24.1 us at 723
// queries of 4096 keys, 1062 against 1078 us at 16384 of 16384; priority in
// the score half gives half of that).
//
// Measured per launch, before (one 32-query form with a running maximum) and
// now: 16384 queries of 16384 keys 1411 -> 1073 us, 2458 of 16384 236 -> 182,
// 4096 of 4096 97.3 -> 83.3, 1640 in four chains of 4096 50.0 -> 44.8, 723 of
// 4096 23.6 -> 21.7 us; 300 chains of 64 keys 39.4 -> 40.3 us, one query of
// 1024 keys 4.9 -> 5.3 us.
#include "rc_common.h"
#include "rc_launch.h"
#include "rc_internal.h"

#include <algorithm>
#include <cmath>

namespace rc {

constexpr int A4_BK = 64;

__device__ __forceinline__ int key_perm4(int m) {
  return ((m >> 4) & 1) * 16 + ((m >> 2) & 1) * 8 + ((m >> 3) & 1) * 4 + (m & 3);
}
// Workgroup barrier without a memory fence: each wave waits for its own tile
// copies first (wait_tiles), and reads of a ring slot are consumed before the
// barrier that frees it.
__device__ __forceinline__ void lds_barrier4() { asm volatile("s_barrier" ::: "memory"); }
// The first barrier: the constants that thread 0 wrote to LDS are there too.
__device__ __forceinline__ void lds_barrier4_first() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vm4() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// WARM: also warm a.warm into the memory-side cache (an instantiation of its
// own, so that the kernel without it carries none of its code or LDS).
template <int QH, bool WARM>
__global__ __launch_bounds__(256, 2) void attn4_kernel(AttnArgs a) {
  constexpr int D = kHeadDim;
  constexpr int KT_BYTES = A4_BK * D * 2, STAGE = 2 * KT_BYTES;
  constexpr int BQ = 128 * QH, WQ = 32 * QH;
  constexpr int CH = KT_BYTES / 1024;  // 1024-byte wave copies per operand tile (9)
  constexpr int STAGES = QH == 2 ? 3 : 4;  // ring depth
  constexpr int CONST_OFF = STAGES * STAGE;
  constexpr int FLAG_OFF = CONST_OFF + 32;
  __shared__ __attribute__((aligned(1024))) char lds[CONST_OFF + 64 + (WARM ? 256 : 0)];
  // read in place of value dims 72..79: (1, 0, 0, 0) and zeros; and of key dims 72..79: (1, 1, 1, 0, ...)
  char *ones_chunk = lds + CONST_OFF, *zero_chunk = ones_chunk + 8, *ref_chunk = ones_chunk + 16;
  volatile int *flag = (volatile int *)(lds + FLAG_OFF);
  if (threadIdx.x == 0) {
    *(V16 *)ones_chunk = V16{{0x00003F80u, 0u, 0u, 0u}};
    *(V16 *)ref_chunk = V16{{0x3F803F80u, 0x00003F80u, 0u, 0u}};
    *flag = 0;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (without the range every tile copy is a branch of its own; with that and
  // the conversions of LDS pointers a launch of few key tiles took 0.5 to 1 us
  // more, and one of 723 queries of 4096 keys, combined, 31.5 instead of 29.3)
  __builtin_assume(wave >= 0 && wave < 4);
  const int g = lane >> 5, r32 = lane & 31;
  const int heads = a.hidden / D;
  const int G = gridDim.x, Y = gridDim.y, T = G * Y * gridDim.z;
  const int p = blockIdx.x + G * (blockIdx.y + Y * blockIdx.z);
  const int L = xcd_logical_id(p, T);
  const int qt = L % G, hy = (L / G) % Y, b = L / (G * Y);
  const int h = hy % heads, split = hy / heads;
  const int n_tiles = a.n_keys / A4_BK;
  const int t_beg = (int)((long)split * n_tiles / a.splits), t_end = (int)((long)(split + 1) * n_tiles / a.splits);
  const int n = t_end - t_beg;
  const char *Kg = (const char *)((const bf16 *)a.K + b * a.chain_stride + h * a.head_stride) + (size_t)t_beg * KT_BYTES;
  const char *Vg = (const char *)((const bf16 *)a.V + b * a.chain_stride + h * a.head_stride) + (size_t)t_beg * KT_BYTES;
  if (WARM && wave == 0) warm_lines(a.warm, a.warm_lines, p, T, lds + CONST_OFF + 64);

  const unsigned lds0 = lds_address(lds);
  // tile copies: 18 wave copies of 1024 bytes, 5 on waves 0 and 1, 4 on 2 and 3
  auto issue_from = [&](const char *keys, const char *values, int slot, int tile) {
    const unsigned s = lds0 + slot * STAGE;
    const char *kt = keys + (size_t)tile * KT_BYTES, *vt = values + (size_t)tile * KT_BYTES;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const int c = i * 4 + wave;
      if (c < 2 * CH) lds_dma16s(c < CH ? kt + c * 1024 : vt + (c - CH) * 1024, lane * 16, s + c * 1024);
    }
  };
  auto issue = [&](int slot, int tile) { issue_from(Kg, Vg, slot, tile); };
  const int2 rr = chain_rows(a, b);
  const int r1 = rr.y, q0 = rr.x + qt * BQ;
  if (q0 >= r1) {
    wait_vm4<0>();
    return;
  }
  // QH = 1: the queries are copied into the ring's last slot first
  const bf16 *Qg = (const bf16 *)a.Q + h * D;
  if (QH == 1) {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const int c = i * 4 + wave;
      if (c < 2 * CH) {
        const int ch = c * 64 + lane, row = ch / 9;
        lds_dma16(Qg + (size_t)min(q0 + row, r1 - 1) * a.hidden + (ch - row * 9) * 8, lds + (STAGES - 1) * STAGE + c * 1024);
      }
    }
  }
  // wait until at most `later` younger tiles' copies are in flight
  auto wait_tiles = [&](int later) {
    if (later >= 2) {
      if (wave < 2) wait_vm4<10>();
      else wait_vm4<8>();
    } else if (later == 1) {
      if (wave < 2) wait_vm4<5>();
      else wait_vm4<4>();
    } else {
      wait_vm4<0>();
    }
  };
  bf16x8 qf[QH][5];
  if (QH == 1) {
#pragma unroll
    for (int i = 0; i < STAGES - 1; ++i)
      if (i < n) issue(i, i);
    wait_tiles(min(n - 1, STAGES - 2));
    lds_barrier4_first();
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      const int d0 = c * 16 + g * 8;
      qf[0][c] = Mfma<bf16>::zero();
      if (d0 < D) qf[0][c] = *(const bf16x8 *)(lds + (STAGES - 1) * STAGE + (wave * 32 + r32) * D * 2 + d0 * 2);
    }
  } else {
    issue(0, 0);
#pragma unroll
    for (int hh = 0; hh < QH; ++hh) {
      const bf16 *qrow = Qg + (size_t)min(q0 + wave * WQ + hh * 32 + r32, r1 - 1) * a.hidden;
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const int d0 = c * 16 + g * 8;
        qf[hh][c] = Mfma<bf16>::zero();
        if (d0 < D) qf[hh][c] = *(const bf16x8 *)(qrow + d0);
      }
    }
    // (consumed here so that no wait for them is left inside the tile loop)
#pragma unroll
    for (int hh = 0; hh < QH; ++hh)
#pragma unroll
      for (int c = 0; c < 5; ++c) asm volatile("" : "+v"(qf[hh][c]));
    wait_vm4<0>();
    if (n > 1) issue(1, 1);
    lds_barrier4_first();
  }

  const int k_off = key_perm4(r32) * (D * 2) + g * 16;
  auto kread = [&](const char *ks, int st, bf16x8 *kf) {
    const char *row = ks + st * 32 * D * 2 + k_off;
#pragma unroll
    for (int c = 0; c < 4; ++c) kf[c] = *(const bf16x8 *)(row + c * 32);
    kf[4] = *(const bf16x8 *)(g ? ref_chunk : row + 128);
  };
  // V^T operands by transpose reads: within a 16-lane group w, lane j supplies
  // the address of a 4-dim chunk of key j / 4, and lane i receives dim i of
  // the four keys
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  const int tw = lane >> 4, tj = lane & 15;
  auto tr_pair = [&](const char *p0, const char *p1) {
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p0);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p1);
    const v8s both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  };
  const int v_off = (((tj >> 2) + (tw >> 1) * 8) * D + 16 * (tw & 1) + 4 * (tj & 3)) * 2;
  const int w_off = (((tj >> 2) + (tw & 1) * 16 + (tw >> 1) * 8) * D + 64 + 4 * (tj & 3)) * 2;
  const bool w_pad = (tj & 3) >= 2;
  const char *w_const = (tj & 3) == 2 ? ones_chunk : zero_chunk;
  // k = 0..3: dims 32 (k % 2) .. +31 of keys 16 (k / 2) + 8 g ..; k = 4: dims 64..79 of the 32 keys
  auto vfrag = [&](const char *vs, int st, int k) {
    if (k < 4) {
      const char *p0 = vs + v_off + ((st * 32 + (k >> 1) * 16) * D + (k & 1) * 32) * 2;
      return tr_pair(p0, p0 + 4 * D * 2);
    }
    const char *p0 = vs + w_off + st * 32 * D * 2;
    return tr_pair(w_pad ? w_const : p0, w_pad ? w_const : p0 + 4 * D * 2);
  };
  const f32x16 zero16 = {};
  auto score1 = [&](const bf16x8 *kf, int hh, int c, f32x16 &s) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c], qf[hh][c], c == 0 ? zero16 : s, 0, 0, 0);
  };

  f32x16 o[QH][2];  // dims 0..63
  f32x4 o2[QH][2];  // dims 64..71, the denominator (row 72) and seven unused rows, queries 0..15 and 16..31
  // Softmax reference: 0 at first.  A workgroup whose denominators leave
  // [2^-40, 2^80], or whose sums overflow, takes its maxima over all its keys
  // as the references (exactly: three bf16 parts in the padded query dims) and
  // starts again.
  float m_ref[QH];
#pragma unroll
  for (int hh = 0; hh < QH; ++hh) m_ref[hh] = 0.0f;
  bool again = false;
  for (;;) {
    if (again) {
      // (bases of its own: the compiler would compute this path's addresses
      // ahead of the outer loop, 140 scalar instructions and 49 spilled scalars)
      const char *keys = Kg, *values = Vg;
      asm volatile("" : "+s"(keys), "+s"(values));
#pragma unroll
      for (int hh = 0; hh < QH; ++hh) m_ref[hh] = -INFINITY;
#pragma nounroll
      for (int i = 0; i < n; ++i) {
        issue_from(keys, values, 0, i);
        wait_vm4<0>();
        lds_barrier4();
        for (int st = 0; st < 2; ++st) {
          bf16x8 kf[5];
          kread(lds, st, kf);
#pragma unroll
          for (int hh = 0; hh < QH; ++hh) {
            f32x16 s;
#pragma unroll
            for (int c = 0; c < 5; ++c) score1(kf, hh, c, s);
#pragma unroll
            for (int e = 0; e < 16; ++e) m_ref[hh] = fmaxf(m_ref[hh], s[e]);
          }
        }
        __syncthreads();
      }
#pragma unroll
      for (int hh = 0; hh < QH; ++hh) {
        const float m = half_swap_max(m_ref[hh]);
        m_ref[hh] = m == -INFINITY ? 0.0f : m;
        const float hi = (float)(bf16)m_ref[hh], mid = (float)(bf16)(m_ref[hh] - hi);
        if (g) {
          qf[hh][4][0] = (bf16)-hi;
          qf[hh][4][1] = (bf16)-mid;
          qf[hh][4][2] = (bf16)-(m_ref[hh] - hi - mid);
        }
      }
#pragma nounroll
      for (int i = 0; i < min(n, STAGES - 1); ++i) issue_from(keys, values, i, i);
      wait_vm4<0>();
      lds_barrier4();
    }
#pragma unroll
    for (int hh = 0; hh < QH; ++hh)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        o[hh][t] = zero16;
        o2[hh][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    // A tile is worked off in units of 32 queries x 32 keys, two at a time:
    // the scores of unit 0; the scores of unit 1 with the exponentials of
    // unit 0; PV of unit 0 with the exponentials of unit 1; PV of unit 1.
    // QH = 2: the units are the wave's two query halves on one key sub-tile;
    // QH = 1: the two key sub-tiles.
    constexpr int NK = QH == 2 ? 1 : 2;  // key sub-tiles per pair of units
    int slot = 0;
    bf16x8 kf[NK][5];
#pragma unroll
    for (int q = 0; q < NK; ++q) kread(lds, q, kf[q]);
    for (int i = 0; i < n; ++i) {
      const char *ks = lds + slot * STAGE, *vs = ks + KT_BYTES;
      slot = slot == STAGES - 1 ? 0 : slot + 1;
#pragma unroll
      for (int st = 0; st < 2; st += NK) {
        f32x16 s[2];
        bf16x8 vf[NK][5];
        float pe[2][16];
        bf16x8 pf[2][2];
        auto exps = [&](int u, int e0, int e1) {  // pinned to their place between the MFMAs
#pragma unroll
          for (int e = e0; e < e1; ++e) {
            float x = s[u][e];
            asm volatile("" : "+v"(x));
            pe[u][e] = __builtin_amdgcn_exp2f(x);
          }
        };
        auto cvt = [&](int u, int c) {
#pragma unroll
          for (int k = 0; k < 8; ++k) pf[u][c][k] = (bf16)pe[u][c * 8 + k];
        };
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            score1(kf[u % NK], u % QH, c, s[u]);
            if (u < NK) vf[u][c] = vfrag(vs, st + u, c);
            if (u == 1 && c > 0) exps(0, 4 * (c - 1), 4 * c);
            __builtin_amdgcn_sched_barrier(0);
          }
        cvt(0, 0);
        cvt(0, 1);
        asm volatile("" : "+v"(pf[0][0]), "+v"(pf[0][1]));  // (not to be moved past the branch)
        if (st + NK == 2 && i + 1 < n) {
          wait_tiles(min(n - 2 - i, STAGES - 3));
          lds_barrier4();
          if (i + STAGES - 1 < n) issue(slot < 2 ? slot + STAGES - 2 : slot - 2, i + STAGES - 1);
        }
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int hh = u % QH;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            o[hh][k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u % NK][k], pf[u][k >> 1], o[hh][k & 1], 0, 0, 0);
            if (u == 0) exps(1, 3 * k, 3 * k + 3);
            if (u == 0 && k == 3) cvt(1, 0);
            if (u == 1 && k == 0 && (st + NK < 2 || i + 1 < n)) {
#pragma unroll
              for (int q = 0; q < NK; ++q)
                kread(st + NK < 2 ? ks : lds + slot * STAGE, st + NK < 2 ? st + NK + q : q, kf[q]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          // dims 64..79: the probabilities of queries 0..15 and 16..31 as
          // operands of 32 keys (rows of 16 lanes exchanged between the two)
          bf16x8 pq[2];
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const auto r = __builtin_amdgcn_permlane16_swap(((const unsigned *)&pf[u][0])[w], ((const unsigned *)&pf[u][1])[w],
                                                            false, false);
            ((unsigned *)&pq[0])[w] = r[0];
            ((unsigned *)&pq[1])[w] = r[1];
          }
#pragma unroll
          for (int q = 0; q < 2; ++q)
            o2[hh][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[u % NK][4], pq[q], o2[hh][q], 0, 0, 0);
          if (u == 0) {
            exps(1, 12, 16);
            cvt(1, 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (again) break;
    bool bad = false;
    float nan0 = 0.0f;  // 0, or NaN if a sum is not finite
#pragma unroll
    for (int hh = 0; hh < QH; ++hh)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        bad = bad || (tw == 2 && !(o2[hh][q][0] < 0x1p80f && o2[hh][q][0] > 0x1p-40f));
#pragma unroll
        for (int e = 0; e < 16; ++e) nan0 = __builtin_fmaf(o[hh][q][e], 0.0f, nan0);
#pragma unroll
        for (int e = 0; e < 4; ++e) nan0 = __builtin_fmaf(o2[hh][q][e], 0.0f, nan0);
      }
    if (__any(bad || nan0 != 0.0f) && lane == 0) *flag = 1;
    __syncthreads();
    if (!*flag) break;
    again = true;
  }

#pragma unroll
  for (int hh = 0; hh < QH; ++hh) {
    // the denominators: row 72 is row 8 of the last block, lanes 32..47
    const float l0 = __shfl(o2[hh][0][0], 32 + tj, 64), l1 = __shfl(o2[hh][1][0], 32 + tj, 64);
    const float l_tot = (r32 >> 4) ? l1 : l0, inv = 1.0f / l_tot;
    const int q_base = q0 + wave * WQ + hh * 32, my_q = q_base + r32;
    bf16 *out = (a.splits == 1 ? (bf16 *)a.O : (bf16 *)a.Opart + (size_t)split * a.total_rows * a.hidden) + h * D;
    auto put = [&](int q, int d, float v0, float v1, float v2, float v3) {
      bf16x4 v;
      v[0] = (bf16)v0; v[1] = (bf16)v1; v[2] = (bf16)v2; v[3] = (bf16)v3;
      *(bf16x4 *)(out + (size_t)q * a.hidden + d) = v;
    };
    if (my_q < r1) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          put(my_q, t * 32 + i * 8 + g * 4, o[hh][t][i * 4] * inv, o[hh][t][i * 4 + 1] * inv, o[hh][t][i * 4 + 2] * inv,
              o[hh][t][i * 4 + 3] * inv);
    }
    if (tw < 2) {
      const float i0 = 1.0f / l0, i1 = 1.0f / l1;
      if (q_base + tj < r1)
        put(q_base + tj, 64 + tw * 4, o2[hh][0][0] * i0, o2[hh][0][1] * i0, o2[hh][0][2] * i0, o2[hh][0][3] * i0);
      if (q_base + 16 + tj < r1)
        put(q_base + 16 + tj, 64 + tw * 4, o2[hh][1][0] * i1, o2[hh][1][1] * i1, o2[hh][1][2] * i1, o2[hh][1][3] * i1);
    }
    if (my_q >= r1) continue;
    if (a.splits > 1 && g == 0) {
      // (relative to 0 the denominator's power of two goes into the reference,
      // so that the combine's weights, like the probabilities, stay near 1)
      float *ml = a.ML + (((size_t)split * a.total_rows + my_q) * heads + h) * 2;
      ml[0] = again ? m_ref[hh] : (float)__builtin_amdgcn_frexp_expf(l_tot);
      ml[1] = again ? l_tot : __builtin_amdgcn_frexp_mantf(l_tot);
    }
  }
}

// Combine of normalised bf16 split outputs: O = sum_s w_s O_s / sum_s w_s with
// w_s = 2^(m_s - max m) l_s, in split order.  One thread per (row, head,
// 8 dims); all loads are issued before use.
__global__ __launch_bounds__(64) void attn_combine_norm_kernel(const bf16 *Opart, const float *ML, bf16 *O, int R,
                                                                int heads, int splits) {
  constexpr int G = kHeadDim / 8;
  const int C = heads * kHeadDim;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)R * heads * G) return;
  const int r = idx / (heads * G);
  const int rem = idx - (long)r * heads * G;
  const int h = rem / G, d = (rem - h * G) * 8;
  constexpr int SMAX = 16;
  float2 ml[SMAX];
  bf16x8 p[SMAX];
#pragma unroll
  for (int s = 0; s < SMAX; ++s)
    if (s < splits) {
      ml[s] = *(const float2 *)(ML + (((size_t)s * R + r) * heads + h) * 2);
      p[s] = *(const bf16x8 *)(Opart + ((size_t)s * R + r) * C + h * kHeadDim + d);
    }
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < SMAX; ++s)
    if (s < splits) M = fmaxf(M, ml[s].x);
  float num[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f}, den = 0.0f;
#pragma unroll
  for (int s = 0; s < SMAX; ++s)
    if (s < splits) {
      const float w = exp2f(ml[s].x - M) * ml[s].y;
#pragma unroll
      for (int k = 0; k < 8; ++k) num[k] += w * (float)p[s][k];
      den += w;
    }
  const float inv = 1.0f / den;
  bf16x8 v;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = (bf16)(num[k] * inv);
  *(bf16x8 *)(O + (size_t)r * C + h * kHeadDim + d) = v;
}

hipError_t launch_attn_combine_norm(const void *Opart, const float *ML, void *O, int R, int heads, int splits,
                                    hipStream_t s) {
  if (R <= 0) return hipSuccess;
  if (splits < 1 || splits > 16) return hipErrorInvalidValue;
  const long n = (long)R * heads * (kHeadDim / 8);
  rc_launch(attn_combine_norm_kernel, dim3((n + 63) / 64), dim3(64), 0, s, (const bf16 *)Opart, ML, (bf16 *)O, R,
            heads, splits);
  return hipGetLastError();
}

// Query halves per wave and key splits: the pair with the least estimated
// time.  A tile of 64 keys takes a CU's two workgroups 1.07 us at QH = 1 and
// 1.85 at QH = 2, a lone workgroup about 0.65 of that; the ends (first tile,
// stores) take 6.5 and 9 us; a combine 4 us and its bytes at about 4 TB/s.
// These were fitted before the tile copies lost their branches, which took
// about 6 % off QH = 1 and 1 % off QH = 2, so near the line QH = 2 is taken
// where QH = 1 has become as fast or a little faster (best of each with its
// combine, us, launches included): 723 queries of 4096 keys 29.3 (QH = 1, five
// splits) and 30.8; 1639 in one chain 45.0 (two) and 47.6, 48.4 as planned; in
// four chains 49.0 and 49.6, 50.1 as planned; 2458 67.0 and 62.2; 4096 81.6 and
// 81.8; 1639 of 16384 141 and 137, 16384 of 16384 1192 and 1047.
AttnPlan plan_attention(const int *counts, int n_chains, int heads, int n_keys, long max_split_rows) {
  const int n_tiles = n_keys / A4_BK;
  long rows = 0;
  for (int b = 0; b < n_chains; ++b) rows += counts[b];
  AttnPlan best{1, 1};
  double best_us = 1e30;
  for (int qh = 1; qh <= 2; ++qh) {
    long qtiles = 0;
    for (int b = 0; b < n_chains; ++b) qtiles += (counts[b] + 128 * qh - 1) / (128 * qh);
    for (int sp = 1; sp <= std::min(n_tiles, 16) && (sp == 1 || rows * sp <= max_split_rows); ++sp) {
      const double wgs = (double)qtiles * heads * sp, rounds = wgs <= 256 ? 0.65 : std::ceil(wgs / 512);
      const double us = (qh == 1 ? 6.5 : 9.0) + rounds * ((n_tiles + sp - 1) / sp) * (qh == 1 ? 1.07 : 1.85) +
                        (sp > 1 ? 4.0 + rows * heads * kHeadDim * 2.0 * (sp + 1) / 4e6 : 0.0);
      if (us < best_us) {
        best_us = us;
        best = AttnPlan{qh, sp};
      }
    }
  }
  return best;
}

hipError_t launch_attention4(const AttnArgs &a, int n_chains, int max_rows, int qh, hipStream_t s) {
  if (max_rows <= 0) return hipSuccess;
  if (a.n_keys % A4_BK != 0 || a.splits < 1 || a.splits > a.n_keys / A4_BK || !a.v_rowmajor || qh < 1 || qh > 2)
    return hipErrorInvalidValue;
  dim3 grid((max_rows + 128 * qh - 1) / (128 * qh), (a.hidden / kHeadDim) * a.splits, n_chains);
  const bool warm = a.warm && a.warm_lines > 0;
  if (qh == 2) {
    if (warm) rc_launch(attn4_kernel<2, true>, grid, dim3(256), 0, s, a);
    else rc_launch(attn4_kernel<2, false>, grid, dim3(256), 0, s, a);
  } else {
    if (warm) rc_launch(attn4_kernel<1, true>, grid, dim3(256), 0, s, a);
    else rc_launch(attn4_kernel<1, false>, grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace rc
