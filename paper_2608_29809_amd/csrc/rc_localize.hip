// Edit-region localisation (Sec. 3.2): cross-attention maps of the delta text
// tokens aggregated over heads and blocks, a per-token-map threshold derived
// from each map's range, union over delta tokens, grid dilation, and the
// stable compaction of the resulting mask into per-chain token lists.
#include "rc_common.h"
#include "rc_launch.h"
#include "rc_elem.h"

#include <climits>

namespace rc {

constexpr int LG_TOK = 16;  // tokens per workgroup, 4 per wave
constexpr int LG_HC = 4;    // heads whose rows a wave loads at once

// Max over the 16 lanes of a DPP row (the steps of row16_sum).
// IEEE maximum (NaN-propagating): one v_maximum3/v_maximum on gfx950, with
// no operand canonicalisation as fmaxf needs.
__device__ __forceinline__ float fmax_(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float row16_max(float v) {
  v = fmax_(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmax_(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmax_(v, dpp_mov<0x141>(v));  // row_half_mirror
  return fmax_(v, dpp_mov<0x140>(v));  // row_mirror
}

// partial[l][tok][j] = sum_h softmax(Z[l][h][tok][:])[delta_j].  One
// workgroup per (16-token tile, layer), each wave 4 tokens.  A row of the
// logits (text_len <= 128 bf16, 16-byte chunks) is spread over one 16-lane
// group (one token per group), so one load instruction covers four
// consecutive rows -- contiguous memory -- and the row's max and sum are
// 16-lane DPP reductions.  A wave issues the rows of LG_HC heads before it
// reduces any (4 KB in flight per wave at 40 VGPRs, eight waves per SIMD).
// The exponent runs on the raw v_exp_f32: its argument z - max is <= 0, so a
// flushed denormal moves a row sum that is >= 1 by less than 2^-126, and the
// row's reciprocal is one v_rcp_f32 (1 ulp).  Lane j of a group owns delta
// column j: it re-reads that one logit (a cache hit) and accumulates its
// probability over the heads in order.
__global__ __launch_bounds__(256) void maps_from_logits_kernel(const uint16_t *Z, int heads, int tokens,
                                                               int text_len, MapsDelta dl, float *partial) {
  const int l = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = lane >> 4, j16 = lane & 15;
  const int tok = blockIdx.x * LG_TOK + wave * 4 + grp;  // this lane group's token
  const int row_vec = text_len / 8;                       // 16-byte chunks per row
  const bool ok = tok < tokens;
  const bool lane_on = j16 < row_vec && ok;
  const bool owner = j16 < dl.n && ok;
  int my_col = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j == j16) my_col = dl.col[j];
  constexpr float kLog2e = 1.4426950408889634f;
  float acc = 0.0f;
  for (int h0 = 0; h0 < heads; h0 += LG_HC) {
    V16 v[LG_HC];
    uint16_t zd[LG_HC];
#pragma unroll
    for (int c = 0; c < LG_HC; ++c) {
      const uint16_t *row = Z + ((size_t)(l * heads + h0 + c) * tokens + tok) * text_len;
      const bool on = h0 + c < heads;
      v[c] = V16{{0u, 0u, 0u, 0u}};
      if (on && lane_on) v[c] = *(const V16 *)(row + j16 * 8);
      zd[c] = (on && owner) ? row[my_col] : (uint16_t)0;
    }
#pragma unroll
    for (int c = 0; c < LG_HC; ++c) {
      const bool on = h0 + c < heads;
      float z[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        z[2 * q] = __uint_as_float(v[c].w[q] << 16);
        z[2 * q + 1] = __uint_as_float(v[c].w[q] & 0xFFFF0000u);
      }
      float m = -INFINITY;
      if (on && lane_on)
        m = fmax_(fmax_(fmax_(z[0], z[1]), fmax_(z[2], z[3])), fmax_(fmax_(z[4], z[5]), fmax_(z[6], z[7])));
      m = row16_max(m);
      const float mc = m * kLog2e;
      float sum = 0.0f;
      if (on && lane_on)
#pragma unroll
        for (int q = 0; q < 8; ++q) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(z[q], kLog2e, -mc));
      sum = row16_sum(sum);
      if (on && owner)
        acc += __builtin_amdgcn_exp2f(__builtin_fmaf(__uint_as_float((uint32_t)zd[c] << 16), kLog2e, -mc)) *
               __builtin_amdgcn_rcpf(sum);
    }
  }
  if (owner) partial[((size_t)l * tokens + tok) * dl.n + j16] = acc;
}

hipError_t launch_maps_from_logits(const uint16_t *logits, int n_layers, int heads, int tokens, int text_len,
                                   const int *delta, int n_delta, float *partial, hipStream_t s) {
  if (text_len % 8 || text_len > 128 || n_delta < 1 || n_delta > 8) return hipErrorInvalidValue;
  MapsDelta dl;
  dl.n = n_delta;
  for (int j = 0; j < 8; ++j) dl.col[j] = j < n_delta ? delta[j] : 0;
  dim3 grid((tokens + LG_TOK - 1) / LG_TOK, n_layers);
  rc_launch(maps_from_logits_kernel, grid, dim3(256), 0, s, logits, heads, tokens, text_len, dl, partial);
  return hipGetLastError();
}

// out[i] = sum_p partial[p][i] in order p = 0, 1, ...  Latency-bound (2.8 MB
// for 28 layers of 4096 x 6): sixteen partials are in flight per thread.
__global__ __launch_bounds__(64) void sum_partials_kernel(const float *partial, int n_parts, int n, float *out) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= n) return;
  float s = 0.0f;
  constexpr int U = 16;
  for (int p0 = 0; p0 < n_parts; p0 += U) {
    float v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = partial[(size_t)min(p0 + k, n_parts - 1) * n + i];
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (p0 + k < n_parts) s += v[k];
  }
  out[i] = s;
}

hipError_t launch_sum_partials(const float *partial, int n_parts, int n, float *out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  rc_launch(sum_partials_kernel, dim3((n + 63) / 64), dim3(64), 0, s, partial, n_parts, n, out);
  return hipGetLastError();
}

// Stable compaction by a 1024-thread workgroup of up to 16 x 1024 tokens, of
// which this thread holds i0 + 1024 k + tid for k < nk (those below `end`),
// selected where bit k of `on` is set: their numbers go to idx[base ..] in
// ascending order.  One ballot per 64 tokens, one scan over the counts of all of
// them; returns the number selected.  cnt: [257] ints of LDS.
// STREAM: the tokens are chains of N laid end to end, numbered within each, and
// the chains that begin here get their offsets, from the last wave, whose lane l
// has chain l, l + 64, ... (b, first token at s) as its next.  word: [256]
// ballots of LDS.
template <bool STREAM>
__device__ __forceinline__ int compact_tokens(unsigned on, int nk, int i0, int base, int *idx, int *cnt, int end = 0,
                                              int N = 1, int *b = nullptr, unsigned *s = nullptr, int *offsets = nullptr,
                                              uint64_t *word = nullptr) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  __syncthreads();  // earlier readers of cnt are done
  for (int k = 0; k < nk; ++k) {
    const uint64_t bal = __ballot((on >> k) & 1u);
    if (lane == 0) {
      cnt[k * 16 + wave] = __popcll(bal);
      if (STREAM) word[k * 16 + wave] = bal;
    }
  }
  __syncthreads();
  if (wave == 0) {  // exclusive scan of nk * 16 <= 256 counts, four per lane
    int c[4], sum = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c[e] = lane * 4 + e < nk * 16 ? cnt[lane * 4 + e] : 0;
      sum += c[e];
    }
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    int pre = inc - sum;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      cnt[lane * 4 + e] = pre;
      pre += c[e];
    }
    if (lane == 63) cnt[256] = inc;
  }
  __syncthreads();
  const int step = STREAM ? 1024 % N : 1024;
  int tok = STREAM ? (i0 + tid) % N : i0 + tid;
  for (int k = 0; k < nk; ++k) {
    const bool sel = (on >> k) & 1u;
    const uint64_t bal = __ballot(sel);
    if (sel) idx[base + cnt[k * 16 + wave] + __popcll(bal & below)] = tok;
    tok += step;
    if (STREAM) tok -= tok >= N ? N : 0;
  }
  if (STREAM && wave == 15)
    for (; *s < (unsigned)(i0 + min(end - i0, nk * 1024)); *b += 64, *s += 64u * N) {
      const int r = (int)*s - i0;
      offsets[*b] = base + cnt[r >> 6] + __popcll(word[r >> 6] & ((1ull << (r & 63)) - 1));
    }
  return cnt[256];
}

__device__ __forceinline__ float row16_fmin(float v) {
  v = fminf(v, dpp_mov<0xB1>(v));
  v = fminf(v, dpp_mov<0x4E>(v));
  v = fminf(v, dpp_mov<0x141>(v));
  return fminf(v, dpp_mov<0x140>(v));
}

// One workgroup per chain: range of each delta map, threshold, union,
// dilation and, for a single chain (idx non-null), the compaction.
//
// Latency-bound (100 KB of maps at 64x64 tokens and six columns).  Every
// column's range comes from one pass: a thread loads all columns of four
// tokens before it uses any, and keeps them for the threshold where the chain
// has no more than 4096 tokens.  The selection is a bit per token (the
// ballots of the waves), so a token's neighbourhood is a shift of a word or
// two per row.  With a pass over memory for each column's range and
// another for its threshold the kernel took 25.8 us at 64x64 tokens and six
// columns, and the compaction another 4.7.  A small call pays for fetching code
// that runs once, so the column count ND is the kernel's: for all counts in one
// kernel a call with one column took 2 to 6 us more than those two passes on
// grids of up to 1024 tokens.
constexpr int kLocTok = 4;  // tokens of a thread loaded together
template <int ND>
__global__ __launch_bounds__(1024) void localize_kernel(const float *maps, int gh, int gw, float threshold, int radius,
                                                        uint8_t *mask, int *idx, int *offsets) {
  __shared__ uint64_t bits[258];       // selection of 64 tokens each, a spare word past the last
  __shared__ float red[2 * ND][64], range[2 * ND];  // per column 2 j: minimum, 2 j + 1: -maximum
  __shared__ int cnt[257];
  const int b = blockIdx.x, tid = threadIdx.x, N = gh * gw;
  const int lane = tid & 63, wave = tid >> 6;
  const float *m = maps + (size_t)b * N * ND;
  const int nk = (N + 1023) / 1024, n_chunk = (nk + kLocTok - 1) / kLocTok;
  float v[kLocTok][ND];
  auto load = [&](int c) {
#pragma unroll
    for (int k = 0; k < kLocTok; ++k) {
      const float *p = m + (size_t)min((c * kLocTok + k) * 1024 + tid, N - 1) * ND;
#pragma unroll
      for (int j = 0; j < ND; ++j) v[k][j] = p[j];
    }
  };
  float lo[ND], nhi[ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) lo[j] = nhi[j] = INFINITY;
  for (int c = 0; c < n_chunk; ++c) {
    load(c);
#pragma unroll
    for (int k = 0; k < kLocTok; ++k)  // (a token past the last is the last again)
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        lo[j] = fminf(lo[j], v[k][j]);
        nhi[j] = fminf(nhi[j], -v[k][j]);
      }
  }
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    lo[j] = row16_fmin(lo[j]);
    nhi[j] = row16_fmin(nhi[j]);
    if ((lane & 15) == 0) {
      red[2 * j][wave * 4 + (lane >> 4)] = lo[j];
      red[2 * j + 1][wave * 4 + (lane >> 4)] = nhi[j];
    }
  }
  __syncthreads();
  if (wave < 2 * ND) {
    float r = red[wave][lane];
    r = row16_fmin(r);
    r = fminf(r, __shfl_xor(r, 16, 64));
    r = fminf(r, __shfl_xor(r, 32, 64));
    if (lane == 0) range[wave] = r;
  }
  __syncthreads();
  unsigned live = 0;  // columns that select (a constant map selects nothing)
  float inv[ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    lo[j] = range[2 * j];
    const float hi = -range[2 * j + 1];
    live |= (unsigned)(hi > lo[j]) << j;
    inv[j] = 1.0f / (hi - lo[j]);
  }
  for (int c = 0; c < n_chunk; ++c) {
    if (n_chunk > 1) load(c);
#pragma unroll
    for (int k = 0; k < kLocTok; ++k) {
      const int i = (c * kLocTok + k) * 1024 + tid;
      bool on = false;
#pragma unroll
      for (int j = 0; j < ND; ++j) on = on || (((live >> j) & 1u) && (v[k][j] - lo[j]) * inv[j] >= threshold);
      const uint64_t bal = __ballot(on && i < N);
      if (lane == 0 && i < N) bits[i >> 6] = bal;
    }
  }
  if (tid == 0) bits[N >> 6] = 0;
  __syncthreads();
  unsigned sel = 0;
  for (int k = 0; k < nk; ++k) {
    const int i = k * 1024 + tid;
    if (i < N) {
      const int y = i / gw, x = i - y * gw;
      const int x0 = max(x - radius, 0), w = min(x + radius, gw - 1) - x0 + 1;
      const int y0 = max(y - radius, 0), y1 = min(y + radius, gh - 1);
      uint64_t any = 0;
      for (int yy = y0; yy <= y1; ++yy) {
        const int p = yy * gw + x0, sh = p & 63;
        uint64_t f = bits[p >> 6] >> sh;
        if (sh) f |= bits[(p >> 6) + 1] << (64 - sh);
        any |= f;
      }
      const unsigned on = (any & ((1ull << w) - 1)) != 0;
      sel |= on << k;
      mask[(size_t)b * N + i] = (uint8_t)on;
    }
  }
  if (idx) {
    const int total = compact_tokens<false>(sel, nk, 0, 0, idx, cnt);
    if (tid == 0) {
      offsets[0] = 0;
      offsets[1] = total;
    }
  }
}

hipError_t launch_localize(const float *maps, int B, int gh, int gw, int n_delta, float threshold, int radius,
                           uint8_t *mask, int *idx, int *offsets, hipStream_t s) {
  if ((long)gh * gw > 16384 || (gh * gw) % 64) return hipErrorInvalidValue;
  int *one = B == 1 ? idx : nullptr;
#define RC_LOC(ND) \
  case ND: rc_launch(localize_kernel<ND>, dim3(B), dim3(1024), 0, s, maps, gh, gw, threshold, radius, mask, one, offsets); break;
  switch (n_delta) {
    RC_LOC(1) RC_LOC(2) RC_LOC(3) RC_LOC(4) RC_LOC(5) RC_LOC(6) RC_LOC(7) RC_LOC(8)
    default: return hipErrorInvalidValue;
  }
#undef RC_LOC
  return B == 1 ? hipGetLastError() : launch_compact(mask, B, gh * gw, idx, offsets, s);
}

// Stable compaction over all chains by one workgroup, 16384 tokens at a time
// (every mask byte of them is loaded before the first is used).  STREAM: all
// chains as one sequence of B N tokens, a barrier and a scan per 16384 tokens;
// else chain by chain, which for short chains takes 1.4 us each: 443 us for 300
// chains of 64 tokens and 125 for 64 of 1024, as one sequence 72 and 60 (a loop
// over 1024 tokens of a chain at a time: 194 and 72).
template <bool STREAM>
__global__ __launch_bounds__(1024) void compact_kernel(const uint8_t *mask, int B, int N, int *idx, int *offsets) {
  __shared__ int cnt[257];
  __shared__ uint64_t word[STREAM ? 256 : 1];
  const int tid = threadIdx.x, end = STREAM ? B * N : N;  // (at most 32767 x 65535)
  int base = 0, b = tid & 63;
  unsigned s = (unsigned)b * N;
  for (int c = 0; c < (STREAM ? 1 : B); ++c) {
    if (!STREAM && tid == 0) offsets[c] = base;
    for (int i0 = 0;;) {
      const int nk = min(16, (end - i0 + 1023) / 1024);
      unsigned on = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int i = i0 + k * 1024 + tid;
        on |= (unsigned)(i < end && mask[(size_t)c * N + min(i, end - 1)] != 0) << k;
      }
      base += STREAM ? compact_tokens<true>(on, nk, i0, base, idx, cnt, end, N, &b, &s, offsets, word)
                     : compact_tokens<false>(on, nk, i0, base, idx, cnt);
      if (end - i0 <= 16384) break;  // (before i0 could overflow)
      i0 += 16384;
    }
  }
  if (tid == 0) offsets[B] = base;
}

// Validity of an active set (device offsets already checked equal to the
// host copy, so every chain's range lies inside idx[0, total)): the first
// position p, in index order, whose token is outside [0, N) or not larger
// than the token before it in the same chain; -1 if there is none.  One
// workgroup; each thread keeps its smallest bad position, then a fixed-order
// reduction; thread 0 writes the verdict.
__global__ __launch_bounds__(1024) void validate_active_kernel(const int *offsets, const int *idx, int B, int N,
                                                               int *verdict) {
  __shared__ int red[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int bad = INT_MAX;
  for (int b = 0; b < B; ++b) {
    const int lo = offsets[b], hi = offsets[b + 1];
    for (int i = lo + tid; i < hi; i += 1024) {
      const int v = idx[i];
      const bool ok = v >= 0 && v < N && (i == lo || idx[i - 1] < v);
      if (!ok) bad = min(bad, i);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bad = min(bad, __shfl_xor(bad, o, 64));
  if (lane == 0) red[wave] = bad;
  __syncthreads();
  if (tid == 0) {
    int m = red[0];
    for (int w = 1; w < 16; ++w) m = min(m, red[w]);
    verdict[0] = m == INT_MAX ? -1 : m;
  }
}

hipError_t launch_validate_active(const int *offsets, const int *idx, int B, int N, int *verdict, hipStream_t s) {
  rc_launch(validate_active_kernel, dim3(1), dim3(1024), 0, s, offsets, idx, B, N, verdict);
  return hipGetLastError();
}

hipError_t launch_compact(const uint8_t *mask, int B, int N, int *idx, int *offsets, hipStream_t s) {
  // one sequence unless a chain fills 16384 tokens by itself (localisation of 32
  // such chains 275 us one by one, 304 in one sequence) or is the only one
  // (65535 tokens: 48.7 and 51.9 us)
  if (B == 1 || N >= 16384) rc_launch(compact_kernel<false>, dim3(1), dim3(1024), 0, s, mask, B, N, idx, offsets);
  else rc_launch(compact_kernel<true>, dim3(1), dim3(1024), 0, s, mask, B, N, idx, offsets);
  return hipGetLastError();
}

}  // namespace rc
