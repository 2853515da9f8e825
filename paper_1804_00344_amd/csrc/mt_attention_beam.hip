// Additive attention of several hypotheses per sentence (K > 1), as two kernels that share the
// sentence's keys and context over its hypotheses:
//   scores   e[m, i] = sum_a va[a] * tanh(P[b,i,a] + q[m,a])   at the valid positions i
//   context  alpha = masked softmax of e, c[m] = sum_i alpha_i Cx[b,i,:]
//
// One workgroup per row (mt_attention.hip) pays two transcendentals per key element and row, and
// its time is that of the compute unit that received the longest sentences: three rows of 80
// positions on one unit are 21 us of its 28 at 64 x 12.
//
// Scores: a workgroup takes up to four positions of a sentence and six of its hypotheses.  With
// c = 2 / ln 2, tanh(p + q) = 1 - 2 / (2^(pc) 2^(qc) + 1): the exponential of a key element is
// shared by the hypotheses and that of a query element by the positions, which leaves per element
// and hypothesis one FMA, and per two of them one reciprocal, v1/d1 + v2/d2 = (v1 d2 + v2 d1) /
// (d1 d2).  The products stay in range while |pc| and |qc| are at most kExpLim; a key vector
// or a query beyond it (wave-uniform, checked for each) is scored by the plain form.
// A wave holds 512 features (8 per lane) of every query; it reduces each hypothesis' sum within
// its 16-lane rows by DPP adds and leaves the four row totals in LDS, where the workgroup's waves
// are added once at the end.
//
// Context: a workgroup takes 256 columns of a sentence for all its hypotheses; its four waves
// split the valid positions, each loading a row's slice once and adding it into every
// hypothesis' sum, and the waves are added through LDS.
//
// Bound by the transcendental and vector instructions of the scores.  Both kernels together
// against one workgroup per row (A = C = 2048, kernel trace): bf16 64 x 12, lengths of mean 25,
// longest 80: 27.9 -> 26.3 us; 128 x 5, mean 30, longest 100: 32.7 -> 27.3; fp32 64 x 12 36.9 ->
// 27.5; fp32 8 x 5, longest 60: 21.4 -> 11.0; bf16 one sentence of 25, beam 5: 12.3 -> 8.9.
#include "mt_internal.h"

namespace mt {

constexpr float kC2 = 2.8853900817779268f;  // 2 / ln 2
constexpr float kExpLim = 30.f;
constexpr int kScoreSlots = 4;  // positions of a workgroup at most
constexpr int kCtxCols = 256;
constexpr int kScoreMaxS = 1024;

typedef uint32_t v4q __attribute__((ext_vector_type(4)));

// eight consecutive elements of a row: one or two 16-byte loads, widened to fp32
template <typename T>
struct Oct {
  static constexpr int NV = (int)sizeof(T) / 2;
  v4q r[NV];
  __device__ __forceinline__ void load(const T *p) {
#pragma unroll
    for (int v = 0; v < NV; ++v) r[v] = ((const v4q *)p)[v];
  }
  __device__ __forceinline__ void get(float (&x)[8]) const {
    if constexpr (NV == 2) {
      __builtin_memcpy(x, r, 32);
    } else {
      bf16x8 h;
      __builtin_memcpy(&h, r, 16);
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (float)h[j];
    }
  }
};

// sum over each 16-lane row, in every lane of the row (bound_ctrl set, though every lane has a
// source: the compiler then folds the move into the add)
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_sum16(float v) {
  v = dpp_add<kDppQuadSwap1>(v);
  v = dpp_add<kDppQuadSwap2>(v);
  v = dpp_add<kDppRowRor4>(v);
  return dpp_add<kDppRowRor8>(v);
}

// grid (tiles of PT <= kScoreSlots positions x hypothesis groups, B), 64 * ceil(A / 512) threads; group g holds
// hypotheses g * kn .. of the sentence (kn <= KB each)
template <typename T, int KB>
__global__ __launch_bounds__(512) void attn_score_kernel(int K, int S, int A, int PT, int kn, const T *__restrict__ P,
                                                         const float *__restrict__ mask, const float *__restrict__ q,
                                                         int ldq, const float *__restrict__ va,
                                                         float *__restrict__ sc) {
  __shared__ float part[8][kScoreSlots][64];  // [wave][position][16-lane row * 16 + hypothesis]
  __shared__ float vpart[8];
  const int b = blockIdx.y;
  const int ng = (K + kn - 1) / kn;
  const int tile = blockIdx.x / ng, k0 = (blockIdx.x % ng) * kn;
  const int nk = K - k0 < kn ? K - k0 : kn;
  const int i0 = tile * PT;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), nw = blockDim.x >> 6;
  // the tile's valid positions
  const float mk = lane < PT && i0 + lane < S ? mask[(size_t)b * S + i0 + lane] : 0.f;
  const int f = wave * 512 + lane * 8;
  const bool on = f < A;
  const int fc = on ? f : A - 8;  // lanes past A: in range, with zero weight
  const T *const Pb = P + (size_t)b * S * A + fc;
  Oct<T> ring[2];
  ring[0].load(Pb + (size_t)i0 * A);
  ring[1].load(Pb + (size_t)(i0 + 1 < S ? i0 + 1 : S - 1) * A);
  const unsigned long long bits = __ballot(mk != 0.f);
  if (bits == 0) return;
  const int last = 63 - __builtin_clzll(bits);

  float vr[8], eq[KB][8];
  float vs = 0.f, qmax = 0.f;
  {
    Oct<float> o;
    o.load(va + fc);
    o.get(vr);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      vs += on ? vr[e] : 0.f;
      vr[e] = on ? -2.0f * vr[e] : 0.f;
    }
  }
  const float *const qb = q + (size_t)(b * K + k0) * ldq + fc;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    Oct<float> o;
    o.load(qb + (size_t)(k < nk ? k : 0) * ldq);
    o.get(eq[k]);
  }
#pragma unroll
  for (int k = 0; k < KB; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = eq[k][e] * kC2;
      qmax = fmaxf(qmax, fabsf(x));
      eq[k][e] = __builtin_amdgcn_exp2f(x);
    }
  // an infinity is out of range here and below, as is a finite value past the limit (the plain form);
  // the maxima pass over a NaN, which makes the sum NaN in either form
  const bool qok = __ballot(!(qmax <= kExpLim)) == 0;
  vs = wave_sum(vs);
  if (lane == 0) vpart[wave] = vs;

  auto score = [&](int p, const Oct<T> &raw) {
    float x[8], hi = 0.f;
    raw.get(x);
#pragma unroll
    for (int e = 0; e < 8; ++e) hi = fmaxf(hi, fabsf(x[e]));
    float tot = 0.f;  // lane r * 16 + k: hypothesis k's sum over 16-lane row r
    if (qok && __ballot(!(hi <= kExpLim / kC2)) == 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = __builtin_amdgcn_exp2f(x[e] * kC2);
#pragma unroll
      for (int k = 0; k < KB; ++k) {  // past nk: computed and not used
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float d0 = __builtin_fmaf(x[e], eq[k][e], 1.0f), d1 = __builtin_fmaf(x[e + 1], eq[k][e + 1], 1.0f);
          const float num = __builtin_fmaf(vr[e + 1], d0, vr[e] * d1);
          acc = __builtin_fmaf(num, rcp_fast(d0 * d1), acc);
        }
        acc = row_sum16(acc);
        tot = (lane & 15) == k ? acc : tot;
      }
    } else {
      for (int k = 0; k < nk; ++k) {
        float acc = 0.f, qv[8];
        Oct<float> o;
        o.load(qb + (size_t)k * ldq);
        o.get(qv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], kC2, qv[e] * kC2)) + 1.0f;
          acc = __builtin_fmaf(vr[e], rcp_fast(d), acc);
        }
        acc = row_sum16(acc);
        tot = (lane & 15) == k ? acc : tot;
      }
    }
    part[wave][p][lane] = tot;
  };
  // rows in order through a two-deep ring; a masked row is loaded (in bounds) and left out
  for (int p = 0; p <= last; p += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (p + d > last) break;
      if ((bits >> (p + d)) & 1) score(p + d, ring[d]);
      const int nx = i0 + p + d + 2;
      ring[d].load(Pb + (size_t)(nx < S ? nx : S - 1) * A);
    }
  }
  __syncthreads();
  float vsum = 0.f;
  for (int w = 0; w < nw; ++w) vsum += vpart[w];
  for (int idx = t; idx < (last + 1) * nk; idx += blockDim.x) {
    const int p = idx / nk, k = idx % nk;
    if (!((bits >> p) & 1)) continue;
    float s = 0.f;
    for (int w = 0; w < nw; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += part[w][p][r * 16 + k];
    sc[(size_t)(b * K + k0 + k) * S + i0 + p] = vsum + s;
  }
}

// four consecutive elements of a context row
template <typename T>
struct Quad;
template <>
struct Quad<float> {
  float4 r;
  __device__ __forceinline__ void load(const float *p) { r = *(const float4 *)p; }
  __device__ __forceinline__ void get(float (&x)[4]) const { x[0] = r.x; x[1] = r.y; x[2] = r.z; x[3] = r.w; }
};
template <>
struct Quad<bf16> {
  uint2 r;
  __device__ __forceinline__ void load(const bf16 *p) { r = *(const uint2 *)p; }
  __device__ __forceinline__ void get(float (&x)[4]) const {
    x[0] = __uint_as_float(r.x << 16); x[1] = __uint_as_float(r.x & 0xffff0000u);
    x[2] = __uint_as_float(r.y << 16); x[3] = __uint_as_float(r.y & 0xffff0000u);
  }
};

// grid (column slices, B), 256 threads; dynamic LDS: max(S * KP, 3 * KB * kCtxCols) floats, KP =
// KB rounded up to a multiple of 4; S <= 64 * NS
template <typename T, int KB, int NS>
__global__ __launch_bounds__(256) void attn_context_kernel(int K, int S, int Cd, const T *__restrict__ Cx,
                                                           const float *__restrict__ mask,
                                                           const float *__restrict__ sc, float *__restrict__ ctx_out,
                                                           int ldc, bf16 *__restrict__ ctx16, int ld16,
                                                           float *__restrict__ alpha_out) {
  constexpr int KP = (KB + 3) / 4 * 4;
  constexpr int U = 4;  // rows in flight per wave
  extern __shared__ __attribute__((aligned(16))) float lds[];
  __shared__ unsigned long long words[NS];  // the valid positions
  float *const al = lds;                    // [S][KP]
  const int b = blockIdx.y;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // ---- requested together: the mask, the scores of the rows k = wave, wave + 4, .., and the
  // first context rows of this wave's positions wave, wave + 4, .. ----
  float mk[NS], row[KP / 4][NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = 64 * s + lane;
    mk[s] = i < S ? mask[(size_t)b * S + i] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < KP / 4; ++r) {
    const int k = wave + 4 * r;
    const float *const rp = sc + (size_t)(b * K + (k < K ? k : 0)) * S;
#pragma unroll
    for (int s = 0; s < NS; ++s) row[r][s] = 64 * s + lane < S ? rp[64 * s + lane] : 0.f;
  }
  const int col = blockIdx.x * kCtxCols + lane * 4;
  const int cc = col < Cd ? col : Cd - 4;
  const T *const Cb = Cx + (size_t)b * S * Cd + cc;
  Quad<T> ring[U];
  auto fetch = [&](int i, Quad<T> &r) { r.load(Cb + (size_t)(i < S ? i : S - 1) * Cd); };  // in bounds; masked rows are left out
#pragma unroll
  for (int u = 0; u < U; ++u) fetch(wave + 4 * u, ring[u]);
  // ---- masked softmax; weights of masked positions are 0 ----
#pragma unroll
  for (int r = 0; r < KP / 4; ++r) {
    const int k = wave + 4 * r;
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < NS; ++s) mx = mk[s] != 0.f ? fmaxf(mx, row[r][s]) : mx;
    mx = wave_max(mx);
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      row[r][s] = mk[s] != 0.f ? exp_fast(row[r][s] - mx) : 0.f;
      sum += row[r][s];
    }
    sum = wave_sum(sum);
    const float inv = sum > 0.f ? 1.0f / sum : 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = 64 * s + lane;
      if (i >= S) continue;
      const float a = k < K ? row[r][s] * inv : 0.f;
      al[i * KP + k] = a;
      if (alpha_out && blockIdx.x == 0 && k < K) alpha_out[(size_t)(b * K + k) * S + i] = a;
    }
  }
  int last = -1;  // the last valid position
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const unsigned long long w = __ballot(mk[s] != 0.f);
    if (w) last = 64 * s + 63 - __builtin_clzll(w);
    if (wave == 0 && lane == 0) words[s] = w;
  }
  __syncthreads();

  float acc[KB][4];
#pragma unroll
  for (int k = 0; k < KB; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[k][e] = 0.f;
  for (int i0 = wave; i0 <= last; i0 += 4 * U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 4 * u;
      if (i <= last && ((words[NS == 1 ? 0 : i >> 6] >> (i & 63)) & 1)) {  // wave-uniform
        float x[4], a[KP];
        ring[u].get(x);
#pragma unroll
        for (int k = 0; k < KP; k += 4) *(float4 *)(a + k) = *(const float4 *)(al + i * KP + k);
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[k][e] = __builtin_fmaf(a[k], x[e], acc[k][e]);
      }
      fetch(i + 4 * U, ring[u]);
    }
  }
  __syncthreads();  // the weights are no longer read
  float *const red = lds;  // [wave - 1][hypothesis][column]
  if (wave > 0) {
#pragma unroll
    for (int k = 0; k < KB; ++k)
      *(float4 *)(red + ((wave - 1) * KB + k) * kCtxCols + lane * 4) = make_float4(acc[k][0], acc[k][1], acc[k][2], acc[k][3]);
  }
  __syncthreads();
  if (wave == 0 && col < Cd) {
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k >= K) continue;
      float4 v = make_float4(acc[k][0], acc[k][1], acc[k][2], acc[k][3]);
#pragma unroll
      for (int w = 0; w < 3; ++w) {
        const float4 o = *(const float4 *)(red + (w * KB + k) * kCtxCols + lane * 4);
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
      }
      const size_t m = (size_t)b * K + k;
      if (ctx_out) *(float4 *)(ctx_out + m * ldc + col) = v;
      if (ctx16) {
        const bf16 h[4] = {to_bf16(v.x), to_bf16(v.y), to_bf16(v.z), to_bf16(v.w)};
        __builtin_memcpy(ctx16 + m * ld16 + col, h, 8);
      }
    }
  }
}

template <typename T, int KB>
static void score_go(int B, int K, int S, int A, int PT, int kn, const T *P, const float *mask, const float *q, int ldq,
                     const float *va, float *sc, hipStream_t st) {
  const dim3 grid((unsigned)((S + PT - 1) / PT * ((K + kn - 1) / kn)), (unsigned)B);
  hipLaunchKernelGGL((attn_score_kernel<T, KB>), grid, dim3(64 * ((A + 511) / 512)), 0, st, K, S, A, PT, kn, P, mask, q,
                     ldq, va, sc);
}

template <typename T, int KB>
static void context_go(int B, int K, int S, int Cd, const T *Cx, const float *mask, const float *sc, float *ctx_out,
                       int ldc, bf16 *ctx16, int ld16, float *alpha_out, hipStream_t st) {
  constexpr int KP = (KB + 3) / 4 * 4;
  const int a = S * KP, r = 3 * KB * kCtxCols;
  const size_t lds = (size_t)(a > r ? a : r) * 4;
  const dim3 grid((unsigned)((Cd + kCtxCols - 1) / kCtxCols), (unsigned)B);
#define MT_CN(NS)                                                                                                 \
  hipLaunchKernelGGL((attn_context_kernel<T, KB, NS>), grid, dim3(256), lds, st, K, S, Cd, Cx, mask, sc, ctx_out, ldc, \
                     ctx16, ld16, alpha_out)
  if (S <= 64) MT_CN(1);
  else if (S <= 128) MT_CN(2);
  else if (S <= 256) MT_CN(4);
  else MT_CN(16);
#undef MT_CN
}

template <typename T>
static hipError_t beam_go(int B, int K, int S, int A, int Cd, const T *P, const T *Cx, const float *mask, const float *q,
                          int ldq, const float *va, float *ctx_out, int ldc, bf16 *ctx16, int ld16, float *alpha_out,
                          float *sc, hipStream_t st) {
  // Positions and hypotheses per workgroup.  us of the score kernel at bf16, A = 2048, for 1, 2, 4
  // and 8 positions: 64 x 12 (length mean 25, longest 80) with 12 hypotheses 23.7 18.2 17.6 19.4,
  // with 6 23.1 16.8 15.5 15.4, with 4 24.0 17.7 16.6 18.4; 128 x 5 (mean 30, longest 100) with 5
  // 22.6 16.6 16.3 18.1; 8 x 5 (mean 25, longest 60) with 5 4.7 4.5 5.6 7.9: more of either shares
  // the exponentials further, fewer leave more waves to cover the latency and even out the units.
  // One position up to 1280 padded ones (the valid ones are not known on the host), four from 5120.
  const long pt = (long)B * S / 1280;
  const int PT = pt < 1 ? 1 : pt > kScoreSlots ? kScoreSlots : (int)pt;
  const int ng = (K + 5) / 6, kn = (K + ng - 1) / ng;
#define MT_SC(KB) score_go<T, KB>(B, K, S, A, PT, kn, P, mask, q, ldq, va, sc, st)
  if (kn <= 2) MT_SC(2);
  else if (kn <= 3) MT_SC(3);
  else if (kn <= 4) MT_SC(4);
  else if (kn <= 5) MT_SC(5);
  else MT_SC(6);
#undef MT_SC
#define MT_CX(KB) context_go<T, KB>(B, K, S, Cd, Cx, mask, sc, ctx_out, ldc, ctx16, ld16, alpha_out, st)
  if (K <= 4) MT_CX(4);
  else if (K <= 6) MT_CX(6);
  else if (K <= 8) MT_CX(8);
  else if (K <= 12) MT_CX(12);
  else MT_CX(16);
#undef MT_CX
  return hipGetLastError();
}

bool attention_beam_ok(int B, int K, int S, int A, int Cd) {
  // the softmax weights of the context kernel fit the 64 KiB of LDS a launch gets by default, and
  // the sentences a grid dimension
  return K <= kKMax && A <= 4096 && A % 8 == 0 && Cd % 4 == 0 && B <= 65535 && S <= kScoreMaxS && ((K + 3) / 4 * 4) * S * 4 <= 65536 - 256;
}

// Which sizes take it: enough positions to pay for the second launch and, with more rows, for the
// units that the row form then fills by itself.  Attention of a step in us between two events (about
// 5 of them are the events'), row form / beam form, mean length 0.4 S unless given, A = 2H; the first
// two lines lie on the beam form's side:
//   A = 2048, bf16: 1 x 5, S 25 15.2 / 11.3; 1 x 16, S 50 21.4 / 15.6; 64 x 12, S 80 31.4 / 30.9, S 160
//     53.8 / 46.4; fp32: 64 x 12, S 80 35.1 / 31.3
//   bf16: 1 x 5, S 10 10.9 / 11.1; 64 x 12, S 25 16.6 / 21.0, S 50 23.2 / 24.5; 256 x 2, S 50 21.9 / 25.4;
//     128 x 5, S 50 21.9 / 24.3; fp32: 128 x 2, all of length 80 31.1 / 37.0
//   A = 512: 1 x 5, length 25 10.4 / 11.3 (fp32); 64 x 16, S 80 21.1 / 26.1 (bf16)
// Of 5808 shapes (K 2..16, B 1..512, S 10..320, A 512..2048, lengths S or of mean 0.4 S, both types)
// 7 are slower than with the row form by more than 3%, by 11% (2 us) at most; with the beam form
// wherever it can run, 1713 were, by up to 57%.  Few hypotheses share few exponentials (K <= 3), and
// more than 12 take the context workgroups the longest; with fewer than 512 features a scoring wave
// has lanes without one (not measured).
bool attention_takes_beam(int B, int K, int S, int A, int Cd) {
  if (K < 2 || A < 512 || !attention_beam_ok(B, K, S, A, Cd)) return false;
  const double w = K <= 3 ? 4.0 : K > 12 ? 2.0 : 1.0;
  const double s = 12.0 + K + w * B * K / 14.0;  // positions at A = 2048; as 1 / sqrt(A) elsewhere
  return (double)S * S * A >= 2048.0 * s * s;
}

hipError_t launch_attention_beam(int B, int K, int S, int A, int Cd, const void *P, const void *Cx, int bf16_io,
                                 const float *mask, const float *q, int ldq, const float *va, float *ctx_out, int ldc,
                                 bf16 *ctx16, int ld16, float *alpha_out, float *sc, hipStream_t st) {
  if (!attention_beam_ok(B, K, S, A, Cd)) return hipErrorInvalidValue;
  if (bf16_io)
    return beam_go<bf16>(B, K, S, A, Cd, (const bf16 *)P, (const bf16 *)Cx, mask, q, ldq, va, ctx_out, ldc, ctx16, ld16,
                         alpha_out, sc, st);
  return beam_go<float>(B, K, S, A, Cd, (const float *)P, (const float *)Cx, mask, q, ldq, va, ctx_out, ldc, ctx16, ld16,
                        alpha_out, sc, st);
}

}  // namespace mt
