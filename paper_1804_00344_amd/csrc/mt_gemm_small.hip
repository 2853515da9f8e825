// Matrix products of a few rows (small batches, the encoder's recurrence):
// out[m, n] = sum_k A[m, k] * W[k, n] (+ bias[n]) for M rows far below what fills the chip with
// output tiles.  The operands, packings and epilogues are those of mt_gemm.hip.
//
// What bounds such a product is the weight matrix, read once (6 MB to 29 MB a launch), and the
// latency of a workgroup's chain of loads.  Tiles of 64 x 128 outputs leave 24 to 40 workgroups
// whose two waves walk the whole depth alone.  Here one workgroup of eight waves owns one
// column block of the packed weights (16 or 32 columns) and 32 rows, and the waves split the
// k-steps in chunks of 64 k (four k-steps): the weights of a chunk go straight into registers, the
// activations through the wave's own part of LDS (no workgroup barrier), both requested one chunk
// ahead; then the eight partial tiles are added through LDS in wave order.  Row groups of 32 share
// a column block's weights in one XCD's L2.  5 rows of the bf16 step: 3072 x 1024 8.2 -> 4.4 us,
// 5120 x 1024 7.8 -> 4.5, 3584 x 2048 11.7 -> 5.5, 512 x 1024 7.4 -> 3.6; fp32 3584 x 2048 38.5 -> 7.9 us
// at 5 rows, 39.5 -> 17.4 at 64.  enc_step_kernel (mt_encoder.hip) splits the depth in the same way.
#include "mt_gemm_common.h"

namespace mt {

constexpr int kSmWaves = 8, kSmThreads = 64 * kSmWaves, kSmRows = 32;

// CB: columns of a workgroup's block; a chunk is 64 k
template <typename CT, typename AT, int CB>
struct SmForm {
  static constexpr int KSTEP = sizeof(CT) == 2 ? 16 : 256 / CB;   // k per MFMA operand vector
  static constexpr int KC = 64;                                   // k per chunk of a wave
  static constexpr int STEPS = KC / KSTEP;                        // k-steps of a chunk
  static constexpr int RB = kSmRows / CB;                         // row blocks
  static constexpr int NACC = CB * CB / 64;
  static constexpr int ROWB = KC * (int)sizeof(CT) + 16;          // padded LDS row of a chunk
};

// PK: columns per block of the packing.  An fp32 workgroup owns 16 columns in either packing: two
// 8-k steps of the 32-column form hold, for one half of the columns, the vectors of a 16-k step.
template <typename CT, typename AT, int PK, int EPI>
__global__ __launch_bounds__(kSmThreads, 4) void gemm_small_kernel(Problems probs) {
  constexpr int BLK = sizeof(CT) == 2 ? 32 : 16;
  using F = SmForm<CT, AT, BLK>;
  typedef __attribute__((__vector_size__(F::NACC * sizeof(float)))) float accv;
  constexpr int PER = F::RB * F::NACC * 64;         // outputs of a workgroup
  constexpr int STG = kSmRows * F::ROWB;            // a wave's LDS chunk
  constexpr int LDSB = STG > PER * 4 ? STG : PER * 4;  // the partial tiles reuse the chunks
  __shared__ __attribute__((aligned(16))) char lds[kSmWaves * LDSB];
  const GemmProblem &P = probs.p[blockIdx.z];
  const int M = pin_s(P.M), N = pin_s(P.N), K = pin_s(P.K), lda = pin_s(P.lda), ldc = pin_s(P.ldc);
  const int KSp = pin_s(P.ldb) / F::KSTEP, KS = K / F::KSTEP;
  const int rgs = (M + kSmRows - 1) / kSmRows;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int rg = id % rgs, nb = id / rgs;  // neighbours share a column block
  if (nb >= (N + BLK - 1) / BLK) return;
  const int m0 = rg * kSmRows;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- this wave's k-steps; the first chunk's weights and the row indices are requested before
  // the row count is waited for ----
  const int s_begin = KS * wave / kSmWaves, s_end = KS * (wave + 1) / kSmWaves;
  const int n = s_end - s_begin;
  typedef u32x4 BSet[F::STEPS];
  BSet b0, b1;
  // weight vector of this lane at k-step s: wp + s * WSTEP
  const size_t wcol = PK == BLK ? (size_t)nb * KSp * 64 + lane
                                : ((size_t)(nb >> 1) * KSp * 2 + (lane >> 5)) * 64 + ((lane >> 4) & 1) * 32 + (nb & 1) * 16 + (lane & 15);
  constexpr int WSTEP = PK == BLK ? 1024 : 2048;
  const char *const wp = (const char *)P.Bp + wcol * 16;
  auto load_b = [&](int c, BSet &b) {
#pragma unroll
    for (int d = 0; d < F::STEPS; ++d) {
      const int s = s_begin + c * F::STEPS + d;
      b[d] = *(const u32x4 *)(wp + (size_t)(s < s_end ? s : KS - 1) * WSTEP);  // past the end: never used
    }
  };
  const int mrow = m0 + (lane & (kSmRows - 1));
  int myrow = mrow;
  if (P.a_idx) myrow = P.a_idx[mrow < M ? mrow : M - 1];
  load_b(0, b0);
  // rows counted on the device, when given, bound the rows read and stored
  const int *const mdp = pin_s(P.m_dev);
  int Mv = M;
  if (mdp) {
    const int md = *(const __attribute__((address_space(1))) int *)mdp;
    Mv = md < M ? md : M;
  }
  if (m0 >= Mv) return;

  // ---- activations: 64-k row pieces into this wave's LDS (16-byte vectors, one row's vectors
  // in consecutive lanes: a load instruction touches the full cache lines of four or eight rows.
  // Loaded as MFMA fragments, 32 rows x 32 bytes, they cost more than the weights: rows lie a
  // power of two apart and met in the same cache channels) ----
  constexpr int VR = F::KC * (int)sizeof(AT) / 16;  // vectors per row piece
  constexpr int RPI = 64 / VR;      // rows per load instruction
  constexpr int NI = kSmRows / RPI;
  if (mrow >= Mv) {
    myrow = 0;
  } else if (P.a_idx && (myrow < 0 || myrow >= P.a_rows)) {
    if (P.err) atomicOr(P.err, 1 << P.err_bit);
    myrow = myrow < 0 ? 0 : P.a_rows - 1;
  }
  int myout = myrow;  // EPI_SCATTER: the (clamped) gather row, or o_idx
  if (EPI == EPI_SCATTER && P.o_idx) myout = P.o_idx[mrow < Mv ? mrow : m0];
  const int vec = lane % VR;
  const char *ap[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
    ap[i] = (const char *)P.A + (size_t)__shfl(myrow, i * RPI + lane / VR, 64) * lda * sizeof(AT);
  u32x4 areg[NI];
  auto load_a = [&](int c) {
    const int k = (s_begin + c * F::STEPS) * F::KSTEP + vec * (16 / (int)sizeof(AT));
    const size_t o = (size_t)(k < K ? k : K - 16 / (int)sizeof(AT)) * sizeof(AT);  // past K: never used
#pragma unroll
    for (int i = 0; i < NI; ++i) areg[i] = *(const u32x4 *)(ap[i] + o);
  };
  char *const mine = lds + wave * LDSB;
  auto store_a = [&]() {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      char *const d = mine + (i * RPI + lane / VR) * F::ROWB;
      if constexpr (sizeof(AT) == sizeof(CT)) {
        *(u32x4 *)(d + vec * 16) = areg[i];
      } else {  // fp32 rows of a bf16 product: four values round to 8 bytes
        float x[4];
        __builtin_memcpy(x, &areg[i], 16);
        bf16 h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = to_bf16(x[j]);
        __builtin_memcpy(d + vec * 8, h, 8);
      }
    }
    // the chunk is read by other lanes of this wave only
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  load_a(0);

  accv acc[F::RB];
#pragma unroll
  for (int i = 0; i < F::RB; ++i)
#pragma unroll
    for (int r = 0; r < F::NACC; ++r) acc[i][r] = 0.f;

  // a second row block without rows (BLK 16, at most 16 rows) is not multiplied
  const bool two = F::RB > 1 && Mv - m0 > BLK;
  const char *const frag = mine + (lane & (BLK - 1)) * F::ROWB + (lane / BLK) * 16;
  auto compute = [&](int c, const BSet &b) {
#pragma unroll
    for (int d = 0; d < F::STEPS; ++d) {
      if (c * F::STEPS + d >= n) break;  // wave-uniform
      u32x4 av[F::RB];
#pragma unroll
      for (int i = 0; i < F::RB; ++i)
        av[i] = *(const u32x4 *)(frag + i * BLK * F::ROWB + d * F::KSTEP * (int)sizeof(CT));
      if constexpr (sizeof(CT) == 2) {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast16<bf16x8>(av[0]), bitcast16<bf16x8>(b[d]), acc[0],
                                                         0, 0, 0);
      } else {
        float fa[F::RB][4], fb[4];
        __builtin_memcpy(fb, &b[d], 16);
#pragma unroll
        for (int i = 0; i < F::RB; ++i) __builtin_memcpy(fa[i], &av[i], 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0][e], fb[e], acc[0], 0, 0, 0);
        if (two) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[F::RB - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[F::RB - 1][e], fb[e], acc[F::RB - 1], 0, 0, 0);
        }
      }
    }
  };
  const int nch = (n + F::STEPS - 1) / F::STEPS;
  auto chunk = [&](int c, const BSet &b, BSet &bn) {
    store_a();
    if (c + 1 < nch) {
      load_b(c + 1, bn);
      load_a(c + 1);
    }
    compute(c, b);
    // the next chunk overwrites what this one's reads took
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  for (int c = 0; c < nch; c += 2) {
    chunk(c, b0, b1);
    if (c + 1 < nch) chunk(c + 1, b1, b0);
  }
  __syncthreads();

  // ---- the waves' partial tiles, added in wave order ----
  float *const red = (float *)lds;
  auto row_of = [&](int e) {
    const int l = e & 63, r = (e >> 6) % F::NACC, i = (e >> 6) / F::NACC;
    return m0 + BLK * i + (BLK == 16 ? (l >> 4) * 4 + r : 8 * (r >> 2) + 4 * (l >> 5) + (r & 3));
  };
#pragma unroll
  for (int i = 0; i < F::RB; ++i)
#pragma unroll
    for (int r = 0; r < F::NACC; ++r) red[wave * PER + (i * F::NACC + r) * 64 + lane] = acc[i][r];
  __syncthreads();
  // EPI_SCATTER: the output row of each element (lane l of every wave holds that of row m0 + l % 32)
  int orow[EPI == EPI_SCATTER ? PER / kSmThreads : 1];
  if constexpr (EPI == EPI_SCATTER) {
#pragma unroll
    for (int q = 0; q < PER / kSmThreads; ++q) orow[q] = __shfl(myout, row_of(tid + kSmThreads * q) - m0, 64);
  }
  const int obf = pin_s(P.out_bf16);
  const float *const biasp = pin_s(P.bias);
  char *const outp = (char *)pin_s(P.out);
#pragma unroll
  for (int q = 0; q < PER / kSmThreads; ++q) {
    const int e = tid + kSmThreads * q;
    float v = red[e];
#pragma unroll
    for (int w = 1; w < kSmWaves; ++w) v += red[w * PER + e];
    // element e = (row block, accumulator r, lane l) of the MFMA output layout
    const int row = row_of(e);
    const int col = nb * BLK + (e & (BLK - 1));
    if (row >= Mv || col >= N) continue;
    if (biasp) v += biasp[col];
    if (EPI == EPI_TANH) v = tanh_fast(v);
    const int orw = EPI == EPI_SCATTER ? orow[q] : row;
    if (obf)
      ((bf16 *)outp)[(size_t)orw * ldc + col] = to_bf16(v);
    else
      ((float *)outp)[(size_t)orw * ldc + col] = v;
  }
}

template <typename CT, typename AT, int PK, int EPI>
static hipError_t go_small(const Problems &ps, int nprob, hipStream_t st) {
  constexpr int BLK = sizeof(CT) == 2 ? 32 : 16;
  int maxg = 0;
  for (int i = 0; i < nprob; ++i) {
    const GemmProblem &p = ps.p[i];
    if (p.K % SmForm<CT, AT, BLK>::KSTEP != 0 || p.K > p.ldb || p.K < 1) return hipErrorInvalidValue;
    const int g = (p.M + kSmRows - 1) / kSmRows * ((p.N + BLK - 1) / BLK);
    maxg = g > maxg ? g : maxg;
  }
  if (maxg == 0) return hipSuccess;
  hipLaunchKernelGGL((gemm_small_kernel<CT, AT, PK, EPI>), dim3(maxg, 1, nprob), dim3(kSmThreads), 0, st, ps);
  return hipGetLastError();
}

template <int EPI>
static hipError_t go_small_e(int bf16_mma, const Problems &ps, int nprob, hipStream_t st) {
  if (bf16_mma)
    return ps.p[0].a_bf16 ? go_small<bf16, bf16, 32, EPI>(ps, nprob, st) : go_small<bf16, float, 32, EPI>(ps, nprob, st);
  return ps.p[0].wblk == 32 ? go_small<float, float, 32, EPI>(ps, nprob, st)
                            : go_small<float, float, 16, EPI>(ps, nprob, st);
}

hipError_t launch_gemm_small(int bf16_mma, const Problems &ps, int nprob, Epilogue epi, hipStream_t st) {
  if (epi == EPI_SCATTER) return go_small_e<EPI_SCATTER>(bf16_mma, ps, nprob, st);
  return epi == EPI_TANH ? go_small_e<EPI_TANH>(bf16_mma, ps, nprob, st) : go_small_e<EPI_STORE>(bf16_mma, ps, nprob, st);
}

}  // namespace mt
