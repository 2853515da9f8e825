// Kernels of the encoder's recurrence (mt_encode): the lists of rows that a position updates, and
// one position of a shallow cell (no layer norm, no transition blocks) as one kernel.
//
// A padded position only carries each direction's state over, so the input products are computed
// at the valid positions alone, and at each position only the rows that are valid there enter
// the recurrent product (a batch's lengths differ: with lengths of mean 25 in a padded length
// of 80, a third of the rows).
#include "mt_gemm_common.h"

namespace mt {

// Block 0: the valid entries of mask [B][S] in increasing order, vrow[j] = b*S + i, and their
// tokens vtok[j]; nvalid their number.  Every token, padding included, is checked against src_V
// (error bit 3).  Block 1 + i: act[i][k] = the sentences valid at position i in increasing
// order, acnt[i] their number.
__global__ __launch_bounds__(1024) void enc_lists_kernel(int B, int S, const float *__restrict__ mask,
                                                         const int32_t *__restrict__ tok, int src_V,
                                                         int32_t *__restrict__ vrow, int32_t *__restrict__ vtok,
                                                         int *__restrict__ nvalid, int32_t *__restrict__ act,
                                                         int *__restrict__ acnt, int32_t *err) {
  __shared__ int wsum[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const bool all = blockIdx.x == 0;
  const int pos = (int)blockIdx.x - 1;
  const int n = all ? B * S : B;
  int base = 0;
  for (int c0 = 0; c0 < n; c0 += 1024) {
    const int i = c0 + t;
    bool ok = false;
    int tk = 0;
    if (i < n) {
      ok = mask[all ? (size_t)i : (size_t)i * S + pos] != 0.f;
      if (all) {
        tk = tok[i];
        if (tk < 0 || tk >= src_V) atomicOr(err, 1 << 3);
      }
    }
    const unsigned long long bal = __ballot(ok);
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int off = base, tot = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      off += w < wave ? wsum[w] : 0;
      tot += wsum[w];
    }
    if (ok) {
      const int j = off + __popcll(bal & ((1ull << lane) - 1ull));
      if (all) {
        vrow[j] = i;
        vtok[j] = tk;
      } else {
        act[(size_t)pos * B + j] = i;
      }
    }
    base += tot;
    __syncthreads();  // wsum is rewritten by the next chunk
  }
  if (t == 0) *(all ? nvalid : acnt + pos) = base;
}

hipError_t launch_enc_lists(int B, int S, const float *mask, const int32_t *tok, int src_V, int32_t *vrow,
                            int32_t *vtok, int *nvalid, int32_t *act, int *acnt, int32_t *err, hipStream_t st) {
  hipLaunchKernelGGL(enc_lists_kernel, dim3(S + 1), dim3(1024), 0, st, B, S, mask, tok, src_V, vrow, vtok, nvalid, act,
                     acnt, err);
  return hipGetLastError();
}

// One position of both directions of a shallow cell: h U, the gates and the new state.
//
// A workgroup owns 16 hidden units (their three gate columns) and 16 RB active rows of one
// direction; its eight waves split the depth as in gemm_small_kernel (16x16 MFMAs, the
// activations staged per wave, partial tiles added through LDS in wave order), and thread t
// finishes one (row, unit) with the three sums it needs, so that the recurrent product is never
// written and the cell needs no launch of its own.  At 64 sentences (RB = 2) and H = 1024 that is 256
// workgroups, one on each compute unit; row groups of a unit block are neighbours, so an XCD
// fetches an eighth of the weights.  What bounds a position is one round of loads behind another
// (the row list, then the rows' states) and the weights themselves, which every launch fetches
// anew (25 MB in fp32, 12.6 MB in bf16): in fp32 8 us a position with one sentence, 11.8 with 64
// of mixed lengths (recurrent product and cell as two launches over all rows: 19.5); in bf16 5 us
// (two launches: 11).
constexpr int kEncWaves = 8, kEncThreads = 64 * kEncWaves, kEncUnits = 16, kEncKC = 64;

// FIRST: the first position, with a zero previous state and no product
template <typename CT, int PK, int RB, bool FIRST>
__global__ __launch_bounds__(kEncThreads) void enc_step_kernel(EncStep P) {
  constexpr bool BF = sizeof(CT) == 2;
  constexpr int kEncRows = 16 * RB;              // rows of a workgroup
  constexpr int KSTEP = BF ? 32 : 16;            // k per MFMA operand vector
  constexpr int STEPS = kEncKC / KSTEP;          // k-steps of a chunk
  constexpr int ROWB = kEncKC * (int)sizeof(CT) + 16;
  constexpr int STG = kEncRows * ROWB;           // a wave's chunk
  constexpr int PER = 3 * RB * 4 * 64;           // partial sums of a wave: gates x row blocks x 16 x 16
  constexpr int LDSB = STG > PER * 4 ? STG : PER * 4;
  __shared__ __attribute__((aligned(16))) char lds[kEncWaves * LDSB];
  const int B = P.B, H = P.H;
  const int rgs = (B + kEncRows - 1) / kEncRows, nu = H / kEncUnits;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int rg = id % rgs, q = id / rgs, dir = q / nu, ub = q % nu;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = dir ? P.pos[1] : P.pos[0], prv = dir ? P.prv[1] : P.prv[0];
  const int r0 = rg * kEncRows;
  CT *const cbase = (CT *)P.ctx;
  const size_t ldc = P.ldc;
  const size_t opos = (size_t)pos * 2 * H + (size_t)dir * H, oprv = (size_t)prv * 2 * H + (size_t)dir * H;

  const int32_t *const act = P.act + (size_t)pos * B;

  // ---- loads that wait for nothing: the first weights, the position's row count and rows, and
  // what a row that is padded here carries over.  Asked for one after another, each of them
  // costs a round trip of about a microsecond ----
  const int KS = (H + KSTEP - 1) / KSTEP;
  const int s_begin = KS * wave / kEncWaves, s_end = KS * (wave + 1) / kEncWaves, n = s_end - s_begin;
  // weight vector of gate g at k-step s: wp[g] + s * WSTEP
  constexpr int WSTEP = PK == 16 ? 1024 : 2048;
  const int KSp = P.ldb / (BF || PK == 16 ? 16 : 8);
  const char *wp[3];
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    const int cb = g * nu + ub;  // 16-column block
    const size_t v = PK == 16 ? (size_t)cb * KSp * 64 + lane
                              : ((size_t)(cb >> 1) * KSp + (lane >> 5)) * 64 + ((lane >> 4) & 1) * 32 + (cb & 1) * 16 + (lane & 15);
    wp[g] = (const char *)(dir ? P.w[1] : P.w[0]) + v * 16;
  }
  typedef u32x4 BSet[STEPS][3];
  BSet b0, b1;
  auto load_b = [&](int c, BSet &w) {
#pragma unroll
    for (int d = 0; d < STEPS; ++d) {
      const int s = s_begin + c * STEPS + d;
      const size_t o = (size_t)(s < s_end ? s : KS - 1) * WSTEP;  // past the end: never used
#pragma unroll
      for (int g = 0; g < 3; ++g) w[d][g] = *(const u32x4 *)(wp[g] + o);
    }
  };
  const int cb_row = r0 + tid / kEncUnits, cb_un = ub * kEncUnits + tid % kEncUnits;
  const int cb_b = cb_row < B ? cb_row : B - 1;
  typedef typename std::conditional<BF, uint16_t, uint32_t>::type bits;  // a state's storage
  uint32_t carried = 0u;
  if constexpr (!FIRST) carried = *(const bits *)(cbase + cb_b * ldc + oprv + cb_un);
  const float cmask = P.mask[(size_t)cb_b * P.S + pos];
  const int ar = r0 + (lane & (kEncRows - 1));
  const int arow_raw = act[ar < B ? ar : B - 1];  // entries past the count are not row numbers
  const int cnt = P.acnt[pos];
  if constexpr (!FIRST) load_b(0, b0);
  asm volatile("" : "+v"(carried));  // loaded with the others, not behind the mask
  if (tid < kEncRows * kEncUnits && cb_row < B && cmask == 0.f) *(bits *)(cbase + cb_b * ldc + opos + cb_un) = (bits)carried;
  if (r0 >= cnt) return;
  const int row_first = __builtin_amdgcn_readfirstlane(arow_raw);  // lane 0: row r0 of the list
  const int arow = ar < cnt ? arow_raw : row_first;

  // ---- this thread's (row, unit) of the MFMA output layout, its input gates and state ----
  const int l = tid & 63, rr = (tid >> 6) & 3, ib = tid >> 8;
  const int lrow = (16 * ib + 4 * (l >> 4) + rr) % kEncRows;
  const int un = ub * kEncUnits + (l & 15);
  const bool live = tid < kEncRows * kEncUnits && r0 + lrow < cnt;
  const int b = __shfl(arow, lrow, 64);
  const float *const xr = P.xe + ((size_t)b * P.S + pos) * 6 * H + (size_t)dir * 3 * H + un;

  float xa, xz, xh, h = 0.f, us[3] = {0.f, 0.f, 0.f};
  if constexpr (FIRST) {
    xa = xr[0]; xz = xr[H]; xh = xr[2 * H];
  } else {
    constexpr int VR = kEncKC * (int)sizeof(CT) / 16, RPI = 64 / VR, NI = kEncRows / RPI;
    const int vec = lane % VR;
    const char *ap[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
      ap[i] = (const char *)(cbase + (size_t)__shfl(arow, i * RPI + lane / VR, 64) * ldc + oprv);
    u32x4 areg[NI];
    auto load_a = [&](int c) {
      constexpr int VK = 16 / (int)sizeof(CT);
      const int k = (s_begin + c * STEPS) * KSTEP + vec * VK;
      // past H: the row's last vector, which meets the packing's zero padding or is never used
      const size_t o = (size_t)(k < H ? k : H - VK) * sizeof(CT);
#pragma unroll
      for (int i = 0; i < NI; ++i) areg[i] = *(const u32x4 *)(ap[i] + o);
    };
    load_a(0);
    xa = xr[0]; xz = xr[H]; xh = xr[2 * H];
    h = BF ? P.sst[((size_t)dir * B + b) * H + un] : (float)cbase[b * ldc + oprv + un];
    char *const mine = lds + wave * LDSB;
    typedef __attribute__((__vector_size__(4 * sizeof(float)))) float accv;
    accv acc[RB][3];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[i][g] = accv{0.f, 0.f, 0.f, 0.f};
    const bool two = cnt - r0 > 16;  // the second row block has rows
    const char *const frag = mine + (lane & 15) * ROWB + (lane >> 4) * 16;
    auto mul = [&](int i, const u32x4(&w)[3], const u32x4 &av) {
      if constexpr (BF) {
#pragma unroll
        for (int g = 0; g < 3; ++g)
          acc[i][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bitcast16<bf16x8>(av), bitcast16<bf16x8>(w[g]), acc[i][g], 0, 0, 0);
      } else {
        float fa[4], fb[3][4];
        __builtin_memcpy(fa, &av, 16);
#pragma unroll
        for (int g = 0; g < 3; ++g) __builtin_memcpy(fb[g], &w[g], 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int g = 0; g < 3; ++g) acc[i][g] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[g][e], acc[i][g], 0, 0, 0);
      }
    };
    auto compute = [&](int c, const BSet &w) {
#pragma unroll
      for (int d = 0; d < STEPS; ++d) {
        if (c * STEPS + d >= n) break;  // wave-uniform
        const u32x4 a0 = *(const u32x4 *)(frag + d * KSTEP * (int)sizeof(CT));
        if (RB == 2 && two) {
          const u32x4 a1 = *(const u32x4 *)(frag + (RB - 1) * 16 * ROWB + d * KSTEP * (int)sizeof(CT));
          mul(0, w[d], a0);
          mul(RB - 1, w[d], a1);
        } else {
          mul(0, w[d], a0);
        }
      }
    };
    const int nch = (n + STEPS - 1) / STEPS;
    auto chunk = [&](int c, const BSet &w, BSet &wn) {
#pragma unroll
      for (int i = 0; i < NI; ++i) *(u32x4 *)(mine + (i * RPI + lane / VR) * ROWB + vec * 16) = areg[i];
      // the chunk is read by other lanes of this wave only
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (c + 1 < nch) {
        load_b(c + 1, wn);
        load_a(c + 1);
      }
      compute(c, w);
      // the next chunk overwrites what this one's reads took
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    for (int c = 0; c < nch; c += 2) {
      chunk(c, b0, b1);
      if (c + 1 < nch) chunk(c + 1, b1, b0);
    }
    __syncthreads();
    float *const red = (float *)lds;  // [wave][gate][row block][accumulator][lane]
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave * PER + ((g * RB + i) * 4 + r) * 64 + lane] = acc[i][g][r];
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      float v = red[g * (PER / 3) + tid];
#pragma unroll
      for (int w = 1; w < kEncWaves; ++w) v += red[w * PER + g * (PER / 3) + tid];
      us[g] = v;
    }
  }
  if (!live) return;
  const float r = sigmoid_fast(xa + us[0]), z = sigmoid_fast(xz + us[1]);
  const float hh = tanh_fast(xh + r * us[2]);
  const float v = (1.0f - z) * hh + z * h;
  Store<CT>::put(cbase + b * ldc + opos + un, v);
  // the fp32 state of a bf16 model is read and written by this thread alone
  if (BF) P.sst[((size_t)dir * B + b) * H + un] = v;
}

static constexpr int enc_row_blocks(int B) { return B <= 32 ? 1 : 2; }

// Up to four workgroups per unit, and fewer of a wide cell, whose row groups each read all of its
// weights (in fp32 at half the states' rate, so the line there lies earlier, and row groups of 32
// that are not full cost most).  us for 24 positions, a product and a cell launch per position
// against one kernel, sentences of full length / of mixed lengths:
//   bf16 H = 256: 512 sentences 277 218 / 252 203, 1024 422 390 / 377 329;  512: 512 426 404 / 364 336,
//   768 564 607 / 496 474;  1024: 160 370 355 / 327 294, 256 476 481 / 411 394, 300 487 552 / 418 431;
//   1536: 160 517 524 / 445 429, 192 624 662 / 483 529;  2048: 96 532 532 / 486 453, 128 594 660 / 515 581
//   fp32 H = 256: 1024 607 598 / 565 484;  512: 384 617 618 / 544 506, 768 985 1201 / 854 936;  768: 160 700
//   571 / 702 541, 192 732 762 / 670 615, 256 871 833 / 747 676, 300 901 1035 / 788 800;  1024: 128 794 678 /
//   728 594, 160 853 934 / 765 732, 256 1247 1281 / 1115 1035;  1536: 32 613 529 / 574 516, 33 712 798 / 696
//   736, 128 1355 1322 / 1189 1181;  2048: 16 614 472 / 571 475, 48 965 1145 / 868 1025
bool enc_step_takes(int bf16_mma, int B, int H) {
  const int rb = enc_row_blocks(B);
  const long wg = (long)((B + 16 * rb - 1) / (16 * rb)) * (H / kEncUnits) * 2;
  if (bf16_mma) return wg <= 1024 && wg * H <= 1600 * 1024;
  return wg <= 1024 && wg * H <= 600 * 1024 && (H <= 1024 || rb == 1);
}

template <typename CT, int PK, int RB>
static hipError_t go_step_rb(const EncStep &p, hipStream_t st) {
  const dim3 grid((unsigned)((p.B + 16 * RB - 1) / (16 * RB) * (p.H / kEncUnits) * 2));
  if (p.first)
    hipLaunchKernelGGL((enc_step_kernel<CT, PK, RB, true>), grid, dim3(kEncThreads), 0, st, p);
  else
    hipLaunchKernelGGL((enc_step_kernel<CT, PK, RB, false>), grid, dim3(kEncThreads), 0, st, p);
  return hipGetLastError();
}

// Rows per workgroup: 16 up to 32 sentences, where groups of 32 leave half of the units idle, else
// 32, which fetch the weights half as often (us for 40 positions with keys and start state, 16 /
// 32 rows: fp32 32 sentences 495 / 636, 64 865 / 787, 128 1393 / 1269; bf16 64 300 / 270, 128 488 /
// 465).
template <typename CT, int PK>
static hipError_t go_step(const EncStep &p, hipStream_t st) {
  return enc_row_blocks(p.B) == 1 ? go_step_rb<CT, PK, 1>(p, st) : go_step_rb<CT, PK, 2>(p, st);
}

hipError_t launch_enc_step(int bf16_mma, const EncStep &p, hipStream_t st) {
  if (p.H % kEncUnits != 0 || p.ldb % 64 != 0 || p.H > p.ldb) return hipErrorInvalidValue;
  if (bf16_mma) return go_step<bf16, 32>(p, st);
  return p.wblk == 32 ? go_step<float, 32>(p, st) : go_step<float, 16>(p, st);
}

}  // namespace mt
