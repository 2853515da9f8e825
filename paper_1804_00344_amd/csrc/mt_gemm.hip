// Matrix products of the decoder step on CDNA4 matrix cores:
// out[m, n] = sum_k A[m, k] * W[k, n] (+ bias[n]), tanh optional, fp32 or bf16 output.
// The A operand may be gathered by a row index (token -> embedding row, backpointer -> state
// row); every problem of one launch has the same A element type.  W is packed at load time
// (mt_load_weights) in the MFMA fragment order of its kernel, zero padded to [K_pad][N_pad]:
//  * fp32 (gemm_f32_kernel): 16 x 16 x 4 MFMAs, both operands straight from global memory;
//  * bf16 (gemm_wd_kernel): 32 x 32 x 16 MFMAs, weights straight from global memory and the
//    activations through a small LDS ring.
// Loads are unconditional and nothing is masked: a row past M reads row 0 and its output row is
// never stored, and a vector past K reads the row's last in-range vector, which meets the zero
// padding of the packed weights (finite x 0 adds nothing).  Epilogues load the bias before any
// store and read the problem fields into scalar registers once: a load between the stores
// would make every store wait for all earlier ones (the memory counter counts both).
#include <algorithm>

#include "mt_gemm_common.h"

namespace mt {

// Tile of a problem whose row count is on the device, where a launch for M rows finds a part of
// them live: each XCD keeps its run of column tiles but walks it row tile by row tile, so that
// its live tiles come first and are spread over its units one by one.  (Column tile by column
// tile, the tiles that end at once let the live ones bunch: 1603 valid of 5120 rows x 2048 x 2048
// in fp32 195 -> 141 us.)  w: the tile's number in launch order, in groups of `per` per workgroup; a
// permutation of the tiles where their columns divide over the XCDs (otherwise the order stays).
__device__ __forceinline__ void counted_tile(int w, int tilesM, int tilesN, int per, int &tm, int &tn) {
  if (tilesN % (kXcds * per) != 0 || (int)gridDim.x * per != tilesM * tilesN) return;
  const int nx = tilesN / kXcds, g = w / per;  // column tiles of an XCD; workgroup
  const int x = g % kXcds, i = g / kXcds * per + w % per;
  tm = i / nx;
  tn = x * nx + i % nx;
}

// Stores of one output tile through a buffer view of its rows: a lane past the last column takes
// an offset beyond the view and rows past the last lie beyond it, so the hardware drops what
// must not be stored and no store is masked or branched around.  (With a row test and a 64-bit
// address around each store the epilogue was 12 instructions a store, which a workgroup runs
// once, from a cold instruction cache: 1024 x 512 x 1024 in 64-row tiles 8.9 -> 8.3 us, in 128-row
// tiles 15.4 -> 13.9.)
struct TileOut {
  __amdgpu_buffer_rsrc_t rs;
  int rowb;  // bytes per output row
  __device__ __forceinline__ TileOut(char *out, int bf, int m0, int rows, int ldc)
      : rs(__builtin_amdgcn_make_buffer_rsrc(out + (size_t)m0 * ldc * (bf ? 2 : 4), 0, rows * ldc * (bf ? 2 : 4), 0x00020000)),
        rowb(ldc * (bf ? 2 : 4)) {}
  // offset of column col in the lane's first row of the tile
  template <bool BF>
  __device__ __forceinline__ int lane_offset(int row, int col, int N) const {
    return col < N ? row * rowb + col * (BF ? 2 : 4) : 0x7ffffff0;
  }
  // row: further rows (compile-time per store); the whole offset is the lane's, which is what the
  // range check compares
  template <bool BF>
  __device__ __forceinline__ void store(float v, int vo, int row) const {
    if constexpr (BF) {
      const bf16 h = to_bf16(v);
      short x;
      __builtin_memcpy(&x, &h, 2);
      __builtin_amdgcn_raw_buffer_store_b16(x, rs, vo + row * rowb, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), rs, vo + row * rowb, 0, 0);
    }
  }
};

// Output rows of an EPI_SCATTER tile.  Its rows increase (see Epilogue), so that the first and the
// last tell whether they are consecutive: then the tile is stored as a plain one at its first
// row.  Sentences of equal length, or the valid positions of long ones, make such tiles.  The rows
// are kept from the prologue: loaded again here, and with each store addressed by itself, two bf16
// products of 768 x 3072 x 1024 took 27.9 us for the 19.8 of a plain store.
struct OutRows {
  int first;
  bool run;
};
__device__ __forceinline__ OutRows out_rows_of(int first, int last, int rows) {
  first = __builtin_amdgcn_readfirstlane(first);
  last = __builtin_amdgcn_readfirstlane(last);
  return {first, last - first == rows - 1};
}

// ---------------------------------------------------------------------------------------
// bf16 operands: weights streamed from global memory straight into registers.
//
// The weights are packed in the MFMA fragment order of the B operand (mt_load_weights): for
// 32-column block nb and 16-k step ks, 64 lanes x 16 bytes at ((nb * KSp + ks) * 64 + lane) * 16,
// lane l holding W[ks * 16 + (l / 32) * 8 + j][nb * 32 + l % 32], j < 8 (KSp = K_pad / 16, K_pad a
// multiple of 128, zero rows beyond K).  One coalesced 16-byte load per lane is one fragment.
//
// Block: 32 MB rows x 128 columns (MB by go_wd), four waves: two column halves of 32 MB x 64 (MB x 2
// blocks of 32x32x16 MFMAs), each shared by two waves.  The block's activation rows
// pass through LDS in stages of 128 k (bf16, an fp32 operand rounded
// on the way), double-buffered from two register stages with one barrier per 8 k-steps; each
// wave's weight fragments come through a register ring refilled D k-steps ahead, so the only
// LDS traffic is the activations (written once; a row's fragment is read by the two waves, one of
// each column half, that own its k-step).
//
// The KW = 2 waves of a column half share its k-steps (of the 8 of a stage, wave kh takes 4), and
// at the end exchange halves of their partial tiles through LDS, each finishing one 32-column
// block.  With one wave per column half, 288 tiles of 768 x 3072 left half of the 1024 SIMDs
// without a wave and the others with nothing to run while one waited: 320 x 3072 x 1024 9.5 -> 8.4
// us, 768 x 5120 x 1024 17.0 -> 15.6, 1024 x 5120 x 1024 26.9 -> 20.7, 768 x 3584 x 2048 22.9 -> 21.0.
constexpr int kWdCols = 128, KW = 2, kWdThreads = 128 * KW;
constexpr int kWdStageK = 128;                   // k per LDS stage (8 k-steps)
constexpr int kWdRowBytes = kWdStageK * 2 + 16;  // padded LDS row of one stage

template <typename AT, int EPI, int D, int MB>
__global__ __launch_bounds__(kWdThreads) void gemm_wd_kernel(Problems probs) {
  constexpr int kWdRows = 32 * MB;
  constexpr int kWdStage = kWdRows * kWdRowBytes;
  constexpr int RP = 4 * MB / KW;  // staged rows per thread
  constexpr int SPS = 8 / KW;      // k-steps per stage and wave
  static_assert(2 * kWdStage >= 4 * MB * 16 * 64 * 4, "the exchange reuses the stages");
  __shared__ __attribute__((aligned(16))) char lds[2 * kWdStage];
  __shared__ __attribute__((aligned(16))) int32_t out_row[EPI == EPI_SCATTER ? kWdRows : 4];
  constexpr int AV = (int)sizeof(AT) / 2;  // 16-byte source loads per 8-k vector
  const GemmProblem &P = probs.p[blockIdx.z];
  // problem fields read once into scalar registers (as references into the argument block
  // they would be re-read, each with a full wait, at every use in the epilogue)
  const int M = pin_s(P.M), N = pin_s(P.N), K = pin_s(P.K), lda = pin_s(P.lda), ldc = pin_s(P.ldc);
  const int KSp = pin_s(P.ldb) / 16;
  const int tilesM = (M + kWdRows - 1) / kWdRows;
  const int tilesN = (N + kWdCols - 1) / kWdCols;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  if (tile >= tilesM * tilesN) return;
  int tm = tile % tilesM, tn = tile / tilesM;  // neighbours share a weight panel
  if (P.m_dev) counted_tile(blockIdx.x, tilesM, tilesN, 1, tm, tn);
  const int m0 = tm * kWdRows, n0 = tn * kWdCols;
  // rows counted on the device, when given, bound the rows read and stored
  const int *const mdp = pin_s(P.m_dev);
  int Mv = M;
  if (mdp) {
    const int md = *(const __attribute__((address_space(1))) int *)mdp;
    Mv = md < M ? md : M;
  }
  if (m0 >= Mv) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 1);  // column half
  const int kh = __builtin_amdgcn_readfirstlane(tid >> 7);

  // ---- activation staging: thread t owns 8-k vector c = t % 16 of rows t / 16 + 8 KW p ----
  const int c = tid & 15;
  const char *a_src[RP];
  {
    int src[RP];
    int orow[RP];
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      const int m = m0 + (tid >> 4) + 8 * KW * p;
      src[p] = m < Mv ? m : 0;  // rows past the count read row 0 (of the gather) and are never stored
    }
    if constexpr (EPI == EPI_SCATTER)
      if (P.o_idx) {
#pragma unroll
        for (int p = 0; p < RP; ++p) orow[p] = P.o_idx[src[p]];
      }
    if (P.a_idx) {
      bool bad = false;
#pragma unroll
      for (int p = 0; p < RP; ++p) src[p] = P.a_idx[src[p]];
#pragma unroll
      for (int p = 0; p < RP; ++p) {
        bad |= src[p] < 0 || src[p] >= P.a_rows;
        src[p] = src[p] < 0 ? 0 : src[p] >= P.a_rows ? P.a_rows - 1 : src[p];
      }
      if (bad && P.err) atomicOr(P.err, 1 << P.err_bit);
    }
#pragma unroll
    for (int p = 0; p < RP; ++p) a_src[p] = (const char *)P.A + (size_t)src[p] * lda * sizeof(AT);
    // EPI_SCATTER: the output row of each stored row, kept for the epilogue (the stages' barriers
    // come before its reads)
    if constexpr (EPI == EPI_SCATTER)
      if (c == 0) {
#pragma unroll
        for (int p = 0; p < RP; ++p) out_row[(tid >> 4) + 8 * KW * p] = P.o_idx ? orow[p] : src[p];
      }
  }
  typedef u32x4 StageRegs[RP][AV];
  auto load_stage = [&](int st, StageRegs &R) {
    const int k = st * kWdStageK + c * 8;
    const int kc = k < K ? k : K - 8;  // past K: the row's last vector (it meets zero weights)
#pragma unroll
    for (int p = 0; p < RP; ++p)
#pragma unroll
      for (int v = 0; v < AV; ++v) R[p][v] = *(const u32x4 *)(a_src[p] + (size_t)kc * sizeof(AT) + 16 * v);
  };
  auto store_stage = [&](int buf, const StageRegs &R) {
    char *base = lds + buf * kWdStage + c * 16;
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      u32x4 val;
      if constexpr (AV == 2)
        val = pack_bf16x8(R[p][0], R[p][1]);
      else
        val = R[p][0];
      *(u32x4 *)(base + ((tid >> 4) + 8 * KW * p) * kWdRowBytes) = val;
    }
  };

  // ---- weight fragments: this wave's blocks nb0, nb0 + 1; ring slot of its n-th k-step is n % D ----
  const int nb0 = (n0 + wave * 64) >> 5;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      (void *)P.Bp, 0, ((N + kWdCols - 1) / kWdCols * kWdCols) * KSp * 32, 0x00020000);
  const int wvo = lane * 16;
  const int wb0 = nb0 * KSp * 1024, wstep1 = KSp * 1024;
  u32x4 ring[D][2];
  const int nst = KSp / 8;
  const int last = nst - 1;
  // the wave's s-th k-step of stage st (past the last: in bounds, never used)
  auto fetch = [&](int st, int s, u32x4(&r)[2]) {
    const int so = wb0 + ((st < last ? st : last) * 8 + kh * SPS + s) * 1024;
    r[0] = __builtin_amdgcn_raw_buffer_load_b128(wrs, wvo, so, 0);
    r[1] = __builtin_amdgcn_raw_buffer_load_b128(wrs, wvo, so + wstep1, 0);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) fetch(d / SPS, d % SPS, ring[d]);

  f32x16 acc[MB][2];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // The wave's k-steps of stage st from LDS buffer buf; the ring slots of stage st are
  // (SPS * (st & 1) + s) % D, static in the two-stage unrolled loop below.  The activation
  // fragments of k-step s + 1 are read before the MFMAs of k-step s (a SIMD holds one or two waves,
  // which meet at the stages' barriers: little else covers the LDS latency).
  const int arow = lane & 31, akoff = (lane >> 5) * 16;
  auto compute = [&](int st, int buf, auto par) {
    const char *base = lds + buf * kWdStage + arow * kWdRowBytes + akoff + kh * (SPS * 32);
    u32x4 af[MB], an[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) af[i] = *(const u32x4 *)(base + i * 32 * kWdRowBytes);
#pragma unroll
    for (int s = 0; s < SPS; ++s) {
      if (s + 1 < SPS) {
#pragma unroll
        for (int i = 0; i < MB; ++i) an[i] = *(const u32x4 *)(base + i * 32 * kWdRowBytes + (s + 1) * 32);
      }
      u32x4(&slot)[2] = ring[(SPS * decltype(par)::value + s) % D];
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast16<bf16x8>(af[i]), bitcast16<bf16x8>(slot[j]),
                                                              acc[i][j], 0, 0, 0);
      fetch(st + D / SPS, s, slot);
      // keep each refill right behind the MFMAs that consumed its slot
      __builtin_amdgcn_sched_barrier(0);
      if (s + 1 < SPS) {
#pragma unroll
        for (int i = 0; i < MB; ++i) af[i] = an[i];
      }
    }
  };

  // Stage st: multiply LDS buffer st & 1, load stage st + 2 into register stage st & 1 and
  // write register stage (st + 1) & 1 (loaded one stage earlier) into the other buffer.
  // Stage indices clamp to the last stage, so the body is branch-free.
  StageRegs s0, s1;
  load_stage(0, s0);
  load_stage(1 < last ? 1 : last, s1);
  store_stage(0, s0);
  __syncthreads();
  auto stage = [&](int st, StageRegs &cur, StageRegs &nxt, auto par) {
    load_stage(st + 2 < last ? st + 2 : last, cur);
    __builtin_amdgcn_sched_barrier(0);
    compute(st, decltype(par)::value, par);
    store_stage(decltype(par)::value ^ 1, nxt);
    __syncthreads();
  };
  int st = 0;
  for (; st + 1 < nst; st += 2) {
    stage(st, s0, s1, std::integral_constant<int, 0>{});
    stage(st + 1, s1, s0, std::integral_constant<int, 1>{});
  }
  if (st < nst) stage(st, s0, s1, std::integral_constant<int, 0>{});

  // ---- epilogue: lane holds D[row = 8*(r/4) + 4*(lane/32) + r%4][col = lane % 32] ----
  // Wave kh finishes column block kh of its half: it leaves the other block's partial sums in LDS
  // and adds the other wave's to its own (the stages are no longer read: the last one ended in a
  // barrier).
  f32x16 fin[MB];
  {
    float *const xw = (float *)lds + (wave * 2 + kh) * (MB * 16 * 64) + lane;
    const float *const xr = (float *)lds + (wave * 2 + (kh ^ 1)) * (MB * 16 * 64) + lane;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xw[(i * 16 + r) * 64] = kh ? acc[i][0][r] : acc[i][1][r];
        fin[i][r] = kh ? acc[i][1][r] : acc[i][0][r];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) fin[i][r] += xr[(i * 16 + r) * 64];
  }
  const int col = n0 + wave * 64 + kh * 32 + (lane & 31);
  const int obf = pin_s(P.out_bf16);
  const float *const biasp = pin_s(P.bias);
  char *const outp = (char *)pin_s(P.out);
  // The bias values are loaded before any store and waited for once: a load between the stores
  // would make every store wait for all earlier stores (the memory counter counts both).
  const float bias = biasp ? ((const __attribute__((address_space(1))) float *)biasp)[col < N ? col : N - 1] : 0.f;
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  const int rows = Mv - m0 < kWdRows ? Mv - m0 : kWdRows;
  const OutRows out_rows = [&] {
    if constexpr (EPI == EPI_SCATTER) return out_rows_of(out_row[0], out_row[rows - 1], rows);
    else return OutRows{m0, true};
  }();
  const TileOut to(outp, obf, out_rows.first, rows, ldc);
  auto epilogue = [&](auto bf) {
    constexpr bool BF = decltype(bf)::value;
    if (EPI == EPI_SCATTER && !out_rows.run) {
      if (col >= N) return;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r0 = i * 32 + 8 * q + 4 * (lane >> 5);
          int32_t orow[4];
          __builtin_memcpy(orow, out_row + (EPI == EPI_SCATTER ? r0 : 0), 16);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (r0 + r >= rows) continue;
            const float v = fin[i][4 * q + r] + bias;
            if constexpr (BF)
              ((__attribute__((address_space(1))) bf16 *)outp)[(size_t)orow[r] * ldc + col] = to_bf16(v);
            else
              ((__attribute__((address_space(1))) float *)outp)[(size_t)orow[r] * ldc + col] = v;
          }
        }
    } else {
      const int vo = to.lane_offset<BF>(4 * (lane >> 5), col, N);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float v = fin[i][r] + bias;
          if (EPI == EPI_TANH) v = tanh_fast(v);
          to.store<BF>(v, vo, i * 32 + 8 * (r >> 2) + (r & 3));
        }
    }
  };
  if (obf)
    epilogue(std::integral_constant<bool, true>{});
  else
    epilogue(std::integral_constant<bool, false>{});
}

template <typename AT, int EPI, int MB>
static hipError_t go_wd_mb(const Problems &ps, int nprob, hipStream_t st) {
  int maxt = 0;
  for (int i = 0; i < nprob; ++i) {
    const int t = ((ps.p[i].M + 32 * MB - 1) / (32 * MB)) * ((ps.p[i].N + kWdCols - 1) / kWdCols);
    maxt = t > maxt ? t : maxt;
  }
  if (maxt == 0) return hipSuccess;
  constexpr int D = 8;  // ring depth: two stages of a wave's k-steps
  hipLaunchKernelGGL((gemm_wd_kernel<AT, EPI, D, MB>), dim3(maxt, 1, nprob), dim3(kWdThreads), 0, st, ps);
  return hipGetLastError();
}

// Rows per tile, 32 MB: the fewest rounds of 256 workgroups (one per compute unit), weighted with
// what a round of such tiles costs against one of MB = 1.  us for MB = 1, 2, 3 (a graph of 20
// launches): bf16 rows 768 x 5120 x 1024 18.7 15.8 18.9, 1024 x 5120 x 1024 23.8 20.8 20.2, 768 x 3584 x 2048
// 24.9 21.8 19.9, 768 x 3072 x 1024 13.7 13.1 12.4, 2048 x 10240 x 2048 162 125 110.  fp32 rows, twice
// the bytes and four conversions a vector, do better in the smaller tiles: 1536 x 3072 x 1024 31.2 27.4
// 30.5, 896 x 5120 x 1024 27.1 24.1 28.2, 768 x 6144 x 512 17.0 16.5 19.0.  Deep products of many fp32 rows
// read those from beyond the L2, once per tile column; tiles of 128 rows halve the weights' share
// (MB = 2 / 4: 2048 x 2048 x 2048 44.7 / 33.1, 2048 x 6144 x 2048 125 / 94, 1792 x 3584 x 2048 69.6 / 59.8, 3072 x
// 3584 x 2048 116 / 105; but 1024 x 3584 x 2048 30.4 / 30.7, 512 x 6144 x 2048 26.7 / 30.1, and 2048 x 1024 x 2048,
// whose 128 tiles leave half of the units idle, 26.9 / 31.1).
//
// At 768 rows 1024 k cost 5.9 us of 3072 columns and 8.7 of 5120 (32 and 37 bytes of operands a
// clock and unit); 6.5 and 7.5 us of a launch do not depend on the depth (row indices, first stage,
// exchange, stores, the last tiles).
template <typename AT, int EPI>
static hipError_t go_wd(const Problems &ps, int nprob, hipStream_t st) {
  constexpr bool F32 = sizeof(AT) == 4;
  static const double cost[3] = {1.0, F32 ? 1.05 : 1.25, F32 ? 1.8 : 1.6};
  for (int i = 0; i < nprob; ++i) {
    const GemmProblem &p = ps.p[i];
    if (p.ldb % kWdStageK != 0 || p.K > p.ldb || p.K % 8 != 0) return hipErrorInvalidValue;
  }
  if constexpr (F32)
    if (ps.p[0].K >= 2048 && ps.p[0].M >= 1792 && (long)((ps.p[0].M + 127) / 128) * ((ps.p[0].N + 127) / 128) >= 224)
      return go_wd_mb<AT, EPI, 4>(ps, nprob, st);
  int best = 1;
  double bc = 0;
  for (int mb = 1; mb <= 3; ++mb) {
    long t = 0;
    for (int i = 0; i < nprob; ++i)
      t += (long)((ps.p[i].M + 32 * mb - 1) / (32 * mb)) * ((ps.p[i].N + kWdCols - 1) / kWdCols);
    const double c = cost[mb - 1] * (double)((t + 255) / 256);
    if (mb == 1 || c <= bc) {
      bc = c;
      best = mb;
    }
  }
  switch (best) {
    case 1: return go_wd_mb<AT, EPI, 1>(ps, nprob, st);
    case 2: return go_wd_mb<AT, EPI, 2>(ps, nprob, st);
    default: return go_wd_mb<AT, EPI, 3>(ps, nprob, st);
  }
}

// ---------------------------------------------------------------------------------------
// fp32 operands: (BLK TA) x (BLK TB) output tiles, each computed by S waves of one workgroup that
// split its k-steps and add their partial sums through LDS; both operands straight from global
// memory (at fp32 rates the MFMAs need only a few bytes per cycle, so no LDS staging).
//
// BLK = 16: v_mfma_f32_16x16x4_f32 takes one fp32 per lane per operand, A lane l holding row
// l % 16 and k (l / 16), B lane l column l % 16 and k (l / 16).  A 16-byte vector per lane holds
// the k quadruple 4 (l / 16) + e, e < 4, of one 16-k step and feeds MFMA e, so the four MFMAs of
// a step cover its 16 k once (the same assignment on both operands).
// BLK = 32: v_mfma_f32_32x32x2f32, A lane l holding row l % 32 and k (l / 32); a 16-byte vector
// holds k = 4 (l / 32) + e of one 8-k step, again feeding MFMA e.  This form sustains a higher
// fraction of the matrix core's rate (86% against 74% in pure-MFMA loops, about 5% more in this
// kernel), at the price of coarser tiles.
// The weights are packed in the order of their form (mt_load_weights picks it per matrix): for
// BLK-column block nb and step ks, 64 lanes x 16 bytes at ((nb * KS + ks) * 64 + lane) * 16
// (KS = K_pad / (256 / BLK)).  The activation vector of lane l is A[row][step k0 + its k
// quadruple], one 16-byte load.  Both come through a register ring refilled D steps ahead.
//
// Tile shape and split are chosen per launch (go_f32) so that the waves spread evenly over the
// chip's 1024 SIMDs: at these shapes the time is set by the SIMD with the most work.
template <int BLK>
struct F32Form {
  static constexpr int KSTEP = 256 / BLK;   // k per step (one 16-byte vector per lane)
  static constexpr int NACC = BLK * BLK / 64;  // accumulator registers per lane per block
  static constexpr int HALF = 64 / BLK;     // lane groups of the k quadruples
};

// WIDE: rows by 64-bit addresses instead of a buffer view, whose offsets have 32 bits (go_f32).
template <int BLK, int TA, int TB, int S, int EPI, int D, int U, bool WIDE = false>
__global__ __launch_bounds__(256) void gemm_f32_kernel(Problems probs) {
  using F = F32Form<BLK>;
  typedef __attribute__((__vector_size__(F::NACC * sizeof(float)))) float accv;
  constexpr int TPB = 4 / S;  // tiles per workgroup (four waves)
  __shared__ __attribute__((aligned(16))) float red[S > 1 ? TPB * (S - 1) * TA * TB * F::NACC * 64 : 1];
  const GemmProblem &P = probs.p[blockIdx.z];
  const int M = pin_s(P.M), N = pin_s(P.N), K = pin_s(P.K), lda = pin_s(P.lda), ldc = pin_s(P.ldc);
  const int KSp = pin_s(P.ldb) / F::KSTEP;
  const int tilesM = (M + BLK * TA - 1) / (BLK * TA);
  const int tilesN = (N + BLK * TB - 1) / (BLK * TB);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = wave % S, slot_t = wave / S;
  const int tile = xcd_remap(blockIdx.x, gridDim.x) * TPB + slot_t;
  // rows counted on the device, when given, bound the rows read and stored
  const int *const mdp = pin_s(P.m_dev);
  int Mv = M;
  if (mdp) {
    const int md = *(const __attribute__((address_space(1))) int *)mdp;
    Mv = md < M ? md : M;
  }
  // a wave without a tile still takes part in the workgroup's barrier below
  const bool has_tile = tile < tilesM * tilesN;
  const int tl = has_tile ? tile : 0;
  int tm = tl % tilesM, tn = tl / tilesM;  // neighbours share a weight panel
  if (mdp && has_tile) counted_tile(blockIdx.x * TPB + slot_t, tilesM, tilesN, TPB, tm, tn);
  const int m0 = tm * BLK * TA, n0 = tn * BLK * TB;
  const bool live = has_tile && m0 < Mv;
  // without a split there is no barrier, so a wave without a tile (or whose rows all lie past
  // the device count) ends here; with one it computes a stand-in tile for the barrier's sake
  if constexpr (S == 1)
    if (!live) return;
  const int lr = lane & (BLK - 1), lk = (lane / BLK) * 4;
  const int ks_begin = part * (KSp / S), ks_end = ks_begin + KSp / S;

  // activation rows of this lane (gathered, clamped; rows past M read row 0, never stored), as
  // byte offsets into a buffer view of A (at most 2^32 - 1 bytes)
  const __amdgpu_buffer_rsrc_t ars =
      __builtin_amdgcn_make_buffer_rsrc((void *)P.A, 0, (int)((uint32_t)P.a_rows * (uint32_t)lda * 4u), 0x00020000);
  typename std::conditional<WIDE, const char *, uint32_t>::type a_off[TA];
  // EPI_SCATTER: the output row of row BLK i + lr of the tile, kept for the epilogue
  int out_row[EPI == EPI_SCATTER ? TA : 1];
  if constexpr (EPI == EPI_SCATTER) {
#pragma unroll
    for (int i = 0; i < TA; ++i) {
      const int m = m0 + BLK * i + lr;
      out_row[i] = P.o_idx && live && m < Mv ? P.o_idx[m] : 0;
    }
  }
#pragma unroll
  for (int i = 0; i < TA; ++i) {
    const int m = m0 + BLK * i + lr;
    int src = m < Mv ? m : 0;
    if (live && P.a_idx && m < Mv) {
      src = P.a_idx[m];
      if (src < 0 || src >= P.a_rows) {
        if (P.err) atomicOr(P.err, 1 << P.err_bit);
        src = src < 0 ? 0 : P.a_rows - 1;
      }
    }
    if (EPI == EPI_SCATTER && !P.o_idx) out_row[EPI == EPI_SCATTER ? i : 0] = src;
    if constexpr (WIDE) a_off[i] = (const char *)P.A + (size_t)src * lda * 4;
    else a_off[i] = (uint32_t)src * (uint32_t)lda * 4u;
  }
  // the view covers the column blocks that exist (the packing pads N further, to N_pad, but a
  // tile may reach past even that): fragments of blocks beyond N read as zero and their
  // columns are never stored
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc((void *)P.Bp, 0, (N + BLK - 1) / BLK * KSp * 1024, 0x00020000);
  const int wvo = lane * 16;
  const int wb0 = (n0 / BLK) * KSp * 1024;
  const int kslast = ks_end - 1;

  struct Slot {
    u32x4 a[TA], b[TB];
  };
  Slot ring[D];
  auto fetch = [&](int ks, Slot &r) {
    const int kc = ks < kslast ? ks : kslast;  // clamped: in bounds, never used
    int k = kc * F::KSTEP + lk;
    k = k < K ? k : K - 4;  // past K: the row's last vector (it meets zero weights)
#pragma unroll
    for (int i = 0; i < TA; ++i) {
      if constexpr (WIDE) r.a[i] = *(const u32x4 *)(a_off[i] + (size_t)k * 4);
      else r.a[i] = __builtin_amdgcn_raw_buffer_load_b128(ars, (int)(a_off[i] + (uint32_t)k * 4u), 0, 0);
    }
#pragma unroll
    for (int j = 0; j < TB; ++j) r.b[j] = __builtin_amdgcn_raw_buffer_load_b128(wrs, wvo, wb0 + (j * KSp + kc) * 1024, 0);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) fetch(ks_begin + d, ring[d]);

  accv acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int r = 0; r < F::NACC; ++r) acc[i][j][r] = 0.f;

  // the ring index of step ks is (ks - ks_begin) % D; the loop advances U steps per iteration
  // ((KSp / S) % U == 0, U a multiple of D).  The compiler drains the memory counter at the loop
  // header, so the longer the body, the rarer the drain.
  for (int ks0 = ks_begin; ks0 < ks_end; ks0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int d = u % D;
      float fa[TA][4], fb[TB][4];
#pragma unroll
      for (int i = 0; i < TA; ++i) __builtin_memcpy(fa[i], &ring[d].a[i], 16);
#pragma unroll
      for (int j = 0; j < TB; ++j) __builtin_memcpy(fb[j], &ring[d].b[j], 16);
      // element e of every vector feeds MFMA e; the TA x TB accumulators alternate between
      // dependent MFMAs
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j) {
            if constexpr (BLK == 16)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
          }
      // the refill of a slot goes behind the MFMAs that read it (hoisted above them, its loads
      // would need fresh registers and a wait for every load in flight)
      __builtin_amdgcn_sched_barrier(0);
      fetch(ks0 + u + D, ring[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- the split's partial sums: parts 1.. write theirs, part 0 adds them in part order ----
  if constexpr (S > 1) {
    constexpr int PER = TA * TB * F::NACC;
    if (part > 0) {
      float *mine = red + (size_t)((slot_t * (S - 1) + part - 1) * PER) * 64;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
          for (int r = 0; r < F::NACC; ++r) mine[((i * TB + j) * F::NACC + r) * 64 + lane] = acc[i][j][r];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int q = 1; q < S; ++q) {
      const float *o = red + (size_t)((slot_t * (S - 1) + q - 1) * PER) * 64;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
          for (int r = 0; r < F::NACC; ++r) acc[i][j][r] += o[((i * TB + j) * F::NACC + r) * 64 + lane];
    }
  }
  if (!live) return;

  // ---- epilogue: lane holds D[row][col = lane % BLK] of each block, row = 4 * (lane / 16) + r
  // (BLK 16) or 8 * (r / 4) + 4 * (lane / 32) + r % 4 (BLK 32); the bias values are loaded before
  // any store and waited for once ----
  const int obf = pin_s(P.out_bf16);
  const float *const biasp = pin_s(P.bias);
  char *const outp = (char *)pin_s(P.out);
  float bias[TB];
#pragma unroll
  for (int j = 0; j < TB; ++j) {
    const int col = n0 + BLK * j + lr;
    bias[j] = biasp ? ((const __attribute__((address_space(1))) float *)biasp)[col < N ? col : N - 1] : 0.f;
  }
  // row of accumulator r within its block
  auto row_of = [&](int r) { return BLK == 16 ? (lane >> 4) * 4 + r : 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  const int rows = Mv - m0 < BLK * TA ? Mv - m0 : BLK * TA;
  OutRows out_rows{m0, true};
  if constexpr (EPI == EPI_SCATTER) {
    int last = 0;
#pragma unroll
    for (int i = 0; i < TA; ++i)
      last = (rows - 1) / BLK == i ? __builtin_amdgcn_readlane(out_row[i], (rows - 1) & (BLK - 1)) : last;
    out_rows = out_rows_of(out_row[0], last, rows);
  }
  const TileOut to(outp, obf, out_rows.first, rows, ldc);
  auto epilogue = [&](auto bf) {
    constexpr bool BF = decltype(bf)::value;
    if (EPI == EPI_SCATTER && !out_rows.run) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int r = 0; r < F::NACC; ++r) {
          const int o = __shfl(out_row[EPI == EPI_SCATTER ? i : 0], row_of(r), 64);
          if (BLK * i + row_of(r) >= rows) continue;
#pragma unroll
          for (int j = 0; j < TB; ++j) {
            const int col = n0 + BLK * j + lr;
            if (col >= N) continue;
            const float v = acc[i][j][r] + bias[j];
            if constexpr (BF)
              ((__attribute__((address_space(1))) bf16 *)outp)[(size_t)o * ldc + col] = to_bf16(v);
            else
              ((__attribute__((address_space(1))) float *)outp)[(size_t)o * ldc + col] = v;
          }
        }
    } else {
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const int vo = to.lane_offset<BF>(BLK == 16 ? (lane >> 4) * 4 : 4 * (lane >> 5), n0 + BLK * j + lr, N);
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
          for (int r = 0; r < F::NACC; ++r) {
            float v = acc[i][j][r] + bias[j];
            if (EPI == EPI_TANH) v = tanh_fast(v);
            to.store<BF>(v, vo, BLK * i + (BLK == 16 ? r : 8 * (r >> 2) + (r & 3)));
          }
      }
    }
  };
  if (obf)
    epilogue(std::integral_constant<bool, true>{});
  else
    epilogue(std::integral_constant<bool, false>{});
}

template <int BLK, int TA, int TB, int S, int EPI>
static hipError_t go_f32_t(const Problems &ps, int nprob, hipStream_t st) {
  int maxw = 0;
  bool deep = TA + TB <= 4;  // ring depth in steps: 8 for small tiles when it divides the steps
  bool long16 = true;        // 16 steps per loop iteration
  for (int i = 0; i < nprob; ++i) {
    const int w = ((ps.p[i].M + BLK * TA - 1) / (BLK * TA)) * ((ps.p[i].N + BLK * TB - 1) / (BLK * TB));
    maxw = w > maxw ? w : maxw;
    const int steps = ps.p[i].ldb / F32Form<BLK>::KSTEP / S;
    deep = deep && steps % 8 == 0;
    long16 = long16 && steps % 16 == 0;
  }
  if (maxw == 0) return hipSuccess;
  constexpr int TPB = 4 / S;
  const dim3 grid((maxw + TPB - 1) / TPB, 1, nprob);
  if constexpr (TA + TB <= 4) {
    if (deep && long16) hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, S, EPI, 8, 16>), grid, dim3(256), 0, st, ps);
    else if (deep) hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, S, EPI, 8, 8>), grid, dim3(256), 0, st, ps);
    else hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, S, EPI, 4, 4>), grid, dim3(256), 0, st, ps);
  } else {
    if (long16) hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, S, EPI, 4, 16>), grid, dim3(256), 0, st, ps);
    else hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, S, EPI, 4, 4>), grid, dim3(256), 0, st, ps);
  }
  return hipGetLastError();
}

// Tile shapes per form: TA x TB blocks of BLK x BLK, k split S.
struct F32Shape {
  int ta, tb, s;
};
static const F32Shape kShapes16[] = {{3, 3, 1}, {3, 4, 1}, {3, 5, 1}, {3, 2, 1}, {2, 4, 1}, {1, 2, 1},
                                     {3, 3, 2}, {3, 4, 2}, {3, 5, 2}, {3, 2, 2}, {1, 2, 4}};
static const F32Shape kShapes32[] = {{1, 3, 1}, {2, 2, 1}, {1, 4, 1}, {2, 3, 1}, {1, 2, 1}, {1, 2, 2}};

// Cost of the best shape of a form for (rows, columns, k-steps): the SIMD with the most work
// receives ceil(waves / 1024) waves of TA * TB / S block-steps each, counted in 16x16x4 MFMA
// time (a 32 x 32 block-step is four 16 x 16 ones at the 32x32x2 form's better rate: 0.95 of
// their time in this kernel at the decoder's shapes).  Also measured there: a k split costs a little more than the same
// work unsplit (its partial sums and the second ring fill), fewer than 6 accumulators leave
// dependent 16x16x4 MFMAs too close together, and between equal costs the shape with more
// waves hides latency better.  A split needs at least 4 steps per part.
static double f32_best(int blk, const long *rows, const long *cols, int nprob, int steps, int *which) {
  const F32Shape *sh = blk == 16 ? kShapes16 : kShapes32;
  const int n = blk == 16 ? (int)(sizeof(kShapes16) / sizeof(kShapes16[0])) : (int)(sizeof(kShapes32) / sizeof(kShapes32[0]));
  double best = -1.0;
  long best_w = 0;
  *which = 0;
  for (int s = 0; s < n; ++s) {
    const F32Shape &h = sh[s];
    if (steps / h.s < 4 || steps % (4 * h.s) != 0) continue;
    long w = 0;
    for (int i = 0; i < nprob; ++i) w += ((rows[i] + blk * h.ta - 1) / (blk * h.ta)) * ((cols[i] + blk * h.tb - 1) / (blk * h.tb));
    w *= h.s;
    const long per = (w + 1023) / 1024;
    double cost = (double)per * h.ta * h.tb / h.s * (h.s > 1 ? 1.05 : 1.0);
    if (blk == 16) cost /= h.ta * h.tb >= 6 ? 1.0 : 0.6;
    else cost *= 4 * 0.95;
    if (best < 0 || cost < best - 1e-9 || (cost < best + 1e-9 && w > best_w)) {
      best = cost;
      best_w = w;
      *which = s;
    }
  }
  return best;
}

int gemm_f32_weight_block(long rows, long N, long K) {
  const long kp = (K + 63) / 64 * 64;
  int w16, w32;
  const double c16 = f32_best(16, &rows, &N, 1, (int)(kp / 16), &w16);
  const double c32 = f32_best(32, &rows, &N, 1, (int)(kp / 8), &w32);
  return (c32 >= 0 && c32 < c16) ? 32 : 16;
}

// Rows that span 4 GiB or more (a large batch's context, states or embeddings) lie beyond what the
// buffer view's 32-bit offsets reach: one tile shape of each form with 64-bit row addresses.
template <int BLK, int TA, int TB, int EPI>
static hipError_t go_f32_wide(const Problems &ps, int nprob, hipStream_t st) {
  long maxw = 0;
  for (int i = 0; i < nprob; ++i)
    maxw = std::max(maxw, (long)((ps.p[i].M + BLK * TA - 1) / (BLK * TA)) * ((ps.p[i].N + BLK * TB - 1) / (BLK * TB)));
  if (maxw == 0) return hipSuccess;
  hipLaunchKernelGGL((gemm_f32_kernel<BLK, TA, TB, 1, EPI, 4, 4, true>), dim3((unsigned)((maxw + 3) / 4), 1, nprob),
                     dim3(256), 0, st, ps);
  return hipGetLastError();
}

template <int EPI>
static hipError_t go_f32(const Problems &ps, int nprob, hipStream_t st) {
  const int blk = ps.p[0].wblk == 32 ? 32 : 16;
  int minsteps = 1 << 30;
  bool wide = false;
  long rows[2], cols[2];
  for (int i = 0; i < nprob; ++i) {
    const GemmProblem &p = ps.p[i];
    if (p.ldb % 64 != 0 || p.K > p.ldb || p.K % 4 != 0 || p.lda % 4 != 0) return hipErrorInvalidValue;
    if ((p.wblk == 32 ? 32 : 16) != blk) return hipErrorInvalidValue;
    const int steps = p.ldb / F32Form<16>::KSTEP * (blk == 32 ? 2 : 1);
    minsteps = steps < minsteps ? steps : minsteps;
    rows[i] = p.M;
    cols[i] = p.N;
    wide = wide || (unsigned long long)p.a_rows * p.lda * 4 > 0xffffffffull;
  }
  if (wide) return blk == 32 ? go_f32_wide<32, 2, 2, EPI>(ps, nprob, st) : go_f32_wide<16, 3, 3, EPI>(ps, nprob, st);
  int bi = 0;
  if (f32_best(blk, rows, cols, nprob, minsteps, &bi) < 0) return hipErrorInvalidValue;
  if (blk == 32) {
    switch (bi) {
      case 0: return go_f32_t<32, 1, 3, 1, EPI>(ps, nprob, st);
      case 1: return go_f32_t<32, 2, 2, 1, EPI>(ps, nprob, st);
      case 2: return go_f32_t<32, 1, 4, 1, EPI>(ps, nprob, st);
      case 3: return go_f32_t<32, 2, 3, 1, EPI>(ps, nprob, st);
      case 4: return go_f32_t<32, 1, 2, 1, EPI>(ps, nprob, st);
      default: return go_f32_t<32, 1, 2, 2, EPI>(ps, nprob, st);
    }
  }
  switch (bi) {
    case 0: return go_f32_t<16, 3, 3, 1, EPI>(ps, nprob, st);
    case 1: return go_f32_t<16, 3, 4, 1, EPI>(ps, nprob, st);
    case 2: return go_f32_t<16, 3, 5, 1, EPI>(ps, nprob, st);
    case 3: return go_f32_t<16, 3, 2, 1, EPI>(ps, nprob, st);
    case 4: return go_f32_t<16, 2, 4, 1, EPI>(ps, nprob, st);
    case 5: return go_f32_t<16, 1, 2, 1, EPI>(ps, nprob, st);
    case 6: return go_f32_t<16, 3, 3, 2, EPI>(ps, nprob, st);
    case 7: return go_f32_t<16, 3, 4, 2, EPI>(ps, nprob, st);
    case 8: return go_f32_t<16, 3, 5, 2, EPI>(ps, nprob, st);
    case 9: return go_f32_t<16, 3, 2, 2, EPI>(ps, nprob, st);
    default: return go_f32_t<16, 1, 2, 4, EPI>(ps, nprob, st);
  }
}

// Few rows take the split-depth kernel of mt_gemm_small.hip, counted in its workgroups (32 rows x
// one column block).  Where the lines lie (us, tiles above against small; 5120 x 1024 s1 product,
// 3584 x 2048 context product, 3072 x 1024 recurrent product):
//  * bf16, 512 workgroups: s1 at 96 rows (480) 8.3 / 6.0 and 128 (640) 8.4 / 7.7, context at 128
//    (448) 12.0 / 8.4 and 256 (896) 12.4 / 13.1, recurrent at 128 (384) 8.6 / 6.5, two recurrent
//    products at 64 rows (384) 8.5 / 6.9 and at 96 (576) 8.7 / 9.0;
//  * fp32 in the 32-column packing, whose tiles are the coarser ones, 896: context at 5 rows 38.5
//    / 7.9, at 128 (896) 39.6 / 29.1, at 256 40.0 / 45.9;
//  * fp32 in the 16-column packing, 256 up to 32 rows, else 512: recurrent at 32 rows (192) 7.1 / 6.7,
//    at 64 (384) 10.6 / 9.8, sample at 128 (512) 8.0 / 6.0, but s1 at 5 rows (320) 6.7 / 8.1 and at 40
//    (640) 10.8 / 13.1, two recurrent products at 5 (384) 7.2 / 8.2.  More than 256 workgroups are two
//    rounds of the units, which only pays where the tiles are poor: at K = 64 768 x 256 (384) 3.9 /
//    4.3 and at K = 256 two of 65 x 768 (288) 4.1 / 5.0 the tiles stay, at K = 128 they cannot split the
//    depth (320 x 512 6.7 / 4.7), from K = 512 to 2048 256 x 1024 x 1024 (512) 10.7 / 9.6, at 4096 128 x 2048
//    (512) 27.3 / 29.4.
static bool small_rows(int bf16_mma, const Problems &ps, int nprob) {
  long wg = 0;
  for (int i = 0; i < nprob; ++i) {
    const GemmProblem &p = ps.p[i];
    if (p.K % 16 != 0 || p.M < 1 || p.wblk != ps.p[0].wblk) return false;
    wg += (long)((p.M + 31) / 32) * ((p.N + (bf16_mma ? 31 : 15)) / (bf16_mma ? 32 : 16));
  }
  const int M = ps.p[0].M, K = ps.p[0].K;
  if (bf16_mma) return wg <= 512;
  if (ps.p[0].wblk == 32) return wg <= 896;
  return wg <= (M > 32 && K >= 128 && K != 256 && K <= 2048 ? 512 : 256);
}

hipError_t launch_gemm(int bf16_mma, const GemmProblem *probs, int nprob, Epilogue epi, hipStream_t st) {
  Problems ps{};
  for (int i = 0; i < nprob; ++i) {
    ps.p[i] = probs[i];
    if (probs[i].a_bf16 != probs[0].a_bf16 || (probs[i].a_bf16 && !bf16_mma)) return hipErrorInvalidValue;
    if (epi == EPI_SCATTER && !probs[i].a_idx) return hipErrorInvalidValue;
  }
  if (small_rows(bf16_mma, ps, nprob)) return launch_gemm_small(bf16_mma, ps, nprob, epi, st);
  if (!bf16_mma) {
    if (epi == EPI_SCATTER) return go_f32<EPI_SCATTER>(ps, nprob, st);
    return epi == EPI_TANH ? go_f32<EPI_TANH>(ps, nprob, st) : go_f32<EPI_STORE>(ps, nprob, st);
  }
  if (epi == EPI_SCATTER)
    return probs[0].a_bf16 ? go_wd<bf16, EPI_SCATTER>(ps, nprob, st) : go_wd<float, EPI_SCATTER>(ps, nprob, st);
  if (probs[0].a_bf16)
    return epi == EPI_TANH ? go_wd<bf16, EPI_TANH>(ps, nprob, st) : go_wd<bf16, EPI_STORE>(ps, nprob, st);
  return epi == EPI_TANH ? go_wd<float, EPI_TANH>(ps, nprob, st) : go_wd<float, EPI_STORE>(ps, nprob, st);
}

}  // namespace mt
