// Definitions shared by the vocabulary projection kernels (single model and fused ensemble):
// tile and list sizes, the wave shape of a workgroup, and the k-step of each operand type.
#pragma once
#include "mt_internal.h"

namespace mt {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kVRows = 64;       // vocabulary rows per wave tile (2 MFMA blocks)
constexpr int kLists = 8;        // candidate buffers per (hypothesis, chunk): 2 lane halves x 4 runs
constexpr int kSampleMax = 2048;  // vocabulary entries of the threshold pass
constexpr float kLog2e = 1.4426950408889634f;

// Hypothesis columns per wave: at most WMAX (64: two 32-column MFMA blocks); a workgroup of HB
// columns runs HB/WH waves per vocabulary run on the same tiles.
template <typename CT, int HB, int WMAX = 64>
struct VShape {
  static constexpr int WH = HB >= WMAX ? WMAX : HB;  // columns per wave
  static constexpr int HBW = WH / 32;            // 32-column MFMA blocks per wave
  static constexpr int NW = 4 * (HB / WH);       // waves per workgroup
  static constexpr int NT = 64 * NW;             // threads per workgroup
};

template <typename CT>
struct VCfg;
template <>
struct VCfg<bf16> {
  static constexpr int KV = 16;  // k per 16-byte vector step
};
template <>
struct VCfg<float> {
  static constexpr int KV = 8;
};

// Stages rows h0 .. h0 + HB - 1 of t [M][E] into LDS rows of rowb bytes (zero beyond M) by NT
// threads.  UB 16-byte vectors per thread are requested together: one load, wait and store after
// another cost a round trip each, 16 of them for the 128 bf16 rows of E = 512 and 32 for 64 fp32
// rows (traces of the pass: bf16 768 x 50k 46.4 -> 44.9 us, 1024 x 50k 62.2 -> 60.3; fp32 40 x 50k 44.0 ->
// 43.0).  VPR: vectors per row if known at compile time, else 0.
template <int HB, int NT, int VPR>
__device__ __forceinline__ void stage_rows(char *lds, int rowb, const char *t, int h0, int M, int vpr_) {
  constexpr int UB = 8;
  const int vpr = VPR > 0 ? VPR : vpr_;
  const int total = HB * vpr;
  for (int base = threadIdx.x; base < total; base += NT * UB) {
    v4u v[UB];
    int r[UB], c[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int idx = base + u * NT;
      r[u] = idx / vpr;
      c[u] = idx - r[u] * vpr;
      const int h = h0 + r[u] < M ? h0 + r[u] : M - 1;  // past M or the last vector: in range, not kept
      v[u] = *(const v4u *)(t + ((size_t)h * vpr + c[u]) * 16);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if (h0 + r[u] >= M) v[u] = v4u{0u, 0u, 0u, 0u};
      if (r[u] < HB) *(v4u *)(lds + r[u] * rowb + c[u] * 16) = v[u];
    }
  }
}

}  // namespace mt
