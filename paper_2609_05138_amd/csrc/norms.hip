// Codebook norms ||w_j||^2 = sum_f W[f][j]^2 (paper, Section 3; the "norms"
// pass of Table 4).  One streaming pass over the feature-major codebook:
// each lane owns the neurons of one 128-bit load per row (four fp32 or eight
// fp16 weights), L lanes cover a row's share of the workgroup, and the waves and
// the 64 / L rows of a wave's load split the rows; squares are exact in fp64 and
// accumulated there in a fixed order, so the result is deterministic and rounded
// to fp32 exactly once.  For an fp16 codebook the norms are those of the stored
// (rounded) weights.  Bound: HBM read bandwidth (4 or 2 B per weight), given
// enough workgroups; a narrow map has few full-width ones, so L shrinks
// with N (rows are then read 256 or 64 bytes at a time).
#include "common.h"

namespace som {
namespace {

constexpr int kChains = 4;      // independent fp64 chains per lane (loads in flight)

typedef _Float16 nh8 __attribute__((ext_vector_type(8)));

template <typename WT>
struct NormLoad;
template <>
struct NormLoad<float> {
  static constexpr int kE = 4;
  static __device__ __forceinline__ void get(const float* p, double (&v)[4]) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
  }
};
template <>
struct NormLoad<_Float16> {
  static constexpr int kE = 8;
  static __device__ __forceinline__ void get(const _Float16* p, double (&v)[8]) {
    const nh8 x = *reinterpret_cast<const nh8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<double>(x[e]);
  }
};

// L lanes per row and V waves: row classes V * 64 / L.
template <typename WT, int L, int V>
__global__ void __launch_bounds__(V * 64)
k_norms(const WT* __restrict__ W, int64_t F, int64_t N, int64_t ldw, float* __restrict__ norms) {
  constexpr int E = NormLoad<WT>::kE;
  constexpr int kRows = 64 / L;            // rows per load instruction
  constexpr int64_t kClasses = V * kRows;
  __shared__ double part[V][L][E];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int piece = lane % L;
  const int64_t col = (static_cast<int64_t>(blockIdx.x) * L + piece) * E;  // first of E neurons
  double s[kChains][E] = {};
  // only groups holding a neuron j < N are read: no load leaves
  // [0, round_up(N, E)) of its row
  if (col < N) {
    const WT* base = W + col;
    int64_t f = wave * kRows + lane / L;
    // the class's rows go to chains 0..3 in turn, in increasing f per chain
    for (; f + (kChains - 1) * kClasses < F; f += kChains * kClasses) {
      double v[kChains][E];
#pragma unroll
      for (int c = 0; c < kChains; ++c) NormLoad<WT>::get(base + (f + c * kClasses) * ldw, v[c]);
#pragma unroll
      for (int c = 0; c < kChains; ++c)
#pragma unroll
        for (int e = 0; e < E; ++e) s[c][e] = fma(v[c][e], v[c][e], s[c][e]);
    }
    // at most three rows remain, one per chain
#pragma unroll
    for (int c = 0; c < kChains - 1; ++c) {
      const int64_t fr = f + c * kClasses;
      if (fr < F) {
        double v[E];
        NormLoad<WT>::get(base + fr * ldw, v);
#pragma unroll
        for (int e = 0; e < E; ++e) s[c][e] = fma(v[e], v[e], s[c][e]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    double t = (s[0][e] + s[1][e]) + (s[2][e] + s[3][e]);
#pragma unroll
    for (int off = L; off < 64; off <<= 1) t += __shfl_xor(t, off, 64);   // the wave's rows of this column
    if (lane < L) part[wave][piece][e] = t;
  }
  __syncthreads();
  if (wave == 0 && lane < L && col < N) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      double t = part[0][lane][e];
#pragma unroll
      for (int w = 1; w < V; ++w) t += part[w][lane][e];
      if (col + e < N) norms[col + e] = static_cast<float>(t);
    }
  }
}

// Lanes per row: 64 where that gives a workgroup per CU, else 16 where that
// gives one for every other CU, else 4.  F = 20,000, fp32: N = 1,024 took 360 us
// with four 64-lane workgroups and 34 us with 64 four-lane ones, N = 16,384
// 420 us (64 workgroups) and 213 us (256 of 16 lanes, 6.2 TB/s); N = 65,536 keeps
// 64 lanes (830 us, 6.3 TB/s).  fp16, N = 65,536: 1,337 us with 128 workgroups of
// 64 lanes.
constexpr int64_t kNormGroups64 = 256, kNormGroups16 = 128;

template <typename WT>
void norms_of(const void* W, int64_t F, int64_t N, int64_t ldw, float* norms, hipStream_t stream) {
  constexpr int64_t E = NormLoad<WT>::kE;
  const WT* w = static_cast<const WT*>(W);
  const int64_t loads = (N + E - 1) / E;   // 128-bit loads per row
  auto groups = [&](int64_t lanes) { return static_cast<uint32_t>((loads + lanes - 1) / lanes); };
  if (groups(64) >= kNormGroups64)
    hipLaunchKernelGGL((k_norms<WT, 64, 8>), dim3(groups(64)), dim3(8 * 64), 0, stream, w, F, N, ldw, norms);
  else if (groups(16) >= kNormGroups16)
    hipLaunchKernelGGL((k_norms<WT, 16, 16>), dim3(groups(16)), dim3(16 * 64), 0, stream, w, F, N, ldw, norms);
  else
    hipLaunchKernelGGL((k_norms<WT, 4, 16>), dim3(groups(4)), dim3(16 * 64), 0, stream, w, F, N, ldw, norms);
}

}  // namespace

hipError_t launch_norms(const void* W, int weights, int64_t F, int64_t N, int64_t ldw, float* norms,
                        hipStream_t stream) {
  if (weights == kWeightsF16)
    norms_of<_Float16>(W, F, N, ldw, norms, stream);
  else
    norms_of<float>(W, F, N, ldw, norms, stream);
  return hipGetLastError();
}

}  // namespace som
