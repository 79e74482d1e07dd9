// Batch-SOM update after the search (paper, Section 3: the best-matching
// unit and its neighbours are updated; Section 6.1, Table 4: a scatter into
// accumulators, a neighbourhood blur, a write-back, then the norms refresh).
// The neighbourhood is the reading stated in include/som.h: a Gaussian of
// width sigma on the rows x cols map grid, truncated at R = ceil(3 sigma) along
// each axis, hence separable into a row blur and a column blur.
//
//  k_accumulate   one wave per document: acc[f][bmu] += 1 for its features and
//                 count[bmu] += 1, as uint32 atomics (exact, order-free)
//  k_taps         g[k] = exp(-k^2 / (2 sigma^2)) for k = 0..R, in fp64, rounded
//                 to fp32 once
//  k_blur_rows    some grid rows of one feature per workgroup, staged in LDS:
//                 t[r][c] = sum_{k=-R..R} g[|k|] acc[r][c+k]  (fixed tap order)
//  k_blur_cols    a strip of 32 or 16 columns of one feature per workgroup, staged
//                 in LDS: v[r][c] = sum_k g[|k|] t[r+k][c]; then either the
//                 blurred counts (den) or the write-back W = v / den where
//                 den > 0 (other units keep their weights)
//  k_blur_stream  R <= 16: one wave per 64-column strip of a feature plane
//                 walks down the rows: row pass from an LDS row buffer,
//                 column pass from an LDS ring of the last 2R+1 results, the
//                 same sums term for term; the accumulators are read once and
//                 the codebook written once.
// Bound: HBM (the two-pass path streams 16 B per element, the streaming one
// 8 B plus a halo of 2R/64 of the reads).
#include "common.h"

namespace som {
namespace {

constexpr int kStrip = 32;  // columns per column-blur workgroup (128 B of fp32)

__global__ void __launch_bounds__(256)
k_accumulate(const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices, int64_t B,
             const int32_t* __restrict__ bmu, int64_t F, int64_t N, uint32_t* __restrict__ acc,
             int64_t ld_acc, uint32_t* __restrict__ count) {
  const int lane = threadIdx.x & 63;
  const int64_t d = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (d >= B) return;
  const int64_t b = bmu[d];
  if (b < 0 || b >= N) return;  // not a unit of this map: ignored
  const int32_t e0 = indptr[d], e1 = indptr[d + 1];
  for (int32_t e = e0 + lane; e < e1; e += 64) {
    const int64_t f = indices[e];
    if (f >= 0 && f < F) atomicAdd(acc + f * ld_acc + b, 1u);
  }
  if (lane == 0) atomicAdd(count + b, 1u);
}

__global__ void k_taps(double sigma, int R, float* __restrict__ g) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > R) return;
  g[k] = sigma > 0 ? static_cast<float>(exp(-static_cast<double>(k) * k / (2.0 * sigma * sigma))) : 1.f;
}

// Both blur passes give each thread eight neighbouring outputs: as the taps are
// walked, one new cell enters the thread's window per tap and feeds eight
// multiply-adds, so an output costs an eighth of an LDS read per tap.  (Reading
// each output's own window, tap by tap, bound both passes on the LDS.)  Whole
// calls, F = 4,000, fp32 weights, before and now: 128^2 map, R = 48 2.80 and
// 0.57 ms; 512^2, R = 17 25.4 and 9.1, R = 48 44.1 and 9.7, R = 192 176 and 23.4.
// What bounds them now: the loads of a row group or strip, which its arithmetic
// waits for, and at R = 192 the multiply-adds.  Cells outside the grid are zero
// in LDS: their terms leave the sums unchanged, which otherwise take the same
// terms in the same order, k = -R..R.
constexpr int kOut = 8;   // outputs per thread

// Output i's tap j reads cell i + j of the window's start; w holds the kOut cells of
// a tap, rotated by the unrolled loop.
template <typename READ>
__device__ __forceinline__ void blur_window(const float* taps, int n, float (&out)[kOut], READ read) {
  // taps[0..n-1]; out[i] = sum_j taps[j] * read(i + j), j ascending
  float w[kOut];
#pragma unroll
  for (int i = 0; i < kOut; ++i) {
    w[i] = read(i);
    out[i] = 0.f;
  }
  int j = 0;
  for (; j + kOut <= n; j += kOut) {
#pragma unroll
    for (int u = 0; u < kOut; ++u) {
      const float g = taps[j + u];
#pragma unroll
      for (int i = 0; i < kOut; ++i) out[i] = fmaf(g, w[(u + i) % kOut], out[i]);
      w[u] = read(j + u + kOut);
    }
  }
  for (; j < n; ++j) {   // fewer than kOut taps: the window shifts by moves
    const float g = taps[j];
#pragma unroll
    for (int i = 0; i < kOut; ++i) out[i] = fmaf(g, w[i], out[i]);
#pragma unroll
    for (int i = 0; i + 1 < kOut; ++i) w[i] = w[i + 1];
    w[kOut - 1] = read(j + kOut);
  }
}

// LDS position of cell c of a row: one float of padding per kOut keeps the
// threads' windows (kOut cells apart) on different banks.
__device__ __host__ __forceinline__ int row_pos(int c) { return c + c / kOut; }

// LDS floats of one padded row: Re cells each side, the columns rounded up to
// whole threads, and the cells the last window reads ahead.
__host__ __device__ inline int blur_row_floats(int cols, int Re) {
  return row_pos((cols + kOut - 1) / kOut * kOut + 2 * Re + kOut) + 1;
}

// Row pass.  in: plane p of the input (uint32 accumulators), rows x cols with
// row stride `cols` inside a plane of stride ld_in; out: fp32 plane of stride
// ld_out.  A workgroup takes `per` rows of one plane; grid (row groups, planes),
// row groups fastest, so that concurrent workgroups spread over one plane rather
// than hitting the same offset of planes a power-of-two stride apart (the same
// memory channels).  Re = min(R, cols - 1).
template <typename IN>
__global__ void __launch_bounds__(256)
k_blur_rows(const IN* __restrict__ in, int64_t ld_in, float* __restrict__ out, int64_t ld_out, int rows, int cols,
            int Re, int per, const float* __restrict__ g) {
  extern __shared__ float lds[];
  float* taps = lds;                            // [2 Re + 1]
  const int stride = blur_row_floats(cols, Re);
  float* cells = lds + (2 * Re + 1);            // [per][stride]
  const int64_t p = blockIdx.y;
  const int r0 = blockIdx.x * per;
  const int nr = rows - r0 < per ? rows - r0 : per;
  for (int j = threadIdx.x; j < 2 * Re + 1; j += blockDim.x) taps[j] = g[j < Re ? Re - j : j - Re];
  for (int i = threadIdx.x; i < nr * stride; i += blockDim.x) cells[i] = 0.f;
  __syncthreads();
  const IN* src = in + p * ld_in + static_cast<int64_t>(r0) * cols;
  for (int i = threadIdx.x; i < nr * cols; i += blockDim.x) {
    const int r = i / cols, c = i - r * cols;
    cells[r * stride + row_pos(c + Re)] = static_cast<float>(src[i]);
  }
  __syncthreads();
  const int groups = (cols + kOut - 1) / kOut;   // threads per row
  float* dst = out + p * ld_out + static_cast<int64_t>(r0) * cols;
  for (int i = threadIdx.x; i < nr * groups; i += blockDim.x) {
    const int r = i / groups, c = (i - r * groups) * kOut;
    const float* row = cells + r * stride;
    float v[kOut];
    blur_window(taps, 2 * Re + 1, v, [&](int k) { return row[row_pos(c + k)]; });
#pragma unroll
    for (int k = 0; k < kOut; ++k)
      if (c + k < cols) dst[r * cols + c + k] = v[k];
  }
}

// Column pass.  MODE 0: den[j] = v (one plane); MODE 1: write-back into the
// codebook.  A workgroup takes a strip of STRIP columns of one plane, all rows
// and Re zero rows each side in LDS, STRIP + STRIP / 8 floats apart, which puts
// the wave's 64 / STRIP row groups (kOut rows apart) on different banks.  Grid
// (strips, planes), strips fastest (see k_blur_rows).  Re = min(R, rows - 1).
// 512 threads: 256 left too few loads in flight beside an 80 KB strip (512^2, R =
// 17: 12.0 ms per call against 9.1)
constexpr int kColThreads = 512;

template <int STRIP>
__host__ __device__ constexpr int blur_col_stride() {
  return STRIP + STRIP / 8;
}

template <typename WT, int MODE, int STRIP>
__global__ void __launch_bounds__(kColThreads)
k_blur_cols(const float* __restrict__ t, int64_t ld_t, int rows, int cols, int Re, const float* __restrict__ g,
            float* __restrict__ den_out, const float* __restrict__ den, WT* __restrict__ W, int64_t ldw) {
  extern __shared__ float lds[];
  constexpr int kStride = blur_col_stride<STRIP>();
  constexpr int kGroups = kColThreads / STRIP;           // row groups in flight
  float* taps = lds;                             // [2 Re + 1]
  float* strip = lds + (2 * Re + 1);             // [rows + 2 Re + 2 kOut][kStride]
  const int64_t p = blockIdx.y;
  const int cx = threadIdx.x % STRIP;
  const int c = blockIdx.x * STRIP + cx;
  const int ry = threadIdx.x / STRIP;
  const float* src = t + p * ld_t;
  for (int j = threadIdx.x; j < 2 * Re + 1; j += kColThreads) taps[j] = g[j < Re ? Re - j : j - Re];
  for (int r = ry; r < rows + 2 * Re + 2 * kOut; r += kGroups) {
    const int rr = r - Re;
    strip[r * kStride + cx] = rr >= 0 && rr < rows && c < cols ? src[static_cast<int64_t>(rr) * cols + c] : 0.f;
  }
  __syncthreads();
  if (c >= cols) return;
  for (int r0 = ry * kOut; r0 < rows; r0 += kGroups * kOut) {
    const float* col = strip + r0 * kStride + cx;
    float v[kOut];
    blur_window(taps, 2 * Re + 1, v, [&](int k) { return col[k * kStride]; });
#pragma unroll
    for (int k = 0; k < kOut; ++k) {
      if (r0 + k >= rows) break;
      const int64_t j = static_cast<int64_t>(r0 + k) * cols + c;
      if (MODE == 0) {
        den_out[j] = v[k];
      } else {
        const float dj = den[j];
        if (dj > 0.f) W[p * ldw + j] = static_cast<WT>(v[k] / dj);
      }
    }
  }
}

// The column pass of maps and radii whose strip with its zero rows exceeds the
// LDS: 32 columns, only the grid's rows in LDS, each output's window tap by tap.
template <typename WT, int MODE>
__global__ void __launch_bounds__(256)
k_blur_cols_tall(const float* __restrict__ t, int64_t ld_t, int rows, int cols, int R, const float* __restrict__ g,
                 float* __restrict__ den_out, const float* __restrict__ den, WT* __restrict__ W, int64_t ldw) {
  extern __shared__ float lds[];
  float* strip = lds;  // [rows][kStrip]
  const int64_t p = blockIdx.y;
  const int c0 = blockIdx.x * kStrip;
  const int cx = threadIdx.x % kStrip;
  const int ry = threadIdx.x / kStrip;          // 8 row lanes
  const int c = c0 + cx;
  const float* src = t + p * ld_t;
  for (int r = ry; r < rows; r += 256 / kStrip)
    strip[r * kStrip + cx] = c < cols ? src[static_cast<int64_t>(r) * cols + c] : 0.f;
  __syncthreads();
  if (c >= cols) return;
  for (int r = ry; r < rows; r += 256 / kStrip) {
    const int lo = r - R < 0 ? -r : -R;
    const int hi = r + R >= rows ? rows - 1 - r : R;
    float s = 0.f;
    for (int k = lo; k <= hi; ++k) s = fmaf(g[k < 0 ? -k : k], strip[(r + k) * kStrip + cx], s);
    const int64_t j = static_cast<int64_t>(r) * cols + c;
    if (MODE == 0) {
      den_out[j] = s;
    } else {
      const float dj = den[j];
      if (dj > 0.f) W[p * ldw + j] = static_cast<WT>(s / dj);
    }
  }
}

constexpr size_t kLdsBytes = 160 * 1024;   // per workgroup

hipError_t launch_blur_rows(const uint32_t* in, int64_t ld_in, float* out, int64_t ld_out, int rows, int cols, int R,
                            const float* g, int64_t planes, hipStream_t stream) {
  const int Re = R < cols - 1 ? R : cols - 1;
  const size_t row = sizeof(float) * blur_row_floats(cols, Re), taps = sizeof(float) * (2 * Re + 1);
  // rows per workgroup: a window of kOut outputs per thread where the row is
  // short, within 64 KB so that two workgroups share a CU
  const int groups = (cols + kOut - 1) / kOut;
  int per = groups < 256 ? 256 / groups : 1;
  while (per > 1 && per * row + taps > 64 * 1024) --per;
  if (per > rows) per = rows;
  const size_t lds = per * row + taps;
  const hipError_t e = allow_lds(&k_blur_rows<uint32_t>, kLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_blur_rows<uint32_t>, dim3(static_cast<uint32_t>((rows + per - 1) / per), static_cast<uint32_t>(planes)),
                     dim3(256), lds, stream, in, ld_in, out, ld_out, rows, cols, Re, per, g);
  return hipGetLastError();
}

// 32-column strips where two of them fit a CU's LDS, else 16 where one does
// (half as many bytes per global read), else the tap-by-tap form.
template <typename WT, int MODE>
hipError_t launch_blur_cols(const float* t, int64_t ld_t, int rows, int cols, int R, const float* g, float* den_out,
                            const float* den, WT* W, int64_t ldw, int64_t planes, hipStream_t stream) {
  const int Re = R < rows - 1 ? R : rows - 1;
  const size_t taps = sizeof(float) * (2 * Re + 1);
  const size_t cells = static_cast<size_t>(rows) + 2 * Re + 2 * kOut;
  const size_t wide = taps + sizeof(float) * cells * blur_col_stride<32>();
  const size_t narrow = taps + sizeof(float) * cells * blur_col_stride<16>();
  const uint32_t np = static_cast<uint32_t>(planes);
  if (wide <= kLdsBytes / 2 || (wide <= kLdsBytes && narrow > kLdsBytes / 2)) {
    const hipError_t e = allow_lds(&k_blur_cols<WT, MODE, 32>, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_blur_cols<WT, MODE, 32>), dim3(static_cast<uint32_t>((cols + 31) / 32), np), dim3(kColThreads), wide,
                       stream, t, ld_t, rows, cols, Re, g, den_out, den, W, ldw);
  } else if (narrow <= kLdsBytes) {
    const hipError_t e = allow_lds(&k_blur_cols<WT, MODE, 16>, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_blur_cols<WT, MODE, 16>), dim3(static_cast<uint32_t>((cols + 15) / 16), np), dim3(kColThreads),
                       narrow, stream, t, ld_t, rows, cols, Re, g, den_out, den, W, ldw);
  } else {
    const size_t tall = sizeof(float) * static_cast<size_t>(rows) * kStrip;
    const hipError_t e = allow_lds(&k_blur_cols_tall<WT, MODE>, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_blur_cols_tall<WT, MODE>), dim3(static_cast<uint32_t>((cols + kStrip - 1) / kStrip), np),
                       dim3(256), tall, stream, t, ld_t, rows, cols, R, g, den_out, den, W, ldw);
  }
  return hipGetLastError();
}

// Streaming blur + write-back (R <= kStreamMaxR, one instantiation per
// radius): one wave owns a strip of 64 columns of one feature plane and
// walks down the grid rows.  Step r loads row r of the strip with its R-wide
// halo (cells outside the grid are zero) into the wave's own LDS row buffer
// and forms the row pass t[r][c] = sum_{k=-R..R} g[|k|] acc[r][c+k]; each
// lane keeps the row-pass results of the last 2R+1 rows in registers (the
// step loop is unrolled by a multiple of 2R+1, so a row's slot is a static
// index), from which the column pass of row r - R,
// sum_{k=-R..R} g[|k|] t[r-R+k][c] (zero rows outside the grid: their slots
// still hold zero), is formed; then the write-back through the blurred
// counts.  Both sums take the same terms in the same order as the two-pass
// kernels; the taps sit in registers and every LDS read has an immediate
// offset.  Rows, and the blurred counts of the rows written back, are loaded
// at least kStreamAhead steps before use; a wave
// touches only its own LDS, so there is no workgroup barrier, and every input
// and output element is read or written once.
constexpr int kStreamMaxR = 16;
constexpr int kStreamAhead = 8;

template <typename WT, int R>
__global__ void __launch_bounds__(64)
k_blur_stream(const uint32_t* __restrict__ acc, int64_t ld_acc, int64_t f0, int rows, int cols,
              const float* __restrict__ g, const float* __restrict__ den, WT* __restrict__ W, int64_t ldw) {
  constexpr int H = 2 * R + 1;
  // steps per unrolled block: a multiple of H (so row r's history slot is
  // the static index (r mod H)), and at least kStreamAhead (the prefetch depth)
  constexpr int U = H * ((kStreamAhead + H - 1) / H);
  __shared__ float rb[64 + 2 * R + 1];  // the current row with its halo
  const int lane = threadIdx.x;
  const int64_t f = f0 + blockIdx.y;
  const int c0 = blockIdx.x * 64;
  const int c = c0 + lane;
  const uint32_t* src = acc + f * ld_acc;
  float tp[R + 1];
#pragma unroll
  for (int i = 0; i <= R; ++i) tp[i] = g[i];
  float hr[H];  // row-pass results of the last H rows: row r in slot r mod H
#pragma unroll
  for (int i = 0; i < H; ++i) hr[i] = 0.f;
  // this lane's two input columns: c0 - R + lane, and c0 - R + 64 + lane for
  // the halo's last 2R cells
  const int ca = c0 - R + lane, cb = c0 - R + 64 + lane;
  const bool va = ca >= 0 && ca < cols, vb = lane < 2 * R && cb >= 0 && cb < cols;
  // Raw words in flight, with the blurred count of the row written back at
  // the step that uses them (row r - R): every lane loads unconditionally
  // (cells outside the grid read element 0 instead), and the selects and the
  // conversion happen when the row is used, so no load is waited for in the
  // step that issues it.
  const bool vc = c < cols;
  uint32_t pa[U], pb[U];
  float pd[U];
#define SOM_STREAM_LOAD(r, a, b, d)                                                                 \
  {                                                                                                \
    const bool in_ = (r) < rows;                                                                   \
    const int rd_ = (r) - R;                                                                       \
    a = src[(in_ && va) ? static_cast<int64_t>(r) * cols + ca : 0];                                \
    b = src[(in_ && vb) ? static_cast<int64_t>(r) * cols + cb : 0];                                \
    d = den[(rd_ >= 0 && rd_ < rows && vc) ? static_cast<int64_t>(rd_) * cols + c : 0];            \
  }
#pragma unroll
  for (int u = 0; u < U; ++u) SOM_STREAM_LOAD(u, pa[u], pb[u], pd[u])
  const int steps = rows + R;
  for (int r0 = 0; r0 < steps; r0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u;
      if (r >= steps) break;
      const bool in = r < rows;
      const float a = (in && va) ? static_cast<float>(pa[u]) : 0.f;
      const float b = (in && vb) ? static_cast<float>(pb[u]) : 0.f;
      const float dj = pd[u];  // blurred count of row r - R (read only when r >= R and c < cols)
      SOM_STREAM_LOAD(r + U, pa[u], pb[u], pd[u])
      // row pass of row r (zero beyond the last row)
      rb[lane] = a;
      if (lane < 2 * R) rb[64 + lane] = b;
      __builtin_amdgcn_wave_barrier();
      float t = 0.f;
#pragma unroll
      for (int j = 0; j <= 2 * R; ++j) t = fmaf(tp[j < R ? R - j : j - R], rb[lane + j], t);
      __builtin_amdgcn_wave_barrier();
      hr[u % H] = r < rows ? t : 0.f;
      // column pass of row r - R: slots (u+1 .. u+H) mod H hold rows r-2R .. r
      // (slots of rows before the first still hold zero)
      if (r >= R) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j <= 2 * R; ++j) s = fmaf(tp[j < R ? R - j : j - R], hr[(u + 1 + j) % H], s);
        if (vc && dj > 0.f) W[f * ldw + static_cast<int64_t>(r - R) * cols + c] = static_cast<WT>(s / dj);
      }
    }
  }
#undef SOM_STREAM_LOAD
}

template <typename WT, int R>
hipError_t launch_stream_r(const uint32_t* acc, int64_t ld_acc, int64_t F, int rows, int cols, const float* taps,
                           const float* den, WT* W, int64_t ldw, hipStream_t stream) {
  const uint32_t strips64 = static_cast<uint32_t>((cols + 63) / 64);
  for (int64_t f0 = 0; f0 < F; f0 += 65535) {  // grid.y holds at most 65535 features
    const uint32_t fc = static_cast<uint32_t>(F - f0 < 65535 ? F - f0 : 65535);
    hipLaunchKernelGGL((k_blur_stream<WT, R>), dim3(strips64, fc), dim3(64), 0, stream, acc, ld_acc, f0, rows, cols,
                       taps, den, W, ldw);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename WT, int R = 0>
hipError_t launch_stream(int r, const uint32_t* acc, int64_t ld_acc, int64_t F, int rows, int cols, const float* taps,
                         const float* den, WT* W, int64_t ldw, hipStream_t stream) {
  if constexpr (R > kStreamMaxR) {
    return hipErrorInvalidValue;
  } else {
    if (r == R) return launch_stream_r<WT, R>(acc, ld_acc, F, rows, cols, taps, den, W, ldw, stream);
    return launch_stream<WT, R + 1>(r, acc, ld_acc, F, rows, cols, taps, den, W, ldw, stream);
  }
}

}  // namespace

size_t update_chunk_planes(int64_t F, int64_t N) {
  int64_t fc = (int64_t(1) << 26) / (N > 0 ? N : 1);  // about 256 MB of fp32 per chunk
  if (fc < 1) fc = 1;
  if (fc > 65535) fc = 65535;  // planes go in grid.y
  if (fc > F) fc = F;
  return static_cast<size_t>(fc);
}

hipError_t launch_update_accumulate(const int32_t* indptr, const int32_t* indices, int64_t B, const int32_t* bmu,
                                    int64_t F, int64_t N, uint32_t* acc, int64_t ld_acc, uint32_t* count,
                                    hipStream_t stream) {
  hipLaunchKernelGGL(k_accumulate, dim3(static_cast<uint32_t>((B + 3) / 4)), dim3(256), 0, stream, indptr, indices,
                     B, bmu, F, N, acc, ld_acc, count);
  return hipGetLastError();
}

hipError_t launch_update_finish(void* W, int weights, int64_t F, int64_t ldw, int rows, int cols, double sigma, int R,
                                const uint32_t* acc, int64_t ld_acc, const uint32_t* count, float* taps,
                                float* den_tmp, float* den, float* chunk, int64_t chunk_planes,
                                hipStream_t stream) {
  const int64_t N = static_cast<int64_t>(rows) * cols;
  hipLaunchKernelGGL(k_taps, dim3(static_cast<uint32_t>(R / 256 + 1)), dim3(256), 0, stream, sigma, R, taps);
  // denominators: the blurred counts
  hipError_t e = launch_blur_rows(count, N, den_tmp, N, rows, cols, R, taps, 1, stream);
  if (e != hipSuccess) return e;
  e = launch_blur_cols<float, 0>(den_tmp, N, rows, cols, R, taps, den, nullptr, nullptr, 0, 1, stream);
  if (e != hipSuccess) return e;
  if (R <= kStreamMaxR) {
    // numerators streamed down 64-column strips, written back through den
    if (weights == kWeightsF16)
      return launch_stream<_Float16>(R, acc, ld_acc, F, rows, cols, taps, den, static_cast<_Float16*>(W), ldw, stream);
    return launch_stream<float>(R, acc, ld_acc, F, rows, cols, taps, den, static_cast<float*>(W), ldw, stream);
  }
  // larger radii: numerators a chunk of features at a time, row pass into the
  // chunk buffer, then the column pass written back through den
  for (int64_t f0 = 0; f0 < F; f0 += chunk_planes) {
    const int64_t fc = F - f0 < chunk_planes ? F - f0 : chunk_planes;
    e = launch_blur_rows(acc + f0 * ld_acc, ld_acc, chunk, N, rows, cols, R, taps, fc, stream);
    if (e != hipSuccess) return e;
    if (weights == kWeightsF16)
      e = launch_blur_cols<_Float16, 1>(chunk, N, rows, cols, R, taps, nullptr, den,
                                        static_cast<_Float16*>(W) + f0 * ldw, ldw, fc, stream);
    else
      e = launch_blur_cols<float, 1>(chunk, N, rows, cols, R, taps, nullptr, den, static_cast<float*>(W) + f0 * ldw,
                                     ldw, fc, stream);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace som
