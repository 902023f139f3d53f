// Cubic-spline rotation: spline coefficients of the sampled PSFs, which the
// cubic orbit build (build_lds.hip) and the cubic gather (build.hip) sample.
//
// The rotation step of Sec. 2 uses SciPy's rotate(), whose default
// interpolation is a cubic spline.  The spline that interpolates a PSF
// extended by zeros, f(x) = sum_m c_m beta3(x - m), has coefficients c that
// are the samples passed through the cubic B-spline interpolation filter.
// Here every sampled PSF P_k is padded by kSplinePad zero pixels per side and
// filtered (float64) along columns, then along rows, with the recursive filter
// for a mirror-symmetric extension of the padded array: gain 6, a causal and an
// anticausal first-order recursion with pole z = sqrt(3) - 2 over the mirrored
// line.  Because the filter is linear, the coefficients of a radially
// interpolated PSF Q = (1-w) P_k + w P_{k+1} are (1-w) C_k + w C_{k+1}, so the
// build blends coefficient pairs exactly as the bilinear build blends sample
// pairs.
//
// Output in scratch: the column pass's float64 results [K][Np][Np] (Np = n + 2
// pad), then radial pairs (C_k, C_{k+1}) rounded to float32, and per PSF the largest
// |coefficient| (which bounds the column for the 16-bit exponents: the spline
// value is a convex combination of coefficients).
#include <math.h>

#include "psflib_internal.h"

namespace psflib {

namespace {

constexpr double kPole = -0.26794919243112270;  // sqrt(3) - 2

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The recursions forget geometrically (|z|^kTail = 5e-19), so a line is cut into
// segments of kSeg samples, one thread each: the causal recursion starts at zero kTail
// samples before the segment and runs kTail past it, the anticausal one back from
// there.  What is dropped is a few 5e-19 of the line's samples more than kTail away:
// below the float64 rounding of the terms kept where the line's contrast is moderate,
// 5e-11 of the faint coefficients where it is 1e-10 (a coronagraph's), under the
// float32 rounding that follows up to 1e-13 (at 1e-14 3e-7); zeros more than kTail
// samples from the nearest other sample stay zero.  A whole
// line per thread (one chain of 4 Np dependent steps through LDS) took 74 us for
// 51 PSFs of 101^2 with the pairs and the maxima in passes of their own, all
// latency; the segments, nine loads of a cached sample per sample, take 21 us.
constexpr int kSeg = 8, kTail = 32;

// Sample index of the mirrored line (period 2 Np - 2; Np >= 25).  Indices in
// [-kTail, Np + kSeg + kTail) are exact, beyond (past the last segment, not
// used) in bounds.
__device__ __forceinline__ int mirror(int i, int Np) {
  i = i < 0 ? -i : i;
  i = i >= Np ? 2 * Np - 2 - i : i;
  i = i < 0 ? -i : i;
  return i < Np ? i : Np - 1;
}

// Coefficients out[0 .. kSeg) of a segment; get(t) is the sample t positions
// after its first, -kTail <= t < kSeg + kTail.
template <typename Get>
__device__ __forceinline__ void spline_segment(Get get, double (&out)[kSeg]) {
  const double z = kPole;
  double y[kSeg + kTail], prev = 0.0, next = 0.0;
#pragma unroll
  for (int t = -kTail; t < 0; ++t) prev = fma(z, prev, 6.0 * get(t));
#pragma unroll
  for (int t = 0; t < kSeg + kTail; ++t) {
    prev = fma(z, prev, 6.0 * get(t));
    y[t] = prev;
  }
#pragma unroll
  for (int t = kSeg + kTail - 1; t >= 0; --t) {
    next = z * (next - y[t]);
    if (t < kSeg) out[t] = next;
  }
}

// Column pass: a workgroup takes tiles of 64 columns by 32 rows of a padded PSF
// (ys workgroups share a PSF's 64 columns), staged in LDS with their kTail
// neighbours, each wave kSeg rows.  A sample that is not finite makes its whole
// column NaN, and with it in the row pass the whole PSF, as a recursion over
// whole lines does.  Sets cmax to zero for the row pass.  (From registers, every
// sample's mirrored row unrolled, the pass is instruction fetches: 20 us for 51
// PSFs of 101^2, 9 us this way.)
constexpr int kTileRows = 4 * kSeg, kColSplit = 4;

__global__ __launch_bounds__(256) void spline_cols_kernel(const float* __restrict__ cube, int n,
                                                          int Np, int tx, int ys,
                                                          double* __restrict__ T,
                                                          float* __restrict__ cmax) {
  __shared__ float tile[kTileRows + 2 * kTail][64];
  __shared__ int bad[4][64];
  const int wgs = tx * ys;
  const int64_t k = blockIdx.x / (unsigned)wgs;
  const int wg = (int)(blockIdx.x % (unsigned)wgs);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int q = wg % tx * 64 + lane;
  if (cmax && wg == 0 && threadIdx.x == 0) cmax[k] = 0.0f;
  const int b = q - kSplinePad;
  const bool inside = (unsigned)b < (unsigned)n;
  const float* col = cube + k * (int64_t)n * n + (inside ? b : 0);
  int mine = 0;
#pragma unroll 8
  for (int a = wave; a < n; a += 4) mine |= !(fabsf(col[(int64_t)a * n]) < INFINITY);
  bad[wave][lane] = inside ? mine : 0;
  double* dst = T + k * (int64_t)Np * Np + q;
  for (int r0 = wg / tx * kTileRows; r0 < Np; r0 += ys * kTileRows) {
#pragma unroll 8
    for (int r = wave; r < kTileRows + 2 * kTail; r += 4) {
      const int a = mirror(r0 + r - kTail, Np) - kSplinePad;
      const bool in = (unsigned)a < (unsigned)n;
      const float v = col[(int64_t)(in ? a : 0) * n];  // no branch: the loads overlap
      tile[r][lane] = inside && in ? v : 0.0f;
    }
    __syncthreads();
    const int i0 = r0 + wave * kSeg;
    if (i0 < Np && q < Np) {
      const bool any = bad[0][lane] | bad[1][lane] | bad[2][lane] | bad[3][lane];
      double out[kSeg];
      spline_segment([&](int t) { return (double)tile[wave * kSeg + kTail + t][lane]; }, out);
#pragma unroll
      for (int t = 0; t < kSeg; ++t)
        if (i0 + t < Np) dst[(int64_t)(i0 + t) * Np] = any ? (double)NAN : out[t];
    }
    __syncthreads();  // the tile is read
  }
}

// Row pass: tiles of kRows rows by kCols columns, staged in LDS with their
// kTail neighbours (odd row stride), a thread per row and segment.  Coefficient
// C_k, rounded to float32, is the first of pair k and the second of pair k - 1;
// the tile's largest |C_k| goes to cmax[k] (bits of non-negative floats order
// as integers; NaNs are skipped).
constexpr int kRows = 16, kCols = 128, kStride = kCols + 2 * kTail + 1;

__global__ __launch_bounds__(256) void spline_rows_kernel(const double* __restrict__ T, int K,
                                                          int Np, int tx, int ty,
                                                          float* __restrict__ pairs,
                                                          float* __restrict__ cmax) {
  static_assert(kRows * kCols / kSeg == 256, "one segment per thread");
  __shared__ double tile[kRows * kStride];
  __shared__ float red[4];
  const int tiles = tx * ty;
  const int64_t k = blockIdx.x / (unsigned)tiles;
  const int tl = (int)(blockIdx.x % (unsigned)tiles);
  const int c0 = (tl % tx) * kCols, i0 = (tl / tx) * kRows;
  const int tid = threadIdx.x;
  const double* src = T + (k * Np + i0) * Np;
  constexpr int W = kCols + 2 * kTail;
  const int rows = Np - i0 < kRows ? Np - i0 : kRows;
  for (int e = tid; e < rows * W; e += 256) {
    const int r = e / W, c = e - r * W;
    tile[r * kStride + c] = src[(int64_t)r * Np + mirror(c0 + c - kTail, Np)];
  }
  int bad = 0;  // a column that is not finite shows in every row
  for (int c = tid; c < Np; c += 256) bad |= !(fabs(src[c]) < (double)INFINITY);
  bad = __syncthreads_or(bad);
  const int r = tid % kRows, c = tid / kRows * kSeg;
  double out[kSeg];
  float m = 0.0f;
  if (r < rows && c0 + c < Np) {
    spline_segment([&](int t) { return tile[r * kStride + c + kTail + t]; }, out);
    if (bad) {
#pragma unroll
      for (int t = 0; t < kSeg; ++t) out[t] = (double)NAN;
    }
#pragma unroll
    for (int t = 0; t < kSeg; ++t)
      if (c0 + c + t < Np) m = fmaxf(m, fabsf((float)out[t]));
  }
  __syncthreads();  // the samples are read: the coefficients take their place
  if (r < rows && c0 + c < Np) {
#pragma unroll
    for (int t = 0; t < kSeg; ++t) tile[r * kStride + c + t] = out[t];
  }
  if (cmax) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((tid & 63) == 0) red[tid >> 6] = m;
  }
  __syncthreads();
  if (cmax && tid == 0)
    atomicMax(reinterpret_cast<unsigned int*>(cmax) + k,
              __float_as_uint(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))));
  const int64_t P = (int64_t)Np * Np;
  const int cols = Np - c0 < kCols ? Np - c0 : kCols;
  for (int e = tid; e < rows * kCols; e += 256) {
    const int rr = e / kCols, cc = e % kCols;
    if (cc >= cols) continue;
    const float v = (float)tile[rr * kStride + cc];
    float* dst = pairs + 2 * (k * P + (int64_t)(i0 + rr) * Np + c0 + cc);
    if (k < K - 1 || K == 1) dst[0] = v;
    if (k > 0) dst[1 - 2 * P] = v;
    if (K == 1) dst[1] = 0.0f;
  }
}

}  // namespace

size_t spline_scratch_bytes(int K, int n) {
  const int64_t Np = (int64_t)n + 2 * kSplinePad, P = Np * Np;
  const int64_t npairs = (K > 1) ? (int64_t)(K - 1) : 1;
  return align256((size_t)K * (size_t)P * 8) + align256((size_t)npairs * (size_t)P * 8);
}

const float* spline_pairs_of(const void* scratch, int K, int n) {
  const int64_t Np = (int64_t)n + 2 * kSplinePad, P = Np * Np;
  return reinterpret_cast<const float*>(reinterpret_cast<const char*>(scratch) +
                                        align256((size_t)K * (size_t)P * 8));
}

hipError_t launch_spline_pairs(const float* cube, int K, int n, void* scratch, float* cmax,
                               hipStream_t s) {
  const int Np = n + 2 * kSplinePad;
  double* T = reinterpret_cast<double*>(scratch);
  float* pairs = const_cast<float*>(spline_pairs_of(scratch, K, n));
  const int cx = (Np + 63) / 64, ct = (Np + kTileRows - 1) / kTileRows;
  const int cy = ct < kColSplit ? ct : kColSplit;
  const int rx = (Np + kCols - 1) / kCols, ry = (Np + kRows - 1) / kRows;
  const int64_t cgrid = (int64_t)K * cx * cy, rgrid = (int64_t)K * rx * ry;
  if (cgrid > INT32_MAX || rgrid > INT32_MAX) return hipErrorInvalidValue;  // above 2^31 x 2048 pixels
  spline_cols_kernel<<<(unsigned)cgrid, 256, 0, s>>>(cube, n, Np, cx, cy, T, cmax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  spline_rows_kernel<<<(unsigned)rgrid, 256, 0, s>>>(T, K, Np, rx, ry, pairs, cmax);
  return hipGetLastError();
}

}  // namespace psflib
