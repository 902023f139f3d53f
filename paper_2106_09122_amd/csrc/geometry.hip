// Scene geometry and radial brackets of every library column, plus the two
// small preparations of the PSF datacube used by the build.
//
// Paper: Sec. 2, Eqs. (2)-(3) (half-pixel-shifted meshgrid scaled by the
// scene pixel scale, flattened row-major), the polar conversion of each field
// point, and the radial interpolation of the datacube (linear or nearest).
#include <math.h>

#include "psflib_internal.h"

namespace psflib {

// Largest value (exact float32 max, for the 16-bit column exponents) and sum
// (float64, a fixed order, for the flux rescale) of each sampled PSF, each where
// asked for.  One workgroup per PSF, four independent loads in flight per thread
// (latency: 51 PSFs of 101^2 take 4 us, 12 with 256 threads and one load each).
__global__ __launch_bounds__(1024) void cube_stats_kernel(const float* __restrict__ cube, int64_t M,
                                                          float* __restrict__ pmax,
                                                          double* __restrict__ sums) {
  __shared__ float red[16];
  __shared__ double red64[16];
  const float* P = cube + (int64_t)blockIdx.x * M;
  float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  double t[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = threadIdx.x; i < M; i += 4 * 1024) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + 1024 * u < M ? P[i + 1024 * u] : 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      m[u] = fmaxf(m[u], v[u]);
      t[u] += (double)v[u];
    }
  }
  float mx = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
  double sum = (t[0] + t[1]) + (t[2] + t[3]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    sum += __shfl_xor(sum, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = mx;
    red64[threadIdx.x >> 6] = sum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      mx = fmaxf(mx, red[w]);
      sum += red64[w];
    }
    if (pmax) pmax[blockIdx.x] = mx;
    if (sums) sums[blockIdx.x] = sum;
  }
}

// pairs[k][p] = (P_k[p], P_{k+1}[p]) for k < max(K-1, 1), so one 8-byte load
// fetches both radial neighbours of a tap (P_1 reads as 0 when K == 1).
__global__ __launch_bounds__(256) void pair_cube_kernel(const float* __restrict__ cube, int K,
                                                        int64_t M, float2* __restrict__ pairs) {
  const int64_t npairs = (K > 1) ? (int64_t)(K - 1) : 1;
  const int64_t total = npairs * M;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * 256) {
    const int64_t k = t / M, p = t - k * M;
    float2 v;
    v.x = cube[k * M + p];
    v.y = (K > 1) ? cube[(k + 1) * M + p] : 0.0f;
    pairs[t] = v;
  }
}

// Radii of up to kRadiiArg samples, passed with the launch; more are read from
// device memory, an upload of its own.
struct RadiiArg {
  double r[kRadiiArg];
};

// One thread per column j (and per padding column up to ncols_pad).
template <bool ARG>
__global__ __launch_bounds__(256) void geometry_kernel(int N, double S, const RadiiArg arg,
                                                       const double* __restrict__ far, int K,
                                                       int interp, int oob,
                                                       const float* __restrict__ pmax,
                                                       int want_exp, ColGeom* __restrict__ geo,
                                                       int64_t ncols_pad,
                                                       int32_t* __restrict__ exps) {
#pragma clang fp contract(off)
  __shared__ double near[ARG ? kRadiiArg : 1];
  if constexpr (ARG) {
    static_assert(kRadiiArg <= 256, "one thread per radius");
    if ((int)threadIdx.x < K) near[threadIdx.x] = arg.r[threadIdx.x];
    __syncthreads();
  }
  const double* radii = ARG ? near : far;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t ncols = (int64_t)N * N;
  if (j >= ncols_pad) return;
  ColGeom g;
  g.pad[0] = g.pad[1] = 0;
  if (j >= ncols) {  // padding column of the 16-bit layout: identically zero
    g.r = 0.0; g.ct = 1.0; g.st = 0.0; g.w = 0.0; g.k = -1; g.e = want_exp ? kZeroColumnExp : 0;
    geo[j] = g;
    if (exps) exps[j] = g.e;
    return;
  }
  const int64_t p = j / N, q = j - p * N;
  // Eqs. (2)-(3): centre offsets (q - (N-1)/2) S and (p - (N-1)/2) S.
  const double C = (double)(N - 1) * 0.5;
  const double x = ((double)q - C) * S;
  const double y = ((double)p - C) * S;
  const double r = sqrt(x * x + y * y);
  double ct = 1.0, st = 0.0;  // atan2(0, 0) = 0
  if (r > 0.0) {
    ct = x / r;
    st = y / r;
  }
  // Radial bracket: Q = (1-w) P_k + w P_{k+1}.
  int k = 0;
  double w = 0.0;
  bool zero = false;
  if (K > 1) {
    if (r <= radii[0]) {
      k = 0; w = 0.0;
    } else if (r >= radii[K - 1]) {
      k = K - 2; w = 1.0;
      if (oob == PSFLIB_OOB_ZERO && r > radii[K - 1]) zero = true;
    } else {
      int lo = 0, hi = K - 1;  // radii[lo] <= r < radii[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (radii[mid] <= r) lo = mid; else hi = mid;
      }
      k = lo;
      const double a = radii[lo], b = radii[lo + 1];
      if (interp == PSFLIB_INTERP_NEAREST)
        w = ((r - a) > (b - r)) ? 1.0 : 0.0;  // ties go to the lower sample
      else
        w = (r - a) / (b - a);
    }
  }
  g.r = r; g.ct = ct; g.st = st; g.w = zero ? 0.0 : w; g.k = zero ? -1 : k;
  g.e = want_exp ? kZeroColumnExp : 0;
  if (want_exp && !zero) {
    // Bound on the column's largest value: bilinear rotation is a convex
    // combination of Q's pixels (or zero), so max_i A_ij <= max Q.
    const double bound = (K == 1) ? (double)pmax[0]
                                  : (1.0 - w) * (double)pmax[k] + w * (double)pmax[k + 1];
    g.e = scale_exponent(bound);
  }
  geo[j] = g;
  if (exps) exps[j] = g.e;
}

__global__ __launch_bounds__(256) void export_geometry_kernel(const ColGeom* __restrict__ geo,
                                                              int64_t ncols,
                                                              double* __restrict__ geom,
                                                              int32_t* __restrict__ kout) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= ncols) return;
  const ColGeom g = geo[j];
  if (geom) {
    geom[4 * j + 0] = g.r;
    geom[4 * j + 1] = g.ct;
    geom[4 * j + 2] = g.st;
    geom[4 * j + 3] = g.w;
  }
  if (kout) kout[j] = g.k;
}

static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

hipError_t launch_cube_stats(const float* cube, int K, int64_t M, float* pmax, double* sums,
                             hipStream_t s) {
  cube_stats_kernel<<<K, 1024, 0, s>>>(cube, M, pmax, sums);
  return hipGetLastError();
}

hipError_t launch_pair_cube(const float* cube, int K, int64_t M, float* pairs, hipStream_t s) {
  const int64_t total = ((K > 1) ? (int64_t)(K - 1) : 1) * M;
  const int64_t want = (total + 255) / 256;
  const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
  pair_cube_kernel<<<grid, 256, 0, s>>>(cube, K, M, reinterpret_cast<float2*>(pairs));
  return hipGetLastError();
}

hipError_t launch_geometry(int N, double S, const double* h_radii, const double* radii, int K, int interp,
                           int oob, const float* pmax, bool want_exp, ColGeom* geo,
                           int64_t ncols_pad, int32_t* exps, hipStream_t s) {
  RadiiArg arg = {};
  const unsigned grid = blocks_for(ncols_pad, 256);
  if (K <= kRadiiArg) {
    for (int k = 0; k < K; ++k) arg.r[k] = h_radii[k];
    geometry_kernel<true><<<grid, 256, 0, s>>>(N, S, arg, nullptr, K, interp, oob, pmax,
                                               want_exp ? 1 : 0, geo, ncols_pad, exps);
  } else {
    geometry_kernel<false><<<grid, 256, 0, s>>>(N, S, arg, radii, K, interp, oob, pmax,
                                                want_exp ? 1 : 0, geo, ncols_pad, exps);
  }
  return hipGetLastError();
}

hipError_t launch_export_geometry(const ColGeom* geo, int64_t ncols, double* geom, int32_t* k,
                                  hipStream_t s) {
  export_geometry_kernel<<<blocks_for(ncols, 256), 256, 0, s>>>(geo, ncols, geom, k);
  return hipGetLastError();
}

}  // namespace psflib
