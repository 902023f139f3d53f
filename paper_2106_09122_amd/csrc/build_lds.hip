// Library build with the radial sample pair staged in LDS (Sec. 2; Eqs. (4)-(5)).
//
// Columns are grouped by their radial bracket k on the device (a counting sort:
// histogram, scan, scatter), so a workgroup can stage the two sampled PSFs it
// needs, P_k and P_{k+1}, once in LDS and build many columns from them.  The
// pair is stored interleaved (one 8-byte LDS read returns both radial
// neighbours of a tap) inside a one-pixel zero border, so the bilinear taps of
// the rotated sample need no per-tap bounds tests.
//
// Coordinates follow the oracle's float64 operations exactly (same products,
// no contraction): per column the products cos*(b-c) and -sin*(b-c) of an
// image column and sin*(a-c), cos*(a-c) of an image row are formed once and
// each element adds them.  The fractional offsets and their complements are
// exact float64 values rounded once to float32; the bilinear weights are their
// float32 products, the radial blend and the weighted sum are float32
// (relative error a few float32 units, as the entries are non-negative
// combinations).
//
// Paths, by what fits:
//  * rotation orbits: the four quarter turns of a scene pixel about the star
//    have bitwise-rotated columns, so one wave forms a base column and writes
//    all four (float32: 16-byte runs straight from registers; 16-bit: rounded
//    into an LDS tile of 8-slot units, slots ordered so that a group holds one
//    quarter turn of 8 base columns).  The pair is staged whole when it fits
//    the LDS; larger pairs (up to 8192 x 8192) are read through a small box per
//    32 x 32 pixel tile, staged by each wave in its own LDS region;
//  * columns in bracket order (sort bounds of the orbits exceeded, pairs that fit
//    the LDS): one wave per column.  The 16-bit forms of these are built as
//    float32 columns into scratch and packed by a second kernel (scale by
//    2^-e_j, round to nearest even, 8 columns per 16 B).
#include <math.h>

#include <type_traits>

#include "psflib_internal.h"

namespace psflib {

// ------------------------------------------------------------ buckets -----
__global__ __launch_bounds__(256) void zero_ints_kernel(int32_t* __restrict__ p, int count) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = 0;
}

// bucket of column j: its bracket k, or nb-1 for an identically zero column.
// Counts are gathered in an LDS histogram per workgroup and added to the
// global counts with one atomic per non-empty bucket (few buckets, many
// columns: direct global atomics would serialise on a handful of addresses).
__device__ __forceinline__ int bucket_of(const ColGeom* __restrict__ geo, int64_t j, int nb) {
  const int k = geo[j].k;
  return k >= 0 ? k : nb - 1;
}

__global__ __launch_bounds__(256) void bucket_count_kernel(const ColGeom* __restrict__ geo,
                                                           int64_t ncols, int nb,
                                                           int32_t* __restrict__ cnt) {
  extern __shared__ int32_t hist[];  // nb
  for (int b = threadIdx.x; b < nb; b += 256) hist[b] = 0;
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < ncols) atomicAdd(hist + bucket_of(geo, j, nb), 1);
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += 256)
    if (hist[b]) atomicAdd(cnt + b, hist[b]);
}

// One workgroup: bucket starts (exclusive scan of the counts) and the work
// items (bucket, first sorted position, length <= kLdsCols).
__global__ __launch_bounds__(1024) void bucket_scan_kernel(const int32_t* __restrict__ cnt, int nb,
                                                           int32_t* __restrict__ bstart,
                                                           int4* __restrict__ items,
                                                           int32_t* __restrict__ nitems) {
  __shared__ int32_t s_cols[1024], s_items[1024];
  const int tid = threadIdx.x;
  const int per = (nb + 1023) / 1024;
  const int b0 = tid * per, b1 = (b0 + per < nb) ? b0 + per : nb;
  int my_cols = 0, my_items = 0;
  for (int b = b0; b < b1; ++b) {
    my_cols += cnt[b];
    my_items += (cnt[b] + kLdsCols - 1) / kLdsCols;
  }
  s_cols[tid] = my_cols;
  s_items[tid] = my_items;
  __syncthreads();
  // inclusive Hillis-Steele scan of both arrays
  for (int off = 1; off < 1024; off <<= 1) {
    int c = 0, it = 0;
    if (tid >= off) {
      c = s_cols[tid - off];
      it = s_items[tid - off];
    }
    __syncthreads();
    s_cols[tid] += c;
    s_items[tid] += it;
    __syncthreads();
  }
  int col = s_cols[tid] - my_cols, item = s_items[tid] - my_items;
  for (int b = b0; b < b1; ++b) {
    bstart[b] = col;
    for (int s = 0; s < cnt[b]; s += kLdsCols) {
      const int len = (cnt[b] - s < kLdsCols) ? cnt[b] - s : kLdsCols;
      items[item++] = make_int4(b, col + s, len, 0);
    }
    col += cnt[b];
  }
  if (tid == 1023) *nitems = s_items[1023];
}

// Positions: a local rank from LDS atomics, one global atomic per non-empty
// bucket to reserve this workgroup's run of positions.  (The order inside a
// bucket only decides which workgroup builds a column, not its values.)
__global__ __launch_bounds__(256) void bucket_scatter_kernel(const ColGeom* __restrict__ geo,
                                                             int64_t ncols, int nb,
                                                             const int32_t* __restrict__ bstart,
                                                             int32_t* __restrict__ cursor,
                                                             int32_t* __restrict__ order) {
  extern __shared__ int32_t sh[];  // nb local counts, then nb bases
  int32_t* lcnt = sh;
  int32_t* base = sh + nb;
  for (int b = threadIdx.x; b < nb; b += 256) lcnt[b] = 0;
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int b = 0, r = 0;
  if (j < ncols) {
    b = bucket_of(geo, j, nb);
    r = atomicAdd(lcnt + b, 1);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nb; q += 256)
    if (lcnt[q]) base[q] = bstart[q] + atomicAdd(cursor + q, lcnt[q]);
  __syncthreads();
  if (j < ncols) order[base[b] + r] = (int32_t)j;
}

// --------------------------------------------------------------- build -----
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Float64 coordinate work of one element, in the oracle's order:
// sx = ct*ux + st*uy, sy = (-st)*ux + ct*uy, col = c + sx, row = c + sy.
struct Tap {
  int idx;           // LDS index of (r0, c0) in the bordered array
  bool ok;           // all four taps inside the bordered array
  float fx, gx, fy, gy;  // fx, 1-fx, fy, 1-fy (float32 of the float64 values)
};

__device__ __forceinline__ Tap tap_coords(double ctux, double mstux, double stuy, double ctuy,
                                          double c, int n, int ls) {
#pragma clang fp contract(off)
  const double sx = ctux + stuy;
  const double sy = mstux + ctuy;
  const double colf = c + sx;
  const double rowf = c + sy;
  const double c0f = floor(colf);
  const double r0f = floor(rowf);
  const double fx = colf - c0f;
  const double fy = rowf - r0f;
  Tap t;
  t.fx = (float)fx;
  t.gx = (float)(1.0 - fx);
  t.fy = (float)fy;
  t.gy = (float)(1.0 - fy);
  // |colf|, |rowf| < 3n, so the integer conversions are exact.  Taps r0, r0+1
  // (c0, c0+1) lie in the bordered array iff -1 <= r0, c0 <= n-1.
  const int c0 = (int)c0f, r0 = (int)r0f;
  t.ok = ((unsigned)(r0 + 1) <= (unsigned)n) && ((unsigned)(c0 + 1) <= (unsigned)n);
  t.idx = t.ok ? (r0 + 1) * ls + (c0 + 1) : 0;
  return t;
}

template <int E, bool FULL>
__global__ __launch_bounds__(1024) void build_lds_kernel(const float* __restrict__ cube, int K,
                                                         const ColGeom* __restrict__ geo,
                                                         const int32_t* __restrict__ order,
                                                         const int4* __restrict__ items,
                                                         const int32_t* __restrict__ nitems,
                                                         int nb, int n, int ls, int64_t M,
                                                         float* __restrict__ A,
                                                         double* __restrict__ tau) {
  // (n+2) rows of pairs (P_k, P_{k+1}) with a zero border, row stride ls >= n+2
  extern __shared__ float2 P2[];
  if ((int)blockIdx.x >= *nitems) return;  // uniform: surplus workgroups of the upper bound
  const int4 it = items[blockIdx.x];
  const int bkt = it.x, start = it.y, len = it.z;
  const bool zero_bucket = bkt == nb - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int np = n + 2;
  if (!zero_bucket) {
    const float* Pk = cube + (int64_t)bkt * M;
    const float* Pk1 = (K > 1) ? Pk + M : nullptr;
    // zero border
    for (int idx = tid; idx < 4 * np; idx += 1024) {
      const int side = idx / np, t = idx % np;
      const int pos = side == 0 ? t : side == 1 ? (np - 1) * ls + t
                    : side == 2 ? t * ls : t * ls + np - 1;
      P2[pos] = make_float2(0.0f, 0.0f);
    }
    // interior, 4 pixels (16 B of each PSF) per thread and step when rows allow
    if ((n & 3) == 0 && (reinterpret_cast<uintptr_t>(cube) & 15) == 0) {
      const int nq = n >> 2;
      for (int q = tid; q < n * nq; q += 1024) {
        const int rr = q / nq, cc = 4 * (q - rr * nq);
        const f32x4 a = *reinterpret_cast<const f32x4*>(Pk + rr * n + cc);
        const f32x4 b = Pk1 ? *reinterpret_cast<const f32x4*>(Pk1 + rr * n + cc)
                            : (f32x4){0.f, 0.f, 0.f, 0.f};
        float2* dst = P2 + (rr + 1) * ls + cc + 1;
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = make_float2(a[e], b[e]);
      }
    } else {
      for (int q = tid; q < n * n; q += 1024) {
        const int rr = q / n, cc = q - rr * n;
        P2[(rr + 1) * ls + cc + 1] = make_float2(Pk[q], Pk1 ? Pk1[q] : 0.0f);
      }
    }
  }
  __syncthreads();
  if (wave >= len) return;  // no barrier below
  const int64_t j = order[start + wave];
  float* col = A + j * M;
  if (zero_bucket) {
    for (int a = 0; a < n; ++a)
#pragma unroll
      for (int v = 0; v < E; ++v) {
        const int b = lane + 64 * v;
        if (FULL || b < n) __builtin_nontemporal_store(0.0f, col + a * n + b);
      }
    if (lane == 0) tau[j] = 0.0;
    return;
  }
  const ColGeom g = geo[j];
  const double c = (double)(n - 1) * 0.5;
  const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
  double ctux[E], mstux[E];
#pragma unroll
  for (int v = 0; v < E; ++v) {
#pragma clang fp contract(off)
    const double ux = (double)(lane + 64 * v) - c;
    ctux[v] = g.ct * ux;
    mstux[v] = (-g.st) * ux;
  }
  double tsum = 0.0;
  for (int a = 0; a < n; ++a) {
    double stuy, ctuy;
    {
#pragma clang fp contract(off)
      const double uy = (double)a - c;
      stuy = g.st * uy;
      ctuy = g.ct * uy;
    }
    float rowsum = 0.0f;
#pragma unroll
    for (int v = 0; v < E; ++v) {
      const int b = lane + 64 * v;
      if (FULL || b < n) {
        const Tap t = tap_coords(ctux[v], mstux[v], stuy, ctuy, c, n, ls);
        const float2 p00 = P2[t.idx], p01 = P2[t.idx + 1];
        const float2 p10 = P2[t.idx + ls], p11 = P2[t.idx + ls + 1];
        const float q00 = fmaf(wk1, p00.y, wk0 * p00.x);
        const float q01 = fmaf(wk1, p01.y, wk0 * p01.x);
        const float q10 = fmaf(wk1, p10.y, wk0 * p10.x);
        const float q11 = fmaf(wk1, p11.y, wk0 * p11.x);
        float val = (t.gy * t.gx) * q00;
        val = fmaf(t.gy * t.fx, q01, val);
        val = fmaf(t.fy * t.gx, q10, val);
        val = fmaf(t.fy * t.fx, q11, val);
        val = t.ok ? val : 0.0f;
        __builtin_nontemporal_store(val, col + a * n + b);
        rowsum += val;
      }
    }
    tsum += (double)rowsum;
  }
  tsum = wave_sum_f64(tsum);
  if (lane == 0) tau[j] = tsum;
}

// ------------------------------------------------------- stable sort -----
constexpr int kSortBlock = 1024;  // columns per block of the stable sort

// Inclusive sum of v over the workgroup's threads (16 waves), fixed order.
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t* tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t u = __shfl_up(v, off, 64);
    if (lane >= off) v += u;
  }
  if (lane == 63) tot[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += tot[w];
  __syncthreads();
  return v;
}

// The work items of a bracket's run of c > 0 positions from `start`, one per
// window of 16 positions, from items[first]: lane of `lanes` takes every lanes-th.
__device__ __forceinline__ void write_items(int4* __restrict__ items, int b, int32_t start, int32_t c,
                                            int32_t first, int lane, int lanes) {
  for (int w = start / 16 * 16 + 16 * lane, i = lane; w < start + c; w += 16 * lanes, i += lanes) {
    const int lo = w > start ? w : start;
    const int hi = (w + 16 < start + c) ? w + 16 : start + c;
    items[first + i] = make_int4(b, lo, hi - lo, w);
  }
}

// The same for up to 1024 brackets, thread b holding bracket b's: a wave per
// bracket (one thread each took 9 of 16 us for 10000 positions of 11 brackets).
__device__ __forceinline__ void write_all_items(int4* __restrict__ items, int nb, int32_t start, int32_t c,
                                                int32_t first, int32_t* s_start, int32_t* s_count,
                                                int32_t* s_first) {
  const int tid = threadIdx.x;
  s_start[tid] = start;
  s_count[tid] = c;
  s_first[tid] = first;
  __syncthreads();
  for (int b = tid >> 6; b < nb; b += 16)
    if (s_count[b] > 0) write_items(items, b, s_start[b], s_count[b], s_first[b], tid & 63, 64);
}

// One workgroup.  cnt[blk][b] becomes the first slot of bucket b's columns of
// block blk (bucket start + the bucket's columns in earlier blocks); items
// (bucket, first slot, length, 16-slot window start) cover every bucket along
// 16-slot windows.
__global__ __launch_bounds__(1024) void sort_scan_kernel(int32_t* __restrict__ cnt, int64_t nblk,
                                                         int nb, int4* __restrict__ items,
                                                         int32_t* __restrict__ nitems) {
  __shared__ int32_t s_cols[1024], s_items[1024], waves[16];
  __shared__ int32_t tot[kLdsMaxBuckets];
  static_assert(kLdsMaxBuckets >= 1024, "write_all_items");
  const int tid = threadIdx.x;
  for (int b = tid; b < nb; b += 1024) {  // independent loads: no store in between
    int32_t run = 0;
    for (int64_t k = 0; k < nblk; ++k) run += cnt[k * nb + b];
    tot[b] = run;
  }
  __syncthreads();
  const int per = (nb + 1023) / 1024;
  const int b0 = tid * per, b1 = (b0 + per < nb) ? b0 + per : nb;
  int my_cols = 0;
  for (int b = b0; b < b1; ++b) my_cols += tot[b];
  const int32_t first = block_scan(my_cols, waves) - my_cols;
  // bucket starts, then the items of each bucket
  int start = first, my_items = 0;
  for (int b = b0; b < b1; ++b) {
    const int c = tot[b];
    if (c > 0) my_items += (start + c - 1) / 16 - start / 16 + 1;
    start += c;
  }
  const int32_t all_items = block_scan(my_items, waves);
  start = first;
  int item = all_items - my_items;
  for (int b = b0; b < b1; ++b) {
    const int c = tot[b];
    int32_t run = start;  // first slot of bucket b in each block
    for (int64_t k0 = 0; k0 < nblk; k0 += 16) {
      int32_t v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = (k0 + u < nblk) ? cnt[(k0 + u) * nb + b] : 0;
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (k0 + u < nblk) {
          cnt[(k0 + u) * nb + b] = run;
          run += v[u];
        }
    }
    if (per > 1 && c > 0) {
      write_items(items, b, start, c, item, 0, 1);
      item += (start + c - 1) / 16 - start / 16 + 1;
    }
    start += c;
  }
  if (tid == 1023) *nitems = all_items;
  if (per == 1) {
    const int32_t c = tid < nb ? tot[tid] : 0;
    __syncthreads();
    write_all_items(items, nb, start - c, c, item, s_cols, tot, s_items);
  }
}

// 16-bit packing: M16[g][i][u] = RN16(A32[8g+u][i] * 2^-e), zeros past ncols.
// Two rows per thread: 8 x 8-byte loads (one per column; 512 B per wave and
// column) and 32 contiguous bytes stored.
template <bool BF16>
__global__ __launch_bounds__(256) void pack16_kernel(const float* __restrict__ A32,
                                                     const ColGeom* __restrict__ geo,
                                                     int64_t M, int64_t ncols,
                                                     u32x4* __restrict__ Mp) {
  const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2;
  const int64_t grp = blockIdx.y;
  if (i0 >= M) return;
  const bool pair = (M % 2) == 0;  // then i0 + 1 < M and the 8-byte loads are aligned
  float v[8][2];
  int32_t ex[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int64_t j = grp * 8 + u;
    v[u][0] = v[u][1] = 0.0f;
    ex[u] = 0;
    if (j < ncols) {
      ex[u] = geo[j].e;
      const float* src = A32 + j * M + i0;
      if (pair) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 t = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(src));
        v[u][0] = t.x;
        v[u][1] = t.y;
      } else {
        v[u][0] = src[0];
        v[u][1] = (i0 + 1 < M) ? src[1] : 0.0f;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (i0 + r >= M) break;
    uint32_t h[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float x = ldexpf(v[u][r], -ex[u]);
      if (BF16) {
        uint32_t w = __float_as_uint(x);
        w += 0x7FFFu + ((w >> 16) & 1u);
        h[u] = w >> 16;
      } else {
        h[u] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x);
      }
    }
    u32x4 pk;
    pk.x = h[0] | (h[1] << 16);
    pk.y = h[2] | (h[3] << 16);
    pk.z = h[4] | (h[5] << 16);
    pk.w = h[6] | (h[7] << 16);
    __builtin_nontemporal_store(pk, Mp + grp * M + i0 + r);
  }
}

// --------------------------------------------- rotation-orbit builds -----
// The scene grid (centre ((N-1)/2, (N-1)/2)) and the PSF grid (centre
// ((n-1)/2, (n-1)/2)) are both invariant under quarter turns.  Turning a
// scene pixel by 90 degrees about the star maps (x, y) to (-y, x) exactly
// (index arithmetic: (p, q) -> (q, N-1-p)), so the turned column has
// cos' = -sin and sin' = cos exactly and the same radius, bracket and
// weight; its source coordinates at image pixel (b', a') = (N-1-a, b) are
// the base column's at (b, a) -- the same float64 products added in the
// other order, which is exact.  Every entry of the turned column is
// therefore bitwise the base column's at the turned image pixel:
//   C1[b][n-1-a] = C2[n-1-a][n-1-b] = C3[n-1-b][a] = C0[a][b]
// for the orbit (j0, j1, j2, j3) of a base column j0 in the quadrant
// x > 0, y >= 0 (the centre pixel of an odd grid is its own orbit).  The
// orbit builds compute C0 once and write all four columns: a quarter of the
// coordinate and interpolation work per stored entry.  Base columns are
// sorted by bracket (stable), cut into windows of 16; a work item is the run
// of one bracket inside a window times a range of image rows (so a launch has
// many more items than compute units), and each wave builds one base column
// over the item's rows.  Column sums: per (row range, base column) partial
// sums in float64, added in row-range order by a last kernel.

// quadrant bases p in [N/2, N), q in [(N+1)/2, N); the centre last (odd N)
struct OrbitGrid {
  int N, plo, qlo, hq;
  int64_t n4;      // base columns with a 4-column orbit
  int64_t nreps;   // n4, plus the centre for odd N
};

__host__ __device__ inline OrbitGrid orbit_grid(int N) {
  OrbitGrid o;
  o.N = N;
  o.plo = N / 2;
  o.qlo = (N + 1) / 2;
  o.hq = N - o.qlo;
  o.n4 = (int64_t)(N - o.plo) * o.hq;
  o.nreps = o.n4 + (N & 1);
  return o;
}

// (columns are fewer than 2^31: 32-bit divisions)
__device__ __forceinline__ int64_t orbit_base(const OrbitGrid& o, int64_t t) {
  if (t < o.n4) {
    const uint32_t r = (uint32_t)t / (uint32_t)o.hq;
    const int64_t p = o.plo + (int64_t)r, q = o.qlo + (int64_t)((uint32_t)t - r * (uint32_t)o.hq);
    return p * o.N + q;
  }
  return (int64_t)(o.N / 2) * o.N + o.N / 2;  // centre
}

// rotation partners of base column j0 = p N + q (k quarter turns)
__device__ __forceinline__ int64_t orbit_member(int64_t j0, int N, int k) {
  const int64_t p = (uint32_t)j0 / (uint32_t)N, q = j0 - p * N;
  switch (k) {
    case 0: return j0;
    case 1: return q * N + (N - 1 - p);
    case 2: return (N - 1 - p) * N + (N - 1 - q);
    default: return (N - 1 - q) * N + p;
  }
}

__device__ __forceinline__ bool orbit_is_centre(int64_t j0, int N) {
  return (N & 1) && j0 == (int64_t)(N / 2) * N + N / 2;
}

// rows of an image-row range: a multiple of 32, about a quarter of the image
static inline int orbit_rows_per_range(int n) {
  const int q = (n + 3) / 4;
  return ((q + 31) / 32) * 32;
}

__global__ __launch_bounds__(kSortBlock) void orbit_count_kernel(const ColGeom* __restrict__ geo,
                                                                 OrbitGrid o, int nb,
                                                                 int32_t* __restrict__ cnt) {
  extern __shared__ int32_t hist[];  // nb
  for (int b = threadIdx.x; b < nb; b += kSortBlock) hist[b] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * kSortBlock + threadIdx.x;
  if (t < o.nreps) atomicAdd(hist + bucket_of(geo, orbit_base(o, t), nb), 1);  // order-free
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += kSortBlock) cnt[(int64_t)blockIdx.x * nb + b] = hist[b];
}

// Lanes of the wave with this lane's bracket (0 <= b < 2^bits; a lane outside the
// set has b < 0 and gets no meaningful mask, nor does it enter another's): one
// ballot per bit of the bracket number, whatever the number of brackets in the wave.
__device__ __forceinline__ uint64_t same_bracket(int b, int bits) {
  uint64_t m = __ballot(b >= 0);
  for (int i = 0; i < bits; ++i) {
    const uint64_t one = __ballot((b >> i) & 1);
    m &= ((b >> i) & 1) ? one : ~one;
  }
  return m;
}

__device__ __forceinline__ int bracket_bits(int nb) { return 32 - __builtin_clz(nb); }

// Stable placement of the base columns: a base's position is its block's first
// position of the bracket plus its rank among the block's earlier bases of the
// same bracket.  Each wave ranks its 64 bases (same_bracket); then the waves take their positions in order, each adding its counts
// to a per-bracket cursor in LDS that starts at the block's first positions.
__global__ __launch_bounds__(kSortBlock) void orbit_scatter_kernel(const ColGeom* __restrict__ geo,
                                                                   OrbitGrid o, int nb,
                                                                   const int32_t* __restrict__ first,
                                                                   int32_t* __restrict__ reps,
                                                                   int32_t* __restrict__ nitems) {
  extern __shared__ int32_t cursor[];  // nb
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int q = tid; q < nb; q += kSortBlock) cursor[q] = first[(int64_t)blockIdx.x * nb + q];
  const int64_t t = (int64_t)blockIdx.x * kSortBlock + tid;
  const bool valid = t < o.nreps;
  const int64_t j0 = valid ? orbit_base(o, t) : 0;
  const int b = valid ? bucket_of(geo, j0, nb) : -1;
  const uint64_t m = same_bracket(b, bracket_bits(nb));
  const int rank = __popcll(m & ((1ull << lane) - 1ull)), count = __popcll(m);
  __syncthreads();
  int pos = 0;
  for (int w = 0; w < kSortBlock / 64; ++w) {
    if (wave == w && valid) {
      pos = cursor[b] + rank;  // every lane reads before the wave's leaders add
      __builtin_amdgcn_wave_barrier();
      if (rank == 0) cursor[b] += count;
    }
    __syncthreads();
  }
  if (valid) {
    reps[pos] = (int32_t)j0;
    if (orbit_is_centre(j0, o.N)) nitems[1] = pos;
  }
}

// The whole sort of up to kSmallSort base columns in up to 1024 brackets in one
// workgroup: the counts of every wave of 64 columns by bracket in LDS, their
// running sums over the waves, the items, the positions; the same order and items
// as the three kernels above.  One launch, 13 us for 4096 columns of 63 brackets
// where the three took 18.
constexpr int kSmallSort = 4096;

__global__ __launch_bounds__(kSortBlock) void orbit_sort_kernel(const ColGeom* __restrict__ geo,
                                                                OrbitGrid o, int nb,
                                                                int32_t* __restrict__ reps,
                                                                int4* __restrict__ items,
                                                                int32_t* __restrict__ nitems) {
  constexpr int C = kSmallSort / kSortBlock;
  extern __shared__ int32_t cnt[];  // [waves of 64 columns][nb]
  __shared__ int32_t tot[16], s_start[kSortBlock], s_count[kSortBlock], s_first[kSortBlock];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = (int)((o.nreps + 63) / 64);
  int64_t j0[C];
  int b[C], rank[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int64_t t = c * kSortBlock + tid;
    j0[c] = t < o.nreps ? orbit_base(o, t) : 0;
    b[c] = t < o.nreps ? bucket_of(geo, j0[c], nb) : -1;
  }
  for (int q = tid; q < nw * nb; q += kSortBlock) cnt[q] = 0;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const uint64_t m = same_bracket(b[c], bracket_bits(nb));
    rank[c] = __popcll(m & ((1ull << lane) - 1ull));
    if (b[c] >= 0 && rank[c] == 0) cnt[(c * 16 + wave) * nb + b[c]] = __popcll(m);
  }
  __syncthreads();
  // bracket `tid`: its columns before every wave, and its total
  int32_t run = 0;
  if (tid < nb) {
#pragma unroll 8
    for (int w = 0; w < nw; ++w) {
      const int32_t v = cnt[w * nb + tid];
      cnt[w * nb + tid] = run;
      run += v;
    }
  }
  const int32_t start = block_scan(run, tot) - run;
  const int32_t mine = run > 0 ? (start + run - 1) / 16 - start / 16 + 1 : 0;
  const int32_t last = block_scan(mine, tot);
  if (tid < nb) {
#pragma unroll 8
    for (int w = 0; w < nw; ++w) cnt[w * nb + tid] += start;
  }
  if (tid == kSortBlock - 1) nitems[0] = last;
  write_all_items(items, nb, start, run, last - mine, s_start, s_count, s_first);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if (b[c] < 0) continue;
    const int32_t pos = cnt[(c * 16 + wave) * nb + b[c]] + rank[c];
    reps[pos] = (int32_t)j0[c];
    if (orbit_is_centre(j0[c], o.N)) nitems[1] = pos;
  }
}

// the partial sums of base position s: row ranges (16-bit) or tiles (float32),
// in order
__device__ __forceinline__ double orbit_sum(const double* __restrict__ part, int nparts,
                                            int64_t nreps, int64_t s) {
  double t = 0.0;
  for (int r0 = 0; r0 < nparts; r0 += 8) {  // 8 loads in flight
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = r0 + u < nparts ? part[(int64_t)(r0 + u) * nreps + s] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) t += v[u];
  }
  return t;
}

// column sums, for every member
__global__ __launch_bounds__(256) void orbit_tau_kernel(const int32_t* __restrict__ reps, OrbitGrid o,
                                                        const double* __restrict__ part, int nparts,
                                                        double* __restrict__ tau) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= o.nreps) return;
  const double t = orbit_sum(part, nparts, o.nreps, s);
  const int64_t j0 = reps[s];
  const int members = orbit_is_centre(j0, o.N) ? 1 : 4;
  for (int k = 0; k < members; ++k) tau[orbit_member(j0, o.N, k)] = t;
}

// The end of a flux-preserving build's first pass: the float32 scale of every
// base column, the PSF's flux over the plain column's sum, and for the 16-bit
// forms the members' exponent from the rescaled bound; identically zero columns
// keep scale 1 and their exponent.
__global__ __launch_bounds__(256) void orbit_scale_kernel(const int32_t* __restrict__ reps, OrbitGrid o,
                                                          const double* __restrict__ part, int nparts,
                                                          int K, ColGeom* __restrict__ geo,
                                                          const OrbitFlux fx) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= o.nreps) return;
  const double old = orbit_sum(part, nparts, o.nreps, s);
  const int64_t j0 = reps[s];
  const ColGeom g = geo[j0];
  if (g.k < 0) {
    fx.colscale[j0] = 1.0f;
    return;
  }
  const double t = (K == 1) ? fx.sums[0] : (1.0 - g.w) * fx.sums[g.k] + g.w * fx.sums[g.k + 1];
  const float sf = (float)((old != 0.0) ? t / old : 1.0);
  fx.colscale[j0] = sf;
  if (!fx.exps) return;
  const double bound = (K == 1) ? (double)fx.pmax[0]
                                : (1.0 - g.w) * (double)fx.pmax[g.k] + g.w * (double)fx.pmax[g.k + 1];
  const int32_t e = scale_exponent(bound * fabs((double)sf));
  const int members = orbit_is_centre(j0, o.N) ? 1 : 4;
  for (int k = 0; k < members; ++k) {
    const int64_t j = orbit_member(j0, o.N, k);
    geo[j].e = e;
    fx.exps[j] = e;
  }
}

// The end of a 16-bit build: workgroups below nsum write column sums and the slot
// maps: base position s in block s/8 of 8 bases, member k in group 4 (s/8) + k,
// slot 32 (s/8) + 8 k + s%8.  Slots without a column (members 1 to 3 of the
// centre of an odd scene, bases that fill up the last block, the slots up to
// ncols_pad) are padding, perm -1; those that the build kernels do not write as
// zeros, whole groups at the end (`tail` of them) and the centre's members, the
// remaining workgroups set to zero.
__global__ __launch_bounds__(256) void orbit16_end_kernel(const int32_t* __restrict__ reps, OrbitGrid o,
                                                          const double* __restrict__ part, int nparts,
                                                          const ColGeom* __restrict__ geo,
                                                          const int32_t* __restrict__ nitems, int nsum,
                                                          int tail, int64_t M, const Orbit16Out out) {
  const int64_t whole = (o.nreps + 7) / 8 * 8;
  if ((int)blockIdx.x >= nsum) {
    const int64_t rowblocks = (M + 255) / 256, wg = (int64_t)blockIdx.x - nsum;
    const int y = (int)(wg / rowblocks);
    const int64_t i = (wg - y * rowblocks) * 256 + threadIdx.x;
    if (i >= M) return;
    uint16_t* Mh = reinterpret_cast<uint16_t*>(out.lib);
    if (y < tail) {
      *reinterpret_cast<u32x4*>(Mh + ((whole / 2 + y) * M + i) * 8) = (u32x4){0u, 0u, 0u, 0u};
    } else {
      const int32_t s = nitems[1];
      Mh[(((int64_t)(s / 8) * 4 + y - tail + 1) * M + i) * 8 + s % 8] = 0;
    }
    return;
  }
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool valid = s < o.nreps;
  if (s < whole) {
    const int64_t j0 = valid ? reps[s] : 0;
    const bool centre = valid && orbit_is_centre(j0, o.N);
    const double t = valid ? orbit_sum(part, nparts, o.nreps, s) : 0.0;
    const int32_t e = valid ? geo[j0].e : kZeroColumnExp;  // the members share the radius
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t slot = (int32_t)((s / 8) * 32 + 8 * k + s % 8);
      const bool column = valid && (k == 0 || !centre);
      const int64_t j = column ? orbit_member(j0, o.N, k) : -1;
      out.perm[slot] = (int32_t)j;
      out.eslot[slot] = e;
      if (column) {
        out.slot_of[j] = slot;
        out.tau[j] = t;
      }
    }
  }
  const int64_t pad = 4 * whole + s;  // fewer than 64 slots
  if (pad < out.ncols_pad) {
    out.perm[pad] = -1;
    out.eslot[pad] = kZeroColumnExp;
  }
}

// the bordered pair (P_k, P_{k+1}) with its zero border, as the LDS build
__device__ __forceinline__ void stage_pair(float2* __restrict__ P2, const float* __restrict__ cube,
                                           int bkt, int K, int n, int ls, int64_t M, int tid) {
  const int np = n + 2;
  const float* Pk = cube + (int64_t)bkt * M;
  const float* Pk1 = (K > 1) ? Pk + M : nullptr;
  for (int idx = tid; idx < 4 * np; idx += 1024) {
    const int side = idx / np, t = idx % np;
    const int pos = side == 0 ? t : side == 1 ? (np - 1) * ls + t : side == 2 ? t * ls : t * ls + np - 1;
    P2[pos] = make_float2(0.0f, 0.0f);
  }
  if ((n & 3) == 0 && (reinterpret_cast<uintptr_t>(cube) & 15) == 0) {
    const int nq = n >> 2;
    for (int q = tid; q < n * nq; q += 1024) {
      const int rr = q / nq, cc = 4 * (q - rr * nq);
      const f32x4 a = *reinterpret_cast<const f32x4*>(Pk + rr * n + cc);
      const f32x4 b = Pk1 ? *reinterpret_cast<const f32x4*>(Pk1 + rr * n + cc) : (f32x4){0.f, 0.f, 0.f, 0.f};
      float2* dst = P2 + (rr + 1) * ls + cc + 1;
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[e] = make_float2(a[e], b[e]);
    }
  } else {
    for (int q = tid; q < n * n; q += 1024) {
      const int rr = q / n, cc = q - rr * n;
      P2[(rr + 1) * ls + cc + 1] = make_float2(Pk[q], Pk1 ? Pk1[q] : 0.0f);
    }
  }
}

// One element of the base column (the LDS build's arithmetic).
__device__ __forceinline__ float orbit_value(const float2* __restrict__ P2, double ctux, double mstux,
                                             double stuy, double ctuy, double c, int n, int ls,
                                             float wk0, float wk1) {
  const Tap t = tap_coords(ctux, mstux, stuy, ctuy, c, n, ls);
  const float2 p00 = P2[t.idx], p01 = P2[t.idx + 1];
  const float2 p10 = P2[t.idx + ls], p11 = P2[t.idx + ls + 1];
  const float q00 = fmaf(wk1, p00.y, wk0 * p00.x);
  const float q01 = fmaf(wk1, p01.y, wk0 * p01.x);
  const float q10 = fmaf(wk1, p10.y, wk0 * p10.x);
  const float q11 = fmaf(wk1, p11.y, wk0 * p11.x);
  float val = (t.gy * t.gx) * q00;
  val = fmaf(t.gy * t.fx, q01, val);
  val = fmaf(t.fy * t.gx, q10, val);
  val = fmaf(t.fy * t.fx, q11, val);
  return t.ok ? val : 0.0f;
}

// Modes of the float32 orbit kernels: the plain build; only the column sums
// (no stores: the first pass of a flux-preserving build); or every value
// multiplied by its column's float32 scale before it is stored and summed
// (the second pass).
constexpr int kPlain = kOrbitPlain, kSumsOnly = kOrbitSumsOnly, kScaled = kOrbitScaled;
// and the first pass that also keeps the base columns (A: the column of base
// position 0), which the 16-bit builds' second pass reads
constexpr int kBases = kOrbitScaled + 1;

// 16-byte run of a column.  VEC (n a multiple of 32): the eight lanes of a tile
// row fill a whole 128-byte line.  Otherwise the run starts at any float and
// the lines at its ends are shared with the next tiles: ordinary stores, so
// that their parts meet in the L2.
template <bool VEC>
__device__ __forceinline__ void store_run(float* p, const f32x4 v) {
  if constexpr (VEC) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
  } else {
    *reinterpret_cast<f32x4u*>(p) = v;
  }
}

// The runs of one row (x[r][0..3] at row a, columns bb ..) in members 0 and 2,
// and of the block's four columns (rows ab ..) in members 1 and 3.
template <bool VEC>
__device__ __forceinline__ void store_row_runs(const float* xr, float* C0, float* C2, int a, int bb,
                                               int n, bool centre) {
  store_run<VEC>(C0 + (int64_t)a * n + bb, (f32x4){xr[0], xr[1], xr[2], xr[3]});
  if (!centre)
    store_run<VEC>(C2 + (int64_t)(n - 1 - a) * n + (n - 4 - bb), (f32x4){xr[3], xr[2], xr[1], xr[0]});
}

template <bool VEC>
__device__ __forceinline__ void store_column_runs(const float (*x)[4], float* C1, float* C3, int ab,
                                                  int bb, int n) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = bb + q;
    store_run<VEC>(C1 + (int64_t)b * n + (n - 4 - ab), (f32x4){x[3][q], x[2][q], x[1][q], x[0][q]});
    store_run<VEC>(C3 + (int64_t)(n - 1 - b) * n + ab, (f32x4){x[0][q], x[1][q], x[2][q], x[3][q]});
    __builtin_amdgcn_sched_barrier(0);
  }
}

// the same entries one by one, for images of fewer than 4 pixels a side
__device__ __forceinline__ void store_block_scalar(const float (*x)[4], float* C0, float* C1, float* C2,
                                                   float* C3, int ab, int bb, int n, bool centre) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int a = ab + r, b = bb + q;
      if (a >= n || b >= n) continue;
      C0[(int64_t)a * n + b] = x[r][q];
      if (centre) continue;
      C1[(int64_t)b * n + (n - 1 - a)] = x[r][q];
      C2[(int64_t)(n - 1 - a) * n + (n - 1 - b)] = x[r][q];
      C3[(int64_t)(n - 1 - b) * n + a] = x[r][q];
    }
}

// First row (column) of the 4 x 4 block that covers v0 .. v0 + 3: with n not a
// multiple of 4 the last block of the image is moved back to end at its edge
// (it forms up to 3 rows or columns of its neighbour again, with the same
// values; they are summed once, by the neighbour).
template <bool VEC>
__device__ __forceinline__ int block_start(int v0, int n) {
  return VEC ? v0 : max(min(v0, n - 4), 0);
}

// What a wave needs of the base column it works on (the same in every lane).
struct OrbitCol {
  int64_t j0, pos;  // column and base position
  double ct, st, w;
  int k;
  float scale;  // flux-preserving scale
};

template <int MODE>
__device__ __forceinline__ OrbitCol load_orbit_col(const int32_t* __restrict__ reps,
                                                   const ColGeom* __restrict__ geo,
                                                   const float* __restrict__ colscale, int64_t sp) {
  OrbitCol o;
  o.j0 = reps[sp];
  o.pos = sp;
  const ColGeom* g = geo + o.j0;
  o.ct = g->ct;
  o.st = g->st;
  o.w = g->w;
  o.k = g->k;
  o.scale = (MODE == kScaled) ? colscale[o.j0] : 1.0f;
  return o;
}

// Tiles of 32 x 32 pixels cover the image; lane (i, k) = (lane / 8, lane % 8)
// of the wave that forms a tile takes the 4 x 4 block at its rows 4i..,
// columns 4k...  The lane then holds four runs of four entries for every
// member (C0, C2 along rows; C1, C3 along the base column's image columns), so
// every store is 16 bytes and each store instruction writes eight runs of 128
// bytes of one member.  value(ctux, mstux, stuy, ctuy) is the entry at the
// block's pixel; the entries' sum is added to tsum.  VEC: n a multiple of 32,
// whole lines.  Otherwise the runs are unaligned and the image's last blocks
// overlap their neighbours (block_start), so that no entry needs a store of
// its own.
template <bool VEC, int MODE, typename Value>
__device__ __forceinline__ void orbit_block(Value value, const OrbitCol& g, double c, int n, int N,
                                            int64_t M, int ab0, int bb0, float* A, double& tsum) {
  const bool centre = orbit_is_centre(g.j0, N);
  float* C0 = A + g.j0 * M;
  float* C1 = A + orbit_member(g.j0, N, 1) * M;
  float* C2 = A + orbit_member(g.j0, N, 2) * M;
  float* C3 = A + orbit_member(g.j0, N, 3) * M;
  const int ab = block_start<VEC>(ab0, n), bb = block_start<VEC>(bb0, n);
  double ctux[4], mstux[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma clang fp contract(off)
    const double ux = (double)(bb + q) - c;
    ctux[q] = g.ct * ux;
    mstux[q] = (-g.st) * ux;
  }
  float x[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int a = ab + r;
    double stuy, ctuy;
    {
#pragma clang fp contract(off)
      const double uy = (double)a - c;
      stuy = g.st * uy;
      ctuy = g.ct * uy;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[r][q] = 0.0f;
      if (VEC || (a < n && bb + q < n)) {  // false for n < 4 only
        x[r][q] = value(ctux[q], mstux[q], stuy, ctuy);
        if constexpr (MODE == kScaled) x[r][q] *= g.scale;
        if (VEC || (a >= ab0 && bb + q >= bb0)) tsum += (double)x[r][q];
      }
      if (q == 1) __builtin_amdgcn_sched_barrier(0);  // two elements in flight
    }
    // the row's runs of C0 and C2
    if (VEC || n >= 4) store_row_runs<VEC>(x[r], C0, C2, a, bb, n, centre);
    // one row of the block at a time: bounds the live coordinate temporaries
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!VEC && n < 4)
    store_block_scalar(x, C0, C1, C2, C3, ab, bb, n, centre);
  else if (!centre)
    store_column_runs<VEC>(x, C1, C3, ab, bb, n);
}

// the modes that store no turned member
constexpr bool base_only(int mode) { return mode == kSumsOnly || mode == kBases; }

// The tile of a base column whose turns are not stored: neighbouring lanes take
// neighbouring pixels, lane (i, k) those at rows a0 + i + 8 p, columns b0 + k + 8
// q, so that the taps of a step lie close together in LDS (1.2 to 1.5 lanes to a
// bank where lanes four pixels apart put 2.3) and the steps past the image's edge
// are left out whole: 101^2 takes 169 steps of 64 pixels a column instead of 256.
// (First pass for 101^2 PSFs of a 101^2 scene with the spline: 186 us with the
// blocks of orbit_block, 154 so.)
template <int MODE, typename Value>
__device__ __forceinline__ void orbit_patch(Value value, const OrbitCol& g, double c, int n, int64_t M,
                                            int a0, int b0, int lane, float* A, double& tsum) {
  const int li = lane >> 3, lk = lane & 7;
  float* C0 = A + g.pos * M;
  double ctux[4], mstux[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma clang fp contract(off)
    const double ux = (double)(b0 + lk + 8 * q) - c;
    ctux[q] = g.ct * ux;
    mstux[q] = (-g.st) * ux;
  }
  auto rows = [&](auto whole) {  // whole: a tile inside the image, no bounds to test
    for (int p = 0; p < 4 && (whole.value || a0 + 8 * p < n); ++p) {  // uniform
      const int a = a0 + li + 8 * p;
      double stuy, ctuy;
      {
#pragma clang fp contract(off)
        const double uy = (double)a - c;
        stuy = g.st * uy;
        ctuy = g.ct * uy;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = b0 + lk + 8 * q;
        if (!whole.value && b0 + 8 * q >= n) break;  // uniform
        if (whole.value || (a < n && b < n)) {
          const float x = value(ctux[q], mstux[q], stuy, ctuy);
          tsum += (double)x;
          if constexpr (MODE == kBases) C0[(int64_t)a * n + b] = x;
        }
        if (q == 1) __builtin_amdgcn_sched_barrier(0);  // two elements in flight
      }
    }
  };
  if (a0 + 32 <= n && b0 + 32 <= n)
    rows(std::true_type{});
  else
    rows(std::false_type{});
}

// a 32 x 32 tile at (a0, b0) of a base column
template <bool VEC, int MODE, typename Value>
__device__ __forceinline__ void orbit_tile(Value value, const OrbitCol& g, double c, int n, int N,
                                           int64_t M, int a0, int b0, int lane, float* A, double& tsum) {
  if constexpr (base_only(MODE)) {
    orbit_patch<MODE>(value, g, c, n, M, a0, b0, lane, A, tsum);
  } else {
    const int ab0 = a0 + 4 * (lane >> 3), bb0 = b0 + 4 * (lane & 7);
    if (ab0 < n && bb0 < n) orbit_block<VEC, MODE>(value, g, c, n, N, M, ab0, bb0, A, tsum);
  }
}

// Float32 orbit build, the pair in LDS.  A workgroup (blockIdx.x: item = run of
// one bracket inside a window of 16 bases; blockIdx.y: a few bases of the
// window) stages the pair and its waves share out the tiles of its bases, so
// that the waves write neighbouring tiles of one column together: where n is
// not a multiple of 32 the tiles' rows and columns share 128-byte lines, and
// the two halves of a line meet in the L2 before it is written back.  Bound by
// the write stream: at 128^2 (1 GiB) 226 us against 250 us with a wave per
// column and row range; at 127^2 465 us against 2475 us with a wave per column
// and a store per entry, 670 us with 16-byte stores, which then evicted half
// lines.
// Four bases give 16 waves of work from 64^2 pixels; smaller images take more,
// so that the pair is staged for a full workgroup.
__host__ __device__ constexpr int orbit_sub(int nt) { return nt == 1 ? 16 : nt == 2 ? 8 : 4; }
template <bool VEC, int MODE>
__global__ __launch_bounds__(1024) void build_orbit_kernel(const float* __restrict__ cube, int K,
                                                           const ColGeom* __restrict__ geo,
                                                           const int32_t* __restrict__ reps,
                                                           const int4* __restrict__ items,
                                                           const int32_t* __restrict__ nitems,
                                                           int nb, int n, int ls, int N, int64_t M,
                                                           int nt, int64_t nreps,
                                                           float* __restrict__ A,
                                                           double* __restrict__ part,
                                                           const float* __restrict__ colscale) {
  extern __shared__ float2 P2[];
  if ((int)blockIdx.x >= *nitems) return;  // uniform: surplus workgroups of the upper bound
  const int4 it = items[blockIdx.x];
  const int sub = orbit_sub(nt);
  const int bkt = it.x, w0 = it.w + sub * (int)blockIdx.y;
  const int first = max(it.y, w0), last = min(it.y + it.z, w0 + sub);
  if (first >= last) return;  // uniform: no base of the item among these
  const bool zero_bucket = bkt == nb - 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (!zero_bucket) stage_pair(P2, cube, bkt, K, n, ls, M, tid);
  __syncthreads();
  const double c = (double)(n - 1) * 0.5;
  const int ntiles = nt * nt, nwork = (last - first) * ntiles;
  if (wave >= nwork) return;  // no barrier below
  OrbitCol g = load_orbit_col<MODE>(reps, geo, colscale, first + wave / ntiles);
  for (int t = wave; t < nwork; t += 16) {  // uniform per wave
    const int sp = first + t / ntiles, tile = t % ntiles;
    const OrbitCol next = load_orbit_col<MODE>(reps, geo, colscale, first + min(t + 16, nwork - 1) / ntiles);
    const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
    const int a0 = 32 * (tile / nt), b0 = 32 * (tile % nt);
    double tsum = 0.0;
    if (zero_bucket)  // identically zero orbit
      orbit_tile<VEC, MODE>([](double, double, double, double) { return 0.0f; }, g, c, n, N, M, a0, b0,
                            lane, A, tsum);
    else
      orbit_tile<VEC, MODE>(
          [&](double ctux, double mstux, double stuy, double ctuy) {
            return orbit_value(P2, ctux, mstux, stuy, ctuy, c, n, ls, wk0, wk1);
          },
          g, c, n, N, M, a0, b0, lane, A, tsum);
    tsum = wave_sum_f64(tsum);
    if (lane == 0) part[(int64_t)tile * nreps + sp] = tsum;
    g = next;
  }
}

// Float32 orbit build for pairs larger than the LDS (n > 141).  The
// rotation map is affine, so a 32 x 32 tile of the base column draws its taps
// from a small box of the bordered pair: every float64 step of the source
// coordinates (the products with the cosine and sine, the two sums) is
// correctly rounded, hence monotone in the pixel's column for a fixed row and
// in its row for a fixed column, so the extreme source rows and columns over a
// tile are those of its four corners, exactly.  The box spans at most
// 31 (|cos| + |sin|) <= 43.85 source units, i.e. at most 45 tap origins and 46
// rows (columns) of the bordered array.  Each wave stages its tile's box in a
// private LDS region, already blended along the radius (the value
// (1-w) P_k + w P_{k+1} at each pixel, formed with the same float32 operations
// as the pair kernels' taps, so the entries are bitwise theirs), then forms the
// tile's 4 x 4 blocks and writes the four quarter turns as build_orbit_kernel
// does.  Sixteen waves per workgroup, 8.6 KiB of LDS each; no workgroup
// barrier (a wave orders its own LDS writes and reads).
constexpr int kFpSpan = 46;                     // box rows or columns, at most
constexpr int kFpStride = kFpSpan + 1;          // odd
constexpr int kFpRegion = kFpSpan * kFpStride;  // floats per wave

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// floor of the source row and column of image pixel (a, b) (tap_coords' steps)
template <typename G>
__device__ __forceinline__ void tap_origin(const G& g, double c, int a, int b, int& r0, int& c0) {
#pragma clang fp contract(off)
  const double ux = (double)b - c, uy = (double)a - c;
  const double ctux = g.ct * ux, mstux = (-g.st) * ux;
  const double stuy = g.st * uy, ctuy = g.ct * uy;
  const double colf = c + (ctux + stuy);
  const double rowf = c + (mstux + ctuy);
  c0 = (int)floor(colf);
  r0 = (int)floor(rowf);
}

// the same for the cubic builds (see build_cubic_orbit_kernel)
constexpr int kCbSpan = 48;                     // box rows or columns, at most
constexpr int kCbStride = kCbSpan + 1;          // odd
constexpr int kCbRegion = kCbSpan * kCbStride;  // floats per wave

// one element from the staged box (origin: bordered row Rlo, column Clo)
__device__ __forceinline__ float box_value(const float* __restrict__ Q, double ctux, double mstux,
                                           double stuy, double ctuy, double c, int n, int base) {
  constexpr int bs = kFpStride;
  const Tap t = tap_coords(ctux, mstux, stuy, ctuy, c, n, bs);
  const int i = t.ok ? t.idx - base : 0;
  const float q00 = Q[i], q01 = Q[i + 1];
  const float q10 = Q[i + bs], q11 = Q[i + bs + 1];
  float val = (t.gy * t.gx) * q00;
  val = fmaf(t.gy * t.fx, q01, val);
  val = fmaf(t.fy * t.gx, q10, val);
  val = fmaf(t.fy * t.fx, q11, val);
  return t.ok ? val : 0.0f;
}

// Stage rows [Rlo, Rlo + bh) x columns [Clo, Clo + bw) of a box into Q (row
// stride kFpStride, kCbStride), each entry the radial blend (1-w) x + w y of its
// pair, formed as the pair kernels form their taps.  Bilinear: bordered indices
// of the sample pair Pk, Pk1 (zero border); cubic: padded indices of the
// coefficient pairs Pc (zero outside the Np x Np array).  A row at a time, lane l
// its column l, 16 rows' loads in flight: the row's offset is a scalar, columns
// outside the array load from past the plane's buffer, which gives zero, so that
// an entry costs the blend and one LDS write.  (Taken 64 entries at a time, with
// an index and bounds for every entry, staging was a third of the kernel's vector
// instructions: 256^2 PSFs, 64^2 scene, float32, 320 us a build against 290 so.)
template <bool CUBIC>
__device__ __forceinline__ void stage_box(float* __restrict__ Q, const float* __restrict__ Pk,
                                          const float* __restrict__ Pk1,
                                          const float2* __restrict__ Pc, int n, int Np, int Rlo,
                                          int Clo, int bh, int bw, float wk0, float wk1, int lane) {
  constexpr int stride = CUBIC ? kCbStride : kFpStride;
  constexpr int kRows = 16, bytes = CUBIC ? 8 : 4;
  const int R0 = __builtin_amdgcn_readfirstlane(CUBIC ? Rlo : Rlo - 1);
  const int rows = __builtin_amdgcn_readfirstlane(bh);
  const int side = CUBIC ? Np : n;
  if (lane >= bw) return;
  const int C = (CUBIC ? Clo : Clo - 1) + lane;
  const uint32_t voff = (unsigned)C < (unsigned)side ? (uint32_t)C * bytes : 0x80000000u;
  const int plane = side * side * bytes;  // side <= 8216
  const __amdgpu_buffer_rsrc_t d0 =
      __builtin_amdgcn_make_buffer_rsrc(CUBIC ? (void*)Pc : (void*)Pk, (short)0, plane, 0x00020000);
  const __amdgpu_buffer_rsrc_t d1 =
      __builtin_amdgcn_make_buffer_rsrc((void*)(Pk1 ? Pk1 : Pk), (short)0, Pk1 ? plane : 0, 0x00020000);
  // rows of the array: [top, end) of the box
  const int top = R0 < 0 ? (-R0 < rows ? -R0 : rows) : 0;
  const int end = side - R0 < rows ? (side - R0 > top ? side - R0 : top) : rows;
  for (int r = 0; r < top; ++r) Q[r * stride + lane] = 0.0f;
  for (int r = end; r < rows; ++r) Q[r * stride + lane] = 0.0f;
  for (int r = top; r < end; r += kRows) {
    float xv[kRows], yv[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int R = R0 + (r + k < end ? r + k : end - 1);  // past the end: the last row again
      const int soff = R * side * bytes;
      if constexpr (CUBIC) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(d0, voff, soff, 0));
        xv[k] = v.x;
        yv[k] = v.y;
      } else {
        xv[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(d0, voff, soff, 0));
        yv[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(d1, voff, soff, 0));
      }
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k)
      if (r + k < end) Q[(r + k) * stride + lane] = fmaf(wk1, yv[k], wk0 * xv[k]);
  }
}

// The waves of the launch walk the (base, tile) pairs independently, tiles of
// one base on neighbouring waves.  Nothing is shared between them; the bases
// are taken in bracket order so that the pairs being read at one time stay in
// the L2 (256^2: 3.7 ms, in natural order 4.6 ms).
// The workgroup's share of the runs, a contiguous range; round i takes the next
// 16, the waves moved on by 5 a round so that none keeps to one place of the
// image (tiles at its corners are cheap).
__device__ __forceinline__ uint32_t box_run(uint32_t i, int wave, uint32_t rounds) {
  return (blockIdx.x * rounds + i) * 16 + (((uint32_t)wave + 5 * i) & 15);
}

template <bool VEC, int MODE>
__global__ __launch_bounds__(1024) void build_orbit_box_kernel(const float* __restrict__ cube, int K,
                                                               const ColGeom* __restrict__ geo,
                                                               const int32_t* __restrict__ reps,
                                                               OrbitGrid o, int n, int64_t M, int nt, int run, uint32_t total,
                                                               float* __restrict__ A,
                                                               double* __restrict__ part,
                                                               const float* __restrict__ colscale) {
  extern __shared__ float QS[];  // 16 regions of kFpRegion floats
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* Q = QS + wave * kFpRegion;
  const double c = (double)(n - 1) * 0.5;
  const int ntiles = nt * nt;
  const int nruns = (ntiles + run - 1) / run;
  const uint32_t rounds = (total + 16 * gridDim.x - 1) / (16 * gridDim.x);
  for (uint32_t i = 0; i < rounds; ++i) {  // no workgroup barrier
    const uint32_t t = box_run(i, wave, rounds);
    if (t >= total) continue;
    const uint32_t sp = t / (uint32_t)nruns;
    const int r = (int)(t - sp * (uint32_t)nruns);
    const OrbitCol g = load_orbit_col<MODE>(reps, geo, colscale, sp);
    double tsum = 0.0;
    for (int tile = r * run; tile < min((r + 1) * run, ntiles); ++tile) {
      const int a0 = 32 * (tile / nt), b0 = 32 * (tile % nt);
      if (g.k < 0) {  // identically zero orbit
        orbit_tile<VEC, MODE>([](double, double, double, double) { return 0.0f; }, g, c, n, o.N, M, a0, b0,
                              lane, A, tsum);
        continue;
      }
      const float* Pk = cube + (int64_t)g.k * M;
      const float* Pk1 = (K > 1) ? Pk + M : nullptr;
      const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
      // the tile's pixels (from the first row and column that its blocks reach)
      // and their box of bordered rows [Rlo, Rlo + bh) and columns [Clo, Clo + bw)
      const int at = base_only(MODE) ? a0 : block_start<VEC>(a0, n), bt = base_only(MODE) ? b0 : block_start<VEC>(b0, n);
      const int ae = (a0 + 32 < n) ? a0 + 32 : n, be = (b0 + 32 < n) ? b0 + 32 : n;
      int rmin, rmax, cmin, cmax;
      {
        int r0, c0;
        tap_origin(g, c, at, bt, r0, c0);
        rmin = rmax = r0;
        cmin = cmax = c0;
#pragma unroll
        for (int k = 1; k < 4; ++k) {
          tap_origin(g, c, (k & 1) ? ae - 1 : at, (k & 2) ? be - 1 : bt, r0, c0);
          rmin = min(rmin, r0);
          rmax = max(rmax, r0);
          cmin = min(cmin, c0);
          cmax = max(cmax, c0);
        }
      }
      const int Rlo = max(rmin + 1, 0), Clo = max(cmin + 1, 0);
      const int bh = min(max(min(rmax + 2, n + 1) - Rlo + 1, 0), kFpSpan);
      const int bw = min(max(min(cmax + 2, n + 1) - Clo + 1, 0), kFpSpan);
      wave_lds_sync();  // the previous tile's reads are done
      stage_box<false>(Q, Pk, Pk1, nullptr, n, 0, Rlo, Clo, bh, bw, wk0, wk1, lane);
      wave_lds_sync();  // the box is staged
      const int base = Rlo * kFpStride + Clo;
      orbit_tile<VEC, MODE>(
            [&](double ctux, double mstux, double stuy, double ctuy) {
              return box_value(Q, ctux, mstux, stuy, ctuy, c, n, base);
            },
            g, c, n, o.N, M, a0, b0, lane, A, tsum);
    }
    tsum = wave_sum_f64(tsum);
    if (lane == 0) part[(int64_t)r * o.nreps + sp] = tsum;
  }
}

// 16-bit rounding of a column's value, scaled by 2^-e (exact)
template <bool BF16>
__device__ __forceinline__ uint16_t round16(float val, int e) {
  const float xs = ldexpf(val, -e);
  if constexpr (BF16) {
    uint32_t w = __float_as_uint(xs);
    w += 0x7FFFu + ((w >> 16) & 1u);  // finite: round to nearest, ties to even
    return (uint16_t)(w >> 16);
  } else {
    return __builtin_bit_cast(uint16_t, (_Float16)xs);
  }
}

// 16-bit store of one unit.  Non-temporal where image rows start on 64 bytes
// (sides that are multiples of 4: 128^2 PSFs, 128^2 scene, 274 us a build against
// 280 with plain stores; 180^2, 90^2 scene, 350 against 365).  On other sides
// every row ends inside a 128-byte line whose rest a neighbouring tile writes
// later: plain stores let the two meet in the L2 (101^2, 128^2 scene: 236 us
// against 272; 181^2, 90^2 scene: 383 against 424).
template <bool LINES>
__device__ __forceinline__ void store_unit(uint16_t* p, const u32x4 w) {
  if constexpr (LINES)
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
  else
    *reinterpret_cast<u32x4*>(p) = w;
}

// 16-bit orbit build.  A window of 16 bases is two blocks; block h's member k is group
// 4 (w0/8 + h) + k, whose unit at an image pixel holds the 8 bases' member
// values there.  The item's rows are walked in tiles of 8 x 32 pixels: every
// wave forms its base column's tile (lane (i, k): row i, columns k + 8 q),
// rounds the values into an LDS tile [2][8][33][8] (unit-major: the 8 bases of
// a block and pixel are one 16-byte LDS word; one unit of padding per row
// keeps the column-wise reads conflict-free), and after one barrier half the
// threads copy the tile's units along rows to members 0 and 2 (runs of 32
// units in rows a and n-1-a) and half along columns to members 1 and 3 (runs
// of 8 units, one 128-byte line, in rows b and n-1-b).  The LDS tile is
// double-buffered, so that one barrier per tile suffices: a tile's buffer is
// written again two tiles later, after every thread has passed the barrier
// behind the copy that read it.  Slots of a block outside the item (the block
// straddles two brackets) are left to the other item: 2-byte stores.  Positions
// past the last base, up to a whole block, are written as zeros with it.
template <bool BF16, bool SCALED, bool LINES>
__global__ __launch_bounds__(1024) void build_orbit16_kernel(const float* __restrict__ cube, int K,
                                                             const ColGeom* __restrict__ geo,
                                                             const int32_t* __restrict__ reps,
                                                             const int4* __restrict__ items,
                                                             const int32_t* __restrict__ nitems,
                                                             int nb, int n, int ls, int64_t M,
                                                             int rpr, int64_t nreps,
                                                             uint16_t* __restrict__ Mh,
                                                             double* __restrict__ part,
                                                             const float* __restrict__ colscale) {
  constexpr int TA = 8, TB = 32, TP = TB + 1;
  constexpr int TILE = 2 * TA * TP * 8;  // uint16 per buffer
  extern __shared__ float2 P2[];  // bordered pair, then the two tile buffers
  if ((int)blockIdx.x >= *nitems) return;  // uniform: surplus workgroups of the upper bound
  const int4 it = items[blockIdx.x];
  const int bkt = it.x, first = it.y, len = it.z, w0 = it.w;
  const bool zero_bucket = bkt == nb - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ra = (int)blockIdx.y * rpr, rb = (ra + rpr < n) ? ra + rpr : n;
  uint16_t* tiles = reinterpret_cast<uint16_t*>(P2 + ((((size_t)(n + 2) * ls) + 1) & ~(size_t)1));
  if (!zero_bucket) stage_pair(P2, cube, bkt, K, n, ls, M, tid);
  const int sp = w0 + wave;
  // the item's positions, the last one with those that fill up its block
  const int end = first + len == nreps ? (first + len + 7) / 8 * 8 : first + len;
  const bool live = sp >= first && sp < end;  // uniform per wave
  const bool base = live && sp < nreps;
  const bool blank = zero_bucket || !base;
  const int h = wave >> 3, u = wave & 7;
  ColGeom g;
  g.ct = 1.0; g.st = 0.0; g.w = 0.0; g.e = 0;
  if (base) g = geo[reps[sp]];
  const float sf = (SCALED && base) ? colscale[reps[sp]] : 1.0f;  // flux-preserving scale
  const double c = (double)(n - 1) * 0.5;
  const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
  const int64_t G0 = (int64_t)(w0 / 8) * 4;
  int lo[2], hi[2];  // the item's slots of each block, relative to the block
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int s0 = w0 + 8 * q;
    lo[q] = (first > s0) ? first - s0 : 0;
    hi[q] = (end < s0 + 8) ? end - s0 : 8;
  }
  const int li = lane >> 3, lk = lane & 7;
  // copy roles: threads 0..511 along rows, 512..1023 along columns
  const bool along_cols = tid >= 512;
  const int cq = (tid & 511) >> 8, crem = tid & 255;
  double tsum = 0.0;
  __syncthreads();  // the pair is staged
  int buf = 0;
  for (int a0 = ra; a0 < rb; a0 += TA) {
    for (int b0 = 0; b0 < n; b0 += TB, buf ^= 1) {
      uint16_t* tile = tiles + buf * TILE;
      if (live) {
        const int a = a0 + li;
        if (a < rb) {
          double stuy, ctuy;
          {
#pragma clang fp contract(off)
            const double uy = (double)a - c;
            stuy = g.st * uy;
            ctuy = g.ct * uy;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (b0 + 8 * q >= n) break;  // uniform
            const int b = b0 + lk + 8 * q;
            if (b >= n) continue;
            double ctux, mstux;
            {
#pragma clang fp contract(off)
              const double ux = (double)b - c;
              ctux = g.ct * ux;
              mstux = (-g.st) * ux;
            }
            float val = blank ? 0.0f
                              : orbit_value(P2, ctux, mstux, stuy, ctuy, c, n, ls, wk0, wk1);
            if constexpr (SCALED) val *= sf;
            tsum += (double)val;
            tile[((h * TA + li) * TP + lk + 8 * q) * 8 + u] = round16<BF16>(val, g.e);
          }
        }
      }
      __syncthreads();
      // one unit per thread: block cq, 8 rows x 32 columns
      if (lo[cq] < hi[cq]) {
        int r, cb;
        if (along_cols) {
          cb = crem >> 3;
          r = crem & 7;
        } else {
          r = crem >> 5;
          cb = crem & 31;
        }
        const int a = a0 + r, b = b0 + cb;
        if (a < rb && b < n) {
          const uint16_t* src = tile + ((cq * TA + r) * TP + cb) * 8;
          uint16_t* dA;
          uint16_t* dB;
          if (along_cols) {
            dA = Mh + ((G0 + 4 * cq + 1) * M + (int64_t)b * n + (n - 1 - a)) * 8;
            dB = Mh + ((G0 + 4 * cq + 3) * M + (int64_t)(n - 1 - b) * n + a) * 8;
          } else {
            dA = Mh + ((G0 + 4 * cq + 0) * M + (int64_t)a * n + b) * 8;
            dB = Mh + ((G0 + 4 * cq + 2) * M + (int64_t)(n - 1 - a) * n + (n - 1 - b)) * 8;
          }
          if (lo[cq] == 0 && hi[cq] == 8) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(src);
            store_unit<LINES>(dA, w);
            store_unit<LINES>(dB, w);
          } else {
            for (int s = lo[cq]; s < hi[cq]; ++s) {
              dA[s] = src[s];
              dB[s] = src[s];
            }
          }
        }
      }
    }
  }
  if (!base) return;
  tsum = wave_sum_f64(tsum);
  if (lane == 0) part[(int64_t)blockIdx.y * nreps + sp] = tsum;
}

// Cubic-spline orbit build: the quarter-turn orbits of the bilinear builds
// (the four members of an orbit sample the spline at the same source points,
// so one base column is computed and four are written), each 32 x 32 pixel
// tile reading its 4 x 4 B-spline taps from a box of the padded coefficient
// pair that the wave stages in its own LDS region.  A pixel's tap origin is
// clamped to padded indices [-3, Np+1] (where that moves it, all its taps lay
// outside the padded array and read zeros, as before the clamp); the clamp and
// the floors are monotone, so the tile's extreme origins are those of its
// corners and the box spans at most 44 + 4 = 48 rows and columns.  The box
// holds the radial blend (1-w) C_k + w C_{k+1} (zero outside the array), and a
// pixel is the 4 x 4 weighted sum of the blend, row by row, in the order of
// the gather form, so both give identical values.
__device__ __forceinline__ int clamp_origin(int v, int Np) { return v < -3 ? -3 : (v > Np + 1 ? Np + 1 : v); }

// clamped tap origin (padded row and column) of image pixel (a, b)
template <typename G>
__device__ __forceinline__ void cubic_origin(const G& g, double c, int a, int b, int Np,
                                             int& r0, int& c0) {
#pragma clang fp contract(off)
  const double ux = (double)b - c, uy = (double)a - c;
  const double pad = (double)kSplinePad;
  const double rowf = c + ((-g.st) * ux + g.ct * uy) + pad;
  const double colf = c + (g.ct * ux + g.st * uy) + pad;
  r0 = clamp_origin((int)floor(rowf), Np);
  c0 = clamp_origin((int)floor(colf), Np);
}

template <bool VEC, int MODE>
__global__ __launch_bounds__(1024) void build_cubic_orbit_kernel(const float2* __restrict__ pairs,
                                                                 int Np,
                                                                 const ColGeom* __restrict__ geo,
                                                                 const int32_t* __restrict__ reps,
                                                                 OrbitGrid o, int n, int64_t M, int nt, int run, uint32_t total,
                                                                 float* __restrict__ A,
                                                                 double* __restrict__ part,
                                                                 const float* __restrict__ colscale) {
  extern __shared__ float QS[];  // 16 regions of kCbRegion floats
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* Q = QS + wave * kCbRegion;
  const double c = (double)(n - 1) * 0.5;
  const double pad = (double)kSplinePad;
  const int ntiles = nt * nt;
  const int nruns = (ntiles + run - 1) / run;
  const uint32_t rounds = (total + 16 * gridDim.x - 1) / (16 * gridDim.x);
  for (uint32_t i = 0; i < rounds; ++i) {  // no workgroup barrier
    const uint32_t t = box_run(i, wave, rounds);
    if (t >= total) continue;
    const uint32_t sp = t / (uint32_t)nruns;
    const int r = (int)(t - sp * (uint32_t)nruns);
    const OrbitCol g = load_orbit_col<MODE>(reps, geo, colscale, sp);
    double tsum = 0.0;
    for (int tile = r * run; tile < min((r + 1) * run, ntiles); ++tile) {
      const int a0 = 32 * (tile / nt), b0 = 32 * (tile % nt);
      if (g.k < 0) {  // identically zero orbit
        orbit_tile<VEC, MODE>([](double, double, double, double) { return 0.0f; }, g, c, n, o.N, M, a0, b0,
                              lane, A, tsum);
        continue;
      }
      const float2* src = pairs + (int64_t)g.k * Np * Np;
      const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
      // the tile's pixels (from the first row and column that its blocks reach)
      // and their box of padded rows [Rlo, Rlo + bh) and columns [Clo, Clo + bw)
      const int at = base_only(MODE) ? a0 : block_start<VEC>(a0, n), bt = base_only(MODE) ? b0 : block_start<VEC>(b0, n);
      const int ae = (a0 + 32 < n) ? a0 + 32 : n, be = (b0 + 32 < n) ? b0 + 32 : n;
      int rmin, rmax, cmin, cmax;
      {
        int r0, c0;
        cubic_origin(g, c, at, bt, Np, r0, c0);
        rmin = rmax = r0;
        cmin = cmax = c0;
#pragma unroll
        for (int k = 1; k < 4; ++k) {
          cubic_origin(g, c, (k & 1) ? ae - 1 : at, (k & 2) ? be - 1 : bt, Np, r0, c0);
          rmin = min(rmin, r0);
          rmax = max(rmax, r0);
          cmin = min(cmin, c0);
          cmax = max(cmax, c0);
        }
      }
      const int Rlo = rmin - 1, Clo = cmin - 1;
      const int bh = min(rmax - rmin + 4, kCbSpan), bw = min(cmax - cmin + 4, kCbSpan);
      wave_lds_sync();  // the previous tile's reads are done
      stage_box<true>(Q, nullptr, nullptr, src, n, Np, Rlo, Clo, bh, bw, wk0, wk1, lane);
      wave_lds_sync();  // the box is staged
      orbit_tile<VEC, MODE>(
            [&](double ctux, double mstux, double stuy, double ctuy) {
#pragma clang fp contract(off)
              const double rowf = c + (mstux + ctuy) + pad;
              const double colf = c + (ctux + stuy) + pad;
              const double r0f = floor(rowf), c0f = floor(colf);
              const int r0 = clamp_origin((int)r0f, Np), c0 = clamp_origin((int)c0f, Np);
              float wy[4], wx[4];
              cubic_weights(rowf - r0f, wy);
              cubic_weights(colf - c0f, wx);
              const float* tp = Q + (r0 - 1 - Rlo) * kCbStride + (c0 - 1 - Clo);
              float V = 0.0f;
#pragma unroll
              for (int dr = 0; dr < 4; ++dr) {
                const float* tr = tp + dr * kCbStride;
                float v = wx[0] * tr[0];
                v = fmaf(wx[1], tr[1], v);
                v = fmaf(wx[2], tr[2], v);
                v = fmaf(wx[3], tr[3], v);
                V = fmaf(wy[dr], v, V);
              }
              return V;
            },
            g, c, n, o.N, M, a0, b0, lane, A, tsum);
    }
    tsum = wave_sum_f64(tsum);
    if (lane == 0) part[(int64_t)r * o.nreps + sp] = tsum;
  }
}

// Copy a tile of TA x 32 units of a whole window to its members: threads 0..511
// along rows, 512..1023 along columns; unit cu of a direction is block cu / (32
// TA), row and column from cu % (32 TA).  Rows end at `ae`; block cq is there when
// 8 cq < left.
template <int TA, bool LINES>
__device__ __forceinline__ void copy_units(const uint16_t* tile, uint16_t* __restrict__ Mh, int64_t G0,
                                           int64_t M, int n, int a1, int ae, int b0, int64_t left, int tid) {
  constexpr int TB = 32, TP = TB + 1;
  const bool along_cols = tid >= 512;
  const int cu = tid & 511, cq = cu / (TA * TB), crem = cu % (TA * TB);
  if (cq >= 2 || 8 * cq >= left) return;
  int r, cb;
  if (along_cols) {
    cb = crem / TA;
    r = crem % TA;
  } else {
    r = crem >> 5;
    cb = crem & 31;
  }
  const int a = a1 + r, b = b0 + cb;
  if (a >= ae || b >= n) return;
  uint16_t* dA;
  uint16_t* dB;
  if (along_cols) {
    dA = Mh + ((G0 + 4 * cq + 1) * M + (int64_t)b * n + (n - 1 - a)) * 8;
    dB = Mh + ((G0 + 4 * cq + 3) * M + (int64_t)(n - 1 - b) * n + a) * 8;
  } else {
    dA = Mh + ((G0 + 4 * cq + 0) * M + (int64_t)a * n + b) * 8;
    dB = Mh + ((G0 + 4 * cq + 2) * M + (int64_t)(n - 1 - a) * n + (n - 1 - b)) * 8;
  }
  const u32x4 w = *reinterpret_cast<const u32x4*>(tile + ((cq * TA + r) * TP + cb) * 8);
  store_unit<LINES>(dA, w);
  store_unit<LINES>(dB, w);
}

// The second pass of a 16-bit flux-preserving build from the base columns that
// the first pass kept (S[position][pixel], float32): a window of 16 bases and a
// range of rows a workgroup, as the 16-bit orbit builds, the values loaded
// instead of formed, the next tile's in flight while a tile is copied.  Bound by
// memory: half the library's bytes read, all of them written.  Forming the values
// again took 202 us for 101^2 PSFs of a 101^2 scene with the spline, this 80.
template <bool BF16, bool LINES>
__global__ __launch_bounds__(1024) void spread_orbit16_kernel(const float* __restrict__ S,
                                                              const ColGeom* __restrict__ geo,
                                                              const int32_t* __restrict__ reps, int n,
                                                              int64_t M, int rpr, int64_t nreps,
                                                              uint16_t* __restrict__ Mh,
                                                              double* __restrict__ part,
                                                              const float* __restrict__ colscale) {
  constexpr int TA = 8, TB = 32, TP = TB + 1;
  constexpr int TILE = 2 * TA * TP * 8;
  __shared__ __attribute__((aligned(16))) uint16_t tiles[2 * TILE];
  const int64_t w0 = (int64_t)blockIdx.x * 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ra = (int)blockIdx.y * rpr, rb = (ra + rpr < n) ? ra + rpr : n;
  const int64_t sp = w0 + wave;
  const int64_t whole = (nreps + 7) / 8 * 8;
  const int h = wave >> 3, u = wave & 7;
  const int li = lane >> 3, lk = lane & 7;
  const bool base = sp < nreps;
  int e = 0;
  float sf = 1.0f;
  if (base) {
    e = geo[reps[sp]].e;
    sf = colscale[reps[sp]];
  }
  const float* src = S + (base ? sp : 0) * M;
  // four values of row a from column b, zeros outside the range or the image
  auto load = [&](int a, int b) -> f32x4 {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!base || a >= rb || b >= n) return v;
    const float* p = src + (int64_t)a * n + b;
    if (b + 4 <= n) return *reinterpret_cast<const f32x4u*>(p);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (b + q < n) v[q] = p[q];
    return v;
  };
  double tsum = 0.0;
  int buf = 0;
  const int64_t G0 = w0 / 8 * 4;
  f32x4 next = load(ra + li, 4 * lk);
  for (int a1 = ra; a1 < rb; a1 += TA) {
    for (int b0 = 0; b0 < n; b0 += TB, buf ^= 1) {  // uniform over the workgroup
      uint16_t* tile = tiles + buf * TILE;
      const f32x4 v = next;
      const bool wrap = b0 + TB >= n;
      next = load(a1 + (wrap ? TA : 0) + li, (wrap ? 0 : b0 + TB) + 4 * lk);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float val = v[q] * sf;
        tsum += (double)val;
        tile[((h * TA + li) * TP + 4 * lk + q) * 8 + u] = round16<BF16>(val, e);
      }
      __syncthreads();  // two buffers: see build_orbit16_kernel
      copy_units<TA, LINES>(tile, Mh, G0, M, n, a1, rb, b0, whole - w0, tid);
    }
  }
  if (!base) return;
  tsum = wave_sum_f64(tsum);
  if (lane == 0) part[(int64_t)blockIdx.y * nreps + sp] = tsum;
}

// 16-bit orbit build for pairs that do not fit the LDS beside the unit tiles
// (n > 131), bilinear or cubic-spline: build_orbit16_kernel's unit tiles and copies,
// with each wave's taps read from a staged box (as build_orbit_box_kernel and
// build_cubic_orbit_kernel) of the 32 x 32 pixels it forms as 32 / TA tiles of
// TA x 32.  LDS: 16 box regions, then the two unit tiles; the cubic boxes are
// larger (48 x 49 floats), so the cubic form takes 4-row tiles (each lane two
// pixels of a tile row) where the bilinear form takes 8-row ones (four).  Every
// wave reads its own bracket's pair, so a workgroup takes a whole window of 16
// bases whatever their brackets, and every store is a whole unit.
template <bool BF16, bool CUBIC, bool SCALED, bool LINES>
__global__ __launch_bounds__(1024) void build_orbit16_box_kernel(const float* __restrict__ src0, int K,
                                                                 const ColGeom* __restrict__ geo,
                                                                 const int32_t* __restrict__ reps,
                                                                 int n, int64_t M, int Np,
                                                                 int rpr, int64_t nreps,
                                                                 uint16_t* __restrict__ Mh,
                                                                 double* __restrict__ part,
                                                                 const float* __restrict__ colscale) {
  constexpr int TA = CUBIC ? 4 : 8, TB = 32, TP = TB + 1;
  constexpr int CPL = (TA * TB) / 64;      // pixels of a tile row per lane
  constexpr int LPR = TB / CPL;            // lanes per tile row
  constexpr int TILE = 2 * TA * TP * 8;    // uint16 per buffer
  constexpr int REGION = CUBIC ? kCbRegion : kFpRegion;
  extern __shared__ float QS[];
  const int64_t w0 = (int64_t)blockIdx.x * 16;  // the window's first base position
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ra = (int)blockIdx.y * rpr, rb = (ra + rpr < n) ? ra + rpr : n;
  uint16_t* tiles = reinterpret_cast<uint16_t*>(QS + 16 * REGION);
  float* Q = QS + wave * REGION;
  const int64_t sp = w0 + wave;
  const int64_t whole = (nreps + 7) / 8 * 8;  // with the positions that fill up the last block
  const bool live = sp < whole;  // uniform per wave
  const int h = wave >> 3, u = wave & 7;
  ColGeom g;
  g.ct = 1.0; g.st = 0.0; g.w = 0.0; g.e = 0; g.k = -1;
  if (sp < nreps) g = geo[reps[sp]];
  const bool blank = g.k < 0;  // an identically zero orbit, or no base
  const float sf = (SCALED && sp < nreps) ? colscale[reps[sp]] : 1.0f;  // flux-preserving scale
  const double c = (double)(n - 1) * 0.5;
  const double pad = (double)kSplinePad;
  const float wk0 = (float)(1.0 - g.w), wk1 = (float)g.w;
  const int pb = blank ? 0 : g.k;
  const float* Pk = CUBIC ? src0 : src0 + (int64_t)pb * M;  // bilinear: the sample pair
  const float* Pk1 = (!CUBIC && K > 1) ? Pk + M : nullptr;
  const float2* Pc = reinterpret_cast<const float2*>(src0) + (CUBIC ? (int64_t)pb * Np * Np : 0);  // cubic
  const int64_t G0 = w0 / 8 * 4;
  const int li = lane / LPR, lk = lane % LPR;
  double tsum = 0.0;
  int buf = 0;
  for (int a0 = ra; a0 < rb; a0 += 32) {
    const int ae = (a0 + 32 < rb) ? a0 + 32 : rb;
    for (int b0 = 0; b0 < n; b0 += TB) {
      const int be = (b0 + TB < n) ? b0 + TB : n;
      int base = 0, Rlo = 0, Clo = 0;
      if (!blank) {  // uniform per wave: stage the box of rows [a0, ae), columns [b0, be)
        int rmin, rmax, cmin, cmax;
        {
          int r0, c0;
          if constexpr (CUBIC) cubic_origin(g, c, a0, b0, Np, r0, c0);
          else tap_origin(g, c, a0, b0, r0, c0);
          rmin = rmax = r0;
          cmin = cmax = c0;
#pragma unroll
          for (int k = 1; k < 4; ++k) {
            if constexpr (CUBIC)
              cubic_origin(g, c, (k & 1) ? ae - 1 : a0, (k & 2) ? be - 1 : b0, Np, r0, c0);
            else
              tap_origin(g, c, (k & 1) ? ae - 1 : a0, (k & 2) ? be - 1 : b0, r0, c0);
            rmin = min(rmin, r0);
            rmax = max(rmax, r0);
            cmin = min(cmin, c0);
            cmax = max(cmax, c0);
          }
        }
        int bh, bw;
        if constexpr (CUBIC) {
          Rlo = rmin - 1;
          Clo = cmin - 1;
          bh = min(rmax - rmin + 4, kCbSpan);
          bw = min(cmax - cmin + 4, kCbSpan);
        } else {
          Rlo = max(rmin + 1, 0);
          Clo = max(cmin + 1, 0);
          bh = min(max(min(rmax + 2, n + 1) - Rlo + 1, 0), kFpSpan);
          bw = min(max(min(cmax + 2, n + 1) - Clo + 1, 0), kFpSpan);
        }
        base = Rlo * kFpStride + Clo;
        stage_box<CUBIC>(Q, Pk, Pk1, Pc, n, Np, Rlo, Clo, bh, bw, wk0, wk1, lane);
        wave_lds_sync();  // the box is staged
      }
      for (int a1 = a0; a1 < ae; a1 += TA, buf ^= 1) {  // uniform over the workgroup
        uint16_t* tile = tiles + buf * TILE;
        if (live) {
          const int a = a1 + li;
          if (a < ae) {
            double stuy, ctuy;
            {
#pragma clang fp contract(off)
              const double uy = (double)a - c;
              stuy = g.st * uy;
              ctuy = g.ct * uy;
            }
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
              if (b0 + LPR * q >= n) break;  // uniform
              const int b = b0 + lk + LPR * q;
              if (b >= n) continue;
              double ctux, mstux;
              {
#pragma clang fp contract(off)
                const double ux = (double)b - c;
                ctux = g.ct * ux;
                mstux = (-g.st) * ux;
              }
              float val = 0.0f;
              if (!blank) {
                if constexpr (CUBIC) {
#pragma clang fp contract(off)
                  const double rowf = c + (mstux + ctuy) + pad;
                  const double colf = c + (ctux + stuy) + pad;
                  const double r0f = floor(rowf), c0f = floor(colf);
                  const int r0 = clamp_origin((int)r0f, Np), c0 = clamp_origin((int)c0f, Np);
                  float wy[4], wx[4];
                  cubic_weights(rowf - r0f, wy);
                  cubic_weights(colf - c0f, wx);
                  const float* t = Q + (r0 - 1 - Rlo) * kCbStride + (c0 - 1 - Clo);
#pragma unroll
                  for (int dr = 0; dr < 4; ++dr) {
                    const float* tr = t + dr * kCbStride;
                    float v = wx[0] * tr[0];
                    v = fmaf(wx[1], tr[1], v);
                    v = fmaf(wx[2], tr[2], v);
                    v = fmaf(wx[3], tr[3], v);
                    val = fmaf(wy[dr], v, val);
                  }
                } else {
                  val = box_value(Q, ctux, mstux, stuy, ctuy, c, n, base);
                }
              }
              if constexpr (SCALED) val *= sf;
              tsum += (double)val;
              tile[((h * TA + li) * TP + lk + LPR * q) * 8 + u] = round16<BF16>(val, g.e);
            }
          }
        }
        __syncthreads();
        copy_units<TA, LINES>(tile, Mh, G0, M, n, a1, ae, b0, whole - w0, tid);
      }
    }
  }
  if (sp >= nreps) return;
  tsum = wave_sum_f64(tsum);
  if (lane == 0) part[(int64_t)blockIdx.y * nreps + sp] = tsum;
}

// ------------------------------------------------------------- launch -----
static int lds_e(int n) { return (n + 63) / 64; }

// LDS row stride (in pairs) of the bordered array: n+2 rounded up to 5 mod 8
// when that still fits.  The taps of a wave follow a rotated line through the
// array; with an even stride, near-vertical lines put lanes two rows apart on
// the same banks, an odd stride spreads them (about 13% fewer LDS cycles over
// random angles at n = 128 in a bank model).
static int lds_stride(int n) {
  const int np = n + 2, ls = np + ((5 - np % 8) + 8) % 8;
  return (size_t)np * ls * sizeof(float2) <= (size_t)kLdsBuildMaxBytes ? ls : np;
}

static bool pair_fits_lds(int n) {
  return (size_t)(n + 2) * (n + 2) * sizeof(float2) <= (size_t)kLdsBuildMaxBytes;
}

bool build_lds_supported(int n, int K, int N) {
  // the bordered pair fits the LDS whole, or the orbit builds stage a box of it per
  // tile (sides are at most 8192: pixel offsets stay in int); the bucket histograms (8
  // B per bucket) must fit the sort kernels' LDS
  if (K > 8192) return false;
  return pair_fits_lds(n) || build_orbit_supported(K, N);
}

static int nbuckets(int K) { return ((K > 1) ? K - 1 : 1) + 1; }

size_t bucket_scratch_bytes(int K, int64_t ncols) {
  const int64_t nb = nbuckets(K);
  const int64_t items_max = (ncols + kLdsCols - 1) / kLdsCols + nb;
  size_t b = 0;
  b += ((size_t)nb * 4 * 3 + 255) & ~(size_t)255;           // cnt, cursor, bstart
  b += ((size_t)items_max * 16 + 16 + 255) & ~(size_t)255;  // items + nitems
  b += ((size_t)ncols * 4 + 255) & ~(size_t)255;            // order
  return b;
}

hipError_t launch_bucket_sort(const ColGeom* geo, int64_t ncols, int K, void* scratch,
                              BucketPlan* plan, hipStream_t s) {
  const int nb = nbuckets(K);
  const int64_t items_max = (ncols + kLdsCols - 1) / kLdsCols + nb;
  char* p = reinterpret_cast<char*>(scratch);
  int32_t* cnt = reinterpret_cast<int32_t*>(p);
  int32_t* cursor = cnt + nb;
  int32_t* bstart = cursor + nb;
  p += ((size_t)nb * 4 * 3 + 255) & ~(size_t)255;
  int4* items = reinterpret_cast<int4*>(p);
  int32_t* nitems = reinterpret_cast<int32_t*>(items + items_max);
  p += ((size_t)items_max * 16 + 16 + 255) & ~(size_t)255;
  int32_t* order = reinterpret_cast<int32_t*>(p);
  // cnt and cursor start at zero (a fill kernel, not hipMemsetAsync, so a
  // captured build replays correctly)
  zero_ints_kernel<<<(unsigned)((2 * nb + 255) / 256), 256, 0, s>>>(cnt, 2 * nb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned cgrid = (unsigned)((ncols + 255) / 256);
  bucket_count_kernel<<<cgrid, 256, (size_t)nb * 4, s>>>(geo, ncols, nb, cnt);
  bucket_scan_kernel<<<1, 1024, 0, s>>>(cnt, nb, bstart, items, nitems);
  bucket_scatter_kernel<<<cgrid, 256, (size_t)nb * 8, s>>>(geo, ncols, nb, bstart, cursor, order);
  plan->order = order;
  plan->items = items;
  plan->nitems = nitems;
  plan->items_max = items_max;
  plan->nb = nb;
  return hipGetLastError();
}

hipError_t launch_pack16(int storage, const float* A32, const ColGeom* geo, int64_t M,
                         int64_t ncols, int64_t ncols_pad, void* lib, hipStream_t s) {
  const dim3 pgrid((unsigned)((M + 511) / 512), (unsigned)(ncols_pad / 8));
  u32x4* Mp = reinterpret_cast<u32x4*>(lib);
  if (storage == PSFLIB_BF16_POW2)
    pack16_kernel<true><<<pgrid, 256, 0, s>>>(A32, geo, M, ncols, Mp);
  else
    pack16_kernel<false><<<pgrid, 256, 0, s>>>(A32, geo, M, ncols, Mp);
  return hipGetLastError();
}

hipError_t launch_build_lds(const float* cube, int K, ColGeom* geo, int n, int N, int64_t M,
                            float* A32, double* tau, void* scratch, hipStream_t s) {
  if (build_orbit_supported(K, N))
    return launch_build_orbit(cube, K, geo, n, N, M, A32, tau, scratch, kPlain, nullptr, s);
  if (!pair_fits_lds(n)) return hipErrorInvalidValue;  // larger pairs: the orbit builds only
  const int64_t ncols = (int64_t)N * N;
  BucketPlan bp;
  hipError_t e = launch_bucket_sort(geo, ncols, K, scratch, &bp, s);
  if (e != hipSuccess) return e;
  const int32_t* order = bp.order;
  const int4* items = bp.items;
  const int32_t* nitems = bp.nitems;
  const int nb = bp.nb;
  const int64_t items_max = bp.items_max;

  const unsigned grid = (unsigned)items_max;
  const bool full = (n % 64) == 0;
  const int ls = lds_stride(n);
  const size_t lds = (size_t)(n + 2) * ls * sizeof(float2);
  const void* fn;
  auto launch = [&](auto kern) -> hipError_t {
    fn = reinterpret_cast<const void*>(kern);
    hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    kern<<<grid, 1024, lds, s>>>(cube, K, geo, order, items, nitems, nb, n, ls, M, A32, tau);
    return hipSuccess;
  };
  switch (lds_e(n)) {
    case 1: e = full ? launch(build_lds_kernel<1, true>) : launch(build_lds_kernel<1, false>); break;
    case 2: e = full ? launch(build_lds_kernel<2, true>) : launch(build_lds_kernel<2, false>); break;
    default: e = launch(build_lds_kernel<3, false>); break;
  }
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

// ------------------------------------------------- orbit launches -----
static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct OrbitPlan {
  OrbitGrid o;
  int nb, rpr, nranges, nt;  // 16-bit: row ranges; float32: tiles per side
  int64_t nblk, items_max;
  int32_t* cnt;
  int4* items;
  int32_t* nitems;  // items; the centre's position
  int32_t* reps;
  double* part;
};

static OrbitPlan orbit_plan(int K, int N, int n, void* scratch) {
  OrbitPlan pl;
  pl.o = orbit_grid(N);
  pl.nb = nbuckets(K);
  pl.rpr = orbit_rows_per_range(n);
  pl.nranges = (n + pl.rpr - 1) / pl.rpr;
  pl.nt = (n + 31) / 32;
  pl.nblk = (pl.o.nreps + kSortBlock - 1) / kSortBlock;
  pl.items_max = (pl.o.nreps + 15) / 16 + 2 * (int64_t)pl.nb + 1;
  char* p = reinterpret_cast<char*>(scratch);
  pl.cnt = reinterpret_cast<int32_t*>(p);
  p += al256((size_t)pl.nblk * pl.nb * 4);
  pl.items = reinterpret_cast<int4*>(p);
  pl.nitems = reinterpret_cast<int32_t*>(pl.items + pl.items_max);
  p += al256((size_t)pl.items_max * 16 + 16);
  pl.reps = reinterpret_cast<int32_t*>(p);
  p += al256((size_t)pl.o.nreps * 4);
  pl.part = reinterpret_cast<double*>(p);
  return pl;
}

size_t build_orbit_scratch_bytes(int K, int N, int n) {
  const OrbitPlan pl = orbit_plan(K, N, n, nullptr);
  return al256((size_t)pl.nblk * pl.nb * 4) + al256((size_t)pl.items_max * 16 + 16) +
         al256((size_t)pl.o.nreps * 4) + al256((size_t)pl.nt * pl.nt * pl.o.nreps * 8);
}

bool build_orbit_supported(int K, int N) {
  const OrbitGrid o = orbit_grid(N);
  const int64_t nblk = (o.nreps + kSortBlock - 1) / kSortBlock;
  return K <= kLdsMaxBuckets - 1 && nblk * nbuckets(K) <= ((int64_t)1 << 24) &&
         (int64_t)N * N < ((int64_t)1 << 31);
}

// Counting sort of the base columns by bracket, and the work items.  One
// workgroup does it while the waves' counts fit its LDS beside other work
// (kSmallSort base columns, scenes up to 128 x 128).
static hipError_t orbit_sort(const ColGeom* geo, const OrbitPlan& pl, hipStream_t s) {
  const size_t lds = (size_t)((pl.o.nreps + 63) / 64) * (size_t)pl.nb * 4;
  if (pl.o.nreps <= kSmallSort && pl.nb <= kSortBlock && lds <= 49152) {
    orbit_sort_kernel<<<1, kSortBlock, lds, s>>>(geo, pl.o, pl.nb, pl.reps, pl.items, pl.nitems);
    return hipGetLastError();
  }
  orbit_count_kernel<<<(unsigned)pl.nblk, kSortBlock, (size_t)pl.nb * 4, s>>>(geo, pl.o, pl.nb, pl.cnt);
  sort_scan_kernel<<<1, 1024, 0, s>>>(pl.cnt, pl.nblk, pl.nb, pl.items, pl.nitems);
  orbit_scatter_kernel<<<(unsigned)pl.nblk, kSortBlock, (size_t)pl.nb * 4, s>>>(
      geo, pl.o, pl.nb, pl.cnt, pl.reps, pl.nitems);
  return hipGetLastError();
}

// What follows the kernel that left the partial sums of a float32 build: the
// scales (first pass of a flux-preserving build) or the column sums.
static hipError_t orbit_finish(const OrbitPlan& pl, int nparts, int mode, int K, ColGeom* geo,
                               const OrbitFlux* fx, double* tau, hipStream_t s) {
  const unsigned grid = (unsigned)((pl.o.nreps + 255) / 256);
  if (mode == kSumsOnly || mode == kBases)
    orbit_scale_kernel<<<grid, 256, 0, s>>>(pl.reps, pl.o, pl.part, nparts, K, geo, *fx);
  else
    orbit_tau_kernel<<<grid, 256, 0, s>>>(pl.reps, pl.o, pl.part, nparts, tau);
  return hipGetLastError();
}

// runs are counted in 32 bits: 2^31 tiles are a library of 2^45 bytes
constexpr int64_t kMaxBoxRuns = (int64_t)1 << 31;

// Tiles that a wave takes at a time (a run): a row of tiles when that leaves
// every one of the 4096 resident waves 8 runs or more (the base's geometry is
// loaded once a run: 256^2 3% faster), else single tiles, which share the work
// out evenly (200^2 PSFs, 64^2 scene: 8% faster).
static int box_run_tiles(const OrbitPlan& pl) {
  return pl.o.nreps * pl.nt >= 8 * 4096 ? pl.nt : 1;
}

// Workgroups of the float32 box kernels: 16 independent waves each, one
// workgroup per CU at a time (its box regions fill the LDS), every workgroup
// walking a contiguous share of the runs.  4096 shares even out the CUs
// (200^2 PSFs, 64^2 scene: 0.35 ms against 0.42 ms with 1024; 256^2: 3.76
// against 3.96 ms), and the workgroups running at one time stay close in
// bracket order.
static unsigned box_grid(int64_t total) {
  const int64_t wgs = (total + 15) / 16;
  return (unsigned)(wgs < 4096 ? wgs : 4096);
}

hipError_t launch_build_orbit(const float* cube, int K, ColGeom* geo, int n, int N, int64_t M,
                              float* A32, double* tau, void* scratch, int mode,
                              const OrbitFlux* fx, hipStream_t s) {
  const OrbitPlan pl = orbit_plan(K, N, n, scratch);
  const float* colscale = fx ? fx->colscale : nullptr;
  if (mode == kSumsOnly && fx->bases) {
    mode = kBases;
    A32 = fx->bases;
  }
  hipError_t e = mode == kScaled ? hipSuccess : orbit_sort(geo, pl, s);  // kept for the second pass
  if (e != hipSuccess) return e;
  const bool vec = (n % 32) == 0;
  if (!pair_fits_lds(n)) {  // a staged box per 32 x 32 tile
    const int run = box_run_tiles(pl), nruns = (pl.nt * pl.nt + run - 1) / run;
    const int64_t total = pl.o.nreps * nruns;
    if (total >= kMaxBoxRuns) return hipErrorInvalidValue;
    const size_t lds = (size_t)16 * kFpRegion * sizeof(float);
    auto launch = [&](auto kern) -> hipError_t {
      const void* fn = reinterpret_cast<const void*>(kern);
      hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (err != hipSuccess) return err;
      kern<<<box_grid(total), 1024, lds, s>>>(cube, K, geo, pl.reps, pl.o, n, M, pl.nt, run, (uint32_t)total, A32, pl.part, colscale);
      return hipGetLastError();
    };
    switch (mode) {
      case kSumsOnly:
        e = launch(build_orbit_box_kernel<false, kSumsOnly>);
        break;
      case kScaled:
        e = vec ? launch(build_orbit_box_kernel<true, kScaled>) : launch(build_orbit_box_kernel<false, kScaled>);
        break;
      case kBases:
        e = launch(build_orbit_box_kernel<false, kBases>);
        break;
      default:
        e = vec ? launch(build_orbit_box_kernel<true, kPlain>) : launch(build_orbit_box_kernel<false, kPlain>);
    }
    if (e != hipSuccess) return e;
    return orbit_finish(pl, nruns, mode, K, geo, fx, tau, s);
  }
  const dim3 grid((unsigned)pl.items_max, (unsigned)(16 / orbit_sub(pl.nt)));
  const int ls = lds_stride(n);
  const size_t lds = (size_t)(n + 2) * ls * sizeof(float2);
  auto launch = [&](auto kern) -> hipError_t {
    const void* fn = reinterpret_cast<const void*>(kern);
    hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    kern<<<grid, 1024, lds, s>>>(cube, K, geo, pl.reps, pl.items, pl.nitems, pl.nb, n, ls, N, M,
                                 pl.nt, pl.o.nreps, A32, pl.part, colscale);
    return hipGetLastError();
  };
  switch (mode) {
    case kSumsOnly:
      e = launch(build_orbit_kernel<false, kSumsOnly>);
      break;
    case kScaled:
      e = vec ? launch(build_orbit_kernel<true, kScaled>) : launch(build_orbit_kernel<false, kScaled>);
      break;
    case kBases:
      e = launch(build_orbit_kernel<false, kBases>);
      break;
    default:
      e = vec ? launch(build_orbit_kernel<true, kPlain>) : launch(build_orbit_kernel<false, kPlain>);
  }
  if (e != hipSuccess) return e;
  return orbit_finish(pl, pl.nt * pl.nt, mode, K, geo, fx, tau, s);
}

// cubic-spline orbit build from staged boxes of the padded coefficient pairs
hipError_t launch_build_cubic_orbit(const float* pairs, int K, ColGeom* geo, int n, int N, int64_t M,
                                    float* A32, double* tau, void* scratch, int mode,
                                    const OrbitFlux* fx, hipStream_t s) {
  const OrbitPlan pl = orbit_plan(K, N, n, scratch);
  const float* colscale = fx ? fx->colscale : nullptr;
  if (mode == kSumsOnly && fx->bases) {
    mode = kBases;
    A32 = fx->bases;
  }
  hipError_t e = mode == kScaled ? hipSuccess : orbit_sort(geo, pl, s);  // kept for the second pass
  if (e != hipSuccess) return e;
  const int Np = n + 2 * kSplinePad;
  const bool vec = (n % 32) == 0;
  const int run = box_run_tiles(pl), nruns = (pl.nt * pl.nt + run - 1) / run;
  const int64_t total = pl.o.nreps * nruns;
  if (total >= kMaxBoxRuns) return hipErrorInvalidValue;
  const size_t lds = (size_t)16 * kCbRegion * sizeof(float);
  const float2* P = reinterpret_cast<const float2*>(pairs);
  auto launch = [&](auto kern) -> hipError_t {
    const void* fn = reinterpret_cast<const void*>(kern);
    hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    kern<<<box_grid(total), 1024, lds, s>>>(P, Np, geo, pl.reps, pl.o, n, M, pl.nt, run, (uint32_t)total, A32, pl.part, colscale);
    return hipGetLastError();
  };
  switch (mode) {
    case kSumsOnly:
      e = launch(build_cubic_orbit_kernel<false, kSumsOnly>);
      break;
    case kScaled:
      e = vec ? launch(build_cubic_orbit_kernel<true, kScaled>) : launch(build_cubic_orbit_kernel<false, kScaled>);
      break;
    case kBases:
      e = launch(build_cubic_orbit_kernel<false, kBases>);
      break;
    default:
      e = vec ? launch(build_cubic_orbit_kernel<true, kPlain>) : launch(build_cubic_orbit_kernel<false, kPlain>);
  }
  if (e != hipSuccess) return e;
  return orbit_finish(pl, nruns, mode, K, geo, fx, tau, s);
}

// 16-bit orbit build: the pair (ending 16-byte aligned), then two 2 x 8 x 33 unit tiles
static size_t orbit16_pair_bytes(int n) {
  return (((size_t)(n + 2) * lds_stride(n) * sizeof(float2)) + 15) & ~(size_t)15;
}
static size_t orbit16_lds_bytes(int n) { return orbit16_pair_bytes(n) + (size_t)2 * (2 * 8 * 33 * 16); }

// LDS of the 16-bit box kernel: 16 box regions, then the two unit tiles
static size_t orbit16_box_lds_bytes(bool cubic) {
  return cubic ? (size_t)16 * kCbRegion * sizeof(float) + (size_t)2 * (2 * 4 * 33 * 16)
               : (size_t)16 * kFpRegion * sizeof(float) + (size_t)2 * (2 * 8 * 33 * 16);
}

static bool orbit16_pair_fits(int n) { return orbit16_lds_bytes(n) <= (size_t)kLdsBuildMaxBytes; }

static_assert((size_t)16 * kFpRegion * sizeof(float) + (size_t)2 * (2 * 8 * 33 * 16) <= kLdsBuildMaxBytes &&
              (size_t)16 * kCbRegion * sizeof(float) + (size_t)2 * (2 * 4 * 33 * 16) <= kLdsBuildMaxBytes,
              "the boxes and unit tiles fit the LDS");

static hipError_t orbit16_end(const OrbitPlan& pl, int64_t M, const ColGeom* geo, const Orbit16Out& out,
                              hipStream_t s) {
  const int64_t whole = (pl.o.nreps + 7) / 8 * 8;
  const int tail = (int)(out.ncols_pad / 8 - whole / 2);  // groups, fewer than 8
  const int nsum = (int)((whole + 255) / 256);
  const int64_t zero = (int64_t)(tail + ((pl.o.N & 1) ? 3 : 0)) * ((M + 255) / 256);
  orbit16_end_kernel<<<(unsigned)(nsum + zero), 256, 0, s>>>(pl.reps, pl.o, pl.part, pl.nranges, geo,
                                                            pl.nitems, nsum, tail, M, out);
  return hipGetLastError();
}

// f(bf16, scaled, lines) as compile-time flags of the 16-bit orbit kernels
template <typename F>
static hipError_t orbit16_form(int storage, int n, const float* colscale, F f) {
  auto on_lines = [&](auto bf, auto scaled) {
    return n % 4 == 0 ? f(bf, scaled, std::true_type{}) : f(bf, scaled, std::false_type{});
  };
  auto on_scale = [&](auto bf) {
    return colscale ? on_lines(bf, std::true_type{}) : on_lines(bf, std::false_type{});
  };
  return storage == PSFLIB_BF16_POW2 ? on_scale(std::true_type{}) : on_scale(std::false_type{});
}

static hipError_t launch_spread16(int storage, const ColGeom* geo, int n, int64_t M, const OrbitPlan& pl,
                                  const Orbit16Out& out, const OrbitFlux& fx, hipStream_t s) {
  const dim3 wgrid((unsigned)((pl.o.nreps + 15) / 16), (unsigned)pl.nranges);
  const hipError_t e = orbit16_form(storage, n, fx.colscale, [&](auto bf, auto, auto lines) {
    spread_orbit16_kernel<bf.value, lines.value><<<wgrid, 1024, 0, s>>>(
        fx.bases, geo, pl.reps, n, M, pl.rpr, pl.o.nreps, reinterpret_cast<uint16_t*>(out.lib), pl.part,
        fx.colscale);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  return orbit16_end(pl, M, geo, out, s);
}

// Base columns worth keeping between the passes.  The cubic values cost more than
// their way through memory at any size (128^2, 176^2 scene, bf16: 0.84 ms against
// 1.22).  Bilinear ones do where the 256 MiB last-level cache cannot hold them: 128^2,
// 128^2 scene, 256 MiB, 283 us kept, 308 formed again; 144^2 scene 401 and 366; 176^2
// 565 and 481.  From boxes (n > 131) kept all the same (256^2, 80^2 scene, 400 MiB: 557
// and 623).  On sides that are not multiples of 4, whose stores of parts of lines
// need the cache too, up to 88 MiB (101^2, 60^2 scene, 35 MiB: 79 and 85; 101^2, 99
// MiB: 180 and 158; 150^2, 60^2 scene, 77 MiB: 144 and 201; 90^2, 174 MiB: 354 and 318).
size_t orbit_bases_bytes(int n, int N, bool cubic) {
  const size_t bytes = (size_t)orbit_grid(N).nreps * (size_t)n * (size_t)n * 4;
  const size_t most = cubic || (n % 4 == 0 && !orbit16_pair_fits(n)) ? ~(size_t)0
                                                                     : (size_t)(n % 4 == 0 ? 256 : 88) << 20;
  return bytes <= most ? bytes : 0;
}

size_t build_lds_scratch_bytes(int K, int N, int n) {
  return build_orbit_supported(K, N) ? build_orbit_scratch_bytes(K, N, n) : bucket_scratch_bytes(K, (int64_t)N * N);
}

hipError_t launch_build_orbit16(int storage, const float* cube, int K, ColGeom* geo, int n, int N,
                                int64_t M, const Orbit16Out& out, void* scratch, const OrbitFlux* fx,
                                hipStream_t s) {
  const OrbitPlan pl = orbit_plan(K, N, n, scratch);
  const float* colscale = fx ? fx->colscale : nullptr;
  hipError_t e = fx ? hipSuccess : orbit_sort(geo, pl, s);  // the first pass has sorted
  if (e != hipSuccess) return e;
  uint16_t* Mh = reinterpret_cast<uint16_t*>(out.lib);
  if (fx && fx->bases) return launch_spread16(storage, geo, n, M, pl, out, *fx, s);
  const dim3 grid((unsigned)pl.items_max, (unsigned)pl.nranges);
  const dim3 wgrid((unsigned)((pl.o.nreps + 15) / 16), (unsigned)pl.nranges);
  if (!orbit16_pair_fits(n)) {  // a staged box per 32 x 32 pixels
    const size_t lds = orbit16_box_lds_bytes(false);
    auto launch = [&](auto kern) -> hipError_t {
      const void* fn = reinterpret_cast<const void*>(kern);
      hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (err != hipSuccess) return err;
      kern<<<wgrid, 1024, lds, s>>>(cube, K, geo, pl.reps, n, M, 0, pl.rpr,
                                   pl.o.nreps, Mh, pl.part, colscale);
      return hipGetLastError();
    };
    e = orbit16_form(storage, n, colscale, [&](auto bf, auto scaled, auto lines) {
      return launch(build_orbit16_box_kernel<bf.value, false, scaled.value, lines.value>);
    });
    if (e != hipSuccess) return e;
    return orbit16_end(pl, M, geo, out, s);
  }
  const int ls = lds_stride(n);
  const size_t lds = orbit16_lds_bytes(n);
  auto launch = [&](auto kern) -> hipError_t {
    const void* fn = reinterpret_cast<const void*>(kern);
    hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    kern<<<grid, 1024, lds, s>>>(cube, K, geo, pl.reps, pl.items, pl.nitems, pl.nb, n, ls, M,
                                 pl.rpr, pl.o.nreps, Mh, pl.part, colscale);
    return hipGetLastError();
  };
  e = orbit16_form(storage, n, colscale, [&](auto bf, auto scaled, auto lines) {
    return launch(build_orbit16_kernel<bf.value, scaled.value, lines.value>);
  });
  if (e != hipSuccess) return e;
  return orbit16_end(pl, M, geo, out, s);
}

hipError_t launch_build_cubic_orbit16(int storage, const float* pairs, int K, ColGeom* geo, int n,
                                      int N, int64_t M, const Orbit16Out& out, void* scratch,
                                      const OrbitFlux* fx, hipStream_t s) {
  const OrbitPlan pl = orbit_plan(K, N, n, scratch);
  const float* colscale = fx ? fx->colscale : nullptr;
  hipError_t e = fx ? hipSuccess : orbit_sort(geo, pl, s);  // the first pass has sorted
  if (e != hipSuccess) return e;
  uint16_t* Mh = reinterpret_cast<uint16_t*>(out.lib);
  if (fx && fx->bases) return launch_spread16(storage, geo, n, M, pl, out, *fx, s);
  const dim3 wgrid((unsigned)((pl.o.nreps + 15) / 16), (unsigned)pl.nranges);
  const size_t lds = orbit16_box_lds_bytes(true);
  const int Np = n + 2 * kSplinePad;
  auto launch = [&](auto kern) -> hipError_t {
    const void* fn = reinterpret_cast<const void*>(kern);
    hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    kern<<<wgrid, 1024, lds, s>>>(pairs, K, geo, pl.reps, n, M, Np, pl.rpr,
                                 pl.o.nreps, Mh, pl.part, colscale);
    return hipGetLastError();
  };
  e = orbit16_form(storage, n, colscale, [&](auto bf, auto scaled, auto lines) {
    return launch(build_orbit16_box_kernel<bf.value, true, scaled.value, lines.value>);
  });
  if (e != hipSuccess) return e;
  return orbit16_end(pl, M, geo, out, s);
}

}  // namespace psflib
