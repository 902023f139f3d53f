// Single-scene products with the library: S = A Z (Sec. 3, Eq. (6)) and the
// adjoint G = A^T g.  Both stream the library once from HBM and are bound by
// memory bandwidth; the scene and image vectors are small and stay in cache.
//
// A is column-major (column j is contiguous), so the forward product is a sum
// of scaled columns.  It is split over (row block, column chunk) workgroups:
// each thread owns 4 consecutive rows (16 bits: up to 8 rows, a row block of
// threads apart) and walks columns with 16 independent 16-byte non-temporal
// loads in flight; the threads of a workgroup are RT along the rows and CT along
// the columns, whose sums are added through LDS, and it writes a partial image;
// a second kernel adds the partials of every row in pairs, in a fixed order.  (Doing that
// sum in the last workgroup to finish each row block needs a device-scope
// release per workgroup, which writes back the XCD's L2: measured slower than
// the extra launch.)  Few columns take one launch: workgroups of 1024 threads
// that walk all of them.  Sums are blocked (16 columns per inner sum) so every
// rounding chain stays short.  Results are bitwise reproducible.
#include <math.h>
#include <stdlib.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>

#include "psflib_internal.h"

namespace psflib {

// ------------------------------------------------------------ forward -----
// Rows i0 .. i0 + 3 of a column, for images whose columns start at 16-byte
// boundaries (kAligned: M % 4 == 0), at any float, or of fewer than 4 pixels
// (kTiny: n = 1).
constexpr int kUnaligned = 0, kAligned = 1, kTiny = 2;

template <int MODE>
__device__ __forceinline__ f32x4 load_rows(const float* __restrict__ p) {
  if constexpr (MODE == kAligned) return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  if constexpr (MODE == kUnaligned) return __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(p));
  return (f32x4){p[0], 0.0f, 0.0f, 0.0f};
}

template <int MODE>
__device__ __forceinline__ void store_rows(float* __restrict__ p, const f32x4 v) {
  if constexpr (MODE == kAligned)
    *reinterpret_cast<f32x4*>(p) = v;
  else if constexpr (MODE == kUnaligned)
    *reinterpret_cast<f32x4u*>(p) = v;
  else
    p[0] = v[0];
}

// First row of the thread whose 4 rows would start at i0: the last thread of
// the image steps back to end with it (its first rows are its neighbour's too,
// with the same values).
template <int MODE>
__device__ __forceinline__ int64_t first_row(int64_t i0, int64_t M) {
  return MODE == kUnaligned && i0 > M - 4 ? M - 4 : i0;
}

// sum_j A[j][i0..i0+3] z(j) over the 16-column blocks c, c + CT, ... of
// [j0, j1), in three levels: 16 columns, 16 blocks, then the rest.
template <int MODE, int CT, typename Z>
__device__ __forceinline__ f32x4 matvec_rows(const float* __restrict__ A, Z z, int64_t M, int64_t i0,
                                             int64_t j0, int64_t j1, int c) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 outer = zero, mid = zero;
  int nblk = 0;
  int64_t j = j0 + 16 * c;
  for (; j + 16 <= j1; j += 16 * CT) {
    f32x4 v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = load_rows<MODE>(A + (j + u) * M + i0);
    f32x4 inner = v[0] * z(j);
#pragma unroll
    for (int u = 1; u < 16; ++u) inner += v[u] * z(j + u);
    mid += inner;
    if (++nblk == 16) {
      outer += mid;
      mid = zero;
      nblk = 0;
    }
  }
  f32x4 inner = zero;
  for (; j < j1; ++j) inner += load_rows<MODE>(A + j * M + i0) * z(j);  // the chunk's last block
  mid += inner;
  return outer + mid;
}

// 256 threads, RT along the rows (4 RT rows per workgroup).  Small images take
// fewer, which leaves fewer threads past the image's end and needs fewer partial
// images for the same number of workgroups (33^2 PSFs, 200^2 scene: 85 -> 35
// us, with the unaligned loads in place of one per float; 127^2: 236 -> 169 us).
template <int MODE, int RT>
__global__ __launch_bounds__(kMvThreads) void matvec_f32_kernel(const float* __restrict__ A,
                                                                const float* __restrict__ Z,
                                                                float* __restrict__ part,
                                                                float* __restrict__ out,
                                                                int64_t M, int64_t ncols,
                                                                int64_t chunk) {
  constexpr int CT = kMvThreads / RT;
  const int r = threadIdx.x % RT, c = __builtin_amdgcn_readfirstlane(threadIdx.x / RT);
  const int64_t row = ((int64_t)blockIdx.x * RT + r) * 4;
  const int64_t i0 = first_row<MODE>(row, M);
  const int64_t j0 = blockIdx.y * chunk;
  const int64_t j1 = (j0 + chunk < ncols) ? j0 + chunk : ncols;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (row < M) acc = matvec_rows<MODE, CT>(A, [=](int64_t j) { return Z[j]; }, M, i0, j0, j1, c);
  if constexpr (CT > 1) {
    __shared__ f32x4 red[CT][RT];
    red[c][r] = acc;
    __syncthreads();
    if (c > 0) return;
#pragma unroll
    for (int k = 1; k < CT; ++k) acc += red[k][r];
  }
  if (row < M) store_rows<MODE>((gridDim.y == 1 ? out : part + blockIdx.y * M) + i0, acc);
}

// One launch for few columns: 1024 threads, 16 along the rows (64 rows per
// workgroup), every column.  The scene is staged in LDS (a wave's lanes are on
// four columns).
constexpr int64_t kMvOneMaxCols32 = 1024, kMvOneMaxCols16 = 2048;

template <int MODE>
__global__ __launch_bounds__(1024) void matvec_one_f32_kernel(const float* __restrict__ A,
                                                              const float* __restrict__ Z,
                                                              float* __restrict__ out, int64_t M,
                                                              int64_t ncols) {
  constexpr int RT = 16, CT = 1024 / RT;
  __shared__ float zs[kMvOneMaxCols32];
  __shared__ f32x4 red[CT][RT];
  for (int j = threadIdx.x; j < ncols; j += 1024) zs[j] = Z[j];
  __syncthreads();
  const int r = threadIdx.x % RT, c = threadIdx.x / RT;
  const int64_t row = ((int64_t)blockIdx.x * RT + r) * 4;
  const int64_t i0 = first_row<MODE>(row, M);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (row < M)
    acc = matvec_rows<MODE, CT>(A, [&](int64_t j) { return zs[j]; }, M, i0, 0, ncols, c);
  red[c][r] = acc;
  // halves of the column threads, in a fixed order
#pragma unroll
  for (int k = CT / 2; k > 0; k >>= 1) {
    __syncthreads();
    if (c < k) red[c][r] += red[c + k][r];
  }
  if (c == 0 && row < M) store_rows<MODE>(out + i0, red[0][r]);
}

// 16-bit storage: element (i, slot s) at ((s/8)*M + i)*8 + s%8, slot s holding
// column perm[s].  One thread per row; one 16-byte load covers 8 slots.  The
// chunk's scene values Z[perm[s]] scaled by 2^eslot[s] are staged in LDS and
// read as broadcasts.
__device__ __forceinline__ float h16_to_f32(uint32_t h, bool bf16) {
  if (bf16) return __uint_as_float(h << 16);
  return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

template <bool BF16>
__device__ __forceinline__ void unpack8(const u32x4 p, float* f) {
  if constexpr (BF16) {
    f[0] = __uint_as_float(p.x << 16);
    f[1] = __uint_as_float(p.x & 0xFFFF0000u);
    f[2] = __uint_as_float(p.y << 16);
    f[3] = __uint_as_float(p.y & 0xFFFF0000u);
    f[4] = __uint_as_float(p.z << 16);
    f[5] = __uint_as_float(p.z & 0xFFFF0000u);
    f[6] = __uint_as_float(p.w << 16);
    f[7] = __uint_as_float(p.w & 0xFFFF0000u);
  } else {
    f[0] = h16_to_f32(p.x & 0xFFFFu, false);
    f[1] = h16_to_f32(p.x >> 16, false);
    f[2] = h16_to_f32(p.y & 0xFFFFu, false);
    f[3] = h16_to_f32(p.y >> 16, false);
    f[4] = h16_to_f32(p.z & 0xFFFFu, false);
    f[5] = h16_to_f32(p.z >> 16, false);
    f[6] = h16_to_f32(p.w & 0xFFFFu, false);
    f[7] = h16_to_f32(p.w >> 16, false);
  }
}

// The sums of one thread: rows src[0..R-1] over the groups g = g0 + c GB, ...
// in steps of CT GB (GB = 16 / R groups per block of 16 loads), in three
// levels: 16 groups, 8 of those, then the rest.  zs holds the 8 scene values of
// group g at 2 (g - g0).
template <bool BF16, int R, int CT>
__device__ __forceinline__ void matvec16_rows(const u32x4* const* src, const f32x4* __restrict__ zs,
                                              int64_t M, int64_t g0, int64_t g1, int c, float* res) {
  constexpr int GB = 16 / R;
  float outer[R], mid[R], inner[R];
#pragma unroll
  for (int r = 0; r < R; ++r) outer[r] = mid[r] = inner[r] = 0.0f;
  auto use = [&](const u32x4* p, int64_t g) {
    const f32x4 za = zs[2 * (g - g0)], zb = zs[2 * (g - g0) + 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float f[8];
      unpack8<BF16>(p[r], f);
      float acc = inner[r];
      acc = fmaf(f[0], za.x, acc);
      acc = fmaf(f[1], za.y, acc);
      acc = fmaf(f[2], za.z, acc);
      acc = fmaf(f[3], za.w, acc);
      acc = fmaf(f[4], zb.x, acc);
      acc = fmaf(f[5], zb.y, acc);
      acc = fmaf(f[6], zb.z, acc);
      acc = fmaf(f[7], zb.w, acc);
      inner[r] = acc;
    }
  };
  int ing = 0, nblk = 0;
  int64_t g = g0 + (int64_t)c * GB;
  for (; g + GB <= g1; g += CT * GB) {
    u32x4 p[GB][R];
#pragma unroll
    for (int u = 0; u < GB; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) p[u][r] = __builtin_nontemporal_load(src[r] + (g + u) * M);
#pragma unroll
    for (int u = 0; u < GB; ++u) use(p[u], g + u);
    ing += GB;
    if (ing == 16) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        mid[r] += inner[r];
        inner[r] = 0.0f;
      }
      ing = 0;
      if (++nblk == 8) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          outer[r] += mid[r];
          mid[r] = 0.0f;
        }
        nblk = 0;
      }
    }
  }
  for (; g < g1; ++g) {  // the chunk's last block
    u32x4 p[R];
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = __builtin_nontemporal_load(src[r] + g * M);
    use(p, g);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) res[r] = outer[r] + (mid[r] + inner[r]);
}

// T threads, RT along the rows; each thread owns R rows, RT apart, so that a
// workgroup reads R RT 16-byte units of every group in one piece, and each
// broadcast of the group's 8 scene values serves R loads.  ZG: groups whose
// scene values the LDS holds.
template <bool BF16, int T, int R, int RT, int ZG>
__global__ __launch_bounds__(T) void matvec_h16_kernel(const u32x4* __restrict__ Mp,
                                                       const int32_t* __restrict__ perm,
                                                       const int32_t* __restrict__ eslot,
                                                       const float* __restrict__ Z,
                                                       float* __restrict__ part,
                                                       float* __restrict__ out, int64_t M,
                                                       int64_t ngroups, int64_t chunk_g) {
  constexpr int CT = T / RT;
  __shared__ f32x4 zs[ZG * 2];
  const int tid = threadIdx.x, t = tid % RT, c = tid / RT;
  const int64_t i0 = (int64_t)blockIdx.x * RT * R + t;
  const int64_t g0 = blockIdx.y * chunk_g;
  const int64_t g1 = (g0 + chunk_g < ngroups) ? g0 + chunk_g : ngroups;
  const int64_t ng = g1 - g0;
  float* zsf = reinterpret_cast<float*>(zs);
  for (int64_t k = tid; k < ng * 8; k += T) {
    const int64_t slot = g0 * 8 + k;
    const int32_t j = perm[slot];
    zsf[k] = (j >= 0) ? ldexpf(Z[j], eslot[slot]) : 0.0f;
  }
  __syncthreads();
  // rows past the image read row M-1 (in bounds) and are not written
  const u32x4* src[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + (int64_t)RT * r;
    src[r] = Mp + (i < M ? i : M - 1);
  }
  float res[R];
  matvec16_rows<BF16, R, CT>(src, zs, M, g0, g1, c, res);
  if constexpr (CT > 1) {
    __shared__ float red[CT][R][RT];
#pragma unroll
    for (int r = 0; r < R; ++r) red[c][r][t] = res[r];
    __syncthreads();
    if (c > 0) return;
#pragma unroll
    for (int k = 1; k < CT; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r) res[r] += red[k][r][t];
  }
  float* dst = (gridDim.y == 1) ? out : part + blockIdx.y * M;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + (int64_t)RT * r;
    if (i < M) dst[i] = res[r];
  }
}

// out[i] = sum over chunks of part[chunk][i].  A workgroup is 64 rows x 4
// quarters of the chunks (whole blocks of 16 partials, loaded together and
// added in pairs: a chain through 16 had up to 1.2 times the error); the quarters'
// sums are added in pairs.
__global__ __launch_bounds__(256) void reduce_rows_kernel(const float* __restrict__ part,
                                                          int64_t nchunks, int64_t M,
                                                          float* __restrict__ out) {
  __shared__ float red[4][64];
  const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + r;
  const int64_t blocks = (nchunks + 15) / 16;
  const int64_t c1 = 16 * (blocks * (q + 1) / 4) < nchunks ? 16 * (blocks * (q + 1) / 4) : nchunks;
  float total = 0.0f;
  if (i < M)
    for (int64_t c0 = 16 * (blocks * q / 4); c0 < c1; c0 += 16) {
      float p[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) p[u] = (c0 + u < c1) ? part[(c0 + u) * M + i] : 0.0f;
#pragma unroll
      for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int u = 0; u < h; ++u) p[u] += p[u + h];
      total += p[0];
    }
  red[q][r] = total;
  __syncthreads();
  if (q == 0 && i < M) out[i] = (red[0][r] + red[1][r]) + (red[2][r] + red[3][r]);
}

// Shape of the product: threads along the rows, rows per thread, row blocks and
// column chunks, about 512 workgroups in all (two per CU), 256 for 16-bit ones
// of 2048 rows (one per CU; 128^2: 80 us against 88-94 us with 192 or 384; those
// of 512 rows, 91^2 PSFs with a 239^2 scene: 145 us with 512, 180 us with 256).
// The number can be overridden with PSFLIB_MV_WORKGROUPS for tuning sweeps.
static int64_t mv_target_workgroups(int rt, int r) {
  static const long env = [] {
    const char* e = getenv("PSFLIB_MV_WORKGROUPS");
    return e ? strtol(e, nullptr, 10) : 0L;
  }();
  if (env > 0) return env;
  return rt * r == 2048 ? kMvTargetWorkgroups16 : kMvTargetWorkgroups32;
}

struct MvShape {
  bool one;  // one launch of 1024-thread workgroups over all columns
  int rt, r;
  int64_t rowblocks, chunk, nchunks;  // chunk: columns (FP32) or 8-column groups (16-bit)
};

static MvShape mv_shape(int storage, int64_t M, int64_t ncols, int64_t ncols_pad) {
  MvShape sh;
  const bool f32 = storage == PSFLIB_FP32;
  const int64_t units = f32 ? ncols : ncols_pad / 8;
  auto padded = [&](int64_t rows) { return (M + rows - 1) / rows * rows; };
  // One launch: up to 16 columns (16-bit: 16 groups) per thread, and images of
  // at most 256 workgroups of 64 rows (32^2: 8.3 us, the launches' rate, against
  // 11; 128^2 PSFs, 32^2 scene, float32 12.3 against 14.9 us, bf16 9.3 against 17;
  // 200^2 PSFs, 40^2 scene: 47 against 44 us).
  if (M <= 16384 && (f32 ? ncols <= kMvOneMaxCols32 : ncols_pad <= kMvOneMaxCols16)) {
    sh.one = true;
    sh.r = f32 ? 4 : 1;
    sh.rt = f32 ? 16 : 64;
    sh.chunk = units;
    sh.nchunks = 1;
    sh.rowblocks = (M + 63) / 64;
    return sh;
  }
  sh.one = false;
  if (f32) {
    // 1024 rows per workgroup; small images of small libraries 512 or 256, whichever
    // leaves few threads past the end (96^2 with 1024: 52 us, with 256: 59 us; 64^2 with
    // 512: 14.5 us, with 1024: 16.1 us; 80^2 with 256: 27 us, with 512: 32 us).  Large
    // libraries of small images read better in the longer pieces (72^2, 181^2 scene: 1024
    // rows 110 us, 512 rows 121; 80^2: 127, 256 rows 145; 56^2, 256^2 scene: 122 and 140;
    // 80^2, 80^2 scene: 29.0 and 25.6).
    sh.r = 4;
    const bool large = (M >= 4608 && ncols >= 8192) || M * ncols >= 100000000;
    sh.rt = M >= 8192 || large ? 256 : padded(512) * 32 <= M * 33 ? 128 : 64;
  } else {
    // 2048 rows where they leave few threads past the end, else 512, and fewer
    // rows per thread for small images (bf16: 101^2, 2048: 39 us, 512: 43 us; 96^2
    // 37 and 31 us); with many columns 2048 rows of smaller images too, and where
    // they leave up to an eighth past the end (64^2, 181^2 scene 43.1 against 50.5; 96^2
    // 96 against 102; 150^2 scene 64^2 36 against 33, 96^2 equal).
    sh.r = 8;
    const bool many = ncols_pad >= 30000;
    sh.rt = M >= (many ? 4096 : 8192) && padded(2048) * (many ? 8 : 11) <= M * (many ? 9 : 12) ? 256 : 64;
    if (sh.rt == 64)
      while (sh.r > 2 && padded(sh.r * 64) * 8 > M * 9 && padded(sh.r * 32) < padded(sh.r * 64)) sh.r /= 2;
  }
  const int64_t rows = (int64_t)sh.r * sh.rt;
  sh.rowblocks = (M + rows - 1) / rows;
  // As many chunks as keep the workgroups within the target: a few more than two a
  // CU cost their CUs a third turn (120^2, 150^2 scene, bf16: 522 workgroups 110 us, 464
  // 99; 96^2, 128^2 scene, float32: 104 and 89).  One chunk a row block more where chunks
  // are so short that the next longer ones, whole blocks of 16, would leave a seventh of
  // the target idle (200^2, 40^2 scene, bf16: 260 workgroups 25 us, 140 32).
  const int64_t target = mv_target_workgroups(sh.rt, sh.r);
  auto chunk_of = [&](int64_t want) {
    const int64_t chunk = ((units + want - 1) / want + 15) / 16 * 16;
    return !f32 && chunk > kMv16MaxChunkGroups ? (int64_t)kMv16MaxChunkGroups : chunk;
  };
  int64_t chunk = chunk_of(std::max<int64_t>(1, target / sh.rowblocks));
  if ((units + chunk - 1) / chunk * sh.rowblocks * 7 < target * 6)
    chunk = chunk_of((target + sh.rowblocks - 1) / sh.rowblocks);
  sh.chunk = chunk;
  sh.nchunks = (units + chunk - 1) / chunk;
  return sh;
}

int64_t matvec_partial_floats(int storage, int64_t M, int64_t ncols, int64_t ncols_pad) {
  const MvShape sh = mv_shape(storage, M, ncols, ncols_pad);
  return sh.nchunks > 1 ? sh.nchunks * M : 0;
}

hipError_t launch_matvec(int storage, const void* lib, const Cols16& cx, const float* Z,
                         int64_t M, int64_t ncols, int64_t ncols_pad, float* partial, float* out,
                         hipStream_t s) {
  const MvShape sh = mv_shape(storage, M, ncols, ncols_pad);
  const dim3 grid((unsigned)sh.rowblocks, (unsigned)sh.nchunks);
  if (storage == PSFLIB_FP32) {
    const float* A = reinterpret_cast<const float*>(lib);
    auto run = [&](auto mode) {
      constexpr int MODE = decltype(mode)::value;
      auto one = [&](auto kern) { kern<<<grid, 1024, 0, s>>>(A, Z, out, M, ncols); };
      auto split = [&](auto kern) { kern<<<grid, kMvThreads, 0, s>>>(A, Z, partial, out, M, ncols, sh.chunk); };
      if (sh.one)
        one(matvec_one_f32_kernel<MODE>);
      else
        sh.rt == 64 ? split(matvec_f32_kernel<MODE, 64>)
        : sh.rt == 128 ? split(matvec_f32_kernel<MODE, 128>) : split(matvec_f32_kernel<MODE, 256>);
    };
    if (M % 4 == 0)
      run(std::integral_constant<int, kAligned>());
    else if (M >= 4)
      run(std::integral_constant<int, kUnaligned>());
    else
      run(std::integral_constant<int, kTiny>());
  } else {
    const int64_t ngroups = ncols_pad / 8;
    const u32x4* Mp = reinterpret_cast<const u32x4*>(lib);
    auto run = [&](auto fmt) {
      constexpr bool BF = decltype(fmt)::value;
      auto go = [&](auto kern, int threads) {
        kern<<<grid, threads, 0, s>>>(Mp, cx.perm, cx.eslot, Z, partial, out, M, ngroups, sh.chunk);
      };
      constexpr int T = kMv16Threads, ZG = kMv16MaxChunkGroups;
      if (sh.one)
        go(matvec_h16_kernel<BF, 1024, 1, 64, (int)kMvOneMaxCols16 / 8>, 1024);
      else if (sh.rt == 256)
        go(matvec_h16_kernel<BF, T, 8, 256, ZG>, T);
      else if (sh.r == 8)
        go(matvec_h16_kernel<BF, T, 8, 64, ZG>, T);
      else if (sh.r == 4)
        go(matvec_h16_kernel<BF, T, 4, 64, ZG>, T);
      else
        go(matvec_h16_kernel<BF, T, 2, 64, ZG>, T);
    };
    if (storage == PSFLIB_BF16_POW2)
      run(std::true_type());
    else
      run(std::false_type());
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || sh.nchunks == 1) return e;
  reduce_rows_kernel<<<(unsigned)((M + 63) / 64), 256, 0, s>>>(partial, sh.nchunks, M, out);
  return hipGetLastError();
}

// ------------------------------------------------------------ adjoint -----
// G_j = sum_i A_ij g_i, bound by the stream of the library.  A workgroup stages
// g of its row block (up to kAdjRows rows) in LDS; its waves then stream whole
// columns (16-bit: 8-slot groups), C of them at a time in rounds of U row steps
// (C U = kAdjLoads loads of 16 bytes per lane), the loads of the next round
// issued before a round is used -- also over the end of a column, whose sum is
// reduced over the wave while the next column is on its way, and while g is
// staged.  C grows for small images, which have few row steps.  SPLIT: the
// waves of a workgroup take the row steps of the same columns in turn and add
// their sums through LDS, where there are too few columns for all the waves.
// Images whose columns do not start at 16-byte boundaries take the same loads,
// unaligned.
constexpr int kAdjLoads = 8;
constexpr int kNonTemporal = 2;  // cache policy of a buffer load

// Sums of V values over the wave, each value in one set of 64 / V lanes:
// value lane / (64 / V) is returned.  Every exchange halves the values.
template <int V>
__device__ __forceinline__ float wave_sums(float (&v)[V], int lane) {
  int off = 32;
#pragma unroll
  for (int n = V; n > 1; n >>= 1, off >>= 1) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int k = 0; k < n / 2; ++k) {
      const float keep = up ? v[k + n / 2] : v[k], send = up ? v[k] : v[k + n / 2];
      v[k] = keep + __shfl_xor(send, off, 64);
    }
  }
  for (; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
  return v[0];
}

// Sum of value q of the workgroup's waves, in pairs.
template <int NW, int V>
__device__ __forceinline__ float waves_sum(const float (&red)[NW][V], int q) {
  static_assert(NW == 8, "pairs of pairs of pairs");
  return ((red[0][q] + red[1][q]) + (red[2][q] + red[3][q])) +
         ((red[4][q] + red[5][q]) + (red[6][q] + red[7][q]));
}

// The block's rows of g on their way into LDS: `units` 16-byte units (at most
// kAdjRows rows), zeros past the last row.  All loads are issued at construction,
// together and before the first round's, so that the copy waits for one of them
// and not for the library (a float at a time in a loop behind the first round's
// loads: 2 to 4 us a call more, 128^2 PSFs of a 24^2 scene, float32, 15.7 against
// 10.5 us, of a 110^2 scene, bf16, 63.1 against 60.2).
struct GRows {
  static constexpr int kUnits = kAdjRows / 4 / kAdjThreads;  // per thread, at most
  f32x4 v[kUnits];
  int units;
  __device__ __forceinline__ GRows(const float* __restrict__ g, int rows, int n, int tid) : units(n) {
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc((void*)g, (short)0, rows * 4, 0x00020000);
#pragma unroll
    for (int k = 0; k < kUnits; ++k)
      if (k * kAdjThreads < units)
        v[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(src, (tid + k * kAdjThreads) * 16, 0, 0));
  }
  __device__ __forceinline__ void store(f32x4* __restrict__ gs, int tid) const {
#pragma unroll
    for (int k = 0; k < kUnits; ++k)
      if (tid + k * kAdjThreads < units) gs[tid + k * kAdjThreads] = v[k];
    __syncthreads();
  }
};

// The rounds of one wave, in order: column groups first, first + stride, ...
// below end, each in `rounds` rounds.  load(buffer, group, round) issues a
// round's loads, use(buffer, round) multiplies them, finish(group) follows a
// group's last round.  Two buffers in turn.
template <typename Buf, typename Load, typename Use, typename Stage, typename Finish>
__device__ __forceinline__ void adjoint_rounds(int64_t first, int64_t end, int64_t stride, int rounds,
                                               Load load, Stage stage, Use use, Finish finish) {
  Buf a, b;
  int64_t grp = first, ngrp = first;
  int r = 0, nr = 0;
  if (first < end) load(a, first, 0);
  stage();
  auto step = [&](Buf& cur, Buf& next) {
    nr = r + 1;
    ngrp = grp;
    if (nr == rounds) {
      nr = 0;
      ngrp += stride;
    }
    if (ngrp < end) load(next, ngrp, nr);
    __builtin_amdgcn_sched_barrier(0);
    use(cur, r);
    if (nr == 0) finish(grp);
    grp = ngrp;
    r = nr;
  };
  while (grp < end) {
    step(a, b);
    if (grp >= end) break;
    step(b, a);
  }
}

// Row steps of 256 rows (4 per lane).  A column's rows of this block are read
// through a buffer that ends with them, so what lies past the end -- rows of a
// step that the image does not fill, steps that fill up a round -- loads as zero
// whatever the library holds there, and the staged g is zero too.  (Reading the
// last rows again with a zero g would turn an infinite entry there into NaN.)
// Buffer loads need no more than the alignment of a float and check every float
// against the end.  (As fast as global loads, 0 to 4% faster: 96^2 54.2 -> 53.7 us,
// 200^2 PSFs with a 128^2 scene 394 -> 380, 128^2 160.8 -> 160.1.)
template <int C, bool SPLIT>
__global__ __launch_bounds__(kAdjThreads, 4) void adjoint_f32_kernel(const float* __restrict__ A,
                                                                     const float* __restrict__ g,
                                                                     float* __restrict__ out,
                                                                     int64_t M, int64_t ncols,
                                                                     int64_t block_rows, int rounds,
                                                                     int64_t per_wg,
                                                                     int64_t out_stride) {
  constexpr int U = kAdjLoads / C;
  constexpr int SUB = U >= 4 ? 4 : U;  // sums per column and component: short rounding chains
  constexpr int NW = kAdjThreads / 64;
  constexpr int W = SPLIT ? NW : 1;  // waves on one group of columns
  extern __shared__ f32x4 gs[];  // [rounds * U * W steps][64]
  __shared__ float red[2][NW][C];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.y * block_rows;
  const int rows = (int)(M - row0 < block_rows ? M - row0 : block_rows);
  const int64_t groups = (ncols + C - 1) / C;
  const int sub = SPLIT ? wave : 0;  // this wave's steps: sub + W k
  struct Buf {
    f32x4 v[U][C];
  };
  auto load = [&](Buf& b, int64_t grp, int r) {
    __amdgpu_buffer_rsrc_t col[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int64_t j = grp * C + c;
      col[c] = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (j < ncols ? j : ncols - 1) * M + row0),
                                                 (short)0, rows * 4, 0x00020000);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = 256 * (sub + W * (r * U + u)) + 4 * lane;
#pragma unroll
      for (int c = 0; c < C; ++c)
        b.v[u][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(col[c], i * 4, 0, kNonTemporal));
    }
  };
  const GRows gr(g + row0, rows, rounds * U * W * 64, tid);
  auto stage = [&]() { gr.store(gs, tid); };
  f32x4 acc[C][SUB] = {};
  auto use = [&](const Buf& b, int r) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const f32x4 gv = gs[(sub + W * (r * U + u)) * 64 + lane];
#pragma unroll
      for (int c = 0; c < C; ++c) acc[c][u % SUB] += b.v[u][c] * gv;
    }
  };
  int buf = 0;
  auto finish = [&](int64_t grp) {
    float sum[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      f32x4 a = acc[c][0];
#pragma unroll
      for (int u = 1; u < SUB; ++u) a += acc[c][u];
      sum[c] = (a[0] + a[1]) + (a[2] + a[3]);
#pragma unroll
      for (int u = 0; u < SUB; ++u) acc[c][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float tot = wave_sums<C>(sum, lane);
    if constexpr (SPLIT) {
      if (lane % (64 / C) == 0) red[buf][wave][lane / (64 / C)] = tot;
      __syncthreads();  // the other buffer's readers are behind the previous one
      if (tid < C && grp * C + tid < ncols) {
        tot = waves_sum(red[buf], tid);
        out[(int64_t)blockIdx.y * out_stride + grp * C + tid] = tot;
      }
      buf ^= 1;
    } else {
      const int64_t j = grp * C + lane / (64 / C);
      if (lane % (64 / C) == 0 && j < ncols) out[(int64_t)blockIdx.y * out_stride + j] = tot;
    }
  };
  const int64_t g0 = (int64_t)blockIdx.x * per_wg, g1 = g0 + per_wg < groups ? g0 + per_wg : groups;
  adjoint_rounds<Buf>(g0 + (SPLIT ? 0 : wave), g1, SPLIT ? 1 : NW, rounds, load, stage, use, finish);
}

// 16-bit: row steps of 64 rows (one per lane, 8 slots in 16 bytes), one group
// at a time in rounds of U steps, through a buffer that ends with the block's
// rows as above.  The sums of group grp belong to slots 8 grp + q, i.e. columns
// perm[8 grp + q]; they are written at the column's index.
template <bool BF16, int U, bool SPLIT>
__global__ __launch_bounds__(kAdjThreads, 4) void adjoint_h16_kernel(const u32x4* __restrict__ Mp,
                                                                     const int32_t* __restrict__ perm,
                                                                     const int32_t* __restrict__ eslot,
                                                                     const float* __restrict__ g,
                                                                     float* __restrict__ out,
                                                                     int64_t M, int64_t ngroups,
                                                                     int64_t block_rows, int rounds,
                                                                     int64_t per_wg,
                                                                     int64_t out_stride,
                                                                     int apply_exp) {
  // Two sums per slot over a round, added to the slot's total when it ends: a chain
  // of U / 2 products, then one of at most 32 rounds (256 steps of 64 rows in one
  // chain had 1.3 times the error, and the rounds cost no time: the loads bound it).
  constexpr int SUB = 2;
  constexpr int NW = kAdjThreads / 64;
  constexpr int W = SPLIT ? NW : 1;  // waves on one group
  extern __shared__ f32x4 gs4[];
  __shared__ float red[2][NW][8];
  const float* gs = reinterpret_cast<const float*>(gs4);  // [rounds * U * W steps][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.y * block_rows;
  const int sub = SPLIT ? wave : 0;  // this wave's steps: sub + W k
  const int rows = (int)(M - row0 < block_rows ? M - row0 : block_rows);
  struct Buf {
    u32x4 v[U];
  };
  auto load = [&](Buf& b, int64_t grp, int r) {
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Mp + grp * M + row0), (short)0, rows * 16, 0x00020000);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = 64 * (sub + W * (r * U + u)) + lane;
      b.v[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, i * 16, 0, kNonTemporal));
    }
  };
  const GRows gr(g + row0, rows, rounds * U * W * 16, tid);
  auto stage = [&]() { gr.store(gs4, tid); };
  float total[8] = {};
  auto use = [&](const Buf& b, int r) {
    float acc[SUB][8] = {};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float gv = gs[(sub + W * (r * U + u)) * 64 + lane];
      float f[8];
      unpack8<BF16>(b.v[u], f);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[u % SUB][q] = fmaf(f[q], gv, acc[u % SUB][q]);
      __builtin_amdgcn_sched_barrier(0);  // one load unpacked at a time
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) total[q] += acc[0][q] + acc[1][q];
  };
  int buf = 0;
  auto finish = [&](int64_t grp) {
    float sum[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      sum[q] = total[q];
      total[q] = 0.0f;
    }
    float tot = wave_sums<8>(sum, lane);
    bool writes = lane % 8 == 0;
    int q = lane / 8;
    if constexpr (SPLIT) {
      if (writes) red[buf][wave][q] = tot;
      __syncthreads();  // the other buffer's readers are behind the previous one
      writes = tid < 8;
      q = tid;
      if (writes) tot = waves_sum(red[buf], q);
      buf ^= 1;
    }
    if (writes) {
      const int64_t slot = grp * 8 + q;
      const int32_t j = perm[slot];
      if (j >= 0) out[(int64_t)blockIdx.y * out_stride + j] = apply_exp ? ldexpf(tot, eslot[slot]) : tot;
    }
  };
  const int64_t g0 = (int64_t)blockIdx.x * per_wg, g1 = g0 + per_wg < ngroups ? g0 + per_wg : ngroups;
  adjoint_rounds<Buf>(g0 + (SPLIT ? 0 : wave), g1, SPLIT ? 1 : NW, rounds, load, stage, use, finish);
}

// out[j] = 2^e_j * sum over row blocks (fixed order), or the plain sum for FP32.
__global__ __launch_bounds__(256) void reduce_cols_kernel(const float* __restrict__ part,
                                                          int64_t nblocks, int64_t stride,
                                                          int64_t ncols,
                                                          const int32_t* __restrict__ exps,
                                                          float* __restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= ncols) return;
  float tot = 0.0f;
  for (int64_t b = 0; b < nblocks; ++b) tot += part[b * stride + j];
  out[j] = exps ? ldexpf(tot, exps[j]) : tot;
}

// Launch shape: row blocks (equal, of whole row steps), columns or groups a
// wave takes at a time, its rounds, and the column groups per workgroup.
struct AdjShape {
  int64_t nb, block_rows, per_wg, grid_x;
  int c, rounds;
  bool split;
  size_t lds;
};

static AdjShape adj_shape(bool f32, int64_t M, int64_t units) {
  AdjShape sh;
  const int64_t step = f32 ? 256 : 64;  // rows per step
  sh.nb = (M + kAdjRows - 1) / kAdjRows;
  sh.block_rows = ((M + sh.nb - 1) / sh.nb + step - 1) / step * step;
  sh.nb = (M + sh.block_rows - 1) / sh.block_rows;
  const int64_t steps = (std::min(M, sh.block_rows) + step - 1) / step;
  const int64_t waves = kAdjThreads / 64;
  auto padded = [](int64_t n, int c) { const int64_t u = kAdjLoads / c; return (n + u - 1) / u * u; };
  // The waves of a workgroup share columns (split) where there are far fewer
  // columns (groups) than resident waves (128^2 PSFs, 20^2 scene, bf16: 11
  // against 31 us), and where a column fills whole rounds of all the waves:
  // 8 KiB at a time of one column then read better than 1 KiB of eight (128^2
  // PSFs, 256^2 scene, fp16: 317 against 330 us; 200^2 and 128^2, fp32, whose
  // rounds would be a fifth empty: 460 against 417 us).  In between, a column per wave
  // makes one round of 192 to 232 workgroups of 8 columns, enough to fill the memory,
  // where shared columns leave some CUs 7 and some 6 of them (128^2, bf16, 112^2 scene,
  // 1568 groups: 62.2 us against 66.3; 116^2 67 against 70; 120^2, 1800, a tie at 71;
  // 124^2, 1928: 77.0 against 74.6; float32, 40^2 18.4 against 19.6, 44^2 a tie at 22;
  // 16-bit columns of one round a wave some longer: 64^2, 122^2 scene, 1864, 22.3
  // against 23.5, 140^2, 2456, 32.6 against 28.1).
  const int64_t share = (steps + waves - 1) / waves, columns = sh.nb * units;
  const int64_t many = f32 || share > kAdjLoads ? 1856 : 2048;
  sh.split = steps >= waves && (columns < 1536 || (columns >= many && share >= kAdjLoads &&
                                                   8 * waves * padded(share, 1) <= 9 * steps));
  const int64_t wsteps = sh.split ? share : steps;
  // columns at a time: as few as leave at most an eighth of a column's rounds
  // empty, but never so many that fewer than 1024 waves have work
  // (16-bit: one group, in rounds of kAdjLoads / c steps)
  const int cmax = f32 ? 8 : 2;
  sh.c = 1;
  while (sh.c < cmax && 8 * padded(wsteps, sh.c) > 9 * wsteps &&
         padded(wsteps, 2 * sh.c) < padded(wsteps, sh.c) &&
         (!f32 || sh.nb * units * (sh.split ? waves : 1) / (2 * sh.c) >= 1024))
    sh.c *= 2;
  const int64_t psteps = padded(wsteps, sh.c);
  sh.rounds = (int)(psteps / (kAdjLoads / sh.c));
  sh.lds = (size_t)psteps * (sh.split ? waves : 1) * step * 4;
  // Workgroups: those resident at once (two per CU), each staging g once, or a
  // multiple of them of about 1 MiB of the library each where it is larger than
  // that, so that the CUs finish together (256^2, bf16: 1.22 ms against 1.30
  // with resident workgroups only; 128^2, bf16, of 0.5 instead of 1 MiB: 89
  // against 85 us; 181^2 PSFs of two row blocks, 200^2 scene: 415 against 404).
  // Float32 libraries of three row blocks and more, whose workgroups' ranges lie
  // further apart, take half as much each (200^2 PSFs, 128^2 scene: 412 against
  // 420 us), and libraries of 2 GiB and more of several long row blocks a quarter
  // (256^2, bf16: 1231 against 1268 us, 160^2 scene, fp16 475 against 489; one row
  // block, 128^2 PSFs, 256^2 scene, bf16: 315 against 310; blocks of 8448 rows, 129^2
  // PSFs, 256^2 scene, float32: 659 against 645).
  const int64_t bytes = columns * std::min(M, sh.block_rows) * (f32 ? 4 : 16);
  const bool far = sh.nb >= 2 && sh.block_rows >= 12288 && bytes >= (int64_t)2 << 30;
  const int64_t turn = (int64_t)(far ? 128 : f32 && sh.nb >= 3 ? 256 : 512) << 20;
  const int64_t turns = std::max<int64_t>(1, (bytes + turn / 2) / turn);
  const int64_t want = std::max<int64_t>(1, 512 * turns / sh.nb);
  const int64_t groups = f32 ? (units + sh.c - 1) / sh.c : units, quantum = sh.split ? 1 : waves;
  sh.per_wg = std::max<int64_t>(1, ((groups + want - 1) / want + quantum - 1) / quantum) * quantum;
  // 16-bit libraries of up to two such turns, shared columns: near that number, the
  // groups per workgroup that leave the fullest CU the fewest, each workgroup
  // costing a tenth of a group more for its copy of g, and a CU with a single
  // workgroup, whose barriers nothing covers, a twentieth (128^2, 160^2 scene: 800
  // workgroups of 4 groups, 16 on the fullest CU, 136 us; 458 of 7, 14 groups, 125;
  // 70^2 scene: 308 of 2, 4 groups, 32.6 us; 206 of 3, 29.2).  Groups of fewer rows
  // gain nothing by it (96^2, 100^2 scene: 31.3 us so, 34.0 by the count).
  if (!f32 && sh.split && turns <= 2 && sh.block_rows >= 12288) {
    const int64_t near = sh.per_wg;
    int64_t best = INT64_MAX;
    for (int64_t p = std::max<int64_t>(1, near / 2); p <= 2 * near; ++p) {
      const int64_t k = (sh.nb * ((groups + p - 1) / p) + 255) / 256;  // workgroups on the fullest CU
      const int64_t cost = k * (10 * p + 1) * (k == 1 ? 21 : 20);
      if (cost < best) {
        best = cost;
        sh.per_wg = p;
      }
    }
  }
  sh.grid_x = (groups + sh.per_wg - 1) / sh.per_wg;
  return sh;
}

int64_t adjoint_partial_floats(int storage, int64_t M, int64_t ncols, int64_t ncols_pad) {
  const bool f32 = storage == PSFLIB_FP32;
  const int64_t nb = adj_shape(f32, M, f32 ? ncols : ncols_pad / 8).nb;
  return nb > 1 ? nb * ncols_pad : 0;
}

hipError_t launch_adjoint(int storage, const void* lib, const Cols16& cx, const float* g,
                          int64_t M, int64_t ncols, int64_t ncols_pad, float* partial, float* out,
                          hipStream_t s) {
  const bool f32 = storage == PSFLIB_FP32;
  const AdjShape sh = adj_shape(f32, M, f32 ? ncols : ncols_pad / 8);
  float* dst = (sh.nb > 1) ? partial : out;
  const int64_t stride = ncols_pad;
  const dim3 grid((unsigned)sh.grid_x, (unsigned)sh.nb);
  if (f32) {
    const float* A = reinterpret_cast<const float*>(lib);
    auto run = [&](auto kern) {
      kern<<<grid, kAdjThreads, sh.lds, s>>>(A, g, dst, M, ncols, sh.block_rows, sh.rounds, sh.per_wg, stride);
    };
    auto pick = [&](auto c) {
      constexpr int C = decltype(c)::value;
      sh.split ? run(adjoint_f32_kernel<C, true>) : run(adjoint_f32_kernel<C, false>);
    };
    switch (sh.c) {
      case 1: pick(std::integral_constant<int, 1>()); break;
      case 2: pick(std::integral_constant<int, 2>()); break;
      case 4: pick(std::integral_constant<int, 4>()); break;
      default: pick(std::integral_constant<int, 8>()); break;
    }
  } else {
    const int64_t ngroups = ncols_pad / 8;
    const u32x4* Mp = reinterpret_cast<const u32x4*>(lib);
    const int apply_exp = (sh.nb > 1) ? 0 : 1;
    auto run = [&](auto kern) {
      kern<<<grid, kAdjThreads, sh.lds, s>>>(Mp, cx.perm, cx.eslot, g, dst, M, ngroups, sh.block_rows,
                                            sh.rounds, sh.per_wg, stride, apply_exp);
    };
    const bool bf = storage == PSFLIB_BF16_POW2;
    auto pick = [&](auto c) {
      constexpr int U = kAdjLoads / decltype(c)::value;
      if (sh.split)
        bf ? run(adjoint_h16_kernel<true, U, true>) : run(adjoint_h16_kernel<false, U, true>);
      else
        bf ? run(adjoint_h16_kernel<true, U, false>) : run(adjoint_h16_kernel<false, U, false>);
    };
    if (sh.c == 1)
      pick(std::integral_constant<int, 1>());
    else
      pick(std::integral_constant<int, 2>());
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || sh.nb == 1) return e;
  reduce_cols_kernel<<<(unsigned)((ncols + 255) / 256), 256, 0, s>>>(
      partial, sh.nb, stride, ncols, f32 ? nullptr : cx.exps, out);
  return hipGetLastError();
}

// ------------------------------------------- allocation-free scratch -----
// Partial sums of psflib_apply_noalloc: a fixed device array on every GPU the
// library runs on, held until the process ends and shared by every such call
// on that GPU.  In host code the array's name is not a device address: the
// address is looked up once per device with hipGetSymbolAddress (that device
// current) and kept, and only that address is passed to kernels.
static __device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float)];

hipError_t noalloc_scratch(int dev, void** ptr) {
  static std::mutex mu;
  static std::map<int, void*> addr;
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(dev);
  if (it != addr.end()) {
    *ptr = it->second;
    return hipSuccess;
  }
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  addr[dev] = p;
  *ptr = p;
  return hipSuccess;
}

// ----------------------------------------------------------- columns ------
template <int STORE>
__global__ __launch_bounds__(256) void get_columns_kernel(const void* __restrict__ lib,
                                                          const int32_t* __restrict__ exps,
                                                          const int32_t* __restrict__ slot_of,
                                                          const int32_t* __restrict__ cols,
                                                          int64_t M, int64_t ncols,
                                                          float* __restrict__ out) {
  const int64_t t = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= M) return;
  const int64_t j = cols[t];
  float v = 0.0f;
  if (j >= 0 && j < ncols) {
    if constexpr (STORE == PSFLIB_FP32) {
      v = reinterpret_cast<const float*>(lib)[j * M + i];
    } else {
      const uint16_t* Mh = reinterpret_cast<const uint16_t*>(lib);
      const int64_t slot = slot_of[j];
      const uint32_t h = Mh[((slot >> 3) * M + i) * 8 + (slot & 7)];
      v = ldexpf(h16_to_f32(h, STORE == PSFLIB_BF16_POW2), exps[j]);
    }
  }
  out[t * M + i] = v;
}

hipError_t launch_get_columns(int storage, const void* lib, const Cols16& cx,
                              const int32_t* cols, int count, int64_t M, int64_t ncols,
                              float* out, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const dim3 grid((unsigned)((M + 255) / 256), (unsigned)count);
  switch (storage) {
    case PSFLIB_FP32:
      get_columns_kernel<PSFLIB_FP32><<<grid, 256, 0, s>>>(lib, cx.exps, cx.slot_of, cols, M, ncols, out);
      break;
    case PSFLIB_BF16_POW2:
      get_columns_kernel<PSFLIB_BF16_POW2><<<grid, 256, 0, s>>>(lib, cx.exps, cx.slot_of, cols, M, ncols, out);
      break;
    default:
      get_columns_kernel<PSFLIB_FP16_POW2><<<grid, 256, 0, s>>>(lib, cx.exps, cx.slot_of, cols, M, ncols, out);
      break;
  }
  return hipGetLastError();
}

// ------------------------------------------------------ column order -----
__global__ __launch_bounds__(256) void identity_order_kernel(int32_t* __restrict__ perm,
                                                             int32_t* __restrict__ eslot,
                                                             int32_t* __restrict__ slot_of,
                                                             const int32_t* __restrict__ exps,
                                                             int64_t ncols, int64_t ncols_pad) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= ncols_pad) return;
  perm[s] = s < ncols ? (int32_t)s : -1;
  eslot[s] = exps[s];
  if (s < ncols) slot_of[s] = (int32_t)s;
}

hipError_t launch_identity_order(int32_t* perm, int32_t* eslot, int32_t* slot_of,
                                 const int32_t* exps, int64_t ncols, int64_t ncols_pad,
                                 hipStream_t s) {
  identity_order_kernel<<<(unsigned)((ncols_pad + 255) / 256), 256, 0, s>>>(perm, eslot, slot_of,
                                                                           exps, ncols, ncols_pad);
  return hipGetLastError();
}

}  // namespace psflib
