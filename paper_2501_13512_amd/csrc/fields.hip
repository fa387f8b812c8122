// Far field of the voxel polarisation (the radiated field of Sec. II's
// current distribution, as used for the RCS comparisons of Sec. III):
//   F(rhat) = (I - rhat rhat) sum_n P_n dV exp(+j k0 rhat . r_n),
// r_n the voxel centre relative to the grid centre; for the face unknowns of
// the rooftop discretisation (`faces`) component c of entry n sits half a
// cell further along axis c, which multiplies component c of the sum by the
// direction's constant exp(+j k0 rhat_c d_c / 2).
//
// The phase factorises over the axes, exp(j k0 (rx px + ry py)) ..., so the
// sum over x of every row (c, z, y) for every direction is a matrix product,
// and only its rows x directions results still need the phase of (y, z).
// With x and its mirror nx - 1 - x taken together,
//   P[x'] e^{j a} + P[x] e^{-j a} = u cos a + j w sin a,  u = P[x'] + P[x],
//   w = P[x'] - P[x],
// the product is real: [u.re, -w.im] and [u.im, w.re] times [cos a; sin a],
// half the operations of the complex one.  It runs on the FP64 matrix
// instructions; cos and sin come from a table per (x, direction).
//
// Few directions, small grids and boxes of one voxel in x leave that product
// mostly padding (192 directions and four pairs of x at a time, three kernels):
// they are summed directly, a sine and cosine per voxel and direction
// (FarShape has the line and both sides).
#include <algorithm>
#include <stdexcept>
#include <string>

#include "krylov_dev.h"

namespace vie {

constexpr int FF_T = 256;          // threads per workgroup
constexpr int FF_ROWS = 16;        // (z, y) rows per workgroup: the matrix instruction's row tile
constexpr int FF_J = 32;           // mirror pairs of x per workgroup
constexpr int FF_NT = 3;           // 16-direction tiles per wavefront
constexpr int FF_DIRS = 4 * FF_NT * 16;   // directions per workgroup
constexpr int FF_LD = 2 * FF_J + 4;       // LDS row of a staged pencil: rows start 8 banks apart
constexpr int FF_PARTS = 512;             // workgroups per direction block, about
constexpr int FF_CHUNK = 2048;            // voxels per workgroup of the direct sum

// Tables and partial sums of the far field that allocates nothing: a fixed
// array of 8 MiB on every GPU the library runs on, held until the process
// ends.  Host code never uses the
// name itself (it is a host-side stand-in there): far_field_scratch_address
// returns the device's own address of its copy.
constexpr int64_t kFarScratchDoubles = int64_t(1) << 20;
static __device__ __align__(256) double scratch[kFarScratchDoubles];

// The phase tables, one row per (table entry, direction):
//   rows [0, jn) and [jn, 2 jn): cos and sin of k0 rx h_j dx, h_j = (nx - 1)/2
//   - j the distance of pair j's members from the grid's centre in cells; 0 in
//   the rows that pad j to jn;
//   then cos and sin of k0 ry y_j (rows 2 jn + 2 y, + 1), then of k0 rz z_j.
__global__ void __launch_bounds__(FF_T) k_far_table(const double* rhat, int ndir, int nx, int ny, int nz, int jn,
                                                    double dx, double dy, double dz, double k0, double* tab) {
  const int i = (int)(blockIdx.x * FF_T + threadIdx.x);
  if (i >= (jn + ny + nz) * ndir) return;
  const int j = i / ndir, dir = i - j * ndir;
  const double* r = rhat + 3 * dir;
  double s = 0.0, c = 0.0;
  if (j < jn) {
    if (2 * j < nx) sincos(k0 * r[0] * ((0.5 * (nx - 1) - j) * dx), &s, &c);
    tab[i] = c;
    tab[(int64_t)jn * ndir + i] = s;
    return;
  }
  const int y = j - jn, z = y - ny;
  if (z < 0)
    sincos(k0 * r[1] * ((y - 0.5 * (ny - 1)) * dy), &s, &c);
  else
    sincos(k0 * r[2] * ((z - 0.5 * (nz - 1)) * dz), &s, &c);
  double* o = tab + (int64_t)(2 * j) * ndir + dir;
  o[0] = c;
  o[ndir] = s;
}

// One workgroup: row tiles of 16 (z, y) rows of the three components, one
// after the other, 32 mirror pairs of x, 192 directions.  The pencils' u and w
// are staged in LDS (real and imaginary result rows as separate row tiles, so
// a lane ends up with both parts of its rows); a wavefront multiplies all six
// row tiles with its 48 directions, applies the phase of (y, z) and adds its
// rows up.  A grid has about FF_PARTS workgroups per direction block (two
// for each compute unit), which bounds the partial sums as well.  Bound by
// the FP64 matrix rate: 128 x 128 x 32 cells and 181 directions take 1.2
// GFLOP, 15 us at that rate; measured 31 us (wavefronts of a workgroup load and
// multiply in turn, two workgroups to a compute unit), 554 us with a sine and
// cosine per voxel and direction.
__global__ void __launch_bounds__(FF_T, 2) k_far_partial(const c128* P, int nx, int ny, int nz, int ndir, int jn,
                                                         int xparts, int per, const double* tab, double* part) {
  typedef double vec4 __attribute__((ext_vector_type(4)));
  __shared__ double a[6][FF_ROWS][FF_LD];
  const int wg = blockIdx.x / xparts, xp = blockIdx.x - wg * xparts;
  const int rows = ny * nz, j0 = xp * FF_J;
  const int jc = min(FF_J, jn - j0);   // pairs staged (a multiple of 4)
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int d0 = blockIdx.y * FF_DIRS + wv * FF_NT * 16;
  int dir[FF_NT];
#pragma unroll
  for (int t = 0; t < FF_NT; ++t) dir[t] = min(d0 + t * 16 + li, ndir - 1);   // past the end: a copy, not stored
  double f[FF_NT][6];
#pragma unroll
  for (int t = 0; t < FF_NT; ++t)
#pragma unroll
    for (int q = 0; q < 6; ++q) f[t][q] = 0.0;
  for (int row0 = wg * per * FF_ROWS; row0 < min((wg + 1) * per * FF_ROWS, rows); row0 += FF_ROWS) {
    double bq[2][FF_NT];
    auto fetch = [&](int k, double* b) {
      const int64_t tr = (int64_t)(k < jc ? j0 + k + lk : jn + j0 + (k - jc) + lk) * ndir;
#pragma unroll
      for (int t = 0; t < FF_NT; ++t) b[t] = tab[tr + dir[t]];
    };
    fetch(0, bq[0]);
    fetch(4, bq[1]);
    __syncthreads();   // the last tile's readers are done
    for (int i = threadIdx.x; i < 3 * FF_ROWS * FF_J; i += FF_T) {
      const int j = i % FF_J, q = i / FF_J, row = q % FF_ROWS, c = q / FF_ROWS;
      if (j >= jc) continue;
      c128 u = mk<double>(0.0, 0.0), w = u;
      const int x = j0 + j, xm = nx - 1 - x;
      if (row0 + row < rows && x <= xm) {
        const c128* p = P + ((int64_t)c * rows + row0 + row) * nx;
        const c128 hi = p[xm], lo = x < xm ? p[x] : u;   // the middle of an odd row stands alone
        u = hi + lo;
        w = hi - lo;
      }
      a[2 * c][row][j] = u.x;
      a[2 * c][row][jc + j] = -w.y;
      a[2 * c + 1][row][j] = u.y;
      a[2 * c + 1][row][jc + j] = w.x;
    }
    __syncthreads();
    if (d0 >= ndir) continue;
    vec4 acc[FF_NT][6];
#pragma unroll
    for (int t = 0; t < FF_NT; ++t)
#pragma unroll
      for (int m = 0; m < 6; ++m) acc[t][m] = vec4{0.0, 0.0, 0.0, 0.0};
    for (int kb = 0; kb < 2 * jc; kb += 8) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = kb + 4 * h;
        double b[FF_NT];
#pragma unroll
        for (int t = 0; t < FF_NT; ++t) b[t] = bq[h][t];
        if (k + 8 < 2 * jc) fetch(k + 8, bq[h]);   // the table two steps ahead
#pragma unroll
        for (int m = 0; m < 6; ++m) {
          const double av = a[m][li][k + lk];
#pragma unroll
          for (int t = 0; t < FF_NT; ++t) acc[t][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b[t], acc[t][m], 0, 0, 0);
        }
      }
    }
    // lane (li, lk) holds rows lk + 4 e of direction li
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = min(row0 + lk + 4 * e, rows - 1), z = row / ny, y = row - z * ny;   // rows past the end are 0
      const double* ty = tab + (int64_t)(2 * (jn + y)) * ndir;
      const double* tz = tab + (int64_t)(2 * (jn + ny + z)) * ndir;
#pragma unroll
      for (int t = 0; t < FF_NT; ++t) {
        const c128 ph = mk<double>(ty[dir[t]], ty[ndir + dir[t]]) * mk<double>(tz[dir[t]], tz[ndir + dir[t]]);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const double re = acc[t][2 * q][e], im = acc[t][2 * q + 1][e];
          f[t][2 * q] += re * ph.x - im * ph.y;
          f[t][2 * q + 1] += re * ph.y + im * ph.x;
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < FF_NT; ++t) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      f[t][q] += __shfl_xor(f[t][q], 16, 64);
      f[t][q] += __shfl_xor(f[t][q], 32, 64);
    }
    if (lk == 0 && d0 + t * 16 + li < ndir) {
      double* o = part + ((int64_t)dir[t] * gridDim.x + blockIdx.x) * 6;
#pragma unroll
      for (int q = 0; q < 6; ++q) o[q] = f[t][q];
    }
  }
}

// The direct sum of one chunk of voxels for one direction.
__global__ void __launch_bounds__(FF_T) k_far_direct(const c128* P, int nx, int ny, int nz, double dx, double dy,
                                                     double dz, double k0, const double* rhat, int nchunk,
                                                     double* part) {
  const int dir = blockIdx.x / nchunk, chunk = blockIdx.x - dir * nchunk;
  const double rx = rhat[3 * dir], ry = rhat[3 * dir + 1], rz = rhat[3 * dir + 2];
  const int64_t nv = (int64_t)nx * ny * nz, xy = (int64_t)nx * ny, v0 = (int64_t)chunk * FF_CHUNK;
  const double cx0 = 0.5 * (nx - 1), cy0 = 0.5 * (ny - 1), cz0 = 0.5 * (nz - 1);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int64_t v = v0 + threadIdx.x; v < v0 + FF_CHUNK && v < nv; v += FF_T) {
    const int z = (int)(v / xy);
    const int64_t r = v - (int64_t)z * xy;
    const int y = (int)(r / nx), x = (int)(r - (int64_t)y * nx);
    double s, c;
    sincos(k0 * (rx * ((x - cx0) * dx) + ry * ((y - cy0) * dy) + rz * ((z - cz0) * dz)), &s, &c);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const c128 p = P[q * nv + v];
      acc[2 * q] += p.x * c - p.y * s;
      acc[2 * q + 1] += p.x * s + p.y * c;
    }
  }
  block_sum<6>(acc);
  if (threadIdx.x == 0) {
    double* o = part + ((int64_t)dir * nchunk + chunk) * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) o[k] = acc[k];
  }
}

template <bool FACES>
__global__ void __launch_bounds__(FF_T) k_far_final(const double* part, int nchunk, const double* rhat, double dx,
                                                    double dy, double dz, double k0, c128* F) {
  const int dir = blockIdx.x;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int c = threadIdx.x; c < nchunk; c += FF_T) {
    const double* p = part + ((int64_t)dir * nchunk + c) * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] += p[k];
  }
  block_sum<6>(acc);
  if (threadIdx.x == 0) {
    const double r[3] = {rhat[3 * dir], rhat[3 * dir + 1], rhat[3 * dir + 2]};
    const double dV = dx * dy * dz, d[3] = {dx, dy, dz};
    double fr[3], fi[3];
    for (int q = 0; q < 3; ++q) {
      double hs = 0.0, hc = 1.0;   // half-cell phase of the component
      if constexpr (FACES) sincos(0.5 * k0 * r[q] * d[q], &hs, &hc);
      fr[q] = (acc[2 * q] * hc - acc[2 * q + 1] * hs) * dV;
      fi[q] = (acc[2 * q] * hs + acc[2 * q + 1] * hc) * dV;
    }
    const double dr = r[0] * fr[0] + r[1] * fr[1] + r[2] * fr[2];
    const double di = r[0] * fi[0] + r[1] * fi[1] + r[2] * fi[2];
    for (int q = 0; q < 3; ++q) F[3 * dir + q] = mk<double>(fr[q] - r[q] * dr, fi[q] - r[q] * di);
  }
}

// The split of one grid and direction count: padded mirror pairs, x parts, row
// tiles and workgroups per direction block, or the direct sum's chunks; doubles
// of scratch per direction.
//
// The direct sum is taken where it is faster, by what the two were measured to
// take (us, on an idle GPU; rounds of 512 workgroups, and what the other
// wavefronts of a direction block add to the first).  Direct / product:
//   5x4x6        1 direction 9.6 / 12.3; 361 10.3 / 15.3
//   16x16x16     1 12.9 / 14.3; 181 15.5 / 15.9; 361 19.8 / 16.7
//   32x32x32     1 13.1 / 16.6; 32 15.7 / 16.8; 48 19.0 / 17.1
//   64x64x64     1 13.6 / 21.4; 8 21.5 / 21.7; 16 32.6 / 21.8
//   128x128x32   1 13.7 / 22.4; 4 20.9 / 22.6; 8 32.4 / 22.9
//   256x256x64   1 41 / 136; 4 125 / 136; 8 236 / 137
//   1x256x256    1 13.5 / 48.1; 128 53.3 / 59.3; 181 72.0 / 66.0; 361 136 / 173
//   2x200x200    1 13.6 / 35.5; 64 38.1 / 40.7; 96 51.7 / 41.1; 361 164 / 128
struct FarShape {
  int jn, xparts, per, parts;
  bool direct;
  int64_t scratch;
  FarShape(int nx, int ny, int nz, int ndir) {
    jn = ((nx + 1) / 2 + 3) / 4 * 4;
    xparts = (jn + FF_J - 1) / FF_J;
    const int64_t tiles = ((int64_t)ny * nz + FF_ROWS - 1) / FF_ROWS;
    per = (int)((tiles * xparts + FF_PARTS - 1) / FF_PARTS);
    parts = (int)((tiles + per - 1) / per) * xparts;
    const int64_t nv = (int64_t)nx * ny * nz, chunks = (nv + FF_CHUNK - 1) / FF_CHUNK;
    const double waves = (ndir + FF_NT * 16 - 1) / (FF_NT * 16);
    const double many = waves <= 4 ? 1 + (waves - 1) / 6 : 1.5 + 0.75 * (waves - 4);
    const double t_product = 11.5 + (0.36 * std::min(jn, FF_J) * per + 4.2 * (per - 1)) * many;
    const double t_direct = 11.0 + (nv < int64_t(1) << 21 ? 0.011 : 0.0138) * (double)(ndir * chunks);
    direct = t_direct < t_product;
    if (direct) parts = (int)chunks;
    scratch = (direct ? 0 : 2 * ((int64_t)jn + ny + nz)) + 6 * (int64_t)parts;
  }
};

int64_t far_field_scratch(int nx, int ny, int nz, int ndir) {
  return std::min<int64_t>(ndir * FarShape(nx, ny, nz, ndir).scratch, kFarScratchDoubles);
}

int64_t far_field_scratch_doubles() { return kFarScratchDoubles; }

void* far_field_scratch_address() {
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr)
    throw std::runtime_error(std::string("far-field scratch address: ") + hipGetErrorString(e));
  return ptr;
}

void far_field(const c128* P, int nx, int ny, int nz, double dx, double dy, double dz, double k0, const double* rhat,
               int ndir, double* part, c128* F, hipStream_t s, bool faces) {
  if (ndir <= 0) return;
  const FarShape f(nx, ny, nz, ndir);
  // as many directions at a time as the scratch holds (a direction's result
  // does not depend on the others taken with it)
  const int most = (int)std::min<int64_t>(kFarScratchDoubles / f.scratch, 65535 * (int64_t)FF_DIRS);
  if (most < 1) throw std::runtime_error("far field: grid too large for its scratch");
  const int tr = f.jn + ny + nz;
  for (int d = 0; d < ndir; d += most) {
    const int n = std::min(most, ndir - d);
    const double* rd = rhat + 3 * (int64_t)d;
    double* sums = part;
    if (f.direct) {
      hipLaunchKernelGGL(k_far_direct, dim3((unsigned)(n * f.parts)), dim3(FF_T), 0, s, P, nx, ny, nz, dx, dy, dz, k0, rd,
                         f.parts, sums);
    } else {
      sums += 2 * (int64_t)tr * n;
      hipLaunchKernelGGL(k_far_table, dim3((unsigned)(((int64_t)tr * n + FF_T - 1) / FF_T)), dim3(FF_T), 0, s, rd, n, nx,
                         ny, nz, f.jn, dx, dy, dz, k0, part);
      hipLaunchKernelGGL(k_far_partial, dim3((unsigned)f.parts, (unsigned)((n + FF_DIRS - 1) / FF_DIRS)), dim3(FF_T), 0, s,
                         P, nx, ny, nz, n, f.jn, f.xparts, f.per, part, sums);
    }
    const auto final_kernel = faces ? k_far_final<true> : k_far_final<false>;
    hipLaunchKernelGGL(final_kernel, dim3(n), dim3(FF_T), 0, s, sums, f.parts, rd, dx, dy, dz, k0, F + 3 * (int64_t)d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw std::runtime_error(std::string("far field launch: ") + hipGetErrorString(e));
  }
}

}  // namespace vie
