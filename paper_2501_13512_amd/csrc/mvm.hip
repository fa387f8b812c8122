// FFT-accelerated product with the discretised VIE operator, and the setup of
// the Green-tensor spectra.
//
// Operator (eqs. (2)-(4) and (6) of the paper, unknown P = J/(j omega eps0)):
//   (A x)_m = x_m / chi_m - sum_n T(m - n) x_n   on the scatterer voxels,
//   (A x)_m = 0                                   on vacuum voxels.
// The sum is a 3-D convolution with the block-Toeplitz kernel T (Sec. I),
// done as a circulant convolution on a (lx, ly, lz) grid with L >= 2n - 1 per
// axis, in five passes over HBM:
//   1. x forward, pruned: rows of nx voxels, zero-padded to lx;
//   2. y forward, pruned: only the nz non-zero z-planes exist;
//   3. z forward + 3x3 symmetric spectral multiply + z inverse, fused in one
//      workgroup per (y-fold, tile of x-folds): the four mirror columns
//      (+-qx, +-qy) of the three components sit in LDS together, so each
//      value of the octant spectrum (q in [0, L/2]^3, parity signs for the
//      odd components: T_xy is odd in x and y, ...) is read once;
//   4. y inverse, cropped to ny rows;
//   5. x inverse, cropped to nx, scaled by 1/(lx ly lz), fused with the
//      local term and the vacuum mask, written as c128.
#include <cmath>
#include <stdexcept>
#include <string>

#include "api_lock.h"
#include "fft_core.h"
#include "krylov_dev.h"
#include "zpass.h"

namespace vie {

int smallest_fft_length(int min_len, bool xy) {
  for (int L : kFftLengths)
    if (L >= min_len && !(xy && L == 36)) return L;
  return -1;
}

// ------------------------------------------------------------------ geometry
template <typename R, int L>
struct Geo {
  static constexpr int T = PlanInfo<L>::max_butterflies;  // threads per pencil
  static constexpr int ES = (int)sizeof(cx<R>);
  // rows (contiguous pencils): ~256 threads, LDS [ROWP][L]
  static constexpr int ROWP = cmax(1, cmin(256 / T, (64 * 1024) / (L * ES)));
  // twiddles held over a row (column) transform: not where their registers cost
  // a wavefront or more (rows of 192x40x96, FP32: 22.6 us without, 30.7 with;
  // columns of 40x192x96: 29.3, 35.3; FP64 columns of 40x72x96: 24.9, 26.6)
  static constexpr bool HOLD = sizeof(R) == 8 || L != 384;
  static constexpr bool HOLD_COL = HOLD && L != 144;
  // pass 5 asks for its vectors before the transform
  static constexpr bool EARLY = HOLD && (sizeof(R) == 4 || L < 72 || L == 256);
  static constexpr int RAD0 = RadInfo<typename Plan<L>::type>::first;
  using RS = RowSlot<RAD0>;                                  // rows with gaps against bank conflicts
  static constexpr int ROWL = RAD0 > 1 ? L + L / RAD0 : L;
  // columns (strided pencils), LDS [L][COLP]: at least 128 contiguous bytes
  // per row of the tile (one full cache line) when 64 KB of LDS allow it,
  // with TC <= T threads per column (several butterflies per thread when
  // T * COLP would exceed 1024 threads)
  static constexpr int LDS_COLS = cmax(1, (64 * 1024) / (L * ES));
  static constexpr int COLP = cmax(1, pow2_floor(cmin(LDS_COLS, cmax(128 / ES, cmin(cmax(16, 256 / T), 512 / T)))));
  static constexpr int TC = cmin(T, cmax(1, 1024 / COLP));
};

// n / d by one multiply-high: m = ceil(2^32 / d) for d >= 2, m = 0 for d = 1.
// With n = q d + r, n m / 2^32 = n / d + n (m - 2^32 / d) / 2^32 and the
// second term is below n / 2^32, so the floor is q whenever n d < 2^32.
// The plane kernels' element, row and plane indices stay far inside that
// range (checked when they are launched).
inline unsigned div_magic(int d) { return d <= 1 ? 0u : (unsigned)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d); }
__device__ __forceinline__ unsigned udiv_m(unsigned n, unsigned m) { return m ? __umulhi(n, m) : n; }

// ------------------------------------------------------------------ kernels
template <typename R>
struct RowArgs {
  int nx, ny, nz, lx, ly;
  int64_t vstride, cstride, wstride;
  const c128* x;
  c128* y;
  const c128* chi_inv;
  cx<R>* work;
  const int* status;
  const cx<R>* tw;
  int mask_input;
  int chi3;   // 1/chi per component ([3][nz][ny][nx]: rooftop faces) instead of per voxel
  // division constants of the plane kernels (udiv_m): nx ny, nx, ny, nz
  unsigned m_pe, m_nx, m_ny, m_nz;
  double scale;
  // BiCGSTAB work fused into pass 1 (in_mode) and pass 5 (out_mode)
  int in_mode, out_mode;
  const c128* r;
  c128* p;
  const c128* v;
  const c128* rhat;
  const c128* s;
  KBatch k;
};

// Pass 1: x forward with zero padding nx -> lx, c128 -> R.  With a fused
// BiCGSTAB update (in_mode 1: p, in_mode 2: s) the new vector is formed in a
// pre-pass that issues all loads of a chunk of elements before storing it to
// HBM and to the pencil's LDS slot; the transform then starts from LDS.
template <typename R, int L>
__global__ void __launch_bounds__((Geo<R, L>::T * Geo<R, L>::ROWP)) k_row_fwd(RowArgs<R> a) {
  using G = Geo<R, L>;
  using RS = typename G::RS;
  constexpr int T = G::T;
  __shared__ cx<R> lds[G::ROWP * G::ROWL];
  const int rows = 3 * a.nz * a.ny;
  const int tiles = (rows + G::ROWP - 1) / G::ROWP;
  const int sys = blockIdx.x / tiles, tile = blockIdx.x - sys * tiles;
  if (!sys_active(a.status, sys)) return;
  const int p = threadIdx.x / T, t = threadIdx.x - p * T;
  const int row = tile * G::ROWP + p;
  const bool valid = row < rows;
  const int rr = valid ? row : 0;
  const int c = rr / (a.nz * a.ny), zy = rr - c * (a.nz * a.ny);
  const int z = zy / a.ny, yy = zy - z * a.ny;
  const int64_t vrow = sys * a.vstride + (int64_t)rr * a.nx;
  cx<R>* w = a.work + sys * a.wstride + ((int64_t)(c * a.nz + z) * a.ly + yy) * a.lx;
  cx<R>* slot = lds + p * G::ROWL;
  const int nx = a.nx;
  const int mode = a.in_mode;
  const TwRegs<R, L, T, G::HOLD> tw(a.tw, t);
  auto st = [&](int k, cx<R> v) { w[k] = v; };
  if (mode == 0) {
    // nothing in the loaders uses a loaded value under its bounds check, so a
    // thread's loads are all in flight together
    const c128* xin = a.x + vrow;
    if (a.mask_input) {
      const c128* chi = a.chi_inv + sys * a.cstride + (int64_t)(a.chi3 ? rr : zy) * nx;
      auto ld = [&](int n) -> cx<R> {
        c128 v = mk<double>(0.0, 0.0), ci = v;
        if (n < nx) {
          v = xin[n];
          ci = chi[n];
        }
        const bool off = ci.x == 0.0 && ci.y == 0.0;
        return cvt<R>(mk<double>(off ? 0.0 : v.x, off ? 0.0 : v.y));
      };
      fft_pencil<R, L, T, -1, false, false, PAD_IN>(ld, st, slot, RS(), t, valid, tw);
    } else {
      auto ld = [&](int n) -> cx<R> {
        c128 v = mk<double>(0.0, 0.0);
        if (n < nx) v = xin[n];
        return cvt<R>(v);
      };
      fft_pencil<R, L, T, -1, false, false, PAD_IN>(ld, st, slot, RS(), t, valid, tw);
    }
    return;
  }
  const KState& ks = a.k.st[sys];
  const bool first = mode == 1 && ks.iters == 0;
  double acc = 0.0;
  constexpr int LH = PadIn<L>::reads;   // elements that the transform reads
  constexpr int E = (LH + T - 1) / T;   // per thread
  constexpr int CH = 4;                // elements per load batch
  c128 rv[CH], pv[CH], vv[CH];
  auto load = [&](int j0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int n = t + (j0 + u) * T;
      if (valid && j0 + u < E && n < nx) {
        rv[u] = a.r[vrow + n];
        if (!first) vv[u] = a.v[vrow + n];
        if (mode == 1 && !first) pv[u] = a.p[vrow + n];
      }
    }
  };
  load(0);   // in flight while alpha is formed
  c128 c1;
  if (mode == 3) {   // alpha from the last product's partials (FIN_ALPHA fused)
    if (!fused_alpha(a.k, sys, tile == 0, &c1)) return;
  } else {
    c1 = mode == 1 ? ks.beta : ks.alpha;
  }
  const c128 c2 = ks.omega;
#pragma unroll
  for (int j0 = 0; j0 < E; j0 += CH) {
    if (j0 > 0) load(j0);
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int n = t + (j0 + u) * T;
      if (valid && j0 + u < E && n < LH) {
        if (n < nx) {
          c128 val;
          if (mode == 1)
            val = first ? rv[u] : rv[u] + c1 * (pv[u] - c2 * vv[u]);   // p = r + beta (p - omega v)
          else
            val = rv[u] - c1 * vv[u];                                    // s = r - alpha v
          a.p[vrow + n] = val;
          slot[slot_at(RS(), n)] = cvt<R>(val);
          acc += abs2(val);
        } else {
          slot[slot_at(RS(), n)] = czero<R>();
        }
      }
    }
  }
  __syncthreads();
  auto ld = [&](int n) -> cx<R> { return slot[slot_at(RS(), n)]; };
  fft_pencil<R, L, T, -1, true, false, PAD_IN>(ld, st, slot, RS(), t, valid, tw);
  if (mode == 2) {
    double sum[1] = {acc};
    write_partial<1>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  }
}

// Pass 5: x inverse, crop lx -> nx, y = x/chi - scale * Q on the mask, 0 off
// it.  The cropped transform lands in LDS; a post-pass issues the loads of
// 1/chi, x and (fused inner products) rhat or s for a chunk of elements
// before storing y.
template <typename R, int L>
__global__ void __launch_bounds__((Geo<R, L>::T * Geo<R, L>::ROWP)) k_row_inv_local(RowArgs<R> a) {
  using G = Geo<R, L>;
  using RS = typename G::RS;
  constexpr int T = G::T;
  __shared__ cx<R> lds[G::ROWP * G::ROWL];
  const int rows = 3 * a.nz * a.ny;
  const int tiles = (rows + G::ROWP - 1) / G::ROWP;
  const int sys = blockIdx.x / tiles, tile = blockIdx.x - sys * tiles;
  if (!sys_active(a.status, sys)) return;
  const int p = threadIdx.x / T, t = threadIdx.x - p * T;
  const int row = tile * G::ROWP + p;
  const bool valid = row < rows;
  const int rr = valid ? row : 0;
  const int c = rr / (a.nz * a.ny), zy = rr - c * (a.nz * a.ny);
  const int z = zy / a.ny, yy = zy - z * a.ny;
  const int64_t vrow = sys * a.vstride + (int64_t)rr * a.nx;
  const c128* chi = a.chi_inv + sys * a.cstride + (int64_t)(a.chi3 ? rr : zy) * a.nx;
  const cx<R>* w = a.work + sys * a.wstride + ((int64_t)(c * a.nz + z) * a.ly + yy) * a.lx;
  cx<R>* slot = lds + p * G::ROWL;
  const int nx = a.nx;
  auto ld = [&](int n) -> cx<R> { return w[n]; };
  auto sts = [&](int k, cx<R> v) {
    if (k < nx) slot[slot_at(RS(), k)] = v;
  };
  const double scale = a.scale;
  const int mode = a.out_mode;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  constexpr int E = (half_padded(L) + T - 1) / T;
  constexpr int CH = 4;
  c128 ci[CH], xv[CH], ov[CH];
  auto load = [&](int j0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int k = t + (j0 + u) * T;
      if (valid && j0 + u < E && k < nx) {
        ci[u] = chi[k];
        xv[u] = a.x[vrow + k];
        if (mode == 1 || mode == 3) ov[u] = a.rhat[vrow + k];
        if (mode == 2 || mode == 4) ov[u] = a.s[vrow + k];
      }
    }
  };
  const TwRegs<R, L, T, G::HOLD> tw(a.tw, t);
  constexpr bool EARLY = G::EARLY && E <= 2 * CH;   // the operands in flight during the transform, where it holds few values
  if (EARLY) load(0);
  fft_pencil<R, L, T, +1, false, true, PAD_OUT>(ld, sts, slot, RS(), t, valid, tw);

#pragma unroll
  for (int j0 = 0; j0 < E; j0 += CH) {
    if (!EARLY || j0 > 0) load(j0);
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int k = t + (j0 + u) * T;
      if (valid && j0 + u < E && k < nx) {
        c128 out = mk<double>(0.0, 0.0);
        if (mode == 3)   // field at every voxel: E_inc + sum T P
          out = ov[u] + scale * cvt<double>(slot[slot_at(RS(), k)]);
        else if (ci[u].x != 0.0 || ci[u].y != 0.0)
          out = xv[u] * ci[u] - scale * cvt<double>(slot[slot_at(RS(), k)]);
        a.y[vrow + k] = out;
        if (mode == 1) {          // <rhat, y>
          const c128 d = cdot1(ov[u], out);
          acc[0] += d.x;
          acc[1] += d.y;
        } else if (mode == 2 || mode == 4) {   // <y, s>, <y, y> (and ||s||^2)
          const c128 d = cdot1(out, ov[u]);
          acc[0] += d.x;
          acc[1] += d.y;
          acc[2] += abs2(out);
          if (mode == 4) acc[3] += abs2(ov[u]);
        }
      }
    }
  }
  if (mode == 1) {
    double sum[2] = {acc[0], acc[1]};
    write_partial<2>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  } else if (mode == 2) {
    double sum[3] = {acc[0], acc[1], acc[2]};
    write_partial<3>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  } else if (mode == 4) {
    write_partial<4>(acc, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  }
}

// ------------------------------------------------------------------ plane passes
// Square transforms (lx = ly <= 128, plane_supported): the x and y transforms of a
// z-plane run in one kernel with the plane in LDS, so passes 1 + 2 become
// k_plane_fwd and passes 4 + 5 become k_plane_inv_local (one launch and one
// trip through HBM fewer each way; same BiCGSTAB fusion as the row kernels).
// A workgroup takes NPL consecutive planes (c, z) of one system; LDS holds
// them as [NPL][L][L + 1] (rows padded against bank conflicts on columns).
// Variant PV sets NPL: 0 as many planes as 48 KB of LDS hold (at most 16),
// 1 at most two (from 48 on one plane with twice the threads), 2 one plane.
// From 96 on every variant is one plane by 1024 threads, the CU's LDS holding
// no second FP64 one.  Fewer planes per workgroup mean more, shorter workgroups: the product's latency falls when few systems are active (two
// 32 x 32 planes of a 16 x 16 box take 3 transform rounds of 32 pencils
// where five planes take 8), at the cost of more workgroups to dispatch.
template <typename R, int L, int PV>
struct PlaneGeo {
  static constexpr int ES = (int)sizeof(cx<R>);
  static constexpr int LP = L + 1;
  static constexpr bool FITS = L * LP * ES <= 150 * 1024;
  static constexpr int NPL_LDS = cmax(1, cmin(16, (48 * 1024) / (L * LP * ES)));
  static constexpr int NPL = PV == 0 ? NPL_LDS : (PV == 1 && L < 48 ? cmin(2, NPL_LDS) : 1);
  static constexpr int BT = L > 64 ? 1024 : (PV == 1 && L >= 48 ? 512 : 256);
  static constexpr int T = PlanInfo<L>::max_butterflies;
  static constexpr int PP = BT / T;
  // where 256 threads take all rows at once, pencils go to sets of 256 in
  // turn: the row phase then leaves whole wavefronts idle, not half the lanes
  // of each
  static constexpr int SET = L / 2 * T <= 256 ? cmin(BT, 256) : BT;
  static constexpr int SP = SET / T;
  static __device__ __forceinline__ int pencil() { return threadIdx.x % SP + threadIdx.x / SET * SP; }
  static __device__ __forceinline__ int place() { return threadIdx.x % SET / SP; }
  static_assert(BT % T == 0, "pencil threads must divide the workgroup");
};

template <typename R, int L, int PV>
__global__ void __launch_bounds__((PlaneGeo<R, L, PV>::BT)) k_plane_fwd(RowArgs<R> a) {
  using G = PlaneGeo<R, L, PV>;
  constexpr int T = G::T, PP = G::PP, LP = G::LP, NPL = G::NPL, BT = G::BT;
  __shared__ cx<R> lds[NPL * L * LP];
  const int planes = 3 * a.nz;
  const int tiles = (planes + NPL - 1) / NPL;
  const int sys = blockIdx.x / tiles, tile = blockIdx.x - sys * tiles;
  if (!sys_active(a.status, sys)) return;
  const int pl0 = tile * NPL, npl = min(NPL, planes - pl0);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int pe = ny * nx;
  const int ne = npl * pe;
  const int64_t v0 = sys * a.vstride + (int64_t)pl0 * pe;
  const int mode = a.in_mode;
  double acc = 0.0;
  const TwRegs<R, L, T> tw(a.tw, G::place());
  // zero the padding columns that the transform reads, of rows y < ny
  const int padw = PadIn<L>::reads - nx;
  for (int e = threadIdx.x; e < npl * ny * padw; e += BT) {
    const int row = e / padw, xx = nx + (e - row * padw);
    const int q = (int)udiv_m((unsigned)row, a.m_ny);
    lds[q * L * LP + (row - q * ny) * LP + xx] = czero<R>();
  }
  auto lds_at = [&](int e) -> cx<R>* {
    const int q = (int)udiv_m((unsigned)e, a.m_pe), rem = e - q * pe, y = (int)udiv_m((unsigned)rem, a.m_nx);
    return lds + (q * L + y) * LP + (rem - y * nx);
  };
  if (mode == 0) {
    const c128* chi = a.chi_inv + sys * a.cstride;
    const bool msk = a.mask_input != 0;
    constexpr int CH = 4;
    for (int e0 = 0; e0 < ne; e0 += CH * BT) {
      c128 v[CH], ci[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int e = e0 + u * BT + (int)threadIdx.x;
        ci[u] = mk<double>(1.0, 0.0);
        if (e < ne) {
          v[u] = a.x[v0 + e];
          if (msk) {
            const int q = (int)udiv_m((unsigned)e, a.m_pe);
            const int zq = pl0 + q;
            const int z = a.chi3 ? zq : zq - nz * (int)udiv_m((unsigned)zq, a.m_nz);
            ci[u] = chi[(int64_t)z * pe + (e - q * pe)];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int e = e0 + u * BT + (int)threadIdx.x;
        if (e < ne) {
          const bool off = ci[u].x == 0.0 && ci[u].y == 0.0;
          *lds_at(e) = cvt<R>(mk<double>(off ? 0.0 : v[u].x, off ? 0.0 : v[u].y));
        }
      }
    }
  } else {
    const KState& ks = a.k.st[sys];
    const bool first = mode == 1 && ks.iters == 0;
    constexpr int CH = 4;
    c128 rv[CH], pv[CH], vv[CH];
    auto load = [&](int e0) {
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int e = e0 + u * BT + (int)threadIdx.x;
        if (e < ne) {
          rv[u] = a.r[v0 + e];
          if (!first) vv[u] = a.v[v0 + e];
          if (mode == 1 && !first) pv[u] = a.p[v0 + e];
        }
      }
    };
    load(0);   // in flight while alpha is formed
    c128 c1;
    if (mode == 3) {   // alpha from the last product's partials (FIN_ALPHA fused)
      if (!fused_alpha(a.k, sys, tile == 0, &c1)) return;
    } else {
      c1 = mode == 1 ? ks.beta : ks.alpha;
    }
    const c128 c2 = ks.omega;
    for (int e0 = 0; e0 < ne; e0 += CH * BT) {
      if (e0 > 0) load(e0);
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int e = e0 + u * BT + (int)threadIdx.x;
        if (e < ne) {
          c128 val;
          if (mode == 1)
            val = first ? rv[u] : rv[u] + c1 * (pv[u] - c2 * vv[u]);   // p = r + beta (p - omega v)
          else
            val = rv[u] - c1 * vv[u];                                    // s = r - alpha v
          a.p[v0 + e] = val;
          *lds_at(e) = cvt<R>(val);
          acc += abs2(val);
        }
      }
    }
  }
  __syncthreads();
  // x transforms of the rows y < ny, in place.  Consecutive lanes take
  // consecutive rows (a row's threads are PP lanes apart), so the threads
  // that a stage with fewer butterflies leaves idle form whole wavefronts,
  // which skip it; the row stride LP keeps the lanes' LDS banks distinct.
  {
    const int p = G::pencil(), t = G::place();
    const int nrows = npl * ny;
    for (int r0 = 0; r0 < nrows; r0 += PP) {
      const int row = r0 + p;
      const bool valid = p < PP && row < nrows;
      const int rr = valid ? row : 0;
      const int rq = (int)udiv_m((unsigned)rr, a.m_ny);
      cx<R>* slot = lds + (rq * L + (rr - rq * ny)) * LP;
      auto ld = [&](int n) -> cx<R> { return slot[n]; };
      auto st = [&](int k, cx<R> v) { slot[k] = v; };
      fft_pencil<R, L, T, -1, true, true, PAD_IN>(ld, st, slot, 1, t, valid, tw);
    }
  }
  // y transforms of the L columns (rows >= ny are zero), out to HBM
  {
    const int p = G::pencil(), t = G::place();
    const int ncols = npl * L;
    cx<R>* w = a.work + sys * a.wstride + (int64_t)pl0 * L * L;
    for (int c0 = 0; c0 < ncols; c0 += PP) {
      const int col = c0 + p;
      const bool valid = t < T && col < ncols;
      const int cc = valid ? col : 0;
      const int q = cc / L, xq = cc - q * L;
      cx<R>* slot = lds + q * L * LP + xq;
      cx<R>* wc = w + (int64_t)q * L * L + xq;
      auto ld = [&](int n) -> cx<R> { return n < ny ? slot[n * LP] : czero<R>(); };
      auto st = [&](int k, cx<R> v) { wc[k * L] = v; };
      fft_pencil<R, L, T, -1, true, false, PAD_IN>(ld, st, slot, LP, t, valid, tw);
    }
  }
  if (mode == 2) {
    double sum[1] = {acc};
    write_partial<1>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  }
}

template <typename R, int L, int PV>
__global__ void __launch_bounds__((PlaneGeo<R, L, PV>::BT)) k_plane_inv_local(RowArgs<R> a) {
  using G = PlaneGeo<R, L, PV>;
  constexpr int T = G::T, PP = G::PP, LP = G::LP, NPL = G::NPL, BT = G::BT;
  __shared__ cx<R> lds[NPL * L * LP];
  const int planes = 3 * a.nz;
  const int tiles = (planes + NPL - 1) / NPL;
  const int sys = blockIdx.x / tiles, tile = blockIdx.x - sys * tiles;
  if (!sys_active(a.status, sys)) return;
  const int pl0 = tile * NPL, npl = min(NPL, planes - pl0);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int pe = ny * nx;
  const int ne = npl * pe;
  const int64_t v0 = sys * a.vstride + (int64_t)pl0 * pe;
  const double scale = a.scale;
  const int mode = a.out_mode;
  const c128* chi = a.chi_inv + sys * a.cstride;
  constexpr int CH = 4;
  c128 ci[CH], xv[CH], ov[CH];
  auto load = [&](int e0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int e = e0 + u * BT + (int)threadIdx.x;
      if (e < ne) {
        const int q = (int)udiv_m((unsigned)e, a.m_pe), zq = pl0 + q;
        ci[u] = chi[(int64_t)(a.chi3 ? zq : zq - nz * (int)udiv_m((unsigned)zq, a.m_nz)) * pe + (e - q * pe)];
        xv[u] = a.x[v0 + e];
        if (mode == 1 || mode == 3) ov[u] = a.rhat[v0 + e];
        if (mode == 2 || mode == 4) ov[u] = a.s[v0 + e];
      }
    }
  };
  const TwRegs<R, L, T> tw(a.tw, G::place());
  load(0);   // in flight during the transforms
  // y inverse of the L columns from HBM, rows k < ny kept in LDS
  {
    const int p = G::pencil(), t = G::place();
    const int ncols = npl * L;
    const cx<R>* w = a.work + sys * a.wstride + (int64_t)pl0 * L * L;
    for (int c0 = 0; c0 < ncols; c0 += PP) {
      const int col = c0 + p;
      const bool valid = t < T && col < ncols;
      const int cc = valid ? col : 0;
      const int q = cc / L, xq = cc - q * L;
      cx<R>* slot = lds + q * L * LP + xq;
      const cx<R>* wc = w + (int64_t)q * L * L + xq;
      auto ld = [&](int n) -> cx<R> { return wc[n * L]; };
      auto st = [&](int k, cx<R> v) {
        if (k < ny) slot[k * LP] = v;
      };
      fft_pencil<R, L, T, +1, false, true, PAD_OUT>(ld, st, slot, LP, t, valid, tw);
    }
  }
  // x inverse of the rows y < ny, in place, cropped to nx (lanes over rows
  // as in the forward kernel)
  {
    const int p = G::pencil(), t = G::place();
    const int nrows = npl * ny;
    for (int r0 = 0; r0 < nrows; r0 += PP) {
      const int row = r0 + p;
      const bool valid = p < PP && row < nrows;
      const int rr = valid ? row : 0;
      const int rq = (int)udiv_m((unsigned)rr, a.m_ny);
      cx<R>* slot = lds + (rq * L + (rr - rq * ny)) * LP;
      auto ld = [&](int n) -> cx<R> { return slot[n]; };
      auto st = [&](int k, cx<R> v) {
        if (k < nx) slot[k] = v;
      };
      fft_pencil<R, L, T, +1, true, true, PAD_OUT>(ld, st, slot, 1, t, valid, tw);
    }
  }
  // y = x/chi - scale Q on the mask, fused inner products
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int e0 = 0; e0 < ne; e0 += CH * BT) {
    if (e0 > 0) load(e0);
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int e = e0 + u * BT + (int)threadIdx.x;
      if (e < ne) {
        const int q = (int)udiv_m((unsigned)e, a.m_pe), rem = e - q * pe, y = (int)udiv_m((unsigned)rem, a.m_nx);
        const cx<R> qv = lds[(q * L + y) * LP + (rem - y * nx)];
        c128 out = mk<double>(0.0, 0.0);
        if (mode == 3)   // field at every voxel: E_inc + sum T P
          out = ov[u] + scale * cvt<double>(qv);
        else if (ci[u].x != 0.0 || ci[u].y != 0.0)
          out = xv[u] * ci[u] - scale * cvt<double>(qv);
        a.y[v0 + e] = out;
        if (mode == 1) {          // <rhat, y>
          const c128 d = cdot1(ov[u], out);
          acc[0] += d.x;
          acc[1] += d.y;
        } else if (mode == 2 || mode == 4) {   // <y, s>, <y, y> (and ||s||^2)
          const c128 d = cdot1(out, ov[u]);
          acc[0] += d.x;
          acc[1] += d.y;
          acc[2] += abs2(out);
          if (mode == 4) acc[3] += abs2(ov[u]);
        }
      }
    }
  }
  if (mode == 1) {
    double sum[2] = {acc[0], acc[1]};
    write_partial<2>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  } else if (mode == 2) {
    double sum[3] = {acc[0], acc[1], acc[2]};
    write_partial<3>(sum, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  } else if (mode == 4) {
    write_partial<4>(acc, a.k.partials, a.k.pstride, a.k.ntile, sys, tile, tiles);
  }
}

// In-place FFT of full-length rows (spectra setup).
template <typename R, int L>
__global__ void __launch_bounds__((Geo<R, L>::T * Geo<R, L>::ROWP)) k_row_full(cx<R>* data, int64_t rows,
                                                                           const cx<R>* tw) {
  using G = Geo<R, L>;
  __shared__ cx<R> lds[G::ROWP * G::ROWL];
  const int p = threadIdx.x / G::T, t = threadIdx.x - p * G::T;
  const int64_t row = (int64_t)blockIdx.x * G::ROWP + p;
  const bool valid = row < rows;
  cx<R>* d = data + (valid ? row : 0) * L;
  auto ld = [&](int n) -> cx<R> { return d[n]; };
  auto st = [&](int k, cx<R> v) { d[k] = v; };
  fft_pencil<R, L, G::T, -1>(ld, st, lds + p * G::ROWL, typename G::RS(), t, valid, tw);
}

// Strided pencils, in place: per system, data[outer][L][inner]; element n of
// column (o, i) at o*L*inner + n*inner + i.  Reads n < n_in (zero beyond),
// writes k < n_out.  Passes 2 and 4, and the y/z passes of the setup.
template <typename R>
struct ColArgs {
  cx<R>* data;
  int outer, inner, n_in, n_out;
  int64_t stride;
  const int* status;
  const cx<R>* tw;
  int nsys;
};

template <typename R, int L, int DIR, int PAD>
__global__ void __launch_bounds__((Geo<R, L>::TC * Geo<R, L>::COLP)) k_col(ColArgs<R> a) {
  using G = Geo<R, L>;
  __shared__ cx<R> lds[G::COLP * L];
  const int64_t cols = (int64_t)a.outer * a.inner;
  const int64_t tiles = (cols + G::COLP - 1) / G::COLP;
  const int sys = (int)(blockIdx.x / tiles);
  const int64_t tile = blockIdx.x - (int64_t)sys * tiles;
  if (!sys_active(a.status, sys)) return;
  const int p = threadIdx.x % G::COLP, t = threadIdx.x / G::COLP;
  const int64_t col = tile * G::COLP + p;
  const bool valid = col < cols;
  const int64_t cc = valid ? col : 0;
  const int64_t o = cc / a.inner, i = cc - o * a.inner;
  cx<R>* base = a.data + sys * a.stride + o * (int64_t)L * a.inner + i;
  const int inner = a.inner, n_in = a.n_in, n_out = a.n_out;
  auto ld = [&](int n) -> cx<R> { return n < n_in ? base[(int64_t)n * inner] : czero<R>(); };
  auto st = [&](int k, cx<R> v) {
    if (k < n_out) base[(int64_t)k * inner] = v;
  };
  const TwRegs<R, L, G::TC, G::HOLD_COL> tw(a.tw, t);
  fft_pencil<R, L, G::TC, DIR, false, false, PAD>(ld, st, lds + p, G::COLP, t, valid, tw);
}

// ------------------------------------------------------------------ launchers
template <typename R>
static void launch_row_fwd(int L, const RowArgs<R>& a, int nsys, hipStream_t s) {
  switch (L) {
#define C(l)                                                                   \
  case l: {                                                                    \
    using G = Geo<R, l>;                                                       \
    const int rows = 3 * a.nz * a.ny, tiles = (rows + G::ROWP - 1) / G::ROWP;  \
    hipLaunchKernelGGL((k_row_fwd<R, l>), dim3(tiles * nsys), dim3(G::T * G::ROWP), 0, s, a); \
    break;                                                                     \
  }
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("x pass", L);
  }
  check_launch("x forward");
}

template <typename R>
static void launch_row_inv(int L, const RowArgs<R>& a, int nsys, hipStream_t s) {
  switch (L) {
#define C(l)                                                                   \
  case l: {                                                                    \
    using G = Geo<R, l>;                                                       \
    const int rows = 3 * a.nz * a.ny, tiles = (rows + G::ROWP - 1) / G::ROWP;  \
    hipLaunchKernelGGL((k_row_inv_local<R, l>), dim3(tiles * nsys), dim3(G::T * G::ROWP), 0, s, a); \
    break;                                                                     \
  }
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("x pass", L);
  }
  check_launch("x inverse");
}

template <typename R, int DIR, int PAD>
static void launch_col(int L, const ColArgs<R>& a, hipStream_t s) {
  switch (L) {
#define C(l)                                                                        \
  case l: {                                                                         \
    using G = Geo<R, l>;                                                            \
    const int64_t cols = (int64_t)a.outer * a.inner;                                \
    const int64_t tiles = (cols + G::COLP - 1) / G::COLP;                           \
    hipLaunchKernelGGL((k_col<R, l, DIR, PAD>), dim3((unsigned)(tiles * a.nsys)), dim3(G::TC * G::COLP), 0, s, a); \
    break;                                                                          \
  }
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("column pass", L);
  }
  check_launch("column pass");
}

#define VIE_PLANE_SMALL(F) F(8) F(12) F(16) F(24) F(32) F(48) F(64)
#define VIE_PLANE_CASES(F) VIE_PLANE_SMALL(F) F(96) F(128)

// Whether a batch's x and y transforms run per plane; `planes` as for
// plane_rule.  Up to 64 always.  A plane of length 96 or 128 takes a CU to
// itself and 8 to 10 us of its time, so few planes are better spread over the
// chip as rows and columns, and so is a round of the 256 CUs that is far from
// full.  Product of 48x48xnz / 64x64xnz, rows and columns against planes, us:
//   96 f32:  93 planes 33.0, 33.4; 96 33.3, 32.1; 144 42.6, 39.3; 255 57.8, 51.9; 258 60.0, 67.3;
//            384 73.3, 74.9; 510 110, 111; 768 146, 146
//      f64:  96 42.0, 41.6; 144 52.3, 47.1; 255 77.6, 69.0; 258 78.6, 86.8; 384 94.5, 94.1 (40x40: 90.1, 91.6);
//            432 134, 132; 510 149, 142; 516 148, 159; 600 185, 188; 660 194, 194; 768 210, 204
//  128 f32:  96 41.1, 34.2; 255 74.7, 67.2; 258 78.3, 83.2; 285 82.3, 84.0; 300 89.9, 89.8 (52x52: 83.2, 85.3);
//            330 93.4, 92.1; 384 99.5, 93.8; 516 157, 158; 768 233, 215
// FP64 planes of length 128 exceed the LDS.  The choice follows the planes of
// one right-hand side (a batch's sums must be those of one alone), so batches
// that fill a little more than a round lose up to 9%: 3 x 48x48x32, 2 x 48x48x48.
bool plane_supported(int lx, int ly, int elem_bytes, int64_t planes) {
  if (lx != ly || lx > 128) return false;
  if (lx > 64) {
    const bool f32 = elem_bytes == 4;
    const int64_t last = (planes - 1) % 256 + 1;   // planes of the last round
    if (planes < 96) return false;
    if (lx == 96 && planes > 256 && (f32 || last < 154)) return false;
    if (lx == 128 && (!f32 || (planes > 256 && planes < 320))) return false;
  }
#define C(l) \
  if (lx == l) return true;
  VIE_PLANE_CASES(C)
#undef C
  return false;
}

template <typename R, int L, int PV>
static void launch_plane_pv(bool fwd, const RowArgs<R>& a, int nsys, hipStream_t s) {
  using G = PlaneGeo<R, L, PV>;
  const int tiles = (3 * a.nz + G::NPL - 1) / G::NPL;
  if constexpr (G::FITS) {
    if (fwd)
      hipLaunchKernelGGL((k_plane_fwd<R, L, PV>), dim3(tiles * nsys), dim3(G::BT), 0, s, a);
    else
      hipLaunchKernelGGL((k_plane_inv_local<R, L, PV>), dim3(tiles * nsys), dim3(G::BT), 0, s, a);
  } else {
    bad_length("plane pass", L);
  }
}

template <typename R>
static void launch_plane(bool fwd, int L, int pv, const RowArgs<R>& a, int nsys, hipStream_t s) {
  if (pv < 0 || pv >= kPlaneVariants) throw std::runtime_error("plane variant out of range");
  // udiv_m's range: element indices below 16 nx ny planes' worth, row
  // indices below 16 ny, plane indices below 3 nz
  const uint64_t pe = (uint64_t)a.nx * (uint64_t)a.ny;
  if (16 * pe * pe >= (1ull << 32) || 16 * (uint64_t)a.ny * a.ny >= (1ull << 32) || 3 * (uint64_t)a.nz * a.nz >= (1ull << 32))
    throw std::runtime_error("plane pass: box too large for its index arithmetic");
  switch (L) {
#define C(l)                                                 \
  case l: {                                                  \
    if (pv == 0)                                             \
      launch_plane_pv<R, l, (l > 64 ? 2 : 0)>(fwd, a, nsys, s); \
    else if (pv == 1)                                        \
      launch_plane_pv<R, l, (l > 64 ? 2 : 1)>(fwd, a, nsys, s); \
    else                                                     \
      launch_plane_pv<R, l, 2>(fwd, a, nsys, s);             \
    break;                                                   \
  }
    VIE_PLANE_CASES(C)
#undef C
    default:
      bad_length("plane pass", L);
  }
  check_launch("plane pass");
}

static void mark(hipEvent_t* ev, int i, hipStream_t s) {
  if (ev && hipEventRecord(ev[i], s) != hipSuccess) throw std::runtime_error("hipEventRecord failed");
}

// The products' transforms take padded axes to be at least half empty.
static void check_padding(int n, int l) {
  if (n < 1 || n > half_padded(l)) throw std::runtime_error("transform length below twice the axis");
}

template <typename R>
static RowArgs<R> row_args(const MvmBatch<R>& b, const KBatch* k, const FuseArgs& f, const c128* x, c128* y,
                           bool mask_input) {
  check_padding(b.nx, b.lx);
  check_padding(b.ny, b.ly);
  check_padding(b.nz, b.lz);
  RowArgs<R> ra{};
  ra.nx = b.nx;
  ra.ny = b.ny;
  ra.nz = b.nz;
  ra.lx = b.lx;
  ra.ly = b.ly;
  ra.vstride = b.vstride;
  ra.cstride = b.cstride;
  ra.wstride = b.wstride;
  ra.x = x;
  ra.y = y;
  ra.chi_inv = b.chi_inv;
  ra.work = b.work;
  ra.status = b.status;
  ra.tw = b.tw->table[b.lx];
  ra.mask_input = mask_input ? 1 : 0;
  ra.chi3 = b.rooftop;
  ra.m_pe = div_magic(b.nx * b.ny);
  ra.m_nx = div_magic(b.nx);
  ra.m_ny = div_magic(b.ny);
  ra.m_nz = div_magic(b.nz);
  ra.scale = 1.0 / ((double)b.lx * (double)b.ly * (double)b.lz);
  ra.r = f.r;
  ra.p = f.p;
  ra.v = f.v;
  ra.rhat = f.rhat;
  ra.s = f.s;
  if (k) ra.k = *k;
  return ra;
}

template <typename R>
void mvm_pass1(const MvmBatch<R>& b, const KBatch* k, const FuseArgs& f, const c128* x, bool mask_input,
               hipStream_t s) {
  if (b.nsys <= 0) return;
  if (f.in_mode == 0 && !x) throw std::runtime_error("mvm_pass1: missing input");
  if (f.in_mode != 0 && (!k || !f.r || !f.v || !f.p))
    throw std::runtime_error("mvm_pass1: missing fused vectors");
  RowArgs<R> ra = row_args<R>(b, k, f, x, nullptr, mask_input);
  ra.in_mode = f.in_mode;
  if (b.plane)
    launch_plane<R>(true, b.lx, b.pvariant, ra, b.nsys, s);
  else
    launch_row_fwd<R>(b.lx, ra, b.nsys, s);
}

template <typename R>
void mvm_mid(const MvmBatch<R>& b, hipStream_t s) {
  if (b.nsys <= 0) return;
  check_padding(b.ny, b.ly);
  check_padding(b.nz, b.lz);
  ColArgs<R> ca{};
  ca.data = b.work;
  ca.outer = 3 * b.nz;
  ca.inner = b.lx;
  ca.n_in = b.ny;
  ca.n_out = b.ly;
  ca.stride = b.wstride;
  ca.status = b.status;
  ca.tw = b.tw->table[b.ly];
  ca.nsys = b.nsys;
  if (!b.plane) launch_col<R, -1, PAD_IN>(b.ly, ca, s);

  ZArgs<R> za{};
  za.nz = b.nz;
  za.ly = b.ly;
  za.lx = b.lx;
  za.variant = b.zvariant;
  za.wstride = b.wstride;
  za.sstride = b.sstride;
  za.work = b.work;
  za.spec = b.spec;
  za.spec_tab = b.spec_tab;
  za.rooftop = b.rooftop;
  za.status = b.status;
  za.tw = b.tw->table[b.lz];
  launch_zconv<R>(b.lz, za, b.nsys, s);

  ca.n_in = b.ly;
  ca.n_out = b.ny;
  if (!b.plane) launch_col<R, +1, PAD_OUT>(b.ly, ca, s);
}

template <typename R>
void mvm_pass5(const MvmBatch<R>& b, const KBatch* k, const FuseArgs& f, const c128* x, c128* y, hipStream_t s) {
  if (b.nsys <= 0) return;
  if (!x || !y) throw std::runtime_error("mvm_pass5: missing vectors");
  if ((f.out_mode == 1 || f.out_mode == 2 || f.out_mode == 4) && !k)
    throw std::runtime_error("mvm_pass5: missing Krylov batch");
  if (((f.out_mode == 1 || f.out_mode == 3) && !f.rhat) || ((f.out_mode == 2 || f.out_mode == 4) && !f.s))
    throw std::runtime_error("mvm_pass5: missing fused vectors");
  RowArgs<R> ra = row_args<R>(b, k, f, x, y, false);
  ra.out_mode = f.out_mode;
  if (b.plane)
    launch_plane<R>(false, b.lx, b.pvariant, ra, b.nsys, s);
  else
    launch_row_inv<R>(b.lx, ra, b.nsys, s);
}

template <typename R>
void mvm(const MvmBatch<R>& b, const c128* x, c128* y, bool mask_input, hipStream_t s, hipEvent_t* ev) {
  if (b.nsys <= 0) return;
  const FuseArgs none{0, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
  mark(ev, 0, s);
  mvm_pass1<R>(b, nullptr, none, x, mask_input, s);
  mark(ev, 1, s);
  if (!ev) {
    mvm_mid<R>(b, s);
  } else {
    // per-pass events for measurement
    ColArgs<R> ca{};
    ca.data = b.work;
    ca.outer = 3 * b.nz;
    ca.inner = b.lx;
    ca.n_in = b.ny;
    ca.n_out = b.ly;
    ca.stride = b.wstride;
    ca.status = b.status;
    ca.tw = b.tw->table[b.ly];
    ca.nsys = b.nsys;
    if (!b.plane) launch_col<R, -1, PAD_IN>(b.ly, ca, s);
    mark(ev, 2, s);
    ZArgs<R> za{};
    za.nz = b.nz;
    za.ly = b.ly;
    za.lx = b.lx;
    za.variant = b.zvariant;
    za.wstride = b.wstride;
    za.sstride = b.sstride;
    za.work = b.work;
    za.spec = b.spec;
    za.spec_tab = b.spec_tab;
    za.rooftop = b.rooftop;
    za.status = b.status;
    za.tw = b.tw->table[b.lz];
    launch_zconv<R>(b.lz, za, b.nsys, s);
    mark(ev, 3, s);
    ca.n_in = b.ly;
    ca.n_out = b.ny;
    if (!b.plane) launch_col<R, +1, PAD_OUT>(b.ly, ca, s);
    mark(ev, 4, s);
  }
  mvm_pass5<R>(b, nullptr, none, x, y, s);
  mark(ev, 5, s);
}

// The z-pass variant of a shape; `cols` counts the columns of every system of
// the batch.  The lines lie where two variants cross.  Measured on 1024 to
// 262144 columns with the kernels alone, 5 us of event overhead with them (us;
// on either side of each line, the variant taken first), and checked with
// products of one problem repeated and of several in turn:
//    32: f32 16384 V2 11.1, V4 11.4; f64 16384 V4 16.0, V2 16.2, 24576 V2 16.1, V4 17.1; f64 rooftop
//        98304 V4 38.3, V2 39.2, 147456 V2 52.6, V4 53.6
//    36: f32 V2 (9216: 10.8, V4 13.1); f64 1024 V2 7.2, V4 7.7, 6144 V4 11.9, V2 12.2,
//        36864 V3 30.3, V4 30.8, 147456 V3 98.9, V4 109
//    48: 3072 f32 V0 8.5, V2 9.1, f64 V4 11.2, V2 11.5; 6144 f32 V2 10.4, V0 10.9, f64 V2 14.3, V4 16.7
//    64: V4 (f32 98304: V2 43.1, V4 45.2 with the spectrum in the caches, but 192x128x32 products of
//        several problems in turn 157, 153; f64 V2 within 1%)
//    72: f32 V2 (65536: 43, V3 57; 262144: 242, V3 253); f64 4096 V0 12.9, V2 13.4, 6144 V2 16.9, V0 18.8,
//        196608 V2 296, V3 314, 262144 V3 465, V2 504; f64 rooftop 16384 V2, 24576 V3 34.0, V2 35.5
//    96: 6144 f32 V0 14.9, V2 15.2, f64 V2 18.8, V0 19.8; 147456 f64 V2 289, V4 311, 196608 f64 V4 429, V2 449;
//        196608 f32 V2 210, V4 218, 262144 f32 V4 311, V2 334
//   128: 3072 V4 15.6, V2 16.7 (f64), 6144 V2 19.1, V4 20.3; 73728 f32 V2 95.4, V4 93.5, 98304 f32 V4 124,
//        V2 129; f32 rooftop 196608 V2 200, V4 219, 262144 V4 330, V2 338; f64 V2 (196608: 457, V4 532)
//   144: f32 36864 V4 55.3, V2 56.9, 65536 V2 113, V4 118, 196608 V2 305, V4 329; f64 V2 (65536: 206, V3 263)
//   192: f32 V4 (65536: 157, V2 168); f64 V2 (1024: 13.2, V4 13.9; 262144: 1428, V4 1560)
//   256: f32 V4 (16384: 45.5, V2 48.0); f64 V2 (196608: 1135, V4 1187), 256x256x128 products V4 3406, V2 3477,
//        rooftop V2 3147, V4 3267
//   from 288 on V4 (f64 288: V4 33.8, V2 39.1 at 4096 columns)
// Tiles of half a cache line (V2 of 96, f32 128, f64 72) rely on both
// halves of a line meeting in the caches, so they end where the work buffer
// leaves the Infinity Cache.  Below 32 V0 and V4 are one.  The mirror columns
// (V1) were ahead in none of 96 shapes of lengths 4 to 256.
int zpass_rule(int elem_bytes, int lz, bool rooftop, int64_t cols) {
  const bool f32 = elem_bytes == 4;
  if (lz < 32) return 0;
  switch (lz) {
    case 32: return cols < (f32 ? 16384 : rooftop ? 131072 : 20480) ? 4 : 2;
    case 36: return f32 || cols < 4096 ? 2 : (cols >= 32768 ? 3 : 4);
    case 48: return cols >= 5120 ? 2 : (f32 ? 0 : 4);
    case 64: return 4;
    case 72:
      if (f32) return 2;
      if (cols < 5120) return 0;
      return cols >= (rooftop ? 20480 : 229376) ? 3 : 2;
    case 96: return cols < (f32 ? 8192 : 5120) ? 0 : (cols >= (f32 || rooftop ? 229376 : 172032) ? 4 : 2);
    case 128: return cols < 5120 || (f32 && cols >= (rooftop ? 229376 : 80000)) ? 4 : 2;
    case 144: return f32 && cols < 57344 ? 4 : 2;
    case 256: return f32 || (!rooftop && cols >= 229376) ? 4 : 2;
    default: return f32 || lz >= 288 ? 4 : 2;
  }
}

// The plane-kernel variant of a shape; `planes` counts the z-planes of the
// three components of every system of the batch.  Few planes want many short
// workgroups, many planes of a small transform fuller ones.  Forward and
// inverse together, with 10 us of event overhead (f32 / f64, us, variants 0, 1, 2):
//   length 16: 384 planes 15.4, 13.6, 14.6 / 15.9, 14.7, 15.7; 6144: 21.2, 28.1, 41.7 / 25.1, 36.8, 59.6
//          24: 576: 29.4, 16.8, 15.5 / 21.9, 18.6, 17.5; 9216: 59.0, 44.7, 52.5 / 60.5, 54.1, 63.7
//          32: 768: 25.6, 18.2, 17.6 / 21.3, 21.1, 19.9; 12288: 84.4, 61.5, 69.1 / 100.6, 100.1, 103.3
//          48: 768: 35.1, 35.0, 26.1 / 29.9, 29.7, 29.5; 3072: 63.8, 63.0, 56.9
// From 48 on variant 1 is one plane by 512 threads; products of 24x24xnz and
// 32x32xnz with variants 1, 2:
//          48 f32: nz 2 14.3, 17.5; 64 20.9, 24.1; 128 29.2, 31.2; 256 56.3, 52.6
//             f64: nz 2 14.6, 18.3; 64 26.2, 29.8; 128 39.2, 38.8; 256 68.7, 63.0
//          64 f32: nz 2 12.5, 15.3; 64 22.2, 24.4; 128 32.2, 33.1; 256 57.5, 55.2
//             f64: nz 2 13.9, 16.2; 64 28.8, 30.6; 96 39.0, 37.7; 256 90.4, 87.1
// `most` is the plane count of the batches that share the choice: a problem's
// own product runs in batches of several right-hand sides too, whose sums
// must be those of one alone.
int plane_rule(int l, int64_t planes, int64_t most) {
  if (l <= 8) return 0;
  if (l <= 16) return planes > 2048 ? 0 : 1;
  if (l <= 32) return planes > 1024 ? 1 : 2;
  return most <= 192 ? 1 : 2;
}

#define VIE_MVM_INST(R)                                                                                           \
  template void mvm<R>(const MvmBatch<R>&, const c128*, c128*, bool, hipStream_t, hipEvent_t*);                  \
  template void mvm_pass1<R>(const MvmBatch<R>&, const KBatch*, const FuseArgs&, const c128*, bool, hipStream_t); \
  template void mvm_mid<R>(const MvmBatch<R>&, hipStream_t);                                                     \
  template void mvm_pass5<R>(const MvmBatch<R>&, const KBatch*, const FuseArgs&, const c128*, c128*, hipStream_t);
VIE_MVM_INST(float)
VIE_MVM_INST(double)
#undef VIE_MVM_INST

int64_t mvm_row_tiles(int lx, int nz, int ny) {
  const int64_t rows = 3 * (int64_t)nz * ny;
  if (lx <= 64) {   // plane kernels: at most one workgroup per plane (a longer plane has more row tiles)
    switch (lx) {
#define C(l)                                                                                 \
  case l: {                                                                                  \
    const int rp = cmin(Geo<float, l>::ROWP, Geo<double, l>::ROWP);                          \
    return std::max<int64_t>((rows + rp - 1) / rp, 3 * (int64_t)nz);                        \
  }
      VIE_PLANE_SMALL(C)
#undef C
    }
  }
  switch (lx) {
#define C(l)                                                                            \
  case l: {                                                                             \
    const int rp = cmin(Geo<float, l>::ROWP, Geo<double, l>::ROWP);                     \
    return (rows + rp - 1) / rp;                                                        \
  }
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("x pass", lx);
  }
}

// ------------------------------------------------------------------ spectra setup
// T(m) of the discretised dyadic Green's function (eq. (1) with the scalar
// Green's function after it), collocated voxels: for m != 0 the dyadic
// (I + grad grad / k0^2) g sampled at the centre separation R times
// k0^2 dV,
//   g [ (1 - j/u - 1/u^2) I + (3/u^2 + 3j/u - 1) Rhat Rhat ],  u = k0 |R|;
// for m = 0 the integral of k0^2 G over the equal-volume sphere,
//   ((2 (1 + j k0 a) exp(-j k0 a) - 3) / 3) I,  a = (3 dV / 4 pi)^(1/3).
// Slot s of an axis of n voxels embedded in length L holds offset s (s < n),
// s - L (s > L - n), nothing otherwise.  Output [6][lz][ly][lx], component
// order xx, xy, xz, yy, yz, zz.
__device__ __forceinline__ int slot_offset(int s, int n, int L, bool* ok) {
  if (s < n) {
    *ok = true;
    return s;
  }
  if (s > L - n) {
    *ok = true;
    return s - L;
  }
  *ok = false;
  return 0;
}

__global__ void k_green_embed(c128* out, int nx, int ny, int nz, int lx, int ly, int lz, double dx, double dy,
                              double dz, double k0) {
  const int64_t npts = (int64_t)lx * ly * lz;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npts) return;
  const int sx = (int)(i % lx);
  const int sy = (int)((i / lx) % ly);
  const int sz = (int)(i / ((int64_t)lx * ly));
  bool okx, oky, okz;
  const int mx = slot_offset(sx, nx, lx, &okx);
  const int my = slot_offset(sy, ny, ly, &oky);
  const int mz = slot_offset(sz, nz, lz, &okz);
  double t[6] = {0, 0, 0, 0, 0, 0};
  double ti[6] = {0, 0, 0, 0, 0, 0};
  if (okx && oky && okz) {
    const double dV = dx * dy * dz;
    if (mx == 0 && my == 0 && mz == 0) {
      const double a = cbrt(3.0 * dV / (4.0 * M_PI));
      const double x = k0 * a;
      double sn, cs;
      sincos(x, &sn, &cs);
      // (1 + j x) exp(-j x) = (cos x + x sin x) + j (x cos x - sin x)
      const double re = (2.0 * (cs + x * sn) - 3.0) / 3.0;
      const double im = 2.0 * (x * cs - sn) / 3.0;
      t[0] = t[3] = t[5] = re;
      ti[0] = ti[3] = ti[5] = im;
    } else {
      const double Rx = mx * dx, Ry = my * dy, Rz = mz * dz;
      const double R = sqrt(Rx * Rx + Ry * Ry + Rz * Rz);
      const double u = k0 * R;
      double sn, cs;
      sincos(u, &sn, &cs);
      const double inv4piR = 1.0 / (4.0 * M_PI * R);
      // pref = k0^2 dV g = k0^2 dV exp(-j u) / (4 pi R)
      const double pr = k0 * k0 * dV * cs * inv4piR, pi = -k0 * k0 * dV * sn * inv4piR;
      const double iu = 1.0 / u, iu2 = iu * iu;
      const double ar = 1.0 - iu2, ai = -iu;          // 1 - j/u - 1/u^2
      const double br = 3.0 * iu2 - 1.0, bi = 3.0 * iu;  // 3/u^2 + 3j/u - 1
      const double rh[3] = {Rx / R, Ry / R, Rz / R};
      const int ci[6] = {0, 0, 0, 1, 1, 2}, cj[6] = {0, 1, 2, 1, 2, 2};
      for (int c = 0; c < 6; ++c) {
        const double rr = rh[ci[c]] * rh[cj[c]];
        double fr = br * rr, fi = bi * rr;
        if (ci[c] == cj[c]) {
          fr += ar;
          fi += ai;
        }
        t[c] = pr * fr - pi * fi;
        ti[c] = pr * fi + pi * fr;
      }
    }
  }
  for (int c = 0; c < 6; ++c) out[c * npts + i] = mk<double>(t[c], ti[c]);
}

__global__ void k_extract_octant(const c128* full, c128* s64, c64* s32, int lx, int ly, int lz, int ncomp) {
  const int ox = lx / 2 + 1, oy = ly / 2 + 1, oz = lz / 2 + 1;
  const int64_t oct = (int64_t)ox * oy * oz;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ncomp * oct) return;
  const int c = (int)(i / oct);
  const int64_t r = i - c * oct;
  const int fx = (int)(r % ox), fy = (int)((r / ox) % oy), fz = (int)(r / ((int64_t)ox * oy));
  const c128 v = full[(int64_t)c * lx * ly * lz + ((int64_t)fz * ly + fy) * lx + fx];
  if (s64) s64[i] = v;
  if (s32) s32[i] = cvt<float>(v);
}

template <int L>
static void launch_row_full_L(c128* data, int64_t rows, const c128* tw, hipStream_t s) {
  using G = Geo<double, L>;
  const int64_t blocks = (rows + G::ROWP - 1) / G::ROWP;
  hipLaunchKernelGGL((k_row_full<double, L>), dim3((unsigned)blocks), dim3(G::T * G::ROWP), 0, s, data, rows, tw);
}

static void launch_row_full(int L, c128* data, int64_t rows, const c128* tw, hipStream_t s) {
  switch (L) {
#define C(l)                                  \
  case l:                                     \
    launch_row_full_L<l>(data, rows, tw, s); \
    break;
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("setup x pass", L);
  }
  check_launch("setup x pass");
}

void green_spectra(int nx, int ny, int nz, int lx, int ly, int lz, double dx, double dy, double dz, double k0,
                   c128* scratch, c128* spec64, c64* spec32, const TwiddleSet<double>& tw, hipStream_t s) {
  const int64_t npts = (int64_t)lx * ly * lz;
  hipLaunchKernelGGL(k_green_embed, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, s, scratch, nx, ny, nz, lx,
                     ly, lz, dx, dy, dz, k0);
  check_launch("green embed");
  launch_row_full(lx, scratch, 6 * (int64_t)ly * lz, tw.table[lx], s);
  ColArgs<double> ca{};
  ca.data = scratch;
  ca.outer = 6 * lz;
  ca.inner = lx;
  ca.n_in = ly;
  ca.n_out = ly;
  ca.stride = 0;
  ca.status = nullptr;
  ca.tw = tw.table[ly];
  ca.nsys = 1;
  launch_col<double, -1, PAD_NONE>(ly, ca, s);
  ca.outer = 6;
  ca.inner = lx * ly;
  ca.n_in = lz;
  ca.n_out = lz;
  ca.tw = tw.table[lz];
  launch_col<double, -1, PAD_NONE>(lz, ca, s);
  const int64_t oct = 6 * (int64_t)(lx / 2 + 1) * (ly / 2 + 1) * (lz / 2 + 1);
  hipLaunchKernelGGL(k_extract_octant, dim3((unsigned)((oct + 255) / 256)), dim3(256), 0, s, scratch, spec64, spec32,
                     lx, ly, lz, 6);
  check_launch("octant");
}

// Rooftop discretisation (Sec. II-A, eq. (5)): the scalar kernel
// k0^2 dV g~(m), g~ the scalar Green's function at the centre separation for
// m != 0 and its mean over the sphere of the cell's volume at m = 0,
//   k0^2 dV g~(0) = (1 + j k0 a) exp(-j k0 a) - 1,  a = (3 dV / 4 pi)^(1/3)
// (the radial integral of r exp(-j k0 r) from 0 to a).  Same slot layout as
// k_green_embed, one component.
__global__ void k_green_embed_scalar(c128* out, int nx, int ny, int nz, int lx, int ly, int lz, double dx, double dy,
                                     double dz, double k0) {
  const int64_t npts = (int64_t)lx * ly * lz;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npts) return;
  const int sx = (int)(i % lx);
  const int sy = (int)((i / lx) % ly);
  const int sz = (int)(i / ((int64_t)lx * ly));
  bool okx, oky, okz;
  const int mx = slot_offset(sx, nx, lx, &okx);
  const int my = slot_offset(sy, ny, ly, &oky);
  const int mz = slot_offset(sz, nz, lz, &okz);
  double re = 0.0, im = 0.0;
  if (okx && oky && okz) {
    const double dV = dx * dy * dz;
    if (mx == 0 && my == 0 && mz == 0) {
      const double x = k0 * cbrt(3.0 * dV / (4.0 * M_PI));
      double sn, cs;
      sincos(x, &sn, &cs);
      re = cs + x * sn - 1.0;
      im = x * cs - sn;
    } else {
      const double Rx = mx * dx, Ry = my * dy, Rz = mz * dz;
      const double R = sqrt(Rx * Rx + Ry * Ry + Rz * Rz);
      double sn, cs;
      sincos(k0 * R, &sn, &cs);
      const double f = k0 * k0 * dV / (4.0 * M_PI * R);
      re = f * cs;
      im = -f * sn;
    }
  }
  out[i] = mk<double>(re, im);
}

// b_j(q) = (1 - exp(-2 pi i q / L_j)) / (k0 d_j) for q in [0, L_j), the three
// axes one after the other: 1 - cos t = 2 sin^2(t / 2) keeps the small
// symbols accurate.
__global__ void k_diff_symbols(c128* s64, c64* s32, int lx, int ly, int lz, double dx, double dy, double dz,
                               double k0) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= lx + ly + lz) return;
  int q = i, L = lx;
  double d = dx;
  if (q >= lx) {
    q -= lx;
    L = ly;
    d = dy;
    if (q >= ly) {
      q -= ly;
      L = lz;
      d = dz;
    }
  }
  double sh, ch, sf, cf;
  sincospi((double)q / L, &sh, &ch);
  sincospi(2.0 * q / L, &sf, &cf);
  const c128 b = mk<double>(2.0 * sh * sh / (k0 * d), sf / (k0 * d));
  if (s64) s64[i] = b;
  if (s32) s32[i] = cvt<float>(b);
}

void green_spectrum_rooftop(int nx, int ny, int nz, int lx, int ly, int lz, double dx, double dy, double dz,
                            double k0, c128* scratch, c128* spec64, c64* spec32, const TwiddleSet<double>& tw,
                            hipStream_t s) {
  const int64_t npts = (int64_t)lx * ly * lz;
  hipLaunchKernelGGL(k_green_embed_scalar, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, s, scratch, nx, ny,
                     nz, lx, ly, lz, dx, dy, dz, k0);
  check_launch("rooftop embed");
  launch_row_full(lx, scratch, (int64_t)ly * lz, tw.table[lx], s);
  ColArgs<double> ca{};
  ca.data = scratch;
  ca.outer = lz;
  ca.inner = lx;
  ca.n_in = ly;
  ca.n_out = ly;
  ca.stride = 0;
  ca.status = nullptr;
  ca.tw = tw.table[ly];
  ca.nsys = 1;
  launch_col<double, -1, PAD_NONE>(ly, ca, s);
  ca.outer = 1;
  ca.inner = lx * ly;
  ca.n_in = lz;
  ca.n_out = lz;
  ca.tw = tw.table[lz];
  launch_col<double, -1, PAD_NONE>(lz, ca, s);
  const int64_t oct = (int64_t)(lx / 2 + 1) * (ly / 2 + 1) * (lz / 2 + 1);
  hipLaunchKernelGGL(k_extract_octant, dim3((unsigned)((oct + 255) / 256)), dim3(256), 0, s, scratch, spec64, spec32,
                     lx, ly, lz, 1);
  check_launch("rooftop octant");
  hipLaunchKernelGGL(k_diff_symbols, dim3((unsigned)((lx + ly + lz + 255) / 256)), dim3(256), 0, s,
                     spec64 ? spec64 + oct : nullptr, spec32 ? spec32 + oct : nullptr, lx, ly, lz, dx, dy, dz, k0);
  check_launch("rooftop symbols");
}

}  // namespace vie
