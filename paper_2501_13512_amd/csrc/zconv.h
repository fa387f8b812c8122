// The z pass with columns in LDS: the column-set variants 0, 2, 3, 4 and the
// mirror-column variant 1, and the launcher of every z-pass kernel.
// Instantiated once per precision (zconv32.hip, zconv64.hip).
#pragma once
#include "fft_core.h"
#include "zpass.h"

namespace vie {

// Pass 3: z forward (nz -> LZ), spectral multiply, z inverse (LZ -> nz).
//
// The spectrum is stored for q in [0, L/2] per axis only; the other octants
// are the same values with a sign (S_ij(L - q) = +-S_ij(q)).  An axis of
// length L is covered by folds f in [0, nfold(L)); fold f stands for column
// f (mirror 0) and column L - f (mirror 1), both using spectral index f.
// For even L fold 0's mirror is the Nyquist column L/2 (spectral index L/2,
// sign +); for odd L fold 0 has no mirror.  A workgroup takes one y-fold and
// ZP consecutive x-folds and transforms all four mirror columns
// (+-qx, +-qy) of the three components, so each spectrum value is loaded
// once and applied to up to 8 points (+-qx, +-qy, qz and LZ - qz).
__host__ __device__ constexpr int nfold(int L) { return (L % 2 == 0) ? L / 2 : (L + 1) / 2; }

struct FoldCol {
  int col;  // column index, -1 if absent
  int sf;   // spectral (octant) index
  int sg;   // parity sign for components odd in this axis
};

__device__ __forceinline__ FoldCol fold_col(int f, int m, int L) {
  if (m == 0) return {f, f, 1};
  if (f > 0) return {L - f, f, -1};
  if ((L & 1) == 0 && L >= 2) return {L / 2, L / 2, 1};
  return {-1, 0, 1};
}

// Variant 0: one tile of ZP columns per workgroup, three components side by
// side; each point loads its spectrum values.  Tiles run along mirror-paired
// rows, chunked per XCD, so the four mirror columns that use one octant
// spectrum value are transformed on one XCD close together in time and the
// value is fetched from HBM about once.
// Column-set variants (V = 0, 2, 3, 4): ZP columns per workgroup, TZ threads
// per column and component, PF: spectrum values loaded into registers
// before the data (their latency overlaps the forward transform).
//   0: wide tiles (up to 1024 threads), max_butterflies threads per column
//   2: one wavefront per component: 64 threads take the columns of half a
//      cache line or more, with no more threads to a column than its first
//      radix keeps busy.  The pass waits on memory, LDS and barriers in
//      turn, so many small workgroups at different points of it hide more
//      than few large ones (see zpass_rule for the times; 144 in FP32 has a
//      geometry of its own, LINE2)
//   3: one cache line of columns, min_butterflies threads, prefetch
//   4: one cache line of columns, max_butterflies threads
// zcol_kernel has the lengths at which variants share a kernel.
template <typename R, int LZ, int V, int K>
struct ZColGeo {
  static constexpr int T = PlanInfo<LZ>::max_butterflies;
  static constexpr int TB = PlanInfo<LZ>::min_butterflies;
  static constexpr int ES = (int)sizeof(cx<R>);
  static constexpr int LDS_ZP = cmax(1, (144 * 1024) / (3 * LZ * ES));
  static constexpr int LINE = cmax(1, pow2_floor(cmin(LDS_ZP, 128 / ES)));
  static constexpr int WIDE = cmax(1, pow2_floor(cmin(LDS_ZP, cmin(64, cmax(128 / ES, 1024 / (3 * T))))));
  static constexpr int WAVE = cmin(64, cmax(64 / ES, 64 / pow2_ceil(TB)));
  // FP32 144 takes V2's place for many columns: one cache line of columns by 16
  // threads each, with the prefetch (196608 columns: V4 329 us, half a line by
  // one wavefront per component 360)
  static constexpr bool LINE2 = V == 2 && sizeof(R) == 4 && LZ == 144;
  static constexpr int ZP = V == 2 && !LINE2 ? WAVE : (V == 0 ? WIDE : LINE);
  static constexpr int TZ = LINE2    ? pow2_ceil(TB)
                            : V == 2 ? cmin(T, 64 / ZP)
                            : V == 3 ? cmin(TB, cmax(1, 1024 / (3 * ZP)))
                                     : cmin(T, pow2_floor(cmax(1, 1024 / (3 * ZP))));
  // the rooftop spectrum is three values a point instead of six: short
  // columns have the registers for it (length 48 FP32, 65536 columns: 27.0 us
  // with the prefetch, 28.7 without)
  static constexpr bool PF = V == 3 || LINE2 || (V == 2 && K == 1 && LZ <= 48);
  // twiddles held in registers over both transforms: not in FP64 beside the
  // prefetched spectrum (64 systems of length 48: 49 us without, 60 with) or
  // for short columns
  static constexpr bool HOLD = !LINE2 && (sizeof(R) == 4 || (!PF && LZ >= 72));
  // wavefronts per SIMD that the registers must leave room for: FP64 beside
  // the prefetched spectrum needs the third (length 48, 65536 columns: 54 us
  // with three, 70 with the two that 170 registers allow)
  static constexpr int WAVES = sizeof(R) == 8 && PF && LZ <= 64 ? 3 : 1;
  static_assert(3 * LZ * ZP * ES <= 150 * 1024, "tile exceeds the LDS");
};

// Variant 1 (mirror columns): geometry.
template <typename R, int LZ>
struct ZGeo {
  static constexpr int T = PlanInfo<LZ>::max_butterflies;
  static constexpr int ES = (int)sizeof(cx<R>);
  static constexpr int ZP = cmax(1, pow2_floor(cmin(64, cmin(1024 / (3 * T), (144 * 1024) / (12 * LZ * ES)))));
};

template <typename R, int LZ>
__global__ void __launch_bounds__((3 * ZGeo<R, LZ>::T * ZGeo<R, LZ>::ZP)) k_zconv_mirror(ZArgs<R> a) {
  using G = ZGeo<R, LZ>;
  constexpr int T = G::T, ZP = G::ZP;
  constexpr int SLOT = LZ * ZP;           // one (mirror, component) pencil set
  __shared__ cx<R> lds[12 * SLOT];        // [mirror 4][component 3][qz][p]
  const int lx = a.lx, ly = a.ly, nz = a.nz;
  const int nfx = nfold(lx), nfy = nfold(ly);
  const int xt = (nfx + ZP - 1) / ZP;
  const int per_sys = nfy * xt;
  const int sys = blockIdx.x / per_sys;
  const int rr = blockIdx.x - sys * per_sys;
  const int fy = rr / xt, ft = rr - fy * xt;
  if (!sys_active(a.status, sys)) return;
  const int comp = threadIdx.x / (T * ZP);
  const int rem = threadIdx.x - comp * (T * ZP);
  const int p = rem % ZP, t = rem / ZP;
  const int fx = ft * ZP + p;
  const bool pvalid = fx < nfx;
  const int64_t plane = (int64_t)ly * lx;
  cx<R>* wsys = a.work + sys * a.wstride + (int64_t)comp * nz * plane;

  // forward along z of the four mirror columns, into LDS
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const FoldCol cxm = fold_col(fx, m & 1, lx), cym = fold_col(fy, m >> 1, ly);
    const bool valid = pvalid && cxm.col >= 0 && cym.col >= 0;
    cx<R>* base = wsys + (valid ? (int64_t)cym.col * lx + cxm.col : 0);
    cx<R>* slot = lds + (m * 3 + comp) * SLOT + p;
    auto ldg = [&](int n) -> cx<R> { return n < nz ? base[n * plane] : czero<R>(); };
    auto sts = [&](int k, cx<R> v) { slot[k * ZP] = v; };
    fft_pencil<R, LZ, T, -1, false, true, PAD_IN>(ldg, sts, slot, ZP, t, valid, a.tw);
  }

  // Q = S X at every point of the four columns; one spectrum load per
  // (fold x, fold y, fold z), reused for its mirrors
  const int64_t ox = lx / 2 + 1, oy = ly / 2 + 1;
  const int64_t oct = ox * oy * (LZ / 2 + 1);
  const cx<R>* spec = a.spec_tab ? a.spec_tab[sys] : a.spec + sys * a.sstride;
  constexpr int NFZ = nfold(LZ);
  for (int i = threadIdx.x; i < NFZ * ZP; i += 3 * T * ZP) {
    const int fz = i / ZP, pp = i - fz * ZP;
    const int fxx = ft * ZP + pp;
    if (fxx >= nfx) continue;
    int64_t o_prev = -1;
    cx<R> sxx, sxy, sxz, syy, syz, szz;
#pragma unroll
    for (int mz = 0; mz < 2; ++mz) {
      const FoldCol czm = fold_col(fz, mz, LZ);
      if (czm.col < 0) continue;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const FoldCol cxm = fold_col(fxx, m & 1, lx), cym = fold_col(fy, m >> 1, ly);
        if (cxm.col < 0 || cym.col < 0) continue;
        const int64_t o = ((int64_t)czm.sf * oy + cym.sf) * ox + cxm.sf;
        if (o != o_prev) {
          sxx = spec[o];
          sxy = spec[oct + o];
          sxz = spec[2 * oct + o];
          syy = spec[3 * oct + o];
          syz = spec[4 * oct + o];
          szz = spec[5 * oct + o];
          o_prev = o;
        }
        const R gxy = R(cxm.sg * cym.sg), gxz = R(cxm.sg * czm.sg), gyz = R(cym.sg * czm.sg);
        const cx<R> axy = gxy * sxy, axz = gxz * sxz, ayz = gyz * syz;
        cx<R>* e = lds + m * 3 * SLOT + czm.col * ZP + pp;
        const cx<R> X = e[0], Y = e[SLOT], Z = e[2 * SLOT];
        e[0] = sxx * X + axy * Y + axz * Z;
        e[SLOT] = axy * X + syy * Y + ayz * Z;
        e[2 * SLOT] = axz * X + ayz * Y + szz * Z;
      }
    }
  }
  __syncthreads();

  // inverse along z, cropped to nz, back to HBM
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const FoldCol cxm = fold_col(fx, m & 1, lx), cym = fold_col(fy, m >> 1, ly);
    const bool valid = pvalid && cxm.col >= 0 && cym.col >= 0;
    cx<R>* base = wsys + (valid ? (int64_t)cym.col * lx + cxm.col : 0);
    cx<R>* slot = lds + (m * 3 + comp) * SLOT + p;
    auto lds_ld = [&](int n) -> cx<R> { return slot[n * ZP]; };
    auto stg = [&](int k, cx<R> v) {
      if (k < nz) base[k * plane] = v;
    };
    fft_pencil<R, LZ, T, +1, true, false, PAD_OUT>(lds_ld, stg, slot, ZP, t, valid, a.tw);
  }
}

// K = 0: the collocated dyadic multiply (six octant spectra of the symmetric
// tensor).  K = 1: the rooftop discretisation, whose spectral operator is
// G'(q) (X_c - conj(b_c) sum_j b_j X_j) with G' = k0^2 dV FFT(g~) (one even
// octant spectrum) and b_j = (1 - exp(-2 pi i q_j / L_j)) / (k0 d_j), the
// symbol of the cell divergence of face values; -conj(b_c) is the symbol of
// the face gradient of cell values.  The spectrum buffer holds the octant of
// G' followed by the full-length tables b_x[lx], b_y[ly], b_z[lz].
template <typename R, int LZ, int V, int K>
__global__ void __launch_bounds__((3 * ZColGeo<R, LZ, V, K>::TZ * ZColGeo<R, LZ, V, K>::ZP), (ZColGeo<R, LZ, V, K>::WAVES))
    k_zconv_col(ZArgs<R> a) {
  using G = ZColGeo<R, LZ, V, K>;
  constexpr int T = G::TZ, ZP = G::ZP;
  constexpr int NT = 3 * T * ZP;
  constexpr int HZ = LZ / 2;
  constexpr int NFT = NT / ZP;                    // fold walkers per column
  constexpr int NF = (HZ + 1 + NFT - 1) / NFT;    // folds per walker
  __shared__ cx<R> lds[3 * LZ * ZP];
  const int cols = a.ly * a.lx;
  const int tiles = (cols + ZP - 1) / ZP;
  // Tile-major logical order (the grid is tiles x systems): each XCD takes
  // a contiguous range of tiles of every system, so the systems still
  // active are spread over all XCDs whichever they are, and the group's
  // shared spectrum columns of a tile are reused from that XCD's L2 by the
  // consecutive workgroups of the other systems.
  const int nsys = (int)gridDim.x / tiles;
  const int g = __builtin_amdgcn_readfirstlane(xcd_chunked(blockIdx.x, gridDim.x));   // uniform
  const int tile = g / nsys, sys = g - tile * nsys;
  if (!sys_active(a.status, sys)) return;
  const int comp = threadIdx.x / (T * ZP);
  const int rem = threadIdx.x - comp * (T * ZP);
  const int p = rem % ZP, t = rem / ZP;
  const TwRegs<R, LZ, T, G::HOLD> tw(a.tw, t);
  const int col = tile * ZP + p;   // logical column
  const bool valid = col < cols;
  // element offsets in 32 bits from the system's base (one system's work
  // buffer holds < 2^31 elements), so loads use a uniform base + offset
  const unsigned plane = (unsigned)a.ly * (unsigned)a.lx;
  unsigned pcol = 0;               // its place in the plane
  if (valid) {
    const int i = col / a.lx;
    pcol = (unsigned)(mirror_paired_row(i, a.ly) * a.lx + (col - i * a.lx));
  }
  cx<R>* const wsys = a.work + sys * a.wstride;
  const unsigned coff = (unsigned)comp * (unsigned)a.nz * plane + pcol;
  cx<R>* slot = lds + comp * LZ * ZP + p;
  const int nz = a.nz;

  // The multiply's view: a thread keeps one column (qx, qy) and walks the
  // z-folds fz = j, j + NFT, ...: each spectrum value serves qz = fz and
  // qz = LZ - fz.
  const int lx = a.lx, ly = a.ly;
  const int hx = lx / 2, hy = ly / 2;
  const int64_t ox = hx + 1, oy = hy + 1;
  const int64_t oct = ox * oy * (HZ + 1);
  const int pp = threadIdx.x % ZP, j0 = threadIdx.x / ZP;
  const int c2 = tile * ZP + pp;
  const bool cvalid = c2 < cols;
  R sx = R(1), sy = R(1);
  const cx<R>* const sp = a.spec_tab ? a.spec_tab[sys] : a.spec + sys * a.sstride;
  unsigned soff = 0;
  cx<R> bx = czero<R>(), by = czero<R>();   // K = 1: difference symbols of the column
  const unsigned oct32 = (unsigned)oct, fzs = (unsigned)(oy * ox);
  if (cvalid) {
    const int i2 = c2 / lx;
    const int qy = mirror_paired_row(i2, ly), qx = c2 - i2 * lx;
    const int fx = qx <= hx ? qx : lx - qx, fy = qy <= hy ? qy : ly - qy;
    sx = qx <= hx ? R(1) : R(-1);
    sy = qy <= hy ? R(1) : R(-1);
    soff = (unsigned)(fy * ox + fx);
    if constexpr (K == 1) {
      bx = *elem(sp, oct32 + (unsigned)qx);
      by = *elem(sp, oct32 + (unsigned)(lx + qy));
    }
  }
  constexpr int NS = K == 1 ? 3 : 6;
  // K = 0: spectrum values (xx, xy, xz, yy, yz, zz, parity signs of qx, qy
  // applied); K = 1: G'(fz), b_z(fz), b_z(LZ - fz)
  auto spec_at = [&](int fz, cx<R>* sv) {
    const unsigned o = soff + (unsigned)fz * fzs;
    if constexpr (K == 1) {
      const unsigned bz0 = oct32 + (unsigned)(lx + ly);
      sv[0] = *elem(sp, o);
      sv[1] = *elem(sp, bz0 + (unsigned)fz);
      sv[2] = *elem(sp, bz0 + (unsigned)(fz == 0 ? 0 : LZ - fz));
    } else {
      sv[0] = *elem(sp, o);
      sv[1] = (sx * sy) * *elem(sp, oct32 + o);
      sv[2] = sx * *elem(sp, 2 * oct32 + o);
      sv[3] = *elem(sp, 3 * oct32 + o);
      sv[4] = sy * *elem(sp, 4 * oct32 + o);
      sv[5] = *elem(sp, 5 * oct32 + o);
    }
  };
  cx<R> pre[G::PF ? NF : 1][NS];
  if constexpr (G::PF) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int fz = j0 + f * NFT;
      if (cvalid && fz <= HZ) spec_at(fz, pre[f]);
    }
  }

  // forward along z into the component's LDS slot
  // first-stage element n = t + (a constant of the unrolled stage): offsets
  // split into a per-thread part and a uniform part
  const unsigned toff = coff + (unsigned)t * plane;
  auto ldg = [&](int n) -> cx<R> {
    return n < nz ? *elem(wsys, toff + (unsigned)(n - t) * plane) : czero<R>();
  };
  auto sts = [&](int k, cx<R> v) { slot[k * ZP] = v; };
  fft_pencil<R, LZ, T, -1, false, true, PAD_IN>(ldg, sts, slot, ZP, t, valid, tw);

  // Q(q) = S(q) X(q), S symmetric 3x3 from the octant with parity signs
  if constexpr (K == 1) if (cvalid) {
    cx<R>* e0 = lds + pp;
    const cx<R> cbx = conj(bx), cby = conj(by);
    auto roof = [&](cx<R>* e, cx<R> gq, cx<R> bz) {
      const cx<R> X = e[0], Y = e[LZ * ZP], Z = e[2 * LZ * ZP];
      const cx<R> d = bx * X + by * Y + bz * Z;   // divergence
      e[0] = gq * (X - cbx * d);
      e[LZ * ZP] = gq * (Y - cby * d);
      e[2 * LZ * ZP] = gq * (Z - conj(bz) * d);
    };
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int fz = j0 + f * NFT;
      if (fz > HZ) break;
      cx<R> sl[NS];
      const cx<R>* sv = sl;
      if constexpr (G::PF)
        sv = pre[f];
      else
        spec_at(fz, sl);
      roof(e0 + fz * ZP, sv[0], sv[1]);
      const int qz2 = LZ - fz;
      if (fz > 0 && qz2 != fz) roof(e0 + qz2 * ZP, sv[0], sv[2]);
    }
  }
  if constexpr (K == 0) if (cvalid) {
    cx<R>* e0 = lds + pp;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int fz = j0 + f * NFT;
      if (fz > HZ) break;
      cx<R> sl[NS];
      const cx<R>* sv = sl;
      if constexpr (G::PF)
        sv = pre[f];
      else
        spec_at(fz, sl);
      const cx<R> sxx = sv[0], sxy = sv[1], sxz = sv[2], syy = sv[3], syz = sv[4], szz = sv[5];
      {
        cx<R>* e = e0 + fz * ZP;   // qz = fz: sz = +1
        const cx<R> X = e[0], Y = e[LZ * ZP], Z = e[2 * LZ * ZP];
        e[0] = sxx * X + sxy * Y + sxz * Z;
        e[LZ * ZP] = sxy * X + syy * Y + syz * Z;
        e[2 * LZ * ZP] = sxz * X + syz * Y + szz * Z;
      }
      const int qz2 = LZ - fz;
      if (fz > 0 && qz2 != fz) {   // qz = LZ - fz: sz = -1
        cx<R>* e = e0 + qz2 * ZP;
        const cx<R> X = e[0], Y = e[LZ * ZP], Z = e[2 * LZ * ZP];
        e[0] = sxx * X + sxy * Y - sxz * Z;
        e[LZ * ZP] = sxy * X + syy * Y - syz * Z;
        e[2 * LZ * ZP] = szz * Z - sxz * X - syz * Y;
      }
    }
  }
  __syncthreads();
  // inverse along z, cropped to nz
  auto lds_ld = [&](int n) -> cx<R> { return slot[n * ZP]; };
  auto stg = [&](int k, cx<R> v) {
    if (k < nz) *elem(wsys, toff + (unsigned)(k - t) * plane) = v;
  };
  fft_pencil<R, LZ, T, +1, true, false, PAD_OUT>(lds_ld, stg, slot, ZP, t, valid, tw);
}

template <typename R, int L, int V, int K>
static void launch_zcol_k(const ZArgs<R>& a, int nsys, hipStream_t s) {
  using G = ZColGeo<R, L, V, K>;
  const int cols = a.ly * a.lx;
  const int blocks = ((cols + G::ZP - 1) / G::ZP) * nsys;
  hipLaunchKernelGGL((k_zconv_col<R, L, V, K>), dim3(blocks), dim3(3 * G::TZ * G::ZP), 0, s, a);
}

template <typename R, int L, int V>
static void launch_zcol(const ZArgs<R>& a, int nsys, hipStream_t s) {
  if (a.rooftop)
    launch_zcol_k<R, L, V, 1>(a, nsys, s);
  else
    launch_zcol_k<R, L, V, 0>(a, nsys, s);
}

// The kernel of a column-set variant: below 32 all are variant 0; where no
// column count is better off with variants 2 and 3 (from 288 on, and 2 at 192
// in FP32) they are variant 4, which also keeps the variants of a length equal
// bit for bit.
template <typename R>
constexpr int zcol_kernel(int l, int v) {
  return l < 32 ? 0 : (l >= 288 || (l == 192 && v == 2 && sizeof(R) == 4)) ? 4 : v;
}

template <typename R>
void launch_zconv(int L, const ZArgs<R>& a, int nsys, hipStream_t s) {
  const int nfy = nfold(a.ly), nfx = nfold(a.lx);
  switch (L) {
#define C(l)                                                                                      \
  case l: {                                                                                       \
    if (a.variant == 1) {                                                                         \
      if (a.rooftop) throw std::runtime_error("z pass: no mirror-column variant for rooftop spectra"); \
      using G = ZGeo<R, l>;                                                                       \
      const int blocks = nfy * ((nfx + G::ZP - 1) / G::ZP) * nsys;                                \
      hipLaunchKernelGGL((k_zconv_mirror<R, l>), dim3(blocks), dim3(3 * G::T * G::ZP), 0, s, a);  \
    } else if (l < 32 || a.variant == 0) {                                                        \
      launch_zcol<R, l, 0>(a, nsys, s);                                                           \
    } else if (a.variant == 2) {                                                                  \
      launch_zcol<R, l, zcol_kernel<R>(l, 2)>(a, nsys, s);                                        \
    } else if (a.variant == 3) {                                                                  \
      launch_zcol<R, l, zcol_kernel<R>(l, 3)>(a, nsys, s);                                        \
    } else {                                                                                      \
      launch_zcol<R, l, zcol_kernel<R>(l, 4)>(a, nsys, s);                                        \
    }                                                                                             \
    break;                                                                                        \
  }
    VIE_L_CASES(C)
#undef C
    default:
      bad_length("z pass", L);
  }
  check_launch("z pass");
}

}  // namespace vie
