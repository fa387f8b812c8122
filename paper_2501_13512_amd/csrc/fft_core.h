// Device FFT core: small DFTs in registers and a compile-time mixed-radix
// Stockham pipeline for one pencil.
//
// The 3-D convolution that accelerates the VIE product (the Toeplitz + FFT
// statement of Sec. I of the paper) is built from 1-D pencils of length
// L = 2^a 3^b.  A pencil is transformed by a chain of radix stages
// (autosort Stockham form): stage s with radix R and p = product of the
// earlier radices reads element b + m*L/R (m < R) for butterfly b, twiddles
// it by w^(m k) with w = exp(-+2 pi i / (p R)), k = b mod p, applies a
// length-R DFT and writes element (b - k) R + k + m p.  The first stage reads
// through a caller-supplied loader (HBM, coalesced across threads) and the
// last stage writes through a caller-supplied storer; the stages in between
// exchange data through LDS.  DIR = -1 is the forward transform
// exp(-2 pi i k n / L), DIR = +1 the unnormalised inverse.
#pragma once
#include "cx.h"

namespace vie {

// ---------------------------------------------------------------- small DFTs
template <int DIR, typename R>
__host__ __device__ __forceinline__ cx<R> rot_q(cx<R> a) {  // a * exp(DIR * i pi / 2)
  return DIR < 0 ? mul_mi(a) : mul_i(a);
}

__host__ __device__ __forceinline__ float fma1(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double fma1(double a, double b, double c) { return __builtin_fma(a, b, c); }
// HALF: the inputs v[RAD/2 ...] are zero (their values are not read), which
// spares the first of the log2(RAD) levels of additions.
// SPLIT: the products of the last level are rounded before they are added, so
// an output's value does not depend on whether its partner (the same product
// with the other sign) is formed as well.
template <bool SPLIT, typename R>
__host__ __device__ __forceinline__ R prod(R a, R b) {
  if constexpr (SPLIT) {
#pragma clang fp contract(off)
    return a * b;
  } else {
    return a * b;
  }
}
template <int RAD, int DIR, bool HALF = false, bool SPLIT = false, typename R>
__host__ __device__ __forceinline__ void dft(cx<R>* v) {
  static_assert(!HALF || RAD % 2 == 0, "an odd radix has no half");
  static_assert(!SPLIT || RAD <= 8, "the last level of radix 16 is not split");
  if constexpr (RAD == 1) {
  } else if constexpr (RAD == 2 && HALF) {
    v[1] = v[0];
  } else if constexpr (RAD == 2) {
    cx<R> a = v[0], b = v[1];
    v[0] = a + b;
    v[1] = a - b;
  } else if constexpr (RAD == 3) {
    const R c = R(-0.5);
    const R s = DIR < 0 ? R(-0.86602540378443864676) : R(0.86602540378443864676);
    cx<R> t1 = v[1] + v[2], t2 = v[1] - v[2];
    cx<R> m = v[0] + c * t1;
    cx<R> j = mk<R>(prod<SPLIT>(-s, t2.y), prod<SPLIT>(s, t2.x));  // i * s * t2
    v[0] = v[0] + t1;
    v[1] = m + j;
    v[2] = m - j;
  } else if constexpr (RAD == 4 && HALF) {
    const cx<R> e = v[0], o0 = v[1], o1 = rot_q<DIR>(v[1]);
    v[0] = e + o0;
    v[2] = e - o0;
    v[1] = e + o1;
    v[3] = e - o1;
  } else if constexpr (RAD == 4) {
    cx<R> e0 = v[0] + v[2], e1 = v[0] - v[2];
    cx<R> o0 = v[1] + v[3], o1 = rot_q<DIR>(v[1] - v[3]);
    v[0] = e0 + o0;
    v[2] = e0 - o0;
    v[1] = e1 + o1;
    v[3] = e1 - o1;
  } else if constexpr (RAD == 8) {
    constexpr int IN = HALF ? 2 : 4;
    cx<R> e[4], o[4];
#pragma unroll
    for (int i = 0; i < IN; ++i) {
      e[i] = v[2 * i];
      o[i] = v[2 * i + 1];
    }
    dft<4, DIR, HALF>(e);
    dft<4, DIR, HALF>(o);
    const R h = R(0.70710678118654752440);
    const R sg = DIR < 0 ? R(-1) : R(1);
    cx<R> t1 = mk<R>(prod<SPLIT>(h, o[1].x - sg * o[1].y), prod<SPLIT>(h, o[1].y + sg * o[1].x));     // w8^1
    cx<R> t2 = rot_q<DIR>(o[2]);                                                                      // w8^2
    cx<R> t3 = mk<R>(prod<SPLIT>(h, -o[3].x - sg * o[3].y), prod<SPLIT>(h, -o[3].y + sg * o[3].x));   // w8^3
    v[0] = e[0] + o[0];
    v[4] = e[0] - o[0];
    v[1] = e[1] + t1;
    v[5] = e[1] - t1;
    v[2] = e[2] + t2;
    v[6] = e[2] - t2;
    v[3] = e[3] + t3;
    v[7] = e[3] - t3;
  } else if constexpr (RAD == 16) {
    constexpr int IN = HALF ? 4 : 8;
    cx<R> e[8], o[8];
#pragma unroll
    for (int i = 0; i < IN; ++i) {
      e[i] = v[2 * i];
      o[i] = v[2 * i + 1];
    }
    dft<8, DIR, HALF>(e);
    dft<8, DIR, HALF>(o);
    const R c1 = R(0.92387953251128675613), s1 = R(0.38268343236508977173);
    const R h = R(0.70710678118654752440);
    const R sg = DIR < 0 ? R(-1) : R(1);
    // w16^k = cos(2 pi k/16) + sg * i sin(2 pi k/16)
    const R cr[8] = {R(1), c1, h, s1, R(0), -s1, -h, -c1};
    const R ci[8] = {R(0), s1, h, c1, R(1), c1, h, s1};
    v[0] = e[0] + o[0];
    v[8] = e[0] - o[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) {
      cx<R> t;
      if (k == 4) {
        t = rot_q<DIR>(o[4]);
      } else {
        const R wr = cr[k], wi = sg * ci[k];
        if (k == 2 && DIR < 0)
          // wi = -wr: which of the two products is fused would be the compiler's
          // choice, which differs with the code around (length 256 in FP32)
          t = mk<R>(fma1(-o[k].y, wi, o[k].x * wr), fma1(o[k].y, wr, o[k].x * wi));
        else
          t = mk<R>(o[k].x * wr - o[k].y * wi, o[k].x * wi + o[k].y * wr);
      }
      v[k] = e[k] + t;
      v[k + 8] = e[k] - t;
    }
  } else {
    static_assert(RAD == 2, "unsupported radix");
  }
}

// ---------------------------------------------------------------- plans
template <int... Rs>
struct Radices {};

template <int L>
struct Plan;
template <> struct Plan<1> { using type = Radices<>; };
template <> struct Plan<2> { using type = Radices<2>; };
template <> struct Plan<3> { using type = Radices<3>; };
template <> struct Plan<4> { using type = Radices<4>; };
template <> struct Plan<6> { using type = Radices<2, 3>; };
template <> struct Plan<8> { using type = Radices<8>; };
template <> struct Plan<12> { using type = Radices<4, 3>; };
template <> struct Plan<16> { using type = Radices<16>; };
template <> struct Plan<24> { using type = Radices<8, 3>; };
template <> struct Plan<32> { using type = Radices<8, 4>; };
template <> struct Plan<36> { using type = Radices<4, 3, 3>; };
template <> struct Plan<48> { using type = Radices<16, 3>; };
template <> struct Plan<64> { using type = Radices<8, 8>; };
template <> struct Plan<72> { using type = Radices<8, 3, 3>; };
template <> struct Plan<96> { using type = Radices<8, 4, 3>; };
template <> struct Plan<128> { using type = Radices<16, 8>; };
template <> struct Plan<144> { using type = Radices<16, 3, 3>; };
template <> struct Plan<192> { using type = Radices<16, 4, 3>; };
template <> struct Plan<256> { using type = Radices<16, 16>; };
template <> struct Plan<288> { using type = Radices<8, 4, 3, 3>; };
template <> struct Plan<384> { using type = Radices<16, 8, 3>; };
template <> struct Plan<512> { using type = Radices<8, 8, 8>; };

template <class Rad>
struct RadInfo;
template <>
struct RadInfo<Radices<>> {
  static constexpr int first = 1;
  static constexpr int nstages = 0;
  static constexpr int rmin = 1 << 30;
  static constexpr int rmax = 1;
};
template <int R0, int... Rs>
struct RadInfo<Radices<R0, Rs...>> {
  static constexpr int first = R0;
  static constexpr int nstages = 1 + sizeof...(Rs);
  static constexpr int rmin = R0 < RadInfo<Radices<Rs...>>::rmin ? R0 : RadInfo<Radices<Rs...>>::rmin;
  static constexpr int rmax = R0 > RadInfo<Radices<Rs...>>::rmax ? R0 : RadInfo<Radices<Rs...>>::rmax;
};

// Largest number of butterflies of any stage = L / smallest radix; a pencil
// uses at most that many threads.  With min_butterflies (L / largest radix)
// threads no thread idles in any stage; stages with more butterflies then
// give each thread several.
template <int L>
struct PlanInfo {
  using rad = typename Plan<L>::type;
  static constexpr int nstages = RadInfo<rad>::nstages;
  static constexpr int max_butterflies = nstages == 0 ? 1 : L / RadInfo<rad>::rmin;
  static constexpr int min_butterflies = nstages == 0 ? 1 : L / RadInfo<rad>::rmax;
};

// ---------------------------------------------------------------- pipeline
// Twiddle table tw[t] = exp(-2 pi i t / L), t < L, in HBM (shared, cached).
//
// A thread's twiddles depend on its place in the pencil only, so they are
// fetched once, before the pencil's data, where the registers allow it
// (TwRegs): loaded at their use they put one more trip to the L2 on the path
// of every stage, and again for every pencil a workgroup takes in turn.  Up to
// 32 registers are spent on them; longer plans load them at their use.
template <class Rad, int L, int T, int P>
struct TwCount {
  static constexpr int value = 0;
};
template <int RAD, int... Rest, int L, int T, int P>
struct TwCount<Radices<RAD, Rest...>, L, T, P> {
  static constexpr int here = P > 1 ? (RAD - 1) * ((L / RAD + T - 1) / T) : 0;
  static constexpr int value = here + TwCount<Radices<Rest...>, L, T, P * RAD>::value;
};

template <typename R, int L, int T, bool HOLD = true>
struct TwRegs {
  static constexpr int count = TwCount<typename Plan<L>::type, L, T, 1>::value;
  static constexpr bool held = HOLD && count * (int)sizeof(cx<R>) <= 32 * 4;
  const cx<R>* __restrict__ tab;
  cx<R> w[held && count > 0 ? count : 1];

  template <int P, int AT, int RAD, int... Rest>
  __device__ __forceinline__ void fetch(int t, Radices<RAD, Rest...>) {
    constexpr int NPT = (L / RAD + T - 1) / T;
    if constexpr (P > 1) {
#pragma unroll
      for (int q = 0; q < NPT; ++q) {
        const int k = (t + q * T) % P;
#pragma unroll
        for (int m = 1; m < RAD; ++m) w[AT + q * (RAD - 1) + m - 1] = tab[(unsigned)(m * k * (L / (P * RAD)))];
      }
    }
    if constexpr (sizeof...(Rest) > 0) fetch<P * RAD, AT + (P > 1 ? NPT * (RAD - 1) : 0)>(t, Radices<Rest...>{});
  }
  // t: the thread's place in its pencil
  __device__ __forceinline__ TwRegs(const cx<R>* __restrict__ tw, int t) : tab(tw) {
    if constexpr (held && count > 0) fetch<1, 0>(t, typename Plan<L>::type{});
  }
  // twiddle m of butterfly t + q T in the stage whose twiddles start at AT
  template <int AT, int RAD, int P>
  __device__ __forceinline__ cx<R> at(int q, int m, int k) const {
    if constexpr (held)
      return w[AT + q * (RAD - 1) + m - 1];
    else
      return tab[(unsigned)(m * k * (L / (P * RAD)))];   // unsigned 32-bit offset from a uniform base
  }
};

// v w (forward) or v conj(w), with its fused operations spelled out: kernels
// that hold their twiddles and kernels that load them agree bit for bit, which
// they need not when the compiler chooses what to contract.
template <int DIR, typename R>
__device__ __forceinline__ cx<R> twiddled(cx<R> v, cx<R> w) {
  const R p = v.y * w.y, q = v.x * w.y;
  return DIR < 0 ? mk<R>(fma1(v.x, w.x, -p), fma1(v.y, w.x, q)) : mk<R>(fma1(v.x, w.x, p), fma1(v.y, w.x, -q));
}

// What half of an even-length pencil is known at compile time: every axis of
// a product is padded to at least twice its voxels less one, so a forward
// transform's upper half of inputs is zero and an inverse's upper half of
// outputs is dropped.
enum Pad { PAD_NONE = 0, PAD_IN = 1, PAD_OUT = 2 };
// elements of a padded pencil that can be voxels
__host__ __device__ constexpr int half_padded(int l) { return l % 2 == 0 ? l / 2 : (l + 1) / 2; }
// PadIn: whether the first stage of a PAD_IN transform leaves out its upper
// inputs, and the elements [0, reads) that it asks its loader for.  Length 3
// has no even first radix: it reads all three, of which two can be voxels.
template <int L>
struct PadIn {
  static constexpr bool half = L % 2 == 0 && RadInfo<typename Plan<L>::type>::first % 2 == 0;
  static constexpr int reads = half ? L / 2 : L;
  static_assert(reads >= half_padded(L), "a voxel would not be read");
};

// Place of element i of a pencil in its LDS slot: consecutive elements LS
// apart, or, for pencils that lie along their lanes (rows), one element left
// out after every RAD.  A stage's butterflies write RAD elements apart, which
// without the gaps is the same banks for all lanes (rows of length 256: 28
// conflict cycles per LDS instruction; the 128x128x32 FP64 product took 176 us
// with them and takes 171).
template <int RAD>
struct RowSlot {};
__device__ __forceinline__ int slot_at(int ls, int i) { return i * ls; }
template <int RAD>
__device__ __forceinline__ int slot_at(RowSlot<RAD>, int i) {
  return RAD > 1 ? i + i / RAD : i;
}

// One stage.  Threads t < T of a pencil cooperate; `lds` points at element 0
// of this pencil's LDS slot and consecutive elements are `ls` apart.  All
// threads of the workgroup must call every stage (barriers inside).
// LDLDS: the loader reads this pencil's LDS slot; STLDS: the storer writes
// it.  Then the first (last) stage separates its reads from its writes by a
// barrier, since the transform runs in place in the slot.
template <typename R, int L, int T, int DIR, int PAD, int RAD, int P, int AT, bool FIRST, bool LAST, bool LDLDS,
          bool STLDS, class Load, class Store, class Slot, bool HOLD>
__device__ __forceinline__ void fft_stage(Load& ld, Store& st, cx<R>* lds, Slot ls, int t, bool tvalid,
                                          const TwRegs<R, L, T, HOLD>& tw) {
  constexpr int NB = L / RAD;
  constexpr int NPT = (NB + T - 1) / T;
  constexpr bool READS_SLOT = !FIRST || LDLDS;
  constexpr bool WRITES_SLOT = !LAST || STLDS;
  constexpr bool HIN = FIRST && PAD == PAD_IN && PadIn<L>::half;
  // the last stage's outputs b + m P, b < P: none of m from here on is kept
  // (radix 16 forms them all: it would spare a ninth of its additions)
  constexpr int MOUT = LAST && PAD == PAD_OUT && L % 2 == 0 && RAD <= 8 ? (RAD + 1) / 2 : RAD;
  cx<R> v[NPT][RAD];
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int b = t + q * T;
    if (tvalid && (NB % T == 0 || b < NB)) {
#pragma unroll
      for (int m = 0; m < (HIN ? RAD / 2 : RAD); ++m) {
        const int idx = b + m * NB;
        if constexpr (FIRST)
          v[q][m] = ld(idx);
        else
          v[q][m] = lds[slot_at(ls, idx)];
      }
    }
  }
  if constexpr (READS_SLOT && WRITES_SLOT) __syncthreads();
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int b = t + q * T;
    if (tvalid && (NB % T == 0 || b < NB)) {
      const int k = (P == 1) ? 0 : (b % P);
      if constexpr (P > 1) {
#pragma unroll
        for (int m = 1; m < RAD; ++m) v[q][m] = twiddled<DIR>(v[q][m], tw.template at<AT, RAD, P>(q, m, k));
      }
      dft<RAD, DIR, HIN, MOUT != RAD>(v[q]);
      const int j = (b - k) * RAD + k;
#pragma unroll
      for (int m = 0; m < MOUT; ++m) {
        if constexpr (LAST)
          st(j + m * P, v[q][m]);
        else
          lds[slot_at(ls, j + m * P)] = v[q][m];
      }
    }
  }
  if constexpr (WRITES_SLOT) __syncthreads();
}

template <typename R, int L, int T, int DIR, int PAD, int P, int AT, bool FIRST, bool LDLDS, bool STLDS, class Load,
          class Store, class Slot, bool HOLD, int RAD, int... Rest>
__device__ __forceinline__ void fft_stages(Load& ld, Store& st, cx<R>* lds, Slot ls, int t, bool tvalid,
                                           const TwRegs<R, L, T, HOLD>& tw, Radices<RAD, Rest...>) {
  constexpr bool LAST = sizeof...(Rest) == 0;
  constexpr int NEXT = AT + (P > 1 ? (RAD - 1) * ((L / RAD + T - 1) / T) : 0);
  fft_stage<R, L, T, DIR, PAD, RAD, P, AT, FIRST, LAST, LDLDS, STLDS>(ld, st, lds, ls, t, tvalid, tw);
  if constexpr (!LAST)
    fft_stages<R, L, T, DIR, PAD, P * RAD, NEXT, false, LDLDS, STLDS>(ld, st, lds, ls, t, tvalid, tw, Radices<Rest...>{});
}

// Transform one pencil of length L: x_n = ld(n) (n < L) -> st(k, X_k).
// Threads t in [0, T) of the pencil take part; tvalid = false threads still
// hit the barriers but touch no data.  The pencil's LDS slot is the exchange
// buffer between stages; see fft_stage for LDLDS / STLDS.  With PAD_IN ld is
// asked for n < PadIn<L>::reads; with PAD_OUT st may not be given k >= L/2.
template <typename R, int L, int T, int DIR, bool LDLDS = false, bool STLDS = false, int PAD = PAD_NONE, class Load,
          class Store, class Slot, bool HOLD>
__device__ __forceinline__ void fft_pencil(Load ld, Store st, cx<R>* lds, Slot ls, int t, bool tvalid,
                                           const TwRegs<R, L, T, HOLD>& tw) {
  using rad = typename Plan<L>::type;
  if constexpr (RadInfo<rad>::nstages == 0) {
    if (tvalid && t == 0) st(0, ld(0));
    if constexpr (STLDS) __syncthreads();
  } else {
    fft_stages<R, L, T, DIR, PAD, 1, 0, true, LDLDS, STLDS>(ld, st, lds, ls, t, tvalid, tw, rad{});
  }
}

// The same with the twiddles fetched on the spot.
template <typename R, int L, int T, int DIR, bool LDLDS = false, bool STLDS = false, int PAD = PAD_NONE, class Load,
          class Store, class Slot>
__device__ __forceinline__ void fft_pencil(Load ld, Store st, cx<R>* lds, Slot ls, int t, bool tvalid,
                                           const cx<R>* __restrict__ tw) {
  const TwRegs<R, L, T> w(tw, t);
  fft_pencil<R, L, T, DIR, LDLDS, STLDS, PAD>(ld, st, lds, ls, t, tvalid, w);
}

}  // namespace vie
