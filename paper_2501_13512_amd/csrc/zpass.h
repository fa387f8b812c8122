// Pieces shared by the z-pass kernels (the product's third pass: z forward,
// spectral multiply, z inverse).
#pragma once
#include <stdexcept>
#include <string>

#include "cx.h"
#include "kernels.h"

namespace vie {

#define VIE_L_CASES(F)                                                                                    \
  F(1) F(2) F(3) F(4) F(6) F(8) F(12) F(16) F(24) F(32) F(36) F(48) F(64) F(72) F(96) F(128) F(144) F(192) F(256) \
      F(288) F(384) F(512)

[[noreturn]] static void bad_length(const char* what, int L) {
  throw std::runtime_error(std::string("unsupported FFT length for ") + what + ": " + std::to_string(L));
}

static void check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw std::runtime_error(std::string("kernel launch failed (") + what + "): " + hipGetErrorString(e));
}

constexpr int pow2_ceil(int v) {
  int p = 1;
  while (p < v) p *= 2;
  return p;
}
constexpr int pow2_floor(int v) {
  int p = 1;
  while (p * 2 <= v) p *= 2;
  return p;
}
constexpr int cmin(int a, int b) { return a < b ? a : b; }
constexpr int cmax(int a, int b) { return a > b ? a : b; }

__device__ __forceinline__ bool sys_active(const int* status, int s) {
  return status == nullptr || status[s] == ST_ACTIVE;
}

template <typename R>
__device__ __forceinline__ cx<R> czero() {
  return mk<R>(R(0), R(0));
}

// Element i of an array whose byte size is below 4 GiB: the byte offset is
// formed in 32 bits, so the access can use a uniform base register plus a
// 32-bit per-lane offset.
template <typename T>
__device__ __forceinline__ T* elem(T* base, unsigned i) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ const T* elem(const T* base, unsigned i) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (unsigned)sizeof(T));
}

// Workgroup b of n runs on XCD b % 8 (round-robin dispatch).  Renumber so
// that each XCD takes one contiguous range of the logical order: work that
// shares data then shares that XCD's L2.
__device__ __forceinline__ int xcd_chunked(int b, int n) {
  constexpr int NX = 8;
  const int q = n / NX, r = n - q * NX;
  const int x = b % NX, l = b / NX;
  return x * q + min(x, r) + l;
}

// Logical row i -> qy in the order 0, 1, L-1, 2, L-2, ...: rows that share
// an octant row of the spectra (qy and L - qy) are adjacent.
__device__ __forceinline__ int mirror_paired_row(int i, int L) {
  if (i == 0) return 0;
  const int k = (i + 1) >> 1;
  return (i & 1) ? k : L - k;
}

template <typename R>
struct ZArgs {
  int nz, ly, lx;
  int variant;   // 0, 2, 3, 4: column sets (ZColGeo); 1: mirror columns
  int rooftop;   // spectral multiply of the rooftop discretisation (column sets only)
  int64_t wstride, sstride;
  cx<R>* work;
  const cx<R>* spec;
  const cx<R>* const* spec_tab;   // per-system spectra (null: spec + sys sstride)
  const int* status;
  const cx<R>* tw;
};

// The z pass in one precision (zconv32.hip, zconv64.hip; a.variant picks the
// kernel).
template <typename R>
void launch_zconv(int L, const ZArgs<R>& a, int nsys, hipStream_t s);

}  // namespace vie
