// Device-side helpers shared by the gfx950 kernels of libfdtd.
#pragma once
#include "fd_internal.h"

#include <type_traits>

namespace fdk {

constexpr float kTwoPiF = 6.28318530717958647692f;

// ------------------------------------------------------------------ Philox
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = 0xD2511F53u * c[0];
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]);
    const uint32_t lo1 = 0xCD9E8D57u * c[2];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]);
    const uint32_t y0 = hi1 ^ c[1] ^ k0;
    const uint32_t y2 = hi0 ^ c[3] ^ k1;
    c[0] = y0; c[1] = lo1; c[2] = y2; c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

__device__ __forceinline__ float u24(uint32_t x) {
  return (static_cast<float>(x >> 8) + 0.5f) * 5.9604644775390625e-8f;  // 2^-24
}

// Three standard normals for (step n, cell o): Box-Muller on the uniform pairs.
__device__ __forceinline__ void normals3(uint32_t n, uint32_t o, uint32_t k0, uint32_t k1, float g[3]) {
  uint32_t c[4] = {n, o, 0u, 2u};
  philox10(c, k0, k1);
  const float r0 = sqrtf(-2.0f * logf(u24(c[0])));
  float s0, c0;
  sincosf(kTwoPiF * u24(c[1]), &s0, &c0);
  const float r1 = sqrtf(-2.0f * logf(u24(c[2])));
  g[0] = r0 * c0;
  g[1] = r0 * s0;
  g[2] = r1 * cosf(kTwoPiF * u24(c[3]));
}

// Field arrays are reached through pointers stored in the plan's descriptor, so
// the compiler cannot infer their address space; every pointer is cast to the
// global space (1) so loads and stores are global_* instructions, and the
// descriptor itself to the constant space (4) so its fields are scalar loads.
typedef __attribute__((address_space(1))) float gf;
typedef __attribute__((address_space(1))) double gd;
typedef __attribute__((address_space(1))) uint8_t gu8;
typedef __attribute__((address_space(4))) fd_desc cdesc;
typedef __attribute__((address_space(4))) fd_mat cmat;
typedef __attribute__((address_space(4))) const float cfloat;

__device__ __forceinline__ gf* G(float* p) { return (gf*)p; }
__device__ __forceinline__ const gf* G(const float* p) { return (const gf*)p; }
__device__ __forceinline__ gd* G(double* p) { return (gd*)p; }
__device__ __forceinline__ const gd* G(const double* p) { return (const gd*)p; }

// A field array indexed with a 32-bit element index: the byte offset is formed
// in 32 bits and zero-extended, so loads and stores take the scalar-base +
// 32-bit vector-offset form (one VGPR per address, no 64-bit address adds).
// Valid for arrays below 4 GiB, which every per-cell array is (at most 2^30
// cells of 4 bytes).
typedef __attribute__((address_space(1))) char gchar;
typedef __attribute__((address_space(1))) const char gcchar;
template <class T>
struct R32 {
  __attribute__((address_space(1))) T* p;
  __device__ __forceinline__ __attribute__((address_space(1))) T& operator[](uint32_t i) const {
    typedef __attribute__((address_space(1))) T gT;
    typedef typename std::conditional<std::is_const<T>::value, gcchar, gchar>::type gb;
    return *(gT*)((gb*)p + (size_t)(i * (uint32_t)sizeof(T)));
  }
};

__device__ __forceinline__ int nxt(int i, int n, int per) { return i + 1 < n ? i + 1 : (per ? 0 : -1); }
__device__ __forceinline__ int prv(int i, int n, int per) { return i > 0 ? i - 1 : (per ? n - 1 : -1); }

// index along an axis after periodic wrap, or -1 beyond a PEC wall
__device__ __forceinline__ int wrap(int i, int n, int per) {
  if (i >= 0 && i < n) return i;
  if (!per) return -1;
  const int r = i % n;
  return r < 0 ? r + n : r;
}

// family of component c within axis w's two stored psi arrays
__device__ __forceinline__ int fam(int c, int w) { return c == (w + 1) % 3 ? 0 : 1; }

// Workgroup barrier for LDS traffic only.  Within a step no workgroup reads
// global memory that another thread of the step writes (inputs and outputs are
// separate buffers), so the barrier waits for outstanding LDS operations but
// not for global loads in flight: loads issued for the next z-plane keep
// streaming across it.
__device__ __forceinline__ void lds_barrier() {
  __asm__ __volatile__("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Deterministic block sum (fixed shuffle tree, then wave partials in order).
__device__ inline double block_sum(double v, double* sred) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  lds_barrier();
  if (lane == 0) sred[w] = v;
  lds_barrier();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) r += sred[q];
  return r;
}

// (hi, lo) += inc as an unevaluated FP32 pair (Knuth's two-sum, then renormalise).
__device__ __forceinline__ void two_sum(float& hi, float& lo, float inc) {
  const float s = hi + inc;
  const float bb = s - hi;
  const float err = (hi - (s - bb)) + (inc - bb);
  const float l = lo + err;
  const float h2 = s + l;
  lo = l - (h2 - s);
  hi = h2;
}

}  // namespace fdk
