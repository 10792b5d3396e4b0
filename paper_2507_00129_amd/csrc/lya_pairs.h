// What the pair kernels (xi and its backward pass) share: bin coordinates as
// 2^20 + x, wave-uniform pixel loads and the hand-out of work.
#pragma once
#include <type_traits>

#include "lya_bin.h"
#include "lya_common.h"

namespace lya {

constexpr unsigned kRunMax = 32;
constexpr int kWaitAll = 0x7fffffff;

// 2^20 and its upper word: 2^20 + x has floor(x) in the low bits of its upper
// word and the fraction in its lower word, in units of 2^-32.
constexpr double kMagic = 1048576.0;
constexpr uint32_t kMagicHi = 0x41300000u;
constexpr double kGuard = 1e-8;        // edge guard, bins (see kUniformRange)
constexpr double kWideGuard = 0.25;    // where every pair in range goes by the edges
constexpr uint32_t kGuard2 = 86u;      // 2 kGuard in units of 2^-32

// How a kernel bins: uniform edges whose first ones are both 0 (the lower-edge tests
// vanish), any uniform edges, or by the edge arrays.
enum : int { kZeroEdges, kUniformEdges, kAnyEdges };
inline int axis_form(const GridDev& g) {
  return g.exact_all ? kAnyEdges : (g.zero_lo_par && g.zero_lo_perp ? kZeroEdges : kUniformEdges);
}

// A lane's interval [lo, hi) on an axis binned by its edges: bin k, or below the first
// edge (k = -1) or from the last one on (k = n).  e[-1] and e[n + 1] are -1 and infinity.
// Consecutive pixels mostly stay in it, two compares, or step to the next one, one load;
// a search from the mean bin width's guess took 6 to 10 dependent loads an axis.
struct EdgeBin {
  double lo, hi;
  int k;
  __device__ __forceinline__ bool holds(double r) const { return (r >= lo) & (r < hi); }
  // From any guess of the bin (a NaN is below the first edge, which does not hold it).
  __device__ __forceinline__ void search(double r, const double* e, int n, int guess) {
    k = bin_exact(r, e, n, guess);
    if (k < 0 && r >= e[n]) k = n;
    lo = e[k];
    hi = e[k + 1];
  }
  // To the neighbouring interval on r's side; the caller looks whether that holds it.
  __device__ __forceinline__ void step(double r, const double* e, int n) {
    const bool up = r >= hi;
    k = up ? min(k + 1, n) : max(k - 1, -1);
    const double at = e[up ? k + 1 : k], from = up ? hi : lo;
    lo = up ? from : at;
    hi = up ? at : from;
  }
};

// Loads through the constant address space: with a wave-uniform address the
// compiler emits scalar (SMEM) loads.  Native vector types are used because
// class copies cannot bind to address-space-qualified objects.
typedef int lya_i16 __attribute__((ext_vector_type(16)));
typedef int lya_i4 __attribute__((ext_vector_type(4)));
typedef int lya_i8 __attribute__((ext_vector_type(8)));
typedef int lya_i2 __attribute__((ext_vector_type(2)));
#define LYA_CONST(T, p) (*(const __attribute__((address_space(4))) T*)(p))

// A pixel of f in scalar registers.
template <typename T> struct UPix { double d; T wd, w; };

// Four FP32 records or two FP64 records (64 bytes) per scalar load.
template <typename T> struct Batch;
template <> struct Batch<float> {
  static constexpr int N = 4;
  UPix<float> r[4];
  __device__ __forceinline__ void load(const XRec32* p) {
    const lya_i16 v = LYA_CONST(lya_i16, p);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      r[u] = UPix<float>{__hiloint2double(v[4 * u + 1], v[4 * u]), __int_as_float(v[4 * u + 2]), __int_as_float(v[4 * u + 3])};
  }
};
template <> struct Batch<double> {
  static constexpr int N = 2;
  UPix<double> r[2];
  __device__ __forceinline__ void load(const Rec64* p) {
    const lya_i16 v = LYA_CONST(lya_i16, p);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      r[u] = UPix<double>{__hiloint2double(v[8 * u + 1], v[8 * u]), __hiloint2double(v[8 * u + 3], v[8 * u + 2]),
                          __hiloint2double(v[8 * u + 5], v[8 * u + 4])};
  }
};
__device__ __forceinline__ UPix<float> load_pix(const XRec32* p) {
  const lya_i4 v = LYA_CONST(lya_i4, p);
  return UPix<float>{__hiloint2double(v[1], v[0]), __int_as_float(v[2]), __int_as_float(v[3])};
}
__device__ __forceinline__ UPix<double> load_pix(const Rec64* p) {
  const lya_i8 v = LYA_CONST(lya_i8, p);
  return UPix<double>{__hiloint2double(v[1], v[0]), __hiloint2double(v[3], v[2]), __hiloint2double(v[5], v[4])};
}

template <typename T> struct RecOf;
template <> struct RecOf<float> { using type = XRec32; };
template <> struct RecOf<double> { using type = Rec64; };

__device__ __forceinline__ uint64_t ballot(bool x) { return __builtin_amdgcn_ballot_w64(x); }
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ double uniform(double x) {
  return __hiloint2double(uniform(__double2hiint(x)), uniform(__double2loint(x)));
}

// Coefficients of a lane without a pixel: up = 2^20 + guard - e0 / dr + 2^-17 |D_i - D_j|,
// ut = 1.5 * 2^20 + 0.5: outside the grid and, for any usual unit of D, off the edge guard,
// which would send every batch of the wave to the exact path (as zeros would: 0.16 ms
// instead of 0.09 for 234 forests of 47 pixels).  Written out: the compiler would keep
// the constants in registers through the pair loop.
__device__ __forceinline__ void past_end(double& cp, double& bt) {
  int c, h, l;
  asm volatile("v_mov_b32_e32 %0, 0x3ee00000\n\tv_mov_b32_e32 %1, 0x41380000\n\tv_mov_b32_e32 %2, 0x80000000"
               : "=v"(c), "=v"(h), "=v"(l));
  cp = __hiloint2double(c, 0);
  bt = __hiloint2double(h, l);
}

// A wave's next `grab` tickets of n, the first of which is returned (~0u: none left),
// from kXiCounters counters beyond the first `base` tickets, the workgroup's own
// counter first.  gone (LDS): counters the workgroup has found empty.  Nobody asks where
// all tickets were dealt out beforehand: a round of 16 atomics that tell 8192 waves so
// was two thirds of a small call's kernel (290 forests of 35 pixels: 83 us, 27 without).
__device__ __forceinline__ unsigned grab_ticket(unsigned* counter, unsigned base, unsigned grab, unsigned n, int* gone) {
  unsigned t = ~0u;
  if (base >= n) return t;
  if ((threadIdx.x & 63) == 0) {
    for (int k = *(volatile int*)gone; k < kXiCounters;) {
      const unsigned w = ((blockIdx.x >> 3) + k) % kXiCounters;
      t = base + (atomicAdd(counter + w * kXiCounterStride, 1u) * kXiCounters + w) * grab;
      if (t < n) break;
      t = ~0u;
      k = max(k + 1, atomicMax(gone, k + 1));
    }
  }
  return (unsigned)uniform((int)t);
}

}  // namespace lya
