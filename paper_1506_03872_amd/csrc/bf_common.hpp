// bf_common.hpp -- what the brute-force kernels share: precisions, the GEMM
// arguments, the bins of pass A and the conversions of the inputs.
#pragma once

#include "mad_common.hpp"
#include "plan.hpp"

namespace mad {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef int i8v __attribute__((ext_vector_type(8)));

enum Prec { kF32 = 0, kBF16 = 1, kFP8 = 2 };

// element bytes, k per MFMA, k per LDS chunk (a 128-byte row slice)
template <int P> struct PrecT;
template <> struct PrecT<kF32> {
  static constexpr int EB = 4, KS = 2, KC = 32;
};
template <> struct PrecT<kBF16> {
  static constexpr int EB = 2, KS = 16, KC = 64;
};
template <> struct PrecT<kFP8> {
  static constexpr int EB = 1, KS = 64, KC = 128;
};

__device__ __forceinline__ uint8_t to_fp8(float x) {
  // round to nearest even into e4m3; |x| < 2^7 after scaling
  const unsigned pk = __builtin_amdgcn_cvt_pk_fp8_f32(x, 0.0f, 0, false);
  return (uint8_t)(pk & 0xff);
}

__device__ __forceinline__ uint16_t to_bf16(float x) {
  // round to nearest even (inputs are finite)
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// norms, rounding floor and scale of one vector from its sums and largest |x|
template <int P>
__device__ __forceinline__ VecInfo vec_info(double s2, double s1, float mx) {
  float scale = 1.0f, eta = 0.0f;
  if (P == kFP8) {
    int e = 0;
    if (mx > 0.0f) (void)frexpf(mx, &e);  // mx < 2^e
    // scaled max < 2^7; 1 / scale stays a normal float (an E8M0 exponent)
    if (e < -119) e = -119;
    scale = ldexpf(1.0f, 7 - e);
    eta = ldexpf(1.0f, -10) / scale;      // half the e4m3 subnormal step
  } else if (P == kBF16) {
    eta = ldexpf(1.0f, -134);
  }
  VecInfo vi;
  vi.n2 = (float)(sqrt(s2) * (1.0 + 1e-6));
  vi.n1 = (float)(s1 * (1.0 + 1e-6));
  vi.eta = eta;
  vi.inv_s = 1.0f / scale;
  return vi;
}

// the scale that vec_info took (a power of two, so its inverse is exact)
template <int P>
__device__ __forceinline__ float vec_scale(const VecInfo& vi) {
  return P == kFP8 ? 1.0f / vi.inv_s : 1.0f;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

struct GemmArgs {
  const void* A;  // rows of Kp elements
  const void* B;
  const VecInfo* ia;
  const VecInfo* ib;
  int64_t m_rows;  // rows of A used
  int64_t a_stride_rows;  // A row i of this pass is row i*stride of the copy
  int64_t m_key;   // row index multiplier for keys (= stride)
  int64_t n, Kp;
  float kappa;     // relative margin factor on ||a||_2 ||b||_2
  float onepu;     // 1 + u
  float d_f;       // d (for the eta * eta term)
  // pass A
  int64_t target;  // rank of the bound that tau is taken at
  unsigned* hist;
  const unsigned* maxes;  // n2, n1, eta maxima of A, then (+4) of B
  int screen;      // 1: no error margin (screening by the computed value)
  int coarse;      // 1: fbin32's bins (screening, or a t-th bound below the
                   // finer ones)
  float mg_max;    // margin upper bound over all pairs (cheap pre-test)
  // pass B
  const unsigned* tau_bits;  // lower bound (float bits)
  float* cval;     // computed value of each survivor
  uint64_t* ckey;
  int64_t ccap;
  unsigned long long* ccount;
};

// monotone 11-bit digit of a non-negative float (exponent and the top 3
// mantissa bits); bin b holds the floats with bits in [b << 20, (b+1) << 20)
__device__ __forceinline__ int fbin32(uint32_t bits) {
  return (int)(bits >> 20) & 2047;
}

// Pass A's bins of the bounds.  Screening takes fbin32's 2048 (their edges
// are part of its result: the pairs it re-ranks are those above one).  The
// certified filter's result does not depend on tau, only its survivors do:
// it counts the lower bounds |c^| - margin in 1024 bins, 32 per octave over
// the 8 octaves below the largest possible |c| (bins 768 up) and 4 per
// octave over the 192 below those, and the upper bounds |c^| + margin in
// 1024 more of the same edges, which say how many pairs will pass.  (With
// fbin32's the edge lay up to 12% under the t-th bound and let 1.7e6 pairs
// through at 1e5 x 1e6 x 256 in bf16.)  fine0 is the first fine digit, a
// multiple of 8, so that it is a coarse edge too; -1: fbin32's bins.
constexpr int kUpperBins = 1024;  // first bin of the upper bounds

struct BoundBins {
  int fine0;
  __device__ __forceinline__ int bin(float v) const {
    const uint32_t bits = __float_as_uint(v);
    if (fine0 < 0) return fbin32(bits);
    const int f = (int)(bits >> 18) - fine0;
    if (f >= 0) return f < 256 ? 768 + f : 1023;
    const int c = 768 - (fine0 >> 3) + (int)(bits >> 21);
    return c > 0 ? c : 0;
  }
  // float bits of the bin's lower edge
  __device__ __forceinline__ unsigned edge(int b) const {
    if (b <= 0) return 0u;
    if (fine0 < 0) return (unsigned)b << 20;
    if (b >= 768) return (unsigned)(fine0 + b - 768) << 18;
    const int c = b - 768 + (fine0 >> 3);
    return c > 0 ? (unsigned)c << 21 : 0u;
  }
  // bins of lower bounds: [0, count)
  __device__ __forceinline__ int count() const {
    return fine0 < 0 ? 2048 : kUpperBins;
  }
};

__device__ __forceinline__ BoundBins bound_bins(const unsigned* maxes,
                                                bool coarse) {
  BoundBins r;
  r.fine0 = -1;
  if (!coarse) {
    // |c| <= ||a||_2 ||b||_2 (a larger value falls in the top bin)
    const float top = __uint_as_float(maxes[0]) * __uint_as_float(maxes[4]);
    const int hi = (int)(__float_as_uint(top) >> 18) | 7;
    r.fine0 = hi > 255 ? hi - 255 : 0;
  }
  return r;
}

// one value of pass A into a histogram
__device__ __forceinline__ void count_bounds(const BoundBins& bins, float c,
                                             float mg, unsigned* hist) {
  const float low = fabsf(c) - mg;
  if (low > 0.0f) atomicAdd(&hist[bins.bin(low)], 1u);
  if (bins.fine0 >= 0)
    atomicAdd(&hist[kUpperBins + bins.bin(fabsf(c) + mg)], 1u);
}

// margin of a pair: a bound on |c^ - c_fp32|
__device__ __forceinline__ float pair_margin(float kappa, float onepu,
                                             float d_f, const VecInfo& va,
                                             const VecInfo& vb) {
  return kappa * va.n2 * vb.n2 + onepu * (va.eta * vb.n1 + vb.eta * va.n1) +
         d_f * va.eta * vb.eta;
}

// the largest margin over all pairs
__device__ __forceinline__ float margin_max(const GemmArgs& g) {
  if (g.screen) return 0.0f;
  VecInfo a{}, b{};
  a.n2 = __uint_as_float(g.maxes[0]);
  a.n1 = __uint_as_float(g.maxes[1]);
  a.eta = __uint_as_float(g.maxes[2]);
  b.n2 = __uint_as_float(g.maxes[4]);
  b.n1 = __uint_as_float(g.maxes[5]);
  b.eta = __uint_as_float(g.maxes[6]);
  return pair_margin(g.kappa, g.onepu, g.d_f, a, b) * (1.0f + 1e-5f);
}

// Pass A, all 256 threads: hands the workgroup's counts (`hist`, in LDS) over
// and returns `pre`: |c| below it reaches neither the bound that g.target of
// all counts so far lie above nor, with its margin, the final tau.  (A bound
// from the workgroup's own values alone stays far below the final one: nearly
// every 64 x 32 block then held a value above it, 2.4 ms instead of 1.0 at
// 1563 x 1e6 x 256 in bf16; no bound, two LDS atomics a pair: 60.5 ms instead
// of 28.3 at 15,625 x 1e6 x 512.)
__device__ __forceinline__ float raise_bound(const GemmArgs& g,
                                             const BoundBins& bins,
                                             float mg_max, unsigned* hist,
                                             unsigned* thr) {
  const int t = threadIdx.x, lane = t & 63;
  __syncthreads();
  for (int b = t; b < 2048; b += 256)
    if (hist[b]) atomicAdd(&g.hist[b], hist[b]);
  // a count read too early only leaves the bound lower
  for (int b = t; b < 2048; b += 256)
    hist[b] = __hip_atomic_load(&g.hist[b], __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (t < 64) {
    const int per = bins.count() / 64;
    const int hi = bins.count() - 1 - per * lane;
    unsigned sum = 0;
    for (int b = hi; b > hi - per; --b) sum += hist[b];
    const unsigned incl = wave_incl_scan(sum);
    const uint64_t reach = __ballot((int64_t)incl >= g.target);
    if (reach && lane == __builtin_ctzll(reach)) {
      unsigned acc = incl - sum;
      int b = hi;
      for (; b > hi - per + 1; --b) {
        acc += hist[b];
        if ((int64_t)acc >= g.target) break;
      }
      *thr = bins.edge(b);
    }
  }
  __syncthreads();
  for (int b = t; b < 2048; b += 256) hist[b] = 0;
  __syncthreads();
  return __uint_as_float(*thr) - mg_max;
}

// E8M0 byte of a vector's power-of-two inverse scale (the MFMA multiplies
// the products of a lane's 32-element K block by 2^(byte - 127) per operand)
__device__ __forceinline__ int e8m0_of(float inv_s) {
  return (int)((__float_as_uint(inv_s) >> 23) & 0xff);
}

// launch of the register-panel GEMM (bf_panel*.hip): pass A (hist) or pass B
// over fragment-ordered copies of A and B
struct PanelArgs {
  GemmArgs g;
  int64_t tiles_n;   // column tiles
  int64_t panels;    // row panels
  int64_t seg;       // column tiles per work item
  int64_t items;     // panels x segments
  const int* sb;     // fp8: E8M0 bytes of B's vectors (padded rows too)
};

// steps of 16 bytes per lane that a vector of d coordinates takes in the
// fragment order, rounded up to a built kernel; 0: no panel kernel for d
int panel_steps(int prec, int64_t d);
// bytes of `rows` vectors in the fragment order (rows padded to 128)
int64_t panel_bytes(int prec, int64_t d, int64_t rows);
hipError_t panel_prepare(const float* X, int64_t rows, int64_t d, int prec,
                         void* out, VecInfo* info, int* scale, hipStream_t st);
hipError_t launch_panel(const GemmArgs& a, int prec, int64_t d, bool hist,
                        const int* sb, hipStream_t st);
// per-precision launches (one file each); grid 0: as many workgroups as fit
hipError_t launch_panel_f32(const PanelArgs& a, int ns, bool hist,
                            int64_t grid, hipStream_t st);
hipError_t launch_panel_bf16(const PanelArgs& a, int ns, bool hist,
                             int64_t grid, hipStream_t st);
hipError_t launch_panel_fp8(const PanelArgs& a, int ns, bool hist,
                            int64_t grid, hipStream_t st);

}  // namespace mad
