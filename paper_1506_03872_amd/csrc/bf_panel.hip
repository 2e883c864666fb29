// bf_panel.hip -- host side of the register-panel GEMM (bf_panel.hpp): which
// inputs it takes, their fragment-ordered copies, and the launch shape.
#include <stdlib.h>

#include "bf_panel.hpp"

namespace mad {

// The panel kernel keeps K in registers: up to 16 steps of 16 bytes per lane
// for 64 rows (K = 256 in bf16, 512 in fp8: 128 VGPRs), in fp32 up to 32
// steps (K = 256), for 32 rows above 20.  Longer vectors stay with the
// LDS-tiled kernel.  Every step count up to 20 is built in fp32, whose time
// follows it (65,536 x 65,536: 8.57 ms at 18 steps, 9.02 at 19, 9.41 at 20);
// the 50 kernels of all precisions are 28 s of the build's 33 on 8 cores and
// 4.6 MB of the library.
int panel_steps(int prec, int64_t d) {
  if (prec == kBF16 && d <= 256) return (int)((d + 15) / 16);
  if (prec == kFP8 && d <= 512) return (int)((d + 63) / 64) * 2;
  if (prec == kF32 && d <= 256) {
    const int ns = (int)((d + 7) / 8);
    return ns <= 20 ? ns : (ns + 1) / 2 * 2;  // even step counts are built
  }
  return 0;
}

int64_t panel_bytes(int prec, int64_t d, int64_t rows) {
  return (rows + 127) / 128 * 4 * (int64_t)panel_steps(prec, d) * 1024;
}

// Fragment order: 16 bytes of lane l = 32 g + r of step s of the 32 vectors
// from 32 b, at ((b NS + s) 64 + l) 16: vector 32 b + r, coordinates 16 s +
// 8 g + 0..7 (bf16), 64 (s / 2) + 32 g + 16 (s % 2) + 0..15 (fp8) or 8 s + 4
// g + 0..3 (fp32), which is the MFMA operand of that lane (fp32: its q-th
// MFMA takes coordinates 8 s + q and 8 s + 4 + q).  A workgroup takes 32
// vectors: it reads them into LDS, 8 lanes sum each one's norms, and every
// thread converts 16-byte pieces in the order they are stored.  Vectors past
// the last are zeros.  (A wave per vector for the norms, as in k_prep, spends
// its time in 18 dependent shuffles a vector: 47 us against 21 at 1e5 x 100 in
// fp8.)
template <int P>
__global__ __launch_bounds__(256) void k_prep_panel(const float* X,
                                                    int64_t rows, int d,
                                                    int ns, char* out,
                                                    VecInfo* info,
                                                    int* e8m0) {
  extern __shared__ float xs[];  // 32 rows at an odd stride
  __shared__ float scale_s[32];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * 32;
  const int ld = d | 1;
  const int live = rows - r0 < 32 ? (rows - r0 > 0 ? (int)(rows - r0) : 0)
                                  : 32;
  const float* x0 = X + r0 * d;
  for (int e = t; e < 32 * d; e += 256) {
    const int r = e / d;
    xs[r * ld + (e - r * d)] = r < live ? x0[e] : 0.0f;
  }
  __syncthreads();
  {  // 8 lanes per vector sum its norms
    const int r = t >> 3, sub = t & 7;
    double s2 = 0.0, s1 = 0.0;
    float mx = 0.0f;
    for (int k = sub; k < d; k += 8) {
      const float f = xs[r * ld + k];
      const double v = f;
      s2 += v * v;
      s1 += fabs(v);
      mx = fmaxf(mx, fabsf(f));
    }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) {
      s2 += __shfl_xor(s2, off, 64);
      s1 += __shfl_xor(s1, off, 64);
      mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    }
    if (sub == 0) {
      const VecInfo vi = vec_info<P>(s2, s1, mx);
      if (r < live) info[r0 + r] = vi;
      scale_s[r] = vec_scale<P>(vi);
      if (P == kFP8) e8m0[r0 + r] = e8m0_of(vi.inv_s);
    }
  }
  __syncthreads();
  i4v* o = (i4v*)(out + (int64_t)blockIdx.x * ns * 1024);
  for (int e = t; e < ns * 64; e += 256) {
    const int s = e >> 6, l = e & 63, r = l & 31, gk = l >> 5;
    const float* x = xs + r * ld;
    const float sc = scale_s[r];
    i4v w = {0, 0, 0, 0};
    if (P == kF32) {
      const int k0 = s * 8 + gk * 4;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        w[q] = __float_as_int(k0 + q < d ? x[k0 + q] : 0.0f);
    } else if (P == kBF16) {
      const int k0 = s * 16 + gk * 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float v = k0 + q < d ? x[k0 + q] : 0.0f;
        w[q >> 1] |= (int)((uint32_t)to_bf16(v) << (16 * (q & 1)));
      }
    } else {
      const int k0 = (s >> 1) * 64 + gk * 32 + (s & 1) * 16;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float v = k0 + q < d ? x[k0 + q] * sc : 0.0f;
        w[q >> 2] |= (int)((uint32_t)to_fp8(v) << (8 * (q & 3)));
      }
    }
    o[e] = w;
  }
}

hipError_t panel_prepare(const float* X, int64_t rows, int64_t d, int prec,
                         void* out, VecInfo* info, int* scale,
                         hipStream_t st) {
  const int ns = panel_steps(prec, d);
  const unsigned g = (unsigned)((rows + 127) / 128 * 4);
  const size_t lds = 32 * 4 * (size_t)(d | 1);  // d <= 512: 64.1 KB
  if (prec == kF32)
    k_prep_panel<kF32><<<g, 256, lds, st>>>(X, rows, (int)d, ns, (char*)out,
                                            info, scale);
  else if (prec == kBF16)
    k_prep_panel<kBF16><<<g, 256, lds, st>>>(X, rows, (int)d, ns, (char*)out,
                                             info, scale);
  else
    k_prep_panel<kFP8><<<g, 256, lds, st>>>(X, rows, (int)d, ns, (char*)out,
                                            info, scale);
  return hipGetLastError();
}

hipError_t launch_panel(const GemmArgs& g, int prec, int64_t d, bool hist,
                        const int* sb, hipStream_t st) {
  PanelArgs a;
  a.g = g;
  a.sb = sb;
  // MAD_BF_GRID overrides the workgroup count, a multiple of 8 (one share
  // per XCD); the result is the same
  int64_t grid = 0;
  if (const char* ev = getenv("MAD_BF_GRID")) grid = atoll(ev) / 8 * 8;
  const int ns = panel_steps(prec, d);
  return prec == kF32    ? launch_panel_f32(a, ns, hist, grid, st)
         : prec == kBF16 ? launch_panel_bf16(a, ns, hist, grid, st)
                         : launch_panel_fp8(a, ns, hist, grid, st);
}

}  // namespace mad
