// bf_panel.hip -- host side of the register-panel GEMM (bf_panel.hpp): which
// inputs it takes, their fragment-ordered copies, and the launch shape.
#include <stdlib.h>

#include "bf_panel.hpp"

namespace mad {

// The panel kernel keeps K in registers: up to 16 steps of 16 bytes per lane
// and 32 rows (K = 256 in bf16, 512 in fp8: 128 VGPRs for 64 rows).  Longer
// vectors, and fp32, whose MFMAs take 64 cycles per 256 bytes of operand and
// are not short of LDS bandwidth, stay with the LDS-tiled kernel.
int panel_steps(int prec, int64_t d) {
  if (prec == kBF16 && d <= 256) return (int)((d + 15) / 16);
  if (prec == kFP8 && d <= 512) return (int)((d + 63) / 64) * 2;
  return 0;
}

int64_t panel_bytes(int prec, int64_t d, int64_t rows) {
  return (rows + 127) / 128 * 4 * (int64_t)panel_steps(prec, d) * 1024;
}

// Fragment order: 16 bytes of lane l = 32 g + r of step s of the 32 vectors
// from 32 b, at ((b NS + s) 64 + l) 16: vector 32 b + r, coordinates 16 s +
// 8 g + 0..7 (bf16) or 64 (s / 2) + 32 g + 16 (s % 2) + 0..15 (fp8), which is
// the MFMA operand of that lane.  A workgroup takes 32 vectors: a wave sums
// the norms of 8 (as k_prep does), then every thread converts 16-byte
// pieces in the order they are stored.  Vectors past the last are zeros.
template <int P>
__global__ __launch_bounds__(256) void k_prep_panel(const float* X,
                                                    int64_t rows, int64_t d,
                                                    int ns, char* out,
                                                    VecInfo* info,
                                                    int* e8m0) {
  __shared__ float scale_s[32];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * 32;
  for (int q = 0; q < 8; ++q) {
    const int64_t r = r0 + wv * 8 + q;
    if (r >= rows) {
      if (lane == 0) {
        scale_s[wv * 8 + q] = 0.0f;
        if (P == kFP8) e8m0[r] = 127;
      }
      continue;
    }
    const float* x = X + r * d;
    double s2 = 0.0, s1 = 0.0;
    float mx = 0.0f;
    for (int64_t k = lane; k < d; k += 64) {
      const double v = x[k];
      s2 += v * v;
      s1 += fabs(v);
      mx = fmaxf(mx, fabsf(x[k]));
    }
    const VecInfo vi = vec_info<P>(wave_sum(s2), wave_sum(s1), wave_max(mx));
    if (lane == 0) {
      info[r] = vi;
      scale_s[wv * 8 + q] = vec_scale<P>(vi);
      if (P == kFP8) e8m0[r] = e8m0_of(vi.inv_s);
    }
  }
  __syncthreads();
  i4v* o = (i4v*)(out + (int64_t)blockIdx.x * ns * 1024);
  for (int e = t; e < ns * 64; e += 256) {
    const int s = e >> 6, l = e & 63, r = l & 31, gk = l >> 5;
    const float* x = X + (r0 + r) * d;
    const float sc = scale_s[r];
    const bool live = r0 + r < rows;
    i4v w = {0, 0, 0, 0};
    if (P == kBF16) {
      const int64_t k0 = (int64_t)s * 16 + gk * 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float v = live && k0 + q < d ? x[k0 + q] : 0.0f;
        w[q >> 1] |= (int)((uint32_t)to_bf16(v) << (16 * (q & 1)));
      }
    } else {
      const int64_t k0 = (int64_t)(s >> 1) * 64 + gk * 32 + (s & 1) * 16;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float v = live && k0 + q < d ? x[k0 + q] * sc : 0.0f;
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
  if (prec == kBF16)
    k_prep_panel<kBF16><<<g, 256, 0, st>>>(X, rows, d, ns, (char*)out, info,
                                           scale);
  else
    k_prep_panel<kFP8><<<g, 256, 0, st>>>(X, rows, d, ns, (char*)out, info,
                                          scale);
  return hipGetLastError();
}

hipError_t launch_panel(const GemmArgs& g, int prec, int64_t d, bool hist,
                        int64_t target, const int* sb, unsigned* thr,
                        hipStream_t st) {
  PanelArgs a;
  a.g = g;
  a.sb = sb;
  a.thr = thr;
  a.target = target;
  const int ns = panel_steps(prec, d);
  const int tn = panel_tile_blocks(ns) * 32;
  a.tiles_n = (g.n + tn - 1) / tn;
  a.panels = (g.m_rows + kPanelRows - 1) / kPanelRows;
  // two workgroups per CU (LDS and registers), a multiple of 8 (one share
  // per XCD); MAD_BF_GRID overrides the count (the result is the same)
  int64_t grid = 256 * 2;
  if (const char* ev = getenv("MAD_BF_GRID")) {
    const int64_t gv = atoll(ev) / 8 * 8;
    if (gv >= 8) grid = gv;
  }
  // column tiles per item: up to 2048 columns, so that loading the rows of A
  // (once per item) is a few percent of it, but a dozen items or more per
  // workgroup while there are tiles enough, so that the last round is short
  int64_t seg = a.tiles_n * a.panels / (grid * 12);
  if (seg > 2048 / tn) seg = 2048 / tn;
  if (seg < 1) seg = 1;
  a.seg = seg;
  a.items = a.panels * ((a.tiles_n + seg - 1) / seg);
  return prec == kBF16
             ? launch_panel_bf16(a, ns, hist, (unsigned)grid, st)
             : launch_panel_fp8(a, ns, hist, (unsigned)grid, st);
}

}  // namespace mad
