// exact_csr.hip -- exhaustive t-MAD (Definition 1) for sparse inputs, the
// exact baseline of Sec. 5.3 for the sparse case.  The paper forms C one
// column at a time with a sparse product whose cost is the number of
// wedges (pairs of entries sharing a coordinate) and keeps a priority queue.
// On power-law inputs nearly all wedges meet at a few coordinates of huge
// degree, so here the coordinates are split in two:
//
//   heavy  the coordinates with the most wedges (deg_A(k) deg_B(k)); their
//          columns are copied into dense m x H and n x H matrices and every
//          pair's heavy part c^H_ij goes through the MFMA brute force;
//   light  the rest; their wedges (i, j, a_ik b_jk) are listed and summed
//          per pair, giving c^L_ij for the pairs P_L that share one.
//
// c_ij = c^H_ij outside P_L and c^H_ij + c^L_ij on it.  With tau_lb a
// lower bound on the t-th largest |c| (the exact values of the heavy part's
// own top-t candidates), the exact top t lies in
//   {pairs with |c^H| >= tau_lb}          (the certified brute-force filter)
//   {pairs of P_L whose bound |c^L| + ||a_i^H|| ||b_j^H|| >= tau_lb}
// whose union is re-ranked with sparse dot products of the candidates.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "mad_common.hpp"
#include "plan.hpp"

namespace mad {

constexpr int64_t kMaxLightWedges = int64_t(1) << 30;
constexpr int64_t kMaxHeavy = 4096;
constexpr int kWedgeSteps = 32;  // wedges per lane of the listing kernel

// Entries per coordinate.  A coordinate that every vector holds takes one
// atomic per entry on one address (12 ns each: 350 us at 30,000 vectors), so
// a workgroup counts in LDS the coordinates that claim a slot of a small
// table first, which the frequent ones do, and adds those counts once
// (16 us); the others go straight to memory.
constexpr int kDegSlots = 2048;

__global__ __launch_bounds__(256) void k_coord_degrees(const int32_t* idx,
                                                       int64_t nnz,
                                                       uint32_t* deg) {
  __shared__ int32_t tag[kDegSlots];
  __shared__ unsigned cnt[kDegSlots];
  for (int s = threadIdx.x; s < kDegSlots; s += 256) {
    tag[s] = -1;
    cnt[s] = 0;
  }
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz;
       e += stride) {
    const int32_t k = idx[e];
    const int s = k & (kDegSlots - 1);
    const int32_t was = atomicCAS(&tag[s], -1, k);
    if (was == -1 || was == k)
      atomicAdd(&cnt[s], 1u);
    else
      atomicAdd(&deg[k], 1u);
  }
  __syncthreads();
  for (int s = threadIdx.x; s < kDegSlots; s += 256)
    if (cnt[s]) atomicAdd(&deg[tag[s]], cnt[s]);
}

// ---------------------------------------------------------------------------
// the heavy / light split on the device
// ---------------------------------------------------------------------------
// Coordinates by their wedges deg_A deg_B, in 2048 bins (exponent and three
// bits of the float): the heavy ones are those of bins >= cut.
__device__ __forceinline__ int wedge_bin(uint64_t w) {
  return w ? (int)(__float_as_uint((float)w) >> 20) : 0;
}

struct SplitHist {
  unsigned long long wedges[2048];
  unsigned count[2048];
};

__global__ __launch_bounds__(256) void k_wedge_hist(const uint32_t* dA,
                                                    const uint32_t* dB,
                                                    int64_t d,
                                                    SplitHist* out) {
  __shared__ SplitHist h;
  for (int b = threadIdx.x; b < 2048; b += 256) {
    h.wedges[b] = 0ull;
    h.count[b] = 0u;
  }
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < d;
       k += stride) {
    const uint64_t w = (uint64_t)dA[k] * dB[k];
    if (!w) continue;
    const int b = wedge_bin(w);
    atomicAdd(&h.wedges[b], (unsigned long long)w);
    atomicAdd(&h.count[b], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < 2048; b += 256)
    if (h.count[b]) {
      atomicAdd(&out->wedges[b], h.wedges[b]);
      atomicAdd(&out->count[b], h.count[b]);
    }
}

// The cut: of the bins that leave at most kMaxLightWedges light wedges and
// 1 to kMaxHeavy heavy coordinates, the one with the least expected time,
// the column times of `pad` (the heavy coordinates, padded to a K step of the
// GEMM that takes them) and wedge_ns per light wedge.  Between cuts of one
// padded width the deepest wins, so that no column is left to padding.  cut =
// -1 when there is none (or no wedge at all).
struct ColumnPad {
  int panel, panel_step;  // widest K of the register-panel GEMM, its K step
  int step;               // K step of the GEMM for longer vectors
  double panel_ns, ns;    // time of a column in each
};

struct SplitCut {
  int64_t cut, live;
  int64_t wedges;
};

__global__ __launch_bounds__(256) void k_split_cut(const SplitHist* h,
                                                   double wedge_ns,
                                                   ColumnPad pad,
                                                   SplitCut* out) {
  __shared__ unsigned long long ws[4], cs[4];
  __shared__ double best[256];
  __shared__ int at[256];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // thread t: bins 2047 - 8 t down to 2040 - 8 t
  unsigned long long w = 0, c = 0;
  for (int q = 0; q < 8; ++q) {
    w += h->wedges[2047 - 8 * t - q];
    c += h->count[2047 - 8 * t - q];
  }
  const unsigned long long wi = wave_incl_scan(w), ci = wave_incl_scan(c);
  if (lane == 63) {
    ws[wv] = wi;
    cs[wv] = ci;
  }
  __syncthreads();
  unsigned long long hw = wi - w, hc = ci - c, total = 0, live = 0;
  for (int u = 0; u < 4; ++u) {
    hw += u < wv ? ws[u] : 0ull;
    hc += u < wv ? cs[u] : 0ull;
    total += ws[u];
    live += cs[u];
  }
  best[t] = 1e300;
  at[t] = -1;
  for (int q = 0; q < 8; ++q) {
    const int b = 2047 - 8 * t - q;
    if (!h->count[b]) continue;
    hw += h->wedges[b];
    hc += h->count[b];
    const unsigned long long light = total - hw;
    if (light > (unsigned long long)kMaxLightWedges ||
        hc > (unsigned long long)kMaxHeavy)
      continue;
    const bool panel = hc <= (unsigned long long)pad.panel;
    const unsigned long long step = panel ? pad.panel_step : pad.step;
    const double cost = (panel ? pad.panel_ns : pad.ns) *
                            (double)((hc + step - 1) / step * step) +
                        wedge_ns * (double)light;
    if (cost < best[t]) {
      best[t] = cost;
      at[t] = b;
    }
  }
  __syncthreads();
  if (t == 0) {
    double m = 1e300;
    int cut = -1;
    for (int u = 0; u < 256; ++u)
      if (best[u] < m) {
        m = best[u];
        cut = at[u];
      }
    out->cut = cut;
    out->live = (int64_t)live;
    out->wedges = (int64_t)total;
  }
}

// Per coordinate: heavy column or -1, the light lists' starts on both sides,
// the light coordinates with wedges and their wedge prefix.  Two passes over
// tiles of 2048 coordinates: sums, then (after launch_scan_parts) positions.
constexpr int kSplitVals = 5;  // heavy, light entries of A, of B, listed
                               // light coordinates, light wedges
constexpr int kSplitPer = 8;
constexpr int kSplitTile = 256 * kSplitPer;

__device__ __forceinline__ void split_add(uint32_t a, uint32_t b, int cut,
                                          int64_t (&v)[kSplitVals]) {
  const uint64_t w = (uint64_t)a * b;
  if (w && wedge_bin(w) >= cut) {
    v[0] += 1;
  } else {
    v[1] += a;
    v[2] += b;
    v[3] += w != 0;
    v[4] += (int64_t)w;
  }
}

__global__ __launch_bounds__(256) void k_split_count(const uint32_t* dA,
                                                     const uint32_t* dB,
                                                     int64_t d,
                                                     const SplitCut* sc,
                                                     int64_t* part) {
  __shared__ int64_t red[4][kSplitVals];
  const int cut = (int)sc->cut;
  const int64_t k0 = (int64_t)blockIdx.x * kSplitTile +
                     (int64_t)threadIdx.x * kSplitPer;
  int64_t v[kSplitVals] = {};
  for (int u = 0; u < kSplitPer; ++u)
    if (k0 + u < d) split_add(dA[k0 + u], dB[k0 + u], cut, v);
#pragma unroll
  for (int q = 0; q < kSplitVals; ++q) {
    const int64_t x = wave_sum(v[q]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = x;
  }
  __syncthreads();
  if (threadIdx.x < kSplitVals) {
    int64_t x = 0;
    for (int w = 0; w < 4; ++w) x += red[w][threadIdx.x];
    part[(int64_t)blockIdx.x * kSplitVals + threadIdx.x] = x;
  }
}

__global__ __launch_bounds__(256) void k_split_fill(
    const uint32_t* dA, const uint32_t* dB, int64_t d, const SplitCut* sc,
    const int64_t* part, const int64_t* tot, int32_t* pos, int64_t* taptr,
    int64_t* tbptr, int32_t* lk, int64_t* wpre) {
  __shared__ int64_t wsum[4][kSplitVals];
  const int cut = (int)sc->cut;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t k0 = (int64_t)blockIdx.x * kSplitTile +
                     (int64_t)threadIdx.x * kSplitPer;
  int64_t v[kSplitVals] = {}, at[kSplitVals];
  for (int u = 0; u < kSplitPer; ++u)
    if (k0 + u < d) split_add(dA[k0 + u], dB[k0 + u], cut, v);
#pragma unroll
  for (int q = 0; q < kSplitVals; ++q) {
    const int64_t incl = wave_incl_scan(v[q]);
    at[q] = incl - v[q];
    if (lane == 63) wsum[wv][q] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSplitVals; ++q) {
    at[q] += part[(int64_t)blockIdx.x * kSplitVals + q];
    for (int w = 0; w < wv; ++w) at[q] += wsum[w][q];
  }
  for (int u = 0; u < kSplitPer && k0 + u < d; ++u) {
    const int64_t k = k0 + u;
    const uint64_t w = (uint64_t)dA[k] * dB[k];
    const bool heavy = w && wedge_bin(w) >= cut;
    pos[k] = heavy ? (int32_t)at[0] : -1;
    taptr[k] = at[1];
    tbptr[k] = at[2];
    if (!heavy && w) {
      lk[at[3]] = (int32_t)k;
      wpre[at[3]] = at[4];
    }
    split_add(dA[k], dB[k], cut, at);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    taptr[d] = tot[1];
    tbptr[d] = tot[2];
    wpre[tot[3]] = tot[4];      // the end, and a sentinel after it
    wpre[tot[3] + 1] = tot[4];
  }
}

// one thread per vector: its heavy entries into column pos[k] of a dense
// row (zero-filled before), and the L2 norms of its heavy and of its light
// entries (x, y of nhl), rounded up; *lmost = the most light entries of a
// vector (cleared before)
__global__ void k_split_rows(const int64_t* ptr, const int32_t* idx,
                             const float* val, int64_t rows,
                             const int32_t* pos, int64_t H, float* dense,
                             float2* nhl, unsigned* lmost) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned light = 0;
  if (r < rows) {
    double sh = 0.0, sl = 0.0;
    for (int64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
      const int32_t p = pos[idx[e]];
      const float v = val[e];
      if (p >= 0) {
        dense[r * H + p] = v;
        sh += (double)v * v;
      } else {
        sl += (double)v * v;
        ++light;
      }
    }
    nhl[r] = make_float2((float)(sqrt(sh) * (1.0 + 1e-6)),
                         (float)(sqrt(sl) * (1.0 + 1e-6)));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned o = __shfl_xor(light, off, 64);
    light = light > o ? light : o;
  }
  if ((threadIdx.x & 63) == 0 && light > *lmost) atomicMax(lmost, light);
}

// the light coordinates' lists of vectors (any order inside a list)
__global__ void k_light_lists(const int64_t* ptr, const int32_t* idx,
                              const float* val, int64_t rows,
                              const int32_t* pos, const int64_t* tptr,
                              uint32_t* cur, uint32_t* trow, float* tval) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  for (int64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
    const int32_t k = idx[e];
    if (pos[k] >= 0) continue;
    const int64_t p = tptr[k] + atomicAdd(&cur[k], 1u);
    trow[p] = (uint32_t)r;
    tval[p] = val[e];
  }
}

// every light wedge: wedge w of light coordinate lk[q] (wpre[q] <= w <
// wpre[q+1]) pairs entry w' / deg_B of A's list with entry w' % deg_B of
// B's list, w' = w - wpre[q]; key i*n + j, value a_ik b_jk (fp32).  A wave
// takes 64 * kWedgeSteps consecutive wedges, lane l every 64th from l.
__global__ __launch_bounds__(256) void k_light_wedges(
    const int32_t* lk, const int64_t* wpre, int64_t nl, int64_t W,
    const int64_t* taptr, const uint32_t* tarow, const float* taval,
    const int64_t* tbptr, const uint32_t* tbrow, const float* tbval,
    int64_t n, uint64_t* keys, float* vals) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t w0 = wave * 64 * kWedgeSteps; w0 < W;
       w0 += nwaves * 64 * kWedgeSteps) {
    int64_t w = w0 + lane;
    if (w >= W) continue;
    // the list holding wedge w: last q with wpre[q] <= w
    int64_t lo = 0, hi = nl;  // wpre[lo] <= w < wpre[hi]
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (wpre[mid] <= w) lo = mid; else hi = mid;
    }
    int64_t q = lo;
    for (int s = 0; s < kWedgeSteps && w < W; ++s, w += 64) {
      while (wpre[q + 1] <= w) ++q;
      const int32_t k = lk[q];
      const int64_t db = tbptr[k + 1] - tbptr[k];
      const int64_t loc = w - wpre[q];
      const int64_t ia = loc / db, jb = loc - ia * db;
      const int64_t pa = taptr[k] + ia, pb = tbptr[k] + jb;
      keys[w] = (uint64_t)tarow[pa] * (uint64_t)n + tbrow[pb];
      vals[w] = taval[pa] * tbval[pb];
    }
  }
}

// pairs of P_L that may reach tau: |c^L| (with its rounding) plus the bound
// ||a_i^H|| ||b_j^H|| on the heavy part
__global__ void k_light_prune(const uint64_t* okey, const int64_t* oval,
                              const int64_t* len, int F, double wslack,
                              int64_t n, const float2* na,
                              const float2* nb, float tau,
                              uint64_t* out, unsigned long long* cnt,
                              int64_t cap) {
  const int64_t L = *len;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < L;
       e += stride) {
    const uint64_t key = okey[e];
    if (key == kEmptyKey) continue;
    const int64_t i = (int64_t)(key / (uint64_t)n);
    const int64_t j = (int64_t)(key - (uint64_t)i * (uint64_t)n);
    const double x = fabs(ldexp((double)oval[e], -F));
    // fp32 products err by at most 2^-24 of sum |a_ik b_jk| <= ||a^L||
    // ||b^L||, the fixed-point sum by 2^-F per wedge of the pair (wslack
    // bounds that), the heavy part by ||a^H|| ||b^H||
    const float2 a = na[i], b = nb[j];  // heavy, light norm
    const double ub = x + 1e-5 * (double)a.y * b.y + wslack +
                      (double)a.x * b.x * (1.0 + 1e-5);
    if (ub >= (double)tau) {
      const unsigned long long p = atomicAdd(cnt, 1ull);
      if ((int64_t)p < cap) out[p] = key;
    }
  }
}

static unsigned grid_of(int64_t n, int per, unsigned cap) {
  int64_t g = (n + per - 1) / per;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

struct ExactWork {
  DeviceBuffer deg, split, pos, ah, bh, norms, lk, wpre, tptr, cur, tlist,
      pairs, acc, tab, cand, fin, misc;
};
static ExactWork g_ex;

// expected times of the split's two parts: a column of the dense product (2 m
// n flops) at the rates measured for the heavy part on each side of the widest
// panel kernel's K, and a light wedge (listed, summed and pruned: 47 to 50 ps
// at 1e7 to 5e8 wedges).  At 3e5 x 3e5: bf16 256 columns 28 ms (1.6e15), 320
// 95 (0.61e15) and 768 192 (0.72e15), at 1e5 x 1e5 4.0 (1.3e15), 9.5 and
// 23.5; fp32 0.14e15 and 0.13e15.  In fp8 the certified margins let whole
// tiles through, and only what a column adds counts: 108 ms with 256 columns,
// 160 with 512 (0.89e15), 222 with 640.
static void split_col_ns(int prec, int64_t m, int64_t n, double* panel,
                         double* longer) {
  const double mn = 2.0 * (double)m * (double)n * 1e9;
  *panel = mn / (prec == 0 ? 1.4e14 : prec == 1 ? 1.3e15 : 0.9e15);
  *longer = mn / (prec == 0 ? 1.3e14 : prec == 1 ? 0.65e15 : 0.8e15);
}
constexpr double kWedgeNs = 0.05;

static ColumnPad column_pad(int prec, int64_t m, int64_t n) {
  ColumnPad p = prec == 0   ? ColumnPad{256, 8, 32}
                : prec == 1 ? ColumnPad{256, 16, 64}
                            : ColumnPad{512, 64, 128};
  split_col_ns(prec, m, n, &p.panel_ns, &p.ns);
  return p;
}

// device_split: cut the coordinates on the device at the least expected
// time; *again = true when the other rule has to be used (no such cut, or
// fewer than t pairs with c != 0 found among the heavy candidates, where the
// pairs with c = 0 that fill the answer depend on the split).  Else the
// host's rule: heavy_req coordinates, or the fewest (a multiple of 64) that
// leave at most kMaxLightWedges.
static hipError_t topk_csr_run(const CsrView& in, int64_t m, int64_t n,
                               int64_t d, int64_t nnzA, int64_t nnzB,
                               int prec, int64_t t, int64_t heavy_req,
                               bool device_split, bool* again, void* out,
                               int64_t* n_out, BfCsrStats* stats,
                               hipStream_t st) {
  hipError_t e;
  ExactWork& w = g_ex;
  struct Events {  // destroyed on every return
    hipEvent_t ev[5] = {};
    Events() {
      for (auto& x : ev) (void)hipEventCreate(&x);
    }
    ~Events() {
      for (auto& x : ev)
        if (x) (void)hipEventDestroy(x);
    }
  } evs;
  hipEvent_t* ev = evs.ev;
  *again = false;
  (void)hipEventRecord(ev[0], st);
  // ---- coordinate degrees and the heavy / light split ---------------------
  const int64_t tiles = (d + kSplitTile - 1) / kSplitTile;
  if ((e = dev_alloc(w.deg, 8 * (size_t)d + 256)) != hipSuccess ||
      (e = dev_alloc(w.misc, 4096)) != hipSuccess ||
      (e = dev_alloc(w.split, sizeof(SplitHist) + 256 +
                                  8 * kSplitVals * (size_t)(tiles + 1))) !=
          hipSuccess ||
      (e = dev_alloc(w.pos, 4 * (size_t)d)) != hipSuccess ||
      (e = dev_alloc(w.tptr, 16 * (size_t)(d + 1))) != hipSuccess ||
      (e = dev_alloc(w.cur, 8 * (size_t)d + 256)) != hipSuccess)
    return e;
  uint32_t* dA = (uint32_t*)w.deg.p;
  uint32_t* dB = dA + d;
  int32_t* dpos = (int32_t*)w.pos.p;
  int64_t* dtaptr = (int64_t*)w.tptr.p;
  int64_t* dtbptr = dtaptr + d + 1;
  {
    FillBatch f{};
    f.count = 2;
    f.p[0] = (uint64_t*)dA;
    f.n[0] = d;
    f.p[1] = (uint64_t*)w.split.p;
    f.n[1] = sizeof(SplitHist) / 8;
    if ((e = launch_fill_multi(f, st)) != hipSuccess) return e;
  }
  k_coord_degrees<<<grid_of(nnzA, 256 * 16, 1024), 256, 0, st>>>(in.a_idx,
                                                                 nnzA, dA);
  k_coord_degrees<<<grid_of(nnzB, 256 * 16, 1024), 256, 0, st>>>(in.b_idx,
                                                                 nnzB, dB);
  int64_t H = 0, W = 0, nl = 0, la = 0, lb = 0;
  double total = 0.0;
  auto sized = [&]() -> hipError_t {  // the arrays that the split sizes
    const int64_t Hc = H > 0 ? H : 1;
    hipError_t r;
    if ((r = dev_alloc(w.ah, 4 * (size_t)m * Hc)) != hipSuccess ||
        (r = dev_alloc(w.bh, 4 * (size_t)n * Hc)) != hipSuccess ||
        (r = dev_alloc(w.norms, 8 * (size_t)(m + n) + 256)) != hipSuccess ||
        (r = dev_alloc(w.lk, 4 * (size_t)(nl + 1))) != hipSuccess ||
        (r = dev_alloc(w.wpre, 8 * (size_t)(nl + 2))) != hipSuccess ||
        (r = dev_alloc(w.tlist, 8 * (size_t)(la + lb + 2))) != hipSuccess)
      return r;
    return hipSuccess;
  };
  if (device_split) {
    SplitHist* hist = (SplitHist*)w.split.p;
    SplitCut* cut = (SplitCut*)(hist + 1);
    int64_t* tot = (int64_t*)((char*)cut + 64);
    int64_t* part = tot + 16;
    k_wedge_hist<<<grid_of(d, 256 * 8, 256), 256, 0, st>>>(dA, dB, d, hist);
    k_split_cut<<<1, 256, 0, st>>>(hist, kWedgeNs, column_pad(prec, m, n),
                                   cut);
    k_split_count<<<(unsigned)tiles, 256, 0, st>>>(dA, dB, d, cut, part);
    if ((e = launch_scan_parts(part, tiles, kSplitVals, tot, st)) !=
        hipSuccess)
      return e;
    struct {
      SplitCut cut;
      char pad[64 - sizeof(SplitCut)];
      int64_t tot[kSplitVals];
    } got;
    if ((e = hipMemcpyAsync(&got, cut, sizeof got, hipMemcpyDeviceToHost,
                            st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
    if (got.cut.live == 0) {  // no coordinate is shared: every c_ij is 0
      if (stats) memset(stats, 0, sizeof *stats);
      return launch_fill_u64((uint64_t*)n_out, 1, 0ull, st);
    }
    if (got.cut.cut < 0) {
      *again = true;
      return hipSuccess;
    }
    H = got.tot[0];
    la = got.tot[1];
    lb = got.tot[2];
    nl = got.tot[3];
    W = got.tot[4];
    total = (double)got.cut.wedges;
    if ((e = sized()) != hipSuccess) return e;
    k_split_fill<<<(unsigned)tiles, 256, 0, st>>>(
        dA, dB, d, cut, part, tot, dpos, dtaptr, dtbptr, (int32_t*)w.lk.p,
        (int64_t*)w.wpre.p);
  } else {
    std::vector<uint32_t> hd(2 * (size_t)d);
    if ((e = hipMemcpyAsync(hd.data(), dA, 8 * (size_t)d,
                            hipMemcpyDeviceToHost, st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
    std::vector<double> wk((size_t)d);
    for (int64_t k = 0; k < d; ++k) {
      wk[k] = (double)hd[k] * (double)hd[d + k];
      total += wk[k];
    }
    std::vector<int32_t> order((size_t)d);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t x, int32_t y) { return wk[x] > wk[y]; });
    int64_t live = 0;
    while (live < d && wk[order[live]] > 0.0) ++live;
    if (live == 0) {  // no coordinate is shared: every c_ij is 0
      if (stats) memset(stats, 0, sizeof *stats);
      return launch_fill_u64((uint64_t*)n_out, 1, 0ull, st);
    }
    if (heavy_req > 0) {
      H = heavy_req < live ? heavy_req : live;
    } else {
      // the fewest heavy coordinates (a multiple of 64) that leave at most
      // kMaxLightWedges light wedges
      double light = total;
      while (H < live && (light > (double)kMaxLightWedges || H % 64 != 0)) {
        light -= wk[order[H]];
        ++H;
      }
    }
    if (H < 1 && live > 0) H = 1;
    if (H > kMaxHeavy) return hipErrorNotSupported;
    std::vector<int32_t> pos((size_t)d, -1);
    for (int64_t h = 0; h < H; ++h) pos[order[h]] = (int32_t)h;
    // light lists: pointer of each coordinate's list, the light coordinates
    // with wedges, and their wedge prefix
    std::vector<int64_t> taptr((size_t)d + 1, 0), tbptr((size_t)d + 1, 0);
    std::vector<int32_t> lk;
    std::vector<int64_t> wpre(1, 0);
    for (int64_t k = 0; k < d; ++k) {
      const bool light = pos[k] < 0;
      taptr[k + 1] = taptr[k] + (light ? hd[k] : 0);
      tbptr[k + 1] = tbptr[k] + (light ? hd[d + k] : 0);
      if (light && wk[k] > 0.0) {
        lk.push_back((int32_t)k);
        wpre.push_back(wpre.back() + (int64_t)hd[k] * (int64_t)hd[d + k]);
      }
    }
    W = wpre.back();
    nl = (int64_t)lk.size();
    la = taptr[d];
    lb = tbptr[d];
    if (W > kMaxLightWedges) return hipErrorNotSupported;
    if ((e = sized()) != hipSuccess) return e;
    wpre.push_back(wpre.back());  // sentinel: wpre[nl + 1] = W
    if ((e = hipMemcpyAsync(dpos, pos.data(), 4 * (size_t)d,
                            hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(dtaptr, taptr.data(), 8 * (size_t)(d + 1),
                            hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(dtbptr, tbptr.data(), 8 * (size_t)(d + 1),
                            hipMemcpyHostToDevice, st)) != hipSuccess ||
        (nl > 0 &&
         (e = hipMemcpyAsync(w.lk.p, lk.data(), 4 * (size_t)nl,
                             hipMemcpyHostToDevice, st)) != hipSuccess) ||
        (e = hipMemcpyAsync(w.wpre.p, wpre.data(), 8 * (size_t)(nl + 2),
                            hipMemcpyHostToDevice, st)) != hipSuccess)
      return e;
    // the vectors above go out of scope
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  }
  // ---- dense heavy columns, light lists, their largest |values| -----------
  const int64_t Hc = H > 0 ? H : 1;
  float2* na = (float2*)w.norms.p;
  float2* nb = na + m;
  uint32_t* curA = (uint32_t*)w.cur.p;
  uint32_t* curB = curA + d;
  uint32_t* tarow = (uint32_t*)w.tlist.p;
  float* taval = (float*)(tarow + la);
  uint32_t* tbrow = (uint32_t*)(taval + la);
  float* tbval = (float*)(tbrow + lb);
  // largest |value| of A's and of B's light lists, then the most light
  // entries of a vector on either side
  float* lmax = (float*)((char*)w.misc.p + 512);
  unsigned* lmost = (unsigned*)(lmax + 2);
  {
    FillBatch f{};
    f.count = 4;
    f.p[0] = (uint64_t*)w.ah.p;
    f.n[0] = (m * Hc + 1) / 2;
    f.p[1] = (uint64_t*)w.bh.p;
    f.n[1] = (n * Hc + 1) / 2;
    f.p[2] = (uint64_t*)curA;
    f.n[2] = d;
    f.p[3] = (uint64_t*)lmax;
    f.n[3] = 2;
    if ((e = launch_fill_multi(f, st)) != hipSuccess) return e;
  }
  k_split_rows<<<grid_of(m, 256, 1u << 30), 256, 0, st>>>(
      in.a_ptr, in.a_idx, in.a_val, m, dpos, Hc, (float*)w.ah.p, na,
      lmost);
  k_split_rows<<<grid_of(n, 256, 1u << 30), 256, 0, st>>>(
      in.b_ptr, in.b_idx, in.b_val, n, dpos, Hc, (float*)w.bh.p, nb,
      lmost + 1);
  k_light_lists<<<grid_of(m, 256, 1u << 30), 256, 0, st>>>(
      in.a_ptr, in.a_idx, in.a_val, m, dpos, dtaptr, curA, tarow, taval);
  k_light_lists<<<grid_of(n, 256, 1u << 30), 256, 0, st>>>(
      in.b_ptr, in.b_idx, in.b_val, n, dpos, dtbptr, curB, tbrow, tbval);
  if ((e = launch_absmax(taval, la, lmax, st)) != hipSuccess ||
      (e = launch_absmax(tbval, lb, lmax + 1, st)) != hipSuccess)
    return e;
  (void)hipEventRecord(ev[1], st);
  // ---- heavy part: certified brute force, then tau_lb ---------------------
  // tau_lb = the t-th largest exact |c| among the candidates of the heavy
  // part's own top t (each is a real pair, so t of them reach it)
  const uint64_t* ck = nullptr;
  int64_t cc = 0;
  BfStats bs;
  memset(&bs, 0, sizeof bs);
  const float* AH = (const float*)w.ah.p;
  const float* BH = (const float*)w.bh.p;
  if ((e = bruteforce_run(AH, m, BH, n, Hc, prec, t, 0, -1.0f, nullptr,
                          nullptr, &ck, &cc, &bs, st)) != hipSuccess)
    return e;
  int64_t* dn = (int64_t*)w.misc.p;
  std::vector<char> tmp((size_t)t * 24);
  if ((e = dev_alloc(w.cand, 24 * (size_t)(t > 1 ? t : 1))) != hipSuccess)
    return e;
  float tau_lb = 0.0f;
  if (cc > 0) {
    if ((e = launch_rerank_topk(ck, cc, nullptr, nullptr, n, 0,
                                t < cc ? t : cc, w.fin, w.cand.p, dn, &in,
                                st)) != hipSuccess)
      return e;
    int64_t got = 0;
    if ((e = hipMemcpyAsync(&got, dn, 8, hipMemcpyDeviceToHost, st)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
    if (got >= t) {
      if ((e = hipMemcpy(tmp.data(), w.cand.p, 24 * (size_t)t,
                         hipMemcpyDeviceToHost)) != hipSuccess)
        return e;
      float c;
      memcpy(&c, tmp.data() + 24 * (size_t)(t - 1) + 16, 4);
      tau_lb = fabsf(c);
    }
  }
  if (device_split && !(tau_lb > 0.0f)) {
    *again = true;
    return hipSuccess;
  }
  // pass B again only when tau_lb is below the threshold it ran with
  const float tau_use = tau_lb * (1.0f - 1e-5f);
  if (tau_use < bs.tau) {
    const float tu = tau_use > 0.0f ? tau_use : 1e-30f;
    if ((e = bruteforce_run(AH, m, BH, n, Hc, prec, t, 0, tu, nullptr,
                            nullptr, &ck, &cc, &bs, st)) != hipSuccess)
      return e;
  }
  const int64_t heavy_cand = cc;
  (void)hipEventRecord(ev[2], st);
  // ---- light part: its wedges summed per pair, then the bound ------------
  int64_t light_cand = 0;
  const size_t pk = 8 * (size_t)(W > 1 ? W : 1);
  const size_t pv = (4 * (size_t)(W > 1 ? W : 1) + 255) / 256 * 256;
  // candidates: heavy survivors, then light survivors (cap: W or 2^27)
  const int64_t lcap = W < (int64_t(1) << 27) ? W : (int64_t(1) << 27);
  const int64_t ccap = heavy_cand + lcap + 1;
  if ((e = dev_alloc(w.tab, 8 * (size_t)ccap + (4 * (size_t)ccap + 255) /
                                                   256 * 256 +
                                16 * (size_t)ccap + 256 +
                                accum_bytes(ccap))) != hipSuccess)
    return e;
  uint64_t* ukeys = (uint64_t*)w.tab.p;
  float* uvals = (float*)((char*)w.tab.p + 8 * (size_t)ccap);
  char* tail = (char*)uvals + (4 * (size_t)ccap + 255) / 256 * 256;
  uint64_t* dkeys = (uint64_t*)tail;
  int64_t* dx = (int64_t*)(dkeys + ccap);
  int64_t* dcnt = (int64_t*)(dx + ccap);
  char* uwork = (char*)(dcnt + 32);
  if (heavy_cand > 0 &&
      (e = hipMemcpyAsync(ukeys, ck, 8 * (size_t)heavy_cand,
                          hipMemcpyDeviceToDevice, st)) != hipSuccess)
    return e;
  if (W > 0) {
    if ((e = dev_alloc(w.pairs, pk + pv)) != hipSuccess ||
        (e = dev_alloc(w.acc, 16 * (size_t)W + 256 + accum_bytes(W))) !=
            hipSuccess)
      return e;
    uint64_t* lkeys = (uint64_t*)w.pairs.p;
    float* lvals = (float*)((char*)w.pairs.p + pk);
    const int64_t per_wave = 64 * kWedgeSteps;
    k_light_wedges<<<grid_of((W + per_wave - 1) / per_wave, 4, 1u << 20), 256,
                     0, st>>>((const int32_t*)w.lk.p,
                              (const int64_t*)w.wpre.p, nl, W, dtaptr, tarow,
                              taval, dtbptr, tbrow, tbval, n, lkeys, lvals);
    // fixed point: |products| < 2^(ea + eb), and a pair has no more of them
    // than either vector has light entries.  (With W, the wedges of all
    // pairs, in its place the slack W 2^-F, which grows as W^2, passed tau
    // at 5.4e8 wedges of lognormal values: 5.4e7 pairs to re-rank at 3e5 x
    // 3e5 and 192 columns, 257 now, and past 2^27 of them an error.)
    struct {
      float amax, bmax;
      unsigned most[2];
    } h;
    if ((e = hipMemcpyAsync(&h, lmax, sizeof h, hipMemcpyDeviceToHost, st)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
    const int64_t per_pair = h.most[0] < h.most[1] ? h.most[0] : h.most[1];
    int ea = 0, eb = 0, lw = 0;
    (void)frexpf(h.amax, &ea);
    (void)frexpf(h.bmax, &eb);
    while ((int64_t(1) << lw) < per_pair) ++lw;
    const int F = 62 - ea - eb - lw;
    uint64_t* okey = (uint64_t*)w.acc.p;
    int64_t* oval = (int64_t*)(okey + W);
    int64_t* lcnt = (int64_t*)(oval + W);
    char* awork = (char*)(lcnt + 32);
    if ((e = launch_accumulate(lkeys, lvals, W, nullptr, F, awork,
                               accum_bytes(W), okey, oval, lcnt, lcnt + 1,
                               st)) != hipSuccess)
      return e;
    unsigned long long* ucnt = (unsigned long long*)(lcnt + 2);
    if ((e = launch_fill_u64((uint64_t*)ucnt, 1, 0ull, st)) != hipSuccess)
      return e;
    k_light_prune<<<grid_of(W, 256 * 8, 8192), 256, 0, st>>>(
        okey, oval, lcnt + 1, F, ldexp((double)per_pair, -F), n, na, nb,
        tau_use,
        ukeys + heavy_cand, ucnt, lcap);
    unsigned long long got = 0;
    if ((e = hipMemcpyAsync(&got, ucnt, 8, hipMemcpyDeviceToHost, st)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
    if ((int64_t)got > lcap) return hipErrorOutOfMemory;
    light_cand = (int64_t)got;
  }
  (void)hipEventRecord(ev[3], st);
  // ---- union without repeats, exact dot products, top t --------------------
  const int64_t nu = heavy_cand + light_cand;
  int64_t distinct = 0;
  if (nu > 0) {
    if ((e = launch_fill_u64((uint64_t*)uvals, (nu + 1) / 2, 0ull, st)) !=
        hipSuccess)
      return e;
    if ((e = launch_accumulate(ukeys, uvals, nu, nullptr, 0, uwork,
                               accum_bytes(ccap), dkeys, dx, dcnt, dcnt + 1,
                               st)) != hipSuccess)
      return e;
    HashTable hsel;
    hsel.keys = dkeys;
    hsel.vals = dx;
    hsel.cap = nu;
    hsel.live = dcnt + 1;
    // the distinct keys to the front of ukeys
    if ((e = launch_dump_scores(hsel, (int64_t*)ukeys, (int64_t*)uwork, nu,
                                dcnt + 2, st)) != hipSuccess)
      return e;
    if ((e = hipMemcpyAsync(&distinct, dcnt + 2, 8, hipMemcpyDeviceToHost,
                            st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
      return e;
  }
  if (distinct > 0) {
    if ((e = launch_rerank_topk(ukeys, distinct, nullptr, nullptr, n, 0,
                                t < distinct ? t : distinct, w.fin, out, n_out,
                                &in, st)) != hipSuccess)
      return e;
  } else {
    if ((e = launch_fill_u64((uint64_t*)n_out, 1, 0ull, st)) != hipSuccess)
      return e;
  }
  (void)hipEventRecord(ev[4], st);
  if ((e = hipEventSynchronize(ev[4])) != hipSuccess) return e;
  if (stats) {
    float f;
    (void)hipEventElapsedTime(&f, ev[0], ev[1]);
    stats->ms_split = f;
    (void)hipEventElapsedTime(&f, ev[1], ev[2]);
    stats->ms_heavy = f;
    (void)hipEventElapsedTime(&f, ev[2], ev[3]);
    stats->ms_light = f;
    (void)hipEventElapsedTime(&f, ev[3], ev[4]);
    stats->ms_final = f;
    stats->heavy = H;
    stats->wedges = (int64_t)total;
    stats->light_wedges = W;
    stats->heavy_candidates = heavy_cand;
    stats->light_candidates = light_cand;
    stats->candidates = distinct;
    stats->tau = tau_use;
  }
  return hipSuccess;
}

hipError_t bruteforce_topk_csr(const CsrView& in, int64_t m, int64_t n,
                               int64_t d, int64_t nnzA, int64_t nnzB,
                               int prec, int64_t t, int64_t heavy_req,
                               void* out, int64_t* n_out, BfCsrStats* stats,
                               hipStream_t st) {
  bool again = heavy_req > 0;
  if (!again) {
    const hipError_t e =
        topk_csr_run(in, m, n, d, nnzA, nnzB, prec, t, 0, true, &again, out,
                     n_out, stats, st);
    // (more candidates than there is room for at this cut: there may be
    // fewer at the host's)
    if (e != hipErrorOutOfMemory && (e != hipSuccess || !again)) return e;
  }
  return topk_csr_run(in, m, n, d, nnzA, nnzB, prec, t, heavy_req, false,
                      &again, out, n_out, stats, st);
}

}  // namespace mad
