// mips.hip -- batched maximum inner product search (MIPS) with diamond
// sampling.
//
// A MIPS query is the MAD problem with a single vector on the B side
// (Sec. 2: a one-column matrix gives MIPS; Sec. 6 runs Alg. 3 once per
// query column).  Query q with budget s_q is exactly the general plan with
// B = {q}: the database tables T1 (i given k) and T3 (k' given i) are shared,
// stage 0 draws k with weight |q_k| v_k from the query's own table, the j
// draw of a one-vector B always returns 0 (its random word is still
// consumed, so sample l of query q uses the Philox block with counter
// (l, q, 0, 0) as in the general plan), the sign of b_kj is the sign of
// q_k, and the fourth edge is q_k'.  Scores are keyed by i alone.
//
// A score is one 64-bit word: the key i + 1 in the low kb bits (kb = bits of
// m) and x in the high 64 - kb bits, two's complement.  Adding inc << kb to
// it never changes its key bits, and x stays exact as long as it fits in 64
// - kb bits, which the exponent F = (general F) - kb guarantees (s_q
// increments of at most max|q| 2^F sum to at most 2^(62 - kb)).
//
// Queries of up to kMaxPartBudget samples sum their scores in LDS:
//   k_mips_query_info   per query: fixed-point exponent, finiteness;
//   k_sample_mips_part  persistent: workgroups walk a list of units (up to
//                       4096 consecutive samples of one query), order a
//                       unit's words by bin (of a hash of i) in LDS and store
//                       them in a row with the bins' offsets;
//   k_mips_bins         one workgroup per (query, bin): the bin's words of
//                       all units into a table in LDS, its distinct keys
//                       out, and, when every key with x > 0 is a candidate
//                       (t'_q >= min(s_q, m), fp32), their dot products;
//   k_mips_post         one workgroup per query (largest budgets first):
//                       the rest of Alg. 2 -- the t'_q largest x (ties by
//                       i), fp32 dot products where k_mips_bins left them,
//                       the t largest |c| (ties by i), in order.
// A sample then costs its table reads and 16 bytes of streamed traffic; in a
// table in memory each new key (97% of them) costs an atomic beyond L2, at
// 2.2e10 a second whatever the table's size.  Longer queries keep that
// table: k_sample_mips inserts by compare-and-swap and k_mips_post scans it.
#include "mad_common.hpp"
#include "plan.hpp"

namespace mad {

constexpr int kPostThreads = 1024;
constexpr int kPostWaves = kPostThreads / 64;
constexpr int kSelBinsM = 2048;
constexpr int kSelDigit = 11;
constexpr int kMaxOutT = 1024;  // t per query
constexpr int kFinCap = 2048;   // final selection list in LDS

// ---------------------------------------------------------------------------
// per query: F from max |q_k| and s_q; live = all entries finite
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mips_query_info(const float* Q,
                                                         int64_t nq,
                                                         int64_t d, int kb,
                                                         MipsQuery* qi,
                                                         MipsCount* qcnt,
                                                         SampleCounters* ctr) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctr->closed = 0;
    ctr->distinct = 0;
  }
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + wv;
  if (q >= nq) return;
  float mx = 0.0f;
  int nonfinite = 0;
  for (int64_t k = lane; k < d; k += 64) {
    const float v = Q[q * d + k];
    nonfinite |= !isfinite(v);
    mx = fmaxf(mx, fabsf(v));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    nonfinite |= __shfl_xor(nonfinite, off, 64);
  }
  if (lane == 0) {
    qi[q].F = fix_exponent(mx, qi[q].s) - kb;  // x shares a slot with i
    qi[q].live = nonfinite ? 0 : 1;
    qcnt[q].pos = 0;
    qcnt[q].rest = 0;
  }
}

hipError_t launch_mips_query_info(const float* Q, int64_t nq, int64_t d,
                                  int kb, MipsQuery* qi, MipsCount* qcnt,
                                  SampleCounters* ctr, hipStream_t st) {
  if (nq <= 0) return hipSuccess;
  k_mips_query_info<<<(unsigned)((nq + 3) / 4), 256, 0, st>>>(
      Q, nq, d, kb, qi, qcnt, ctr);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sampling: a persistent grid over the chunk list
// ---------------------------------------------------------------------------
size_t mips_sample_lds_bytes(int L0, int64_t d) {
  return ((size_t)8 << L0) + (size_t)4 * (size_t)d;
}

// Samples l0 + e[u] (e[u] < count) of query q: key i, increment and whether
// the diamond closes.  t0s, qs: the query's stage-0 table and row, in LDS.
template <int U>
__device__ __forceinline__ void mips_draws(const MipsArgs& a, int32_t q,
                                           int64_t l0, int e0, int step,
                                           int count, int F,
                                           const uint64_t* t0s,
                                           const float* qs,
                                           uint32_t (&key)[U],
                                           int64_t (&inc)[U],
                                           bool (&closed)[U]) {
  uint64_t e1[U], e3[U], U1[U], U3[U];
  uint32_t sg[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = e0 + u * step;
    const uint64_t l = (uint64_t)(l0 + (e < count ? e : 0));
    const Philox4 r = philox4x64_10(l, (uint64_t)q, 0ull, 0ull, a.seed, 0ull);
    const uint32_t s0 = slot_of(r.w0, a.L0);
    const uint32_t k = draw_entry(t0s[s0], s0, r.w0).pos;
    U1[u] = r.w1;
    U3[u] = r.w3;
    sg[u] = sign_bit(qs[k]);  // b_kj of the one-vector B is q_k
    e1[u] = a.T1[((uint64_t)k << a.L1) + slot_of(r.w1, a.L1)];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const Drawn di = draw_entry(e1[u], slot_of(U1[u], a.L1), U1[u]);
    key[u] = di.pos;
    sg[u] ^= di.sgn;
    e3[u] = a.T3[((uint64_t)di.pos << a.L3) + slot_of(U3[u], a.L3)];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const Drawn dk = draw_entry(e3[u], slot_of(U3[u], a.L3), U3[u]);
    const float v = qs[dk.pos];
    sg[u] ^= dk.sgn;
    closed[u] = e0 + u * step < count && v != 0.0f;
    inc[u] = 0;
    if (closed[u]) {
      const int64_t mag = (int64_t)rint(ldexp((double)v, F));
      inc[u] = sg[u] ? -mag : mag;
    }
  }
}

template <int U>
__global__ __launch_bounds__(256) void k_sample_mips(MipsArgs a) {
  extern __shared__ uint64_t sm[];
  const int N0 = 1 << a.L0;
  uint64_t* t0s = sm;
  float* qs = (float*)(sm + N0);
  unsigned long long nclosed = 0, ncreated = 0;
  for (int64_t c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const MipsChunk ch = a.chunks[c];
    const MipsQuery qi = a.qi[ch.q];
    if (!qi.live || !(a.t0tot[ch.q] > 0.0)) continue;  // uniform per block
    __syncthreads();  // the previous chunk is done with the LDS copies
    const uint64_t* t0g = a.T0q + ((int64_t)ch.q << a.L0);
    for (int e = threadIdx.x; e < N0; e += blockDim.x) t0s[e] = t0g[e];
    for (int64_t k = threadIdx.x; k < a.d; k += blockDim.x)
      qs[k] = a.Q[(int64_t)ch.q * a.d + k];
    __syncthreads();
    unsigned long long* hs = (unsigned long long*)(a.hslot + qi.hoff);
    const uint32_t hmask = qi.hmask;
    const int kb = a.kb;
    const uint64_t kmask = (1ull << kb) - 1;
    for (int base = threadIdx.x; base < ch.count; base += 256 * U) {
      uint32_t key[U], slot[U];
      int64_t inc[U];
      bool closed[U];
      mips_draws<U>(a, ch.q, ch.l0, base, 256, ch.count, qi.F, t0s, qs, key,
                    inc, closed);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        slot[u] = (uint32_t)mix64(key[u]) & hmask;
        nclosed += closed[u];
      }
      // claim an empty slot with key and increment in one swap; a slot
      // that already holds the key takes the increment by an add
      bool pend[U], add[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        pend[u] = closed[u];
        add[u] = false;
      }
      bool any = true;
      while (any) {
        unsigned long long prev[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          prev[u] = pend[u] ? atomicCAS(hs + slot[u], 0ull,
                                        ((uint64_t)inc[u] << kb) |
                                            ((uint64_t)key[u] + 1))
                            : 0ull;
        any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!pend[u]) continue;
          if (prev[u] == 0ull) {
            ++ncreated;
            pend[u] = false;
          } else if ((prev[u] & kmask) == (uint64_t)key[u] + 1) {
            add[u] = inc[u] != 0;
            pend[u] = false;
          } else {
            slot[u] = (slot[u] + 1) & hmask;
            any = true;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (add[u]) atomicAdd(hs + slot[u], (uint64_t)inc[u] << kb);
    }
  }
  __shared__ unsigned long long part[2][4];
  nclosed = wave_sum(nclosed);
  ncreated = wave_sum(ncreated);
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = nclosed;
    part[1][threadIdx.x >> 6] = ncreated;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long cc = part[0][0] + part[0][1] + part[0][2] +
                                  part[0][3];
    const unsigned long long dd = part[1][0] + part[1][1] + part[1][2] +
                                  part[1][3];
    if (cc) atomicAdd(&a.ctr->closed, cc);
    if (dd) atomicAdd(&a.ctr->distinct, dd);
  }
}

hipError_t launch_sample_mips(const MipsArgs& a, int unroll, int grid,
                              hipStream_t st) {
  if (a.nchunks <= 0) return hipSuccess;
  const size_t lds = mips_sample_lds_bytes(a.L0, a.d);
  int64_t g = grid < a.nchunks ? grid : a.nchunks;
  if (g < 1) g = 1;
  switch (unroll) {
    case 1: k_sample_mips<1><<<(unsigned)g, 256, lds, st>>>(a); break;
    case 2: k_sample_mips<2><<<(unsigned)g, 256, lds, st>>>(a); break;
    case 8: k_sample_mips<8><<<(unsigned)g, 256, lds, st>>>(a); break;
    default: k_sample_mips<4><<<(unsigned)g, 256, lds, st>>>(a); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sampling of the LDS-summed queries: a persistent grid over the units.
// Bound by the two random lines of a sample (T1[k], T3[i]); 512 threads so
// that the unit's 32 KB of words leaves 16 waves or more on a CU.
// ---------------------------------------------------------------------------
constexpr int kPartThreads = 512;

// Bin of key i, one of 2^lb: the top bits of a hash, so that every bin gets
// its share of the samples wherever the weight of the database lies, and a
// query's bins are unions of the bins of a query that has more.  (Ranges of
// i, on 1e6 x 128 rows ordered by norms falling as i^-0.5: most samples in a
// few bins, 22.9 ms for 4096 queries of 1e3 to 1e5 samples, 4.7 on the same
// rows in random order; 4.7 in either order with the hash.)  The factors are
// odd, near 2^32 over the golden ratio and over the square root of 2.
__device__ __forceinline__ uint32_t mips_bin(uint32_t i, int lb) {
  uint32_t h = i * 0x9E3779B1u;
  h = (h ^ (h >> 15)) * 0xB504F333u;
  return (uint32_t)(((uint64_t)h << lb) >> 32);
}

size_t mips_part_lds_bytes(int L0, int64_t d) {
  return (size_t)8 * kMipsUnit + mips_sample_lds_bytes(L0, d);
}

template <int U>
__global__ __launch_bounds__(kPartThreads) void k_sample_mips_part(
    MipsArgs a) {
  extern __shared__ uint64_t sm[];
  __shared__ unsigned cur[kMaxBins + 1];
  const int N0 = 1 << a.L0;
  uint64_t* words = sm;
  uint64_t* t0s = sm + kMipsUnit;
  float* qs = (float*)(t0s + N0);
  const int t = threadIdx.x;
  const uint64_t kmask = (1ull << a.kb) - 1;
  unsigned long long nclosed = 0;
  for (int64_t c = blockIdx.x; c < a.nunits; c += gridDim.x) {
    const MipsChunk ch = a.units[c];
    const MipsQuery qi = a.qi[ch.q];
    if (!qi.live || !(a.t0tot[ch.q] > 0.0)) continue;  // uniform per block
    __syncthreads();  // the previous unit is done with the LDS copies
    const uint64_t* t0g = a.T0q + ((int64_t)ch.q << a.L0);
    for (int e = t; e < N0; e += kPartThreads) t0s[e] = t0g[e];
    for (int64_t k = t; k < a.d; k += kPartThreads)
      qs[k] = a.Q[(int64_t)ch.q * a.d + k];
    for (int b = t; b <= qi.bins; b += kPartThreads) cur[b] = 0;
    __syncthreads();
    for (int base = t; base < ch.count; base += kPartThreads * U) {
      uint32_t key[U];
      int64_t inc[U];
      bool closed[U];
      mips_draws<U>(a, ch.q, ch.l0, base, kPartThreads, ch.count, qi.F, t0s,
                    qs, key, inc, closed);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = base + u * kPartThreads;
        if (e >= ch.count) continue;
        words[e] = closed[u] ? ((uint64_t)inc[u] << a.kb) |
                                   ((uint64_t)key[u] + 1)
                             : 0ull;
        if (closed[u]) atomicAdd(&cur[mips_bin(key[u], qi.lb)], 1u);
        nclosed += closed[u];
      }
    }
    __syncthreads();
    // starts of the bins, to the offsets and as write cursors
    uint16_t* offs = a.offs + qi.ooff +
                     (ch.l0 / a.unit) * (int64_t)(qi.bins + 1);
    if (t < 64) {
      unsigned carry = 0;
      for (int b0 = 0; b0 <= qi.bins; b0 += 64) {
        const int b = b0 + t;
        const unsigned v = b < qi.bins ? cur[b] : 0u;
        const unsigned incl = wave_incl_scan(v);
        if (b <= qi.bins) {
          cur[b] = carry + incl - v;
          offs[b] = (uint16_t)(carry + incl - v);
        }
        carry += __shfl(incl, 63, 64);
      }
    }
    __syncthreads();
    const unsigned total = cur[qi.bins];
    constexpr int kPer = kMipsUnit / kPartThreads;
    uint64_t w[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int e = t + r * kPartThreads;
      w[r] = e < ch.count ? words[e] : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r)
      if (w[r])
        words[atomicAdd(
            &cur[mips_bin((uint32_t)(w[r] & kmask) - 1u, qi.lb)], 1u)] = w[r];
    __syncthreads();
    // regions start on 16 bytes and hold an even number of words: the pair
    // after an odd total is not read
    ulonglong2* o = (ulonglong2*)(a.part + qi.poff + ch.l0);
    const ulonglong2* in = (const ulonglong2*)words;
    for (unsigned e = t; e < (total + 1) / 2; e += kPartThreads) o[e] = in[e];
  }
  __shared__ unsigned long long part[kPartThreads / 64];
  nclosed = wave_sum(nclosed);
  if ((t & 63) == 0) part[t >> 6] = nclosed;
  __syncthreads();
  if (t == 0) {
    unsigned long long cc = 0;
    for (int w = 0; w < kPartThreads / 64; ++w) cc += part[w];
    if (cc) atomicAdd(&a.ctr->closed, cc);
  }
}

// ---------------------------------------------------------------------------
// verification: c = a_i . q in fp32, 16 lanes per candidate, kVerU
// candidates of a lane group at once (their row loads in flight together),
// rows read as float4 when `vec` (d a multiple of 4, A on 16 bytes)
// ---------------------------------------------------------------------------
constexpr int kVerU = 4;

__device__ __forceinline__ void mips_dots(const float* const (&ar)[kVerU],
                                          const bool (&need)[kVerU],
                                          const float* qs, int64_t d,
                                          bool vec, int gl,
                                          float (&acc)[kVerU]) {
#pragma unroll
  for (int u = 0; u < kVerU; ++u) acc[u] = 0.0f;
  if (vec) {
    for (int64_t k = gl * 4; k < d; k += 64) {
      const float4 y = *(const float4*)(qs + k);
      float4 x[kVerU];
#pragma unroll
      for (int u = 0; u < kVerU; ++u)
        x[u] = need[u] ? *(const float4*)(ar[u] + k)
                       : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
      for (int u = 0; u < kVerU; ++u) {
        acc[u] = fmaf(x[u].x, y.x, acc[u]);
        acc[u] = fmaf(x[u].y, y.y, acc[u]);
        acc[u] = fmaf(x[u].z, y.z, acc[u]);
        acc[u] = fmaf(x[u].w, y.w, acc[u]);
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < kVerU; ++u)
      if (need[u])
        for (int64_t k = gl; k < d; k += 16)
          acc[u] = fmaf(ar[u][k], qs[k], acc[u]);
  }
#pragma unroll
  for (int u = 0; u < kVerU; ++u)
#pragma unroll
    for (int off = 8; off > 0; off >>= 1)
      acc[u] += __shfl_xor(acc[u], off, 64);
}

// ---------------------------------------------------------------------------
// one (query, bin) per workgroup: the bin's words of every unit of the query
// into an open-addressing table in LDS, then its distinct keys out, those
// with x > 0 from the front of the query's region and the rest from its
// back.  A bin expects at most about 1024 words and the table has 2048
// slots; words that do not fit (keys that the hash puts in one bin) are
// taken in halves, quarters, ... of the keys' hashes, each in a pass of its
// own.  What bounds it is a chain of eight or so memory latencies per item,
// so it wants workgroups in flight more than slots: 2.51 ms at 4096 queries
// of 1e3 to 1e5 samples on 1e6 x 128, 3.49 ms with 4096 slots.
//
// The items go through the bins in order, all queries of a bin together, so
// that the rows a bin verifies (1/128 of the database for a query of 1e5
// samples: 4 MB at 1e6 x 128) are shared in L2 by the queries instead of
// being fetched for each.
// ---------------------------------------------------------------------------
constexpr int kBinThreads = 256;
constexpr int kBinSlots = 2048;  // 16 KB: 8 workgroups on a CU
constexpr int kBinProbes = 128;  // a longer chain counts as a full table

__global__ __launch_bounds__(kBinThreads) void k_mips_bins(MipsArgs a) {
  // the query row (fused verification)
  extern __shared__ __attribute__((aligned(16))) float qs[];
  __shared__ __attribute__((aligned(16))) uint64_t tab[kBinSlots];
  __shared__ unsigned nwords, npos, nrest;
  __shared__ unsigned gpos, grest;
  __shared__ int full;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const MipsItem it = a.items[blockIdx.x];
  const MipsQuery qi = a.qi[it.q];
  if (!qi.live || !(a.t0tot[it.q] > 0.0)) return;
  const int64_t units = (qi.s + a.unit - 1) / a.unit;
  const int64_t ostep = qi.bins + 1;
  const uint16_t* offs = a.offs + qi.ooff + it.bin;
  const uint64_t kmask = (1ull << a.kb) - 1;
  if (t == 0) nwords = 0;
  __syncthreads();
  unsigned mine = 0;
  for (int64_t u = t; u < units; u += kBinThreads)
    mine += (unsigned)offs[u * ostep + 1] - (unsigned)offs[u * ostep];
  mine = wave_sum(mine);
  if (lane == 0 && mine) atomicAdd(&nwords, mine);
  const bool fused = a.lp == 0 && qi.tp >= qi.ccap;
  if (fused)
    for (int64_t k = t; k < a.d; k += kBinThreads)
      qs[k] = a.Q[(int64_t)it.q * a.d + k];
  __syncthreads();
  const unsigned words = nwords;
  if (words == 0) return;
  unsigned slots = 256;
  while (slots < 2 * words && slots < (unsigned)kBinSlots) slots <<= 1;
  const bool vec = (a.d & 3) == 0 && ((uintptr_t)a.A & 15) == 0;
  uint64_t* region = a.hslot + qi.hoff;
  // 16 lanes per unit, more when there are fewer than 16 units
  int lw = 8;
  while (lw > 4 && (kBinThreads >> lw) < units) --lw;
  int depth = 0;       // this pass: keys whose hash starts with the
  uint64_t prefix = 0; // `depth` bits `prefix`
  while (true) {
    for (unsigned e = t; e < slots; e += kBinThreads) tab[e] = 0ull;
    if (t == 0) {
      full = 0;
      npos = 0;
      nrest = 0;
    }
    __syncthreads();
    for (int64_t u = t >> lw; u < units; u += kBinThreads >> lw) {
      const unsigned st = offs[u * ostep], en = offs[u * ostep + 1];
      const uint64_t* in = a.part + qi.poff + u * a.unit;
      for (unsigned e = st + (t & ((1 << lw) - 1)); e < en; e += 1u << lw) {
        const uint64_t w = in[e];
        const uint64_t h = mix64((w & kmask) - 1);
        if (depth && (h >> (64 - depth)) != prefix) continue;
        unsigned slot = (unsigned)h & (slots - 1);
        for (int probe = 0;; ++probe) {
          if (probe == kBinProbes) {
            full = 1;
            break;
          }
          const uint64_t prev =
              atomicCAS((unsigned long long*)&tab[slot], 0ull, w);
          if (prev == 0ull) break;
          if (((prev ^ w) & kmask) == 0) {
            atomicAdd((unsigned long long*)&tab[slot], w & ~kmask);
            break;
          }
          slot = (slot + 1) & (slots - 1);
        }
      }
    }
    __syncthreads();
    if (full) {  // uniform; mix64 is one to one, so halving ends
      ++depth;
      prefix <<= 1;
      __syncthreads();
      continue;
    }
    // the keys with x > 0 to the front of the table (through registers)
    constexpr int kPer = kBinSlots / kBinThreads;
    uint64_t w[kPer];
    unsigned cp = 0, cr = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const unsigned e = t + r * kBinThreads;
      w[r] = e < slots ? tab[e] : 0ull;
      cp += (int64_t)w[r] >> a.kb > 0;
      cr += w[r] != 0ull && (int64_t)w[r] >> a.kb <= 0;
    }
    const unsigned ip = wave_incl_scan(cp), ir = wave_incl_scan(cr);
    unsigned bp = 0, br = 0;
    if (lane == 63) {
      bp = atomicAdd(&npos, ip);
      br = atomicAdd(&nrest, ir);
    }
    unsigned at = __shfl(bp, 63, 64) + ip - cp;
    unsigned rt = __shfl(br, 63, 64) + ir - cr;
    __syncthreads();  // every slot is in registers, the counts are whole
    if (t == 0) {
      gpos = npos ? atomicAdd(&a.qcnt[it.q].pos, npos) : 0u;
      grest = nrest ? atomicAdd(&a.qcnt[it.q].rest, nrest) : 0u;
    }
    __syncthreads();
    const int64_t back = qi.ccap - 1 - (int64_t)grest;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      if (w[r] == 0ull) continue;
      if ((int64_t)w[r] >> a.kb > 0)
        tab[at++] = w[r];
      else
        region[back - (int64_t)rt++] = w[r];
    }
    __syncthreads();
    const unsigned np = npos;
    for (unsigned e = t; e < np; e += kBinThreads)
      region[(int64_t)gpos + e] = tab[e];
    if (fused) {
      float* sc = a.sc + qi.soff + gpos;
      const int grp = lane >> 4, gl = lane & 15;
      constexpr unsigned kRound = kBinThreads / 16;
      for (unsigned r0 = wv * 4; r0 < np; r0 += kRound * kVerU) {
        bool need[kVerU];
        const float* ar[kVerU];
        float acc[kVerU];
#pragma unroll
        for (int u = 0; u < kVerU; ++u) {
          const unsigned e = r0 + grp + u * kRound;
          need[u] = e < np;
          ar[u] = a.A + (int64_t)((tab[need[u] ? e : r0] & kmask) - 1) * a.d;
        }
        mips_dots(ar, need, qs, a.d, vec, gl, acc);
#pragma unroll
        for (int u = 0; u < kVerU; ++u)
          if (need[u] && gl == 0) sc[r0 + grp + u * kRound] = acc[u];
      }
    }
    if (depth == 0) break;
    // the next part of the hash range, as wide as it can be
    ++prefix;
    while (depth > 0 && !(prefix & 1)) {
      prefix >>= 1;
      --depth;
    }
    if (depth == 0) break;
    __syncthreads();
  }
}

hipError_t launch_sample_mips_part(const MipsArgs& a, int unroll, int grid,
                                   hipStream_t st) {
  if (a.nunits <= 0) return hipSuccess;
  const size_t lds = mips_part_lds_bytes(a.L0, a.d);
  int64_t g = grid < a.nunits ? grid : a.nunits;
  if (g < 1) g = 1;
  switch (unroll) {
    case 1:
      k_sample_mips_part<1><<<(unsigned)g, kPartThreads, lds, st>>>(a);
      break;
    case 2:
      k_sample_mips_part<2><<<(unsigned)g, kPartThreads, lds, st>>>(a);
      break;
    case 8:
      k_sample_mips_part<8><<<(unsigned)g, kPartThreads, lds, st>>>(a);
      break;
    default:
      k_sample_mips_part<4><<<(unsigned)g, kPartThreads, lds, st>>>(a);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_mips_bins(const MipsArgs& a, hipStream_t st) {
  if (a.nitems <= 0) return hipSuccess;
  k_mips_bins<<<(unsigned)a.nitems, kBinThreads, (size_t)4 * a.d, st>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// postprocessing helpers (1024 threads)
// ---------------------------------------------------------------------------
struct PostShared {
  unsigned h[kSelBinsM];
  unsigned long long scan[kPostThreads];
  unsigned wcnt[kPostWaves];
  unsigned long long base;
  int chosen;
  unsigned long long before;
};

// Slot of this thread among the takers of one round of the whole block, in
// thread order, after `ps.base`; advances ps.base by the round's count.
__device__ int64_t block_take(bool take, PostShared& ps) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t ball = __ballot(take);
  if (lane == 0) ps.wcnt[wv] = (unsigned)__popcll(ball);
  __syncthreads();
  unsigned before = 0, total = 0;
  for (int w = 0; w < kPostWaves; ++w) {
    const unsigned c = ps.wcnt[w];
    before += w < wv ? c : 0u;
    total += c;
  }
  const int64_t slot = (int64_t)ps.base + before +
                       __popcll(ball & ((1ull << lane) - 1));
  __syncthreads();
  if (threadIdx.x == 0) ps.base += total;
  __syncthreads();
  return slot;
}

// First slot of this thread's `cnt` takers among those of one round of the
// whole block, in thread order, after `ps.base`; advances ps.base by the
// round's count.
__device__ int64_t block_take_n(unsigned cnt, PostShared& ps) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned incl = wave_incl_scan(cnt);
  if (lane == 63) ps.wcnt[wv] = incl;
  __syncthreads();
  unsigned before = 0, total = 0;
  for (int w = 0; w < kPostWaves; ++w) {
    const unsigned c = ps.wcnt[w];
    before += w < wv ? c : 0u;
    total += c;
  }
  const int64_t slot = (int64_t)ps.base + before + (incl - cnt);
  __syncthreads();
  if (threadIdx.x == 0) ps.base += total;
  __syncthreads();
  return slot;
}

// Threshold of an exact selection of k of n elements by (primary desc,
// key asc): the elements taken are those with take(p, key) true.  Digits
// of kSelDigit bits, from bit `top` of the primary down, then the 32-bit
// key.  Keys are unique, so the key phase always ends the search.
struct SelThr {
  uint64_t pp, pm;
  uint32_t kp, km;
  int key_phase;
};

__device__ __forceinline__ bool sel_take(uint64_t p, uint32_t kk,
                                         const SelThr& s) {
  const uint64_t pmv = p & s.pm;
  if (pmv != s.pp) return pmv > s.pp;
  if (!s.key_phase) return true;
  return (kk & s.km) <= s.kp;
}

template <class PrimOf, class KeyOf>
__device__ SelThr block_select(const PrimOf& prim, const KeyOf& key,
                               int64_t n, int64_t k, int top,
                               PostShared& ps) {
  const int t = threadIdx.x;
  SelThr s{0, 0, 0, 0, 0};
  int64_t k_rem = k;
  int shift = top - kSelDigit > 0 ? top - kSelDigit : 0;
  bool done = k_rem >= n;
  while (!done) {
    for (int b = t; b < kSelBinsM; b += kPostThreads) ps.h[b] = 0;
    __syncthreads();
    for (int64_t e = t; e < n; e += kPostThreads) {
      const uint64_t p = prim(e);
      if ((p & s.pm) != s.pp) continue;
      if (!s.key_phase) {
        atomicAdd(&ps.h[(p >> shift) & (kSelBinsM - 1)], 1u);
      } else {
        const uint32_t kk = key(e);
        if ((kk & s.km) != s.kp) continue;
        atomicAdd(&ps.h[(kk >> shift) & (kSelBinsM - 1)], 1u);
      }
    }
    __syncthreads();
    // bins in selection order; thread t owns positions 2t, 2t + 1
    const int b0 = s.key_phase ? 2 * t : kSelBinsM - 1 - 2 * t;
    const int b1 = s.key_phase ? 2 * t + 1 : kSelBinsM - 2 - 2 * t;
    const unsigned v0 = ps.h[b0], v1 = ps.h[b1];
    ps.scan[t] = (unsigned long long)v0 + v1;
    if (t == 0) ps.chosen = -1;
    __syncthreads();
    for (int off = 1; off < kPostThreads; off <<= 1) {
      const unsigned long long o = t >= off ? ps.scan[t - off] : 0ull;
      __syncthreads();
      ps.scan[t] += o;
      __syncthreads();
    }
    const unsigned long long excl = ps.scan[t] - v0 - v1;
    if ((long long)excl < k_rem && (long long)(excl + v0) >= k_rem) {
      ps.chosen = b0;
      ps.before = excl;
    } else if ((long long)(excl + v0) < k_rem &&
               (long long)(excl + v0 + v1) >= k_rem) {
      ps.chosen = b1;
      ps.before = excl + v0;
    }
    __syncthreads();
    const int b = ps.chosen;
    const unsigned nbin = b >= 0 ? ps.h[b] : 0u;
    const unsigned long long bef = ps.before;
    __syncthreads();
    if (b < 0) break;  // cannot happen while k_rem <= matching count
    k_rem -= (int64_t)bef;
    if (!s.key_phase) {
      s.pp |= (uint64_t)b << shift;
      s.pm |= (uint64_t)(kSelBinsM - 1) << shift;
    } else {
      s.kp |= (uint32_t)b << shift;
      s.km |= (uint32_t)(kSelBinsM - 1) << shift;
    }
    if ((int64_t)nbin == k_rem) {
      done = true;
    } else if (shift == 0) {
      if (s.key_phase) done = true;
      s.key_phase = 1;
      shift = 32 - kSelDigit;
    } else {
      shift = shift > kSelDigit ? shift - kSelDigit : 0;
    }
  }
  return s;
}

// Histograms over the bits of a float >= 0 shifted right by 20 (exponent
// and three mantissa bits, kSelBinsM bins): bin(v) is monotone in v, and
// every v in bin b is at least edge(b), the float with bits b << 20.
__device__ __forceinline__ unsigned fbin(uint32_t bits) { return bits >> 20; }
__device__ __forceinline__ float fbin_edge(int b) {
  return __uint_as_float((uint32_t)b << 20);
}

// The bin b of the histogram ps.h that holds the k-th largest value: bins
// above b hold fewer than k values, bins from b up at least k.  Wave 0
// searches (32 bins per lane, from the top); ps.chosen = b (-1 when the
// histogram holds fewer than k values) and ps.before = the count in bins
// >= b.  The histogram must be complete; synchronise before reading.
__device__ void hist_kth_bin(PostShared& ps, int64_t k) {
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  const int hi = kSelBinsM - 1 - 32 * lane;
  unsigned long long sum = 0;
  for (int b = hi; b > hi - 32; --b) sum += ps.h[b];
  const unsigned long long incl = wave_incl_scan(sum);
  const uint64_t reach = __ballot((long long)incl >= k);
  if (lane == 0 && reach == 0) ps.chosen = -1;
  if (reach == 0) return;
  if (lane != __builtin_ctzll(reach)) return;
  unsigned long long acc = incl - sum;
  for (int b = hi; b > hi - 32; --b) {
    acc += ps.h[b];
    if ((long long)acc >= k) {
      ps.chosen = b;
      ps.before = acc;
      return;
    }
  }
}

// ---------------------------------------------------------------------------
// post: one workgroup per query
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kPostThreads) void k_mips_post(MipsArgs a) {
  extern __shared__ __attribute__((aligned(16))) float qs[];  // query row
  __shared__ PostShared ps;
  __shared__ uint32_t fk[kMaxOutT];
  __shared__ uint64_t fx[kMaxOutT];
  __shared__ float fc[kMaxOutT];
  __shared__ uint32_t lk[kFinCap];  // final-selection list: keys,
  __shared__ float lc[kFinCap];     // c,
  __shared__ int32_t le[kFinCap];   // positions in the verified arrays
  __shared__ unsigned nl;
  const int t = threadIdx.x;
  const int64_t q = a.order[blockIdx.x];
  const MipsQuery qi = a.qi[q];
  if (!qi.live || !(a.t0tot[q] > 0.0) || qi.s <= 0) {
    if (t == 0) {
      a.n_out[q] = qi.live ? 0 : -1;
      a.qstats[q].n_pos = 0;
      a.qstats[q].n_cand = 0;
      a.qstats[q].n_fp32 = 0;
    }
    return;
  }
  for (int64_t k = t; k < a.d; k += kPostThreads) qs[k] = a.Q[q * a.d + k];
  const uint64_t kmask = (1ull << a.kb) - 1;
  // candidates (Omega_s): the keys with x > 0.  k_mips_bins has listed them;
  // a table in memory is scanned, and its words compacted in slot order
  const uint64_t* cw = a.hslot + qi.hoff;
  int64_t npos = 0;
  if (qi.bins) {
    npos = (int64_t)a.qcnt[q].pos;
    __syncthreads();
  } else {
    const uint64_t* hs = cw;
    uint64_t* lw = a.cw + qi.coff;
    const int64_t cap = (int64_t)qi.hmask + 1;
    if (t == 0) ps.base = 0;
    __syncthreads();
    // kScanPer consecutive slots per thread and round (the table capacity
    // is a power of two of at least 1024 slots, so rounds are whole)
    constexpr int kScanPer = 8;
    for (int64_t r0 = 0; r0 < cap; r0 += kPostThreads * kScanPer) {
      const int64_t e0 = r0 + (int64_t)t * kScanPer;
      uint64_t w[kScanPer];
      unsigned cnt = 0;
#pragma unroll
      for (int u = 0; u < kScanPer; ++u) {
        w[u] = e0 + u < cap ? hs[e0 + u] : 0ull;
        cnt += (int64_t)w[u] >> a.kb > 0;
      }
      int64_t pos = block_take_n(cnt, ps);
#pragma unroll
      for (int u = 0; u < kScanPer; ++u)
        if ((int64_t)w[u] >> a.kb > 0) {
          if (pos < qi.ccap) lw[pos] = w[u];
          ++pos;
        }
    }
    npos = (int64_t)ps.base;
    cw = lw;
  }
  if (npos > qi.ccap) npos = qi.ccap;  // cannot happen: distinct <= s_q, m
  // candidate selection (Omega_t'): the t'_q largest x, ties by i
  // ascending; when all are taken, the candidate words serve as they are
  const bool cut = npos > qi.tp;
  uint64_t* sel = a.sw + qi.soff;
  float* sc = a.sc + qi.soff;
  uint32_t* sab = a.sab + qi.soff;
  int64_t nsel = npos;
  if (cut) {
    const SelThr thr = block_select(
        [&](int64_t e) { return cw[e] >> a.kb; },
        [&](int64_t e) { return (uint32_t)(cw[e] & kmask) - 1u; }, npos,
        qi.tp, 64, ps);
    nsel = qi.tp;
    __syncthreads();
    if (t == 0) ps.base = 0;
    __syncthreads();
    for (int64_t r0 = 0; r0 < npos; r0 += kPostThreads) {
      const int64_t e = r0 + t;
      const uint64_t w = e < npos ? cw[e] : 0;
      const bool take =
          e < npos &&
          sel_take(w >> a.kb, (uint32_t)(w & kmask) - 1u, thr);
      const int64_t pos = block_take(take, ps);
      if (take && pos < qi.scap) sel[pos] = w;
    }
    cw = sel;
  }
  if (nsel > qi.scap) nsel = qi.scap;
  __syncthreads();
  auto key_of = [&](int64_t e) { return (uint32_t)(cw[e] & kmask) - 1u; };
  const int lane = t & 63, wv = t >> 6, grp = lane >> 4, gl = lane & 15;
  const int64_t tq = a.t < nsel ? a.t : nsel;
  // low-precision screen (when the plan asks for one and more than t
  // candidates remain): c^ of every candidate from the bf16 / fp8 rows and
  // the bound mg on |c^ - c_fp32|; tau <= the t-th largest lower bound
  // |c^| - mg; only candidates with |c^| + mg >= tau are verified in fp32.
  // Every other candidate has |c_fp32| < tau <= the fp32 |c| of t others,
  // so the top t is the one the fp32 verification of all of them gives.
  // tau is the lower edge of the histogram bin that holds the t-th largest
  // lower bound (at most that bound), from a histogram the screen pass
  // fills as it goes.
  const bool screen = a.lp != 0 && nsel > tq;
  float tau = 0.0f;
  for (int b = t; b < kSelBinsM; b += kPostThreads) ps.h[b] = 0;
  __syncthreads();
  if (screen) {
    const int64_t rowb = a.Kp * (a.lp == 1 ? 2 : 1);  // bytes per row
    const uint4* qrow = (const uint4*)((const char*)a.Qlp + q * rowb);
    const VecInfo vq = a.iq[q];
    // kScrU rounds of 4 candidates per wave at once, as in verification below
    constexpr int kScrU = 4;
    const int64_t round = kPostWaves * 4;
    for (int64_t e0 = (int64_t)wv * 4; e0 < nsel; e0 += round * kScrU) {
      const uint4* arow[kScrU];
      int64_t iu[kScrU];
      float acc[kScrU];
      VecInfo va[kScrU];  // loaded with the rows, used by lane gl = 0
#pragma unroll
      for (int u = 0; u < kScrU; ++u) {
        const int64_t e = e0 + grp + u * round;
        iu[u] = (int64_t)key_of(e < nsel ? e : e0);
        arow[u] = (const uint4*)((const char*)a.Alp + iu[u] * rowb);
        acc[u] = 0.0f;
        if (gl == 0) va[u] = a.ia[iu[u]];
      }
      for (int64_t c16 = gl; c16 < rowb / 16; c16 += 16) {
        const uint4 y = qrow[c16];
        uint4 x[kScrU];
#pragma unroll
        for (int u = 0; u < kScrU; ++u) x[u] = arow[u][c16];
#pragma unroll
        for (int u = 0; u < kScrU; ++u)
          acc[u] = lowp_dot16(x[u], y, a.lp, acc[u]);
      }
#pragma unroll
      for (int u = 0; u < kScrU; ++u) {
#pragma unroll
        for (int off = 8; off > 0; off >>= 1)
          acc[u] += __shfl_xor(acc[u], off, 64);
        const int64_t e = e0 + grp + u * round;
        if (e < nsel && gl == 0) {
          const float c = acc[u] * va[u].inv_s * vq.inv_s;
          const float mg = a.kappa * va[u].n2 * vq.n2 +
                           a.onepu * (va[u].eta * vq.n1 + vq.eta * va[u].n1) +
                           a.d_f * va[u].eta * vq.eta;
          const float lo = fabsf(c) - mg;
          atomicAdd(&ps.h[fbin(__float_as_uint(lo > 0.0f ? lo : 0.0f))], 1u);
          sab[e] = 0;  // |c| of the candidates verified below
          sc[e] = fabsf(c) + mg;
        }
      }
    }
    __syncthreads();
    hist_kth_bin(ps, tq);
    __syncthreads();
    tau = ps.chosen > 0 ? fbin_edge(ps.chosen) : 0.0f;
    if (t == 0) nl = 0;
    __syncthreads();
    for (int b = t; b < kSelBinsM; b += kPostThreads) ps.h[b] = 0;
    // the candidates left to verify (upper bound >= tau), listed in LDS
    for (int64_t e = t; e < nsel; e += kPostThreads)
      if (sc[e] >= tau) {
        const unsigned p = atomicAdd(&nl, 1u);
        if (p < (unsigned)kFinCap) le[p] = (int32_t)e;
      }
  }
  if (t == 0) ps.base = 0;
  __syncthreads();
  // verify the listed candidates, or (no screen, or a list that did not
  // fit) every candidate whose bound reaches tau
  const bool via_list = screen && nl <= (unsigned)kFinCap;
  const int64_t nv = via_list ? (int64_t)nl : nsel;
  // verification, and a histogram of |c| filled as the values come
  unsigned nfp = 0;
  if (qi.bins && a.lp == 0 && qi.tp >= qi.ccap) {  // done by k_mips_bins
    for (int64_t e = t; e < nsel; e += kPostThreads) {
      atomicAdd(&ps.h[fbin(__float_as_uint(fabsf(sc[e])))], 1u);
      ++nfp;
    }
  } else {
    const int64_t round = kPostWaves * 4;  // candidates per block round
    const bool vec = (a.d & 3) == 0 && ((uintptr_t)a.A & 15) == 0;
    for (int64_t r0 = (int64_t)wv * 4; r0 < nv; r0 += round * kVerU) {
      bool need[kVerU];
      int64_t ev[kVerU];
      const float* ar[kVerU];
      float acc[kVerU];
#pragma unroll
      for (int u = 0; u < kVerU; ++u) {
        const int64_t r = r0 + grp + u * round;
        ev[u] = r < nv ? (via_list ? (int64_t)le[r] : r) : 0;
        need[u] = r < nv && (via_list || !screen || sc[ev[u]] >= tau);
        ar[u] = a.A + (int64_t)key_of(ev[u]) * a.d;
      }
      mips_dots(ar, need, qs, a.d, vec, gl, acc);
#pragma unroll
      for (int u = 0; u < kVerU; ++u)
        if (need[u] && gl == 0) {
          const uint32_t ab = __float_as_uint(fabsf(acc[u]));
          sc[ev[u]] = acc[u];
          if (screen) sab[ev[u]] = ab;
          atomicAdd(&ps.h[fbin(ab)], 1u);
          ++nfp;
        }
    }
  }
  // |c| bits; a screened-out candidate's are 0
  auto abs_of = [&](int64_t e) {
    return screen ? sab[e] : __float_as_uint(fabsf(sc[e]));
  };
  if (nfp) atomicAdd((unsigned long long*)&ps.base, (unsigned long long)nfp);
  __syncthreads();
  const int64_t n_fp32 = (int64_t)ps.base;
  // final selection: the t largest |c|, ties by i ascending.  The
  // histogram gives the bin b of the t-th largest |c|; the candidates of
  // bins >= b (every one verified: a screened-out candidate keeps |c| = 0
  // and b >= 1) go to an LDS list where each one's rank is counted
  // directly.  A list that would not fit, or b = 0, takes the digit
  // selection over all candidates instead.
  const bool cut3 = nsel > tq;
  bool listed = false;
  if (cut3) {
    hist_kth_bin(ps, tq);
    if (t == 0) nl = 0;
    __syncthreads();
    const int b3 = ps.chosen;
    listed = b3 >= 1 && ps.before <= (unsigned long long)kFinCap;
    __syncthreads();
    if (listed) {
      for (int64_t e = t; e < nsel; e += kPostThreads) {
        const uint32_t ab = abs_of(e);
        if ((int)fbin(ab) >= b3) {
          const unsigned p = atomicAdd(&nl, 1u);
          lk[p] = key_of(e);
          lc[p] = sc[e];
          le[p] = (int32_t)e;
        }
      }
      __syncthreads();
      const int n = (int)nl;
      for (int e = t; e < n; e += kPostThreads) {
        const uint32_t ae = __float_as_uint(fabsf(lc[e]));
        const uint32_t ke = lk[e];
        int rank = 0;
        for (int u = 0; u < n; ++u) {
          const uint32_t au = __float_as_uint(fabsf(lc[u]));
          rank += au > ae || (au == ae && lk[u] < ke);
        }
        if (rank < tq) {
          fk[rank] = ke;
          fx[rank] = cw[le[e]] >> a.kb;
          fc[rank] = lc[e];
        }
      }
      __syncthreads();
    }
  }
  if (!listed) {
    SelThr thr3{0, 0, 0, 0, 0};
    if (cut3)
      thr3 = block_select([&](int64_t e) { return (uint64_t)abs_of(e); },
                          key_of, nsel, tq, 32, ps);
    __syncthreads();
    if (t == 0) ps.base = 0;
    __syncthreads();
    for (int64_t r0 = 0; r0 < nsel; r0 += kPostThreads) {
      const int64_t e = r0 + t;
      const bool live = e < nsel;
      const uint64_t p = live ? abs_of(e) : 0;
      const uint32_t kk = live ? key_of(e) : 0;
      const bool take = live && (!cut3 || sel_take(p, kk, thr3));
      const int64_t pos = block_take(take, ps);
      if (take && pos < tq) {
        fk[pos] = kk;
        fx[pos] = cw[e] >> a.kb;
        fc[pos] = sc[e];
      }
    }
    __syncthreads();
  }
  // rank order (|c| desc, i asc) and output
  struct Pair {
    int64_t i, j;
    float c, x;
  };
  Pair* o = (Pair*)a.out + q * a.t;
  for (int64_t e = t; e < tq; e += kPostThreads) {
    const float ae = fabsf(fc[e]);
    const uint32_t ke = fk[e];
    int64_t rank = 0;
    for (int64_t u = 0; u < tq; ++u) {
      const float au = fabsf(fc[u]);
      rank += au > ae || (au == ae && fk[u] < ke);
    }
    Pair pr;
    pr.i = (int64_t)ke;
    pr.j = q;
    pr.c = fc[e];
    pr.x = (float)ldexp((double)(int64_t)fx[e], -qi.F);
    o[rank] = pr;
  }
  if (t == 0) {
    a.n_out[q] = tq;
    a.qstats[q].n_pos = npos;
    a.qstats[q].n_cand = nsel;
    a.qstats[q].n_fp32 = n_fp32;
  }
}

hipError_t launch_mips_post(const MipsArgs& a, hipStream_t st) {
  if (a.nq <= 0) return hipSuccess;
  if (a.t > kMaxOutT) return hipErrorInvalidValue;
  k_mips_post<<<(unsigned)a.nq, kPostThreads, (size_t)4 * a.d, st>>>(a);
  return hipGetLastError();
}

// every key of query q's scores, for parity checks
__global__ void k_mips_dump(const uint64_t* hs, int kb, int64_t cap,
                            int64_t* keys, int64_t* xfix, int64_t out_cap,
                            int64_t* count) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const uint64_t kmask = (1ull << kb) - 1;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < cap;
       e += stride) {
    const uint64_t w = hs[e];
    if (w == 0) continue;
    const unsigned long long p = atomicAdd((unsigned long long*)count, 1ull);
    if ((int64_t)p < out_cap) {
      keys[p] = (int64_t)(w & kmask) - 1;
      xfix[p] = (int64_t)w >> kb;
    }
  }
}

hipError_t launch_mips_dump(const MipsArgs& a, int64_t q, int64_t* keys,
                            int64_t* xfix, int64_t cap, int64_t* count,
                            hipStream_t st) {
  MipsQuery qi;
  MipsCount qc;
  hipError_t e = hipMemcpy(&qi, a.qi + q, sizeof qi, hipMemcpyDeviceToHost);
  if (e == hipSuccess)
    e = hipMemcpy(&qc, a.qcnt + q, sizeof qc, hipMemcpyDeviceToHost);
  if (e == hipSuccess)
    e = launch_fill_u64((uint64_t*)count, 1, 0ull, st);
  if (e != hipSuccess) return e;
  // a table of slots; or the listed keys, x > 0 from the front of the
  // region and the rest from its back
  const uint64_t* hs = a.hslot + qi.hoff;
  const uint64_t* from[2] = {hs, hs + (qi.ccap - (int64_t)qc.rest)};
  const int64_t len[2] = {
      qi.bins ? (int64_t)qc.pos : qi.s > 0 ? (int64_t)qi.hmask + 1 : 0,
      qi.bins ? (int64_t)qc.rest : 0};
  for (int r = 0; r < 2; ++r) {
    if (len[r] <= 0) continue;
    int64_t blocks = (len[r] + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    k_mips_dump<<<(unsigned)blocks, 256, 0, st>>>(from[r], a.kb, len[r], keys,
                                                  xfix, cap, count);
  }
  return hipGetLastError();
}

}  // namespace mad
