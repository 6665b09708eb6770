// Block-wide radix select on fp32 bit patterns (positive floats: unsigned order = float order)
// and the fp64 re-evaluation of a token's score.  Shared by the dense and the candidate-list
// selection kernels; all functions are called by every thread of a 1024-thread workgroup.
#pragma once
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"

namespace sagekv {

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / kWave;

struct TopkShared {
  int hist[kHistBins];
  int wave_tot[kTopkWaves];
  int pick[2];  // bin, rank left inside it
};

// Logit scratch layout: [row][chunk][head][chunk tokens], so a score workgroup writes one
// contiguous block and the readers still take 16 bytes per head per thread.
__device__ __forceinline__ int64_t logit_index(const RowGeom& geo, int n_chunks, int chunk_tokens, int row, int g,
                                               int64_t tok) {
  const int shift = __builtin_ctz((unsigned)chunk_tokens);
  const int64_t chunk = tok >> shift;
  return ((((int64_t)row * n_chunks + chunk) * geo.G + g) << shift) + (tok - (chunk << shift));
}

// Exact softmax statistics of one head of a row from its per-chunk partials (max, sum exp(x - max)), `stride` floats apart:
// M = overall maximum of the fp32 logits, Z = sum_i exp(l_i - M) combined in fp64.  Called by all 64
// lanes of a wave; every lane gets the result.  PartialLoads: the first 128 chunks' partials, asked for early.
struct PartialLoads {
  float2 v[2];
};
__device__ __forceinline__ PartialLoads load_partials(const float* pr, int stride, int n_chunks) {
  const int lane = threadIdx.x & 63;
  PartialLoads l;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    l.v[u] = make_float2(-INFINITY, 0.f);
    if (lane + 64 * u < n_chunks) l.v[u] = *reinterpret_cast<const float2*>(pr + (int64_t)(lane + 64 * u) * stride);
  }
  return l;
}
__device__ __forceinline__ RowStat merge_partials_wave(const PartialLoads& l, const float* pr, int stride, int n_chunks) {
  const int lane = threadIdx.x & 63;
  float M = fmaxf(l.v[0].x, l.v[1].x);
  for (int i = lane + 128; i < n_chunks; i += 64) M = fmaxf(M, pr[(int64_t)i * stride]);
  M = wave_combine<true, 1>(M);
  double z = 0.0;
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (64 * u < n_chunks) z += l.v[u].y == 0.f ? 0.0 : (double)l.v[u].y * exp((double)l.v[u].x - (double)M);
#pragma unroll 1
  for (int i = lane + 128; i < n_chunks; i += 64) {
    const float2 v = *reinterpret_cast<const float2*>(pr + (int64_t)i * stride);
    z += (double)v.y * exp((double)v.x - (double)M);
  }
  z = group_sum_f64<64>(z);
  RowStat st;
  st.M = M;
  st.Z = z;
  st.invZ = (float)(1.0 / z);
  return st;
}

// The same from the partials of the one-sweep dense path.
__device__ inline RowStat merge_partials_wave(const ChunkPartial* pr, int n_chunks) {
  const int lane = threadIdx.x & 63;
  float M = -INFINITY;
  for (int i = lane; i < n_chunks; i += 64) M = fmaxf(M, pr[i].max);
  M = wave_combine<true, 1>(M);
  double z = 0.0;
#pragma unroll 1
  for (int i = lane; i < n_chunks; i += 64) z += pr[i].sum * exp((double)pr[i].max - (double)M);
  z = group_sum_f64<64>(z);
  RowStat st;
  st.M = M;
  st.Z = z;
  st.invZ = (float)(1.0 / z);
  return st;
}

// Largest digit b such that count(digits >= b) >= k_rem; returns b and the rank left inside it (0 and 1 if there are fewer
// than k_rem).  A barrier has to lie between an earlier block scan on wave_tot and this.
__device__ inline void pick_digit(const int* hist, int* wave_tot, int* pick /* [2] */, int nb, int k_rem, int* bin,
                                  int* rem) {
  const int t = threadIdx.x;
  const int i0 = nb - 1 - 2 * t, i1 = nb - 2 - 2 * t;  // descending digits
  const int c0 = i0 >= 0 ? hist[i0] : 0;
  const int c1 = i1 >= 0 ? hist[i1] : 0;
  int tot;
  const int incl = block_scan_incl(c0 + c1, wave_tot, &tot);
  const int before = incl - c0 - c1;
  if (before < k_rem && k_rem <= incl) {  // one thread, or none (everybody has read an earlier pick before the scan's barrier)
    const bool first = k_rem <= before + c0;
    pick[0] = first ? i0 : i1;
    pick[1] = k_rem - before - (first ? 0 : c0);
  }
  __syncthreads();
  const bool found = k_rem >= 1 && k_rem <= tot;
  *bin = found ? pick[0] : 0;
  *rem = found ? pick[1] : 1;
}
__device__ inline void pick_digit(TopkShared& sh, int nb, int k_rem, int* bin, int* rem) {
  pick_digit(sh.hist, sh.wave_tot, sh.pick, nb, k_rem, bin, rem);
}

__device__ inline void hist_pass(TopkShared& sh, const float* cand, int64_t E, uint32_t prefix, uint32_t mask, int shift,
                          int nbits) {
  for (int b = threadIdx.x; b < kHistBins; b += kTopkThreads) sh.hist[b] = 0;
  __syncthreads();
  const uint32_t dm = (1u << nbits) - 1u;
  for (int64_t i0 = threadIdx.x; i0 < E; i0 += 4 * kTopkThreads) {  // four independent loads in flight
    uint32_t key[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + (int64_t)u * kTopkThreads;
      key[u] = i < E ? __float_as_uint(cand[i]) : ~prefix;  // a key that never matches the prefix
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + (int64_t)u * kTopkThreads;
      if (i < E && (key[u] & mask) == prefix) atomicAdd(&sh.hist[(key[u] >> shift) & dm], 1);
    }
  }
  __syncthreads();
}

// k-th largest key among cand[0..E) and how many elements equal to it belong to the top k.
// first_hist_ready: sh.hist already holds the histogram of the first digit.
__device__ inline void radix_select(TopkShared& sh, const float* cand, int64_t E, int k, bool first_hist_ready,
                             uint32_t* tau, int* quota) {
  int bin, rem = k;
  if (!first_hist_ready) hist_pass(sh, cand, E, 0u, 0u, 20, 11);
  pick_digit(sh, 1 << 11, rem, &bin, &rem);
  uint32_t prefix = (uint32_t)bin << 20;
  hist_pass(sh, cand, E, prefix, 0xFFF00000u, 9, 11);
  pick_digit(sh, 1 << 11, rem, &bin, &rem);
  prefix |= (uint32_t)bin << 9;
  hist_pass(sh, cand, E, prefix, 0xFFFFFE00u, 0, 9);
  pick_digit(sh, 1 << 9, rem, &bin, &rem);
  *tau = prefix | (uint32_t)bin;
  *quota = rem;
}

// Ordered output of a selection kept as a bitmap in LDS (16-byte aligned): writes first + (index of
// the j-th set bit) to out[j] for j < k.  Every thread takes one, two or four consecutive words per round: a thread's
// words are gone through bit by bit, so a short bitmap is spread over all of them.
__device__ inline void bitmap_compact(const uint32_t* bitmap, int n_words, int first, int32_t* out, int k,
                                      int* wave_tot) {
  const int per = n_words <= kTopkThreads ? 1 : n_words <= 2 * kTopkThreads ? 2 : 4;
  int run = 0;
  for (int w0 = 0; w0 < n_words; w0 += per * kTopkThreads) {
    const int w = w0 + per * (int)threadIdx.x;
    uint32_t word[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) word[j] = j < per && w + j < n_words ? bitmap[w + j] : 0u;
    const int cnt = __popc(word[0]) + __popc(word[1]) + __popc(word[2]) + __popc(word[3]);
    int tot;
    if (w0 > 0) __syncthreads();  // wave_tot
    const int incl = block_scan_incl(cnt, wave_tot, &tot);
    int pos = run + incl - cnt;
    run += tot;
    int at = first + w * 32;
#pragma unroll 1
    for (int j = 0; j < per; ++j, at += 32) {
      uint32_t x = j == 0 ? word[0] : j == 1 ? word[1] : j == 2 ? word[2] : word[3];
      while (x) {
        const int b = __ffs(x) - 1;
        x &= x - 1;
        if (pos < k) out[pos] = (int32_t)(at + b);
        ++pos;
      }
    }
  }
}

template <int DT>
__device__ inline double elem_f64(const void* base, int64_t i);
template <>
__device__ inline double elem_f64<DT_BF16>(const void* base, int64_t i) {
  return (double)__uint_as_float((uint32_t)((const uint16_t*)base)[i] << 16);
}
template <>
__device__ inline double elem_f64<DT_F32>(const void* base, int64_t i) {
  return (double)((const float*)base)[i];
}

// Score of token `tok` of the row in fp64 (heads g_lo .. g_hi-1 of the group), rounded once to fp32.
// row_stats: the exact (M, Z) of the row's G heads (global or LDS).
template <int DT>
__device__ inline float refined_score(const RowGeom& geo, const void* q_last, const void* K, const PageMap& pm,
                                   int64_t ks_problem, int64_t ks_head, int64_t ks_token, const RowStat* row_stats,
                                   int prob, int c, int64_t tok, int g_lo, int g_hi) {
  const int D = geo.D, G = geo.G;
  const int64_t k_off = kv_offset(pm, pm.ks_page, ks_problem, ks_head, ks_token, prob, c, tok);
  const double inv = 1.0 / sqrt((double)D);
  double tot = 0.0;
  for (int g = g_lo; g < g_hi; ++g) {
    const int64_t q_off = ((int64_t)prob * geo.Hq + c * G + g) * D;
    double acc = 0.0;
    for (int j = 0; j < D; ++j) acc += elem_f64<DT>(q_last, q_off + j) * elem_f64<DT>(K, k_off + j);
    const RowStat st = row_stats[g];
    tot += exp(acc * inv - (double)st.M) / st.Z;
  }
  return (float)tot;
}

// One head's share of that value computed by one whole wave: lanes split head_dim, fp64 tree reduction (the fp64
// sum order differs from the sequential one by ~1e-16 relative, far below fp32 rounding).
template <int DT>
__device__ inline double refined_term_wave(const RowGeom& geo, const void* q_last, const void* K, const PageMap& pm,
                                           int64_t ks_problem, int64_t ks_head, int64_t ks_token, const RowStat& st,
                                           int prob, int c, int64_t tok, int g) {
  const int D = geo.D, lane = threadIdx.x & 63;
  const int64_t k_off = kv_offset(pm, pm.ks_page, ks_problem, ks_head, ks_token, prob, c, tok);
  const int64_t q_off = ((int64_t)prob * geo.Hq + c * geo.G + g) * D;
  double acc = 0.0;
  for (int j = lane; j < D; j += 64) acc += elem_f64<DT>(q_last, q_off + j) * elem_f64<DT>(K, k_off + j);
  acc = group_sum_f64<64>(acc);
  return exp(acc * (1.0 / sqrt((double)D)) - (double)st.M) / st.Z;
}
template <int DT>
__device__ inline float refined_score_wave(const RowGeom& geo, const void* q_last, const void* K, const PageMap& pm,
                                        int64_t ks_problem, int64_t ks_head, int64_t ks_token, const RowStat* row_stats,
                                        int prob, int c, int64_t tok, int g_lo, int g_hi) {
  double tot = 0.0;
  for (int g = g_lo; g < g_hi; ++g)
    tot += refined_term_wave<DT>(geo, q_last, K, pm, ks_problem, ks_head, ks_token, row_stats[g], prob, c, tok, g);
  return (float)tot;
}

// ---- normalisers of the one-sweep dense path ----------------------------------------------------
// The score pass knows nothing about a row before its sweep, so its chunk sums hold fp32 terms only.  Once a head's (M, Z) are
// merged, the terms heavy enough FOR THE ROW (heavy_logit_threshold: at most 1.4 M^2 of them) are exchanged for ones
// with an fp64 exponent: only chunks whose maximum reaches the threshold can hold one; their logits are looked through again
// in scratch.  (A rule on a term's share of its own chunk, applied in the score pass, calls every token of a flat chunk heavy
// once the logits share an offset: 256 rows x 8192 tokens, 4 heads, logits around -30: 718 us that way, 223 so.)
// A wave takes every sixteenth segment of 256 tokens of a head, one step further for the next head (neighbouring segments and
// a segment's heads tend to be heavy together).  Latency bound, two memory round trips (logits, then keys): a segment's
// logits are asked for one segment ahead, and a wave collects the heavy terms of its segments, up to a batch, before it
// takes them.  Few instructions on purpose, each thing in one place: the code runs once per row and is fetched cold.
constexpr int kExactTokens = 256;
constexpr int kExactBatch = 256;  // at least one segment's
constexpr int kExactMost = 2048;  // times the heads: heavy terms a wave takes exactly; beyond: as fp32 terms
struct ExactSums {
  double change[kTopkWaves][64];  // what a wave's terms change in Z of each head
  int tok[kTopkWaves][kExactBatch];
  unsigned char head[kTopkWaves][kExactBatch];
};

// A batch of a wave: 16 of its segments from seg0 on for each of the heads g0 .. g0 + 3, one (segment, head) per lane.
struct ExactItem {
  int g, seg;
};
__device__ __forceinline__ ExactItem exact_item(int g0, int seg0, int lane) {
  const int g = g0 + (lane & 3);
  return ExactItem{g, seg0 + kTopkWaves * (lane >> 2) + (((int)(threadIdx.x >> 6) - g) & (kTopkWaves - 1))};
}
// The maximum of the chunk that this lane's item lies in.
__device__ __forceinline__ float exact_maximum(const DenseRows& in, int row, int g0, int g_hi, int seg0) {
  const ExactItem it = exact_item(g0, seg0, threadIdx.x & 63);
  const int ch = it.seg >> __builtin_ctz((unsigned)in.chunk / kExactTokens);
  return it.g < g_hi && ch < in.n_chunks ? in.partials[((int64_t)row * in.geo.G + it.g) * in.n_chunks + ch].max : -INFINITY;
}

// Four elements of a row, and a product of such fours in fp64.
template <int DT>
struct FourElems {
  typedef uint2 type;
};
template <>
struct FourElems<DT_F32> {
  typedef uint4 type;
};
template <int DT>
__device__ __forceinline__ typename FourElems<DT>::type four_elems(const void* base, int64_t i) {
  return *reinterpret_cast<const typename FourElems<DT>::type*>((const char*)base + i * Elem<DT>::bytes);
}
template <int DT>
__device__ __forceinline__ double dot_f64(const typename FourElems<DT>::type& a, const typename FourElems<DT>::type& b, double acc) {
  if constexpr (DT == DT_BF16) {
    acc += (double)bf16_lo(a.x) * (double)bf16_lo(b.x) + (double)bf16_hi(a.x) * (double)bf16_hi(b.x);
    return acc + ((double)bf16_lo(a.y) * (double)bf16_lo(b.y) + (double)bf16_hi(a.y) * (double)bf16_hi(b.y));
  } else {
    acc += (double)__uint_as_float(a.x) * (double)__uint_as_float(b.x) + (double)__uint_as_float(a.y) * (double)__uint_as_float(b.y);
    return acc + ((double)__uint_as_float(a.z) * (double)__uint_as_float(b.z) + (double)__uint_as_float(a.w) * (double)__uint_as_float(b.w));
  }
}

// A wave's first cnt listed terms: exp(l - M) - (the fp32 term in the merged sum), l = the logit in fp64, added to its changes.
// Sixteen lanes share a term, four elements at a time, two terms in flight (fp32: one, registers).  Called by all 64 lanes
// of a wave.
template <int DT>
__device__ __forceinline__ void exact_terms_wave(const DenseRows& in, ExactSums& sh, int cnt, int row, const RowStat* stat) {
  typedef typename FourElems<DT>::type Four;
  constexpr int U = DT == DT_BF16 ? 2 : 1;
  const int D = in.geo.D, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, sub = lane & 15;
  const int prob = row / in.geo.Hkv, c = row % in.geo.Hkv, chunk_shift = __builtin_ctz((unsigned)in.chunk);
  const double inv = 1.0 / sqrt((double)D);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
  for (int e0 = 0; e0 < cnt; e0 += 4 * U) {
    Four k0[U], k1[U], q0[U], q1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + 4 * u + grp < cnt ? e0 + 4 * u + grp : cnt - 1;
      const int64_t ko = kv_offset(in.pm, in.pm.ks_page, in.ks_problem, in.ks_head, in.ks_token, prob, c, sh.tok[wave][e]) + 4 * sub;
      const int64_t qo = ((int64_t)prob * in.geo.Hq + c * in.geo.G + sh.head[wave][e]) * D + 4 * sub;
      k0[u] = four_elems<DT>(in.K, ko);
      q0[u] = four_elems<DT>(in.q_last, qo);
      k1[u] = D > 64 ? four_elems<DT>(in.K, ko + 64) : Four{};
      q1[u] = D > 64 ? four_elems<DT>(in.q_last, qo + 64) : Four{};
    }
    // lanes 0 and 1 of a group: the terms' fp64 exponentials, lanes 2 and 3: their fp32 ones as they were merged
    const int e = e0 + 4 * (sub & 1) + grp;
    const bool mine = sub < 4 && (sub & 1) < U && e < cnt;
    const int g = sh.head[wave][e < cnt ? e : cnt - 1];
    const float M = stat[g].M;
    float x = 0.f, mc = M;
    if (mine && sub >= 2) {
      x = in.logits[logit_index(in.geo, in.n_chunks, in.chunk, row, g, sh.tok[wave][e])];
      mc = in.partials[((int64_t)row * in.geo.G + g) * in.n_chunks + (sh.tok[wave][e] >> chunk_shift)].max;
    }
    double l = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double a = group_sum_f64<16>(dot_f64<DT>(k1[u], q1[u], dot_f64<DT>(k0[u], q0[u], 0.0)));
      l = sub == u ? a * inv : l;
    }
    const double ex = exp((sub >= 2 ? (double)mc : l) - (double)M);
    if (mine) unsafeAtomicAdd(&sh.change[wave][g], sub >= 2 ? -(double)exp_fast(x - mc) * ex : ex);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// What the heavy terms change in Z of heads g_lo .. g_hi of a row (stat, thr: their merged statistics and
// heavy_logit_threshold of them, in LDS; max: exact_maximum of the first batch, asked for early).  Called by every thread of a
// 1024-thread workgroup; begins with a barrier.  before(): called by all of them where there are heavy terms.  True (workgroup-uniform):
// exact_apply has to follow.
template <int DT, class Before>
__device__ __forceinline__ bool exact_changes(const DenseRows& in, ExactSums& sh, int row, int g_lo, int g_hi, const RowStat* stat,
                                              const float* thr, float max, Before before) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  bool any = false;
  for (int g = g_lo; g < g_hi; ++g) any |= thr[g] <= stat[g].M;
  if (!any) return false;  // no term of any head is heavy
  before();
  sh.change[wave][lane] = 0.0;
  const int n_seg = in.n_chunks * (in.chunk / kExactTokens);
  int taken = 0, listed = 0;  // wave-uniform
  bool end = false;
  for (int g0 = g_lo, seg0 = 0; !end;) {  // the last round only takes what is listed
    unsigned long long todo = 0ull;
    end = seg0 >= n_seg;
    if (!end) {
      const int g = g0 + (lane & 3);
      if (g0 > g_lo || seg0 > 0) max = exact_maximum(in, row, g0, g_hi, seg0);
      todo = __ballot(g < g_hi && max >= thr[g < g_hi ? g : g_lo]);
    }
    auto logits_of = [&](const ExactItem& it) -> float4 {
      const int64_t tok = (int64_t)it.seg * kExactTokens + 4 * lane;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (tok < in.geo.L)
        v = *reinterpret_cast<const float4*>(in.logits + logit_index(in.geo, in.n_chunks, in.chunk, row, it.g, tok));
      return v;
    };
    ExactItem it = {g_lo, 0}, it_next = it;
    float4 next = make_float4(0.f, 0.f, 0.f, 0.f);
    if (todo) {
      it_next = exact_item(g0, seg0, __ffsll(todo) - 1);
      next = logits_of(it_next);
    }
    do {
      unsigned long long heavy[4] = {0ull, 0ull, 0ull, 0ull};
      int total = 0;
      if (todo) {
        const float x[4] = {next.x, next.y, next.z, next.w};
        it = it_next;
        todo &= todo - 1;
        if (todo) {
          it_next = exact_item(g0, seg0, __ffsll(todo) - 1);
          next = logits_of(it_next);
        }
        const float th = thr[it.g];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          heavy[e] = __ballot((int64_t)it.seg * kExactTokens + 4 * lane + e < in.geo.L && x[e] >= th);
          total += __popcll(heavy[e]);
        }
        if (taken + total > kExactMost * (g_hi - g_lo)) continue;
        taken += total;
      }
      if (listed > 0 && (end || listed + total > kExactBatch)) {
        exact_terms_wave<DT>(in, sh, listed, row, stat);
        listed = 0;
      }
      if (total > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int w = listed + __popcll(heavy[e] & ((1ull << lane) - 1ull));
          if ((heavy[e] >> lane) & 1ull) {
            sh.tok[wave][w] = it.seg * kExactTokens + 4 * lane + e;
            sh.head[wave][w] = (unsigned char)it.g;
          }
          listed += __popcll(heavy[e]);
        }
      }
    } while (todo);
    g0 += 4;
    if (g0 >= g_hi) g0 = g_lo, seg0 += 16 * kTopkWaves;
  }
  return true;
}
// Adds the changes to the statistics; begins and ends with a barrier.
__device__ __forceinline__ void exact_apply(const ExactSums& sh, int g_lo, int g_hi, RowStat* stat) {
  const int tid = threadIdx.x;
  __syncthreads();
  if (tid >= g_lo && tid < g_hi) {
    double z = stat[tid].Z;
#pragma unroll
    for (int w = 0; w < kTopkWaves; ++w) z += sh.change[w][tid];
    stat[tid].Z = z;
    stat[tid].invZ = (float)(1.0 / z);
  }
  __syncthreads();
}

// f(head, token, logit), logits in fours from a token on (-inf: past the row's end), for the heads g_lo .. g_hi - 1 with which(head), which has to be
// the same for all threads.
template <class Which, class F>
__device__ __forceinline__ void each_four(const DenseRows& in, int row, int g_lo, int g_hi, Which which, F f) {
  constexpr int U = 4;  // loads in flight
  const int quads = (int)((in.geo.L + 3) >> 2);
#pragma unroll 1
  for (int g = g_lo, q = threadIdx.x; g < g_hi;) {
    float4 x[U];
    int gu[U], tok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      while (g < g_hi && !which(g)) ++g;  // workgroup-uniform (q at its start)
      gu[u] = g;
      tok[u] = 4 * q;
      x[u] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (g < g_hi && q < quads) x[u] = *reinterpret_cast<const float4*>(in.logits + logit_index(in.geo, in.n_chunks, in.chunk, row, g, tok[u]));
      q += kTopkThreads;
      if (q - (int)threadIdx.x >= quads) q = threadIdx.x, ++g;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (gu[u] >= g_hi) continue;  // workgroup-uniform
      float l[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) l[e] = tok[u] + e < in.geo.L ? l[e] : -INFINITY;
      f(gu[u], tok[u], l);
    }
  }
}

// Higher thresholds (thr) for the heads that have more heavy terms than are worth taking.  heavy_logit_threshold is the safe choice where a few terms
// hold most of a head's mass.  Hundreds of terms over it are all small ones (logits that share an offset, where every tenth token reaches
// it), and their errors average out: what is left out may be as much as keeps sqrt(sum w_i^2) over ALL terms left out within sqrt(theta), the same
// bound on Z's error.  That sum comes from the numbers of logits in steps of 1/8 below the maximum, each taken at its step's middle (the last, open one
// at its upper edge), so it does not depend on any order.  bins: 64 per head.  Called by every thread of a 1024-thread workgroup; begins and ends with a barrier.
// A term costs one CU some 10 ns.  8 rows x 8192 tokens x 4 heads of N(60, 1) have 6600 terms each over the thresholds and 820 over the raised ones,
// and Z's error goes from 0.5e-7 to 1e-7; whole passes 141 and 50.5 us (24.4 at N(0, 1)), 64 rows x 8192 x 16 heads 532 and 181 (77), 64 x 2048 x 4
// 148 and 57 (25), fp32 8 x 8192 x 4 210 and 63 (29).
template <class Which>
__device__ __forceinline__ void raise_thresholds(const DenseRows& in, int* bins, int row, int g_lo, int g_hi, const RowStat* stat, float* thr, Which which) {
  const int tid = threadIdx.x, lane = tid & 63;
  __syncthreads();
  for (int b = tid; b < 64 * (g_hi - g_lo); b += kTopkThreads) bins[b] = 0;
  __syncthreads();
  each_four(in, row, g_lo, g_hi, which, [&](int g, int, const float (&l)[4]) {
    const float M = stat[g].M;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float step = 8.f * (M - l[e]);
      if (step < 63.f) atomicAdd(&bins[64 * (g - g_lo) + (int)fmaxf(step, 0.f)], 1);  // (the rest, often nearly all, would meet in one place)
    }
  });
  __syncthreads();
  for (int g = g_lo + (tid >> 6); g < g_hi; g += kTopkWaves) {  // a wave per head
    if (!which(g)) continue;
    const float M = stat[g].M, t = thr[g];
    const int in_step = lane < 63 ? bins[64 * (g - g_lo) + lane] : 0;
    const float above = group_sum<64>((float)in_step);
    if (group_sum<64>((float)lane <= 8.f * (M - t) ? (float)in_step : 0.f) <= 64.f) continue;  // few terms: all of them are taken
    // sum w_i^2 of a step, then of those below it too, times Z^2
    float left = lane < 63 ? (float)in_step * exp_fast(-0.25f * ((float)lane + 0.5f)) : ((float)in.geo.L - above) * exp_fast(-0.25f * 63.f);
#pragma unroll
    for (int o = 1; o < 64; o *= 2) {
      const float more = __shfl_down(left, o);
      left += lane + o < 64 ? more : 0.f;
    }
    const unsigned long long enough = __ballot(left <= (float)stat[g].Z * exp_fast(t - M));  // theta Z^2
    if (enough && lane == 0) thr[g] = fmaxf(t, M - 0.125f * (float)(__ffsll(enough) - 1));
  }
  __syncthreads();
}

// ---- selection among scores held in registers ---------------------------------------------------
// N scores per thread of a 1024-thread workgroup, -1: no element.  All functions are called by every thread.
constexpr int kMaxBand = 1024;  // elements around the k-th that are ranked exactly among themselves

struct RegSelect {
  union {
    int hist[2][kHistBins];
    double term[kMaxBand];  // refine_band: fp64 terms of a batch of (member, head)
  };
  int wave_tot[kTopkWaves], pick[2];
  int red[2][kTopkWaves];  // ~smallest, largest key of each wave
  int band_tok[kMaxBand];
  float band_v[kMaxBand];
  int n_band, n_above;
};

// Bracket of the k-th largest score: its bit pattern lies in [*tlo, *thi], at most 2^9 apart (2^-14 relative).
// Two histograms over the keys' own range: 2048 bins from the smallest to the largest key, then 2048 bins
// inside the bin that holds the k-th.  (Digits of the bit pattern would put most of a row into a few bins: the
// LDS atomics of a wave then serialise on one address.)  Also clears n_band and n_above.
// each(f) calls f(score) for the thread's scores, any number of times, in any order, with -1 where there is none.
// TWO false: the first histogram only, *tlo = the lower edge of the k-th score's bin (a lower bound of it).
template <bool TWO, class Each>
__device__ __forceinline__ void bracket_kth(RegSelect& sh, Each each, int k, uint32_t* tlo, uint32_t* thi) {
  const int tid = threadIdx.x, wave = tid >> 6;
  int4* h4 = reinterpret_cast<int4*>(&sh.hist[0][0]);
  for (int b = tid; b < (TWO ? 2 : 1) * kHistBins / 4; b += kTopkThreads) h4[b] = make_int4(0, 0, 0, 0);
  int mn = 0x7FFFFFFF, mx = -1;
  each([&](float v) {
    const int key = __float_as_int(v);
    if (key >= 0) mn = key < mn ? key : mn;
    mx = key > mx ? key : mx;
  });
  const int wmn = wave_max_i(~mn), wmx = wave_max_i(mx);
  if ((tid & 63) == 0) {
    sh.red[0][wave] = wmn;
    sh.red[1][wave] = wmx;
  }
  if (tid == 0) sh.n_band = sh.n_above = 0;
  __syncthreads();
  int e = sh.red[(tid >> 4) & 1][tid & 15];  // rows 0, 2 of the wave: ~smallest, rows 1, 3: largest
  e = max(e, dpp_rot_i32<0x128>(e));         // row_ror
  e = max(e, dpp_rot_i32<0x124>(e));
  e = max(e, dpp_rot_i32<0x122>(e));
  e = max(e, dpp_rot_i32<0x121>(e));
  mn = ~__builtin_amdgcn_readlane(e, 0);
  mx = __builtin_amdgcn_readlane(e, 16);
  const uint32_t range = mx >= mn ? (uint32_t)(mx - mn) : 0u;
  const int s1 = range < (uint32_t)kHistBins ? 0 : 21 - __clz((int)range);  // range >> s1 < 2048
  each([&](float v) {
    const int key = __float_as_int(v);
    if (key >= 0) atomicAdd(&sh.hist[0][(uint32_t)(key - mn) >> s1], 1);
  });
  __syncthreads();
  int bin, rem;
  pick_digit(sh.hist[0], sh.wave_tot, sh.pick, kHistBins, k, &bin, &rem);
  const int base = mn + (int)((uint32_t)bin << s1);
  if (!TWO || s1 == 0) {
    *tlo = (uint32_t)base;
    *thi = (uint32_t)base + ((1u << s1) - 1u);
    return;
  }
  const int s2 = s1 > 11 ? s1 - 11 : 0;
  each([&](float v) {
    const int key = __float_as_int(v);
    if (key >= 0 && (int)((uint32_t)(key - mn) >> s1) == bin) atomicAdd(&sh.hist[1][(uint32_t)(key - base) >> s2], 1);
  });
  __syncthreads();
  pick_digit(sh.hist[1], sh.wave_tot, sh.pick, kHistBins, rem, &bin, &rem);
  *tlo = (uint32_t)base + ((uint32_t)bin << s2);
  *thi = *tlo + ((1u << s2) - 1u);
}

// fp64 scores of the band's members (band_tok) into band_v: 16 lanes take a (member, head) term, the terms are added
// in head order.  Ends with a barrier.
template <int DT>
__device__ __forceinline__ void refine_band(RegSelect& sh, int nb, const RowGeom& geo, const void* q_last, const void* K,
                                            const PageMap& pm, int64_t ks_problem, int64_t ks_head, int64_t ks_token,
                                            const RowStat* stats, int prob, int c, int g_lo, int g_hi) {
  typedef typename FourElems<DT>::type Four;
  const int D = geo.D, tid = threadIdx.x, sub = tid & 15, heads = g_hi - g_lo, per = kMaxBand / heads;
  const double inv = 1.0 / sqrt((double)D);
  for (int m0 = 0; m0 < nb; m0 += per) {
    const int cnt = nb - m0 < per ? nb - m0 : per;
#pragma unroll 1
    for (int t = tid >> 4; t < cnt * heads; t += kTopkThreads / 16) {
      const int g = g_lo + t % heads;
      const int64_t ko = kv_offset(pm, pm.ks_page, ks_problem, ks_head, ks_token, prob, c, sh.band_tok[m0 + t / heads]) + 4 * sub;
      const int64_t qo = ((int64_t)prob * geo.Hq + c * geo.G + g) * D + 4 * sub;
      const Four k0 = four_elems<DT>(K, ko), q0 = four_elems<DT>(q_last, qo);
      Four k1 = {}, q1 = {};
      if (D > 64) k1 = four_elems<DT>(K, ko + 64), q1 = four_elems<DT>(q_last, qo + 64);
      const double l = group_sum_f64<16>(dot_f64<DT>(k1, q1, dot_f64<DT>(k0, q0, 0.0))) * inv;
      if (sub == 0) sh.term[t] = exp(l - (double)stats[g].M) / stats[g].Z;
    }
    __syncthreads();
    for (int t = tid; t < cnt; t += kTopkThreads) {
      double tot = 0.0;
      for (int g = 0; g < heads; ++g) tot += sh.term[t * heads + g];
      sh.band_v[m0 + t] = (float)tot;
    }
    __syncthreads();
  }
}

// The heavy terms of a row whose logits pass through registers, listed there as they are met (a few dozen at most, as a rule), and taken
// together with the band: exact_changes and refine_band in one round trip to the keys, where the lists hold what there is.  One after the
// other they took 8 of a row's 20 us (256 rows x 8192 tokens, k = 1788, four sink tokens); a whole pass 207 -> 204, over 8 rows 29.7 -> 27.6,
// 128 rows x 8192 x 7 heads 128 -> 122.6.
constexpr int kHeavyList = 512;
constexpr int kHeavyMost = 4096;  // with raised thresholds, see raise_thresholds
struct HeavyList {  // in the order in which the waves met them
  int n;
  int tok[kHeavyMost];
  float logit[kHeavyMost];
  double exact[kHeavyMost];  // the logit in fp64
  unsigned char head[kHeavyMost];
  // What a head's terms change in its Z (exact term - the one in the merged sum) in units of 2^-46 of the largest term: a sum of integers does not
  // depend on the waves' order.  (Sums in the order of head and token, from every term's place among the keys: 64 rows x 8192 x 16 heads,
  // queries x 6, 500 terms a row, 97.5 us for the pass, so 87.)
  unsigned long long change[64];
};

// fp64 scores of the band's members into band_v after the listed terms have gone into the statistics (stat, in LDS).  Every 16 lanes
// take one logit.  nb * heads <= kMaxBand, hv.n <= kHeavyMost, hv.change = 0.  Begins (hv.n, band_tok) after a barrier, ends with one.
template <int DT>
__device__ __forceinline__ void refine_band_exact(RegSelect& sh, HeavyList& hv, int nb, const DenseRows& in, int row, int g_lo, int g_hi, RowStat* stat) {
  typedef typename FourElems<DT>::type Four;
  const RowGeom& geo = in.geo;
  const int D = geo.D, tid = threadIdx.x, sub = tid & 15, heads = g_hi - g_lo, n_heavy = hv.n, n = n_heavy + nb * heads;
  const int prob = row / geo.Hkv, c = row % geo.Hkv, chunk_shift = __builtin_ctz((unsigned)in.chunk);
  const double inv = 1.0 / sqrt((double)D);
  constexpr int U = DT == DT_BF16 ? 2 : 1, kGroups = kTopkThreads / 16;
#pragma unroll 1
  for (int t0 = tid >> 4; t0 < n; t0 += U * kGroups) {
    Four k0[U], k1[U], q0[U], q1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && n <= kGroups) continue;  // workgroup-uniform: a term a group at most
      const int t = t0 + u * kGroups < n ? t0 + u * kGroups : t0;
      const bool heavy = t < n_heavy;
      const int b = heavy ? 0 : t - n_heavy;
      const int tok = heavy ? hv.tok[t] : sh.band_tok[b / heads], g = heavy ? hv.head[t] : g_lo + b % heads;
      const int64_t ko = kv_offset(in.pm, in.pm.ks_page, in.ks_problem, in.ks_head, in.ks_token, prob, c, tok) + 4 * sub;
      const int64_t qo = ((int64_t)prob * geo.Hq + c * geo.G + g) * D + 4 * sub;
      k0[u] = four_elems<DT>(in.K, ko);
      q0[u] = four_elems<DT>(in.q_last, qo);
      k1[u] = D > 64 ? four_elems<DT>(in.K, ko + 64) : Four{};
      q1[u] = D > 64 ? four_elems<DT>(in.q_last, qo + 64) : Four{};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && n <= kGroups) continue;
      const int t = t0 + u * kGroups;
      const double l = group_sum_f64<16>(dot_f64<DT>(k1[u], q1[u], dot_f64<DT>(k0[u], q0[u], 0.0))) * inv;
      if (sub == 0 && t < n) *(t < n_heavy ? &hv.exact[t] : &sh.term[t - n_heavy]) = l;
    }
  }
  __syncthreads();
  if (n_heavy > 0) {  // a term per thread: sixteen lanes waiting for one's exponentials took longer than the dot products
    for (int t = tid; t < n_heavy; t += kTopkThreads) {
      const int g = hv.head[t];
      const float mc = in.partials[((int64_t)row * geo.G + g) * in.n_chunks + (hv.tok[t] >> chunk_shift)].max;
      const double M = (double)stat[g].M;
      const double x = exp(hv.exact[t] - M) - (double)exp_fast(hv.logit[t] - mc) * exp((double)mc - M);
      atomicAdd(&hv.change[g], (unsigned long long)__double2ll_rn(x * 0x1p46));
    }
    __syncthreads();
    if (tid >= g_lo && tid < g_hi) {
      const double z = stat[tid].Z + (double)(long long)hv.change[tid] * 0x1p-46;
      stat[tid].Z = z;
      stat[tid].invZ = (float)(1.0 / z);
    }
    __syncthreads();
  }
  for (int b = tid; b < nb * heads; b += kTopkThreads) {
    const RowStat& st = stat[g_lo + b % heads];
    sh.term[b] = exp(sh.term[b] - (double)st.M) / st.Z;
  }
  __syncthreads();
  for (int t = tid; t < nb; t += kTopkThreads) {
    double tot = 0.0;
    for (int g = 0; g < heads; ++g) tot += sh.term[t * heads + g];
    sh.band_v[t] = (float)tot;
  }
  __syncthreads();
}

}  // namespace sagekv
