// Eviction pass, selection stage (paper Sec. 2 Step 2 "top-k", Step 3 "Concat"):
// per row, the k candidates with the largest score, ties to the lower index, written in
// ascending position between the sink and the recent window; then the gather of K and V.
//
// row_select_kernel: one-sweep dense path, rows whose scores one workgroup holds in registers.
//
// topk_kernel: one 1024-thread workgroup per row; two passes over the row's scores (steps 1 and
// 2) on the usual route, all with aligned 16-byte loads.
//   1. coarse bracket of the k-th score: the first two digits (11 + 11 bits) of a radix select on
//      the fp32 bit patterns of the scores (all positive, so the unsigned order is the float
//      order).  The first digit's histogram was built by many workgroups in the combine stage; the
//      second is an LDS histogram over the row.  The k-th score is then known to 2^-13 relative.
//   2. one scan counts the scores above a relative band around that bracket and lists the band's
//      members; those are re-evaluated in fp64 (dot products, exp, fp64-combined normalisers),
//      patched into the score row and ranked exactly among themselves (score descending, index
//      ascending), so the decision near the threshold does not depend on fp32 summation order.
//      The exact threshold is the (k - #above)-th of them.
//   3. only if the band holds more than kDenseBand members (a row of near-ties) or the refined
//      threshold sits on the band's edge: patch the band, exact radix select of the whole row.
//   4. ordered output.  Usual route: the band scan has marked every score above the band in an LDS
//      bitmap (one bit per candidate, rows of up to 512K candidates), the selected band members
//      are added, and a prefix sum over the bitmap's population counts gives the positions: the
//      row is read twice in all.  General route or longer rows: every wave counts and then writes
//      a contiguous part of the row.  Both keep the output ascending and give ties to the lowest
//      indices.
#include "device_utils.h"
#include "kernels.h"
#include "radix_select.h"

namespace sagekv {

namespace {

constexpr int kDenseBand = 1024;  // band members whose exact ranking is done among themselves

// A row of fp32 scores read with aligned 16-byte loads.  "Quad" q holds row elements 4q - head ..
// 4q - head + 3; quads q_lo .. q_hi-1 lie fully inside the row and are read with one vector load
// each, several in flight per thread.  The at most six elements before and after them are the
// row's edge elements: first edge = elements 0 .. n_first-1, last edge = elements last0 .. E-1.
// One workgroup (one CU) owns a row, so the passes below are bound by instruction issue as much
// as by the CU's load path: per element they spend two to four vector instructions, counts go
// through wave ballots into scalar registers.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4* GlobalQuads;  // global memory: 16-byte vector loads

struct QuadRow {
  const float* cand;
  GlobalQuads quads;  // quads[q] for q_lo <= q < q_hi
  int head;           // floats between the 16-byte boundary below cand and cand
  int q_lo, q_hi;
  int n_first, last0, E;
};

__device__ inline QuadRow quad_row(const float* cand, int E) {
  QuadRow r;
  r.cand = cand;
  r.head = (int)((reinterpret_cast<uintptr_t>(cand) >> 2) & 3);
  r.quads = (GlobalQuads)(cand - r.head);
  r.q_lo = r.head ? 1 : 0;
  r.q_hi = (r.head + E) >> 2;
  if (r.q_hi < r.q_lo) r.q_hi = r.q_lo;
  r.n_first = 4 * r.q_lo - r.head < E ? 4 * r.q_lo - r.head : E;
  r.last0 = 4 * r.q_hi - r.head > r.n_first ? 4 * r.q_hi - r.head : r.n_first;
  r.E = E;
  return r;
}

// Row index of the edge element that thread `t` (0..7) looks after, or -1: threads 0..3 the first
// edge, 4..7 the last one.
__device__ inline int edge_index(const QuadRow& r, int t) {
  if (t < 4) return t < r.n_first ? t : -1;
  return r.last0 + (t - 4) < r.E ? r.last0 + (t - 4) : -1;
}

constexpr int kQuadUnroll = 8;  // quads in flight per thread: 32 scores

// LDS histogram of digit (key >> shift) & (2^nbits - 1) over the keys that match `prefix` under `mask`.
__device__ inline void hist_pass_quads(TopkShared& sh, const QuadRow& r, uint32_t prefix, uint32_t mask, int shift,
                                       int nbits) {
  for (int b = threadIdx.x; b < kHistBins; b += kTopkThreads) sh.hist[b] = 0;
  __syncthreads();
  const uint32_t dm = (1u << nbits) - 1u;
  const int ei = threadIdx.x < 8 ? edge_index(r, threadIdx.x) : -1;
  uint32_t ekey = ~prefix;
  if (ei >= 0) ekey = __float_as_uint(r.cand[ei]);
  for (int q0 = r.q_lo + threadIdx.x; q0 < r.q_hi; q0 += kQuadUnroll * kTopkThreads) {
    u32x4 v[kQuadUnroll];
#pragma unroll
    for (int u = 0; u < kQuadUnroll; ++u) {
      const int q = q0 + u * kTopkThreads;
      v[u] = r.quads[q < r.q_hi ? q : r.q_hi - 1];
    }
#pragma unroll
    for (int u = 0; u < kQuadUnroll; ++u) {
      const bool valid = q0 + u * kTopkThreads < r.q_hi;
      const uint32_t key[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (valid && (key[e] & mask) == prefix) atomicAdd(&sh.hist[(key[e] >> shift) & dm], 1);
    }
  }
  if (ei >= 0 && (ekey & mask) == prefix) atomicAdd(&sh.hist[(ekey >> shift) & dm], 1);
  __syncthreads();
}

__device__ inline int lanes_below(unsigned long long ballot) {  // set bits of `ballot` in lanes below this one
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

// One selection list (one per row, group-sum, or one per (row, query head)) from its score row.  p.ghist: the first digit's
// histogram is there; null: it is taken here.
template <int DT>
__device__ __forceinline__ void topk_list(const TopkParams& p, uint32_t* bitmap /* bit i + head: candidate i is selected (head: see QuadRow) */,
                                          int list) {
  __shared__ TopkShared sh;
  const int tid = threadIdx.x;
  const int row = list / p.n_lists, gl = list % p.n_lists;
  const int g_lo = p.n_lists > 1 ? gl : 0, g_hi = p.n_lists > 1 ? gl + 1 : p.geo.G;
  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int S = p.S, W = p.W, k = p.k;
  const int64_t L = p.geo.L;
  const int E = (int)(L - S - W);
  const int n_kept = S + p.n_lists * k + W;
  int32_t* kept_row = p.kept_idx + (int64_t)row * n_kept;
  int32_t* kept = kept_row + gl * k;  // this list's k slots start at kept[S]
  float* cand = p.scores + (int64_t)list * p.pitch + S;
  const RowStat* row_stats = p.stats + (int64_t)row * p.geo.G;

  if (gl == 0) {
    for (int t = tid; t < S; t += kTopkThreads) kept_row[t] = t;
    for (int t = tid; t < W; t += kTopkThreads) kept_row[S + p.n_lists * k + t] = (int32_t)(L - W + t);
  }
  if (k == 0) return;
  const QuadRow qr = quad_row(cand, E);
  const int edge_i = tid < 8 ? edge_index(qr, tid) : -1;  // this thread's edge element, if any

  // 1. bracket of the k-th fp32 score: its first 22 bits
  if (p.ghist) {
    for (int b = tid; b < kHistBins; b += kTopkThreads) sh.hist[b] = p.ghist[(int64_t)list * kHistBins + b];
    __syncthreads();
  } else {
    hist_pass_quads(sh, qr, 0u, 0u, 20, 11);
  }
  uint32_t tau;
  int quota;
  {
    int bin, rem;
    pick_digit(sh, 1 << 11, k, &bin, &rem);
    tau = (uint32_t)bin << 20;
    hist_pass_quads(sh, qr, tau, 0xFFF00000u, 9, 11);
    pick_digit(sh, 1 << 11, rem, &bin, &rem);
    tau |= (uint32_t)bin << 9;
    quota = rem;
  }

  // 2. the band around it.  Scores above the band are selected whatever their exact value; the
  //    members of the band are re-evaluated in fp64 (and patched into the score row).  With a band
  //    of at most kDenseBand members the exact threshold is found among them alone: it is the
  //    (k - #above)-th largest refined value, provided it still lies strictly inside the band
  //    (then no score outside the band can compare differently).  Anything else (a huge band of
  //    near-ties, a refined value on the band's edge) takes the general route: patch, then a full
  //    radix select of the patched row.
  // (below 2^-126 the scores sit on the 2^-149 grid: the band is at least kDenormSlack wide each way)
  const float lo = __uint_as_float(tau) * (1.0f - p.band) - kDenormSlack,
              hi = __uint_as_float(tau | 0x1FFu) * (1.0f + p.band) + kDenormSlack;
  __shared__ int band_i[kDenseBand];
  __shared__ float band_v[kDenseBand];
  __shared__ int n_band, n_above, short_ok;
  __shared__ uint32_t short_tau;
  __shared__ int short_quota;
  const int n_words = (qr.head + E + 31) >> 5;
  const bool use_bitmap = n_words * 4 <= p.bitmap_bytes;
  if (tid == 0) n_band = n_above = short_ok = 0;
  if (use_bitmap)
    for (int w = tid; w < n_words; w += kTopkThreads) bitmap[w] = 0u;
  __syncthreads();
  {
    auto member = [&](int i) {
      const int t = atomicAdd(&n_band, 1);
      if (t < kDenseBand) band_i[t] = i;
    };
    float ev = -1.f;
    if (edge_i >= 0) ev = cand[edge_i];
    int above = 0;  // wave-uniform: counted through ballots
    for (int q0 = qr.q_lo + (tid & ~63); q0 < qr.q_hi; q0 += kQuadUnroll * kTopkThreads) {  // wave-uniform trip count
      u32x4 v[kQuadUnroll];
#pragma unroll
      for (int u = 0; u < kQuadUnroll; ++u) {
        const int q = q0 + (tid & 63) + u * kTopkThreads;
        v[u] = qr.quads[q < qr.q_hi ? q : qr.q_hi - 1];
      }
#pragma unroll
      for (int u = 0; u < kQuadUnroll; ++u) {
        const int q = q0 + (tid & 63) + u * kTopkThreads;
        const bool valid = q < qr.q_hi;
        const float x[4] = {__uint_as_float(v[u].x), __uint_as_float(v[u].y), __uint_as_float(v[u].z),
                            __uint_as_float(v[u].w)};
        uint32_t nib = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool gt = valid && x[e] > hi;
          above += __popcll(__ballot(gt));
          nib |= gt ? 1u << e : 0u;
          if (valid && !gt && x[e] >= lo) member(4 * q - qr.head + e);
        }
        if (use_bitmap && nib) atomicOr(&bitmap[q >> 3], nib << (4 * (q & 7)));
      }
    }
    if ((tid & 63) == 0 && above) atomicAdd(&n_above, above);
    if (edge_i >= 0) {
      if (ev > hi) {
        atomicAdd(&n_above, 1);
        if (use_bitmap) atomicOr(&bitmap[(edge_i + qr.head) >> 5], 1u << ((edge_i + qr.head) & 31));
      } else if (ev >= lo) {
        member(edge_i);
      }
    }
  }
  __syncthreads();
  const int nb = n_band, r = k - n_above;
  bool general = nb > kDenseBand || r < 1 || r > nb;
  if (!general) {
    if (nb <= 4 * kTopkWaves) {  // the usual handful: one wave per member
      for (int t = tid >> 6; t < nb; t += kTopkWaves) {
        const int i = band_i[t];
        const float v = refined_score_wave<DT>(p.geo, p.q_last, p.K, p.pm, p.ks_problem, p.ks_head, p.ks_token, row_stats,
                                               prob, c, S + i, g_lo, g_hi);
        if ((tid & 63) == 0) {
          band_v[t] = v;
          cand[i] = v;
        }
      }
    } else {
      for (int t = tid; t < nb; t += kTopkThreads) {
        const int i = band_i[t];
        const float v = refined_score<DT>(p.geo, p.q_last, p.K, p.pm, p.ks_problem, p.ks_head, p.ks_token, row_stats, prob, c,
                                          S + i, g_lo, g_hi);
        band_v[t] = v;
        cand[i] = v;
      }
    }
    __syncthreads();
    for (int t = tid; t < nb; t += kTopkThreads) {
      const float v = band_v[t];
      const int i = band_i[t];
      int rank = 0, greater = 0;
      for (int u = 0; u < nb; ++u) {
        greater += band_v[u] > v;
        rank += band_v[u] > v || (band_v[u] == v && band_i[u] < i);
      }
      if (rank == r - 1 && v > lo && v < hi) {  // the threshold element, strictly inside the band
        short_tau = __float_as_uint(v);
        short_quota = r - greater;
        short_ok = 1;
      }
      if (use_bitmap && rank < r) atomicOr(&bitmap[(i + qr.head) >> 5], 1u << ((i + qr.head) & 31));
    }
    __syncthreads();
    general = !short_ok;
    if (!general) {
      if (use_bitmap) {  // 4., usual route
        bitmap_compact(bitmap, n_words, S - qr.head, kept + S, k, sh.wave_tot);
        return;
      }
      tau = short_tau;
      quota = short_quota;
    }
  } else {
    for (int i0 = tid; i0 < E; i0 += 4 * kTopkThreads) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * kTopkThreads;
        v[u] = i < E ? cand[i] : -1.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * kTopkThreads;
        if (v[u] >= lo && v[u] <= hi)
          cand[i] = refined_score<DT>(p.geo, p.q_last, p.K, p.pm, p.ks_problem, p.ks_head, p.ks_token, row_stats, prob, c,
                                          S + i, g_lo, g_hi);
      }
    }
  }
  __syncthreads();

  // 3. general route: exact threshold by a radix select over the patched scores
  if (general) radix_select(sh, cand, E, k, false, &tau, &quota);

  // 4., general route or a row too long for the bitmap.  Every wave owns a contiguous sixteenth of the row's quads (wave 0 also
  //    the first edge, the last wave the last edge): it first counts its keys above and equal to
  //    the threshold, the sixteen counts give every wave its first output slot, then it reads its
  //    part again (cache-hot) and writes the selected positions in order; ties go to the lowest
  //    indices.  No workgroup barrier inside either loop.  Keys are compared as signed integers
  //    (scores are non-negative floats), so -1 stands for "no element".
  __shared__ int wave_gt[kTopkWaves], wave_eq[kTopkWaves];
  const int lane = tid & 63, wave = tid >> 6;
  const int itau = (int)tau;
  const int seg = ((qr.q_hi - qr.q_lo + kTopkWaves - 1) / kTopkWaves + 63) / 64 * 64;  // quads per wave
  const int seg_lo = qr.q_lo + wave * seg;
  const int seg_hi = seg_lo + seg < qr.q_hi ? seg_lo + seg : qr.q_hi;
  // edge elements as one more round of the first / the last wave: lanes 0..3 hold one element each
  int edge_key = -1, edge_at = 0;
  if (wave == 0 || wave == kTopkWaves - 1) {
    const int ei = lane < 4 ? edge_index(qr, (wave == 0 ? 0 : 4) + lane) : -1;
    if (ei >= 0) {
      edge_key = (int)__float_as_uint(cand[ei]);
      edge_at = ei;
    }
  }
  {
    int n_gt = 0, n_eq = 0;  // wave-uniform
    for (int q0 = seg_lo; q0 < seg_hi; q0 += kQuadUnroll * 64) {
      u32x4 v[kQuadUnroll];
#pragma unroll
      for (int u = 0; u < kQuadUnroll; ++u) {
        const int q = q0 + lane + u * 64;
        v[u] = qr.quads[q < seg_hi ? q : seg_hi - 1];
      }
#pragma unroll
      for (int u = 0; u < kQuadUnroll; ++u) {
        const bool valid = q0 + lane + u * 64 < seg_hi;
        const int key[4] = {(int)v[u].x, (int)v[u].y, (int)v[u].z, (int)v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          n_gt += __popcll(__ballot(valid && key[e] > itau));
          n_eq += __popcll(__ballot(valid && key[e] == itau));
        }
      }
    }
    n_gt += __popcll(__ballot(edge_key > itau));
    n_eq += __popcll(__ballot(edge_key == itau));
    if (lane == 0) {
      wave_gt[wave] = n_gt;
      wave_eq[wave] = n_eq;
    }
  }
  __syncthreads();
  int run_sel = 0, run_eq = 0;  // selected / equal keys before this wave's part (wave-uniform)
  for (int w = 0; w < wave; ++w) {
    run_sel += wave_gt[w];
    run_eq += wave_eq[w];
  }
  run_sel += run_eq < quota ? run_eq : quota;
  // one round: every lane holds four keys (key[e] = -1: none) of row elements at0 .. at0+3
  auto round = [&](const int (&key)[4], int at0) {
    bool sel[4];
    unsigned long long any_eq = 0ull;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sel[e] = key[e] > itau;
      any_eq |= __ballot(key[e] == itau);
    }
    if (any_eq) {  // rare: equal keys are selected while the quota lasts, lowest indices first
      int mine = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += key[e] == itau;
      int incl = mine;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      int before = run_eq + incl - mine;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (key[e] == itau) {
          sel[e] = before < quota;
          ++before;
        }
      run_eq += __shfl(incl, 63);
    }
    int pos = run_sel, total = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long b = __ballot(sel[e]);
      pos += lanes_below(b);
      total += __popcll(b);
    }
    if (sel[0] | sel[1] | sel[2] | sel[3]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (sel[e]) {
          if (pos < k) kept[S + pos] = (int32_t)(S + at0 + e);
          ++pos;
        }
    }
    run_sel += total;
  };
  if (wave == 0) {
    const int key[4] = {edge_key, -1, -1, -1};
    round(key, edge_at);
  }
  for (int q0 = seg_lo; q0 < seg_hi; q0 += kQuadUnroll * 64) {
    u32x4 v[kQuadUnroll];
#pragma unroll
    for (int u = 0; u < kQuadUnroll; ++u) {
      const int q = q0 + lane + u * 64;
      v[u] = qr.quads[q < seg_hi ? q : seg_hi - 1];
    }
#pragma unroll
    for (int u = 0; u < kQuadUnroll; ++u) {
      const int q = q0 + lane + u * 64;
      const bool valid = q < seg_hi;
      const int key[4] = {valid ? (int)v[u].x : -1, valid ? (int)v[u].y : -1, valid ? (int)v[u].z : -1,
                          valid ? (int)v[u].w : -1};
      round(key, 4 * q - qr.head);
    }
  }
  if (wave == kTopkWaves - 1) {
    const int key[4] = {edge_key, -1, -1, -1};
    round(key, edge_at);
  }
}

template <int DT>
__global__ __launch_bounds__(kTopkThreads) void topk_kernel(TopkParams p) {
  extern __shared__ __align__(16) uint32_t bitmap[];
  const int list = blockIdx.x;
  if (p.gate.row_flag && (*p.gate.n_flagged == 0 || p.gate.row_flag[list / p.n_lists] == 0)) return;  // gated launch: only the flagged rows
  topk_list<DT>(p, bitmap, list);
}

// ---- one-sweep dense path, whole row in one workgroup ------------------------------------------
// Statistics (fp64 merge of the chunks' partials), scores, top-k and ordered output of one selection list, the
// list's scores held in registers: thread t owns the quads t, t + 1024, ... of the row (4 consecutive tokens
// each).  Latency bound (one workgroup per list, a chain of memory round trips and barriers), so it replaces the
// launches of the general route below for rows of up to 24576 tokens (24 registers of scores per thread):
// statistics + combine + top-k took 21 + 11 + 23 us for 256 rows of 8192 tokens, this kernel 29, now 22; 9.5 + 4.5 + 15.3 and 14, then 10.7, for
// 2 rows of 4096.  Of the 22 and the 10.7, 3.5 and 2.4 go into the normalisers' heavy terms, and 1.6 into fp64 scores: both are left out
// where the band around the k-th score holds no more than is selected of it (2 rows x 4096, k = 188: a whole pass 19.9 -> 17.8 us, three
// such rows in four).  Calls of few, longer rows: see shortlist_kernel.
template <int DT, int NQ, bool SCORES>
__global__ __launch_bounds__(kTopkThreads) void row_select_kernel(RowSelectParams p) {
  constexpr int N = 4 * NQ;
  __shared__ ExactSums sh_exact;
  __shared__ RegSelect sh;
  __shared__ HeavyList heavy;
  __shared__ RowStat s_stat[64];  // up to 64 heads per KV head
  __shared__ float s_thr[64];
  __shared__ __align__(16) uint32_t bitmap[NQ * kTopkThreads * 4 / 32];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int list = blockIdx.x;
  const int row = list / p.n_lists, gl = list % p.n_lists;
  const RowGeom& geo = p.in.geo;
  const int G = geo.G, S = p.S, W = p.W, k = p.k, L = (int)geo.L;
  const int g_lo = p.n_lists > 1 ? gl : 0, g_hi = p.n_lists > 1 ? gl + 1 : G;
  const int prob = row / geo.Hkv, c = row % geo.Hkv;
  int32_t* kept_row = p.kept_idx + (int64_t)row * (S + p.n_lists * k + W);
  int32_t* kept = kept_row + S + gl * k;

  if (gl == 0) {
    for (int t = tid; t < S; t += kTopkThreads) kept_row[t] = t;
    for (int t = tid; t < W; t += kTopkThreads) kept_row[S + p.n_lists * k + t] = L - W + t;
  }
  if (k == 0 && !SCORES) return;
  // the logits of HB heads at a time, the next ones in flight while the current ones are used; the first are asked for
  // once a wave has done its part of the statistics
  constexpr int HB = NQ <= 2 ? 4 : NQ <= 4 ? 2 : 1;
  float4 x[2][HB][NQ];
  auto load_heads = [&](int g0, float4 (&dst)[HB][NQ]) {
#pragma unroll
    for (int h = 0; h < HB; ++h)
      if (g0 + h < g_hi) {
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
          const int tok = 4 * (u * kTopkThreads + tid);
          if (tok < L) dst[h][u] = *reinterpret_cast<const float4*>(p.in.logits + logit_index(geo, p.in.n_chunks, p.in.chunk, row, g0 + h, tok));
        }
      }
  };
  if (tid == 0 && p.flag) {
    p.flag[list] = 0;
    if (list == 0) *p.marker = kFlagsPerList;
  }
  const float max0 = exact_maximum(p.in, row, g_lo, g_hi, 0);
  for (int g = g_lo + wave; g < g_hi; g += kTopkWaves) {  // one wave per head
    const RowStat st = merge_partials_wave(p.in.partials + ((int64_t)row * G + g) * p.in.n_chunks, p.in.n_chunks);
    if ((tid & 63) == 0) {
      s_stat[g] = st;
      s_thr[g] = heavy_logit_threshold(st.M, (float)st.Z);
    }
  }
  for (int w = tid; w < (int)(sizeof(bitmap) / 4); w += kTopkThreads) bitmap[w] = 0u;
  if (tid == 0) heavy.n = 0;
  if (tid < 64) heavy.change[tid] = 0ull;
  // The heavy terms change a normaliser by a few 1e-6 at most: scores that are written out have them in, the selection
  // only needs them where it comes to fp64 scores.
  auto exact = [&]() {
    if (exact_changes<DT>(p.in, sh_exact, row, g_lo, g_hi, s_stat, s_thr, max0, [] {})) exact_apply(sh_exact, g_lo, g_hi, s_stat);
  };
  if (SCORES) exact();
  load_heads(g_lo, x[0]);
  if (!SCORES) __syncthreads();

  auto note = [&](int t, int g, int tok, float l) {
    if (t < kHeavyMost) {
      heavy.tok[t] = tok;
      heavy.logit[t] = l;
      heavy.head[t] = (unsigned char)g;
    }
  };
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = 0.f;
  auto add_heads = [&](int g0, const float4 (&src)[HB][NQ]) {
#pragma unroll
    for (int h = 0; h < HB; ++h)
      if (g0 + h < g_hi) {
        const float M = s_stat[g0 + h].M, inv = s_stat[g0 + h].invZ, thr = SCORES ? INFINITY : s_thr[g0 + h];
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
          const int tok = 4 * (u * kTopkThreads + tid);
          if (tok < L) {
            const float top = fmaxf(fmaxf(src[h][u].x, src[h][u].y), fmaxf(src[h][u].z, src[h][u].w));
            if (!SCORES && top >= thr) {  // rare
              const float l[4] = {src[h][u].x, src[h][u].y, src[h][u].z, src[h][u].w};
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (l[e] >= thr && tok + e < L) note(atomicAdd(&heavy.n, 1), g0 + h, tok + e, l[e]);
            }
            v[4 * u] += exp_times(src[h][u].x - M, inv);
            v[4 * u + 1] += exp_times(src[h][u].y - M, inv);
            v[4 * u + 2] += exp_times(src[h][u].z - M, inv);
            v[4 * u + 3] += exp_times(src[h][u].w - M, inv);
          }
        }
      }
  };
  for (int g = g_lo; g < g_hi; g += 2 * HB) {
    if (g + HB < g_hi) load_heads(g + HB, x[1]);
    add_heads(g, x[0]);
    if (g + HB >= g_hi) break;
    if (g + 2 * HB < g_hi) load_heads(g + 2 * HB, x[0]);
    add_heads(g + HB, x[1]);
  }
  float* out = SCORES ? p.scores + (int64_t)list * p.pitch : nullptr;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int tok = 4 * ((i >> 2) * kTopkThreads + tid) + (i & 3);
    if (SCORES && tok < L) out[tok] = v[i];
    if (tok < S || tok >= L - W) v[i] = -1.f;
  }
  if (k == 0) return;

  // the k-th score's bracket, and the band around it (see topk_kernel)
  uint32_t tlo, thi;
  bracket_kth<true>(sh, [&](auto f) {
#pragma unroll
    for (int i = 0; i < N; ++i) f(v[i]);
  }, k, &tlo, &thi);
  const float lo = __uint_as_float(tlo) * (1.0f - p.band) - kDenormSlack,
              hi = __uint_as_float(thi) * (1.0f + p.band) + kDenormSlack;
  int above = 0;  // wave-uniform
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    uint32_t nib = 0u;
    const int q = u * kTopkThreads + tid;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = v[4 * u + e];
      const bool gt = x > hi;
      above += __popcll(__ballot(gt));
      nib |= gt ? 1u << e : 0u;
      if (!gt && x >= 0.f && x >= lo) {
        const int t = atomicAdd(&sh.n_band, 1);
        if (t < kMaxBand) sh.band_tok[t] = 4 * q + e;
      }
    }
    if (nib) atomicOr(&bitmap[q >> 3], nib << (4 * (q & 7)));
  }
  if ((tid & 63) == 0 && above) atomicAdd(&sh.n_above, above);
  __syncthreads();
  const int nb = sh.n_band, r = k - sh.n_above;
  bool general = nb > kMaxBand || r < 1 || r > nb;
  const bool whole = !SCORES && !general && nb == r;  // the whole band is selected: no need to rank it
  bool together = !SCORES && !general && nb * (g_hi - g_lo) <= kMaxBand;
  if (whole) {
    for (int t = tid; t < nb; t += kTopkThreads) atomicOr(&bitmap[sh.band_tok[t] >> 5], 1u << (sh.band_tok[t] & 31));
    __syncthreads();
  } else if (!SCORES) {
    if (heavy.n > kHeavyList) {
      auto any = [&](int g) { return s_thr[g] <= s_stat[g].M; };
      raise_thresholds(p.in, sh.hist[0], row, g_lo, g_hi, s_stat, s_thr, any);  // (the histograms are done with)
      if (tid == 0) heavy.n = 0;
      __syncthreads();
      each_four(p.in, row, g_lo, g_hi, any, [&](int g, int tok, const float (&l)[4]) {
        const float thr = s_thr[g];
        unsigned long long in[4];
        int cnt = 0, at = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          in[e] = __ballot(l[e] >= thr);
          cnt += __popcll(in[e]);
        }
        if (cnt == 0) return;  // wave-uniform
        if ((tid & 63) == 0) at = atomicAdd(&heavy.n, cnt);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (l[e] >= thr) note(at + lanes_below(in[e]), g, tok + e, l[e]);
          at += __popcll(in[e]);
        }
      });
      __syncthreads();
      together &= heavy.n <= kHeavyMost;
    }
    if (!together) exact();
  }
  if (!whole && !general) {
    if (together)
      refine_band_exact<DT>(sh, heavy, nb, p.in, row, g_lo, g_hi, s_stat);
    else
      refine_band<DT>(sh, nb, geo, p.in.q_last, p.in.K, p.in.pm, p.in.ks_problem, p.in.ks_head, p.in.ks_token, s_stat, prob, c, g_lo, g_hi);
    if (tid == 0) sh.n_band = 0;  // now: 1 = the threshold lies strictly inside the band
    __syncthreads();
    for (int t = tid; t < nb; t += kTopkThreads) {
      const float x = sh.band_v[t];
      const int tok = sh.band_tok[t];
      if (SCORES) out[tok] = x;
      int rank = 0;
      for (int u = 0; u < nb; ++u) rank += sh.band_v[u] > x || (sh.band_v[u] == x && sh.band_tok[u] < tok);
      if (rank == r - 1 && x > lo && x < hi) sh.n_band = 1;
      if (rank < r) atomicOr(&bitmap[tok >> 5], 1u << (tok & 31));
    }
    __syncthreads();
    general = sh.n_band == 0;
  }
  if (general) {
    if (tid == 0 && p.flag) p.flag[list] = 1;
    // near-ties by the thousand, or a refined threshold on the band's edge: refine the whole band in place, then an
    // exact radix select over the registers; equal scores go to the lowest tokens while the quota lasts
    __syncthreads();
    for (int w = tid; w < (int)(sizeof(bitmap) / 4); w += kTopkThreads) bitmap[w] = 0u;
#pragma unroll 1
    for (int i = 0; i < N; ++i) {
      float x = 0.f;
      const int tok = 4 * ((i >> 2) * kTopkThreads + tid) + (i & 3);
#pragma unroll
      for (int j = 0; j < N; ++j) x = j == i ? v[j] : x;
      if (x >= 0.f && x >= lo && x <= hi) {
        x = refined_score<DT>(geo, p.in.q_last, p.in.K, p.in.pm, p.in.ks_problem, p.in.ks_head, p.in.ks_token, s_stat, prob, c, tok, g_lo, g_hi);
        if (SCORES) out[tok] = x;
      }
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] = j == i ? x : v[j];
    }
    uint32_t prefix = 0u, mask = 0u;
    int rem = k, bin;
    for (int digit = 0; digit < 3; ++digit) {
      const int shift = digit == 0 ? 20 : digit == 1 ? 9 : 0, bits = digit == 2 ? 9 : 11;
      for (int b = tid; b < kHistBins; b += kTopkThreads) sh.hist[0][b] = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const uint32_t key = __float_as_uint(v[i]);
        if (v[i] >= 0.f && (key & mask) == prefix) atomicAdd(&sh.hist[0][(key >> shift) & ((1u << bits) - 1u)], 1);
      }
      __syncthreads();
      pick_digit(sh.hist[0], sh.wave_tot, sh.pick, 1 << bits, rem, &bin, &rem);
      prefix |= (uint32_t)bin << shift;
      mask |= ((1u << bits) - 1u) << shift;
    }
    int before = 0;  // equal scores in front of the quads at hand
#pragma unroll 1
    for (int u = 0; u < NQ; ++u) {
      float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < N; ++j)
        if ((j >> 2) == u) x[j & 3] = v[j];
      const int q = u * kTopkThreads + tid;
      int eq = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) eq += __float_as_uint(x[e]) == prefix;
      int tot;
      __syncthreads();  // wave_tot
      int at = before + block_scan_incl(eq, sh.wave_tot, &tot) - eq;
      uint32_t nib = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool same = __float_as_uint(x[e]) == prefix;
        if (__float_as_int(x[e]) > (int)prefix || (same && at < rem)) nib |= 1u << e;
        at += same;
      }
      if (nib) atomicOr(&bitmap[q >> 3], nib << (4 * (q & 7)));
      before += tot;
    }
    __syncthreads();
  }
  bitmap_compact(bitmap, (L + 31) >> 5, 0, kept, k, sh.wave_tot);
}

// Longer rows: the same statistics, for the combine stage.
template <int DT>
__global__ __launch_bounds__(kTopkThreads) void row_stats_kernel(RowStatsParams p) {
  __shared__ ExactSums sh;
  __shared__ RowStat s_stat[64];
  __shared__ float s_thr[64];
  const int tid = threadIdx.x, row = blockIdx.x, G = p.in.geo.G;
  for (int b = tid; b < kHistBins * p.n_lists; b += kTopkThreads) p.ghist[(int64_t)row * p.n_lists * kHistBins + b] = 0;
  const float max0 = exact_maximum(p.in, row, 0, G, 0);
  for (int g = tid >> 6; g < G; g += kTopkWaves) {
    const RowStat st = merge_partials_wave(p.in.partials + ((int64_t)row * G + g) * p.in.n_chunks, p.in.n_chunks);
    if ((tid & 63) == 0) {
      s_stat[g] = st;
      s_thr[g] = heavy_logit_threshold(st.M, (float)st.Z);
    }
  }
  if (exact_changes<DT>(p.in, sh, row, 0, G, s_stat, s_thr, max0, [] {})) exact_apply(sh, 0, G, s_stat);
  if (tid < G) p.stats[(int64_t)row * G + tid] = s_stat[tid];
}

// ---- one-sweep dense path, a row spread over many workgroups -------------------------------------
// First launch: a workgroup per list and kShortTokens tokens turns the logits into scores and hands on the few that can be
// among the k best: those at or above a threshold that every workgroup of a list finds for itself, from the same sample of the list's own
// scores.  More workgroups, one per list or several that share its heads, take the heavy terms into the normalisers (exact_changes), which only the fp64
// scores of the band around the k-th need: 1e-6 of a score against the band's 2e-4.  Heads with heavy terms in nearly every chunk have hundreds of
// them and raise their thresholds; whole passes over N(60, 1), us, with one workgroup per list that takes every term, and this: 8 rows x 32K x 4 heads
// 95 and 44.7 (39.3 at N(0, 1)), x 16 heads 267 and 55 (53), 32 x 32K x 7 heads 183 and 103 (92), fp32 8 x 30000 x 4 131 and 58 (53).
// Latency bound: 6.6 us for 8 rows x 32K tokens x 4 heads, of them 2.2 for partials and logits, 1.4 exponentials, 2.4 the threshold; the
// second launch 5.8 (13.5 for 8 rows x 128K, k = 3580, of them 2.0 to collect the scores, 2.9 bracket, 1.7 band, 3.5 fp64 scores, 2.2
// output).  Together they stand for statistics, combine and top-k in launches of their own, 4.5 + 7 + 13.5, and for a whole pass over those rows
// 51.4 -> 37.3 us.  The sample is 128 runs of 16 tokens, 64 bytes of a head's logits each: 512 runs of four cost every workgroup
// four times the lines (4.0 us instead of 2.2, 10.6 instead of 4.5 with 32 rows).  NQ = 2: half as many workgroups where a CU
// would get more than one (32 rows x 32K: 25 us and 12 under the profiler).
template <int DT, int HB, int NQ>
__global__ __launch_bounds__(kTopkThreads) void shortlist_kernel(ShortlistParams p) {
  __shared__ union {
    ExactSums exact;
    RegSelect sel;
  } sh_u;
  __shared__ RowStat s_stat[64];
  __shared__ float s_thr[64];
  __shared__ int n_out;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int list = blockIdx.y, part = (int)blockIdx.x - p.n_exact, row = list / p.n_lists, gl = list % p.n_lists;
  const RowGeom& geo = p.in.geo;
  const int G = geo.G, L = (int)geo.L;
  const int g_lo = p.n_lists > 1 ? gl : 0, g_hi = p.n_lists > 1 ? gl + 1 : G;
  const ChunkPartial* partials = p.in.partials + (int64_t)row * G * p.in.n_chunks;
  if (part < 0) {
    const int per = (g_hi - g_lo + p.n_exact - 1) / p.n_exact, lo = g_lo + per * (int)blockIdx.x, hi = lo + per < g_hi ? lo + per : g_hi;
    if (lo >= hi) return;
    __shared__ bool s_many[64];
    const float max0 = exact_maximum(p.in, row, lo, hi, 0);
    for (int g = lo + wave; g < hi; g += kTopkWaves) {
      const ChunkPartial* pr = partials + (int64_t)g * p.in.n_chunks;
      const RowStat st = merge_partials_wave(pr, p.in.n_chunks);
      const float thr = heavy_logit_threshold(st.M, (float)st.Z);
      int n = 0;  // chunks that hold heavy terms
      if (thr <= st.M)  // wave-uniform, rare
        for (int i = 0; i < p.in.n_chunks; i += 64) n += __popcll(__ballot(i + lane < p.in.n_chunks && pr[i + lane].max >= thr));
      if (lane == 0) {
        s_stat[g] = st;
        s_thr[g] = thr;
        s_many[g] = 8 * n > 7 * p.in.n_chunks;
      }
    }
    auto raise = [&] {
      bool many = false;
      for (int g = lo; g < hi; ++g) many |= s_many[g];
      if (many) raise_thresholds(p.in, reinterpret_cast<int*>(&sh_u), row, lo, hi, s_stat, s_thr, [&](int g) { return s_many[g]; });
    };
    if (exact_changes<DT>(p.in, sh_u.exact, row, lo, hi, s_stat, s_thr, max0, raise)) exact_apply(sh_u.exact, lo, hi, s_stat);
    if (tid >= lo && tid < hi) p.stats[(int64_t)row * G + tid] = s_stat[tid];
    return;
  }
  constexpr int kPart = 4 * NQ * kTopkThreads;
  const int tok0 = part * kPart + 4 * tid;  // this thread's first four tokens of NQ times four,
  const int run0 = 16 * (p.first_run + (int)(((tid >> 2) * p.step) >> 16)) + 4 * (tid & 3);  // and its four of the sample
  const bool sampled = tid < 4 * p.n_runs;
  float4 x[HB][NQ], y[HB];
  auto load = [&](int g0) {
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      y[h] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < NQ; ++u) x[h][u] = y[h];
      if (g0 + h < g_hi) {
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
          const int tok = tok0 + 4 * u * kTopkThreads;
          if (tok < L) x[h][u] = *reinterpret_cast<const float4*>(p.in.logits + logit_index(geo, p.in.n_chunks, p.in.chunk, row, g0 + h, tok));
        }
        if (sampled) y[h] = *reinterpret_cast<const float4*>(p.in.logits + logit_index(geo, p.in.n_chunks, p.in.chunk, row, g0 + h, run0));
      }
    }
  };
  load(g_lo);
  for (int g = g_lo + (kTopkWaves - 1 - wave); g < g_hi; g += kTopkWaves) {  // (the last waves hold no sample)
    const RowStat st = merge_partials_wave(partials + (int64_t)g * p.in.n_chunks, p.in.n_chunks);
    if (lane == 0) s_stat[g] = st;
  }
  if (tid == 0) n_out = 0;
  __syncthreads();
  float v[NQ][4], w[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < NQ; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[u][e] = 0.f;
  auto add = [](float (&a)[4], const float4& l, float M, float inv) {
    a[0] += exp_times(l.x - M, inv);
    a[1] += exp_times(l.y - M, inv);
    a[2] += exp_times(l.z - M, inv);
    a[3] += exp_times(l.w - M, inv);
  };
  for (int g0 = g_lo;;) {
#pragma unroll
    for (int h = 0; h < HB; ++h)
      if (g0 + h < g_hi) {
        const float M = s_stat[g0 + h].M, inv = s_stat[g0 + h].invZ;
        if (sampled) add(w, y[h], M, inv);
#pragma unroll
        for (int u = 0; u < NQ; ++u) add(v[u], x[h][u], M, inv);
      }
    g0 += HB;
    if (g0 >= g_hi) break;
    load(g0);
  }
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const int tok = tok0 + 4 * u * kTopkThreads;
    if (tok < L) *reinterpret_cast<float4*>(p.scores + (int64_t)list * p.pitch + tok) = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
  }
  uint32_t tlo = 0u, thi;
  if (p.rank > 0)  // (0: everything passes)
    bracket_kth<false>(sh_u.sel, [&](auto f) {
#pragma unroll
      for (int e = 0; e < 4; ++e) f(sampled ? w[e] : -1.f);
    }, p.rank, &tlo, &thi);
  const float tau = __uint_as_float(tlo);
  bool ok[NQ][4];
  unsigned long long bal[NQ][4];
  int n_wave = 0;
#pragma unroll
  for (int u = 0; u < NQ; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int tok = tok0 + 4 * u * kTopkThreads + e;
      ok[u][e] = tok >= p.S && tok < L - p.W && v[u][e] >= tau;
      bal[u][e] = __ballot(ok[u][e]);
      n_wave += __popcll(bal[u][e]);
    }
  int base = 0;
  if (lane == 0 && n_wave) base = atomicAdd(&n_out, n_wave);
  base = __builtin_amdgcn_readfirstlane(base);
  uint2* out = p.cand + ((int64_t)list * p.n_parts + part) * kPart;
#pragma unroll
  for (int u = 0; u < NQ; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (ok[u][e]) out[base + lanes_below(bal[u][e])] = make_uint2(__float_as_uint(v[u][e]), (uint32_t)(tok0 + 4 * u * kTopkThreads + e));
      base += __popcll(bal[u][e]);
    }
  __syncthreads();
  if (tid == 0) {
    p.count[(int64_t)list * p.n_parts + part] = n_out;
    if (part == 0) p.tau[list] = tau;
  }
}

// Second launch: a workgroup per list selects among the scores handed on, in registers, as row_select_kernel does.  Where they do
// not do (a threshold that turned out too high or far too low, a band of near-ties), the same workgroup goes through the list's
// score row instead.
template <int DT, int NPT>
__global__ __launch_bounds__(kTopkThreads) void shortlist_select_kernel(ShortlistParams p, TopkParams tp) {
  __shared__ RegSelect sh;
  __shared__ RowStat s_stat[64];
  __shared__ int part_off[kShortParts + 1];
  extern __shared__ __align__(16) uint32_t bitmap[];
  const int tid = threadIdx.x, list = blockIdx.x;
  const int row = list / p.n_lists, gl = list % p.n_lists;
  const RowGeom& geo = tp.geo;
  const int G = geo.G, S = tp.S, W = tp.W, k = tp.k, L = (int)geo.L, E = L - S - W;
  const int g_lo = p.n_lists > 1 ? gl : 0, g_hi = p.n_lists > 1 ? gl + 1 : G;
  const int prob = row / geo.Hkv, c = row % geo.Hkv;
  int32_t* kept_row = tp.kept_idx + (int64_t)row * (S + p.n_lists * k + W);
  int32_t* kept = kept_row + S + gl * k;

  const int raw = tid < p.n_parts ? p.count[(int64_t)list * p.n_parts + tid] : 0;
  const float tau = p.tau[list];
  if (tid >= g_lo && tid < g_hi) s_stat[tid] = p.stats[(int64_t)row * G + tid];
  if (gl == 0) {
    for (int t = tid; t < S; t += kTopkThreads) kept_row[t] = t;
    for (int t = tid; t < W; t += kTopkThreads) kept_row[S + p.n_lists * k + t] = L - W + t;
  }
  if (tid == 0 && p.flag) {
    p.flag[list] = 0;
    if (list == 0) *p.marker = kFlagsPerList;
  }
  const int n_words = (E + 31) >> 5;
  for (int w = tid; w < n_words; w += kTopkThreads) bitmap[w] = 0u;
  int n_c;
  const int incl = block_scan_incl(raw, sh.wave_tot, &n_c);
  if (tid < p.n_parts) part_off[tid] = incl - raw;
  if (tid == 0) part_off[p.n_parts] = n_c;
  __syncthreads();
  bool ok = n_c >= k && n_c <= NPT * kTopkThreads;
  if (ok) {
    const uint2* in = p.cand + (int64_t)list * p.n_parts * p.part_tokens;
    float v[NPT];
    int tok[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      v[u] = -1.f;
      tok[u] = S;
      const int j0 = u * kTopkThreads + (tid & ~63), j = j0 + (tid & 63);  // a wave's 64 lie in one part or a few adjacent ones
      if (j0 < n_c) {
        int at = -1;  // the last part that begins at or before j0
        for (int q = 0; q < p.n_parts; q += 64) at += __popcll(__ballot(q + (tid & 63) < p.n_parts && part_off[q + (tid & 63)] <= j0));
        int from = part_off[at], to = part_off[at + 1];
        while (__any(j >= to && j < n_c)) {
          if (j >= to && j < n_c) {
            ++at;
            from = to;
            to = part_off[at + 1];
          }
        }
        if (j < n_c) {
          const uint2 r = in[(int64_t)at * p.part_tokens + (j - from)];
          v[u] = __uint_as_float(r.x);
          tok[u] = (int)r.y;
        }
      }
    }
    uint32_t tlo, thi;
    bracket_kth<true>(sh, [&](auto f) {
#pragma unroll
      for (int u = 0; u < NPT; ++u) f(v[u]);
    }, k, &tlo, &thi);
    const float lo = __uint_as_float(tlo) * (1.0f - tp.band) - kDenormSlack,
                hi = __uint_as_float(thi) * (1.0f + tp.band) + kDenormSlack;
    int above = 0;  // wave-uniform
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const bool gt = v[u] > hi;
      above += __popcll(__ballot(gt));
      if (gt) {
        atomicOr(&bitmap[(tok[u] - S) >> 5], 1u << ((tok[u] - S) & 31));
      } else if (v[u] >= 0.f && v[u] >= lo) {
        const int t = atomicAdd(&sh.n_band, 1);
        if (t < kMaxBand) sh.band_tok[t] = tok[u];
      }
    }
    if ((tid & 63) == 0 && above) atomicAdd(&sh.n_above, above);
    __syncthreads();
    const int nb = sh.n_band, r = k - sh.n_above;
    // (what was not handed on scores below tau: none of it reaches the band; tau = 0: everything was handed on)
    ok = (lo >= tau || tau == 0.f) && nb <= kMaxBand && r >= 1 && r <= nb;
    if (ok && nb == r) {  // the whole band is selected: no need to rank it
      for (int t = tid; t < nb; t += kTopkThreads) atomicOr(&bitmap[(sh.band_tok[t] - S) >> 5], 1u << ((sh.band_tok[t] - S) & 31));
      __syncthreads();
    } else if (ok) {
      refine_band<DT>(sh, nb, geo, tp.q_last, tp.K, tp.pm, tp.ks_problem, tp.ks_head, tp.ks_token, s_stat, prob, c, g_lo, g_hi);
      if (tid == 0) sh.n_band = 0;  // now: 1 = the threshold lies strictly inside the band
      __syncthreads();
      for (int t = tid; t < nb; t += kTopkThreads) {
        const float x = sh.band_v[t];
        const int i = sh.band_tok[t];
        int rank = 0;
        for (int u = 0; u < nb; ++u) rank += sh.band_v[u] > x || (sh.band_v[u] == x && sh.band_tok[u] < i);
        if (rank == r - 1 && x > lo && x < hi) sh.n_band = 1;
        if (rank < r) atomicOr(&bitmap[(i - S) >> 5], 1u << ((i - S) & 31));
      }
      __syncthreads();
      ok = sh.n_band != 0;
    }
  }
  if (ok) {
    bitmap_compact(bitmap, n_words, S, kept, k, sh.wave_tot);
  } else {
    if (tid == 0 && p.flag) p.flag[list] = 1;
    __syncthreads();
    topk_list<DT>(tp, bitmap, list);
  }
}

// ---- gather -----------------------------------------------------------------------------------
constexpr int kGatherThreads = 256;
constexpr int kGatherTokens = 64;  // reduced-cache rows one workgroup copies
// From so many bytes written on, the rows are stored nontemporally.  Plain stores leave the Infinity Cache (256 MB) full of lines that
// have yet to go to memory, and whoever streams next pays for them at a multiple of their bytes (see the filtering pass's
// candidates); nontemporal ones go out during the gather.  So it depends on what follows, us, plain and nontemporal (inputs in
// rotation, "1 GB": a read of that much, as a model's weights are between a pass and the step's attention, and between steps):
//   rows x tokens, MB written    pass after pass   pass, 1 GB, step, 1 GB   pass, step, 1 GB
//   256 x   8K, 134                194   182           733   731               469   470
//   256 x   8K, 268                229   215           787   781               518   525
//   256 x  32K, 101                413   406           951   949               691   692
//   256 x  32K, 201                460   448          1014  1009               744   753
//   256 x  32K, 268                503   483          1056  1049               784   793
//   256 x  64K, 537                969   921          1539  1527              1231  1242
//   256 x 128K, 537               1545  1519          2153  2127              1875  1871
//   256 x 128K, 1057              1802  1780          2453  2460              2189  2167
// Where the step reads the cache right behind the pass, it would have found some of it on the chip: 1 % is lost there.  With less
// written the gain goes (64 rows x 8K, 67 MB: 69 and 71 pass after pass).
// Beyond so many bytes of keys the stores are plain: there the totals are even (256 x 128K, 537 MB, a pass and 256 steps: 23.6 ms
// either way, inputs in rotation 1521 and 1517 us a pass), and a pass that stands between steps ends later by what it
// does not leave to them, 1503 and 1522 us.
constexpr int64_t kStreamGather = 96ll << 20, kStreamGatherKeys = 6ll << 30;

template <int LPT, bool STREAM>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(GatherParams p, int eb) {
  const int row = blockIdx.y;
  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int sub = threadIdx.x / LPT, cl = threadIdx.x % LPT;
  constexpr int TPI = kGatherThreads / LPT;  // tokens per iteration
  const int64_t row_bytes = (int64_t)p.geo.D * eb;
  const CacheRow Kc = cache_row(p.Kc, p.cpm, false, prob, c, row, p.cap, (int)row_bytes, eb);
  const CacheRow Vc = cache_row(p.Vc, p.cpm, true, prob, c, row, p.cap, (int)row_bytes, eb);
  const int32_t* kept = p.kept_idx + (int64_t)row * p.n_kept;
  const int t0 = blockIdx.x * kGatherTokens;
  constexpr int NIT = kGatherTokens / TPI;
  // all of a thread's loads are issued before its first store: positions first, then the rows
  // (streaming loads: the full cache is not read again)
  int64_t src[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int t = t0 + it * TPI + sub;
    src[it] = kept[t < p.n_kept ? t : p.n_kept - 1];
  }
  uint4 a[NIT], b[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int64_t i = src[it] < 0 ? 0 : (src[it] >= p.geo.L ? p.geo.L - 1 : src[it]);  // never read outside the row
    const int64_t ko = kv_offset(p.pm, p.pm.ks_page, p.ks_problem, p.ks_head, p.ks_token, prob, c, i);
    const int64_t vo = kv_offset(p.pm, p.pm.vs_page, p.vs_problem, p.vs_head, p.vs_token, prob, c, i);
    a[it] = ld16_stream((const char*)p.K + ko * eb + cl * 16);
    b[it] = ld16_stream((const char*)p.V + vo * eb + cl * 16);
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int t = t0 + it * TPI + sub;
    if (t < p.n_kept) {
      if (STREAM) {
        st16_stream(Kc.at(t) + cl * 16, a[it]);
        st16_stream(Vc.at(t) + cl * 16, b[it]);
      } else {
        st16(Kc.at(t) + cl * 16, a[it]);
        st16(Vc.at(t) + cl * 16, b[it]);
      }
    }
  }
}

}  // namespace

// Room for one bit per candidate, whatever the row's alignment.
static int64_t bitmap_bytes(const TopkParams& p) { return ((p.geo.L - p.S - p.W + 3 + 31) / 32 + 3) / 4 * 16; }

template <int DT, int NPT>
static hipError_t launch_shortlist_select(const ShortlistParams& p, const TopkParams& tp, unsigned lists, hipStream_t s) {
  static uint64_t done = 0;
  const hipError_t e = allow_dynamic_lds((const void*)shortlist_select_kernel<DT, NPT>, kShortMax / 8 + 16, &done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((shortlist_select_kernel<DT, NPT>), dim3(lists), dim3(kTopkThreads), tp.bitmap_bytes, s, p, tp);
  return hipGetLastError();
}

template <int DT>
static hipError_t launch_shortlist_t(const ShortlistParams& p, const TopkParams& tp, unsigned lists, hipStream_t s) {
  const dim3 grid((unsigned)(p.n_parts + p.n_exact), lists);
  const int heads = p.n_lists > 1 ? 1 : p.in.geo.G;
#define SAGEKV_LAUNCH(HB)                                                                              \
  if (p.part_tokens == kShortTokens)                                                                   \
    hipLaunchKernelGGL((shortlist_kernel<DT, HB, 1>), grid, dim3(kTopkThreads), 0, s, p);              \
  else                                                                                                 \
    hipLaunchKernelGGL((shortlist_kernel<DT, HB, 2>), grid, dim3(kTopkThreads), 0, s, p)
  if (heads == 1) {
    SAGEKV_LAUNCH(1);
  } else if (heads <= 4 || p.part_tokens != kShortTokens) {
    SAGEKV_LAUNCH(4);
  } else {
    hipLaunchKernelGGL((shortlist_kernel<DT, 8, 1>), grid, dim3(kTopkThreads), 0, s, p);
  }
#undef SAGEKV_LAUNCH
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // 6 beside 8: 8 rows x 128K, k = 1788 79.4 -> 78.8 us, 8 x 32K, k = 2600 42.1 -> 41.7; 12 beside 16 (8 x 128K, k = 3580; 4 x 128K x 7) was even
  return p.expect <= 4 * kTopkThreads    ? launch_shortlist_select<DT, 4>(p, tp, lists, s)
         : p.expect <= 6 * kTopkThreads  ? launch_shortlist_select<DT, 6>(p, tp, lists, s)
         : p.expect <= 8 * kTopkThreads  ? launch_shortlist_select<DT, 8>(p, tp, lists, s)
                                         : launch_shortlist_select<DT, 16>(p, tp, lists, s);
}

hipError_t launch_shortlist(const ShortlistParams& p, const TopkParams& tp0, hipStream_t s) {
  const RowGeom& geo = p.in.geo;
  if (geo.G > 64 || p.n_parts > kShortParts || p.n_exact < 1 || (p.part_tokens != kShortTokens && p.part_tokens != 2 * kShortTokens) || geo.L - tp0.S - tp0.W > kShortMax) return hipErrorInvalidValue;
  TopkParams tp = tp0;
  tp.ghist = nullptr;
  tp.bitmap_bytes = (int)bitmap_bytes(tp);
  const unsigned lists = (unsigned)(geo.n_problems * geo.Hkv * p.n_lists);
  return geo.dtype == DT_BF16 ? launch_shortlist_t<DT_BF16>(p, tp, lists, s) : launch_shortlist_t<DT_F32>(p, tp, lists, s);
}

hipError_t launch_topk(const TopkParams& p0, hipStream_t s) {
  constexpr int kMaxBitmap = 64 * 1024;
  static uint64_t done_bf16 = 0, done_f32 = 0;
  hipError_t e = p0.geo.dtype == DT_BF16 ? allow_dynamic_lds((const void*)topk_kernel<DT_BF16>, kMaxBitmap, &done_bf16)
                                         : allow_dynamic_lds((const void*)topk_kernel<DT_F32>, kMaxBitmap, &done_f32);
  if (e != hipSuccess) return e;
  TopkParams p = p0;
  const int64_t need = bitmap_bytes(p);
  p.bitmap_bytes = need <= kMaxBitmap ? (int)need : 0;
  const int lists = p.geo.n_problems * p.geo.Hkv * p.n_lists;
  if (p.geo.dtype == DT_BF16)
    hipLaunchKernelGGL(topk_kernel<DT_BF16>, dim3((unsigned)lists), dim3(kTopkThreads), p.bitmap_bytes, s, p);
  else
    hipLaunchKernelGGL(topk_kernel<DT_F32>, dim3((unsigned)lists), dim3(kTopkThreads), p.bitmap_bytes, s, p);
  return hipGetLastError();
}

hipError_t launch_row_select(const RowSelectParams& p, hipStream_t s) {
  if (p.in.geo.L > kRowSelectMax || p.in.geo.G > 64) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(p.in.geo.n_problems * p.in.geo.Hkv * p.n_lists));
  const int quads = (int)((p.in.geo.L + 4 * kTopkThreads - 1) / (4 * kTopkThreads));  // per thread
#define SAGEKV_LAUNCH(NQ)                                                                                       \
  if (p.in.geo.dtype == DT_BF16 && p.scores)                                                                       \
    hipLaunchKernelGGL((row_select_kernel<DT_BF16, NQ, true>), grid, dim3(kTopkThreads), 0, s, p);              \
  else if (p.in.geo.dtype == DT_BF16)                                                                              \
    hipLaunchKernelGGL((row_select_kernel<DT_BF16, NQ, false>), grid, dim3(kTopkThreads), 0, s, p);             \
  else if (p.scores)                                                                                            \
    hipLaunchKernelGGL((row_select_kernel<DT_F32, NQ, true>), grid, dim3(kTopkThreads), 0, s, p);               \
  else                                                                                                          \
    hipLaunchKernelGGL((row_select_kernel<DT_F32, NQ, false>), grid, dim3(kTopkThreads), 0, s, p)
  if (quads <= 1) {
    SAGEKV_LAUNCH(1);
  } else if (quads <= 2) {
    SAGEKV_LAUNCH(2);
  } else if (quads <= 4) {
    SAGEKV_LAUNCH(4);
  } else {
    SAGEKV_LAUNCH(6);
  }
#undef SAGEKV_LAUNCH
  return hipGetLastError();
}

hipError_t launch_row_stats(const RowStatsParams& p, hipStream_t s) {
  if (p.in.geo.G > 64) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(p.in.geo.n_problems * p.in.geo.Hkv));
  if (p.in.geo.dtype == DT_BF16)
    hipLaunchKernelGGL(row_stats_kernel<DT_BF16>, grid, dim3(kTopkThreads), 0, s, p);
  else
    hipLaunchKernelGGL(row_stats_kernel<DT_F32>, grid, dim3(kTopkThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_gather(const GatherParams& p, hipStream_t s) {
  const int rows = p.geo.n_problems * p.geo.Hkv;
  const int eb = p.geo.dtype == DT_BF16 ? 2 : 4;
  const int lpt = p.geo.D * eb / 16;
  dim3 grid((unsigned)((p.n_kept + kGatherTokens - 1) / kGatherTokens), (unsigned)rows);
  const int64_t token_bytes = (int64_t)rows * p.geo.D * eb;
  const bool stream = 2 * token_bytes * p.n_kept > kStreamGather && token_bytes * p.geo.L <= kStreamGatherKeys;
#define SAGEKV_LAUNCH(LPT)                                                                          \
  if (stream)                                                                                        \
    hipLaunchKernelGGL((gather_kernel<LPT, true>), grid, dim3(kGatherThreads), 0, s, p, eb);         \
  else                                                                                               \
    hipLaunchKernelGGL((gather_kernel<LPT, false>), grid, dim3(kGatherThreads), 0, s, p, eb)
  switch (lpt) {
    case 8: SAGEKV_LAUNCH(8); break;
    case 16: SAGEKV_LAUNCH(16); break;
    case 32: SAGEKV_LAUNCH(32); break;
    default: return hipErrorInvalidValue;
  }
#undef SAGEKV_LAUNCH
  return hipGetLastError();
}

}  // namespace sagekv
