// Fast eviction path (paper Sec. 2 Step 2, same result as the dense path): instead of writing
// every token's logits during the K stream and reading them back, keep only the few tokens that
// can reach the top-k.
//
//   sample_*_kernel   a strided sample of each row -> approximate softmax statistics (M^, Z^) per
//                     head and a conservative threshold tau^ on the approximate score: a sample
//                     quantile chosen so that, four sigma low, 1.15 k tokens of the row still pass.
//   (score pass)      score_mfma_kernel in SCORE_FILTER mode: exact logits, exact softmax partials;
//                     tokens whose approximate score reaches tau^ are kept, with their exact fp32 logits,
//                     in the slots of their score chunk (no global atomics) or, once a chunk has used
//                     its slots up, in the row's overflow pool.
//   topk_cand_kernel  exact (M, Z) per head from the partials and the bound rho * tau^ on the exact
//                     score of every token that was dropped; exact scores of the candidates (in registers),
//                     bracket of the k-th score, fp64 re-evaluation and exact ranking of the few candidates around
//                     it, then an LDS bitmap turns the unordered selection into ascending positions.  The
//                     row is only accepted if its k-th score clears the bound, i.e. if no dropped token
//                     could have been selected; otherwise it is flagged and the dense stages redo it.
//   cand_split_pq_kernel + topk_cand_pq_kernel
//                     the same for one list per query head: a workgroup per row splits the row's candidates
//                     into the heads' lists, then a workgroup per (row, head) selects its list.
#include "device_utils.h"
#include "kernels.h"
#include "radix_select.h"

namespace sagekv {

namespace {

constexpr int kFastMaxG = 16;
constexpr float kHeavyShare = 0.01f;  // see sample_stats_kernel (0.3 % and 0.1 % measured worse)

// Per row: approximate softmax statistics of every head from the sampled logits; per selection list
// (one per row, or one per query head): approximate scores of the sampled candidates and a lower bound
// of their rank-th largest (within 1/2048 of their range) = the list's filter threshold.
//
// One workgroup per row: latency bound, a chain of barriers.  The sampled logits are read once: a thread holds NI
// items, an item being the logits of one head quad (4 heads, 16 bytes) of one sample slot, and always the same
// quad.  NI = 0: more items than registers (9 to 16 heads and more than 262144 candidates), they are read from memory in
// every pass.  NI = 18 spills 2 of its 128 registers (17 to 19 when this was measured) and is still ahead of that (a pass over one row of 300000 tokens x
// 8 heads 90 us and 93, two rows of 200000 x 16 heads 112 and 119).
template <int GQ, int NI>
__global__ __launch_bounds__(kTopkThreads) void sample_stats_kernel(SampleParams p) {
  __shared__ RegSelect sh;
  __shared__ float red[4][4 * GQ][kTopkWaves];

  const int row = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // per-query lists: the heads 4 blockIdx.y .. + 3, a list each; else all of them (G: heads from there on)
  const bool per_head = GQ == 1 && p.n_lists > 1;
  const int h0 = per_head ? 4 * (int)blockIdx.y : 0, G = p.geo.G - h0, rec = GQ == 1 ? p.Gs : 4 * GQ;
  const int n_slots = 64 * (p.nA + p.nB + p.nC), lo_b = 64 * p.nA, nB = 64 * p.nB;
  const int qd = tid % GQ;  // this thread's head quad
  const float* slog = p.samp_logit + (int64_t)row * n_slots * rec + 4 * qd + h0;
  if (tid == 0) {
    p.row_fail[row] = 0;
    p.ovf_count[row] = 0;
    if (row == 0) *p.n_fail = 0;
  }
  // slot of item i, and the tokens of the row it stands for (0 = outside the part its block samples)
  auto slot_of = [&](int i) { return tid / GQ + i * (kTopkThreads / GQ); };
  auto weight = [&](int s) -> float {
    const int b = s >> 6, t = s & 63;
    if (s >= n_slots) return 0.f;
    if (b < p.nA) return t < p.validA ? p.wA : 0.f;
    if (b < p.nA + p.nB) return p.wB;
    return n_slots - s <= p.validC ? p.wC : 0.f;
  };
  auto load = [&](int s) { return *reinterpret_cast<const f32x4_t*>(slog + (int64_t)s * rec); };
  f32x4_t x[NI > 0 ? NI : 1];  // logits, later exp(logit - M)
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    x[i] = f32x4_t{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (weight(slot_of(i)) > 0.f) x[i] = load(slot_of(i));
  }
  const int n_items = (n_slots * GQ + kTopkThreads - 1) / kTopkThreads;
  // f(item's four values, slot, weight) for the thread's items
  auto each = [&](auto f) {
    if (NI > 0) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float w = weight(slot_of(i));
        if (w > 0.f) f(x[i], slot_of(i), w);
      }
    } else {
      for (int i = 0; i < n_items; ++i) {
        const float w = weight(slot_of(i));
        if (w > 0.f) {
          f32x4_t v = load(slot_of(i));
          f(v, slot_of(i), w);
        }
      }
    }
  };
  // Over the lanes that share a quad, then the waves: all[] gets the heads' results (wave-uniform), v[] this thread's quad's.
  // Ends before its barrier's buffer may be written again: every call has its own.
  auto reduce = [&](float (&v)[4], float (&all)[4 * GQ], float (*buf)[kTopkWaves], auto maximum) {
    constexpr bool MAX = decltype(maximum)::value;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = wave_combine<MAX, GQ>(v[r]);
      if (lane < GQ) buf[4 * qd + r][wave] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      const float x = row_combine<MAX, 1>(buf[4 * q + (lane >> 4)][lane & 15]);
#pragma unroll
      for (int r = 0; r < 4; ++r) all[4 * q + r] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), 16 * r));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = all[r];
#pragma unroll
      for (int q = 1; q < GQ; ++q) v[r] = qd == q ? all[4 * q + r] : v[r];
    }
  };
  typedef std::integral_constant<bool, true> Max;
  typedef std::integral_constant<bool, false> Sum;

  // approximate softmax statistics: M^ = max, Z^ = sum of weight * exp(l - M^)
  float M4[4], Mall[4 * GQ], Z4[4], Zall[4 * GQ], z4[4], zall[4 * GQ], h4[4], hall[4 * GQ];
#pragma unroll
  for (int r = 0; r < 4; ++r) M4[r] = -INFINITY, Z4[r] = z4[r] = h4[r] = 0.f;
  each([&](f32x4_t& v, int, float) {
#pragma unroll
    for (int r = 0; r < 4; ++r) M4[r] = fmaxf(M4[r], v[r]);
  });
  reduce(M4, Mall, red[0], Max());
  auto expo = [&](const f32x4_t& v) {
    return f32x4_t{exp_fast(v[0] - M4[0]), exp_fast(v[1] - M4[1]), exp_fast(v[2] - M4[2]), exp_fast(v[3] - M4[3])};
  };
  each([&](f32x4_t& v, int, float w) {
    const f32x4_t e = expo(v);
#pragma unroll
    for (int r = 0; r < 4; ++r) Z4[r] += w * e[r];
    v = e;  // (registers: from here on the exponentials; from memory: a copy)
  });
  reduce(Z4, Zall, red[1], Sum());  // first estimate of Z^, refined below
  // A sampled token that would alone stand for more than 1 % of the head's mass is a heavy token, and heavy
  // tokens are rare: it is counted once, not once per token it was meant to represent.  (Attention mass sits on
  // few tokens; scaling such a token up by the sampling rate would put the head's normaliser off by a large
  // factor and the row could not be certified.  Under-counting only lets a few more candidates through.)
  each([&](f32x4_t& v, int, float w) {
    const f32x4_t e = NI > 0 ? v : expo(v);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool heavy = w * e[r] > kHeavyShare * Z4[r];
      z4[r] += (heavy ? 1.f : w) * e[r];
      h4[r] += heavy && w > 1.f ? w * e[r] : 0.f;  // a token that stands for itself alone (the sink) is no surprise
    }
  });
#pragma unroll
  for (int r = 0; r < 4; ++r) {  // (one barrier for both sums: the first goes to its buffer before the second's)
    h4[r] = wave_combine<false, GQ>(h4[r]);
    if (lane < GQ) red[3][4 * qd + r][wave] = h4[r];
  }
  reduce(z4, zall, red[2], Sum());
  float I4[4], heavy_share = 0.f;  // largest share of a head's first estimate that came from heavy tokens
#pragma unroll
  for (int q = 0; q < GQ; ++q) {
    const float x = row_combine<false, 1>(red[3][4 * q + (lane >> 4)][lane & 15]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int g = 4 * q + r;
      hall[g] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), 16 * r));
      if (g < G) heavy_share = fmaxf(heavy_share, hall[g] / Zall[g]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) I4[r] = 4 * qd + r < G ? 1.0f / z4[r] : 0.f;  // padding heads add nothing to a score
  if (tid < GQ) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * tid + r < G) {
        p.samp_stats[(int64_t)row * p.geo.G + h0 + 4 * tid + r] = make_float2(M4[r], I4[r]);
        p.heavy_thr[(int64_t)row * p.geo.G + h0 + 4 * tid + r] = heavy_logit_threshold(M4[r], z4[r]);
      }
  }
  // A heavy-tailed row (the sample met heavy tokens) has heads whose normalisers are known with
  // very different accuracy, whatever the sampler does about the heavy tokens it saw: some head
  // has others it did not see.  The summed score then needs a threshold further down: the rank
  // grows with the largest heavy share, up to twice the planned one (the candidate capacity is
  // planned for that).  Per-query lists do not need it: a head's own scale cancels.
  int rank = p.rank;
  if (!per_head) {
    const float grow = fminf(1.f, 4.f * fmaxf(0.f, heavy_share - 0.04f));
    rank = (int)((float)p.rank * (1.f + grow));
    if (rank > nB) rank = nB;
  }

  // group-sum: the threshold is on the summed approximate score; per-query: on the head's own.  Every thread takes part for
  // every item (the quads of a slot sit in adjacent lanes); -1: not a sampled candidate, or not this thread's.
  const int lists = per_head ? (G < 4 ? G : 4) : 1;
  for (int li = 0; li < lists; ++li) {
    auto score = [&](const f32x4_t& e, int s) -> float {
      float a = 0.f;
      bool mine;
      if (per_head) {
        mine = true;
#pragma unroll
        for (int r = 0; r < 4; ++r) a = li == r ? e[r] * I4[r] : a;
      } else {
        mine = qd == 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) a += e[r] * I4[r];
        if (GQ >= 2) a += __shfl_xor(a, 1);
        if (GQ >= 4) a += __shfl_xor(a, 2);
      }
      return mine && s >= lo_b && s < lo_b + nB ? a : -1.f;
    };
    uint32_t tlo = 0u, thi;
    if (rank >= 1 && p.rank <= nB) {  // rank beyond the sample: everything passes (the row is then redone densely)
      bracket_kth<false>(sh, [&](auto f) {
        if (NI > 0) {
#pragma unroll
          for (int i = 0; i < NI; ++i) f(score(x[i], slot_of(i)));
        } else {
          for (int i = 0; i < n_items; ++i) {
            const int s = slot_of(i) < n_slots ? slot_of(i) : n_slots - 1;
            f(score(expo(load(s)), slot_of(i)));
          }
        }
      }, rank, &tlo, &thi);
    }
    if (tid == 0) p.samp_tau[(int64_t)row * p.n_lists + h0 + li] = __uint_as_float(tlo);
    __syncthreads();  // the histogram is cleared for the next list
  }
}

// The row cannot be certified (reason: 1 too many / too few candidates, 2 too few reach the bound,
// 3 the k-th score does not clear the bound, 4 a band of near-ties): the dense stages redo it.  Several
// lists of a row may flag it; the count of flagged rows goes up once.
__device__ __forceinline__ void flag_row(const TopkCandParams& p, int row, int reason) {
  if (atomicExch(&p.row_fail[row], reason) == 0) atomicAdd(p.n_fail, 1);
}

// Shared state of the candidate selection kernels.
struct CandShared {
  RegSelect rs;
  float sM[kFastMaxG], sInv[kFastMaxG];
  RowStat stat[kFastMaxG];  // exact statistics of the row's heads
  double rho[kFastMaxG], flushed[kFastMaxG];
  float bound[kFastMaxG];   // per-query lists: the bound of each head's list,
  float thr[kFastMaxG];     // and the same bound as a logit of that head
  int n_list[kFastMaxG];    // per-query lists: candidates each list has kept
  int n_over;               // candidates in the row's overflow pool
  int chunk_off[1025];
};

// What a row's selection starts from, all of it asked for at once: thread t's chunk's candidate count, wave g's head's partials
// and sampled statistics.
struct RowStart {
  int raw;
  PartialLoads part;
  float2 samp;
};
__device__ __forceinline__ RowStart row_start(const TopkCandParams& p, int row) {
  const int tid = threadIdx.x, g = __builtin_amdgcn_readfirstlane(tid >> 6), G = p.geo.G, words = chunk_line_words(G);
  const float* lines = p.lines + (int64_t)row * p.n_chunks * words;
  RowStart r = {};
  if (tid < p.n_chunks) r.raw = __float_as_int(lines[(int64_t)tid * words + words - 1]);
  if (g < G) {
    r.part = load_partials(lines + 2 * g, words, p.n_chunks);
    r.samp = p.samp_stats[(int64_t)row * G + g];
  }
  return r;
}

// Exact softmax statistics of the row's heads, one wave per head, from the partials of the filtering pass; and how
// far the sampled statistics were off: rho = (exact weight) / (sampled weight).  A barrier has to follow.
__device__ __forceinline__ void exact_stats(const TopkCandParams& p, CandShared& s, int row, const RowStart& r) {
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), G = p.geo.G;
  if (g >= G) return;
  const int words = chunk_line_words(G);
  const RowStat st = merge_partials_wave(r.part, p.lines + (int64_t)row * p.n_chunks * words + 2 * g, words, p.n_chunks);
  if ((threadIdx.x & 63) == 0) {
    s.stat[g] = st;
    s.sM[g] = st.M;
    s.sInv[g] = st.invZ;
    p.stats[(int64_t)row * G + g] = st;
    s.rho[g] = exp((double)r.samp.x - (double)st.M) / (st.Z * (double)r.samp.y);
    s.flushed[g] = 0x1p-126 * (double)r.samp.y;  // the filter's exponentials come out as 0 below 2^-126
  }
}

// Candidates per score chunk -> offsets of a dense list (s.chunk_off): the chunks' own slots first, the row's overflow pool
// behind them.  Returns how many there are; -1 (workgroup-uniform): far more than planned, or fewer than k.
__device__ __forceinline__ int candidate_offsets(const TopkCandParams& p, CandShared& s, int row, int raw) {
  const int tid = threadIdx.x;
  const int v = raw < p.cap_c ? raw : p.cap_c;
  if (tid == 0) s.n_over = 0;
  __syncthreads();
  if (raw > v) atomicAdd(&s.n_over, raw - v);  // rare
  int tot;
  const int incl = block_scan_incl(v, s.rs.wave_tot, &tot);
  const int n_over = s.n_over;  // (all added before the scan's barrier)
  if (tid < p.n_chunks) s.chunk_off[tid] = incl - v;
  if (tid == 0) s.chunk_off[p.n_chunks] = tot;
  __syncthreads();
  const int n_all = tot + n_over;
  return n_all > p.cap || n_all < p.k || n_over > p.cap_o ? -1 : n_all;
}

// Records of N candidates of the dense list (those at n_all or beyond: any record).  The searches advance in step, so
// that their LDS reads overlap.
template <int N>
__device__ __forceinline__ void candidate_slots(const TopkCandParams& p, const CandShared& s, int64_t row_slots, int n_all,
                                                const int (&dj)[N], int64_t (&slot)[N]) {
  const int n_primary = s.chunk_off[p.n_chunks];
  int at[N];  // chunk with chunk_off[ch] <= dj < chunk_off[ch + 1]
#pragma unroll
  for (int u = 0; u < N; ++u) at[u] = 0;
  for (int step = 1 << (31 - __clz(p.n_chunks)); step > 0; step >>= 1) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int next = at[u] + step;
      if (s.chunk_off[next < p.n_chunks ? next : p.n_chunks] <= dj[u] && next < p.n_chunks) at[u] = next;
    }
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
    slot[u] = dj[u] >= n_all       ? row_slots
              : dj[u] >= n_primary ? row_slots + (int64_t)p.n_chunks * p.cap_c + (dj[u] - n_primary)
                                   : row_slots + (int64_t)at[u] * p.cap_c + (dj[u] - s.chunk_off[at[u]]);
}

// Sink and recent positions of a row's kept list.
__device__ __forceinline__ void write_ends(const TopkCandParams& p, int row) {
  int32_t* kept_row = p.kept_idx + (int64_t)row * (p.S + p.n_lists * p.k + p.W);
  for (int t = threadIdx.x; t < p.S; t += kTopkThreads) kept_row[t] = t;
  for (int t = threadIdx.x; t < p.W; t += kTopkThreads)
    kept_row[p.S + p.n_lists * p.k + t] = (int32_t)(p.geo.L - p.W + t);
}
// The dense stages that redo a flagged row add to its lists' first-digit histograms.
__device__ __forceinline__ void clear_histograms(const TopkCandParams& p, int row) {
  for (int b = threadIdx.x; b < kHistBins * p.n_lists; b += kTopkThreads) p.ghist[(int64_t)row * p.n_lists * kHistBins + b] = 0;
}

// The k best of a list's n_c candidates, certified against `bound`: every token outside the list scores below it.
// each(f) calls f(score, token) for the thread's candidates, -1 for none, every lane of a wave equally often.
// s.stat[g_lo .. g_hi) holds the heads' statistics; `kept` = the list's k output slots.  False: the row was flagged.
template <int DT, class Each>
__device__ __forceinline__ bool select_list(const TopkCandParams& p, CandShared& s, uint32_t* bitmap, int row, int g_lo,
                                            int g_hi, int n_c, float bound, Each each, int32_t* kept) {
  const int tid = threadIdx.x;
  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int S = p.S, k = p.k;
  const int64_t E = p.geo.L - S - p.W;
  if (n_c < k) {
    if (tid == 0) flag_row(p, row, 2);
    return false;
  }
  const int n_words = (int)((E + 31) / 32);
  for (int w = tid; w < n_words; w += kTopkThreads) bitmap[w] = 0u;
  // the k-th score's bracket, then the candidates within the band around it are re-scored in fp64 and
  // ranked exactly (score descending, index ascending); everything above the band is selected
  uint32_t tlo, thi;
  bracket_kth<true>(s.rs, [&](auto f) { each([&](float v, int) { f(v); }); }, k, &tlo, &thi);
  const float lo = __uint_as_float(tlo) * (1.0f - p.band) - kDenormSlack,
              hi = __uint_as_float(thi) * (1.0f + p.band) + kDenormSlack;
  // the row is certified only if no token outside the list can reach the band
  if (!(lo * (1.0f - p.band) > bound)) {
    if (tid == 0) flag_row(p, row, 3);
    return false;
  }
  int n_above = 0;  // wave-uniform
  each([&](float v, int tok) {
    const bool above = v > hi;
    if (above) {
      const int pos = tok - S;
      atomicOr(&bitmap[pos >> 5], 1u << (pos & 31));
    } else if (v >= 0.f && v >= lo) {
      const int t = atomicAdd(&s.rs.n_band, 1);
      if (t < kMaxBand) s.rs.band_tok[t] = tok;
    }
    n_above += __popcll(__ballot(above));
  });
  if ((tid & 63) == 0 && n_above) atomicAdd(&s.rs.n_above, n_above);
  __syncthreads();
  const int nb = s.rs.n_band, r = k - s.rs.n_above;
  if (nb > kMaxBand || r < 1 || r > nb) {  // a degenerate row of (nearly) equal scores: dense path
    if (tid == 0) flag_row(p, row, 4);
    return false;
  }
  refine_band<DT>(s.rs, nb, p.geo, p.q_last, p.K, p.pm, p.ks_problem, p.ks_head, p.ks_token, s.stat, prob, c, g_lo, g_hi);
  for (int t = tid; t < nb; t += kTopkThreads) {
    const float v = s.rs.band_v[t];
    const int tok = s.rs.band_tok[t];
    int rank = 0;
    for (int u = 0; u < nb; ++u) rank += s.rs.band_v[u] > v || (s.rs.band_v[u] == v && s.rs.band_tok[u] < tok);
    if (rank < r) atomicOr(&bitmap[(tok - S) >> 5], 1u << ((tok - S) & 31));
  }
  __syncthreads();
  bitmap_compact(bitmap, n_words, S, kept + S, k, s.rs.wave_tot);
  return true;
}

// One list per row, one workgroup per row.  Latency bound: a chain of dependent memory round trips (counts ->
// records -> the band's keys) and barriers on as many CUs as the call has rows.  So a row's candidates are read
// once and kept in registers, up to NPT per thread, their loads batched and in flight while the statistics are merged;
// selecting among scores in memory (three radix passes and a band pass, each with its own round trips, all
// of a row's keys in a few histogram bins) took 45 us for 8 rows of 128K tokens and 71 for 256, this 28 and 36, and 22
// and 27 with one barrier per reduction and the row's first loads together (row_start).
// GQ: head quads of a record.  More than NPT * 1024 candidates (peaked rows): scores and tokens go through memory.  (NPT = 24 with 9
// to 16 heads spills 7 registers; through memory it would be about even: 313 and 310 us, two rows of 400000 tokens, k = 16000.)
template <int DT, int NPT, int GQ>
__global__ __launch_bounds__(kTopkThreads) void topk_cand_kernel(TopkCandParams p) {
  constexpr int UB = GQ == 1 ? 4 : GQ == 2 ? 2 : 1;  // candidates per batch of loads
  static_assert(NPT % UB == 0, "whole batches");
  __shared__ CandShared s;
  extern __shared__ __align__(16) uint32_t bitmap[];  // one bit per eviction candidate of the row
  const int row = blockIdx.x, tid = threadIdx.x, G = p.geo.G;
  const RowStart start = row_start(p, row);
  const float tau = p.samp_tau[row];
  write_ends(p, row);
  exact_stats(p, s, row, start);
  if (p.k == 0) return;
  const int n_all = candidate_offsets(p, s, row, start.raw);
  if (n_all < 0) {
    clear_histograms(p, row);
    if (tid == 0) flag_row(p, row, 1);
    return;
  }
  const int64_t row_slots = (int64_t)row * p.slots_per_row;
  struct Batch {
    float4 lg[UB][GQ];
    int32_t tok[UB];
  };
  auto load_batch = [&](int u0, Batch& b) {
    int64_t slot[UB];
    int dj[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) dj[u] = (u0 + u) * kTopkThreads + tid;
    candidate_slots<UB>(p, s, row_slots, n_all, dj, slot);
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      b.tok[u] = p.cand_idx[slot[u]];
#pragma unroll
      for (int q = 0; q < GQ; ++q) b.lg[u][q] = *reinterpret_cast<const float4*>(p.cand_logit + (slot[u] * GQ + q) * 4);
    }
  };
  // exact fp32 score, same arithmetic and order as the dense combine stage
  auto score = [&](const float4 (&lg)[GQ]) -> float {
    float a = 0.f;
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      const float x[4] = {lg[q].x, lg[q].y, lg[q].z, lg[q].w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (q * 4 + e < G) a += exp_times(x[e] - s.sM[q * 4 + e], s.sInv[q * 4 + e]);
    }
    return a;
  };
  Batch b[2];
  load_batch(0, b[0]);
  // A token the filter dropped had approximate score < tau^, so its exact score is below rho * tau^
  // (plus what exponentials flushed to zero could hide, plus fp32 slack), rho the worst head's.
  float bound;
  {
    double rho = 0.0, fl = 0.0;
    for (int g = 0; g < G; ++g) {
      const double r = s.rho[g];
      rho = r > rho || !(r == r) ? r : rho;
      fl += s.flushed[g];
    }
    bound = (float)(rho * ((double)tau + fl) * 1.001);
  }
  int32_t* kept = p.kept_idx + (int64_t)row * (p.S + p.k + p.W);
  bool ok;
  if (n_all <= NPT * kTopkThreads) {
    float v[NPT];
    int32_t tok[NPT];
#pragma unroll
    for (int u0 = 0; u0 < NPT; u0 += UB) {
      const int n = u0 / UB;
      if (u0 + UB < NPT && (u0 + UB) * kTopkThreads < n_all) load_batch(u0 + UB, b[(n + 1) & 1]);
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        v[u0 + u] = -1.f;
        tok[u0 + u] = p.S;
        if ((u0 + u) * kTopkThreads + tid < n_all) {
          v[u0 + u] = score(b[n & 1].lg[u]);
          tok[u0 + u] = b[n & 1].tok[u];
        }
      }
    }
    ok = select_list<DT>(p, s, bitmap, row, 0, G, n_all, bound, [&](auto f) {
#pragma unroll
      for (int i = 0; i < NPT; ++i) f(v[i], tok[i]);
    }, kept);
  } else {
    float* cs = p.cand_score + (int64_t)row * p.cs_pitch;
    int32_t* ci = p.cand_pos + (int64_t)row * p.cs_pitch;
    for (int u0 = 0; u0 * kTopkThreads < n_all; u0 += UB) {
      load_batch(u0, b[0]);
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int dj = (u0 + u) * kTopkThreads + tid;
        if (dj < n_all) {
          cs[dj] = score(b[0].lg[u]);
          ci[dj] = b[0].tok[u];
        }
      }
    }
    // (a thread reads back what it wrote: no barrier needed)
    ok = select_list<DT>(p, s, bitmap, row, 0, G, n_all, bound, [&](auto f) {
      for (int j0 = 0; j0 < n_all; j0 += kTopkThreads) {
        const bool in = j0 + tid < n_all;
        f(in ? cs[j0 + tid] : -1.f, in ? ci[j0 + tid] : p.S);
      }
    }, kept);
  }
  if (!ok) clear_histograms(p, row);
}

// Per-query lists, first launch: one workgroup per row splits the row's candidates into the lists
// (a list re-reading all of the row's records costs more than everything else it does) and leaves
// each list's count and bound in list_info; count -1: nothing to select for this row.  List g gets the LOGIT of
// head g and the token of every candidate that can reach the list's bound.
// Registers are capped in both launches so that two workgroups share a CU (8 waves per SIMD): the
// kernels are chains of dependent memory round trips, a second resident workgroup fills the waits.
template <int DT>
__global__ __launch_bounds__(kTopkThreads, 8) void cand_split_pq_kernel(TopkCandParams p) {
  __shared__ CandShared s;
  const int row = blockIdx.x, tid = threadIdx.x, G = p.geo.G;
  const RowStart start = row_start(p, row);
  write_ends(p, row);
  clear_histograms(p, row);
  if (tid < kFastMaxG) s.n_list[tid] = 0;
  exact_stats(p, s, row, start);
  if (p.k == 0) return;
  const int n_all = candidate_offsets(p, s, row, start.raw);
  // A token the filter dropped for head g had approximate probability < tau^_g, so its exact one is below the
  // list's bound.  exp(x - M) / Z >= bd  <=>  x >= M + log(bd Z); lowered by more than fp32 rounding can move either side
  if (tid < G) {
    const double bd = s.rho[tid] * ((double)p.samp_tau[(int64_t)row * G + tid] + s.flushed[tid]) * 1.001;
    s.bound[tid] = (float)bd;
    s.thr[tid] = (float)((double)s.stat[tid].M + log(bd * s.stat[tid].Z) - 1e-4);
  }
  if (n_all < 0) {
    if (tid == 0) flag_row(p, row, 1);
    if (tid < G) p.list_info[(int64_t)row * G + tid] = make_float2(__int_as_float(-1), 0.f);
    return;
  }
  __syncthreads();  // s.thr
  float* cs0 = p.cand_score + (int64_t)row * p.n_lists * p.cs_pitch;
  int32_t* ci0 = p.cand_pos + (int64_t)row * p.n_lists * p.cs_pitch;
  const int64_t row_slots = (int64_t)row * p.slots_per_row;
  for (int d0 = 0; d0 < n_all; d0 += 4 * kTopkThreads) {
    int64_t slot[4];
    int dj[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) dj[u] = d0 + u * kTopkThreads + tid;
    candidate_slots<4>(p, s, row_slots, n_all, dj, slot);
    int32_t ti[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) ti[u] = p.cand_idx[slot[u]];
    // four heads at a time: their logits are one 16-byte load per candidate
    for (int g4 = 0; g4 < G; g4 += 4) {
      float4 lg[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        lg[u] = *reinterpret_cast<const float4*>(p.cand_logit + slot[u] * p.Gs + g4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int g = g4 + e;
        if (g >= G) break;  // workgroup-uniform
        float* cs = cs0 + (int64_t)g * p.cs_pitch;
        int32_t* ci = ci0 + (int64_t)g * p.cs_pitch;
        const float thr = s.thr[g];
        float x[4];
        unsigned long long bal[4];
        int n_wave = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[u] = e == 0 ? lg[u].x : e == 1 ? lg[u].y : e == 2 ? lg[u].z : lg[u].w;
          bal[u] = __ballot(dj[u] < n_all && x[u] >= thr);
          n_wave += __popcll(bal[u]);
        }
        if (n_wave) {  // wave-uniform
          int base = 0;
          if ((tid & 63) == 0) base = atomicAdd(&s.n_list[g], n_wave);
          base = __shfl(base, 0);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if ((bal[u] >> (tid & 63)) & 1ull) {
              const int pos = base + __popcll(bal[u] & ((1ull << (tid & 63)) - 1ull));
              cs[pos] = x[u];
              ci[pos] = ti[u];
            }
            base += __popcll(bal[u]);
          }
        }
      }
    }
  }
  __syncthreads();
  if (tid < G) p.list_info[(int64_t)row * G + tid] = make_float2(__int_as_float(s.n_list[tid]), s.bound[tid]);
}

// Per-query lists, second launch: one workgroup per (row, head); a list's candidates in registers, up to NPT per thread.
template <int DT, int NPT>
__global__ __launch_bounds__(kTopkThreads, 8) void topk_cand_pq_kernel(TopkCandParams p) {
  __shared__ CandShared s;
  extern __shared__ __align__(16) uint32_t bitmap[];
  const int list = blockIdx.x, tid = threadIdx.x, G = p.geo.G;
  const int row = list / G, g = list % G;
  const float2 info = p.list_info[list];
  const RowStat st = p.stats[(int64_t)row * G + g];
  const int n_c = __float_as_int(info.x);
  if (n_c < 0) return;
  float* cs = p.cand_score + (int64_t)list * p.cs_pitch;
  const int32_t* ci = p.cand_pos + (int64_t)list * p.cs_pitch;
  if (tid == 0) s.stat[g] = st;  // (select_list has barriers before it is read)
  int32_t* kept = p.kept_idx + (int64_t)row * (p.S + G * p.k + p.W) + g * p.k;
  if (n_c <= NPT * kTopkThreads) {
    float v[NPT];
    int32_t tok[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const int j = u * kTopkThreads + tid;
      v[u] = -1.f;
      tok[u] = p.S;
      if (j < n_c) {
        v[u] = cs[j];
        tok[u] = ci[j];
      }
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u)  // exact fp32 scores, same arithmetic as the dense stages
      if (u * kTopkThreads + tid < n_c) v[u] = exp_times(v[u] - st.M, st.invZ);
    select_list<DT>(p, s, bitmap, row, g, g + 1, n_c, info.y, [&](auto f) {
#pragma unroll
      for (int i = 0; i < NPT; ++i) f(v[i], tok[i]);
    }, kept);
  } else {
    for (int j = tid; j < n_c; j += kTopkThreads) cs[j] = exp_times(cs[j] - st.M, st.invZ);
    select_list<DT>(p, s, bitmap, row, g, g + 1, n_c, info.y, [&](auto f) {
      for (int j0 = 0; j0 < n_c; j0 += kTopkThreads) {
        const bool in = j0 + tid < n_c;
        f(in ? cs[j0 + tid] : -1.f, in ? ci[j0 + tid] : p.S);
      }
    }, kept);
  }
}

}  // namespace

template <int GQ>
void launch_sample_stats(const SampleParams& p, unsigned rows, unsigned parts, int items, hipStream_t s) {
  const dim3 grid(rows, parts), block(kTopkThreads);
  if (items <= 3) {
    hipLaunchKernelGGL((sample_stats_kernel<GQ, 3>), grid, block, 0, s, p);
  } else if (items <= 6) {
    hipLaunchKernelGGL((sample_stats_kernel<GQ, 6>), grid, block, 0, s, p);
  } else if (items <= 9 || GQ == 1) {  // (one quad: the largest sample is 9 items per thread)
    hipLaunchKernelGGL((sample_stats_kernel<GQ, 9>), grid, block, 0, s, p);
  } else if constexpr (GQ > 1) {
    if (items <= 18)
      hipLaunchKernelGGL((sample_stats_kernel<GQ, 18>), grid, block, 0, s, p);
    else
      hipLaunchKernelGGL((sample_stats_kernel<GQ, 0>), grid, block, 0, s, p);
  }
}

hipError_t launch_sample(const SampleParams& p, hipStream_t s) {
  const int rows = p.geo.n_problems * p.geo.Hkv;
  if (p.geo.dtype != DT_BF16 || p.geo.G > kFastMaxG || p.nB * 64 > 8192) return hipErrorInvalidValue;
  hipError_t e = launch_sample_logits(p, s);
  if (e != hipSuccess) return e;
  // One workgroup per row; with several lists per row one for every four of them, as the thresholds are found one after the other (whole pass,
  // us, one per row and so: 112 rows x 128K x 7 lists 841 and 822, 64 x 32K x 7 247 and 227, 64 x 32K x 4 185 and 184).
  const int gq = p.n_lists > 1 ? 1 : p.Gs / 4 > 2 ? 4 : p.Gs / 4;  // head quads of a record that a workgroup takes, as a power of two
  const unsigned parts = p.n_lists > 1 ? (unsigned)(p.geo.G + 3) / 4 : 1;
  const int items = (64 * (p.nA + p.nB + p.nC) * gq + kTopkThreads - 1) / kTopkThreads;
  if (gq == 1) launch_sample_stats<1>(p, (unsigned)rows, parts, items, s);
  else if (gq == 2) launch_sample_stats<2>(p, (unsigned)rows, parts, items, s);
  else launch_sample_stats<4>(p, (unsigned)rows, parts, items, s);
  return hipGetLastError();
}

template <int NPT, int GQ>
hipError_t launch_topk_cand_t(const TopkCandParams& p, unsigned rows, size_t lds, hipStream_t s) {
  static uint64_t done = 0;
  const hipError_t e = allow_dynamic_lds((const void*)topk_cand_kernel<DT_BF16, NPT, GQ>, 128 * 1024, &done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((topk_cand_kernel<DT_BF16, NPT, GQ>), dim3(rows), dim3(kTopkThreads), lds, s, p);
  return hipGetLastError();
}
template <int NPT>
hipError_t launch_topk_cand_n(const TopkCandParams& p, unsigned rows, size_t lds, hipStream_t s) {
  return p.Gs == 4   ? launch_topk_cand_t<NPT, 1>(p, rows, lds, s)
         : p.Gs == 8 ? launch_topk_cand_t<NPT, 2>(p, rows, lds, s)
                     : launch_topk_cand_t<NPT, 4>(p, rows, lds, s);
}
template <int NPT>
hipError_t launch_topk_pq_t(const TopkCandParams& p, unsigned lists, size_t lds, hipStream_t s) {
  static uint64_t done = 0;
  const hipError_t e = allow_dynamic_lds((const void*)topk_cand_pq_kernel<DT_BF16, NPT>, 128 * 1024, &done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((topk_cand_pq_kernel<DT_BF16, NPT>), dim3(lists), dim3(kTopkThreads), lds, s, p);
  return hipGetLastError();
}

hipError_t launch_topk_cand(const TopkCandParams& p, hipStream_t s) {
  const unsigned rows = (unsigned)(p.geo.n_problems * p.geo.Hkv);
  const int64_t E = p.geo.L - p.S - p.W;
  // the bitmap (one bit per candidate, up to 128 KiB) sits next to about 30 KiB of static LDS; a CU has 160 KiB
  const size_t lds = (size_t)((E + 31) / 32) * 4;
  if (lds > 128 * 1024 || p.geo.G > kFastMaxG) return hipErrorInvalidValue;
  // registers per thread for the candidates a list is expected to have (see TopkCandParams::expect): a row that has
  // more than that goes through memory, at about the pace that all of them had before
  if (p.n_lists > 1) {
    hipLaunchKernelGGL(cand_split_pq_kernel<DT_BF16>, dim3(rows), dim3(kTopkThreads), 0, s, p);
    const unsigned lists = rows * (unsigned)p.n_lists;
    return p.expect <= 4 * kTopkThreads ? launch_topk_pq_t<4>(p, lists, lds, s) : launch_topk_pq_t<12>(p, lists, lds, s);
  }
  return p.expect <= 4 * kTopkThreads    ? launch_topk_cand_n<4>(p, rows, lds, s)
         : p.expect <= 12 * kTopkThreads ? launch_topk_cand_n<12>(p, rows, lds, s)
                                         : launch_topk_cand_n<24>(p, rows, lds, s);
}

}  // namespace sagekv
