// C ABI of the library: argument checks, workspace layout, launch order.
#include "../../include/sagekv.h"
#include "../../include/sagekv_bench.h"

#include <math.h>
#include <stdint.h>

#include <mutex>
#include <vector>

#include "kernels.h"

using namespace sagekv;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Relative half-width of the band around the coarse k-th score whose members are re-scored in
// fp64.  fp32 scores carry a relative error of a few 1e-6 at most with logits of ordinary size (dot products of <= 128
// exact products summed pairwise, one exp, one multiply per head; on the one-sweep path also the heads' normalisers, whose heavy terms
// are put right only for the fp64 scores), so 2^-12 leaves two orders
// of magnitude of margin while the band still holds only a handful of candidates per row.  Dot products and normalisers
// are off in proportion to the logits, about 1.2e-7 |l| each: at |l| = 500 both together reach half of the band, which is what two scores
// may be off by towards each other.  (Offsets to +-1000, queries x 1 to 70, 33 thousand calls against fp64: no list differed by more than 1e-6 on this route.)
constexpr float kBand = 1.0f / 4096.0f;

constexpr int64_t kFillScores = 256, kFill = 512;  // see score_chunk
constexpr int64_t kShortFrom = 8192, kExactFill = 224;  // see shortlist_plan

// Sizes of the fast (pre-filtered) eviction path for one descriptor; ok = the path applies.
struct FastPlan {
  bool ok;
  int nA, nB, nC, validA, validC, rank, cap, Gs;
  int expect;  // candidates a list usually has at most
  int cap_c;  // candidate slots each score chunk owns; what does not fit goes to the row's overflow pool (cap slots)
  int64_t stepB;
  float wA, wB, wC;
};

// Tokens one workgroup of the first pass over K covers: 1024, less where the call is too small for that to fill the
// chip.  At most 1024 chunks per row (the candidate selection gives each a thread).
// At least 512 workgroups, two per CU (filtering pass over 8 rows of 32768 tokens: 22 us with 512 workgroups of 512
// tokens, 24.7 with 256 of 1024, 27 with 1024 of 256; as the pass is now 18.7 with 512 and 20.3 with 1024; a whole pass of the one-sweep path
// over 8 rows x 32K 37.3 with 512 and 38.1 with 256, 32 x 8192 43.2 and 44.7).  256 do for a dense call that returns every score, whose
// statistics are merged by one workgroup per row (8 rows of 30000 tokens x 4 heads: 65.3 us with chunks of 512 tokens, 67.6 with 256).
int score_chunk(const sagekv_select_desc* d, int64_t fill) {
  const int64_t rows = (int64_t)d->n_problems * d->n_kv_heads;
  int chunk = d->dtype == SAGEKV_BF16 ? kScoreChunk : 512;
  while (chunk > 256 && rows * ((d->L + chunk - 1) / chunk) < fill && (d->L + chunk / 2 - 1) / (chunk / 2) <= 1024) chunk /= 2;
  return chunk;
}

FastPlan fast_plan(const sagekv_select_desc* d) {
  FastPlan f = {};
  const int G = d->n_q_heads / d->n_kv_heads;
  const int64_t E = d->L - d->n_sink - d->n_recent;
  f.ok = d->dtype == SAGEKV_BF16 && G <= 16 && d->k > 0 && E <= 1048576 && d->L <= 1024 * (int64_t)kScoreChunk &&
         !(d->flags & SAGEKV_SELECT_DENSE);
  if (!f.ok) return f;
  const int lists = d->head_mode == SAGEKV_HEADS_PER_QUERY ? G : 1;
  // sample: runs of 16 consecutive tokens, about 1/64 of the candidates (64 to 512 runs); the
  // sample is read from HBM on top of the full pass over K, so its share is kept small
  int64_t nb = E / 4096;
  f.nB = (int)(nb < 16 ? 16 : (nb > 128 ? 128 : nb));
  f.stepB = ((E - 16) << 16) / (4 * f.nB - 1);  // between 16-token runs
  f.nA = d->n_sink > 0 ? 1 : 0;
  f.validA = d->n_sink < 64 ? d->n_sink : 64;
  // the recent window is where a trained model puts much of its attention: up to its last 512 tokens
  // are all sampled
  f.nC = d->n_recent >= 512 ? 8 : (d->n_recent + 63) / 64;
  f.validC = d->n_recent < 64 * f.nC ? d->n_recent : 64 * f.nC;
  f.wA = f.nA ? (float)d->n_sink / (float)f.validA : 0.f;
  f.wB = (float)E / (float)(64 * f.nB);
  f.wC = (float)d->n_recent / (float)f.validC;
  // Threshold = the rank-th largest approximate score among the n sampled candidates.  About
  // rank * E / n tokens of the row exceed it, with relative sigma 1/sqrt(rank); the rank is the
  // smallest whose 4-sigma low side still keeps (1 + margin) k tokens: rank - 4 sqrt(rank) >=
  // (1 + margin) k n / E.  The margin covers the error of the sampled softmax normalisers; the
  // bound on a dropped token's score takes the worst head's, so it grows with the group size
  // (15 % at G = 4, 20 % at G = 8, 46 % at G = 16: measured, a redone row costs far more than the
  // extra candidates).
  const double margin = 0.10 + 0.0125 * (double)G + (G > 8 ? 0.02 * (double)(G - 8) : 0.0);
  const double r0 = (1.0 + margin) * (double)d->k * (double)(64 * f.nB) / (double)E;
  const double x = 2.0 + sqrt(4.0 + r0);
  f.rank = (int)ceil(x * x);
  f.expect = (int)(((double)f.rank + 4.0 * sqrt((double)f.rank)) * (double)f.wB);
  // Room for the candidates: about rank * wB tokens pass a list's threshold, 4 sigma high side
  // (rank + 4 sqrt(rank)) * wB; per-query lists share one candidate list per row (their union).
  // (a heavy-tailed row may raise its rank to twice the planned one, see sample_stats_kernel)
  const double high = (2.0 * (double)f.rank + 4.0 * sqrt(2.0 * (double)f.rank)) * (double)f.wB;
  const double planned = 2.5 * (double)d->k;
  int64_t cap = (int64_t)ceil(high > planned ? high : planned) * lists + 4096;
  f.cap = (int)(cap < E ? cap : E);
  // k is a large share of the row: the filter would be expected to keep half of it or more
  if (2.0 * lists * (double)f.rank * (double)f.wB > (double)E || 5 * (int64_t)d->k * lists > E) {
    f.ok = false;
    return f;
  }
  f.Gs = G <= 4 ? 4 : G <= 8 ? 8 : 16;  // whole, aligned 16-byte quads, a power of two of them
  // A chunk's own slots: twice the candidates an average chunk is expected to keep (rank * wB tokens
  // per list over the row's chunks), so that only chunks where the candidates crowd (a needle
  // cluster, the tokens next to the recent window of a trained model) reach into the overflow pool.
  const int chunk = score_chunk(d, kFill);
  const int64_t n_chunks = (d->L + chunk - 1) / chunk;
  const double per_chunk = (double)f.rank * (double)f.wB * lists / (double)n_chunks;
  int cap_c = 32;
  while (cap_c < 2.0 * per_chunk + 16.0 && cap_c < chunk) cap_c *= 2;
  f.cap_c = cap_c;
  return f;
}

// Rows of the one-sweep dense path whose selection is spread over many workgroups (shortlist_kernel); ok = that applies.
struct ShortlistPlan {
  bool ok;
  int n_parts, part_tokens, n_exact, first_run, n_runs, rank, expect;
  int64_t step;
};

ShortlistPlan shortlist_plan(const sagekv_select_desc* d) {
  ShortlistPlan s = {};
  const int64_t E = d->L - d->n_sink - d->n_recent;
  const int64_t lists = (int64_t)d->n_problems * (d->head_mode == SAGEKV_HEADS_PER_QUERY ? d->n_q_heads : d->n_kv_heads);
  auto parts = [&](int tokens) { return (d->L + tokens - 1) / tokens; };
  s.part_tokens = lists * (parts(kShortTokens) + 1) <= 256 ? kShortTokens : 2 * kShortTokens;  // one workgroup per CU
  s.n_parts = (int)parts(s.part_tokens);
  // The heads' heavy terms by as many workgroups as there are CUs for: with logits that share an offset one has to look through a whole row's (8 rows x
  // 32K x 16 heads, N(60, 1), with raised thresholds: 136 us with one, 55 so).  Not on all 256: the others would start later (32 rows x 32K x 4
  // heads, N(0, 1): 84 us with 224 workgroups in all, 87.5 with 256).
  const int64_t heads = d->head_mode == SAGEKV_HEADS_PER_QUERY ? 1 : d->n_q_heads / d->n_kv_heads, free_cus = kExactFill / lists - s.n_parts;
  s.n_exact = (int)(free_cus < 1 ? 1 : free_cus < heads ? free_cus : heads);
  if (d->k < 1 || E > kShortMax || d->L > (int64_t)kShortParts * kShortTokens) return s;
  // the sample: runs of 16 tokens, aligned (64 bytes of a head's logits), all of them candidates
  const int64_t r0 = ((int64_t)d->n_sink + 15) / 16, r1 = (d->L - d->n_recent) / 16;
  const int64_t runs = r1 > r0 ? r1 - r0 : 0;
  s.first_run = (int)r0;
  s.n_runs = (int)(runs < kShortRuns ? runs : kShortRuns);
  s.step = s.n_runs ? (runs << 16) / s.n_runs : 0;
  // Threshold = the rank-th largest of the n sampled scores.  About rank * E / n tokens of the row reach it, with a relative
  // sigma of sqrt((1 - n / E) / rank); the rank is the smallest whose 4-sigma low side keeps 1.1 k tokens (scores of neighbours are
  // not quite independent).
  const double n = 16.0 * s.n_runs, f = n / (double)E;
  const double mean = 1.1 * (double)d->k * f, c = 4.0 * sqrt(f < 1.0 ? 1.0 - f : 0.0);
  const double x = 0.5 * (c + sqrt(c * c + 4.0 * mean));
  s.rank = (int)ceil(x * x);
  double most = (double)E;
  if (s.rank < n) {
    most = ((double)s.rank + c * sqrt((double)s.rank)) / f;
    if (most > (double)E) most = (double)E;
  } else {
    s.rank = 0;  // everything passes
  }
  s.expect = (int)ceil(most);
  // Registers of the selecting workgroup, and longer rows than one workgroup selects from faster (row_select_kernel): from 8192 tokens on, more with fewer
  // heads a list,
  // while the first launch has a CU for every workgroup, us, row_select_kernel and this: 8 rows x 8192 28.9 29.9, x 10000 32.7 30.6, x 24000
  // 46.9 35.6, 32 x 24000 81 71, 64 x 24000 180 180, 128 x 16384 160 170 (4 heads); 8 rows of 64 dims, fp32, 1 head x 9000 22.2 24.4, x 12000 23.0 25.1, x
  // 16000 25.7 25.2, 2 heads x 12000 25.1 27.2, x 16000 28.3 27.2, 3 x 9000 26.1 27.6, x 12000 28.4 27.9, 4 x 9000 28.2 28.9, x 12000 30.8 29.8, bf16 1 x 12000
  // 22.9 23.5, x 16000 23.9 23.3, 2 x 9000 23.3 23.2, x 16000 24.9 24.6; from kRowSelectMax tokens on, up to the logits of
  // 256 rows x 32K x 4 heads, wherever the pre-filtered path is the alternative (few_rows), else as select_layout says.
  const int64_t from = heads == 1 ? 14336 : heads == 2 ? 12288 : heads == 3 ? 10240 : kShortFrom;
  s.ok = s.expect <= 16 * 1024 &&
         (d->L > kRowSelectMax ? 4 * (int64_t)d->n_problems * d->n_q_heads * d->L <= 128ll << 20
                               : d->L > from && lists * (s.n_parts + 1) <= 256);
  return s;
}

struct SelectLayout {
  // small: the pre-filtered path applies to the descriptor; rows it cannot certify (and calls that
  // ask for every score) take the two-sweep dense path, which needs no logit scratch.  The layout is that of the path that one_sweep says.
  bool small;
  size_t logits /* one_sweep */, scores, partials /* one_sweep: ChunkPartial, else the chunks' lines */, stats, ghist, total;
  // pre-filtered path (n_fail: whenever small)
  size_t samp_logit, samp_stats, heavy_thr, samp_tau, list_info, ovf_count, cand_idx, cand_logit, cand_score, cand_pos,
      row_fail, n_fail;
  // one-sweep dense path, many workgroups per row
  size_t short_cand, short_count, short_tau, flags;
  int64_t slots_per_row, cs_pitch;
  FastPlan fast;
  ShortlistPlan list;
  bool one_sweep;  // the one-sweep dense path (small: for a call of few rows),
  bool shortlist;  // with the shortlist launches
  int64_t Lp;
  int n_chunks, chunk, rows, G, n_lists;
};

bool check_select(const sagekv_select_desc* d, sagekv_status* st) {
  *st = SAGEKV_ERR_INVALID_ARG;
  if (!d) return false;
  if (d->n_problems < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads) return false;
  if (d->L < 1 || d->L > 0x7FFFFFF0ll) return false;
  if (d->n_sink < 0 || d->n_recent < 1 || d->k < 0) return false;
  if ((int64_t)d->n_sink + d->n_recent + d->k > d->L) return false;
  if (d->head_mode != SAGEKV_HEADS_GROUP_SUM && d->head_mode != SAGEKV_HEADS_PER_QUERY) return false;
  const int64_t lists = d->head_mode == SAGEKV_HEADS_PER_QUERY ? d->n_q_heads / d->n_kv_heads : 1;
  if ((int64_t)d->compact_capacity < (int64_t)d->n_sink + d->n_recent + lists * d->k) return false;
  if (d->flags & ~(uint32_t)SAGEKV_SELECT_DENSE) return false;
  *st = SAGEKV_ERR_UNSUPPORTED;
  if (d->dtype != SAGEKV_BF16 && d->dtype != SAGEKV_F32) return false;
  if (d->head_dim != 64 && d->head_dim != 128) return false;
  if (d->n_q_heads / d->n_kv_heads > 64) return false;
  // rows (and selection lists) index one grid dimension of the launches
  if ((int64_t)d->n_problems * d->n_kv_heads * lists > 65535) return false;
  const int epl = d->dtype == SAGEKV_BF16 ? 8 : 4;  // 16-byte alignment of every token row
  const int64_t strides[6] = {d->k_stride_problem, d->k_stride_head, d->k_stride_token,
                              d->v_stride_problem, d->v_stride_head, d->v_stride_token};
  for (int i = 0; i < 6; ++i)
    if (strides[i] < 0 || strides[i] % epl) return false;
  if (d->k_stride_token < d->head_dim || d->v_stride_token < d->head_dim) return false;
  *st = SAGEKV_OK;
  return true;
}

// Calls that the pre-filtered path could serve, but the one-sweep dense path serves faster: its logits (`bytes`) stay in the caches between
// its passes, and it has two launches in between instead of five.  Whole passes, us, pre-filtered and dense:
//   rows x tokens, heads     MB                      rows x tokens, heads     MB
//   8 x 8K, 4                 1    43.5   28.9       64 x 2K, 4                2    40.7   22.8
//   8 x 32K, 4                4    49.8   37.3       256 x 4K, 4              17     118     92
//   4 x 128K, 7              15    81.2   66.0       256 x 8K, 4              34     188    171
//   8 x 128K, 4              17    92.2   86.8       512 x 8K, 4              67     325    315
//   32 x 32K, 4              17    93.2   88.3       1024 x 8K, 4            134     635    635
//   16 x 98304, 4            25     109    110       512 x 8K, 7             117     344    348
//   8 x 256K, 4              34     139    146       8 x 32K, 16              21    88.6   65.3
//   16 x 64K, 4, 64 dims     17    59.1   53.3       32 x 32K, 7              29    92.0   88.7
//   16 x 128K, 4, 64 dims    34    78.8   89.9       64 x 20000, 7            36     110    110
//   per-query lists: 32 x 32K, 7 29 160 126, 64 x 32K, 7 59 246 243, 32 x 32K, 4 17 116 104, 64 x 32K, 4 34 186 187
// Rows too long for row_select_kernel with few heads have more keys and more workgroups of the shortlist's first launch in as many bytes of logits:
//   64 x 40000, 1             10     140    139       40 x 40000, 2 (64 dims) 13 66.0 64.1      24 x 50000, 4 (64 dims) 19 57.3 58.6
//   8 x 400000, 1             13     167    171       32 x 65536, 2            17     117    120
//   24 x 92424, 1, 64 dims     9    74.6   76.2       40 x 54961, 2            18     122    128
bool few_rows(const sagekv_select_desc* d, int G, bool per_query) {
  const double mb = 4e-6 * (double)d->n_problems * d->n_q_heads * (double)d->L;
  if (d->L <= kShortFrom) return mb <= 68.0;
  if (G > 4 || per_query) return mb <= 30.0;
  if (d->L <= kRowSelectMax) return mb <= 20.0;
  return mb <= (G == 1 ? 8.5 : G == 2 ? 13.0 : 18.5);
}

// Workspace layout.  Descriptors the pre-filtered path cannot serve get the one-sweep dense path's
// scratch (every token's fp32 logits: G * 4 bytes per token).  All others get: a score row per
// selection list (used by the rows that have to be redone, and by calls that ask for scores_out
// through the caller's array instead), the candidate records (a few slots per score chunk and an
// overflow pool per row) and small per-row arrays.  The dense candidate arrays of the final
// selection live in the list's score row while it is not in use.
// few: a call that calls for it (few_rows, rows too long for row_select_kernel) gets the one-sweep dense path with the shortlist launches
// and their scratch; without, the paths that make do with less.
SelectLayout select_layout(const sagekv_select_desc* d, bool own_scores, bool few) {
  SelectLayout l = {};
  l.rows = d->n_problems * d->n_kv_heads;
  l.G = d->n_q_heads / d->n_kv_heads;
  l.n_lists = d->head_mode == SAGEKV_HEADS_PER_QUERY ? l.G : 1;
  l.Lp = (d->L + 3) / 4 * 4;
  l.fast = fast_plan(d);
  l.small = l.fast.ok;
  l.list = shortlist_plan(d);
  few = few && own_scores;
  l.one_sweep = !l.small || (few && few_rows(d, l.G, l.n_lists > 1) && (l.list.ok || d->L <= kRowSelectMax));
  // Calls the pre-filtered path does not serve, more than kRowSelectMax tokens: up to two workgroups of the first launch per CU, one with
  // 64 dims.  Whole passes, us, statistics, combine and top-k in launches of their own and this, by workgroups: 7 per-query lists of 27000 tokens, 280
  // 58.5 54.2, 420 75.8 68.0, 1680 213 217, 4200 512 523; 4 lists of 30000, 480 119 115, 3840 787 797; rows of 32000 x 4 heads, 320 213 210, 640 386
  // 388; of 64 dims, 320 128 132, 500 180 183, 600 211 218.
  const int64_t first = (int64_t)l.rows * l.n_lists * (l.list.n_parts + 1);
  l.shortlist = few && l.list.ok && l.one_sweep && (l.small || d->L <= kRowSelectMax || first <= (d->head_dim == 64 ? 256 : 512));
  l.chunk = score_chunk(d, l.one_sweep && !few ? kFillScores : kFill);
  l.n_chunks = (int)((d->L + l.chunk - 1) / l.chunk);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes);
    return at;
  };
  const size_t rows = (size_t)l.rows;
  l.n_fail = take(l.small ? sizeof(int) : 0);  // first: at the same place whatever path a call takes
  l.logits = take(l.one_sweep ? rows * l.n_chunks * l.G * l.chunk * sizeof(float) : 0);
  l.partials = take(rows * l.n_chunks * (l.one_sweep ? l.G * sizeof(ChunkPartial) : chunk_line_words(l.G) * sizeof(float)));
  l.stats = take(rows * l.G * sizeof(RowStat));
  l.ghist = take(rows * l.n_lists * kHistBins * sizeof(int));
  bool cs_in_scores = false;
  const size_t lists = rows * l.n_lists;
  if (l.small && l.one_sweep) l.flags = take(lists * sizeof(int));
  if (l.shortlist) {
    l.short_cand = take(lists * l.list.n_parts * l.list.part_tokens * sizeof(uint2));
    l.short_count = take(lists * l.list.n_parts * sizeof(int));
    l.short_tau = take(lists * sizeof(float));
  }
  if (!l.one_sweep) {
    const FastPlan& f = l.fast;
    const size_t ns = (size_t)64 * (f.nA + f.nB + f.nC);
    l.samp_logit = take(rows * ns * f.Gs * sizeof(float));
    l.samp_stats = take(rows * l.G * sizeof(float2));
    l.heavy_thr = take(rows * l.G * sizeof(float));
    l.samp_tau = take(rows * l.n_lists * sizeof(float));
    l.list_info = take(rows * l.n_lists * sizeof(float2));
    l.slots_per_row = ((int64_t)l.n_chunks * f.cap_c + f.cap + 31) / 32 * 32;  // a chunk's slots (cap_c >= 32) are whole lines
    l.ovf_count = take(rows * sizeof(int));
    l.cand_idx = take(rows * l.slots_per_row * sizeof(int32_t));
    l.cand_logit = take(rows * l.slots_per_row * f.Gs * sizeof(float));
    l.row_fail = take(rows * sizeof(int));
    cs_in_scores = 2 * (int64_t)f.cap <= l.Lp;
    l.cs_pitch = cs_in_scores ? l.Lp : f.cap;
    if (!cs_in_scores) {
      l.cand_score = take(rows * l.n_lists * f.cap * sizeof(float));
      l.cand_pos = take(rows * l.n_lists * f.cap * sizeof(int32_t));
    }
  }
  // last, so that no other offset depends on whether the caller brought its own score rows
  // (one-sweep rows whose selection holds its scores in registers need none)
  own_scores = own_scores && (!l.one_sweep || l.shortlist || d->L > kRowSelectMax);
  l.scores = take(own_scores ? rows * l.n_lists * l.Lp * sizeof(float) : 0);
  if (cs_in_scores) {  // the first half of a list's score row: exact scores, the second: token indices
    l.cand_score = l.scores;
    l.cand_pos = l.scores + (size_t)l.fast.cap * sizeof(float);
  }
  l.total = off;
  return l;
}

int decode_lists(const sagekv_decode_desc* d) {
  return d->head_mode == SAGEKV_HEADS_PER_QUERY ? d->n_q_heads / d->n_kv_heads : 1;
}

bool check_decode(const sagekv_decode_desc* d, sagekv_status* st) {
  *st = SAGEKV_ERR_INVALID_ARG;
  if (!d) return false;
  if (d->n_problems < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads) return false;
  if (d->n_sink < 0 || d->n_recent < 1 || d->k < 0) return false;
  if (d->head_mode != SAGEKV_HEADS_GROUP_SUM && d->head_mode != SAGEKV_HEADS_PER_QUERY) return false;
  if ((int64_t)d->compact_capacity < (int64_t)d->n_sink + d->n_recent + (int64_t)decode_lists(d) * d->k) return false;
  *st = SAGEKV_ERR_UNSUPPORTED;
  if ((int64_t)d->n_problems * d->n_kv_heads > 65535) return false;  // rows index one grid dimension
  if (d->dtype != SAGEKV_BF16 && d->dtype != SAGEKV_F32) return false;
  if (d->head_dim != 64 && d->head_dim != 128) return false;
  *st = SAGEKV_OK;
  return true;
}

struct DecodeLayout {
  size_t part_ml, part_acc, total;
  int max_splits, rows, G;
};

// Splits per row.  With about one row per CU or more, a single 8-wave workgroup per row fills
// the chip and needs no merge launch; otherwise enough workgroups to fill 256 CUs several times
// over (fp32: see slices_f32), at least 128 tokens each.  Short rows are not worth the merge launch:
// bf16 up to 256 tokens, a single pass (8 rows x 4 heads x 256 tokens 9.2 us split, 7.7 whole; 4 rows x 7 heads 8.7 and 7.7; before
// the slice kernel had its present form 10.3 and 8.4, 9.6 and 8.2, and at
// 512 tokens 10.5 and 11.0, 10.45 and 10.5), fp32 up to 384 tokens of head_dim 64, 192 of 128 (2 rows x 2 heads x 300 and 400 tokens 9.5 and 9.3 us
// split, 7.2 and 8.1 whole, 512 even; 4 rows x 4 heads x 512 10.0 and 11.0; head_dim 128, 160 tokens: 8 rows x 4 heads 10.4 and 8.0, 4 x 7
// 12.2 and 10.1, 256 tokens 10.5 and 9.7, 12.2 and 12.5).
constexpr int kFillDecode = 2048;

// fp32: a slice of 128 tokens is one block for each of its workgroup's waves, with nothing in flight while they start and merge.  So one
// workgroup per CU of 8 waves (128 dims), two of 4 (64 dims), of as many tokens as that takes; where many rows do not divide them, the slices whose
// rounds of workgroups, each as long as its blocks and one and a half more, are the shortest in all.  us, slices as for bf16 and so: 64 rows x 2048 tokens of 128 dims
// 31.8 and 25.4 (1 head), 34 and 26 (2), 41.8 and 31 (7), 16 x 4096 18.8 and 16 (1), 150 x 4000 143.6 and 123.7 (7; with 2 slices 161), of 64 dims
// 64 x 2048 x 7 heads 24.6 and 20.7, 16 x 8000 x 1 19 and 16, 100 x 3000 x 5 80 and 42.
int slices_f32(int rows, int len, int head_dim) {
  const int fill = head_dim == 128 ? 256 : 512, first = fill / rows > 1 ? fill / rows : 1;
  int best = first, least = 0x7FFFFFFF;
  if (20 * rows <= 3 * fill) return first;  // they leave 15 % of the workgroups idle at most
  for (int n = first; n < 4 * first + 4; ++n) {
    const int blocks = (len + 128 * n - 1) / (128 * n), cost = (rows * n + fill - 1) / fill * (2 * blocks + 3);
    if (cost < least) best = n, least = cost;
  }
  return best;
}

int splits_for(int rows, int len, int dtype, int head_dim, int want) {
  if (rows >= kWholeRows) return 1;
  if (dtype == SAGEKV_BF16 ? len <= 256 : (int64_t)len * head_dim <= 384 * 64) return 1;
  int most = (len + 127) / 128;
  int n = want < most ? want : most;
  return n < 1 ? 1 : n;
}

DecodeLayout decode_layout(const sagekv_decode_desc* d) {
  DecodeLayout l;
  l.rows = d->n_problems * d->n_kv_heads;
  l.G = d->n_q_heads / d->n_kv_heads;
  // (room for kFillDecode workgroups, whatever a call uses: scratch sizes are part of the interface)
  l.max_splits = splits_for(l.rows, d->compact_capacity, d->dtype, d->head_dim, (kFillDecode + l.rows - 1) / l.rows);
  size_t off = 0;
  l.part_ml = off;
  off = align_up(off + (size_t)l.rows * l.max_splits * l.G * sizeof(float2));
  l.part_acc = off;
  off = align_up(off + (size_t)l.rows * l.max_splits * l.G * d->head_dim * sizeof(float));
  l.total = l.max_splits > 1 ? off : 0;  // one split per row writes `out` directly
  return l;
}

// ---- stage timing -----------------------------------------------------------------------------
struct Timing {
  int n_calls = 0;
  int next_select = 0, next_decode = 0;
  std::vector<hipEvent_t> sel;  // [n_calls][SAGEKV_N_STAGES][2]
  std::vector<hipEvent_t> dec;  // [n_calls][2]
  std::vector<uint32_t> sel_mask;  // [n_calls] stages that recorded both events
  uint32_t stages = ~0u;           // select stages to bracket
  bool decode = true;              // bracket decode calls
} g_timing;

struct StageTimer {
  hipEvent_t* ev = nullptr;
  uint32_t* mask = nullptr;
  hipStream_t s;
  StageTimer(int which, hipStream_t stream) : s(stream) {
    if (g_timing.n_calls == 0) return;
    if (which == 0 && g_timing.next_select < g_timing.n_calls) {
      mask = &g_timing.sel_mask[g_timing.next_select];
      *mask = 0;
      ev = &g_timing.sel[(size_t)g_timing.next_select++ * SAGEKV_N_STAGES * 2];
    }
    if (which == 1 && g_timing.decode && g_timing.next_decode < g_timing.n_calls)
      ev = &g_timing.dec[(size_t)g_timing.next_decode++ * 2];
  }
  bool on(int stage) const { return ev && (!mask || ((g_timing.stages >> stage) & 1u)); }
  void begin(int stage) {
    if (on(stage)) (void)hipEventRecord(ev[stage * 2], s);
  }
  void end(int stage) {
    if (!on(stage)) return;
    (void)hipEventRecord(ev[stage * 2 + 1], s);
    if (mask) *mask |= 1u << stage;
  }
};

sagekv_status dev(hipError_t e) { return e == hipSuccess ? SAGEKV_OK : SAGEKV_ERR_DEVICE; }

// Checks the page description of a reduced cache of `capacity` tokens per row and turns it into the
// kernels' page map.
sagekv_status compact_page_map(const sagekv_paged_kv* pg, int dtype, int n_kv_heads, int head_dim, int64_t capacity,
                               PageMap* pm) {
  if (!pg || !pg->block_table || pg->n_pages < 1) return SAGEKV_ERR_INVALID_ARG;
  const int ps = pg->page_size;
  if (ps < 16 || (ps & (ps - 1))) return SAGEKV_ERR_INVALID_ARG;
  if (pg->table_pitch < (capacity + ps - 1) / ps) return SAGEKV_ERR_INVALID_ARG;
  const int64_t page_elems = (int64_t)n_kv_heads * ps * head_dim;
  if (pg->k_stride_page < page_elems || pg->v_stride_page < page_elems) return SAGEKV_ERR_INVALID_ARG;
  const int epl = dtype == SAGEKV_BF16 ? 8 : 4;
  if ((uintptr_t)pg->block_table & 3u || pg->k_stride_page % epl || pg->v_stride_page % epl) return SAGEKV_ERR_UNSUPPORTED;
  pm->table = pg->block_table;
  pm->pitch = pg->table_pitch;
  pm->ks_page = pg->k_stride_page;
  pm->vs_page = pg->v_stride_page;
  pm->shift = __builtin_ctz((unsigned)ps);
  pm->n_pages = pg->n_pages;
  return SAGEKV_OK;
}

// Scratch of sagekv_decode_step_static: the split partials of a decode step, for callers that cannot
// hand over device memory.  Every GPU the library runs on holds its own copy of this array at its
// own address; in host code the name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[SAGEKV_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU, once looked up

// Device address of the scratch array on the current GPU (looked up once per device, with that
// device current).
sagekv_status static_scratch(void** ptr) {
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return SAGEKV_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SAGEKV_ERR_DEVICE;
    g_scratch_ptr[device] = p;
  }
  *ptr = g_scratch_ptr[device];
  return SAGEKV_OK;
}

// Every cache and query row is read and written 16 bytes per lane.
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// `ring` (nullable, device): the count of appended tokens lives on the device; slot and len are then
// derived in the kernels and the launch moves the count on.
sagekv_status run_decode(const sagekv_decode_desc* d, const void* q, const void* q_sink, const void* k_new,
                         const void* v_new,
                         void* Kc, void* Vc, int slot, int len, int32_t* ring, float* out, void* ws,
                         size_t ws_bytes, hipStream_t s, const PageMap* cpm = nullptr) {
  if (!aligned16(q) || !aligned16(q_sink) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(Kc) ||
      !aligned16(Vc) || ((uintptr_t)out & 3u) || !aligned16(ws) || ((uintptr_t)ring & 3u))
    return SAGEKV_ERR_UNSUPPORTED;
  const DecodeLayout l = decode_layout(d);
  if (l.total > 0 && (!ws || ws_bytes < l.total)) return SAGEKV_ERR_WORKSPACE;
  DecodeParams p = {};
  p.n_problems = d->n_problems;
  p.Hq = d->n_q_heads;
  p.Hkv = d->n_kv_heads;
  p.G = l.G;
  p.D = d->head_dim;
  p.dtype = d->dtype;
  p.q = q;
  p.q_sink = q_sink;
  p.qs_S = q_sink ? d->n_sink : 0;
  p.Kc = Kc;
  p.Vc = Vc;
  p.k_new = k_new;
  p.v_new = v_new;
  p.slot = slot;
  p.len = len;
  p.cap = d->compact_capacity;
  // with the count on the device the length of a growing row is not known here: as many slices as
  // the full capacity would take (a fixed-size window has its one length either way)
  const int longest = ring && d->grow_recent ? d->compact_capacity : len;
  p.n_splits = splits_for(l.rows, longest, d->dtype, d->head_dim,
                          d->dtype == SAGEKV_BF16 ? (kFillDecode + l.rows - 1) / l.rows : slices_f32(l.rows, longest, d->head_dim));
  if (p.n_splits > l.max_splits) p.n_splits = l.max_splits;
  p.tokens_per_split = split_tokens(len, p.n_splits);
  p.ring = ring;
  p.ring_base = d->n_sink + decode_lists(d) * d->k;
  p.ring_W = d->n_recent;
  p.ring_grow = d->grow_recent;
  p.ring_advance = ring != nullptr;
  if (cpm) p.cpm = *cpm;
  // a reduced cache that cannot stay in L2 / Infinity Cache between steps is streamed (measured: +8 %)
  p.pq_S = d->n_sink;
  p.pq_k = decode_lists(d) > 1 ? d->k : 0;
  p.stream_loads = 2.0 * l.rows * len * d->head_dim * (d->dtype == SAGEKV_BF16 ? 2 : 4) > 192.0 * 1024 * 1024;
  p.part_ml = (float2*)((char*)ws + l.part_ml);
  p.part_acc = (float*)((char*)ws + l.part_acc);
  p.out = out;
  p.scale = (float)(1.0 / sqrt((double)d->head_dim));
  StageTimer t(1, s);
  t.begin(0);
  hipError_t e = launch_decode(p, s);
  t.end(0);
  return dev(e);
}

}  // namespace

extern "C" {

sagekv_status sagekv_paper_budget(int32_t B, int32_t G, int32_t* n_sink, int32_t* k, int32_t* n_recent) {
  if (!n_sink || !k || !n_recent || G < 1 || B < 4 * (int64_t)G) return SAGEKV_ERR_INVALID_ARG;
  const int32_t share = B / (2 * G);  // >= 2
  int32_t pow2 = 1;
  while (pow2 <= share / 2) pow2 *= 2;
  *n_sink = B / 4;
  *k = pow2;
  *n_recent = B - B / 4 - G * pow2;
  return SAGEKV_OK;
}

const char* sagekv_status_string(sagekv_status s) {
  switch (s) {
    case SAGEKV_OK: return "ok";
    case SAGEKV_ERR_INVALID_ARG: return "invalid argument";
    case SAGEKV_ERR_UNSUPPORTED: return "unsupported configuration";
    case SAGEKV_ERR_WORKSPACE: return "workspace missing or too small";
    case SAGEKV_ERR_DEVICE: return "HIP launch failed";
    case SAGEKV_ERR_SCRATCH_LIMIT: return "problem exceeds the library's built-in scratch (SAGEKV_STATIC_SCRATCH_BYTES)";
  }
  return "unknown status";
}

size_t sagekv_select_workspace_bytes(const sagekv_select_desc* desc) {
  sagekv_status st;
  if (!check_select(desc, &st)) return 0;
  const size_t n = select_layout(desc, true, true).total, less = select_layout(desc, true, false).total;
  return n > less ? n : less;
}

}  // extern "C"

namespace {

sagekv_status select_impl(const sagekv_select_desc* d, const PageMap& pm, const void* q_last, const void* K,
                          const void* V, void* Kc, void* Vc, int32_t* kept_idx, float* scores_out, void* workspace,
                          size_t workspace_bytes, void* hip_stream, const PageMap* out_pm = nullptr) {
  sagekv_status st;
  if (!check_select(d, &st)) return st;
  if (!q_last || !K || !V || !Kc || !Vc || !kept_idx) return SAGEKV_ERR_INVALID_ARG;
  if (!aligned16(q_last) || !aligned16(K) || !aligned16(V) || !aligned16(Kc) || !aligned16(Vc) ||
      ((uintptr_t)kept_idx & 3u) || ((uintptr_t)scores_out & 15u) || !aligned16(workspace))
    return SAGEKV_ERR_UNSUPPORTED;
  SelectLayout l = select_layout(d, scores_out == nullptr, false);
  if (!workspace || workspace_bytes < l.total) return SAGEKV_ERR_WORKSPACE;
  if (scores_out == nullptr) {
    const SelectLayout few = select_layout(d, true, true);
    if (few.one_sweep && workspace_bytes >= few.total) l = few;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  // per-token scores are only produced by the dense stages
  const bool fast = !l.one_sweep && scores_out == nullptr;

  RowGeom geo;
  geo.n_problems = d->n_problems;
  geo.Hq = d->n_q_heads;
  geo.Hkv = d->n_kv_heads;
  geo.G = l.G;
  geo.D = d->head_dim;
  geo.dtype = d->dtype;
  geo.L = d->L;
  geo.Lp = l.Lp;

  float* scores = scores_out ? scores_out : (float*)(ws + l.scores);
  const int64_t pitch = scores_out ? d->L : l.Lp;
  float* lines = (float*)(ws + l.partials);
  RowStat* stats = (RowStat*)(ws + l.stats);
  int* ghist = (int*)(ws + l.ghist);
  const float scale = (float)(1.0 / sqrt((double)d->head_dim));

  StageTimer t(0, s);
  hipError_t e;

  ScoreParams sp = {};
  sp.geo = geo;
  sp.q_last = q_last;
  sp.K = K;
  sp.ks_problem = d->k_stride_problem;
  sp.ks_head = d->k_stride_head;
  sp.ks_token = d->k_stride_token;
  sp.pm = pm;
  sp.logits = (float*)(ws + l.logits);
  sp.lines = lines;
  sp.chunk_partials = (ChunkPartial*)(ws + l.partials);
  sp.n_chunks = l.n_chunks;
  sp.chunk = l.chunk;
  sp.g0 = 0;
  sp.scale = scale;
  sp.stats = stats;
  sp.scores = scores;
  sp.pitch = pitch;
  sp.ghist = ghist;
  sp.S = d->n_sink;
  sp.W = d->n_recent;
  sp.n_lists = l.n_lists;

  StatsParams tp = {};
  tp.lines = lines;
  tp.stats = stats;
  tp.ghist = ghist;
  tp.G = l.G;
  tp.n_chunks = l.n_chunks;
  tp.n_lists = l.n_lists;

  TopkParams kp = {};
  kp.geo = geo;
  kp.scores = scores;
  kp.pitch = pitch;
  kp.ghist = ghist;
  kp.stats = stats;
  kp.q_last = q_last;
  kp.K = K;
  kp.ks_problem = d->k_stride_problem;
  kp.ks_head = d->k_stride_head;
  kp.ks_token = d->k_stride_token;
  kp.pm = pm;
  kp.kept_idx = kept_idx;
  kp.S = d->n_sink;
  kp.W = d->n_recent;
  kp.k = d->k;
  kp.n_lists = l.n_lists;
  kp.band = kBand;

  // The sample stage: approximate softmax statistics and filter thresholds for the pre-filtered path; both
  // that path and the two-sweep path take from it which terms of a softmax sum need an fp64 exponent.
  auto run_sample = [&]() -> hipError_t {
    const FastPlan& f = l.fast;
    SampleParams mp = {};
    mp.geo = geo;
    mp.q_last = q_last;
    mp.K = K;
    mp.ks_problem = d->k_stride_problem;
    mp.ks_head = d->k_stride_head;
    mp.ks_token = d->k_stride_token;
    mp.pm = pm;
    mp.S = d->n_sink;
    mp.W = d->n_recent;
    mp.k = d->k;
    mp.nA = f.nA;
    mp.nB = f.nB;
    mp.nC = f.nC;
    mp.stepB = f.stepB;
    mp.validA = f.validA;
    mp.validC = f.validC;
    mp.wA = f.wA;
    mp.wB = f.wB;
    mp.wC = f.wC;
    mp.rank = f.rank;
    mp.n_lists = l.n_lists;
    mp.Gs = f.Gs;
    mp.samp_logit = (float*)(ws + l.samp_logit);
    mp.samp_stats = (float2*)(ws + l.samp_stats);
    mp.heavy_thr = (float*)(ws + l.heavy_thr);
    mp.samp_tau = (float*)(ws + l.samp_tau);
    mp.row_fail = (int*)(ws + l.row_fail);
    mp.ovf_count = (int*)(ws + l.ovf_count);
    mp.n_fail = (int*)(ws + l.n_fail);
    mp.scale = scale;
    t.begin(SAGEKV_STAGE_SAMPLE);
    const hipError_t es = launch_sample(mp, s);
    t.end(SAGEKV_STAGE_SAMPLE);
    return es;
  };

  if (fast) {
    // ---- pre-filtered path: sample, one filtering pass over K, selection among the candidates
    const FastPlan& f = l.fast;
    float2* samp_stats = (float2*)(ws + l.samp_stats);
    float* samp_tau = (float*)(ws + l.samp_tau);
    int* row_fail = (int*)(ws + l.row_fail);
    e = run_sample();
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    sp.heavy_thr = (const float*)(ws + l.heavy_thr);

    ScoreParams fp = sp;
    fp.filt.samp_stats = samp_stats;
    fp.filt.samp_tau = samp_tau;
    fp.filt.ovf_count = (int*)(ws + l.ovf_count);
    fp.filt.cand_idx = (int32_t*)(ws + l.cand_idx);
    fp.filt.cand_logit = (float*)(ws + l.cand_logit);
    fp.filt.cap_c = f.cap_c;
    fp.filt.cap_o = f.cap;
    fp.filt.slots_per_row = l.slots_per_row;
    fp.filt.Gs = f.Gs;
    fp.filt.n_lists = l.n_lists;
    fp.filt.S = d->n_sink;
    fp.filt.W = d->n_recent;
    t.begin(SAGEKV_STAGE_SCORE);
    e = launch_score_filter(fp, s);
    t.end(SAGEKV_STAGE_SCORE);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;

    TopkCandParams cp = {};
    cp.geo = geo;
    cp.lines = lines;
    cp.stats = stats;
    cp.samp_stats = samp_stats;
    cp.samp_tau = samp_tau;
    cp.ghist = ghist;
    cp.cand_idx = fp.filt.cand_idx;
    cp.cand_logit = fp.filt.cand_logit;
    cp.cap_c = f.cap_c;
    cp.cap_o = f.cap;
    cp.slots_per_row = l.slots_per_row;
    cp.n_chunks = l.n_chunks;
    cp.cand_score = (float*)(ws + l.cand_score);
    cp.cand_pos = (int32_t*)(ws + l.cand_pos);
    cp.cs_pitch = l.cs_pitch;
    cp.list_info = (float2*)(ws + l.list_info);
    cp.cap = f.cap;
    cp.Gs = f.Gs;
    cp.expect = f.expect;
    cp.n_lists = l.n_lists;
    cp.q_last = q_last;
    cp.K = K;
    cp.ks_problem = d->k_stride_problem;
    cp.ks_head = d->k_stride_head;
    cp.ks_token = d->k_stride_token;
    cp.pm = pm;
    cp.kept_idx = kept_idx;
    cp.row_fail = row_fail;
    cp.n_fail = (int*)(ws + l.n_fail);
    cp.S = d->n_sink;
    cp.W = d->n_recent;
    cp.k = d->k;
    cp.band = kBand;
    t.begin(SAGEKV_STAGE_TOPK);
    e = launch_topk_cand(cp, s);
    t.end(SAGEKV_STAGE_TOPK);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;

    // Rows that could not be certified: a second pass over their K turns the now exact (M, Z) into
    // every token's score, then the dense selection.  Both launches are gated by the rows' flags:
    // with nothing flagged they are a handful of workgroups that look at the flags and leave.
    t.begin(SAGEKV_STAGE_REDO);
    sp.gate.row_flag = row_fail;
    sp.gate.n_flagged = (int*)(ws + l.n_fail);
    e = launch_score(sp, SCORE_SCORES, s);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    kp.gate = sp.gate;
    e = launch_topk(kp, s);
    t.end(SAGEKV_STAGE_REDO);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
  } else if (!l.one_sweep) {
    // ---- every score is asked for, no logit scratch: two sweeps over K (partials, then scores)
    e = run_sample();  // for heavy_thr (it also clears the flags; the marker below follows it)
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    sp.heavy_thr = (const float*)(ws + l.heavy_thr);
    if (launch_fill_u32(ws + l.n_fail, 1, 0xFFFFFFFFu, s) != hipSuccess) return SAGEKV_ERR_DEVICE;
    t.begin(SAGEKV_STAGE_SCORE);
    e = launch_score(sp, SCORE_PARTIALS, s);
    t.end(SAGEKV_STAGE_SCORE);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    t.begin(SAGEKV_STAGE_STATS);
    e = launch_stats(tp, l.rows, s);
    t.end(SAGEKV_STAGE_STATS);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    t.begin(SAGEKV_STAGE_COMBINE);
    e = launch_score(sp, SCORE_SCORES, s);
    t.end(SAGEKV_STAGE_COMBINE);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    t.begin(SAGEKV_STAGE_TOPK);
    e = launch_topk(kp, s);
    t.end(SAGEKV_STAGE_TOPK);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
  } else {
    // ---- one-sweep dense path: logits to scratch, statistics, scores, selection
    t.begin(SAGEKV_STAGE_SCORE);
    e = launch_score(sp, SCORE_LOGITS, s);
    t.end(SAGEKV_STAGE_SCORE);
    if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    DenseRows in = {};
    in.geo = geo;
    in.logits = sp.logits;
    in.partials = sp.chunk_partials;
    in.n_chunks = l.n_chunks;
    in.chunk = l.chunk;
    in.q_last = q_last;
    in.K = K;
    in.ks_problem = d->k_stride_problem;
    in.ks_head = d->k_stride_head;
    in.ks_token = d->k_stride_token;
    in.pm = pm;
    int* const flags = l.small ? (int*)(ws + l.flags) : nullptr;
    int* const marker = l.small ? (int*)(ws + l.n_fail) : nullptr;
    if (l.shortlist) {
      ShortlistParams hp = {};
      hp.in = in;
      hp.stats = stats;
      hp.scores = scores;
      hp.pitch = pitch;
      hp.cand = (uint2*)(ws + l.short_cand);
      hp.count = (int*)(ws + l.short_count);
      hp.tau = (float*)(ws + l.short_tau);
      hp.flag = flags;
      hp.marker = marker;
      hp.n_parts = l.list.n_parts;
      hp.part_tokens = l.list.part_tokens;
      hp.n_exact = l.list.n_exact;
      hp.S = d->n_sink;
      hp.W = d->n_recent;
      hp.n_lists = l.n_lists;
      hp.first_run = l.list.first_run;
      hp.n_runs = l.list.n_runs;
      hp.rank = l.list.rank;
      hp.step = l.list.step;
      hp.expect = l.list.expect;
      t.begin(SAGEKV_STAGE_TOPK);
      e = launch_shortlist(hp, kp, s);
      t.end(SAGEKV_STAGE_TOPK);
      if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    } else if (d->L <= kRowSelectMax) {
      RowSelectParams rp = {};
      rp.in = in;
      rp.scores = scores_out;
      rp.pitch = pitch;
      rp.kept_idx = kept_idx;
      rp.S = d->n_sink;
      rp.W = d->n_recent;
      rp.k = d->k;
      rp.n_lists = l.n_lists;
      rp.band = kBand;
      rp.flag = flags;
      rp.marker = marker;
      t.begin(SAGEKV_STAGE_TOPK);
      e = launch_row_select(rp, s);
      t.end(SAGEKV_STAGE_TOPK);
      if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    } else {
      RowStatsParams xp = {in, stats, ghist, l.n_lists};
      t.begin(SAGEKV_STAGE_STATS);
      e = launch_row_stats(xp, s);
      t.end(SAGEKV_STAGE_STATS);
      if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
      CombineParams cp = {};
      cp.geo = geo;
      cp.logits = sp.logits;
      cp.n_chunks = l.n_chunks;
      cp.chunk = l.chunk;
      cp.stats = stats;
      cp.scores = scores;
      cp.pitch = pitch;
      cp.ghist = ghist;
      cp.S = d->n_sink;
      cp.W = d->n_recent;
      cp.n_lists = l.n_lists;
      t.begin(SAGEKV_STAGE_COMBINE);
      e = launch_combine(cp, s);
      t.end(SAGEKV_STAGE_COMBINE);
      if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
      t.begin(SAGEKV_STAGE_TOPK);
      e = launch_topk(kp, s);
      t.end(SAGEKV_STAGE_TOPK);
      if (e != hipSuccess) return SAGEKV_ERR_DEVICE;
    }
  }

  GatherParams gp = {};
  gp.geo = geo;
  gp.K = K;
  gp.V = V;
  gp.ks_problem = d->k_stride_problem;
  gp.ks_head = d->k_stride_head;
  gp.ks_token = d->k_stride_token;
  gp.vs_problem = d->v_stride_problem;
  gp.vs_head = d->v_stride_head;
  gp.vs_token = d->v_stride_token;
  gp.pm = pm;
  gp.kept_idx = kept_idx;
  gp.Kc = Kc;
  gp.Vc = Vc;
  gp.n_kept = d->n_sink + l.n_lists * d->k + d->n_recent;
  gp.cap = d->compact_capacity;
  if (out_pm) gp.cpm = *out_pm;
  t.begin(SAGEKV_STAGE_GATHER);
  e = launch_gather(gp, s);
  t.end(SAGEKV_STAGE_GATHER);
  return dev(e);
}

}  // namespace

extern "C" {

sagekv_status sagekv_select(const sagekv_select_desc* d, const void* q_last, const void* K, const void* V, void* Kc,
                            void* Vc, int32_t* kept_idx, float* scores_out, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
  const PageMap none = {nullptr, 0, 0, 0, 0, 0};
  return select_impl(d, none, q_last, K, V, Kc, Vc, kept_idx, scores_out, workspace, workspace_bytes, hip_stream);
}

}  // extern "C"

namespace {
// Page map of a paged FULL cache (the strides inside a page come from the select descriptor).
sagekv_status input_page_map(const sagekv_select_desc* d, const sagekv_paged_kv* pg, PageMap* pm) {
  if (!pg || !pg->block_table || pg->n_pages < 1) return SAGEKV_ERR_INVALID_ARG;
  if ((uintptr_t)pg->block_table & 3u) return SAGEKV_ERR_UNSUPPORTED;
  const int ps = pg->page_size;
  if (ps < 16 || (ps & (ps - 1))) return SAGEKV_ERR_INVALID_ARG;
  if (pg->table_pitch < (d->L + ps - 1) / ps) return SAGEKV_ERR_INVALID_ARG;
  const int epl = d->dtype == SAGEKV_BF16 ? 8 : 4;
  if (pg->k_stride_page < 0 || pg->v_stride_page < 0 || pg->k_stride_page % epl || pg->v_stride_page % epl)
    return SAGEKV_ERR_UNSUPPORTED;
  pm->table = pg->block_table;
  pm->pitch = pg->table_pitch;
  pm->ks_page = pg->k_stride_page;
  pm->vs_page = pg->v_stride_page;
  pm->shift = __builtin_ctz((unsigned)ps);
  pm->n_pages = pg->n_pages;
  return SAGEKV_OK;
}
}  // namespace

extern "C" {

sagekv_status sagekv_select_paged(const sagekv_select_desc* d, const sagekv_paged_kv* pg, const void* q_last,
                                  const void* K_pool, const void* V_pool, void* Kc, void* Vc, int32_t* kept_idx,
                                  float* scores_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_select(d, &st)) return st;
  PageMap pm;
  st = input_page_map(d, pg, &pm);
  if (st != SAGEKV_OK) return st;
  return select_impl(d, pm, q_last, K_pool, V_pool, Kc, Vc, kept_idx, scores_out, workspace, workspace_bytes,
                     hip_stream);
}

sagekv_status sagekv_select_into_pages(const sagekv_select_desc* d, const sagekv_paged_kv* in_pages,
                                       const sagekv_paged_kv* out_pages, const void* q_last, const void* K,
                                       const void* V, void* Kc_pool, void* Vc_pool, int32_t* kept_idx,
                                       float* scores_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_select(d, &st)) return st;
  PageMap in_pm = {nullptr, 0, 0, 0, 0, 0}, out_pm;
  if (in_pages) {
    st = input_page_map(d, in_pages, &in_pm);
    if (st != SAGEKV_OK) return st;
  }
  st = compact_page_map(out_pages, d->dtype, d->n_kv_heads, d->head_dim, d->compact_capacity, &out_pm);
  if (st != SAGEKV_OK) return st;
  return select_impl(d, in_pm, q_last, K, V, Kc_pool, Vc_pool, kept_idx, scores_out, workspace, workspace_bytes,
                     hip_stream, &out_pm);
}

sagekv_status sagekv_select_redone_rows(const sagekv_select_desc* d, const void* workspace, size_t workspace_bytes,
                                        void* hip_stream, int32_t* n_rows) {
  sagekv_status st;
  if (!check_select(d, &st)) return st;
  if (!n_rows) return SAGEKV_ERR_INVALID_ARG;
  const SelectLayout l = select_layout(d, true, false);
  if (!workspace || workspace_bytes < l.total) return SAGEKV_ERR_WORKSPACE;
  *n_rows = -1;
  if (!l.small) return SAGEKV_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  if (hipStreamSynchronize(s) != hipSuccess) return SAGEKV_ERR_DEVICE;
  int n = 0;  // -1: the last call went through the dense stages for every row
  if (hipMemcpy(&n, (const char*)workspace + l.n_fail, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
    return SAGEKV_ERR_DEVICE;
  if (n == kFlagsPerList) {  // one flag per list
    const SelectLayout f = select_layout(d, true, true);
    if (workspace_bytes < f.total) return SAGEKV_ERR_WORKSPACE;
    const int lists = l.rows * l.n_lists;
    int flags[1024], last = -1;
    n = 0;
    for (int i0 = 0; i0 < lists; i0 += 1024) {
      const int cnt = lists - i0 < 1024 ? lists - i0 : 1024;
      if (hipMemcpy(flags, (const char*)workspace + f.flags + i0 * sizeof(int), cnt * sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
        return SAGEKV_ERR_DEVICE;
      for (int i = 0; i < cnt; ++i)
        if (flags[i] != 0 && (i0 + i) / l.n_lists != last) {
          last = (i0 + i) / l.n_lists;
          ++n;
        }
    }
  }
  *n_rows = n;
  return SAGEKV_OK;
}

sagekv_status sagekv_append(const sagekv_decode_desc* d, const void* k_new, const void* v_new, void* Kc, void* Vc,
                            int32_t n_appended, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!k_new || !v_new || !Kc || !Vc || n_appended < 0) return SAGEKV_ERR_INVALID_ARG;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(Kc) || !aligned16(Vc)) return SAGEKV_ERR_UNSUPPORTED;
  const int base = d->n_sink + decode_lists(d) * d->k;
  const int64_t slot = d->grow_recent ? (int64_t)base + d->n_recent + n_appended : base + n_appended % d->n_recent;
  if (slot >= d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  DecodeParams p = {};
  p.n_problems = d->n_problems;
  p.Hkv = d->n_kv_heads;
  p.D = d->head_dim;
  p.dtype = d->dtype;
  p.Kc = Kc;
  p.Vc = Vc;
  p.k_new = k_new;
  p.v_new = v_new;
  p.slot = (int)slot;
  p.cap = d->compact_capacity;
  return dev(launch_append(p, (hipStream_t)hip_stream));
}

size_t sagekv_decode_workspace_bytes(const sagekv_decode_desc* desc) {
  sagekv_status st;
  if (!check_decode(desc, &st)) return 0;
  return decode_layout(desc).total;
}

sagekv_status sagekv_decode_attn(const sagekv_decode_desc* d, const void* q, const void* Kc, const void* Vc,
                                 int32_t len, float* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !Kc || !Vc || !out || len < 1 || len > d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  return run_decode(d, q, nullptr, nullptr, nullptr, const_cast<void*>(Kc), const_cast<void*>(Vc), -1, len, nullptr, out,
                    workspace, workspace_bytes, (hipStream_t)hip_stream);
}

sagekv_status sagekv_decode_attn_window(const sagekv_decode_desc* d, const void* q, const void* q_sink, const void* Kc,
                                        const void* Vc, int32_t len, float* out, void* workspace,
                                        size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !q_sink || !Kc || !Vc || !out || len < 1 || len > d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  return run_decode(d, q, q_sink, nullptr, nullptr, const_cast<void*>(Kc), const_cast<void*>(Vc), -1, len, nullptr, out,
                    workspace, workspace_bytes, (hipStream_t)hip_stream);
}

sagekv_status sagekv_decode_step(const sagekv_decode_desc* d, const void* q, const void* k_new, const void* v_new,
                                 void* Kc, void* Vc, int32_t n_appended, float* out, void* workspace,
                                 size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !k_new || !v_new || !Kc || !Vc || !out || n_appended < 0) return SAGEKV_ERR_INVALID_ARG;
  const int base = d->n_sink + decode_lists(d) * d->k;
  const int64_t slot = d->grow_recent ? (int64_t)base + d->n_recent + n_appended : base + n_appended % d->n_recent;
  const int64_t len = d->grow_recent ? slot + 1 : (int64_t)base + d->n_recent;
  if (slot >= d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  return run_decode(d, q, nullptr, k_new, v_new, Kc, Vc, (int)slot, (int)len, nullptr, out, workspace, workspace_bytes,
                    (hipStream_t)hip_stream);
}

sagekv_status sagekv_decode_step_static(const sagekv_decode_desc* d, const void* q, const void* k_new, const void* v_new,
                                        void* Kc, void* Vc, int32_t n_appended, float* out, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !k_new || !v_new || !Kc || !Vc || !out || n_appended < 0) return SAGEKV_ERR_INVALID_ARG;
  const int base = d->n_sink + decode_lists(d) * d->k;
  const int64_t slot = d->grow_recent ? (int64_t)base + d->n_recent + n_appended : base + n_appended % d->n_recent;
  const int64_t len = d->grow_recent ? slot + 1 : (int64_t)base + d->n_recent;
  if (slot >= d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  if (decode_layout(d).total > (size_t)SAGEKV_STATIC_SCRATCH_BYTES) return SAGEKV_ERR_SCRATCH_LIMIT;
  void* ws = nullptr;
  st = static_scratch(&ws);
  if (st != SAGEKV_OK) return st;
  return run_decode(d, q, nullptr, k_new, v_new, Kc, Vc, (int)slot, (int)len, nullptr, out, ws,
                    (size_t)SAGEKV_STATIC_SCRATCH_BYTES, (hipStream_t)hip_stream);
}

sagekv_status sagekv_decode_attn_paged(const sagekv_decode_desc* d, const sagekv_paged_kv* pages, const void* q,
                                       const void* Kc_pool, const void* Vc_pool, int32_t len, float* out,
                                       void* workspace, size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !Kc_pool || !Vc_pool || !out || len < 1 || len > d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  PageMap cpm;
  st = compact_page_map(pages, d->dtype, d->n_kv_heads, d->head_dim, d->compact_capacity, &cpm);
  if (st != SAGEKV_OK) return st;
  return run_decode(d, q, nullptr, nullptr, nullptr, const_cast<void*>(Kc_pool), const_cast<void*>(Vc_pool), -1, len,
                    nullptr, out, workspace, workspace_bytes, (hipStream_t)hip_stream, &cpm);
}

sagekv_status sagekv_decode_step_paged(const sagekv_decode_desc* d, const sagekv_paged_kv* pages, const void* q,
                                       const void* k_new, const void* v_new, void* Kc_pool, void* Vc_pool,
                                       int32_t n_appended, int32_t* ring_state, float* out, void* workspace,
                                       size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !k_new || !v_new || !Kc_pool || !Vc_pool || !out || (!ring_state && n_appended < 0))
    return SAGEKV_ERR_INVALID_ARG;
  PageMap cpm;
  st = compact_page_map(pages, d->dtype, d->n_kv_heads, d->head_dim, d->compact_capacity, &cpm);
  if (st != SAGEKV_OK) return st;
  const int base = d->n_sink + decode_lists(d) * d->k;
  if (ring_state) {
    const int len = d->grow_recent ? d->compact_capacity : base + d->n_recent;
    return run_decode(d, q, nullptr, k_new, v_new, Kc_pool, Vc_pool, 0, len, ring_state, out, workspace,
                      workspace_bytes, (hipStream_t)hip_stream, &cpm);
  }
  const int64_t slot = d->grow_recent ? (int64_t)base + d->n_recent + n_appended : base + n_appended % d->n_recent;
  const int64_t len = d->grow_recent ? slot + 1 : (int64_t)base + d->n_recent;
  if (slot >= d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  return run_decode(d, q, nullptr, k_new, v_new, Kc_pool, Vc_pool, (int)slot, (int)len, nullptr, out, workspace,
                    workspace_bytes, (hipStream_t)hip_stream, &cpm);
}

sagekv_status sagekv_decode_step_ring(const sagekv_decode_desc* d, const void* q, const void* k_new, const void* v_new,
                                      void* Kc, void* Vc, int32_t* ring_state, float* out, void* workspace,
                                      size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !k_new || !v_new || !Kc || !Vc || !out || !ring_state) return SAGEKV_ERR_INVALID_ARG;
  const int base = d->n_sink + decode_lists(d) * d->k;
  // the longest row this step can attend (a growing row's length is only known on the device)
  const int len = d->grow_recent ? d->compact_capacity : base + d->n_recent;
  return run_decode(d, q, nullptr, k_new, v_new, Kc, Vc, 0, len, ring_state, out, workspace,
                    workspace_bytes, (hipStream_t)hip_stream);
}

sagekv_status sagekv_decode_step_window(const sagekv_decode_desc* d, const void* q, const void* q_sink,
                                        const void* k_new, const void* v_new, void* Kc, void* Vc, int32_t n_appended,
                                        float* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  sagekv_status st;
  if (!check_decode(d, &st)) return st;
  if (!q || !q_sink || !k_new || !v_new || !Kc || !Vc || !out || n_appended < 0) return SAGEKV_ERR_INVALID_ARG;
  const int base = d->n_sink + decode_lists(d) * d->k;
  const int64_t slot = d->grow_recent ? (int64_t)base + d->n_recent + n_appended : base + n_appended % d->n_recent;
  const int64_t len = d->grow_recent ? slot + 1 : (int64_t)base + d->n_recent;
  if (slot >= d->compact_capacity) return SAGEKV_ERR_INVALID_ARG;
  return run_decode(d, q, q_sink, k_new, v_new, Kc, Vc, (int)slot, (int)len, nullptr, out, workspace, workspace_bytes,
                    (hipStream_t)hip_stream);
}

sagekv_status sagekv_stage_timing_enable(int32_t n_calls) {
  for (hipEvent_t e : g_timing.sel) (void)hipEventDestroy(e);
  for (hipEvent_t e : g_timing.dec) (void)hipEventDestroy(e);
  g_timing.sel.clear();
  g_timing.dec.clear();
  g_timing.sel_mask.clear();
  g_timing.n_calls = 0;
  g_timing.next_select = g_timing.next_decode = 0;
  if (n_calls <= 0) return SAGEKV_OK;
  g_timing.sel.resize((size_t)n_calls * SAGEKV_N_STAGES * 2);
  g_timing.dec.resize((size_t)n_calls * 2);
  g_timing.sel_mask.assign((size_t)n_calls, 0u);
  for (hipEvent_t& e : g_timing.sel)
    if (hipEventCreate(&e) != hipSuccess) return SAGEKV_ERR_DEVICE;
  for (hipEvent_t& e : g_timing.dec)
    if (hipEventCreate(&e) != hipSuccess) return SAGEKV_ERR_DEVICE;
  g_timing.n_calls = n_calls;
  return SAGEKV_OK;
}

sagekv_status sagekv_stage_timing_stages(uint32_t select_stage_mask, int32_t decode) {
  g_timing.stages = select_stage_mask;
  g_timing.decode = decode != 0;
  return SAGEKV_OK;
}

sagekv_status sagekv_stage_timing_read(int32_t which, int32_t call, float* ms) {
  if (!ms || call < 0) return SAGEKV_ERR_INVALID_ARG;
  if (which == 0) {
    if (call >= g_timing.next_select) return SAGEKV_ERR_INVALID_ARG;
    hipEvent_t* ev = &g_timing.sel[(size_t)call * SAGEKV_N_STAGES * 2];
    for (int i = 0; i < SAGEKV_N_STAGES; ++i) {
      ms[i] = 0.f;
      if (!(g_timing.sel_mask[call] & (1u << i))) continue;
      if (hipEventSynchronize(ev[2 * i + 1]) != hipSuccess) return SAGEKV_ERR_DEVICE;
      if (hipEventElapsedTime(&ms[i], ev[2 * i], ev[2 * i + 1]) != hipSuccess) return SAGEKV_ERR_DEVICE;
    }
    return SAGEKV_OK;
  }
  if (which == 1) {
    if (call >= g_timing.next_decode) return SAGEKV_ERR_INVALID_ARG;
    hipEvent_t* ev = &g_timing.dec[(size_t)call * 2];
    if (hipEventSynchronize(ev[1]) != hipSuccess) return SAGEKV_ERR_DEVICE;
    if (hipEventElapsedTime(&ms[0], ev[0], ev[1]) != hipSuccess) return SAGEKV_ERR_DEVICE;
    return SAGEKV_OK;
  }
  return SAGEKV_ERR_INVALID_ARG;
}

}  // extern "C"
