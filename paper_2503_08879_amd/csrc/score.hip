// Eviction pass, scoring stage (paper Sec. 2 Step 2: attention scores of the last token's
// query against the cached keys).
//
//   score_f32_kernel, score_mfma_kernel (bf16)
//                   stream K once: logit[g][i] = q[g].K[i]/sqrt(d) for the G heads of a row.  What a
//                   pass leaves behind depends on its mode (ScoreMode): fp32 logits + per-chunk softmax
//                   partials (max, sum exp) for the one-sweep dense path; partials + the records of
//                   the tokens that pass the sample threshold (pre-filtered path); partials only, or
//                   every token's score from known (M, Z) (two-sweep dense path: rows the pre-filter
//                   could not certify, without a logit scratch).
//   sample_logits_kernel  logits of the sampled blocks of the pre-filtered path.
//   stats_kernel    merges the partials of a row into (M, Z) per head, in fp64 (two-sweep path).
//   combine_kernel  score[i] = sum_g exp(logit[g][i] - M_g) / Z_g  (fp32) and the first radix
//                   histogram of the candidates' scores, merged across workgroups with atomics.
#include "device_utils.h"
#include "kernels.h"
#include "radix_select.h"

namespace sagekv {

namespace {

constexpr int kScoreThreads = 256;
constexpr int kScoreWaves = kScoreThreads / kWave;
constexpr int64_t kWriteThrough = 1ll << 30;
// Logits of the one-sweep path go through L2 at once over more than this many bytes of keys, up to four heads: later they would be evicted in the
// middle of the stream, a few lines at a time.  (Nothing stored: 82 us for 256 rows x 8192 tokens x 4 heads, 537 MB; stored 97, through L2 92.)  Whole
// pass, us, left and written through: 64 rows x 8192 (134 MB) 68.7 and 69.4, 96 rows 96.0 and 95.9, 128 rows 118 and 117, 192 rows 166 and 163,
// 256 rows 214 and 211, 512 rows 421 and 416, 256 x 16K 419 and 413, 32 x 32K 88.2 and 87.1.  With more heads a store holds half lines of two heads:
// 128 rows x 8192 x 7 heads 129 and 131, 16 x 64K 91 and 94.
constexpr int64_t kLogitsThrough = 200000000;
constexpr int kGatedRowBlocks = 16;  // y-blocks of a gated score / combine launch
// A score workgroup takes a chunk of BPW blocks of 64 tokens per wave (BPW = 1, 2, 4: 256, 512, 1024 tokens).

// fp32 caches.  Products and sums in fp64 (the same four cycles as in fp32), so a logit is rounded once.  Eight lanes share a token, four or two
// 16-byte chunks each, and its eight parts are summed while heads and lanes change places: lane s of the eight ends with head s's
// logit (up to eight heads a launch).  A wave takes batches of 32 tokens (16 with 128 dims), lane group t of eight the tokens 4 t .. 4 t + 3 (2 t, 2 t + 1), so that a
// lane stores four (two) logits at once; the next batch's loads are in flight meanwhile.  (With 16 or 32 lanes per token and every head's logit summed over all of
// them in fp32 the pass was bound by vector instructions. Whole calls, us: 8 rows x 32K x 4 heads of 128 dims 66.3 and 53.8, 64 x 16K x 4 182
// and 169, 16 x 32K x 7 117 and 102, in pages 4 x 16K x 7 61.5 and 50.6, 64 x 8192 x 4 of 64 dims 67.3 and 59.7; plain loads instead of streaming
// ones 113 us for the pass over 64 x 16K, 100 so.)
//
// The softmax partial of the chunk is taken after the last block, from the logits in registers.
//
// 64 dims and seven heads would take 172 registers, two workgroups a CU: held to the 168 of three, without a spill, 64 rows x 40000 218 -> 196 us.  (Eight heads
// take 190: held to 168 they spill 32, 224 -> 228.)
template <int D, int GB, int BPW>
__global__ __launch_bounds__(kScoreThreads, D == 64 && GB == 7 ? 3 : 2) void score_f32_kernel(ScoreParams p) {
  constexpr int NC = D / 32;            // chunks of a token per lane
  constexpr int U = D == 64 ? 4 : 2;    // a lane group's tokens of a batch
  constexpr int NB = 64 * BPW / (8 * U);  // batches per wave
  constexpr int kChunk = 64 * BPW * kScoreWaves;
  __shared__ __attribute__((aligned(16))) double qd[GB * D];
  __shared__ float part_m[kScoreWaves][GB];
  __shared__ double part_s[kScoreWaves][GB];

  const int row = blockIdx.y;
  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t8 = lane >> 3, sl = lane & 7;
  const int64_t L = p.geo.L;
  const int64_t wave_base = (int64_t)blockIdx.x * kChunk + (int64_t)wave * BPW * 64;
  float qv[(GB * D + kScoreThreads - 1) / kScoreThreads];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(qv) / 4); ++i) {
    const int at = threadIdx.x + i * kScoreThreads;
    qv[i] = at < GB * D ? ((const float*)p.q_last)[((int64_t)prob * p.geo.Hq + c * p.geo.G + p.g0) * D + at] : 0.f;
  }
  uint4 kv[2][U][NC];
  auto load_batch = [&](int n, uint4 (&dst)[U][NC]) {
    if (wave_base + 8 * U * n < L) {  // wave-uniform
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int64_t tok = wave_base + 8 * U * n + U * t8 + u;
        tok = tok < L ? tok : L - 1;  // tail: re-read the last token, masked below
        const char* a = (const char*)p.K + kv_offset(p.pm, p.pm.ks_page, p.ks_problem, p.ks_head, p.ks_token, prob, c, tok) * 4 + sl * 16;
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) dst[u][ch] = ld16_stream(a + ch * 128);
      }
    }
  };
  load_batch(0, kv[0]);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(qv) / 4); ++i)
    if ((int)threadIdx.x + i * kScoreThreads < GB * D) qd[threadIdx.x + i * kScoreThreads] = (double)qv[i];
  __syncthreads();

  float xs[NB][U];  // of head sl; -INFINITY: no token
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int64_t tok0 = wave_base + 8 * U * n + U * t8;
    if (n + 1 < NB) load_batch(n + 1, kv[(n + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) xs[n][u] = -INFINITY;
    if (wave_base + 8 * U * n < L) {
#pragma unroll
      for (int uu = 0; uu < U; uu += 2) {
#pragma unroll
        for (int hh = 0; hh < GB; hh += 4) {
          asm volatile("" ::: "memory");  // the queries are read again, not held for the other tokens
          double a[2][4];
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < 4; ++h) a[u][h] = 0.0;
#pragma unroll
          for (int ch = 0; ch < NC; ++ch) {
            double kd[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              uint4 k = kv[n & 1][uu + u][ch];
              if (GB > 4) asm volatile("" : "+v"(k.x), "+v"(k.y), "+v"(k.z), "+v"(k.w));  // converted again for the other four heads, not held
              kd[u][0] = (double)__uint_as_float(k.x);
              kd[u][1] = (double)__uint_as_float(k.y);
              kd[u][2] = (double)__uint_as_float(k.z);
              kd[u][3] = (double)__uint_as_float(k.w);
            }
#pragma unroll
            for (int h = 0; h < 4 && hh + h < GB; ++h) {
              const double* q = qd + (hh + h) * D + (ch * 8 + sl) * 4;
#pragma unroll
              for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[u][h] = fma(kd[u][e], q[e], a[u][h]);
            }
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const float r = (float)(eight_lane_sums<GB>(a[u], sl) * (1.0 / sqrt((double)D)));
            xs[n][uu + u] = hh == 0 || sl >= 4 ? r : xs[n][uu + u];
          }
        }
      }
      // (past the row's end, inside the chunk's scratch: the last token's again)
      if (sl < GB)
      {
        float* at = p.logits + logit_index(p.geo, p.n_chunks, p.chunk, row, p.g0 + sl, tok0);
        if constexpr (U == 4)
          *reinterpret_cast<float4*>(at) = make_float4(xs[n][0], xs[n][1], xs[n][2], xs[n][3]);
        else
          *reinterpret_cast<float2*>(at) = make_float2(xs[n][0], xs[n][1]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (tok0 + u >= L) xs[n][u] = -INFINITY;
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // (max, sum) of the chunk: the lanes of a head -> wave -> workgroup
  float m = -INFINITY;
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int u = 0; u < U; ++u) m = fmaxf(m, xs[n][u]);
  m = fmaxf(m, dpp_f32<0x128>(m));  // row_ror:8
  m = swap32_max(swap16_max(m));
  if (lane < GB) part_m[wave][lane] = m;
  __syncthreads();
  float M = -INFINITY;
  if (sl < GB) {
#pragma unroll
    for (int w = 0; w < kScoreWaves; ++w) M = fmaxf(M, part_m[w][sl]);
  }
  M = M == -INFINITY ? 0.f : M;  // nothing but -inf: the sum is 0
  double z = 0.0;
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int u = 0; u < U; ++u) z += (double)exp_fast(xs[n][u] - M);
  z += dpp_f64<0x128>(z);
  z += swap16_f64(z);
  z = swap32_sum_f64(z);
  if (lane < GB) part_s[wave][lane] = z;
  __syncthreads();
  if (threadIdx.x < GB) {
    const int g = threadIdx.x;
    float mm = part_m[0][g];
    double zz = 0.0;
#pragma unroll
    for (int w = 0; w < kScoreWaves; ++w) {
      mm = fmaxf(mm, part_m[w][g]);
      zz += part_s[w][g];
    }
    p.chunk_partials[((int64_t)row * p.geo.G + p.g0 + g) * p.n_chunks + blockIdx.x] = ChunkPartial{zz, mm, 0.f};
  }
}

// bf16 scoring on the matrix cores.  The dot products of a 16-token tile against the group's
// query heads are one 16x16x(head_dim) product: A = queries (heads in rows, zero padded),
// B = keys (tokens in columns), fp32 accumulate.  MFMA operands want a lane to hold 8
// consecutive elements of ONE token per column lane, while coalesced loads give adjacent lanes
// adjacent 16-byte chunks of the SAME token, so each wave stages its 64-token block through a
// private, XOR-swizzled LDS buffer (conflict free both ways).  GPAD = heads padded to 4, 8 or
// 16: the operand's rows repeat them 16/GPAD times and a lane takes the product of the tile of its slot, so that
// 16/GPAD tiles share a set of four registers, after a block every lane owns 4 logits and all stores are coalesced.
//
// MODE (ScoreMode) says what the pass leaves behind:
//   SCORE_LOGITS    every logit, to the scratch of the one-sweep dense path, and the softmax partials;
//   SCORE_FILTER    the pre-filtered path: nothing is written per token.  A lane keeps its logits only for
//                   tokens whose approximate score (sample statistics) reaches the row's conservative
//                   threshold, and appends (index, logits) to the chunk's candidate slots, or, once those
//                   are used up, to the row's overflow pool;
//   SCORE_PARTIALS  the softmax partials only;
//   SCORE_SCORES    with (M, Z) of every head known: every token's score (summed over the group, or one
//                   row per head), and the first radix histogram of the candidates' scores.
//
// PAGED: the chunk's pages (at most 64: pages hold 16 tokens or more) are looked up once, one per
// lane, and every load takes its page from the lane that holds it.
// One score chunk (64 * BPW * kScoreWaves tokens of row `row`) by one workgroup of kScoreThreads threads.
//
// The block loop is rolled where nothing is kept per token: unrolled, each block would have its own body for heavy terms.  The partials
// of 9 to 16 heads of 128 dims took 276 registers so, and a CU one workgroup, with nobody to cover its LDS and MFMA
// phases; rolled, and held to the 256 of two workgroups, they fit without spilling.  A pass that also returns every score, unrolled and
// rolled, us: 8 rows x 32K tokens x 16 heads 102.5 and 99.8, 64 x 32K 291 and 268, 256 x 32K 906 and 829, 64 x 128K 838 and 766 (12
// heads 832 and 754); with at most 8 heads and with 64 dims the two are even.
template <int D, int GPAD, int MODE, bool PAGED, int BPW>
__device__ __forceinline__ void score_mfma_chunk(const ScoreParams& p, int gb, int row, int chunk) {
  constexpr int CH = D / 8;         // 16-byte chunks per token
  constexpr int TPL = 64 / CH;      // tokens per coalesced wave load
  constexpr int NLOAD = 64 / TPL;   // loads per 64-token block
  constexpr int KSTEPS = D / 32;    // MFMA k-steps per tile
  constexpr int TILES = 16 / GPAD;  // 16-token tiles per accumulator
  constexpr int NACC = 4 / TILES;   // accumulators per block
  constexpr bool FILTER = MODE == SCORE_FILTER;
  constexpr bool KEEP = MODE == SCORE_LOGITS || MODE == SCORE_SCORES;  // per-token values held to the end
  constexpr bool PARTIALS = MODE == SCORE_FILTER || MODE == SCORE_PARTIALS;  // running sums (SCORE_LOGITS: at the end)
  constexpr bool HEAVY = PARTIALS;
  constexpr int kChunk = 64 * BPW * kScoreWaves;
  // heavy terms per register of a lane, and tile, up to which they are taken one by one (a round of four 0.3 us, a tile's products 1 us
  // with 128 dims, 0.6 with 64).  64 rows x 32K tokens of N(60, 1) logits, all tiles / up to 1 / 2 / 3 terms, us: 4 heads of 128 dims 223 175 168 167,
  // 7 heads 264 213 185 183, 16 heads 350 327 267 261
  constexpr int kThin = D == 128 ? 3 : 2;
  constexpr int kAddUnroll = GPAD == 16 && (FILTER || D == 128) ? 1 : 4;  // (four exponentials side by side: spills)
  constexpr int kBlockUnroll = PARTIALS ? 1 : BPW;

  __shared__ uint4 lds[kScoreWaves][64 * CH];
  __shared__ float2 part[kScoreWaves][4][4];
  // FILTER: a wave collects its candidates in LDS and stores them in runs, see `flush`
  constexpr int GQ = GPAD / 4;                                       // float4s in a record (Gs = GPAD)
  constexpr int kStash = GPAD == 4 ? 128 : GPAD == 8 ? 96 : 48;      // room for at least two accumulators' tokens
  __shared__ float4 stash_rec[FILTER ? kScoreWaves : 1][FILTER ? kStash * GQ : 1];
  __shared__ int32_t stash_tok[FILTER ? kScoreWaves : 1][FILTER ? kStash : 1];
  __shared__ int n_kept_wg;  // candidates this workgroup has stored so far
  static_assert(!FILTER || sizeof(lds) + sizeof(part) + sizeof(stash_rec) + sizeof(stash_tok) + sizeof(n_kept_wg) <= 80 * 1024,
                "two workgroups share a CU's 160 KB");

  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tq = lane / CH, cl = lane % CH;  // load role: token sub-index, chunk
  const int n = lane & 15, j = lane >> 4;    // MFMA role: column (token), k-group / row block
  const int64_t L = p.geo.L;
  uint4* buf = lds[wave];

  const char* Krow = (const char*)p.K + ((int64_t)prob * p.ks_problem + (int64_t)c * p.ks_head) * 2;
  const int64_t tok_bytes = p.ks_token * 2;
  int my_page = 0, first_page = 0;
  if (PAGED) {
    Krow = (const char*)p.K + (int64_t)c * p.ks_head * 2;
    first_page = (int)(((int64_t)chunk * kChunk) >> p.pm.shift);
    const int last_page = (int)((L - 1) >> p.pm.shift);
    const int pg = first_page + lane < last_page ? first_page + lane : last_page;
    my_page = page_of(p.pm, prob, (int64_t)pg << p.pm.shift);
  }
  // The waves of a workgroup take the chunk's 64-token blocks round robin, so the workgroup reads
  // one contiguous 64 KiB run at a time; the first block's loads go out before anything else.
  const int64_t wave_base = (int64_t)chunk * kChunk + (int64_t)wave * 64;
  constexpr int64_t kBlockStride = 64 * kScoreWaves;
  const int64_t lane_off = (int64_t)tq * tok_bytes + cl * 16;
  uint4 kv[NLOAD];
  // the block of 64 tokens from tb on (tb wave-uniform, < L).  Load i covers the TPL tokens from tb + i * TPL on, which
  // share a page: its address is a wave-uniform base plus the lane's offset, but for the row's last, partial block.
  auto load_block = [&](int64_t tb) {
    if (tb + 64 <= L) {
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) {
        const char* base;
        if (PAGED) {
          const int64_t tok = tb + i * TPL;
          const int pid = __builtin_amdgcn_readlane(my_page, (int)(tok >> p.pm.shift) - first_page);
          base = Krow + ((int64_t)pid * p.pm.ks_page * 2 + (tok & ((1 << p.pm.shift) - 1)) * tok_bytes);
        } else {
          base = Krow + (tb + i * TPL) * tok_bytes;
        }
        kv[i] = ld16_stream(base + lane_off);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) {
        int64_t tok = tb + i * TPL + tq;
        tok = tok < L ? tok : L - 1;  // re-read the last token, masked below
        if (PAGED) {
          const int pid = __shfl(my_page, (int)(tok >> p.pm.shift) - first_page);
          kv[i] = ld16_stream(Krow + ((int64_t)pid * p.pm.ks_page * 2 + (tok & ((1 << p.pm.shift) - 1)) * tok_bytes) + cl * 16);
        } else {
          kv[i] = ld16_stream(Krow + tok * tok_bytes + cl * 16);
        }
      }
    }
  };
  if (wave_base < L) load_block(wave_base);
  // A operand: lane (row m = n, k-group j) holds q[head m % GPAD][8*(4*kc + j) ..+8]
  const int my_head = n % GPAD, tslot = (4 * j) / GPAD;
  uint4 qa[KSTEPS];
#pragma unroll
  for (int kc = 0; kc < KSTEPS; ++kc) {
    qa[kc] = make_uint4(0u, 0u, 0u, 0u);
    if (my_head < gb) {
      const int h = c * p.geo.G + p.g0 + my_head;
      qa[kc] = ld16((const char*)p.q_last + (((int64_t)prob * p.geo.Hq + h) * D + (4 * kc + j) * 8) * 2);
    }
  }

  // each lane ends up with the logits of heads hbase .. hbase+3
  const int hbase = (4 * j) % GPAD;
  float m[4], sum[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    m[r] = -INFINITY;
    sum[r] = 0.f;
  }

  // softmax weights of this lane's 4 heads: the sample's (M^, 1/Z^) for the filter, the exact (M, 1/Z)
  // for the scores; the row's filter threshold(s)
  float fM[4] = {0.f, 0.f, 0.f, 0.f}, fInv[4] = {0.f, 0.f, 0.f, 0.f}, ftau = 0.f;
  // terms with an fp64 exponent (ScoreParams::heavy_thr): the passes that follow a sample stage.  (The one-sweep
  // dense pass, SCORE_LOGITS, knows nothing about the row yet: exact_changes takes them once the partials are merged.)
  float hthr[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
  if (HEAVY && p.heavy_thr) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (hbase + r < gb) hthr[r] = p.heavy_thr[(int64_t)row * p.geo.G + p.g0 + hbase + r];
  }
  float ftau_h[4] = {INFINITY, INFINITY, INFINITY, INFINITY};  // per-query lists: a threshold per head
  const bool per_head = FILTER && p.filt.n_lists > 1;
  if (FILTER) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (hbase + r < gb) {
        const float2 st = p.filt.samp_stats[(int64_t)row * p.geo.G + hbase + r];
        fM[r] = st.x;
        fInv[r] = st.y;
        if (per_head) ftau_h[r] = p.filt.samp_tau[(int64_t)row * p.geo.G + hbase + r];
      }
    if (!per_head) ftau = p.filt.samp_tau[row];
    if (threadIdx.x == 0) n_kept_wg = 0;
    __syncthreads();
  }
  if (MODE == SCORE_SCORES) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (hbase + r < gb) {
        const RowStat st = p.stats[(int64_t)row * p.geo.G + p.g0 + hbase + r];
        fM[r] = st.M;
        fInv[r] = st.invZ;
      }
  }
  // FILTER: this chunk's own candidate slots, and the row's overflow pool behind all chunks' slots
  const int64_t row_slots = (int64_t)row * p.filt.slots_per_row;
  const int64_t slot_base = row_slots + (int64_t)chunk * p.filt.cap_c;
  const int64_t ovf_base = row_slots + (int64_t)p.n_chunks * p.filt.cap_c;
  // The wave's collected candidates into the next free slots.  In runs, because these few bytes cost what the write-backs of
  // their lines cost, not what the store instructions do (stored over and over into 16 KB that stay in L2, the pass takes what it takes
  // with nothing stored).  Nothing stored / stored as met / in runs: 64 rows x 40K tokens in pages, 7 heads 117 / 137 / 124 us,
  // 112 rows x 128K, 7 lists 549 / 625 / 605, 8 rows x 128K, 4 heads 49 / 52 / 48 (with the lines of the partials).
  // Over more than kWriteThrough bytes of keys they are written through L2 at once, not left for it to evict in the middle of
  // the stream; a small call's selection finds them in the caches.  Whole
  // pass, left and written through, us: 64 rows x 40K in pages (0.6 GB) 169 and 171, 96 x 32K (0.8 GB) 206 and 206, 128 x 32K (1.1 GB) 256
  // and 255, 64 x 128K (2.1 GB) 418 and 411, 256 x 32K (2.1 GB) 479 and 472, 112 x 128K with 7 lists (3.8 GB) 871 and 848, 256 x 128K (8.6 GB)
  // 1542 and 1522.
  int n_stash = 0;  // wave-uniform
  auto flush = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int base = 0;
    if (lane == 0) base = atomicAdd(&n_kept_wg, n_stash);  // LDS counter
    base = __builtin_amdgcn_readfirstlane(base);
    int fit = p.filt.cap_c - base, room = 0;  // candidates that take the chunk's own slots, and the pool's
    fit = fit < 0 ? 0 : fit < n_stash ? fit : n_stash;
    int64_t over = 0;
    if (fit < n_stash) {  // rare: the chunk's own slots are used up
      int o = 0;
      if (lane == 0) o = atomicAdd(&p.filt.ovf_count[row], n_stash - fit);
      o = __builtin_amdgcn_readfirstlane(o);
      room = o < p.filt.cap_o ? p.filt.cap_o - o : 0;  // pool full: dropped, the row is redone
      over = ovf_base + o - fit;
    }
    const int last = room < n_stash - fit ? fit + room : n_stash;
    for (int i = lane; i < last * GQ; i += 64) {
      const int e = i / GQ;
      const int64_t slot = e < fit ? slot_base + base + e : over + e;
      const float4 rec = stash_rec[wave][i];
      if (p.filt.write_through && e < fit)  // (descriptor of the run, bounds not used: the slots are the chunk's own)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, rec),
                                               __builtin_amdgcn_make_buffer_rsrc(p.filt.cand_logit + (slot_base + base) * (4 * GQ), 0, -1, 0x00027000),
                                               i * 16, 0, 16 /* sc1 */);
      else
        reinterpret_cast<float4*>(p.filt.cand_logit)[slot * GQ + i % GQ] = rec;
      if (i % GQ == 0) p.filt.cand_idx[slot] = stash_tok[wave][e];
    }
    n_stash = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  const unsigned long long before_mine = (1ull << (((j - j % GQ) << 4) | n)) - 1ull;  // lanes that count tokens before this lane's
  constexpr unsigned long long kCounting = GPAD == 4 ? ~0ull : GPAD == 8 ? 0x0000FFFF0000FFFFull : 0xFFFFull;  // one lane per token

  // Software pipeline: the loads of block b+1 are issued right after block b went to LDS, so
  // their latency overlaps block b's MFMA phase.  Loads and stores share one in-order completion counter, so a
  // store inside the loop puts its write-ack latency on the critical path of the next block: what is kept per token stays
  // in registers until the wave has loaded its last block, and the filter stores only when its stash is full (`flush`; with 6.8 thousand
  // candidates in a row of 128K tokens, 13 per wave, after the loop).
  // HEAVY: this lane's share of the heavy terms of heads j + 4 i: sum of exp(l - heavy_m) in fp64
  bool seen_heavy = false;
  double heavy_m[GQ], heavy_z[GQ];
#pragma unroll
  for (int i = 0; i < GQ; ++i) heavy_m[i] = -INFINITY, heavy_z[i] = 0.0;
  float xs[KEEP ? BPW : 1][NACC][4];
#pragma unroll kBlockUnroll
  for (int blk = 0; blk < BPW; ++blk) {
    const int64_t tok_base = wave_base + (int64_t)blk * kBlockStride;
    if (tok_base < L) {  // wave-uniform
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // previous block's LDS reads are done
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) {
        const int t = i * TPL + tq;
        buf[t * CH + (cl ^ (t & (CH - 1)))] = kv[i];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (blk + 1 < BPW && tok_base + kBlockStride < L) {
        int64_t next = tok_base + kBlockStride;
        asm volatile("" : "+s"(next));  // the addresses of later blocks are not computed (and held) up front
        load_block(next);
      }
      // Row m of the A operand is head m % GPAD whatever the tile slot, so a tile's product holds every head's logits 16 / GPAD
      // times over and each lane takes the tile of its slot.  (One accumulator for the tiles, with A zero but for the slot's rows:
      // a chain of 16 / GPAD times as many products, and as many copies of A in registers.)
      f32x4_t acc[NACC];
#pragma unroll
      for (int a = 0; a < NACC; ++a) {
#pragma unroll
        for (int ts = 0; ts < TILES; ++ts) {
          const int t = (a * TILES + ts) * 16 + n;
          f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kc = 0; kc < KSTEPS; ++kc) {
            const uint4 b = buf[t * CH + ((4 * kc + j) ^ (n & (CH - 1)))];
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qa[kc]), __builtin_bit_cast(bf16x8_t, b), d, 0, 0, 0);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[a][r] = ts == 0 || tslot == ts ? d[r] : acc[a][r];
        }
      }
      // lane (j, n), accumulator a, register r: row 4j + r = (tile slot, head), column n = token
      bool any_heavy = false;
#pragma unroll
      for (int a = 0; a < NACC; ++a) {
        const int64_t tok = tok_base + (a * TILES + (4 * j) / GPAD) * 16 + n;
        float approx = 0.f;
        int any_head = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = acc[a][r] * p.scale;
          xs[KEEP ? blk : 0][a][r] = x;
          if (MODE != SCORE_LOGITS && tok < L && hbase + r < gb) {
            if (PARTIALS) {
              const float mn = fmaxf(m[r], x);
              const bool hv = HEAVY && x >= hthr[r];  // rare: its term is added below, with an fp64 exponent
              any_heavy |= hv;
              sum[r] = sum[r] * exp_fast(m[r] - mn) + (hv ? 0.f : exp_fast(x - mn));
              m[r] = mn;
            }
            if (FILTER) {
              const float pr = exp_fast(x - fM[r]) * fInv[r];
              approx += pr;
              any_head |= !(pr < ftau_h[r]);
            }
            if (MODE == SCORE_SCORES) xs[KEEP ? blk : 0][a][r] = exp_times(x - fM[r], fInv[r]);
          } else if (MODE == SCORE_SCORES) {
            xs[KEEP ? blk : 0][a][r] = 0.f;
          }
        }
        if (FILTER) {
          // the heads of a token sit in GPAD/4 lanes (same n, adjacent j): combine their parts
          unsigned long long reach;
          if (per_head) {
            reach = __ballot(any_head != 0);
            if (GPAD >= 8) reach |= (reach >> 16) & 0x0000FFFF0000FFFFull;
            if (GPAD >= 16) reach |= reach >> 32;
          } else {
            if (GPAD >= 8) approx = swap16_sum(approx);
            if (GPAD >= 16) approx = swap32_sum(approx);
            reach = __ballot(!(approx < ftau));
          }
          const unsigned long long bal = reach & __ballot(tok >= p.filt.S && tok < L - p.filt.W) & kCounting;
          if (bal) {  // wave-uniform
            if (n_stash + 64 / GQ > kStash) flush();
            if ((bal >> (((j - j % GQ) << 4) | n)) & 1ull) {  // every lane of the token
              const int pos = n_stash + __popcll(bal & before_mine);
              stash_rec[wave][pos * GQ + j % GQ] = make_float4(xs[0][a][0], xs[0][a][1], xs[0][a][2], xs[0][a][3]);
              if (j % GQ == 0) stash_tok[wave][pos] = (int32_t)tok;
            }
            n_stash += __popcll(bal);
          }
        }
      }
      if (HEAVY && (FILTER ? __builtin_expect(__any(any_heavy), 0) : __any(any_heavy))) {  // wave-uniform, rare: out of the filter's straight line
        // The block is still in LDS: the fp64 logits of a 16-token tile for every head are D / 4 steps of
        // v_mfma_f64_16x16x4 on the operands at hand (element e of everybody's 16 bytes per step), about 1 us a tile.  (Listing the
        // terms and reading their keys again after the last block, sixteen lanes per dot product: 5.7 us for the chunk that holds a
        // row's sink tokens, which is what the whole launch of a small call then waits for.)  Terms strewn thin over the tiles, as logits
        // that share an offset have them, are taken one by one: with tiles alone the pass over 256 rows x 32K tokens of N(60, 1) logits took
        // 688 us instead of 463 at N(0, 1), so 467 (with the list, and the other kernels of that time, 612).
        seen_heavy = true;
        unsigned long long hv[NACC][4];  // lanes whose logit is a heavy term: lane (j', n), register r: head 4 (j' % GQ) + r
#pragma unroll
        for (int a = 0; a < NACC; ++a)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            hv[a][r] = __ballot(tok_base + (a * TILES + (4 * j) / GPAD) * 16 + n < L && hbase + r < gb && xs[0][a][r] >= hthr[r]);
        // a term's logit l into the sums of its head, in the lane of its column
        auto add = [](double& hm, double& hz, bool take, double l) {
          double ex = 0.0;
          if (__any(take && hz > 0.0)) ex = exp(l > hm ? hm - l : l - hm);  // (usually everybody's first)
          if (take) {
            hz = l > hm ? hz * ex + 1.0 : hz + ex;
            hm = l > hm ? l : hm;
          }
        };
#pragma unroll 1
        for (int a = 0; a < NACC; ++a) {
          unsigned long long h[4], any = 0ull;
          int rounds = 0, tiles = 0;  // terms in the fullest register, tiles that hold any
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            h[r] = hv[0][r];
#pragma unroll
            for (int aa = 1; aa < NACC; ++aa) h[r] = a == aa ? hv[aa][r] : h[r];
            any |= h[r];
            const int cnt = __popcll(h[r]);
            rounds = cnt > rounds ? cnt : rounds;
          }
          if (!any) continue;
          constexpr unsigned long long kTile = GQ < 4 ? (1ull << (16 * GQ % 64)) - 1ull : ~0ull;  // the lanes of a tile's rows
#pragma unroll
          for (int ts = 0; ts < TILES; ++ts) tiles += (any >> (16 * GQ * ts)) & kTile ? 1 : 0;
          if (rounds <= kThin * tiles) {
            // one by one: dot products on the vector ALU, four at a time, those of heads j + 4 i by the 16 lanes of group j
            unsigned long long left = j == 0 ? h[0] : j == 1 ? h[1] : j == 2 ? h[2] : h[3];
#pragma unroll 1
            for (; rounds > 0; --rounds) {
              const bool have = left != 0ull;
              const int bit = have ? __ffsll(left) - 1 : 0, i = (bit >> 4) % GQ, t = (a * TILES + (bit >> 4) / GQ) * 16 + (bit & 15);
              left &= left - 1ull;
              const int c = n * CH / 16;  // this lane's 16 bytes of the key; 64 dims: the lower or the upper half of them
              uint4 kb = buf[t * CH + (c ^ (t & (CH - 1)))], qb;
              const int from = ((c & 3) << 4) | (4 * i + j);  // the lane that holds the query's
#pragma unroll
              for (int kc = 0; kc < KSTEPS; ++kc) {
                const uint4 x = make_uint4(__shfl(qa[kc].x, from), __shfl(qa[kc].y, from), __shfl(qa[kc].z, from), __shfl(qa[kc].w, from));
                if (kc == 0 || c >> 2 == kc) qb = x;
              }
              if (CH == 8 && (n & 1)) kb.x = kb.z, kb.y = kb.w, qb.x = qb.z, qb.y = qb.w;
              double l = (double)bf16_lo(qb.x) * (double)bf16_lo(kb.x) + (double)bf16_hi(qb.x) * (double)bf16_hi(kb.x) +
                         (double)bf16_lo(qb.y) * (double)bf16_lo(kb.y) + (double)bf16_hi(qb.y) * (double)bf16_hi(kb.y);
              if (CH == 16)
                l += (double)bf16_lo(qb.z) * (double)bf16_lo(kb.z) + (double)bf16_hi(qb.z) * (double)bf16_hi(kb.z) +
                     (double)bf16_lo(qb.w) * (double)bf16_lo(kb.w) + (double)bf16_hi(qb.w) * (double)bf16_hi(kb.w);
              l = group_sum_f64<16>(l) * (1.0 / sqrt((double)D));
              double hm = heavy_m[0], hz = heavy_z[0];
#pragma unroll
              for (int ii = 1; ii < GQ; ++ii) hm = i == ii ? heavy_m[ii] : hm, hz = i == ii ? heavy_z[ii] : hz;
              add(hm, hz, have && n == (bit & 15), l);
#pragma unroll
              for (int ii = 0; ii < GQ; ++ii)
                if (i == ii) heavy_m[ii] = hm, heavy_z[ii] = hz;
            }
            continue;
          }
#pragma unroll 1
          for (int ts = 0; ts < TILES; ++ts) {
            if (!((any >> (16 * GQ * ts)) & kTile)) continue;
            typedef double f64x4_t __attribute__((ext_vector_type(4)));
            f64x4_t d = {0.0, 0.0, 0.0, 0.0};  // register i of lane (j, n): row 4 i + j = head (4 i + j) % GPAD, token n
#pragma unroll
            for (int kc = 0; kc < KSTEPS; ++kc) {
              const uint4 b = buf[((a * TILES + ts) * 16 + n) * CH + ((4 * kc + j) ^ (n & (CH - 1)))];
              uint32_t qw[4] = {qa[kc].x, qa[kc].y, qa[kc].z, qa[kc].w};
              const uint32_t bw[4] = {b.x, b.y, b.z, b.w};
              asm volatile("" : "+v"(qw[0]), "+v"(qw[1]), "+v"(qw[2]), "+v"(qw[3]));  // not converted (and held) up front
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_lo(qw[e]), (double)bf16_lo(bw[e]), d, 0, 0, 0);
                d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_hi(qw[e]), (double)bf16_hi(bw[e]), d, 0, 0, 0);
              }
            }
            const unsigned long long own = j == 0 ? h[0] : j == 1 ? h[1] : j == 2 ? h[2] : h[3];  // heads j + 4 i
#pragma unroll kAddUnroll
            for (int i = 0; i < GQ; ++i) {
              double hm = heavy_m[0], hz = heavy_z[0], l = d[0];
#pragma unroll
              for (int ii = 1; ii < GQ; ++ii) hm = i == ii ? heavy_m[ii] : hm, hz = i == ii ? heavy_z[ii] : hz, l = i == ii ? d[ii] : l;
              add(hm, hz, (own >> (16 * (GQ * ts + i) + n)) & 1ull, l * (1.0 / sqrt((double)D)));
#pragma unroll
              for (int ii = 0; ii < GQ; ++ii)
                if (i == ii) heavy_m[ii] = hm, heavy_z[ii] = hz;
            }
          }
        }
      }
      // one block ahead is enough, and all that the registers of two workgroups per CU hold: without this the passes
      // that have no branch here load two blocks ahead (300-400 registers, one workgroup per CU)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the heavy terms join the sums of the lanes that hold their heads (the staging buffer is free after the last block)
  if (HEAVY && seen_heavy) {
    double2* hb = reinterpret_cast<double2*>(buf);  // [head][token column]
    static_assert(GPAD * 16 * sizeof(double2) <= sizeof(lds[0]), "heavy sums fit the staging buffer");
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int i = 0; i < GQ; ++i) hb[(j + 4 * i) * 16 + n] = make_double2(heavy_m[i], heavy_z[i]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
    for (int r = 0; r < 4; ++r) {
      const double2 h = hb[((4 * j) % GPAD + r) * 16 + n];
      if (j < GQ && h.y > 0.0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i == r) {
            const float mn = fmaxf(m[i], (float)h.x);
            const double x = h.x - (double)mn;  // usually the rounding of the maximum: the exponential's series to x^3
            double ex = 1.0 + x * (1.0 + x * (0.5 + x * (1.0 / 6.0)));
            if (__any(fabs(x) > 0x1p-10)) ex = exp(x);
            sum[i] = sum[i] * exp_fast(m[i] - mn) + (float)(h.y * ex);
            m[i] = mn;
          }
      }
    }
  }
  if (MODE == SCORE_LOGITS) {
#pragma unroll
    for (int blk = 0; blk < BPW; ++blk) {
      const bool in = wave_base + (int64_t)blk * kBlockStride < L;  // wave-uniform: the block exists
#pragma unroll
      for (int a = 0; a < NACC; ++a) {
        const int64_t tok = wave_base + (int64_t)blk * kBlockStride + (a * TILES + (4 * j) / GPAD) * 16 + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float& x = xs[KEEP ? blk : 0][a][r];
          if (in && tok < L && hbase + r < gb) {
            float* at = p.logits + logit_index(p.geo, p.n_chunks, p.chunk, row, p.g0 + hbase + r, tok);
            if (GPAD == 4 && p.logits_through)
              __hip_atomic_store(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
              *at = x;
          } else {
            x = -INFINITY;
          }
        }
      }
    }
    // softmax partial of the chunk: lanes -> row blocks of 16 -> workgroup
    __shared__ double part_z[MODE == SCORE_LOGITS ? kScoreWaves : 1][4][4];
    const int j0 = (hbase / 4), jstep = GPAD / 4;  // the row blocks that share this one's heads
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float M = -INFINITY;
#pragma unroll
      for (int blk = 0; blk < BPW; ++blk)
#pragma unroll
        for (int a = 0; a < NACC; ++a) M = fmaxf(M, xs[KEEP ? blk : 0][a][r]);
      M = group16_max(M);
      if (n == 0) part[wave][j][r].x = M;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float M = -INFINITY;
#pragma unroll
      for (int w = 0; w < kScoreWaves; ++w)
#pragma unroll
        for (int jj = 0; jj < 4; jj += jstep) M = fmaxf(M, part[w][j0 + jj][r].x);
      M = M == -INFINITY ? 0.f : M;  // nothing but -inf (heads past the group among them): the sum is 0
      double z = 0.0;
#pragma unroll
      for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int blk = 0; blk < BPW; ++blk) z += (double)exp_fast(xs[KEEP ? blk : 0][a][r] - M);
      z = group_sum_f64<16>(z);
      if (n == 0) part_z[wave][j][r] = z;
    }
    __syncthreads();
    if ((int)threadIdx.x < gb) {
      const int g = threadIdx.x;
      float M = -INFINITY;
      double z = 0.0;
      for (int w = 0; w < kScoreWaves; ++w)
        for (int jj = 0; jj < 4; jj += jstep) {
          M = fmaxf(M, part[w][g / 4 + jj][g % 4].x);
          z += part_z[w][g / 4 + jj][g % 4];
        }
      p.chunk_partials[((int64_t)row * p.geo.G + p.g0 + g) * p.n_chunks + chunk] = ChunkPartial{z, M, 0.f};
    }
    return;
  }
  if (MODE == SCORE_SCORES) {
    // xs holds exp(l - M) / Z of this lane's heads.  One list per row: the group's sum (the lanes that
    // share a token add up, ascending heads within a lane); one list per head: each value is a score.
    __shared__ int hist[kHistBins];
    const bool per_q = p.n_lists > 1;
    const bool rep = (4 * j) % GPAD == 0;
    const int64_t cand_lo = p.S, cand_hi = L - p.W;
    if (!per_q) {
#pragma unroll
      for (int blk = 0; blk < BPW; ++blk)
#pragma unroll
        for (int a = 0; a < NACC; ++a) {
          float v = (xs[KEEP ? blk : 0][a][0] + xs[KEEP ? blk : 0][a][1]) + (xs[KEEP ? blk : 0][a][2] + xs[KEEP ? blk : 0][a][3]);
          if (GPAD >= 8) v += __shfl_xor(v, 16);
          if (GPAD >= 16) v += __shfl_xor(v, 32);
          xs[KEEP ? blk : 0][a][0] = v;
        }
    }
    const int n_pass = per_q ? gb : 1;  // histogram passes: one list at a time through the LDS histogram
    for (int li = 0; li < n_pass; ++li) {
      for (int b = threadIdx.x; b < kHistBins; b += kScoreThreads) hist[b] = 0;
      __syncthreads();
      const int64_t list = (int64_t)row * p.n_lists + (per_q ? p.g0 + li : 0);
      float* out = p.scores + list * p.pitch;
      // the lane that holds this list's value of a token: the counting lane (sum), or head li's lane and register
      const bool mine = per_q ? (hbase <= li && li < hbase + 4) : rep;
      const int r_sel = per_q ? (li - hbase) & 3 : 0;
#pragma unroll
      for (int blk = 0; blk < BPW; ++blk)
#pragma unroll
        for (int a = 0; a < NACC; ++a) {
          const int64_t tok = wave_base + (int64_t)blk * kBlockStride + (a * TILES + (4 * j) / GPAD) * 16 + n;
          float v = xs[KEEP ? blk : 0][a][0];
          if (per_q) {
            v = r_sel == 1 ? xs[KEEP ? blk : 0][a][1] : v;
            v = r_sel == 2 ? xs[KEEP ? blk : 0][a][2] : v;
            v = r_sel == 3 ? xs[KEEP ? blk : 0][a][3] : v;
          }
          if (mine && tok < L) {
            out[tok] = v;
            if (tok >= cand_lo && tok < cand_hi) atomicAdd(&hist[(__float_as_uint(v) >> 20) & (kHistBins - 1)], 1);
          }
        }
      __syncthreads();
      int* gh = p.ghist + list * kHistBins;
      for (int b = threadIdx.x; b < kHistBins; b += kScoreThreads) {
        const int v = hist[b];
        if (v) atomicAdd(&gh[b], v);
      }
      __syncthreads();
    }
    return;
  }

  if (FILTER && n_stash) flush();
  // (max, sum) of the chunk: the 16 lanes of a row block share their heads
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float M = group16_max(m[r]);
    float sm = (m[r] == -INFINITY) ? 0.f : sum[r] * exp_fast(m[r] - M);
    sm = group_sum<16>(sm);
    if (n == 0) part[wave][j][r] = make_float2(M, sm);
  }
  __syncthreads();
  // the chunk's line, whole: thread t writes word t
  const int words = chunk_line_words(p.geo.G), t = threadIdx.x;
  if (t < words) {
    float v = 0.f;
    if (t < 2 * gb) {
      const int g = t >> 1;
      float2 pw[kScoreWaves][16 / GPAD];
      float M = -INFINITY, sm = 0.f;
#pragma unroll
      for (int w = 0; w < kScoreWaves; ++w)
#pragma unroll
        for (int ts = 0; ts < TILES; ++ts) {
          pw[w][ts] = part[w][ts * GQ + g / 4][g % 4];
          M = fmaxf(M, pw[w][ts].x);
        }
#pragma unroll
      for (int w = 0; w < kScoreWaves; ++w)
#pragma unroll
        for (int ts = 0; ts < TILES; ++ts) sm += (pw[w][ts].x == -INFINITY) ? 0.f : pw[w][ts].y * exp_fast(pw[w][ts].x - M);
      v = t & 1 ? sm : M;
    }
    if (FILTER && t == words - 1) v = __int_as_float(n_kept_wg);
    p.lines[((int64_t)row * p.n_chunks + chunk) * words + t] = v;
  }
}

// Workgroups per CU that the registers are held to.  The filter and the partials over chunks of 1024 tokens of 64 dims: three, 168
// registers, at the price of up to 20 spilled ones in the code for heavy terms with 9 to 16 heads (3 with 5 to 8); left alone they take 173 and 187,
// and two workgroups.  256 rows x 32K tokens x 16 heads, two and three, us: N(0, 1) logits 390 and 372, queries x 6 547 and 494, N(60, 1) 650 and
// 564; 7 heads 305 and 284, 365 and 347, 397 and 352; scores of 16 heads 499 and 477, 582 and 517, 751 and 667.  Smaller chunks are for calls
// that do not fill three.
template <int D, int GPAD, int MODE, int BPW>
constexpr int score_workgroups() {
  if (GPAD == 16 && (MODE == SCORE_LOGITS || MODE == SCORE_SCORES)) return 1;  // every token's values are held to the end
  return D == 64 && BPW == 4 && (MODE == SCORE_FILTER || MODE == SCORE_PARTIALS) ? 3 : 2;
}

// grid (chunks, rows).  A gated launch (rows the pre-filter could not certify, usually none) has a
// few y-blocks only, each walking over all rows and working on the flagged ones: an empty launch
// then costs a handful of workgroups instead of one per (chunk, row).
template <int D, int GPAD, int MODE, bool PAGED, int BPW>
__global__ __launch_bounds__(kScoreThreads, (score_workgroups<D, GPAD, MODE, BPW>())) void score_mfma_kernel(ScoreParams p, int gb) {
  if (MODE != SCORE_FILTER && p.gate.row_flag) {
    if (*p.gate.n_flagged == 0) return;  // the usual case: nothing to redo
    const int rows = p.geo.n_problems * p.geo.Hkv;
    for (int row = blockIdx.y; row < rows; row += gridDim.y) {
      if (p.gate.row_flag[row] == 0) continue;  // workgroup-uniform
      score_mfma_chunk<D, GPAD, MODE, PAGED, BPW>(p, gb, row, (int)blockIdx.x);
      __syncthreads();  // the chunk's last LDS reads, before the next row's writes
    }
    return;
  }
  // Workgroups go to the eight XCDs in turn.  Where a row has a multiple of eight chunks, its first one (the sink
  // tokens: heavy terms, a longer tail) would always meet the same XCD: the first eight chunks are rotated by the row.
  // (All chunks rotated: 1.41 instead of 1.28 ms at 256 rows x 128 chunks, the stream over K loses its order.)
  const unsigned chunk = blockIdx.x < 8 && gridDim.x >= 8 ? (blockIdx.x + blockIdx.y) & 7u : blockIdx.x;
  score_mfma_chunk<D, GPAD, MODE, PAGED, BPW>(p, gb, (int)blockIdx.y, (int)chunk);
}

// Logits of the sampled blocks (fast path): one wave per 64-token block, logits to samp_logit[row][slot][Gs] (16 bytes per
// lane).  A block is four tiles of 16 consecutive tokens (sample_token), and a lane loads its MFMA B operands straight from
// memory: the four (two) 64-byte pieces of a token go to four lanes, and the tile's 4 (2) KB are one run all the same; no LDS,
// little code, the pages of a lane's four tokens looked up together (with a table load in front of every load of keys the
// stage took 29 us instead of 23 for 64 rows x 40K tokens in pages).
// Plain loads: nontemporal ones take 37 instead of 49 us over 256 rows x 32K tokens, but the filtering pass after them then
// takes 370 instead of 343 (over 256 x 128K 52 and 75, 1400 and 1270): it is left to push out what the last writer's lines hold of the
// Infinity Cache.
template <int D, int GPAD, bool PAGED>
__global__ __launch_bounds__(kScoreThreads, 4) void sample_logits_kernel(SampleParams p) {
  constexpr int KSTEPS = D / 32, TILES = 16 / GPAD, NACC = 4 / TILES;
  const int row = blockIdx.y;
  const int prob = row / p.geo.Hkv, c = row % p.geo.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, j = lane >> 4;
  const int64_t L = p.geo.L;
  const int blk = blockIdx.x * kScoreWaves + wave;
  if (blk >= p.nA + p.nB + p.nC) return;  // wave-uniform; no workgroup barrier below
  const char* base = (const char*)p.K + ((PAGED ? 0 : (int64_t)prob * p.ks_problem) + (int64_t)c * p.ks_head) * 2 + 16 * j;
  int64_t at[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    int64_t tok = sample_token(p, blk, 16 * t) + n;
    tok = tok < 0 ? 0 : (tok < L ? tok : L - 1);
    at[t] = PAGED ? (int64_t)page_of(p.pm, prob, tok) * p.pm.ks_page + (tok & ((1 << p.pm.shift) - 1)) * p.ks_token : tok * p.ks_token;
  }
  uint4 kv[4][KSTEPS];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int kc = 0; kc < KSTEPS; ++kc) kv[t][kc] = ld16(base + at[t] * 2 + 64 * kc);
  const int my_head = n % GPAD, tslot = (4 * j) / GPAD;
  uint4 qa[KSTEPS];
#pragma unroll
  for (int kc = 0; kc < KSTEPS; ++kc) {
    qa[kc] = make_uint4(0u, 0u, 0u, 0u);
    if (my_head < p.geo.G) qa[kc] = ld16((const char*)p.q_last + (((int64_t)prob * p.geo.Hq + c * p.geo.G + my_head) * D + (4 * kc + j) * 8) * 2);
  }
  const int hbase = (4 * j) % GPAD;
  float* out = p.samp_logit + ((int64_t)row * (p.nA + p.nB + p.nC) + blk) * 64 * GPAD;
#pragma unroll
  for (int a = 0; a < NACC; ++a) {
    f32x4_t acc;  // as in score_mfma_chunk: every tile's product holds all heads, a lane takes the tile of its slot
#pragma unroll
    for (int ts = 0; ts < TILES; ++ts) {
      f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < KSTEPS; ++kc)
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qa[kc]), __builtin_bit_cast(bf16x8_t, kv[a * TILES + ts][kc]), d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = ts == 0 || tslot == ts ? d[r] : acc[r];
    }
    *reinterpret_cast<float4*>(out + ((a * TILES + tslot) * 16 + n) * GPAD + hbase) =
        make_float4(acc[0] * p.scale, acc[1] * p.scale, acc[2] * p.scale, acc[3] * p.scale);
  }
}

__global__ __launch_bounds__(64) void stats_kernel(StatsParams p) {
  const int lane = threadIdx.x, row = blockIdx.x;
  if (p.ghist)
    for (int b = lane; b < kHistBins * p.n_lists; b += 64) p.ghist[(int64_t)row * p.n_lists * kHistBins + b] = 0;
  for (int g = 0; g < p.G; ++g) {
    const int stride = chunk_line_words(p.G);
    const float* pr = p.lines + (int64_t)row * p.n_chunks * stride + 2 * g;
    const RowStat st = merge_partials_wave(load_partials(pr, stride, p.n_chunks), pr, stride, p.n_chunks);
    if (lane == 0) p.stats[(int64_t)row * p.G + g] = st;
  }
}

constexpr int kCombineThreads = 256;
constexpr int kMaxG = 64;

__global__ __launch_bounds__(kCombineThreads) void combine_kernel(CombineParams p) {
  __shared__ int hist[kHistBins];
  __shared__ float sM[kMaxG], sInv[kMaxG];
  const int tid = threadIdx.x;
  const int row = blockIdx.y;
  const int G = p.geo.G;
  const int64_t L = p.geo.L;
  for (int b = tid; b < kHistBins; b += kCombineThreads) hist[b] = 0;
  if (tid < G) {
    RowStat st = p.stats[(int64_t)row * G + tid];
    sM[tid] = st.M;
    sInv[tid] = st.invZ;
  }
  __syncthreads();
  // group-sum: one score row per KV head; per-query: blockIdx.z picks the head, one row each
  const int g_lo = p.n_lists > 1 ? blockIdx.z : 0, g_hi = p.n_lists > 1 ? g_lo + 1 : G;
  const int64_t list = (int64_t)row * p.n_lists + (p.n_lists > 1 ? g_lo : 0);
  float* out = p.scores + list * p.pitch;
  const int64_t cand_lo = p.S, cand_hi = L - p.W;
  const bool vec_out = (p.pitch & 3) == 0;
  const int64_t base = (int64_t)blockIdx.x * kCombineChunk;
#pragma unroll
  for (int it = 0; it < kCombineChunk / (kCombineThreads * 4); ++it) {
    const int64_t tok = base + (int64_t)it * kCombineThreads * 4 + tid * 4;
    if (tok >= L) break;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int g = g_lo; g < g_hi; ++g) {
      const float4 x = *reinterpret_cast<const float4*>(p.logits + logit_index(p.geo, p.n_chunks, p.chunk, row, g, tok));
      const float M = sM[g], inv = sInv[g];
      acc[0] += exp_times(x.x - M, inv);
      acc[1] += exp_times(x.y - M, inv);
      acc[2] += exp_times(x.z - M, inv);
      acc[3] += exp_times(x.w - M, inv);
    }
    if (vec_out && tok + 3 < L) {
      *reinterpret_cast<float4*>(out + tok) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (tok + j < L) out[tok + j] = acc[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t t = tok + j;
      if (t >= cand_lo && t < cand_hi) atomicAdd(&hist[(__float_as_uint(acc[j]) >> 20) & (kHistBins - 1)], 1);
    }
  }
  __syncthreads();
  int* gh = p.ghist + list * kHistBins;
  for (int b = tid; b < kHistBins; b += kCombineThreads) {
    int v = hist[b];
    if (v) atomicAdd(&gh[b], v);
  }
}

template <int D, int BPW>
hipError_t launch_score_g(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  switch (gb) {
#define SAGEKV_CASE(N) \
  case N:              \
    hipLaunchKernelGGL((score_f32_kernel<D, N, BPW>), grid, dim3(kScoreThreads), 0, s, p); \
    break;
    SAGEKV_CASE(1) SAGEKV_CASE(2) SAGEKV_CASE(3) SAGEKV_CASE(4)
    SAGEKV_CASE(5) SAGEKV_CASE(6) SAGEKV_CASE(7) SAGEKV_CASE(8)
#undef SAGEKV_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_score_f32(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  switch (p.chunk) {
    case 256: return launch_score_g<D, 1>(p, gb, grid, s);
    case 512: return launch_score_g<D, 2>(p, gb, grid, s);
    default: return hipErrorInvalidValue;
  }
}

template <int D, int MODE, bool PAGED, int BPW>
hipError_t launch_score_mfma_p(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  if (gb <= 4)
    hipLaunchKernelGGL((score_mfma_kernel<D, 4, MODE, PAGED, BPW>), grid, dim3(kScoreThreads), 0, s, p, gb);
  else if (gb <= 8)
    hipLaunchKernelGGL((score_mfma_kernel<D, 8, MODE, PAGED, BPW>), grid, dim3(kScoreThreads), 0, s, p, gb);
  else
    hipLaunchKernelGGL((score_mfma_kernel<D, 16, MODE, PAGED, BPW>), grid, dim3(kScoreThreads), 0, s, p, gb);
  return hipGetLastError();
}

template <int D, int MODE, int BPW>
hipError_t launch_score_mfma_b(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  return p.pm.table ? launch_score_mfma_p<D, MODE, true, BPW>(p, gb, grid, s)
                    : launch_score_mfma_p<D, MODE, false, BPW>(p, gb, grid, s);
}

template <int D, int MODE>
hipError_t launch_score_mfma(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  if constexpr (MODE != SCORE_SCORES) {
    if (p.chunk == 256) return launch_score_mfma_b<D, MODE, 1>(p, gb, grid, s);
    if (p.chunk == 512) return launch_score_mfma_b<D, MODE, 2>(p, gb, grid, s);
  }
  return launch_score_mfma_b<D, MODE, kScoreChunk / (64 * kScoreWaves)>(p, gb, grid, s);
}

template <int MODE>
hipError_t launch_score_mfma_d(const ScoreParams& p, int gb, dim3 grid, hipStream_t s) {
  return p.geo.D == 128 ? launch_score_mfma<128, MODE>(p, gb, grid, s) : launch_score_mfma<64, MODE>(p, gb, grid, s);
}

}  // namespace

// Fast path: bf16, G <= 16 (one launch covers the group).
hipError_t launch_score_filter(const ScoreParams& p0, hipStream_t s) {
  const int rows = p0.geo.n_problems * p0.geo.Hkv;
  dim3 grid((unsigned)p0.n_chunks, (unsigned)rows);
  ScoreParams p = p0;
  p.g0 = 0;
  p.gate.row_flag = nullptr;
  if (p.geo.dtype != DT_BF16 || p.geo.G > 16) return hipErrorInvalidValue;
  p.filt.write_through = (int64_t)rows * p.geo.L * p.geo.D * 2 > kWriteThrough;
  return launch_score_mfma_d<SCORE_FILTER>(p, p.geo.G, grid, s);
}

hipError_t launch_sample_logits(const SampleParams& p, hipStream_t s) {
  const int rows = p.geo.n_problems * p.geo.Hkv;
  const int nb = p.nA + p.nB + p.nC;
  if (p.geo.dtype != DT_BF16 || p.geo.G > 16) return hipErrorInvalidValue;
  dim3 grid((unsigned)((nb + kScoreWaves - 1) / kScoreWaves), (unsigned)rows);
#define SAGEKV_LAUNCH(DD, GP)                                                                                  \
  if (p.pm.table)                                                                                               \
    hipLaunchKernelGGL((sample_logits_kernel<DD, GP, true>), grid, dim3(kScoreThreads), 0, s, p);               \
  else                                                                                                          \
    hipLaunchKernelGGL((sample_logits_kernel<DD, GP, false>), grid, dim3(kScoreThreads), 0, s, p)
  if (p.geo.D == 128) {
    if (p.geo.G <= 4) {
      SAGEKV_LAUNCH(128, 4);
    } else if (p.geo.G <= 8) {
      SAGEKV_LAUNCH(128, 8);
    } else {
      SAGEKV_LAUNCH(128, 16);
    }
  } else {
    if (p.geo.G <= 4) {
      SAGEKV_LAUNCH(64, 4);
    } else if (p.geo.G <= 8) {
      SAGEKV_LAUNCH(64, 8);
    } else {
      SAGEKV_LAUNCH(64, 16);
    }
  }
#undef SAGEKV_LAUNCH
  return hipGetLastError();
}

int max_group_per_launch() { return 8; }

// Dense passes.  bf16: any mode, gated or not; fp32 caches: SCORE_LOGITS over every row only.
hipError_t launch_score(const ScoreParams& p0, ScoreMode mode, hipStream_t s) {
  const int rows = p0.geo.n_problems * p0.geo.Hkv;
  const bool bf16 = p0.geo.dtype == DT_BF16;
  if (mode == SCORE_FILTER || (!bf16 && (mode != SCORE_LOGITS || p0.gate.row_flag))) return hipErrorInvalidValue;
  // scores: whole kScoreChunk chunks, whatever the first pass used; the others p.chunk tokens per workgroup
  const unsigned nx = mode == SCORE_SCORES ? (unsigned)((p0.geo.L + kScoreChunk - 1) / kScoreChunk) : (unsigned)p0.n_chunks;
  dim3 grid(nx, (unsigned)(p0.gate.row_flag && rows > kGatedRowBlocks ? kGatedRowBlocks : rows));
  const int per_launch = bf16 ? 16 : max_group_per_launch();
  for (int g0 = 0; g0 < p0.geo.G; g0 += per_launch) {
    ScoreParams p = p0;
    p.g0 = g0;
    const int gb = p0.geo.G - g0 < per_launch ? p0.geo.G - g0 : per_launch;
    hipError_t e;
    if (!bf16)
      e = p.geo.D == 128 ? launch_score_f32<128>(p, gb, grid, s) : launch_score_f32<64>(p, gb, grid, s);
    else if (mode == SCORE_LOGITS) {
      p.logits_through = gb <= 4 && (int64_t)rows * p.geo.L * p.geo.D * 2 > kLogitsThrough;
      e = launch_score_mfma_d<SCORE_LOGITS>(p, gb, grid, s);
    } else if (mode == SCORE_PARTIALS)
      e = launch_score_mfma_d<SCORE_PARTIALS>(p, gb, grid, s);
    else
      e = launch_score_mfma_d<SCORE_SCORES>(p, gb, grid, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_stats(const StatsParams& p, int rows, hipStream_t s) {
  hipLaunchKernelGGL(stats_kernel, dim3((unsigned)rows), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_combine(const CombineParams& p, hipStream_t s) {
  const int rows = p.geo.n_problems * p.geo.Hkv;
  const unsigned nx = (unsigned)((p.geo.L + kCombineChunk - 1) / kCombineChunk);
  hipLaunchKernelGGL(combine_kernel, dim3(nx, (unsigned)rows, (unsigned)p.n_lists), dim3(kCombineThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace sagekv
