// Decoding over the reduced cache (paper Sec. 2 Step 4): the new token's (k, v) replaces the
// oldest entry of the recent window, then every query head attends over the reduced row.
//
// decode_*_kernel: grid (splits, rows).  A workgroup streams its slice of Kc and Vc once for all
// G heads of the row (16-byte loads), keeps an online softmax per wave or lane
// group and merges them -> workgroup.  With one split per row (many rows: all
// layers of a step in one launch) one workgroup (usually 8 waves) owns the whole row and
// writes `out` itself; with few rows the row is split, partials (max, sum, acc[G][d]) go to scratch and
// combine_kernel merges them.  (A last-workgroup-done merge inside one kernel needs a device
// scope fence in every workgroup, which on this multi-XCD part writes back and invalidates
// L2: measured ~8x slower than two launches.)  The appended token is read from k_new / v_new
// directly and stored to its slot by the workgroup that owns it, so append and attention are
// one launch.
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"

namespace sagekv {

namespace {

// Slot of the new token, attended length and slice size of this launch: the host's values, or
// derived from the device-side count of appended tokens.
struct StepGeom {
  int slot, len, tokens_per_split, n_appended;
};
// late: a fixed-size window with its count on the device.  Only the slot depends on the count, so its load need not be
// waited for in front of everything else: the first loads go out with slot = -1 and late_slot() fills it in.  (One
// layer's step, 8 rows x 4096 tokens: 15.8 -> 14.5 us together with the queries' loads in front of K's and V's and
// the maxima over DPP instead of shuffles; 11.3 with the loads of SliceLoads and the shared factors of the merge, 11.0 with its bounded loads.)
__device__ __forceinline__ bool slot_is_late(const DecodeParams& p) { return p.ring && !p.ring_grow; }
__device__ __forceinline__ int late_slot(const DecodeParams& p, StepGeom& s, int n_appended) {
  s.n_appended = n_appended;
  s.slot = p.k_new ? ring_position(p.ring_base, p.ring_W, 0, p.cap, n_appended < 0 ? 0 : n_appended).slot : -1;
  return s.slot;
}
template <bool LATE = false>
__device__ __forceinline__ StepGeom step_geom(const DecodeParams& p) {
  StepGeom s = {p.k_new ? p.slot : -1, p.len, p.tokens_per_split, 0};
  if (LATE && slot_is_late(p)) {
    s.slot = -1;
  } else if (p.ring) {
    s.n_appended = p.ring[0];
    const RingPos r = ring_position(p.ring_base, p.ring_W, p.ring_grow, p.cap, s.n_appended < 0 ? 0 : s.n_appended);
    s.slot = p.k_new ? r.slot : -1;
    s.len = r.len;
    s.tokens_per_split = split_tokens(r.len, p.n_splits);
  }
  return s;
}

// Source addresses of the 16-byte loads of a bf16 decode wave.  The wave's it-th block holds the tokens
// t_begin + (wave + it * NW) * BT ..+ BT of the row; load i covers TPL consecutive ones of them, which lie in one
// 16-token group and so in one page.  PAGED: the page ids of the next 64 groups sit in one register, a group
// per lane, filled once per 64 groups; a load takes its id by readlane.  (Looking the page up per load puts a
// table load in front of every block's K and V loads, and loads complete in order: waiting for the table
// means waiting for every K and V load already in flight.  448 rows x 8192 tokens x 7 heads in pages of 16:
// 724 us, 2.6 TB/s; with the ids in a register 294 us, 6.4 TB/s, which is what the strided layout takes.)
template <bool PAGED, int ROWB, int BT, int NW, int TPL>
struct BlockSource {
  static constexpr int GPB = BT / 16;  // 16-token groups per block
  CacheRow K, V;
  int t_begin, t_end, slot, wave, my_page;

  // page ids of the 64 groups from block it0 on (it0 * GPB a multiple of 64); every lane takes part
  __device__ __forceinline__ void fill_pages(int it0) {
    if (!PAGED) return;
    const int lane = threadIdx.x & 63;
    int tok = t_begin + (wave + (it0 + lane / GPB) * NW) * BT + (lane % GPB) * 16;
    tok = tok < t_end ? tok : t_begin;  // past the slice: its loads are clamped to t_begin as well
    const int pid = K.tab[tok >> K.shift];
    my_page = pid < 0 ? 0 : (pid >= K.n_pages ? K.n_pages - 1 : pid);
  }
  __device__ __forceinline__ bool refill_before(int it) const { return PAGED && ((it * GPB) & 63) == 0; }
  // this lane's token of load i of block it; tokens past the slice become one that is inside it: its first, in pages the first
  // of the group my_page was filled for
  __device__ __forceinline__ int token(int it, int i, int tq) const {
    const int b0 = t_begin + (wave + it * NW) * BT, tok = b0 + i * TPL + tq;
    const int g0 = b0 + (i * TPL) / 16 * 16;
    return tok < t_end ? tok : PAGED && g0 < t_end ? g0 : t_begin;
  }
  __device__ __forceinline__ const char* at(const CacheRow& r, const char* fresh, int it, int i, int tq) const {
    const int tok = token(it, i, tq);
    if (!PAGED) return tok == slot ? fresh : r.base + (int64_t)tok * ROWB;
    const int pid = __builtin_amdgcn_readlane(my_page, (it * GPB + (i * TPL) / 16) & 63);
    const char* page = r.base + (int64_t)pid * r.page_bytes;
    return tok == slot ? fresh : page + (int64_t)(tok & ((1 << r.shift) - 1)) * ROWB;
  }
  // the slot has become known after the first block was loaded without it: the lanes that hold the new token's
  // place (a lane past the slice may, through its replacement) take the new token
  template <int NLOAD>
  __device__ __forceinline__ void patch_first(uint4 (&k)[NLOAD], uint4 (&v)[NLOAD], const char* kn, const char* vn, int tq, int cl) const {
    const int b0 = t_begin + wave * BT;
    if ((slot < b0 || slot >= b0 + BT) && slot != t_begin) return;  // wave-uniform
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      if (token(0, i, tq) == slot) {
        k[i] = ld16(kn + cl * 16);
        v[i] = ld16(vn + cl * 16);
      }
  }
};

// Called once per row of a launch whose workgroups own whole rows: the last row to finish advances
// the device-side count (for sliced rows the merge launch does).  Every wave has read ring[0] and used the value (in its
// addresses, or, where the slot is late, in the slot's comparison) before the barriers that come before this, so the store
// cannot overtake a reader; a launch without a new token uses it only here, in the one thread that stores.  The next launch
// on the stream sees it.  Only the counter itself is exchanged between workgroups: relaxed atomics, no
// cache-wide fence.
__device__ __forceinline__ void row_done(const DecodeParams& p, const StepGeom& sg) {
  if (!p.ring || !p.ring_advance) return;
  const int rows = (int)gridDim.y;
  const int ticket = __hip_atomic_fetch_add(&p.ring[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (ticket == rows - 1) {
    __hip_atomic_store(&p.ring[1], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p.ring[0], sg.n_appended + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// End of a decode workgroup that owns its whole row: the row is done.  (Sliced rows are completed
// by the merge launch.)
__device__ __forceinline__ void finish_row(const DecodeParams& p, const StepGeom& sg) {
  if (p.n_splits == 1 && threadIdx.x == 0) row_done(p, sg);
}

// fp32 caches.  Both products and the sums in fp64 (an fp32 logit of magnitude 100 would be off by 2.5e-5, and so would its softmax weight);
// fp64 and fp32 multiply-adds take the same four cycles.  Bound by vector instructions, so nothing is done twice: eight lanes share a
// token (four, or two, 16-byte chunks each), a logit's eight parts are summed while heads and lanes change places, and lane s of the eight ends
// with head s's logit, whose weight it computes once and leaves in LDS for the lanes that hold V's chunks (16 bytes of a token each).
// A wave works on blocks of 16 or 32 tokens.  (With 16 or 32 lanes per token, every head's logit summed over all of them and its weight
// computed in all of them, fp32 accumulators, and that kernel now, us: 2 rows x 2 heads x 256 tokens of 64 dims 7.5 and 6.7, 8 rows x 4 x
// 512 of 128 18.5 and 9.7, 4 x 7 x 2048 28.4 and 12.2, 256 x 4 x 4096 281 and 188, 128 x 7 x 2048 132 and 85.5, in pages 256 x 4 x 2048 233
// and 103; errors 5 to 30 % smaller.)
template <int D, int GB, int NW, int BT, bool PG>
__global__ __launch_bounds__(NW * 64) void decode_f32_kernel(DecodeParams p, int g0) {
  constexpr int ROWB = D * 4, CH = D / 4, GPB = BT / 16;
  constexpr bool LATE_V = GB >= 6;  // V's block after the logits, not with K's: else registers spill
  constexpr int NG = BT / 8, NC = CH / 8;             // K: groups of 8 tokens, a lane's chunks of a token
  constexpr int TPL = 64 / CH, NV = BT / TPL;         // V: tokens per load, loads
  constexpr int GP = (GB + 1) / 2 * 2;                // weights of a token in LDS: whole 16-byte pairs
  constexpr int kThreads = NW * 64, NQ = (GB * D + kThreads - 1) / kThreads;
  __shared__ __attribute__((aligned(16))) double qd[2][GB * D];  // queries; 1: the one the sink tokens are scored with
  __shared__ __attribute__((aligned(16))) double pw[NW][BT][GP];
  __shared__ uint4 s_new[2 * CH];  // the new token's key and value
  __shared__ float s_acc[NW][GB][D];
  __shared__ float s_m[NW][GB];
  __shared__ double s_l[NW][GB];

  const int row = blockIdx.y, split = blockIdx.x;
  const int prob = row / p.Hkv, c = row % p.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t8 = lane >> 3, sl = lane & 7;   // K role: token of a group, share of a token; head, once the logits are summed
  const int tq = lane / CH, cl = lane % CH;  // V role: token of a load, chunk
  const int64_t head0 = (int64_t)prob * p.Hq + c * p.G + g0;

  StepGeom sg = step_geom<true>(p);
  int ring_n = 0;
  if (slot_is_late(p)) ring_n = p.ring[0];  // on its way while the first loads are issued
  const int t_begin = split * sg.tokens_per_split;
  const int t_end = min(sg.len, t_begin + sg.tokens_per_split);
  const int nblk = (t_end - t_begin + BT - 1) / BT;
  const CacheRow Kr = cache_row(p.Kc, p.cpm, false, prob, c, row, p.cap, ROWB, 4);
  const CacheRow Vr = cache_row(p.Vc, p.cpm, true, prob, c, row, p.cap, ROWB, 4);

  // loads complete in order: the queries first, then the new token, then K and V
  float qv[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int at = tid + i * kThreads;
    qv[i] = at < GB * D ? ((const float*)p.q)[head0 * D + at] : 0.f;
  }
  const bool value = tid >= CH;  // threads 0 .. 2 CH - 1: a chunk of the new key or value
  uint4 fresh = make_uint4(0u, 0u, 0u, 0u);
  if (p.k_new && tid < 2 * CH) fresh = ld16((const char*)(value ? p.v_new : p.k_new) + (int64_t)row * ROWB + (tid % CH) * 16);
  // PG: page ids of the 64 groups of 16 tokens from block it0 on, one per lane
  int my_page = 0;
  auto fill_pages = [&](int it0) {
    int tok = t_begin + (wave + (it0 + lane / GPB) * NW) * BT + (lane % GPB) * 16;
    tok = tok < t_end ? tok : t_begin;
    const int pid = Kr.tab[tok >> Kr.shift];
    my_page = pid < 0 ? 0 : (pid >= Kr.n_pages ? Kr.n_pages - 1 : pid);
  };
  // token `at` of block it (at - lane's part is wave-uniform: `base`); past the slice one that is inside it
  auto token = [&](int it, int base, int at) {
    const int b0 = t_begin + (wave + it * NW) * BT, g16 = b0 + base / 16 * 16;
    return b0 + at < t_end ? b0 + at : PG && g16 < t_end ? g16 : t_begin;
  };
  auto address = [&](const CacheRow& r, int it, int base, int tok) -> const char* {
    if (!PG) return r.base + (int64_t)tok * ROWB;
    const int pid = __builtin_amdgcn_readlane(my_page, (it * GPB + base / 16) & 63);
    return r.base + (int64_t)pid * r.page_bytes + (int64_t)(tok & ((1 << r.shift) - 1)) * ROWB;
  };
  uint4 kv[NG][NC], vv[NV];
  auto load_k = [&](int it) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const char* a = address(Kr, it, 8 * g, token(it, 8 * g, 8 * g + t8)) + sl * 16;
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) kv[g][ch] = ld16(a + ch * 128);
    }
  };
  auto load_v = [&](int it) {
#pragma unroll
    for (int i = 0; i < NV; ++i) vv[i] = ld16(address(Vr, it, i * TPL, token(it, i * TPL, i * TPL + tq)) + cl * 16);
  };
  if (wave < nblk) {
    if (PG) fill_pages(0);
    load_k(0);
    if (!LATE_V) load_v(0);
  }
#pragma unroll
  for (int i = 0; i < NQ; ++i)
    if (tid + i * kThreads < GB * D) qd[0][tid + i * kThreads] = (double)qv[i];
  if (p.q_sink)
    for (int at = tid; at < GB * D; at += kThreads) qd[1][at] = (double)((const float*)p.q_sink)[head0 * D + at];
  int slot = sg.slot;
  if (slot_is_late(p)) slot = late_slot(p, sg, ring_n);
  if (tid < 2 * CH) {
    s_new[tid] = fresh;
    if (slot >= t_begin && slot < t_end) st16((value ? Vr : Kr).at(slot) + (tid % CH) * 16, fresh);  // Step 4: the new token enters the window
  }
  __syncthreads();

  float m = -INFINITY;  // of head sl
  double l = 0.0, acc[GB][4];
#pragma unroll
  for (int g = 0; g < GB; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[g][e] = 0.0;

  for (int b = wave, it = 0; b < nblk; b += NW, ++it) {
    const int b0 = t_begin + b * BT;
    // whatever the cache holds in the new token's place was loaded, by lanes past the slice too: the token itself instead
    const bool patch = slot >= 0 && ((slot >= b0 && slot < b0 + BT) || (b0 + BT > t_end && (slot == t_begin || (PG && slot >= b0 - 16 && slot < t_end))));
    if (patch) {  // wave-uniform
#pragma unroll
      for (int g = 0; g < NG; ++g)
        if (token(it, 8 * g, 8 * g + t8) == slot) {
#pragma unroll
          for (int ch = 0; ch < NC; ++ch) kv[g][ch] = s_new[ch * 8 + sl];
        }
    }

    // logits: lane's parts, two groups at a time
    double x[NG];  // of head sl, token 8 g + t8
    auto logits = [&](auto sink) {
#pragma unroll
      for (int gg = 0; gg < NG; gg += 2) {
#pragma unroll
        for (int hh = 0; hh < GB; hh += 4) {
          asm volatile("" ::: "memory");  // the queries are read again, not held for the other groups
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
              kd[u][0] = (double)__uint_as_float(kv[gg + u][ch].x);
              kd[u][1] = (double)__uint_as_float(kv[gg + u][ch].y);
              kd[u][2] = (double)__uint_as_float(kv[gg + u][ch].z);
              kd[u][3] = (double)__uint_as_float(kv[gg + u][ch].w);
            }
#pragma unroll
            for (int h = 0; h < 4 && hh + h < GB; ++h) {
              const int at = (hh + h) * D + (ch * 8 + sl) * 4;
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const double* q = qd[0] + at;
                if constexpr (decltype(sink)::value) q = qd[b0 + 8 * (gg + u) + t8 < p.qs_S ? 1 : 0] + at;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[u][h] = fma(kd[u][e], q[e], a[u][h]);
              }
            }
          }
          // over the eight lanes of a token; lane s keeps head s
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const double r = eight_lane_sums<GB>(a[u], sl);
            x[gg + u] = hh == 0 || sl >= 4 ? r : x[gg + u];
          }
        }
      }
    };
    if (p.q_sink && b0 < p.qs_S)  // wave-uniform: the block holds sink tokens
      logits(std::integral_constant<bool, true>());
    else
      logits(std::integral_constant<bool, false>());
    if (LATE_V) load_v(it);
    const bool more = b + NW < nblk;
    if (more) {
      if (PG && (((it + 1) * GPB) & 63) == 0) fill_pages(it + 1);
      load_k(it + 1);
    }

    // softmax weights, once per (token, head)
    float bm = -INFINITY;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int tok = b0 + 8 * g + t8;
      const bool in = sl < GB && tok < t_end && head_attends(p.pq_S, p.pq_k, p.G, g0 + sl, tok);
      x[g] = in ? x[g] * (1.0 / sqrt((double)D)) : -INFINITY;
      bm = fmaxf(bm, (float)x[g]);
    }
    bm = fmaxf(bm, dpp_f32<0x128>(bm));  // row_ror:8
    bm = swap32_max(swap16_max(bm));
    const float mn = fmaxf(m, bm);
    const float corr = mn == -INFINITY ? 1.f : exp_fast(m - mn);  // head with nothing to attend yet
    l *= (double)corr;
    m = mn;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the last block's weights are read
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const float w = x[g] == -INFINITY ? 0.f : exp_fast((float)(x[g] - (double)mn));
      l += (double)w;
      if (sl < GB) pw[wave][8 * g + t8][sl] = (double)w;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // P.V on the lanes that hold V's chunks
    if (patch) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (token(it, i * TPL, i * TPL + tq) == slot) vv[i] = s_new[CH + cl];
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const double f = (double)__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(corr), g));
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[g][e] *= f;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double v[4] = {(double)__uint_as_float(vv[i].x), (double)__uint_as_float(vv[i].y), (double)__uint_as_float(vv[i].z),
                           (double)__uint_as_float(vv[i].w)};
#pragma unroll
      for (int g = 0; g < GB; ++g) {
        const double w = pw[wave][i * TPL + tq][g];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[g][e] = fma(w, v[e], acc[g][e]);
      }
    }
    if (!LATE_V && more) load_v(it + 1);
  }

  // the wave's totals: over the lanes that share a chunk of V, and those that share a head
#pragma unroll
  for (int g = 0; g < GB; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double a = acc[g][e];
      if (CH == 16) a += swap16_f64(a);
      a = swap32_sum_f64(a);
      if (tq == 0) s_acc[wave][g][cl * 4 + e] = (float)a;
    }
  l += dpp_f64<0x128>(l);
  l += swap16_f64(l);
  l = swap32_sum_f64(l);
  if (lane < GB) {
    s_m[wave][lane] = m;
    s_l[wave][lane] = l;
  }
  __syncthreads();

  // the waves' parts, added in fp64; one split: finish here, else write this split's partial
  const bool single = p.n_splits == 1;
  float* pa = p.part_acc + (((int64_t)row * p.n_splits + split) * p.G + g0) * D;
  float2* pml = p.part_ml + ((int64_t)row * p.n_splits + split) * p.G + g0;
  for (int it = tid; it < GB * D; it += kThreads) {
    const int g = it / D, j = it % D;
    float M = s_m[0][g];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][g]);
    double a = 0.0, ls = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const double f = s_m[w][g] == -INFINITY ? 0.0 : (double)exp_fast(s_m[w][g] - M);
      a += (double)s_acc[w][g][j] * f;
      ls += s_l[w][g] * f;
    }
    if (single) {
      p.out[(head0 + g) * D + j] = (float)(a / ls);
    } else {
      pa[(int64_t)g * D + j] = M == -INFINITY ? 0.f : (float)a;  // (nothing attended here: see combine_kernel)
      if (j == 0) pml[g] = make_float2(M, (float)ls);
    }
  }
  finish_row(p, sg);
}

// bf16 decode with the q.K products on the matrix cores.  Per 32-token block a wave stages K
// through XOR-swizzled LDS into v_mfma_f32_16x16x32_bf16 (A = queries, zero padded to GPAD heads),
// so a lane ends with the 4 logits of one token: the softmax weights are computed once per
// (token, head) instead of once per lane, then handed through LDS to the lanes that hold the V
// chunks (16 lanes per token, fp32 FMA accumulation).  K and V of block b+1 are both in flight
// while block b is processed (two 8-load register buffers per wave).  STREAM: the reduced cache
// does not fit the on-chip caches between steps, read it with streaming loads.
template <int D, int GPAD, int NW, bool STREAM, bool PG>
__global__ __launch_bounds__(NW * 64) void decode_mfma_kernel(DecodeParams p, int g0, int gb) {
  constexpr int BT = GPAD > 4 ? 16 : 32;                   // tokens per block (registers: acc is GPAD x 8)
  constexpr int CH = D / 8, TPL = 64 / CH, NLOAD = BT / TPL, KSTEPS = D / 32;
  constexpr int TILES = 16 / GPAD;                         // 16-token tiles sharing the accumulator rows
  constexpr int NT = BT / 16;                              // tiles per block (<= TILES for GPAD <= 8)
  constexpr int ROWB = D * 2, EPL = 8;
  constexpr int kThreads = NW * 64;
  static_assert(NT <= TILES, "one accumulator per block");

  __shared__ uint4 kbuf[NW][BT * CH];
  __shared__ float pbuf[NW][BT][GPAD];
  __shared__ float cbuf[NW][GPAD];
  __shared__ float2 s_ml[NW][GPAD];

  const int row = blockIdx.y, split = blockIdx.x;
  const int prob = row / p.Hkv, c = row % p.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tq = lane / CH, cl = lane % CH;  // load / PV role: token sub-index, 16-byte chunk
  const int n = lane & 15, j = lane >> 4;    // MFMA role: column (token), row block

  const CacheRow Kr = cache_row(p.Kc, p.cpm, false, prob, c, row, p.cap, ROWB, 2);
  const CacheRow Vr = cache_row(p.Vc, p.cpm, true, prob, c, row, p.cap, ROWB, 2);
  const char* kn = p.k_new ? (const char*)p.k_new + (int64_t)row * ROWB : nullptr;
  const char* vn = p.v_new ? (const char*)p.v_new + (int64_t)row * ROWB : nullptr;
  StepGeom sg = step_geom<true>(p);
  int ring_n = 0;
  if (slot_is_late(p)) ring_n = p.ring[0];  // on its way while the first loads are issued
  const int t_begin = split * sg.tokens_per_split;
  const int t_end = min(sg.len, t_begin + sg.tokens_per_split);

  // accumulator rows 4j..4j+3 = (tile slot, heads hbase..hbase+3); slots >= NT stay empty
  const int hbase = (4 * j) % GPAD, tile = (4 * j) / GPAD;
  const int t_mine = tile * 16 + n;  // this lane's token within the block (MFMA role)
  float m_run[4], l_part[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    m_run[r] = -INFINITY;
    l_part[r] = 0.f;
  }
  float acc[GPAD][EPL];
#pragma unroll
  for (int g = 0; g < GPAD; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;

  uint4* buf = kbuf[wave];
  const int nblk = (t_end - t_begin + BT - 1) / BT;
  uint4 kv[NLOAD], vv[NLOAD];
  BlockSource<PG, ROWB, BT, NW, TPL> src = {Kr, Vr, t_begin, t_end, sg.slot, wave, 0};
  auto load_block = [&](int it, uint4* dst, const CacheRow& base, const char* fresh) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const char* a = src.at(base, fresh, it, i, tq) + cl * 16;
      dst[i] = STREAM ? ld16_stream(a) : ld16(a);
    }
  };
  if (wave < nblk) {  // first blocks in flight before anything else is waited for
    src.fill_pages(0);
    load_block(0, kv, Kr, kn);
    load_block(0, vv, Vr, vn);
  }
  if (slot_is_late(p)) {
    src.slot = late_slot(p, sg, ring_n);
    src.patch_first(kv, vv, kn, vn, tq, cl);
  }
  const int slot = src.slot;
  if (slot >= t_begin && slot < t_end && tid < CH) {  // Step 4: the new token enters the window
    st16(Kr.at(slot) + tid * 16, ld16(kn + tid * 16));
    st16(Vr.at(slot) + tid * 16, ld16(vn + tid * 16));
  }
  // A operand of tile slot ts, k-step kc, kept in LDS (registers are short here): lane (row m = n,
  // k-group j) reads q[head m % GPAD][8*(4*kc + j) ..+8] if m / GPAD == ts, zeros otherwise
  // Set 1 holds the query the sink tokens are scored with, when the caller gives one.
  __shared__ uint4 qbuf[2][NT][KSTEPS][64];
  for (int it = tid; it < (p.q_sink ? 2 : 1) * NT * KSTEPS * 64; it += kThreads) {
    const int l = it & 63, kc = (it >> 6) % KSTEPS, ts = (it / (64 * KSTEPS)) % NT, set = it / (64 * KSTEPS * NT);
    const int m = l & 15, jj = l >> 4;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (m % GPAD < gb && m / GPAD == ts) {
      const int h = c * p.G + g0 + m % GPAD;
      v = ld16((const char*)(set ? p.q_sink : p.q) + (((int64_t)prob * p.Hq + h) * D + (4 * kc + jj) * 8) * 2);
    }
    qbuf[set][ts][kc][l] = v;
  }
  __syncthreads();
  for (int b = wave, it = 0; b < nblk; b += NW, ++it) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // last block's LDS reads are done
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int t = i * TPL + tq;
      buf[t * CH + (cl ^ (t & (CH - 1)))] = kv[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const bool more = b + NW < nblk;
    if (more) {
      if (src.refill_before(it + 1)) src.fill_pages(it + 1);
      load_block(it + 1, kv, Kr, kn);
    }

    // logits of the block
    f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f}, ds = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const bool sink_blk = p.q_sink && t_begin + b * BT < p.qs_S;  // wave-uniform: the block holds sink tokens
#pragma unroll
    for (int ts = 0; ts < NT; ++ts) {
      const int t = ts * 16 + n;
#pragma unroll
      for (int kc = 0; kc < KSTEPS; ++kc) {
        const uint4 bb = buf[t * CH + ((4 * kc + j) ^ (n & (CH - 1)))];
        const uint4 qv = qbuf[0][ts][kc][lane];
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qv), __builtin_bit_cast(bf16x8_t, bb), d,
                                                    0, 0, 0);
        if (sink_blk) {
          const uint4 qs = qbuf[1][ts][kc][lane];
          ds = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qs), __builtin_bit_cast(bf16x8_t, bb),
                                                       ds, 0, 0, 0);
        }
      }
    }
    const int tok = t_begin + b * BT + t_mine;
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[r] = (tile < NT && tok < t_end && hbase + r < gb && head_attends(p.pq_S, p.pq_k, p.G, g0 + hbase + r, tok))
                 ? (sink_blk && tok < p.qs_S ? ds[r] : d[r]) * p.scale
                 : -INFINITY;

    // online softmax, once per (token, head); lanes with the same heads agree on the maximum
    float corr[4], pw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float bm = x[r];
      bm = group16_max(bm);
#pragma unroll
      for (int o = 16 * (GPAD / 4); o < 64; o <<= 1) bm = fmaxf(bm, __shfl_xor(bm, o));
      const float mn = fmaxf(m_run[r], bm);
      corr[r] = (mn == -INFINITY) ? 1.f : exp_fast(m_run[r] - mn);
      pw[r] = (x[r] == -INFINITY) ? 0.f : exp_fast(x[r] - mn);
      l_part[r] = l_part[r] * corr[r] + pw[r];
      m_run[r] = mn;
    }
    if (tile < NT) *reinterpret_cast<float4*>(&pbuf[wave][t_mine][hbase]) = make_float4(pw[0], pw[1], pw[2], pw[3]);
    if (n == 0 && j < GPAD / 4)
      *reinterpret_cast<float4*>(&cbuf[wave][hbase]) = make_float4(corr[0], corr[1], corr[2], corr[3]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // P.V on the lanes that hold the V chunks
#pragma unroll
    for (int g4 = 0; g4 < GPAD / 4; ++g4) {
      const float4 c4 = *reinterpret_cast<const float4*>(&cbuf[wave][g4 * 4]);
      const float cr[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g4 * 4 + r][e] *= cr[r];
    }
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      if (GPAD > 4) __builtin_amdgcn_sched_barrier(0);  // keep the unrolled steps apart: registers
      const int t_local = i * TPL + tq;
      float vf[EPL];
      unpack16(vv[i], vf);
      if (more) {  // the register is free: V of the next block, as early as possible
        const char* a = src.at(Vr, vn, it + 1, i, tq) + cl * 16;
        vv[i] = STREAM ? ld16_stream(a) : ld16(a);
      }
#pragma unroll
      for (int g4 = 0; g4 < GPAD / 4; ++g4) {
        const float4 p4 = *reinterpret_cast<const float4*>(&pbuf[wave][t_local][g4 * 4]);
        const float pp[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[g4 * 4 + r][e] = fmaf(pp[r], vf[e], acc[g4 * 4 + r][e]);
      }
    }
  }

  // wave totals: sum of weights per head, accumulators over the TPL token groups
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float ls = group_sum<16>(l_part[r]);
#pragma unroll
    for (int o = 16 * (GPAD / 4); o < 64; o <<= 1) ls += __shfl_xor(ls, o);
    if (n == 0 && j < GPAD / 4) s_ml[wave][hbase + r] = make_float2(m_run[r], ls);
  }
  __syncthreads();  // every wave is done with its K buffer: reuse it for the accumulators
  float* s_acc = reinterpret_cast<float*>(&kbuf[0][0]);  // [NW][GPAD][D]
  static_assert(GPAD * D * 4 <= BT * CH * 16 + 0 * NW, "accumulators fit the K buffers");
#pragma unroll
  for (int g = 0; g < GPAD; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      float a = acc[g][e];
#pragma unroll
      for (int o = CH; o < 64; o <<= 1) a += __shfl_xor(a, o);
      if (tq == 0) s_acc[((wave * GPAD) + g) * D + cl * EPL + e] = a;
    }
  __syncthreads();

  const bool single = p.n_splits == 1;
  float* pa = p.part_acc + (((int64_t)row * p.n_splits + split) * p.G + g0) * D;
  float2* pml = p.part_ml + ((int64_t)row * p.n_splits + split) * p.G + g0;
  for (int it = tid; it < gb * D; it += kThreads) {
    const int g = it / D, jj = it % D;
    float M = s_ml[0][g].x;
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_ml[w][g].x);
    float a = 0.f, ls = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2 ml = s_ml[w][g];
      const float f = (ml.x == -INFINITY) ? 0.f : exp_fast(ml.x - M);
      a += s_acc[((w * GPAD) + g) * D + jj] * f;
      ls += ml.y * f;
    }
    if (single) {
      p.out[((int64_t)prob * p.Hq + c * p.G + g0 + g) * D + jj] = a / ls;
    } else {
      pa[(int64_t)g * D + jj] = a;
      if (jj == 0) pml[g] = make_float2(M, ls);
    }
  }
  finish_row(p, sg);
}

// bf16 decode with BOTH products on the matrix cores.  q.K as in decode_mfma_kernel.  The softmax
// weights of a 32-token block are rounded to bf16 (as the values are) and written to LDS as
// P[head][token]; V goes through the wave's staging buffer like K, and a lane gets the MFMA B operand
// V[8 tokens][its dim] with two transposed LDS reads (ds_read_b64_tr_b16: lane s of a 16-lane group
// addresses 4 dims of token s / 4 and receives dim s of 4 tokens).
// out[head][dim] accumulates in one 16x16 tile per 16 dims, rows = heads, so the accumulator does not
// grow with the group size and the vector ALU no longer does G x head_dim multiply-adds per token.
__device__ __forceinline__ uint32_t bf16_rne(float f) {  // finite, non-negative input
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// Loads of that kernel.  A wave's it-th block holds the BT tokens from first(it) on; where all of them are in the slice, load i is
// a wave-uniform address + 16 bytes per lane, and nothing else is computed per load: the new token is not looked for in
// the addresses, the one block that holds its slot is patched afterwards.  (One layer's step spent 1.9 us on 16 times 13
// address instructions and on eight rounds of kernel arguments before its first key was asked for.)
// PAGED: as BlockSource.
template <bool PG, bool STREAM, int D, int BT, int NW>
struct SliceLoads {
  static constexpr int ROWB = D * 2, CH = D / 8, TPL = 64 / CH, NLOAD = BT / TPL, GPB = BT / 16;
  int t_begin, t_end, slot, wave, lane;
  // paged: this problem's block table; page ids of the 64 groups at hand
  const int32_t* tab;
  int shift, n_pages, my_page;

  __device__ __forceinline__ int first(int it) const { return t_begin + (wave + it * NW) * BT; }
  __device__ __forceinline__ void fill_pages(int it0) {
    if (!PG) return;
    int tok = first(it0 + lane / GPB) + (lane % GPB) * 16;
    tok = tok < t_end ? tok : t_begin;
    const int pid = tab[tok >> shift];
    my_page = pid < 0 ? 0 : (pid >= n_pages ? n_pages - 1 : pid);
  }
  __device__ __forceinline__ bool refill_before(int it) const { return PG && ((it * GPB) & 63) == 0; }
  // this lane's token of load i; past the slice one that is inside it (its first, in pages the first of the group)
  __device__ __forceinline__ int token(int it, int i) const {
    const int b0 = first(it), tok = b0 + i * TPL + lane / CH, g0 = b0 + (i * TPL) / 16 * 16;
    return tok < t_end ? tok : PG && g0 < t_end ? g0 : t_begin;
  }
  __device__ __forceinline__ uint4 ld(const char* p) const { return STREAM ? ld16_stream(p) : ld16(p); }
  // base: the row's first token, or the pool advanced to the row's KV head
  __device__ __forceinline__ void load(int it, const char* base, int64_t page_bytes, uint4 (&dst)[NLOAD]) const {
    const int b0 = first(it);
    if (b0 + BT <= t_end) {  // wave-uniform
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) {
        const int tok = b0 + i * TPL;
        const char* p = base + (int64_t)tok * ROWB;
        if (PG)
          p = base + (int64_t)__builtin_amdgcn_readlane(my_page, (it * GPB + (i * TPL) / 16) & 63) * page_bytes +
              (int64_t)(tok & ((1 << shift) - 1)) * ROWB;
        dst[i] = ld(p + lane * 16);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) {
        const int tok = token(it, i);
        const char* p = base + (int64_t)tok * ROWB;
        if (PG)
          p = base + (int64_t)__builtin_amdgcn_readlane(my_page, (it * GPB + (i * TPL) / 16) & 63) * page_bytes +
              (int64_t)(tok & ((1 << shift) - 1)) * ROWB;
        dst[i] = ld(p + (lane % CH) * 16);
      }
    }
  }
  // Does the block hold the new token (or, past the slice's end, a stand-in that is the new token)?  wave-uniform
  __device__ __forceinline__ bool holds_slot(int it) const {
    const int b0 = first(it);
    return slot >= 0 && ((slot >= b0 && slot < b0 + BT) || (slot == t_begin && b0 + BT > t_end));
  }
  // fresh: this lane's 16 bytes of the new token, loaded early
  __device__ __forceinline__ void patch(int it, const uint4& fresh, uint4 (&dst)[NLOAD]) const {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      if (token(it, i) == slot) dst[i] = fresh;
  }
};

template <int D, int GPAD, int NW, bool STREAM, bool PG>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) void decode_pv_mfma_kernel(DecodeParams p, int g0, int gb) {
  constexpr int BT = 32;
  constexpr int CH = D / 8, TPL = 64 / CH, NLOAD = BT / TPL, KSTEPS = D / 32;
  constexpr int TILES = 16 / GPAD;                       // 16-token tiles sharing a q.K accumulator
  constexpr int NT = BT / 16;                            // token tiles per block
  constexpr int NACC = NT > TILES ? NT / TILES : 1;      // q.K accumulators per block
  constexpr int NDT = D / 16;                            // output tiles (16 dims each)
  constexpr int ROWB = D * 2;
  constexpr int kThreads = NW * 64;
  static_assert(GPAD * D * 4 <= BT * CH * 16, "accumulators fit the staging buffers");

  __shared__ uint4 kbuf[NW][BT * CH];  // K staging, then V staging, at the end the waves' accumulators
  __shared__ __attribute__((aligned(16))) unsigned short pT[NW][16][BT];  // weights, bf16, [head][token]
  __shared__ float2 s_ml[NW][GPAD];

  const int row = blockIdx.y, split = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tq = lane / CH, cl = lane % CH;  // load role: token sub-index, 16-byte chunk
  const int n = lane & 15, j = lane >> 4;    // MFMA role: column, row block / k-group
  const int64_t head0 = (int64_t)row * p.G + g0;  // = problem * Hq + KV head * G + g0

  SliceLoads<PG, STREAM, D, BT, NW> src;
  const char *Kb, *Vb;
  if (PG) {
    const int prob = row / p.Hkv, c = row % p.Hkv;
    Kb = (const char*)p.Kc + ((int64_t)c << p.cpm.shift) * ROWB;
    Vb = (const char*)p.Vc + ((int64_t)c << p.cpm.shift) * ROWB;
    src.tab = p.cpm.table + (int64_t)prob * p.cpm.pitch;
    src.shift = p.cpm.shift;
    src.n_pages = p.cpm.n_pages;
  } else {
    Kb = (const char*)p.Kc + (int64_t)row * p.cap * ROWB;
    Vb = (const char*)p.Vc + (int64_t)row * p.cap * ROWB;
  }
  const int64_t k_page = PG ? p.cpm.ks_page * 2 : 0, v_page = PG ? p.cpm.vs_page * 2 : 0;
  StepGeom sg = step_geom<true>(p);
  int ring_n = 0;
  if (slot_is_late(p)) ring_n = p.ring[0];  // on its way while the first loads are issued
  const int t_begin = split * sg.tokens_per_split;
  const int t_end = min(sg.len, t_begin + sg.tokens_per_split);
  const int nblk = (t_end - t_begin + BT - 1) / BT;
  src.t_begin = t_begin, src.t_end = t_end, src.slot = sg.slot, src.wave = wave, src.lane = lane, src.my_page = 0;

  // The queries' loads go out first, then K's, then V's: loads complete in order, so each is waited for when it is
  // needed and no later one with it.
  // A operand of the q.K product, the same for every tile: lane (row m = n, k-group j) holds q[head m % GPAD][8*(4*kc + j) ..+8], so a
  // product holds every head's logits 16 / GPAD times over and a lane takes the tile of its slot.
  uint4 qa[KSTEPS], qs[KSTEPS];  // qs: the query the sink tokens are scored with, when the caller gives one
  {
    const int64_t at = ((head0 + n % GPAD) * D + 8 * j) * 2;
    const bool mine = n % GPAD < gb;
#pragma unroll
    for (int kc = 0; kc < KSTEPS; ++kc) {
      qa[kc] = qs[kc] = make_uint4(0u, 0u, 0u, 0u);
      if (mine) qa[kc] = ld16((const char*)p.q + at + 64 * kc);
    }
    if (p.q_sink && mine) {
#pragma unroll
      for (int kc = 0; kc < KSTEPS; ++kc) qs[kc] = ld16((const char*)p.q_sink + at + 64 * kc);
    }
  }
  uint4 k_fresh = make_uint4(0u, 0u, 0u, 0u), v_fresh = k_fresh;  // this lane's chunk of the new token
  if (p.k_new) {
    k_fresh = ld16((const char*)p.k_new + (int64_t)row * ROWB + cl * 16);
    v_fresh = ld16((const char*)p.v_new + (int64_t)row * ROWB + cl * 16);
  }
  uint4 kv[NLOAD], vv[NLOAD];
  if (wave < nblk) {
    src.fill_pages(0);
    src.load(0, Kb, k_page, kv);
    src.load(0, Vb, v_page, vv);
  }

  // q.K accumulator a, register r of lane (j, n): head hbase + r, token tile a * TILES + tslot, column n
  const int hbase = (4 * j) % GPAD, tslot = (4 * j) / GPAD;
  float m_run[4], l_part[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    m_run[r] = -INFINITY;
    l_part[r] = 0.f;
  }
  f32x4_t acc[NDT];  // out[head 4j + r][dim 16 * nd + n]
#pragma unroll
  for (int nd = 0; nd < NDT; ++nd) acc[nd] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  uint4* buf = kbuf[wave];
  reinterpret_cast<uint4*>(&pT[wave][0][0])[lane] = make_uint4(0u, 0u, 0u, 0u);  // rows of absent heads stay 0

  if (slot_is_late(p)) src.slot = late_slot(p, sg, ring_n);
  const int slot = src.slot;
  if (slot >= t_begin && slot < t_end && tid < CH) {  // Step 4: the new token enters the window
    const CacheRow Kr = cache_row(p.Kc, p.cpm, false, row / p.Hkv, row % p.Hkv, row, p.cap, ROWB, 2);
    const CacheRow Vr = cache_row(p.Vc, p.cpm, true, row / p.Hkv, row % p.Hkv, row, p.cap, ROWB, 2);
    st16(Kr.at(slot) + tid * 16, k_fresh);
    st16(Vr.at(slot) + tid * 16, v_fresh);
  }

  // V staging swizzle (16-byte chunk ^= vswz(token)): the four tokens a 16-lane group reads together
  // land in different banks
  auto vswz = [](int t) { return CH == 16 ? (((t & 3) << 1) | (((t >> 3) & 1) << 3)) : ((t & 3) << 1); };

  for (int b = wave, it = 0; b < nblk; b += NW, ++it) {
    const bool patch = src.holds_slot(it);  // wave-uniform, one block of the row
    if (patch) src.patch(it, k_fresh, kv);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // last block's reads of the buffer are done
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int t = i * TPL + tq;
      buf[t * CH + (cl ^ (t & (CH - 1)))] = kv[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const bool more = b + NW < nblk;
    if (more) {
      if (src.refill_before(it + 1)) src.fill_pages(it + 1);
      src.load(it + 1, Kb, k_page, kv);
    }

    const int tok0 = t_begin + b * BT;
    f32x4_t d[NACC];
    auto qk = [&](const uint4 (&q)[KSTEPS], f32x4_t (&out)[NACC]) {
#pragma unroll
      for (int ts = 0; ts < NT; ++ts) {
        const int t = ts * 16 + n;
        f32x4_t x = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < KSTEPS; ++kc) {
          const uint4 bb = buf[t * CH + ((4 * kc + j) ^ (n & (CH - 1)))];
          x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, q[kc]), __builtin_bit_cast(bf16x8_t, bb), x, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) out[ts / TILES][r] = ts % TILES == 0 || tslot == ts % TILES ? x[r] : out[ts / TILES][r];
      }
    };
    qk(qa, d);
    if (p.q_sink && tok0 < p.qs_S) {  // wave-uniform: the block holds sink tokens
      f32x4_t ds[NACC];
      qk(qs, ds);
#pragma unroll
      for (int a = 0; a < NACC; ++a)
        if (tok0 + (a * TILES + tslot) * 16 + n < p.qs_S) d[a] = ds[a];
    }
    float x[NACC][4];
#pragma unroll
    for (int a = 0; a < NACC; ++a) {
      const int tile = a * TILES + tslot, tok = tok0 + tile * 16 + n;
      const bool in = tile < NT && tok < t_end;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[a][r] = in && hbase + r < gb ? d[a][r] * p.scale : -INFINITY;
      if (p.pq_k > 0) {  // per-query rows: a list's token belongs to one head (see head_attends)
        const int u = tok - p.pq_S;
        if (u >= 0 && u < p.G * p.pq_k) {
          const int own = u / p.pq_k - g0 - hbase;
#pragma unroll
          for (int r = 0; r < 4; ++r) x[a][r] = own == r ? x[a][r] : -INFINITY;
        }
      }
    }
    // online softmax, once per (token, head); lanes with the same heads agree on the maximum
    float corr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float bm = x[0][r];
#pragma unroll
      for (int a = 1; a < NACC; ++a) bm = fmaxf(bm, x[a][r]);
      bm = group16_max(bm);
      if (GPAD <= 4) bm = swap16_max(bm);
      if (GPAD <= 8) bm = swap32_max(bm);
      const float mn = fmaxf(m_run[r], bm);
      corr[r] = (mn == -INFINITY) ? 1.f : exp_fast(m_run[r] - mn);
      float lsum = 0.f;
#pragma unroll
      for (int a = 0; a < NACC; ++a) {
        const uint32_t pb = (x[a][r] == -INFINITY) ? 0u : bf16_rne(exp_fast(x[a][r] - mn));
        lsum += __uint_as_float(pb << 16);  // the denominator sums the weights the numerator uses
        const int tile = a * TILES + tslot;
        if (tile < NT) pT[wave][hbase + r][tile * 16 + n] = (unsigned short)pb;
      }
      l_part[r] = l_part[r] * corr[r] + lsum;
      m_run[r] = mn;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // weights visible; q.K reads of the buffer done

    // V of the block into the staging buffer, V of the next block into the registers
    if (patch) src.patch(it, v_fresh, vv);
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int t = i * TPL + tq;
      buf[t * CH + (cl ^ vswz(t))] = vv[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (more) src.load(it + 1, Vb, v_page, vv);

    // out += P.V: A = weights [head n][tokens 8j..8j+7], B = values [tokens 8j..8j+7][dim 16 nd + n]
    const uint4 pa = *reinterpret_cast<const uint4*>(&pT[wave][n][8 * j]);
#pragma unroll
    for (int nd = 0; nd < NDT; ++nd) {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[nd][r] *= corr[r];  // rows 4j + r are heads hbase + r for every j in use
      // transposed LDS read: lane s of a 16-lane group gives the address of 4 dims of token s / 4
      // and receives its own dim of 4 tokens
      typedef short v4s_t __attribute__((ext_vector_type(4)));
      const int tu = 8 * j + (n >> 2);                       // first token this lane addresses
      const int cch = (2 * nd + ((n & 3) >> 1)) ^ vswz(tu);  // vswz(tu) = vswz(tu + 4)
      const unsigned short* b16 = reinterpret_cast<const unsigned short*>(buf);
      const v4s_t x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) v4s_t*)(b16 + (tu * CH + cch) * 8 + (n & 1) * 4));
      const v4s_t x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) v4s_t*)(b16 + ((tu + 4) * CH + cch) * 8 + (n & 1) * 4));
      struct { v4s_t a, b; } pair = {x0, x1};
      const uint4 vb = __builtin_bit_cast(uint4, pair);
      acc[nd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pa), __builtin_bit_cast(bf16x8_t, vb),
                                                        acc[nd], 0, 0, 0);
    }
  }

  // wave totals: sum of weights per head over the lanes that share it
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float ls = group_sum<16>(l_part[r]);
    if (GPAD <= 4) ls = swap16_sum(ls);
    if (GPAD <= 8) ls = swap32_sum(ls);
    if (n == 0 && j < GPAD / 4) s_ml[wave][hbase + r] = make_float2(m_run[r], ls);
  }
  // a wave's accumulators go to its own staging buffer, [GPAD][D]
  constexpr int kAccStride = BT * CH * 4;  // floats between the waves' buffers
  float* s_acc = reinterpret_cast<float*>(&kbuf[0][0]);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int nd = 0; nd < NDT; ++nd)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * j + r < GPAD) s_acc[wave * kAccStride + (4 * j + r) * D + nd * 16 + n] = acc[nd][r];
  __syncthreads();

  const bool single = p.n_splits == 1;
  const int64_t part = ((int64_t)row * p.n_splits + split) * p.G + g0;
#pragma unroll
  for (int i0 = 0; i0 < GPAD * D; i0 += kThreads) {
    const int g = (i0 + tid) / D, jj = tid % D;
    if (g >= gb) break;
    float2 ml[NW];
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      ml[w] = s_ml[w][g];
      M = fmaxf(M, ml[w].x);
    }
    float a = 0.f, ls = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = (ml[w].x == -INFINITY) ? 0.f : exp_fast(ml[w].x - M);
      a += s_acc[w * kAccStride + g * D + jj] * f;
      ls += ml[w].y * f;
    }
    if (single) {
      p.out[(head0 + g) * D + jj] = a / ls;
    } else {
      p.part_acc[(part + g) * D + jj] = M == -INFINITY ? 0.f : a;  // (nothing attended here: see combine_kernel)
      if (jj == 0) p.part_ml[part + g] = make_float2(M, ls);
    }
  }
  finish_row(p, sg);
}

// Merge launch: out[head g][dim j] of a row from its slices, sum_s acc_s e^{m_s - M} / sum_s l_s e^{m_s - M}; a workgroup per (row,
// head), one thread per dim.  Latency bound: one memory round trip for up to 32 slices, all loads ahead of their first use, and few
// instructions: a wave's lanes take a slice's (m, l) each and share the factors by readlane (a thread that reads and
// exponentiates every slice's for itself executes three times as many; 8 rows x 4 heads x 32 slices of 128 dims 3.0 us so, 2.05 with the factors shared).
__global__ __launch_bounds__(128) void combine_kernel(DecodeParams p) {
  const int row = blockIdx.x, g = blockIdx.y, j = threadIdx.x, sl = threadIdx.x & 31;
  // every slice kernel of the step has finished: the device-side count of appended tokens moves on
  if (p.ring && p.ring_advance && row == 0 && g == 0 && j == 0) p.ring[0] = p.ring[0] + 1;
  if (j >= p.D) return;  // wave-uniform
  const int64_t first = (int64_t)row * p.n_splits * p.G + g;
  const float2* ml = p.part_ml + first;
  // Slices in which the head attends nothing (per-query rows) come with factor 0 and, lest a value in them that is no number
  // enters as 0 times it, with zeros.  Slices past the last read as 0 by the buffer's bound: the last one read again, even times 0, would make an infinite output
  // NaN.  (It also saves the address arithmetic: a step over 8 rows x 4096 tokens x 4 heads 10.1 -> 9.7 us.)
  const int step = p.G * p.D * (int)sizeof(float);  // bytes
  const auto acc = __builtin_amdgcn_make_buffer_rsrc(p.part_acc + first * p.D, 0, (p.n_splits - 1) * step + p.D * (int)sizeof(float), 0x00027000);
  float M = -INFINITY, num = 0.f;
  double den = 0.0;
  for (int s0 = 0; s0 < p.n_splits; s0 += 32) {
    float2 v = make_float2(-INFINITY, 0.f);
    if (s0 + sl < p.n_splits) v = ml[(int64_t)(s0 + sl) * p.G];
    float av[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) av[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(acc, (s0 + u) * step + j * (int)sizeof(float), 0, 0));
    const float Mn = fmaxf(M, swap16_max(row_combine<true, 1>(v.x)));  // both halves of the wave hold the same 32 slices
    if (Mn == -INFINITY) continue;  // nothing attended in these slices (uniform over the workgroup)
    const float f = v.x == -INFINITY ? 0.f : exp_fast(v.x - Mn);
    const float f0 = M == -INFINITY ? 0.f : exp_fast(M - Mn);
    den = den * f0 + group_sum_f64<32>((double)v.y * f);  // (a tree of rounded fp32 products is 1 % further off over four slices)
    num *= f0;
#pragma unroll
    for (int u = 0; u < 32; ++u)
      num = fmaf(av[u], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), u)), num);
    M = Mn;
  }
  p.out[((int64_t)row * p.G + g) * p.D + j] = num / (float)den;
}

template <int LPT>
__global__ __launch_bounds__(64) void append_kernel(DecodeParams p, int row_bytes) {
  const int row = blockIdx.x, tid = threadIdx.x;
  if (tid >= LPT) return;
  const int prob = row / p.Hkv, c = row % p.Hkv, eb = row_bytes / p.D;
  const CacheRow Kr = cache_row(p.Kc, p.cpm, false, prob, c, row, p.cap, row_bytes, eb);
  const CacheRow Vr = cache_row(p.Vc, p.cpm, true, prob, c, row, p.cap, row_bytes, eb);
  st16(Kr.at(p.slot) + tid * 16, ld16((const char*)p.k_new + (int64_t)row * row_bytes + tid * 16));
  st16(Vr.at(p.slot) + tid * 16, ld16((const char*)p.v_new + (int64_t)row * row_bytes + tid * 16));
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = v;
}

template <int D, int GB, bool PG>
void launch_decode_f32_g(const DecodeParams& p, int g0, dim3 grid, hipStream_t s) {
  if constexpr (D == 128) {
    hipLaunchKernelGGL((decode_f32_kernel<D, GB, 8, 16, PG>), grid, dim3(512), 0, s, p, g0);
  } else if (p.n_splits > 1) {
    hipLaunchKernelGGL((decode_f32_kernel<D, GB, 4, 32, PG>), grid, dim3(256), 0, s, p, g0);
  } else if constexpr (GB <= 2) {
    hipLaunchKernelGGL((decode_f32_kernel<D, GB, 8, 16, PG>), grid, dim3(512), 0, s, p, g0);
  } else {
    hipLaunchKernelGGL((decode_f32_kernel<D, GB, 8, 32, PG>), grid, dim3(512), 0, s, p, g0);
  }
}

template <int D, bool PG>
hipError_t launch_decode_f32(const DecodeParams& p, int g0, int gb, dim3 grid, hipStream_t s) {
  switch (gb) {
    case 1: launch_decode_f32_g<D, 1, PG>(p, g0, grid, s); break;
    case 2: launch_decode_f32_g<D, 2, PG>(p, g0, grid, s); break;
    case 3: launch_decode_f32_g<D, 3, PG>(p, g0, grid, s); break;
    case 4: launch_decode_f32_g<D, 4, PG>(p, g0, grid, s); break;
    case 5: launch_decode_f32_g<D, 5, PG>(p, g0, grid, s); break;
    case 6: launch_decode_f32_g<D, 6, PG>(p, g0, grid, s); break;
    case 7: launch_decode_f32_g<D, 7, PG>(p, g0, grid, s); break;
    case 8: launch_decode_f32_g<D, 8, PG>(p, g0, grid, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D, bool STREAM, bool PG>
hipError_t launch_decode_mfma_s(const DecodeParams& p, int g0, int gb, dim3 grid, hipStream_t s) {
  // One workgroup per row (many rows): 8 waves, one workgroup per CU; a row split over several
  // workgroups: 4 waves.  (For 256 < rows <= 512, 4-wave workgroups that are all resident at once
  // were measured no faster than two rounds of 8-wave ones.)
  // Up to 4 heads with whole rows, P.V on the vector ALU is a little faster (measured 86 vs 89 us
  // per step at 256 rows x 4096 tokens); with more heads, or short slices, P.V on the matrix cores
  // wins clearly (448 rows x 1024 tokens x 7 heads: 47 vs 68 us).
  const bool big = p.n_splits == 1;
  // more rows than CUs: 4-wave workgroups, two resident per CU, beat two rounds of 8-wave ones
  // (measured 43 vs 47 us at 448 rows x 1024 tokens x 7 heads)
  const bool wide = big && grid.y <= 256;
  if (gb <= 4) {
    // few short rows that took the split kernel before they were whole (more than 128 tokens): latency, P.V on the matrix
    // cores (8 rows x 256 tokens: 8.4 vs 9.8 us); shorter ones keep their fp32 weights
    if (big && grid.y < kWholeRows && p.len > 128)
      hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 4, 8, STREAM, PG>), grid, dim3(512), 0, s, p, g0, gb);
    else if (big) hipLaunchKernelGGL((decode_mfma_kernel<D, 4, 8, STREAM, PG>), grid, dim3(512), 0, s, p, g0, gb);
    else hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 4, 4, STREAM, PG>), grid, dim3(256), 0, s, p, g0, gb);
  } else if (gb <= 8) {
    if (wide) hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 8, 8, STREAM, PG>), grid, dim3(512), 0, s, p, g0, gb);
    else hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 8, 4, STREAM, PG>), grid, dim3(256), 0, s, p, g0, gb);
  } else {
    if (wide) hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 16, 8, STREAM, PG>), grid, dim3(512), 0, s, p, g0, gb);
    else hipLaunchKernelGGL((decode_pv_mfma_kernel<D, 16, 4, STREAM, PG>), grid, dim3(256), 0, s, p, g0, gb);
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_decode_mfma(const DecodeParams& p, int g0, int gb, dim3 grid, hipStream_t s) {
  if (p.cpm.table)
    return p.stream_loads ? launch_decode_mfma_s<D, true, true>(p, g0, gb, grid, s)
                          : launch_decode_mfma_s<D, false, true>(p, g0, gb, grid, s);
  return p.stream_loads ? launch_decode_mfma_s<D, true, false>(p, g0, gb, grid, s)
                        : launch_decode_mfma_s<D, false, false>(p, g0, gb, grid, s);
}

}  // namespace

hipError_t launch_decode(const DecodeParams& p, hipStream_t s) {
  const int rows = p.n_problems * p.Hkv;
  dim3 grid((unsigned)p.n_splits, (unsigned)rows);
  const int per_launch = p.dtype == DT_BF16 ? 16 : max_group_per_launch();  // heads one launch handles
  for (int g0 = 0; g0 < p.G; g0 += per_launch) {
    const int gb = p.G - g0 < per_launch ? p.G - g0 : per_launch;
    DecodeParams q = p;
    if (g0 > 0) q.k_new = nullptr;  // the first launch already stored the new token
    if (g0 + per_launch < p.G) q.ring_advance = 0;  // the last launch of the step moves the ring on
    hipError_t e;
    if (p.dtype == DT_BF16)
      e = p.D == 128 ? launch_decode_mfma<128>(q, g0, gb, grid, s) : launch_decode_mfma<64>(q, g0, gb, grid, s);
    else
      e = p.cpm.table ? (p.D == 128 ? launch_decode_f32<128, true>(q, g0, gb, grid, s) : launch_decode_f32<64, true>(q, g0, gb, grid, s))
                      : (p.D == 128 ? launch_decode_f32<128, false>(q, g0, gb, grid, s) : launch_decode_f32<64, false>(q, g0, gb, grid, s));
    if (e != hipSuccess) return e;
  }
  if (p.n_splits > 1) {
    hipLaunchKernelGGL(combine_kernel, dim3((unsigned)rows, (unsigned)p.G), dim3(128), 0, s, p);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t launch_append(const DecodeParams& p, hipStream_t s) {
  const int rows = p.n_problems * p.Hkv;
  const int eb = p.dtype == DT_BF16 ? 2 : 4;
  const int row_bytes = p.D * eb;
  switch (row_bytes / 16) {
    case 8: hipLaunchKernelGGL(append_kernel<8>, dim3((unsigned)rows), dim3(64), 0, s, p, row_bytes); break;
    case 16: hipLaunchKernelGGL(append_kernel<16>, dim3((unsigned)rows), dim3(64), 0, s, p, row_bytes); break;
    case 32: hipLaunchKernelGGL(append_kernel<32>, dim3((unsigned)rows), dim3(64), 0, s, p, row_bytes); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// A fill kernel instead of a memset: the calls may be recorded into a HIP graph.
hipError_t launch_fill_u32(void* ptr, size_t n, uint32_t value, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t want = (n + 255) / 256;
  unsigned grid = (unsigned)(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid), dim3(256), 0, s, (uint32_t*)ptr, n, value);
  return hipGetLastError();
}

}  // namespace sagekv
