// gfx950 kernels of libsplash_attn besides the attend kernel (attend.hpp) and
// the DOP regroup (dop.hip): split planner, LSE combine, page gather and
// device-data checks, and the launchers.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "device_types.hpp"
#include "kernels.hpp"
#include "splash_common.hpp"

namespace splash {

// ============================================================== planner ===

// Pages of tile t: its whole causal prefix, or under a shard its keys in
// [key_begin[b], min(prefix, key_end[b])) (key_begin a page boundary), or
// for the top-k variant its list entries in groups of 64.
__device__ __forceinline__ int32_t dev_tile_pages(const int32_t* seq_lens, int32_t q_chunk, int32_t t,
                                                  const int32_t* key_begin, const int32_t* key_end,
                                                  const int32_t* topk_count) {
  if (topk_count) return ceil_div(topk_count[t], kPage);
  int32_t b = t / q_chunk, i = t - b * q_chunk;
  int32_t L = tile_keys(seq_lens[b], q_chunk, i);
  if (key_end) {
    const int32_t hi = min(L, key_end[b]), lo = key_begin[b];
    return hi > lo ? ceil_div(hi, kPage) - lo / kPage : 0;
  }
  return L > 0 ? ceil_div(L, kPage) : 0;
}

// Whole-wave reductions of the device library (DPP based, no LDS round trips).
extern "C" __device__ __attribute__((const)) long long __ockl_wfred_add_i64(long long);
extern "C" __device__ __attribute__((const)) long long __ockl_wfred_min_i64(long long);
extern "C" __device__ __attribute__((const)) float __ockl_wfred_max_f32(float);
extern "C" __device__ __attribute__((const)) float __ockl_wfred_add_f32(float);

// Inclusive scan of one int per lane over the wave with DPP moves: prefix
// sums inside each row of 16 lanes (shifts 1, 2, 4, 8), then the row totals
// are broadcast into the following rows.
__device__ __forceinline__ int32_t wave_incl_scan(int32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
  return x;
}

// Inclusive running max of one non-negative int per lane over the wave (the
// same DPP pattern as the scan, with max for the add).
__device__ __forceinline__ int32_t wave_incl_max(int32_t x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));  // row_shr:1
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));  // row_shr:2
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));  // row_shr:4
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));  // row_shr:8
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // row_bcast:15 -> rows 1, 3
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));  // row_bcast:31 -> rows 2, 3
  return x;
}

// Exclusive block scan of one int per thread (1024 threads); returns the
// exclusive prefix and writes the block total to *total.
__device__ int32_t block_exclusive_scan(int32_t v, int32_t* wave_buf, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t inc = wave_incl_scan(v);
  if (lane == 63) wave_buf[wave] = inc;
  __syncthreads();
  if (wave == 0) {
    const int32_t x = lane < 16 ? wave_buf[lane] : 0;
    const int32_t run = wave_incl_scan(x);
    if (lane < 16) wave_buf[lane] = run - x;
    if (lane == 15) wave_buf[16] = run;
  }
  __syncthreads();
  int32_t res = wave_buf[wave] + inc - v;
  *total = wave_buf[16];
  __syncthreads();
  return res;
}

// Three exclusive block scans at once (one set of barriers for the three).
__device__ void block_exclusive_scan3(int32_t a, int32_t b, int32_t c, int32_t* wave_buf, int32_t* ea, int32_t* eb,
                                      int32_t* ec, int32_t* ta, int32_t* tb, int32_t* tc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b), ic = wave_incl_scan(c);
  if (lane == 63) {
    wave_buf[wave] = ia;
    wave_buf[17 + wave] = ib;
    wave_buf[34 + wave] = ic;
  }
  __syncthreads();
  if (wave == 0) {
    const int32_t xa = lane < 16 ? wave_buf[lane] : 0, xb = lane < 16 ? wave_buf[17 + lane] : 0,
                  xc = lane < 16 ? wave_buf[34 + lane] : 0;
    const int32_t ra = wave_incl_scan(xa), rb = wave_incl_scan(xb), rc = wave_incl_scan(xc);
    if (lane < 16) {
      wave_buf[lane] = ra - xa;
      wave_buf[17 + lane] = rb - xb;
      wave_buf[34 + lane] = rc - xc;
    }
    if (lane == 15) {
      wave_buf[16] = ra;
      wave_buf[33] = rb;
      wave_buf[50] = rc;
    }
  }
  __syncthreads();
  *ea = wave_buf[wave] + ia - a;
  *eb = wave_buf[17 + wave] + ib - b;
  *ec = wave_buf[34 + wave] + ic - c;
  *ta = wave_buf[16];
  *tb = wave_buf[33];
  *tc = wave_buf[50];
  __syncthreads();
}

__global__ __launch_bounds__(1024) void plan_kernel(PlanLaunch p) {
  __shared__ int32_t s_pages[kPlanLdsTiles];
  __shared__ int32_t s_ufirst[kPlanLdsTiles + 1];  // first unit of each tile (cached case)
  __shared__ int32_t s_sfirst[kPlanLdsTiles];      // first partial slot of each tile (cached case)
  __shared__ int64_t s_w[16][kNumCandidates + 1], s_s[16][kNumCandidates + 1];  // units, split units per tile slice
  __shared__ int32_t s_m[16][kNumCandidates + 1];  // tiles of at most pair_pages
  __shared__ int32_t s_lhist[kMaxUnitPages + 1];  // units per length
  __shared__ int32_t s_lbase[kMaxUnitPages + 1];  // next queue slot per length
  __shared__ int32_t s_q[kMaxWorkers];            // fold plan: pages of each rank (0 past the last tile)
  __shared__ int32_t s_rt[kMaxWorkers];           // fold plan: tile of each rank
  __shared__ int32_t s_pm[kMaxWorkers / 2];       // fold plan: running max of the pair loads
  __shared__ int64_t s_red64[16];
  __shared__ int32_t s_red32[16];
  __shared__ int64_t s_cost[kNumCandidates + 1];
  __shared__ int32_t s_list[kNumCandidates + 1];  // candidate index of each distinct size
  __shared__ int32_t s_nd;                        // number of distinct sizes
  __shared__ UDiv s_udiv[kNumCandidates + 1];      // their division magic
  __shared__ int32_t s_cand[kNumCandidates + 1];
  __shared__ int32_t s_parts[kNumCandidates];  // parts of each candidate
  __shared__ int32_t s_scan[51];
  __shared__ int32_t s_chunk;
  __shared__ int64_t s_best;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t T = p.B * p.q_chunk;
  const bool cached = T <= kPlanLdsTiles;
  // A shard's result is always a partial: every unit writes a partial slot
  // (the combine turns each tile's parts into its fp32 result), and tiles
  // with no key in the shard are listed for the combine with no parts.
  const bool shard = p.key_end != nullptr;
  // tiles with no key (a shard's, or a top-k row with an empty list) are
  // listed for the combine with no parts, which writes out = 0, lse = -inf
  const bool list_empty = shard || p.topk_count != nullptr;
  int32_t* hdr = p.ws.header;
  auto pages_of = [&](int32_t t) -> int32_t {
    return cached ? s_pages[t] : dev_tile_pages(p.seq_lens, p.q_chunk, t, p.key_begin, p.key_end, p.topk_count);
  };

  // 1. page counts (cached), total and largest tile.
  int64_t tot = 0;
  int32_t mx = 0;
  for (int32_t t = tid; t < T; t += 1024) {
    const int32_t P = dev_tile_pages(p.seq_lens, p.q_chunk, t, p.key_begin, p.key_end, p.topk_count);
    if (cached) s_pages[t] = P;
    tot += P;
    mx = P > mx ? P : mx;
  }
  // the candidates' part counts: k + 1 for k < 64, then the geometric
  // recurrence of plan_candidate_parts (uniform, unrolled; lane i of wave 1
  // keeps step i)
  static_assert(kNumCandidates >= 64 && kNumCandidates - 64 <= 64, "candidate layout");
  if (wave == 0) s_parts[lane] = lane + 1;
  if (wave == 1) {
    int32_t parts = 64, mine = 0;
#pragma unroll
    for (int i = 0; i < kNumCandidates - 64; ++i) {
      parts += parts / 8;
      if (lane == i) mine = parts;
    }
    if (lane < kNumCandidates - 64) s_parts[64 + lane] = mine;
  }
  tot = __ockl_wfred_add_i64(tot);
  mx = __ockl_wfred_max_i32(mx);
  if (lane == 0) { s_red64[wave] = tot; s_red32[wave] = mx; }
  __syncthreads();
  tot = 0; mx = 0;
  for (int w = 0; w < 16; ++w) { tot += s_red64[w]; mx = s_red32[w] > mx ? s_red32[w] : mx; }
  const int64_t total_pages = tot;
  const int32_t max_pages = mx > 0 ? mx : 1;

  // 2. unit size: evaluate every candidate (and a forced size), take the argmin.
  // Wave 0 lists the distinct candidate sizes (a size equal to the previous
  // candidate's is left out: the argmin keeps the smaller index on ties
  // anyway).  Then every wave counts units and split units of listed
  // candidates over a slice of the tiles: with at most 64 sizes lane j of
  // wave w takes size j over the tiles t = w + 16i, otherwise sizes
  // 64 (w >> 3) + j over t = (w & 7) + 8i.  The slices meet in LDS; wave 0
  // adds them up, prices every size (one lane each) and takes the argmin.
  if (wave == 0) {
    int32_t nd = 0, before = 0;  // before: the last size of the round before
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = 64 * r + lane;
      int32_t ck = 0;
      if (k < kNumCandidates) {
        ck = plan_candidate_size(s_parts[k], max_pages, p.unit_cap);
      }
      const int32_t up = __shfl_up(ck, 1, 64), prev = lane == 0 ? before : up;
      before = __shfl(ck, 63, 64);
      if (k < kNumCandidates) {
        if (prev == ck) ck = 0;  // (sizes are at least 1, so k = 0 stays)
      } else if (k == kNumCandidates && p.forced_chunk > 0) {
        ck = p.forced_chunk < p.unit_cap ? p.forced_chunk : p.unit_cap;
      }
      if (k <= kNumCandidates) s_cand[k] = ck;
      const uint64_t keep = __builtin_amdgcn_ballot_w64(ck > 0);
      const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(keep >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)keep, 0));
      if (ck > 0) {
        s_list[nd + below] = k;
        s_udiv[nd + below] = udiv_make((uint32_t)ck);  // once per size (at most unit_cap <= kMaxUnitPages)
      }
      nd += __builtin_popcountll(keep);
    }
    if (lane == 0) {
      s_nd = nd;
      s_cost[kNumCandidates] = INT64_MAX;
    }
  }
  __syncthreads();
  const int nd = s_nd;
  const bool wide = nd > 64;
  const int nsl = wide ? 8 : 16;  // tile slices
  {
    // With at most 32 sizes, 64 / np2 lanes share a size (np2: nd rounded up
    // to a power of two), each taking every (64 / np2)-th tile of the slice;
    // their sums meet by shuffles.  (uniform per wave)
    const int np2 = wide ? 64 : (nd <= 1 ? 1 : 1 << (32 - __builtin_clz((unsigned)(nd - 1))));
    const int sub = 64 / np2;
    const int j = wide ? 64 * (wave >> 3) + lane : (lane & (np2 - 1));
    const int part = wide ? 0 : lane / np2;
    const int slice = wide ? (wave & 7) : wave;
    int64_t W = 0, S = 0;
    int32_t M = 0;
    if (j < nd) {
      const int32_t ck = s_cand[s_list[j]];
      const UDiv ud = s_udiv[j];
      const uint32_t pair = (uint32_t)pair_pages(ck, max_pages, p.pair_spread, shard, kPlanCosts);
      auto count = [&](int32_t P) {
        const int32_t n = (int32_t)udiv((uint32_t)(P + ck - 1), ud);  // ceil(P / c)
        W += n;
        S += (n > 1 || shard) ? n : 0;
        M += (uint32_t)(P - 1) < pair ? 1 : 0;  // 1 .. pair pages
      };
      if (cached) {
#pragma unroll 4
        for (int32_t t = slice + nsl * part; t < T; t += nsl * sub) count(s_pages[t]);
      } else {
        for (int32_t t = slice + nsl * part; t < T; t += nsl * sub)
          count(dev_tile_pages(p.seq_lens, p.q_chunk, t, p.key_begin, p.key_end, p.topk_count));
      }
    }
    for (int off = np2; off < 64; off <<= 1) {
      W += __shfl_xor(W, off, 64);
      S += __shfl_xor(S, off, 64);
      M += __shfl_xor(M, off, 64);
    }
    if (j < nd && part == 0) {
      s_w[slice][j] = W;
      s_s[slice][j] = S;
      s_m[slice][j] = M;
    }
  }
  __syncthreads();
  if (wave == 0) {
    // price every listed size (lane j, then j + 64), then the first minimum
    // (smallest candidate index on ties): the key puts the cost above the
    // candidate index (costs stay far below 2^56)
    int64_t best = INT64_MAX;
    for (int j = lane; j < nd; j += 64) {
      const int k = s_list[j];
      const int32_t ck = s_cand[k];
      int64_t W = 0, S = 0;
      int32_t M = 0;
      for (int sl = 0; sl < nsl; ++sl) {
        W += s_w[sl][j];
        S += s_s[sl][j];
        M += s_m[sl][j];
      }
      const bool ok = S <= p.ws.max_partials && W <= p.ws.max_units;
      const int64_t cost = ok ? plan_cost(ck, W, S, M, total_pages, max_pages, p.G, kPlanCosts) : INT64_MAX;
      if (k == kNumCandidates) s_cost[kNumCandidates] = cost;
      const int64_t key = (cost == INT64_MAX || k == kNumCandidates) ? INT64_MAX : ((cost << 7) | k);
      best = key < best ? key : best;
    }
    best = __ockl_wfred_min_i64(best);
    int bk = best == INT64_MAX ? kNumCandidates : (int)(best & 127);
    if (lane == 0) {
      if (bk >= kNumCandidates) bk = 0;
      s_best = best == INT64_MAX ? INT64_MAX : (best >> 7);
      if (p.forced_chunk > 0 && s_cost[kNumCandidates] != INT64_MAX) bk = kNumCandidates;
      s_chunk = s_cand[bk];
    }
  }
  __syncthreads();
  const int32_t c = s_chunk;

  // 2b. the fold plan (at most one tile per worker, no forced size): rank
  // the tiles by pages, then price every cap (thread C - 1 takes cap C) and
  // keep the cheapest; taken when it beats every unit size.  The busiest worker under cap C is
  // max(16 C + U, max_{j < nl(C)} v_j - 16 C) with v_j = 16 (q_j + q_{G-1-j})
  // + U + U [q_{G-1-j} > 0] independent of C, so a running max of v over j
  // and a binary search for nl(C) = #{r : q_r > C} price a cap in O(log G).
  bool fold = p.forced_chunk == 0 && !shard &&
              fold_applicable(T, p.G, kMaxWorkers, max_pages, total_pages, s_best, kPlanCosts, p.unit_cap);
  int32_t cap = 0, nl = 0;
  if (fold) {
    // counting sort of the tiles by pages, longest first: the histogram, the
    // number of tiles with more pages (thread i takes pages kMaxUnitPages -
    // i), then one atomic per tile (tiles of equal pages in whatever order
    // the atomics give; it decides only which worker runs which of them)
    for (int32_t i = tid; i <= kMaxUnitPages; i += 1024) s_lhist[i] = 0;
    __syncthreads();
    if (tid < T) atomicAdd(&s_lhist[s_pages[tid]], 1);  // 0 <= pages <= kMaxUnitPages
    __syncthreads();
    int32_t longer;
    s_lbase[kMaxUnitPages - tid] = block_exclusive_scan(s_lhist[kMaxUnitPages - tid], s_scan, &longer);
    if (tid == 0) s_lbase[0] = longer;  // empty tiles last
    __syncthreads();
    if (tid < T) {
      const int32_t P = s_pages[tid], r = atomicAdd(&s_lbase[P], 1);
      s_q[r] = P;
      s_rt[r] = tid;
    } else if (tid < p.G) {
      s_q[tid] = 0;
    }
    __syncthreads();
    const int32_t U = kPlanCosts.unit_x16, half = p.G / 2;
    int32_t v = 0;
    if (tid < half) {
      const int32_t qk = s_q[p.G - 1 - tid];
      v = 16 * (s_q[tid] + qk) + U + (qk > 0 ? U : 0);
    }
    v = wave_incl_max(v);  // running max inside the wave, then over the waves before
    if (lane == 63) s_red32[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v = s_red32[w] > v ? s_red32[w] : v;
    if (tid < half) s_pm[tid] = v;
    __syncthreads();
    auto count_long = [&](int32_t C) {  // first rank with q_r <= C (q descends)
      int32_t lo = 0, hi = T;
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (s_q[mid] > C) lo = mid + 1; else hi = mid;
      }
      return lo;
    };
    const int32_t C = tid + 1;
    int64_t key = INT64_MAX;
    if (C < s_q[0]) {
      const int32_t n = count_long(C);
      if (2 * n <= p.G && 2 * n <= p.ws.max_partials) {
        int64_t mk = 16 * (int64_t)C + U;
        if (n > 0 && (int64_t)s_pm[n - 1] - 16 * C > mk) mk = (int64_t)s_pm[n - 1] - 16 * C;
        const int64_t cost = (int64_t)p.G * (mk + kPlanCosts.split_x16) + 2 * (int64_t)n * kPlanCosts.combine_x16;
        key = (cost << 10) | (kMaxUnitPages - C);  // ties: the larger cap
      }
    }
    key = __ockl_wfred_min_i64(key);
    __syncthreads();  // every wave is past its reads of s_red32
    if (lane == 0) s_red64[wave] = key;
    __syncthreads();
    key = INT64_MAX;
    for (int w = 0; w < 16; ++w) key = s_red64[w] < key ? s_red64[w] : key;
    fold = key != INT64_MAX && (key >> 10) < s_best;
    if (fold) {
      cap = kMaxUnitPages - (int32_t)(key & 1023);
      nl = count_long(cap);
    }
  }
  auto tile_units = [&](int32_t t, int32_t P, int32_t* n, int32_t* sp) {
    if (fold) {
      *n = P > cap ? 2 : (P > 0 ? 1 : 0);
      *sp = P > cap ? 2 : 0;
    } else {
      *n = P > 0 ? ceil_div(P, c) : 0;
      *sp = (*n > 1 || shard) ? *n : 0;
    }
  };

  // 3. scan units / partial slots / split tiles over the tiles, write the list.
  int32_t carry_u = 0, carry_s = 0, carry_f = 0;
  for (int32_t base = 0; base < T; base += 1024) {
    const int32_t t = base + tid;
    const int32_t P = t < T ? pages_of(t) : 0;
    int32_t n = 0, sp = 0;
    if (t < T) tile_units(t, P, &n, &sp);
    const int32_t f = (sp > 0 || (list_empty && t < T && P == 0)) ? 1 : 0;
    int32_t tu, ts, tf, eu, es, ef;
    block_exclusive_scan3(n, sp, f, s_scan, &eu, &es, &ef, &tu, &ts, &tf);
    eu += carry_u;
    es += carry_s;
    ef += carry_f;
    if (t < T) {
      if (cached) {
        s_ufirst[t] = eu;
        s_sfirst[t] = es;
      } else {
        for (int32_t u = 0; u < n && eu + u < p.ws.max_units; ++u) {
          int4 rec;
          rec.x = t;
          rec.y = unit_begin(P, n, u);
          rec.z = unit_begin(P, n, u + 1);
          rec.w = (n > 1 || shard) ? es + u : -1;
          p.ws.units[eu + u] = rec;
        }
      }
      p.ws.indptr[t] = es < p.ws.max_partials ? es : p.ws.max_partials;
      if (f) {
        // the same (clamped) range as indptr[t], indptr[t + 1]
        const int32_t mp = p.ws.max_partials;
        const int32_t r0 = es < mp ? es : mp, r1 = es + sp < mp ? es + sp : mp;
        p.ws.split_list[ef] = make_int4(t, r0, r1 - r0, 0);
      }
    }
    carry_u += tu;
    carry_s += ts;
    carry_f += tf;
  }
  // 4. unit records.  A fold plan writes them worker by worker (worker r:
  // its own tile, or the head of it, then the tail it takes over) together
  // with each worker's first unit.  Otherwise (cached case) one thread per
  // unit finds its tile by binary search over the first-unit offsets; with
  // more units than workers the queue is ordered longest unit first (a
  // counting sort over unit lengths; the order among units of equal length
  // is whatever the LDS atomics give, and does not change any result); the
  // attend kernel deals it to its workers in a snake, which pairs the longest
  // units of one pass with the shortest of the next the way a
  // longest-processing-time-first schedule would; with at most one unit per
  // worker every unit starts at once: tile order.
  if (fold) {
    __syncthreads();  // partial offsets of every tile
    const int32_t r = tid;
    const bool own = r < T && s_q[r] > 0, tail = r < p.G && r >= p.G - nl;
    int32_t total;
    const int32_t base = block_exclusive_scan((int32_t)own + (int32_t)tail, s_scan, &total);
    if (own) {
      const int32_t t = s_rt[r], P = s_q[r];
      p.ws.units[base] = r < nl ? make_int4(t, 0, cap, s_sfirst[t]) : make_int4(t, 0, P, -1);
    }
    if (tail) {
      const int32_t j = p.G - 1 - r, t = s_rt[j];
      p.ws.units[base + (int32_t)own] = make_int4(t, cap, s_q[j], s_sfirst[t] + 1);
    }
    if (r < p.G) hdr[kHdrWorkerTable + r] = base;
    if (r == 0) hdr[kHdrWorkerTable + p.G] = total;
  } else if (cached) {
    if (tid == 0) s_ufirst[T] = carry_u;
    for (int32_t i = tid; i <= kMaxUnitPages; i += 1024) s_lhist[i] = 0;
    __syncthreads();
    const int32_t NU = carry_u < p.ws.max_units ? carry_u : p.ws.max_units;
    auto unit_rec = [&](int32_t ug) {
      int32_t lo = 0, hi = T - 1;  // last tile with s_ufirst[t] <= ug
      while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (s_ufirst[mid] <= ug) lo = mid; else hi = mid - 1;
      }
      const int32_t t = lo, u = ug - s_ufirst[t];
      const int32_t P = s_pages[t];
      const int32_t n = s_ufirst[t + 1] - s_ufirst[t];
      const int32_t es = s_sfirst[t];
      int4 rec;
      rec.x = t;
      rec.y = unit_begin(P, n, u);
      rec.z = unit_begin(P, n, u + 1);
      rec.w = (n > 1 || shard) ? es + u : -1;
      return rec;
    };
    const bool lpt = NU > p.G;  // uniform
    // With query chunks the rows of a request read the same pages: the
    // queue keeps a request's units together (requests ordered by their
    // longest unit), unit index major, so that the rows of one page range sit
    // side by side and run on one XCD (see the attend kernel's dealing),
    // whose L2 serves the pages to every row.  Request b's range start sits
    // in s_q[b], its key in s_rt[b] (the fold plan's arrays, free here).
    const bool grouped = lpt && p.q_chunk > 1 && p.B <= kMaxWorkers && !shard;
    if (grouped) {
      for (int32_t b = tid; b < p.B; b += 1024) {
        const int32_t t0 = b * p.q_chunk, t1 = t0 + p.q_chunk;
        int32_t key = 0;
        for (int32_t t = t0; t < t1; ++t) {
          const int32_t n = s_ufirst[t + 1] - s_ufirst[t];
          if (n > 0) key = max(key, ceil_div(s_pages[t], n));
        }
        s_rt[b] = key;
        const int32_t cnt = s_ufirst[t1] - s_ufirst[t0];
        if (cnt > 0) atomicAdd(&s_lhist[key], cnt);  // 1 <= key <= kMaxUnitPages
      }
    } else {
      for (int32_t ug = tid; ug < NU; ug += 1024) {
        const int4 rec = unit_rec(ug);
        if (lpt) atomicAdd(&s_lhist[rec.z - rec.y], 1);  // 1 <= length <= kMaxUnitPages
        else p.ws.units[ug] = rec;
      }
    }
    __syncthreads();
    if (lpt) {
      // queue offset of each length: the number of longer units (thread i
      // takes length kMaxUnitPages - i)
      static_assert(kMaxUnitPages == 1024, "one thread per unit length");
      const int32_t len = kMaxUnitPages - tid;
      int32_t unused;
      s_lbase[len] = block_exclusive_scan(s_lhist[len], s_scan, &unused);
      __syncthreads();
      if (grouped) {
        for (int32_t b = tid; b < p.B; b += 1024) {
          const int32_t cnt = s_ufirst[(b + 1) * p.q_chunk] - s_ufirst[b * p.q_chunk];
          if (cnt > 0) s_q[b] = atomicAdd(&s_lbase[s_rt[b]], cnt);
        }
        __syncthreads();
        for (int32_t ug = tid; ug < NU; ug += 1024) {
          const int4 rec = unit_rec(ug);
          const int32_t b = rec.x / p.q_chunk, i = rec.x - b * p.q_chunk, u = ug - s_ufirst[rec.x];
          // rank in unit-major order: sum_r min(u, n_r) + #{r < i : n_r > u}
          int32_t rank = 0;
          for (int32_t r = 0; r < p.q_chunk; ++r) {
            const int32_t t = b * p.q_chunk + r, n = s_ufirst[t + 1] - s_ufirst[t];
            rank += min(u, n) + ((r < i && n > u) ? 1 : 0);
          }
          p.ws.units[s_q[b] + rank] = rec;
        }
      } else {
        for (int32_t ug = tid; ug < NU; ug += 1024) {
          const int4 rec = unit_rec(ug);
          p.ws.units[atomicAdd(&s_lbase[rec.z - rec.y], 1)] = rec;
        }
      }
    }
  }
  if (tid == 0) {
    p.ws.indptr[T] = carry_s;
    hdr[kHdrGrab] = 0;
    hdr[kHdrDone] = 0;
    hdr[kHdrUnits] = carry_u < p.ws.max_units ? carry_u : p.ws.max_units;
    hdr[kHdrPartials] = carry_s;
    hdr[kHdrChunk] = fold ? 0 : c;
    hdr[kHdrSplitTiles] = carry_f;
    hdr[kHdrTotalPages] = total_pages > INT32_MAX ? INT32_MAX : (int32_t)total_pages;
    // every split tile has at most this many parts
    hdr[kHdrMaxParts] = fold ? (nl > 0 ? 2 : 1) : (max_pages + c - 1) / c;
    hdr[kHdrSchedule] = fold ? p.G : 0;
    hdr[kHdrFoldCap] = fold ? cap : 0;
  }
}

// ============================================================== combine ===

constexpr int kCombineQuarters = 4;  // waves per (row, head): 128 columns each
constexpr int kCombineRowParts = 8;  // at most this many parts: one wave per (row, head)
//
// The standalone merge of fp32 partials by split offsets (splash_mla_combine).
// Four wave slots per (request, chunk row, head), 128 columns each (2 per
// lane).  With at most 8 parts every lane loads all parts' LSEs and its
// columns of all parts at once; with more, the LSEs are reduced across the
// lanes first and sixteen parts' columns are in flight at a time.
__global__ __launch_bounds__(256) void combine_kernel(CombineLaunch c) {
  const int lane = threadIdx.x & 63;
  const int64_t wave_global = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  if (c.B <= 0) return;
  const size_t stride = (size_t)c.q_chunk * c.H;  // between parts
  // output row of (item b, chunk row qi): b * q_chunk + qi, or its place
  // among the shards
  auto out_row = [&](int b, int qi) -> size_t {
    const size_t r = (size_t)b * c.q_chunk + qi;
    if (c.num_shards <= 0) return r;
    const size_t rb = r / (size_t)c.tile_q, ri = r - rb * (size_t)c.tile_q;
    return (rb * c.num_shards + c.shard) * c.tile_q + ri;
  };
  // One wave per (item, row, head) with at most kCombineRowParts parts: 8
  // columns per lane, every part's LSE and columns loaded at once, so the row
  // costs one round trip to memory for its data and no cross-lane reduction.
  auto row_merge = [&](int b, int s0, int np, int qi, int hh) {
    const size_t base = (size_t)qi * c.H + hh;
    const size_t orow = out_row(b, qi) * c.H + hh;
    const float* plse = c.partial_lse + base;
    f32x4 v[kCombineRowParts][2];
    float w[kCombineRowParts];
    const float* prow = c.partials + base * kDimV + 8 * lane;
#pragma unroll
    for (int u = 0; u < kCombineRowParts; ++u) {
      w[u] = -INFINITY;
      v[u][0] = v[u][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (u < np) {  // uniform
        w[u] = plse[(size_t)(s0 + u) * stride];
        const f32x4* src = (const f32x4*)(prow + (size_t)(s0 + u) * stride * kDimV);
        v[u][0] = src[0];
        v[u][1] = src[1];
      }
    }
    float M = -INFINITY, wsum = 0.f;
#pragma unroll
    for (int u = 0; u < kCombineRowParts; ++u) M = fmaxf(M, w[u]);
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    if (M > -INFINITY) {
#pragma unroll
      for (int u = 0; u < kCombineRowParts; ++u) {
        const float wu = __expf(w[u] - M);  // 0 past the last part
        wsum += wu;
        acc0 += wu * v[u][0];
        acc1 += wu * v[u][1];
      }
    }
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    if (c.out_f32) {
      f32x4* dst = (f32x4*)((float*)c.out + orow * kDimV + 8 * lane);
      dst[0] = acc0 * inv;
      dst[1] = acc1 * inv;
    } else {
      u32x4 o4;
      o4[0] = pack_bf16x2(acc0[0] * inv, acc0[1] * inv);
      o4[1] = pack_bf16x2(acc0[2] * inv, acc0[3] * inv);
      o4[2] = pack_bf16x2(acc1[0] * inv, acc1[1] * inv);
      o4[3] = pack_bf16x2(acc1[2] * inv, acc1[3] * inv);
      *(u32x4*)((uint16_t*)c.out + orow * kDimV + 8 * lane) = o4;
    }
    if (lane == 0 && c.out_lse) c.out_lse[orow] = wsum > 0.f ? M + __logf(wsum) : -INFINITY;
  };
  // one (request or tile, row, head, quarter) item
  auto combine_item = [&](int b, int s0, int s1, int quarter, int qi, int hh) {
    const size_t orow = out_row(b, qi) * c.H + hh;
    const int nparts = s1 - s0;
    const size_t base = (size_t)qi * c.H + hh;
    const float* plse = c.partial_lse + base;
    const int col = 128 * quarter + 2 * lane;
    // the lane's 2 columns of part s (fp32 partials: this path serves the
    // standalone merge)
    auto part2 = [&](int sp) -> f32x2 { return *(const f32x2*)(c.partials + ((size_t)sp * stride + base) * kDimV + col); };
    float M = -INFINITY, wsum = 0.f;
    f32x2 acc = {0.f, 0.f};
    if (nparts <= 8) {
      // few parts: every lane loads every part's LSE itself (the same 32
      // bytes for the whole wave) together with its 2 columns of every part,
      // so the row costs one round trip to memory and no cross-lane reduction
      f32x2 v[8];
      float w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        w[u] = -INFINITY;
        v[u] = (f32x2){0.f, 0.f};
        if (u < nparts) {  // uniform
          w[u] = plse[(size_t)(s0 + u) * stride];
          v[u] = part2(s0 + u);
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) M = fmaxf(M, w[u]);
      if (M > -INFINITY) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float wu = __expf(w[u] - M);  // 0 past the last part
          wsum += wu;
          acc += wu * v[u];
        }
      }
    } else {
      for (int s = s0 + lane; s < s1; s += 64) M = fmaxf(M, plse[(size_t)s * stride]);
      M = __ockl_wfred_max_f32(M);
      if (M > -INFINITY)
        for (int s = s0 + lane; s < s1; s += 64) wsum += __expf(plse[(size_t)s * stride] - M);
      wsum = __ockl_wfred_add_f32(wsum);
      // many parts: sixteen parts' columns in flight at a time
      if (M > -INFINITY) {
        constexpr int kU = 16;
        int s = s0;
        for (; s + kU <= s1; s += kU) {
          f32x2 v[kU];
          float w[kU];
#pragma unroll
          for (int u = 0; u < kU; ++u) {
            v[u] = part2(s + u);
            w[u] = plse[(size_t)(s + u) * stride];
          }
#pragma unroll
          for (int u = 0; u < kU; ++u) acc += __expf(w[u] - M) * v[u];
        }
        if (s < s1) {
          // the remaining parts: independent loads, clamped to a valid part
          f32x2 v[kU];
          float w[kU];
#pragma unroll
          for (int u = 0; u < kU; ++u) {
            const int su = s + u < s1 ? s + u : s1 - 1;
            v[u] = part2(su);
            w[u] = s + u < s1 ? plse[(size_t)su * stride] : -INFINITY;
          }
#pragma unroll
          for (int u = 0; u < kU; ++u) acc += __expf(w[u] - M) * v[u];
        }
      }
    }
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    if (c.out_f32)
      *(f32x2*)((float*)c.out + orow * kDimV + col) = acc * inv;
    else
      *(unsigned*)((uint16_t*)c.out + orow * kDimV + col) = pack_bf16x2(acc[0] * inv, acc[1] * inv);
    if (lane == 0 && quarter == 0 && c.out_lse) c.out_lse[orow] = wsum > 0.f ? M + __logf(wsum) : -INFINITY;
  };
  {
    // one wave per (request, row, head), which takes the one-round-trip row
    // merge when the request has at most kCombineRowParts parts and
    // otherwise the four quarters in turn
    const int64_t per_b = (int64_t)c.q_chunk * c.H;
    for (int64_t item = wave_global; item < (int64_t)c.B * per_b; item += nwaves) {
      const int b = (int)(item / per_b);
      const int row = (int)(item - (int64_t)b * per_b);
      const int qi = row / c.H, hh = row - qi * c.H;
      const int s0 = c.indptr[b], s1 = c.indptr[b + 1];
      if (s1 <= s0 && !c.write_empty) continue;
      if (s1 - s0 <= kCombineRowParts) {
        row_merge(b, s0, s1 - s0, qi, hh);
      } else {
        for (int quarter = 0; quarter < kCombineQuarters; ++quarter) combine_item(b, s0, s1, quarter, qi, hh);
      }
    }
  }
}

// The merge of one step's split partials (splash_mla_combine_splits): the
// attend kernel's fp16 partials with their quarter exponents, the split
// tiles listed by the planner.  Every (tile, chunk row, head) row is one
// item; a lane holds 8 of its 512 columns (quarter lane / 16).  With at most
// kMergeWaveParts parts per tile (the plan's bound), or with at least
// kMergeWaveItems items of at most kMergeWaveLongParts parts (items enough
// to fill the chip with waves, so a workgroup per item would only queue
// them), a wave takes an item alone; otherwise a workgroup takes it and its
// four waves split the parts.  Either way parts go kMergeBatch at a time,
// one memory round trip per batch, against a running maximum of their LSEs
// (the sums rescaled when it grows); the four waves of a workgroup meet in
// LDS.  Few registers, so that many waves hide the round trips.
constexpr int kMergeWaveParts = 4;
constexpr int kMergeWaveItems = 8192;
constexpr int kMergeWaveLongParts = 16;
constexpr int kMergeBatch = 4;
__global__ __launch_bounds__(256) void merge_splits_kernel(CombineLaunch c) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t nitems = (int64_t)(*c.item_count) * c.q_chunk * c.H;
  if (nitems == 0) return;
  const int max_parts = *c.max_parts;
  const bool by_wave = max_parts <= kMergeWaveParts ||
                       (nitems >= kMergeWaveItems && max_parts <= kMergeWaveLongParts);  // uniform
  const size_t stride = (size_t)c.q_chunk * c.H;          // between parts
  const int qsh = 8 * (lane >> 4);
  // parts first, first + step, ... of an item: running max m, weight sum,
  // column sums
  auto accumulate = [&](const int4& rec, size_t base, int first, int step, float& m, float& ssum, f32x4& acc0,
                        f32x4& acc1) {
    const int s0 = rec.y, np = rec.z;
    const float* plse = c.partial_lse + base;
    const uint16_t* prow = c.partials_h + base * kDimV + 8 * lane;
    for (int u0 = first; u0 < np; u0 += step * kMergeBatch) {
      u32x4 raw[kMergeBatch];
      float wu[kMergeBatch];
      uint32_t ew[kMergeBatch];
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) {
        const int u = u0 + step * k;
        raw[k] = (u32x4){0, 0, 0, 0};
        wu[k] = -INFINITY;
        ew[k] = 0;
        if (u < np) {  // uniform
          const size_t r = (size_t)(s0 + u) * stride;
          raw[k] = *(const u32x4*)(prow + r * kDimV);
          wu[k] = plse[r];
          ew[k] = c.part_exp[r + base];
        }
      }
      float bm = -INFINITY;
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) bm = fmaxf(bm, wu[k]);
      if (bm > -INFINITY) {  // uniform
        const float mn = fmaxf(m, bm), rs = __expf(m - mn);  // 0 while m is -inf
        acc0 *= rs;
        acc1 *= rs;
        ssum *= rs;
        m = mn;
#pragma unroll
        for (int k = 0; k < kMergeBatch; ++k) {
          const int e = (int)((ew[k] >> qsh) & 255u);
          const float sc = __expf(wu[k] - m);  // 0 for parts past the end
          ssum += sc;
          acc0 += sc * unpack_f16x4(raw[k][0], raw[k][1], e);
          acc1 += sc * unpack_f16x4(raw[k][2], raw[k][3], e);
        }
      }
    }
  };
  auto store = [&](const int4& rec, int qi, int hh, float M, float wsum, const f32x4& acc0, const f32x4& acc1) {
    size_t r = (size_t)rec.x * c.q_chunk + qi;
    if (c.num_shards > 0) {
      const size_t rb = r / (size_t)c.tile_q, ri = r - rb * (size_t)c.tile_q;
      r = (rb * c.num_shards + c.shard) * c.tile_q + ri;
    }
    const size_t orow = r * c.H + hh;
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    if (c.out_f32) {
      f32x4* dst = (f32x4*)((float*)c.out + orow * kDimV + 8 * lane);
      dst[0] = acc0 * inv;
      dst[1] = acc1 * inv;
    } else {
      u32x4 o4;
      o4[0] = pack_bf16x2(acc0[0] * inv, acc0[1] * inv);
      o4[1] = pack_bf16x2(acc0[2] * inv, acc0[3] * inv);
      o4[2] = pack_bf16x2(acc1[0] * inv, acc1[1] * inv);
      o4[3] = pack_bf16x2(acc1[2] * inv, acc1[3] * inv);
      *(u32x4*)((uint16_t*)c.out + orow * kDimV + 8 * lane) = o4;
    }
    if (lane == 0 && c.out_lse) c.out_lse[orow] = wsum > 0.f ? M + __logf(wsum) : -INFINITY;
  };
  const int64_t per_tile = (int64_t)c.q_chunk * c.H;
  if (by_wave) {
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t item = (int64_t)blockIdx.x * 4 + w; item < nitems; item += nwaves) {
      const int64_t ri = item / per_tile;
      const int row = (int)(item - ri * per_tile), qi = row / c.H, hh = row - qi * c.H;
      const int4 rec = c.item_list[ri];
      float m = -INFINITY, ssum = 0.f;
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
      accumulate(rec, (size_t)qi * c.H + hh, 0, 1, m, ssum, acc0, acc1);
      store(rec, qi, hh, m, ssum, acc0, acc1);
    }
    return;
  }
  __shared__ f32x4 s_acc[4][64][2];
  __shared__ float s_ms[4][2];
  for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
    const int64_t ri = item / per_tile;
    const int row = (int)(item - ri * per_tile), qi = row / c.H, hh = row - qi * c.H;
    const int4 rec = c.item_list[ri];
    float m = -INFINITY, ssum = 0.f;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    accumulate(rec, (size_t)qi * c.H + hh, w, 4, m, ssum, acc0, acc1);
    s_acc[w][lane][0] = acc0;
    s_acc[w][lane][1] = acc1;
    if (lane == 0) {
      s_ms[w][0] = m;
      s_ms[w][1] = ssum;
    }
    __syncthreads();
    if (w == 0) {
      float M = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) M = fmaxf(M, s_ms[v][0]);
      float wsum = 0.f;
      acc0 = acc1 = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (M > -INFINITY) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float f = __expf(s_ms[v][0] - M);  // 0 for a wave without parts
          wsum += f * s_ms[v][1];
          acc0 += f * s_acc[v][lane][0];
          acc1 += f * s_acc[v][lane][1];
        }
      }
      store(rec, qi, hh, M, wsum, acc0, acc1);
    }
    __syncthreads();  // s_acc and s_ms are free for the next item
  }
}

// =============================================================== gather ===
//
// Dense copy of every history through the page-address arithmetic of the
// attend kernel: token j of request b is row (block_table[b][j>>6] << 6) |
// (j & 63).  One block per request; 16-byte copies.
__global__ __launch_bounds__(256) void gather_kernel(const uint8_t* kv, const int32_t* bt, const int32_t* seq_lens,
                                                     int32_t B, int32_t bt_stride, int32_t row_bytes,
                                                     uint8_t* dense) {
  const int b = blockIdx.x;
  size_t off = 0;
  for (int r = 0; r < b; ++r) off += (size_t)seq_lens[r];
  const int s = seq_lens[b];
  const int chunks = row_bytes / 16;
  for (int64_t e = threadIdx.x; e < (int64_t)s * chunks; e += blockDim.x) {
    const int j = (int)(e / chunks), ch = (int)(e - (int64_t)j * chunks);
    const int phys = bt[(size_t)b * bt_stride + (j >> 6)];
    const uint8_t* src = kv + ((size_t)phys * kPage + (j & 63)) * row_bytes + ch * 16;
    *(u32x4*)(dense + (off + j) * row_bytes + ch * 16) = *(const u32x4*)src;
  }
}

// ================================================================ check ===
//
// Validates device data: q_chunk <= seq_lens[b] and every used block-table
// entry in [0, num_pages); under a shard also 0 <= key_begin[b] <= key_end[b]
// with key_begin[b] a page boundary, and only the shard's pages are used.
// Writes the smallest failing request + 1 (or 0).
// latent_kv (the fp8 latent-row pool, else null): once every page entry of a
// request is in range, each of its rows' four tile scales must be a positive
// normal power of two no larger than 2^63.
__global__ __launch_bounds__(256) void check_kernel(const int32_t* bt, const int32_t* seq_lens,
                                                    const int32_t* key_begin, const int32_t* key_end, int32_t B,
                                                    int32_t q_chunk, int32_t bt_stride, int32_t num_pages,
                                                    const uint8_t* latent_kv, int32_t* result) {
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    const int s = seq_lens[b];
    bool bad = s < q_chunk || (int64_t)(s + kPage - 1) / kPage > bt_stride;
    int lo = 0, hi = s;
    if (key_end) {
      lo = key_begin[b];
      hi = min(s, key_end[b]);
      bad = bad || lo < 0 || (lo & (kPage - 1)) != 0 || key_end[b] < lo;
    }
    if (!bad && hi > lo) {
      const int np = (hi + kPage - 1) / kPage;
      for (int k = lo / kPage + threadIdx.x; k < np; k += blockDim.x) {
        const int v = bt[(size_t)b * bt_stride + k];
        if (v < 0 || v >= num_pages) bad = true;
      }
    }
    if (latent_kv && !__syncthreads_or(bad) && hi > lo) {
      for (int j = lo + threadIdx.x; j < hi; j += blockDim.x) {
        const size_t row = (size_t)bt[(size_t)b * bt_stride + (j >> 6)] * kPage + (j & (kPage - 1));
        const u32x4 sc = *(const u32x4*)(latent_kv + row * kLatentRowBytes + 512);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint32_t e = (sc[t] >> 23) & 0xFF;
          if ((sc[t] & 0x807FFFFFu) != 0 || e == 0 || e > 127 + 63) bad = true;
        }
      }
    }
    if (bad) atomicMin(result, b + 1);
  }
}

__global__ void init_check(int32_t* result) { *result = INT32_MAX; }

// Top-k variant: every row's count in [0, topk], every used position in the
// row's visible prefix [0, s_b - q_chunk + i], and its page's block-table
// entry in [0, num_pages); with the fp8 latent-row pool (latent_kv non-null)
// also each listed row's four tile scales a positive normal power of two
// no larger than 2^63.
// Writes the smallest failing row + 1 (or 0).
__global__ __launch_bounds__(256) void topk_check_kernel(const int32_t* bt, const int32_t* seq_lens,
                                                         const int32_t* idx, const int32_t* count, int32_t N,
                                                         int32_t q_chunk, int32_t topk, int32_t bt_stride,
                                                         int32_t num_pages, const uint8_t* latent_kv,
                                                         int32_t* result) {
  for (int n = blockIdx.x; n < N; n += gridDim.x) {
    const int b = n / q_chunk, i = n - b * q_chunk;
    const int s = seq_lens[b], c = count[n];
    const int vis = s - q_chunk + i + 1;
    bool bad = s < q_chunk || (int64_t)(s + kPage - 1) / kPage > bt_stride || c < 0 || c > topk;
    if (!bad) {
      for (int e = threadIdx.x; e < c; e += blockDim.x) {
        const int pos = idx[(size_t)n * topk + e];
        if (pos < 0 || pos >= vis) {
          bad = true;
        } else {
          const int pg = bt[(size_t)b * bt_stride + (pos >> 6)];
          if (pg < 0 || pg >= num_pages) {
            bad = true;
          } else if (latent_kv) {
            const size_t row = (size_t)pg * kPage + (pos & (kPage - 1));
            const u32x4 sc = *(const u32x4*)(latent_kv + row * kLatentRowBytes + 512);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const uint32_t ex = (sc[t] >> 23) & 0xFF;
              if ((sc[t] & 0x807FFFFFu) != 0 || ex == 0 || ex > 127 + 63) bad = true;
            }
          }
        }
      }
    }
    if (bad) atomicMin(result, n + 1);
  }
}

// ============================================================ launchers ===

hipError_t launch_plan(const PlanLaunch& p, hipStream_t s) {
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_attend(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  // fp8 caches: QK on the fp8 pipe unless the caller asked for the exact one
  const bool topk = a.topk_idx != nullptr;
  if (a.kv_dtype == 2 && a.exact_qk) (topk ? launch_attend_exact_latent_topk : launch_attend_exact_latent)(a, workers, s);
  else if (a.kv_dtype == 1 && a.exact_qk) (topk ? launch_attend_exact_fp8_topk : launch_attend_exact_fp8)(a, workers, s);
  else if (a.kv_dtype == 2) (topk ? launch_attend_latent_topk : launch_attend_latent)(a, workers, s);
  else if (a.kv_dtype == 1) (topk ? launch_attend_fp8_topk : launch_attend_fp8)(a, workers, s);
  else (topk ? launch_attend_bf16_topk : launch_attend_bf16)(a, workers, s);
  return hipGetLastError();
}

hipError_t launch_combine(const CombineLaunch& c, hipStream_t s) {
  if (c.item_list) {
    // the step's split tiles (their number is on the device): a block per
    // (tile, row, head) up to the bound, the kernel strides over the rest
    int64_t blocks = (int64_t)c.B * c.q_chunk * c.H;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(merge_splits_kernel, dim3((unsigned)blocks), dim3(256), 0, s, c);
    return hipGetLastError();
  }
  int64_t items = (int64_t)c.B * c.q_chunk * c.H * kCombineQuarters;
  int64_t blocks = (items + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(combine_kernel, dim3((unsigned)blocks), dim3(256), 0, s, c);
  return hipGetLastError();
}

hipError_t launch_gather(const void* kv, const int32_t* bt, const int32_t* seq_lens, int32_t B, int32_t bt_stride,
                         int32_t row_bytes, void* dense, hipStream_t s) {
  hipLaunchKernelGGL(gather_kernel, dim3(B), dim3(256), 0, s, (const uint8_t*)kv, bt, seq_lens, B, bt_stride,
                     row_bytes, (uint8_t*)dense);
  return hipGetLastError();
}

hipError_t launch_topk_check(const int32_t* bt, const int32_t* seq_lens, const int32_t* idx, const int32_t* count,
                             int32_t N, int32_t q_chunk, int32_t topk, int32_t bt_stride, int32_t num_pages,
                             const void* latent_kv, int32_t* result, hipStream_t s) {
  hipLaunchKernelGGL(init_check, dim3(1), dim3(1), 0, s, result);
  int blocks = N < 1024 ? N : 1024;
  hipLaunchKernelGGL(topk_check_kernel, dim3(blocks), dim3(256), 0, s, bt, seq_lens, idx, count, N, q_chunk, topk,
                     bt_stride, num_pages, (const uint8_t*)latent_kv, result);
  return hipGetLastError();
}

hipError_t launch_check(const int32_t* bt, const int32_t* seq_lens, const void* latent_kv, const int32_t* key_begin,
                        const int32_t* key_end, int32_t B, int32_t q_chunk, int32_t bt_stride, int32_t num_pages,
                        int32_t* result, hipStream_t s) {
  hipLaunchKernelGGL(init_check, dim3(1), dim3(1), 0, s, result);
  int blocks = B < 1024 ? B : 1024;
  hipLaunchKernelGGL(check_kernel, dim3(blocks), dim3(256), 0, s, bt, seq_lens, key_begin, key_end, B, q_chunk,
                     bt_stride, num_pages, (const uint8_t*)latent_kv, result);
  return hipGetLastError();
}

}  // namespace splash
