// Sampling epilogues of the two model calls of Algorithm 1, on fp32 logits.
//
// Drafting call: row 0 gives x_{n+1} (an ordinary sample, not part of the draft), row t gives
// draft t; the rows' ln-sum-exp is kept so that the validation call can evaluate d_t(x).
// Validation call: accept draft t iff  ln r_t + ln d_t(x) < ln p_t(x)  (r < min(1, p/d)), in
// order; the first reject is replaced by a draw from the normalised (p_t - d_t)_+; if all k are
// accepted one more token is drawn from the last row.  Then kv_len += 1 + a: rows of rejected
// drafts stay in the cache as dead entries.
//
// Every "draw" is a Gumbel-max: argmax_j (score_j - ln(-ln u_j)), u_j from Philox4x32-10 with
// key = seed and counter = (j/4, iteration, row | purpose << 8, sequence id); an argmax is
// independent of reduction order, so wavefront reductions give the same winner as a serial loop.
// Ties go to the lowest index, a NaN loses against every number.  temperature == 0 is greedy (argmax of the logits).
//
// Top-k sampling (the paper's sampler, Experimental setup: k = 10, and 25 for pass@10): the draft
// and the target distribution are each the softmax over the row's own K largest logits, zero
// elsewhere; ties at the boundary keep the lower indices.  A row's filter is two numbers found by
// a radix select over order-preserving integer keys: the key of the K-th largest logit and the
// highest index that may still be kept among the logits equal to it.  Entries outside the filter
// are skipped by every scan (ln-sum-exp, draws, residual) and have probability zero in the accept
// test.  K = 0 is no filter (key 0, every index allowed).
#include <type_traits>

#include "pass_internal.h"

namespace pass {

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    // one 32 x 32 -> 64 bit multiply per product (v_mad_u64_u32) instead of a high and a low one
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// top 23 bits -> (bits + 0.5) * 2^-23, in (0,1), exact in fp32
__device__ __forceinline__ float u01(uint32_t x) { return ((float)(x >> 9) + 0.5f) * (1.0f / 8388608.0f); }
// The per-element transcendentals use the hardware exp2 / log2 (absolute error around 1e-6 on
// the scores in play), inside the fp32 margin the decision comparison allows; the ln-sum-exp
// totals, the accept test and the merges of partial sums, a handful of values per row, stay precise.
__device__ __forceinline__ float gumbel(float u) { return -__logf(-__logf(u)); }

struct Best {
  float s;
  int idx;
};
__device__ __forceinline__ Best better(Best a, Best b) {
  // larger score wins, any number wins against a NaN; equal scores: lower index; idx < 0 means "no candidate"
  if (b.idx < 0) return a;
  if (a.idx < 0) return b;
  const bool nan_a = a.s != a.s, nan_b = b.s != b.s;
  if (b.s > a.s || (nan_a && !nan_b) || ((b.s == a.s || (nan_a && nan_b)) && b.idx < a.idx)) return b;
  return a;
}
__device__ __forceinline__ Best wave_best(Best v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    Best t;
    t.s = __shfl_xor(v.s, o);
    t.idx = __shfl_xor(v.idx, o);
    v = better(v, t);
  }
  return v;
}

struct MaxSum {
  float m, s;  // running max and sum of exp(a - m)
};
__device__ __forceinline__ MaxSum ms_merge(MaxSum a, MaxSum b) {
  if (b.m == -INFINITY) return a;
  if (a.m == -INFINITY) return b;
  MaxSum r;
  r.m = fmaxf(a.m, b.m);
  r.s = a.s * expf(a.m - r.m) + b.s * expf(b.m - r.m);
  return r;
}
__device__ __forceinline__ MaxSum wave_ms(MaxSum v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    MaxSum t;
    t.m = __shfl_xor(v.m, o);
    t.s = __shfl_xor(v.s, o);
    v = ms_merge(v, t);
  }
  return v;
}

constexpr int kEpiThreads = 1024;
constexpr int kEpiWaves = kEpiThreads / 64;

__device__ Best block_best(Best v, Best *sh) {
  v = wave_best(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  v = sh[threadIdx.x & (kEpiWaves - 1)];  // sixteen wavefronts' results in four exchanges
#pragma unroll
  for (int o = kEpiWaves / 2; o > 0; o >>= 1) {
    Best t;
    t.s = __shfl_xor(v.s, o);
    t.idx = __shfl_xor(v.idx, o);
    v = better(v, t);
  }
  return v;
}
__device__ MaxSum block_ms(MaxSum v, MaxSum *sh) {
  v = wave_ms(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  v = sh[threadIdx.x & (kEpiWaves - 1)];
#pragma unroll
  for (int o = kEpiWaves / 2; o > 0; o >>= 1) {
    MaxSum t;
    t.m = __shfl_xor(v.m, o);
    t.s = __shfl_xor(v.s, o);
    v = ms_merge(v, t);
  }
  return v;
}

// Walk NR logits rows of V entries in groups of four consecutive entries ("quads", the unit one
// Philox call covers): f(quad index, values[NR][4], number of valid entries).  A thread takes
// quads threadIdx.x, + kEpiThreads, ... in ascending order.  When V is a multiple of 4 a quad is
// one 16-byte load and the loads of four quads are issued before the first is used (indices
// clamped, results of quads that do not exist dropped): a load under a condition would be
// waited for on the spot, and a row is only V / (4 * kEpiThreads) quads deep per thread.
template <int NR, typename F>
__device__ __forceinline__ void scan_rows(const float *const (&rows)[NR], int V, F &&f) {
  if ((V & 3) == 0) {
    constexpr int U = 4;
    const int V4 = V >> 2;
    for (int q0 = threadIdx.x; q0 < V4; q0 += U * kEpiThreads) {
      float4 v[U][NR];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < NR; ++r) v[u][r] = ((const float4 *)rows[r])[min(q0 + u * kEpiThreads, V4 - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * kEpiThreads;
        if (q < V4) {
          float x[NR][4];
#pragma unroll
          for (int r = 0; r < NR; ++r) { x[r][0] = v[u][r].x; x[r][1] = v[u][r].y; x[r][2] = v[u][r].z; x[r][3] = v[u][r].w; }
          f(q, x, 4);
        }
      }
    }
  } else {
    for (int q = threadIdx.x; q * 4 < V; q += kEpiThreads) {
      const int n = min(4, V - q * 4);
      float x[NR][4];
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[r][e] = rows[r][q * 4 + min(e, n - 1)];
      f(q, x, n);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// top-k filter
// ---------------------------------------------------------------------------------------------
// order-preserving key of a logit: a > b  <=>  key(a) > key(b); -0 and +0 share a key
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
struct RowFilter {
  uint32_t key;  // key of the K-th largest logit (0: keep everything)
  int tie_max;   // highest index kept among the logits whose key equals `key`
};
__device__ __forceinline__ bool kept(const RowFilter &f, float l, int j) {
  uint32_t k = order_key(l);
  return k > f.key || (k == f.key && j <= f.tie_max);
}

constexpr int kSelBins = 2048;  // 11 + 11 + 10 bits
struct SelectShared {
  int hist[kSelBins];
  int wave_tot[kEpiWaves];
  int bin, rank;
};

// Exclusive prefix sum over the threads of the workgroup, in thread order.
__device__ int block_exclusive_scan(int v, int *wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int off = 0;
  for (int w = 0; w < wave; ++w) off += wave_tot[w];
  return off + inc - v;
}

// The histogram holds counts per digit; find the digit that contains the rank-th largest element
// (rank >= 1, counted from the top digit down) and the rank inside that digit.
__device__ void find_digit(SelectShared &sh, int n_bins, int rank, int &digit, int &rank_in) {
  const int bpt = n_bins / kEpiThreads;           // bins per thread (n_bins is a multiple of 512)
  const int hi = n_bins - threadIdx.x * bpt - 1;  // thread 0 owns the top bins
  int local = 0;
  for (int i = 0; i < bpt; ++i) local += sh.hist[hi - i];
  const int above = block_exclusive_scan(local, sh.wave_tot);
  if (above < rank && rank <= above + local) {
    int acc = above;
    for (int i = 0; i < bpt; ++i) {
      int c = sh.hist[hi - i];
      if (rank <= acc + c) { sh.bin = hi - i; sh.rank = rank - acc; break; }
      acc += c;
    }
  }
  __syncthreads();
  digit = sh.bin;
  rank_in = sh.rank;
  __syncthreads();
}

// Filter of one row for top-K sampling, by the whole workgroup: three counting passes over the
// row (it sits in L2: the LM head has just written it).  K <= 0 or K >= V: no filter.
__device__ RowFilter select_top_k(const float *row, int V, int K, SelectShared &sh) {
  RowFilter f;
  f.key = 0;
  f.tie_max = V;
  if (K <= 0 || K >= V) return f;
  const float *const rows[1] = {row};
  uint32_t prefix = 0, mask = 0;
  int rank = K;
  const int shifts[3] = {21, 10, 0}, bits[3] = {11, 11, 10};
  for (int pass = 0; pass < 3; ++pass) {
    const int n_bins = 1 << bits[pass];
    for (int i = threadIdx.x; i < kSelBins; i += kEpiThreads) sh.hist[i] = 0;
    __syncthreads();
    const int shift = shifts[pass];
    scan_rows<1>(rows, V, [&](int q4, const float (&x)[1][4], int n) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e < n) {
          uint32_t k = order_key(x[0][e]);
          if ((k & mask) == prefix) atomicAdd(&sh.hist[(k >> shift) & (n_bins - 1)], 1);
        }
      }
    });
    __syncthreads();
    int digit, rank_in;
    find_digit(sh, n_bins < kEpiThreads ? kEpiThreads : n_bins, rank, digit, rank_in);
    prefix |= (uint32_t)digit << shift;
    mask |= (uint32_t)(n_bins - 1) << shift;
    if (pass == 2) {
      // `rank_in` of the sh.hist[digit] logits equal to the threshold are kept: the lowest indices
      const int n_equal = sh.hist[digit];
      f.key = prefix;
      if (rank_in < n_equal) {
        // rare (exactly equal logits across the boundary): one thread walks the row in index order
        if (threadIdx.x == 0) {
          int seen = 0, j = 0;
          for (; j < V; ++j)
            if (order_key(row[j]) == prefix && ++seen == rank_in) break;
          sh.bin = j;
        }
        __syncthreads();
        f.tie_max = sh.bin;
        __syncthreads();
      }
    }
    rank = rank_in;
  }
  return f;
}

// Gumbel-max over softmax(logits * inv_t) (or plain argmax when greedy) fused with ln-sum-exp.
__device__ void sample_row(const float *logits, int V, bool greedy, float inv_t, uint32_t k0, uint32_t k1,
                           uint32_t c1, uint32_t c2, uint32_t c3, const RowFilter &flt, Best &best, MaxSum &ms) {
  best.s = -INFINITY;
  best.idx = -1;
  ms.m = -INFINITY;
  ms.s = 0.f;
  const float *const rows[1] = {logits};
  scan_rows<1>(rows, V, [&](int q4, const float (&x)[1][4], int n) {
    uint32_t rnd[4] = {0, 0, 0, 0};
    if (!greedy) philox4x32_10((uint32_t)q4, c1, c2, c3, k0, k1, rnd);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e < n && kept(flt, x[0][e], q4 * 4 + e)) {
        float l = x[0][e];
        float a = l * inv_t;
        if (a > ms.m) {
          ms.s = (ms.m == -INFINITY) ? 1.f : ms.s * __expf(ms.m - a) + 1.f;
          ms.m = a;
        } else {
          ms.s += __expf(a - ms.m);
        }
        Best c;
        c.s = greedy ? l : a + gumbel(u01(rnd[e]));
        c.idx = q4 * 4 + e;
        best = better(best, c);
      }
    }
  });
}

// A slot's counters, requested at the start of a kernel: read where they are needed they are two trips to memory at its end
struct SlotCounts {
  int n_gen, gen_limit, frozen, kv_len;
  uint32_t iter;
};
__device__ __forceinline__ SlotCounts slot_counts(const Params &p, int slot) {
  return SlotCounts{p.n_gen[slot], p.gen_limit[slot], p.frozen[slot], p.kv_len[slot], p.iter[slot]};
}
// x_{n+1} is accepted unconditionally: it joins the sequence, its predecessor's K/V stay
__device__ __forceinline__ void commit_first(const Params &p, const SampleArgs &a, int slot, int token, const SlotCounts &n) {
  p.first[slot] = token;
  const int frozen = n.n_gen >= n.gen_limit;
  p.frozen[slot] = frozen;
  if (a.commit && !frozen) {
    p.kv_len[slot] = n.kv_len + 1;
    p.pending[slot] = token;
    if (n.n_gen < p.gen_cap) p.gen[(size_t)slot * p.gen_cap + n.n_gen] = token;
    p.n_gen[slot] = n.n_gen + 1;
  }
}
// The accepted drafts and the final token y join the sequence.  By one wavefront, a token per lane; `draft`: lane t's draft t + 1.
__device__ __forceinline__ void commit_verified(const Params &p, const SampleArgs &a, int slot, int acc, int y, int draft, const SlotCounts &n) {
  const int t = threadIdx.x & 63;
  if (t > acc) return;  // acc <= k < 16
  const int x = t < acc ? draft : y;
  const bool live = a.commit && !n.frozen;
  p.last_out[slot * (kMaxK + 1) + t] = x;
  if (live && n.n_gen + t < p.gen_cap) p.gen[(size_t)slot * p.gen_cap + n.n_gen + t] = x;
  if (t != 0) return;
  p.n_acc[slot] = acc;
  if (live) {
    p.n_gen[slot] = n.n_gen + acc + 1;
    p.kv_len[slot] = n.kv_len + 1 + acc;  // K/V of x_{n+1} and of the accepted drafts are kept
    p.pending[slot] = y;
    p.iter[slot] = n.iter + 1;
  }
}
__device__ __forceinline__ int lane_draft(const Params &p, int slot) { return p.drafts[slot * kMaxK + min((int)(threadIdx.x & 63), kMaxK - 1)]; }

__global__ __launch_bounds__(kEpiThreads) void draft_epilogue_kernel(Params p, SampleArgs a, int R) {
  __shared__ Best sh_b[kEpiWaves];
  __shared__ MaxSum sh_m[kEpiWaves];
  __shared__ SelectShared sh_sel;
  int m = blockIdx.x, b = m / R, r = m % R;
  int slot = p.step_slots[b];
  if (a.stats_only && r == 0) return;  // row 0 of an externally drafted block is the last token, not a draft
  const float *logits = p.draft_logits + ((size_t)slot * (1 + p.k) + r) * p.V;
  bool greedy = a.temperature == 0.f;
  float inv_t = greedy ? 1.f : 1.f / a.temperature;
  const RowFilter flt = select_top_k(logits, p.V, greedy ? 0 : a.top_k, sh_sel);
  if (threadIdx.x == 0) {  // the validation call evaluates d_t through the same filter
    p.flt_key_d[slot * (kMaxK + 1) + r] = flt.key;
    p.flt_tie_d[slot * (kMaxK + 1) + r] = flt.tie_max;
  }
  const SlotCounts n = slot_counts(p, slot);
  Best best;
  MaxSum ms;
  sample_row(logits, p.V, greedy, inv_t, a.seed_lo, a.seed_hi, n.iter, (uint32_t)(r + a.row_base) | (PURPOSE_DRAFT << 8),
             p.seq_id[slot], flt, best, ms);
  best = block_best(best, sh_b);
  ms = block_ms(ms, sh_m);
  if (threadIdx.x == 0) {
    p.logz_d[slot * (kMaxK + 1) + r] = ms.m + logf(ms.s);
    if (a.stats_only) {
      // the tokens were drafted elsewhere
    } else if (r > 0) {
      p.drafts[slot * kMaxK + (r - 1)] = best.idx;
    } else {
      commit_first(p, a, slot, best.idx, n);
    }
  }
}

// ln-sum-exp (over the row's filter) and argmax of every validation row
__global__ __launch_bounds__(kEpiThreads) void verify_stats_kernel(Params p, SampleArgs a, int R) {
  __shared__ Best sh_b[kEpiWaves];
  __shared__ MaxSum sh_m[kEpiWaves];
  int m = blockIdx.x, b = m / R, r = m % R;
  int slot = p.step_slots[b];
  const float *logits = p.verify_logits + ((size_t)slot * (1 + p.k) + r) * p.V;
  __shared__ SelectShared sh_sel;
  bool greedy = a.temperature == 0.f;
  float inv_t = greedy ? 1.f : 1.f / a.temperature;
  const RowFilter flt = select_top_k(logits, p.V, greedy ? 0 : a.top_k, sh_sel);
  if (threadIdx.x == 0) {
    p.flt_key_p[slot * (kMaxK + 1) + r] = flt.key;
    p.flt_tie_p[slot * (kMaxK + 1) + r] = flt.tie_max;
  }
  Best best;
  MaxSum ms;
  sample_row(logits, p.V, true, inv_t, 0, 0, 0, 0, 0, flt, best, ms);
  best = block_best(best, sh_b);
  ms = block_ms(ms, sh_m);
  if (threadIdx.x == 0) {
    p.logz_p[slot * (kMaxK + 1) + r] = ms.m + logf(ms.s);
    p.argmax_p[slot * (kMaxK + 1) + r] = best.idx;
  }
}

__global__ __launch_bounds__(kEpiThreads) void verify_decide_kernel(Params p, SampleArgs a) {
  __shared__ Best sh_b[kEpiWaves];
  __shared__ int sh_a;
  const int slot = p.step_slots[blockIdx.x];
  const int k = p.k_act, V = p.V;  // rows of this call; the logits buffers keep the stride 1 + p.k
  const bool greedy = a.temperature == 0.f;
  const float inv_t = greedy ? 1.f : 1.f / a.temperature;
  const float *P = p.verify_logits + (size_t)slot * (1 + p.k) * V;
  const float *Dl = p.draft_logits + (size_t)slot * (1 + p.k) * V;
  const float *zp = p.logz_p + slot * (kMaxK + 1), *zd = p.logz_d + slot * (kMaxK + 1);
  const int32_t *drafts = p.drafts + slot * kMaxK;
  const SlotCounts n = slot_counts(p, slot);
  const int draft = lane_draft(p, slot);
  const uint32_t it = n.iter, sid = p.seq_id[slot];
  // row filters (top-k) found by the two statistics kernels; greedy never filters
  auto filter_p = [&](int row) {
    RowFilter f;
    f.key = greedy ? 0u : p.flt_key_p[slot * (kMaxK + 1) + row];
    f.tie_max = greedy ? V : p.flt_tie_p[slot * (kMaxK + 1) + row];
    return f;
  };
  auto filter_d = [&](int row) {
    RowFilter f;
    f.key = greedy ? 0u : p.flt_key_d[slot * (kMaxK + 1) + row];
    f.tie_max = greedy ? V : p.flt_tie_d[slot * (kMaxK + 1) + row];
    return f;
  };

  if (threadIdx.x == 0) {
    int acc = 0;
    for (int t = 1; t <= k; ++t) {
      int x = drafts[t - 1];
      bool ok;
      if (greedy) {
        ok = x == p.argmax_p[slot * (kMaxK + 1) + (t - 1)];
      } else {
        // a token outside a row's filter has probability zero there
        const float pl = P[(size_t)(t - 1) * V + x], dl = Dl[(size_t)t * V + x];
        float lp = kept(filter_p(t - 1), pl, x) ? pl * inv_t - zp[t - 1] : -INFINITY;
        float ld = kept(filter_d(t), dl, x) ? dl * inv_t - zd[t] : -INFINITY;
        uint32_t rnd[4];
        philox4x32_10(0u, it, (uint32_t)t | (PURPOSE_ACCEPT << 8), sid, a.seed_lo, a.seed_hi, rnd);
        ok = logf(u01(rnd[0])) + ld < lp;
      }
      if (!ok) break;
      acc += 1;
    }
    sh_a = acc;
  }
  __syncthreads();
  const int acc = sh_a;
  int y;
  if (greedy) {
    y = p.argmax_p[slot * (kMaxK + 1) + acc];
  } else if (acc == k) {
    Best best;
    MaxSum ms;
    sample_row(P + (size_t)k * V, V, false, inv_t, a.seed_lo, a.seed_hi, it, (uint32_t)(k + 1) | (PURPOSE_BONUS << 8),
               sid, filter_p(k), best, ms);
    y = block_best(best, sh_b).idx;
  } else {
    const float *pr = P + (size_t)acc * V, *dr = Dl + (size_t)(acc + 1) * V;
    const float z_p = zp[acc], z_d = zd[acc + 1];
    const uint32_t c2 = (uint32_t)(acc + 1) | (PURPOSE_RESIDUAL << 8);
    const RowFilter fp = filter_p(acc), fd = filter_d(acc + 1);
    Best best;
    best.s = -INFINITY;
    best.idx = -1;
    const float *const rows[2] = {pr, dr};
    scan_rows<2>(rows, V, [&](int q4, const float (&x)[2][4], int n_valid) {
      uint32_t rnd[4];
      philox4x32_10((uint32_t)q4, it, c2, sid, a.seed_lo, a.seed_hi, rnd);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e < n_valid) {
          const int j = q4 * 4 + e;
          float w = (kept(fp, x[0][e], j) ? __expf(x[0][e] * inv_t - z_p) : 0.f) -
                    (kept(fd, x[1][e], j) ? __expf(x[1][e] * inv_t - z_d) : 0.f);
          if (w > 0.f) {
            Best c;
            c.s = __logf(w) + gumbel(u01(rnd[e]));
            c.idx = q4 * 4 + e;
            best = better(best, c);
          }
        }
      }
    });
    best = block_best(best, sh_b);
    if (best.idx < 0) {
      // residual empty through rounding: draw from p_t with the same counters
      MaxSum ms;
      sample_row(pr, V, false, inv_t, a.seed_lo, a.seed_hi, it, c2, sid, fp, best, ms);
      best = block_best(best, sh_b);
      if (threadIdx.x == 0) atomicAdd(p.fallbacks, 1);
    }
    y = best.idx;
  }
  if (threadIdx.x < 64) commit_verified(p, a, slot, acc, y, draft, n);
}

// ---------------------------------------------------------------------------------------------
// The same epilogues for large vocabularies, every row spread over workgroups.  One workgroup per row is bound by the
// vector arithmetic of a single compute unit (exp, Philox, two logarithms per entry: 17 to 26 us for 32000 entries),
// while 250 units idle.  Here a workgroup takes 1024 entries of a row (4096 of very long rows) and leaves (max, sum, best) in a workspace; the kernel that follows merges the parts in order and goes on:
//   drafting    part, commit
//   validation  part, commit (greedy); part, draw, commit (sampled): the workgroups of `draw` each find the accept
//               count for themselves, then take their entries of the residual or bonus draw
// With top-k sampling a kernel of one workgroup per row finds the rows' filters first.  Every draw is an argmax over the
// same scores as above, whoever computes them.
// Measured at 32000 entries, seven rows, one sequence, T = 0.8: drafting 25.0 us -> 4.7 + 4.0, validation
// 16.4 + 25.3 -> 4.7 + 6.4 + 3.9; one greedy row: 17.2 -> 4.6 + 4.0 and 16.2 -> 4.6 + 4.0.
// ---------------------------------------------------------------------------------------------
// quads of four entries per thread of a part: one while that makes no more parts than the workspace holds (32000
// entries: 32 parts; with four per thread, eight parts, row_part and verify_draw took 8.8 and 13.6 us instead of 4.7 and 6.4), else four
constexpr int kPartThreads = 256;

// Wavefront reductions through DPP.  OP(v, the other lane's v) is only applied where the other lane exists; lane 63 ends
// with the result, which is handed to every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {  // masked rows get their own value back
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false);
}
template <typename F>
__device__ __forceinline__ void dpp_steps(F &&f) {
  f(std::integral_constant<int, 0xB1>{}, std::integral_constant<int, 0xF>{});   // quad_perm [1,0,3,2]
  f(std::integral_constant<int, 0x4E>{}, std::integral_constant<int, 0xF>{});   // quad_perm [2,3,0,1]
  f(std::integral_constant<int, 0x141>{}, std::integral_constant<int, 0xF>{});  // row_half_mirror
  f(std::integral_constant<int, 0x140>{}, std::integral_constant<int, 0xF>{});  // row_mirror
  f(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});  // row_bcast:15 into rows 1 and 3
  f(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});  // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ float lane63(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); }
__device__ __forceinline__ float wave_max_dpp(float v) {
  dpp_steps([&](auto C, auto R) { v = fmaxf(v, __uint_as_float(dpp_u32<C.value, R.value>(__float_as_uint(v)))); });
  return lane63(v);
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  dpp_steps([&](auto C, auto R) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), C.value, R.value, 0xF, false));
  });
  return lane63(v);
}
// A candidate as an integer that orders like better(): larger score first, a NaN last, then the lower index; 0 = no candidate
__device__ __forceinline__ uint64_t best_key(float s, int idx) { return (uint64_t)(s == s ? order_key(s) : 0u) << 32 | (uint32_t)~idx; }
__device__ __forceinline__ int key_index(uint64_t key) { return key ? (int)~(uint32_t)key : -1; }
__device__ __forceinline__ uint64_t wave_key_dpp(uint64_t k) {
  dpp_steps([&](auto C, auto R) {
    const uint64_t o = (uint64_t)dpp_u32<C.value, R.value>((uint32_t)(k >> 32)) << 32 | dpp_u32<C.value, R.value>((uint32_t)k);
    k = o > k ? o : k;
  });
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(k >> 32), 63) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)k, 63);
}
// (max, sum of exp) of the wavefront's lanes; a lane with no entry has max -inf and sum 0
__device__ __forceinline__ MaxSum wave_ms_dpp(float mx, float sum) {
  const float m = wave_max_dpp(mx);
  return MaxSum{m, wave_sum_dpp(mx == -INFINITY ? 0.f : sum * expf(mx - m))};
}

__device__ __forceinline__ RowFilter read_filter(const uint32_t *key, const int32_t *tie, int at, bool filtered, int V) {
  RowFilter f;
  f.key = filtered ? key[at] : 0u;
  f.tie_max = filtered ? tie[at] : V;
  return f;
}

__global__ __launch_bounds__(kEpiThreads) void row_filter_kernel(Params p, SampleArgs a, int R, int verify) {
  __shared__ SelectShared sh_sel;
  const int m = blockIdx.x, slot = p.step_slots[m / R], r = m % R;
  if (a.stats_only && r == 0) return;
  const float *row = (verify ? p.verify_logits : p.draft_logits) + ((size_t)slot * (1 + p.k) + r) * p.V;
  const RowFilter f = select_top_k(row, p.V, a.top_k, sh_sel);
  if (threadIdx.x == 0) {
    (verify ? p.flt_key_p : p.flt_key_d)[slot * (kMaxK + 1) + r] = f.key;
    (verify ? p.flt_tie_p : p.flt_tie_d)[slot * (kMaxK + 1) + r] = f.tie_max;
  }
}

// What U quads of a row (quads lo, lo + stride, ..., values in v) give: sum of exp over their maximum, and the best candidate
// (the draw when `draw`, else the largest logit).  A quad beyond the row counts for nothing.
template <int U>
__device__ __forceinline__ void score_quads(const float4 (&v)[U], int lo, int stride, int V4, const RowFilter &flt, float inv_t, bool draw,
                                            const SampleArgs &a, uint32_t it, uint32_t c2, uint32_t sid, float &mx, float &sum, uint64_t &key) {
  float l[4 * U];
  uint32_t keep = 0;
  mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = lo + u * stride;
    l[4 * u] = v[u].x; l[4 * u + 1] = v[u].y; l[4 * u + 2] = v[u].z; l[4 * u + 3] = v[u].w;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (q < V4 && kept(flt, l[4 * u + e], q * 4 + e)) {
        keep |= 1u << (4 * u + e);
        mx = fmaxf(mx, l[4 * u + e] * inv_t);
      }
  }
  sum = 0.f;
  key = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = lo + u * stride;
    uint32_t rnd[4] = {0, 0, 0, 0};
    if (draw && (keep >> (4 * u) & 15u)) philox4x32_10((uint32_t)q, it, c2, sid, a.seed_lo, a.seed_hi, rnd);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (keep >> (4 * u + e) & 1u) {
        const float x = l[4 * u + e], s = x * inv_t;
        sum += mx == -INFINITY ? 0.f : __expf(s - mx);
        const uint64_t k = best_key(draw ? s + gumbel(u01(rnd[e])) : x, q * 4 + e);
        key = k > key ? k : key;
      }
  }
}

// Part blockIdx.x of row blockIdx.y: (max, sum of exp, best candidate).  Validation rows keep the argmax of the
// logits as best, drafting rows the draw (also an argmax of the logits when greedy).
template <int U>
__global__ __launch_bounds__(kPartThreads) void row_part_kernel(Params p, SampleArgs a, int R, int verify, int filtered) {
  __shared__ float sh_m[4], sh_s[4];
  __shared__ uint64_t sh_k[4];
  const int m = blockIdx.y, slot = p.step_slots[m / R], r = m % R;
  if (a.stats_only && r == 0) return;
  const float *row = (verify ? p.verify_logits : p.draft_logits) + ((size_t)slot * (1 + p.k) + r) * p.V;
  const bool greedy = a.temperature == 0.f;
  const float inv_t = greedy ? 1.f : 1.f / a.temperature;
  const int at = slot * (kMaxK + 1) + r;
  const int V4 = p.V >> 2, lo = blockIdx.x * (U * kPartThreads) + threadIdx.x;
  float4 v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = ((const float4 *)row)[min(lo + u * kPartThreads, V4 - 1)];
  const RowFilter flt = read_filter(verify ? p.flt_key_p : p.flt_key_d, verify ? p.flt_tie_p : p.flt_tie_d, at, filtered, p.V);
  float mx, sum;
  uint64_t key;
  score_quads<U>(v, lo, kPartThreads, V4, flt, inv_t, !greedy && !verify, a, p.iter[slot], (uint32_t)(r + a.row_base) | (PURPOSE_DRAFT << 8),
                 p.seq_id[slot], mx, sum, key);
  const MaxSum ms = wave_ms_dpp(mx, sum);
  key = wave_key_dpp(key);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sh_m[wave] = ms.m; sh_s[wave] = ms.s; sh_k[wave] = key; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const float t = fmaxf(fmaxf(sh_m[0], sh_m[1]), fmaxf(sh_m[2], sh_m[3]));
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      total += sh_m[w] == -INFINITY ? 0.f : sh_s[w] * expf(sh_m[w] - t);
      key = sh_k[w] > key ? sh_k[w] : key;
    }
    p.row_parts[(size_t)m * kRowParts + blockIdx.x] = make_float4(t, total, __uint_as_float((uint32_t)(key >> 32)), __uint_as_float((uint32_t)key));
  }
}

// ln-sum-exp and best index of a row from its parts (lane i holds part i), by one wavefront; every lane gets both
__device__ __forceinline__ float4 load_part(const Params &p, int m, int parts) {
  return p.row_parts[(size_t)m * kRowParts + min((int)(threadIdx.x & 63), parts - 1)];
}
__device__ __forceinline__ void merge_parts(float4 v, int parts, float &logz, int &idx) {
  const bool own = (int)(threadIdx.x & 63) < parts;
  const MaxSum ms = wave_ms_dpp(own ? v.x : -INFINITY, own ? v.y : 0.f);
  const uint64_t key = wave_key_dpp(own ? (uint64_t)__float_as_uint(v.z) << 32 | __float_as_uint(v.w) : 0);
  logz = ms.m + logf(ms.s);
  idx = key_index(key);
}

__global__ __launch_bounds__(1024) void draft_commit_kernel(Params p, SampleArgs a, int R, int parts, int filtered) {
  const int b = blockIdx.x, slot = p.step_slots[b], r = threadIdx.x >> 6;  // a wavefront per row (R <= 16)
  if (r >= R || (a.stats_only && r == 0)) return;
  float logz;
  int idx;
  const SlotCounts n = slot_counts(p, slot);
  merge_parts(load_part(p, b * R + r, parts), parts, logz, idx);
  if ((threadIdx.x & 63) != 0) return;
  p.logz_d[slot * (kMaxK + 1) + r] = logz;
  if (!filtered) {  // the validation call evaluates d_t through the same filter
    p.flt_key_d[slot * (kMaxK + 1) + r] = 0u;
    p.flt_tie_d[slot * (kMaxK + 1) + r] = p.V;
  }
  if (a.stats_only) return;  // the tokens were drafted elsewhere
  if (r > 0) {
    p.drafts[slot * kMaxK + (r - 1)] = idx;
  } else {
    commit_first(p, a, slot, idx, n);
  }
}

// Accept test of draft t by lane t - 1.  What it needs of memory is requested before the rows' parts are merged.
struct AcceptOperands {
  int x;         // the draft
  float pl, dl;  // its logit in the target and in the draft row
  RowFilter fp, fd;
  float zd;
};
__device__ __forceinline__ AcceptOperands accept_operands(const Params &p, int slot, bool filtered, bool greedy) {
  const int t = min((int)(threadIdx.x & 63) + 1, max(p.k_act, 1)), V = p.V, base = slot * (kMaxK + 1);
  AcceptOperands o;
  o.x = p.drafts[slot * kMaxK + t - 1];
  if (greedy || p.k_act == 0) return o;
  const int x = clamp_token(p, o.x);
  o.pl = p.verify_logits[((size_t)slot * (1 + p.k) + t - 1) * V + x];
  o.dl = p.draft_logits[((size_t)slot * (1 + p.k) + t) * V + x];
  o.fp = read_filter(p.flt_key_p, p.flt_tie_p, base + t - 1, filtered, V);
  o.fd = read_filter(p.flt_key_d, p.flt_tie_d, base + t, true, V);
  o.zd = p.logz_d[base + t];
  return o;
}
// How many drafts are accepted, in every lane of the calling wavefront.  zp, argmax: of the validation rows (LDS).
__device__ __forceinline__ int count_accepted(const Params &p, const SampleArgs &a, int slot, const AcceptOperands &o, const float *zp,
                                              const int *argmax) {
  const int lane = threadIdx.x & 63;
  bool ok = false;
  if (lane < p.k_act) {
    const int t = lane + 1;
    if (a.temperature == 0.f) {
      ok = o.x == argmax[t - 1];
    } else {
      // a token outside a row's filter has probability zero there
      const float inv_t = 1.f / a.temperature;
      const float lp = kept(o.fp, o.pl, o.x) ? o.pl * inv_t - zp[t - 1] : -INFINITY;
      const float ld = kept(o.fd, o.dl, o.x) ? o.dl * inv_t - o.zd : -INFINITY;
      uint32_t rnd[4];
      philox4x32_10(0u, p.iter[slot], (uint32_t)t | (PURPOSE_ACCEPT << 8), p.seq_id[slot], a.seed_lo, a.seed_hi, rnd);
      ok = logf(u01(rnd[0])) + ld < lp;
    }
  }
  return __builtin_ctzll(~__builtin_amdgcn_ballot_w64(ok));  // lanes k .. 63 count as rejected (k < 16)
}

// the validation rows' ln-sum-exp and argmax into LDS, by a workgroup of four wavefronts (R <= 16: four rows each)
__device__ __forceinline__ void merge_rows(const Params &p, int b, int R, int parts, float *zp, int *argmax) {
  const int wave = threadIdx.x >> 6;
  float4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = load_part(p, b * R + min(wave + 4 * i, R - 1), parts);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = wave + 4 * i;
    if (r >= R) break;
    float logz;
    int idx;
    merge_parts(v[i], parts, logz, idx);
    if ((threadIdx.x & 63) == 0) { zp[r] = logz; argmax[r] = idx; }
  }
  __syncthreads();
}

// Quad q of the draw that follows the accept chain: the extra token's row `vp` (bonus), or the residual (p_t - d_t)_+
__device__ __forceinline__ uint64_t draw_quad(const SampleArgs &a, int q, float4 vp, float4 vd, const RowFilter &fp, const RowFilter &fd,
                                              float z_p, float z_d, bool bonus, float inv_t, uint32_t it, uint32_t c2, uint32_t sid) {
  const float xp[4] = {vp.x, vp.y, vp.z, vp.w}, xd[4] = {vd.x, vd.y, vd.z, vd.w};
  uint32_t rnd[4];
  philox4x32_10((uint32_t)q, it, c2, sid, a.seed_lo, a.seed_hi, rnd);
  uint64_t key = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = q * 4 + e;
    uint64_t c = 0;
    if (bonus) {
      if (kept(fp, xp[e], j)) c = best_key(xp[e] * inv_t + gumbel(u01(rnd[e])), j);
    } else {
      const float w = (kept(fp, xp[e], j) ? __expf(xp[e] * inv_t - z_p) : 0.f) - (kept(fd, xd[e], j) ? __expf(xd[e] * inv_t - z_d) : 0.f);
      if (w > 0.f) c = best_key(__logf(w) + gumbel(u01(rnd[e])), j);
    }
    key = c > key ? c : key;
  }
  return key;
}

// Part blockIdx.x of the draw that follows the accept chain of slot blockIdx.y: the residual (p_t - d_t)_+ of the first
// rejected draft, or the extra token's row when all were accepted.
template <int U>
__global__ __launch_bounds__(kPartThreads) void verify_draw_kernel(Params p, SampleArgs a, int R, int parts, int filtered) {
  __shared__ uint64_t sh_k[4];
  __shared__ float zp[kMaxK + 1];
  __shared__ int argmax[kMaxK + 1], sh_acc;
  const int b = blockIdx.y, slot = p.step_slots[b], k = p.k_act, V = p.V, base = slot * (kMaxK + 1);
  const AcceptOperands ops = accept_operands(p, slot, filtered, false);
  merge_rows(p, b, R, parts, zp, argmax);
  if (threadIdx.x < 64) {
    const int n = count_accepted(p, a, slot, ops, zp, argmax);
    if (threadIdx.x == 0) sh_acc = n;
    if (blockIdx.x == 0) {
      if (threadIdx.x == 0) p.n_acc[slot] = n;
      if ((int)threadIdx.x < R) { p.logz_p[base + threadIdx.x] = zp[threadIdx.x]; p.argmax_p[base + threadIdx.x] = argmax[threadIdx.x]; }
    }
  }
  __syncthreads();
  const int acc = sh_acc;
  const bool bonus = acc == k;
  const float inv_t = 1.f / a.temperature;
  const float *pr = p.verify_logits + ((size_t)slot * (1 + p.k) + acc) * V;
  const float *dr = bonus ? pr : p.draft_logits + ((size_t)slot * (1 + p.k) + acc + 1) * V;
  const int V4 = V >> 2, lo = blockIdx.x * (U * kPartThreads) + threadIdx.x;
  float4 vp[U], vd[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = min(lo + u * kPartThreads, V4 - 1);
    vp[u] = ((const float4 *)pr)[q];
    vd[u] = ((const float4 *)dr)[q];
  }
  const RowFilter fp = read_filter(p.flt_key_p, p.flt_tie_p, base + acc, filtered, V);
  const RowFilter fd = bonus ? fp : read_filter(p.flt_key_d, p.flt_tie_d, base + acc + 1, true, V);
  const float z_p = zp[acc], z_d = bonus ? 0.f : p.logz_d[base + acc + 1];
  const uint32_t it = p.iter[slot], sid = p.seq_id[slot], c2 = (uint32_t)(acc + 1) | ((bonus ? PURPOSE_BONUS : PURPOSE_RESIDUAL) << 8);
  uint64_t key = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = lo + u * kPartThreads;
    if (q >= V4) continue;
    const uint64_t c = draw_quad(a, q, vp[u], vd[u], fp, fd, z_p, z_d, bonus, inv_t, it, c2, sid);
    key = c > key ? c : key;
  }
  key = wave_key_dpp(key);
  if ((threadIdx.x & 63) == 0) sh_k[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < 4; ++w) key = sh_k[w] > key ? sh_k[w] : key;
    p.draw_parts[(size_t)b * kRowParts + blockIdx.x] = key;
  }
}

__global__ __launch_bounds__(kPartThreads) void verify_commit_kernel(Params p, SampleArgs a, int R, int parts, int filtered) {
  __shared__ float zp[kMaxK + 1];
  __shared__ int argmax[kMaxK + 1];
  __shared__ uint64_t sh_k[4];
  const int b = blockIdx.x, slot = p.step_slots[b], base = slot * (kMaxK + 1);
  const SlotCounts n = slot_counts(p, slot);
  const int draft = lane_draft(p, slot);
  int acc, y;
  if (a.temperature == 0.f) {
    const AcceptOperands ops = accept_operands(p, slot, filtered, true);
    merge_rows(p, b, R, parts, zp, argmax);
    if (threadIdx.x >= 64) return;
    acc = count_accepted(p, a, slot, ops, zp, argmax);
    y = argmax[acc];
    if ((int)threadIdx.x < R) { p.logz_p[base + threadIdx.x] = zp[threadIdx.x]; p.argmax_p[base + threadIdx.x] = argmax[threadIdx.x]; }
  } else {
    const uint64_t part = p.draw_parts[(size_t)b * kRowParts + min((int)(threadIdx.x & 63), parts - 1)];
    acc = p.n_acc[slot];
    y = key_index(wave_key_dpp(part));  // (the last part repeated changes nothing); the same in every wavefront
    if (y < 0 && acc < p.k_act) {
      // residual empty through rounding: draw from p_t with the same counters
      const RowFilter f = read_filter(p.flt_key_p, p.flt_tie_p, base + acc, filtered, p.V);
      const float *row = p.verify_logits + ((size_t)slot * (1 + p.k) + acc) * p.V;
      uint64_t key = 0;
      for (int q = threadIdx.x; q * 4 < p.V; q += kPartThreads) {
        uint32_t rnd[4];
        philox4x32_10((uint32_t)q, n.iter, (uint32_t)(acc + 1) | (PURPOSE_RESIDUAL << 8), p.seq_id[slot], a.seed_lo, a.seed_hi, rnd);
        for (int e = 0; e < 4; ++e) {
          const float x = row[q * 4 + e];
          if (!kept(f, x, q * 4 + e)) continue;
          const uint64_t c = best_key(x * (1.f / a.temperature) + gumbel(u01(rnd[e])), q * 4 + e);
          key = c > key ? c : key;
        }
      }
      key = wave_key_dpp(key);
      if ((threadIdx.x & 63) == 0) sh_k[threadIdx.x >> 6] = key;
      __syncthreads();
      for (int w = 0; w < 4; ++w) key = sh_k[w] > key ? sh_k[w] : key;
      y = key_index(key);
      if (threadIdx.x == 0) atomicAdd(p.fallbacks, 1);
    }
  }
  if (threadIdx.x < 64) commit_verified(p, a, slot, acc, y, draft, n);
}

// ---------------------------------------------------------------------------------------------
// And for small vocabularies without a filter: a wavefront per row, a workgroup per slot, so that the drafting epilogue
// needs no barrier and the validation epilogue no second kernel.  Both are chains of latencies (slot, logits, reductions,
// counters, one after the other), so whatever does not depend on the link before is requested ahead of it.
// Measured at 512 entries, three rows, greedy (a workgroup of 1024 threads per row, and a second kernel that decides -> here):
// drafting 6.3 us -> 3.2, validation 5.1 + 2.1 -> 3.0.
// ---------------------------------------------------------------------------------------------
constexpr int kSmallQuads = 4;  // quads of a row per lane: rows of up to 1024 entries

template <int U>
__device__ __forceinline__ void load_row(const float *row, int V4, float4 (&v)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = ((const float4 *)row)[min((int)(threadIdx.x & 63) + u * 64, V4 - 1)];
}

template <int U>
__global__ __launch_bounds__(1024) void draft_small_kernel(Params p, SampleArgs a, int R) {
  const int slot = p.step_slots[blockIdx.x], r = threadIdx.x >> 6;
  if (a.stats_only && r == 0) return;
  const bool greedy = a.temperature == 0.f;
  float4 v[U];
  load_row<U>(p.draft_logits + ((size_t)slot * (1 + p.k) + r) * p.V, p.V >> 2, v);
  const SlotCounts n = slot_counts(p, slot);
  float mx, sum;
  uint64_t key;
  score_quads<U>(v, threadIdx.x & 63, 64, p.V >> 2, RowFilter{0u, p.V}, greedy ? 1.f : 1.f / a.temperature, !greedy, a, n.iter,
                 (uint32_t)(r + a.row_base) | (PURPOSE_DRAFT << 8), p.seq_id[slot], mx, sum, key);
  const MaxSum ms = wave_ms_dpp(mx, sum);
  const int idx = key_index(wave_key_dpp(key));
  if ((threadIdx.x & 63) != 0) return;
  const int at = slot * (kMaxK + 1) + r;
  p.logz_d[at] = ms.m + logf(ms.s);
  p.flt_key_d[at] = 0u;  // the validation call evaluates d_t through the same filter
  p.flt_tie_d[at] = p.V;
  if (a.stats_only) return;  // the tokens were drafted elsewhere
  if (r > 0) p.drafts[slot * kMaxK + (r - 1)] = idx;
  else commit_first(p, a, slot, idx, n);
}

template <int U>
__global__ __launch_bounds__(1024) void verify_small_kernel(Params p, SampleArgs a, int R) {
  __shared__ float zp[kMaxK + 1];
  __shared__ int argmax[kMaxK + 1], sh_acc;
  __shared__ uint64_t sh_k[2][kMaxK + 1];
  const int slot = p.step_slots[blockIdx.x], r = threadIdx.x >> 6, lane = threadIdx.x & 63, base = slot * (kMaxK + 1);
  const int V = p.V, V4 = V >> 2, k = p.k_act;
  const bool greedy = a.temperature == 0.f;
  const float inv_t = greedy ? 1.f : 1.f / a.temperature;
  const RowFilter all{0u, V};
  float4 v[U];
  load_row<U>(p.verify_logits + ((size_t)slot * (1 + p.k) + r) * V, V4, v);
  const SlotCounts n = slot_counts(p, slot);
  const AcceptOperands ops = accept_operands(p, slot, false, greedy);
  float mx, sum;
  uint64_t key;
  score_quads<U>(v, lane, 64, V4, all, inv_t, false, a, 0, 0, 0, mx, sum, key);
  const MaxSum ms = wave_ms_dpp(mx, sum);
  const int idx = key_index(wave_key_dpp(key));
  if (lane == 0) {
    const float logz = ms.m + logf(ms.s);
    zp[r] = logz;
    argmax[r] = idx;
    p.logz_p[base + r] = logz;
    p.argmax_p[base + r] = idx;
  }
  __syncthreads();
  if (r == 0) {
    const int acc = count_accepted(p, a, slot, ops, zp, argmax);
    if (lane == 0) sh_acc = acc;
  }
  __syncthreads();
  const int acc = sh_acc;
  int y;
  if (greedy) {
    y = argmax[acc];
  } else {
    const bool bonus = acc == k;
    const float4 *pr = (const float4 *)(p.verify_logits + ((size_t)slot * (1 + p.k) + acc) * V);
    const float4 *dr = bonus ? pr : (const float4 *)(p.draft_logits + ((size_t)slot * (1 + p.k) + acc + 1) * V);
    const RowFilter fd = bonus ? all : read_filter(p.flt_key_d, p.flt_tie_d, base + acc + 1, true, V);
    const float z_d = bonus ? 0.f : p.logz_d[base + acc + 1];
    const uint32_t it = n.iter, sid = p.seq_id[slot], c2 = (uint32_t)(acc + 1) | ((bonus ? PURPOSE_BONUS : PURPOSE_RESIDUAL) << 8);
    auto draw = [&](bool whole_row, uint64_t (&sh)[kMaxK + 1]) {
      uint64_t best = 0;
      for (int q = threadIdx.x; q < V4; q += R * 64) {
        const uint64_t c = draw_quad(a, q, pr[q], dr[q], all, fd, zp[acc], z_d, whole_row, inv_t, it, c2, sid);
        best = c > best ? c : best;
      }
      best = wave_key_dpp(best);
      if (lane == 0) sh[r] = best;
      __syncthreads();
      for (int w = 0; w < R; ++w) best = sh[w] > best ? sh[w] : best;
      return key_index(best);
    };
    y = draw(bonus, sh_k[0]);
    if (y < 0) {  // the same in every thread
      // residual empty through rounding: draw from p_t with the same counters
      y = draw(true, sh_k[1]);
      if (!bonus && threadIdx.x == 0) atomicAdd(p.fallbacks, 1);
    }
  }
  if (r == 0) commit_verified(p, a, slot, acc, y, ops.x, n);
}

// Rows of a multiple of four entries, more than 4096 of them, are spread over workgroups; shorter ones stay with one (5 to 6 us,
// what the first of two kernels would take).  Returns the parts, 0 for one workgroup per row.
static int row_parts_of(const Params &p, int &u) {
  const int V4 = p.V / 4;
  u = (V4 + kPartThreads - 1) / kPartThreads <= kRowParts ? 1 : 4;
  const int parts = (V4 + u * kPartThreads - 1) / (u * kPartThreads);
  return p.V % 4 == 0 && p.V > 4096 && parts <= kRowParts ? parts : 0;
}

// Rows that a wavefront each takes: a multiple of four entries, at most 1024 (four quads a lane; beyond, a workgroup has the
// wavefronts to take a quad per thread), no filter (the selection of the K-th largest is a workgroup's).  Returns the quads per lane, 0 if not.
static int small_quads_of(const Params &p, const SampleArgs &a) {
  const bool filtered = a.temperature != 0.f && a.top_k > 0 && a.top_k < p.V;
  if (filtered || p.V % 4 != 0 || p.V > 256 * kSmallQuads) return 0;
  return p.V <= 256 ? 1 : p.V <= 512 ? 2 : kSmallQuads;
}
template <typename F>
static void with_quads(int u, F &&f) {
  if (u == 1) f(std::integral_constant<int, 1>{});
  else if (u == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, kSmallQuads>{});
}

void launch_draft_epilogue(const Params &p, const SampleArgs &a, int B, int R, hipStream_t s) {
  int u;
  if (const int quads = small_quads_of(p, a)) {
    with_quads(quads, [&](auto U) { draft_small_kernel<U.value><<<B, R * 64, 0, s>>>(p, a, R); });
    return;
  }
  const int parts = row_parts_of(p, u);
  if (!parts) {
    draft_epilogue_kernel<<<B * R, kEpiThreads, 0, s>>>(p, a, R);
    return;
  }
  const int filtered = a.temperature != 0.f && a.top_k > 0 && a.top_k < p.V;
  if (filtered) row_filter_kernel<<<B * R, kEpiThreads, 0, s>>>(p, a, R, 0);
  if (u == 1) row_part_kernel<1><<<dim3(parts, B * R), kPartThreads, 0, s>>>(p, a, R, 0, filtered);
  else row_part_kernel<4><<<dim3(parts, B * R), kPartThreads, 0, s>>>(p, a, R, 0, filtered);
  draft_commit_kernel<<<B, R * 64, 0, s>>>(p, a, R, parts, filtered);
}

void launch_verify_epilogue(const Params &p, const SampleArgs &a, int B, int R, hipStream_t s) {
  int u;
  if (const int quads = small_quads_of(p, a)) {
    with_quads(quads, [&](auto U) { verify_small_kernel<U.value><<<B, R * 64, 0, s>>>(p, a, R); });
    return;
  }
  const int parts = row_parts_of(p, u);
  if (!parts) {
    verify_stats_kernel<<<B * R, kEpiThreads, 0, s>>>(p, a, R);
    verify_decide_kernel<<<B, kEpiThreads, 0, s>>>(p, a);
    return;
  }
  const int filtered = a.temperature != 0.f && a.top_k > 0 && a.top_k < p.V;
  if (filtered) row_filter_kernel<<<B * R, kEpiThreads, 0, s>>>(p, a, R, 1);
  if (u == 1) row_part_kernel<1><<<dim3(parts, B * R), kPartThreads, 0, s>>>(p, a, R, 1, filtered);
  else row_part_kernel<4><<<dim3(parts, B * R), kPartThreads, 0, s>>>(p, a, R, 1, filtered);
  if (a.temperature != 0.f) {
    if (u == 1) verify_draw_kernel<1><<<dim3(parts, B), kPartThreads, 0, s>>>(p, a, R, parts, filtered);
    else verify_draw_kernel<4><<<dim3(parts, B), kPartThreads, 0, s>>>(p, a, R, parts, filtered);
  }
  verify_commit_kernel<<<B, kPartThreads, 0, s>>>(p, a, R, parts, filtered);
}

// The uniforms the epilogues attach to indices j0 .. j0 + n of one (sequence, iteration, row,
// purpose): the same generator and the same bits-to-float step as the draws above use.
__global__ void rng_uniforms_kernel(float *out, uint32_t j0, int n, uint32_t k0, uint32_t k1, uint32_t c1, uint32_t c2,
                                    uint32_t c3) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;  // quad of indices within the chunk; j0 % 4 == 0
  if (q * 4 >= n) return;
  uint32_t rnd[4];
  philox4x32_10(j0 / 4 + (uint32_t)q, c1, c2, c3, k0, k1, rnd);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (q * 4 + e < n) out[q * 4 + e] = u01(rnd[e]);
}

void launch_rng_uniforms(float *out, uint32_t j0, int n, uint64_t seed, uint32_t seq_id, uint32_t iteration,
                         uint32_t row, uint32_t purpose, hipStream_t s) {
  const int quads = (n + 3) / 4;
  rng_uniforms_kernel<<<(quads + 255) / 256, 256, 0, s>>>(out, j0, n, (uint32_t)seed, (uint32_t)(seed >> 32), iteration,
                                                         row | (purpose << 8), seq_id);
}

}  // namespace pass
