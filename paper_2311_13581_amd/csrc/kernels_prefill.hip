// Prompt pass ("initial prompt sequence" of Algorithm 1) as a compute-bound problem.
//
// The decode kernels stream every weight once per call of at most 64 rows; a prompt of thousands
// of tokens pushed through them re-reads the model dozens of times and leaves the matrix cores
// idle.  Here up to 2048 prompt rows go through each layer in one pass:
//
//   gemm_tile_kernel   a workgroup of eight wavefronts computes 256 x 128 (or 192 x 128) output features x
//                      rows; both operands stream from memory straight into a ring of LDS stages.  Accumulators
//                      stay in the register file for the whole K loop, one fixed summation order.  Same operand
//                      formats and the same fused epilogues as the decode GEMM (RMSNorm scale, rotary embedding and
//                      K/V page writes, SiLU * up, residual add with (hi, lo) of the next norm's input).  Where the
//                      tiles would leave compute units idle, K is cut into slices whose sums tile_reduce_kernel adds.
//   attn_prefill_kernel causal attention of a block of 32 (or 16) query rows of one head over the
//                      paged cache, without a split of the keys across workgroups: the four
//                      wavefronts take alternate 32-key steps and merge once at the end.  K and V
//                      tiles are used for all row groups of the block.
//   attn_prefill_shared_kernel  the same for passes of more than 512 rows: 128 rows per workgroup,
//                      the K and V tiles of a step fetched once into LDS for all four wavefronts.
#include "lds_copy.h"
#include "pass_internal.h"

namespace pass {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// value of the lane 8 columns further in the same row of 16 (row_ror 8): lo half <-> hi half
__device__ __forceinline__ float other_half(float v) { return dpp_mov<0x128>(v); }

// sum over the sixteen lanes of a row, in each of them
__device__ __forceinline__ float row_total(float v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  return v + dpp_mov<0x140>(v);  // row_mirror
}

template <int I> struct ic { static constexpr int value = I; };

enum { TILE_QKV = 0, TILE_RESID = 1, TILE_GATEUP = 2, TILE_PART = 3 };

struct TileArgs {
  const u32x4 *W;             // packed weight tiles [strip][K/32][64 lanes]
  const u32x4 *X;             // activation rows as (hi, lo) tiles [ceil(M/8)][K/32][64 lanes][8]
  int M, K, n_strips;
  int layer;
  const uint16_t *gain_next;  // RESID: gain of the norm that follows
  PrefillSegs segs;           // QKV: whose rows these are (K/V go to that sequence's pages)
  int tiles_m, tiles_n;
  int panel;                  // row tiles of a panel: tiles are walked panel by panel, features outside, rows inside
  int slices, kt_slice;       // PART: slices of K and k-steps of each
  float *part;                // PART: [slice][M][16 * n_strips] sums over a slice of K
};

// What becomes of four consecutive output features n .. n + 3 (n % 4 == 0) of row m, `inv` = 1 / rms of the row.
__device__ __forceinline__ void finish_qkv(const Params &p, const PrefillWs &w, const TileArgs &a, int m, int n, floatx4 v) {
  const int which = n / p.D;        // 0 q, 1 k, 2 v
  const int c = n - which * p.D;    // column inside the projection
  const int head = c / p.hd, dim = c - head * p.hd;
  if (which < 2) {
    const int half = p.hd / 2;
    const float *cs = p.rope_cos + (size_t)m * half + dim / 2;
    const float *sn = p.rope_sin + (size_t)m * half + dim / 2;
    const float x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3];
    v[0] = x0 * cs[0] - x1 * sn[0];
    v[1] = x0 * sn[0] + x1 * cs[0];
    v[2] = x2 * cs[1] - x3 * sn[1];
    v[3] = x2 * sn[1] + x3 * cs[1];
  }
  if (which == 0) {
    *(floatx4 *)(w.q + (size_t)m * p.D + c) = v;
    return;
  }
  // pages tiled (k_tile, v_tile); bf16 storage
  // (the rows of a 16-row group share a block: the index is uniform over the wavefront)
  const int sb = __builtin_amdgcn_readfirstlane(m / kPrefillBlockRows), sr = m % kPrefillBlockRows;
  if (sr >= a.segs.rows[sb]) return;  // a padding row: nothing to cache
  const int pos = a.segs.pos[sb] + sr;
  const int page = p.block_table[(size_t)a.segs.slot[sb] * p.pages_per_seq + (pos >> p.page_shift)];
  const size_t hbase = ((size_t)a.layer * p.n_pages + page) * p.H + head;
  const int off = pos & (p.page_size - 1);
  if (which == 1) {
    uint2 pk;
    pk.x = pack2_bf16(v[0], v[1]);
    pk.y = pack2_bf16(v[2], v[3]);
    *(uint2 *)((uint16_t *)p.k_pool + hbase * p.page_size * p.hd + k_tile(p, off, dim)) = pk;
  } else {
    uint16_t *vp = (uint16_t *)p.v_pool + hbase * p.page_size * p.hd + v_tile(p, off, dim);
#pragma unroll
    for (int r = 0; r < 4; ++r) vp[8 * r] = f32_to_bf16(v[r]);
  }
}
// residual add, (hi, lo) of h * gain of the next norm; returns the four features' share of sum h^2
__device__ __forceinline__ float finish_resid(const Params &p, const uint16_t *gain_next, int m, int n, floatx4 y) {
  float *hp = p.h + (size_t)m * p.d + n;
  const floatx4 hv = *(floatx4 *)hp + y;
  *(floatx4 *)hp = hv;
  float tv[4], ss = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    tv[r] = hv[r] * bf16_to_f32(gain_next[n + r]);
    ss += hv[r] * hv[r];
  }
  store_split4(p.xg, m, p.d, n, tv);
  return ss;
}
// silu(gate) * up of FFN features f .. f + 3
__device__ __forceinline__ void finish_gateup(const Params &p, int m, int f, floatx4 yg, floatx4 yu, float inv) {
  float tv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float gt = yg[r] * inv, up = yu[r] * inv;
    tv[r] = gt / (1.0f + __expf(-gt)) * up;
  }
  store_split4(p.act_x, m, p.F, f, tv);
}

// The tiled GEMM.  Y[rows][features] += W . X over k-steps of 32; a workgroup of eight wavefronts owns 16 * WF * SW
// features x 16 * WR * RG rows, a wavefront SW strips of 16 features x RG groups of 16 rows.
// Both operands of a k-step go straight from memory to LDS, into a ring of three stages, two steps ahead of their
// use.  The (hi, lo) halves of an activation row are two B operands (a weight fragment is read once for both), so a
// k-step is 2 * SW * RG MFMAs per wavefront.  The two halves' sums have accumulators of their own: in a common one the
// sum is rounded twice as often (2047 rows, error of the sums alone relative to the result: K = 4096 5.7e-7 against 4.0e-7,
// K = 11008 9.5e-7 against 6.7e-7, the whole product 2.63e-6 against 2.54e-6).  That holds the tile to 128 rows: the larger
// ones (256 x 256, 384 x 128) took 2 to 6 % less time of a prompt pass, with one accumulator.
// The wavefronts form two groups, one wavefront of each group per SIMD, that alternate: while one group reads the
// fragments of its next k-step out of LDS and requests a later stage, the other keeps the matrix cores busy; the
// workgroup meets after every half step.  Timeline of half steps: group 0 reads step t in 2t and multiplies in
// 2t + 1, group 1 reads it in 2t + 1 and multiplies in 2t + 2.  A stage is overwritten by requests issued two half
// steps after group 0's reads (one after group 1's) have returned; its copies have landed, in every wavefront, at
// the meeting before group 0 reads it (each group waits for its own at the end of half step 2t - 1).
// STEP: calls that carry few rows (PrefillWs::few), which would otherwise go through the decode kernels, are as exact as
// there.  The products of a k-step are added to a sum over three steps, and that to the whole sum (a matrix instruction
// rounds its accumulator four times, an addition once).  100 rows, error of the sums: K = 4096 1.1e-7, K = 11008 1.6e-7
// (decode kernels 0.95e-7 to 1.36e-7 and 1.2e-7; two accumulators 1.5e-7 and 2.2e-7).  Logits on top of a prompt of 100 tokens, two
// 7B layers, distance from 64 bits, mean of 60 seeds: 1.12e-4 (decode kernels 1.28e-4, two accumulators 1.36e-4).  6 % more time.
// Bound by power.  Against a form that kept weight fragments in registers and staged the activations through registers
// (4 wavefronts, 256 x 64 tiles): QKV 363 -> 291 us, Wo 124 -> 113, gate/up 633 -> 552, down 326 -> 263 (7B shapes, 2047 rows).
template <int EPI, int WF, int WR, int SW, int RG, bool STEP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_tile_kernel(Params p, PrefillWs w, TileArgs a) {
  constexpr int TS = WF * SW, TG = WR * RG;         // strips and 16-row groups of the tile
  constexpr int NC = (TS + 2 * TG + 7) / 8;         // 1 KB copies of a wavefront per step
  constexpr int ROWS = TG * 16;
  constexpr bool NORM = (EPI == TILE_QKV || EPI == TILE_GATEUP);
  static_assert(WF * WR == 8, "eight wavefronts");
  static_assert(EPI != TILE_GATEUP || SW % 2 == 0, "a wavefront needs a gate strip and its up strip");
  __shared__ u32x4 s0[TS + 2 * TG][64], s1[TS + 2 * TG][64], s2[TS + 2 * TG][64];  // weight tiles, then activation fragments
  __shared__ float s_inv[ROWS], s_part[512];

  // tile of this workgroup: consecutive workgroup ids go to different dies (XCDs), each with its own L2; every die
  // gets a contiguous eighth of the tiles in panel order, so its workgroups share weight and activation tiles
  const int n_tiles = a.tiles_m * a.tiles_n * a.slices;
  const int die = blockIdx.x & 7, rem = n_tiles & 7;
  int t = die * (n_tiles >> 3) + min(die, rem) + (int)(blockIdx.x >> 3);
  const int slice = t / (a.tiles_m * a.tiles_n);
  t -= slice * a.tiles_m * a.tiles_n;
  const int pnl = t / (a.panel * a.tiles_n);
  t -= pnl * a.panel * a.tiles_n;
  const int gm = min(a.panel, a.tiles_m - pnl * a.panel);
  const int tn = t / gm, tm = pnl * a.panel + t % gm;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wf = wave % WF, wr = wave / WF;
  const int c = lane & 15, kq = lane >> 4;
  const int KT = a.K >> 5, n_groups = (a.M + 7) >> 3;
  const int kt0 = slice * a.kt_slice, kt1 = min(KT, kt0 + a.kt_slice);
  const int m0 = tm * ROWS;

  // sources of this wavefront's copies: tiles wave * NC .. of the stage (past its end: the last one again).  Strips past
  // the end repeat the last one, row groups past the end the last one (in bounds; their results are dropped).  Fragment
  // (16-row group, half): lane (c, kq) takes the slot of row c & 7 of 8-row group c >> 3.
  const u32x4 *src[NC];
  int dst[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    dst[i] = min(wave * NC + i, TS + 2 * TG - 1);
    if (dst[i] < TS) {
      src[i] = a.W + ((size_t)min(tn * TS + dst[i], a.n_strips - 1) * KT) * 64 + lane;
    } else {
      const int f = dst[i] - TS, rg = f >> 1, half = f & 1;
      const int g8 = min(tm * TG * 2 + 2 * rg + (c >> 3), n_groups - 1);
      src[i] = a.X + (size_t)g8 * KT * 64 + kq * 16 + half * 8 + (c & 7);
    }
  }
  auto issue = [&](u32x4 (*st)[64], int kt) __attribute__((always_inline)) {
    const size_t off = (size_t)min(kt, kt1 - 1) * 64;  // steps past the end repeat the last one (never read)
#pragma unroll
    for (int i = 0; i < NC; ++i) copy_to_lds(src[i] + off, &st[dst[i]][0]);
  };
  issue(s0, kt0);
  issue(s1, kt0 + 1);

  // 1 / rms of the tile's rows from the producer's partial sums of h^2
  if constexpr (NORM) {
    constexpr int TH = 512 / ROWS;
    const int row = tid % ROWS, th = tid / ROWS;
    float ss = 0.f;
    if (m0 + row < a.M) {
      // eight requests at a time (indices past the end repeat the last partial and are dropped)
      for (int i0 = th; i0 < w.np; i0 += 8 * TH) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p.ssq[(size_t)min(i0 + u * TH, w.np - 1) * w.rows + m0 + row];
#pragma unroll
        for (int u = 0; u < 8; ++u) ss += (i0 + u * TH < w.np) ? v[u] : 0.f;
      }
    }
    s_part[tid] = ss;
    __syncthreads();
    if (tid < ROWS) {
      float tot = 0.f;
#pragma unroll
      for (int j = 0; j < TH; ++j) tot += s_part[j * ROWS + tid];
      s_inv[tid] = 1.0f / sqrtf(tot / (float)p.d + p.eps);
    }
    // published by the meetings of the main loop
  }

  floatx4 acc[STEP ? 1 : 2][STEP ? 1 : SW][STEP ? 1 : RG];
  float sum[STEP ? SW : 1][STEP ? RG : 1][4], three[STEP ? SW : 1][STEP ? RG : 1][4];
#pragma unroll
  for (int s = 0; s < SW; ++s)
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      if constexpr (STEP)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[s][g][r] = 0.f;
      else acc[0][s][g] = acc[1][s][g] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

  auto step = [&](const u32x4 (*st)[64], u32x4 (*nxt)[64], int kt, auto first) __attribute__((always_inline)) {
    bf16x8 av[SW], bv[RG][2];
#pragma unroll
    for (int s = 0; s < SW; ++s) av[s] = __builtin_bit_cast(bf16x8, st[wf * SW + s][lane]);
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h) bv[g][h] = __builtin_bit_cast(bf16x8, st[TS + (wr * RG + g) * 2 + h][lane]);
    issue(nxt, kt + 2);
    wait_lds_reads();
    if (grp) wait_copies<NC>();
    meet();
    __builtin_amdgcn_s_setprio(1);
    if constexpr (!STEP) {
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int s = 0; s < SW; ++s) acc[h][s][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[s], bv[g][h], acc[h][s][g], 0, 0, 0);
    } else {
      // two strips of a row group at a time, the additions two turns later, one product beside two of them
      constexpr int TURNS = RG * SW / 2;
      floatx4 y[3][2];
#pragma unroll
      for (int b = 0; b < TURNS + 2; ++b)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (b < TURNS) {
            const int g = b / (SW / 2), s = b % (SW / 2) * 2 + (u & 1);
            y[b % 3][u & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[s], bv[g][u < 2], u < 2 ? floatx4{0.f, 0.f, 0.f, 0.f} : y[b % 3][u & 1], 0, 0, 0);
          }
          if (b >= 2) {
            const int g = (b - 2) / (SW / 2), s = (b - 2) % (SW / 2) * 2 + (u >> 1);
#pragma unroll
            for (int r = 2 * (u & 1); r < 2 * (u & 1) + 2; ++r) {
              three[s][g][r] = first.value ? y[(b - 2) % 3][u >> 1][r] : three[s][g][r] + y[(b - 2) % 3][u >> 1][r];
              asm volatile("" : "+v"(three[s][g][r]));  // added here: the compiler would keep the products of several steps
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (!grp) wait_copies<NC>();
    meet();
  };
  wait_copies<NC>();
  wait_lds_reads();
  meet();
  if (grp) meet();
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (STEP)
#pragma unroll
      for (int s = 0; s < SW; ++s)
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[s][g][r] += three[s][g][r];
  };
  int kt = kt0;
  for (; kt + 2 < kt1; kt += 3) {
    step(s0, s2, kt, ic<1>{});
    step(s1, s0, kt + 1, ic<0>{});
    step(s2, s1, kt + 2, ic<0>{});
    fold();
  }
  if (kt < kt1) {
    step(s0, s2, kt, ic<1>{});
    if (kt + 1 < kt1) step(s1, s0, kt + 1, ic<0>{});
    fold();
  }
  if (!grp) meet();
  wait_copies<0>();  // no copy may land in LDS that the next workgroup already owns

  auto total = [&](int s, int g) __attribute__((always_inline)) {
    if constexpr (STEP) return floatx4{sum[s][g][0], sum[s][g][1], sum[s][g][2], sum[s][g][3]};
    else return acc[0][s][g] + acc[1][s][g];
  };
  // lane (c, kq) holds Y[row 16 g + c][features 16 strip + 4 kq .. + 3]
  const int strip0 = tn * TS + wf * SW;
#pragma unroll
  for (int g = 0; g < RG; ++g) {
    const int lr = (wr * RG + g) * 16 + c, m = m0 + lr;
    const bool row_live = m < a.M;
    float inv = 1.f;
    if constexpr (NORM) inv = s_inv[lr];
    float ss = 0.f;
    if constexpr (EPI == TILE_GATEUP) {
#pragma unroll
      for (int s = 0; s < SW; s += 2)
        if (row_live && strip0 + s + 1 < a.n_strips)
          finish_gateup(p, m, ((strip0 + s) >> 1) * 16 + 4 * kq, total(s, g), total(s + 1, g), inv);
    } else {
#pragma unroll
      for (int s = 0; s < SW; ++s) {
        const int n = (strip0 + s) * 16 + 4 * kq;
        if (row_live && strip0 + s < a.n_strips) {
          if constexpr (EPI == TILE_RESID)
            ss += finish_resid(p, a.gain_next, m, n, total(s, g));
          else if constexpr (EPI == TILE_QKV)
            finish_qkv(p, w, a, m, n, total(s, g) * inv);
          else
            *(floatx4 *)(a.part + ((size_t)slice * a.M + m) * (a.n_strips * 16) + n) = total(s, g);
        }
      }
    }
    if constexpr (EPI == TILE_RESID) {
      // partial sum of h^2 over this wavefront's 16 * SW features, one per row
      const int part = tn * WF + wf;
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (lane < 16 && row_live && strip0 < a.n_strips) p.ssq[(size_t)part * w.rows + m] = ss;
    }
  }
}

// Adds the SL slices of a product that was split along K (in slice order) and finishes it as the fused epilogues do.
// One workgroup: 16 rows x 64 features (a gate strip, its up strip, twice); thread = (row, four features), sixteen
// neighbouring threads of a row, so that a slice is read in runs of 256 bytes (sixteen rows side by side, 16 bytes of
// each, kept the address unit busy four times as long).  What belongs to a row is summed across its sixteen lanes.
// Bound by the slices' bytes and, for the small ones, by the launch and two trips to memory.  Measured (7B, before ->
// now): 100 rows gate/up, two slices, 12.5 -> 7.4 us, QKV, four, 9.2 -> 7.4; 511 rows Wo and down, four, 14.0 -> 11.0; 836 rows, two, 20.6 -> 13.8.
template <int EPI, int SL>
__global__ __launch_bounds__(256) void tile_reduce_kernel(Params p, PrefillWs w, TileArgs a) {
  const int qd = threadIdx.x & 15, m = blockIdx.y * 16 + (threadIdx.x >> 4), n = blockIdx.x * 64 + qd * 4, N = a.n_strips * 16;
  const bool live = m < a.M && n < N;
  const int mc = min(m, a.M - 1);
  const size_t stride = (size_t)a.M * N, at = (size_t)mc * N + min(n, N - 4);
  floatx4 v[SL];
#pragma unroll
  for (int i = 0; i < SL; ++i) v[i] = *(const floatx4 *)(a.part + i * stride + at);
  float inv = 1.f;
  if constexpr (EPI != TILE_RESID) {
    // the partial sums lie row beside row: thread (group, row) here
    __shared__ float s_part[16][17];
    const int r = min((int)blockIdx.y * 16 + qd, a.M - 1);
    float ss = 0.f;
    for (int i0 = threadIdx.x >> 4; i0 < w.np; i0 += 64) {  // four requests at a time (indices past the end repeat the last partial, dropped)
      float t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = p.ssq[(size_t)min(i0 + 16 * u, w.np - 1) * w.rows + r];
#pragma unroll
      for (int u = 0; u < 4; ++u) ss += i0 + 16 * u < w.np ? t[u] : 0.f;
    }
    s_part[threadIdx.x >> 4][qd] = ss;
    __syncthreads();
    inv = 1.0f / sqrtf(row_total(s_part[qd][threadIdx.x >> 4]) / (float)p.d + p.eps);
  }
  floatx4 y = v[0];
#pragma unroll
  for (int i = 1; i < SL; ++i) y += v[i];
  if constexpr (EPI == TILE_QKV) {
    if (live) finish_qkv(p, w, a, m, n, y * inv);
  } else if constexpr (EPI == TILE_GATEUP) {
    // quads 0..3 gate, 4..7 up of one strip pair, 8..11 gate, 12..15 up of the next: the up quad is four lanes on
    floatx4 up;
#pragma unroll
    for (int r = 0; r < 4; ++r) up[r] = dpp_mov<0x104>(y[r]);  // row_shl 4
    if (!(qd & 4) && live) finish_gateup(p, m, (n >> 5) * 16 + (n & 15), y, up, inv);
  } else {
    const float ss = row_total(live ? finish_resid(p, a.gain_next, m, n, y) : 0.f);
    if (qd == 0 && m < a.M) p.ssq[(size_t)blockIdx.x * w.rows + m] = ss;
  }
}

// Shapes of the tiled GEMM: 256 x 128 and 192 x 128 features x rows, and what a k-step takes when every compute unit has one.
struct TileShape { int ts, strips_per_wave; float step_us; };
constexpr int kTileRows = 128;
constexpr TileShape kTileShapes[2] = {{16, 4, 0.74f}, {12, 6, 0.57f}};
struct TilePlan { int shape, slices; };

// Which tile and how many slices of K.  The tiles run in rounds of one per compute unit (256), a round takes the
// steps of a tile; what a shape leaves idle in its last round decides, as long as the weights do not have to be
// waited for.  Slices fill the chip when there are fewer tiles than units; their sums cost a write, a read and a
// launch.  `want` > 0 asks for a tile, whole or in slices, whatever it costs (the workspace still has to hold the sums).
TilePlan plan_tiles(int n_strips, int K, int M, size_t part_floats, int want) {
  const int KT = K / 32;
  const int most = want == 2 || want == 5 ? 1 : want == 4 ? 2 : 8;
  TilePlan best{want == 3 || want == 5, 1};
  float best_us = 1e30f;
  for (int s = 0; s < 2; ++s) {
    const TileShape &t = kTileShapes[s];
    if (want && s != (want == 3 || want == 5)) continue;
    const int tiles = ((n_strips + t.ts - 1) / t.ts) * ((M + kTileRows - 1) / kTileRows);
    for (int ks = 1; ks <= most; ++ks) {
      const int kts = (KT + ks - 1) / ks;
      if ((KT + kts - 1) / kts != ks) continue;  // every slice has steps
      if (ks > 1 && (size_t)ks * M * n_strips * 16 > part_floats) continue;
      if (want) { best.slices = ks; continue; }  // as many as asked for, or as there are
      if (kts < 8 && ks > 1) continue;
      const float rounds = (float)((tiles * ks + 255) / 256);
      float us = rounds * (kts * t.step_us + 4.f);
      const float stream = (float)n_strips * K * 32 / 5.0e6f;  // the weights at 5 TB/s
      if (us < stream) us = stream;
      if (ks > 1) us += 4.f + (float)ks * M * n_strips * 16 * 8 / 4.0e6f;
      if (us < best_us) { best_us = us; best = TilePlan{s, ks}; }
    }
  }
  return best;
}

// Launches a product with its epilogue; returns the number of partial sums of h^2 per row that RESID leaves.
template <int EPI>
int launch_tile(const Params &p, const PrefillWs &w, TileArgs a, hipStream_t s) {
  const TilePlan pl = plan_tiles(a.n_strips, a.K, a.M, w.part_floats, w.strips_opt);
  const TileShape &t = kTileShapes[pl.shape];
  a.tiles_n = (a.n_strips + t.ts - 1) / t.ts;
  a.tiles_m = (a.M + kTileRows - 1) / kTileRows;
  // a die works on 32 tiles at a time: about 1024 rows x 1024 features re-read the least per multiply-add
  a.panel = w.panel ? w.panel : 1024 / kTileRows;
  const int KT = a.K / 32;
  a.kt_slice = (KT + pl.slices - 1) / pl.slices;
  a.slices = (KT + a.kt_slice - 1) / a.kt_slice;
  a.part = w.part;
  const int grid = a.tiles_n * a.tiles_m * a.slices;
  auto go = [&](auto E) {
    constexpr int e = decltype(E)::value;
    const bool step = w.few;
    if (pl.shape == 1 && step) gemm_tile_kernel<e, 2, 4, 6, 2, true><<<grid, 512, 0, s>>>(p, w, a);
    else if (pl.shape == 1) gemm_tile_kernel<e, 2, 4, 6, 2, false><<<grid, 512, 0, s>>>(p, w, a);
    else if (step) gemm_tile_kernel<e, 4, 2, 4, 4, true><<<grid, 512, 0, s>>>(p, w, a);
    else gemm_tile_kernel<e, 4, 2, 4, 4, false><<<grid, 512, 0, s>>>(p, w, a);
  };
  if (a.slices == 1) {
    go(ic<EPI>{});
    return (a.n_strips + t.strips_per_wave - 1) / t.strips_per_wave;
  }
  go(ic<TILE_PART>{});
  auto add = [&](auto SL) { tile_reduce_kernel<EPI, decltype(SL)::value><<<dim3((a.n_strips + 3) / 4, (a.M + 15) / 16), 256, 0, s>>>(p, w, a); };
  switch (a.slices) {
    case 2: add(ic<2>{}); break;
    case 3: add(ic<3>{}); break;
    case 4: add(ic<4>{}); break;
    case 5: add(ic<5>{}); break;
    case 6: add(ic<6>{}); break;
    case 7: add(ic<7>{}); break;
    default: add(ic<8>{}); break;
  }
  return (a.n_strips + 3) / 4;
}

// ---------------------------------------------------------------------------------------------
// Causal attention of RG * 16 consecutive prompt rows of one head (bf16 cache, head_dim 128, pages
// tiled).  Scores S^T[key][row] = K[key][:] . Q[row][:] with K rows as the MFMA A operand (key
// order inside the two 16-key tiles chosen so that a lane ends up with 8 consecutive keys) and 16
// query rows as the columns of the B operand; the probabilities of 8 consecutive keys feed
// O^T[dim][row] += V^T[dim][key] P[key][row] with one 16-byte load of the tiled V page as A
// operand.  Queries and probabilities keep fp32-like precision as (hi, lo) bf16 pairs; unlike the
// decode kernel, which puts the two halves of 8 rows side by side in the 16 columns, the halves go
// into separate MFMAs here: S = K q_hi + K q_lo accumulate into one score tile, the softmax runs
// once per (row, key) (side by side it runs in the hi and in the lo column, and that vector
// arithmetic, not the matrix cores, bounds the kernel), and P_hi, P_lo are two B operands that
// accumulate into one output tile.  A wavefront walks 32-key steps base = 32 * wave, + 128, ...
// with online softmax; wavefronts 1..3 leave (max, sum, accumulator) in LDS and wavefront 0 merges
// the four in wavefront order, normalises and stores the rows as (hi, lo) pairs for the Wo GEMM.
// ---------------------------------------------------------------------------------------------
template <int RG>  // groups of 16 rows per workgroup
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_prefill_kernel(Params p, PrefillWs w, int layer, PrefillAttn a) {
  constexpr int HD = 128, RQ = 16 * RG;
  __shared__ float s_m[3][RQ], s_l[3][RQ];
  __shared__ __align__(16) float s_acc[3][RQ][HD];

  constexpr int SUB = kPrefillBlockRows / RQ;
  const int blk = blockIdx.x / SUB, first = (SUB - 1 - blockIdx.x % SUB) * RQ;  // rows with the most keys first
  const int head = blockIdx.y;
  const int nr = min(RQ, a.rows[blk] - first);
  if (nr <= 0) return;  // uniform over the workgroup
  const int slot = a.slot[blk], r0 = a.row[blk] + first;  // r0: row of the pass, at position `at` of the sequence
  const int at = a.pos[blk] + first;
  const int k_hi = at + nr;  // keys 0 .. k_hi - 1 are visible to the block's last row

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ml = lane & 15, g = lane >> 4;
  const uint16_t *kpool = (const uint16_t *)p.k_pool, *vpool = (const uint16_t *)p.v_pool;

  // query fragments: column ml = row rg * 16 + ml, scaled by 1/sqrt(hd), as separate hi and lo operands
  u32x4 qh[RG][4], ql[RG][4];
  {
    const float scale = rsqrtf((float)HD);
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const int rr = rg * 16 + ml;
      const bool live = rr < nr;
      const float *qp = w.q + (size_t)(r0 + (live ? rr : 0)) * p.D + head * HD + g * 8;
      floatx4 raw[4][2];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        raw[j][0] = *(const floatx4 *)(qp + j * 32);
        raw[j][1] = *(const floatx4 *)(qp + j * 32 + 4);
      }
      const float sc_q = live ? scale : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          qh[rg][j][2 * h] = split2_bf16(raw[j][h][0] * sc_q, raw[j][h][1] * sc_q, true);
          qh[rg][j][2 * h + 1] = split2_bf16(raw[j][h][2] * sc_q, raw[j][h][3] * sc_q, true);
          ql[rg][j][2 * h] = split2_bf16(raw[j][h][0] * sc_q, raw[j][h][1] * sc_q, false);
          ql[rg][j][2 * h + 1] = split2_bf16(raw[j][h][2] * sc_q, raw[j][h][3] * sc_q, false);
        }
    }
  }

  floatx4 o[RG][8];
  float m_run[RG], l_run[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    m_run[rg] = -INFINITY;
    l_run[rg] = 0.f;
#pragma unroll
    for (int db = 0; db < 8; ++db) o[rg][db] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  for (int base = wave * 32; base < k_hi; base += 128) {
    // one page holds the 32 keys (page_size is a multiple of 32); the lookup is wavefront-uniform
    const int page = p.block_table[(size_t)slot * p.pages_per_seq + (base >> p.page_shift)];
    const int poff = base & (p.page_size - 1);
    const size_t hbase = ((size_t)layer * p.n_pages + page) * p.H + head;
    const uint16_t *kp = kpool + (hbase * HD * p.page_size + poff * 8);    // K[dim / 8][key][8]
    const uint16_t *vp = vpool + (hbase * p.page_size + poff) * HD;        // V[key / 8][dim][8]
    u32x4 kt[2][4], vt[8];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int key = (ml >> 2) * 8 + t * 4 + (ml & 3);  // key slot ml of tile t
#pragma unroll
      for (int j = 0; j < 4; ++j) kt[t][j] = *(const u32x4 *)(kp + ((j * 4 + g) * p.page_size + key) * 8);
    }
#pragma unroll
    for (int db = 0; db < 8; ++db) vt[db] = *(const u32x4 *)(vp + (g * HD + db * 16 + ml) * 8);
    __builtin_amdgcn_sched_barrier(0);  // all sixteen requests leave before anything is computed

#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      // a row group whose last row comes before this step's first key sees none of the step
      if (base > at + rg * 16 + 15) continue;
      floatx4 sc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kt[t][j]),
                                                          __builtin_bit_cast(bf16x8, qh[rg][j]), sc[t], 0, 0, 0);
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kt[t][j]),
                                                          __builtin_bit_cast(bf16x8, ql[rg][j]), sc[t], 0, 0, 0);
        }
      }
      // lane (column ml, g) holds the scores of row rg * 16 + ml for keys base + 8g + 4t + r
      const int rr = rg * 16 + ml;
      float sv[8];
      float m_blk = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = base + 8 * g + 4 * t + r;
          const bool ok = (rr < nr) && (key <= at + rr);
          const float v = ok ? sc[t][r] : -INFINITY;
          sv[4 * t + r] = v;
          m_blk = fmaxf(m_blk, v);
        }
      m_blk = fmaxf(m_blk, __shfl_xor(m_blk, 16));
      m_blk = fmaxf(m_blk, __shfl_xor(m_blk, 32));
      const float m_new = fmaxf(m_run[rg], m_blk);
      const float alpha = (m_run[rg] == -INFINITY) ? 0.f : __expf(m_run[rg] - m_new);
      float pv[8], psum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pv[i] = (sv[i] == -INFINITY) ? 0.f : __expf(sv[i] - m_new);
        psum += pv[i];
      }
      l_run[rg] = l_run[rg] * alpha + psum;
      m_run[rg] = m_new;
      u32x4 ph, pl;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ph[i] = pack2_bf16(pv[2 * i], pv[2 * i + 1]);
        pl[i] = pack2_bf16(pv[2 * i] - __uint_as_float(ph[i] << 16), pv[2 * i + 1] - __uint_as_float(ph[i] & 0xffff0000u));
      }
      // once the running maxima have settled alpha is 1 in every lane: skip the rescaling then
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
        for (int db = 0; db < 8; ++db) o[rg][db] *= alpha;
      }
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        o[rg][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt[db]),
                                                            __builtin_bit_cast(bf16x8, ph), o[rg][db], 0, 0, 0);
        o[rg][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt[db]),
                                                            __builtin_bit_cast(bf16x8, pl), o[rg][db], 0, 0, 0);
      }
    }
  }

  // a row's sum of probabilities is spread over the four g groups; lane (ml, g) holds dims
  // db * 16 + 4g + r of row rg * 16 + ml
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    l_run[rg] += __shfl_xor(l_run[rg], 16);
    l_run[rg] += __shfl_xor(l_run[rg], 32);
  }
  if (wave > 0) {
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const int rr = rg * 16 + ml;
      if (g == 0) { s_m[wave - 1][rr] = m_run[rg]; s_l[wave - 1][rr] = l_run[rg]; }
#pragma unroll
      for (int db = 0; db < 8; ++db) *(floatx4 *)&s_acc[wave - 1][rr][db * 16 + 4 * g] = o[rg][db];
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const int rr = rg * 16 + ml;
      if (rr >= nr) continue;
      float m_n = m_run[rg];
#pragma unroll
      for (int j = 0; j < 3; ++j) m_n = fmaxf(m_n, s_m[j][rr]);
      // row rr always sees key 0, so m_n is finite
      float f0 = (m_run[rg] == -INFINITY) ? 0.f : __expf(m_run[rg] - m_n);
      float l_n = l_run[rg] * f0;
      floatx4 acc[8];
#pragma unroll
      for (int db = 0; db < 8; ++db) acc[db] = o[rg][db] * f0;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const float mj = s_m[j][rr];
        const float f = (mj == -INFINITY) ? 0.f : __expf(mj - m_n);
        l_n += s_l[j][rr] * f;
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[db] += *(const floatx4 *)&s_acc[j][rr][db * 16 + 4 * g] * f;
      }
      const float inv_l = 1.0f / l_n;
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        const float tv[4] = {acc[db][0] * inv_l, acc[db][1] * inv_l, acc[db][2] * inv_l, acc[db][3] * inv_l};
        store_split4(p.attn_x, r0 + rr, p.D, head * HD + db * 16 + 4 * g, tv);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Long prompts: the same attention with the K/V tiles shared by the workgroup.  In the kernel above
// every block of 32 rows pulls all earlier keys through its compute unit's L1 on its own, and at
// thousands of rows that traffic out of L2 bounds it.  Here a workgroup owns 128 rows, 32 per
// wavefront; all four wavefronts walk the same 32-key steps, whose K and V tiles (16 KB) the four copy
// straight into LDS in fragment order, one step ahead, so that every wavefront reads a fragment as 1 KB
// of consecutive 16-byte words.  A wavefront skips the steps past its own last row but keeps copying
// and meeting the barriers.  No merge at the end: every wavefront owns its rows.
//
// The softmax's vector arithmetic costs as much as the MFMAs, so it is kept short: scores come out in
// base-2 logarithms (log2 e is folded into the queries), only steps that reach past the wavefront's
// first row are masked, and the reference the exponentials are taken against is not the running
// maximum: it is moved (an exchange between lanes, a rescaling of the accumulators) only when a score
// exceeds it by more than 8, which for most rows is the first step only.  Probabilities up to 2^8
// keep the relative precision of their (hi, lo) halves, and the quotient at the end does not care.
//
// Blocks differ in their number of keys: the first half of the grid takes the longer ones, longest first,
// the second half the shorter ones, shortest first, so that where all workgroups are resident at once
// (two per compute unit) the shortest shares a unit with the longest (97 us; longest first throughout 108,
// other interleavings 105 to 112).
// Measured per 7B layer (2047 rows): 155 -> 95 us against running maxima, masks everywhere and tiles
// through registers; 13B, rows 2048 .. 4095: 465 -> 305.  Also tried: 64-key steps (the same), 16 rows per
// wavefront with three or four wavefronts per SIMD (5 % slower at 2047 rows, 20 % at 4096).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_prefill_shared_kernel(Params p, PrefillWs w, int layer, PrefillAttn a) {
  constexpr int HD = 128, RG = 2, RW = 16 * RG, RQ = 4 * RW;  // 32 rows per wavefront, 128 per workgroup
  constexpr int STEP = 32;                                    // keys per step
  __shared__ u32x4 sK0[8][64], sK1[8][64], sV0[8][64], sV1[8][64];

  const int head = blockIdx.x, n_blk = gridDim.y, half = (n_blk + 1) / 2;
  const int blk = (int)blockIdx.y < half ? (int)blockIdx.y : n_blk - 1 - ((int)blockIdx.y - half);
  const int slot = a.slot[blk], rows = a.rows[blk];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ml = lane & 15, g = lane >> 4;
  const int r0w = a.row[blk] + wave * RW;        // first row of this wavefront (of the pass), at position `at` of the sequence
  const int at = a.pos[blk] + wave * RW;
  const int nr = max(0, min(RW, rows - wave * RW));  // its rows (0: the prompt ends before them)
  const int k_all = a.pos[blk] + rows;               // keys visible to the workgroup's last row
  const int k_own = nr ? at + nr : 0;                // keys visible to this wavefront's last row
  const uint16_t *kpool = (const uint16_t *)p.k_pool, *vpool = (const uint16_t *)p.v_pool;

  // this wavefront's share of a step: K fragments 2 * wave, 2 * wave + 1 (fragment t * 4 + j: 16 key slots of half t, dims
  // j * 32 ..) and the V fragments of dim blocks 2 * wave, 2 * wave + 1
  auto issue = [&](u32x4 (*dK)[64], u32x4 (*dV)[64], int base) __attribute__((always_inline)) {
    const int page = p.block_table[(size_t)slot * p.pages_per_seq + (base >> p.page_shift)];
    const int poff = base & (p.page_size - 1);
    const size_t hbase = ((size_t)layer * p.n_pages + page) * p.H + head;
    const uint16_t *kp = kpool + (hbase * HD * p.page_size + poff * 8);    // K[dim / 8][key][8]
    const uint16_t *vp = vpool + (hbase * p.page_size + poff) * HD;        // V[key / 8][dim][8]
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int f = wave * 2 + i, key = (ml >> 2) * 8 + (f >> 2) * 4 + (ml & 3);  // key slot ml of half f >> 2
      copy_to_lds(kp + (((f & 3) * 4 + g) * p.page_size + key) * 8, &dK[f][0]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      copy_to_lds(vp + (g * HD + (wave * 2 + i) * 16 + ml) * 8, &dV[wave * 2 + i][0]);
  };
  issue(sK0, sV0, 0);

  u32x4 qh[RG][4], ql[RG][4];
  {
    const float scale = rsqrtf((float)HD) * 1.4426950408889634f;
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const int rr = rg * 16 + ml;
      const bool live = rr < nr;
      const float *qp = w.q + (size_t)(live ? r0w + rr : a.row[blk]) * p.D + head * HD + g * 8;
      floatx4 raw[4][2];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        raw[j][0] = *(const floatx4 *)(qp + j * 32);
        raw[j][1] = *(const floatx4 *)(qp + j * 32 + 4);
      }
      const float sc_q = live ? scale : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          qh[rg][j][2 * h] = split2_bf16(raw[j][h][0] * sc_q, raw[j][h][1] * sc_q, true);
          qh[rg][j][2 * h + 1] = split2_bf16(raw[j][h][2] * sc_q, raw[j][h][3] * sc_q, true);
          ql[rg][j][2 * h] = split2_bf16(raw[j][h][0] * sc_q, raw[j][h][1] * sc_q, false);
          ql[rg][j][2 * h + 1] = split2_bf16(raw[j][h][2] * sc_q, raw[j][h][3] * sc_q, false);
        }
    }
  }

  floatx4 o[RG][8];
  float m_ref[RG], l_run[RG];  // reference of the exponentials (the same in a row's four lanes), this lane's sum
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    m_ref[rg] = -__FLT_MAX__;  // no score is lower: the first step moves it.  Not -inf: a row past the last one has all its
    l_run[rg] = 0.f;           //   keys masked in some steps, and -inf - -inf would not be a number
#pragma unroll
    for (int db = 0; db < 8; ++db) o[rg][db] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  auto scores = [&](floatx4 (&sc)[RG][2], const u32x4 (*dK)[64]) __attribute__((always_inline)) {
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
#pragma unroll
      for (int t = 0; t < 2; ++t) sc[rg][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8 kf = __builtin_bit_cast(bf16x8, dK[t * 4 + j][lane]);
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) sc[rg][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, qh[rg][j]), sc[rg][t], 0, 0, 0);
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) sc[rg][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, ql[rg][j]), sc[rg][t], 0, 0, 0);
      }
  };
  // lane (ml, g) holds the scores of row rg * 16 + ml for keys base + 8g + 4t + r; turns them into (hi, lo) probabilities
  auto softmax = [&](floatx4 (&sc)[RG][2], u32x4 (&ph)[RG], u32x4 (&pl)[RG], int base, bool masked) __attribute__((always_inline)) {
    float top[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      if (masked) {
        const int last = at + rg * 16 + ml - base - 8 * g;  // the row's last key, counted from this lane's first
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) sc[rg][t][r] = 4 * t + r <= last ? sc[rg][t][r] : -INFINITY;
      }
      top[rg] = fmaxf(fmaxf(fmaxf(sc[rg][0][0], sc[rg][0][1]), fmaxf(sc[rg][0][2], sc[rg][0][3])),
                      fmaxf(fmaxf(sc[rg][1][0], sc[rg][1][1]), fmaxf(sc[rg][1][2], sc[rg][1][3])));
    }
    bool above = false;
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) above |= top[rg] > m_ref[rg] + 8.f;
    if (__builtin_amdgcn_ballot_w64(above) != 0) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        float m = fmaxf(top[rg], m_ref[rg]);
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
        const float alpha = __builtin_amdgcn_exp2f(m_ref[rg] - m);
        m_ref[rg] = m;
        l_run[rg] *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) o[rg][db] *= alpha;
      }
    }
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      float pv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pv[i] = __builtin_amdgcn_exp2f(sc[rg][i >> 2][i & 3] - m_ref[rg]);
      l_run[rg] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ph[rg][i] = pack2_bf16(pv[2 * i], pv[2 * i + 1]);
        pl[rg][i] = pack2_bf16(pv[2 * i] - __uint_as_float(ph[rg][i] << 16), pv[2 * i + 1] - __uint_as_float(ph[rg][i] & 0xffff0000u));
      }
    }
  };
  auto output = [&](const u32x4 (&ph)[RG], const u32x4 (&pl)[RG], const u32x4 (*dV)[64]) __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const bf16x8 vf = __builtin_bit_cast(bf16x8, dV[db][lane]);
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) o[rg][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, ph[rg]), o[rg][db], 0, 0, 0);
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) o[rg][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, pl[rg]), o[rg][db], 0, 0, 0);
    }
  };
  // The step's tiles have landed (every wavefront waits for its own copies, and for its reads of the step before, then
  // they meet); the other stage, which everybody has finished reading, is filled with the next step's.
  auto step = [&](const u32x4 (*dK)[64], const u32x4 (*dV)[64], u32x4 (*nK)[64], u32x4 (*nV)[64], int base) __attribute__((always_inline)) {
    wait_copies<0>();
    wait_lds_reads();
    meet();
    if (base + STEP < k_all) issue(nK, nV, base + STEP);
    if (base >= k_own) return;  // past this wavefront's last row
    const bool masked = base + STEP > at + 1;  // some row of this wavefront does not see all of the step
    floatx4 sc[RG][2];
    u32x4 ph[RG], pl[RG];
    scores(sc, dK);
    softmax(sc, ph, pl, base, masked);
    output(ph, pl, dV);
  };
  for (int base = 0; base < k_all; base += 2 * STEP) {
    step(sK0, sV0, sK1, sV1, base);
    if (base + STEP < k_all) step(sK1, sV1, sK0, sV0, base + STEP);
  }

  // lane (ml, g) holds dims db * 16 + 4g + r of row rg * 16 + ml; a row's sum of probabilities is
  // spread over the four g groups
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    const int rr = rg * 16 + ml;
    float l = l_run[rg];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (rr >= nr) continue;
    const float inv_l = 1.0f / l;  // every live row sees key 0
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const float tv[4] = {o[rg][db][0] * inv_l, o[rg][db][1] * inv_l, o[rg][db][2] * inv_l, o[rg][db][3] * inv_l};
      store_split4(p.attn_x, r0w + rr, p.D, head * HD + db * 16 + 4 * g, tv);
    }
  }
}

}  // namespace

void launch_prefill_qkv(const Params &p, const PrefillWs &w, const void *W, int layer, const PrefillSegs &segs, int M,
                        hipStream_t s) {
  TileArgs a{(const u32x4 *)W, (const u32x4 *)p.xg, M, p.d, 3 * p.D / 16, layer, nullptr, segs, 0, 0, 0, 1, 0, nullptr};
  launch_tile<TILE_QKV>(p, w, a, s);
}
int launch_prefill_resid(const Params &p, const PrefillWs &w, const void *W, const uint16_t *X, int K, const void *gain_next, int M,
                         hipStream_t s) {
  TileArgs a{(const u32x4 *)W, (const u32x4 *)X, M, K, p.d / 16, 0, (const uint16_t *)gain_next, PrefillSegs{}, 0, 0, 0, 1, 0, nullptr};
  return launch_tile<TILE_RESID>(p, w, a, s);
}
void launch_prefill_gateup(const Params &p, const PrefillWs &w, const void *W, int M, hipStream_t s) {
  TileArgs a{(const u32x4 *)W, (const u32x4 *)p.xg, M, p.d, 2 * p.F / 16, 0, nullptr, PrefillSegs{}, 0, 0, 0, 1, 0, nullptr};
  launch_tile<TILE_GATEUP>(p, w, a, s);
}
void launch_prefill_attention(const Params &p, const PrefillWs &w, int layer, const PrefillAttn &a, bool shared, hipStream_t s) {
  if (a.n == 0) return;
  if (shared)
    attn_prefill_shared_kernel<<<dim3(p.H, a.n), 256, 0, s>>>(p, w, layer, a);
  else if (w.attn_rows == 16)
    attn_prefill_kernel<1><<<dim3(a.n * (kPrefillBlockRows / 16), p.H), 256, 0, s>>>(p, w, layer, a);
  else
    attn_prefill_kernel<2><<<dim3(a.n * (kPrefillBlockRows / 32), p.H), 256, 0, s>>>(p, w, layer, a);
}

// Row assembly of a tiled pass that carries rows of several sequences (see PrefillSegs): h (fp32), (hi, lo) of
// h * gain of the first norm, partial sums of h^2 (partial 0 carries the whole row), rotary table at the row's
// own position.  Padding rows are assembled like any other (their token is whatever `p.prefill_ids` holds for
// them, position 0): rows are independent, and nothing of a padding row is ever cached or read.
__global__ __launch_bounds__(256) void assemble_prefill_segs_kernel(Params p, const uint16_t *tok_emb, const uint16_t *gain0,
                                                                    PrefillSegs segs, int ssq_parts, int ssq_stride) {
  __shared__ float red[4];
  const int m = blockIdx.x, sb = m / kPrefillBlockRows, sr = m % kPrefillBlockRows;
  const int pos = sr < segs.rows[sb] ? segs.pos[sb] + sr : 0;
  const uint16_t *src = tok_emb + (size_t)clamp_token(p, p.prefill_ids[m]) * p.d;
  float ss = 0.f;
  for (int c0 = threadIdx.x * 8; c0 < p.d; c0 += 256 * 8) {
    const uint4 sv = *(const uint4 *)(src + c0), gv = *(const uint4 *)(gain0 + c0);
    const uint32_t sw[4] = {sv.x, sv.y, sv.z, sv.w}, gw[4] = {gv.x, gv.y, gv.z, gv.w};
    float v[8], x[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(sw[e] << 16);
      v[2 * e + 1] = __uint_as_float(sw[e] & 0xffff0000u);
      x[2 * e] = v[2 * e] * __uint_as_float(gw[e] << 16);
      x[2 * e + 1] = v[2 * e + 1] * __uint_as_float(gw[e] & 0xffff0000u);
    }
    float4 *hp = (float4 *)(p.h + (size_t)m * p.d + c0);
    hp[0] = make_float4(v[0], v[1], v[2], v[3]);
    hp[1] = make_float4(v[4], v[5], v[6], v[7]);
    const float x0[4] = {x[0], x[1], x[2], x[3]}, x1[4] = {x[4], x[5], x[6], x[7]};
    store_split4(p.xg, m, p.d, c0, x0);
    store_split4(p.xg, m, p.d, c0 + 4, x1);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  for (int i = threadIdx.x; i < ssq_parts; i += 256)
    p.ssq[(size_t)i * ssq_stride + m] = (i == 0) ? (red[0] + red[1] + red[2] + red[3]) : 0.f;
  const int half = p.hd / 2;
  for (int i = threadIdx.x; i < half; i += 256) {
    double sn, cs;
    sincos((double)pos * p.rope_theta[i], &sn, &cs);
    p.rope_cos[(size_t)m * half + i] = (float)cs;
    p.rope_sin[(size_t)m * half + i] = (float)sn;
  }
}

void launch_assemble_prefill_segs(const Params &p, const void *tok_emb, const void *gain0, const PrefillSegs &segs, int M,
                                  int ssq_parts, int ssq_stride, hipStream_t s) {
  assemble_prefill_segs_kernel<<<M, 256, 0, s>>>(p, (const uint16_t *)tok_emb, (const uint16_t *)gain0, segs, ssq_parts, ssq_stride);
}

}  // namespace pass
