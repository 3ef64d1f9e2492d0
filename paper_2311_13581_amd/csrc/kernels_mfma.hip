// Matrix-core path of the (1+k)-row decode step for bf16 models on gfx950.
//
// The step is bound by streaming the weights once (Section 2.2 of the paper: a few extra rows
// cost about as much as one row because decoding is memory-bound).  Every weight matrix is
// repacked at load time into tiles of 16 output features x 32 input features, stored in the lane
// order of v_mfma_f32_16x16x32_bf16's A operand, so that one wavefront fetches a tile as 64
// adjacent 16-byte loads (1 KB, fully coalesced) and a strip of 16 output features is one
// contiguous run of K/32 KB.  The M <= 64 activation rows are the B operand (rows padded to 16
// per MFMA).  A workgroup of 4 to 16 wavefronts owns one to four strips (or pairs of a gate and an up
// strip; up to eight strips for calls with more than 8 rows) and splits K among its wavefronts;
// the next trip's weight tiles are requested before the current trip computes (calls with more than
// 8 rows: through rings of LDS stages); partial tiles are reduced through LDS in a fixed order (deterministic).  No workgroup shares weights with another,
// and the activation rows (tens of KB) sit in every XCD's L2, so the block-to-XCD mapping needs
// no special order.
//
// Activations keep fp32-like precision although the matrix core takes bf16: every activation x
// is carried as a pair (hi, lo) of bf16 values, hi = bf16(x), lo = bf16(x - hi).  Eight rows fill
// one 16-column MFMA: columns 0..7 take the hi halves, columns 8..15 the lo halves of the same
// rows, and the epilogue adds column j+8 to column j.  So a (1+k)-row call with k <= 7 costs one
// MFMA and one activation load per weight tile, and nothing but the weights and the K/V cache is
// ever rounded to 8 bits of mantissa (the paper's bfloat16 is read as the storage format of the
// model, Training details).  Activation buffers are laid out for that, in tiles like the weights:
// [group of 8 rows][K/32][4][hi, lo][xr][8]: eight consecutive features (k/8 % 4 of the k-tile) of
// the hi halves of xr rows, then of their lo halves.  xr is 8, where a wavefront fetches its B operand
// of a k-tile as 1 KB of whole cache lines in lane order, and the call's rows if these are fewer
// (Params::xr, xs_index).
//
// Fused epilogues:
//   QKV     : RMSNorm scale, rotary embedding, q (fp32) to the workspace, K/V rows (bf16) into
//             the paged cache
//   RESID   : residual add into h (fp32), (hi, lo) of h * gain of the next norm, per-strip
//             partial sums of h^2
//   GATEUP  : RMSNorm scale, silu(gate) * up as (hi, lo)
//   LOGITS  : RMSNorm scale, fp32 logits into the slot's logits rows
// RMSNorm has no kernel: the producer stores (hi, lo) of h * gain and partial sums of h^2; the
// consumer multiplies its accumulators by rsqrt(mean(h^2) + eps), which commutes with the GEMM.
#include <limits.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "lds_copy.h"
#include "pass_internal.h"

namespace pass {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));


// ---------------------------------------------------------------------------------------------
// Weight repacking: plain [N][K] bf16 -> tiles [strip][K/32][64 lanes][8], lane l of a tile holds
// row (l % 16), columns (l / 16) * 8 .. + 8 of the tile.  Destination strip = off + stride * s.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_tiles_kernel(const uint4 *src, uint4 *dst, int N, int K,
                                                         int strip_off, int strip_stride) {
  const int KT = K / 32;
  size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;  // one 16-byte chunk each
  size_t total = (size_t)(N / 16) * KT * 64;
  if (idx >= total) return;
  int lane = (int)(idx & 63);
  size_t tile = idx >> 6;
  int kt = (int)(tile % KT);
  int s = (int)(tile / KT);
  int row = s * 16 + (lane & 15);
  int col = kt * 32 + (lane >> 4) * 8;
  size_t dstrip = (size_t)strip_off + (size_t)strip_stride * s;
  dst[(dstrip * KT + kt) * 64 + lane] = src[((size_t)row * K + col) / 8];
}

void launch_pack_tiles(const uint16_t *src, uint16_t *dst, int N, int K, int strip_off, int strip_stride,
                       hipStream_t s) {
  size_t total = (size_t)(N / 16) * (K / 32) * 64;
  pack_tiles_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const uint4 *)src, (uint4 *)dst, N, K,
                                                                      strip_off, strip_stride);
}

// ---------------------------------------------------------------------------------------------
// Coded weights: the same tiles in 12 bits a weight, without loss.
// A decode-sized product is bound by the bytes of its weights, and a trained (or random) matrix uses few of the 256
// exponents a bf16 value can have.  A coded tile holds each weight's low byte (the exponent's last bit and the mantissa)
// as it is, and its high byte (sign and the exponent's upper seven bits) as a sign and an index into a table of eight
// values per matrix: 12 bytes a lane instead of 16, which twelve byte operations turn back into the tile's 16.  Eight
// values of the upper seven bits are 16 octaves: of normally distributed weights one in ten thousand falls outside.  Up to two
// of those per tile stand in a fix word beside it (place and bits); a tile with more is read in its plain form.  What a
// product multiplies is bit for bit the plain weight.
// Measured at 5 rows (7B shapes, us, plain -> coded): QKV 17.6 -> 14.6, gate/up 29.0 -> 23.0, LM head 41.2 -> 31.4, Wo
// 8.1 -> 7.4, down 17.4 -> 16.1 (beside activation tiles with room for 8 rows; xs_index has what tiles of 5 give).
// ---------------------------------------------------------------------------------------------
typedef uint32_t u32x3 __attribute__((ext_vector_type(3), aligned(4)));
constexpr int kCodedTile = 768;  // bytes
template <bool Z> struct LaneTile { typedef u32x4 T; };  // what a lane holds of a weight tile
template <> struct LaneTile<true> { typedef uint32_t T __attribute__((ext_vector_type(3))); };
// Weights that the table does not hold: two words per tile.  The first: bits 0..15 the weight, 16..18 its place among the lane's
// eight, 19..24 the lane, 25 set where there is one.  The second: the same for another, or, with bit 31 set, how many more there
// are (bits 24..30) and where in the matrix's overflow list they stand (bits 0..23).
constexpr uint32_t kFixValid = 1u << 25, kFixMore = 1u << 31;
constexpr int kFixMost = 128;  // of a tile
// Fix words of a strip stand by k-tile modulo 4, so that those of a wavefront (every 4th, 8th or 16th k-tile) lie close.
__host__ __device__ constexpr int fix_stride(int KT) { return (KT + 3) / 4 * 4; }
__device__ __forceinline__ int fix_index(int KT, int kt) { return (kt & 3) * (fix_stride(KT) / 4) + (kt >> 2); }

__device__ __forceinline__ u32x4 decode_tile(LaneTile<true>::T c, uint32_t lut0, uint32_t lut1) {
  const uint32_t h0 = __builtin_amdgcn_perm(lut1, lut0, c[2] & 0x07070707u) | ((c[2] << 4) & 0x80808080u);
  const uint32_t h1 = __builtin_amdgcn_perm(lut1, lut0, (c[2] >> 4) & 0x07070707u) | (c[2] & 0x80808080u);
  u32x4 t;
  t[0] = __builtin_amdgcn_perm(h0, c[0], 0x05010400u);
  t[1] = __builtin_amdgcn_perm(h0, c[0], 0x07030602u);
  t[2] = __builtin_amdgcn_perm(h1, c[1], 0x05010400u);
  t[3] = __builtin_amdgcn_perm(h1, c[1], 0x07030602u);
  return t;
}
// puts the weight of a (wavefront-uniform) fix word into its place
__device__ __forceinline__ void fix_weight(u32x4 &t, uint32_t w, int lane) {
  const bool mine = lane == (int)((w >> 19) & 63);
  const uint32_t e = (w >> 16) & 7, sh = (e & 1) * 16, keep = 0xffff0000u >> sh, v = (w & 0xffffu) << sh;
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) t[q] = mine & ((e >> 1) == q) ? (t[q] & keep) | v : t[q];
}
// the tile's two words applied (both wavefront-uniform).  The overflow list comes through scalar loads: the requests for the next
// tiles stay in flight.
__device__ __forceinline__ void fix_tile(u32x4 &t, uint32_t w0, uint32_t w1, const uint32_t *more, int lane) {
  typedef const __attribute__((address_space(4))) uint32_t *Uniform;
  const Uniform list = (Uniform)(uintptr_t)(more + (w1 & 0xffffff));
  const int left = w1 & kFixMore ? (w1 >> 24) & 127 : w1 ? 1 : 0;
  for (int i = 0;; ++i) {  // (one copy of the body: it stands in a kernel once per strip and unrolled k-tile)
    fix_weight(t, w0, lane);
    if (i == left) break;
    w0 = w1 & kFixMore ? list[i] : w1;
  }
}

// How often each value of the upper seven exponent bits occurs in a matrix of packed tiles (in every step-th 16 bytes: the
// table need not be the best there is).
__global__ __launch_bounds__(256) void exponents_kernel(const uint4 *src, size_t n, size_t step, uint32_t *hist) {
  __shared__ uint32_t h[128];
  if (threadIdx.x < 128) h[threadIdx.x] = 0;
  __syncthreads();
  for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * step; i < n; i += (size_t)gridDim.x * 256 * step) {
    const uint4 v = src[i];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      atomicAdd(&h[(w[q] >> 8) & 127], 1u);
      atomicAdd(&h[(w[q] >> 24) & 127], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 128 && h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}
void launch_exponents(const void *src, size_t weights, uint32_t *hist, hipStream_t s) {
  const size_t n = weights / 8, step = std::max<size_t>(1, n >> 16) | 1;  // odd: no lane of a tile is left out
  exponents_kernel<<<128, 256, 0, s>>>((const uint4 *)src, n, step, hist);
}

// Packed tiles -> coded tiles and fix words, a wavefront per four tiles.  counts[0]: entries of the overflow list taken so far, counts[1]:
// set where the copy does not hold the matrix (the list is full, or a tile has more than kFixMost weights outside the table).  load: what
// the tile's strip has outside in the k-tiles that go with this one.
__device__ __forceinline__ void code_tile(const uint4 v, const Coded &z, size_t tile, uint2 *words, uint32_t *load, uint32_t *counts, int lane) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  const uint32_t first = z.lut0 & 255, base = (z.lut0 >> 8 & 255) - 1;  // the table: `first`, then a run from base + 1 (coded_table)
  uint32_t c[3] = {0, 0, 0};
  uint64_t out[8];
  int n = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t b = (w[e >> 1] >> ((e & 1) * 16)) & 0xffffu, up = (b >> 8) & 127;
    const uint32_t d = up - base;
    const bool run = d - 1 < 7;
    c[e >> 2] |= (b & 255) << ((e & 3) * 8);
    c[2] |= ((run ? d : 0) | (b >> 15) << 3) << ((e & 3) * 8 + (e >> 2) * 4);
    out[e] = __ballot(!run && up != first);
    n += __popcll(out[e]);
  }
  *(u32x3 *)((char *)z.tiles + tile * kCodedTile + lane * 12) = u32x3{c[0], c[1], c[2]};
  if (n == 0) {
    if (lane == 0) *words = make_uint2(0, 0);
    return;
  }
  if (lane == 0) atomicAdd(load, (uint32_t)n);
  uint32_t at = 0;
  if (n > 2) {
    if (lane == 0) at = atomicAdd(&counts[0], (uint32_t)n - 1);
    at = __shfl((int)at, 0);
    if (n > kFixMost || (size_t)at + n - 1 > z.more_room) {
      if (lane == 0) counts[1] = 1;
      return;
    }
  }
  if (n != 2 && lane == 0) words->y = n == 1 ? 0 : kFixMore | (uint32_t)(n - 1) << 24 | at;
  int before = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (out[e] >> lane & 1) {
      const int i = before + __popcll(out[e] & ((1ull << lane) - 1));  // its number among the tile's
      const uint32_t word = ((w[e >> 1] >> ((e & 1) * 16)) & 0xffffu) | (uint32_t)e << 16 | (uint32_t)lane << 19 | kFixValid;
      if (i == 0) words->x = word;
      else if (n == 2) words->y = word;
      else z.more[at + i - 1] = word;
    }
    before += __popcll(out[e]);
  }
}
__global__ __launch_bounds__(256) void code_tiles_kernel(const uint4 *src, Coded z, int KT, size_t tiles, uint32_t *counts) {
  const int lane = threadIdx.x & 63;
  const size_t tile0 = ((size_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 4;
  uint4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = src[(tile0 + i < tiles ? tile0 + i : tiles - 1) * 64 + lane];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const size_t tile = tile0 + i, strip = tile / KT;
    const int kt = (int)(tile - strip * KT);
    if (tile < tiles) code_tile(v[i], z, tile, z.fix + strip * fix_stride(KT) + fix_index(KT, kt), z.load + strip * 4 + (kt & 3), counts, lane);
  }
}
void launch_code_tiles(const void *src, const Coded &z, int N, int K, uint32_t *counts, hipStream_t s) {
  const size_t tiles = (size_t)(N / 16) * (K / 32);
  code_tiles_kernel<<<(unsigned)((tiles + 15) / 16), 256, 0, s>>>((const uint4 *)src, z, K / 32, tiles, counts);
}
// Whether the products of up to 8 rows gain by a copy with that many weights outside its table (load: [N / 16][4], the weights of a strip
// whose k-tiles agree modulo 4, which the same wavefronts read).  A wavefront puts them in one after the other, 0.10 to 0.14 us each,
// while the other wavefronts of its workgroup wait at the end.
// Over all: gate/up of d 4096, 5 rows, 29.3 us plain, with 0.04 weights of a tile outside (normally distributed ones) 24.0, 0.3 25.5, 0.55 27.1, 0.8
// 32.4, one in every tile 33.5, two 47.7.  In one place: a tile with 32 outside 24.0 us, with 64 26.2, with 128 39.5; a strip with one
// row of zeros (32 in every tile) 177, with two 342.  Twice what there is on average, and 12, is beyond what chance
// does to normally distributed weights (60 to 190 in a million outside, by their scale).
bool coded_pays_for(const uint32_t *load, int N, int K, float *outside) {
  uint64_t all = 0;
  uint32_t most = 0;
  const size_t n = (size_t)N / 16 * 4;
  for (size_t i = 0; i < n; ++i) { all += load[i]; most = std::max(most, load[i]); }
  *outside = (float)((double)all * 512 / ((double)N * K));
  return *outside <= 0.4f && most <= 12 + 2 * all / n;
}
// The table of a matrix: the eight values that leave the fewest weights outside, a run of eight or zero's and a run of seven.
void coded_table(const uint32_t *hist, uint32_t *lut0, uint32_t *lut1) {
  uint64_t best = 0;
  int at = 0, zero = 0;
  for (int z = 0; z < 2; ++z)
    for (int b = z; b + 8 - z <= 128; ++b) {
      uint64_t in = z ? hist[0] : 0;
      for (int i = 0; i < 8 - z; ++i) in += hist[b + i];
      if (in > best) { best = in; at = b; zero = z; }
    }
  uint8_t t[8];
  for (int i = 0; i < 8; ++i) t[i] = (uint8_t)(zero ? (i ? at + i - 1 : 0) : at + i);
  memcpy(lut0, t, 4);
  memcpy(lut1, t + 4, 4);
}

// ---------------------------------------------------------------------------------------------
// Row assembly for the matrix-core path: h (fp32), (hi, lo) of h * gain of the first norm,
// partial sums of h^2 (partial 0 carries the whole row, the others are zero), rotary table,
// row tables.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void assemble_mfma_kernel(Params p, const uint16_t *tok_emb,
                                                            const uint16_t *lookahead, const uint16_t *gain0,
                                                            int mode, int R, int ssq_parts, int ssq_stride,
                                                            int row_tables) {
  __shared__ float red[4];
  int m = blockIdx.x, b = m / R, r = m % R;
  int slot = p.step_slots[b];
  int pos = p.kv_len[slot] + r;
  if (m == 0 && threadIdx.x == 0 && mode != MODE_PREFILL) p.clock[mode == MODE_DRAFT ? 0 : 1] = wall_clock64();
  const bool dead = row_is_dead(p, mode, slot, R);
  const uint16_t *src;
  if (mode == MODE_PREFILL) {
    src = tok_emb + (size_t)p.prefill_ids[r] * p.d;
  } else if (r == 0) {
    src = tok_emb + (size_t)clamp_token(p, p.pending[slot]) * p.d;
  } else if (mode == MODE_DRAFT) {
    // look-ahead embedding r (Section 2.2.1), or the fixed token of the paper's second baseline
    src = p.la_token >= 0 ? tok_emb + (size_t)p.la_token * p.d : lookahead + (size_t)(r - 1) * p.d;
  } else {
    src = tok_emb + (size_t)clamp_token(p, p.drafts[slot * kMaxK + (r - 1)]) * p.d;
  }
  // eight consecutive features per thread and trip: one 16-byte load of the embedding row and of
  // the gain, two 16-byte stores of h, one 16-byte store each of the hi and the lo tile slots
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
    uint4 hi, lo;
    hi.x = split2_bf16(x[0], x[1], true); lo.x = split2_bf16(x[0], x[1], false);
    hi.y = split2_bf16(x[2], x[3], true); lo.y = split2_bf16(x[2], x[3], false);
    hi.z = split2_bf16(x[4], x[5], true); lo.z = split2_bf16(x[4], x[5], false);
    hi.w = split2_bf16(x[6], x[7], true); lo.w = split2_bf16(x[6], x[7], false);
    uint16_t *xh = p.xg + xs_index(m, p.d, c0, p.xr);
    *(uint4 *)xh = hi;
    *(uint4 *)(xh + kXsLo * p.xr) = lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  for (int i = threadIdx.x; i < ssq_parts; i += 256)
    p.ssq[(size_t)i * ssq_stride + m] = (i == 0) ? (red[0] + red[1] + red[2] + red[3]) : 0.f;
  int half = p.hd / 2;
  for (int i = threadIdx.x; i < half; i += 256) {
    double sn, cs;
    sincos((double)pos * p.rope_theta[i], &sn, &cs);
    p.rope_cos[(size_t)m * half + i] = (float)cs;
    p.rope_sin[(size_t)m * half + i] = (float)sn;
  }
  if (threadIdx.x == 0 && row_tables) {
    p.row_pos[m] = dead ? 0 : pos;
    p.row_slot[m] = dead ? -1 : slot;
    p.row_page[m] = dead ? -1 : p.block_table[(size_t)slot * p.pages_per_seq + (pos >> p.page_shift)];
    p.row_out[m] = slot * (1 + p.k) + r;
  }
}

void launch_assemble_mfma(const Params &p, const void *tok_emb, const void *lookahead, const void *gain0, int mode,
                          int B, int R, hipStream_t s) {
  assemble_mfma_kernel<<<B * R, 256, 0, s>>>(p, (const uint16_t *)tok_emb, (const uint16_t *)lookahead,
                                             (const uint16_t *)gain0, mode, R, p.d / 16, kMaxRows, 1);
}

// ---------------------------------------------------------------------------------------------
// The streaming GEMM
// ---------------------------------------------------------------------------------------------
enum { EPI_QKV = 0, EPI_RESID = 1, EPI_GATEUP = 2, EPI_LOGITS = 3, EPI_PARTIAL = 4, EPI_GATEUP_SAVE = 5 };

template <int I> struct nb_c { static constexpr int value = I; };

struct GemmArgs {
  const u32x4 *W;             // packed weight tiles
  const uint16_t *X;          // activation rows as (hi, lo) tiles [ceil(M/8)][K/32][4][hi, lo][p.xr][8]
  int M, K;
  int layer;
  const uint16_t *gain_next;  // RESID: gain of the norm that follows
  float *logits;              // LOGITS: base of the [slot][1+k][V] logits
  int kt_split;               // PARTIAL: k-tiles per workgroup row (blockIdx.y picks the slice of K); else 0
  float *partial;             // PARTIAL: [gridDim.y][kMaxRows][N] sums over the slice of K
  int n_strips;               // strips of the matrix (the last workgroup may own fewer blocks)
  int ldy;                    // PARTIAL: features per row of `partial`
  float *gu_save;             // GATEUP_SAVE: [M][2F] gate | up before the activation (what its derivative needs)
  Coded z;                    // the matrix in its coded form, read in place of W where the kernel says so
};

// What follows the K loop, for the register and the LDS-ring form alike.  All that the epilogue reads from memory is requested
// together and early (the register form: behind the first trip's requests; the ring form: behind the last tile): with one workgroup a
// compute unit nothing else hides the trips.  One after the other they took, after the K loop, 1.9 us of the QKV product's 15.5 at 5 rows, 1.0 of
// gate/up's 23.8, and at 40 rows 5.3 of 27.4 and 4.7 of 36.9.
// MB: row groups whose partial tiles the areas of LDS take at a time.
template <int MT, int EPI, int WAVES, int NB, int NS, int MB>
struct Epilogue {
  static constexpr bool GU = (EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE);
  static constexpr int PER = GU ? 2 : 1;  // strips per block
  static constexpr bool NORM = (EPI != EPI_RESID && EPI != EPI_PARTIAL);
  static_assert(NS == NB * PER, "strips of a workgroup");
  static constexpr int UNITS = (MB * NB + WAVES - 1) / WAVES;  // (row group, block) pairs of a wavefront per batch of row groups
  // The partial sums of h^2 (written by the producer of X, [strip][kMaxRows]) in rounds.  Few rows: a value a lane and request, lane
  // (ml & 7) has row ml & 7, the two halves of the columns and the four groups of lanes take alternate partials.  More rows: four rows a lane,
  // 16 lanes a partial.
  static constexpr int ASKED = NORM ? (MT == 1 ? 8 : 16) : 1;
  static constexpr int ROUND = WAVES * 64;  // partials of a round, in either form
  floatx4 norm[ASKED];
  float2 cs[UNITS], sn[UNITS];  // QKV
  int pos[UNITS], page[UNITS], out[UNITS];  // QKV; LOGITS
  floatx4 h[UNITS];             // RESID
  uint2 gain[UNITS];

  // row and first feature of the wavefront's j-th unit of the batch that begins with row group mt0; false: there is none
  __device__ __forceinline__ static bool unit(int j, int mt0, int strip0, int n_strips, int &mt, int &blk, int &strip) {
    const int u = (threadIdx.x >> 6) + j * WAVES;
    const int mb = u / NB;
    blk = u - mb * NB;
    mt = mt0 + mb;
    strip = strip0 + blk * PER;
    return u < MB * NB && mt < MT && strip < n_strips;
  }
  __device__ __forceinline__ void ask_norm(const Params &p, int round) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int NP = p.d / 16;
    // through a buffer descriptor: indices past the end read as zero
    const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc((void *)p.ssq, 0, NP * kMaxRows * 4, 0x00020000);
#pragma unroll
    for (int u = 0; u < ASKED; ++u) {
      if constexpr (MT == 1) {
        const int i = round * ROUND + u * WAVES * 8 + wave * 8 + (lane >> 4) * 2 + ((lane >> 3) & 1);
        norm[u][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sr, (i * kMaxRows + (lane & 7)) * 4, 0, 0));
      } else {
        const int i = round * ROUND + u * WAVES * 4 + wave * 4 + (lane >> 4), row = (lane & 15) * 4;
        norm[u] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(sr, row < MT * 8 ? (i * kMaxRows + row) * 4 : 0x40000000, 0, 0));
      }
    }
  }
  __device__ __forceinline__ void ask_units(const Params &p, const GemmArgs &a, int mt0, int strip0) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < UNITS; ++j) {
      int mt, blk, strip;
      unit(j, mt0, strip0, a.n_strips, mt, blk, strip);
      const int m = min(mt, MT - 1) * 8 + (lane & 7), n = min(strip, a.n_strips - 1) * 16 + 4 * g;
      if constexpr (EPI == EPI_QKV) {
        const int half = p.hd / 2, at = m * half + (n - n / p.hd * p.hd) / 2;  // (projections are whole heads)
        cs[j] = *(const float2 *)(p.rope_cos + at);
        sn[j] = *(const float2 *)(p.rope_sin + at);
        pos[j] = p.row_pos[m];
        page[j] = p.row_page[m];
      } else if constexpr (EPI == EPI_LOGITS) {
        out[j] = p.row_out[m];
      } else if constexpr (EPI == EPI_RESID) {
        h[j] = *(const floatx4 *)(p.h + (size_t)m * p.d + n);
        gain[j] = *(const uint2 *)(a.gain_next + n);
      }
    }
  }
  __device__ __forceinline__ void ask(const Params &p, const GemmArgs &a, int strip0) {
    if constexpr (NORM) ask_norm(p, 0);
    ask_units(p, a, 0, strip0);
  }

  // acc: this wavefront's sums over its k-tiles; red: [WAVES] areas of `red_stride` 16-byte words, one of each wavefront's own
  __device__ __forceinline__ void finish(const Params &p, const GemmArgs &a, floatx4 (&acc)[NS][MT], floatx4 *red, int red_stride,
                                         float (*red_ss)[MT * 8], int strip0) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ml = lane & 15, g = lane >> 4;
    // Per batch of 8-row groups (as many as the areas take): every wavefront posts its partial tiles, then the
    // (row group, block) pairs are shared out: a wavefront reduces a pair's tiles in a fixed order, adds the lo columns to
    // the hi columns and runs the fused epilogue.  Lanes with ml < 8 hold Y[m = mt*8 + ml][n0 + 4g .. 4g+3].
#pragma unroll
    for (int mt0 = 0; mt0 < MT; mt0 += MB) {
      if (mt0 > 0) {
        __syncthreads();  // the previous batch has been read
        ask_units(p, a, mt0, strip0);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (mt0 + mb < MT) red[(size_t)wave * red_stride + (mb * NS + s) * 64 + lane] = acc[s][mt0 + mb < MT ? mt0 + mb : 0];
      if constexpr (NORM) {
        if (mt0 == 0) {
          floatx4 ss = {0.f, 0.f, 0.f, 0.f};
          for (int round = 0;;) {
#pragma unroll
            for (int u = 0; u < ASKED; ++u) {
              if constexpr (MT == 1) ss[0] += norm[u][0];
              else ss += norm[u];
            }
            if (++round * ROUND >= p.d / 16) break;
            ask_norm(p, round);
          }
          if constexpr (MT == 1) {
            ss[0] += __shfl_xor(ss[0], 8);
            ss[0] += __shfl_xor(ss[0], 16);
            ss[0] += __shfl_xor(ss[0], 32);
            if (lane < 8) red_ss[wave][lane] = ss[0];
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              ss[r] += __shfl_xor(ss[r], 16);
              ss[r] += __shfl_xor(ss[r], 32);
            }
            if (lane < MT * 2) *(floatx4 *)&red_ss[wave][lane * 4] = ss;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < UNITS; ++j) {
        int mt, blk, strip;
        if (!unit(j, mt0, strip0, a.n_strips, mt, blk, strip)) continue;  // past the rows, or a block that does not exist
        const int mb = mt - mt0;
        floatx4 y[PER];
#pragma unroll
        for (int s = 0; s < PER; ++s) {
          y[s] = red[(mb * NS + blk * PER + s) * 64 + lane];
#pragma unroll
          for (int w = 1; w < WAVES; ++w) y[s] += red[(size_t)w * red_stride + (mb * NS + blk * PER + s) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) y[s][r] += __shfl_xor(y[s][r], 8);
        }
        const int m = mt * 8 + (ml & 7);
        float inv = 1.f;
        if constexpr (NORM) {
          float ss = 0.f;
#pragma unroll
          for (int w = 0; w < WAVES; ++w) ss += red_ss[w][m];
          inv = 1.0f / sqrtf(ss / (float)p.d + p.eps);
        }
        const bool live = m < a.M && ml < 8;

        if constexpr (EPI == EPI_LOGITS) {
          if (live) {
            float *o = a.logits + (size_t)out[j] * p.V + strip * 16 + 4 * g;
            *(floatx4 *)o = y[0] * inv;
          }
        } else if constexpr (GU) {
          if (live) {
            // strips 2b (gate) and 2b+1 (up) of the interleaved matrix both belong to features 16b..16b+15
            int f0 = (blockIdx.x * NB + blk) * 16 + 4 * g;
            float t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float gt = y[0][r] * inv, up = y[1][r] * inv;
              t[r] = gt / (1.0f + __expf(-gt)) * up;
            }
            store_split4(p.act_x, m, p.F, f0, t, p.xr);
            if constexpr (EPI == EPI_GATEUP_SAVE) {
              *(floatx4 *)(a.gu_save + (size_t)m * 2 * p.F + f0) = y[0] * inv;
              *(floatx4 *)(a.gu_save + (size_t)m * 2 * p.F + p.F + f0) = y[1] * inv;
            }
          }
        } else if constexpr (EPI == EPI_PARTIAL) {
          // sums over this workgroup's slice of K; the slices are added up by resid_reduce_kernel
          if (live)
            *(floatx4 *)(a.partial + ((size_t)blockIdx.y * kMaxRows + m) * a.ldy + strip * 16 + 4 * g) = y[0];
        } else if constexpr (EPI == EPI_RESID) {
          int n = strip * 16 + 4 * g;
          float ss = 0.f;
          if (live) {
            floatx4 hv = h[j] + y[0];
            *(floatx4 *)(p.h_out + (size_t)m * p.d + n) = hv;
            const uint32_t gw[2] = {gain[j].x, gain[j].y};
            float t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              t[r] = hv[r] * __uint_as_float(r & 1 ? gw[r >> 1] & 0xffff0000u : gw[r >> 1] << 16);
              ss += hv[r] * hv[r];
            }
            store_split4(p.xg, m, p.d, n, t, p.xr);
          }
          ss += __shfl_xor(ss, 16);
          ss += __shfl_xor(ss, 32);
          if (lane < 8) p.ssq[(size_t)strip * kMaxRows + m] = ss;  // rows >= M get 0
        } else {  // EPI_QKV
          if (live) {
            int n = strip * 16 + 4 * g;       // column in [0, 3D)
            int which = n / p.D;              // 0 q, 1 k, 2 v
            int c = n - which * p.D;          // column inside the projection
            int head = c / p.hd, dim = c - head * p.hd;
            floatx4 v = y[0] * inv;
            if (which < 2) {
              float x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3];
              v[0] = x0 * cs[j].x - x1 * sn[j].x;
              v[1] = x0 * sn[j].x + x1 * cs[j].x;
              v[2] = x2 * cs[j].y - x3 * sn[j].y;
              v[3] = x2 * sn[j].y + x3 * cs[j].y;
            }
            if (which == 0) {
              *(floatx4 *)(p.qkv + (size_t)m * 3 * p.D + c) = v;
            } else if (page[j] >= 0) {  // a dead row (see row_is_dead) has no place in the cache
              // the cache is bf16 storage: the one place besides the weights where values are rounded
              const int off = pos[j] & (p.page_size - 1);
              uint16_t *pool = (uint16_t *)(which == 1 ? p.k_pool : p.v_pool) + (((size_t)a.layer * p.n_pages + page[j]) * p.H + head) * p.page_size * p.hd;
              if (p.kv_tiled && which == 2) {
#pragma unroll
                for (int r = 0; r < 4; ++r) pool[v_tile(p, off, dim + r)] = f32_to_bf16(v[r]);
              } else {
                uint2 pk;
                pk.x = pack2_bf16(v[0], v[1]);
                pk.y = pack2_bf16(v[2], v[3]);
                *(uint2 *)(pool + (p.kv_tiled ? k_tile(p, off, dim) : (size_t)off * p.hd + dim)) = pk;
              }
            }
          }
        }
      }
    }
  }
};

// byte offset of a lane's 16 bytes in a k-tile of a group of rows that has room for xr of them
__device__ __forceinline__ int x_lane(int lane, int xr) { return ((lane >> 4) * 2 * xr + (lane & 7) + (lane >> 3 & 1) * xr) * 16; }

// Calls of up to 8 rows: one MFMA column block, operands through registers.  A workgroup owns NB output blocks (a block is
// one strip of 16 features, or the gate strip and the up strip of 16 FFN features) and its wavefronts share K: wavefront w
// takes k-tiles w, w + WAVES, ..., U of them a trip, and requests a trip while it computes the one before.  The last trip may
// hold k-tiles past the end: those are requested too (clamped), so that nothing is waited for one by one, and not computed.
// Bound by how evenly the weights are spread over the compute units: a unit takes in about 30 GB/s of weights and the
// activation tile of 8 rows that goes with NB strips costs a third of a weight tile (one with room for fewer rows
// less, by its lines: down on coded weights, d 4096, one strip a workgroup, 16.6 -> 15.3 us at 5 rows and 16.4 -> 14.6 at 1; with several
// strips a workgroup 1 to 2 %), the chip 6.9 TB/s.  Which NB, WAVES and U that asks for: few_rows_shape.
// The sums of a strip have WAVES x NA accumulators, at least 4 for QKV and gate/up and 16 for the other products (fewer
// would round more often).
template <int EPI, int WAVES>
constexpr int few_rows_chains() {
  constexpr int need = (EPI == EPI_QKV || EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE) ? 4 : 16;
  return need > WAVES ? need / WAVES : 1;
}
template <int EPI, int WAVES, int U, int NB, bool Z>
__global__ __launch_bounds__(WAVES * 64) void gemm_mfma_kernel(Params p, GemmArgs a) {
  constexpr int NS = NB * ((EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE) ? 2 : 1);  // strips
  constexpr int NA = few_rows_chains<EPI, WAVES>();
  constexpr int G = NA > U ? NA / U : 1;  // trips until an accumulator's turn comes again
  __shared__ floatx4 red[WAVES * NS * 64];
  __shared__ float red_ss[WAVES][8];
  Epilogue<1, EPI, WAVES, NB, NS, 1> epilogue;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ml = lane & 15;  // MFMA column = pseudo-row
  const int KT = a.K >> 5;   // k-tiles of K (strip stride)
  const int strip0 = blockIdx.x * NS;

  floatx4 acc[NA][NS];
#pragma unroll
  for (int c = 0; c < NA; ++c)
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[c][s] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Activation loads go through a buffer descriptor: a lane whose pseudo-row belongs to a row >= M gets an out-of-range
  // offset and the hardware returns zeros without touching memory.  All loads are unconditional instructions, so
  // outstanding requests are counted exactly and a trip can wait for its operands while the next trip's stay in flight.
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)a.X, 0, 16 * a.K * 2, 0x00020000);
  const int xtile = p.xr * 128;  // bytes of a k-tile of the rows
  const int xoff = (ml & 7) < a.M ? x_lane(lane, p.xr) : 0x40000000;  // byte offset of this lane's 16 bytes in k-tile 0
  typedef typename LaneTile<Z>::T Tile;
  const char *wp[NS];  // strips past the end repeat the last one (in bounds; their results are dropped)
#pragma unroll
  for (int s = 0; s < NS; ++s)
    wp[s] = (const char *)(Z ? a.z.tiles : a.W) + (size_t)(NB > 1 ? min(strip0 + s, a.n_strips - 1) : strip0 + s) * KT * (64 * 4 * (Z ? 3 : 4));

  Tile av[2][U][NS];
  u32x4 bv[2][U];
  auto load = [&](int buf, int trip) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kt = min(wave + (trip * U + u) * WAVES, KT - 1);
      bv[buf][u] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff, kt * xtile, 0);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if constexpr (Z) av[buf][u][s] = __builtin_nontemporal_load((const u32x3 *)(wp[s] + ((size_t)kt * 64 + lane) * 12));
        else av[buf][u][s] = __builtin_nontemporal_load((const u32x4 *)wp[s] + (size_t)kt * 64 + lane);
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // requested here: left alone, the scheduler moves the requests behind the products
  };
  // coded weights: lane j holds the fix words of this wavefront's j-th k-tile (no more than 64 of them: the launcher sees to it)
  u32x2 fix[Z ? NS : 1];
  auto mma = [&](int buf, int g, int u, int trip) __attribute__((always_inline)) {
    u32x4 w[NS];
    if constexpr (Z) {
      const int j = trip * U + u;
      uint32_t w0[NS], any = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        w[s] = decode_tile(av[buf][u][s], a.z.lut0, a.z.lut1);
        w0[s] = (uint32_t)__builtin_amdgcn_readlane((int)fix[s][0], j);
        any |= w0[s];
      }
      if (__builtin_expect(any != 0, 0)) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (w0[s])
            fix_tile(w[s], w0[s], (uint32_t)__builtin_amdgcn_readlane((int)fix[s][1], j), a.z.more, lane);
      }
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) w[s] = av[buf][u][s];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      floatx4 &c = acc[(g * U + u) % NA][s];
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s]), __builtin_bit_cast(bf16x8, bv[buf][u]), c, 0, 0, 0);
    }
  };
  const int trips = (KT + WAVES * U - 1) / (WAVES * U);
  constexpr int STEP = G > 2 ? G : 2;  // trips per turn of the loop: whole turns of the accumulators and of the two buffers
  int t = 0;
  load(0, 0);
  if constexpr (Z) {  // behind the first trip's requests, ahead of the second's
    const int kt = min(wave + lane * WAVES, KT - 1);
#pragma unroll
    for (int s = 0; s < NS; ++s)
      fix[s] = *(const u32x2 *)(a.z.fix + (size_t)min(strip0 + s, a.n_strips - 1) * fix_stride(KT) + fix_index(KT, kt));
    __builtin_amdgcn_sched_barrier(0);
  }
  epilogue.ask(p, a, strip0);
  __builtin_amdgcn_sched_barrier(0);
  for (; t + STEP < trips; t += STEP) {  // (all of these are full)
#pragma unroll
    for (int g = 0; g < STEP; ++g) {
      load((g + 1) & 1, t + g + 1);
#pragma unroll
      for (int u = 0; u < U; ++u) mma(g & 1, g, u, t + g);
    }
  }
  // the last one to STEP trips, each number of them in a line of its own (a request under a condition would be waited for)
  auto rest = [&](auto self, auto gc) __attribute__((always_inline)) -> void {
    constexpr int g = decltype(gc)::value;
    if constexpr (g + 1 < STEP) {
      if (t + g + 1 < trips) {
        load((g + 1) & 1, t + g + 1);
#pragma unroll
        for (int u = 0; u < U; ++u) mma(g & 1, g, u, t + g);
        self(self, nb_c<g + 1>{});
        return;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (wave + ((t + g) * U + u) * WAVES < KT) mma(g & 1, g, u, t + g);
  };
  rest(rest, nb_c<0>{});
  floatx4 sum[NS][1];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    sum[s][0] = acc[0][s];
#pragma unroll
    for (int c = 1; c < NA; ++c) sum[s][0] += acc[c][s];
  }
  epilogue.finish(p, a, sum, red, NS * 64, red_ss, strip0);
}

// Calls with more than 8 rows (and slices of K of any call): the same product with both operands in LDS rings.  Such a call pulls two to three times
// the weights' bytes out of L2 as activation rows, every workgroup all of its rows once, and through registers a compute
// unit draws no more than 36 B per clock whatever is in flight (measured); copies from memory to LDS run at 59.
// Every wavefront owns a ring of D stages of one k-tile (its NS weight tiles and MT activation groups, 1 KB each), fills
// it by itself and reads it by itself: no barrier before the final reduction, and the wavefronts' rings together keep
// up to 150 KB of requests in flight per compute unit with no registers spent on them, so that more strips fit a
// workgroup.  The areas of the reduction are the rings themselves.
// Measured on 7B shapes (operands through registers -> rings), 40 rows: QKV 30.1 -> 29.2 us, gate/up 39.0 -> 38.0, Wo and
// down slices 17.3 -> 16.6 on average, LM head 60.7 -> 51.6; 64 rows: QKV 40.3 -> 37.5, gate/up 78.6 -> 53.9, LM head
// 108.7 -> 78.2.  Bound by the unit's vector memory path all the same: its returns are in order, so a row out of L2 waits
// for the weights requested before it.
constexpr int kRingWaves = 4;  // (eight wavefronts with two stages each: 3 to 5 % slower in every product)
constexpr int kRingFixTiles = 64;  // k-tiles a wavefront of a product on coded weights may have: their fix words wait in LDS
constexpr int ring_stages(int waves, int stage) { return waves * stage * 3 <= 156 * 1024 ? 3 : (waves * stage * 2 <= 156 * 1024 ? 2 : 1); }
// on coded weights two where a stage is large (three: 1 to 4 % slower), more where two would hold too little
constexpr int coded_ring_stages(int stage) { return stage >= 5 * 1024 ? 2 : (stage >= 4 * 1024 ? 3 : 4); }

template <int MT, int EPI, int WAVES, int NB, bool Z>
__global__ __launch_bounds__(WAVES * 64) void gemm_rows_kernel(Params p, GemmArgs a) {
  constexpr int PER = (EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE) ? 2 : 1;
  constexpr int NS = NB * PER, T = NS + MT;
  constexpr int TILE = Z ? kCodedTile : 1024, STAGE = NS * TILE + MT * 1024;  // bytes
  constexpr int D = Z ? coded_ring_stages(STAGE) : ring_stages(WAVES, STAGE);
  __shared__ u32x4 ring[WAVES * D * STAGE / 16];
  __shared__ uint32_t fixes[Z ? WAVES : 1][Z ? NS : 1][Z ? 2 * kRingFixTiles : 1];  // fix words of the wavefront's k-tiles
  __shared__ __align__(16) float red_ss[WAVES][MT * 8];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KT = a.K >> 5;                                        // k-tiles of the whole K (strip stride)
  const int kbase = (EPI == EPI_PARTIAL) ? blockIdx.y * a.kt_split : 0;     // first k-tile this workgroup walks
  const int KTl = (EPI == EPI_PARTIAL) ? min(a.kt_split, KT - kbase) : KT;  // how many (the last slice may hold fewer)
  const int strip0 = blockIdx.x * NS;

  // strips past the end repeat the last one (in bounds; their results are dropped).  Rows >= M of the last group hold
  // whatever the buffer holds: a column of the product depends on its own row only, and those columns are dropped.
  const char *wp[NS];
  const u32x4 *xp[MT];
#pragma unroll
  for (int s = 0; s < NS; ++s) 
    wp[s] = (const char *)(Z ? a.z.tiles : a.W) + ((size_t)min(strip0 + s, a.n_strips - 1) * KT + kbase + wave) * TILE + min(lane, TILE / 16 - 1) * 16;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) xp[mt] = (const u32x4 *)a.X + ((size_t)mt * KT + kbase + wave) * 64 + lane;
  const int xr = MT == 1 ? p.xr : 8;  // (one group: the rows that are not there have no place in memory, theirs in LDS holds anything)
  const char *x1 = (const char *)a.X + (size_t)(kbase + wave) * (xr * 128) + x_lane(lane, xr);
  char *mine = (char *)ring + wave * (D * STAGE);

  // The sums lose as little as with eight wavefronts or more sharing K: either two accumulators per tile, one of the
  // wavefront's even and one of its odd k-tiles, or, where the registers do not hold those, a product of one k-tile at a
  // time that is added to the sum as a whole (a matrix instruction rounds its accumulator four times, an addition once).
  // K = 4096, error of the sums relative to the result: 1.3e-7 and 1.2e-7; with one accumulator 1.9e-7, in 1 % less time at 40
  // rows (gate/up 37.5 us against 38.0) and 14 % less at 64 (46.2 against 53.9).
  constexpr bool PAIRS = NS * MT <= 30;
  floatx4 acc[NS][MT], odd[PAIRS ? NS : 1][PAIRS ? MT : 1];
  float sum[PAIRS ? 1 : NS][PAIRS ? 1 : MT][4];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if constexpr (PAIRS) acc[s][mt] = odd[s][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
      else
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[s][mt][r] = 0.f;
    }

  // this wavefront's k-tiles: wave, wave + WAVES, ...  (the workgroup walks its strips front to back)
  const int n = (KTl - wave + WAVES - 1) / WAVES;
  auto issue = [&](int i, char *st) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if constexpr (MT > 1) copy_to_lds<false>(xp[mt] + (size_t)i * WAVES * 64, st + NS * TILE + mt * 1024);
      else if ((lane & 7) < xr) copy_to_lds<false>(x1 + (size_t)i * WAVES * (xr * 128), st + NS * TILE);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!Z || lane < kCodedTile / 16) copy_to_lds<true>(wp[s] + (size_t)i * WAVES * TILE, st + s * TILE);
    }
  };
  if constexpr (Z) {  // the run of n fix words of every strip, ahead of the first stage
    const int f0 = fix_index(KT, kbase + wave);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t *fp = (const uint32_t *)(a.z.fix + (size_t)min(strip0 + s, a.n_strips - 1) * fix_stride(KT) + f0);
#pragma unroll
      for (int h = 0; h < 2 * kRingFixTiles; h += 64)
        if (h < 2 * n) copy1_to_lds(fp + min(h + lane, 2 * n - 1), &fixes[wave][s][h]);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < n) issue(d, mine + d * STAGE);
  int at = 0;
  uint32_t marks = 0;
  auto tile = [&](int i, auto &into) __attribute__((always_inline)) {
    char *st = mine + at * STAGE;
    const int left = n - 1 - i;  // stages requested after this one: min(left, D - 1)
    if (left >= D - 1) wait_copies<(D - 1) * T>();
    else if (D > 3 && left == 2) wait_copies<(D > 3 ? 2 * T : 0)>();
    else if (D > 2 && left == 1) wait_copies<(D > 2 ? T : 0)>();
    else wait_copies<0>();
    u32x4 av[NS], bv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) bv[mt] = ((const u32x4 *)(st + NS * TILE + mt * 1024))[lane];
    typename LaneTile<Z>::T cv[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (Z) {
        cv[s] = *(const u32x3 *)(st + s * TILE + lane * 12);
      } else {
        cv[s] = ((const u32x4 *)(st + s * TILE))[lane];
      }
    }
    if (i + D < n) {
      wait_lds_reads();  // the stage has been read: it can be filled again
      issue(i + D, st);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (Z) {
      if (i == 0) {  // the fix words came ahead of the first stage: lane j learns which strips of the wavefront's j-th k-tile have any
#pragma unroll
        for (int s = 0; s < NS; ++s) marks |= (fixes[wave][s][2 * min(lane, n - 1)] ? 1u : 0u) << s;
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) av[s] = decode_tile(cv[s], a.z.lut0, a.z.lut1);
      const uint32_t mark = (uint32_t)__builtin_amdgcn_readlane((int)marks, i);
      if (__builtin_expect(mark != 0, 0)) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (mark >> s & 1)
            fix_tile(av[s], __builtin_amdgcn_readfirstlane(fixes[wave][s][2 * i]), __builtin_amdgcn_readfirstlane(fixes[wave][s][2 * i + 1]), a.z.more, lane);
      }
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) av[s] = cv[s];
    }
    auto product = [&](int s, int mt, floatx4 c) __attribute__((always_inline)) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[s]), __builtin_bit_cast(bf16x8, bv[mt]), c, 0, 0, 0);
    };
    if constexpr (PAIRS) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) into[s][mt] = product(s, mt, into[s][mt]);
    } else {
      floatx4 y[2][MT];
#pragma unroll
      for (int s = 0; s <= NS; ++s) {  // a strip's products, beside the additions of the strip before
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          if (s < NS) y[s & 1][mt] = product(s < NS ? s : 0, mt, floatx4{0.f, 0.f, 0.f, 0.f});
          if (s > 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) into[s - 1][mt][r] += y[(s - 1) & 1][mt][r];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    at = at + 1 == D ? 0 : at + 1;
  };
  if constexpr (PAIRS) {
    int i = 0;
    for (; i + 1 < n; i += 2) {
      tile(i, acc);
      tile(i + 1, odd);
    }
    if (i < n) tile(i, acc);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[s][mt] += odd[s][mt];
  } else {
    for (int i = 0; i < n; ++i) tile(i, sum);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[s][mt] = floatx4{sum[s][mt][0], sum[s][mt][1], sum[s][mt][2], sum[s][mt][3]};
  }
  constexpr int MB = D * STAGE / (NS * 1024) < MT ? D * STAGE / (NS * 1024) : MT;  // row groups whose partial tiles fit a wavefront's ring
  Epilogue<MT, EPI, WAVES, NB, NS, MB> epilogue;
  epilogue.ask(p, a, strip0);
  epilogue.finish(p, a, acc, (floatx4 *)ring, D * STAGE / 16, red_ss, strip0);
}

// Launch shape of the decode-sized GEMMs: GemmTuning (a member of the context, so two contexts
// never share a setting).  Defaults chosen by sweeping the benchmark on MI355X.
GemmTuning::GemmTuning()
    : waves{0, 0, 0, 0, 0},        // QKV, Wo, gate/up, LM head, down; 0 = by the count of blocks (few_rows_shape)
      unroll{1, 1, 1, 1, 1},
      big_blocks{0, 0, 0, 0, 0},   // 0 = by the count of blocks (ring_shape)
      split_ks(-1) {}              // -1 = by the rows (launch_resid_split)

int GemmTuning::set(int kind, int w, int u) {
  if (kind < 0 || kind > 4) return -1;
  if (w != 4 && w != 8 && w != 16) return -1;
  if (u != 1 && u != 2 && u != 4) return -1;
  waves[kind] = w;
  unroll[kind] = u;
  return 0;
}

int GemmTuning::set_big(int kind, int w, int blocks) {  // (the wavefronts are fixed: kRingWaves)
  if (kind < 0 || kind > 4) return -1;
  if (w != 4 && w != 8 && w != 16) return -1;
  if (blocks < 0 || blocks > 8) return -1;
  big_blocks[kind] = blocks;
  return 0;
}

int GemmTuning::set_split(int ks) {
  if (ks < 0 || ks > 8) return -1;
  split_ks = ks;
  return 0;
}

// Launch shape of a call of up to 8 rows: output blocks per workgroup, wavefronts, k-tiles per trip.  A compute unit should
// own as many blocks as any other and share the activation tile between them, with some 24 weight tiles or more requested
// at a time; where the blocks do not divide evenly among the 256 units, smaller workgroups even it out.
struct FewShape { int w, u, nb; };
static FewShape few_rows_shape(int epi, int n) {
  switch (epi) {
    case EPI_QKV:  // one workgroup a unit, or two (d 5120: 960 strips, four a workgroup 25.8 us, one in workgroups of 4
                   // wavefronts 31.3; 4096: 17.7 and, of 8, 20.4; 2048: 7.2 and 7.9; 1024: 4.5 and 5.2)
      if (n <= 256) return {8, 2, 1};
      if (n <= 512) return {4, 2, 2};
      if (n <= 768) return {8, 2, 3};
      if (n <= 1024) return {8, 1, 4};
      return {n % 256 ? 4 : 8, 1, 1};  // two rounds and more: one strip as ever (d 6144, 1152 strips, 46.6 us; three a workgroup 40.3)
    case EPI_GATEUP:
    case EPI_GATEUP_SAVE:  // (against one pair and one tile a trip in workgroups of 4, us: d 1024, 172 pairs 4.7 and 5.1; 2048, 344 9.8
                           // and 10.3, 448 11.4 both; 3072, 440 15.8 both; 4096, 588 25.5 and 30.8; 5120, 860 43.7 and 49.4, 1120 59.6 and
                           // 61.2; 8192, 1792 137 and 142)
      if (n <= 256) return {4, 2, 1};
      if (n <= 384) return {4, 1, 2};
      if (n <= 512) return {4, 1, 1};
      if (n <= 768) return {8, 1, 3};
      if (n <= 1024) return {8, 1, 4};
      return {8, 2, 1};
    case EPI_LOGITS:  // many rounds: two strips share the activation tile (V 32000: 41.3 us, one strip of 16 wavefronts 47.0; d 5120 51.4
                      // and 58.2; d 1024, V 2000, 125 strips, one a workgroup of 8: 3.7 and 3.8)
      return n <= 256 ? FewShape{8, 2, 1} : FewShape{4, 2, 2};
    default:  // Wo and down: 16 features a workgroup while there are units for them (d 4096: Wo 8.2 us, 16 wavefronts 8.7; 2048:
              // 5.0 and, of 8 with one tile a trip, 5.1), two strips beyond (d 5120, 320 strips: Wo 12.6 us, one strip 15.8; d 8192, 512: 25.6 and 25.1)
      return n <= 256 ? FewShape{8, 4, 1} : FewShape{16, 1, 2};
  }
}
// Whether a product of the ring form gains by coded weights.  Small ones only wait longer for their first tile (Wo d 2048 at 16 rows
// 6.5 us, coded 7.1; QKV 8.2 and 8.7; but Wo d 4096 12.6 and 10.5).
static bool coded_pays(int n_strips, int K) { return (int64_t)n_strips * 16 * K >= 1 << 24; }
// What a strip costs it, a plain one being 1, with that many weights of a tile outside the table: its four wavefronts put those in one by one, and
// beyond 0.16 of a tile the plain matrix is faster (gate/up d 4096, us, plain and coded: 16 rows 31.0, with 0.04 outside 25.8, 0.14 28.0, 0.3 33.7,
// 0.55 42.9; 40 rows 37.0, 33.6, 36.2, 41.9, 50.9).
static float coded_strip(float outside) { return 0.75f + 2.0f * std::max(0.0f, outside - 0.04f); }
// Slices of K of Wo and down in calls of up to 8 rows, and strips per workgroup; 1 = whole K.  Fewer strips than units leave
// units idle, 257 to 511 strips give some of them two: then the product is bound by those, and slices over all of them pay for
// the kernel that adds their sums.  In us, fitted to d 1024 .. 5120 (K up to 3.5 d): a unit takes 0.033 us per KB of weights and 0.010
// per KB of activation tile, the chip 6.9 TB/s, both kernels together 5.2.  The choice is within 9 % of the fastest there, within 6 % at
// d 6656 and 8192; d 6144 (384 strips) stays whole where two slices of three strips would take 10 % less (one K in six 21 %).
// d 5120, K 13760: 38.0 us whole in one strip a workgroup, 28 in two, 25.6 in slices; d 2048, K 5504: 9.4 and 8.1.
// On coded weights a strip takes 0.027 a KB and the start and end of both kernels 7.3 (5 rows, whole and in slices: d 3072, K 8192 10.8 and 13.5,
// 10752 15.0 and 15.8; d 4096, 8192 12.3 and 16.4, 14336 18.6 and 21.6; d 5120, 5120 13.2 and 14.2, 10240 21.8 and 20.5, 13824 28.0 and 24.5;
// d 6144, 6144 15.1 and 17.2, 16384 33.1 and 31.1; d 8192, 8192 20.2 and 24.1, 22016 55.4 and 51.0).
static int few_rows_slices(int n, int K, int d, int F, bool coded, bool slices_coded, int &nb_best) {
  const int KT = K / 32;
  float whole = n <= 256 ? 2.8f + K * (1.1e-3f + 0.7e-6f * n) : 3.0f + ((n + 1) / 2 + 255) / 256 * K * 1.97e-3f;
  if (coded) whole = n <= 256 ? 2.8f + K * (0.8e-3f + 1.3e-6f * n) : 3.0f + ((n + 1) / 2 + 255) / 256 * K * 1.73e-3f;
  float best = 0.95f * whole;
  int ks_best = 1;
  for (int ks = 2; ks <= 8; ++ks) {
    const int kts = (KT + ks - 1) / ks;
    if ((KT + kts - 1) / kts != ks || kts < 8) continue;
    if ((size_t)ks * d > (size_t)2 * F) continue;  // the slices' sums borrow the generic path's gate/up workspace
    for (int nb : {1, 2, 3, 4, 5, 6, 8}) {
      const float rounds = ((n + nb - 1) / nb * ks + 255) / 256;
      const float us = slices_coded ? 7.3f + std::max(rounds * (nb * 0.027f + 0.0125f) * kts, (float)n * K * 24 / 6.9e6f)
                                    : 5.2f + std::max(rounds * (nb * 0.033f + 0.010f) * kts, (float)n * K * 32 / 6.9e6f);
      if (us < best) { best = us; ks_best = ks; nb_best = nb; }
    }
  }
  return ks_best;
}
// The same on coded weights: eight wavefronts, and blocks by the rounds of 256 workgroups times what a workgroup takes in per k-tile,
// three quarters of a tile per strip and the activation tile.  Residual products as above.  (Measured against the plain tiles in
// their best shape, us: QKV d 2048 7.2 and 7.3, 4096 14.9 and 17.7, 5120 21.1 and 25.8; gate/up d 2048, 344 blocks, two a workgroup
// 9.3 and 9.9, 4096, 688, three 23.8 and 29.1, 5120, 860, four 35.1 and 43.5, 1120, three 49.9 and 59.6; LM head V 32000, four, d 1024 10.3
// and 12.3, 4096 31.7 and 41.4, V 24000, two, 26.2 and 31.8; Wo d 4096 6.9 and 8.1, 5120 11.9 and 12.6; down K 11008 15.3 and
// 17.5: their four k-tiles a trip take 2 % less than two.)
static int coded_blocks(int n, int per) {
  int best = 1;
  auto cost = [&](int nb) { return ((n + nb - 1) / nb + 255) / 256 * (3 * per * nb + 4); };
  for (int nb = 2; nb <= 4; ++nb)
    if (cost(nb) < cost(best)) best = nb;
  return best;
}
// whether a wavefront's lanes hold the fix words of all its k-tiles (64 of them) in the shapes of launch_coded
static bool coded_fits(int epi, int n_blocks, int K) { return (K >> 5) <= 64 * (epi == EPI_RESID && n_blocks > 256 ? 16 : 8); }
static bool few_rows_read_coded(const GemmTuning &tn, int kind, int epi, const Coded &z, int n_blocks, int K) {
  return !tn.waves[kind] && z.tiles && coded_fits(epi, n_blocks, K);  // (a launch shape that was asked for is one of the plain form)
}
template <int EPI>
static void launch_coded(const Params &p, const GemmArgs &a, int n_blocks, hipStream_t s) {
  auto go = [&](auto W, auto U, auto B) {
    constexpr int w = decltype(W)::value, u = decltype(U)::value, nb = decltype(B)::value;
    gemm_mfma_kernel<EPI, w, u, nb, true><<<(n_blocks + nb - 1) / nb, w * 64, 0, s>>>(p, a);
  };
  if constexpr (EPI == EPI_RESID) {
    if (n_blocks <= 256) go(nb_c<8>{}, nb_c<4>{}, nb_c<1>{});
    else go(nb_c<16>{}, nb_c<1>{}, nb_c<2>{});
  } else {
    constexpr int U = EPI == EPI_QKV ? 2 : 1;  // k-tiles a trip where a workgroup has two or three blocks
    switch (coded_blocks(n_blocks, EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE ? 2 : 1)) {
      case 1: go(nb_c<8>{}, nb_c<2>{}, nb_c<1>{}); break;
      case 2: go(nb_c<8>{}, nb_c<U>{}, nb_c<2>{}); break;
      case 3: go(nb_c<8>{}, nb_c<U>{}, nb_c<3>{}); break;
      default: go(nb_c<8>{}, nb_c<1>{}, nb_c<4>{}); break;
    }
  }
}
template <int EPI>
static void launch_few(const Params &p, const GemmArgs &a, int n_blocks, FewShape sh, hipStream_t s) {
  auto go = [&](auto W, auto U, auto B) {
    constexpr int w = decltype(W)::value, u = decltype(U)::value, nb = decltype(B)::value;
    gemm_mfma_kernel<EPI, w, u, nb, false><<<(n_blocks + nb - 1) / nb, w * 64, 0, s>>>(p, a);
  };
  constexpr bool GU = (EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE);
  const int key = sh.w * 100 + sh.u * 10 + sh.nb;
  if constexpr (EPI == EPI_QKV) {
    if (key == 422) return go(nb_c<4>{}, nb_c<2>{}, nb_c<2>{});
    if (key == 823) return go(nb_c<8>{}, nb_c<2>{}, nb_c<3>{});
    if (key == 814) return go(nb_c<8>{}, nb_c<1>{}, nb_c<4>{});
  } else if constexpr (GU) {
    if (key == 412) return go(nb_c<4>{}, nb_c<1>{}, nb_c<2>{});
    if (key == 813) return go(nb_c<8>{}, nb_c<1>{}, nb_c<3>{});
    if (key == 814) return go(nb_c<8>{}, nb_c<1>{}, nb_c<4>{});
  } else if constexpr (EPI == EPI_LOGITS) {
    if (key == 422) return go(nb_c<4>{}, nb_c<2>{}, nb_c<2>{});
  } else {
    if (key == 1612) return go(nb_c<16>{}, nb_c<1>{}, nb_c<2>{});
  }
  if constexpr (EPI == EPI_GATEUP_SAVE) {  // nobody asks for a launch shape of this one: those of few_rows_shape
    if (key == 411) return go(nb_c<4>{}, nb_c<1>{}, nb_c<1>{});
    if (key == 421) return go(nb_c<4>{}, nb_c<2>{}, nb_c<1>{});
    return go(nb_c<8>{}, nb_c<2>{}, nb_c<1>{});
  } else {
    switch (sh.w * 10 + sh.u) {
      case 161: return go(nb_c<16>{}, nb_c<1>{}, nb_c<1>{});
      case 162: return go(nb_c<16>{}, nb_c<2>{}, nb_c<1>{});
      case 164: return go(nb_c<16>{}, nb_c<4>{}, nb_c<1>{});
      case 81: return go(nb_c<8>{}, nb_c<1>{}, nb_c<1>{});
      case 82: return go(nb_c<8>{}, nb_c<2>{}, nb_c<1>{});
      case 84: return go(nb_c<8>{}, nb_c<4>{}, nb_c<1>{});
      case 41: return go(nb_c<4>{}, nb_c<1>{}, nb_c<1>{});
      case 42: return go(nb_c<4>{}, nb_c<2>{}, nb_c<1>{});
      default: return go(nb_c<4>{}, nb_c<4>{}, nb_c<1>{});
    }
  }
}

// Blocks a workgroup of the ring form may own: its sums (of the 512 registers that one wavefront per SIMD has) and two
// stages of its ring must fit.
constexpr int kRingCodedGroups = 6;  // row groups up to which the ring form takes coded weights
constexpr bool ring_fits(int strips, int mt) { return strips * mt <= 64 && kRingWaves * 2 * (strips + mt) <= 156; }

template <int MT, int EPI>
static void launch_rows_mt(const Params &p, const GemmArgs &a, dim3 grid, int nb, bool coded, hipStream_t s) {
  constexpr int PER = (EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE) ? 2 : 1;
  auto go = [&](auto B) {
    constexpr int NB = decltype(B)::value;
    if constexpr (ring_fits(NB * PER, MT)) {
      if constexpr (MT <= kRingCodedGroups && NB * PER * MT <= 30) {
        if (coded) return gemm_rows_kernel<MT, EPI, kRingWaves, NB, true><<<grid, kRingWaves * 64, 0, s>>>(p, a);
      }
      gemm_rows_kernel<MT, EPI, kRingWaves, NB, false><<<grid, kRingWaves * 64, 0, s>>>(p, a);
    }
  };
  switch (nb) {
    case 1: go(nb_c<1>{}); break;
    case 2: go(nb_c<2>{}); break;
    case 3: go(nb_c<3>{}); break;
    case 4: go(nb_c<4>{}); break;
    case 5: go(nb_c<5>{}); break;
    case 6: go(nb_c<6>{}); break;
    default: go(nb_c<8>{}); break;
  }
}
// Blocks per workgroup (1 .. 6 or 8), and whether the product reads coded weights.  A workgroup pulls all M rows whatever it owns, and a
// compute unit holds one: the product takes (rounds of 256 workgroups) x (operand tiles per k-tile).  Products added step by step (sums
// past 30 tiles) cost a quarter more, and with the decoding beside them too much.  On coded weights a strip is three quarters of a tile, and
// a second round costs a quarter more unless two workgroups fit a unit's LDS (gate/up an eighth).  Against a plain product added step by step, which
// owns eight strips a workgroup, coded strips in two rounds lose that gain with K (k-tiles: of a workgroup).  `want` > 0 asks for a number.
// Measured without and with the copies, us: 40 rows, d 4096, QKV 26.0 and 23.8, gate/up (688 blocks) 36.1 and 33.7, Wo 15.4 and 14.7, down
// 25.1 and 23.6 (with the kernel that adds the slices); 16 rows 19.2 and 17.1, 30.7 and 25.6, 12.6 and
// 10.5, 19.3 and 18.2, 46.4 and 35.7; d 5120, 24 rows, 860 blocks 47.8 and 42.5; 48 rows, d 4096, QKV 28.3 and 26.3.  LM head, V 32000, eight strips
// plain and four coded: 32 rows, d 1024 20.0 and 19.9, 2048 31.9 and 27.7, 3072 37.2 and 37.3, 4096 49.4 and 47.7, 5120 59.3 and 60.7, 6144 69.8 and
// 71.4, 8192 88.7 and 92.5; 40 rows 22.2 and 21.9, 33.2 and 30.7, 40.2 and 42.0, 53.0 and 54.2, 62.5 and 67.8, 74.4 and 78.1, 94.2 and 101.5.
struct RingShape { int nb; bool coded; };
static RingShape ring_shape(int want, int n_blocks, int per, int mt, int slices, int kts, bool coded, float outside) {
  const float strip = coded_strip(outside);
  RingShape best{1, false};
  float best_cost = 1e30f;
  float rounds_lose = 1;
  for (int z = 0; z <= (coded ? 1 : 0); ++z) {
    if (z && best.nb * per * mt > 30) rounds_lose = kts <= 64 ? 1.0f : kts <= 128 ? 1.05f : 1.1f;
    for (int nb : {1, 2, 3, 4, 5, 6, 8}) {
      const int ns = nb * per, rounds = ((n_blocks + nb - 1) / nb * slices + 255) / 256;
      if (!ring_fits(ns, mt) || (z && ns * mt > 30)) continue;
      float cost = rounds * ((z ? strip : 1.0f) * ns + mt);
      if (ns * mt > 30) cost *= 1.28f;
      if (z && rounds > 1) cost *= 8 * (0.75f * ns + mt) + 2 * ns > 79 ? 1.25f : per == 2 ? 1.12f : rounds_lose;
      if (want) cost = (float)std::abs(nb - want) + (coded && z == (strip > 1) ? 0.5f : 0.0f);  // the nearest, in the cheaper form
      if (cost < best_cost) { best_cost = cost; best = RingShape{nb, z != 0}; }
    }
  }
  return best;
}
// kts: k-tiles of a workgroup
static RingShape rows_shape(const Coded &z, int M, int n_blocks, int per, int K, int kts, int want, int slices) {
  const int mt = (M + 7) / 8;
  const bool coded = z.tiles && mt <= kRingCodedGroups && coded_pays(n_blocks * per, K) && kts <= kRingFixTiles * kRingWaves;
  return ring_shape(want, n_blocks, per, mt, slices, kts, coded, z.outside);
}
template <int EPI>
static void launch_rows(const Params &p, const GemmArgs &a, int n_blocks, int want, int slices, hipStream_t s) {
  constexpr int PER = (EPI == EPI_GATEUP || EPI == EPI_GATEUP_SAVE) ? 2 : 1;
  const int mt = (a.M + 7) / 8;
  const auto [nb, z] = rows_shape(a.z, a.M, n_blocks, PER, a.K, EPI == EPI_PARTIAL ? a.kt_split : a.K >> 5, want, slices);
  const dim3 grid((n_blocks + nb - 1) / nb, slices);
  switch (mt) {
    case 1: if constexpr (EPI == EPI_PARTIAL) launch_rows_mt<1, EPI>(p, a, grid, nb, z, s); break;
    case 2: launch_rows_mt<2, EPI>(p, a, grid, nb, z, s); break;
    case 3: launch_rows_mt<3, EPI>(p, a, grid, nb, z, s); break;
    case 4: launch_rows_mt<4, EPI>(p, a, grid, nb, z, s); break;
    case 5: launch_rows_mt<5, EPI>(p, a, grid, nb, z, s); break;
    case 6: launch_rows_mt<6, EPI>(p, a, grid, nb, z, s); break;
    case 7: launch_rows_mt<7, EPI>(p, a, grid, nb, z, s); break;
    default: launch_rows_mt<8, EPI>(p, a, grid, nb, z, s); break;
  }
}

template <int EPI>
static void launch_gemm_epi(const Params &p, const GemmTuning &tn, const GemmArgs &a, int n_strips, hipStream_t s,
                            int kind = EPI) {
  constexpr int PER = (EPI == EPI_GATEUP) ? 2 : 1;
  const int n_blocks = n_strips / PER;
  if (a.M <= 8) {
    if (few_rows_read_coded(tn, kind, EPI, a.z, n_blocks, a.K)) return launch_coded<EPI>(p, a, n_blocks, s);
    return launch_few<EPI>(p, a, n_blocks, tn.waves[kind] ? FewShape{tn.waves[kind], tn.unroll[kind], 1} : few_rows_shape(EPI, n_blocks), s);
  }
  launch_rows<EPI>(p, a, n_blocks, tn.big_blocks[kind], 1, s);
}

// ---------------------------------------------------------------------------------------------
// Residual projections (Wo, down) in slices of K.  Calls with more than 8 rows: N = d gives only d/16 strips,
// one per compute unit at best, and every workgroup would have to pull all M activation rows
// through its L1: that traffic, not HBM, bounds the kernel.  So K is cut into KS slices across
// workgroups that own that many times the strips (7B: 4 slices, 4 strips; 8 and 8 took 23.2 us for down where
// these take 22.0, 2 and 2 took 27.7).  Calls of up to 8 rows: where the strips alone leave units idle (few_rows_slices).  The slices'
// sums go to a workspace and this kernel adds them in slice order (deterministic), then does what
// the fused epilogue does: residual add into h, (hi, lo) of h * gain of the next norm, per-strip
// partial sums of h^2.  One workgroup per strip of 16 features: thread = (row, 4 features).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void resid_reduce_kernel(Params p, const float *partial, int KS, int M,
                                                           const uint16_t *gain_next) {
  const int strip = blockIdx.x, m = threadIdx.x >> 2, n = strip * 16 + (threadIdx.x & 3) * 4;
  float ss = 0.f;
  if (m < M) {
    const size_t at = (size_t)m * p.d + n;
    floatx4 hv = *(const floatx4 *)(p.h + at);
    floatx4 part[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)  // all slices requested at once (index clamped, surplus dropped)
      part[ks] = *(const floatx4 *)(partial + ((size_t)min(ks, KS - 1) * kMaxRows + m) * p.d + n);
    floatx4 y = part[0];
#pragma unroll
    for (int ks = 1; ks < 8; ++ks)
      if (ks < KS) y += part[ks];
    hv += y;
    *(floatx4 *)(p.h_out + at) = hv;
    float t[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      t[r] = hv[r] * bf16_to_f32(gain_next[n + r]);
      ss += hv[r] * hv[r];
    }
    store_split4(p.xg, m, p.d, n, t, p.xr);
  }
  ss += __shfl_xor(ss, 1);
  ss += __shfl_xor(ss, 2);
  if ((threadIdx.x & 3) == 0) p.ssq[(size_t)strip * kMaxRows + m] = ss;  // rows >= M get 0
}

// Slices of K of a residual product (1: whole), k-tiles of a slice, strips per workgroup (0: by cost)
struct ResidSlices { int ks, kts, nb; };
static ResidSlices resid_slices(const Params &p, const GemmTuning &tn, int kind, const Coded &z, int M, int K) {
  const int n_strips = p.d / 16, KT = K >> 5;
  int KS = tn.split_ks, nb = tn.big_blocks[kind];
  if (KS < 0 && M > 8) KS = 4;
  if (KS < 0 && tn.waves[kind]) KS = 1;  // a launch shape of the whole product was asked for
  if (KS < 0) {
    int best = 0;
    const bool coded = z.tiles && coded_fits(EPI_RESID, n_strips, K);
    KS = few_rows_slices(n_strips, K, p.d, p.F, coded, coded && coded_pays(n_strips, K) && coded_strip(z.outside) <= 1, best);
    if (!nb) nb = best;
  }
  if (KS < 2) return {1, KT, nb};
  // K need not divide evenly, the last slice holds what is left (40 rows, down of d 4096, K 9408, 294 k-tiles: 22.5 us in
  // slices of 74, 74, 74 and 72, 31.7 whole; d 5120, K 13760: 32.9 and 56.1)
  const int kts = (KT + KS - 1) / KS;
  KS = (KT + kts - 1) / kts;
  if (KS < 2 || (size_t)KS * p.d > (size_t)2 * p.F) return {1, KT, nb};  // the slices' sums borrow the generic path's gate/up workspace
  return {KS, kts, nb};
}
static bool launch_resid_split(const Params &p, const GemmTuning &tn, const GemmArgs &a0, int kind, hipStream_t s) {
  const ResidSlices sl = resid_slices(p, tn, kind, a0.z, a0.M, a0.K);
  if (sl.ks < 2) return false;
  GemmArgs a = a0;
  a.kt_split = sl.kts;
  a.partial = p.gu;
  a.ldy = p.d;
  launch_rows<EPI_PARTIAL>(p, a, p.d / 16, sl.nb, sl.ks, s);
  resid_reduce_kernel<<<p.d / 16, 256, 0, s>>>(p, a.partial, sl.ks, a.M, a.gain_next);
  return true;
}
static int resid_kind(const Params &p, int K) { return K == p.F ? 4 : 1; }  // the down projection has its own shape

void launch_gemm_qkv(const Params &p, const GemmTuning &tn, const Matrix &W, int layer, int M, hipStream_t s) {
  GemmArgs a{(const u32x4 *)W.tiles, p.xg, M, p.d, layer, nullptr, nullptr, 0, nullptr, 3 * p.D / 16, 0, nullptr, W.coded};
  launch_gemm_epi<EPI_QKV>(p, tn, a, 3 * p.D / 16, s);
}
void launch_gemm_resid(const Params &p, const GemmTuning &tn, const Matrix &W, const uint16_t *X, int K,
                       const void *gain_next, int M, hipStream_t s) {
  GemmArgs a{(const u32x4 *)W.tiles, X, M, K, 0, (const uint16_t *)gain_next, nullptr, 0, nullptr, p.d / 16, 0, nullptr, W.coded};
  if (launch_resid_split(p, tn, a, resid_kind(p, K), s)) return;
  launch_gemm_epi<EPI_RESID>(p, tn, a, p.d / 16, s, resid_kind(p, K));
}
void launch_gemm_gateup(const Params &p, const GemmTuning &tn, const Matrix &W, int M, hipStream_t s) {
  GemmArgs a{(const u32x4 *)W.tiles, p.xg, M, p.d, 0, nullptr, nullptr, 0, nullptr, 2 * p.F / 16, 0, nullptr, W.coded};
  launch_gemm_epi<EPI_GATEUP>(p, tn, a, 2 * p.F / 16, s);
}
void launch_gemm_logits(const Params &p, const GemmTuning &tn, const Matrix &W, float *logits, int M, hipStream_t s) {
  GemmArgs a{(const u32x4 *)W.tiles, p.xg, M, p.d, 0, nullptr, logits, 0, nullptr, p.V / 16, 0, nullptr, W.coded};
  launch_gemm_epi<EPI_LOGITS>(p, tn, a, p.V / 16, s);
}

bool gemm_reads_coded(const Params &p, const GemmTuning &tn, int kind, const Coded &z, int M) {
  const bool resid = kind == 1 || kind == 4;
  const int K = kind == 1 ? p.D : kind == 4 ? p.F : p.d, per = kind == 2 ? 2 : 1;
  const int n_blocks = (kind == 0 ? 3 * p.D : kind == 2 ? p.F : kind == 3 ? p.V : p.d) / 16;
  if (resid) {
    const ResidSlices sl = resid_slices(p, tn, resid_kind(p, K), z, M, K);
    if (sl.ks > 1) return rows_shape(z, M, n_blocks, 1, K, sl.kts, sl.nb, sl.ks).coded;
    kind = resid_kind(p, K);
  }
  if (M <= 8) return few_rows_read_coded(tn, kind, resid ? EPI_RESID : EPI_QKV, z, n_blocks, K);
  return rows_shape(z, M, n_blocks, per, K, K >> 5, tn.big_blocks[kind], 1).coded;
}


// ---------------------------------------------------------------------------------------------
// What the training of the look-ahead embeddings adds (kernels_train.hip has the rest).
// ---------------------------------------------------------------------------------------------
// The gate/up GEMM that also keeps gate | up before the activation, in the decode call's launch shapes.
void launch_gemm_gateup_save(const Params &p, const Matrix &W, float *gu_save, int M, hipStream_t s) {
  GemmArgs a{(const u32x4 *)W.tiles, p.xg, M, p.d, 0, nullptr, nullptr, 0, nullptr, 2 * p.F / 16, 0, gu_save, W.coded};
  const int n_blocks = p.F / 16;
  if (M <= 8 && a.z.tiles && coded_fits(EPI_GATEUP_SAVE, n_blocks, a.K)) launch_coded<EPI_GATEUP_SAVE>(p, a, n_blocks, s);
  else if (M <= 8) launch_few<EPI_GATEUP_SAVE>(p, a, n_blocks, few_rows_shape(EPI_GATEUP_SAVE, n_blocks), s);
  else launch_rows<EPI_GATEUP_SAVE>(p, a, n_blocks, 0, 1, s);
}

// Plain product Y = X W^T on packed tiles: X as (hi, lo) tiles of K features, W packed [N][K], Y fp32.
// K is cut into KS slices across workgroups (the last one may be shorter); slice ks leaves its
// sums in part[ks][kMaxRows][N] and the consumer adds the slices in order.  Needs N % 64 == 0; returns the KS it
// used (plain_gemm_slices: what the consumer must add up).
int plain_gemm_slices(int N, int K) {
  const int KT = K / 32, wgs = N / 64;
  int best = 1;
  for (int ks = 1; ks <= 8; ks *= 2) {
    if (KT / ks < 8) break;
    best = ks;
    if (wgs * ks >= 256) break;  // one workgroup per compute unit: each pulls its slice of the rows once
  }
  const int kts = (KT + best - 1) / best;
  return (KT + kts - 1) / kts;  // every slice holds something
}
bool gemm_plain_reads_coded(const Coded &z, int M, int N, int K) {
  const int KT = K / 32, KS = plain_gemm_slices(N, K);
  return rows_shape(z, M, N / 16, 1, K, (KT + KS - 1) / KS, 0, KS).coded;
}
int launch_gemm_plain(const Params &p, const Matrix &W, const uint16_t *X, int M, int N, int K, float *part, hipStream_t s) {
  const int KT = K / 32, KS = plain_gemm_slices(N, K);
  GemmArgs a{(const u32x4 *)W.tiles, X, M, K, 0, nullptr, nullptr, (KT + KS - 1) / KS, part, N / 16, N, nullptr, W.coded};
  launch_rows<EPI_PARTIAL>(p, a, N / 16, 0, KS, s);
  return KS;
}

// Packed tiles of W [N][K] -> packed tiles of its transpose [K][N] (the backward pass multiplies by
// W^T with the same kernels).  One 16-byte chunk of the destination per thread: row k of W^T, eight
// consecutive n.  Run once when training is set up.
__global__ __launch_bounds__(256) void transpose_packed_kernel(const uint16_t *src, uint16_t *dst, int N, int K) {
  const int KT = K / 32, NT = N / 32;  // k-tiles of the source, of the destination
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x, total = (size_t)(K / 16) * NT * 64;
  if (idx >= total) return;
  const int lane = (int)(idx & 63);
  const size_t tile = idx >> 6;
  const int nt = (int)(tile % NT), ks = (int)(tile / NT);  // destination k-tile (over n), strip (over k)
  const int k = ks * 16 + (lane & 15), n0 = nt * 32 + (lane >> 4) * 8;
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int n = n0 + e;
    v[e] = src[((((size_t)(n >> 4) * KT + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (n & 15)) << 3) + (k & 7)];
  }
  uint4 o;
  o.x = v[0] | (uint32_t)v[1] << 16; o.y = v[2] | (uint32_t)v[3] << 16;
  o.z = v[4] | (uint32_t)v[5] << 16; o.w = v[6] | (uint32_t)v[7] << 16;
  *(uint4 *)(dst + idx * 8) = o;
}
void launch_transpose_packed(const void *src, void *dst, int N, int K, hipStream_t s) {
  const size_t total = (size_t)(K / 16) * (N / 32) * 64;
  transpose_packed_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const uint16_t *)src, (uint16_t *)dst, N, K);
}

}  // namespace pass
