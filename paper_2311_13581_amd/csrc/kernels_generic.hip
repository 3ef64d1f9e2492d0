// Generic kernels of the (1+k)-row decode step: any storage type, fp32 activations.
// They carry the fp32 configuration and any shape the matrix-core path does not take.
#include "pass_internal.h"

namespace pass {

// ---------------------------------------------------------------------------------------------
// Row assembly (Section 2.2.1: the look-ahead embeddings are appended after the sequence;
// Algorithm 1: drafting call on (x_n, [LA]_1..[LA]_k), validation call on (x_{n+1}, drafts)).
// Row m = b*R + r belongs to slot step_slots[b] at position kv_len[slot] + r.
// Also fills the rotary table of the step (angles in double: pos * base^(-2i/hd), the
// frequencies from the table made at create).
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void assemble_kernel(Params p, const T *tok_emb, const T *lookahead, int mode,
                                                       int R) {
  int m = blockIdx.x, b = m / R, r = m % R;
  int slot = p.step_slots[b];
  int pos = p.kv_len[slot] + r;
  if (m == 0 && threadIdx.x == 0 && mode != MODE_PREFILL) p.clock[mode == MODE_DRAFT ? 0 : 1] = wall_clock64();
  const bool dead = row_is_dead(p, mode, slot, R);
  const T *src;
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
  float *dst = p.h + (size_t)m * p.d;
  for (int i = threadIdx.x; i < p.d; i += blockDim.x) dst[i] = load_f(src, i);
  int half = p.hd / 2;
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    double sn, cs;
    sincos((double)pos * p.rope_theta[i], &sn, &cs);
    p.rope_cos[(size_t)m * half + i] = (float)cs;
    p.rope_sin[(size_t)m * half + i] = (float)sn;
  }
  if (threadIdx.x == 0) {
    p.row_pos[m] = dead ? 0 : pos;
    p.row_slot[m] = dead ? -1 : slot;
    p.row_out[m] = slot * (1 + p.k) + r;
  }
}

void launch_assemble(const Params &p, int dtype, const void *tok_emb, const void *lookahead, int mode, int B,
                     int R, hipStream_t s) {
  if (dtype == PASS_F32)
    assemble_kernel<float><<<B * R, 256, 0, s>>>(p, (const float *)tok_emb, (const float *)lookahead, mode, R);
  else
    assemble_kernel<bf16_t><<<B * R, 256, 0, s>>>(p, (const bf16_t *)tok_emb, (const bf16_t *)lookahead, mode, R);
}

// ---------------------------------------------------------------------------------------------
// RMSNorm: out = x * rsqrt(mean(x^2) + eps) * gain
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float *x, const T *gain, float *out, int d, float eps) {
  __shared__ float red[4];
  const float *xr = x + (size_t)blockIdx.x * d;
  float ss = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) ss += xr[i] * xr[i];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = red[0] + red[1] + red[2] + red[3];
  float inv = 1.0f / sqrtf(tot / (float)d + eps);
  float *o = out + (size_t)blockIdx.x * d;
  for (int i = threadIdx.x; i < d; i += 256) o[i] = xr[i] * inv * load_f(gain, i);
}

void launch_rmsnorm(const Params &p, int dtype, const float *x, const void *gain, float *out, int M, hipStream_t s) {
  if (dtype == PASS_F32)
    rmsnorm_kernel<float><<<M, 256, 0, s>>>(x, (const float *)gain, out, p.d, p.eps);
  else
    rmsnorm_kernel<bf16_t><<<M, 256, 0, s>>>(x, (const bf16_t *)gain, out, p.d, p.eps);
}

// ---------------------------------------------------------------------------------------------
// Skinny GEMM, generic: out[m][n] (+)= sum_k X[m][k] W[n][k].  One wavefront per output column,
// lanes stride over K in chunks of 8 elements (K % 8 == 0), rows in blocks of 8.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void load8(const float *w, float (&o)[8]) {
  float4 a = *(const float4 *)w, b = *(const float4 *)(w + 4);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t *w, float (&o)[8]) {
  uint4 v = *(const uint4 *)w;
  o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
  o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
  o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xffff0000u);
  o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xffff0000u);
}

template <typename T>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const float *X, const T *W, float *out, int M, int N,
                                                           int K, int ldc, const int32_t *rowmap, int accumulate) {
  constexpr int MB = 8;
  int lane = threadIdx.x & 63;
  int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  int n_waves = gridDim.x * 4;
  for (int n = wave; n < N; n += n_waves) {
    const T *wr = W + (size_t)n * K;
    for (int m0 = 0; m0 < M; m0 += MB) {
      int mr = min(MB, M - m0);
      float acc[MB];
#pragma unroll
      for (int i = 0; i < MB; ++i) acc[i] = 0.f;
      for (int k0 = lane * 8; k0 < K; k0 += 64 * 8) {
        float w[8];
        load8(wr + k0, w);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          if (i < mr) {
            float x[8];
            load8(X + (size_t)(m0 + i) * K + k0, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[i] = fmaf(w[e], x[e], acc[i]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) acc[i] = wave_sum(acc[i]);
      if (lane == 0) {
        for (int i = 0; i < mr; ++i) {
          int row = rowmap ? rowmap[m0 + i] : (m0 + i);
          float *o = out + (size_t)row * ldc + n;
          *o = accumulate ? (*o + acc[i]) : acc[i];
        }
      }
    }
  }
}

void launch_gemm_generic(int dtype, const float *X, const void *W, float *out, int M, int N, int K, int ldc,
                         const int32_t *rowmap, int accumulate, hipStream_t s) {
  int blocks = (N + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  if (dtype == PASS_F32)
    gemm_generic_kernel<float><<<blocks, 256, 0, s>>>(X, (const float *)W, out, M, N, K, ldc, rowmap, accumulate);
  else
    gemm_generic_kernel<bf16_t><<<blocks, 256, 0, s>>>(X, (const bf16_t *)W, out, M, N, K, ldc, rowmap, accumulate);
}

// ---------------------------------------------------------------------------------------------
// Rotary embedding on q and k (interleaved pairs), K/V rows written to the paged cache at the
// row's position.  q is rotated in place in the qkv workspace.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void rope_kv_kernel(Params p, int layer) {
  int m = blockIdx.x;
  int slot = p.row_slot[m], pos = p.row_pos[m];
  int half = p.hd / 2;
  float *q = p.qkv + (size_t)m * 3 * p.D;
  float *kk = q + p.D;
  float *vv = q + 2 * p.D;
  T *kpool = (T *)p.k_pool, *vpool = (T *)p.v_pool;
  for (int idx = threadIdx.x; idx < p.H * half; idx += blockDim.x) {
    int h = idx / half, i = idx % half;
    float cs = p.rope_cos[(size_t)m * half + i], sn = p.rope_sin[(size_t)m * half + i];
    int e = h * p.hd + 2 * i;
    float q0 = q[e], q1 = q[e + 1];
    q[e] = q0 * cs - q1 * sn;
    q[e + 1] = q0 * sn + q1 * cs;
    if (slot < 0) continue;  // a dead row (see row_is_dead) has no place in the cache
    float k0 = kk[e], k1 = kk[e + 1];
    size_t off = kv_offset(p, layer, slot, pos, h) + 2 * i;
    store_f(kpool, off, k0 * cs - k1 * sn);
    store_f(kpool, off + 1, k0 * sn + k1 * cs);
    store_f(vpool, off, vv[e]);
    store_f(vpool, off + 1, vv[e + 1]);
  }
}

void launch_rope_kv(const Params &p, int dtype, int layer, int M, hipStream_t s) {
  if (dtype == PASS_F32)
    rope_kv_kernel<float><<<M, 256, 0, s>>>(p, layer);
  else
    rope_kv_kernel<bf16_t><<<M, 256, 0, s>>>(p, layer);
}

// act = silu(gate) * up
__global__ __launch_bounds__(256) void silu_mul_kernel(const float *gu, float *act, int F) {
  int m = blockIdx.y;
  int f = blockIdx.x * 256 + threadIdx.x;
  if (f < F) {
    float g = gu[(size_t)m * 2 * F + f], u = gu[(size_t)m * 2 * F + F + f];
    float v = g / (1.0f + __expf(-g)) * u;
    act[(size_t)m * F + f] = v;
  }
}

void launch_silu_mul(const Params &p, int M, hipStream_t s) {
  dim3 grid((p.F + 255) / 256, M);
  silu_mul_kernel<<<grid, 256, 0, s>>>(p.gu, p.act, p.F);
}

// ---------------------------------------------------------------------------------------------
// The decode step's GEMMs with everything around them folded in (five kernels per layer instead of ten; a call of the
// tiny fp32 model is a chain of dependent launches of 2 to 5 us each and nothing else):
//   QKV     RMSNorm, rotary embedding, q to the workspace, K/V rows into the paged cache
//   RESID   residual add into h
//   GATEUP  RMSNorm, silu(gate) * up
//   LOGITS  RMSNorm, logits of row m into row rowmap[m]
// One wavefront per pair of output columns (a rotary pair; a gate column and its up column; two neighbours), lanes
// stride over K in chunks of VEC elements, MB rows at a time.  RMSNorm: the dot product runs over x * gain and is
// scaled by 1 / rms at the end, the sum of x^2 comes out of the same pass over the row (every wavefront reads all of
// every row anyway).  A row's arithmetic depends on the shape only, not on what shares its call.  Rows past the last one
// repeat it and are dropped, so that all loads are unconditional and leave together; what the epilogue needs is
// requested before the loop.  Measured on the tiny model (d 256, three rows),
// per call: 25 kernels and 104 us -> 13 and 50 us, with the attention merge of one split gone as well.
// ---------------------------------------------------------------------------------------------
enum { ROW_QKV = 0, ROW_RESID = 1, ROW_GATEUP = 2, ROW_LOGITS = 3 };

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}
// sum over the wavefront, in every lane
__device__ __forceinline__ float wave_total(float v) {
  v = dpp_add<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
  v = dpp_add<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  v = dpp_add<0x141, 0xF>(v);  // row_half_mirror
  v = dpp_add<0x140, 0xF>(v);  // row_mirror: every lane has its row of 16
  v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3: lane 63 has all
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
template <int VEC>
__device__ __forceinline__ void load_vec(const float *w, float (&o)[VEC]) {
#pragma unroll
  for (int i = 0; i < VEC; i += 4) {
    const float4 a = *(const float4 *)(w + i);
    o[i] = a.x; o[i + 1] = a.y; o[i + 2] = a.z; o[i + 3] = a.w;
  }
}
template <int VEC>
__device__ __forceinline__ void load_vec(const bf16_t *w, float (&o)[VEC]) {
#pragma unroll
  for (int i = 0; i < VEC; i += 4) {
    const uint2 a = *(const uint2 *)(w + i);
    o[i] = __uint_as_float(a.x << 16); o[i + 1] = __uint_as_float(a.x & 0xffff0000u);
    o[i + 2] = __uint_as_float(a.y << 16); o[i + 3] = __uint_as_float(a.y & 0xffff0000u);
  }
}

struct RowGemm {
  const float *X;       // [M][K]
  const void *W, *gain; // [N][K], [K] (RESID: unused)
  float *out;           // RESID: h, GATEUP: act, LOGITS: logits; QKV: the qkv workspace
  const int32_t *rowmap;
  int M, N, K, layer;   // N: output columns (GATEUP: gate and up together)
};

template <typename T, int EPI, int VEC, int MB>
__global__ __launch_bounds__(256) void row_gemm_kernel(Params p, RowGemm a) {
  constexpr bool NORM = (EPI != ROW_RESID);
  const int lane = threadIdx.x & 63;
  const int pr = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // pair of columns
  const int c0 = EPI == ROW_GATEUP ? pr : 2 * pr;
  const int n_pairs = (a.N + 1) / 2;
  if (pr >= n_pairs) return;
  const int c1 = EPI == ROW_GATEUP ? a.N / 2 + pr : min(2 * pr + 1, a.N - 1);
  const T *w0 = (const T *)a.W + (size_t)c0 * a.K, *w1 = (const T *)a.W + (size_t)c1 * a.K, *gn = (const T *)a.gain;
  for (int m0 = 0; m0 < a.M; m0 += MB) {
    const int mine = min(m0 + (lane < MB ? lane : 0), a.M - 1);  // the row this lane finishes
    // what the epilogue of that row needs
    int slot = 0, pos = 0, page = 0, orow = mine;
    float cs = 0.f, sn = 0.f, h0 = 0.f, h1 = 0.f;
    const int proj = EPI == ROW_QKV ? c0 / p.D : 0;       // 0 q, 1 k, 2 v
    const int col = c0 - proj * p.D;
    if constexpr (EPI == ROW_QKV) {
      const int half = p.hd / 2, i = (col % p.hd) >> 1;
      slot = p.row_slot[mine];
      pos = p.row_pos[mine];
      cs = p.rope_cos[(size_t)mine * half + i];
      sn = p.rope_sin[(size_t)mine * half + i];
      page = p.block_table[(size_t)max(slot, 0) * p.pages_per_seq + (pos >> p.page_shift)];
    } else if constexpr (EPI == ROW_RESID) {
      h0 = a.out[(size_t)mine * a.N + c0];
      h1 = a.out[(size_t)mine * a.N + c1];
    } else if constexpr (EPI == ROW_LOGITS) {
      orow = a.rowmap[mine];
    }
    float s0[MB], s1[MB], sq[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) s0[i] = s1[i] = sq[i] = 0.f;
    for (int k0 = lane * VEC; k0 < a.K; k0 += 64 * VEC) {
      float u[VEC], v[VEC], g[VEC], x[MB][VEC];
      load_vec<VEC>(w0 + k0, u);
      load_vec<VEC>(w1 + k0, v);
      if constexpr (NORM) load_vec<VEC>(gn + k0, g);
#pragma unroll
      for (int i = 0; i < MB; ++i) load_vec<VEC>(a.X + (size_t)min(m0 + i, a.M - 1) * a.K + k0, x[i]);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          float t = x[i][e];
          if constexpr (NORM) {
            sq[i] = fmaf(t, t, sq[i]);
            t *= g[e];
          }
          s0[i] = fmaf(u[e], t, s0[i]);
          s1[i] = fmaf(v[e], t, s1[i]);
        }
    }
    // lane i < MB ends with the two columns of row m0 + i
    float y0 = 0.f, y1 = 0.f, ss = 0.f;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const float t0 = wave_total(s0[i]), t1 = wave_total(s1[i]);
      y0 = lane == i ? t0 : y0;
      y1 = lane == i ? t1 : y1;
      if constexpr (NORM) {
        const float tq = wave_total(sq[i]);
        ss = lane == i ? tq : ss;
      }
    }
    if (lane >= MB || m0 + lane >= a.M) continue;
    if constexpr (NORM) {
      const float inv = 1.0f / sqrtf(ss / (float)a.K + p.eps);
      y0 *= inv;
      y1 *= inv;
    }
    if constexpr (EPI == ROW_QKV) {
      float *q = a.out + (size_t)mine * 3 * p.D;
      const float r0 = proj < 2 ? y0 * cs - y1 * sn : y0, r1 = proj < 2 ? y0 * sn + y1 * cs : y1;
      if (proj == 0) {
        *(float2 *)(q + col) = make_float2(r0, r1);
      } else if (slot >= 0) {  // a dead row (see row_is_dead) has no place in the cache
        const int head = col / p.hd, dim = col - head * p.hd;
        T *pool = (T *)(proj == 1 ? p.k_pool : p.v_pool);
        const size_t off = ((((size_t)a.layer * p.n_pages + page) * p.H + head) * p.page_size + (pos & (p.page_size - 1))) * (size_t)p.hd + dim;
        store_f(pool, off, r0);
        store_f(pool, off + 1, r1);
      }
    } else if constexpr (EPI == ROW_GATEUP) {
      a.out[(size_t)mine * (a.N / 2) + pr] = y0 / (1.0f + __expf(-y0)) * y1;
    } else if constexpr (EPI == ROW_RESID) {
      a.out[(size_t)mine * a.N + c0] = h0 + y0;
      if (c1 != c0) a.out[(size_t)mine * a.N + c1] = h1 + y1;
    } else {
      a.out[(size_t)orow * a.N + c0] = y0;
      if (c1 != c0) a.out[(size_t)orow * a.N + c1] = y1;
    }
  }
}

template <int V> struct vec_c { static constexpr int value = V; };

template <typename T, int EPI>
static void launch_row_gemm(const Params &p, const RowGemm &a, hipStream_t s) {
  const int grid = ((a.N + 1) / 2 + 3) / 4;
  // Chunks: 16 bytes of a weight row per lane, so that a wavefront's loads are whole lines (fp32 in chunks of 8: d 4096, 8 rows
  // 1.70 ms a call pair against 1.20); bf16 of a row of fewer than 512 in chunks of 4, or half of the lanes would have nothing
  // to do.  (The chunk decides the order of a row's sums: it follows type and K alone.)
  // Rows: as few blocks of up to eight as hold them, all of one size, because a row past the last one costs as much as any.
  // fp32, d 4096, two layers, a call pair: 5 rows in a block of eight 1.53 ms, now 0.98; 9 rows in two blocks of eight 2.53,
  // now 1.53.  With a wavefront per column and the norm, the rotary embedding and the activation in kernels of their own: 1.43
  // and 2.20.
  const int blocks = (a.M + 7) / 8, rows = (a.M + blocks - 1) / blocks;
  auto go = [&](auto V) {
    constexpr int VEC = decltype(V)::value;
    switch (rows) {
      case 1: row_gemm_kernel<T, EPI, VEC, 1><<<grid, 256, 0, s>>>(p, a); break;
      case 2: row_gemm_kernel<T, EPI, VEC, 2><<<grid, 256, 0, s>>>(p, a); break;
      case 3: row_gemm_kernel<T, EPI, VEC, 3><<<grid, 256, 0, s>>>(p, a); break;
      case 4: row_gemm_kernel<T, EPI, VEC, 4><<<grid, 256, 0, s>>>(p, a); break;
      case 5: row_gemm_kernel<T, EPI, VEC, 5><<<grid, 256, 0, s>>>(p, a); break;
      case 6: row_gemm_kernel<T, EPI, VEC, 6><<<grid, 256, 0, s>>>(p, a); break;
      case 7: row_gemm_kernel<T, EPI, VEC, 7><<<grid, 256, 0, s>>>(p, a); break;
      default: row_gemm_kernel<T, EPI, VEC, 8><<<grid, 256, 0, s>>>(p, a); break;
    }
  };
  if (sizeof(T) == 4 || a.K < 512) go(vec_c<4>{});
  else if constexpr (sizeof(T) == 2) go(vec_c<8>{});
}
template <int EPI>
static void launch_row_gemm_dt(int dtype, const Params &p, const RowGemm &a, hipStream_t s) {
  if (dtype == PASS_F32) launch_row_gemm<float, EPI>(p, a, s);
  else launch_row_gemm<bf16_t, EPI>(p, a, s);
}
void launch_row_qkv(const Params &p, int dtype, const void *gain, const void *W, int layer, int M, hipStream_t s) {
  launch_row_gemm_dt<ROW_QKV>(dtype, p, RowGemm{p.h, W, gain, p.qkv, nullptr, M, 3 * p.D, p.d, layer}, s);
}
void launch_row_resid(const Params &p, int dtype, const float *X, const void *W, int K, int M, hipStream_t s) {
  launch_row_gemm_dt<ROW_RESID>(dtype, p, RowGemm{X, W, nullptr, p.h, nullptr, M, p.d, K, 0}, s);
}
void launch_row_gateup(const Params &p, int dtype, const void *gain, const void *W, int M, hipStream_t s) {
  launch_row_gemm_dt<ROW_GATEUP>(dtype, p, RowGemm{p.h, W, gain, p.act, nullptr, M, 2 * p.F, p.d, 0}, s);
}
void launch_row_logits(const Params &p, int dtype, const void *gain, const void *W, float *logits, int M, hipStream_t s) {
  launch_row_gemm_dt<ROW_LOGITS>(dtype, p, RowGemm{p.h, W, gain, logits, p.row_out, M, p.V, p.d, 0}, s);
}

// ---------------------------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------------------------
struct PokeArgs {
  int32_t *ptr[16];
  int32_t val[16];
  int n;
};
__global__ void poke_kernel(PokeArgs a) {
  int i = threadIdx.x;
  if (i < a.n) *a.ptr[i] = a.val[i];
}
void launch_poke(int32_t *const *ptrs, const int32_t *vals, int n, hipStream_t s) {
  PokeArgs a;
  a.n = n;
  for (int i = 0; i < n; ++i) { a.ptr[i] = ptrs[i]; a.val[i] = vals[i]; }
  poke_kernel<<<1, 16, 0, s>>>(a);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, size_t n) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}
// Reads n16 16-byte words and drops them: the yardstick of pass_plain_read.  Every workgroup owns
// a contiguous segment (the pattern that reads fastest on this device), 8 requests per thread in
// flight.  `never` is 0: the store only keeps the loads alive.
typedef uint32_t rd_u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void plain_read_kernel(const rd_u32x4 *src, size_t n16, int never, uint32_t *sink) {
  constexpr int U = 8;
  const size_t per = (n16 + gridDim.x - 1) / gridDim.x;
  const size_t lo = per * blockIdx.x, hi = min(n16, lo + per);
  uint32_t acc = 0;
  size_t i = lo + threadIdx.x;
  for (; i + (U - 1) * 256 < hi; i += U * 256) {
    rd_u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= v[u][u & 3];
  }
  for (; i < hi; i += 256) acc ^= __builtin_nontemporal_load(src + i)[0];
  if (never && acc == 0x9e3779b9u) *sink = acc;
}

void launch_plain_read(const void *src, size_t bytes, uint32_t *sink, hipStream_t s) {
  plain_read_kernel<<<2048, 256, 0, s>>>((const rd_u32x4 *)src, bytes / 16, 0, sink);
}

void launch_fill_i32(int32_t *p, int32_t v, size_t n, hipStream_t s) {
  if (n == 0) return;
  // chunks of 2^30 elements keep the grid size inside 32 bits
  for (size_t done = 0; done < n; done += (size_t)1 << 30) {
    size_t m = n - done < ((size_t)1 << 30) ? n - done : (size_t)1 << 30;
    fill_i32_kernel<<<(unsigned)((m + 255) / 256), 256, 0, s>>>(p + done, v, m);
  }
}

}  // namespace pass
