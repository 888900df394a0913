// Projections of few token rows (M <= 64, bf16): the suffix pass, where a layer is one pass over its weights.
//
// Bound: HBM (weight bytes) and, from about 32 rows on, the rate at which L2 feeds a compute unit with activations.
// A load instruction costs by the cache lines it touches: one that takes 16 bytes from each of 16 rows runs at a fifth
// of the rate of one that takes 1 KB in one piece (measured: gate/up of the 8B shape at 64 rows 126 us against
// 77 us with only the operands' layout changed).  So both operands are kept in blocks of 16 rows x 32 columns, each
// block the 1 KB that a wave loads for one MFMA operand in lane order: block (r/16, k/32) of a matrix with K columns is at
// ((r/16) * K/32 + k/32) * 512 elements, element ((k%32)/8 * 16 + r%16) * 8 + k%8 inside it.  Weights are packed that way
// when they are set; activations are written that way by the step in front (they live in the workspace only), up to eight
// rows as rows (few_rows_row_major).
//
// No LDS ring: a wave streams both operands straight to registers, PF steps ahead; the waves of a workgroup split
// the contraction (neighbouring chunks, so that a workgroup reads 512 contiguous bytes and more per row block) and
// add up through LDS in wave order.  A workgroup that has whole sums applies the step that follows (RoPE + KV write,
// residual + what the next RMSNorm needs, SwiGLU) itself: no partial sums in memory, no reduction launch.
// RMSNorm is split: the producer of the residual stream h also writes a = bf16(h * gain) and, per 16 columns,
// the row's sum of squares; the projection that reads a scales its sums by rsqrt(mean(h^2) + eps).
#include "dsk_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

enum { EP_ROPE = 0, EP_SWIGLU = 1, EP_RES = 2, EP_PART = 3 };

// Activations of few_rows_row_major(M) rows stand in rows instead of blocks, and so do their sums of squares ([M][K/16]
// instead of [K/16][64]).
__device__ __forceinline__ int64_t act_at(int64_t m, int64_t k, int64_t K, int rows) { return rows ? m * K + k : block_at(m, k, K); }
__device__ __forceinline__ int ssq_at(int m, int part, int K, int rows) { return rows ? m * (K >> 4) + part : part * 64 + m; }

struct StreamArgs {
  const bf16_t* X;  // blocks, rows up to a multiple of 16; or rows (x_rows)
  const bf16_t* W;  // blocks
  int M, N, K, x_rows;
  const float* ssq; float eps;  // EP_ROPE, EP_SWIGLU: row factor of the RMSNorm in front, from sums of squares (ssq_at)
  bf16_t* out;                  // EP_ROPE: q rows, stride ldq; EP_SWIGLU: [M, N/2], EP_RES: a = h * gain, both in blocks or rows as X
  int64_t ldq;
  const float2* cs; bf16_t* k_rows; bf16_t* v_rows; int Hq, Hkv, dh;
  const void* R; int r_f32; void* C; int c_f32;         // EP_RES: C = sum + R, row-major
  const bf16_t* gain; float* ssq_out;                   // EP_RES: both null when nothing follows
  float* P;                                             // EP_PART: [splits][M][N]; experts: [E][M][N]
  // Expert layers: blockIdx.z is the expert; it is left out when no token has chosen it.  Strides in elements.
  const int32_t* experts; int n_entries;
  int64_t x_expert, w_expert, out_expert;
};

__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v) {
  bf16x4 o;
  o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
  return o;
}

// What a quad of the residual stream (row m, columns n .. n+3) reads besides its sum, requested before the sum is there: behind
// it these were two round trips to memory one after the other, at the end of every launch (one row through four 8B layers 359.8 ->
// 357.6 us, with the rotary pairs of QKV).
struct ResidualIn { u32x4 r; bf16x4 g; };  // r: as it lies, four fp32 or (in the lower half) four bf16
__device__ __forceinline__ ResidualIn residual_in(int m, int n, int N, bool in, const void* R, int r_f32, const bf16_t* gain) {
  ResidualIn q = {};
  const int64_t at = (int64_t)m * N + n;
  if (in) {
    if (r_f32) {
      q.r = *(const u32x4*)((const float*)R + at);
    } else {
      const u32x2 r = *(const u32x2*)((const bf16_t*)R + at);
      q.r[0] = r[0]; q.r[1] = r[1];
    }
    if (gain) q.g = *(const bf16x4*)(gain + n);
  }
  return q;
}

// v[n..n+3] of row m: + R, C, and the next norm's share; the four lanes of a 16-column group are at lane ^ X1, lane ^ X2
template <int X1, int X2>
__device__ __forceinline__ void residual_quad(f32x4 v, const ResidualIn& q, int m, int n, int N, bool in, int r_f32, void* C,
                                              int c_f32, bool norm, bf16_t* a, int a_rows, float* ssq_out) {
  const int64_t at = (int64_t)m * N + n;
  if (in) {
    if (r_f32) {
      v += __builtin_bit_cast(f32x4, q.r);
    } else {
      const bf16x4 r = __builtin_bit_cast(bf16x4, u32x2{q.r[0], q.r[1]});
      v[0] += (float)r[0]; v[1] += (float)r[1]; v[2] += (float)r[2]; v[3] += (float)r[3];
    }
    if (C) {
      if (c_f32) *(f32x4*)((float*)C + at) = v;
      else *(bf16x4*)((bf16_t*)C + at) = to_bf16x4(v);
    }
  }
  if (!norm) return;
  float ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  ss += __shfl_xor(ss, X1, 64);
  ss += __shfl_xor(ss, X2, 64);
  if (in) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= (float)q.g[e];
    *(bf16x4*)(a + act_at(m, n, N, a_rows)) = to_bf16x4(v);
    if (n % 16 == 0) ssq_out[ssq_at(m, n / 16, N, a_rows)] = ss;
  }
}

// Wave tile: MT blocks of 16 rows x NT blocks of 16 columns, KS x 32 of the contraction per step.  EP_ROPE and EP_SWIGLU
// take their column blocks in pairs that a lane combines: the halves (i, i + dh/2) of a head, or gate and up (packed in
// blocks of 32 rows each).
template <int MT, int NT, int KW, int PF, int KS, int EP>
__global__ void __launch_bounds__(64 * KW, 1) stream_kernel(StreamArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  f32x4* red = (f32x4*)smem_raw;                          // [KW][MT * NT][64]
  f32x4* red_ss = red + KW * MT * NT * 64;                // [KW][16]: sums of squares of rows 4 * i ..
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int kw = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr bool PAIRS = EP == EP_ROPE || EP == EP_SWIGLU;
  if (p.experts) {
    bool chosen = false;
    for (int i = tid; i < p.n_entries; i += 64 * KW) chosen |= p.experts[i] == (int)blockIdx.z;
    if (!__syncthreads_or(chosen)) return;
    p.X += blockIdx.z * p.x_expert;
    p.W += blockIdx.z * p.w_expert;
    if (EP == EP_PART) p.P += blockIdx.z * p.out_expert;
    else p.out += blockIdx.z * p.out_expert;
  }
  const int unit0 = blockIdx.x * (NT / 2);
  const int half = p.dh >> 1, per_head = half >> 4, n_rot = (p.Hq + p.Hkv) * per_head;
  auto col0 = [&](int j) {
    if (EP == EP_ROPE) {
      const int u = unit0 + j / 2;
      return u < n_rot ? u / per_head * p.dh + u % per_head * 16 + (j & 1) * half : (p.Hq + p.Hkv) * p.dh + 32 * (u - n_rot) + (j & 1) * 16;
    }
    if (EP == EP_SWIGLU) {
      const int u = unit0 + j / 2;
      return (u >> 1) * 64 + (u & 1) * 16 + (j & 1) * 32;
    }
    return (int)blockIdx.x * 16 * NT + 16 * j;
  };
  const int kb = p.K >> 5;  // k blocks
  uint32_t wo[NT], xo[MT];
#pragma unroll
  for (int j = 0; j < NT; ++j) wo[j] = ((uint32_t)(col0(j) >> 4) * kb * 64 + lane) * 16;
#pragma unroll
  for (int i = 0; i < MT; ++i) xo[i] = ((uint32_t)i * kb * 64 + lane) * 16;
  // rows: a lane's eight values of its row (the last one for those past it), 64 bytes a block
  const bool x_rows = MT == 1 && p.x_rows;
  if (x_rows) xo[0] = ((uint32_t)min(r16, p.M - 1) * p.K + 8 * g) * 2;
  const int x_step = x_rows ? 64 : 1024;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // steps of this workgroup's share of the contraction (blockIdx.y of gridDim.y shares); K is a multiple of 64
  const int n_steps_all = kb / KS;
  const int begin = (int)((int64_t)n_steps_all * blockIdx.y / gridDim.y), end = (int)((int64_t)n_steps_all * (blockIdx.y + 1) / gridDim.y);
  bf16x8 fw[PF][KS][NT], fx[PF][KS][MT];
  auto load = [&](int s, int c) {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int b = c * KS + q;
      const char* wb = (const char*)p.W + (int64_t)b * 1024;
      const char* xb = (const char*)p.X + (int64_t)b * x_step;
#pragma unroll
      for (int j = 0; j < NT; ++j) fw[s][q][j] = __builtin_nontemporal_load((const bf16x8*)(wb + wo[j]));
#pragma unroll
      for (int i = 0; i < MT; ++i) fx[s][q][i] = *(const bf16x8*)(xb + xo[i]);
    }
  };
  // What the epilogue of the wave's item (one at most) reads: in flight under the contraction
  static_assert((EP != EP_RES && EP != EP_ROPE) || MT * (PAIRS ? NT / 2 : NT) <= KW, "one item a wave");
  ResidualIn res;
  f32x4 cs[2];  // four (cos, sin)
  if ((EP == EP_RES || EP == EP_ROPE) && kw < MT * (PAIRS ? NT / 2 : NT)) {
    const int m = 16 * (kw % MT) + r16, c0 = col0(PAIRS ? kw / MT * 2 : kw / MT);
    if (EP == EP_RES) res = residual_in(m, c0 + 4 * g, p.N, m < p.M, p.R, p.r_f32, p.gain);
    if (EP == EP_ROPE && m < p.M && c0 < (p.Hq + p.Hkv) * p.dh) {
      const f32x4* src = (const f32x4*)(p.cs + (int64_t)m * half + c0 % p.dh + 4 * g);
      cs[0] = src[0];
      cs[1] = src[1];
    }
  }
#pragma unroll
  for (int s = 0; s < PF; ++s) {
    load(s, min(begin + kw + s * KW, end - 1));
    __builtin_amdgcn_sched_barrier(0);
  }
  if (PAIRS && x_rows) {
    // Sums of squares in rows: a wave per row, 32 lanes each every 32nd part, added up as below.  (As columns of 64 a row's parts
    // lie in a cache line each.)
    static_assert(MT > 1 || KW == 8, "a wave per row, 32 lanes as the groups of 16 lanes below");
    const int parts = p.K >> 4;
    float s = 0.f;
    if (kw < p.M && lane < 32) {
      for (int q = lane; q < parts; q += 8 * 32) {
        float b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = q + u * 32 < parts ? p.ssq[kw * parts + q + u * 32] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += b[u];
      }
    }
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if (lane < 32 && lane % 4 == 0) ((float*)red_ss)[lane / 4 * 64 + kw] = s;
  } else if (PAIRS) {
    // Sums of squares: four rows a lane, eight loads in flight.  One load at a time took longer than the matrix (25 us instead
    // of 18.6 us for QKV over 64 rows, 58 us instead of 43.7 us for gate/up); requested in front of the operands: 49 us.
    const float* src = p.ssq + 4 * r16;
    const int parts = p.K >> 4;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (4 * r16 < 16 * MT) {
      for (int q = tid >> 4; q < parts; q += 8 * 4 * KW) {
        f32x4 b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = q + u * 4 * KW < parts ? *(const f32x4*)(src + (q + u * 4 * KW) * 64) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 8; ++u) s += b[u];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] += __shfl_xor(s[e], 16, 64);
      s[e] += __shfl_xor(s[e], 32, 64);
    }
    if (lane < 16) red_ss[kw * 16 + lane] = s;
  }
  // Where a load is under a condition the compiler counts on the path without it, and waits at a step's first operands for
  // nearly all that is in flight; the same where it mixes the loads of two steps.  So the loop has no conditions, the last
  // steps, 2 * PF - 1 at most, come behind it, and no load crosses into another step's.
  // (Four 8B layers, 64 rows 545 -> 536 us, one row 357.6 -> 355.6; a Mixtral layer over 64 rows 582 -> 575.)
  auto step = [&](int s) {
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[s][q][j], fx[s][q][i], acc[j][i], 0, 0, 0);
  };
  int c = begin + kw;
  for (; c + (2 * PF - 1) * KW < end; c += PF * KW) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      step(s);
      load(s, c + (s + PF) * KW);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < 2 * PF - 1; ++s) {
    if (c + s * KW < end) {
      step(s % PF);
      if (s + PF < 2 * PF - 1 && c + (s + PF) * KW < end) load(s, c + (s + PF) * KW);
    }
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) red[(kw * MT * NT + j * MT + i) * 64 + lane] = acc[j][i];
  __syncthreads();
  auto total = [&](int j, int i) {
    f32x4 v = red[(j * MT + i) * 64 + lane];
#pragma unroll
    for (int k = 1; k < KW; ++k) v += red[(k * MT * NT + j * MT + i) * 64 + lane];
    return v;
  };
  for (int it = kw; it < MT * (PAIRS ? NT / 2 : NT); it += KW) {
    const int i = it % MT, jj = it / MT, m = 16 * i + r16;
    const bool in = m < p.M;
    if (!PAIRS) {
      const int n = col0(jj) + 4 * g;
      const f32x4 v = total(jj, i);
      if (EP == EP_PART) {
        if (in) *(f32x4*)(p.P + ((int64_t)blockIdx.y * p.M + m) * p.N + n) = v;
      } else {
        residual_quad<16, 32>(v, res, m, n, p.N, in, p.r_f32, p.C, p.c_f32, p.gain, p.out, x_rows, p.ssq_out);
      }
      continue;
    }
    f32x4 x0 = total(2 * jj, i), x1 = total(2 * jj + 1, i);
    if (!in) continue;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < KW; ++k) s += ((const float*)red_ss)[k * 64 + m];
    const float rs = rsqrtf(s / (float)p.K + p.eps);
    x0 *= rs;
    x1 *= rs;
    if (EP == EP_SWIGLU) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x0[e]));
        o[e] = x0[e] * sig * x1[e];
      }
      *(bf16x4*)(p.out + act_at(m, 16 * (unit0 + jj) + 4 * g, p.N >> 1, x_rows)) = to_bf16x4(o);
    } else {
      const int c0 = col0(2 * jj), rot_cols = (p.Hq + p.Hkv) * p.dh, kvw = p.Hkv * p.dh;
      if (c0 < rot_cols) {
        const int head = c0 / p.dh, i0 = c0 % p.dh + 4 * g;
        f32x4 y0, y1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float co = cs[e / 2][e % 2 * 2], si = cs[e / 2][e % 2 * 2 + 1];
          y0[e] = x0[e] * co - x1[e] * si;
          y1[e] = x1[e] * co + x0[e] * si;
        }
        bf16_t* dst = head < p.Hq ? p.out + (int64_t)m * p.ldq + head * p.dh + i0
                                  : p.k_rows + (int64_t)m * kvw + (head - p.Hq) * p.dh + i0;
        *(bf16x4*)dst = to_bf16x4(y0);
        *(bf16x4*)(dst + half) = to_bf16x4(y1);
      } else {
        bf16_t* dst = p.v_rows + (int64_t)m * kvw + (c0 - rot_cols) + 4 * g;
        *(bf16x4*)dst = to_bf16x4(x0);
        *(bf16x4*)(dst + 16) = to_bf16x4(x1);
      }
    }
  }
}

// What stream_kernel's EP_RES does, for a contraction split over workgroups (partial sums P, added in split order).  One
// thread per 4 columns of a row.
__global__ void __launch_bounds__(256) few_residual_kernel(const float* __restrict__ P, int splits, const void* R, int r_f32,
                                                           void* C, int c_f32, const bf16_t* __restrict__ gain,
                                                           bf16_t* __restrict__ a, float* __restrict__ ssq_out, int M, int N) {
  const int i = blockIdx.x * 256 + threadIdx.x, quads = N / 4;
  const bool in = i < M * quads;
  const int m = in ? i / quads : 0, n = in ? (i - m * quads) * 4 : 0;
  const ResidualIn q = residual_in(m, n, N, in, R, r_f32, gain);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (in) {
    f32x4 b[4];
    const int64_t stride = (int64_t)M * N;
    const float* src = P + (int64_t)m * N + n;
    for (int k = 0; k < splits; k += 4) {  // four at a time in flight
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k + u < splits) b[u] = *(const f32x4*)(src + (k + u) * stride);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k + u < splits) v += b[u];
    }
  }
  residual_quad<1, 2>(v, q, m, n, N, in, r_f32, C, c_f32, gain, a, 0, ssq_out);
}

// Router of an expert layer on the prepared rows a (blocks or rows; the RMSNorm factor is applied to the logits), one workgroup per
// token: eight experts at a time, every thread eight columns of each, sums over the workgroup in a fixed order.  Same
// rules as the router over rows (moe.hip): fp32 logits, equal ones to the lower expert, NaN last.
__global__ void __launch_bounds__(256) few_route_kernel(const bf16_t* __restrict__ a, const float* __restrict__ ssq, float eps,
                                                        const bf16_t* __restrict__ wr, int32_t* __restrict__ experts,
                                                        float* __restrict__ gates, int a_rows, int d, int E, int top_k) {
  __shared__ float part[4][9];
  __shared__ float logit[DSK_MOE_MAX_EXPERTS];
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float ss = 0.f;
  for (int q = tid; q < d / 16; q += 256) ss += ssq[ssq_at(t, q, d, a_rows)];
  for (int e0 = 0; e0 < E; e0 += 8) {
    float acc[9] = {};
    for (int c = tid; c < d / 8; c += 256) {
      const bf16x8 x = *(const bf16x8*)(a + act_at(t, 8 * c, d, a_rows));
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bf16x8 w = *(const bf16x8*)(wr + (int64_t)min(e0 + e, E - 1) * d + 8 * c);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[e] = fmaf((float)x[u], (float)w[u], acc[e]);
      }
    }
    acc[8] = ss;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc[e] += __shfl_xor(acc[e], o, 64);
      if (lane == 0) part[wave][e] = acc[e];
    }
    __syncthreads();
    if (tid < 8 && e0 + tid < E) {
      const float rs = rsqrtf((part[0][8] + part[1][8] + part[2][8] + part[3][8]) / (float)d + eps);
      const float v = (part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid]) * rs;
      logit[e0 + tid] = v == v ? v : -3.0e38f;
    }
    __syncthreads();
  }
  if (tid != 0) return;
  float best[DSK_MOE_MAX_TOP_K];
  float sum = 0.f;
  for (int j = 0; j < top_k; ++j) {
    int at = 0;
    for (int e = 1; e < E; ++e)
      if (logit[e] > logit[at]) at = e;  // strictly greater: the lower index keeps a tie
    best[j] = logit[at];
    logit[at] = -INFINITY;               // below every real entry (a NaN logit counts as -3e38)
    experts[t * top_k + j] = at;
    sum += expf(best[j] - best[0]);
  }
  const float inv = 1.0f / sum;
  for (int j = 0; j < top_k; ++j) gates[t * top_k + j] = expf(best[j] - best[0]) * inv;
}

// C = h + sum_j gates[t][j] * y[experts[t][j]][t], and the next norm's share, as few_residual_kernel
__global__ void __launch_bounds__(256) few_combine_kernel(const float* __restrict__ y, const int32_t* __restrict__ experts,
                                                          const float* __restrict__ gates, int top_k, int E, const void* R, void* C,
                                                          int c_f32, const bf16_t* __restrict__ gain, bf16_t* __restrict__ a, int a_rows,
                                                          float* __restrict__ ssq_out, int M, int N) {
  const int i = blockIdx.x * 256 + threadIdx.x, quads = N / 4;
  const bool in = i < M * quads;
  const int m = in ? i / quads : 0, n = in ? (i - m * quads) * 4 : 0;
  const ResidualIn q = residual_in(m, n, N, in, R, 1, gain);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (in) {
    for (int j = 0; j < top_k; ++j) {
      const int e = min(max(experts[m * top_k + j], 0), E - 1);  // always inside y, whatever the table holds
      v += *(const f32x4*)(y + ((int64_t)e * M + m) * N + n) * gates[m * top_k + j];
    }
  }
  residual_quad<1, 2>(v, q, m, n, N, in, 1, C, c_f32, gain, a, a_rows, ssq_out);
}

// The input norm of a call's first layer and the call's rotary table: workgroups 0 .. n_norm-1, and those behind them.
__global__ void __launch_bounds__(256) few_norm_rope_kernel(const void* h, int h_f32, const bf16_t* __restrict__ gain,
                                                            bf16_t* __restrict__ a, int a_rows, float* __restrict__ ssq_out, int M,
                                                            int N, int n_norm, RopeJob rope) {
  if ((int)blockIdx.x >= n_norm) {
    rope_entry(rope, (int64_t)((int)blockIdx.x - n_norm) * 256 + threadIdx.x);
    return;
  }
  const int i = blockIdx.x * 256 + threadIdx.x, quads = N / 4;
  const bool in = i < M * quads;
  const int m = in ? i / quads : 0, n = in ? (i - m * quads) * 4 : 0;
  residual_quad<1, 2>(f32x4{0.f, 0.f, 0.f, 0.f}, residual_in(m, n, N, in, h, h_f32, gain), m, n, N, in, h_f32, nullptr, 0, gain, a, a_rows, ssq_out);
}

template <int MT, int NT, int KW, int PF, int KS, int EP>
hipError_t launch_stream(const StreamArgs& p, int tiles, int splits, hipStream_t s, int n_experts = 1) {
  auto kern = stream_kernel<MT, NT, KW, PF, KS, EP>;
  constexpr int lds = KW * MT * NT * 1024 + KW * 256;
  if constexpr (lds > 64 << 10) {
    static bool configured = false;
    if (!configured) {
      hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
      configured = true;
    }
  }
  hipLaunchKernelGGL(kern, dim3(tiles, splits, n_experts), dim3(64 * KW), lds, s, p);
  return hipGetLastError();
}

// A projection with residual runs unsplit on 16-column tiles (every compute unit gets one at the 8B width) as long as
// that many tiles re-reading the activations stay cheap; beyond 180 MB of such reads the contraction is split over about 256
// workgroups of 64 columns, and a reduction launch adds up.  8B shape: O over 64 rows (134 MB of reads) 13.6 us against
// 10.6 us + 4.9 us split; down over 64 rows (470 MB) 40 us against 24.6 us + 4.9 us, over 32 (235 MB) 31.8 against 21.6 + 4.8,
// over 16 (117 MB) 24.0 unsplit.  Other widths, us a layer unsplit -> split: down over 64 rows, 3072 wide (201 MB) 92.2 -> 92.1; O over
// 64 rows, 5120 wide (210 MB) 160.8 -> 155.9; O over 40 rows, 6144 wide (226 MB) 190.0 -> 186.7; O over 32 rows, 8192 wide (268 MB)
// 314.0 -> 308.3.
int residual_splits(int M, int N, int K) {
  const int rows = (M + 15) / 16 * 16;
  if (rows <= 16 || (int64_t)(N / 16) * rows * K * 2 <= (int64_t)180 << 20) return 0;
  const int tiles = N / 64, splits = (256 + tiles - 1) / tiles;
  return splits > K / 512 ? (K / 512 > 0 ? K / 512 : 1) : splits;
}

}  // namespace

// Widths in whole blocks, heads in whole pairs of blocks.
bool few_rows_supported(int M, int d, int F, int Hq, int Hkv, int dh) {
  return M >= 1 && M <= 64 && d % 64 == 0 && F % 64 == 0 && dh % 32 == 0 && Hq * dh % 64 == 0;
}

// A block holds 16 rows whatever M is, and what an unfilled one costs is its cache lines: eight a load, against one a row where
// the activations stand in rows; a row's sums of squares likewise.  8B shape, us a launch, blocks against rows: one row QKV
// 12.2 -> 10.8, O 8.8 -> 7.9, gate/up 40.5 -> 37.8, down 22.8 -> 19.9; eight rows 12.2 -> 11.6, 8.7 -> 8.1, 40.4 -> 39.4, 22.6 ->
// 20.7; twelve rows (activations alone) 12.4 -> 12.8, 8.9 -> 9.0, 40.5 -> 41.7, 23.1 -> 22.9.
bool few_rows_row_major(int M) { return M <= 8; }

int64_t few_rows_workspace_bytes(int d, int K_max) {
  const int s = residual_splits(64, d, K_max);
  return (int64_t)(s > 0 ? s : 1) * 64 * d * 4;
}

hipError_t launch_few_norm(const void* h, int h_f32, const void* gain, void* a, float* ssq, int M, int d, const RopeJob* rope,
                           hipStream_t s) {
  const int n_norm = (M * (d / 4) + 255) / 256;
  const RopeJob job = rope ? *rope : RopeJob{};
  hipLaunchKernelGGL(few_norm_rope_kernel, dim3(n_norm + rope_blocks(job)), dim3(256), 0, s, h, h_f32, (const bf16_t*)gain, (bf16_t*)a,
                     (int)few_rows_row_major(M), ssq, M, d, n_norm, job);
  return hipGetLastError();
}

hipError_t launch_few_qkv(const void* a, const float* ssq, float eps, const void* W, void* qkv, int64_t ldq, const float2* cs,
                          void* k_rows, void* v_rows, int M, int d, int Hq, int Hkv, int dh, hipStream_t s) {
  StreamArgs p = {};
  p.X = (const bf16_t*)a; p.W = (const bf16_t*)W; p.M = M; p.x_rows = few_rows_row_major(M); p.N = (Hq + 2 * Hkv) * dh; p.K = d; p.ssq = ssq; p.eps = eps;
  p.out = (bf16_t*)qkv; p.ldq = ldq; p.cs = cs; p.k_rows = (bf16_t*)k_rows; p.v_rows = (bf16_t*)v_rows;
  p.Hq = Hq; p.Hkv = Hkv; p.dh = dh;
  const int tiles = p.N / 32;
  switch ((M + 15) / 16) {
    case 1: return launch_stream<1, 2, 8, 2, 2, EP_ROPE>(p, tiles, 1, s);
    case 2: return launch_stream<2, 2, 8, 2, 2, EP_ROPE>(p, tiles, 1, s);
    case 3: return launch_stream<3, 2, 8, 2, 2, EP_ROPE>(p, tiles, 1, s);
    default: return launch_stream<4, 2, 8, 2, 2, EP_ROPE>(p, tiles, 1, s);
  }
}

// Up to 16 rows: 32-column tiles; more: 128-column tiles (224 workgroups at the 8B width), which read the activations
// a quarter as often (8B shape, 64 rows 45 us against 57 us; with one step in flight instead of two 50 us; 32 rows 42.0 against 47.3;
// 12 rows 43.2 against 42.2).  With 17 to 32 rows only where there are enough of them for the chip.
hipError_t launch_few_swiglu(const void* a, const float* ssq, float eps, const void* W, void* act, int M, int N, int K,
                             hipStream_t s) {
  StreamArgs p = {};
  p.X = (const bf16_t*)a; p.W = (const bf16_t*)W; p.M = M; p.x_rows = few_rows_row_major(M); p.N = N; p.K = K; p.ssq = ssq; p.eps = eps; p.out = (bf16_t*)act;
  switch ((M + 15) / 16) {
    case 1: return launch_stream<1, 2, 8, 2, 2, EP_SWIGLU>(p, N / 32, 1, s);
    case 2: return N / 128 >= 192 ? launch_stream<2, 8, 4, 2, 1, EP_SWIGLU>(p, N / 128, 1, s)
                                  : launch_stream<2, 2, 8, 2, 2, EP_SWIGLU>(p, N / 32, 1, s);
    case 3: return launch_stream<3, 8, 4, 2, 1, EP_SWIGLU>(p, N / 128, 1, s);
    default: return launch_stream<4, 8, 4, 2, 1, EP_SWIGLU>(p, N / 128, 1, s);
  }
}

hipError_t launch_few_residual(const void* x, const void* W, const void* R, int r_f32, void* C, int c_f32, const void* gain,
                               void* a, float* ssq, int M, int N, int K, void* ws, int64_t ws_bytes, hipStream_t s) {
  StreamArgs p = {};
  p.X = (const bf16_t*)x; p.W = (const bf16_t*)W; p.M = M; p.x_rows = few_rows_row_major(M); p.N = N; p.K = K;
  p.R = R; p.r_f32 = r_f32; p.C = C; p.c_f32 = c_f32; p.gain = (const bf16_t*)gain; p.out = (bf16_t*)a; p.ssq_out = ssq;
  p.P = (float*)ws;
  const int mt = (M + 15) / 16, splits = residual_splits(M, N, K);
  if (splits > 0) {
    if (!ws || (int64_t)splits * M * N * 4 > ws_bytes) return hipErrorNotSupported;
    hipError_t e = mt == 2 ? launch_stream<2, 4, 8, 2, 1, EP_PART>(p, N / 64, splits, s)
                   : mt == 3 ? launch_stream<3, 4, 8, 2, 1, EP_PART>(p, N / 64, splits, s)
                           : launch_stream<4, 4, 8, 2, 1, EP_PART>(p, N / 64, splits, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(few_residual_kernel, dim3((M * (N / 4) + 255) / 256), dim3(256), 0, s, (const float*)ws, splits, R, r_f32,
                       C, c_f32, (const bf16_t*)gain, (bf16_t*)a, ssq, M, N);
    return hipGetLastError();
  }
  switch (mt) {
    case 1: return launch_stream<1, 1, 8, 2, 2, EP_RES>(p, N / 16, 1, s);
    case 2: return launch_stream<2, 1, 8, 2, 2, EP_RES>(p, N / 16, 1, s);
    case 3: return launch_stream<3, 1, 8, 2, 2, EP_RES>(p, N / 16, 1, s);
    default: return launch_stream<4, 1, 8, 2, 2, EP_RES>(p, N / 16, 1, s);
  }
}

hipError_t launch_few_route(const void* a, const float* ssq, float eps, const void* wr, int32_t* experts, float* gates, int n,
                            int d, int E, int top_k, hipStream_t s) {
  if (E < 1 || E > DSK_MOE_MAX_EXPERTS || top_k < 1 || top_k > DSK_MOE_MAX_TOP_K || top_k > E) return hipErrorNotSupported;
  hipLaunchKernelGGL(few_route_kernel, dim3(n), dim3(256), 0, s, (const bf16_t*)a, ssq, eps, (const bf16_t*)wr, experts, gates,
                     (int)few_rows_row_major(n), d, E, top_k);
  return hipGetLastError();
}

// The expert MLPs over all rows (a few rows hit most experts, and what it costs is the weights): one launch per projection
// over every expert that some token has chosen (Mixtral width, 64 rows: 332 + 150 us for 2.8 GB; expert by expert with a
// reduction behind each, 32 launches, 730 us; one row streams two experts of the eight).  Tiles as wide as still give the chip 256
// workgroups read the activations (of down 1.8 MB a workgroup at 64 rows) less often: down in 128- instead of 64-column tiles over 64
// rows 166.5 -> 149.7 us, over 40 161 -> 150, over 24 (32-column tiles before) 169 -> 146; gate/up over 24 rows 321 -> 304; down over 12
// rows in 64- instead of 16-column tiles 145.7 -> 129.8 (over 4 rows, five experts or six, 98 against 82: up to eight rows 16 columns).  act: [E][rows up to 16][F],
// blocks or rows (few_rows_row_major); y: [E][M][d].
hipError_t launch_few_experts(const void* a, const float* ssq, float eps, const void* wgu, const void* wd, void* act, float* y,
                              const int32_t* experts, int M, int d, int F, int E, int top_k, hipStream_t s) {
  StreamArgs p = {};
  p.X = (const bf16_t*)a; p.W = (const bf16_t*)wgu; p.M = M; p.x_rows = few_rows_row_major(M); p.N = 2 * F; p.K = d; p.ssq = ssq; p.eps = eps; p.out = (bf16_t*)act;
  p.experts = experts; p.n_entries = M * top_k;
  p.w_expert = 2 * (int64_t)F * d; p.out_expert = (int64_t)(M + 15) / 16 * 16 * F;
  hipError_t e;
  const int chosen = M * top_k < E ? M * top_k : E;  // experts that run, at most
  switch ((M + 15) / 16) {
    case 1: e = launch_stream<1, 2, 8, 2, 2, EP_SWIGLU>(p, p.N / 32, 1, s, E); break;
    case 2:
      e = (int64_t)p.N / 128 * chosen >= 192 ? launch_stream<2, 8, 4, 2, 1, EP_SWIGLU>(p, p.N / 128, 1, s, E)
                                             : launch_stream<2, 2, 8, 2, 2, EP_SWIGLU>(p, p.N / 32, 1, s, E);
      break;
    case 3: e = launch_stream<3, 8, 4, 2, 1, EP_SWIGLU>(p, p.N / 128, 1, s, E); break;
    default: e = launch_stream<4, 8, 4, 2, 1, EP_SWIGLU>(p, p.N / 128, 1, s, E); break;
  }
  if (e != hipSuccess) return e;
  p.X = (const bf16_t*)act; p.x_expert = p.out_expert;
  p.W = (const bf16_t*)wd; p.w_expert = (int64_t)d * F;
  p.N = d; p.K = F; p.P = y; p.out_expert = (int64_t)M * d;
  const bool wide = d % 128 == 0 && (int64_t)d / 128 * chosen >= 256;
  switch ((M + 15) / 16) {
    case 1:
      return M > 8 && (int64_t)d / 64 * chosen >= 256 ? launch_stream<1, 4, 8, 2, 1, EP_PART>(p, d / 64, 1, s, E)
                                                      : launch_stream<1, 1, 8, 2, 2, EP_PART>(p, d / 16, 1, s, E);
    case 2:
      return wide ? launch_stream<2, 8, 4, 2, 1, EP_PART>(p, d / 128, 1, s, E) : launch_stream<2, 2, 8, 2, 2, EP_PART>(p, d / 32, 1, s, E);
    case 3:
      return wide ? launch_stream<3, 8, 4, 2, 1, EP_PART>(p, d / 128, 1, s, E) : launch_stream<3, 4, 8, 2, 1, EP_PART>(p, d / 64, 1, s, E);
    default:
      return wide ? launch_stream<4, 8, 4, 2, 1, EP_PART>(p, d / 128, 1, s, E) : launch_stream<4, 4, 8, 2, 1, EP_PART>(p, d / 64, 1, s, E);
  }
}

hipError_t launch_few_combine(const float* y, const int32_t* experts, const float* gates, int top_k, int E, const float* h, void* C,
                              int c_f32, const void* gain, void* a, float* ssq, int M, int d, hipStream_t s) {
  hipLaunchKernelGGL(few_combine_kernel, dim3((M * (d / 4) + 255) / 256), dim3(256), 0, s, y, experts, gates, top_k, E,
                     (const void*)h, C, c_f32, (const bf16_t*)gain, (bf16_t*)a, (int)few_rows_row_major(M), ssq, M, d);
  return hipGetLastError();
}
