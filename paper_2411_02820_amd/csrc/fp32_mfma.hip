// fp32 models on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 products, fp32 accumulation): the
// projections with what surrounds them in a layer (RMSNorm in front, residual / RoPE + KV write / SwiGLU behind) and
// causal attention.
//
// What bounds these: the fp32 workload is small (128 tokens, width 256), every launch is a few microseconds of latency
// and next to no arithmetic.  So a layer is five launches, every workgroup's loads go straight to registers (nothing to
// share that the caches do not hold), and the contraction is split over the waves of a workgroup so that a
// chain of loads is two to six long instead of forty; and since one matrix instruction is 32 cycles for 2048 flops, the chains
// of those count as well: narrow tiles, eight waves for the keys of a launch that few workgroups make.  The whole fp32 workload
// (2 layers over 128 tokens, 4 over 16) takes 0.190 ms; with wide tiles, four waves for the keys and the rotary table in a launch
// of its own 0.220 ms; on the plain-ALU kernels with separate norm, RoPE and SwiGLU launches 1.43 ms (projections 41 us, attention
// 44 us a launch).
// Error against 64 bits 1.4e-7 (2-norm; plain kernels 3.0e-7).  More chunks in flight (six instead of three): no gain.
#include "dsk_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct Fp32Gemm {
  const float* A; int64_t lda;
  const float* W; int64_t ldw;
  float* C; int64_t ldc;
  const float* R; int64_t ldr;
  int M, N, K;
  int units;  // of 32 columns of W (unit_cols), of 16 on narrow tiles
  const float* gain; float eps;                     // RMSNorm in front (NORM)
  int gu_block;                                     // EP_SWIGLU
  const float2* cs; float* k_rows; float* v_rows;   // EP_ROPE
  int Hq, Hkv, dh;
  RopeJob job;                                      // EP_ROPE, job.cs set: the table is still to be filled (and cs is job.cs)
};

enum { EP_PLAIN = 0, EP_SWIGLU = 1, EP_ROPE = 2 };

// Columns of W come in units of two sides c0 and c1 of 8 * CT columns, paired so that a lane holds what its epilogue
// combines: neighbours; gate and up of the same FFN index; or the two halves of rotary pairs.  CT = 2: a 16-column tile for
// either side; CT = 1: one tile for both.
template <int EP, int CT>
__device__ __forceinline__ void unit_cols(const Fp32Gemm& p, int u, int* c0, int* c1) {
  constexpr int UP = 8 * CT;
  if (EP == EP_SWIGLU) {
    const int f = UP * u, gb = p.gu_block;
    *c0 = f / gb * 2 * gb + f % gb;
    *c1 = *c0 + gb;
  } else if (EP == EP_ROPE) {
    const int half = p.dh >> 1, per = half / UP, n_rot = (p.Hq + p.Hkv) * per;
    if (u < n_rot) {
      *c0 = u / per * p.dh + u % per * UP;
      *c1 = *c0 + half;
    } else {
      *c0 = (p.Hq + p.Hkv) * p.dh + 2 * UP * (u - n_rot);
      *c1 = *c0 + UP;
    }
  } else {
    *c0 = 2 * UP * u;
    *c1 = *c0 + UP;
  }
}

// One lane's share of unit u: x0, x1 = four consecutive columns of row m behind c0 and c1, at column offset q4; cs: the
// (cos, sin) of the four pairs of a rotated unit.
template <int EP, int CT>
__device__ __forceinline__ void unit_store(const Fp32Gemm& p, int m, int u, int q4, f32x4 x0, f32x4 x1, const float2* cs) {
  constexpr int UP = 8 * CT;
  int c0, c1;
  unit_cols<EP, CT>(p, u, &c0, &c1);
  if (EP == EP_SWIGLU) {
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = x0[e] / (1.0f + __expf(-x0[e])) * x1[e];
    *(f32x4*)(p.C + (int64_t)m * p.ldc + UP * u + q4) = o;
  } else if (EP == EP_ROPE) {
    const int half = p.dh >> 1, rot_cols = (p.Hq + p.Hkv) * p.dh, kvw = p.Hkv * p.dh;
    if (c0 < rot_cols) {
      const int head = c0 / p.dh, i0 = c0 % p.dh + q4;
      f32x4 y0, y1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 c = cs[e];
        y0[e] = x0[e] * c.x - x1[e] * c.y;
        y1[e] = x1[e] * c.x + x0[e] * c.y;
      }
      float* dst = head < p.Hq ? p.C + (int64_t)m * p.ldc + head * p.dh + i0 : p.k_rows + (int64_t)m * kvw + (head - p.Hq) * p.dh + i0;
      *(f32x4*)dst = y0;
      *(f32x4*)(dst + half) = y1;
    } else {
      float* dst = p.v_rows + (int64_t)m * kvw + (c0 - rot_cols) + q4;
      *(f32x4*)dst = x0;
      *(f32x4*)(dst + UP) = x1;
    }
  } else {
#pragma unroll
    for (int t = 0; t < CT; ++t) {  // CT = 1: the unit's 16 columns are the lanes' four by four
      const int n = (t ? c1 : c0) + q4;
      if (n >= p.N) continue;  // N is a multiple of 4
      f32x4 v = t ? x1 : x0;
      if (p.R) v += *(const f32x4*)(p.R + (int64_t)m * p.ldr + n);
      *(f32x4*)(p.C + (int64_t)m * p.ldc + n) = v;
    }
  }
}

// C = epilogue(norm(A) W^T).  A workgroup of WM x WN x KW waves: wave tiles of 16*TM rows and U units (32*U columns),
// KW waves share one such tile and split the contraction.  A lane loads four consecutive k of row lane%16 (16 bytes;
// k = 16*chunk + 4*(lane/16) + j feeds MFMA j, the same assignment for both operands), so a chunk of 16 k is
// one load per 16 rows and four MFMAs per tile pair; PF chunks are in flight.  W rows are the MFMA A operand: register r of
// a lane is column 4*(lane/16) + r of row lane%16.
// NORM: the rows are scaled by rsqrt(mean(a^2) + eps) behind the contraction and by the gain in front of it; the sum of
// squares falls out of the loads, every wave (with its KW peers) reads its rows whole.
template <int TM, int U, int WM, int WN, int KW, int PF, bool NORM, int EP, int CT>
__global__ void __launch_bounds__(64 * WM * WN * KW) gemm_fp32_kernel(Fp32Gemm p) {
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = wave % KW, wt = wave / KW, wm = wt % WM, wn = wt / WM;
  const int m0 = (blockIdx.y * WM + wm) * 16 * TM, u0 = (blockIdx.x * WN + wn) * U;
  const float* ap[TM];
  static_assert(CT == 2 || (U == 1 && KW > 1), "the halves of a narrow unit meet in LDS");
  constexpr int NT = CT * U;  // column tiles
  const float* wp[NT];
#pragma unroll
  for (int i = 0; i < TM; ++i) ap[i] = p.A + (int64_t)min(m0 + 16 * i + r16, p.M - 1) * p.lda + 4 * g;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    int c0, c1;
    unit_cols<EP, CT>(p, min(u0 + u, p.units - 1), &c0, &c1);
    if (CT == 1 && r16 >= 8) c0 = c1 - 8;  // row r16 of the tile is column c1 + r16 - 8
    wp[CT * u] = p.W + (int64_t)min(c0 + r16, p.N - 1) * p.ldw + 4 * g;
    if (CT == 2) wp[CT * u + 1] = p.W + (int64_t)min(c1 + r16, p.N - 1) * p.ldw + 4 * g;
  }
  f32x4 acc[TM][NT];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ss[TM] = {};
  f32x4 fa[PF][TM], fw[PF][NT], fg[PF];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const int n_chunks = (p.K + 15) / 16;
  auto load = [&](int s, int c) {
    if (c >= n_chunks) return;  // uniform over the wave
    const bool in = 16 * c + 4 * g < p.K;  // K is a multiple of 4: a lane's four values are all inside or all outside
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[s][i] = in ? *(const f32x4*)(ap[i] + 16 * c) : zero;
#pragma unroll
    for (int j = 0; j < NT; ++j) fw[s][j] = in ? *(const f32x4*)(wp[j] + 16 * c) : zero;
    if (NORM) fg[s] = in ? *(const f32x4*)(p.gain + 16 * c + 4 * g) : zero;
  };
#pragma unroll
  for (int s = 0; s < PF; ++s) load(s, kw + s * KW);
  constexpr int UP = 8 * CT;  // columns of a unit on either side
  // The rotary pairs of a small tile, while the operands arrive: read behind the reduction they cost a round trip to memory,
  // and the table in a launch of its own 3.5 us a call.  The workgroups of head 0 write it for the layers that follow.  Not on
  // the larger tiles: there the registers of the angles leave a compute unit two workgroups instead of three (and the LDS of the
  // pairs three instead of four), in every layer (QKV over 1024 rows, 1536 columns of 512: 50.5 us, with both 60.5; 500 rows 18.2
  // and 20.4).
  constexpr bool PAIRS = EP == EP_ROPE && TM * U == 1;
  __shared__ float2 pairs[PAIRS ? WM * WN : 1][TM][U][16][UP];
  if (PAIRS) {
    const int half = p.dh >> 1, per = half / UP, n_rot = (p.Hq + p.Hkv) * per;
    for (int q = kw * 64 + lane; q < TM * U * 16 * UP; q += KW * 64) {
      const int i = q / (U * 16 * UP), u = q / (16 * UP) % U, row = q / UP % 16, m = m0 + 16 * i + row, k = (u0 + u) % per * UP + q % UP;
      if (m >= p.M || u0 + u >= n_rot) continue;
      if (p.job.cs) {
        const float2 c = rope_pair(p.job, m, k);
        if (u0 + u < per) p.job.cs[(int64_t)m * half + k] = c;
        pairs[wt][i][u][row][q % UP] = c;
      } else {
        pairs[wt][i][u][row][q % UP] = p.cs[(int64_t)m * half + k];
      }
    }
  }
  for (int c = kw; c < n_chunks; c += PF * KW) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      if (c + s * KW < n_chunks) {
        if (NORM) {
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const f32x4 x = fa[s][i];
            ss[i] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
            fa[s][i] = x * fg[s];
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[s][j][k], fa[s][i][k], acc[i][j], 0, 0, 0);
        load(s, c + (s + PF) * KW);
      }
    }
  }
  if (NORM) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      ss[i] += __shfl_xor(ss[i], 16, 64);
      ss[i] += __shfl_xor(ss[i], 32, 64);
    }
  }
  const float inv_k = 1.0f / (float)p.K;
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + 16 * i + r16;
      if (m >= p.M) continue;
      const float rs = NORM ? 1.0f / sqrtf(ss[i] * inv_k + p.eps) : 1.0f;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u0 + u < p.units) {
          const int half = p.dh >> 1;
          const float2* cs = EP == EP_ROPE ? p.cs + (int64_t)m * half + (u0 + u) * 16 % half + 4 * g : nullptr;
          unit_store<EP, 2>(p, m, u0 + u, 4 * g, acc[i][2 * u] * rs, acc[i][2 * u + 1] * rs, cs);
        }
    }
  } else {
    // partial sums of the KW waves meet in LDS and are added in wave order
    __shared__ f32x4 red[WM * WN][KW][TM * NT][64];
    __shared__ float red_ss[WM * WN][KW][TM * 16];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < NT; ++j) red[wt][kw][i * NT + j][lane] = acc[i][j];
      if (NORM && g == 0) red_ss[wt][kw][i * 16 + r16] = ss[i];
    }
    __syncthreads();
    for (int it = kw; it < TM * U; it += KW) {  // (row block, unit) pairs go round the KW waves
      const int i = it / U, u = it % U, m = m0 + 16 * i + r16;
      if (m >= p.M || u0 + u >= p.units) continue;
      constexpr bool MEET = CT == 1 && EP != EP_PLAIN;  // two lanes' sums are one lane's unit
      if (MEET && g >= 2) continue;
      const int j0 = i * NT + CT * u, j1 = CT == 2 ? j0 + 1 : j0, l1 = MEET ? lane + 32 : lane;
      f32x4 x0 = red[wt][0][j0][lane], x1 = red[wt][0][j1][l1];
      float s = NORM ? red_ss[wt][0][i * 16 + r16] : 0.f;
#pragma unroll
      for (int k = 1; k < KW; ++k) {
        x0 += red[wt][k][j0][lane];
        if (CT == 2 || MEET) x1 += red[wt][k][j1][l1];
        if (NORM) s += red_ss[wt][k][i * 16 + r16];
      }
      const float rs = NORM ? 1.0f / sqrtf(s * inv_k + p.eps) : 1.0f;
      const float2* cs = PAIRS           ? &pairs[wt][i][u][r16][4 * g]
                         : EP == EP_ROPE ? p.cs + (int64_t)m * (p.dh >> 1) + (u0 + u) * UP % (p.dh >> 1) + 4 * g
                                         : nullptr;
      unit_store<EP, CT>(p, m, u0 + u, 4 * g, x0 * rs, x1 * rs, cs);
    }
  }
}

template <int TM, int U, int WM, int WN, int KW, int PF, bool NORM, int EP, int CT = 2>
hipError_t launch_tiled(const Fp32Gemm& p, hipStream_t s) {
  const dim3 grid((p.units + U * WN - 1) / (U * WN), (p.M + 16 * TM * WM - 1) / (16 * TM * WM));
  hipLaunchKernelGGL((gemm_fp32_kernel<TM, U, WM, WN, KW, PF, NORM, EP, CT>), grid, dim3(64 * WM * WN * KW), 0, s, p);
  return hipGetLastError();
}

// Three tilings, by how many workgroups a problem has: 128 x 128 per workgroup (64 x 64 wave tiles, the matrix pipe
// is the bound) once that makes 256 of them, one per compute unit; 16 x 32 with the contraction split over eight waves
// while that stays within 1024, four per compute unit (latency is the bound); 32 x 64 over four waves in between.
enum { FP32_LARGE, FP32_MEDIUM, FP32_SMALL };
int fp32_tiling(const Fp32Gemm& p) {
  auto groups = [&](int rows, int units) { return (int64_t)((p.M + rows - 1) / rows) * ((p.units + units - 1) / units); };
  return groups(128, 4) >= 256 ? FP32_LARGE : groups(16, 1) <= 1024 ? FP32_SMALL : FP32_MEDIUM;
}
template <bool NORM, int EP>
hipError_t launch_fp32(const Fp32Gemm& p, hipStream_t s) {
  switch (fp32_tiling(p)) {
    case FP32_LARGE: return launch_tiled<4, 2, 2, 2, 1, 2, NORM, EP>(p, s);
    case FP32_SMALL:
      // One column tile a workgroup while that leaves no compute unit a second one: half the matrix instructions behind one
      // another, which is what a wave of these takes longest for (16 rows of the fp32 workload, us: down 5.7 -> 4.5, O 3.9 ->
      // 3.7, QKV 4.9 -> 4.5, gate/up 4.9 -> 4.4).
      if ((int64_t)((p.M + 15) / 16) * p.units * 2 <= 256) {
        Fp32Gemm q = p;
        q.units *= 2;
        return launch_tiled<1, 1, 1, 1, 8, 3, NORM, EP, 1>(q, s);
      }
      return launch_tiled<1, 1, 1, 1, 8, 3, NORM, EP>(p, s);
    default: return launch_tiled<2, 2, 1, 1, 4, 2, NORM, EP>(p, s);
  }
}

// Causal attention, one workgroup per 16 queries of one (sequence, q head); its NW waves take every NW-th chunk of
// 32 keys with a running softmax of their own and merge through LDS in wave order.  Scores are computed transposed
// (keys are the MFMA rows), so a lane owns one query (lane%16) and four keys of a 16-key tile (4*(lane/16) + r), which is
// the operand layout of P^T in O^T += V^T P^T: register r feeds MFMA r, with V read as rows 4*(lane/16) + r.
template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW) attn_fp32_kernel(const float* __restrict__ q, int64_t ldq, const float* __restrict__ k_rows,
                                                        const float* __restrict__ v_rows, float* __restrict__ out,
                                                        const int32_t* __restrict__ q_cu, const int32_t* __restrict__ p_cu,
                                                        int n_seqs, int64_t own_row0, int Hq, int Hkv) {
  constexpr int NC = DH / 16;
  extern __shared__ f32x4 red_o[];  // [NW][NC][64]
  __shared__ float red_m[NW][16], red_l[NW][16];
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int head = blockIdx.y, kvh = head / (Hq / Hkv);
  int tile = blockIdx.x, b = 0, q_begin = 0, q_end = 0;
  for (;; ++b) {
    q_begin = q_cu[b];
    q_end = q_cu[b + 1];
    const int nt = (q_end - q_begin + 15) / 16;
    if (tile < nt || b + 1 >= n_seqs) break;
    tile -= nt;
  }
  const int q0 = q_begin + 16 * tile;
  if (q0 >= q_end) return;
  const int qi = min(q0 + r16, q_end - 1);
  const int64_t ldkv = (int64_t)Hkv * DH;
  const int64_t pre0 = p_cu ? p_cu[b] : 0;
  const int n_pre = p_cu ? p_cu[b + 1] - p_cu[b] : 0;
  const int64_t own0 = own_row0 + q_begin;
  const int visible = n_pre + qi - q_begin + 1;                        // keys this lane's query sees
  const int n_keys = n_pre + min(q0 + 15, q_end - 1) - q_begin + 1;    // keys of the workgroup
  auto row_of = [&](int j) { return j < n_pre ? pre0 + j : own0 + (j - n_pre); };

  const float scale = 1.0f / sqrtf((float)DH);
  f32x4 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) qf[c] = *(const f32x4*)(q + (int64_t)qi * ldq + head * DH + 16 * c + 4 * g) * scale;
  f32x4 o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  for (int j0 = 32 * wave; j0 < n_keys; j0 += 32 * NW) {
    f32x4 kf[2][NC];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float* kp = k_rows + row_of(min(j0 + 16 * t + r16, n_keys - 1)) * ldkv + kvh * DH + 4 * g;
#pragma unroll
      for (int c = 0; c < NC; ++c) kf[t][c] = *(const f32x4*)(kp + 16 * c);
    }
    float vf[2][4][NC];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* vp = v_rows + row_of(min(j0 + 16 * t + 4 * g + r, n_keys - 1)) * ldkv + kvh * DH + r16;
#pragma unroll
        for (int c = 0; c < NC; ++c) vf[t][r][c] = vp[16 * c];
      }
    // (All 32 keys, also where the chunk has 16 or fewer: with a branch around the second 16, 1024 keys took 37.8 us instead of
    // 34.9 and 128 keys 6.3 instead of 5.9, heads of 64; 144 keys 6.4 instead of 6.8.)
    f32x4 s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][c][k], qf[c][k], s[t], 0, 0, 0);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (j0 + 16 * t + 4 * g + r >= visible) s[t][r] = -INFINITY;
        mx = fmaxf(mx, s[t][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx);
    const float m_safe = m_new == -INFINITY ? 0.f : m_new;  // no key of this wave is visible to the query yet
    const float corr = expf(m - m_safe);
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[t][r] = expf(s[t][r] - m_safe);
        sum += s[t][r];
      }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    l = l * corr + sum;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] *= corr;
    // A probability of 0 takes a key out of the product only while its V row is finite: where a chunk holds keys that
    // some of the 16 queries may not see, and one of its rows is not, the sum is taken key by key instead.
    bool by_key = false;
    if (j0 + 31 >= n_pre + q0 - q_begin + 1) {  // uniform: past what the first query sees
      float z = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < NC; ++c) z = fmaf(vf[t][r][c], 0.f, z);
      by_key = __builtin_amdgcn_ballot_w64(z != 0.f) != 0;
    }
    if (!by_key) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][r][c], s[t][r], o[c], 0, 0, 0);
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          for (int gg = 0; gg < 4; ++gg) {
            const int j = j0 + 16 * t + 4 * gg + r;
            const float pj = __shfl(s[t][r], 16 * gg + r16, 64);
            if (j < visible) {
              const float* vp = v_rows + row_of(j) * ldkv + kvh * DH + 4 * g;
#pragma unroll
              for (int c = 0; c < NC; ++c) o[c] += *(const f32x4*)(vp + 16 * c) * pj;
            }
          }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) red_o[(wave * NC + c) * 64 + lane] = o[c];
  if (g == 0) {
    red_m[wave][r16] = m;
    red_l[wave][r16] = l;
  }
  __syncthreads();
  if (q0 + r16 >= q_end) return;
  float M = red_m[0][r16];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmaxf(M, red_m[w][r16]);  // finite: wave 0 holds key 0, which every query sees
  float wgt[NW], den = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wgt[w] = expf(red_m[w][r16] - M);
    den += red_l[w][r16] * wgt[w];
  }
  const float inv = 1.0f / den;
  for (int c = wave; c < NC; c += NW) {
    f32x4 x = red_o[c * 64 + lane] * wgt[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) x += red_o[(w * NC + c) * 64 + lane] * wgt[w];
    *(f32x4*)(out + (int64_t)qi * Hq * DH + head * DH + 16 * c + 4 * g) = x * inv;
  }
}

bool rows16(const void* p, int64_t ld) { return (((uintptr_t)p) & 15) == 0 && (ld & 3) == 0; }

Fp32Gemm plain_args(const void* A, int64_t lda, const void* W, int64_t ldw, void* C, int64_t ldc, int M, int N, int K) {
  Fp32Gemm p = {};
  p.A = (const float*)A; p.lda = lda; p.W = (const float*)W; p.ldw = ldw; p.C = (float*)C; p.ldc = ldc;
  p.M = M; p.N = N; p.K = K; p.units = (N + 31) / 32;
  return p;
}

}  // namespace

// Rows must be whole 16-byte pieces (K, N and all strides multiples of 4 elements); what is not runs on the plain-ALU
// kernel.  65535: the grid's row dimension, in the smallest row tile.
bool gemm_fp32_supported(const void* A, int64_t lda, const void* W, int64_t ldw, const void* C, int64_t ldc, const void* R,
                         int64_t ldr, int M, int N, int K) {
  return K % 4 == 0 && N % 4 == 0 && rows16(A, lda) && rows16(W, ldw) && rows16(C, ldc) && (!R || rows16(R, ldr)) &&
         M <= 16 * 65535;
}

hipError_t launch_gemm_fp32(const void* A, int64_t lda, const void* W, int64_t ldw, void* C, int64_t ldc, const void* R,
                            int64_t ldr, int M, int N, int K, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  Fp32Gemm p = plain_args(A, lda, W, ldw, C, ldc, M, N, K);
  p.R = (const float*)R; p.ldr = ldr;
  return launch_fp32<false, EP_PLAIN>(p, s);
}

// Whether QKV over M rows runs on the tiling that can fill the rotary table as well.
bool gemm_fp32_takes_rope(int M, int Hq, int Hkv, int dh) {
  Fp32Gemm p = {};
  p.M = M; p.units = ((Hq + 2 * Hkv) * dh + 31) / 32;
  return fp32_tiling(p) == FP32_SMALL;
}

// job (gemm_fp32_takes_rope): fill the rotary table cs on the way
hipError_t launch_gemm_fp32_norm_rope(const float* h, const void* gain, float eps, const void* wqkv, void* qkv, const float2* cs,
                                      void* k_rows, void* v_rows, int M, int d, int Hq, int Hkv, int dh, const RopeJob* job, hipStream_t s) {
  const int N = (Hq + 2 * Hkv) * dh;
  Fp32Gemm p = plain_args(h, d, wqkv, d, qkv, N, M, N, d);
  p.gain = (const float*)gain; p.eps = eps;
  p.cs = cs; p.k_rows = (float*)k_rows; p.v_rows = (float*)v_rows; p.Hq = Hq; p.Hkv = Hkv; p.dh = dh;
  if (job) p.job = *job;
  return launch_fp32<true, EP_ROPE>(p, s);
}

hipError_t launch_gemm_fp32_norm_swiglu(const float* h, const void* gain, float eps, const void* wgu, void* act, int M, int d,
                                        int F, int gu_block, hipStream_t s) {
  Fp32Gemm p = plain_args(h, d, wgu, d, act, F, M, 2 * F, d);
  p.gain = (const float*)gain; p.eps = eps; p.gu_block = gu_block; p.units = F / 16;
  return launch_fp32<true, EP_SWIGLU>(p, s);
}

bool attn_fp32_supported(const AttnArgs& a) {
  return (a.dh == 64 || a.dh == 128) && rows16(a.q, a.ldq) && rows16(a.k_rows, 4) && rows16(a.v_rows, 4) && rows16(a.out, 4);
}

hipError_t launch_attn_fp32(const AttnArgs& a, hipStream_t s) {
  if (a.n_q <= 0) return hipSuccess;
  int64_t tiles = 0;
  int max_keys = 0;
  for (int b = 0; b < a.n_seqs; ++b) {
    const int len = a.q_cu_host[b + 1] - a.q_cu_host[b], keys = len + (a.p_cu_host ? a.p_cu_host[b + 1] - a.p_cu_host[b] : 0);
    tiles += (len + 15) / 16;
    if (keys > max_keys) max_keys = keys;
  }
  // Waves of a workgroup, a chunk of 32 keys each: four while that takes them one chunk.  Past that eight shorten the chain of
  // chunks, which pays where it is what a launch takes: with heads of 128 always (four waves' registers leave one workgroup a
  // compute unit, so eight are twice as many in flight), with heads of 64 while no compute unit gets a second workgroup
  // (three of four waves fit there, one of eight).  Four -> eight waves, us:
  //   heads of 64: 144 keys, 36 workgroups 7.9 -> 6.8, 252 8.7 -> 7.7, 288 9.7 -> 10.7, 2304 34.0 -> 57.9;  512 keys, 256 workgroups
  //   13.8 -> 12.4;  1024 keys, 256 workgroups 22.9 -> 20.3, 512 34.9 -> 37.0
  //   heads of 128: 144 keys, 36 workgroups 12.6 -> 10.9, 2304 94.9 -> 91.1;  1024 keys, 512 workgroups 78.0 -> 66.8
  const bool eight = max_keys > 128 && (a.dh == 128 || tiles * a.Hq <= 256);
  auto launch = [&](auto kern, int nw) -> hipError_t {
    const int lds = nw * a.dh / 16 * 1024;
    if (lds > 48 << 10) {
      const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, a.Hq), dim3(64 * nw), lds, s, (const float*)a.q, a.ldq, (const float*)a.k_rows,
                       (const float*)a.v_rows, (float*)a.out, a.q_cu, a.p_cu, a.n_seqs, a.own_row0, a.Hq, a.Hkv);
    return hipGetLastError();
  };
  if (eight) return a.dh == 64 ? launch(attn_fp32_kernel<64, 8>, 8) : launch(attn_fp32_kernel<128, 8>, 8);
  return a.dh == 64 ? launch(attn_fp32_kernel<64, 4>, 4) : launch(attn_fp32_kernel<128, 4>, 4);
}
