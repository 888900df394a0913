// Attention of few queries (at most 128 per sequence against a long cache: the suffix pass, a generation step; or the prefill
// of a short prompt), bf16.
//
// Bound: the rate at which K and V arrive from HBM, and how soon the first of them do; then the softmax arithmetic of the
// resident wave or two per SIMD.  So: the q heads of a kv group and their queries form one list of columns (query-major)
// that is cut into 16-column MFMA tiles, and a workgroup reads K and V of its key range once for all of its columns; the key
// ranges are cut so that about 256 workgroups run; K and V go to a ring of LDS stages by direct loads (heads of 128: two stages of
// 64 KB, both in flight at the start, one beside the stage in work from then on); V is read from LDS through the transposing read, so no transposed copy of the prefix is
// made (it was a launch of its own over all prefix rows).
// Scores are transposed, S^T = K Q^T on v_mfma_f32_16x16x32_bf16: a lane owns one column and keys 4*(lane/16) + r of a
// 16-key tile.  The contraction index of O^T += V^T P^T is numbered so that the two key tiles of a 32-key step are the
// lane's eight values as they stand: index 8g + e is key 16*(e/4) + 4g + e%4, and the V operand follows with two transposing
// reads of four keys each.
// 8B shape, per layer, against a transposed copy and 32x32x16 tiles before: 64 queries and 8192 keys 21.2 us (31), one query and
// 4096 keys 7.2 us (17), and the merge of the key ranges 5 us in both.  Of the 21.2 us the loads alone take 10, the partial
// outputs 4; runs of 64 keys per wave and stage (two independent steps to schedule) instead of 32 took 25 -> 22.5 us, four column
// tiles per wave with one wave per SIMD take 35.
// 128 queries for each of eight sequences of 1k to 8k keys: 153 us, one key range per workgroup (before: transposed copy 35,
// attention 153, merge 15).  The sequences have 26 to 63 stages and one key range each, so the launch lasts as long as the longest of
// them: an even share would be 50 stages.
#include <math.h>

#include <type_traits>

#include "dsk_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// the top bit of each bf16 half of x: set where the half is Inf or NaN (exponent all ones)
__device__ __forceinline__ uint32_t non_finite(uint32_t x) { return ((x & 0x7F807F80u) + 0x00800080u) & 0x80008000u; }

struct FewParams {
  const bf16_t* q; int64_t ldq;
  const bf16_t* k; const bf16_t* v;
  bf16_t* out; int out_blocks;
  float* part_o; float* part_ml;  // splits > 1: [n_q][Hq][splits][dh], [n_q][Hq][splits][2]
  const int32_t* q_cu; const int32_t* p_cu;
  int n_seqs; int own_row0; int Hq, Hkv; int splits; int range;  // key ranges: `splits` of `range` stages each
  float c;  // softmax scale * log2(e)
};

// QG groups of waves take 16*QT columns each, the KH waves of a group every KH-th run of 32*KS keys of a stage; NST stages in the
// ring.
template <int DH, int QT, int QG, int KH, int KS, int NST>
__global__ void __launch_bounds__(64 * QG * KH) attn_few_kernel(FewParams p) {
  constexpr int NW = QG * KH, KW = 32 * KS, KEYS = KW * KH;  // keys per wave and per stage
  constexpr int SLOTS = DH / 8, RPI = 64 / SLOTS;  // 16-byte slots per row, rows per wave load
  constexpr int INST = KEYS / RPI / NW;            // loads per wave, stage and matrix
  constexpr int NKS = DH / 32, NDT = DH / 16;
  static_assert(KEYS % (RPI * NW) == 0, "stage / wave mismatch");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ int v_cleared[NW];         // the wave has cleared elements of V (below)
  bf16_t* sK = (bf16_t*)smem_raw;       // [NST][KEYS][DH]
  bf16_t* sV = sK + NST * KEYS * DH;    // [NST][KEYS][DH]
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave % QG, kh = wave / QG;
  const int G = p.Hq / p.Hkv;

  // kv head innermost: with eight of them each die serves one, and the column blocks of a key range share its L2
  const int kvh = blockIdx.x % p.Hkv, z = blockIdx.x / p.Hkv % p.splits;
  int blk = blockIdx.x / p.Hkv / p.splits, b = 0, q_begin = 0, q_len = 0;
  constexpr int COLS = 16 * QT * QG;
  for (;; ++b) {
    q_begin = p.q_cu[b];
    q_len = p.q_cu[b + 1] - q_begin;
    const int nb = (q_len * G + COLS - 1) / COLS;
    if (blk < nb || b + 1 >= p.n_seqs) break;
    blk -= nb;
  }
  const int n_cols = q_len * G;
  if (blk * COLS >= n_cols) return;  // cannot happen for a well-formed grid
  const int pre_begin = p.p_cu ? p.p_cu[b] : 0, n_pre = p.p_cu ? p.p_cu[b + 1] - pre_begin : 0;
  const int own_begin = p.own_row0 + q_begin;
  const int n_keys = n_pre + min(n_cols - 1, blk * COLS + COLS - 1) / G + 1;  // keys some column of the workgroup sees
  // stages of this key range
  const int n_stages_all = (n_keys + KEYS - 1) / KEYS;
  const int st0 = min(z * p.range, n_stages_all), st1 = min(st0 + p.range, n_stages_all);
  // the first of them with a key that some column does not see
  const int st_masked = max(st0, (n_pre + blk * COLS / G + 1) / KEYS);

  const int ldkv = p.Hkv * DH;
  const bf16_t* kb = p.k + kvh * DH;
  const bf16_t* vb = p.v + kvh * DH;
  const uint32_t sK_lds = (uint32_t)(uintptr_t)sK, sV_lds = (uint32_t)(uintptr_t)sV;
  // Slot swizzles, applied where a row is fetched.  K: 16 lanes read one slot of 16 consecutive rows.  V: 32 lanes of the
  // transposing read take a 32-byte pair of slots from each of 8 consecutive rows.
  auto kswz = [](int row) { return DH == 128 ? row & 15 : (row >> 1) & 7; };
  auto vswz = [](int row) { return DH == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1; };
  auto load_to = [](uint32_t dst, const void* src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(src) : "memory", "m0");
  };
  // A stage inside the prefix: the lanes' byte offsets from its first row are those of every stage, so its loads take a scalar base and
  // no arithmetic per lane.  (The swizzles repeat after KP and VP loads of RPI rows.)
  constexpr int KP = INST < 16 / RPI ? INST : 16 / RPI, VP = INST < 8 / RPI ? INST : 8 / RPI;
  uint32_t k_off[KP], v_off[VP];
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    const int r = RPI * (wave * INST + i) + lane / SLOTS;
    k_off[i] = (uint32_t)(r * ldkv + (lane % SLOTS ^ kswz(r)) * 8) * 2u;
  }
#pragma unroll
  for (int i = 0; i < VP; ++i) {
    const int r = RPI * (wave * INST + i) + lane / SLOTS;
    v_off[i] = (uint32_t)(r * ldkv + (lane % SLOTS ^ vswz(r)) * 8) * 2u;
  }
  auto load_off = [](uint32_t dst, uint32_t off, const void* base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(base) : "memory", "m0");
  };
  auto issue = [&](int st) {
    const uint32_t at = (uint32_t)(((st - st0) % NST * KEYS + RPI * wave * INST) * DH) * 2u;
    if ((st + 1) * KEYS <= n_pre) {
      const int64_t row0 = (int64_t)(pre_begin + st * KEYS) * ldkv;
#pragma unroll
      for (int i = 0; i < INST; ++i) {
        load_off(sK_lds + at + i * 1024, k_off[i % KP], kb + row0 + (int64_t)(i / KP * KP) * RPI * ldkv);
        load_off(sV_lds + at + i * 1024, v_off[i % VP], vb + row0 + (int64_t)(i / VP * VP) * RPI * ldkv);
      }
    } else {
      int lane_s = lane;
      asm volatile("" : "+v"(lane_s));  // nothing of this path is kept in registers over the loop
#pragma unroll
      for (int i = 0; i < INST; ++i) {
        const int r = RPI * (wave * INST + i) + lane_s / SLOTS, s = lane_s % SLOTS;
        const int j = min(st * KEYS + r, n_keys - 1);  // rows past the end repeat the last one and are masked
        const int64_t row = j < n_pre ? pre_begin + j : own_begin + (j - n_pre);
        load_to(sK_lds + at + i * 1024, kb + row * ldkv + (s ^ kswz(r)) * 8);
        load_to(sV_lds + at + i * 1024, vb + row * ldkv + (s ^ vswz(r)) * 8);
      }
    }
  };

  // columns of this wave: column index -> query col / G, q head kvh * G + col % G
  bf16x8 qf[QT][NKS];
  int visible[QT], qrow[QT], head[QT];
  bool active = false;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int first = blk * COLS + (qg * QT + t) * 16, col = min(first + r16, n_cols - 1);
    active |= first < n_cols;
    qrow[t] = q_begin + col / G;
    head[t] = kvh * G + col % G;
    visible[t] = n_pre + col / G + 1;
    const bf16_t* qp = p.q + (int64_t)qrow[t] * p.ldq + head[t] * DH + 8 * g;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[t][ks] = *(const bf16x8*)(qp + 32 * ks);
  }
  f32x4 o[QT][NDT];
  float m[QT], l[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int cleared = 0;
  // The queries first, waited for alone: the compiler does not see the direct loads, and its own wait would otherwise be
  // for all of the ring.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
#pragma unroll
  for (int s = 0; s < NST; ++s)
    if (st0 + s < st1) issue(st0 + s);

  constexpr int PER = 2 * INST;  // loads per wave and stage
  for (int st = st0; st < st1; ++st) {
    // the stages behind this one may still be in flight
    const int behind = min(st == st0 ? NST - 1 : NST - 2, st1 - 1 - st);
    if (behind >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * PER) : "memory");
    else if (behind == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
    else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int stage = (st - st0) % NST, key0 = st * KEYS + KW * kh;
    // A probability of 0 takes a key out of O only while its V row is finite.  In stages that not every column sees whole, a
    // wave clears the elements that are not finite in the rows it has loaded itself; the columns that see them get them at the end.
    // (Suffix pass of one row, 8B: 95.8 -> 96.2 us a layer; of 64 rows 135.9 -> 136.1 us.)
    if (st >= st_masked) {
      bf16_t* mine = sV + (stage * KEYS + RPI * wave * INST) * DH + lane * 8;
      u32x4 x[INST];
      uint32_t any = 0;
#pragma unroll
      for (int i = 0; i < INST; ++i) {
        x[i] = *(const u32x4*)(mine + i * 512);
        any |= non_finite(x[i][0]) | non_finite(x[i][1]) | non_finite(x[i][2]) | non_finite(x[i][3]);
      }
      if (__builtin_amdgcn_ballot_w64(any != 0) != 0) {
#pragma unroll
        for (int i = 0; i < INST; ++i) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t t = non_finite(x[i][e]);
            x[i][e] &= ~(t | (t - (t >> 15)));
          }
          *(u32x4*)(mine + i * 512) = x[i];
        }
        cleared = 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
    // The one barrier of a stage: the stage is there for every wave, and every wave is past the one in front (its reads have
    // returned), which takes the next loads.  With a second barrier behind the MFMAs, and addresses worked out per lane: 8 x 128
    // queries (49523 keys in all) 174 us instead of 153, 4 x 100 queries and 4096 keys each 51.6 instead of 46.0, 64 queries and
    // 8192 keys 21.8 instead of 21.2.  What bounds it now, one thing left out at a time (timing only): no tile loads 0.83 of the time,
    // no reads of K 0.87, no exponentials 0.95, no reads of V 1.0.  Measured without gain: the scores of the next stage beside the
    // exponentials of this one (153 us, and 3 us more at the start), fragments read four or six ahead of their MFMAs.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (st > st0 && st + NST - 1 < st1) issue(st + NST - 1);
    if (active && key0 < n_keys) {
      const bf16_t* kt = sK + (stage * KEYS + KW * kh) * DH;
      const bf16_t* vt = sV + (stage * KEYS + KW * kh) * DH;
      // Straight-line stretches, the rare cases (masks, a moving reference) in branches between them, so that the
      // scheduler can run exponentials, V reads and MFMAs of the wave's steps side by side.
      f32x4 s[QT][2 * KS];
      float mx[QT];
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int h = 0; h < 2 * KS; ++h) s[t][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 2 * KS; ++h)
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const int row = 16 * h + r16;
          const bf16x8 kf = *(const bf16x8*)(kt + row * DH + ((4 * ks + g) ^ kswz(row)) * 8);
#pragma unroll
          for (int t = 0; t < QT; ++t) s[t][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[t][ks], s[t][h], 0, 0, 0);
        }
      if (key0 + KW > n_pre) {  // own rows (or the end) among the keys: a mask per column
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
          for (int h = 0; h < 2 * KS; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (key0 + 16 * h + 4 * g + r >= visible[t]) s[t][h][r] = -INFINITY;
      }
      bool moves = false;
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        mx[t] = s[t][0][0];
#pragma unroll
        for (int h = 0; h < 2 * KS; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx[t] = fmaxf(mx[t], s[t][h][r]);
        moves |= !((mx[t] - m[t]) * p.c <= 8.0f);
      }
      // The exponentials' reference follows the true maximum only when that exceeds it by more than 2^8 in the exponent
      // (attn_mfma.hip), so as long as no lane sees that the four lanes of a column need not agree on the maximum.
      if (__builtin_amdgcn_ballot_w64(moves) != 0) {
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          float x = fmaxf(mx[t], __shfl_xor(mx[t], 16, 64));
          x = fmaxf(x, __shfl_xor(x, 32, 64));
          const float m_true = fmaxf(m[t], x);
          const bool keep = (m_true - m[t]) * p.c <= 8.0f;  // false for m = -inf
          const float m_new = keep ? m[t] : m_true;
          const float alpha = keep ? 1.0f : __builtin_amdgcn_exp2f((m[t] - (m_new == -INFINITY ? 0.f : m_new)) * p.c);
          l[t] *= alpha;
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) o[t][dt] *= alpha;
          m[t] = m_new;
        }
      }
      bf16x8 pf[QT][KS];
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const float mc = m[t] == -INFINITY ? 0.f : m[t] * p.c;
#pragma unroll
        for (int h = 0; h < 2 * KS; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float e = __builtin_amdgcn_exp2f(s[t][h][r] * p.c - mc);
            l[t] += e;
            pf[t][h / 2][4 * (h % 2) + r] = (bf16_t)e;
          }
      }
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          // lane i of a group of 16 names 8 bytes of row i/4 and receives column i of the four rows
          s16x4 vf[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int row = 32 * k + 16 * h + 4 * g + (r16 >> 2), slot = 2 * dt + ((r16 & 3) >> 1);
            const bf16_t* src = vt + row * DH + (slot ^ vswz(row)) * 8 + (r16 & 1) * 4;
            vf[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)src);
          }
          typedef __attribute__((ext_vector_type(8))) short s16x8;
          const bf16x8 vfrag = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[0], vf[1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
          for (int t = 0; t < QT; ++t) o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfrag, pf[t][k], o[t][dt], 0, 0, 0);
        }
    }
  }

  // What the clearing took out: a visible key of any weight makes its column's sum Inf or NaN.
  if (lane == 0) v_cleared[wave] = cleared;
  __syncthreads();
  int any_cleared = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) any_cleared |= v_cleared[w];
  if (any_cleared) {
    for (int st = st_masked; st < st1; ++st)
      for (int j = st * KEYS + KW * kh, end = min(j + KW, n_keys); j < end; ++j) {
        const bf16_t* row = vb + (int64_t)(j < n_pre ? pre_begin + j : own_begin + (j - n_pre)) * ldkv + 4 * g;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const bf16x4 v = *(const bf16x4*)(row + 16 * dt);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = (float)v[e];
#pragma unroll
            for (int t = 0; t < QT; ++t)
              if (!(fabsf(x) < INFINITY) && j < visible[t]) o[t][dt][e] += x;
          }
        }
      }
  }

  // the KH waves of a group merge through LDS (the ring is idle), each its share of the output columns
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    l[t] += __shfl_xor(l[t], 16, 64);
    l[t] += __shfl_xor(l[t], 32, 64);
  }
  f32x4* red = (f32x4*)smem_raw;                    // [QG][KH][NDT][64]
  float2* red_ml = (float2*)(red + NW * NDT * 64);  // [QG][KH][16]
#pragma unroll
  for (int t = 0; t < QT; ++t) {  // one column tile at a time
    __syncthreads();
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) red[((qg * KH + kh) * NDT + dt) * 64 + lane] = o[t][dt];
    if (g == 0) red_ml[(qg * KH + kh) * 16 + r16] = make_float2(m[t], l[t]);
    __syncthreads();
    if (blk * COLS + (qg * QT + t) * 16 + r16 < n_cols) {
      float M = -INFINITY, den = 0.f, w[KH];
#pragma unroll
      for (int k = 0; k < KH; ++k) M = fmaxf(M, red_ml[(qg * KH + k) * 16 + r16].x);
      const float m_safe = M == -INFINITY ? 0.f : M;
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        const float2 ml = red_ml[(qg * KH + k) * 16 + r16];
        w[k] = __builtin_amdgcn_exp2f((ml.x - m_safe) * p.c);
        den += ml.y * w[k];
      }
      const int64_t qh = (int64_t)qrow[t] * p.Hq + head[t];
      const float inv = 1.0f / den;
      if (st0 < st1) {  // a range past this sequence's keys only says so (m = -inf): nothing reads its outputs
        for (int dt = kh; dt < NDT; dt += KH) {
          f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < KH; ++k) x += red[((qg * KH + k) * NDT + dt) * 64 + lane] * w[k];
          const int d = 16 * dt + 4 * g;
          if (p.splits > 1) {
            *(f32x4*)(p.part_o + (qh * p.splits + z) * DH + d) = x;
          } else {
            x *= inv;
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (bf16_t)x[e];
            *(bf16x4*)(p.out + (p.out_blocks ? block_at(qrow[t], head[t] * DH + d, p.Hq * DH) : qh * DH + d)) = v;
          }
        }
      }
      if (p.splits > 1 && kh == 0 && g == 0) *(float2*)(p.part_ml + (qh * p.splits + z) * 2) = make_float2(M, den);
    }
  }
}

template <int DH, int QT, int QG, int KH, int KS, int NST>
hipError_t launch_few(const FewParams& p, int64_t blocks, hipStream_t s) {
  auto kern = attn_few_kernel<DH, QT, QG, KH, KS, NST>;
  constexpr int ring = NST * 32 * KS * KH * DH * 2 * 2, merge = QG * KH * (DH / 16 * 1024 + 128);
  constexpr int lds = ring > merge ? ring : merge;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  DSK_LAUNCH_TIMED(kern, dim3((unsigned)blocks), dim3(64 * QG * KH), lds, s, p);
  return hipGetLastError();
}

}  // namespace

// Sequences of at most 128 queries; or a call too small to fill the chip with the 128-query workgroups of attn_mfma.hip (at
// most 256 of them, up to 1024 queries) over short key ranges: there the transposed copy, a launch of its own, and the
// latency of few wide workgroups weigh more.  A layer of the 8B shape over one prompt of 333 / 512 / 768 / 1024 tokens:
// 241 -> 240, 289 -> 278, 399 -> 384, 472 -> 458 us; a 70B layer over 512 tokens 793 -> 776 us.  Past it the 32-query waves of
// attn_mfma.hip do more per LDS read: 2048 tokens 798 there, 812 here, 8 x 512 tokens 1375 and 1389 us.
// A chunked layer's later chunks need the transposed rows of this one.
bool attn_few_supported(const AttnArgs& a) {
  if ((a.dh != 128 && a.dh != 64) || (a.ldq & 7) || a.own_row0 + a.n_q >= ((int64_t)1 << 31) || a.keep_vt) return false;
  const bool small = a.n_q <= 1024 && (int64_t)a.n_q * a.Hq <= 256 * 128;
  for (int b = 0; b < a.n_seqs; ++b) {
    const int len = a.q_cu_host[b + 1] - a.q_cu_host[b];
    if (len > 128 && (!small || len + (a.p_cu_host ? a.p_cu_host[b + 1] - a.p_cu_host[b] : 0) > 1024)) return false;
  }
  return true;
}

hipError_t launch_attn_few(const AttnArgs& a, int* splits_out, hipStream_t s) {
  if (a.n_q <= 0) return hipSuccess;
  const int G = a.Hq / a.Hkv;
  int max_len = 0;
  int64_t max_keys = 0;
  for (int b = 0; b < a.n_seqs; ++b) {
    const int len = a.q_cu_host[b + 1] - a.q_cu_host[b];
    const int64_t keys = len + (a.p_cu_host ? a.p_cu_host[b + 1] - a.p_cu_host[b] : 0);
    if (len > max_len) max_len = len;
    if (keys > max_keys) max_keys = keys;
  }
  // columns per workgroup: 16 (four waves share the keys), 64, or 128 (32 per wave: a fragment feeds two MFMAs)
  const int cols = max_len * G <= 16 ? 16 : max_len * G <= 64 ? 64 : 128;
  const int max_stages = (int)((max_keys + 127) / 128);  // every form has stages of 128 keys
  // Key ranges, the same length for all sequences (short ones leave the last ranges empty): the length that by this count
  // ends first, with one workgroup per compute unit, 4 us for a workgroup's start and end, 3 us per stage (1 us with 16
  // columns) and the partial outputs written and read at 5 TB/s.
  int splits = 1, range = max_stages;
  int64_t blocks = 0;
  float best_us = 1e30f;
  for (int want = 1; want <= 32 && want <= max_stages; ++want) {
    const int len = (max_stages + want - 1) / want, sp = (max_stages + len - 1) / len;
    if (sp != want) continue;
    if (sp > 1 && (!a.ws || (int64_t)a.n_q * sp * a.Hq * (a.dh + 2) * 4 > a.ws_bytes)) break;
    int64_t busy = 0, all = 0;
    for (int b = 0; b < a.n_seqs; ++b) {
      const int64_t q_len = a.q_cu_host[b + 1] - a.q_cu_host[b];
      const int64_t keys = q_len + (a.p_cu_host ? a.p_cu_host[b + 1] - a.p_cu_host[b] : 0);
      const int64_t col_blocks = (q_len * G + cols - 1) / cols * a.Hkv;
      busy += col_blocks * (((keys + 127) / 128 + len - 1) / len);
      all += col_blocks;
    }
    float us = (float)((busy + 255) / 256) * (len * (cols == 16 ? 1.f : 3.f) + 4.f);
    if (sp > 1) us += 5.f + (float)busy * cols * a.dh * 8.f / 5.0e6f;
    if (us < best_us) {
      best_us = us;
      splits = sp;
      range = len;
      blocks = all;
    }
  }
  FewParams p;
  p.q = (const bf16_t*)a.q; p.ldq = a.ldq; p.k = (const bf16_t*)a.k_rows; p.v = (const bf16_t*)a.v_rows;
  p.out = (bf16_t*)a.out; p.out_blocks = a.out_blocks; p.q_cu = a.q_cu; p.p_cu = a.p_cu; p.n_seqs = a.n_seqs;
  p.own_row0 = (int)a.own_row0; p.Hq = a.Hq; p.Hkv = a.Hkv; p.splits = splits; p.range = range;
  p.c = (float)(1.4426950408889634 / sqrt((double)a.dh));
  p.part_o = splits > 1 ? (float*)a.ws : nullptr;
  p.part_ml = splits > 1 ? p.part_o + (int64_t)a.n_q * a.Hq * splits * a.dh : nullptr;
  *splits_out = splits;
  hipError_t e;
  blocks *= splits;
  if (a.dh == 128)
    e = cols == 16 ? launch_few<128, 1, 1, 4, 1, 2>(p, blocks, s)
                   : cols == 64 ? launch_few<128, 1, 4, 2, 2, 2>(p, blocks, s) : launch_few<128, 2, 4, 2, 2, 2>(p, blocks, s);
  else
    e = cols == 16 ? launch_few<64, 1, 1, 4, 1, 4>(p, blocks, s)
                   : cols == 64 ? launch_few<64, 1, 4, 2, 2, 3>(p, blocks, s) : launch_few<64, 2, 4, 2, 2, 3>(p, blocks, s);
  if (e != hipSuccess || splits == 1) return e;
  return launch_attn_combine(p.part_o, p.part_ml, a.out, a.out_blocks, a.n_q, a.Hq, a.dh, splits, p.c, s);
}
