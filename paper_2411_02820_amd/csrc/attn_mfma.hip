// bf16 MFMA flash attention for gfx950: causal grouped-query attention over packed sequences,
// keys taken from up to two row ranges of a cache layer (a fully visible prefix range and the
// queries' own causal range), online softmax in fp32.
//
// A workgroup of NW waves (4 are used) owns 32*NW query rows of one (sequence, q head); each wave 32 of them.
// Keys are walked in tiles of 64 cache rows (aligned to multiples of 64), staged in two-stage LDS rings
// by direct global->LDS loads (global_load_lds_dwordx4):
//   K tile  [64 keys][dh]   - rows permuted (perm_key), see below
//   Vt tile [dh][64 keys]   - from a transposed copy of V kept in the model's workspace
// Both the row permutation and the 16-byte slot swizzle are applied on the global side (which address a
// lane fetches), since the LDS destination of such a load is fixed by the lane id.
// Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_16x16x32_bf16 (K rows as the MFMA A
// operand, Q rows as B): a lane then owns TWO queries (lane%16 of the wave's two 16-query tiles) and 16 keys of each
// 64-key tile; a row sum stays in the lane until the end, and a row maximum is exchanged between the four lanes of a query only when
// one of them is far above the reference.  With the K-row permutation a lane's scores of two neighbouring 16-row tiles are 8
// consecutive keys (32*half + 8*(lane/16) + 0..7), i.e. exactly the B-operand layout of P^T for O^T += Vt P^T, and the
// matching Vt fragment is one 16-byte LDS read.  The output accumulator O^T[d][q] keeps the query in the
// lane as well, so rescaling by the running maximum is a per-lane scalar multiply.
// Bound: LDS reads (a 1 KB fragment feeds 32 cycles of MFMA, which is what LDS delivers to four SIMDs) and, in a layer, the power
// limit.  The 16x16x32 instruction sustains some 10 % more flops than the 32x32x16 one there: us a launch, before -> after, one 8B
// context of 2048 rows 58.2 -> 55.9, 4096 161 -> 153, 8192 545 -> 515 (1067 TFLOP/s causal), 16384 2100 -> 2004; a layer over 16384 rows
// 7205 -> 7124.  Fragments read three or four ahead instead of two, and a higher wave priority in phase 2: no gain.
//
// Few queries against many keys (the suffix pass) would leave most CUs idle, so the key tiles of a
// workgroup can be split over blockIdx.z; each split writes its unnormalised fp32 output with its running
// maximum and sum, and a second kernel merges the splits in a fixed order.
#include "dsk_internal.h"
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int BKV = 64;  // keys per tile

struct AttnParams {
  const bf16_t* q; int64_t ldq;
  const bf16_t* k; const bf16_t* vt; int64_t ldvt;
  bf16_t* out;
  float* part_o; float* part_ml;  // split mode: [n_q][Hq][splits][dh] and [n_q][Hq][splits][2]
  const int32_t* q_cu; const int32_t* p_cu;
  int n_seqs; int own_row0; int Hq, Hkv; int total_tiles; int splits;
  float c;         // softmax scale * log2(e)
  int k_row_max;   // last cache row that may be read
};

// key offset inside a 64-key tile that stands in LDS row rho: bits 4, 3, 2 of the row are bits 2, 4, 3 of the key
__device__ __forceinline__ int perm_key(int rho) { return (rho & 0x23) | ((rho & 0xC) << 1) | ((rho & 0x10) >> 2); }

template <int DH, bool SPLIT, int NW>
__global__ void __launch_bounds__(64 * NW, 8 / NW) attn_bf16_kernel(AttnParams p) {
  constexpr int BQ = 32 * NW;  // query rows per workgroup: 32 per wave
  constexpr int KCH = DH / 8;             // 16-byte slots per K row
  constexpr int K_RPI = 64 / KCH;         // K rows per wave load instruction
  constexpr int K_INST = BKV / K_RPI / NW; // per wave
  constexpr int V_INST = DH / 8 / NW;     // Vt rows are 64 keys = 8 slots -> 8 rows per instruction
  constexpr int NKS = DH / 32, NDT = DH / 16;  // steps of 32 along the head, output tiles of 16
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* sK = (bf16_t*)smem_raw;        // [2][BKV * DH]  K ring
  bf16_t* sV = sK + 2 * BKV * DH;        // [2][DH * BKV]  Vt ring

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 15, g = lane >> 4;
  // ---- which (head, sequence, query tile).  Workgroups are handed out in blockIdx.x order, round-robin over
  //      the 8 XCDs (each with its own L2).  Late query tiles carry the most key tiles, so they come first for
  //      every head (a heavy workgroup started late would run on alone at the end), and with a head count
  //      that is a multiple of 8 each XCD serves a fixed eighth of the heads, so the q heads of one kv group
  //      read their K and Vt through the same L2. ----
  int h, rank;
  {
    const int L = blockIdx.x;
    if ((p.Hq & 7) == 0) {
      const int hpx = p.Hq >> 3, j = L >> 3;
      h = (L & 7) * hpx + j % hpx;
      rank = j / hpx;
    } else {
      h = L % p.Hq;
      rank = L / p.Hq;
    }
  }
  const int kvh = h / (p.Hq / p.Hkv);
  // Tiles are handed out from the end of the packed batch.  A strict heaviest-first order over all sequences (tiles
  // by their index inside the sequence, from host-built tables) was measured on a batch of eight ragged prefixes:
  // no change (1.895 ms per launch either way), so the plain order stays.
  int tile = p.total_tiles - 1 - rank;
  int b = 0, seq_begin = 0, seq_end = 0;
  for (;; ++b) {
    seq_begin = p.q_cu[b];
    seq_end = p.q_cu[b + 1];
    int nt = (seq_end - seq_begin + BQ - 1) / BQ;
    if (tile < nt || b + 1 >= p.n_seqs) break;
    tile -= nt;
  }
  const int q0 = seq_begin + tile * BQ;  // first query row (packed index) of this workgroup
  if (q0 >= seq_end) return;              // cannot happen for a well-formed grid
  const int qw0 = q0 + 32 * wave;  // first query row of this wave
  const bool wave_active = qw0 < seq_end;
  const int qi[2] = {min(qw0 + lq, seq_end - 1), min(qw0 + 16 + lq, seq_end - 1)};  // this lane's queries (clamped for the padding rows)

  const int own_begin = p.own_row0 + seq_begin;
  const int wave_lim_min = p.own_row0 + min(qw0, seq_end - 1);       // smallest limit in the wave
  const int wave_lim_max = p.own_row0 + min(qw0 + 31, seq_end - 1);  // largest limit in the wave
  const int blk_lim = p.own_row0 + min(q0 + BQ, seq_end) - 1;
  const int pre_begin = p.p_cu ? p.p_cu[b] : 0, pre_end = p.p_cu ? p.p_cu[b + 1] : 0;
  const int ta0 = pre_begin / BKV, nA = pre_end > pre_begin ? (pre_end - 1) / BKV - ta0 + 1 : 0;
  const int tb0 = own_begin / BKV, nB = blk_lim / BKV - tb0 + 1;
  const int n_tiles = nA + nB;
  // key-tile range of this split
  int it_begin = 0, it_end = n_tiles;
  if (SPLIT) {
    const int per = (n_tiles + p.splits - 1) / p.splits;
    it_begin = min(n_tiles, (int)blockIdx.z * per);
    it_end = min(n_tiles, it_begin + per);
  }

  // ---- Q fragments (B operand): query = 16*qt + lane%16, d = 32*ks + 8*(lane/16) .. +7 ----
  bf16x8 qf[2][NKS];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const bf16_t* qp = p.q + (int64_t)qi[qt] * p.ldq + h * DH + 8 * g;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[qt][ks] = *(const bf16x8*)(qp + 32 * ks);
  }

  // ---- tile loads, direct to LDS.  K: LDS row rho (MFMA row) holds key offset perm_key(rho); slot s of a
  //      row holds chunk s ^ kswz(rho).  Vt: LDS row d, slot s holds key chunk s ^ vswz(d).  A 16-byte
  //      fragment read is served 16 lanes (consecutive rows, one slot index) per cycle over 64 banks, so the
  //      16 lanes must land in 16 different 16-byte bank groups: a 256-byte row covers all banks and needs 16
  //      different slots (xor with row % 16); 128-byte rows come two per bank sweep and need 8 different
  //      slots per row pair (xor with (row / 2) % 8). ----
  auto kswz = [](int row) { return DH * 2 == 256 ? (row & 15) : ((row >> 1) & 7); };
  auto vswz = [](int d) { return (d >> 1) & 7; };
  // A load instruction takes a scalar base (tile origin) plus a 32-bit per-lane byte offset that is the same
  // for every tile; only a tile that reaches past the last readable cache row needs per-lane clamping.
  const int ldkv = p.Hkv * DH;
  const bf16_t* k_base = p.k + kvh * DH;
  const bf16_t* vt_base = p.vt + (int64_t)kvh * DH * p.ldvt;
  const uint32_t sK_lds = (uint32_t)(uintptr_t)sK, sV_lds = (uint32_t)(uintptr_t)sV;
  uint32_t k_off[K_INST], v_off[V_INST];
#pragma unroll
  for (int i = 0; i < K_INST; ++i) {
    const int rho = K_RPI * (wave * K_INST + i) + lane / KCH, s = lane % KCH;
    k_off[i] = (uint32_t)(perm_key(rho) * ldkv + (s ^ kswz(rho)) * 8) * 2u + 4096u - 1024u * i;
  }
#pragma unroll
  for (int i = 0; i < V_INST; ++i) {
    const int d = 8 * (wave * V_INST + i) + (lane >> 3), s = lane & 7;
    v_off[i] = (uint32_t)(d * (int)p.ldvt + (s ^ vswz(d)) * 8) * 2u + 4096u - 1024u * i;
  }
  // LDS destination of a direct load = M0 + instruction offset + 16 * lane, and the instruction offset also
  // adds to the global address.  The load instructions of a tile write LDS pieces 1024 bytes apart, so they
  // share one M0 value and differ in the instruction offset (the lane offsets k_off / v_off compensate it on
  // the global side, biased by 4096 so that they stay non-negative).  M0 is written once per group of
  // loads: a write to M0 has to wait until earlier direct loads have consumed the old value.
  auto set_m0 = [](uint32_t dst) { asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(dst) : "memory", "m0"); };
  auto lds_load = [](uint32_t voff, const void* base, int i) {
    switch (i) {
      case 0: asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base) : "memory"); break;
      case 1: asm volatile("global_load_lds_dwordx4 %0, %1 offset:1024" : : "v"(voff), "s"(base) : "memory"); break;
      case 2: asm volatile("global_load_lds_dwordx4 %0, %1 offset:2048" : : "v"(voff), "s"(base) : "memory"); break;
      default: asm volatile("global_load_lds_dwordx4 %0, %1 offset:3072" : : "v"(voff), "s"(base) : "memory"); break;
    }
  };
  auto tile_row0 = [&](int it) { return (it < nA ? ta0 + it : tb0 + (it - nA)) * BKV; };
  // i-th load instruction of a K tile / a Vt tile; the first one of a tile sets M0
  static_assert(K_INST <= 4 && V_INST <= 4 && K_RPI * DH * 2 == 1024, "instruction offsets assume 1024-byte pieces");
  auto issue_k1 = [&](int it, int i) {
    const int r0 = tile_row0(it), stage = (it - it_begin) & 1;
    const char* base = (const char*)(k_base + (int64_t)r0 * ldkv) - 4096;
    uint32_t off = k_off[i];
    if (r0 + BKV - 1 > p.k_row_max) {
      const int rho = K_RPI * (wave * K_INST + i) + lane / KCH, s = lane % KCH;
      off = (uint32_t)(min(perm_key(rho), p.k_row_max - r0) * ldkv + (s ^ kswz(rho)) * 8) * 2u + 4096u - 1024u * i;
    }
    if (i == 0) set_m0(sK_lds + (uint32_t)(stage * BKV * DH + K_RPI * wave * K_INST * DH) * 2u);
    lds_load(off, base, i);
  };
  auto issue_v1 = [&](int it, int i) {
    const int r0 = tile_row0(it), stage = (it - it_begin) & 1;
    if (i == 0) set_m0(sV_lds + (uint32_t)(stage * DH * BKV + 8 * wave * V_INST * BKV) * 2u);
    lds_load(v_off[i], (const char*)(vt_base + r0) - 4096, i);
  };
  auto issue_k = [&](int it) {
#pragma unroll
    for (int i = 0; i < K_INST; ++i) issue_k1(it, i);
  };
  auto issue_v = [&](int it) {
#pragma unroll
    for (int i = 0; i < V_INST; ++i) issue_v1(it, i);
  };
  // A wave has nothing to do in tiles that lie wholly beyond the causal limit of all its queries; those are
  // the last tiles of the range, so the wave's active tiles are [it_begin, act_end).
  int act_end = it_begin;
  if (wave_active) act_end = max(it_begin, min(it_end, nA + wave_lim_max / BKV - tb0 + 1));

  f32x4 o[NDT][2];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) o[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // running state of the lane's two queries: m = reference maximum, mc = m * c (0 while no key was visible), l = sum over this
  // lane's keys
  float m[2] = {-INFINITY, -INFINITY}, mc[2] = {0.f, 0.f}, l[2] = {0.f, 0.f};

  constexpr int NF = 4 * NKS;    // K fragments of a tile, each the operand of two MFMAs (one per 16 queries)
  constexpr int NV = 2 * NDT;    // Vt fragments
  // fragment j of K: LDS rows 16 * (j % 4) .., head-dim step j / 4; of Vt: d-tile j % NDT, key half j / NDT: consecutive MFMAs go to
  // different accumulators
  auto k_frag = [&](const bf16_t* kt_s, int j) {
    const int row = 16 * (j % 4) + lq;
    return *(const bf16x8*)(kt_s + row * DH + (((4 * (j / 4) + g) ^ kswz(row)) * 8));
  };
  auto v_frag = [&](const bf16_t* vt_s, int j) {
    const int d = 16 * (j % NDT) + lq;
    return *(const bf16x8*)(vt_s + d * BKV + (((4 * (j / NDT) + g) ^ vswz(d)) * 8));
  };
  // masks the scores of tile `it` where a key is outside the visible range of the lane's query;
  // register r of row tile kt is key r0 + 32*(kt/2) + 8*(lane/16) + 4*(kt%2) + r
  auto mask = [&](int it, f32x4 (*s)[2]) {
    const int r0 = tile_row0(it);
    const bool segA = it < nA;
    const int lo = segA ? pre_begin : own_begin;
    const bool full = r0 >= lo && r0 + BKV - 1 <= (segA ? pre_end - 1 : wave_lim_min);
    if (!full) {
      const int kb = r0 + 8 * g;
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const int hi = segA ? pre_end - 1 : p.own_row0 + qi[qt];
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int key = kb + 32 * (kt >> 1) + 4 * (kt & 1) + r;
            s[kt][qt][r] = (key >= lo && key <= hi) ? s[kt][qt][r] : -INFINITY;
          }
      }
    }
  };
  // A query has its 64 scores of a tile in four lanes (lane%16 alike).
  // The exponentials are taken relative to a reference maximum m that follows the true running maximum
  // lazily: it moves only when the true maximum exceeds it by more than 2^8 in the exponent, so that
  // probabilities stay below 2^8 and the accumulated sums and outputs rarely need rescaling.  The
  // normalised result does not depend on the reference.  While no lane's own maximum is that far above, nothing is exchanged.
  auto new_max = [&](const float* mx) {
    const bool far = (mx[0] - m[0]) * p.c > 8.0f || (mx[1] - m[1]) * p.c > 8.0f;  // true for m = -inf and a visible key
    if (__builtin_amdgcn_ballot_w64(far) == 0) return;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float x = fmaxf(mx[qt], __shfl_xor(mx[qt], 16, 64));
      x = fmaxf(x, __shfl_xor(x, 32, 64));
      const float m_true = fmaxf(m[qt], x);
      const bool keep = (m_true - m[qt]) * p.c <= 8.0f;  // false for m = -inf (first visible key)
      const float m_new = keep ? m[qt] : m_true;
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = keep ? 1.0f : __builtin_amdgcn_exp2f((m[qt] - m_safe) * p.c);
      mc[qt] = m_safe * p.c;
      m[qt] = m_new;
      l[qt] *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) o[dt][qt] *= alpha;
    }
  };

  // One key tile.  The matrix pipe and the vector ALU of a SIMD run side by side only when their
  // instructions alternate in the instruction stream, so the two matrix phases of a tile are interleaved,
  // MFMA by MFMA, with the vector work of the neighbouring tile:
  //   phase 1:  S(it+1) = K(it+1) Q^T      with   P(it) = exp2(S(it) c - m c), row sums, bf16 packing
  //   phase 2:  O^T += Vt(it) P(it)^T       with   row maximum of S(it+1)
  // s_i holds the masked scores of tile `it` (m, mc already include it), s_n receives tile it+1.
  // Fragments are read from LDS two ahead.
  auto tile_step = [&](auto has_next_c, int it, f32x4 (*s_i)[2], f32x4 (*s_n)[2]) {
    constexpr bool HN = decltype(has_next_c)::value;
    float psum[2] = {0.f, 0.f};
    u32x4 pf[2][2];  // [key half][query tile]
    {
      const bf16_t* kt_s = sK + ((it + 1 - it_begin) & 1) * BKV * DH;
      constexpr int PPF = 16 / NF;  // pairs of scores per fragment
      bf16x8 kf[NF];
      if (HN) {
        kf[0] = k_frag(kt_s, 0);
        kf[1] = k_frag(kt_s, 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        if (HN && j + 2 < NF) kf[j + 2] = k_frag(kt_s, j + 2);
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          if (HN) {
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            s_n[j % 4][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j], qf[qt][j / 4], j < 4 ? z : s_n[j % 4][qt], 0, 0, 0);
          }
#pragma unroll
        for (int e = 0; e < PPF; ++e) {
          const int idx = j * PPF + e, kt = idx / 4, qt = idx / 2 % 2, r = idx % 2 * 2;
          const float e0 = __builtin_amdgcn_exp2f(s_i[kt][qt][r] * p.c - mc[qt]);
          const float e1 = __builtin_amdgcn_exp2f(s_i[kt][qt][r + 1] * p.c - mc[qt]);
          psum[qt] += e0;
          psum[qt] += e1;
          bf16x2 pk = {(bf16_t)e0, (bf16_t)e1};
          uint32_t pku = __builtin_bit_cast(uint32_t, pk);
          // keeps this arithmetic between the neighbouring MFMAs (its results are first used in phase 2, and
          // the optimiser would otherwise move it there)
          asm volatile("" : "+v"(pku), "+v"(psum[qt]));
          pf[kt >> 1][qt][(kt & 1) * 2 + (r >> 1)] = pku;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    l[0] += psum[0];
    l[1] += psum[1];
    if (HN) mask(it + 1, s_n);
    {
      const bf16_t* vt_s = sV + ((it - it_begin) & 1) * DH * BKV;
      constexpr int EPF = 32 / NV;  // scores per fragment
      bf16x8 vf[NV];
      vf[0] = v_frag(vt_s, 0);
      vf[1] = v_frag(vt_s, 1);
      float mx[2] = {-INFINITY, -INFINITY};
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if (j + 2 < NV) vf[j + 2] = v_frag(vt_s, j + 2);
        const int dt = j % NDT, hf = j / NDT;
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j], __builtin_bit_cast(bf16x8, pf[hf][qt]), o[dt][qt], 0, 0, 0);
        if (HN) {
#pragma unroll
          for (int e = 0; e < EPF; ++e) {
            const int idx = j * EPF + e;
            mx[idx / 16] = fmaxf(mx[idx / 16], s_n[idx % 16 / 4][idx / 16][idx % 4]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (HN) new_max(mx);
    }
  };

  // Per tile and workgroup one barrier: after it K(it+1) and Vt(it) are complete in LDS and every wave is
  // done with K(it) and Vt(it-1), whose ring stages the loads issued next overwrite.
  // The loads the barrier released go out right behind it, in one burst (about 55 cycles each): spread between
  // the MFMAs of phase 1 they cost the wave more than that (measured with per-phase timestamps).
  auto tile_sync = [&](int it) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): as a builtin the compiler accounts for it
    __syncthreads();
    if (it + 2 < it_end) issue_k(it + 2);
    if (it + 1 < it_end) issue_v(it + 1);
  };

  f32x4 s_a[4][2], s_b[4][2];
#pragma unroll
  for (int kt = 0; kt < 4; ++kt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) s_a[kt][qt] = s_b[kt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (it_begin < it_end) {
    // the first two K tiles and the first Vt tile are requested together, behind the Q fragments, and waited for
    // once: one round trip to memory at the start of a workgroup instead of two (the wait is for everything: the
    // compiler's own count for the Q fragments cannot see the direct-to-LDS loads, so a partial wait would be turned
    // into a full one in front of the first use of Q anyway)
    issue_k(it_begin);
    if (it_begin + 1 < it_end) issue_k(it_begin + 1);
    issue_v(it_begin);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): as a builtin the compiler accounts for it
    __syncthreads();
    if (it_begin < act_end) {
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const bf16x8 kf = k_frag(sK, j);
        if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // not all fragments at once: registers
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) s_a[j % 4][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[qt][j / 4], s_a[j % 4][qt], 0, 0, 0);
      }
      mask(it_begin, s_a);
      float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx[qt] = fmaxf(mx[qt], s_a[kt][qt][r]);
      new_max(mx);
    }
  }
  {
    // steady state in pairs so that the two score buffers swap roles without copies; then the wave's last
    // active tile (no successor to score); then the tiles this wave only helps to load
    int it = it_begin;
    for (; it + 2 < act_end; it += 2) {
      tile_sync(it);
      tile_step(std::true_type{}, it, s_a, s_b);
      tile_sync(it + 1);
      tile_step(std::true_type{}, it + 1, s_b, s_a);
    }
    if (it + 1 < act_end) {
      tile_sync(it);
      tile_step(std::true_type{}, it, s_a, s_b);
      tile_sync(it + 1);
      tile_step(std::false_type{}, it + 1, s_b, s_a);
      it += 2;
    } else if (it < act_end) {
      tile_sync(it);
      tile_step(std::false_type{}, it, s_a, s_b);
      it += 1;
    }
    for (; it < it_end; ++it) tile_sync(it);
  }

  // ---- store: register e of d-tile dt is out[q][16*dt + 4*(lane/16) + e] ----
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    float l_tot = l[qt] + __shfl_xor(l[qt], 16, 64);
    l_tot += __shfl_xor(l_tot, 32, 64);
    const int64_t qrow = qw0 + 16 * qt + lq;
    if (!wave_active || qrow >= seq_end) continue;
    if (SPLIT) {
      float* po = p.part_o + ((qrow * p.Hq + h) * p.splits + blockIdx.z) * DH;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) *(f32x4*)(po + 16 * dt + 4 * g) = o[dt][qt];
      if (g == 0) {
        float* pm = p.part_ml + ((qrow * p.Hq + h) * p.splits + blockIdx.z) * 2;
        pm[0] = m[qt];
        pm[1] = l_tot;
      }
    } else {
      const float inv = 1.0f / l_tot;
      bf16_t* op = p.out + qrow * p.Hq * DH + h * DH;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(o[dt][qt][e] * inv);
        *(bf16x4*)(op + 16 * dt + 4 * g) = v;
      }
    }
  }
}

__device__ __forceinline__ int64_t out_at(int q, int k, int width, int out_blocks) {
  return out_blocks ? block_at(q, k, width) : (int64_t)q * width + k;
}

// out[q][h][:] = sum_s o_s * 2^((m_s - M) c) / sum_s l_s * 2^((m_s - M) c), M = max_s m_s; one wave per (q, h).
template <int DH>
__global__ void __launch_bounds__(64) attn_combine_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                          bf16_t* __restrict__ out, int out_blocks, int Hq, int splits, float c) {
  const int64_t qh = (int64_t)blockIdx.x * Hq + blockIdx.y;
  const float* ml = part_ml + qh * splits * 2;
  float M = -INFINITY;
  for (int s = 0; s < splits; ++s) M = fmaxf(M, ml[2 * s]);
  float den = 0.f, acc[DH / 64] = {};
  for (int s = 0; s < splits; ++s) {
    const float ms = ml[2 * s];
    if (ms == -INFINITY) continue;  // this split saw no visible key
    const float w = __builtin_amdgcn_exp2f((ms - M) * c);
    den += ml[2 * s + 1] * w;
#pragma unroll
    for (int a = 0; a < DH / 64; ++a) acc[a] += part_o[(qh * splits + s) * DH + threadIdx.x + 64 * a] * w;
  }
  const float inv = 1.0f / den;
#pragma unroll
  for (int a = 0; a < DH / 64; ++a) out[out_at(blockIdx.x, blockIdx.y * DH + threadIdx.x + 64 * a, Hq * DH, out_blocks)] = (bf16_t)(acc[a] * inv);
}

// The same for at most MAXS splits, with every partial result requested before the first is used: the merge is a
// chain of small dependent steps, and what it takes is the round trips to memory, not the arithmetic.  Same sums in
// the same order as above.
template <int DH, int MAXS>
__global__ void __launch_bounds__(64) attn_combine_batched_kernel(const float* __restrict__ part_o,
                                                                  const float* __restrict__ part_ml, bf16_t* __restrict__ out,
                                                                  int out_blocks, int Hq, int splits, float c) {
  const int64_t qh = (int64_t)blockIdx.x * Hq + blockIdx.y;
  const float* ml = part_ml + qh * splits * 2;
  float ms[MAXS], ls[MAXS], po[MAXS][DH / 64];
#pragma unroll
  for (int s = 0; s < MAXS; ++s) {
    const bool on = s < splits;
    ms[s] = on ? ml[2 * s] : -INFINITY;
    ls[s] = on ? ml[2 * s + 1] : 0.f;
#pragma unroll
    for (int a = 0; a < DH / 64; ++a) po[s][a] = on ? part_o[(qh * splits + s) * DH + threadIdx.x + 64 * a] : 0.f;
  }
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < MAXS; ++s) M = fmaxf(M, ms[s]);
  float den = 0.f, acc[DH / 64] = {};
#pragma unroll
  for (int s = 0; s < MAXS; ++s) {
    if (ms[s] == -INFINITY) continue;  // not a split, or one that saw no visible key
    const float w = __builtin_amdgcn_exp2f((ms[s] - M) * c);
    den += ls[s] * w;
#pragma unroll
    for (int a = 0; a < DH / 64; ++a) acc[a] += po[s][a] * w;
  }
  const float inv = 1.0f / den;
#pragma unroll
  for (int a = 0; a < DH / 64; ++a) out[out_at(blockIdx.x, blockIdx.y * DH + threadIdx.x + 64 * a, Hq * DH, out_blocks)] = (bf16_t)(acc[a] * inv);
}

// Vt[(kvh*dh + d)*ldvt + row] = V[row][kvh*dh + d] for the valid rows, 0 for the others, over whole
// 64-row tiles.  valid(row) = row < n_pre || own_row0 <= row < own_row0 + n_own.
__global__ void __launch_bounds__(256) transpose_v_kernel(const bf16_t* __restrict__ v_rows, bf16_t* __restrict__ vt,
                                                          int64_t ldvt, int width, int64_t n_pre, int64_t own_row0,
                                                          int64_t n_own, int64_t tile0) {
  __shared__ bf16_t tile[64][66];
  const int64_t r0 = ((int64_t)blockIdx.x + tile0) * 64;
  const int c0 = blockIdx.y * 64;
  const int tid = threadIdx.x;
  {
    const int r = tid >> 3, ch = tid & 7;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int rr = r + 32 * half;
      const int64_t row = r0 + rr;
      const bool valid = row < n_pre || (row >= own_row0 && row < own_row0 + n_own);
      bf16x8 x;
      if (valid) x = *(const bf16x8*)(v_rows + row * width + c0 + ch * 8);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (bf16_t)0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) tile[rr][ch * 8 + e] = x[e];
    }
  }
  __syncthreads();
  {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int id = tid + 256 * half, d = id >> 3, rc = id & 7;
      bf16x8 x;
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = tile[rc * 8 + e][d];
      *(bf16x8*)(vt + (int64_t)(c0 + d) * ldvt + r0 + rc * 8) = x;
    }
  }
}

}  // namespace

// how many calls split the keys over workgroups, how many of those had at most 64 queries per sequence, and how many calls
// the kernel for few queries (attn_few.hip) took
static int64_t g_split_launches = 0, g_split_64_launches = 0, g_few_launches = 0;
void attn_mfma_counts(int64_t* split, int64_t* split_64, int64_t* few, int reset) {
  if (split) *split = g_split_launches;
  if (split_64) *split_64 = g_split_64_launches;
  if (few) *few = g_few_launches;
  if (reset) g_split_launches = g_split_64_launches = g_few_launches = 0;
}

// fp32 scratch for the split mode: n_q * splits <= kMaxSplitRows partial rows of (dh + 2) floats per q head
constexpr int64_t kMaxSplitRows = 4096;
int64_t attn_mfma_workspace_bytes(int Hq, int dh) { return kMaxSplitRows * Hq * (dh + 2) * 4; }

hipError_t launch_transpose_v(const void* v_rows, void* vt, int64_t ldvt, int width, int64_t n_pre, int64_t own_row0,
                              int64_t n_own, int64_t first_row, hipStream_t s) {
  const int64_t end = own_row0 + n_own, tile0 = first_row / 64;
  if (end <= tile0 * 64) return hipSuccess;
  dim3 grid((unsigned)((end + 63) / 64 - tile0), width / 64);
  hipLaunchKernelGGL(transpose_v_kernel, grid, dim3(256), 0, s, (const bf16_t*)v_rows, (bf16_t*)vt, ldvt, width, n_pre,
                     own_row0, n_own, tile0);
  return hipGetLastError();
}

template <int DH, bool SPLIT, int NW>
hipError_t launch_attn(const AttnParams& p, dim3 grid, hipStream_t s) {
  auto kern = attn_bf16_kernel<DH, SPLIT, NW>;
  constexpr int lds = (2 * BKV * DH + 2 * DH * BKV) * 2;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  DSK_LAUNCH_TIMED(kern, grid, dim3(64 * NW), lds, s, p);
  return hipGetLastError();
}

hipError_t launch_attn_combine(const float* part_o, const float* part_ml, void* out, int out_blocks, int n_q, int Hq, int dh,
                               int splits, float c, hipStream_t s) {
  const dim3 grid(n_q, Hq);
  bf16_t* o = (bf16_t*)out;
  if (dh == 128 && splits <= 16)
    hipLaunchKernelGGL((attn_combine_batched_kernel<128, 16>), grid, dim3(64), 0, s, part_o, part_ml, o, out_blocks, Hq, splits, c);
  else if (dh == 128 && splits <= 32)
    hipLaunchKernelGGL((attn_combine_batched_kernel<128, 32>), grid, dim3(64), 0, s, part_o, part_ml, o, out_blocks, Hq, splits, c);
  else if (dh == 128)
    hipLaunchKernelGGL(attn_combine_kernel<128>, grid, dim3(64), 0, s, part_o, part_ml, o, out_blocks, Hq, splits, c);
  else if (splits <= 32)
    hipLaunchKernelGGL((attn_combine_batched_kernel<64, 32>), grid, dim3(64), 0, s, part_o, part_ml, o, out_blocks, Hq, splits, c);
  else
    hipLaunchKernelGGL(attn_combine_kernel<64>, grid, dim3(64), 0, s, part_o, part_ml, o, out_blocks, Hq, splits, c);
  return hipGetLastError();
}

hipError_t launch_attn_mfma_bf16(const AttnArgs& a, hipStream_t s) {
  if (a.n_q <= 0) return hipSuccess;
  if (attn_few_supported(a)) {
    int splits = 1;
    hipError_t e = launch_attn_few(a, &splits, s);
    if (e == hipSuccess) ++g_few_launches;
    if (e == hipSuccess && splits > 1) {
      ++g_split_launches;
      bool up_to_64 = true;
      for (int b = 0; b < a.n_seqs; ++b) up_to_64 &= a.q_cu_host[b + 1] - a.q_cu_host[b] <= 64;
      if (up_to_64) ++g_split_64_launches;
    }
    return e;
  }
  // (few rows, whose result goes out in blocks, are all with the kernel above)
  if (a.out_blocks || (a.dh != 128 && a.dh != 64) || !a.vt || (a.ldq & 7) || a.own_row0 + a.n_q >= ((int64_t)1 << 31))
    return hipErrorNotSupported;
  // per-lane tile offsets are 32-bit byte offsets
  if ((int64_t)a.dh * a.ldvt * 2 >= ((int64_t)1 << 32) || (int64_t)BKV * a.Hkv * a.dh * 2 >= ((int64_t)1 << 32))
    return hipErrorNotSupported;
  AttnParams p;
  p.q = (const bf16_t*)a.q; p.ldq = a.ldq; p.k = (const bf16_t*)a.k_rows; p.vt = (const bf16_t*)a.vt; p.ldvt = a.ldvt;
  p.out = (bf16_t*)a.out; p.q_cu = a.q_cu; p.p_cu = a.p_cu; p.n_seqs = a.n_seqs; p.own_row0 = (int)a.own_row0;
  p.Hq = a.Hq; p.Hkv = a.Hkv;
  // 4-wave workgroups (128 queries).  8-wave workgroups halve the tile loads a wave issues per key tile and are
  // faster when the kernel is timed alone (+14 % at 8k tokens) but slower inside the layer, behind the projections
  // (25.05 -> 25.26 ms for eight 8B layers at 8k tokens, 58.3 -> 59.5 ms at 16k), so only this shape is built.
  auto count_tiles = [&](int bq) {
    int64_t t = 0;
    for (int b = 0; b < a.n_seqs; ++b) t += (a.q_cu_host[b + 1] - a.q_cu_host[b] + bq - 1) / bq;
    return t;
  };
  constexpr int nw = 4;
  int64_t max_keys = 0;
  for (int b = 0; b < a.n_seqs; ++b) {
    const int len = a.q_cu_host[b + 1] - a.q_cu_host[b];
    int64_t keys = len + (a.p_cu_host ? a.p_cu_host[b + 1] - a.p_cu_host[b] : 0);
    if (keys > max_keys) max_keys = keys;
  }
  p.c = (float)(1.4426950408889634 / sqrt((double)a.dh));
  p.k_row_max = (int)(a.own_row0 + a.n_q - 1);
  const int key_tiles = (int)((max_keys + BKV - 1) / BKV) + 1;
  const int total = (int)count_tiles(32 * nw);
  const int64_t blocks = (int64_t)total * a.Hq;
  // split the key tiles when the grid alone cannot fill the chip
  int splits = 1;
  if (a.ws && blocks < 512 && key_tiles >= 8) {
    // about two workgroups per CU; measured on 64 queries against 8k and 16k keys: 16 splits beat 8 and 32
    // (more splits pay more for partial outputs and the per-workgroup start-up than they gain in parallelism)
    splits = (int)((512 + blocks - 1) / blocks);
    if (splits > key_tiles / 4) splits = key_tiles / 4;
    while (splits > 1 && ((int64_t)a.n_q * splits > kMaxSplitRows ||
                          (int64_t)a.n_q * splits * a.Hq * (a.dh + 2) * 4 > a.ws_bytes))
      --splits;
  }
  p.total_tiles = total;
  p.splits = splits;
  p.part_o = nullptr;
  p.part_ml = nullptr;
  if (splits > 1) {
    p.part_o = (float*)a.ws;
    p.part_ml = p.part_o + (int64_t)a.n_q * a.Hq * splits * a.dh;
    dim3 grid((unsigned)blocks, 1, splits);
    ++g_split_launches;
    hipError_t e = a.dh == 128 ? launch_attn<128, true, 4>(p, grid, s) : launch_attn<64, true, 4>(p, grid, s);
    if (e != hipSuccess) return e;
    return launch_attn_combine(p.part_o, p.part_ml, p.out, 0, a.n_q, a.Hq, a.dh, splits, p.c, s);
  }
  dim3 grid((unsigned)total * a.Hq);
  return a.dh == 128 ? launch_attn<128, false, 4>(p, grid, s) : launch_attn<64, false, 4>(p, grid, s);
}
