// bf16 MFMA GEMM for gfx950:  C[M,N] = A[M,K] * W[N,K]^T  (+ R), fp32 accumulation, bf16 output.
//
// Both operands are K-contiguous, so both feed the MFMA with 16-byte vectors and no transposition.  Two kernels:
// gemm16_bf16_kernel on v_mfma_f32_16x16x32_bf16 for more than 64 rows (tiles of 128, 192 or 256 rows x 256 columns, the
// contraction split over workgroups where the tiles do not fill the chip: gemm_plan), gemm_bf16_kernel on
// v_mfma_f32_32x32x16_bf16 for 64 rows and fewer of row-major weights (K-split tiles) and for gate/up over up to 256 rows.
// (Few rows of a model's own weights: few_rows.hip.)  A workgroup owns a BM x BN tile of C and walks K in steps of 64
// through a two-stage
// LDS ring (W up to four: w_stages) filled by direct global->LDS loads (global_load_lds_dwordx4: no staging registers, no
// ds_write).  The loads of k-tile kt+2 go out, between MFMAs, as soon as a barrier shows that every wave
// has read k-tile kt out of the stage they overwrite; fragments are read from LDS one or two k-steps ahead
// of the MFMAs that use them.  Two schedules of the 32x32x16 kernel (SCHED): 0 frees the stage before the last k-step
// (one barrier per k-tile; any tile shape), 1 frees it before k-step 2 of 4 and spreads the loads over two
// k-steps (two barriers; the 128 x 128 tile, where it is up to 25 % faster).
//
// LDS rows hold 64 bf16 = eight 16-byte slots.  A wave load instruction fills 64 consecutive slots
// (8 rows); the swizzle is applied on the global side: the lane that fills slot p of row r fetches chunk
// p ^ ((r >> 1) & 7).  With that, the 16 lanes that one LDS cycle serves (rows r..r+15 at one k chunk)
// touch 16 different 16-byte bank groups of the 256-byte LDS line.
//
// W rows play the MFMA "A" role and activation rows the "B" role: a lane then holds four consecutive
// output columns of one row in four consecutive accumulator registers (the epilogue regroups them through LDS so
// that stores cover whole rows of the tile).
// Workgroup ids are remapped so that each XCD (own L2) works on a compact patch of the tile grid.
//
// 64 rows and fewer are a weight-streaming problem: a 64 x 64 tile, K split over blockIdx.y so that enough workgroups
// stream W to fill HBM; each split writes an fp32 partial tile and a second kernel adds the partials in a fixed
// order (deterministic), applies the residual and rounds.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "dsk_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int BK = 64;        // k extent of one LDS stage
constexpr int CH = BK / 8;    // 16-byte slots per LDS row
constexpr int RPI = 64 / CH;  // rows filled by one wave load instruction
constexpr int NSTAGE = 2;
constexpr int N_XCD = 8;
constexpr int GROUP_M = 4;    // M-tiles per scheduling group

__device__ __forceinline__ int slot(int row, int chunk) { return (row * CH + (chunk ^ ((row >> 1) & (CH - 1)))) * 8; }

// W in blocks (WB; block_at in dsk_internal.h): a k-tile of 64 columns is two 1 KB blocks per 16 rows.  Each goes to LDS as
// it is, in one wave load of 1 KB in a row, and a fragment is read back in lane order: no swizzle, no conflicts.  The
// other way round, fetching blocks piecewise into the row layout, lets a load touch 64 bytes of a line at a time and
// costs the large GEMMs 10 % (8192 x 28672 x 4096).
constexpr int BLK = 512;  // elements of a block
template <bool WB> __device__ __forceinline__ int w_step() { return WB ? 32 : 2; }  // bytes of W per k of a tile's origin

// C[m][n..n+3] = v (+ R[m][n..n+3]); R and C are bf16 or fp32 as the epilogue flags say.
__device__ __forceinline__ void store_quad(void* C, int64_t ldc, const void* R, int64_t ldr, int m, int n, f32x4 v, int epi) {
  if (epi & EPI_RESIDUAL) {
    if (epi & EPI_R_F32) {
      f32x4 r = *(const f32x4*)((const float*)R + (int64_t)m * ldr + n);
      v += r;
    } else {
      bf16x4 r = *(const bf16x4*)((const bf16_t*)R + (int64_t)m * ldr + n);
      v[0] += (float)r[0]; v[1] += (float)r[1]; v[2] += (float)r[2]; v[3] += (float)r[3];
    }
  }
  if (epi & EPI_C_F32) {
    *(f32x4*)((float*)C + (int64_t)m * ldc + n) = v;
  } else {
    bf16x4 o;
    o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
    *(bf16x4*)((bf16_t*)C + (int64_t)m * ldc + n) = o;
  }
}

// PARTIAL: write the fp32 accumulators of this K split to P[split][M][N] instead of the bf16 result.
// EPI_SWIGLU (run-time flag; wave tiles of two 32-column MFMA tiles): W holds gate and up
// rows interleaved in blocks of 32 (packed rows 64b..64b+31 = gate rows 32b.., the next 32 = the same up
// rows), so the two MFMA tiles of a wave are gate and up of the same 32 FFN indices at the same
// lane/register; the epilogue writes silu(gate)*up to C[M, N/2].
// SCHED: software-pipeline schedule of the k loop, see the top of the file.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool PARTIAL, int SCHED, bool WB>
__global__ void __launch_bounds__(WAVES_M* WAVES_N * 64)
    gemm_bf16_kernel(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W, int64_t ldw,
                     void* __restrict__ C, int64_t ldc, const void* __restrict__ R, int64_t ldr,
                     float* __restrict__ P, int M, int N, int K, int epi, int tiles_m, int tiles_n, int kt_per_split) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;  // wave tile
  constexpr int TM = WTM / 32, TN = WTN / 32;            // 32x32 MFMA tiles per wave
  constexpr int A_INST = BM / RPI / NW, W_INST = BN / RPI / NW;
  constexpr int NKS = BK / 16;
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile/wave mismatch");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* sA = (bf16_t*)smem_raw;      // [NSTAGE][BM][BK]
  bf16_t* sW = sA + NSTAGE * BM * BK;  // [NSTAGE][BN][BK]

  // ---- workgroup -> tile, XCD-aware: consecutive ids go to different XCDs, so give each XCD a
  //      contiguous range of the (grouped) tile order ----
  const int nb = gridDim.x;
  int pid = blockIdx.x;
  {
    const int q = nb / N_XCD, rem = nb % N_XCD;
    const int xcd = pid % N_XCD, loc = pid / N_XCD;
    pid = (xcd < rem) ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
  }
  const int per_group = GROUP_M * tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GROUP_M;
  const int gsz = min(GROUP_M, tiles_m - first_m);
  const int in_group = pid - group * per_group;
  const int tm = first_m + in_group % gsz;
  const int tn = in_group / gsz;
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  // ---- per-lane global source of each wave load instruction: a 32-bit byte offset from the (uniform) matrix
  //      base, so that the loads use the scalar-base + vector-offset address form and the walk along K only
  //      moves the scalar base ----
  const int lr = lane / CH, lp = lane % CH;
  uint32_t a_off[A_INST], w_off[W_INST];
#pragma unroll
  for (int i = 0; i < A_INST; ++i) {
    int row = RPI * (wave * A_INST + i) + lr;
    a_off[i] = (uint32_t)(((int64_t)min(m0 + row, M - 1) * lda + (lp ^ ((row >> 1) & (CH - 1))) * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < W_INST; ++i) {
    const int row = RPI * (wave * W_INST + i) + lr, blk = wave * W_INST + i;  // WB: block blk % 2 of rows 16 * (blk / 2) ..
    w_off[i] = WB ? (uint32_t)(min(n0 / 16 + blk / 2, N / 16 - 1) * (int)(ldw / 32) + blk % 2) * (BLK * 2u) + lane * 16u
                  : (uint32_t)(((int64_t)min(n0 + row, N - 1) * ldw + (lp ^ ((row >> 1) & (CH - 1))) * 8) * 2);
  }
  typedef __attribute__((address_space(3))) void lds_void;
  typedef const __attribute__((address_space(1))) void glb_void;
  constexpr int PER_TILE = A_INST + W_INST;  // load instructions per wave per k-tile
  // global_load_lds_dwordx4 in its scalar-base + 32-bit vector-offset form; M0 carries the LDS byte address
  // of the 1 KB the wave fills (lane i lands at M0 + 16*i)
  const uint32_t sA_lds = (uint32_t)(uintptr_t)sA, sW_lds = (uint32_t)(uintptr_t)sW;
  auto issue_load = [&](int stage, int k0, int idx) {
    const bool is_a = idx < A_INST;
    const int li = is_a ? idx : idx - A_INST;
    const char* base = is_a ? (const char*)A + (int64_t)k0 * 2 : (const char*)W + (int64_t)k0 * w_step<WB>();
    const uint32_t voff = is_a ? a_off[li] : w_off[li];
    const uint32_t dst = is_a ? sA_lds + (uint32_t)(stage * BM * BK + RPI * (wave * A_INST + li) * BK) * 2
                              : sW_lds + (uint32_t)(stage * BN * BK + RPI * (wave * W_INST + li) * BK) * 2;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(dst), "v"(voff), "s"(base)
                 : "memory", "m0");
  };
  auto issue_loads = [&](int stage, int k0) {
#pragma unroll
    for (int i = 0; i < PER_TILE; ++i) issue_load(stage, k0, i);
  };

  f32x16 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  const int frag_row = lane & 31, frag_hi = lane >> 5;
  auto load_frags = [&](const bf16_t* a_s, const bf16_t* w_s, int ks, bf16x8* xf, bf16x8* wf) {
    const int ch = ks * 2 + frag_hi;
#pragma unroll
    for (int i = 0; i < TM; ++i) xf[i] = *(const bf16x8*)(a_s + slot(wm * WTM + i * 32 + frag_row, ch));
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int r = wn * WTN + j * 32 + frag_row;
      wf[j] = *(const bf16x8*)(w_s + (WB ? ((r >> 4) * 2 + (ch >> 2)) * BLK + ((ch & 3) * 16 + (r & 15)) * 8 : slot(r, ch)));
    }
  };

  // ---- K range of this workgroup ----
  const int KT_all = K / BK;
  const int kt_begin = PARTIAL ? (int)blockIdx.y * kt_per_split : 0;
  const int kt_end = PARTIAL ? min(KT_all, kt_begin + kt_per_split) : KT_all;

  // Software pipeline over k-tiles with ONE barrier per tile, placed between the MFMAs of k-step NKS-2 and
  // NKS-1: by then every LDS read of the current tile has been issued and waited for, so the barrier both
  // publishes tile kt+1 (each wave has waited for its own loads) and frees the current stage for the loads of
  // tile kt+2.  After the barrier a wave still owns the MFMAs of the last k-step (fragments already in
  // registers) and issues the first fragment reads of tile kt+1 under them, so the restart after a barrier
  // never waits on LDS.
  const int n_kt = kt_end - kt_begin;
  issue_loads(0, kt_begin * BK);
  if (n_kt > 1) {
    issue_loads(1, (kt_begin + 1) * BK);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_TILE) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  if constexpr (SCHED == 1) {
    // Early-freed stage, for k-tiles of four k-steps.  Fragments are read two k-steps ahead (sets 1 and 2 during
    // k-step 0, set 3 during k-step 1), so every LDS read of the tile has returned before k-step 2: the barrier
    // there frees the stage, and the loads of tile t+2 go out one per two MFMAs over k-steps 2 and 3 instead of
    // all in the last one.  A second barrier before k-step 3 publishes tile t+1: its loads were issued a whole
    // tile earlier, and only the LD loads issued since the first barrier may still be in flight.
    static_assert(NKS == 4 && PER_TILE % 2 == 0, "schedule written for four k-steps");
    constexpr int NM = TN * TM;
    constexpr int LD = PER_TILE / 2;  // loads per wave in each of the last two k-steps
    bf16x8 xs[NKS][TM], ws[NKS][TN];
    load_frags(sA, sW, 0, xs[0], ws[0]);
    auto tile_step = [&](int t, auto has_next, auto has_next2) {
      const int stage = t & 1;
      const bf16_t* a_s = sA + stage * BM * BK;
      const bf16_t* w_s = sW + stage * BN * BK;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks == 2) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
        if (ks == 3) {
          if (has_next2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LD) : "memory");
          else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int m = j * TM + i;
            if (m == (NM >= 8 ? 2 : 1)) {
              __builtin_amdgcn_sched_barrier(0);
              if (ks == 0) { load_frags(a_s, w_s, 1, xs[1], ws[1]); load_frags(a_s, w_s, 2, xs[2], ws[2]); }
              if (ks == 1) load_frags(a_s, w_s, 3, xs[3], ws[3]);
              if (ks == 3 && has_next) load_frags(sA + (stage ^ 1) * BM * BK, sW + (stage ^ 1) * BN * BK, 0, xs[0], ws[0]);
              __builtin_amdgcn_sched_barrier(0);
            }
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ws[ks][j], xs[ks][i], acc[j][i], 0, 0, 0);
            if (ks >= 2 && has_next2) {
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int q = m * LD / NM; q < (m + 1) * LD / NM; ++q)
                issue_load(stage, (kt_begin + t + 2) * BK, (ks - 2) * LD + q);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int t = 0;
    for (; t + 2 < n_kt; ++t) tile_step(t, std::true_type{}, std::true_type{});
    if (t + 1 < n_kt) { tile_step(t, std::true_type{}, std::false_type{}); ++t; }
    if (t < n_kt) tile_step(t, std::false_type{}, std::false_type{});
  } else {
    bf16x8 xf[2][TM], wf[2][TN];
    load_frags(sA, sW, 0, xf[0], wf[0]);
    // one k-tile; the two flags are compile-time so that the steady-state loop body is a single basic block
    // (precise s_waitcnt counts) and the tail tiles are peeled
    auto tile_step = [&](int t, auto has_next, auto has_next2) {
      const int stage = t & 1;
      const bf16_t* a_s = sA + stage * BM * BK;
      const bf16_t* w_s = sW + stage * BN * BK;
  #pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int cur = ks & 1;
        constexpr int NM = TN * TM;
        constexpr int LEAD = NM >= 8 ? 2 : 1;  // MFMAs issued before the next fragment reads
        if (ks + 1 == NKS) {
          // all reads of this tile are done; tile t+1 has landed (only its loads are outstanding)
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          __syncthreads();
          if (has_next)
            load_frags(sA + (stage ^ 1) * BM * BK, sW + (stage ^ 1) * BN * BK, 0, xf[cur ^ 1], wf[cur ^ 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
  #pragma unroll
        for (int j = 0; j < TN; ++j)
  #pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int m = j * TM + i;
            if (ks + 1 < NKS && m == LEAD) {
              // Fragment reads of the next k-step go out after the first MFMAs of this one: the s_waitcnt the
              // compiler puts in front of this k-step then only covers reads issued a whole k-step earlier, and
              // the new reads have the remaining MFMAs to land.
              __builtin_amdgcn_sched_barrier(0);
              load_frags(a_s, w_s, ks + 1, xf[cur ^ 1], wf[cur ^ 1]);
              __builtin_amdgcn_sched_barrier(0);
            }
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[cur][j], xf[cur][i], acc[j][i], 0, 0, 0);
            if (ks + 1 == NKS && has_next2) {
              // the loads of tile t+2 (its stage was freed by the barrier) go out one by one between the MFMAs of
              // the last k-step: a wave that queues several vector-memory instructions back to back cannot issue
              // its MFMAs until the address unit has taken them
              __builtin_amdgcn_sched_barrier(0);
  #pragma unroll
              for (int q = m * PER_TILE / NM; q < (m + 1) * PER_TILE / NM; ++q)
                issue_load(stage, (kt_begin + t + 2) * BK, q);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int t = 0;
    for (; t + 2 < n_kt; ++t) tile_step(t, std::true_type{}, std::true_type{});
    if (t + 1 < n_kt) { tile_step(t, std::true_type{}, std::false_type{}); ++t; }
    if (t < n_kt) tile_step(t, std::false_type{}, std::false_type{});

  }

  // ---- epilogue: accumulator register 4q+e of tile (j,i) is C[m][n + e],
  //      m = tile row base + lane%32, n = tile col base + 8q + 4*(lane/32) ----
  // Wave tiles of 64 columns go through LDS (free by now: every wave has read its last fragments before the last
  // barrier, and no load is in flight): stored straight from the accumulators, a store instruction would touch
  // 32 rows with 8 or 16 bytes each; staged, a wave writes 32 x 64 fp32 values to a padded region of its own and
  // reads them back row by row, so that 16 lanes cover one output row (128 contiguous bytes of bf16, 256 of fp32)
  // and the residual is read the same way.  Only the wave itself touches its region: no barrier.
  if constexpr (!PARTIAL && TN == 2) {
    constexpr int ROW_F = 64 + 4;  // floats per staged row: 16-byte pad, conflict-free for 16 lanes at a time
    float* stage = (float*)smem_raw + wave * (32 * ROW_F);
    static_assert(NW * 32 * ROW_F * 4 <= NSTAGE * (BM + BN) * BK * 2, "staging region fits the tile ring");
    const bool swiglu = (epi & EPI_SWIGLU) != 0;
    // the lane's indices are derived here from an opaque copy of the lane id: computed before the k loop (where the
    // compiler would otherwise hoist them) they would take the kernel from 248 to 252 registers, i.e. to all 512
    // of a SIMD for its two waves, and no other kernel's wave (a copy, a pacing kernel) could share the CU
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int frag_row = lane_e & 31, frag_hi = lane_e >> 5;
    const int rr = lane_e >> 4, c4 = (lane_e & 15) * 4;  // read-back: 4 rows per instruction, 4 columns per lane
    const int rr_s = lane_e >> 3, c4_s = (lane_e & 7) * 4;  // SwiGLU: 32 result columns per row, 8 rows per instruction
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (swiglu) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = acc[0][i][4 * q + e], u = acc[1][i][4 * q + e];
            const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
            o[e] = g * sig * u;
          }
          *(f32x4*)(stage + frag_row * ROW_F + 8 * q + 4 * frag_hi) = o;
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4 o = {acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
            *(f32x4*)(stage + frag_row * ROW_F + j * 32 + 8 * q + 4 * frag_hi) = o;
          }
      }
      __builtin_amdgcn_wave_barrier();
      const int mb = m0 + wm * WTM + i * 32;
      if (swiglu) {
        const int fb = (n0 + wn * WTN) / 2;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int r = it * 8 + rr_s, m = mb + r, f = fb + c4_s;
          const f32x4 v = *(const f32x4*)(stage + r * ROW_F + c4_s);
          if (m < M && f < N / 2) {
            bf16x4 o;
            o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
            *(bf16x4*)((bf16_t*)C + (int64_t)m * ldc + f) = o;
          }
        }
      } else {
        const int n = n0 + wn * WTN + c4;
        // the eight residual quads of this 32-row block are requested together, then added and stored: one
        // memory round trip per block instead of one per store
        f32x4 res[8];
        if (epi & EPI_RESIDUAL) {
#pragma unroll
          for (int it = 0; it < 8; ++it) {
            const int m = min(mb + it * 4 + rr, M - 1), nn = min(n, N - 4);  // clamped: masked below
            if (epi & EPI_R_F32) {
              res[it] = *(const f32x4*)((const float*)R + (int64_t)m * ldr + nn);
            } else {
              const bf16x4 rb = *(const bf16x4*)((const bf16_t*)R + (int64_t)m * ldr + nn);
              res[it][0] = (float)rb[0]; res[it][1] = (float)rb[1]; res[it][2] = (float)rb[2]; res[it][3] = (float)rb[3];
            }
          }
        }
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int r = it * 4 + rr, m = mb + r;
          f32x4 v = *(const f32x4*)(stage + r * ROW_F + c4);
          if (epi & EPI_RESIDUAL) v += res[it];
          if (m < M && n < N) store_quad(C, ldc, nullptr, 0, m, n, v, epi & ~(EPI_RESIDUAL | EPI_R_F32));  // N % 4 == 0
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm * WTM + i * 32 + frag_row;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + wn * WTN + j * 32 + 8 * q + 4 * frag_hi;
        if (n >= N) continue;  // N is a multiple of 4
        float v0 = acc[j][i][4 * q], v1 = acc[j][i][4 * q + 1], v2 = acc[j][i][4 * q + 2], v3 = acc[j][i][4 * q + 3];
        if (PARTIAL) {
          f32x4 o = {v0, v1, v2, v3};
          *(f32x4*)(P + ((int64_t)blockIdx.y * M + m) * N + n) = o;
        } else {
          f32x4 v = {v0, v1, v2, v3};
          store_quad(C, ldc, R, ldr, m, n, v, epi);
        }
      }
    }
  }
}

// The same GEMM on v_mfma_f32_16x16x32_bf16 (wave tiles of 64 columns, no K split).  Under a bf16 GEMM on random
// data the chip sits at its power limit, and a register-only loop of this instruction sustains about 10 % more
// flops there than the 32x32x16 one (the 16x16 accumulator tile is read and written half as often per flop).
// W rows are the MFMA "A" operand again: lane l holds row l%16 and the eight k values 8*(l/16)..+7 of a 32-wide
// k-step; accumulator register r of tile (j,i) is C[m][n + r], m = 16i + l%16, n = 16j + 4*(l/16).
// Schedule per k-tile (two k-steps of 32 MFMAs): the fragments of k-step 1 are read during k-step 0; a barrier
// between the k-steps frees the stage; the loads of A of tile t+2 and of W of the tile that takes this one's stage (w_stages) are
// spread over the MFMAs of k-step 1; a barrier in
// the middle of k-step 1 publishes tile t+1, whose first fragments are read during the rest of it.
// GROUPED (the expert projections of a mixture-of-experts layer): the token rows are sorted by expert, and row tile
// tm of the grid is described by tile_tab[tm] = {expert, first row, end of the expert's rows, scheduling group} (built on the
// device; tile_tab[tiles_m] = numbers of tiles that exist, and of low ones behind them; expert < 0: no such tile, the workgroup leaves); the
// expert's matrix is W + expert * w_group_stride.  a_row (optional): sorted row r is row a_row[r] of A's a_rows rows, so
// that the rows are read where they are (gathered into a buffer first they cost 38 us more at 8192 tokens).
// LOW (down): the table may end in low tiles, 128 x 128, for experts' last rows (moe_low_tiles has the rule and its figures).
// ROPE (the QKV projection, heads of 128, weights in blocks): a wave's 64 columns are 32 rotary pairs of one head (elements
// p0 .. p0 + 31 and their partners 64 further on: tiles j and j + 2, the same lane and register), so that the epilogue
// rotates the fp32 sums and writes q to C and k and v straight to their cache rows.  The separate pass read and wrote
// every row once more (33 us for 8192 rows of the 8B shape); a layer over 4096 rows 1432 -> 1421 us, over eight ragged
// contexts (49523 rows) 18.60 -> 18.42 ms, a Mixtral layer over 8192 rows 5958 -> 5925 us, a 70B one 10489 -> 10461 us.
struct RopeOut {
  const float2* cs;  // [M][64] (cos, sin)
  bf16_t *k, *v;     // [M][Hkv * 128]
  int Hq, Hkv;
};
// DIRECT (unsplit 256-row tiles, weights in blocks, w_direct): a wave loads its fragments of W straight to registers, and only A
// goes through LDS, in a ring of four stages.  W is requested 1.5 k-tiles ahead; the compiler's waits, which count these loads
// but not those of A between them, leave some 0.8 of a k-tile of that (vmcnt 6 to 11 where 13 to 19 newer loads are in flight).
// What bounds the large projections is power, and with all operands zero the other form is the faster
// one (8192 x 28672 x 4096 1912 against 1800 TFLOP/s).  On data this form is, because it moves less: 128 KB of LDS reads and
// 32 KB of writes per k-tile instead of 192 and 64 (a fragment of W comes twice from L1, not twice through LDS; requests to
// L2 the same within 4 %), and because an MFMA shares an operand with the one before it.  8192 rows, both forms in turn:
// down 662 -> 638 us, QKV 297 -> 292, O 246.5 -> 245, gate/up 1262 -> 1250; 70B QKV, down and gate/up 1005 -> 988, 2635 -> 2624 and
// 5160 -> 4996; same sums, same order.
// Measured without gain: 2, 3 or 6 fragments of A ahead, and the lines of W touched 4 to 8 k-tiles early (faster on zeros).
//
// Stages of W in LDS (not DIRECT; A has two).  Lower tiles have less to compute on a k-tile of W, which is the same 32 KB for every
// height, so with two stages they wait for it: W runs further ahead, as far as LDS goes (128 rows 160 KB, 192 rows 144 KB).  us a
// launch, two stages -> these: 128 rows QKV over 1024 rows 64.4 -> 60.3, O over 1500 rows 73.0 -> 68.3; 192 rows gate/up over 333 rows 81.5
// -> 77.8 (70B 307.7 -> 296.0), QKV over 1500 rows 73.9 -> 72.7.  256 rows with three stages: 0.5 to 1 % slower (gate/up over 4096 rows
// 628.8 -> 632.9), so they keep two.  Up to 128 rows of a dense projection keep two as well: one row tile streams W once, from HBM,
// and what fills a longer ring in front of the loop holds up the first k-tile.  us, four stages -> two: 96 rows QKV 19.9 -> 19.0, O 17.0 ->
// 16.3, down 32.3 -> 31.9, 70B O 37.4 -> 34.4, a 2048-wide shape's down 16.0 -> 14.8; over 128 rows O 17.7 -> 17.0, 70B O 39.2 -> 36.0,
// QKV 20.8 and 70B QKV 41.9 -> 42.4.  From 129 rows on four: over 160 rows QKV 22.6 -> 22.2, O 17.6 -> 18.2, a layer the same; 230 rows
// 208.5 -> 205.6.
template <int BM> constexpr int w_stages() { return BM == 128 ? 4 : BM == 192 ? 3 : 2; }
template <int BM, int BN, bool DIRECT, int WS = w_stages<BM>()> constexpr int lds16() { return (DIRECT ? 4 * BM : NSTAGE * BM + WS * BN) * BK * 2; }
// One tile: rows m0 .. of A up to row M, columns n0 .. of the product with W.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool WB, bool GROUPED, bool ROPE, bool DIRECT, int WS = w_stages<BM>()>
__device__ __forceinline__ void gemm16_tile(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W, int64_t ldw, void* C,
                                            int64_t ldc, const void* __restrict__ R, int64_t ldr, int m0, int n0, int M, int M_all, int N,
                                            int K, int epi, int kt_per_split, const int32_t* __restrict__ a_row, int a_rows,
                                            const RopeOut& ro) {
  static_assert(!ROPE || (WB && !GROUPED && BN % 128 == 0 && BN / WAVES_N == 64), "two waves a head");
  static_assert(!DIRECT || (WB && BM == 256 && BN / WAVES_N == 64), "W straight to registers: from blocks, four column tiles a wave");
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int TM = WTM / 16, TN = WTN / 16;  // 16x16 MFMA tiles per wave
  constexpr int A_INST = BM / RPI / NW, W_INST = BN / RPI / NW;
  constexpr int PER_TILE = A_INST + W_INST;
  constexpr int NM = TM * TN;                  // MFMAs per k-step
  constexpr int NF = TM + TN;                  // fragment reads per k-step
  constexpr int A_STAGES = 4;                  // DIRECT: stages of A alone
  static_assert(WTN == 64 && BK == 64 && TM % 2 == 0 && BM % (RPI * NW) == 0, "written for 64-column wave tiles, two k-steps");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* sA = (bf16_t*)smem_raw;
  bf16_t* sW = sA + NSTAGE * BM * BK;  // [WS][BN][BK], not DIRECT

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  f32x4 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;
  const int frow = lane & 15, fq = lane >> 4;
  // 16-column block of the tile that feeds the wave's column tile j
  auto col_block = [&](int j) { return ROPE ? wn / 2 * 8 + wn % 2 * 2 + j / 2 * 4 + j % 2 : wn * WTN / 16 + j; };
  // k-tiles of this workgroup: all of them, or share blockIdx.y of a contraction split over workgroups (C then holds
  // one fp32 plane of M x N partial sums per share)
  const int kt0 = (int)blockIdx.y * kt_per_split, n_kt = min(K / BK - kt0, kt_per_split);
  if (!GROUPED) C = (char*)C + (int64_t)blockIdx.y * M_all * ldc * ((epi & EPI_C_F32) ? 4 : 2);

  const int lr = lane / CH, lp = lane % CH;
  uint32_t a_off[A_INST];
#pragma unroll
  for (int i = 0; i < A_INST; ++i) {
    int row = RPI * (wave * A_INST + i) + lr;
    int ar = min(m0 + row, M - 1);
    if (GROUPED && a_row) ar = min(max(a_row[ar], 0), a_rows - 1);  // always inside A, whatever the table holds
    a_off[i] = (uint32_t)(((int64_t)ar * lda + (lp ^ ((row >> 1) & (CH - 1))) * 8) * 2);
  }
  const uint32_t sA_lds = (uint32_t)(uintptr_t)sA;

  if constexpr (DIRECT) {
    // W frag of column tile j: 1 KB blocks, two per k-tile and 16 columns
    uint32_t w_off[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
      w_off[j] = (uint32_t)min(n0 / 16 + col_block(j), N / 16 - 1) * (uint32_t)(ldw / 32) * (BLK * 2u) + lane * 16u;
    const auto w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, (uint32_t)((int64_t)N * ldw * 2), 0x00027000);
    bf16x8 wf[2][2][TN], xf[2 * TM];
    // tiles past the end repeat the last one: no branch splits the loop, and nothing uses what they bring
    auto load_w = [&](int buf, int t, int ks, int j) {
      const int at = (kt0 + min(t, n_kt - 1)) * (BK * 32) + ks * (BLK * 2);
      wf[buf][ks][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_off[j], at, 0));
    };
    auto load_a = [&](int t, int i) {
      const char* base = (const char*)A + (int64_t)(kt0 + min(t, n_kt - 1)) * (BK * 2);
      const uint32_t dst = sA_lds + (uint32_t)(t % A_STAGES * BM * BK + RPI * (wave * A_INST + i) * BK) * 2;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :
                   : "s"(dst), "v"(a_off[i]), "s"(base)
                   : "memory", "m0");
    };
    constexpr int NX = 2 * TM, AHEAD = 4;  // activation fragments of a k-tile; read AHEAD of their MFMAs
    const bf16_t* x_at[2] = {sA + slot(wm * WTM + frow, fq), sA + slot(wm * WTM + frow, 4 + fq)};
    auto read_x = [&](int stage, int f) { xf[f] = *(const bf16x8*)(x_at[f / TM] + stage * BM * BK + f % TM * 16 * BK); };

    // Loads return in the order in which they were issued.  The compiler counts those of W, not the direct ones of A, and
    // may move the former: so no wait counts on its order.  Whatever of W is requested behind pin() follows the loads of A in
    // front of it, and landed() lets the compiler wait for such loads of W, hence for that A too.
    auto pin = [&] { asm volatile("" : "+v"(w_off[0]), "+v"(w_off[1]), "+v"(w_off[2]), "+v"(w_off[3]) : : "memory"); };
    auto landed = [&](bf16x8* w) { asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]) : : "memory"); };
#pragma unroll
    for (int i = 0; i < 2 * A_INST; ++i) load_a(i / A_INST, i % A_INST);
    pin();
#pragma unroll
    for (int f = 0; f < 3 * TN; ++f) {
      load_w(f / (2 * TN), f / (2 * TN), f / TN % 2, f % TN);
      if (f == TN - 1) pin();
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < A_INST; ++i) load_a(2, i);
    pin();
    landed(wf[0][0]);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) read_x(0, f);

    auto tile_step = [&](auto buf_, int t) {
      constexpr int buf = buf_();
      const int stage = t % A_STAGES, next = (t + 1) % A_STAGES;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < NX; ++f) {
        if (f == NX - AHEAD) {
          // A(t + 1) is older than this k-step's W, so it has landed for every wave; and every wave is past its reads of
          // tile t - 1, whose stage takes A(t + 3)
          landed(wf[buf][1]);
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        const int i = f % TM, ks = f / TM;
#pragma unroll
        for (int u = 0; u < TN; ++u) {
          const int j = f & 1 ? TN - 1 - u : u;  // there and back: one operand changes from each MFMA to the next
          acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[buf][ks][j], xf[f], acc[j][i], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (u == 0) {
            if (f + AHEAD < NX) read_x(stage, f + AHEAD);
            else read_x(next, f + AHEAD - NX);
          }
          if (u == 2 && i < TN) {
            if (ks == 0) load_w(buf ^ 1, t + 1, 1, i);
            else load_w(buf, t + 2, 0, i);
          }
          if (u == 3 && f >= NX - AHEAD) {
            constexpr int per = A_INST / AHEAD;
#pragma unroll
            for (int q = 0; q < per; ++q) load_a(t + 3, (f - (NX - AHEAD)) * per + q);
            if (f == NX - 1) pin();
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    int t = 0;
    do {  // at least two k-tiles
      tile_step(std::integral_constant<int, 0>{}, t);
      tile_step(std::integral_constant<int, 1>{}, t + 1);
      t += 2;
    } while (t + 1 < n_kt);
    if (t < n_kt) tile_step(std::integral_constant<int, 0>{}, t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the epilogue's staging takes the ring
    __syncthreads();
  } else {
    uint32_t w_off[W_INST];
#pragma unroll
    for (int i = 0; i < W_INST; ++i) {
      const int row = RPI * (wave * W_INST + i) + lr, blk = wave * W_INST + i;  // WB: block blk % 2 of rows 16 * (blk / 2) ..
      w_off[i] = WB ? (uint32_t)(min(n0 / 16 + blk / 2, N / 16 - 1) * (int)(ldw / 32) + blk % 2) * (BLK * 2u) + lane * 16u
                    : (uint32_t)(((int64_t)min(n0 + row, N - 1) * ldw + (lp ^ ((row >> 1) & (CH - 1))) * 8) * 2);
    }
    const uint32_t sW_lds = (uint32_t)(uintptr_t)sW;
    // load idx of a k-tile step: A of k-tile ta to stage sa, then W of k-tile tw to stage sw
    auto issue_load = [&](int sa, int ta, int sw, int tw, int idx) {
      const bool is_a = idx < A_INST;
      const int li = is_a ? idx : idx - A_INST;
      const char* base = is_a ? (const char*)A + (int64_t)(kt0 + ta) * (BK * 2) : (const char*)W + (int64_t)(kt0 + tw) * (BK * w_step<WB>());
      const uint32_t voff = is_a ? a_off[li] : w_off[li];
      const uint32_t dst = is_a ? sA_lds + (uint32_t)(sa * BM * BK + RPI * (wave * A_INST + li) * BK) * 2
                                : sW_lds + (uint32_t)(sw * BN * BK + RPI * (wave * W_INST + li) * BK) * 2;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :
                   : "s"(dst), "v"(voff), "s"(base)
                   : "memory", "m0");
    };

    // fragment f of a k-step, in the order the MFMAs (j outer, i inner) first need them: W 0, X 0..TM-1, W 1..TN-1
    bf16x8 xs[2][TM], ws[2][TN];
    auto read_frag = [&](const bf16_t* a_s, const bf16_t* w_s, int ks, int f) {
      const int ch = ks * 4 + fq;
      const int j = f == 0 ? 0 : f - TM;
      if (f >= 1 && f <= TM) xs[ks][f - 1] = *(const bf16x8*)(a_s + slot(wm * WTM + (f - 1) * 16 + frow, ch));
      else {
        ws[ks][j] = *(const bf16x8*)(w_s + (WB ? (col_block(j) * 2 + ks) * BLK + lane * 8 : slot(wn * WTN + j * 16 + frow, ch)));
      }
    };

    // Loads return in order.  In front of the loop: tile 0, tile 1, then W alone of the tiles up to WS - 1; only tile 0 is waited for.
#pragma unroll
    for (int i = 0; i < PER_TILE; ++i) issue_load(0, 0, 0, 0, i);
    if (n_kt >= WS) {
#pragma unroll
      for (int i = 0; i < PER_TILE; ++i) issue_load(1, 1, 1, 1, i);
#pragma unroll
      for (int u = 2; u < WS; ++u)
#pragma unroll
        for (int i = A_INST; i < PER_TILE; ++i) issue_load(0, 0, u, u, i);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_TILE + (WS - 2) * W_INST) : "memory");
    } else if (WS > 2 && n_kt > 1) {
#pragma unroll
      for (int i = 0; i < PER_TILE; ++i) issue_load(1, 1, 1, 1, i);
      if (n_kt > 2) {
#pragma unroll
        for (int i = A_INST; i < PER_TILE; ++i) issue_load(0, 0, 2, 2, i);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_TILE + W_INST) : "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_TILE) : "memory");
      }
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    static_assert(WS >= 2 && WS <= 4, "a contraction shorter than the ring: three k-tiles at most");
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) read_frag(sA, sW, 0, f);

    // k-tile t (stage w_at of W) brings A of t + 2 (n_ld = A_INST loads) and W of t + WS (n_ld = PER_TILE).  The wait in the middle of
    // k-step 1 is for A(t + 1) and W(t + 1).  Behind A(t + 1) come the loads of W that its step issued after it (w_behind: W(t + WS - 1),
    // or nothing more where W had ended) and the loads issued since; W(t + 1) is older where WS > 2 (for t = 0, where tile 1 ends with it, it is
    // followed by W of the tiles from 2 on, no fewer loads), and is W(t + WS - 1) itself where WS = 2.
    int w_at = 0;
    auto tile_step = [&](int t, auto has_next, auto n_ld_, auto w_behind) {
      constexpr int n_ld = n_ld_(), newer = NM / 2 * n_ld / NM + w_behind();
      const int stage = t & 1, w_next = w_at + 1 == WS ? 0 : w_at + 1;
      const bf16_t* a_s = sA + stage * BM * BK;
      const bf16_t* w_s = sW + w_at * BN * BK;
      const bf16_t* a_n = sA + (stage ^ 1) * BM * BK;
      const bf16_t* w_n = sW + w_next * BN * BK;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        if (ks == 1) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int m = j * TM + i;
            if (ks == 1 && m == NM / 2) {
              asm volatile("s_waitcnt vmcnt(%0)" ::"n"(newer) : "memory");
              __builtin_amdgcn_s_barrier();
              asm volatile("" ::: "memory");
            }
            // fragment reads between the MFMAs: k-step 1's during k-step 0 (done a quarter before its end), the
            // next tile's first ones during the second half of k-step 1
            if (ks == 0 && m >= 1) {
              constexpr int D = NM * 3 / 4 - 1;
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int f = min(NF, (m - 1) * NF / D); f < min(NF, m * NF / D); ++f) read_frag(a_s, w_s, 1, f);
              __builtin_amdgcn_sched_barrier(0);
            }
            if (ks == 1 && has_next && m > NM / 2) {
              constexpr int D = NM / 2 - 2;
              const int mm = m - NM / 2;
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int f = min(NF, (mm - 1) * NF / D); f < min(NF, mm * NF / D); ++f) read_frag(a_n, w_n, 0, f);
              __builtin_amdgcn_sched_barrier(0);
            }
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws[ks][j], xs[ks][i], acc[j][i], 0, 0, 0);
            if (ks == 1 && n_ld > 0) {
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int q = m * n_ld / NM; q < (m + 1) * n_ld / NM; ++q) issue_load(stage, t + 2, w_at, t + WS, q);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      w_at = w_next;
    };
    int t = 0;
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, A_INST> a_only{};
    constexpr std::integral_constant<int, PER_TILE> a_and_w{};
    constexpr std::integral_constant<int, (WS > 2 ? W_INST : 0)> w_last{};
    for (; t + WS < n_kt; ++t) tile_step(t, std::true_type{}, a_and_w, w_last);
    if (WS > 2 && t + 2 < n_kt) { tile_step(t, std::true_type{}, a_only, w_last); ++t; }
    if (WS > 3 && t + 2 < n_kt) { tile_step(t, std::true_type{}, a_only, none); ++t; }
    if (t + 1 < n_kt) { tile_step(t, std::true_type{}, none, none); ++t; }
    if (t < n_kt) tile_step(t, std::false_type{}, none, none);
  }

  // ---- epilogue through the wave's own LDS region, 32 rows at a time (as in the 32x32 kernel) ----
  constexpr int ROW_F = 64 + 4;
  float* stage_f = (float*)smem_raw + wave * (32 * ROW_F);
  static_assert(NW * 32 * ROW_F * 4 <= lds16<BM, BN, DIRECT, WS>(), "staging region fits the tile ring");
  const bool swiglu = (epi & EPI_SWIGLU) != 0;
  int lane_e = lane;
  asm volatile("" : "+v"(lane_e));  // indices derived after the k loop: not kept in registers across it
  const int er = lane_e & 15, eq = lane_e >> 4;
  const int rr = lane_e >> 4, c4 = (lane_e & 15) * 4;
  const int rr_s = lane_e >> 3, c4_s = (lane_e & 7) * 4;
  if constexpr (ROPE) {
    const int head = n0 / 128 + wn / 2, p0 = wn % 2 * 32;
    if (head >= ro.Hq + 2 * ro.Hkv) return;  // uniform over the wave; no barrier follows
    const bool rotates = head < ro.Hq + ro.Hkv;
    bf16_t* out = head < ro.Hq ? (bf16_t*)C + head * 128 : rotates ? ro.k + (head - ro.Hq) * 128 : ro.v + (head - ro.Hq - ro.Hkv) * 128;
    const int64_t ldo = head < ro.Hq ? ldc : ro.Hkv * 128;
    f32x4 cs[2][2][2][2];  // [ib % 2][h][j][.]: (cos, sin) of the lane's four pairs, requested one block of 32 rows ahead
    auto request = [&](int ib) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int m = min(m0 + wm * WTM + ib * 32 + 16 * h + er, M - 1);
          const f32x4* src = (const f32x4*)(ro.cs + (int64_t)m * 64 + p0 + 16 * j + 4 * eq);
          cs[ib % 2][h][j][0] = src[0];
          cs[ib % 2][h][j][1] = src[1];
        }
    };
    if (rotates) request(0);
#pragma unroll
    for (int ib = 0; ib < TM / 2; ++ib) {
      if (rotates && ib + 1 < TM / 2) request(ib + 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = 2 * ib + h;
        float* rowp = stage_f + (16 * h + er) * ROW_F + 4 * eq;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 y1 = acc[j][i], y2 = acc[j + 2][i];
          if (rotates) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float c = cs[ib % 2][h][j][e / 2][e % 2 * 2], sn = cs[ib % 2][h][j][e / 2][e % 2 * 2 + 1];
              const float a = y1[e], b = y2[e];
              y1[e] = a * c - b * sn;
              y2[e] = b * c + a * sn;
            }
          }
          *(f32x4*)(rowp + 16 * j) = y1;
          *(f32x4*)(rowp + 16 * (j + 2)) = y2;
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int r = it * 4 + rr, m = m0 + wm * WTM + ib * 32 + r;
        const f32x4 v = *(const f32x4*)(stage_f + r * ROW_F + c4);
        if (m < M) store_quad(out, ldo, nullptr, 0, m, p0 + (c4 & 31) + (c4 & 32) * 2, v, EPI_STORE);
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
#pragma unroll
  for (int ib = 0; ib < TM / 2; ++ib) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = 2 * ib + h;
      float* rowp = stage_f + (16 * h + er) * ROW_F + 4 * eq;
      if (swiglu) {
        // gate rows are the first 32 W rows of the wave's 64, up rows the next 32: tiles j and j + TN/2
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = acc[j][i][e], u = acc[j + TN / 2][i][e];
            const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
            o[e] = g * sig * u;
          }
          *(f32x4*)(rowp + 16 * j) = o;
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4*)(rowp + 16 * j) = acc[j][i];
      }
    }
    __builtin_amdgcn_wave_barrier();
    const int mb = m0 + wm * WTM + ib * 32;
    if (swiglu) {
      const int fb = (n0 + wn * WTN) / 2;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = it * 8 + rr_s, m = mb + r, f = fb + c4_s;
        const f32x4 v = *(const f32x4*)(stage_f + r * ROW_F + c4_s);
        if (m < M && f < N / 2) {
          bf16x4 o;
          o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
          *(bf16x4*)((bf16_t*)C + (int64_t)m * ldc + f) = o;
        }
      }
    } else {
      const int n = n0 + wn * WTN + c4;
      f32x4 res[8];
      if (epi & EPI_RESIDUAL) {
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int m = min(mb + it * 4 + rr, M - 1), nn = min(n, N - 4);
          if (epi & EPI_R_F32) {
            res[it] = *(const f32x4*)((const float*)R + (int64_t)m * ldr + nn);
          } else {
            const bf16x4 rb = *(const bf16x4*)((const bf16_t*)R + (int64_t)m * ldr + nn);
            res[it][0] = (float)rb[0]; res[it][1] = (float)rb[1]; res[it][2] = (float)rb[2]; res[it][3] = (float)rb[3];
          }
        }
      }
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int r = it * 4 + rr, m = mb + r;
        f32x4 v = *(const f32x4*)(stage_f + r * ROW_F + c4);
        if (epi & EPI_RESIDUAL) v += res[it];
        if (m < M && n < N) store_quad(C, ldc, nullptr, 0, m, n, v, epi & ~(EPI_RESIDUAL | EPI_R_F32));
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool WB, bool GROUPED = false, bool ROPE = false, bool DIRECT = false, bool LOW = false,
          int WS = w_stages<BM>()>
__global__ void __launch_bounds__(WAVES_M* WAVES_N * 64)
    gemm16_bf16_kernel(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W_all, int64_t ldw,
                       void* C, int64_t ldc, const void* __restrict__ R, int64_t ldr, int M_all, int N, int K,
                       int epi, int tiles_m, int tiles_n, int kt_per_split, const int4* __restrict__ tile_tab,
                       int64_t w_group_stride, const int32_t* __restrict__ a_row, int a_rows, RopeOut ro) {
  int pid = blockIdx.x;
  int nb = gridDim.x;
  bool behind = false;
  if constexpr (GROUPED) {
    // the grid is sized for the worst case; the tiles that exist are the first ones of the table, and only their
    // workgroups are spread over the dies (the rest, the highest block ids, leave at once).  Low tiles that stand behind all
    // others are spread by themselves.
    const int4 counts = tile_tab[tiles_m];
    nb = min(counts.x, tiles_m) * tiles_n;
    if (LOW && pid >= nb) {
      behind = true;
      pid -= nb;
      nb = min(counts.y, tiles_m - min(counts.x, tiles_m)) * ((N + MOE_LOW_COLS - 1) / MOE_LOW_COLS);
    }
    if (pid >= nb) return;
  }
  {
    const int q = nb / N_XCD, rem = nb % N_XCD;
    const int xcd = pid % N_XCD, loc = pid / N_XCD;
    pid = (xcd < rem) ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
  }
  if constexpr (GROUPED) {
    int4 te;
    int n0;
    if (behind) {
      const int cols = (N + MOE_LOW_COLS - 1) / MOE_LOW_COLS;
      te = tile_tab[min(tile_tab[tiles_m].x, tiles_m) + pid / cols];
      n0 = pid % cols * MOE_LOW_COLS;
    } else {
      // A scheduling group is of one expert, and a balanced expert is one group: a die then streams that expert's W once.  In
      // groups of four, which straddle experts, gate/up over 16384 rows of eight experts (8B widths) took 2949 us (2833), down
      // 1687 (1650).  The workgroups of a group are one range of ids, whatever its size.
      const int packed = tile_tab[pid / tiles_n].w;
      const int first_m = packed & ((1 << MOE_GROUP_SHIFT) - 1), gsz = packed >> MOE_GROUP_SHIFT, in_group = pid - first_m * tiles_n;
      te = tile_tab[first_m + in_group % gsz];
      n0 = in_group / gsz * BN;
    }
    if (te.x < 0) return;  // uniform over the workgroup, before any barrier
    const bf16_t* W = W_all + (int64_t)te.x * w_group_stride;
    if constexpr (LOW) {
      if (behind) {
        gemm16_tile<MOE_LOW_ROWS, MOE_LOW_COLS, 4, 2, WB, GROUPED, ROPE, false>(A, lda, W, ldw, C, ldc, R, ldr, te.y, n0, te.z, M_all, N, K, epi,
                                                                               kt_per_split, a_row, a_rows, ro);
        return;
      }
    }
    gemm16_tile<BM, BN, WAVES_M, WAVES_N, WB, GROUPED, ROPE, DIRECT>(A, lda, W, ldw, C, ldc, R, ldr, te.y, n0, te.z, M_all, N, K, epi,
                                                                    kt_per_split, a_row, a_rows, ro);
  } else {
    const int per_group = GROUP_M * tiles_n, group = pid / per_group, first_m = group * GROUP_M;
    const int gsz = min(GROUP_M, tiles_m - first_m), in_group = pid - group * per_group;
    gemm16_tile<BM, BN, WAVES_M, WAVES_N, WB, GROUPED, ROPE, DIRECT, WS>(A, lda, W_all, ldw, C, ldc, R, ldr, (first_m + in_group % gsz) * BM,
                                                                        in_group / gsz * BN, M_all, M_all, N, K, epi, kt_per_split, a_row,
                                                                        a_rows, ro);
  }
}

// Sum over the K splits of the quads at P + k * stride, k = 0 .. splits-1, added in split order.  The reductions are
// short chains of dependent steps on little data: what they take is round trips to memory, so the loads of four
// splits are requested together.
__device__ __forceinline__ f32x4 sum_splits(const float* __restrict__ p, int64_t stride, int splits) {
  f32x4 a = *(const f32x4*)p;
  int k = 1;
  for (; k + 3 < splits; k += 4) {
    f32x4 b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = *(const f32x4*)(p + (k + u) * stride);
#pragma unroll
    for (int u = 0; u < 4; ++u) a += b[u];
  }
  {  // the last one to three splits, requested together as well
    f32x4 b[3];
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (k + u < splits) b[u] = *(const f32x4*)(p + (k + u) * stride);
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (k + u < splits) a += b[u];
  }
  return a;
}
// C[m][n] = bf16( sum_s P[s][m][n] (+ R[m][n]) ), the partials added in split order.
__global__ void __launch_bounds__(256) splitk_reduce_kernel(const float* __restrict__ P, void* __restrict__ C, int64_t ldc,
                                                            const void* __restrict__ R, int64_t ldr, int M, int N,
                                                            int splits, int epi) {
  const int64_t quads = (int64_t)M * (N / 4);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= quads) return;
  const int m = (int)(i / (N / 4)), n = (int)(i - (int64_t)m * (N / 4)) * 4;
  const f32x4 s = sum_splits(P + (int64_t)m * N + n, (int64_t)M * N, splits);
  store_quad(C, ldc, R, ldr, m, n, s, epi);
}

// The QKV projection's partial sums, followed by what rope_kv_write_kernel does: q and k heads rotated with the (cos, sin)
// table of the tokens (pairs (i, i + dh/2)), q written to the qkv buffer, rotated k and v to the rows of the cache.
// One thread per 4 rotary pairs, or per 4 values of v.
__global__ void __launch_bounds__(256) splitk_reduce_rope_kernel(const float* __restrict__ P, bf16_t* __restrict__ qkv, int64_t ldq,
                                                                 const float2* __restrict__ cs, bf16_t* __restrict__ k_rows,
                                                                 bf16_t* __restrict__ v_rows, int M, int N, int splits, int Hq,
                                                                 int Hkv, int dh) {
  const int half = dh / 2, kvw = Hkv * dh;
  const int rot_units = (Hq + Hkv) * (half / 4), v_units = kvw / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)M * (rot_units + v_units)) return;
  const int m = (int)(i / (rot_units + v_units)), u = (int)(i - (int64_t)m * (rot_units + v_units));
  const float* row = P + (int64_t)m * N;
  const int64_t stride = (int64_t)M * N;
  auto store = [](bf16_t* dst, f32x4 v) {
    bf16x4 o;
    o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
    *(bf16x4*)dst = o;
  };
  if (u < rot_units) {
    const int head = u / (half / 4), i0 = (u % (half / 4)) * 4;
    const f32x4 x1 = sum_splits(row + head * dh + i0, stride, splits), x2 = sum_splits(row + head * dh + i0 + half, stride, splits);
    f32x4 y1, y2;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2 c = cs[(int64_t)m * half + i0 + e];
      y1[e] = x1[e] * c.x - x2[e] * c.y;
      y2[e] = x2[e] * c.x + x1[e] * c.y;
    }
    bf16_t* dst = head < Hq ? qkv + (int64_t)m * ldq + head * dh + i0 : k_rows + (int64_t)m * kvw + (head - Hq) * dh + i0;
    store(dst, y1);
    store(dst + half, y2);
  } else {
    const int j = (u - rot_units) * 4;
    store(v_rows + (int64_t)m * kvw + j, sum_splits(row + (Hq + Hkv) * dh + j, stride, splits));
  }
}

// The partial sums of a projection with residual whose result feeds an RMSNorm, one workgroup per token row: writes the
// fp32 residual stream h = sums + R and xn = h * rsqrt(mean(h^2) + eps) * g in bf16.  d <= 1024 * NCH, a multiple of 4.
template <int NCH>
__global__ void __launch_bounds__(256) splitk_reduce_rmsnorm_kernel(const float* __restrict__ P, float* h, const void* R, int r_f32,
                                                                    const bf16_t* __restrict__ g, bf16_t* __restrict__ xn, int M,
                                                                    int d, int splits, float eps) {
  __shared__ float part[4];
  const int m = blockIdx.x;
  f32x4 v[NCH];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int n = (threadIdx.x + c * 256) * 4;
    if (n >= d) continue;
    f32x4 a = sum_splits(P + (int64_t)m * d + n, (int64_t)M * d, splits);
    if (r_f32) {
      a += *(const f32x4*)((const float*)R + (int64_t)m * d + n);
    } else {
      const bf16x4 r = *(const bf16x4*)((const bf16_t*)R + (int64_t)m * d + n);
      a[0] += (float)r[0]; a[1] += (float)r[1]; a[2] += (float)r[2]; a[3] += (float)r[3];
    }
    *(f32x4*)(h + (int64_t)m * d + n) = a;
    v[c] = a;
    ss += a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float r = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)d + eps);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int n = (threadIdx.x + c * 256) * 4;
    if (n >= d) continue;
    const bf16x4 gg = *(const bf16x4*)(g + n);
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16_t)(v[c][e] * r * (float)gg[e]);
    *(bf16x4*)(xn + (int64_t)m * d + n) = o;
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool PARTIAL, int SCHED, bool WB>
hipError_t launch_form(const void* A, int64_t lda, const void* W, int64_t ldw, void* C, int64_t ldc, const void* R, int64_t ldr,
                  float* P, int M, int N, int K, int epi, int splits, int kt_per_split, hipStream_t s) {
  auto kern = gemm_bf16_kernel<BM, BN, WAVES_M, WAVES_N, PARTIAL, SCHED, WB>;
  constexpr int lds = NSTAGE * (BM + BN) * BK * 2;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  DSK_LAUNCH_TIMED(kern, dim3(tiles_m * tiles_n, splits), dim3(WAVES_M * WAVES_N * 64), lds, s, (const bf16_t*)A, lda,
                   (const bf16_t*)W, ldw, C, ldc, R, ldr, P, M, N, K, epi, tiles_m, tiles_n, kt_per_split);
  return hipGetLastError();
}

// W in rows or in blocks, as the caller has it.  (The 64-row tiles meet blocks only in a model that was created under
// "force_generic" with a head_dim the attention kernels do not take and runs without it.)
template <int BM, int BN, int WAVES_M, int WAVES_N, bool PARTIAL, int SCHED = 0>
hipError_t launch(const void* A, int64_t lda, const void* W, int64_t ldw, int w_blocks, void* C, int64_t ldc, const void* R, int64_t ldr,
                  float* P, int M, int N, int K, int epi, int splits, int kt_per_split, hipStream_t s) {
  return w_blocks ? launch_form<BM, BN, WAVES_M, WAVES_N, PARTIAL, SCHED, true>(A, lda, W, ldw, C, ldc, R, ldr, P, M, N, K, epi, splits, kt_per_split, s)
                  : launch_form<BM, BN, WAVES_M, WAVES_N, PARTIAL, SCHED, false>(A, lda, W, ldw, C, ldc, R, ldr, P, M, N, K, epi, splits, kt_per_split, s);
}

// Whether a launch of unsplit 256-row tiles takes W in blocks straight to registers (DIRECT); rows: those that share W, of an
// expert the average.  Some 220 launches, widths of 1024 to 8192 and 512 to 16384 rows, both forms in turn; time of DIRECT over
// that of the other form:
//   QKV, O and down: contractions of 4096 and longer 0.95 to 1.00 (2048 rows, QKV 4096 wide 93.3 -> 90.9 us; 8192 rows, down 14336
//   long 662 -> 638), of 3584 0.98 to 1.00, of 3072 and 2048 0.97 to 1.01 (layers 3072 wide over 4096 and 8192 rows 1.01), of 1024 1.00
//   to 1.01.
//   gate/up, whose W is the longest stream for its rows: 4096 wide 1.02 at 1536 rows, 1.01 at 4096, 0.99 at 8192, 0.985 at 16384;
//   5120 wide 1.02 at 1024, 1.00 at 6144, 0.986 at 7000; 8192 wide 1.01 at 1024, 0.99 at 2048, 0.97 at 8192; 2048 wide 1.01 to 1.03.
//   Experts: one row tile each 1.02 to 1.06 (W comes once, from HBM, and wants the longer lead); more than one: down 0.96 to 1.02,
//   mean 0.98, gate/up 0.97 to 1.02, mean 1.00.
// Lower tiles and split contractions keep the other form: half as many MFMAs share a fragment of W, or few k-tiles share the start (O
// over 1536 rows, 128-row tiles, 62.7 -> 64.9 us; down over 333 rows, 192-row tiles in eight splits, 54.4 -> 55.1 us; unsplit
// 192-row tiles were not measured).  (The loop of DIRECT wants two k-tiles at least.)
std::atomic<int64_t> g_direct_launches{0};
bool w_direct(int64_t rows, int K, bool gate_up) {
  if (gate_up) return K >= 8192 ? rows >= 1536 : K >= 3584 && rows * K >= (int64_t)1 << 25;
  return K >= 3584 && rows > 256;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool WB, bool DIRECT = false, int WS = w_stages<BM>()>
hipError_t launch16_form(const void* A, int64_t lda, const void* W, int64_t ldw, void* C, int64_t ldc, const void* R, int64_t ldr,
                         int M, int N, int K, int epi, int splits, int kt_per_split, hipStream_t s) {
  auto kern = gemm16_bf16_kernel<BM, BN, WAVES_M, WAVES_N, WB, false, false, DIRECT, false, WS>;
  constexpr int lds = lds16<BM, BN, DIRECT, WS>();
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  DSK_LAUNCH_TIMED(kern, dim3(tiles_m * tiles_n, splits), dim3(WAVES_M * WAVES_N * 64), lds, s, (const bf16_t*)A, lda,
                   (const bf16_t*)W, ldw, C, ldc, R, ldr, M, N, K, epi, tiles_m, tiles_n, kt_per_split, (const int4*)nullptr,
                   (int64_t)0, (const int32_t*)nullptr, 0, RopeOut{});
  g_direct_launches += DIRECT;
  return hipGetLastError();
}

template <int BM, bool DIRECT>
hipError_t launch16_rope(const void* A, const void* W, void* qkv, const RopeOut& ro, int M, int K, hipStream_t s) {
  auto kern = gemm16_bf16_kernel<BM, 256, 2, 4, true, false, true, DIRECT>;
  constexpr int lds = lds16<BM, 256, DIRECT>();
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int N = (ro.Hq + 2 * ro.Hkv) * 128, tiles_m = (M + BM - 1) / BM, tiles_n = (N + 255) / 256;
  DSK_LAUNCH_TIMED(kern, dim3(tiles_m * tiles_n), dim3(512), lds, s, (const bf16_t*)A, (int64_t)K, (const bf16_t*)W, (int64_t)K, qkv,
                   (int64_t)N, (const void*)nullptr, (int64_t)0, M, N, K, (int)EPI_STORE, tiles_m, tiles_n, K / BK,
                   (const int4*)nullptr, (int64_t)0, (const int32_t*)nullptr, 0, ro);
  g_direct_launches += DIRECT;
  return hipGetLastError();
}

// bm: rows of the tile (128, 192 or 256; 256 columns).  splits > 1: fp32 partial planes in C, epi = EPI_C_F32.
hipError_t launch16(int bm, const void* A, int64_t lda, const void* W, int64_t ldw, int w_blocks, void* C, int64_t ldc, const void* R,
                    int64_t ldr, int M, int N, int K, int epi, int splits, int kt_per_split, hipStream_t s) {
#define DSK_FORM(BM, WS)                                                                                                             \
  (w_blocks ? launch16_form<BM, 256, 2, 4, true, false, WS>(A, lda, W, ldw, C, ldc, R, ldr, M, N, K, epi, splits, kt_per_split, s)   \
            : launch16_form<BM, 256, 2, 4, false, false, WS>(A, lda, W, ldw, C, ldc, R, ldr, M, N, K, epi, splits, kt_per_split, s))
  if (bm == 256 && w_blocks && splits == 1 && w_direct(M, K, epi & EPI_SWIGLU))
    return launch16_form<256, 256, 2, 4, true, true>(A, lda, W, ldw, C, ldc, R, ldr, M, N, K, epi, 1, kt_per_split, s);
  return bm == 128 ? (M <= 128 ? DSK_FORM(128, 2) : DSK_FORM(128, 4)) : bm == 192 ? DSK_FORM(192, 3) : DSK_FORM(256, 2);
#undef DSK_FORM
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool DIRECT, bool LOW = false>
hipError_t launch16_grouped(const void* A, int64_t lda, const int32_t* a_row, int a_rows, const void* W, int64_t ldw,
                            int64_t w_group_stride, void* C, int64_t ldc, int N, int K, int epi, const int4* tile_tab, int tile_rows,
                            int low_tiles, hipStream_t s) {
  auto kern = gemm16_bf16_kernel<BM, BN, WAVES_M, WAVES_N, true, true, false, DIRECT, LOW>;
  constexpr int own = lds16<BM, BN, DIRECT>(), of_low = lds16<MOE_LOW_ROWS, MOE_LOW_COLS, false>(), lds = LOW && of_low > own ? of_low : own;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_n = (N + BN - 1) / BN;
  const int low_n = (N + MOE_LOW_COLS - 1) / MOE_LOW_COLS;
  DSK_LAUNCH_TIMED(kern, dim3(tile_rows * tiles_n + low_tiles * (low_n - tiles_n)), dim3(WAVES_M * WAVES_N * 64), lds, s, (const bf16_t*)A, lda,
                   (const bf16_t*)W, ldw, C, ldc, (const void*)nullptr, (int64_t)0, 0, N, K, epi, tile_rows, tiles_n,
                   K / BK, tile_tab, w_group_stride, a_row, a_rows, RopeOut{});
  g_direct_launches += DIRECT;
  return hipGetLastError();
}

int g_variant = 0;

// How a projection over more than 64 rows runs: tile rows (256 columns) and over how many workgroups its contraction is
// split.  A tile of 256 x 256 needs the fewest operand bytes per flop and is the best one where it fills the chip; where
// it does not, a lower tile makes better-filled rounds, and below one round the contraction is split (fp32 partial
// planes, fixed-order reduction).  The times below, in microseconds, are fits to measurements on the 8B projections over 96
// to 3000 rows with cold weights (in brackets the 128 x 128 tiles with split contraction this replaces):
//   QKV 333 rows 32.8 [43.0], 1500 rows 71.7 [91.7], 3000 rows 140 [165];  O 333 rows 27.8 [35.8], 3000 rows 85 [96];
//   down 333 rows 55 [81], 700 rows 85 [135], 1500 rows 149 [207].
// The times of 256-row tiles are those of the form that brings W through LDS; where w_direct takes the other one they are 0 to 5 %
// too long.  Those of 128- and 192-row tiles are of two stages of W; with the stages that these have now (w_stages) they are up to 6 %
// too long.  The choices reflect neither.
struct GemmPlan { int bm, splits, per, head_rows, rest_bm; };

// the best single launch and its time (a matter of the sizes alone: the scratch holds every split, gemm_mfma_split_bytes)
float plan_one(int M, int N, int K, bool may_split, bool full_tile, GemmPlan* plan) {
  const int KT = K / BK, bms[3] = {256, 192, 128};
  const bool fills = (int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 192;  // gemm_mfma_uses_prefill_tile
  GemmPlan best = {256, 1, KT, 0, 0};
  float best_us = 1e30f;
  for (int i = 0; i < 3; ++i) {
    const int bm = bms[i];
    if (full_tile && bm != 256) break;
    const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + 255) / 256);
    const int max_sp = fills || !may_split || tiles > 128 ? 1 : (int)(256 / tiles);
    for (int want = 1; want <= max_sp && (want == 1 || KT / want >= 4); ++want) {
      const int per = (KT + want - 1) / want, sp = (KT + per - 1) / per;
      if (sp != want) continue;
      const float rounds = (float)(tiles * sp) / 256.0f, fill = rounds < 1.f ? rounds : 1.f;
      // microseconds per k-tile of 64: busier chips clock lower and share the L2s
      const float kt_us = bm == 256 ? 1.08f + 0.42f * fill : bm == 192 ? 0.97f + 0.30f * fill : 0.85f + 0.15f * fill;
      // a last round that is not full costs most of a full one; less with lower tiles
      const float whole = floorf(rounds), frac = rounds - whole;
      const float tail = bm == 256 ? 0.75f + 0.25f * frac : bm == 192 ? 0.53f + 0.2f * frac : 0.45f + 0.4f * frac;
      const float n_rounds = rounds <= 1.f ? 1.f : whole + (frac > 0.f ? tail : 0.f);
      float us = n_rounds * (per * kt_us + 4.f);
      if (sp > 1) us += 4.5f + (float)sp * M * N * 8.f / 5.0e6f;
      if (us < best_us * 0.99f) {
        best_us = us;
        best = {bm, sp, per, 0, 0};
      }
    }
  }
  *plan = best;
  return best_us;
}

// ... and where a last round would stay partly empty, the rows of the whole rounds (head_rows, 256-row tiles) and the rest run as
// two launches, the rest in tiles of rest_bm rows.  Neither is split and both are the same kernel, so that a row's sums keep
// their order whatever the number of rows around it.  QKV over 4096 rows (1.5 rounds) 174 -> 162 us, over 8500 rows 348 -> 325 us;
// down over 13300 rows (3.25 rounds) 1271 -> 1184 us.
GemmPlan gemm_plan(int M, int N, int K, bool may_split) {
  GemmPlan best, head, rest;
  const float us = plan_one(M, N, K, may_split, false, &best);
  const int tiles_n = (N + 255) / 256;
  const int64_t rounds = (int64_t)((M + 255) / 256) * tiles_n / 256;
  const int64_t head_rows = rounds * 256 / tiles_n * 256;
  if (best.splits == 1 && rounds >= 1 && head_rows >= 256 && M - head_rows > 64) {
    const float two = plan_one((int)head_rows, N, K, false, true, &head) +
                      plan_one((int)(M - head_rows), N, K, false, false, &rest) + 2.f;
    if (two < us * 0.97f) best = {256, 1, K / BK, (int)head_rows, rest.bm};
  }
  return best;
}

}  // namespace

void gemm_mfma_set_variant(int v) { g_variant = v; }
int64_t gemm_mfma_direct_launches(int reset) { return reset ? g_direct_launches.exchange(0) : g_direct_launches.load(); }

// How a projection over few token rows (M <= 64) is split: 64x64 tiles and about 768 workgroups; a very wide N
// (the gate/up projection) has enough 64x128 tiles to fill the chip with few splits, which halves the share of the
// token rows in the tile loads (measured on M = 64, N = 28672, K = 4096: 54 us against 64 us; narrower shapes are
// best left as they are).  Returns whether the K-split path can run (more than one split, partials fit in ws).
static bool small_m_plan(int M, int N, int K, int64_t ws_bytes, bool* wide, int* splits, int* per) {
  const int KT = K / BK;
  *wide = (N + 127) / 128 >= 192;
  const int tiles = ((M + 63) / 64) * (*wide ? (N + 127) / 128 : (N + 63) / 64);
  int sp = ((*wide ? 512 : 768) + tiles - 1) / tiles;
  sp = max(1, min(sp, KT / 2));
  *per = (KT + sp - 1) / sp;
  *splits = (KT + *per - 1) / *per;
  return *splits > 1 && (int64_t)*splits * M * N * 4 <= ws_bytes;
}

// The fused gate/up epilogue needs whole 64-column gate/up blocks (few rows have kernels of their own, few_rows.hip).
bool gemm_mfma_swiglu_supported(int M, int N, int K) { return M > 64 && N % 64 == 0 && K >= BK && K % BK == 0; }

// 64 token rows x (splits x N) floats: about 768 tiles of 64 columns (+ one more split's worth) for the 64x64
// tiling, up to 4 splits of a wide N for the 64x128 tiling
int64_t gemm_mfma_workspace_bytes(int max_n) { return (int64_t)64 * 4 * ((int64_t)768 * 64 + (int64_t)4 * max_n); }

// What the partial planes of a split contraction take at most for up to max_m rows.  plan_one splits tiles so far that 256
// workgroups run, each with 256 x 256 sums or fewer, and gives every one of them at least four k-tiles.
int64_t gemm_mfma_split_bytes(int64_t max_m, int N, int K) {
  if (max_m <= 64) return 0;
  const int64_t most = (int64_t)256 * 256 * 256 * 4, shares = K / BK / 4 > 1 ? K / BK / 4 : 1;
  const int64_t bytes = max_m * N * shares * 4;
  return bytes < most ? bytes : most;
}

void gemm_mfma_plan(int M, int N, int K, int may_split, int32_t* plan) {
  const GemmPlan p = gemm_plan(M, N, K, may_split);
  plan[0] = p.bm; plan[1] = p.splits; plan[2] = p.head_rows; plan[3] = p.rest_bm;
}

// Whether a projection makes at least 192 tiles of 256 x 256: it fills the chip with them or with lower tiles of the same
// kernel, and its contraction is not split (what the timing hook and the roofline figure are about).
bool gemm_mfma_uses_prefill_tile(int M, int N) {
  return M > 64 && (int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 192;
}

hipError_t launch_gemm_mfma_bf16(const void* A, int64_t lda, const void* W, int64_t ldw, int w_blocks, void* C, int64_t ldc,
                                 const void* R, int64_t ldr, int M, int N, int K, int epi, void* ws, int64_t ws_bytes,
                                 hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K < BK || K % BK || N % 4 || (lda & 7) || (ldw & 7) || (ldc & 3) || ((epi & EPI_RESIDUAL) && (ldr & 3)))
    return hipErrorNotSupported;
  // rows are addressed by 32-bit byte offsets from the matrix base
  if ((int64_t)M * lda * 2 >= ((int64_t)1 << 32) || (int64_t)N * ldw * 2 >= ((int64_t)1 << 32)) return hipErrorNotSupported;
  const int KT = K / BK;
  int variant = g_variant;
  if (epi & EPI_SWIGLU) {
    if (!gemm_mfma_swiglu_supported(M, N, K)) return hipErrorNotSupported;
    // up to 256 rows the 128 x 128 tiles, which fill the chip twice over (two workgroups per compute unit).  us, 8B gate/up, against
    // the 128 x 256 tiles of the plan: 96 rows 59 against 69, 128 rows 60 against 71; since those have four stages of W they are the
    // faster ones from 129 rows on (160 rows 69.5 against 65.2, 200 rows 70.4 against 67.4, 256 rows 77.0 against 70.6; 70B, 256 x 256
    // tiles of the plan, 200 rows 273 against 213), which the line does not reflect
    if (variant == 2 || (variant == 0 && M <= 256))
      return launch<128, 128, 2, 2, false, 1>(A, lda, W, ldw, w_blocks, C, ldc, R, ldr, nullptr, M, N, K, epi, 1, KT, s);
    if (variant == 1) return launch16(256, A, lda, W, ldw, w_blocks, C, ldc, R, ldr, M, N, K, epi, 1, KT, s);
  }
  if (variant == 0 && M > 64) {
    const GemmPlan p = gemm_plan(M, N, K, ws != nullptr && !(epi & EPI_SWIGLU));
    if (p.head_rows > 0) {
      // a pair of events taken for this call spans both launches
      const hipEvent_t stop = g_launch_ev_stop;
      g_launch_ev_stop = nullptr;
      hipError_t e = launch16(256, A, lda, W, ldw, w_blocks, C, ldc, R, ldr, p.head_rows, N, K, epi, 1, KT, s);
      if (e != hipSuccess) return e;
      g_launch_ev_stop = stop;
      const int64_t r = p.head_rows;
      return launch16(p.rest_bm, (const bf16_t*)A + r * lda, lda, W, ldw, w_blocks, (char*)C + r * ldc * (epi & EPI_C_F32 ? 4 : 2), ldc,
                      R ? (const char*)R + r * ldr * (epi & EPI_R_F32 ? 4 : 2) : nullptr, ldr, M - p.head_rows, N, K, epi, 1, KT, s);
    }
    if (p.splits == 1) return launch16(p.bm, A, lda, W, ldw, w_blocks, C, ldc, R, ldr, M, N, K, epi, 1, KT, s);
    if (ws_bytes < gemm_mfma_split_bytes(M, N, K)) return hipErrorNotSupported;
    hipError_t e = launch16(p.bm, A, lda, W, ldw, w_blocks, ws, N, nullptr, 0, M, N, K, EPI_C_F32, p.splits, p.per, s);
    if (e != hipSuccess) return e;
    const int64_t quads = (int64_t)M * (N / 4);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, (const float*)ws, C, ldc, R, ldr,
                       M, N, p.splits, epi);
    return hipGetLastError();
  }
  if (variant == 0) variant = 3;
  switch (variant) {
    case 3: {  // weight streaming: K split over workgroups, fp32 partial planes, fixed-order reduce
      bool wide;
      int splits, per;
      if (ws && small_m_plan(M, N, K, ws_bytes, &wide, &splits, &per)) {
        hipError_t e = wide ? launch<64, 128, 1, 4, true>(A, lda, W, ldw, w_blocks, C, ldc, R, ldr, (float*)ws, M, N, K, epi, splits, per, s)
                            : launch<64, 64, 1, 2, true>(A, lda, W, ldw, w_blocks, C, ldc, R, ldr, (float*)ws, M, N, K, epi, splits, per, s);
        if (e != hipSuccess) return e;
        const int64_t quads = (int64_t)M * (N / 4);
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, (const float*)ws,
                           C, ldc, R, ldr, M, N, splits, epi);
        return hipGetLastError();
      }
      return launch<64, 64, 1, 2, false>(A, lda, W, ldw, w_blocks, C, ldc, R, ldr, nullptr, M, N, K, epi, 1, KT, s);
    }
    // the two prefill tilings by request: the 256x256 tile on the 16x16x32 MFMA (1), the 128x128 tile on the 32x32x16 MFMA (2)
    case 2: return launch<128, 128, 2, 2, false, 1>(A, lda, W, ldw, w_blocks, C, ldc, R, ldr, nullptr, M, N, K, epi, 1, KT, s);
    default: return launch16(256, A, lda, W, ldw, w_blocks, C, ldc, R, ldr, M, N, K, epi, 1, KT, s);
  }
}

// Row tile of the grouped projections: 256 rows, lower where an expert has fewer (all its rows in one tile, with room for
// the spread of a balanced router).  The lines are from tiles with two stages of W.
int moe_tile_rows_for(int64_t n_rows, int E) {
  const int64_t avg = n_rows / E;
  return avg <= 104 ? 128 : avg <= 168 ? 192 : 256;
}

// Projections of a mixture-of-experts layer over token rows sorted by expert: one launch over all experts.
// tile_tab[0..tile_rows) describes the tiles of tile_m rows and tile_tab[tile_rows] holds their number (see the kernel);
// rows of C are the sorted slots, rows of A too unless a_row says where they are.  low_tiles: how many low tiles the table may hold (0:
// it holds none).
// epi: EPI_SWIGLU (C bf16 [slots, N/2]) or EPI_C_F32 / EPI_STORE (C [slots, N]); no residual.
hipError_t launch_gemm_mfma_grouped(const void* A, int64_t lda, int64_t a_rows, const int32_t* a_row, const void* W, int64_t ldw,
                                    int w_blocks, int64_t w_group_stride, void* C, int64_t ldc, int N, int K, int epi,
                                    const void* tile_tab, int tile_m, int tile_rows, int low_tiles, int64_t rows_per_expert, hipStream_t s) {
  if (tile_rows <= 0) return hipSuccess;
  // (a model the tensor-core path takes has its weights in blocks)
  if (!w_blocks || K < BK || K % BK || N % 64 || (lda & 7) || (ldw & 7) || (ldc & 3) || (epi & EPI_RESIDUAL)) return hipErrorNotSupported;
  if (a_rows * lda * 2 >= ((int64_t)1 << 32) || (int64_t)N * ldw * 2 >= ((int64_t)1 << 32)) return hipErrorNotSupported;
  const bool direct = w_direct(rows_per_expert, K, false);
  auto f = tile_m == 128   ? launch16_grouped<128, 256, 2, 4, false>
           : tile_m == 192 ? launch16_grouped<192, 256, 2, 4, false>
           : low_tiles     ? (direct ? launch16_grouped<256, 256, 2, 4, true, true> : launch16_grouped<256, 256, 2, 4, false, true>)
           : direct        ? launch16_grouped<256, 256, 2, 4, true>
                           : launch16_grouped<256, 256, 2, 4, false>;
  return f(A, lda, a_row, (int)a_rows, W, ldw, w_group_stride, C, ldc, N, K, epi, (const int4*)tile_tab, tile_rows, low_tiles, s);
}

// More than 64 rows, dense operands: whether the contraction is split, i.e. a reduction runs behind the projection, which
// can then do the step that follows (the two launchers below).
bool gemm_mfma_splits(int M, int N, int K) {
  return g_variant == 0 && M > 64 && K >= BK && K % BK == 0 && N % 8 == 0 && (int64_t)M * K * 2 < ((int64_t)1 << 32) &&
         (int64_t)N * K * 2 < ((int64_t)1 << 32) && gemm_plan(M, N, K, true).splits > 1;
}

// QKV + RoPE + KV write: q rows in qkv [M, N], k and v only in the cache
hipError_t launch_gemm_split_rope(const void* A, const void* W, int w_blocks, void* qkv, const float2* cs, void* k_rows, void* v_rows,
                                  int M, int K, int Hq, int Hkv, int dh, void* ws, int64_t ws_bytes, hipStream_t s) {
  const int N = (Hq + 2 * Hkv) * dh;
  if (!ws || dh % 8 || !gemm_mfma_splits(M, N, K) || ws_bytes < gemm_mfma_split_bytes(M, N, K)) return hipErrorNotSupported;
  const GemmPlan p = gemm_plan(M, N, K, true);
  hipError_t e = launch16(p.bm, A, K, W, K, w_blocks, ws, N, nullptr, 0, M, N, K, EPI_C_F32, p.splits, p.per, s);
  if (e != hipSuccess) return e;
  const int64_t units = (int64_t)M * ((Hq + Hkv) * (dh / 8) + Hkv * dh / 4);
  hipLaunchKernelGGL(splitk_reduce_rope_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s, (const float*)ws,
                     (bf16_t*)qkv, (int64_t)N, cs, (bf16_t*)k_rows, (bf16_t*)v_rows, M, N, p.splits, Hq, Hkv, dh);
  return hipGetLastError();
}

// The same step where the contraction is not split: in the projection's epilogue.
bool gemm_mfma_rope_supported(int M, int N, int K, int w_blocks, int dh) {
  return g_variant == 0 && w_blocks && dh == 128 && M > 64 && K >= BK && K % BK == 0 && (int64_t)M * K * 2 < ((int64_t)1 << 32) &&
         (int64_t)N * K * 2 < ((int64_t)1 << 32);
}

hipError_t launch_gemm_rope(const void* A, const void* W, void* qkv, const float2* cs, void* k_rows, void* v_rows, int M, int K, int Hq,
                            int Hkv, hipStream_t s) {
  const int N = (Hq + 2 * Hkv) * 128;
  if (!gemm_mfma_rope_supported(M, N, K, 1, 128)) return hipErrorNotSupported;
  const GemmPlan p = gemm_plan(M, N, K, false);
  auto run = [&](int bm, int64_t r0, int64_t rows) {
    const RopeOut ro = {cs + r0 * 64, (bf16_t*)k_rows + r0 * Hkv * 128, (bf16_t*)v_rows + r0 * Hkv * 128, Hq, Hkv};
    auto f = bm == 128   ? launch16_rope<128, false>
             : bm == 192 ? launch16_rope<192, false>
             : w_direct(rows, K, false) ? launch16_rope<256, true>
                                            : launch16_rope<256, false>;
    return f((const bf16_t*)A + r0 * K, W, (bf16_t*)qkv + r0 * N, ro, (int)rows, K, s);
  };
  if (p.head_rows == 0) return run(p.bm, 0, M);
  const hipEvent_t stop = g_launch_ev_stop;  // a pair of events taken for this call spans both launches
  g_launch_ev_stop = nullptr;
  const hipError_t e = run(256, 0, p.head_rows);
  if (e != hipSuccess) return e;
  g_launch_ev_stop = stop;
  return run(p.rest_bm, p.head_rows, M - p.head_rows);
}

// h [M, d] fp32 = x W^T + R and xn [M, d] = rmsnorm(h) * g; d <= 8192
hipError_t launch_gemm_split_norm(const void* A, const void* W, int w_blocks, float* h, const void* R, int r_f32, const void* g, void* xn,
                                  float eps, int M, int d, int K, void* ws, int64_t ws_bytes, hipStream_t s) {
  if (!ws || d > 8192 || !gemm_mfma_splits(M, d, K) || ws_bytes < gemm_mfma_split_bytes(M, d, K)) return hipErrorNotSupported;
  const GemmPlan p = gemm_plan(M, d, K, true);
  hipError_t e = launch16(p.bm, A, K, W, K, w_blocks, ws, d, nullptr, 0, M, d, K, EPI_C_F32, p.splits, p.per, s);
  if (e != hipSuccess) return e;
  if (d <= 4096)
    hipLaunchKernelGGL(splitk_reduce_rmsnorm_kernel<4>, dim3(M), dim3(256), 0, s, (const float*)ws, h, R, r_f32, (const bf16_t*)g,
                       (bf16_t*)xn, M, d, p.splits, eps);
  else
    hipLaunchKernelGGL(splitk_reduce_rmsnorm_kernel<8>, dim3(M), dim3(256), 0, s, (const float*)ws, h, R, r_f32, (const bf16_t*)g,
                       (bf16_t*)xn, M, d, p.splits, eps);
  return hipGetLastError();
}
