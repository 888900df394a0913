// Internal declarations shared by the HIP sources of libdsk (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "dsk.h"

typedef __bf16 bf16_t;

// ---- element conversion (fp32 math everywhere; storage is float or bf16) ----
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return (bf16_t)x; }  // RNE (v_cvt_pk_bf16_f32)

// ---- packed weight layout ----
// QKV rows are [Wq; Wk; Wv].  Gate and up rows are interleaved in blocks of gu_block rows:
// packed rows [2*gu_block*j, 2*gu_block*j+gu_block) hold gate rows [gu_block*j, ..+gu_block),
// the next gu_block packed rows hold the same up rows, so that a GEMM tile owns gate and up of
// the same FFN index.
// The projections of a bf16 model are kept in blocks of 16 rows x 32 columns (dsk_model::w_blocks), each in the lane order of
// an MFMA operand: what the few-row kernels stream (few_rows.hip), and as good as rows for the tiled GEMMs.  Matrices
// whose widths are no whole blocks (fp32 models, test shapes) stay row-major.
__host__ __device__ inline int64_t block_at(int64_t r, int64_t k, int64_t K) {  // element offset of (r, k), K columns
  return ((r >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (r & 15)) * 8 + (k & 7);
}
struct LayerWeights {
  void* g1;
  void* wqkv;  // [(Hq+2Hkv)*dh, d]
  void* wo;    // [d, Hq*dh]
  void* g2;
  void* wgu;   // [2F, d] interleaved; a mixture-of-experts layer: [E][2F, d]
  void* wd;    // [d, F]; a mixture-of-experts layer: [E][d, F]
  void* wr;    // router [E, d] of a mixture-of-experts layer
};

constexpr int DSK_MAX_E_CHUNKS = 16;

// The rotary table of a call: cs[t][j] = (cos, sin) of pos[t] * theta[j], angle and sincos in fp64, stored as fp32.  The
// first norm of a bf16 call, and the first QKV projection of an fp32 one, fills it as well (a launch less in front of them).
struct RopeJob { const int32_t* pos; const double* theta; float2* cs; int T, half; };
__device__ __forceinline__ float2 rope_pair(const RopeJob& j, int t, int k) {  // of token t, pair k
  double s, c;
  sincos((double)j.pos[t] * j.theta[k], &s, &c);
  return make_float2((float)c, (float)s);
}
__device__ __forceinline__ void rope_entry(const RopeJob& j, int64_t i) {
  if (i >= (int64_t)j.T * j.half) return;
  const int t = (int)(i / j.half);
  j.cs[i] = rope_pair(j, t, (int)(i - (int64_t)t * j.half));
}
inline unsigned rope_blocks(const RopeJob& j) { return (unsigned)(((int64_t)j.T * j.half + 255) / 256); }

struct dsk_model {
  dsk_config_t cfg;
  int elem;         // bytes per element
  int64_t max_tokens;
  int64_t max_kv_rows;
  int gu_block;
  int n_qkv;        // (Hq+2Hkv)*dh
  LayerWeights* layers;
  int w_blocks;     // projections are in blocks (see above)
  int64_t weight_bytes;
  // workspace
  void* xn;         // [maxT, d]      normalised activations
  void* qkv;        // [maxT, n_qkv]
  void* attn;       // [maxT, Hq*dh]
  void* gu;         // [maxT, 2F], or what split_ws needs
  void* act;        // [maxT, F]
  float* h;         // [maxT, d]      residual stream between the layers of one call, kept in fp32
  void* e_stage;    // [maxT, d]      landing buffer for an E cache that arrives from pinned host memory
  float2* rope_cs;  // [maxT, dh/2]   cos, sin
  double* theta;    // [dh/2]         rope_base^(-2i/dh)
  void* vt;         // [Hkv*dh, ldvt] transposed V of the layer in flight (bf16 MFMA attention)
  int64_t ldvt;     // max_kv_rows rounded up to 64
  float* ssq;       // sums of squares of the few-row pass (RMSNorm split in two): [d/16][64], up to eight rows [rows][d/16]
  void* gemm_ws;    // fp32 partial tiles of the K-split small-M GEMM
  int64_t gemm_ws_bytes;
  void* split_ws;   // the same for more than 64 rows: gu where nothing else uses it there, else gemm_ws; large enough for
                    // every split, so that how a call is split does not hang on max_tokens
  int64_t split_ws_bytes;
  void* attn_ws;    // fp32 partial outputs of the key-split attention
  int64_t attn_ws_bytes;
  // mixture-of-experts layers (cfg.n_experts > 0)
  int32_t* moe_experts;  // [maxT, top_k] chosen experts
  float* moe_gates;      // [maxT, top_k] their gate weights
  int32_t* moe_slot;     // [maxT, top_k] row of the entry once the rows are grouped by expert
  int32_t* moe_src;      // [maxT*top_k]  token of every grouped row
  void* moe_tab;         // int4 [2][moe_tile_rows + 1] row tiles of the grouped projections and their numbers, gate/up's and down's
  int moe_tile_rows;
  float* moe_y;          // expert outputs, fp32: [maxT*top_k, d] grouped, or [E][n][d] when every expert runs over all rows
  int64_t moe_y_rows;
  int64_t workspace_bytes;
  // load pipeline
  hipStream_t load_stream;
  hipEvent_t ev_entry, ev_e, ev_all, ev_stage_free;
  hipEvent_t ev_e_chunk[DSK_MAX_E_CHUNKS];  // arrival of the row chunks of a host-resident E cache
  int32_t* chunk_cu;                        // device [DSK_MAX_E_CHUNKS][4]: {0, rows before the chunk, 0, rows of the chunk}
  hipEvent_t* ev_kv;        // [L]
  unsigned char* pending;   // [L] 1 if ev_kv[l] must be waited for by the suffix
  int any_pending;
  int load_mode;
  double throttle_gbps;        // > 0: loads are paced to this rate (emulates a slower link); 0 = off
  unsigned long long* pace_t0; // device: start time of the current call's loads (constant-rate clock ticks)
  int64_t paced_bytes;         // bytes handed to the load stream since pace_t0 was taken
};

// epilogues of the GEMM family
// bit 0: add R; bit 1: R is fp32 (else the model dtype); bit 2: C is fp32 (else the model dtype)
// bit 3 (bf16 MFMA kernel only): W is the interleaved gate/up matrix, C[M, N/2] = silu(gate) * up
enum { EPI_STORE = 0, EPI_RESIDUAL = 1, EPI_R_F32 = 2, EPI_C_F32 = 4, EPI_SWIGLU = 8 };

// ---- launchers (each validates nothing: the C-ABI layer has checked shapes) ----
// C[M,N] = A[M,K] * W[N,K]^T (+ R[M,N] when epi has EPI_RESIDUAL); row strides in elements.  w_blocks: W is in blocks.
hipError_t launch_gemm_generic(int dtype, const void* A, int64_t lda, const void* W, int64_t ldw, int w_blocks, void* C,
                               int64_t ldc, const void* R, int64_t ldr, int M, int N, int K, int epi, hipStream_t s);
// fp32 on the matrix instruction (fp32_mfma.hip).  The first asks whether rows are whole 16-byte pieces; the plain-ALU
// kernel takes the others.  The fused two: C = epilogue(rmsnorm(h) W^T) with RoPE + KV write (head_dim a multiple of 32)
// or SwiGLU (gate and up interleaved in blocks of 16 or 32) behind the projection.
bool gemm_fp32_supported(const void* A, int64_t lda, const void* W, int64_t ldw, const void* C, int64_t ldc, const void* R,
                         int64_t ldr, int M, int N, int K);
hipError_t launch_gemm_fp32(const void* A, int64_t lda, const void* W, int64_t ldw, void* C, int64_t ldc, const void* R,
                            int64_t ldr, int M, int N, int K, hipStream_t s);
hipError_t launch_gemm_fp32_norm_rope(const float* h, const void* gain, float eps, const void* wqkv, void* qkv, const float2* cs,
                                      void* k_rows, void* v_rows, int M, int d, int Hq, int Hkv, int dh, const RopeJob* job, hipStream_t s);
bool gemm_fp32_takes_rope(int M, int Hq, int Hkv, int dh);
hipError_t launch_gemm_fp32_norm_swiglu(const float* h, const void* gain, float eps, const void* wgu, void* act, int M, int d,
                                        int F, int gu_block, hipStream_t s);
// bf16 MFMA GEMM; returns hipErrorNotSupported when the shape is outside what it handles.
// ws: optional fp32 scratch for the partial tiles of a split contraction: gemm_mfma_workspace_bytes up to 64 rows,
// gemm_mfma_split_bytes beyond.
hipError_t launch_gemm_mfma_bf16(const void* A, int64_t lda, const void* W, int64_t ldw, int w_blocks, void* C, int64_t ldc,
                                 const void* R, int64_t ldr, int M, int N, int K, int epi, void* ws, int64_t ws_bytes,
                                 hipStream_t s);
int64_t gemm_mfma_workspace_bytes(int max_n);
int64_t gemm_mfma_split_bytes(int64_t max_m, int N, int K);  // scratch with which every split of up to max_m > 64 rows fits
bool gemm_mfma_swiglu_supported(int M, int N, int K);
// More than 64 rows with the contraction split over workgroups: the reduction does the step that follows, RoPE + KV write, or
// the RMSNorm of h = x W^T + R (d <= 8192).
bool gemm_mfma_splits(int M, int N, int K);
hipError_t launch_gemm_split_rope(const void* A, const void* W, int w_blocks, void* qkv, const float2* cs, void* k_rows, void* v_rows,
                                  int M, int K, int Hq, int Hkv, int dh, void* ws, int64_t ws_bytes, hipStream_t s);
// The QKV projection with RoPE + KV write in its epilogue (heads of 128, weights in blocks, contraction not split).
bool gemm_mfma_rope_supported(int M, int N, int K, int w_blocks, int dh);
hipError_t launch_gemm_rope(const void* A, const void* W, void* qkv, const float2* cs, void* k_rows, void* v_rows, int M, int K, int Hq,
                            int Hkv, hipStream_t s);
hipError_t launch_gemm_split_norm(const void* A, const void* W, int w_blocks, float* h, const void* R, int r_f32, const void* g, void* xn,
                                  float eps, int M, int d, int K, void* ws, int64_t ws_bytes, hipStream_t s);
// Few token rows (M <= 64, bf16, few_rows.hip): weights and activations in blocks, the step that follows a projection (and
// the RMSNorm in front of it) done by the projection.  a = bf16(h * gain) and ssq [d/16][64] its sums of squares; up to
// eight rows (few_rows_row_major) every activation in rows instead of blocks, and ssq [M][d/16].
bool few_rows_supported(int M, int d, int F, int Hq, int Hkv, int dh);
bool few_rows_row_major(int M);
int64_t few_rows_workspace_bytes(int d, int K_max);
// rope: also fills the rotary table (may be null)
hipError_t launch_few_norm(const void* h, int h_f32, const void* gain, void* a, float* ssq, int M, int d, const RopeJob* rope,
                           hipStream_t s);
hipError_t launch_few_qkv(const void* a, const float* ssq, float eps, const void* W, void* qkv, int64_t ldq, const float2* cs,
                          void* k_rows, void* v_rows, int M, int d, int Hq, int Hkv, int dh, hipStream_t s);
// act [M, N/2] (laid out as a) = silu(gate) * up
hipError_t launch_few_swiglu(const void* a, const float* ssq, float eps, const void* W, void* act, int M, int N, int K,
                             hipStream_t s);
// C (row-major) = x W^T + R; with gain: a and ssq for the next projection
hipError_t launch_few_residual(const void* x, const void* W, const void* R, int r_f32, void* C, int c_f32, const void* gain,
                               void* a, float* ssq, int M, int N, int K, void* ws, int64_t ws_bytes, hipStream_t s);
// expert layers: router on prepared rows, the chosen experts' MLPs (act [E][M up to 16][F] in blocks, y [E][M][d] fp32), their
// gate-weighted sum on the residual stream
hipError_t launch_few_route(const void* a, const float* ssq, float eps, const void* wr, int32_t* experts, float* gates, int n,
                            int d, int E, int top_k, hipStream_t s);
hipError_t launch_few_experts(const void* a, const float* ssq, float eps, const void* wgu, const void* wd, void* act, float* y,
                              const int32_t* experts, int M, int d, int F, int E, int top_k, hipStream_t s);
hipError_t launch_few_combine(const float* y, const int32_t* experts, const float* gates, int top_k, int E, const float* h, void* C,
                              int c_f32, const void* gain, void* a, float* ssq, int M, int d, hipStream_t s);

// x is fp32 when x_f32 is set, else the model dtype; g and y are the model dtype
hipError_t launch_rmsnorm(int dtype, const void* x, int x_f32, const void* g, void* y, int T, int d, float eps, hipStream_t s);
extern thread_local int g_last_hip_error;  // hipError_t of the last failed HIP call on this thread
// Timing of single launches (the "time_gemm" hook): when set, the next tensor-core GEMM or attention launch on this
// thread attaches the two events to its own dispatch (they receive the kernel's start and stop times; no extra
// packets go into the stream) and clears the pair.
extern thread_local hipEvent_t g_launch_ev_start, g_launch_ev_stop;
#define DSK_LAUNCH_TIMED(kern, grid, block, lds, stream, ...)                                                        \
  do {                                                                                                               \
    if (g_launch_ev_start || g_launch_ev_stop) {                                                                     \
      hipExtLaunchKernelGGL(kern, grid, block, lds, stream, g_launch_ev_start, g_launch_ev_stop, 0, __VA_ARGS__);    \
      g_launch_ev_start = g_launch_ev_stop = nullptr;                                                                \
    } else {                                                                                                         \
      hipLaunchKernelGGL(kern, grid, block, lds, stream, __VA_ARGS__);                                               \
    }                                                                                                                \
  } while (0)

// K and V rows of layers first .. first+n-1 (bytes of each) from one device cache into another, one launch (splice.hip)
hipError_t launch_splice(const void* src, int64_t src_stride, int64_t src_v, void* dst, int64_t dst_stride, int64_t dst_v, int first,
                         int n, int64_t bytes, int background, hipStream_t s);
// pacing of the load stream against the 100 MHz constant-rate clock
hipError_t launch_pace_start(unsigned long long* t0, hipStream_t s);
hipError_t launch_pace_wait(const unsigned long long* t0, unsigned long long ticks, hipStream_t s);
hipError_t launch_rope_table(const RopeJob& rope, hipStream_t s);
// RMSNorm of the first layer and the rotary table in one launch, where norm_takes_rope says so (bf16)
bool norm_takes_rope(int dtype, int d);
hipError_t launch_rmsnorm_rope(const void* x, const void* g, void* y, int T, int d, float eps, const RopeJob& rope, hipStream_t s);
// rotates q (in place) and k of qkv [T, n_qkv]; writes rotated k and v to the cache rows row0..row0+T-1
hipError_t launch_rope_kv_write(int dtype, void* qkv, const float2* cs, void* k_rows, void* v_rows, int T, int Hq,
                                int Hkv, int dh, hipStream_t s);
// act[t,f] = silu(gate) * up from the interleaved gate/up GEMM output gu [T, 2F]
hipError_t launch_swiglu(int dtype, const void* gu, void* act, int T, int F, int gu_block, hipStream_t s);

// Causal grouped-query attention over packed sequences.  Query token i of sequence b (rows q_cu[b]..)
// sees cache rows p_cu[b] .. p_cu[b+1]-1 (all of them; p_cu may be NULL: no such segment) and rows
// own_row0 + q_cu[b] .. own_row0 + i.  q rows have stride ldq elements, out rows Hq*dh.
struct AttnArgs {
  const void* q; int64_t ldq;
  const void* k_rows; const void* v_rows;  // layer base of K and V rows (row stride Hkv*dh)
  void* out;
  const int32_t* q_cu; const int32_t* p_cu; const int32_t* q_cu_host; const int32_t* p_cu_host; int n_seqs;
  int64_t own_row0; int n_q; int Hq, Hkv, dh;
  const void* vt; int64_t ldvt;  // transposed V (see launch_transpose_v; not read where attn_few_supported); NULL: not available
  int keep_vt = 0;               // later calls rely on the transposed copy of this call's rows
  int out_blocks = 0;            // out in blocks (block_at, Hq*dh columns) instead of rows
  void* ws; int64_t ws_bytes;    // fp32 scratch for key-split partial results (attn_mfma_workspace_bytes); optional
};
bool attn_fp32_supported(const AttnArgs& a);
hipError_t launch_attn_fp32(const AttnArgs& a, hipStream_t s);
hipError_t launch_attn_generic(int dtype, const AttnArgs& a, hipStream_t s);
hipError_t launch_attn_mfma_bf16(const AttnArgs& a, hipStream_t s);
// Few queries per sequence (attn_few.hip; launch_attn_mfma_bf16 hands such calls over): no transposed V needed.
bool attn_few_supported(const AttnArgs& a);
hipError_t launch_attn_few(const AttnArgs& a, int* splits, hipStream_t s);
// merges key-split partial results [n_q][Hq][splits][dh] / [..][2]
hipError_t launch_attn_combine(const float* part_o, const float* part_ml, void* out, int out_blocks, int n_q, int Hq, int dh,
                               int splits, float c, hipStream_t s);
int64_t attn_mfma_workspace_bytes(int Hq, int dh);
// vt[(c)*ldvt + row] = v_rows[row][c] for valid rows (row < n_pre or own_row0 <= row < own_row0+n_own), 0 otherwise,
// over the whole 64-row tiles from the one that holds first_row up to own_row0+n_own (earlier tiles of vt are left as
// they are); width = Hkv*dh must be a multiple of 64.
hipError_t launch_transpose_v(const void* v_rows, void* vt, int64_t ldvt, int width, int64_t n_pre, int64_t own_row0,
                              int64_t n_own, int64_t first_row, hipStream_t s);
// cu[0..3] = {a, b, c, d} on the device (sequence boundaries of a row chunk, set in stream order)
hipError_t launch_set_int4(int32_t* dst, int a, int b, int c, int d, hipStream_t s);

hipError_t launch_fill_normal(void* dst, int64_t n, uint64_t seed, uint64_t stream_id, float std, float offset,
                              int64_t idx0, int dtype, hipStream_t s);
// weight (re)packing: logical tensor rows <-> packed rows.  map: 0 identity + row_off, 1 gate rows, 2 up rows.
hipError_t launch_pack_rows(int dtype, void* packed, const void* logical, int64_t rows, int64_t cols, int map,
                            int gu_block, int64_t row_off, int blocks, int to_packed, hipStream_t s);
hipError_t launch_fill_weight(int dtype, void* packed, int64_t rows, int64_t cols, int map, int gu_block, int64_t row_off, int blocks,
                              uint64_t seed, uint64_t stream_id, float std, float offset, hipStream_t s);

// mixture-of-experts MLP: router, grouping by expert, grouped projections, gate-weighted sum (moe.hip, gemm_mfma.hip)
hipError_t launch_moe_route(int dtype, const void* xn, const void* wr, int32_t* experts, float* gates, int n, int d, int E,
                            int top_k, hipStream_t s);
// tile_tab: two tables of int4 [tile_rows_max + 1], gate/up's and down's (the last entry of each receives its numbers of tiles)
hipError_t launch_moe_place(const int32_t* experts, int32_t* slot_of, int32_t* src_token, void* tile_tab, int n, int top_k,
                            int E, int tile_m, int down_tiles_n, int tile_rows_max, hipStream_t s);
hipError_t moe_low_tile_count(unsigned long long* count);  // low tiles that calls on this device have written to tables
// Tiles of a scheduling group, at most (a Mixtral layer over 4096, 6000, 8192 tokens, us: four 3055, 4095, 5988; eight 3015, 3987, 5897;
// twelve 3007, 3974, 5915; twenty-four 3004, 3987, 5906: from eight on it does not matter), and the place of their number in the table.
constexpr int MOE_GROUP_MOST = 12, MOE_GROUP_SHIFT = 20;
int moe_tile_rows_for(int64_t n_rows, int E);
// Low tiles: an expert's last rows where they are no more than MOE_LOW_ROWS and its other tiles have MOE_HIGH_ROWS.
constexpr int MOE_HIGH_ROWS = 256, MOE_LOW_ROWS = 128, MOE_LOW_COLS = 128;
// rows of the grouped projections' tile table for n_rows rows over E experts in tiles of tile_m (every expert may end in a
// partial tile)
inline int moe_tile_table_rows(int64_t n_rows, int E, int tile_m) { return (int)((n_rows + tile_m - 1) / tile_m) + E; }
hipError_t launch_moe_combine(const float* y, const float* h_mid, const float* gates, const int32_t* experts,
                              const int32_t* slot_of, void* out, int out_f32, int n, int d, int top_k, int64_t y_rows,
                              hipStream_t s);
hipError_t launch_gemm_mfma_grouped(const void* A, int64_t lda, int64_t a_rows, const int32_t* a_row, const void* W, int64_t ldw,
                                    int w_blocks, int64_t w_group_stride, void* C, int64_t ldc, int N, int K, int epi,
                                    const void* tile_tab, int tile_m, int tile_rows, int low_tiles, int64_t rows_per_expert,
                                    hipStream_t s);

// tuning knobs (dsk_set_option)
void gemm_mfma_set_variant(int v);
int64_t gemm_mfma_direct_launches(int reset);
void attn_mfma_counts(int64_t* split, int64_t* split_64, int64_t* few, int reset);
bool gemm_mfma_uses_prefill_tile(int M, int N);
void gemm_mfma_plan(int M, int N, int K, int may_split, int32_t* plan);  // dsk_gemm_plan
