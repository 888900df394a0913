// Mixture-of-experts MLP (the Mixtral receiver of Sec. 5.4): router, grouping of the token rows by expert, and the
// gate-weighted sum of the expert outputs.  The expert projections themselves run on the GEMM kernels.
//
// Routing as in Mixtral: router logits = xn * Wr^T in fp32, the top_k experts of a token by logit (equal logits go to
// the lower expert index), gate weights = softmax over the chosen logits.
#include "dsk_internal.h"

namespace {

constexpr int MAX_K = DSK_MOE_MAX_TOP_K;

template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> { typedef __attribute__((ext_vector_type(8))) __bf16 type; };
template <> struct Vec8<float> { typedef __attribute__((ext_vector_type(8))) float type; };

// One wave per token: the E dot products one after the other (the row of xn stays in the cache), each reduced over
// the wave in a fixed order, then the top_k choice and the softmax on values every lane holds.
template <typename T>
__global__ void __launch_bounds__(256) moe_route_kernel(const T* __restrict__ xn, const T* __restrict__ wr,
                                                        int32_t* __restrict__ experts, float* __restrict__ gates, int n,
                                                        int d, int E, int top_k) {
  typedef typename Vec8<T>::type vec8;
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= n) return;
  float best_v[MAX_K];
  int best_e[MAX_K];
#pragma unroll
  for (int j = 0; j < MAX_K; ++j) { best_v[j] = -INFINITY; best_e[j] = -1; }
  const T* x = xn + (int64_t)t * d;
  // the token's row is read once and kept in registers (widths up to 512 * XCH; wider rows are re-read per expert)
  constexpr int XCH = 8;
  const bool in_regs = d <= 512 * XCH;
  vec8 xr[XCH];
  if (in_regs) {
#pragma unroll
    for (int i = 0; i < XCH; ++i) {
      const int c = lane * 8 + 512 * i;
      if (c < d) xr[i] = *(const vec8*)(x + c);
    }
  }
  for (int e = 0; e < E; ++e) {
    const T* w = wr + (int64_t)e * d;
    float acc = 0.f;
    if (in_regs) {
      // same products in the same order as the loop below
      vec8 wv[XCH];
#pragma unroll
      for (int i = 0; i < XCH; ++i) {
        const int c = lane * 8 + 512 * i;
        if (c < d) wv[i] = *(const vec8*)(w + c);
      }
#pragma unroll
      for (int i = 0; i < XCH; ++i) {
        const int c = lane * 8 + 512 * i;
        if (c < d) {
#pragma unroll
          for (int u = 0; u < 8; ++u) acc = fmaf(to_f32(xr[i][u]), to_f32(wv[i][u]), acc);
        }
      }
    } else {
      for (int c = lane * 8; c < d; c += 512) {
        const vec8 a = *(const vec8*)(x + c), b = *(const vec8*)(w + c);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fmaf(to_f32(a[u]), to_f32(b[u]), acc);
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (!(acc == acc)) acc = -3.0e38f;  // a NaN logit ranks last: every list entry below is then a real expert
    // insert into the descending list; strictly greater only, so that an earlier expert keeps its place on a tie
    float v = acc;
    int id = e;
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) {
      if (j < top_k && v > best_v[j]) {
        const float tv = best_v[j];
        const int te = best_e[j];
        best_v[j] = v; best_e[j] = id;
        v = tv; id = te;
      }
    }
  }
  if (lane == 0) {
    float p[MAX_K], sum = 0.f;
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) {
      p[j] = j < top_k ? expf(best_v[j] - best_v[0]) : 0.f;
      sum += p[j];
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int j = 0; j < MAX_K; ++j)
      if (j < top_k) {
        experts[(int64_t)t * top_k + j] = best_e[j];
        gates[(int64_t)t * top_k + j] = p[j] * inv;
      }
  }
}

// The same choice on the matrix cores, for bf16 rows of whole 32-element steps and more than a few tokens: one workgroup per
// 16 tokens, its four waves take every fourth step of the contraction (v_mfma_f32_16x16x32_bf16, fp32 accumulation; experts
// are the MFMA rows in NT blocks of 16), partial logits meet in LDS in wave order.  Bound by reading the rows once (67 MB at
// 8192 x 4096); the kernel above re-reads all router weights per token from the L2s: 41 us there, with this one 19 us.
template <int NT>
__global__ void __launch_bounds__(256) moe_route_mfma_kernel(const bf16_t* __restrict__ xn, const bf16_t* __restrict__ wr,
                                                             int32_t* __restrict__ experts, float* __restrict__ gates, int n, int d,
                                                             int E, int top_k) {
  typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  constexpr int PF = NT <= 2 ? 8 : 4;  // steps in flight
  __shared__ float part[4][16][16 * NT + 1];
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4, wave = tid >> 6;
  const int t0 = blockIdx.x * 16;
  const bf16_t* x = xn + (int64_t)min(t0 + r16, n - 1) * d + 8 * g;
  const bf16_t* w[NT];
  f32x4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    w[j] = wr + (int64_t)min(16 * j + r16, E - 1) * d + 8 * g;
    acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int steps = d / 32;
  for (int s0 = wave; s0 < steps; s0 += 4 * PF) {
    bf16x8 fx[PF], fw[PF][NT];
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (s0 + 4 * u < steps) {
        fx[u] = *(const bf16x8*)(x + (s0 + 4 * u) * 32);
#pragma unroll
        for (int j = 0; j < NT; ++j) fw[u][j] = *(const bf16x8*)(w[j] + (s0 + 4 * u) * 32);
      }
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (s0 + 4 * u < steps)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[u][j], fx[u], acc[j], 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][r16][16 * j + 4 * g + r] = acc[j][r];
  __syncthreads();
  for (int i = tid; i < 16 * E; i += 256) {
    const int t = i / E, e = i - t * E;
    const float v = part[0][t][e] + part[1][t][e] + part[2][t][e] + part[3][t][e];
    part[0][t][e] = v == v ? v : -3.0e38f;  // only this thread reads and writes the entry
  }
  __syncthreads();
  if (tid >= 16 || t0 + tid >= n) return;
  float* logit = part[0][tid];
  const int64_t at = (int64_t)(t0 + tid) * top_k;
  float best[MAX_K], sum = 0.f;
#pragma unroll
  for (int j = 0; j < MAX_K; ++j) {
    if (j >= top_k) break;
    int b = 0;
    for (int e = 1; e < E; ++e)
      if (logit[e] > logit[b]) b = e;  // strictly greater: the lower index keeps a tie
    best[j] = logit[b];
    logit[b] = -INFINITY;
    experts[at + j] = b;
    sum += expf(best[j] - best[0]);
  }
  const float inv = 1.0f / sum;
#pragma unroll
  for (int j = 0; j < MAX_K; ++j) {
    if (j >= top_k) break;
    gates[at + j] = expf(best[j] - best[0]) * inv;
  }
}

// Groups the n*top_k (token, choice) entries by expert, keeping token order inside an expert (so the result does not
// depend on timing).  One workgroup per expert e: it counts the entries of every expert (LDS histogram), derives the
// first slot of its own rows and the first row tile of its own tiles, then walks the entries in order and gives the
// j-th entry of expert e the slot first + j.  slot_of[entry] = slot, src_token[slot] = token.  tile_tab[r], r <
// tile_rows_max: {expert, first slot of the tile, end of the expert's slots, first tile of its scheduling group | tiles of
// that << MOE_GROUP_SHIFT}, the tiles of all experts back to back, behind them low ones,
// expert -1 past the last tile; tile_tab[tile_rows_max] = {number of tiles, number of low ones} (the GEMM spreads exactly those over the
// chip: a grid sized for the worst case would leave the dies that get its empty end idle).  With tiles of MOE_HIGH_ROWS a second
// table behind the first is the down projection's, tiles_n column tiles wide.
//
// Low tiles (128 x 128): down has few column tiles, so an expert's partly filled last tiles decide how many rounds of workgroups it
// takes; balanced experts with whole tiles to the row fill whole rounds, and the few rows that some have beyond them cost one more.
// Where an expert's last rows fit a low tile, and the rounds are fewer so (a low tile taken for half a high one), they run as low
// tiles behind all others.  The rule is on the counts, i.e. on the device.  us, eight experts of the 8B widths, down over 2048, 4096, 6300,
// 8192 tokens: 614 -> 467, 938 -> 812, 1327 -> 1181, 1681 -> 1515; 1100, 2400 and 3200 tokens, where the rounds are as many, keep the
// high ones (low ones as 128 x 256 tiles whatever the rounds: 2400 tokens 635 -> 696).  Half as wide as the others because what a
// low tile takes is its stream of W, and one compute unit draws only so much: 128 x 256 tiles took 526, 862, 1288, 1559.
// Gate/up has seven times the column tiles and streams an expert's W once for all its row tiles: low tiles behind the others stream
// it again (2400 tokens 1069 -> 1077), low tiles in the expert's group 1069 -> 1024 there, but 843 -> 890 over 2048 tokens.
__device__ inline bool moe_low_tiles(int n_plain, int n_high, int n_low, int tiles_n) {
  constexpr int CUS = 256;
  if (n_low == 0) return false;
  const int64_t plain = ((int64_t)n_plain * tiles_n + CUS - 1) / CUS, high = (int64_t)n_high * tiles_n;
  const int64_t rounds = (high + CUS - 1) / CUS, left = (int64_t)n_low * tiles_n - (rounds * CUS - high);  // what the last round has no room for
  return 2 * rounds + (left > 0 ? (2 * left + CUS - 1) / CUS : 0) < 2 * plain;
}
__device__ unsigned long long low_tiles_written;  // by all calls on this device
constexpr int PLACE_T = 1024;  // threads: the walk is a chain of rounds, wider ones make it shorter (256: 23 us at 8192 tokens)
__global__ void __launch_bounds__(PLACE_T) moe_place_kernel(const int32_t* __restrict__ experts, int32_t* __restrict__ slot_of,
                                                        int32_t* __restrict__ src_token, int4* __restrict__ tile_tab,
                                                        int n_entries, int top_k, int E, int tile_m, int tiles_n, int tile_rows_max) {
  __shared__ int hist[DSK_MOE_MAX_EXPERTS];
  __shared__ int wave_cnt[2][4][PLACE_T / 64];
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < DSK_MOE_MAX_EXPERTS) hist[tid] = 0;
  __syncthreads();
  for (int base = tid; base < n_entries; base += 4 * PLACE_T) {
    int x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = base + PLACE_T * q < n_entries ? experts[base + PLACE_T * q] : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((unsigned)x[q] < (unsigned)E) atomicAdd(&hist[x[q]], 1);  // the router only writes experts below E
  }
  __syncthreads();
  // an expert's tiles, and whether its last one may be low
  __shared__ int tiles_of[DSK_MOE_MAX_EXPERTS];
  if (tid < E) {
    const int plain = (hist[tid] + tile_m - 1) / tile_m;
    const bool low = tile_m == MOE_HIGH_ROWS && plain > 0 && hist[tid] - (plain - 1) * tile_m <= MOE_LOW_ROWS;
    tiles_of[tid] = 2 * plain + low;
  }
  __syncthreads();
  // [0]: without low tiles; [1]: with them
  int first = 0, n_high[2] = {0, 0}, high0[2] = {0, 0}, n_low = 0, low0 = 0;
  for (int x = 0; x < E; ++x) {
    const int plain = tiles_of[x] >> 1, low = tiles_of[x] & 1;
    if (x == e) {
      high0[0] = n_high[0];
      high0[1] = n_high[1];
      low0 = n_low;
    }
    if (x < e) first += hist[x];
    n_high[0] += plain;
    n_high[1] += plain - low;
    n_low += low;
  }
  const int mine = hist[e], my_low = tiles_of[e] & 1, my_high[2] = {tiles_of[e] >> 1, (tiles_of[e] >> 1) - my_low};
  // One table: the expert's `high` tiles from entry at0 on, and its low one at low_at (< 0: none); n_at, n_behind: all experts' tiles of
  // either kind.  Scheduling groups: an expert's tiles in as few as the most allows, the first ones longer by a tile where they are
  // not equal.
  auto write_table = [&](int4* tab, int at0, int high, int low_at, int n_at, int n_behind) {
    const int n_groups = max((high + MOE_GROUP_MOST - 1) / MOE_GROUP_MOST, 1), least = high / n_groups;
    const int longer = (high - n_groups * least) * (least + 1);  // tiles of the longer ones
    for (int r = tid; r < high; r += PLACE_T) {
      const int size = r < longer ? least + 1 : least, from = r < longer ? 0 : longer, g0 = from + (r - from) / size * size;
      if (at0 + r < tile_rows_max) tab[at0 + r] = make_int4(e, first + r * tile_m, first + mine, (at0 + g0) | size << MOE_GROUP_SHIFT);
    }
    if (tid == 0 && low_at >= 0 && low_at < tile_rows_max) tab[low_at] = make_int4(e, first + high * tile_m, first + mine, 0);
    if (e == E - 1) {
      for (int r = n_at + n_behind + tid; r < tile_rows_max; r += PLACE_T) tab[r] = make_int4(-1, 0, 0, 0);
      if (tid == 0) tab[tile_rows_max] = make_int4(min(n_at, tile_rows_max), min(n_behind, max(tile_rows_max - n_at, 0)), 0, 0);
    }
  };
  write_table(tile_tab, high0[0], my_high[0], -1, n_high[0], 0);
  if (tile_m == MOE_HIGH_ROWS) {
    const bool low = moe_low_tiles(n_high[0], n_high[1], n_low, tiles_n);
    write_table(tile_tab + tile_rows_max + 1, high0[low], my_high[low], low && my_low ? n_high[1] + low0 : -1, n_high[low], low ? n_low : 0);
    if (low && e == E - 1 && tid == 0) atomicAdd(&low_tiles_written, (unsigned long long)n_low);
  }
  // rounds of 4 * PLACE_T entries, four groups of PLACE_T in entry order; a thread's four entries are requested together (the
  // walk is a chain of short rounds: what it takes is the round trips to memory)
  int running = 0;
  int buf = 0;
  for (int base = 0; base < n_entries; base += 4 * PLACE_T, buf ^= 1) {
    int ex[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = base + PLACE_T * q + tid;
      ex[q] = i < n_entries ? experts[i] : -1;
    }
    unsigned long long mask[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mask[q] = __ballot(ex[q] == e);
      if (lane == 0) wave_cnt[buf][q][wave] = __popcll(mask[q]);
    }
    __syncthreads();  // the other buffer is written in the next round, after every wave has passed this barrier
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int before = __popcll(mask[q] & ((1ull << lane) - 1ull));
      int total = 0;
#pragma unroll
      for (int w = 0; w < PLACE_T / 64; ++w) {
        const int c = wave_cnt[buf][q][w];
        if (w < wave) before += c;
        total += c;
      }
      if (ex[q] == e) {
        const int i = base + PLACE_T * q + tid;
        const int slot = first + running + before;
        slot_of[i] = slot;
        src_token[slot] = i / top_k;
      }
      running += total;
    }
  }
}

// out[t][:] = h_mid[t][:] + sum_j gates[t][j] * y[row(t, j)][:], j in the order of the router's list (highest logit
// first).  row(t, j) = slot_of[t*top_k + j] when the rows are grouped by expert, experts[t*top_k + j] * n + t when
// every expert ran over all n rows.  y and h_mid are fp32; out is fp32 or the model dtype.
template <typename TO>
__global__ void __launch_bounds__(256) moe_combine_kernel(const float* __restrict__ y, const float* __restrict__ h_mid,
                                                          const float* __restrict__ gates,
                                                          const int32_t* __restrict__ experts,
                                                          const int32_t* __restrict__ slot_of, TO* __restrict__ out, int n,
                                                          int d, int top_k, int64_t y_rows) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const int quads = d / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)n * quads) return;
  const int t = (int)(i / quads), c = (int)(i - (int64_t)t * quads) * 4;
  f32x4 acc = *(const f32x4*)(h_mid + (int64_t)t * d + c);
  for (int j = 0; j < top_k; ++j) {
    int64_t row = slot_of ? (int64_t)slot_of[(int64_t)t * top_k + j] : (int64_t)experts[(int64_t)t * top_k + j] * n + t;
    row = row < 0 ? 0 : (row >= y_rows ? y_rows - 1 : row);  // always inside y, whatever the tables hold
    const float g = gates[(int64_t)t * top_k + j];
    const f32x4 v = *(const f32x4*)(y + row * d + c);
    acc[0] = fmaf(g, v[0], acc[0]); acc[1] = fmaf(g, v[1], acc[1]);
    acc[2] = fmaf(g, v[2], acc[2]); acc[3] = fmaf(g, v[3], acc[3]);
  }
  TO* o = out + (int64_t)t * d + c;
#pragma unroll
  for (int u = 0; u < 4; ++u) o[u] = from_f32<TO>(acc[u]);
}

}  // namespace

hipError_t launch_moe_route(int dtype, const void* xn, const void* wr, int32_t* experts, float* gates, int n, int d, int E,
                            int top_k, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (E < 1 || E > DSK_MOE_MAX_EXPERTS || top_k < 1 || top_k > MAX_K || top_k > E || d % 8) return hipErrorNotSupported;
  const dim3 grid((unsigned)((n + 3) / 4));
  if (dtype == DSK_BF16 && d % 32 == 0 && n > 64) {
    auto kern = E <= 16 ? moe_route_mfma_kernel<1> : E <= 32 ? moe_route_mfma_kernel<2> : moe_route_mfma_kernel<4>;
    hipLaunchKernelGGL(kern, dim3((n + 15) / 16), dim3(256), 0, s, (const bf16_t*)xn, (const bf16_t*)wr, experts, gates, n, d, E, top_k);
  } else if (dtype == DSK_BF16)
    hipLaunchKernelGGL(moe_route_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)xn, (const bf16_t*)wr, experts, gates,
                       n, d, E, top_k);
  else
    hipLaunchKernelGGL(moe_route_kernel<float>, grid, dim3(256), 0, s, (const float*)xn, (const float*)wr, experts, gates, n,
                       d, E, top_k);
  return hipGetLastError();
}

hipError_t moe_low_tile_count(unsigned long long* count) { return hipMemcpyFromSymbol(count, HIP_SYMBOL(low_tiles_written), sizeof *count); }

hipError_t launch_moe_place(const int32_t* experts, int32_t* slot_of, int32_t* src_token, void* tile_tab, int n, int top_k,
                            int E, int tile_m, int tiles_n, int tile_rows_max, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(moe_place_kernel, dim3(E), dim3(PLACE_T), 0, s, experts, slot_of, src_token, (int4*)tile_tab, n * top_k,
                     top_k, E, tile_m, tiles_n, tile_rows_max);
  return hipGetLastError();
}

hipError_t launch_moe_combine(const float* y, const float* h_mid, const float* gates, const int32_t* experts,
                              const int32_t* slot_of, void* out, int out_f32, int n, int d, int top_k, int64_t y_rows,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t units = (int64_t)n * (d / 4);
  const dim3 grid((unsigned)((units + 255) / 256));
  if (out_f32)
    hipLaunchKernelGGL(moe_combine_kernel<float>, grid, dim3(256), 0, s, y, h_mid, gates, experts, slot_of, (float*)out, n, d,
                       top_k, y_rows);
  else
    hipLaunchKernelGGL(moe_combine_kernel<bf16_t>, grid, dim3(256), 0, s, y, h_mid, gates, experts, slot_of, (bf16_t*)out, n,
                       d, top_k, y_rows);
  return hipGetLastError();
}
