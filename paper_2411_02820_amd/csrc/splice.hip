// Splice of device-resident layers: K and V rows of a run of layers copied from the sender's cache into the receiver's in
// one launch.  Bound: HBM, every byte read and written once.  Copying layer by layer cost the host about 10 us per copy
// call (48 calls in front of the first kernel of an 8B pass, 4 in front of a 0.2 ms fp32 one) and left the GPU waiting.
#include "dsk_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4;

// blockIdx.y: (layer, K or V) of the run; four 16-byte pieces per thread in flight.  The rows are next read by the suffix
// pass, long after the caches have turned over: they bypass them.
__global__ void __launch_bounds__(256) splice_kernel(const char* __restrict__ src, int64_t src_stride, int64_t src_v,
                                                     char* __restrict__ dst, int64_t dst_stride, int64_t dst_v, int first,
                                                     int64_t pieces) {
  const int l = first + (blockIdx.y >> 1), v = blockIdx.y & 1;
  const i32x4* s = (const i32x4*)(src + l * src_stride + v * src_v);
  i32x4* d = (i32x4*)(dst + l * dst_stride + v * dst_v);
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pieces; i += 4 * step) {
    i32x4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * step < pieces) x[u] = __builtin_nontemporal_load(s + i + u * step);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * step < pieces) __builtin_nontemporal_store(x[u], d + i + u * step);
  }
}

}  // namespace

// Layers first .. first + n - 1, `bytes` (a multiple of 16) of K and of V each; all addresses and strides 16-byte aligned.
// About 2048 workgroups in all, fewer when there is less than 16 KB for each: 32 layers of 8192 8B rows in 489 us, 4.4 TB/s
// (copied layer by layer: 767 us).  Next to a recomputation (`background`) 128: at full rate the copy holds up the kernels it
// runs beside, and it has the recomputation's time to finish.  8192 rows, 32 8B layers of which one is recomputed, both ways
// in turn: 7837 us (quartiles 7828-7857) against 7915 (7905-7928); eight recomputed: 29672 (29633-29701) and 29712
// (29669-29800); over 1024 rows and at the 70B width no difference.
hipError_t launch_splice(const void* src, int64_t src_stride, int64_t src_v, void* dst, int64_t dst_stride, int64_t dst_v, int first,
                         int n, int64_t bytes, int background, hipStream_t s) {
  if (n <= 0 || bytes <= 0) return hipSuccess;
  int64_t gx = ((background ? 128 : 2048) + 2 * n - 1) / (2 * n);
  if (gx > (bytes + 16383) / 16384) gx = (bytes + 16383) / 16384;
  hipLaunchKernelGGL(splice_kernel, dim3((unsigned)gx, 2 * n), dim3(256), 0, s, (const char*)src, src_stride, src_v, (char*)dst,
                     dst_stride, dst_v, first, bytes / 16);
  return hipGetLastError();
}
