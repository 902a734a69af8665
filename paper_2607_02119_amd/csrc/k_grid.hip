// K3: delay-pattern de-interleave / interleave between a per-request stream
// buffer [T][K] (token of codebook k emitted at step t) and the frame grid
// [K][F] (Sec. 2.1: stream k is offset by d_k steps, so frame f of codebook k
// was emitted at step f + d_k).
//
// Two forms.  A thread per token divides 64-bit indices three times, but a small
// batch fills more of the chip with it.  A thread per frame (de-interleave) or
// step (interleave) walks its K codebooks, eight loads in flight: no division,
// the grid side contiguous over the lanes, the stream side in whole lines (a
// lane's K tokens are neighbours).  Small batches are bound by the launch and one
// memory round trip, and a thread with K tokens makes K / 8 of them.
#include "mcd_internal.h"

namespace mcd {
namespace {

constexpr int kWalk = 8;                   // codebooks in flight per thread

// The row form's range, token form / row form in us (de-interleave of n requests
// x F frames x K): at least a wave per request; from five codebooks on 32768
// rows (8 x 300 x 32 2.8 / 4.7, 64 x 300 x 16 3.3 / 3.6, 64 x 700 x 16 4.4 / 4.1,
// 256 x 700 x 16 14.0 / 8.6); three and four always (64 x 64 x 4 2.5 / 2.4, 2000 x
// 1500 x 3 27.4 / 20.1); one and two in small batches only (64 x 64 x 1 2.42 /
// 2.30, 2000 x 300 x 1 3.8 / 6.4, 2000 x 300 x 2 5.6 / 6.9).
bool by_rows(int64_t n_req, int64_t len, int32_t K) {
  if (len < 64) return false;
  if (K <= 2) return n_req * len < 65536;
  return K <= 4 || n_req * len >= 32768;
}

// Interleave: two codebooks from 2^20 rows on too (2000 x 700 9.9 / 9.0, 2000 x
// 300 5.6 / 6.7), and more than eight only with 16-byte stores (2000 x 1500 x 9
// 74.2 / 76.4, 64 x 1500 x 9 4.6 / 5.4, x 12 5.4 / 4.2).
bool by_rows_interleave(int64_t n_req, int64_t len, int32_t K, bool vec) {
  if (K == 2 && len >= 64 && n_req * len >= 1 << 20) return true;
  return by_rows(n_req, len, K) && (vec || K <= 8);
}

__global__ __launch_bounds__(256) void deinterleave_rows(const int32_t *__restrict__ streams,
                                                         int32_t n_req, int32_t T, int32_t K,
                                                         Delays d, int32_t F,
                                                         int32_t *__restrict__ grid) {
  const int32_t f = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (f >= F) return;
  for (int32_t r = blockIdx.y; r < n_req; r += gridDim.y) {
    const int32_t *src = streams + (size_t)r * T * K + (size_t)f * K;
    int32_t *dst = grid + (size_t)r * K * F + f;
    for (int k0 = 0; k0 < K; k0 += kWalk) {
      int32_t v[kWalk];
#pragma unroll
      for (int j = 0; j < kWalk; ++j)
        if (k0 + j < K) v[j] = src[(size_t)d.d[k0 + j] * K + k0 + j];
#pragma unroll
      for (int j = 0; j < kWalk; ++j)
        if (k0 + j < K) dst[(size_t)(k0 + j) * F] = v[j];
    }
  }
}

// VEC: K is a multiple of four and the streams are 16-byte aligned
template <bool VEC>
__global__ __launch_bounds__(256) void interleave_rows(const int32_t *__restrict__ grid,
                                                       int32_t n_req, int32_t F, int32_t K,
                                                       Delays d, int32_t T, int32_t pad_id,
                                                       int32_t *__restrict__ streams) {
  const int32_t t = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (t >= T) return;
  for (int32_t r = blockIdx.y; r < n_req; r += gridDim.y) {
    const int32_t *src = grid + (size_t)r * K * F;
    int32_t *dst = streams + ((size_t)r * T + t) * K;
    for (int k0 = 0; k0 < K; k0 += kWalk) {
      int32_t v[kWalk];
#pragma unroll
      for (int j = 0; j < kWalk; ++j) {
        v[j] = pad_id;
        if (k0 + j < K) {
          const int32_t f = t - d.d[k0 + j];
          if (f >= 0 && f < F) v[j] = src[(size_t)(k0 + j) * F + f];
        }
      }
      if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < kWalk; j += 4)
          if (k0 + j < K)
            *reinterpret_cast<int4 *>(dst + k0 + j) = make_int4(v[j], v[j + 1], v[j + 2], v[j + 3]);
      } else {
#pragma unroll
        for (int j = 0; j < kWalk; ++j)
          if (k0 + j < K) dst[k0 + j] = v[j];
      }
    }
  }
}

__global__ __launch_bounds__(256) void deinterleave_kernel(const int32_t *__restrict__ streams,
                                                           int32_t n_req, int32_t T, int32_t K,
                                                           Delays d, int32_t F,
                                                           int32_t *__restrict__ grid) {
  const size_t total = (size_t)n_req * K * F;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const int32_t f = (int32_t)(i % F);
    const int32_t k = (int32_t)((i / F) % K);
    const size_t r = i / ((size_t)F * K);
    grid[i] = streams[(r * T + (size_t)(f + d.d[k])) * K + k];
  }
}

__global__ __launch_bounds__(256) void interleave_kernel(const int32_t *__restrict__ grid,
                                                         int32_t n_req, int32_t F, int32_t K,
                                                         Delays d, int32_t T, int32_t pad_id,
                                                         int32_t *__restrict__ streams) {
  const size_t total = (size_t)n_req * T * K;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const int32_t k = (int32_t)(i % K);
    const int32_t t = (int32_t)((i / K) % T);
    const size_t r = i / ((size_t)K * T);
    const int32_t f = t - d.d[k];
    streams[i] = (f >= 0 && f < F) ? grid[(r * K + k) * F + f] : pad_id;
  }
}

// One thread per frame or step, in blocks of whole waves: one per request up to
// 256; then of 64 while the batch is small, so that it spreads over the compute
// units (64 x 1500 x 8, de-interleave: 4.0 us, with blocks of 256 4.3); else as
// few as 256 threads allow, of equal size (2000 x 300 x 8: 19.1 us with 44 frames
// in the second block, 13.1 with blocks of 64).
struct RowGrid {
  dim3 grid, block;
  RowGrid(int32_t len, int32_t n_req) {
    const unsigned l = (unsigned)len, blocks = (l + 255) / 256;
    const bool small = l > 256 && (int64_t)len * n_req < 131072;
    const unsigned nt = small ? 64 : ((l + blocks - 1) / blocks + 63) / 64 * 64;
    block = dim3(nt);
    grid = dim3((l + nt - 1) / nt, (unsigned)(n_req < 32768 ? n_req : 32768));
  }
};

unsigned blocks_for(size_t total) {
  size_t b = (total + 255) / 256;
  if (b > 65536) b = 65536;
  return (unsigned)(b ? b : 1);
}

}  // namespace

hipError_t launch_deinterleave(const int32_t *streams, int32_t n_req, int32_t T, int32_t K,
                               const Delays &d, int32_t F, int32_t *grid, hipStream_t st) {
  const size_t total = (size_t)n_req * K * F;
  if (total == 0) return hipSuccess;
  if (by_rows(n_req, F, K)) {
    const RowGrid g(F, n_req);
    hipLaunchKernelGGL(deinterleave_rows, g.grid, g.block, 0, st, streams, n_req, T, K, d, F, grid);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(deinterleave_kernel, dim3(blocks_for(total)), dim3(256), 0, st, streams,
                     n_req, T, K, d, F, grid);
  return hipGetLastError();
}

hipError_t launch_interleave(const int32_t *grid, int32_t n_req, int32_t F, int32_t K,
                             const Delays &d, int32_t T, int32_t pad_id, int32_t *streams,
                             hipStream_t st) {
  const size_t total = (size_t)n_req * T * K;
  if (total == 0) return hipSuccess;
  const bool vec = K % 4 == 0 && reinterpret_cast<uintptr_t>(streams) % 16 == 0;
  if (by_rows_interleave(n_req, T, K, vec)) {
    const RowGrid g(T, n_req);
    if (vec)
      hipLaunchKernelGGL(interleave_rows<true>, g.grid, g.block, 0, st, grid, n_req, F, K, d, T,
                         pad_id, streams);
    else
      hipLaunchKernelGGL(interleave_rows<false>, g.grid, g.block, 0, st, grid, n_req, F, K, d, T,
                         pad_id, streams);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(interleave_kernel, dim3(blocks_for(total)), dim3(256), 0, st, grid, n_req,
                     F, K, d, T, pad_id, streams);
  return hipGetLastError();
}

}  // namespace mcd
