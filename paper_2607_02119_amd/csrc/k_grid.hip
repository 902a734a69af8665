// K3: delay-pattern de-interleave / interleave between a per-request stream
// buffer [T][K] (token of codebook k emitted at step t) and the frame grid
// [K][F] (Sec. 2.1: stream k is offset by d_k steps, so frame f of codebook k
// was emitted at step f + d_k).
//
// A thread owns one frame (de-interleave) or one step (interleave) of a request
// and walks its K codebooks, eight loads in flight: no index division, the grid
// side contiguous over the lanes, the stream side in whole lines (a lane's K
// tokens are neighbours).  Bound by the launch and one memory round trip:
// 64 requests of 1500 steps x 8 (6 MB moved) took 6.9 and 5.4 us with one
// thread per token, which divided 64-bit indices three times.  Requests
// shorter than a wave keep one thread per token.
#include "mcd_internal.h"

namespace mcd {
namespace {

constexpr int kWalk = 8;                   // codebooks in flight per thread
constexpr int kShort = 64;                 // frames or steps below which a thread has one token

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

// One thread per frame or step: blocks of 64 threads while the batch is small,
// so that it spreads over the compute units.
struct RowGrid {
  dim3 grid, block;
  RowGrid(int32_t len, int32_t n_req) {
    const unsigned nt = (int64_t)len * n_req >= 256 * 512 ? 256u : 64u;
    block = dim3(nt);
    grid = dim3(((unsigned)len + nt - 1) / nt, (unsigned)(n_req < 32768 ? n_req : 32768));
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
  if (F >= kShort) {
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
  if (T >= kShort) {
    const RowGrid g(T, n_req);
    if (K % 4 == 0 && reinterpret_cast<uintptr_t>(streams) % 16 == 0)
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
