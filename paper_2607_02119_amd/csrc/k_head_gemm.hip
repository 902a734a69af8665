// K1 dispatch, and the fp32 path: codebook-head projection with the CFG merge
// and temperature fused into the epilogue, and the text-head projection with a
// fused (max, lowest argmax) epilogue.
//
//   logits[g][n] = sum_h hidden[row(g)][h] * W[n][h]         (Sec. 2.1, n = k*V + v)
//   pair p (GEMM rows 2p, 2p+1 = Main, Companion):
//     scores[p][n] = (w * l_main + (1 - w) * l_comp) / T    (Eq. 1, Sec. 2.4)
//   solo row j:  scores[n_pairs + j][n] = l / T;  T = 0 (greedy): no division
//   text rows:   per row and 32-column part, the largest logit and its lowest id.
//
// bf16 heads run on the streaming kernel (k_stream.hip) up to 128 GEMM rows;
// above, audio rows there too or in 256 x 256 tiles, whichever costs less, and
// text rows in 256 x 128 tiles (k_mfma.hip).  fp32 heads (true fp32 products)
// run on the fp32 matrix instruction here.
#include "gemm_common.h"

namespace mcd {
namespace {

// fp32 path: true fp32 products on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: lane l holds row or column l % 16 at k = l / 16).
//
// A workgroup owns 16 MB rows and 16 NB columns; its four waves take the k16
// groups of H in turn and their sums meet in LDS.  A lane loads 16 bytes, four
// consecutive k of its row or column, so one load feeds four MFMAs (their k
// order is permuted alike on both sides) and a load instruction reads whole
// 64-byte segments; loads of four groups are in flight together, the first
// weights before the plan is read.  Small heads (4 rows, 4096 columns, H 256)
// are bound by that chain of latencies: this form takes it from 46 us (one
// thread per column, walking its weight row in 4-byte loads) to 4.1 us.
//
// Rows and columns past the end repeat the last one and are not stored.  H
// need not be a multiple of 16 or 4 and the buffers only need 4-byte
// alignment: the last group is read element by element.
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kF32Groups = 4;              // k16 groups in flight per wave
constexpr int kF32Waves = 4;

template <int MB, int NB, bool TEXT>
__global__ __launch_bounds__(256) void head_gemm_f32(HeadView hv, StepView sv) {
  constexpr int U = kF32Groups, BM = 16 * MB, BN = 16 * NB, CP = BN + 1;
  __shared__ float part[kF32Waves][BM][CP];
  __shared__ float4 rowp[BM / 2];
  const int32_t *rows = sv.plan + kPlanHeader + (TEXT ? sv.Mg : 0);
  const int M = TEXT ? sv.n_text : sv.Mg;
  const int N = TEXT ? hv.V_text : hv.N;
  const float *Wp = static_cast<const float *>(TEXT ? hv.W_text : hv.W);
  const float *X = static_cast<const float *>(sv.hidden);
  const int H = hv.H;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM;
  const int c = lane & 15, kq = 4 * (lane >> 4);
  const int G = H / 16;                    // whole k16 groups

  const float *wp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) wp[j] = Wp + (size_t)min(n0 + 16 * j + c, N - 1) * H + kq;
  floatx4 wv[U][NB];
  auto load_w = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u * kF32Waves;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        wv[u][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (g < G) wv[u][j] = *reinterpret_cast<const float4_a4 *>(wp[j] + 16 * g);
      }
    }
  };
  load_w(wave);

  if (!plan_ok(sv)) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0)
      atomicOr(sv.status, (uint32_t)MCD_DEV_BAD_PLAN);
    return;
  }
  const float *xp[MB];
  float xs[MB];                            // 0 for a row outside the batch
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int r = rows[min(m0 + 16 * i + c, M - 1)];
    const bool ok = r >= 0 && r < sv.R;
    if (!ok) atomicOr(sv.status, (uint32_t)MCD_DEV_BAD_PLAN);
    xp[i] = X + (size_t)(ok ? r : 0) * H + kq;
    xs[i] = ok ? 1.0f : 0.0f;
  }
  if constexpr (!TEXT) {
    if (tid < BM / 2) rowp[tid] = pair_params(sv, rows, m0 + 2 * tid);
  }

  floatx4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  auto multiply = [&](const floatx4 (&a)[MB], const floatx4 (&b)[NB]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
  };
  for (int g0 = wave; g0 < G; g0 += U * kF32Waves) {
    floatx4 xv[U][MB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u * kF32Waves;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        xv[u][i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (g < G && xs[i] != 0.0f) xv[u][i] = *reinterpret_cast<const float4_a4 *>(xp[i] + 16 * g);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) multiply(xv[u], wv[u]);
    load_w(g0 + U * kF32Waves);
  }
  if (16 * G < H && wave == G % kF32Waves) {   // the last, partial group
    floatx4 a[MB], b[NB];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = 16 * G + kq + e < H;
#pragma unroll
      for (int i = 0; i < MB; ++i) a[i][e] = (in && xs[i] != 0.0f) ? xp[i][16 * G + e] : 0.0f;
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j][e] = in ? wp[j][16 * G + e] : 0.0f;
    }
    multiply(a, b);
  }
  // lane l holds rows 4 (l / 16) .. + 3 of column l % 16 of every block
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * i + kq + r][16 * j + c] = acc[i][j][r];
  __syncthreads();
  auto sum = [&](int row, int col) __attribute__((always_inline)) {
    float v = part[0][row][col];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) v += part[w][row][col];
    return v;
  };
  if constexpr (!TEXT) {
    for (int item = tid; item < BM / 2 * BN; item += 256) {
      const int q = item / BN, col = item % BN, n = n0 + col;
      if (n >= N || m0 + 2 * q >= M) continue;
      const float b = hv.bias ? hv.bias[n] : 0.0f;
      const float v0 = sum(2 * q, col) + b, v1 = sum(2 * q + 1, col) + b;
      const float4 pr = rowp[q];
      const int o0 = __float_as_int(pr.z), o1 = __float_as_int(pr.w);
      if (o1 == -2) {
        sv.scores[(size_t)o0 * N + n] = fmaf(pr.x, v0, (1.0f - pr.x) * v1) * pr.y;
      } else {
        if (o0 >= 0) sv.scores[(size_t)o0 * N + n] = v0 * pr.x;
        if (o1 >= 0) sv.scores[(size_t)o1 * N + n] = v1 * pr.y;
      }
    }
  } else {
    static_assert(BN == kTextPartCols, "one text part per workgroup and row");
    for (int item = tid; item < BM * BN; item += 256) {   // 32 lanes per row
      const int row = item / BN, col = item % BN, n = n0 + col, g = m0 + row;
      float bv = -INFINITY;
      int bi = INT32_MAX;
      if (n < N) {
        bv = sum(row, col);
        bi = n;
      }
      for (int off = 1; off < 32; off <<= 1) {
        const float ov = __shfl_xor(bv, off);
        const int oi = __shfl_xor(bi, off);
        better(bv, bi, ov, oi);
      }
      if (col == 0 && g < M) {
        sv.text_val[(size_t)g * sv.text_parts + blockIdx.x] = bv;
        sv.text_idx[(size_t)g * sv.text_parts + blockIdx.x] = bi;
      }
    }
  }
}

// 16 columns per workgroup (a text part, 32, for the text head); as few row
// blocks as hold the rows, up to 64 rows, and row tiles beyond.
template <bool TEXT>
hipError_t launch_f32(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  constexpr int NB = TEXT ? 2 : 1;
  const unsigned tn = (unsigned)((N + 16 * NB - 1) / (16 * NB));
  if (M <= 16)
    hipLaunchKernelGGL((head_gemm_f32<1, NB, TEXT>), dim3(tn), dim3(256), 0, st, hv, sv);
  else if (M <= 32)
    hipLaunchKernelGGL((head_gemm_f32<2, NB, TEXT>), dim3(tn), dim3(256), 0, st, hv, sv);
  else
    hipLaunchKernelGGL((head_gemm_f32<4, NB, TEXT>), dim3(tn, (unsigned)((M + 63) / 64)),
                       dim3(256), 0, st, hv, sv);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_head_gemm_part(const HeadView &hv, const StepView &sv, bool text,
                                 hipStream_t st) {
  const int M = text ? sv.n_text : sv.Mg;
  if (M == 0) return hipSuccess;
  if (hv.dtype == MCD_F32) {
    return text ? launch_f32<true>(hv, sv, M, hv.V_text, st)
                : launch_f32<false>(hv, sv, M, hv.N, st);
  }
  return M <= 128 ? launch_stream_gemm(hv, sv, text, st) : launch_mfma_gemm(hv, sv, text, st);
}

hipError_t launch_head_gemm(const HeadView &hv, const StepView &sv, hipStream_t st) {
  hipError_t e = launch_head_gemm_part(hv, sv, false, st);
  if (e == hipSuccess) e = launch_head_gemm_part(hv, sv, true, st);
  return e;
}

}  // namespace mcd
