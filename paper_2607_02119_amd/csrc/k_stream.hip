// K1, weight-streaming path (text batches of at most 128 rows, and audio
// batches of any number of rows where 256 x 256 tiles would take longer):
// codebook-head projection
// with the CFG merge and temperature fused into the epilogue, or the text-head
// projection with a fused (max, lowest argmax) epilogue.
//
//   logits[g][n] = sum_h hidden[row(g)][h] * W[n][h]         (Sec. 2.1, n = k*V + v)
//   pair p (GEMM rows 2p, 2p+1 = Main, Companion):
//     scores[p][n] = (w * l_main + (1 - w) * l_comp) / T    (Eq. 1, Sec. 2.4)
//   solo row j:  scores[n_pairs + j][n] = l / T;  T = 0 (greedy): no division
//   text rows:   per row and 32-column part, the largest logit and its lowest id.
#include "pc_tile.h"

namespace mcd {
namespace {

template <int BM, int BN, bool TEXT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4))) void head_gemm_pc(
    HeadView hv, StepView sv) {
  __shared__ __attribute__((aligned(1024))) char lds[PcShape<BM, BN>::kLds];
  pc_tile<BM, BN, TEXT>(hv, sv, blockIdx.x, lds);
}

template <int BM, int BN, bool TEXT>
hipError_t launch_pc(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  hipLaunchKernelGGL((head_gemm_pc<BM, BN, TEXT>), dim3(tm * tn), dim3(512), 0, st, hv, sv);
  return hipGetLastError();
}

// Up to 32 rows the hidden states are few and the weights' HBM reads bound the
// tile: 64-column tiles when 128-column ones would leave compute units idle,
// else 128-column ones.
template <bool TEXT>
hipError_t launch_few_rows(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  if ((N + 127) / 128 < 256) return launch_pc<32, 64, TEXT>(hv, sv, M, N, st);
  return launch_pc<32, wide_columns(32), TEXT>(hv, sv, M, N, st);
}

// More rows: a tile takes in (BM + BN) x H x 2 bytes, and that rate bounds it,
// so a launch takes about rounds of 256 compute units x (BM + BN).  The shape
// with the least of that; the larger of equals (fewer re-reads).  Measured (H
// 4096, us, 32 x 64 / 64 x 64 / 64 x 96 / 128 x 64 tiles, the choice marked):
// 128 rows of 2048 columns 18.0* / 21.6 / 27.1 / 29.1; of 8192 32.7 / 26.7* /
// 29.0 / 32.1; of 12288 44.8 / 44.8 / 29.5* / 33.7; of 16384 61.5 / 49.9 / 56.0
// / 38.8*; of 32768 54 with 128 x 128; 512 rows of 16384 70 with 128 x 256.
struct TileShape {
  int bm, bn;
};
constexpr TileShape kShapes[] = {{128, 256}, {128, 128}, {128, 64}, {64, 256},
                                 {64, 128},  {64, 96},   {64, 64},  {32, 64}};

int64_t cost_of(const TileShape &t, int M, int N) {
  const int64_t tiles = (int64_t)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  return (tiles + 255) / 256 * (t.bm + t.bn);
}

int best_shape(int M, int N) {
  int best = -1;
  for (int i = 0; i < (int)(sizeof kShapes / sizeof kShapes[0]); ++i) {
    if (M <= 64 && kShapes[i].bm > 64) continue;   // rows of padding
    if (best < 0 || cost_of(kShapes[i], M, N) < cost_of(kShapes[best], M, N)) best = i;
  }
  return best;
}

template <bool TEXT>
hipError_t launch_tiles(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  if (M <= 32) return launch_few_rows<TEXT>(hv, sv, M, N, st);
  switch (best_shape(M, N)) {
    case 0: return launch_pc<128, 256, TEXT>(hv, sv, M, N, st);
    case 1: return launch_pc<128, 128, TEXT>(hv, sv, M, N, st);
    case 2: return launch_pc<128, 64, TEXT>(hv, sv, M, N, st);
    case 3: return launch_pc<64, 256, TEXT>(hv, sv, M, N, st);
    case 4: return launch_pc<64, 128, TEXT>(hv, sv, M, N, st);
    case 5: return launch_pc<64, 96, TEXT>(hv, sv, M, N, st);
    case 6: return launch_pc<64, 64, TEXT>(hv, sv, M, N, st);
    default: return launch_pc<32, 64, TEXT>(hv, sv, M, N, st);
  }
}

}  // namespace

int64_t stream_cost(int32_t M, int32_t N) { return cost_of(kShapes[best_shape(M, N)], M, N); }

hipError_t launch_stream_gemm(const HeadView &hv, const StepView &sv, bool text,
                              hipStream_t st) {
  return text ? launch_tiles<true>(hv, sv, sv.n_text, hv.V_text, st)
              : launch_tiles<false>(hv, sv, sv.Mg, hv.N, st);
}

}  // namespace mcd
