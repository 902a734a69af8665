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
  pc_tile<BM, BN, TEXT, true>(hv, sv, blockIdx.x, lds);
}

template <int BM, int BN, bool TEXT>
hipError_t launch_pc(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  hipLaunchKernelGGL((head_gemm_pc<BM, BN, TEXT>), dim3(tm * tn), dim3(512), 0, st, hv, sv);
  return hipGetLastError();
}

template <int BM, int BN>
constexpr StreamTile tile_of() {
  return StreamTile{BM, BN, PcShape<BM, BN>::SW};
}

// More than 32 rows: a tile takes in (BM + BN) x H x 2 bytes, and that rate bounds it,
// so a launch takes about rounds of 256 compute units x (BM + BN).  The shape
// with the least of that; the larger of equals (fewer re-reads).  Measured (H
// 4096, us, 32 x 64 / 64 x 64 / 64 x 96 / 128 x 64 tiles, the choice marked):
// 128 rows of 2048 columns 18.0* / 21.6 / 27.1 / 29.1; of 8192 32.7 / 26.7* /
// 29.0 / 32.1; of 12288 44.8 / 44.8 / 29.5* / 33.7; of 16384 61.5 / 49.9 / 56.0
// / 38.8*; of 32768 54 with 128 x 128; 512 rows of 16384 70 with 128 x 256.
constexpr StreamTile kShapes[] = {tile_of<128, 256>(), tile_of<128, 128>(), tile_of<128, 64>(),
                                  tile_of<64, 256>(),  tile_of<64, 128>(),  tile_of<64, 96>(),
                                  tile_of<64, 64>(),   tile_of<32, 64>()};

int64_t cost_of(const StreamTile &t, int M, int N) {
  const int64_t tiles = (int64_t)((M + t.rows - 1) / t.rows) * ((N + t.cols - 1) / t.cols);
  return (tiles + 255) / 256 * (t.rows + t.cols);
}

const StreamTile &best_shape(int M, int N) {
  const StreamTile *best = nullptr;
  for (const StreamTile &t : kShapes) {
    if (M <= 64 && t.rows > 64) continue;   // rows of padding
    if (!best || cost_of(t, M, N) < cost_of(*best, M, N)) best = &t;
  }
  return *best;
}

template <bool TEXT>
hipError_t launch_tiles(const HeadView &hv, const StepView &sv, int M, int N, hipStream_t st) {
  const StreamTile t = stream_tile(M, N, TEXT && sv.Mg > 0);
  if constexpr (TEXT)
    if (t.rows == 32 && t.cols == 256) return launch_pc<32, 256, TEXT>(hv, sv, M, N, st);
  switch (t.rows * 1000 + t.cols) {
    case 128256: return launch_pc<128, 256, TEXT>(hv, sv, M, N, st);
    case 128128: return launch_pc<128, 128, TEXT>(hv, sv, M, N, st);
    case 128064: return launch_pc<128, 64, TEXT>(hv, sv, M, N, st);
    case 64256: return launch_pc<64, 256, TEXT>(hv, sv, M, N, st);
    case 64128: return launch_pc<64, 128, TEXT>(hv, sv, M, N, st);
    case 64096: return launch_pc<64, 96, TEXT>(hv, sv, M, N, st);
    case 64064: return launch_pc<64, 64, TEXT>(hv, sv, M, N, st);
    case 32128: return launch_pc<32, 128, TEXT>(hv, sv, M, N, st);
    default: return launch_pc<32, 64, TEXT>(hv, sv, M, N, st);
  }
}

}  // namespace

int64_t stream_cost(int32_t M, int32_t N) { return cost_of(best_shape(M, N), M, N); }

// Up to 32 rows the hidden states are few and the weights' HBM reads bound the
// tile: 64-column tiles when 128-column ones would leave compute units idle,
// else 128-column ones.  Beside audio tiles of another launch, which take a
// compute unit's whole LDS, tiles that take all of it too: two of the smaller
// ones leave a unit at different times, and it stands half empty until both
// have (24 text rows of 151936 beside 1024 / 2048 audio rows of 32768, H 4096:
// 471 / 727 us with 128-column tiles, 443 / 689 with 256).
StreamTile stream_tile(int32_t M, int32_t N, bool beside) {
  if (M > 32) return best_shape(M, N);
  if (beside) return tile_of<32, 256>();
  return (N + 127) / 128 < 256 ? tile_of<32, 64>() : tile_of<32, wide_columns(32)>();
}

int32_t stream_stages(int rows, int cols) {
  if (rows == 32 && cols == 128) return tile_of<32, 128>().stages;
  for (const StreamTile &t : kShapes)
    if (t.rows == rows && t.cols == cols) return t.stages;
  return 0;
}

hipError_t launch_stream_gemm(const HeadView &hv, const StepView &sv, bool text,
                              hipStream_t st) {
  return text ? launch_tiles<true>(hv, sv, sv.n_text, hv.V_text, st)
              : launch_tiles<false>(hv, sv, sv.Mg, hv.N, st);
}

}  // namespace mcd
