// K1 for a mixed batch in one launch, streaming tiles for both parts: the
// audio rows' projection with the CFG merge and temperature (Sec. 2.1, Eq. 1,
// Sec. 2.4) and the text rows' projection with its (max, lowest argmax)
// partials (Sec. 2.4: the text head takes no CFG).
#pragma once

#include "pc_tile.h"

namespace mcd {
namespace {

// Workgroups [0, n_audio) run BMA x BNA audio tiles, the rest BMT x BNT text
// tiles.  Two launches on two streams instead cost a fork and a join of events
// in every step.  Steps in two launches and in one: 95 audio rows of 7021
// columns with 9 text rows of 32003 (H 1600) 55.5 and 41.2 us; 16 audio rows
// of 8192 with 4 of 32000 (H 1024) 53.8 and 25.9; 512 audio rows of 32768 with
// 24 of 151936 (H 4096, two launches with 256 x 256 audio tiles) 374 and 339.
template <int BMA, int BNA, int BMT, int BNT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4))) void
head_gemm_mixed_pc(HeadView hv, StepView sv, int n_audio) {
  constexpr int LA = PcShape<BMA, BNA>::kLds, LT = PcShape<BMT, BNT>::kLds;
  __shared__ __attribute__((aligned(1024))) char lds[LA > LT ? LA : LT];
  const int b = blockIdx.x;
  if (b < n_audio) pc_tile<BMA, BNA, false, false>(hv, sv, b, lds);
  else pc_tile<BMT, BNT, true, false>(hv, sv, b - n_audio, lds);
}

template <int BMA, int BNA, int BMT, int BNT>
hipError_t launch_mixed_pc(const HeadView &hv, const StepView &sv, hipStream_t st) {
  const int n_audio = ((sv.Mg + BMA - 1) / BMA) * ((hv.N + BNA - 1) / BNA);
  const int n_text = (hv.V_text + BNT - 1) / BNT;   // one row tile: at most BMT text rows
  hipLaunchKernelGGL((head_gemm_mixed_pc<BMA, BNA, BMT, BNT>), dim3((unsigned)(n_audio + n_text)),
                     dim3(512), 0, st, hv, sv, n_audio);
  return hipGetLastError();
}

// Tile widths by each part on its own, not by the cost rule of its own launch
// (stream_tile): 64 columns where 128-column tiles are fewer than the compute
// units, wide ones otherwise; audio rows beyond 128 in 128 x 256 row tiles.
// The other part's tiles fill the units that this leaves idle.  Where both are
// small the rule costs time: 256 audio rows of 4096 columns with 8 text rows of
// 8000 (H 4096) take 61 us so and 44 with 32 x 64 audio tiles.
inline bool wide_audio(int32_t Mg, int32_t N) { return Mg > 128 || (N + 127) / 128 >= 256; }
inline bool wide_text(int32_t V_text) { return (V_text + 127) / 128 >= 256; }
// rows of a part's tiles
inline int mixed_rows(int32_t M) { return M <= 32 ? 32 : M <= 64 ? 64 : 128; }

template <int BMA, int BMT>
hipError_t launch_mixed_rows(const HeadView &hv, const StepView &sv, hipStream_t st) {
  const bool wa = wide_audio(sv.Mg, hv.N), wt = wide_text(hv.V_text);
  constexpr int WA = wide_columns(BMA), WT = wide_columns(BMT);
  if (wa) return wt ? launch_mixed_pc<BMA, WA, BMT, WT>(hv, sv, st)
                    : launch_mixed_pc<BMA, WA, BMT, 64>(hv, sv, st);
  return wt ? launch_mixed_pc<BMA, 64, BMT, WT>(hv, sv, st)
            : launch_mixed_pc<BMA, 64, BMT, 64>(hv, sv, st);
}

template <int BMT>
hipError_t launch_mixed_text(const HeadView &hv, const StepView &sv, hipStream_t st) {
  switch (mixed_rows(sv.Mg)) {
    case 32: return launch_mixed_rows<32, BMT>(hv, sv, st);
    case 64: return launch_mixed_rows<64, BMT>(hv, sv, st);
    default: return launch_mixed_rows<128, BMT>(hv, sv, st);
  }
}

}  // namespace
}  // namespace mcd
