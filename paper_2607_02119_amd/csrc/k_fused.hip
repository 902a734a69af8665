// How a batch of audio and text rows runs (mixed_form), and K1 for such a batch
// in one launch with wide audio tiles: the audio rows' projection with the CFG
// merge and temperature (Sec. 2.1, Eq. 1, Sec. 2.4) in 256 x 256 MFMA tiles,
// and the text rows' projection with its (max, lowest argmax) partials in the
// four-wave streaming tiles of stream_tile.h (Sec. 2.4: the text head takes no
// CFG).
//
// Workgroups [0, n_audio) run audio tiles, the rest text tiles.  Workgroups
// are dispatched in index order, so the longer audio tiles start first and
// the text tiles fill the compute units as they free up.  One launch on one
// stream replaces two concurrent launches on two streams, and with them the
// cross-stream fork and join of every step.  Audio sums are those of the audio
// rows alone in the same tiles; text sums agree with those of a text launch,
// whose tiles split and walk k otherwise, within fp32 rounding.
#include "mfma2_tile.h"
#include "mixed_tile.h"

namespace mcd {
namespace {

template <int BNT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void head_gemm_mixed(
    HeadView hv, StepView sv, int n_audio) {
  constexpr int LA = M2Shape::kLds, LT = DmaShape<128, BNT>::kLds;
  __shared__ __attribute__((aligned(1024))) char lds[LA > LT ? LA : LT];
  const int b = blockIdx.x;
  if (b < n_audio) mfma2_tile(hv, sv, b, n_audio, lds);
  else dma_tile<128, BNT>(hv, sv, b - n_audio, lds);
}

template <int BNT>
hipError_t launch_mixed(const HeadView &hv, const StepView &sv, int n_audio, hipStream_t st) {
  const int n_text = (hv.V_text + BNT - 1) / BNT;   // one row tile of 128 text rows
  hipLaunchKernelGGL((head_gemm_mixed<BNT>), dim3((unsigned)(n_audio + n_text)), dim3(256), 0,
                     st, hv, sv, n_audio);
  return hipGetLastError();
}

enum class Mixed { kTwoLaunches, kStreaming, kWideAudio };

// Fewer text rows (at most 64) beside many 256 x 256 audio tiles: two launches,
// where those save more than a fork and a join cost against 128 x 256 streaming
// tiles, in the unit of stream_cost (384 a streaming tile; a wide one 710 to 730,
// less where H is long and its prologue and epilogue weigh less).
//
// A text part of a round or more fills the gaps of either's last round, so that
// the tiles count and not their rounds.  Streaming tiles for both / two
// launches, us, audio rows of 32768 columns, text rows of 151936: H 4096, 768
// with 64 419 / 413, 1024 with 64 484 / 466, 1536 with 64 622 / 581, 1024 with 24
// 455 / 448, 1280 with 24 527 / 516, 1800 with 24 692 / 653, 512 with 24 321 / 344,
// 896 with 64, whose 256 x 256 tiles are one eighth padding, 429 / 450.  H 2560:
// 768 with 64 297 / 299, 1664 with 24 450 / 429.  H 2048: 1024 with 64 267 / 273,
// 1664 with 24 351 / 350, 1800 with 24 385 / 366.  H 1600: 1024 with 64 224 / 234,
// 1536 with 64 287 / 279, 1664 with 24 293 / 298, 1800 with 24 326 / 311.
//
// A smaller one adds tiles to the last round, or a round.  With 8 text rows of
// 8000: 1024 rows 275 / 308, 1536 423 / 433, 1800 524 / 495, 2048 562 / 549; 1800 at
// H 2560 388 / 357, at H 2048 295 / 300; 2432 at H 1600 323 / 318, at H 1024
// 222 / 233; 2048 at H 1024 211 / 188.  2048 with 64 of 32003 605 / 594, at H 1024 211 / 220.
bool two_launches(int32_t Mg, int32_t N, int32_t n_text, int32_t V_text, int32_t H) {
  if (n_text > 64) return false;
  const int64_t wide = tiles_256(Mg, N), rows = tiles_128x256(Mg, N);
  if (text_fills(n_text, V_text)) {   // two rounds of text tiles fill more than one
    const int64_t w = V_text <= 511 * 256 ? 730 : H >= 2048 ? 710 : 718;
    return wide * w < rows * 384 &&
           (wide >= 768 || (wide >= 512 && H >= 2560) || (wide >= 384 && n_text > 32 && H >= 3072));
  }
  auto with_text = [](int64_t tiles, int64_t cost, int64_t text) {
    return (tiles + 255) / 256 * cost + (tiles % 256 == 0 ? text : 0);
  };
  return wide >= 1024 && (n_text <= 32 || H >= 1536) &&
         with_text(wide, H >= 2560 ? 710 : H >= 1536 ? 722 : 730, 210) < with_text(rows, 384, 160) &&
         mfma_tile(Mg, N, false, false).stages == 0;
}

// More than 64 text rows (one row tile of 128) beside at least one round of 256
// x 256 audio tiles: those two in one launch.  Where the line lies (steps, H
// 4096): 768 audio rows of 32768 columns with 128 text rows of 151936 take 455
// us so and 465 in streaming tiles.  Otherwise streaming tiles in one launch.
Mixed mixed_form(int32_t Mg, int32_t N, int32_t n_text, int32_t V_text, int32_t H) {
  if (Mg < 1 || n_text < 1 || n_text > 128) return Mixed::kTwoLaunches;
  const int64_t n_audio = tiles_256(Mg, N);
  if (Mg > 128 && n_text > 64 && n_audio >= 256)
    return n_audio > (1 << 20) ? Mixed::kTwoLaunches : Mixed::kWideAudio;
  if (n_audio > (1 << 18) || two_launches(Mg, N, n_text, V_text, H)) return Mixed::kTwoLaunches;
  return Mixed::kStreaming;
}

// Columns of the text tiles beside 256 x 256 audio tiles: narrow where 128
// columns make less than one round, wide where they make more.
int beside_wide_audio(int32_t V_text) {
  const int t128 = (V_text + 127) / 128;
  return t128 < 256 ? 64 : t128 == 256 ? 128 : 256;
}

}  // namespace

hipError_t launch_mixed_gemm(const HeadView &hv, const StepView &sv, hipStream_t st,
                             bool *launched) {
  const Mixed form = hv.dtype == MCD_BF16
                         ? mixed_form(sv.Mg, hv.N, sv.n_text, hv.V_text, hv.H)
                         : Mixed::kTwoLaunches;
  *launched = form != Mixed::kTwoLaunches;
  if (form == Mixed::kTwoLaunches) return hipSuccess;
  if (form == Mixed::kStreaming) {
    switch (mixed_rows(sv.n_text)) {
      case 32: return launch_mixed_text_32(hv, sv, st);
      case 64: return launch_mixed_text_64(hv, sv, st);
      default: return launch_mixed_text_128(hv, sv, st);
    }
  }
  const int n_audio = (int)tiles_256(sv.Mg, hv.N);
  switch (beside_wide_audio(hv.V_text)) {
    case 64: return launch_mixed<64>(hv, sv, n_audio, st);
    case 128: return launch_mixed<128>(hv, sv, n_audio, st);
    default: return launch_mixed<256>(hv, sv, n_audio, st);
  }
}

ProjectionRoute projection_route(int32_t Mg, int32_t N, int32_t n_text, int32_t V_text,
                                 int32_t H) {
  ProjectionRoute r{0, {0, 0, 0}, {0, 0, 0}};
  const bool both = Mg > 0 && n_text > 0;
  auto part = [&](int32_t M, int32_t cols, bool text) {   // of launch_head_gemm_part
    ++r.launches;
    return M <= 128 ? stream_tile(M, cols, text && both) : mfma_tile(M, cols, text, text_fills(n_text, V_text));
  };
  switch (both ? mixed_form(Mg, N, n_text, V_text, H) : Mixed::kTwoLaunches) {
    case Mixed::kStreaming: {
      const int ra = mixed_rows(Mg), rt = mixed_rows(n_text);
      const int ca = wide_audio(Mg, N) ? wide_columns(ra) : 64;
      const int ct = wide_text(V_text) ? wide_columns(rt) : 64;
      return ProjectionRoute{1, {ra, ca, stream_stages(ra, ca)}, {rt, ct, stream_stages(rt, ct)}};
    }
    case Mixed::kWideAudio: {
      const int ct = beside_wide_audio(V_text);
      const int stages = ct == 64 ? DmaShape<128, 64>::SW
                         : ct == 128 ? DmaShape<128, 128>::SW : DmaShape<128, 256>::SW;
      return ProjectionRoute{1, {256, 256, 0}, {128, ct, stages}};
    }
    case Mixed::kTwoLaunches: break;
  }
  if (Mg > 0) r.audio = part(Mg, N, false);
  if (n_text > 0) r.text = part(n_text, V_text, true);
  return r;
}

}  // namespace mcd

extern "C" void mcd_projection_route(int32_t Mg, int32_t N, int32_t n_text, int32_t V_text,
                                     int32_t H, int32_t out[7]) {
  const mcd::ProjectionRoute r = mcd::projection_route(Mg, N, n_text, V_text, H);
  const int32_t w[7] = {r.launches,   r.audio.rows, r.audio.cols, r.audio.stages,
                        r.text.rows,  r.text.cols,  r.text.stages};
  for (int i = 0; i < 7; ++i) out[i] = w[i];
}
