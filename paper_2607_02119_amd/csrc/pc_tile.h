// Tile body of the K1 weight-streaming path, copying and computing waves apart:
// codebook-head projection with the CFG merge and temperature fused into the
// epilogue (TEXT = false), or the text-head projection with a fused (max, lowest
// argmax) epilogue; the formulas are at the head of k_stream.hip.
#pragma once

#include "stream_tile.h"

namespace mcd {
namespace {

// A workgroup has eight waves, two per SIMD.  Waves 0-3 only read fragments
// from LDS and issue MFMAs; waves 4-7 only bring in slices of 64 k (128 bytes
// of every weight and hidden row of the tile): waves 4-5 copy the weights
// global -> LDS, non-temporal, SW stages deep; waves 6-7 load the hidden rows
// into registers HL slices ahead and write them to a ring of SA stages.
//
// The buffers are sized by bytes in flight: hidden rows come from L2, but behind
// the weights' HBM reads in the compute unit's in-order return path, so every
// byte takes 1.5 - 2 us under load, and 100 GB/s per compute unit would need 150 -
// 200 KiB under way.  The registers of the loading waves hold the hidden rows'
// part of it, the LDS the weights' part; neither costs the computing waves a
// stall, where a wave that also computes adds its copies and LDS writes to its
// MFMAs.  The loops take in 42 - 50 GB/s with about that much under way, so
// this is not all that bounds them.
//
// The computing waves split a slice by columns and k: KSPLIT k groups of
// 4 / KSPLIT column groups.  One barrier per slice: at the barrier of slice st,
// slice st + 1 has landed and every fragment of slice st is in registers (it
// stands before the MFMAs of the last k16 step), so stage st is filled again
// at once.  LDS layout of a slice as in stream_tile.h.
template <int BM, int BN>
struct PcShape {
  static constexpr int SK = kDmaSK, ROWB = SK * 2, NT = 512;
  // k groups, for at most 128 accumulators per lane: four (every fragment is read
  // by one wave only) up to 64 x 128 outputs, two up to 128 x 128, else one
  static constexpr int KSPLIT = BM * BN <= 64 * 128 ? 4 : BM * BN <= 128 * 128 ? 2 : 1;
  static constexpr int CSPLIT = 4 / KSPLIT, KS = 4 / KSPLIT;   // column groups, k16 steps per slice
  static constexpr int WN = BN / CSPLIT;                       // columns per wave
  static constexpr int MB = BM / 32, NB = WN / 32;
  static constexpr int WST = BN * ROWB, AST = BM * ROWB;
  static constexpr int WIW = WST / 1024 / 2, AIA = AST / 1024 / 2;   // copies per wave and slice
  // 32 rows: half of the LDS, so that two tiles share a compute unit and the
  // start and end of one run under the other's loop (24 text rows, 151936 x
  // 4096: 207 us at one tile per compute unit, 200 at two, 210 with 256
  // columns; 6.2 TB/s).  In one launch with taller audio tiles the workgroup
  // takes their LDS, and a compute unit has one.
  static constexpr int kBudget = (BM == 32 && BN <= 128 ? 80 : 160) * 1024;
  static constexpr int SA = BN == 64 ? 3 : 2;
  static constexpr int HL = BM == 128 ? 6 : 8;   // hidden slices in flight in registers
  // Of the up to 16 weight stages that fit, at most six in the smaller tiles and
  // eight in the others: the weight waves fill the ring before the first hidden
  // rows are asked for, which then return behind it, and a tile of few slices
  // waits for both.  All that fit / eight / six, us, at H 1024, 1600, 4096: 64
  // rows of 16384 columns (64 x 64) 11.5 / 10.8 / 10.3, 14.6 / 14.0 / 13.5, 29.1
  // / 28.9 / 28.0; 200 of 8192 (128 x 64) 12.6 / 11.7 / 11.7, 16.7 / 15.2 / 15.1,
  // 30.3 / 28.9 / 29.7; 64 of 32768 (64 x 128, eight fit) at H 1600 - / 21.6 /
  // 22.1.
  static constexpr int SW0 = (kBudget - SA * AST) / WST;
  static constexpr int SWM = BM * BN < 128 * 64 ? 6 : 8, SWV = 63 / WIW + 1;   // counter range
  static constexpr int SW1 = SW0 < SWM ? SW0 : SWM, SW = SW1 < SWV ? SW1 : SWV;
  static constexpr int CP = BN + 4;        // padded row pitch of the sums (floats)
  static constexpr int kRing = SW * WST + SA * AST;
  static constexpr int kParams = (BM / 2) * 16;
  static constexpr int kEpi = KSPLIT * BM * CP * 4 + kParams;
  static constexpr int kLds = kRing > kEpi ? kRing : kEpi;
  static_assert(SW >= 3 && (SW - 1) * WIW < 64 && kLds <= 160 * 1024, "ring depths");
};

// Columns of a tile when 128-column tiles make more than one round: 256, half
// the hidden-state bytes per weight byte, or 128 for 32 rows, whose hidden
// states are few.
constexpr int wide_columns(int bm) { return bm == 32 ? 128 : 256; }

// One BM x BN tile (tile index bx: row tile bx % tiles_m, column tile
// bx / tiles_m) with 512 threads and the workgroup's LDS buffer `lds` of
// PcShape<BM, BN>::kLds bytes (1024-byte aligned).
// ALONE: no other tiles in the launch.
template <int BM, int BN, bool TEXT, bool ALONE>
__device__ __forceinline__ void pc_tile(const HeadView &hv, const StepView &sv, int bx, char *lds) {
  using S_ = PcShape<BM, BN>;
  constexpr int SK = S_::SK, MB = S_::MB, NB = S_::NB, ROWB = S_::ROWB, KS = S_::KS;
  constexpr int WST = S_::WST, AST = S_::AST, SW = S_::SW, SA = S_::SA, CP = S_::CP;
  constexpr int WIW = S_::WIW, AIA = S_::AIA, HL = S_::HL;
  float4 *const rowp = reinterpret_cast<float4 *>(lds + S_::kLds - S_::kParams);

  const int32_t *rows = sv.plan + kPlanHeader + (TEXT ? sv.Mg : 0);
  const int M = TEXT ? sv.n_text : sv.Mg;
  const int N = TEXT ? hv.V_text : hv.N;
  const int H = hv.H;
  const int NST = H / SK;
  const int tiles_m = (M + BM - 1) / BM;
  // Several row tiles: workgroups are dealt to the 8 XCDs in turn, so the
  // index is remapped to give each XCD a contiguous run of tiles (one more in
  // the first XCDs where the runs are not equal), in which the row tiles of a
  // column tile are neighbours, run at the same time and walk k in the same
  // order: they share that column tile's weights through the L2.
  if (tiles_m > 1) {
    const int ntiles = tiles_m * ((N + BN - 1) / BN);
    bx = (bx % 8) * (ntiles / 8) + min(bx % 8, ntiles % 8) + bx / 8;
  }
  const int tile_m = bx % tiles_m, tile_n = bx / tiles_m;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q2 = tid - 384;                // row pair of a thread of waves 6-7
  PairLoads praw{0.0f, 0.0f, 0.0f, 0, false, false};
  float *const C = reinterpret_cast<float *>(lds);

  if (wave >= 4) {
    // ---- copying waves ----
    // Tiles walk k from offsets of their own (see stream_tile.h).
    const int kskew = (int)(((unsigned)tile_n * 7u) % (unsigned)NST);
    const int seg_r = lane >> 3, seg_c = lane & 7;
    wait_vmem_and_lds<0>();
    if (wave < 6) {
      // the weights depend on nothing but the tile, so they start before the
      // plan is read
      const __bf16 *Wp = static_cast<const __bf16 *>(TEXT ? hv.W_text : hv.W);
      const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds +
                            (uint32_t)((wave - 4) * WIW * 1024);
      const __bf16 *src[WIW];
      static_for<0, WIW>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const int r = ((wave - 4) * WIW + q) * 8 + seg_r;
        src[q] = Wp + (size_t)min(n0 + r, N - 1) * H + ((seg_c ^ ((r >> 1) & 7)) * 8);
      });
      auto issue = [&](int st) __attribute__((always_inline)) {
        int ks = st + kskew;
        ks = ks >= NST ? ks - NST : ks;
        const uint32_t sb = ring + (uint32_t)((st % SW) * WST);
        static_for<0, WIW>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          lds_copy16_stream(src[q] + ks * SK, sb + (uint32_t)(q * 1024));
        });
      };
      for (int st = 0; st < SW; ++st)
        if (st < NST) issue(st);
      if (!plan_ok(sv)) {
        wait_vmem_and_lds<0>();  // no copy may still be landing in this workgroup's LDS
        return;
      }
      // slice 0 has landed, then slice st + 1 for every st
      wait_slices<WIW, SW - 1>(NST - 1);
      block_barrier_no_vmem_wait();
      for (int st = 0; st < NST; ++st) {
        wait_slices<WIW, SW - 2>(max(NST - 2 - st, 0));
        block_barrier_no_vmem_wait();
        if (st + SW < NST) issue(st + SW);
      }
    } else {
      if (!plan_ok(sv)) return;
      const __bf16 *X = static_cast<const __bf16 *>(sv.hidden);
      // all row loads first (the copy sources and, for the epilogue, the rows
      // of a GEMM row pair per thread), then the checks
      // Rows past the end (never stored) repeat the last one, whose lines then come
      // from L1.  In wide tiles, several row tiles of them and a round or two of
      // tiles with no text rows beside, they go on at the first row: a last row
      // tile with lighter loads runs ahead of its neighbours, which share its
      // weights through L2 (200 / 130 rows of 32768 columns, H 1600: 37.3 / 39.6 us
      // with the last row, 34.7 / 34.6 so; 270 of 16384 33.1 / 30.1).  Elsewhere the
      // unit that it frees early is worth more (95 of 8192 in 128 x 64 tiles 11.2 /
      // 11.9; beside 8 text rows of 8000 1150 of 32768, H 2048, 176.7 / 182.9).
      int prow[AIA];
      auto rows_at = [&](auto &&row) __attribute__((always_inline)) {
        static_for<0, AIA>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          prow[q] = rows[row(m0 + ((wave - 6) * AIA + q) * 8 + seg_r)];
        });
      };
      auto clamped = [&](int g) __attribute__((always_inline)) { return min(g, M - 1); };
      if constexpr (ALONE && BM == 128 && BN >= 128) {
        const int tiles = tiles_m * ((N + BN - 1) / BN);
        if (tiles_m > 1 && tiles >= 128 && tiles <= 512 && sv.n_text == 0)
          rows_at([&](int g) __attribute__((always_inline)) { return g < M ? g : g - M; });
        else
          rows_at(clamped);
      } else {
        rows_at(clamped);
      }
      const int g0 = m0 + 2 * min(q2, BM / 2 - 1);
      int pr0 = 0, pr1 = 0;
      if constexpr (!TEXT) {
        pr0 = rows[min(g0, sv.Mg - 1)];
        pr1 = rows[min(g0 + 1, sv.Mg - 1)];
      }
      bool bad = false;
      const __bf16 *src[AIA];
      static_for<0, AIA>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const int r = ((wave - 6) * AIA + q) * 8 + seg_r;
        const bool ok = prow[q] >= 0 && prow[q] < sv.R;
        bad |= !ok;
        src[q] = X + (size_t)(ok ? prow[q] : 0) * H + ((seg_c ^ ((r >> 1) & 7)) * 8);
      });
      if constexpr (!TEXT) praw = pair_params_load(sv, g0, pr0, pr1);
      if (bad) atomicOr(sv.status, (uint32_t)MCD_DEV_BAD_PLAN);
      // Loads past the last slice re-load it (clamped; never stored), so that
      // every iteration issues the same loads and the compiler's waits for
      // them stay exact.
      char *const ring = lds + SW * WST + (wave - 6) * AIA * 1024 + lane * 16;
      auto load = [&](int st, u32x4 (&b)[AIA]) __attribute__((always_inline)) {
        int ks = min(st, NST - 1) + kskew;
        ks = ks >= NST ? ks - NST : ks;
        static_for<0, AIA>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          b[q] = *reinterpret_cast<const u32x4 *>(src[q] + ks * SK);
        });
      };
      auto store = [&](int st, const u32x4 (&b)[AIA]) __attribute__((always_inline)) {
        if (st >= NST) return;
        static_for<0, AIA>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          *reinterpret_cast<u32x4 *>(ring + (st % SA) * AST + q * 1024) = b[q];
        });
      };
      // buffer j holds the slices s >= SA with (s - SA) % HL == j; the first
      // SA slices go straight through buffers 0 .. SA - 1
      u32x4 hb[HL][AIA];
      static_for<0, SA>([&](auto jc) __attribute__((always_inline)) {
        load(decltype(jc)::value, hb[decltype(jc)::value]);
      });
      static_for<SA, HL>([&](auto jc) __attribute__((always_inline)) {
        load(SA + decltype(jc)::value, hb[decltype(jc)::value]);
      });
      static_for<0, SA>([&](auto jc) __attribute__((always_inline)) {
        store(decltype(jc)::value, hb[decltype(jc)::value]);
        load(SA + decltype(jc)::value, hb[decltype(jc)::value]);
      });
      wait_vmem_and_lds<63>();             // its writes
      block_barrier_no_vmem_wait();
      // after the barrier of slice st its stage is free for slice st + SA
      auto iteration = [&](int st, u32x4 (&b)[AIA]) __attribute__((always_inline)) {
        wait_vmem_and_lds<63>();
        block_barrier_no_vmem_wait();
        store(st + SA, b);
        load(st + SA + HL, b);
      };
      int st0 = 0;
      for (; st0 + HL <= NST; st0 += HL) {
        static_for<0, HL>([&](auto jc) __attribute__((always_inline)) {
          iteration(st0 + decltype(jc)::value, hb[decltype(jc)::value]);
        });
      }
      static_for<0, HL - 1>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        if (st0 + j < NST) iteration(st0 + j, hb[j]);
      });
    }
    // the copies are invisible to the compiler; the last iteration waited for
    // all of them, and this drain makes that explicit before LDS is reused
    wait_vmem_and_lds<0>();
    __syncthreads();
    if (!TEXT && q2 >= 0 && q2 < BM / 2) rowp[q2] = pair_params_finish(sv, praw);
  } else {
    // ---- computing waves ----
    if (!plan_ok(sv)) {
      if (blockIdx.x == 0 && tid == 0) atomicOr(sv.status, (uint32_t)MCD_DEV_BAD_PLAN);
      return;
    }
    const int ch = wave % S_::CSPLIT, kh = wave / S_::CSPLIT;
    floatx16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // lane l holds row (column) l % 32 and the 8 consecutive k of chunk
    // 2 (kh KS + step) + l / 32; the swizzle depends on l % 32 only
    const int frow = lane & 31;
    int foff[KS];
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2)
      foff[s2] = frow * ROWB + (((2 * (kh * KS + s2) + (lane >> 5)) ^ ((frow >> 1) & 7)) * 16);
    const char *const wring = lds + ch * S_::WN * ROWB, *const aring = lds + SW * WST;
    constexpr int NM = MB * NB, NR = MB + NB;
    bf16x8 fa[2][MB], fb[2][NB];
    auto read = [&](auto rc, int st, int off, auto bc) __attribute__((always_inline)) {
      constexpr int r = decltype(rc)::value, buf = decltype(bc)::value;
      if constexpr (r < NB)
        fb[buf][r] = *reinterpret_cast<const bf16x8 *>(wring + (st % SW) * WST + off + r * 32 * ROWB);
      else
        fa[buf][r - NB] = *reinterpret_cast<const bf16x8 *>(aring + (st % SA) * AST + off +
                                                            (r - NB) * 32 * ROWB);
    };
    // MFMAs of one k16 step from buffer buf; the fragments of the next step
    // (stage of slice st, offset off) are read between them
    auto step = [&](auto bc, int st, int off) __attribute__((always_inline)) {
      constexpr int buf = decltype(bc)::value;
      static_for<0, NM>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value, i = m / NB, j = m % NB;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
        static_for<0, NR>([&](auto rc) __attribute__((always_inline)) {
          constexpr int r = decltype(rc)::value;
          if constexpr (r * NM / NR == m) read(rc, st, off, std::integral_constant<int, 1 - buf>{});
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    auto arrive = [&]() __attribute__((always_inline)) {
      wait_vmem_and_lds<63>();             // this wave's fragment reads
      block_barrier_no_vmem_wait();
    };
    arrive();
    static_for<0, NR>([&](auto rc) __attribute__((always_inline)) {
      read(rc, 0, foff[0], std::integral_constant<int, 0>{});
    });
    if constexpr (KS == 1) {
      int st = 0;
      for (; st + 2 <= NST; st += 2) {     // past the end: read, never used
        arrive();
        step(std::integral_constant<int, 0>{}, st + 1, foff[0]);
        arrive();
        step(std::integral_constant<int, 1>{}, st + 2, foff[0]);
      }
      if (st < NST) {
        arrive();
        step(std::integral_constant<int, 0>{}, st + 1, foff[0]);
      }
    } else {
      for (int st = 0; st < NST; ++st) {   // past the end: read, never used
        static_for<0, KS>([&](auto sc) __attribute__((always_inline)) {
          constexpr int s2 = decltype(sc)::value;
          if constexpr (s2 + 1 == KS) arrive();
          step(std::integral_constant<int, (s2 & 1)>{}, s2 + 1 == KS ? st + 1 : st, foff[(s2 + 1) % KS]);
        });
      }
    }
    wait_vmem_and_lds<0>();
    __syncthreads();
    // the k groups' sums side by side in LDS (the rings are free)
    float *Cl = C + (kh * BM + (lane >> 5) * 4) * CP + ch * S_::WN + frow;
    static_for<0, MB * NB * 16>([&](auto fc) __attribute__((always_inline)) {
      constexpr int f = decltype(fc)::value;
      constexpr int i = f / (NB * 16), j = (f / 16) % NB, r = f % 16;
      Cl[(i * 32 + (r >> 2) * 8 + (r & 3)) * CP + j * 32] = acc[i][j][r];
    });
  }
  epilogue_from_lds<BM, BN, CP, TEXT, S_::KSPLIT, S_::NT>(hv, sv, C, rowp, m0, n0, M, N);
}

}  // namespace
}  // namespace mcd
