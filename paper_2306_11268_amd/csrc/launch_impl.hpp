// Per-size choice and launch of the separable passes: which kernel, tile width
// and schedule each (FFT length, kind, axis) takes.
#pragma once

#include "kernels_impl.hpp"
#include "sep_impl.hpp"

namespace lr {

// ---------------------------------------------------------------------------
// Per-size launchers (explicitly instantiated in one translation unit per size)
// ---------------------------------------------------------------------------

// Vectors per workgroup by FFT length (the workgroup has T * N2 threads).
template <int N> struct TileT;
template <> struct TileT<64>   { static constexpr int T = 16; };
template <> struct TileT<100>  { static constexpr int T = 16; };
template <> struct TileT<128>  { static constexpr int T = 16; };
template <> struct TileT<200>  { static constexpr int T = 32; };  // column seed pass 132 -> 121 us, map 143 -> 124, last pass of a map 126 -> 115 against 16 (its covered columns alone 61 -> 71)
template <> struct TileT<256>  { static constexpr int T = 8; };
template <> struct TileT<350>  { static constexpr int T = 32; };  // 14 slots: T * 14 threads must be whole waves
template <> struct TileT<400>  { static constexpr int T = 8; };
template <> struct TileT<500>  { static constexpr int T = 16; };  // 20 slots: T * 20 threads must be whole waves
template <> struct TileT<512>  { static constexpr int T = 8; };
template <> struct TileT<1000> { static constexpr int T = 8; };
template <> struct TileT<1024> { static constexpr int T = 8; };

template <int N>
using CfgFor = Cfg<typename PlanFor<N>::type, TileT<N>::T>;
template <int N>
using RowCfgFor = Cfg<typename RowPlanFor<N>::type, TileT<N>::T>;

// Vectors per workgroup of the separable layer passes, by kind and axis where
// a measured sweep preferred another width than the size default (fields and
// tables do not depend on it).
template <int N, int KIND, int AXIS>
struct LayerTile {
  static constexpr int T = TileT<N>::T;
};
template <> struct LayerTile<200, kFwdMid, kCol> { static constexpr int T = 32; };
template <> struct LayerTile<200, kPropOnce, kRow> { static constexpr int T = 32; };
template <> struct LayerTile<200, kBwdMid, kCol> { static constexpr int T = 16; };
template <> struct LayerTile<200, kFwdMid, kRow> { static constexpr int T = 8; };
template <> struct LayerTile<200, kBwdMid, kRow> { static constexpr int T = 8; };
template <> struct LayerTile<200, kBwdLast, kCol> { static constexpr int T = 32; };
// 400: the column layer passes at 16 vectors (pitch 17: the A-item and
// B-item reads of a 16-lane group fall in distinct bank pairs; at 8 vectors
// two B-items share each group's pairs), four-wave workgroups of 55 KB, 8
// waves per CU against 10 (5-layer training step, batch 500: adjoint column
// passes 576 -> 485 us and 391 -> 337 us; forward, padded fields only, 320 in
// 400, batch 100: 68 -> 67)
template <> struct LayerTile<400, kFwdMid, kCol> { static constexpr int T = 16; };
template <> struct LayerTile<400, kBwdMid, kCol> { static constexpr int T = 16; };
template <> struct LayerTile<400, kBwdLast, kCol> { static constexpr int T = 16; };
// The widths from here on serve padded fields (a field that fills the grid runs
// these kinds on sep_pass); measured with the aperture at 0.8 of the grid, 5
// layers, against the size default.
// 500: the forward passes in one ten-wave workgroup of 32 vectors per CU
// instead of one five-wave workgroup of 16 (a 68 KB five-wave workgroup
// leaves no room for a second one on a CU): first pass 210 -> 165 us, rows 361
// -> 304, columns 349 -> 282 (batch 200)
template <> struct LayerTile<500, kPropOnce, kRow> { static constexpr int T = 32; };
template <> struct LayerTile<500, kFwdMid, kRow> { static constexpr int T = 32; };
template <> struct LayerTile<500, kFwdMid, kCol> { static constexpr int T = 32; };
// 512: the adjoint row pass at 16 vectors, 143.5 -> 128 us (batch 64; the first
// pass is even at 54.5)
template <> struct LayerTile<512, kPropOnce, kRow> { static constexpr int T = 16; };
template <> struct LayerTile<512, kBwdMid, kRow> { static constexpr int T = 16; };
// 1000: first pass 84 -> 71 us, rows 148 -> 123, columns 135 -> 111 (batch 16)
template <> struct LayerTile<1000, kPropOnce, kRow> { static constexpr int T = 16; };
template <> struct LayerTile<1000, kFwdMid, kRow> { static constexpr int T = 16; };
template <> struct LayerTile<1000, kFwdMid, kCol> { static constexpr int T = 16; };
// (the adjoint passes keep the default: at 32 vectors of 500 and 16 of 1000 their
// registers, capped at 168 for ten waves, spill)

template <int N, int KIND, int AXIS>
using LayerCfg = Cfg<std::conditional_t<AXIS == kRow, typename RowPlanFor<N>::type, typename PlanFor<N>::type>,
                     LayerTile<N, KIND, AXIS>::T>;

// The forward row layer pass at 200 points runs on wave tiles: each wave's
// loads cover 8 whole 64-byte runs of its rows.
template <int N, int KIND, int AXIS>
constexpr bool wave_tile_kind() {
  return N == 200 && AXIS == kRow && KIND == kFwdMid;
}

// Passes of a slot-ordered field that run on register-resident items
// (sep_impl.hpp) rather than on tiles in shared memory, where they measured
// faster (tile -> register, us; batch 500 at 64, 100 and 200 points, 300 at
// 128, 200 at 256 and 500, 100 at 400, 64 at 350 and 512, 16 at 1000 and 1024):
//   detector-plane row passes, every length: last forward 13.4 -> 12.6 (100),
//     29.8 -> 25.6 (200), 82 -> 45 (350, full map), 105 -> 55 (500), 126 -> 65
//     (1000, full map); adjoint seed 105 -> 56 (350), 177 -> 98 (500);
//   row layer passes: forward 16.3 -> 13.6 (64), 32 -> 24 (128), 64 -> 52 (256),
//     84 -> 67 (400), 313 -> 280 (500), 145 -> 113 (1000), but 82 -> 84 (200);
//     adjoint 22.4 -> 19.9 (64), 49.5 -> 42 (128), 127 -> 110 (200), 105 -> 95
//     (256), 127 -> 99 (400), 231 -> 199 (1000), but 42 -> 47 (100: items of 4
//     values, seven rounds of them); even at 500, where one-wave tiles of its own
//     kernel measured 442 next to the other passes of this table and these 445;
//   first row pass: 20 -> 18 (128), 46 -> 39 (256), 57 -> 45 (400), 84 -> 63
//     (1000), but 63 -> 65 (200) and 23 -> 27 (100), where the natural row is
//     staged for short items, and even at 64;
//   forward column pass: 30 -> 26 (100), 28 -> 25 (128), 78 -> 50 (256), 80 -> 71
//     (400), 349 -> 301 (500), 136 -> 134 (1000), but 84 -> 86 (200), 122.5 -> 126
//     (1024) and even at 64;
//   adjoint column passes: 20 -> 19 (64), 132 -> 103 (256), 625 -> 580 (500),
//     236 -> 215 (512), but 42 -> 44 (100), 134 -> 137 (200), 75 -> 83 (350), 111 ->
//     118 (400), 236 -> 288 (1000) and even at 128 and 1024: there the tile
//     passes' two barriers a propagation outweigh their fewer waves.
template <int N, int KIND, int AXIS>
constexpr bool sep_kind() {
  constexpr bool SHORT = N == 100 || N == 200;
  if (KIND == kFwdLast || KIND == kBwdFirst) return AXIS == kRow;
  if (AXIS == kRow && KIND == kBwdMid) return N != 100;
  if (AXIS == kRow) return KIND != kBwdLast && !SHORT;
  if (KIND == kFwdMid) return N != 64 && N != 200 && N != 1024;
  return (KIND == kBwdMid || KIND == kBwdLast) && (N == 64 || N == 256 || N == 500 || N == 512);
}
// Vectors per workgroup of those passes (rows: one wave, or four at 40 slots;
// columns: four waves, or eight at 40 slots), and the exchange of the
// accumulating kinds: complex values where the A-items are of at most 25 (the barriers
// and the shared-memory instructions saved, and a prefetched input, outweigh
// the waves: 400 points, adjoint row pass 116 -> 101 us), else one component.
template <int N, int KIND, int AXIS>
struct SepFor {
  using PL = typename PlanFor<N>::type;
  static constexpr bool ACC = KIND == kBwdMid || KIND == kBwdLast;
  using type = std::conditional_t<AXIS == kRow,
                                  Sep<PL, kRow, (PL::N2 <= 32 ? 64 : 256) / PL::N2, true, !(ACC && PL::N1 <= 25)>,
                                  Sep<PL, kCol, (PL::N2 <= 32 ? 256 : 512) / PL::N2, ACC, !ACC>>;
};

// The column kinds take the tile passes where a batch leaves the CUs fewer than
// two register workgroups each (12-64 columns each, against 8-32): at half of
// that and below they measured 5-30% slower (100 points, 16 samples, forward 11.5
// us on tiles, 13.7; 256, 8 samples, 11.1 and 12.5, adjoint 15.1 and 16.8; 512, 8
// samples, 22.6 and 24.9, last adjoint 32.6 and 41.8; 1000, 4 samples, 36.8 and
// 43.4).  Forward at 350 and 500 points, where a tile is alone on its CU, the
// register passes are even from one sample on; the adjoint ones at 500 are
// slower up to about 28 samples (16: 60 and 70) and, the last, 128 (64: 145 and
// 154).  At 512 the adjoint layer pass is the slower one again past 128 samples
// (256: 809 and 833, 500: 1536 and 1652).
template <int N, int KIND, int AXIS>
bool use_sep(int batch) {
  if constexpr (!sep_kind<N, KIND, AXIS>()) {
    return false;
  } else if constexpr (AXIS == kRow) {
    return true;
  } else {
    constexpr int T = SepFor<N, KIND, AXIS>::type::T;
    constexpr bool ACC = KIND == kBwdMid || KIND == kBwdLast;
    constexpr int least = !ACC && (N == 350 || N == 500) ? 0 : N == 500 ? (KIND == kBwdLast ? 21 : 5) : 2;  // per CU
    const long long groups = (long long)((N + T - 1) / T) * batch;
    if (N == 512 && KIND == kBwdMid && groups > 16ll * device_cus()) return false;
    return groups >= (long long)least * device_cus();
  }
}

// FULL: a slot-ordered field.
template <int N, int KIND, int AXIS, bool FULL>
hipError_t launch_fr(const PassArgs& a, hipStream_t st) {
  if constexpr (FULL && sep_kind<N, KIND, AXIS>()) {
    if (use_sep<N, KIND, AXIS>(a.batch)) {
      using G = typename SepFor<N, KIND, AXIS>::type;
      if constexpr (KIND == kFwdLast || KIND == kBwdFirst) {
        if (a.ntiles < 1 || a.batch < 1) return hipErrorInvalidValue;
        hipLaunchKernelGGL((sep_detector_pass<G, KIND>), dim3(a.ntiles * a.batch), dim3(G::P), 0, st, a);
      } else {
        if (a.workers < 1 || (KIND == kPropOnce && !a.in_real)) return hipErrorInvalidValue;
        hipLaunchKernelGGL((sep_pass<G, KIND>), dim3(8 * ((a.workers + 7) / 8)), dim3(G::P), 0, st, a);
      }
      return hipGetLastError();
    }
  }
  if constexpr (FULL && AXIS == kRow && sep_kind<N, KIND, AXIS>()) {
    return hipErrorInvalidValue;  // (row kinds have no second variant)
  } else if constexpr (FULL && wave_tile_kind<N, KIND, AXIS>()) {
    if (a.workers < 1) return hipErrorInvalidValue;
    const dim3 grid(8 * ((a.workers + 7) / 8));
    hipLaunchKernelGGL((wave_pass<typename PlanFor<N>::type, KIND, AXIS>), grid, dim3(64), 0, st, a);
  } else if constexpr (KIND == kFwdLast || KIND == kBwdFirst) {
    using C = std::conditional_t<AXIS == kRow, RowCfgFor<N>, CfgFor<N>>;
    const dim3 grid(work_grid(a.ntiles, (a.batch + a.spg - 1) / a.spg));
    hipLaunchKernelGGL((detector_pass<C, KIND, AXIS, FULL>), grid, dim3(C::P), 0, st, a);
  } else {
    using C = LayerCfg<N, KIND, AXIS>;
    if (a.workers < 1) return hipErrorInvalidValue;
    const dim3 grid(8 * ((a.workers + 7) / 8));
    hipLaunchKernelGGL((fresnel_pass<C, KIND, AXIS, FULL>), grid, dim3(C::P), 0, st, a);
  }
  return hipGetLastError();
}

template <int N, int KIND, int AXIS>
int slots_sep() {
  static int per_cu = 0;
  if (per_cu == 0) {
    using G = typename SepFor<N, KIND, AXIS>::type;
    per_cu = resident_per_cu(reinterpret_cast<const void*>(&sep_pass<G, KIND>), G::P);
  }
  return per_cu * device_cus();
}
template <int N, int KIND, int AXIS, bool FULL>
int slots_fr(int full) {
  if constexpr (FULL && sep_kind<N, KIND, AXIS>()) {
    if (use_sep<N, KIND, AXIS>(full)) return slots_sep<N, KIND, AXIS>();
  }
  static int per_cu = 0;
  if (per_cu == 0) {
    if constexpr (FULL && AXIS == kRow && sep_kind<N, KIND, AXIS>()) {
      return 0;
    } else if constexpr (FULL && wave_tile_kind<N, KIND, AXIS>()) {
      per_cu = resident_per_cu(reinterpret_cast<const void*>(&wave_pass<typename PlanFor<N>::type, KIND, AXIS>), 64);
    } else {
      using C = LayerCfg<N, KIND, AXIS>;
      per_cu = resident_per_cu(reinterpret_cast<const void*>(&fresnel_pass<C, KIND, AXIS, FULL>), C::P);
    }
  }
  return per_cu * device_cus();
}

template <int N, int KIND>
int slots_fr_axis(Axis axis, int full) {
  if (full) return axis == kRow ? slots_fr<N, KIND, kRow, true>(full) : slots_fr<N, KIND, kCol, true>(full);
  return axis == kRow ? slots_fr<N, KIND, kRow, false>(0) : slots_fr<N, KIND, kCol, false>(0);
}

template <int N, int KIND>
int tile_fr_axis(Axis axis, int full) {
  if constexpr (sep_kind<N, KIND, kRow>()) {
    if (axis == kRow && full) return SepFor<N, KIND, kRow>::type::T;
  }
  if constexpr (sep_kind<N, KIND, kCol>()) {
    if (axis == kCol && full && use_sep<N, KIND, kCol>(full)) return SepFor<N, KIND, kCol>::type::T;
  }
  if constexpr (KIND == kFwdLast || KIND == kBwdFirst) return TileT<N>::T;
  if (axis == kRow) return full && wave_tile_kind<N, KIND, kRow>() ? 8 : LayerTile<N, KIND, kRow>::T;
  return full && wave_tile_kind<N, KIND, kCol>() ? 8 : LayerTile<N, KIND, kCol>::T;
}

// Vectors per workgroup of a separable pass (full: samples of a call on a
// slot-ordered field, 0 for a padded one).
template <int N>
int tile_fr_n(PassKind kind, Axis axis, int full) {
  switch (kind) {
    case kPropOnce: return tile_fr_axis<N, kPropOnce>(axis, full);
    case kFwdMid: return tile_fr_axis<N, kFwdMid>(axis, full);
    case kBwdMid: return tile_fr_axis<N, kBwdMid>(axis, full);
    case kBwdLast: return tile_fr_axis<N, kBwdLast>(axis, full);
    case kFwdLast: return tile_fr_axis<N, kFwdLast>(axis, full);
    case kBwdFirst: return tile_fr_axis<N, kBwdFirst>(axis, full);
  }
  return 0;
}

template <int N>
int slots_fr_n(PassKind kind, Axis axis, int full) {
  switch (kind) {
    case kPropOnce: return slots_fr_axis<N, kPropOnce>(axis, full);
    case kFwdMid: return slots_fr_axis<N, kFwdMid>(axis, full);
    case kBwdMid: return slots_fr_axis<N, kBwdMid>(axis, full);
    case kBwdLast: return slots_fr_axis<N, kBwdLast>(axis, full);
    default: return 0;
  }
}

template <int N, int KIND>
hipError_t launch_fr_axis(Axis axis, const PassArgs& a, hipStream_t st) {
  if (a.full) return axis == kRow ? launch_fr<N, KIND, kRow, true>(a, st) : launch_fr<N, KIND, kCol, true>(a, st);
  return axis == kRow ? launch_fr<N, KIND, kRow, false>(a, st) : launch_fr<N, KIND, kCol, false>(a, st);
}

template <int N>
hipError_t launch_fr_n(PassKind kind, Axis axis, const PassArgs& a, hipStream_t st) {
  if (a.full && a.n != N) return hipErrorInvalidValue;
  switch (kind) {
    case kPropOnce: return launch_fr_axis<N, kPropOnce>(axis, a, st);
    case kFwdMid: return launch_fr_axis<N, kFwdMid>(axis, a, st);
    case kFwdLast: return launch_fr_axis<N, kFwdLast>(axis, a, st);
    case kBwdFirst: return launch_fr_axis<N, kBwdFirst>(axis, a, st);
    case kBwdMid: return launch_fr_axis<N, kBwdMid>(axis, a, st);
    case kBwdLast: return launch_fr_axis<N, kBwdLast>(axis, a, st);
  }
  return hipErrorInvalidValue;
}

// Whether the row layer passes of a forward or backward call read row-major
// tables (sep_pass) rather than the [col][row] ones of the tile passes.
template <int N>
bool row_major_n(bool backward) { return backward ? sep_kind<N, kBwdMid, kRow>() : sep_kind<N, kFwdMid, kRow>(); }

template <int N>
TileShape shape_n() { return TileShape{CfgFor<N>::T, CfgFor<N>::S}; }

// The slot order of the separable passes' stored fields: rows and columns
// use the same plan, so one map serves both axes.
template <int N>
SlotMap slot_map_n() {
  using PL = typename PlanFor<N>::type;
  static_assert(std::is_same_v<PL, typename RowPlanFor<N>::type>, "stored slot order needs one plan for both axes");
  return SlotMap{PL::N1, PL::N2, PL::PFA ? 1 : 0};
}

}  // namespace lr
