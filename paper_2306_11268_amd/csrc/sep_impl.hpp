// Separable (Fresnel) layer and detector passes on register-resident items, for a
// layer that fills the grid (slot order, plan.hpp): the detector-plane rows at
// every length, the layer passes where they measured faster than the tile
// passes (sep_kind, launch_impl.hpp).
//
// The tile passes of kernels_impl.hpp keep a complex tile of N x T values in
// shared memory: at 350, 500 and 1000 points 68-104 KB, one workgroup of 5-7
// waves per CU, too few to hide any latency.  Here a lane keeps its A-item and
// then its B-items in registers, fields move between registers and global
// memory directly, and shared memory holds only the exchange between the two
// (exchange.hpp), one float component at a time: half the bytes.  The
// arithmetic and its order are those of the tile passes.
//
//   rows:    a workgroup transforms R whole rows, consecutive lanes
//            consecutive A-items; one wave where N2 <= 32 (no barriers);
//   columns: T columns, consecutive lanes consecutive columns, in four (or
//            eight) waves: a workgroup of 5, 6, 7 or 10 waves puts one more on
//            some SIMDs, always the same ones, so at 168 registers (three
//            waves a SIMD) a second five-wave workgroup does not fit a CU.  At
//            20 slots 12 columns fill 240 of 256 lanes, at 14 slots 18 fill 252.
#pragma once

#include "exchange.hpp"
#include "kernels_impl.hpp"

namespace lr {

// The left-over quarter round of B-items as one item per lane quad (the
// Good-Thomas 4 x Q split of b_spectral_quad).
template <class IT>
struct QuadItems {
  static constexpr int Q = IT::N2 / 4;
  static constexpr bool ON = IT::N2 % 4 == 0 && Q % 2 == 1 && Q > 1 && (IT::N1 % IT::N2) * 4 == IT::N2;
  static constexpr int E1 = ON ? Q * inv_mod(Q % 4, 4) : 0;
  static constexpr int E2 = ON ? 4 * inv_mod(4 % Q, Q) : 0;
};

// Geometry of a workgroup.  Entry (vector, k1, j) of the exchange buffer:
// rows v*PR + k1*P1 + j, columns (k1*P1 + j)*T + v.
template <class PL_, int AXIS_, int T_, bool REPEAT_ = AXIS_ == kRow, bool SPLIT_ = true>
struct Sep : Items<PL_, true> {
  using PL = PL_;
  using IT = Items<PL_, true>;
  using QI = QuadItems<IT>;
  static constexpr int AXIS = AXIS_;
  static constexpr bool ROWS = AXIS_ == kRow;
  static constexpr int T = T_;
  static constexpr int P = (T_ * IT::N2 + 63) / 64 * 64;
  static_assert(ROWS || P % 64 == 0, "whole waves");
  // lanes past the T vectors: in a one-wave workgroup they repeat the first
  // items of vector 0; else (SPARE) their A side is the exchange area's padding
  // column and on the B side they repeat item 0
  static constexpr bool SPARE = P != T_ * IT::N2 && P > 64;
  static constexpr int PR = IT::N1 * IT::P1 + (64 + IT::N2 - IT::N1 * IT::P1 % 64) % 64;
  static constexpr int SA = ROWS ? IT::P1 : IT::P1 * T_;  // A side: stride of k1
  static constexpr int SQ = ROWS ? 1 : T_;                // B side: stride of j
  static constexpr int BUF = ROWS ? T_ * PR : IT::N1 * IT::P1 * T_;
  static constexpr bool SPLIT = SPLIT_;  // exchange one component at a time
  using Elem = std::conditional_t<SPLIT_, float, float2>;
  static constexpr int IBW = QI::ON ? IT::IB - 1 : IT::IB;  // rounds of whole items
  static constexpr bool REPEAT = REPEAT_;  // exchange.hpp: repeat an item instead of branching
  static constexpr bool PARTIAL = !IT::FULL_ROUNDS && !QI::ON;
  // staged chirp (entry k1*P1 + k2); the widest items read the cached table in
  // global memory instead, which is in lane order for a Cooley-Tukey plan
  static constexpr bool TAB_LDS = PL_::PFA || IT::N < 512;
  static constexpr int TAB = TAB_LDS ? IT::N1 * IT::P1 : 1;
  static constexpr int Z = QI::ON ? QI::Q : 1;
};

template <class G>
struct SepLane {
  int v;     // vector of the tile
  int j;     // slot of the A-item
  int s;     // slot of the B-items
  int ab;    // A-side base
  int quad;  // lane index of the quad split
  bool act;
  __device__ __forceinline__ SepLane() {
    const int tid = (int)threadIdx.x;
    act = G::T * G::N2 == G::P || tid < G::T * G::N2;
    quad = act ? tid : tid - G::T * G::N2;
    v = G::ROWS ? (act ? tid / G::N2 : 0) : quad % G::T;
    j = G::ROWS ? (act ? tid - v * G::N2 : quad) : quad / G::T;
    s = j;
    if (G::SPARE && !act) {
      j = G::N2;
      s = 0;
    }
    ab = G::ROWS ? v * G::PR + j : j * G::T + v;
  }
  __device__ __forceinline__ int b_base(int k1) const {
    return G::ROWS ? v * G::PR + k1 * G::P1 : k1 * G::P1 * G::T + v;
  }
};

// One 1-D propagation of the lane's A-item, in place.  CONJ: the conjugate
// table.
template <class G, bool CONJ>
__device__ __forceinline__ void sep_prop(typename G::Elem* buf, const float2* tab, const float2* __restrict__ gtab,
                                         const SepLane<G>& ln, float2 (&x)[G::N1]) {
  using IT = typename G::IT;
  using QI = typename G::QI;
  constexpr int N1 = G::N1;
  constexpr int N2 = G::N2;
  constexpr int IBW = G::IBW;
  constexpr int Q = QI::Q;
  auto chirp = [&](int k1, int k2) -> float2 {
    if constexpr (G::TAB_LDS) {
      return tab[k1 * G::P1 + k2];
    } else {
      return ld(gtab, (unsigned)(k1 + N1 * k2));
    }
  };
  auto times = [](float2 u, float2 h) { return CONJ ? cmulc(u, h) : cmul(u, h); };
  const int s = opaque<IT>(ln.s);
  auto has = [&](auto ic) { return G::REPEAT || N2 * (ic.value + 1) <= N1 || IT::item(s, ic.value); };
  auto item = [&](auto ic) { return IT::template item_of<G::REPEAT>(s, ic.value); };
  // quad split: lane q of item (vector qv, k1 = qk) holds elements (Q*q + 4*m) mod N2
  int q = 0, qk = 0, qb = 0;
  if constexpr (QI::ON) {
    const int t = opaque<IT>(ln.quad);
    q = t & 3;
    const int qi = t >> 2;
    const int qv = G::ROWS ? qi / Q : qi % G::T;
    qk = N2 * (G::IB - 1) + (G::ROWS ? qi - qv * Q : qi / G::T);
    qb = G::ROWS ? qv * G::PR + qk * G::P1 : qk * G::P1 * G::T + qv;
  }
  auto qe = [&](auto m) {
    const int e = Q * q + 4 * decltype(m)::value;
    return e >= N2 ? e - N2 : e;
  };

  Dft<N1, -1>::run(x);
  phase<IT>();
  float2 y[IBW][N2];
  float2 z[G::Z];
  // (a barrier after the last read where lanes repeat an item: they read
  // entries another lane rewrites next)
  constexpr bool GUARD = (G::REPEAT && G::PARTIAL) || G::SPARE;
  if constexpr (G::SPLIT) {
    static_for<0, 2>([&](auto c) {
      static_for<0, N1>([&](auto k) { buf[ln.ab + G::SA * k.value] = c.value ? x[k.value].y : x[k.value].x; });
      exchange_sync<G::P>();
      static_for<0, IBW>([&](auto ic) {
        if (!has(ic)) return;
        const int b = ln.b_base(item(ic));
        static_for<0, N2>([&](auto e) {
          const float f = buf[b + G::SQ * e.value];
          if constexpr (c.value) y[ic.value][e.value].y = f; else y[ic.value][e.value].x = f;
        });
      });
      if constexpr (QI::ON) {
        static_for<0, Q>([&](auto m) {
          const float f = buf[qb + G::SQ * qe(m)];
          if constexpr (c.value) z[m.value].y = f; else z[m.value].x = f;
        });
      }
      if constexpr (c.value == 0 || GUARD) exchange_sync<G::P>();
    });
  } else {
    static_for<0, N1>([&](auto k) { buf[ln.ab + G::SA * k.value] = x[k.value]; });
    exchange_sync<G::P>();
    static_for<0, IBW>([&](auto ic) {
      if (!has(ic)) return;
      const int b = ln.b_base(item(ic));
      static_for<0, N2>([&](auto e) { y[ic.value][e.value] = buf[b + G::SQ * e.value]; });
    });
    if constexpr (QI::ON) static_for<0, Q>([&](auto m) { z[m.value] = buf[qb + G::SQ * qe(m)]; });
    if constexpr (GUARD) exchange_sync<G::P>();
  }
  phase<IT>();
  static_for<0, IBW>([&](auto ic) {
    if (!has(ic)) return;
    const int k1 = item(ic);
    float2(&u)[N2] = y[ic.value];
    item_forward<IT>(k1, u);
    static_for<0, N2>([&](auto k2) {
      u[k2.value] = times(u[k2.value], chirp(k1, k2.value));
      if constexpr (k2.value % 8 == 7) phase<IT>();
    });
    phase<IT>();
    item_inverse<IT>(k1, u);
  });
  if constexpr (QI::ON) {
    const float s1 = (q & 1) ? -1.f : 1.f;
    const float s2 = (q & 2) ? -1.f : 1.f;
    const bool l3 = q == 3;
    static_for<0, Q>([&](auto m) { z[m.value] = cmul(z[m.value], root_at<G::N>((unsigned)(qk * qe(m)))); });
    Dft<Q, -1>::run(z);
    quad_butterfly<2, Q>(z, s2);
    static_for<0, Q>([&](auto m) {
      const float2 u = z[m.value];
      z[m.value] = l3 ? c2(u.y, -u.x) : u;
    });
    quad_butterfly<1, Q>(z, s1);
    const int k4 = ((q & 1) << 1) | (q >> 1);
    static_for<0, Q>([&](auto m) {
      const int f = (QI::E1 * k4 + QI::E2 * decltype(m)::value) % N2;
      z[m.value] = times(z[m.value], chirp(qk, f));
    });
    quad_butterfly<1, Q>(z, s1);
    static_for<0, Q>([&](auto m) {
      const float2 u = z[m.value];
      z[m.value] = l3 ? c2(-u.y, u.x) : u;
    });
    quad_butterfly<2, Q>(z, s2);
    Dft<Q, 1>::run(z);
    static_for<0, Q>([&](auto m) { z[m.value] = cmul(z[m.value], root_at<G::N>((unsigned)(G::N - qk * qe(m)))); });
    phase<IT>();
  }
  if constexpr (G::SPLIT) {
    static_for<0, 2>([&](auto c) {
      static_for<0, IBW>([&](auto ic) {
        if (!has(ic)) return;
        const int b = ln.b_base(item(ic));
        static_for<0, N2>([&](auto e) {
          buf[b + G::SQ * e.value] = c.value ? y[ic.value][e.value].y : y[ic.value][e.value].x;
        });
      });
      if constexpr (QI::ON) {
        static_for<0, Q>([&](auto m) { buf[qb + G::SQ * qe(m)] = c.value ? z[m.value].y : z[m.value].x; });
      }
      exchange_sync<G::P>();
      static_for<0, N1>([&](auto k) {
        const float f = buf[ln.ab + G::SA * k.value];
        if constexpr (c.value) x[k.value].y = f; else x[k.value].x = f;
      });
      if constexpr (c.value == 0) exchange_sync<G::P>();
    });
  } else {
    static_for<0, IBW>([&](auto ic) {
      if (!has(ic)) return;
      const int b = ln.b_base(item(ic));
      static_for<0, N2>([&](auto e) { buf[b + G::SQ * e.value] = y[ic.value][e.value]; });
    });
    if constexpr (QI::ON) static_for<0, Q>([&](auto m) { buf[qb + G::SQ * qe(m)] = z[m.value]; });
    exchange_sync<G::P>();
    static_for<0, N1>([&](auto k) { x[k.value] = buf[ln.ab + G::SA * k.value]; });
  }
  phase<IT>();
  Dft<N1, 1>::run(x);
  phase<IT>();
}

// Chirp into shared memory in B-item order (visible after the next barrier).
template <class G>
__device__ __forceinline__ void sep_stage(float2* tab, const float2* __restrict__ gtab) {
  if constexpr (G::TAB_LDS) {
    for (int i = (int)threadIdx.x; i < G::N; i += G::P) {
      const int k1 = i / G::N2;
      const int k2 = i - k1 * G::N2;
      tab[k1 * G::P1 + k2] = gtab[G::PL::freq(k1, k2)];
    }
  }
}

// ---------------------------------------------------------------------------
// Layer passes (kFwdMid, kBwdMid, kBwdLast) on either axis and the first pass
// (kPropOnce, rows): schedule and arguments as fresnel_pass.  Modulation
// tables and dphi partials lie as the fields do ([y][x] slots).
// ---------------------------------------------------------------------------
// Waves per SIMD asked of the compiler: four (128 registers) for the forward
// kinds, two (256) for the adjoint kinds, which hold two fields, the next
// sample's input and the accumulators.
template <int KIND>
constexpr int sep_waves() { return KIND == kBwdMid || KIND == kBwdLast ? 2 : 4; }

template <class G, int KIND>
__global__ void __launch_bounds__(G::P, sep_waves<KIND>()) sep_pass(PassArgs a) {
  using IT = typename G::IT;
  using PL = typename G::PL;
  constexpr int N = G::N;
  constexpr int N1 = G::N1;
  constexpr int N2 = G::N2;
  constexpr bool ROWS = G::ROWS;
  constexpr bool ACC = KIND == kBwdMid || KIND == kBwdLast;
  constexpr int POL = field_load_policy<N>();
  constexpr int STEP = ROWS ? N2 : N2 * N;  // stored distance of consecutive A-item elements
  static_assert(KIND == kFwdMid || ACC || (KIND == kPropOnce && ROWS), "layer kinds, and the first row pass");
  __shared__ typename G::Elem buf[G::BUF];
  __shared__ float2 tab[G::TAB];

  // columns: XCD-contiguous ranks share lines in one L2; rows: dispatch order,
  // or the tile-major persistent order at 1000 points (as fresnel_pass)
  const int G8 = (int)gridDim.x;
  const int l = (int)blockIdx.x;
  const int rank = ACC && ROWS && N == 1000 ? persistent_rank(l, G8, a.ntiles, a.lanes)
                   : ROWS                   ? l
                                            : (l & 7) * (G8 >> 3) + (l >> 3);
  if (rank >= a.workers) return;
  const SepLane<G> ln;
  const size_t nn = (size_t)N * N;
  const int total = a.ntiles * a.batch;
  sep_stage<G>(tab, a.tab);
  if constexpr (G::TAB_LDS) exchange_sync<G::P>();

  float acc[ACC ? N1 : 1];
  if constexpr (ACC) {
    static_for<0, N1>([&](auto k) { acc[k.value] = 0.f; });
  }
  // elements at which G can be nonzero (layer L of a region loss, column passes)
  unsigned gmask = ~0u;
  if constexpr (ACC && !ROWS) {
    if (a.live) {
      gmask = 0u;
      static_for<0, N1>([&](auto k) {
        if (ln.act && ld(a.live, PL::pos_of_slot(ln.j + N2 * k.value)) != 0ull) gmask |= 1u << k.value;
      });
    }
  }
  // stored offset of this lane's A-item, in es-byte elements
  auto base = [&](int vec, bool ok, int es) -> unsigned {
    const int j = opaque<IT>(ln.j);
    return ok ? (unsigned)(ROWS ? vec * N + j : j * N + vec) * (unsigned)es : kOutOfRange;
  };
  auto load = [&](const float2* p, unsigned o, unsigned mask, float2(&x)[N1]) {
    const Rsrc r = make_rsrc(p, (unsigned)nn * 8u);
    static_for<0, N1>([&](auto k) {
      x[k.value] = bload_so<POL>(r, ((mask >> k.value) & 1u) ? o : kOutOfRange, STEP * 8 * k.value);
    });
  };

  // (accumulating kinds with the registers for it) W_{l-1} of the next item, in
  // flight while the current one is finished
  constexpr bool PREFETCH = ACC && !G::SPLIT;
  float2 pf[PREFETCH ? N1 : 1];
  auto prefetch = [&](int it, bool more) {
    if constexpr (PREFETCH) {
      phase<IT>();
      const int vec = (it % a.ntiles) * G::T + ln.v;
      load(a.act_in + (size_t)(it / a.ntiles) * nn, base(vec, more && vec < a.nvec && (!G::SPARE || ln.act), 8), ~0u, pf);
      phase<IT>();
    }
  };
  auto item = [&](int it) {
    const int tile = it % a.ntiles;
    const int b = it / a.ntiles;
    const int vec = tile * G::T + ln.v;
    const bool vok = vec < a.nvec && (!G::SPARE || ln.act);
    const float2* in = static_cast<const float2*>(a.in) + (size_t)b * nn;
    const unsigned o = base(vec, vok, 8);
    float2 x[N1];
    if constexpr (ACC) {
      // A_l from the saved input of the forward pass; the adjoint of the
      // first-axis half of hop l+1 of G
      float2 ar[N1];
      if constexpr (PREFETCH) {
        static_for<0, N1>([&](auto k) { ar[k.value] = pf[k.value]; });
        load(in, o, gmask, x);
        phase<IT>();
        sep_prop<G, false>(buf, tab, a.tab, ln, ar);
      } else {
        load(a.act_in + (size_t)b * nn, o, ~0u, ar);
        sep_prop<G, false>(buf, tab, a.tab, ln, ar);
        load(in, base(vec, vok, 8), gmask, x);
      }
      // h = conj(M_l) G_l and dphi_l += Im(conj(A_l) h)
      const Rsrc rm = make_rsrc(a.mod, (unsigned)nn * 8u);
      const unsigned om = base(vec, vok, 8);
      float2 m[PREFETCH ? N1 : 1];
      if constexpr (PREFETCH) {
        static_for<0, N1>([&](auto k) { m[k.value] = bload_keep_so(rm, om, STEP * 8 * k.value); });
      }
      phase<IT>();
      sep_prop<G, true>(buf, tab, a.tab, ln, x);
      static_for<0, N1>([&](auto k) {
        float2 w;
        if constexpr (PREFETCH) w = m[k.value]; else w = bload_keep_so(rm, om, STEP * 8 * k.value);
        const float2 h = cmulc(x[k.value], w);
        acc[k.value] += ar[k.value].x * h.y - ar[k.value].y * h.x;
        x[k.value] = h;
        if constexpr (!PREFETCH && k.value % 8 == 7) phase<IT>();
      });
      phase<IT>();
      const int next = it + a.workers;
      prefetch(next < total ? next : it, next < total);
      if constexpr (KIND == kBwdMid) sep_prop<G, true>(buf, tab, a.tab, ln, x);
    } else if constexpr (KIND == kFwdMid) {
      load(in, o, ~0u, x);
      sep_prop<G, false>(buf, tab, a.tab, ln, x);
      const Rsrc rm = make_rsrc(a.mod, (unsigned)nn * 8u);
      const unsigned om = base(vec, vok, 8);
      static_for<0, N1>([&](auto k) {
        x[k.value] = cmul(x[k.value], bload_keep_so(rm, om, STEP * 8 * k.value));
        if constexpr (k.value % 8 == 7) phase<IT>();
      });
      sep_prop<G, false>(buf, tab, a.tab, ln, x);
    } else {
      // natural amplitudes: stored row vec is natural row pos_of_slot(vec);
      // along it, slot order is natural for a Cooley-Tukey plan, else the row
      // goes through the exchange buffer (at most N <= PR floats a row)
      const Rsrc r = make_rsrc(static_cast<const float*>(a.in) + (size_t)b * nn, (unsigned)nn * 4u);
      const unsigned on = vok ? (unsigned)(PL::pos_of_slot(vec) * N + ln.j) * 4u : kOutOfRange;
      static_assert(G::SPLIT, "rows are staged through a float buffer");
      float f[N1];
      static_for<0, N1>([&](auto k) {
        f[k.value] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)on, N2 * 4 * k.value, POL));
      });
      if constexpr (PL::PFA) {
        float* const row = buf + ln.v * G::PR;
        static_for<0, N1>([&](auto k) { row[ln.j + N2 * k.value] = f[k.value]; });
        exchange_sync<G::P>();
        const int p0 = PL::pos_base(ln.j);
        static_for<0, N1>([&](auto k) { f[k.value] = row[PL::pos_at(p0, k.value)]; });
        exchange_sync<G::P>();
      }
      static_for<0, N1>([&](auto k) { x[k.value] = c2(f[k.value], 0.f); });
      sep_prop<G, false>(buf, tab, a.tab, ln, x);
    }
    if constexpr (KIND != kBwdLast) {
      const Rsrc ro = make_rsrc(a.out + (size_t)b * nn, (unsigned)nn * 8u);
      const unsigned os = base(vec, vok && ln.act, 8);
      static_for<0, N1>([&](auto k) { bstore_so(ro, os, STEP * 8 * k.value, x[k.value]); });
    }
  };
  if constexpr (ACC) {
    if (rank < total) prefetch(rank, true);
    for (int it = rank; it < total; it += a.workers) item(it);
    // one partial per lane of workgroups (the tile is fixed)
    const int vec = (rank % a.ntiles) * G::T + ln.v;
    const unsigned o = base(vec, ln.act && vec < a.nvec, 4);
    const Rsrc dp = make_rsrc(a.dphi_part + (size_t)(rank / a.ntiles) * nn, (unsigned)nn * 4u);
    static_for<0, N1>([&](auto k) { bstore_f_so(dp, o, STEP * 4 * k.value, acc[k.value]); });
  } else {
    if (rank < total) item(rank);
  }
}

// ---------------------------------------------------------------------------
// Detector-plane row passes (kFwdLast, kBwdFirst): as detector_pass.  Natural
// rows (gradient, skip field, outputs) move through the exchange buffer one
// component at a time where slot order is not natural.
// ---------------------------------------------------------------------------
template <class G, int KIND>
__global__ void __launch_bounds__(G::P, sep_waves<kFwdMid>()) sep_detector_pass(PassArgs a) {
  using IT = typename G::IT;
  using PL = typename G::PL;
  constexpr int N = G::N;
  constexpr int N1 = G::N1;
  constexpr int N2 = G::N2;
  constexpr int R = G::T;
  constexpr int POL = field_load_policy<N>();
  static_assert(G::ROWS && (KIND == kFwdLast || KIND == kBwdFirst), "detector-plane row passes");
  static_assert(!G::SPARE || !PL::PFA, "spare lanes hold no row values to stage");
  __shared__ float buf[G::BUF];
  __shared__ float2 tab[G::TAB];
  __shared__ float rsum[KIND == kFwdLast ? R * kMaxRegions : 1];

  const int tile = (int)blockIdx.x % a.ntiles;
  const int b = (int)blockIdx.x / a.ntiles;
  if (b >= a.batch) return;
  const SepLane<G> ln;
  const int tid = (int)threadIdx.x;
  const size_t nn = (size_t)N * N;
  sep_stage<G>(tab, a.tab);
  if constexpr (G::TAB_LDS) exchange_sync<G::P>();

  // stored row of tile row i: the covered-first permutation, or consecutive
  const int nrows = a.vperm ? a.nact : N;
  auto stored = [&](int i) { return i < nrows ? (a.vperm ? a.vperm[i] : i) : 0; };
  const bool vok = tile * R + ln.v < nrows && (!G::SPARE || ln.act);
  const int vec = stored(tile * R + ln.v);
  const int y = PL::pos_of_slot(vec);  // natural row
  float* const row = buf + ln.v * G::PR;
  // byte offsets in a natural array: this lane's coalesced run q = j + N2*m of
  // row y (consecutive lanes, consecutive pixels)
  auto nat = [&](bool ok, int es) -> unsigned { return ok ? (unsigned)((y * N + opaque<IT>(ln.j)) * es) : kOutOfRange; };
  // A-item order <-> the lane's natural run
  auto to_items = [&](float(&f)[N1]) {
    if constexpr (PL::PFA) {
      exchange_sync<G::P>();
      static_for<0, N1>([&](auto m) { row[ln.j + N2 * m.value] = f[m.value]; });
      exchange_sync<G::P>();
      const int p0 = PL::pos_base(opaque<IT>(ln.j));
      static_for<0, N1>([&](auto k) { f[k.value] = row[PL::pos_at(p0, k.value)]; });
      exchange_sync<G::P>();
    }
  };
  auto to_run = [&](float(&f)[N1]) {
    if constexpr (PL::PFA) {
      exchange_sync<G::P>();
      const int p0 = PL::pos_base(opaque<IT>(ln.j));
      static_for<0, N1>([&](auto k) { row[PL::pos_at(p0, k.value)] = f[k.value]; });
      exchange_sync<G::P>();
      static_for<0, N1>([&](auto m) { f[m.value] = row[ln.j + N2 * m.value]; });
    }
  };

  float2 x[N1];
  {
    const Rsrc rin = make_rsrc(static_cast<const float2*>(a.in) + (size_t)b * nn, (unsigned)nn * 8u);
    const unsigned o = vok ? (unsigned)(vec * N + ln.j) * 8u : kOutOfRange;
    static_for<0, N1>([&](auto k) { x[k.value] = bload_so<POL>(rin, o, N2 * 8 * k.value); });
  }
  // rest of the last hop: U_D
  sep_prop<G, false>(buf, tab, a.tab, ln, x);
  if (a.skip) {
    const Rsrc rs = make_rsrc(a.skip + (size_t)b * nn, (unsigned)nn * 8u);
    const unsigned o = nat(vok, 8);
    static_for<0, 2>([&](auto c) {
      float f[N1];
      static_for<0, N1>([&](auto m) { f[m.value] = bload_f_so(rs, o, N2 * 8 * m.value + 4 * c.value); });
      to_items(f);
      static_for<0, N1>([&](auto k) {
        if constexpr (c.value) x[k.value].y += f[k.value]; else x[k.value].x += f[k.value];
      });
    });
  }

  if constexpr (KIND == kBwdFirst) {
    // seed G_D = 2 (dL/dI) U_D
    if (a.grad_int) {
      const Rsrc rg = make_rsrc(a.grad_int + (size_t)b * nn, (unsigned)nn * 4u);
      const unsigned o = nat(vok, 4);
      float f[N1];
      static_for<0, N1>([&](auto m) { f[m.value] = bload_f_so(rg, o, N2 * 4 * m.value); });
      to_items(f);
      static_for<0, N1>([&](auto k) { x[k.value] = cscale(x[k.value], 2.f * f[k.value]); });
    } else {
      // dL/dI is dL/dS_k on region k: sum over the regions covering the pixel
      const float* __restrict__ gs = a.grad_sums + (size_t)b * a.K;
      const unsigned long long vmask = vok ? ld(a.row_mask, y) : 0ull;
      const int p0 = PL::pos_base(ln.j);
      static_for<0, N1>([&](auto k) {
        float g = 0.f;
        if (vmask) {
          unsigned long long m = vmask & ld(a.col_mask, PL::pos_at(p0, k.value));
          while (m) {
            g += gs[__builtin_ctzll(m)];
            m &= m - 1;
          }
        }
        x[k.value] = cscale(x[k.value], 2.f * g);
      });
    }
    phase<IT>();
    sep_prop<G, true>(buf, tab, a.tab, ln, x);
    const Rsrc ro = make_rsrc(a.out + (size_t)b * nn, (unsigned)nn * 8u);
    const unsigned o = vok && ln.act ? (unsigned)(vec * N + ln.j) * 8u : kOutOfRange;
    static_for<0, N1>([&](auto k) { bstore_so(ro, o, N2 * 8 * k.value, x[k.value]); });
  } else {
    if (a.field_out) {
      const Rsrc ro = make_rsrc(a.field_out + (size_t)b * nn, (unsigned)nn * 8u);
      float re[N1];
      float im[N1];
      static_for<0, N1>([&](auto k) { re[k.value] = x[k.value].x; });
      to_run(re);
      static_for<0, N1>([&](auto k) { im[k.value] = x[k.value].y; });
      to_run(im);
      const unsigned o = nat(vok && ln.act, 8);
      static_for<0, N1>([&](auto m) { bstore_so(ro, o, N2 * 8 * m.value, c2(re[m.value], im[m.value])); });
    }
    float f[N1];
    static_for<0, N1>([&](auto k) { f[k.value] = cabs2(x[k.value]); });
    to_run(f);
    if (a.intensity) {
      const Rsrc ro = make_rsrc(a.intensity + (size_t)b * nn, (unsigned)nn * 4u);
      const unsigned o = nat(vok && ln.act, 4);
      if (a.accumulate) {
        static_for<0, N1>([&](auto m) { bstore_f_so(ro, o, N2 * 4 * m.value, f[m.value] + bload_f_so(ro, o, N2 * 4 * m.value)); });
      } else {
        static_for<0, N1>([&](auto m) { bstore_f_so(ro, o, N2 * 4 * m.value, f[m.value]); });
      }
    }
    if (a.sums_part) {
      // one run per (region, row) over the natural row in shared memory, the
      // rows added in order
      exchange_sync<G::P>();
      if (!G::SPARE || ln.act) static_for<0, N1>([&](auto m) { row[ln.j + N2 * m.value] = f[m.value]; });
      exchange_sync<G::P>();
      const int K = a.K;
      const int side = a.det_size;
      for (int i = tid; i < K * R; i += G::P) {
        const int k = i / R;
        const int rr = i - k * R;
        const int2 c = a.regions[k];  // (y0, x0)
        float run = 0.f;
        if (tile * R + rr < nrows && (unsigned)(PL::pos_of_slot(stored(tile * R + rr)) - c.x) < (unsigned)side) {
          for (int d = 0; d < side; ++d) run += buf[rr * G::PR + c.y + d];
        }
        rsum[i] = run;
      }
      exchange_sync<G::P>();
      for (int k = tid; k < K; k += G::P) {
        float part = 0.f;
        for (int rr = 0; rr < R; ++rr) part += rsum[k * R + rr];
        a.sums_part[((size_t)b * a.ntiles + tile) * K + k] = part;
      }
    }
  }
}

}  // namespace lr
