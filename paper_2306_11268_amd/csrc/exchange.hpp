// The exchange between the two register steps of a transform, for the passes
// that keep a lane's items in registers (as_impl.hpp, sep_impl.hpp): lane slot
// s of a vector holds A-item s (N1 values) and, on the other side, the B-items
// s, s + N2, ... (N2 values each).
#pragma once

#include "tile.hpp"

namespace lr {

// Barrier between shared-memory phases of a workgroup of P threads.  One wave
// needs no hardware barrier and no wait: its shared-memory accesses complete
// in order, so only the compiler has to keep them in order.
template <int P>
__device__ __forceinline__ void exchange_sync() {
  if constexpr (P == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  } else {
    __syncthreads();
  }
}

// Rounds of B-items per lane (item k1 = s + N2*ic in round ic).
template <class PL, bool FENCED = false>
struct Items {
  using Plan = PL;
  static constexpr int N = PL::N;
  static constexpr int N1 = PL::N1;
  static constexpr int N2 = PL::N2;
  static constexpr int IB = (N1 + N2 - 1) / N2;
  static constexpr bool FULL_ROUNDS = N1 % N2 == 0;
  static constexpr int P1 = N2 + 1;  // exchange pitch of a B-item
  static constexpr bool LONG = FENCED || N1 > 16 || N2 * IB > 16;
  static_assert(N2 % 2 == 0, "odd exchange pitch");
  // Whether lane s has an item in round ic, and the item it works on: row
  // passes (REPEAT) let a lane past the last item repeat one of that round's
  // items, the same values from and to the same shared-memory entries, because
  // a branch around the item kept the compiler from scheduling the arrays live
  // across it (100-400 bytes of scratch); column passes, where whole waves are
  // past the last item, branch (500 points: 54 us against 106 with repeats).
  static __device__ __forceinline__ bool item(int s, int ic) { return FULL_ROUNDS || s + N2 * ic < N1; }
  template <bool REPEAT>
  static __device__ __forceinline__ int item_of(int s, int ic) {
    constexpr int last = N1 - N2 * (IB - 1);  // items of the last round
    return N2 * ic + (!REPEAT || FULL_ROUNDS || ic + 1 < IB ? s : s % last);
  }
};

// Exchange of one vector's A-item (x) with its B-items (y).  The A side of
// element k1 is buf[ab + SA*k1], the B side of element q of round ic
// buf[bb[ic] + SQ*q].  A to_vector after a to_items, and the other way round,
// rewrites only entries that the same lane read last and needs no barrier
// between them.  A to_vector after a to_vector writes entries that other lanes
// read on their A side: the first of them is called with AGAIN, which ends it
// with a barrier.  SPLIT: one component
// at a time through a float buffer (half the shared memory, three times the
// barriers), else a float2 buffer.  s: the lane's slot (B-items).
// SPARE: the workgroup has lanes that repeat item 0.
template <class IT, int P, bool SPLIT, bool REPEAT, bool SPARE, int SA, int SQ>
struct Exchange {
  using Elem = std::conditional_t<SPLIT, float, float2>;
  static constexpr int N1 = IT::N1;
  static constexpr int N2 = IT::N2;
  static constexpr int IB = IT::IB;
  static __device__ __forceinline__ bool has(int s, int ic) { return REPEAT || IT::item(s, ic); }
  static __device__ __forceinline__ void to_items(Elem* buf, int s, int ab, const int (&bb)[IB], const float2 (&x)[N1],
                                                  float2 (&y)[IB][N2]) {
    if constexpr (SPLIT) {
      static_for<0, 2>([&](auto c) {
        static_for<0, N1>([&](auto k) { buf[ab + SA * k.value] = c.value ? x[k.value].y : x[k.value].x; });
        exchange_sync<P>();
        static_for<0, IB>([&](auto ic) {
          if (!has(s, ic.value)) return;
          static_for<0, N2>([&](auto q) {
            const float v = buf[bb[ic.value] + SQ * q.value];
            if constexpr (c.value) y[ic.value][q.value].y = v; else y[ic.value][q.value].x = v;
          });
        });
        if constexpr (c.value == 0) exchange_sync<P>();
      });
    } else {
      static_for<0, N1>([&](auto k) { buf[ab + SA * k.value] = x[k.value]; });
      exchange_sync<P>();
      static_for<0, IB>([&](auto ic) {
        if (!has(s, ic.value)) return;
        static_for<0, N2>([&](auto q) { y[ic.value][q.value] = buf[bb[ic.value] + SQ * q.value]; });
      });
    }
    // lanes that repeat an item read entries another lane rewrites next
    if constexpr ((REPEAT && !IT::FULL_ROUNDS) || SPARE) exchange_sync<P>();
  }
  template <bool AGAIN = false>
  static __device__ __forceinline__ void to_vector(Elem* buf, int s, int ab, const int (&bb)[IB], const float2 (&y)[IB][N2],
                                                   float2 (&x)[N1]) {
    if constexpr (SPLIT) {
      static_for<0, 2>([&](auto c) {
        static_for<0, IB>([&](auto ic) {
          if (!has(s, ic.value)) return;
          static_for<0, N2>([&](auto q) {
            buf[bb[ic.value] + SQ * q.value] = c.value ? y[ic.value][q.value].y : y[ic.value][q.value].x;
          });
        });
        exchange_sync<P>();
        static_for<0, N1>([&](auto k) {
          const float v = buf[ab + SA * k.value];
          if constexpr (c.value) x[k.value].y = v; else x[k.value].x = v;
        });
        if constexpr (c.value == 0) exchange_sync<P>();
      });
    } else {
      static_for<0, IB>([&](auto ic) {
        if (!has(s, ic.value)) return;
        static_for<0, N2>([&](auto q) { buf[bb[ic.value] + SQ * q.value] = y[ic.value][q.value]; });
      });
      exchange_sync<P>();
      static_for<0, N1>([&](auto k) { x[k.value] = buf[ab + SA * k.value]; });
    }
    if constexpr (AGAIN) exchange_sync<P>();
  }
};

// Long items (more than 16 values of a vector or of its items per lane): an
// index goes through an empty asm statement, so that roots and addresses
// derived from it are formed next to their use, not hoisted and kept live, and
// scheduling barriers between the phases of a pass do the same for loads.
// Short items have the registers, and their root and table loads are better
// in flight early (64 points: column pass 14.7 -> 13.6 us); in the persistent
// kinds (FENCED) they too would be kept live across the samples (256 points,
// adjoint row pass 46 -> 60 us).
template <class IT>
__device__ __forceinline__ int opaque(int v) {
  if constexpr (IT::LONG) asm volatile("" : "+v"(v));
  return v;
}
template <class IT>
__device__ __forceinline__ void phase() {
  if constexpr (IT::LONG) __builtin_amdgcn_sched_barrier(0);
}

// Cooley-Tukey twiddles exp(-2*pi*i*k1*j/N) in pairs (j, j + 1) by item:
// consecutive lanes (items k1) read consecutive 16-byte entries, N2/2 loads a
// B-item, each root rounded once.  Read one by one out of the table of N
// roots (entry k1*j: a gather, N2 - 1 loads) they held the passes up: every
// load waits behind the field loads in flight (500 points, 200 samples:
// forward row pass 306 -> 280 us, adjoint column pass 620 -> 550).
template <class PL>
struct RootPairs {
  float4 w[PL::N2 / 2 * PL::N1];
};
// factor: of every entry, the exact ones included.
template <class PL>
constexpr RootPairs<PL> make_root_pairs(double factor) {
  RootPairs<PL> t{};
  for (int p = 0; p < PL::N2 / 2; ++p)
    for (int k1 = 0; k1 < PL::N1; ++k1) {
      const cdbl a = unit_root(static_cast<long long>(k1) * (2 * p), PL::N, -1);
      const cdbl b = unit_root(static_cast<long long>(k1) * (2 * p + 1), PL::N, -1);
      float4& e = t.w[p * PL::N1 + k1];
      const double ga = factor * (k1 * p == 0 ? 1.0 : root_gain<PL::N>());
      const double gb = factor * (k1 == 0 ? 1.0 : root_gain<PL::N>());
      e.x = static_cast<float>(ga * a.re);
      e.y = static_cast<float>(ga * a.im);
      e.z = static_cast<float>(gb * b.re);
      e.w = static_cast<float>(gb * b.im);
    }
  return t;
}
template <class PL>
struct ItemRoots {
  static constexpr RootPairs<PL> table = make_root_pairs<PL>(1.0);
};
// The same over N^2, for the inverse transform of a hop: its factor then costs no
// rounding of its own (and N1 products a lane less than on the output).  Where
// 1/N^2 is a float there is nothing to gain, and plans without a table scale
// the output.  The factor also takes out the mean gain of the hop's four
// transforms (root_gain): 2.8e-8 at 100, 200 and 400 points, 5.2e-8 with half
// transforms at 400, 2.4e-8 at 500.
template <class PL, bool HALF>
struct ScaledRoots {
  static constexpr bool ON = !PL::PFA && PL::N2 < 32 && (PL::N & (PL::N - 1)) != 0;
  static constexpr double gain = PL::N == 500 ? 2.4e-8 : HALF ? 5.2e-8 : 2.8e-8;
  static constexpr double factor = (1.0 - gain) / ((double)PL::N * PL::N);
  static constexpr RootPairs<PL> table = make_root_pairs<PL>(factor);
};
// Multiply a B-item by its twiddles (INV: their conjugates), eight values at a
// time so that the roots are not all live at once.  Items of 32 or more values
// take the products w^(k1*j) = w^(k1*(j mod 8)) * w^(8*k1*(j/8)) instead: 7 +
// N2/8 - 1 loads, one more rounding (<= 1.5 ulp) (1000 points: column pass 133
// against 155 us; 1024: row pass 93 against 96).
// Roots: the table, ItemRoots or ScaledRoots.
template <class IT, bool INV, class Table = ItemRoots<typename IT::Plan>>
__device__ __forceinline__ void item_twiddle(int k1, float2 (&y)[IT::N2]) {
  using PL = typename IT::Plan;
  constexpr int N2 = IT::N2;
  constexpr bool SCALED = !std::is_same_v<Table, ItemRoots<PL>>;
  static_assert(!SCALED || N2 < 32, "long items have no scaled table");
  if constexpr (N2 >= 32) {
    auto root = [&](int m) { return root_at<IT::N>(INV ? (unsigned)(IT::N - k1 * m) : (unsigned)(k1 * m)); };
    float2 lo[8];
    static_for<1, 8>([&](auto i) { lo[i.value] = root(i.value); });
    static_for<0, N2 / 8>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if constexpr (b == 0) {
        static_for<1, 8>([&](auto i) { y[i.value] = cmul(y[i.value], lo[i.value]); });
      } else {
        const float2 hi = root(8 * b);
        y[8 * b] = cmul(y[8 * b], hi);
        static_for<1, 8>([&](auto i) { y[8 * b + i.value] = cmul(y[8 * b + i.value], cmul(lo[i.value], hi)); });
      }
      phase<IT>();
    });
  } else static_for<0, N2 / 2>([&](auto pc) {
    constexpr int p = decltype(pc)::value;
    const float4 w = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(Table::table.w) +
                                                      (unsigned)(p * IT::N1 + k1) * 16u);
    auto times = [](float2 u, float2 r) { return INV ? cmulc(u, r) : cmul(u, r); };
    if constexpr (p > 0) y[2 * p] = times(y[2 * p], c2(w.x, w.y));
    else if constexpr (SCALED) y[0] = cscale(y[0], static_cast<float>(Table::factor));
    y[2 * p + 1] = times(y[2 * p + 1], c2(w.z, w.w));
    if constexpr (p % 4 == 3) phase<IT>();
  });
}
template <class IT>
__device__ __forceinline__ void item_forward(int k1, float2 (&y)[IT::N2]) {
  if constexpr (!IT::Plan::PFA) {
    item_twiddle<IT, false>(opaque<IT>(k1), y);
    phase<IT>();
  }
  Dft<IT::N2, -1>::run(y);
  phase<IT>();
}
template <class IT, class Table = ItemRoots<typename IT::Plan>>
__device__ __forceinline__ void item_inverse(int k1, float2 (&y)[IT::N2]) {
  Dft<IT::N2, 1>::run(y);
  phase<IT>();
  if constexpr (!IT::Plan::PFA) {
    item_twiddle<IT, true, Table>(opaque<IT>(k1), y);
    phase<IT>();
  }
}

}  // namespace lr
