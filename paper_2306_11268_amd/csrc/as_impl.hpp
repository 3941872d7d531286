// Angular-spectrum passes (non-separable transfer functions) for gfx950.
//
// A hop is FFT_x of every row, then per column FFT_y, x H, IFFT_y, then IFFT_x
// of every row.  Between passes a sample is stored as n rows of N x-spectrum
// values in natural frequency order ([B][n][N]); only the n rows inside the
// aperture carry data.  With the Cooley-Tukey plans (AsPlanFor) positions and
// frequencies are natural, so a lane's elements lie at one per-lane base plus
// compile-time offsets in every array a pass touches, and no array is staged
// through shared memory (350 points: the last paragraph):
//
//   A-item j of a vector: positions j + N2*k, k < N1;
//   B-item k1: frequencies k1 + N1*k2, k2 < N2, and on its other side the
//     elements j < N2 it exchanges with the A-items.
//
// Shared memory holds only that exchange; for the longer plans one float
// component at a time (real parts, then imaginary parts): half the bytes of a
// complex tile, so twice the resident waves, which is what bounds these
// passes (the 1024-point column tile of complex values in both directions
// held 74 KB per 4 waves: 8 waves per CU).  Entry (k1, j) of a vector is at
// k1*(N2+1) + j (N2 is even), which spreads the B-side reads of a wave over all
// banks.
//
// Measured (10 layers, 512 in 1024, batch 64, one MI355X; before: tiles staged
// through shared memory): column pass 285 -> 156 us (2109 VALU instructions
// per lane, 132 us at the measured issue rate), row layer pass 175 -> 95 us
// (537 MB at 5.6 TB/s, the rate of a large copy), the network 5.08 -> 2.79 ms;
// 5 layers of training, 200 in 400, batch 100: 1.60 -> 0.98 ms.
//
// With a field zero padded to twice its size (HALF: n = N/2, N1 divisible by
// 4) a lane's elements inside the aperture are exactly k = N1/4 .. 3*N1/4 - 1:
// the A-step runs HalfDft, and half of the loads, stores and products vanish.
//
// 350 points keep their Good-Thomas plan: the twiddles of 25 x 14 added 7% to
// the rounding error of a transform (9.4e-8 -> 1.01e-7).  Rows then move as
// natural runs and take the plan's order through the exchange area; columns
// address their rows and table rows one by one.  5 layers, batch 64: 511 -> 475 us
// against 25 x 14 with twiddles (a single hop 101 -> 104).
#pragma once

#include "exchange.hpp"
#include "kernels_impl.hpp"

namespace lr {

template <class PL, bool FENCED = false>
struct AsItems : Items<PL, FENCED> {
  // frequency of element k2 of item k1: freq_at<k2>(freq_base(k1))
  static __device__ __forceinline__ int freq_base(int k1) { return PL::PFA ? k1 * PL::E1 % PL::N : k1; }
  template <int K2>
  static __device__ __forceinline__ int freq_at(int base) {
    if constexpr (PL::PFA) {
      const int f = base + K2 * PL::E2 % PL::N;
      return f >= PL::N ? f - PL::N : f;
    } else {
      return base + PL::N1 * K2;
    }
  }
  // elements of an A-item inside a half aperture (HALF), or all of them
  static constexpr int K0(bool half) { return half ? PL::N1 / 4 : 0; }
  static constexpr int KN(bool half) { return half ? PL::N1 / 2 : PL::N1; }
};

// A-step of the elements u[0..KN) a lane holds (HALF: the middle half).
template <class IT, bool HALF>
__device__ __forceinline__ void as_a_forward(const float2 (&u)[IT::KN(HALF)], float2 (&x)[IT::N1]) {
  if constexpr (HALF) {
    HalfDft<IT::N1>::forward(u, x);
  } else {
    static_for<0, IT::N1>([&](auto k) { x[k.value] = u[k.value]; });
    Dft<IT::N1, -1>::run(x);
  }
}
template <class IT, bool HALF>
__device__ __forceinline__ void as_a_inverse(float2 (&x)[IT::N1], float2 (&u)[IT::KN(HALF)]) {
  if constexpr (HALF) {
    HalfDft<IT::N1>::inverse(x, u);
  } else {
    Dft<IT::N1, 1>::run(x);
    static_for<0, IT::N1>([&](auto k) { u[k.value] = x[k.value]; });
  }
}

// ---------------------------------------------------------------------------
// Row passes.  A workgroup transforms R whole rows; lane (r, j), j < N2, holds
// A-item j of row r, consecutive lanes consecutive elements, so every access
// of a wave covers N2 consecutive values of R rows.  R*N2 is one wave where
// N2 allows (no barriers at all; 60 of 64 lanes at N2 = 10 and 20, 56 at 14),
// 6 rows in four waves (240 of 256 lanes) at N2 = 40.
// ---------------------------------------------------------------------------
template <class PL>
struct AsRows : AsItems<PL> {
  using IT = AsItems<PL>;
  static constexpr int R = (IT::N2 <= 32 ? 64 : 256) / IT::N2;
  static constexpr int P = (R * IT::N2 + 63) / 64 * 64;
  static constexpr bool SPARE = P != R * IT::N2 && P > 64;
  static_assert(!SPARE || !PL::PFA, "spare lanes hold no run of a row");
  // row pitch: at least the exchange area, and = N2 mod 64, so that the rows
  // of a wave tile the banks on the A side
  static constexpr int PR = IT::N1 * IT::P1 + (64 + IT::N2 - IT::N1 * IT::P1 % 64) % 64;
  // one component at a time where the complex buffer would keep fewer than
  // 16 waves resident per CU
  static constexpr bool SPLIT = R * PR * 8 > 10 * 1024 * (P / 64);
  // waves per SIMD asked of the compiler: 4 where a lane's items fit in 128
  // registers, one less for the 40-value items and for the accumulating kinds
  static constexpr int WAVES = IT::N2 * IT::IB > 32 ? 3 : 4;
  static constexpr int WAVES_ACC = WAVES - 1;
  // and two for the middle backward kind of the Good-Thomas plan: its reordered
  // items, the accumulators and a second transform do not fit in three waves'
  // 168 registers (350x350: 36 us at three, 24 at two with a batch of 16; 94
  // and 67 with 64). The last layer's kind has one transform and keeps three
  // (54 and 62 us with 64).
  static constexpr int WAVES_MID = PL::PFA ? 2 : WAVES_ACC;
  static_assert(R * PR * (SPLIT ? 4 : 8) + R * kMaxRegions * 4 < 64 * 1024, "static shared memory");
};

template <class PL, int KIND, bool HALF>
__global__ void __launch_bounds__(AsRows<PL>::P, KIND == kAsRowBwdMid    ? AsRows<PL>::WAVES_MID
                                                 : KIND == kAsRowBwdLast ? AsRows<PL>::WAVES_ACC
                                                                         : AsRows<PL>::WAVES)
    as_row_pass(PassArgs a) {
  using W = AsRows<PL>;
  using IT = AsItems<PL, KIND == kAsRowBwdMid || KIND == kAsRowBwdLast>;
  using EX = Exchange<IT, W::P, W::SPLIT, true, W::SPARE, W::P1, 1>;
  constexpr int N = W::N;
  constexpr int N1 = W::N1;
  constexpr int N2 = W::N2;
  constexpr int IB = W::IB;
  constexpr int R = W::R;
  constexpr int KN = W::KN(HALF);
  constexpr bool ACC = (KIND == kAsRowBwdMid || KIND == kAsRowBwdLast);
  constexpr bool SPECTRAL_IN = (KIND == kAsRowMid || KIND == kAsRowLast || KIND == kAsRowIfft || ACC);
  constexpr bool FWD_OUT = (KIND == kAsRowFirst || KIND == kAsRowMid || KIND == kAsRowBwdFirst ||
                            KIND == kAsRowBwdMid);
  __shared__ typename EX::Elem buf[R * W::PR];
  __shared__ float rsum[KIND == kAsRowLast ? R * kMaxRegions : 1];

  const int rank = (int)blockIdx.x;
  if (rank >= a.workers) return;
  const int tid = (int)threadIdx.x;
  // the lanes past the R rows store nothing: in a one-wave workgroup they repeat
  // the first items of row 0 (the same values to the same shared-memory
  // entries, no branch); else (SPARE) their A side is the exchange area's
  // padding column and on the B side they repeat item 0
  const bool act = R * N2 == W::P || tid < R * N2;
  const int r = act ? tid / N2 : 0;
  const int j0 = act ? tid - r * N2 : (W::SPARE ? N2 : tid - R * N2);
  const int s0 = W::SPARE && !act ? 0 : j0;
  const int n = a.n;
  const int off = a.off;
  const size_t nn = (size_t)n * n;
  const int total = a.ntiles * a.batch;
  const int ab = r * W::PR + j0;
  int bb[IB];
  static_for<0, IB>([&](auto ic) { bb[ic.value] = r * W::PR + W::P1 * IT::template item_of<true>(s0, ic.value); });

  float acc[ACC ? KN : 1];
  if constexpr (ACC) {
    static_for<0, KN>([&](auto k) { acc[k.value] = 0.f; });
  }

  auto item = [&](int it) {
    const int tile = it % a.ntiles;
    const int b = it / a.ntiles;
    const int j = opaque<IT>(j0);
    const int s = opaque<IT>(s0);
    const int vec = tile * R + r;
    const bool vok = vec < n && (!W::SPARE || act);
    auto pos_ok = [&](int jj, auto k) { return HALF || (unsigned)(jj + N2 * decltype(k)::value - off) < (unsigned)n; };
    // f(k, byte offset per lane, scalar byte offset) for the elements of this
    // lane's A-item in an n x n natural array of es-byte values; the per-lane
    // offset is out of range outside the aperture
    auto each_if = [&](bool ok, int es, auto&& f) {
      const int jj = opaque<IT>(j);
      const int row = vec * n + jj;  // HALF: element k is aperture position jj + N2*k
      if constexpr (HALF) {
        const unsigned base = ok ? (unsigned)(row * es) : kOutOfRange;
        static_for<0, KN>([&](auto k) { f(k, base, N2 * k.value * es); });
      } else {
        static_for<0, KN>([&](auto k) {
          f(k, ok && pos_ok(jj, k) ? (unsigned)((row + N2 * k.value - off) * es) : kOutOfRange, 0);
        });
      }
    };
    auto each = [&](int es, auto&& f) { each_if(vok, es, f); };
    auto each_out = [&](int es, auto&& f) { each_if(vok && act, es, f); };
    // spectrum element (round ic, k2) of this row: frequency k1 + N1*k2
    auto spec_base = [&](bool ok, int ic) -> unsigned {
      return ok ? (unsigned)(vec * N + IT::template item_of<true>(s, ic)) * 8u : kOutOfRange;
    };
    // Good-Thomas plans: arrays move as runs j + N2*m, m < N1, in natural order
    // (consecutive lanes, consecutive values) and take the plan's order through
    // the row's exchange area, one component at a time.
    [[maybe_unused]] auto reorder = [&](auto&& write, auto&& read) {
      if constexpr (PL::PFA) {
        float* const line = reinterpret_cast<float*>(buf) + r * W::PR;
        static_for<0, 2>([&](auto c) {
          exchange_sync<W::P>();
          write(c, line);
          exchange_sync<W::P>();
          read(c, line);
        });
        exchange_sync<W::P>();
      }
    };
    auto run_write = [&](float2* v) {
      return [v, j](auto c, float* line) {
        static_for<0, N1>([&](auto m) { line[j + N2 * m.value] = c.value ? v[m.value].y : v[m.value].x; });
      };
    };
    auto run_read = [&](float2* v) {
      return [v, j](auto c, float* line) {
        static_for<0, N1>([&](auto m) {
          const float f = line[j + N2 * m.value];
          if constexpr (c.value) v[m.value].y = f; else v[m.value].x = f;
        });
      };
    };
    // a run of positions into A-item order, and back
    auto to_item = [&](float2(&v)[KN]) {
      if constexpr (PL::PFA) {
        const int p0 = PL::pos_base(opaque<IT>(j));
        reorder(run_write(v), [&](auto c, float* line) {
          static_for<0, N1>([&](auto k) {
            const float f = line[PL::pos_at(p0, k.value)];
            if constexpr (c.value) v[k.value].y = f; else v[k.value].x = f;
          });
        });
      }
    };
    auto to_run = [&](float2(&v)[KN]) {
      if constexpr (PL::PFA) {
        const int p0 = PL::pos_base(opaque<IT>(j));
        reorder([&](auto c, float* line) {
          static_for<0, N1>([&](auto k) { line[PL::pos_at(p0, k.value)] = c.value ? v[k.value].y : v[k.value].x; });
        }, run_read(v));
      }
    };
    if constexpr (KIND == kAsRowLast) {
      // sums only: rows no region covers contribute nothing
      if (!a.intensity && !a.field_out && !a.saved_ud) {
        if (!a.sums_part) return;
        const bool hit = vok && a.row_mask[vec] != 0ull;
        bool any;
        if constexpr (W::P == 64) any = __any(hit) != 0; else any = __syncthreads_or(hit) != 0;
        if (!any) {
          for (int k = tid; k < a.K; k += W::P) a.sums_part[((size_t)b * a.ntiles + tile) * a.K + k] = 0.f;
          return;
        }
      }
    }

    float2 u[KN];
    if constexpr (SPECTRAL_IN) {
      const Rsrc rin = make_rsrc(static_cast<const float2*>(a.in) + (size_t)b * n * N, (unsigned)(n * N) * 8u);
      float2 y[IB][N2];
      if constexpr (PL::PFA) {
        float2 run[N1];
        const unsigned base = vec < n ? (unsigned)(vec * N + j) * 8u : kOutOfRange;
        static_for<0, N1>([&](auto m) { run[m.value] = bload_so<2>(rin, base, N2 * 8 * m.value); });
        const int jb = opaque<IT>(s);
        reorder(run_write(run), [&](auto c, float* line) {
          static_for<0, IB>([&](auto ic) {
            const int fb = IT::freq_base(IT::template item_of<true>(jb, ic.value));
            static_for<0, N2>([&](auto k2) {
              const float f = line[IT::template freq_at<k2.value>(fb)];
              if constexpr (c.value) y[ic.value][k2.value].y = f; else y[ic.value][k2.value].x = f;
            });
          });
        });
      } else {
        static_for<0, IB>([&](auto ic) {
          const unsigned base = spec_base(vec < n, ic.value);
          static_for<0, N2>([&](auto k2) { y[ic.value][k2.value] = bload_so<2>(rin, base, N1 * 8 * k2.value); });
        });
      }
      const int ji = opaque<IT>(s);
      static_for<0, IB>([&](auto ic) {
        item_inverse<IT>(IT::template item_of<true>(ji, ic.value), y[ic.value]);
      });
      phase<IT>();
      float2 x[N1];
      // (the last adjoint pass goes straight to the next sample's to_vector)
      EX::template to_vector<ACC && !FWD_OUT>(buf, s, ab, bb, y, x);
      phase<IT>();
      as_a_inverse<IT, HALF>(x, u);
      phase<IT>();
      to_run(u);
      if constexpr (KIND == kAsRowMid || ACC) {
        const Rsrc rmod = make_rsrc(a.mod, (unsigned)nn * 8u);
        if constexpr (KIND == kAsRowMid) {
          each(8, [&](auto k, unsigned o, int so) { u[k.value] = cmul(u[k.value], bload_keep_so(rmod, o, so)); });
          if (a.act_out) {
            const Rsrc ro = make_rsrc(a.act_out + (size_t)b * nn, (unsigned)nn * 8u);
            each_out(8, [&](auto k, unsigned o, int so) { bstore_so(ro, o, so, u[k.value]); });
          }
        } else {
          const Rsrc ra = make_rsrc(a.act_in + (size_t)b * nn, (unsigned)nn * 8u);
          each(8, [&](auto k, unsigned o, int so) {
            const float2 ul = bload_so<2>(ra, o, so);
            acc[k.value] += ul.x * u[k.value].y - ul.y * u[k.value].x;
          });
          if constexpr (KIND == kAsRowBwdMid) {
            phase<IT>();
            each(8, [&](auto k, unsigned o, int so) { u[k.value] = cmulc(u[k.value], bload_keep_so(rmod, o, so)); });
          }
        }
      }
    } else if constexpr (KIND == kAsRowBwdFirst) {
      // seed G_D = 2 (dL/dI) U_D; off the regions of a region loss U_D is not read
      const Rsrc rud = make_rsrc(a.ud_in + (size_t)b * nn, (unsigned)nn * 8u);
      if (a.grad_int) {
        const Rsrc rg = make_rsrc(a.grad_int + (size_t)b * nn, (unsigned)nn * 4u);
        each(8, [&](auto k, unsigned o, int so) { u[k.value] = bload_so<2>(rud, o, so); });
        each(4, [&](auto k, unsigned o, int so) {
          // (zero, not 0 * U_D, where dL/dI is zero: U_D may be infinite or NaN there)
          const float g = bload_f_so(rg, o, so);
          u[k.value] = g != 0.f ? cscale(u[k.value], 2.f * g) : c2(0.f, 0.f);
        });
      } else {
        const float* __restrict__ gs = a.grad_sums + (size_t)b * a.K;
        const unsigned long long vmask = vok ? a.row_mask[vec] : 0ull;
        each(8, [&](auto k, unsigned o, int so) {
          float g = 0.f;
          if (vmask && pos_ok(j, k)) {
            unsigned long long m = vmask & a.col_mask[j + N2 * (k.value + IT::K0(HALF)) - off];
            while (m) {
              g += gs[__builtin_ctzll(m)];
              m &= m - 1;
            }
          }
          // (zero, not 0 * U_D, where no region is)
          const float2 v = bload_so<2>(rud, g != 0.f ? o : kOutOfRange, so);
          u[k.value] = cscale(v, 2.f * g);
        });
      }
    } else {  // kAsRowFirst: natural amplitudes or fields
      if (a.in_real) {
        const Rsrc ri = make_rsrc(static_cast<const float*>(a.in) + (size_t)b * nn, (unsigned)nn * 4u);
        each(4, [&](auto k, unsigned o, int so) { u[k.value] = c2(bload_f_so(ri, o, so), 0.f); });
      } else {
        const Rsrc ri = make_rsrc(static_cast<const float2*>(a.in) + (size_t)b * nn, (unsigned)nn * 8u);
        each(8, [&](auto k, unsigned o, int so) { u[k.value] = bload_so<2>(ri, o, so); });
      }
    }

    if constexpr (FWD_OUT) {
      phase<IT>();
      to_item(u);
      float2 x[N1];
      as_a_forward<IT, HALF>(u, x);
      phase<IT>();
      float2 y[IB][N2];
      EX::to_items(buf, s, ab, bb, x, y);
      phase<IT>();
      const int jf = opaque<IT>(s);
      const Rsrc ro = make_rsrc(a.out + (size_t)b * n * N, (unsigned)(n * N) * 8u);
      // centred: position p holds frequency (p + N/2) mod N, a rotation of k2 by N2/2
      const int rot = a.spec_centred ? N * 4 : 0;
      if constexpr (PL::PFA) {
        static_for<0, IB>([&](auto ic) { item_forward<IT>(IT::template item_of<true>(jf, ic.value), y[ic.value]); });
        float2 run[N1];
        reorder([&](auto c, float* line) {
          static_for<0, IB>([&](auto ic) {
            const int fb = IT::freq_base(IT::template item_of<true>(jf, ic.value));
            static_for<0, N2>([&](auto k2) {
              line[IT::template freq_at<k2.value>(fb)] = c.value ? y[ic.value][k2.value].y : y[ic.value][k2.value].x;
            });
          });
        }, run_read(run));
        const unsigned base = (unsigned)(vec * N + j) * 8u;
        static_for<0, N1>([&](auto m) {
          constexpr int f = N2 * decltype(m)::value;  // frequency j + f
          const bool low = f + N2 <= N / 2 || (f < N / 2 && j + f < N / 2);
          const unsigned at = base + (unsigned)(f * 8 + (low ? rot : -rot));
          bstore_so(ro, vok && act ? at : kOutOfRange, 0, run[m.value]);
        });
      } else static_for<0, IB>([&](auto ic) {
        item_forward<IT>(IT::template item_of<true>(jf, ic.value), y[ic.value]);
        const unsigned base = spec_base(vok && act && IT::item(jf, ic.value), ic.value);
        static_for<0, N2>([&](auto k2) {
          bstore_so(ro, base, N1 * 8 * k2.value + (k2.value < N2 / 2 ? rot : -rot), y[ic.value][k2.value]);
        });
      });
    } else if constexpr (KIND == kAsRowIfft) {
      const Rsrc ro = make_rsrc(a.out + (size_t)b * nn, (unsigned)nn * 8u);
      each_out(8, [&](auto k, unsigned o, int so) { bstore_so(ro, o, so, u[k.value]); });
    } else if constexpr (KIND == kAsRowLast) {
      if (a.skip) {
        const Rsrc rs = make_rsrc(a.skip + (size_t)b * nn, (unsigned)nn * 8u);
        each(8, [&](auto k, unsigned o, int so) {
          const float2 s = bload_so<2>(rs, o, so);
          u[k.value] = cadd(u[k.value], s);
        });
      }
      if (a.field_out) {
        const Rsrc ro = make_rsrc(a.field_out + (size_t)b * nn, (unsigned)nn * 8u);
        each_out(8, [&](auto k, unsigned o, int so) { bstore_so(ro, o, so, u[k.value]); });
      }
      if (a.saved_ud) {
        const Rsrc ro = make_rsrc(a.saved_ud + (size_t)b * nn, (unsigned)nn * 8u);
        each_out(8, [&](auto k, unsigned o, int so) { bstore_so(ro, o, so, u[k.value]); });
      }
      if (a.intensity) {
        const Rsrc ro = make_rsrc(a.intensity + (size_t)b * nn, (unsigned)nn * 4u);
        each_out(4, [&](auto k, unsigned o, int so) {
          float v = cabs2(u[k.value]);
          if (a.accumulate) v += bload_f_so(ro, o, so);
          bstore_f_so(ro, o, so, v);
        });
      }
      if (a.sums_part) {
        // |U|^2 by aperture position (the row pitch holds n <= N values),
        // then one run per (region, row) and the rows added in order
        float* const pix = reinterpret_cast<float*>(buf);
        exchange_sync<W::P>();
        static_for<0, KN>([&](auto k) {
          if (vok && pos_ok(j, k)) pix[r * W::PR + j + N2 * (k.value + IT::K0(HALF)) - off] = cabs2(u[k.value]);
        });
        exchange_sync<W::P>();
        const int K = a.K;
        const int side = a.det_size;
        for (int i = tid; i < K * R; i += W::P) {
          const int k = i / R;
          const int rr = i - k * R;
          const int2 c = a.regions[k];  // (y0, x0)
          float run = 0.f;
          if (tile * R + rr < n && (unsigned)(tile * R + rr - c.x) < (unsigned)side) {
            for (int d = 0; d < side; ++d) run += pix[rr * W::PR + c.y + d];
          }
          rsum[i] = run;
        }
        exchange_sync<W::P>();
        for (int k = tid; k < K; k += W::P) {
          float part = 0.f;
          for (int rr = 0; rr < R; ++rr) part += rsum[k * R + rr];
          a.sums_part[((size_t)b * a.ntiles + tile) * K + k] = part;
        }
      }
    }
  };
  // accumulating kinds run persistently, the others take one item
  if constexpr (ACC) {
    for (int it = rank; it < total; it += a.workers) item(it);
  } else {
    if (rank < total) item(rank);
  }
  if constexpr (ACC) {
    // one partial per lane of workgroups (the tile is fixed): row-major, natural
    const int j = j0;
    const int vec = (rank % a.ntiles) * R + r;
    const Rsrc dp = make_rsrc(a.dphi_part + (size_t)(rank / a.ntiles) * nn, (unsigned)nn * 4u);
    static_for<0, KN>([&](auto k) {
      const int q = j + N2 * (k.value + IT::K0(HALF)) - off;
      bstore_f(dp, act && vec < n && (unsigned)q < (unsigned)n ? (unsigned)(vec * n + q) * 4u : kOutOfRange,
               acc[k.value]);
    });
  }
}

// ---------------------------------------------------------------------------
// Column passes.  A workgroup transforms T spectrum columns of one sample;
// consecutive lanes take consecutive columns.  The transfer function is read
// from the caller's table H[ky][kx] in natural order; an even table
// (H[N - ky] = H[ky]) is read at its rows ky <= N/2 only.  FAR: forward
// transform only, x table, stored at [(ky + N/2) mod N][kx position].
//
// Work order, the ranks of an XCD contiguous: at the power-of-two lengths
// pairs of neighbouring tiles sample by sample, pair after pair (an XCD reads
// an eighth of the table, which stays in its L2: 156 against 161 us at 1024,
// 64 samples of 512 rows; 31.5 against 33.9 at 512); at the others, whose
// rows do not end on 128-byte lines, every tile of a sample, so that tiles
// sharing a line run together (500 points, 32 samples: 54.2 against 60.8 us;
// 400: 44.8 against 45.9; 200: 45.3 against 48.1).
// ---------------------------------------------------------------------------
template <class PL, int T>
struct AsCols : AsItems<PL> {
  using IT = AsItems<PL>;
  static constexpr int P = (T * IT::N2 + 63) / 64 * 64;
  // the lanes past the T columns: their A side is the exchange area's padding
  // column, on the B side they repeat item 0, and they store nothing
  static constexpr bool SPARE = P != T * IT::N2;
  static constexpr int LDS = IT::N1 * IT::P1 * T;
  static constexpr bool PAIRS = (IT::N & (IT::N - 1)) == 0;
  static constexpr bool SPLIT = LDS * 8 > 10 * 1024 * (P / 64);  // as for the rows
  static constexpr int WAVES = IT::N2 * IT::IB > 32 ? 3 : 4;
};

template <class PL, int T, bool HALF, bool FAR>
__global__ void __launch_bounds__((AsCols<PL, T>::P), (AsCols<PL, T>::WAVES)) as_col_pass(PassArgs a) {
  using W = AsCols<PL, T>;
  using IT = AsItems<PL>;
  using EX = Exchange<IT, W::P, W::SPLIT, false, W::SPARE, W::P1 * T, T>;
  constexpr int N = W::N;
  constexpr int N1 = W::N1;
  constexpr int N2 = W::N2;
  constexpr int IB = W::IB;
  constexpr int KN = W::KN(HALF);
  using Scaled = ScaledRoots<PL, HALF>;
  constexpr bool SCALED = Scaled::ON;  // 1/N^2 in the inverse roots, else on the output
  __shared__ typename EX::Elem buf[W::LDS];

  const int per = (int)gridDim.x >> 3;
  const int item = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (item >= a.workers) return;
  int tile;
  int b;
  if constexpr (W::PAIRS) {
    // (pair, sample, tile of the pair); a last odd tile is a pair of one
    const int pair = item / (2 * a.batch);
    const int rest = item - pair * 2 * a.batch;
    const bool whole = 2 * pair + 1 < a.ntiles;
    b = whole ? rest >> 1 : rest;
    tile = 2 * pair + (whole ? rest & 1 : 0);
  } else {
    b = item / a.ntiles;
    tile = item - b * a.ntiles;
  }

  const int tid = (int)threadIdx.x;
  const bool act = !W::SPARE || tid < T * N2;
  const int v = (act ? tid : tid - T * N2) % T;
  const int j = act ? tid / T : N2;
  const int s = act ? j : 0;
  const int n = a.n;
  const int off = a.off;
  const int vec = tile * T + v;
  const bool vok = vec < N && act;
  const int ab = j * T + v;
  int bb[IB];
  static_for<0, IB>([&](auto ic) { bb[ic.value] = IT::template item_of<false>(s, ic.value) * W::P1 * T + v; });
  // f(k, byte offset per lane, scalar byte offset) of this lane's A-item: rows
  // pos - off of column vec
  auto each = [&](auto&& f) {
    const int jj = opaque<IT>(j);
    if constexpr (HALF) {
      const unsigned base = vok ? (unsigned)(jj * N + vec) * 8u : kOutOfRange;
      static_for<0, KN>([&](auto k) { f(k, base, N2 * k.value * N * 8); });
    } else {
      const int p0 = PL::pos_base(jj);
      static_for<0, KN>([&](auto k) {
        const int q = PL::pos_at(p0, k.value) - off;
        f(k, vok && (unsigned)q < (unsigned)n ? (unsigned)(q * N + vec) * 8u : kOutOfRange, 0);
      });
    }
  };

  const Rsrc rin = make_rsrc(static_cast<const float2*>(a.in) + (size_t)b * n * N, (unsigned)(n * N) * 8u);
  float2 u[KN];
  each([&](auto k, unsigned o, int so) { u[k.value] = bload_so<2>(rin, o, so); });
  float2 x[N1];
  as_a_forward<IT, HALF>(u, x);
  phase<IT>();
  float2 y[IB][N2];
  EX::to_items(buf, s, ab, bb, x, y);
  phase<IT>();

  // rows ky = k1 + N1*k2; the mirrored row N - ky = (N1 - k1) + N1*(N2 - 1 - k2)
  const Rsrc rt = make_rsrc(a.tab, (unsigned)(N * N) * 8u);
  const float sg = a.conj_tab ? -1.f : 1.f;  // (one product, not a branch per value)
  const bool sym = a.tab_sym != 0;
  int kx = vec;
  if constexpr (FAR) kx = vec + N / 2 < N ? vec + N / 2 : vec - N / 2;  // centred columns
  static_for<0, IB>([&](auto ic) {
    if (!IT::item(s, ic.value)) return;
    const int k1 = s + N2 * ic.value;
    float2(&z)[N2] = y[ic.value];
    item_forward<IT>(k1, z);
    const bool col = vec < N;  // (spare lanes repeat an item, table and all)
    const int fb = IT::freq_base(k1);
    const unsigned lo = col ? (unsigned)(k1 * N + kx) * 8u : kOutOfRange;
    const unsigned hi = col && sym ? (unsigned)((N1 - k1) * N + kx) * 8u : lo;
    static_for<0, N2>([&](auto k2) {
      constexpr int up = N1 * N * 8 * decltype(k2)::value;
      constexpr int down = N1 * N * 8 * (N2 - 1 - decltype(k2)::value);
      float2 h;
      if constexpr (PL::PFA) {
        const int ky = IT::template freq_at<k2.value>(fb);
        const int row = sym && ky > N / 2 ? N - ky : ky;
        h = bload_keep_so(rt, col ? (unsigned)(row * N + kx) * 8u : kOutOfRange, 0);
      } else {
        h = k2.value < N2 / 2 ? bload_keep_so(rt, lo, up) : bload_keep_so(rt, hi, sym ? down : up);
      }
      z[k2.value] = cmul(z[k2.value], c2(h.x, sg * h.y));
      if constexpr (k2.value % 8 == 7) phase<IT>();  // eight table values in flight
    });
    if constexpr (FAR) {
      const Rsrc ro = make_rsrc(a.out + (size_t)b * N * N, (unsigned)(N * N) * 8u);
      const unsigned out = vok ? (unsigned)(k1 * N + vec) * 8u : kOutOfRange;
      static_for<0, N2>([&](auto k2) {
        if constexpr (PL::PFA) {
          const int ky = IT::template freq_at<k2.value>(fb);
          const int row = ky < N / 2 ? ky + N / 2 : ky - N / 2;
          bstore_so(ro, vok ? (unsigned)(row * N + vec) * 8u : kOutOfRange, 0, z[k2.value]);
        } else {
          constexpr int row = N1 * ((decltype(k2)::value + N2 / 2) % N2);  // (ky + N/2) mod N = k1 + row
          bstore_so(ro, out, row * N * 8, z[k2.value]);
        }
      });
    } else {
      phase<IT>();
      item_inverse<IT, std::conditional_t<SCALED, Scaled, ItemRoots<PL>>>(k1, z);
    }
  });
  if constexpr (!FAR) {
    EX::to_vector(buf, s, ab, bb, y, x);
    phase<IT>();
    as_a_inverse<IT, HALF>(x, u);
    const Rsrc ro = make_rsrc(a.out + (size_t)b * n * N, (unsigned)(n * N) * 8u);
    each([&](auto k, unsigned o, int so) {
      if constexpr (SCALED) bstore_so(ro, o, so, u[k.value]); else bstore_so(ro, o, so, cscale(u[k.value], a.scale));
    });
  }
}

// Columns per workgroup: 128-byte segments of every row (at 1024 points 8
// columns, four waves instead of eight, measured 181 against 156 us for 64
// samples of 512 rows; 32 columns at 256 and 512 5% slower), more where that
// would not be whole waves; at 100, 200 and 500 points, whose rows do not end
// on 128-byte lines, as many as fill 256 lanes (a five-wave workgroup leaves
// SIMDs uneven, sep_impl.hpp): 200 points 48 -> 41 us for 200 samples, 250 in
// 500 47 -> 37 us for 32 (at 400, whose rows do, 45 -> 54 us, so not there).
// Far field of 100 and 200: whole waves.
template <int N, bool FAR> struct AsColT { static constexpr int T = 16; };
template <> struct AsColT<100, false> { static constexpr int T = 25; };
template <> struct AsColT<200, false> { static constexpr int T = 25; };
template <> struct AsColT<100, true> { static constexpr int T = 32; };
template <> struct AsColT<200, true> { static constexpr int T = 32; };
template <bool FAR> struct AsColT<350, FAR> { static constexpr int T = 32; };
template <bool FAR> struct AsColT<500, FAR> { static constexpr int T = 12; };

template <int N, bool FAR>
using AsPlan = typename std::conditional_t<FAR, FarPlanFor<N>, AsPlanFor<N>>::type;

// n = N/2 centred and N1 divisible by 4: HalfDft.  Its roots add 2-4% to the
// rounding of a transform at 20 values, where a whole transform has none
// (Good-Thomas 4 x 5).  A hop at 400 makes up for it (ScaledRoots; 1.94e-7 before
// half transforms, 1.92e-7 now, against 64 bits), one at 200 does not (1.77e-7
// -> 1.83e-7) and takes whole transforms: 100 in 200, 5 layers, batch 200, 263 ->
// 287 us.
template <int N, bool FAR = false>
constexpr bool as_half_plan() { return AsPlan<N, FAR>::N1 % 4 == 0 && N != 200; }
template <int N, bool FAR>
bool as_half(const PassArgs& a) {
  return as_half_plan<N, FAR>() && 2 * a.n == N && 4 * a.off == N;
}

template <int N, int KIND, bool FAR>
hipError_t launch_as_rows(const PassArgs& a, hipStream_t st) {
  using PL = AsPlan<N, FAR>;
  if constexpr (as_half_plan<N, FAR>()) {
    if (as_half<N, FAR>(a)) {
      hipLaunchKernelGGL((as_row_pass<PL, KIND, true>), dim3(a.workers), dim3(AsRows<PL>::P), 0, st, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((as_row_pass<PL, KIND, false>), dim3(a.workers), dim3(AsRows<PL>::P), 0, st, a);
  return hipGetLastError();
}
template <int N, int KIND>
hipError_t launch_as_row(const PassArgs& a, hipStream_t st) {
  if (a.workers < 1 || a.n < 1 || a.n > N || a.off != (N - a.n) / 2) return hipErrorInvalidValue;
  if constexpr (KIND == kAsRowFirst) {
    if (a.spec_centred) return launch_as_rows<N, KIND, true>(a, st);
  }
  return launch_as_rows<N, KIND, false>(a, st);
}

template <int N, bool FAR, bool HALF>
hipError_t launch_as_cols(const PassArgs& args, hipStream_t st) {
  using PL = AsPlan<N, FAR>;
  constexpr int T = AsColT<N, FAR>::T;
  constexpr int P = AsCols<PL, T>::P;
  constexpr int tiles = (N + T - 1) / T;
  // a launch holds fewer than 2^32 threads: batches past that (of apertures a
  // few rows high) go in several
  constexpr int most = static_cast<int>(0xffffffffu / (static_cast<unsigned>(P) * tiles)) - 8;
  PassArgs a = args;
  a.ntiles = tiles;
  for (long long b = 0; b < args.batch; b += most) {
    a.batch = static_cast<int>(std::min<long long>(most, args.batch - b));
    a.workers = tiles * a.batch;
    a.in = static_cast<const float2*>(args.in) + (size_t)b * a.n * N;
    a.out = args.out + (size_t)b * (FAR ? N : a.n) * N;
    hipLaunchKernelGGL((as_col_pass<PL, T, HALF, FAR>), dim3(8 * ((a.workers + 7) / 8)), dim3(P), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <int N, bool FAR>
hipError_t launch_as_col(const PassArgs& a, hipStream_t st) {
  if (a.batch < 1 || a.n < 1 || a.n > N || a.off != (N - a.n) / 2) return hipErrorInvalidValue;
  if constexpr (as_half_plan<N, FAR>()) {
    if (as_half<N, FAR>(a)) return launch_as_cols<N, FAR, true>(a, st);
  }
  return launch_as_cols<N, FAR, false>(a, st);
}

template <int N>
hipError_t launch_as_n(AsPassKind kind, const PassArgs& a, hipStream_t st) {
  switch (kind) {
    case kAsRowFirst: return launch_as_row<N, kAsRowFirst>(a, st);
    case kAsCol: return launch_as_col<N, false>(a, st);
    case kAsRowMid: return launch_as_row<N, kAsRowMid>(a, st);
    case kAsRowLast: return launch_as_row<N, kAsRowLast>(a, st);
    case kAsRowBwdFirst: return launch_as_row<N, kAsRowBwdFirst>(a, st);
    case kAsRowBwdMid: return launch_as_row<N, kAsRowBwdMid>(a, st);
    case kAsRowBwdLast: return launch_as_row<N, kAsRowBwdLast>(a, st);
    case kAsRowIfft: return launch_as_row<N, kAsRowIfft>(a, st);
    case kAsColFar: return launch_as_col<N, true>(a, st);
  }
  return hipErrorInvalidValue;
}

// Rows per workgroup, and resident workgroups of an accumulating row kind.
template <int N>
int as_rows_n(bool far) { return far ? AsRows<AsPlan<N, true>>::R : AsRows<AsPlan<N, false>>::R; }
template <int N>
int slots_as_n(AsPassKind kind, bool half) {
  using PL = AsPlan<N, false>;
  static int cache[2][2] = {};
  const int m = kind == kAsRowBwdMid ? 0 : 1;
  int& c = cache[m][half ? 1 : 0];
  if (c == 0) {
    const void* k = m == 0 ? reinterpret_cast<const void*>(&as_row_pass<PL, kAsRowBwdMid, false>)
                           : reinterpret_cast<const void*>(&as_row_pass<PL, kAsRowBwdLast, false>);
    if constexpr (as_half_plan<N>()) {
      if (half)
        k = m == 0 ? reinterpret_cast<const void*>(&as_row_pass<PL, kAsRowBwdMid, true>)
                   : reinterpret_cast<const void*>(&as_row_pass<PL, kAsRowBwdLast, true>);
    }
    c = resident_per_cu(k, AsRows<PL>::P);
  }
  return c * device_cus();
}

}  // namespace lr
