// Helper kernels and the size dispatch of the pass kernels.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "tile.hpp"

namespace lr {

// Per-size entry points, defined in kern_size.hip (one object per size).
template <int N> hipError_t launch_fr_n(PassKind, Axis, const PassArgs&, hipStream_t);
template <int N> int slots_fr_n(PassKind, Axis, int);
template <int N> int tile_fr_n(PassKind, Axis, int);
template <int N> hipError_t launch_as_n(AsPassKind, const PassArgs&, hipStream_t);
template <int N> int as_rows_n(bool);
template <int N> int slots_as_n(AsPassKind, bool);
template <int N> TileShape shape_n();
template <int N> SlotMap slot_map_n();
template <int N> bool row_major_n(bool);
template <int N> hipError_t launch_field_fwd_n(const FieldArgs&, hipStream_t);

// ---------------------------------------------------------------------------
// Helper kernels
// ---------------------------------------------------------------------------

struct OrientArg { int o[64]; };

// mod[l][sq][sv] = gamma * exp(j*phi_l[y][x]) with (q, vec) = (sm.pos(sq),
// sm.pos(sv)) and (y, x) = (q, vec), or (vec, q) when transposed.
__device__ __forceinline__ void prep_mod_body(const float* __restrict__ phi, int layers, int n, float gamma,
                                              const OrientArg& orient, SlotMap sm, float2* __restrict__ mod) {
  const size_t nn = (size_t)n * n;
  const size_t total = nn * layers;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int l = (int)(i / nn);
    const size_t r = i - (size_t)l * nn;
    const int sq = (int)(r / n);
    const int q = sm.pos(sq);
    const int vec = sm.pos((int)(r - (size_t)sq * n));
    const bool tr = orient.o[l < 64 ? l : 63] != 0;
    const int y = tr ? vec : q;
    const int x = tr ? q : vec;
    float s, c;
    sincosf(phi[(size_t)l * nn + (size_t)y * n + x], &s, &c);
    mod[i] = c2(gamma * c, gamma * s);
  }
}

// sums[b][k] (one wave each): the per-tile partial sums, lane l adding tiles
// l, l + 64, ... and the lanes a fixed butterfly.  One thread per sum walked
// up to 256 tiles one load at a time (20 us for 1000 sums of 67 tiles).
__global__ void __launch_bounds__(256) finish_sums_kernel(const float* __restrict__ part, int batch, int ntiles, int K,
                                                          float* __restrict__ sums, int accumulate) {
  const int lane = threadIdx.x & 63;
  for (unsigned i = blockIdx.x * 4 + (threadIdx.x >> 6); i < (unsigned)(batch * K); i += gridDim.x * 4) {
    const unsigned b = i / K;
    const int k = (int)(i - b * K);
    float s = 0.f;
    for (int tl = lane; tl < ntiles; tl += 64) s += part[((size_t)b * ntiles + tl) * K + k];
    s = wave_sum(s);
    if (lane == 0) sums[i] = accumulate ? sums[i] + s : s;
  }
}

// Loss of the detector sums, averaged over the batch, and its gradient
// dL/dS.  kind 0: softmax cross-entropy, -log p_t.  kind 1: the paper's
// ||softmax(S) - onehot(t)||^2, whose gradient goes through the softmax
// Jacobian: dL/dS_j = p_j (d_j - sum_i d_i p_i), d = 2 (p - t) / B.
// One workgroup; sample b is handled by thread b % 1024 and the per-thread
// losses are summed in a fixed order.  An out-of-range label makes the loss NaN.
__global__ void __launch_bounds__(1024) loss_kernel(int kind, const float* __restrict__ sums,
                                                    const int32_t* __restrict__ labels, int batch, int K,
                                                    float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ float red[16];
  float my = 0.f;
  const float invb = 1.0f / (float)batch;
  for (int b = threadIdx.x; b < batch; b += 1024) {
    const float* s = sums + (size_t)b * K;
    float mx = s[0];
    for (int k = 1; k < K; ++k) mx = fmaxf(mx, s[k]);
    float z = 0.f;
    for (int k = 0; k < K; ++k) z += expf(s[k] - mx);
    const float lz = logf(z);
    const int tl = labels[b];
    const bool valid = (unsigned)tl < (unsigned)K;
    float lb;
    if (kind == 0) {
      lb = lz + mx - (valid ? s[tl] : 0.f);
      if (grad) {
        for (int k = 0; k < K; ++k) grad[(size_t)b * K + k] = (expf(s[k] - mx - lz) - (k == tl ? 1.f : 0.f)) * invb;
      }
    } else {
      lb = 0.f;
      float c = 0.f;  // sum_i d_i p_i
      for (int k = 0; k < K; ++k) {
        const float p = expf(s[k] - mx - lz);
        const float r = p - (k == tl ? 1.f : 0.f);
        lb += r * r;
        c += 2.f * r * invb * p;
      }
      if (grad) {
        for (int k = 0; k < K; ++k) {
          const float p = expf(s[k] - mx - lz);
          const float d = 2.f * (p - (k == tl ? 1.f : 0.f)) * invb;
          grad[(size_t)b * K + k] = p * (d - c);
        }
      }
    }
    my += valid ? lb : __builtin_nanf("");
  }
  const float tot = block_sum<1024>(my, red);
  if (threadIdx.x == 0 && loss) *loss = tot * invb;
}

// Codesign layer (§3.2): per pixel, w = softmax((logits + noise) / tau) over
// the K device levels; the phase is sum_k w_k levels_k, or (hard) the level
// of the largest logits + noise, the first on ties.  The gradient (the soft
// Jacobian, also the straight-through gradient of the hard layer) is
// dL/dlogit_j = w_j (levels_j - sum_k w_k levels_k) dL/dphi / tau.
//
// A streaming pass over the scores: G = 1 .. 64 lanes hold a pixel's scores in
// registers (lane l levels l, l + G, ...; as many lanes as K needs, so that a
// wave carries 64 / G pixels), read once, U pixels in flight per lane group,
// every exponential formed once.  A lane adds its levels in order and the
// lanes add up in halves, from 32 apart to 1, whatever G is.  One wave per
// pixel, one pixel at a time, was held by the latency of its loads and its
// chain of reductions: 200 000 pixels of 256 levels 134 -> 67 us forward
// (410 MB, 6.1 TB/s) and 168 -> 108 us backward (615 MB, 5.7 TB/s), 300 000
// of 64 levels 76 -> 39 and 72 -> 48.  16-byte loads, whose lanes hold
// neighbouring levels, gain nothing at 256 levels and 13 us at 64, but they
// change the order of a pixel's sums, which the gradient's level minus mean
// makes visible (1e-4 of the largest value).
constexpr int kCodesignMaxLevels = 1024;

// Reductions over groups of G lanes: across lanes D apart, from G/2 to 1.
template <int D>
__device__ __forceinline__ float lane_across(float x) {
  if constexpr (D == 1) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
  } else if constexpr (D == 2) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
  } else if constexpr (D == 8) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xF, 0xF, false));  // row_ror:8
  } else if constexpr (D == 4 || D == 16) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), (D << 10) | 0x1F));  // xor D
  } else {
    return __shfl_xor(x, 32, 64);
  }
}
template <int G, class Op>
__device__ __forceinline__ float group_reduce(float x, Op op) {
  if constexpr (G >= 64) x = op(x, lane_across<32>(x));
  if constexpr (G >= 32) x = op(x, lane_across<16>(x));
  if constexpr (G >= 16) x = op(x, lane_across<8>(x));
  if constexpr (G >= 8) x = op(x, lane_across<4>(x));
  if constexpr (G >= 4) x = op(x, lane_across<2>(x));
  if constexpr (G >= 2) x = op(x, lane_across<1>(x));
  return x;
}

template <int G, int N>
__device__ __forceinline__ void codesign_read(const float* __restrict__ p, int K, int lane, bool ok, float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = ok && lane + G * i < K ? p[lane + G * i] : 0.f;
}

// BWD: out [count][K] = dL/dlogits; else out [count] = phases.
template <int G, int N, int U, bool BWD>
__global__ void __launch_bounds__(256) codesign_kernel(const float* __restrict__ logits, const float* __restrict__ noise,
                                                       const float* __restrict__ levels, int K, long long count,
                                                       float inv_tau, int hard, const float* __restrict__ grad_phi,
                                                       float* __restrict__ out) {
  constexpr int PER = 256 / G;  // lane groups per workgroup
  const int lane = threadIdx.x % G;
  const int group = threadIdx.x / G;
  auto fmax2 = [](float a, float b) { return fmaxf(a, b); };
  auto fsum2 = [](float a, float b) { return a + b; };
  float lv[N];
  codesign_read<G, N>(levels, K, lane, true, lv);
  const long long step = (long long)gridDim.x * PER * U;
  for (long long p0 = ((long long)blockIdx.x * U) * PER + group; p0 < count + group; p0 += step) {
    float sc[U][N];
    float nz[U][N];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long p = p0 + (long long)u * PER;
      codesign_read<G, N>(logits + p * K, K, lane, p < count, sc[u]);
      codesign_read<G, N>(noise + p * K, K, lane, p < count, nz[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long p = p0 + (long long)u * PER;
      float smax = -INFINITY;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        sc[u][i] = lane + G * i < K ? sc[u][i] + nz[u][i] : -INFINITY;
        smax = fmaxf(smax, sc[u][i]);
      }
      smax = group_reduce<G>(smax, fmax2);
      if (!BWD && hard) {
        // the first level reaching the maximum, and its phase
        int kb = K;
#pragma unroll
        for (int i = N - 1; i >= 0; --i) {
          const int k = lane + G * i;
          if (k < K && sc[u][i] == smax) kb = k;
        }
        // (level indices are exact in float32)
        const float kf = group_reduce<G>((float)kb, [](float a, float b) { return fminf(a, b); });
        const int k = (int)kf;
        if (lane == 0 && p < count) out[p] = levels[k < K ? k : 0];  // (none reaches it only for NaN scores)
        continue;
      }
      const float ymax = smax * inv_tau;
      float es = 0.f;
      float ws = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float e = lane + G * i < K ? expf(sc[u][i] * inv_tau - ymax) : 0.f;
        es += e;
        ws += e * lv[i];
        sc[u][i] = e;
      }
      es = group_reduce<G>(es, fsum2);
      ws = group_reduce<G>(ws, fsum2);
      if constexpr (!BWD) {
        if (lane == 0 && p < count) out[p] = ws / es;
      } else {
        const float inv_s = 1.f / es;
        const float mean = ws * inv_s;
        const float gs = p < count ? grad_phi[p] * inv_tau : 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) sc[u][i] = sc[u][i] * inv_s * (lv[i] - mean) * gs;
        if (p < count) {
          float* o = out + p * K;
#pragma unroll
          for (int i = 0; i < N; ++i)
            if (lane + G * i < K) o[lane + G * i] = sc[u][i];
        }
      }
    }
  }
}

struct CodesignArgs {
  const float* logits;
  const float* noise;
  const float* levels;
  int K;
  long long count;
  float inv_tau;
  int hard;
  const float* grad_phi;
  float* out;
  hipStream_t st;
};
template <int G, int N, int U>
static void launch_codesign_shape(const CodesignArgs& a) {
  constexpr int PER = 256 / G * U;  // pixels per workgroup and round
  long long blocks = (a.count + PER - 1) / PER;
  if (blocks > 65536) blocks = 65536;
  const dim3 grid((unsigned)blocks);
  if (a.grad_phi) {
    hipLaunchKernelGGL((codesign_kernel<G, N, U, true>), grid, dim3(256), 0, a.st, a.logits, a.noise, a.levels, a.K,
                       a.count, a.inv_tau, a.hard, a.grad_phi, a.out);
  } else {
    hipLaunchKernelGGL((codesign_kernel<G, N, U, false>), grid, dim3(256), 0, a.st, a.logits, a.noise, a.levels,
                       a.K, a.count, a.inv_tau, a.hard, a.grad_phi, a.out);
  }
}

// One Adam step on every element: m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// phi -= lr * (m / bc1) / (sqrt(v / bc2) + eps), bc = 1 - beta^t.
__global__ void adam_kernel(float* __restrict__ phi, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, long long count, float lr, float b1, float b2, float eps,
                            float bc1, float bc2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    phi[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  }
}

// dphi_l[y][x] = sum over groups of part_l[g][sq][sv], oriented (transposed:
// q = x) and in the slot order sm ((q, vec) = (sm.pos(sq), sm.pos(sv))), for
// every layer l = blockIdx.y in one launch; part_l starts at
// part + l * layer_stride.  A workgroup covers 64 consecutive elements with 4
// slices of 64 threads; slice s sums groups s, s+4, s+8, ... in order and the
// four partial sums are added in slice order, so the result does not depend
// on scheduling.  A layer with no groups gets zeros.
struct ReduceArg {
  int groups[64];
  int transposed[64];
};
__global__ void __launch_bounds__(256) reduce_dphi_kernel(const float* __restrict__ part, size_t layer_stride,
                                                          ReduceArg arg, int n, SlotMap sm, float* __restrict__ out) {
  __shared__ float red[4][64];
  const int l = blockIdx.y;
  const int groups = arg.groups[l];
  const float* __restrict__ pl = part + (size_t)l * layer_stride;
  const size_t nn = (size_t)n * n;
  const int lane = threadIdx.x & 63;
  const int slice = threadIdx.x >> 6;
  const size_t i = (size_t)blockIdx.x * 64 + lane;
  float s = 0.f;
  if (i < nn) {
    int g = slice;
    for (; g + 12 < groups; g += 16) {
      const float a0 = pl[(size_t)g * nn + i];
      const float a1 = pl[(size_t)(g + 4) * nn + i];
      const float a2 = pl[(size_t)(g + 8) * nn + i];
      const float a3 = pl[(size_t)(g + 12) * nn + i];
      s += a0;
      s += a1;
      s += a2;
      s += a3;
    }
    for (; g < groups; g += 4) s += pl[(size_t)g * nn + i];
  }
  red[slice][lane] = s;
  __syncthreads();
  if (slice == 0 && i < nn) {
    const float r = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    const int sq = (int)(i / n);
    const int q = sm.pos(sq);
    const int v = sm.pos((int)(i - (size_t)sq * n));
    out[(size_t)l * nn + (arg.transposed[l] ? (size_t)v * n + q : (size_t)q * n + v)] = r;
  }
}

// Region corners, per-row / per-column coverage masks (natural indices) and
// the covered-first permutations of the stored rows and columns (slot order
// sm): stored indices whose natural row / column a region covers, in
// ascending order, then the others.  Run by one workgroup of 1024 threads,
// thread i handles row i and column i (n <= 1024).
__device__ void set_regions_body(const Regions& reg, int n, SlotMap sm, int2* dst, unsigned long long* row_mask,
                                 unsigned long long* col_mask, int* row_perm, int* col_perm, int (*wave_count)[16]) {
  const int i = threadIdx.x;
  if (i < reg.K) dst[i] = make_int2(reg.y0[i], reg.x0[i]);
  auto masks = [&](int p, unsigned long long& rm, unsigned long long& cm) {
    rm = 0;
    cm = 0;
    for (int k = 0; k < reg.K; ++k) {
      if ((unsigned)(p - reg.y0[k]) < (unsigned)reg.s) rm |= 1ull << k;
      if ((unsigned)(p - reg.x0[k]) < (unsigned)reg.s) cm |= 1ull << k;
    }
  };
  unsigned long long rm = 0, cm = 0;
  if (i < n) {
    masks(i, rm, cm);
    row_mask[i] = rm;
    col_mask[i] = cm;
    masks(sm.pos(i), rm, cm);  // coverage of stored index i
  }
  const bool rc = i < n && rm != 0;
  const bool cc = i < n && cm != 0;
  const int lane = i & 63;
  const int wave = i >> 6;
  const unsigned long long rb = __ballot(rc);
  const unsigned long long cb = __ballot(cc);
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  if (lane == 0) {
    wave_count[0][wave] = __popcll(rb);
    wave_count[1][wave] = __popcll(cb);
  }
  __syncthreads();
  int r_rank = __popcll(rb & below), c_rank = __popcll(cb & below), r_total = 0, c_total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) {
      r_rank += wave_count[0][w];
      c_rank += wave_count[1][w];
    }
    r_total += wave_count[0][w];
    c_total += wave_count[1][w];
  }
  if (i < n) {
    // r_rank = covered rows before i, so i - r_rank uncovered rows precede it
    row_perm[rc ? r_rank : r_total + (i - r_rank)] = i;
    col_perm[cc ? c_rank : c_total + (i - c_rank)] = i;
  }
}

// Separable Fresnel chirps in natural frequency order from the 2-D table H
// (N x N): x chirp H[0][f], y chirp H[f][0] * conj(H[0][0]) (so the two
// carry exp(jkz) once), each with the 1/N of the inverse DFT folded in.
__device__ __forceinline__ void prep_chirps_body(const float2* __restrict__ H, int N, float2* __restrict__ cx,
                                                 float2* __restrict__ cy) {
  const float inv = 1.0f / (float)N;
  const float2 h00c = c2(H[0].x, -H[0].y);
  for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < N; f += gridDim.x * blockDim.x) {
    cx[f] = cscale(H[f], inv);
    cy[f] = cscale(cmul(H[(size_t)f * N], h00c), inv);
  }
}

// Per-call tables in one launch: the modulation of every layer (all
// workgroups), the separable chirps when H is given, and, when the call reads
// detector regions, the region tables (workgroup 0).  Workgroups of 1024
// threads.
__global__ void __launch_bounds__(1024) prep_layers_kernel(const float* __restrict__ phi, int layers, int n, float gamma,
                                                           OrientArg orient, SlotMap sm, float2* __restrict__ mod,
                                                           Regions reg,
                                                           int2* dst, unsigned long long* row_mask,
                                                           unsigned long long* col_mask, int* row_perm, int* col_perm,
                                                           const float2* __restrict__ H, int nfft,
                                                           float2* __restrict__ cx, float2* __restrict__ cy) {
  __shared__ int wave_count[2][16];
  if (blockIdx.x == 0 && dst) set_regions_body(reg, n, sm, dst, row_mask, col_mask, row_perm, col_perm, wave_count);
  if (H) prep_chirps_body(H, nfft, cx, cy);
  if (phi) prep_mod_body(phi, layers, n, gamma, orient, sm, mod);
}

// Detector readout from a field: one workgroup per (sample, region).
__global__ void __launch_bounds__(256) readout_kernel(const float2* __restrict__ field, int n, Regions reg,
                                                      float* __restrict__ sums) {
  __shared__ float red[4];
  const int b = blockIdx.y;
  const int k = blockIdx.x;
  const int K = reg.K;
  const int s = reg.s;
  const float2* f = field + (size_t)b * n * n;
  const int ry = reg.y0[k];
  const int rx = reg.x0[k];
  float my = 0.f;
  for (int e = threadIdx.x; e < s * s; e += 256) {
    const int dy = e / s;
    const int dx = e - dy * s;
    my += cabs2(f[(size_t)(ry + dy) * n + rx + dx]);
  }
  const float tot = block_sum<256>(my, red);
  if (threadIdx.x == 0) sums[(size_t)b * K + k] = tot;
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------

bool fft_size_supported(int N) {
  switch (N) {
    case 64:
    case 100:
    case 128:
    case 200:
    case 256:
    case 350:
    case 400:
    case 500:
    case 512:
    case 1000:
    case 1024:
      return true;
    default:
      return false;
  }
}

TileShape tile_shape(int N, int) {
  switch (N) {
    case 64: return shape_n<64>();
    case 100: return shape_n<100>();
    case 128: return shape_n<128>();
    case 200: return shape_n<200>();
    case 256: return shape_n<256>();
    case 350: return shape_n<350>();
    case 400: return shape_n<400>();
    case 500: return shape_n<500>();
    case 512: return shape_n<512>();
    case 1000: return shape_n<1000>();
    case 1024: return shape_n<1024>();
    default: return TileShape{0, 0};
  }
}

SlotMap slot_map(int N) {
  switch (N) {
    case 64: return slot_map_n<64>();
    case 100: return slot_map_n<100>();
    case 128: return slot_map_n<128>();
    case 200: return slot_map_n<200>();
    case 256: return slot_map_n<256>();
    case 350: return slot_map_n<350>();
    case 400: return slot_map_n<400>();
    case 500: return slot_map_n<500>();
    case 512: return slot_map_n<512>();
    case 1000: return slot_map_n<1000>();
    case 1024: return slot_map_n<1024>();
    default: return SlotMap{0, 0, 0};
  }
}

bool row_major_rows(int N, bool backward) {
  switch (N) {
    case 64: return row_major_n<64>(backward);
    case 100: return row_major_n<100>(backward);
    case 128: return row_major_n<128>(backward);
    case 200: return row_major_n<200>(backward);
    case 256: return row_major_n<256>(backward);
    case 350: return row_major_n<350>(backward);
    case 400: return row_major_n<400>(backward);
    case 500: return row_major_n<500>(backward);
    case 512: return row_major_n<512>(backward);
    case 1000: return row_major_n<1000>(backward);
    case 1024: return row_major_n<1024>(backward);
    default: return false;
  }
}

bool field_forward_supported(int N) { return N == 64 || N == 100 || N == 128 || N == 200; }

bool field_forward_preferred(int N, int batch) {
  if (!field_forward_supported(N) || N == 200) return false;
  if (N == 64) return true;
  int dev = 0;
  int cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return false;
  return batch >= cus;
}

hipError_t launch_field_forward(int N, const FieldArgs& a, hipStream_t st) {
  switch (N) {
    case 64: return launch_field_fwd_n<64>(a, st);
    case 100: return launch_field_fwd_n<100>(a, st);
    case 128: return launch_field_fwd_n<128>(a, st);
    case 200: return launch_field_fwd_n<200>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fresnel_pass(int N, PassKind kind, Axis axis, const PassArgs& a, hipStream_t st) {
  switch (N) {
    case 64: return launch_fr_n<64>(kind, axis, a, st);
    case 100: return launch_fr_n<100>(kind, axis, a, st);
    case 128: return launch_fr_n<128>(kind, axis, a, st);
    case 200: return launch_fr_n<200>(kind, axis, a, st);
    case 256: return launch_fr_n<256>(kind, axis, a, st);
    case 350: return launch_fr_n<350>(kind, axis, a, st);
    case 400: return launch_fr_n<400>(kind, axis, a, st);
    case 500: return launch_fr_n<500>(kind, axis, a, st);
    case 512: return launch_fr_n<512>(kind, axis, a, st);
    case 1000: return launch_fr_n<1000>(kind, axis, a, st);
    case 1024: return launch_fr_n<1024>(kind, axis, a, st);
    default: return hipErrorInvalidValue;
  }
}

int fresnel_pass_tile(int N, PassKind kind, Axis axis, int full) {
  switch (N) {
    case 64: return tile_fr_n<64>(kind, axis, full);
    case 100: return tile_fr_n<100>(kind, axis, full);
    case 128: return tile_fr_n<128>(kind, axis, full);
    case 200: return tile_fr_n<200>(kind, axis, full);
    case 256: return tile_fr_n<256>(kind, axis, full);
    case 350: return tile_fr_n<350>(kind, axis, full);
    case 400: return tile_fr_n<400>(kind, axis, full);
    case 500: return tile_fr_n<500>(kind, axis, full);
    case 512: return tile_fr_n<512>(kind, axis, full);
    case 1000: return tile_fr_n<1000>(kind, axis, full);
    case 1024: return tile_fr_n<1024>(kind, axis, full);
    default: return 0;
  }
}

int fresnel_pass_slots(int N, PassKind kind, Axis axis, int full) {
  switch (N) {
    case 64: return slots_fr_n<64>(kind, axis, full);
    case 100: return slots_fr_n<100>(kind, axis, full);
    case 128: return slots_fr_n<128>(kind, axis, full);
    case 200: return slots_fr_n<200>(kind, axis, full);
    case 256: return slots_fr_n<256>(kind, axis, full);
    case 350: return slots_fr_n<350>(kind, axis, full);
    case 400: return slots_fr_n<400>(kind, axis, full);
    case 500: return slots_fr_n<500>(kind, axis, full);
    case 512: return slots_fr_n<512>(kind, axis, full);
    case 1000: return slots_fr_n<1000>(kind, axis, full);
    case 1024: return slots_fr_n<1024>(kind, axis, full);
    default: return 0;
  }
}

hipError_t launch_as_pass(int N, AsPassKind kind, const PassArgs& a, hipStream_t st) {
  switch (N) {
    case 64: return launch_as_n<64>(kind, a, st);
    case 100: return launch_as_n<100>(kind, a, st);
    case 128: return launch_as_n<128>(kind, a, st);
    case 200: return launch_as_n<200>(kind, a, st);
    case 256: return launch_as_n<256>(kind, a, st);
    case 350: return launch_as_n<350>(kind, a, st);
    case 400: return launch_as_n<400>(kind, a, st);
    case 500: return launch_as_n<500>(kind, a, st);
    case 512: return launch_as_n<512>(kind, a, st);
    case 1000: return launch_as_n<1000>(kind, a, st);
    case 1024: return launch_as_n<1024>(kind, a, st);
    default: return hipErrorInvalidValue;
  }
}


int as_row_tile(int N, bool far) {
  switch (N) {
    case 64: return as_rows_n<64>(far);
    case 100: return as_rows_n<100>(far);
    case 128: return as_rows_n<128>(far);
    case 200: return as_rows_n<200>(far);
    case 256: return as_rows_n<256>(far);
    case 350: return as_rows_n<350>(far);
    case 400: return as_rows_n<400>(far);
    case 500: return as_rows_n<500>(far);
    case 512: return as_rows_n<512>(far);
    case 1000: return as_rows_n<1000>(far);
    case 1024: return as_rows_n<1024>(far);
    default: return 0;
  }
}

int as_pass_slots(int N, AsPassKind kind, bool half) {
  switch (N) {
    case 64: return slots_as_n<64>(kind, half);
    case 100: return slots_as_n<100>(kind, half);
    case 128: return slots_as_n<128>(kind, half);
    case 200: return slots_as_n<200>(kind, half);
    case 256: return slots_as_n<256>(kind, half);
    case 350: return slots_as_n<350>(kind, half);
    case 400: return slots_as_n<400>(kind, half);
    case 500: return slots_as_n<500>(kind, half);
    case 512: return slots_as_n<512>(kind, half);
    case 1000: return slots_as_n<1000>(kind, half);
    case 1024: return slots_as_n<1024>(kind, half);
    default: return 0;
  }
}

// ---------------------------------------------------------------------------
// Layer normalisation of intensity maps (per sample, over count values).
// Chunk c of sample b covers values [c * kLnChunk, min(count, (c+1) * kLnChunk)).
// ---------------------------------------------------------------------------
// The chunk sits in registers between the two sums (16 values a thread), in
// 16-byte pieces where the maps allow (VEC); the chunks are merged by one wave
// in a fixed order, inside the last kernel for maps of up to kLnFuse chunks.
// (64 maps of 350 x 350: 32 -> 16 us forward, 32 -> 26 us backward; 16 of 1000 x
// 1000: 104 -> 35 and 106 -> 49; before,
// every value was read twice by the first kernel, a thread per sample walked
// its chunks and the last kernel divided 64-bit indices per value.)
constexpr int kLnThreads = 256;
constexpr int kLnPer = kLnChunk / kLnThreads;  // values per thread of a chunk
constexpr int kLnFuse = 256;

// f(i, offset, valid) for this thread's values of chunk c (offset inside the
// sample); VEC: runs of four consecutive values.
template <bool VEC, class F>
__device__ __forceinline__ void ln_values(int c, long long count, F&& f) {
  const long long lo = (long long)c * kLnChunk;
#pragma unroll
  for (int i = 0; i < kLnPer; ++i) {
    const long long o = VEC ? lo + 4 * ((i / 4) * kLnThreads + (int)threadIdx.x) + i % 4
                            : lo + i * kLnThreads + (int)threadIdx.x;
    f(i, o, o < count);
  }
}
template <bool VEC>
__device__ __forceinline__ void ln_read(const float* __restrict__ x, int c, long long count, float (&v)[kLnPer]) {
  if constexpr (VEC) {
    const long long lo = (long long)c * kLnChunk;
#pragma unroll
    for (int i = 0; i < kLnPer / 4; ++i) {
      const long long o = lo + 4 * (i * kLnThreads + (int)threadIdx.x);
      const float4 q = o < count ? *reinterpret_cast<const float4*>(x + o) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[4 * i] = q.x;
      v[4 * i + 1] = q.y;
      v[4 * i + 2] = q.z;
      v[4 * i + 3] = q.w;
    }
  } else {
    ln_values<VEC>(c, count, [&](int i, long long o, bool ok) { v[i] = ok ? x[o] : 0.f; });
  }
}

// g == nullptr: part = (chunk mean, sum of squared deviations from it);
// otherwise part = (sum of g, sum of g * y) with y = x the normalised map.
template <bool VEC>
__global__ void __launch_bounds__(kLnThreads) ln_partial_kernel(const float* __restrict__ x,
                                                                const float* __restrict__ g, long long count,
                                                                int nchunks, float2* __restrict__ part) {
  __shared__ float red[kLnThreads / 64];
  const int c = blockIdx.x;
  const int b = blockIdx.y;
  const size_t base = (size_t)b * (size_t)count;
  float v[kLnPer];
  ln_read<VEC>(x + base, c, count, v);
  float s1 = 0.f;
  float s2 = 0.f;
  if (g == nullptr) {
    const long long left = count - (long long)c * kLnChunk;
    const float n = (float)(left < kLnChunk ? left : kLnChunk);
#pragma unroll
    for (int i = 0; i < kLnPer; ++i) s1 += v[i];
    const float mean = block_sum<kLnThreads>(s1, red) / n;
    ln_values<VEC>(c, count, [&](int i, long long, bool ok) {
      const float d = ok ? v[i] - mean : 0.f;
      s2 += d * d;
    });
    const float m2 = block_sum<kLnThreads>(s2, red);
    if (threadIdx.x == 0) part[(size_t)b * nchunks + c] = c2(mean, m2);
  } else {
    float gv[kLnPer];
    ln_read<VEC>(g + base, c, count, gv);
#pragma unroll
    for (int i = 0; i < kLnPer; ++i) {
      s1 += gv[i];
      s2 += gv[i] * v[i];
    }
    const float a = block_sum<kLnThreads>(s1, red);
    const float bsum = block_sum<kLnThreads>(s2, red);
    if (threadIdx.x == 0) part[(size_t)b * nchunks + c] = c2(a, bsum);
  }
}

// One wave merges the chunks of a sample: lane l takes chunks l, l + 64, ... in
// order, then the lanes merge in a fixed butterfly.  Forward: chunk means and
// squared-deviation sums by the pairwise update of Chan et al., returning
// (mean, 1/sqrt(M2 / count + eps)); backward: (mean of g, mean of g * y).
__device__ __forceinline__ float2 ln_merge(const float2* __restrict__ p, long long count, int nchunks, float eps,
                                           bool backward) {
  const int lane = threadIdx.x & 63;
  if (backward) {
    float a = 0.f;
    float m = 0.f;
    for (int c = lane; c < nchunks; c += 64) {
      a += p[c].x;
      m += p[c].y;
    }
    return c2(wave_sum(a) / (float)count, wave_sum(m) / (float)count);
  }
  float n_a = 0.f;
  float mean = 0.f;
  float m2 = 0.f;
  // (an empty side leaves the other as it is)
  auto merge = [&](float n_b, float mean_b, float m2_b) {
    const float n = n_a + n_b;
    const float w = n > 0.f ? n_b / n : 0.f;
    const float delta = mean_b - mean;
    mean = n_a > 0.f ? mean + delta * w : mean_b;
    m2 = m2 + m2_b + (n_a > 0.f && n_b > 0.f ? delta * delta * (n_a * w) : 0.f);
    n_a = n;
  };
  for (int c = lane; c < nchunks; c += 64) {
    const long long left = count - (long long)c * kLnChunk;
    merge((float)(left < kLnChunk ? left : kLnChunk), p[c].x, p[c].y);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float nb = __shfl_xor(n_a, o, 64);
    const float mb = __shfl_xor(mean, o, 64);
    const float qb = __shfl_xor(m2, o, 64);
    if (nb > 0.f) merge(nb, mb, qb);
  }
  // every lane merged the same chunks, in its own order: lane 0's result
  mean = __shfl(mean, 0, 64);
  m2 = __shfl(m2, 0, 64);
  return c2(mean, 1.f / sqrtf(m2 / (float)count + eps));
}

__global__ void __launch_bounds__(64) ln_combine_kernel(const float2* __restrict__ part, long long count, int nchunks,
                                                        float eps, int backward, float2* __restrict__ out) {
  const int b = blockIdx.x;
  const float2 r = ln_merge(part + (size_t)b * nchunks, count, nchunks, eps, backward != 0);
  if (threadIdx.x == 0) out[b] = r;
}

// Forward: y = (x - mean) * rstd.  Backward (g != nullptr, x = y the
// normalised map): dx = rstd * (g - mean(g) - y * mean(g * y)).  A workgroup
// per chunk and sample; FUSE: it merges the sample's partials itself (part),
// and chunk 0's writes them to the statistics.
template <bool VEC, bool FUSE>
__global__ void __launch_bounds__(kLnThreads) ln_apply_kernel(const float* __restrict__ x, const float* __restrict__ g,
                                                              const float2* __restrict__ part, float2* stats,
                                                              const float2* __restrict__ stats2, long long count,
                                                              int nchunks, float eps, float* __restrict__ out) {
  __shared__ float2 merged;
  const int c = blockIdx.x;
  const int b = blockIdx.y;
  const size_t base = (size_t)b * (size_t)count;
  float v[kLnPer];
  float gv[kLnPer];
  ln_read<VEC>(x + base, c, count, v);
  if (g) ln_read<VEC>(g + base, c, count, gv);
  float2 s;
  float2 s2;
  if constexpr (FUSE) {
    if (threadIdx.x < 64) {
      const float2 r = ln_merge(part + (size_t)b * nchunks, count, nchunks, eps, g != nullptr);
      if (threadIdx.x == 0) {
        merged = r;
        if (!g && c == 0) stats[b] = r;
      }
    }
    __syncthreads();
    s = g ? stats[b] : merged;
    s2 = merged;
  } else {
    s = stats[b];
    s2 = g ? stats2[b] : c2(0.f, 0.f);
  }
#pragma unroll
  for (int i = 0; i < kLnPer; ++i) v[i] = g ? s.y * (gv[i] - s2.x - v[i] * s2.y) : (v[i] - s.x) * s.y;
  if constexpr (VEC) {
    const long long lo = (long long)c * kLnChunk;
#pragma unroll
    for (int i = 0; i < kLnPer / 4; ++i) {
      const long long o = lo + 4 * (i * kLnThreads + (int)threadIdx.x);
      if (o < count) *reinterpret_cast<float4*>(out + base + o) = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
  } else {
    ln_values<VEC>(c, count, [&](int i, long long o, bool ok) {
      if (ok) out[base + o] = v[i];
    });
  }
}

// The three kernels of either direction (g null: forward).  The in-place forms
// (out = x, or out = g) read a chunk whole before they write it.
template <bool VEC>
static hipError_t launch_ln(const float* x, const float* g, int batch, long long count, float eps, float* out,
                            float2* stats, float2* part, float2* stats2, hipStream_t st) {
  const int nchunks = (int)ln_chunks(count);
  const dim3 grid(nchunks, batch);
  hipLaunchKernelGGL(ln_partial_kernel<VEC>, grid, dim3(kLnThreads), 0, st, x, g, count, nchunks, part);
  if (nchunks <= kLnFuse) {
    hipLaunchKernelGGL((ln_apply_kernel<VEC, true>), grid, dim3(kLnThreads), 0, st, x, g, part, stats, stats2, count,
                       nchunks, eps, out);
  } else {
    hipLaunchKernelGGL(ln_combine_kernel, dim3(batch), dim3(64), 0, st, part, count, nchunks, eps, g ? 1 : 0,
                       g ? stats2 : stats);
    hipLaunchKernelGGL((ln_apply_kernel<VEC, false>), grid, dim3(kLnThreads), 0, st, x, g, part, stats, stats2, count,
                       nchunks, eps, out);
  }
  return hipGetLastError();
}
// Every map starts on 16 bytes and is a whole number of float4.
static bool ln_vec(const void* a, const void* b, const void* c, long long count) {
  auto ok = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  return count % 4 == 0 && ok(a) && ok(b) && ok(c);
}

hipError_t launch_layer_norm(const float* x, int batch, long long count, float eps, float* y, float2* stats,
                             float2* part, hipStream_t st) {
  if (batch < 1 || batch > 65535 || count < 1 || ln_chunks(count) > (1 << 30)) return hipErrorInvalidValue;
  return ln_vec(x, y, nullptr, count) ? launch_ln<true>(x, nullptr, batch, count, eps, y, stats, part, nullptr, st)
                                      : launch_ln<false>(x, nullptr, batch, count, eps, y, stats, part, nullptr, st);
}

hipError_t launch_layer_norm_backward(const float* g, const float* y, const float2* stats, int batch,
                                      long long count, float* dx, float2* part, float2* stats2, hipStream_t st) {
  if (batch < 1 || batch > 65535 || count < 1 || ln_chunks(count) > (1 << 30)) return hipErrorInvalidValue;
  float2* s = const_cast<float2*>(stats);  // (only read in this direction)
  return ln_vec(g, y, dx, count) ? launch_ln<true>(y, g, batch, count, 0.f, dx, s, part, stats2, st)
                                 : launch_ln<false>(y, g, batch, count, 0.f, dx, s, part, stats2, st);
}

hipError_t launch_prep_layers(const float* phi, int layers, int n, float gamma, const int* orient_host, SlotMap sm,
                              float2* mod, const Regions* regions, int2* dst, unsigned long long* row_mask,
                              unsigned long long* col_mask, int* row_perm, int* col_perm, const float2* H, int nfft,
                              float2* chirp_x, float2* chirp_y, hipStream_t st) {
  if (n < 1 || n > 1024 || layers < 0 || layers > 64 || (H && (nfft < n || !chirp_x || !chirp_y)))
    return hipErrorInvalidValue;
  if (sm.N1 != 0 && sm.N1 * sm.N2 != n) return hipErrorInvalidValue;
  if (regions && (regions->K < 1 || regions->K > kMaxRegions)) return hipErrorInvalidValue;
  OrientArg o{};
  for (int l = 0; l < layers; ++l) o.o[l] = orient_host[l];
  Regions r{};
  if (regions) r = *regions;
  const size_t total = (size_t)n * n * layers;
  int blocks = (int)((total + 1023) / 1024);
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(prep_layers_kernel, dim3(blocks), dim3(1024), 0, st, layers > 0 ? phi : nullptr, layers, n,
                     gamma, o, sm, mod, r, regions ? dst : nullptr, row_mask, col_mask, row_perm, col_perm, H, nfft,
                     chirp_x, chirp_y);
  return hipGetLastError();
}

hipError_t launch_finish_sums(const float* part, int batch, int ntiles, int K, float* sums, int accumulate,
                              hipStream_t st) {
  // (a launch holds fewer than 2^32 threads; more sums than 2^22 workgroups of
  // four take further rounds)
  const unsigned blocks = std::min((static_cast<unsigned>(batch * K) + 3) / 4, 1u << 22);
  hipLaunchKernelGGL(finish_sums_kernel, dim3(blocks), dim3(256), 0, st, part, batch, ntiles, K, sums,
                     accumulate);
  return hipGetLastError();
}

hipError_t launch_loss(int kind, const float* sums, const int32_t* labels, int batch, int K, float* grad, float* loss,
                       hipStream_t st) {
  hipLaunchKernelGGL(loss_kernel, dim3(1), dim3(1024), 0, st, kind, sums, labels, batch, K, grad, loss);
  return hipGetLastError();
}

hipError_t launch_codesign(const float* logits, const float* noise, const float* levels, int K, long long count,
                           float tau, int hard, const float* grad_phi, float* phi_or_grad, hipStream_t st) {
  if (K < 1 || K > kCodesignMaxLevels) return hipErrorInvalidValue;
  if (count <= 0) return hipSuccess;
  const CodesignArgs a{logits, noise, levels, K, count, 1.f / tau, hard, grad_phi, phi_or_grad, st};
  if (K <= 1) launch_codesign_shape<1, 1, 4>(a);
  else if (K <= 2) launch_codesign_shape<2, 1, 4>(a);
  else if (K <= 4) launch_codesign_shape<4, 1, 4>(a);
  else if (K <= 8) launch_codesign_shape<8, 1, 4>(a);
  else if (K <= 16) launch_codesign_shape<16, 1, 4>(a);
  else if (K <= 32) launch_codesign_shape<32, 1, 4>(a);
  else if (K <= 64) launch_codesign_shape<64, 1, 4>(a);
  else if (K <= 128) launch_codesign_shape<64, 2, 4>(a);
  else if (K <= 256) launch_codesign_shape<64, 4, 2>(a);
  else if (K <= 512) launch_codesign_shape<64, 8, 2>(a);
  else launch_codesign_shape<64, 16, 1>(a);
  return hipGetLastError();
}

hipError_t launch_adam(float* phi, const float* g, float* m, float* v, long long count, float lr, float b1, float b2,
                       float eps, float bc1, float bc2, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  long long blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)blocks), dim3(256), 0, st, phi, g, m, v, count, lr, b1, b2, eps, bc1,
                     bc2);
  return hipGetLastError();
}

hipError_t launch_reduce_dphi(const float* part, size_t layer_stride, const int* groups, const int* transposed,
                              int layers, int n, SlotMap sm, float* out, hipStream_t st) {
  if (layers < 1 || layers > 64) return hipErrorInvalidValue;
  if (sm.N1 != 0 && sm.N1 * sm.N2 != n) return hipErrorInvalidValue;
  ReduceArg arg{};
  for (int l = 0; l < layers; ++l) {
    arg.groups[l] = groups[l];
    arg.transposed[l] = transposed[l];
  }
  const size_t nn = (size_t)n * n;
  const int blocks = (int)((nn + 63) / 64);
  hipLaunchKernelGGL(reduce_dphi_kernel, dim3(blocks, layers), dim3(256), 0, st, part, layer_stride, arg, n, sm, out);
  return hipGetLastError();
}


hipError_t launch_readout(const float2* field, int batch, int n, const Regions& r, float* sums, hipStream_t st) {
  hipLaunchKernelGGL(readout_kernel, dim3(r.K, batch), dim3(256), 0, st, field, n, r, sums);
  return hipGetLastError();
}

}  // namespace lr
