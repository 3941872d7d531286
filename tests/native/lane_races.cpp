// Shared-memory races between the waves of a workgroup, found on the host: a pass
// kernel compiled as plain C++ runs lane after lane (its control flow does not
// depend on the data), every access to its shared memory is recorded with the
// number of barriers the lane has passed, and two accesses of different waves
// to one word in the same interval between barriers, a read and a write, are a
// race.  (Two writes are not counted: lanes past the last item or vector
// repeat another lane's and write the same values.)  Lanes of one wave are in
// lockstep and cannot race.  Lanes that end with different barrier counts are
// an error too.
//
//   clang++ -fsanitize=thread -c ... -DLR_FFT_N=<size>, linked without the sanitizer:
//   the access hooks it calls are the ones below.
#include <hip/hip_runtime.h>

#include <unordered_map>
#include <vector>

#include "../../paper_2306_11268_amd/csrc/as_impl.hpp"
#include "../../paper_2306_11268_amd/csrc/launch_impl.hpp"

namespace {
struct Access { unsigned readers = 0, writers = 0; };  // waves
std::unordered_map<uint64_t, Access> seen;
bool recording = false;
unsigned lane_wave = 0;
const char* stack_hi = nullptr;
long races = 0;
}  // namespace

#define HOOK extern "C" __attribute__((no_sanitize("thread"), used))
static __attribute__((no_sanitize("thread"))) void access_(void* p, int bytes, bool write) {
  if (!recording) return;
  const char* c = static_cast<const char*>(p);
  const char* here = reinterpret_cast<const char*>(&p);
  if (c >= here - 4096 && c < stack_hi) return;  // the lane's own registers
  recording = false;                             // (the map's accesses are not the kernel's)
  for (uintptr_t w = reinterpret_cast<uintptr_t>(c) / 4; w <= (reinterpret_cast<uintptr_t>(c) + bytes - 1) / 4; ++w) {
    Access& a = seen[(static_cast<uint64_t>(w) << 16) | static_cast<unsigned>(lane_epoch)];
    const unsigned others = ~(1u << lane_wave);
    if ((write ? a.readers : a.writers) & others) ++races;
    (write ? a.writers : a.readers) |= 1u << lane_wave;
  }
  recording = true;
}
#define HOOKS(n)                                                        \
  HOOK void __tsan_read##n(void* p) { access_(p, n, false); }           \
  HOOK void __tsan_write##n(void* p) { access_(p, n, true); }           \
  HOOK void __tsan_unaligned_read##n(void* p) { access_(p, n, false); } \
  HOOK void __tsan_unaligned_write##n(void* p) { access_(p, n, true); } \
  HOOK void __tsan_read_write##n(void* p) { access_(p, n, true); }      \
  HOOK void __tsan_unaligned_read_write##n(void* p) { access_(p, n, true); }
HOOKS(1)
HOOKS(2)
HOOKS(4)
HOOKS(8)
HOOKS(16)
HOOK void __tsan_read_range(void* p, long n) { access_(p, (int)n, false); }
HOOK void __tsan_write_range(void* p, long n) { access_(p, (int)n, true); }
HOOK void __tsan_func_entry(void*) {}
HOOK void __tsan_func_exit() {}
HOOK void __tsan_init() {}
HOOK void __tsan_vptr_update(void**, void*) {}
HOOK void __tsan_vptr_read(void**) {}
HOOK void* __tsan_memcpy(void* d, const void* s, size_t n) { return __builtin_memmove(d, s, n); }
HOOK void* __tsan_memmove(void* d, const void* s, size_t n) { return __builtin_memmove(d, s, n); }
HOOK void* __tsan_memset(void* d, int c, size_t n) {
  for (size_t i = 0; i < n; ++i) static_cast<volatile char*>(d)[i] = (char)c;
  return d;
}

namespace {
using namespace lr;
constexpr int N = LR_FFT_N;

std::vector<float> some(1 << 22, 1.f);  // stands for every array a kernel reads directly
std::vector<unsigned long long> masks(N, 1ull);
std::vector<int> perm(N, 0);
std::vector<int2> regions(kMaxRegions, int2{0, 0});

PassArgs args(int n, int tiles, int workers) {
  PassArgs a{};
  a.n = n;
  a.off = (N - n) / 2;
  a.nvec = n;
  a.batch = 3;
  a.spg = 1;
  a.full = n == N;
  a.in = some.data();
  a.out = reinterpret_cast<float2*>(some.data());
  a.tab = reinterpret_cast<const float2*>(some.data());
  a.mod = reinterpret_cast<const float2*>(some.data());
  a.act_in = reinterpret_cast<const float2*>(some.data());
  a.act_out = a.out;
  a.dphi_part = some.data();
  a.skip = a.mod;
  a.ud_in = a.mod;
  a.grad_int = some.data();
  a.intensity = some.data();
  a.field_out = a.out;
  a.sums_part = some.data();
  a.grad_sums = some.data();
  a.row_mask = masks.data();
  a.col_mask = masks.data();
  a.regions = regions.data();
  a.K = 3;
  a.det_size = 2;
  a.in_real = 1;
  a.ntiles = tiles;
  a.workers = workers;
  a.lanes = 1;
  return a;
}

// One workgroup of P lanes; its persistent loop takes every item of its tile.
template <class K>
__attribute__((no_sanitize("thread"))) bool run(const char* what, K kernel, int P, unsigned grid, const PassArgs& a) {
  seen.clear();
  races = 0;
  int epochs = -1;
  bool even = true;
  gridDim = {grid, 1, 1};
  blockDim = {static_cast<unsigned>(P), 1, 1};
  blockIdx = {0, 0, 0};
  char top;
  stack_hi = &top + 65536;
  for (int t = 0; t < P; ++t) {
    threadIdx = {static_cast<unsigned>(t), 0, 0};
    lane_wave = static_cast<unsigned>(t) / 64;
    lane_epoch = 0;
    recording = true;
    kernel(a);
    recording = false;
    even = even && (epochs < 0 || epochs == lane_epoch);
    epochs = lane_epoch;
  }
  const bool ok = races == 0 && even && !seen.empty();
  std::printf("%s N=%d P=%d barriers=%d words=%zu races=%ld%s %s\n", what, N, P, epochs, seen.size(), races,
              even ? "" : " uneven barriers", ok ? "ok" : "FAIL");
  return ok;
}

template <int KIND, bool HALF>
bool as_row(const char* what) {
  using PL = typename AsPlanFor<N>::type;
  const int n = HALF ? N / 2 : N;
  const int tiles = (n + AsRows<PL>::R - 1) / AsRows<PL>::R;
  if (AsRows<PL>::P == 64) return true;
  constexpr bool acc = KIND == kAsRowBwdMid || KIND == kAsRowBwdLast;
  return run(what, &as_row_pass<PL, KIND, HALF>, AsRows<PL>::P, tiles * 3, args(n, tiles, acc ? tiles : tiles * 3));
}
template <bool HALF>
bool as_rows() {
  return as_row<kAsRowFirst, HALF>("as first") & as_row<kAsRowMid, HALF>("as mid") &
         as_row<kAsRowLast, HALF>("as last") & as_row<kAsRowIfft, HALF>("as ifft") &
         as_row<kAsRowBwdFirst, HALF>("as bwd first") & as_row<kAsRowBwdMid, HALF>("as bwd mid") &
         as_row<kAsRowBwdLast, HALF>("as bwd last");
}
template <bool HALF, bool FAR>
bool as_col() {
  using PL = AsPlan<N, FAR>;
  constexpr int T = AsColT<N, FAR>::T;
  const int tiles = (N + T - 1) / T;
  return run(FAR ? "as far" : "as col", &as_col_pass<PL, T, HALF, FAR>, AsCols<PL, T>::P, (tiles * 3 + 7) / 8 * 8,
             args(HALF ? N / 2 : N, tiles, tiles * 3));
}

template <int KIND, int AXIS>
bool sep(const char* what) {
  if constexpr (sep_kind<N, KIND, AXIS>()) {
    using G = typename SepFor<N, KIND, AXIS>::type;
    if (G::P == 64) return true;
    const int tiles = (N + G::T - 1) / G::T;
    constexpr bool acc = KIND == kBwdMid || KIND == kBwdLast;
    if constexpr (KIND == kFwdLast || KIND == kBwdFirst) {
      return run(what, &sep_detector_pass<G, KIND>, G::P, tiles * 3, args(N, tiles, tiles * 3));
    } else {
      return run(what, &sep_pass<G, KIND>, G::P, (tiles * 3 + 7) / 8 * 8, args(N, tiles, acc ? tiles : tiles * 3));
    }
  }
  return true;
}
}  // namespace

int main() {
  bool ok = as_rows<false>() & as_col<false, false>() & as_col<false, true>();
  if constexpr (as_half_plan<N>()) ok &= as_rows<true>() & as_col<true, false>();
  if constexpr (as_half_plan<N, true>()) ok &= as_col<true, true>();
  ok &= sep<kPropOnce, kRow>("sep first row") & sep<kFwdMid, kRow>("sep mid row") & sep<kBwdMid, kRow>("sep bwd row") &
        sep<kFwdLast, kRow>("sep last row") & sep<kBwdFirst, kRow>("sep seed row") &
        sep<kFwdMid, kCol>("sep mid col") & sep<kBwdMid, kCol>("sep bwd col") & sep<kBwdLast, kCol>("sep bwd last col");
  std::printf(ok ? "ALL OK\n" : "FAILURES\n");
  return ok ? 0 : 1;
}
