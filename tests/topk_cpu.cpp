// The top-k kernels on the CPU (tests/cpu_hip): a call whose scratch another
// call uses in between, as two streams on one scratch would.  Results of the
// first call are then undefined, its accesses are not: the vectors and the
// scratch lie against pages that may not be touched.  With the workspace that
// is reported and with the smallest that is taken.  Prints "ok".
#include <sys/mman.h>

#include <algorithm>
#include <numeric>
#include <random>

#include "../paper_2409_17836_amd/csrc/lossy.hip"

using namespace lmgc;

// `bytes` (a multiple of 16) with 64 MB of untouchable pages on both sides.
static char* guarded(size_t bytes) {
  const size_t gap = 64 << 20, page = 4096, body = (bytes + page - 1) / page * page;
  char* p = (char*)mmap(nullptr, 2 * gap + body, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (p == MAP_FAILED || mprotect(p + gap, body, PROT_READ | PROT_WRITE)) abort();
  return p + gap + body - bytes;
}

struct Vec {
  int64_t n, k;
  float *v, *out;
  std::vector<float> want;
};

// n values: 3000 above the threshold, `same` that share its leading 23 bits,
// the rest below; k falls among the `same`.
static Vec make(int64_t n, int same, int seed) {
  std::mt19937 rng(seed);
  Vec x{n, 3000 + same / 2, (float*)guarded(n * 4), (float*)guarded(n * 4), {}};
  std::vector<int> at(n);
  std::iota(at.begin(), at.end(), 0);
  std::shuffle(at.begin(), at.end(), rng);
  for (int64_t i = 0; i < n; i++) {
    uint32_t bits;
    const float base = i < 3000 ? 1e-2f : 5e-4f;
    memcpy(&bits, &base, 4);
    bits = (bits & 0xFFFFFF00u) | (rng() & 0xFF);
    if (i >= 3000 + same) bits = rng() % 0x39000000u;
    bits |= (rng() & 1) << 31;
    memcpy(&x.v[at[i]], &bits, 4);
  }
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return mag_key(x.v[a]) > mag_key(x.v[b]); });
  x.want.assign(n, 0.f);
  for (int64_t i = 0; i < x.k; i++) x.want[order[i]] = x.v[order[i]];
  return x;
}

static void check(bool ok, const char* what, int at) {
  if (ok) return;
  printf("%s (after launch %d)\n", what, at);
  exit(1);
}

int main() {
  Vec small = make(40000, 900, 1), large = make(60000, 900, 2), ties = make(48000, 4000, 3);
  Vec* pairs[][2] = {{&small, &large}, {&large, &small}, {&small, &ties}, {&ties, &large}};
  size_t bytes = 0;
  char* ws = nullptr;
  auto topk = [&](Vec& x) { launch_sparsify_topk(x.v, x.n, x.k, x.out, ws, bytes, nullptr); };
  auto same = [](const Vec& x) { return !memcmp(x.out, x.want.data(), x.n * 4); };
  for (size_t b : {lossy_workspace_bytes(), lossy_min_workspace_bytes()}) {
    bytes = b;
    ws = guarded((b + 15) / 16 * 16);
    for (auto& p : pairs) {
      if (b != lossy_workspace_bytes() && &p != &pairs[2]) continue;  // one pair has both routes
      Vec &first = *p[0], &second = *p[1];
      for (int stop = -1;; stop++) {  // launches of `first` before `second` runs
        int launched = 0;
        bool ran = false;
        cpu_hip::after_launch = [&](const char*) {
          if (ran || launched++ != stop) return;
          ran = true;
          topk(second);
        };
        topk(first);
        cpu_hip::after_launch = nullptr;
        if (stop < 0) check(same(first), "a call alone is wrong", stop);
        if (stop >= 0 && !ran) break;
        if (ran) check(same(second), "an uninterrupted call is wrong", stop);
      }
    }
  }
  printf("ok\n");
  return 0;
}
