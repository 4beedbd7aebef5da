// The serialisation kernel on the CPU (tests/cpu_hip) against a token-by-token
// reference: every value width, byte order, group length and number of
// separators, streams that end at, before and after the edges of a thread's
// four tokens and of a block, ranges of windows that start anywhere and run
// into the padding, with and without bins; few and many tokens per thread.
// Values and outputs lie against pages that may not be touched.  Prints "ok".
#include <sys/mman.h>

#include <random>

#include "../paper_2409_17836_amd/csrc/serialize.hip"

using namespace lmgc;

struct Guarded {  // `bytes` that end (but for their alignment) at an untouchable page
  char *map, *p;
  size_t len;
  explicit Guarded(size_t bytes, size_t align) {
    const size_t page = 4096, body = (bytes + page - 1) / page * page;
    len = body + 2 * page;
    map = (char*)mmap(nullptr, len, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == MAP_FAILED || (body && mprotect(map + page, body, PROT_READ | PROT_WRITE))) abort();
    p = map + page + body - (bytes + align - 1) / align * align;
  }
  ~Guarded() { munmap(map, len); }
};

static void reference(const uint8_t* v, int64_t n, const lmgc_serial_params& sp, std::vector<int>& tok,
                      std::vector<uint8_t>& sym) {
  const int bpv = sp.bytes_per_value, nsep = sp.sep2_id >= 0 ? 2 : 1;
  auto put = [&](int id, int bin) { tok.push_back(id), sym.push_back((uint8_t)bin); };
  const int64_t nbytes = n * bpv;
  for (int64_t b = 0; b < nbytes; b++) {
    const uint8_t x = v[b / bpv * bpv + (sp.msb_first ? bpv - 1 - b % bpv : b % bpv)];
    put(sp.hex_ids[x >> 4], x >> 4);
    put(sp.hex_ids[x & 15], x & 15);
    if (sp.bytes_per_group > 0 && ((b + 1) % sp.bytes_per_group == 0 || b + 1 == nbytes))
      for (int i = 0; i < nsep; i++) put(i ? sp.sep2_id : sp.sep_id, 16 + i);
  }
}

template <int R>
static void check(const Guarded& vals, int64_t n, const lmgc_serial_params& sp, const std::vector<int>& tok,
                  const std::vector<uint8_t>& sym, int64_t first, int64_t count, bool want_sym) {
  const int64_t len = count * sp.window, t0 = first * sp.window;
  Guarded t(len * 4, 16), s(len, 4);
  memset(t.p, 0xEE, len * 4);
  memset(s.p, 0xEE, len);
  launch_rounds<R>(n ? vals.p : nullptr, n, sp, first, count, (int32_t*)t.p, want_sym ? (uint8_t*)s.p : nullptr, nullptr);
  for (int64_t i = 0; i < len; i++) {
    const bool in = t0 + i < (int64_t)tok.size();
    const int want = in ? tok[t0 + i] : sp.pad_id, bin = in ? sym[t0 + i] : 255;
    if (((int32_t*)t.p)[i] == want && (!want_sym || (uint8_t)s.p[i] == bin)) continue;
    printf("rounds %d n %lld bpv %d bpg %d sep2 %d msb %d window %d range %lld+%lld: token %lld\n", R, (long long)n,
           sp.bytes_per_value, sp.bytes_per_group, sp.sep2_id, sp.msb_first, sp.window, (long long)first,
           (long long)count, (long long)i);
    exit(1);
  }
}

int main() {
  std::mt19937 rng(1);
  for (int bpv : {1, 2, 4})
    for (int bpg : {0, 1, 2, 3, 4, 5, 8, 100, 255})
      for (int sep2 : {-1, 44})
        for (int64_t bytes : {4, 8, 20, 452, 456, 460, 1816, 1820, 1824, 2044, 2048, 4096, 5000}) {
          const int64_t n = bytes / bpv;
          Guarded vals(n * bpv, bpv);
          for (int64_t i = 0; i < n * bpv; i++) vals.p[i] = (char)rng();
          lmgc_serial_params sp{};
          sp.bytes_per_value = bpv, sp.bytes_per_group = bpg, sp.msb_first = (int)(rng() & 1);
          sp.sep_id = 32, sp.sep2_id = sep2, sp.pad_id = 7;
          for (int i = 0; i < 16; i++) sp.hex_ids[i] = 100 + i;
          std::vector<int> tok;
          std::vector<uint8_t> sym;
          reference((uint8_t*)vals.p, n, sp, tok, sym);
          const int windows[] = {1, 100, 256, 1000, 1023};
          sp.window = windows[rng() % 5];
          if (sp.window == 1 && tok.size() > 3000) sp.window = 1024;
          const int64_t nw = ((int64_t)tok.size() + sp.window - 1) / sp.window;
          check<1>(vals, n, sp, tok, sym, 0, nw, true);
          check<4>(vals, n, sp, tok, sym, 0, nw, true);
          const int64_t first = rng() % nw, count = 1 + rng() % (nw - first);
          check<1>(vals, n, sp, tok, sym, first, count, rng() & 1);
          check<4>(vals, n, sp, tok, sym, first, count, rng() & 1);
        }
  printf("ok\n");
  return 0;
}
