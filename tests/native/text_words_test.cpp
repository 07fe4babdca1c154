// text_words.hpp near the largest text (2^31 - 3 bytes), where the end of a
// position's 64-byte word no longer fits an int, and at ordinary positions,
// against bit-by-bit loops in 64 bits.
#include "text_words.hpp"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::printf("FAILED %s line %d\n", #c, __LINE__);           \
      std::exit(1);                                               \
    }                                                             \
  } while (0)

namespace {
constexpr int kMaxText = 0x7ffffffd;  // 2^31 - 3

// the words of bytes [b, e) as a span's marking loop visits them
void check_span(int b, int e) {
  const int64_t w0 = b >> 6, words = (e >> 6) - w0 + 1;
  std::vector<unsigned long long> got(words), want(words);
  int steps = 0;
  for (int i = b; i < e;) {
    CHECK(++steps <= words);
    const int stop = anon::word_stop(i, e);
    CHECK(stop > i && stop <= e && (stop - 1) >> 6 == i >> 6);
    got[(i >> 6) - w0] |= anon::word_mask(i, stop);
    i = stop;
  }
  for (int64_t i = b; i < e; ++i) want[(i >> 6) - w0] |= 1ull << (i & 63);
  CHECK(got == want);
}

// a window of `n` bytes from `base` on whose bits past the text are set, as
// zero padding sets those of the not-a-space class
void check_runs(int base, int n, int text_end, unsigned seed) {
  std::mt19937_64 rng(seed);
  std::vector<uint64_t> words(n / 64);
  for (auto& w : words) w = rng() | rng() | rng();
  for (int64_t o = 0; o < n; ++o)
    if (base + o >= text_end) words[o >> 6] |= 1ull << (o & 63);
  for (int64_t p = base; p <= text_end && p < (int64_t)base + n; ++p)
    for (int64_t lim : {(int64_t)text_end, p, p + 1, p + 63, p + 64, p + 65, p + 200}) {
      if (lim < p || lim > text_end) continue;
      int64_t q = p;
      while (q < lim && ((words[(q - base) >> 6] >> ((q - base) & 63)) & 1)) ++q;
      CHECK(anon::set_run_end(words.data(), base, (int)p, (int)lim) == q);
    }
}
}  // namespace

int main() {
  for (int64_t n = (int64_t(1) << 31) - 200; n <= kMaxText; ++n)
    for (int len : {1, 2, 3, 17, 62, 63, 64, 65, 66, 130, 199})
      if (n - len >= 0) check_span((int)(n - len), (int)n);
  for (int b = 0; b < 130; ++b)
    for (int e = b + 1; e < 330; ++e) check_span(b, e);
  std::printf("PASS spans\n");
  // the window of the last 4096-byte tile: 64 bytes before, 448 after it
  for (int end = kMaxText - 62; end <= kMaxText; ++end) {
    const int tile = (end - 1) & ~4095;
    check_runs(tile - 64, 64 + 4096 + 448, end, (unsigned)end);
  }
  check_runs(-64, 1024, 900, 1);
  std::printf("PASS runs\nALL PASSED\n");
}
