// Word arithmetic on bitmaps over a text, a bit per byte, 64 bytes to a word.
// Positions are ints: a text may be as long as 2^31 - 3 bytes, so its last
// word can end at 2^31, and no expression here passes its limit argument.
// constexpr, so that kernels and host tests share it.
#pragma once
#include <cstdint>

namespace anon {

// One past the last byte of i's word, at most e (i < e).
[[gnu::always_inline]] constexpr int word_stop(int i, int e) { return e - i <= 64 - (i & 63) ? e : (i | 63) + 1; }

// The bits of bytes [i, stop) of i's word, stop = word_stop(i, .).
[[gnu::always_inline]] constexpr unsigned long long word_mask(int i, int stop) {
  return (stop - i == 64 ? ~0ull : (1ull << (stop - i)) - 1) << (i & 63);
}

// End of the run of set bits from p on, at most lim (base <= p <= lim); bit o
// of the words is the byte at base + o.
[[gnu::always_inline]] constexpr int set_run_end(const uint64_t* words, int base, int p, int lim) {
  while (p < lim) {
    const int o = p - base, left = 64 - (o & 63);
    const uint64_t stop = ~words[o >> 6] >> (o & 63);
    const int run = stop ? __builtin_ctzll(stop) : left;
    if (lim - p <= run) return lim;
    p += run;
    if (stop) return p;
  }
  return p;
}

}  // namespace anon
