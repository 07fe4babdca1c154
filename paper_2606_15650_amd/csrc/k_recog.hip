// Pattern recognizers beside the NER model (the paper's detector pairs the
// transformer with regular-expression recognizers, Sec. II stage 2) and the
// merge of overlapping detections into whole-entity spans.
//
// Nine recognizers, each a rule at one start byte of a record (W = word bytes
// [A-Za-z0-9_], LABEL = [A-Za-z0-9-], LOCAL = [A-Za-z0-9._%+-]):
//   0 URL       "http://" or "https://" at a word start, then >= 1 non-space bytes
//   1 EMAIL     maximal LOCAL run, '@', >= 1 "label." groups, then an all-letter
//               top label of >= 2 bytes not followed by a LABEL byte (longest)
//   2 IPV4      four dot-separated octets 0..255 without leading zeros, at word
//               boundaries
//   3 MAC       six hex pairs separated by ':', at word boundaries
//   4 HASH      a hex run of exactly 32, 40 or 64 bytes at word boundaries
//   5 CVE       "CVE-" + 4 digits + '-' + 4..7 digits at word boundaries
//   6 HOSTNAME  dotted LABEL run not preceded by LABEL or '.', ending at a label
//               equal to one of eight top labels, not followed by LABEL (longest)
//   7 IPV6      an address in an RFC 4291 (section 2.2) text form: the maximal
//               run of hex digits, ':' and '.' from a hex digit or ':' not
//               preceded by W, ':' or '.', without its trailing dots, not
//               followed by W
//   8 CPE       "cpe:/" + part [aho] or "cpe:2.3:" + part [aho*-] at a word
//               start, the part not followed by a component byte C =
//               [A-Za-z0-9._~%*?!\-], then the maximal run of C and ':'
// Every start byte where a rule matches gives one candidate span.
//
// Merge: NER spans and candidates sharing a byte form one span, their union
// (transitively; spans that only touch stay apart), typed by its longest
// member, then NER before recognizers (in the order above), then the leftmost.
//
// The rules are tried at anchors only: every match holds one byte that few
// bytes equal, at a place that fixes its start -- the '@' of an e-mail, the
// first '.' of a hostname or an IPv4 address, the first ':' of a URL, MAC,
// IPv6 or CPE, the '-' after "CVE", and for a hash the first aligned 16-byte
// block of hex digits inside it.  A workgroup stages 4096 bytes (16 per
// thread) with 64 bytes before and 448 after in LDS, lists its anchors (about
// one byte in forty), and runs the rules on them with the lanes packed.
//
// Merge: two bitmaps over the text, S (a span begins here) and J (this byte
// and the one before it lie in one span).  A union begins where S holds and J
// does not, and ends at the first byte after it where J does not hold.  The
// begins are counted per tile, their ranks number the unions, and a 64-bit
// atomic max per union over its members' keys (length, priority, begin, type)
// picks its type.
//
// Bound by the rules' scans and by launches: a byte costs one read and half a
// bit of bitmap traffic, where per-byte counters, flags, keys and their
// three-kernel scans moved about 140 bytes of memory per text byte over 20
// launches.  4.9 MB of text with its NER spans in 4096 records: 467 ->
// 35 us (the rules 22).
#include "kernels.hpp"
#include "text_words.hpp"

namespace anon {
namespace {

__device__ __forceinline__ bool is_digit(uint8_t c) { return c >= '0' && c <= '9'; }
__device__ __forceinline__ bool is_letter(uint8_t c) { return (c | 0x20) >= 'a' && (c | 0x20) <= 'z'; }
__device__ __forceinline__ bool is_word(uint8_t c) { return is_digit(c) || is_letter(c) || c == '_'; }
__device__ __forceinline__ bool is_label(uint8_t c) { return is_digit(c) || is_letter(c) || c == '-'; }
__device__ __forceinline__ bool is_local(uint8_t c) {
  return is_digit(c) || is_letter(c) || c == '.' || c == '_' || c == '%' || c == '+' || c == '-';
}
__device__ __forceinline__ bool is_hex(uint8_t c) {
  return is_digit(c) || ((c | 0x20) >= 'a' && (c | 0x20) <= 'f');
}
__device__ __forceinline__ bool is_space(uint8_t c) { return c == ' ' || (c >= '\t' && c <= '\r'); }

constexpr int kTile = 4096;                   // text bytes per match workgroup, 16 per thread
constexpr int kBefore = 64, kAfter = 448;     // staged before and after the tile
constexpr int kWin = kBefore + kTile + kAfter;
constexpr int kWinWords = kWin / 64;

// Byte classes kept as bitmaps of the staged window, a bit per byte: a run's
// end is then one count of trailing zeros per 64 bytes instead of a load, a
// range test and a branch per byte.
enum Class { C_LABEL, C_LOCAL, C_HEX, C_LETTER, C_TEXT /* not a space */, C_COUNT };
__device__ __forceinline__ bool in_class(uint8_t c, int k) {
  return k == C_LABEL ? is_label(c) : k == C_LOCAL ? is_local(c) : k == C_HEX ? is_hex(c) : k == C_LETTER ? is_letter(c)
                                                                                               : !is_space(c);
}

// One record's bytes [lo, hi) of the text; positions are absolute (texts are
// below 2^31 - 2 bytes: a position and the one past it fit an int, the end of
// its 64-byte word may not, see text_words.hpp).  Bytes inside the workgroup's
// staged window [wlo, whi) are read from LDS (window position of byte i:
// i - base), the rest (long runs past the window) from global memory.
struct Rec {
  const uint8_t* t;
  int lo, hi;
  const uint8_t* win;
  const uint64_t (*cls)[kWinWords];
  int base, wlo, whi;
  __device__ uint8_t at(int i) const { return (i >= wlo && i < whi) ? win[i - base] : t[i]; }
  __device__ bool word_start(int p) const { return is_word(at(p)) && (p == lo || !is_word(at(p - 1))); }
  __device__ bool word_end(int q) const { return q == hi || !is_word(at(q)); }
  // bytes p .. p + N - 1, p >= lo, are inside the record and pass f(i, byte):
  // inside the window the loads are independent (no early exit), so they cost
  // one LDS latency
  template <int N, typename F>
  __device__ bool all(int p, F f) const {
    if (hi - p < N) return false;
    bool ok = true;
    if (p >= wlo && whi - p >= N) {
      const uint8_t* q = win + (p - base);
#pragma unroll
      for (int i = 0; i < N; ++i) ok = f(i, q[i]) && ok;
    } else {
      for (int i = 0; i < N && ok; ++i) ok = f(i, t[p + i]);
    }
    return ok;
  }
  template <int N>
  __device__ bool has(int p, const char (&s)[N]) const {
    return all<N - 1>(p, [&](int i, uint8_t c) { return c == (uint8_t)s[i]; });
  }
  // end of the run of class k from p on, at most hi
  template <int K>
  __device__ int run_end(int p) const {
    const int lim = min(hi, whi);
    if (p >= wlo && p < lim) {
      p = set_run_end(cls[K], base, p, lim);
      if (p < lim) return p;
    }
    p = min(p, hi);
    while (p < hi && in_class(at(p), K)) ++p;  // past the window
    return p;
  }
  // start of the run of class k that ends before p, at least lo
  template <int K>
  __device__ int run_begin(int p) const {
    const int lim = max(lo, wlo);
    while (p > lim && p <= whi) {
      const int o = p - 1 - base;
      const uint64_t stop = ~cls[K][o >> 6] << (63 - (o & 63));
      if (stop) {
        p -= __clzll((long long)stop);
        if (p > lim) return p;
        break;
      }
      p -= (o & 63) + 1;
    }
    p = max(p, lo);
    while (p > lo && in_class(at(p - 1), K)) --p;
    return p;
  }
};

__device__ int match_url(const Rec& r, int p) {
  if (!r.word_start(p)) return -1;
  int q;
  if (r.has(p, "https://")) q = p + 8;
  else if (r.has(p, "http://")) q = p + 7;
  else return -1;
  const int e = r.run_end<C_TEXT>(q);
  return e > q ? e : -1;
}

// Whether the label [s, e) is one of the eight top labels.
__device__ bool top_listed(const Rec& r, int s, int e) {
  switch (e - s) {
    case 3: return r.has(s, "lan") || r.has(s, "net") || r.has(s, "org");
    case 4: return r.has(s, "corp");
    case 5: return r.has(s, "intra") || r.has(s, "local");
    case 7: return r.has(s, "example");
    case 8: return r.has(s, "internal");
    default: return false;
  }
}

// Dotted LABEL groups from i on: the top label (a listed one, or at least two
// letters) may be any label but the first; the longest successful domain is
// the last success in order.
template <bool LISTED>
__device__ int dotted_domain(const Rec& r, int i) {
  int best = -1;
  bool first = true;
  while (true) {
    const int j = r.run_end<C_LABEL>(i);
    if (!first && (LISTED ? top_listed(r, i, j) : j - i >= 2 && r.run_end<C_LETTER>(i) >= j)) best = j;
    if (j == i || j >= r.hi || r.at(j) != '.') return best;
    first = false;
    i = j + 1;
  }
}

// p: the start of a LOCAL run, maximal to the left
__device__ int match_email(const Rec& r, int p) {
  const int q = r.run_end<C_LOCAL>(p);
  if (q == r.hi || r.at(q) != '@') return -1;
  return dotted_domain<false>(r, q + 1);
}

// p: the start of a LABEL run, maximal to the left
__device__ int match_hostname(const Rec& r, int p) {
  if (p > r.lo && r.at(p - 1) == '.') return -1;
  return dotted_domain<true>(r, p);
}

// End of a valid octet spanning the whole digit run at i, else -1.
__device__ int octet(const Rec& r, int i) {
  int e = i;
  int v = 0;
  while (e < r.hi && is_digit(r.at(e)) && e - i < 4) v = v * 10 + (r.at(e++) - '0');
  const int c = e - i;
  if (c < 1 || c > 3 || (c > 1 && r.at(i) == '0') || v > 255) return -1;
  return e;
}

__device__ int match_ipv4(const Rec& r, int p) {
  if (!is_digit(r.at(p)) || !r.word_start(p)) return -1;
  int i = p;
  for (int k = 0; k < 4; ++k) {
    const int e = octet(r, i);
    if (e < 0) return -1;
    if (k == 3) return r.word_end(e) ? e : -1;
    if (e == r.hi || r.at(e) != '.') return -1;
    i = e + 1;
  }
  return -1;
}

__device__ int match_mac(const Rec& r, int p) {
  if (!r.word_start(p) || !r.all<17>(p, [](int k, uint8_t c) { return k % 3 == 2 ? c == ':' : is_hex(c); })) return -1;
  return r.word_end(p + 17) ? p + 17 : -1;
}

__device__ int match_hash(const Rec& r, int p) {
  if (!r.word_start(p)) return -1;
  const int e = r.run_end<C_HEX>(p), c = e - p;
  return ((c == 32 || c == 40 || c == 64) && r.word_end(e)) ? e : -1;
}

__device__ int match_cve(const Rec& r, int p) {
  if (!r.word_start(p) || r.hi - p < 9 || !r.has(p, "CVE-")) return -1;
  for (int k = 0; k < 4; ++k)
    if (!is_digit(r.at(p + 4 + k))) return -1;
  if (r.at(p + 8) != '-') return -1;
  int e = p + 9;
  while (e < r.hi && is_digit(r.at(e)) && e - (p + 9) < 8) ++e;
  const int c = e - (p + 9);
  return (c >= 4 && c <= 7 && r.word_end(e)) ? e : -1;
}

__device__ __forceinline__ bool is_cpe(uint8_t c) {
  return is_digit(c) || is_letter(c) || c == '.' || c == '_' || c == '~' || c == '%' || c == '*' || c == '?' ||
         c == '!' || c == '\\' || c == '-';
}

__device__ int match_cpe(const Rec& r, int p) {
  if (!r.word_start(p)) return -1;
  int q;
  bool v23;
  if (r.has(p, "cpe:/")) q = p + 5, v23 = false;
  else if (r.has(p, "cpe:2.3:")) q = p + 8, v23 = true;
  else return -1;
  if (q == r.hi) return -1;
  const uint8_t part = r.at(q);
  if (!(part == 'a' || part == 'h' || part == 'o' || (v23 && (part == '*' || part == '-')))) return -1;
  ++q;
  if (q < r.hi && is_cpe(r.at(q))) return -1;
  while (q < r.hi && (is_cpe(r.at(q)) || r.at(q) == ':')) ++q;
  return q;
}

// Four octets separated by '.', exactly covering [i, end).
__device__ bool dotted_quad(const Rec& r, int i, int end) {
  for (int k = 0; k < 4; ++k) {
    const int e = octet(r, i);
    if (e < 0) return false;
    if (k == 3) return e == end;
    if (e >= end || r.at(e) != '.') return false;
    i = e + 1;
  }
  return false;
}

// The address text S = [p, s) is read group by group: 1-4 hex digits, a ':'
// after every group but the last, one "::" at most (standing for at least
// one zero group, so at most seven written groups), and a dotted quad, worth
// two groups, only as the text's last group.  An address text is at most 45
// bytes long, so a longer S is rejected while it is scanned.
__device__ int match_ipv6(const Rec& r, int p) {
  const uint8_t c0 = r.at(p);
  if (!is_hex(c0) && c0 != ':') return -1;
  if (p > r.lo) {
    const uint8_t c = r.at(p - 1);
    if (is_word(c) || c == ':' || c == '.') return -1;
  }
  // The first group has at most 4 hex digits and a ':' follows it (a lone
  // group or a dotted quad alone is no address), so hashes, IPv4 addresses
  // and words are rejected after at most 5 bytes.
  int e = p, s = p;
  bool colon = false;
  while (e < r.hi) {
    const uint8_t c = r.at(e);
    if (c == '.') {
      if (!colon) return -1;
      ++e;
      continue;
    }
    if (c == ':') colon = true;
    else if (!is_hex(c)) break;
    else if (!colon && e - p >= 4) return -1;
    s = ++e;
    if (s - p > 45) return -1;
  }
  if (!colon || !r.word_end(s)) return -1;
  int groups = 0;
  bool dbl = false;
  int i = p;
  if (c0 == ':') {
    if (s - p < 2 || r.at(p + 1) != ':') return -1;
    dbl = true;
    i = p + 2;
  }
  while (i < s) {
    int j = i;
    while (j < s && is_hex(r.at(j))) ++j;
    if (j < s && r.at(j) == '.') {
      if (!dotted_quad(r, i, s)) return -1;
      groups += 2;
      break;
    }
    if (j == i || j - i > 4) return -1;
    ++groups;
    i = j;
    if (i == s) break;
    ++i;  // the ':' after the group
    if (i == s) return -1;
    if (r.at(i) == ':') {
      if (dbl) return -1;
      dbl = true;
      if (++i == s) break;
    }
  }
  return (dbl ? groups <= 7 : groups == 8) ? s : -1;
}

constexpr int kRecognizers = kNumRecognizers;
constexpr int kTileWords = kTile / 64;
// matches of a tile: an anchor gives at most two, a 16-byte block and a record
// start (no anchor) one each
__host__ __device__ constexpr int64_t tile_entries(int64_t bytes) { return 2 * bytes + (bytes + 15) / 16; }
constexpr int kTileEntries = (int)tile_entries(kTile);
struct RecTypes {
  int t[kRecognizers];  // type index per recognizer, 0 = off
};

// 60-bit union key of a span: longest first, then lowest priority (NER 0,
// recognizer k -> k+1), then leftmost begin (offset inside the record); the
// low byte carries the type.
__device__ __forceinline__ unsigned long long span_key(int len, int prio, int local_begin, int type) {
  return ((unsigned long long)min(len, 0xFFFFFF) << 36) | ((unsigned long long)(15 - prio) << 32) |
         ((unsigned long long)(0xFFFFFF - min(local_begin, 0xFFFFFF)) << 8) | (unsigned long long)type;
}

// Record b's bytes, clamped to the text [0, n) (a malformed cu_bytes is
// flagged by rx_init_kernel and cannot send a read outside the text).
__device__ __forceinline__ void record_bounds(const int64_t* cu, int b, int64_t n, int& lo, int& hi) {
  const int64_t l = min(max(cu[b], (int64_t)0), n);
  lo = (int)l;
  hi = (int)min(max(cu[b + 1], l), n);
}

// Clears the bitmaps and checks cu_bytes: it must rise from 0 to n, and
// records must be shorter than 16 MiB (the union key holds lengths in 24
// bits).
__global__ __launch_bounds__(256) void rx_init_kernel(unsigned long long* maps, int64_t words,
                                                      const int64_t* __restrict__ cu, int B, int64_t n,
                                                      uint32_t* err) {
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = i0; i < words; i += (int64_t)gridDim.x * 256) maps[i] = 0;
  for (int64_t b = i0; b <= B; b += (int64_t)gridDim.x * 256) {
    const int64_t x = cu[b];
    if ((b == 0 && x != 0) || (b == B && x != n)) raise_error(err, ANON_ERR_TEXT);
    if (b < B && (cu[b + 1] < x || cu[b + 1] - x >= (int64_t(1) << 24))) raise_error(err, ANON_ERR_TEXT);
  }
}

// Span [b, e), e > b, into the bitmaps.
__device__ __forceinline__ void mark_span(const RecogBuffers& w, int b, int e) {
  atomicOr(&w.begins[b >> 6], 1ull << (b & 63));
  for (int i = b + 1; i < e;) {
    const int stop = word_stop(i, e);
    atomicOr(&w.joins[i >> 6], word_mask(i, stop));
    i = stop;
  }
}

// The same by a whole wave, a word per lane and step, where a span is long
// enough: an 8 MB one by a thread of its own took 9 ms.
constexpr int kLongSpan = 1024;
__device__ __forceinline__ void mark_long_span(const RecogBuffers& w, int b, int e, int lane) {
  if (lane == 0) atomicOr(&w.begins[b >> 6], 1ull << (b & 63));
  for (int word = ((b + 1) >> 6) + lane; word <= (e - 1) >> 6; word += 64) {
    const int i = max(b + 1, word * 64);
    atomicOr(&w.joins[word], word_mask(i, word_stop(i, e)));
  }
}

// An NER span's global [b, e); false (and the error bit) outside its record.
__device__ __forceinline__ bool ner_span(const anon_span& s, const int64_t* cu, int B, int64_t n, int n_types, int& b,
                                         int& e, uint32_t* err) {
  if (s.record < 0 || s.record >= B || s.type < 1 || s.type > n_types) {
    raise_error(err, ANON_ERR_SPAN);
    return false;
  }
  int lo, hi;
  record_bounds(cu, s.record, n, lo, hi);
  if (s.begin < 0 || s.end <= s.begin || s.end > hi - lo) {
    raise_error(err, ANON_ERR_SPAN);
    return false;
  }
  b = lo + (int)s.begin;
  e = lo + (int)s.end;
  return true;
}

// 16 bytes of text from p on (zeros past n)
__device__ __forceinline__ uint4 text16(const uint8_t* __restrict__ text, int64_t p, int64_t n) {
  if (n - p >= 16) return load16(text + p);
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (p + i < n) w[i >> 2] |= (uint32_t)text[p + i] << (8 * (i & 3));
  return uint4{w[0], w[1], w[2], w[3]};
}

// Class bits of 16 staged bytes (and of the anchors among them), four bytes at
// a time: the classes byte by byte took three times the instructions.
__device__ __forceinline__ uint32_t class_bits(const uint4& v, uint32_t (&m)[C_COUNT]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t anchors = 0;
#pragma unroll
  for (int k = 0; k < C_COUNT; ++k) m[k] = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t lower = w[i] | 0x20202020u;
    const uint32_t digit = bytes_between(w[i], '0', '9'), letter = bytes_between(lower, 'a', 'z');
    const uint32_t dash = bytes_equal(w[i], '-'), dot = bytes_equal(w[i], '.');
    const uint32_t label = digit | letter | dash;
    const uint32_t local = label | dot | bytes_equal(w[i], '_') | bytes_equal(w[i], '%') | bytes_equal(w[i], '+');
    const uint32_t space = bytes_equal(w[i], ' ') | bytes_between(w[i], '\t', '\r');
    m[C_LABEL] |= byte_bits(label) << (4 * i);
    m[C_LOCAL] |= byte_bits(local) << (4 * i);
    m[C_HEX] |= byte_bits(digit | bytes_between(lower, 'a', 'f')) << (4 * i);
    m[C_LETTER] |= byte_bits(letter) << (4 * i);
    m[C_TEXT] |= byte_bits(~space & 0x80808080u) << (4 * i);
    anchors |= byte_bits(dash | dot | bytes_equal(w[i], ':') | bytes_equal(w[i], '@')) << (4 * i);
  }
  return anchors;
}

constexpr int kBounds = 64;  // records of a tile whose boundaries are staged

// Blocks below n_tiles: the matches of a tile's anchors, stored in the tile's
// entry slots and marked in the bitmaps.  The blocks above: the NER spans.
// Each wave takes rules of its own (hostnames, IPv4, the ':' rules, the
// others), so that a wave's lanes run one rule's scan: with one list for all,
// every wave ran every rule's scan in turn (65 us for a lone tile).
__global__ __launch_bounds__(256) void rx_match_kernel(const uint8_t* __restrict__ text,
                                                       const int64_t* __restrict__ cu, int B, int64_t n, RecTypes rt,
                                                       int n_tiles, const anon_span* __restrict__ ner,
                                                       const int* __restrict__ ner_cu, int ner_cap, int n_types,
                                                       RecogBuffers w, uint32_t* err) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x >= n_tiles) {
    const int total = min(ner_cu[B], ner_cap);
    for (int64_t i0 = (int64_t)(blockIdx.x - n_tiles) * 256; i0 < total; i0 += (int64_t)(gridDim.x - n_tiles) * 256) {
      int b = 0, e = 0;
      const bool ok = i0 + tid < total && ner_span(ner[i0 + tid], cu, B, n, n_types, b, e, err);
      if (ok && e - b <= kLongSpan) mark_span(w, b, e);
      for (uint64_t m = __ballot(ok && e - b > kLongSpan); m; m &= m - 1) {
        const int of = __ffsll((unsigned long long)m) - 1;
        mark_long_span(w, __shfl(b, of, 64), __shfl(e, of, 64), lane);
      }
    }
    return;
  }
  // Anchor lists (offset within the tile, for the last list also the rule's
  // kind).  Every position is in one list at most, every 16-byte block's start
  // once more; only a malformed cu_bytes, whose records can start at one
  // byte, could fill them.
  enum { L_DOT, L_COLON, L_OTHER, L_COUNT };
  enum { K_AT, K_DASH, K_HEX, K_REC };
  constexpr int kDots = kTile / 2 + 1;  // a '.' after a LABEL byte
  constexpr int kList = kTile + kTile / 16;
  __shared__ __align__(16) uint8_t win[kWin];
  __shared__ __align__(16) uint64_t cls[C_COUNT][kWinWords];
  __shared__ uint16_t list[kDots + 2 * kList];
  __shared__ int n_list[L_COUNT], n_entries, bound[kBounds + 1];
  const int64_t p0 = (int64_t)blockIdx.x * kTile;
  const int base = (int)p0 - kBefore, wlo = max(base, 0), whi = (int)min(p0 + kTile + kAfter, n);
  uint32_t my_hex = 0, my_anchors = 0;
  auto stage = [&](int piece, const uint4& v) {  // 16 bytes and their class bits
    uint32_t m[C_COUNT];
    my_anchors = class_bits(v, m);
    my_hex = m[C_HEX];
    *(uint4*)(win + piece * 16) = v;
#pragma unroll
    for (int k = 0; k < C_COUNT; ++k) ((uint16_t*)cls[k])[piece] = (uint16_t)m[k];
  };
  // the text travels while the records of the tile's first and last byte are
  // looked for
  const uint4 mine = text16(text, p0 + tid * 16, n);
  const int halo = tid < kBefore / 16 ? tid : (kBefore + kTile) / 16 + tid - 64;  // (waves 0 and 1)
  const bool has_halo = tid < kBefore / 16 || (tid >= 64 && tid < 64 + kAfter / 16);
  uint4 other{0, 0, 0, 0};
  if (has_halo && p0 - kBefore + halo * 16 >= 0) other = text16(text, p0 - kBefore + halo * 16, n);
  if (tid < L_COUNT) n_list[tid] = 0;
  if (tid == 0) n_entries = 0;
  const int2 rr = wg_find_records(cu, B, p0, min(p0 + kTile, n) - 1);
  const int r0 = rr.x, r1 = max(rr.y, rr.x);
  if (has_halo) stage(halo, other);
  stage(kBefore / 16 + tid, mine);
  const bool few = r1 - r0 < kBounds;
  if (few && tid <= r1 - r0 + 1) bound[tid] = (int)min(max(cu[r0 + tid], (int64_t)0), n);
  __syncthreads();
  // anchors, with what their neighbours must be for any rule
  const uint8_t* me = win + kBefore + tid * 16;
  const auto first = [](int l) { return l == L_DOT ? 0 : kDots + (l - L_COLON) * kList; };
  const auto room = [](int l) { return l == L_DOT ? kDots : kList; };
  auto push = [&](int l, int v) {
    const int k = atomicAdd(&n_list[l], 1);
    if (k < room(l)) list[first(l) + k] = (uint16_t)v;
  };
  {
    for (uint32_t m = my_anchors; m; m &= m - 1) {
      const int i = __ffs(m) - 1, off = tid * 16 + i;
      const uint8_t c = me[i], prev = me[i - 1], next = me[i + 1];
      if (c == '.') {
        if (is_label(prev)) push(L_DOT, off);
      } else if (c == '@') {
        if (is_local(prev)) push(L_OTHER, off | (K_AT << 12));
      } else if (c == '-') {
        if (prev == 'E') push(L_OTHER, off | (K_DASH << 12));
      } else if (is_hex(prev) || next == ':' || ((prev == 'p' || prev == 's') && next == '/')) {
        push(L_COLON, off);
      }
    }
    if (my_hex == 0xffff && ((const uint16_t*)cls[C_HEX])[kBefore / 16 + tid - 1] != 0xffff)
      push(L_OTHER, (tid * 16) | (K_HEX << 12));
  }
  // record starts: a hash there may follow the last record's hex digits
  wg_each_record(cu, r0, r1, [&](int r) {
    const int64_t x = cu[r];
    if (x >= p0 && x < min(p0 + kTile, n) && cu[r + 1] > x && is_hex(win[kBefore + (x - p0)]))
      push(L_OTHER, (int)(x - p0) | (K_REC << 12));
  });
  __syncthreads();

  auto record = [&](int a) {  // of the anchor at byte a
    int x = r0, y = r1;
    while (x < y) {
      const int m = (x + y + 1) >> 1;
      if ((few ? (int64_t)bound[m - r0] : cu[m]) <= a) x = m;
      else y = m - 1;
    }
    int lo, hi;
    if (few) lo = bound[x - r0], hi = max(bound[x - r0 + 1], lo);
    else record_bounds(cu, x, n, lo, hi);
    return Rec{text, lo, hi, win, cls, base, wlo, whi};
  };
  const int entry_room = (int)tile_entries(min((int64_t)kTile, n - p0));
  auto emit = [&](const Rec& r, int rule, int p, int e) {
    if (e < 0) return;
    mark_span(w, p, e);
    const int slot = atomicAdd(&n_entries, 1);
    if (slot < entry_room)
      w.entries[(size_t)blockIdx.x * kTileEntries + slot] =
          RecogEntry{p, 0, span_key(e - p, 1 + rule, p - r.lo, rt.t[rule])};
  };
  const int li = wave < 2 ? (int)L_DOT : wave == 2 ? (int)L_COLON : (int)L_OTHER;
  const int nl = min(n_list[li], room(li));
  for (int k = lane; k < nl; k += 64) {
    const int v = list[first(li) + k], a = (int)p0 + (v & 0xfff);
    const Rec r = record(a);
    if (a < r.lo || a >= r.hi) continue;  // only with a malformed cu_bytes
    if (wave == 0) {
      const int s = r.run_begin<C_LABEL>(a);
      if (rt.t[6] && s < a) emit(r, 6, s, match_hostname(r, s));
    } else if (wave == 1) {
      int s = a;
      while (s > r.lo && a - s < 4 && is_digit(r.at(s - 1))) --s;
      if (rt.t[2] && s < a) emit(r, 2, s, match_ipv4(r, s));
    } else if (wave == 2) {
      const uint8_t prev = a > r.lo ? r.at(a - 1) : 0;
      if (rt.t[0] && prev == 'p' && a - r.lo >= 4) emit(r, 0, a - 4, match_url(r, a - 4));
      if (rt.t[0] && prev == 's' && a - r.lo >= 5) emit(r, 0, a - 5, match_url(r, a - 5));
      const int mac = a - r.lo >= 2 && is_hex(prev) ? match_mac(r, a - 2) : -1;
      if (rt.t[3]) emit(r, 3, a - 2, mac);
      // (six groups not followed by ':' are no address)
      if (rt.t[7] && !(mac >= 0 && (mac == r.hi || r.at(mac) != ':'))) {
        int s = a;
        while (s > r.lo && a - s < 5 && is_hex(r.at(s - 1))) --s;
        if (a - s < 5) emit(r, 7, s, match_ipv6(r, s));
      }
      if (rt.t[8] && prev == 'e' && a - r.lo >= 3) emit(r, 8, a - 3, match_cpe(r, a - 3));
    } else {
      const int kind = v >> 12;
      if (kind == K_AT) {
        const int s = r.run_begin<C_LOCAL>(a);
        if (rt.t[1] && s < a) emit(r, 1, s, match_email(r, s));
      } else if (kind == K_DASH) {
        if (rt.t[5] && a - r.lo >= 3) emit(r, 5, a - 3, match_cve(r, a - 3));
      } else if (rt.t[4]) {
        const int s = kind == K_HEX ? r.run_begin<C_HEX>(a) : r.lo;
        emit(r, 4, s, match_hash(r, s));
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    w.n_entries[blockIdx.x] = min(n_entries, entry_room);
    w.rec0[blockIdx.x] = r0;
  }
}

// A wave per tile: its unions' begins (left in `begins`), their rank within
// the tile at every 64-byte word, their count, and their keys cleared.
__global__ __launch_bounds__(256) void rx_count_kernel(RecogBuffers w, int n_tiles, int64_t words) {
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (tile >= n_tiles) return;
  const int64_t i = (int64_t)tile * kTileWords + lane;
  unsigned long long u = 0;
  if (i < words) w.begins[i] = u = w.begins[i] & ~w.joins[i];
  const int c = __popcll(u);
  int x = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (i < words) w.word_rank[i] = (uint16_t)(x - c);
  const int total = __shfl(x, 63, 64);
  if (lane == 0) w.tile_count[tile] = total;
  for (int k = lane; k < total; k += 64) w.keys[(size_t)tile * kTile + k] = 0;
}

// The unions of p's tile that begin at or before byte p: the rank, counted from
// 1, of the union that holds p; 0 if it began in an earlier tile.
__device__ __forceinline__ int union_rank(const RecogBuffers& w, int p) {
  const unsigned long long u = w.begins[p >> 6] & (~0ull >> (63 - (p & 63)));
  return w.word_rank[p >> 6] + __popcll(u);
}

// The key slot of the union that holds byte p.
__device__ __forceinline__ size_t union_slot(const RecogBuffers& w, int p) {
  int tile = p / kTile, k = union_rank(w, p);
  while (k == 0 && tile > 0) k = w.tile_count[--tile];
  return (size_t)tile * kTile + max(k - 1, 0);
}

// The last tile before `tile` where a union begins, -1 if there is none, by a
// whole wave, 64 tiles a step.
__device__ __forceinline__ int last_begin_tile(const RecogBuffers& w, int tile, int lane) {
  for (int top = tile; top > 0; top -= 64) {
    const int t = top - 1 - lane;
    const uint64_t some = __ballot(t >= 0 && w.tile_count[max(t, 0)] > 0);
    if (some) return top - __ffsll((unsigned long long)some);
  }
  return -1;
}

// Block 0: the prefix of the tiles' union counts.  The next blocks: every
// match's key into its union, a wave per tile.  The rest: the NER spans' keys.
// A tile's matches before its first union's begin are in one union, which
// began in an earlier tile: that tile is looked for once, and one atomic takes
// their largest key.  (64 tiles to a workgroup left most CUs idle on dense
// text: 1.2 MB of IPv6 addresses of three bytes 228 us, of IPv4 addresses 112.)
__global__ __launch_bounds__(256) void rx_members_kernel(const int64_t* __restrict__ cu, int B, int64_t n, int n_tiles,
                                                         int entry_blocks, const anon_span* __restrict__ ner,
                                                         const int* __restrict__ ner_cu, int ner_cap, int n_types,
                                                         RecogBuffers w) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (blockIdx.x == 0) {
    __shared__ int pre[257];
    const int per = (n_tiles + 255) / 256, a = min(n_tiles, tid * per), b = min(n_tiles, a + per);
    int s = 0;
    for (int i = a; i < b; ++i) s += w.tile_count[i];
    pre[tid + 1] = s;
    if (tid == 0) pre[0] = 0;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
      const int x = tid >= o ? pre[tid + 1 - o] : 0;
      __syncthreads();
      pre[tid + 1] += x;
      __syncthreads();
    }
    int run = pre[tid];
    for (int i = a; i < b; ++i) {
      w.tile_pre[i] = run;
      run += w.tile_count[i];
    }
    if (tid == 0) w.tile_pre[n_tiles] = pre[256];
    return;
  }
  if ((int)blockIdx.x <= entry_blocks) {
    const int tile = (blockIdx.x - 1) * 4 + (tid >> 6);
    if (tile >= n_tiles) return;
    const int total = w.n_entries[tile];
    unsigned long long earlier = 0;  // of the union that began before the tile
    for (int i = lane; i < total; i += 64) {
      const RecogEntry e = w.entries[(size_t)tile * kTileEntries + i];
      if (e.p / kTile == tile && union_rank(w, e.p) == 0) earlier = max(earlier, e.key);
      else atomicMax(&w.keys[union_slot(w, e.p)], e.key);  // (a match may begin before its anchor's tile)
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) earlier = max(earlier, (unsigned long long)__shfl_xor(earlier, o, 64));
    if (earlier) {
      const int t = last_begin_tile(w, tile, lane);
      if (lane == 0 && t >= 0) atomicMax(&w.keys[(size_t)t * kTile + w.tile_count[t] - 1], earlier);
    }
    return;
  }
  const int total = min(ner_cu[B], ner_cap);
  const int first = entry_blocks + 1;
  for (int64_t i = (int64_t)(blockIdx.x - first) * 256 + tid; i < total; i += (int64_t)(gridDim.x - first) * 256) {
    const anon_span s = ner[i];
    int b, e;
    if (!ner_span(s, cu, B, n, n_types, b, e, nullptr)) continue;
    atomicMax(&w.keys[union_slot(w, b)], span_key(e - b, 0, (int)s.begin, s.type));
  }
}

// A wave per tile writes its unions as spans, their records looked for among
// the tile's (in all 4096: 8 us of a call, now 4.5); the blocks above write
// cu_spans[b] = unions beginning before record b's first byte.
__global__ __launch_bounds__(256) void rx_emit_kernel(const int64_t* __restrict__ cu, int B, int64_t n, int n_tiles,
                                                      int tile_blocks, RecogBuffers w, int64_t words, anon_span* out,
                                                      int cap, int* cu_spans, uint32_t* err) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= tile_blocks) {
    const int b = (blockIdx.x - tile_blocks) * 256 + tid;
    if (b > B) return;
    const int total = w.tile_pre[n_tiles];
    const int64_t x = b == B ? n : min(max(cu[b], (int64_t)0), n);
    cu_spans[b] = x == n ? total
                         : w.tile_pre[x / kTile] + w.word_rank[x >> 6] +
                               __popcll(w.begins[x >> 6] & ((1ull << (x & 63)) - 1));
    if (b == B && total > cap) raise_error(err, ANON_ERR_SPAN_CAP);
    return;
  }
  const int tile = blockIdx.x * 4 + (tid >> 6), lane = tid & 63;
  const int64_t i = (int64_t)tile * kTileWords + lane;
  if (tile >= n_tiles) return;
  unsigned long long u = i < words ? w.begins[i] : 0;
  int k = i < words ? w.word_rank[i] : 0, b = w.rec0[tile];
  const int last = tile + 1 < n_tiles ? w.rec0[tile + 1] : B - 1;
  int64_t next = -1;  // the first byte past record b
  auto write = [&](int p, int e) {
    if (next <= p) {  // largest index of [b, last] with cu <= p
      int top = last;
      while (b < top) {
        const int m = (b + top + 1) >> 1;
        if (cu[m] <= p) b = m;
        else top = m - 1;
      }
      next = cu[b + 1];
    }
    out[w.tile_pre[tile] + k] =
        anon_span{b, (int)(w.keys[(size_t)tile * kTile + k] & 0xff), p - cu[b], e - cu[b]};
  };
  int far = -1;  // where the end of a long union, the word's last, is yet to be looked for
  for (; u; u &= u - 1, ++k) {
    if (w.tile_pre[tile] + k >= cap) break;
    const int p = (int)(i * 64) + __ffsll(u) - 1;
    // its end: the first byte after p not joined to the one before it
    int j = (p + 1) >> 6;
    unsigned long long open = ~w.joins[j] & (~0ull << ((p + 1) & 63));
    for (int more = 0; open == 0 && more < 3; ++more) open = ~w.joins[++j];
    if (open == 0) {
      far = j + 1;
      break;
    }
    write(p, j * 64 + __ffsll(open) - 1);
  }
  for (uint64_t m = __ballot(far >= 0); m; m &= m - 1) {
    // by the whole wave, 64 words a step (the text's last word is not all
    // joined); one after the other, an 8 MB union's took 11 ms
    const int of = __ffsll((unsigned long long)m) - 1;
    for (int j0 = __shfl(far, of, 64); j0 < words; j0 += 64) {
      const unsigned long long open = j0 + lane < words ? ~w.joins[j0 + lane] : 0;
      const uint64_t some = __ballot(open != 0);
      if (!some) continue;
      const int at = __ffsll((unsigned long long)some) - 1;
      const int e = (j0 + at) * 64 + __shfl(__ffsll(open) - 1, at, 64);
      if (lane == of) write((int)(i * 64) + __ffsll(u) - 1, e);
      break;
    }
  }
}

}  // namespace

static int64_t recog_tiles(int64_t n) { return (n + kTile - 1) / kTile; }
static int64_t recog_words(int64_t n) { return n / 64 + 1; }  // a bit per byte and one past the end

size_t recog_workspace_bytes(int64_t n) {
  Carver k(nullptr, SIZE_MAX);
  recog_layout(n, k);
  return k.used + 256;
}

RecogBuffers recog_layout(int64_t n, Carver& k) {
  const int64_t tiles = recog_tiles(n), words = recog_words(n);
  RecogBuffers w;
  w.begins = k.take<unsigned long long>(2 * words);
  w.joins = w.begins + words;
  w.word_rank = k.take<uint16_t>(words);
  w.n_entries = k.take<int>(tiles + 1);
  w.tile_count = k.take<int>(tiles + 1);
  w.tile_pre = k.take<int>(tiles + 1);
  w.rec0 = k.take<int>(tiles + 1);
  w.keys = k.take<unsigned long long>(n);
  w.entries = k.take<RecogEntry>(tiles > 0 ? (tiles - 1) * kTileEntries + tile_entries(n - (tiles - 1) * kTile) : 0);
  return w;
}

void launch_recognize(const uint8_t* text, const int64_t* cu_bytes, int B, int64_t n,
                      const int rec_types[kNumRecognizers],
                      const anon_span* ner, const int* ner_cu, int ner_cap, int n_types, const RecogBuffers& w,
                      anon_span* out, int cap, int* cu_spans, uint32_t* err, hipStream_t s) {
  RecTypes rt;
  for (int k = 0; k < kRecognizers; ++k) rt.t[k] = rec_types[k];
  const int tiles = (int)recog_tiles(n);
  const int64_t words = recog_words(n);
  const bool have_ner = ner && ner_cu && ner_cap > 0;
  // the NER spans' count is on the device: enough blocks for it in a few
  // rounds, and none that idles in its thousands when the capacity is large
  const int ner_blocks = have_ner ? std::min(ceil_div(ner_cap, 256), 1024) : 0;
  const int tile_blocks = ceil_div(tiles, 4);
  hipLaunchKernelGGL(rx_init_kernel, dim3(std::max(1, std::min(ceil_div(std::max<int64_t>(2 * words, B + 1), 256), 2048))),
                     dim3(256), 0, s, w.begins, 2 * words, cu_bytes, B, n, err);
  if (tiles + ner_blocks > 0)
    hipLaunchKernelGGL(rx_match_kernel, dim3(tiles + ner_blocks), dim3(256), 0, s, text, cu_bytes, B, n, rt, tiles,
                       ner, ner_cu, ner_cap, n_types, w, err);
  if (tiles > 0)
    hipLaunchKernelGGL(rx_count_kernel, dim3(tile_blocks), dim3(256), 0, s, w, tiles, words);
  hipLaunchKernelGGL(rx_members_kernel, dim3(1 + tile_blocks + (tiles > 0 ? ner_blocks : 0)), dim3(256), 0, s,
                     cu_bytes, B, n, tiles, tile_blocks, ner, ner_cu, ner_cap, n_types, w);
  hipLaunchKernelGGL(rx_emit_kernel, dim3(tile_blocks + ceil_div(B + 1, 256)), dim3(256), 0, s, cu_bytes, B, n, tiles,
                     tile_blocks, w, words, out, cap, cu_spans, err);
}

}  // namespace anon
