// Schema-aware whole-field spans without NER: the paper's configuration that
// maps named fields straight to pseudonyms and bypasses inference (Sec. II;
// Sec. IV-A; App. C, Table VI with and without the configuration).
//
// Records are "Field: value" lines.  A line (a maximal run of bytes without
// '\n', never crossing a record boundary) holds a field if its first ':' is
// directly followed by ' '; the name is the bytes before the ':', the value
// the bytes after ": " up to the end of the line.  A configured name with a
// non-empty value gives one span of the configured type over the value.
//
// A workgroup takes 8192 bytes, 32 per thread, staged in LDS with the 448
// after them, and keeps '\n', ':' and record starts as bitmaps: a line's
// colon and a value's end are one count of trailing zeros away.  The lines
// are listed, so that whole waves of them are looked at, and a name is looked
// up by a key of its eight dwords.  A tile's fields are stored in byte order,
// which is record-major; the tiles' counts are scanned, and a wave per tile
// writes the spans.
//
// Bound by instructions (three quarters of the match's time is vector issue):
// one read of the text and 16 bytes per field, where a thread per byte read
// three bytes each, wrote an int flag, scanned the flags in three kernels and
// tested every line a second time.  128 MB in 16,384 records: 4.8 ms -> 0.11
// ms, 91 us of it the match (16 bytes a thread, lines taken where they began
// and every name compared in full: 215).
#include <algorithm>

#include "kernels.hpp"

namespace anon {
namespace {

constexpr int kTile = 8192;
constexpr int kAfter = 448;                 // staged past the tile
constexpr int kWin = kTile + kAfter;
constexpr int kWinWords = kWin / 64;
constexpr int kTileFields = kTile / 4;      // (a field has 4 bytes at least: "x: v")

__device__ __forceinline__ int find_in(const int64_t* cu, int a, int c, int64_t p) {
  while (a < c) {  // largest index of [a, c] with cu <= p
    const int m = (a + c + 1) >> 1;
    if (cu[m] <= p) a = m;
    else c = m - 1;
  }
  return a;
}

// First set bit at or after o of two bitmaps of the window, kWin if none.
__device__ __forceinline__ int next_bit(const uint64_t* x, const uint64_t* y, int o) {
  for (int w = o >> 6; w < kWinWords; ++w) {
    uint64_t v = x[w] | y[w];
    if (w == o >> 6) v &= ~0ull << (o & 63);
    if (v) return w * 64 + __ffsll((unsigned long long)v) - 1;
  }
  return kWin;
}

// 64 bits from o on of two bitmaps of the window, o < kTile + 1.
__device__ __forceinline__ uint64_t bits_from(const uint64_t* x, const uint64_t* y, int o) {
  const int w = o >> 6, s = o & 63;
  const uint64_t lo = x[w] | y[w], hi = x[w + 1] | y[w + 1];
  return s ? lo >> s | hi << (64 - s) : lo;
}

__global__ __launch_bounds__(256) void fd_match_kernel(const uint8_t* __restrict__ text,
                                                       const int64_t* __restrict__ cu, int B, int64_t n,
                                                       FieldTable ft, FieldBuffers out) {
  __shared__ __align__(16) uint8_t win[kWin + 48];  // (names are read as 36 bytes)
  __shared__ __align__(16) uint64_t nl[kWinWords], colon[kWinWords], rec[kWinWords];
  __shared__ uint16_t lines[kTile];
  __shared__ int ws[4];
  const int tid = threadIdx.x;
  const int64_t p0 = (int64_t)blockIdx.x * kTile;
  const int whi = (int)min((int64_t)kWin, n - p0);  // staged bytes of text
  auto load = [&](int piece) {
    const int64_t p = p0 + piece * 16;
    if (n - p >= 16) return load16(text + p);
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (p + i < n) w[i >> 2] |= (uint32_t)text[p + i] << (8 * (i & 3));
    return uint4{w[0], w[1], w[2], w[3]};
  };
  auto stage = [&](int piece, uint4 v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t mn = 0, mc = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mn |= byte_bits(bytes_equal(w[i], '\n')) << (4 * i);
      mc |= byte_bits(bytes_equal(w[i], ':')) << (4 * i);
    }
    *(uint4*)(win + piece * 16) = uint4{w[0], w[1], w[2], w[3]};
    ((uint16_t*)nl)[piece] = (uint16_t)mn;
    ((uint16_t*)colon)[piece] = (uint16_t)mc;
    ((uint16_t*)rec)[piece] = 0;
    return mn;
  };
  // the text and the byte before this thread's (a line break there starts a
  // line) travel while the record of the tile's first byte is looked for
  const int64_t mine = p0 + tid * 32;
  const uint4 v0 = load(2 * tid), v1 = load(2 * tid + 1);
  const uint4 v2 = tid < kAfter / 16 ? load(kTile / 16 + tid) : uint4{0, 0, 0, 0};
  const uint8_t before = mine > 0 && mine < n ? text[mine - 1] : 0;
  const int r0 = wg_find_record(cu, B, p0);
  uint32_t my_nl = stage(2 * tid, v0);
  my_nl |= stage(2 * tid + 1, v1) << 16;
  if (tid < kAfter / 16) stage(kTile / 16 + tid, v2);
  const bool after_break = before == '\n';
  __syncthreads();
  // record starts of the window
  wg_each_record_to(cu, B, r0, p0 + whi - 1, [&](int b) {
    const int64_t c = cu[b];
    if (c >= p0 && c < p0 + whi) atomicOr((uint32_t*)rec + ((c - p0) >> 5), 1u << ((c - p0) & 31));
  });
  uint32_t starts = (my_nl << 1) | (after_break ? 1u : 0u) | ((const uint32_t*)rec)[tid];
  if (mine == 0) starts |= 1;  // the text's first byte
  starts &= ~my_nl;            // (an empty line)
  if (n - mine < 32) starts &= n > mine ? (1u << (n - mine)) - 1 : 0;
  // the field of the line that begins at byte o of the tile (type 0: none)
  auto field_of = [&](int o) {
    const FieldEntry none{0, 0, 0, 0};
    // the name ends at a ':' before any line break or record start after it:
    // all within 64 bytes, two words (searched for to the window's end, 4.9 MB
    // of lines of one byte without a ':' took 139 us a call, now 22)
    const uint64_t at_colon = bits_from(colon, colon, o), at_stop = bits_from(nl, rec, o + 1);
    const int len = at_colon ? __ffsll((unsigned long long)at_colon) - 1 : 64, c = o + len;
    const int room = at_stop ? __ffsll((unsigned long long)at_stop) : 65;  // the line's bytes, as far as seen
    if (len > kFieldNameMax || len >= room || c + 1 >= whi || win[c + 1] != ' ' || room == len + 1) return none;
    uint32_t d[kFieldNameMax / 4];
    const uint32_t* q = (const uint32_t*)(win + (o & ~3));
    uint32_t lo = q[0];
#pragma unroll
    for (int i = 0; i < kFieldNameMax / 4; ++i) {
      const uint32_t hi = q[i + 1];
      const uint32_t v = __builtin_amdgcn_alignbyte(hi, lo, o & 3);
      const int left = len - 4 * i;
      d[i] = left >= 4 ? v : left <= 0 ? 0 : v & ((1u << (8 * left)) - 1);
      lo = hi;
    }
    // the first of equal names, as configured: by the names' keys, the whole
    // name only where a key is equal (another name's key: the next equal one)
    const uint32_t key = field_key(d, len);
    int type = 0;
    for (int from = 0; from < ft.n && !type;) {
      int hit = kFieldsMax;
      for (int k = ft.n - 1; k >= 0; --k)
        if (ft.key[k] == key && k >= from) hit = k;
      if (hit == kFieldsMax) break;
      uint32_t diff = ft.len[hit] ^ len;
#pragma unroll
      for (int i = 0; i < kFieldNameMax / 4; ++i) diff |= ((const uint32_t*)ft.name[hit])[i] ^ d[i];
      if (diff == 0) type = ft.type[hit];
      from = hit + 1;
    }
    if (!type) return none;
    // the value: up to the next line break, record start or the text's end
    const int vb = c + 2, stop = next_bit(nl, rec, vb);
    int64_t ve = stop;
    if (stop >= whi) {
      ve = p0 + whi;  // past the window, byte by byte inside the record
      if (ve < n) {
        const int64_t hi = min(max(cu[find_in(cu, r0, B - 1, p0 + o) + 1], ve), n);
        while (ve < hi && text[ve] != '\n') ++ve;
      }
      ve -= p0;
    }
    if (ve <= vb) return none;
    return FieldEntry{(int)p0 + o, (int)(p0 + vb), (int)(p0 + ve), type};
  };
  // the lines' first bytes, in order
  const int lane = tid & 63, wave = tid >> 6;
  {
    const int own = __popc(starts);
    int x = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    int at = x - own;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (w < wave) at += ws[w];
    for (; starts; starts &= starts - 1) lines[at++] = (uint16_t)(tid * 32 + __ffs(starts) - 1);
  }
  const int n_lines = ws[0] + ws[1] + ws[2] + ws[3];
  int total = 0;  // fields found so far
  FieldEntry* to = out.entries + (size_t)blockIdx.x * kTileFields;
  const int room = (int)min((int64_t)kTileFields, (n - p0 + 3) / 4);
  __syncthreads();
  for (int l0 = 0; l0 < n_lines; l0 += 256) {
    FieldEntry f{0, 0, 0, 0};
    if (l0 + tid < n_lines) f = field_of(lines[l0 + tid]);
    const uint64_t some = __ballot(f.type > 0);
    if (lane == 0) ws[wave] = __popcll((unsigned long long)some);
    __syncthreads();
    int at = total + __popcll((unsigned long long)(some & ((1ull << lane) - 1)));
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w < wave) at += ws[w];
      total += ws[w];
    }
    if (f.type > 0 && at < room) to[at] = f;
    __syncthreads();
  }
  if (tid == 0) {
    out.counts[blockIdx.x] = min(total, room);
    out.rec0[blockIdx.x] = r0;
  }
}

// A wave per tile writes its spans (pre: exclusive prefix of the tiles'
// counts); the blocks above check cu_bytes and write cu_spans[b] = fields
// before record b.
__global__ __launch_bounds__(256) void fd_emit_kernel(const int64_t* __restrict__ cu, int B, int64_t n, int n_tiles,
                                                      int tile_blocks, FieldBuffers w, anon_span* out, int cap,
                                                      int* cu_spans, uint32_t* err) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= tile_blocks) {
    const int b = (blockIdx.x - tile_blocks) * 256 + tid;
    if (b > B) return;
    const int64_t c = cu[b], x = min(max(c, (int64_t)0), n);
    if ((b == 0 && c != 0) || (b == B && c != n) || (b < B && cu[b + 1] < c)) raise_error(err, ANON_ERR_TEXT);
    const int total = w.counts[n_tiles], tile = (int)(x / kTile);
    int k = total;
    if (x < n) {
      const FieldEntry* e = w.entries + (size_t)tile * kTileFields;
      int a = 0, c = w.counts[tile + 1] - w.counts[tile];  // first entry at or after x
      while (a < c) {
        const int m = (a + c) >> 1;
        if (e[m].line < x) a = m + 1;
        else c = m;
      }
      k = w.counts[tile] + a;
    }
    cu_spans[b] = k;
    if (b == B && total > cap) raise_error(err, ANON_ERR_SPAN_CAP);
    return;
  }
  const int tile = blockIdx.x * 4 + (tid >> 6), lane = tid & 63;
  if (tile >= n_tiles) return;
  const int first = w.counts[tile], cnt = w.counts[tile + 1] - first;
  const int ra = w.rec0[tile], rb = tile + 1 < n_tiles ? w.rec0[tile + 1] : B - 1;
  for (int i = lane; i < cnt && first + i < cap; i += 64) {
    const FieldEntry e = w.entries[(size_t)tile * kTileFields + i];
    const int r = find_in(cu, ra, rb, e.line);
    out[first + i] = anon_span{r, e.type, e.begin - cu[r], e.end - cu[r]};
  }
}

}  // namespace

FieldBuffers field_layout(int64_t n, Carver& k) {
  const int64_t tiles = (n + kTile - 1) / kTile;
  FieldBuffers w;
  w.entries = k.take<FieldEntry>((n + 3) / 4);
  w.counts = k.take<int>(tiles + 1);
  w.rec0 = k.take<int>(tiles + 1);
  return w;
}

size_t field_workspace_bytes(int64_t n) {
  Carver k(nullptr, SIZE_MAX);
  field_layout(n, k);
  return k.used + 256;
}

// An empty text has no tile.
__global__ void fd_empty_kernel(int* counts) { counts[0] = 0; }

void launch_field_spans(const uint8_t* text, const int64_t* cu_bytes, int B, int64_t n, const FieldTable& ft,
                        const FieldBuffers& w, anon_span* out, int cap, int* cu_spans, uint32_t* err,
                        hipStream_t s) {
  const int tiles = (int)((n + kTile - 1) / kTile), tile_blocks = ceil_div(tiles, 4);
  if (tiles > 0) {
    hipLaunchKernelGGL(fd_match_kernel, dim3(tiles), dim3(256), 0, s, text, cu_bytes, B, n, ft, w);
    launch_scan_counts(w.counts, tiles, s);
  } else {
    hipLaunchKernelGGL(fd_empty_kernel, dim3(1), dim3(1), 0, s, w.counts);
  }
  hipLaunchKernelGGL(fd_emit_kernel, dim3(tile_blocks + ceil_div(B + 1, 256)), dim3(256), 0, s, cu_bytes, B, n, tiles,
                     tile_blocks, w, out, cap, cu_spans, err);
}

}  // namespace anon
