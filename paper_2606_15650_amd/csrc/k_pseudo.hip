// Pseudonym substitution on the GPU (the paper's Sec. II stage 3).
//
// Every entity span is replaced by "[" TYPE "_" slug "]", slug = the first n
// lowercase hex digits of HMAC-SHA256(key, entity bytes).  HMAC (RFC 2104)
// is computed with the SHA-256 states after the key^ipad and key^opad blocks
// precomputed once per key, so a message of up to 55 bytes costs two
// compressions.  A device hash table (open addressing, insert-only) caches
// entity bytes -> digest across calls; because the digest is a pure function
// of the bytes, a lost insert race or a full table only costs a recompute and
// never changes the output.
//
// Substitution is two-pass: a per-record pass validates the spans and lays
// out each pseudonym's output offset and the record's output length, a scan
// turns lengths into output offsets, and a per-record block writes every
// output byte (copied text or pseudonym character) at its final position.
#include <algorithm>

#include "kernels.hpp"

namespace anon {

// FIPS 180-4 Sec. 4.2.2 round constants and Sec. 5.3.3 initial hash value.
#define ANON_SHA256_K                                                                                         \
  {0x428a2f98u, 0x71374491u, 0xb5c0fbcfu, 0xe9b5dba5u, 0x3956c25bu, 0x59f111f1u, 0x923f82a4u, 0xab1c5ed5u, \
   0xd807aa98u, 0x12835b01u, 0x243185beu, 0x550c7dc3u, 0x72be5d74u, 0x80deb1feu, 0x9bdc06a7u, 0xc19bf174u, \
   0xe49b69c1u, 0xefbe4786u, 0x0fc19dc6u, 0x240ca1ccu, 0x2de92c6fu, 0x4a7484aau, 0x5cb0a9dcu, 0x76f988dau, \
   0x983e5152u, 0xa831c66du, 0xb00327c8u, 0xbf597fc7u, 0xc6e00bf3u, 0xd5a79147u, 0x06ca6351u, 0x14292967u, \
   0x27b70a85u, 0x2e1b2138u, 0x4d2c6dfcu, 0x53380d13u, 0x650a7354u, 0x766a0abbu, 0x81c2c92eu, 0x92722c85u, \
   0xa2bfe8a1u, 0xa81a664bu, 0xc24b8b70u, 0xc76c51a3u, 0xd192e819u, 0xd6990624u, 0xf40e3585u, 0x106aa070u, \
   0x19a4c116u, 0x1e376c08u, 0x2748774cu, 0x34b0bcb5u, 0x391c0cb3u, 0x4ed8aa4au, 0x5b9cca4fu, 0x682e6ff3u, \
   0x748f82eeu, 0x78a5636fu, 0x84c87814u, 0x8cc70208u, 0x90befffau, 0xa4506cebu, 0xbef9a3f7u, 0xc67178f2u}

namespace {

constexpr uint32_t kH0[8] = {0x6a09e667u, 0xbb67ae85u, 0x3c6ef372u, 0xa54ff53au,
                             0x510e527fu, 0x9b05688cu, 0x1f83d9abu, 0x5be0cd19u};

__host__ __device__ __forceinline__ uint32_t rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }

// One SHA-256 compression of the 16 big-endian words w into state st.
__host__ __device__ inline void sha256_compress(uint32_t st[8], const uint32_t win[16]) {
  constexpr uint32_t K[64] = ANON_SHA256_K;
  uint32_t w[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) w[i] = win[i];
  uint32_t a = st[0], b = st[1], c = st[2], d = st[3], e = st[4], f = st[5], g = st[6], h = st[7];
#pragma unroll
  for (int i = 0; i < 64; ++i) {
    uint32_t wi;
    if (i < 16) {
      wi = w[i];
    } else {
      const uint32_t x15 = w[(i + 1) & 15], x2 = w[(i + 14) & 15];
      const uint32_t s0 = rotr(x15, 7) ^ rotr(x15, 18) ^ (x15 >> 3);
      const uint32_t s1 = rotr(x2, 17) ^ rotr(x2, 19) ^ (x2 >> 10);
      wi = w[i & 15] = w[i & 15] + s0 + w[(i + 9) & 15] + s1;
    }
    const uint32_t S1 = rotr(e, 6) ^ rotr(e, 11) ^ rotr(e, 25);
    const uint32_t ch = (e & f) ^ (~e & g);
    const uint32_t t1 = h + S1 + ch + K[i] + wi;
    const uint32_t S0 = rotr(a, 2) ^ rotr(a, 13) ^ rotr(a, 22);
    const uint32_t mj = (a & b) ^ (a & c) ^ (b & c);
    const uint32_t t2 = S0 + mj;
    h = g;
    g = f;
    f = e;
    e = d + t1;
    d = c;
    c = b;
    b = a;
    a = t1 + t2;
  }
  st[0] += a;
  st[1] += b;
  st[2] += c;
  st[3] += d;
  st[4] += e;
  st[5] += f;
  st[6] += g;
  st[7] += h;
}

// SHA-256 continued from `st` (which has already absorbed `prefix` bytes)
// over msg[0..len); the final state is left in st.
__host__ __device__ inline void sha256_tail(uint32_t st[8], uint64_t prefix, const uint8_t* msg, int64_t len) {
  uint32_t w[16];
  int64_t pos = 0;
  while (len - pos >= 64) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      w[i] = ((uint32_t)msg[pos + 4 * i] << 24) | ((uint32_t)msg[pos + 4 * i + 1] << 16) |
             ((uint32_t)msg[pos + 4 * i + 2] << 8) | (uint32_t)msg[pos + 4 * i + 3];
    sha256_compress(st, w);
    pos += 64;
  }
  const int rem = (int)(len - pos);
  const uint64_t bits = (prefix + (uint64_t)len) * 8u;
  // final one or two blocks: remaining bytes, 0x80, zeros, 64-bit length
  const int nblk = rem < 56 ? 1 : 2;
  for (int blk = 0; blk < nblk; ++blk) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      uint32_t v = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = blk * 64 + 4 * i + j;
        uint32_t byte = 0;
        if (k < rem) byte = msg[pos + k];
        else if (k == rem) byte = 0x80;
        v = (v << 8) | byte;
      }
      w[i] = v;
    }
    if (blk == nblk - 1) {
      w[14] = (uint32_t)(bits >> 32);
      w[15] = (uint32_t)bits;
    }
    sha256_compress(st, w);
  }
}

__device__ __forceinline__ void hmac_outer(const PcacheDev& pc, const uint32_t (&st)[8], uint32_t out[8]) {
  uint32_t w[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) w[i] = st[i];
  w[8] = 0x80000000u;
#pragma unroll
  for (int i = 9; i < 15; ++i) w[i] = 0;
  w[15] = (64 + 32) * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = pc.opad[i];
  sha256_compress(out, w);
}

__device__ inline void hmac_sha256(const PcacheDev& pc, const uint8_t* msg, int64_t len, uint32_t out[8]) {
  uint32_t st[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = pc.ipad[i];
  sha256_tail(st, 64, msg, len);
  hmac_outer(pc, st, out);
}

constexpr int kMaxEntity = 96;
constexpr int kMsgWords = kMaxEntity / 4;

// HMAC of an entity of at most kMaxEntity bytes held in registers (m: its
// bytes, little-endian dwords, zeros past len).
__device__ inline void hmac_words(const PcacheDev& pc, const uint32_t (&m)[kMsgWords], int len, uint32_t out[8]) {
  uint32_t st[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = pc.ipad[i];
  // the padded message: m, 0x80, zeros, the bit count in the last block's end
  auto word = [&](int i) {  // i a constant after unrolling
    const uint32_t v = i < kMsgWords ? m[i] : 0;
    const uint32_t pad = (len >> 2) == i ? 0x80u << (8 * (len & 3)) : 0;
    return __builtin_bswap32(v | pad);
  };
  // the blocks of the message, then the outer one, by one compression's code
  // (a copy of it for each is more than the instruction cache holds)
  const int blocks = len < 56 ? 1 : 2;
#pragma unroll 1
  for (int blk = 0; blk <= blocks; ++blk) {
    const bool outer = blk == blocks;
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t pad = i == 8 ? 0x80000000u : i == 15 ? (64 + 32) * 8 : 0;
      w[i] = outer ? (i < 8 ? st[i & 7] : pad) : blk == 0 ? word(i) : word(16 + i);
    }
    if (blk == blocks - 1) w[15] = (64 + (uint32_t)len) * 8;
    if (outer) {
#pragma unroll
      for (int i = 0; i < 8; ++i) st[i] = pc.opad[i];
    }
    sha256_compress(st, w);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = st[i];
}

// Table entry: state, length, fingerprint, entity bytes, digest, and for the
// mapping export the smallest type the entity was pseudonymized under and the
// first and last call that met it.
struct __align__(16) Entry {
  uint32_t state;  // 0 empty, 1 being written, 2 ready; above them 30 bits of fp
  uint32_t len;
  uint64_t fp;
  uint8_t bytes[kMaxEntity];
  uint32_t digest[8];
  int32_t type;
  uint32_t first, last, pad;
};
static_assert(sizeof(Entry) == 160 && sizeof(Entry) == sizeof(PcacheEntryView), "entry layout");

__device__ __forceinline__ bool preserved(const PcacheDev& pc, int type) {
  return (pc.preserve[(type >> 5) & 3] >> (type & 31)) & 1u;
}

// A later meeting of a ready entry: keep the smallest type and the last call
// (read first: most meetings of a popular entity change neither).
__device__ __forceinline__ void touch(Entry* e, int type, uint32_t call) {
  if (__hip_atomic_load(&e->type, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > type) atomicMin(&e->type, type);
  if (__hip_atomic_load(&e->last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < call) atomicMax(&e->last, call);
}
constexpr int kMaxProbe = 32;

// An entity's bytes in registers: 16-byte loads, the last ones byte by byte
// where they would pass the text's end, zeros past len.
__device__ __forceinline__ void load_entity(const uint8_t* text, int64_t at, int len, int64_t text_end,
                                            uint32_t (&m)[kMsgWords]) {
#pragma unroll
  for (int c = 0; c < kMsgWords / 4; ++c) {
    uint32_t w[4] = {0, 0, 0, 0};
    if (16 * c < len) {
      const int64_t p = at + 16 * c;
      if (text_end - p >= 16) {
        const uint4 v = load16(text + p);
        w[0] = v.x, w[1] = v.y, w[2] = v.z, w[3] = v.w;
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (16 * c + i < len) w[i >> 2] |= (uint32_t)text[p + i] << (8 * (i & 3));
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int left = len - 16 * c - 4 * i;
      m[4 * c + i] = left >= 4 ? w[i] : left <= 0 ? 0 : w[i] & ((1u << (8 * left)) - 1);
    }
  }
}

// 64-bit mix of the entity's dwords and length (table position and first
// comparison only; equal bytes are compared in full).  The multipliers are
// those of MurmurHash3's 64-bit finalizer (A. Appleby, public domain).
__device__ __forceinline__ uint64_t fingerprint(const uint32_t (&m)[kMsgWords], int len) {
  uint64_t h = 0x9e3779b97f4a7c15ull * (uint64_t)(len + 1);
#pragma unroll
  for (int i = 0; i < kMsgWords; i += 2)
    if (4 * i < len) {
      h = (h ^ (m[i] | ((uint64_t)m[i + 1] << 32))) * 0xff51afd7ed558ccdull;
      h ^= h >> 32;
    }
  h *= 0xc4ceb9fe1a85ec53ull;
  return h ^ (h >> 29);
}

// Entry bytes past its length are zero, as in m.
__device__ __forceinline__ bool same_bytes(const Entry* e, const uint32_t (&m)[kMsgWords], int len) {
  uint32_t diff = 0;
#pragma unroll
  for (int c = 0; c < kMsgWords / 4; ++c)
    if (16 * c < len) {
      const uint4 v = *(const uint4*)(e->bytes + 16 * c);
      diff |= (v.x ^ m[4 * c]) | (v.y ^ m[4 * c + 1]) | (v.z ^ m[4 * c + 2]) | (v.w ^ m[4 * c + 3]);
    }
  return diff == 0;
}

// Each span's output offset within its record, its pseudonym's length and
// where the text goes on after it.  A span is valid if it lies in the record
// and begins at or after the end of the last valid, not preserved one.
//
// A wave takes `per` records, one for up to 16,384 of them.  64 spans of a
// record at a time are laid out as if all were valid (prefix sums); only if one
// turns out not to be does lane 0 go through them one by one.  16,384 records
// of 7.8 KB: 46 -> 11 us against a thread per record, whose reads of
// neighbouring records' spans shared no cache line.  Of more records most have
// few spans, and a wave for each would wait for its reads alone (a million
// empty ones: 144 us against 5.5 of a thread each): a lane reads a record's
// bounds, and lays out up to kFewSpans by itself.
constexpr int kFewSpans = 8;
template <bool SEVERAL>  // records to a wave
__global__ __launch_bounds__(256) void ps_layout_kernel(PcacheDev pc, const int64_t* __restrict__ cu_bytes, int B,
                                                        int per, const anon_span* __restrict__ spans,
                                                        const int* __restrict__ cu_spans, int span_cap,
                                                        int64_t* __restrict__ out_len, int64_t* __restrict__ sp_out,
                                                        int* __restrict__ sp_plen, int64_t* __restrict__ sp_in_end,
                                                        uint32_t* err) {
  const int lane = threadIdx.x & 63;
  const int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per;
  const int tail = pc.slug > 0 ? pc.slug + 1 : 0;
  // spans [i0, i1) of record b in their order, after acc bytes of growth and a
  // replaced span's end at prev_end (the error is raised once: 6144 invalid
  // spans in 1024 records met on its word for 64 us)
  auto one_by_one = [&](int b, int64_t in_len, int i0, int i1, int64_t& acc, int64_t& prev_end) {
    bool bad = false;
    for (int i = i0; i < i1; ++i) {
      const anon_span q = spans[i];
      const bool valid = q.record == b && q.type >= 1 && q.type <= pc.n_types && q.begin >= prev_end &&
                         q.end >= q.begin && q.end <= in_len;
      if (valid && !preserved(pc, q.type)) {
        const int n = 2 + (pc.name_off[q.type] - pc.name_off[q.type - 1]) + tail;
        sp_out[i] = q.begin + acc;
        sp_plen[i] = n;
        sp_in_end[i] = q.end;
        acc += n - (q.end - q.begin);
        prev_end = q.end;
      } else {
        bad |= !valid;
        sp_out[i] = prev_end + acc;
        sp_plen[i] = 0;
        sp_in_end[i] = prev_end;
      }
    }
    if (bad) raise_error(err, ANON_ERR_SPAN);
  };
  auto bounds = [&](int64_t b, int64_t& in_len, int& s0, int& s1) {
    in_len = cu_bytes[b + 1] - cu_bytes[b];
    if (in_len < 0) {
      raise_error(err, ANON_ERR_SPAN);
      in_len = 0;
    }
    s0 = cu_spans[b], s1 = cu_spans[b + 1];
    if (s1 > span_cap) raise_error(err, ANON_ERR_SPAN_CAP);
    s0 = min(max(s0, 0), span_cap);
    s1 = min(max(s1, s0), span_cap);
  };
  // record b by the whole wave
  auto by_wave = [&](int b, int64_t in_len, int s0, int s1) {
    int64_t acc = 0, prev_end = 0;
    for (int c0 = s0; c0 < s1; c0 += 64) {
      const int s = c0 + lane;
      const bool in = s < s1;
      anon_span sp{b, 0, 0, 0};
      if (in) sp = spans[s];
      const bool typed = sp.type >= 1 && sp.type <= pc.n_types;
      const bool keep = in && typed && preserved(pc, sp.type);
      const int plen = in && typed && !keep ? 2 + (pc.name_off[sp.type] - pc.name_off[sp.type - 1]) + tail : 0;
      // ends of the replaced spans up to and before this lane's, the growth likewise
      int64_t e = plen > 0 ? sp.end : 0, d = plen > 0 ? plen - (sp.end - sp.begin) : 0;
      const int64_t own = d;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(e, o, 64), z = __shfl_up(d, o, 64);
        if (lane >= o) {
          e = max(e, y);
          d += z;
        }
      }
      int64_t before = __shfl_up(e, 1, 64);
      before = lane > 0 ? max(before, prev_end) : prev_end;
      const bool ok = !in || (sp.record == b && typed && sp.begin >= before && sp.end >= sp.begin && sp.end <= in_len);
      if (__all(ok)) {
        const int64_t a = acc + d - own;
        if (in) {
          // a preserved type: the span's bytes are copied like the text around it
          sp_out[s] = (plen > 0 ? sp.begin : before) + a;
          sp_plen[s] = plen;
          sp_in_end[s] = plen > 0 ? sp.end : before;
        }
        acc += __shfl(d, 63, 64);
        prev_end = max(prev_end, __shfl(e, 63, 64));
        continue;
      }
      if (lane == 0) one_by_one(b, in_len, c0, min(c0 + 64, s1), acc, prev_end);
      acc = __shfl(acc, 0, 64);
      prev_end = __shfl(prev_end, 0, 64);
    }
    if (lane == 0) out_len[b] = in_len + acc;
  };
  int64_t in_len = 0;
  int s0 = 0, s1 = 0;
  if constexpr (!SEVERAL) {
    if (first >= B) return;
    bounds(first, in_len, s0, s1);
    by_wave((int)first, in_len, s0, s1);
    return;
  }
  const int b = (int)first + lane;  // this lane's record
  const bool mine = lane < per && first + lane < B;
  if (mine) bounds(b, in_len, s0, s1);
  const bool few = s1 - s0 <= kFewSpans;
  if (mine && few) {
    int64_t acc = 0, prev_end = 0;
    one_by_one(b, in_len, s0, s1, acc, prev_end);
    out_len[b] = in_len + acc;
  }
  for (uint64_t todo = __ballot(mine && !few); todo; todo &= todo - 1) {
    const int of = __ffsll((unsigned long long)todo) - 1;
    by_wave((int)first + of, __shfl(in_len, of, 64), __shfl(s0, of, 64), __shfl(s1, of, 64));
  }
}

// A thread per span, the grid striding over the spans there are (their count
// is on the device, the capacity may be far above it).  The entity is read
// once into registers with 16-byte loads, and hashed, compared and stored
// from there.  The counters are summed per workgroup into one of
// kCounterSlots slots, where every wave's two atomics met on one line.  Bound
// by the latency of text, probe and entry, each found by the one before, and
// for new entities by fences: a slot's state carries 30 bits of its
// fingerprint, so that only a slot that is nearly surely the entity's is read
// behind a fence or waited for.  us per call, cold being a first meeting:
//   139,000 spans of 359 entities in 128 MB: 46, cold 131 (a thread per
//     span, bytewise: 160, 265)
//   120,000 spans, nearly all of an entity each: cold 120 (every occupied slot
//     behind a fence, every slot being written waited for: 396; neither
//     waiting nor tags: 167)
// Three waves a SIMD, and one copy of the compression for an entity's blocks
// (hmac_words): 57 -> 49 for the hits.
__global__ __launch_bounds__(256, 3) void ps_hash_kernel(PcacheDev pc, const uint8_t* __restrict__ text,
                                                      const int64_t* __restrict__ cu_bytes, int B,
                                                      const anon_span* __restrict__ spans,
                                                      const int* __restrict__ cu_spans, int span_cap,
                                                      const int* __restrict__ sp_plen,
                                                      uint32_t* __restrict__ digests) {
  __shared__ int tally[3];
  const int n = min(cu_spans[B], span_cap);
  const int64_t text_end = cu_bytes[B];
  if (threadIdx.x < 3) tally[threadIdx.x] = 0;
  __syncthreads();
  int lookups = 0, hits = 0, inserts = 0;
  Entry* table = (Entry*)pc.table;
  for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < n; s += (int64_t)gridDim.x * 256) {
    if (sp_plen[s] <= 0) continue;
    const anon_span sp = spans[s];
    const int64_t at = cu_bytes[sp.record] + sp.begin, len64 = sp.end - sp.begin;
    uint32_t dg[8];
    if (len64 > kMaxEntity) {
      hmac_sha256(pc, text + at, len64, dg);
    } else {
      const int len = (int)len64;
      uint32_t m[kMsgWords];
      load_entity(text, at, len, text_end, m);
      const uint64_t fp = pc.enabled ? fingerprint(m, len) : 0;
      const uint32_t tag = (uint32_t)(fp >> 32) & ~3u;
      bool have = false;
      if (pc.enabled) {
        ++lookups;
        uint64_t slot = fp & pc.mask;
        for (int i = 0; i < kMaxProbe; ++i, slot = (slot + 1) & pc.mask) {
          Entry* e = table + slot;
          const uint32_t stt = __hip_atomic_load(&e->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (stt == 0) break;
          if (stt != (tag | 2)) continue;
          // a ready entry: this fence pairs with its writer's release fence, so
          // the entry's fields read below are the ones written before "ready"
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          if (e->fp == fp && e->len == (uint32_t)len && same_bytes(e, m, len)) {
#pragma unroll
            for (int k = 0; k < 8; ++k) dg[k] = e->digest[k];
            have = true;
            ++hits;
            touch(e, sp.type, pc.call);
            break;
          }
        }
      }
      if (!have) {
        hmac_words(pc, m, len, dg);
        if (pc.enabled) {
          // In rounds of the wave: every lane goes on to a slot that it can
          // claim, to its entity, or to a slot that is being written; then one
          // release fence publishes all that were claimed (a fence is a cache
          // write-back on this part).  A slot being written that has this
          // entity's tag may be getting this very entity, so it is looked at
          // again, a bounded number of times: else the many lanes of one
          // frequent new entity fill kMaxProbe slots with it, and an entity
          // whose place is the first of them finds no room.
          uint64_t slot = fp & pc.mask;
          int probe = 0, waits = 0;
          bool open = true;
          while (__any(open)) {
            Entry* claimed = nullptr;
            while (open) {
              if (probe >= kMaxProbe) {
                open = false;
                break;
              }
              Entry* e = table + slot;
              // claiming an empty slot reads nothing of another writer's, so the
              // claim needs no ordering (waiting is a load: many waves wait for
              // one frequent new entity)
              uint32_t expected = 0;
              if (waits > 0) expected = __hip_atomic_load(&e->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              if (expected == 0 && __hip_atomic_compare_exchange_strong(&e->state, &expected, tag | 1, __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                claimed = e;
                break;
              }
              if (expected == (tag | 2)) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                if (e->fp == fp && e->len == (uint32_t)len && same_bytes(e, m, len)) {
                  touch(e, sp.type, pc.call);
                  open = false;
                  break;
                }
              } else if (expected == (tag | 1) && waits < kMaxProbe) {
                ++waits;
                break;
              }
              ++probe;
              slot = (slot + 1) & pc.mask;
            }
            if (claimed) {
              claimed->len = (uint32_t)len;
              claimed->fp = fp;
#pragma unroll
              for (int c = 0; c < kMsgWords / 4; ++c)
                *(uint4*)(claimed->bytes + 16 * c) = uint4{m[4 * c], m[4 * c + 1], m[4 * c + 2], m[4 * c + 3]};
#pragma unroll
              for (int k = 0; k < 8; ++k) claimed->digest[k] = dg[k];
              claimed->type = sp.type;
              claimed->first = claimed->last = pc.call;
              __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
              __hip_atomic_store(&claimed->state, tag | 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              ++inserts;
              open = false;
            }
          }
        }
      }
    }
    uint4* to = (uint4*)(digests + (size_t)s * 8);
    to[0] = uint4{dg[0], dg[1], dg[2], dg[3]};
    to[1] = uint4{dg[4], dg[5], dg[6], dg[7]};
  }
  if (lookups) atomicAdd(&tally[0], lookups);
  if (hits) atomicAdd(&tally[1], hits);
  if (inserts) atomicAdd(&tally[2], inserts);
  __syncthreads();
  if (threadIdx.x < 3 && tally[threadIdx.x])
    atomicAdd(&pc.counters[8 * (blockIdx.x % kCounterSlots) + threadIdx.x], (unsigned long long)tally[threadIdx.x]);
}

// Record blockIdx.x's output, every gridDim.y-th block of kChunks 16-byte chunks
// (chunks are aligned in memory).  A chunk that lies in copied text is one
// unaligned 16-byte load and one store; the others (a span begins or ends in
// them, or the record does) are listed and done a byte per thread, so that
// they do not hold up the copying lanes.  The record's spans are searched in
// LDS (if at most kStaged; else in memory).  128 MB in 16,384 records: 730 ->
// 105 us (2.4 TB/s read and written) against a byte and a search per thread.
constexpr int kStaged = 512;
constexpr int kChunks = 512;  // a step of a workgroup: two chunks a thread, both in flight

__global__ __launch_bounds__(256) void ps_write_kernel(PcacheDev pc, const uint8_t* __restrict__ text,
                                                       const int64_t* __restrict__ cu_bytes,
                                                       const anon_span* __restrict__ spans,
                                                       const int* __restrict__ cu_spans, int span_cap,
                                                       const int64_t* __restrict__ sp_out,
                                                       const int* __restrict__ sp_plen,
                                                       const int64_t* __restrict__ sp_in_end,
                                                       const uint32_t* __restrict__ digests,
                                                       const int64_t* __restrict__ cu_out, uint8_t* __restrict__ out,
                                                       int64_t out_cap, uint32_t* err) {
  __shared__ int64_t l_out[kStaged], l_end[kStaged];
  __shared__ int l_plen[kStaged];
  __shared__ int list[kChunks], n_list;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int64_t o0 = cu_out[b], n_out = cu_out[b + 1] - o0;
  const int lead = (int)((uintptr_t)(out + o0) & 15);  // bytes of the first chunk before the record
  const int64_t chunks = n_out > 0 ? (n_out + lead + 15) / 16 : 0;
  if ((int64_t)blockIdx.y * kChunks >= chunks) return;
  if (tid == 0 && o0 + n_out > out_cap) raise_error(err, ANON_ERR_OUT_CAP);
  const int64_t room = min(n_out, out_cap - o0);  // bytes of the record that are written
  const int s0 = min(max(cu_spans[b], 0), span_cap);
  const int ns = min(max(cu_spans[b + 1], s0), span_cap) - s0;
  const bool staged = ns <= kStaged;
  if (staged)
    for (int i = tid; i < ns; i += 256) {
      l_out[i] = sp_out[s0 + i];
      l_plen[i] = sp_plen[s0 + i];
      l_end[i] = sp_in_end[s0 + i];
    }
  const uint8_t* in = text + cu_bytes[b];
  const int64_t in_len = max(cu_bytes[b + 1] - cu_bytes[b], (int64_t)0);
  auto pos = [&](int i) { return staged ? l_out[i] : sp_out[s0 + i]; };
  auto last_at = [&](int64_t j) {  // last span whose pseudonym starts at or before output byte j
    int lo = 0, hi = ns - 1, sel = -1;
    while (lo <= hi) {
      const int mid = (lo + hi) >> 1;
      if (pos(mid) <= j) sel = mid, lo = mid + 1;
      else hi = mid - 1;
    }
    return sel;
  };
  for (int64_t c0 = (int64_t)blockIdx.y * kChunks; c0 < chunks; c0 += (int64_t)gridDim.y * kChunks) {
    if (tid == 0) n_list = 0;
    __syncthreads();
    int64_t src[kChunks / 256];  // where the thread's chunks are copied from, -1: not, -2: listed
#pragma unroll
    for (int k = 0; k < kChunks / 256; ++k) {
      const int64_t c = c0 + k * 256 + tid, j0 = c * 16 - lead;
      src[k] = c < chunks && j0 < room ? -2 : -1;
      if (src[k] == -1 || j0 < 0 || j0 + 16 > room) continue;
      const int sel = last_at(j0);
      const int64_t stop = sel + 1 < ns ? pos(sel + 1) : n_out;
      int64_t from = j0;
      bool gap = true;
      if (sel >= 0) {
        const int64_t past = j0 - pos(sel) - (staged ? l_plen[sel] : sp_plen[s0 + sel]);
        gap = past >= 0;
        from = (staged ? l_end[sel] : sp_in_end[s0 + sel]) + past;
      }
      if (gap && stop - j0 >= 16 && in_len - from >= 16) src[k] = from;
    }
    uint4 v[kChunks / 256];
#pragma unroll
    for (int k = 0; k < kChunks / 256; ++k)
      if (src[k] >= 0) v[k] = load16(in + src[k]);
#pragma unroll
    for (int k = 0; k < kChunks / 256; ++k) {
      const int c = k * 256 + tid;
      if (src[k] >= 0) *(uint4*)(out + o0 + (c0 + c) * 16 - lead) = v[k];
      else if (src[k] == -2) list[atomicAdd(&n_list, 1)] = c;
    }
    __syncthreads();
    const int todo = n_list * 16;
    for (int q = tid; q < todo; q += 256) {
      const int64_t j = (c0 + list[q >> 4]) * 16 - lead + (q & 15);
      if (j < 0 || j >= room) continue;
      const int sel = last_at(j);
      uint8_t ch;
      if (sel < 0) {
        ch = j < in_len ? in[j] : 0;
      } else {
        const int64_t k = j - pos(sel);
        const int plen = staged ? l_plen[sel] : sp_plen[s0 + sel];
        if (k < plen) {
          const int typ = spans[s0 + sel].type;
          const int n0 = pc.name_off[typ - 1], tl = pc.name_off[typ] - n0;
          if (k == 0) ch = '[';
          else if (k == plen - 1) ch = ']';
          else if (k <= tl) ch = pc.names[n0 + k - 1];
          else if (k == tl + 1) ch = '_';
          else {
            const int h = (int)(k - tl - 2);
            const uint32_t v = (digests[(size_t)(s0 + sel) * 8 + (h >> 3)] >> (28 - 4 * (h & 7))) & 15;
            ch = (uint8_t)(v < 10 ? '0' + v : 'a' + v - 10);
          }
        } else {
          const int64_t i = (staged ? l_end[sel] : sp_in_end[s0 + sel]) + (k - plen);
          ch = i < in_len ? in[i] : 0;
        }
      }
      out[o0 + j] = ch;
    }
    __syncthreads();
  }
}

}  // namespace

size_t pcache_entry_bytes() { return sizeof(Entry); }

// Known-answer check of the host SHA-256/HMAC code (RFC 4231 Sec. 4.3).
bool hmac_selftest() {
  const char* key = "Jefe";
  const char* msg = "what do ya want for nothing?";
  const uint32_t want[8] = {0x5bdcc146u, 0xbf60754eu, 0x6a042426u, 0x089575c7u,
                            0x5a003f08u, 0x9d273983u, 0x9dec58b9u, 0x64ec3843u};
  uint32_t ip[8], op[8];
  sha256_hmac_midstates((const uint8_t*)key, 4, ip, op);
  sha256_tail(ip, 64, (const uint8_t*)msg, 28);
  uint32_t w[16] = {0};
  for (int i = 0; i < 8; ++i) w[i] = ip[i];
  w[8] = 0x80000000u;
  w[15] = (64 + 32) * 8;
  sha256_compress(op, w);
  for (int i = 0; i < 8; ++i)
    if (op[i] != want[i]) return false;
  return true;
}

void sha256_hmac_midstates(const uint8_t* key, size_t key_len, uint32_t ipad[8], uint32_t opad[8]) {
  uint8_t k0[64] = {0};
  if (key_len > 64) {
    uint32_t st[8];
    for (int i = 0; i < 8; ++i) st[i] = kH0[i];
    sha256_tail(st, 0, key, (int64_t)key_len);
    for (int i = 0; i < 8; ++i) {
      k0[4 * i] = (uint8_t)(st[i] >> 24);
      k0[4 * i + 1] = (uint8_t)(st[i] >> 16);
      k0[4 * i + 2] = (uint8_t)(st[i] >> 8);
      k0[4 * i + 3] = (uint8_t)st[i];
    }
  } else {
    for (size_t i = 0; i < key_len; ++i) k0[i] = key[i];
  }
  uint32_t wi[16], wo[16];
  for (int i = 0; i < 16; ++i) {
    uint32_t a = 0, b = 0;
    for (int j = 0; j < 4; ++j) {
      a = (a << 8) | (uint8_t)(k0[4 * i + j] ^ 0x36);
      b = (b << 8) | (uint8_t)(k0[4 * i + j] ^ 0x5c);
    }
    wi[i] = a;
    wo[i] = b;
  }
  for (int i = 0; i < 8; ++i) ipad[i] = opad[i] = kH0[i];
  sha256_compress(ipad, wi);
  sha256_compress(opad, wo);
}

void launch_ps_layout(const PcacheDev& pc, const int64_t* cu_bytes, int B, const anon_span* spans,
                      const int* cu_spans, int span_cap, int64_t* out_len, int64_t* sp_out, int* sp_plen,
                      int64_t* sp_in_end, uint32_t* err, hipStream_t s) {
  if (B <= 0) return;
  const int per = std::min(ceil_div(B, 16384), 64);
  hipLaunchKernelGGL(per > 1 ? ps_layout_kernel<true> : ps_layout_kernel<false>, dim3(ceil_div(B, (int64_t)4 * per)),
                     dim3(256), 0, s, pc, cu_bytes, B, per, spans, cu_spans, span_cap, out_len, sp_out, sp_plen,
                     sp_in_end, err);
}

void launch_ps_hash(const PcacheDev& pc, const uint8_t* text, const int64_t* cu_bytes, int B, const anon_span* spans,
                    const int* cu_spans, int span_cap, const int* sp_plen, uint8_t* digests, hipStream_t s) {
  if (span_cap <= 0 || pc.slug == 0) return;
  hipLaunchKernelGGL(ps_hash_kernel, dim3(std::min(ceil_div(span_cap, 256), 2048)), dim3(256), 0, s, pc, text, cu_bytes, B, spans,
                     cu_spans, span_cap, sp_plen, (uint32_t*)digests);
}

void launch_ps_write(const PcacheDev& pc, const uint8_t* text, const int64_t* cu_bytes, int B,
                     const anon_span* spans, const int* cu_spans, int span_cap, const int64_t* sp_out,
                     const int* sp_plen, const int64_t* sp_in_end, const uint8_t* digests, const int64_t* cu_out,
                     uint8_t* out, int64_t out_cap, uint32_t* err, hipStream_t s) {
  if (B <= 0) return;
  // few records: several workgroups for each, which leave at once if it is short
  const int split = std::max(1, std::min(2048 / B, 64));
  hipLaunchKernelGGL(ps_write_kernel, dim3(B, split), dim3(256), 0, s, pc, text, cu_bytes, spans, cu_spans, span_cap,
                     sp_out, sp_plen, sp_in_end, (const uint32_t*)digests, cu_out, out, out_cap, err);
}

}  // namespace anon
