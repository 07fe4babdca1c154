// BIO span decoding on the GPU, plus the device-wide exclusive scans that
// compact variable-length outputs.
//
// Decoding is token-parallel.  A token opens a span iff its label is not O
// and it is B-t, or it is the first token of its record, or the previous
// token's type differs (so an I-t without an open span of type t opens one).
// The flags are kept as bits with their ranks, 4096 tokens to a workgroup;
// the workgroups' counts give every span its index in record-major order, and
// the opening token then walks forward over the following I-t tokens of its
// record (labels staged in LDS) to find the span's last token.  Every token
// is visited by at most one walk, so the work is O(T).
//
// Bound by latency and launches: a call moves 2.5 bytes per token beyond the
// spans themselves (labels read twice, a quarter byte of flags and ranks
// written and read), and takes two launches where an int flag per token, a
// three-kernel scan of them and a record search per labelled token took six.
// 978,000 tokens in 4096 records: 38 -> 11.5 us (6 in each kernel).
#include "kernels.hpp"

namespace anon {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename T>
__device__ T block_exclusive_scan(T v, T* sh, T* total) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {
    const T x = tid >= o ? sh[tid - o] : T(0);
    __syncthreads();
    sh[tid] += x;
    __syncthreads();
  }
  const T incl = sh[tid];
  *total = sh[kScanThreads - 1];
  __syncthreads();
  return incl - v;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const T* __restrict__ in, int64_t n,
                                                                   T* __restrict__ part) {
  __shared__ T sh[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) s += in[base + i];
  T total;
  block_exclusive_scan<T>(s, sh, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Single workgroup: exclusive scan of the per-tile sums; writes the grand
// total to out[n].
template <typename T>
__global__ __launch_bounds__(1024) void scan_parts_kernel(T* __restrict__ part, int nparts, T* __restrict__ out,
                                                          int64_t n) {
  __shared__ T sh[1024];
  const int tid = threadIdx.x;
  const int per = (nparts + 1023) / 1024;
  const int a = min(nparts, tid * per), b = min(nparts, a + per);
  T s = 0;
  for (int i = a; i < b; ++i) s += part[i];
  sh[tid] = s;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const T x = tid >= o ? sh[tid - o] : T(0);
    __syncthreads();
    sh[tid] += x;
    __syncthreads();
  }
  T run = sh[tid] - s;
  for (int i = a; i < b; ++i) {
    const T v = part[i];
    part[i] = run;
    run += v;
  }
  if (tid == 1023) out[n] = sh[1023];
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(const T* __restrict__ in, int64_t n,
                                                                  const T* __restrict__ part, T* __restrict__ out) {
  __shared__ T sh[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T v[kScanItems];
  T s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = base + i < n ? in[base + i] : T(0);
    s += v[i];
  }
  T total;
  T run = block_exclusive_scan<T>(s, sh, &total) + part[blockIdx.x];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) out[base + i] = run;
    run += v[i];
  }
}

template <typename T>
void exclusive_scan(const T* in, T* out, int64_t n, void* temp, hipStream_t s) {
  const int nparts = (int)((n + kScanTile - 1) / kScanTile);
  T* part = (T*)temp;
  if (nparts > 0) hipLaunchKernelGGL(scan_reduce_kernel<T>, dim3(nparts), dim3(kScanThreads), 0, s, in, n, part);
  hipLaunchKernelGGL(scan_parts_kernel<T>, dim3(1), dim3(1024), 0, s, part, nparts, out, n);
  if (nparts > 0)
    hipLaunchKernelGGL(scan_apply_kernel<T>, dim3(nparts), dim3(kScanThreads), 0, s, in, n, (const T*)part, out);
}

// Exclusive prefix of n values in place or into out, out[n] = their sum, by
// one workgroup: 4 consecutive values per thread and step, so a step of 4096
// values is one coalesced load, a wave scan and two barriers.  For the counts
// of tiles or records, which are few: 31,250 take 19 us (a run of values per
// thread, read one after the other, took 55).
template <typename T>
__global__ __launch_bounds__(1024) void scan_one_kernel(const T* in, T* out, int n) {
  __shared__ T ws[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  T carry = 0;
  for (int at = 0; at < n; at += 4096) {
    const int i = at + tid * 4;
    T v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = i + k < n ? in[i + k] : T(0);
    const T s = v[0] + v[1] + v[2] + v[3];
    T x = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const T y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    T run = carry + x - s;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w < wave) run += ws[w];
      carry += ws[w];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < n) out[i + k] = run;
      run += v[k];
    }
    __syncthreads();
  }
  if (tid == 0) out[n] = carry;
}

constexpr int kTile = 4096;           // tokens per workgroup, 16 per thread
constexpr int kDirectTiles = 4096;    // up to here the writers sum the tiles before theirs themselves

__device__ __forceinline__ int clean_label(int lab, int n_types, uint32_t* err) {
  if (lab > 2 * n_types) {
    raise_error(err, ANON_ERR_LABEL);
    return 0;
  }
  return lab;
}

// Exclusive sum of v over the workgroup's 256 threads and its total.
__device__ __forceinline__ int wg_exclusive(int v, int* total) {
  __shared__ int ws[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) ws[wave] = x;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) base += ws[w];
    all += ws[w];
  }
  *total = all;
  __syncthreads();
  return base + x - v;
}

// 16 labels from t0 on (zeros past T), byte i in bits 8 (i mod 4) of word i/4
__device__ __forceinline__ uint4 load_labels(const uint8_t* labels, int t0, int T) {
  if (T - t0 >= 16) return load16(labels + t0);
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i < T - t0) w[i >> 2] |= (uint32_t)labels[t0 + i] << (8 * (i & 3));
  return uint4{w[0], w[1], w[2], w[3]};
}

// Opening flags of a tile of tokens: 16 bits per thread, their rank within
// the tile, and the tile's count.  A token's record start matters only where
// an I-t follows a token of type t, and is looked up in the tile's own record
// boundaries (a bitmap in LDS), so no token searches the boundary array.
__global__ __launch_bounds__(256) void bio_flags_kernel(const uint8_t* __restrict__ labels,
                                                        const int* __restrict__ cu, int B, int T, int n_types,
                                                        uint16_t* __restrict__ bits, uint16_t* __restrict__ rank,
                                                        int* __restrict__ counts, int* __restrict__ rec0,
                                                        uint32_t* err) {
  __shared__ uint32_t starts[kTile / 32];
  const int tid = threadIdx.x, base = blockIdx.x * kTile, last = base + kTile - 1, t0 = base + tid * 16;
  const uint4 lv = load_labels(labels, t0, T);
  const uint32_t l[4] = {lv.x, lv.y, lv.z, lv.w};
  int prev = t0 > 0 && t0 < T ? labels[t0 - 1] : 0;
  if (tid < kTile / 32) starts[tid] = 0;
  // record boundaries inside the tile
  const int first = wg_find_record(cu, B, base);
  __syncthreads();
  wg_each_record_to(cu, B, first, min(last, T - 1), [&](int b) {
    const int c = cu[b];
    if (c >= base && c <= last) atomicOr(&starts[(c - base) >> 5], 1u << ((c - base) & 31));
  });
  const uint32_t rs = starts[tid >> 1] >> ((tid & 1) * 16);
  uint32_t f = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int raw = (l[i >> 2] >> (8 * (i & 3))) & 0xff;
    const int lab = clean_label(raw, n_types, err), typ = (lab + 1) >> 1;
    const int ptyp = prev > 2 * n_types ? 0 : (prev + 1) >> 1;
    if (lab != 0 && ((lab & 1) || t0 + i == 0 || ((rs >> i) & 1) || ptyp != typ)) f |= 1u << i;
    prev = raw;
  }
  int total;
  const int r = wg_exclusive(__popc(f), &total);
  if (t0 < T) {
    bits[t0 >> 4] = (uint16_t)f;
    rank[t0 >> 4] = (uint16_t)r;
  }
  if (tid == 0) {
    counts[blockIdx.x] = total;
    rec0[blockIdx.x] = first;
  }
}

// Last token of a span whose tokens up to e are known to be in it: sixteen
// labels a load, four loads at once while the record has as many (a span of
// 100,000 tokens 12.4 -> 1.0 ms against a label at a time).
constexpr int kNear = 32;  // tokens looked at one by one before
__device__ __forceinline__ int run_end(const uint8_t* __restrict__ labels, int e, int end_tok, int cont) {
  const uint32_t c4 = (uint32_t)cont * 0x01010101u;
  while (end_tok - e > 64) {
    uint4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = load16(labels + e + 1 + 16 * i);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w[4] = {v[i].x ^ c4, v[i].y ^ c4, v[i].z ^ c4, v[i].w ^ c4};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (w[k]) return e + (__ffs(w[k]) - 1) / 8;
        e += 4;
      }
    }
  }
  while (e + 1 < end_tok && labels[e + 1] == cont) ++e;
  return e;
}

// Spans of a tile (blocks below n_tiles) and the record offsets (the blocks
// above).  With SCANNED, counts already holds the exclusive prefix over the
// tiles; else each block sums the counts before its tile (at most
// kDirectTiles of them), which saves a launch.
template <bool SCANNED>
__global__ __launch_bounds__(256) void bio_write_kernel(const uint8_t* __restrict__ labels,
                                                        const int* __restrict__ tok_off, const int* __restrict__ cu,
                                                        int B, int T, int n_tiles, const uint16_t* __restrict__ bits,
                                                        const uint16_t* __restrict__ rank,
                                                        const int* __restrict__ counts, const int* __restrict__ rec0,
                                                        anon_span* __restrict__ spans, int span_cap,
                                                        int* __restrict__ cu_spans, uint32_t* err) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= n_tiles) {
    // cu_spans[b]: spans opened before the record's first token
    __shared__ int pre[SCANNED ? 1 : kDirectTiles + 1];
    if constexpr (!SCANNED) {
      constexpr int PER = kDirectTiles / 256;
      int c[PER], s = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int k = tid * PER + i;
        c[i] = k < n_tiles ? counts[k] : 0;
        s += c[i];
      }
      int total;
      s = wg_exclusive(s, &total);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        pre[tid * PER + i] = s;
        s += c[i];
      }
      if (tid == 0) pre[kDirectTiles] = total;
      __syncthreads();
    }
    const int b = (blockIdx.x - n_tiles) * 256 + tid;
    if (b > B) return;
    const int t = min(max(cu[b], 0), T), tile = t / kTile;
    int n;
    if constexpr (SCANNED) n = counts[min(tile, n_tiles)];
    else n = pre[min(tile, kDirectTiles)];
    if (t < T) n += rank[t >> 4] + __popc(bits[t >> 4] & ((1u << (t & 15)) - 1));
    else if (tile < n_tiles) n = SCANNED ? counts[tile + 1] : pre[tile + 1];
    cu_spans[b] = n;
    if (b == B && (SCANNED ? counts[n_tiles] : pre[n_tiles]) > span_cap) raise_error(err, ANON_ERR_SPAN_CAP);
    return;
  }
  const int base = blockIdx.x * kTile, last = min(base + kTile - 1, T - 1), t0 = base + tid * 16;
  __shared__ __align__(16) uint8_t lab[kTile];
  uint32_t f = 0;
  int idx = 0;
  if (t0 < T) {
    f = bits[t0 >> 4];
    idx = rank[t0 >> 4];
  }
  *(uint4*)(lab + tid * 16) = load_labels(labels, t0, T);
  if constexpr (SCANNED) {
    idx += counts[blockIdx.x];
  } else {
    int s = 0, total;
    for (int k = tid; k < (int)blockIdx.x; k += 256) s += counts[k];
    wg_exclusive(s, &total);
    idx += total;
  }
  // the tile's records lie between its first and the next tile's first
  const int r0 = rec0[blockIdx.x], r1 = (int)blockIdx.x + 1 < n_tiles ? rec0[blockIdx.x + 1] : B - 1;
  __syncthreads();
  int a = r0, next = -1;  // the span's record and the first token past it
  for (; f; f &= f - 1, ++idx) {
    if (idx >= span_cap) break;
    const int t = t0 + __ffs(f) - 1;
    if (next <= t) {  // largest index of [a, r1] with cu <= t
      int c = r1;
      while (a < c) {
        const int m = (a + c + 1) >> 1;
        if (cu[m] <= t) a = m;
        else c = m - 1;
      }
      next = cu[a + 1];
    }
    const int end_tok = min(next, T);
    const int typ = (lab[t - base] + 1) >> 1, cont = 2 * typ;  // I-typ continues the span
    int e = t;
    const int near = min(min(end_tok - 1, last), t + kNear);
    while (e < near && lab[e + 1 - base] == cont) ++e;
    if (e == near) e = run_end(labels, e, end_tok, cont);
    spans[idx] = anon_span{a, typ, tok_off[2 * t], tok_off[2 * e + 1]};
  }
}

}  // namespace

size_t scan_temp_bytes(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile + 1) * sizeof(int64_t); }

void launch_exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, void* temp, hipStream_t s) {
  // one launch while a workgroup's steps of 4096 (2.4 us each) cost less than
  // the tiled scan's three launches (16,384 values: 10 us against 15)
  if (n <= 16384) hipLaunchKernelGGL(scan_one_kernel<int64_t>, dim3(1), dim3(1024), 0, s, in, out, (int)n);
  else exclusive_scan<int64_t>(in, out, n, temp, s);
}

size_t bio_layout(int T, Carver& k, BioBuffers& w) {
  const int tiles = ceil_div(T, kTile);
  w.bits = k.take<uint16_t>(ceil_div(T, 16));
  w.rank = k.take<uint16_t>(ceil_div(T, 16));
  w.counts = k.take<int>((size_t)2 * (tiles + 1));
  w.rec0 = w.counts + tiles + 1;
  return k.used;
}

void launch_scan_counts(int* counts, int n, hipStream_t s) {
  hipLaunchKernelGGL(scan_one_kernel<int>, dim3(1), dim3(1024), 0, s, counts, counts, n);
}

void launch_bio(const uint8_t* labels, const int* tok_off, const int* cu_seqlens, int B, int T, int n_types,
                const BioBuffers& w, anon_span* spans, int span_cap, int* cu_spans, uint32_t* err, hipStream_t s) {
  const int tiles = ceil_div(T, kTile), grid = tiles + ceil_div(B + 1, 256);
  if (tiles > 0)
    hipLaunchKernelGGL(bio_flags_kernel, dim3(tiles), dim3(256), 0, s, labels, cu_seqlens, B, T, n_types, w.bits,
                       w.rank, w.counts, w.rec0, err);
  if (tiles > kDirectTiles) {
    launch_scan_counts(w.counts, tiles, s);
    hipLaunchKernelGGL(bio_write_kernel<true>, dim3(grid), dim3(256), 0, s, labels, tok_off, cu_seqlens, B, T, tiles,
                       w.bits, w.rank, w.counts, w.rec0, spans, span_cap, cu_spans, err);
  } else {
    hipLaunchKernelGGL(bio_write_kernel<false>, dim3(grid), dim3(256), 0, s, labels, tok_off, cu_seqlens, B, T,
                       tiles, w.bits, w.rank, w.counts, w.rec0, spans, span_cap, cu_spans, err);
  }
}

}  // namespace anon
