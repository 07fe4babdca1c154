// Row-wise kernels of the encoder: embedding + LayerNorm, LayerNorm, the
// token-classification head (argmax and top-2 margin), type conversions and
// the window gather / owner-window merge for long records.
//
// A 64-lane wave owns a token row (LayerNorm of a large batch: two rows);
// lane i holds VEC consecutive elements (4 where the row length allows) of
// each chunk of 64*VEC elements, so every load and store is a contiguous wave
// access (see RowMap).  LayerNorm statistics are FP32 and two-pass (mean, then
// mean of squared deviations) with a fixed order of the sums, so a row's
// result never depends on the other rows of the batch.  The classifier runs
// on the FP32 matrix cores, 16 tokens per wave.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace anon {
namespace {

__device__ __forceinline__ float ldf(const float* p) { return *p; }
__device__ __forceinline__ float ldf(const bf16_t* p) { return static_cast<float>(*p); }

// Record containing packed token t (largest b with cu[b] <= t), robust to
// malformed cu_seqlens (the result is then only clamped, never out of range).
__device__ __forceinline__ int find_record(const int* cu, int B, int t) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cu[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The same by a whole wave for a wave-uniform t: 64 boundaries a step, so two
// dependent reads for up to 4096 records instead of twelve.
__device__ __forceinline__ int wave_find_record(const int* cu, int B, int t, int lane) {
  int lo = 0, n = B;
  while (n > 1) {
    const int step = (n + 63) / 64, i = lane * step;
    const uint64_t below = __ballot(lane == 0 || (i < n && cu[lo + i] <= t));
    const int k = 63 - __clzll((long long)below);
    lo += k * step;
    n = min(step, n - k * step);
  }
  return lo;
}

// A lane owns NPL elements of a row in chunks of VEC consecutive columns:
// element i sits at column (i / VEC) * 64 * VEC + lane * VEC + i % VEC, so
// every chunk is one 16-byte (fp32) or 8-byte (bf16) access and each wave
// access covers a contiguous span of the row.
template <int NPL>
struct RowMap {
  static constexpr int VEC = NPL % 4 == 0 ? 4 : NPL;
  __device__ static int col(int i, int lane) { return (i / VEC) * 64 * VEC + lane * VEC + i % VEC; }
};

template <int NPL>
__device__ __forceinline__ void load_row(const float* src, int lane, float (&v)[NPL]) {
  typedef RowMap<NPL> RM;
#pragma unroll
  for (int c = 0; c < NPL / RM::VEC; ++c) {
    if constexpr (RM::VEC == 4) {
      const floatx4 x = *(const floatx4*)(src + RM::col(c * 4, lane));
#pragma unroll
      for (int k = 0; k < 4; ++k) v[c * 4 + k] = x[k];
    } else {
#pragma unroll
      for (int k = 0; k < RM::VEC; ++k) v[c * RM::VEC + k] = src[RM::col(c * RM::VEC + k, lane)];
    }
  }
}

template <int NPL>
__device__ __forceinline__ void load_row(const bf16_t* src, int lane, float (&v)[NPL]) {
  typedef RowMap<NPL> RM;
#pragma unroll
  for (int c = 0; c < NPL / RM::VEC; ++c) {
    if constexpr (RM::VEC == 4) {
      const bf16x4 x = __builtin_nontemporal_load((const bf16x4*)(src + RM::col(c * 4, lane)));
#pragma unroll
      for (int k = 0; k < 4; ++k) v[c * 4 + k] = static_cast<float>(x[k]);
    } else {
#pragma unroll
      for (int k = 0; k < RM::VEC; ++k) v[c * RM::VEC + k] = static_cast<float>(src[RM::col(c * RM::VEC + k, lane)]);
    }
  }
}

// LayerNorm of the row in v (lane-owned elements, RowMap order) with gain gv
// and shift bv in the same order, written to row `row` of out (and out_q).
template <int NPL>
__device__ __forceinline__ void ln_store(float (&v)[NPL], const float (&gv)[NPL], const float (&bv)[NPL], float eps,
                                         int h, int lane, size_t row, void* out, ElemType out_t, fp8_t* out_q,
                                         float q_inv_scale, bf16_t* out_b = nullptr) {
  typedef RowMap<NPL> RM;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) s += v[i];
  const float mean = wave_sum(s) / (float)h;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    const float d = v[i] - mean;
    q += d * d;
  }
  const float var = wave_sum(q) / (float)h;
  const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
  for (int c = 0; c < NPL / RM::VEC; ++c) {
    float y[RM::VEC];
    const int c0 = RM::col(c * RM::VEC, lane);
#pragma unroll
    for (int k = 0; k < RM::VEC; ++k)
      y[k] = gv[c * RM::VEC + k] * ((v[c * RM::VEC + k] - mean) * rstd) + bv[c * RM::VEC + k];
    if (out_t == ET_F32) {
#pragma unroll
      for (int k = 0; k < RM::VEC; ++k) ((float*)out)[row * h + c0 + k] = y[k];
      if (out_b) {  // the same values rounded, beside them
#pragma unroll
        for (int k = 0; k < RM::VEC; ++k) out_b[row * h + c0 + k] = static_cast<bf16_t>(y[k]);
      }
    } else {
      bf16_t yb[RM::VEC];
#pragma unroll
      for (int k = 0; k < RM::VEC; ++k) yb[k] = static_cast<bf16_t>(y[k]);
      if constexpr (RM::VEC == 4) {
        __builtin_nontemporal_store(bf16x4{yb[0], yb[1], yb[2], yb[3]}, (bf16x4*)((bf16_t*)out + row * h + c0));
      } else {
#pragma unroll
        for (int k = 0; k < RM::VEC; ++k) ((bf16_t*)out)[row * h + c0 + k] = yb[k];
      }
      if (out_q) {
#pragma unroll
        for (int k = 0; k < RM::VEC; ++k)
          out_q[row * h + c0 + k].v = f32_to_e4m3(static_cast<float>(yb[k]) * q_inv_scale);
      }
    }
  }
}

// A wave takes one token: its table row is requested before its record is
// looked for, by the whole wave.  Bound by the gathered table rows and the
// output: 874,505 rows of 768, ids spread over 30,522, 841 -> 660 us against a
// search by each lane ahead of the row (6.1 TB/s); two or four rows a wave,
// with one search, were 8 and 28% slower than one.
template <int NPL>
__global__ __launch_bounds__(256) void embed_ln_kernel(const int* __restrict__ ids, const int* __restrict__ cu,
                                                       int B, int T_cap, const float* __restrict__ tok,
                                                       const float* __restrict__ pos, const float* __restrict__ g,
                                                       const float* __restrict__ b, float eps, int vocab,
                                                       int max_pos, void* out, ElemType out_t, fp8_t* out_q,
                                                       float q_inv_scale, int* pos_out, bf16_t* out_b,
                                                       uint32_t* err, const int* t_dev) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= live_rows(T_cap, t_dev)) return;
  constexpr int h = NPL * 64;
  int id = ids[t];
  if (id < 0 || id >= vocab) {
    if (lane == 0) raise_error(err, ANON_ERR_TOKEN_ID);
    id = 0;
  }
  float v[NPL];
  load_row<NPL>(tok + (size_t)id * h, lane, v);
  const int r = wave_find_record(cu, B, t, lane);
  const int p = min(max(t - cu[r], 0), max_pos - 1);
  if (pos_out && lane == 0) pos_out[t] = p;
  if (pos) {  // learned absolute positions (no table: positions enter elsewhere)
    float w[NPL];
    load_row<NPL>(pos + (size_t)p * h, lane, w);
#pragma unroll
    for (int i = 0; i < NPL; ++i) v[i] += w[i];
  }
  float gv[NPL], bv[NPL];
  load_row<NPL>(g, lane, gv);
  load_row<NPL>(b, lane, bv);
  ln_store<NPL>(v, gv, bv, eps, h, lane, t, out, out_t, out_q, q_inv_scale, out_b);
}

// RPW rows per wave: every row's loads are issued before the first
// reduction, so more bytes are in flight per wave.
template <typename TY, int NPL, int RPW>
__global__ __launch_bounds__(256) void layernorm_kernel(const TY* __restrict__ y, const float* __restrict__ g,
                                                        const float* __restrict__ b, float eps, int rows_cap,
                                                        void* out, ElemType out_t, fp8_t* out_q, float q_inv_scale,
                                                        const int* rows_dev) {
  const int lane = threadIdx.x & 63;
  const int rows = live_rows(rows_cap, rows_dev);
  const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW;
  if (row0 >= rows) return;
  constexpr int h = NPL * 64;
  float v[RPW][NPL], gv[NPL], bv[NPL];
#pragma unroll
  for (int k = 0; k < RPW; ++k)
    if (row0 + k < rows) load_row<NPL>(y + (size_t)(row0 + k) * h, lane, v[k]);
  load_row<NPL>(g, lane, gv);
  load_row<NPL>(b, lane, bv);
#pragma unroll
  for (int k = 0; k < RPW; ++k)
    if (row0 + k < rows) ln_store<NPL>(v[k], gv, bv, eps, h, lane, row0 + k, out, out_t, out_q, q_inv_scale);
}

template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>());
  }
}

constexpr int kMaxLabels = 64;

// Token classifier on the FP32 matrix cores (C <= 16 NB labels): a wave forms
// z^T = Wc x^T for 16 tokens with v_mfma_f32_16x16x4_f32, exact products of
// the FP32 head and the (bf16 or FP32) hidden state, FP32 sums.  Lane group q
// (16 lanes) feeds k-index q of every MFMA from the 16-element slice q & 1 of
// each 32-column chunk, its elements 2e + (q >> 1).  Then lane l holds the
// logits of token (l & 15) for classes n*16 + (l/16)*4 + r; the four groups
// merge their top-2 with two exchanges (ties to the lowest class).
//
// The head is laid out in LDS once per workgroup in the order in which lanes
// read it (every read 1 KB without conflicts); the hidden state comes straight
// from memory, kAheadX pairs of chunks in flight.  Bound by latency for a
// small batch and by the MFMAs for a large one, for which two waves a SIMD are
// too few: bf16 rows of 768, 17 labels, us per launch
//   tokens                                            112  18,052  162,529  874,505
//   32x32x2 MFMAs, each chunk's loads waited for     31.1    38.0    107.6      562
//   8 waves a workgroup, 4 pairs in flight           15.3    31.4    109.6      600
//   16 waves, 2 pairs                                13.7    27.2     90.6      517
// (FP32 rows, 123,714 tokens: 145.6, 115.5, 110.0.)
constexpr int kClsWaves = 16;
template <typename TX, int H, int NB>
__global__ __launch_bounds__(kClsWaves * 64) void classifier_mfma_kernel(
    const TX* __restrict__ x, const float* __restrict__ wc, const float* __restrict__ bc, int T_cap, int C,
    uint8_t* __restrict__ labels, float* __restrict__ logits, float* __restrict__ margin, const int* t_dev) {
  constexpr int kPairs = H / 64, kAheadX = 2;
  static_assert(kPairs % kAheadX == 0, "the ring divides the chunks");
  __shared__ floatx4 head[kPairs * 2 * NB * 2 * 64];  // [chunk][n][half][lane] of 4 values
  const int tid = threadIdx.x, lane = tid & 63;
  const int T = live_rows(T_cap, t_dev);
  const int tiles = (T + 15) / 16;
  const int q = lane >> 4, r16 = lane & 15, slice = (q & 1) * 16;
  const bool odd_k = q >> 1;
  typedef TX vec8 __attribute__((ext_vector_type(8)));
  vec8 xv[kAheadX][4];  // pairs of chunks of 16 elements
  auto row = [&](int tile) {  // rows past T re-read row T-1, never stored
    return x + (size_t)max(min(tile * 16 + r16, T - 1), 0) * H + slice;
  };
  auto load = [&](auto slot, const TX* xr, int p) {
#pragma unroll
    for (int e = 0; e < 4; ++e) xv[decltype(slot)::value][e] = *(const vec8*)(xr + p * 64 + (e >> 1) * 32 + (e & 1) * 8);
  };
  int tile = blockIdx.x + gridDim.x * (tid >> 6);
  const TX* xr = row(tile);
  static_for<kAheadX>([&](auto d) { load(d, xr, decltype(d)::value); });
  for (int i = tid; i < NB * 16 * (H / 4); i += kClsWaves * 64) {
    const int c = (i & 15) + i / (16 * (H / 4)) * 16;  // class (16 to a wave: their places' banks differ)
    const int k = (i >> 4) % (H / 4) * 4;              // columns k..k+3
    const floatx4 v = c < C ? *(const floatx4*)(wc + (size_t)c * H + k) : floatx4{0.f, 0.f, 0.f, 0.f};
    const int chunk = k >> 5, in = k & 15, sl = (k >> 4) & 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // element in + j: half (in+j)/8, place (in+j)/2 % 4, of group sl or 2 + sl
      const int e = (in + j) >> 1, group = sl + 2 * (j & 1);
      ((float*)(head + ((chunk * NB + (c >> 4)) * 2 + (e >> 2)) * 64 + group * 16 + (c & 15)))[e & 3] = v[j];
    }
  }
  __syncthreads();
  floatx4 wv[2][NB][2];  // of this chunk and the next
  auto read = [&](floatx4 (&w)[NB][2], int chunk) {
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int f = 0; f < 2; ++f) w[n][f] = head[((chunk * NB + n) * 2 + f) * 64 + lane];
  };
  read(wv[0], 0);
  for (; tile < tiles; tile += gridDim.x * kClsWaves) {
    const int t0 = tile * 16;
    floatx4 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < kPairs; p0 += kAheadX) {
      static_for<kAheadX>([&](auto slot) {
        constexpr int D = decltype(slot)::value;
        const int p = p0 + D;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int next = p * 2 + c + 1 < kPairs * 2 ? p * 2 + c + 1 : 0;  // (chunk 0 for the next tile)
          read(wv[1 - c], next);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x0 = static_cast<float>(xv[D][2 * c + (e >> 2)][(2 * e) & 7]);
            const float x1 = static_cast<float>(xv[D][2 * c + (e >> 2)][(2 * e + 1) & 7]);
            const float xe = odd_k ? x1 : x0;
#pragma unroll
            for (int n = 0; n < NB; ++n)
              acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[c][n][e >> 2][e & 3], xe, acc[n], 0, 0, 0);
          }
        }
        if (p + kAheadX < kPairs) load(slot, xr, p + kAheadX);
        __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the next MFMAs)
      });
    }
    xr = row(tile + gridDim.x * kClsWaves);
    static_for<kAheadX>([&](auto d) { load(d, xr, decltype(d)::value); });
    float best = -INFINITY, second = -INFINITY;
    int arg = 0;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = n * 16 + q * 4 + r;  // increasing
        if (c < C) {
          const float z = acc[n][r] + bc[c];
          if (logits && t0 + r16 < T) logits[(size_t)(t0 + r16) * C + c] = z;
          if (z > best) {
            second = best;
            best = z;
            arg = c;
          } else if (z > second) {
            second = z;
          }
        }
      }
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
      const float ob = __shfl_xor(best, o, 64), os = __shfl_xor(second, o, 64);
      const int oa = __shfl_xor(arg, o, 64);
      if (best > ob) {
        second = fmaxf(second, ob);
      } else if (ob > best) {
        second = fmaxf(os, best);
        best = ob;
        arg = oa;
      } else {
        arg = min(arg, oa);
        second = best;
      }
    }
    if (q == 0 && t0 + r16 < T) {
      labels[t0 + r16] = (uint8_t)arg;
      if (margin) margin[t0 + r16] = C > 1 ? best - second : INFINITY;
    }
  }
}

template <typename TX, int NPL>
__global__ __launch_bounds__(256) void classifier_kernel(const TX* __restrict__ x, const float* __restrict__ wc,
                                                         const float* __restrict__ bc, int T_cap, int C,
                                                         uint8_t* __restrict__ labels, float* __restrict__ logits,
                                                         float* __restrict__ margin, const int* t_dev) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= live_rows(T_cap, t_dev)) return;
  constexpr int h = NPL * 64;
  float xv[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) xv[i] = ldf(x + (size_t)t * h + lane + 64 * i);
  float best = -INFINITY, second = -INFINITY, mine = 0.f;
  int arg = 0;
  for (int c = 0; c < C; ++c) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NPL; ++i) s += xv[i] * wc[(size_t)c * h + lane + 64 * i];
    const float z = wave_sum(s) + bc[c];
    if (lane == c) mine = z;
    if (z > best) {
      second = best;
      best = z;
      arg = c;
    } else if (z > second) {
      second = z;
    }
  }
  if (logits && lane < C) logits[(size_t)t * C + lane] = mine;
  if (lane == 0) {
    labels[t] = (uint8_t)arg;
    if (margin) margin[t] = C > 1 ? best - second : INFINITY;
  }
}

// Four elements a thread and step, four steps in flight: 855,000 x 768 bf16
// 1504 -> 659 us (6 TB/s) (an element per thread, stores of 4 bytes, before).  out
// need not be aligned to more than its elements.
struct __attribute__((packed, aligned(4))) Out4 {
  floatx4 v;
};
template <typename TX>
__global__ __launch_bounds__(256) void to_f32_kernel(const TX* __restrict__ x, float* __restrict__ out, int64_t n) {
  typedef TX vec4 __attribute__((ext_vector_type(4)));
  const int64_t i0 = (int64_t)blockIdx.x * 4096 + threadIdx.x * 4;
  if (((int64_t)blockIdx.x + 1) * 4096 <= n) {
    vec4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __builtin_nontemporal_load((const vec4*)(x + i0 + k * 1024));
#pragma unroll
    for (int k = 0; k < 4; ++k) ((Out4*)(out + i0 + k * 1024))->v = __builtin_convertvector(v[k], floatx4);
    return;
  }
  for (int k = 0; k < 4; ++k)
    for (int e = 0; e < 4; ++e)
      if (i0 + k * 1024 + e < n) out[i0 + k * 1024 + e] = ldf(x + i0 + k * 1024 + e);
}

// dst[c][r] = src[r][c] * inv_scale, converted to the storage type.
template <typename TD>
__global__ __launch_bounds__(256) void transpose_convert_kernel(const float* __restrict__ src, int rows, int cols,
                                                                TD* __restrict__ dst, float inv_scale) {
  __shared__ float tile[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    tile[k][tx] = (r < rows && c < cols) ? src[(size_t)r * cols + c] : 0.f;
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int c = c0 + k, r = r0 + tx;
    if (c < cols && r < rows) {
      const float v = tile[tx][k] * inv_scale;
      if constexpr (sizeof(TD) == 4) dst[(size_t)c * rows + r] = v;
      else if constexpr (sizeof(TD) == 2) dst[(size_t)c * rows + r] = static_cast<bf16_t>(v);
      else dst[(size_t)c * rows + r].v = f32_to_e4m3(v);
    }
  }
}

__global__ void window_gather_kernel(const int* __restrict__ ids, const int* __restrict__ cu,
                                     const int4* __restrict__ win, int* __restrict__ w_ids) {
  const int4 w = win[blockIdx.x];  // (record, start in record, length, first window token)
  const int src = cu[w.x] + w.y;
  for (int i = threadIdx.x; i < w.z; i += blockDim.x) w_ids[w.w + i] = ids[src + i];
}

// 256 tokens a workgroup: each thread finds its token's row, then the rows'
// logits are copied value by value, so that a wave's accesses are contiguous
// (a thread copying its token's row alone: 28 us for 146,000 tokens of 17
// labels, now 12 us).
__global__ __launch_bounds__(256) void window_merge_kernel(const int* __restrict__ cu, int B,
                                                           const int* __restrict__ rec_win0,
                                                           const int4* __restrict__ win, int window, int stride,
                                                           const uint8_t* __restrict__ wl,
                                                           const float* __restrict__ wz,
                                                           const float* __restrict__ wm, int C,
                                                           uint8_t* __restrict__ labels, float* __restrict__ logits,
                                                           float* __restrict__ margin, int T) {
  __shared__ int from[256];
  const int t0 = blockIdx.x * 256, tid = threadIdx.x, t = t0 + tid;
  // the record of the wave's first token, then on from there
  int b = wave_find_record(cu, B, min(t0 + (tid & ~63), T - 1), tid & 63);
  if (t < T) {
    if (b + 1 < B && cu[b + 1] <= t) {  // largest index of [b + 1, B) with cu <= t
      int top = B - 1;
      ++b;
      if (b < top && cu[b + 1] > t) top = b;  // (most often the next record)
      while (b < top) {
        const int m = (b + top + 1) >> 1;
        if (cu[m] <= t) b = m;
        else top = m - 1;
      }
    }
    const int i = t - cu[b];
    const int nw = rec_win0[b + 1] - rec_win0[b];
    const int half = (window - stride) / 2;
    int k = i >= half ? (i - half) / stride : 0;
    k = min(k, nw - 1);
    const int4 w = win[rec_win0[b] + k];
    const int src = w.w + (i - w.y);
    labels[t] = wl[src];
    if (margin) margin[t] = wm[src];
    from[tid] = src;
  }
  if (!logits) return;
  __syncthreads();
  const int n = min(256, T - t0) * C;
  for (int i = tid; i < n; i += 256) {
    const int k = i / C;
    logits[(size_t)t0 * C + i] = wz[(size_t)from[k] * C + (i - k * C)];
  }
}

__global__ void fill_u8_kernel(uint8_t* p, uint8_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Values uniform in [-1, 1) from a 32-bit integer hash of the element index
// (the "lowbias32" mixer of Chris Wellons' hash-prospector): operands with
// the bit statistics of real activations, so that timed kernels draw the
// power (and run at the clock) they do on real data.
__global__ void fill_random_kernel(void* p, ElemType t, int64_t n, uint32_t seed) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    uint32_t x = (uint32_t)i ^ (uint32_t)(i >> 32) * 0x9e3779b9u ^ seed;
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    const float v = (float)(x >> 8) * (1.0f / 8388608.0f) - 1.0f;
    if (t == ET_F32) ((float*)p)[i] = v;
    else if (t == ET_BF16) ((bf16_t*)p)[i] = static_cast<bf16_t>(v);
    else ((fp8_t*)p)[i].v = f32_to_e4m3(v);
  }
}

#define ANON_NPL_SWITCH(NPLV, ...)            \
  switch (NPLV) {                             \
    case 1: { constexpr int NPL = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int NPL = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int NPL = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int NPL = 8; __VA_ARGS__; } break;   \
    case 12: { constexpr int NPL = 12; __VA_ARGS__; } break; \
    case 16: { constexpr int NPL = 16; __VA_ARGS__; } break; \
    default: break;                           \
  }

}  // namespace

void launch_embed_ln(const int* ids, const int* cu_seqlens, int B, int T, const float* tok_emb, const float* pos_emb,
                     const float* g, const float* b, float eps, int vocab, int max_pos, int h, void* out,
                     ElemType out_t, fp8_t* out_q, float q_inv_scale, uint32_t* err, hipStream_t s, int* pos_out,
                     const int* t_dev, bf16_t* out_b) {
  if (T <= 0) return;
  ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((embed_ln_kernel<NPL>), dim3(ceil_div(T, 4)), dim3(256), 0, s, ids,
                                             cu_seqlens, B, T, tok_emb, pos_emb, g, b, eps, vocab, max_pos, out,
                                             out_t, out_q, q_inv_scale, pos_out, out_b, err, t_dev));
}

void launch_layernorm(const void* y, ElemType y_t, const float* g, const float* b, float eps, int rows, int h,
                      void* out, ElemType out_t, fp8_t* out_q, float q_inv_scale, hipStream_t s,
                      const int* rows_dev) {
  if (rows <= 0) return;
  // One row per wave while the launch is bound by the latency of a row (137
  // rows of 768: 3.7 us against 4.1 with two; 21,608: 14.6, 15.7) or a row has
  // the bytes of two (FP32: 126,000 rows 101 us, 104); two BF16 rows where the
  // bytes in flight count (162,000: 84 us against 92; 855,000: 444, 492).
  if (y_t == ET_F32) {
    ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((layernorm_kernel<float, NPL, 1>), dim3(ceil_div(rows, 4)), dim3(256),
                                               0, s, (const float*)y, g, b, eps, rows, out, out_t, out_q, q_inv_scale,
                                               rows_dev));
  } else if (rows < 65536) {
    ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((layernorm_kernel<bf16_t, NPL, 1>), dim3(ceil_div(rows, 4)), dim3(256),
                                               0, s, (const bf16_t*)y, g, b, eps, rows, out, out_t, out_q,
                                               q_inv_scale, rows_dev));
  } else {
    ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((layernorm_kernel<bf16_t, NPL, 2>), dim3(ceil_div(rows, 8)), dim3(256),
                                               0, s, (const bf16_t*)y, g, b, eps, rows, out, out_t, out_q,
                                               q_inv_scale, rows_dev));
  }
}

void launch_classifier(const void* x, ElemType x_t, const float* wc_t, const float* bc, int T, int h, int C,
                       uint8_t* labels, float* logits, float* margin, hipStream_t s, const int* t_dev) {
  if (T <= 0) return;
  if (C <= 32) {
    // a workgroup per tile of 16 tokens up to one per CU, then a wave each
    const int blocks = std::min(ceil_div(T, 16), 256);
#define ANON_CLS_MFMA_N(TX, HV, NB)                                                                               \
  hipLaunchKernelGGL((classifier_mfma_kernel<TX, HV, NB>), dim3(blocks), dim3(kClsWaves * 64), 0, s, (const TX*)x,   \
                     wc_t, bc, T, C, labels, logits, margin, t_dev)
#define ANON_CLS_MFMA(HV)                                   \
  case HV:                                                  \
    if (x_t == ET_F32 && C <= 16) ANON_CLS_MFMA_N(float, HV, 1); \
    else if (x_t == ET_F32) ANON_CLS_MFMA_N(float, HV, 2);  \
    else if (C <= 16) ANON_CLS_MFMA_N(bf16_t, HV, 1);       \
    else ANON_CLS_MFMA_N(bf16_t, HV, 2);                    \
    return;
    switch (h) {
      ANON_CLS_MFMA(128)
      ANON_CLS_MFMA(256)
      ANON_CLS_MFMA(512)
      ANON_CLS_MFMA(768)
      ANON_CLS_MFMA(1024)
      default:
        break;
    }
#undef ANON_CLS_MFMA_N
#undef ANON_CLS_MFMA
  }
  if (x_t == ET_F32) {
    ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((classifier_kernel<float, NPL>), dim3(ceil_div(T, 4)), dim3(256), 0,
                                               s, (const float*)x, wc_t, bc, T, C, labels, logits, margin, t_dev));
  } else {
    ANON_NPL_SWITCH(h / 64, hipLaunchKernelGGL((classifier_kernel<bf16_t, NPL>), dim3(ceil_div(T, 4)), dim3(256), 0,
                                               s, (const bf16_t*)x, wc_t, bc, T, C, labels, logits, margin, t_dev));
  }
}

void launch_to_f32(const void* x, ElemType t, float* out, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  const int grid = (int)((n + 4095) / 4096);
  if (t == ET_F32) hipLaunchKernelGGL(to_f32_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)x, out, n);
  else hipLaunchKernelGGL(to_f32_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)x, out, n);
}

void launch_transpose_convert(const float* src, int rows, int cols, void* dst, ElemType t, float inv_scale,
                              hipStream_t s) {
  dim3 grid(ceil_div(cols, 32), ceil_div(rows, 32));
  if (t == ET_F32)
    hipLaunchKernelGGL(transpose_convert_kernel<float>, grid, dim3(256), 0, s, src, rows, cols, (float*)dst,
                       inv_scale);
  else if (t == ET_BF16)
    hipLaunchKernelGGL(transpose_convert_kernel<bf16_t>, grid, dim3(256), 0, s, src, rows, cols, (bf16_t*)dst,
                       inv_scale);
  else
    hipLaunchKernelGGL(transpose_convert_kernel<fp8_t>, grid, dim3(256), 0, s, src, rows, cols, (fp8_t*)dst,
                       inv_scale);
}

void launch_window_gather(const int* ids, const int* cu_seqlens, const int4* windows, int n_windows, int* w_ids,
                          hipStream_t s) {
  if (n_windows <= 0) return;
  hipLaunchKernelGGL(window_gather_kernel, dim3(n_windows), dim3(256), 0, s, ids, cu_seqlens, windows, w_ids);
}

void launch_window_merge(const int* cu_seqlens, int B, const int* rec_win0, const int4* windows, int window,
                         int stride, const uint8_t* w_labels, const float* w_logits, const float* w_margin, int C,
                         uint8_t* labels, float* logits, float* margin, int T, hipStream_t s) {
  if (T <= 0) return;
  hipLaunchKernelGGL(window_merge_kernel, dim3(ceil_div(T, 256)), dim3(256), 0, s, cu_seqlens, B, rec_win0, windows,
                     window, stride, w_labels, w_logits, w_margin, C, labels, logits, margin, T);
}

void launch_fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_u8_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, s, p, v, n);
}

void launch_fill_random(void* p, ElemType t, int64_t n, uint32_t seed, hipStream_t s) {
  if (n <= 0) return;
  const int64_t blocks = std::min<int64_t>(ceil_div(n, 256), 65536);
  hipLaunchKernelGGL(fill_random_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, t, n, seed);
}

}  // namespace anon
