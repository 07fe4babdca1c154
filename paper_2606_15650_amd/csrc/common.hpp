// Shared definitions of the gfx950 kernels and the host runtime of libanon.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/anon.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));

// One FP8-E4M3 (OCP "fn") value in a byte.
struct fp8_t {
  uint8_t v;
};

namespace anon {

// Thread-local last error string; set_error returns `st` for chaining.
anon_status set_error(anon_status st, const std::string& msg);
void clear_error();

#define ANON_HIP_CHECK(expr)                                                             \
  do {                                                                                   \
    hipError_t _e = (expr);                                                              \
    if (_e != hipSuccess)                                                                \
      return ::anon::set_error(ANON_EDEVICE, std::string(#expr ": ") + hipGetErrorString(_e)); \
  } while (0)

// Per-device error word (bits ANON_ERR_*): kernels that check device data
// take its address and raise bits instead of reading or writing out of bounds.
__device__ __forceinline__ void raise_error(uint32_t* err, uint32_t bit) {
  if (err) atomicOr(err, bit);
}

// Address of the current device's error word (allocated once per device),
// or the word set for the calling thread by set_thread_error_word.
uint32_t* error_word_ptr();
// Route the error bits of this thread's later launches to `w` (device
// memory, the caller's); nullptr restores the per-device word.
void set_thread_error_word(uint32_t* w);

constexpr int kWave = 64;

// Rows a launch computes: its capacity `cap` (the grid is sized for it), or,
// when `dev` is given, the count held in device memory clamped to [0, cap].
// A graph captured for a token bucket reads the batch's count this way.
__device__ __forceinline__ int live_rows(int cap, const int* dev) {
  return dev ? max(0, min(*dev, cap)) : cap;
}

__device__ __forceinline__ float bf16_to_float(bf16_t x) { return static_cast<float>(x); }
__device__ __forceinline__ bf16_t float_to_bf16(float x) { return static_cast<bf16_t>(x); }

// FP32 -> OCP E4M3FN, round to nearest even, saturating at +-448.
__device__ __forceinline__ uint8_t f32_to_e4m3(float v) {
  v = fminf(fmaxf(v, -448.0f), 448.0f);
  return (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(v, v, 0, false) & 0xff);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// The same sums in registers: the halves and the rows of 16 are exchanged by
// permlane swaps; once all rows are equal in lanes 8 apart, a rotation by 4
// finds what an exchange with lane ^ 4 would, and so on.  (Bits as above; the
// six exchanges through LDS were a fifth of a small LayerNorm.)
template <>
__device__ __forceinline__ float wave_sum(float v) {
#ifdef __HIP_DEVICE_COMPILE__
  auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x128, 0xf, 0xf, true));  // row_ror:8
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x124, 0xf, 0xf, true));
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x122, 0xf, 0xf, true));
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x121, 0xf, 0xf, true));
#endif
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Largest b in [0, B) with cu[b] <= p (0 if there is none), by the whole
// workgroup: every thread samples one boundary per round, so 65,536 records
// take two dependent loads with 256 threads instead of sixteen.  All threads
// call it with the same arguments and get the same result; a malformed cu
// gives some index of [0, B).
template <typename T>
__device__ __forceinline__ int wg_find_record(const T* cu, int B, T p) {
  const int nt = blockDim.x, tid = threadIdx.x;
  int lo = 0, n = B;
  while (n > 1) {
    const int step = (n + nt - 1) / nt, at = tid * step;
    const int cnt = __syncthreads_count(at < n && (at == 0 || cu[lo + at] <= p));
    lo += (cnt - 1) * step;
    n = min(step, n - (cnt - 1) * step);
  }
  return lo;
}

// The records of two positions p <= q by the same steps.
template <typename T>
__device__ __forceinline__ int2 wg_find_records(const T* cu, int B, T p, T q) {
  const int nt = blockDim.x, tid = threadIdx.x;
  int lo = 0, n = B, lo2 = 0, n2 = B;
  while (n > 1 || n2 > 1) {
    const int step = (n + nt - 1) / nt, at = tid * step, step2 = (n2 + nt - 1) / nt, at2 = tid * step2;
    const T c = at < n ? cu[lo + at] : 0, c2 = at2 < n2 ? cu[lo2 + at2] : 0;
    const int cnt = __syncthreads_count(at < n && (at == 0 || c <= p));
    const int cnt2 = __syncthreads_count(at2 < n2 && (at2 == 0 || c2 <= q));
    lo += (cnt - 1) * step;
    n = min(step, n - (cnt - 1) * step);
    lo2 += (cnt2 - 1) * step2;
    n2 = min(step2, n2 - (cnt2 - 1) * step2);
  }
  return int2{lo, lo2};
}

// f(b) for the records b of [r0, r1] by the whole workgroup, in no order; for
// what only the last of the records that begin at one place need do.  (Where a
// workgroup has few bytes or tokens and more than 1024 records, most are
// empty: runs of as many records as there are threads that begin where the
// record after them does are left out.  A million empty records at one place
// cost a read of two of them per thread and 65,536; one after the other, 256
// at a time, they took 2 ms.)
template <typename T, typename F>
__device__ __forceinline__ void wg_each_record(const T* cu, int r0, int r1, F f) {
  const int nt = blockDim.x, tid = threadIdx.x, lane = tid & 63;
  if (r1 - r0 < 1024) {
    for (int b = r0 + tid; b <= r1; b += nt) f(b);
    return;
  }
  for (int64_t s = r0; s <= r1; s += (int64_t)nt * nt) {
    const int64_t a = s + (int64_t)tid * nt;  // this thread's run
    uint64_t some = __ballot(a <= r1 && cu[a] != cu[min(a + nt, (int64_t)r1 + 1)]);
    for (; some; some &= some - 1) {  // the wave's runs that are not of one place
      const int64_t run = s + (int64_t)(tid - lane + __ffsll((unsigned long long)some) - 1) * nt;
      for (int j = lane; j < nt; j += 64)
        if (run + j <= r1) f((int)(run + j));
    }
  }
}

// The same for the records from r0 on that begin at or before p, r0 the record
// of a byte or token; most often they are few, and no second search is made.
// Ends with a barrier.
template <typename T, typename F>
__device__ __forceinline__ void wg_each_record_to(const T* cu, int B, int r0, T p, F f) {
  const int b = r0 + (int)threadIdx.x;
  const bool in = b < B && cu[b] <= p;
  if (in) f(b);
  if (!__syncthreads_or(in && threadIdx.x == blockDim.x - 1)) return;
  wg_each_record(cu, r0 + (int)blockDim.x, wg_find_record(cu, B, p), f);
  __syncthreads();
}

// The bytes' bit 7 gathered into four bits (a multiplication).
__device__ __forceinline__ uint32_t byte_bits(uint32_t flags) { return (flags >> 7) * 0x10204080u >> 28; }
// Bit 7 of each byte of w: the byte equals c / lies in [lo, hi], lo >= 1, hi <= 127.
__device__ __forceinline__ uint32_t bytes_equal(uint32_t w, uint8_t c) {
  const uint32_t x = w ^ (c * 0x01010101u);
  return ~(((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu);
}
__device__ __forceinline__ uint32_t bytes_between(uint32_t w, uint8_t lo, uint8_t hi) {
  const uint32_t x = w & 0x7f7f7f7fu;
  return (x + (128 - lo) * 0x01010101u) & ~(x + (127 - hi) * 0x01010101u) & ~w & 0x80808080u;
}

// 16 bytes from an address of any alignment
__device__ __forceinline__ uint4 load16(const uint8_t* p) {
  uint4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

// 16 bytes per lane from global memory straight into LDS
// (global_load_lds_dwordx4): lane i's bytes land at l + 16 i, where l is
// the same for the whole wave.
__device__ __forceinline__ void dma16(const void* g, char* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}

// s_waitcnt vmcnt(n) alone (expcnt and lgkmcnt left at their maxima)
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Workspace carving: consecutive 256-byte aligned sub-buffers.
struct Carver {
  char* base;
  size_t used = 0;
  size_t cap;
  Carver(void* b, size_t c) : base((char*)b), cap(c) {}
  template <typename T>
  T* take(size_t n) {
    size_t off = align_up(used, 256);
    used = off + n * sizeof(T);
    return base ? (T*)(base + off) : nullptr;
  }
  bool ok() const { return used <= cap; }
};

// Kernel-class timing (anon_prof_*).
enum KClass { KC_QKV = 0, KC_ATTN, KC_OPROJ, KC_FFN1, KC_FFN2, KC_LN, KC_EMBED, KC_CLS, KC_COUNT };
struct ProfScope {
  int kc;
  hipStream_t s;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  double flops;
  ProfScope(int kc, hipStream_t s, double flops);
  ~ProfScope();
};

}  // namespace anon
