// Dense GEMMs of the encoder on CDNA4 matrix cores, with fused epilogues.
//
// C[M,N] = A[M,K] * W[N,K]^T, A = packed token activations (no padding), W =
// a weight matrix stored transposed so that both operands are K-contiguous.
// One workgroup owns a BM x BN output tile; its waves form a WGM x WGN grid
// and each wave accumulates (BM/WGM) x (BN/WGN) with 32x32 MFMA tiles:
//   fp32: v_mfma_f32_32x32x2_f32      (K step 2)
//   bf16: v_mfma_f32_32x32x16_bf16    (K step 16)
//   fp8 : v_mfma_scale_f32_32x32x64_f8f6f4 with E4M3 operands (K step 64)
// Two main loops: BF16/FP8 operands stream global -> LDS directly through a
// ring of K tiles (XOR-swizzled rows; three forms of it, see gemm_dma_kernel);
// FP32 operands go through registers into double-buffered, padded LDS.  In
// both the MFMA operands of the next k-step are read from LDS while those of
// this one are multiplied.
//
// The K loop always runs in increasing k with one MFMA shape per precision,
// so each output element's sum is formed in the same order whatever the tile
// shape or the row's position in the batch (batch invariance; tile
// configurations are interchangeable bit for bit).
//
// Epilogues: bias (+ exact scaling of the Q columns by 1/sqrt(d)); bias + GELU;
// bias + residual added in FP32 and rounded once to the output type.
#include <math.h>

#include <algorithm>

#include "kernels.hpp"

namespace anon {
namespace {

template <typename T>
struct Mfma;

template <>
struct Mfma<float> {
  typedef float frag;
  static constexpr int KI = 2, KPL = 1;
  __device__ static floatx16 mma(frag a, frag b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mfma<bf16_t> {
  typedef bf16x8 frag;
  static constexpr int KI = 16, KPL = 8;
  __device__ static floatx16 mma(frag a, frag b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mfma<fp8_t> {
  typedef intx8 frag;
  static constexpr int KI = 64, KPL = 32;
  // operand formats 0/0 = E4M3 x E4M3; block scales 127 = 2^0 (unscaled)
  __device__ static floatx16 mma(frag a, frag b, floatx16 c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
  }
};

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16_t* p) { return static_cast<float>(*p); }
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ void st(bf16_t* p, float v) { *p = static_cast<bf16_t>(v); }
__device__ __forceinline__ void st(fp8_t* p, float v) { p->v = f32_to_e4m3(v); }

// GELU(v) = v/2 (1 + erf(v / sqrt 2)) with erf from Abramowitz & Stegun
// formula 7.1.26 (rational approximation, |error| <= 1.5e-7): far below the
// bf16 output rounding and the FP32 path's 1e-4 logit tolerance, and a third
// of the instructions of a full-precision erff in an epilogue that runs
// once per output element.
__device__ __forceinline__ float gelu_erf(float v) {
  // Phi(v) = 1 - q for v >= 0 and q for v < 0, with q = P(t) exp(-v^2/2) / 2,
  // t = 1 / (1 + p |v| / sqrt 2); the 1/2 and 1/sqrt 2 are folded into the
  // constants, and exp(-v^2/2) = exp2(-(v sqrt(log2(e)/2))^2)
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, fabsf(v), 1.0f));
  const float P = ((((0.5f * 1.061405429f * t - 0.5f * 1.453152027f) * t + 0.5f * 1.421413741f) * t -
                    0.5f * 0.284496736f) * t + 0.5f * 0.254829592f) * t;
  const float sv = v * 0.84932180028801904f;
  const float r = v * (P * __builtin_amdgcn_exp2f(-(sv * sv)));
  // v - r for v >= 0 and r for v < 0: since q <= 1/2, r = v q lies between
  // 0 and v/2, so the wanted value is always the larger of the two
  return fmaxf(v - r, r);
}

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous run of tiles so that the tiles sharing an A row-block (and the
// weight panel) meet in the same L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
  const int X = 8;
  const int per = nb / X, rem = nb % X;
  const int x = bid % X, loc = bid / X;
  return x * per + min(x, rem) + loc;
}

// Linear tile index -> (row block, column block), in groups of `gm` row
// blocks walked column by column: the tiles in flight on one XCD then share
// a few A row blocks and a few weight column panels, a working set that fits
// its L2, instead of cycling through the whole weight matrix per row block.
__device__ __forceinline__ void group_tile(int t, int ntm, int ntn, int gm, int& mb, int& nb) {
  const int per_group = gm * ntn;
  const int g = t / per_group, r = t - g * per_group;
  const int m0 = g * gm, gsz = min(ntm - m0, gm);
  mb = m0 + r % gsz;
  nb = r / gsz;
}

struct DevParams {
  const void* A;
  const void* W;
  const float* bias;
  const void* resid;
  void* C;
  int M, N, K;
  float qscale;
  int qcols;
  float acc_scale;
  float out_inv_scale;
  int group_m;
  int ldc;            // output row stride (elements)
  const int* pos;     // EPI_ROPE: position of each row within its record
  const float* rope;  // EPI_ROPE: [max_pos][64] cos (first 32) and sin (last 32)
  int rope_cols;      // EPI_ROPE: columns below this are rotated
  const int* m_dev;   // non-null: rows to compute (device), M is the grid's capacity
};

// The MFMAs take the weight fragment as their first operand, so each
// accumulator holds a 32x32 block of C^T: lane l, register r holds row
// (l & 31) and column (r/4)*8 + (l/32)*4 + r%4 of the block -- four
// consecutive columns of one row per register quad.
//
// Epilogue: once the K loop is done, the operand LDS is reused.  Each wave
// forms its outputs -- bias, Q scaling, GELU or the residual (copied first
// into the LDS slots its outputs take, added in FP32, rounded once) -- and
// parks them in its own LDS region in the output type, then writes the
// region back with 16-byte row-contiguous stores.  Loads come before stores wherever possible: on
// this architecture loads and stores share one counter, so a load issued
// after a store waits for the store to be acknowledged.  The region holds
// whole 32-row strips (see Staging::NS).  Rows are unpadded, with 16-byte chunks
// XOR-permuted by the row (chunk c of row r in slot c ^ (r mod 16)) so that
// the 32 rows a register quad spans land on distinct bank groups.
template <typename TO, int EPI, int TM, int TN, int NW, int SMEM>
struct Staging {
  // output columns of a wave: the gated epilogue writes one of each pair
  // of 32-column sub-blocks
  static constexpr int OTN = EPI == EPI_GEGLU ? TN / 2 : TN;
  static constexpr int ROWB = OTN * 32 * (int)sizeof(TO);       // bytes per staged row
  static constexpr int CPR = ROWB / 16;                          // 16-byte chunks per row
  static constexpr int SWZ = (CPR < 16 ? CPR : 16) - 1;
  static constexpr int STRIP = 32 * ROWB;                        // one 32-row strip of one wave
  static constexpr int FIT = SMEM / (NW * STRIP) < TM ? SMEM / (NW * STRIP) : TM;
  // strips per pass: the residual epilogue loads, so it stages as much as
  // fits before its first store; the others load nothing after the bias and
  // go strip by strip, one strip's stores draining under the next's math
  static constexpr int NS = EPI == EPI_RESID ? FIT : 1;
  static_assert(NS >= 1 && CPR >= 2 && (CPR & (CPR - 1)) == 0, "epilogue staging does not fit");
  static_assert((NS * 32 * CPR) % 64 == 0, "write-back covers whole waves");
};

template <typename T>
__device__ __forceinline__ void ld4(const T* p, float (&v)[4]);
template <>
__device__ __forceinline__ void ld4(const float* p, float (&v)[4]) {
  const floatx4 x = *(const floatx4*)p;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = x[e];
}
template <>
__device__ __forceinline__ void ld4(const bf16_t* p, float (&v)[4]) {
  const bf16x4 x = *(const bf16x4*)p;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = static_cast<float>(x[e]);
}

__device__ __forceinline__ void st4(float* p, const float (&v)[4]) { *(floatx4*)p = floatx4{v[0], v[1], v[2], v[3]}; }
__device__ __forceinline__ void st4(bf16_t* p, const float (&v)[4]) {
  *(bf16x4*)p = bf16x4{static_cast<bf16_t>(v[0]), static_cast<bf16_t>(v[1]), static_cast<bf16_t>(v[2]),
                       static_cast<bf16_t>(v[3])};
}
__device__ __forceinline__ void st4(fp8_t* p, const float (&v)[4]) {
  float c[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) c[e] = fminf(fmaxf(v[e], -448.0f), 448.0f);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w, true);
  *(int*)p = w;
}

// Bias of a lane's columns (loaded before any store).
template <int TN>
__device__ __forceinline__ void load_bias(const DevParams& p, int lane, int wcol0, floatx4 (&bias)[TN][4]) {
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[j][q] = *(const floatx4*)(p.bias + wcol0 + j * 32 + q * 8 + (lane >> 5) * 4);
}

// Applies the epilogue to a wave's (TM*32) x (TN*32) accumulator block whose
// top-left output element is (wrow0, wcol0).
template <typename TO, typename TR, int EPI, int TM, int TN, int NW, int SMEM>
__device__ __forceinline__ void epilogue(const DevParams& p, floatx16 (&acc)[TM][TN], char* smem, int wave, int lane,
                                         int M, int wrow0, int wcol0,
                                         const floatx4 (&bias)[TN][4]) {
  typedef Staging<TO, EPI, TM, TN, NW, SMEM> SG;
  constexpr int ROWB = SG::ROWB, CPR = SG::CPR, SWZ = SG::SWZ, NS = SG::NS;
  const int N = p.N;
  constexpr bool PAIRED = EPI == EPI_ROPE || EPI == EPI_GEGLU;
  static_assert(!PAIRED || TN % 2 == 0, "paired epilogues need whole 64-column blocks per wave");
  static_assert(EPI != EPI_GEGLU || sizeof(TO) >= 2, "the gated epilogue writes bf16 or fp32");
  // where this wave's outputs start in a row of C
  const int ocol0 = EPI == EPI_GEGLU ? wcol0 / 2 : wcol0;
  char* stg = smem + wave * (SMEM / NW / 1024 * 1024);
  const int lrow = lane & 31, lq = (lane >> 5) * 4;
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += NS) {
    if constexpr (EPI == EPI_RESID) {
      // 0. the residual of strips [i0, i0 + NS) straight into the staging
      // slots its outputs take (residual and output have one element size):
      // 16-byte row-contiguous global -> LDS copies, lane l of a copy taking
      // slot l % CPR of staged row (copy rows) + l / CPR, i.e. the chunk
      // that the row's XOR permutation puts there.  Read per lane in the
      // accumulator layout instead, every load would touch 32 rows for 16
      // bytes of each.
      static_assert(sizeof(TR) == sizeof(TO), "the residual is staged in the output's layout");
      static_assert(ROWB <= 1024 && 1024 % ROWB == 0, "whole staged rows per copy instruction");
      constexpr int RPC = 1024 / ROWB;  // staged rows per copy instruction
      const int nss = min(TM - i0, NS);  // strips of this pass
      const int crow = lane / CPR, cslot = lane % CPR;
      // a uniform base row (rows past M re-read row M-1, which the clamped
      // base keeps at or below every lane's row) and 32-bit lane offsets
      const int brow = min(wrow0 + i0 * 32, M - 1);
      const char* rbase = (const char*)p.resid + ((size_t)brow * N + wcol0) * sizeof(TR);
#pragma unroll
      for (int t = 0; t < NS * 32 / RPC; ++t) {
        if (t * RPC >= nss * 32) break;
        const int srow = t * RPC + crow;
        const int grow = min(wrow0 + (i0 + (srow >> 5)) * 32 + (srow & 31), M - 1);
        const uint32_t off = (uint32_t)((grow - brow) * N * (int)sizeof(TR) + (cslot ^ (srow & SWZ)) * 16);
        dma16(rbase + off, stg + t * 1024);
      }
      wait_vmcnt<0>();
    }
    // 1. outputs of strips [i0, i0 + NS) into LDS
#pragma unroll
    for (int is = 0; is < NS && i0 + is < TM; ++is) {
      const int i = i0 + is;
      const int srow = is * 32 + lrow;  // staged row
      const int grow = min(wrow0 + i * 32 + lrow, M - 1);
      if constexpr (PAIRED) {
        // sub-blocks j and j+1 hold the two members of each pair: columns
        // c and c + 32 of a 64-column head block (RoPE), or the input and
        // the gate half of the gated MLP (weights interleaved in 32-column
        // blocks)
        int prow = 0;
        if constexpr (EPI == EPI_ROPE) prow = p.pos[grow];
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          const bool rot = EPI == EPI_ROPE && wcol0 + j * 32 < p.rope_cols;
          const bool qs = EPI == EPI_ROPE && wcol0 + j * 32 < p.qcols;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int d0 = q * 8 + lq;  // index within the 32-column sub-block
            float a[4], b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              a[e] = acc[i][j][q * 4 + e] * p.acc_scale + bias[j][q][e];
              b[e] = acc[i][j + 1][q * 4 + e] * p.acc_scale + bias[j + 1][q][e];
            }
            if constexpr (EPI == EPI_ROPE) {
              if (rot) {
                const floatx4 cs = *(const floatx4*)(p.rope + (size_t)prow * 64 + d0);
                const floatx4 sn = *(const floatx4*)(p.rope + (size_t)prow * 64 + 32 + d0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const float x1 = a[e], x2 = b[e];
                  a[e] = x1 * cs[e] - x2 * sn[e];
                  b[e] = x2 * cs[e] + x1 * sn[e];
                }
              }
              if (qs) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  a[e] *= p.qscale;
                  b[e] *= p.qscale;
                }
              }
              const int ba = (j * 32 + d0) * (int)sizeof(TO), bb = ((j + 1) * 32 + d0) * (int)sizeof(TO);
              st4((TO*)(stg + srow * ROWB + (((ba >> 4) ^ (srow & SWZ)) * 16) + (ba & 15)), a);
              st4((TO*)(stg + srow * ROWB + (((bb >> 4) ^ (srow & SWZ)) * 16) + (bb & 15)), b);
            } else {
              float y[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = gelu_erf(a[e]) * b[e];
              const int by = ((j / 2) * 32 + d0) * (int)sizeof(TO);
              st4((TO*)(stg + srow * ROWB + (((by >> 4) ^ (srow & SWZ)) * 16) + (by & 15)), y);
            }
          }
        }
        continue;
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        // the Q columns are whole 32-column blocks (qcols is a multiple of 64)
        const bool qs = EPI == EPI_BIAS && wcol0 + j * 32 < p.qcols;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int cl = j * 32 + q * 8 + lq;  // column within the wave's block
          const int byte = cl * (int)sizeof(TO);
          const int chunk = (byte >> 4) ^ (srow & SWZ);
          char* slot = stg + srow * ROWB + chunk * 16 + (byte & 15);
          float rv[4] = {0.f, 0.f, 0.f, 0.f};
          if constexpr (EPI == EPI_RESID) ld4((const TR*)slot, rv);  // staged above
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float x = acc[i][j][q * 4 + e] * p.acc_scale + bias[j][q][e];
            if (EPI == EPI_BIAS) {
              if (qs) x *= p.qscale;
            } else if (EPI == EPI_GELU) {
              x = gelu_erf(x);
              // FP8 output: the activation is a bf16 value first (as in the
              // BF16 path), then scaled and rounded to E4M3
              if (sizeof(TO) == 1) x = static_cast<float>(static_cast<bf16_t>(x)) * p.out_inv_scale;
            } else {
              x += rv[e];
            }
            v[e] = x;
          }
          st4((TO*)slot, v);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // 2. the strips back to memory, 16 bytes per lane, row-contiguous
    constexpr int NCH = NS * 32 * CPR;
#pragma unroll
    for (int c0 = 0; c0 < NCH; c0 += 64) {
      const int c = c0 + lane;  // NCH is a multiple of 64
      const int srow = c / CPR, cc = c % CPR;
      const int i = i0 + srow / 32;  // past TM only in a last, partial pass
      const int grow = wrow0 + i * 32 + (srow & 31);
      const intx4 v = *(const intx4*)(stg + srow * ROWB + ((cc ^ (srow & SWZ)) * 16));
      // (single-use streams: the next kernel reads them from memory)
      if (i < TM && grow < M)
        __builtin_nontemporal_store(v, (intx4*)((char*)p.C + ((size_t)grow * p.ldc + ocol0) * sizeof(TO) + cc * 16));
    }
    if (i0 + NS < TM) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
  }
}

// Register-staged kernel (FP32 operands): the next K tile is fetched into
// registers while the current one is multiplied from double-buffered,
// row-padded LDS (16 bytes of padding per row keeps the 16-byte fragment
// reads of 16 lanes on distinct banks).
template <typename TI, typename TO, typename TR, int EPI, int BM, int BN, int BK, int WGM, int WGN, int OCC>
__global__ __launch_bounds__(WGM* WGN * 64, OCC) void gemm_kernel(DevParams p) {
  typedef Mfma<TI> MF;
  typedef typename MF::frag frag;
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int EPC = 16 / (int)sizeof(TI);  // elements per 16-byte chunk
  constexpr int CPR = BK / EPC;              // chunks per tile row
  constexpr int LDK = BK + EPC;              // padded LDS row (16 bytes)
  constexpr int A_CH = BM * CPR / NT, B_CH = BN * CPR / NT;
  constexpr int NKS = BK / MF::KI;
  static_assert((BM * CPR) % NT == 0 && (BN * CPR) % NT == 0, "tile/threads mismatch");
  static_assert(TM >= 1 && TN >= 1 && BK % MF::KI == 0, "bad tile");
  constexpr int OPND_BYTES = 2 * (BM + BN) * LDK * (int)sizeof(TI);
  __shared__ __align__(16) char smem[OPND_BYTES];
  TI(*As)[BM * LDK] = reinterpret_cast<TI(*)[BM * LDK]>(smem);
  TI(*Bs)[BN * LDK] = reinterpret_cast<TI(*)[BN * LDK]>(smem + 2 * BM * LDK * sizeof(TI));

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int N = p.N, K = p.K;
  // the tiles of the rows to compute; with a device row count the grid may
  // hold more workgroups, which leave at once, and the live tiles are spread
  // over the XCDs as in a launch of exactly their number
  const int M = live_rows(p.M, p.m_dev);
  const int ntn = N / BN;
  const int ntm = (M + BM - 1) / BM;
  if ((int)blockIdx.x >= ntm * ntn) return;
  int mb, nb;
  group_tile(xcd_remap(blockIdx.x, ntm * ntn), ntm, ntn, p.group_m, mb, nb);
  const int m0 = mb * BM, n0 = nb * BN;

  const TI* __restrict__ A = (const TI*)p.A;
  const TI* __restrict__ W = (const TI*)p.W;

  intx4 ra[A_CH], rb[B_CH];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int c = tid + i * NT, r = c / CPR, cc = c % CPR;
      // rows past M (last tile only) re-read row M-1: their results are
      // never stored, and the load needs no branch
      const int gm = min(m0 + r, M - 1);
      ra[i] = *(const intx4*)(A + (size_t)gm * K + k0 + cc * EPC);
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int c = tid + i * NT, r = c / CPR, cc = c % CPR;
      rb[i] = *(const intx4*)(W + (size_t)(n0 + r) * K + k0 + cc * EPC);
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int c = tid + i * NT, r = c / CPR, cc = c % CPR;
      *(intx4*)&As[buf][r * LDK + cc * EPC] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int c = tid + i * NT, r = c / CPR, cc = c % CPR;
      *(intx4*)&Bs[buf][r * LDK + cc * EPC] = rb[i];
    }
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int KT = K / BK;
  gload(0);
  lstore(0);
  __syncthreads();
  const int arow = wm * WTM + (lane & 31), brow = wn * WTN + (lane & 31);
  const int kofs = (lane >> 5) * MF::KPL;
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < KT) gload((kt + 1) * BK);
    const TI* as = As[buf];
    const TI* bs = Bs[buf];
    frag a[2][TM], b[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[0][i] = *(const frag*)&as[(arow + i * 32) * LDK + kofs];
#pragma unroll
    for (int j = 0; j < TN; ++j) b[0][j] = *(const frag*)&bs[(brow + j * 32) * LDK + kofs];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int cur = ks & 1;
      if (ks + 1 < NKS) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          a[cur ^ 1][i] = *(const frag*)&as[(arow + i * 32) * LDK + (ks + 1) * MF::KI + kofs];
#pragma unroll
        for (int j = 0; j < TN; ++j)
          b[cur ^ 1][j] = *(const frag*)&bs[(brow + j * 32) * LDK + (ks + 1) * MF::KI + kofs];
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(b[cur][j], a[cur][i], acc[i][j]);
    }
    if (kt + 1 < KT) lstore(buf ^ 1);
    __syncthreads();
  }
  floatx4 bias[TN][4];
  load_bias(p, lane, n0 + wn * WTN, bias);
  epilogue<TO, TR, EPI, TM, TN, WGM * WGN, OPND_BYTES>(p, acc, smem, wave, lane, M, m0 + wm * WTM, n0 + wn * WTN, bias);
}

// LDS-ring kernel (BF16 / FP8 operands).  Each K tile travels from global
// memory straight into LDS (global_load_lds_dwordx4: no register staging),
// ST tiles deep, so the loads of tile k+ST-1 are in flight while tile k is
// multiplied.  One barrier per K tile: after it, every wave's copy of tile k
// has landed and every wave has finished reading tile k-1, whose slot then
// takes tile k+ST-1.
//
// kAhead: the two operands have slots of their own, three for A and two for
// W, and run at different distances: A two K tiles ahead, W one.  An
// activation row block is read from beyond the L2 (1-2 us under load) by the
// few tiles of its row, while a weight panel is shared by every row block in
// flight and mostly hits it, so the same 160 KB that a two-stage ring leaves
// a fifth of free cover the longer latency.  Every refill is branch-free
// inside the MFMA block (the last three tiles are peeled), so its issue hides
// behind the MFMAs; in the two-stage ring the refill's branch split the block
// and the eight copies went out with the matrix pipe idle.  At 855,055 rows
// of the base encoder (256x256x64): QKV 2.99 -> 2.79 ms, output projection
// 1.17 -> 1.14, FFN1 4.76 -> 4.57, FFN2 3.64 -> 3.42 per launch; one tile
// alone on the chip, K = 3072: 60.7 -> 54.2 us (a K tile 2690 -> 2380 clocks,
// 2048 of them MFMA).  At full load the shader clock falls (QKV 1.76 GHz, output
// projection 1.96, FFN1 1.89, FFN2 1.74) and a K tile takes 2400-2600 of its
// clocks, so the matrix pipe is 80-85% busy outside the epilogue.  What holds
// the rest is not settled: a library's kernel does the output projection and
// FFN2 shapes, without the residual, in 0.98 and 3.01 ms.  A layout of 4
// waves of 128x128 with its accumulators pinned in AGPRs reads a third less
// LDS but has nothing to run while its one wave per SIMD waits: 3.06 / 1.29 /
// 4.80 / 3.59 ms with the same ring, not kept.
//
// Where the epilogue stages no more than a wave's own part of A's third slot
// (stays()), a workgroup keeps its CU for every 256th tile: the next tile's
// first copies, all but those into that slot, travel during the epilogue.  855,055 rows: FFN1 4.71 -> 4.54 ms, QKV
// 2.76 -> 2.72; the epilogue itself (the GELU is 92 of its clocks per element
// and wave) still runs with the matrix pipe idle, and two workgroups of 128x256
// tiles per CU, which overlap it, lose more in the main loop (QKV of 200,000
// rows 644 us against 789, FFN1 1037 against 1087).  FP8 spills with it.
//
// kTileRegs: for batches so small that a CU has one tile and what counts is
// how long one K tile takes.  With one or four 32x32 blocks in a workgroup a
// k-step is a single MFMA, too short to cover the LDS reads of the next, and
// one or two waves do not issue copies fast enough.  So the fragments of a
// whole K tile are read under the MFMAs of the tile before, eight waves share
// the copies, and a tile costs one barrier and no other wait.  137 rows of the
// base encoder: 5.2, 5.4, 5.8 and 12.1 us -> 4.8, 4.6, 5.3 and 8.7 for the four
// GEMMs of a layer (a K tile of 128 530 clocks instead of 900); deeper rings
// change nothing.
//
// LDS layout: rows of BK elements, unpadded, with the 16-byte chunks of a
// row XOR-permuted by a function of the row (chunk c of row r sits in slot
// c ^ swz(r)): a 16-lane group reading the same logical chunk of 16
// consecutive rows then touches 16 distinct 16-byte bank groups, and one
// wave's load instruction fills 1024 contiguous bytes.
template <int CPR>
__device__ __forceinline__ int lds_swz(int r) {
  static_assert(CPR == 4 || CPR == 8 || CPR == 16, "rows of 64, 128 or 256 bytes");
  return CPR == 16 ? r & 15 : CPR == 8 ? (r >> 1) & 7 : (r >> 2) & 3;
}

// dma16 with the source given as a uniform base, a lane offset and a uniform
// offset (buffer_load_dwordx4 ... lds): no 64-bit address is formed per lane,
// so a refill in the main loop is one instruction.  The descriptor covers
// 2 GiB from the base; the callers' offsets stay inside their matrix.
__device__ __forceinline__ void buf16(const char* base, uint32_t voff, int soff, char* l) {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000),
                                           (__attribute__((address_space(3))) void*)l, 16, voff, soff, 0, 0);
#endif
}
// p, known to be the same for every lane, in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// Waits until at most `left` K tiles (of LPT load instructions each) issued
// after the wanted one are in flight; MAX of them is the ring's steady state,
// fewer remain at the end of the K loop, where nothing is issued any more.
template <int MAX, int LPT>
__device__ __forceinline__ void wait_tiles(int left) {
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (left >= MAX) wait_vmcnt<MAX * LPT>();
    else wait_tiles<MAX - 1, LPT>(left);
  }
}

// Instruction order of one k-step (a scheduling region): the next k-step's
// fragment reads go out two per MFMA from the first MFMA on, so their
// latency hides behind the rest of the step's MFMA chain; then the ring
// refill loads (last k-step of a tile), two per MFMA; then the other MFMAs.
template <int NMF, int NRD, int NVM>
__device__ __forceinline__ void sched_step() {
  constexpr int RG = (NRD + 1) / 2, VG = (NVM + 1) / 2;
#pragma unroll
  for (int r = 0; r < NRD / 2; ++r) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // DS read
  }
  if constexpr (NRD % 2) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
#pragma unroll
  for (int v = 0; v < NVM / 2; ++v) {
    if (RG + v < NMF) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x010, 2, 0);  // VMEM
  }
  if constexpr (NVM % 2) {
    if (RG + VG - 1 < NMF) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
  }
  if constexpr (NMF > RG + VG) __builtin_amdgcn_sched_group_barrier(0x008, NMF - RG - VG, 0);
}

// "Ring stages" of the ring that runs A two K tiles and W one K tile ahead
// (see gemm_dma_kernel).
constexpr int kAhead = -1;
// A ring of ST - kTileRegs stages for a few tiles on an empty chip (see
// gemm_dma_kernel): kLoaders waves load, WGM x WGN of them multiply.
constexpr int kTileRegs = 100;
constexpr int kLoaders = 8;

// Whether a workgroup stays for several tiles, by the kernel and by its
// launch: it has a CU to itself, and its epilogue needs no more LDS than A's
// third slot (BM x BK).  BF16: the 256x256 tiles but with the residual
// epilogue, with the gated one, which writes half as many columns, all of one
// workgroup per CU.
template <typename TI, typename TO, int EPI, int BM, int BN, int BK, int WGM, int WGN, int ST, int OCC>
constexpr bool stays() {
  if constexpr (ST == kAhead && OCC == 1 && sizeof(TI) == 2 && EPI != EPI_RESID)
    return BM * BK * (int)sizeof(TI) >=
           WGM * WGN * Staging<TO, EPI, BM / WGM / 32, BN / WGN / 32, WGM * WGN, 1 << 20>::STRIP;
  return false;
}

template <typename TI, typename TO, typename TR, int EPI, int BM, int BN, int BK, int WGM, int WGN, int ST,
          int OCC>
__global__ __launch_bounds__(ST >= kTileRegs ? kLoaders * 64 : WGM* WGN * 64, OCC) void gemm_dma_kernel(DevParams p) {
  typedef Mfma<TI> MF;
  typedef typename MF::frag frag;
  constexpr int NC = WGM * WGN;  // waves that multiply; NW: that load
  constexpr int NW = ST >= kTileRegs ? kLoaders : NC;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int EPC = 16 / (int)sizeof(TI);    // elements per 16-byte chunk
  constexpr int CPR = BK / EPC;                // chunks per row
  constexpr int ROWB = BK * (int)sizeof(TI);   // bytes per row
  constexpr int RPI = 64 / CPR;                // rows per wave load instruction
  constexpr int A_INS = BM / RPI / NW, B_INS = BN / RPI / NW;
  constexpr int LPT = A_INS + B_INS;           // load instructions per wave per K tile
  constexpr int A_BYTES = BM * ROWB, STAGE = (BM + BN) * ROWB;
  constexpr int NKS = BK / MF::KI;             // MFMA k-steps per K tile
  constexpr int NCH = MF::KPL * (int)sizeof(TI) / 16;  // chunks per lane fragment
  constexpr int CPS = MF::KI / EPC;            // chunks per k-step
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile/waves mismatch");
  static_assert(TM >= 1 && TN >= 1 && BK % MF::KI == 0 && (ST >= 2 || ST == kAhead), "bad tile");
  constexpr bool AHEAD = ST == kAhead, WHOLE = ST >= kTileRegs;
  constexpr int SL = WHOLE ? ST - kTileRegs : ST;  // stages
  static_assert(AHEAD || (SL - 1) * LPT < 64, "vmcnt range");
  constexpr bool PERSIST = stays<TI, TO, EPI, BM, BN, BK, WGM, WGN, ST, OCC>();
  constexpr int SMEM = AHEAD ? 3 * A_BYTES + 2 * (STAGE - A_BYTES) : SL * STAGE;
  static_assert(SMEM <= 160 * 1024, "LDS ring exceeds the CU's 160 KB");
  __shared__ __align__(1024) char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int N = p.N, K = p.K;
  // the tiles of the rows to compute; with a device row count the grid may
  // hold more workgroups, which leave at once, and the live tiles are spread
  // over the XCDs as in a launch of exactly their number
  const int M = live_rows(p.M, p.m_dev);
  const int ntn = N / BN;
  const int ntm = (M + BM - 1) / BM;
  if ((int)blockIdx.x >= ntm * ntn) return;
  // this lane's source of each load instruction, as a byte offset from the
  // tile's first row at k = 0 (uniform bases stay in scalar registers; rows
  // past M, in the last row block only, re-read row M-1: never stored, no
  // branch)
  int m0, n0;
  const char *abase, *bbase;
  uint32_t ga[A_INS], gb[B_INS];
  auto go_to = [&](int tile) {
    int mb, nb;
    group_tile(xcd_remap(tile, ntm * ntn), ntm, ntn, p.group_m, mb, nb);
    m0 = mb * BM, n0 = nb * BN;
    abase = (const char*)p.A + (size_t)m0 * K * sizeof(TI);
    bbase = (const char*)p.W + (size_t)n0 * K * sizeof(TI);
    const int rl = lane / CPR, slot = lane % CPR;
#pragma unroll
    for (int i = 0; i < A_INS; ++i) {
      const int r = (wave * A_INS + i) * RPI + rl;
      ga[i] = (uint32_t)((min(m0 + r, M - 1) - m0) * K + (slot ^ lds_swz<CPR>(r)) * EPC) * (uint32_t)sizeof(TI);
    }
#pragma unroll
    for (int i = 0; i < B_INS; ++i) {
      const int r = (wave * B_INS + i) * RPI + rl;
      gb[i] = (uint32_t)(r * K + (slot ^ lds_swz<CPR>(r)) * EPC) * (uint32_t)sizeof(TI);
    }
  };
  go_to(blockIdx.x);
  auto issue = [&](int kt, int stage) {
    char* sa = smem + stage * STAGE + wave * A_INS * 1024;
    char* sb = smem + stage * STAGE + A_BYTES + wave * B_INS * 1024;
    const char* ak = abase + (size_t)kt * BK * sizeof(TI);
    const char* bk = bbase + (size_t)kt * BK * sizeof(TI);
#pragma unroll
    for (int i = 0; i < A_INS; ++i) dma16(ak + ga[i], sa + i * 1024);
#pragma unroll
    for (int i = 0; i < B_INS; ++i) dma16(bk + gb[i], sb + i * 1024);
  };

  // fragment addresses: row (lane & 31) of each 32-row sub-tile; the swizzle
  // is the same for rows 32 apart, so one slot offset per (k-step, chunk)
  const int ra = wm * WTM + (lane & 31), rb = wn * WTN + (lane & 31);
  int aoff[NKS][NCH], boff[NKS][NCH];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int kc = ks * CPS + (lane >> 5) * NCH + q;
      aoff[ks][q] = ra * ROWB + (kc ^ lds_swz<CPR>(ra)) * 16;
      boff[ks][q] = A_BYTES + rb * ROWB + (kc ^ lds_swz<CPR>(rb)) * 16;
    }
  auto rdfrag = [&](const char* base, const int (&off)[NCH], int sub) {
    frag f;
    if constexpr (NCH == 1) {
      f = *(const frag*)(base + off[0] + sub * 32 * ROWB);
    } else {
      const intx4 lo = *(const intx4*)(base + off[0] + sub * 32 * ROWB);
      const intx4 hi = *(const intx4*)(base + off[1] + sub * 32 * ROWB);
      f = frag{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
    return f;
  };

  floatx16 acc[TM][TN];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  clear();

  const int KT = K / BK;
  // The ring holds up to ST tiles in flight or resident.
  if constexpr (!AHEAD && !WHOLE) {
#pragma unroll
    for (int s = 0; s < ST; ++s)
      if (s < KT) issue(s, s);
    wait_tiles<ST - 1, LPT>(KT - 1);
    __builtin_amdgcn_s_barrier();
  }

  if constexpr (AHEAD) {
    // B tiles run one tile ahead in two slots, A tiles two ahead in three:
    // during tile kt's last k-step its two slots are free and take B of tile
    // kt+2 and A of tile kt+3.
    static_assert(NKS % 2 == 0, "the fragment buffers of a k-step are the same in every tile");
    constexpr int B0 = 3 * A_BYTES, B_BYTES = BN * ROWB;
    const char *ua, *ub;
    auto issue_a = [&](int kt, int slot) {
#pragma unroll
      for (int i = 0; i < A_INS; ++i)
        buf16(ua, ga[i], kt * BK * (int)sizeof(TI), smem + slot * A_BYTES + (wave * A_INS + i) * 1024);
    };
    auto issue_b = [&](int kt, int slot) {
#pragma unroll
      for (int i = 0; i < B_INS; ++i)
        buf16(ub, gb[i], kt * BK * (int)sizeof(TI), smem + B0 + slot * B_BYTES + (wave * B_INS + i) * 1024);
    };
    auto start = [&] {  // all of a tile's first copies but those into A's third slot
      ua = uniform_ptr(abase);
      ub = uniform_ptr(bbase);
      issue_b(0, 0);
      issue_a(0, 0);
      if (KT > 1) {
        issue_b(1, 1);
        issue_a(1, 1);
      }
    };
    start();
    int tile = blockIdx.x;
    for (;;) {
      if (KT > 2) {
        issue_a(2, 2);
        wait_vmcnt<2 * A_INS + B_INS>();
      } else if (KT > 1) {
        wait_vmcnt<A_INS + B_INS>();
      } else {
        wait_vmcnt<0>();
      }
      __builtin_amdgcn_s_barrier();
      frag fa[2][TM], fb[2][TN];
      auto read_a = [&](int set, int slot, int ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[set][i] = rdfrag(smem + slot * A_BYTES, aoff[ks], i);
      };
      auto read_b = [&](int set, int slot, int ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[set][j] = rdfrag(smem + B0 - A_BYTES + slot * B_BYTES, boff[ks], j);
      };
      read_a(0, 0, 0);
      read_b(0, 0, 0);
      int sa = 0, sb = 0;  // this tile's slots
      // one tile with LEFT tiles after it (3: three or more)
      auto body = [&](int kt, auto leftc) {
        constexpr int LEFT = decltype(leftc)::value;
        constexpr int NRD = (TM + TN) * NCH;
        const int na = sa == 2 ? 0 : sa + 1;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const int cur = ks & 1;
          if (ks + 1 < NKS) {
            read_a(cur ^ 1, sa, ks + 1 < NKS ? ks + 1 : 0);
            read_b(cur ^ 1, sb, ks + 1 < NKS ? ks + 1 : 0);
          } else if constexpr (LEFT > 0) {
            // this wave's reads of the tile have returned and tile kt+1 has
            // landed (of the later issues only A of kt+2 may be in flight);
            // after the barrier both hold for every wave
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) (vmcnt, expcnt at maxima)
            wait_vmcnt<(LEFT > 1 ? A_INS : 0)>();
            __builtin_amdgcn_s_barrier();
            read_a(cur ^ 1, na, 0);
            read_b(cur ^ 1, sb ^ 1, 0);
            if constexpr (LEFT > 1) issue_b(kt + 2, sb);
            if constexpr (LEFT > 2) issue_a(kt + 3, sa);
          }
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(fb[cur][j], fa[cur][i], acc[i][j]);
          if (ks + 1 < NKS) sched_step<TM * TN, NRD, 0>();
          else sched_step<TM * TN, (LEFT > 0 ? NRD : 0), (LEFT > 2 ? LPT : LEFT > 1 ? B_INS : 0)>();
        }
        sa = na;
        sb ^= 1;
      };
      int kt = 0;
      for (; kt + 3 < KT; ++kt) body(kt, std::integral_constant<int, 3>());
      if (kt + 2 < KT) body(kt++, std::integral_constant<int, 2>());
      if (kt + 1 < KT) body(kt++, std::integral_constant<int, 1>());
      if constexpr (PERSIST) {
        const int row0 = m0 + wm * WTM, col0 = n0 + wn * WTN;
        floatx4 bias[TN][4];
        load_bias(p, lane, col0, bias);  // (there before the copies below, which it would wait for)
        body(kt, std::integral_constant<int, 0>());
        wait_vmcnt<0>();
        __syncthreads();  // every wave has read the ring to its end
        tile += gridDim.x;
        const bool more = tile < ntm * ntn;
        if (more) {
          go_to(tile);
          start();
        }
        epilogue<TO, TR, EPI, TM, TN, NW, A_BYTES>(p, acc, smem + 2 * A_BYTES, wave, lane, M, row0, col0, bias);
        if (!more) return;
        clear();
      } else {
        body(kt, std::integral_constant<int, 0>());
        break;
      }
    }
  } else if constexpr (WHOLE) {
    const char* const ua = uniform_ptr(abase);
    const char* const ub = uniform_ptr(bbase);
    auto refill = [&](int kt, int slot) {
      char* l = smem + slot * STAGE;
#pragma unroll
      for (int i = 0; i < A_INS; ++i)
        buf16(ua, ga[i], kt * BK * (int)sizeof(TI), l + (wave * A_INS + i) * 1024);
#pragma unroll
      for (int i = 0; i < B_INS; ++i)
        buf16(ub, gb[i], kt * BK * (int)sizeof(TI), l + A_BYTES + (wave * B_INS + i) * 1024);
    };
    frag fa[2][NKS][TM], fb[2][NKS][TN];
    const bool computes = wave < NC;
    auto read = [&](auto set, int slot) {
      if (!computes) return;
      const char* base = smem + slot * STAGE;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[decltype(set)::value][ks][i] = rdfrag(base, aoff[ks], i);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[decltype(set)::value][ks][j] = rdfrag(base, boff[ks], j);
      }
    };
#pragma unroll
    for (int s = 0; s < SL - 1; ++s)
      if (s < KT) refill(s, s);
    wait_tiles<SL - 2, LPT>(KT - 1);
    __builtin_amdgcn_s_barrier();
    read(std::integral_constant<int, 0>(), 0);
    int slot = 0;
    // tile kt, its fragments in set P or on their way there
    auto body = [&](int kt, auto set) {
      constexpr int P = decltype(set)::value;
      const int next = slot + 1 == SL ? 0 : slot + 1;
      // this wave has used tile kt-1 and its part of tile kt+1 has landed;
      // after the barrier that is so for every wave: tile kt-1's slot is free
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 1 < KT) {
        wait_tiles<SL - 3, LPT>(KT - 2 - kt);
        __builtin_amdgcn_s_barrier();
        if (kt + SL - 1 < KT) refill(kt + SL - 1, slot == 0 ? SL - 1 : slot - 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (computes) {
        // (past the last tile the reads find an older one and are not used)
        read(std::integral_constant<int, P ^ 1>(), next);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(fb[P][ks][j], fa[P][ks][i], acc[i][j]);
        sched_step<NKS * TM * TN, NKS * (TM + TN) * NCH, 0>();
      }
      slot = next;
    };
    for (int kt = 0; kt < KT; kt += 2) {
      body(kt, std::integral_constant<int, 0>());
      if (kt + 1 < KT) body(kt + 1, std::integral_constant<int, 1>());
    }
  } else {
  // Fragments are double-buffered across k-steps, also across tiles: the
  // buffer of a k-step is the parity of its global k-step index, a
  // compile-time value once the tile loop is unrolled by two.
  frag fa[2][TM], fb[2][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[0][i] = rdfrag(smem, aoff[0], i);
#pragma unroll
  for (int j = 0; j < TN; ++j) fb[0][j] = rdfrag(smem, boff[0], j);
  int stage = 0;
  // One K tile.  During its last k-step the next tile is made ready: wait for
  // it, barrier (every wave has then also finished reading this tile, whose
  // slot takes tile kt+ST), and read its first fragments while this tile's
  // last MFMAs run.
  auto tile_body = [&](int kt, auto tpar) {
    constexpr int TP = decltype(tpar)::value;
    const char* base = smem + stage * STAGE;
    const int nstage = stage + 1 == ST ? 0 : stage + 1;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int cur = (TP * NKS + ks) & 1;
      if (ks + 1 < NKS) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[cur ^ 1][i] = rdfrag(base, aoff[ks + 1 < NKS ? ks + 1 : 0], i);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[cur ^ 1][j] = rdfrag(base, boff[ks + 1 < NKS ? ks + 1 : 0], j);
      } else {
        // this wave's reads of the tile have returned before anyone may
        // overwrite it; tile kt+1 has landed for this wave.  (No instruction
        // crosses this point: the previous k-step's MFMAs stay ahead of the
        // wait, covering the latency of the reads it waits for.)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) (vmcnt, expcnt at maxima)
        wait_tiles<ST - 2, LPT>(KT - 2 - kt);
        __builtin_amdgcn_s_barrier();
        if (kt + ST < KT) issue(kt + ST, stage);
        const char* nbase = smem + nstage * STAGE;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[cur ^ 1][i] = rdfrag(nbase, aoff[0], i);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[cur ^ 1][j] = rdfrag(nbase, boff[0], j);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(fb[cur][j], fa[cur][i], acc[i][j]);
      // (with two workgroups per CU the hardware interleaves them better)
      if constexpr (OCC == 1) {
        if (ks + 1 < NKS) sched_step<TM * TN, (TM + TN) * NCH, 0>();
        else sched_step<TM * TN, (TM + TN) * NCH, LPT>();
      }
    }
    stage = nstage;
  };
  for (int kt = 0; kt < KT; kt += 2) {
    tile_body(kt, std::integral_constant<int, 0>());
    if (kt + 1 < KT) tile_body(kt + 1, std::integral_constant<int, 1>());
  }
  }
  // no refill is in flight (the last tiles issue none); every wave must have
  // finished reading the ring before the staging below reuses it
  __syncthreads();
  if (wave >= NC) return;
  floatx4 bias[TN][4];
  load_bias(p, lane, n0 + wn * WTN, bias);
  epilogue<TO, TR, EPI, TM, TN, NC, SMEM>(p, acc, smem, wave, lane, M, m0 + wm * WTM, n0 + wn * WTN, bias);
}

struct Cfg {
  int bm, bn, bk, wgm, wgn, st, occ;
  const char* name;
};

// Whether a tile serves an epilogue: the paired epilogues need an even
// number of 32-column sub-blocks per wave, and one 32-row output strip per
// wave must fit the kernel's LDS (mirrors Staging).
constexpr bool staging_fits(int bm, int bn, int bk, int wgm, int wgn, int st, int in_bytes, int out_bytes, int epi) {
  const int tn = bn / wgn / 32;
  if ((epi == EPI_ROPE || epi == EPI_GEGLU) && tn % 2 != 0) return false;
  const int smem = st >= kTileRegs ? (st - kTileRegs) * (bm + bn) * bk * in_bytes : st == kAhead ? (3 * bm + 2 * bn) * bk * in_bytes : st == 0 ? 2 * (bm + bn) * (bk + 16 / in_bytes) * in_bytes : st * (bm + bn) * bk * in_bytes;
  const int otn = epi == EPI_GEGLU ? tn / 2 : tn;
  return smem >= wgm * wgn * 32 * otn * 32 * out_bytes;
}

// Tile configurations per input type; index = GemmParams::config.
// Columns: BM, BN, BK, wave grid WGM x WGN, LDS ring stages (0: the
// register-staged kernel), workgroups per CU the registers are sized for.
#define ANON_BF16_CFGS(X)                                      \
  X(0, 256, 256, 64, 4, 2, 0, 2, "bf16_256x256x64_w4x2")       \
  X(1, 256, 128, 32, 4, 2, 0, 2, "bf16_256x128x32_w4x2")       \
  X(2, 128, 256, 32, 2, 4, 0, 2, "bf16_128x256x32_w2x4")       \
  X(3, 256, 256, 32, 4, 2, 3, 1, "bf16_256x256x32_w4x2_s3")    \
  X(4, 256, 128, 64, 4, 2, 3, 1, "bf16_256x128x64_w4x2_s3")    \
  X(5, 128, 256, 64, 2, 4, 3, 1, "bf16_128x256x64_w2x4_s3")    \
  X(6, 256, 128, 32, 4, 2, 3, 2, "bf16_256x128x32_w4x2_s3")    \
  X(7, 128, 256, 32, 2, 4, 3, 2, "bf16_128x256x32_w2x4_s3")    \
  X(8, 256, 256, 64, 4, 2, 2, 1, "bf16_256x256x64_w4x2_s2")    \
  X(9, 256, 256, 32, 4, 2, 4, 1, "bf16_256x256x32_w4x2_s4")    \
  X(10, 256, 128, 32, 4, 2, 4, 1, "bf16_256x128x32_w4x2_s4")    \
  X(11, 256, 256, 64, 2, 4, kAhead, 1, "bf16_256x256x64_w2x4_a") \
  X(12, 192, 256, 64, 2, 4, kAhead, 1, "bf16_192x256x64_w2x4_a") \
  X(13, 128, 256, 64, 2, 4, kAhead, 1, "bf16_128x256x64_w2x4_a") \
  X(14, 128, 128, 64, 2, 2, kAhead, 2, "bf16_128x128x64_w2x2_a") \
  X(15, 64, 128, 64, 2, 2, kAhead, 2, "bf16_64x128x64_w2x2_a")   \
  X(16, 64, 64, 64, 2, 2, kAhead, 4, "bf16_64x64x64_w2x2_a")     \
  X(17, 64, 64, 128, 2, 2, kAhead, 2, "bf16_64x64x128_w2x2_a")   \
  X(18, 32, 64, 128, 1, 2, kAhead, 2, "bf16_32x64x128_w1x2_a")   \
  X(19, 64, 64, 64, 2, 1, kAhead, 2, "bf16_64x64x64_w2x1_a") \
  X(20, 32, 64, 128, 1, 2, kTileRegs + 4, 1, "bf16_32x64x128_w1x2_r4") \
  X(21, 32, 32, 128, 1, 1, kTileRegs + 3, 1, "bf16_32x32x128_w1x1_r3") \
  X(22, 64, 64, 128, 2, 2, kTileRegs + 4, 1, "bf16_64x64x128_w2x2_r4")
#define ANON_F32_CFGS(X)                                 \
  X(0, 128, 128, 32, 2, 2, 0, 2, "f32_128x128x32_w2x2") \
  X(1, 64, 64, 32, 2, 2, 0, 2, "f32_64x64x32_w2x2")     \
  X(2, 128, 128, 16, 2, 2, 0, 2, "f32_128x128x16_w2x2") \
  X(3, 256, 128, 16, 2, 2, 0, 1, "f32_256x128x16_w2x2")
#define ANON_FP8_CFGS(X)                                    \
  X(0, 256, 256, 64, 4, 2, 0, 2, "fp8_256x256x64_w4x2")     \
  X(1, 256, 256, 64, 4, 2, 3, 1, "fp8_256x256x64_w4x2_s3")  \
  X(2, 256, 256, 128, 4, 2, 2, 1, "fp8_256x256x128_w4x2_s2") \
  X(3, 256, 128, 128, 4, 2, 3, 1, "fp8_256x128x128_w4x2_s3") \
  X(4, 256, 128, 64, 4, 2, 3, 2, "fp8_256x128x64_w4x2_s3")  \
  X(5, 128, 256, 64, 2, 4, 3, 2, "fp8_128x256x64_w2x4_s3")  \
  X(6, 256, 256, 64, 4, 2, 4, 1, "fp8_256x256x64_w4x2_s4")  \
  X(7, 256, 256, 128, 2, 4, kAhead, 1, "fp8_256x256x128_w2x4_a") \
  X(8, 128, 256, 128, 2, 4, kAhead, 1, "fp8_128x256x128_w2x4_a") \
  X(9, 128, 128, 128, 2, 2, kAhead, 2, "fp8_128x128x128_w2x2_a") \
  X(10, 64, 128, 128, 2, 2, kAhead, 2, "fp8_64x128x128_w2x2_a")  \
  X(11, 64, 64, 128, 2, 2, kAhead, 4, "fp8_64x64x128_w2x2_a")    \
  X(12, 32, 64, 256, 1, 2, kTileRegs + 4, 1, "fp8_32x64x256_w1x2_r4") \
  X(13, 32, 32, 256, 1, 1, kTileRegs + 3, 1, "fp8_32x32x256_w1x1_r3")

#define ANON_CFG_ROW(i, bm, bn, bk, wgm, wgn, st, occ, name) {bm, bn, bk, wgm, wgn, st, occ, name},
const Cfg kCfgBF16[] = {ANON_BF16_CFGS(ANON_CFG_ROW)};
const Cfg kCfgF32[] = {ANON_F32_CFGS(ANON_CFG_ROW)};
const Cfg kCfgFP8[] = {ANON_FP8_CFGS(ANON_CFG_ROW)};

const Cfg* cfgs(ElemType t, int* n) {
  if (t == ET_BF16) {
    *n = (int)(sizeof(kCfgBF16) / sizeof(Cfg));
    return kCfgBF16;
  }
  if (t == ET_F32) {
    *n = (int)(sizeof(kCfgF32) / sizeof(Cfg));
    return kCfgF32;
  }
  *n = (int)(sizeof(kCfgFP8) / sizeof(Cfg));
  return kCfgFP8;
}

template <typename TI, typename TO, typename TR, int EPI, int BM, int BN, int BK, int WGM, int WGN, int ST, int OCC>
bool run(const GemmParams& g, hipStream_t s) {
  if constexpr (!staging_fits(BM, BN, BK, WGM, WGN, ST, (int)sizeof(TI), (int)sizeof(TO), EPI)) {
    return false;  // no pairs in a wave's columns, or the output strips do not fit the LDS
  } else {
  // tile order: by default, groups of 8 row blocks when a row block spans 8
  // or more column blocks (its weight panels would otherwise cycle through
  // the XCD's L2 once per row block), else plain row-major order
  const int gm = g.group_m > 0 ? g.group_m : (g.N / BN >= 8 ? 8 : 1);
  DevParams p{g.A, g.W, g.bias, g.resid, g.C, g.M, g.N, g.K, g.qscale, g.qcols, g.acc_scale, g.out_inv_scale, gm,
              g.ldc > 0 ? g.ldc : (g.epi == EPI_GEGLU ? g.N / 2 : g.N), g.pos, g.rope, g.rope_cols, g.m_dev};
  const int tiles = ((g.M + BM - 1) / BM) * (g.N / BN);
  constexpr bool PERSIST = stays<TI, TO, EPI, BM, BN, BK, WGM, WGN, ST, OCC>();
  if constexpr (ST == 0) {
    hipLaunchKernelGGL((gemm_kernel<TI, TO, TR, EPI, BM, BN, BK, WGM, WGN, OCC>), dim3(tiles),
                       dim3(WGM * WGN * 64), 0, s, p);
  } else {
    static_assert(sizeof(TI) <= 2, "the LDS ring kernel serves BF16 and FP8 operands");
    hipLaunchKernelGGL((gemm_dma_kernel<TI, TO, TR, EPI, BM, BN, BK, WGM, WGN, ST, OCC>),
                       dim3(PERSIST ? std::min(tiles, 256) : tiles),
                       dim3((ST >= kTileRegs ? kLoaders : WGM * WGN) * 64), 0, s, p);
  }
  return true;
  }
}

#define ANON_CFG_CASE(i, bm, bn, bk, wgm, wgn, st, occ, name) \
  case i:                                                      \
    return run<TI, TO, TR, EPI, bm, bn, bk, wgm, wgn, st, occ>(g, s);

template <typename TI, typename TO, typename TR, int EPI>
bool dispatch_tile(const GemmParams& g, int ci, hipStream_t s) {
  if constexpr (sizeof(TI) == 2) {
    switch (ci) { ANON_BF16_CFGS(ANON_CFG_CASE) }
  } else if constexpr (sizeof(TI) == 4) {
    switch (ci) { ANON_F32_CFGS(ANON_CFG_CASE) }
  } else {
    switch (ci) { ANON_FP8_CFGS(ANON_CFG_CASE) }
  }
  return false;
}

template <typename TI>
bool dispatch_epi(const GemmParams& g, int ci, hipStream_t s) {
  // Supported (epilogue, output, residual) combinations per input type.
  if constexpr (sizeof(TI) == 4) {
    if (g.epi == EPI_BIAS && g.out == ET_F32) return dispatch_tile<TI, float, float, EPI_BIAS>(g, ci, s);
    if (g.epi == EPI_GELU && g.out == ET_F32) return dispatch_tile<TI, float, float, EPI_GELU>(g, ci, s);
    if (g.epi == EPI_RESID && g.res == ET_F32 && g.out == ET_F32)
      return dispatch_tile<TI, float, float, EPI_RESID>(g, ci, s);
    if (g.epi == EPI_ROPE && g.out == ET_F32) return dispatch_tile<TI, float, float, EPI_ROPE>(g, ci, s);
    if (g.epi == EPI_GEGLU && g.out == ET_F32) return dispatch_tile<TI, float, float, EPI_GEGLU>(g, ci, s);
  } else {
    if constexpr (sizeof(TI) == 2) {
      // the ModernBERT-style encoder: rotary QKV, gated MLP, FP32 residual stream
      if (g.epi == EPI_ROPE && g.out == ET_BF16) return dispatch_tile<TI, bf16_t, float, EPI_ROPE>(g, ci, s);
      if (g.epi == EPI_GEGLU && g.out == ET_BF16) return dispatch_tile<TI, bf16_t, float, EPI_GEGLU>(g, ci, s);
      if (g.epi == EPI_RESID && g.res == ET_F32 && g.out == ET_F32)
        return dispatch_tile<TI, float, float, EPI_RESID>(g, ci, s);
    }
    if (g.epi == EPI_BIAS && g.out == ET_BF16) return dispatch_tile<TI, bf16_t, float, EPI_BIAS>(g, ci, s);
    if constexpr (sizeof(TI) == 2) {
      if (g.epi == EPI_GELU && g.out == ET_BF16) return dispatch_tile<TI, bf16_t, float, EPI_GELU>(g, ci, s);
    } else {
      if (g.epi == EPI_GELU && g.out == ET_FP8) return dispatch_tile<TI, fp8_t, float, EPI_GELU>(g, ci, s);
    }
    if (g.epi == EPI_RESID && g.res == ET_BF16 && g.out == ET_BF16)
      return dispatch_tile<TI, bf16_t, bf16_t, EPI_RESID>(g, ci, s);
  }
  return false;
}

}  // namespace

int gemm_num_configs(ElemType in) {
  int n;
  cfgs(in, &n);
  return n;
}

const char* gemm_config_name(ElemType in, int config) {
  int n;
  const Cfg* c = cfgs(in, &n);
  return (config >= 0 && config < n) ? c[config].name : "?";
}

bool gemm_config_fits(ElemType in, int config, int N, int K) {
  int n;
  const Cfg* c = cfgs(in, &n);
  if (config < 0 || config >= n) return false;
  return N % c[config].bn == 0 && K % c[config].bk == 0;
}

static int elem_bytes(ElemType t) { return t == ET_F32 ? 4 : (t == ET_BF16 ? 2 : 1); }

bool gemm_config_launchable(const GemmParams& g, int config) {
  int n;
  const Cfg* c = cfgs(g.in, &n);
  if (config < 0 || config >= n) return false;
  const Cfg& k = c[config];
  const int64_t tiles = ((int64_t)g.M + k.bm - 1) / k.bm * (g.N / k.bn);
  return tiles * (k.st >= kTileRegs ? kLoaders : k.wgm * k.wgn) * 64 <= 0xffffffffll;
}

bool gemm_config_serves(const GemmParams& g, int config) {
  int n;
  const Cfg* c = cfgs(g.in, &n);
  if (!gemm_config_fits(g.in, config, g.N, g.K)) return false;
  const Cfg& k = c[config];
  return staging_fits(k.bm, k.bn, k.bk, k.wgm, k.wgn, k.st, elem_bytes(g.in), elem_bytes(g.out), g.epi);
}

// Estimated time (us) of the tiles worth choosing, fitted to launches of the
// base and large encoders' GEMMs at 16 to 50,000 rows on all 256 CUs (bf16 K
// 768 and 3072, FP8 K 1024 and 4096, FP32 K 768 and 3072).  With kt = 128-byte steps of K:
//   f0 + f1 kt  a launch whose tiles all start at once (latency of one tile)
//   g0 + g1 kt  each further tile per CU, all CUs busy
//   gelu        added to both by the GELU epilogue
// Whole: tiles of one workgroup per CU, so a last, partly filled round costs
// between the first and the second figure.  Pair: at most two per CU, whose
// second tile costs a round as soon as one CU has it.  Fine: tiles so small
// that the CUs' loads even out.  Step: each further tile on any CU costs a
// round.  Both: two tiles of a CU share its matrix cores to the end, so a
// third starts with the fourth.
enum TileFill { kWhole, kPair, kFine, kStep, kBoth };
struct TileCost {
  int config;
  float f0, f1, g0, g1, gelu;
  TileFill fill;
};
const TileCost kCostBF16[] = {
    {11, 5.1f, 1.06f, 5.3f, 1.6f, 5.0f, kWhole},   {12, 3.8f, 0.9f, 4.0f, 1.35f, 3.8f, kWhole},
    {13, 1.4f, 0.825f, 2.7f, 1.03f, 3.0f, kWhole}, {14, 2.7f, 0.506f, 0.7f, 0.53f, 1.0f, kPair},
    {15, 0.6f, 0.508f, 1.27f, 0.303f, 0.6f, kPair}, {16, 0.5f, 0.406f, 0.3f, 0.19f, 0.4f, kFine},
    {17, 2.5f, 0.261f, 0.65f, 0.2f, 0.4f, kFine},  {18, 2.9f, 0.2f, 0.96f, 0.134f, 0.4f, kFine},
    {19, 0.5f, 0.46f, 0.3f, 0.25f, 0.4f, kFine},   {20, 3.27f, 0.128f, 1.8f, 0.15f, 0.3f, kStep},
    {21, 3.25f, 0.114f, 0.74f, 0.13f, 0.3f, kStep}, {22, 3.45f, 0.14f, 0.2f, 0.3f, 0.3f, kStep},
};
const TileCost kCostFP8[] = {
    {7, 6.3f, 1.02f, 8.0f, 1.25f, 9.0f, kWhole},   {8, 2.0f, 0.875f, 3.2f, 0.9f, 3.5f, kWhole},
    {9, 3.1f, 0.53f, 0.7f, 0.54f, 1.1f, kPair},    {10, 3.7f, 0.25f, 0.7f, 0.34f, 0.5f, kFine},
    {11, 3.1f, 0.19f, 0.34f, 0.2f, 0.3f, kFine},   {12, 3.25f, 0.14f, 1.5f, 0.167f, 0.3f, kStep},
    {13, 3.23f, 0.121f, 0.93f, 0.121f, 0.3f, kStep},
};

const TileCost kCostF32[] = {
    {0, 5.0f, 2.13f, 3.7f, 1.91f, 0.5f, kBoth},
    {1, 3.5f, 0.73f, 0.53f, 0.578f, 0.3f, kStep},
    {2, 5.0f, 2.29f, 6.0f, 1.83f, 0.5f, kStep},
};

static float tile_cost(const TileCost& t, const Cfg& c, const GemmParams& g, int rows) {
  const float kt = (float)g.K * elem_bytes(g.in) / 128.f;
  const float ge = g.epi == EPI_GELU || g.epi == EPI_GEGLU ? t.gelu : 0.f;
  const float one = t.f0 + t.f1 * kt + ge, more = t.g0 + t.g1 * kt + ge;
  const float r = (float)(((int64_t)rows + c.bm - 1) / c.bm * (g.N / c.bn)) / 256.f;  // tiles per CU
  if (t.fill == kWhole) {
    const float full = floorf(r);
    return full * more + (r > full ? one + (more - one) * (r - full) : 0.f);
  }
  if (r <= 1.f) return one;
  if (t.fill == kFine) return one + (r - 1.f) * more;
  if (t.fill == kStep) return one + (ceilf(r) - 1.f) * more;
  if (t.fill == kBoth) return ceilf(r / 2.f) * 2.f * more;
  return one + (r < 2.f ? 1.f : ceilf(2.f * r) * 0.5f - 1.f) * more;
}

int default_gemm_config(const GemmParams& g) {
  // The cheapest tile for this many rows by the estimate above, else the
  // first configuration that serves the shape and epilogue.  One tile shape
  // for every size leaves most CUs idle on a small batch: with 256x256 tiles
  // alone, a record of 137 tokens runs its four GEMMs of a layer on 3 to 12
  // workgroups (20, 20, 25 and 61 us on the base shapes); the tiles chosen
  // here take 4.8, 4.6, 5.3 and 8.7 us, and at 2,094 rows 13, 7, 17 and 22
  // instead of 21, 21, 27 and 63.  At 8,192 rows and above the choice is
  // worth 0-25% (the last round of 256x256 tiles), from 21,608 rows on it is
  // mostly the 256x256 tile.  FP32: 137 rows 56, 56, 57 and 210 us with
  // 128x128 tiles alone, 21, 21, 22 and 74 with 64x64; 4,096 rows 192, 58, 197
  // and 209 -> 135, 47, 154 and 175; 21,608 rows keep 128x128.
  const int n = gemm_num_configs(g.in);
  int nc;
  const Cfg* cs = cfgs(g.in, &nc);
  int best = -1;
  float best_t = 0.f;
  auto consider = [&](const TileCost& t) {
    if (!gemm_config_serves(g, t.config) || !gemm_config_launchable(g, t.config)) return;
    // M is what a captured launch may hold, its row count on the device what
    // a replay brings: then the mean over the quarters of M counts.  8,192
    // rows at most, FFN2 of the base encoder with 4,096 / 8,192 brought:
    // 128x256 tiles (best when full) 41 / 42.5 us, 128x128 27 / 44.4.  The
    // server's buckets halve and the smallest that holds a batch is replayed,
    // so all but its smallest are half full at least; with the mean over
    // 50-100% instead, a replay of four base layers took, at 51 / 75 / 100%
    //   2,048 rows at most   278 / 327 / 355 us   (here 272 / 348 / 370)
    //   4,096                396 / 454 / 499      (360 / 462 / 512)
    //   8,192                534 / 674 / 796      (522 / 679 / 806)
    // and 512, 1,024 and 16,384 the same: no gain, and 5-20% lost below half.
    float us = 0.f;
    for (int q = g.m_dev ? 1 : 4; q <= 4; ++q) us += tile_cost(t, cs[t.config], g, (int)((int64_t)g.M * q / 4));
    if (best < 0 || us < best_t) best = t.config, best_t = us;
  };
  if (g.in == ET_BF16)
    for (const TileCost& t : kCostBF16) consider(t);
  else if (g.in == ET_FP8)
    for (const TileCost& t : kCostFP8) consider(t);
  else
    for (const TileCost& t : kCostF32) consider(t);
  if (best >= 0) return best;
  for (int c = 0; c < n; ++c)
    if (gemm_config_serves(g, c) && gemm_config_launchable(g, c)) return c;
  return -1;
}

bool launch_gemm(const GemmParams& g, hipStream_t s) {
  int ci = g.config;
  // (a tile kept for fewer rows: a launch holds less than 2^32 threads)
  if (ci < 0 || (gemm_config_serves(g, ci) && !gemm_config_launchable(g, ci))) ci = default_gemm_config(g);
  if (ci < 0 || !gemm_config_serves(g, ci)) {
    set_error(ANON_EINVAL, "gemm: no tile configuration divides N=" + std::to_string(g.N) + " K=" +
                               std::to_string(g.K));
    return false;
  }
  if ((g.epi == EPI_BIAS || g.epi == EPI_ROPE) && (g.qcols % 64 != 0 || g.rope_cols % 64 != 0)) {
    set_error(ANON_EINVAL, "gemm: scaled and rotated columns must be whole 64-column blocks");
    return false;
  }
  if (g.M <= 0) return true;
  bool ok = false;
  if (g.in == ET_F32) ok = dispatch_epi<float>(g, ci, s);
  else if (g.in == ET_BF16) ok = dispatch_epi<bf16_t>(g, ci, s);
  else ok = dispatch_epi<fp8_t>(g, ci, s);
  if (!ok) set_error(ANON_EINVAL, "gemm: unsupported type/epilogue combination");
  return ok;
}

}  // namespace anon
