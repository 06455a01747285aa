// What the two families of stage-1 kernels on the matrix cores share: operand types, the kernels' parameters, the
// partial record, and the seeds' own keys and values.
#pragma once

#include <math.h>

#include "common.hpp"

namespace vista {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short i16x4;

constexpr int kTile = kTileItems;    // items per tile
// A record: [four O registers][lane][4], then [lane][l, m]: five stores of 8 or 16 bytes a lane and block, and two loads a
// record in a wave of the merge, which is bound by the latency of the longest user's records.  (A register a row, 18 stores and
// six loads of 4 bytes, and the maximum moved record by record, measured together: one user of 7001 items 21.1 -> 20.7 us a call, jagged
// batch of 768 597 items 171.4 -> 170.0, 8 users of a million items 1586 -> 1580, SiLU, S = 128, 500 003 items 102.1 -> 101.2, d = 64,
// S = 100, 300 007 items 67.0 -> 66.4.  The merge alone is slower by it where every compute unit reads: 32 768 blocks over 14 M items of
// d = 256 116 -> 122 us, eight long users 12.1 -> 12.7; 5.8 -> 5.4, 12.3 -> 11.8 and 12.3 -> 11.6 in the first, second and fourth call.)
constexpr int kRecFloats = 18 * 64;
constexpr int kRecSums = 16 * 64;    // where l and m are

struct MfmaSummarizeParams {
  const uint16_t* X;
  const int64_t* offsets;
  const uint16_t* Q;
  int64_t q_user_stride;
  const uint16_t* Wk;
  const uint16_t* Wv;
  float* partials;
  int B, S, H;
  int nqb;        // query blocks = ceil(S / 32)
  int wph;        // waves per head (the workgroup has HPW wph of them)
  int64_t N;
  int seg;
  int nhg;        // head groups = H / HPW
  float c;        // scale * log2(e)
  float* Ks;      // self term: K', V' of the seeds, formed beside the history, or null
  float* Vs;
  int64_t self_rows;
};

union Pack8 {
  bf16x8 v;
  uint4 u;
  uint16_t h[8];
  uint32_t w[4];
};

__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 r = __builtin_convertvector(f, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// acc + 0: NaN if either number of the pair is infinite or NaN
__device__ __forceinline__ float dot2_zero(uint32_t pk, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), bf16x2{}, acc, false);
}

__device__ __forceinline__ float dot2_self(uint32_t pk, float acc) {
  const bf16x2 v = __builtin_bit_cast(bf16x2, pk);
  return __builtin_amdgcn_fdot2_f32_bf16(v, v, acc, false);
}

// An instruction whose result is pinned comes before whatever is pinned later in the program.
template <typename T>
__device__ __forceinline__ void pin(T& v) { asm volatile("" : "+v"(v)); }

// LDS-only workgroup barrier: global loads in flight (the X prefetch) stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Register i of a lane in half hf holds row 4 hf + acc_row0(i) of the 32x32 accumulator.
__device__ __forceinline__ constexpr int acc_row0(int i) { return 8 * (i / 4) + (i % 4); }

template <int V>
struct Int { static constexpr int value = V; };

constexpr int kXBuf = 3;             // ring depth of the X tiles in LDS (and of the projected tiles in the plain kernels)

// Self term: K' = Q W_k and V' = Q W_v of the seeds in fp32 (bf16 inputs, products exact, fp32 sums).
// A unit is 32 seeds x 32 channels of both, formed by one wave: the seeds' rows read once as the A operand, the
// weights 16 bytes a lane and turned by the matrix core as in the main kernel.
__device__ __forceinline__ void self_kv_unit(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Wk,
                                             const uint16_t* __restrict__ Wv, float* __restrict__ Ks,
                                             float* __restrict__ Vs, int64_t rows, int d, int64_t unit) {
  const int nc = d / 32;
  const int64_t r0 = unit / nc * 32;
  const int c0 = int(unit % nc) * 32;
  if (r0 >= rows) return;
  const int lane = threadIdx.x & 63, hf = lane >> 5, l32 = lane & 31;
  const int64_t qrow = r0 + l32 < rows ? r0 + l32 : rows - 1;   // rows past the end repeat the last; not stored
  const uint16_t* q = Q + qrow * d + 8 * hf;
  const int wrow = (l32 & 16) | ((l32 & 4) << 1) | ((l32 & 8) >> 1) | (l32 & 3);
  const uint16_t* src[2] = {Wk + wrow * d + c0 + 8 * hf, Wv + wrow * d + c0 + 8 * hf};
  Pack8 sel[2];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int j = 0; j < 8; ++j) sel[e].h[j] = (l32 == 16 * e + 8 * hf + j) ? 0x3F80 : 0;
  f32x16 acc[2] = {{0}, {0}};
#pragma unroll 2
  for (int k = 0; k < d; k += 32) {
    float rest = 0.f;
    Pack8 x[2], raw[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      x[e].u = *reinterpret_cast<const uint4*>(q + k + 16 * e);
#pragma unroll
      for (int m = 0; m < 2; ++m) raw[m][e].u = *reinterpret_cast<const uint4*>(src[m] + k * d + 16 * e);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      f32x16 t = {0};
      t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(raw[m][0].v, sel[0].v, t, 0, 0, 0);
      t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(raw[m][1].v, sel[1].v, t, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 8; ++e) rest = dot2_zero(raw[m][e / 4].w[e % 4], rest);
      const bool finite = __builtin_amdgcn_ballot_w64(rest != 0.f) == 0;     // (else not turned: see summarize_wave)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        Pack8 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w.w[j] = cvt_pk_bf16(t[8 * e + 2 * j], t[8 * e + 2 * j + 1]);
        if (!finite) {
          const uint16_t* W = (m ? Wv : Wk) + int64_t(k + 16 * e + 8 * hf) * d + c0 + l32;
#pragma unroll
          for (int j = 0; j < 8; ++j) w.h[j] = W[j * d];
        }
        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[e].v, w.v, acc[m], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t r = r0 + acc_row0(i) + 4 * hf;
    if (r < rows) {
      Ks[r * d + c0 + l32] = acc[0][i];
      Vs[r * d + c0 + l32] = acc[1][i];
    }
  }
}

// The kernels of the shapes whose operands are kept whole (split_mfma.hip); one_head: a head a workgroup (d = 64, 128, S <= 256).
hipError_t launch_split(MfmaSummarizeParams& p, int d, bool one_head, int64_t G, hipStream_t s);

}  // namespace vista
