// Stage 1 on the matrix cores with operands kept whole, gfx950: the bf16 softmax shapes outside the fixed seed counts.
//
// The stream, the waves' roles and the partial records are those of summarize_mfma.hip: a workgroup walks a segment of the
// history for HPW heads, a head has a K wave, a V wave and, for many seeds, waves that only attend; an X tile of 32
// items goes from HBM straight into LDS, is projected two tiles ahead, and every wave attends over it for its own
// query blocks, items on the matrix rows and queries on the columns.
//
// The fixed seed counts keep K, V and the softmax weights as bf16 operands.  Any other seed
// count (and d = 64) keeps them whole, as one thread per query on the vector unit did before: each is
// two fp16 terms, 22 bits and a sign.  Scores take two products (the seeds are bf16, one fp16 term), P V
// three, the scale is applied to the fp32 keys.  fp16 has these bits from 2^-3 to 2^16 only, so everything is brought there by powers of two, which
// change no bit: queries and keys by a unit of the seeds (users' own: of each user's), values by their column of W_v and by the first tile of a user's piece, weights by
// a whole-number reference of each row's own, which is one more product (ones times -m).  That is 19 binary places, and a row may need
// others: its items of large weight may have no value, its own values may be small beside its neighbours'.  So what the terms leave of a row at most
// is held against what the row came to when a piece ends, and a piece with a row that is not known to 2^-19 by that, with keys, values or queries outside fp16,
// infinite or NaN, is formed again in fp32 (pieces_in_fp32), by the wave that found it.
// us a call, 48 users, 300 007 items, d = 64, S = 100, three bf16 terms / two fp16 terms: unit scale 66.2 / 56.1, items 0.7 of whose variance is common to a user
// 66.1 / 56.1, seeds 3 times as large 76.8 / 59.2, items 300 times, seeds 1 / 300 66.1 / 55.9; 1 200 028 items 199 / 150, d = 256 1102 / 845, d = 256, S = 500
// 2706 / 2066.  Users of some 80 to 180 items at d = 256, S = 100 to 200 are 4 to 8 % slower, 101 / 109 and 87 / 91: the check, and every other tile a ragged one.  A reference that all rows
// share (2^-4, scores up to 19.75 and every row's best on the first tile not below 0, else tile by tile with a look for the maximum) was 53.2 at unit scale, 65.4 and
// 67.9 in the second and third call, and gave rows wrong by 33 % where an item without a value scored 19 above the others.
// Error of the result before its bf16 rounding against fp64 (2-norm; d = 64 to 256, one user
// of 700 and of 3001 items, scores up to 6 / 25 / 100): 3.0-3.7 and 5.2-5.7 / 3.8-5.2 and 5.6-7.3 / 5.3-8.9 and 7.2-9.8 e-7; three bf16
// terms 3.7-4.3 and 6.3-7.6 / 5.8-8.1 and 9.7-14 / 8.0-14 and 12-16 e-7.  (Two bf16 terms, 16 bits, were ten times that.)
// What such a wave spends its time on is vector issue: a product keeps the matrix pipe for 32 clocks, in which some
// six plain vector instructions or three exponentials go beside it, so a tile stands in an order that pairs them.
#include "stage1_mfma.hpp"

namespace vista {

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

namespace {

constexpr float kHalfMost2 = 4.29e9f;            // 65 500^2: squared sums below keep every term finite in fp16
constexpr float kQueryMost2 = 4096.f;            // (2^6)^2, of a query in its unit, beyond which it is taken in fp32: a key's last bit, 2^-25, times it stays below 2^-19
constexpr float kKeyMost2 = 8100.f;              // 90^2: a query's numbers below 2^-17 lose up to 2^-25 each, which meets keys of at most this
// Weights are 2^(s - m), m a whole number of each row's own that puts its best weight to 2^12..2^13 when it is taken and is raised when a weight
// would pass 2^kTopWeight (fp16 ends at 2^16).  A plain tile has scores within +-kPlainScore (by |q| |k|), so that m - s is within fp32's exponents.
constexpr float kTopWeight = 15.75f;
constexpr float kBestWeight = 12.f;
constexpr float kFirstReference = -8.f, kFirstBest = 8.f;      // a piece begins with this one, which stays where the first tile's best weight is 2^8 to 2^kTopWeight
constexpr float kPlainScore = 54.f;
// What fp16 terms leave of a weight is at most 2^-25 (weights from 2^-3 up have 22 bits and a sign).  So over a piece of n items a row's sum is
// wrong by at most 2^-25 sum |v| <= 2^-25 (n sum |v|^2)^1/2, and a row that is not 2^19 times that is not known well enough: (2^-6)^2.
// Of a value at most 2^-25 is left too, which matters where a row's own values are small beside the others of their columns: its mean has to be
// 2^-2.5, which is 2^20 times sqrt(32) of these, or a quarter of what n values of the mean size (2^-0.5 at least; 2^7.5 is usual) come to where
// they point anywhere, as what is left of them does: (2^-2.5)^2, (2^-0.5)^2, (2^-2)^2.
constexpr float kWeightsLost2 = 2.4414062e-4f, kValuesLost2 = 0.03125f, kValueMean2 = 0.5f, kMeanLost2 = 0.0625f;

// One 32-wide operand of a tile: the two k-halves of its two fp16 terms, 22 bits and a sign.
struct Operand {
  Pack8 hi[2];
  Pack8 lo[2];
};

__device__ __forceinline__ uint32_t cvt_pk_f16(float a, float b) {
  f32x2 f = {a, b};
  f16x2 r = __builtin_convertvector(f, f16x2);
  return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ float f16_lo(uint32_t w) { return float(__builtin_bit_cast(f16x2, w)[0]); }
__device__ __forceinline__ float f16_hi(uint32_t w) { return float(__builtin_bit_cast(f16x2, w)[1]); }

// fp32 pair (a, b) as two fp16 pairs, both rounded to nearest: what is left is 2^-24 of the value, or 2^-25 where that is more.
// (v_fma_mix_f32 takes an fp16 operand and fp32 ones at full rate; mixlo and mixhi, which would also round, run at half of it.)
__device__ __forceinline__ void split_pk(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = cvt_pk_f16(a, b);
  float ra, rb;
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(hi), "v"(a));
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(hi), "v"(b));
  lo = cvt_pk_f16(ra, rb);
}

__device__ __forceinline__ float dot2_self_f16(uint32_t pk, float acc) {
  const f16x2 v = __builtin_bit_cast(f16x2, pk);
  return __builtin_amdgcn_fdot2(v, v, acc, false);
}

__device__ __forceinline__ f32x16 mfma_f16(const bf16x8& a, const bf16x8& b, f32x16 acc) {     // (eight fp16 numbers each)
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
}

// acc += K Q with K = hi + lo and Q one term
__device__ __forceinline__ f32x16 mma_scores(const Operand& a, const bf16x8 (&b)[2], f32x16 acc) {
#pragma unroll
  for (int q = 0; q < 2; ++q) acc = mfma_f16(a.lo[q].v, b[q], acc);
#pragma unroll
  for (int q = 0; q < 2; ++q) acc = mfma_f16(a.hi[q].v, b[q], acc);
  return acc;
}

// acc += A B, both hi + lo; lo is at most 2^-11 of hi, so what is left out (lo lo) is 2^-24 of the product at most
__device__ __forceinline__ f32x16 mma(const Operand& a, const Operand& b, f32x16 acc) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    acc = mfma_f16(a.lo[q].v, b.hi[q].v, acc);
    acc = mfma_f16(a.hi[q].v, b.lo[q].v, acc);
    acc = mfma_f16(a.hi[q].v, b.hi[q].v, acc);
  }
  return acc;
}

// v of lane i with that of another lane of the same sixteen, in registers: 1, 2, then those in reverse order of eight and of sixteen.
template <int CTRL>
__device__ __forceinline__ uint32_t turned(uint32_t v) { return uint32_t(__builtin_amdgcn_update_dpp(int(v), int(v), CTRL, 0xF, 0xF, false)); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, turned<0xB1>(v));
  v = max(v, turned<0x4E>(v));
  v = max(v, turned<0x141>(v));
  v = max(v, turned<0x140>(v));
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(r[0], r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max(h[0], h[1]);
}
// of this lane and the one in the other half
__device__ __forceinline__ float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float wave_sum(float v) {
  auto other = [](float x, auto ctrl) { return __uint_as_float(turned<decltype(ctrl)::value>(__float_as_uint(x))); };
  v += other(v, Int<0xB1>{});
  v += other(v, Int<0x4E>{});
  v += other(v, Int<0x141>{});
  v += other(v, Int<0x140>{});
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Largest of a lane's sixteen, three a time.
__device__ __forceinline__ float max16(const f32x16& s) {
  float t[2] = {s[0], s[1]};
#pragma unroll
  for (int i = 2; i < 14; i += 4) {
    t[0] = fmaxf(fmaxf(t[0], s[i]), s[i + 2]);
    t[1] = fmaxf(fmaxf(t[1], s[i + 1]), s[i + 3]);
  }
  return fmaxf(fmaxf(t[0], t[1]), fmaxf(s[14], s[15]));
}

// Shared memory of one workgroup.  WREG: a projecting wave keeps its D x 32 weight operands in registers instead of in LDS.
// Two slots of projected tiles are enough: a tile is published into the slot of the one whose operands every wave has
// read, one tile ago, and the barrier in between orders the two.
template <int D, int HPW, bool WREG>
struct SplitLds {
  uint4 xbuf[kXBuf][(D / 8) * 32];    // X tiles: [16-byte chunk][item], filled by direct global->LDS loads
  uint4 kvbuf[2][HPW][2][4][64];      // projected tiles: [slot][head][K|V][term, half of the 16 registers][lane]
  float knorm[2][HPW][64];            // squared norm of the scaled key rows (half per lane); infinite where fp16 does not hold them
  float vnorm[2][HPW][64];            // that of the value columns, infinite too
  int4 vunit[HPW][8];                 // a channel's published values times two to this and its piece's unit are its values
  int punit[4][HPW];                  // units of four pieces, by their number: the one attended over and the two that may be published beside it
  int qunit[4][HPW];                  // and of users' own queries: two to this is what they are divided by
  int redo;                           // some wave has records to form again
  uint4 wop[WREG ? 1 : HPW * 2 * (D / 16) * 64];   // projection weights as MFMA operands: [head][K|V][k-slice][lane]
};

// Partial records of a finished piece; slot = segment + user.
template <int NQB>
__device__ __forceinline__ void write_record(const MfmaSummarizeParams& p, int64_t slot, int h, int block, int lane, const f32x16 (&o)[NQB],
                                             const float (&l)[NQB], const float (&m)[NQB]) {
  char* rec = reinterpret_cast<char*>(p.partials + ((slot * p.H + h) * p.nqb + block) * kRecFloats);
  const uint32_t lane_off = uint32_t(lane) * 16;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    if (block + qb >= p.nqb) break;                    // a block past the last query has no record
    char* r = rec + size_t(qb) * kRecFloats * 4;       // scalar
#pragma unroll
    for (int i = 0; i < 16; i += 4)
      *reinterpret_cast<float4*>(r + i * 256 + lane_off) = make_float4(o[qb][i], o[qb][i + 1], o[qb][i + 2], o[qb][i + 3]);
    *reinterpret_cast<float2*>(r + kRecSums * 4 + lane_off / 2) = make_float2(half_sum(l[qb]), m[qb]);
  }
}

// The pieces whose records a wave has marked (m NaN) once more, with everything in fp32 and a running maximum: for keys, values and queries of any
// size, infinite and NaN ones included, and for rows that two fp16 terms leave too little of.  Each wave by itself, from memory; only the weights
// stand in LDS, where the tiles were.
template <int D, int NQB, int HPW, bool WREG>
__device__ __forceinline__ void pieces_in_fp32(const MfmaSummarizeParams& p, SplitLds<D, HPW, WREG>& sm, int64_t g, int h, int hl, int qblock,
                                                int64_t seg_begin, int64_t seg_end) {
  constexpr int KS = D / 16, kOps = HPW * 2 * KS * 64;       // [head][K|V][k-slice][lane]
  static_assert(sizeof(uint4) * kOps <= sizeof(sm.xbuf) + sizeof(sm.kvbuf), "the flag that all waves look at is behind the tiles");
  uint4* w = reinterpret_cast<uint4*>(&sm);
  const int lane = threadIdx.x & 63, hf = lane >> 5, l32 = lane & 31;
#pragma unroll 1
  for (int e = threadIdx.x; e < kOps; e += blockDim.x) {
    const int ks = (e >> 6) % KS, m = (e >> 6) / KS % 2, head = (e >> 6) / (2 * KS);
    const uint16_t* W = (m ? p.Wv : p.Wk) + (16 * ks + 8 * hf) * D + 32 * (h - hl + head) + l32;
    Pack8 t;
#pragma unroll
    for (int j = 0; j < 8; ++j) t.h[j] = W[j * D];
    w[e] = t.u;
  }
  lds_barrier();
  w += hl * 2 * KS * 64 + lane;
  f32x16 o[NQB];
  float l[NQB], m[NQB];
  auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      o[qb] = f32x16{0};
      l[qb] = 0.f;
      m[qb] = kLowest;
    }
  };
  reset();
  TileCursor c;
  c.init(p.offsets, p.B, find_user_wave(p.offsets, p.B, seg_begin), seg_begin, seg_end);
  bool marked = false, first = true;
#pragma unroll 1
  while (c.valid) {
    if (first) {
      const float* rec = p.partials + (((g + c.user) * p.H + h) * p.nqb + (qblock < p.nqb ? qblock : 0)) * kRecFloats;
      const float at = __hip_atomic_load(rec + kRecSums + 2 * lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      marked = qblock < p.nqb && __builtin_amdgcn_ballot_w64(__builtin_isnan(at)) != 0;
    }
    if (!marked) {                                       // to the piece's last tile
      c.skip(c.tiles_left - 1);
      c.advance(p.offsets, p.B, seg_end);
      continue;
    }
    const int rows = c.rows(), nvl = rows - 4 * hf;      // register i holds a row of the piece iff acc_row0(i) < nvl
    const uint16_t* x = p.X + (c.row + (l32 < rows ? l32 : rows - 1)) * D + 8 * hf;
    f32x16 k = {0}, v = {0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Pack8 t, wk, wv;
      t.u = *reinterpret_cast<const uint4*>(x + 16 * ks);
      wk.u = w[ks * 64];
      wv.u = w[(KS + ks) * 64];
      k = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wk.v, t.v, k, 0, 0, 0);
      v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.v, wv.v, v, 0, 0, 0);
    }
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      int q = qblock * 32 + qb * 32 + l32;
      if (q > p.S - 1) q = p.S - 1;
      const uint16_t* row = p.Q + p.q_user_stride * c.user + int64_t(q) * D + 32 * h + 4 * hf;
      f32x16 s = {0};
#pragma unroll
      for (int i = 0; i < 16; ++i)
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[i] * p.c, __uint_as_float(uint32_t(row[acc_row0(i)]) << 16), s, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (acc_row0(i) >= nvl) s[i] = -INFINITY;
      float top = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) top = fmaxf(top, s[i]);
      top = half_max(top);
      const float mnew = fmaxf(m[qb], top);
      const float alpha = __builtin_amdgcn_exp2f(m[qb] - mnew);
      l[qb] *= alpha;
#pragma unroll
      for (int i = 0; i < 16; ++i) o[qb][i] *= alpha;
      m[qb] = mnew;
      // rows past the piece are left out of the product, not only given weight 0: they may be infinite.  Sums of the tile first: weights of
      // nearly one, added to thousands one by one, would all be rounded the same way
      f32x16 t = {0};
      float lsum[2] = {0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float e = acc_row0(i) < nvl ? __builtin_amdgcn_exp2f(s[i] - mnew) : 0.f;
        t = __builtin_amdgcn_mfma_f32_32x32x2f32(acc_row0(i) < nvl ? v[i] : 0.f, e, t, 0, 0, 0);
        lsum[i & 1] += e;
      }
      l[qb] += lsum[0] + lsum[1];
#pragma unroll
      for (int i = 0; i < 16; ++i) o[qb][i] += t[i];
    }
    const bool last = c.tiles_left == 1;
    const int user = c.user;
    c.advance(p.offsets, p.B, seg_end);
    first = last;
    if (last) {
      write_record<NQB>(p, g + user, h, qblock, lane, o, l, m);
      reset();
    }
  }
}

// Body of one wave; ROLE 0 forms K^T, ROLE 1 forms V, ROLE 2 forms nothing and only attends.
template <int D, int NQB, int HPW, int FW, bool WREG, int ROLE>
__device__ __forceinline__ void split_wave(const MfmaSummarizeParams& p, SplitLds<D, HPW, WREG>& sm, int64_t g, int h, int hl,
                                           int qblock, int64_t seg_begin, int64_t seg_end) {
  constexpr bool PROJ = ROLE < 2;        // this wave projects
  constexpr int WR = PROJ ? ROLE : 0;    // its slot in the weight and K/V buffers (unused otherwise)
  constexpr int NT = FW * 64;            // threads that move X: the first FW waves
  constexpr int CH = D / 8;              // 16-byte chunks per row
  constexpr int KS = D / 16;             // k-slices of the projection
  constexpr int CPT = kTile * CH / NT;   // X chunks each of them moves per tile
  static_assert(kTile * CH % NT == 0, "tile must split evenly over the fetching waves");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int hf = lane >> 5;
  const int l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Projection weights of this wave's head as MFMA operands, in registers or parked in LDS
  // (each wave reads back only what it wrote).  Element j of slice ks is
  // W[16 ks + 8 hf + j][32 h + l32].
  bf16x8 wreg[WREG ? KS : 1];
  auto keep_weights = [&](int ks, const uint4& u) __attribute__((always_inline)) {
    Pack8 t;
    t.u = u;
    if constexpr (WREG) wreg[ks] = t.v; else sm.wop[((hl * 2 + WR) * KS + ks) * 64 + lane] = t.u;
  };
  // Rows of 32 columns are read 16 bytes a lane and turned by the matrix core: a 32 x 32 block times a
  // 0/1 selector lands in accumulator layout with the lane on the block's column.  The lane picks its
  // row so that registers 0..7 and 8..15 come out as two operands (row of register i, half hf:
  // 16 (i / 8) + 8 hf + i % 8).  Two loads a block instead of sixteen 2-byte ones; bit for bit the
  // same operands (a product with 1.0 is exact) as long as the weights are finite: an infinite or NaN
  // entry would spoil its whole row of the block (0 times it is NaN), so such weights go the other way.
  const uint16_t* W = ROLE ? p.Wv : p.Wk;
  const bool wide_rows = (reinterpret_cast<uintptr_t>(W) & 15) == 0;
  Pack8 wraw[PROJ ? KS / 2 : 1][2];
  auto request_weights = [&]() __attribute__((always_inline)) {
    if constexpr (PROJ) {
      if (wide_rows) {
        const int row = (l32 & 16) | ((l32 & 4) << 1) | ((l32 & 8) >> 1) | (l32 & 3);
        const uint16_t* src = W + row * D + 32 * h + 8 * hf;
#pragma unroll
        for (int b = 0; b < KS / 2; ++b)
#pragma unroll
          for (int q = 0; q < 2; ++q) wraw[b][q].u = *reinterpret_cast<const uint4*>(src + 32 * b * D + 16 * q);
      }
    }
  };
  auto settle_weights = [&]() __attribute__((always_inline)) {
    if constexpr (PROJ) {
      bool turned = wide_rows;
      if (wide_rows) {
        float rest[4] = {0.f, 0.f, 0.f, 0.f};      // stay 0 over finite weights, NaN otherwise
#pragma unroll
        for (int b = 0; b < KS / 2; ++b)
#pragma unroll
          for (int e = 0; e < 8; ++e) rest[e % 4] = dot2_zero(wraw[b][e / 4].w[e % 4], rest[e % 4]);
        turned = __builtin_amdgcn_ballot_w64((rest[0] + rest[1]) + (rest[2] + rest[3]) != 0.f) == 0;
      }
      if (turned) {
        Pack8 sel[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int j = 0; j < 8; ++j) sel[q].h[j] = (l32 == 16 * q + 8 * hf + j) ? 0x3F80 : 0;
#pragma unroll
        for (int b = 0; b < KS / 2; ++b) {
          f32x16 t = {0};
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wraw[b][0].v, sel[0].v, t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wraw[b][1].v, sel[1].v, t, 0, 0, 0);
#pragma unroll
          for (int q = 0; q < 2; ++q)
            keep_weights(2 * b + q,
                         make_uint4(cvt_pk_bf16(t[8 * q], t[8 * q + 1]), cvt_pk_bf16(t[8 * q + 2], t[8 * q + 3]),
                                    cvt_pk_bf16(t[8 * q + 4], t[8 * q + 5]), cvt_pk_bf16(t[8 * q + 6], t[8 * q + 7])));
        }
      } else {
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks) {
          Pack8 t;
#pragma unroll
          for (int j = 0; j < 8; ++j) t.h[j] = W[(16 * ks + 8 * hf + j) * D + 32 * h + l32];
          if constexpr (WREG) {
#pragma unroll
            for (int k2 = 0; k2 < KS; ++k2)
              if (k2 == ks) wreg[k2] = t.v;
          } else {
            keep_weights(ks, t.u);
          }
        }
      }
    }
  };

  // A channel's values are published times two powers of two that bring them to some 2^4 whatever the size of the weights and of a user's
  // items: by the norm of its column of W_v, and by 2^4, or, where the first tile of a piece has numbers above 2^8
  // by that or none above 1, by what takes its largest to 2^6: what fp16 cuts off, 2^-25, is then below what fp32 sums of a channel are known to.
  float vchannel = 1.f, vscale = 1.f;
  bool odd_column = false;           // weights too large or too small for that, or not finite
  auto settle_values = [&]() __attribute__((always_inline)) {
    if constexpr (ROLE == 1) {
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        Pack8 w;
        if constexpr (WREG) w.v = wreg[ks]; else w.u = sm.wop[((hl * 2 + WR) * KS + ks) * 64 + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) part[j] = dot2_self(w.w[j], part[j]);
      }
      float n2 = (part[0] + part[1]) + (part[2] + part[3]);
      n2 = half_sum(n2);
      const int e = (int(__float_as_uint(n2) >> 23) - 127) >> 1;       // floor of log2 of the norm
      const bool usual = n2 >= 8.6361686e-37f && n2 <= 1.1579209e36f;   // about 2^-120 .. 2^120; no column of zeros, nothing infinite or NaN
      vchannel = usual ? __uint_as_float(uint32_t(127 - e) << 23) : 1.f;
      odd_column = !usual && n2 != 0.f;
      if (hf == 0) reinterpret_cast<int*>(sm.vunit[hl])[l32] = usual ? e : 0;
    }
  };
  // The unit of the queries, the same for all waves of a head: a power of two that brings the largest number of eight rows to 1..2; keys are published
  // by the inverse.  Users' own queries have units of their own, which the K wave forms two tiles ahead with the piece's first keys.
  const bool own = p.q_user_stride != 0;
  float qunit = 1.f, kunit = 1.f;        // queries are taken times the first, keys times the second, the inverse of their user's
  uint2 qsome = make_uint2(0, 0);
  auto request_some = [&](int user) __attribute__((always_inline)) {
    qsome = *reinterpret_cast<const uint2*>(p.Q + p.q_user_stride * user + int64_t((lane >> 3) * p.S >> 3) * D + 32 * h + 4 * (lane & 7));
  };
  auto unit_of_some = [&]() __attribute__((always_inline)) {
    const uint32_t a = qsome.x & 0x7FFF7FFFu, b = qsome.y & 0x7FFF7FFFu;
    const uint32_t top = wave_max(max(max(a & 0xFFFFu, a >> 16), max(b & 0xFFFFu, b >> 16)));
    const int e = int(top >> 7) - 127;
    return top == 0 || e > 100 ? 0 : e < -100 ? -100 : e;        // (0 for an infinite or NaN one too)
  };
  auto power_of_two = [](int e) __attribute__((always_inline)) { return __uint_as_float(uint32_t(127 + e) << 23); };
  int pieces_out = 0;                // pieces published so far
  auto start_piece = [&](const f32x16& acc) __attribute__((always_inline)) {
    if constexpr (ROLE == 0) {
      if (own) {
        const int e = unit_of_some();
        kunit = power_of_two(e);
        if (lane == 0) sm.qunit[pieces_out & 3][hl] = e;
        ++pieces_out;
      }
    }
    if constexpr (ROLE == 1) {
      float most[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) most[i % 4] = fmaxf(most[i % 4], fabsf(acc[i]));
      const float mine = fmaxf(fmaxf(most[0], most[1]), fmaxf(most[2], most[3])) * vchannel;
      int up = 4;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(mine <= 256.f)) != 0 || __builtin_amdgcn_ballot_w64(mine >= 1.f) == 0, 0)) {
        const uint32_t top = wave_max(__float_as_uint(mine) & 0x7FFFFFFFu);
        if (top >= 0x20000000u && top < 0x5F800000u) up = 6 - (int(top >> 23) - 127);      // 2^-63 .. 2^64
      }
      vscale = ldexpf(vchannel, up);
      if (lane == 0) sm.punit[pieces_out & 3][hl] = -up;
      ++pieces_out;
    }
  };

  const int qbase = qblock * 32;         // first query of this wave
  bf16x8 qop[NQB][2];                    // (once settled, the bits of fp16 numbers)
  float qmax2 = 0.f;
  auto request_queries = [&](int user) __attribute__((always_inline)) {
    const char* Qb = reinterpret_cast<const char*>(p.Q + p.q_user_stride * user + 32 * h) + 8 * hf;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      int q = qbase + qb * 32 + l32;
      if (q > p.S - 1) q = p.S - 1;              // columns past the last query repeat it; never read back
      const char* row = Qb + q * (D * 2);
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        Pack8 t;
        // dh index of element j: 16 part + 4 hf + 8 (j / 4) + j % 4 -> two runs of four
        const uint2 a = *reinterpret_cast<const uint2*>(row + 32 * part);
        const uint2 b = *reinterpret_cast<const uint2*>(row + 32 * part + 16);
        t.w[0] = a.x; t.w[1] = a.y; t.w[2] = b.x; t.w[3] = b.y;
        qop[qb][part] = t.v;
      }
    }
  };
  bool coarse = false;                   // some query number lost bits
  float bound2 = 0.f;                    // keys of no larger squared norm have scores within kPlainScore
  bool lost_queries = false;             // queries beyond what fp16 terms take
  auto settle_queries = [&]() __attribute__((always_inline)) {
    float worst = 0.f, rest = 0.f;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      float n2 = 0.f;
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        Pack8 t;
        t.v = qop[qb][part];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float a = __uint_as_float(t.w[j] << 16) * qunit, b = __uint_as_float(t.w[j] & 0xFFFF0000u) * qunit;
          n2 = fmaf(a, a, n2);
          n2 = fmaf(b, b, n2);
          t.w[j] = cvt_pk_f16(a, b);
          rest = fmaxf(rest, fmaxf(fabsf(a - f16_lo(t.w[j])), fabsf(b - f16_hi(t.w[j]))));
        }
        qop[qb][part] = t.v;
      }
      n2 = half_sum(n2);
      worst = n2 <= kQueryMost2 ? fmaxf(worst, n2) : INFINITY;
    }
    qmax2 = __uint_as_float(wave_max(__float_as_uint(worst)));     // (not negative)
    lost_queries = __builtin_amdgcn_ballot_w64(qmax2 == INFINITY) != 0;
    coarse = __builtin_amdgcn_ballot_w64(rest != 0.f) != 0;
    bound2 = fminf(kPlainScore * kPlainScore / qmax2, coarse ? kKeyMost2 : kHalfMost2);
  };

  // ---- the segment as one stream of tiles (TileCursor: scalar state, offsets read through
  // uniform loads).  `ca` names the tile being attended over, `cf` runs three tiles ahead
  // and names the tile whose rows are requested from HBM.
  using Cursor = TileCursor;
  auto cursor_init = [&](Cursor& c) __attribute__((always_inline)) {
    c.init(p.offsets, p.B, find_user_wave(p.offsets, p.B, seg_begin), seg_begin, seg_end);
  };
  auto cursor_advance = [&](Cursor& c) __attribute__((always_inline)) { c.advance(p.offsets, p.B, seg_end); };
  // whether the tile it then names is the first of a piece
  auto cursor_enters = [&](Cursor& c) __attribute__((always_inline)) {
    const bool last = c.tiles_left == 1;
    cursor_advance(c);
    return last && c.valid ? 1 : 0;
  };

  f32x16 o[NQB];
  float l[NQB], m[NQB];
  int mode = 0;                  // 0 fresh piece, 1 reference m, 2 not for fp16 terms: nothing more is done for the piece, its record is formed again
  bool redo = false;             // this wave has such records
  float safe2 = -1.f;            // bound2, or less than any where a row's m is out of the way
  float vsum = 0.f;              // this lane's share of the squared norms of the values so far
  int tiles = 0;                 // of the piece so far
  // scores come out of the matrix core less m: one more product, of ones at k = 0 with -m there (fp16 holds whole numbers to 2048)
  Pack8 ones, mop[NQB];
  ones.u = make_uint4(hf == 0 ? 0x3C00u : 0u, 0u, 0u, 0u);
  auto set_reference = [&](int qb) __attribute__((always_inline)) {
    mop[qb].u = make_uint4(hf == 0 ? cvt_pk_f16(-m[qb], 0.f) : 0u, 0u, 0u, 0u);
  };
  auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[qb][i] = 0.f;
      l[qb] = 0.f;
      m[qb] = kFirstReference;
      set_reference(qb);
    }
    mode = 0;
    safe2 = bound2;
    vsum = 0.f;
    tiles = 0;
  };

  // HBM -> LDS movement of X without a stop in registers (global_load_lds, 16 bytes
  // per lane: lane i of a wave lands at the wave's LDS base + 16 i).  Tile t lives in
  // xbuf[t % 3]; the rows of tile t+3 are requested at the top of tile t into the
  // buffer tile t has vacated and must have landed by the end of tile t+1, so a
  // load has two tile periods.  Rows past the piece are clamped to its last row.
  auto fetch_rows = [&](const char* base, int last, int xb) __attribute__((always_inline)) {   // last: last valid row
    if (wave >= FW) return;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int slot = k * NT + tid;                         // LDS slot = chunk * 32 + item
      int rel = slot & 31;
      if (rel > last) rel = last;
      const uint32_t voff = uint32_t(rel) * (D * 2) + uint32_t(slot >> 5) * 16;
      // Written as assembly so that the completion wait is the explicit vmcnt wait at
      // the end of the next tile, not a conservative one before the next LDS read.
      const uint32_t lds_base = uint32_t(reinterpret_cast<uintptr_t>(
          (void __attribute__((address_space(3)))*)(&sm.xbuf[xb][k * NT + wave * 64])));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :
                   : "s"(lds_base), "v"(voff), "s"(base)
                   : "memory", "m0");
    }
  };
  auto fetch = [&](const Cursor& c, int xb) __attribute__((always_inline)) {
    fetch_rows(reinterpret_cast<const char*>(p.X) + c.row * (D * 2), c.rows() - 1, xb);
  };
  // k-slices [ks0, ks1) of this wave's projection of the X tile in xbuf[buf]
  auto project = [&](int buf, int ks0, int ks1, f32x16& acc) __attribute__((always_inline)) {
    if constexpr (PROJ) {
#pragma unroll
      for (int ks = ks0; ks < ks1; ++ks) {
        Pack8 x, w;
        x.u = sm.xbuf[buf][(2 * ks + hf) * 32 + l32];
        if constexpr (WREG) w.v = wreg[ks]; else w.u = sm.wop[((hl * 2 + WR) * KS + ks) * 64 + lane];
        acc = ROLE ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, w.v, acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.v, x.v, acc, 0, 0, 0);
      }
    }
  };
  // hand the projected tile to the partner waves: operands (+ key norms), a pair of registers at a time
  auto publish_pair = [&](const f32x16& acc, int i, Operand& r, float& n2) __attribute__((always_inline)) {
    const float c = ROLE ? vscale : p.c * kunit;           // the keys' scale, in fp32
    uint32_t& pk = r.hi[i / 8].w[(i % 8) / 2];
    split_pk(acc[i] * c, acc[i + 1] * c, pk, r.lo[i / 8].w[(i % 8) / 2]);
    n2 = dot2_self_f16(pk, n2);
  };
  auto publish_pairs = [&](int buf, const f32x16& acc, Operand& r, float n2) __attribute__((always_inline)) {
    if constexpr (PROJ) {
      bool lost = !(n2 <= kHalfMost2) || (ROLE == 1 && odd_column);
      if (ROLE == 1 && __builtin_expect(__builtin_amdgcn_ballot_w64(n2 == 0.f) != 0, 0)) {      // (nothing but zeros is well kept)
        float any = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) any = fmaxf(any, fabsf(acc[i]));
        lost |= n2 == 0.f && any > 0.f;
      }
      if (lost) n2 = INFINITY;
      if (ROLE == 0) sm.knorm[buf][hl][lane] = n2; else sm.vnorm[buf][hl][lane] = n2;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        sm.kvbuf[buf][hl][WR][q][lane] = r.hi[q].u;
        sm.kvbuf[buf][hl][WR][2 + q][lane] = r.lo[q].u;
      }
    }
  };
  auto publish = [&](int buf, const f32x16& acc) __attribute__((always_inline)) {
    if constexpr (PROJ) {
      Operand r;
      float n2 = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) publish_pair(acc, i, r, n2);
      publish_pairs(buf, acc, r, n2);
    }
  };
  float vn2 = 0.f;          // squared norm of half a value column of the tile being attended over
  auto unsafe_tile = [&](float kn2) __attribute__((always_inline)) { return __builtin_amdgcn_ballot_w64(!(kn2 <= safe2)) != 0; };

  // everything the workgroup starts from is requested before any of it is waited for
  request_weights();
  if (!own) {
    request_some(0);
    request_queries(0);
  }
  Cursor ca, cf;
  cursor_init(ca);
  cf = ca;

  // Common case: a full tile, bounded scores, another tile behind it.  Straight-line
  // code (one scheduling region per tile): two projection MFMAs of the next tile ride
  // along with every query block of this one.
  Operand kk, vv;    // K/V operands of the tile being attended over
  float kn2 = 0.f;          // its squared key norm (this lane's item)
  // Operands of tile t+1 (ring slot i1) come out of LDS while tile t is still being worked on,
  // into the registers tile t has just finished with: K (and the norms) once the last scores
  // of the tile are issued, V after its last P.V product.  They were published one tile ago
  // and the barrier at the start of tile t made them visible, so by the next barrier they
  // are in registers and the next tile starts without a round trip to LDS.
  auto read_operand = [&](Operand& r, int i1, int which) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      r.hi[q].u = sm.kvbuf[i1][hl][which][q][lane];
      r.lo[q].u = sm.kvbuf[i1][hl][which][2 + q][lane];
    }
  };
  auto read_k = [&](int i1) __attribute__((always_inline)) {
    read_operand(kk, i1, 0);
    kn2 = sm.knorm[i1][hl][lane] + sm.knorm[i1][hl][lane ^ 32];
    vn2 = sm.vnorm[i1][hl][lane];
  };
  auto read_v = [&](int i1) __attribute__((always_inline)) {
    read_operand(vv, i1, 1);
  };
  int odd = 0;              // tile index mod 2
  // slot of tile t+2 in the ring of the X tiles, slots of tiles t+1 and t+2 among the operands; r = tile index mod 3
  struct Slots { int x2, kv1, kv2; };
  auto slots = [&](int r) __attribute__((always_inline)) {
    const int i1 = r == kXBuf - 1 ? 0 : r + 1, i2 = i1 == kXBuf - 1 ? 0 : i1 + 1;
    return Slots{i2, odd ^ 1, odd};
  };
  f32x16 nx = {0};          // scores less m of the first block of the tile to come, where that is a plain one
  // the next n slices of a projection, the operand of the one behind them requested
  auto project_some = [&](int buf, int n, int& ks, Pack8& xr, f32x16& acc) __attribute__((always_inline)) {
    if constexpr (PROJ) {
#pragma unroll
      for (int i = 0; i < n; ++i) {
        if (ks >= KS) break;
        Pack8 w;
        if constexpr (WREG) w.v = wreg[ks]; else w.u = sm.wop[((hl * 2 + WR) * KS + ks) * 64 + lane];
        acc = ROLE ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(xr.v, w.v, acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.v, xr.v, acc, 0, 0, 0);
        pin(acc);
        ++ks;
        if (ks < KS) xr.u = sm.xbuf[buf][(2 * ks + hf) * 32 + l32];
      }
    }
  };
  // product j of five; the reference last, so that the sums before it are of the scores' own size
  auto score_product = [&](int qb, int j, const f32x16& s) __attribute__((always_inline)) {
    if (j == 4) return mfma_f16(ones.v, mop[qb].v, s);
    return mfma_f16((j < 2 ? kk.lo[j & 1] : kk.hi[j & 1]).v, qop[qb][j & 1], j ? s : f32x16{0});
  };
  // which of the tiles t + 2, t + 3 and t + 4, from the lowest bit, are the first of their piece
  int firsts = 0, user2 = 0, user3 = 0, user4 = 0;      // and whose they are
  // A plain tile, in an order of its own (pin): every pair of exponentials, its split and its sum stand between two products, those of the
  // next block's scores, of the block before with the values and of the projection.  A tile ends with the first scores of the next
  // one (nx) and its last block's products, beside the projected tile's own split.
  // Where a weight would leave fp16's range, or a piece's first tile has none in the middle of it, the row's reference is moved before the exponentials.
  // straight: no piece starts within the tiles on their way.
  auto fast_tile = [&](int r, auto straight) __attribute__((always_inline)) {
    const Slots at = slots(r);
    f32x16 acc = {0};
    int ks = 0;
    Pack8 xr;
    if constexpr (PROJ) xr.u = sm.xbuf[at.x2][hf * 32 + l32];
    Operand before;      // weights of the block before
    auto score = [&](int qb, int j, f32x16& s) __attribute__((always_inline)) {
      s = score_product(qb, j, s);
      pin(s);
    };
    auto second = [&](int qb, const Operand& w, int j) __attribute__((always_inline)) {
      const int q = j / 3;
      o[qb] = mfma_f16((j % 3 == 0 ? vv.lo[q] : vv.hi[q]).v, (j % 3 == 1 ? w.lo[q] : w.hi[q]).v, o[qb]);
      pin(o[qb]);
    };
    vsum += vn2;
    ++tiles;
    if (NQB == 1) read_k(at.kv1);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      f32x16 sc = nx;
      float top = max16(sc);
      const float low = mode == 0 ? kFirstBest : -INFINITY;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(top > kTopWeight || top < low) != 0, 0)) {
        top = half_max(top);
        const float by = top > kTopWeight || top < low ? floorf(top) - kBestWeight : 0.f, alpha = __builtin_amdgcn_exp2f(-by);
        m[qb] += by;
        l[qb] *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sc[i] -= by;
          o[qb][i] *= alpha;
        }
        set_reference(qb);
      }
      f32x16 nn;
      float ev[16], lsum[2] = {0.f, 0.f};
      Operand cur;
      const bool more = qb + 1 < NQB;
      if (NQB > 1 && !more) read_k(at.kv1);      // this tile's scores are all issued
#pragma unroll
      for (int st = 0; st < 9; ++st) {
        if (st < 8) {
#pragma unroll
          for (int e = 2 * st; e < 2 * st + 2; ++e) { ev[e] = __builtin_amdgcn_exp2f(sc[e]); pin(ev[e]); }
        }
        if (st > 0) {
          const int i = 2 * st - 2;
          uint32_t hi, lo;
          split_pk(ev[i], ev[i + 1], hi, lo);
          pin(lo);
          cur.hi[i / 8].w[(i % 8) / 2] = hi;
          cur.lo[i / 8].w[(i % 8) / 2] = lo;
          lsum[0] += ev[i];
          lsum[1] += ev[i + 1];
          pin(lsum[0]);
          pin(lsum[1]);
        }
        if (more && ((st & 1) || st == 8)) score(qb + 1, st / 2, nn);
        if (qb > 0 && st < 6) second(qb - 1, before, st);
        if (!more && st > 5) second(qb, cur, st - 6);
        if (st < 8) project_some(at.x2, ((qb * 8 + st + 1) * KS) / (NQB * 8) - ((qb * 8 + st) * KS) / (NQB * 8), ks, xr, acc);
      }
      l[qb] += lsum[0] + lsum[1];
      before = cur;
      if (more) nx = nn;
    }
    if constexpr (!decltype(straight)::value) {
      if (firsts & 1) start_piece(acc);
    }
    Operand pub;
    float n2 = 0.f;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      if (st < 3) second(NQB - 1, before, 3 + st);
      else score(0, st - 3, nx);
      if constexpr (PROJ) {
        publish_pair(acc, 2 * st, pub, n2);
        pin(n2);
      }
    }
    mode = 1;
    read_v(at.kv1);
    if constexpr (PROJ) publish_pairs(at.kv2, acc, pub, n2);
  };

  // the accumulators in the values' own units
  int pieces_done = 0;
  auto scale_values = [&]() __attribute__((always_inline)) {
    const int unit = sm.punit[pieces_done & 3][hl];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int4 u = sm.vunit[hl][2 * g4 + hf];        // channels 8 g4 + 4 hf + 0..3: rows of registers 4 g4..
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        o[qb][4 * g4] = ldexpf(o[qb][4 * g4], u.x + unit);
        o[qb][4 * g4 + 1] = ldexpf(o[qb][4 * g4 + 1], u.y + unit);
        o[qb][4 * g4 + 2] = ldexpf(o[qb][4 * g4 + 2], u.z + unit);
        o[qb][4 * g4 + 3] = ldexpf(o[qb][4 * g4 + 3], u.w + unit);
      }
    }
  };
  // whether every row of this wave is known well enough (the accumulators in the terms' units)
  auto rows_known = [&]() __attribute__((always_inline)) {
    const float v2 = wave_sum(vsum);
    const float n = 32.f * float(tiles);
    const float by_l = v2 == 0.f ? 0.f : v2 >= kValueMean2 * n ? fminf(kValuesLost2, kMeanLost2 * v2 / (n * n)) : kValuesLost2;
    const float by_n = kWeightsLost2 * n * v2;
    bool bad = !(v2 < INFINITY);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) part[i % 4] = fmaf(o[qb][i], o[qb][i], part[i % 4]);
      const float o2 = half_sum((part[0] + part[1]) + (part[2] + part[3])), ls = half_sum(l[qb]);
      bad |= !(o2 >= by_n && o2 >= by_l * ls * ls && o2 < INFINITY);
    }
    return __builtin_amdgcn_ballot_w64(bad) == 0;
  };
  // Any tile: ragged tail, scores beyond the bound, last tile of the segment.
  auto slow_tile = [&](int r, int nvalid) __attribute__((always_inline)) {
    const Slots at = slots(r);
    const int nvl = nvalid - 4 * hf;
    if (__builtin_expect(lost_queries || __builtin_amdgcn_ballot_w64(!(kn2 < INFINITY) || (coarse && kn2 > kKeyMost2)) != 0, 0)) mode = 2;
    if (__builtin_expect(mode != 2, 1)) {
      if (mode == 0) {
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) m[qb] = kLowest;
      }
      vsum += vn2;
      ++tiles;
      f32x16 sc[NQB];
      float top[NQB];
      bool raise = false;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) sc[qb] = mma_scores(kk, qop[qb], f32x16{0});
      if (nvalid < kTile) {
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (acc_row0(i) >= nvl) sc[qb][i] = -INFINITY;
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) top[qb] = max16(sc[qb]);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        top[qb] = half_max(top[qb]);
        raise |= top[qb] - m[qb] > kTopWeight;
      }
      if (__builtin_amdgcn_ballot_w64(raise) != 0) {
        bool out = false;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const float mq = top[qb] - m[qb] > kTopWeight ? floorf(top[qb]) - kBestWeight : m[qb];
          const float alpha = __builtin_amdgcn_exp2f(m[qb] - mq);      // 0 on a piece's first tile (m lowest)
          l[qb] *= alpha;
#pragma unroll
          for (int i = 0; i < 16; ++i) o[qb][i] *= alpha;
          m[qb] = mq;
          set_reference(qb);
          out |= !(fabsf(mq) <= kPlainScore + kBestWeight + 1.f);
        }
        safe2 = __builtin_amdgcn_ballot_w64(out) != 0 ? -1.f : bound2;
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        Operand pw;
        float lsum[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float ea = __builtin_amdgcn_exp2f(sc[qb][i] - m[qb]), eb = __builtin_amdgcn_exp2f(sc[qb][i + 1] - m[qb]);
          split_pk(ea, eb, pw.hi[i / 8].w[(i % 8) / 2], pw.lo[i / 8].w[(i % 8) / 2]);
          lsum[0] += ea;
          lsum[1] += eb;
        }
        l[qb] += lsum[0] + lsum[1];
        o[qb] = mma(vv, pw, o[qb]);
      }
      mode = 1;
    }
    read_k(at.kv1);
    read_v(at.kv1);
    // the tile two ahead (past the end of the segment: a repeat of its last tile, never used)
    f32x16 acc = {0};
    project(at.x2, 0, KS, acc);
    if (firsts & 1) start_piece(acc);
    publish(at.kv2, acc);
  };

  // partial record of a finished piece: slot = segment + user
  auto write_partial = [&](int user) __attribute__((always_inline)) {
    if (mode == 2 || !rows_known()) {
      redo = true;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) m[qb] = NAN;
    } else {
      scale_values();
    }
    ++pieces_done;
    write_record<NQB>(p, g + user, h, qbase / 32, lane, o, l, m);
  };

  if (!ca.valid) return;               // only with invalid offsets (whole workgroup)
  reset_state();

  // Waits until at most `pending` of this wave's newest vector-memory operations
  // are outstanding (s_waitcnt vmcnt only; the other counters are left alone).
  auto wait_vm = [&](auto n_c) __attribute__((always_inline)) {
    constexpr int n = decltype(n_c)::value;
    __builtin_amdgcn_s_waitcnt((n & 0xF) | ((n >> 4) << 14) | 0x0F70);
  };

  // Tile t lives in ring slot t mod 3, as raw rows (xbuf) and, projected, as operands
  // (kvbuf, slot t mod 2).  While tile t is attended over, tile t+2 is projected and published, the
  // operands of tile t+1 move into registers, the rows of tile t+3 land and those of tile
  // t+4 are requested into the slot whose rows (tile t+1) were projected one tile ago.
  // ---- prologue: tiles 0, 1, 2 requested; 0 and 1 landed, projected and published
  fetch(cf, 0);
  const int first1 = cursor_enters(cf);
  fetch(cf, 1);
  const int user1 = cf.user;
  firsts = cursor_enters(cf);
  user2 = cf.user;
  fetch(cf, 2);
  firsts |= cursor_enters(cf) << 1;
  user3 = cf.user;
  if (own) {
    request_some(ca.user);
    request_queries(ca.user);
  }
  settle_weights();
  settle_values();
  {
    const int e = unit_of_some();
    kunit = power_of_two(e);
    qunit = power_of_two(-e);
  }
  settle_queries();
  safe2 = bound2;
  wait_vm(Int<CPT>{});
  lds_barrier();
  {
    f32x16 acc = {0};
    project(0, 0, KS, acc);
    start_piece(acc);
    publish(0, acc);
    f32x16 acc1 = {0};
    project(1, 0, KS, acc1);
    if (first1) {
      if (own && ROLE == 0) request_some(user1);
      start_piece(acc1);
    }
    publish(1, acc1);
  }
  lds_barrier();              // slot 0's rows are projected by everyone, its operands are visible
  fetch(cf, 0);               // tile 3
  firsts |= cursor_enters(cf) << 2;
  user4 = cf.user;
  read_k(0);
  read_v(0);
  wait_vm(Int<CPT>{});        // tile 2 has landed

  // One barrier per tile on either route (waves may take different routes: the bound
  // depends on each wave's queries).  Runs of plain tiles (full, bounded scores, not
  // the last of their piece) stay in the inner loop, whose body is straight-line
  // code with the accumulators updated in place; every other tile leaves it, takes
  // the general route and does the piece bookkeeping.
  int r = 0;              // ring slot of the tile being attended over
  bool drain = false;     // other vector-memory traffic (record stores, query loads) is in flight
  // Tile t+3 (requested one tile ago) must have landed before the next barrier; the
  // request just issued for tile t+4 may stay in flight.  Loads complete in order
  // among themselves but not with respect to stores, so after a record write
  // everything is drained once.
  auto end_of_tile = [&]() __attribute__((always_inline)) {
    if (drain) wait_vm(Int<0>{}); else wait_vm(Int<CPT>{});
    drain = false;
    firsts = (firsts >> 1) | (cursor_enters(cf) << 2);
    user2 = user3;
    user3 = user4;
    user4 = cf.user;
  };
  // Start of a tile: the barrier, then the request for tile t+4.
  auto begin_tile = [&]() __attribute__((always_inline)) {
    lds_barrier();
    fetch(cf, r == kXBuf - 1 ? 0 : r + 1);
    if constexpr (ROLE == 0)
      if (own && (firsts & 1)) request_some(user2);
  };
  // whether the tile whose operands are in registers is a plain one
  bool unsafe = unsafe_tile(kn2);
  auto is_plain = [&]() __attribute__((always_inline)) {
    return !(ca.tiles_left == 1 || mode == 2 || unsafe);
  };
  bool plain = is_plain();
  auto first_scores = [&]() __attribute__((always_inline)) {       // a plain tile behind another one has them already
#pragma unroll
    for (int j = 0; j < 5; ++j) nx = score_product(0, j, nx);
  };
  if (plain) first_scores();
  for (;;) {
    // Plain tiles while the tile being requested is a full one of the same piece: no cursor in the loop, whose
    // branches and state moves would be on every wave between two barriers.
    if (plain) {
      const int run = cf.straight(ca);
      const char* base = reinterpret_cast<const char*>(p.X) + cf.row * (D * 2);
      int n = 0;
      while (n < run && plain) {
        // The loop's head on a cache line: d = 128, 300 007 items, S = 300 212 -> 200 us a call, S = 400 232 -> 228, S = 100 and 200 the same; d = 256 loses
        // (S = 100 317 -> 323), d = 64 is the same.
        if constexpr (D == 128) asm volatile(".p2align 6");
        lds_barrier();
        fetch_rows(base, kTile - 1, r == kXBuf - 1 ? 0 : r + 1);
        base += kTile * D * 2;
        fast_tile(r, Int<1>{});
        if (drain) wait_vm(Int<0>{}); else wait_vm(Int<CPT>{});
        drain = false;
        ++n;
        r = r == kXBuf - 1 ? 0 : r + 1;
        odd ^= 1;
        unsafe = unsafe_tile(kn2);
        plain = !unsafe;
      }
      ca.skip(n);
      cf.skip(n);
      plain = is_plain();
    }
    while (__builtin_expect(plain, 1)) {
      begin_tile();
      fast_tile(r, Int<0>{});
      end_of_tile();
      --ca.tiles_left;
      ca.row += kTile;
      r = r == kXBuf - 1 ? 0 : r + 1;
      odd ^= 1;
      unsafe = unsafe_tile(kn2);
      plain = is_plain();
    }
    begin_tile();
    const bool last_in_piece = ca.tiles_left == 1;
    const int nvalid = last_in_piece ? ca.tail : kTile;
    slow_tile(r, nvalid);
    end_of_tile();
    const int done_user = ca.user;
    cursor_advance(ca);
    if (last_in_piece) {
      write_partial(done_user);
      reset_state();
      if (own && ca.valid) {
        request_queries(ca.user);
        qunit = power_of_two(-sm.qunit[pieces_done & 3][hl]);
        settle_queries();
        safe2 = bound2;
      }
      drain = true;
    }
    r = r == kXBuf - 1 ? 0 : r + 1;
    odd ^= 1;
    if (!ca.valid) break;
    unsafe = unsafe_tile(kn2);
    plain = is_plain();
    if (plain) first_scores();
  }
  if (redo) sm.redo = 1;
}


// NQB query blocks a wave; the first FW waves fetch X.  At d = 64 a wave of one block has 168 registers, so that three fit a SIMD.
template <int D, int NQB, int HPW, int FW, bool WREG>
__global__ __launch_bounds__(512, D == 64 && NQB == 1 ? 3 : 2) void split_mfma_kernel(MfmaSummarizeParams p) {
  __shared__ SplitLds<D, HPW, WREG> sm;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept scalar
  const int hl = wave / p.wph;
  // slot 0 projects K, slot 1 projects V, the others only attend; the slots of successive heads are
  // turned by two so that every SIMD (wave id mod 4) gets its share of projecting waves
  int slot = wave - hl * p.wph + 2 * hl;
  while (slot >= p.wph) slot -= p.wph;

  // XCD-aware block -> (segment, head group): the head groups of one segment
  // share an XCD (and its L2) because their block ids differ by multiples of 8.
  const int64_t id = blockIdx.x;
  const int64_t grp = id / (8 * p.nhg);
  const int idl = int(id - grp * 8 * p.nhg);
  const int64_t g = grp * 8 + (idl & 7);
  const int hg = idl >> 3;
  const int h = hg * HPW + hl;
  const int64_t seg_begin = g * p.seg;
  if (seg_begin >= p.N) return;          // padding blocks of the last group (whole workgroup)
  const int64_t seg_end = (seg_begin + p.seg < p.N) ? seg_begin + p.seg : p.N;
  // the seeds' own keys and values, as in summarize_mfma_kernel
  if (__builtin_expect(p.Ks != nullptr, 0)) {
    const int64_t groups = (p.N + p.seg - 1) / p.seg * p.nhg, units = (p.self_rows + 31) / 32 * (D / 32);
    for (int64_t u = int64_t(wave) * groups + g * p.nhg + hg; u < units; u += groups * (blockDim.x >> 6))
      self_kv_unit(p.Q, p.Wk, p.Wv, p.Ks, p.Vs, p.self_rows, D, u);
  }
  // All roles run the same sequence of barriers; only the MFMA operand order differs.
  const int qblock = slot * NQB;
  if (threadIdx.x == 0) sm.redo = 0;      // (set behind the first tile's barrier at the earliest)
  if (slot == 0)
    split_wave<D, NQB, HPW, FW, WREG, 0>(p, sm, g, h, hl, qblock, seg_begin, seg_end);
  else if (slot == 1)
    split_wave<D, NQB, HPW, FW, WREG, 1>(p, sm, g, h, hl, qblock, seg_begin, seg_end);
  else
    split_wave<D, NQB, HPW, FW, WREG, 2>(p, sm, g, h, hl, qblock, seg_begin, seg_end);
  __builtin_amdgcn_s_waitcnt(0x0F70);     // rows still on their way to LDS, records
  lds_barrier();
  if (__builtin_expect(sm.redo != 0, 0)) pieces_in_fp32<D, NQB, HPW, WREG>(p, sm, g, h, hl, qblock, seg_begin, seg_end);
}

template <int D, int NQB, int HPW, int FW, bool WREG>
hipError_t launch_kernel(MfmaSummarizeParams& p, int wph, int64_t G, hipStream_t s) {
  p.wph = wph;
  p.nhg = p.H / HPW;
  const int64_t blocks = (G + 7) / 8 * 8 * p.nhg;
  return launch(split_mfma_kernel<D, NQB, HPW, FW, WREG>, dim3(unsigned(blocks)), dim3(HPW * wph * 64), 0, s, p);
}

}  // namespace

hipError_t launch_split(MfmaSummarizeParams& p, int d, bool one_head, int64_t G, hipStream_t s) {
  const int w1 = p.nqb < 4 ? 4 : p.nqb, w2 = p.nqb < 3 ? 2 : (p.nqb + 1) / 2;   // waves per head at one, two query blocks
  if (one_head) {
    const int w = p.nqb < 2 ? 2 : p.nqb;
    if (d == 64) return w < 4 ? launch_kernel<64, 1, 1, 2, true>(p, w, G, s) : launch_kernel<64, 1, 1, 4, true>(p, w, G, s);
    return w < 4 ? launch_kernel<128, 1, 1, 2, true>(p, w, G, s) : launch_kernel<128, 1, 1, 4, true>(p, w, G, s);
  }
  if (d == 64) {
    if (p.nqb <= 2) return launch_kernel<64, 1, 2, 4, true>(p, 2, G, s);
    if (p.nqb <= 8) return launch_kernel<64, 2, 2, 4, true>(p, w2, G, s);
    return launch_kernel<64, 2, 1, 4, true>(p, w2, G, s);
  }
  if (d == 128) {
    if (p.nqb <= 2) return launch_kernel<128, 1, 2, 4, true>(p, 2, G, s);
    if (p.nqb <= 8) return launch_kernel<128, 2, 2, 4, true>(p, w2, G, s);
    return launch_kernel<128, 2, 1, 4, true>(p, w2, G, s);
  }
  if (p.nqb <= 8) return launch_kernel<256, 1, 1, 4, true>(p, w1, G, s);
  return launch_kernel<256, 2, 1, 4, false>(p, w2, G, s);
}

}  // namespace vista
