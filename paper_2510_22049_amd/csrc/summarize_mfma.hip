// Stage 1 on the matrix cores (bf16 MFMA, fp32 accumulate), gfx950.
//
// One workgroup streams one flat segment of the packed history for HPW heads.
// Each head is served by a pair of waves.  Per tile of 32 items:
//   1. the X tile (32 x D bf16) goes from HBM straight into LDS (direct
//      global->LDS loads, three tiles deep, no stop in registers);
//   2. wave "K" of a pair forms K_h^T = (scale*log2e W_k,h)^T X^T, wave "V" forms
//      V_h = X W_v,h -- D / 16 32x32x16 MFMAs each, weights held in registers (as LDS operands only
//      with four query blocks a wave at d = 256) -- and both hand the bf16
//      result to their partner through LDS;
//   3. each wave owns half of the S queries: for every block of 32 queries
//      S^T = K_h Q_h^T (items x queries), p = 2^(s - m), O^T += V_h^T P^T.
// With items on the MFMA row index and queries on the column index, every lane
// owns one query column: the softmax statistics are per-lane scalars, the
// fp32 score registers turn into the bf16 P operand without any shuffle, and
// the projected K^T / V accumulators already are the next MFMA's A operand.
// The projection of tile t+1 rides along with the attention over tile t, and
// the tiles of all pieces (user x segment) of the segment form one stream.
// Where a pair would leave a wave with more than four query blocks (S = 512) or
// with too few waves per compute unit (D = 256), a head gets more waves instead:
// the K and V waves plus others that only attend, the queries shared by all.  At D = 256, S = 512 they are shared
// unevenly in long softmax histories and in workgroups of half the heads: two blocks to a projecting wave, whose weights take
// 64 registers, six to the others, which comes to 24 MFMAs a tile for each of the four.
// (Sixteen waves of two query blocks and 128 registers each, four to a SIMD, were 7 to 10 %
// slower than eight of four: twice the operand reads from LDS and idle attend-only waves.)
//
// Softmax reference.  Scores are kept in base-2 units.  While every score of a
// tile is provably inside [-60, 60] (Cauchy-Schwarz: |q| |k| <= 60) the
// reference maximum stays at the constant 0 and no per-score subtraction or
// maximum is needed; 2^s cannot overflow, underflow or lose relative precision
// there.  A tile that fails the test switches the piece to the usual running
// maximum with rescaling.  Both routes evaluate the same softmax exactly.
//
// Each piece ends with one partial record (O, l, m) per head; merge_mfma_kernel
// combines a user's records in ascending segment order.
#include "stage1_mfma.hpp"

namespace vista {

constexpr float kSafeBound2 = 3600.f;  // (60)^2: |q|^2 |k|^2 below this keeps 2^s in range

__device__ __forceinline__ float dot2_ones(uint32_t pk, float acc) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), ones, acc, false);
}

// One 32-wide operand of a tile: the two k-halves of its bf16 value.
struct Operand {
  Pack8 hi[2];
};

// acc += K Q
__device__ __forceinline__ f32x16 mma_exact_b(const Operand& a, const bf16x8 (&b)[2], f32x16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[0].v, b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[1].v, b[1], acc, 0, 0, 0);
  return acc;
}

// acc += A B
__device__ __forceinline__ f32x16 mma(const Operand& a, const Operand& b, f32x16 acc) {
#pragma unroll
  for (int q = 0; q < 2; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[q].v, b.hi[q].v, acc, 0, 0, 0);
  return acc;
}

// One block of 32 queries against one tile of 32 items.  `general` and `masked`
// are wave-uniform; the MFMAs sit on the common path so the accumulators keep
// one register assignment whichever route a tile takes.
__device__ __forceinline__ void attend_block(const Operand& k, const Operand& v,
                                             const bf16x8 (&q)[2], f32x16& o, float& l, float& m, bool general,
                                             bool masked, int nvl) {
  // nvl = valid items of the tile minus 4 hf: register i is valid iff acc_row0(i) < nvl
  f32x16 s = {0};
  s = mma_exact_b(k, q, s);
  if (general) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (acc_row0(i) >= nvl) s[i] = -INFINITY;
    float tmax = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float mnew = fmaxf(m, tmax);
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    l *= alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] *= alpha;
    m = mnew;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] -= mnew;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(s[i]);
  if (masked) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (acc_row0(i) >= nvl) s[i] = 0.f;
  }
  Operand p;
#pragma unroll
  for (int i = 0; i < 16; i += 2) {
    const uint32_t pk = cvt_pk_bf16(s[i], s[i + 1]);
    l = dot2_ones(pk, l);
    p.hi[i / 8].w[(i % 8) / 2] = pk;
  }
  o = mma(v, p, o);
}

// Shared memory of one workgroup.  WREG: a projecting wave keeps its D x 32 weight operands in
// registers (D / 4 of them) instead of in LDS, which halves the operand reads of a projection: with the
// weights in LDS at D = 256, 32 users and 500 000 items took 242 us instead of 222 at S = 128 and 308
// instead of 296 at S = 256.
template <int D, int HPW, bool WREG>
struct SummarizeLds {
  uint4 xbuf[kXBuf][(D / 8) * 32];    // X tiles: [16-byte chunk][item], filled by direct global->LDS loads
  uint4 kvbuf[kXBuf][HPW][2][2][64];  // projected tiles: [ring slot][head][K|V][half of the 16 registers][lane]
  float knorm[kXBuf][HPW][64];        // squared norm of the scaled key rows (half per lane)
  uint4 wop[WREG ? 1 : HPW * 2 * (D / 16) * 64];   // projection weights as MFMA operands: [head][K|V][k-slice][lane]
};

// Body of one wave; ROLE 0 forms K^T, ROLE 1 forms V, ROLE 2 forms nothing and only attends
// (the further waves of a head when its queries are spread over more than two).  The tile loop is
// software-pipelined: while the wave attends over tile t (VALU-heavy) it also
// issues the projection MFMAs of tile t+1, and the X rows of tiles t+2 / t+3 are
// on their way from HBM (registers) into the LDS buffer tile t has vacated.  One
// LDS-only barrier per tile orders the two double-buffered exchanges.
// ATTN selects what is made of a score: VISTA_ATTN_SOFTMAX as described above, or
// VISTA_ATTN_SILU, the pointwise form SiLU(s) v of App. B: no reference maximum, no
// denominator, no norm test; the key weights then carry -scale*log2(e), so a score leaves the
// MFMA as t = -s log2(e) and SiLU(s) = -ln(2) t / (1 + 2^t); the weight handed to the second
// product is t / (1 + 2^t) and the constant joins the 1/L_b of the merge.
template <int D, int NQB, int HPW, int FW, bool WREG, bool ALLF, int ROLE, int ATTN, bool ORDERED>
__device__ __forceinline__ void summarize_wave(const MfmaSummarizeParams& p, SummarizeLds<D, HPW, WREG>& sm,
                                               int64_t g, int h, int hl, int qblock, int64_t seg_begin,
                                               int64_t seg_end) {
  constexpr bool PROJ = ROLE < 2;        // this wave projects
  constexpr bool SILU = ATTN == VISTA_ATTN_SILU;
  constexpr int WR = PROJ ? ROLE : 0;    // its slot in the weight and K/V buffers (unused otherwise)
  constexpr int NT = FW * 64;            // threads that move X: the first FW waves
  constexpr int CH = D / 8;              // 16-byte chunks per row
  constexpr int KS = D / 16;             // k-slices of the projection
  constexpr int CPT = kTile * CH / NT;   // X chunks each of them moves per tile
  static_assert(kTile * CH % NT == 0, "tile must split evenly over the fetching waves");
  constexpr int KPB = (KS + NQB - 1) / NQB;   // projection k-slices issued per query block

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int hf = lane >> 5;
  const int l32 = lane & 31;

  // Projection weights of this wave's head as MFMA operands, in registers or parked in LDS
  // (each wave reads back only what it wrote).  Element j of slice ks is
  // W[16 ks + 8 hf + j][32 h + l32]; the key weights carry scale*log2(e), so the
  // scores leave the MFMA in base-2 units.
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
        const float c = ROLE ? 1.f : p.c;
#pragma unroll
        for (int b = 0; b < KS / 2; ++b) {
          f32x16 t = {0};
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wraw[b][0].v, sel[0].v, t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wraw[b][1].v, sel[1].v, t, 0, 0, 0);
#pragma unroll
          for (int q = 0; q < 2; ++q)
            keep_weights(2 * b + q,
                         make_uint4(cvt_pk_bf16(t[8 * q] * c, t[8 * q + 1] * c), cvt_pk_bf16(t[8 * q + 2] * c, t[8 * q + 3] * c),
                                    cvt_pk_bf16(t[8 * q + 4] * c, t[8 * q + 5] * c), cvt_pk_bf16(t[8 * q + 6] * c, t[8 * q + 7] * c)));
        }
      } else {
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks) {
          Pack8 t;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint16_t w = W[(16 * ks + 8 * hf + j) * D + 32 * h + l32];
            t.h[j] = ROLE ? w : f32_to_bf16_bits(__uint_as_float(uint32_t(w) << 16) * p.c);
          }
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

  const int qbase = qblock * 32;         // first query of this wave
  bf16x8 qop[NQB][2];
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
  auto settle_queries = [&]() __attribute__((always_inline)) {
    if constexpr (!SILU) {
      float worst = 0.f;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        float n2 = 0.f;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          Pack8 t;
          t.v = qop[qb][part];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            float f = __uint_as_float(uint32_t(t.h[j]) << 16);
            n2 = fmaf(f, f, n2);
          }
        }
        n2 += __shfl_xor(n2, 32, 64);
        worst = fmaxf(worst, n2);
      }
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) worst = fmaxf(worst, __shfl_xor(worst, off, 64));
      qmax2 = worst;
    }
  };

  // ---- the segment as one stream of tiles (TileCursor: scalar state, offsets read through
  // uniform loads).  `ca` names the tile being attended over, `cf` runs three tiles ahead
  // and names the tile whose rows are requested from HBM.
  using Cursor = TileCursor;
  auto cursor_init = [&](Cursor& c) __attribute__((always_inline)) {
    c.init(p.offsets, p.B, find_user_wave(p.offsets, p.B, seg_begin), seg_begin, seg_end);
  };
  auto cursor_advance = [&](Cursor& c) __attribute__((always_inline)) { c.advance(p.offsets, p.B, seg_end); };

  f32x16 o[NQB];
  float l[NQB], m[NQB];
  // plain tiles keep their share of the denominators in lacc (register qb % 4 of either accumulator);
  // the general route folds it into l first
  constexpr int NLA = (NQB + 3) / 4;     // pairs of accumulators: one register of each per query block
  constexpr int NLR = NQB < 4 ? NQB : 4;
  f32x4 lacc[NLA][2];
  uint2 onesrow[NLR];
#pragma unroll
  for (int r = 0; r < NLR; ++r) {
    const uint32_t w = (lane & 3) == r ? 0x3F803F80u : 0u;
    onesrow[r] = make_uint2(w, w);
  }
  int mode = 0;  // 0 fresh piece, 1 constant reference 0, 2 running maximum
  auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[qb][i] = 0.f;
      l[qb] = 0.f;
      m[qb] = 0.f;
    }
#pragma unroll
    for (int a = 0; a < NLA; ++a) lacc[a][0] = lacc[a][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    mode = 0;
  };

  // HBM -> LDS movement of X without a stop in registers (global_load_lds, 16 bytes
  // per lane: lane i of a wave lands at the wave's LDS base + 16 i).  Tile t lives in
  // xbuf[t % 3]; the rows of tile t+3 are requested at the top of tile t into the
  // buffer tile t has vacated and must have landed by the end of tile t+1, so a
  // load has two tile periods.  Rows past the piece are clamped to its last row.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto fetch_rows = [&](const char* base, int last, int xb) __attribute__((always_inline)) {   // last: last valid row
    if (!ALLF && wave >= FW) return;
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
  // hand the projected tile to the partner waves: bf16 operand halves (+ key norms)
  auto publish = [&](int buf, const f32x16& acc) __attribute__((always_inline)) {
    if constexpr (PROJ) {
      Operand r;
      float n2 = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const uint32_t pk = cvt_pk_bf16(acc[i], acc[i + 1]);
        if (ROLE == 0 && !SILU) n2 = dot2_self(pk, n2);
        r.hi[i / 8].w[(i % 8) / 2] = pk;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) sm.kvbuf[buf][hl][WR][q][lane] = r.hi[q].u;
      if (ROLE == 0 && !SILU) sm.knorm[buf][hl][lane] = n2;
    }
  };
  auto unsafe_tile = [&](float kn2) __attribute__((always_inline)) {
    if constexpr (SILU) return false;
    return __builtin_amdgcn_ballot_w64(kn2 * qmax2 > kSafeBound2) != 0;
  };

  // everything the workgroup starts from is requested before any of it is waited for
  request_weights();
  if (p.q_user_stride == 0) request_queries(0);
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
    for (int q = 0; q < 2; ++q) r.hi[q].u = sm.kvbuf[i1][hl][which][q][lane];
  };
  auto read_k = [&](int i1) __attribute__((always_inline)) {
    read_operand(kk, i1, 0);
    if constexpr (!SILU) kn2 = sm.knorm[i1][hl][lane] + sm.knorm[i1][hl][lane ^ 32];
  };
  auto read_v = [&](int i1) __attribute__((always_inline)) {
    read_operand(vv, i1, 1);
  };
  // slots of tiles t+1 and t+2 in a ring of the X tiles and of the operands, r = tile index mod 3
  struct Slots { int x2, kv1, kv2; };
  auto slots = [&](int r) __attribute__((always_inline)) {
    const int i1 = r == kXBuf - 1 ? 0 : r + 1, i2 = i1 == kXBuf - 1 ? 0 : i1 + 1;
    return Slots{i2, i1, i2};
  };
  auto free_tile = [&](int r) __attribute__((always_inline)) {
    const Slots at = slots(r);
    f32x16 acc = {0};
    // scores run one query block ahead of the exponentials that consume them
    f32x16 nx = {0};
    nx = mma_exact_b(kk, qop[0], nx);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      if (qb == NQB - 1) read_k(at.kv1);     // the last scores of this tile are already issued
      const f32x16 sc = nx;
      if (qb + 1 < NQB) {
        const f32x16 z = {0};
        nx = mma_exact_b(kk, qop[qb + 1], z);
      }
      if (qb * KPB < KS) project(at.x2, qb * KPB, qb * KPB + KPB < KS ? qb * KPB + KPB : KS, acc);
      Operand pp;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        float ea = __builtin_amdgcn_exp2f(sc[i]), eb = __builtin_amdgcn_exp2f(sc[i + 1]);
        if constexpr (SILU) {
          ea = sc[i] * __builtin_amdgcn_rcpf(1.f + ea);
          eb = sc[i + 1] * __builtin_amdgcn_rcpf(1.f + eb);
        }
        pp.hi[i / 8].w[(i % 8) / 2] = cvt_pk_bf16(ea, eb);
      }
      // The denominator on the matrix core: a 4x4x4 product (16 blocks, one per four lanes)
      // whose A block has ones in row qb % 4 adds a lane's own four packed weights into register
      // qb % 4 of that lane -- the lane-local partial sum a chain of adds would form, taken over
      // the bf16 weights the numerator uses.  It issues like one plain vector instruction for four
      // weights; two accumulators take turns so that consecutive products do not wait for each
      // other.
      if constexpr (!SILU) {
        const i16x4 sel = __builtin_bit_cast(i16x4, onesrow[qb % 4]);
#pragma unroll
        for (int part = 0; part < 4; ++part) {
          const Pack8& src = pp.hi[part / 2];
          const uint2 pw = make_uint2(src.w[2 * (part & 1)], src.w[2 * (part & 1) + 1]);
          f32x4& a = lacc[qb / 4][part & 1];
          a = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(sel, __builtin_bit_cast(i16x4, pw), a, 0, 0, 0);
        }
      }
      o[qb] = mma(vv, pp, o[qb]);
    }
    read_v(at.kv1);
    publish(at.kv2, acc);
  };
  // The same in an order of its own (pin).  A product keeps the matrix pipe for 32 clocks and the issue port for some 11, and
  // exponentials run beside it (four products and sixteen v_exp_f32 take what the exponentials do alone); products in a row wait for the
  // pipe.  Left to itself the compiler ends a tile in runs of ten and more of them.  So the second product of a block and its denominators
  // wait for the exponentials of the next block, and a pair is packed a few instructions behind its exponentials.
  static_assert(!ORDERED || !SILU, "ordered_tile forms softmax weights");
  auto ordered_tile = [&](int r) __attribute__((always_inline)) {
    const Slots at = slots(r);
    f32x16 acc = {0};
    int ks = 0;
    Pack8 xr;
    if constexpr (PROJ) xr.u = sm.xbuf[at.x2][hf * 32 + l32];
    auto proj = [&](int n) __attribute__((always_inline)) {      // n slices of the projection
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
          if (ks < KS) xr.u = sm.xbuf[at.x2][(2 * ks + hf) * 32 + l32];
        }
      }
    };
    Pack8 before[2];          // packed weights of the block before
    auto small = [&](int qb, int part) __attribute__((always_inline)) {
      const i16x4 sel = __builtin_bit_cast(i16x4, onesrow[qb % 4]);
      const Pack8& src = before[part / 2];
      const uint2 pw = make_uint2(src.w[2 * (part & 1)], src.w[2 * (part & 1) + 1]);
      f32x4& a = lacc[qb / 4][part & 1];
      a = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(sel, __builtin_bit_cast(i16x4, pw), a, 0, 0, 0);
      pin(a);
    };
    auto second = [&](int qb, int half) __attribute__((always_inline)) {
      o[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv.hi[half].v, before[half].v, o[qb], 0, 0, 0);
      pin(o[qb]);
    };
    const f32x16 zero = {0};
    f32x16 nx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk.hi[0].v, qop[0][0], zero, 0, 0, 0);
    nx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk.hi[1].v, qop[0][1], nx, 0, 0, 0);
    pin(nx);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const f32x16 sc = nx;
      float ev[16];
      Pack8 cur[2];
      auto E = [&](int i) __attribute__((always_inline)) { ev[i] = __builtin_amdgcn_exp2f(sc[i]); pin(ev[i]); };
      auto P = [&](int i) __attribute__((always_inline)) {
        uint32_t t = cvt_pk_bf16(ev[i], ev[i + 1]);
        pin(t);
        cur[i / 8].w[(i % 8) / 2] = t;
      };
      const bool more = qb + 1 < NQB;
      auto next = [&](int half) __attribute__((always_inline)) {
        if (!more) return;
        nx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk.hi[half].v, qop[(qb + 1) % NQB][half], half ? nx : zero, 0, 0, 0);
        pin(nx);
      };
      auto share = [&](int i) __attribute__((always_inline)) { proj((i + 1) * KPB / 4 - i * KPB / 4); };
      next(0);
      E(0); E(1); E(2);
      if (qb > 0) { small(qb - 1, 0); second(qb - 1, 0); }
      P(0); E(3); E(4); E(5);
      if (qb > 0) small(qb - 1, 1);
      share(0);
      P(2); E(6); E(7); P(4);
      share(1);
      next(1);
      if (!more) read_k(at.kv1);
      E(8); P(6); E(9); E(10);
      if (qb > 0) { small(qb - 1, 2); second(qb - 1, 1); }
      P(8); E(11); E(12);
      if (qb > 0) small(qb - 1, 3);
      share(2);
      P(10); E(13); E(14); P(12); E(15);
      share(3);
      P(14);
      before[0] = cur[0];
      before[1] = cur[1];
    }
    second(NQB - 1, 0);
    small(NQB - 1, 0); small(NQB - 1, 1);
    second(NQB - 1, 1);
    small(NQB - 1, 2); small(NQB - 1, 3);
    read_v(at.kv1);
    publish(at.kv2, acc);
  };
  auto fast_tile = [&](int r) __attribute__((always_inline)) {
    if constexpr (ORDERED) ordered_tile(r); else free_tile(r);
  };

  // Any tile: ragged tail, scores beyond the bound, last tile of the segment.
  auto slow_tile = [&](int r, int nvalid, bool unsafe) __attribute__((always_inline)) {
    const Slots at = slots(r);
    const int nvl = nvalid - 4 * hf;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      l[qb] += lacc[qb / 4][0][qb % 4] + lacc[qb / 4][1][qb % 4];
      lacc[qb / 4][0][qb % 4] = lacc[qb / 4][1][qb % 4] = 0.f;
    }
    if constexpr (SILU) {
      // pointwise form: scores, weights (rows past the piece's end get weight 0), second product
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        f32x16 sc = {0};
        sc = mma_exact_b(kk, qop[qb], sc);
        Operand pp;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          float wa = sc[i] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(sc[i]));
          float wb = sc[i + 1] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(sc[i + 1]));
          if (acc_row0(i) >= nvl) wa = 0.f;
          if (acc_row0(i + 1) >= nvl) wb = 0.f;
          pp.hi[i / 8].w[(i % 8) / 2] = cvt_pk_bf16(wa, wb);
        }
        o[qb] = mma(vv, pp, o[qb]);
      }
      mode = 1;
    } else {
    const bool general = mode == 2 || unsafe;
    if (mode != 2) {   // the reference so far: nothing (fresh piece) or the constant 0
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) m[qb] = (general && mode == 0) ? kLowest : 0.f;
    }
    mode = general ? 2 : 1;
    const bool masked = nvalid < kTile;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
      attend_block(kk, vv, qop[qb], o[qb], l[qb], m[qb], general, masked, nvl);
    }
    read_k(at.kv1);
    read_v(at.kv1);
    // the tile two ahead (past the end of the segment: a repeat of its last tile, never used)
    f32x16 acc = {0};
    project(at.x2, 0, KS, acc);
    publish(at.kv2, acc);
  };

  // partial record of a finished piece: slot = segment + user
  auto write_partial = [&](int user) __attribute__((always_inline)) {
    const int64_t slot = g + user;
    char* rec = reinterpret_cast<char*>(p.partials + ((slot * p.H + h) * p.nqb + (qbase / 32)) * kRecFloats);
    const uint32_t lane_off = uint32_t(lane) * 16;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      if (qbase / 32 + qb >= p.nqb) break;               // a block past the last query has no record
      char* r = rec + size_t(qb) * kRecFloats * 4;       // scalar
#pragma unroll
      for (int i = 0; i < 16; i += 4)
        *reinterpret_cast<float4*>(r + i * 256 + lane_off) = make_float4(o[qb][i], o[qb][i + 1], o[qb][i + 2], o[qb][i + 3]);
      *reinterpret_cast<float2*>(r + kRecSums * 4 + lane_off / 2) =
          make_float2(l[qb] + __shfl_xor(l[qb], 32, 64), (mode == 2) ? m[qb] : 0.f);
    }
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
  // (kvbuf).  While tile t is attended over, tile t+2 is projected and published, the
  // operands of tile t+1 move into registers, the rows of tile t+3 land and those of tile
  // t+4 are requested into the slot whose rows (tile t+1) were projected one tile ago.
  // ---- prologue: tiles 0, 1, 2 requested; 0 and 1 landed, projected and published
  fetch(cf, 0);
  cursor_advance(cf);
  fetch(cf, 1);
  cursor_advance(cf);
  fetch(cf, 2);
  cursor_advance(cf);
  if (p.q_user_stride != 0) request_queries(ca.user);
  settle_weights();
  settle_queries();
  wait_vm(Int<CPT>{});
  lds_barrier();
  {
    f32x16 acc = {0};
    project(0, 0, KS, acc);
    publish(0, acc);
    f32x16 acc1 = {0};
    project(1, 0, KS, acc1);
    publish(1, acc1);
  }
  lds_barrier();              // slot 0's rows are projected by everyone, its operands are visible
  fetch(cf, 0);               // tile 3
  cursor_advance(cf);
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
    cursor_advance(cf);
  };
  // Start of a tile: the barrier, then the request for tile t+4.
  auto begin_tile = [&]() __attribute__((always_inline)) {
    lds_barrier();
    fetch(cf, r == kXBuf - 1 ? 0 : r + 1);
  };
  // whether the tile whose operands are in registers is a plain one
  bool unsafe = unsafe_tile(kn2);
  auto is_plain = [&]() __attribute__((always_inline)) {
    if constexpr (SILU) return ca.tiles_left != 1;
    return !(ca.tiles_left == 1 || mode == 2 || unsafe);
  };
  bool plain = is_plain();
  for (;;) {
    // Plain tiles while the tile being requested is a full one of the same piece: no cursor in the loop.  Its
    // branches and state moves are on every wave between two barriers; without this loop 8 users of a
    // million items take 1720 us instead of 1652, two layers at d = 256 27.4 ms instead of 24.0.
    if (plain) {
      const int run = cf.straight(ca);
      const char* base = reinterpret_cast<const char*>(p.X) + cf.row * (D * 2);
      int n = 0;
      while (n < run && plain) {
        lds_barrier();
        fetch_rows(base, kTile - 1, r == kXBuf - 1 ? 0 : r + 1);
        base += kTile * D * 2;
        mode = 1;
        fast_tile(r);
        if (drain) wait_vm(Int<0>{}); else wait_vm(Int<CPT>{});
        drain = false;
        ++n;
        r = r == kXBuf - 1 ? 0 : r + 1;
        unsafe = unsafe_tile(kn2);
        plain = !unsafe;
      }
      ca.skip(n);
      cf.skip(n);
      plain = is_plain();
    }
    while (__builtin_expect(plain, 1)) {
      begin_tile();
      mode = 1;
      fast_tile(r);
      end_of_tile();
      --ca.tiles_left;
      ca.row += kTile;
      r = r == kXBuf - 1 ? 0 : r + 1;
      unsafe = unsafe_tile(kn2);
      plain = is_plain();
    }
    begin_tile();
    const bool last_in_piece = ca.tiles_left == 1;
    const int nvalid = last_in_piece ? ca.tail : kTile;
    slow_tile(r, nvalid, unsafe);
    end_of_tile();
    const int done_user = ca.user;
    cursor_advance(ca);
    if (last_in_piece) {
      write_partial(done_user);
      reset_state();
      if (p.q_user_stride != 0 && ca.valid) {
        request_queries(ca.user);
        settle_queries();
      }
      drain = true;
    }
    r = r == kXBuf - 1 ? 0 : r + 1;
    if (!ca.valid) break;
    unsafe = unsafe_tile(kn2);
    plain = is_plain();
  }
}

// MAXT: largest workgroup of the instantiation (it bounds the registers of a wave).  The first FW waves
// fetch X (ALLF: that is every wave).
// NQB query blocks to a projecting wave, NQA to one that only attends.  OCC: waves on a SIMD that the registers have to leave
// room for, as far as the workgroups that fit the LDS can fill them (the two-wave workgroups of D = 256, S = 64 cannot, and take
// 295 registers).
template <int D, int NQB, int NQA, int HPW, int FW, bool WREG, int MAXT, int ATTN, int OCC, bool ORDERED>
__global__ __launch_bounds__(MAXT, OCC) void summarize_mfma_kernel(MfmaSummarizeParams p) {
  __shared__ SummarizeLds<D, HPW, WREG> sm;

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
  // The seeds' own keys and values, which the merge needs: units of them go round the workgroups' first waves, then their
  // second and so on.  A kernel in front of this one was a launch and 6 us of latency: 500 003 items, SiLU, S = 128 106.3 ->
  // 100.5 us a call without it; 7000 items, d = 128, S = 256 33.8 -> 24.9; 100 users with queries of their own, 60 000 items,
  // d = 256, S = 512 255 -> 243.  They come before the history because what they need would have to be kept through it
  // otherwise, and every call would pay (behind it, calls without the self term: SiLU, d = 128, S = 256, 300 users, 9557
  // items 103.4 us instead of 97.9; S = 64, 110 users, 117 964 items 36.3 instead of 35.7).  Marked as unlikely, they stand behind
  // the streaming code instead of in front of it (softmax, S = 128, 64 users, 1 000 000 items 157.2 -> 155.3 us, others the same).
  if (__builtin_expect(p.Ks != nullptr, 0)) {
    const int64_t groups = (p.N + p.seg - 1) / p.seg * p.nhg, units = (p.self_rows + 31) / 32 * (D / 32);
    for (int64_t u = int64_t(wave) * groups + g * p.nhg + hg; u < units; u += groups * (blockDim.x >> 6))
      self_kv_unit(p.Q, p.Wk, p.Wv, p.Ks, p.Vs, p.self_rows, D, u);
  }
  // All roles run the same sequence of barriers; only the MFMA operand order differs.
  if (slot == 0)
    summarize_wave<D, NQB, HPW, FW, WREG, MAXT == 64 * FW, 0, ATTN, ORDERED>(p, sm, g, h, hl, 0, seg_begin, seg_end);
  else if (slot == 1)
    summarize_wave<D, NQB, HPW, FW, WREG, MAXT == 64 * FW, 1, ATTN, ORDERED>(p, sm, g, h, hl, NQB, seg_begin, seg_end);
  else if constexpr (MAXT != HPW * 128)      // (two waves per head: there is no third slot)
    summarize_wave<D, NQA, HPW, FW, WREG, MAXT == 64 * FW, 2, ATTN, ORDERED>(p, sm, g, h, hl, 2 * NQB + (slot - 2) * NQA, seg_begin, seg_end);
}

// Merge of a user's partial records in a fixed order, so the result is bitwise reproducible.
// Softmax form: with m the running maximum of the m_c,
// out = sum_c 2^(m_c - m) O_c / sum_c 2^(m_c - m) l_c; the self term (Ks != null) is one more
// record (m = own score, l = 1, O = own value), taken last.  SiLU form: out =
// (-ln 2 sum_c O_c + SiLU(own score) own value) / L_b (the records hold sums of
// t / (1 + 2^t) v with t = -s log2 e).  Four waves per (user, head, query block): wave w owns
// accumulator registers 4w..4w+3, i.e. channels 8w + 4 hf + 0..3.
// RG = 1: the four are one block and walk the user's records in ascending order.
// RG = 4: each of the four is a block of four waves; wave r takes the r-th run of the records,
// ascending, and the runs' sums are combined in ascending order.  (No codec: its scale spans the four.)
// Columns past the last query are computed and not stored.
template <bool SILU, int RG>
__global__ __launch_bounds__(256) void merge_mfma_kernel(const float* __restrict__ partials,
                                                              const int64_t* __restrict__ offsets, int B, int S, int d,
                                                              int H, int seg, int64_t N, int64_t G,
                                                              uint16_t* __restrict__ out, int* status,
                                                              int check_offsets, const uint16_t* __restrict__ Q,
                                                              int64_t q_user_stride, const float* __restrict__ Ks,
                                                              const float* __restrict__ Vs, float scale,
                                                              float* __restrict__ out_scales) {
  __shared__ float amax_part[8][32];
  __shared__ float group[RG > 1 ? RG - 1 : 1][6][64];       // (m, l, o0..o3) of the later groups
  const int nqb = (S + 31) / 32;
  const int blk = RG > 1 ? blockIdx.x >> 2 : blockIdx.x;
  const int qb = blk % nqb, h = (blk / nqb) % H, b = blk / (nqb * H);
  // The first block publishes the status word: the offsets are checked here unless the host has.
  if (blockIdx.x == 0) {
    int bad = 0;
    if (check_offsets)
      for (int u = threadIdx.x; u <= B; u += blockDim.x) {
        const int64_t o = offsets[u];
        bad |= (u == 0 && o != 0) || (u == B && o != N) || (u < B && offsets[u + 1] < o);
      }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) *status = bad ? int(VISTA_ERR_OFFSETS) : int(VISTA_OK);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w = RG > 1 ? blockIdx.x & 3 : wave, rg = RG > 1 ? wave : 0;
  const int hf = lane >> 5, l32 = lane & 31;
  const bool live = rg == 0 && qb * 32 + l32 < S;           // this lane stores
  const int64_t begin = offsets[b], end = offsets[b + 1];
  uint16_t* dst = out + (int64_t(b) * S + qb * 32 + l32) * d + 32 * h + 8 * w + 4 * hf;
  // cache codec (out_scales != null): `out` holds int8 codes, one scale per (token, head)
  int8_t* dst8 = reinterpret_cast<int8_t*>(out) + (int64_t(b) * S + qb * 32 + l32) * d + 32 * h + 8 * w + 4 * hf;
  if (end <= begin) {
    if (!live) return;
    if (out_scales) {
      *reinterpret_cast<uint32_t*>(dst8) = 0u;
      if (w == 0 && hf == 0) out_scales[(int64_t(b) * S + qb * 32 + l32) * H + h] = 0.f;
    } else {
      *reinterpret_cast<uint2*>(dst) = make_uint2(0u, 0u);
    }
    return;
  }
  int64_t g0 = segment_of(begin, seg), g1 = segment_of(end - 1, seg);
  if (g0 < 0) g0 = 0;
  if (g1 > G - 1) g1 = G - 1;
  // the query's own key and value (self term): score in the units of the records' m
  float s_self = 0.f, vs[4] = {0.f, 0.f, 0.f, 0.f};
  if (Ks) {
    const int i = qb * 32 + l32 < S ? qb * 32 + l32 : S - 1;
    const uint16_t* q = Q + q_user_stride * b + int64_t(i) * d + 32 * h;
    const int64_t srow = (q_user_stride ? int64_t(b) * S : 0) + i;
    const float* ks = Ks + srow * d + 32 * h;
#pragma unroll 8
    for (int c = 0; c < 32; ++c) s_self = fmaf(__uint_as_float(uint32_t(q[c]) << 16), ks[c], s_self);
    s_self *= scale;
#pragma unroll
    for (int r = 0; r < 4; ++r) vs[r] = Vs[srow * d + 32 * h + 8 * w + 4 * hf + r];
  }
  // One pass with a running maximum (rescaled once a batch); the loads of a batch are all issued before the first is
  // used, so that a long user is not a chain of dependent round trips.  (Sixteen: jagged batch 2 % slower a call.)
  constexpr int kBatch = 8;
  float m = kLowest, l = 0.f, o0 = 0.f, o1 = 0.f, o2 = 0.f, o3 = 0.f;
  const int64_t run = (g1 - g0 + RG) / RG;                  // records per group
  const int64_t r0 = g0 + rg * run;
  if (g1 > r0 + run - 1) g1 = r0 + run - 1;
  const int64_t stride = int64_t(H) * nqb * kRecFloats;     // from one segment's record to the next one's
  for (int64_t g = r0; g <= g1; g += kBatch) {
    const int left = int(g1 - g < kBatch ? g1 - g : kBatch);           // records behind the first
    const float* r = partials + (((g + b) * H + h) * nqb + qb) * kRecFloats;
    float4 o[kBatch];
    float2 lm[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float* at = r + (u <= left ? u : left) * stride;           // past the last: the last again, at no weight
      lm[u] = *reinterpret_cast<const float2*>(at + kRecSums + lane * 2);
      o[u] = *reinterpret_cast<const float4*>(at + w * 256 + lane * 4);
    }
    __builtin_amdgcn_sched_barrier(0);
    float wgt[kBatch];
    if (SILU) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) wgt[u] = u <= left ? 1.f : 0.f;
    } else {
      float mn = m;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) mn = u <= left ? fmaxf(mn, lm[u].y) : mn;
      const float keep = exp2f(m - mn);                     // 0 before the first record (m lowest), 1 while the maximum stands
      m = mn;
      l *= keep; o0 *= keep; o1 *= keep; o2 *= keep; o3 *= keep;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) wgt[u] = u <= left ? exp2f(lm[u].y - mn) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {     // ascending segment order
      if (u > left) o[u] = make_float4(0.f, 0.f, 0.f, 0.f);   // (they may be infinite: a weight of 0 is not enough)
      if (!SILU) l = fmaf(lm[u].x, wgt[u], l);
      o0 = fmaf(o[u].x, wgt[u], o0);
      o1 = fmaf(o[u].y, wgt[u], o1);
      o2 = fmaf(o[u].z, wgt[u], o2);
      o3 = fmaf(o[u].w, wgt[u], o3);
    }
  }
  if (RG > 1) {
    if (rg > 0) {
      float* x = &group[rg - 1][0][lane];
      x[0] = m; x[64] = l; x[128] = o0; x[192] = o1; x[256] = o2; x[320] = o3;
    }
    __syncthreads();
    if (rg > 0) return;
#pragma unroll
    for (int r = 0; r < RG - 1; ++r) {
      const float* x = &group[r][0][lane];
      float keep = 1.f, wgt = 1.f;
      if (!SILU) {
        const float mn = fmaxf(m, x[0]);
        keep = exp2f(m - mn);
        wgt = exp2f(x[0] - mn);             // 0 for an empty group (m lowest)
        m = mn;
      }
      l = fmaf(x[64], wgt, l * keep);
      o0 = fmaf(x[128], wgt, o0 * keep);
      o1 = fmaf(x[192], wgt, o1 * keep);
      o2 = fmaf(x[256], wgt, o2 * keep);
      o3 = fmaf(x[320], wgt, o3 * keep);
    }
  }
  float inv;
  if (SILU) {
    inv = 1.f / float(end - begin);
    const float wself = Ks ? s_self / (1.f + expf(-s_self)) : 0.f;
    o0 = fmaf(o0, -0.69314718056f, wself * vs[0]);
    o1 = fmaf(o1, -0.69314718056f, wself * vs[1]);
    o2 = fmaf(o2, -0.69314718056f, wself * vs[2]);
    o3 = fmaf(o3, -0.69314718056f, wself * vs[3]);
  } else {
    if (Ks) {
      const float mn = fmaxf(m, s_self);
      const float keep = exp2f(m - mn), wgt = exp2f(s_self - mn);
      l = fmaf(l, keep, wgt);
      o0 = fmaf(vs[0], wgt, o0 * keep);
      o1 = fmaf(vs[1], wgt, o1 * keep);
      o2 = fmaf(vs[2], wgt, o2 * keep);
      o3 = fmaf(vs[3], wgt, o3 * keep);
    }
    inv = 1.f / l;
  }
  if (RG == 1 && out_scales) {
    // Sec. 3.1's quantisation, fused: the head's 32 channels of a token sit in this block's
    // eight (wave, half) groups of four; their largest magnitude goes through LDS.
    const float y0 = o0 * inv, y1 = o1 * inv, y2 = o2 * inv, y3 = o3 * inv;
    amax_part[2 * w + hf][l32] = fmaxf(fmaxf(fabsf(y0), fabsf(y1)), fmaxf(fabsf(y2), fabsf(y3)));
    __syncthreads();
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) amax = fmaxf(amax, amax_part[k][l32]);
    const float q = amax > 0.f ? 127.f / amax : 0.f;
    auto code = [&](float y) __attribute__((always_inline)) {
      return uint32_t(int(fminf(fmaxf(rintf(y * q), -127.f), 127.f))) & 0xFFu;
    };
    if (!live) return;
    *reinterpret_cast<uint32_t*>(dst8) = code(y0) | (code(y1) << 8) | (code(y2) << 16) | (code(y3) << 24);
    if (w == 0 && hf == 0) out_scales[(int64_t(b) * S + qb * 32 + l32) * H + h] = amax > 0.f ? amax / 127.f : 0.f;
    return;
  }
  if (!live) return;
  uint2 pk;
  pk.x = uint32_t(f32_to_bf16_bits(o0 * inv)) | (uint32_t(f32_to_bf16_bits(o1 * inv)) << 16);
  pk.y = uint32_t(f32_to_bf16_bits(o2 * inv)) | (uint32_t(f32_to_bf16_bits(o3 * inv)) << 16);
  *reinterpret_cast<uint2*>(dst) = pk;
}

// The same as a kernel of its own, for the paths whose main kernel does not form them.  It is a few launches' worth of
// latency: one thread per output walking 2-byte loads took 33 us for 128 seeds of width 128, this takes 6.
__global__ __launch_bounds__(256) void self_kv_mfma_kernel(const uint16_t* __restrict__ Q,
                                                           const uint16_t* __restrict__ Wk,
                                                           const uint16_t* __restrict__ Wv, float* __restrict__ Ks,
                                                           float* __restrict__ Vs, int64_t rows, int d) {
  self_kv_unit(Q, Wk, Wv, Ks, Vs, rows, d, int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6));
}

// ------------------------------------------------------------------ host side

// 16-byte loads of seeds and weights; other alignments and types keep one thread per output.
bool mfma_self_kv_supported(const vista_summarize_desc& d, const void* Q, const void* Wk, const void* Wv) {
  return d.dtype == VISTA_BF16 && d.d % 32 == 0 &&
         ((reinterpret_cast<uintptr_t>(Q) | reinterpret_cast<uintptr_t>(Wk) | reinterpret_cast<uintptr_t>(Wv)) & 15) == 0;
}

hipError_t mfma_self_kv(const vista_summarize_desc& d, const void* Q, const void* Wk, const void* Wv, float* Ks,
                        float* Vs, hipStream_t s) {
  const int64_t rows = d.q_user_stride ? int64_t(d.B) * d.S : d.S;
  const int64_t units = (rows + 31) / 32 * (d.d / 32);
  return launch(self_kv_mfma_kernel, dim3(unsigned((units + 3) / 4)), dim3(256), 0, s, static_cast<const uint16_t*>(Q),
                static_cast<const uint16_t*>(Wk), static_cast<const uint16_t*>(Wv), Ks, Vs, rows, d.d);
}

// The shapes whose K, V and softmax weights are bf16 operands.
bool mfma_summarize_supported(const vista_summarize_desc& d) {
  if (d.dtype != VISTA_BF16 || d.attn == VISTA_ATTN_QLA) return false;
  if (!(d.d == 128 && d.H == 4) && !(d.d == 256 && d.H == 8)) return false;
  return d.S == 64 || d.S == 128 || d.S == 256 || d.S == 512;
}

// The other bf16 softmax shapes of the same head width: any seed count, K, V and weights as split
// operands (split_mfma.hip).
bool mfma_split_supported(const vista_summarize_desc& d) {
  if (d.dtype != VISTA_BF16 || d.attn != VISTA_ATTN_SOFTMAX || mfma_summarize_supported(d)) return false;
  return (d.d == 64 && d.H == 2) || (d.d == 128 && d.H == 4) || (d.d == 256 && d.H == 8);
}

// Short histories go to workgroups of half the heads, so of half the waves.  A tile then takes one wave's time a
// SIMD instead of two, and twice the workgroups find compute units idle; once they are all busy the rows are
// merely fetched twice.  us a call, whole / half workgroups, few users: d = 128, S = 256, 7001 items 26.5 / 20.8,
// 60 000 42.7 / 35.4, 200 000 65.8 / 61.8, 400 000 104 / 106; S = 64, 60 000 23.7 / 21.3, 140 000 30.0 / 29.6, 200 000 35.3 /
// 36.2; S = 128, 100 000 33.9 / 31.4, 200 000 45.5 / 45.5; S = 512, 80 000 52.5 / 50.7, 200 000 92.2 / 95.4.  The SiLU form at
// S = 128 has sixteen waves beyond: 60 000 29.4 / 28.4, 80 000 32.2 / 33.2.  At d = 256 a tile is twice the bytes and four groups of
// heads share the chip as it is: S = 64, 7001 18.2 / 17.9, 15 000 21.4 / 23.1; S = 128, 15 000 24.6 / 22.8, 20 000 25.8 / 26.0; S = 256,
// 15 000 31.4 / 28.8, 25 000 35.4 / 36.0; S = 512, 30 000 53.7 / 51.1, 45 000 62.1 / 62.2; SiLU, S = 128, 13 845 24.1 / 25.5.
// Users count too: a workgroup of half the heads walks twice the items, so twice the users, and at every change of user its one
// wave a SIMD goes through a ragged tile, a record and, with queries of their own, their load with nobody beside it.  Each user
// beyond the first counts as some items, few in the SiLU form, whose ragged tiles cost what full ones do, many where a wave holds six
// blocks of queries.  Lognormal users, whole / half: softmax, d = 256, S = 512, 64 of 24 576 items 74.0 / 84.2, queries of their own
// 84.1 / 99.7; 8 of 31 744 52.3 / 48.2; d = 128, S = 512, 96 of 43 008 with queries of their own 69 / 78; S = 64, 200 of 65 536 30.8 / 33.5,
// SiLU, S = 256, 110 of 22 937 63 / 49.  Up to `few` items any number of users is faster in halves (200 of 2048, d = 256, S = 512
// 205 / 182; own 287 / 260).  Over 6350 calls (1 to 300 users) ten take halves that are 3 to 6 % behind, 154 whole ones.
static int64_t short_limit(const vista_summarize_desc& d) {
  const bool silu = d.attn == VISTA_ATTN_SILU;
  if (d.d == 256) return d.S == 64 ? 8192 : d.S == 512 ? (silu ? 20480 : 32768) : silu ? 12288 : 16384;
  if (silu && d.S == 128) return 65536;
  return d.S == 256 ? 229376 : d.S == 512 ? 98304 : 131072;
}
static bool short_history(const vista_summarize_desc& d, int64_t limit) {
  const bool silu = d.attn == VISTA_ATTN_SILU, own = d.q_user_stride != 0;
  const int64_t few = d.d == 128 ? 12288 : d.S < 256 ? 4096 : 6144;
  int64_t user;
  if (d.d == 256)
    user = d.S == 64 ? 2048 : silu ? 384 : d.S < 512 ? 192 : own ? 3072 : 2048;
  else if (silu)
    user = d.S == 128 ? (own ? 768 : 320) : 128;
  else
    user = d.S == 512 ? (own ? 1024 : 768) : own ? 640 : 384;
  return d.total_items <= few || d.total_items + user * int64_t(d.B - 1) <= limit;
}
static bool short_history(const vista_summarize_desc& d) { return short_history(d, short_limit(d)); }

// The shortest of these go to workgroups of one head with half the query blocks a wave (or, of one block, half the waves), in
// segments that make one workgroup a compute unit: a tile takes half the time again, and a wave's code, which such a call walks
// cold, is half as long.  Beyond, rows are fetched and users are changed once more for nothing, the sooner the more users there are;
// with some way to the limit above, where halves are no better than whole ones.  us a call, halves / one head: d = 128, S = 256, one
// user of 2000 items 16.6 / 13.9, of 7001 20.3 / 17.5, of 30 000 30.0 / 24.5, of 64 000 37 / 37; 64 users of 8000 in all 28.5 / 24.2, of 48 000
// 36.3 / 35.6; S = 128, SiLU, one user of 15 000 19.5 / 15.6, 300 of 20 000 4 to 9 % faster, of 32 000 8 to 11 % slower; S = 64, 64 users of
// 12 000 3 % faster, of 32 000 11 % slower; S = 512, 30 users of 60 000 52.4 / 47.1; d = 256, S = 512, one user of 7001 34.5 / 30.8, 8 of 8000 19 %
// faster, 300 of 20 000 6 % slower.  (At d = 256 up to S = 128 a half already is one head of one block a wave.)
static bool one_head_history(const vista_summarize_desc& d) {
  const bool silu = d.attn == VISTA_ATTN_SILU;
  if ((d.d == 256 && d.S < 256) || !short_history(d, short_limit(d) / 8 * 7)) return false;
  if (d.d == 256 || d.S == 512) return true;
  const double few = d.S == 64 ? 16384 : d.S == 128 ? (silu ? 53248 : 49152) : silu ? 40960 : 57344;
  return double(d.total_items) <= few * (0.4 + 0.6 * 32.0 / (double(d.B) + 31.0));
}

// How the heads of a segment are shared out.
enum class Heads { kWhole, kHalf, kOne };

// Head groups (workgroups per segment) and workgroups resident on a compute unit, as launched below.
static int head_groups(const vista_summarize_desc& d, Heads heads) {
  const int nqb = (d.S + 31) / 32;
  if (heads == Heads::kOne) return d.H;
  if (mfma_summarize_supported(d))
    return (d.d == 256 ? 4 : nqb > 8 ? 2 : 1) * (heads == Heads::kHalf ? 2 : 1);
  if (d.d == 256) return 8;
  return nqb > 8 ? d.H : d.H / 2;
}
static int resident_workgroups(const vista_summarize_desc& d, Heads heads) {
  // One head, split operands: another one shares the compute unit where its segment would be longer than 512 items, a third (d = 64, waves
  // of 168 registers) than 1600; eight waves have it to themselves.  us a call with one / two / three: d = 64, S = 100, 48 users of 300 007 items 71.9 / 57.3
  // / 55.1, of 100 000 38.0 / 34.6 / 34.4, of 60 000 31.0 / 29.8 / 31.1; S = 200, 180 000 64.3 / 67.2 / 74.0; d = 128, S = 100, 120 000 70.2 / 55.9 / 66.7,
  // 60 000 47.1 / 40.3 / 46.9; S = 250, 30 000 36.8 / 44.7 / 52.1.
  if (heads == Heads::kOne && mfma_split_supported(d)) {
    const int64_t alone = d.total_items * d.H / 256;
    return d.S > 128 || alone <= 512 ? 1 : d.d == 64 && alone > 1600 ? 3 : 2;
  }
  // Two fit, but two cold starts on a compute unit have to pay: a segment of 768 items for one does it with the split
  // operands (d = 64, S = 40: 60 000 items in 23.8 us with one, 24.5 with two, 100 000 in 26.4 and 28.0, 200 000 in 37.2 and 33.3), 2048 at d = 256.
  if (mfma_split_supported(d)) return d.d != 256 && d.S <= 128 && d.total_items > 768 * 256 / head_groups(d, Heads::kWhole) ? 2 : 1;
  return d.d == 256 && d.S == 64 && d.total_items > 131072 ? 2 : 1;
}

// Split operands: one head a workgroup and one block a wave, three to eight waves, beside two heads and two blocks.  us a call, two
// heads / one: d = 64, S = 100, 30 users of 30 000 items 25.4 / 23.4, of 150 000 41.8 / 40.5, 48 of 300 007 55.3 to 55.8 / 55.0 to 55.9, of 450 000 70.6 / 71.6, of 600 000
// 85.8 / 87.6; S = 200, 30 of 60 000 40.0 / 35.7, of 200 000 65.4 / 65.2, of 300 007 83.1 / 89.6; d = 128, S = 100, 30 of 60 000 43.1 / 41.4, of
// 120 000 55.4 / 55.9, of 200 000 73.8 / 77.7; S = 205, one of 53 749 45.4 / 40.7; S = 250, one of 15 000 30.4 / 24.6, of 55 300 46.6 / 43.6, 30 of 30 000
// 40.0 / 37.4, of 55 000 55.3 / 50.7, of 60 000 51.1 / 53.0.  One and two blocks in all
// make two waves, which is worth it in short histories: d = 64, S = 40, one of 15 000 17.7 / 16.9, 30 of 30 000 20.3 / 21.8; d = 128, S = 40, 30 of
// 7001 24.1 / 22.7, of 15 000 21.7 / 24.8.
static bool one_head_split(const vista_summarize_desc& d) {
  const int64_t nqb = (d.S + 31) / 32, N = d.total_items;
  if (d.d == 256 || nqb > 8) return false;
  if (nqb <= 2) return N <= (d.d == 64 ? 16384 : 8192);
  if (d.d == 64) return N * nqb <= 1300000;
  return N <= 125000 && double(N) * (double(nqb) * sqrt(double(nqb))) <= 1500000.0;
}

static Heads fitted_heads(const vista_summarize_desc& d) {
  if (mfma_split_supported(d)) return one_head_split(d) ? Heads::kOne : Heads::kWhole;
  if (!mfma_summarize_supported(d)) return Heads::kWhole;
  return one_head_history(d) ? Heads::kOne : short_history(d) ? Heads::kHalf : Heads::kWhole;
}

// Segment size of the matrix-core kernels where the caller leaves it open: the history is cut so that
// the workgroups fill the chip k times, k the smallest count that keeps a segment at or below 32768
// items, a multiple of 32, at least 128 (short histories: see below).  Longer segments mean fewer records to write and merge: 8
// users of a million items (d = 128, S = 256) take 1650 us at this limit, 1669 at 16384 and 1704 or more
// at 8192; one layer at d = 256, S = 512 over 14 M items 11.9, 12.0 and 12.25 ms.  Below 128 items a
// workgroup's set-up and record outweigh its tiles: one user of 7001 items takes 24.8 us at 64, 21.9
// at 96 and 20.8 at 128.
int mfma_summarize_segment(const vista_summarize_desc& d) {
  const int64_t N = d.total_items;
  const Heads heads = fitted_heads(d);
  const int64_t units = 256 * resident_workgroups(d, heads) / head_groups(d, heads);
  constexpr int64_t kMost = 32768, kLeast = 128;
  int64_t k = (N + units * kMost - 1) / (units * kMost);
  if (k < 1) k = 1;
  int64_t s = (N + units * k - 1) / (units * k);
  s = (s + 31) / 32 * 32;
  if (heads == Heads::kHalf && d.d == 128 && d.S < 512) {
    // Few workgroups: a longer segment is more tiles for each, a shorter one more records to write and merge, so the
    // best length goes with the square root: 1.5 sqrt(N), which is beyond both the least length and an even share of the
    // chip from 9200 to 28 700 items.  (15 000 items, d = 128, S = 256: 27.7 us at 128, 24.8 at 192, 24.3 at 256; 30 000: 34.4 at
    // 128, 28.6 at 256, 31.4 at 512.  The other shapes have no such range.)
    const int64_t r = (int64_t(1.5 * sqrt(double(N))) + 16) / 32 * 32;
    if (s < r) s = r;
  }
  return int(s < kLeast ? kLeast : s);
}

// How the heads of G segments are shared out.  Segments fitted here follow fitted_heads; one head a workgroup is for them alone, as
// halves hold their queries in the waves that whole workgroups do and so leave the score bound at the same tiles.  Where the caller names their
// size, or the workspace leaves the base schedule, both kinds walk the same tiles of the same users, and halves win while each has
// a compute unit.  At d = 128 two of them share one, and in a short history nothing is lost beyond (a user is a record and a ragged tile
// of it, 128 items).  Half / whole, mean over 1 to 200 users and segments of 64 to 4096 items: softmax, d = 128, S = 256, 60 halves 0.73, 240
// 0.75, 500 0.95; S = 512, 120 0.77, 240 0.80; S = 128 in segments of 8192, 260 1.06; d = 256, S = 256, 64 halves 0.83, 240 0.86, 480 1.05; S = 512
// 0.82, 0.86, 1.02.  At d = 256 up to 288 are well in segments of up to 256 (0.84 to 0.99), 1.1 to 1.2 in longer ones; S = 64 is 0.99 for 240,
// 1.04 in long segments.
static Heads heads_of_workgroups(const vista_summarize_desc& d, int seg, int64_t G) {
  if (mfma_split_supported(d)) return d.segment_items == 0 && seg == mfma_summarize_segment(d) ? fitted_heads(d) : Heads::kWhole;
  if (!mfma_summarize_supported(d)) return Heads::kWhole;
  if (seg == mfma_summarize_segment(d)) {
    const Heads heads = fitted_heads(d);
    return heads == Heads::kOne && d.segment_items > 0 ? Heads::kHalf : heads;
  }
  const bool few = d.total_items + 128 * int64_t(d.B) <= short_limit(d);
  const int64_t halves = G * head_groups(d, Heads::kHalf);
  const bool half = d.d == 128 ? few || halves <= 256 : few ? halves <= 288 : halves <= 256 && d.S != 64;
  return half ? Heads::kHalf : Heads::kWhole;
}

// Whether the seeds' own keys and values are formed beside the history.  With workgroups on nearly every compute unit the
// main kernel's waves do it as fast as a kernel of its own, without its launch and cold start; with fewer, only a few units
// for each are worth it, and queries of their own for many users over few items go to the kernel that fills the chip.  us a
// call, in front / beside, queries of their own: 250 workgroups, d = 128, S = 256, 40 000 items, 32 users (4 units a workgroup) 46.6 /
// 43.4, 128 users (16) 90.6 / 86.2; 256, d = 256, S = 512, 8000 items, 128 users (64) 302 / 296.  126, d = 128, S = 256, 8000 items: 8 users
// (2) 39.3 / 34.6, 32 users (8) 44.7 / 44.0, 128 users (32) 86.5 / 96.6.  32, 2000 items: 2 users (2) 29.3 / 25.5, 8 users (8) 36.0 / 36.5, 32
// users (32) 47.5 / 67.9.  Split operands: d = 64, S = 100, 63 workgroups, 32 users (3) 35.4 / 31.8; 250, 128 users (3) 43.6 / 38.7;
// d = 256, S = 200, 256, 32 users (6) 103.2 / 95.5.  Of 1152 calls five take the kernel in front where beside is 5 to 13 % faster.
static bool self_beside_history(const vista_summarize_desc& d, int seg, int64_t G, int64_t rows) {
  const int64_t units = (rows + 31) / 32 * (d.d / 32), groups = G * head_groups(d, heads_of_workgroups(d, seg, G));
  return units <= (groups >= 240 ? 64 : 4) * groups;
}

static size_t partial_bytes(const vista_summarize_desc& d, int seg) {
  int64_t G = (d.total_items + seg - 1) / seg;
  return size_t(G + d.B) * d.H * ((d.S + 31) / 32) * kRecFloats * sizeof(float);
}

// [header][seg_user][partial records][K' of the seeds][V' of the seeds]
size_t mfma_summarize_workspace(const vista_summarize_desc& d, int seg) {
  const int64_t G = (d.total_items + seg - 1) / seg;
  return kHeaderBytes + plan_bytes(G) + ((partial_bytes(d, seg) + 255) & ~size_t(255)) + 2 * self_kv_bytes(d);
}

template <int D, int NQB, int HPW, int FW, bool WREG, int MAXT, int ATTN, int NQA = NQB, int OCC = MAXT / 256, bool ORDERED = false>
static hipError_t launch_main(MfmaSummarizeParams& p, int wph, int64_t G, hipStream_t s) {
  p.wph = wph;
  p.nhg = p.H / HPW;
  const int64_t groups = (G + 7) / 8;
  const int64_t blocks = groups * 8 * p.nhg;
  return launch(summarize_mfma_kernel<D, NQB, NQA, HPW, FW, WREG, MAXT, ATTN, OCC, ORDERED>, dim3(unsigned(blocks)),
                dim3(HPW * wph * 64), 0, s, p);
}

template <int ATTN>
static hipError_t launch_for_shape(MfmaSummarizeParams& p, const vista_summarize_desc& desc, int64_t G, hipStream_t s) {
  const int d = desc.d;
  // Four query blocks a wave at d = 128, softmax: the tile in its own order (ordered_tile).  us a call, free / ordered: S = 256, jagged batch
  // 169.2 / 168.9, 8 users of a million items 1573 / 1560, 300 users of 300 003 107.8 / 107.5, one of 7001 20.56 / 20.43; S = 512, 100 users
  // of 300 003 135.9 / 134.7, with queries of their own 146.1 / 146.2.  With queries of their own at S = 256 the registers of
  // their load are spilled in the loop (8 users 84.4 / 84.7, 300 users 120.7 / 122.4): those stay free.  So do one and two blocks a
  // wave (S = 64 66.9 / 67.8, S = 128 equal) and d = 256 (S = 128 225 / 230, S = 512 435 / 450), where a wave has less to put between its
  // products or attends without projecting.  The SiLU form has no such tile.
  constexpr bool softmax = ATTN == VISTA_ATTN_SOFTMAX;
  const bool shared = p.q_user_stride == 0;
  const Heads heads = heads_of_workgroups(desc, p.seg, G);
  if (heads == Heads::kOne) {
    if (d == 128) {
      if (p.nqb <= 2) return launch_main<128, 1, 1, 2, true, 128, ATTN, 1, 2>(p, 2, G, s);
      if (p.nqb <= 4) return launch_main<128, 1, 1, 4, true, 256, ATTN, 1, 2>(p, 4, G, s);
      if (p.nqb <= 8) return launch_main<128, 2, 1, 4, true, 256, ATTN, 2, 2>(p, 4, G, s);
      return launch_main<128, 2, 1, 8, true, 512, ATTN, 2, 2>(p, 8, G, s);
    }
    if (p.nqb <= 8) return launch_main<256, 1, 1, 8, true, 512, ATTN, 1, 2>(p, 8, G, s);
    return launch_main<256, 2, 1, 8, true, 512, ATTN, 2, 2>(p, 8, G, s);
  }
  if (heads == Heads::kHalf) {
    if (d == 128) {
      if (p.nqb <= 2) return launch_main<128, 1, 2, 4, true, 256, ATTN, 1, 2>(p, 2, G, s);
      if (p.nqb <= 4) return launch_main<128, 2, 2, 4, true, 256, ATTN, 2, 2>(p, 2, G, s);
      if (p.nqb <= 8 && shared) return launch_main<128, 4, 2, 4, true, 256, ATTN, 4, 2, softmax>(p, 2, G, s);
      if (p.nqb <= 8) return launch_main<128, 4, 2, 4, true, 256, ATTN, 4, 2>(p, 2, G, s);
      return launch_main<128, 4, 1, 4, true, 256, ATTN, 4, 2, softmax>(p, 4, G, s);
    }
    if (p.nqb <= 2) return launch_main<256, 1, 1, 2, true, 128, ATTN, 1, 2>(p, 2, G, s);
    if (p.nqb <= 4) return launch_main<256, 1, 1, 4, true, 256, ATTN, 1, 2>(p, 4, G, s);
    if (p.nqb <= 8) return launch_main<256, 2, 1, 4, true, 256, ATTN, 2, 2>(p, 4, G, s);
    return launch_main<256, 2, 1, 4, true, 256, ATTN, 6, 2>(p, 4, G, s);
  }
  if (d == 128) {
    // SiLU's two transcendentals a score leave the vector unit the bound: one block a wave feeds it better than
    // two, sixteen waves of them at S = 128 (115 -> 108 us over 500 003 items; softmax the other way, 87 -> 92;
    // at S = 64 eight waves hold one block each as it is).  Sixteen waves of two blocks lose to eight of four:
    // 149 -> 182 us at S = 256, 251 -> 281 at 512; at d = 256 364 -> 361 and, S = 512, 337 -> 356.
    if constexpr (ATTN == VISTA_ATTN_SILU)
      if (p.nqb == 4) return launch_main<128, 1, 4, 8, true, 1024, ATTN>(p, 4, G, s);
    if (p.nqb <= 2) return launch_main<128, 1, 4, 8, true, 512, ATTN>(p, 2, G, s);
    if (p.nqb <= 4) return launch_main<128, 2, 4, 8, true, 512, ATTN>(p, 2, G, s);
    if (p.nqb <= 8 && shared) return launch_main<128, 4, 4, 8, true, 512, ATTN, 4, 2, softmax>(p, 2, G, s);
    if (p.nqb <= 8) return launch_main<128, 4, 4, 8, true, 512, ATTN>(p, 2, G, s);
    return launch_main<128, 4, 2, 8, true, 512, ATTN, 4, 2, softmax>(p, 4, G, s);
  }
  // Two workgroups of four waves on a compute unit: their barriers are not in step (209 -> 167 us over 500 000 items,
  // SiLU form 143 -> 112 over 300 000; with the weights in LDS there was room for one).
  if (p.nqb <= 2) return launch_main<256, 1, 2, 4, true, 256, ATTN, 1, 2>(p, 2, G, s);
  if (p.nqb <= 4) return launch_main<256, 1, 2, 8, true, 512, ATTN>(p, 4, G, s);
  if (p.nqb <= 8) return launch_main<256, 2, 2, 8, true, 512, ATTN>(p, 4, G, s);
  // At S = 512 either four blocks a wave, the weights in LDS, or 2 + 2 + 6 + 6, which leaves the projecting waves registers for
  // the weights.  Softmax: 421 -> 413 us over 500 000 items, two layers over 14 M items with the rest of the path 22.8 -> 22.35
  // ms.  SiLU keeps four each: its vector work is three times as long in a wave of six blocks as beside it (100 000 items in segments
  // of 4096 250 us against 261, 300 000 of 8192 481 against 505, 262 144 at the default 278 against 284).
  if constexpr (ATTN == VISTA_ATTN_SILU) {
    return launch_main<256, 4, 2, 8, false, 512, ATTN>(p, 4, G, s);
  } else {
    // The waves of six blocks are late at every change of user, more so where they load the queries anew: 0.5 to 1 us a change
    // with shared queries, 1.5 to 3 with queries of their own, against 2 % of the call.  So short histories and short users
    // keep four blocks each.  us a call, four each / uneven, lognormal users: shared queries, 32 of 16 000 items 51.7 / 52.5, of
    // 40 000 69.5 / 68.9, of 80 000 101.3 / 99.3; 300 of 40 000 214 / 218, of 320 000 420 / 417; own, 4 of 24 000 53.4 / 55.5, of 80 000
    // 96.0 / 96.2; 32 of 40 000 76.0 / 78.5, of 160 000 168 / 167; 200 of 160 000 269 / 274, of 1 280 000 1164 / 1139.
    const bool own = p.q_user_stride != 0;
    if (p.N < (own ? 65536 : 24576) || p.N < (own ? 4096 : 1024) * int64_t(p.B))
      return launch_main<256, 4, 2, 8, false, 512, ATTN>(p, 4, G, s);
    return launch_main<256, 2, 2, 8, true, 512, ATTN, 6>(p, 4, G, s);
  }
}

template <bool SILU, int RG>
static hipError_t launch_merge(const MfmaSummarizeParams& p, const SummarizeArgs& a, const float* Ks, const float* Vs,
                               int64_t blocks) {
  const vista_summarize_desc& d = a.desc;
  return launch(merge_mfma_kernel<SILU, RG>, dim3(unsigned(RG > 1 ? 4 * blocks : blocks)), dim3(256), 0, a.stream, p.partials, a.offsets,
                d.B, d.S, d.d, d.H, a.seg, d.total_items, a.G, static_cast<uint16_t*>(a.out),
                reinterpret_cast<int*>(a.workspace), a.offsets_checked ? 0 : 1, p.Q, d.q_user_stride, Ks, Vs,
                SILU ? a.scale_plain : a.scale_log2, a.out_scales);
}

vista_status mfma_summarize(const SummarizeArgs& a) {
  const vista_summarize_desc& d = a.desc;
  const bool silu = d.attn == VISTA_ATTN_SILU;
  MfmaSummarizeParams p;
  p.X = static_cast<const uint16_t*>(a.X);
  p.offsets = a.offsets;
  p.Q = static_cast<const uint16_t*>(a.Q);
  p.q_user_stride = d.q_user_stride;
  p.Wk = static_cast<const uint16_t*>(a.Wk);
  p.Wv = static_cast<const uint16_t*>(a.Wv);
  p.partials = reinterpret_cast<float*>(a.workspace + kHeaderBytes + plan_bytes(a.G));
  p.B = d.B;
  p.S = d.S;
  p.nqb = (d.S + 31) / 32;
  p.H = d.H;
  p.N = d.total_items;
  p.seg = a.seg;
  p.c = silu ? -a.scale_log2 : a.scale_log2;
  p.Ks = p.Vs = nullptr;
  p.self_rows = 0;
  float* Ks = nullptr;
  float* Vs = nullptr;
  if (d.flags & VISTA_FLAG_SELF_TERM) {
    Ks = reinterpret_cast<float*>(reinterpret_cast<char*>(p.partials) + ((partial_bytes(d, a.seg) + 255) & ~size_t(255)));
    Vs = Ks + self_kv_bytes(d) / sizeof(float);
    const int64_t rows = d.q_user_stride ? int64_t(d.B) * d.S : d.S;
    if (mfma_self_kv_supported(d, a.Q, a.Wk, a.Wv) && self_beside_history(d, a.seg, a.G, rows)) {
      p.Ks = Ks;
      p.Vs = Vs;
      p.self_rows = rows;
    } else if (launch_self_kv(d, a.Q, a.Wk, a.Wv, Ks, Vs, a.stream) != hipSuccess) {
      return VISTA_ERR_HIP;
    }
  }
  const int64_t merge_blocks = int64_t(d.B) * d.H * p.nqb;
  if ((a.G + 7) / 8 * 8 * 8 > 0x7FFFFFFF || merge_blocks > 0x7FFFFFFF) return VISTA_ERR_UNSUPPORTED;
  if (a.G > 0) {
    const hipError_t e = mfma_split_supported(d) ? launch_split(p, d.d, heads_of_workgroups(d, a.seg, a.G) == Heads::kOne, a.G, a.stream)
                         : silu          ? launch_for_shape<VISTA_ATTN_SILU>(p, d, a.G, a.stream)
                                         : launch_for_shape<VISTA_ATTN_SOFTMAX>(p, d, a.G, a.stream);
    if (e != hipSuccess) return VISTA_ERR_HIP;
  }
  // Few blocks: four times as many, and four waves to a user's records.  A merge is bound by what a
  // compute unit can read (about 20 GB/s each when all do), so it wants them all.
  const bool wide = merge_blocks <= 512 && !a.out_scales;
  auto merge = [&](auto four) {
    constexpr int RG = decltype(four)::value;
    return silu ? launch_merge<true, RG>(p, a, Ks, Vs, merge_blocks) : launch_merge<false, RG>(p, a, Ks, Vs, merge_blocks);
  };
  const hipError_t e = wide ? merge(Int<4>{}) : merge(Int<1>{});
  return e == hipSuccess ? VISTA_OK : VISTA_ERR_HIP;
}

}  // namespace vista
