// Both stages on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums), for
// fp32 and bf16 storage and any head width that is a multiple of 16: the fp32 configurations and the
// shapes the bf16 kernels do not take.  Calls here are small and bound by latency -- launches, round
// trips to memory, serial chains -- so the aim is few kernels, everything a workgroup needs requested
// at once, and no chain longer than a tile.
//
// Operand layout of one 16x16x4 product, lane = 16 g + c: A holds A[row c][k g], B holds B[k g][col c],
// register r of the accumulator is D[row 4 g + r][col c].  The order in which the four k of a step are
// taken is free as long as A and B agree: scores take channel 16 a + 4 g + b in step (a, b), so a lane's
// four steps are 16 consecutive bytes; P V takes item 16 t + 4 g + r in step (t, r), so the score
// accumulators are the B operand as they stand.
//
// Measured (MI355X): 1 user x 1024 items, d = 64, one head, 16 seeds, then 32 candidates, both stages
// fp32: 1628 us with one thread per query and per (candidate, head), 16 us here; 8 users, 8000 items,
// 4 heads, 64 seeds: 1349 and 20 us.  Error against fp64 1.8e-7 (2-norm), 2.5e-7 before.
#include "common.hpp"

namespace vista {

typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

constexpr int kRows = 64;        // items of a tile
constexpr int kChunk = 64;       // input channels staged at a time
constexpr int kXRow = kChunk + 4;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4(const bf16_t* p) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xFFFF0000u), __uint_as_float(t.y << 16),
                     __uint_as_float(t.y & 0xFFFF0000u));
}
__device__ __forceinline__ void store4(float* p, const f32x4& v) { *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void store4(bf16_t* p, const f32x4& v) {
  *reinterpret_cast<uint2*>(p) = make_uint2(uint32_t(f32_to_bf16_bits(v[0])) | (uint32_t(f32_to_bf16_bits(v[1])) << 16),
                                            uint32_t(f32_to_bf16_bits(v[2])) | (uint32_t(f32_to_bf16_bits(v[3])) << 16));
}
__device__ __forceinline__ float at(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

struct HistoryParams {
  const void* X;
  const int64_t* offsets;
  const void* Q;
  int64_t q_user_stride;
  const void* Wk;
  const void* Wv;
  float* partials;       // [slot][head][query][dh + 2]: O, l, m
  int B, S, d, H;
  int64_t N;
  int seg;
  float scale;           // softmax: scale * log2(e);  SiLU: scale
};

// One workgroup: a segment, a head, 64 U queries (a wave 16 U of them).  Per tile of 64 items: the
// tile's rows and the head's weights pass through LDS in chunks of 64 input channels (the weights stay
// where d <= 64), wave w forms K and V of items 16 w .. 16 w + 15, and after a barrier every wave
// attends over the tile for its own queries with a running maximum.  dh = 16 DT.
template <typename T, int DT, int U, bool SILU>
__global__ __launch_bounds__(256) void history_f32_kernel(HistoryParams p) {
  constexpr int kRow = 16 * DT + 4;      // 4 rows are 16 banks apart: column and row reads spread over the banks
  __shared__ __align__(16) float xs[kRows * kXRow];
  __shared__ __align__(16) float ws[2][kChunk * kRow];
  __shared__ __align__(16) float ks[kRows * kRow];
  __shared__ __align__(16) float vs[kRows * kRow];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int h = blockIdx.y, d = p.d;
  const T* X = static_cast<const T*>(p.X);
  const T* W[2] = {static_cast<const T*>(p.Wk) + h * 16 * DT, static_cast<const T*>(p.Wv) + h * 16 * DT};
  const int64_t seg_begin = int64_t(blockIdx.x) * p.seg;
  const int64_t seg_end = seg_begin + p.seg < p.N ? seg_begin + p.seg : p.N;

  const int q0 = (int(blockIdx.z) * 4 * U + wave) * 16;         // unit u holds queries q0 + 64 u + c
  float4 q[U][DT];
  auto load_queries = [&](int user) __attribute__((always_inline)) {
    const T* Q = static_cast<const T*>(p.Q) + p.q_user_stride * user + h * 16 * DT + 4 * g;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int i = q0 + 64 * u + c;
      if (i > p.S - 1) i = p.S - 1;
#pragma unroll
      for (int a = 0; a < DT; ++a) {
        q[u][a] = load4(Q + int64_t(i) * d + 16 * a);
        q[u][a].x *= p.scale; q[u][a].y *= p.scale; q[u][a].z *= p.scale; q[u][a].w *= p.scale;
      }
    }
  };
  f32x4 o[U][DT];
  float l[U], m[U];
  auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      l[u] = 0.f;
      m[u] = SILU ? 0.f : kLowest;
#pragma unroll
      for (int n = 0; n < DT; ++n) o[u][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto flush = [&](int user) __attribute__((always_inline)) {
    const int64_t slot = int64_t(blockIdx.x) + user;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = q0 + 64 * u + c;
      l[u] += __shfl_xor(l[u], 16, 64);
      l[u] += __shfl_xor(l[u], 32, 64);
      if (i < p.S) {
        float* dst = p.partials + ((slot * p.H + h) * p.S + i) * (16 * DT + 2);
#pragma unroll
        for (int n = 0; n < DT; ++n) {
          *reinterpret_cast<float2*>(dst + 16 * n + 4 * g) = make_float2(o[u][n][0], o[u][n][1]);
          *reinterpret_cast<float2*>(dst + 16 * n + 4 * g + 2) = make_float2(o[u][n][2], o[u][n][3]);
        }
        if (g == 0) *reinterpret_cast<float2*>(dst + 16 * DT) = make_float2(l[u], m[u]);
      }
    }
  };

  if (p.q_user_stride == 0) load_queries(0);
  int wuser = find_user_wave(p.offsets, p.B, seg_begin), user = -1;
  int64_t wpos = seg_begin;
  reset();
  for (int64_t r0 = seg_begin; r0 < seg_end; r0 += kRows) {
    const int rows = seg_end - r0 < kRows ? int(seg_end - r0) : kRows;
    f32x4 acc[2][DT];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int n = 0; n < DT; ++n) acc[e][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < d; k0 += kChunk) {
      const int cols = d - k0 < kChunk ? d - k0 : kChunk;
      const bool weights = d > kChunk || r0 == seg_begin;
      float4 x[4], w[2][DT];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = i * 256 + tid, r = e >> 4, k = 4 * (e & 15);
        x[i] = r < rows && k < cols ? load4(X + (r0 + r) * d + k0 + k) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      if (weights) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < DT; ++i) {
            const int f = i * 256 + tid, k = f / (4 * DT), n = 4 * (f % (4 * DT));
            w[e][i] = k < cols ? load4(W[e] + int64_t(k0 + k) * d + n) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
      }
      __syncthreads();                     // the previous chunk and the previous tile's K, V are no longer read
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = i * 256 + tid;
        *reinterpret_cast<float4*>(xs + (e >> 4) * kXRow + 4 * (e & 15)) = x[i];
      }
      if (weights) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < DT; ++i) {
            const int f = i * 256 + tid;
            *reinterpret_cast<float4*>(ws[e] + f / (4 * DT) * kRow + 4 * (f % (4 * DT))) = w[e][i];
          }
      }
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (16 * a >= cols) break;
        const float4 xa = load4(xs + (16 * wave + c) * kXRow + 16 * a + 4 * g);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int k = (16 * a + 4 * g + b) * kRow + c;
#pragma unroll
          for (int n = 0; n < DT; ++n) {
            acc[0][n] = mfma4(at(xa, b), ws[0][k + 16 * n], acc[0][n]);
            acc[1][n] = mfma4(at(xa, b), ws[1][k + 16 * n], acc[1][n]);
          }
        }
      }
    }
#pragma unroll
    for (int n = 0; n < DT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ks[(16 * wave + 4 * g + r) * kRow + 16 * n + c] = acc[0][n][r];
        vs[(16 * wave + 4 * g + r) * kRow + 16 * n + c] = acc[1][n][r];
      }
    __syncthreads();
    // the pieces (users) that meet this tile
    Piece pc;
    while (next_piece(p.offsets, p.B, r0 + rows, wuser, wpos, pc)) {
      if (pc.user != user) {
        if (user >= 0) {
          flush(user);
          reset();
        }
        user = pc.user;
        if (p.q_user_stride != 0) load_queries(user);
      }
      const int lo = int(pc.begin - r0), hi = int(pc.end - r0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q0 + 64 * u >= p.S) break;                     // (wave-uniform)
        f32x4 s[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (16 * t + 16 <= lo || 16 * t >= hi) continue;
#pragma unroll
          for (int a = 0; a < DT; ++a) {
            const float4 ka = load4(ks + (16 * t + c) * kRow + 16 * a + 4 * g);
#pragma unroll
            for (int b = 0; b < 4; ++b) s[t] = mfma4(at(ka, b), at(q[u][a], b), s[t]);
          }
        }
        if (SILU) {
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int i = 16 * t + 4 * g + r;
              s[t][r] = i >= lo && i < hi ? s[t][r] / (1.f + expf(-s[t][r])) : 0.f;
            }
        } else {
          float top = -INFINITY;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int i = 16 * t + 4 * g + r;
              if (i < lo || i >= hi) s[t][r] = -INFINITY;
              top = fmaxf(top, s[t][r]);
            }
          top = fmaxf(top, __shfl_xor(top, 16, 64));
          top = fmaxf(top, __shfl_xor(top, 32, 64));
          const float mn = fmaxf(m[u], top), alpha = exp2f(m[u] - mn);   // 0 on the first tile (m lowest)
          m[u] = mn;
          l[u] *= alpha;
#pragma unroll
          for (int n = 0; n < DT; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[u][n][r] *= alpha;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              s[t][r] = exp2f(s[t][r] - mn);
              l[u] += s[t][r];
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (16 * t + 16 <= lo || 16 * t >= hi) continue;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            // rows of other users in the tile are left out of the product, not only given weight 0: theirs
            // may be infinite
            const int i = 16 * t + 4 * g + r;
            const bool mine = i >= lo && i < hi;
#pragma unroll
            for (int n = 0; n < DT; ++n) o[u][n] = mfma4(mine ? vs[i * kRow + 16 * n + c] : 0.f, s[t][r], o[u][n]);
          }
        }
      }
    }
  }
  if (user >= 0) flush(user);
}

// The same for segments of 32 items and up to 64 queries, the smallest calls: eight waves share out the products that four waves
// of the kernel above run one after another (a wave there forms 2 x DT blocks of K and V for its 16 items, and with 16 seeds one wave
// attends over all 64 items while three wait).  Here a wave forms one matrix's blocks of 16 items, every other one of DT, and
// attends over 16 items for 16 queries; the two waves that share queries combine their sums when a piece ends.  1 user x 1024 items, d =
// 64, one head, 16 seeds, fp32, with
// the candidates: 18.6 -> 16.3 us.
constexpr int kShortRows = 32, kShortQueries = 64, kShortThreads = 512;
template <typename T, int DT, bool SILU>
__global__ __launch_bounds__(kShortThreads) void history_f32_short_kernel(HistoryParams p) {
  constexpr int kRow = 16 * DT + 4;
  __shared__ __align__(16) float xs[kShortRows * kXRow];
  __shared__ __align__(16) float ws[2][kChunk * kRow];
  __shared__ __align__(16) float ks[kShortRows * kRow];
  __shared__ __align__(16) float vs[kShortRows * kRow];
  __shared__ float other[4][4 * DT + 2][64];           // the later 16 items' O, l, m of the four query units
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int h = blockIdx.y, d = p.d;
  const T* X = static_cast<const T*>(p.X);
  const T* W[2] = {static_cast<const T*>(p.Wk) + h * 16 * DT, static_cast<const T*>(p.Wv) + h * 16 * DT};
  const int64_t seg_begin = int64_t(blockIdx.x) * p.seg;
  const int64_t seg_end = seg_begin + p.seg < p.N ? seg_begin + p.seg : p.N;

  const int q0 = 16 * (wave & 3), half = wave >> 2;    // this wave attends over items 16 half .. 16 half + 15
  const bool attends = q0 < p.S;
  float4 q[DT];
  auto load_queries = [&](int user) __attribute__((always_inline)) {
    const int i = q0 + c < p.S ? q0 + c : p.S - 1;
    const T* Q = static_cast<const T*>(p.Q) + p.q_user_stride * user + int64_t(i) * d + h * 16 * DT + 4 * g;
#pragma unroll
    for (int a = 0; a < DT; ++a) {
      q[a] = load4(Q + 16 * a);
      q[a].x *= p.scale; q[a].y *= p.scale; q[a].z *= p.scale; q[a].w *= p.scale;
    }
  };
  f32x4 o[DT];
  float l, m;
  auto reset = [&]() __attribute__((always_inline)) {
    l = 0.f;
    m = SILU ? 0.f : kLowest;
#pragma unroll
    for (int n = 0; n < DT; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // (the whole workgroup is here together: pieces are the same for all waves)
  auto flush = [&](int user) __attribute__((always_inline)) {
    float* x = &other[wave & 3][0][lane];
    if (half == 1) {
#pragma unroll
      for (int n = 0; n < DT; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[64 * (4 * n + r)] = o[n][r];
      x[64 * 4 * DT] = l;
      x[64 * (4 * DT + 1)] = m;
    }
    __syncthreads();
    if (half == 0 && q0 + c < p.S) {
      const float l2 = x[64 * 4 * DT], m2 = x[64 * (4 * DT + 1)];
      const float mn = SILU ? 0.f : fmaxf(m, m2);
      const float a0 = SILU ? 1.f : exp2f(m - mn), a1 = SILU ? 1.f : exp2f(m2 - mn);    // 0 for sixteen items of other users (m lowest)
      float sum = l * a0 + l2 * a1;
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      float* dst = p.partials + (((int64_t(blockIdx.x) + user) * p.H + h) * p.S + q0 + c) * (16 * DT + 2);
#pragma unroll
      for (int n = 0; n < DT; ++n) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = o[n][r] * a0 + x[64 * (4 * n + r)] * a1;
        *reinterpret_cast<float2*>(dst + 16 * n + 4 * g) = make_float2(v[0], v[1]);
        *reinterpret_cast<float2*>(dst + 16 * n + 4 * g + 2) = make_float2(v[2], v[3]);
      }
      if (g == 0) *reinterpret_cast<float2*>(dst + 16 * DT) = make_float2(sum, mn);
    }
    __syncthreads();                       // before the next piece's sums come to the same place
  };

  if (p.q_user_stride == 0) load_queries(0);
  int wuser = find_user_wave(p.offsets, p.B, seg_begin), user = -1;
  int64_t wpos = seg_begin;
  reset();
  for (int64_t r0 = seg_begin; r0 < seg_end; r0 += kShortRows) {
    const int rows = seg_end - r0 < kShortRows ? int(seg_end - r0) : kShortRows;
    constexpr int NB = (DT + 1) / 2;
    f32x4 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int item0 = 16 * (wave & 1), e0 = (wave >> 1) & 1, n0 = wave >> 2;      // its blocks of K or V: n0, n0 + 2, ...
    for (int k0 = 0; k0 < d; k0 += kChunk) {
      const int cols = d - k0 < kChunk ? d - k0 : kChunk;
      const bool weights = d > kChunk || r0 == seg_begin;
      constexpr int NW = (DT + 1) / 2;
      float4 w[2][NW];
      const int xr = tid >> 4, xk = 4 * (tid & 15);
      const float4 x = xr < rows && xk < cols ? load4(X + (r0 + xr) * d + k0 + xk) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (weights) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < NW; ++i) {
            const int f = i * kShortThreads + tid, k = f / (4 * DT), n = 4 * (f % (4 * DT));
            w[e][i] = f < kChunk * 4 * DT && k < cols ? load4(W[e] + int64_t(k0 + k) * d + n) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
      }
      __syncthreads();                     // the previous chunk and the previous tile's K, V are no longer read
      *reinterpret_cast<float4*>(xs + xr * kXRow + xk) = x;
      if (weights) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < NW; ++i) {
            const int f = i * kShortThreads + tid;
            if (f < kChunk * 4 * DT) *reinterpret_cast<float4*>(ws[e] + f / (4 * DT) * kRow + 4 * (f % (4 * DT))) = w[e][i];
          }
      }
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (16 * a >= cols) break;
        const float4 xa = load4(xs + (item0 + c) * kXRow + 16 * a + 4 * g);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const float* wrow = ws[e0] + (16 * a + 4 * g + b) * kRow + c;
#pragma unroll
          for (int n = 0; n < NB; ++n)
            if (n0 + 2 * n < DT) acc[n] = mfma4(at(xa, b), wrow[16 * (n0 + 2 * n)], acc[n]);
        }
      }
    }
    float* kv = e0 ? vs : ks;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (n0 + 2 * n < DT) kv[(item0 + 4 * g + r) * kRow + 16 * (n0 + 2 * n) + c] = acc[n][r];
    __syncthreads();
    // the pieces (users) that meet this tile
    Piece pc;
    while (next_piece(p.offsets, p.B, r0 + rows, wuser, wpos, pc)) {
      if (pc.user != user) {
        if (user >= 0) {
          flush(user);
          reset();
        }
        user = pc.user;
        if (p.q_user_stride != 0) load_queries(user);
      }
      const int lo = int(pc.begin - r0), hi = int(pc.end - r0);
      if (!attends || 16 * half + 16 <= lo || 16 * half >= hi) continue;       // (wave-uniform)
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int a = 0; a < DT; ++a) {
        const float4 ka = load4(ks + (16 * half + c) * kRow + 16 * a + 4 * g);
#pragma unroll
        for (int b = 0; b < 4; ++b) s = mfma4(at(ka, b), at(q[a], b), s);
      }
      float top = -INFINITY;
      bool mine[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * half + 4 * g + r;
        mine[r] = i >= lo && i < hi;
        if (SILU) {
          s[r] = mine[r] ? s[r] / (1.f + expf(-s[r])) : 0.f;
        } else {
          if (!mine[r]) s[r] = -INFINITY;
          top = fmaxf(top, s[r]);
        }
      }
      if (!SILU) {
        top = fmaxf(top, __shfl_xor(top, 16, 64));
        top = fmaxf(top, __shfl_xor(top, 32, 64));
        const float mn = fmaxf(m, top), alpha = exp2f(m - mn);   // 0 on the first tile (m lowest)
        m = mn;
        l *= alpha;
#pragma unroll
        for (int n = 0; n < DT; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[n][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[r] = exp2f(s[r] - mn);
          l += s[r];
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // rows of other users in the tile are left out of the product, not only given weight 0: theirs
        // may be infinite
        const int i = 16 * half + 4 * g + r;
#pragma unroll
        for (int n = 0; n < DT; ++n) o[n] = mfma4(mine[r] ? vs[i * kRow + 16 * n + c] : 0.f, s[r], o[n]);
      }
    }
  }
  if (user >= 0) flush(user);
}

// Stage 2: one wave scores 16 candidates of one (user, head) against the user's summaries, 64 keys at a
// time with a running maximum; keys and values come straight from memory (a user's summaries of a head
// are a few tens of kilobytes that its waves share through the caches).
template <typename T, int DT>
__global__ __launch_bounds__(64) void candidates_f32_kernel(const T* __restrict__ cand, const T* __restrict__ summ,
                                                            T* __restrict__ out, int C, int S, int d, int H,
                                                            float scale_log2, int self_term) {
  const int lane = threadIdx.x, g = lane >> 4, c = lane & 15;
  const int nc = (C + 15) / 16;
  const int64_t unit = blockIdx.x;
  const int h = int(unit % H);
  const int c0 = int(unit / H % nc) * 16;
  const int64_t b = unit / (int64_t(H) * nc);
  const int ci = c0 + c < C ? c0 + c : C - 1;              // candidates past the end repeat the last; not stored
  const T* qrow = cand + (b * C + ci) * d + h * 16 * DT;
  const T* Y = summ + b * S * d + h * 16 * DT;
  float4 q[DT], own[DT];
#pragma unroll
  for (int a = 0; a < DT; ++a) {
    own[a] = load4(qrow + 16 * a + 4 * g);                 // channels 16 a + 4 g + 0..3: operand and accumulator order
    q[a] = make_float4(own[a].x * scale_log2, own[a].y * scale_log2, own[a].z * scale_log2, own[a].w * scale_log2);
  }
  f32x4 o[DT];
#pragma unroll
  for (int n = 0; n < DT; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kLowest, l = 0.f;
  for (int j0 = 0; j0 < S; j0 += 64) {
    f32x4 s[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (j0 + 16 * t >= S) continue;
      const int j = j0 + 16 * t + c < S ? j0 + 16 * t + c : S - 1;
#pragma unroll
      for (int a = 0; a < DT; ++a) {
        const float4 y = load4(Y + int64_t(j) * d + 16 * a + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[t] = mfma4(at(y, e), at(q[a], e), s[t]);
      }
    }
    float top = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (j0 + 16 * t + 4 * g + r >= S) s[t][r] = -INFINITY;
        top = fmaxf(top, s[t][r]);
      }
    top = fmaxf(top, __shfl_xor(top, 16, 64));
    top = fmaxf(top, __shfl_xor(top, 32, 64));
    const float mn = fmaxf(m, top), alpha = exp2f(m - mn);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int n = 0; n < DT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n][r] *= alpha;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (j0 + 16 * t >= S) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pw = exp2f(s[t][r] - mn);
        l += pw;
        const int i = j0 + 16 * t + 4 * g + r;
        const T* y = Y + int64_t(i < S ? i : S - 1) * d + c;   // (weight 0 past the last key)
#pragma unroll
        for (int n = 0; n < DT; ++n) o[n] = mfma4(to_f32(y[16 * n]), pw, o[n]);
      }
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (self_term) {                       // one more key and value: the candidate itself (Eq. 3)
    float s = 0.f;
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(at(q[a], e), at(own[a], e), s);
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    const float mn = fmaxf(m, s), alpha = exp2f(m - mn), pw = exp2f(s - mn);
    l = fmaf(l, alpha, pw);
#pragma unroll
    for (int n = 0; n < DT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n][r] = fmaf(o[n][r], alpha, pw * at(own[n], r));
  }
  if (c0 + c >= C) return;
  const float inv = 1.f / l;
  T* dst = out + (b * C + c0 + c) * d + h * 16 * DT + 4 * g;
#pragma unroll
  for (int n = 0; n < DT; ++n) store4(dst + 16 * n, o[n] * inv);
}

template <typename T, int DT, bool SILU>
hipError_t launch_history(const HistoryParams& p, int64_t G, hipStream_t s) {
  if (p.seg <= kShortRows && p.S <= kShortQueries)
    return launch(history_f32_short_kernel<T, DT, SILU>, dim3(unsigned(G), unsigned(p.H)), dim3(kShortThreads), 0, s, p);
  const int u = p.S <= 64 ? 1 : p.S <= 128 ? 2 : 4;        // query units of a wave
  const dim3 grid(unsigned(G), unsigned(p.H), unsigned((p.S + 64 * u - 1) / (64 * u)));
  switch (u) {
    case 1: return launch(history_f32_kernel<T, DT, 1, SILU>, grid, dim3(256), 0, s, p);
    case 2: return launch(history_f32_kernel<T, DT, 2, SILU>, grid, dim3(256), 0, s, p);
    default: return launch(history_f32_kernel<T, DT, 4, SILU>, grid, dim3(256), 0, s, p);
  }
}

template <typename T, bool SILU>
hipError_t launch_history_dt(const HistoryParams& p, int64_t G, hipStream_t s) {
  switch (p.d / p.H / 16) {
    case 1: return launch_history<T, 1, SILU>(p, G, s);
    case 2: return launch_history<T, 2, SILU>(p, G, s);
    case 3: return launch_history<T, 3, SILU>(p, G, s);
    default: return launch_history<T, 4, SILU>(p, G, s);
  }
}

template <typename T>
hipError_t launch_candidates(const vista_attend_desc& d, float scale_log2, const void* cand, const void* summ, void* out,
                             hipStream_t s) {
  const int64_t units = int64_t(d.B) * d.H * ((d.C + 15) / 16);
  const dim3 grid(static_cast<unsigned>(units));
  const T* q = static_cast<const T*>(cand);
  const T* y = static_cast<const T*>(summ);
  T* o = static_cast<T*>(out);
  const int self = d.flags & VISTA_FLAG_SELF_TERM;
  switch (d.d / d.H / 16) {
    case 1: return launch(candidates_f32_kernel<T, 1>, grid, dim3(64), 0, s, q, y, o, d.C, d.S, d.d, d.H, scale_log2, self);
    case 2: return launch(candidates_f32_kernel<T, 2>, grid, dim3(64), 0, s, q, y, o, d.C, d.S, d.d, d.H, scale_log2, self);
    case 3: return launch(candidates_f32_kernel<T, 3>, grid, dim3(64), 0, s, q, y, o, d.C, d.S, d.d, d.H, scale_log2, self);
    default: return launch(candidates_f32_kernel<T, 4>, grid, dim3(64), 0, s, q, y, o, d.C, d.S, d.d, d.H, scale_log2, self);
  }
}

// four elements at a time: 16 bytes of fp32, 8 of bf16
bool aligned4(int32_t dtype, const void* p) { return (reinterpret_cast<uintptr_t>(p) & (dtype == VISTA_BF16 ? 7 : 15)) == 0; }

}  // namespace

bool f32_history_supported(const vista_summarize_desc& d) {
  return d.attn != VISTA_ATTN_QLA && d.d / d.H % 16 == 0 && !mfma_summarize_supported(d);
}

bool f32_history_aligned(const vista_summarize_desc& d, const void* X, const void* Q, const void* Wk, const void* Wv) {
  return aligned4(d.dtype, X) && aligned4(d.dtype, Q) && aligned4(d.dtype, Wk) && aligned4(d.dtype, Wv);
}

// Segment size where the caller leaves it open: workgroups (segments x heads x query blocks) for every
// compute unit, a multiple of the 64-item tile, at most 8192 items.
int f32_history_segment(const vista_summarize_desc& d) {
  const int64_t N = d.total_items;
  // Segments of 32 items (history_f32_short_kernel) while a user has few records to merge and the heads leave room on the chip.  Both
  // stages, 64 / 32 items: one user of 1024 items, one head 18.6 / 16.3 us, of 2048 18.3 / 17.7, of 4096 20.2 / 20.9, of 8000 22.9 / 26.6; six of
  // 1024 in all 20.8 / 18.1, of 8000 21.3 / 20.2; two heads, 48 seeds, six of 4096 18.6 / 16.6, of 8000 19.0 / 20.0.
  if (d.S <= kShortQueries && N * d.H <= 8192 && N <= 1536 * int64_t(d.B)) return kShortRows;
  int64_t units = 256 / (int64_t(d.H) * ((d.S + 255) / 256));
  if (units < 32) units = 32;
  int64_t s = (N + units - 1) / units;
  s = (s + kRows - 1) / kRows * kRows;
  return int(s < kRows ? kRows : s > 8192 ? 8192 : s);
}

hipError_t f32_history(const SummarizeArgs& a, float* partials) {
  const vista_summarize_desc& d = a.desc;
  const bool silu = d.attn == VISTA_ATTN_SILU;
  HistoryParams p;
  p.X = a.X;
  p.offsets = a.offsets;
  p.Q = a.Q;
  p.q_user_stride = d.q_user_stride;
  p.Wk = a.Wk;
  p.Wv = a.Wv;
  p.partials = partials;
  p.B = d.B; p.S = d.S; p.d = d.d; p.H = d.H;
  p.N = d.total_items;
  p.seg = a.seg;
  p.scale = silu ? a.scale_plain : a.scale_log2;
  if (d.dtype == VISTA_BF16)
    return silu ? launch_history_dt<bf16_t, true>(p, a.G, a.stream) : launch_history_dt<bf16_t, false>(p, a.G, a.stream);
  return silu ? launch_history_dt<float, true>(p, a.G, a.stream) : launch_history_dt<float, false>(p, a.G, a.stream);
}

// (a wave per unit, and the runtime takes fewer than 2^32 threads: beyond, one thread per candidate and head)
bool f32_candidates_supported(const vista_attend_desc& d, const void* cand, const void* summ, const void* out) {
  return d.d / d.H % 16 == 0 && aligned4(d.dtype, cand) && aligned4(d.dtype, summ) && aligned4(d.dtype, out) &&
         int64_t(d.B) * d.H * ((int64_t(d.C) + 15) / 16) * 64 <= 0xFFFFFFFF;
}

hipError_t f32_candidates(const vista_attend_desc& d, float scale_log2, const void* cand, const void* summ, void* out,
                          hipStream_t s) {
  return d.dtype == VISTA_BF16 ? launch_candidates<bf16_t>(d, scale_log2, cand, summ, out, s)
                               : launch_candidates<float>(d, scale_log2, cand, summ, out, s);
}

}  // namespace vista
