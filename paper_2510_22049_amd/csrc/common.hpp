// Shared device helpers of libvista: storage types, the split-L piece walk and
// the launch-error check.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <utility>

#include "vista.h"

namespace vista {

// bf16 travels as its 16 bit pattern; fp32 as float.
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float(uint32_t(v.bits) << 16); }

// Round-to-nearest-even fp32 -> bf16 (finite values; the paths never produce NaN).
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}
__device__ __forceinline__ void store_as(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_as(bf16_t* p, float v) { p->bits = f32_to_bf16_bits(v); }

constexpr float kLog2e = 1.4426950408889634f;
// A running maximum starts here and not at minus infinity: a tile or segment whose scores are all minus
// infinity then weighs nothing (2^(-inf - lowest) = 0), where -inf - (-inf) would be NaN.
constexpr float kLowest = -3.402823466e38f;
constexpr int kHeaderBytes = 256;  // workspace header: int32 device status at byte 0
// Workspace layout of vista_summarize: [header 256 B][seg_user int32[G], padded to 256 B][path-specific data]
__host__ __device__ inline size_t plan_bytes(int64_t G) { return (size_t(G) * sizeof(int) + 255) & ~size_t(255); }

// ---------------------------------------------------------------------------
// Split-L piece walk (pure function of offsets and the segment size).
// Segment g owns flat rows [g*seg, min((g+1)*seg, N)).  find_user returns the
// last user whose first row is <= row; the walk then visits the non-empty
// intersections of the segment with consecutive users.  Every row handed to a
// caller lies inside the segment, hence inside [0, N), whatever offsets hold.
// ---------------------------------------------------------------------------
// offsets[] entries are read at workgroup-uniform addresses; telling the compiler
// so keeps the whole piece walk (and everything derived from it) in scalar registers.
// The walk is also compiled for the host (vista_summarize_schedule reports it).
__host__ __device__ __forceinline__ int64_t load_uniform(const int64_t* p) {
  const int64_t v = *p;
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v)));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v) >> 32));
  return int64_t((uint64_t(hi) << 32) | lo);
#else
  return v;
#endif
}

__host__ __device__ __forceinline__ int find_user(const int64_t* __restrict__ offsets, int B, int64_t row) {
  int lo = 0, hi = B;  // invariant: offsets[lo] <= row (offsets[0] = 0), answer in [lo, hi)
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (load_uniform(offsets + mid) <= row) lo = mid; else hi = mid;
  }
  return lo;
}

// The same search by a whole wave (all lanes active, `row` wave-uniform): 64 probes a step, so up to 64
// users take one round trip to memory and 4096 take two.  Any offsets keep the answer in [0, B).
__device__ __forceinline__ int find_user_wave(const int64_t* __restrict__ offsets, int B, int64_t row) {
  int lo = 0, n = B;                     // the answer lies in [lo, lo + n)
  while (n > 1) {
    const int step = (n + 63) / 64;
    const int at = int(threadIdx.x & 63) * step;                    // lane i looks at user lo + i step
    const bool below = at > 0 && at < n && offsets[lo + at] <= row; // lane 0 holds by the invariant
    const int last = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(below) | 1ull);   // last lane not beyond the row
    lo += last * step;
    n = n - last * step < step ? n - last * step : step;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// row / seg, the segment of a row: 32-bit division where the row allows, a tenth of the instructions of the 64-bit one.  (No call
// was measurably faster by it: jagged batch 169.7 us both ways, one user of 7001 items 20.4, quasi-linear form 71.5.)
__device__ __forceinline__ int64_t segment_of(int64_t row, int seg) {
  return (uint64_t(row) >> 32) == 0 ? int64_t(uint32_t(row) / uint32_t(seg)) : row / seg;
}

struct Piece {
  int user;
  int64_t begin, end;  // flat rows [begin, end)
};

// Advances to the next piece of segment [pos, seg_end); returns false when done.
// `user` and `pos` carry the walk state between calls.
__host__ __device__ __forceinline__ bool next_piece(const int64_t* __restrict__ offsets, int B, int64_t seg_end,
                                                    int& user, int64_t& pos, Piece& out) {
  while (pos < seg_end && user < B) {
    int64_t uend = load_uniform(offsets + user + 1);
    if (uend > pos) {
      int64_t e = uend < seg_end ? uend : seg_end;
      out.user = user;
      out.begin = pos;
      out.end = e;
      pos = e;
      if (uend <= seg_end) ++user;
      return true;
    }
    ++user;
  }
  return false;
}

// A segment as one stream of tiles of `kTileItems` rows.  A tile never spans two
// users: the cursor walks the pieces of the segment and cuts each into tiles, the
// last of which may be ragged.  When the cursor runs off the segment it stays on
// its last tile (still in bounds) with valid = false.  All state is scalar.
constexpr int kTileItems = 32;
struct TileCursor {
  int wuser;        // piece walk: next user to look at
  int64_t wpos;     // piece walk: next flat row (= end of the current piece)
  int user;         // user of the current piece
  int64_t row;      // first row of the current tile
  int tiles_left;   // tiles of the current piece not yet passed, this one included
  int tail;         // valid rows of the piece's last tile, 1..32
  bool valid;

  __host__ __device__ __forceinline__ void enter(const Piece& pc) {
    const int64_t len = pc.end - pc.begin;            // 1 .. segment size: fits 32 bits
    user = pc.user;
    row = pc.begin;
    tiles_left = int((len + kTileItems - 1) / kTileItems);
    tail = int(len - int64_t(tiles_left - 1) * kTileItems);
  }
  // first_user: the user owning row seg_begin (last user whose first row is <= seg_begin)
  __host__ __device__ __forceinline__ void init(const int64_t* __restrict__ offsets, int B, int first_user,
                                                int64_t seg_begin, int64_t seg_end) {
    wuser = first_user;
    wpos = seg_begin;
    Piece pc;
    pc.user = 0;
    pc.begin = seg_begin;
    pc.end = seg_begin + 1;          // overwritten unless offsets are invalid; stays inside [0, N)
    valid = next_piece(offsets, B, seg_end, wuser, wpos, pc);
    enter(pc);
  }
  __host__ __device__ __forceinline__ void advance(const int64_t* __restrict__ offsets, int B, int64_t seg_end) {
    if (!valid) return;
    if (tiles_left > 1) {
      --tiles_left;
      row += kTileItems;
    } else {
      Piece nx;
      if (next_piece(offsets, B, seg_end, wuser, wpos, nx))
        enter(nx);
      else
        valid = false;               // stays on its last tile
    }
  }
  // Full tiles this cursor can still pass, its current one included, before the last tile of its piece:
  // while `behind` (a cursor some tiles earlier in the stream) is in the same piece, both walk them
  // by adding to `row`, with no look at the pieces (skip).
  __host__ __device__ __forceinline__ int straight(const TileCursor& behind) const {
    return valid && wpos == behind.wpos && user == behind.user ? tiles_left - 1 : 0;
  }
  __host__ __device__ __forceinline__ void skip(int n) {
    tiles_left -= n;
    row += int64_t(n) * kTileItems;
  }
  // valid rows of the current tile
  __host__ __device__ __forceinline__ int rows() const { return tiles_left == 1 ? tail : kTileItems; }
};

template <typename Tuple, size_t... I>
inline void fill_arg_pointers(void** ptrs, Tuple& vals, std::index_sequence<I...>) {
  ((ptrs[I] = static_cast<void*>(&std::get<I>(vals))), ...);
}

// Launches a kernel and reports this launch's own status (an error left behind by an
// earlier, unrelated call of the application is neither reported nor cleared).
template <typename... KArgs, typename... Args>
inline hipError_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                         Args... args) {
  std::tuple<KArgs...> vals{static_cast<KArgs>(args)...};
  void* ptrs[sizeof...(KArgs) > 0 ? sizeof...(KArgs) : 1];
  fill_arg_pointers(ptrs, vals, std::index_sequence_for<KArgs...>{});
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, stream);
}

#define VISTA_LAUNCH(...)                                              \
  do {                                                                 \
    if (::vista::launch(__VA_ARGS__) != hipSuccess) return VISTA_ERR_HIP; \
  } while (0)

// Launchers implemented in the kernel files (host side).
struct SummarizeArgs {
  vista_summarize_desc desc;
  int seg;            // resolved segment size
  int64_t G;          // segments
  const int* seg_user; // [G] first user of each segment (written by the plan kernel); null: found in the kernel
  bool offsets_checked; // the host mirror has been checked: the device need not
  float scale_log2;   // scale * log2(e)
  float scale_plain;  // scale
  const void* X;
  const int64_t* offsets;
  const void* Q;
  const void* Wk;
  const void* Wv;
  void* out;
  float* out_scales;  // non-null: out receives int8 codes and this their scales [B, S, H] (cache codec)
  char* workspace;
  hipStream_t stream;
};

size_t generic_summarize_workspace(const vista_summarize_desc& d, int seg);
// fp32 matrix instructions (plain_mfma.hip); the merge is the plain path's
bool f32_history_supported(const vista_summarize_desc& d);
bool f32_history_aligned(const vista_summarize_desc& d, const void* X, const void* Q, const void* Wk, const void* Wv);
int f32_history_segment(const vista_summarize_desc& d);
hipError_t f32_history(const SummarizeArgs& a, float* partials);
size_t f32_summarize_workspace(const vista_summarize_desc& d, int seg);
vista_status f32_summarize(const SummarizeArgs& a);
bool f32_candidates_supported(const vista_attend_desc& d, const void* cand, const void* summ, const void* out);
hipError_t f32_candidates(const vista_attend_desc& d, float scale_log2, const void* cand, const void* summ, void* out,
                          hipStream_t s);
size_t self_kv_bytes(const vista_summarize_desc& d);
hipError_t launch_self_kv(const vista_summarize_desc& d, const void* Q, const void* Wk, const void* Wv, float* Ks,
                          float* Vs, hipStream_t s);
bool mfma_self_kv_supported(const vista_summarize_desc& d, const void* Q, const void* Wk, const void* Wv);
hipError_t mfma_self_kv(const vista_summarize_desc& d, const void* Q, const void* Wk, const void* Wv, float* Ks,
                        float* Vs, hipStream_t s);
vista_status generic_summarize(const SummarizeArgs& a);
bool mfma_summarize_supported(const vista_summarize_desc& d);
bool mfma_split_supported(const vista_summarize_desc& d);
int mfma_summarize_segment(const vista_summarize_desc& d);
size_t mfma_summarize_workspace(const vista_summarize_desc& d, int seg);
vista_status mfma_summarize(const SummarizeArgs& a);

bool mfma_qla_supported(const vista_summarize_desc& d);
int mfma_qla_segment(const vista_summarize_desc& d);
vista_status mfma_qla_state(const SummarizeArgs& a, float* partials);
// dz: dZs [B][H][32][32] fp32 (device); writes dK and dV rows of every item
vista_status mfma_qla_backward_items(const SummarizeArgs& a, const float* dz, void* d_keys, void* d_values);
size_t qla_backward_workspace(const vista_summarize_desc& d, int seg);
vista_status qla_backward(const SummarizeArgs& a, const void* d_out, void* d_queries, void* d_keys, void* d_values,
                          void* d_self_keys, void* d_self_values);

// summaries either as `summ` (dtype) or, when codes != null, as int8 codes with fp32 scales [B, S, H]
vista_status generic_target_attend(const vista_attend_desc& d, float scale_log2, const void* cand,
                                   const void* summ, const int8_t* codes, const float* scales, void* out,
                                   hipStream_t s);
vista_status generic_quantize(const vista_codec_desc& d, const void* y, int8_t* codes, float* scales, hipStream_t s);
bool mfma_target_attend_supported(const vista_attend_desc& d);
vista_status mfma_target_attend(const vista_attend_desc& d, float scale_log2, const void* cand,
                                const void* summ, const int8_t* codes, const float* scales, void* out,
                                hipStream_t s);

vista_status generic_sglu_ffn(const vista_ffn_desc& d, float eps, const void* y, const void* Wg,
                              const void* Wu, const void* Wo, void* out, hipStream_t s);
bool mfma_sglu_ffn_supported(const vista_ffn_desc& d);
vista_status mfma_sglu_ffn(const vista_ffn_desc& d, float eps, const void* y, const void* Wg,
                           const void* Wu, const void* Wo, void* out, hipStream_t s);

// Validates offsets on the device (status word) and records, for every segment,
// the user that owns its first row (seg_user[g], int32), so that the main
// kernels start their piece walk without a search.
hipError_t launch_plan(const int64_t* offsets, int B, int64_t N, int seg, int64_t G, int* status, int* seg_user,
                       hipStream_t s);

}  // namespace vista
