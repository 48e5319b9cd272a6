// Shared host-side declarations of libvardrop (context, error plumbing, small helpers).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>
#include "../../include/vardrop.h"

static const int kProfPairs = 4096;   // event pairs held between two vardrop_profile_read calls

struct vardrop_ctx {
  int device;
  int last_hip_error;
  int prof_kid;          // kernel whose launches are bracketed by events (-1: none)
  int prof_n;            // pairs recorded since the last read
  int prof_stride;       // every prof_stride-th launch of the selected kernel is bracketed
  int prof_seen;         // launches of the selected kernel seen since it was selected
  hipEvent_t* prof_ev;   // 2 * kProfPairs events, created on first use
  short* prof_kids;      // kernel id of every recorded pair
  hipEvent_t prof_e0, prof_e1;   // the pair the next launch is to be given (null: launch untimed)
  hipEvent_t signal_event[64];   // vardrop_signal_after: the next launch of kernel id i carries signal_event[i] (null: none)
                                 // as the completion event of its own dispatch
  void* twiddle;         // device: k-DFH cosine / sine table in matrix-fragment order (kTwiddleBytes)
  int twiddle_L;         // window length the table currently holds (0: none),
  int twiddle_fmin;      //   its first candidate bin
  int twiddle_F;         //   its number of candidate bins
  int twiddle_r2;        //   and whether it is laid out for the radix-2 kernel
  int lds_per_block;     // bytes of LDS one workgroup may use
  int num_cus;           // compute units of the device
  void* static_scratch;  // device address, on this context's device, of the static scratch array of sample.hip
};

static const int kMaxHashL = 1024;                    // longest window vardrop_hash takes
static const size_t kTwiddleBytes = (size_t)2 << 20;   // 32 contraction steps x 16 bin tiles x 4 KiB

#define VD_HIP(ctx, call)                                   \
  do {                                                      \
    hipError_t e__ = (call);                                \
    if (e__ != hipSuccess) {                                \
      (ctx)->last_hip_error = (int)e__;                     \
      return VARDROP_EHIP;                                  \
    }                                                       \
  } while (0)

#define VD_LAUNCH_CHECK(ctx) VD_HIP(ctx, hipGetLastError())

// Per-kernel timing.  While the context is profiling kernel `kid` (or all kernels), a VdTimer in scope hands the one
// launch issued through VD_KERNEL during its lifetime a pair of events that the runtime ties to that dispatch itself
// (hipExtLaunchKernelGGL): their difference is the kernel's own execution time, as a profiler's kernel trace reports
// it, with no extra packet on the stream.  Costs one integer compare otherwise.
static const int kProfAll = -2;
struct VdTimer {
  vardrop_ctx* ctx;
  bool active;
  bool signal;
  VdTimer(vardrop_ctx* c, int kid, hipStream_t) : ctx(c), active(false), signal(false) {
    if (kid >= 0 && kid < 64 && c->signal_event[kid]) {     // (a launch that signals is not timed)
      signal = true;
      c->prof_e0 = nullptr;
      c->prof_e1 = c->signal_event[kid];
      c->signal_event[kid] = nullptr;
      return;
    }
    if ((c->prof_kid == kid || c->prof_kid == kProfAll) && c->prof_ev && c->prof_n < kProfPairs &&
        (c->prof_seen++ % c->prof_stride) == 0) {
      active = true;
      c->prof_kids[c->prof_n] = (short)kid;
      c->prof_e0 = c->prof_ev[2 * c->prof_n];
      c->prof_e1 = c->prof_ev[2 * c->prof_n + 1];
    }
  }
  ~VdTimer() {
    if (active) {
      ++ctx->prof_n;
      ctx->prof_e0 = ctx->prof_e1 = nullptr;
    }
    if (signal) ctx->prof_e1 = nullptr;
  }
};
#define VD_KERNEL(ctx, kernel, grid, block, lds, s, ...)                                                        \
  do {                                                                                                          \
    if ((ctx)->prof_e1) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, (ctx)->prof_e0, (ctx)->prof_e1, 0, __VA_ARGS__); \
    else hipLaunchKernelGGL(kernel, grid, block, lds, s, __VA_ARGS__);                                          \
  } while (0)

// Token count of a call.  It is either the host integer `bound` itself (n_dev == nullptr) or an int32 in device
// memory that every kernel of the call reads, with `bound` as its upper limit (what the buffers were sized for).
// Returns false when the device value lies outside [0, bound]: the kernel then returns without writing to memory,
// and the first workgroup of the kernel that was handed `status` raises it.
__device__ inline bool vd_count(const int32_t* n_dev, int bound, int& n, int32_t* status = nullptr) {
  n = bound;
  if (!n_dev) return true;
  n = *n_dev;
  if ((unsigned)n <= (unsigned)bound) return true;
  if (status && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0 && threadIdx.y == 0) *status = 1;
  return false;
}

// Workgroups are handed to the eight accelerator dies (XCDs) in turn, and every die has an L2 of its
// own.  These helpers turn a workgroup's linear id into its place in an order in which each die works
// through ONE contiguous range of the tiles, so that tiles sharing an operand meet in the same L2
// instead of each die fetching its own copy from memory.
__device__ static inline int xcd_range_start(int xcd, int total) { return xcd * (total >> 3) + min(xcd, total & 7); }
__device__ static inline int xcd_contiguous(int id, int total) { return xcd_range_start(id & 7, total) + (id >> 3); }

__host__ __device__ static inline size_t vd_align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline bool vd_aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }
__host__ __device__ static inline int vd_ceil_div(int a, int b) { return (a + b - 1) / b; }

// Number of K slices of the weight-gradient GEMMs (K = M = B*n rows).  They share a launch with the input gradient.
// Few tokens: the 64 x 128 weight-gradient tiles walk over K beside 128-row input-gradient tiles, one workgroup per
// compute unit, in slices of at most 4608 rows: one slice up to there, so that no partial products exist (a second slice
// makes that launch 3.5 us shorter at the Traffic shape and costs a 5 us launch that sums the slices).  Many tokens:
// 128 x 128 tiles for both, two workgroups per compute unit, and enough slices for that (counted as twice as many 64-row
// tiles), at least 256 rows each.  Slices are a multiple of the 64-row stage.
// (Host and device: with a device-side token count the kernels evaluate it themselves.)
static const int kFewSliceRows = 4608;      // few tokens: rows of a slice at most
static const int kManySlices = 8;           // many tokens: slices at most
__host__ __device__ static inline int vd_attn_bf16_weight_tiles(int d) { return vd_ceil_div(d, 64) * vd_ceil_div(d, 128) * 4; }
// `many`: which of the two the launch was made for (with a device-side count: by its bound)
__host__ __device__ static inline int vd_attn_bf16_splitk(int d, long long M, bool many, int* kchunk) {
  int s;
  if (many) {
    s = vd_ceil_div(512, vd_attn_bf16_weight_tiles(d));
    if (s > kManySlices) s = kManySlices;
    while (s > 1 && M / s < 256) --s;
  } else {
    s = vd_ceil_div((int)M, kFewSliceRows);
  }
  if (s < 1) s = 1;
  int chunk = (int)vd_align_up((size_t)vd_ceil_div((int)M, s), 64);
  if (chunk < 64) chunk = 64;
  s = M > 0 ? vd_ceil_div((int)M, chunk) : 1;
  if (kchunk) *kchunk = chunk;
  return s;
}
// Many tokens begin at 512 input-gradient tiles of 128 rows, and earlier, from 148 on, where that adds no launch (more than
// 4608 rows have several slices either way, a d of 1024 has one either way), d gives the weight gradients tiles enough, and
// the launch needs fewer rounds of the chip: 512 places for the many-token workgroups, 256 for the others.
// Whole backward, few -> many with the sum of slices, B = 32, us:
//   One round: d = 256 53.4 -> 51.8 at 9600 rows, 66.7 -> 63.9 at 12800 (49.5 -> 50.8 for d = 320 at 6400); d = 384 63.4 -> 62.7 at
//     8544; d = 448 55.2 -> 51.3 at 4800; d = 512 58.4 -> 55.7 at 4800, 71.5 -> 68.7 at 8000; d = 640 84.6 -> 73.0 at 4800; d =
//     704 92.7 -> 83.5 at 4704; d = 768 106 -> 87.0 at 4640; d = 1024 71.2 -> 60.8 at 2400, 94.2 -> 83.9 at 4000.
//   Two rounds against four: d = 512 138 -> 131 at 13440; d = 704 109 -> 104 at 5248; d = 768 126 -> 122 at 7680; d = 832 128 -> 111 at
//     5472; d = 960 142 -> 125 at 4800; d = 1024 152 -> 133 at 4800.
//   Two against three that are full for the most part (over 680 of 768 places): d = 320 129 -> 121 at 18784; d = 384 134 -> 130 at
//     17056; d = 448 102 -> 96.2 at 11040; d = 512 107 -> 105 at 10560, 114 -> 109 at 12000; d = 576 110 -> 107 at 8448; d = 640
//     101 -> 103 at 7424, 123 -> 121 at 9216; but d = 704 93.5 -> 101 at 4864 and d = 256 187 -> 188 at 32000.
//   Two against three that are not: d = 384 92.0 -> 96.1 at 12800; d = 448 87.1 -> 89.7 at 9920; d = 512 93.0 -> 96.0 at 8320; d = 576
//     75.5 -> 80.9 at 5504, 85.2 -> 92.9 at 6656; d = 640 90.7 -> 96.2 at 6272 (but d = 320 93.4 -> 91.7 at 15360).
//   Two against two: d = 320 74.2 -> 78.8 at 10464, d = 384 77.7 -> 84.6 at 11104, d = 448 69.6 -> 77.0 at 7360.
//   Up to 4608 rows: d = 512 29.2 -> 38.2 at 2048, 37.5 -> 42.4 at 3328, 41.8 -> 44.9 at 4096; d = 768 53.4 -> 61.7, 69.6 -> 68.9, 78.7 ->
//     76.4; d = 640 51.1 -> 54.4, 62.3 -> 60.8, 67.1 -> 64.1; d = 384 27.5 -> 34.1, 35.3 -> 36.5, 38.6 -> 37.9; d = 256 24.1 -> 28.0,
//     33.0 -> 30.3, 36.9 -> 30.9.  What the later of these would gain, a device-side count of half its bound would lose.
// With a device-side count the bound decides.  Counts near it gain as above, counts far below it lose: d = 512, bound 6144
// rows, 6080 rows 67.8 -> 65.5, 4160 56.3 -> 57.1, 3200 40.6 -> 45.6; bound 6880, 4000 rows 45.2 -> 47.3, 704 28.5 -> 38.2; bound
// 8320, 8000 rows 77.1 -> 73.9, 6400 68.8 -> 67.3, 4160 55.8 -> 56.8.
static inline bool vd_attn_bf16_many_tokens(int d, long long M) {
  const int cols = vd_ceil_div(d, 128), weight_tiles = vd_attn_bf16_weight_tiles(d);
  const long long tiles = (long long)vd_ceil_div((int)M, 128) * cols;
  if (tiles >= 512) return true;
  if (tiles < 148 || d < 256 || (M <= kFewSliceRows && weight_tiles < 512)) return false;
  const long long many = tiles + 4 * cols * cols * vd_attn_bf16_splitk(d, M, true, nullptr);
  const long long few = tiles + weight_tiles * vd_attn_bf16_splitk(d, M, false, nullptr);
  return many <= 512 || few > 768 || (few > 680 && d >= 320 && d <= 640);
}
// Bias gradients: the copy wavefronts of the weight-gradient tiles add up the columns of their right-hand operand while they
// wait (GemmBf16::sum0 ..), or the two launches of colsum.hip read that operand again.  With few tokens, one workgroup a compute unit,
// the launch is as long as one weight-gradient tile's chain of slices while there are places for all tiles, and the sums lengthen every
// slice of it by about 0.1 us: inside only for short chains, or with a tenth more tiles than places.  Whole backward, launches of
// their own -> inside, us:
//   d = 64 25.7 -> 25.4 at 1536 rows, 24.4 -> 25.1 at 1792, 34.6 -> 42.0 at 4096; d = 128 23.8 -> 23.0 at 1536, 26.9 -> 27.5 at 2048, 37.6 ->
//   43.2 at 4096; d = 192 27.0 -> 26.6 at 1792, 28.2 -> 28.7 at 2048; d = 256 31.8 -> 30.9 at 2048, 36.8 -> 38.5 at 3072; d = 384 35.3 -> 34.6 at
//   2304, 45.0 -> 46.2 at 3072; d = 512 27.1 -> 20.6 at 256, 39.5 -> 38.8 at 2560, 48.2 -> 50.2 at 3584;
//   several slices, whose sum runs anyway: two of 2560 d = 64 33.4 -> 33.7, d = 128 36.7 -> 34.5, d = 256 45.9 -> 43.9; two of 3072 d = 128 38.2 ->
//   39.0, d = 256 46.8 -> 47.6; two of 4096 d = 64 40.0 -> 44.8, d = 256 50.9 -> 54.1;
//   more tiles than places: d = 512 61.5 -> 65.0 at 4608 (272 tiles), d = 192 57.5 -> 59.8 at 12 288 (264), d = 384 58.1 -> 56.4 at 6144 (288),
//   d = 320 1.08x at 12 288 (468), d = 448 1.08x at 8192 (480), from d = 576 on 1.1-1.25x at every count.  Many tokens: 1.01-1.14x.
static inline bool vd_attn_bf16_sums_inside(int d, long long M, bool many, int splitk, int kchunk, int num_cus) {
  const long long tiles = (long long)vd_ceil_div(d, 128) * ((M + 127) / 128) + (long long)vd_attn_bf16_weight_tiles(d) * splitk;
  int rows = d < 384 ? 1024 + 4 * d : 2560;
  if (splitk > 1) rows = rows + 1000 < 3000 ? rows + 1000 : 3000;
  return many || kchunk <= rows || 10 * tiles >= 11ll * num_cus;
}
// Most slices of any count of up to M rows.  The few-token side has more than kManySlices only while one column of tiles
// (d <= 128) keeps it going past 36864 rows: 15 at its end, 511 tiles.  Grows with M.
static inline int vd_attn_bf16_max_splitk(int d, long long M) {
  const long long few_end = 511ll / vd_ceil_div(d, 128) * 128;
  const int s = vd_ceil_div((int)(M < few_end ? M : few_end), kFewSliceRows);
  return s > kManySlices ? s : kManySlices;
}
size_t vd_attn_bf16_partial_offset(int B, int n, int d, int H);
size_t vd_attn_bf16_ws_bytes(int B, int n, int d, int H);

// device address of the static scratch array (sample.hip) on the current device; 0 or the hipError_t
int vd_static_scratch_address(void** out);

size_t vd_attn_f32_ws_bytes(int B, int n, int d);

// attention back ends (attn_f32.hip, attn_bf16.hip); argument checks are done by the caller
// K slices of the embedding's weight gradient dWe = z^T dxs (K = M = B * n_sel rows, L x d results): a slice fewer is a partial
// product fewer to write and to sum (1.1 us at 720 x 512), a longer slice 0.45 us per 64 rows, which meet at s^2 = 2600 M / (L d).
// At most 16, at least 128 rows each, and no more than leave all tiles resident together (10 272 rows of 1024 x 1024 with five of 128
// tiles 48.1 us, with four 35.7).  dWe and its sum back to back, with slices that gave the chip two workgroups a compute unit and two copy
// stages -> with these and three stages, us: 24.8 -> 15.4 (3008 rows, 720 x 512; inside a step 18 -> 16), 33.8 -> 22.9 (10 272), 33.3 -> 25.3
// (10 272, 1024 x 512), 21.8 -> 15.4 (27 584, 96 x 512), 9.4 -> 8.7 (3680, 96 x 512; inside a step 11.4 -> 11.4), 7.9 -> 8.0 (800, 240 x 512), 18.3 ->
// 18.9 (10 272, 240 x 1024).  (Host and device.)
__host__ __device__ static inline int vd_embed_splitk(int L, int d, long long M, int* kchunk) {
  const int most = 512 / (vd_ceil_div(L, 64) * vd_ceil_div(d, 128));       // slices whose tiles are resident together
  int s = 1;
  while (s < 16 && s < most && (long long)(s + 1) * (s + 1) * L * d <= 2600 * M) ++s;
  while (s > 1 && M / s < 128) --s;
  int chunk = (int)vd_align_up((size_t)vd_ceil_div((int)M, s), 64);
  if (chunk < 64) chunk = 64;
  if (kchunk) *kchunk = chunk;
  return M > 0 ? vd_ceil_div((int)M, chunk) : 1;
}

// A count that may live in device memory (see vd_count): with dev != nullptr the `n` of the call is its bound.
struct VdDevCount {
  const int32_t* dev;
  int32_t* status;
};
int vd_attn_fwd_f32(vardrop_ctx*, const float* xs, int B, int n, int d, int H,
                    const float* const W[4], const float* const bias[4],
                    float* y, void* saved, void* ws, hipStream_t s, VdDevCount dn = {nullptr, nullptr});
int vd_attn_bwd_f32(vardrop_ctx*, const float* dy, const float* xs, int B, int n, int d, int H,
                    const float* const W[4], const void* saved, float* dxs,
                    float* const dW[4], float* const db[4], void* ws, hipStream_t s, VdDevCount dn = {nullptr, nullptr});
int vd_attn_fwd_bf16(vardrop_ctx*, const void* xs, int B, int n, int d, int H,
                     const void* const W[4], const void* const bias[4],
                     void* y, void* saved, void* ws, hipStream_t s,
                     const int32_t* sel = nullptr, int N = 0, void* xs_out = nullptr, VdDevCount dn = {nullptr, nullptr});
int vd_attn_bwd_bf16(vardrop_ctx*, const void* dy, const void* xs, int B, int n, int d, int H,
                     const void* const W[4], const void* saved, void* dxs,
                     float* const dW[4], float* const db[4], void* ws, hipStream_t s, VdDevCount dn = {nullptr, nullptr});
// column sums of up to four [rows][d] matrices (colsum.hip)
int vd_colsum(vardrop_ctx*, int dtype, const void* const src[4], float* const dst[4], long long rows, int d,
              void* scratch, hipStream_t s, VdDevCount dn, int n_max, int n_mul, int nz = 4);
// gather / scatter with an optional device-side count (gather.hip); argument checks are done by the caller
int vd_gather(vardrop_ctx*, const void* tokens, int B, int N, int d, int dtype, const int32_t* sel, int n_sel,
              void* out, hipStream_t s, VdDevCount dn = {nullptr, nullptr});
