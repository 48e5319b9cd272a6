// Column sums of the bias gradients: dbq, dbk, dbv, dbo = column sums of dQ, dK, dV, dy (in bf16 where the gradient launch does not form
// them: vd_attn_bf16_sums_inside), dbe = column sums of dxs in fp32.
//
// Bound by reading the four [rows][d] matrices once.  One thread per column walks all rows serially and leaves the chip
// empty (2 700 us for four bf16 matrices of 10272 x 512); here the rows are cut into slices, a workgroup sums one slice
// of one matrix with 16-byte loads, several rows in flight, and a second small kernel adds the slices in order, so
// the result does not depend on scheduling: 10.9 + 4.8 us at that size (3.9 TB/s for the first).
#include "common.h"
#include "bf16_mfma.h"

namespace {

constexpr int kMaxSlices = 64;
constexpr int kSliceRows = 64;      // rows per slice at least: below that a slice is mostly its start and its end

struct ColSum {
  const void* src[4];
  float* dst[4];
  float* part;                      // [4][slices][d] when slices > 1
  long long rows;
  int d, slices;
  const int32_t* n_dev;             // device-side token count: rows = n_mul * n, cut into the same number of slices
  int n_max, n_mul;
};

template <int EPU> __device__ inline void add_unit(float (&s)[EPU], const u32x4& v);
template <> __device__ inline void add_unit<4>(float (&s)[4], const u32x4& v) {
#pragma unroll
  for (int w = 0; w < 4; ++w) s[w] += __uint_as_float(v[w]);
}
template <> __device__ inline void add_unit<8>(float (&s)[8], const u32x4& v) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    s[2 * w] += __uint_as_float(v[w] << 16);
    s[2 * w + 1] += __uint_as_float(v[w] & 0xffff0000u);
  }
}

// EPU elements per 16-byte unit: 8 (bf16) or 4 (fp32).  grid (slices, 4 matrices, blocks of 64 units), 256 threads = four rows.
template <int EPU>
__global__ __launch_bounds__(256) void colsum_kernel(ColSum a) {
  __shared__ float red[3][64][EPU + 1];
  float* dst = a.dst[blockIdx.y];
  if (!dst) return;
  if (a.n_dev) {
    int n;
    if (!vd_count(a.n_dev, a.n_max, n)) return;
    a.rows = (long long)a.n_mul * n;
  }
  const long long chunk = (a.rows + a.slices - 1) / a.slices;
  const long long r0 = blockIdx.x * chunk, r1 = min(a.rows, r0 + chunk);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int units = a.d / EPU, u = blockIdx.z * 64 + lane;
  const u32x4* src = reinterpret_cast<const u32x4*>(a.src[blockIdx.y]) + min(u, units - 1);
  float s[EPU] = {};
  long long r = r0 + wave;
  for (; r + 28 < r1; r += 32) {                 // eight rows of this wavefront in flight
    u32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = src[(r + 4 * i) * units];
#pragma unroll
    for (int i = 0; i < 8; ++i) add_unit<EPU>(s, v[i]);
  }
  for (; r < r1; r += 4) add_unit<EPU>(s, src[r * units]);
  if (wave > 0) {
#pragma unroll
    for (int e = 0; e < EPU; ++e) red[wave - 1][lane][e] = s[e];
  }
  __syncthreads();
  if (wave > 0 || u >= units) return;
  float* out = (a.slices > 1 ? a.part + ((long long)blockIdx.y * a.slices + blockIdx.x) * a.d : dst) + u * EPU;
#pragma unroll
  for (int e = 0; e < EPU; ++e) out[e] = ((s[e] + red[0][lane][e]) + red[1][lane][e]) + red[2][lane][e];
}

// dst[z][c] = sum over the slices, in order inside each of 16 groups and then over the groups.  grid (columns / 16, 4),
// 256 threads: at most four loads a thread, all in flight (with four groups of 16 loads: 6.0 us instead of 4.8).
__global__ __launch_bounds__(256) void colsum_finish_kernel(ColSum a) {
  __shared__ float red[16][17];
  float* dst = a.dst[blockIdx.y];
  if (!dst) return;
  if (a.n_dev) {
    int n;
    if (!vd_count(a.n_dev, a.n_max, n)) return;
  }
  const int col = threadIdx.x & 15, group = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + col;
  const float* p = a.part + (long long)blockIdx.y * a.slices * a.d + min(c, a.d - 1);
  constexpr int PER = kMaxSlices / 16;
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = group * PER + i < a.slices ? p[(long long)(group * PER + i) * a.d] : 0.f;
  float s = v[0];
#pragma unroll
  for (int i = 1; i < PER; ++i) s += v[i];
  red[group][col] = s;
  __syncthreads();
  if (group == 0 && c < a.d) {
#pragma unroll
    for (int g = 1; g < 16; ++g) s += red[g][col];
    dst[c] = s;
  }
}

}  // namespace

// Column sums of the first nz of up to four [rows][d] matrices of the given type (rows whole 16-byte units, 16-byte aligned) into dst[z]
// (fp32, null: skipped).  `scratch`: nz * min(64, rows / 64) * d floats, 16-byte aligned, free to be overwritten.
int vd_colsum(vardrop_ctx* ctx, int dtype, const void* const src[4], float* const dst[4], long long rows, int d,
              void* scratch, hipStream_t s, VdDevCount dn, int n_max, int n_mul, int nz) {
  ColSum c = {};
  for (int z = 0; z < 4; ++z) {
    c.src[z] = src[z];
    c.dst[z] = dst[z];
  }
  c.part = (float*)scratch;      // 4 nz slices d bytes (all four matrices: at most rows d / 4)
  c.rows = rows; c.d = d;
  c.n_dev = dn.dev; c.n_max = n_max; c.n_mul = n_mul;
  const long long want = rows / kSliceRows;
  c.slices = want > kMaxSlices ? kMaxSlices : (want < 1 ? 1 : (int)want);
  const int epu = dtype == VARDROP_BF16 ? 8 : 4;
  const dim3 grid(c.slices, nz, vd_ceil_div(d / epu, 64));
  if (dtype == VARDROP_BF16) hipLaunchKernelGGL(colsum_kernel<8>, grid, dim3(256), 0, s, c);
  else hipLaunchKernelGGL(colsum_kernel<4>, grid, dim3(256), 0, s, c);
  VD_LAUNCH_CHECK(ctx);
  if (c.slices > 1) {
    hipLaunchKernelGGL(colsum_finish_kernel, dim3(vd_ceil_div(d, 16), nz), dim3(256), 0, s, c);
    VD_LAUNCH_CHECK(ctx);
  }
  return VARDROP_OK;
}
