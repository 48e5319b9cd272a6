// fp32 GEMMs on the matrix cores, shared by the fp32 attention back end and the fp32 embedding (gemm_f32.hip).
#ifndef VARDROP_GEMM_F32_H
#define VARDROP_GEMM_F32_H
#include "common.h"

// Up to four batch entries, or up to three accumulated segments.  Named fields rather than arrays, so that the
// argument block is never indexed at run time.
struct GemmF32 {
  const float *A0, *A1, *A2, *A3;
  const float *B0, *B1, *B2, *B3;
  float *C0, *C1, *C2, *C3;
  const float *bias0, *bias1, *bias2, *bias3;
  int lda, ldb, ldc;
  int M, N, K;
  int nz;             // batch entries (matrices)
  int nseg;           // > 1: segments accumulate into C0 (then nz is 1)
  float* part;        // weight gradients of several K slices: slice s of matrix z goes to part + (z * slices + s) * M * N
  // device-side token count (n_dev != nullptr, see vd_count): M (n_role 0) or K (n_role 1) is n_mul * n
  const int32_t* n_dev;
  int32_t* status;
  int n_max, n_mul, n_role;
  void count(const VdDevCount& dn, bool give_status, int nmax, int mul, int role) {
    n_dev = dn.dev; status = give_status ? dn.status : nullptr; n_max = nmax; n_mul = mul; n_role = role;
  }
  void set(int z, const float* a, const float* b, float* c, const float* bias) {
    switch (z) {
      case 0: A0 = a; B0 = b; C0 = c; bias0 = bias; break;
      case 1: A1 = a; B1 = b; C1 = c; bias1 = bias; break;
      case 2: A2 = a; B2 = b; C2 = c; bias2 = bias; break;
      default: A3 = a; B3 = b; C3 = c; bias3 = bias; break;
    }
  }
};

// K slices of a weight gradient over K rows in `nz` matrices of M x N (tiles of 64 x 64): enough workgroups to give every
// compute unit one, slices of at least 256 rows, at most 32 slices.  Grows with K.
__host__ __device__ static inline int vd_f32_splitk(int M, int N, int nz, long long K) {
  const int tiles = nz * vd_ceil_div(M, 64) * vd_ceil_div(N, 64);
  int s = vd_ceil_div(256, tiles);
  if (s > 32) s = 32;
  if (s > K / 256) s = (int)(K / 256);
  return s < 1 ? 1 : s;
}

// C[z] = A[z] B[z] (+ bias[z]), A k-contiguous [M][K], B k-contiguous [N][K] (b_kc) or n-contiguous [K][N]
int vd_gemm_f32(vardrop_ctx*, int kid, const GemmF32& g, bool b_kc, hipStream_t s);
// C[z] = A[z]^T B[z], A [K][M] and B [K][N], K cut into slices by vd_f32_splitk (g.part: room for that many partial
// products); one launch, and a second one that sums the slices when there are several
int vd_gemm_f32_wgrad(vardrop_ctx*, int kid, const GemmF32& g, hipStream_t s);
// the input gradient gx (k-contiguous operands, segments) and the weight gradients gw in one launch (+ the slice sum)
int vd_gemm_f32_bwd_pair(vardrop_ctx*, const GemmF32& gx, const GemmF32& gw, hipStream_t s);
#endif  // VARDROP_GEMM_F32_H
