// fp32 back end of the multi-head attention (Eq. 3), forward and backward, on v_mfma_f32_32x32x2_f32 (fp32 operands and
// accumulation; the projections and their gradients are the GEMMs of gemm_f32.hip).
//
// As in the bf16 back end the work runs on transposed tiles: S^T = K q^T puts one query on a lane, so softmax statistics are
// per-lane scalars and the score registers are, unchanged, the right-hand operand of the next product (register r of a
// half-wavefront holds token 8 (r / 4) + 4 half + r % 4 of the block, and the instruction contracts one token per half).
// A wavefront owns 32 queries (or keys), four share blocks of 32 tokens of two head slices in LDS, double-buffered.
// Bound by the fp32 matrix rate: 2 (forward) and 7 (backward) products of 32 x 32 x d_k per block pair, 64 clocks per
// 32 x 32 x 2.  The row-per-thread multiply-add kernels this replaced took 155 us forward and 318 us backward at
// B = 32, n = 104, d = 512, H = 8.
#include "bf16_mfma.h"
#include "gemm_f32.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SdpaF32 {
  const float *q, *k, *v, *o, *dout;
  float *out, *lse, *dq, *dk, *dv;
  int n, d, H, B;
  float scale;
  const int32_t* n_dev;         // device-side token count (then n is its bound, see vd_count)
};

// Tiles [32 tokens][DH] fp32 in LDS, rows 16 bytes apart from a multiple of 64: a row read takes the same 16-byte chunk of 16
// consecutive rows, which then cover all 64 banks, and a read of 32 consecutive dimensions of a row has its address in one
// register and a constant offset per row (an XOR swizzle needs a register per row: spills in the backward).
template <int DH>
struct Tile {
  static constexpr int kChunks = DH / 4, kPitch = DH * 4 + 16, kBytes = 32 * kPitch;
  static constexpr int kUnits = (32 * kChunks + 255) / 256;         // 16-byte units per thread
  // rows [j0, j0 + 32) of a head slice, zeros from row n on
  static __device__ inline void fetch(f32x4 (&v)[kUnits], const float* p, int ld, int j0, int n) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const int i = u * 256 + threadIdx.x, row = j0 + i / kChunks;
      const bool in = i < 32 * kChunks && row < n;
      const f32x4 w = *reinterpret_cast<const f32x4*>(p + (long long)(in ? row : 0) * ld + (i % kChunks) * 4);
      v[u] = in ? w : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  static __device__ inline void put(unsigned char* lds, const f32x4 (&v)[kUnits]) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const int i = u * 256 + threadIdx.x;
      if (i < 32 * kChunks) *reinterpret_cast<f32x4*>(lds + i / kChunks * kPitch + i % kChunks * 16) = v[u];
    }
  }
};
// a lane's own row as the right-hand operand: head dimensions 8 g + 4 half + e
template <int DH>
__device__ inline void own_row(f32x4 (&f)[DH / 8], const float* p, int ld, int row, int n, int half) {
  const bool in = row < n;
#pragma unroll
  for (int g = 0; g < DH / 8; ++g) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(p + (long long)(in ? row : 0) * ld + 8 * g + 4 * half);
    f[g] = in ? w : f32x4{0.f, 0.f, 0.f, 0.f};
  }
}
// acc += tile rows (32 tokens) x own row: tokens become the rows of the result
template <int DH>
__device__ inline floatx16 rows_times(const unsigned char* tile, const f32x4 (&f)[DH / 8], int col, int half) {
  floatx16 acc = zero16();
#pragma unroll
  for (int g = 0; g < DH / 8; ++g) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(tile + col * Tile<DH>::kPitch + (2 * g + half) * 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], f[g][e], acc, 0, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  return acc;
}
// acc[dt] += tile^T (dimensions 32 dt .. as rows) x the 32 tokens in registers p
template <int DH>
__device__ inline void cols_times(floatx16 (&acc)[(DH + 31) / 32], const unsigned char* tile, const floatx16& p, int col, int half) {
#pragma unroll
  for (int dt = 0; dt < (DH + 31) / 32; ++dt) {
    const int dim = DH < 32 ? col & (DH - 1) : 32 * dt + col;       // (16 dimensions: rows 16.. of the result repeat them, unused)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int token = 8 * (r >> 2) + 4 * half + (r & 3);
      const float a = *reinterpret_cast<const float*>(tile + token * Tile<DH>::kPitch + dim * 4);
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, p[r], acc[dt], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);         // (LDS reads of later products requested from here on would cost registers)
  }
}
// accumulator (rows = head dimensions, column = this lane's token) -> row of the head slice
template <int DH>
__device__ inline void store_row(float* row, const floatx16 (&acc)[(DH + 31) / 32], int half, float mul) {
#pragma unroll
  for (int dt = 0; dt < (DH + 31) / 32; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (32 * dt + 8 * q < DH) {
        const f32x4 w = {acc[dt][4 * q] * mul, acc[dt][4 * q + 1] * mul, acc[dt][4 * q + 2] * mul, acc[dt][4 * q + 3] * mul};
        *reinterpret_cast<f32x4*>(row + 32 * dt + 8 * q + 4 * half) = w;
      }
}
// This workgroup's block of 128 tokens, head and window; each die works through whole (window, head) pairs.
__device__ inline bool block_f32(SdpaF32& a, int parts, int& xb, int& h, int& b) {
  int n;
  if (!vd_count(a.n_dev, a.n, n)) return false;
  a.n = n;
  const int gx = parts * ((n + 127) >> 7), total = gx * a.H * a.B;
  if ((int)blockIdx.x >= total) return false;
  const int t = xcd_contiguous(blockIdx.x, total);
  xb = t % gx;
  h = (t / gx) % a.H;
  b = t / (gx * a.H);
  return true;
}

template <int DH>
__global__ __launch_bounds__(256) void sdpa_fwd_f32(SdpaF32 a) {
  typedef Tile<DH> T;
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * T::kBytes];      // two buffers of K, V
  int qb, h, b;
  if (!block_f32(a, 1, qb, h, b)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int n = a.n, ld = a.d;
  const long long base = (long long)b * n * ld + h * DH;
  const float *kp = a.k + base, *vp = a.v + base;
  const int q0 = qb * 128 + wave * 32, qi = q0 + col;
  const int nb = (n + 31) >> 5;
  f32x4 rk[T::kUnits], rv[T::kUnits], qf[DH / 8];
  T::fetch(rk, kp, ld, 0, n);
  T::fetch(rv, vp, ld, 0, n);
  own_row<DH>(qf, a.q + base, ld, qi, n, half);
  floatx16 acc[(DH + 31) / 32];
#pragma unroll
  for (auto& x : acc) x = zero16();
  float m = -INFINITY, l = 0.f;
  T::put(smem, rk);
  T::put(smem + T::kBytes, rv);
  for (int j = 0; j < nb; ++j) {
    const unsigned char* ks = smem + (j & 1) * 2 * T::kBytes;
    __syncthreads();                           // block j is in; everyone is done with block j - 1
    if (j + 1 < nb) {
      T::fetch(rk, kp, ld, 32 * (j + 1), n);
      T::fetch(rv, vp, ld, 32 * (j + 1), n);
    }
    if (q0 < n) {                              // (the last block's wavefronts past the end only help to load)
      floatx16 st = rows_times<DH>(ks, qf, col, half);
      float mt = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        st[r] = j * 32 + 8 * (r >> 2) + 4 * half + (r & 3) < n ? st[r] * a.scale : -INFINITY;
        mt = fmaxf(mt, st[r]);
      }
      mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
      const float mn = fmaxf(m, mt);           // finite: every block holds a key
      if (__any(mn != m)) {
        const float alpha = expf(m - mn);
        l *= alpha;
#pragma unroll
        for (auto& x : acc)
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] *= alpha;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        st[r] = expf(st[r] - mn);
        l += st[r];
      }
      m = mn;
      cols_times<DH>(acc, ks + T::kBytes, st, col, half);
    }
    if (j + 1 < nb) {
      unsigned char* nx = smem + ((j + 1) & 1) * 2 * T::kBytes;
      T::put(nx, rk);
      T::put(nx + T::kBytes, rv);
    }
  }
  l += __shfl_xor(l, 32, 64);
  if (qi < n) {
    store_row<DH>(a.out + base + (long long)qi * ld, acc, half, 1.f / l);
    if (half == 0) a.lse[((long long)b * a.H + h) * n + qi] = m + logf(l);
  }
}

// dQ of 128 queries: S^T = K q^T and dP^T = V dO^T, dS^T in registers, dQ^T += K^T dS^T.
template <int DH>
__device__ __forceinline__ void bwd_dq_f32(const SdpaF32& a, int qb, int h, int b, unsigned char* smem) {
  typedef Tile<DH> T;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int n = a.n, ld = a.d;
  const long long base = (long long)b * n * ld + h * DH;
  const float *kp = a.k + base, *vp = a.v + base;
  const int q0 = qb * 128 + wave * 32, qi = q0 + col;
  const int nb = (n + 31) >> 5;
  f32x4 rk[T::kUnits], rv[T::kUnits], qf[DH / 8], df[DH / 8];
  T::fetch(rk, kp, ld, 0, n);
  T::fetch(rv, vp, ld, 0, n);
  own_row<DH>(qf, a.q + base, ld, qi, n, half);
  own_row<DH>(df, a.dout + base, ld, qi, n, half);
  float D = 0.f;                               // rowsum(dO * O)
  {
    f32x4 of[DH / 8];
    own_row<DH>(of, a.o + base, ld, qi, n, half);
#pragma unroll
    for (int g = 0; g < DH / 8; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) D = fmaf(df[g][e], of[g][e], D);
    D += __shfl_xor(D, 32, 64);
  }
  const float lse = qi < n ? a.lse[((long long)b * a.H + h) * n + qi] : INFINITY;
  floatx16 acc[(DH + 31) / 32];
#pragma unroll
  for (auto& x : acc) x = zero16();
  T::put(smem, rk);
  T::put(smem + T::kBytes, rv);
  for (int j = 0; j < nb; ++j) {
    const unsigned char* ks = smem + (j & 1) * 2 * T::kBytes;
    __syncthreads();
    if (j + 1 < nb) {
      T::fetch(rk, kp, ld, 32 * (j + 1), n);
      T::fetch(rv, vp, ld, 32 * (j + 1), n);
    }
    if (q0 < n) {
      floatx16 st = rows_times<DH>(ks, qf, col, half);
      const floatx16 dp = rows_times<DH>(ks + T::kBytes, df, col, half);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = expf(fmaf(st[r], a.scale, -lse));
        st[r] = p * (dp[r] - D) * a.scale;
      }
      if (j * 32 + 32 > n) {                   // (a key past the end scores 0: its p = exp(-lse) may be infinite, so its zeros
#pragma unroll                                 //  in K would not drop it)
        for (int r = 0; r < 16; ++r)
          st[r] = j * 32 + 8 * (r >> 2) + 4 * half + (r & 3) < n ? st[r] : 0.f;
      }
      cols_times<DH>(acc, ks, st, col, half);
    }
    if (j + 1 < nb) {
      unsigned char* nx = smem + ((j + 1) & 1) * 2 * T::kBytes;
      T::put(nx, rk);
      T::put(nx + T::kBytes, rv);
    }
  }
  if (qi < n) store_row<DH>(a.dq + base + (long long)qi * ld, acc, half, 1.f);
}

// dK and dV of 128 keys: S = Q k^T and dP = dO v^T (lane = key), P and dS in registers, dV^T += dO^T P, dK^T += Q^T dS.
// rowsum(dO * O) of a block's queries is formed by the threads that copy dO.
template <int DH>
__device__ __forceinline__ void bwd_dkv_f32(const SdpaF32& a, int kb, int h, int b, unsigned char* smem, float (*stat)[2][32]) {
  typedef Tile<DH> T;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int n = a.n, ld = a.d;
  const long long base = (long long)b * n * ld + h * DH;
  const float *qp = a.q + base, *dp_ = a.dout + base, *op = a.o + base;
  const float* lp = a.lse + ((long long)b * a.H + h) * n;
  const int k0 = kb * 128 + wave * 32, kj = k0 + col;
  const int nb = (n + 31) >> 5;
  f32x4 rq[T::kUnits], rd[T::kUnits], ro[T::kUnits], kf[DH / 8], vf[DH / 8];
  float rl = INFINITY;
  auto load = [&](int j) {
    T::fetch(rq, qp, ld, 32 * j, n);
    T::fetch(rd, dp_, ld, 32 * j, n);
    T::fetch(ro, op, ld, 32 * j, n);
    const int i = 32 * j + (int)threadIdx.x;
    if (threadIdx.x < 32) rl = i < n ? lp[i] : INFINITY;       // a query past the end: its probabilities are zero
  };
  auto store = [&](int buf) {
    T::put(smem + buf * 2 * T::kBytes, rq);
    T::put(smem + buf * 2 * T::kBytes + T::kBytes, rd);
    if (threadIdx.x < 32) stat[buf][0][threadIdx.x] = rl;
#pragma unroll
    for (int u = 0; u < T::kUnits; ++u) {
      float s = rd[u][0] * ro[u][0];
#pragma unroll
      for (int e = 1; e < 4; ++e) s = fmaf(rd[u][e], ro[u][e], s);
#pragma unroll
      for (int x = 1; x < T::kChunks; x <<= 1) s += __shfl_xor(s, x, 64);
      const int i = u * 256 + threadIdx.x;
      if (i < 32 * T::kChunks && i % T::kChunks == 0) stat[buf][1][i / T::kChunks] = s;
    }
  };
  load(0);
  own_row<DH>(kf, a.k + base, ld, kj, n, half);
  own_row<DH>(vf, a.v + base, ld, kj, n, half);
  floatx16 ak[(DH + 31) / 32], av[(DH + 31) / 32];
#pragma unroll
  for (auto& x : ak) x = zero16();
#pragma unroll
  for (auto& x : av) x = zero16();
  store(0);
  for (int j = 0; j < nb; ++j) {
    const unsigned char* qs = smem + (j & 1) * 2 * T::kBytes;
    const float (*st2)[32] = stat[j & 1];
    __syncthreads();
    if (j + 1 < nb) load(j + 1);
    if (k0 < n) {
      floatx16 p = rows_times<DH>(qs, kf, col, half);
      floatx16 ds = rows_times<DH>(qs + T::kBytes, vf, col, half);
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 ls = *reinterpret_cast<const f32x4*>(&st2[0][8 * r4 + 4 * half]);
        const f32x4 D = *reinterpret_cast<const f32x4*>(&st2[1][8 * r4 + 4 * half]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * r4 + e;
          p[r] = expf(fmaf(p[r], a.scale, -ls[e]));
          ds[r] = p[r] * (ds[r] - D[e]) * a.scale;
        }
      }
      cols_times<DH>(av, qs + T::kBytes, p, col, half);
      cols_times<DH>(ak, qs, ds, col, half);
    }
    if (j + 1 < nb) store((j + 1) & 1);
  }
  if (kj < n) {
    store_row<DH>(a.dk + base + (long long)kj * ld, ak, half, 1.f);
    store_row<DH>(a.dv + base + (long long)kj * ld, av, half, 1.f);
  }
}

// Both parts of the backward in one launch: of the workgroups of a (window, head), the first half takes keys, the rest queries.
template <int DH>
__global__ __launch_bounds__(256, DH <= 64 ? 2 : 1) void sdpa_bwd_f32(SdpaF32 a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * Tile<DH>::kBytes];
  __shared__ __attribute__((aligned(16))) float stat[2][2][32];
  int xb, h, b;
  if (!block_f32(a, 2, xb, h, b)) return;
  const int blocks = (a.n + 127) >> 7;
  if (xb < blocks) bwd_dkv_f32<DH>(a, xb, h, b, smem, stat);
  else bwd_dq_f32<DH>(a, xb - blocks, h, b, smem);
}

template <int DH>
int launch_core(vardrop_ctx* ctx, const SdpaF32& a, bool backward, hipStream_t s) {
  const long long grid = (long long)(backward ? 2 : 1) * vd_ceil_div(a.n, 128) * a.H * a.B;
  if (grid >= (1ll << 31)) return VARDROP_EUNSUPPORTED;
  VdTimer timer(ctx, backward ? VARDROP_K_SDPA_BWD : VARDROP_K_SDPA_FWD, s);
  if (backward) VD_KERNEL(ctx, sdpa_bwd_f32<DH>, dim3((unsigned)grid), dim3(256), 0, s, a);
  else VD_KERNEL(ctx, sdpa_fwd_f32<DH>, dim3((unsigned)grid), dim3(256), 0, s, a);
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}
int run_core(vardrop_ctx* ctx, const SdpaF32& a, bool backward, hipStream_t s) {
  switch (a.d / a.H) {
    case 16: return launch_core<16>(ctx, a, backward, s);
    case 32: return launch_core<32>(ctx, a, backward, s);
    case 64: return launch_core<64>(ctx, a, backward, s);
    case 128: return launch_core<128>(ctx, a, backward, s);
    default: return VARDROP_EUNSUPPORTED;
  }
}
GemmF32 projection(int M, int d) {
  GemmF32 g = {};
  g.lda = g.ldb = g.ldc = d;
  g.M = M; g.N = d; g.K = d;
  g.nz = 1; g.nseg = 1;
  return g;
}

}  // namespace

// saved: q, k, v, o ([M][d] fp32 each, M = B*n) then lse [B][H][n]
int vd_attn_fwd_f32(vardrop_ctx* ctx, const float* xs, int B, int n, int d, int H,
                    const float* const W[4], const float* const bias[4],
                    float* y, void* saved, void* ws, hipStream_t s, VdDevCount dn) {
  (void)ws;
  const long long M = (long long)B * n;
  float* q = (float*)saved;
  float* o = q + 3 * M * d;
  SdpaF32 a = {};
  a.q = q; a.k = q + M * d; a.v = q + 2 * M * d;
  a.out = o; a.lse = o + M * d;
  a.n = n; a.d = d; a.H = H; a.B = B; a.scale = 1.0f / sqrtf((float)(d / H));
  a.n_dev = dn.dev;
  GemmF32 g = projection((int)M, d);
  g.nz = 3;
  for (int z = 0; z < 3; ++z) g.set(z, xs, W[z], q + z * M * d, bias[z]);
  g.count(dn, true, n, B, 0);
  int rc = vd_gemm_f32(ctx, VARDROP_K_GEMM_QKV, g, false, s);
  if (rc || (rc = run_core(ctx, a, false, s))) return rc;
  GemmF32 go = projection((int)M, d);
  go.set(0, o, W[3], y, bias[3]);
  go.count(dn, false, n, B, 0);
  return vd_gemm_f32(ctx, VARDROP_K_GEMM_OUT, go, false, s);
}

size_t vd_attn_f32_ws_bytes(int B, int n, int d) {
  const size_t M = (size_t)B * n;
  const int slices = vd_f32_splitk(d, d, 4, (long long)M);
  return vd_align_up(4 * M * d * sizeof(float), 256) + (slices > 1 ? (size_t)4 * slices * d * d * sizeof(float) : 0);
}

// ws: dO, dq, dk, dv ([M][d] fp32 each), then the partial products of the weight gradients
int vd_attn_bwd_f32(vardrop_ctx* ctx, const float* dy, const float* xs, int B, int n, int d, int H,
                    const float* const W[4], const void* saved, float* dxs,
                    float* const dW[4], float* const db[4], void* ws, hipStream_t s, VdDevCount dn) {
  const long long M = (long long)B * n;
  const float* q = (const float*)saved;
  const float* o = q + 3 * M * d;
  float* dO = (float*)ws;
  float* dqkv[3] = {dO + M * d, dO + 2 * M * d, dO + 3 * M * d};
  GemmF32 g = projection((int)M, d);           // dO = dy Wo^T
  g.set(0, dy, W[3], dO, nullptr);
  g.count(dn, true, n, B, 0);
  int rc = vd_gemm_f32(ctx, VARDROP_K_GEMM_DO, g, true, s);
  if (rc) return rc;
  SdpaF32 a = {};
  a.q = q; a.k = q + M * d; a.v = q + 2 * M * d; a.o = o; a.dout = dO;
  a.lse = const_cast<float*>(o + M * d);
  a.dq = dqkv[0]; a.dk = dqkv[1]; a.dv = dqkv[2];
  a.n = n; a.d = d; a.H = H; a.B = B; a.scale = 1.0f / sqrtf((float)(d / H));
  a.n_dev = dn.dev;
  if ((rc = run_core(ctx, a, true, s))) return rc;
  GemmF32 gx = projection((int)M, d);          // dxs = dq Wq^T + dk Wk^T + dv Wv^T
  gx.nseg = 3;
  for (int z = 0; z < 3; ++z) gx.set(z, dqkv[z], W[z], z == 0 ? dxs : nullptr, nullptr);
  gx.count(dn, false, n, B, 0);
  GemmF32 gw = {};                             // dWq, dWk, dWv, dWo = xs^T dq, xs^T dk, xs^T dv, o^T dy
  for (int z = 0; z < 3; ++z) gw.set(z, xs, dqkv[z], dW[z], nullptr);
  gw.set(3, o, dy, dW[3], nullptr);
  gw.lda = gw.ldb = gw.ldc = d;
  gw.M = d; gw.N = d; gw.K = (int)M;
  gw.nz = 4; gw.nseg = 1;
  gw.part = (float*)((char*)ws + vd_align_up((size_t)4 * M * d * sizeof(float), 256));
  gw.count(dn, false, n, B, 1);
  if ((rc = vd_gemm_f32_bwd_pair(ctx, gx, gw, s))) return rc;
  if (db[0] || db[1] || db[2] || db[3]) {
    // (the dO rows of the workspace have served their purpose)
    const void* src[4] = {dqkv[0], dqkv[1], dqkv[2], dy};
    return vd_colsum(ctx, VARDROP_F32, src, db, M, d, dO, s, dn, n, B);
  }
  return VARDROP_OK;
}
