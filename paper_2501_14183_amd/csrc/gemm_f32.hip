// fp32 GEMMs: fp32 operands, results and accumulation; the products are formed on the bf16 matrix instruction where K is long.
//
// v_mfma_f32_32x32x2_f32 has a sixteenth of the bf16 rate and bounded these products (83-90 of its 157 TFLOP/s).  An fp32
// number of magnitude 2^-110 and more is exactly the sum of three bf16 numbers: hi, mid, lo, each the nearest one to what is left.
// Every product of two of those is exact in fp32, and six of the nine are formed: hi hi, which has accumulators of its own, and
// hi mid, mid hi, mid mid, hi lo, lo hi in a second set, added at the end.  Of the others mid lo and lo mid are at most 2^-25
// of the full one each, of either sign.  So a product by itself is off by at most 2 units of 2^-24 (1.69 over four million pairs,
// rms 0.43) where the fp32 instruction rounds it once (1, rms 0.42); with parts cut off instead of rounded it was 7.2, rms 1.02, and
// always short.  A running sum is rounded once per 16 k instead of eight times, which counts where many terms make the result:
// 1.3e-7 of the result's norm from fp64 against 4.0e-7 for 3392 x 512 x 512, 1.7e-7 against 5.2e-7 with K = 3392, 1.5e-7 against
// 3.8e-7 with scales spread over 2^24 along k, and 4.0-6.1e-7 against 8.6-14e-7 in the outputs of an attention layer.
// What three bf16 numbers do not hold is found and computed once more with the fp32 instruction, a tile at a time: a number with
// bits below 2^-133, the smallest bf16 number (lower bits of the remainder are set then), and infinities and NaN
// (inf - inf: the result is not finite, as where hi rounds to infinity).  They come out as with that instruction alone.
//
// Tiles of 64 x 64, four wavefronts of one 32 x 32 block each, for the sake of many workgroups (a selection of a few thousand
// token rows is 400 tiles).  What bounds it: a slice of 32 k costs the LDS 24 KB of writes at 80 bytes a clock and 48 KB of
// reads at 256 (500 clocks, one after the other), a SIMD 384 clocks of matrix instructions and 104 vector instructions of
// splitting; three workgroups share a compute unit and reach 1080 clocks a slice.  3328 x 512 x 1536: 66 -> 50 us, the
// gradient launch of the same layer 150 -> 102 us (by parts cut off 47 and 98).  Tried: mid lo and lo mid too, with which a
// product by itself is as good as the fp32 instruction's: forward and backward of the layer 86 + 158 -> 93 + 174 us; one LDS
// buffer and four workgroups 47 and 107; fp32 by asynchronous copies, split behind the LDS read by every wavefront for itself
// 53 and 116 (128 x 64 tiles: 61 and 115).
// Global memory goes through registers, where it is split, into two LDS buffers of 32 k: edges and unaligned rows are
// handled there with zeros, so the inner loop has no masks; loads are issued two slices ahead, one barrier per slice.
#include "bf16_mfma.h"
#include "gemm_f32.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kT = 64, kK = 32;              // tile edge, k per LDS buffer
constexpr int kOperand = kT * kK * 4;        // bytes of one fp32 operand in one buffer
constexpr int kPlane = kT * kK * 2;          // bytes of one bf16 part of an operand in one buffer
constexpr int kLds = 2 * 2 * 3 * kPlane;     // two buffers of two operands in three parts

template <typename T>
__device__ inline T pick(int z, T p0, T p1, T p2, T p3) { return z == 0 ? p0 : (z == 1 ? p1 : (z == 2 ? p2 : p3)); }

struct DimsF32 {
  int M, K, splitk, kchunk;
};

// The product's dimensions with a device-side count resolved; false: nothing to do.
__device__ inline bool resolve_f32(const GemmF32& g, DimsF32& dm, bool wgrad) {
  dm.M = g.M;
  dm.K = g.K;
  if (g.n_dev) {
    int n;
    if (!vd_count(g.n_dev, g.n_max, n, g.status)) return false;
    if (g.n_role == 0) dm.M = g.n_mul * n;
    else dm.K = g.n_mul * n;
  }
  dm.splitk = wgrad ? vd_f32_splitk(g.M, g.N, g.nz, dm.K) : 1;
  dm.kchunk = wgrad ? (int)vd_align_up((size_t)vd_ceil_div(dm.K, dm.splitk), kK) : dm.K;
  return true;
}

// One operand's slice of 32 k travels as two 16-byte units per thread.
//   KC (rows contiguous in k): LDS [64 rows][32 k], 16-byte chunk position XORed with (row / 2) % 8 (a read takes one
//      chunk of 16 consecutive rows; two rows share 256 bytes);
//   otherwise (rows contiguous in m or n): LDS [32 k][64], chunk position XORed with 8 on k rows 4..7 of every 8 (a read
//      takes 32 consecutive columns of rows k and k + 4).
// VEC: rows are 16-byte aligned and their extent along the contiguous index is a multiple of 4.
// What lies outside is zeroed on the way into LDS (`in`: one bit per unit, or per element), not here: a use of the loaded
// values right behind the loads would wait for them in front of the slice's matrix instructions.
template <bool KC, bool VEC>
__device__ inline void fetch(f32x4 (&v)[2], uint32_t& in_bits, const float* __restrict__ P, int ld, int r0, int rows, int k0, int kend) {
  in_bits = 0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = u * 256 + threadIdx.x;
    const int row = KC ? r0 + (i >> 3) : k0 + (i >> 4);                // index of the strided dimension
    const int c = KC ? k0 + 4 * (i & 7) : r0 + 4 * (i & 15);           // first index of the contiguous one
    const int row_end = KC ? rows : kend, c_end = KC ? kend : rows;
    const bool ok = row < row_end;
    const float* p = P + (long long)(ok ? row : 0) * ld;
    if constexpr (VEC) {
      const bool in = ok && c < c_end;
      v[u] = *reinterpret_cast<const f32x4*>(p + (in ? c : 0));
      in_bits |= in ? 1u << u : 0u;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = ok && c + e < c_end;
        v[u][e] = p[in ? c + e : 0];
        in_bits |= in ? 1u << (4 * u + e) : 0u;
      }
    }
  }
}
// The same for a slice that lies inside [0, kend) (VEC): a scalar base that moves with the slice plus an offset per thread that
// does not.  Rows or columns past the end repeat the last ones; their results are not stored.
template <bool KC>
__device__ inline void unit_offsets(uint32_t (&off)[2], int ld, int r0, int rows) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = u * 256 + threadIdx.x;
    off[u] = KC ? (uint32_t)(min(i >> 3, rows - 1 - r0) * ld + 4 * (i & 7)) * 4u : (uint32_t)((i >> 4) * ld + min(4 * (i & 15), rows - 4 - r0)) * 4u;
  }
}
template <bool KC>
__device__ inline void fetch_inside(f32x4 (&v)[2], const float* __restrict__ P, int ld, int r0, int k0, const uint32_t (&off)[2]) {
  const char* base = reinterpret_cast<const char*>(P + (KC ? (long long)r0 * ld + k0 : (long long)k0 * ld + r0));
#pragma unroll
  for (int u = 0; u < 2; ++u) v[u] = *reinterpret_cast<const f32x4*>(base + off[u]);
}
// The three bf16 parts of a unit (four fp32 values) as 8 bytes each, to the planes of the operand.  `lost` collects what is left
// for the last part: the lower 16 bits of that say whether it is more than a bf16 number holds.
//   KC: plane [64 rows][32 k], 64-byte rows, 16-byte chunk position XORed with swz_kc<32>(row)
//   otherwise: plane [32 k][64], 128-byte rows, chunk position XORed with swz_nc<64>(k)
template <bool KC>
__device__ inline void put_split(unsigned char* lds, const f32x4 (&v)[2], uint32_t& lost) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = u * 256 + threadIdx.x;
    const int c = KC ? i & 7 : i & 15, row = KC ? i >> 3 : i >> 4;
    const int addr = row * (KC ? 64 : 128) + (((c >> 1) ^ (KC ? swz_kc<kK>(row) : swz_nc<kT>(row))) * 16) + (c & 1) * 8;
    u32x2 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      const float x0 = v[u][e], x1 = v[u][e + 1];
      const uint32_t hw = pack2(x0, x1);
      const float r0 = x0 - __uint_as_float(hw << 16), r1 = x1 - __uint_as_float(hw & 0xffff0000u);   // exact
      const uint32_t mw = pack2(r0, r1);
      const uint32_t l0 = __float_as_uint(r0 - __uint_as_float(mw << 16)), l1 = __float_as_uint(r1 - __uint_as_float(mw & 0xffff0000u));
      lost |= l0 | l1;
      h[e >> 1] = hw;
      m[e >> 1] = mw;
      l[e >> 1] = __builtin_amdgcn_perm(l1, l0, 0x07060302u);
    }
    *reinterpret_cast<u32x2*>(lds + addr) = h;
    *reinterpret_cast<u32x2*>(lds + kPlane + addr) = m;
    *reinterpret_cast<u32x2*>(lds + 2 * kPlane + addr) = l;
  }
}
// k = 16 ks + 8 half + 0..7 of row / column mn0 + lane % 32 of a plane
template <bool KC>
__device__ inline Frag frag_split(const unsigned char* plane, int mn0, int ks, int lane) {
  Frag f;
  const int half = lane >> 5;
  if constexpr (KC) {
    const int row = mn0 + (lane & 31);
    f.q = *reinterpret_cast<const u32x4*>(plane + row * 64 + (((2 * ks + half) ^ swz_kc<kK>(row)) * 16));
  } else {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    const int mn = mn0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int rd = 0; rd < 2; ++rd) {
      const int k = 16 * ks + 8 * half + 4 * rd + ((lane & 15) >> 2);
      const unsigned char* p = plane + k * 128 + (((mn >> 3) ^ swz_nc<kT>(k)) * 16) + ((mn >> 2) & 1) * 8;
      f.d[rd] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
    }
  }
  return f;
}
template <bool KC, bool VEC>
__device__ inline void put(unsigned char* lds, const f32x4 (&v)[2], uint32_t in_bits) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = u * 256 + threadIdx.x;
    const int addr = KC ? (i >> 3) * 128 + (((i & 7) ^ ((i >> 4) & 7)) * 16)
                        : (i >> 4) * 256 + (((i & 15) ^ ((((i >> 4) >> 2) & 1) << 3)) * 16);
    f32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (in_bits >> (VEC ? u : 4 * u + e)) & 1u ? v[u][e] : 0.f;
    *reinterpret_cast<f32x4*>(lds + addr) = w;
  }
}
// k = 8 g + 4 half + e of row / column `mn` of the tile, e = 0..3: both halves of a wavefront and both operands agree on
// this order of k, which is all the contraction needs
template <bool KC>
__device__ inline f32x4 frag(const unsigned char* lds, int mn, int g, int half) {
  if constexpr (KC) {
    return *reinterpret_cast<const f32x4*>(lds + mn * 128 + (((2 * g + half) ^ ((mn >> 1) & 7)) * 16));
  } else {
    f32x4 v;
    const unsigned char* p = lds + (8 * g + 4 * half) * 256 + (((mn >> 2) ^ (half << 3)) * 16) + (mn & 3) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float*>(p + e * 256);
    return v;
  }
}

// One tile of the product: by bf16 parts (SPLIT; `lost`: see put_split), or with the fp32 instruction.
template <bool AKC, bool BKC, bool VEC, bool SPLIT>
__device__ __forceinline__ floatx16 gemm_f32_sum(const GemmF32& g, const DimsF32& dm, int bx, int by, int bz, unsigned char* smem, uint32_t& lost) {
  static_assert(VEC || !SPLIT, "by parts: aligned rows");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
  const int z = bz / dm.splitk, slice = bz - z * dm.splitk;
  const int m0 = by * kT, n0 = bx * kT;
  const int kbeg = slice * dm.kchunk, kend = min(dm.K, kbeg + dm.kchunk);
  const int nk = kend > kbeg ? (kend - kbeg + kK - 1) / kK : 0;
  const int nseg = g.nseg > 1 ? g.nseg : 1;
  const int total = nk * nseg;
  // (values, not references into the argument block: selecting among addresses would put a copy of it into private memory)
  const float *A1 = g.A1, *A2 = g.A2, *B1 = g.B1, *B2 = g.B2;
  const float* A0 = pick(z, g.A0, A1, A2, g.A3);
  const float* B0 = pick(z, g.B0, B1, B2, g.B3);
  const int lda = g.lda, ldb = g.ldb, M = dm.M, N = g.N;
  floatx16 acc = zero16(), low = zero16();     // low: the products of smaller parts
  constexpr int operand = SPLIT ? 3 * kPlane : kOperand;
  f32x4 ra[2][2], rb[2][2];
  uint32_t ia[2], ib[2];
  int fk = kbeg, fseg = 0;                     // fetch cursor
  const float *Ap = A0, *Bp = B0;
  uint32_t offa[2], offb[2];
  if constexpr (SPLIT) {
    unit_offsets<AKC>(offa, lda, m0, M);
    unit_offsets<BKC>(offb, ldb, n0, N);
  }
  auto load = [&](int s) {
    if (SPLIT && fk + kK <= kend) {
      fetch_inside<AKC>(ra[s], Ap, lda, m0, fk, offa);
      fetch_inside<BKC>(rb[s], Bp, ldb, n0, fk, offb);
    } else {
      fetch<AKC, VEC>(ra[s], ia[s], Ap, lda, m0, M, fk, kend);
      fetch<BKC, VEC>(rb[s], ib[s], Bp, ldb, n0, N, fk, kend);
      if constexpr (SPLIT) {                   // (the last slice of a K that is not a multiple of 32)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (!((ia[s] >> u) & 1u)) ra[s][u] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (!((ib[s] >> u) & 1u)) rb[s][u] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
    fk += kK;
    if (fk >= kend && fseg + 1 < nseg) {       // (past the last slice: everything is outside and becomes zeros)
      fk = kbeg;
      ++fseg;
      Ap = fseg == 1 ? A1 : A2;
      Bp = fseg == 1 ? B1 : B2;
    }
  };
  auto store = [&](int s) {
    if constexpr (SPLIT) {
      put_split<AKC>(smem + s * 2 * operand, ra[s], lost);
      put_split<BKC>(smem + s * 2 * operand + operand, rb[s], lost);
    } else {
      put<AKC, VEC>(smem + s * 2 * operand, ra[s], ia[s]);
      put<BKC, VEC>(smem + s * 2 * operand + operand, rb[s], ib[s]);
    }
  };
  auto compute = [&](int buf) {
    const unsigned char* la = smem + buf * 2 * operand;
    const unsigned char* lb = la + operand;
    if constexpr (SPLIT) {
#pragma unroll
      for (int ks = 0; ks < kK / 16; ++ks) {
        Frag a[3], b[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          a[p] = frag_split<AKC>(la + p * kPlane, wm * 32, ks, lane);
          b[p] = frag_split<BKC>(lb + p * kPlane, wn * 32, ks, lane);
        }
        acc = mfma(a[0], b[0], acc);
        low = mfma(a[0], b[2], low);
        low = mfma(a[2], b[0], low);
        low = mfma(a[1], b[1], low);
        low = mfma(a[0], b[1], low);
        low = mfma(a[1], b[0], low);
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < kK / 8; ++q) {
      const f32x4 a = frag<AKC>(la, wm * 32 + col, q, half), b = frag<BKC>(lb, wn * 32 + col, q, half);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
    }
  };
  // Two slices per round, loads and stores without conditions (a load that some path skips would make the compiler wait
  // for the newest loads where it needs the ones before): slices past the end are never read.
  if (total > 0) {
    load(0);
    load(1);
    store(0);
  }
  for (int t = 0; t + 2 <= total; t += 2) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      __syncthreads();                         // slice t + s is in; everyone is done with slice t + s - 1
      load(s);
      compute(s);
      store(1 - s);
      if constexpr (SPLIT) {
        // matrix instructions first, each followed by its share of the next slice's split: one wavefront keeps both pipes busy
        constexpr int RD = (AKC ? 3 : 6) + (BKC ? 3 : 6);
        __builtin_amdgcn_sched_group_barrier(0x100, RD, 0);
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, RD, 0);
#pragma unroll
        for (int i = 0; i < 11; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
          __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        }
      }
    }
  }
  if (total & 1) {
    __syncthreads();
    compute(0);
  }
  if constexpr (SPLIT) acc += low;
  return acc;
}

template <bool AKC, bool BKC, bool VEC, bool SPLIT>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32& g, const DimsF32& dm, int bx, int by, int bz, unsigned char* smem) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
  const int z = bz / dm.splitk, m0 = by * kT, n0 = bx * kT;
  uint32_t lost = 0;
  floatx16 acc = gemm_f32_sum<AKC, BKC, VEC, SPLIT>(g, dm, bx, by, bz, smem, lost);
  if constexpr (SPLIT) {
    bool good = (lost & 0xffffu) == 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) good = good && fabsf(acc[r]) < INFINITY;
    if (__syncthreads_or(!good)) acc = gemm_f32_sum<AKC, BKC, VEC, false>(g, dm, bx, by, bz, smem, lost);
  }
  const float* bias = pick(z, g.bias0, g.bias1, g.bias2, g.bias3);
  float* C = pick(z, g.C0, g.C1, g.C2, g.C3);
  int ldc = g.ldc;
  if (dm.splitk > 1) {
    C = g.part + (long long)bz * dm.M * g.N;
    ldc = g.N;
  }
  const int n = n0 + wn * 32 + col;
  if (n < g.N) {
    const float bv = bias ? bias[n] : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + wm * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
      if (m < dm.M) C[(long long)m * ldc + n] = acc[r] + bv;
    }
  }
}

// (by parts: three workgroups a compute unit, the most its LDS holds; left to itself the compiler takes registers for two)
template <bool AKC, bool BKC, bool VEC, bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 3 : 1) void gemm_f32_kernel(GemmF32 g) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[SPLIT ? kLds : 4 * kOperand];
  DimsF32 dm;
  if (!resolve_f32(g, dm, !AKC)) return;
  const int gx = (g.N + kT - 1) / kT, gy = (dm.M + kT - 1) / kT;
  const int total = gx * gy * g.nz * dm.splitk;
  if ((int)blockIdx.x >= total) return;        // (a grid sized for the bound of a device-side count)
  const int t = xcd_contiguous(blockIdx.x, total);
  gemm_f32_tile<AKC, BKC, VEC, SPLIT>(g, dm, t % gx, (t / gx) % gy, t / (gx * gy), smem);
}

// Input gradient and weight gradients of one layer depend on the same dQ, dK, dV and on nothing of each other: one
// launch, the weight-gradient tiles (K = all tokens: the longer chains) first.
template <bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 3 : 1) void gemm_f32_bwd_pair_kernel(GemmF32 gx, GemmF32 gw) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[SPLIT ? kLds : 4 * kOperand];
  DimsF32 dx, dw;
  if (!resolve_f32(gx, dx, false) || !resolve_f32(gw, dw, true)) return;
  const int wn = (gw.N + kT - 1) / kT, wm = (dw.M + kT - 1) / kT, nw = wn * wm * gw.nz * dw.splitk;
  const int xn = (gx.N + kT - 1) / kT, xm = (dx.M + kT - 1) / kT, nx = xn * xm;
  if ((int)blockIdx.x < nw) {
    const int t = xcd_contiguous(blockIdx.x, nw);
    gemm_f32_tile<false, false, true, SPLIT>(gw, dw, t % wn, (t / wn) % wm, t / (wn * wm), smem);
  } else if ((int)blockIdx.x < nw + nx) {
    const int t = xcd_contiguous(blockIdx.x - nw, nx);
    gemm_f32_tile<true, true, true, SPLIT>(gx, dx, t % xn, t / xn, 0, smem);
  }
}

// C[z][i] = sum over the slices, in order (a single slice was written as the result itself)
__global__ __launch_bounds__(256) void sum_slices_f32_kernel(GemmF32 g) {
  DimsF32 dm;
  if (!resolve_f32(g, dm, true) || dm.splitk <= 1) return;
  const int z = blockIdx.y;
  const long long count = (long long)g.M * g.N;
  const float* p = g.part + z * dm.splitk * count;
  float* C = pick(z, g.C0, g.C1, g.C2, g.C3);
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256) {
    float s = 0.f;
    int k = 0;
    for (; k + 8 <= dm.splitk; k += 8) {       // eight loads in flight, added in slice order
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p[(k + e) * count + i];
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e];
    }
    for (; k < dm.splitk; ++k) s += p[k * count + i];
    C[(i / g.N) * g.ldc + i % g.N] = s;
  }
}

bool aligned4(const GemmF32& g, bool a_kc, bool b_kc) {
  bool ok = g.lda % 4 == 0 && g.ldb % 4 == 0 && (a_kc ? g.K : g.M) % 4 == 0 && (b_kc ? g.K : g.N) % 4 == 0;
  const void* p[8] = {g.A0, g.A1, g.A2, g.A3, g.B0, g.B1, g.B2, g.B3};
  for (const void* q : p) ok = ok && vd_aligned(q, 16);
  return ok;
}

int sum_slices(vardrop_ctx* ctx, const GemmF32& g, int bound, hipStream_t s) {
  if (bound <= 1) return VARDROP_OK;
  const long long blocks = ((long long)g.M * g.N + 255) / 256;
  VdTimer timer(ctx, VARDROP_K_REDUCE_DW, s);
  VD_KERNEL(ctx, sum_slices_f32_kernel, dim3((unsigned)(blocks > 1024 ? 1024 : blocks), g.nz), dim3(256), 0, s, g);
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}

// By parts where a tile walks over at least 256 k; the gradient launch of a layer, where its input-gradient tiles do (3 d), weight
// gradients of few rows included.  Forward and backward of an attention layer, fp32 instruction -> by parts everywhere:
//   d = 64: 16.1 -> 18.0 and 19.5 -> 20.8 us (36 rows), 25.8 -> 27.4 and 38.3 -> 38.4 (3200), 45.3 -> 46.5 and 82.3 -> 80.8 (9600): two
//     slices a tile, the longer start and end of the parts cost more than they save;
//   d = 128: 20.6 -> 21.9 and 27.7 -> 27.9 (36), 37.6 -> 37.7 and 58.9 -> 56.6 (3200), 71.2 -> 70.8 and 140.9 -> 131.1 (9600);
//   d = 192: 23.4 -> 24.0 and 33.2 -> 32.4 (36), 43.1 -> 42.0 and 65.8 -> 60.8 (3200), 104.8 -> 98.5 and 215.0 -> 193.1 (9600);
//   d = 256: 26.1 -> 26.0 and 38.2 -> 35.9 (36), 26.9 -> 26.6 and 39.4 -> 37.6 (256), 53.6 -> 48.8 and 79.6 -> 70.3 (3200);
//   d = 512: 37.7 -> 35.0 and 62.2 -> 56.2 (36), 102 -> 84.4 and 196 -> 154 (3200); d = 1024: 308 -> 239 and 628 -> 479 (3200).
// With only the gradient launch by parts, d = 96 to 224: -4 to 0 % of the backward at 9 to 80 rows, -5 to -11 % from 3200 on.
// (With a device-side count its bound decides.)  Offsets within a tile have 32 bits there: up to 64 rows of 2^24.
bool by_parts(const GemmF32& g, long long k) { return k >= 256 && g.lda <= (1 << 24) && g.ldb <= (1 << 24); }

template <bool AKC, bool BKC>
int launch_f32(vardrop_ctx* ctx, int kid, const GemmF32& g, int slices, hipStream_t s) {
  const long long grid = (long long)vd_ceil_div(g.N, kT) * vd_ceil_div(g.M, kT) * g.nz * slices;
  if (grid >= (1ll << 31)) return VARDROP_EUNSUPPORTED;
  VdTimer timer(ctx, kid, s);
  if (!aligned4(g, AKC, BKC)) VD_KERNEL(ctx, (gemm_f32_kernel<AKC, BKC, false, false>), dim3((unsigned)grid), dim3(256), 0, s, g);
  else if (by_parts(g, AKC ? (long long)g.K * (g.nseg > 1 ? g.nseg : 1) : g.K / slices)) VD_KERNEL(ctx, (gemm_f32_kernel<AKC, BKC, true, true>), dim3((unsigned)grid), dim3(256), 0, s, g);
  else VD_KERNEL(ctx, (gemm_f32_kernel<AKC, BKC, true, false>), dim3((unsigned)grid), dim3(256), 0, s, g);
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}

}  // namespace

int vd_gemm_f32(vardrop_ctx* ctx, int kid, const GemmF32& g, bool b_kc, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return VARDROP_OK;
  return b_kc ? launch_f32<true, true>(ctx, kid, g, 1, s) : launch_f32<true, false>(ctx, kid, g, 1, s);
}

int vd_gemm_f32_wgrad(vardrop_ctx* ctx, int kid, const GemmF32& g, hipStream_t s) {
  const int slices = vd_f32_splitk(g.M, g.N, g.nz, g.K);
  const int rc = launch_f32<false, false>(ctx, kid, g, slices, s);
  return rc ? rc : sum_slices(ctx, g, slices, s);
}

int vd_gemm_f32_bwd_pair(vardrop_ctx* ctx, const GemmF32& gx, const GemmF32& gw, hipStream_t s) {
  if (!aligned4(gx, true, true) || !aligned4(gw, false, false)) return VARDROP_EUNSUPPORTED;
  const int slices = vd_f32_splitk(gw.M, gw.N, gw.nz, gw.K);
  const long long grid = (long long)vd_ceil_div(gx.N, kT) * vd_ceil_div(gx.M, kT) +
                         (long long)vd_ceil_div(gw.N, kT) * vd_ceil_div(gw.M, kT) * gw.nz * slices;
  if (grid >= (1ll << 31)) return VARDROP_EUNSUPPORTED;
  {
    VdTimer timer(ctx, VARDROP_K_GEMM_DW_DXS, s);
    if (by_parts(gx, 3ll * gx.K)) VD_KERNEL(ctx, gemm_f32_bwd_pair_kernel<true>, dim3((unsigned)grid), dim3(256), 0, s, gx, gw);
    else VD_KERNEL(ctx, gemm_f32_bwd_pair_kernel<false>, dim3((unsigned)grid), dim3(256), 0, s, gx, gw);
  }
  VD_LAUNCH_CHECK(ctx);
  return sum_slices(ctx, gw, slices, s);
}
