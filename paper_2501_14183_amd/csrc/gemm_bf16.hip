// bf16 GEMMs of the attention back end on v_mfma_f32_32x32x16_bf16: projections, their input and
// weight gradients, and the sum of K slices.
#include "bf16_mfma.h"
#include "gemm_bf16.h"

namespace {

// out[z][i] = sum_s part[(z * splitk + s)][i], slices added in ascending order
struct SplitkReduce {
  const float* part;
  float* out[4];
  long long count;     // elements per matrix
  const float* sum_part;   // and of the column sums that ride along (nullptr: none), N a matrix
  float* sum[4];
  int N;
  int blocks;          // workgroups of a matrix; those behind them add up its column sums
  int splitk;
  // device-side token count: the slice count is the one the weight-gradient kernel derived from it (d = dn_d)
  const int32_t* n_dev;
  int n_max, n_mul, dn_d, many;
};
// One matrix of `stride` elements per slice, always `splitk` partial products (no direct result): its first count0
// elements go to out0, the next count1 to out1 (nullable).  With a device-side count the slices follow the
// embedding's rule (M = dn_m rows, N = dn_n columns).
struct SplitkReduceRows {
  const float* part;
  float* out0;
  float* out1;
  long long count0, count1, stride;
  int splitk;
  const int32_t* n_dev;
  int n_max, n_mul, dn_m, dn_n;
};
// add(get(0)), add(get(1)), ... add(get(n - 1)) in order, up to eight in flight.  (A loop that takes four at a time and the rest one by
// one waits four times for seven slices; one branch per slice costs a single slice 0.3 us.)
template <int U, typename GET, typename ADD>
__device__ __forceinline__ void add_slices_fixed(int k0, GET get, ADD add) {
  decltype(get(0)) v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = get(k0 + u);
#pragma unroll
  for (int u = 0; u < U; ++u) add(v[u]);
}
template <typename GET, typename ADD>
__device__ __forceinline__ void add_slices(int n, GET get, ADD add) {
  int k0 = 0;
  for (; k0 + 8 <= n; k0 += 8) add_slices_fixed<8>(k0, get, add);
  switch (n - k0) {
    case 1: add_slices_fixed<1>(k0, get, add); break;
    case 2: add_slices_fixed<2>(k0, get, add); break;
    case 3: add_slices_fixed<3>(k0, get, add); break;
    case 4: add_slices_fixed<4>(k0, get, add); break;
    case 5: add_slices_fixed<5>(k0, get, add); break;
    case 6: add_slices_fixed<6>(k0, get, add); break;
    case 7: add_slices_fixed<7>(k0, get, add); break;
    default: break;
  }
}
__global__ __launch_bounds__(256) void splitk_reduce_rows_kernel(SplitkReduceRows a) {
  int splitk = a.splitk;
  if (a.n_dev) {
    int n;
    if (!vd_count(a.n_dev, a.n_max, n)) return;
    splitk = n == 0 ? 0 : vd_embed_splitk(a.dn_m, a.dn_n, (long long)a.n_mul * n, nullptr);   // no tokens: zero gradients
  }
  const long long total = a.count0 + (a.out1 ? a.count1 : 0);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    const float* p = a.part + i;
    float s = 0.f;
    add_slices(splitk, [&](int k) { return p[(long long)k * a.stride]; }, [&](float v) { s += v; });
    if (i < a.count0) a.out0[i] = s; else a.out1[i - a.count0] = s;
  }
}
__global__ __launch_bounds__(256) void splitk_reduce_kernel(SplitkReduce a) {
  int splitk = a.splitk;
  if (a.n_dev) {
    int n;
    if (!vd_count(a.n_dev, a.n_max, n)) return;
    splitk = vd_attn_bf16_splitk(a.dn_d, (long long)a.n_mul * n, a.many != 0, nullptr);
    if (splitk <= 1 && n > 0) return;            // a single slice was written as the result itself
    if (n == 0) splitk = 0;                      // no tokens: the gradients are zero
  }
  const int z = blockIdx.y;
  if ((int)blockIdx.x >= a.blocks) {
    const int c = ((int)blockIdx.x - a.blocks) * blockDim.x + threadIdx.x;
    float* dst = z == 0 ? a.sum[0] : (z == 1 ? a.sum[1] : (z == 2 ? a.sum[2] : a.sum[3]));
    if (!dst || c >= a.N) return;
    const float* p = a.sum_part + (long long)z * splitk * a.N + c;
    float s = 0.f;
    add_slices(splitk, [&](int k) { return p[(long long)k * a.N]; }, [&](float v) { s += v; });
    dst[c] = s;
    return;
  }
  const long long n4 = a.count >> 2;
  const float4* src = reinterpret_cast<const float4*>(a.part) + (long long)z * splitk * n4;
  float4* dst = reinterpret_cast<float4*>(z == 0 ? a.out[0] : (z == 1 ? a.out[1] : (z == 2 ? a.out[2] : a.out[3])));
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (long long)a.blocks * blockDim.x) {
    float4 s = splitk > 0 ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    add_slices(splitk - 1, [&](int k) { return src[(long long)(k + 1) * n4 + i]; },
               [&](const float4& v) { s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w; });
    dst[i] = s;
  }
}

// ================================================================== GEMM with asynchronous LDS fill
// C[z] = op(A[z]) * op(B[z]) (+ bias[z]) in bf16, the sum over up to three segments into C[0], or
// (SPLIT) an fp32 partial product per K slice.  Each operand is either k-contiguous ([M][K] / [N][K])
// or mn-contiguous ([K][M] / [K][N]).
//
// Global memory is copied straight into LDS (dma16_buf: every lane names its own 16
// source bytes, the wavefront's 64 chunks land in 1 KB of consecutive LDS), NS stages deep, so
// that the copies of the next NS-1 slices are in flight while the matrix cores work on the
// current one and no register or LDS-store instruction is spent on staging.  Because the LDS side
// of a copy is fixed, the bank swizzle is applied on the source side: LDS chunk position p of a row
// holds source chunk p ^ pattern(row).
//   k-contiguous operand:  LDS tile [row][BK], fragments are 16-byte reads (row = lane % 32,
//                          chunk 2*ks + lane / 32), pattern chosen so that eight consecutive rows
//                          spread over all banks.
//   mn-contiguous operand: LDS tile [k][W]; fragments come from the transposing read
//                          ds_read_b64_tr_b16, in which, inside each group of 16 lanes, lane s names
//                          four consecutive columns of k-row s / 4 at column block s % 4, and lane j
//                          receives column j of the four k-rows.  A slice that reaches past the end
//                          of K (weight gradients: K is the token count) is copied from clamped
//                          rows and the left operand's fragments are masked.
// Fragment reads and the wait counters are written out by hand: the compiler would otherwise wait
// for every outstanding copy before any LDS read.
// The product is formed transposed (the B fragment is the left operand of the instruction), so a
// lane owns one output row and four consecutive columns per register quad; the tile goes through
// LDS once more so that global stores are whole 16-byte chunks of consecutive rows.
// The dimensions a kernel works with: those of the argument block, or what a device-side token count makes of them.
// waits until at most min(ahead, A) * LPS of this wavefront's copies are still in flight
template <int A, int LPS>
__device__ __forceinline__ void wait_ahead(int ahead) {
  if constexpr (A <= 0) {
    wait_vm<0>();
  } else {
    if (ahead >= A) wait_vm<A * LPS>();
    else wait_ahead<A - 1, LPS>(ahead);
  }
}
constexpr int kGemmThreads = 512;     // four computing wavefronts and four copy wavefronts
struct GemmDims {
  int M, K, splitk, kchunk, rs_n;
};
// KH (a 64-row tile of fp32 partial products from mn-contiguous operands on 64-k stages): the four computing
// wavefronts are two column halves x two halves of every K slice instead of 2 x 2 blocks of the tile.  A wavefront
// then owns all 64 rows, reads 2 KB + 2 KB of fragments per 16-k step instead of 1 KB + 2 KB for half the matrix
// instructions' worth of it (32 KB of LDS reads per slice instead of 48 KB, which is what bounds this tile), and
// the two K halves are added through LDS before the epilogue, lower half first.
// SUMS: column sums of B as well (GemmBf16::sum0 ..).
template <bool AKC, bool BKC, bool SPLIT, int BM, int BK, int NS, bool KH = false, bool SUMS = false>
__device__ __forceinline__ void gemm_async_tile(const GemmBf16& g, const GemmDims& dm, const int bx, const int by, const int bz) {
  static_assert(!SUMS || (SPLIT && !BKC), "column sums: of a weight gradient's right-hand operand");
  static_assert(!KH || (!AKC && !BKC && SPLIT && BM == 64 && BK == 64), "K halves: 64-row weight-gradient tiles on 64-k stages");
  constexpr int BN = 128, MI = KH ? 2 : BM / 64, KS = BK / 16;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int IA = A_BYTES / 4096, IB = B_BYTES / 4096, LPS = IA + IB;   // 1 KB copies per wavefront and stage
  constexpr int CH = BK / 8;                                              // 16-byte chunks per k-contiguous row
  constexpr int RPI = 64 / CH;                                            // ... and rows per copy instruction
  constexpr int CHA = BM / 8, RPA = 64 / CHA;                             // the same for an [k][BM] tile
  constexpr int CHB = BN / 8, RPB = 64 / CHB;                             // and an [k][BN] tile
  constexpr int OPK = (AKC ? MI : 2 * MI) + (BKC ? 2 : 4);                // LDS reads per 16-k step
  constexpr int ES = SPLIT ? 4 : 2;                                       // output element size
  constexpr int CPITCH = BN * ES + 16;                                    // LDS row pitch of the output tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = KH ? 0 : (wave >> 1) & 1, wn = wave & 1;
  const int kh = KH ? (wave >> 1) & 1 : 0;                                // which two of a slice's four 16-k steps
  constexpr int MROWS = KH ? BM : BM / 2;                                 // tile rows a computing wavefront covers
  const int col = lane & 31, half = lane >> 5;
  const int zb = SPLIT ? bz / dm.splitk : bz;
  const int kbeg = SPLIT ? (bz % dm.splitk) * dm.kchunk : 0;
  const int kend = SPLIT ? min(dm.K, kbeg + dm.kchunk) : dm.K;
  const int m0 = by * BM, n0 = bx * BN;
  const int nseg = g.nseg > 1 ? g.nseg : 1;
  const int nk = (kend - kbeg + BK - 1) / BK;
  const int total = nseg * nk;
  const int zsel = g.nseg > 1 ? 0 : zb;
  const bf16_t* A1 = g.A1; const bf16_t* B1 = g.B1;
  const bf16_t* A2 = g.A2; const bf16_t* B2 = g.B2;
  const bf16_t* A0 = zsel == 0 ? g.A0 : (zsel == 1 ? A1 : (zsel == 2 ? A2 : g.A3));
  const bf16_t* B0 = zsel == 0 ? g.B0 : (zsel == 1 ? B1 : (zsel == 2 ? B2 : g.B3));

  // ---- the copy wavefronts.  Wavefronts 4-7 do nothing but issue the asynchronous copies; wavefronts 0-3 never touch
  // global memory inside the loop.  A copy instruction holds its wavefront until the memory pipeline takes it
  // (300-500 clocks per slice for a wavefront's share), which would otherwise be time in which that wavefront
  // issues neither LDS reads nor matrix instructions; one wavefront alone cannot issue a whole slice fast enough
  // (about 32 bytes per clock), four reach the pipeline's 64-74.
  const bool producer = wave >= 4;
  const int w4 = wave & 3;
  // Source offsets (bytes) of this copy wavefront's share from a scalar base that moves with the slice: copy u fills LDS
  // bytes [1024 (4 u + w4), + 1024) of the operand
  //   k-contiguous: clamped row * ld + chunk * 8
  //   mn-contiguous: k-row (krowX + u * 4 * RPx) * ld + column; only in a slice that reaches past kend the k-row is clamped
  // (scalar slice offset and 32-bit lane offsets: see dma16_buf; with 64-bit addresses the copies bounded every tile)
  static_assert((NS - 2) * LPS < 64, "the copy counter holds at most 63");
  uint32_t goffA[IA], goffB[IB];
  uint32_t coffA[AKC ? 1 : IA], coffB[BKC ? 1 : IB];              // the column's part of it (mn-contiguous)
  int krowA = 0, krowB = 0;
  if (producer) {
#pragma unroll
    for (int u = 0; u < IA; ++u) {
      if constexpr (AKC) {
        const int row = (u * 4 + w4) * RPI + lane / CH;
        goffA[u] = (uint32_t)(min(m0 + row, dm.M - 1) * g.lda + ((lane % CH) ^ swz_kc<BK>(row)) * 8) * 2u;
      } else {
        const int krow = (u * 4 + w4) * RPA + lane / CHA;
        if (u == 0) krowA = krow;
        coffA[u] = (uint32_t)min(m0 + ((lane % CHA) ^ swz_nc<BM>(krow)) * 8, dm.M - 8) * 2u;
        goffA[u] = (uint32_t)(krow * g.lda) * 2u + coffA[u];
      }
    }
#pragma unroll
    for (int u = 0; u < IB; ++u) {
      if constexpr (BKC) {
        const int row = (u * 4 + w4) * RPI + lane / CH;
        goffB[u] = (uint32_t)(min(n0 + row, g.N - 1) * g.ldb + ((lane % CH) ^ swz_kc<BK>(row)) * 8) * 2u;
      } else {
        const int krow = (u * 4 + w4) * RPB + lane / CHB;
        if (u == 0) krowB = krow;
        coffB[u] = (uint32_t)min(n0 + ((lane % CHB) ^ swz_nc<BN>(krow)) * 8, g.N - 8) * 2u;
        goffB[u] = (uint32_t)(krow * g.ldb) * 2u + coffB[u];
      }
    }
  }
  // ---- fragment addresses (LDS bytes relative to a stage)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  uint32_t addrA[MI][AKC ? KS : 1], addrB[2][BKC ? KS : 1];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if constexpr (AKC) {
      const int ra = wm * MROWS + i * 32 + col;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) addrA[i][ks] = lds0 + ra * (BK * 2) + (((2 * ks + half) ^ swz_kc<BK>(ra)) * 16);
    } else {
      const int krow = 8 * half + ((lane & 15) >> 2);
      const int mn = wm * MROWS + i * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      addrA[i][0] = lds0 + krow * (BM * 2) + (((mn >> 3) ^ swz_nc<BM>(krow)) * 16) + ((mn >> 2) & 1) * 8 + kh * 32 * BM * 2;
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if constexpr (BKC) {
      const int rb = wn * 64 + j * 32 + col;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        addrB[j][ks] = lds0 + A_BYTES + rb * (BK * 2) + (((2 * ks + half) ^ swz_kc<BK>(rb)) * 16);
    } else {
      const int krow = 8 * half + ((lane & 15) >> 2);
      const int mn = wn * 64 + j * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      addrB[j][0] = lds0 + A_BYTES + krow * (BN * 2) + (((mn >> 3) ^ swz_nc<BN>(krow)) * 16) + ((mn >> 2) & 1) * 8 + kh * 32 * BN * 2;
    }
  }

  floatx16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = zero16();

  // ---- copy cursor (copy wavefront)
  int fseg = 0, fk = kbeg;
  copy_src Ap = copy_source(A0), Bp = copy_source(B0);
#define VD_ISSUE_STAGE(BUF)                                                                        \
  {                                                                                                \
    unsigned char* sp = smem + (BUF) * STAGE + w4 * 1024;                                          \
    const uint32_t sa = (uint32_t)(AKC ? fk : fk * g.lda) * 2u, sb = (uint32_t)(BKC ? fk : fk * g.ldb) * 2u;\
    if ((AKC && BKC) || fk + BK <= kend) {                                                         \
      _Pragma("unroll") for (int u = 0; u < IA; ++u) dma16_buf(Ap, goffA[u], sa, sp + u * 4096);   \
      _Pragma("unroll") for (int u = 0; u < IB; ++u) dma16_buf(Bp, goffB[u], sb, sp + A_BYTES + u * 4096);\
    } else {                                                                                       \
      const int last = kend - 1 - fk;                                                              \
      _Pragma("unroll") for (int u = 0; u < IA; ++u) {                                             \
        if constexpr (AKC) dma16_buf(Ap, goffA[u], sa, sp + u * 4096);                             \
        else dma16_buf(Ap, (uint32_t)(min(krowA + u * 4 * RPA, last) * g.lda) * 2u + coffA[u], sa, sp + u * 4096);\
      }                                                                                            \
      _Pragma("unroll") for (int u = 0; u < IB; ++u) {                                             \
        if constexpr (BKC) dma16_buf(Bp, goffB[u], sb, sp + A_BYTES + u * 4096);                   \
        else dma16_buf(Bp, (uint32_t)(min(krowB + u * 4 * RPB, last) * g.ldb) * 2u + coffB[u], sb, sp + A_BYTES + u * 4096);\
      }                                                                                            \
    }                                                                                              \
    fk += BK;                                                                                      \
    if (fk >= kend) {                                                                              \
      fk = kbeg;                                                                                   \
      ++fseg;                                                                                      \
      Ap = copy_source(fseg == 1 ? A1 : A2);                                                       \
      Bp = copy_source(fseg == 1 ? B1 : B2);                                                       \
    }                                                                                              \
  }
  // Column sums of B, by the copy wavefronts (which sizes: vd_attn_bf16_sums_inside; a launch of their own that reads B again took 11.5 + 5.0 us
  // for the four of 10 272 x 512, 5.7 + 2.3 for one of 3008 x 512; here dense training at 10 272 rows 196 -> 183 us a step, the
  // embedding of 3008 windows of 720 samples 35.0 -> 32.1).  Lane c + 16 j of copy wavefront w4 takes the eight columns of 16-byte chunk c in k-rows
  // BK / 4 w4 + j + {0, 4, ..} of every slice, adds those of a slice up first and the slices in order.
  float* sum_out = nullptr;
  float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (SUMS) {
    if (by == 0) sum_out = zsel == 0 ? g.sum0 : (zsel == 1 ? g.sum1 : (zsel == 2 ? g.sum2 : g.sum3));
  }
  if (producer) {
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < total) VD_ISSUE_STAGE(s)
    for (int t0 = 0; t0 < total; t0 += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int t = t0 + s;
        if (t < total) {
          // slice t has landed once at most `ahead` younger stages are still in flight
          const int ahead = min(total - 1 - t, NS - 2);
          wait_ahead<NS - 2, LPS>(ahead);
          __builtin_amdgcn_s_barrier();     // slice t is in; everyone is done with slice t-1, whose buffer is filled next
          if (t + NS - 1 < total) VD_ISSUE_STAGE((s + NS - 1) % NS)
          if constexpr (SUMS) {
            if (sum_out) {
              const int krow = (BK / 4) * w4 + (lane >> 4), live = kend - (kbeg + t * BK) - krow;
              const uint32_t at = lds0 + s * STAGE + A_BYTES + krow * (BN * 2) + (((lane & 15) ^ swz_nc<BN>(krow)) * 16);
              Frag f[4];
              lds_read16(f[0].q, at);
              lds_read16_at<4 * BN * 2>(f[1].q, at);
              if constexpr (BK == 64) {
                lds_read16_at<8 * BN * 2>(f[2].q, at);
                lds_read16_at<12 * BN * 2>(f[3].q, at);
                wait_lds<0>(f[0], f[1], f[2], f[3]);
              } else {
                wait_lds<0>(f[0], f[1]);
              }
#pragma unroll
              for (int i = 0; i < BK / 16; ++i)
                if (live <= 4 * i) f[i].q = u32x4{0u, 0u, 0u, 0u};       // (a k-row past the end repeats the last one)
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                float v = bf2f(f[0].h[e]) + bf2f(f[1].h[e]);
                if constexpr (BK == 64) v += bf2f(f[2].h[e]) + bf2f(f[3].h[e]);
                csum[e] += v;
              }
            }
          }
        }
      }
    }
  } else {
  for (int t0 = 0; t0 < total; t0 += NS) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int t = t0 + s;
      if (t < total) {
        __builtin_amdgcn_s_barrier();     // the copy wavefront has seen slice t land
        const uint32_t so = s * STAGE;
        // valid k of this lane's first fragment; only the last slice of an mn-contiguous A can fall short
        int kvalid = 8;
        if constexpr (!AKC) kvalid = t == total - 1 ? kend - (kbeg + (nk - 1) * BK + 8 * half + 32 * kh) : 8 + 16 * KS;
        Frag fa[2][2], fb[2][2];
#define VD_READ_STEP(KS_, SET)                                                                     \
  {                                                                                                \
    _Pragma("unroll") for (int i = 0; i < MI; ++i) {                                               \
      if constexpr (AKC) {                                                                         \
        lds_read16(fa[SET][i].q, addrA[i][AKC ? (KS_) : 0] + so);                                  \
      } else {                                                                                     \
        lds_read8_tr<(KS_) * 16 * BM * 2>(fa[SET][i].d[0], addrA[i][0] + so);                      \
        lds_read8_tr<(KS_) * 16 * BM * 2 + 4 * BM * 2>(fa[SET][i].d[1], addrA[i][0] + so);         \
      }                                                                                            \
    }                                                                                              \
    _Pragma("unroll") for (int j = 0; j < 2; ++j) {                                                \
      if constexpr (BKC) {                                                                         \
        lds_read16(fb[SET][j].q, addrB[j][BKC ? (KS_) : 0] + so);                                  \
      } else {                                                                                     \
        lds_read8_tr<(KS_) * 16 * BN * 2>(fb[SET][j].d[0], addrB[j][0] + so);                      \
        lds_read8_tr<(KS_) * 16 * BN * 2 + 4 * BN * 2>(fb[SET][j].d[1], addrB[j][0] + so);         \
      }                                                                                            \
    }                                                                                              \
  }
#define VD_MFMA_STEP(KS_, SET, PENDING)                                                            \
  {                                                                                                \
    if constexpr (MI == 2) wait_lds<PENDING>(fa[SET][0], fa[SET][1], fb[SET][0], fb[SET][1]);      \
    else wait_lds<PENDING>(fa[SET][0], fb[SET][0], fb[SET][1]);                                    \
    if constexpr (!AKC) {                                                                          \
      if (kvalid - 16 * (KS_) < 8) {                                                               \
        _Pragma("unroll") for (int i = 0; i < MI; ++i) mask_frag(fa[SET][i], kvalid - 16 * (KS_)); \
      }                                                                                            \
    }                                                                                              \
    _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                 \
      _Pragma("unroll") for (int j = 0; j < 2; ++j) acc[i][j] = mfma(fb[SET][j], fa[SET][i], acc[i][j]); \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
        VD_READ_STEP(0, 0)
        if constexpr (KS == 2 || KH) {
          VD_READ_STEP(1, 1)
          VD_MFMA_STEP(0, 0, OPK)
          VD_MFMA_STEP(1, 1, 0)
        } else {
          VD_READ_STEP(1, 1)
          VD_MFMA_STEP(0, 0, OPK)
          VD_READ_STEP(2, 0)
          VD_MFMA_STEP(1, 1, OPK)
          VD_READ_STEP(3, 1)
          VD_MFMA_STEP(2, 0, OPK)
          VD_MFMA_STEP(3, 1, 0)
        }
#undef VD_READ_STEP
#undef VD_MFMA_STEP
      }
    }
  }
  }
#undef VD_ISSUE_STAGE

  // ---- epilogue.  acc[i][j] register 4*q4 + e is C[wm*MROWS + i*32 + col][wn*64 + j*32 + 8*q4 + 4*half + e]
  // of the tile; it is written to LDS (with the bias), then stored as 16-byte chunks of whole rows.
  const bf16_t* bias = SPLIT ? nullptr : (zsel == 0 ? g.bias0 : (zsel == 1 ? g.bias1 : (zsel == 2 ? g.bias2 : g.bias3)));
  __syncthreads();                        // every wavefront is done reading the last slice
  float* csum_lds = reinterpret_cast<float*>(smem + BM * CPITCH);         // [4 copy wavefronts][128 columns], behind the tile
  if constexpr (SUMS) {
    if (sum_out && producer) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        csum[e] += __shfl_xor(csum[e], 16, 64);
        csum[e] += __shfl_xor(csum[e], 32, 64);
        if (lane < 16) csum_lds[w4 * BN + 8 * lane + e] = csum[e];
      }
    }
  }
  if constexpr (KH) {
    // the upper K half hands its sums over through LDS; the lower half adds them to its own (lower + upper)
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (!producer && kh == 1 - pass) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
            for (int i = 0; i < MI; ++i) {
              float4* p = reinterpret_cast<float4*>(smem + (i * 32 + col) * CPITCH + (wn * 64 + j * 32 + 8 * q4 + 4 * half) * 4);
              if (pass == 0) {
                *p = make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
              } else {
                const float4 v = *p;
                acc[i][j][4 * q4] += v.x; acc[i][j][4 * q4 + 1] += v.y; acc[i][j][4 * q4 + 2] += v.z; acc[i][j][4 * q4 + 3] += v.w;
              }
            }
      }
      if (pass == 0) __syncthreads();
    }
    // (a lane of the lower half reads and rewrites only its own elements: no barrier in between)
  }
  if (!producer && kh == 0)
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if constexpr (SPLIT) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int i = 0; i < MI; ++i)
          *reinterpret_cast<float4*>(smem + (wm * MROWS + i * 32 + col) * CPITCH + (wn * 64 + j * 32 + 8 * q4 + 4 * half) * 4) =
              make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
    } else {
#pragma unroll
      for (int g2 = 0; g2 < 4; g2 += 2) {
        float bv[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        if (bias) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int n = n0 + wn * 64 + j * 32 + 8 * (g2 + e) + 4 * half;
            if (n < g.N) {                         // N is a multiple of 8: a quad is inside or outside
              const u32x2 b4 = *reinterpret_cast<const u32x2*>(bias + n);
              bv[e][0] = __uint_as_float(b4.x << 16); bv[e][1] = __uint_as_float(b4.x & 0xffff0000u);
              bv[e][2] = __uint_as_float(b4.y << 16); bv[e][3] = __uint_as_float(b4.y & 0xffff0000u);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          u32x2 o[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 4 * (g2 + e);
            o[e].x = pack2(acc[i][j][r] + bv[e][0], acc[i][j][r + 1] + bv[e][1]);
            o[e].y = pack2(acc[i][j][r + 2] + bv[e][2], acc[i][j][r + 3] + bv[e][3]);
          }
          *reinterpret_cast<u32x4*>(smem + (wm * MROWS + i * 32 + col) * CPITCH + (wn * 64 + j * 32 + 8 * (g2 + half)) * 2) = quads16(o[0], o[1]);
        }
      }
    }
  __syncthreads();
  constexpr int CPR = BN * ES / 16;          // 16-byte chunks per tile row
  constexpr int EPC = 16 / ES;               // elements per chunk
  unsigned char* Cb;
  long long ldc_bytes;
  if constexpr (SPLIT) {
    if (dm.splitk > 1 || g.force_part) {      // partial product of slice bz % splitk of matrix bz / splitk
      Cb = reinterpret_cast<unsigned char*>(g.part) + (long long)bz * dm.M * g.N * 4;
      ldc_bytes = (long long)g.N * 4;
    } else {                 // a single slice is the result itself
      Cb = reinterpret_cast<unsigned char*>(zsel == 0 ? g.C0 : (zsel == 1 ? g.C1 : (zsel == 2 ? g.C2 : g.C3)));
      ldc_bytes = (long long)g.ldc * 4;
    }
  } else {
    Cb = reinterpret_cast<unsigned char*>(zsel == 0 ? g.C0 : (zsel == 1 ? g.C1 : (zsel == 2 ? g.C2 : g.C3)));
    ldc_bytes = (long long)g.ldc * 2;
  }
  if constexpr (SUMS) {
    const int c = threadIdx.x - 256;
    if (sum_out && producer && c < BN && n0 + c < g.N) {
      if (dm.splitk > 1) sum_out = g.sum_part + (long long)bz * g.N;
      sum_out[n0 + c] = ((csum_lds[c] + csum_lds[BN + c]) + csum_lds[2 * BN + c]) + csum_lds[3 * BN + c];
    }
  }
  if (producer) return;                   // (no barrier follows)
#pragma unroll
  for (int u = 0; u < BM * CPR / 256; ++u) {
    const int idx = u * 256 + threadIdx.x;
    const int row = idx / CPR, c = idx % CPR;
    if (m0 + row < dm.M && n0 + c * EPC < g.N) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(smem + row * CPITCH + c * 16);
      *reinterpret_cast<u32x4*>(Cb + (long long)(m0 + row) * ldc_bytes + (long long)(n0 + c * EPC) * ES) = v;
    }
  }
  if constexpr (!SPLIT) {
    // per-head row sums of C * rs_o (see GemmBf16) from the rounded tile in LDS: a pair of neighbouring lanes
    // takes the two 32-column halves of one head of one row, each in ascending column order
    if (g.rs_out) {
#pragma unroll
      for (int u = 0; u < BM * 4 / 256; ++u) {
        const int idx = u * 256 + threadIdx.x;
        const int row = idx >> 2, c0 = ((idx >> 1) & 1) * 64 + (idx & 1) * 32;
        const int m = m0 + row;
        const bool live = m < dm.M && n0 + c0 < g.N;
        float p = 0.f;
        if (live) {
          const bf16_t* orow = g.rs_o + (long long)m * g.ldc + n0 + c0;
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4) {
            const u32x4 cv = *reinterpret_cast<const u32x4*>(smem + row * CPITCH + (c0 + 8 * v4) * 2);
            const u32x4 ov = *reinterpret_cast<const u32x4*>(orow + 8 * v4);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              p = fmaf(__uint_as_float(cv[w] << 16), __uint_as_float(ov[w] << 16), p);
              p = fmaf(__uint_as_float(cv[w] & 0xffff0000u), __uint_as_float(ov[w] & 0xffff0000u), p);
            }
          }
        }
        p += __shfl_xor(p, 1, 64);
        if (live && (idx & 1) == 0) {
          const int b = m / dm.rs_n;
          const long long i = ((long long)b * g.rs_H + ((n0 + c0) >> 6)) * dm.rs_n + (m - b * dm.rs_n);
          g.rs_out[i] = g.rs_mul * p;
          if (g.rs_aux_out) g.rs_aux_out[i] = g.rs_aux_mul * g.rs_aux_in[i];
        }
      }
    }
  }
}

// LDS a workgroup of the asynchronous GEMM needs: the staging ring, or the output tile (and column sums behind it) if that is larger
template <bool SPLIT, int BM, int BK, int NS, bool SUMS = false>
constexpr int gemm_async_lds() {
  constexpr int ring = NS * (BM + 128) * BK * 2, out = BM * (128 * (SPLIT ? 4 : 2) + 16) + (SUMS ? 4 * 128 * 4 : 0);
  return ring > out ? ring : out;
}
template <bool SPLIT, int BM, int BK, int NS, bool SUMS = false>
constexpr int gemm_async_lds_v = gemm_async_lds<SPLIT, BM, BK, NS, SUMS>();
// The product's dimensions, with a device-side token count (GemmBf16::n_dev) resolved; false: nothing to do.  EMBED: K slices by the
// embedding's rule (n_role 2), else by the attention's.  (Both in one kernel: code that the gradient launch never runs, and with
// some versions of it that launch takes 2-4 % longer: 55.5 -> 57.9 us of a backward pass of 3584 rows of 576.)
template <bool EMBED>
__device__ __forceinline__ bool gemm_resolve(const GemmBf16& g, GemmDims& dm) {
  dm.M = g.M; dm.K = g.K; dm.splitk = g.splitk; dm.kchunk = g.kchunk; dm.rs_n = g.rs_n;
  if (!g.n_dev) return true;
  int n;
  if (!vd_count(g.n_dev, g.n_max, n, g.status)) return false;
  if (g.n_role == 0) {
    dm.M = g.n_mul * n;
    dm.rs_n = n;
  } else {
    dm.K = g.n_mul * n;
    int kchunk = 64;
    if constexpr (EMBED) dm.splitk = vd_embed_splitk(g.M, g.N, (long long)dm.K, &kchunk);
    else dm.splitk = vd_attn_bf16_splitk(g.M, (long long)dm.K, g.many != 0, &kchunk);
    dm.kchunk = kchunk;
  }
  // (no tokens: an input gradient has no rows to write; a weight gradient is all zeros, which its tiles write
  // themselves: a product over no slices)
  if (g.n_role != 0 && dm.K == 0) {
    dm.splitk = 1;
    dm.kchunk = 64;
    return dm.M > 0;
  }
  return dm.M > 0 && dm.K > 0;
}
// One-dimensional grid of at least nz * tiles workgroups (more when the launch was sized for the bound of a
// device-side count: the surplus returns at once).
template <bool AKC, bool BKC, bool SPLIT, int BM, int BK, int NS, bool SUMS = false>
// (wavefronts a SIMD: two or three workgroups share a compute unit)
__global__ __launch_bounds__(kGemmThreads, BM == 128 || NS > 2 ? 4 : 6) void gemm_async_kernel(GemmBf16 g, int nz) {
  GemmDims dm;
  if (!gemm_resolve<SPLIT>(g, dm)) return;
  // tiles in the order n fastest, then m, then batch entry: a die's range shares its rows of A
  const int gx = (g.N + 127) >> 7, gy = (dm.M + BM - 1) / BM;
  const int total = gx * gy * nz * (SPLIT ? dm.splitk : 1);
  if ((int)blockIdx.x >= total) return;
  const int t = xcd_contiguous(blockIdx.x, total);
  gemm_async_tile<AKC, BKC, SPLIT, BM, BK, NS, false, SUMS>(g, dm, t % gx, (t / gx) % gy, t / (gx * gy));
}
// The input gradient (gx: k-contiguous operands, up to three accumulated segments) and the weight
// gradients (gw: mn-contiguous operands, K slices, fp32 partial products) depend on the same dQ, dK,
// dV and on nothing of each other, so they share one launch.
// Tile shapes of the two kinds of workgroup: rows, k per copy stage, stages (BN = 128 always).
template <int BMX_, int BKX_, int NSX_, int BMW_, int BKW_, int NSW_, bool KHW_, bool SUMS_>
struct PairCfg {
  static constexpr int BMX = BMX_, BKX = BKX_, NSX = NSX_, BMW = BMW_, BKW = BKW_, NSW = NSW_;
  static constexpr bool SUMS = SUMS_;              // bias gradients as well
  static constexpr bool KHW = KHW_;                // the weight-gradient tiles' wavefronts split every K slice in halves
  static constexpr int ldsx = gemm_async_lds_v<false, BMX_, BKX_, NSX_>, ldsw = gemm_async_lds_v<true, BMW_, BKW_, NSW_, SUMS_>;
  static constexpr int lds = ldsx > ldsw ? ldsx : ldsw;
};
// few tokens: 128-row input-gradient tiles beside 64-row weight-gradient tiles (wavefronts in K halves), both on
// three 64-k stages (96 KB of LDS; with two stages an input-gradient tile waits 1000 of 1700 clocks per slice for
// its copies), one slice;
// many tokens: 128-row tiles for both, input gradients on two 64-k stages (whole 128-byte lines of their k-contiguous rows;
// on four 32-k stages 174 -> 161 us at 15 400 rows of 768, 34.2 -> 30.6 at 6080 of 512), weight gradients on four 32-k stages
// (two of 64 k: 168 us) (64 KB); three or four 64-k stages leave one workgroup a compute unit: 192 us
template <bool SUMS> using PairSmall = PairCfg<128, 64, 3, 64, 64, 3, true, SUMS>;
template <bool SUMS> using PairLarge = PairCfg<128, 64, 2, 128, 32, 4, false, SUMS>;
template <typename CFG>
__global__ __launch_bounds__(kGemmThreads, CFG::KHW ? 2 : 4) void gemm_bwd_pair_kernel(GemmBf16 gx, GemmBf16 gw, int nzw) {
  // Each die takes a contiguous range of the input-gradient tiles (n fastest: a range shares its rows
  // of dQ, dK, dV) and a contiguous range of the weight-gradient tiles (n, then m, then K slice, then
  // matrix: a range shares its K slice of both operands).  The kind whose tiles walk over more K comes first, so that a late
  // start never meets a long tile (with the input gradient always first, at 15 400 rows of 768 its 726 tiles of 36 slices held
  // up the 288 weight-gradient tiles of 120: 161 us, 127 this way).  Whole backward, input gradient first -> by this rule:
  //   many tokens: d = 512 106 -> 102 us at 10 272 rows, 343 -> 310 at 27 584; d = 768 274 -> 257 at 15 400; d = 1024 259 -> 236 at 9600,
  //     153 -> 141 at 5760, but 124 -> 132 at 4224 (32 tiles more than the chip has places);
  //   few tokens: d = 512 and less within 0.3 %; d = 576 53.3 -> 47.4 at 3520, d = 640 52.3 -> 50.5 at 2784, d = 832 104 -> 98.4 at 4576;
  //     d = 704 55.0 -> 56.7 at 3200, d = 768 57.4 -> 58.9 at 3200, 59.7 -> 62.2 at 3520 (264 and 288 weight-gradient tiles on 256 places),
  //     81.8 -> 80.8 at 4224.
  GemmDims dx, dw;
  const bool has_x = gemm_resolve<false>(gx, dx);
  if (!gemm_resolve<false>(gw, dw)) return;          // (an invalid count; with no tokens only the weight-gradient tiles run)
  if (!has_x) dx.M = 0;
  constexpr int BMX = CFG::BMX, BMW = CFG::BMW;
  const int gxn = (gx.N + 127) >> 7, gwn = (gw.N + 127) >> 7, gwm = (dw.M + BMW - 1) / BMW;
  const int nx = gxn * ((dx.M + BMX - 1) / BMX), nw = gwn * gwm * nzw * dw.splitk;
  if ((int)blockIdx.x >= nx + nw) return;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const bool w_first = dw.kchunk > 3 * gx.K;
  const int n1 = w_first ? nw : nx;
  const int cnt1 = (n1 >> 3) + (xcd < (n1 & 7) ? 1 : 0), start1 = xcd_range_start(xcd, n1);
  const bool first = slot < cnt1;
  const int t = first ? start1 + slot : xcd_range_start(xcd, nx + nw) - start1 + (slot - cnt1);
  if (first != w_first) {
    gemm_async_tile<true, true, false, BMX, CFG::BKX, CFG::NSX>(gx, dx, t % gxn, t / gxn, 0);
  } else {
    gemm_async_tile<false, false, true, BMW, CFG::BKW, CFG::NSW, CFG::KHW, CFG::SUMS>(gw, dw, t % gwn, (t / gwn) % gwm, t / (gwn * gwm));
  }
}

// Tile and pipeline depth of the asynchronous GEMM: 128 x 128 tiles once there are enough of them to
// keep every compute unit busy with two workgroups; otherwise 64 x 128 tiles, three stages deep while
// two workgroups still fit beside each other in LDS (at most 512 tiles), else two stages and three
// workgroups per compute unit.
template <bool AKC, bool BKC, bool SPLIT, int BM, int NS, bool SUMS = false>
int launch_gemm_async_cfg(vardrop_ctx* ctx, int kid, const GemmBf16& g, int nz, hipStream_t s) {
  constexpr int BK = 64;
  constexpr int lds = gemm_async_lds<SPLIT, BM, BK, NS, SUMS>();
  static int configured_device = -1;     // raising the dynamic LDS limit is a per-device, per-function setting
  if (configured_device != ctx->device) {
    VD_HIP(ctx, hipFuncSetAttribute((const void*)gemm_async_kernel<AKC, BKC, SPLIT, BM, BK, NS, SUMS>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    configured_device = ctx->device;
  }
  // (with a device-side count g.M or g.K and g.splitk hold the bounds the grid is sized for)
  const long long grid = (long long)vd_ceil_div(g.N, 128) * vd_ceil_div(g.M, BM) * nz * (SPLIT ? g.splitk : 1);
  if (grid >= (1ll << 31)) return VARDROP_EUNSUPPORTED;
  {
    VdTimer timer(ctx, kid, s);
    VD_KERNEL(ctx, (gemm_async_kernel<AKC, BKC, SPLIT, BM, BK, NS, SUMS>), dim3((unsigned)grid), dim3(kGemmThreads), lds, s, g, nz);
  }
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}
// one launch for the input gradient gx and the sliced weight gradients gw (nzw matrices)
template <typename CFG>
int launch_gemm_bwd_pair_cfg(vardrop_ctx* ctx, const GemmBf16& gx, const GemmBf16& gw, int nzw, hipStream_t s) {
  constexpr int lds = CFG::lds;
  static int configured_device = -1;
  if (configured_device != ctx->device) {
    VD_HIP(ctx, hipFuncSetAttribute((const void*)gemm_bwd_pair_kernel<CFG>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    configured_device = ctx->device;
  }
  const int gxn = vd_ceil_div(gx.N, 128), gxm = vd_ceil_div(gx.M, CFG::BMX);
  const int gwn = vd_ceil_div(gw.N, 128), gwm = vd_ceil_div(gw.M, CFG::BMW);
  const int nx = gxn * gxm, nw = gwn * gwm * nzw * gw.splitk;
  {
    VdTimer timer(ctx, VARDROP_K_GEMM_DW_DXS, s);
    VD_KERNEL(ctx, gemm_bwd_pair_kernel<CFG>, dim3(nx + nw), dim3(kGemmThreads), lds, s, gx, gw, nzw);
  }
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}
int launch_gemm_bwd_pair(vardrop_ctx* ctx, const GemmBf16& gx, const GemmBf16& gw, int nzw, hipStream_t s) {
  if (gx.K % 64 != 0 || gx.N % 8 != 0 || (long long)gx.M * gx.lda >= (1ll << 31) || (long long)gx.N * gx.ldb >= (1ll << 31) ||
      gw.M % 8 != 0 || gw.N % 8 != 0 || gw.kchunk % 64 != 0 || gw.splitk < 1 ||
      (long long)gw.K * gw.lda >= (1ll << 31) || (long long)gw.K * gw.ldb >= (1ll << 31))
    return VARDROP_EUNSUPPORTED;
  // (with a device-side count the choice is made for its bound, tiles and slices alike)
  const bool sums = gw.sum0 || gw.sum1 || gw.sum2 || gw.sum3;
  if (gw.many) return sums ? launch_gemm_bwd_pair_cfg<PairLarge<true>>(ctx, gx, gw, nzw, s) : launch_gemm_bwd_pair_cfg<PairLarge<false>>(ctx, gx, gw, nzw, s);
  return sums ? launch_gemm_bwd_pair_cfg<PairSmall<true>>(ctx, gx, gw, nzw, s) : launch_gemm_bwd_pair_cfg<PairSmall<false>>(ctx, gx, gw, nzw, s);
}

template <bool BKC>
int launch_gemm_async(vardrop_ctx* ctx, int kid, const GemmBf16& g, int nz, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return VARDROP_OK;
  if ((g.K % 64 != 0 && (BKC || !g.a_kpad)) || g.N % 8 != 0 || (long long)g.M * g.lda >= (1ll << 31) ||
      (long long)g.K * g.ldb >= (1ll << 31))
    return VARDROP_EUNSUPPORTED;
  if (g.rs_out && (nz != 1 || g.nseg > 1 || g.N % 64 != 0 || g.rs_n <= 0 || g.M % g.rs_n != 0)) return VARDROP_EUNSUPPORTED;
  const long long t128 = (long long)vd_ceil_div(g.N, 128) * vd_ceil_div(g.M, 128) * nz;
  const long long t64 = (long long)vd_ceil_div(g.N, 128) * vd_ceil_div(g.M, 64) * nz;
  if (t128 >= 512) return launch_gemm_async_cfg<true, BKC, false, 128, 2>(ctx, kid, g, nz, s);
  if (t64 <= 512) return launch_gemm_async_cfg<true, BKC, false, 64, 3>(ctx, kid, g, nz, s);
  return launch_gemm_async_cfg<true, BKC, false, 64, 2>(ctx, kid, g, nz, s);
}

}  // namespace

int vd_gemm_bf16(vardrop_ctx* ctx, int kid, const GemmBf16& g, int nz, bool b_k_contiguous, hipStream_t s) {
  return b_k_contiguous ? launch_gemm_async<true>(ctx, kid, g, nz, s) : launch_gemm_async<false>(ctx, kid, g, nz, s);
}

int vd_gemm_bf16_bwd_pair(vardrop_ctx* ctx, const GemmBf16& gx, const GemmBf16& gw, int nzw, hipStream_t s) {
  return launch_gemm_bwd_pair(ctx, gx, gw, nzw, s);
}

int vd_gemm_bf16_wgrad_split(vardrop_ctx* ctx, int kid, const GemmBf16& g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return VARDROP_OK;
  if (g.M % 8 != 0 || g.N % 8 != 0 || g.splitk < 1 || g.kchunk % 64 != 0 || (g.n_dev && g.n_role != 2) ||
      (long long)g.K * g.lda >= (1ll << 31) || (long long)g.K * g.ldb >= (1ll << 31))
    return VARDROP_EUNSUPPORTED;
  // (three stages: with two 20.9 -> 15.0 us and their sum at 27 584 rows of 96 x 512, 26.6 -> 25.5 at 10 272 of 720 x 512)
  if (g.sum0) return launch_gemm_async_cfg<false, false, true, 64, 3, true>(ctx, kid, g, 1, s);
  return launch_gemm_async_cfg<false, false, true, 64, 3>(ctx, kid, g, 1, s);
}

int vd_gemm_bf16_sum_rows(vardrop_ctx* ctx, const float* part, float* out0, long long count0, float* out1, long long count1,
                          long long stride, int splitk, hipStream_t s, const GemmBf16* like) {
  SplitkReduceRows r = {};
  if (like && like->n_dev) {
    r.n_dev = like->n_dev;
    r.n_max = like->n_max;
    r.n_mul = like->n_mul;
    r.dn_m = like->M;
    r.dn_n = like->N;
  }
  r.part = part;
  r.out0 = out0;
  r.out1 = out1;
  r.count0 = count0;
  r.count1 = count1;
  r.stride = stride;
  r.splitk = splitk;
  {
    VdTimer timer(ctx, VARDROP_K_REDUCE_DW, s);
    VD_KERNEL(ctx, splitk_reduce_rows_kernel, dim3((unsigned)((count0 + count1 + 255) / 256)), dim3(256), 0, s, r);
  }
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}

int vd_gemm_bf16_sum_slices(vardrop_ctx* ctx, const float* part, float* const out[4], long long count, int splitk,
                            hipStream_t s, const GemmBf16& gw, int nz) {
  SplitkReduce r = {};
  if (gw.n_dev) {
    r.n_dev = gw.n_dev;
    r.n_max = gw.n_max;
    r.n_mul = gw.n_mul;
    r.dn_d = gw.M;
    r.many = gw.many;
  }
  r.sum_part = gw.sum_part;
  r.sum[0] = gw.sum0; r.sum[1] = gw.sum1; r.sum[2] = gw.sum2; r.sum[3] = gw.sum3;
  r.N = gw.N;
  r.part = part;
  for (int z = 0; z < nz; ++z) r.out[z] = out[z];
  r.count = count;
  r.splitk = splitk;
  r.blocks = vd_ceil_div((int)(count / 4), 256);
  {
    VdTimer timer(ctx, VARDROP_K_REDUCE_DW, s);
    const bool sums = r.sum_part && (r.sum[0] || r.sum[1] || r.sum[2] || r.sum[3]);
    VD_KERNEL(ctx, splitk_reduce_kernel, dim3(r.blocks + (sums ? vd_ceil_div(r.N, 256) : 0), nz), dim3(256), 0, s, r);
  }
  VD_LAUNCH_CHECK(ctx);
  return VARDROP_OK;
}
