// Grouping by hash and stratified sampling (Sec. 3.3, Eq. 1-2).
//
// Every quantity the step needs of a variate n is a count over all variates m:
//   start(n) = #{h_m < h_n}                        its group's place in the order of hashes,
//   size(n)  = #{h_m = h_n}                        the group's size,
//   rank(n)  = #{h_m = h_n, (u_m, m) < (u_n, n)}   its place in the random order of the group,
// with u[n] from Philox4x32-10, counter (n, 0, step_lo, step_hi), key (seed_lo, seed_hi), or a caller's key.  n is kept
// when rank(n) < n_i(size).  Counting needs no order, no atomics on shared buckets and no exchange between workgroups,
// so it spreads over the chip (N = 8192: 28 us with all hashes different, 35 with 1756 groups, 63 with one):
//   1. rank_kernel: a workgroup owns 16 (above 4096 variates 32) variates; its wavefronts share out the m.  The result
//      is left packed in group_id[n].
//   2. select_kernel, one workgroup: dense group ids (a bitmap of the occupied starts and its prefix sums) and the kept
//      variates in ascending order.
// Up to 192 variates one workgroup does both in one launch.
// Measured (both launches; before: one workgroup ordering the variates in LDS): N = 32 3.0 us (8.1), 321 4.3 + 1.8
// (9.5), 862 6.3 + 2.1 (14.0), 2048 8.9 + 4.7 (25.5), 8192 34 + 5.8 (142).
#include <type_traits>
#include "common.h"

namespace {

constexpr int kMaxN = 8192;
constexpr int kSmallSample = 192;           // variates one workgroup handles in one launch
                                            // (192: 7.0 us, two launches 6.3 and 1-2 us more for a call alone; 220: 8.8
                                            // against 6.5, 256: 10.0 against 6.4; 137: 5.7 against 6.1)

__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     uint32_t k0, uint32_t k1, uint32_t& r0, uint32_t& r1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    c0 = hi1 ^ c1 ^ k0;
    c1 = lo1;
    c2 = hi0 ^ c3 ^ k1;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  r0 = c0;
  r1 = c1;
}

// Inclusive prefix sum over the 64 lanes: four shifts inside the rows of 16 lanes, then the last lane of a row is
// added to the next row and lane 31 to the upper half (lanes a step does not reach add zero).
__device__ inline int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return v;
}
struct SampleArgs {
  const uint64_t* hash;
  int32_t* group_id;
  int32_t* sel;
  int32_t* counts;
  int N;
  uint32_t gs, num, den;
  uint32_t seed_lo, seed_hi, step_lo, step_hi;
  const uint64_t* ext_keys;   // optional: key of variate n that orders the members of a group, instead of a Philox draw
  uint64_t* step_dev;         // optional: the step counter lives in device memory (read here instead of step_lo / step_hi)
  int advance;                //   and is incremented once the draw is done, so that a recorded launch draws anew when replayed
};

// members kept from a group of `size` (Eq. 1 with the optional keep ratio)
__device__ inline uint32_t keep_count(uint32_t size, const SampleArgs& a) {
  uint64_t by_ratio = ((uint64_t)size * a.num + a.den - 1) / a.den;
  if (by_ratio < 1) by_ratio = 1;
  uint32_t keep = by_ratio < size ? (uint32_t)by_ratio : size;
  if (a.gs != 0 && keep > a.gs) keep = a.gs;
  return keep;
}

__device__ inline void read_step(SampleArgs& a) {
  if (a.step_dev) {
    const uint64_t step = *a.step_dev;
    a.step_lo = (uint32_t)step;
    a.step_hi = (uint32_t)(step >> 32);
  }
}
// the key that orders variate n inside its group
__device__ inline uint64_t member_key(const SampleArgs& a, int n) {
  if (a.ext_keys) return a.ext_keys[n];
  uint32_t r0, r1;
  philox4x32_10((uint32_t)n, 0u, a.step_lo, a.step_hi, a.seed_lo, a.seed_hi, r0, r1);
  return ((uint64_t)r0 << 32) | r1;
}
// What rank_kernel leaves for select_kernel: start (13 bits), kept, first of its group.
constexpr uint32_t kStartMask = 0x1fffu, kKept = 0x2000u, kFirst = 0x4000u;
__device__ inline uint32_t pack_rank(const SampleArgs& a, int start, int size, int rank) {
  return (uint32_t)start | ((uint32_t)rank < keep_count((uint32_t)size, a) ? kKept : 0u) | (rank == 0 ? kFirst : 0u);
}

// ---- step 2: `nt` threads (a multiple of 64), thread t holds the packed results of variates t, t + nt, ... in v.
struct SelectLds {
  uint32_t bits[kMaxN / 32];                // which starts are occupied,
  int before[kMaxN / 32];                   // groups that start before a word of them,
  int kept[8 * 16];                         // kept variates of a wavefront's 64, then of all before
};
template <int E>
__device__ inline void select_phase(const SampleArgs& a, const uint32_t (&v)[E], SelectLds& s, int nt) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6, N = a.N;
  for (int i = tid; i < kMaxN / 32; i += nt) s.bits[i] = 0;
  __syncthreads();
  unsigned long long kept[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool live = e * nt + tid < N;
    if (live && (v[e] & kFirst)) atomicOr(&s.bits[(v[e] & kStartMask) >> 5], 1u << (v[e] & 31));
    kept[e] = __ballot(live && (v[e] & kKept));
    if (lane == 0) s.kept[e * nw + wave] = __popcll(kept[e]);
  }
  __syncthreads();
  if (wave == 0) {                          // kept variates before every wavefront's share: at most 128 counts
    const int n = E * nw;
    const int c0 = 2 * lane < n ? s.kept[2 * lane] : 0, c1 = 2 * lane + 1 < n ? s.kept[2 * lane + 1] : 0;
    const int incl = wave_inclusive_sum(c0 + c1);
    if (2 * lane < n) s.kept[2 * lane] = incl - c0 - c1;
    if (2 * lane + 1 < n) s.kept[2 * lane + 1] = incl - c1;
    if (lane == 63) a.counts[0] = incl;
  }
  if (wave == nw - 1) {                     // groups before every word of the bitmap
    int c[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c[i] = __popc(s.bits[4 * lane + i]);
      sum += c[i];
    }
    const int incl = wave_inclusive_sum(sum);
    int run = incl - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s.before[4 * lane + i] = run;
      run += c[i];
    }
    if (lane == 63) a.counts[1] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = e * nt + tid;
    if (n < N) {
      const uint32_t start = v[e] & kStartMask;
      a.group_id[n] = s.before[start >> 5] + __popc(s.bits[start >> 5] & ((1u << (start & 31)) - 1u));
      if (v[e] & kKept) a.sel[s.kept[e * nw + wave] + __popcll(kept[e] & ((1ull << lane) - 1ull))] = n;
    }
  }
  // (every launch of the step that reads the counter has done so: this one is the last)
  if (tid == 0 && a.step_dev && a.advance) *a.step_dev = *a.step_dev + 1;
}

// ---- step 1.  T variates per workgroup: lane l of every wavefront counts for variate l % T over one of the 64 / T
// values of m that a wavefront takes at a time.  Two passes.  The first compares 32 bits of the hashes, the topmost that
// any of them uses (all of them, for most): smaller ones count towards start, equal ones flag the m for the second, which
// compares whole hashes and the members' keys.  The keys are drawn for the flagged m only.
// Bound by the vector pipe (the first pass: N^2 / 64 comparisons of about six instructions, spread over the chip) and, for
// few variates, by the latency of its five phases.
constexpr int kRankThreads = 1024;
template <int T>
__global__ __launch_bounds__(kRankThreads) void rank_kernel(SampleArgs a) {
  constexpr int NT = kRankThreads, M = 64 / T, STEP = (NT / 64) * M;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int N = a.N, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t* __restrict__ hash = a.hash;
  uint64_t* hs = reinterpret_cast<uint64_t*>(smem);                    // [N] hashes
  uint64_t* us = hs + N;                                               // [N] keys of the listed variates; before that
  uint32_t* ks = reinterpret_cast<uint32_t*>(us);                      //     [N] 32 bits of the hashes and
  uint8_t* flag = reinterpret_cast<uint8_t*>(ks + N);                  //     [N] flags of the variates to list
  uint16_t* list = reinterpret_cast<uint16_t*>(us + N);                // [N]
  int* cnt = reinterpret_cast<int*>(smem + (((size_t)N * 18 + 15) & ~(size_t)15));   // [3][T],
  int* nlist = cnt + 3 * T;                                            // the list's length,
  int* level = nlist + 1;                                              // and how many bytes the widest hash has beyond 4
  read_step(a);
  const int n = blockIdx.x * T + lane % T;
  const bool valid = n < N;                   // (lanes past the end count for variate N - 1 and are not written)
  if (tid < 3 * T + 2) cnt[tid] = 0;
  uint32_t high = 0;
  for (int i = tid; i < N; i += 4 * NT) {     // (four loads in flight)
    uint64_t h[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) h[u] = hash[min(i + u * NT, N - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * NT < N) {
        hs[i + u * NT] = h[u];
        ks[i + u * NT] = (uint32_t)h[u];
        flag[i + u * NT] = 0;
        high |= (uint32_t)(h[u] >> 32);
      }
  }
  const uint64_t kn = member_key(a, valid ? n : N - 1);
  __syncthreads();
  if (__any(high != 0)) {
    const int l = __any(high >> 24) ? 4 : (__any(high >> 16) ? 3 : (__any(high >> 8) ? 2 : 1));
    if (lane == 0) atomicMax(level, l);
  }
  __syncthreads();
  const int shift = 8 * *level;
  if (shift) {
    for (int i = tid; i < N; i += NT) ks[i] = (uint32_t)(hs[i] >> shift);
    __syncthreads();
  }
  const uint64_t hn = hs[valid ? n : N - 1];
  int lt = 0, eq = 0, rank = 0;
  {
    const uint32_t k32 = (uint32_t)(hn >> shift);
    const int full = N / (4 * STEP) * (4 * STEP);
    int m = wave * M + lane / T;
    for (; m < full; m += 4 * STEP) {         // (four reads in flight)
      uint32_t km[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) km[u] = ks[m + u * STEP];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        lt += km[u] < k32 ? 1 : 0;
        if (km[u] == k32) flag[m + u * STEP] = 1;
      }
    }
    for (; m < N; m += STEP) {
      const uint32_t km = ks[m];
      lt += km < k32 ? 1 : 0;
      if (km == k32) flag[m] = 1;
    }
  }
  __syncthreads();
  for (int i0 = tid - lane; i0 < N; i0 += NT) {          // the list: its order does not matter to a count
    const int m = i0 + lane;
    const bool in = m < N && flag[m];
    const unsigned long long b = __ballot(in);
    if (b) {
      int base = 0;
      if (lane == 0) base = atomicAdd(nlist, __popcll(b));
      base = __builtin_amdgcn_readfirstlane(base);
      if (in) list[base + __popcll(b & ((1ull << lane) - 1ull))] = (uint16_t)m;
    }
  }
  __syncthreads();
  const int L = *nlist;
  for (int i = tid; i < L; i += NT) us[i] = member_key(a, list[i]);
  __syncthreads();
  auto count = [&](int m, uint64_t h, uint64_t u) {
    const bool same = h == hn;
    lt += h < hn && (uint32_t)(h >> shift) == (uint32_t)(hn >> shift) ? 1 : 0;      // (not counted in the first pass)
    eq += same ? 1 : 0;
    rank += (same && (u < kn || (u == kn && m < n))) ? 1 : 0;
  };
  {
    const int full = L / (4 * STEP) * (4 * STEP);
    int i = wave * M + lane / T;
    for (; i < full; i += 4 * STEP) {
      int m[4];
      uint64_t u4[4], h4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        m[u] = list[i + u * STEP];
        u4[u] = us[i + u * STEP];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) h4[u] = hs[m[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u) count(m[u], h4[u], u4[u]);
    }
    for (; i < L; i += STEP) count(list[i], hs[list[i]], us[i]);
  }
#pragma unroll
  for (int off = T; off < 64; off <<= 1) {
    lt += __shfl_xor(lt, off, 64);
    eq += __shfl_xor(eq, off, 64);
    rank += __shfl_xor(rank, off, 64);
  }
  if (lane < T) {
    atomicAdd(&cnt[lane], lt);
    atomicAdd(&cnt[T + lane], eq);
    atomicAdd(&cnt[2 * T + lane], rank);
  }
  __syncthreads();
  if (tid < T && valid) a.group_id[n] = (int32_t)pack_rank(a, cnt[tid], cnt[T + tid], cnt[2 * T + tid]);
}
template <int E>
__global__ __launch_bounds__(1024) void select_kernel(SampleArgs a) {
  __shared__ SelectLds s;
  uint32_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = e * (int)blockDim.x + (int)threadIdx.x;
    v[e] = n < a.N ? (uint32_t)a.group_id[n] : 0u;
  }
  select_phase<E>(a, v, s, blockDim.x);
}
// Up to 192 variates: wavefront w counts for the variates of block w % nb of 64 over one of 16 / nb parts of them.
__global__ __launch_bounds__(1024) void sample_small_kernel(SampleArgs a) {
  __shared__ uint64_t hs[kSmallSample], us[kSmallSample];
  __shared__ int cnt[3][kSmallSample];
  __shared__ SelectLds s;
  const int N = a.N, tid = threadIdx.x, wave = tid >> 6, nb = (N + 63) >> 6;
  const int n = (wave % nb) * 64 + (tid & 63), part = wave / nb, parts = 16 / nb;
  read_step(a);
  if (tid < N) {
    hs[tid] = a.hash[tid];
    us[tid] = member_key(a, tid);
  }
  if (tid < 3 * kSmallSample) cnt[0][tid] = 0;
  __syncthreads();
  if (n < N && part < parts) {
    const uint64_t hn = hs[n], kn = us[n];
    int lt = 0, eq = 0, rank = 0;
    const int per = (N + parts - 1) / parts;
#pragma unroll 4
    for (int m = part * per; m < min(N, (part + 1) * per); ++m) {
      const uint64_t h = hs[m], u = us[m];
      lt += h < hn ? 1 : 0;
      eq += h == hn ? 1 : 0;
      rank += (h == hn && (u < kn || (u == kn && m < n))) ? 1 : 0;
    }
    atomicAdd(&cnt[0][n], lt);
    atomicAdd(&cnt[1][n], eq);
    atomicAdd(&cnt[2][n], rank);
  }
  __syncthreads();
  uint32_t v[1] = {tid < N ? pack_rank(a, cnt[0][tid], cnt[1][tid], cnt[2][tid]) : 0u};
  select_phase<1>(a, v, s, blockDim.x);
}

size_t rank_lds(int N, int T) { return (((size_t)N * 18 + 15) & ~(size_t)15) + (size_t)(3 * T + 2) * sizeof(int); }

int run_sample(vardrop_ctx* ctx, const uint64_t* hash, int N,
               uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
               uint64_t seed, uint64_t step, const uint64_t* ext_keys,
               int32_t* group_id, int32_t* sel, int32_t* counts, int32_t* counts_host, void* stream,
               uint64_t* step_dev = nullptr, int advance = 0) {
  if (!ctx || !hash || !group_id || !sel || !counts) return VARDROP_EINVAL;
  if (N < 1) return VARDROP_EINVAL;
  if (ratio_den == 0 || ratio_num > ratio_den) return VARDROP_EINVAL;
  if (N > kMaxN) return VARDROP_EUNSUPPORTED;
  SampleArgs a;
  a.hash = hash;
  a.group_id = group_id;
  a.sel = sel;
  a.counts = counts;
  a.N = N;
  a.gs = gs;
  a.num = ratio_num;
  a.den = ratio_den;
  a.seed_lo = (uint32_t)seed;
  a.seed_hi = (uint32_t)(seed >> 32);
  a.step_lo = (uint32_t)step;
  a.step_hi = (uint32_t)(step >> 32);
  a.ext_keys = ext_keys;
  a.step_dev = step_dev;
  a.advance = advance;
  hipStream_t s = (hipStream_t)stream;
  VdTimer timer(ctx, VARDROP_K_SAMPLE, s);
  if (N <= kSmallSample) {
    VD_KERNEL(ctx, sample_small_kernel, dim3(1), dim3(1024), 0, s, a);
    VD_LAUNCH_CHECK(ctx);
  } else {
    // A workgroup owns 16 variates, and 32 above 4096: at most one workgroup per compute unit.
    // (timed as one: the first launch carries the start event, the second the completion)
#define VD_RANK(T)                                                                                                 \
  {                                                                                                                \
    const size_t lds = rank_lds(N, T);                                                                             \
    if (lds > 65536) VD_HIP(ctx, hipFuncSetAttribute((const void*)rank_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
    if (ctx->prof_e0) hipExtLaunchKernelGGL(rank_kernel<T>, dim3(vd_ceil_div(N, T)), dim3(kRankThreads), lds, s, ctx->prof_e0, nullptr, 0, a); \
    else hipLaunchKernelGGL(rank_kernel<T>, dim3(vd_ceil_div(N, T)), dim3(kRankThreads), lds, s, a);               \
  }
    if (N <= 4096) VD_RANK(16)
    else VD_RANK(32)
#undef VD_RANK
    VD_LAUNCH_CHECK(ctx);
#define VD_SELECT(E, NT)                                                                                           \
  {                                                                                                                \
    if (ctx->prof_e1) hipExtLaunchKernelGGL(select_kernel<E>, dim3(1), dim3(NT), 0, s, nullptr, ctx->prof_e1, 0, a); \
    else hipLaunchKernelGGL(select_kernel<E>, dim3(1), dim3(NT), 0, s, a);                                         \
  }
    if (N <= 1024) VD_SELECT(1, vd_ceil_div(N, 64) * 64)
    else if (N <= 2048) VD_SELECT(2, 1024)
    else if (N <= 4096) VD_SELECT(4, 1024)
    else VD_SELECT(8, 1024)
#undef VD_SELECT
    VD_LAUNCH_CHECK(ctx);
  }
  if (counts_host)
    VD_HIP(ctx, hipMemcpyAsync(counts_host, counts, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  return VARDROP_OK;
}

// ---- deterministic representatives: keys from the distance to the group's mean spectrum, by one workgroup per group
// (that of its first member, the lowest variate index; the others return).  The members are listed in ascending
// order, one thread per candidate bin adds their values in that order and divides by the group size, then one thread
// per member adds up its squared distances in ascending bins.
// Single-precision IEEE operations without fused multiply-add throughout: these values decide which
// members are kept, and the test oracle evaluates them in the same arithmetic and order.
// Bound by its serial chains: loads of 32 members (or bins) are in flight while the sums go on in order, of four blocks of hashes
// while the group is listed.  With the distances of N = 2048, F = 85, 120 groups the whole call takes 16.7 us (17.9 with eight loads and one
// block), of one group of 2048 84 (103), of 8192 341 (415).  A piece of the rows at a time through LDS instead: 180 and 711 us.
// key[n] = bits of sum_f (abar[n][f] - mean[f])^2 in the upper half: non-negative floats order like their bit patterns
__global__ __launch_bounds__(256) void group_distance_kernel(const uint64_t* __restrict__ hash, const float* __restrict__ abar,
                                                            float* __restrict__ mean, uint64_t* __restrict__ keys, int N, int F) {
  __shared__ uint16_t list[kMaxN];
  __shared__ int wcnt[16];
  const int n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t h = hash[n];
  int earlier = 0;
  {                                                      // (four loads in flight; past n: n - 1 again)
    int m0 = 0;
    for (; m0 + 256 < n; m0 += 4 * 256) {
      uint64_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = hash[min(m0 + u * 256 + tid, n - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) earlier |= v[u] == h ? 1 : 0;
    }
    if (m0 + tid < n) earlier |= hash[m0 + tid] == h ? 1 : 0;
  }
  if (__syncthreads_or(earlier)) return;
  int size = 0;
  // the list: four blocks of 256 at a time, the last one alone
  const auto collect = [&](int m0, auto blocks) {
    constexpr int U = decltype(blocks)::value;
    uint64_t v[U];
    unsigned long long b[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = hash[min(m0 + u * 256 + tid, N - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      in[u] = m0 + u * 256 + tid < N && v[u] == h;
      b[u] = __ballot(in[u]);
      if (lane == 0) wcnt[u * 4 + wave] = __popcll(b[u]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int at = size;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w < wave) at += wcnt[u * 4 + w];
        size += wcnt[u * 4 + w];
      }
      if (in[u]) list[at + __popcll(b[u] & ((1ull << lane) - 1ull))] = (uint16_t)(m0 + u * 256 + tid);
    }
    __syncthreads();
  };
  {
    int m0 = n;
    for (; m0 + 256 < N; m0 += 4 * 256) collect(m0, std::integral_constant<int, 4>());
    if (m0 < N) collect(m0, std::integral_constant<int, 1>());
  }
  float* mu = mean + (long long)n * F;                   // (a group's mean lies at its first member's place)
  for (int f = tid; f < F; f += 256) {
    float acc = 0.f;
    int i = 0;
    for (; i + 32 <= size; i += 32) {
      float x[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) x[u] = abar[(long long)list[i + u] * F + f];
#pragma unroll
      for (int u = 0; u < 32; ++u) acc = acc + x[u];
    }
    for (; i + 8 <= size; i += 8) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = abar[(long long)list[i + u] * F + f];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = acc + x[u];
    }
    for (; i < size; ++i) acc = acc + abar[(long long)list[i] * F + f];
    mu[f] = acc / (float)size;                           // (correctly rounded: the compiler's default for fp32 division)
  }
  __threadfence_block();
  __syncthreads();
  for (int i = tid; i < size; i += 256) {
    const float* row = abar + (long long)list[i] * F;
    float d = 0.f;
    {
#pragma clang fp contract(off)                  // product and sum are rounded separately (no fused multiply-add)
      int f = 0;
      for (; f + 32 <= F; f += 32) {
        float x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) x[u] = row[f + u] - mu[f + u];
#pragma unroll
        for (int u = 0; u < 32; ++u) {
          const float sq = x[u] * x[u];
          d = d + sq;
        }
      }
      for (; f + 8 <= F; f += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = row[f + u] - mu[f + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float sq = x[u] * x[u];
          d = d + sq;
        }
      }
      for (; f < F; ++f) {
        const float t = row[f] - mu[f];
        const float sq = t * t;
        d = d + sq;
      }
    }
    keys[list[i]] = (uint64_t)__float_as_uint(d) << 32;
  }
}

}  // namespace

extern "C" size_t vardrop_sample_workspace_bytes(int) { return 0; }

extern "C" int vardrop_sample(vardrop_ctx* ctx, const uint64_t* hash, int N,
                              uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
                              uint64_t seed, uint64_t step,
                              int32_t* group_id, int32_t* sel, int32_t* counts, int32_t* counts_host,
                              void* ws, size_t ws_bytes, void* stream) {
  (void)ws;
  (void)ws_bytes;
  return run_sample(ctx, hash, N, gs, ratio_num, ratio_den, seed, step, nullptr, group_id, sel, counts, counts_host, stream);
}

extern "C" int vardrop_sample_dev(vardrop_ctx* ctx, const uint64_t* hash, int N,
                                  uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
                                  uint64_t seed, uint64_t* step_dev, int advance,
                                  int32_t* group_id, int32_t* sel, int32_t* counts,
                                  void* ws, size_t ws_bytes, void* stream) {
  (void)ws;
  (void)ws_bytes;
  if (!step_dev || !vd_aligned(step_dev, 8)) return VARDROP_EINVAL;
  return run_sample(ctx, hash, N, gs, ratio_num, ratio_den, seed, 0, nullptr, group_id, sel, counts, nullptr, stream,
                    step_dev, advance);
}

namespace {
int run_sample_nearest(vardrop_ctx* ctx, const uint64_t* hash, const float* abar, int N, int F,
                       uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
                       int32_t* group_id, int32_t* sel, int32_t* counts, int32_t* counts_host,
                       float* mean, uint64_t* keys, void* stream) {
  // (run_sample's argument checks come first: nothing is launched for arguments it refuses)
  if (!hash || !group_id || !sel || !counts || N < 1 || ratio_den == 0 || ratio_num > ratio_den) return VARDROP_EINVAL;
  if (N > kMaxN) return VARDROP_EUNSUPPORTED;
  hipLaunchKernelGGL(group_distance_kernel, dim3(N), dim3(256), 0, (hipStream_t)stream, hash, abar, mean, keys, N, F);
  VD_LAUNCH_CHECK(ctx);
  return run_sample(ctx, hash, N, gs, ratio_num, ratio_den, 0, 0, keys, group_id, sel, counts, counts_host, stream);
}

// Scratch of the entry point that allocates nothing: [N][F] floats, a group's mean in the row of its first member
// (N F <= kStaticMeanFloats), followed by the distance keys ([N] uint64, N <= kMaxN).  Part of the code object, one copy per device, held until
// the process ends; every call on a device uses it, so calls that overlap on one device race.
constexpr size_t kStaticMeanFloats = (size_t)1 << 20;
constexpr size_t kStaticScratchBytes = kStaticMeanFloats * sizeof(float) + (size_t)kMaxN * sizeof(uint64_t);
}  // namespace
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of the scratch array on the current device (the array's name is only a host-side stand-in for it).
int vd_static_scratch_address(void** out) {
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) return (int)(e != hipSuccess ? e : hipErrorInvalidSymbol);
  *out = p;
  return 0;
}

extern "C" int vardrop_sample_nearest_noalloc(vardrop_ctx* ctx, const uint64_t* hash, const float* abar, int N, int F,
                                              uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
                                              int32_t* group_id, int32_t* sel, int32_t* counts, void* stream) {
  if (!ctx || !abar || F < 1) return VARDROP_EINVAL;
  if (N > kMaxN || (N >= 1 && (size_t)N * (size_t)F > kStaticMeanFloats)) return VARDROP_EUNSUPPORTED;   // beyond the static scratch
  if (!ctx->static_scratch) return VARDROP_EHIP;             // its address could not be taken when the context was made
  float* mean = (float*)ctx->static_scratch;
  uint64_t* keys = (uint64_t*)((char*)ctx->static_scratch + kStaticMeanFloats * sizeof(float));
  return run_sample_nearest(ctx, hash, abar, N, F, gs, ratio_num, ratio_den, group_id, sel, counts, nullptr, mean, keys, stream);
}

extern "C" size_t vardrop_sample_nearest_workspace_bytes(int N, int F) {
  if (N < 1 || F < 1) return 0;
  return vd_align_up((size_t)N * F * sizeof(float), 256) + vd_align_up((size_t)N * sizeof(uint64_t), 256);
}

extern "C" int vardrop_sample_nearest(vardrop_ctx* ctx, const uint64_t* hash, const float* abar, int N, int F,
                                      uint32_t gs, uint32_t ratio_num, uint32_t ratio_den,
                                      int32_t* group_id, int32_t* sel, int32_t* counts, int32_t* counts_host,
                                      void* ws, size_t ws_bytes, void* stream) {
  if (!ctx || !abar || F < 1) return VARDROP_EINVAL;
  if (N >= 1 && (!ws || !vd_aligned(ws, 256) || ws_bytes < vardrop_sample_nearest_workspace_bytes(N, F))) return VARDROP_EWORKSPACE;
  float* mean = (float*)ws;
  uint64_t* keys = (uint64_t*)((char*)ws + vd_align_up((size_t)N * F * sizeof(float), 256));
  return run_sample_nearest(ctx, hash, abar, N, F, gs, ratio_num, ratio_den, group_id, sel, counts, counts_host, mean, keys, stream);
}
