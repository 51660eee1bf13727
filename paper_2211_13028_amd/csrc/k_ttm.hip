// Mode-k tensor-times-matrix on the (A, K, B) view of a C-order tensor:
//   Y[a, i, b] = sum_k M[i, k] X[a, k, b]
// (Sec. 2.1: the mode-k unfolding of X x_k M is M times the unfolding of X).
// No unfolding is materialised: for each a, X[a] is a row-major K x B matrix,
// so the contraction is a strided-batched GEMM whose HBM reads are whole rows.
//
//  * ttm_generic: VALU kernel for every dtype and shape (one output column per
//    thread, m split into register tiles, M chunks broadcast from LDS).
//  * ttm_split_f32: matrix-core kernel for binary32 X (B >= 64, m <= 64): three
//    bfloat16 terms a value, X streamed once, M split and staged in LDS.
//  * ttm_mfma_f32, ttm_mfma_f32_grouped: binary32 products, M read from L2, for a short K or few rows
//    of M on the 16-byte grid, and for the small contractions of one launch.
//  * ttm_mfma_bf16: bfloat16 X (B >= 64, m <= 64), M staged in LDS, operands re-packed in registers so
//    that each lane holds 8 consecutive k of one column; ttm_mfma_bf16_direct: the same with
//    M read from the caches, for small tensors on the 16-byte grid.
//  * ttm_mfma_last: the last mode (B == 1), X in rows of K contiguous values.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace rt {

namespace {

// ------------------------------------------------------------------ generic VALU
constexpr int kGenThreads = 256;
constexpr int kGenKC = 64;

// acc[ii] += sum over k in [kb, ke) of M(i0 + ii, k) X[a, k, b] for this thread's column
// (xp = &X[a, 0, b]).  A chunk of M is staged in LDS; its global loads are all issued
// into registers before the first LDS store, and X is read kXB rows at a time, so the
// loads of a chunk are in flight together instead of one latency each.
constexpr int kXB = 8;
static_assert(kGenKC % kXB == 0, "X blocks must tile the M chunk");
template <typename TX, typename TC, int MT>
__device__ __forceinline__ void generic_accumulate(const TX* __restrict__ xp, int64_t B, const TC* __restrict__ M,
                                                   int64_t m, int64_t K, int64_t i0, int64_t kb, int64_t ke,
                                                   bool mtrans, bool active, TC (&sM)[MT][kGenKC], TC (&acc)[MT]) {
  constexpr int kPer = MT * kGenKC / kWave;  // M elements per thread at the smallest block (one wave)
  const int nth = static_cast<int>(blockDim.x);
  for (int64_t k0 = kb; k0 < ke; k0 += kGenKC) {
    // binary32, four rows of M: the sums of 64 k are added up (one chain over a long K rounds more).
    // Not with more rows, which hold the registers of waves in flight (a 256^3 projection step, whose
    // expansions have K = 24 and m = 256: 586 us with such sums, 531 without).
    constexpr bool kSums = std::is_same<TC, float>::value && MT == 4;
    TC part[MT];
#pragma unroll
    for (int ii = 0; ii < MT; ++ii) part[ii] = kSums ? TC(0) : acc[ii];
    TC mv[kPer];
#pragma unroll
    for (int rep = 0; rep < kPer; ++rep) {
      const int t = static_cast<int>(threadIdx.x) + rep * nth;
      const int ii = t / kGenKC, kk = t % kGenKC;
      mv[rep] = (t < MT * kGenKC && i0 + ii < m && k0 + kk < ke)
                    ? (mtrans ? M[(k0 + kk) * m + i0 + ii] : M[(i0 + ii) * K + k0 + kk])
                    : TC(0);
    }
    __syncthreads();
#pragma unroll
    for (int rep = 0; rep < kPer; ++rep) {
      const int t = static_cast<int>(threadIdx.x) + rep * nth;
      if (t < MT * kGenKC) sM[t / kGenKC][t % kGenKC] = mv[rep];
    }
    __syncthreads();
    if (active) {
      const int kend = static_cast<int>((ke - k0) < kGenKC ? (ke - k0) : kGenKC);
      for (int kk0 = 0; kk0 < kend; kk0 += kXB) {
        TC xv[kXB];
#pragma unroll
        for (int u = 0; u < kXB; ++u)
          xv[u] = (kk0 + u < kend) ? static_cast<TC>(Load<TX>::get(xp, (k0 + kk0 + u) * B)) : TC(0);
#pragma unroll
        for (int u = 0; u < kXB; ++u)
#pragma unroll
          for (int ii = 0; ii < MT; ++ii) part[ii] = fma(sM[ii][kk0 + u], xv[u], part[ii]);
      }
    }
#pragma unroll
    for (int ii = 0; ii < MT; ++ii) acc[ii] = kSums ? acc[ii] + part[ii] : part[ii];
  }
}

// one block: columns bx blockDim.x .., rows MT by .., part bz of K
template <typename TX, typename TC, int MT>
__device__ __forceinline__ void generic_block(const TX* __restrict__ X, int64_t A, int64_t K, int64_t B,
                                              const TC* __restrict__ M, int64_t m, int64_t kper, bool mtrans,
                                              TC* __restrict__ Y, int64_t bx, int64_t by, int64_t bz,
                                              TC (&sM)[MT][kGenKC]) {
  const int64_t col = bx * blockDim.x + threadIdx.x;
  const int64_t i0 = by * MT;
  const int64_t kb = bz * kper;
  const int64_t ke = (kb + kper < K) ? kb + kper : K;
  const bool active = col < A * B;
  const int64_t a = active ? col / B : 0;
  const int64_t b = active ? col - a * B : 0;
  TC acc[MT];
#pragma unroll
  for (int ii = 0; ii < MT; ++ii) acc[ii] = TC(0);
  generic_accumulate<TX, TC, MT>(X + a * K * B + b, B, M, m, K, i0, kb, ke, mtrans, active, sM, acc);
  if (active) {
    TC* y = Y + bz * A * m * B;
#pragma unroll
    for (int ii = 0; ii < MT; ++ii)
      if (i0 + ii < m) y[a * m * B + (i0 + ii) * B + b] = acc[ii];
  }
}

template <typename TX, typename TC, int MT>
__global__ __launch_bounds__(kGenThreads) void ttm_generic_kernel(const TX* __restrict__ X, int64_t A, int64_t K,
                                                                  int64_t B, const TC* __restrict__ M, int64_t m,
                                                                  int64_t kper, bool mtrans, TC* __restrict__ Y) {
  __shared__ TC sM[MT][kGenKC];
  generic_block<TX, TC, MT>(X, A, K, B, M, m, kper, mtrans, Y, blockIdx.x, blockIdx.y, blockIdx.z, sM);
}

// Several such contractions with few output columns (one wave a block, four rows of M) in one
// launch: the blocks of job q start at blk0.  They are bound by their latency, so one after the
// other they take a launch's time each (the second level of a 701 x 523 x 389 binary32
// sketch, with its sums: 46 us in six launches, 28 in three).
constexpr int kGenGroupRows = 4;
struct GenJob {
  const void* X;
  const void* M;
  void* out;
  int64_t A, K, B, m, kper, blk0, gx, gy;
};
struct GenJobTable {
  GenJob j[kMaxF32Group];
  int count;
};
template <typename T>
__global__ __launch_bounds__(kWave) void ttm_generic_group_kernel(GenJobTable tab) {
  __shared__ T sM[kGenGroupRows][kGenKC];
  int q = 0;
  for (int t = 1; t < tab.count; ++t)
    if (static_cast<int64_t>(blockIdx.x) >= tab.j[t].blk0) q = t;
  const GenJob& J = tab.j[q];
  const int64_t local = blockIdx.x - J.blk0;
  const int64_t bx = local % J.gx, rest = local / J.gx;
  generic_block<T, T, kGenGroupRows>(static_cast<const T*>(J.X), J.A, J.K, J.B, static_cast<const T*>(J.M), J.m, J.kper,
                                     false, static_cast<T*>(J.out), bx, rest % J.gy, rest / J.gy, sM);
}

// Split sums of several jobs in one launch: job q covers the flat indices [off_q, off_q + n_q).
template <typename T>
struct SumJob {
  const T* first;
  const T* rest;
  T* Y;
  int64_t n, off;
  int ksplit;
};
template <typename T>
struct SumJobTable {
  SumJob<T> j[kMaxF32Group];
  int count;
};
template <typename T>
__global__ __launch_bounds__(256) void sum_splits_grouped_kernel(SumJobTable<T> tab, int64_t total) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; g < total; g += stride) {
    int q = 0;
    for (int t = 1; t < tab.count; ++t)
      if (g >= tab.j[t].off) q = t;
    const SumJob<T>& J = tab.j[q];
    const int64_t i = g - J.off;
    T acc = J.first[i];
    for (int k = 1; k < J.ksplit; ++k) acc += J.rest[(k - 1) * J.n + i];
    J.Y[i] = acc;
  }
}
template <typename T>
hipError_t split_sums(const std::vector<SplitSum>& sums, hipStream_t st) {
  for (size_t i0 = 0; i0 < sums.size(); i0 += kMaxF32Group) {
    SumJobTable<T> tab{};
    int64_t total = 0;
    for (size_t i = i0; i < sums.size() && tab.count < kMaxF32Group; ++i) {
      tab.j[tab.count++] = SumJob<T>{static_cast<const T*>(sums[i].first), static_cast<const T*>(sums[i].rest),
                                     static_cast<T*>(sums[i].Y), sums[i].n, total, sums[i].ksplit};
      total += sums[i].n;
    }
    const unsigned g = static_cast<unsigned>(ceil_div(total, 256) > 8192 ? 8192 : ceil_div(total, 256));
    sum_splits_grouped_kernel<T><<<g, 256, 0, st>>>(tab, total);
  }
  return hipGetLastError();
}

template <typename TC>
__global__ __launch_bounds__(256) void generic_sum_kernel(const TC* __restrict__ part, int ksplit, int64_t n,
                                                          TC* __restrict__ Y) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride) {
    TC s = part[i];
    for (int k = 1; k < ksplit; ++k) s += part[k * n + i];
    Y[i] = s;
  }
}

// split K over grid.z when there are too few output columns to fill the chip
int generic_ksplit(int64_t A, int64_t K, int64_t B) {
  const int64_t cols = A * B;
  int ks = 1;
  while (cols * ks < 131072 && K / (2 * ks) >= 64 && ks < 64) ks *= 2;
  return ks;
}

// few output columns: one-wave blocks, so that more CUs share the work
int generic_threads(int64_t A, int64_t B) { return A * B < 32768 ? kWave : kGenThreads; }

template <typename TX, typename TC>
hipError_t generic_dispatch(const TX* X, int64_t A, int64_t K, int64_t B, const TC* M, int64_t m, TC* Y, TC* ws,
                            hipStream_t st, bool mtrans) {
  const int64_t cols = A * B;
  const int threads = generic_threads(A, B);
  const unsigned gx = static_cast<unsigned>(ceil_div(cols, threads));
  const int ks = generic_ksplit(A, K, B);
  const int64_t kper = ceil_div(K, ks);
  TC* out = (ks > 1) ? ws : Y;
  if (m <= 4 || threads == kWave) {
    // (few output columns: 4-row tiles, so that more waves share the rows of m)
    const unsigned gy = static_cast<unsigned>(ceil_div(m, 4));
    ttm_generic_kernel<TX, TC, 4><<<dim3(gx, gy, ks), threads, 0, st>>>(X, A, K, B, M, m, kper, mtrans, out);
  } else if (m <= 8) {
    const unsigned gy = static_cast<unsigned>(ceil_div(m, 8));
    ttm_generic_kernel<TX, TC, 8><<<dim3(gx, gy, ks), threads, 0, st>>>(X, A, K, B, M, m, kper, mtrans, out);
  } else {
    const unsigned gy = static_cast<unsigned>(ceil_div(m, 16));
    ttm_generic_kernel<TX, TC, 16><<<dim3(gx, gy, ks), threads, 0, st>>>(X, A, K, B, M, m, kper, mtrans, out);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || ks == 1) return e;
  const int64_t n = A * m * B;
  const unsigned g2 = static_cast<unsigned>(ceil_div(n, 256) > 4096 ? 4096 : ceil_div(n, 256));
  generic_sum_kernel<TC><<<g2, 256, 0, st>>>(out, ks, n, Y);
  return hipGetLastError();
}

template <typename T>
hipError_t generic_group(const GenericContraction* c, int count, std::vector<SplitSum>& sums, hipStream_t st) {
  GenJobTable tab{};
  int64_t blocks = 0;
  for (int i = 0; i < count; ++i) {
    const int ks = generic_ksplit(c[i].A, c[i].K, c[i].B);
    GenJob& J = tab.j[tab.count++];
    J.X = c[i].X;
    J.M = c[i].M;
    J.out = ks > 1 ? c[i].ws : c[i].Y;
    J.A = c[i].A; J.K = c[i].K; J.B = c[i].B; J.m = c[i].m;
    J.kper = ceil_div(J.K, ks);
    J.blk0 = blocks;
    J.gx = ceil_div(J.A * J.B, kWave);
    J.gy = ceil_div(J.m, kGenGroupRows);
    blocks += J.gx * J.gy * ks;
    const int64_t n = J.A * J.m * J.B;
    if (ks > 1) sums.push_back(SplitSum{c[i].ws, static_cast<const T*>(c[i].ws) + n, c[i].Y, n, ks});
  }
  ttm_generic_group_kernel<T><<<static_cast<unsigned>(blocks), kWave, 0, st>>>(tab);
  return hipGetLastError();
}

// grouped form: job found by binary search over blk0; one wave per workgroup

template <typename TX, typename TC, int MT>
__global__ __launch_bounds__(kWave) void ttm_grouped_kernel(const GTtmJob* __restrict__ jobs,
                                                             const int32_t* __restrict__ blkjob) {
  __shared__ TC sM[MT][kGenKC];
  const int64_t blk = blockIdx.x;
  const GTtmJob J = jobs[blkjob[blk]];
  const int64_t local = blk - J.blk0;
  const int64_t cb = local / J.mtiles, mtile = local - cb * J.mtiles;
  const int64_t A = J.A, K = J.K, B = J.B, m = J.m;
  const TX* X = static_cast<const TX*>(J.X);
  const TC* M = static_cast<const TC*>(J.M);
  const int64_t col = cb * kWave + threadIdx.x;
  const int64_t i0 = mtile * MT;
  const bool active = col < A * B;
  const int64_t a = active ? col / B : 0;
  const int64_t b = active ? col - a * B : 0;
  TC acc[MT];
#pragma unroll
  for (int ii = 0; ii < MT; ++ii) acc[ii] = TC(0);
  // compact loops (few registers, several waves per SIMD for the many small jobs of a batch)
  const TX* xp = X + a * K * B + b;
  for (int64_t k0 = 0; k0 < K; k0 += kGenKC) {
    __syncthreads();
    for (int t = threadIdx.x; t < MT * kGenKC; t += kWave) {
      const int ii = t / kGenKC, kk = t % kGenKC;
      sM[ii][kk] = (i0 + ii < m && k0 + kk < K) ? (J.mtrans ? M[(k0 + kk) * m + i0 + ii] : M[(i0 + ii) * K + k0 + kk])
                                                : TC(0);
    }
    __syncthreads();
    if (active) {
      const int kend = static_cast<int>((K - k0) < kGenKC ? (K - k0) : kGenKC);
      for (int kk = 0; kk < kend; ++kk) {
        const TC x = static_cast<TC>(Load<TX>::get(xp, (k0 + kk) * B));
#pragma unroll
        for (int ii = 0; ii < MT; ++ii) acc[ii] = fma(sM[ii][kk], x, acc[ii]);
      }
    }
  }
  if (active) {
    TC* y = static_cast<TC*>(J.Y);
#pragma unroll
    for (int ii = 0; ii < MT; ++ii)
      if (i0 + ii < m) y[a * m * B + (i0 + ii) * B + b] = acc[ii];
  }
}

// ------------------------------------------------------------------ MFMA
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));  // at any bfloat16 boundary

constexpr int kMfmaThreads = 256;  // 4 waves, one 128-column unit each
constexpr int kUnitCols = 128;

// Where part ks of a contraction of n results goes: the first one into the result itself, the others
// behind one another (so a contraction in two parts needs the space of one).
__device__ __forceinline__ float* part_of(float* Y, float* rest, int64_t ks, int64_t n) {
  return ks == 0 ? Y : rest + (ks - 1) * n;
}

// Work unit = (a, 128-column chunk, k-split part).  Y (or a split-K partial) is
// written for rows i < m only.
// One work unit (a wave) of the binary32 contraction; unit < A * chunks * ksplit.
// (binary32 products: the small grouped contractions of the sketch's dimension tree, and short K or
// few rows of M)
template <int MT, bool VM, int DEPTH, bool SUMS>
__device__ __forceinline__ void ttm_f32_unit(const float* __restrict__ X, int64_t A, int64_t K, int64_t B,
                                             const float* __restrict__ Mop, int64_t m, int64_t chunks, int ksplit,
                                             int64_t kper, float* __restrict__ Y, float* __restrict__ rest, int64_t unit) {
  const int lane = threadIdx.x % kWave;
  const int ks = static_cast<int>(unit % ksplit);
  const int64_t ac = unit / ksplit;
  const int64_t a = ac / chunks;
  const int64_t b0 = (ac - a * chunks) * kUnitCols;
  const int j = lane % 16, q = lane / 16;
  const int64_t kbeg = ks * kper;
  const int64_t kend = (kbeg + kper < K) ? kbeg + kper : K;

  f32x4 acc[MT][2][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[mt][g][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  const float* xa = X + a * K * B;
  const bool colok0 = (b0 + 4 * j) < B;
  const bool colok1 = (b0 + 64 + 4 * j) < B;
  // The wave takes k in blocks of 16.  Product s of a block sums over the four k that
  // lane groups q = 0..3 hold, k = k0 + 4 q + s, so a lane's share of the M tile for the
  // whole block is four consecutive k: one 16-byte load per tile when K % 4 == 0 (VM).
  // The lane loads the X rows k0 + 4 q + s (s = 0..3), columns b0 + 4 j .. and
  // b0 + 64 + 4 j ...  Loads carry no conditions: a row past kend reads row kend - 1 and
  // is zeroed before use, and a lane past B reads column b0 (its products land only in
  // output columns that are not stored).
  const int64_t c0off = colok0 ? b0 + 4 * j : b0, c1off = colok1 ? b0 + 64 + 4 * j : b0;
  const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
  // DEPTH blocks in flight: set P holds the block DEPTH steps ahead of the one multiplied
  f32x4 n0[DEPTH][4], n1[DEPTH][4];
  float nw[DEPTH][MT][4];
  const auto load_block = [&](int64_t k0, auto Pc) {
    constexpr int P = decltype(Pc)::value;
    const int64_t kl = k0 + 4 * q;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t kc = (kl + s < kend) ? kl + s : kend - 1;
      n0[P][s] = *reinterpret_cast<const f32x4*>(xa + kc * B + c0off);
      n1[P][s] = *reinterpret_cast<const f32x4*>(xa + kc * B + c1off);
    }
    if constexpr (VM) {
      // kl is a multiple of 4, so kl < kend <= K gives kl <= K - 4; a block past K reads
      // the last four k of the row instead (zeroed before use)
      const int64_t km = (kl <= K - 4) ? kl : K - 4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(Mop + (mt * 16 + j) * K + km);
#pragma unroll
        for (int s = 0; s < 4; ++s) nw[P][mt][s] = v[s];
      }
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int s = 0; s < 4; ++s) nw[P][mt][s] = Mop[(mt * 16 + j) * K + ((kl + s < kend) ? kl + s : kend - 1)];
    }
  };
  const auto block = [&](int64_t k0, auto Pc) {
    constexpr int P = decltype(Pc)::value;
    f32x4 y0[4], y1[4];
    float w[4][MT];
    const int64_t kl = k0 + 4 * q;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool kin = kl + s < kend;
      y0[s] = kin ? n0[P][s] : zero4;
      y1[s] = kin ? n1[P][s] : zero4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) w[s][mt] = kin ? nw[P][mt][s] : 0.f;
    }
    // the block DEPTH steps ahead goes out before this block's products (the scheduler may
    // move neither the operand take-over below it nor it into the products)
    __builtin_amdgcn_sched_barrier(0);
    load_block(k0 + 16 * DEPTH, Pc);  // past kend: rows kend - 1 again, never used
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SUMS) {
      // sums of eight k each, added on the vector ALU: one chain over a long K rounds more (K = 80, normal
      // data: 1.6e-7 of the result's norm, 7.5e-8 in these sums)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f32x4 part[2][4];
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t)
              part[s % 2][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][mt], (g == 0 ? y0 : y1)[s][t],
                                                                    s < 2 ? zero4 : part[s % 2][t], 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            acc[mt][g][t] += part[0][t] + part[1][t];
            // formed here: moved past the loop's branches, it would keep the parts in registers
            asm volatile("" : "+v"(acc[mt][g][t]));
          }
        }
      return;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          acc[mt][0][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][mt], y0[s][t], acc[mt][0][t], 0, 0, 0);
          acc[mt][1][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][mt], y1[s][t], acc[mt][1][t], 0, 0, 0);
        }
      }
    }
  };
  constexpr auto sets = std::make_integer_sequence<int, DEPTH>{};
  if (kbeg < kend) for_each_index([&](auto Pc) { load_block(kbeg + 16 * decltype(Pc)::value, Pc); }, sets);
  for (int64_t k0 = kbeg; k0 < kend; k0 += 16 * DEPTH)
    for_each_index(
        [&](auto Pc) {
          const int64_t kb = k0 + 16 * decltype(Pc)::value;
          if (kb < kend) block(kb, Pc);
        },
        sets);
  float* ya = part_of(Y, rest, ks, A * m * B) + a * m * B;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t i = mt * 16 + 4 * q + v;
      if (i >= m) continue;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int64_t c = b0 + 64 * g + 4 * j;
        if (c < B) {
          f32x4 o = f32x4{acc[mt][g][0][v], acc[mt][g][1][v], acc[mt][g][2][v], acc[mt][g][3][v]};
          *reinterpret_cast<f32x4u*>(ya + i * B + c) = o;
        }
      }
    }
  }
}

// ------------------------------------------------------------------ binary32 as three bfloat16 terms
// The binary32 contraction on the bfloat16 matrix cores, at binary32 accuracy.  Every value is
// the exact sum of three bfloat16 terms, x = h + m + l (each the rounding to nearest of what is
// left, 8 bits at a time: the splitting of Henry, Tang and Heinecke, ARITH 2019), and of the nine
// products of x and M the six of relative size 2^-16 or more are kept (hh, hm, mh, mm, hl, lh); the
// dropped ones are below 2^-24 of |x M|, half a unit in the last place of binary32, with random
// signs.  A 16x16x32 bfloat16 product takes a quarter of the time a k of 16x16x4 binary32 ones do, so
// six of them take 0.375 of it.
//
// Per block of 32 k the five small products are summed by themselves, smallest first, and that sum is
// added on the vector ALU: the matrix cores cut an addend to the accumulator off where the vector ALU
// rounds, and every product that they add to the whole sum costs it one more rounding.  Error of
// the result's norm against 64 bits, over that of binary32 products on the matrix cores: normal data
// 0.38 (K = 64), 0.45 (100), 0.59 (267), 0.58 (1024), 0.44 (4096); values exp(5 N), whose sums are mostly
// one product, 0.99 .. 1.13 (with all six products added to the accumulator 1.13 .. 1.6, and normal
// data 0.65 .. 0.85); a single product (K = 1) 1.02.  Cost: 460 -> 478 us for 1024 x 524288
// with m = 49, nothing measurable for three row tiles of M or fewer.
//
// A wave owns 64 columns of one slab (lane j: four consecutive columns, at any 4-byte
// boundary) and takes k in blocks of 32: lane group q loads the rows k0 + 8 q .. + 7, converts
// them pairwise (the packed pair is what the B operand holds: two k of one column), and has the
// next block in flight during the block's products.  The four waves of a workgroup share the k
// range; M is split while it is staged in LDS, 64 k at a time, double-buffered.
//
// Bound: HBM (1024 x 1024 x 512 with m = 49: 0.165 ms of matrix-core time at peak against 0.36 ms
// of reading at 6.3 TB/s); the binary32 products before were bound by the matrix cores.  One after
// the other, 1024 x 524288 with m = 49: 544 -> 478 us; 512 x 768 x 640 with m = 36 338 -> 213;
// 128^4 with m = 27 285 -> 255 (first mode), 273 -> 232 (second).
//
// X and M are scaled by 2^24 before they are split, so that all terms of the smallest subnormal are
// normal bfloat16 values, and the results are scaled back.  What that cannot hold (an infinity, which
// splits into NaN; values above 2^104, results above 2^80) gives a result that is not finite, and the
// wave then takes its columns once more, with binary32 products: one infinity in X of 1024 x
// 524288 costs 46 us, one in every 195 rows of every column 840.
constexpr float kSplitUp = 0x1p24f, kSplitDown = 0x1p-48f;
constexpr int kSplitCols = 64;
constexpr int kSplitWin = 64;                // k of M per staged window
constexpr int kSplitStride = kSplitWin + 8;  // bfloat16 per staged row: 16-byte groups, rows 36 banks apart
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// the three terms of two values, packed in pairs
__device__ __forceinline__ void split3(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  const auto round2 = [](float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  };
  const auto low = [](uint32_t v) { return __uint_as_float(v << 16); };
  const auto high = [](uint32_t v) { return __uint_as_float(v & 0xffff0000u); };
  h = round2(x0, x1);
  const float r0 = x0 - low(h), r1 = x1 - high(h);  // exact
  m = round2(r0, r1);
  l = round2(r0 - low(m), r1 - high(m));
}

template <int MT, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void ttm_split_f32_kernel(
    const float* __restrict__ X, int64_t A, int64_t K, int64_t B, const float* __restrict__ Mop, int64_t m,
    int64_t chunks, int64_t groups, int64_t kper, float* __restrict__ Y, float* __restrict__ rest) {
  __shared__ __align__(16) uint16_t sM[2][3][16 * MT * kSplitStride];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int j = lane % 16, q = lane / 16;
  int je = j, qe = q;
  const int64_t ks = blockIdx.x / groups;
  const int64_t unit_raw = (blockIdx.x - ks * groups) * (NT / kWave) + tid / kWave;
  const bool active = unit_raw < A * chunks;
  const int64_t unit = active ? unit_raw : 0;
  const int64_t a = unit / chunks;
  const int64_t col_raw = (unit - a * chunks) * kSplitCols + 4 * j;
  // A lane whose columns run past B takes the last four.  It stores only those from col_raw on:
  // the others are its neighbour's, in another wave where a chunk begins, and a wave that takes its
  // columns once more (see the end) rounds them differently.
  const int64_t col = col_raw + 4 <= B ? col_raw : B - 4;
  const int64_t kbeg = ks * kper;
  const int64_t kend = (kbeg + kper < K) ? kbeg + kper : K;
  const float* xa = X + a * K * B + col;

  f32x4 acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The lane's rows of a block, at xp (advanced by 32 rows a block: forming each row's address
  // from its number cost more issue slots than the conversion).  In the range's last block rows
  // past kend read row kend - 1 again; M is zero there.
  f32x4 rn[8];
  const float* xp = xa + (kbeg + 8 * q) * B;
  const auto load = [&](int64_t k0) {
    if (k0 + 32 <= kend) {
#pragma unroll
      for (int t = 0; t < 8; ++t) rn[t] = *reinterpret_cast<const f32x4u*>(xp + t * B);
    } else if (k0 < kend) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int64_t k = k0 + 8 * q + t;
        rn[t] = *reinterpret_cast<const f32x4u*>(xa + (k < kend ? k : kend - 1) * B);
      }
    }
    xp += 32 * B;
  };
  // staging: group g = NT i + tid of a window is row g / 16, k = kw + 4 (g % 16) ..
  constexpr int kGroups = 16 * MT * (kSplitWin / 4), kPer = (kGroups + NT - 1) / NT;
  f32x4 sv[kPer];
  const auto group_at = [&](int row, int64_t k) {  // zero past the range
    const float* src = Mop + static_cast<int64_t>(row) * K + k;
    f32x4 v;
    if (k + 4 <= kend) {
      v = *reinterpret_cast<const f32x4u*>(src);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = k + c < kend ? src[c] : 0.f;
    }
    return v;
  };
  const auto stage_load = [&](int64_t kw) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int g = i * NT + tid;
      if (g < kGroups) sv[i] = group_at(g / 16, kw + 4 * (g % 16));
    }
  };
  const auto stage_store = [&](int b) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int g = i * NT + tid;
      if (g >= kGroups) break;
      uint32_t t[3][2];
      split3(sv[i][0] * kSplitUp, sv[i][1] * kSplitUp, t[0][0], t[1][0], t[2][0]);
      split3(sv[i][2] * kSplitUp, sv[i][3] * kSplitUp, t[0][1], t[1][1], t[2][1]);
#pragma unroll
      for (int p = 0; p < 3; ++p)
        *reinterpret_cast<uint2*>(&sM[b][p][(g / 16) * kSplitStride + 4 * (g % 16)]) = make_uint2(t[p][0], t[p][1]);
    }
  };
  load(kbeg);
  stage_load(kbeg);
  stage_store(0);
  __syncthreads();
  int buf = 0, half = 0;
  for (int64_t k0 = kbeg; k0 < kend; k0 += 32) {
    // window: the blocks k0 - 32 half and the one after it
    const bool more = k0 + (kSplitWin - 32 * half) < kend;
    if (half == 0 && more) stage_load(k0 + kSplitWin);
    u32x4 xt[3][4];  // terms of the lane's four columns, 8 k each
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t h, md, l;
        split3(rn[2 * w][c] * kSplitUp, rn[2 * w + 1][c] * kSplitUp, h, md, l);
        xt[0][c][w] = h;
        xt[1][c][w] = md;
        xt[2][c][w] = l;
      }
    __builtin_amdgcn_sched_barrier(0);
    load(k0 + 32);
    __builtin_amdgcn_sched_barrier(0);
    // The columns in pairs: the small products of a pair, then the large ones of the next pair, then
    // the pair's addition, whose operands the matrix cores have finished by then; the terms of the
    // next row tile are read during the second pair's products.
    const uint16_t* mw = &sM[buf][0][j * kSplitStride + 32 * half + 8 * q];
    const auto read_m = [&](bf16x8 (&mv)[3], int mt) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
        mv[p] = *reinterpret_cast<const bf16x8*>(mw + (p * 16 * MT + 16 * mt) * kSplitStride);
    };
    const auto large = [&](int mt, int c0, bf16x8 mv) {
#pragma unroll
      for (int c = c0; c < c0 + 2; ++c)
        acc[mt][c] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(mv, __builtin_bit_cast(bf16x8, xt[0][c]), acc[mt][c], 0, 0, 0);
    };
    bf16x8 mv[3], nx[3];
    read_m(mv, 0);
    large(0, 0, mv[0]);
#pragma unroll
    for (int pair = 0; pair < 2 * MT; ++pair) {
      constexpr int kTm[5] = {2, 0, 1, 1, 0}, kTx[5] = {0, 2, 1, 0, 1};
      const int mt = pair / 2, c0 = 2 * (pair % 2);
      if (c0 == 2 && mt + 1 < MT) {
        read_m(nx, mt + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x4 low[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int e = 0; e < 5; ++e)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          low[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mv[kTm[e]], __builtin_bit_cast(bf16x8, xt[kTx[e]][c0 + c]),
                                                           low[c], 0, 0, 0);
      if (c0 == 0) {
        large(mt, 2, mv[0]);
      } else if (mt + 1 < MT) {
        large(mt + 1, 0, nx[0]);
#pragma unroll
        for (int p = 0; p < 3; ++p) mv[p] = nx[p];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[mt][c0 + c] += low[c];
    }
    // the sums are formed here: moved past the branches below, they would keep every `low` in registers
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(acc[mt][c]));
    half ^= 1;
    if (half == 0 || k0 + 32 >= kend) {
      if (more) stage_store(buf ^ 1);
      lds_barrier();  // the window is read by every wave and the next one staged; loads of X stay in flight
      buf ^= 1;
    }
  }
  if (!active) return;
  // (nothing of what follows is formed before the loop, whose registers it would take)
  asm volatile("" : "+v"(je), "+v"(qe));
  // results outside the range of the terms (see above): once more with binary32 products
  bool again = false;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        again = again || !isfinite(acc[mt][c][v]);
        acc[mt][c][v] *= kSplitDown;
      }
  }
  if (__any(again)) {
    // the rows of X as above, the next block in flight; product t of a block sums over the k of
    // the four lane groups, k0 + 8 q + t, so a lane's share of M is eight consecutive k
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    xp = xa + (kbeg + 8 * qe) * B;
    load(kbeg);
    for (int64_t k0 = kbeg; k0 < kend; k0 += 32) {
      const int64_t kl = k0 + 8 * qe;
      f32x4 x[8];
      f32x4 w[MT][2];
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = (kl + t < kend) ? rn[t] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int h = 0; h < 2; ++h) w[mt][h] = group_at(16 * mt + je, kl + 4 * h);
      __builtin_amdgcn_sched_barrier(0);
      load(k0 + 32);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[mt][t / 4][t % 4], x[t][c], acc[mt][c], 0, 0, 0);
    }
  }
  if (col_raw >= B) return;
  float* ya = part_of(Y, rest, ks, A * m * B) + a * m * B + col;
  if (col == col_raw) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = 16 * mt + 4 * qe + v;
        if (i < m) *reinterpret_cast<f32x4u*>(ya + i * B) = f32x4{acc[mt][0][v], acc[mt][1][v], acc[mt][2][v], acc[mt][3][v]};
      }
  } else {
    const int skip = static_cast<int>(col_raw - col);  // columns that the lane before stores
#pragma unroll
    for (int c = 1; c < 4; ++c) {
      if (c < skip) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t i = 16 * mt + 4 * qe + v;
          if (i < m) ya[i * B + c] = acc[mt][c][v];
        }
    }
  }
}

// Binary32 products, one block of 16 k in flight (see launch_ttm_mfma_ws for the sizes that take them).
template <int MT, bool VM>
__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(MT == 4 ? 1 : 2))) void ttm_mfma_f32_kernel(
    const float* __restrict__ X, int64_t A, int64_t K, int64_t B, const float* __restrict__ Mop, int64_t m,
    int64_t chunks, float* __restrict__ Y) {
  const int64_t unit = static_cast<int64_t>(blockIdx.x) * (kMfmaThreads / kWave) + threadIdx.x / kWave;
  if (unit < A * chunks) ttm_f32_unit<MT, VM, 1, MT == 1>(X, A, K, B, Mop, m, chunks, 1, (K + 3) / 4 * 4, Y, nullptr, unit);
}

// Independent binary32 contractions of one shape class in one launch: job q owns the
// units [unit0_q, unit0_q + A_q chunks_q ksplit_q).
struct F32Job {
  const float* X;
  const float* Mop;
  float* Y;
  float* rest;
  int64_t A, K, B, m, chunks, kper, unit0;
  int ksplit;
};
struct F32JobTable {
  F32Job j[kMaxF32Group];
  int count;
};
template <int MT, bool VM>
__global__ __launch_bounds__(kMfmaThreads) void ttm_mfma_f32_grouped_kernel(F32JobTable tab) {
  const int64_t unit = static_cast<int64_t>(blockIdx.x) * (kMfmaThreads / kWave) + threadIdx.x / kWave;
  int q = 0;
  for (int t = 1; t < tab.count; ++t)
    if (unit >= tab.j[t].unit0) q = t;
  const F32Job& J = tab.j[q];
  const int64_t local = unit - J.unit0;
  if (local >= J.A * J.chunks * J.ksplit) return;
  ttm_f32_unit<MT, VM, 3, false>(J.X, J.A, J.K, J.B, J.Mop, J.m, J.chunks, J.ksplit, J.kper, J.Y, J.rest, local);
}

// Last-mode contraction (B == 1): Y[a, i] = sum_k X[a, k] M[i, k], a GEMM with
// the long contiguous rows of X as the reduction axis.  A wave owns 64 rows of X
// (four 16-row MFMA tiles) and reads them with 16-byte loads along k, at whatever boundary the
// rows start; the packed operand supplies the 16-row tiles of M.  A lane's 16 bytes are its
// share of one or four products: 8 k of one 16x16x32 bfloat16 product, or one k of four 16x16x4
// binary32 ones (k = k0 + 4 q + s in product s).  (bfloat16 X, and binary32 rows that are not a
// multiple of four long, ran on the vector ALU before, a thread a row: the core
// step of a 160 x 96 x 336 bfloat16 tensor 222 us, now 43; of a 161 x 119 x 267 binary32 one 195, now 53)
template <typename TX>
struct LastIO;
template <>
struct LastIO<float> {
  typedef f32x4 vec_t;
  typedef f32x4u load_t;
  static constexpr int kPer = 4;  // k a lane
  static __device__ __forceinline__ vec_t zero() { return vec_t{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ vec_t part(const float* p, int n) {  // the first n values
    vec_t v = zero();
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < n) v[c] = p[c];
    return v;
  }
  static __device__ __forceinline__ f32x4 mac(vec_t m, vec_t x, f32x4 acc, int c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(m[c], x[c], acc, 0, 0, 0);
  }
  static constexpr int kMacs = 4;
};
template <>
struct LastIO<bf16_t> {
  typedef u32x4 vec_t;
  typedef u32x4u load_t;
  static constexpr int kPer = 8;
  static __device__ __forceinline__ vec_t zero() { return vec_t{0u, 0u, 0u, 0u}; }
  static __device__ __forceinline__ vec_t part(const bf16_t* p, int n) {
    vec_t v = zero();
#pragma unroll
    for (int w = 0; w < 4; ++w)
      v[w] = (2 * w < n ? p[2 * w] : 0u) | (2 * w + 1 < n ? static_cast<uint32_t>(p[2 * w + 1]) << 16 : 0u);
    return v;
  }
  static __device__ __forceinline__ f32x4 mac(vec_t m, vec_t x, f32x4 acc, int) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, x), acc, 0,
                                                   0, 0);
  }
  static constexpr int kMacs = 1;
};

template <typename TX, int MT, bool PARTS, bool EVEN>
__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(MT == 1 ? 4 : MT >= 3 ? 2 : EVEN ? 4 : 3))) void
ttm_mfma_last_kernel(const TX* __restrict__ X, int64_t A, int64_t K, const TX* __restrict__ Mop, int64_t m, int ksplit,
                     int64_t kper, float* __restrict__ Y) {
  typedef LastIO<TX> IO;
  typedef typename IO::vec_t vec_t;
  constexpr int kBlock = 4 * IO::kPer;  // k a step
  const int lane = threadIdx.x % kWave;
  const int64_t unit = static_cast<int64_t>(blockIdx.x) * (kMfmaThreads / kWave) + threadIdx.x / kWave;
  const int64_t groups = (A + 63) / 64;
  if (unit >= groups * ksplit) return;
  const int ks = static_cast<int>(unit % ksplit);
  const int64_t a0 = (unit / ksplit) * 64;
  const int r16 = lane % 16, q = lane / 16;
  const int64_t kbeg = ks * kper;
  const int64_t kend = (kbeg + kper < K) ? kbeg + kper : K;
  // PARTS: sums of 64 k, added up in `sum`
  f32x4 acc[MT][4], sum[PARTS ? MT : 1][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int at = 0; at < 4; ++at) acc[mt][at] = sum[PARTS ? mt : 0][at] = f32x4{0.f, 0.f, 0.f, 0.f};
  const auto close_part = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int at = 0; at < 4; ++at) {
        sum[PARTS ? mt : 0][at] += acc[mt][at];
        acc[mt][at] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  // The next step's k are loaded while the current ones are multiplied.  A row past A reads row
  // A - 1 (its products land only in output rows that are not stored); in the range's last step
  // k past kend is zero in both operands.  EVEN (binary32 on the 16-byte grid): the loads carry no
  // conditions, k past kend reads the range's last four and is zeroed when it is taken over.
  const TX* xr[4];
#pragma unroll
  for (int at = 0; at < 4; ++at) {
    const int64_t a = a0 + 16 * at + r16;
    xr[at] = X + ((a < A) ? a : A - 1) * K + IO::kPer * q;
  }
  const TX* mr = Mop + r16 * K + IO::kPer * q;
  vec_t nx[4], nw[MT];
  const auto load = [&](int64_t k0) {
    if constexpr (EVEN) {
      const int64_t kc = (k0 + IO::kPer * q < kend) ? k0 : kend - IO::kPer * (q + 1);
#pragma unroll
      for (int at = 0; at < 4; ++at) nx[at] = *reinterpret_cast<const vec_t*>(xr[at] + kc);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nw[mt] = *reinterpret_cast<const vec_t*>(mr + 16 * mt * K + kc);
    } else if (k0 + kBlock <= kend) {
#pragma unroll
      for (int at = 0; at < 4; ++at) nx[at] = *reinterpret_cast<const typename IO::load_t*>(xr[at] + k0);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nw[mt] = *reinterpret_cast<const typename IO::load_t*>(mr + 16 * mt * K + k0);
    } else if (k0 < kend) {
      const int64_t left = kend - (k0 + IO::kPer * q);
      const int n = left < 0 ? 0 : (left < IO::kPer ? static_cast<int>(left) : IO::kPer);
#pragma unroll
      for (int at = 0; at < 4; ++at) nx[at] = IO::part(xr[at] + k0, n);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nw[mt] = IO::part(mr + 16 * mt * K + k0, n);
    }
  };
  load(kbeg);
  for (int64_t k0 = kbeg; k0 < kend; k0 += kBlock) {
    vec_t xv[4], mv[MT];
#pragma unroll
    for (int at = 0; at < 4; ++at) xv[at] = nx[at];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) mv[mt] = nw[mt];
    if constexpr (EVEN) {
      const bool kin = k0 + IO::kPer * q < kend;
#pragma unroll
      for (int at = 0; at < 4; ++at) xv[at] = kin ? xv[at] : IO::zero();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) mv[mt] = kin ? mv[mt] : IO::zero();
    }
    __builtin_amdgcn_sched_barrier(0);
    load(k0 + kBlock);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < IO::kMacs; ++c)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int at = 0; at < 4; ++at) acc[mt][at] = IO::mac(mv[mt], xv[at], acc[mt][at], c);
    if (PARTS && (k0 - kbeg) % 64 == 64 - kBlock) close_part();
  }
  if constexpr (PARTS) close_part();
  float* y = Y + static_cast<int64_t>(ks) * A * m;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int at = 0; at < 4; ++at) {
      const int64_t a = a0 + 16 * at + r16;
      if (a >= A) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = 16 * mt + 4 * q + v;
        if (i < m) y[a * m + i] = (PARTS ? sum[PARTS ? mt : 0][at] : acc[mt][at])[v];
      }
    }
}

__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

// bfloat16 contraction on 16x16x32 products.  A wave owns 128 columns of one slab (lane j: eight
// consecutive columns, at any 2-byte boundary) and takes k in blocks of 32: lane group q loads
// the rows k0 + 8 q .. + 7, with the next block in flight during the block's products, and packs
// the eight k of a column just before its products (which keeps two waves on a SIMD).  The waves
// of a workgroup share the k range, and M is staged in LDS 64 k at a time, double-buffered, zero
// past the range.  Bound: HBM.  Rows off the 16-byte grid ran on the vector ALU before, at a
// twentieth of the rate: the core step of 293 x 544 x 387 took 456 us, now 67.
// With four row tiles the registers do not suffice: with 512 threads five are put aside around the
// loop, with 256 also a part of the next window of M, once in 64 k.
template <int MT, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void ttm_mfma_bf16_kernel(
    const bf16_t* __restrict__ X, int64_t A, int64_t K, int64_t B, const bf16_t* __restrict__ Mop, int64_t m,
    int64_t chunks, int64_t groups, int64_t kper, float* __restrict__ Y, float* __restrict__ rest) {
  __shared__ __align__(16) uint16_t sM[2][16 * MT * kSplitStride];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int j = lane % 16, q = lane / 16;
  const int64_t ks = blockIdx.x / groups;
  const int64_t unit_raw = (blockIdx.x - ks * groups) * (NT / kWave) + tid / kWave;
  const bool active = unit_raw < A * chunks;
  const int64_t unit = active ? unit_raw : 0;
  const int64_t a = unit / chunks;
  const int64_t col_raw = (unit - a * chunks) * kUnitCols + 8 * j;
  // a lane whose columns run past B takes the last eight: its results repeat its neighbour's
  const int64_t col = col_raw + 8 <= B ? col_raw : B - 8;
  const int64_t kbeg = ks * kper;
  const int64_t kend = (kbeg + kper < K) ? kbeg + kper : K;
  const bf16_t* xa = X + a * K * B + col;

  f32x4 acc[MT][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // as in the binary32 kernel: the lane's rows of a block at xp; in the range's last block rows
  // past kend read row kend - 1 again (zeroed when the block is taken over)
  u32x4 rn[8];
  const bf16_t* xp = xa + (kbeg + 8 * q) * B;
  const auto load = [&](int64_t k0) {
    if (k0 + 32 <= kend) {
#pragma unroll
      for (int t = 0; t < 8; ++t) rn[t] = *reinterpret_cast<const u32x4u*>(xp + t * B);
    } else if (k0 < kend) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int64_t k = k0 + 8 * q + t;
        rn[t] = *reinterpret_cast<const u32x4u*>(xa + (k < kend ? k : kend - 1) * B);
      }
    }
    xp += 32 * B;
  };
  // staging: group g = NT i + tid of a window is row g / 8, k = kw + 8 (g % 8) ..
  constexpr int kGroups = 16 * MT * (kSplitWin / 8), kPer = (kGroups + NT - 1) / NT;
  u32x4 sv[kPer];
  const auto stage_load = [&](int64_t kw) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int g = i * NT + tid;
      if (g >= kGroups) break;
      const int64_t k = kw + 8 * (g % 8);
      const bf16_t* src = Mop + static_cast<int64_t>(g / 8) * K + k;
      if (k + 8 <= kend) {
        sv[i] = *reinterpret_cast<const u32x4u*>(src);
      } else {
#pragma unroll
        for (int w = 0; w < 4; ++w)
          sv[i][w] = (k + 2 * w < kend ? src[2 * w] : 0u) |
                     (k + 2 * w + 1 < kend ? static_cast<uint32_t>(src[2 * w + 1]) << 16 : 0u);
      }
    }
  };
  const auto stage_store = [&](int b) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int g = i * NT + tid;
      if (g >= kGroups) break;
      *reinterpret_cast<u32x4*>(&sM[b][(g / 8) * kSplitStride + 8 * (g % 8)]) = sv[i];
    }
  };
  load(kbeg);
  stage_load(kbeg);
  stage_store(0);
  __syncthreads();
  int buf = 0, half = 0;
  for (int64_t k0 = kbeg; k0 < kend; k0 += 32) {
    const bool more = k0 + (kSplitWin - 32 * half) < kend;
    if (half == 0 && more) stage_load(k0 + kSplitWin);
    u32x4 r[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) r[t] = rn[t];
    if (k0 + 32 > kend) {
#pragma unroll
      for (int t = 0; t < 8; ++t)
        if (k0 + 8 * q + t >= kend) r[t] = u32x4{0u, 0u, 0u, 0u};
    }
    __builtin_amdgcn_sched_barrier(0);
    load(k0 + 32);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 mv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      mv[mt] = *reinterpret_cast<const bf16x8*>(&sM[buf][(16 * mt + j) * kSplitStride + 32 * half + 8 * q]);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4 op;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t lo = r[2 * w][c / 2], hi = r[2 * w + 1][c / 2];
        op[w] = (c % 2 == 0) ? pack_lo(lo, hi) : pack_hi(lo, hi);
      }
      const bf16x8 bv = __builtin_bit_cast(bf16x8, op);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mv[mt], bv, acc[mt][c], 0, 0, 0);
    }
    half ^= 1;
    if (half == 0 || k0 + 32 >= kend) {
      if (more) stage_store(buf ^ 1);
      lds_barrier();  // the window is read by every wave and the next one staged; loads of X stay in flight
      buf ^= 1;
    }
  }
  if (!active || col_raw >= B) return;
  float* ya = part_of(Y, rest, ks, A * m * B) + a * m * B + col;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t i = 16 * mt + 4 * q + v;
      if (i >= m) continue;
      f32x4u* dst = reinterpret_cast<f32x4u*>(ya + i * B);
      dst[0] = f32x4{acc[mt][0][v], acc[mt][1][v], acc[mt][2][v], acc[mt][3][v]};
      dst[1] = f32x4{acc[mt][4][v], acc[mt][5][v], acc[mt][6][v], acc[mt][7][v]};
    }
}

// The same with the lane's share of M (eight k of a row) read from the caches beside its rows of X,
// for rows on the 16-byte grid (B and K multiples of eight): without the LDS windows a wave starts its
// products as soon as its own loads are there.  Bound: latency, for the small contractions that run
// here (see bf16_direct_ok).
template <int MT>
__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(2))) void ttm_mfma_bf16_direct_kernel(
    const bf16_t* __restrict__ X, int64_t A, int64_t K, int64_t B, const bf16_t* __restrict__ Mop, int64_t m,
    int64_t chunks, int ksplit, int64_t kper, float* __restrict__ Y, float* __restrict__ rest) {
  const int lane = threadIdx.x % kWave;
  const int64_t unit = static_cast<int64_t>(blockIdx.x) * (kMfmaThreads / kWave) + threadIdx.x / kWave;
  if (unit >= A * chunks * ksplit) return;
  const int ks = static_cast<int>(unit % ksplit);
  const int64_t ac = unit / ksplit;
  const int64_t a = ac / chunks;
  const int j = lane % 16, q = lane / 16;
  const int64_t col = (ac - a * chunks) * kUnitCols + 8 * j;
  const int64_t kbeg = ks * kper;
  const int64_t kend = (kbeg + kper < K) ? kbeg + kper : K;
  f32x4 acc[MT][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The next 32 k are loaded while the current ones are multiplied.  Loads carry no conditions: a
  // block past kend reads the last 8 k of the range (zeroed before use; kbeg and kend are
  // multiples of 8), and columns past B are the last 8 (their products are not stored).
  const bf16_t* xa = X + a * K * B + (col < B ? col : B - 8);
  const bf16_t* ma = Mop + j * K;
  u32x4 rn[8], nw[MT];
  const auto load = [&](int64_t k0) {
    const int64_t k = k0 + 8 * q;
    const int64_t kc = (k < kend) ? k : kend - 8;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) nw[mt] = *reinterpret_cast<const u32x4*>(ma + 16 * mt * K + kc);
#pragma unroll
    for (int t = 0; t < 8; ++t) rn[t] = *reinterpret_cast<const u32x4*>(xa + (kc + t) * B);
  };
  if (kbeg < kend) load(kbeg);
  const u32x4 zero4 = u32x4{0u, 0u, 0u, 0u};
  for (int64_t k0 = kbeg; k0 < kend; k0 += 32) {
    const bool kin = k0 + 8 * q < kend;
    u32x4 r[8], mv[MT];
#pragma unroll
    for (int t = 0; t < 8; ++t) r[t] = kin ? rn[t] : zero4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) mv[mt] = kin ? nw[mt] : zero4;
    __builtin_amdgcn_sched_barrier(0);
    load(k0 + 32);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4 op;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t lo = r[2 * w][c / 2], hi = r[2 * w + 1][c / 2];
        op[w] = (c % 2 == 0) ? pack_lo(lo, hi) : pack_hi(lo, hi);
      }
      const bf16x8 bv = __builtin_bit_cast(bf16x8, op);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, mv[mt]), bv, acc[mt][c], 0, 0, 0);
    }
  }
  if (col >= B) return;
  float* ya = part_of(Y, rest, ks, A * m * B) + a * m * B + col;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t i = 16 * mt + 4 * q + v;
      if (i >= m) continue;
      f32x4u* dst = reinterpret_cast<f32x4u*>(ya + i * B);
      dst[0] = f32x4{acc[mt][0][v], acc[mt][1][v], acc[mt][2][v], acc[mt][3][v]};
      dst[1] = f32x4{acc[mt][4][v], acc[mt][5][v], acc[mt][6][v], acc[mt][7][v]};
    }
}

// Y = sum of the split parts in part order (binary32), stored as TO
template <typename TO>
__global__ __launch_bounds__(256) void sum_splits_kernel(const float* first, const float* __restrict__ rest, int ksplit,
                                                         int64_t n, TO* Y) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride) {
    float s = first[i];
    for (int k = 1; k < ksplit; ++k) s += rest[(k - 1) * n + i];
    Y[i] = static_cast<TO>(s);
  }
}

struct MfmaPlan {
  int64_t chunks;
  int ksplit;
  int64_t kper;
};

MfmaPlan mfma_plan(rt_dtype xdt, int64_t A, int64_t K, int64_t B, int64_t m, int64_t unit_cols) {
  MfmaPlan p;
  p.chunks = ceil_div(B, unit_cols);
  const int64_t units = A * p.chunks;
  const int64_t kgran = (xdt == RT_BF16 || unit_cols == kSplitCols) ? 32 : 4;
  int ks = 1;
  // aim for >= 2048 waves (8 per CU) when K is long enough to split; short K
  // (>= 64 per part) is split too while the partial sums stay under a quarter
  // of the input read
  // (an input that stays in the caches may split down to 32 per part)
  const int64_t in_bytes = A * K * B * (xdt == RT_BF16 ? 2 : 4);
  const bool cached = in_bytes <= (int64_t(32) << 20);
  while (units * ks < 2048 && ks < 16) {
    const int64_t kp = K / (ks * 2);
    const int64_t part_bytes = 2 * ks * A * m * B * 4;
    if (kp >= 256 || (kp >= 64 && part_bytes * 4 <= in_bytes) || (cached && kp >= 32 && part_bytes <= in_bytes))
      ks *= 2;
    else
      break;
  }
  p.ksplit = ks;
  p.kper = ceil_div(ceil_div(K, ks), kgran) * kgran;
  return p;
}

}  // namespace

size_t ttm_generic_ws(rt_dtype xdt, int64_t A, int64_t K, int64_t B, int64_t m) {
  const int ks = generic_ksplit(A, K, B);
  if (ks == 1) return 0;
  return align256(static_cast<size_t>(ks) * A * m * B * (xdt == RT_F64 ? 8 : 4));
}

hipError_t launch_ttm_generic(const void* X, rt_dtype xdt, int64_t A, int64_t K, int64_t B, const void* M,
                              int64_t m, void* Y, void* ws, hipStream_t st, bool mtrans) {
  if (A * B == 0 || m == 0) return hipSuccess;
  switch (xdt) {
    case RT_F64:
      return generic_dispatch<double, double>(static_cast<const double*>(X), A, K, B,
                                              static_cast<const double*>(M), m, static_cast<double*>(Y),
                                              static_cast<double*>(ws), st, mtrans);
    case RT_F32:
      return generic_dispatch<float, float>(static_cast<const float*>(X), A, K, B, static_cast<const float*>(M),
                                            m, static_cast<float*>(Y), static_cast<float*>(ws), st, mtrans);
    case RT_BF16:
      return generic_dispatch<bf16_t, float>(static_cast<const bf16_t*>(X), A, K, B,
                                             static_cast<const float*>(M), m, static_cast<float*>(Y),
                                             static_cast<float*>(ws), st, mtrans);
    case RT_F8E4M3:
      return generic_dispatch<f8_t, float>(static_cast<const f8_t*>(X), A, K, B, static_cast<const float*>(M), m,
                                           static_cast<float*>(Y), static_cast<float*>(ws), st, mtrans);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_ttm_generic_group(const GenericContraction* c, int count, rt_dtype dt, std::vector<SplitSum>& sums,
                                    hipStream_t st) {
  if (dt != RT_F32 && dt != RT_F64) return hipErrorInvalidValue;
  bool few = count > 1 && count <= kMaxF32Group;
  for (int i = 0; i < count; ++i)
    if (c[i].A * c[i].B == 0 || c[i].m == 0 || generic_threads(c[i].A, c[i].B) != kWave) few = false;
  if (few) return dt == RT_F32 ? generic_group<float>(c, count, sums, st) : generic_group<double>(c, count, sums, st);
  for (int i = 0; i < count; ++i) {
    const hipError_t e = launch_ttm_generic(c[i].X, dt, c[i].A, c[i].K, c[i].B, c[i].M, c[i].m, c[i].Y, c[i].ws, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_split_sums(const std::vector<SplitSum>& sums, rt_dtype dt, hipStream_t st) {
  if (sums.empty()) return hipSuccess;
  if (dt == RT_F32) return split_sums<float>(sums, st);
  return dt == RT_F64 ? split_sums<double>(sums, st) : hipErrorInvalidValue;
}

int64_t ttm_mfma_mpad(int64_t m) { return ceil_div(m, 16) * 16; }

bool ttm_mfma_ok(rt_dtype xdt, int64_t A, int64_t K, int64_t B, int64_t m) {
  if (m < 1 || m > 64 || A < 1 || K < 1) return false;
  // rows off the 16-byte grid: the split kernel takes them too, but a contraction with few columns
  // is faster on the vector ALU, whose waves share the rows of M (80 x 49 x 49 over its first
  // mode: 7 us against 9; 250 x 310 x 190 over its second: 42 against 25)
  if (xdt == RT_F32) return B >= 64 && (B % 4 == 0 || A * ceil_div(B, 64) >= 256);
  if (xdt == RT_BF16) return B >= 64 && ((B % 8 == 0 && K % 8 == 0) || A * ceil_div(B, 64) >= 256);
  return false;
}

size_t ttm_mfma_ws(rt_dtype xdt, int64_t A, int64_t K, int64_t B, int64_t m, bool grouped) {
  // (a binary32 contraction that leaves a group and runs alone has as many units or more, and so
  // as many parts or fewer)
  const int64_t unit_cols = (xdt == RT_F32 && !grouped) ? kSplitCols : kUnitCols;
  const int ks = mfma_plan(xdt, A, K, B, m, unit_cols).ksplit;
  if (ks == 1) return 0;
  return align256(static_cast<size_t>(ks - 1) * A * m * B * sizeof(float));
}

namespace {
// Where binary32 products take less time than the three-term ones, which convert every value of X
// and multiply a block of 32 k whatever part of it exists:
//  * up to 16 k (64 x 4 x 4096 with m = 8: 8 us against 12; 16 x 262144, m = 36: 17 and 21);
//  * one 16-row tile of M, whose products are few: 400 x 262144 with m = 8 77 us against 84, 48 x 262144 15
//    and 19, 200 x 400 x 640 34 and 42.  Below 512 units of 128 columns they are alike or the
//    split over k of the other gains more (400 x 4096: 23 against 10), and from 4096 units on
//    HBM bounds both, but for short K (64 x 1048576: 75 and 65; 20 x 1048576: 33 and 39).
bool f32_products_ok(int64_t A, int64_t K, int64_t B, int64_t m) {
  if (B % 4 != 0) return false;
  const int64_t units = A * ceil_div(B, kUnitCols);
  return K <= 16 || (m <= 16 && units >= 512 && (units < 4096 || K <= 24));
}

// Where the bfloat16 contraction reads M from the caches: rows on the 16-byte grid, and too few units
// or too short a K to gain from sharing M (208 x 80 x 112 with m = 60: 11 us, 18 with M in LDS; 480 x 65536:
// 20 and 30; 208 x 512 x 512, m = 60: 32 and 35; 480 x 262144, m = 60: 70 and 61; 208 x 1048576: 170 and 167).
bool bf16_direct_ok(int64_t units, int64_t K, int64_t B) {
  return B % 8 == 0 && K % 8 == 0 && (units < 2048 || (units < 8192 && K <= 256));
}

hipError_t launch_f32_products(const float* X, int64_t A, int64_t K, int64_t B, const float* Mop, int64_t m, float* Y,
                               hipStream_t st) {
  const int64_t chunks = ceil_div(B, kUnitCols);
  const unsigned grid = static_cast<unsigned>(ceil_div(A * chunks, kMfmaThreads / kWave));
#define RT_F32(MTV, VMV) ttm_mfma_f32_kernel<MTV, VMV><<<grid, kMfmaThreads, 0, st>>>(X, A, K, B, Mop, m, chunks, Y)
#define RT_F32_VM(MTV)                \
  do {                                \
    if (K % 4 == 0) RT_F32(MTV, true); \
    else RT_F32(MTV, false);          \
  } while (0)
  switch (ttm_mfma_mpad(m) / 16) {
    case 1: RT_F32_VM(1); break;
    case 2: RT_F32_VM(2); break;
    case 3: RT_F32_VM(3); break;
    default: RT_F32_VM(4); break;
  }
#undef RT_F32_VM
#undef RT_F32
  return hipGetLastError();
}
hipError_t launch_bf16_direct(const bf16_t* X, int64_t A, int64_t K, int64_t B, const bf16_t* Mop, int64_t m,
                              const MfmaPlan& p, float* Y, float* rest, hipStream_t st) {
  const unsigned grid = static_cast<unsigned>(ceil_div(A * p.chunks * p.ksplit, kMfmaThreads / kWave));
#define RT_DIRECT(MTV)                                                                                          \
  ttm_mfma_bf16_direct_kernel<MTV><<<grid, kMfmaThreads, 0, st>>>(X, A, K, B, Mop, m, p.chunks, p.ksplit, p.kper, \
                                                                  Y, rest)
  switch (ttm_mfma_mpad(m) / 16) {
    case 1: RT_DIRECT(1); break;
    case 2: RT_DIRECT(2); break;
    case 3: RT_DIRECT(3); break;
    default: RT_DIRECT(4); break;
  }
#undef RT_DIRECT
  return hipGetLastError();
}

// The kernels that stage M in LDS; the waves of a workgroup share the k range.
hipError_t launch_staged(const void* X, rt_dtype xdt, int64_t A, int64_t K, int64_t B, const void* Mop, int64_t m,
                         const MfmaPlan& p, float* Y, float* rest, hipStream_t st) {
  const int MT = static_cast<int>(ttm_mfma_mpad(m) / 16);
  const int64_t units = A * p.chunks;
  // Binary32: eight waves a workgroup read 2 KB of a row together and split M once for all, but the
  // prologue of the one such workgroup that a CU holds is exposed.  Rows of 131072 columns on gain from
  // 256 k on (2 x 512 x 131072, m = 36: 119 us with four, 112 with eight; 2 x 1024 x 131072, m = 49: 247 and
  // 232; K = 128, m = 27: 256 and 281).  Shorter ones lose, the more the shorter (16 x 512 x 16384, m = 36:
  // 108 and 124; 40 x 1024 x 2048, m = 49: 103 and 117), but for four row tiles and a long K, where four
  // waves wait for M (32 x 1024 x 8192: 241 and 230, 64 x 1024 x 4096: 238 and 233; 512 x 1024 x 640: 299 and 325).
  // A row past the last whole tile on the vector ALU instead of a padded tile (m = 49) was no faster here,
  // unlike with binary32 products.
  // bfloat16: eight for four row tiles of M, which with four waves do not fit the registers (1024 x
  // 262144 with m = 60: 140 us with four, 119 with eight), except in the small contractions, where
  // the second workgroup of a CU is worth more (24576 columns, K = 208: 17.4 and 18.6; 98304: 23.0 and 22.4).
  const bool wide = xdt == RT_BF16 ? MT == 4 && units * K >= 150000
                                   : (B >= 131072 ? p.kper >= 256 : MT == 4 && B >= 4096 && p.kper > 768);
  const int64_t groups = ceil_div(units, wide ? 8 : 4);
  const unsigned grid = static_cast<unsigned>(groups * p.ksplit);
#define RT_TTM(KERNEL, TX, MTV, NTV)                                                                      \
  KERNEL<MTV, NTV><<<grid, NTV, 0, st>>>(static_cast<const TX*>(X), A, K, B, static_cast<const TX*>(Mop), \
                                         m, p.chunks, groups, p.kper, Y, rest)
#define RT_TTM_ANY(MTV)                                                    \
  do {                                                                     \
    if (xdt == RT_BF16) RT_TTM(ttm_mfma_bf16_kernel, bf16_t, MTV, 256);    \
    else if (wide) RT_TTM(ttm_split_f32_kernel, float, MTV, 512);          \
    else RT_TTM(ttm_split_f32_kernel, float, MTV, 256);                    \
  } while (0)
  if (xdt == RT_BF16 && wide) {
    RT_TTM(ttm_mfma_bf16_kernel, bf16_t, 4, 512);
  } else {
    switch (MT) {
      case 1: RT_TTM_ANY(1); break;
      case 2: RT_TTM_ANY(2); break;
      case 3: RT_TTM_ANY(3); break;
      default: RT_TTM_ANY(4); break;
    }
  }
#undef RT_TTM_ANY
#undef RT_TTM
  return hipGetLastError();
}
}  // namespace

hipError_t launch_ttm_mfma_ws(const void* X, rt_dtype xdt, int64_t A, int64_t K, int64_t B, const void* Mop,
                              int64_t m, float* Y, void* ws, hipStream_t st, std::vector<SplitSum>* later) {
  if (xdt == RT_F32 && f32_products_ok(A, K, B, m) && reinterpret_cast<uintptr_t>(X) % 16 == 0)
    return launch_f32_products(static_cast<const float*>(X), A, K, B, static_cast<const float*>(Mop), m, Y, st);
  const MfmaPlan p = mfma_plan(xdt, A, K, B, m, xdt == RT_F32 ? kSplitCols : kUnitCols);
  float* rest = static_cast<float*>(ws);
  hipError_t e;
  if (xdt == RT_BF16 && bf16_direct_ok(A * p.chunks, K, B) && reinterpret_cast<uintptr_t>(X) % 16 == 0)
    e = launch_bf16_direct(static_cast<const bf16_t*>(X), A, K, B, static_cast<const bf16_t*>(Mop), m, p, Y, rest, st);
  else
    e = launch_staged(X, xdt, A, K, B, Mop, m, p, Y, rest, st);
  if (e != hipSuccess || p.ksplit == 1) return e;
  const int64_t n = A * m * B;
  if (later) {
    later->push_back(SplitSum{Y, rest, Y, n, p.ksplit});
    return hipSuccess;
  }
  const unsigned g2 = static_cast<unsigned>(ceil_div(n, 256) > 8192 ? 8192 : ceil_div(n, 256));
  sum_splits_kernel<float><<<g2, 256, 0, st>>>(Y, rest, p.ksplit, n, Y);
  return hipGetLastError();
}

hipError_t launch_ttm_mfma_f32_group(const F32Contraction* c, int count, std::vector<SplitSum>& sums, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  // one launch needs one kernel instance: every job with the same tile count and M load, and
  // rows that start on 16-byte boundaries
  int mt0 = -1;
  bool vm0 = true, same = count <= kMaxF32Group;
  for (int i = 0; i < count && same; ++i) {
    const int mt = static_cast<int>(ttm_mfma_mpad(c[i].m) / 16);
    const bool vm = c[i].K % 4 == 0;
    if (c[i].B % 4 != 0 || reinterpret_cast<uintptr_t>(c[i].X) % 16 != 0) same = false;
    if (i == 0) {
      mt0 = mt;
      vm0 = vm;
    } else if (mt != mt0 || vm != vm0) {
      same = false;
    }
  }
  if (!same || count == 1) {
    for (int i = 0; i < count; ++i) {
      const hipError_t e =
          launch_ttm_mfma_ws(c[i].X, RT_F32, c[i].A, c[i].K, c[i].B, c[i].Mop, c[i].m, c[i].Y, c[i].ws, st, &sums);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  F32JobTable tab{};
  tab.count = count;
  int64_t units = 0;
  for (int i = 0; i < count; ++i) {
    const MfmaPlan p = mfma_plan(RT_F32, c[i].A, c[i].K, c[i].B, c[i].m, kUnitCols);
    F32Job& J = tab.j[i];
    J.X = c[i].X;
    J.Mop = c[i].Mop;
    J.Y = c[i].Y;
    J.rest = static_cast<float*>(c[i].ws);
    J.A = c[i].A; J.K = c[i].K; J.B = c[i].B; J.m = c[i].m;
    J.chunks = p.chunks;
    J.kper = p.kper;
    J.ksplit = p.ksplit;
    J.unit0 = units;
    units += c[i].A * p.chunks * p.ksplit;
    if (p.ksplit > 1) sums.push_back(SplitSum{J.Y, J.rest, J.Y, c[i].A * c[i].m * c[i].B, p.ksplit});
  }
  const unsigned grid = static_cast<unsigned>(ceil_div(units, kMfmaThreads / kWave));
#define RT_LAUNCH_GROUP(MTV)                                                                     \
  if (vm0)                                                                                       \
    ttm_mfma_f32_grouped_kernel<MTV, true><<<grid, kMfmaThreads, 0, st>>>(tab);                  \
  else                                                                                           \
    ttm_mfma_f32_grouped_kernel<MTV, false><<<grid, kMfmaThreads, 0, st>>>(tab)
  switch (mt0) {
    case 1: RT_LAUNCH_GROUP(1); break;
    case 2: RT_LAUNCH_GROUP(2); break;
    case 3: RT_LAUNCH_GROUP(3); break;
    default: RT_LAUNCH_GROUP(4); break;
  }
#undef RT_LAUNCH_GROUP
  return hipGetLastError();
}

bool ttm_mfma_last_ok(rt_dtype xdt, int64_t A, int64_t K, int64_t m) {
  return (xdt == RT_F32 || xdt == RT_BF16) && A >= 1 && m >= 1 && m <= 64 && K >= 4;
}

bool ttm_mfma_last_pays(rt_dtype xdt, int64_t A, int64_t K, int64_t m) {
  if (!ttm_mfma_last_ok(xdt, A, K, m)) return false;
  if (xdt == RT_F32) return K % 4 == 0 || A * K > 400000 || (m <= 16 && K >= 64);
  return A * K > 200000 || (K >= 32 && (K >= 64 || K % 8 == 0 || m <= 32));
}

namespace {
struct LastPlan {
  int ksplit;
  int64_t kper;
};
LastPlan last_plan(rt_dtype xdt, int64_t A, int64_t K, int64_t m) {
  LastPlan p;
  const int64_t units = ceil_div(A, 64);
  int ks = 1;
  while (units * ks < 2048 && K / (ks * 2) >= 64 && ks < 16 && 2 * ks * A * m * 4 <= A * K * 4) ks *= 2;
  p.ksplit = ks;
  const int64_t step = xdt == RT_F32 ? 16 : 32;  // k a step of the kernel: the parts of K are whole steps
  p.kper = ceil_div(ceil_div(K, ks), step) * step;
  return p;
}
}  // namespace

size_t ttm_mfma_last_ws(int64_t A, int64_t K, int64_t m, bool f64_out) {
  const LastPlan p = last_plan(RT_F32, A, K, m);  // (the split is the same for both types)
  return (p.ksplit == 1 && !f64_out) ? 0 : align256(static_cast<size_t>(p.ksplit) * A * m * sizeof(float));
}

hipError_t launch_ttm_mfma_last(const void* X, rt_dtype xdt, int64_t A, int64_t K, const void* Mop, int64_t m, float* Y,
                                void* ws, hipStream_t st, double* Y64, std::vector<SplitSum>* later) {
  const LastPlan p = last_plan(xdt, A, K, m);
  float* out = (p.ksplit == 1 && !Y64) ? Y : static_cast<float*>(ws);
  const int64_t units = ceil_div(A, 64) * p.ksplit;
  const unsigned grid = static_cast<unsigned>(ceil_div(units, kMfmaThreads / kWave));
  const int MT = static_cast<int>(ttm_mfma_mpad(m) / 16);
  // Rows off the 16-byte grid are summed in parts of 64 k: one chain over a long K rounds more than the
  // parts that the vector-ALU kernel splits it into (1.76e-7 against 1.53e-7 of the
  // norm at K = 267; 1.42e-7 in parts).  On the grid, one chain with loads that carry no conditions is
  // faster for up to two row tiles (112 x 768 x 784 with m = 24: 81 us, 91 in parts).  For more, the
  // parts, with such loads where X stays in the caches (1521 x 384 with m = 55: 17.9 us, 19.5 with
  // conditions; 5332 x 784, m = 39: 21.0 and 22.5; 20000 x 384, m = 55: 45.0 and 41.7; 100000 x 784: 207 and 174).
  const bool grid16 = xdt == RT_F32 && K % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  const bool even = grid16 && (MT < 3 || A * K <= (int64_t(1) << 22));
#define RT_LAST(TXV, MTV, PV, EV)                                                                                 \
  ttm_mfma_last_kernel<TXV, MTV, PV, EV><<<grid, kMfmaThreads, 0, st>>>(                                          \
      static_cast<const TXV*>(X), A, K, static_cast<const TXV*>(Mop), m, p.ksplit, p.kper, out)
#define RT_LAUNCH_LAST(MTV)                                \
  do {                                                     \
    if (xdt != RT_F32) RT_LAST(bf16_t, MTV, false, false); \
    else if (even) RT_LAST(float, MTV, (MTV >= 3), true);  \
    else RT_LAST(float, MTV, true, false);                 \
  } while (0)
  switch (MT) {
    case 1: RT_LAUNCH_LAST(1); break;
    case 2: RT_LAUNCH_LAST(2); break;
    case 3: RT_LAUNCH_LAST(3); break;
    default: RT_LAUNCH_LAST(4); break;
  }
#undef RT_LAUNCH_LAST
#undef RT_LAST
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || (p.ksplit == 1 && !Y64)) return e;
  const int64_t n = A * m;
  if (later && !Y64) {
    later->push_back(SplitSum{out, out + n, Y, n, p.ksplit});
    return hipSuccess;
  }
  const unsigned g2 = static_cast<unsigned>(ceil_div(n, 256) > 8192 ? 8192 : ceil_div(n, 256));
  if (Y64)
    sum_splits_kernel<double><<<g2, 256, 0, st>>>(out, out + n, p.ksplit, n, Y64);
  else
    sum_splits_kernel<float><<<g2, 256, 0, st>>>(out, out + n, p.ksplit, n, Y);
  return hipGetLastError();
}

int64_t ttm_grouped_blocks(int64_t A, int64_t B, int64_t m, int mt) {
  return ceil_div(A * B, kWave) * ceil_div(m, mt);
}

hipError_t launch_ttm_grouped(const GTtmJob* jobs, const int32_t* blkjob, int count, int64_t total_blocks,
                              rt_dtype xdt, int mt, hipStream_t st) {
  if (count == 0 || total_blocks == 0) return hipSuccess;
  const unsigned g = static_cast<unsigned>(total_blocks);
#define RT_G(TX, TC, MTV) ttm_grouped_kernel<TX, TC, MTV><<<g, kWave, 0, st>>>(jobs, blkjob)
  // the row tile must be exactly the one the block counts were computed with
  if (mt != 8 && mt != 16 && mt != 32) return hipErrorInvalidValue;
  switch (xdt) {
    case RT_F64:
      if (mt == 8) RT_G(double, double, 8); else if (mt == 16) RT_G(double, double, 16); else RT_G(double, double, 32);
      break;
    case RT_F32:
      if (mt == 8) RT_G(float, float, 8); else if (mt == 16) RT_G(float, float, 16); else RT_G(float, float, 32);
      break;
    case RT_BF16:
      if (mt == 8) RT_G(bf16_t, float, 8); else if (mt == 16) RT_G(bf16_t, float, 16); else RT_G(bf16_t, float, 32);
      break;
    default:
      return hipErrorInvalidValue;
  }
#undef RT_G
  return hipGetLastError();
}

}  // namespace rt
