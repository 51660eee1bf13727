// First level of the all-at-once sketch (Alg. 4.4 sketch step with the
// dimension tree of Sec. 4.4): one streaming pass over X, viewed as (A, P, Q)
// with P, Q the sizes of the last two modes, computes both
//   Z = X x_d Phi_d        (the node shared by every sketch that contracts mode d)
//   W = X x_{d-1} Phi_{d-1} (the node of the mode-d sketch)
// so X is read from HBM exactly once for all modes; every later contraction of
// the tree runs on Z or W, which are smaller by I_d/s_d and I_{d-1}/s_{d-1}.
//
// Layout: a 256-thread workgroup owns one slab X[a] (or a row range of it) and a
// range of up to 64*NQ columns.  Lane l holds columns q0 + l + 64*j (coalesced
// row reads), the matching Phi_Q entries in registers, and W accumulators for
// its columns; each row's Z values are reduced across the wave.  Phi_P[:, p]
// is wave-uniform (scalar loads).  Row ranges or column ranges split over
// several workgroups produce partial sums that a second kernel adds in a fixed
// order.
#include <algorithm>

#include "kernels.hpp"

namespace rt {

namespace {

constexpr int kZWThreads = 256;
constexpr int kZWWaves = kZWThreads / kWave;

template <typename TX, typename TC, int NQ, int SMAX>
__global__ __launch_bounds__(kZWThreads) void sketch_zw_kernel(const TX* __restrict__ X, int64_t A, int64_t P,
                                                               int64_t Q, const TC* __restrict__ phiP, int sP,
                                                               const TC* __restrict__ phiQ, int sQ,
                                                               int64_t rows_per_block, int qblocks, int pblocks,
                                                               TC* __restrict__ Zo, TC* __restrict__ Wo) {
  extern __shared__ unsigned char zw_smem[];
  TC* sW = reinterpret_cast<TC*>(zw_smem);  // [waves][sP][64*NQ]
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t blk = blockIdx.x;
  const int qblk = static_cast<int>(blk % qblocks);
  const int64_t rest = blk / qblocks;
  const int pblk = static_cast<int>(rest % pblocks);
  const int64_t a = rest / pblocks;
  const int64_t q0 = static_cast<int64_t>(qblk) * 64 * NQ;
  const bool needZ = Zo != nullptr, needW = Wo != nullptr;

  TC phq[NQ][SMAX];
  TC wacc[NQ][SMAX];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int64_t q = q0 + lane + 64 * j;
#pragma unroll
    for (int c = 0; c < SMAX; ++c) {
      phq[j][c] = (needZ && q < Q && c < sQ) ? phiQ[c * Q + q] : TC(0);
      wacc[j][c] = TC(0);
    }
  }
  const int64_t pbeg = static_cast<int64_t>(pblk) * rows_per_block;
  const int64_t pend = (pbeg + rows_per_block < P) ? pbeg + rows_per_block : P;
  const TX* xa = X + a * P * Q;
  TC* zrow = needZ ? Zo + (static_cast<int64_t>(qblk) * A + a) * P * sQ : nullptr;
  for (int64_t p = pbeg + wave; p < pend; p += kZWWaves) {
    TC x[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int64_t q = q0 + lane + 64 * j;
      x[j] = (q < Q) ? static_cast<TC>(Load<TX>::get(xa, p * Q + q)) : TC(0);
    }
    if (needW) {
#pragma unroll
      for (int c = 0; c < SMAX; ++c) {
        const TC f = (c < sP) ? phiP[c * P + p] : TC(0);
#pragma unroll
        for (int j = 0; j < NQ; ++j) wacc[j][c] = fma(f, x[j], wacc[j][c]);
      }
    }
    if (needZ) {
      TC z[SMAX];
#pragma unroll
      for (int c = 0; c < SMAX; ++c) {
        TC s = TC(0);
#pragma unroll
        for (int j = 0; j < NQ; ++j) s = fma(x[j], phq[j][c], s);
        z[c] = s;
      }
#pragma unroll
      for (int c = 0; c < SMAX; ++c)
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) z[c] += __shfl_xor(z[c], off);
      // lane c stores z[c]
      TC mine = TC(0);
#pragma unroll
      for (int c = 0; c < SMAX; ++c)
        if (lane == c) mine = z[c];
      if (lane < sQ) zrow[p * sQ + lane] = mine;
    }
  }
  if (!needW) return;
  const int width = 64 * NQ;
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int c = 0; c < SMAX; ++c)
      if (c < sP) sW[(wave * sP + c) * width + lane + 64 * j] = wacc[j][c];
  __syncthreads();
  TC* wout = Wo + (static_cast<int64_t>(pblk) * A + a) * sP * Q;
  for (int idx = threadIdx.x; idx < sP * width; idx += kZWThreads) {
    const int c = idx / width, col = idx % width;
    const int64_t q = q0 + col;
    if (q >= Q) continue;
    TC s = TC(0);
    for (int w = 0; w < kZWWaves; ++w) s += sW[(w * sP + c) * width + col];
    wout[c * Q + q] = s;
  }
}

template <typename TC>
__global__ __launch_bounds__(256) void sum_parts_kernel(const TC* __restrict__ part, int parts, int64_t n,
                                                        TC* __restrict__ out) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride) {
    TC s = part[i];
    for (int k = 1; k < parts; ++k) s += part[k * n + i];
    out[i] = s;
  }
}

// ------------------------------------------------------------------ bfloat16 / FP8 on matrix cores
// Same two contractions on MFMA (v_mfma_f32_16x16x32_bf16, binary32 accumulation).
// FP8 e4m3 data is widened exactly to bfloat16 as it is loaded, so it streams at
// one byte per element and multiplies as the FP8 values themselves.
// A wave owns 128 columns of a slab X[a]; CW waves side by side cover the column block (up to 512
// columns) and the workgroup takes 4 / CW slabs (a short last mode keeps all waves busy).  All
// waves step through the same rows, 32 at a time:
//  * W^T tile: out[c][q] = sum_p PhiP[c][p] X[p][q].  Each lane loads an 8 x 8
//    block (8 rows, 8 consecutive columns, 16 bytes per row) and re-packs it in
//    registers into 8 operands holding 8 consecutive p of one column; the wave
//    keeps its 16 x 128 accumulator for the whole row range (no cross-wave sum).
//  * Z tile: out[p][c] = sum_q X[p][q] PhiQ[c][q] over the wave's 128 columns,
//    with the X rows staged row-major in the wave's LDS area as the A operand;
//    the CW waves' partial Z rows are added in LDS in a fixed order, one
//    barrier per step (double-buffered partials).
// The next 32 rows are loaded while the current ones are used.  Rows may start at any boundary:
// a group of eight columns that the row's end cuts runs into the next row (masked when it is
// taken over), except in the tensor's last rows, where it is loaded entry by entry.  Rows beyond P and
// operand rows beyond s are zero.  P, Q >= 16, s <= 8.  EVEN (P, Q multiples of eight): groups lie
// wholly inside or outside the range, and the loads carry no conditions at all: one past the
// range reads the last group in it, zeroed when it is taken over (260 us for 1024 x 1024 x 512
// bfloat16 sketches, 281 with the other form).  (Sizes off the 16-byte grid ran on the
// vector-ALU pass before: all sketches of a 682 x 960 x 138 bfloat16 tensor 413 us, now 92)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(1)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr int kZWColsMfma = 512;
constexpr int kTileStride = 136;  // bf16 per staged row: 128 columns + 8 padding (spreads LDS banks)

// Raw loads of eight consecutive entries and their widening to bfloat16 pairs.  The widening
// happens when a prefetched block is used, so the loads stay in flight across the previous step.
// part: the first n of them, the others zero.
template <typename TX>
struct BlockIO;

template <>
struct BlockIO<bf16_t> {
  typedef u32x4 raw_t;  // 8 bfloat16
  static __device__ __forceinline__ raw_t load(const bf16_t* p) { return *reinterpret_cast<const u32x4u*>(p); }
  static __device__ __forceinline__ raw_t part(const bf16_t* p, int n) {
    raw_t v;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      v[w] = (2 * w < n ? p[2 * w] : 0u) | (2 * w + 1 < n ? static_cast<uint32_t>(p[2 * w + 1]) << 16 : 0u);
    return v;
  }
  static __device__ __forceinline__ u32x4 widen(raw_t v) { return v; }
};

// FP8 e4m3: 8 bytes per row, widened exactly to bfloat16 (every e4m3 value is a
// bfloat16 value) by the hardware conversion, so the products are the FP8 ones
template <>
struct BlockIO<f8_t> {
  typedef u32x2 raw_t;
  static __device__ __forceinline__ raw_t load(const f8_t* p) { return *reinterpret_cast<const u32x2u*>(p); }
  static __device__ __forceinline__ raw_t part(const f8_t* p, int n) {
    raw_t v = u32x2{0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < n) v[e / 4] |= static_cast<uint32_t>(p[e]) << (8 * (e % 4));
    return v;
  }
  static __device__ __forceinline__ u32x4 widen(raw_t v) {
    return u32x4{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[0], 1.0f, false)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[0], 1.0f, true)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[1], 1.0f, false)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[1], 1.0f, true))};
  }
};

// entries of a group of eight that lie before `end` (first: entry 0)
__device__ __forceinline__ int group_count(int64_t first, int64_t end) {
  return first + 8 <= end ? 8 : (first < end ? static_cast<int>(end - first) : 0);
}

template <typename TX, bool EVEN, int CW>
__global__ __launch_bounds__(kZWThreads) __attribute__((amdgpu_waves_per_eu(3))) void sketch_zw_bf16_mfma_kernel(
    const TX* __restrict__ X, int64_t A, int64_t P, int64_t Q, const bf16_t* __restrict__ phiP, int sP,
    const bf16_t* __restrict__ phiQ, int sQ, int64_t rows_per_block, int64_t qcols, int qblocks, int pblocks,
    float* __restrict__ Zo, float* __restrict__ Wo) {
  typedef BlockIO<TX> IO;
  constexpr int kSlabs = kZWWaves / CW;
  __shared__ __align__(16) bf16_t tile[kZWWaves][32 * kTileStride];
  __shared__ float zpart[2][CW > 1 ? kZWWaves : 1][CW > 1 ? 32 * 16 : 1];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t blk = blockIdx.x;
  const int qblk = static_cast<int>(blk % qblocks);
  const int64_t rest = blk / qblocks;
  const int pblk = static_cast<int>(rest % pblocks);
  const int64_t a_raw = (rest / pblocks) * kSlabs + wave / CW;
  const int64_t a = a_raw < A ? a_raw : A - 1;
  const int64_t q0 = static_cast<int64_t>(qblk) * qcols;
  const int64_t qend = (q0 + qcols < Q) ? q0 + qcols : Q;
  const int64_t qw = q0 + 128 * (wave % CW);  // this wave's columns
  const bool on = a_raw < A && qw < qend;     // waves past the last slab or column only keep the barriers
  const bool needZ = Zo != nullptr, needW = Wo != nullptr;
  const int li = lane % 16, kg = lane / 16;
  const int64_t pbeg = static_cast<int64_t>(pblk) * rows_per_block;
  const int64_t pend = (pbeg + rows_per_block < P) ? pbeg + rows_per_block : P;
  const TX* xa = X + a * P * Q;
  float* zout = needZ ? Zo + (static_cast<int64_t>(qblk) * A + a) * P * sQ : nullptr;
  bf16_t* my = tile[wave];
  const int64_t qc = qw + 8 * li;
  const int ncol = group_count(qc, qend);
  u32x4 cmask;  // the lane's columns that exist
#pragma unroll
  for (int w = 0; w < 4; ++w) cmask[w] = (2 * w < ncol ? 0xffffu : 0u) | (2 * w + 1 < ncol ? 0xffff0000u : 0u);

  // loop-invariant PhiQ operands of the Z product: row c = li, 8 columns per k group
  u32x4 bq[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int64_t qk = qw + 32 * ks + 8 * kg;
    const int n = needZ ? group_count(qk, qend) : 0;
    const bf16_t* src = phiQ + static_cast<int64_t>(li) * Q + qk;
    bq[ks] = n == 8 ? BlockIO<bf16_t>::load(src) : BlockIO<bf16_t>::part(src, n);
  }
  f32x4 wacc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) wacc[c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Lane (li, kg) loads rows p0 + 8 kg + t (t < 8), columns qc..qc+7, and the PhiP operand of the
  // W product (row c = li, columns p0 + 8 kg ..).  A column group past qend reads the row's last
  // eight entries; such values are masked when the block is taken over.  In the range's last step
  // a row past pend reads row pend - 1 (zeroed when taken over).
  const int64_t qcc = ncol > 0 ? qc : Q - 8;
  typename IO::raw_t rn[8];
  u32x4 ppn = u32x4{0u, 0u, 0u, 0u};
  const TX* xp = xa + (pbeg + 8 * kg) * Q + qcc;  // the lane's rows of the next step
  const bf16_t* fp = phiP + (needW ? static_cast<int64_t>(li) * P + pbeg + 8 * kg : 0);
  const auto load = [&](int64_t pb) {
    if constexpr (EVEN) {
      const int64_t p = pb + 8 * kg;
      const int64_t pc = p < pend ? p : pend - 8;
      // without W the load reads an entry of PhiQ (in bounds: Z is then computed) and is unused
      ppn = BlockIO<bf16_t>::load(needW ? phiP + static_cast<int64_t>(li) * P + pc
                                        : phiQ + static_cast<int64_t>(li) * Q + (Q - 8));
#pragma unroll
      for (int t = 0; t < 8; ++t) rn[t] = IO::load(xa + (pc + t) * Q + qcc);
      return;
    }
    if (pb + 32 <= pend && !(a == A - 1 && pb + 32 >= P)) {
      if (needW) ppn = BlockIO<bf16_t>::load(fp);
#pragma unroll
      for (int t = 0; t < 8; ++t) rn[t] = IO::load(xp + t * Q);
    } else if (pb < pend) {
      const int left = static_cast<int>(pend - pb) - 8 * kg;  // rows of the lane's group that exist
      if (needW) ppn = BlockIO<bf16_t>::part(fp, left);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const TX* src = t < left ? xp + t * Q : xa + (pend - 1) * Q + qcc;
        rn[t] = (ncol == 8 || ncol == 0) ? IO::load(src) : IO::part(src, ncol);
        __builtin_amdgcn_sched_barrier(0);  // (the rows' entry loads all at once need too many registers)
      }
    }
    xp += 32 * Q;
    fp += 32;
  };
  if (CW > 1 && !on)  // a wave without columns adds zeros
    for (int g = lane; g < 2 * 512; g += kWave) zpart[g / 512][wave][g % 512] = 0.f;
  if (CW > 1) __syncthreads();
  if (on) load(pbeg);
  int buf = 0;
  for (int64_t pb = pbeg; pb < pend; pb += 32) {
    if (on) {
      u32x4 r[8];
      const bool in = pb + 8 * kg < pend;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        r[t] = IO::widen(rn[t]);
        if constexpr (EVEN) {
          r[t] = (in && ncol > 0) ? r[t] : u32x4{0u, 0u, 0u, 0u};
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) r[t][w] &= cmask[w];
          if (pb + 8 * kg + t >= pend) r[t] = u32x4{0u, 0u, 0u, 0u};
        }
      }
      const u32x4 pp = (!EVEN || in) ? ppn : u32x4{0u, 0u, 0u, 0u};
      __builtin_amdgcn_sched_barrier(0);
      load(pb + 32);
      __builtin_amdgcn_sched_barrier(0);
      if (needZ) {
        __builtin_amdgcn_wave_barrier();  // the previous step's reads of the staging area stay above
#pragma unroll
        for (int t = 0; t < 8; ++t) *reinterpret_cast<u32x4*>(my + (8 * kg + t) * kTileStride + 8 * li) = r[t];
        __builtin_amdgcn_wave_barrier();  // cross-lane: stores before the reads below
        f32x4 zacc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) {
            const u32x4 xr = *reinterpret_cast<const u32x4*>(my + (16 * mt + li) * kTileStride + 32 * ks + 8 * kg);
            zacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xr),
                                                                __builtin_bit_cast(bf16x8, bq[ks]), zacc[mt], 0, 0, 0);
          }
        // D layout: row 16 mt + 4 kg + v, column c = li (addressed from the wave's own row, with one
        // offset a lane: eight of them, kept through the loop, spilled registers)
        const int left = pend - pb < 32 ? static_cast<int>(pend - pb) : 32, zoff = 4 * kg * sQ + li;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = 16 * mt + 4 * kg + v;
            if constexpr (CW > 1)
              zpart[buf][wave][row * 16 + li] = zacc[mt][v];
            else if (li < sQ && row < left)
              (zout + (pb + 16 * mt + v) * sQ)[zoff] = zacc[mt][v];
          }
      }
      if (needW) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          u32x4 op;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t lo = r[2 * w][c / 2], hi = r[2 * w + 1][c / 2];
            op[w] = (c % 2 == 0) ? ((lo & 0xffffu) | (hi << 16)) : ((lo >> 16) | (hi & 0xffff0000u));
          }
          wacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pp),
                                                            __builtin_bit_cast(bf16x8, op), wacc[c], 0, 0, 0);
        }
      }
    }
    if (CW > 1 && needZ) {
      lds_barrier();  // the next rows' loads stay in flight
      // the waves of a slab finish 32 / CW rows of the step each, eight at a time: lane -> (row, c < 8)
      const int first = wave - wave % CW, c = lane % 8;
#pragma unroll
      for (int i = 0; i < 4 / CW; ++i) {
        const int row = (32 / CW) * (wave % CW) + 8 * i + lane / 8;
        const int64_t p = pb + row;
        if (c < sQ && p < pend && a_raw < A) {
          float z = zpart[buf][first][row * 16 + c];
#pragma unroll
          for (int w = 1; w < CW; ++w) z += zpart[buf][first + w][row * 16 + c];
          zout[p * sQ + c] = z;
        }
      }
      buf ^= 1;
    }
  }
  if (!needW || !on || ncol == 0) return;
  // W^T accumulators: row cp = 4 kg + v, column qc + c
  float* wout = Wo + (static_cast<int64_t>(pblk) * A + a) * sP * Q;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int cp = 4 * kg + v;
    if (cp >= sP) continue;
    float* dst = wout + static_cast<int64_t>(cp) * Q + qc;
    if (ncol == 8) {
      reinterpret_cast<f32x4u*>(dst)[0] = f32x4{wacc[0][v], wacc[1][v], wacc[2][v], wacc[3][v]};
      reinterpret_cast<f32x4u*>(dst)[1] = f32x4{wacc[4][v], wacc[5][v], wacc[6][v], wacc[7][v]};
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (c < ncol) dst[c] = wacc[c][v];
    }
  }
}

// ------------------------------------------------------------------ binary32 on matrix cores
// The same pass for binary32 X with v_mfma_f32_16x16x4f32.  A wave owns 128 columns of a
// slab X[a]; CW waves side by side cover the column block (up to 512 columns) and the
// workgroup takes 4 / CW slabs, so a tensor whose last mode is short keeps its four waves busy
// (with all four side by side, 128^4 binary32, W alone: 432 us; 216 now).  All waves step
// through the same rows, 16 at a time.  Lane (li, kg) loads row 4t + kg of each row quad t as
// two 16-byte groups (columns 4 li.. and 64 + 4 li..):
//  * W^T: A = PhiP[c][p] (one value per lane), B = the loaded groups, component c
//    giving columns 4 n + c, so four MFMAs cover 64 columns per row quad;
//  * Z: the 16 x 128 tile is staged row-major in the wave's LDS area, 64 columns at a
//    time, and read back with lane (row li, 4 consecutive columns at 4 kg) as A; PhiQ is B, staged in
//    LDS once per workgroup (read from the caches, the 16 rows of a lane group touched 16
//    cache lines per load every step).  Partial Z rows are added across the CW waves in LDS
//    (fixed order).
// PhiP is staged in LDS 64 rows at a time, the next 64 in flight during the current ones.  Rows off the 16-byte
// grid sum W^T over 16 rows, then over those sums, and Z in eight parts: with one chain each the
// rounding errors were 1.4 times those of the vector-ALU pass that they ran on before.  (On the
// aligned path, which always had one chain, the shorter ones halve the error of a decomposition
// and cost 2 % of the pass.)
// VEC: Q % 4 == 0 and X 16-byte aligned, so a 16-byte group lies in one row and on its
// boundary.  Otherwise the groups are loaded at whatever 4-byte boundary they start at, run into
// the next row where the last one is cut by the row's end (masked when it is taken over), and
// are loaded entry by entry in the last rows of the tensor.  (701 x 523 x 389 binary32 on the
// vector-ALU pass instead: 297 us; 192 now,
// 3 TB/s)
// P, A arbitrary, Q >= 4; s <= 8.
constexpr int kF32Stride = 68;  // floats per staged row: 64 + 4 padding (rows four banks apart)
constexpr int kPhiQRows = 8;
constexpr int kPhiQStride = kZWColsMfma + 8;     // floats per row: 16-byte rows, rows 8 banks apart
constexpr int kPhiPWin = 64;                     // rows of PhiP per staged window

// Rows 8 .. 15 of a W^T product are padding, so the sums of two accumulators fit in one register
// each: the lower half of the lanes holds rows 0 .. 7 of the first, the upper half those of the
// second.  add_pair adds both accumulators to such a sum and clears them; split_pair gives them back.
__device__ __forceinline__ void add_pair(f32x4& sum, f32x4& a, f32x4& b) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[v]), __float_as_uint(b[v]), false, false);
    sum[v] += __uint_as_float(both[0]);
    a[v] = 0.f;
    b[v] = 0.f;
  }
}
__device__ __forceinline__ void split_pair(const f32x4& sum, f32x4& a, f32x4& b) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    a[v] = sum[v];
    b[v] = __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(sum[v]), 0u, false, false)[1]);
  }
}

template <bool NZ, bool NW, bool VEC, int CW>
__global__ __launch_bounds__(kZWThreads) __attribute__((amdgpu_waves_per_eu(3))) void sketch_zw_f32_mfma_kernel(
    const float* __restrict__ X, int64_t A, int64_t P, int64_t Q, const float* __restrict__ phiP, int sP,
    const float* __restrict__ phiQ, int sQ, int64_t rows_per_block, int64_t qcols, int qblocks, int pblocks,
    float* __restrict__ Zo, float* __restrict__ Wo) {
  constexpr int kSlabs = kZWWaves / CW;
  __shared__ __align__(16) float tile[NZ ? kZWWaves : 1][NZ ? 16 * kF32Stride : 4];
  __shared__ float zpart[2][NZ && CW > 1 ? kZWWaves : 1][NZ && CW > 1 ? 16 * 16 : 1];
  __shared__ __align__(16) float sPhiQ[NZ ? kPhiQRows * kPhiQStride : 4];  // PhiQ rows < 8 of the block's columns
  __shared__ float sPhiP[2][NW ? kPhiPWin * 16 : 1];  // window of PhiP, [p][c]
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t blk = blockIdx.x;
  const int qblk = static_cast<int>(blk % qblocks);
  const int64_t rest = blk / qblocks;
  const int pblk = static_cast<int>(rest % pblocks);
  const int64_t a_raw = (rest / pblocks) * kSlabs + wave / CW;
  const int64_t a = a_raw < A ? a_raw : A - 1;
  const int64_t q0 = static_cast<int64_t>(qblk) * qcols;
  const int64_t qend = (q0 + qcols < Q) ? q0 + qcols : Q;
  const int64_t qw = q0 + 128 * (wave % CW);
  const bool on = a_raw < A && qw < qend;  // waves past the last slab or column only keep the barriers
  const int li = lane % 16, kg = lane / 16;
  const int64_t pbeg = static_cast<int64_t>(pblk) * rows_per_block;
  const int64_t pend = (pbeg + rows_per_block < P) ? pbeg + rows_per_block : P;
  const float* xa = X + a * P * Q;
  float* my = tile[NZ ? wave : 0];
  const int64_t qc[2] = {qw + 4 * li, qw + 64 + 4 * li};
  const bool ok[2] = {qc[0] < qend, qc[1] < qend};

  f32x4 wacc[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) wacc[j][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // !VEC: sums of 16 rows each (add_pair)
  f32x4 wsum[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h) wsum[j][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  const auto flush_w = [&]() {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) add_pair(wsum[j][h], wacc[j][2 * h], wacc[j][2 * h + 1]);
  };

  // The next step's rows are loaded while the current step is multiplied.  Loads carry no
  // per-lane conditions: a row past pend reads row pend - 1 and a column group past qend the
  // last group of the row; such values are zeroed when the step is taken over.
  const int64_t qlast = Q - 4;
  const int64_t qcc[2] = {ok[0] ? qc[0] : qlast, ok[1] ? qc[1] : qlast};
  f32x4 rn[4][2];
  const auto load_step = [&](int64_t pb) {
    // groups cut by the end of the tensor's last row are loaded entry by entry
    const bool tail = !VEC && a == A - 1 && pb + 16 >= P;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t p = pb + 4 * t + kg;
      const int64_t pc = (p < pend) ? p : pend - 1;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float* src = xa + pc * Q + qcc[j];
        if constexpr (VEC) {
          rn[t][j] = *reinterpret_cast<const f32x4*>(src);
        } else if (!tail) {
          rn[t][j] = *reinterpret_cast<const f32x4u*>(src);
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) rn[t][j][c] = src[qcc[j] + c < Q ? c : 0];
        }
      }
    }
  };
  if (on) load_step(pbeg);  // in flight while the factors are staged
  // thread: rows pl + 16 u of the window, column c of PhiP; zero past pend
  const int pl = threadIdx.x % 16, pcol = threadIdx.x / 16;
  float pv[kPhiPWin / 16];
  const auto phip_load = [&](int64_t pw) {
#pragma unroll
    for (int u = 0; u < kPhiPWin / 16; ++u) {
      const int64_t p = pw + pl + 16 * u;
      pv[u] = p < pend ? phiP[static_cast<int64_t>(pcol) * P + p] : 0.f;
    }
  };
  const auto phip_store = [&](int b) {
#pragma unroll
    for (int u = 0; u < kPhiPWin / 16; ++u) sPhiP[b][(pl + 16 * u) * 16 + pcol] = pv[u];
  };
  if constexpr (NW) {
    phip_load(pbeg);
    phip_store(0);
  }
  if constexpr (NZ && CW > 1) {
    if (!on)  // a wave without columns adds zeros
      for (int g = lane; g < 2 * 256; g += kWave) zpart[g / 256][wave][g % 256] = 0.f;
  }
  if constexpr (NZ) {
    // PhiQ (sQ <= 8) for the block's columns, zero past sQ and past qend
    constexpr int kV = VEC ? 4 : 1, kRow = 128 * CW / kV;
    for (int g = threadIdx.x; g < kPhiQRows * kRow; g += kZWThreads) {
      const int c = g / kRow, q = kV * (g % kRow);
      const float* src = phiQ + static_cast<int64_t>(c) * Q + q0 + q;
      const bool in = c < sQ && q0 + q < qend;
      if constexpr (VEC)
        *reinterpret_cast<f32x4*>(&sPhiQ[c * kPhiQStride + q]) =
            in ? *reinterpret_cast<const f32x4*>(src) : f32x4{0.f, 0.f, 0.f, 0.f};
      else
        sPhiQ[c * kPhiQStride + q] = in ? *src : 0.f;
    }
  }
  __syncthreads();
  int buf = 0, win = 0;
  for (int64_t pb = pbeg; pb < pend; pb += 16) {
    const int step = static_cast<int>((pb - pbeg) / 16) % (kPhiPWin / 16);  // of the window
    const bool more = pb - 16 * step + kPhiPWin < pend;
    if (NW && step == 0 && more) phip_load(pb + kPhiPWin);
    if (on) {
      f32x4 r[4][2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool pin = pb + 4 * t + kg < pend;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if constexpr (VEC) {
            r[t][j] = (ok[j] && pin) ? rn[t][j] : f32x4{0.f, 0.f, 0.f, 0.f};
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) r[t][j][c] = (pin && qc[j] + c < qend) ? rn[t][j][c] : 0.f;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      load_step(pb + 16);  // past pend: clamped, never used
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (NW) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float pp = sPhiP[win][(16 * step + 4 * t + kg) * 16 + li];  // zero past pend
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              wacc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(pp, r[t][j][c], wacc[j][c], 0, 0, 0);
        }
        if constexpr (!VEC) flush_w();
      }
      if constexpr (NZ) {
        f32x4 zacc = f32x4{0.f, 0.f, 0.f, 0.f}, zp[4];
        // the 16 x 128 tile in two halves of 64 columns (a 16 x 64 stage per wave)
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
          if (kb % 4 == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) zp[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            __builtin_amdgcn_wave_barrier();  // the previous half's reads of the stage stay above
#pragma unroll
            for (int t = 0; t < 4; ++t)
              *reinterpret_cast<f32x4*>(my + (4 * t + kg) * kF32Stride + 4 * li) = r[t][kb / 4];
            __builtin_amdgcn_wave_barrier();  // cross-lane: stores before the reads below
          }
          const int qk = 128 * (wave % CW) + 16 * kb + 4 * kg;
          f32x4 bq = *reinterpret_cast<const f32x4*>(&sPhiQ[(li & (kPhiQRows - 1)) * kPhiQStride + qk]);
          if (li >= kPhiQRows) bq = f32x4{0.f, 0.f, 0.f, 0.f};
          const f32x4 xr = *reinterpret_cast<const f32x4*>(my + li * kF32Stride + 16 * (kb % 4) + 4 * kg);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            f32x4& z = VEC ? zacc : zp[c];
            z = __builtin_amdgcn_mfma_f32_16x16x4f32(xr[c], bq[c], z, 0, 0, 0);
          }
          if (!VEC && kb % 4 == 3) zacc += (zp[0] + zp[1]) + (zp[2] + zp[3]);
        }
        // D layout: row 4 kg + v, column c = li
        if constexpr (CW > 1) {
#pragma unroll
          for (int v = 0; v < 4; ++v) zpart[buf][wave][(4 * kg + v) * 16 + li] = zacc[v];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int64_t p = pb + 4 * kg + v;
            if (li < sQ && p < pend) Zo[((static_cast<int64_t>(qblk) * A + a) * P + p) * sQ + li] = zacc[v];
          }
        }
      }
    }
    // the next window is stored before the last step's barrier: its area was last read in the
    // window before this one
    const bool turn = NW && step == kPhiPWin / 16 - 1 && more;
    if (turn) phip_store(win ^ 1);
    if constexpr (NZ && CW > 1) {
      lds_barrier();  // the next rows' loads stay in flight
      // the waves of a slab finish 16 / CW rows of the step each: lane -> (row, c)
      constexpr int kZRows = 16 / CW;
      const int row = kZRows * (wave % CW) + lane / 8, c = lane % 8;
      const int64_t p = pb + row;
      if (lane / 8 < kZRows && c < sQ && p < pend && a_raw < A) {
        const int first = wave - wave % CW;
        float z = zpart[buf][first][row * 16 + c];
#pragma unroll
        for (int w = 1; w < CW; ++w) z += zpart[buf][first + w][row * 16 + c];
        Zo[((static_cast<int64_t>(qblk) * A + a) * P + p) * sQ + c] = z;
      }
      buf ^= 1;
    }
    if (turn) {
      if constexpr (!(NZ && CW > 1)) lds_barrier();
      win ^= 1;
    }
  }
  if (!NW || !on) return;
  if constexpr (!VEC) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) split_pair(wsum[j][h], wacc[j][2 * h], wacc[j][2 * h + 1]);
  }
  float* wout = Wo + (static_cast<int64_t>(pblk) * A + a) * sP * Q;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (!ok[j]) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int cp = 4 * kg + v;
      if (cp >= sP) continue;
      float* dst = wout + static_cast<int64_t>(cp) * Q + qc[j];
      if constexpr (VEC) {
        *reinterpret_cast<f32x4*>(dst) = f32x4{wacc[j][0][v], wacc[j][1][v], wacc[j][2][v], wacc[j][3][v]};
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (qc[j] + c < qend) dst[c] = wacc[j][c][v];
      }
    }
  }
}

int nq_max(rt_dtype xdt) { return xdt == RT_F64 ? 4 : 8; }

int pick_nq(rt_dtype xdt, int64_t Q) {
  const int64_t need = ceil_div(Q, 64);
  const int mx = nq_max(xdt);
  int nq = 1;
  while (nq < need && nq < mx) nq *= 2;
  return nq;
}

template <typename TX, typename TC>
hipError_t zw_dispatch(const TX* X, int64_t A, int64_t P, int64_t Q, const TC* phiP, int sP, const TC* phiQ, int sQ,
                       TC* Zo, TC* Wo, const ZWPlan& plan, int nq, hipStream_t st) {
  const int smax = (sP > sQ ? sP : sQ) <= 4 ? 4 : 8;
  const int64_t blocks = A * plan.pblocks * plan.qblocks;
  const size_t shmem = Wo ? static_cast<size_t>(kZWWaves) * sP * 64 * nq * sizeof(TC) : 0;
#define RT_ZW(NQV, SV)                                                                                        \
  sketch_zw_kernel<TX, TC, NQV, SV><<<static_cast<unsigned>(blocks), kZWThreads, shmem, st>>>(               \
      X, A, P, Q, phiP, sP, phiQ, sQ, plan.rows_per_block, static_cast<int>(plan.qblocks),                      \
      static_cast<int>(plan.pblocks), Zo, Wo)
  if (smax == 4) {
    switch (nq) {
      case 1: RT_ZW(1, 4); break;
      case 2: RT_ZW(2, 4); break;
      case 4: RT_ZW(4, 4); break;
      default: RT_ZW(8, 4); break;
    }
  } else {
    switch (nq) {
      case 1: RT_ZW(1, 8); break;
      case 2: RT_ZW(2, 8); break;
      case 4: RT_ZW(4, 8); break;
      default: RT_ZW(8, 8); break;
    }
  }
#undef RT_ZW
  return hipGetLastError();
}

}  // namespace

bool sketch_zw_ok(rt_dtype, int64_t sP, int64_t sQ) { return sP >= 1 && sQ >= 1 && sP <= 8 && sQ <= 8; }

// Where binary32 rows off the 16-byte grid are faster on the vector ALU, given the row ranges of all
// slabs.  A matrix-core step of 16 rows takes a wave about 2 us however small the grid is; the vector ALU
// splits the rows among up to 2048 workgroups but reduces every row of Z across a wave.  200 rows of 90
// columns with s = 5: 15 us against 36 for 24 slabs, 36 and 36 for 192, 53 and 37 for 384; s = 3: 13 and 36,
// 23 and 36, 35 and 36.  Past 256 columns a lane of the vector ALU has eight of them (300 x 510, s = 5:
// 25 and 34 for 24 slabs, 49 and 37 for 96).
static bool zw_few_slabs(int64_t ranges, int64_t Q, int64_t s) {
  return Q % 4 != 0 && ranges < (s <= 4 ? (Q <= 256 ? 400 : 200) : (Q <= 256 ? 200 : 64));
}

ZWPlan sketch_zw_plan(rt_dtype xdt, int64_t A, int64_t P, int64_t Q, int64_t sP, int64_t sQ, bool needZ,
                      bool needW) {
  ZWPlan p;
  // (below 16 entries a row or 16 rows, most of a step's matrix-core tile would be padding)
  p.mfma = xdt != RT_F64 && Q >= 16 && P >= 16;
  const bool mf32 = xdt == RT_F32;
  const int nq = pick_nq(xdt, Q);
  p.qblocks = p.mfma ? ceil_div(Q, kZWColsMfma) : ceil_div(Q, 64 * nq);
  p.qcols = p.mfma ? kZWColsMfma : 64 * nq;
  p.waves_per_slab = kZWWaves;
  if (p.mfma) {
    // the column blocks share the 128-column units evenly, and a block of one or two units leaves
    // waves for further slabs
    const int64_t units = ceil_div(ceil_div(Q, 128), p.qblocks);
    p.qcols = 128 * units;
    p.waves_per_slab = units > 2 ? 4 : static_cast<int>(units);
  }
  if (p.mfma) {
    // Row split for the matrix-core pass: 768 workgroups are resident at once
    // (3 per CU).  Cost in units of "one row per resident workgroup":
    //   rows_per_block * max(1, workgroups / 768)  +  partial-W traffic of pb row ranges,
    // with the W partials (written and re-read, binary32) converted at the bytes of X that one
    // row of the resident workgroups is (512 columns each, over their slabs).  A grid of at
    // least one full round streams at about the same rate whether its last round is full or not (the
    // pass is bound by HBM), so rounds count fractionally; a grid below one round is
    // bound by its longest workgroup.  (Counting the last round as full chose three row
    // ranges for 1024 x 1024 x 512 binary32, 20 us per decomposition slower than one.)
    const int64_t resident = 768;
    const int64_t step = mf32 ? 16 : 32;  // rows per step of the kernel
    const double row_bytes = static_cast<double>(resident) * kZWColsMfma * (mf32 ? 4 : 2);
    const int64_t slab_groups = ceil_div(A, kZWWaves / p.waves_per_slab);
    double best = 0.0;
    int64_t best_rows = 0;
    for (int64_t pb = 1; pb <= 64; ++pb) {
      const int64_t rows = ceil_div(ceil_div(P, pb), step) * step;
      const int64_t pbs = ceil_div(P, rows);
      if (pbs != pb || (pb > 1 && rows < 128)) continue;
      const int64_t wgs = slab_groups * p.qblocks * pb;
      const double rounds = wgs > resident ? static_cast<double>(wgs) / resident : 1.0;
      const double t = rounds * rows +
                       (pb > 1 && needW ? 2.0 * pb * A * sP * Q * 4.0 / row_bytes : 0.0);
      if (best_rows == 0 || t < best) {
        best = t;
        best_rows = rows;
      }
    }
    p.rows_per_block = best_rows ? best_rows : ceil_div(P, step) * step;
    if (mf32 && zw_few_slabs(A * ceil_div(P, p.rows_per_block), Q, std::max(sP, sQ))) {
      p.mfma = false;
      p.qblocks = ceil_div(Q, 64 * nq);
      p.qcols = 64 * nq;
      p.waves_per_slab = kZWWaves;
    }
  }
  if (!p.mfma) {
    int64_t pb = 1;
    const int64_t target = 2048;
    if (A * p.qblocks < target) pb = ceil_div(target, A * p.qblocks);
    int64_t maxpb = ceil_div(P, 16);  // keep at least 16 rows per block
    // (and, where a matrix-core pass would sum W in a few parts, no longer chain of parts: 33 of them, P = 520,
    // had 1.2 times its error)
    if (mf32 && P >= 16 && Q >= 16) maxpb = std::min<int64_t>(maxpb, 16);
    if (pb > maxpb) pb = maxpb;
    if (pb < 1) pb = 1;
    p.rows_per_block = ceil_div(P, pb);
  }
  p.pblocks = ceil_div(P, p.rows_per_block);
  const size_t esz = (xdt == RT_F64) ? 8 : 4;
  size_t ws = 0;
  if (needZ && p.qblocks > 1) ws += align256(static_cast<size_t>(p.qblocks) * A * P * sQ * esz);
  if (needW && p.pblocks > 1) ws += align256(static_cast<size_t>(p.pblocks) * A * sP * Q * esz);
  p.ws_bytes = ws;
  return p;
}

hipError_t launch_sketch_zw(const void* X, rt_dtype xdt, int64_t A, int64_t P, int64_t Q, const void* phiP, int64_t sP,
                            const void* phiQ, int64_t sQ, const void* phiP16, const void* phiQ16, void* Z, void* W,
                            const ZWPlan& plan, void* ws, hipStream_t st) {
  const int nq = pick_nq(xdt, Q);
  const size_t esz = (xdt == RT_F64) ? 8 : 4;
  char* wsp = static_cast<char*>(ws);
  void* zdst = Z;
  void* wdst = W;
  if (Z && plan.qblocks > 1) {
    zdst = wsp;
    wsp += align256(static_cast<size_t>(plan.qblocks) * A * P * sQ * esz);
  }
  if (W && plan.pblocks > 1) {
    wdst = wsp;
    wsp += align256(static_cast<size_t>(plan.pblocks) * A * sP * Q * esz);
  }
  hipError_t e;
  const int isP = static_cast<int>(sP), isQ = static_cast<int>(sQ);
  if (plan.mfma) {
    const int64_t groups = ceil_div(A, kZWWaves / plan.waves_per_slab) * plan.pblocks * plan.qblocks;
    const unsigned g = static_cast<unsigned>(groups);
    if (xdt == RT_F32) {
      const bool vec = Q % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
#define RT_ZWF(NZV, NWV, VV, CWV)                                                                                    \
  sketch_zw_f32_mfma_kernel<NZV, NWV, VV, CWV><<<g, kZWThreads, 0, st>>>(                                            \
      static_cast<const float*>(X), A, P, Q, static_cast<const float*>(phiP16), isP, static_cast<const float*>(phiQ16), \
      isQ, plan.rows_per_block, plan.qcols, static_cast<int>(plan.qblocks), static_cast<int>(plan.pblocks),           \
      static_cast<float*>(zdst), static_cast<float*>(wdst))
#define RT_ZWF_W(NZV, NWV, VV)                            \
  do {                                                    \
    if (plan.waves_per_slab == 1) RT_ZWF(NZV, NWV, VV, 1); \
    else if (plan.waves_per_slab == 2) RT_ZWF(NZV, NWV, VV, 2); \
    else RT_ZWF(NZV, NWV, VV, 4);                         \
  } while (0)
#define RT_ZWF_V(NZV, NWV)                 \
  do {                                     \
    if (vec) RT_ZWF_W(NZV, NWV, true);     \
    else RT_ZWF_W(NZV, NWV, false);        \
  } while (0)
      if (zdst && wdst) RT_ZWF_V(true, true);
      else if (zdst) RT_ZWF_V(true, false);
      else RT_ZWF_V(false, true);
#undef RT_ZWF_V
#undef RT_ZWF_W
#undef RT_ZWF
    }
    else {
      const bool even = P % 8 == 0 && Q % 8 == 0;
#define RT_ZWB(TXV, EV, CWV)                                                                                  \
  sketch_zw_bf16_mfma_kernel<TXV, EV, CWV><<<g, kZWThreads, 0, st>>>(                                         \
      static_cast<const TXV*>(X), A, P, Q, static_cast<const bf16_t*>(phiP16), isP,                           \
      static_cast<const bf16_t*>(phiQ16), isQ, plan.rows_per_block, plan.qcols, static_cast<int>(plan.qblocks), \
      static_cast<int>(plan.pblocks), static_cast<float*>(zdst), static_cast<float*>(wdst))
#define RT_ZWB_T(EV, CWV)                              \
  do {                                                 \
    if (xdt == RT_F8E4M3) RT_ZWB(f8_t, EV, CWV);       \
    else RT_ZWB(bf16_t, EV, CWV);                      \
  } while (0)
#define RT_ZWB_E(CWV)                 \
  do {                                \
    if (even) RT_ZWB_T(true, CWV);    \
    else RT_ZWB_T(false, CWV);        \
  } while (0)
      if (plan.waves_per_slab == 1) RT_ZWB_E(1);
      else if (plan.waves_per_slab == 2) RT_ZWB_E(2);
      else RT_ZWB_E(4);
#undef RT_ZWB_E
#undef RT_ZWB_T
#undef RT_ZWB
    }
    e = hipGetLastError();
  } else
  switch (xdt) {
    case RT_F64:
      e = zw_dispatch<double, double>(static_cast<const double*>(X), A, P, Q, static_cast<const double*>(phiP), isP,
                                      static_cast<const double*>(phiQ), isQ, static_cast<double*>(zdst),
                                      static_cast<double*>(wdst), plan, nq, st);
      break;
    case RT_F32:
      e = zw_dispatch<float, float>(static_cast<const float*>(X), A, P, Q, static_cast<const float*>(phiP), isP,
                                    static_cast<const float*>(phiQ), isQ, static_cast<float*>(zdst),
                                    static_cast<float*>(wdst), plan, nq, st);
      break;
    case RT_BF16:
      e = zw_dispatch<bf16_t, float>(static_cast<const bf16_t*>(X), A, P, Q, static_cast<const float*>(phiP), isP,
                                     static_cast<const float*>(phiQ), isQ, static_cast<float*>(zdst),
                                     static_cast<float*>(wdst), plan, nq, st);
      break;
    default:
      e = zw_dispatch<f8_t, float>(static_cast<const f8_t*>(X), A, P, Q, static_cast<const float*>(phiP), isP,
                                   static_cast<const float*>(phiQ), isQ, static_cast<float*>(zdst),
                                   static_cast<float*>(wdst), plan, nq, st);
      break;
  }
  if (e != hipSuccess) return e;
  // fixed-order sums of the partials
  if (Z && plan.qblocks > 1) {
    const int64_t n = A * P * sQ;
    const unsigned g = static_cast<unsigned>(ceil_div(n, 256) > 4096 ? 4096 : ceil_div(n, 256));
    if (xdt == RT_F64)
      sum_parts_kernel<double><<<g, 256, 0, st>>>(static_cast<const double*>(zdst), static_cast<int>(plan.qblocks), n,
                                                  static_cast<double*>(Z));
    else
      sum_parts_kernel<float><<<g, 256, 0, st>>>(static_cast<const float*>(zdst), static_cast<int>(plan.qblocks), n,
                                                 static_cast<float*>(Z));
  }
  if (W && plan.pblocks > 1) {
    const int64_t n = A * sP * Q;
    const unsigned g = static_cast<unsigned>(ceil_div(n, 256) > 4096 ? 4096 : ceil_div(n, 256));
    if (xdt == RT_F64)
      sum_parts_kernel<double><<<g, 256, 0, st>>>(static_cast<const double*>(wdst), static_cast<int>(plan.pblocks), n,
                                                  static_cast<double*>(W));
    else
      sum_parts_kernel<float><<<g, 256, 0, st>>>(static_cast<const float*>(wdst), static_cast<int>(plan.pblocks), n,
                                                 static_cast<float*>(W));
  }
  return hipGetLastError();
}

}  // namespace rt
