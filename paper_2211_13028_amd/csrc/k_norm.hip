// Relative reconstruction error by explicit residual, in binary64 (Sec. 5):
// the host contracts all modes but the first into T = G x_2 U_2 ... x_d U_d
// (r1 x prod_{k>1} I_k), and this kernel streams X once, reconstructing each
// element as U_1[i, :] . T[:, b] and accumulating ||X - X_hat||^2, ||X||^2 and the
// count of non-finite entries.  Fixed-order reductions (bitwise reproducible).
#include "kernels.hpp"

namespace rt {

namespace {

constexpr int kRThreads = 256;
constexpr int kRCols = 256;   // columns per workgroup: 64 per wave
constexpr int kRChunk = 64;   // rows of U_1 staged in LDS at a time: four 16-row blocks

typedef double rr_f64x4 __attribute__((ext_vector_type(4)));

// Four consecutive entries of a row of X, widened to binary64 when they are used.
template <typename TX>
struct Quad {
  TX v[4];
};
template <typename TX, bool VEC>
__device__ __forceinline__ Quad<TX> load_quad(const TX* __restrict__ p, int n) {
  Quad<TX> q;
  if constexpr (VEC) {
    typedef TX vec_t __attribute__((ext_vector_type(4)));
    const vec_t v = *reinterpret_cast<const vec_t*>(p);
#pragma unroll
    for (int c = 0; c < 4; ++c) q.v[c] = v[c];
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) q.v[c] = p[c < n ? c : 0];
  }
  return q;
}

// A wave owns 64 columns b of the (I1, Brest) view and walks the rows of its range 16 at a
// time.  X_hat of the 16 x 64 block is 4 KS binary64 16x16x4 products: T stays in registers
// as the B operand for the whole range, U_1 (staged in LDS, kRChunk rows at a time) is A.
// Column group c takes the columns b0 + 4 n + c, so a lane's four results of one row are
// four consecutive entries of X: one 16-byte load (binary32) per row, the next block's in
// flight during the products.
//
// Bound: FP64 matrix rate and HBM nearly alike (2 r1 flops per entry against its bytes).
// The row-per-step vector form that this replaces read each U_1 entry from LDS once per
// column of a thread: LDS held it at a fifth of the FP64 rate.  640 x 512 x 480 binary32,
// r = 24: 466 us before, 209 us now (7.6 GFLOP, 36 TFLOP/s; 3.0 TB/s).
//
// A block whose rows and columns all exist and whose entries are all finite takes the
// unmasked path; other blocks mask entry by entry.
template <typename TX, int KS, bool VEC>
__global__ __launch_bounds__(kRThreads) void recon_residual_kernel(const TX* __restrict__ X, int64_t I1, int64_t Brest,
                                                                   const double* __restrict__ U1,
                                                                   const double* __restrict__ T, int r1,
                                                                   int64_t rows, double* __restrict__ part) {
  constexpr int kStride = 4 * KS + 2;
  __shared__ double sU[kRChunk * kStride];
  __shared__ double red[3][kRThreads / kWave];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int r16 = lane % 16, q = lane / 16;
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * kRCols + 64 * wave;
  const int64_t col = b0 + 4 * r16;  // the lane's four columns
  const int ncol = col + 4 <= Brest ? 4 : (col < Brest ? static_cast<int>(Brest - col) : 0);
  const bool wave_on = b0 < Brest, cols_full = b0 + 64 <= Brest;
  const int64_t ibeg = static_cast<int64_t>(blockIdx.y) * rows;
  const int64_t iend = (ibeg + rows < I1) ? ibeg + rows : I1;
  double t[KS][4];
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int k = 4 * s + q;
      t[s][c] = (k < r1 && c < ncol) ? T[static_cast<int64_t>(k) * Brest + col + c] : 0.0;
    }
  double s_res[2] = {0.0, 0.0}, s_x[2] = {0.0, 0.0}, s_bad = 0.0;
  // loads are clamped into the range (row iend - 1, the row's last whole group or its entry
  // 0); what they read there is masked
  const int64_t colc = ncol > 0 ? col : 0;
  Quad<TX> xn[4];
  const auto load = [&](int64_t i0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t i = (i0 + q + 4 * v < iend) ? i0 + q + 4 * v : iend - 1;
      xn[v] = load_quad<TX, VEC>(X + i * Brest + colc, ncol);
    }
  };
  if (wave_on && ibeg < iend) load(ibeg);
  for (int64_t c0 = ibeg; c0 < iend; c0 += kRChunk) {
    __syncthreads();
    for (int idx = threadIdx.x; idx < kRChunk * 4 * KS; idx += kRThreads) {
      const int ii = idx / (4 * KS), k = idx % (4 * KS);
      sU[ii * kStride + k] = (c0 + ii < iend && k < r1) ? U1[(c0 + ii) * r1 + k] : 0.0;
    }
    __syncthreads();
    if (!wave_on) continue;
    for (int64_t i0 = c0; i0 < c0 + kRChunk && i0 < iend; i0 += 16) {
      Quad<TX> x[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = xn[v];
      __builtin_amdgcn_sched_barrier(0);
      load(i0 + 16);  // past iend: clamped, never used
      __builtin_amdgcn_sched_barrier(0);
      rr_f64x4 xh[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) xh[c] = rr_f64x4{0.0, 0.0, 0.0, 0.0};
      const double* u = sU + (i0 - c0 + r16) * kStride + q;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const double av = u[4 * s];
#pragma unroll
        for (int c = 0; c < 4; ++c) xh[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, t[s][c], xh[c], 0, 0, 0);
      }
      // result v of lane (r16, q): row q + 4 v, columns col .. col + 3
      bool fine = cols_full && i0 + 16 <= iend;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < 4; ++c) fine = fine && isfinite(Load<TX>::get(x[v].v, c));
      if (__all(fine)) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double xv = static_cast<double>(Load<TX>::get(x[v].v, c));
            const double d = xv - xh[c][v];
            s_res[c % 2] = fma(d, d, s_res[c % 2]);
            s_x[c % 2] = fma(xv, xv, s_x[c % 2]);
          }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (i0 + q + 4 * v >= iend || c >= ncol) continue;
            const double xv = static_cast<double>(Load<TX>::get(x[v].v, c));
            if (!isfinite(xv)) {
              s_bad += 1.0;
              continue;
            }
            const double d = xv - xh[c][v];
            s_res[c % 2] = fma(d, d, s_res[c % 2]);
            s_x[c % 2] = fma(xv, xv, s_x[c % 2]);
          }
      }
    }
  }
  // fixed-order block reduction
  double sr = s_res[0] + s_res[1], sx = s_x[0] + s_x[1];
  for (int off = 32; off >= 1; off >>= 1) {
    sr += __shfl_xor(sr, off);
    sx += __shfl_xor(sx, off);
    s_bad += __shfl_xor(s_bad, off);
  }
  if (lane == 0) { red[0][wave] = sr; red[1][wave] = sx; red[2][wave] = s_bad; }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0.0;
    for (int i = 0; i < kRThreads / kWave; ++i) s += red[threadIdx.x][i];
    part[(static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = s;
  }
}

// Workgroup 0: out[0], out[1], out[3] = the sums of the residual's partials.  Workgroup 1:
// out[2] = ||G||^2, eight loads of a thread in flight (one dependent load at a time on 256
// threads took 24 us for 24^3 entries).
constexpr int kFinishThreads = 1024;
__global__ __launch_bounds__(kFinishThreads) void residual_finish_kernel(const double* __restrict__ part,
                                                                         int64_t blocks,
                                                                         const double* __restrict__ g, int64_t ng,
                                                                         double* __restrict__ out) {
  constexpr int kWaves = kFinishThreads / kWave;
  __shared__ double red[3][kWaves];
  double s[3] = {0.0, 0.0, 0.0};
  if (blockIdx.x == 0) {
    for (int64_t i = threadIdx.x; i < blocks; i += kFinishThreads)
      for (int k = 0; k < 3; ++k) s[k] += part[i * 3 + k];
  } else {
    for (int64_t i0 = threadIdx.x; i0 < ng; i0 += 8 * kFinishThreads) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t i = i0 + u * kFinishThreads;
        v[u] = i < ng ? g[i] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s[0] = fma(v[u], v[u], s[0]);
    }
  }
  for (int k = 0; k < 3; ++k)
    for (int off = 32; off >= 1; off >>= 1) s[k] += __shfl_xor(s[k], off);
  if (threadIdx.x % kWave == 0)
    for (int k = 0; k < 3; ++k) red[k][threadIdx.x / kWave] = s[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < 3; ++k)
      for (int w = 0; w < kWaves; ++w) v[k] += red[k][w];
    if (blockIdx.x == 0) {
      out[0] = v[0];
      out[1] = v[1];
      out[3] = v[2];
    } else {
      out[2] = v[0];
    }
  }
}

// Row ranges: enough workgroups for four a CU, at least 128 rows each (every range loads its
// share of T again, r1 binary64 values a column: at 128 rows that is half of binary32 X's
// bytes at r1 = 32, and it comes from the caches for the later ranges).
int64_t residual_rows(int64_t I1, int64_t Brest) {
  const int64_t cb = ceil_div(Brest, kRCols);
  int64_t ranges = 1;
  while (cb * ranges < 1024 && I1 / (2 * ranges) >= 128) ranges *= 2;
  return ceil_div(ceil_div(I1, ranges), 16) * 16;
}

template <typename TX>
hipError_t dispatch(const TX* X, int64_t I1, int64_t Brest, const double* U1, const double* T, int64_t r1,
                    double* part, hipStream_t st) {
  const int r = static_cast<int>(r1);
  const int64_t rows = residual_rows(I1, Brest);
  const dim3 grid(static_cast<unsigned>(ceil_div(Brest, kRCols)), static_cast<unsigned>(ceil_div(I1, rows)));
  // whole-group loads need every row to start on a group boundary
  const bool vec = Brest % 4 == 0 && reinterpret_cast<uintptr_t>(X) % (4 * sizeof(TX)) == 0;
#define RT_RR(KSV)                                                                                             \
  if (vec)                                                                                                     \
    recon_residual_kernel<TX, KSV, true><<<grid, kRThreads, 0, st>>>(X, I1, Brest, U1, T, r, rows, part);      \
  else                                                                                                         \
    recon_residual_kernel<TX, KSV, false><<<grid, kRThreads, 0, st>>>(X, I1, Brest, U1, T, r, rows, part)
  // products of four k: r1 rounded up to one of five lengths
  if (r <= 8) { RT_RR(2); }
  else if (r <= 16) { RT_RR(4); }
  else if (r <= 24) { RT_RR(6); }
  else if (r <= 32) { RT_RR(8); }
  else { RT_RR(16); }
#undef RT_RR
  return hipGetLastError();
}

}  // namespace

size_t recon_residual_ws(int64_t I1, int64_t Brest) {
  return align256(static_cast<size_t>(ceil_div(Brest, kRCols) * ceil_div(I1, residual_rows(I1, Brest))) * 3 *
                  sizeof(double));
}

hipError_t launch_recon_residual(const void* X, rt_dtype xdt, int64_t I1, int64_t Brest, const double* U1,
                                 const double* T, int64_t r1, const double* G, int64_t ng, double* out, void* ws,
                                 hipStream_t st) {
  double* part = static_cast<double*>(ws);
  hipError_t e;
  switch (xdt) {
    case RT_F64: e = dispatch(static_cast<const double*>(X), I1, Brest, U1, T, r1, part, st); break;
    case RT_F32: e = dispatch(static_cast<const float*>(X), I1, Brest, U1, T, r1, part, st); break;
    case RT_BF16: e = dispatch(static_cast<const bf16_t*>(X), I1, Brest, U1, T, r1, part, st); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const int64_t blocks = ceil_div(Brest, kRCols) * ceil_div(I1, residual_rows(I1, Brest));
  residual_finish_kernel<<<2, kFinishThreads, 0, st>>>(part, blocks, G, ng, out);
  return hipGetLastError();
}

}  // namespace rt
