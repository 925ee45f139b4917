// The deep part of the Wide & Deep click-through-rate model (Appendix C,
// "Click-through-rate prediction"): an MLP over the concatenated field
// embeddings, forward and backward in fp64 on the matrix cores.
//
// The products are the only dense contractions of the store's tasks; they
// run on v_mfma_f64_16x16x4f64, whose operands and results a wavefront holds
// as: lane l passes a = A[l % 16][l / 16] (16 x 4) and b = B[l / 16][l % 16]
// (4 x 16) and holds c[v] = C[l / 16 + 4 v][l % 16] of the 16 x 16 result.
#pragma once

#include "common.hpp"
#include "push.hpp"

namespace adapm {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ GEMM
// C[M][N] = op(A)[M][K] op(B)[K][N], all sums in fp64.
// op(A)[m][k] = TA ? A[k * lda + m] : A[m * lda + k]; op(B) likewise with
// TB.  B's elements are fp32 (the dense parameters) or fp64.
//
// A workgroup computes a TM x TN tile of C (128 x 128, 64 x 128 or 64 x 64),
// each of its four wavefronts a quarter as products of 16 x 16, with no LDS
// and no barrier: a fp64 16x16x4 product occupies its matrix core for 64
// cycles, so a wave's 64 products of 16 K steps (128 x 128) take 4,096 cycles
// and need 12-16 KB of operands, which the L1 and L2 deliver in a fifth of
// that time; each wave loads the next K step's operands into a second
// register set while the matrix cores work on the current one, and waits for
// nobody.  Which k a lane group multiplies is free as long as both operands
// agree, and so are the rows and columns of a product: lane group g takes the
// KK neighbouring k at KK g of a step, and lane position r the MI
// neighbouring rows (NJ columns) at MI r (NJ r), so that every load is a
// vector of neighbouring elements and a lane stores neighbouring results.
// Counters of the products of a step of 8,192 samples (1,664 and 1,024 wide):
// matrix cores busy 82-91% of the time, 58-65 TFLOP/s.  Staging the operands through LDS with a barrier per
// 16 K steps reached 52-57, and 39 where the fp32 operand was converted next
// to its load, which then was waited for at once.
//
// Rows and columns past the end are clamped to the last ones that exist: the
// lanes compute and store those results twice, with equal bits, and no access
// needs a predicate.  Only the last K step, and products with fewer rows or
// columns than one lane's vector, load element by element.
//
// Tiles are dealt to the dies in contiguous runs (xcd_slot), so the tiles
// that share A's rows, and the slices of a split K, stay in one L2.  With S > 1
// slices of K, slice z writes its partial product to C + z * M * N (EPI_NONE
// only); k_sum_slices adds them in slice order.
//
// EPI_BIAS_RELU: C = max(product + bias[n], 0), a forward layer.
// EPI_RELU_MASK: C = H[m][n] > 0 ? product : 0, the gradient of the layer
// below (H its activations, same shape and stride as C).
constexpr int GEMM_BK = 16;   // K slices are multiples of this
enum { EPI_NONE = 0, EPI_BIAS_RELU = 1, EPI_RELU_MASK = 2 };

// n neighbouring elements (8, 16 or 32 bytes), aligned like one element.
template <typename T, int n>
__device__ __forceinline__ void load_elems(const T* __restrict__ p, T* out) {
  if constexpr (n == 4 && sizeof(T) == 8) {
    load_elems<T, 2>(p, out);
    load_elems<T, 2>(p + 2, out + 2);
  } else {
    typedef T vec __attribute__((ext_vector_type(n), aligned(sizeof(T))));
    const vec x = *reinterpret_cast<const vec*>(p);
#pragma unroll
    for (int e = 0; e < n; ++e) out[e] = x[e];
  }
}

// One wave's operand of a K step: v[kk][i] is element i of the lane's ROWS
// neighbouring rows (columns of B) at k = KK g + kk.  KMAJOR: memory rows run
// along k (the lane's rows are neighbours in memory), else along the rows.
template <typename T, int KK, int ROWS, bool KMAJOR>
struct GemmOperand {
  T v[KK][ROWS];
  __device__ __forceinline__ void load(const T* __restrict__ p, int64_t ld) {   // p: the lane's first element
    if constexpr (KMAJOR) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) load_elems<T, ROWS>(p + kk * ld, v[kk]);
    } else {
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        T x[KK];
        load_elems<T, KK>(p + i * ld, x);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) v[kk][i] = x[kk];
      }
    }
  }
  // element by element: rows clamped to nr - 1, zeros from k = kend on
  __device__ __forceinline__ void load_edge(const T* __restrict__ base, int64_t ld, int64_t row, int64_t nr, int64_t k,
                                            int64_t kend) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const int64_t r = row + i < nr ? row + i : nr - 1;
        const int64_t q = k + kk;
        v[kk][i] = q < kend ? base[KMAJOR ? q * ld + r : r * ld + q] : T(0);
      }
  }
};

template <bool TA, bool TB, typename BT, int TM, int TN, int EPI>
__global__ __launch_bounds__(BLOCK, 2) void k_gemm_f64(int64_t M, int64_t N, int64_t K, const double* __restrict__ A,
                                                       int64_t lda, const BT* __restrict__ B, int64_t ldb,
                                                       double* __restrict__ C, int64_t ldc, int64_t kslice, int gx,
                                                       int gy, const float* __restrict__ bias,
                                                       const double* __restrict__ H) {
  constexpr int MI = TM / 32, NJ = TN / 32;   // products of a wave along m and n
  constexpr int KK = sizeof(BT) == 4 ? 4 : 2; // k per lane group and step (two register sets have to fit)
  constexpr int STEP = 4 * KK;
  const int lane = threadIdx.x % WAVE;
  const int wave = threadIdx.x / WAVE;
  const int r = lane % 16, g = lane / 16;
  const int id = (int)xcd_slot(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(id / gx % gy) * TM + (wave / 2) * (TM / 2);
  const int64_t n0 = (int64_t)(id % gx) * TN + (wave % 2) * (TN / 2);
  const int64_t z = id / (gx * gy);
  const int64_t kbeg = z * kslice;
  const int64_t kend = kbeg + kslice < K ? kbeg + kslice : K;
  C += z * M * N;
  // first row (column) of lane position q, so that the vector stays inside
  const bool vec = M >= MI && N >= NJ;
  auto row_of = [&](int q) -> int64_t {
    const int64_t m = m0 + MI * q;
    return !vec || m < M - MI ? m : M - MI;
  };
  auto col_of = [&](int q) -> int64_t {
    const int64_t n = n0 + NJ * q;
    return !vec || n < N - NJ ? n : N - NJ;
  };
  const int64_t row = row_of(r), col = col_of(r);
  const double* pa = A + (TA ? (kbeg + KK * g) * lda + row : row * lda + kbeg + KK * g);
  const BT* pb = B + (TB ? col * ldb + kbeg + KK * g : (kbeg + KK * g) * ldb + col);
  const int64_t da = TA ? STEP * lda : STEP, db = TB ? STEP : STEP * ldb;

  struct Set {
    GemmOperand<double, KK, MI, TA> a;
    GemmOperand<BT, KK, NJ, !TB> b;
  } set[2];
  auto load = [&](Set& x) {
    x.a.load(pa, lda);
    x.b.load(pb, ldb);
    pa += da;
    pb += db;
  };

  f64x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto products = [&](const Set& x) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      double b[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = (double)x.b.v[kk][j];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a.v[kk][i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  // whole steps in vectors, two at a time through the two sets, then the rest
  const int64_t nfull = vec && kbeg < kend ? (kend - kbeg) / STEP : 0;
  if (nfull > 0) load(set[0]);
  for (int64_t s = 0; s < nfull; s += 2) {
    if (s + 1 < nfull) load(set[1]);
    products(set[0]);
    if (s + 2 < nfull) load(set[0]);
    if (s + 1 < nfull) products(set[1]);
  }
  for (int64_t k0 = kbeg + nfull * STEP; k0 < kend; k0 += STEP) {
    set[0].a.load_edge(A, lda, row, M, k0 + KK * g, kend);
    set[0].b.load_edge(B, ldb, col, N, k0 + KK * g, kend);
    products(set[0]);
  }
  // result v of product (i, j): lane position g + 4 v along m, r along n
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      int64_t m = row_of(g + 4 * v) + i;
      m = m < M ? m : M - 1;
      double* out = C + m * ldc + col;
      const double* h = EPI == EPI_RELU_MASK ? H + m * ldc + col : nullptr;
      double x[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) x[j] = acc[i][j][v];
      if (vec) {
        if constexpr (EPI == EPI_BIAS_RELU) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            x[j] += (double)bias[col + j];
            x[j] = x[j] > 0.0 ? x[j] : 0.0;
          }
        } else if constexpr (EPI == EPI_RELU_MASK) {
          double hv[NJ];
          load_elems<double, NJ>(h, hv);
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            if (!(hv[j] > 0.0)) x[j] = 0.0;
        }
        typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
        for (int j = 0; j < NJ; j += 2) *reinterpret_cast<f64x2u*>(out + j) = f64x2u{x[j], x[j + 1]};
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          if (col + j >= N) continue;
          if constexpr (EPI == EPI_BIAS_RELU) {
            x[j] += (double)bias[col + j];
            x[j] = x[j] > 0.0 ? x[j] : 0.0;
          } else if constexpr (EPI == EPI_RELU_MASK) {
            if (!(h[j] > 0.0)) x[j] = 0.0;
          }
          out[j] = x[j];
        }
      }
    }
}

// out[i] = sum over z of part[z * count + i], z = 0 .. S-1 in order.
__global__ __launch_bounds__(BLOCK) void k_sum_slices(const double* __restrict__ part, int64_t S, int64_t count,
                                                      double* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
    double t = 0.0;
    int64_t z = 0;
    for (; z + 4 <= S; z += 4) {
      double x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = part[(z + q) * count + i];
#pragma unroll
      for (int q = 0; q < 4; ++q) t += x[q];
    }
    for (; z < S; ++z) t += part[z * count + i];
    out[i] = t;
  }
}

// ------------------------------------------------------------------ inputs and head
// X[b][f * E + c] = W[key(b, f)][c] in fp64 (zero rows for skipped samples):
// one group of L lanes per (sample, field) row.
template <int L, int NV, int VW>
__global__ __launch_bounds__(BLOCK) void k_wd_gather(const float* __restrict__ W, int64_t ld,
                                                     const int64_t* __restrict__ keys, int64_t B, int F, int E,
                                                     const uint8_t* __restrict__ ok, double* __restrict__ X) {
  constexpr int GPB = BLOCK / L;
  const int gl = threadIdx.x % L;
  const int64_t n = B * F;
  for (int64_t i = (int64_t)blockIdx.x * GPB + threadIdx.x / L; i < n; i += (int64_t)gridDim.x * GPB) {
    const int64_t b = i / F;
    const bool valid = ok[b];
    const float* row = W + (valid ? keys[i] : 0) * ld;
    double* out = X + i * E;   // row b, field f: X + (b * F + f) * E
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int c = (gl + v * L) * VW;
      if (c < E) {
        float x[VW];
        if (valid) load_frag<VW>(row + c, x);
#pragma unroll
        for (int e = 0; e < VW; ++e)
          if (c + e < E) out[c + e] = valid ? (double)x[e] : 0.0;
      }
    }
  }
}

// One wavefront per sample: logit = h_L . w + c + sum of the F wide weights
// (field order), the logistic loss, dlogit = sigmoid(logit) - label (0 for
// skipped samples) and dH_L = dlogit w, masked by h_L > 0 when h_L is a
// ReLU layer (relu = 0: no hidden layer, h_L is the input x itself).
__global__ __launch_bounds__(BLOCK) void k_wd_head(const double* __restrict__ H, int64_t Hn,
                                                   const float* __restrict__ w, const float* __restrict__ c,
                                                   const float* __restrict__ W, int64_t ld, int E,
                                                   const int64_t* __restrict__ keys, int F,
                                                   const float* __restrict__ label, const uint8_t* __restrict__ ok,
                                                   int64_t B, int relu, double* __restrict__ dlogit,
                                                   double* __restrict__ dH, double* __restrict__ loss_part) {
  const int lane = threadIdx.x % WAVE;
  double lsum = 0.0;
  for (int64_t b = (int64_t)blockIdx.x * WAVES_PER_BLOCK + threadIdx.x / WAVE; b < B;
       b += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const double* h = H + b * Hn;
    const bool valid = ok[b];
    // the wide weights, one field per lane, added in field order
    double wide = 0.0;
    for (int f0 = 0; f0 < F; f0 += WAVE) {
      const int nf = F - f0 < WAVE ? F - f0 : WAVE;
      const float x = valid && lane < nf ? W[keys[b * F + f0 + lane] * ld + E] : 0.0f;
      for (int f = 0; f < nf; ++f) wide += (double)__shfl(x, f, WAVE);
    }
    double s = 0.0;
    int64_t n0 = lane;
    for (; n0 + 7 * WAVE < Hn; n0 += 8 * WAVE) {   // eight loads in flight
      double x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = h[n0 + q * WAVE];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += x[q] * (double)w[n0 + q * WAVE];
    }
    for (; n0 < Hn; n0 += WAVE) s += h[n0] * (double)w[n0];
    s = group_sum<WAVE>(s);
    const double logit = s + (double)c[0] + wide;
    const double y = (double)label[b];
    double g = 0.0;
    if (valid) {
      // softplus(z) - y z, and sigmoid(z) - y, in forms that do not overflow
      const double sp = logit > 0.0 ? logit + log1p(exp(-logit)) : log1p(exp(logit));
      if (lane == 0) lsum += sp - y * logit;
      g = (logit >= 0.0 ? 1.0 / (1.0 + exp(-logit)) : exp(logit) / (1.0 + exp(logit))) - y;
    }
    if (lane == 0) dlogit[b] = g;
    n0 = lane;
    for (; n0 + 7 * WAVE < Hn; n0 += 8 * WAVE) {
      double x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = h[n0 + q * WAVE];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int64_t n = n0 + q * WAVE;
        dH[b * Hn + n] = (!relu || x[q] > 0.0) ? g * (double)w[n] : 0.0;
      }
    }
    for (; n0 < Hn; n0 += WAVE) dH[b * Hn + n0] = (!relu || h[n0] > 0.0) ? g * (double)w[n0] : 0.0;
  }
  __shared__ double sm[WAVES_PER_BLOCK];
  lsum = block_sum_double(lsum, sm);
  if (threadIdx.x == 0) loss_part[blockIdx.x] = lsum;
}

// Column sums out[n] = sum_b A[b][n] s[b] (s = 1 without a scale), in two
// deterministic stages: block (x, y) sums rows [y R, (y + 1) R) of 64 columns
// into part[y][n], each of its four wavefronts every fourth row with eight
// loads in flight, the wavefronts' sums added in order; then the parts are
// added likewise.  Bound by reading A once: 128 rows per block give a batch of
// 8,192 x 1,024 its 1,024 workgroups (256 rows of 256 columns, one load in
// flight per thread, took 77 us for its 67 MB; a single column, 8 KB, as long).
constexpr int64_t COLSUM_ROWS = 128;
constexpr int COLSUM_COLS = 64;

__device__ __forceinline__ void colsum_block(const double* __restrict__ A, int64_t r0, int64_t r1, int64_t cols,
                                             const double* __restrict__ s, double* __restrict__ out) {
  __shared__ double sm[WAVES_PER_BLOCK][COLSUM_COLS];
  const int64_t n = (int64_t)blockIdx.x * COLSUM_COLS + threadIdx.x % WAVE;
  const int w = threadIdx.x / WAVE;
  const bool in = n < cols;
  double t = 0.0;
  int64_t r = r0 + w;
  for (; r + 7 * WAVES_PER_BLOCK < r1; r += 8 * WAVES_PER_BLOCK) {
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = in ? A[(r + q * WAVES_PER_BLOCK) * cols + n] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) t += s ? x[q] * s[r + q * WAVES_PER_BLOCK] : x[q];
  }
  for (; r < r1; r += WAVES_PER_BLOCK) {
    const double x = in ? A[r * cols + n] : 0.0;
    t += s ? x * s[r] : x;
  }
  sm[w][threadIdx.x % WAVE] = t;
  __syncthreads();
  if (w == 0 && in) {
    double a = sm[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < WAVES_PER_BLOCK; ++q) a += sm[q][threadIdx.x];
    out[n] = a;
  }
}

__global__ __launch_bounds__(BLOCK) void k_colsum_part(const double* __restrict__ A, int64_t rows, int64_t cols,
                                                       const double* __restrict__ s, double* __restrict__ part) {
  const int64_t r0 = (int64_t)blockIdx.y * COLSUM_ROWS;
  const int64_t r1 = r0 + COLSUM_ROWS < rows ? r0 + COLSUM_ROWS : rows;
  colsum_block(A, r0, r1, cols, s, part + (int64_t)blockIdx.y * cols);
}

__global__ __launch_bounds__(BLOCK) void k_colsum_final(const double* __restrict__ part, int64_t nparts, int64_t cols,
                                                        double* __restrict__ out) {
  colsum_block(part, 0, nparts, cols, nullptr, out);
}

// Per-occurrence gradient rows at the occurrence's sorted position:
// [dX[b][f E .. f E + E) | dlogit[b] | 0 ...] rounded to fp32 (zeros for
// skipped samples, whose occurrences sort last and are not merged).
__global__ __launch_bounds__(BLOCK) void k_wd_rows(const double* __restrict__ dX, const double* __restrict__ dlogit,
                                                   int64_t B, int F, int E, int dim, const uint32_t* __restrict__ rank,
                                                   float* __restrict__ grads) {
  const int64_t n = B * F;
  for (int64_t i = (int64_t)blockIdx.x * WAVES_PER_BLOCK + threadIdx.x / WAVE; i < n;
       i += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const int lane = threadIdx.x % WAVE;
    const int64_t b = i / F;
    float* out = grads + (int64_t)rank[i] * dim;
    const double* src = dX + i * E;
    for (int c = lane; c < dim; c += WAVE)
      out[c] = c < E ? (float)src[c] : (c == E ? (float)dlogit[b] : 0.0f);
  }
}

// Per-element AdaGrad of the dense buffer from its fp64 gradient, rounded
// once to fp32.
__global__ __launch_bounds__(BLOCK) void k_dense_adagrad(float* __restrict__ w, float* __restrict__ acc,
                                                         const double* __restrict__ g, int64_t n, float lr,
                                                         float eps) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) {
    float wi = w[i], ai = acc[i];
    adagrad_elem(wi, ai, (float)g[i], lr, eps);
    w[i] = wi;
    acc[i] = ai;
  }
}

}  // namespace adapm
