// Training of the manifold parameterisation (Sec. "Manifold Construction",
// eq. "loss"; Sec. "Training Details"): encoder q_b = E2 ELU(E1 u_b + c1) + c2,
// decoder g(x_p, q_b) at every point of every snapshot of the batch, loss =
// mean (g - u)^2, gradients by the reverse-mode chain rule written out layer
// by layer, and Adam with bias correction on FP32 master parameters.
//
// The decoder's rows are (snapshot, point) pairs, snapshot-major: row
// b * P + p.  Layer activations a_l = ELU(z_l) are kept for the backward
// pass (ELU'(z) is recovered from a: 1 where a > 0, a + 1 otherwise).  The
// matrix products run on the matrix cores through gemm.hpp, in bfloat16 with
// FP32 accumulation (FP32 when the net's precision is FP32); the first layer
// (K = m + r), the output layer and every reduction over rows are plain
// FP32 kernels with a fixed summation order.
#include <algorithm>

#include "common.hpp"
#include "gemm.hpp"
#include "train_fused.hpp"

namespace crom {

constexpr int MAX_SPLITS = 256;  // split-K partial tiles at most

// ---------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------
template <class T>
__global__ void convert_kernel(const float* __restrict__ a, T* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = (T)a[i];
}

// c[b][u] = b1[u] + sum_k W1[u][m + k] q[b][k]  (FP64 accumulation)
__global__ void fold_kernel(const float* __restrict__ W1, const float* __restrict__ b1, const float* __restrict__ q,
                            int B, int W, int m, int r, float* __restrict__ c) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < B * W; i += gridDim.x * blockDim.x) {
    const int b = i / W, u = i % W;
    double s = b1[u];
    for (int k = 0; k < r; ++k) s += (double)W1[u * (m + r) + m + k] * q[b * r + k];
    c[i] = (float)s;
  }
}

// a1[row][u] = ELU(sum_i W1[u][i] x[p][i] + c[b][u]),  row = b * P + p.
// A thread takes 8 consecutive units of one row (W is a multiple of 8); the
// x-columns of W1 are staged in LDS, and every load of a thread is issued
// before its arithmetic (m is a compile-time constant).
constexpr int EW_MAX_W = 256;  // widest layer of the compiled shapes
constexpr int EW_MAX_MD = 3;   // largest m and d

// Sine networks (SINE): a1 = sin(z), and g1 = cos(z) for the backward.
template <class T, int M, bool SINE = false>
__global__ __launch_bounds__(256) void layer1_kernel(const float* __restrict__ W1, const float* __restrict__ c,
                                                     const float* __restrict__ x, int64_t P, int64_t rows, int W,
                                                     int r, T* __restrict__ a1, T* __restrict__ g1) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  __shared__ float wx[EW_MAX_W * M];
  for (int i = threadIdx.x; i < W * M; i += blockDim.x) wx[i] = W1[(i / M) * (M + r) + i % M];
  __syncthreads();
  const int G = W / 8;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows * G; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = i / G;
    const int u0 = (int)(i - row * G) * 8;
    const int64_t b = row / P, p = row - b * P;
    float xv[M];
#pragma unroll
    for (int k = 0; k < M; ++k) xv[k] = x[p * M + k];
    const float4 c0 = *reinterpret_cast<const float4*>(&c[b * W + u0]);
    const float4 c1 = *reinterpret_cast<const float4*>(&c[b * W + u0 + 4]);
    const float cz[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    vec8 o, oc;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float z = cz[e];
#pragma unroll
      for (int k = 0; k < M; ++k) z += wx[(u0 + e) * M + k] * xv[k];
      if constexpr (SINE) {
        const float rz = reduce_2pi(z);
        o[e] = (T)__sinf(rz);
        oc[e] = (T)__cosf(rz);
      } else {
        o[e] = (T)(z > 0.0f ? z : __expf(z) - 1.0f);
      }
    }
    *reinterpret_cast<vec8*>(&a1[row * W + u0]) = o;
    if constexpr (SINE) *reinterpret_cast<vec8*>(&g1[row * W + u0]) = oc;
  }
}

// g[row][o] = sum_u Wout[o][u] a[row][u] + bout[o]: one thread per row,
// 8 units per load, in unit order; Wout staged in LDS.
template <class T, int D>
__global__ __launch_bounds__(256) void output_kernel(const T* __restrict__ a, const float* __restrict__ Wout,
                                                     const float* __restrict__ bout, int64_t rows, int W,
                                                     float* __restrict__ g) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  __shared__ float wo[EW_MAX_W * D];
  for (int i = threadIdx.x; i < W * D; i += blockDim.x) wo[i] = Wout[i];
  __syncthreads();
  for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < rows;
       row += (int64_t)gridDim.x * blockDim.x) {
    float s[D];
#pragma unroll
    for (int o = 0; o < D; ++o) s[o] = 0.0f;
    for (int u0 = 0; u0 < W; u0 += 8) {
      const vec8 v = *reinterpret_cast<const vec8*>(&a[row * W + u0]);
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int o = 0; o < D; ++o) s[o] += wo[o * W + u0 + e] * (float)v[e];
    }
#pragma unroll
    for (int o = 0; o < D; ++o) g[row * D + o] = s[o] + bout[o];
  }
}

// dg = 2 (g - u) / n and per-block partial sums of (g - u)^2
__global__ void mse_kernel(const float* __restrict__ g, const float* __restrict__ u, int64_t n,
                           float* __restrict__ dg, double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float e = g[i] - u[i];
    dg[i] = 2.0f * e / (float)n;
    s += (double)e * e;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// loss = sum of the block partials / n: each thread adds a strided quarter
// of them, then a fixed-order tree.
__global__ __launch_bounds__(256) void mse_final_kernel(const double* __restrict__ part, int nb, int64_t n,
                                                         float* loss) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(sh[0] / (double)n);
}

// dz[row][u] = (sum_o dg[row][o] Wout[o][u]) * ELU'(a[row][u]); 8 units
// of one row per thread, Wout staged in LDS.
// Sine networks (SINE): `a` holds the stored cos(z) and scales dz directly.
template <class T, int D, bool SINE = false>
__global__ __launch_bounds__(256) void dz_last_kernel(const float* __restrict__ dg, const float* __restrict__ Wout,
                                                      const T* __restrict__ a, int64_t rows, int W,
                                                      T* __restrict__ dz) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  __shared__ float wo[EW_MAX_W * D];
  for (int i = threadIdx.x; i < W * D; i += blockDim.x) wo[i] = Wout[i];
  __syncthreads();
  const int G = W / 8;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows * G; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = i / G;
    const int u0 = (int)(i - row * G) * 8;
    float d[D];
#pragma unroll
    for (int o = 0; o < D; ++o) d[o] = dg[row * D + o];
    const vec8 av = *reinterpret_cast<const vec8*>(&a[row * W + u0]);
    vec8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float s = 0.0f;
#pragma unroll
      for (int o = 0; o < D; ++o) s += d[o] * wo[o * W + u0 + e];
      out[e] = (T)(SINE ? s * (float)av[e] : s * elu_d1_from_a((float)av[e]));
    }
    *reinterpret_cast<vec8*>(&dz[row * W + u0]) = out;
  }
}

// Weighted column sums over row segments, in two fixed-order passes.
//   out[seg][k][col] = sum over rows of the segment of w_k(row) X[row][col]
// with w_0 = 1 and w_k = wt[(row % wmod) * wstride + k - 1] (k = 1..nw-1).
// Pass 1: block (chunk, seg) sums `chunk_rows` rows of its segment.  Its
// threads split into row groups; a thread adds the rows of its group for
// VEC consecutive columns (VEC = 16 bytes of X when the rows are aligned,
// else 1), in FP32, then the groups are added in group order in FP64.
// Pass 2 adds the chunks in a fixed order.
template <class T, int VEC>
__global__ __launch_bounds__(256) void colsum_kernel(const T* __restrict__ X, int64_t ldx, int cols,
                                                     int64_t seg_rows, int chunk_rows,
                                                     const float* __restrict__ wt, int64_t wmod, int wstride,
                                                     int nw, double* __restrict__ part) {
  __shared__ double sh[4][256];
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const int ch = blockIdx.x, seg = blockIdx.y, chunks = gridDim.x;
  const int64_t r0 = (int64_t)ch * chunk_rows;
  const int64_t r1 = min(seg_rows, r0 + chunk_rows);
  const int tid = threadIdx.x;
  for (int c0 = 0; c0 < cols; c0 += 256 * VEC) {
    const int cw = min(256 * VEC, cols - c0);       // columns of this pass
    const int tpr = (cw + VEC - 1) / VEC;           // threads per row
    const int G = 256 / tpr;                        // row groups
    const int cv = tid % tpr, rg = tid / tpr;
    const int col = c0 + cv * VEC;
    float s[4][VEC];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int e = 0; e < VEC; ++e) s[k][e] = 0.0f;
    if (rg < G) {
#pragma unroll 4
      for (int64_t r = r0 + rg; r < r1; r += G) {
        const int64_t row = seg * seg_rows + r;
        float v[VEC];
        if constexpr (VEC > 1) {
          const vec_t x = *reinterpret_cast<const vec_t*>(&X[row * ldx + col]);
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[e] = (float)x[e];
        } else {
          v[0] = (float)X[row * ldx + col];
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[0][e] += v[e];
        for (int k = 1; k < nw; ++k) {
          const float w = wt[(row % wmod) * wstride + (k - 1)];
#pragma unroll
          for (int e = 0; e < VEC; ++e) s[k][e] += v[e] * w;
        }
      }
    }
    for (int e = 0; e < VEC; ++e) {
      for (int k = 0; k < nw; ++k) sh[k][tid] = rg < G ? (double)s[k][e] : 0.0;
      __syncthreads();
      if (tid < tpr && c0 + tid * VEC + e < cols) {
        for (int k = 0; k < nw; ++k) {
          double a = 0.0;
          for (int q = 0; q < G; ++q) a += sh[k][q * tpr + tid];
          part[(((int64_t)seg * chunks + ch) * nw + k) * cols + c0 + tid * VEC + e] = a;
        }
      }
      __syncthreads();
    }
  }
}

// Pass 2: out[seg][k][col] = sum over chunks, in chunk order within each of
// 4 interleaved lanes, then the 4 lanes in order.
__global__ __launch_bounds__(256) void colsum_final_kernel(const double* __restrict__ part, int segs, int chunks,
                                                           int nw, int cols, double* __restrict__ out) {
  __shared__ double sh[4][64];
  const int n_out = nw * cols;
  const int o = blockIdx.x * 64 + (threadIdx.x & 63), lane4 = threadIdx.x >> 6, seg = blockIdx.y;
  double a = 0.0;
  if (o < n_out) {
#pragma unroll 8
    for (int c = lane4; c < chunks; c += 4) a += part[((int64_t)seg * chunks + c) * n_out + o];
  }
  sh[lane4][threadIdx.x & 63] = a;
  __syncthreads();
  if (threadIdx.x < 64 && o < n_out)
    out[(int64_t)seg * n_out + o] = ((sh[0][threadIdx.x] + sh[1][threadIdx.x]) + sh[2][threadIdx.x]) + sh[3][threadIdx.x];
}

constexpr int COLSUM_CHUNKS = 2048;  // partial sums per column sum at most
// Chunks of a snapshot's rows in the column sums (at most COLSUM_CHUNKS, or
// one per segment, in all).
static int row_chunks(int64_t rows, int segs) {
  const int64_t chunks = (rows + 255) / 256, cap = max(1, COLSUM_CHUNKS / segs);
  return (int)(chunks > cap ? cap : chunks < 1 ? 1 : chunks);
}

// Column sums of X [segs * seg_rows][cols] (leading dimension ldx) per
// segment, weighted as in colsum_kernel, into out [segs][nw][cols] (FP64).
template <class T>
static void colsum(const T* X, int64_t ldx, int cols, int segs, int64_t seg_rows, const float* wt, int64_t wmod,
                   int wstride, int nw, double* part, double* out, hipStream_t st) {
  const int chunks = row_chunks(seg_rows, segs);
  const int chunk_rows = (int)((seg_rows + chunks - 1) / chunks);
  constexpr int VEC = 16 / (int)sizeof(T);
  if (cols % VEC == 0 && ldx % VEC == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0)
    hipLaunchKernelGGL((colsum_kernel<T, VEC>), dim3(chunks, segs), dim3(256), 0, st, X, ldx, cols, seg_rows,
                       chunk_rows, wt, wmod, wstride, nw, part);
  else
    hipLaunchKernelGGL((colsum_kernel<T, 1>), dim3(chunks, segs), dim3(256), 0, st, X, ldx, cols, seg_rows,
                       chunk_rows, wt, wmod, wstride, nw, part);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((nw * cols + 63) / 64, segs), dim3(256), 0, st, part, segs, chunks,
                     nw, cols, out);
}

// First-layer gradients from the per-snapshot sums S[b][0][u] = sum_p dz1,
// S[b][1 + i][u] = sum_p dz1 x_p[i] (i < m):
//   dW1[u][i] = sum_b S[b][1+i][u]; dW1[u][m+k] = sum_b S[b][0][u] q[b][k];
//   db1[u] = sum_b S[b][0][u];  dq[b][k] = sum_u S[b][0][u] W1[u][m+k]
// One wave per output, its lanes over the sum (a thread per output, with
// the sum as a chain of dependent loads, took 22 us for 16 snapshots).
__global__ __launch_bounds__(256) void layer1_grad_kernel(const double* __restrict__ S, const float* __restrict__ q,
                                                          const float* __restrict__ W1, int B, int W, int m, int r,
                                                          float* __restrict__ dW1, float* __restrict__ db1,
                                                          float* __restrict__ dq) {
  const int nw = 1 + m, lane = threadIdx.x & 63;
  for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < W * (m + r) + W + B * r; i += gridDim.x * 4) {
    double s = 0.0;
    float* out;
    if (i < W * (m + r)) {
      const int u = i / (m + r), k = i % (m + r);
      for (int b = lane; b < B; b += 64)
        s += k < m ? S[((int64_t)b * nw + 1 + k) * W + u] : S[((int64_t)b * nw) * W + u] * (double)q[b * r + (k - m)];
      out = dW1 + i;
    } else if (i < W * (m + r) + W) {
      const int u = i - W * (m + r);
      for (int b = lane; b < B; b += 64) s += S[((int64_t)b * nw) * W + u];
      out = db1 + u;
    } else {
      const int j = i - W * (m + r) - W, b = j / r, k = j % r;
      for (int u = lane; u < W; u += 64) s += S[((int64_t)b * nw) * W + u] * (double)W1[u * (m + r) + m + k];
      out = dq + j;
    }
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) s += __shfl_xor(s, w);
    if (lane == 0) *out = (float)s;
  }
}
// A launch holds fewer than 2^32 threads: from some 4 million outputs (524,000
// snapshots of 8 latents) on, its waves take several.
static dim3 layer1_grid(int W, int m, int r, int B) {
  return dim3((unsigned)std::min<int64_t>(1 << 20, ((int64_t)W * (m + r) + W + (int64_t)B * r + 3) / 4));
}

__global__ void d2f_kernel(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = (float)a[i];
}

// Adam with bias correction (Kingma & Ba), FP32 state.
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// ---------------------------------------------------------------------------
// host-side plumbing
// ---------------------------------------------------------------------------
static unsigned grid_for(int64_t n, int threads = 256) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > 16384) b = 16384;
  return (unsigned)b;
}

// The square hidden-layer products in bfloat16 at widths whose weights fit
// a wave's registers go through rowgemm_kernel; returns false otherwise.
template <bool FWD>
static bool row_gemm(int W, const void* X, const void* Wt, const float* bias, const void* gate, void* C,
                     int64_t rows, hipStream_t st, crom_status* s, bool sine = false, void* G = nullptr) {
  RowGemmArgs g{static_cast<const __bf16*>(X), static_cast<const __bf16*>(Wt), bias,
                static_cast<const __bf16*>(gate), static_cast<__bf16*>(C), rows, static_cast<__bf16*>(G)};
  const int64_t tiles = (rows + 15) / 16;
  int64_t blocks = (tiles + 3) / 4;
  if (blocks > 1024) blocks = 1024;  // four workgroups of four waves per CU, looping over row tiles
  if (blocks < 1) blocks = 1;
  if (W == 128 && sine) hipLaunchKernelGGL((rowgemm_kernel<128, FWD, true>), dim3((unsigned)blocks), dim3(256), 0, st, g);
  else if (W == 32 && sine) hipLaunchKernelGGL((rowgemm_kernel<32, FWD, true>), dim3((unsigned)blocks), dim3(256), 0, st, g);
  else if (W == 128) hipLaunchKernelGGL((rowgemm_kernel<128, FWD>), dim3((unsigned)blocks), dim3(256), 0, st, g);
  else if (W == 32) hipLaunchKernelGGL((rowgemm_kernel<32, FWD>), dim3((unsigned)blocks), dim3(256), 0, st, g);
  else return false;
  *s = hip_check(hipGetLastError(), "row gemm launch");
  return true;
}

// dW = X^T Y over `rows` rows for the 128-wide hidden layers in bfloat16:
// wgrad_kernel partials (at most MAX_SPLITS workgroups), then their sum in
// workgroup order.  Returns false for other widths.
static bool wgrad(int W, const void* X, const void* Y, int64_t rows, float* part, float* dW, hipStream_t st,
                  crom_status* s) {
  if (W != 128) return false;
  constexpr int KS = 32;
  int64_t nblk = (rows + KS - 1) / KS;
  if (nblk > MAX_SPLITS) nblk = MAX_SPLITS;
  if (nblk < 1) nblk = 1;
  int64_t per = (rows + nblk - 1) / nblk;
  per = (per + KS - 1) / KS * KS;
  nblk = per > 0 ? (rows + per - 1) / per : 1;
  if (nblk < 1) nblk = 1;
  hipLaunchKernelGGL((wgrad_kernel<128>), dim3((unsigned)nblk), dim3(256), 0, st, static_cast<const __bf16*>(X),
                     static_cast<const __bf16*>(Y), rows, per, part);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((W * W + 63) / 64)), dim3(256), 0, st, part, (int)nblk,
                     W, W, dW, (int64_t)W, 0, (int)EPI_NONE, nullptr);
  *s = hip_check(hipGetLastError(), "weight gradient launch");
  return true;
}

template <class T, bool TA, bool TB, int EPI>
static crom_status gemm(GemmArgs g, hipStream_t st) {
  constexpr int BK = sizeof(T) == 2 ? 64 : 32;  // the kernel's K tile
  dim3 grid((g.N + 63) / 64, (g.M + 63) / 64, 1);
  if (g.part) {
    // split K so that there are a few hundred blocks
    const int64_t tiles = (int64_t)grid.x * grid.y;
    int splits = (int)((1024 + tiles - 1) / tiles);
    const int maxs = (g.K + BK - 1) / BK;
    if (splits > maxs) splits = maxs;
    if (splits > MAX_SPLITS) splits = MAX_SPLITS;
    if (splits < 1) splits = 1;
    int kc = (g.K + splits - 1) / splits;
    kc = (kc + BK - 1) / BK * BK;
    splits = (g.K + kc - 1) / kc;
    g.kchunk = kc;
    grid.z = splits;
    if (EPI == EPI_DELU) return fail(CROM_ERR_INVALID_ARG, "split-K carries no gate");
    hipLaunchKernelGGL((gemm_kernel<T, TA, TB, EPI_NONE>), grid, dim3(256), 0, st, g);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(((int64_t)g.M * g.N + 63) / 64)), dim3(256), 0, st,
                       g.part, splits, g.M, g.N, g.C, g.ldc, g.accumulate, EPI, g.bias);
  } else {
    g.kchunk = g.K;
    hipLaunchKernelGGL((gemm_kernel<T, TA, TB, EPI>), grid, dim3(256), 0, st, g);
  }
  return hip_check(hipGetLastError(), "gemm launch");
}

static GemmArgs gemm_args(int M, int N, int K, const void* A, int64_t lda, const void* B, int64_t ldb) {
  GemmArgs g{};
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = A;
  g.lda = lda;
  g.B = B;
  g.ldb = ldb;
  return g;
}

// Workspace carving (256-byte aligned pieces).
struct Carve {
  char* base;
  size_t off;
  template <class U>
  U* take(size_t count) {
    U* p = reinterpret_cast<U*>(base ? base + off : nullptr);
    off = (off + count * sizeof(U) + 255) & ~size_t(255);
    return p;
  }
};

constexpr int MSE_BLOCKS = 1024;

// The shapes the fused pass is compiled for: its LDS holds one activation
// tile per product and the registers its weight gradients, four at most.
// Forward and backward of 3 latents at 4,999 points took 382 us layer by layer
// and take 147 (with the forward's latents in one launch), the gradients of 16
// snapshots of 16,384 points 0.92 ms and 0.25.  A block of rows never crosses a
// snapshot, so thousands of snapshots of fewer than some 30 points, which no
// field has, are the exception: backward of 10,000 snapshots of 20 points in
// bfloat16 0.97 ms layer by layer and 1.22 here, of 40 points 1.54 and 1.16; FP32
// 1.80 and 2.55, 3.29 and 2.54; at 1,000 snapshots of 20 points 0.31 and 0.15.
static bool fused_shape(const crom_net* n) {
  return n->width == TF_W && n->m == 2 && n->d == 1 && n->act == CROM_ACT_ELU && n->depth >= 3 && n->depth <= 5;
}

// Rows of a snapshot that one workgroup of the fused pass sums at a time.
// Training: colsum's chunks (whose FP32 sums the encoder's gradient repeats
// bit for bit in bfloat16; in FP32 nothing hangs on it, and single blocks
// share out evenly).  A vector-Jacobian product has no such follower: while there
// are compute units for it, one block of rows per workgroup (120 instead of
// 60 workgroups for 3 latents at 4,999 points: 54 -> 35 us, and 7 -> 14 us to
// add their gradients).
template <class T>
static int64_t fused_chunk_rows(int64_t P, int B, bool vjp) {
  constexpr int ROWS = FusedTile<T>::ROWS;
  const int64_t blocks = (P + ROWS - 1) / ROWS * B;
  if (sizeof(T) == 2 ? vjp && blocks <= TF_MAX_WG : blocks <= 8 * TF_MAX_WG) return ROWS;
  return (P + row_chunks(P, B) - 1) / row_chunks(P, B);
}

// The most chunks fused_chunk_rows leaves for any smaller B and P too: what
// the workspace is sized for, so that it holds a smaller last batch.
template <class T>
static int64_t fused_max_items(int64_t P, int B, bool vjp) {
  constexpr int ROWS = FusedTile<T>::ROWS;
  const int64_t blocks = (P + ROWS - 1) / ROWS * B;
  const int64_t chunks = std::min<int64_t>((P + 255) / 256 * B, std::max(COLSUM_CHUNKS, B));
  const int64_t single = sizeof(T) == 4 ? 8 * TF_MAX_WG : vjp ? TF_MAX_WG : 0;  // blocks that are a chunk each
  return std::min(blocks, std::max(chunks, single));
}

// The decoder's forward and backward over B snapshots x P points.  q: [B][r]
// FP32 latents.  dg_in: when not NULL the caller's dL/dg [B*P][D] (no loss);
// otherwise u [B][P] gives the MSE loss and dL/dg.  Writes grad_dec (natural
// parameter layout) and dq [B][r].
template <class T>
struct DecoderPass {
  T *a[16], *dz0, *dz1, *wt[16];
  T* gt[16];  // sine networks: cos(z_l) of each hidden layer
  float *c, *g, *dg, *part;
  double *cpart, *csum, *mpart;
  void* frags;  // the fused pass: packed weights, sums carried between blocks, first activations
  f32x4* carry;
  T* a0;
  static size_t vjp_bytes(const crom_net* n, int B, int64_t P) {
    Carve cv{nullptr, 0};
    DecoderPass d;
    d.carve(cv, n, B, P, true);
    return cv.off;
  }
  void carve(Carve& cv, const crom_net* n, int B, int64_t P, bool vjp) {
    const int64_t rows = (int64_t)B * P;
    const int W = n->width, depth = n->depth, D = n->d;
    if (fused_shape(n)) {
      const int64_t items = fused_max_items<T>(P, B, vjp), wgs = items < TF_MAX_WG ? items : TF_MAX_WG;
      frags = cv.take<f32x4>((size_t)(depth - 1) * 2 * FusedTile<T>::FRAGS);
      c = cv.take<float>((size_t)B * W);
      part = cv.take<float>((size_t)wgs * (depth - 1) * TF_MAT);
      carry = cv.take<f32x4>((size_t)wgs * 3 * TF_THREADS);
      a0 = cv.take<T>((size_t)wgs * FusedTile<T>::ROWS * FusedTile<T>::LD);
      cpart = cv.take<double>((size_t)items * 3 * W);
      mpart = cv.take<double>((size_t)wgs * tf_out(depth - 1));
      csum = cv.take<double>((size_t)B * 3 * W);
      return;
    }
    for (int l = 0; l < depth; ++l) a[l] = cv.take<T>((size_t)rows * W);
    for (int l = 0; l < depth; ++l) gt[l] = n->act == CROM_ACT_SINE ? cv.take<T>((size_t)rows * W) : nullptr;
    dz0 = cv.take<T>((size_t)rows * W);
    dz1 = cv.take<T>((size_t)rows * W);
    for (int l = 1; l < depth; ++l) wt[l] = cv.take<T>((size_t)W * W);
    c = cv.take<float>((size_t)B * W);
    g = cv.take<float>((size_t)rows * D);
    dg = cv.take<float>((size_t)rows * D);
    part = cv.take<float>((size_t)MAX_SPLITS * W * W);
    const int nw = 1 + n->m > D ? 1 + n->m : D;
    const int nmax = nw > 1 + D ? nw : 1 + D;
    cpart = cv.take<double>((size_t)(B > COLSUM_CHUNKS ? B : COLSUM_CHUNKS) * nmax * W);
    csum = cv.take<double>((size_t)B * nmax * W);
    mpart = cv.take<double>(MSE_BLOCKS);
  }
};

template <class T, int L>
static crom_status fused_fwd_bwd(const crom_net* n, const float* x, int B, int64_t P, const float* q, const float* u,
                                 const float* dg_in, float* grad, float* dq, float* loss, DecoderPass<T>& ws, hipStream_t st) {
  using F = FusedTile<T>;
  const int r = n->r;
  const ParamIndex pi = param_index(2, r, 1, TF_W, L + 1);
  hipLaunchKernelGGL(fused_prep_kernel<T>, dim3((L * 2 * F::FRAGS + 255) / 256), dim3(256), 0, st, n->params, pi, L, q,
                     B, r, static_cast<typename F::frag*>(ws.frags), ws.c);
  FusedArgs a{};
  a.params = n->params;
  a.pi = pi;
  a.frags = ws.frags;
  a.x = x;
  a.c = ws.c;
  a.u = dg_in ? nullptr : u;
  a.dg_in = dg_in;
  a.P = P;
  a.r = r;
  a.chunk_rows = fused_chunk_rows<T>(P, B, dg_in != nullptr);
  a.chunks = (int)((P + a.chunk_rows - 1) / a.chunk_rows);  // rounding up may leave the last ones without rows
  a.items = (int64_t)B * a.chunks;
  a.n = (float)((int64_t)B * P);
  a.part = ws.part;
  a.carry = ws.carry;
  a.a0 = ws.a0;
  a.spart = ws.cpart;
  a.opart = ws.mpart;
  const int wgs = (int)(a.items < TF_MAX_WG ? a.items : TF_MAX_WG);
  auto k = fused_train_kernel<T, L>;
  crom_status s = set_lds(k, (int)sizeof(FusedLds<T, L>));
  if (s != CROM_OK) return s;
  hipLaunchKernelGGL(k, dim3(wgs), dim3(TF_THREADS), sizeof(FusedLds<T, L>), st, a);
  FusedReduceArgs f{ws.part, ws.mpart, ws.cpart, wgs, L, a.chunks, pi, grad, dg_in ? nullptr : loss,
                    (double)((int64_t)B * P), ws.csum, B};
  hipLaunchKernelGGL(fused_reduce_kernel, dim3(L * TF_MAT / 64 + ((1 + L) * TF_W + 2 + 63) / 64 +
                                                (unsigned)std::min<int64_t>(1 << 20, (int64_t)B * (3 * TF_W / 64))),
                     dim3(TF_LANES * 64), 0, st, f);
  hipLaunchKernelGGL(layer1_grad_kernel, layer1_grid(TF_W, 2, r, B), dim3(256), 0, st, ws.csum, q,
                     n->params + pi.w[0], B, TF_W, 2, r, grad + pi.w[0], grad + pi.b[0], dq);
  return hip_check(hipGetLastError(), "fused training pass");
}

template <class T>
static crom_status decoder_fwd_bwd(const crom_net* n, const float* x, int B, int64_t P, const float* q,
                                   const float* u, const float* dg_in, float* grad, float* dq, float* loss,
                                   DecoderPass<T>& ws, hipStream_t st) {
  const int W = n->width, depth = n->depth, D = n->d, m = n->m, r = n->r;
  const int64_t rows = (int64_t)B * P;
  const ParamIndex pi = param_index(m, r, D, W, depth);
  const float* prm = n->params;
  const bool sine = n->act == CROM_ACT_SINE;  // bfloat16 row kernels only (checked at entry)
  crom_status s = CROM_OK;
  if (fused_shape(n)) {
    if (depth == 3) return fused_fwd_bwd<T, 2>(n, x, B, P, q, u, dg_in, grad, dq, loss, ws, st);
    if (depth == 4) return fused_fwd_bwd<T, 3>(n, x, B, P, q, u, dg_in, grad, dq, loss, ws, st);
    return fused_fwd_bwd<T, 4>(n, x, B, P, q, u, dg_in, grad, dq, loss, ws, st);
  }
  // weights in the GEMM precision
  for (int l = 1; l < depth; ++l)
    hipLaunchKernelGGL((convert_kernel<T>), dim3(grid_for((int64_t)W * W)), dim3(256), 0, st, prm + pi.w[l], ws.wt[l],
                       (int64_t)W * W);
  // ---- forward ----
  hipLaunchKernelGGL(fold_kernel, dim3(grid_for((int64_t)B * W)), dim3(256), 0, st, prm + pi.w[0], prm + pi.b[0], q,
                     B, W, m, r, ws.c);
  if (W > EW_MAX_W || W % 8 != 0 || m > EW_MAX_MD || D > EW_MAX_MD) return fail(CROM_ERR_UNSUPPORTED, "training shape");
  {
    const dim3 grid(grid_for(rows * W / 8));
    T* g1 = ws.gt[0];
    if (sine) {
      if (m == 1) hipLaunchKernelGGL((layer1_kernel<T, 1, true>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
      else if (m == 2) hipLaunchKernelGGL((layer1_kernel<T, 2, true>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
      else hipLaunchKernelGGL((layer1_kernel<T, 3, true>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
    } else {
      if (m == 1) hipLaunchKernelGGL((layer1_kernel<T, 1>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
      else if (m == 2) hipLaunchKernelGGL((layer1_kernel<T, 2>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
      else hipLaunchKernelGGL((layer1_kernel<T, 3>), grid, dim3(256), 0, st, prm + pi.w[0], ws.c, x, P, rows, W, r, ws.a[0], g1);
    }
  }
  for (int l = 1; l < depth; ++l) {
    if constexpr (sizeof(T) == 2) {
      if (row_gemm<true>(W, ws.a[l - 1], ws.wt[l], prm + pi.b[l], nullptr, ws.a[l], rows, st, &s, sine, ws.gt[l])) {
        if (s != CROM_OK) return s;
        continue;
      }
    }
    GemmArgs g = gemm_args((int)rows, W, W, ws.a[l - 1], W, ws.wt[l], W);
    g.bias = prm + pi.b[l];
    if constexpr (sizeof(T) == 2) {
      g.Cb = reinterpret_cast<__bf16*>(ws.a[l]);
      g.ldcb = W;
    } else {
      g.C = reinterpret_cast<float*>(ws.a[l]);
      g.ldc = W;
    }
    if ((s = gemm<T, false, true, EPI_BIAS_ELU>(g, st)) != CROM_OK) return s;
  }
  if (D == 1)
    hipLaunchKernelGGL((output_kernel<T, 1>), dim3(grid_for(rows)), dim3(256), 0, st, ws.a[depth - 1],
                       prm + pi.w[depth], prm + pi.b[depth], rows, W, ws.g);
  else
    hipLaunchKernelGGL((output_kernel<T, 3>), dim3(grid_for(rows)), dim3(256), 0, st, ws.a[depth - 1],
                       prm + pi.w[depth], prm + pi.b[depth], rows, W, ws.g);
  const float* dg = dg_in;
  if (!dg_in) {
    hipLaunchKernelGGL(mse_kernel, dim3(MSE_BLOCKS), dim3(256), 0, st, ws.g, u, rows * D, ws.dg, ws.mpart);
    hipLaunchKernelGGL(mse_final_kernel, dim3(1), dim3(256), 0, st, ws.mpart, MSE_BLOCKS, rows * D, loss);
    dg = ws.dg;
  }
  // ---- backward: output layer ----
  {
    // dWout[o][u] = sum_rows dg[row][o] a[row][u]; dbout[o] = sum dg[row][o]
    // (column sums of a weighted by dg, and of dg itself)
    colsum<T>(ws.a[depth - 1], W, W, 1, rows, dg, rows, D, 1 + D, ws.cpart, ws.csum, st);
    // csum[1 + o][u] = dWout[o][u]
    hipLaunchKernelGGL(d2f_kernel, dim3(grid_for((int64_t)D * W)), dim3(256), 0, st, ws.csum + W, grad + pi.w[depth],
                       (int64_t)D * W);
    colsum<float>(dg, D, D, 1, rows, nullptr, 1, 0, 1, ws.cpart, ws.csum, st);
    hipLaunchKernelGGL(d2f_kernel, dim3(1), dim3(64), 0, st, ws.csum, grad + pi.b[depth], (int64_t)D);
    if (sine && D == 1)
      hipLaunchKernelGGL((dz_last_kernel<T, 1, true>), dim3(grid_for(rows * W / 8)), dim3(256), 0, st, dg,
                         prm + pi.w[depth], ws.gt[depth - 1], rows, W, ws.dz0);
    else if (sine)
      hipLaunchKernelGGL((dz_last_kernel<T, 3, true>), dim3(grid_for(rows * W / 8)), dim3(256), 0, st, dg,
                         prm + pi.w[depth], ws.gt[depth - 1], rows, W, ws.dz0);
    else if (D == 1)
      hipLaunchKernelGGL((dz_last_kernel<T, 1>), dim3(grid_for(rows * W / 8)), dim3(256), 0, st, dg,
                         prm + pi.w[depth], ws.a[depth - 1], rows, W, ws.dz0);
    else
      hipLaunchKernelGGL((dz_last_kernel<T, 3>), dim3(grid_for(rows * W / 8)), dim3(256), 0, st, dg,
                         prm + pi.w[depth], ws.a[depth - 1], rows, W, ws.dz0);
  }
  // ---- hidden layers ----
  T* dz = ws.dz0;
  T* dzn = ws.dz1;
  for (int l = depth - 1; l >= 1; --l) {
    // dW_l = dz^T a_{l-1}  (split over rows)
    bool wg = false;
    if constexpr (sizeof(T) == 2) {
      wg = wgrad(W, dz, ws.a[l - 1], rows, ws.part, grad + pi.w[l], st, &s);
      if (s != CROM_OK) return s;
    }
    if (!wg) {
      GemmArgs gw = gemm_args(W, W, (int)rows, dz, W, ws.a[l - 1], W);
      gw.C = grad + pi.w[l];
      gw.ldc = W;
      gw.part = ws.part;
      if ((s = gemm<T, true, false, EPI_NONE>(gw, st)) != CROM_OK) return s;
    }
    // db_l = column sums of dz
    colsum<T>(dz, W, W, 1, rows, nullptr, 1, 0, 1, ws.cpart, ws.csum, st);
    hipLaunchKernelGGL(d2f_kernel, dim3(grid_for(W)), dim3(256), 0, st, ws.csum, grad + pi.b[l], (int64_t)W);
    // dz_{l-1} = (dz W_l) * ELU'(a_{l-1})
    bool done = false;
    if constexpr (sizeof(T) == 2) {
      done = row_gemm<false>(W, dz, ws.wt[l], nullptr, sine ? ws.gt[l - 1] : ws.a[l - 1], dzn, rows, st, &s, sine);
      if (s != CROM_OK) return s;
    }
    if (done) {
      T* t = dz;
      dz = dzn;
      dzn = t;
      continue;
    }
    GemmArgs gd = gemm_args((int)rows, W, W, dz, W, ws.wt[l], W);
    gd.gate = ws.a[l - 1];
    gd.ldg = W;
    if constexpr (sizeof(T) == 2) {
      gd.Cb = reinterpret_cast<__bf16*>(dzn);
      gd.ldcb = W;
    } else {
      gd.C = reinterpret_cast<float*>(dzn);
      gd.ldc = W;
    }
    if ((s = gemm<T, false, false, EPI_DELU>(gd, st)) != CROM_OK) return s;
    T* t = dz;
    dz = dzn;
    dzn = t;
  }
  // ---- first layer: per-snapshot sums of dz1 and of dz1 * x_i ----
  {
    const int nw = 1 + m;
    colsum<T>(dz, W, W, B, P, x, P, m, nw, ws.cpart, ws.csum, st);
    hipLaunchKernelGGL(layer1_grad_kernel, layer1_grid(W, m, r, B), dim3(256), 0, st,
                       ws.csum, q, prm + pi.w[0], B, W, m, r, grad + pi.w[0], grad + pi.b[0], dq);
  }
  return hip_check(hipGetLastError(), "decoder backward");
}

// Encoder: E1 [hidden][n_in], c1 [hidden], E2 [r][hidden], c2 [r] (FP32).
template <class T>
struct EncoderPass {
  T *ub, *dh;  // the snapshots (bfloat16 only) and the hidden layer's gradient as operands of dE1
  float *q, *dq, *h32, *kpart;
  void carve(Carve& cv, const crom_encoder* e, int B) {
    ub = sizeof(T) == 2 ? cv.take<T>((size_t)B * e->n_in) : nullptr;
    dh = cv.take<T>((size_t)B * e->hidden);
    q = cv.take<float>((size_t)B * e->r);
    dq = cv.take<float>((size_t)B * e->r);
    h32 = cv.take<float>((size_t)B * e->hidden);
    kpart = cv.take<float>((size_t)MAX_SPLITS * B * e->hidden);
  }
};

static ParamIndex enc_index(const crom_encoder* e) {
  ParamIndex pi{};
  pi.w[0] = 0;
  pi.b[0] = (int64_t)e->hidden * e->n_in;
  pi.w[1] = pi.b[0] + e->hidden;
  pi.b[1] = pi.w[1] + (int64_t)e->r * e->hidden;
  return pi;
}

// First layer of the dense encoder, split over K: part[z][b][n] = the products
// of u [B][K] and E1 [N][K] over K-range z (a multiple of the K tile), FP32.
// One wave per 16 snapshots x 16 units and range; the operands are read as
// FP32 and rounded here (converting E1 and u first, in launches of their own,
// read and wrote 29 MB more: 23 us for 16,384 -> 256 against 8).  Bfloat16:
// ub (NULL: none) also receives u in bfloat16.  Same operands, K order and
// ranges as gemm_kernel with split K.
template <class T>
__global__ __launch_bounds__(256) void enc_part_kernel(const float* __restrict__ u, const float* __restrict__ E1, int B,
                                                       int N, int64_t K, int64_t kchunk, int vec, T* __restrict__ ub,
                                                       float* __restrict__ part) {
  constexpr bool BF = sizeof(T) == 2;
  constexpr int STEP = BF ? 32 : 4, E = STEP / 4;  // K of one product; K per lane
  typedef T frag __attribute__((ext_vector_type(E)));
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int bt = (B + 15) / 16, b0 = (int)(blockIdx.x % bt) * 16, n0 = ((int)(blockIdx.x / bt) * 4 + (threadIdx.x >> 6)) * 16;
  if (n0 >= N) return;
  const int64_t k0 = blockIdx.y * kchunk, k1 = k0 + kchunk < K ? k0 + kchunk : K;
  auto load = [&](const float* row, bool ok, int64_t k) {
    frag f;
    if constexpr (BF) {
      if (vec && ok && k + 8 <= k1) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(row + k), y = *reinterpret_cast<const f32x4*>(row + k + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f[e] = (T)x[e];
          f[4 + e] = (T)y[e];
        }
        return f;
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) f[e] = ok && k + e < k1 ? (T)row[k + e] : (T)0.0f;
    return f;
  };
  const int b = b0 + lr, n = n0 + lr;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int64_t ks = k0; ks < k1; ks += STEP) {
    const int64_t k = ks + E * lg;
    const frag x = load(u + (int64_t)b * K, b < B, k), y = load(E1 + (int64_t)n * K, n < N, k);
    if constexpr (BF) {
      if (ub && n0 == 0 && b < B) {
        if (vec && K % 8 == 0 && k + 8 <= k1) {
          *reinterpret_cast<frag*>(&ub[(int64_t)b * K + k]) = x;
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
            if (k + e < k1) ub[(int64_t)b * K + k + e] = x[e];
        }
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc, 0, 0, 0);
    } else {
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], y[0], acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = b0 + 4 * lg + v;
    if (row < B && n < N) part[((int64_t)blockIdx.y * B + row) * N + n] = acc[v];
  }
}

// q [B][r] = h [B][K] E2^T + c2, FP32 products in K order, one wave per 16 x 16
// outputs; q2 (NULL: none): a second copy.
__global__ __launch_bounds__(64) void enc_latent_kernel(const float* __restrict__ h, const float* __restrict__ E2,
                                                        const float* __restrict__ c2, int B, int r, int K,
                                                        float* __restrict__ q, float* __restrict__ q2) {
  const int lr = threadIdx.x & 15, lg = threadIdx.x >> 4;
  const int b = blockIdx.x * 16 + lr, n = blockIdx.y * 16 + lr;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int U = 16;  // products whose operands are in flight together
  for (int k0 = 0; k0 < K; k0 += 4 * U) {
    float x[U], y[U];
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int k = k0 + 4 * s + lg;
      x[s] = b < B && k < K ? h[(int64_t)b * K + k] : 0.0f;
      y[s] = n < r && k < K ? E2[(int64_t)n * K + k] : 0.0f;
    }
#pragma unroll
    for (int s = 0; s < U; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s], y[s], acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = blockIdx.x * 16 + 4 * lg + v;
    if (row < B && n < r) {
      const float t = acc[v] + c2[n];
      q[row * r + n] = t;
      if (q2) q2[row * r + n] = t;
    }
  }
}

template <class T>
static crom_status encoder_fwd(const crom_encoder* e, const float* u, int B, EncoderPass<T>& ws, float* q_out,
                               hipStream_t st) {
  const ParamIndex pi = enc_index(e);
  const float* prm = e->params;
  // h = ELU(u E1^T + c1)  [B][hidden]: few rows, long K, so K is split
  constexpr int BK = sizeof(T) == 2 ? 64 : 32;
  const int64_t tiles = (int64_t)((e->hidden + 63) / 64) * ((B + 63) / 64);
  int64_t splits = std::min<int64_t>({(1024 + tiles - 1) / tiles, ((int64_t)e->n_in + BK - 1) / BK, MAX_SPLITS});
  if (splits < 1) splits = 1;
  const int64_t kc = (((int64_t)e->n_in + splits - 1) / splits + BK - 1) / BK * BK;
  splits = (e->n_in + kc - 1) / kc;
  const int vec = e->n_in % 4 == 0 && (reinterpret_cast<uintptr_t>(u) | reinterpret_cast<uintptr_t>(prm)) % 16 == 0;
  hipLaunchKernelGGL(enc_part_kernel<T>, dim3((unsigned)((int64_t)((B + 15) / 16) * ((e->hidden + 63) / 64)), (unsigned)splits),
                     dim3(256), 0, st, u, prm, B, e->hidden, (int64_t)e->n_in, kc, vec, ws.ub, ws.kpart);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(((int64_t)B * e->hidden + 63) / 64)), dim3(256), 0, st,
                     ws.kpart, (int)splits, B, e->hidden, ws.h32, (int64_t)e->hidden, 0, (int)EPI_BIAS_ELU,
                     prm + pi.b[0]);
  // q = h E2^T + c2 (FP32 product of the FP32 activations)
  hipLaunchKernelGGL(enc_latent_kernel, dim3((B + 15) / 16, (e->r + 15) / 16), dim3(64), 0, st, ws.h32, prm + pi.w[1],
                     prm + pi.b[1], B, e->r, e->hidden, ws.q, q_out);
  return hip_check(hipGetLastError(), "encoder forward");
}

// Backward of the dense encoder's small layers, one wave per 16 hidden units
// and chunk of snapshots (nine launches of the general products and sums took
// 60 us for 16 snapshots and 256 units):
//   dz1 [B][hidden] = (dq E2) * ELU'(h), in T (FP32 products in K order),
//   dc1 = sum_b dz1,  dE2 [r][hidden] = dq^T h,  dc2 = sum_b dq  (FP64 sums).
// A wave takes 4 us for every 16 snapshots, a chain of dependent loads: all
// 100,000 in one wave took 23 ms.  One chunk writes the gradients; of several, each
// leaves its sums in part [chunk][N (1 + r) + r] (dc1, dE2, dc2), which
// enc_bwd_final_kernel adds up.
template <class T>
__global__ __launch_bounds__(64) void enc_bwd_kernel(const float* __restrict__ dq, const float* __restrict__ E2,
                                                     const float* __restrict__ h, int B, int chunk, int r, int N,
                                                     T* __restrict__ dz1, float* __restrict__ dc1,
                                                     float* __restrict__ dE2, float* __restrict__ dc2,
                                                     double* __restrict__ part) {
  constexpr int RM = 16;  // largest latent size
  const int lr = threadIdx.x & 15, lg = threadIdx.x >> 4;
  const int n = blockIdx.x * 16 + lr;
  const int c0 = blockIdx.y * chunk, c1 = B - c0 < chunk ? B : c0 + chunk;
  double s1 = 0.0, s2[RM];
#pragma unroll
  for (int k = 0; k < RM; ++k) s2[k] = 0.0;
  for (int b0 = c0; b0 < c1; b0 += 16) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k0 = 0; k0 < RM; k0 += 4) {
      const int k = k0 + lg;
      const float x = b0 + lr < c1 && k < r ? dq[(b0 + lr) * r + k] : 0.0f;
      const float y = n < N && k < r ? E2[(int64_t)k * N + n] : 0.0f;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int b = b0 + 4 * lg + v;
      if (b >= c1 || n >= N) continue;
      const float hv = h[(int64_t)b * N + n], z = acc[v] * elu_d1_from_a(hv);
      dz1[(int64_t)b * N + n] = (T)z;
      s1 += (double)z;
#pragma unroll
      for (int k = 0; k < RM; ++k)
        if (k < r) s2[k] += (double)dq[b * r + k] * (double)hv;
    }
  }
  auto groups = [](double s) {
    s += __shfl_xor(s, 16);
    return s + __shfl_xor(s, 32);
  };
  double* p = gridDim.y > 1 ? part + blockIdx.y * ((int64_t)N * (1 + r) + r) : nullptr;
  s1 = groups(s1);
#pragma unroll
  for (int k = 0; k < RM; ++k) s2[k] = groups(s2[k]);
  if (lg == 0 && n < N) {
    if (p) p[n] = s1;
    else dc1[n] = (float)s1;
#pragma unroll
    for (int k = 0; k < RM; ++k) {
      if (k >= r) continue;
      if (p) p[(int64_t)N * (1 + k) + n] = s2[k];
      else dE2[(int64_t)k * N + n] = (float)s2[k];
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < r) {
    double s = 0.0;
    for (int b = c0; b < c1; ++b) s += (double)dq[b * r + threadIdx.x];
    if (p) p[(int64_t)N * (1 + r) + threadIdx.x] = s;
    else dc2[threadIdx.x] = (float)s;
  }
}

// One wave per gradient, its lanes over the chunks.
__global__ __launch_bounds__(256) void enc_bwd_final_kernel(const double* __restrict__ part, int chunks, int r, int N,
                                                            float* __restrict__ dc1, float* __restrict__ dE2,
                                                            float* __restrict__ dc2) {
  const int64_t n_out = (int64_t)N * (1 + r) + r, o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (o >= n_out) return;
  double s = 0.0;
  for (int c = lane; c < chunks; c += 64) s += part[c * n_out + o];
#pragma unroll
  for (int w = 1; w < 64; w <<= 1) s += __shfl_xor(s, w);
  if (lane != 0) return;
  if (o < N) dc1[o] = (float)s;
  else if (o < (int64_t)N * (1 + r)) dE2[o - N] = (float)s;
  else dc2[o - (int64_t)N * (1 + r)] = (float)s;
}

template <class T>
static crom_status encoder_bwd(const crom_encoder* e, const float* u, int B, const float* dq, float* grad,
                               EncoderPass<T>& ws, hipStream_t st) {
  const ParamIndex pi = enc_index(e);
  // chunks of 64 snapshots, of more where there would be over 1,024; their
  // sums take the place of the forward's partial products, MAX_SPLITS FP32
  // values for each of the B x hidden
  const int chunk = std::max(64, ((B - 1) / 1024 + 16) / 16 * 16), chunks = (B - 1) / chunk + 1;
  static_assert((1 + 2 * 16) * 8 <= MAX_SPLITS * 4 * 64, "a chunk's sums fit (r <= 16, one unit)");
  double* part = reinterpret_cast<double*>(ws.kpart);
  hipLaunchKernelGGL(enc_bwd_kernel<T>, dim3((e->hidden + 15) / 16, chunks), dim3(64), 0, st, dq, e->params + pi.w[1],
                     ws.h32, B, chunk, e->r, e->hidden, ws.dh, grad + pi.b[0], grad + pi.w[1], grad + pi.b[1], part);
  if (chunks > 1)
    hipLaunchKernelGGL(enc_bwd_final_kernel, dim3((unsigned)(((int64_t)e->hidden * (1 + e->r) + e->r + 3) / 4)), dim3(256),
                       0, st, part, chunks, e->r, e->hidden, grad + pi.b[0], grad + pi.w[1], grad + pi.b[1]);
  // dE1 = dz1^T u  [hidden][n_in]
  const void* ut = ws.ub ? static_cast<const void*>(ws.ub) : u;
  GemmArgs g = gemm_args(e->hidden, e->n_in, B, ws.dh, e->hidden, ut, e->n_in);
  g.C = grad + pi.w[0];
  g.ldc = e->n_in;
  return gemm<T, true, false, EPI_NONE>(g, st);
}

// ---------------------------------------------------------------------------
// Convolutional encoder (Sec. "Network Details"): the snapshot as a 1D vector
// of its P points with d channels; 1D convolutions (kernel 6, stride 4, d
// output channels, no padding, ELU) until the length is the smallest one not
// below 32 / d; flattened channel-major; a dense layer of `hidden` values
// (ELU) and a linear dense layer to r.  FP32 storage, FP32 products inside a
// convolution window or a dense row, FP64 sums over the batch and over
// positions for the weight gradients (fixed order: deterministic).
// Parameters, FP32, in order: per convolution W [d][d][6], b [d]; then
// E1 [hidden][L d], c1 [hidden], E2 [r][hidden], c2 [r].
// ---------------------------------------------------------------------------
constexpr int CONV_K = 6, CONV_S = 4, CONV_MAXL = 16;

struct ConvShape {
  int d, nl, hidden, r;
  int64_t len[CONV_MAXL + 1];  // len[0] = P
  int64_t w[CONV_MAXL], b[CONV_MAXL], e1, c1, e2, c2, count;
};

static ConvShape conv_shape(int64_t P, int d, int hidden, int r) {
  ConvShape c{};
  c.d = d;
  c.hidden = hidden;
  c.r = r;
  c.len[0] = P;
  int64_t L = P;
  while (L >= CONV_K && c.nl < CONV_MAXL) {
    const int64_t nxt = (L - CONV_K) / CONV_S + 1;
    if (nxt * d < 32) break;
    c.len[++c.nl] = nxt;
    L = nxt;
  }
  int64_t o = 0;
  for (int l = 0; l < c.nl; ++l) {
    c.w[l] = o;
    o += (int64_t)d * d * CONV_K;
    c.b[l] = o;
    o += d;
  }
  c.e1 = o;
  o += (int64_t)hidden * L * d;
  c.c1 = o;
  o += hidden;
  c.e2 = o;
  o += (int64_t)r * hidden;
  c.c2 = o;
  o += r;
  c.count = o;
  return c;
}

__device__ __forceinline__ float elu_f(float z) { return z > 0.0f ? z : expm1f(z); }
__device__ __forceinline__ float delu_from_act(float a) { return a > 0.0f ? 1.0f : a + 1.0f; }

// y[b][o][j] = ELU(bias[o] + sum_{c,k} W[o][c][k] x(b, c, 4 j + k)), with
// x(b, c, i) = x[b * xb + c * xc + i * xi].
__global__ __launch_bounds__(256) void conv_fwd_kernel(const float* __restrict__ x, int64_t xb, int64_t xc,
                                                      int64_t xi, const float* __restrict__ W,
                                                      const float* __restrict__ bias, int B, int d, int64_t Lo,
                                                      float* __restrict__ y) {
  const int64_t total = (int64_t)B * d * Lo;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e % Lo, bo = e / Lo;
    const int o = (int)(bo % d), b = (int)(bo / d);
    float s = bias[o];
    for (int c = 0; c < d; ++c) {
      const float* xp = x + b * xb + c * xc + (CONV_S * j) * xi;
      const float* wp = W + ((int64_t)o * d + c) * CONV_K;
#pragma unroll
      for (int k = 0; k < CONV_K; ++k) s += wp[k] * xp[k * xi];
    }
    y[e] = elu_f(s);
  }
}

// The two dense layers on top, a workgroup per snapshot: h = ELU(E1 x + c1)
// (n_mid values), q = E2 h + c2 (n_out), each output one thread's sum in input
// order; q2 (NULL: none): a second copy of q.
__global__ __launch_bounds__(256) void dense_fwd_kernel(const float* __restrict__ x, const float* __restrict__ E1,
                                                       const float* __restrict__ c1, const float* __restrict__ E2,
                                                       const float* __restrict__ c2, int B, int64_t n_in, int n_mid, int n_out,
                                                       float* __restrict__ h, float* __restrict__ q,
                                                       float* __restrict__ q2) {
  auto row = [](const float* W, float bias, const float* in, int64_t n) {
    float s = bias;
#pragma unroll 8
    for (int64_t i = 0; i < n; ++i) s += W[i] * in[i];
    return s;
  };
  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    for (int o = threadIdx.x; o < n_mid; o += blockDim.x)
      h[b * n_mid + o] = elu_f(row(E1 + o * n_in, c1[o], x + b * n_in, n_in));
    __syncthreads();
    for (int o = threadIdx.x; o < n_out; o += blockDim.x) {
      const float s = row(E2 + (int64_t)o * n_mid, c2[o], h + b * n_mid, n_mid);
      q[b * n_out + o] = s;
      if (q2) q2[b * n_out + o] = s;
    }
  }
}

// Backward of one dense layer, an output per thread:
//   dW[o][i] = sum_b dy[b][o] x[b][i], db[o] = sum_b dy[b][o] (FP64 sums over b in order),
//   dx[b][i] = (sum_o dy[b][o] W[o][i]) * ELU'(a[b][i])  (dx NULL: none)
__global__ __launch_bounds__(256) void dense_bwd_kernel(const float* __restrict__ dy, const float* __restrict__ x,
                                                       const float* __restrict__ W, const float* __restrict__ a, int B,
                                                       int64_t n_in, int n_out, float* __restrict__ dW,
                                                       float* __restrict__ db, float* __restrict__ dx) {
  const int64_t nw = (int64_t)n_out * n_in, total = nw + n_out + (dx ? (int64_t)B * n_in : 0);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    if (e < nw) {
      const int64_t o = e / n_in, i = e % n_in;
      double s = 0.0;
      for (int b = 0; b < B; ++b) s += (double)dy[(int64_t)b * n_out + o] * (double)x[(int64_t)b * n_in + i];
      dW[e] = (float)s;
    } else if (e < nw + n_out) {
      const int64_t o = e - nw;
      double s = 0.0;
      for (int b = 0; b < B; ++b) s += (double)dy[(int64_t)b * n_out + o];
      db[o] = (float)s;
    } else {
      const int64_t j = e - nw - n_out, i = j % n_in, b = j / n_in;
      float s = 0.0f;
#pragma unroll 8
      for (int o = 0; o < n_out; ++o) s += dy[b * n_out + o] * W[(int64_t)o * n_in + i];
      dx[j] = s * delu_from_act(a[j]);
    }
  }
}

// Backward of one convolution.  Blocks (e, chunk) of the first d*d*6 + d rows
// of the grid: e < d*d*6 takes W[o][c][k] = sum_{b,j} dz[b][o][j] x(b, c, 4 j +
// k), e = d*d*6 + o the bias sum_{b,j} dz[b][o][j], over the chunk's contiguous
// share of the (b, j) pairs (each thread a fixed stride in FP64, then a tree in
// LDS) into part[e][chunk]; conv_wgrad_final_kernel sums the chunks in order.
// The other blocks: the input gradient, gated by the ELU of the layer below
// (dzp NULL: none),
//   dzp[b][c][i] = ELU'(a[b][c][i]) sum_o sum_{k: i = 4 j + k, 0 <= j < Lo} dz[b][o][j] W[o][c][k].
constexpr int CONV_RED = 256, CONV_CHUNKS = 64;
__global__ __launch_bounds__(CONV_RED) void conv_bwd_kernel(const float* __restrict__ dz, const float* __restrict__ x,
                                                           int64_t xb, int64_t xc, int64_t xi,
                                                           const float* __restrict__ W, const float* __restrict__ a,
                                                           int B, int d, int64_t Li, int64_t Lo,
                                                           double* __restrict__ part, float* __restrict__ dzp) {
  __shared__ double red[CONV_RED];
  const int e = blockIdx.x / CONV_CHUNKS, chunk = blockIdx.x % CONV_CHUNKS;
  const int nw = d * d * CONV_K;
  if (e >= nw + d) {
    const int64_t total = (int64_t)B * d * Li;
    const int64_t first = blockIdx.x - (int64_t)(nw + d) * CONV_CHUNKS, blocks = gridDim.x - (int64_t)(nw + d) * CONV_CHUNKS;
    for (int64_t p = first * blockDim.x + threadIdx.x; p < total; p += blocks * blockDim.x) {
      const int64_t i = p % Li, bc = p / Li, b = bc / d;
      const int c = (int)(bc % d);
      float s = 0.0f;
      for (int k = (int)(i % CONV_S); k < CONV_K; k += CONV_S) {
        const int64_t j = (i - k) / CONV_S;
        if (i < k || j >= Lo) continue;
        for (int o = 0; o < d; ++o) s += dz[(b * d + o) * Lo + j] * W[((int64_t)o * d + c) * CONV_K + k];
      }
      dzp[p] = s * delu_from_act(a[p]);
    }
    return;
  }
  const int64_t n = (int64_t)B * Lo;
  const int64_t per = (n + CONV_CHUNKS - 1) / CONV_CHUNKS;
  const int64_t t0 = chunk * per, t1 = t0 + per < n ? t0 + per : n;
  double s = 0.0;
  if (e < nw) {
    const int o = e / (d * CONV_K), c = (e / CONV_K) % d, k = e % CONV_K;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += CONV_RED) {
      const int64_t b = t / Lo, j = t % Lo;
      s += (double)dz[(b * d + o) * Lo + j] * (double)x[b * xb + c * xc + (CONV_S * j + k) * xi];
    }
  } else {
    const int o = e - nw;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += CONV_RED) {
      const int64_t b = t / Lo, j = t % Lo;
      s += (double)dz[(b * d + o) * Lo + j];
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = CONV_RED / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(int64_t)e * CONV_CHUNKS + chunk] = red[0];
}

// The weight and bias gradients of every convolution (a block each: W then b,
// one after another in `grad`) from their partials.
__global__ __launch_bounds__(64) void conv_wgrad_final_kernel(const double* __restrict__ part, int n,
                                                             float* __restrict__ grad) {
  part += (int64_t)blockIdx.x * n * CONV_CHUNKS;
  grad += (int64_t)blockIdx.x * n;
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    double s = 0.0;
#pragma unroll 16
    for (int c = 0; c < CONV_CHUNKS; ++c) s += part[(int64_t)e * CONV_CHUNKS + c];
    grad[e] = (float)s;
  }
}

struct ConvPass {
  float* a[CONV_MAXL + 1];  // a[l] = ELU(conv_l) [B][d][len[l]], l >= 1
  float *h, *q, *dq, *dh, *dz[2];
  double* wpart;  // [convolutions][d*d*6 + d][CONV_CHUNKS] weight-gradient partials
  void carve(Carve& cv, const ConvShape& c, int B) {
    wpart = cv.take<double>((size_t)c.nl * (c.d * c.d * CONV_K + c.d) * CONV_CHUNKS);
    for (int l = 1; l <= c.nl; ++l) a[l] = cv.take<float>((size_t)B * c.d * c.len[l]);
    const int64_t top = c.nl ? c.len[1] : c.len[0];
    h = cv.take<float>((size_t)B * c.hidden);
    dh = cv.take<float>((size_t)B * c.hidden);
    q = cv.take<float>((size_t)B * c.r);
    dq = cv.take<float>((size_t)B * c.r);
    dz[0] = cv.take<float>((size_t)B * c.d * top);
    dz[1] = cv.take<float>((size_t)B * c.d * top);
  }
};

// Strides of the activation entering convolution l (l = 0: the snapshot
// [B][P][d], point-major; else [B][d][len]).
static void conv_in(const ConvShape& c, const float* u, const ConvPass& w, int l, const float** x, int64_t* xb,
                    int64_t* xc, int64_t* xi) {
  if (l == 0) {
    *x = u;
    *xb = c.len[0] * c.d;
    *xc = 1;
    *xi = c.d;
  } else {
    *x = w.a[l];
    *xb = c.d * c.len[l];
    *xc = c.len[l];
    *xi = 1;
  }
}

static crom_status conv_encoder_fwd(const ConvShape& c, const float* prm, const float* u, int B, ConvPass& w,
                                    float* q_out, hipStream_t st) {
  for (int l = 0; l < c.nl; ++l) {
    const float* x;
    int64_t xb, xc, xi;
    conv_in(c, u, w, l, &x, &xb, &xc, &xi);
    hipLaunchKernelGGL(conv_fwd_kernel, dim3(grid_for((int64_t)B * c.d * c.len[l + 1])), dim3(256), 0, st, x, xb,
                       xc, xi, prm + c.w[l], prm + c.b[l], B, c.d, c.len[l + 1], w.a[l + 1]);
  }
  // the flattened top: [B][d][L] is [B][L d] channel-major; with no
  // convolution the snapshot itself ([B][P d], point-major)
  const float* flat = c.nl ? w.a[c.nl] : u;
  hipLaunchKernelGGL(dense_fwd_kernel, dim3((unsigned)std::min(B, 1 << 20)), dim3(256), 0, st, flat, prm + c.e1,
                     prm + c.c1, prm + c.e2, prm + c.c2, B, c.len[c.nl] * c.d, c.hidden, c.r, w.h, w.q, q_out);
  return hip_check(hipGetLastError(), "convolutional encoder forward");
}

static crom_status conv_encoder_bwd(const ConvShape& c, const float* prm, const float* u, int B, const float* dq,
                                    float* grad, ConvPass& w, hipStream_t st) {
  const float* flat = c.nl ? w.a[c.nl] : u;
  const int64_t n_flat = c.len[c.nl] * c.d;
  // last layer: dE2, dc2; dh = (dq E2) ELU'(h)
  hipLaunchKernelGGL(dense_bwd_kernel, dim3(grid_for((int64_t)(c.r + B) * c.hidden + c.r)), dim3(256), 0, st, dq, w.h,
                     prm + c.e2, w.h, B, (int64_t)c.hidden, c.r, grad + c.e2, grad + c.c2, w.dh);
  // dense layer: dE1, dc1; the top convolution's output gradient
  hipLaunchKernelGGL(dense_bwd_kernel, dim3(grid_for((int64_t)(c.hidden + B) * n_flat + c.hidden)), dim3(256), 0, st,
                     w.dh, flat, prm + c.e1, c.nl ? w.a[c.nl] : nullptr, B, n_flat, c.hidden, grad + c.e1, grad + c.c1,
                     c.nl ? w.dz[0] : nullptr);
  if (c.nl == 0) return hip_check(hipGetLastError(), "convolutional encoder backward");
  const int nwb = c.d * c.d * CONV_K + c.d;  // a convolution's weights and biases, adjacent in the parameters
  int cur = 0;
  for (int l = c.nl - 1; l >= 0; --l) {  // convolution l: len[l] -> len[l + 1]
    const float* x;
    int64_t xb, xc, xi;
    conv_in(c, u, w, l, &x, &xb, &xc, &xi);
    const unsigned dx_blocks = l > 0 ? grid_for((int64_t)B * c.d * c.len[l]) : 0;
    hipLaunchKernelGGL(conv_bwd_kernel, dim3(nwb * CONV_CHUNKS + dx_blocks), dim3(CONV_RED), 0, st, w.dz[cur], x, xb, xc,
                       xi, prm + c.w[l], l > 0 ? w.a[l] : nullptr, B, c.d, c.len[l], c.len[l + 1],
                       w.wpart + (size_t)l * nwb * CONV_CHUNKS, w.dz[1 - cur]);
    cur = 1 - cur;
  }
  hipLaunchKernelGGL(conv_wgrad_final_kernel, dim3(c.nl), dim3(64), 0, st, w.wpart, nwb, grad);
  return hip_check(hipGetLastError(), "convolutional encoder backward");
}

static ConvShape conv_of(const crom_net* n, const crom_encoder* e) {
  return conv_shape(e->n_in / n->d, n->d, e->hidden, e->r);
}

static bool bf_mode(const crom_net* n) { return n->precision != CROM_PREC_FP32; }

template <class T>
static size_t train_bytes_t(const crom_net* n, const crom_encoder* e, int B) {
  Carve cv{nullptr, 0};
  DecoderPass<T> d;
  d.carve(cv, n, B, e->n_in / n->d, false);
  if (e->kind == CROM_ENC_CONV) {
    ConvPass cp;
    cp.carve(cv, conv_of(n, e), B);
  } else {
    EncoderPass<T> en;
    en.carve(cv, e, B);
  }
  return cv.off + 256;
}

static crom_status check_enc(const crom_net* n, const crom_encoder* e) {
  if (!e || !e->params) return fail(CROM_ERR_INVALID_ARG, "encoder and its params are required");
  if (e->n_in < 1 || e->hidden < 1 || e->r != n->r || e->n_in % n->d != 0)
    return fail(CROM_ERR_INVALID_ARG, "encoder shape: r must match the net and n_in = P * d");
  if (e->kind != CROM_ENC_DENSE && e->kind != CROM_ENC_CONV) return fail(CROM_ERR_INVALID_ARG, "encoder kind");
  if (e->kind == CROM_ENC_CONV && conv_of(n, e).nl < 1)
    return fail(CROM_ERR_INVALID_ARG, "the convolutional encoder needs room for one convolution (P d values)");
  return CROM_OK;
}

template <class T>
static crom_status train_grads_t(const crom_net* n, const crom_encoder* e, const float* u, const float* x, int B,
                                 float* grad_dec, float* grad_enc, float* loss, float* q_out, void* ws,
                                 hipStream_t st) {
  Carve cv{reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255)), 0};
  const int64_t P = e->n_in / n->d;
  DecoderPass<T> d;
  d.carve(cv, n, B, P, false);
  if (e->kind == CROM_ENC_CONV) {
    const ConvShape c = conv_of(n, e);
    ConvPass cp;
    cp.carve(cv, c, B);
    crom_status s = conv_encoder_fwd(c, e->params, u, B, cp, q_out, st);
    if (s != CROM_OK) return s;
    s = decoder_fwd_bwd<T>(n, x, B, P, cp.q, u, nullptr, grad_dec, cp.dq, loss, d, st);
    if (s != CROM_OK) return s;
    return conv_encoder_bwd(c, e->params, u, B, cp.dq, grad_enc, cp, st);
  }
  EncoderPass<T> en;
  en.carve(cv, e, B);
  crom_status s = encoder_fwd<T>(e, u, B, en, q_out, st);
  if (s != CROM_OK) return s;
  s = decoder_fwd_bwd<T>(n, x, B, P, en.q, u, nullptr, grad_dec, en.dq, loss, d, st);
  if (s != CROM_OK) return s;
  return encoder_bwd<T>(e, u, B, en.dq, grad_enc, en, st);
}

}  // namespace crom

using namespace crom;

extern "C" {

size_t crom_encoder_param_count(int32_t n_in, int32_t hidden, int32_t r) {
  if (n_in < 1 || hidden < 1 || r < 1) return 0;
  return (size_t)hidden * n_in + hidden + (size_t)r * hidden + r;
}

size_t crom_conv_encoder_param_count(int64_t P, int32_t d, int32_t hidden, int32_t r) {
  if (P < 1 || d < 1 || hidden < 1 || r < 1) return 0;
  const ConvShape c = conv_shape(P, d, hidden, r);
  return c.nl < 1 ? 0 : (size_t)c.count;
}

crom_status crom_train_workspace(const crom_net* net, const crom_encoder* enc, int32_t B, size_t* bytes) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if (net->act != CROM_ACT_ELU &&
      (net->act != CROM_ACT_SINE || net->precision == CROM_PREC_FP32 || (net->width != 32 && net->width != 128)))
    return fail(CROM_ERR_UNSUPPORTED, "training kernels: ELU networks, or sine networks of width 32 or 128 in bfloat16");
  if ((s = check_enc(net, enc)) != CROM_OK) return s;
  if (B < 1 || !bytes) return fail(CROM_ERR_INVALID_ARG, "B >= 1 and bytes are required");
  *bytes = bf_mode(net) ? train_bytes_t<__bf16>(net, enc, B) : train_bytes_t<float>(net, enc, B);
  return CROM_OK;
}

crom_status crom_train_grads(const crom_net* net, const crom_encoder* enc, const float* u, const float* x, int32_t B,
                             float* grad_dec, float* grad_enc, float* loss, float* q_out, void* ws, size_t ws_bytes,
                             void* stream) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if (net->act != CROM_ACT_ELU &&
      (net->act != CROM_ACT_SINE || net->precision == CROM_PREC_FP32 || (net->width != 32 && net->width != 128)))
    return fail(CROM_ERR_UNSUPPORTED, "training kernels: ELU networks, or sine networks of width 32 or 128 in bfloat16");
  if ((s = check_enc(net, enc)) != CROM_OK) return s;
  if (B < 1 || !u || !x || !grad_dec || !grad_enc || !loss || !ws)
    return fail(CROM_ERR_INVALID_ARG, "u, x, gradients, loss and ws are required");
  size_t need = 0;
  crom_train_workspace(net, enc, B, &need);
  if (ws_bytes < need) return fail(CROM_ERR_WORKSPACE, "workspace too small");
  hipStream_t st = static_cast<hipStream_t>(stream);
  return bf_mode(net) ? train_grads_t<__bf16>(net, enc, u, x, B, grad_dec, grad_enc, loss, q_out, ws, st)
                      : train_grads_t<float>(net, enc, u, x, B, grad_dec, grad_enc, loss, q_out, ws, st);
}

crom_status crom_adam_step(float* params, const float* grad, float* m, float* v, int64_t n, int64_t t, float lr,
                           float beta1, float beta2, float eps, void* stream) {
  if (n < 0 || t < 1) return fail(CROM_ERR_INVALID_ARG, "n >= 0 and t >= 1");
  if (n == 0) return CROM_OK;
  if (!params || !grad || !m || !v) return fail(CROM_ERR_INVALID_ARG, "params, grad, m and v are required");
  const float c1 = (float)(1.0 - pow((double)beta1, (double)t));
  const float c2 = (float)(1.0 - pow((double)beta2, (double)t));
  hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n)), dim3(256), 0, static_cast<hipStream_t>(stream), params, grad, m,
                     v, n, lr, beta1, beta2, eps, c1, c2);
  return hip_check(hipGetLastError(), "adam launch");
}

crom_status crom_train_step(const crom_net* net, void* packed, float* dec_grad, float* dec_m, float* dec_v,
                            const crom_encoder* enc, float* enc_grad, float* enc_m, float* enc_v, int64_t t,
                            const float* u, const float* x, int32_t B, float lr, float* loss, void* ws,
                            size_t ws_bytes, void* stream) {
  crom_status s = crom_train_grads(net, enc, u, x, B, dec_grad, enc_grad, loss, nullptr, ws, ws_bytes, stream);
  if (s != CROM_OK) return s;
  if (!dec_m || !dec_v || !enc_m || !enc_v) return fail(CROM_ERR_INVALID_ARG, "Adam moments are required");
  const int64_t nd = (int64_t)crom_net_param_count(net->m, net->r, net->d, net->width, net->depth);
  const int64_t ne = enc->kind == CROM_ENC_CONV ? conv_of(net, enc).count
                                                : (int64_t)crom_encoder_param_count(enc->n_in, enc->hidden, enc->r);
  s = crom_adam_step(const_cast<float*>(net->params), dec_grad, dec_m, dec_v, nd, t, lr, 0.9f, 0.999f, 1e-8f, stream);
  if (s != CROM_OK) return s;
  s = crom_adam_step(enc->params, enc_grad, enc_m, enc_v, ne, t, lr, 0.9f, 0.999f, 1e-8f, stream);
  if (s != CROM_OK) return s;
  if (packed) return crom_net_pack(net, packed, stream);
  return CROM_OK;
}

static int64_t enc_count(const crom_net* net, const crom_encoder* enc) {
  return enc->kind == CROM_ENC_CONV ? conv_of(net, enc).count
                                    : (int64_t)crom_encoder_param_count(enc->n_in, enc->hidden, enc->r);
}

crom_status crom_train_state_offsets(const crom_net* net, const crom_encoder* enc, crom_train_state_layout* out) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if ((s = check_enc(net, enc)) != CROM_OK) return s;
  if (!out) return fail(CROM_ERR_INVALID_ARG, "out is NULL");
  const size_t nd = 4 * crom_net_param_count(net->m, net->r, net->d, net->width, net->depth);
  const size_t ne = 4 * (size_t)enc_count(net, enc);
  size_t o = 0;
  auto take = [&o](size_t n) {
    const size_t at = o;
    o = (o + n + 255) & ~size_t(255);
    return at;
  };
  out->dec_params = take(nd);
  out->dec_grad = take(nd);
  out->dec_m = take(nd);
  out->dec_v = take(nd);
  out->enc_params = take(ne);
  out->enc_grad = take(ne);
  out->enc_m = take(ne);
  out->enc_v = take(ne);
  out->total = o;
  return CROM_OK;
}

size_t crom_train_state_bytes(const crom_net* net, const crom_encoder* enc) {
  crom_train_state_layout L;
  return crom_train_state_offsets(net, enc, &L) == CROM_OK ? L.total : 0;
}

crom_status crom_train_step_state(const crom_net* net, const crom_encoder* enc, void* state, void* packed, int64_t t,
                                  const float* u, const float* x, int32_t B, float lr, float* loss, void* ws,
                                  size_t ws_bytes, void* stream) {
  crom_train_state_layout L;
  crom_status s = crom_train_state_offsets(net, enc, &L);
  if (s != CROM_OK) return s;
  if (!state) return fail(CROM_ERR_INVALID_ARG, "state is NULL");
  if (reinterpret_cast<uintptr_t>(state) & 255) return fail(CROM_ERR_INVALID_ARG, "state must be 256-byte aligned");
  char* b = static_cast<char*>(state);
  crom_net n = *net;
  n.params = reinterpret_cast<const float*>(b + L.dec_params);
  crom_encoder e = *enc;
  e.params = reinterpret_cast<float*>(b + L.enc_params);
  return crom_train_step(&n, packed, reinterpret_cast<float*>(b + L.dec_grad), reinterpret_cast<float*>(b + L.dec_m),
                         reinterpret_cast<float*>(b + L.dec_v), &e, reinterpret_cast<float*>(b + L.enc_grad),
                         reinterpret_cast<float*>(b + L.enc_m), reinterpret_cast<float*>(b + L.enc_v), t, u, x, B, lr,
                         loss, ws, ws_bytes, stream);
}

crom_status crom_encode_workspace(const crom_net* net, const crom_encoder* enc, int32_t B, size_t* bytes) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if (net->act != CROM_ACT_ELU &&
      (net->act != CROM_ACT_SINE || net->precision == CROM_PREC_FP32 || (net->width != 32 && net->width != 128)))
    return fail(CROM_ERR_UNSUPPORTED, "training kernels: ELU networks, or sine networks of width 32 or 128 in bfloat16");
  if ((s = check_enc(net, enc)) != CROM_OK) return s;
  if (B < 1 || !bytes) return fail(CROM_ERR_INVALID_ARG, "B >= 1 and bytes are required");
  Carve cv{nullptr, 0};
  if (enc->kind == CROM_ENC_CONV) {
    ConvPass cp;
    cp.carve(cv, conv_of(net, enc), B);
  } else if (bf_mode(net)) {
    EncoderPass<__bf16> en;
    en.carve(cv, enc, B);
  } else {
    EncoderPass<float> en;
    en.carve(cv, enc, B);
  }
  *bytes = cv.off + 256;
  return CROM_OK;
}

crom_status crom_encode(const crom_net* net, const crom_encoder* enc, const float* u, int32_t B, float* q, void* ws,
                        size_t ws_bytes, void* stream) {
  size_t need = 0;
  crom_status s = crom_encode_workspace(net, enc, B, &need);
  if (s != CROM_OK) return s;
  if (!u || !q || !ws) return fail(CROM_ERR_INVALID_ARG, "u, q and ws are required");
  if (ws_bytes < need) return fail(CROM_ERR_WORKSPACE, "workspace too small");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Carve cv{reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255)), 0};
  if (enc->kind == CROM_ENC_CONV) {
    const ConvShape c = conv_of(net, enc);
    ConvPass cp;
    cp.carve(cv, c, B);
    return conv_encoder_fwd(c, enc->params, u, B, cp, q, st);
  }
  if (bf_mode(net)) {
    EncoderPass<__bf16> en;
    en.carve(cv, enc, B);
    return encoder_fwd<__bf16>(enc, u, B, en, q, st);
  }
  EncoderPass<float> en;
  en.carve(cv, enc, B);
  return encoder_fwd<float>(enc, u, B, en, q, st);
}

crom_status crom_decode_vjp_workspace(const crom_net* net, int32_t B, int64_t P, size_t* bytes) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if (net->act != CROM_ACT_ELU &&
      (net->act != CROM_ACT_SINE || net->precision == CROM_PREC_FP32 || (net->width != 32 && net->width != 128)))
    return fail(CROM_ERR_UNSUPPORTED, "training kernels: ELU networks, or sine networks of width 32 or 128 in bfloat16");
  if (B < 1 || P < 1 || !bytes) return fail(CROM_ERR_INVALID_ARG, "B >= 1, P >= 1 and bytes are required");
  *bytes = (bf_mode(net) ? DecoderPass<__bf16>::vjp_bytes(net, B, P) : DecoderPass<float>::vjp_bytes(net, B, P)) + 256;
  return CROM_OK;
}

crom_status crom_decode_vjp(const crom_net* net, const float* x, int64_t P, const float* q, int32_t B,
                            const float* dg, float* grad_params, float* grad_q, void* ws, size_t ws_bytes,
                            void* stream) {
  crom_status s = check_net(net, false);
  if (s != CROM_OK) return s;
  if (net->act != CROM_ACT_ELU &&
      (net->act != CROM_ACT_SINE || net->precision == CROM_PREC_FP32 || (net->width != 32 && net->width != 128)))
    return fail(CROM_ERR_UNSUPPORTED, "training kernels: ELU networks, or sine networks of width 32 or 128 in bfloat16");
  if (B < 1 || P < 1) return fail(CROM_ERR_INVALID_ARG, "B >= 1 and P >= 1");
  if (!x || !q || !dg || !grad_params || !grad_q || !ws)
    return fail(CROM_ERR_INVALID_ARG, "x, q, dg, grad_params, grad_q and ws are required");
  size_t need = 0;
  crom_decode_vjp_workspace(net, B, P, &need);
  if (ws_bytes < need) return fail(CROM_ERR_WORKSPACE, "workspace too small");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Carve cv{reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255)), 0};
  if (bf_mode(net)) {
    DecoderPass<__bf16> d;
    d.carve(cv, net, B, P, true);
    return decoder_fwd_bwd<__bf16>(net, x, B, P, q, nullptr, dg, grad_params, grad_q, nullptr, d, st);
  }
  DecoderPass<float> d;
  d.carve(cv, net, B, P, true);
  return decoder_fwd_bwd<float>(net, x, B, P, q, nullptr, dg, grad_params, grad_q, nullptr, d, st);
}

}  // extern "C"
