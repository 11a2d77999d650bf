// The decoder's training pass at width 128 in bfloat16, forward and backward
// in one kernel (d = 1, m = 2, ELU, 3 to 5 hidden layers).
//
// Layer by layer through memory (row_gemm, wgrad, column sums: every layer's
// 67 MB of activations for 16 x 16,384 rows written once and read two or
// three times) the pass was bound by HBM traffic and by some 40 launches:
// 0.82 ms for 16 snapshots of 16,384 points.  Here a workgroup carries 128
// rows through all layers and back with the activations in LDS and every
// weight gradient in accumulators, so that memory sees the points, the
// snapshots and one partial gradient per workgroup: MEASURED.
// What bounds it now is vector work (the ELU and its slope, the bfloat16
// conversions: about 27 k of the 35 k cycles a block takes), then LDS.
//
// Split.  Eight waves, two per SIMD, so that one wave's products meet the
// other's epilogue.  In a layer's product a wave takes 32 output units of 64
// rows (units on the MFMA M dimension, rows on N): its weight fragments (32
// registers, L2) feed four products each.  In a weight gradient (K = rows,
// fragments by LDS transpose reads) it takes a 64 x 32 block of dW, 32
// accumulators per layer; the bias gradient is a product with ones.
// LDS holds as many 128-row tiles as there are products in one direction:
// the last layer's activations stay in registers, dz_l takes the place of
// a_l, and a_0 is computed again for the first weight gradient (a fifth tile
// would not fit).
//
// The operands, the K order of every product, the epilogues, the output
// layer's sum (unit order) and the sums of dz_0 (16 row groups per chunk, in
// FP32, then FP64) are those of the layerwise kernels, which other shapes
// take: the latents' gradient, on which the encoder's bfloat16 operands
// depend, comes out with the same bits on either path.
#pragma once

#include "common.hpp"
#include "gemm.hpp"

namespace crom {

constexpr int TF_W = 128, TF_ROWS = 128, TF_LD = TF_W + 8;  // LDS row: 4 banks further on than the one before
constexpr int TF_THREADS = 512, TF_MAX_WG = 256;            // one workgroup per compute unit
constexpr int TF_FRAGS = (TF_W / 16) * (TF_W / 32) * 64;    // 16-byte fragments of one weight matrix
constexpr int TF_MAT = TF_W * TF_W + TF_W;                  // a layer's partial gradient: dW, then db

struct FusedArgs {
  const float* params;
  ParamIndex pi;
  const bf16x8* frags;  // [layer][forward, backward][mt][kb][lane], packed by fused_prep_kernel
  const float* x;       // [P][2]
  const float* c;       // [B][W] first-layer fold
  const float* u;       // [B][P] snapshots, or NULL:
  const float* dg_in;   // [B][P] the caller's cotangent
  int64_t P;
  int r, chunks, chunk_rows;  // per snapshot, as colsum splits its rows
  int64_t items;              // B * chunks
  float n;                    // B * P
  float* part;                // [workgroups][layers][TF_MAT]
  double* spart;              // [items][3][W]: sums of dz_0, dz_0 x_0, dz_0 x_1
  double* opart;              // [workgroups][2 W + 2]: dWout (two halves of the rows), dbout, sum of squares
};

// Weight fragments of every hidden-to-hidden layer (bfloat16, forward and
// transposed) and the per-snapshot fold of the first layer
// c[b][u] = b1[u] + sum_k W1[u][2 + k] q[b][k] (FP64 accumulation).
__global__ __launch_bounds__(256) void fused_prep_kernel(const float* __restrict__ params, ParamIndex pi, int L,
                                                         const float* __restrict__ q, int B, int r,
                                                         bf16x8* __restrict__ frags, float* __restrict__ c) {
  constexpr int KB = TF_W / 32;
  const int nf = L * 2 * TF_FRAGS;
  for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < nf + B * TF_W; f += gridDim.x * blockDim.x) {
    if (f < nf) {
      const int l = f & 63, kb = (f >> 6) % KB, mt = (f >> 6) / KB % (TF_W / 16), dir = f / TF_FRAGS % 2;
      const float* Wl = params + pi.w[1 + f / (2 * TF_FRAGS)];
      const int m = 16 * mt + (l & 15), k = 32 * kb + 8 * (l >> 4);
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (__bf16)(dir ? Wl[(k + e) * TF_W + m] : Wl[m * TF_W + k + e]);
      frags[f] = v;
    } else {
      const int i = f - nf, b = i / TF_W, un = i % TF_W;
      const float* W1 = params + pi.w[0];
      double s = params[pi.b[0] + un];
      for (int k = 0; k < r; ++k) s += (double)W1[un * (2 + r) + 2 + k] * q[b * r + k];
      c[i] = (float)s;
    }
  }
}

template <int L>
struct FusedLds {
  __bf16 X[L][TF_ROWS * TF_LD];
  float wx[2][TF_W], c[TF_W], bias[L][TF_W], wo[TF_W], xs[2][TF_ROWS], dg[TF_ROWS];
  double red[2][2];
};

template <int L>
__global__ __launch_bounds__(TF_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void fused_train_kernel(
    FusedArgs a) {
  constexpr int KB = TF_W / 32;
  extern __shared__ __align__(16) char lds_raw[];
  FusedLds<L>& s = *reinterpret_cast<FusedLds<L>*>(lds_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
  const int wm = wave & 3, wn = wave >> 2;          // products: M-tiles 2 wm, 2 wm + 1; rows 64 wn ..
  const int mq = (wave >> 2) * 64, nq = (wave & 3) * 32;  // weight gradients: rows mq .., columns nq .. of dW
  for (int i = tid; i < TF_W; i += TF_THREADS) {
    const float* W1 = a.params + a.pi.w[0];
    s.wx[0][i] = W1[i * (2 + a.r)];
    s.wx[1][i] = W1[i * (2 + a.r) + 1];
#pragma unroll
    for (int l = 0; l < L; ++l) s.bias[l][i] = a.params[a.pi.b[1 + l] + i];
    s.wo[i] = a.params[a.pi.w[L + 1] + i];
  }
  const float bout = a.params[a.pi.b[L + 1]];

  f32x4 dw[L][4][2], db[L];
  float dwo[2][4];
  double sq = 0.0, sdg = 0.0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    db[l] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) dw[l][i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) dwo[i][v] = 0.0f;

  // Tile `slot` of the activations, its offset formed where it is used: the
  // compiler would otherwise keep every slot's per-lane addresses in
  // registers, and the accumulators leave none.
  auto tile = [&](int slot) {
    int o = slot * TF_ROWS * TF_LD;
    asm volatile("" : "+s"(o));
    return &s.X[0][0] + o;
  };
  bf16x8 A[2][KB];  // this wave's weight fragments of the coming product
  const int fo = 2 * wm * KB * 64 + lane;
  auto load_a = [&](int l, int dir) {
    int o = (l * 2 + dir) * TF_FRAGS;
    asm volatile("" : "+s"(o));
    const bf16x8* f = a.frags + o + fo;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) A[i][kb] = f[(i * KB + kb) * 64];
  };
  auto product = [&](const __bf16* X, f32x4 (&acc)[2][4]) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      acc[0][n] = acc[1][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(&X[(64 * wn + 16 * n + lr) * TF_LD + 32 * kb + 8 * lg]);
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i][kb], b, acc[i][n], 0, 0, 0);
      }
    }
  };
  // this lane's 4 consecutive units of M-tile 2 wm + i in its row of N-tile n
  auto at = [&](int i, int n) { return (64 * wn + 16 * n + lr) * TF_LD + 16 * (2 * wm + i) + 4 * lg; };
  // fragment of 16 columns from c0 of rows 32 kk ..: lane (lg, lr) receives rows 8 lg .. 8 lg + 7 of column c0 + lr
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  auto columns = [&](const __bf16* X, int kk, int c0) {
    const __bf16* p = X + (32 * kk + 8 * lg + (lr >> 2)) * TF_LD + c0 + 4 * (lr & 3);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * TF_LD));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  const s16x8 ones_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  // dw += dz^T a over the block's rows, db += dz^T 1 (one of this wave's M-tiles)
  auto weight_grad = [&](const __bf16* Z, const __bf16* Y, f32x4 (&d)[4][2], f32x4& b) {
#pragma unroll
    for (int kk = 0; kk < TF_ROWS / 32; ++kk) {
      bf16x8 y[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) y[j] = columns(Y, kk, nq + 16 * j);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16x8 z = columns(Z, kk, mq + 16 * i);
#pragma unroll
        for (int j = 0; j < 2; ++j) d[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(z, y[j], d[i][j], 0, 0, 0);
      }
      const bf16x8 zb = columns(Z, kk, mq + 16 * (wave & 3));
      b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zb, __builtin_bit_cast(bf16x8, ones_bits), b, 0, 0, 0);
    }
  };
  auto elu = [](float z) { return z > 0.0f ? z : __expf(z) - 1.0f; };
  // a_0 of the block, 8 units of a row per step
  auto first_layer = [&]() {
#pragma unroll
    for (int t = 0; t < TF_ROWS * TF_W / 8 / TF_THREADS; ++t) {
      const int row = t * (TF_THREADS / 16) + (tid >> 4), u0 = (tid & 15) * 8;
      const float x0 = s.xs[0][row], x1 = s.xs[1][row];
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float z = s.c[u0 + e];
        z += s.wx[0][u0 + e] * x0;
        z += s.wx[1][u0 + e] * x1;
        o[e] = (__bf16)elu(z);
      }
      *reinterpret_cast<bf16x8*>(&s.X[0][row * TF_LD + u0]) = o;
    }
  };

  for (int64_t item = blockIdx.x; item < a.items; item += gridDim.x) {
    const int64_t b = item / a.chunks, ch = item - b * a.chunks;
    const int64_t p0 = ch * a.chunk_rows;
    const int64_t p1 = p0 + a.chunk_rows < a.P ? p0 + a.chunk_rows : a.P;
    // a chunk past the last row (the rounded chunk size may leave one) sums nothing
    float sum[3][4];  // of dz_0 and dz_0 x_k over rows rg, rg + 16, ..., units 4 cv ..
    const int cv = tid & 31, rg = tid >> 5;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[k][e] = 0.0f;
    for (int64_t r0 = p0; r0 < p1; r0 += TF_ROWS) {
      const int valid = p1 - r0 < TF_ROWS ? (int)(p1 - r0) : TF_ROWS;
      // rows past the chunk repeat its last one and carry dz = 0
      if (tid < TF_ROWS) {
        const int64_t p = r0 + (tid < valid ? tid : valid - 1);
        s.xs[0][tid] = a.x[2 * p];
        s.xs[1][tid] = a.x[2 * p + 1];
      } else if (tid < TF_ROWS + TF_W) {
        s.c[tid - TF_ROWS] = a.c[b * TF_W + tid - TF_ROWS];
      }
      load_a(0, 0);
      __syncthreads();
      first_layer();
      __syncthreads();

      // ---- forward
      uint2 top[2][4];  // a_L at this lane's entries
#pragma unroll
      for (int l = 1; l <= L; ++l) {
        f32x4 acc[2][4];
        product(tile(l - 1), acc);
        load_a(l < L ? l : L - 1, l < L ? 0 : 1);
        __bf16* out = tile(l < L ? l : 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 bv = *reinterpret_cast<const f32x4*>(&s.bias[l - 1][16 * (2 * wm + i) + 4 * lg]);
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            bf16x4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = (__bf16)elu(acc[i][n][v] + bv[v]);
            *reinterpret_cast<bf16x4*>(&out[at(i, n)]) = o;
            if (l == L) top[i][n] = __builtin_bit_cast(uint2, o);
          }
        }
        __syncthreads();
      }

      // ---- output layer and dL/dg, one thread per row, in unit order
      if (tid < TF_ROWS) {
        float d = 0.0f;
        if (tid < valid) {
          const int64_t row = b * a.P + r0 + tid;
          if (a.u) {
            float g = 0.0f;
#pragma unroll 4
            for (int u0 = 0; u0 < TF_W; u0 += 8) {
              const bf16x8 v = *reinterpret_cast<const bf16x8*>(&s.X[0][tid * TF_LD + u0]);
#pragma unroll
              for (int e = 0; e < 8; ++e) g += s.wo[u0 + e] * (float)v[e];
            }
            const float e = (g + bout) - a.u[row];
            d = 2.0f * e / a.n;
            sq += (double)e * e;
          } else {
            d = a.dg_in[row];
          }
          sdg += (double)d;
        }
        s.dg[tid] = d;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4 wv = *reinterpret_cast<const f32x4*>(&s.wo[16 * (2 * wm + i) + 4 * lg]);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const int row = 64 * wn + 16 * n + lr;
          const float d = s.dg[row];
          const bf16x4 av = __builtin_bit_cast(bf16x4, top[i][n]);
          bf16x4 o;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float t = d * wv[v];
            o[v] = (__bf16)(row < valid ? t * elu_d1_from_a((float)av[v]) : 0.0f);
            dwo[i][v] += d * (float)av[v];
          }
          *reinterpret_cast<bf16x4*>(&s.X[0][at(i, n)]) = o;
        }
      }
      __syncthreads();

      // ---- backward: dz_l in X[0] (l = L) or X[l]; a_{l-1} in X[l - 1]
#pragma unroll
      for (int l = L; l >= 1; --l) {
        const __bf16* Z = tile(l == L ? 0 : l);
        __bf16* G = tile(l - 1);
        f32x4 acc[2][4];
        product(Z, acc);
        if (l > 1) load_a(l - 2, 1);
        uint2 o[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const bf16x4 gv = *reinterpret_cast<const bf16x4*>(&G[at(i, n)]);
            bf16x4 t;
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = (__bf16)(acc[i][n][v] * elu_d1_from_a((float)gv[v]));
            o[i][n] = __builtin_bit_cast(uint2, t);
          }
        weight_grad(Z, G, dw[l - 1], db[l - 1]);
        __syncthreads();  // dz_l and a_{l-1} have been read
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int n = 0; n < 4; ++n) *reinterpret_cast<uint2*>(&G[at(i, n)]) = o[i][n];
        if (l == 2) first_layer();  // a_0 again, where dz_L was
        __syncthreads();
      }

      // ---- sums of dz_0 over the block, continuing the chunk's
#pragma unroll
      for (int t = 0; t < TF_ROWS / 16; ++t) {
        const int row = rg + 16 * t;
        const bf16x4 z = *reinterpret_cast<const bf16x4*>(&s.X[0][row * TF_LD + 4 * cv]);
        const float x0 = s.xs[0][row], x1 = s.xs[1][row];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = (float)z[e];
          sum[0][e] += v;
          sum[1][e] += v * x0;
          sum[2][e] += v * x1;
        }
      }
      __syncthreads();  // before the next block's points
    }
    // the chunk's 16 row groups in order (X[1] is free until the next block's second layer)
    float* sh = reinterpret_cast<float*>(s.X[1]);  // [3][16][W]
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<f32x4*>(&sh[(k * 16 + rg) * TF_W + 4 * cv]) = f32x4{sum[k][0], sum[k][1], sum[k][2], sum[k][3]};
    __syncthreads();
    if (tid < 3 * TF_W) {
      const int k = tid / TF_W, col = tid % TF_W;
      double t = 0.0;
#pragma unroll
      for (int g = 0; g < 16; ++g) t += (double)sh[(k * 16 + g) * TF_W + col];
      a.spart[item * 3 * TF_W + tid] = t;
    }
    __syncthreads();
  }

  // ---- this workgroup's partial gradients
  float* part = a.part + (size_t)blockIdx.x * L * TF_MAT;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    float* d = part + l * TF_MAT;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) d[(mq + 16 * i + 4 * lg + v) * TF_W + nq + 16 * j + lr] = dw[l][i][j][v];
    if (lr == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) d[TF_W * TF_W + mq + 16 * (wave & 3) + 4 * lg + v] = db[l][v];
    }
  }
  double* op = a.opart + (size_t)blockIdx.x * (2 * TF_W + 2);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double t = (double)dwo[i][v];
#pragma unroll
      for (int m = 1; m < 16; m <<= 1) t += __shfl_xor(t, m);
      if (lr == 0) op[wn * TF_W + 16 * (2 * wm + i) + 4 * lg + v] = t;
    }
  if (wave < 2) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      sdg += __shfl_xor(sdg, m);
      sq += __shfl_xor(sq, m);
    }
    if (lane == 0) {
      s.red[wave][0] = sdg;
      s.red[wave][1] = sq;
    }
  }
  __syncthreads();
  if (tid < 2) op[2 * TF_W + tid] = s.red[0][tid] + s.red[1][tid];
}

// Sums the workgroups' partials in order (4 interleaved lanes per output,
// then the lanes): blocks [0, nb_w) the layers' dW and db, then dWout, dbout
// and the loss, then S[seg][3][W] from the chunks.
struct FusedReduceArgs {
  const float* part;
  const double *opart, *spart;
  int wgs, L, chunks;
  ParamIndex pi;
  float* grad;
  float* loss;  // NULL: none
  double n;
  double* S;
  int segs;
};
__global__ __launch_bounds__(256) void fused_reduce_kernel(FusedReduceArgs a) {
  __shared__ double sh[4][64];
  const int t = threadIdx.x & 63, l4 = threadIdx.x >> 6;
  const int nb_w = a.L * TF_MAT / 64, nb_o = (TF_W + 2 + 63) / 64;
  const int blk = blockIdx.x;
  if (blk < nb_w) {  // FP32 partials, summed in FP32
    float* shf = reinterpret_cast<float*>(sh);
    const int e = blk * 64 + t, l = e / TF_MAT, i = e % TF_MAT;
    const size_t stride = (size_t)a.L * TF_MAT;
    float s = 0.0f;
#pragma unroll 8
    for (int z = l4; z < a.wgs; z += 4) s += a.part[z * stride + e];
    shf[l4 * 64 + t] = s;
    __syncthreads();
    if (threadIdx.x < 64)
      a.grad[(i < TF_W * TF_W ? a.pi.w[1 + l] + i : a.pi.b[1 + l] + i - TF_W * TF_W)] =
          ((shf[t] + shf[64 + t]) + shf[128 + t]) + shf[192 + t];
    return;
  }
  double s = 0.0;
  if (blk < nb_w + nb_o) {
    const int o = (blk - nb_w) * 64 + t;
    if (o < TF_W + 2) {
      for (int z = l4; z < a.wgs; z += 4) {
        const double* p = a.opart + (size_t)z * (2 * TF_W + 2);
        s += o < TF_W ? p[o] + p[TF_W + o] : p[TF_W + o];
      }
    }
    sh[l4][t] = s;
    __syncthreads();
    if (threadIdx.x < 64 && o < TF_W + 2) {
      s = ((sh[0][t] + sh[1][t]) + sh[2][t]) + sh[3][t];
      if (o < TF_W) a.grad[a.pi.w[a.L + 1] + o] = (float)s;
      else if (o == TF_W) a.grad[a.pi.b[a.L + 1]] = (float)s;
      else if (a.loss) *a.loss = (float)(s / a.n);
    }
    return;
  }
  const int i = (blk - nb_w - nb_o) * 64 + t, seg = i / (3 * TF_W), o = i % (3 * TF_W);  // 3 W is a multiple of 64
  const double* p = a.spart + (size_t)seg * a.chunks * 3 * TF_W + o;
#pragma unroll 8
  for (int ch = l4; ch < a.chunks; ch += 4) s += p[(size_t)ch * 3 * TF_W];
  sh[l4][t] = s;
  __syncthreads();
  if (threadIdx.x < 64) a.S[i] = ((sh[0][t] + sh[1][t]) + sh[2][t]) + sh[3][t];
}

}  // namespace crom
