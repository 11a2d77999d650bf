// The decoder's training pass at width 128, forward and backward in one kernel
// (d = 1, m = 2, ELU, 3 to 5 hidden layers), in bfloat16 and in FP32.
//
// Layer by layer through memory (row_gemm, wgrad, column sums: every layer's
// activations written once and read two or three times) the pass was bound by
// HBM traffic and by some 40 launches: 0.82 ms in bfloat16 for 16 snapshots of
// 16,384 points, 0.56 ms in FP32 for 5 of 9,797.  Here a workgroup carries 128
// rows (FP32: 64) through all layers and back with the activations in LDS and
// every weight gradient in accumulators, so that memory sees the points, the
// snapshots and one partial gradient per workgroup: 0.206 ms and 0.26 ms.
// In bfloat16, of the 62 k cycles a block of rows takes, vector instructions
// (the ELU and its slope, the conversions) are issued in about 25 k, products
// in 13 k and LDS is busy in 24 k; the rest waits, at 16 barriers and for LDS.
// In FP32 the products bound it: 100 k of 150 k cycles.
//
// Split.  Eight waves, two per SIMD, so that one wave's products meet the
// other's epilogue.  In a layer's product a wave takes 32 output units of
// half the rows (units on the MFMA M dimension, rows on N), its weight
// fragments streaming through 32 registers from L2.  In a weight gradient
// (K = rows; bfloat16 fragments by LDS transpose reads) it takes a 64 x 32
// block of dW, 32 accumulators per layer; the bias gradient is a product with
// ones, 32 rows in FP32 and FP64 from there (the layerwise column sums: 16 or
// 32; kept in LDS it also frees registers: 258 -> 246 us for the gradients of
// 16 snapshots of 16,384 points, FP32 training step 301 -> 303).  LDS holds as
// many tiles of rows as there are products in one direction: the last layer's
// activations stay in registers, dz_l takes the place of a_l, and a_0, whose
// place dz_L takes (a fifth tile would not fit), waits in memory and comes back
// while the upper layers' gradients are formed.
//
// In bfloat16 the operands, the K order of every product, the epilogues, the
// output layer's sum (unit order) and the sums of dz_0 (16 row groups per
// chunk, in FP32, then FP64) are those of the layerwise kernels, which other
// shapes take: the latents' gradient, on which the encoder's bfloat16
// operands depend, comes out with the same bits on either path.
#pragma once

#include "common.hpp"
#include "gemm.hpp"

namespace crom {

constexpr int TF_W = 128;
constexpr int TF_THREADS = 512, TF_MAX_WG = 256;  // one workgroup per compute unit
constexpr int TF_MAT = TF_W * TF_W;               // a layer's partial dW
// a workgroup's FP64 partials: dWout (two halves of the rows), dbout, sum of squares, the layers' db
constexpr int tf_out(int L) { return (2 + L) * TF_W + 2; }

// Rows of a block (the LDS holds a tile of them per product), the LDS row
// (padded: 8 or 4 banks further on than the one before), K of one 16-byte
// fragment per lane and the K-blocks of a product.
template <class T>
struct FusedTile {
  static constexpr bool BF = sizeof(T) == 2;
  static constexpr int ROWS = BF ? 128 : 64, LD = TF_W + (BF ? 16 : 4), E = 16 / (int)sizeof(T), KQ = TF_W / (4 * E);
  static constexpr int FRAGS = (TF_W / 16) * KQ * 64;  // 16-byte fragments of one weight matrix
  static constexpr int NT = ROWS / 32;                 // N-tiles of a wave's product
  typedef T frag __attribute__((ext_vector_type(E)));
  typedef T vec8 __attribute__((ext_vector_type(8), aligned(16)));
  typedef T vec4 __attribute__((ext_vector_type(4), aligned(8)));
};

struct FusedArgs {
  const float* params;
  ParamIndex pi;
  const void* frags;    // [layer][forward, backward][mt][kb][lane], packed by fused_prep_kernel
  const float* x;       // [P][2]
  const float* c;       // [B][W] first-layer fold
  const float* u;       // [B][P] snapshots, or NULL:
  const float* dg_in;   // [B][P] the caller's cotangent
  int64_t P;
  int64_t chunk_rows;         // of a snapshot's rows, as colsum splits them
  int r, chunks;
  int64_t items;              // B * chunks
  float n;                    // B * P
  float* part;                // [workgroups][layers][TF_MAT]
  f32x4* carry;               // [workgroups][3][TF_THREADS]: a chunk's sums of dz_0 between its blocks
  void* a0;                   // [workgroups][ROWS][LD]: a_0 of the block, as it lies in LDS
  double* spart;              // [items][3][W]: sums of dz_0, dz_0 x_0, dz_0 x_1
  double* opart;              // [workgroups][tf_out(layers)]
};

// Weight fragments of every hidden-to-hidden layer (forward and transposed; the
// rows of a pair of M-tiles are dealt so that a lane ends with 8 consecutive
// units: one 16-byte LDS access) and the per-snapshot fold of the first layer
// c[b][u] = b1[u] + sum_k W1[u][2 + k] q[b][k] (FP64 accumulation).
template <class T>
__global__ __launch_bounds__(256) void fused_prep_kernel(const float* __restrict__ params, ParamIndex pi, int L,
                                                         const float* __restrict__ q, int B, int r,
                                                         typename FusedTile<T>::frag* __restrict__ frags,
                                                         float* __restrict__ c) {
  using F = FusedTile<T>;
  const int nf = L * 2 * F::FRAGS;
  for (int64_t j = blockIdx.x * blockDim.x + threadIdx.x; j < nf + (int64_t)B * TF_W; j += gridDim.x * blockDim.x) {
    if (j < nf) {
      const int f = (int)j, l = f & 63, kb = (f >> 6) % F::KQ, mt = (f >> 6) / F::KQ % (TF_W / 16), dir = f / F::FRAGS % 2;
      const float* Wl = params + pi.w[1 + f / (2 * F::FRAGS)];
      const int m = 32 * (mt >> 1) + 8 * (l >> 2 & 3) + 4 * (mt & 1) + (l & 3), k = F::E * (4 * kb + (l >> 4));
      typename F::frag v;
#pragma unroll
      for (int e = 0; e < F::E; ++e) v[e] = (T)(dir ? Wl[(k + e) * TF_W + m] : Wl[m * TF_W + k + e]);
      frags[f] = v;
    } else {
      const int64_t i = j - nf, b = i / TF_W;
      const int un = (int)(i % TF_W);
      const float* W1 = params + pi.w[0];
      double s = params[pi.b[0] + un];
      for (int k = 0; k < r; ++k) s += (double)W1[un * (2 + r) + 2 + k] * q[b * r + k];
      c[i] = (float)s;
    }
  }
}

// Sum over the 16 lanes of a DPP row, in every lane (rotations by 8, 4, 2, 1):
// the first STEPS rotations' sums in FP32, the others in FP64.
template <int CTRL>
__device__ __forceinline__ unsigned row_rot(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL, class V>
__device__ __forceinline__ V plus_rot(V v) {
  if constexpr (sizeof(V) == 4) {
    return v + __uint_as_float(row_rot<CTRL>(__float_as_uint(v)));
  } else {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = row_rot<CTRL>((unsigned)b), hi = row_rot<CTRL>((unsigned)(b >> 32));
    return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
  }
}
template <int STEPS>
__device__ __forceinline__ double row16_sum(float f) {
  static_assert(STEPS == 2 || STEPS == 4, "");
  f = plus_rot<0x124>(plus_rot<0x128>(f));
  if constexpr (STEPS == 4) return (double)plus_rot<0x121>(plus_rot<0x122>(f));
  else return plus_rot<0x121>(plus_rot<0x122>((double)f));
}

// *p += v in LDS, without waiting for the old value (one lane per address)
__device__ __forceinline__ void lds_add(double* p, double v) {
  __builtin_amdgcn_ds_atomic_fadd_f64((__attribute__((address_space(3))) double*)p, v);
}

template <class T, int L>
struct FusedLds {
  static constexpr int ROWS = FusedTile<T>::ROWS;
  T X[L][ROWS * FusedTile<T>::LD];
  float wx[2][TF_W], c[TF_W], bias[L][TF_W], wo[TF_W], xs[2][ROWS];
  float dg[ROWS];             // the block's snapshot values (or cotangents), then dL/dg
  double dwo[2][TF_W];        // dWout, two halves of the rows
  double db[L][TF_W];
  double loss[ROWS][2];       // per row of a block: sums of dL/dg and of the squared errors
};

template <class T, int L>
__global__ __launch_bounds__(TF_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void fused_train_kernel(
    FusedArgs a) {
  using F = FusedTile<T>;
  using frag = typename F::frag;
  using vec8 = typename F::vec8;
  constexpr int ROWS = F::ROWS, LD = F::LD, KQ = F::KQ, E = F::E, NT = F::NT, RING = 4;
  extern __shared__ __align__(16) char lds_raw[];
  FusedLds<T, L>& s = *reinterpret_cast<FusedLds<T, L>*>(lds_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
  const int wm = wave & 3, wn = wave >> 2;          // products: M-tiles 2 wm, 2 wm + 1; rows 16 NT wn ..
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

  if (tid < ROWS) s.loss[tid][0] = s.loss[tid][1] = 0.0;
  if (tid < 2 * TF_W) (&s.dwo[0][0])[tid] = 0.0;
  if (tid < L * TF_W) (&s.db[0][0])[tid] = 0.0;

  f32x4 dw[L][4][2];
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) dw[l][i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // Tile `slot` of the activations, its offset formed where it is used: the
  // compiler would otherwise keep every slot's per-lane addresses in
  // registers, and the accumulators leave none.
  auto tile = [&](int slot) {
    int o = slot * ROWS * LD;
    asm volatile("" : "+s"(o));
    return &s.X[0][0] + o;
  };
  // This wave's weight fragments: a ring of four K-blocks.  As soon as a
  // block has been used, its place takes the block four further on: of this
  // product (FP32 has eight) or of the next one, whose loads so have the rest
  // of this product, its epilogue and a barrier to arrive.
  frag A[2][RING];
  const int fo = 2 * wm * KQ * 64 + lane;
  auto frags = [&](int l, int dir) {
    int o = (l * 2 + dir) * F::FRAGS;
    asm volatile("" : "+s"(o));
    return reinterpret_cast<const frag*>(a.frags) + o + fo;
  };
  auto load_a = [&](const frag* f, int kb) {
#pragma unroll
    for (int i = 0; i < 2; ++i) A[i][kb % RING] = f[(i * KQ + kb) * 64];
  };
  // acc = W X over the wave's rows: the layer (l, dir), then (nl, ndir) comes
  auto product = [&](const T* X, f32x4 (&acc)[2][NT], int l, int dir, int nl, int ndir) {
    const T* p = X + (16 * NT * wn + lr) * LD + E * lg;
    const frag* f = KQ > RING ? frags(l, dir) : nullptr;
    const frag* fn = frags(nl, ndir);
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[0][n] = acc[1][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kb = 0; kb < KQ; ++kb) {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const frag b = *reinterpret_cast<const frag*>(&p[16 * n * LD + 4 * E * kb]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if constexpr (F::BF) {
            acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i][kb % RING], b, acc[i][n], 0, 0, 0);
          } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
              acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[i][kb % RING][e], b[e], acc[i][n], 0, 0, 0);
          }
        }
      }
      if (kb + RING < KQ) load_a(f, kb + RING);
      else load_a(fn, kb + RING - KQ);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // this lane's 8 consecutive units (4 i + v of its two M-tiles) in its row of N-tile n
  const int u8 = 32 * wm + 8 * lg;
  auto at = [&](int n) { return (16 * (NT * wn + n) + lr) * LD + u8; };
  // fragment of 16 columns from c0 for the K-block kk of rows.  bfloat16 (32
  // rows): lane (lg, lr) receives rows 8 lg .. 8 lg + 7 of column c0 + lr, by
  // transpose reads; FP32 (4 rows): row lg of column c0 + lr.
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  constexpr int KR = F::BF ? 32 : 4;
  auto columns = [&](const T* X, int kk, int c0) {
    if constexpr (F::BF) {
      const T* p = X + (KR * kk + 8 * lg + (lr >> 2)) * LD + c0 + 4 * (lr & 3);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * LD));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    } else {
      return X[(KR * kk + lg) * LD + c0 + lr];
    }
  };
  auto mfma = [](auto x, auto y, f32x4 c) {
    if constexpr (F::BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
  };
  auto ones = []() {
    if constexpr (F::BF) {
      const s16x8 v = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
      return __builtin_bit_cast(bf16x8, v);
    } else {
      return 1.0f;
    }
  };
  // dw += dz^T a over the block's rows, db += dz^T 1 (one of this wave's
  // M-tiles): products with ones over 32 rows, FP64 from there
  auto weight_grad = [&](const T* Z, const T* Y, f32x4 (&d)[4][2], double* db) {
    constexpr int GROUP = 32 / KR;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 b = zero;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int kk = 0; kk < ROWS / KR; ++kk) {
      decltype(ones()) y[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) y[j] = columns(Y, kk, nq + 16 * j);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto z = columns(Z, kk, mq + 16 * i);
#pragma unroll
        for (int j = 0; j < 2; ++j) d[i][j] = mfma(z, y[j], d[i][j]);
      }
      b = mfma(columns(Z, kk, mq + 16 * (wave & 3)), ones(), b);
      if (kk % GROUP == GROUP - 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] += (double)b[v];
        b = zero;
      }
    }
    if (lr == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) lds_add(&db[mq + 16 * (wave & 3) + 4 * lg + v], t[v]);
    }
  };
  // the thread's index, opaque: the addresses formed from it are computed in
  // the phase that uses them instead of being kept (spilled) across the loop
  auto self = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  auto elu = [](float z) { return z > 0.0f ? z : __expf(z) - 1.0f; };
  // a_0 of the block, 8 units of a row per step, and its copy in memory
  T* a0 = static_cast<T*>(a.a0) + (size_t)blockIdx.x * ROWS * LD;
  auto first_layer = [&]() {
    const int me = self();
#pragma unroll
    for (int t = 0; t < ROWS * TF_W / 8 / TF_THREADS; ++t) {
      const int row = t * (TF_THREADS / 16) + (me >> 4), u0 = (me & 15) * 8;
      const float x0 = s.xs[0][row], x1 = s.xs[1][row];
      vec8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float z = s.c[u0 + e];
        z += s.wx[0][u0 + e] * x0;
        z += s.wx[1][u0 + e] * x1;
        o[e] = (T)elu(z);
      }
      *reinterpret_cast<vec8*>(&s.X[0][row * LD + u0]) = o;
      *reinterpret_cast<vec8*>(&a0[row * LD + u0]) = o;
    }
  };
  // ... and back into tile 0, straight to LDS: a wave's load fills 1 KB in lane order
  auto reload_a0 = [&]() {
    constexpr int STEP = 64 * E, LOADS = ROWS * LD / STEP;
    static_assert(LOADS * STEP == ROWS * LD, "whole wave loads");
    const int w = __builtin_amdgcn_readfirstlane(wave), me = self() & 63;
    for (int i = w; i < LOADS; i += TF_THREADS / 64)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a0 + i * STEP + E * me),
                                       (__attribute__((address_space(3))) void*)(&s.X[0][i * STEP]), 16, 0, 0);
  };

  // the block's points and snapshot values (rows past the chunk repeat its
  // last one and carry dz = 0) and its snapshot's fold, loaded a block ahead
  int64_t item = blockIdx.x, b, p0, p1, r0;  // the grid has at most `items` workgroups
  float in0, in1 = 0.0f, in2 = 0.0f;
  auto chunk = [&]() {
    b = item / a.chunks;
    p0 = (item - b * a.chunks) * a.chunk_rows;
    p1 = p0 + a.chunk_rows < a.P ? p0 + a.chunk_rows : a.P;
    r0 = p0;
  };
  auto fetch = [&]() {
    const int me = self();
    if (me < ROWS) {
      const int64_t p = r0 + me < p1 ? r0 + me : p1 - 1;
      in0 = a.x[2 * p];
      in1 = a.x[2 * p + 1];
      in2 = (a.u ? a.u : a.dg_in)[b * a.P + p];
    } else if (me < ROWS + TF_W) {
      in0 = a.c[b * TF_W + me - ROWS];
    }
  };
  auto place = [&]() {
    const int me = self();
    if (me < ROWS) {
      s.xs[0][me] = in0;
      s.xs[1][me] = in1;
      s.dg[me] = in2;
    } else if (me < ROWS + TF_W) {
      s.c[me - ROWS] = in0;
    }
  };
  chunk();
  fetch();
  place();
#pragma unroll
  for (int kb = 0; kb < RING; ++kb) load_a(frags(0, 0), kb);
  __syncthreads();

  while (true) {
      const int valid = p1 - r0 < ROWS ? (int)(p1 - r0) : ROWS;
      first_layer();
      __syncthreads();

      // ---- forward
      vec8 top[NT];  // a_L at this lane's entries
#pragma unroll
      for (int l = 1; l <= L; ++l) {
        f32x4 acc[2][NT];
        product(tile(l - 1), acc, l - 1, 0, l < L ? l : L - 1, l < L ? 0 : 1);
        T* out = tile(l < L ? l : 0);
        const f32x4 bv[2] = {*reinterpret_cast<const f32x4*>(&s.bias[l - 1][u8]),
                             *reinterpret_cast<const f32x4*>(&s.bias[l - 1][u8 + 4])};
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          vec8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (T)elu(acc[e >> 2][n][e & 3] + bv[e >> 2][e & 3]);
          *reinterpret_cast<vec8*>(&out[at(n)]) = o;
          if (l == L) top[n] = o;
        }
        __syncthreads();
      }

      // ---- output layer and dL/dg, one thread per row, in unit order
      if (tid < ROWS) {
        const int row = self();
        float d = s.dg[row];
        double e2 = 0.0;
        if (a.u) {
          float g = 0.0f;
          const T* X = tile(0) + row * LD;
          // uniform addresses: scalar loads, operands of the products
          const __attribute__((address_space(4))) float* wo =
              (const __attribute__((address_space(4))) float*)(a.params + a.pi.w[L + 1]);
          constexpr int CH = F::BF ? 8 : 4;
#pragma unroll
          for (int h = 0; h < TF_W; h += 8 * CH) {
            vec8 v[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) v[i] = *reinterpret_cast<const vec8*>(&X[h + 8 * i]);
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
              for (int e = 0; e < 8; ++e) g += wo[h + 8 * i + e] * (float)v[i][e];
          }
          const float e = (g + bout) - d;
          d = 2.0f * e / a.n;
          e2 = (double)e * e;
        }
        if (row >= valid) d = 0.0f;
        s.dg[row] = d;
        s.loss[row][0] += (double)d;
        if (row < valid) s.loss[row][1] += e2;
      }
      __syncthreads();
      {
        T* Z = tile(0);
        const int me = self(), half = me >> 8, u0 = 32 * (me >> 6 & 3) + 8 * (me >> 4 & 3), row0 = 16 * NT * half + (me & 15);
        float dwo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) dwo[e] = 0.0f;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const int row = row0 + 16 * n;
          const float d = s.dg[row];
          vec8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float t = d * s.wo[u0 + e], av = (float)top[n][e];
            o[e] = (T)(t * elu_d1_from_a(av));
            dwo[e] += d * av;
          }
          uint32_t bits[2 * sizeof(T)];
          __builtin_memcpy(bits, &o, sizeof bits);
#pragma unroll
          for (int e = 0; e < 2 * (int)sizeof(T); ++e) bits[e] = row < valid ? bits[e] : 0u;
          __builtin_memcpy(&o, bits, sizeof bits);
          *reinterpret_cast<vec8*>(&Z[row * LD + u0]) = o;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double t = row16_sum<F::BF ? 2 : 4>(dwo[e]);  // 16 (FP32: 32) rows in FP32
          if ((me & 15) == 0) lds_add(&s.dwo[half][u0 + e], t);
        }
      }
      __syncthreads();

      // ---- backward: dz_l in X[0] (l = L) or X[l]; a_{l-1} in X[l - 1]
#pragma unroll
      for (int l = L; l >= 1; --l) {
        const T* Z = tile(l == L ? 0 : l);
        T* G = tile(l - 1);
        f32x4 acc[2][NT];
        // after the last product: the next block's first
        product(Z, acc, l - 1, 1, l > 1 ? l - 2 : 0, l > 1 ? 1 : 0);
        vec8 o[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const vec8 gv = *reinterpret_cast<const vec8*>(&G[at(n)]);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[n][e] = (T)(acc[e >> 2][n][e & 3] * elu_d1_from_a((float)gv[e]));
        }
        weight_grad(Z, G, dw[l - 1], s.db[l - 1]);
        __syncthreads();  // dz_l and a_{l-1} have been read
        if (l == L) reload_a0();  // where dz_L was
#pragma unroll
        for (int n = 0; n < NT; ++n) *reinterpret_cast<vec8*>(&G[at(n)]) = o[n];
        if (l == 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // a_0 has arrived
        __syncthreads();
      }

      // ---- sums of dz_0 and dz_0 x_k over the block, continuing the chunk's;
      // the next block's inputs meanwhile
      f32x4 sum[3];
      const int me = self(), cv = me & 31, rg = me >> 5;  // rows rg, rg + 16, ..., units 4 cv ..
      f32x4* carry = a.carry + (size_t)blockIdx.x * 3 * TF_THREADS + me;
#pragma unroll
      for (int k = 0; k < 3; ++k) sum[k] = r0 > p0 ? carry[k * TF_THREADS] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      const int64_t done = item;
      bool more = true;
      r0 += ROWS;
      const bool last = r0 >= p1;  // of its chunk
      if (last) {
        item += gridDim.x;
        more = item < a.items;
        if (more) chunk();
      }
      if (more) fetch();
      {
        const T* X = tile(0) + 4 * cv;
#pragma unroll
        for (int t = 0; t < ROWS / 16; ++t) {
          const int row = rg + 16 * t;
          const typename F::vec4 z = *reinterpret_cast<const typename F::vec4*>(&X[row * LD]);
          const float x0 = s.xs[0][row], x1 = s.xs[1][row];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = (float)z[e];
            sum[0][e] += v;
            sum[1][e] += v * x0;
            sum[2][e] += v * x1;
          }
        }
      }
      if (last) {  // the chunk's 16 row groups in order, through a tile that is free here
        float* sh = reinterpret_cast<float*>(tile(1));  // [3][16][W]
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<f32x4*>(&sh[(k * 16 + rg) * TF_W + 4 * cv]) = sum[k];
        __syncthreads();
        if (tid < 3 * TF_W) {
          const int k = me / TF_W, col = me % TF_W;
          double t = 0.0;
#pragma unroll
          for (int g = 0; g < 16; ++g) t += (double)sh[(k * 16 + g) * TF_W + col];
          a.spart[done * 3 * TF_W + me] = t;
        }
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) carry[k * TF_THREADS] = sum[k];
        __syncthreads();
      }
      if (!more) break;
      place();
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
  }
  double* op = a.opart + (size_t)blockIdx.x * tf_out(L);
  if (tid < 2 * TF_W) op[tid] = (&s.dwo[0][0])[tid];
  if (tid < L * TF_W) op[2 * TF_W + 2 + tid] = (&s.db[0][0])[tid];
  if (wave == 0) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      double t = s.loss[lane][k] + (ROWS > 64 ? s.loss[(lane + 64) % ROWS][k] : 0.0);
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) t += __shfl_xor(t, m);
      if (lane == 0) op[2 * TF_W + k] = t;
    }
  }
}

// Sums the workgroups' partials in order (16 interleaved lanes per output,
// then the lanes; four lanes kept too few loads in flight: 28 us for the 67 MB
// of 256 workgroups): blocks [0, nb_w) the layers' dW, then dWout, dbout, the
// loss and the layers' db, then S[seg][3][W] from the chunks.
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
constexpr int TF_LANES = 16;
__global__ __launch_bounds__(TF_LANES * 64) void fused_reduce_kernel(FusedReduceArgs a) {
  __shared__ double sh[TF_LANES][64];
  const int t = threadIdx.x & 63, lane = threadIdx.x >> 6;
  auto total = [&](auto* v) {  // the lanes' sums of output t, in order
    auto s = v[t];
#pragma unroll
    for (int l = 1; l < TF_LANES; ++l) s += v[64 * l + t];
    return s;
  };
  const int nb_w = a.L * TF_MAT / 64, n_o = (1 + a.L) * TF_W + 2, nb_o = (n_o + 63) / 64;
  const int blk = blockIdx.x;
  if (blk < nb_w) {  // FP32 partials, summed in FP32
    float* shf = reinterpret_cast<float*>(sh);
    const int e = blk * 64 + t, l = e / TF_MAT, i = e % TF_MAT;
    const size_t stride = (size_t)a.L * TF_MAT;
    float s = 0.0f;
#pragma unroll 8
    for (int z = lane; z < a.wgs; z += TF_LANES) s += a.part[z * stride + e];
    shf[lane * 64 + t] = s;
    __syncthreads();
    if (threadIdx.x < 64)
      a.grad[a.pi.w[1 + l] + i] = total(shf);
    return;
  }
  double s = 0.0;
  if (blk < nb_w + nb_o) {
    const int o = (blk - nb_w) * 64 + t;
    if (o < n_o) {
      for (int z = lane; z < a.wgs; z += TF_LANES) {
        const double* p = a.opart + (size_t)z * tf_out(a.L);
        s += o < TF_W ? p[o] + p[TF_W + o] : p[TF_W + o];
      }
    }
    sh[lane][t] = s;
    __syncthreads();
    if (threadIdx.x < 64 && o < n_o) {
      s = total(&sh[0][0]);
      if (o < TF_W) a.grad[a.pi.w[a.L + 1] + o] = (float)s;
      else if (o == TF_W) a.grad[a.pi.b[a.L + 1]] = (float)s;
      else if (o > TF_W + 1) a.grad[a.pi.b[1 + (o - TF_W - 2) / TF_W] + (o - TF_W - 2) % TF_W] = (float)s;
      else if (a.loss) *a.loss = (float)(s / a.n);
    }
    return;
  }
  const int64_t stride = (int64_t)(gridDim.x - nb_w - nb_o) * 64;
  for (int64_t i = (int64_t)(blk - nb_w - nb_o) * 64 + t; i - t < (int64_t)a.segs * 3 * TF_W; i += stride) {
    const int64_t seg = i / (3 * TF_W), o = i % (3 * TF_W);  // 3 W is a multiple of 64
    const double* p = a.spart + seg * a.chunks * 3 * TF_W + o;
    s = 0.0;
#pragma unroll 8
    for (int ch = lane; ch < a.chunks; ch += TF_LANES) s += p[(size_t)ch * 3 * TF_W];
    sh[lane][t] = s;
    __syncthreads();
    if (threadIdx.x < 64) a.S[i] = total(&sh[0][0]);
    __syncthreads();
  }
}

}  // namespace crom
