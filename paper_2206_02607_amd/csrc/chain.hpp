// Decoder values of 128-wide networks in the BF16 mode with the activations in
// registers: Engine's value pass (same operands, K order, epilogues and output
// sums, so the same bits) arranged for many points.
//
// What bounds it: a value column has five vector instructions of epilogue and
// three of hi/lo split for every three matrix instructions' share of it, so
// the vector ALU is busy about as long as the matrix cores, and Engine runs
// the two in turn: its layers' output units are split over the waves, so two
// workgroup barriers and an LDS round trip separate them.  Here a wave owns
// its points through all layers.  The K order of the packed weights is such
// that a lane's sums of two M-tiles are its B fragment of the next layer, so
// activations never leave the registers; the epilogue of one pair of M-tiles
// is in one instruction stream with the products of the next, across layers
// too; LDS carries only weights and parameters.  Eight waves (two per SIMD)
// share a layer's hi and lo fragments, 64 KB, and the next layer's arrive by
// direct loads in a second buffer meanwhile: one barrier per layer.
//
// 2D decoder, one latent: 2^20 points 364 us in Engine, 349 us here (1.18
// PFLOP/s of products, the rate of a large matrix product on this card),
// 65,536 points 29.6 and 26.2 us.  Without the interleaving (each epilogue
// after its own products) 400 us; a stated pattern of one product and four or
// five vector instructions, or a higher priority of one wave of a SIMD, changes
// nothing (348 to 354 us).
#pragma once

#include "common.hpp"
#include "engine.hpp"

namespace crom {

template <class S>
struct Chain {
  static constexpr int W = S::W, M = S::M, R = S::R, MTILES = W / 16, KB = W / 32;
  static_assert(W == 128 && S::D == 1, "a layer's weights twice in LDS; one output");
  static constexpr int NW = 8, THREADS = NW * 64, CUS = 256;
  // points of a workgroup per N-tile of its waves
  static constexpr int TILE = NW * PT;
  static constexpr int LAYER = (int)Packing<S, PREC_BF16>::LAYER_BYTES;  // hi, then lo fragments
  using PC = ParamCache<S>;
  static constexpr int FOLDS = 3;
  static constexpr int FOLD_OFF = 2 * LAYER, PAR_OFF = FOLD_OFF + FOLDS * W * 4;
  static __host__ __device__ constexpr int lds_bytes(int depth) { return PAR_OFF + PC::bytes(depth); }

  // Packed layer h into weight buffer `buf`, straight to LDS; arrived() waits
  // for this wave's share, a barrier for the others'.
  static __device__ __forceinline__ void fetch(char* lds, const char* __restrict__ packed, int h, int buf) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int PER = LAYER / 1024 / NW;
    const char* src = packed + (size_t)h * LAYER + w * PER * 1024;
    char* dst = lds + buf * LAYER + w * PER * 1024;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i * 1024 + lane * 16),
                                       (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, 0, 0);
  }
  static __device__ __forceinline__ void arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

  // First-layer fold of a latent into a slot (threads 0 .. W-1).
  static __device__ __forceinline__ void fold(char* lds, const float* par, const double* __restrict__ q, int slot) {
    const int u = threadIdx.x;
    if (u >= W) return;
    const float* W1 = par + PC::W1(0);
    double s = (double)(par + PC::B1())[u];
#pragma unroll
    for (int k = 0; k < R; ++k) s += (double)W1[u * (M + R) + M + k] * q[k];
    reinterpret_cast<float*>(lds + FOLD_OFF)[slot * W + u] = (float)s;
  }

  // A wave's NT 16-point tiles.
  template <int NT>
  struct Tile {
    using E = Engine<S, Cols<M, R, 1, 0, false, D2_NONE, 0>, NT, 4, PREC_BF16, 2>;  // the epilogue
    struct Acts {
      bf16x8 hi[NT][KB], lo[NT][KB];
    };
    struct Pair {  // two M-tiles of a layer's sums
      f32x4 z[2][NT];
    };

    static __device__ __forceinline__ void activate(Pair& p) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float z[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) z[t] = p.z[m][t][v];
          E::epilogue(z);
#pragma unroll
          for (int t = 0; t < NT; ++t) p.z[m][t][v] = z[t];
        }
    }
    // A pair's activations, split, into K-block kb.
    static __device__ __forceinline__ void pack(Acts& a, int kb, Pair p) {
      activate(p);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint32_t h[4], l[4];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            float r0, r1, d0, d1;
            h[2 * m + i] = bf16_pair(p.z[m][t][2 * i], p.z[m][t][2 * i + 1], r0, r1);
            l[2 * m + i] = bf16_pair(p.z[m][t][2 * i] - r0, p.z[m][t][2 * i + 1] - r1, d0, d1);
          }
        a.hi[t][kb] = __builtin_bit_cast(bf16x8, uint4{h[0], h[1], h[2], h[3]});
        a.lo[t][kb] = __builtin_bit_cast(bf16x8, uint4{l[0], l[1], l[2], l[3]});
      }
    }
    // A pair's share of the output layer.
    static __device__ __forceinline__ void dot(float (&part)[NT], const float* Wout, int mp, Pair p) {
      activate(p);
      const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
      for (int t = 0; t < NT; ++t) part[t] = 0.0f;
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float w = Wout[(2 * mp + m) * 16 + lg * 4 + v];
#pragma unroll
          for (int t = 0; t < NT; ++t) part[t] += w * p.z[m][t][v];
        }
    }
    static __device__ __forceinline__ void start(Pair& p, const float* bias, int mp) {
      const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const f32x4 bv = *reinterpret_cast<const f32x4*>(&bias[(2 * mp + m) * 16 + lg * 4]);
#pragma unroll
        for (int t = 0; t < NT; ++t) p.z[m][t] = bv;
      }
    }
    // Products of K-blocks K0 .. K1-1 for pair mp.
    template <int K0, int K1>
    static __device__ __forceinline__ void products(Pair& p, const Acts& in, const bf16x8* wf, int mp) {
#pragma unroll
      for (int kb = K0; kb < K1; ++kb) {
        bf16x8 ah[2], al[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          ah[m] = wf[((2 * mp + m) * KB + kb) * 64];
          al[m] = wf[(MTILES * KB + (2 * mp + m) * KB + kb) * 64];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            p.z[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[m], in.hi[t][kb], p.z[m][t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            p.z[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[m], in.lo[t][kb], p.z[m][t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            p.z[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[m], in.hi[t][kb], p.z[m][t], 0, 0, 0);
      }
    }
    // One layer.  The last pair of a layer's sums stays in c, to be finished
    // beside the next layer's first products.
    static __device__ __forceinline__ void layer(Acts& in, Acts& out, Pair& c, const bf16x8* wf, const float* bias) {
      Pair p[2];
      start(p[0], bias, 0);
      products<0, KB - 1>(p[0], in, wf, 0);
      pack(in, KB - 1, c);
      products<KB - 1, KB>(p[0], in, wf, 0);
#pragma unroll
      for (int mp = 1; mp < KB; ++mp) {
        start(p[mp & 1], bias, mp);
        products<0, KB>(p[mp & 1], in, wf, mp);
        pack(out, mp - 1, p[(mp - 1) & 1]);
      }
      c = p[(KB - 1) & 1];
    }
    static __device__ __forceinline__ void last_layer(Acts& in, float (&part)[KB][NT], const Pair& c,
                                                      const bf16x8* wf, const float* bias, const float* Wout) {
      Pair p[2];
      start(p[0], bias, 0);
      products<0, KB - 1>(p[0], in, wf, 0);
      pack(in, KB - 1, c);
      products<KB - 1, KB>(p[0], in, wf, 0);
#pragma unroll
      for (int mp = 1; mp < KB; ++mp) {
        start(p[mp & 1], bias, mp);
        products<0, KB>(p[mp & 1], in, wf, mp);
        dot(part[mp - 1], Wout, mp - 1, p[(mp - 1) & 1]);
      }
      dot(part[KB - 1], Wout, KB - 1, p[(KB - 1) & 1]);
    }

    // g[t]: the network's value at this wave's points 16 t + lane % 16 (x[t]).
    // On entry buffer `buf` receives layer 0 (fetch; not awaited) and the fold
    // slot is written (not awaited); `next` tells whether another pass
    // follows, whose layer 0 is fetched.  mid() runs once the pass is under
    // way: loads issued there are awaited with the next layer.  Returns the
    // buffer of the next pass.  depth >= 2.
    template <class Mid>
    static __device__ __forceinline__ int run(char* lds, const float* par, const char* __restrict__ packed, int depth,
                                              const float (&x)[2][M], int slot, int buf, bool next, float (&g)[NT],
                                              Mid&& mid) {
      const int lane = threadIdx.x & 63, lg = lane >> 4;
      const float* fold_v = reinterpret_cast<const float*>(lds + FOLD_OFF) + slot * W;
      const float* W1 = par + PC::W1(0);
      arrived();
      __syncthreads();
      mid();
      Acts a, b;
      Pair c;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int u = (2 * kb + m) * 16 + lg * 4 + v;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              float lin = 0.0f;
#pragma unroll
              for (int i = 0; i < M; ++i) lin += W1[u * (M + R) + i] * x[t][i];
              c.z[m][t][v] = lin + fold_v[u];
            }
          }
        if (kb < KB - 1) pack(a, kb, c);
      }
      auto begin = [&](int h) {  // layer h: its weights are here and the other buffer is read
        if (h > 0) {
          arrived();
          __syncthreads();
        }
        if (h + 1 < depth - 1) fetch(lds, packed, h + 1, buf ^ 1);
        else if (next) fetch(lds, packed, 0, buf ^ 1);
        const bf16x8* wf = reinterpret_cast<const bf16x8*>(lds + buf * LAYER) + lane;
        buf ^= 1;
        return wf;
      };
      int h = 0;
      for (; h + 2 < depth - 1; h += 2) {
        layer(a, b, c, begin(h), par + PC::BH(h));
        layer(b, a, c, begin(h + 1), par + PC::BH(h + 1));
      }
      if (h + 1 < depth - 1) {
        layer(a, b, c, begin(h), par + PC::BH(h));
        a = b;
        ++h;
      }
      float part[KB][NT];  // per pair of M-tiles, as four waves sum them
      last_layer(a, part, c, begin(h), par + PC::BH(h), par + PC::WOUT(depth));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float s = (par + PC::BOUT(depth))[0];
#pragma unroll
        for (int mp = 0; mp < KB; ++mp) {
          float p = part[mp][t];
          p += __shfl_xor(p, 16);
          p += __shfl_xor(p, 32);
          s += p;
        }
        g[t] = s;
      }
      return buf;
    }
  };
};

// Which workgroup takes which points.  An item is a group of 256 points of one
// of `sets` latent sets; the items go round the compute units, and a last
// round that is at most half full is cut into items of 128 points (one tile
// per wave), which take 0.6 of the time.
struct ChainPlan {
  int64_t groups;  // per set
  int64_t full;    // items of 256 points in whole rounds (and the tail, where it is not cut)
  int64_t halves;  // items of 128 points
  int blocks;
  __host__ static ChainPlan of(int64_t P, int64_t sets, int cus) {
    ChainPlan c;
    c.groups = (P + 255) / 256;
    const int64_t items = c.groups * sets, tail = items % cus;
    const bool cut = tail > 0 && 2 * tail <= cus;
    c.full = cut ? items - tail : items;
    c.halves = cut ? 2 * tail : 0;
    c.blocks = (int)(items >= cus ? cus : (cut ? c.halves : items));
    return c;
  }
};

// Whether Chain takes `sets` latent sets at P points, or Engine with 64 points
// per workgroup.  Where a compute unit has n of Engine's batches, Engine takes
// 13.8, 16.5, 21.4 and 29 us for n = 1 .. 4 (2D, one latent; up to three are
// resident together and hide each other's waits) and about 6.4 us for each
// more; Chain 27 us for the first 256 points, 22 us for each more and 12 for a
// cut last round.  So never below n = 4, and from there by the rounds: in
// Engine's batches a whole round of Chain costs 4 * 0.87 and a cut one 2.2 *
// 0.87 (65,536 points 29.6 and 26.2 us, 65,537 31.5 and 37.7, 131,072 52.6 and
// 48.1).  The sine's epilogue is longer: 0.97 (65,536 points 29.9 and 28.2 us,
// 82,000 39.1 and 40.1, 100,000 47.1 and 49.3, 131,072 53.7 and 50.1).  The
// packed weights go straight to LDS, 16 bytes per lane: at a lesser alignment
// Engine takes them, through registers.
template <class S>
static bool chain_takes(int depth, int64_t P, int64_t sets, const char* packed) {
  using C = Chain<S>;
  if (depth < 2 || C::lds_bytes(depth) > LDS_MAX || reinterpret_cast<uintptr_t>(packed) % 16 != 0) return false;
  const int64_t n = ((P + 63) / 64 * sets + C::CUS - 1) / C::CUS;
  const ChainPlan c = ChainPlan::of(P, sets, C::CUS);
  const int64_t rounds = c.full / C::CUS, rest = c.full % C::CUS;
  const int64_t tenths = 40 * rounds + (c.halves ? 22 : rest ? 40 : 0);
  return n >= 4 && tenths * (S::ACT == ACT_SINE ? 97 : 87) < n * 1000;
}

// Decoder values for latents q [sets][K][R] at points x [P]: per set and point
// sink.begin(), then for each of the K latents sink.load(set, k, p) while the
// pass runs and sink.take(value), then sink.store(set, p).  The lane that holds
// a point's value calls the sink; lanes without a point (p < 0) do not.
template <class S, class Sink>
__device__ __forceinline__ void chain_sweep(char* lds, const float* params, const ParamIndex& pi,
                                            const char* __restrict__ packed, int depth, const float* __restrict__ x,
                                            int64_t P, const double* __restrict__ q, int K, const ChainPlan& plan,
                                            Sink& sink) {
  using C = Chain<S>;
  float* par = reinterpret_cast<float*>(lds + C::PAR_OFF);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  struct Item {
    int64_t set, p0;  // p0: the workgroup's first point
    bool half, valid;
  };
  const int64_t bid = blockIdx.x, nblk = gridDim.x;
  const int64_t nf = bid < plan.full ? (plan.full - bid + nblk - 1) / nblk : 0;
  auto item = [&](int64_t n) {
    Item it;
    it.half = n >= nf;
    int64_t g = bid + n * nblk, off = 0;
    it.valid = n < nf || (n == nf && bid < plan.halves);
    if (it.half) {
      g = plan.full + (bid >> 1);
      off = (bid & 1) * C::TILE;
    }
    it.set = g / plan.groups;
    it.p0 = (g - it.set * plan.groups) * 256 + off;
    return it;
  };
  // x of this lane's columns of an item (points past the end: the last one)
  auto points = [&](const Item& it, float (&xv)[2][S::M]) {
    const int per = it.half ? PT : 2 * PT;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      int64_t p = it.p0 + wave * per + (it.half ? 0 : t * PT) + (lane & 15);
      if (p >= P) p = P - 1;
#pragma unroll
      for (int i = 0; i < S::M; ++i) xv[t][i] = x[p * S::M + i];
    }
  };
  Item it = item(0);
  if (!it.valid) return;
  C::fetch(lds, packed, 0, 0);
  C::PC::load(par, params, pi, depth, C::THREADS);
  __syncthreads();
  C::fold(lds, par, q + it.set * K * S::R, 0);
  float xv[2][S::M];
  points(it, xv);
  int buf = 0, slot = 0;
  for (int64_t n = 0; it.valid; ++n) {
    const Item nx = item(n + 1);
    float xn[2][S::M];
    const int per = it.half ? PT : 2 * PT;
    int64_t p = it.p0 + wave * per + lane;
    if (lane >= per || p >= P) p = -1;
    sink.begin();
    for (int k = 0; k < K; ++k) {
      const bool more = k + 1 < K, next = more || nx.valid;
      // The next pass's fold.  Its slot was last read two folds ago, before
      // the barrier that began the previous pass.
      const double* qn = q + (more ? it.set * K + k + 1 : nx.set * K) * S::R;
      const bool refold = next && qn != q + (it.set * K + k) * S::R;
      const int slot_n = refold ? (slot + 1) % C::FOLDS : slot;
      if (refold) C::fold(lds, par, qn, slot_n);
      auto mid = [&] {
        if (p >= 0) sink.load(it.set, k, p);
        if (!more && nx.valid) points(nx, xn);
      };
      float v;
      if (it.half) {
        float g[1];
        buf = C::template Tile<1>::run(lds, par, packed, depth, xv, slot, buf, next, g, mid);
        v = g[0];
      } else {
        float g[2];
        buf = C::template Tile<2>::run(lds, par, packed, depth, xv, slot, buf, next, g, mid);
        v = lane < PT ? g[0] : g[1];
      }
      if (p >= 0) sink.take(v);
      slot = slot_n;
    }
    if (p >= 0) sink.store(it.set, p);
    it = nx;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < S::M; ++i) xv[t][i] = xn[t][i];
  }
}

}  // namespace crom
