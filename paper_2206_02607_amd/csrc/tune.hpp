// Launch shapes of the value/derivative decode kernels (shared by the
// decode entry points and the fused decode-residual kernel of the sample
// selection).
#pragma once

#include "engine.hpp"

namespace crom {

// Launch shape of the decode kernels per decoder width and arithmetic:
// waves per workgroup, weight fragments (-1: by register estimate, 2:
// streamed one K-block ahead) and the waves per SIMD the register
// allocation must leave room for.  Measured on the 12-column 2D BF16 decode
// (1M points): 4 waves holding a layer's fragments 381 TFLOP/s (380
// registers, one workgroup per CU); 8 waves held to 128 registers 553;
// 4 waves (two M-tiles each, so every activation fragment read from LDS
// feeds two products) with streamed fragments held to 256 registers 633
// (two workgroups per CU); 2 waves 488.
// NBV: 16-point batches per workgroup of the value-only decode.  2D FP32,
// 65,536 points: 32 per workgroup 96.3 us, 64 86.2 us, 128 90.2 us.  2D BF16,
// 1,000, 16,384 and 49,152 points: 64 per workgroup 13.4, 13.8 and 21.4 us, 128
// 20.1, 20.1 and 25.0 us; more points than that are Chain's.
template <class S, int PREC>
struct DecodeTune {
  static constexpr int NW = S::W <= 32 ? 2 : (S::W <= 128 ? 4 : 8);
  static constexpr int PF = -1;
  static constexpr int WPE = 1;
  static constexpr int NBV = 4;
};
template <>
struct DecodeTune<Shape<128, 2, 8, 1>, PREC_BF16> {
  static constexpr int NW = 4, PF = 2, WPE = 2, NBV = 4;
};
template <>
struct DecodeTune<Shape<128, 2, 8, 1>, PREC_BF16_PURE> {
  static constexpr int NW = 4, PF = 2, WPE = 2, NBV = 4;
};
template <>
struct DecodeTune<Shape<128, 2, 8, 1, ACT_SINE>, PREC_BF16> {
  static constexpr int NW = 4, PF = 2, WPE = 2, NBV = 4;
};

// Values of 128-wide networks in BF16 mode (where Chain does not take them):
// the launch shape measured for the 2D decoder, with 16 latent values too
// (16,385 points 25.7 -> 15.5 us, 65,537 points 61.6 -> 32 us).
template <class S, int PREC>
struct ValueTune {
  using T = DecodeTune<S, PREC>;
  static constexpr bool W128 = S::W == 128 && S::D == 1 && PREC == PREC_BF16;
  static constexpr int PF = W128 ? 2 : T::PF, WPE = W128 ? 2 : T::WPE;
};

}  // namespace crom
