// Workgroup shape of the 16-bit decoder backward (oo_bwd16.hip).
#pragma once

#include "oo_mlp.h"

namespace oo {

constexpr int kPlane = 4 * kWave;  // elements of one plane of a fragment
constexpr int kFrag = 2 * kPlane;  // elements of a fragment

struct Bwd16Layout {
  int KB0;                   // input chunks
  size_t w, a0, x, y, total; // byte offsets: packed weights, inputs, deltas, activations
};

// waves: wave tiles of a workgroup, whose inputs stay for the whole tile;
// nput: wave tiles whose deltas and activations the exchange buffers hold
// at a time.
__host__ __device__ inline Bwd16Layout bwd16_layout(int K0, int H, int n_layers, int waves, int nput) {
  Bwd16Layout b;
  b.KB0 = (K0 + 31) / 32;
  size_t o = (size_t)bias_floats(n_layers, H) * sizeof(float);
  b.w = o;
  o += (size_t)packed_weight_elems<f16>(n_layers, K0, H) * 2;
  b.a0 = o;
  o += (size_t)waves * b.KB0 * kFrag * 2;
  b.x = o;
  o += (size_t)nput * (H / 32) * kFrag * 2;
  b.y = o;
  o += (size_t)nput * (H / 32) * kFrag * 2;
  b.total = o;
  return b;
}

// Workgroup shape: eight waves (128 queries); for the 128-wide decoders of
// three or four hidden layers four, whose dW blocks need the registers of
// one wave per SIMD. The exchange buffers hold every wave's operands where
// that fits beside the weights, else a share of the waves at a time. The
// widest inputs (over 96) of four 128-wide hidden layers fit in neither way:
// waves = 0, and the caller runs the kernel that reads its weights from L2.
struct Bwd16Shape {
  int waves, nput;
  size_t lds;
};
inline Bwd16Shape bwd16_shape(const MlpArgs& M) {
  Bwd16Shape s;
  s.waves = M.H == 128 && M.n_layers > 3 ? 4 : 8;
  for (s.nput = s.waves; s.nput >= 2; s.nput /= 2) {
    s.lds = bwd16_layout(M.K0, M.H, M.n_layers, s.waves, s.nput).total;
    if (s.lds <= (size_t)160 * 1024) return s;
  }
  s.waves = 0;
  return s;
}

}  // namespace oo
