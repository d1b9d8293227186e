// The decoder's forward on matrix cores, shared by the fused query kernels,
// the standalone decoder and the disparity predictor: weights packed into
// LDS in fragment order, biases beside them, and the layer chain on NT
// tiles of 16 queries.
#pragma once

#include "oo_device.h"
#include "oo_internal.h"

namespace oo {

// ---------------------------------------------------------------------------
// Decoder forward on one wave's tiles of 16 queries.
// ---------------------------------------------------------------------------

// Weight fragments: packed in LDS in fragment order (zero padded), or read
// straight from the row-major matrices. Packed layout: layer 0 first
// ((H/16) x KB0 fragments), then each hidden layer ((H/16) x (H/32)), then
// the output layer (H/32); one fragment is 64 lanes x 8 elements.
template <class MT, bool WLDS>
struct WFrag {
  const MT* lds;
  int KB0;
  __device__ inline typename FragT<MT>::type get(const MlpArgs& M, int layer, int m, int kb, int lane) const {
    if constexpr (WLDS) {
      const int MH = M.H / 16, KH = M.H / 32;
      int base, KB;
      if (layer == 0) {
        base = 0;
        KB = KB0;
      } else {
        base = MH * KB0 + (layer - 1) * MH * KH;
        KB = KH;
      }
      return *reinterpret_cast<const typename FragT<MT>::type*>(lds + ((base + m * KB + kb) * kWave + lane) * 8);
    } else {
      const int n_in = layer == 0 ? M.K0 : M.H;
      const int n_out = layer == M.n_layers - 1 ? M.n_out : M.H;
      return wfrag_global<MT>(launder_ptr(reinterpret_cast<const MT*>(M.W[layer])), n_out, n_in, n_in, m, kb, lane);
    }
  }
};

// Layer biases kept in LDS next to the weights, H floats per hidden layer
// and 16 (zero padded) for the output layer: an output tile's bias is then
// one 16-byte LDS read per lane instead of predicated loads from L2.
__host__ __device__ inline int bias_floats(int n_layers, int H) { return (n_layers - 1) * H + 16; }

__device__ inline void load_biases_lds(const MlpArgs& M, float* bias) {
  for (int e = threadIdx.x; e < bias_floats(M.n_layers, M.H); e += blockDim.x) {
    const int layer = e / M.H, i = e % M.H;
    bias[e] = layer < M.n_layers - 1 || i < M.n_out ? M.b[layer][i] : 0.0f;
  }
}

__device__ inline f32x4 bias_tile(const float* bias, int m, int lane) {
  return *reinterpret_cast<const f32x4*>(bias + 16 * m + 4 * (lane >> 4));
}

// The layers after the first on NT N-tiles of 16 queries: acc holds the first
// layer's sums (before its ReLU), out gets the output tile per N-tile (rows
// 0..2 = RGB in lanes 0..15). The bias is the C operand of a layer's first
// MFMA, so no accumulator is copied or initialised.
template <class MT, int H, int NT, class WSrc>
__device__ inline void mlp_rest(const MlpArgs& M, const WSrc& W, const float* bias, int lane,
                                f32x4 (&acc)[H / 16][NT], f32x4 out[NT]) {
  typedef typename FragT<MT>::type frag;
  constexpr int MH = H / 16, KH = H / 32;
  // hidden layers H -> H
  for (int layer = 1; layer < M.n_layers - 1; ++layer) {
    const float* lb = bias + layer * H;
    frag bf[KH][NT];
#pragma unroll
    for (int kb = 0; kb < KH; ++kb)
#pragma unroll
      for (int t = 0; t < NT; ++t) bf[kb][t] = chain_frag<MT>(acc[2 * kb][t], acc[2 * kb + 1][t], true);
#pragma unroll
    for (int kb = 0; kb < KH; ++kb) {
      frag a[MH];
      f32x4 bt[MH];
#pragma unroll
      for (int m = 0; m < MH; ++m) {
        a[m] = W.get(M, layer, m, kb, lane);
        if (kb == 0) bt[m] = bias_tile(lb, m, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MH; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = mma(a[m], bf[kb][t], kb == 0 ? bt[m] : acc[m][t]);
    }
  }
  // output layer H -> 3
  const int lo = M.n_layers - 1;
  const f32x4 bt = bias_tile(bias + lo * H, 0, lane);
#pragma unroll
  for (int kb = 0; kb < KH; ++kb) {
    const frag a = W.get(M, lo, 0, kb, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      out[t] = mma(a, chain_frag<MT>(acc[2 * kb][t], acc[2 * kb + 1][t], true), kb == 0 ? bt : out[t]);
  }
}

// Runs the MLP on NT N-tiles of 16 queries and returns the output tile per
// N-tile. input(kb, t) is the B operand of the first layer: K-chunk kb < KB0
// of N-tile t.
// KB is KB0 where the caller knows it at compile time, else 0.
template <class MT, int H, int NT, int KB, class WSrc, class In>
__device__ inline void mlp_forward_tiles(const MlpArgs& M, const WSrc& W, const float* bias, int KB0, int lane,
                                         In&& input, f32x4 out[NT]) {
  // M is a kernel argument: indexing its arrays reads the argument segment.
  typedef typename FragT<MT>::type frag;
  constexpr int MH = H / 16;
  f32x4 acc[MH][NT];
  // layer 0: K0 -> H. Each K-chunk's weight fragments are all read before
  // its MFMAs, so their LDS latency overlaps instead of stalling every pair
  // of MFMAs.
  auto chunk = [&](int kb, bool first) {
    frag bf[NT], a[MH];
    f32x4 bt[MH];
#pragma unroll
    for (int t = 0; t < NT; ++t) bf[t] = input(kb, t);
#pragma unroll
    for (int m = 0; m < MH; ++m) {
      a[m] = W.get(M, 0, m, kb, lane);
      if (first) bt[m] = bias_tile(bias, m, lane);
    }
    __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink each read to its MFMAs)
#pragma unroll
    for (int m = 0; m < MH; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[m][t] = mma(a[m], bf[t], first ? bt[m] : acc[m][t]);
  };
  chunk(0, true);
  if constexpr (KB > 0) {
#pragma unroll
    for (int kb = 1; kb < KB; ++kb) chunk(kb, false);
  } else {
    for (int kb = 1; kb < KB0; ++kb) chunk(kb, false);
  }
  mlp_rest<MT, H, NT>(M, W, bias, lane, acc, out);
}

// Packs every layer's weights in fragment order: put(f, lane, frag) gets
// lane `lane`'s 8 elements of packed fragment f (zeros outside the matrix).
// A wave takes whole fragments, four at a time, so eight 4-element loads per
// lane are in flight and no index is divided per element. (With one load and
// three divisions per element the pack was most of a small launch: 1,000
// queries through 20-64-64-3 in FP32 took 24.2 us, now 14.4.) Rows that are
// not aligned for 4-element loads go element by element.
template <class MT, class Put>
__device__ inline void pack_layers(const MlpArgs& M, Put&& put) {
  typedef MT v4 __attribute__((ext_vector_type(4)));
  constexpr int U = 4;
  const int lane = threadIdx.x & 63, r16 = lane & 15, g4 = 4 * (lane >> 4);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int KB0 = (M.K0 + 31) / 32, KH = M.H / 32, MH = M.H / 16;
  const int F = MH * KB0 + (M.n_layers - 2) * MH * KH + KH;
  bool vec = true;
  for (int i = 0; i < M.n_layers; ++i) vec = vec && reinterpret_cast<uintptr_t>(M.W[i]) % sizeof(v4) == 0;
  for (int f0 = wave; f0 < F; f0 += U * waves) {
    v4 v[U][2];
    bool ok[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int f = f0 + u * waves, layer = 0, KB = KB0;
      f = f < F ? f : F - 1;
      while (f >= MH * KB && layer < M.n_layers - 1) {
        f -= MH * KB;
        KB = KH;
        ++layer;
      }
      const int n_in = layer == 0 ? M.K0 : M.H, n_out = layer == M.n_layers - 1 ? M.n_out : M.H;
      const MT* src = reinterpret_cast<const MT*>(M.W[layer]);
      const int row = 16 * (f / KB) + r16;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = 32 * (f % KB) + 16 * h + g4;
        ok[u][h] = row < n_out && col < n_in;  // n_in is a multiple of 4
        const MT* p = src + (ok[u][h] ? (int64_t)row * n_in + col : 0);
        if (vec) {
          v[u][h] = *reinterpret_cast<const v4*>(p);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) v[u][h][j] = p[j];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f0 + u * waves;
      if (f < F) {
        typename FragT<MT>::type a;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j) a[4 * h + j] = ok[u][h] ? v[u][h][j] : from_f32<MT>(0.0f);
        put(f, lane, a);
      }
    }
  }
}

template <class MT>
__device__ inline void pack_weights_lds(const MlpArgs& M, MT* lds) {
  typedef typename FragT<MT>::type frag;
  pack_layers<MT>(M, [&](int f, int lane, const frag& a) { reinterpret_cast<frag*>(lds)[f * kWave + lane] = a; });
}

template <class MT>
__host__ __device__ inline int packed_weight_elems(int n_layers, int K0, int H) {
  return ((H / 16) * ((K0 + 31) / 32) + (n_layers - 2) * (H / 16) * (H / 32) + H / 32) * kWave * 8;
}

// RGB of the 16 NT queries from q0 on.
template <int NT>
__device__ inline void store_rgb(const f32x4 out[NT], int64_t q0, int64_t Q, int lane, float* rgb) {
  if (lane < 16) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int64_t q = q0 + 16 * t + lane;
      if (q < Q) {
        rgb[3 * q + 0] = out[t][0];
        rgb[3 * q + 1] = out[t][1];
        rgb[3 * q + 2] = out[t][2];
      }
    }
  }
}

// Grid of the tile kernels for a workgroup using lds bytes: one workgroup
// per tile up to the resident count, so that a small batch spreads over the
// chip (xcd_tiles hands out the tiles to match).
inline int tile_grid(int64_t n_tiles, size_t lds) {
  // LDS per CU on gfx950 is 160 KiB: one or two workgroups fit per CU.
  const int per_cu = lds * 2 <= (size_t)160 * 1024 ? 2 : 1;
  int64_t g = (int64_t)device_cus() * per_cu;
  if (g > n_tiles) g = n_tiles;
  if (g >= 8) g -= g % 8;
  return (int)(g > 0 ? g : 1);
}

inline size_t bias_bytes(const MlpArgs& M) { return (size_t)bias_floats(M.n_layers, M.H) * sizeof(float); }

}  // namespace oo
