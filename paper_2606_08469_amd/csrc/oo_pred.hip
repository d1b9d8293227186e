// Forward of the disparity predictor (Sec. 3.3 disparity equation, Sec. 3.5
// hash-grid network) on the matrix cores: for the residual step's queries,
// and for the render and encode entry points.
#include <hip/hip_runtime.h>

#include "oo_mlp.h"

namespace oo {

// ---------------------------------------------------------------------------
// Disparity predictor on the matrix cores: each wave encodes 64 queries'
// positions (hash grid) and lookup directions into its FP32 activation tile
// and runs the predictor's MLP on it like the decoder's, writing d per
// query. FP32 path: 16x16x4 FP32 MFMA, weights from L2. 16-bit path
// (SPLIT): every operand is split into two BF16 parts, x = hi + lo with
// hi = bf16(x) and lo = bf16(x - hi) (about 16 significant bits, FP32's
// exponent range), and each product is hi hi + hi lo + lo hi on 16x16x32
// BF16 MFMA with FP32 accumulation: three MFMAs of 16 cycles for each
// eight FP32 ones of 32. The weights are split once per workgroup into LDS.
// hi + lo holds x to 2^-16 relative (each part rounds to 8 significant
// bits) and the dropped lo lo term is below 2^-16 of the product, so each
// product carries at most about 3 * 2^-16 relative error. (A plain 16-bit
// predictor moves shifted lookups across triangle edges often enough to
// break its gradients' agreement.)
// ---------------------------------------------------------------------------

// Packs the predictor's FP32 weights into LDS in fragment order, split into
// BF16 hi (at hi) and lo (at hi + the packed size) parts.
__device__ inline void pack_weights_split(const MlpArgs& M, bf16* hi, int total_elems) {
  pack_layers<float>(M, [&](int f, int lane, const f32x8& w) {
    bf16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h[i] = from_f32<bf16>(w[i]);
      l[i] = from_f32<bf16>(w[i] - to_f32(h[i]));
    }
    reinterpret_cast<bf16x8*>(hi)[f * kWave + lane] = h;
    reinterpret_cast<bf16x8*>(hi + total_elems)[f * kWave + lane] = l;
  });
}

__device__ __forceinline__ void split8(const float (&v)[8], bf16x8& h, bf16x8& l) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bf16 a = from_f32<bf16>(v[i]);
    h[i] = a;
    l[i] = from_f32<bf16>(v[i] - to_f32(a));
  }
}

// acc += A B with A, B split: hi hi + hi lo + lo hi.
__device__ __forceinline__ f32x4 mma_split(const bf16x8& ah, const bf16x8& al, const bf16x8& bh, const bf16x8& bl,
                                           f32x4 c) {
  c = mma(ah, bh, c);
  c = mma(ah, bl, c);
  return mma(al, bh, c);
}

// The predictor's MLP (width 64) on N-tiles t0 .. t0+NT-1 with split
// operands; out[t] rows 0.. = d in lanes 0..15. The input's first K-chunk
// (the 32 hash features) comes from the wave's one-chunk FP32 tile; the
// second holds only the unit direction (inputs 32..34, input 35 zero),
// which the lanes of group 0 take from the lane that owns the query, so the
// tile needs half the LDS.
static_assert(kDispK == 36, "the predictor's input is 32 hash features, the unit direction and a zero");
template <int NT>
__device__ inline void disp_mlp_split(const MlpArgs& M, const WFrag<bf16, true>& Wh, const WFrag<bf16, true>& Wl,
                                      const float* bias, const float* htile, const float u[3], int t0, int lane,
                                      f32x4 out[NT]) {
  constexpr int MH = kDispH / 16, KH = kDispH / 32;
  f32x4 acc[MH][NT];
#pragma unroll
  for (int m = 0; m < MH; ++m) {
    const f32x4 bt = bias_tile(bias, m, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[m][t] = bt;
  }
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    bf16x8 bh[NT], bl[NT], ah[MH], al[MH];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float v[8];
      if (kb == 0) {
        const f32x8 x = htile_get<float>(htile, 1, t0 + t, 0, lane);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = x[i];
      } else {
        // slot i < 4 of group g holds input 32 + 4g + i; the rest are >= 48
        const int src = 16 * (t0 + t) + (lane & 15);
        const float s0 = __shfl(u[0], src), s1 = __shfl(u[1], src), s2 = __shfl(u[2], src);
        const bool g0 = (lane >> 4) == 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.0f;
        v[0] = g0 ? s0 : 0.0f;
        v[1] = g0 ? s1 : 0.0f;
        v[2] = g0 ? s2 : 0.0f;
      }
      split8(v, bh[t], bl[t]);
    }
#pragma unroll
    for (int m = 0; m < MH; ++m) {
      ah[m] = Wh.get(M, 0, m, kb, lane);
      al[m] = Wl.get(M, 0, m, kb, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < MH; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[m][t] = mma_split(ah[m], al[m], bh[t], bl[t], acc[m][t]);
  }
  // ReLU'd outputs of tiles (2kb, 2kb+1) are the next layer's chunk kb
  auto chain = [&](int kb, int t, bf16x8& h, bf16x8& l) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = fmaxf(acc[2 * kb][t][j], 0.0f);
      v[4 + j] = fmaxf(acc[2 * kb + 1][t][j], 0.0f);
    }
    split8(v, h, l);
  };
  for (int layer = 1; layer < M.n_layers - 1; ++layer) {
    bf16x8 bh[KH][NT], bl[KH][NT];
#pragma unroll
    for (int kb = 0; kb < KH; ++kb)
#pragma unroll
      for (int t = 0; t < NT; ++t) chain(kb, t, bh[kb][t], bl[kb][t]);
#pragma unroll
    for (int m = 0; m < MH; ++m) {
      const f32x4 bt = bias_tile(bias + layer * kDispH, m, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[m][t] = bt;
    }
#pragma unroll
    for (int kb = 0; kb < KH; ++kb) {
      bf16x8 ah[MH], al[MH];
#pragma unroll
      for (int m = 0; m < MH; ++m) {
        ah[m] = Wh.get(M, layer, m, kb, lane);
        al[m] = Wl.get(M, layer, m, kb, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MH; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = mma_split(ah[m], al[m], bh[kb][t], bl[kb][t], acc[m][t]);
    }
  }
  const int lo = M.n_layers - 1;
  const f32x4 bo = bias_tile(bias + lo * kDispH, 0, lane);
#pragma unroll
  for (int t = 0; t < NT; ++t) out[t] = bo;
#pragma unroll
  for (int kb = 0; kb < KH; ++kb) {
    const bf16x8 ah = Wh.get(M, lo, 0, kb, lane), al = Wl.get(M, lo, 0, kb, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      bf16x8 bh, bl;
      chain(kb, t, bh, bl);
      out[t] = mma_split(ah, al, bh, bl, out[t]);
    }
  }
}

template <bool SPLIT>
__global__ __launch_bounds__(256) void disparity_fwd_kernel(const DispArgs G, const MlpArgs P, const QuerySrc src,
                                                            int64_t Q, float* __restrict__ d_out) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int NT = 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int KB0 = (P.K0 + 31) / 32;
  const int KBT = SPLIT ? 1 : KB0;  // K-chunks the FP32 tile holds
  const int wl_elems = SPLIT ? packed_weight_elems<bf16>(P.n_layers, P.K0, P.H) : 0;
  float* const bias = reinterpret_cast<float*>(smem);
  bf16* const wl = reinterpret_cast<bf16*>(bias + bias_floats(P.n_layers, kDispH));
  float* const htile = reinterpret_cast<float*>(wl + 2 * wl_elems) + wave * (4 * KBT * kWave * 8);
  load_biases_lds(P, bias);
  if (SPLIT) pack_weights_split(P, wl, wl_elems);
  {  // zero the K padding of this lane's row once
    const float z[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = P.K0; k < 32 * KBT; k += 4) htile_put4<float>(htile, KBT, lane, k, z);
  }
  __syncthreads();
  const WFrag<float, false> W{nullptr, KB0};
  const WFrag<bf16, true> Wh{wl, KB0}, Wlo{wl + wl_elems, KB0};
  const int64_t n_tiles = (Q + 63) / 64;
  const TileRange tr = xcd_tiles(n_tiles, waves, wave);
  for (int64_t tile = tr.first; tile < tr.end; tile += tr.stride) {
    const int64_t q = tile * 64 + lane;
    float x[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f}, u[3];
    if (q < Q) load_query(src, q, x, d);
    unit_dir3(d, u);
    float a[kDispK];
    disparity_input(G, x, u, a);
#pragma unroll
    for (int k = 0; k < (SPLIT ? 32 : kDispK); k += 4) htile_put4<float>(htile, KBT, lane, k, &a[k]);
    wave_lds_sync();
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += NT) {
      f32x4 out[NT];
      if constexpr (SPLIT)
        disp_mlp_split<NT>(P, Wh, Wlo, bias, htile, u, t0, lane, out);
      else
        mlp_forward_tiles<float, kDispH, NT, (kDispK + 31) / 32>(
            P, W, bias, KB0, lane, [&](int kb, int t) { return htile_get<float>(htile, KB0, t0 + t, kb, lane); }, out);
      if (lane < 16) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int64_t qq = tile * 64 + 16 * (t0 + t) + lane;
          if (qq < Q) d_out[qq] = out[t][0];
        }
      }
    }
    wave_lds_sync();
  }
}

hipError_t launch_disparity_fwd(const DispArgs& G, oo_dtype md, const QuerySrc& src, int64_t Q, float* d_out,
                                hipStream_t st) {
  if (Q == 0) return hipSuccess;
  MlpArgs P{};
  P.n_layers = G.n_layers;
  P.K0 = kDispK;
  P.E = 0;
  P.H = kDispH;
  P.n_out = 1;
  for (int i = 0; i < kMaxLayers; ++i) {
    P.W[i] = i < G.n_layers ? G.W[i] : nullptr;
    P.b[i] = i < G.n_layers ? G.b[i] : nullptr;
  }
  // four-wave workgroups, two per CU: four 16 KiB FP32 tiles, or for the
  // split variant the hi and lo weight copies (2 x 18 KiB) and four 8 KiB
  // one-chunk tiles
  const bool split = md != OO_F32;
  constexpr int waves = 4;
  const size_t wbytes = split ? (size_t)2 * packed_weight_elems<bf16>(P.n_layers, P.K0, P.H) * sizeof(bf16) : 0;
  const int kbt = split ? 1 : (P.K0 + 31) / 32;
  const size_t lds = bias_bytes(P) + wbytes + (size_t)waves * 4 * kbt * kWave * 8 * sizeof(float);
  const int grid = tile_grid((Q + 63) / 64, lds);
  if (split) {
    allow_lds((const void*)disparity_fwd_kernel<true>, lds);
    hipLaunchKernelGGL(disparity_fwd_kernel<true>, dim3(grid), dim3(64 * waves), lds, st, G, P, src, Q, d_out);
  } else {
    allow_lds((const void*)disparity_fwd_kernel<false>, lds);
    hipLaunchKernelGGL(disparity_fwd_kernel<false>, dim3(grid), dim3(64 * waves), lds, st, G, P, src, Q, d_out);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The predictor for single queries (render and encode): FP32 MFMA whose sums
// run in the order of the inputs. v_mfma_f32_16x16x4_f32 adds its four
// products to C one after the other, each with one rounding, so a layer
// z = b + sum_k W[k] a[k] taken four consecutive k at a time is the plain
// FMA chain over k, to the bit. Step s takes inputs 4 s + g (lane group g);
// output row 4 g + j of tile m holds unit 16 m + 4 j + g, so that register j
// of tile m is, unchanged, the operand of step 4 m + j of the next layer.
// The weights are packed once per workgroup into LDS, four steps per 16-byte
// read. Bound by the gathers of the hash entries. (One lane per query with
// the weights read from memory by every wave took 1.0 ms of a 1280x720
// render; this takes 0.23.)
// ---------------------------------------------------------------------------
constexpr int kPredStride = 80;  // floats between inputs of the [input][query] tile: no bank conflicts
constexpr int kPredWaves = 4;
constexpr int kPredQ0 = (kDispK / 4 + 3) / 4;  // 16-byte groups of steps, first layer (3) and hidden ones (4)
constexpr int kPredQH = kDispH / 16;

__host__ __device__ inline int predict_frags(int n_layers) {
  return 4 * kPredQ0 + (n_layers - 2) * 4 * kPredQH + kPredQH;  // the output layer has one tile
}

__global__ __launch_bounds__(64 * kPredWaves) void predict_kernel(const DispArgs G, const QuerySrc src, int64_t Q,
                                                                  float* __restrict__ out, int64_t stride) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int MH = kDispH / 16, NT = 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, r16 = lane & 15;
  const bool two = G.n_layers == 3;
  const int F = predict_frags(G.n_layers);
  f32x4* const wl = reinterpret_cast<f32x4*>(smem);
  float* const bias = reinterpret_cast<float*>(wl + F * kWave);  // [n_layers - 1][64], then the output's
  float* const tile = bias + 3 * kDispH + wave * kDispK * kPredStride;
  for (int f = wave; f < F; f += kPredWaves) {
    const int layer = f < MH * kPredQ0 ? 0 : (two && f < MH * (kPredQ0 + kPredQH) ? 1 : 2);  // 2: the output layer
    const int e = layer == 0 ? f : (layer == 1 ? f - MH * kPredQ0 : f - MH * kPredQ0 - (two ? MH * kPredQH : 0));
    const int per = layer == 0 ? kPredQ0 : kPredQH, m = e / per, sq = e % per;
    const int n_in = layer == 0 ? kDispK : kDispH, n_out = layer == 2 ? 1 : kDispH;
    const float* W = layer == 0 ? G.W[0] : (layer == 1 || !two ? G.W[1] : G.W[2]);
    const int row = 16 * m + 4 * (r16 & 3) + (r16 >> 2);
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int col = 4 * (4 * sq + i) + g;
      const bool ok = row < n_out && col < n_in;
      v[i] = ok ? W[row * n_in + col] : 0.0f;
    }
    wl[f * kWave + lane] = v;
  }
  for (int e = threadIdx.x; e < kDispH; e += blockDim.x) {
    bias[e] = G.b[0][e];
    if (two) bias[kDispH + e] = G.b[1][e];
  }
  if (threadIdx.x == 0) bias[2 * kDispH] = (two ? G.b[2] : G.b[1])[0];
  __syncthreads();
  const f32x4* const w1 = wl + MH * kPredQ0 * kWave;
  const f32x4* const wo = w1 + (two ? MH * kPredQH * kWave : 0);
  const TileRange tr = xcd_tiles((Q + 63) / 64, kPredWaves, wave);
  for (int64_t it = tr.first; it < tr.end; it += tr.stride) {
    const int64_t q = it * 64 + lane;
    float x[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f}, u[3];
    if (q < Q) load_query(src, q, x, d);
    unit_dir3(d, u);
    {
      float a[kDispK];
      disparity_input(G, x, u, a);
#pragma unroll
      for (int k = 0; k < kDispK; ++k) tile[k * kPredStride + lane] = a[k];
    }
    wave_lds_sync();
#pragma unroll 1
    for (int t0 = 0; t0 < 4; t0 += NT) {
      f32x4 acc[MH][NT], o[NT];
      auto init = [&](int layer) {  // unit 16 m + 4 j + g
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float b = bias[layer * kDispH + 16 * m + 4 * j + g];
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[m][t][j] = b;
          }
      };
      init(0);
#pragma unroll
      for (int sq = 0; sq < kPredQ0; ++sq) {
        f32x4 w[MH];
#pragma unroll
        for (int m = 0; m < MH; ++m) w[m] = wl[(m * kPredQ0 + sq) * kWave + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int s = 4 * sq + i;
          if (4 * s >= kDispK) break;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float b = tile[(4 * s + g) * kPredStride + 16 * (t0 + t) + r16];
#pragma unroll
            for (int m = 0; m < MH; ++m)
              acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[m][i], b, acc[m][t], 0, 0, 0);
          }
        }
      }
      float h[MH][NT][4];  // operand of step 4 m + j
      auto relu = [&] {
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) h[m][t][j] = fmaxf(acc[m][t][j], 0.0f);
      };
      relu();
      if (two) {
        init(1);
#pragma unroll
        for (int sq = 0; sq < kPredQH; ++sq) {
          f32x4 w[MH];
#pragma unroll
          for (int m = 0; m < MH; ++m) w[m] = w1[(m * kPredQH + sq) * kWave + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int m = 0; m < MH; ++m)
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[m][i], h[sq][t][i], acc[m][t], 0, 0, 0);
        }
        relu();
      }
      const float bo = bias[2 * kDispH];
#pragma unroll
      for (int t = 0; t < NT; ++t) o[t] = f32x4{bo, bo, bo, bo};  // row 0 is the output
#pragma unroll
      for (int sq = 0; sq < kPredQH; ++sq) {
        const f32x4 w = wo[sq * kWave + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int t = 0; t < NT; ++t) o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], h[sq][t][i], o[t], 0, 0, 0);
      }
      if (lane < 16) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int64_t qq = it * 64 + 16 * (t0 + t) + lane;
          if (qq < Q) out[qq * stride] = o[t][0];
        }
      }
    }
    wave_lds_sync();
  }
}

hipError_t launch_predict(const DispArgs& G, const QuerySrc& src, int64_t Q, float* out, int64_t stride,
                          hipStream_t st) {
  if (Q == 0) return hipSuccess;
  const size_t lds = (size_t)predict_frags(G.n_layers) * kWave * sizeof(f32x4) +
                     (3 * kDispH + kPredWaves * kDispK * kPredStride) * sizeof(float);
  allow_lds((const void*)predict_kernel, lds);
  hipLaunchKernelGGL(predict_kernel, dim3(tile_grid((Q + 63) / 64, lds)), dim3(64 * kPredWaves), lds, st, G, src, Q,
                     out, stride);
  return hipGetLastError();
}

}  // namespace oo
