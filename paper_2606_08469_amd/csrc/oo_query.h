// The fused query kernel (oo_query_fwd, and the residual forward's queries),
// instantiated for one decoder type per source file.
#pragma once

#include "oo_mlp.h"

namespace oo {

// ---------------------------------------------------------------------------
// Fused query: encode 64 queries per wave into LDS, decode them there.
// ---------------------------------------------------------------------------
// Queries q < n_idx also store their node index per level in idx_out
// (level-major [L][n_idx]) and their octahedral coordinates in uv_out, which
// the residual backward reads instead of descending and mapping again.
// In the paper's scheme the stored indices are the eight corner cells'
// nodes per level ([L][8][n_idx]) and the query's position is kept too
// (pos_out, [n_idx]); the scatter recomputes the trilinear weights from it.
// With 16-bit operands the level features are kept as well (O.rows,
// [L C / 4][n_idx][4]: a wave's stores are contiguous), so that the backward
// gathers no texels.
// MODE as for encode_kernel; with the shift rgb[3 q] holds query q's
// disparity when the kernel starts (the wave that reads it writes the
// radiance there). MODE 3: the shift with the disparity predicted here, one
// lane per query, for a radiance array that is one of the inputs (every wave
// reads its queries before it writes their radiance). 1280x720 FP16 queries
// take 1.70 ms that way, 1.22 after the predictor's own kernel.
// Streaming (64-wide layers with the weights in LDS, node scheme): the first layer takes
// the inputs chunk by chunk while the gathers of the next levels are in
// flight, so a wave's tile holds one chunk of 32 and the LDS holds more waves:
// gathers, conversions and MFMAs of different waves overlap. 1280x720 queries,
// 72 inputs, three hidden layers: FP32 two or three waves per SIMD in place of
// one, 309 -> 282 us; FP16 four in place of two, 72 -> 68 us (144 registers,
// which allow three only, 73 us). At width 128 the sums of the first layer
// alone take 128 registers, which leaves the two waves that whole tiles
// allow too; the paper scheme's encode takes so many itself that streaming
// spills them (1280x720 queries in FP16: 0.56 ms, whole tiles 0.28).
constexpr bool query_streams(int H, bool wlds, int mode) { return H == 64 && wlds && mode == 0; }
// Waves per workgroup: FP32 takes one workgroup per CU, up to twelve waves
// where the registers (168) do without scratch memory to speak of, 16-bit two
// of eight waves (128 registers).
template <class MT>
constexpr int query_waves(int H, bool wlds, int mode) {
  return query_streams(H, wlds, mode) && sizeof(MT) == 4 ? 12 : 8;
}
template <class MT>
constexpr int query_waves_per_simd(int H, bool wlds, int mode) {
  return query_waves<MT>(H, wlds, mode) / 4 * (query_streams(H, wlds, mode) && sizeof(MT) == 2 ? 2 : 1);
}

// KEEP: queries q < n_idx of this launch are the backward's. The residual
// forward runs the others in a launch of their own, without the stores, where
// that pays (split_queries).
template <class MT, int C, int H, bool WLDS, int MODE, bool KEEP>
__global__ __launch_bounds__(64 * query_waves<MT>(H, WLDS, MODE))
    __attribute__((amdgpu_waves_per_eu(query_waves_per_simd<MT>(H, WLDS, MODE)))) void query_kernel(
    const TreeArgs T, const MlpArgs M, const QuerySrc src, int64_t Q, float* rgb, const QueryOut O, const DispArgs G) {
  int32_t* __restrict__ idx_out = O.idx;
  float2* __restrict__ uv_out = O.uv;
  float4* __restrict__ pos_out = O.pos;
  const int64_t n_idx = O.n_idx;
  MT* const brows = reinterpret_cast<MT*>(O.rows);
  typedef MT v4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // N-tiles per decoder pass: all four with 16-bit operands, LDS weights
  // and 64-wide layers (each weight fragment read then serves four MFMAs;
  // at width 128 the accumulators would spill)
  constexpr int NT = sizeof(MT) == 2 && WLDS && H == 64 ? 4 : 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int KB0 = (M.K0 + 31) / 32;
  constexpr bool STREAM = query_streams(H, WLDS, MODE);
  constexpr int MH = H / 16;
  const int KBT = STREAM ? 1 : KB0;  // chunks the wave's tile holds
  const int wl_elems = WLDS ? packed_weight_elems<MT>(M.n_layers, M.K0, M.H) : 0;
  float* const bias = reinterpret_cast<float*>(smem);
  MT* wl = reinterpret_cast<MT*>(bias + bias_floats(M.n_layers, H));
  MT* htile = wl + wl_elems + wave * (4 * KBT * kWave * 8);
  load_biases_lds(M, bias);
  if (WLDS) pack_weights_lds<MT>(M, wl);
  if (!STREAM) {  // zero the K padding of this lane's row once
    const float z[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = M.K0; k < 32 * KB0; k += 4) htile_put4<MT>(htile, KB0, lane, k, z);
  }
  __syncthreads();
  const WFrag<MT, WLDS> W{wl, KB0};
  const int64_t n_tiles = (Q + 63) / 64;
  const TileRange tr = xcd_tiles(n_tiles, waves, wave);
  for (int64_t tile = tr.first; tile < tr.end; tile += tr.stride) {
    const int64_t q = tile * 64 + lane;
    const bool valid = q < Q;
    float x[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
    if (valid) load_query(src, q, x, d);
    float s, t;
    octa(d, s, t);
    const bool keep = KEEP && q < Q && q < n_idx;
    f32x4 acc0[STREAM ? MH : 1][4];  // the first layer's sums
    if constexpr (STREAM) {
#pragma unroll
      for (int m = 0; m < MH; ++m) {
        const f32x4 b = bias_tile(bias, m, lane);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc0[m][t] = b;
      }
    }
    // Inputs k .. k + 3 of this lane's query, in the order of k. Streaming,
    // each full chunk of 32 goes through the first layer at once.
    auto input4 = [&](int k, const float* v) {
      htile_put4<MT>(htile, KBT, lane, STREAM ? k & 31 : k, v);
      if constexpr (STREAM) {
        if ((k & 31) != 28) return;
        wave_lds_sync();
#pragma unroll
        for (int t0 = 0; t0 < 4; t0 += NT) {
          typename FragT<MT>::type b[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) b[t] = htile_get<MT>(htile, 1, t0 + t, 0, lane);
#pragma unroll
          for (int m = 0; m < MH; ++m) {
            const auto a = W.get(M, 0, m, k >> 5, lane);
#pragma unroll
            for (int t = 0; t < NT; ++t) acc0[m][t0 + t] = mma(a, b[t], acc0[m][t0 + t]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        wave_lds_sync();
      }
    };
    if (keep) uv_out[q] = make_float2(s, t);
    if constexpr (MODE > 0) {
      float u[3] = {0.f, 0.f, 0.f}, disp = 0.0f;
      if constexpr (MODE >= 2) {
        unit_dir3(d, u);
        if constexpr (MODE == 3)
          disp = predict_lane(G, x, u);
        else if (valid)
          disp = rgb[3 * q];
      }
      if (keep) pos_out[q] = make_float4(x[0], x[1], x[2], disp);
      encode_paper<MT, C, MODE >= 2>(T, valid, x, s, t, [&](int l, const float* h, const int (&node)[8], auto& last) {
#pragma unroll
        for (int c = 0; c < C; c += 4) input4(l * C + c, &h[c]);
        if (keep) {
#pragma unroll
          for (int d = 0; d < 8; ++d) idx_out[(l * 8 + d) * n_idx + q] = node[d];  // coalesced across lanes
          if constexpr (sizeof(MT) == 2)
            if (brows)
#pragma unroll
              for (int c = 0; c < C; c += 4)
                *reinterpret_cast<v4*>(brows + (((l * C + c) >> 2) * n_idx + q) * 4) = last.round4(c);
        }
      }, disp, u);
    } else {
      encode_pipelined<MT, C>(T, valid, x, s, t, [&](int l, const float* h, int node, auto& last) {
#pragma unroll
        for (int c = 0; c < C; c += 4) input4(l * C + c, &h[c]);
        if (keep) {
          idx_out[l * n_idx + q] = node;  // level-major: coalesced across lanes
          if constexpr (sizeof(MT) == 2)
            if (brows)
#pragma unroll
              for (int c = 0; c < C; c += 4)
                *reinterpret_cast<v4*>(brows + (((l * C + c) >> 2) * n_idx + q) * 4) = last.round4(c);
        }
      });
    }
    // the decoder's surface attributes follow the level features
    for (int k = 0; k < M.E; k += 4) {
      float g4[4] = {0.f, 0.f, 0.f, 0.f};
      if (valid) load_attr4(src, q, k, g4);
      input4(M.K0 - M.E + k, g4);
    }
    if constexpr (STREAM) {  // the rest of the last chunk
      const float z[4] = {0.f, 0.f, 0.f, 0.f};
      for (int k = M.K0; k & 31; k += 4) input4(k, z);
    }
    wave_lds_sync();
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += NT) {
      f32x4 out[NT];
      if constexpr (STREAM) {
        f32x4 acc[MH][NT];
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[m][t] = acc0[m][t0 + t];
        mlp_rest<MT, H, NT>(M, W, bias, lane, acc, out);
      } else {
        mlp_forward_tiles<MT, H, NT, 0>(
            M, W, bias, KB0, lane, [&](int kb, int t) { return htile_get<MT>(htile, KB0, t0 + t, kb, lane); }, out);
      }
      store_rgb<NT>(out, tile * 64 + 16 * t0, Q, lane, rgb);
    }
    wave_lds_sync();
  }
}

// The shape without weights in LDS: as many 64-query tiles as fit, up to 8.
template <class MT>
static void tile_launch_shape_plain(const MlpArgs& M, int64_t Q, int& waves, size_t& lds, int& grid) {
  const int KB0 = (M.K0 + 31) / 32;
  const size_t tile_bytes = (size_t)4 * KB0 * kWave * 8 * sizeof(MT);
  const size_t bb = bias_bytes(M);
  waves = 8;
  while (waves > 1 && bb + waves * tile_bytes > (size_t)max_lds()) --waves;
  lds = bb + waves * tile_bytes;
  grid = tile_grid((Q + 63) / 64, lds);
}

// Workgroup shape for the tile kernels: up to query_waves, each with a 64-query
// activation tile, plus the packed weights when they fit next to them.
template <class MT>
static void tile_launch_shape(const MlpArgs& M, int mode, int64_t Q, bool& wlds, int& waves, size_t& lds, int& grid) {
  const int KB0 = query_streams(M.H, true, mode) ? 1 : (M.K0 + 31) / 32;
  const size_t tile_bytes = (size_t)4 * KB0 * kWave * 8 * sizeof(MT);
  const size_t wbytes = (size_t)packed_weight_elems<MT>(M.n_layers, M.K0, M.H) * sizeof(MT);
  const size_t bb = bias_bytes(M);
  const size_t cap = (size_t)max_lds() - bb;
  waves = query_waves<MT>(M.H, true, mode);
  wlds = true;
  while (waves > 4 && wbytes + waves * tile_bytes > cap) --waves;
  if (wlds && wbytes + waves * tile_bytes > cap) wlds = false;
  if (!wlds) {
    tile_launch_shape_plain<MT>(M, Q, waves, lds, grid);
    return;
  }
  // more than eight waves: the number that wastes least of the last round of
  // a CU's tiles (a CU with 64 tiles has eight full rounds of 8, but 5 1/3 of
  // 12: 2^20 queries take 343 us with 8 and 384 with 12; with 57 tiles, eight
  // rounds of 8 or five of 12, 295 and 282), the larger of equals
  if (waves > 8) {
    const int64_t n = ((Q + 63) / 64 + device_cus() - 1) / device_cus();
    int best = 8;
    for (int w = 9; w <= waves; ++w)
      if ((n + w - 1) / w * w <= (n + best - 1) / best * best) best = w;
    waves = best;
  }
  lds = bb + wbytes + waves * tile_bytes;
  grid = tile_grid((Q + 63) / 64, lds);
}

// Whether the Q - n queries after the first n run in a launch of their own,
// whose kernel stores nothing for the backward. It pays where it costs no
// more rounds of the chip (tiles that a workgroup has time for, idle ones
// among them), or where the second launch is long enough to make up for one
// that is mostly idle: eight rounds, or three with streamed 16-bit layers,
// whose rounds the stores slow down by a fifth. Training steps back to back,
// without the split and with it: FP32, 128-wide, 4,000 points x 8 354 and 455
// us, 100,000 x 4 1414 and 1488; FP16, 64-wide, 60,000 x 3 257 and 264, 200,000
// x 4 619 and 588, 262,144 x 4 694 and 652. Of 52 sizes drawn at random the rule
// takes the faster way, or one within 2% of it, in 51.
template <class MT>
static bool split_queries(const MlpArgs& M, int mode, int64_t n, int64_t Q) {
  int64_t rounds = 0;
  auto slots = [&](int64_t q) {
    bool wlds;
    int waves, grid;
    size_t lds;
    tile_launch_shape<MT>(M, mode, q, wlds, waves, lds, grid);
    const int64_t tiles = (q + 63) / 64, round = (int64_t)grid * waves;
    rounds = tiles / round;
    return (tiles + round - 1) / round * waves;
  };
  const int64_t all = slots(Q), kept = slots(n), rest = slots(Q - n);
  return kept + rest <= all || rounds >= (query_streams(M.H, true, mode) && sizeof(MT) == 2 ? 3 : 8);
}

template <class MT, int C, int H, int MODE, bool KEEP>
static hipError_t launch_query_p(const TreeArgs& T, const MlpArgs& M, const QuerySrc& src, int64_t Q, float* rgb,
                                 const QueryOut& O, const DispArgs& G, hipStream_t st) {
  bool wlds;
  int waves, grid;
  size_t lds;
  tile_launch_shape<MT>(M, MODE, Q, wlds, waves, lds, grid);
  if (wlds && MODE >= 2) {  // the shifted variants: keep one of each
    wlds = false;
    tile_launch_shape_plain<MT>(M, Q, waves, lds, grid);
  }
  if (wlds) {
    auto k = query_kernel<MT, C, H, true, MODE >= 2 ? 1 : MODE, KEEP>;
    allow_lds((const void*)k, lds);
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * waves), lds, st, T, M, src, Q, rgb, O, G);
  } else {
    auto k = query_kernel<MT, C, H, false, MODE, KEEP>;
    allow_lds((const void*)k, lds);
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * waves), lds, st, T, M, src, Q, rgb, O, G);
  }
  return hipGetLastError();
}

// Whether Q rows of `width` floats from out on share memory with a caller's
// queries.
inline bool overlaps(const float* out, int width, const QuerySrc& src, int64_t Q) {
  const uintptr_t o = reinterpret_cast<uintptr_t>(out), oe = o + sizeof(float) * width * Q;
  const auto hit = [&](const float* p, int64_t w) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return p && a < oe && o < a + sizeof(float) * w * Q;
  };
  return hit(src.xA, 3) || hit(src.dA, 3) || hit(src.gA, src.E);
}

template <class MT, int C, int H>
static hipError_t launch_query_t(const TreeArgs& T, const MlpArgs& M, const QuerySrc& src, int64_t Q, float* rgb,
                                 const QueryOut& O, const DispArgs& G, hipStream_t st) {
  if (T.interp == OO_INTERP_PAPER && G.n_levels > 0) {
    if (overlaps(rgb, 3, src, Q)) return launch_query_p<MT, C, H, 3, false>(T, M, src, Q, rgb, O, G, st);
    const hipError_t e = launch_predict(G, src, Q, rgb, 3, st);
    return e != hipSuccess ? e : launch_query_p<MT, C, H, 2, false>(T, M, src, Q, rgb, O, G, st);
  }
  const bool paper = T.interp == OO_INTERP_PAPER;
  if (O.n_idx > 0) {
    int64_t n = O.n_idx < Q ? O.n_idx : Q;
    if (n < Q && !split_queries<MT>(M, paper, n, Q)) n = Q;
    const hipError_t e = paper ? launch_query_p<MT, C, H, 1, true>(T, M, src, n, rgb, O, G, st)
                               : launch_query_p<MT, C, H, 0, true>(T, M, src, n, rgb, O, G, st);
    if (e != hipSuccess || n == Q) return e;
    QuerySrc rest = src;  // sorted positions n ..
    rest.idx += n;
    return paper ? launch_query_p<MT, C, H, 1, false>(T, M, rest, Q - n, rgb + 3 * n, O, G, st)
                 : launch_query_p<MT, C, H, 0, false>(T, M, rest, Q - n, rgb + 3 * n, O, G, st);
  }
  return paper ? launch_query_p<MT, C, H, 1, false>(T, M, src, Q, rgb, O, G, st)
               : launch_query_p<MT, C, H, 0, false>(T, M, src, Q, rgb, O, G, st);
}

template <class MT>
hipError_t launch_query_m(const TreeArgs& T, const MlpArgs& M, const QuerySrc& src, int64_t Q, float* rgb,
                          const QueryOut& O, const DispArgs& G, hipStream_t st) {
  if (Q == 0) return hipSuccess;
  if (T.C == 4)
    return M.H == 64 ? launch_query_t<MT, 4, 64>(T, M, src, Q, rgb, O, G, st)
                     : launch_query_t<MT, 4, 128>(T, M, src, Q, rgb, O, G, st);
  return M.H == 64 ? launch_query_t<MT, 8, 64>(T, M, src, Q, rgb, O, G, st)
                   : launch_query_t<MT, 8, 128>(T, M, src, Q, rgb, O, G, st);
}

}  // namespace oo
