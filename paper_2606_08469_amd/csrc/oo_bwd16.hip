// The decoder backward with 16-bit operands: recompute, delta chain and the
// weight gradients.
//
// Every wave carries 16 queries of its own through the whole chain in
// registers, from the level features that the forward kept and the caller's
// surface attributes: the hidden layers, then the gradient back through the
// transposed weights. Only the weight gradients need the workgroup: dW of a
// layer is contracted over all its queries, each wave owning a block of dW
// tiles in registers for the whole kernel, so activations and deltas pass
// through LDS once per layer, two barriers each. The next tile's inputs and
// seeds are loaded while this one is worked on.
//
// One packed copy of the weights serves both directions. A fragment is kept
// as two planes of 4 elements per lane (its slots 0-3 and 4-7); the forward
// reads both planes in order, and the transposed operand of the backward is
// read with ds_read_tr16_b64: of every 16 lanes, lane i receives element
// i % 4 of what lanes i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4 address.
// The same read turns a layer's activations, stored as the operands they
// are, into the [neuron][queries] operands of dW.
//
// Bound by LDS reads and the two barriers per layer; the matrix cores are a
// third busy. 262,144 queries, 88 features, two 128-wide hidden layers in
// FP16: 96 us, where one kernel that shared 64 queries between its waves and
// gathered the features again took 335 us; 32,768 queries, 48 inputs, four
// 128-wide layers: 63 us after 403 us. A bias sum needs an accumulator of its
// own per layer: one shared by all layers, a column each, is 1% faster but
// lets an infinite delta of one layer make the others' sums NaN (zero times
// infinity).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "oo_bwd16.h"

namespace oo {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) s16x4* lds_s16x4;

template <class MT>
__device__ __forceinline__ typename FragT<MT>::type join(const s16x4& lo, const s16x4& hi) {
  union {
    s16x4 s[2];
    typename FragT<MT>::type f;
  } u;
  u.s[0] = lo;
  u.s[1] = hi;
  return u.f;
}

// Fragment as stored: slots 0-3 and 4-7 of this lane.
template <class MT>
__device__ __forceinline__ typename FragT<MT>::type plane_frag(const MT* f, int lane) {
  return join<MT>(*reinterpret_cast<const s16x4*>(f + 4 * lane), *reinterpret_cast<const s16x4*>(f + kPlane + 4 * lane));
}

template <class MT>
__device__ __forceinline__ void put_planes(MT* f, int lane, const typename FragT<MT>::type& a) {
  union {
    typename FragT<MT>::type f;
    s16x4 s[2];
  } u;
  u.f = a;
  *reinterpret_cast<s16x4*>(f + 4 * lane) = u.s[0];
  *reinterpret_cast<s16x4*>(f + kPlane + 4 * lane) = u.s[1];
}

// One plane read transposed: `at` is the lane's own element offset
// (tr_offset), and lane (g, r) receives element r % 4 of lanes
// 16 (r / 4) + 4 g .. + 3 of the plane.
template <class MT>
__device__ __forceinline__ s16x4 tr_plane(const MT* plane, int at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(const_cast<MT*>(plane) + at));
}
__device__ __forceinline__ int tr_offset(int lane) {
  const int g = lane >> 4, k = (lane >> 2) & 3, p = lane & 3;
  return (p * 16 + 4 * g + k) * 4;
}

}  // namespace

// NW waves, NHH hidden-to-hidden layers. nput < NW (the largest decoders):
// the exchange buffers take the waves' operands in NW / nput turns.
template <class MT, int H, int NW, int NHH>
__global__ __launch_bounds__(64 * NW) void bwd16_kernel(const MlpArgs M, const int LC, const BwdArgs A,
                                                        const ParamLayout PL, const int nput) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef typename FragT<MT>::type frag;
  constexpr int MH = H / 16, KH = H / 32, NL = NHH + 2;
  // dW blocks: RB row tiles x CB column tiles per wave, NC column blocks
  constexpr int RB = MH / 4, NC = NW / 4, CB = MH / NC, CB0 = 8 / NC, UO = (MH + NW - 1) / NW;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = RB * (wave / NC), cset = wave % NC;
  const int K0 = M.K0, NK0 = (K0 + 15) / 16;
  const Bwd16Layout lay = bwd16_layout(K0, H, NL, NW, nput);
  const int KB0 = lay.KB0;
  float* const bias = reinterpret_cast<float*>(smem);
  MT* const wl = reinterpret_cast<MT*>(smem + lay.w);
  MT* const A0 = reinterpret_cast<MT*>(smem + lay.a0);
  MT* const A0w = A0 + wave * KB0 * kFrag;
  MT* const X = reinterpret_cast<MT*>(smem + lay.x);
  MT* const Y = reinterpret_cast<MT*>(smem + lay.y);
  load_biases_lds(M, bias);
  pack_layers<MT>(M, [&](int f, int ln, const frag& a) { put_planes<MT>(wl + (size_t)f * kFrag, ln, a); });
  // fragment (0, 0) of hidden layer 1 + hh, or (hh = NHH) of the output layer
  auto layer_w = [&](int hh) { return wl + (MH * KB0 + hh * MH * KH) * kFrag; };

  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  constexpr int NHA = NHH > 0 ? NHH : 1;
  f32x4 acc0[RB][CB0], accH[NHA][RB][CB], accO[UO], db0[RB], dbH[NHA][RB], dbO;
  float* const part = A.partials + (int64_t)blockIdx.x * PL.P;
  // Visits every dW and db tile this wave owns: tile(acc, rows, columns,
  // offset of the matrix, row tile, column tile); a bias is a matrix of one
  // column.
  auto each_tile = [&](auto&& tile) {
    const int dk = K0, dh = H;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int cb = 0; cb < CB0; ++cb)
        if (cset * CB0 + cb < NK0) tile(acc0[rb][cb], H, dk, PL.w_off[0], row0 + rb, cset * CB0 + cb);
      if (cset == 0) tile(db0[rb], H, 1, PL.b_off[0], row0 + rb, 0);
#pragma unroll
      for (int hh = 0; hh < NHH; ++hh) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) tile(accH[hh][rb][cb], H, dh, PL.w_off[1 + hh], row0 + rb, cset * CB + cb);
        if (cset == 0) tile(dbH[hh][rb], H, 1, PL.b_off[1 + hh], row0 + rb, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < UO; ++u)
      if (wave + NW * u < MH) tile(accO[u], 3, dh, PL.w_off[NL - 1], 0, wave + NW * u);
    if (wave == 0) tile(dbO, 3, 1, PL.b_off[NL - 1], 0, 0);
  };
  // the sums start from what this workgroup's earlier launches left (every
  // column of a bias tile holds the bias sum)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    db0[rb] = z4;
#pragma unroll
    for (int cb = 0; cb < CB0; ++cb) acc0[rb][cb] = z4;
#pragma unroll
    for (int h = 0; h < NHH; ++h) {
      dbH[h][rb] = z4;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) accH[h][rb][cb] = z4;
    }
  }
#pragma unroll
  for (int u = 0; u < UO; ++u) accO[u] = z4;
  dbO = z4;
  if (A.accumulate) {
    const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
    each_tile([&](f32x4& acc, int n_out, int n_in, int64_t off, int mm, int nk) {
      const int k = n_in == 1 ? 0 : 16 * nk + r16;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = 16 * mm + 4 * g + j;
        const bool in = n < n_out && k < n_in;
        const float v = part[off + (in ? n * n_in + k : 0)];
        acc[j] = in ? v : 0.0f;
      }
    });
  }
  frag ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = from_f32<MT>(1.0f);
  __syncthreads();

  // ---- inputs: a lane's two runs of four inputs per chunk, and the seeds ----
  s16x4 raw[4][2];
  float sd[3];
  int src_q = -1;  // source query, whose surface attributes the decoder reads
  const MT* const rows = reinterpret_cast<const MT*>(A.rows);
  auto load = [&](int64_t tile) {
    const int lane = threadIdx.x & 63;
    const int64_t q = tile * 16 * NW + wave * 16 + (lane & 15);
    const int64_t qc = q < A.Q ? q : A.Q - 1;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {  // (columns past L C read the first ones: masked below)
        const int col = 32 * kb + 16 * hf + 4 * (lane >> 4);
        raw[kb][hf] = *reinterpret_cast<const s16x4*>(rows + ((col < LC ? col >> 2 : 0) * A.ldn + qc) * 4);
      }
#pragma unroll
    for (int i = 0; i < 3; ++i) sd[i] = A.seeds[3 * qc + i];
    if (K0 > LC) src_q = A.order[qc];
  };
  const int64_t n_tiles = (A.Q + 16 * NW - 1) / (16 * NW);
  const TileRange rng = xcd_tiles(n_tiles, 1, 0);
  if (rng.first < rng.end) load(rng.first);
  for (int64_t tile = rng.first; tile < rng.end; tile += rng.stride) {
    // lane-derived addresses are loop-invariant: recomputed per tile rather
    // than held in registers across the loop
    const int lane = launder_lane(threadIdx.x) & 63, g = lane >> 4, r16 = lane & 15, tr = tr_offset(lane);
    const int64_t q = tile * 16 * NW + wave * 16 + r16;
    const bool valid = q < A.Q;
    // ---- 1. this tile's inputs into LDS, the next one's on their way ------
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      if (kb < KB0)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const s16x4 zero = {0, 0, 0, 0};
          const bool in = valid && 32 * kb + 16 * hf + 4 * g < LC;
          *reinterpret_cast<s16x4*>(A0w + (kb * 2 + hf) * kPlane + 4 * lane) = in ? raw[kb][hf] : zero;
        }
    if (valid && src_q >= 0 && src_q < A.n_src) {  // surface attributes, in the caller's query order
      const int E = K0 - LC;
      const float* const gp = src_q < A.nA ? A.gA + (int64_t)E * src_q : A.gB + E * (src_q - A.nA);
      for (int k = 4 * g; k < E; k += 16) {
        typedef MT v4 __attribute__((ext_vector_type(4)));
        const int col = LC + k;
        v4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = from_f32<MT>(gp[k + j]);
        *reinterpret_cast<s16x4*>(A0w + (col >> 4) * kPlane + 4 * ((col & 12) * 4 + r16)) = __builtin_bit_cast(s16x4, v);
      }
    }
    frag sf;  // seeds of the output layer, rows 0 .. 2
#pragma unroll
    for (int i = 0; i < 8; ++i) sf[i] = from_f32<MT>(i < 3 && g == 0 && valid ? sd[i < 3 ? i : 0] : 0.0f);
    if (tile + rng.stride < rng.end) load(tile + rng.stride);
    wave_lds_sync();

    // ---- 2. hidden layers ---------------------------------------------------
    // acc[m] = sum over chunks kb < KB of read(kb, m) b(kb), from c_in(m).
    // Four row tiles a step, the next step's operand reads in flight while
    // this step's products run.
    f32x4 acc[MH];
    auto products = [&](auto kbs, auto&& read, auto&& b, auto&& c_in) {
      constexpr int KB = decltype(kbs)::value, S = KB * (MH / 4);
      frag a[2][4];
#pragma unroll
      for (int m = 0; m < 4; ++m) a[0][m] = read(0, m);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int kb = s / (MH / 4), m0 = s % (MH / 4) * 4;
        if (s + 1 < S) {
          const int kb1 = (s + 1) / (MH / 4), m1 = (s + 1) % (MH / 4) * 4;
#pragma unroll
          for (int m = 0; m < 4; ++m) a[(s + 1) & 1][m] = read(kb1, m1 + m);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m0 + m] = mma(a[s & 1][m], b(kb), kb == 0 ? c_in(m0 + m) : acc[m0 + m]);
      }
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, KH> Hid;
    frag act[NHH + 1][KH];  // ReLU'd outputs of the hidden layers, as operands
    for (int kb = 0; kb < KB0; ++kb) {
      const frag b = plane_frag<MT>(A0w + kb * kFrag, lane);
      products(One{}, [&](int, int m) { return plane_frag<MT>(wl + (m * KB0 + kb) * kFrag, lane); },
               [&](int) { return b; }, [&](int m) { return kb == 0 ? bias_tile(bias, m, lane) : acc[m]; });
    }
#pragma unroll
    for (int kb = 0; kb < KH; ++kb) act[0][kb] = chain_frag<MT>(acc[2 * kb], acc[2 * kb + 1], true);
#pragma unroll
    for (int hh = 0; hh < NHH; ++hh) {
      const MT* Wh = layer_w(hh);
      products(Hid{}, [&](int kb, int m) { return plane_frag<MT>(Wh + (m * KH + kb) * kFrag, lane); },
               [&](int kb) { return act[hh][kb]; }, [&](int m) { return bias_tile(bias + (hh + 1) * H, m, lane); });
#pragma unroll
      for (int kb = 0; kb < KH; ++kb) act[hh + 1][kb] = chain_frag<MT>(acc[2 * kb], acc[2 * kb + 1], true);
    }

    // ---- 3. backward --------------------------------------------------------
    // operand rows 16 m .. + 15 over the queries of wave tiles 2 c and 2 c + 1
    // of a buffer with K chunks per wave tile
    auto queries_frag = [&](const MT* buf, int K, int c, int m) {
      const MT* p = buf + (2 * c * K * 2 + m) * kPlane;
      return join<MT>(tr_plane<MT>(p, tr), tr_plane<MT>(p + K * kFrag, tr));
    };
    // this wave's dW block and db rows of a layer with H outputs: deltas in X
    // (wave tiles c0 .. c0 + nput / 2 - 1 pairs), activations in buf
    auto contract = [&](auto& accw, f32x4 (&db)[RB], const MT* buf, int K, int ncols) {
      constexpr int CBn = sizeof(accw[0]) / sizeof(f32x4);
      for (int c = 0; c < nput / 2; ++c) {
        frag a[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) a[rb] = queries_frag(X, KH, c, row0 + rb);
#pragma unroll
        for (int cb = 0; cb < CBn; ++cb)
          if (cset * CBn + cb < ncols) {
            const frag b = queries_frag(buf, K, c, cset * CBn + cb);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) accw[rb][cb] = mma(a[rb], b, accw[rb][cb]);
          }
        if (cset == 0)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) db[rb] = mma(a[rb], ones, db[rb]);
      }
    };
    // delta of a layer's input (operands df) from acc = W^T delta: ReLU'(z)
    // = 1 where the activation is positive
    frag df[KH];
    auto mask = [&](const frag (&a)[KH]) {
#pragma unroll
      for (int kb = 0; kb < KH; ++kb) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (!(to_f32(a[kb][i]) > 0.0f)) acc[2 * kb + (i >> 2)][i & 3] = 0.0f;
        df[kb] = chain_frag<MT>(acc[2 * kb], acc[2 * kb + 1], false);
      }
    };
    const MT* const Xw = X, *const Yw = Y;
    // Exchange of one layer's deltas xs (nx chunks) and activations ys: the
    // waves put theirs in nput at a time, and use(t0) reads all of them.
    auto exchange = [&](auto& xs, auto* ys, auto&& use) {
      constexpr int nx = sizeof(xs) / sizeof(frag);
      for (int t0 = 0; t0 < NW; t0 += nput) {
        if (wave >= t0 && wave < t0 + nput) {
          MT* const xw = const_cast<MT*>(Xw) + (wave - t0) * KH * kFrag;
          MT* const yw = const_cast<MT*>(Yw) + (wave - t0) * KH * kFrag;
#pragma unroll
          for (int kb = 0; kb < nx; ++kb) put_planes<MT>(xw + kb * kFrag, lane, xs[kb]);
          if constexpr (!std::is_same<decltype(ys), const int*>::value)
#pragma unroll
            for (int kb = 0; kb < KH; ++kb) put_planes<MT>(yw + kb * kFrag, lane, (*ys)[kb]);
        }
        __syncthreads();
        use(t0);
        __syncthreads();  // every wave has read the buffers
      }
    };
    // output layer
    frag sfa[1] = {sf};
    exchange(sfa, &act[NHH], [&](int) {
      for (int c = 0; c < nput / 2; ++c) {
        const frag a = queries_frag(X, KH, c, 0);
#pragma unroll
        for (int u = 0; u < UO; ++u)
          if (wave + NW * u < MH) accO[u] = mma(a, queries_frag(Y, KH, c, wave + NW * u), accO[u]);
        if (wave == 0) dbO = mma(a, ones, dbO);
      }
    });
    {
      const MT* Wo = layer_w(NHH);
      const s16x4 zero = {0, 0, 0, 0};
      products(One{}, [&](int, int m) { return join<MT>(tr_plane<MT>(Wo + m * kPlane, tr), zero); },
               [&](int) { return sf; }, [&](int) { return z4; });
      mask(act[NHH]);
    }
#pragma unroll
    for (int hh = NHH - 1; hh >= 0; --hh) {
      exchange(df, &act[hh], [&](int) { contract(accH[hh], dbH[hh], Y, KH, MH); });
      // acc = W^T df, from the forward's fragments
      const MT* Wh = layer_w(hh);
      products(Hid{},
               [&](int kb, int m) {
                 const MT* p = Wh + (2 * kb * KH * 2 + m) * kPlane;
                 return join<MT>(tr_plane<MT>(p, tr), tr_plane<MT>(p + KH * kFrag, tr));
               },
               [&](int kb) { return df[kb]; }, [&](int) { return z4; });
      mask(act[hh]);
    }
    exchange(df, (const int*)nullptr, [&](int t0) { contract(acc0, db0, A0 + t0 * KB0 * kFrag, KB0, NK0); });
    {
      // dh = W_0^T delta over the level-feature rows only: the surface
      // attributes are inputs, not parameters
      const int MK = (LC + 15) / 16;
#pragma unroll 2
      for (int m = 0; m < MK; ++m) {
        f32x4 d = z4;
#pragma unroll
        for (int kb = 0; kb < KH; ++kb) {
          const MT* p = wl + (2 * kb * KB0 * 2 + m) * kPlane;
          d = mma(join<MT>(tr_plane<MT>(p, tr), tr_plane<MT>(p + KB0 * kFrag, tr)), df[kb], d);
        }
        const int k = 16 * m + 4 * g;
        if (valid && k < LC) *reinterpret_cast<float4*>(A.dh + q * LC + k) = make_float4(d[0], d[1], d[2], d[3]);
      }
    }
  }

  const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  each_tile([&](f32x4& acc, int n_out, int n_in, int64_t off, int mm, int nk) {
    const int k = n_in == 1 ? r16 : 16 * nk + r16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = 16 * mm + 4 * g + j;
      if (n < n_out && k < n_in) part[off + n * n_in + k] = acc[j];
    }
  });
}

template <class MT, int H>
static hipError_t launch_bwd16_t(const MlpArgs& M, int LC, const BwdArgs& A, const ParamLayout& PL, int grid,
                                 hipStream_t st) {
  const Bwd16Shape s = bwd16_shape(M);
  constexpr int NWD = H == 128 ? 4 : 8;  // three or four hidden layers
  auto k = M.n_layers == 2   ? bwd16_kernel<MT, H, 8, 0>
           : M.n_layers == 3 ? bwd16_kernel<MT, H, 8, 1>
           : M.n_layers == 4 ? bwd16_kernel<MT, H, NWD, 2>
                             : bwd16_kernel<MT, H, NWD, 3>;
  allow_lds((const void*)k, s.lds);
  hipLaunchKernelGGL(k, dim3(grid), dim3(64 * s.waves), s.lds, st, M, LC, A, PL, s.nput);
  return hipGetLastError();
}

hipError_t launch_bwd16(const MlpArgs& M, oo_dtype md, int LC, const BwdArgs& A, const ParamLayout& PL, int grid,
                        hipStream_t st) {
  if (md == OO_F16)
    return M.H == 64 ? launch_bwd16_t<f16, 64>(M, LC, A, PL, grid, st) : launch_bwd16_t<f16, 128>(M, LC, A, PL, grid, st);
  return M.H == 64 ? launch_bwd16_t<bf16, 64>(M, LC, A, PL, grid, st) : launch_bwd16_t<bf16, 128>(M, LC, A, PL, grid, st);
}

}  // namespace oo
