// Forward kernels: standalone encoding, the fused encode + decode query, the residual assembly with its FP64 loss
// reduction, and the FP32 -> FP16/BF16 parameter cast.
#include <hip/hip_runtime.h>

#include "oo_device.h"
#include "oo_internal.h"
#include "oo_mlp.h"

namespace oo {

// ---------------------------------------------------------------------------
// Standalone encoding: one thread per query, h written row-major to memory.
// ---------------------------------------------------------------------------
// MODE: 0 node + bilinear, 1 the paper's scheme, 2 the paper's scheme with
// the disparity shift (FP32 features; the first entry of each row holds the
// query's disparity when the kernel starts, see launch_predict).
template <class TT, class HT, int C, int MODE>
__global__ __launch_bounds__(256) void encode_kernel(const TreeArgs T, const float* __restrict__ x,
                                                     const float* __restrict__ dir, int64_t B,
                                                     HT* __restrict__ h_out, int32_t* __restrict__ idx_out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = q < B;
  float xq[3] = {0.f, 0.f, 0.f}, dq[3] = {0.f, 0.f, 1.f};
  if (valid) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      xq[a] = x[3 * q + a];
      dq[a] = dir[3 * q + a];
    }
  }
  typedef HT vC __attribute__((ext_vector_type(C)));
  if constexpr (MODE > 0) {
    // the eight cells around x per level, barycentric vertex maps
    float s, t;
    octa(dq, s, t);
    float u[3] = {0.f, 0.f, 0.f}, disp = 0.0f;
    if constexpr (MODE == 2) {
      unit_dir3(dq, u);
      if (valid) disp = to_f32(h_out[q * (int64_t)(T.L * C)]);
    }
    const int L = T.L;
    HT* hrow = h_out + (valid ? q : 0) * (int64_t)(L * C);
    encode_paper<TT, C, MODE == 2>(T, valid, xq, s, t, [&](int l, const float* h, const int (&node)[8], auto&) {
      if (!valid) return;
      vC v;
#pragma unroll
      for (int c = 0; c < C; ++c) v[c] = from_f32<HT>(h[c]);
      *reinterpret_cast<vC*>(hrow + l * C) = v;
      if (idx_out) {
        int4* o = reinterpret_cast<int4*>(idx_out + (q * L + l) * 8);
        o[0] = make_int4(node[0], node[1], node[2], node[3]);
        o[1] = make_int4(node[4], node[5], node[6], node[7]);
      }
    }, disp, u);
    return;
  }
  int idx[kMaxLevels];
  descend(T, valid, xq, idx);
  if (!valid) return;
  float s, t;
  octa(dq, s, t);
  const int L = T.L;
  HT* hrow = h_out + q * (int64_t)(L * C);
#pragma unroll
  for (int l0 = 0; l0 < kMaxLevels; l0 += 4) {
    if (l0 >= L) break;
    float h[4][C];
    gather_levels<TT, C, 4>(T, l0, &idx[l0], s, t, h);
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) {
      const int l = l0 + gi;
      if (l < L) {
        vC v;
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = from_f32<HT>(h[gi][c]);
        *reinterpret_cast<vC*>(hrow + l * C) = v;
        if (idx_out) idx_out[q * L + l] = idx[l];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Shifted encode of the residual's sorted queries into decoder input rows:
// one thread per query (the paper's scheme with the disparity shift, each
// query's disparity read from O.disp). Row q of h_rows (K0 = L C + E
// entries of MT) holds the level features, then the surface attributes;
// queries q < n_idx also leave what the backward reads (corner nodes,
// octahedral coordinates, position and disparity, lookup direction), as
// the fused query does. Without the decoder's registers the encode runs at
// several more waves per SIMD, which its dependent gathers need; the
// standalone decoder then reads the rows.
// ---------------------------------------------------------------------------
template <class TT, class MT, int C>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(C == 4 ? 4 : 3))) void encode_rows_kernel(const TreeArgs T, const QuerySrc src, int64_t Q, int K0,
                                                          int E, MT* __restrict__ h_rows, const QueryOut O) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = q < Q;
  float x[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
  if (valid) load_query(src, q, x, d);
  float s, t;
  octa(d, s, t);
  float u[3];
  unit_dir3(d, u);
  const float disp = valid ? O.disp[q] : 0.0f;
  const bool keep = q < O.n_idx;
  if (keep) {
    O.uv[q] = make_float2(s, t);
    O.wdir[q] = make_float4(u[0], u[1], u[2], 0.0f);
    O.pos[q] = make_float4(x[0], x[1], x[2], disp);
  }
  typedef MT vC __attribute__((ext_vector_type(C)));
  MT* const row = h_rows + (valid ? q : 0) * (int64_t)K0;
  MT* const brow = keep ? reinterpret_cast<MT*>(O.rows) : nullptr;
  typedef MT v4 __attribute__((ext_vector_type(4)));
  encode_paper<TT, C, true>(T, valid, x, s, t, [&](int l, const float* h, const int (&node)[8], auto& last) {
    if (valid) {
      vC v;
#pragma unroll
      for (int c = 0; c < C; ++c) v[c] = from_f32<MT>(h[c]);
      *reinterpret_cast<vC*>(row + l * C) = v;
    }
    if (keep)
#pragma unroll
      for (int dd = 0; dd < 8; ++dd) O.idx[(l * 8 + dd) * O.n_idx + q] = node[dd];  // coalesced across lanes
    if constexpr (sizeof(MT) == 2)
      if (brow)
#pragma unroll
        for (int c = 0; c < C; c += 4)
          *reinterpret_cast<v4*>(brow + (((l * C + c) >> 2) * O.n_idx + q) * 4) = last.round4(c);
  }, disp, u);
  if (!valid) return;
  for (int k = 0; k < E; k += 4) {
    float g4[4];
    load_attr4(src, q, k, g4);
    v4 v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = from_f32<MT>(g4[c]);
    *reinterpret_cast<v4*>(row + K0 - E + k) = v;
  }
}

// ---------------------------------------------------------------------------
// Residual assembly (rendering-equation RHS) and loss partials.
// ---------------------------------------------------------------------------

// One group of G lanes per LHS point (G = N rounded up to a power of two,
// at most 64): lane k of the group weighs secondary sample k (and k + G, ...)
// so the per-sample inputs are read coalesced; the group sums its products
// with lane shuffles in a fixed order. The group leader forms
// T = Le + (1/N) sum_k w_k * L(x2_k) and r = L - T and writes the outputs;
// each block leaves one FP64 partial of sum r^2 (or (r / rho)^2).
__global__ __launch_bounds__(256) void combine_kernel(const ResidualArgs A, int G, const float* __restrict__ Lq,
                                                      const int32_t* __restrict__ rank, float* __restrict__ lhs_out, float* __restrict__ rhs_out,
                                                      float* __restrict__ resid_out, double* __restrict__ partials) {
  __shared__ double red[4];
  const int64_t gid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  const int64_t b = gid / G;
  const int k0 = (int)(gid % G);
  const bool valid = b < A.B;
  float s[3] = {0.f, 0.f, 0.f};
  if (valid && !A.target_override && A.N > 0) {
    float n[3], wo[3], alb[3] = {A.albedo[3 * b], A.albedo[3 * b + 1], A.albedo[3 * b + 2]};
    load_unit(A.n + 3 * b, n);
    load_unit(A.wo + 3 * b, wo);
    const float alpha = A.rough[b];
    for (int k = k0; k < A.N; k += G) {
      const int64_t bk = b * A.N + k;
      float wi[3], w[3];
      load_unit(A.wi + 3 * bk, wi);
      bsdf_weight(n, wo, wi, alb, alpha, A.F0, A.pdf ? A.pdf[bk] : 1.0f, w);
      const int64_t qk = A.B + bk;
      const float* Lk = Lq + 3 * (rank ? (int64_t)rank[qk] : qk);
#pragma unroll
      for (int c = 0; c < 3; ++c) s[c] += w[c] * Lk[c];
    }
  }
  for (int off = G >> 1; off > 0; off >>= 1)
#pragma unroll
    for (int c = 0; c < 3; ++c) s[c] += __shfl_xor(s[c], off, G);
  double acc = 0.0;
  if (valid && k0 == 0) {
    const float* Lb = Lq + 3 * (rank ? (int64_t)rank[b] : b);
    float L[3] = {Lb[0], Lb[1], Lb[2]};
    float T[3];
    if (A.target_override) {
#pragma unroll
      for (int c = 0; c < 3; ++c) T[c] = A.target_override[3 * b + c];
    } else {
      const float invN = A.N > 0 ? 1.0f / (float)A.N : 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) T[c] = A.Le[3 * b + c] + s[c] * invN;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float r = L[c] - T[c];
      lhs_out[3 * b + c] = L[c];
      rhs_out[3 * b + c] = T[c];
      resid_out[3 * b + c] = r;
      double rr = (double)r;
      if (A.loss_kind == 1) {
        const double rho = fmax((double)L[c] + (double)T[c], 0.0) + (double)A.eps;
        rr /= rho;
      }
      acc += rr * rr;
    }
  }
  // fixed order: within each wave by shuffles, then the four waves in turn
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Fixed-order sum of the block partials: loss = sum / (3B). One workgroup, so
// a chain of latencies: 32,768 partials take 10 us with 16 in flight per
// thread, 34 one by one.
__global__ __launch_bounds__(256) void loss_reduce_kernel(const double* __restrict__ partials, int n, int64_t B,
                                                          double* __restrict__ loss) {
  __shared__ double red[256];
  double acc = 0.0;
  constexpr int U = 16;  // partials in flight per thread, added in the plain loop's order
  for (int i0 = threadIdx.x; i0 < n; i0 += 256 * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i0 + 256 * u < n ? partials[i0 + 256 * u] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = B > 0 ? red[0] / (3.0 * (double)B) : 0.0;
}

// Eight elements per thread and iteration (two 16-byte loads, one store of
// 8 x sizeof(DT) bytes) when both pointers allow it, both loads issued before
// either is converted; the tail and unaligned arrays go element by element.
template <class DT>
__global__ __launch_bounds__(256) void cast_kernel(const float* __restrict__ src, DT* __restrict__ dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t nv = 0;
  if ((reinterpret_cast<uintptr_t>(src) % 16) == 0 && (reinterpret_cast<uintptr_t>(dst) % (8 * sizeof(DT))) == 0) {
    nv = n / 8;
    typedef DT v8 __attribute__((ext_vector_type(8)));
    for (int64_t i = i0; i < nv; i += stride) {
      // streamed once: non-temporal loads and stores keep the masters and
      // the working copy from displacing cached data
      typedef float f4 __attribute__((ext_vector_type(4)));
      const f4 a = __builtin_nontemporal_load(reinterpret_cast<const f4*>(src) + 2 * i);
      const f4 b = __builtin_nontemporal_load(reinterpret_cast<const f4*>(src) + 2 * i + 1);
      v8 o;
      o[0] = from_f32<DT>(a.x);
      o[1] = from_f32<DT>(a.y);
      o[2] = from_f32<DT>(a.z);
      o[3] = from_f32<DT>(a.w);
      o[4] = from_f32<DT>(b.x);
      o[5] = from_f32<DT>(b.y);
      o[6] = from_f32<DT>(b.z);
      o[7] = from_f32<DT>(b.w);
      __builtin_nontemporal_store(o, reinterpret_cast<v8*>(dst) + i);
    }
  }
  for (int64_t i = 8 * nv + i0; i < n; i += stride) dst[i] = from_f32<DT>(src[i]);
}

// Node indices the residual forward stored for its backward queries
// ([L][Qb], sorted positions), returned per source query ([Qb][L]). Sorted
// position p holds source query order[p]; a value outside [0, Qb) is skipped.
// With K = 8 (the paper's scheme) each level holds the eight corners:
// [L][8][Qb] in, [Qb][L][8] out.
__global__ __launch_bounds__(256) void saved_nodes_kernel(const int32_t* __restrict__ nidx,
                                                          const int32_t* __restrict__ order, int64_t Qb, int L, int K,
                                                          int32_t* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= Qb) return;
  const int64_t q = order[p];
  if (q < 0 || q >= Qb) return;
  for (int l = 0; l < L; ++l)
    for (int k = 0; k < K; ++k) out[(q * L + l) * K + k] = nidx[((int64_t)l * K + k) * Qb + p];
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

template <class TT, class HT, int C>
static hipError_t launch_encode_t(const TreeArgs& T, const float* x, const float* d, int64_t B, void* h,
                                  int32_t* idx, const DispArgs& G, hipStream_t st) {
  const int64_t blocks = (B + 255) / 256;
  HT* hp = reinterpret_cast<HT*>(h);
  if (T.interp != OO_INTERP_PAPER)
    hipLaunchKernelGGL((encode_kernel<TT, HT, C, 0>), dim3((unsigned)blocks), dim3(256), 0, st, T, x, d, B, hp, idx);
  else if (G.n_levels == 0)
    hipLaunchKernelGGL((encode_kernel<TT, HT, C, 1>), dim3((unsigned)blocks), dim3(256), 0, st, T, x, d, B, hp, idx);
  else if constexpr (sizeof(HT) == 4) {  // the shifted encoding writes FP32 features only
    const hipError_t e = launch_predict(G, QuerySrc{x, d, B, x, d}, B, hp, (int64_t)T.L * C, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((encode_kernel<TT, HT, C, 2>), dim3((unsigned)blocks), dim3(256), 0, st, T, x, d, B, hp, idx);
  } else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <class TT, int C>
static hipError_t launch_encode_h(const TreeArgs& T, const float* x, const float* d, int64_t B, void* h,
                                  oo_dtype hd, int32_t* idx, const DispArgs& G, hipStream_t st) {
  switch (hd) {
    case OO_F32: return launch_encode_t<TT, float, C>(T, x, d, B, h, idx, G, st);
    case OO_F16: return launch_encode_t<TT, f16, C>(T, x, d, B, h, idx, G, st);
    default: return launch_encode_t<TT, bf16, C>(T, x, d, B, h, idx, G, st);
  }
}

hipError_t launch_encode(const TreeArgs& T, oo_dtype td, const float* x, const float* d, int64_t B, void* h,
                         oo_dtype hd, int32_t* idx, const DispArgs& G, hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (td == OO_F32)
    return T.C == 4 ? launch_encode_h<float, 4>(T, x, d, B, h, hd, idx, G, st)
                    : launch_encode_h<float, 8>(T, x, d, B, h, hd, idx, G, st);
  if (td == OO_F16)
    return T.C == 4 ? launch_encode_h<f16, 4>(T, x, d, B, h, hd, idx, G, st)
                    : launch_encode_h<f16, 8>(T, x, d, B, h, hd, idx, G, st);
  return T.C == 4 ? launch_encode_h<bf16, 4>(T, x, d, B, h, hd, idx, G, st)
                  : launch_encode_h<bf16, 8>(T, x, d, B, h, hd, idx, G, st);
}

static int combine_group(int N) {
  int G = 1;
  while (G < N && G < 64) G <<= 1;
  return G;
}

int combine_blocks(int64_t B, int N) { return (int)((B * combine_group(N) + 255) / 256); }

hipError_t launch_combine(const ResidualArgs& A, const float* Lq, const int32_t* rank, float* lhs, float* rhs,
                          float* resid, double* partials, double* loss, hipStream_t st) {
  const int G = combine_group(A.target_override ? 0 : A.N);
  const int nb = combine_blocks(A.B, A.target_override ? 0 : A.N);
  if (nb > 0)
    hipLaunchKernelGGL(combine_kernel, dim3(nb), dim3(256), 0, st, A, G, Lq, rank, lhs, rhs, resid, partials);
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, st, partials, nb, A.B, loss);
  return hipGetLastError();
}

hipError_t launch_saved_nodes(const int32_t* nidx, const int32_t* order, int64_t Qb, int L, int K, int32_t* out,
                              hipStream_t st) {
  if (Qb == 0) return hipSuccess;
  hipLaunchKernelGGL(saved_nodes_kernel, dim3((unsigned)((Qb + 255) / 256)), dim3(256), 0, st, nidx, order, Qb, L,
                     K, out);
  return hipGetLastError();
}

hipError_t launch_cast(const float* src, void* dst, oo_dtype dt, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  // one 8-element vector per thread (measured faster than a smaller grid
  // striding over the array); arrays beyond 2^33 elements stride
  int64_t blocks = (n / 8 + 255) / 256;
  if (blocks > (1 << 22)) blocks = 1 << 22;
  if (blocks < 1) blocks = 1;
  if (dt == OO_F32)
    hipLaunchKernelGGL(cast_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, src, (float*)dst, n);
  else if (dt == OO_F16)
    hipLaunchKernelGGL(cast_kernel<f16>, dim3((unsigned)blocks), dim3(256), 0, st, src, (f16*)dst, n);
  else
    hipLaunchKernelGGL(cast_kernel<bf16>, dim3((unsigned)blocks), dim3(256), 0, st, src, (bf16*)dst, n);
  return hipGetLastError();
}

template <class TT, class MT, int C>
static void launch_encode_rows_t(const TreeArgs& T, const QuerySrc& src, int64_t Q, int K0, int E, void* h_rows,
                                 const QueryOut& O, hipStream_t st) {
  hipLaunchKernelGGL((encode_rows_kernel<TT, MT, C>), dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, st, T, src, Q,
                     K0, E, reinterpret_cast<MT*>(h_rows), O);
}

hipError_t launch_encode_rows(const TreeArgs& T, oo_dtype td, const MlpArgs& M, const QuerySrc& src, int64_t Q,
                              void* h_rows, const QueryOut& O, hipStream_t st) {
  if (Q == 0) return hipSuccess;
  // the tables and the decoder share one dtype in the product paths
  if (td == OO_F32)
    T.C == 4 ? launch_encode_rows_t<float, float, 4>(T, src, Q, M.K0, M.E, h_rows, O, st)
             : launch_encode_rows_t<float, float, 8>(T, src, Q, M.K0, M.E, h_rows, O, st);
  else if (td == OO_F16)
    T.C == 4 ? launch_encode_rows_t<f16, f16, 4>(T, src, Q, M.K0, M.E, h_rows, O, st)
             : launch_encode_rows_t<f16, f16, 8>(T, src, Q, M.K0, M.E, h_rows, O, st);
  else
    T.C == 4 ? launch_encode_rows_t<bf16, bf16, 4>(T, src, Q, M.K0, M.E, h_rows, O, st)
             : launch_encode_rows_t<bf16, bf16, 8>(T, src, Q, M.K0, M.E, h_rows, O, st);
  return hipGetLastError();
}

}  // namespace oo
