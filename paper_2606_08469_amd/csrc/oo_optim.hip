// Optimiser step over the FP32 masters (Adam, lazy over feature-map blocks
// no query read, fused with the working-copy refresh and the gradient
// clear), and the marking of the nodes a residual batch read.
#include <hip/hip_runtime.h>

#include "oo_device.h"
#include "oo_internal.h"

namespace oo {

// Four elements per thread ("quads") over the concatenated segments: segment
// s owns the quads [first[s], first[s + 1]). A quad reads the block flag of
// its first element; blocks are whole multiples of 4 elements (every table
// block is res^2 C or (res+1)^2 C with C in {4, 8}), so the four elements
// share it. The last quad of a segment may hold fewer than four elements.
// Segments whose arrays are all 16-byte aligned (8-byte for a 16-bit working
// copy) move each array as one vector per quad.
__device__ inline float adam_update(const AdamArgs& A, float& p, float& m, float& v, float g) {
  m = A.b1 * m + (1.0f - A.b1) * g;
  v = A.b2 * v + (1.0f - A.b2) * g * g;
  p = p - A.lr * (m * A.inv_c1) / (sqrtf(v * A.inv_c2) + A.eps);
  return p;
}

// Any quad of any segment.
template <class WT>
__device__ inline void adam_quad(const AdamArgs& A, int64_t tq) {
  int s = 0;
  while (s + 1 < A.n_segs && tq >= A.first[s + 1]) ++s;
  const AdamSeg& S = A.seg[s];
  const int64_t i0 = (tq - A.first[s]) * 4;
  if (S.touched && !S.touched[i0 / S.block]) return;
  for (int64_t i = i0; i < i0 + 4 && i < S.n; ++i) {
    float p = S.param[i], m = S.m[i], v = S.v[i];
    adam_update(A, p, m, v, S.grad[i]);
    S.m[i] = m;
    S.v[i] = v;
    S.param[i] = p;
    S.grad[i] = 0.0f;
    if (S.work) reinterpret_cast<WT*>(S.work)[i] = from_f32<WT>(p);
  }
}

// Bound by memory: 34 bytes move per updated element with a 16-bit working
// copy. The masters, moments and gradients are as good as gone from the
// caches when they are next read, so their loads and stores bypass them, and
// each workgroup takes 256 quads and ends instead of looping. 262 million
// elements (8.9 GB) take 1.61 ms, 5.5 TB/s. With one quad per thread: 1571 us
// (1679 if the working copy is stored through the caches); without the cache
// bypass 1761, looping over 16,384 workgroups 1868, neither (and a search of
// the segments and a 64-bit division per thread) 2112.
// A workgroup has two waves, each thread two quads one after the other: where
// few maps were read, the time goes to starting waves that find nothing to do
// (the same elements, a thousandth of them read: 156 us; with four waves of
// one quad per thread 271, a tenth read 225 and 305, all of them 1709 and
// 1703; with four quads per thread 97, 213 and 1739 to 1826).
constexpr int kAdamThreads = 128, kAdamQuads = 2;
template <class WT>
__global__ __launch_bounds__(kAdamThreads) void adam_kernel(const AdamArgs A) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef WT w4 __attribute__((ext_vector_type(4)));
  const int64_t total = A.first[A.n_segs];
  constexpr int per = kAdamThreads * kAdamQuads;
  for (int64_t base = (int64_t)blockIdx.x * per; base < total; base += (int64_t)gridDim.x * per) {
    int s = 0;
    while (s + 1 < A.n_segs && base >= A.first[s + 1]) ++s;
    const AdamSeg& S = A.seg[s];
    const int64_t q0 = base - A.first[s];
    if (!S.vec || (q0 + per) * 4 > S.n) {  // several segments, a short quad or unaligned arrays
      for (int64_t q = base + threadIdx.x; q < base + per && q < total; q += kAdamThreads) adam_quad<WT>(A, q);
      continue;
    }
    uint32_t go[kAdamQuads];
#pragma unroll
    for (int u = 0; u < kAdamQuads; ++u) {
      const int64_t i0 = (q0 + kAdamThreads * u + threadIdx.x) * 4;
      go[u] = S.touched ? S.touched[S.shift >= 0 ? i0 >> S.shift : i0 / S.block] : 1u;
    }
#pragma unroll
    for (int u = 0; u < kAdamQuads; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      if (!go[u]) continue;
      const int64_t i0 = (q0 + kAdamThreads * u + threadIdx.x) * 4;
      f4* const pp = reinterpret_cast<f4*>(S.param + i0);
      f4* const mp = reinterpret_cast<f4*>(S.m + i0);
      f4* const vp = reinterpret_cast<f4*>(S.v + i0);
      f4* const gp = reinterpret_cast<f4*>(S.grad + i0);
      const f4 p0 = __builtin_nontemporal_load(pp), m0 = __builtin_nontemporal_load(mp);
      const f4 v0 = __builtin_nontemporal_load(vp), g = __builtin_nontemporal_load(gp);
      f4 p, m, v;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float pj = p0[j], mj = m0[j], vj = v0[j];
        adam_update(A, pj, mj, vj, g[j]);
        p[j] = pj;
        m[j] = mj;
        v[j] = vj;
      }
      __builtin_nontemporal_store(p, pp);
      __builtin_nontemporal_store(m, mp);
      __builtin_nontemporal_store(v, vp);
      __builtin_nontemporal_store(f4{0.f, 0.f, 0.f, 0.f}, gp);
      if (S.work) {
        w4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = from_f32<WT>(p[j]);
        __builtin_nontemporal_store(w, reinterpret_cast<w4*>(reinterpret_cast<WT*>(S.work) + i0));
      }
    }
  }
}

hipError_t launch_adam(const AdamArgs& A, oo_dtype wd, hipStream_t st) {
  const int64_t total = A.first[A.n_segs];
  if (total == 0) return hipSuccess;
  constexpr int per = kAdamThreads * kAdamQuads;
  int64_t blocks = (total + per - 1) / per;
  if (blocks > 1 << 22) blocks = 1 << 22;  // (2^32 elements; more loop)
  if (wd == OO_F16)
    hipLaunchKernelGGL(adam_kernel<f16>, dim3((unsigned)blocks), dim3(kAdamThreads), 0, st, A);
  else if (wd == OO_BF16)
    hipLaunchKernelGGL(adam_kernel<bf16>, dim3((unsigned)blocks), dim3(kAdamThreads), 0, st, A);
  else
    hipLaunchKernelGGL(adam_kernel<float>, dim3((unsigned)blocks), dim3(kAdamThreads), 0, st, A);
  return hipGetLastError();
}

// touched[node] = 1 for every stored node index of the n backward queries
// ([rows][n], rows = levels x corners) that lies in [0, n_nodes).
__global__ __launch_bounds__(256) void touched_kernel(const int32_t* __restrict__ nidx, int64_t n, int64_t rows,
                                                      int64_t n_nodes, uint32_t* __restrict__ touched) {
  const int64_t total = n * rows, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
    const int32_t v = nidx[e];
    if (v >= 0 && v < n_nodes) touched[v] = 1u;
  }
}

hipError_t launch_touched(const int32_t* nidx, int64_t n, int64_t rows, int64_t n_nodes, uint32_t* touched,
                          hipStream_t st) {
  const int64_t total = n * rows;
  if (total == 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 256 * 64) blocks = 256 * 64;
  hipLaunchKernelGGL(touched_kernel, dim3((unsigned)blocks), dim3(256), 0, st, nidx, n, rows, n_nodes, touched);
  return hipGetLastError();
}

}  // namespace oo
