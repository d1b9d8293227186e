// Standalone decoder (oo_mlp_fwd, and the residual's decoder over the shifted
// encode's rows).
#include <hip/hip_runtime.h>

#include "oo_mlp.h"

namespace oo {

// ---------------------------------------------------------------------------
// Standalone decoder: every wave decodes 16 NT rows of h at a time.
//
// A lane's share of a first-layer operand chunk is two runs of four
// consecutive inputs of one row, so the operands come straight from memory
// as 4-element loads (a 16-row, 32-byte-wide block per instruction; the two
// runs of a chunk share their 64-byte sectors). No activation tile is kept
// in LDS: the weights and biases are all it holds, so eight waves fit beside
// the 119 KB of a 48-128-128-128-128-3 decoder too (five with a tile each).
// Bound by MFMA issue and the conversions between layers (two waves per SIMD
// overlap one tile's loads with the other's products): 2^20 rows of
// 88-128-128-3 in FP16 take 64 us (88 with tiles staged through LDS), 0.92
// PFLOP/s.
// ---------------------------------------------------------------------------
template <class MT, bool WLDS>
__host__ __device__ constexpr int mlp_ntiles() {
  // with 16-bit operands and the weights in LDS each weight fragment read
  // serves four MFMAs (the other variants would spill)
  return sizeof(MT) == 2 && WLDS ? 4 : 2;
}

template <class MT, int H, int KB0, bool WLDS>
__global__ __launch_bounds__(512) void mlp_kernel(const MlpArgs M, const MT* __restrict__ h, int64_t Q,
                                                  float* __restrict__ rgb) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef typename FragT<MT>::type frag;
  typedef uint32_t raw __attribute__((ext_vector_type(sizeof(MT))));  // four inputs
  constexpr int NT = mlp_ntiles<MT, WLDS>();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  float* const bias = reinterpret_cast<float*>(smem);
  MT* wl = reinterpret_cast<MT*>(bias + bias_floats(M.n_layers, H));
  load_biases_lds(M, bias);
  if (WLDS) pack_weights_lds<MT>(M, wl);
  __syncthreads();
  const WFrag<MT, WLDS> W{wl, KB0};
  const TileRange tr = xcd_tiles((Q + 16 * NT - 1) / (16 * NT), waves, wave);
  for (int64_t tile = tr.first; tile < tr.end; tile += tr.stride) {
    const int64_t q0 = tile * 16 * NT;
    raw b0[KB0][NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int64_t q = q0 + 16 * t + (lane & 15);
      const MT* row = h + (q < Q ? q : Q - 1) * (int64_t)M.K0;  // rows past Q are decoded and dropped
#pragma unroll
      for (int kb = 0; kb < KB0; ++kb)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int col = 32 * kb + 16 * half + 4 * (lane >> 4);  // K0 is a multiple of 4
          b0[kb][t][half] = *reinterpret_cast<const raw*>(row + (col < M.K0 ? col : 0));
        }
    }
    // operand chunk kb of N-tile t; inputs past K0 are zeros
    auto input = [&](int kb, int t) {
      union {
        raw r[2];
        frag f;
      } u;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        u.r[half] = b0[kb][t][half];
        if (kb == KB0 - 1) {
          const bool in = 32 * kb + 16 * half + 4 * (lane >> 4) < M.K0;
#pragma unroll
          for (int j = 0; j < (int)(sizeof(raw) / 4); ++j) u.r[half][j] = in ? u.r[half][j] : 0u;
        }
      }
      return u.f;
    };
    f32x4 out[NT];
    mlp_forward_tiles<MT, H, NT, KB0>(M, W, bias, KB0, lane, input, out);
    store_rgb<NT>(out, q0, Q, lane, rgb);
  }
}

// An attribute of the current device, or `otherwise` where it cannot be read.
static int device_attribute(hipDeviceAttribute_t a, int otherwise) {
  int dev = 0, v = 0;
  return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, a, dev) == hipSuccess && v > 0 ? v : otherwise;
}

int device_cus() {
  static const int cus = device_attribute(hipDeviceAttributeMultiprocessorCount, 256);
  return cus;
}

int max_lds() {
  static const int lds = device_attribute(hipDeviceAttributeMaxSharedMemoryPerBlock, 65536);
  return lds;
}

template <class MT, int H, int KB0>
static hipError_t launch_mlp_k(const MlpArgs& M, const void* h, int64_t Q, float* rgb, hipStream_t st) {
  // 16-bit weights always fit in LDS (132 KB at most), and so do FP32 ones
  // but for the widest decoders of three or more 128-wide hidden layers
  constexpr bool may_not_fit = sizeof(MT) == 4 && H == 128;
  const size_t wbytes = (size_t)packed_weight_elems<MT>(M.n_layers, M.K0, M.H) * sizeof(MT);
  const bool wlds = !may_not_fit || bias_bytes(M) + wbytes <= (size_t)max_lds();
  const size_t lds = bias_bytes(M) + (wlds ? wbytes : 0);
  const int rows = 16 * (wlds ? mlp_ntiles<MT, true>() : mlp_ntiles<MT, false>());
  int64_t grid = (Q + rows - 1) / rows;  // one eight-wave workgroup per CU
  if (grid > device_cus()) grid = device_cus();
  if (grid >= 8) grid -= grid % 8;
  auto k = mlp_kernel<MT, H, KB0, true>;
  if constexpr (may_not_fit)
    if (!wlds) k = mlp_kernel<MT, H, KB0, false>;
  allow_lds((const void*)k, lds);
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(512), lds, st, M, reinterpret_cast<const MT*>(h), Q, rgb);
  return hipGetLastError();
}

template <class MT, int H>
static hipError_t launch_mlp_t(const MlpArgs& M, const void* h, int64_t Q, float* rgb, hipStream_t st) {
  switch ((M.K0 + 31) / 32) {  // K0 <= 128
    case 1: return launch_mlp_k<MT, H, 1>(M, h, Q, rgb, st);
    case 2: return launch_mlp_k<MT, H, 2>(M, h, Q, rgb, st);
    case 3: return launch_mlp_k<MT, H, 3>(M, h, Q, rgb, st);
    default: return launch_mlp_k<MT, H, 4>(M, h, Q, rgb, st);
  }
}

hipError_t launch_mlp(const MlpArgs& M, oo_dtype md, const void* h, int64_t Q, float* rgb, hipStream_t st) {
  if (Q == 0) return hipSuccess;
  if (md == OO_F32) return M.H == 64 ? launch_mlp_t<float, 64>(M, h, Q, rgb, st) : launch_mlp_t<float, 128>(M, h, Q, rgb, st);
  if (md == OO_F16) return M.H == 64 ? launch_mlp_t<f16, 64>(M, h, Q, rgb, st) : launch_mlp_t<f16, 128>(M, h, Q, rgb, st);
  return M.H == 64 ? launch_mlp_t<bf16, 64>(M, h, Q, rgb, st) : launch_mlp_t<bf16, 128>(M, h, Q, rgb, st);
}

}  // namespace oo
