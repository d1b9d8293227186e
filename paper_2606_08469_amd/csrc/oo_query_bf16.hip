#include <hip/hip_runtime.h>

#include "oo_query.h"

namespace oo {

hipError_t launch_query_bf16(const TreeArgs& T, const MlpArgs& M, const QuerySrc& src, int64_t Q, float* rgb,
                            const QueryOut& O, const DispArgs& G, hipStream_t st) {
  return launch_query_m<bf16>(T, M, src, Q, rgb, O, G, st);
}

}  // namespace oo
