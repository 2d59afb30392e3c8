// The bf16-triple multi-channel kernels for these filter sizes (multi_split.h).
#include "multi_split.h"

namespace dconv {
#define DCONV_LAUNCHER(K)                                                                    \
  hipError_t launch_split_k##K(const MultiPlan &p, const float *I, const float *F, float *O, \
                               const TileArgs &a, hipStream_t st) {                          \
    return launch_split_k<K>(p, I, F, O, a, st, std::make_integer_sequence<int, kNumSplit>{}); \
  }
DCONV_LAUNCHER(4)
DCONV_LAUNCHER(5)
}  // namespace dconv
