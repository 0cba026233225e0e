// Pruned 3x3 conv, lean kernel for any pattern library (mask-testing form):
// fp32 or bf16, stride 1, dilation 1, pad 1.
//
// The channel-chunk kernel it takes these layers from reads every weight by a
// scalar load of its own inside the tap tests and stages per workgroup behind
// a barrier per chunk.
#include "conv_pp_lean.hpp"

namespace pp {

hipError_t launch_lean_gen(int id, const LeanParams& p, int n, bool bf16, hipStream_t st) {
#define PP_G(ID, R, CC, WS, V4)                                                                              \
  case ID:                                                                                                   \
    return bf16 ? kern::launch_lean_tiling<R, CC, 8, WS, V4, true, false, 1, 1, true>(p, n, st)              \
                : kern::launch_lean_tiling<R, CC, 8, WS, V4, false, false, 1, 1, true>(p, n, st);
  switch (id) {
    PP_GRECIPES(PP_G)
    default:
      return hipErrorInvalidValue;
  }
#undef PP_G
}

}  // namespace pp
