// Instantiation of the four-right-hand-side kernel for LinkBF16 links.
#include "stencil_kernels.hpp"

namespace bri {

hipError_t launch_bf16_rows(const StencilArgs &a, bool dag, int mode, hipStream_t st) {
    return dag ? launch_rows<LinkBF16, true>(a, mode, st) : launch_rows<LinkBF16, false>(a, mode, st);
}

}  // namespace bri
