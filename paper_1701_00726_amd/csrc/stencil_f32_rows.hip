// Instantiation of the four-right-hand-side kernel for LinkF32 links.
#include "stencil_kernels.hpp"

namespace bri {

hipError_t launch_f32_rows(const StencilArgs &a, bool dag, int mode, hipStream_t st) {
    return dag ? launch_rows<LinkF32, true>(a, mode, st) : launch_rows<LinkF32, false>(a, mode, st);
}

}  // namespace bri
