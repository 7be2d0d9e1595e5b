// Instantiation of the four-right-hand-side kernel for LinkF64 links.
#include "stencil_kernels.hpp"

namespace bri {

hipError_t launch_f64_rows(const StencilArgs &a, bool dag, int mode, hipStream_t st) {
    return dag ? launch_rows<LinkF64, true>(a, mode, st) : launch_rows<LinkF64, false>(a, mode, st);
}

}  // namespace bri
