// Kernel A of the compress path for fp16 storage (see compress_gq.h).
#include "compress_gq.h"

namespace lsp {
hipError_t launch_gq_f16(CompressGroup& g, int32_t r, int32_t d, const RawCall& raw, hipStream_t st) {
    return launch_gq<F16>(g, r, d, raw, st);
}
}  // namespace lsp
