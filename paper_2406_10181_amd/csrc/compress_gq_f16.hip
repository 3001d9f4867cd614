// Kernel A of the compress path for fp16 storage (see compress_gq.h).
#include "compress_gq.h"

namespace lsp {
hipError_t launch_gq_f16(CompressGroup& g, const RawCall& raw, hipStream_t st) {
    return launch_gq<F16>(g, raw, st);
}
}  // namespace lsp
