// Kernel A of the compress path for bf16 storage (see compress_gq.h).
#include "compress_gq.h"

namespace lsp {
hipError_t launch_gq_bf16(CompressGroup& g, int32_t r, int32_t d, const RawCall& raw, hipStream_t st) {
    return launch_gq<BF16>(g, r, d, raw, st);
}
}  // namespace lsp
