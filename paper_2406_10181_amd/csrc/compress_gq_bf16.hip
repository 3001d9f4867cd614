// Kernel A of the compress path for bf16 storage (see compress_gq.h) in calls on raw projectors, whose plan is used once and is built sooner without
// the tiles that compress_mm.hip walks (4096 x 4096, r = 512, d = 8, raw: 50.6 us, with tiles and that kernel 55.2).
#include "compress_gq.h"

namespace lsp {
hipError_t launch_gq_bf16(CompressGroup& g, const RawCall& raw, hipStream_t st) {
    return launch_gq<BF16>(g, raw, st);
}
}  // namespace lsp
