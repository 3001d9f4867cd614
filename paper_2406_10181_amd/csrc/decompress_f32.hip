// Decompress and apply, estimation bias for fp32 storage (see decompress.h).
#include "decompress.h"

namespace lsp {
hipError_t launch_apply_f32(ApplyGroup& g, int32_t r, int32_t d, hipStream_t st) { return launch_d_shape<F32>(g, r, d, st); }
hipError_t launch_bias_f32(ApplyGroup& g, int32_t r, int32_t d, float* partial, hipStream_t st) { return launch_bias_shape<F32>(g, r, d, partial, st); }
}  // namespace lsp
