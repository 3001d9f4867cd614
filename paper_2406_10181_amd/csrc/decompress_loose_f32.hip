// k_expand_loose for fp32 storage (see decompress_loose.h).
#include "decompress_loose.h"

namespace lsp {
template <> hipError_t launch_loose<F32>(const ApplyGroup& g, unsigned grid, bool eight, bool norms, hipStream_t st) { return launch_loose_d<F32, 2>(g, grid, eight, norms, st); }
}  // namespace lsp
