// k_expand_loose for fp16 storage (see decompress_loose.h).
#include "decompress_loose.h"

namespace lsp {
template <> hipError_t launch_loose<F16>(const ApplyGroup& g, unsigned grid, bool eight, bool norms, hipStream_t st) { return launch_loose_d<F16, 2>(g, grid, eight, norms, st); }
}  // namespace lsp
