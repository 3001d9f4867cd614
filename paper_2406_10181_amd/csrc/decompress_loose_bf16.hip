// k_expand_loose for bf16 storage (see decompress_loose.h).
#include "decompress_loose.h"

namespace lsp {
template <> hipError_t launch_loose<BF16>(const ApplyGroup& g, unsigned grid, bool eight, bool norms, hipStream_t st) { return launch_loose_d<BF16, 2>(g, grid, eight, norms, st); }
}  // namespace lsp
