// Decompress and apply, estimation bias where rows begin anywhere, or d is none of 2, 4, 8, 16: k_expand_loose (decompress.h), for every d from 2 to kLooseEntries.
#pragma once

#include "decompress.h"

namespace lsp {

template <typename D, int LP, int DD, bool NORMS, WideForm FORM>
static hipError_t launch_loose_kernel(const ApplyGroup& g, unsigned grid, hipStream_t st) {
    constexpr auto kern = k_expand_loose<D, LP, DD, NORMS, FORM>;
    constexpr size_t ents = (size_t)4 * LP * DD * sizeof(int2);
    hipError_t e;
    if ((e = allow_dynamic_lds<kern, (size_t)1024 * 16 * LP + ents>()) != hipSuccess) return e;
    const size_t lds = (size_t)(g.r + 3) / 4 * 4 * 16 * LP + ents;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), lds, st, g);
    return hipGetLastError();
}

template <typename D, int DD>
static hipError_t launch_loose_d(const ApplyGroup& g, unsigned grid, bool eight, bool norms, hipStream_t st) {
    if (g.d != DD) {
        if constexpr (DD < kLooseEntries) return launch_loose_d<D, DD + 1>(g, grid, eight, norms, st);
        else return hipErrorInvalidValue;
    }
    const bool deep = grid <= kResidentDeep;
    if (eight) return norms ? launch_loose_kernel<D, 2, DD, true, kDeep>(g, grid, st) : launch_loose_kernel<D, 2, DD, false, kDeep>(g, grid, st);
    if (deep) return norms ? launch_loose_kernel<D, 4, DD, true, kDeep>(g, grid, st) : launch_loose_kernel<D, 4, DD, false, kDeep>(g, grid, st);
    return norms ? launch_loose_kernel<D, 4, DD, true, kTwo>(g, grid, st) : launch_loose_kernel<D, 4, DD, false, kTwo>(g, grid, st);
}

}  // namespace lsp
