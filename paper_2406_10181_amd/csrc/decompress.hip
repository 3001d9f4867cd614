// Decompress and apply, estimation bias: what does not depend on the storage type (decompress.h has the kernels).
#include "decompress.h"

namespace lsp {

// Adds the workgroups' sums in order (in double) and forms the bias:
// out[0] = ||P S Q^T - G||_F^2, out[1] = ||G||_F^2, out[2] = sqrt(out[0] / out[1]).
__global__ __launch_bounds__(256) void k_bias_finish(const float2* __restrict__ partial, int count, float* __restrict__ out) {
    __shared__ double sx[256], sy[256];
    double x = 0.0, y = 0.0;
    for (int k = threadIdx.x; k < count; k += 256) { x += (double)partial[k].x; y += (double)partial[k].y; }
    sx[threadIdx.x] = x; sy[threadIdx.x] = y;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) { sx[threadIdx.x] += sx[threadIdx.x + off]; sy[threadIdx.x] += sy[threadIdx.x + off]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = (float)sx[0]; out[1] = (float)sy[0];
        out[2] = (float)sqrt(sx[0] / sy[0]);
    }
}

int64_t bias_blocks(int64_t m, int64_t n, int32_t r, int32_t d) {
    return bias_eight_rows(m, n, r, d, 2) || bias_eight_rows(m, n, r, d, 4) ? (m + 7) / 8 : (m + 15) / 16;
}

hipError_t launch_apply_f32(ApplyGroup& g, int32_t r, int32_t d, hipStream_t st);
hipError_t launch_apply_f16(ApplyGroup& g, int32_t r, int32_t d, hipStream_t st);
hipError_t launch_apply_bf16(ApplyGroup& g, int32_t r, int32_t d, hipStream_t st);
hipError_t launch_bias_f32(ApplyGroup& g, int32_t r, int32_t d, float* partial, hipStream_t st);
hipError_t launch_bias_f16(ApplyGroup& g, int32_t r, int32_t d, float* partial, hipStream_t st);
hipError_t launch_bias_bf16(ApplyGroup& g, int32_t r, int32_t d, float* partial, hipStream_t st);

hipError_t launch_bias(ApplyGroup& g, int32_t r, int32_t d, lsp_dtype dtype, float* partial, float* out, hipStream_t st) {
    const int64_t m = g.p[0].m;
    const bool eight = bias_eight_rows(m, g.p[0].n, r, d, dtype == LSP_F32 ? 4 : 2);
    hipError_t e;
    switch (dtype) {
        case LSP_F32:  e = launch_bias_f32(g, r, d, partial, st); break;
        case LSP_F16:  e = launch_bias_f16(g, r, d, partial, st); break;
        default:       e = launch_bias_bf16(g, r, d, partial, st); break;
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bias_finish, dim3(1), dim3(256), 0, st, reinterpret_cast<float2*>(partial), (int)(eight ? (m + 7) / 8 : (m + 15) / 16), out);
    return hipGetLastError();
}

hipError_t launch_decompress(ApplyGroup& g, int32_t r, int32_t d, lsp_dtype dtype, hipStream_t st) {
    switch (dtype) {
        case LSP_F32:  return launch_apply_f32(g, r, d, st);
        case LSP_F16:  return launch_apply_f16(g, r, d, st);
        default:       return launch_apply_bf16(g, r, d, st);
    }
}

__global__ __launch_bounds__(256) void k_validate(const int32_t* __restrict__ idx, int64_t count, int r, int32_t* flag) {
    int bad = 0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < count; k += (int64_t)gridDim.x * 256) {
        const int v = idx[k];
        bad |= (v < 0 || v >= r);
    }
    if (bad) *flag = 1;
}

__global__ void k_clear_flag(int32_t* flag) { *flag = 0; }

hipError_t launch_validate(const int32_t* idx, int64_t count, int32_t r, int32_t* flag, hipStream_t st) {
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, st, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(k_validate, dim3((unsigned)(blocks > 2048 ? 2048 : blocks)), dim3(256), 0, st, idx, count, (int)r, flag);
    return hipGetLastError();
}

}  // namespace lsp
