// Per-row preparation of the prompt pass: row log-sum-exps that come from outside.
#include "vatp_device.h"

namespace vatp {

namespace {

// Row log-sum-exp handed in by an upstream attention kernel (natural logarithm) -> base 2.
__global__ __launch_bounds__(256) void lse_to_base2_kernel(const float *__restrict__ lse,
                                                           float *__restrict__ lse2, BatchMeta meta,
                                                           int n_heads, int cap)
{
    const int b = blockIdx.z, h = blockIdx.y;
    const int r = blockIdx.x * 256 + threadIdx.x;
    const size_t unit = static_cast<size_t>(b) * n_heads + h;
    if (r < meta.len[b]) lse2[unit * cap + r] = lse[unit * cap + r] * kLog2e;
}

}  // namespace

hipError_t launch_lse_to_base2(const float *lse, float *lse2, const BatchMeta &meta, const Geometry &g,
                               hipStream_t st)
{
    if (g.max_len <= 0) return hipSuccess;
    const int q_heads = g.n_heads * g.group;           // one row log-sum-exp per query head
    hipLaunchKernelGGL(lse_to_base2_kernel, dim3((g.max_len + 255) / 256, q_heads, g.batch), dim3(256), 0, st, lse,
                       lse2, meta, q_heads, g.cap);
    return hipGetLastError();
}

}  // namespace vatp
