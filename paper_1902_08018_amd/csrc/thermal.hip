// thermal.hip -- the thermal step of the model (Sec. 2.1, Eq. 1):
//
//     T_{k+1} = A T_k + B u_k,   A sparse (CSR), B diagonal,
//
// evaluated every millisecond (light and dark stages) on about 3.7e5
// temperatures before the deformation GEMV.  One lane per row: the row's
// products and b_i u_i are summed in FP64 (the kernel is bound by HBM, so the
// wide arithmetic costs nothing) and the state is stored as FP32.  Per row the
// kernel moves its CSR entries (8 B each), its row pointer, b_i, u_i, T_i and
// the new T_i (the gathered neighbours of a mesh come from cache).
#include <hip/hip_runtime.h>

#include "../../include/wh.h"
#include "wh_ctx.hpp"
#include "wh_internal.hpp"

namespace wh {
namespace {

// Lanes of a workgroup: 512 where that gives every CU one, else 64.  A small
// system's time is that of its gathers in the CUs that have some, so it is
// spread over as many as there are.  us a step, 64 / 256 / 512 lanes: 5,000
// rows of 7 entries 2.9 / 3.7 / 4.4 (rows of 27 4.3 / 6.9 / 11.6), 60,000 of 5
// 3.0 / 3.4 / 3.6, 100,000 of 5 3.7 / 3.8 / 3.7, 131,072 of 5 3.9 / 4.0 / 3.7.
constexpr unsigned kThermalThreads = 512, kThermalThreadsSmall = 64;
// entries of a row read together: the rows of a two-dimensional mesh have five
constexpr int kThermalBatch = 5;

// One lane per row.  A launch is short (the 608 x 608 mesh: 369,664 rows, all
// resident at once), so it is bound by memory latency: the row's pointers, its
// entries, the entries' temperatures, and the launch itself (1.6 us empty, 2.8
// without entries).  A batch of entries is loaded before any of its
// temperatures, and those before the first product, so a mesh row waits twice
// for its entries and not twice an entry.  The new state is stored past the
// cache: it is read by the next launch, whose XCDs' L2s would not share it,
// and the kernel's end need not write it back.  608 x 608, 100 steps, us a
// step: one entry at a time 6.5, batches of 2 / 3 / 4 / 5 / 6 / 8 with the
// streaming store 6.1 / 5.8 / 6.5 / 5.2 / 5.6 / 6.4, batches of 5 with an
// ordinary store 5.6; 512 lanes a workgroup 5.1, 1024 5.8.  The workgroup
// taking all its rows' entries in order through LDS took 8.2.
__global__ void __launch_bounds__(kThermalThreads) thermal_step_kernel(
    uint32_t n, uint32_t nnz, const uint32_t* __restrict__ row_ptr, const uint32_t* __restrict__ col,
    const float* __restrict__ val, const float* __restrict__ b, const float* __restrict__ T,
    const float* __restrict__ u, float* __restrict__ T_next)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        // entries outside [0, nnz) and columns outside [0, n) are skipped: a
        // malformed matrix gives wrong values, never a stray access
        const uint32_t p0 = row_ptr[i] < nnz ? row_ptr[i] : nnz;
        const uint32_t p1 = row_ptr[i + 1] < nnz ? row_ptr[i + 1] : nnz;
        const float bi = b[i], ui = u[i];
        double s = 0.0;
        for (uint32_t p = p0; p < p1; p += kThermalBatch) {
            uint32_t j[kThermalBatch];
            float v[kThermalBatch], t[kThermalBatch];
            const uint32_t left = p1 - p;
#pragma unroll
            for (uint32_t k = 0; k < kThermalBatch; ++k) {
                const uint32_t q = k < left ? p + k : p1 - 1; // past the row: its last entry again
                j[k] = col[q];
                v[k] = val[q];
            }
#pragma unroll
            for (uint32_t k = 0; k < kThermalBatch; ++k) {
                const bool counts = k < left && j[k] < n;
                const float x = T[counts ? j[k] : 0u];
                t[k] = counts ? x : 0.0f;
                v[k] = counts ? v[k] : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < kThermalBatch; ++k)
                s = __builtin_fma((double)v[k], (double)t[k], s);
            if (left <= kThermalBatch)
                break; // p + kThermalBatch may wrap
        }
        s = __builtin_fma((double)bi, (double)ui, s);
        __builtin_nontemporal_store((float)s, T_next + i);
    }
}

struct ThermalGrid {
    unsigned groups, threads;
};

ThermalGrid thermal_grid(uint32_t n, int num_cus)
{
    const unsigned threads = (uint64_t)n < (uint64_t)kThermalThreads * num_cus ? kThermalThreadsSmall : kThermalThreads;
    const uint64_t g = ((uint64_t)n + threads - 1) / threads;
    return ThermalGrid{(unsigned)(g < (1u << 20) ? (g ? g : 1) : (1u << 20)), threads};
}

} // namespace
} // namespace wh

using namespace wh;

extern "C" wh_status wh_thermal_step(wh_ctx* ctx, uint32_t n, uint32_t nnz, const uint32_t* d_row_ptr,
                                     const uint32_t* d_col, const float* d_val, const float* d_b, const float* d_T,
                                     const float* d_u, float* d_T_next, void* stream)
{
    WH_GUARD(ctx);
    if (!d_row_ptr || !d_b || !d_T || !d_u || !d_T_next || (nnz && (!d_col || !d_val)))
        return WH_ERR_INVALID;
    if (d_T == d_T_next)
        return WH_ERR_INVALID; // every row reads its neighbours' old values
    if (n == 0)
        return WH_OK;
    const ThermalGrid g = thermal_grid(n, ctx->num_cus);
    hipLaunchKernelGGL(thermal_step_kernel, dim3(g.groups), dim3(g.threads), 0,
                       static_cast<hipStream_t>(stream), n, nnz, d_row_ptr, d_col, d_val, d_b, d_T, d_u, d_T_next);
    return device_error(ctx, hipGetLastError());
}

extern "C" wh_status wh_thermal_run(wh_ctx* ctx, uint32_t n, uint32_t nnz, const uint32_t* d_row_ptr,
                                    const uint32_t* d_col, const float* d_val, const float* d_b, float* d_T,
                                    const float* d_U, uint64_t ldu, uint32_t steps, float* d_work, void* stream)
{
    WH_GUARD(ctx);
    if (!d_row_ptr || !d_b || !d_T || !d_work || (steps && !d_U) || (nnz && (!d_col || !d_val)))
        return WH_ERR_INVALID;
    if (d_T == d_work || ldu < n)
        return WH_ERR_INVALID;
    if (n == 0 || steps == 0)
        return WH_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // ping-pong between d_T and d_work; an odd count ends with a copy back
    float* cur = d_T;
    float* nxt = d_work;
    const ThermalGrid g = thermal_grid(n, ctx->num_cus);
    for (uint32_t k = 0; k < steps; ++k) {
        hipLaunchKernelGGL(thermal_step_kernel, dim3(g.groups), dim3(g.threads), 0, st, n, nnz,
                           d_row_ptr, d_col, d_val, d_b, cur, d_U + (uint64_t)k * ldu, nxt);
        float* t = cur;
        cur = nxt;
        nxt = t;
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && cur != d_T)
        e = hipMemcpyAsync(d_T, cur, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st);
    return device_error(ctx, e);
}
