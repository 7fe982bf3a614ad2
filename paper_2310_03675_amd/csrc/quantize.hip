// Hadamard-domain quantization, the kernel for any shape (gfx950), and the fill kernel.
//
// Paper, Methodology section: y = x H along the contraction dimension with
// H = BlockDiag(H_k,..,H_k) in Sylvester form; Q(y) with alpha calibrated on
// the maximum of the tensor; nearest or stochastic rounding.
//
// Two passes over the source tensors, up to six (tensor, axis) pairs of any shapes in a launch:
//   pass 1  transform in registers, reduce max|y|
//   pass 2  transform again, scale, round, clamp, pack, store codes
// The transformed values never go to memory.  It serves what the tuned kernels
// (quantize_fast.hip, quantize_dual.hip) do not take -- odd contraction lengths, column counts that
// are no multiples of 4 -- and sets of small tensors, which are bound by latency: by the number
// of launches and by the chain of one wave's work.

#include "common.hpp"
#include "quantize_any.hpp"

#include <limits.h>

namespace hdqt {

namespace {

template <bool QUANT>
__global__ __launch_bounds__(any::kThreads) void fwht_any_kernel(AnyBatch b)
{
    __shared__ float red[any::kThreads / kWave];
    __shared__ float lds[any::kLdsFloats];
    const AnyHeader h = whole_args(b.h);
    // (a grid holds 2^32 threads)
    for (int64_t vb = blockIdx.x; vb < h.total; vb += gridDim.x) {
        any::batch_block<QUANT>(b, h, (int)vb, red, lds);
        if (vb + gridDim.x < h.total) __syncthreads();
    }
}

__global__ void zero2_kernel(uint32_t* a, int64_t na, uint32_t* b, int64_t nb)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na + nb;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i < na) a[i] = 0u;
        else b[i - na] = 0u;
    }
}

} // namespace

hipError_t launch_zero2(uint32_t* a, int64_t na, uint32_t* b, int64_t nb, hipStream_t stream)
{
    if (!b) nb = 0;
    const int64_t blocks = (na + nb + 255) / 256;
    const int grid = blocks < 1 ? 1 : blocks < 2048 ? (int)blocks : 2048;
    ProfileScope ps(K_FILL, stream);
    hipLaunchKernelGGL(zero2_kernel, dim3(grid), dim3(256), 0, stream, a, na, b, nb);
    return hipGetLastError();
}

bool plan_any(const QuantArgs& q, AnyBatch* b)
{
    AnyHeader& h = b->h;
    if (h.n == kMaxAny) return false;
    AnyPlan p{};
    int64_t count;
    if (q.axis) {
        p.per = make_divisor((uint32_t)((q.cols + 7) / 8));
        count = (q.rows * (int64_t)p.per.d + any::kThreads - 1) / any::kThreads;
    } else {
        // as many of the four waves side by side as there are columns for (32 columns are one
        // 128-byte line of a row); block orders above 64 need them on top of each other
        p.wc = q.log2n > 6 || q.cols <= 8 ? 1 : q.cols <= 16 ? 2 : 4;
        p.per = make_divisor((uint32_t)((q.cols + 8 * p.wc - 1) / (8 * p.wc)));
        const int64_t tall = 64 * (4 / p.wc);
        count = (int64_t)p.per.d * ((q.rows + tall - 1) / tall);
    }
    if (count + h.total >= ((int64_t)1 << 31)) return false;
    if (!h.n)
        for (int k = 0; k < kMaxAny; ++k) h.first[k] = INT_MAX;
    h.first[h.n] = h.total;
    p.count = (int)count;
    b->t[h.n] = {q, p};
    h.total += p.count;
    ++h.n;
    return true;
}

hipError_t launch_any(const AnyBatch& b, int pass, hipStream_t stream)
{
    const dim3 grid((unsigned)(b.h.total < (1 << 23) ? b.h.total : (1 << 23)));
    ProfileScope ps(pass == 1 ? K_ANY_ABSMAX : K_ANY_QUANT, stream);
    if (pass == 1) hipLaunchKernelGGL(fwht_any_kernel<false>, grid, dim3(any::kThreads), 0, stream, b);
    else hipLaunchKernelGGL(fwht_any_kernel<true>, grid, dim3(any::kThreads), 0, stream, b);
    return hipGetLastError();
}

} // namespace hdqt
