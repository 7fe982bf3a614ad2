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

template <bool QUANT, bool MANY>
__global__ __launch_bounds__(any::kThreads) void fwht_any_kernel(AnyBatch b)
{
    __shared__ float red[any::kThreads / kWave];
    __shared__ float lds[any::kLdsFloats];
    const AnyHeader h = whole_args(b.h);
    // (a grid holds 2^32 threads)
    for (int64_t vb = blockIdx.x; vb < h.total; vb += gridDim.x) {
        any::batch_block<QUANT, MANY>(b, h, (int)vb, red, lds);
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
    p.count = p.pieces = (int)count;
    p.steps = 1;
    b->t[h.n] = {q, p};
    h.total += p.count;
    ++h.n;
    return true;
}

// Workgroups that run at a time (73 registers a thread with a second piece on its way: six to a CU), and the most
// pieces that one takes: with two rounds of them or more, four at most (three and eight measured alike).  Only where at least
// half of the pieces are along axis 0, whose eight rows a thread are eight loads; along axis 1 a piece is two, and more waves in
// flight do better.  us without / with: axis 0 5000 x 1269 22.6 / 21.6, 5000 x 3277 45.8 / 37.5, at order 256 5120 x 3201 88.9 / 68.9;
// weight gradients of 99 features and outputs 32064 rows 42.9 / 40.3, 64129 64.4 / 53.1; steps of 4000 x 561 x 561 52.2 / 50.5,
// 60001 x 77 x 50 80.9 / 75.5; of 70 random sets of a layer's tensors just above the line 66 gain 1 to 13 % and two lose 1.  Axis 1
// alone 22231 x 301 17.8 / 18.4, forward products of 12544 x 502 x 32 21.0 / 23.
constexpr int kAnyPlaces = 1536, kAnyMostSteps = 4;

void finish_any(AnyBatch* b)
{
    AnyHeader& h = b->h;
    const int rounds = h.total / kAnyPlaces, steps = rounds < kAnyMostSteps ? rounds : kAnyMostSteps;
    int down = 0;
    for (int k = 0; k < h.n; ++k) down += b->t[k].q.axis ? 0 : b->t[k].p.pieces;
    if (steps < 2 || down < h.total - down) return;
    h.total = 0;
    for (int k = 0; k < h.n; ++k) {
        AnyPlan& p = b->t[k].p;
        p.steps = steps;
        p.count = (p.pieces + steps - 1) / steps;
        h.first[k] = h.total;
        h.total += p.count;
    }
}

hipError_t launch_any(const AnyBatch& b, int pass, hipStream_t stream)
{
    const dim3 grid((unsigned)(b.h.total < (1 << 23) ? b.h.total : (1 << 23)));
    ProfileScope ps(pass == 1 ? K_ANY_ABSMAX : K_ANY_QUANT, stream);
    const bool many = b.h.n && b.t[0].p.steps > 1;
    if (pass == 1 && many) hipLaunchKernelGGL((fwht_any_kernel<false, true>), grid, dim3(any::kThreads), 0, stream, b);
    else if (pass == 1) hipLaunchKernelGGL((fwht_any_kernel<false, false>), grid, dim3(any::kThreads), 0, stream, b);
    else if (many) hipLaunchKernelGGL((fwht_any_kernel<true, true>), grid, dim3(any::kThreads), 0, stream, b);
    else hipLaunchKernelGGL((fwht_any_kernel<true, false>), grid, dim3(any::kThreads), 0, stream, b);
    return hipGetLastError();
}

} // namespace hdqt
