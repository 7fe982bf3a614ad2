// Layout changes around the matmuls, pure data movement, one launch each:
//   unfolding of a convolution's input into the matrix the matmuls take, for the layers whose
//   geometry the activation-source kernels do not read directly (strides, windows that leave K
//   off a multiple of 64, tiny images): X[(b, yo, xo), c*kh*kw + ty*kw + tx] =
//   act[b, c, yo*stride + ty - ph, xo*stride + tx - pw], zero outside the image;
//   its adjoint, the gradient of the matrix folded back onto the activation;
//   and [batch, rows, cols] -> [batch, cols, rows], the layout of pixels x channels against that of
//   images (channel planes).
#include "common.hpp"

namespace hdqt {

namespace {

constexpr int kThreads = 256;

// ---- unfolding: a thread has one column of X (its channel and tap are worked out once) and kRows
// rows of it, kUnroll loads in flight.  (A row at a time, with the divisions of every element in front
// of a single load: 330 us for the ten such layers of a ResNet-18 at batch 128, 270 MB of
// matrices; now 170.)
constexpr int kRows = 32;          // per thread
constexpr int kUnroll = 8;

__global__ __launch_bounds__(kThreads) void im2col_kernel(Im2colArgs a, int width, int log2w, uint32_t n_col)
{
    const int K = a.C * a.kh * a.kw, khw = a.kh * a.kw;
    // (runs of rows and, fastest, of columns on one axis of the grid: the others hold 65535 workgroups,
    // 2097120 rows of more than 128 columns)
    const uint32_t run = blockIdx.x / n_col;
    const int k = (int)(blockIdx.x - run * n_col) * width + ((int)threadIdx.x & (width - 1));
    if (k >= K) return;
    const int c = k / khw, tap = k - c * khw, ty = tap / a.kw, tx = tap - ty * a.kw;
    const int side = kThreads >> log2w;                  // rows of the workgroup at a time
    const int64_t per_image = (int64_t)a.Ho * a.Wo;
    int64_t m = (int64_t)run * ((int64_t)side * kRows) + ((int)threadIdx.x >> log2w);
    const int64_t b = m / per_image;
    int yo = (int)((m - b * per_image) / a.Wo), xo = (int)(m - b * per_image - (int64_t)yo * a.Wo);
    // (an image and its next: the offsets inside one fit 32 bits)
    const int64_t image = (int64_t)a.C * a.H * a.W;
    const float* src = a.act + b * image + (int64_t)c * a.H * a.W;
    float* dst = a.X + m * K + k;
    const int64_t step = (int64_t)side * K;
    for (int r0 = 0; r0 < kRows; r0 += kUnroll) {
        float v[kUnroll];
#pragma unroll
        for (int r = 0; r < kUnroll; ++r) {
            const int y = yo * a.stride + ty - a.ph, x = xo * a.stride + tx - a.pw;
            const bool in = m + (int64_t)(r0 + r) * side < a.M && y >= 0 && y < a.H && x >= 0 && x < a.W;
            v[r] = in ? src[y * a.W + x] : 0.0f;
            xo += side;
            while (xo >= a.Wo) {
                xo -= a.Wo;
                if (++yo == a.Ho) { yo = 0; src += image; }
            }
        }
#pragma unroll
        for (int r = 0; r < kUnroll; ++r) {
            if (m + (int64_t)(r0 + r) * side < a.M) *dst = v[r];
            dst += step;
        }
    }
}

// ---- folding: a workgroup has 32 pixels of the activation (of the batch's pixels in a row) and 64
// channels.  Lanes are channels, so that the kh * kw elements a lane adds up for a pixel lie in the
// lines its neighbours read too, and which taps there are is the same for the whole wave; the sums
// turn through LDS and leave as runs of pixels.  The taps are added from the window's end to its
// start, i.e. in the order of the matrix rows.
//
// A pixel has at most ceil(kh / stride) x ceil(kw / stride) taps, whose loads go out NY x NX at a time:
// all of them, or (NY = 1, larger windows) along one row of the window.  Of those that fall outside
// the matrix a zero is added.  128 x 64 x 32 x 32, window 3, stride 2: 94 -> 68 us against a loop over
// the window that loads and adds tap by tap.
constexpr int kFoldPixels = 32, kFoldChannels = 64;

__device__ __forceinline__ int last_tap(int at, int k, int stride)      // largest t < k, t = at modulo stride
{
    return k - 1 - (k - 1 + stride - at % stride) % stride;
}

template <int NY, int NX>
__global__ __launch_bounds__(kThreads) void col2im_kernel(Im2colArgs a)
{
    __shared__ float turn[kFoldChannels][kFoldPixels + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int khw = a.kh * a.kw, K = a.C * khw, HW = a.H * a.W;
    const int c0 = (int)blockIdx.y * kFoldChannels, c = c0 + lane < a.C ? c0 + lane : a.C - 1;
    const int lane_off = c * khw;
    // (a grid holds 2^32 threads; the activation of a strided layer has more pixels than its matrix rows)
    for (int64_t p0 = (int64_t)blockIdx.x * kFoldPixels; p0 < a.M; p0 += (int64_t)gridDim.x * kFoldPixels) {
        // (the same in every lane) the wave's first pixel
        const int64_t p_first = p0 + wave * (kFoldPixels / 4);
        int64_t b = p_first / HW;
        int y = (int)((uint32_t)(p_first - b * HW) / (uint32_t)a.W), x = (int)(p_first - b * HW) - y * a.W;
        for (int i = 0; i < kFoldPixels / 4; ++i) {
            if (p_first + i >= a.M) break;
            float sum = 0.0f;
            // the last tap whose matrix row or column is a whole number of strides away, and every
            // stride-th before it
            const int ty_last = last_tap(y + a.ph, a.kh, a.stride), tx_last = last_tap(x + a.pw, a.kw, a.stride);
            for (int ty0 = ty_last; ty0 >= 0; ty0 -= NY * a.stride)
                for (int tx0 = tx_last; tx0 >= 0; tx0 -= NX * a.stride) {
                    float v[NY * NX];
#pragma unroll
                    for (int u = 0; u < NY * NX; ++u) {
                        const int ty = ty0 - u / NX * a.stride, tx = tx0 - u % NX * a.stride;
                        const int yo = (y + a.ph - ty) / a.stride, xo = (x + a.pw - tx) / a.stride;
                        const bool ok = ty >= 0 && tx >= 0 && y + a.ph >= ty && x + a.pw >= tx && yo < a.Ho && xo < a.Wo;
                        const float* row = a.X + (ok ? ((b * a.Ho + yo) * a.Wo + xo) * (int64_t)K + ty * a.kw + tx : 0);
                        v[u] = row[lane_off];
                        if (!ok) v[u] = 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < NY * NX; ++u) sum += v[u];
                }
            turn[lane][wave * (kFoldPixels / 4) + i] = sum;
            if (++x == a.W) {
                x = 0;
                if (++y == a.H) { y = 0; ++b; }
            }
        }
        __syncthreads();
        const int64_t p = p0 + (lane & 31);
        if (p < a.M) {
            const int64_t bp = p / HW, at = p - bp * HW;
            for (int i = 0; i < kFoldChannels / 8; ++i) {
                const int ch = wave * (kFoldChannels / 4) + 2 * i + (lane >> 5);
                if (c0 + ch < a.C) a.out[(bp * a.C + c0 + ch) * HW + at] = turn[ch][lane & 31];
            }
        }
        if (p0 + (int64_t)gridDim.x * kFoldPixels < a.M) __syncthreads();
    }
}

// ---- transposition: 64 x 64 elements through LDS, whole lines on both sides
constexpr int kTurn = 64;

__global__ __launch_bounds__(kThreads) void transpose_kernel(const float* src, float* dst, int64_t rows, int64_t cols)
{
    __shared__ float turn[kTurn][kTurn + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * kTurn, r0 = (int64_t)blockIdx.y * kTurn;
    src += (int64_t)blockIdx.z * rows * cols;
    dst += (int64_t)blockIdx.z * rows * cols;
    float v[kTurn / 4];
#pragma unroll
    for (int i = 0; i < kTurn / 4; ++i) {
        const int64_t r = r0 + 4 * i + wave;
        v[i] = r < rows && c0 + lane < cols ? src[r * cols + c0 + lane] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < kTurn / 4; ++i) turn[4 * i + wave][lane] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTurn / 4; ++i) {
        const int64_t c = c0 + 4 * i + wave;
        if (c < cols && r0 + lane < rows) dst[c * rows + r0 + lane] = turn[lane][4 * i + wave];
    }
}

} // namespace

hipError_t launch_im2col(const Im2colArgs& a, hipStream_t stream)
{
    const int64_t K = (int64_t)a.C * a.kh * a.kw;
    int log2w = 5;
    while (log2w < 8 && (1 << log2w) < K) ++log2w;
    const int width = 1 << log2w;
    const int64_t tall = (int64_t)(kThreads / width) * kRows;
    const int64_t n_col = (K + width - 1) / width, runs = (a.M + tall - 1) / tall;
    ProfileScope ps(K_IM2COL, stream);
    hipLaunchKernelGGL(im2col_kernel, dim3((unsigned)(n_col * runs)), dim3(kThreads), 0, stream, a, width, log2w,
                       (uint32_t)n_col);
    return hipGetLastError();
}

hipError_t launch_col2im(const Im2colArgs& a, hipStream_t stream)
{
    const int64_t runs = (a.M + kFoldPixels - 1) / kFoldPixels;
    const unsigned across = (unsigned)((a.C + kFoldChannels - 1) / kFoldChannels);
    const dim3 grid((unsigned)(runs < (1 << 23) ? runs : (1 << 23)), across);
    ProfileScope ps(K_COL2IM, stream);
    const int ny = (a.kh + a.stride - 1) / a.stride, nx = (a.kw + a.stride - 1) / a.stride, n = ny > nx ? ny : nx;
    if (n == 1) hipLaunchKernelGGL((col2im_kernel<1, 1>), grid, dim3(kThreads), 0, stream, a);
    else if (n == 2) hipLaunchKernelGGL((col2im_kernel<2, 2>), grid, dim3(kThreads), 0, stream, a);
    else if (n == 3) hipLaunchKernelGGL((col2im_kernel<3, 3>), grid, dim3(kThreads), 0, stream, a);
    else hipLaunchKernelGGL((col2im_kernel<1, 3>), grid, dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_transpose(const float* src, float* dst, int64_t batch, int64_t rows, int64_t cols, hipStream_t stream)
{
    const dim3 grid((unsigned)((cols + kTurn - 1) / kTurn), (unsigned)((rows + kTurn - 1) / kTurn), (unsigned)batch);
    ProfileScope ps(K_TRANSPOSE, stream);
    hipLaunchKernelGGL(transpose_kernel, grid, dim3(kThreads), 0, stream, src, dst, rows, cols);
    return hipGetLastError();
}

} // namespace hdqt
