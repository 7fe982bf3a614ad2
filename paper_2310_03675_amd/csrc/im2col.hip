// Layout changes around the matmuls, pure data movement, one launch each:
//   unfolding of a convolution's input into the matrix the matmuls take, for the layers whose
//   geometry the activation-source kernels do not read directly (strides, windows that leave K
//   off a multiple of 64, tiny images): X[(b, yo, xo), c*kh*kw + ty*kw + tx] =
//   act[b, c, yo*stride + ty - ph, xo*stride + tx - pw], zero outside the image;
//   its adjoint, the gradient of the matrix folded back onto the activation;
//   and [batch, rows, cols] -> [batch, cols, rows], the layout of pixels x channels against that of
//   images (channel planes).
#include "common.hpp"

#include <limits.h>

namespace hdqt {

namespace {

constexpr int kThreads = 256;

// ---- unfolding through LDS: a workgroup has TX x TY windows of one image (a tile of the matrix rows) and CB
// channels.  It fetches the part of the activation under them as runs of a row's pixels and writes CB * kh *
// kw neighbours in each matrix row, 16 bytes a lane; where a column's element lies in LDS stands in a
// table.  What bounds it is writing X.  Of windows that leave pixels out (1 x 1 with stride 2) only those
// under a window are fetched.  At batch 128, us a call, with a thread's column at a time and now (4.9 TB/s:
// the floor): 64 x 32 x 32, stride 2, window 3 42 / 26 (22), window 1 11.4 / 8.7 (8.6); 256 x 8 x 8, stride 2,
// window 1 9.2 / 4.3 (2.1); 96 x 14 x 14, stride 1, window 3 31 / 21 (20).
struct UnfoldTile {
    int TY, CB;             // windows on top of each other; channels
    int sy, sx;             // from a window to the next in LDS: the stride, or the window where that is less
    int plane;              // floats per channel in LDS
    Divisor TX, across, down, blocks;              // (tiles of an image; blocks of channels)
    Divisor width, height, step_y, step_x;         // of a plane; sy, sx
    Divisor taps, kw, units;                       // kh * kw; stores per matrix row
};
constexpr int kTileLds = 32 * 1024;
constexpr int64_t kTiles = (int64_t)1 << 22;       // (a grid holds 2^32 threads)

__global__ __launch_bounds__(kThreads) void im2col_tile_kernel(Im2colArgs a, UnfoldTile t)
{
    extern __shared__ __attribute__((aligned(16))) float part[];
    const int tid = threadIdx.x;
    const int khw = (int)t.taps.d, K = a.C * khw;
    const uint32_t i1 = divide(blockIdx.x, t.blocks), i2 = divide(i1, t.across), b = divide(i2, t.down);
    const int c0 = (int)(blockIdx.x - i1 * t.blocks.d) * t.CB, xo0 = (int)((i1 - i2 * t.across.d) * t.TX.d);
    const int yo0 = (int)(i2 - b * t.down.d) * t.TY;
    const int cn = a.C - c0 < t.CB ? a.C - c0 : t.CB, TY = a.Ho - yo0 < t.TY ? a.Ho - yo0 : t.TY;
    int* column = reinterpret_cast<int*>(part);
    float* patch = part + (t.CB * khw + 3 & ~3);
    for (int q = tid; q < cn * khw; q += kThreads) {
        const uint32_t c = divide((uint32_t)q, t.taps), tap = (uint32_t)q - c * t.taps.d, ty = divide(tap, t.kw);
        column[q] = (int)(c * t.plane + ty * t.width.d + tap - ty * t.kw.d);
    }
    {
        constexpr int UNROLL = 8;
        const int total = cn * t.plane, yb = yo0 * a.stride - a.ph, xb = xo0 * a.stride - a.pw;
        const float* src = a.act + ((int64_t)b * a.C + c0) * a.H * a.W;
        for (int i0 = tid; i0 < total; i0 += kThreads * UNROLL) {
            float v[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const uint32_t i = (uint32_t)(i0 + u * kThreads), line = divide(i, t.width), j = i - line * t.width.d;
                const uint32_t c = divide(line, t.height), r = line - c * t.height.d;
                const int y = yb + (int)r + (int)divide(r, t.step_y) * (a.stride - t.sy);
                const int x = xb + (int)j + (int)divide(j, t.step_x) * (a.stride - t.sx);
                const bool in = (int)i < total && y >= 0 && y < a.H && x >= 0 && x < a.W;
                // (an image's offsets fit 32 bits)
                v[u] = in ? src[((int)c * a.H + y) * a.W + x] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (i0 + u * kThreads < total) patch[i0 + u * kThreads] = v[u];
        }
    }
    __syncthreads();

    const int have = cn * khw / 4;                     // (K and c0 * khw are multiples of 4)
    const int total = TY * (int)(t.TX.d * t.units.d);
    float* dst = a.X + (((int64_t)b * a.Ho + yo0) * a.Wo + xo0) * K + (int64_t)c0 * khw;
#pragma unroll 4
    for (int i = tid; i < total; i += kThreads) {
        const uint32_t row = divide((uint32_t)i, t.units), ry = divide(row, t.TX);
        const int unit = i - (int)(row * t.units.d), rx = (int)(row - ry * t.TX.d);
        if (unit >= have || xo0 + rx >= a.Wo) continue;
        const float* from = patch + (int)ry * t.sy * (int)t.width.d + rx * t.sx;
        float* to = dst + ((int64_t)(int)ry * a.Wo + rx) * K + unit * 4;
        const int4 at = *reinterpret_cast<const int4*>(column + 4 * unit);
        *reinterpret_cast<float4*>(to) = make_float4(from[at.x], from[at.y], from[at.z], from[at.w]);
    }
}

// ---- unfolding for every geometry (rows of X that are no whole 16-byte units, where a tile's stores would be
// single elements: 16 x 3 x 224 x 224, window 7, stride 2 50 us against 43; windows whose part of the activation
// does not fit LDS; tiles that do not pay, see unfold_tiles_pay): a thread has one column of X (its channel and
// tap are worked out once) and kRows rows of it, kUnroll loads in flight.  (A row at a time, with the divisions of
// every element in front of a single load: 330 us for the ten such layers of a ResNet-18 at batch 128, 270 MB
// of matrices; this way 170.)
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

// ---- folding through LDS: a workgroup has a tile of TX x TY pixels of one image and CB channels.  The
// elements that it adds up are CB * kh * kw neighbours in each of the matrix rows whose window meets the
// tile; they are fetched as whole runs of 16 bytes a lane, and a thread then picks its pixel's taps, at
// the same places for every channel, and writes runs of pixels.  What bounds it is memory: the matrix is
// read once (rows at the tiles' edges up to three times, from the caches).  Fetched from memory tap by
// tap, lanes kh * kw elements apart, every load spread over 18 lines and a pixel's chain of loads and
// index divisions was all a wave had in flight.  At batch 128, us a call, then and now (4.9 TB/s: the floor):
// 64 x 32 x 32, stride 2, window 3 69 / 27 (22), window 1 37 / 8.6 (8.6); 128 x 16 x 16, stride 2, window 3
// 36 / 13.4 (11); 512 x 4 x 4, stride 1, window 3 19 / 9.3 (8.6).
// At most NY x NX taps meet in a pixel; they are added from the window's end to its start, i.e. in the order
// of the matrix rows, a zero for those outside the matrix.
struct FoldTile {
    int TY, log2p;          // pixel rows of a tile; lanes are dealt 2^log2p pixels
    int CB, pitch;          // channels, floats per matrix row in LDS
    int rows_x;             // matrix rows side by side that the tile's pixels meet
    Divisor TX, stride, across, down, blocks;      // (across, down: tiles of an image; blocks of channels)
    Divisor units, row_x;   // loads per matrix row; rows_x
};

__device__ __forceinline__ int last_tap(int r, int k, const Divisor& stride)      // largest t < k, t = r modulo stride
{
    const uint32_t over = (uint32_t)(k - 1 - r) + stride.d;
    return k - 1 - (int)(over - divide(over, stride) * stride.d);
}

template <int NY, int NX, bool WIDE>
__global__ __launch_bounds__(kThreads) void col2im_tile_kernel(Im2colArgs a, FoldTile t)
{
    extern __shared__ __attribute__((aligned(16))) float part[];
    const int tid = threadIdx.x;
    const int khw = a.kh * a.kw, K = a.C * khw, HW = a.H * a.W;
    const uint32_t i1 = divide(blockIdx.x, t.blocks), i2 = divide(i1, t.across), b = divide(i2, t.down);
    const int c0 = (int)(blockIdx.x - i1 * t.blocks.d) * t.CB, x0 = (int)((i1 - i2 * t.across.d) * t.TX.d);
    const int y0 = (int)(i2 - b * t.down.d) * t.TY;
    const int cn = a.C - c0 < t.CB ? a.C - c0 : t.CB, TX = (int)t.TX.d, s = (int)t.stride.d;
    const int y_end = a.H - y0 < t.TY ? a.H : y0 + t.TY, x_end = a.W - x0 < TX ? a.W : x0 + TX;

    // the matrix rows that meet the tile
    const int yb = y0 + a.ph - a.kh, xb = x0 + a.pw - a.kw;
    const int yo_lo = yb < 0 ? 0 : (int)divide((uint32_t)yb, t.stride) + 1, xo_lo = xb < 0 ? 0 : (int)divide((uint32_t)xb, t.stride) + 1;
    const int yo_in = (int)divide((uint32_t)(y_end - 1 + a.ph), t.stride), xo_in = (int)divide((uint32_t)(x_end - 1 + a.pw), t.stride);
    const int yo_hi = yo_in < a.Ho ? yo_in : a.Ho - 1, xo_hi = xo_in < a.Wo ? xo_in : a.Wo - 1;
    {
        constexpr int PER = WIDE ? 4 : 1, UNROLL = WIDE ? 4 : 8;
        const int have = cn * khw / PER;                  // (wide: K and c0 * khw are multiples of 4)
        const int total = (yo_hi - yo_lo + 1) * t.rows_x * (int)t.units.d;      // (<= 0: no row meets it)
        const float* src = a.X + (((int64_t)b * a.Ho + yo_lo) * a.Wo + xo_lo) * K + (int64_t)c0 * khw;
        for (int i0 = tid; i0 < total; i0 += kThreads * UNROLL) {
            float4 v[UNROLL];
            int at[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const uint32_t i = (uint32_t)(i0 + u * kThreads), row = divide(i, t.units), ry = divide(row, t.row_x);
                const int unit = (int)(i - row * t.units.d), rx = (int)(row - ry * t.row_x.d);
                const bool in = (int)i < total && unit < have && xo_lo + rx <= xo_hi;
                at[u] = in ? (int)row * t.pitch + unit * PER : -1;
                const float* from = src + ((int64_t)(int)ry * a.Wo + rx) * K + unit * PER;
                if constexpr (WIDE) v[u] = in ? *reinterpret_cast<const float4*>(from) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                else v[u].x = in ? *from : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                if (at[u] < 0) continue;
                if constexpr (WIDE) *reinterpret_cast<float4*>(part + at[u]) = v[u];
                else part[at[u]] = v[u].x;
            }
        }
    }
    __syncthreads();

    const int p = tid & ((1 << t.log2p) - 1), py = (int)divide((uint32_t)p, t.TX);
    const int y = y0 + py, x = x0 + p - py * TX;
    if (y >= y_end) return;       // (x < x_end or another tile's column)
    if (x >= x_end) return;
    const int qy = (int)divide((uint32_t)(y + a.ph), t.stride), qx = (int)divide((uint32_t)(x + a.pw), t.stride);
    const int ry = y + a.ph - qy * s, rx = x + a.pw - qx * s;
    const int ty0 = last_tap(ry, a.kh, t.stride), tx0 = last_tap(rx, a.kw, t.stride);
    // (a multiple of the stride, minus one stride where the pixel lies between the windows)
    const int yo0 = qy - ((int)divide((uint32_t)(ty0 - ry + s), t.stride) - 1), xo0 = qx - ((int)divide((uint32_t)(tx0 - rx + s), t.stride) - 1);
    int at[NY * NX];
    bool ok[NY * NX];
#pragma unroll
    for (int u = 0; u < NY * NX; ++u) {
        const int j = u / NX, i = u % NX;
        const int ty = ty0 - j * s, tx = tx0 - i * s, yo = yo0 + j, xo = xo0 + i;
        ok[u] = ty >= 0 && tx >= 0 && yo >= 0 && yo < a.Ho && xo >= 0 && xo < a.Wo;
        at[u] = ok[u] ? ((yo - yo_lo) * t.rows_x + (xo - xo_lo)) * t.pitch + ty * a.kw + tx : 0;
    }
    const int side = kThreads >> t.log2p;
    float* out = a.out + ((int64_t)b * a.C + c0) * HW + (int64_t)y * a.W + x;
#pragma unroll 4
    for (int ch = tid >> t.log2p; ch < cn; ch += side) {
        float sum = 0.0f;
#pragma unroll
        for (int u = 0; u < NY * NX; ++u) {
            const float v = part[at[u] + ch * khw];
            sum += ok[u] ? v : 0.0f;
        }
        out[(int64_t)ch * HW] = sum;
    }
}

// ---- folding for every geometry (windows of more than three strides; such strides and windows that a
// tile's matrix rows do not fit LDS; images of fewer than four pixels): a workgroup has 32 pixels of the
// activation (of the batch's pixels in a row) and 64 channels.  Lanes are channels, so that the kh * kw
// elements a lane adds up for a pixel lie in the lines its neighbours read too, and which taps there are is
// the same for the whole wave; the sums turn through LDS and leave as runs of pixels.  The loads of a
// pixel's taps go out NY x NX at a time: all of them, or (NY = 1) along one row of a larger window.
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

namespace {

// Whether tiles are the faster way, us with a thread's column at a time / in tiles.  Over 1800 random geometries (half of
// them not looked at for the rule) all in tiles take 1.14 times as long as none (899 lose more than 5 %), with this rule
// 0.92 (95 lose).  A workgroup costs 0.9 ns whatever it writes: not where
// images hold few windows (18436 x 384 x 1 x 1, window 1, 17.2 / 106; 29865 x 208 x 1 x 2 19.7 / 142; 16384 x 64 x 2 x 2, window 3, 40 /
// 54) or little of X comes of them.  Of windows up to two wide a thread's column reads a line of every plane per
// element and tiles gain most (422 x 384 x 22 x 14, window 1, 298 / 107).  Wider ones share lines between the lanes; there tiles
// need pixels that several windows read (398 x 72 x 3 x 96, window 4, stride 4, 16.6 / 31.6; H = 1 with a window of 3 x 3, two
// thirds of them padding, 44 / 66) and workgroups for every CU (7 x 154 x 8 x 62, window 4, stride 2, 140 of them, 9.4 / 14.7).
bool unfold_tiles_pay(const Im2colArgs& a, int64_t windows, int64_t written, int64_t fetched, int64_t workgroups)
{
    if (windows < 16 || written < 1024) return false;
    return a.kw <= 2 || (2 * written >= 3 * fetched && workgroups >= 400);
}

// How the tiles are cut; false where a tile of one row of windows and four channels does not fit, or tiles do not pay.
// Tiles of whole matrix rows of an image where they are short, up to 128 of them and 64 KB of X (16 KB: 26 -> 31
// us for 64 x 32 x 32, window 3, stride 2); the channels that fit 32 KB then, but runs of at least 256 bytes.
bool plan_unfold_tile(const Im2colArgs& a, UnfoldTile* t, unsigned* grid, size_t* lds)
{
    const int64_t khw = (int64_t)a.kh * a.kw, most_floats = kTileLds / 4;
    const int64_t across = ((int64_t)a.Wo + 63) / 64, TX = ((int64_t)a.Wo + across - 1) / across;
    int64_t TY = 1;
    while (2 * TY * TX <= 128 && 2 * TY * TX * khw * (a.C < 16 ? a.C : 16) <= 16384 && TY < a.Ho) TY *= 2;
    // (coordinates of a tile's last window, also one behind the image, fit 32 bits)
    if (((int64_t)a.Ho + TY) * a.stride + a.kh >= INT_MAX || ((int64_t)a.Wo + TX) * a.stride + a.kw >= INT_MAX) return false;
    const int64_t sy = a.stride < a.kh ? a.stride : a.kh, sx = a.stride < a.kw ? a.stride : a.kw;
    for (; TY >= 1; TY /= 2) {
        const int64_t height = (TY - 1) * sy + a.kh, width = (TX - 1) * sx + a.kw;
        for (int64_t most = 64; most >= 4; most /= 2) {
            const int64_t CB = most < a.C ? most : a.C, seg = (CB * khw + 3) / 4 * 4, floats = seg + CB * height * width;
            if (floats > most_floats) continue;
            if (CB < a.C && CB * khw * 4 < 256 && TY > 1) break;
            const int64_t blocks = (a.C + CB - 1) / CB, down = (a.Ho + TY - 1) / TY, batch = a.M / ((int64_t)a.Ho * a.Wo);
            if (across * down > kTiles || across * down * blocks > kTiles / batch) return false;
            const int64_t windows = TX * (TY < a.Ho ? TY : a.Ho);
            if (!unfold_tiles_pay(a, windows, windows * CB * khw, CB * height * width, across * down * blocks * batch)) return false;
            const auto div = [](int64_t d) { return make_divisor((uint32_t)d); };
            *t = {(int)TY, (int)CB, (int)sy, (int)sx, (int)(height * width), div(TX), div(across), div(down), div(blocks),
                  div(width), div(height), div(sy), div(sx), div(khw), div(a.kw), div(CB * khw / 4)};
            *grid = (unsigned)(across * down * blocks * batch);
            *lds = (size_t)floats * 4;
            return true;
        }
    }
    return false;
}

} // namespace

hipError_t launch_im2col(const Im2colArgs& a, hipStream_t stream)
{
    ProfileScope ps(K_IM2COL, stream);
    const int64_t K = (int64_t)a.C * a.kh * a.kw;
    UnfoldTile t;
    unsigned tiles;
    size_t lds;
    // (X itself is on a 16-byte boundary)
    if (K % 4 == 0 && plan_unfold_tile(a, &t, &tiles, &lds)) {
        hipLaunchKernelGGL(im2col_tile_kernel, dim3(tiles), dim3(kThreads), lds, stream, a, t);
        return hipGetLastError();
    }
    int log2w = 5;
    while (log2w < 8 && (1 << log2w) < K) ++log2w;
    const int width = 1 << log2w;
    const int64_t tall = (int64_t)(kThreads / width) * kRows;
    const int64_t n_col = (K + width - 1) / width, runs = (a.M + tall - 1) / tall;
    hipLaunchKernelGGL(im2col_kernel, dim3((unsigned)(n_col * runs)), dim3(kThreads), 0, stream, a, width, log2w,
                       (uint32_t)n_col);
    return hipGetLastError();
}

namespace {

// How the tiles are cut; false where a tile of one pixel row and four channels does not fit, or has too few pixels.
// Tiles of whole image rows where they are short, up to 128 pixels (64 or 256: 32.6 and 26.7 us for 128 x 64 x
// 32 x 32, window 3, stride 2, which takes 26.7; its 1 x 1 neighbour 9.8 and 11.8 against 8.6); the channels
// that fit 32 KB then (48 KB: 13.4 -> 13.7 and 9.3 -> 10.4 us at 16 x 16 and 4 x 4 images), but runs of a line
// at least (of 512 bytes: tiles of two rows for 96 x 14 x 14, window 3, 46 us instead of 26).
bool plan_fold_tile(const Im2colArgs& a, FoldTile* t, unsigned* grid, size_t* lds)
{
    const int64_t khw = (int64_t)a.kh * a.kw, most_rows = kTileLds / 4;
    const int64_t across = ((int64_t)a.W + 63) / 64, TX = ((int64_t)a.W + across - 1) / across;
    int64_t TY = 1;
    while (2 * TY * TX <= 128 && TY < a.H) TY *= 2;
    const auto rows = [&](int64_t pixels, int k, int out) {
        const int64_t r = (pixels + k - 2) / a.stride + 1;
        return r < out ? r : (int64_t)out;
    };
    for (; TY >= 1; TY /= 2) {
        const int64_t ny = rows(TY, a.kh, a.Ho), nx = rows(TX, a.kw, a.Wo);
        if (ny > most_rows || nx > most_rows || ny * nx > most_rows || khw > most_rows) continue;
        for (int64_t most = 64; most >= 4; most /= 2) {
            const int64_t CB = most < a.C ? most : a.C;
            int64_t pitch = (CB * khw + 3) / 4 * 4;
            if (pitch % 8 == 0) pitch += 4;      // (an odd number of 16-byte units: a column's rows in different banks)
            if (ny * nx * pitch * 4 > kTileLds) continue;
            if (CB < a.C && CB * khw * 4 < 128 && TY > 1) break;
            const int64_t blocks = (a.C + CB - 1) / CB, down = (a.H + TY - 1) / TY, batch = a.M / ((int64_t)a.H * a.W);
            const bool wide = a.C * khw % 4 == 0;
            if (across * down > kTiles || across * down * blocks > kTiles / batch) return false;
            // (a workgroup for three pixels: 18436 x 384 x 1 x 1, window 1, 44 / 101 us, 38580 x 144 x 1 x 1, window 3, 60 / 150.  Of
            // 1800 random geometries 93 lose more than 5 % without this line, 13 with it)
            if (TX * (TY < a.H ? TY : a.H) < 4) return false;
            int log2p = 0;
            while ((1 << log2p) < TX * TY) ++log2p;
            *t = {(int)TY, log2p, (int)CB, (int)pitch, (int)nx, make_divisor((uint32_t)TX), make_divisor((uint32_t)a.stride),
                  make_divisor((uint32_t)across), make_divisor((uint32_t)down), make_divisor((uint32_t)blocks),
                  make_divisor((uint32_t)(wide ? CB * khw / 4 : CB * khw)), make_divisor((uint32_t)nx)};
            *grid = (unsigned)(across * down * blocks * batch);
            *lds = (size_t)(ny * nx * pitch * 4);
            return true;
        }
    }
    return false;
}

template <int N>
void launch_fold_tile(const Im2colArgs& a, const FoldTile& t, unsigned grid, size_t lds, hipStream_t stream)
{
    const bool wide = (int64_t)a.C * a.kh * a.kw % 4 == 0;      // (X itself is on a 16-byte boundary)
    if (wide) hipLaunchKernelGGL((col2im_tile_kernel<N, N, true>), dim3(grid), dim3(kThreads), lds, stream, a, t);
    else hipLaunchKernelGGL((col2im_tile_kernel<N, N, false>), dim3(grid), dim3(kThreads), lds, stream, a, t);
}

} // namespace

hipError_t launch_col2im(const Im2colArgs& a, hipStream_t stream)
{
    ProfileScope ps(K_COL2IM, stream);
    // (strides up to 2^31 - 1: no sum)
    const int ny = (a.kh - 1) / a.stride + 1, nx = (a.kw - 1) / a.stride + 1, n = ny > nx ? ny : nx;
    FoldTile t;
    unsigned tiles;
    size_t lds;
    if (n <= 3 && plan_fold_tile(a, &t, &tiles, &lds)) {
        if (n == 1) launch_fold_tile<1>(a, t, tiles, lds, stream);
        else if (n == 2) launch_fold_tile<2>(a, t, tiles, lds, stream);
        else launch_fold_tile<3>(a, t, tiles, lds, stream);
        return hipGetLastError();
    }
    const int64_t runs = (a.M + kFoldPixels - 1) / kFoldPixels;
    const unsigned across = (unsigned)((a.C + kFoldChannels - 1) / kFoldChannels);
    const dim3 grid((unsigned)(runs < (1 << 23) ? runs : (1 << 23)), across);
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
