// Input gradient of a convolution, folded onto the activation (gfx950): the integer product of the
// codes of G [pixels, N] and W [C * kh * kw, N], its kh * kw columns of a channel added up where
// they meet in the activation, dequantized once.
//
//   dAct[b, c, y, x] = sum over taps (ty, tx) and tiles of N of
//                      clamp(sum over the tile of G[b, y - ty + ph, x - tx + pw, n] W[c, ty, tx, n])
//
// The sums over the tiles and over the taps are both plain integer sums, so a pixel and a channel
// have ONE contraction of kh * kw * N codes: the channel's line of W codes (its taps lie one behind
// the other) against the rows of G around the pixel, zeros outside the image.  Nothing is computed
// for halo pixels and no accumulator leaves its register before it is finished.  (Before, each
// workgroup multiplied a 128 x 128 tile of the unfolded product, halo rows included, wrote its
// accumulators to LDS and gathered nine of them per output: 174 us for 262144 x 576 x 64, bound by
// those passes through LDS and the barriers around them.)
//
// A workgroup owns 256 pixels and 64 channels; a wave 32 pixels and all 64 channels (two MFMA
// blocks, channels as rows, so that a store writes 32 neighbouring pixels).  Where that leaves CUs idle what counts
// is a wave's chain: half the channels and half the waves per workgroup, four times the workgroups.  W goes through LDS,
// unpacked once per workgroup, 256 codes of the contraction at a time, double-buffered; a wave's
// rows of G go straight to its registers, four steps ahead: the nine shifted reads of a row hit
// the CU's L1.  What is left is the clamp: one vector instruction per tile sum.

#include "common.hpp"

namespace hdqt {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef short v2s __attribute__((ext_vector_type(2)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

constexpr int kStep = 32;                 // codes per MFMA
constexpr int kChunk = 256;               // codes of the contraction per LDS buffer
constexpr int kSteps = kChunk / kStep;
constexpr int kAhead = 4;                 // steps of G in flight, and in hand
constexpr int kPitch = kChunk + 16;       // bytes of a channel's line in LDS
constexpr uint32_t kOutside = 0x80000000u;      // operands are smaller than 2 GB

static_assert(kSteps == 2 * kAhead, "a chunk is two groups of G");

__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const uint8_t* q, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(q), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ int clamp3(int v, int lo, int hi)      // (plain C++: see gemm_fast.hip)
{
    const int t = v < lo ? lo : v;
    return t > hi ? hi : t;
}

// SAT8: tiles of one step, 8-bit accumulators: two tile sums per saturating conversion, added by
// one dot product (see EPI_SAT8_S32 in gemm_fast.hip); else tiles of whole steps and a
// compare-select clamp, totals times 256.
// BLOCKS: 32-channel blocks of a workgroup; its waves are 4 per block (one 16-byte unit of W per thread and chunk).
template <bool SAT8, int BLOCKS>
__global__ __launch_bounds__(256 * BLOCKS, 4) void gemm_fold_kernel(GemmArgs g)
{
    constexpr int kBlocks = BLOCKS, kWaves = 4 * BLOCKS, kPixels = 32 * kWaves, kChannels = 32 * kBlocks;
    static_assert(kChannels * kSteps == 64 * kWaves, "one unit of W per thread and chunk");
    __shared__ __attribute__((aligned(16))) uint8_t Ws[2][kChannels][kPitch];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int N = (int)g.D, W = g.fW, H = g.fH, khw = g.fkh * g.fkw;
    const int ph = (g.fkh - 1) / 2, pw = (g.fkw - 1) / 2;
    const int total_codes = khw * N;
    const int pitch = N / 2;                                     // bytes of a line (N % 32 == 0)
    const __amdgpu_buffer_rsrc_t rsG = operand_rsrc(g.qA, g.RA * g.pitchA), rsW = operand_rsrc(g.qB, g.RB * g.pitchB);

    // ---- the lane's pixel
    const int64_t pixel = (int64_t)blockIdx.x * kPixels + wave * 32 + (lane & 31);
    const bool live = pixel < g.RA;
    const uint32_t hw = (uint32_t)(H * W);
    const uint32_t img = (uint32_t)pixel / hw, at = (uint32_t)pixel - img * hw;
    const int y = (int)(at / (uint32_t)W), x = (int)(at - (uint32_t)y * (uint32_t)W);

    // ---- the stream of G: eight bytes per lane and step, kAhead steps at a time
    int f_n = 0, f_ty = 0, f_tx = 0, f_left = total_codes;       // position of the next step
    uint32_t f_row = kOutside;                                   // byte of the source pixel's row
    auto locate = [&] {
        const int yy = y - f_ty + ph, xx = x - f_tx + pw;
        const bool ok = live && yy >= 0 && yy < H && xx >= 0 && xx < W;
        f_row = ok ? (uint32_t)((int)pixel + (ph - f_ty) * W + (pw - f_tx)) * (uint32_t)pitch + 8 * half : kOutside;
    };
    locate();
    auto fetch_g = [&](v2u (&v)[kAhead]) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            // (behind the end of the contraction: zeros)
            const uint32_t off = f_left > 0 && f_row != kOutside ? f_row + (uint32_t)(f_n >> 1) : kOutside;
            v[i] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rsG, off, 0, 0));
            f_left -= kStep;
            f_n += kStep;
            if (f_n >= N) {
                f_n = 0;
                if (++f_tx == g.fkw) { f_tx = 0; ++f_ty; }
                locate();
            }
        }
    };

    // ---- the stream of W: thread -> channel tid / 8 of the workgroup's, unit tid % 8 of the chunk
    const int w_row = tid >> 3, w_unit = tid & 7;
    const int64_t channel0 = (int64_t)blockIdx.y * kChannels;
    const bool w_live = channel0 + w_row < g.fC;
    const uint32_t w_line = w_live ? (uint32_t)(channel0 + w_row) * (uint32_t)(khw * pitch) + 16 * w_unit : 0u;
    int w_code = w_unit * kStep;                                 // of the next chunk's unit
    auto fetch_w = [&]() -> uint4 {
        const uint32_t off = w_live && w_code < total_codes ? w_line + (uint32_t)((w_code - w_unit * kStep) >> 1) : kOutside;
        w_code += kChunk;
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsW, off, 0, 0));
    };
    // codes times 16 as bytes, even positions first inside each eight bytes of the source, so that
    // a lane's 16 bytes of a step are those of the eight bytes of G it multiplies
    auto store_w = [&](const uint4& u, int buf) {
        const uint32_t m = 0xF0F0F0F0u;
        uint8_t* dst = &Ws[buf][w_row][w_unit * kStep];
        *reinterpret_cast<uint4*>(dst) = make_uint4((u.x << 4) & m, (u.y << 4) & m, u.x & m, u.y & m);
        *reinterpret_cast<uint4*>(dst + 16) = make_uint4((u.z << 4) & m, (u.w << 4) & m, u.z & m, u.w & m);
    };
    auto frag_w = [&](int buf, int block, int step) -> v4i {
        return *reinterpret_cast<const v4i*>(&Ws[buf][block * 32 + (lane & 31)][step * kStep + half * 16]);
    };
    auto frag_g = [&](v2u v) -> v4i {
        const uint32_t m = 0xF0F0F0F0u;
        return v4i{(int)((v[0] << 4) & m), (int)((v[1] << 4) & m), (int)(v[0] & m), (int)(v[1] & m)};
    };

    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    v16i total[kBlocks], part[kBlocks];
#pragma unroll
    for (int c = 0; c < kBlocks; ++c) { total[c] = zero; part[c] = zero; }
    const int lo = g.acc_lo_scaled, hi = g.acc_hi_scaled, s = (int)g.s;
    int m_n = 0, m_tile = 0;             // the multiplied step: codes into the tap, into the tile
    // steps `first` .. of the chunk in `buf`, `steps` of them (none behind the end of the contraction)
    auto multiply = [&](const v2u (&v)[kAhead], int buf, int first, int steps) {
        if constexpr (SAT8) {
#pragma unroll
            for (int i = 0; i < kAhead; i += 2) {
                if (i >= steps) break;   // (a step behind the end is zero on both sides)
                const v4i g0 = frag_g(v[i]), g1 = frag_g(v[i + 1]);
#pragma unroll
                for (int c = 0; c < kBlocks; ++c) {
                    const v16i p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(frag_w(buf, c, first + i), g0, zero, 0, 0, 0);
                    const v16i p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(frag_w(buf, c, first + i + 1), g1, zero, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const v2s pk = __builtin_amdgcn_cvt_pk_i16(p0[r], p1[r]);
                        total[c][r] = __builtin_amdgcn_sdot4(__builtin_bit_cast(int, pk), 0x01000100, total[c][r], false);
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                if (i >= steps) break;
                const v4i gf = frag_g(v[i]);
#pragma unroll
                for (int c = 0; c < kBlocks; ++c)
                    part[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(frag_w(buf, c, first + i), gf, part[c], 0, 0, 0);
                m_n += kStep;
                m_tile += kStep;
                const bool tap_ends = m_n >= N;
                if (tap_ends || m_tile >= s) {
                    m_tile = 0;
                    if (tap_ends) m_n = 0;
#pragma unroll
                    for (int c = 0; c < kBlocks; ++c) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) total[c][r] += clamp3(part[c][r], lo, hi);
                        part[c] = zero;
                    }
                }
            }
        }
    };

    // ---- chunk by chunk; one barrier each: a buffer is overwritten two chunks after it was filled,
    // behind the barrier that every wave passes when it has read it
    const int chunks = (total_codes + kChunk - 1) / kChunk;
    v2u even[kAhead], odd[kAhead];
    uint4 w_next = fetch_w();
    fetch_g(even);
    for (int q = 0; q < chunks; ++q) {
        store_w(w_next, q & 1);
        __syncthreads();
        w_next = fetch_w();
        const int left = (total_codes - q * kChunk) / kStep;
        fetch_g(odd);
        multiply(even, q & 1, 0, left);
        fetch_g(even);
        multiply(odd, q & 1, kAhead, left - kAhead);
    }

    if (!live) return;
    const float dq = (g.scaleA[0] * g.scaleB[0]) * g.inv_n;
    // from the workgroup's first image and channel: less than (kPixels + hw) * fC elements
    const uint32_t first = (uint32_t)((int64_t)blockIdx.x * kPixels), img0 = first / hw;
    const int64_t base = ((int64_t)img0 * g.fC + channel0) * hw;
    const int64_t off = (int64_t)(img - img0) * g.fC * hw + at + 4 * half * (int64_t)hw;
    auto value = [&](int c, int r) { return (float)(SAT8 ? total[c][r] : total[c][r] >> 8) * dq; };
    auto channel = [](int c, int r) { return 32 * c + 8 * (r >> 2) + (r & 3); };       // (of the lower half's lanes)
    if (channel0 + kChannels <= g.fC && !g.mask_src && (int64_t)(kPixels + hw) * g.fC < ((int64_t)1 << 31)) {
        // Nothing is tested per element and a store's address is a uniform one plus the lane's: the stores are one run.
#pragma unroll
        for (int c = 0; c < kBlocks; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) (g.out + base + (int64_t)channel(c, r) * hw)[(uint32_t)off] = value(c, r);
        return;
    }
#pragma unroll
    for (int c = 0; c < kBlocks; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (channel0 + channel(c, r) + 4 * half >= g.fC) continue;
            const int64_t o = base + (int64_t)channel(c, r) * hw + off;
            float f = value(c, r);
            if (g.mask_src && !(g.mask_src[o] > 0.0f)) f = 0.0f;
            g.out[o] = f;
        }
}

} // namespace

// What hdqt_conv_bwd promises to take, which is less than the kernel above could: it divides by any width
// and has neither row tiles nor 16-bit totals.  A caller takes a refusal as the sign to unfold, and the
// unfolded gradient is rounded term by term; which layers that concerns is part of their results.
bool gemm_fold_plan(GemmArgs* g, int64_t batch, int C, int H, int W, int kh, int kw)
{
    auto pow2 = [](int64_t v) { return v > 0 && (v & (v - 1)) == 0; };
    if (batch < 1 || C < 1 || H < 1 || W < 1 || kh < 1 || kw < 1 || kh % 2 == 0 || kw % 2 == 0) return false;
    if (!pow2(W) || W > 128 || kh * kw > 128 || kh > 15 || kw > 15) return false;
    if (g->RA != batch * (int64_t)H * W || g->RB != (int64_t)C * kh * kw || g->D % kStep != 0) return false;
    if (batch * (int64_t)C * H * W >= ((int64_t)1 << 40)) return false;
    // images of a power of two up to 128 pixels, images of 256, or rows so short that 128 pixels hold the
    // window's, and at most 65535 such pieces
    const int64_t hw = (int64_t)H * W;
    int64_t parts;
    if (hw <= 128) {
        if (!pow2(hw)) return false;
        parts = (batch + 128 / hw - 1) / (128 / hw);
    } else if (hw == 256 && kh * kw <= 9 && kh * kw > 1 && g->D <= 128 && batch <= 65535) {
        parts = batch;
    } else {
        const int rows_out = 128 / W - (kh - 1);
        if (rows_out < 1) return false;
        parts = batch * ((H + rows_out - 1) / rows_out);
    }
    if (parts > 65535) return false;
    // a pixel's and a column's total fits 16 bits; the kh * kw of them, times 256, then fit the kernel's 32
    const int64_t tile_sum = g->s * (((int64_t)1 << (g->bA - 1)) * ((int64_t)1 << (g->bB - 1)));
    const int64_t per_tile = tile_sum < (int64_t)g->acc_hi + 1 ? tile_sum : (int64_t)g->acc_hi + 1;
    if (per_tile > 32767 || per_tile * g->n_tiles > 32767) return false;
    g->splits = 1;
    g->tiles_per_split = g->n_tiles;
    g->fold = 1;
    g->fbatch = batch; g->fC = C; g->fH = H; g->fW = W; g->fkh = kh; g->fkw = kw;
    return gemm_fast_eligible(*g);
}

// Workgroups of 256 pixels and 64 channels below which the chip has too few of them.  Over 900 layers (windows of
// 1 x 1 to 5 x 5, 32 to 512 codes a tap), large workgroups / a quarter of that each, geometric means and ranges of the
// times' ratio: 1.53 (0.90 to 2.06) below 64 workgroups, 1.35 (1.02 to 1.94) below 128, 1.14 (0.88 to 1.93) below 192, 1.00 (0.72 to 1.44)
// from there to 255, 1.16 (0.73 to 1.77) at 256 to 340, where which is ahead changes with the layer.
constexpr int64_t kFewWorkgroups = 192;

hipError_t launch_gemm_fold(const GemmArgs& g_in, hipStream_t stream)
{
    GemmArgs g = g_in;
    const int64_t lo = (int64_t)g.acc_lo * 256, hi = (int64_t)g.acc_hi * 256;
    g.acc_lo_scaled = lo < INT32_MIN ? INT32_MIN : (int)lo;
    g.acc_hi_scaled = hi > INT32_MAX ? INT32_MAX : (int)hi;
    const int64_t wide = ((g.RA + 255) / 256) * ((g.fC + 63) / 64);
    const int blocks = wide < kFewWorkgroups ? 1 : 2;
    const dim3 grid((unsigned)((g.RA + 128 * blocks - 1) / (128 * blocks)), (unsigned)((g.fC + 32 * blocks - 1) / (32 * blocks)));
    const dim3 block(256 * blocks);
    ProfileScope ps(g.profile_tag ? K_GEMM_I4_FWD + (g.profile_tag - 1) : K_GEMM_I4, stream);
    const bool sat8 = g.s == kStep && g.acc_hi == 127;
    if (sat8 && blocks == 1) hipLaunchKernelGGL((gemm_fold_kernel<true, 1>), grid, block, 0, stream, g);
    else if (sat8) hipLaunchKernelGGL((gemm_fold_kernel<true, 2>), grid, block, 0, stream, g);
    else if (blocks == 1) hipLaunchKernelGGL((gemm_fold_kernel<false, 1>), grid, block, 0, stream, g);
    else hipLaunchKernelGGL((gemm_fold_kernel<false, 2>), grid, block, 0, stream, g);
    return hipGetLastError();
}

} // namespace hdqt
