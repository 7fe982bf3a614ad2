// Integer matmul of packed codes through the 6-bit floating-point matrix instructions (gfx950), for products that
// are large in all three dimensions.
//
// A 4-bit code is a 6-bit float (e2m3) exactly: patterns 0 .. 8 are the values 0, 1/8, .. 1 in equal steps, and the
// sign is a bit of its own.  Products of two are whole 64ths, and sums of 64 of them, and totals below 2^24, are exact
// in binary32, whatever the order.  v_mfma_scale_f32_32x32x64_f8f6f4 does twice the multiply-adds per cycle of
// v_mfma_i32_32x32x32_i8 on such operands, a tile of 64 codes is one instruction, and a fragment is 24 bytes a lane
// instead of 32.
//
// Two kernels.  expand_kernel lays the codes out as fragments: [panel of 128 rows][stage of 128 codes][half of a
// stage][block of 32 rows] of 1536 bytes, 16 bytes of each lane and then 8 of each, so that a stage of a panel is 12 KB in
// a row and goes to LDS without passing through registers.  gemm_six_kernel: a workgroup has a 128 x 128 tile of the
// output, eight waves of 64 x 32, stages double-buffered in LDS.
//
// What bounds it (counters, 8192 cubed): where tiles are clamped, vector issue and matrix pipe one after the other, busy in 75 and
// 28 % of the cycles; the fragment reads take 31 % of the LDS's.  Without clamps nothing is busy all the time, the LDS in
// 53 % of the cycles, the matrix pipe in 48: the waves spend 60 % of theirs waiting for the next stage and at its barrier.
// 8192 cubed with tiles of 64: gemm_i4_kernel 850 to 930 us, lines_gemm_i4_kernel 683, this one 470 to 540 and expand_kernel 34; without
// clamps 565, 454, and 320 to 350 and 34.  (Three stages in LDS, and waves of 64 x 64, change nothing where tiles are clamped.)
//
// Clamp of a 64-code tile to 8 bits: the sum arrives as (sum + 128.5) / 256, v_cvt_pknorm_u16_f32 clamps two of them
// to [0, 1] and leaves clamp(sum) + 128 in the high byte of each half ((q + 0.5) * 65535 / 256 lies in
// [256 q + 127, 256 q + 128] for q < 256), and v_msad_u8 adds 255 minus those two bytes to the total: one vector
// instruction per sum, as in gemm_i4_kernel, but none on the matrix pipe (its v_dot4c is).
#include "gemm_lines.hpp"

namespace hdqt {

namespace {

constexpr int kPanel = 128, kStage = 128;                   // rows and codes of a stage of one operand
constexpr int kBlockBytes = 1536, kStageBytes = 8 * kBlockBytes;
constexpr int kThreads = 512, kExpandThreads = 256;

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

struct SixArgs {
    const uint8_t *fA, *fB;          // fragments
    int64_t panel_bytes;             // of one panel: stages * kStageBytes
    uint32_t stages, n_rt, n_ct, per_xcd;
    Divisor group;                   // 8 * n_ct tiles
    const float *scaleA, *scaleB;
    float inv_n;
    lines::OutArgs to;
};

struct ExpandArgs {
    const uint8_t* codes[2];
    uint8_t* frags[2];
    int64_t rows[2], pitch, panel_bytes;
    uint32_t first, stages;          // workgroups of the first operand
};

// four nibbles (two's complement) in the low 16 bits -> four 6-bit floats in 24
__device__ __forceinline__ uint32_t six_of(uint32_t x)
{
    uint32_t y = (x & 0xFFu) | ((x & 0xFF00u) << 4);
    y = (y & 0x00F00Fu) | ((y & 0x0F00F0u) << 2);
    const uint32_t neg = (y >> 3) & 0x041041u;
    // (a nibble below zero: inverted and one added, at most 8, no carry)
    return ((y ^ (neg * 15u)) + neg) | (neg << 5);
}

// A wave turns 32 rows x 64 codes into one block; a workgroup's four waves read 128 bytes of every row.
__global__ __launch_bounds__(kExpandThreads) void expand_kernel(ExpandArgs e)
{
    const int which = blockIdx.x >= e.first;
    const uint32_t id = blockIdx.x - (which ? e.first : 0);
    // (two stages, four half stages, per workgroup)
    const uint32_t pairs = (e.stages + 1) / 2, rb = id / pairs, pair = id - rb * pairs;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t half = pair * 4 + wave, stage = half >> 1;
    if (stage >= e.stages) return;
    const int64_t row = (int64_t)rb * 32 + (lane & 31);
    uint4 c = make_uint4(0, 0, 0, 0);
    const int64_t at = (int64_t)half * 32 + (lane >> 5) * 16;
    if (row < e.rows[which] && at < e.pitch) c = *reinterpret_cast<const uint4*>(e.codes[which] + row * e.pitch + at);
    uint32_t s[8] = {six_of(c.x & 0xFFFFu), six_of(c.x >> 16), six_of(c.y & 0xFFFFu), six_of(c.y >> 16),
                     six_of(c.z & 0xFFFFu), six_of(c.z >> 16), six_of(c.w & 0xFFFFu), six_of(c.w >> 16)};
    uint32_t w[6];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        w[3 * k] = s[4 * k] | (s[4 * k + 1] << 24);
        w[3 * k + 1] = (s[4 * k + 1] >> 8) | (s[4 * k + 2] << 16);
        w[3 * k + 2] = (s[4 * k + 2] >> 16) | (s[4 * k + 3] << 8);
    }
    uint8_t* dst = e.frags[which] + (int64_t)(rb >> 2) * e.panel_bytes + (int64_t)stage * kStageBytes +
                   ((half & 1) * 4 + (rb & 3)) * kBlockBytes;
    *reinterpret_cast<uint4*>(dst + lane * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint2*>(dst + 1024 + lane * 8) = make_uint2(w[4], w[5]);
}

__device__ __forceinline__ v8i fragment(const uint8_t* block, int lane)
{
    const uint4 a = *reinterpret_cast<const uint4*>(block + lane * 16);
    // (volatile: the compiler would read this part of two fragments at once, and then move it to where it belongs)
    const v2i b = *(const volatile __attribute__((address_space(3))) v2i*)(block + 1024 + lane * 8);
    return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, b[0], b[1], 0, 0};
}

// scale bytes: 2^-1 on either side, so that products of codes (in 64ths) come out in 256ths; 1 without
template <bool SAT>
__device__ __forceinline__ v16f multiply(v8i a, v8i b, v16f c)
{
    constexpr int kScale = SAT ? 0x7E7E7E7E : 0x7F7F7F7F;
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, kScale, 0, kScale);
}

// SAT: tiles of 64 codes clamped to 8 bits; else plain sums.
template <bool SAT, bool STREAM>
__global__ __launch_bounds__(kThreads, 4) void gemm_six_kernel(SixArgs g)
{
    __shared__ __align__(16) uint8_t lds[2][2 * kStageBytes];
    // Workgroups go to the eight XCDs in turn: each gets a run of tiles of its own, in groups of eight rows of tiles
    // column by column, so that the 64 tiles it works on at a time share sixteen panels in its L2.
    const uint32_t idx = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
    if (idx >= g.n_rt * g.n_ct) return;
    const uint32_t grp = divide(idx, g.group), in = idx - grp * g.group.d;
    const uint32_t tall = g.n_rt - 8 * grp < 8 ? g.n_rt - 8 * grp : 8, ct = in / tall, rt = 8 * grp + in - ct * tall;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = wave >> 2, wc = wave & 3;
    // waves 0-3 bring A's panel, 4-7 B's, 3 KB each
    const uint8_t* src = wave < 4 ? g.fA + rt * g.panel_bytes + wave * 3072 : g.fB + ct * g.panel_bytes + (wave - 4) * 3072;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(src), 0, (int)(g.panel_bytes - (wave & 3) * 3072), 0x00020000);
    auto bring = [&](uint32_t s, int buf) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)&lds[buf][wave * 3072 + j * 1024], 16, lane * 16,
                (int)(s * kStageBytes) + j * 1024, 0, 0);
    };

    v16f base;
#pragma unroll
    for (int i = 0; i < 16; ++i) base[i] = SAT ? 128.5f / 256.0f : 0.0f;
    const float scale = *g.scaleA * *g.scaleB * g.inv_n;
    uint32_t tot[2][16] = {};
    v16f sum[2] = {base, base};
    auto stage = [&](uint32_t s, int buf) {
        // The stage has arrived (every wave waits for its own part of it, which the barrier alone does not ask for), and
        // nobody reads the other buffer any more: what a wave read of it has gone into its products.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const uint8_t* a0 = &lds[buf][2 * wr * kBlockBytes];
        const uint8_t* b0 = &lds[buf][kStageBytes + wc * kBlockBytes];
        const v8i b[2] = {fragment(b0, lane), fragment(b0 + 4 * kBlockBytes, lane)};
        const v8i a[2][2] = {{fragment(a0, lane), fragment(a0 + 4 * kBlockBytes, lane)},
                             {fragment(a0 + kBlockBytes, lane), fragment(a0 + 5 * kBlockBytes, lane)}};
        // (behind all reads of the stage: the compiler has reads of LDS wait for everything on its way there)
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < g.stages) bring(s + 1, buf ^ 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (SAT) {
                const v16f d0 = multiply<SAT>(a[i][0], b[0], base), d1 = multiply<SAT>(a[i][1], b[1], base);
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    tot[i][r] = __builtin_amdgcn_msad_u8(
                        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pknorm_u16(d0[r], d1[r])), 0xFF00FF00u, tot[i][r]);
                __builtin_amdgcn_sched_barrier(0);      // (registers for one block's sums)
            } else {
                sum[i] = multiply<SAT>(a[i][0], b[0], sum[i]);
                sum[i] = multiply<SAT>(a[i][1], b[1], sum[i]);
            }
        }
    };
    bring(0, 0);
    for (uint32_t s = 0; s < g.stages; s += 2) {
        stage(s, 0);
        if (s + 1 < g.stages) stage(s + 1, 1);
    }

    // (each of the 2 * stages tiles added 255 - (clamped sum + 128))
    int acc[2][1][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][0][r] = SAT ? (int)(254u * g.stages - tot[i][r]) : (int)(sum[i][r] * 64.0f);
    lines::write_totals<STREAM, false, 2, 1>(g.to, 0, (int64_t)rt * kPanel + wr * 64, (int64_t)ct * kPanel + wc * 32, lane, scale, acc);
}

} // namespace

int64_t gemm_six_bytes(const GemmArgs& g)
{
    const int64_t stages = (g.D + kStage - 1) / kStage;
    return ((g.RA + kPanel - 1) / kPanel + (g.RB + kPanel - 1) / kPanel) * stages * kStageBytes;
}

bool gemm_six_shape(int64_t RA, int64_t RB, int64_t D)
{
    return D % 32 == 0 && RA >= 256 && RB >= 256 && D >= 512;      // (rows of codes of whole 16-byte pieces)
}

// Against lines_gemm_i4_kernel, from 100 products of 12 to 120 10^9 multiply-adds and 2^39 (us, integer kernel / this one with
// expand_kernel): what it saves grows with the products, what it pays with the codes that are laid out anew and with the outputs,
// which it stores in pieces of 128 bytes (the other: 256).  Clamped 8192 cubed 683 / 508, 4096 cubed 88 / 78, 4137 x 4005 x 2080
// 60 / 53.5, 4736 x 2944 x 1216 32.3 / 34.0, 2432 x 14976 x 512 32.9 / 44.4; not clamped 8192 cubed 454 / 352, 10752 x 2048 x 3648
// 84 / 71, 4137 x 4005 x 2080 44.6 / 42.8, 4096 cubed 64.5 / 67.9, 3712 x 13568 x 768 47.1 / 63.9.  Of the 100 four fall on the
// wrong side, by up to 5 us (4096 x 4096 x 2048 not clamped 35.0 / 40.2).
static bool pays(const GemmArgs& g)
{
    const double codes = 1e-6 * (double)(g.RA + g.RB) * (double)g.D, outputs = 1e-6 * (double)g.RA * (double)g.RB;
    const double products = 1e-3 * outputs * (double)g.D;
    return g.acc_hi == 127 ? 0.382 * products - 3.3 - 0.11 * codes - 0.204 * outputs > 0.0
                           : 0.256 * products - 2.9 - 0.123 * codes - 0.197 * outputs > 0.0;
}

// The products that are multiplied here, whose workspaces hold the codes' other form.  (Two lines have to be passed: `pays`, where
// lines_gemm_i4_kernel is what multiplies otherwise -- not unclamped tiles of 24 or 33 codes, for which there is only the
// generic kernel, 6825 x 2768 x 1792 1987 / 54 us -- and the estimate that was drawn against gemm_i4_kernel, which multiplied them
// otherwise then: the least gain of outputs that fill whole half rounds of its workgroups still keeps products away of which
// `pays` makes next to nothing, 0.2 us for 2048 x 4096 x 2048 clamped.  Tiles of 128 or 256 in 8-bit accumulators, two and four
// chained instructions and fewer clamps, have no instance: nothing multiplies large products in them so far.)
bool gemm_six_eligible(const GemmArgs& g)
{
    if (!gemm_six_shape(g.RA, g.RB, g.D)) return false;
    if (g.bA > 4 || g.bB > 4 || g.splits > 1 || g.fold || g.mask_src || g.out_bf16) return false;
    const bool clamped = g.s == 64 && g.acc_lo == -128 && g.acc_hi == 127;
    const bool plain = g.acc_hi == INT_MAX && g.D <= 16384;      // totals of at most 2^20
    if (!(clamped || plain) || (gemm_packed_eligible(g) && !pays(g))) return false;
    const double codes = (double)(g.RA + g.RB) * (double)g.D, products = (double)g.RA * (double)g.RB * (double)g.D;
    const double gain = (clamped ? 7.5e-10 : 4.4e-10) * products - (clamped ? 6.5 : 8.0) - 2.8e-7 * codes;
    const int64_t stages = (g.D + kStage - 1) / kStage, n_rt = (g.RA + kPanel - 1) / kPanel, n_ct = (g.RB + kPanel - 1) / kPanel;
    double least = 0.0;
    if (n_rt * n_ct % 256 == 0 && (clamped || (g.RB >= g.RA && stages <= 8))) {
        least = 1.4 / 512 * (double)(n_rt * n_ct);
        if (clamped && least < 3.0) least = 3.0;
    }
    if (gain < least) return false;
    // a panel's bytes in 31 bits, and grids of less than 2^32 threads (with what they are rounded up by)
    return stages * kStageBytes < ((int64_t)1 << 31) && (n_rt * n_ct + 7) * kThreads < ((int64_t)1 << 32) &&
           4 * (n_rt + n_ct) * ((stages + 1) / 2) * kExpandThreads < ((int64_t)1 << 32);
}

hipError_t launch_gemm_six(const GemmArgs& g, void* frags, hipStream_t stream)
{
    SixArgs k{};
    k.stages = (uint32_t)((g.D + kStage - 1) / kStage);
    k.panel_bytes = (int64_t)k.stages * kStageBytes;
    k.n_rt = (uint32_t)((g.RA + kPanel - 1) / kPanel); k.n_ct = (uint32_t)((g.RB + kPanel - 1) / kPanel);
    k.per_xcd = (k.n_rt * k.n_ct + 7) / 8;
    k.group = make_divisor(8 * k.n_ct);
    k.fA = static_cast<uint8_t*>(frags); k.fB = k.fA + k.n_rt * k.panel_bytes;
    k.to = lines::out_args(g);
    k.scaleA = g.scaleA; k.scaleB = g.scaleB; k.inv_n = g.inv_n;
    ExpandArgs e{};
    e.codes[0] = g.qA; e.codes[1] = g.qB;
    e.frags[0] = static_cast<uint8_t*>(frags); e.frags[1] = e.frags[0] + k.n_rt * k.panel_bytes;
    e.rows[0] = g.RA; e.rows[1] = g.RB;
    e.pitch = g.pitchA; e.panel_bytes = k.panel_bytes; e.stages = k.stages;
    const uint32_t pairs = (k.stages + 1) / 2;
    e.first = 4 * k.n_rt * pairs;
    {
        ProfileScope ps(K_EXPAND, stream);
        hipLaunchKernelGGL(expand_kernel, dim3(e.first + 4 * k.n_ct * pairs), dim3(kExpandThreads), 0, stream, e);
    }
    ProfileScope ps(g.profile_tag ? K_GEMM_I4_FWD + (g.profile_tag - 1) : K_GEMM_I4, stream);
    const dim3 grid(8 * k.per_xcd), block(kThreads);
    const bool sat = g.acc_hi == 127;
    if (sat && g.stream_out) hipLaunchKernelGGL((gemm_six_kernel<true, true>), grid, block, 0, stream, k);
    else if (sat) hipLaunchKernelGGL((gemm_six_kernel<true, false>), grid, block, 0, stream, k);
    else if (g.stream_out) hipLaunchKernelGGL((gemm_six_kernel<false, true>), grid, block, 0, stream, k);
    else hipLaunchKernelGGL((gemm_six_kernel<false, false>), grid, block, 0, stream, k);
    return hipGetLastError();
}

} // namespace hdqt
