// Integer matmul of packed codes whose lines go straight to LDS (gfx950): 8-bit accumulators over tiles of 32 or 64, and tiles
// that cannot saturate.
//
// A workgroup of four waves has a 128 x 128 tile of the output (128 x 64 up to 64 columns), a wave 64 x 64 (32 x 64) of it; a
// stage is 128 codes of every line, packed as they are, brought by buffer_load ... lds.  A wave opens the codes it multiplies:
// six instructions per fragment and step, against sixteen clamps per block.  12 or 16 KB a stage leave room for three stages and
// three or four workgroups on a CU, which is what short contractions of wide outputs want: one workgroup's stores run under
// the others' loads and clamps, and an XCD writes a run of the output of its own.  gemm_i4_kernel (two workgroups of eight
// waves, codes opened on their way to LDS, a workgroup walking along its strip of the output) / this one, us: 65536 x 1152 x 128
// 66.6 / 56.6 (302 MB of stores: 5.3 TB/s), 8192 x 4096 x 128 38.5 / 26.7, 40000 x 425 x 256 28.1 / 17.3, 262144 x 64 x 576 34.4 / 30.6,
// 2048 x 4608 x 512 20.4 / 17.7, 320 x 128 x 32768 in parts 18.6 / 15.7; tiles that cannot saturate 68160 x 576 x 672 70 / 41.  What
// bounds the long contractions is the clamp, one vector instruction per sum and half of it on the matrix pipe: 4096 cubed
// 136 / 125.
#include "gemm_lines.hpp"

#include <type_traits>

namespace hdqt {

namespace {

using namespace lines;

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef short v2s __attribute__((ext_vector_type(2)));

constexpr int kStage = 128, kLine = kStage / 2;     // codes of a line in a stage, and their bytes
constexpr int kRows = 128, kWaves = 4;

enum Clamp { CLAMP_32, CLAMP_64, CLAMP_NONE };

// The packed codes of two 32-code steps of the wave's blocks, 8 bytes a lane and step: step 0 at `a` and `b` in LDS, step 1 in
// the next piece of 16 bytes.  (One statement with its own wait: the compiler would have reads of LDS wait for every load on
// its way there, the next stages' too.  The wait hides behind the products of the steps before.)
struct Codes22 { v2i a[2][2], b[2][2]; };
__device__ __forceinline__ void read_steps(uint32_t a, uint32_t b, Codes22& r)
{
    asm volatile("ds_read_b64 %0, %8\n\tds_read_b64 %4, %9\n\tds_read_b64 %1, %10\n\tds_read_b64 %5, %11\n\t"
                 "ds_read_b64 %2, %8 offset:2048\n\tds_read_b64 %6, %9 offset:2048\n\t"
                 "ds_read_b64 %3, %10 offset:2048\n\tds_read_b64 %7, %11 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r.a[0][0]), "=&v"(r.a[0][1]), "=&v"(r.a[1][0]), "=&v"(r.a[1][1]), "=&v"(r.b[0][0]), "=&v"(r.b[0][1]),
                   "=&v"(r.b[1][0]), "=&v"(r.b[1][1])
                 : "v"(a), "v"(b), "v"(a ^ 16u), "v"(b ^ 16u)
                 : "memory");
}
struct Codes12 { v2i a[1][2], b[2][2]; };
__device__ __forceinline__ void read_steps(uint32_t a, uint32_t b, Codes12& r)
{
    asm volatile("ds_read_b64 %0, %6\n\tds_read_b64 %2, %7\n\tds_read_b64 %1, %8\n\tds_read_b64 %3, %9\n\t"
                 "ds_read_b64 %4, %7 offset:2048\n\tds_read_b64 %5, %9 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r.a[0][0]), "=&v"(r.a[0][1]), "=&v"(r.b[0][0]), "=&v"(r.b[0][1]), "=&v"(r.b[1][0]), "=&v"(r.b[1][1])
                 : "v"(a), "v"(b), "v"(a ^ 16u), "v"(b ^ 16u)
                 : "memory");
}

// 16 codes as bytes of 16 * code, even positions first (the same order on either side)
__device__ __forceinline__ v4i open(v2i w)
{
    const uint32_t m = 0xF0F0F0F0u, x = (uint32_t)w[0], y = (uint32_t)w[1];
    return v4i{(int)((x << 4) & m), (int)((y << 4) & m), (int)(x & m), (int)(y & m)};
}

// Two tiles' sums, times 256: saturated to 16 bits, their high bytes are the clamped sums.
__device__ __forceinline__ int add_clamped(int total, int p0, int p1)
{
    const v2s pk = __builtin_amdgcn_cvt_pk_i16(p0, p1);
    return __builtin_amdgcn_sdot4(__builtin_bit_cast(int, pk), 0x01000100, total, false);
}

template <int CLAMP, bool STREAM, bool NARROW, bool MASK, bool TAIL, int kStages = 3>
__global__ __launch_bounds__(kThreads, kStages > 3 ? 2 : NARROW ? 4 : MASK || TAIL ? 2 : 3) void lines_gemm_i4_kernel(LinesArgs g)
{
    constexpr int kCols = NARROW ? 64 : 128, kBlocks = NARROW ? 1 : 2;      // blocks of a wave one above the other; two side by side
    constexpr int kPanelA = kRows * kLine, kPanelB = kCols * kLine, kStageBytes = kPanelA + kPanelB;
    constexpr int kBringA = kRows / 16 / kWaves, kBringB = kCols / 16 / kWaves;      // loads of a wave per stage, sixteen lines each
    __shared__ __align__(1024) uint8_t lds[kStages * kStageBytes];
    const Place at = place_of(g, kStage);
    if (!at.there) return;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = NARROW ? wave : wave >> 1, wc = NARROW ? 0 : wave & 1;
    const int64_t rowA = (int64_t)at.rt * kRows, rowB = (int64_t)at.ct * kCols, begin = (int64_t)at.s_begin * kLine;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.qA + rowA * g.pitch + begin), 0,
                                                                         bytes_left(g.RA, rowA, g.pitch, begin), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.qB + rowB * g.pitch + begin), 0,
                                                                         bytes_left(g.RB, rowB, g.pitch, begin), 0x00020000);
    // The piece of a line that goes to a lane's place is its number turned by the line's, so that the reads of sixteen
    // lines' pieces spread over all banks (four lines of LDS are all banks once).
    const uint32_t piece = 16 * ((lane & 3) ^ ((lane >> 4) & 3)), off = (lane >> 2) * (uint32_t)g.pitch + piece;
    const int64_t line_left = g.pitch - begin;
    auto bring = [&](uint32_t s, uint32_t to) {
        const uint32_t o = (int64_t)s * kLine + piece < line_left ? off + s * kLine : kOutside;
#pragma unroll
        for (int j = 0; j < kBringA; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsA, (__attribute__((address_space(3))) void*)(lds + to + (wave * kBringA + j) * 1024), 16,
                o + (wave * kBringA + j) * 16 * (uint32_t)g.pitch, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < kBringB; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsB, (__attribute__((address_space(3))) void*)(lds + to + kPanelA + (wave * kBringB + j) * 1024), 16,
                o + (wave * kBringB + j) * 16 * (uint32_t)g.pitch, 0, 0, 0);
    };

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int frow = lane & 31;
    const uint32_t turn = 16 * ((frow >> 2) & 3) + 8 * (lane >> 5);
    const uint32_t fa = lds0 + (wr * 32 * kBlocks + frow) * kLine + turn, fb = lds0 + kPanelA + (wc * 64 + frow) * kLine + turn;

    const float scale = *g.scaleA * *g.scaleB * g.inv_n;
    const v16i zero = {};
    int tot[kBlocks][2][16] = {};
    v16i sum[kBlocks][2] = {};           // CLAMP_NONE
    uint32_t buf = 0;
    bring(0, 0);
#pragma unroll
    for (int k = 1; k < kStages - 1; ++k)
        if (at.n_stages > (uint32_t)k) bring(k, k * kStageBytes);
    for (uint32_t s = 0; s < at.n_stages; ++s) {
        // The stage has arrived (every wave waits for its own part of it), and nobody reads the buffer any more that the next
        // loads go to: a wave's reads of it were waited for where they stand.
        if (s + kStages - 2 < at.n_stages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 2) * (kBringA + kBringB)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + kStages - 1 < at.n_stages) bring(s + kStages - 1, buf == 0 ? (kStages - 1) * kStageBytes : buf - kStageBytes);
        std::conditional_t<NARROW, Codes12, Codes22> q[2];
        auto read = [&](int p) {
            read_steps((fa + buf) ^ (32 * p), (fb + buf) ^ (32 * p), q[p]);
            // codes behind the line's end (the next line's): nothing on one side is enough
            const int64_t valid = g.D - ((int64_t)(at.s_begin + s) * kStage + 64 * p + 16 * (lane >> 5));
            if (TAIL && (int64_t)(at.s_begin + s + 1) * kStage > g.D) {
#pragma unroll
                for (int i = 0; i < kBlocks; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int d = 0; d < 2; ++d)
                            if (32 * t + 8 * d >= valid) q[p].a[i][t][d] = 0;
            }
        };
        if constexpr (CLAMP == CLAMP_64) {
            read(0);
            read(1);
#pragma unroll
            for (int i = 0; i < kBlocks; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    v16i p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(open(q[0].a[i][0]), open(q[0].b[j][0]), zero, 0, 0, 0);
                    v16i p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(open(q[1].a[i][0]), open(q[1].b[j][0]), zero, 0, 0, 0);
                    p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(open(q[0].a[i][1]), open(q[0].b[j][1]), p0, 0, 0, 0);
                    p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(open(q[1].a[i][1]), open(q[1].b[j][1]), p1, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[i][j][r] = add_clamped(tot[i][j][r], p0[r], p1[r]);
                    __builtin_amdgcn_sched_barrier(0);      // (registers for one block's fragments)
                }
        } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                read(p);
                v4i a[kBlocks][2], b[2][2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
#pragma unroll
                    for (int i = 0; i < kBlocks; ++i) a[i][t] = open(q[p].a[i][t]);
#pragma unroll
                    for (int j = 0; j < 2; ++j) b[j][t] = open(q[p].b[j][t]);
                }
                if constexpr (CLAMP == CLAMP_NONE) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < kBlocks; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j)
                                sum[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][t], b[j][t], sum[i][j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const v16i p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][0], b[j][0], zero, 0, 0, 0);
                            const v16i p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][1], b[j][1], zero, 0, 0, 0);
#pragma unroll
                            for (int r = 0; r < 16; ++r) tot[i][j][r] = add_clamped(tot[i][j][r], p0[r], p1[r]);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        buf = buf == (kStages - 1) * kStageBytes ? 0 : buf + kStageBytes;
    }
    if constexpr (CLAMP == CLAMP_NONE) {
#pragma unroll
        for (int i = 0; i < kBlocks; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[i][j][r] = sum[i][j][r] >> 8;       // (exact: products carry the factor 16 * 16)
    }
    write_totals<STREAM, MASK, kBlocks, 2>(g.to, at.share, rowA + wr * 32 * kBlocks, rowB + wc * 64, lane, scale, tot);
}

} // namespace

// What gemm_i4_kernel keeps of these: tiles asked whether they can saturate (gemm_fast_tests_tiles), lines that are no whole
// dwords, bfloat16 outputs, and a mask behind lines that end inside 32 codes.  Of 331 drawn products (3- and 4-bit codes, 32 to
// 168000 rows and columns, contractions of 8 to 16384) the 170 that come here are faster by 27 to 38 % in the median; the one class that
// is not is a narrow output's very long contraction in parts (576 x 64 x 262144 32.0 / 32.9, x 131072 21.7 / 21.4).
bool gemm_packed_eligible(const GemmArgs& g)
{
    if (g.bA > 4 || g.bB > 4 || g.fold || g.out_bf16) return false;
    if (g.D % 8 != 0 || (g.D % 32 != 0 && g.mask_src)) return false;
    const bool clamped = g.acc_hi == 127 && (g.s == 32 || g.s == 64), plain = g.acc_hi == INT_MAX && g.s % 32 == 0;
    if (!(clamped || plain) || gemm_fast_tests_tiles(g)) return false;
    return gemm_fast_eligible(g) && lines_grid(g, kRows, g.RB <= 64 ? 64 : 128);
}

hipError_t launch_gemm_packed(const GemmArgs& g, hipStream_t stream)
{
    const bool narrow = g.RB <= 64, masked = g.mask_src && g.splits == 1, tail = g.D % 32 != 0;
    const LinesArgs k = lines_args(g, kRows, narrow ? 64 : 128, kStage);
    const int clamp = g.acc_hi != 127 ? CLAMP_NONE : g.s == 32 ? CLAMP_32 : CLAMP_64;
    ProfileScope ps(g.profile_tag ? K_GEMM_I4_FWD + (g.profile_tag - 1) : K_GEMM_I4, stream);
    const dim3 grid(8 * k.per_xcd), block(kThreads);
#define HDQT_PACKED3(CL, ST, NA)                                                                                       \
    do {                                                                                                               \
        if (tail) hipLaunchKernelGGL((lines_gemm_i4_kernel<CL, ST, NA, false, true>), grid, block, 0, stream, k);        \
        else if (masked) hipLaunchKernelGGL((lines_gemm_i4_kernel<CL, ST, NA, true, false>), grid, block, 0, stream, k); \
        else hipLaunchKernelGGL((lines_gemm_i4_kernel<CL, ST, NA, false, false>), grid, block, 0, stream, k);            \
    } while (0)
#define HDQT_PACKED(CL)                                                                                                \
    do {                                                                                                               \
        if (g.stream_out && narrow) HDQT_PACKED3(CL, true, true);                                                      \
        else if (g.stream_out) HDQT_PACKED3(CL, true, false);                                                          \
        else if (narrow) HDQT_PACKED3(CL, false, true);                                                                \
        else HDQT_PACKED3(CL, false, false);                                                                           \
    } while (0)
    if (clamp == CLAMP_32) HDQT_PACKED(CLAMP_32);
    else if (clamp == CLAMP_64) HDQT_PACKED(CLAMP_64);
    else HDQT_PACKED(CLAMP_NONE);
#undef HDQT_PACKED
#undef HDQT_PACKED3
    return hipGetLastError();
}

} // namespace hdqt
