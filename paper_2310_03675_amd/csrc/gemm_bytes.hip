// Integer matmul of codes with a byte each (5 to 8 bits), in tiles that are whole stages of 128 codes or one tile (gfx950).
//
// A workgroup of four waves has a 128 x 128 tile of the output, a wave 64 x 64 of it (2 x 2 MFMA blocks, running tile and
// totals apart).  A stage is 128 codes of every line: whole 128-byte lines, eight lanes to a line, straight to LDS
// (buffer_load ... lds); codes need no unpacking.  What bounds it (4096 cubed, parts of the kernel left out in a scratch copy):
// the MFMAs alone take 54 us, at the clock the chip holds on full-range bytes, the loads alone 55, the LDS reads 34, all of it
// 81.  With stages of 64 codes the loads alone were 80 us: a load costs a CU by the lines it touches, not by its bytes.
// A 256 x 128 tile of eight waves with three stages in LDS moves less (48) and ends where this one does (86 us), and
// wastes more at an output's edges.  gemm_i4_kernel, which brings codes through registers: 4096 cubed, tiles of 256 in 16
// bits, 104 us, here 88; 3000 x 3100 x 2992 72 / 57; 512 x 4608 x 2048 in four parts 26.2 / 24.3.
#include "gemm_lines.hpp"

#include <type_traits>

namespace hdqt {

namespace {

using namespace lines;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kTile = 128;                  // rows and columns of a workgroup's part of the output
constexpr int kStage = 128;                 // codes of a row in a stage
constexpr int kPanelBytes = kTile * kStage; // a stage of one operand
constexpr int kStageBytes = 2 * kPanelBytes;
constexpr int kWaves = kThreads / 64;
constexpr int kBring = kTile / 8 / kWaves;  // loads of a wave per stage and operand, eight lines each

// four fragments of one 32-code step: two blocks of 32 rows on either side
// (One statement with its own wait: the compiler would have reads of LDS wait for every load on its way there, the next
// stage's too.  The wait hides behind the products of the step before.)
struct Step { v4i a0, a1, b0, b1; };
__device__ __forceinline__ Step read_step(uint32_t a, uint32_t b)
{
    Step s;
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %2, %5\n\tds_read_b128 %1, %4 offset:4096\n\tds_read_b128 %3, %5 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(s.a0), "=&v"(s.a1), "=&v"(s.b0), "=&v"(s.b1)
                 : "v"(a), "v"(b)
                 : "memory");
    return s;
}

// kStages in LDS: two, with two workgroups on a CU, or three where there is one workgroup for a CU at most, which has
// nothing else to do while its next stage is on its way.
template <bool STREAM, int kStages>
__global__ __launch_bounds__(kThreads, kStages == 2 ? 2 : 1) void gemm_bytes_kernel(LinesArgs g)
{
    __shared__ __align__(1024) uint8_t lds[kStages * kStageBytes];
    const Place p = place_of(g, kStage);
    if (!p.there) return;
    const uint32_t n_stages = p.n_stages;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = wave >> 1, wc = wave & 1;
    // a wave brings eight rows at a time, eight lanes to a row
    const int64_t rowA = (int64_t)p.rt * kTile, rowB = (int64_t)p.ct * kTile, begin = (int64_t)p.s_begin * kStage;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.qA + rowA * g.pitch + begin), 0,
                                                                         bytes_left(g.RA, rowA, g.pitch, begin), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.qB + rowB * g.pitch + begin), 0,
                                                                         bytes_left(g.RB, rowB, g.pitch, begin), 0x00020000);
    const int lrow = lane >> 3;
    // The piece of a row that goes to a lane's place is its number turned by the row's, so that a fragment's reads
    // spread over the banks (two rows of LDS are all banks once).
    const int turn = (lane >> 4) & 3;
    uint32_t off[2], code[2];               // of even and odd groups of eight rows
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        code[j] = 16 * ((lane & 7) ^ (turn + 4 * j));
        off[j] = (uint32_t)(lrow + 8 * j) * (uint32_t)g.pitch + code[j];
    }
    const int64_t d_left = g.D - begin;
    const uint32_t hop = wave * kBring * 8 * (uint32_t)g.pitch;
    auto bring = [&](uint32_t s, uint32_t at) {
        uint32_t o[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) o[j] = (int64_t)s * kStage + code[j] < d_left ? off[j] + s * kStage : kOutside;
#pragma unroll
        for (int j = 0; j < kBring; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsA, (__attribute__((address_space(3))) void*)(lds + at + (wave * kBring + j) * 1024), 16,
                o[j & 1] + (hop + (j >> 1) * 16 * (uint32_t)g.pitch), 0, 0, 0);
#pragma unroll
        for (int j = 0; j < kBring; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsB, (__attribute__((address_space(3))) void*)(lds + at + kPanelBytes + (wave * kBring + j) * 1024), 16,
                o[j & 1] + (hop + (j >> 1) * 16 * (uint32_t)g.pitch), 0, 0, 0);
    };

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int frow = lane & 31;
    const uint32_t k0 = 16 * ((lane >> 5) ^ ((frow >> 1) & 7));
    const uint32_t fa = lds0 + (wr * 64 + frow) * kStage, fb = lds0 + kPanelBytes + (wc * 64 + frow) * kStage;

    const float scale = *g.scaleA * *g.scaleB * g.inv_n;
    const v16i zero = {};
    v16i part[2][2] = {};
    int tot[2][2][16] = {};
    uint32_t at = 0;
    auto stage = [&](uint32_t s, auto fresh) {
        // The stage has arrived (every wave waits for its own part of it), and nobody reads the buffer any more that the next
        // loads go to: a wave's reads of it were waited for where they stand.
        if (kStages > 2 && s + 1 < n_stages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kBring) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t before = at == 0 ? (kStages - 1) * kStageBytes : at - kStageBytes;
        if (s + kStages - 1 < n_stages) bring(s + kStages - 1, before);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const Step q = read_step(fa + at + (k0 ^ (32 * k)), fb + at + (k0 ^ (32 * k)));
            const bool f = fresh.value && k == 0;
            part[0][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(q.a0, q.b0, f ? zero : part[0][0], 0, 0, 0);
            part[1][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(q.a1, q.b0, f ? zero : part[1][0], 0, 0, 0);
            part[0][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(q.a0, q.b1, f ? zero : part[0][1], 0, 0, 0);
            part[1][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(q.a1, q.b1, f ? zero : part[1][1], 0, 0, 0);
        }
        at = at == (kStages - 1) * kStageBytes ? 0 : at + kStageBytes;
    };
    bring(0, 0);
    if (kStages > 2 && n_stages > 1) bring(1, kStageBytes);
    for (uint32_t s = 0; s < n_stages;) {
        const uint32_t end = s + g.stages_per_tile < n_stages ? s + g.stages_per_tile : n_stages;
        stage(s, std::true_type{});
        for (++s; s < end; ++s) stage(s, std::false_type{});
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int v = part[i][j][r], t = v < g.lo ? g.lo : v;
                    tot[i][j][r] += t > g.hi ? g.hi : t;
                }
    }

    write_totals<STREAM, false, 2, 2>(g.to, p.share, rowA + wr * 64, rowB + wc * 64, lane, scale, tot);
}

} // namespace

// Of 148 products with 5- to 8-bit codes, drawn over 32 to 150000 rows and columns and contractions of 128 to 32768, in one part
// and in many, that this kernel multiplies instead of gemm_i4_kernel it is faster for all but one, by 26 % in the median (us,
// that one first: 65536 x 1152 x 128 65 / 55, 4096 x 1000 x 4096 45.3 / 38.4, 1152 x 128 x 65536 34.0 / 28.3, 8192 x 4096 x 256 41.9 / 28.3).
// The one is an output larger than the memory-side cache, whose rows are neither whole lines nor many tiles wide: 153856 x 425 x 256
// 83 / 95, x 512 117 / 125, but 110000 x 425 x 512 85 / 53, 153856 x 448 x 512 113 / 71, 65536 x 1150 x 256 83 / 76.
// (Masks are applied by the pass behind it, as for gemm_i4_kernel's byte codes; bfloat16 outputs, tiles that are no whole stages
// and lines that are no whole 16-byte pieces stay there.)
bool gemm_bytes_eligible(const GemmArgs& g)
{
    if (g.bA <= 4 || g.bB <= 4 || g.fold || g.out_bf16) return false;
    if (g.D % 16 != 0 || (g.n_tiles > 1 && g.s % kStage != 0)) return false;
    if (!g.stream_out && g.splits == 1 && g.RB <= 4 * kTile && 4 * g.RA * g.RB > ((int64_t)240 << 20)) return false;
    return gemm_fast_eligible(g) && lines_fit(g, kTile, kTile, kStage);
}

hipError_t launch_gemm_bytes(const GemmArgs& g, hipStream_t stream)
{
    const LinesArgs k = lines_args(g, kTile, kTile, kStage);
    ProfileScope ps(g.profile_tag ? K_GEMM_I4_FWD + (g.profile_tag - 1) : K_GEMM_I4, stream);
    const dim3 grid(8 * k.per_xcd), block(kThreads);
    if (g.stream_out) hipLaunchKernelGGL((gemm_bytes_kernel<true, 2>), grid, block, 0, stream, k);
    else if (k.tiles <= 256) hipLaunchKernelGGL((gemm_bytes_kernel<false, 3>), grid, block, 0, stream, k);
    else hipLaunchKernelGGL((gemm_bytes_kernel<false, 2>), grid, block, 0, stream, k);
    return hipGetLastError();
}

} // namespace hdqt
