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
#include "common.hpp"

#include <type_traits>

namespace hdqt {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kTile = 128;                  // rows and columns of a workgroup's part of the output
constexpr int kStage = 128;                 // codes of a row in a stage
constexpr int kPanelBytes = kTile * kStage; // a stage of one operand
constexpr int kStageBytes = 2 * kPanelBytes;
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kBring = kTile / 8 / kWaves;  // loads of a wave per stage and operand, eight lines each
constexpr uint32_t kOutside = 0x80000000u;

struct BytesArgs {
    const uint8_t *qA, *qB;
    int64_t pitch, RA, RB, D;
    uint32_t n_rt, n_ct, tiles, per_xcd;
    Divisor group, out_tiles;
    uint32_t stages_per_tile, part_stages;
    int lo, hi;
    const float *scaleA, *scaleB;
    float inv_n;
    float* out;
    int32_t *acc_out, *partial;
};

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
__global__ __launch_bounds__(kThreads, kStages == 2 ? 2 : 1) void gemm_bytes_kernel(BytesArgs g)
{
    __shared__ __align__(16) uint8_t lds[kStages * kStageBytes];
    // Workgroups go to the eight XCDs in turn: each gets a run of tiles of its own (part by part of a split contraction), in
    // groups of eight rows of tiles column by column, whose panels its L2 holds.
    const uint32_t idx = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
    if (idx >= g.tiles) return;
    const uint32_t share = divide(idx, g.out_tiles), it = idx - share * g.out_tiles.d;
    const uint32_t grp = divide(it, g.group), in = it - grp * g.group.d;
    const uint32_t tall = g.n_rt - 8 * grp < 8 ? g.n_rt - 8 * grp : 8, ct = in / tall, rt = 8 * grp + in - ct * tall;
    const uint32_t stages_all = (uint32_t)((g.D + kStage - 1) / kStage), s_begin = share * g.part_stages;
    const uint32_t n_stages = stages_all - s_begin < g.part_stages ? stages_all - s_begin : g.part_stages;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = wave >> 1, wc = wave & 1;
    // a wave brings eight rows at a time, eight lanes to a row
    auto left = [&](int64_t rows, int64_t first) {
        const int64_t n = (rows - first) * g.pitch - (int64_t)s_begin * kStage;
        return (int)(n < (int64_t)kOutside ? n : (int64_t)kOutside - 1);
    };
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(g.qA + (int64_t)rt * kTile * g.pitch + (int64_t)s_begin * kStage), 0, left(g.RA, (int64_t)rt * kTile), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(g.qB + (int64_t)ct * kTile * g.pitch + (int64_t)s_begin * kStage), 0, left(g.RB, (int64_t)ct * kTile), 0x00020000);
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
    const int64_t d_left = g.D - (int64_t)s_begin * kStage;
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

    // Stores through a descriptor that ends with the output: rows beyond it are dropped by the range check, columns by an
    // offset outside (a branch around every store was 1 us of a small product: 40 KB of instructions).
    const int64_t row0 = (int64_t)rt * kTile + wr * 64, col0 = (int64_t)ct * kTile + wc * 64, at0 = row0 * g.RB + col0;
    const int64_t room = 4 * (g.RA * g.RB - at0);
    const int bytes = room <= 0 ? 0 : (int)(room < (int64_t)kOutside ? room : (int64_t)kOutside - 1);
    uint32_t lane_off[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t col = 32 * j + (lane & 31);
        lane_off[j] = col0 + col < g.RB ? 4 * (4 * (lane >> 5) * (uint32_t)g.RB + (uint32_t)col) : kOutside;
    }
    auto store = [&](void* base, auto value, auto nt) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(base) + 4 * at0, 0, bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    __builtin_amdgcn_raw_buffer_store_b32(value(tot[i][j][r]), rs, lane_off[j] + 4 * (32 * i + 8 * (r >> 2) + (r & 3)) * (uint32_t)g.RB, 0, nt.value);
    };
    auto number = [](int acc) { return (uint32_t)acc; };
    auto scaled = [scale](int acc) { return __float_as_uint((float)acc * scale); };
    if (g.partial) {
        store(g.partial + (int64_t)share * g.RA * g.RB, number, std::integral_constant<int, 0>{});
        return;
    }
    if (g.out) store(g.out, scaled, std::integral_constant<int, STREAM ? 2 : 0>{});
    if (g.acc_out) store(g.acc_out, number, std::integral_constant<int, 0>{});
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
    const int64_t tiles = ((g.RA + kTile - 1) / kTile) * ((g.RB + kTile - 1) / kTile) * g.splits;
    return gemm_fast_eligible(g) && (tiles + 7) * kThreads < ((int64_t)1 << 32);
}

hipError_t launch_gemm_bytes(const GemmArgs& g, hipStream_t stream)
{
    BytesArgs k{};
    k.qA = g.qA; k.qB = g.qB; k.pitch = g.pitchA; k.RA = g.RA; k.RB = g.RB; k.D = g.D;
    k.n_rt = (uint32_t)((g.RA + kTile - 1) / kTile); k.n_ct = (uint32_t)((g.RB + kTile - 1) / kTile);
    k.tiles = k.n_rt * k.n_ct * (uint32_t)g.splits;
    k.per_xcd = (k.tiles + 7) / 8;
    k.group = make_divisor(8 * k.n_ct);
    k.out_tiles = make_divisor(k.n_rt * k.n_ct);
    k.stages_per_tile = (uint32_t)((g.s + kStage - 1) / kStage);
    k.part_stages = (uint32_t)((g.tiles_per_split * g.s + kStage - 1) / kStage);
    k.lo = g.acc_lo; k.hi = g.acc_hi;
    k.scaleA = g.scaleA; k.scaleB = g.scaleB; k.inv_n = g.inv_n;
    k.out = g.out; k.acc_out = g.acc_out; k.partial = g.splits > 1 ? g.partial : nullptr;
    ProfileScope ps(g.profile_tag ? K_GEMM_I4_FWD + (g.profile_tag - 1) : K_GEMM_I4, stream);
    const dim3 grid(8 * k.per_xcd), block(kThreads);
    if (g.stream_out) hipLaunchKernelGGL((gemm_bytes_kernel<true, 2>), grid, block, 0, stream, k);
    else if (k.tiles <= 256) hipLaunchKernelGGL((gemm_bytes_kernel<false, 3>), grid, block, 0, stream, k);
    else hipLaunchKernelGGL((gemm_bytes_kernel<false, 2>), grid, block, 0, stream, k);
    return hipGetLastError();
}

} // namespace hdqt
