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
// bounds the long contractions is the clamp, one vector instruction per sum and half of it on the matrix pipe: 4096 cubed of
// codes that fill their range 125.5 / 128.5.
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
constexpr int kStages = 3;                          // in LDS

// TEST_32: CLAMP_32 where a tile is asked first whether it can saturate at all (see below)
enum Clamp { CLAMP_32, CLAMP_64, CLAMP_NONE, TEST_32 };

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

// The same, times 256, plus 255 for each of the two that saturates upwards.
__device__ __forceinline__ int add_clamped_scaled(int total, int p0, int p1)
{
    const v2s ones = {1, 1};
    return __builtin_amdgcn_sdot2(__builtin_amdgcn_cvt_pk_i16(p0, p1), ones, total, false);
}

// TEST_32.  A tile whose sums provably stay inside the accumulator is not clamped: by Cauchy and Schwarz |sum a_k b_k| <=
// sqrt(sum a_k^2 sum b_k^2), so with nA the largest sum of squares over a wave's lines of A in this tile and nB over its lines of
// B, nA nB <= 127^2 means that none of them can, and the matrix core adds the tile straight onto the totals.  These carry the
// factor 256 of the opened codes throughout; a clamped tile that saturates upwards adds 32767 where 127 * 256 is meant, 255 too
// many, so a total is 256 (T + p) - p with p <= 255 of them (at most 255 tiles a part): p = -total mod 256.
// A wave squares the lines that it brought itself, 32 of either operand, at the end of the stage before: its own loads are all
// it waits for, and the next barrier makes the largest sums known along with the codes.  A workgroup whose first stage holds a tile
// that has to be clamped asks no more: codes that fill their range pass nowhere, and then the test is pure cost.
// Largest sums of squares, by stage (even, odd), operand, wave that brought the lines, tile and quarter of the lines:
constexpr int kNormWords = 16, kNorms = 2 * 2 * kWaves * kNormWords;
struct Quad { v4i u[4]; };
__device__ __forceinline__ Quad read_own(uint32_t a, uint32_t b)
{
    Quad q;
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:1024\n\tds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:1024\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(q.u[0]), "=&v"(q.u[1]), "=&v"(q.u[2]), "=&v"(q.u[3])
                 : "v"(a), "v"(b)
                 : "memory");
    return q;
}
__device__ __forceinline__ void lds_write(uint32_t at, int v)
{
    asm volatile("ds_write_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" ::"v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ int lds_read(uint32_t at)
{
    int v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(at) : "memory");
    return v;
}
__device__ __forceinline__ int squares(v4i w)
{
    int n = __builtin_amdgcn_sdot8(w[0], w[0], 0, false);
    n = __builtin_amdgcn_sdot8(w[1], w[1], n, false);
    n = __builtin_amdgcn_sdot8(w[2], w[2], n, false);
    return __builtin_amdgcn_sdot8(w[3], w[3], n, false);
}
template <int CTRL>
__device__ __forceinline__ int max_dpp(int x)
{
    const int y = __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
    return x > y ? x : y;
}

template <int CLAMP, bool STREAM, bool NARROW, bool MASK, bool TAIL>
__global__ __launch_bounds__(kThreads, NARROW ? 4 : MASK || TAIL ? 2 : 3) void lines_gemm_i4_kernel(LinesArgs g)
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
    v16i sum[kBlocks][2] = {};           // CLAMP_NONE, TEST_32
    uint32_t buf = 0;
    bring(0, 0);
    if (at.n_stages > 1) bring(1, kStageBytes);
    // TEST_32: where the largest sums are, and the word that says that the test was given up
    [[maybe_unused]] __shared__ int norms[CLAMP == TEST_32 ? kNorms + 1 : 1];
    const uint32_t norm0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)norms, norm_off = norm0 + 4 * kNorms;
    // the largest sums of squares of the wave's own lines of the stage in `from`, to the words of stage s
    [[maybe_unused]] auto square_own = [&](uint32_t s, uint32_t from) {
        const uint32_t own = lds0 + from + wave * 2048 + lane * 16;
        const Quad q = read_own(own, own + kPanelA);
        const int a0 = squares(q.u[0]), a1 = squares(q.u[1]), b0 = squares(q.u[2]), b1 = squares(q.u[3]);
        int na = a0 > a1 ? a0 : a1, nb = b0 > b1 ? b0 : b1;
        // (a lane's piece is the line's number (lane % 4) ^ (lane / 16 % 4): the sixteen lines of a load, four to sixteen lanes)
        na = max_dpp<0x124>(max_dpp<0x128>(na));       // row_ror:8, row_ror:4
        nb = max_dpp<0x124>(max_dpp<0x128>(nb));
        const uint32_t quarter = (lane >> 4) & 3, tile = (lane & 3) ^ quarter, w = (s & 1) * (2 * kWaves) + wave;
        const int second = (lane & 4) != 0;            // lanes 0-3 of sixteen write A's, lanes 4-7 B's
        if ((lane & 8) == 0) lds_write(norm0 + 4 * ((w + second * kWaves) * kNormWords + tile * 4 + quarter), second ? nb : na);
    };
    bool clamped = false;                 // (wave-uniform) some tile went through the clamp
    uint32_t s = 0;
    if constexpr (CLAMP == TEST_32) {
        if (threadIdx.x == 0) lds_write(norm_off, 0);
        if (at.n_stages > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBringA + kBringB) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        square_own(0, 0);
        for (; s < at.n_stages; ++s) {
            // (the wave's own part of the stage has arrived: its lines were squared)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (s && __builtin_amdgcn_readfirstlane(lds_read(norm_off))) break;      // (the same in every wave)
            const uint32_t after = buf == 2 * kStageBytes ? 0 : buf + kStageBytes;
            if (s + 2 < at.n_stages) bring(s + 2, buf == 0 ? 2 * kStageBytes : buf - kStageBytes);
            // lanes 0-31 the two waves that brought the wave's lines of A, lanes 32-63 those of B
            const int op = lane >> 5, from = 2 * (op ? wc : wr) + ((lane >> 4) & 1);
            int m = lds_read(norm0 + 4 * (((s & 1) * 2 + op) * kWaves * kNormWords + from * kNormWords + (lane & 15)));
            m = max_dpp<0x4E>(max_dpp<0xB1>(m));       // the four quarters of the lines
            const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)m, (uint32_t)m, false, false);
            m = (int)(r16[0] > r16[1] ? r16[0] : r16[1]);
            int any_no = 0;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int a0 = __builtin_amdgcn_readlane(m, 8 * p), a1 = __builtin_amdgcn_readlane(m, 8 * p + 4);
                const int b0 = __builtin_amdgcn_readlane(m, 32 + 8 * p), b1 = __builtin_amdgcn_readlane(m, 36 + 8 * p);
                // Two flags whose relation the compiler cannot see: as if and else the two ways of updating the totals meet in a
                // join that copies all of them on both sides.
                const int ok = __builtin_amdgcn_readfirstlane((a0 * b0 <= 127 * 127 && a1 * b1 <= 127 * 127) ? 1 : 0);
                int no;
                asm volatile("s_xor_b32 %0, %1, 1" : "=s"(no) : "s"(ok) : "scc");
                any_no |= no;
                Codes22 q;
                read_steps((fa + buf) ^ (32 * p), (fb + buf) ^ (32 * p), q);
                v4i a[2][2], b[2][2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i) { a[i][t] = open(q.a[i][t]); b[i][t] = open(q.b[i][t]); }
                if (ok) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j)
                                sum[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][t], b[j][t], sum[i][j], 0, 0, 0);
                }
                if (no) {
                    clamped = true;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const v16i p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][0], b[j][0], zero, 0, 0, 0);
                            const v16i p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][1], b[j][1], zero, 0, 0, 0);
#pragma unroll
                            for (int r = 0; r < 16; ++r) sum[i][j][r] = add_clamped_scaled(sum[i][j][r], p0[r], p1[r]);
                        }
                }
            }
            if (s == 0 && any_no && lane == 0) lds_write(norm_off, 1);
            if (s + 1 < at.n_stages) {
                if (s + 2 < at.n_stages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBringA + kBringB) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                square_own(s + 1, after);
            }
            buf = after;
        }
        if (s < at.n_stages) clamped = true;
    }
    const uint32_t s_given_up = s;
    for (; s < at.n_stages; ++s) {
        // The stage has arrived (every wave waits for its own part of it), and nobody reads the buffer any more that the next
        // loads go to: a wave's reads of it were waited for where they stand.
        // (TEST_32 gives up behind a stage's barrier)
        if (CLAMP != TEST_32 || s != s_given_up) {
            if (s + 1 < at.n_stages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBringA + kBringB) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        if (s + 2 < at.n_stages) bring(s + 2, buf == 0 ? 2 * kStageBytes : buf - kStageBytes);
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
                            for (int r = 0; r < 16; ++r) {
                                if constexpr (CLAMP == TEST_32) sum[i][j][r] = add_clamped_scaled(sum[i][j][r], p0[r], p1[r]);
                                else tot[i][j][r] = add_clamped(tot[i][j][r], p0[r], p1[r]);
                            }
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        buf = buf == 2 * kStageBytes ? 0 : buf + kStageBytes;
    }
    if constexpr (CLAMP == CLAMP_NONE || CLAMP == TEST_32) {
#pragma unroll
        for (int i = 0; i < kBlocks; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    // (exact: products carry the factor 16 * 16)
                    const int v = sum[i][j][r], p = CLAMP == TEST_32 && clamped ? -v & 255 : 0;
                    tot[i][j][r] = ((v + p) >> 8) - p;
                }
    }
    write_totals<STREAM, MASK, kBlocks, 2>(g.to, at.share, rowA + wr * 32 * kBlocks, rowB + wc * 64, lane, scale, tot);
}

} // namespace

// Workgroups with tiles of 128 x 128.
static int64_t wide_workgroups(const GemmArgs& g) { return ((g.RA + 127) / 128) * ((g.RB + 127) / 128) * g.splits; }

// Tiles of 128 x 64 for up to 64 columns, and where those of 128 x 128 would be two to a CU at most: eight waves there do not
// hide a stage's trip (32768 x 128 x 320 9.7 / 9.0, 8192 x 512 x 256 8.7 / 8.0, 320 x 128 x 32768 in parts 16.2 / 14.8, 4096 x 1152 x 128
// 9.8 / 10.0).  Where nothing is clamped the second reading of A's lines shows, and the line comes earlier (23845 x 192 x 4096, 374
// workgroups, 32.7 / 30.6, 174 x 16256 x 1024, 254, 9.9 / 9.1, but 18995 x 373 x 1088, 447, 15.0 / 16.5, 8404 x 832 x 5640, 462, 49.8 / 62.0).
static bool narrow_tiles(const GemmArgs& g) { return g.RB <= 64 || wide_workgroups(g) <= (g.acc_hi == 127 ? 512 : 384); }

// What gemm_i4_kernel keeps of these: lines that are no whole dwords, bfloat16 outputs, parts of no whole stages (tiles of 96 or
// 160 codes), a mask behind lines that end inside 32 codes, and, of the products whose tiles are asked whether they can saturate,
// those whose lines end inside 32 codes (a line's last piece brings codes of the next line, and the testing loop has no place to
// clear them before they are squared) and those of up to 512 workgroups: eight waves each do better there than four (65536 x
// 128 x 1152, test passed 19.6 / 20.5, failed 24.4 / 26.3; with clamps and tiles of 128 x 64 24.0 and 24.2), not beyond: of 60 drawn
// products this kernel takes 0.83 of the time in the median where the test passes and 0.96 to 0.98 where it does not, 1.07 at the worst
// (131072 x 128 x 576 passed 26.9 / 25.0, 2496 x 5179 x 6016 178 / 190 on codes with a deviation of 1.5, 4096 cubed 125.5 / 132 on
// those, 125.5 / 128.5 on uniform ones and 86 / 85 passed).  Of 331 drawn products (3- and 4-bit codes, 32 to
// 168000 rows and columns, contractions of 8 to 16384) the 170 that come here are faster by 27 to 38 % in the median; the one
// class that is not is a narrow output's very long contraction in parts (576 x 64 x 262144 32.0 / 32.9, x 131072 21.7 / 21.4).
bool gemm_packed_eligible(const GemmArgs& g)
{
    if (g.bA > 4 || g.bB > 4 || g.fold || g.out_bf16) return false;
    if (g.D % 8 != 0 || (g.D % 32 != 0 && g.mask_src)) return false;
    const bool clamped = g.acc_hi == 127 && (g.s == 32 || g.s == 64), plain = g.acc_hi == INT_MAX && g.s % 32 == 0;
    if (!(clamped || plain) || (gemm_fast_tests_tiles(g) && (g.D % 32 != 0 || wide_workgroups(g) <= 512))) return false;
    return gemm_fast_eligible(g) && lines_fit(g, kRows, narrow_tiles(g) ? 64 : 128, kStage);
}

hipError_t launch_gemm_packed(const GemmArgs& g, hipStream_t stream)
{
    const bool narrow = narrow_tiles(g), masked = g.mask_src != nullptr, tail = g.D % 32 != 0;
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
    if (gemm_fast_tests_tiles(g)) {
        if (g.stream_out) hipLaunchKernelGGL((lines_gemm_i4_kernel<TEST_32, true, false, false, false>), grid, block, 0, stream, k);
        else hipLaunchKernelGGL((lines_gemm_i4_kernel<TEST_32, false, false, false, false>), grid, block, 0, stream, k);
    } else if (clamp == CLAMP_32) HDQT_PACKED(CLAMP_32);
    else if (clamp == CLAMP_64) HDQT_PACKED(CLAMP_64);
    else HDQT_PACKED(CLAMP_NONE);
#undef HDQT_PACKED
#undef HDQT_PACKED3
    return hipGetLastError();
}

} // namespace hdqt
