// Integer matmul for products that cannot fill the chip with 128 x 128 tiles (gfx950).
//
// Same arithmetic as gemm_fast.hip: packed 4-bit codes or a byte per code, v_mfma_i32_32x32x32_i8,
// every tile of s codes clamped to the accumulator, 32-bit totals, dequantized once.
//
// What bounds these products is a chain, not a rate: with 128 x 128 tiles a layer of 128 x 561 x 561
// has five workgroups, each of whose SIMDs multiplies, clamps and adds 18 steps of 8 blocks one
// after the other (11 us), and a split contraction adds a launch.  Here a workgroup owns one
// block of 32 x 32 outputs and its four waves share the contraction between them, whole tiles
// each; the totals meet in LDS, so that nothing is left for a second launch.  The operands go
// from memory straight to the registers the matrix core reads (16 bytes a lane and load, halves of which change
// places across the wave), four steps ahead of the multiplication and without a barrier.  Every
// element is fetched once per 32 rows of the other operand: small products live in the L2 caches.
// Up to three products share a launch (a layer's forward product and both gradients).

#include "common.hpp"
#include "ragged.hpp"

#include <limits.h>
#include <type_traits>

namespace hdqt {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef short v2s __attribute__((ext_vector_type(2)));

constexpr int kStep = 32;            // codes per MFMA
constexpr int kWaves = 4;            // waves of a workgroup (eight: 2947 x 561 x 561 17.3 us instead of 13.7,
                                     // 4096 x 512 x 256 15.0 / 10.0, long contractions the same)

// MODE_TILES: tiles of whole steps, compare-select clamp.  MODE_SAT8: tiles of one step, 8-bit
// accumulators, packed codes: two tile sums per saturating conversion, added by one dot product
// (see EPI_SAT8_S32 in gemm_fast.hip).  MODE_HALF: tiles of 16 codes, two per step.
enum Mode { MODE_TILES = 0, MODE_SAT8 = 1, MODE_HALF = 2 };
constexpr int kModeWide = 4;

// How the codes come from memory: FETCH_LINES 16 bytes of a line of its own per lane, FETCH_RAGGED the same where
// lines do not start on a dword, FETCH_STAGED 64 bytes of a line per four lanes, through LDS.
enum Fetch { FETCH_LINES = 0, FETCH_RAGGED = 1, FETCH_STAGED = 2 };
constexpr int kStageLine = 80;               // bytes from line to line in LDS (of 64: the reads of eight lines meet no bank twice)
constexpr int kStage = 2 * 32 * kStageLine;  // bytes per wave (and its totals, in the end)

// codes at any byte address
struct __attribute__((packed)) Bytes4 { uint32_t v; };
struct __attribute__((packed)) Bytes8 { uint32_t x, y; };
struct __attribute__((packed, aligned(4))) Words4 { uint32_t w[4]; };

// The 8 bytes of codes at byte `at` of an operand, of which `codes` (any number, also none) lie
// inside their line, the others as zeros: the 8 bytes up to the line's end (or the operand's first 8,
// where that would begin in front of it; operands have at least 8), shifted into place.
template <bool WIDE>
__device__ __forceinline__ uint64_t load_tail(const uint8_t* q, uint32_t at, int codes)
{
    constexpr int kBits = WIDE ? 8 : 4;
    if (codes <= 0) return 0;
    if (codes > 64 / kBits) codes = 64 / kBits;
    const uint32_t bytes = (uint32_t)(codes * kBits + 7) / 8, end = at + bytes, start = end > 8 ? end - 8 : 0;
    const Bytes8 b = *reinterpret_cast<const Bytes8*>(q + start);
    const uint64_t w = ((uint64_t)b.y << 32 | b.x) >> (8 * (at - start));
    return codes * kBits == 64 ? w : w & (((uint64_t)1 << (codes * kBits)) - 1);
}

// A lane's 16 codes of a step: 2 dwords, 4 with a byte per code.  (One value, not an array: that
// way a group of them stays in registers whatever the branches around the loads.)
template <bool WIDE>
using Codes = uint32_t __attribute__((ext_vector_type(WIDE ? 4 : 2)));

// The step at code k: the lane's half of it, or (HALF) its halves of the step's two tiles.  `line` is
// the byte of the lane's line in the operand, `left` the codes of the line from k on (TAIL: fewer
// than a step's).
template <bool WIDE, bool HALF, bool TAIL>
__device__ __forceinline__ Codes<WIDE> load_step(const uint8_t* q, uint32_t line, int k, int half, int left)
{
    constexpr int N = WIDE ? 4 : 2, PER = HALF ? N / 2 : N;              // dwords, dwords of one run
    const uint32_t k_byte = (uint32_t)(WIDE ? k : k >> 1);
    const uint8_t* step = q + k_byte;                                    // (the same in every lane)
    Codes<WIDE> w;
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        // dwords i and i + 1: of one run, or (HALF, packed) one of either tile
        const int code = HALF ? 16 * (i / PER) + 8 * half : 16 * half + 4 * (WIDE ? i : 0);
        const uint32_t at = line + (uint32_t)(WIDE ? code : code >> 1);
        if constexpr (TAIL && PER == 1) {
            w[0] = (uint32_t)load_tail<WIDE>(q, k_byte + at, left - code);
            w[1] = (uint32_t)load_tail<WIDE>(q, k_byte + at + 8, left - code - 16);
        } else if constexpr (TAIL) {
            const uint64_t two = load_tail<WIDE>(q, k_byte + at, left - code);
            w[i] = (uint32_t)two;
            w[i + 1] = (uint32_t)(two >> 32);
        } else if constexpr (PER == 1) {
            w[0] = reinterpret_cast<const Bytes4*>(step + at)->v;
            w[1] = reinterpret_cast<const Bytes4*>(step + 8 + at)->v;
        } else {
            const Bytes8 two = *reinterpret_cast<const Bytes8*>(step + at);
            w[i] = two.x;
            w[i + 1] = two.y;
        }
    }
    return w;
}

// the upper half of the wave's v and the lower half's w change places
__device__ __forceinline__ void swap_halves(uint32_t v, uint32_t w, uint32_t& x, uint32_t& y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, w, false, false);
    x = r[0];
    y = r[1];
}

// N units of 32 bytes of a lane's line from byte k on, 16 bytes a lane: the lower half of the wave has a
// unit's first 16, the upper half the others.  What these loads cost is not their bytes but that every
// lane's are in a line of its own: with 8 bytes a lane a CU took some 80 cycles for each, three times
// what its matrix cores needed for the step.
// RAGGED: lines that do not start on a dword.  Loads of 16 bytes from such addresses cost twice, so the aligned
// dwords are fetched and shifted into place; the dword behind a lane's four is the first of the lane that
// has the next 16 bytes, and the last unit's upper half fetches its fourth whole from where it is.  (2074 x 355 x 555, packed: 7.3 us.)
template <bool RAGGED, int N>
__device__ __forceinline__ void load_units(const uint8_t* q, uint32_t line, uint32_t k, int half, Words4 (&out)[N])
{
    const uint8_t* p = q + k;                                            // (the same in every lane)
    const uint32_t at = RAGGED ? ragged_at(line, half) : line + 16 * (uint32_t)half, phase = line & 3u;
#pragma unroll
    for (int u = 0; u < N; ++u) out[u] = *reinterpret_cast<const Words4*>(p + (at + 32 * u));
    if constexpr (RAGGED) {
        const uint32_t last = reinterpret_cast<const Bytes4*>(p + ragged_last_at(line, 32 * N))->v;
        Words4 d[N];
#pragma unroll
        for (int u = 0; u < N; ++u) d[u] = out[u];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            uint32_t of_upper, of_lower;
            swap_halves(d[u].w[0], d[u + 1 < N ? u + 1 : u].w[0], of_lower, of_upper);
            const uint32_t next = half ? of_lower : of_upper;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[u].w[i] = __builtin_amdgcn_alignbyte(i < 3 ? d[u].w[i < 3 ? i + 1 : 3] : next, d[u].w[i], phase);
        }
        if (half) out[N - 1].w[3] = last;
    }
}

// A unit's codes: two steps of packed codes, one with a byte per code.  A lane has 16 consecutive bytes where
// the matrix core wants its share of either half: half the dwords change places with the other half of the wave.
template <bool WIDE, bool HALF>
__device__ __forceinline__ void unit_codes(const Words4& u, Codes<WIDE>* c)
{
    uint32_t x[4];
    if constexpr (!WIDE && HALF) {           // tiles of 16: dwords 0, 1 are the first tile's of the step, one per half
        swap_halves(u.w[0], u.w[1], x[0], x[2]);
        swap_halves(u.w[2], u.w[3], x[1], x[3]);
    } else if constexpr (!WIDE || HALF) {    // 16 bytes are a step, or a tile: two dwords per half
        swap_halves(u.w[0], u.w[2], x[0], x[2]);
        swap_halves(u.w[1], u.w[3], x[1], x[3]);
    } else {
        for (int i = 0; i < 4; ++i) x[i] = u.w[i];
    }
    if constexpr (WIDE) {
        c[0] = Codes<WIDE>{x[0], x[1], x[2], x[3]};
    } else {
        c[0] = Codes<WIDE>{x[0], x[1]};
        c[1] = Codes<WIDE>{x[2], x[3]};
    }
}

// the fragment(s) the matrix core wants: packed codes as bytes 16 * code, even positions first
template <bool WIDE>
__device__ __forceinline__ v4i whole(Codes<WIDE> w)
{
    if constexpr (WIDE) {
        return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
    } else {
        const uint32_t m = 0xF0F0F0F0u;
        return v4i{(int)((w[0] << 4) & m), (int)((w[1] << 4) & m), (int)(w[0] & m), (int)(w[1] & m)};
    }
}

template <bool WIDE>
__device__ __forceinline__ long tile_half(Codes<WIDE> w, int t)
{
    const uint32_t m = 0xF0F0F0F0u;
    v2i p;
    if constexpr (WIDE) p = t ? v2i{(int)w[2], (int)w[3]} : v2i{(int)w[0], (int)w[1]};
    else p = v2i{(int)(((t ? w[1] : w[0]) << 4) & m), (int)((t ? w[1] : w[0]) & m)};
    return __builtin_bit_cast(long, p);
}

__device__ __forceinline__ int clamp3(int v, int lo, int hi)      // (plain C++: see gemm_fast.hip)
{
    const int t = v < lo ? lo : v;
    return t > hi ? hi : t;
}

// One product as this kernel wants it: everything that is the same for all its workgroups is worked
// out on the host (a 64-bit division on the device is a hundred instructions), and the kernel has it in one
// trip to its arguments (2947 x 561 x 561, both passes of the quantizer included, 24.5 -> 22.0 us).
struct SmallArgs {
    const uint8_t *qA, *qB;
    const float *scaleA, *scaleB;
    float* out;
    uint16_t* out_bf16;
    int32_t* acc_out;
    const float* mask_src;
    int pitchA, pitchB, RA, RB, D;
    int acc_lo_scaled, acc_hi_scaled;
    float inv_n;
    int mode;                        // Mode, + kModeWide with a byte per code
    int unit, units;                 // what the waves share out (a tile, or a step), and how many there are
    int steps_per_tile;
    int ragged;                      // lines that do not start on a dword
    Divisor n_ct;                    // blocks along a row of the output
};

// (see common.hpp: the arguments in one go)
__device__ __forceinline__ SmallArgs whole_args(const SmallArgs& x)
{
    const SmallArgs g = x;
    asm volatile("" ::"s"(g.qA), "s"(g.qB), "s"(g.scaleA), "s"(g.scaleB), "s"(g.out), "s"(g.out_bf16), "s"(g.acc_out),
                 "s"(g.mask_src), "s"(g.pitchA), "s"(g.pitchB), "s"(g.RA), "s"(g.RB), "s"(g.D), "s"(g.acc_lo_scaled),
                 "s"(g.acc_hi_scaled), "s"(g.inv_n), "s"(g.mode), "s"(g.unit), "s"(g.units), "s"(g.steps_per_tile),
                 "s"(g.ragged),
                 "s"(g.n_ct.d), "s"(g.n_ct.mul), "s"(g.n_ct.sh1), "s"(g.n_ct.sh2));
    return g;
}

// The totals of a wave: the 32 x 32 block at (row0, col0), codes [k_begin, k_end), whole tiles.
//
// STAGED: chunks of 64 bytes of every line go through the wave's own piece of LDS, in which four lanes fetch a line's
// 64 bytes and two read them: a load's lanes then touch 16 lines instead of 32, and what a CU takes for it (77 cycles
// otherwise) no longer decides.  That costs every chain a trip through LDS per chunk, so it is for launches with
// enough of them per CU (launch_gemm_small).
template <bool WIDE, int MODE, int FETCH>
__device__ __forceinline__ v16i contract(const SmallArgs& g, int row0, int col0, int k_begin, int k_end, uint8_t* stage)
{
    constexpr bool RAGGED = FETCH == FETCH_RAGGED;
    constexpr bool HALF = MODE == MODE_HALF;
    // steps per group of loads (tiles of 16 keep the sums of two a step; staged: what is left of a chunk)
    constexpr int G = FETCH == FETCH_STAGED ? (WIDE ? 2 : 4) : WIDE || HALF ? 2 : 4;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    // (rows outside the operands: the last one, nothing of it is written)
    const int ra = row0 + (lane & 31), rb = col0 + (lane & 31);
    const uint32_t la = (uint32_t)(ra < g.RA ? ra : g.RA - 1) * (uint32_t)g.pitchA;
    const uint32_t lb = (uint32_t)(rb < g.RB ? rb : g.RB - 1) * (uint32_t)g.pitchB;
    struct Group {
        Codes<WIDE> a[G], b[G];
    };
    const int whole_steps = k_end > k_begin ? (k_end - k_begin) / kStep : 0, k_whole = k_begin + whole_steps * kStep;
    constexpr int PER_UNIT = WIDE ? 1 : 2, N = G / PER_UNIT;
    // a group of whole steps
    auto fetch = [&](Group& f, int k) {
        Words4 a[N], b[N];
        load_units<RAGGED, N>(g.qA, la, (uint32_t)(WIDE ? k : k >> 1), half, a);
        load_units<RAGGED, N>(g.qB, lb, (uint32_t)(WIDE ? k : k >> 1), half, b);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            unit_codes<WIDE, HALF>(a[u], f.a + u * PER_UNIT);
            unit_codes<WIDE, HALF>(b[u], f.b + u * PER_UNIT);
        }
    };
    // what is left of the whole steps, fewer than a group; behind them zeros (a tile of them adds nothing)
    auto fetch_rest = [&](Group& f, int k) {
#pragma unroll
        for (int i = 0; i < G; i += PER_UNIT) {
            const int at = k + kStep * i;
#pragma unroll
            for (int j = 0; j < PER_UNIT; ++j) f.a[i + j] = f.b[i + j] = 0;
            if (at + kStep * PER_UNIT <= k_whole) {
                Words4 a[1], b[1];
                load_units<RAGGED, 1>(g.qA, la, (uint32_t)(WIDE ? at : at >> 1), half, a);
                load_units<RAGGED, 1>(g.qB, lb, (uint32_t)(WIDE ? at : at >> 1), half, b);
                unit_codes<WIDE, HALF>(a[0], f.a + i);
                unit_codes<WIDE, HALF>(b[0], f.b + i);
            } else if (at < k_whole) {
                f.a[i] = load_step<WIDE, HALF, false>(g.qA, la, at, half, 0);
                f.b[i] = load_step<WIDE, HALF, false>(g.qB, lb, at, half, 0);
            }
        }
    };
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int lo = g.acc_lo_scaled, hi = g.acc_hi_scaled;
    const int steps_per_tile = g.steps_per_tile;
    int in_tile = 0;
    v16i total = zero, part = zero;          // part: the sums of the running tile (MODE_TILES)
    auto finish_tile = [&] {
        in_tile = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] += clamp3(part[r], lo, hi);
        part = zero;
    };
    // the first `valid` steps of a group count; COUNT: how many there are at most
    auto multiply = [&](const Group& f, int valid, auto count) {
        constexpr int COUNT = decltype(count)::value;
#pragma unroll
        for (int i = 0; i < COUNT; i += MODE == MODE_SAT8 ? 2 : 1) {
            if constexpr (MODE == MODE_SAT8) {
                const v16i p0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(whole<WIDE>(f.a[i]), whole<WIDE>(f.b[i]), zero, 0, 0, 0);
                v16i p1 = zero;
                if (i + 1 < COUNT) {
                    const int j = i + 1 < G ? i + 1 : 0;
                    p1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(whole<WIDE>(f.a[j]), whole<WIDE>(f.b[j]), zero, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const v2s pk = __builtin_amdgcn_cvt_pk_i16(p0[r], p1[r]);
                    total[r] = __builtin_amdgcn_sdot4(__builtin_bit_cast(int, pk), 0x01000100, total[r], false);
                }
            } else if constexpr (HALF) {
                const v16i p0 = __builtin_amdgcn_mfma_i32_32x32x16_i8(tile_half<WIDE>(f.a[i], 0), tile_half<WIDE>(f.b[i], 0), zero, 0, 0, 0);
                const v16i p1 = __builtin_amdgcn_mfma_i32_32x32x16_i8(tile_half<WIDE>(f.a[i], 1), tile_half<WIDE>(f.b[i], 1), zero, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r) total[r] += clamp3(p0[r], lo, hi) + clamp3(p1[r], lo, hi);
            } else {
                part = __builtin_amdgcn_mfma_i32_32x32x32_i8(whole<WIDE>(f.a[i]), whole<WIDE>(f.b[i]), part, 0, 0, 0);
                if (i < valid && ++in_tile == steps_per_tile) finish_tile();
            }
        }
    };
    Group now, next;
    if constexpr (FETCH == FETCH_STAGED) {
        constexpr int CHUNK = 2 * PER_UNIT * kStep;                      // codes of 64 bytes
        const int chunks = (k_whole - k_begin) / CHUNK, k_rest = k_begin + chunks * CHUNK;
        const int quarter = lane & 3, line = lane >> 2;
        const uint8_t *pa[2], *pb[2];                                    // lines `line` and line + 16
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = row0 + line + 16 * i, c = col0 + line + 16 * i;
            pa[i] = g.qA + ((uint32_t)(r < g.RA ? r : g.RA - 1) * (uint32_t)g.pitchA + 16 * quarter);
            pb[i] = g.qB + ((uint32_t)(c < g.RB ? c : g.RB - 1) * (uint32_t)g.pitchB + 16 * quarter);
        }
        Words4 r[4];
        auto load = [&](int k) {
            const int at = WIDE ? k : k >> 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                r[i] = *reinterpret_cast<const Words4*>(pa[i] + at);
                r[2 + i] = *reinterpret_cast<const Words4*>(pb[i] + at);
            }
        };
        uint8_t* put = stage + line * kStageLine + 16 * quarter;
        const uint8_t* take = stage + (lane & 31) * kStageLine + 16 * half;
        if (chunks) load(k_begin);
        for (int c = 0; c < chunks; ++c) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4*>(put + i * 16 * kStageLine) = make_uint4(r[i].w[0], r[i].w[1], r[i].w[2], r[i].w[3]);
            if (c + 1 < chunks) load(k_begin + (c + 1) * CHUNK);
            // LDS operations of one wave are carried out in order; the fences keep the compiler from moving
            // them across each other
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            Words4 u[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 x = *reinterpret_cast<const uint4*>(take + (i >> 1) * 32 * kStageLine + (i & 1) * 32);
                u[i] = Words4{{x.x, x.y, x.z, x.w}};
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                unit_codes<WIDE, HALF>(u[i], now.a);
                unit_codes<WIDE, HALF>(u[2 + i], now.b);
                multiply(now, PER_UNIT, std::integral_constant<int, PER_UNIT>{});
            }
        }
        if (k_rest < k_whole) fetch_rest(next, k_rest);
        if (k_rest < k_whole) multiply(next, (k_whole - k_rest) / kStep, std::integral_constant<int, G>{});
    } else {
        const int full = whole_steps / G;        // groups
        if (full) {
            // (the loop's loads are unconditional: the compiler can count them and waits for the older ones only)
            fetch(now, k_begin);
            for (int done = 1; done < full; ++done) {
                fetch(next, k_begin + done * G * kStep);
                multiply(now, G, std::integral_constant<int, G>{});
                now = next;
            }
        }
        const int rest = whole_steps - full * G;
        if (rest) fetch_rest(next, k_whole - rest * kStep);
        if (full) multiply(now, G, std::integral_constant<int, G>{});
        if (rest) multiply(next, rest, std::integral_constant<int, G>{});
    }
    if (k_whole < k_end) {                   // the line ends inside a step
        Group last{};
        last.a[0] = load_step<WIDE, HALF, true>(g.qA, la, k_whole, half, k_end - k_whole);
        last.b[0] = load_step<WIDE, HALF, true>(g.qB, lb, k_whole, half, k_end - k_whole);
        multiply(last, 1, std::integral_constant<int, 1>{});
    }
    if (MODE == MODE_TILES && in_tile) finish_tile();
    if (!WIDE && MODE != MODE_SAT8) {        // (exact: every sum carries the factor 16 * 16)
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] >>= 8;
    }
    return total;
}

struct SmallBatch {
    int first[kMaxSmallBatch];       // a product's first workgroup, INT_MAX behind the last product
    SmallArgs g[kMaxSmallBatch];
};

template <bool STAGED>
__global__ __launch_bounds__(64 * kWaves, 4) void gemm_small_kernel(SmallBatch b)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[kWaves][kStage];
    int p = 0, local = (int)blockIdx.x;
#pragma unroll
    for (int j = 1; j < kMaxSmallBatch; ++j) {
        const bool beyond = (int)blockIdx.x >= b.first[j];
        p = beyond ? j : p;
        local = beyond ? (int)blockIdx.x - b.first[j] : local;
    }
    const SmallArgs g = whole_args(b.g[p]);
    const int rt = (int)divide((uint32_t)local, g.n_ct), ct = local - rt * (int)g.n_ct.d;
    const int row0 = rt * 32, col0 = ct * 32;
    const float scaleA = g.scaleA[0], scaleB = g.scaleB[0];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));

    // the wave's share of the contraction
    const int k_begin = g.units * wave / kWaves * g.unit;
    int k_end = g.units * (wave + 1) / kWaves * g.unit;
    if (k_end > g.D) k_end = g.D;

    uint8_t* stage = lds[wave];
    v16i total;
#define HDQT_CONTRACT(WIDE, MODE)                                                                        \
    total = g.ragged ? contract<WIDE, MODE, FETCH_RAGGED>(g, row0, col0, k_begin, k_end, stage)                             \
                     : contract<WIDE, MODE, STAGED ? FETCH_STAGED : FETCH_LINES>(g, row0, col0, k_begin, k_end, stage)
    switch (g.mode) {
    case MODE_TILES: HDQT_CONTRACT(false, MODE_TILES); break;
    case MODE_SAT8: HDQT_CONTRACT(false, MODE_SAT8); break;
    case MODE_HALF:
        // (launch_gemm_small sends none to the staged kernel)
        if constexpr (STAGED) total = v16i{};
        else HDQT_CONTRACT(false, MODE_HALF);
        break;
    case MODE_TILES + kModeWide: HDQT_CONTRACT(true, MODE_TILES); break;
    default: HDQT_CONTRACT(true, MODE_HALF); break;
    }
#undef HDQT_CONTRACT

#pragma unroll
    for (int r = 0; r < 16; ++r) reinterpret_cast<int*>(stage)[r * 64 + lane] = total[r];
    __syncthreads();
    const float dq = (scaleA * scaleB) * g.inv_n;
    const int col = col0 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 16 / kWaves; ++i) {
        const int r = wave * (16 / kWaves) + i;
        int v = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) v += reinterpret_cast<const int*>(lds[w])[r * 64 + lane];
        const int row = row0 + 8 * (r >> 2) + (r & 3) + 4 * (lane >> 5);
        if (row < g.RA && col < g.RB) {
            const int64_t o = (int64_t)row * g.RB + col;
            float f = (float)v * dq;
            if (g.acc_out) g.acc_out[o] = v;
            if (g.out_bf16) g.out_bf16[o] = (uint16_t)bf16_bits(f);
            if (g.out) {
                if (g.mask_src && !(g.mask_src[o] > 0.0f)) f = 0.0f;
                g.out[o] = f;
            }
        }
    }
}

int mode_of(const GemmArgs& g)
{
    if (g.s < kStep) return MODE_HALF + (g.bA > 4 ? kModeWide : 0);
    if (g.bA <= 4 && g.s == kStep && g.acc_hi == 127) return MODE_SAT8;
    return MODE_TILES + (g.bA > 4 ? kModeWide : 0);
}

// What the waves share out: tiles, or steps where a step holds two tiles or nothing is clamped.
int64_t unit_of(const GemmArgs& g) { return g.s < kStep || g.acc_hi == INT_MAX ? kStep : g.s; }

// The products this kernel is the faster one for, by an estimate in us of what a call takes longer with it than
// with the large tiles' kernel (gemm_fast.hip, and the sum over a split contraction's parts): a sum over what
// the product has of
//   here: steps of a wave's chain; steps, and blocks, per CU; the same steps where lines do not start on a
//     dword; rounds of workgroups (four per CU) beyond the first;
//   there: stages in a row; the second launch, and the slices' elements (10^6), of a split; the output's elements;
//     the stages again where rows are no whole dwords; tiles per place of the chip;
// and a difference of what any launch takes.  The coefficients are least squares over 900 forward products and
// gradients of random sizes (outputs of 16 to 20000 rows and columns, contractions from 16 to 20000) and settings, each
// timed with its quantization and both kernels: the choice takes 0.3 % more time than the better of the two would,
// always this kernel 6.8 %, never 13.7 %.  Over others than the fit's, codes alone: 0.9 % over 250 of the
// same ranges, nothing over 200 with contractions of 20000 to 300000.  There / here: 3505 x 456 x 640 23.8 / 9.2 us, 667 x 320 x
// 2080 17.5 / 5.2, 467 x 3208 x 576 in tiles of 16 17.2 / 10.2, but 8513 x 1396 x 64 15.4 / 25.7, 250 x 200 x 64384 22 / 105.
// A product that shares its launch with others does not pay for one here (an empty kernel: 1.6 us).
// With a byte per code and long tiles a wave that gets fewer tiles than another leaves its SIMD idle, and the steps per
// CU are those of the longest share: 2304 x 586 x 16987 in one tile 149 / 292, 1920 x 600 x 5632 39 / 59.  Over 1005 such products
// in one to some dozen tiles the choice then takes 1.6 % more time than the better kernel, otherwise 3.3 %.  Not so with packed codes, whose long
// tiles cost less a step than the fit's short ones (28 x 115 x 16248 in one tile 94 / 46, 800 x 832 x 8384 54 / 28): there
// the even share is the better estimate (0.4 % against 2 to 21 %).
struct Estimate {
    double here[5], there[6], launch;
};
constexpr Estimate kEstimates[4] = {
    {{0.127, 0.0171, 0.316, 0.0080, 0.0}, {1.175, 2.70, 1.484, 0.0, 0.186, 1.746}, -3.12},          // MODE_SAT8
    {{0.172, 0.0159, 0.711, 0.0056, 0.800}, {0.565, 2.84, 1.223, 2.514, 0.083, 0.0}, -3.97},        // MODE_TILES
    {{0.295, 0.0252, 1.079, 0.0046, 0.348}, {1.802, 4.30, 1.081, 2.692, 0.0, 4.412}, -3.40},        // MODE_HALF
    {{0.229, 0.0316, 0.489, 0.0349, 1.323}, {1.228, 2.83, 0.315, 1.227, 0.698, 7.491}, -3.13}};     // a byte per code
constexpr double kLaunchUs = 1.6;

bool faster_here(const GemmArgs& g, bool alone)
{
    const bool wide = g.bA > 4, half = g.s < kStep, ragged = g.D % (wide ? 4 : 8) != 0;
    const Estimate& e = kEstimates[wide ? 3 : half ? 2 : mode_of(g) == MODE_SAT8 ? 0 : 1];
    const int64_t blocks = ((g.RA + 31) / 32) * ((g.RB + 31) / 32), steps = (g.D + kStep - 1) / kStep, rounds = (blocks + 1023) / 1024;
    // (masked outputs: 4096 x 640 x 128 takes 17.9 to 20.2 us here and 19.2 to 19.6 there, with the mask's own pass)
    if (g.mask_src && blocks > 2048) return false;
    const int64_t unit = unit_of(g), longest = ((g.D + unit - 1) / unit + kWaves - 1) / kWaves * (unit / kStep);
    const double busy = (double)(wide && unit > kStep ? kWaves * (longest < steps ? longest : steps) : steps);
    const double per_cu = (double)blocks / 256.0, outputs = 1e-6 * (double)g.RA * (double)g.RB;
    const double here = e.here[0] * (double)steps / kWaves + (e.here[1] + (g.pitchA % 4 != 0 ? e.here[3] : 0.0)) * busy * per_cu +
                        e.here[2] * per_cu + e.here[4] * (double)(rounds - 1) + e.launch - (alone ? 0.0 : kLaunchUs);
    const int64_t across = g.RB <= 64 && !wide && !half ? 64 : 128, stages = (steps + 3) / 4;
    const int64_t tiles = ((g.RA + 127) / 128) * ((g.RB + across - 1) / across), places = (tiles * g.splits + 511) / 512;
    const double in_a_row = (double)((stages + g.splits - 1) / g.splits * places);
    const double there = (e.there[0] + (ragged ? e.there[4] : 0.0)) * in_a_row + e.there[3] * outputs +
                         (g.splits > 1 ? e.there[1] + e.there[2] * g.splits * outputs : 0.0) + e.there[5] * (double)(tiles * g.splits) / 512.0;
    return here <= there;
}

// (32-bit offsets into the operands)
bool small_enough(const GemmArgs& g, bool alone)
{
    if ((g.RA + g.RB) * (g.pitchA + g.pitchB) >= ((int64_t)1 << 31)) return false;
    return faster_here(g, alone);
}

} // namespace

bool gemm_small_eligible(const GemmArgs& g, bool alone)
{
    if (g.fold || (g.bA > 4) != (g.bB > 4)) return false;      // packed or bytes, the same on both sides
    if (g.s != 16 && g.s % kStep != 0) return false;
    if (g.RA * g.pitchA < 8 || g.RB * g.pitchB < 8) return false;      // (see load_tail)
    if (mode_of(g) == MODE_SAT8) return small_enough(g, alone);       // unscaled totals: covered by the API's range check
    // a tile's sum and the totals, times 256 with packed codes, must stay inside int32
    const int64_t max_prod = ((int64_t)1 << (g.bA - 1)) * ((int64_t)1 << (g.bB - 1)), room = g.bA > 4 ? ((int64_t)1 << 31) : ((int64_t)1 << 23);
    const int64_t tile_max = g.s * max_prod, acc_max = (int64_t)g.acc_hi + 1;
    const int64_t n_tiles = (g.D + g.s - 1) / g.s;
    return tile_max < room && (tile_max < acc_max ? tile_max : acc_max) * n_tiles < room && small_enough(g, alone);
}

hipError_t launch_gemm_small(const GemmArgs* gs, int n, hipStream_t stream)
{
    if (n < 1 || n > kMaxSmallBatch) return hipErrorInvalidValue;
    SmallBatch b{};
    int64_t total = 0, work = 0, staged_blocks = 0;
    bool packed_halves = false, paired = true, all_aligned = true;
    for (int k = 0; k < kMaxSmallBatch; ++k) b.first[k] = INT_MAX;
    for (int k = 0; k < n; ++k) {
        const GemmArgs& g = gs[k];
        SmallArgs& a = b.g[k];
        const int64_t f = g.bA > 4 ? 1 : 256, lo = (int64_t)g.acc_lo * f, hi = (int64_t)g.acc_hi * f;
        a.qA = g.qA; a.qB = g.qB; a.scaleA = g.scaleA; a.scaleB = g.scaleB;
        a.out = g.out; a.out_bf16 = g.out_bf16; a.acc_out = g.acc_out; a.mask_src = g.mask_src;
        // (all below 2^31: small_enough)
        a.pitchA = (int)g.pitchA; a.pitchB = (int)g.pitchB;
        a.RA = (int)g.RA; a.RB = (int)g.RB; a.D = (int)g.D;
        a.acc_lo_scaled = lo < INT_MIN ? INT_MIN : (int)lo;
        a.acc_hi_scaled = hi > INT_MAX ? INT_MAX : (int)hi;
        a.inv_n = g.inv_n;
        a.mode = mode_of(g);
        a.unit = (int)unit_of(g);
        a.units = (int)((g.D + a.unit - 1) / a.unit);
        a.steps_per_tile = (int)(g.s / kStep);
        a.ragged = g.pitchA % 4 != 0 || g.pitchB % 4 != 0;
        const int64_t blocks = ((g.RA + 31) / 32) * ((g.RB + 31) / 32), steps = (g.D + kStep - 1) / kStep;
        const bool aligned = g.pitchA % 64 == 0 && g.pitchB % 64 == 0;
        if (!a.ragged && (aligned || a.mode != MODE_SAT8)) {
            work += blocks * steps;
            staged_blocks += blocks;
        }
        all_aligned &= aligned;
        packed_halves |= a.mode == MODE_HALF;
        paired &= a.mode == MODE_SAT8;
        a.n_ct = make_divisor((uint32_t)((g.RB + 31) / 32));
        b.first[k] = (int)total;
        total += (int64_t)a.n_ct.d * ((g.RA + 31) / 32);
    }
    ProfileScope ps(n > 1 ? K_GEMM_SMALL : gs[0].profile_tag ? K_GEMM_I4_FWD + (gs[0].profile_tag - 1) : K_GEMM_I4, stream);
    // Steps of blocks from which the launch waits for its loads' lanes rather than for one chain, lanes / staged in us of 360
    // products.  In pairs (MODE_SAT8) the steps of lines of whole 64 bytes count, where a chunk is one piece of a line: 2304 x 256
    // x 8192 (147456) 27.4 / 22.6, 798 x 657 x 4864 (79800) 16.6 / 14.0, 434 x 1236 x 3840 (65520) 13.7 / 12.3, 5992 x 152 x 1152 (33840)
    // 8.5 / 8.7, and never below one block per CU (575 x 445 x 9344, 252 blocks, 10.8 / 12.5); of other lines 1800 x 1920 x
    // 1472 (157320) takes 21.6 / 23.0, 736 x 1152 x 6464 (167256) 23.6 / 24.9, 592 x 1096 x 10816 (224770) 33.5 / 31.6.  The other modes,
    // whose steps take longer: tiles of 64 579 x 830 x 1792 (27664) 7.4 / 6.8, 7333 x 99 x 2304 (66240) 15.4 / 12.5; bytes 3251 x
    // 83 x 3328 (31824) 14.4 / 10.8, 1262 x 1555 x 1024 (62720) 18.4 / 13.6; where a chunk lies over two pieces later: bytes
    // 1924 x 1345 x 544 (44591) 12.5 / 13.3, 7027 x 95 x 2512 (52140) 20.7 / 17.4.  Not for packed codes in tiles of 16, whose two
    // sums a step leave no registers for it (1280 x 2304 x 192, a step, 35 / 40).
    const int64_t least = paired ? 64000 : all_aligned ? 24000 : 50000;
    const bool staged = !packed_halves && work >= least && (!paired || staged_blocks >= 256);
    if (staged) hipLaunchKernelGGL(gemm_small_kernel<true>, dim3((unsigned)total), dim3(64 * kWaves), 0, stream, b);
    else hipLaunchKernelGGL(gemm_small_kernel<false>, dim3((unsigned)total), dim3(64 * kWaves), 0, stream, b);
    return hipGetLastError();
}

} // namespace hdqt
