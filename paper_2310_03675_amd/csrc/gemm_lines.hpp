// What the kernels that bring the lines of both operands straight to LDS have in common (gemm_bytes.hip, gemm_packed.hip).
#pragma once
#include "common.hpp"

#include <limits.h>

namespace hdqt {
namespace lines {

constexpr uint32_t kOutside = 0x80000000u;
constexpr int kThreads = 256;               // four waves

// where the totals of a product go
struct OutArgs {
    int64_t RA, RB;
    float* out;
    const float* mask_src;
    int32_t *acc_out, *partial;
    int partial16;
};
inline OutArgs out_args(const GemmArgs& g)
{
    return {g.RA, g.RB, g.out, g.mask_src, g.acc_out, g.splits > 1 ? g.partial : nullptr, g.partial16};
}

struct LinesArgs {
    const uint8_t *qA, *qB;
    int64_t pitch, RA, RB, D;
    uint32_t n_rt, n_ct, tiles, per_xcd;
    Divisor group, out_tiles;
    uint32_t stages_per_tile, part_stages;
    int lo, hi, fin_shift;                  // clamp of a tile's sum, factor left in a total
    const float *scaleA, *scaleB;
    float inv_n;
    OutArgs to;
};

// tile: rows and columns of a workgroup's part of the output; stage: codes of a line in LDS
inline LinesArgs lines_args(const GemmArgs& g, int64_t tile_rows, int64_t tile_cols, int64_t stage)
{
    LinesArgs k{};
    k.qA = g.qA; k.qB = g.qB; k.pitch = g.pitchA; k.RA = g.RA; k.RB = g.RB; k.D = g.D;
    k.n_rt = (uint32_t)((g.RA + tile_rows - 1) / tile_rows); k.n_ct = (uint32_t)((g.RB + tile_cols - 1) / tile_cols);
    k.tiles = k.n_rt * k.n_ct * (uint32_t)g.splits;
    k.per_xcd = (k.tiles + 7) / 8;
    k.group = make_divisor(8 * k.n_ct);
    k.out_tiles = make_divisor(k.n_rt * k.n_ct);
    k.stages_per_tile = (uint32_t)((g.s + stage - 1) / stage);
    k.part_stages = (uint32_t)((g.tiles_per_split * g.s + stage - 1) / stage);
    k.lo = g.acc_lo; k.hi = g.acc_hi;
    k.scaleA = g.scaleA; k.scaleB = g.scaleB; k.inv_n = g.inv_n;
    k.to = out_args(g);
    return k;
}
// Grids of less than 2^32 threads (with what they are rounded up by), and parts of whole stages: tiles_per_split tiles then end
// where the next part begins, so that no part begins at or behind a line's end (all but the last have fewer than n_tiles tiles
// together) and none has more codes than those by which its totals were found to fit 16 bits.
inline bool lines_fit(const GemmArgs& g, int64_t tile_rows, int64_t tile_cols, int64_t stage)
{
    if (g.splits > 1 && g.tiles_per_split * g.s % stage != 0) return false;
    const int64_t tiles = ((g.RA + tile_rows - 1) / tile_rows) * ((g.RB + tile_cols - 1) / tile_cols) * g.splits;
    return (tiles + 7) * kThreads < ((int64_t)1 << 32);
}

// Workgroups go to the eight XCDs in turn: each gets a run of tiles of its own (part by part of a split contraction), in
// groups of eight rows of tiles column by column, whose panels its L2 holds.
struct Place {
    uint32_t share, rt, ct;          // part of the contraction, row and column of tiles
    uint32_t s_begin, n_stages;      // the part's stages
    bool there;
};
__device__ __forceinline__ Place place_of(const LinesArgs& g, uint32_t stage)
{
    Place p;
    const uint32_t idx = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
    p.there = idx < g.tiles;
    p.share = divide(idx, g.out_tiles);
    const uint32_t it = idx - p.share * g.out_tiles.d;
    const uint32_t grp = divide(it, g.group), in = it - grp * g.group.d;
    const uint32_t tall = g.n_rt - 8 * grp < 8 ? g.n_rt - 8 * grp : 8;
    p.ct = in / tall;
    p.rt = 8 * grp + in - p.ct * tall;
    const uint32_t all = (uint32_t)((g.D + stage - 1) / stage);
    p.s_begin = p.share * g.part_stages;
    if (p.s_begin > all) p.s_begin = all;
    p.n_stages = all - p.s_begin < g.part_stages ? all - p.s_begin : g.part_stages;
    return p;
}

// bytes of an operand from a panel's first line and a part's first byte on, for the range check of its descriptor
__device__ __forceinline__ int bytes_left(int64_t rows, int64_t first, int64_t pitch, int64_t begin)
{
    const int64_t n = (rows - first) * pitch - begin;
    return n <= 0 ? 0 : (int)(n < (int64_t)kOutside ? n : (int64_t)kOutside - 1);
}

// A wave's totals, RBLK x CBLK blocks of 32 x 32 at (row0, col0), to where they belong.  Stores through a descriptor that ends
// with the output: rows beyond it are dropped by the range check, columns by an offset outside (a branch around every store
// costs 2.5 us of a small product).
template <bool STREAM, bool MASK, int RBLK, int CBLK>
__device__ __forceinline__ void write_totals(const OutArgs& g, uint32_t share, int64_t row0, int64_t col0, int lane, float scale,
                                             const int (&tot)[RBLK][CBLK][16])
{
    const int64_t at0 = row0 * g.RB + col0, room = g.RA * g.RB - at0;
    uint32_t off[CBLK];              // elements
#pragma unroll
    for (int j = 0; j < CBLK; ++j) {
        const int64_t col = 32 * j + (lane & 31);
        off[j] = col0 + col < g.RB ? 4 * (lane >> 5) * (uint32_t)g.RB + (uint32_t)col : kOutside / 4;
    }
    auto range = [room](int64_t size) {
        return room <= 0 ? 0 : (int)(size * room < (int64_t)kOutside ? size * room : (int64_t)kOutside - 1);
    };
    auto each = [&](auto put) {
#pragma unroll
        for (int i = 0; i < RBLK; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < CBLK; ++j)
                    put(off[j] + (32 * i + 8 * (r >> 2) + (r & 3)) * (uint32_t)g.RB, tot[i][j][r], (i * 16 + r) * CBLK + j);
    };
    if (g.partial) {
        const int64_t slice = (int64_t)share * g.RA * g.RB + at0;
        if (g.partial16) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                reinterpret_cast<int16_t*>(g.partial) + slice, 0, range(2), 0x00020000);
            // (an offset outside in elements is one in units of 2 bytes only with the bit above)
            each([&](uint32_t o, int acc, int) {
                __builtin_amdgcn_raw_buffer_store_b16((short)acc, rs, o >= kOutside / 4 ? kOutside : 2 * o, 0, 0);
            });
        } else {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(g.partial + slice, 0, range(4), 0x00020000);
            each([&](uint32_t o, int acc, int) { __builtin_amdgcn_raw_buffer_store_b32((uint32_t)acc, rs, 4 * o, 0, 0); });
        }
        return;
    }
    if (g.out) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(g.out + at0, 0, range(4), 0x00020000);
        if constexpr (MASK) {
            const __amdgpu_buffer_rsrc_t ms = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.mask_src) + at0, 0, range(4), 0x00020000);
            float m[RBLK * CBLK * 16];
            each([&](uint32_t o, int, int at) { m[at] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ms, 4 * o, 0, STREAM ? 2 : 0)); });
            each([&](uint32_t o, int acc, int at) {
                __builtin_amdgcn_raw_buffer_store_b32(m[at] > 0.0f ? __float_as_uint((float)acc * scale) : 0u, rs, 4 * o, 0, STREAM ? 2 : 0);
            });
        } else {
            each([&](uint32_t o, int acc, int) {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)acc * scale), rs, 4 * o, 0, STREAM ? 2 : 0);
            });
        }
    }
    if (g.acc_out) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(g.acc_out + at0, 0, range(4), 0x00020000);
        each([&](uint32_t o, int acc, int) { __builtin_amdgcn_raw_buffer_store_b32((uint32_t)acc, rs, 4 * o, 0, 0); });
    }
}

} // namespace lines
} // namespace hdqt
