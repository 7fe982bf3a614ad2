// Hadamard-domain quantization of one tensor along BOTH axes from one read
// (gfx950).
//
// A training step needs every activation and gradient tensor quantized twice:
// along its rows for one matmul and along its columns for another (X along K
// for the forward product and along M for the weight gradient; G along N for
// the input gradient and along M for the weight gradient).  The two results
// are the paper's quantizer Q applied in two Hadamard domains; they share
// nothing but the source, and the source is what costs: the kernels are
// HBM-bound.  Here pass 1 computes both maxima and pass 2 both code sets from a
// single read of the tensor each.  The results are bit-identical to two
// single-axis quantizations.
//
// A wave holds a tile of 64 rows x 64 columns in registers, 64 values per lane:
// lane (rg, cg) = (lane / 8, lane % 8) has rows 8*rg + i (i < 8) of columns
// 32*h + 4*cg + j (h < 2, j < 4).  Both transforms run on that one layout:
//   along the columns of a row (axis 1): strides 1, 2 pair registers (j),
//     strides 4, 8, 16 pair lanes (lane xor 1, 2, 4), stride 32 pairs registers (h);
//   along the rows of a column (axis 0): strides 1, 2, 4 pair registers (i),
//     strides 8, 16, 32 pair lanes (lane xor 8, 16, 32).
// The stages that pair lanes through DPP are single multiply-adds that leave the
// upper lane's result negated (see stage_fma8); the sign a lane has accumulated,
// (-1)^popcount(lane & 7) after axis 1 and (-1)^(lane bit 3) after axis 0, is
// folded into the reciprocal step the lane quantizes with.
// The axis-1 transform is done row by row on copies (eight values at a time),
// the axis-0 transform then in place.  No LDS is involved.  (Pass 2 of a convolution source is another matter,
// see below.)
// Requires rows and cols multiples of 64 and block orders up to 64.  Codes of up to
// 4 bits are packed two per byte; the WIDE instances write codes of 5 to 8 bits, one
// per byte (both axes of a tensor, and all tensors of a launch, on the same side).

#include "common.hpp"
#include "lane_ops.hpp"
#include "quantize_any.hpp"

namespace hdqt {

namespace {

using namespace lanes;

constexpr int kThreads = 256;
constexpr int kTile = 64;

constexpr int kPieces = 7;               // 16-byte pieces of a patch per lane, in flight (four workgroups' patches fill the LDS)
constexpr int kPatchFloats = 256 * kPieces;      // of LDS that hold it
__host__ __device__ inline int tile_patch_floats(const DualArgs& q) { return (q.pCN * q.pCP + 3) & ~3; }      // (kConvTiles)

// LDS operations of one wave are carried out in order; this keeps the compiler from moving reads above the
// writes of other lanes.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct Tile {
    float v[2][4][8];        // [h][j][i]
};

struct DualCtx {
    const DualArgs* q;
    int cg, rg;
    int log2n_row, log2n_col;      // block orders; compile-time 6 in the kernel instances for n = 64
    float c1, c2, c4, c8;          // -1 where the lane bit is set, else +1
    float inv_row, inv_col;        // reciprocal steps, times the lane's accumulated sign
    float qmin_row, qmax_row, qmin_col, qmax_col;
};

__device__ __forceinline__ void tile_load(Tile& t, const DualArgs& q, const DualCtx& x, int64_t row0,
                                          int64_t col0)
{
    // a uniform address per (i, h) plus one 32-bit offset per lane (cols < 2^26: quantize_dual_eligible):
    // one 64-bit vector addition per row of the tile is all that is left of the address arithmetic
    // (buffer loads with scalar offsets take that out too, 21 instructions of 1711, and change no time)
    const float* base = q.T + row0 * q.cols + col0;
    const uint32_t lo = (uint32_t)(x.rg * 8) * (uint32_t)q.cols + (uint32_t)(x.cg * 4);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 a = *reinterpret_cast<const float4*>(&(base + i * q.cols + 32 * h)[lo]);
            t.v[h][0][i] = a.x; t.v[h][1][i] = a.y; t.v[h][2][i] = a.z; t.v[h][3][i] = a.w;
        }
}

// The same tile when the source is an activation and the tensor its im2col matrix.
// The 64 rows of a tile are 64 consecutive pixels of one image (whole image rows when
// W <= 64, a 64-pixel run of one row otherwise), its 64 columns a run of (channel, tap)
// pairs: everything the tile reads lies in a patch of pCN channels x pPH rows x pPW
// pixels, zero border included.  The wave copies the patch into its own piece of LDS
// with coalesced reads, then gathers its 64 x 64 values from there: an element's patch
// address is (row part of its pixel) + (column part of its channel and tap).
// The activation is read from HBM about once per pass instead of kh*kw times.
//
// Two ways to it (dual_conv_plan).  Where the patch is at most kPieces 16-byte pieces a lane, kConvLines: its rows are padded
// to whole pieces on either side and pieces lie one after the other, so piece u of the
// patch is the same place of every tile relative to the tile's first: a lane works out its pieces once,
// and a wave of pass 2 goes through pSteps tiles.  (Working them out for each tile was a quarter of the kernel's vector
// instructions.)  Pass 1, which has little else to do, is better off with a tile a wave, more of them in flight:
// 262144 x 576 52 -> 42 us, in steps 85.
struct PatchPieces {
    int off[kPieces];                    // bytes from the image's element (c_lo, y_first - ph, x_first - lead)
    int y[kPieces];                      // four times the patch row (far outside for pieces that hold nothing), plus 1 for
                                         // pieces left of the tile's own columns and 2 for those right of them
};

struct PatchPlace {                      // of one tile, the same in every lane
    const float* img;
    int x, y, c_lo;                      // x_first - lead, y_first - ph
    int at;                              // in pieces: bytes of (c_lo, y, x) from `img` (images of less than 2^31 bytes)
    int beside;                          // 1: the tile's columns start an image row, 2: they end one, 3: both
};

__device__ __forceinline__ void patch_pieces(PatchPieces& p, const DualArgs& q, int lane)
{
    const int wt = q.cW < kTile ? q.cW : kTile;
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const uint32_t u = 64 * k + lane;
        const uint32_t c = (u * q.pInvCh) >> 20, rest = u - c * q.pPerCh;          // (below 2^20 / pPerCh: dual_conv_plan)
        const uint32_t y = (rest * q.pInvRow) >> 20, x = (rest - y * q.pPerRow) * 4;
        p.off[k] = 4 * (((int)c * q.cH + (int)y) * q.cW + (int)x);
        const int beside = (int)x < q.pLead ? 1 : (int)x >= q.pLead + wt ? 2 : 0;
        p.y[k] = u < q.pPieces && (int)y < q.pPH ? 4 * (int)y + beside : INT_MIN / 2;
    }
}

__device__ __forceinline__ PatchPlace patch_place(const DualArgs& q, uint32_t row0, uint32_t col0)
{
    PatchPlace a;
    const int W = q.cW, H = q.cH;
    const uint32_t b = divide(row0, q.dHW), rem = row0 - b * q.dHW.d;
    const int y_first = (int)divide(rem, q.dW), x_first = (int)rem - y_first * W;
    a.c_lo = (int)divide(col0, q.dTaps);
    a.y = y_first - (q.ckh - 1) / 2;
    a.img = q.T + (int64_t)b * q.cC * H * W;
    a.x = x_first - q.pLead;
    a.at = (int)(4u * (uint32_t)((a.c_lo * H + a.y) * W + a.x));
    a.beside = (x_first == 0 ? 1 : 0) | (x_first + kTile >= W ? 2 : 0);
    return a;
}

// (what lies outside the image is asked for beyond its end, where a buffer load returns zeros)
__device__ __forceinline__ void patch_load(float4 (&v)[kPieces], const PatchPieces& p, const PatchPlace& a, const DualArgs& q)
{
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.img), 0, 4 * q.cC * q.cH * q.cW, 0x00020000);
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const bool in = (uint32_t)(p.y[k] + 4 * a.y) < 4u * (uint32_t)q.cH && !(p.y[k] & a.beside);
        v[k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, in ? p.off[k] + a.at : -16, 0, 0));
    }
}

// Into LDS; returns the values' sign bits, put together.
__device__ __forceinline__ uint32_t patch_store(const float4 (&v)[kPieces], float* patch, int lane)
{
    uint32_t signs = 0;
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        signs |= (as_u(v[k].x) | as_u(v[k].y)) | (as_u(v[k].z) | as_u(v[k].w));
        *reinterpret_cast<float4*>(patch + 4 * (64 * k + lane)) = v[k];
    }
    return signs;
}

// Column parts of the tile's 64 columns, one per lane, in bytes.
__device__ __forceinline__ void column_table(int* coltab, const DualArgs& q, int c_lo, uint32_t col0, int lane)
{
    const uint32_t k = col0 + (uint32_t)lane;
    const uint32_t c = divide(k, q.dTaps), tap = k - c * q.dTaps.d;
    const uint32_t ty = divide(tap, q.dkw), tx = tap - ty * q.dkw.d;
    coltab[lane] = 4 * (((int)c - c_lo) * q.pCP + (int)ty * q.pPW + (int)tx + q.pLead - (q.ckw - 1) / 2);
}

// (of a patch in pieces)
__device__ __forceinline__ int* column_parts(float* patch) { return reinterpret_cast<int*>(patch + kPatchFloats); }

__device__ __forceinline__ const float* at_byte(const float* p, int bytes)
{
    return reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + bytes);
}

// The tile in registers from the patch: pixel 8*rg + i of the tile is (image row off / Wt, position off % Wt),
// Wt = min(W, 64), a power of two.  With Wt >= 8 the lane's eight pixels are neighbours
// in one image row: eight consecutive patch words per column.
__device__ __forceinline__ void tile_gather(Tile& t, const DualArgs& q, const float* patch, const int* coltab, int lane)
{
    int shift = q.cW >= kTile ? 6 : 31 - __builtin_clz((unsigned)q.cW), PW = q.pPW;
    const int off = lane & ~7, cg = lane & 7;
    if (shift >= 3) {
        const float* base = patch + (off >> shift) * PW + (off & ((1 << shift) - 1));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int4 cp = *reinterpret_cast<const int4*>(coltab + 32 * h + 4 * cg);
            const float* p[4] = {at_byte(base, cp.x), at_byte(base, cp.y), at_byte(base, cp.z), at_byte(base, cp.w)};
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) t.v[h][j][i] = p[j][i];
        }
    } else {
        asm volatile("" : "+s"(PW), "+s"(shift));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int4 cp = *reinterpret_cast<const int4*>(coltab + 32 * h + 4 * cg);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float* p = patch + ((off + i) >> shift) * PW + ((off + i) & ((1 << shift) - 1));
                t.v[h][0][i] = *at_byte(p, cp.x);
                t.v[h][1][i] = *at_byte(p, cp.y);
                t.v[h][2][i] = *at_byte(p, cp.z);
                t.v[h][3][i] = *at_byte(p, cp.w);
            }
        }
    }
}

// Any other patch, kConvTiles: row by row, unpadded, for tiles in registers in both passes.  In pieces these take more LDS than
// four workgroups have, and their rows meet on the same banks.  Both passes over 75 M elements of 64 channels, tiles in registers / pieces in
// two or three parts (in units of 64 pieces with the best padding): 3 x 1 in images 32 wide 132 / 233 us (155), 1 x 3 in 8 95 / 149 (145),
// 5 x 3 in 64 92 / 118 (97), 9 x 3 in 64 90 / 117 (143).
constexpr int kPatchUnroll = 6;

// Returns whether a value of the patch has its sign bit set (the same in every lane).
__device__ __forceinline__ bool tile_load_conv(Tile& t, const DualArgs& q, int64_t row0, int64_t col0, float* patch, int lane)
{
    uint32_t signs = 0;
    const int W = q.cW, H = q.cH, C = q.cC, kw = q.ckw, pw = (kw - 1) / 2;
    const int PH = q.pPH, PW = q.pPW;
    int* coltab = reinterpret_cast<int*>(patch + tile_patch_floats(q));
    const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)row0);
    const uint32_t k0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)col0);
    const PatchPlace at = patch_place(q, m0, k0);
    const int x_first = at.x + pw;

    // ---- patch: row r = (channel c_lo + r / PH, image row y_first - ph + r % PH).  The tile's own
    // columns are whole image rows, or 64 pixels from a multiple of 64 on: four pixels per lane and
    // load, kPatchUnroll loads in flight (every address is clamped into the activation, so no load
    // is conditional).  (One pixel per lane and load cost 64 times the twelve instructions of its
    // address and border test, a third of the kernel: 262144 x 576 from 256 x 64 x 32 x 32, pass 1
    // 143 -> 91 us, pass 2 180 -> 135 us.)
    const int wt = W < kTile ? W : kTile;
    const int rows_total = q.pCN * PH;
    // (r / PH for r below 2^20 / PH: dual_conv_plan)
    const uint32_t inv_ph = ((1u << 20) + (uint32_t)PH - 1) / (uint32_t)PH;
    auto source = [&](int r, int& off) {          // whether row r lies in the activation, and where
        const int c_rel = (int)(((uint32_t)r * inv_ph) >> 20);
        const int gy = at.y + r - c_rel * PH, c = at.c_lo + c_rel;
        const int gyc = gy < 0 ? 0 : (gy >= H ? H - 1 : gy), cc = c >= C ? C - 1 : c;
        off = (cc * H + gyc) * W;
        return gy == gyc && c < C;
    };
    if (wt >= 4) {
        const int log2u = 29 - __builtin_clz((unsigned)wt);      // (wt is a power of two) units of four pixels per row
        const int units = rows_total << log2u;
        for (int u0 = 0; u0 < units; u0 += 64 * kPatchUnroll) {
            float4 v[kPatchUnroll];
            int dst[kPatchUnroll];
#pragma unroll
            for (int k = 0; k < kPatchUnroll; ++k) {
                const int u = u0 + 64 * k + lane, r = u >> log2u, xq = (u - (r << log2u)) * 4;
                int off;
                const bool in = source(r, off);
                v[k] = *reinterpret_cast<const float4*>(at.img + off + x_first + xq);
                if (!in) v[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                dst[k] = u < units ? r * PW + pw + xq : -1;
            }
#pragma unroll
            for (int k = 0; k < kPatchUnroll; ++k) {
                if (dst[k] < 0) continue;
                signs |= (as_u(v[k].x) | as_u(v[k].y)) | (as_u(v[k].z) | as_u(v[k].w));
                float* d = patch + dst[k];
                d[0] = v[k].x; d[1] = v[k].y; d[2] = v[k].z; d[3] = v[k].w;
            }
        }
    }
    // ---- the window's columns beside them (all columns of images one or two pixels wide): zeros
    // next to a whole image row, else pixels one by one
    const int n_side = wt >= 4 ? kw - 1 : PW;
    if (n_side) {
        const uint32_t inv_ns = ((1u << 20) + (uint32_t)n_side - 1) / (uint32_t)n_side;
        for (int e = lane; e < rows_total * n_side; e += 64) {
            const int r = (int)(((uint32_t)e * inv_ns) >> 20), k = e - r * n_side;
            const int px = wt >= 4 && k >= pw ? wt + k : k, gx = at.x + px;
            float v = 0.0f;
            if (gx >= 0 && gx < W) {
                int off;
                const bool in = source(r, off);
                v = at.img[off + gx];
                if (!in) v = 0.0f;
            }
            signs |= as_u(v);
            patch[r * PW + px] = v;
        }
    }
    column_table(coltab, q, at.c_lo, k0, lane);
    wave_order();
    tile_gather(t, q, patch, coltab, lane);
    return __builtin_amdgcn_ballot_w64((int)signs < 0) != 0;
}

// Random bits of stochastic rounding for the lane's elements of one tile row: four
// consecutive elements at h = 0 (index e, e % 4 == 0) and four at h = 1 (index
// e + 32).  Each group lies in one Philox block (block e/8, words (e%8)/2 and
// (e%8)/2 + 1), and lanes cg and cg ^ 1 need the same two blocks, the even lane the
// lower words, the odd lane the upper ones.  So the even lane computes the block of
// h = 0, the odd lane that of h = 1, and they trade the halves the other needs:
// one Philox call per lane and row instead of two.
__device__ __forceinline__ void random_words(int64_t e, bool odd, uint32_t tensor_id, uint32_t k0,
                                             uint32_t k1, uint32_t w_h0[2], uint32_t w_h1[2])
{
    const uint64_t blk = ((uint64_t)e >> 3) + (odd ? 4u : 0u);
    uint32_t r[4];
    philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), tensor_id, 0u, k0, k1, r);
    const uint32_t send0 = odd ? r[0] : r[2], send1 = odd ? r[1] : r[3];
    const uint32_t recv0 = __float_as_uint(lane_xor<1>(__uint_as_float(send0)));
    const uint32_t recv1 = __float_as_uint(lane_xor<1>(__uint_as_float(send1)));
    w_h0[0] = odd ? recv0 : r[0];
    w_h0[1] = odd ? recv1 : r[1];
    w_h1[0] = odd ? r[2] : recv0;
    w_h1[1] = odd ? r[3] : recv1;
}

// Axis 1 for the lane's row 8*rg + i of the tile: transform, then absmax (pass
// 1) or codes (pass 2).
template <bool QUANT, bool STOCH, bool WIDE>
__device__ __forceinline__ void row_line(const Tile& t, int i, const DualCtx& x, int64_t row0,
                                         int64_t col0, float& amax)
{
    const DualArgs& q = *x.q;
    const int log2n = x.log2n_row;
    float w[8];              // index 4*h + j
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[4 * h + j] = t.v[h][j][i];
    if (log2n >= 1) {
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            const float a = w[k], c = w[k + 1];
            w[k] = a + c;
            w[k + 1] = a - c;
        }
    }
    if (log2n >= 2) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (!(k & 2)) {
                const float a = w[k], c = w[k + 2];
                w[k] = a + c;
                w[k + 2] = a - c;
            }
    }
    if (log2n >= 3) {
        stage_fma8<1>(w, x.c1);
    }
    if (log2n >= 4) {
        stage_fma8<2>(w, x.c2);
    }
    if (log2n >= 5) {
        stage_fma8<4>(w, x.c4);
    }
    if (!QUANT) {
        // max(|a + c|, |a - c|) = |a| + |c|, also after rounding: the last stage of
        // pass 1 needs no differences
        if (log2n >= 6) {
#pragma unroll
            for (int k = 0; k < 4; ++k) amax = fmaxf(amax, fabsf(w[k]) + fabsf(w[k + 4]));
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) amax = fmaxf(amax, fabsf(w[k]));
        }
        return;
    }
    if (log2n >= 6) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float a = w[k], c = w[k + 4];
            w[k] = a + c;
            w[k + 4] = a - c;
        }
    }
    const int64_t row = row0 + x.rg * 8 + i;
    const float magic = kMagic + (WIDE ? 128.0f : 8.0f);
    uint32_t both = 0;       // the lane's eight codes: low half h = 0, high half h = 1
    uint32_t rnd[2][2] = {{0u, 0u}, {0u, 0u}};
    if (STOCH)
        random_words(row * q.cols + col0 + x.cg * 4, (x.cg & 1) != 0, q.tid_row, q.seed_row_lo,
                     q.seed_row_hi, rnd[0], rnd[1]);
    if constexpr (WIDE) {
        // one byte per code: the lane's four codes of each half are a dword.  Lanes cg and
        // cg ^ 1 trade one of them: the even lane ends up with columns 4cg .. 4cg+7, the odd
        // one with columns 32+4(cg-1) .. 32+4cg+3, eight bytes per lane and store.
        uint32_t word[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t cw[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = (rnd[h][j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
                cw[j] = code_word<STOCH>(w[4 * h + j], x.inv_row, x.qmin_row, x.qmax_row, magic, u);
            }
            word[h] = pack_bytes(cw);
        }
        const bool odd = (x.cg & 1) != 0;
        const uint32_t other = __float_as_uint(lane_xor<1>(__uint_as_float(odd ? word[0] : word[1])));
        const uint2 pair = odd ? make_uint2(other, word[1]) : make_uint2(word[0], other);
        const int byte_off = odd ? 32 + 4 * (x.cg - 1) : 4 * x.cg;
        *reinterpret_cast<uint2*>(q.codes_row + row * q.cols + col0 + byte_off) = pair;
        return;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t* w01 = rnd[h];
        // 0x4B400000 << 4j has no bits in the low 16: the low half of the sum is the
        // four offset nibbles
        uint32_t acc = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t u = (w01[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
            acc += code_word<STOCH>(w[4 * h + j], x.inv_row, x.qmin_row, x.qmax_row, magic, u) << (4 * j);
        }
        both |= (acc & 0xFFFFu) << (16 * h);
    }
    both ^= 0x88888888u;
    // Lanes cg and cg ^ 1 trade halves: the even one ends up with columns
    // 4cg .. 4cg+7 (bytes 2cg .. 2cg+3 of the row's 32), the odd one with columns
    // 32+4(cg-1) .. 32+4cg+3 (bytes 16+2(cg-1) ..).
    const uint32_t other = __float_as_uint(lane_xor<1>(__uint_as_float(both)));
    const bool odd = (x.cg & 1) != 0;
    const uint32_t word = __builtin_amdgcn_perm(other, both, odd ? 0x03020706u : 0x05040100u);
    const int byte_off = odd ? 16 + 2 * (x.cg - 1) : 2 * x.cg;
    // (uniform address of the tile's row i, 32-bit offset of the lane's row group and bytes)
    const uint32_t lo = (uint32_t)(x.rg * 8) * (uint32_t)(q.cols >> 1) + (uint32_t)byte_off;
    *reinterpret_cast<uint32_t*>(&(q.codes_row + (row0 + i) * (q.cols >> 1) + (col0 >> 1))[lo]) = word;
}

// Axis 0 on the whole tile, in place.  The two lanes of a swap stage carry the
// same sign (it depends on lane bit 3 only), so those stages need no care.
// MAX_ONLY (pass 1, block order 64): the last stage is replaced by |lo| + |hi| of
// the swapped-in pairs, returned as a running maximum; the tile is then spent.
template <bool MAX_ONLY>
__device__ __forceinline__ float col_transform(Tile& t, int log2n, float c8)
{
    float m = 0.0f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float* v = t.v[h][j];
            butterfly8(v, log2n);
            if (log2n > 3) stage_fma8<8>(v, c8);
            if (log2n > 4) {
#pragma unroll
                for (int i = 0; i < 8; i += 2) stage_swap<false>(v[i], v[i + 1]);
            }
            if (MAX_ONLY) {
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    const v2u r = __builtin_amdgcn_permlane32_swap(as_u(v[i]), as_u(v[i + 1]), false, false);
                    m = fmaxf(m, fabsf(as_f(r[0])) + fabsf(as_f(r[1])));
                }
            } else if (log2n > 5) {
#pragma unroll
                for (int i = 0; i < 8; i += 2) stage_swap<true>(v[i], v[i + 1]);
            }
        }
    return m;
}

template <bool STOCH, bool WIDE>
__device__ __forceinline__ void col_codes(const Tile& t, const DualCtx& x, int64_t row0, int64_t col0)
{
    const DualArgs& q = *x.q;
    const float magic = kMagic + (WIDE ? 128.0f : 8.0f);
    const int64_t pitch = WIDE ? q.rows : q.rows >> 1;
    uint32_t cw[2][4][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        uint32_t rnd[2][2] = {{0u, 0u}, {0u, 0u}};
        if (STOCH)
            random_words((row0 + x.rg * 8 + i) * q.cols + col0 + x.cg * 4, (x.cg & 1) != 0, q.tid_col,
                         q.seed_col_lo, q.seed_col_hi, rnd[0], rnd[1]);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = (rnd[h][j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
                cw[h][j][i] = code_word<STOCH>(t.v[h][j][i], x.inv_col, x.qmin_col, x.qmax_col, magic, u);
            }
    }
    // column 32h + 4cg + j, rows 8rg .. 8rg+7: one dword (two with a byte per code); the
    // eight rg lanes of a column write 32 (64) consecutive bytes
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (WIDE) {
                uint8_t* dst = q.codes_col + (col0 + 32 * h + x.cg * 4 + j) * pitch + row0 + x.rg * 8;
                *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bytes(cw[h][j]), pack_bytes(cw[h][j] + 4));
            } else {
                const uint32_t lo = (uint32_t)(x.cg * 4) * (uint32_t)pitch + (uint32_t)(x.rg * 4);
                uint8_t* dst = &(q.codes_col + (col0 + 32 * h + j) * pitch + (row0 >> 1))[lo];
                *reinterpret_cast<uint32_t*>(dst) = pack_nibbles(cw[h][j]);
            }
        }
}

// Both maxima of the workgroup into their records (see QMeta).
__device__ __forceinline__ void record_max2(float m_row, float m_col, QMeta* meta_row,
                                            QMeta* meta_col, float (*smem)[2], int local, int dense)
{
    m_row = wave_max(m_row);
    m_col = wave_max(m_col);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { smem[wave][0] = m_row; smem[wave][1] = m_col; }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int which = threadIdx.x;
        float r = smem[0][which];
        for (int w = 1; w < kThreads / kWave; ++w) r = fmaxf(r, smem[w][which]);
        record_word(r, which ? meta_col : meta_row, local, dense);
    }
}

// ---- the two phases of a tile, shared by the two-launch and the one-launch kernels

template <bool N64>
__device__ __forceinline__ void dual_setup(DualCtx& x, const DualArgs& q, int lane)
{
    x.q = &q;
    // with the block orders known at compile time the stage conditions, the branches around
    // them and the register copies at their joins disappear (about a tenth of the kernel)
    x.log2n_row = N64 ? 6 : q.log2n_row;
    x.log2n_col = N64 ? 6 : q.log2n_col;
    x.cg = lane & 7;
    x.rg = lane >> 3;
    x.c1 = (lane & 1) ? -1.0f : 1.0f;
    x.c2 = (lane & 2) ? -1.0f : 1.0f;
    x.c4 = (lane & 4) ? -1.0f : 1.0f;
    x.c8 = (lane & 8) ? -1.0f : 1.0f;
    x.inv_row = x.inv_col = 0.0f;
    x.qmin_row = (float)(-(1 << (q.b_row - 1)));
    x.qmax_row = (float)((1 << (q.b_row - 1)) - 1);
    x.qmin_col = (float)(-(1 << (q.b_col - 1)));
    x.qmax_col = (float)((1 << (q.b_col - 1)) - 1);
}

// reciprocal steps (with the lane's accumulated signs) from the two scalings;
// one thread of the grid publishes the scales
__device__ __forceinline__ void dual_set_scaling(DualCtx& x, const DualArgs& q, const Scaling& s_row,
                                                 const Scaling& s_col, bool publisher)
{
    // signs accumulated by the stage_fma8 stages that actually run
    float sg_row = 1.0f;
    if (x.log2n_row >= 3) sg_row *= x.c1;
    if (x.log2n_row >= 4) sg_row *= x.c2;
    if (x.log2n_row >= 5) sg_row *= x.c4;
    x.inv_row = s_row.inv * sg_row;
    x.inv_col = x.log2n_col > 3 ? s_col.inv * x.c8 : s_col.inv;
    if (publisher && threadIdx.x == 0) {
        q.meta_row->scale = s_row.scale;
        q.meta_col->scale = s_col.scale;
        if (q.scale_row_out) *q.scale_row_out = s_row.scale;
        if (q.scale_col_out) *q.scale_col_out = s_col.scale;
    }
}

template <int CTRL>
__device__ __forceinline__ float add_dpp(float x)
{
    return x + dpp_move<CTRL>(x);
}

// Both maxima of a tile without negative values, block orders 8 to 64.  The largest output of a
// block is then its sum, in the order of the butterfly's own output 0: by induction over the stages no
// |a +- c| exceeds the sum of the values below it, because rounding is monotone (an infinity gives
// infinity and a NaN a block that counts for nothing, both ways).  So the sums replace the butterflies,
// one addition per pair instead of two outputs: 190 vector instructions a tile instead of 900.  What a
// convolution reads is what a rectifier wrote, and these passes are bound by vector issue:
// 262144 x 576 from 256 x 64 x 32 x 32 91 -> 49 us, 32768 x 320 from 256 x 64 x 1 x 128 15 -> 8.
__device__ __forceinline__ void sums_absmax(const Tile& t, const DualCtx& x, float& amax_row, float& amax_col)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float s[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s[h] = (t.v[h][0][i] + t.v[h][1][i]) + (t.v[h][2][i] + t.v[h][3][i]);
            s[h] = add_dpp<0xB1>(s[h]);                                   // lane ^ 1
            if (x.log2n_row > 3) s[h] = add_dpp<0x4E>(s[h]);              // lane ^ 2
            if (x.log2n_row > 4) s[h] = add_dpp<0x141>(s[h]);             // the other quad of eight lanes
        }
        if (x.log2n_row > 5) amax_row = fmaxf(amax_row, s[0] + s[1]);
        else amax_row = fmaxf(amax_row, fmaxf(s[0], s[1]));
    }
    float c[8];                                                           // of column 32h + 4cg + j: c[4h + j]
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float* v = t.v[k >> 2][k & 3];
        c[k] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        if (x.log2n_col > 3) c[k] = add_dpp<0x128>(c[k]);                 // lane ^ 8
    }
    // (a swap brings the two halves of a pair into one lane: c[k]'s in the lower lanes, c[k + 1]'s in the upper)
    int n = 8;
    if (x.log2n_col > 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const v2u r = __builtin_amdgcn_permlane16_swap(as_u(c[2 * k]), as_u(c[2 * k + 1]), false, false);
            c[k] = as_f(r[0]) + as_f(r[1]);
        }
        n = 4;
    }
    if (x.log2n_col > 5) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const v2u r = __builtin_amdgcn_permlane32_swap(as_u(c[2 * k]), as_u(c[2 * k + 1]), false, false);
            c[k] = as_f(r[0]) + as_f(r[1]);
        }
        n = 2;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (k < n) amax_col = fmaxf(amax_col, c[k]);
}

// both maxima of a tile; `t` is spent afterwards
__device__ __forceinline__ void dual_absmax(Tile& t, const DualCtx& x, int64_t row0, int64_t col0,
                                            float& amax_row, float& amax_col)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) row_line<false, false, false>(t, i, x, row0, col0, amax_row);
    if (x.log2n_col > 5) {
        amax_col = fmaxf(amax_col, col_transform<true>(t, x.log2n_col, x.c8));
    } else {
        col_transform<false>(t, x.log2n_col, x.c8);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) amax_col = fmaxf(amax_col, fabsf(t.v[h][j][i]));
    }
}

// both code sets of a tile; `t` is spent afterwards
template <bool ST_ROW, bool ST_COL, bool WIDE>
__device__ __forceinline__ void dual_codes(Tile& t, const DualCtx& x, int64_t row0, int64_t col0)
{
    float unused = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) row_line<true, ST_ROW, WIDE>(t, i, x, row0, col0, unused);
    col_transform<false>(t, x.log2n_col, x.c8);
    col_codes<ST_COL, WIDE>(t, x, row0, col0);
}

// ---- pass 2 of a convolution source: every lane has a whole line of its wave's tile, first a row (64 columns),
// then a column (64 rows), so that both transforms and the packing stay inside the lane.  The patch is in LDS
// anyway, and gathering it twice is cheaper than pairing lanes: an addition of two registers takes two
// cycles a wave here, one with a lane move four and a lane swap eight (measured at four waves per SIMD).
// Pass 2 of 262144 x 576 from 256 x 64 x 32 x 32 136 -> 99 us, of 32768 x 320 from 256 x 64 x 1 x 128 18.7 -> 16.4.
// What bounds it is still vector issue: 1550 instructions a tile keep the ALU busy in all of the kernel's cycles (counters), the LDS
// is busy in 46 % of them, a quarter of that with bank conflicts.  Not for
// an ordinary source: its tile would have to go through LDS too, 17 KB a wave, which leaves two waves per SIMD
// (the 65536 x 1152 x 128 step 259 -> 265 us).

// Lane's row (AXIS 1) or column (AXIS 0) of the tile.
template <int AXIS>
__device__ __forceinline__ void line_gather(float (&v)[kTile], const DualArgs& q, float* patch, int lane)
{
    const int* coltab = column_parts(patch);
    const int PW = q.pPW, shift = q.cW >= kTile ? 6 : 31 - __builtin_clz((unsigned)q.cW), mask = (1 << shift) - 1;
    if (AXIS == 1) {
        const float* base = patch + (lane >> shift) * PW + (lane & mask);
#pragma unroll
        for (int k = 0; k < kTile; k += 4) {
            const int4 cp = *reinterpret_cast<const int4*>(coltab + k);
            v[k] = *at_byte(base, cp.x); v[k + 1] = *at_byte(base, cp.y);
            v[k + 2] = *at_byte(base, cp.z); v[k + 3] = *at_byte(base, cp.w);
        }
    } else {
        const float* base = at_byte(patch, coltab[lane]);
        if (shift >= 3) {
#pragma unroll
            for (int k = 0; k < kTile; k += 8) {
                const float* p = base + ((k >> shift) * PW + (k & mask));
#pragma unroll
                for (int i = 0; i < 8; ++i) v[k + i] = p[i];
            }
        } else {
            int pitch = PW, sh = shift;
            asm volatile("" : "+s"(pitch), "+s"(sh));     // (keeps 64 addresses of narrow images out of the common path)
#pragma unroll
            for (int k = 0; k < kTile; ++k) v[k] = base[(k >> sh) * pitch + (k & ((1 << sh) - 1))];
        }
    }
}

__device__ __forceinline__ void butterfly64(float (&v)[kTile], int log2n)
{
#pragma unroll
    for (int s = 0; s < 6; ++s)
        if (log2n > s) {
#pragma unroll
            for (int k = 0; k < kTile; ++k)
                if (!(k & (1 << s))) {
                    const float a = v[k], c = v[k + (1 << s)];
                    v[k] = a + c;
                    v[k + (1 << s)] = a - c;
                }
        }
}

// Codes of a line, 32 (WIDE: 64) consecutive bytes.  `random(g, u)` gives the random 16 bits of its elements 8g .. 8g+7.
// They leave by way of LDS, neighbouring lanes with neighbouring pieces of a line.
template <bool STOCH, bool WIDE, typename Random>
__device__ __forceinline__ void line_codes(const float (&v)[kTile], float inv, float qmin, float qmax, uint8_t* dst, int64_t pitch,
                                           uint4* words, int lane, Random random)
{
    constexpr int kPieces = WIDE ? 4 : 2;        // 16-byte pieces of a line
    const float magic = kMagic + (WIDE ? 128.0f : 8.0f);
    uint32_t out[4];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        uint32_t u[8] = {}, cw[8];
        if (STOCH) random(g, u);
#pragma unroll
        for (int i = 0; i < 8; ++i) cw[i] = code_word<STOCH>(v[8 * g + i], inv, qmin, qmax, magic, u[i]);
        if constexpr (WIDE) {
            out[2 * (g & 1)] = pack_bytes(cw);
            out[2 * (g & 1) + 1] = pack_bytes(cw + 4);
            if (g & 1) words[lane * kPieces + (g >> 1)] = make_uint4(out[0], out[1], out[2], out[3]);
        } else {
            out[g & 3] = pack_nibbles_chain(cw);
            if ((g & 3) == 3) words[lane * kPieces + (g >> 2)] = make_uint4(out[0], out[1], out[2], out[3]);
        }
    }
    wave_order();
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int at = 64 * k + lane, line = at / kPieces;
        *reinterpret_cast<uint4*>(dst + line * pitch + 16 * (at % kPieces)) = words[at];
    }
    wave_order();
}

// Both code sets of a tile.  `piece`: the wave's LDS: patch, column table, codes on their way out.
template <bool ST_ROW, bool ST_COL, bool WIDE, bool N64>
__device__ __forceinline__ void line_tile(const DualArgs& q, const Scaling& s_row, const Scaling& s_col, int64_t row0,
                                          int64_t col0, float* piece, int lane)
{
    const int half = WIDE ? 0 : 1;
    uint4* const words = reinterpret_cast<uint4*>(piece + kPatchFloats + kTile);
    float v[kTile];
    line_gather<1>(v, q, piece, lane);
    butterfly64(v, N64 ? 6 : q.log2n_row);
    {
        const int64_t row = row0 + lane;
        const uint64_t blk = (uint64_t)(row * q.cols + col0) >> 3;
        line_codes<ST_ROW, WIDE>(v, s_row.inv, (float)(-(1 << (q.b_row - 1))), (float)((1 << (q.b_row - 1)) - 1),
                                 q.codes_row + ((row0 * q.cols + col0) >> half), q.cols >> half, words, lane, [&](int g, uint32_t (&u)[8]) {
                                     uint32_t r[4];
                                     philox4x32_10((uint32_t)(blk + g), (uint32_t)((blk + g) >> 32), q.tid_row, 0u,
                                                   q.seed_row_lo, q.seed_row_hi, r);
#pragma unroll
                                     for (int i = 0; i < 8; ++i) u[i] = (r[i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
                                 });
    }
    line_gather<0>(v, q, piece, lane);
    uint4* const blocks = reinterpret_cast<uint4*>(piece);      // (the patch has been read)
    butterfly64(v, N64 ? 6 : q.log2n_col);
    line_codes<ST_COL, WIDE>(v, s_col.inv, (float)(-(1 << (q.b_col - 1))), (float)((1 << (q.b_col - 1)) - 1),
                             q.codes_col + ((col0 * q.rows + row0) >> half), q.rows >> half, words, lane, [&](int g, uint32_t (&u)[8]) {
                                 // eight lanes need the same eight blocks, of rows 8g .. 8g+7 at their columns: each
                                 // makes one, and they are handed over through LDS
                                 const uint64_t blk = (uint64_t)((row0 + 8 * g + (lane & 7)) * q.cols + col0 + (lane & ~7)) >> 3;
                                 uint32_t r[4];
                                 philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), q.tid_col, 0u, q.seed_col_lo,
                                               q.seed_col_hi, r);
                                 blocks[lane] = make_uint4(r[0], r[1], r[2], r[3]);
                                 wave_order();
                                 const uint16_t* mine = reinterpret_cast<const uint16_t*>(blocks + (lane & ~7)) + (lane & 7);
#pragma unroll
                                 for (int i = 0; i < 8; ++i) u[i] = mine[8 * i];
                                 wave_order();
                             });
}

// One launch covers up to kMaxBatch tensors: the workgroups of tensor k are
// [first[k], first[k+1]) of a one-dimensional grid, numbered along its columns first.
// Small tensors (a layer's weights) ride along with a large one instead of paying
// for a launch of their own.
struct DualBatch {
    int first[kMaxDualBatch + 1];        // (behind the last tensor: the workgroups of all)
    Divisor gx[kMaxDualBatch];   // workgroups along the columns
    int WC[kMaxDualBatch];       // waves side by side in a workgroup (1, 2 or 4)
    int words[kMaxDualBatch];    // dense: pass 1's workgroups, whose maxima stand side by side
    int steps[kMaxDualBatch];    // convolution sources: tiles a wave takes one after the other
    int lds_per_wave;            // floats of LDS per wave (convolution sources), a multiple of 4
    int dense;                   // the maxima stand side by side (see QMeta)
    int spread;                  // pass 2: every spread-th workgroup of the grid is one of tensor 0 (0: off)
    DualArgs t[kMaxDualBatch];
};

// (see common.hpp: the arguments in one go)
template <int CONV>
__device__ __forceinline__ DualArgs whole_args(const DualArgs& x)
{
    const DualArgs q = x;
    asm volatile("" ::"s"(q.T), "s"(q.rows), "s"(q.cols), "s"(q.log2n_row), "s"(q.log2n_col), "s"(q.b_row), "s"(q.clip_row),
                 "s"(q.tid_row), "s"(q.b_col), "s"(q.clip_col), "s"(q.tid_col), "s"(q.seed_row_lo), "s"(q.seed_row_hi),
                 "s"(q.seed_col_lo), "s"(q.seed_col_hi), "s"(q.meta_row), "s"(q.meta_col), "s"(q.codes_row), "s"(q.codes_col),
                 "s"(q.scale_row_out), "s"(q.scale_col_out));
    if constexpr (CONV != 0)
        asm volatile("" ::"s"(q.conv), "s"(q.cC), "s"(q.cH), "s"(q.cW), "s"(q.ckh), "s"(q.ckw), "s"(q.pPH), "s"(q.pPW), "s"(q.pCN), "s"(q.pCP),
                     "s"(q.pLead), "s"(q.dHW.mul), "s"(q.dHW.sh1), "s"(q.dHW.sh2));
    if constexpr (CONV == kConvLines)
        asm volatile("" ::"s"(q.pPieces), "s"(q.pPerCh), "s"(q.pPerRow), "s"(q.pInvCh), "s"(q.pInvRow));
    return q;
}

// Workgroup number -> number in the tensor-after-tensor order.  With `spread`, the workgroups of
// tensor 0 (the stochastically rounded one of a per-tensor launch: twice the vector
// instructions per tile, a tenth of the bytes) stand at every spread-th place of the grid
// instead of in front of it, so that they run beside the memory-bound tiles of the others,
// not before them.
__device__ __forceinline__ int batch_order(const DualBatch& b)
{
    const int bid = (int)blockIdx.x;
    if (!b.spread) return bid;
    const int c0 = b.first[1], slot = bid / b.spread;
    if (bid - slot * b.spread == 0 && slot < c0) return slot;
    const int before = slot + 1 < c0 ? slot + 1 : c0;      // tensor 0's workgroups at or before this place
    return bid - before + c0;
}

// Wave w of a workgroup owns the tile at columns [64*wc, 64*wc + 64) of the
// workgroup's strip and rows [64*wr, 64*wr + 64), (wc, wr) = (w % WC, w / WC).
// One tile per wave and no register prefetch: what hides the memory latency is
// the number of resident waves, and a second tile in registers halves it
// (measured: 67 us against 85 us for pass 1 of a 65536 x 1152 tensor).
//
// ROUND selects the rounding of pass 2: bit 0 = stochastic along the rows, bit 1 =
// along the columns; kRoundPerTensor = every tensor of the launch is either nearest on
// both axes or stochastic on both, told by its own flags (a layer's X and W next to
// its G), so that the short, arithmetic-heavy stochastic tensor shares a launch with
// the long, memory-bound ones instead of running after them on a half-empty chip.
constexpr int kRoundPerTensor = 4;
constexpr int kRoundWide = 8;        // added to ROUND: codes of 5 to 8 bits, one per byte

// A convolution source: the workgroups' tiles, four rows of tiles high, are numbered strip by strip, and a
// workgroup takes one of them in pass 1, `steps` in a row in pass 2; its waves lie above each other.
template <bool QUANT, int ROUND, bool N64>
__device__ __forceinline__ void conv_block(const DualBatch& b, int k, int vb, float (*red)[2], float* lds)
{
    constexpr bool kStRow = (ROUND & 1) != 0, kStCol = (ROUND & 2) != 0, kWide = (ROUND & kRoundWide) != 0;
    const DualArgs q = whole_args<kConvLines>(b.t[k]);
    const int count = b.first[k + 1] - b.first[k];
    int local = vb - b.first[k];
    if (QUANT) local = count - 1 - local;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float* const piece = lds + wave * b.lds_per_wave;
    const int dense = b.dense ? b.words[k] : 0;
    Maxima max_row{}, max_col{};
    if (QUANT) {
        max_row = fetch_maxima(q.meta_row, dense);
        max_col = fetch_maxima(q.meta_col, dense);
    }
    const uint32_t strips = b.gx[k].d, row_tiles = (uint32_t)(q.rows / kTile);
    const uint32_t first = (uint32_t)local * (uint32_t)b.steps[k];
    uint32_t by = divide(first, b.gx[k]), strip = first - by * strips;
    PatchPieces pieces;
    auto live = [&](uint32_t y) { return 4 * y + (uint32_t)wave < row_tiles; };
    patch_pieces(pieces, q, lane);
    Scaling s_row{}, s_col{};
    if (QUANT) {
        s_row = scaling_of(max_row, q.meta_row, q.clip_row, q.b_row, dense);
        s_col = scaling_of(max_col, q.meta_col, q.clip_col, q.b_col, dense);
        if (local == 0 && threadIdx.x == 0) {
            q.meta_row->scale = s_row.scale;
            q.meta_col->scale = s_col.scale;
            if (q.scale_row_out) *q.scale_row_out = s_row.scale;
            if (q.scale_col_out) *q.scale_col_out = s_col.scale;
        }
    }
    DualCtx x;
    if (!QUANT) dual_setup<N64>(x, q, lane);
    float amax_row = 0.0f, amax_col = 0.0f;
    const int steps = QUANT ? b.steps[k] : 1;
    for (int step = 0; step < steps && live(by); ++step) {
        int l = lane;
        asm volatile("" : "+v"(l));      // (what follows from the lane is worked out where it is used, not kept for the loop)
        const int64_t row0 = (int64_t)(4 * by + wave) * kTile, col0 = (int64_t)strip * kTile;
        const PatchPlace at = patch_place(q, (uint32_t)row0, (uint32_t)col0);
        float4 v[kPieces];
        patch_load(v, pieces, at, q);
        const uint32_t signs = patch_store(v, piece, l);
        column_table(column_parts(piece), q, at.c_lo, (uint32_t)col0, l);
        wave_order();
        if (++strip == strips) { strip = 0; ++by; }
        if (QUANT) {
            line_tile<kStRow, kStCol, kWide, N64>(q, s_row, s_col, row0, col0, piece, l);
        } else {
            const bool negative = __builtin_amdgcn_ballot_w64((int)signs < 0) != 0;
            Tile t;
            tile_gather(t, q, piece, column_parts(piece), l);
            if (!negative && x.log2n_row >= 3 && x.log2n_col >= 3) sums_absmax(t, x, amax_row, amax_col);
            else dual_absmax(t, x, row0, col0, amax_row, amax_col);
            wave_order();
        }
    }
    if (!QUANT) record_max2(amax_row, amax_col, q.meta_row, q.meta_col, red, local, b.dense);
}

template <bool QUANT, int ROUND, bool N64, int CONV>
__device__ __forceinline__ void dual_block(const DualBatch& b, int k, int vb, float (*red)[2], float* lds)
{
    if (CONV == kConvLines && b.t[k].conv) {
        conv_block<QUANT, ROUND, N64>(b, k, vb, red, lds);
        return;
    }
    const DualArgs q = whole_args<CONV == kConvTiles ? kConvTiles : 0>(b.t[k]);
    const int count = b.first[k + 1] - b.first[k];
    // pass 2 walks a tensor from its end to its start: it begins with what pass 1
    // read last, which is most likely still in the memory-side cache
    int local = vb - b.first[k];
    if (QUANT) local = count - 1 - local;
    const int WC = b.WC[k];
    const uint32_t by32 = divide((uint32_t)local, b.gx[k]);
    const int64_t by = by32, bx = (uint32_t)local - by32 * b.gx[k].d;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int log2wc = WC >> 1, wc = wave & (WC - 1), wr = wave >> log2wc, WR = 4 >> log2wc;      // (WC is 1, 2 or 4)
    const int64_t col0 = (bx * WC + wc) * kTile;
    const int64_t row0 = (by * WR + wr) * kTile;
    // rows % 64 == cols % 64 == 0: a tile is entirely inside the tensor or entirely outside
    const bool live = col0 < q.cols && row0 < q.rows;

    DualCtx x;
    dual_setup<N64>(x, q, lane);
    const int dense = b.dense ? b.words[k] : 0;
    Maxima max_row{}, max_col{};         // (on their way before the tile)
    if (QUANT) {
        max_row = fetch_maxima(q.meta_row, dense);
        max_col = fetch_maxima(q.meta_col, dense);
    }
    Tile t;
    bool signs = true;                   // (of an ordinary source nobody asks: its passes wait for memory)
    if (live) {
        if (CONV == kConvTiles && q.conv) signs = tile_load_conv(t, q, row0, col0, lds + wave * b.lds_per_wave, lane);
        else tile_load(t, q, x, row0, col0);
    }
    if (QUANT) {
        const Scaling s_row = scaling_of(max_row, q.meta_row, q.clip_row, q.b_row, dense);
        const Scaling s_col = scaling_of(max_col, q.meta_col, q.clip_col, q.b_col, dense);
        dual_set_scaling(x, q, s_row, s_col, local == 0);
        if (live) dual_codes<(ROUND & 1) != 0, (ROUND & 2) != 0, (ROUND & kRoundWide) != 0>(t, x, row0, col0);
    } else {
        float amax_row = 0.0f, amax_col = 0.0f;
        if (CONV == kConvTiles && !signs && x.log2n_row >= 3 && x.log2n_col >= 3) sums_absmax(t, x, amax_row, amax_col);
        else if (live) dual_absmax(t, x, row0, col0, amax_row, amax_col);
        record_max2(amax_row, amax_col, q.meta_row, q.meta_col, red, local, b.dense);
    }
}

template <bool QUANT, int ROUND, bool N64, int CONV>
__global__ __launch_bounds__(kThreads, CONV == kConvLines ? 4 : 1) void fwht_dual_kernel(DualBatch b, AnyBatch ride)
{
    __shared__ float red[kThreads / kWave][2];
    extern __shared__ __attribute__((aligned(16))) float lds[];      // CONV: one patch per wave; riders' exchange

    if ((int)blockIdx.x >= b.first[kMaxDualBatch]) {
        any::batch_block<QUANT, false>(ride, hdqt::whole_args(ride.h), (int)blockIdx.x - b.first[kMaxDualBatch], &red[0][0], lds);
        return;
    }
    const int vb = QUANT ? batch_order(b) : (int)blockIdx.x;
    int k = 0;
#pragma unroll
    for (int j = 1; j < kMaxDualBatch; ++j) k = vb >= b.first[j] ? j : k;
    if constexpr ((ROUND & 7) == kRoundPerTensor) {
        // two complete bodies, chosen per workgroup: sharing anything between them
        // (one load, one setup) lets the compiler keep both paths' registers alive
        if (b.t[k].st_row) dual_block<QUANT, 3 | (ROUND & kRoundWide), N64, CONV>(b, k, vb, red, lds);
        else dual_block<QUANT, ROUND & kRoundWide, N64, CONV>(b, k, vb, red, lds);
    } else {
        dual_block<QUANT, ROUND, N64, CONV>(b, k, vb, red, lds);
    }
}

// floats of LDS of a wave: patch, column table; pass 2 by lines: codes on their way out
int conv_floats(const DualArgs& q, bool quant)
{
    if (q.conv == kConvTiles) return tile_patch_floats(q) + kTile;
    return kPatchFloats + kTile + (!quant ? 0 : q.b_row > 4 ? 16 * kTile : 8 * kTile);
}

bool all_order_64(const DualArgs* qs, int n)
{
    for (int k = 0; k < n; ++k)
        if (qs[k].log2n_row != 6 || qs[k].log2n_col != 6) return false;
    return true;
}

// waves of a workgroup side by side, and the workgroups of a tensor
int waves_across(const DualArgs& q)
{
    const int64_t strips = q.cols / kTile;
    if (q.conv == kConvLines) return 1;
    return (strips % 4 == 0) ? 4 : (strips % 2 == 0) ? 2 : 1;
}

bool make_batch(const DualArgs* qs, int n, bool dense, const AnyBatch* ride, bool quant, DualBatch* b)
{
    if (n < 1 || n > kMaxDualBatch) return false;
    b->dense = dense ? 1 : 0;
    int64_t total = 0;
    int lds = 0;
    for (int k = 0; k < n; ++k) {
        const DualArgs& q = qs[k];
        const int WC = waves_across(q);
        const int64_t gx = q.cols / kTile / WC, tiles = dual_workgroups(q);
        const int64_t steps = q.conv == kConvLines && quant ? q.pSteps : 1, wgs = (tiles + steps - 1) / steps;
        b->t[k] = q;
        if (q.conv) {
            const int need = conv_floats(q, quant);
            if (need > lds) lds = need;
        }
        b->first[k] = (int)total;
        b->gx[k] = make_divisor((uint32_t)gx);
        b->WC[k] = WC;
        b->words[k] = (int)tiles;
        b->steps[k] = (int)steps;
        total += wgs;
        if (total >= ((int64_t)1 << 30)) return false;
    }
    if (ride && ride->h.total >= (1 << 30)) return false;
    for (int k = n; k <= kMaxDualBatch; ++k) b->first[k] = (int)total;
    b->lds_per_wave = lds;
    b->spread = 0;
    return true;
}

} // namespace

int64_t dual_workgroups(const DualArgs& q)
{
    const int WC = waves_across(q);
    const int64_t tall = (int64_t)kTile * (4 / WC);
    return (q.cols / kTile / WC) * ((q.rows + tall - 1) / tall);
}

// Geometries the im2col source takes: odd windows, and tiles of 64 pixels that are whole
// image rows (W a power of two up to 64, H*W a multiple of 64) or lie inside one row
// (W a multiple of 64); the patch of a tile must fit the wave's share of LDS.
constexpr int kMaxPatchFloats = 3008;      // 12 KB per wave with the column table

bool dual_conv_plan(DualArgs* q)
{
    const int W = q->cW, H = q->cH, kh = q->ckh, kw = q->ckw;
    if (q->cC < 1 || H < 1 || W < 1 || kh < 1 || kw < 1 || kh % 2 == 0 || kw % 2 == 0) return false;
    if (kh > 15 || kw > 15) return false;
    const bool row_run = (W % kTile == 0);
    const bool whole_rows = (W < kTile) && (kTile % W == 0) && (((int64_t)H * W) % kTile == 0);
    if (!row_run && !whole_rows) return false;
    // one image is indexed with 32 bits
    if ((int64_t)q->cC * H * W >= ((int64_t)1 << 31) || q->rows >= ((int64_t)1 << 31) || q->cols >= ((int64_t)1 << 31))
        return false;
    if (q->rows % ((int64_t)H * W) != 0 || q->cols != (int64_t)q->cC * kh * kw) return false;
    q->pPH = (row_run ? 1 : kTile / W) + kh - 1;
    q->pPW = (row_run ? kTile : W) + kw - 1;
    // (what is refused has always been told from one channel more than some windows need)
    if (((kTile - 1) / (kh * kw) + 2) * q->pPH * q->pPW > kMaxPatchFloats) return false;
    q->pCN = (kTile - 2) / (kh * kw) + 2;      // 64 columns that start at any tap of a channel
    q->dHW = make_divisor((uint32_t)(H * W)); q->dW = make_divisor((uint32_t)W);
    q->dTaps = make_divisor((uint32_t)(kh * kw)); q->dkw = make_divisor((uint32_t)kw);
    q->pLead = (kw - 1) / 2;
    q->pCP = q->pPH * q->pPW;
    q->conv = kConvTiles;
    // By lines where a row is a whole number of pieces, one image is addressed with 31 bits and the patch is no more than a
    // lane's pieces in flight.  Seven pieces behind every channel put the columns of a tile on different banks (two or
    // three of 64 lanes on one, up to eight without them); one, or none, where seven would make it longer than that.
    const int wt = row_run ? kTile : W, lead = (q->pLead + 3) & ~3;
    const uint32_t per_row = (uint32_t)(wt + 2 * lead) / 4, bare = per_row * (uint32_t)q->pPH, most = 64u * kPieces / (uint32_t)q->pCN;
    if (W < 4 || (int64_t)q->cC * H * W >= ((int64_t)1 << 29) || bare > most) return true;
    q->conv = kConvLines;
    const uint32_t per_ch = bare + 7 <= most ? bare + 7 : bare + 1 <= most ? bare + 1 : bare;
    q->pLead = lead; q->pPW = 4 * (int)per_row; q->pCP = 4 * (int)per_ch;
    q->pPieces = per_ch * (uint32_t)q->pCN; q->pPerCh = per_ch; q->pPerRow = per_row;
    q->pInvCh = ((1u << 20) + per_ch - 1) / per_ch;
    q->pInvRow = ((1u << 20) + per_row - 1) / per_row;
    // pass 2: as many tiles a wave as make one round of the chip's workgroups
    const int64_t tiles = q->cols / kTile * ((q->rows / kTile + 3) / 4);
    int64_t places = (160 << 10) / (4 * (int64_t)sizeof(float) * conv_floats(*q, true));
    places = 256 * (places < 1 ? 1 : places > 4 ? 4 : places);
    q->pSteps = (int)((tiles + places - 1) / places);
    return true;
}

bool quantize_dual_eligible(const DualArgs& q)
{
    if (q.cols >= ((int64_t)1 << 26) || q.rows >= ((int64_t)1 << 26)) return false;      // 32-bit lane offsets
    return (q.rows % kTile == 0) && (q.cols % kTile == 0) && q.log2n_row <= 6 && q.log2n_col <= 6 &&
           q.b_row <= 8 && q.b_col <= 8 && (q.b_row <= 4) == (q.b_col <= 4) &&
           (q.rows / kTile) * (q.cols / kTile) < ((int64_t)1 << 30);
}

// The way of a convolution source among the tensors (a launch has one at most), 0 without one.
int conv_among(const DualArgs* qs, int n)
{
    int conv = 0;
    for (int k = 0; k < n; ++k)
        if (qs[k].conv) conv = qs[k].conv;
    return conv;
}

// Dynamic LDS of a launch: the patches of a convolution source, or the riders' exchange
size_t launch_lds(const DualBatch& b, const AnyBatch* ride)
{
    size_t lds = (size_t)(kThreads / kWave) * b.lds_per_wave;
    if (ride && ride->h.n && lds < any::kLdsFloats) lds = any::kLdsFloats;
    return lds * sizeof(float);
}

// Pass 1 (all maxima) of n tensors and the riders in one launch; without `dense` their
// calibration records must be zero.
hipError_t launch_dual_pass1(const DualArgs* qs, int n, bool dense, const AnyBatch* ride, hipStream_t stream)
{
    static const AnyBatch none{};
    if (!ride) ride = &none;
    DualBatch b;
    if (!make_batch(qs, n, dense, ride, false, &b)) return hipErrorInvalidValue;
    const int id = n > 1 ? K_DUAL_ABSMAX_BATCH
                         : (qs[0].profile_tag ? K_DUAL_ABSMAX_X + (qs[0].profile_tag - 1) : K_DUAL_ABSMAX);
    ProfileScope ps(id, stream);
    const dim3 grid((unsigned)(b.first[n] + ride->h.total)), block(kThreads);
    const size_t lds = launch_lds(b, ride);
    const bool n64 = all_order_64(qs, n);
    const int conv = conv_among(qs, n);
#define HDQT_LAUNCH_PASS1(CONV)                                                                     \
    do {                                                                                            \
        if (n64) hipLaunchKernelGGL((fwht_dual_kernel<false, 0, true, CONV>), grid, block, lds, stream, b, *ride); \
        else hipLaunchKernelGGL((fwht_dual_kernel<false, 0, false, CONV>), grid, block, lds, stream, b, *ride); \
    } while (0)
    if (conv == kConvLines) HDQT_LAUNCH_PASS1(kConvLines);
    else if (conv == kConvTiles) HDQT_LAUNCH_PASS1(kConvTiles);
    else HDQT_LAUNCH_PASS1(0);
#undef HDQT_LAUNCH_PASS1
    return hipGetLastError();
}

// Whether the tensors can share a pass-2 launch: same rounding modes everywhere, or each
// tensor nearest on both axes or stochastic on both; and all of them with packed 4-bit
// codes or all with a byte per code.
bool dual_pass2_batchable(const DualArgs* qs, int n)
{
    bool same = true, paired = true;
    for (int k = 0; k < n; ++k) {
        if ((qs[k].b_row <= 4) != (qs[0].b_row <= 4)) return false;
        if (qs[k].st_row != qs[0].st_row || qs[k].st_col != qs[0].st_col) same = false;
        if (qs[k].st_row != qs[k].st_col) paired = false;
    }
    return same || paired;
}

// Pass 2 (both code sets) of n tensors in one launch (see dual_pass2_batchable).
hipError_t launch_dual_pass2(const DualArgs* qs, int n, bool dense, const AnyBatch* ride, hipStream_t stream)
{
    static const AnyBatch none{};
    if (!ride) ride = &none;
    DualBatch b;
    if (!make_batch(qs, n, dense, ride, true, &b) || !dual_pass2_batchable(qs, n)) return hipErrorInvalidValue;
    bool same = true;
    for (int k = 1; k < n; ++k)
        if (qs[k].st_row != qs[0].st_row || qs[k].st_col != qs[0].st_col) same = false;
    const int id = n > 1 ? K_DUAL_QUANT_BATCH
                         : (qs[0].profile_tag ? K_DUAL_QUANT_X + (qs[0].profile_tag - 1) : K_DUAL_QUANT);
    ProfileScope ps(id, stream);
    const dim3 grid((unsigned)(b.first[n] + ride->h.total)), block(kThreads);
    const bool n64 = all_order_64(qs, n);
    const size_t lds = launch_lds(b, ride);
    const int conv = conv_among(qs, n);
#define HDQT_LAUNCH_ORDER(ROUND, CONV)                                                               \
    do {                                                                                            \
        if (n64) hipLaunchKernelGGL((fwht_dual_kernel<true, ROUND, true, CONV>), grid, block, lds, stream, b, *ride); \
        else hipLaunchKernelGGL((fwht_dual_kernel<true, ROUND, false, CONV>), grid, block, lds, stream, b, *ride); \
    } while (0)
#define HDQT_LAUNCH_PASS2(ROUND)                                                                     \
    do {                                                                                            \
        if (conv == kConvLines) HDQT_LAUNCH_ORDER(ROUND, kConvLines);                               \
        else if (conv == kConvTiles) HDQT_LAUNCH_ORDER(ROUND, kConvTiles);                          \
        else HDQT_LAUNCH_ORDER(ROUND, 0);                                                           \
    } while (0)
    const int mode = !same ? kRoundPerTensor : (qs[0].st_row ? 1 : 0) | (qs[0].st_col ? 2 : 0);
    // A stochastic tensor in front of nearest ones: its workgroups among theirs (see batch_order),
    // over the first three quarters of the grid (a heavy workgroup among the last ones is the
    // kernel's tail: spread over the whole grid the launch took 102 us instead of 95.6) and at
    // an odd distance: workgroups go to the eight XCDs in turn, and at a distance of 8 (6) every
    // heavy one lands on the same XCD (on four of them): 122 (100) us.  At 7: 93.4 us.
    if (mode == kRoundPerTensor && qs[0].st_row && b.first[1] > 0) {
        bool rest_nearest = true;
        for (int k = 1; k < n; ++k) rest_nearest = rest_nearest && !qs[k].st_row;
        int64_t q = (int64_t)b.first[n] * 3 / (4 * (int64_t)b.first[1]);
        if (q % 2 == 0) --q;
        if (rest_nearest && q >= 3 && q < ((int64_t)1 << 30)) b.spread = (int)q;
    }
    if (qs[0].b_row > 4) {
        switch (mode) {
        case kRoundPerTensor: HDQT_LAUNCH_PASS2(kRoundPerTensor | kRoundWide); break;
        case 3: HDQT_LAUNCH_PASS2(3 | kRoundWide); break;
        case 1: HDQT_LAUNCH_PASS2(1 | kRoundWide); break;
        case 2: HDQT_LAUNCH_PASS2(2 | kRoundWide); break;
        default: HDQT_LAUNCH_PASS2(0 | kRoundWide); break;
        }
    } else {
        switch (mode) {
        case kRoundPerTensor: HDQT_LAUNCH_PASS2(kRoundPerTensor); break;
        case 3: HDQT_LAUNCH_PASS2(3); break;
        case 1: HDQT_LAUNCH_PASS2(1); break;
        case 2: HDQT_LAUNCH_PASS2(2); break;
        default: HDQT_LAUNCH_PASS2(0); break;
        }
    }
#undef HDQT_LAUNCH_PASS2
#undef HDQT_LAUNCH_ORDER
    return hipGetLastError();
}

// (A one-launch variant for small tensors -- tile kept in registers across a grid-wide barrier --
// was built and measured: correct, but the cooperative launch it needs for a guaranteed
// co-resident grid costs about 25 us more than an ordinary launch on this stack, more than the
// launch it saves.)

} // namespace hdqt
