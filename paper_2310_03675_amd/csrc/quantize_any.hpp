// Hadamard-domain quantization of a tensor of any shape along one axis: the device side shared by
// the batch kernel (quantize.hip) and the launches in which small tensors ride along with a large
// one (quantize_dual.hip).
//
// A thread holds eight consecutive contraction indices and nothing else, so a small tensor is
// spread over as many waves as it has (a layer of 64 x 256 x 128: 44 workgroups for its six code
// sets instead of 4 waves with 64 values a lane).
//   axis 1: thread = eight codes of one line; larger strides pair neighbouring lanes.  Lines of
//     any length: a line's last thread holds what is left, the codes behind it are zeros.
//   axis 0: lane (rg, cg) = (lane / 8, lane % 8) has rows 8 rg .. 8 rg + 7 of column cg of the
//     wave's 64 x 8 piece; strides 8, 16, 32 pair lanes, 64 and 128 pair waves through LDS.
// What bounds a small launch is one chain of trips: to the arguments, to the tensor, in pass 2 to the
// maxima.  The arguments come in two trips (whole_args), the maxima are on their way before the
// tensor, nothing is divided (Divisor) and no reduction goes through LDS permutes: the step of 64 x 256 x 128
// 14.4 -> 10.7 us together with the product's kernel, quantize of 1315 x 362 7.5 -> 6.2 us, of which an empty
// kernel has 1.6 a launch.
// The butterfly runs with strides 1, 2, 4, ..., n/2 in that order: this fixes the binary32
// rounding to the balanced pairwise tree over the signed terms in natural index order.
#pragma once
#include "common.hpp"
#include "lane_ops.hpp"

namespace hdqt {
namespace any {

using namespace lanes;

constexpr int kThreads = 256;
constexpr int kRandPitch = 5;                                // dwords per row of random halfwords
constexpr int kLdsFloats = 8 * kThreads;                     // cross-wave exchange; the random words of
static_assert(4 * 64 * kRandPitch <= kLdsFloats, "four waves' random words fit the exchange buffer");

// rows of any length in bytes or elements: dwords at any address
struct __attribute__((packed, aligned(4))) Float4 { float x, y, z, w; };
struct __attribute__((packed)) Dword { uint32_t v; };

// The eight halfwords of elements e .. e+7 (e & 7 == 0: one Philox block, else two).
__device__ __forceinline__ void random8(const QuantArgs& q, uint64_t e, uint32_t r[4])
{
    const uint64_t blk = e >> 3;
    philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), q.tensor_id, 0u, q.seed_lo, q.seed_hi, r);
    if ((q.cols & 7) == 0) return;       // (uniform) e is a multiple of 8 then
    uint32_t n[4];
    philox4x32_10((uint32_t)(blk + 1), (uint32_t)((blk + 1) >> 32), q.tensor_id, 0u, q.seed_lo, q.seed_hi, n);
    // the 16 halfwords from number e & 7 on
    const uint32_t sh = (uint32_t)e & 7u;
    const uint32_t m4 = (sh & 4) ? ~0u : 0u, m2 = (sh & 2) ? ~0u : 0u;
    const uint32_t w[8] = {r[0], r[1], r[2], r[3], n[0], n[1], n[2], n[3]};
    uint32_t x[6], y[5];
#pragma unroll
    for (int k = 0; k < 6; ++k) x[k] = (w[k + 2] & m4) | (w[k] & ~m4);
#pragma unroll
    for (int k = 0; k < 5; ++k) y[k] = (x[k + 1] & m2) | (x[k] & ~m2);
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = __builtin_amdgcn_alignbyte(y[k + 1], y[k], 2 * (sh & 1));
}

// eight codes of one line, `count` of them inside it (zero bits behind them)
__device__ __forceinline__ void store8(const QuantArgs& q, const uint32_t cw[8], uint8_t* dst, int count)
{
    if (q.b <= 4) {
        uint32_t w = pack_nibbles(cw);
        if (count >= 8) {
            reinterpret_cast<Dword*>(dst)->v = w;
        } else {
            // (a zero behind the line is no zero where the step's inverse is infinite)
            w &= (1u << (4 * count)) - 1u;
            for (int k = 0; 2 * k < count; ++k) dst[k] = (uint8_t)(w >> (8 * k));
        }
    } else {
        const uint32_t w0 = pack_bytes(cw), w1 = pack_bytes(cw + 4);
        if (count >= 8) {
            reinterpret_cast<Dword*>(dst)[0].v = w0;
            reinterpret_cast<Dword*>(dst)[1].v = w1;
        } else {
            for (int k = 0; k < count; ++k) dst[k] = (uint8_t)((k < 4 ? w0 : w1) >> (8 * (k & 3)));
        }
    }
}

__device__ __forceinline__ void emit(const QuantArgs& q, const float v[8], const uint32_t rnd[4], float inv,
                                     uint8_t* dst, int count)
{
    const float qminf = (float)(-(1 << (q.b - 1))), qmaxf = (float)((1 << (q.b - 1)) - 1);
    const float magic = kMagic + (q.b <= 4 ? 8.0f : 128.0f);
    uint32_t cw[8];
    if (q.stochastic) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            cw[i] = code_word<true>(v[i], inv, qminf, qmaxf, magic, sr_halfword(rnd, (uint32_t)i));
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) cw[i] = code_word<false>(v[i], inv, qminf, qmaxf, magic, 0u);
    }
    store8(q, cw, dst, count);
}

// Eight values of a thread, where they come from (number of the first element, of the random bits) and where their
// codes go (bytes).
struct Eight {
    float v[8];
    int64_t from, to;
    int count;                           // of them inside the tensor
    bool last;                           // of a line
};

// The zeros behind a line whose codes are padded (a few bytes of one thread in a line's many).  Written before the transform: behind the codes
// they cost fwht_dual_kernel<true, 4, true, 0>, which takes such tensors along, 30 registers and its fourth wave per SIMD
// (65536 x 1152 x 128's step 252.6 / 254.9 us).
__device__ __forceinline__ void zeros_behind(const QuantArgs& q, const Eight& t)
{
    if (!t.last || !t.count) return;
    uint8_t* dst = q.codes + t.to + (q.b <= 4 ? (t.count + 1) >> 1 : t.count);
#pragma unroll 1
    for (int k = 0; k < q.pad; ++k) dst[k] = 0;
}

// Those of a workgroup's piece of the tensor, loads only.
template <int AXIS>
__device__ __forceinline__ void load8(Eight& t, const QuantArgs& q, const AnyPlan& p, int piece, int64_t pitch)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = q.b <= 4 ? 4 : 8;    // bytes of eight codes
    t.count = 0;
    if (AXIS) {
        // (the workgroup's first line: a 32-bit division wherever that is enough)
        const int64_t base = (int64_t)piece * kThreads;
        const int64_t line0 = piece < (1 << 23) ? (int64_t)divide((uint32_t)base, p.per) : base / (int64_t)p.per.d;
        const uint32_t at = (uint32_t)(base - line0 * p.per.d) + (uint32_t)tid;
        const uint32_t down = divide(at, p.per);
        const uint32_t j = at - down * p.per.d;
        const int64_t line = line0 + down;
        t.from = line * q.cols + 8 * (int64_t)j;
        const float* src = q.T + t.from;
        if (line < q.rows) {
            const int64_t left = q.cols - 8 * (int64_t)j;
            t.count = left < 8 ? (int)left : 8;
        }
        if (t.count == 8) {
            const Float4 lo = reinterpret_cast<const Float4*>(src)[0], hi = reinterpret_cast<const Float4*>(src)[1];
            t.v[0] = lo.x; t.v[1] = lo.y; t.v[2] = lo.z; t.v[3] = lo.w;
            t.v[4] = hi.x; t.v[5] = hi.y; t.v[6] = hi.z; t.v[7] = hi.w;
        } else {
            // (seven at most; with an eighth the compiler makes its load one with the eighth of a whole piece, three loads
            // then: 9431 x 301 10.1 / 10.8 us, 18863 x 301 with nothing else changed 16.0 / 16.6)
#pragma unroll
            for (int i = 0; i < 7; ++i) t.v[i] = i < t.count ? src[i] : 0.0f;
            t.v[7] = 0.0f;
        }
        t.to = line * pitch + (int64_t)j * per;
        t.last = j + 1 == p.per.d;
    } else {
        const uint32_t across = divide((uint32_t)piece, p.per);
        const int64_t by = across, bx = (uint32_t)piece - across * p.per.d;
        const int wc = wave & (p.wc - 1), wr = wave >> (p.wc >> 1);      // (wc: 1, 2 or 4)
        const int rg = lane >> 3, cg = lane & 7;
        const int64_t row0 = (by * (4 >> (p.wc >> 1)) + wr) * 64, col0 = (bx * p.wc + wc) * 8;       // the wave's piece
        const int64_t row = row0 + rg * 8, col = col0 + cg;
        if (col < q.cols && row < q.rows) {
            const int64_t left = q.rows - row;
            t.count = left < 8 ? (int)left : 8;
        }
        // (clamped addresses: every load is unconditional)
        const int64_t rc = t.count ? row : 0, cc = t.count ? col : 0;
        const float* src = q.T + rc * q.cols + cc;
#pragma unroll
        for (int i = 0; i < 8; ++i) t.v[i] = src[(i < t.count ? i : 0) * q.cols];
        t.from = (row + cg) * q.cols + col0;
        t.to = col * pitch + (row >> 3) * per;
        t.last = row + 8 >= q.rows;
    }
}

// Their transform, and in pass 2 their random bits.
template <bool QUANT, int AXIS>
__device__ __forceinline__ void transform8(Eight& t, const QuantArgs& q, uint32_t (&rnd)[4], float* lds)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float (&v)[8] = t.v;
    if (AXIS) {
        butterfly8(v, q.log2n);
        if (q.log2n > 3) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = stage_dpp<1>(v[i], (uint32_t)(lane & 1) << 31);
        }
        if (q.log2n > 4) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = stage_dpp<2>(v[i], (uint32_t)(lane & 2) << 30);
        }
        if (q.log2n > 5) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = stage_dpp<4>(v[i], (uint32_t)(lane & 4) << 29);
        }
        if (q.log2n > 6) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = stage_dpp<8>(v[i], (uint32_t)(lane & 8) << 28);
        }
        if (q.log2n > 7) {
#pragma unroll
            for (int i = 0; i < 8; i += 2) stage_swap<false>(v[i], v[i + 1]);
        }
        if (QUANT && q.stochastic) random8(q, (uint64_t)t.from, rnd);
    } else {
        const int rg = lane >> 3, cg = lane & 7;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = i < t.count ? v[i] : 0.0f;
        butterfly8(v, q.log2n);
        if (q.log2n > 3) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = stage_dpp<8>(v[i], (uint32_t)(lane & 8) << 28);
        }
        if (q.log2n > 4) {
#pragma unroll
            for (int i = 0; i < 8; i += 2) stage_swap<false>(v[i], v[i + 1]);
        }
        if (q.log2n > 5) {
#pragma unroll
            for (int i = 0; i < 8; i += 2) stage_swap<true>(v[i], v[i + 1]);
        }
        // strides 64 and 128: the partner is another wave (four waves on top of each other: plan_any)
        for (int st = 6; st < q.log2n; ++st) {
            const int mask = 64 << (st - 6);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; ++i) lds[i * kThreads + tid] = v[i];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float other = lds[i * kThreads + (tid ^ mask)];
                v[i] = (tid & mask) ? other - v[i] : v[i] + other;
            }
        }
        if (QUANT && q.stochastic) {
            // the wave's 64 rows of eight halfwords: lane (rg, cg) draws row 8 rg + cg, then
            // reads column cg of its own eight rows
            if (q.log2n > 6) __syncthreads();
            uint32_t* words = reinterpret_cast<uint32_t*>(lds) + wave * 64 * kRandPitch;
            random8(q, (uint64_t)t.from, rnd);
            // LDS operations of one wave are carried out in order; the fences keep the compiler
            // from moving reads above the writes of other lanes, and writes above the last piece's reads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < 4; ++k) words[(rg * 8 + cg) * kRandPitch + k] = rnd[k];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint16_t* half = reinterpret_cast<const uint16_t*>(words);
#pragma unroll
            for (int i = 0; i < 8; i += 2)
                rnd[i >> 1] = (uint32_t)half[(rg * 8 + i) * 2 * kRandPitch + cg] |
                              (uint32_t)half[(rg * 8 + i + 1) * 2 * kRandPitch + cg] << 16;
        }
    }
}

__device__ __forceinline__ void publish(const QuantArgs& q, const Scaling& sc, int local)
{
    if (local == 0 && threadIdx.x == 0) {
        q.meta->scale = sc.scale;
        if (q.scale_out) *q.scale_out = sc.scale;
    }
}

__device__ __forceinline__ float largest8(const Eight& t, float amax)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(t.v[i]));
    return amax;
}

// One workgroup of one tensor: transform, then the maximum (returned) or the codes.  `local` is
// the workgroup's number within the tensor, `p` how the tensor is cut (plan_any).  Here it has one piece of it.
template <bool QUANT>
__device__ __forceinline__ float block(const QuantArgs& q, const AnyPlan& p, int local, float* lds)
{
    const int64_t pitch = (q.b <= 4 ? ((q.axis ? q.cols : q.rows) + 1) >> 1 : (q.axis ? q.cols : q.rows)) + q.pad;
    Maxima maxima{};
    if (QUANT) maxima = fetch_maxima(q.meta, p.dense);
    Eight t;
    uint32_t rnd[4] = {0, 0, 0, 0};
    if (q.axis) {
        load8<1>(t, q, p, local, pitch);
        if (QUANT) zeros_behind(q, t);
        transform8<QUANT, 1>(t, q, rnd, lds);
    } else {
        load8<0>(t, q, p, local, pitch);
        if (QUANT) zeros_behind(q, t);
        transform8<QUANT, 0>(t, q, rnd, lds);
    }
    if (!QUANT) return largest8(t, 0.0f);
    const Scaling sc = scaling_of(maxima, q.meta, q.clip, q.b, p.dense);
    publish(q, sc, local);
    if (t.count) emit(q, t.v, rnd, sc.inv, q.codes + t.to, t.count);
    return 0.0f;
}

// Here p.steps pieces one after the other, the next one's values on their way while this one's are worked on: in a
// tensor of thousands of pieces the trips and the scaling in front of a piece took most of its time (finish_any says where).
// (Not with the axis told apart inside the loop: where its two sides meet the compiler copies every value.  p.pieces and
// p.steps are not among whole_args' members: with them there these sets gain nothing, and small ones lose a little.)
template <bool QUANT, int AXIS>
__device__ __forceinline__ float block_of_many(const QuantArgs& q, const AnyPlan& p, int local, float* lds)
{
    const int64_t pitch = (q.b <= 4 ? ((AXIS ? q.cols : q.rows) + 1) >> 1 : (AXIS ? q.cols : q.rows)) + q.pad;
    Maxima maxima{};
    if (QUANT) maxima = fetch_maxima(q.meta, p.dense);
    int piece = local * p.steps;
    const int last = piece + p.steps < p.pieces ? piece + p.steps : p.pieces;
    Eight next;
    load8<AXIS>(next, q, p, piece, pitch);
    Scaling sc{};
    float amax = 0.0f;
    for (bool first = true; piece < last; ++piece, first = false) {
        Eight t = next;
        if (piece + 1 < last) load8<AXIS>(next, q, p, piece + 1, pitch);
        uint32_t rnd[4] = {0, 0, 0, 0};
        if (QUANT) zeros_behind(q, t);
        transform8<QUANT, AXIS>(t, q, rnd, lds);
        if (QUANT) {
            if (first) {
                sc = scaling_of(maxima, q.meta, q.clip, q.b, p.dense);
                publish(q, sc, local);
            }
            if (t.count) emit(q, t.v, rnd, sc.inv, q.codes + t.to, t.count);
        } else {
            amax = largest8(t, amax);
        }
    }
    return amax;
}

// both passes of workgroup `vb` of a batch; `red`: one float per wave
template <bool QUANT, bool MANY>
__device__ __forceinline__ void batch_block(const AnyBatch& b, const AnyHeader& h, int vb, float* red, float* lds)
{
    int k = 0, local = vb;
#pragma unroll
    for (int j = 1; j < kMaxAny; ++j) {
        const bool beyond = vb >= h.first[j];
        k = beyond ? j : k;
        local = beyond ? vb - h.first[j] : local;
    }
    const AnyTensor t = whole_args(b.t[k]);
    if (QUANT) local = t.p.count - 1 - local;      // what pass 1 read last is in the caches still
    float m;
    if constexpr (!MANY) m = block<QUANT>(t.q, t.p, local, lds);
    else m = t.q.axis ? block_of_many<QUANT, 1>(t.q, t.p, local, lds) : block_of_many<QUANT, 0>(t.q, t.p, local, lds);
    if (!QUANT) record_max(m, t.q.meta, red, local, t.p.dense);
}

} // namespace any
} // namespace hdqt
