// Shared declarations of the HDQT device library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hdqt {

constexpr int kMaxHadamard = 256;   // largest supported block order
constexpr int kWave = 64;

// Per-operand calibration record in the workspace.  `scale` is the value of one code step,
// written by pass 2; max|y| is reduced in one of two ways, the same for every tensor of a launch:
//   * up to kDenseMost workgroups of pass 1 store their maxima side by side, one word each, and
//     every wave of pass 2 reads them all.  Nothing has to be cleared beforehand: the launch
//     that clears the records is 2.5 us and a gap, one of six of a small layer's step.
//   * more workgroups use integer atomicMax on the bit patterns (non-negative floats order like
//     unsigned integers) in a record that was cleared.  Atomics on one address are serialised,
//     so the workgroups spread over 64 slots, each on its own 128-byte line; pass 2 reads one
//     slot per lane and finishes the reduction inside the wave.
constexpr int kAmaxSlots = 64;
constexpr int kAmaxSlotStride = 32;     // dwords
constexpr int kDenseMost = 1024;        // sixteen words per lane of pass 2
struct QMeta {
    float scale;
    uint32_t pad[31];
    uint32_t amax[kAmaxSlots * kAmaxSlotStride];
};
constexpr int64_t kQMetaDwords = sizeof(QMeta) / 4;

// One quantize request, resolved by the host.
struct QuantArgs {
    const float* T;
    int64_t rows, cols;     // source tensor, row-major
    int axis;               // 1: contraction along a row, 0: along a column
    int log2n;              // log2 of the block order actually used
    int b;                  // code width
    int stochastic;         // 0 nearest-even, 1 stochastic
    float clip;
    uint32_t tensor_id;
    uint32_t seed_lo, seed_hi;
    QMeta* meta;            // device
    uint8_t* codes;         // device, packed, contraction-major
    float* scale_out;       // device, may alias &meta->scale, may be null
    int pad;                // bytes of zeros behind a line of codes (any-shape kernel only)
};

// n / d for any 32-bit n, by multiplication (Granlund and Montgomery, PLDI'94, with the round-up
// multiplier): a handful of scalar instructions instead of some forty vector ones.
struct Divisor {
    uint32_t d, mul, sh1, sh2;
};
inline Divisor make_divisor(uint32_t d)
{
    uint32_t l = 0;
    while (((uint64_t)1 << l) < d) ++l;
    const uint64_t mul = ((((uint64_t)1 << l) - d) << 32) / d + 1;      // (2^(32 + l) / d, rounded up, minus 2^32)
    return {d, (uint32_t)mul, l < 1 ? l : 1, l < 1 ? 0 : l - 1};
}
__host__ __device__ __forceinline__ uint32_t divide(uint32_t n, const Divisor& v)
{
    const uint32_t t = (uint32_t)(((uint64_t)v.mul * n) >> 32);
    return (t + ((n - t) >> v.sh1)) >> v.sh2;
}

// How the any-shape kernel cuts one tensor of a launch (plan_any).
struct AnyPlan {
    int count;              // its workgroups
    int dense;              // `count` if the maxima stand side by side, 0 for atomic slots
    int wc;                 // axis 0: waves side by side in a workgroup (1, 2 or 4)
    Divisor per;            // axis 1: threads per line; axis 0: pieces along the columns
    int pieces, steps;      // of 2048 values; how many of them a workgroup takes one after the other
};
constexpr int kMaxAny = 6;
struct AnyTensor {
    QuantArgs q;
    AnyPlan p;
};
struct AnyHeader {
    int first[kMaxAny];     // a tensor's first workgroup in the launch, INT_MAX behind the last tensor
    int n;
    int total;              // workgroups
};
struct AnyBatch {
    AnyHeader h;
    AnyTensor t[kMaxAny];
};

// One tensor quantized along both axes from one read ("row" = axis 1, along the
// columns; "col" = axis 0, along the rows).
enum ConvWay { kConvLines = 1, kConvTiles = 2 };      // how a convolution source is read: see quantize_dual.hip

struct DualArgs {
    const float* T;
    int64_t rows, cols;
    int log2n_row, log2n_col;
    int b_row, st_row;
    float clip_row;
    uint32_t tid_row;
    int b_col, st_col;
    float clip_col;
    uint32_t tid_col;
    uint32_t seed_row_lo, seed_row_hi;   // Philox key per axis
    uint32_t seed_col_lo, seed_col_hi;
    QMeta* meta_row;
    QMeta* meta_col;
    uint8_t* codes_row;     // [rows, cols/2]
    uint8_t* codes_col;     // [cols, rows/2]
    float* scale_row_out;   // may be null
    float* scale_col_out;
    int pad_row, pad_col;   // of its halves, where the any-shape kernel has them
    int profile_tag;        // which tensor of the step this is (timing table only): 0 none, 1 X, 2 W, 3 G
    // Convolution source (conv != 0): T points at an activation [batch, C, H, W] and the
    // tensor that is quantized is its im2col matrix for a kh x kw window, stride 1, zero
    // padding (kh - 1) / 2 and (kw - 1) / 2: row = pixel (b, y, x), column c*kh*kw + ty*kw + tx
    // holds act[b, c, y + ty - ph, x + tx - pw].  rows = batch*H*W, cols = C*kh*kw.
    int conv;               // 0 or one of ConvWay
    int cC, cH, cW, ckh, ckw;
    int pPH, pPW, pCN;      // the part of the activation a 64 x 64 tile reads: rows, row length in LDS, channels
    int pCP, pLead;         // distance of its channels in LDS; of a row's first pixel from the row's start
    // kConvLines alone:
    uint32_t pPieces, pPerCh, pPerRow;       // 16-byte pieces of the part, of a channel, of a row
    uint32_t pInvCh, pInvRow;                // 2^20 / pPerCh and / pPerRow, rounded up
    int pSteps;             // tiles a wave of pass 2 takes one after the other
    // both:
    Divisor dHW, dW, dTaps, dkw;
};

struct GemmArgs {
    const uint8_t* qA;      // [RA, pitchA] packed codes
    const uint8_t* qB;      // [RB, pitchB]
    int64_t pitchA, pitchB;
    int bA, bB;
    int64_t RA, RB, D;
    int64_t s;              // tile length in codes
    int s_pad;              // tile length rounded up to the MFMA K granularity
    int64_t n_tiles;        // ceil(D / s)
    int acc_lo, acc_hi;     // accumulator range [-2^(a-1), 2^(a-1)-1]
    int acc_lo_scaled, acc_hi_scaled;   // the same bounds times 256 (set by the 4-bit fast path)
    int jA, jB, fin_shift;              // 16-bit saturation path: operand factors 2^jA, 2^jB; 16 - acc_bits
    const float* scaleA;    // device scalars
    const float* scaleB;
    float inv_n;            // 1 / n_eff (a power of two)
    float* out;             // [RA, RB] or null
    uint16_t* out_bf16;     // [RA, RB] bfloat16 patterns or null: the same values, narrowed (nearest even)
    const float* mask_src;  // null, or a tensor of the fp32 output's shape: the output is written
                            // where mask_src > 0 and +0 elsewhere (the rectifier's backward pass
                            // behind an input gradient); the integer outputs are not masked
    bool padded;            // D is an odd contraction with zeros behind it (asked for masked products only)
    int32_t* acc_out;       // [RA, RB] or null
    int partial16;          // the slices hold 16-bit integers (a part's totals fit: parts of few tiles)
    int32_t* partial;       // [splits, RA, RB] when splits > 1: one slice per part of the contraction;
                            // second reading of the accumulator: [n_tiles, RA, RB], every tile's sums
    uint32_t* tile_max;     // second reading only: max |tile sum| per tile, zero beforehand
    int req_bits;           // second reading in the matrix-core kernel: a, and the clamp bounds
    float req_lo, req_hi;   // -2^(a-1) and 2^(a-1) - 1, each plus 1.5 * 2^23
    int stream_out;         // output too large to stay cached, in whole lines: written with streaming stores
    int profile_tag;        // which matmul of the step this is (timing table only): 0 none, 1 + kind
    int splits;             // workgroups sharing one output tile along the contraction
    int64_t tiles_per_split;
    // Fold (fold != 0): the product is the gradient of an im2col matrix, qA holds the codes of
    // G [batch*H*W pixels, D], qB those of W [C*kh*kw, D], and what is written is the gradient
    // of the activation, out[batch, C, H, W]: the accumulators of a pixel's kh*kw taps are
    // added up (exact integers) and dequantized once (gemm_fold.hip).
    int fold;
    int fC, fH, fW, fkh, fkw;
    int64_t fbatch;
};
// fills the fold fields from the geometry; false if the kernel does not take it
bool gemm_fold_plan(GemmArgs* g, int64_t batch, int C, int H, int W, int kh, int kw);
hipError_t launch_gemm_fold(const GemmArgs& g, hipStream_t stream);

// Unfolding of an activation [batch, C, H, W] into X [M = batch*Ho*Wo, K = C*kh*kw] (im2col.hip)
struct Im2colArgs {
    const float* act;
    float* X;
    int64_t M;              // rows of X; of launch_col2im: pixels of the activation, batch*H*W
    int C, H, W, kh, kw, stride, ph, pw, Ho, Wo;
    float* out;             // launch_col2im: the activation's gradient, X that of the matrix
};
hipError_t launch_im2col(const Im2colArgs& a, hipStream_t stream);
hipError_t launch_col2im(const Im2colArgs& a, hipStream_t stream);
// dst[batch, cols, rows] = src[batch, rows, cols] transposed
hipError_t launch_transpose(const float* src, float* dst, int64_t batch, int64_t rows, int64_t cols, hipStream_t stream);

// Launchers (host).  Each returns the hipError_t of its last launch.
// any-shape kernel: add a tensor to a batch (false: it is full); a launch of a whole batch
bool plan_any(const QuantArgs& q, AnyBatch* b);
// the workgroups of a batch that nothing is added to any more
void finish_any(AnyBatch* b);
hipError_t launch_any(const AnyBatch& b, int pass, hipStream_t stream);
hipError_t launch_gemm(const GemmArgs& g, hipStream_t stream);
// Second reading of the low-bit accumulator: every tile's partial sums to g.partial and their
// maxima to g.tile_max, then Q with acc_bits per tile and the sum over tiles (see gemm.hip).
hipError_t launch_gemm_requant(const GemmArgs& g, int acc_bits, hipStream_t stream);
// The same result without storing a tile sum, for the shapes the matrix-core kernel takes
// (gemm_requant_fast_eligible): pass 1 multiplies and keeps only g.tile_max, pass 2 multiplies
// again and quantizes every tile sum with its tile's maximum as it leaves the matrix core.
// With a split contraction pass 2 writes its parts' totals to g.partial ([splits, RA, RB]),
// which launch_reduce then adds; g.inv_n carries the factor 2^-(a-1) in that case and here.
bool gemm_requant_fast_eligible(const GemmArgs& g, int acc_bits);
hipError_t launch_gemm_requant_fast(const GemmArgs& g, int acc_bits, int pass, hipStream_t stream);
constexpr int kMaxDualBatch = 3;
// the two passes of the two-axis quantization, each for up to kMaxDualBatch tensors in one launch
// ("ride": tensors of the any-shape kernel that share the launch; dense: the maxima of every tensor
// of the launch stand side by side, see QMeta)
hipError_t launch_dual_pass1(const DualArgs* qs, int n, bool dense, const AnyBatch* ride, hipStream_t stream);
hipError_t launch_dual_pass2(const DualArgs* qs, int n, bool dense, const AnyBatch* ride, hipStream_t stream);
int64_t dual_workgroups(const DualArgs& q);
bool dual_pass2_batchable(const DualArgs* qs, int n);
// fills the patch extents of a convolution source; false if the kernels do not take the geometry
bool dual_conv_plan(DualArgs* q);
// zero a[0, na) and b[0, nb) (b may be null) in one launch
hipError_t launch_zero2(uint32_t* a, int64_t na, uint32_t* b, int64_t nb, hipStream_t stream);
// sum the `splits` slices of `partial` ([splits, count]); the totals go to acc_out
// (nullable) and, dequantized, to out (nullable)
// out_bf16 (nullable): the dequantized totals narrowed to bfloat16
hipError_t launch_reduce(const int32_t* partial, int splits, int64_t count, const float* scaleA,
                         const float* scaleB, float inv_n, float* out, uint16_t* out_bf16,
                         int32_t* acc_out, hipStream_t stream, const float* mask_src = nullptr,
                         bool slices16 = false);
bool reduce_takes_slices16(int splits, int64_t count);
// out[e] = mask_src[e] > 0 ? out[e] : +0 (for the matmul paths that do not mask in their epilogue)
hipError_t launch_relu_mask(float* out, const float* mask_src, int64_t count, hipStream_t stream);
// whether the matrix-core kernel applies g.mask_src in its own epilogue
bool gemm_fast_masks(const GemmArgs& g);

// Optional per-kernel timing (off by default).  When enabled through the C ABI,
// every launch is bracketed by two HIP events on its stream.
enum KernelId {
    K_FILL = 0, K_ROW_ABSMAX, K_ROW_QUANT, K_COL_ABSMAX, K_COL_QUANT, K_ANY_ABSMAX,
    K_ANY_QUANT, K_GEMM_ALIGNED, K_GEMM_GENERIC, K_REDUCE, K_GEMM_I4, K_DUAL_ABSMAX, K_DUAL_QUANT,
    K_GEMM_I4_FWD, K_GEMM_I4_BWD_INPUT, K_GEMM_I4_BWD_WEIGHT,
    K_DUAL_ABSMAX_X, K_DUAL_ABSMAX_W, K_DUAL_ABSMAX_G, K_DUAL_QUANT_X, K_DUAL_QUANT_W, K_DUAL_QUANT_G,
    K_DUAL_ABSMAX_BATCH, K_DUAL_QUANT_BATCH, K_REQUANT_TILES, K_REQUANT_SUM, K_IM2COL, K_RELU_MASK,
    K_GEMM_RAGGED, K_GEMM_SMALL, K_COL2IM, K_TRANSPOSE, K_EXPAND,
    K_COUNT
};
bool quantize_fast_eligible(const QuantArgs& q);
hipError_t launch_quantize_fast(const QuantArgs& q, hipStream_t stream);
bool quantize_dual_eligible(const DualArgs& q);
// products that cannot fill the chip with large tiles: up to kMaxSmallBatch of them in one launch,
// never split (gemm_small.hip)
constexpr int kMaxSmallBatch = 3;
bool gemm_small_eligible(const GemmArgs& g, bool alone = true);      // alone: no other product in the launch
hipError_t launch_gemm_small(const GemmArgs* gs, int n, hipStream_t stream);
// large products of packed codes through the 6-bit floating-point matrix instructions, and the scratch they
// need for the codes in that form (gemm_six.hip)
bool gemm_six_shape(int64_t RA, int64_t RB, int64_t D);
bool gemm_six_eligible(const GemmArgs& g);
int64_t gemm_six_bytes(const GemmArgs& g);
hipError_t launch_gemm_six(const GemmArgs& g, void* frags, hipStream_t stream);
bool gemm_fast_eligible(const GemmArgs& g);
// whether gemm_i4_kernel asks of every tile if it can saturate (EPI_CERT8_S32)
bool gemm_fast_tests_tiles(const GemmArgs& g);
// products of codes with a byte each that fill the chip with whole tiles (gemm_bytes.hip)
bool gemm_bytes_eligible(const GemmArgs& g);
hipError_t launch_gemm_bytes(const GemmArgs& g, hipStream_t stream);
// the same of packed codes, in tiles whose clamps are known to act or not to (gemm_packed.hip)
bool gemm_packed_eligible(const GemmArgs& g);
hipError_t launch_gemm_packed(const GemmArgs& g, hipStream_t stream);
hipError_t launch_gemm_fast(const GemmArgs& g, hipStream_t stream);
const char* kernel_name(int id);
bool profiling_enabled();
void profile_begin(int id, hipStream_t stream);
void profile_end(int id, hipStream_t stream);
struct ProfileScope {
    int id; hipStream_t stream; bool on;
    ProfileScope(int i, hipStream_t s) : id(i), stream(s), on(profiling_enabled()) { if (on) profile_begin(id, stream); }
    ~ProfileScope() { if (on) profile_end(id, stream); }
};

// ---- device helpers -------------------------------------------------------

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies
// and a Weyl key schedule.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        // (exclusive or of three: one instruction, which the compiler does not find by itself)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Random 16 bits of element e: half-word (e & 1) of word ((e >> 1) & 3) of `blk`.
__device__ __forceinline__ uint32_t sr_halfword(const uint32_t blk[4], uint32_t e_low3)
{
    const uint32_t w = blk[(e_low3 >> 1) & 3];
    return (w >> (16 * (e_low3 & 1))) & 0xFFFFu;
}

// alpha * 2^(b-1): one correctly rounded division.  A binary64 quotient of two
// binary32 values rounds to binary32 without double-rounding error (53 >= 2*24+2).
// binary32 -> bfloat16 pattern, nearest, ties to even (finite values; a carry out of the
// fraction moves to the next binade or to infinity, which is the correctly rounded result)
__device__ __forceinline__ uint32_t bf16_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ float inverse_step(float amax_clipped, int b)
{
    const double levels = (double)(1 << (b - 1));
    return (float)(levels / (double)amax_clipped);
}

// A block of kernel arguments, all of it asked for at once.  Left to itself the compiler asks for a
// member where it is first used, one after the other, and a trip to an argument takes some hundred
// cycles: a good part of what a launch of a few workgroups takes.  (The statement only wants the
// members in registers; pointers stay pointers, whose address space the compiler knows.)
__device__ __forceinline__ AnyHeader whole_args(const AnyHeader& x)
{
    const AnyHeader h = x;
    static_assert(kMaxAny == 6, "every member is named below");
    asm volatile("" ::"s"(h.first[0]), "s"(h.first[1]), "s"(h.first[2]), "s"(h.first[3]), "s"(h.first[4]), "s"(h.first[5]),
                 "s"(h.n), "s"(h.total));
    return h;
}

__device__ __forceinline__ AnyTensor whole_args(const AnyTensor& x)
{
    const AnyTensor t = x;
    asm volatile("" ::"s"(t.q.T), "s"(t.q.rows), "s"(t.q.cols), "s"(t.q.axis), "s"(t.q.log2n), "s"(t.q.b), "s"(t.q.stochastic),
                 "s"(t.q.clip), "s"(t.q.tensor_id), "s"(t.q.seed_lo), "s"(t.q.seed_hi), "s"(t.q.meta), "s"(t.q.codes),
                 "s"(t.q.scale_out), "s"(t.q.pad), "s"(t.p.count), "s"(t.p.dense), "s"(t.p.wc), "s"(t.p.per.d), "s"(t.p.per.mul),
                 "s"(t.p.per.sh1), "s"(t.p.per.sh2));
    return t;
}

// ---- calibration helpers --------------------------------------------------

// Largest of the wave's values, none of which is negative or NaN (such floats order like their bit
// patterns), in every lane: moves inside rows of sixteen lanes, then lane swaps.  (Six LDS permutes, one
// waiting for the other, take 600 cycles, of which a launch of a small tensor has two such reductions.)
__device__ __forceinline__ uint32_t wave_max_bits(uint32_t m)
{
    auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));       // lane ^ 1
    m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));       // lane ^ 2
    m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, true));      // the other four of eight
    m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xF, 0xF, true));      // the other eight of sixteen
    const auto r16 = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    m = larger(r16[0], r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return larger(r32[0], r32[1]);
}

__device__ __forceinline__ float wave_max(float m) { return __uint_as_float(wave_max_bits(__float_as_uint(m))); }

// The workgroup's maximum into its record.  dense: the word of its own (number `local`); else
// one atomicMax into slot local % 64, and only if it can raise the slot.
__device__ __forceinline__ void record_word(float m, QMeta* meta, int local, int dense)
{
    const uint32_t bits = __float_as_uint(m);
    if (dense) {
        meta->amax[local] = bits;
        return;
    }
    uint32_t* target = &meta->amax[((uint32_t)local % kAmaxSlots) * kAmaxSlotStride];
    if (bits > __hip_atomic_load(target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(target, bits);
}

// The same from every thread's maximum (256 threads).  `smem` holds one float per wave.
__device__ __forceinline__ void record_max(float m, QMeta* meta, float* smem, int local, int dense)
{
    m = wave_max(m);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) smem[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = smem[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmaxf(r, smem[w]);
        record_word(r, meta, local, dense);
    }
}

struct Scaling {
    float inv;      // alpha * 2^(b-1); 0 for an all-zero tensor (every code is then 0)
    float scale;    // value of one code step
};

// Must be reached by whole waves: lane l reads slot l, or the words l, l + 64, ... of `dense`.  In two
// halves, so that a caller has the words on their way before the loads of its tensor.
struct Maxima {
    uint32_t w[4];           // (clamped: four loads in flight, a word twice does no harm)
};

__device__ __forceinline__ Maxima fetch_maxima(const QMeta* meta, int dense)
{
    const int lane = threadIdx.x & 63;
    Maxima x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int at = 64 * k + lane;
        // (the slots: one load, and three of a word that every lane reads, rather than a branch)
        x.w[k] = meta->amax[dense ? (at < dense ? at : dense - 1) : (k ? 0 : lane * kAmaxSlotStride)];
    }
    return x;
}

// From one of the record's largest values in every lane.
__device__ __forceinline__ Scaling scaling_from(uint32_t slot, float clip, int b)
{
    const float amax = __uint_as_float(wave_max_bits(slot));
    const float amax_c = clip * amax;
    Scaling s;
    const bool zero = (amax_c == 0.0f);
    s.inv = zero ? 0.0f : inverse_step(amax_c, b);
    s.scale = zero ? 0.0f : amax_c / (float)(1 << (b - 1));
    return s;
}

__device__ __forceinline__ Scaling scaling_of(const Maxima& x, const QMeta* meta, float clip, int b, int dense)
{
    const int lane = threadIdx.x & 63;
    auto larger = [](uint32_t p, uint32_t q) { return p > q ? p : q; };
    uint32_t slot = larger(larger(x.w[0], x.w[1]), larger(x.w[2], x.w[3]));
    for (int i = 256; i < dense; i += 256) {
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int at = i + 64 * k + lane;
            w[k] = meta->amax[at < dense ? at : dense - 1];
        }
        slot = larger(slot, larger(larger(w[0], w[1]), larger(w[2], w[3])));
    }
    return scaling_from(slot, clip, b);
}

// Where the maxima always stand in slots.  (An ordinary load that stays where it is written: the compiler moves others
// to where the value is needed.)
__device__ __forceinline__ uint32_t fetch_slot(const QMeta* meta)
{
    return __hip_atomic_load(&meta->amax[(threadIdx.x & 63) * kAmaxSlotStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

__device__ __forceinline__ void publish_scale(const QuantArgs& q, const Scaling& s)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        q.meta->scale = s.scale;
        if (q.scale_out) *q.scale_out = s.scale;
    }
}

} // namespace hdqt
