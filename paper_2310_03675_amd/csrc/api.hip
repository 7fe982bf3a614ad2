// C ABI of the HDQT library: argument validation, workspace planning and the
// sequence of launches of each entry point.  See include/hdqt.h for the
// contract of every function.

#include "../../include/hdqt.h"
#include "common.hpp"

#include <limits.h>
#include <mutex>

namespace {

thread_local int g_last_hip_error = 0;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }
inline bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int check_operand(const hdqt_operand_t* op)
{
    if (!op) return HDQT_EINVAL_NULL;
    if (op->b < 2 || op->b > 8) return HDQT_EINVAL_BITS;
    if (op->round != HDQT_ROUND_NEAREST && op->round != HDQT_ROUND_STOCHASTIC)
        return HDQT_EINVAL_ROUND;
    if (!(op->clip > 0.0f) || op->clip > 1.0f) return HDQT_EINVAL_CLIP;
    return HDQT_OK;
}

int check_hadamard(int had_block)
{
    if (!is_pow2(had_block) || had_block > hdqt::kMaxHadamard) return HDQT_EINVAL_HADAMARD;
    return HDQT_OK;
}

// Per dimension: the kernels put up to one workgroup per 64 rows on the y axis of the
// grid, which holds 65535.
constexpr int64_t kMaxDim = (int64_t)65535 * 64 + 1;
constexpr int64_t kMaxElems = (int64_t)1 << 40;      // per tensor

int check_dims2(int64_t rows, int64_t cols)
{
    if (rows <= 0 || cols <= 0 || rows >= kMaxDim || cols >= kMaxDim) return HDQT_EINVAL_DIM;
    if (rows > kMaxElems / cols) return HDQT_EINVAL_DIM;
    return HDQT_OK;
}

// Range checks of the integer matmul: one tile's exact sum and the sum of all
// (clamped) tiles must both fit in 32 bits.
int check_accumulation(int64_t D, int64_t s, int acc_bits, int bA, int bB)
{
    if (s < 1) return HDQT_EINVAL_TILE;
    if (acc_bits < 2 || acc_bits > 32) return HDQT_EINVAL_ACC;
    const int64_t s_eff = s < D ? s : D;
    const int64_t max_prod = ((int64_t)1 << (bA - 1)) * ((int64_t)1 << (bB - 1));
    if (s_eff > (((int64_t)1 << 31) - 1) / max_prod) return HDQT_EINVAL_TILE;
    const int64_t tile_max = s_eff * max_prod;
    const int64_t acc_max = (int64_t)1 << (acc_bits - 1);
    const int64_t per_tile = tile_max < acc_max ? tile_max : acc_max;
    const int64_t n_tiles = (D + s_eff - 1) / s_eff;
    if (n_tiles > (((int64_t)1 << 31) - 1) / per_tile) return HDQT_EINVAL_ACC;
    return HDQT_OK;
}

struct Orientation {
    int64_t RA, RB, D;
    int64_t a_rows, a_cols, b_rows, b_cols;
    int a_axis, b_axis;
};

int orient(int kind, int64_t M, int64_t K, int64_t N, Orientation* o)
{
    switch (kind) {
    case HDQT_GEMM_FWD:          // A = X[M,K] along K, B = W[K,N] along K
        *o = {M, N, K, M, K, K, N, 1, 0};
        return HDQT_OK;
    case HDQT_GEMM_BWD_INPUT:    // A = G[M,N] along N, B = W[K,N] along N
        *o = {M, K, N, M, N, K, N, 1, 1};
        return HDQT_OK;
    case HDQT_GEMM_BWD_WEIGHT:   // A = X[M,K] along M, B = G[M,N] along M
        *o = {K, N, M, M, K, M, N, 0, 0};
        return HDQT_OK;
    default:
        return HDQT_EINVAL_AXIS;
    }
}

int check_gemm(int kind, int64_t M, int64_t K, int64_t N, const hdqt_params_t* p, Orientation* o)
{
    if (!p) return HDQT_EINVAL_NULL;
    int rc = orient(kind, M, K, N, o);
    if (rc) return rc;
    if (M <= 0 || K <= 0 || N <= 0 || M >= kMaxDim || K >= kMaxDim || N >= kMaxDim)
        return HDQT_EINVAL_DIM;
    if ((rc = check_dims2(M, K)) || (rc = check_dims2(K, N)) || (rc = check_dims2(M, N))) return rc;
    if ((rc = check_hadamard(p->had_block))) return rc;
    if ((rc = check_operand(&p->A)) || (rc = check_operand(&p->B))) return rc;
    return check_accumulation(o->D, p->s, p->acc_bits, p->A.b, p->B.b);
}

int log2i(int v)
{
    int k = 0;
    while ((1 << k) < v) ++k;
    return k;
}

int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return HDQT_EHIP;
}

// Parts the contraction is split into when the output has too few tiles to fill the chip.
// The matmul kernels keep two workgroups per CU resident (512 on the chip); every part
// writes an int32 slice of the output that a second pass reads back.  The number of parts is
// the one a simple cost model likes best: the multiplication at the rate the kernels reach
// on a full chip (0.8 POP/s on whole 128 x 128 tiles), slowed down in proportion when
// fewer than 512 workgroups exist, plus one more launch and the slices written and read at
// the 8 TB/s that data of this size gets from the caches.  (A weight gradient with nine
// output tiles takes all the parts it can get; a forward product that already has one
// workgroup per CU takes none; a 2048 x 4608 x 512 product with 64 tiles takes eight.)
int choose_splits(int64_t RA, int64_t RB, int64_t D, int64_t n_tiles)
{
    const int64_t blocks = ((RA + 127) / 128) * ((RB + 127) / 128);
    if (blocks >= 512 || n_tiles < 8) return 1;
    int64_t most = 512 / blocks;
    if (most > n_tiles / 4) most = n_tiles / 4;
    if (most > 1024) most = 1024;
    const double ops = 2.0 * 128.0 * 128.0 * (double)blocks * (double)D;      // what the tiles cost, padding included
    const double slice_us = 8.0 * (double)RA * (double)RB / 8.0e6;            // one slice, written and read
    double best_t = 0.0;
    int best = 1;
    for (int64_t c = 1; c <= most; ++c) {
        const double fill = (double)(blocks * c) / 512.0;
        double t = ops / (0.8e9 * (fill < 1.0 ? fill : 1.0));
        if (c > 1) t += 4.0 + slice_us * (double)c;
        if (c == 1 || t < best_t) { best_t = t; best = (int)c; }
    }
    return best;
}

// Codes that a call keeps to itself lie in lines of whole 16-byte pieces where the contraction is odd, zeros behind them: the
// product then runs over codes(D) of them, in tiles that end with whole pieces or are one tile as before.  (Odd contractions
// are quantized by the any-shape kernel alone, which writes the zeros.  Lines that start on any byte go through a shift per
// fragment in the matmul kernels, and do not go straight to LDS.  Steps, unpadded / padded, us: 64000 x 99 x 99 99.2 / 86.2, 16384 x
// 405 x 243 99.0 / 85.0, 8192 x 1001 x 333 95 / 86, 4097 x 27 x 64 17.4 / 15.5, 131072 x 27 x 64 without input gradient 56.2 / 53.8,
// 1000 x 301 x 77 14.9 / 14.0, 1000000 x 3 x 64 345 / 300, 3 x 2048 x 2048 28.8 / 28.5; but 1 x 4096 x 4096 58.8 / 59.3: a single
// position, whose zeros are fifteen stores to a code, stays alone.  The codes that hdqt_workspace_layout and a saved activation describe lie as ever.)
// A workspace that has room for the codes without the zeros is enough: they then lie without.
struct Lines {
    bool padded;
    int64_t codes(int64_t D) const { return padded && (D & 1) && D > 1 ? (D + 31) / 32 * 32 : D; }
    int64_t tile(int64_t D, int64_t s) const { return s < D ? s : codes(D); }
    int64_t pitch(int64_t D, int b) const { return hdqt_codes_pitch(codes(D), b); }
    int pad(int64_t D, int b) const { return (int)(pitch(D, b) - hdqt_codes_pitch(D, b)); }
};
constexpr Lines kAsTheyAre{false};

constexpr size_t kMetaBytes = (sizeof(hdqt::QMeta) + 255) / 256 * 256;

hdqt::QuantArgs make_quant_args(const float* T, int64_t rows, int64_t cols, int axis, int n_eff,
                                const hdqt_operand_t* op, uint64_t seed, hdqt::QMeta* meta, void* codes,
                                float* scale_out, Lines lines = kAsTheyAre)
{
    hdqt::QuantArgs q{};
    q.T = T; q.rows = rows; q.cols = cols; q.axis = axis;
    q.log2n = log2i(n_eff);
    q.b = op->b; q.stochastic = (op->round == HDQT_ROUND_STOCHASTIC);
    q.clip = op->clip; q.tensor_id = op->tensor_id;
    q.seed_lo = (uint32_t)seed; q.seed_hi = (uint32_t)(seed >> 32);
    q.meta = meta; q.codes = static_cast<uint8_t*>(codes); q.scale_out = scale_out;
    q.pad = lines.pad(axis ? cols : rows, op->b);
    return q;
}

hdqt::DualArgs make_dual_args(const float* T, int64_t rows, int64_t cols, int n1,
                              const hdqt_operand_t* op1, uint64_t seed1, int n0,
                              const hdqt_operand_t* op0, uint64_t seed0, hdqt::QMeta* meta1,
                              hdqt::QMeta* meta0, void* codes1, void* codes0, float* scale1_out,
                              float* scale0_out, int profile_tag, Lines lines1 = kAsTheyAre, Lines lines0 = kAsTheyAre)
{
    hdqt::DualArgs d{};
    d.profile_tag = profile_tag;
    d.T = T; d.rows = rows; d.cols = cols;
    d.log2n_row = log2i(n1); d.log2n_col = log2i(n0);
    d.b_row = op1->b; d.st_row = (op1->round == HDQT_ROUND_STOCHASTIC);
    d.clip_row = op1->clip; d.tid_row = op1->tensor_id;
    d.b_col = op0->b; d.st_col = (op0->round == HDQT_ROUND_STOCHASTIC);
    d.clip_col = op0->clip; d.tid_col = op0->tensor_id;
    d.seed_row_lo = (uint32_t)seed1; d.seed_row_hi = (uint32_t)(seed1 >> 32);
    d.seed_col_lo = (uint32_t)seed0; d.seed_col_hi = (uint32_t)(seed0 >> 32);
    d.meta_row = meta1; d.meta_col = meta0;
    d.codes_row = static_cast<uint8_t*>(codes1); d.codes_col = static_cast<uint8_t*>(codes0);
    d.scale_row_out = scale1_out; d.scale_col_out = scale0_out;
    d.pad_row = lines1.pad(cols, op1->b);
    d.pad_col = lines0.pad(rows, op0->b);
    return d;
}

// rows and columns of the im2col matrix; false if the geometry is not a valid one
bool conv_matrix_shape(const hdqt_conv_t* geo, int64_t* M, int64_t* K)
{
    if (!geo || geo->batch < 1 || geo->channels < 1 || geo->height < 1 || geo->width < 1 || geo->kh < 1 ||
        geo->kw < 1)
        return false;
    const int64_t hw = (int64_t)geo->height * geo->width;
    if (geo->batch > kMaxDim / hw) return false;
    *M = geo->batch * hw;
    *K = (int64_t)geo->channels * geo->kh * geo->kw;
    return *M < kMaxDim && *K < kMaxDim;
}

// Make `d` read its tensor from the activation `geo` describes; false if the two-axis
// kernels do not take that geometry.
bool set_conv_source(hdqt::DualArgs* d, const hdqt_conv_t* geo)
{
    d->cC = geo->channels; d->cH = geo->height; d->cW = geo->width;
    d->ckh = geo->kh; d->ckw = geo->kw;
    return hdqt::dual_conv_plan(d);
}

// Everything one call quantizes, at most kMaxSet (tensor, axis) pairs: tensors along both axes
// (whole) and along one.
struct QuantSet {
    hdqt::DualArgs both[hdqt::kMaxDualBatch];
    hdqt::QuantArgs one[hdqt::kMaxAny];
    int n_both = 0, n_one = 0;
    void add(const hdqt::DualArgs& d) { both[n_both++] = d; }
    void add(const hdqt::QuantArgs& q) { one[n_one++] = q; }
};

hdqt::QuantArgs half_of(const hdqt::DualArgs& d, int axis)
{
    hdqt::QuantArgs q{};
    q.T = d.T; q.rows = d.rows; q.cols = d.cols; q.axis = axis;
    q.log2n = axis ? d.log2n_row : d.log2n_col;
    q.b = axis ? d.b_row : d.b_col; q.stochastic = axis ? d.st_row : d.st_col;
    q.clip = axis ? d.clip_row : d.clip_col; q.tensor_id = axis ? d.tid_row : d.tid_col;
    q.seed_lo = axis ? d.seed_row_lo : d.seed_col_lo; q.seed_hi = axis ? d.seed_row_hi : d.seed_col_hi;
    q.meta = axis ? d.meta_row : d.meta_col; q.codes = axis ? d.codes_row : d.codes_col;
    q.scale_out = axis ? d.scale_row_out : d.scale_col_out;
    q.pad = axis ? d.pad_row : d.pad_col;
    return q;
}

// Where the any-shape kernel is the faster one (us of whole calls, the tuned kernels first):
// Elements, over all pairs, up to which a whole set goes to it: a 512 x 512 x 512 step 27.4 / 20.5,
// 1024 x 1024 x 512 39.1 / 34.2; 2048 x 1152 x 128 (5.5 M) 35.4 / 36.8, 8192 x 1152 x 128 70.1 / 84.4.
constexpr int64_t kAnySet = (int64_t)1 << 22;
// Elements up to which a pair that has a tuned single-axis kernel joins the any-shape pairs of the
// set, which saves the two launches of its own: G of a 131072 x 27 x 64 step (8.4 M) 86.5 / 80.1,
// of 8192 x 1000 x 300 142.8 / 119.4; both operands of 2816 x 2816 x 2816 (7.9 M each) 86.3 / 83.5.
constexpr int64_t kAnyPair = (int64_t)1 << 23;
// The same along axis 0 with orders above 64, where the any-shape kernel pairs waves through LDS
// (the tuned kernel takes 16.5 us at least, 21 with stochastic rounding).  At order 256: X of a
// forward call of 2048 x 1152 x 128 (2.4 M) 35.4 / 29.7, of 65536 x 64 x 64 (4.2 M) 40.3 / 42.4, of
// 16384 x 512 x 64 (8.4 M) 53.4 / 71.0; stochastically, G of a backward call of 65536 x 64 x 64
// 59.5 / 56.5, a 12288 x 512 tensor (6.3 M) on both axes 45.6 / 50.8.
constexpr int64_t kAnyDeep = (int64_t)7 << 19, kAnyDeepStochastic = (int64_t)5 << 20;
// Elements of two such pairs that make up a set, up to which they go there together (stochastic rounding at
// seven tenths): X and G of a weight gradient of 13056 x 256 x 256 (6.7 M) 50.6 / 58.5, of 6144 x 512 x 768
// (3.1 M and, stochastically, 4.7 M) 62.0 / 68.5, of 16384 x 128 x 192 (2.1 and 3.1 M) 52.6 / 46.2.
constexpr int64_t kAnyDeepTwo = (int64_t)5 << 20;
// Workgroups (2048 values) up to which a pair goes there although no other tensor shares the
// launches.  Up to kDenseMost the record need not be cleared: 4096 x 512 along axis 0 11.5 / 10.8, but
// 6144 x 512 13.4 / 14.9 and 4096 x 2048 20.2 / 23.7.  Along axis 0 with stochastic rounding a little
// more: G of a 5312 x 3520 x 512 layer without input gradient (1328) 53.8 / 51.9, 8192 x 512 (2048)
// 15.9 / 17.7.  Half of it with orders above 64 along axis 0 (4096 x 512 16.7 / 18.0), and where a
// tensor with launches of its own has the records cleared anyway.
constexpr int64_t kAnyLone = hdqt::kDenseMost, kAnyLoneStochastic = kAnyLone * 11 / 8;
// Not where much of a strip of the tuned kernel along axis 0, of 64 rows and 128 columns (64, 32 for narrow
// tensors), is wasted: G of 24640 x 320 x 192 without input gradient 41.5 / 39.  Rows that are no whole
// strips go there too since its codes leave in 16-byte stores at any pitch: 5000 x 1000 14.8 / 20.3, 9002 x 512
// 12.5 / 16.8, stochastically 15.8 / 17.7, 20000 x 128 13.8 / 13.8; with a byte per code and stochastic rounding,
// which gains least (9002 x 512 16.9 / 18.2, 2200 x 1024 12.9 / 12.9), they stay.
bool whole_strips(const hdqt::QuantArgs& q)
{
    if (q.axis || q.log2n > 6) return true;
    if (q.rows % 64 != 0 && q.b > 4 && q.stochastic) return false;
    const int64_t across = q.cols > 96 ? 128 : q.cols > 32 ? 64 : 32, padded = (q.cols + across - 1) / across * across;
    return 7 * padded <= 8 * q.cols;
}
// Elements up to which a tensor rounded stochastically on both axes leaves the two-axis kernel's
// launch of a layer's tensors (64 values of two random streams a lane: its few waves end last) for
// the any-shape workgroups beside it: G of 2048 x 4608 x 512 (1 M) 110.7 / 105.1, of 2048 x 1152 x 128
// 35.9 / 31.8; of 16384 x 1152 x 128 (2.1 M) 105.9 / 123.0.
constexpr int64_t kAnyStochastic = (int64_t)1 << 20;

// Quantizes a set: one launch per pass for all tensors that the two-axis and the any-shape kernel
// take (two for pass 2 where the rounding modes do not go together), two launches per tensor that
// its single-axis kernel is the faster one for.  `records`, `record_bytes`: the calibration records of all of them.
int run_quantize_set(const QuantSet& s, void* records, size_t record_bytes, hipStream_t stream)
{
    int64_t work = 0;
    for (int k = 0; k < s.n_both; ++k) work += 2 * s.both[k].rows * s.both[k].cols;
    for (int k = 0; k < s.n_one; ++k) work += s.one[k].rows * s.one[k].cols;
    const bool small = work <= kAnySet;

    hdqt::DualArgs dual[hdqt::kMaxDualBatch];
    hdqt::QuantArgs alone[hdqt::kMaxAny];
    hdqt::AnyBatch any{};
    int n_dual = 0, n_alone = 0;
    auto deep = [](const hdqt::QuantArgs& q) { return !q.axis && q.log2n > 6; };
    bool fits = true;        // (2^31 workgroups: tensors of more than a card's memory)
    auto place = [&](const hdqt::QuantArgs& q) {
        const int64_t most = !deep(q) ? kAnyPair : q.stochastic ? kAnyDeepStochastic : kAnyDeep;
        if (q.rows * q.cols <= most || !hdqt::quantize_fast_eligible(q)) fits = hdqt::plan_any(q, &any) && fits;
        else alone[n_alone++] = q;
    };
    for (int k = 0; k < s.n_both; ++k) {
        const hdqt::DualArgs& d = s.both[k];
        const bool leaves = s.n_both > 1 && d.st_row && d.st_col && d.rows * d.cols <= kAnyStochastic;
        if (d.conv || (!small && !leaves && hdqt::quantize_dual_eligible(d))) {
            dual[n_dual++] = d;
        } else {
            place(half_of(d, 1));
            place(half_of(d, 0));
        }
    }
    for (int k = 0; k < s.n_one; ++k) place(s.one[k]);
    if (!fits) return HDQT_EINVAL_DIM;
    if (any.h.n == 1 && !n_dual && hdqt::quantize_fast_eligible(any.t[0].q) && whole_strips(any.t[0].q)) {
        const hdqt::QuantArgs& q = any.t[0].q;
        int64_t most = q.axis || !q.stochastic ? kAnyLone : kAnyLoneStochastic;
        if (n_alone || (deep(q) && !q.stochastic)) most /= 2;
        if (any.h.total > most) {
            alone[n_alone++] = q;
            any.h.n = any.h.total = 0;
        }
    }
    if (any.h.n == 2 && !n_dual && !n_alone && deep(any.t[0].q) && deep(any.t[1].q)) {
        int64_t sum = 0;
        for (int k = 0; k < 2; ++k) sum += any.t[k].q.rows * any.t[k].q.cols * (any.t[k].q.stochastic ? 7 : 10) / 10;
        if (sum > kAnyDeepTwo && hdqt::quantize_fast_eligible(any.t[0].q) && hdqt::quantize_fast_eligible(any.t[1].q)) {
            for (int k = 0; k < 2; ++k) alone[n_alone++] = any.t[k].q;
            any.h.n = any.h.total = 0;
        }
    }

    const bool ride = n_dual && any.h.total < (1 << 20);
    if (!ride) hdqt::finish_any(&any);
    // maxima side by side, and nothing to clear, if every tensor has few enough workgroups
    bool dense = n_alone == 0;
    for (int k = 0; k < n_dual; ++k) dense = dense && hdqt::dual_workgroups(dual[k]) <= hdqt::kDenseMost;
    for (int k = 0; k < any.h.n; ++k) dense = dense && any.t[k].p.count <= hdqt::kDenseMost;
    for (int k = 0; k < any.h.n; ++k) any.t[k].p.dense = dense ? any.t[k].p.count : 0;
    hipError_t e = hipSuccess;
    if (!dense) e = hdqt::launch_zero2(static_cast<uint32_t*>(records), (int64_t)(record_bytes / 4), nullptr, 0, stream);

    if (n_dual) {
        const hdqt::AnyBatch* riders = ride ? &any : nullptr;
        if (e == hipSuccess) e = hdqt::launch_dual_pass1(dual, n_dual, dense, riders, stream);
        // Pass 2: all in one launch if the rounding modes go together, the last tensor (a layer's
        // G) first: its tiles take longest (two random streams) and start while the chip fills.
        hdqt::DualArgs ord[hdqt::kMaxDualBatch];
        for (int k = 0; k < n_dual; ++k) ord[k] = dual[(k + n_dual - 1) % n_dual];
        if (hdqt::dual_pass2_batchable(ord, n_dual)) {
            if (e == hipSuccess) e = hdqt::launch_dual_pass2(ord, n_dual, dense, riders, stream);
        } else {
            int done = 0;
            while (done < n_dual && e == hipSuccess) {
                int take = n_dual - done;
                while (take > 1 && !hdqt::dual_pass2_batchable(dual + done, take)) --take;
                e = hdqt::launch_dual_pass2(dual + done, take, dense, done ? nullptr : riders, stream);
                done += take;
            }
        }
    }
    if (any.h.n && !ride) {
        if (e == hipSuccess) e = hdqt::launch_any(any, 1, stream);
        if (e == hipSuccess) e = hdqt::launch_any(any, 2, stream);
    }
    for (int k = 0; k < n_alone && e == hipSuccess; ++k) e = hdqt::launch_quantize_fast(alone[k], stream);
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

// Resolve tile length, accumulator range and the split of the contraction.
hdqt::GemmArgs plan_gemm(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                         const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff,
                         int acc_bits, int64_t s, float* out, int32_t* acc_out, int profile_tag = 0,
                         uint16_t* out_bf16 = nullptr, bool keep_tiles = false)
{
    hdqt::GemmArgs g{};
    g.profile_tag = profile_tag;
    g.qA = static_cast<const uint8_t*>(qA); g.qB = static_cast<const uint8_t*>(qB);
    g.pitchA = hdqt_codes_pitch(D, bA); g.pitchB = hdqt_codes_pitch(D, bB);
    g.bA = bA; g.bB = bB; g.RA = RA; g.RB = RB; g.D = D;
    // a contraction of one tile may as well end on a step of the matrix-core kernel: the codes
    // behind a row's end count as zeros (K = 27 in tiles of 32: one step instead of the generic
    // kernel)
    g.s = s < D ? s : (keep_tiles ? D : (D + 31) / 32 * 32);
    g.acc_lo = acc_bits >= 32 ? INT_MIN : -(1 << (acc_bits - 1));
    g.acc_hi = acc_bits >= 32 ? INT_MAX : (1 << (acc_bits - 1)) - 1;
    if (!keep_tiles) {
        // Tiles that cannot saturate need not be kept apart: while m * s products of the
        // largest magnitude, 2^(bA-1) * 2^(bB-1) each, fit the accumulator, the clamp of a
        // group of m tiles changes nothing and the sum over the group is the sum of its
        // tiles' sums.  Groups of 256 or 128 codes are whole stages of the matrix-core kernel
        // (16-bit accumulators with 4-bit inputs, 32-bit ones with any inputs).
        const int64_t max_prod = ((int64_t)1 << (bA - 1)) * ((int64_t)1 << (bB - 1));
        for (int64_t grp = 256; grp >= 128; grp /= 2)
            if (g.s < grp && grp % g.s == 0 && grp <= D && grp * max_prod <= (int64_t)g.acc_hi) {
                g.s = grp;
                break;
            }
    }
    // The parts of a split contraction are chosen from the tiles as they stand here; parts
    // begin on a stage of the matrix-core kernel (128 codes) when the tile length divides
    // one: every 16-byte load of a part then lies inside one 64-byte run of its row
    // (measured on the benchmark layer's weight gradient: 37 -> 40 tiles per part, 35.7 ->
    // 33.1 us), and a tile of 16 codes never starts in the middle of a 32-code step.
    const int64_t plan_tiles = (D + g.s - 1) / g.s;
    g.splits = choose_splits(RA, RB, D, plan_tiles);
    int64_t part_tiles = (plan_tiles + g.splits - 1) / g.splits;
    if (g.splits > 1 && g.s < 128 && 128 % g.s == 0) {
        const int64_t q = 128 / g.s;
        part_tiles = (part_tiles + q - 1) / q * q;
    }
    const int64_t part_codes = part_tiles * g.s;
    if (!keep_tiles) {
        // Tiles that cannot saturate at all: every clamp is the identity and the result is the
        // plain integer product, so the tiles may as well be longer (the kernels clamp at tile
        // ends: 2048 codes are 16 stages of the matrix-core kernel between two clamps) and the
        // accumulator 32 bits wide -- as long as the product itself, times the factor 256 the
        // packed-code kernel carries, stays inside int32, and a part of a split contraction
        // stays a whole number of tiles (fewer, longer parts would leave compute units idle:
        // the weight gradient of the 65536 x 1152 x 128 layer with 8-bit codes and 32-bit
        // accumulators fell from 52 parts to 8).
        const int64_t max_prod = ((int64_t)1 << (bA - 1)) * ((int64_t)1 << (bB - 1));
        const int64_t room = (bA <= 4 && bB <= 4) ? ((int64_t)1 << 22) : ((int64_t)1 << 31);
        if (g.s % 128 == 0 && g.s * max_prod <= (int64_t)g.acc_hi && D * max_prod < room) {
            while (g.s * 2 <= 2048 && g.s * 2 <= D && (g.splits == 1 || part_codes % (g.s * 2) == 0))
                g.s *= 2;
            g.acc_lo = INT_MIN;
            g.acc_hi = INT_MAX;
        }
    }
    g.s_pad = (int)((g.s + 15) / 16 * 16);
    g.n_tiles = (D + g.s - 1) / g.s;
    g.scaleA = scaleA; g.scaleB = scaleB;
    g.inv_n = 1.0f / (float)n_eff;
    g.out = out; g.acc_out = acc_out; g.out_bf16 = out_bf16;
    // An output larger than half the 256 MB memory-side cache cannot stay there until
    // someone reads it; written normally it would sit there dirty and be written back
    // in the middle of the next kernel's reads (measured: the pass over X that follows
    // the input gradient of the 65536 x 1152 layer takes 90 us instead of 53 us).
    // Rows that are no whole 128-byte lines are the exception: a streaming store that ends inside
    // a line does not wait for the neighbour that fills it (input gradients of 31936 x 1150 x 128
    // 140 us, written normally 53, 16000 x 2298 x 48 129 / 42; rows of whole half lines lose it from
    // 512 MB on: 69248 x 1136 x 128 128 / 118, 138496 x 1136 x 128, 600 MB, 214 / 220).
    const int64_t row = RB * (out ? (int64_t)sizeof(float) : (int64_t)sizeof(uint16_t)), out_bytes = RA * row;
    g.stream_out = row % 128 == 0 ? out_bytes >= ((int64_t)128 << 20) : row % 64 == 0 && out_bytes >= ((int64_t)512 << 20);
    g.tiles_per_split = g.splits > 1 ? part_codes / g.s : g.n_tiles;
    g.splits = (int)((g.n_tiles + g.tiles_per_split - 1) / g.tiles_per_split);
    return g;
}

// Bytes of workspace the matmul needs: with a split contraction every part writes
// its totals to a slice of its own ([splits, RA, RB] int32), summed by a second pass.
size_t partial_bytes(int64_t RA, int64_t RB, int64_t D, int64_t s)
{
    const int64_t s_eff = s < D ? s : D;
    int splits = choose_splits(RA, RB, D, (D + s_eff - 1) / s_eff);
    // plan_gemm may merge tiles into groups of 128 or 256 codes; whatever it decides fits
    for (int64_t grp = 128; grp <= 256; grp *= 2)
        if (s_eff < grp && grp % s_eff == 0 && grp <= D) {
            const int alt = choose_splits(RA, RB, D, (D + grp - 1) / grp);
            if (alt > splits) splits = alt;
        }
    return splits > 1 ? (size_t)splits * (size_t)(RA * RB) * sizeof(int32_t) : 0;
}

// Bytes that a call does without if it has to, but is faster with: the codes of a large product expanded for the
// 6-bit matrix instructions.
size_t expanded_bytes(int64_t RA, int64_t RB, int64_t D, int bA, int bB, int acc_bits, int64_t s)
{
    if (!hdqt::gemm_six_shape(RA, RB, D)) return 0;
    const hdqt::GemmArgs g = plan_gemm(nullptr, nullptr, bA, bB, nullptr, nullptr, RA, RB, D, 1, acc_bits, s, nullptr, nullptr);
    return hdqt::gemm_six_eligible(g) ? (size_t)hdqt::gemm_six_bytes(g) : 0;
}

int run_planned_gemm(hdqt::GemmArgs g, void* ws, size_t ws_bytes, hipStream_t stream)
{
    hipError_t e;
    // (asked for also where the small products' kernel then does without: which one multiplies is
    // not the caller's to know)
    if (g.splits > 1 && (!ws || ws_bytes < (size_t)g.splits * (size_t)(g.RA * g.RB) * sizeof(int32_t)))
        return HDQT_EWORKSPACE;
    if (hdqt::gemm_small_eligible(g)) {
        e = hdqt::launch_gemm_small(&g, 1, stream);
        return e == hipSuccess ? HDQT_OK : hip_fail(e);
    }
    if (hdqt::gemm_six_eligible(g) && ws && (int64_t)ws_bytes >= hdqt::gemm_six_bytes(g)) {
        e = hdqt::launch_gemm_six(g, ws, stream);
        return e == hipSuccess ? HDQT_OK : hip_fail(e);
    }
    if (g.splits > 1) {
        g.partial = static_cast<int32_t*>(ws);
        // A part of few tiles has totals of 16 bits: slices of half the bytes (the matrix-core
        // kernel's packed-code instances write them, the many-slices pass reads them).
        const int64_t max_prod = ((int64_t)1 << (g.bA - 1)) * ((int64_t)1 << (g.bB - 1));
        const int64_t tile_sum = g.s * max_prod;
        const int64_t per_tile = tile_sum < (int64_t)g.acc_hi + 1 ? tile_sum : (int64_t)g.acc_hi + 1;
        g.partial16 = (hdqt::gemm_fast_eligible(g) && g.bA <= 4 &&
                       per_tile * g.tiles_per_split <= 32767 &&
                       hdqt::reduce_takes_slices16(g.splits, g.RA * g.RB)) ? 1 : 0;
        e = hdqt::launch_gemm(g, stream);
        if (e != hipSuccess) return hip_fail(e);
        e = hdqt::launch_reduce(g.partial, g.splits, g.RA * g.RB, g.scaleA, g.scaleB, g.inv_n, g.out,
                                g.out_bf16, g.acc_out, stream, g.mask_src, g.partial16 != 0);
        return e == hipSuccess ? HDQT_OK : hip_fail(e);
    }
    e = hdqt::launch_gemm(g, stream);
    if (e != hipSuccess) return hip_fail(e);
    // the rectifier's mask, where the matmul's own epilogue does not apply it
    if (g.mask_src && g.out && !hdqt::gemm_fast_masks(g)) {
        const int64_t count = g.fold ? g.fbatch * g.fC * g.fH * g.fW : g.RA * g.RB;
        e = hdqt::launch_relu_mask(g.out, g.mask_src, count, stream);
    }
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

// Products that do not depend on one another, in this order: the small ones in one launch, the
// others one by one, each with its own slices' workspace.
struct PlannedGemm { hdqt::GemmArgs g; void* ws; size_t ws_bytes; };

int run_planned_gemms(const PlannedGemm* ps, int n, hipStream_t stream)
{
    hdqt::GemmArgs small[hdqt::kMaxSmallBatch];
    int n_small = 0, n_near = 0;
    for (int k = 0; k < n; ++k) n_near += hdqt::gemm_small_eligible(ps[k].g, false);
    const bool alone = n_near < 2;
    for (int k = 0; k < n; ++k)
        if (hdqt::gemm_small_eligible(ps[k].g, alone)) small[n_small++] = ps[k].g;
    if (n_small) {
        const hipError_t e = hdqt::launch_gemm_small(small, n_small, stream);
        if (e != hipSuccess) return hip_fail(e);
    }
    for (int k = 0; k < n; ++k) {
        if (hdqt::gemm_small_eligible(ps[k].g, alone)) continue;
        const int rc = run_planned_gemm(ps[k].g, ps[k].ws, ps[k].ws_bytes, stream);
        if (rc) return rc;
    }
    return HDQT_OK;
}

int run_gemm_codes(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                   const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff, int acc_bits,
                   int64_t s, float* out, uint16_t* out_bf16, int32_t* acc_out, void* workspace,
                   size_t workspace_bytes, void* stream)
{
    if (!qA || !qB || !scaleA || !scaleB || (!out && !out_bf16 && !acc_out)) return HDQT_EINVAL_NULL;
    if (RA <= 0 || RB <= 0 || D <= 0 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim)
        return HDQT_EINVAL_DIM;
    int rc;
    if ((rc = check_dims2(RA, D)) || (rc = check_dims2(RB, D)) || (rc = check_dims2(RA, RB)))
        return rc;
    if (bA < 2 || bA > 8 || bB < 2 || bB > 8) return HDQT_EINVAL_BITS;
    if (!is_pow2(n_eff) || n_eff > hdqt::kMaxHadamard || D % n_eff != 0)
        return HDQT_EINVAL_HADAMARD;
    if ((rc = check_accumulation(D, s, acc_bits, bA, bB))) return rc;
    if (misaligned(qA) || misaligned(qB) || misaligned(out) || misaligned(out_bf16) ||
        misaligned(acc_out) || misaligned(workspace))
        return HDQT_EALIGN;
    return run_planned_gemm(plan_gemm(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, acc_bits, s,
                                      out, acc_out, 0, out_bf16),
                            workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

// What a call needs of a layout's total.
size_t least_bytes(const hdqt_ws_layout_t& L, const hdqt_params_t* prm)
{
    return align_up(L.acc + partial_bytes(L.RA, L.RB, L.D, prm->s) + 256, 256);
}

int run_gemm(int kind, const float* P, const float* Q, float* out, int64_t M, int64_t K, int64_t N,
             const hdqt_params_t* prm, int32_t* acc_out, void* ws, size_t ws_bytes, void* stream_v,
             uint16_t* out_bf16 = nullptr, const float* mask_src = nullptr)
{
    hdqt_ws_layout_t L;
    int rc = hdqt_workspace_layout(kind, M, K, N, prm, &L);
    if (rc) return rc;
    if (!P || !Q || (!out && !out_bf16 && !acc_out)) return HDQT_EINVAL_NULL;
    if (!ws || ws_bytes < least_bytes(L, prm)) return HDQT_EWORKSPACE;
    if (misaligned(P) || misaligned(Q) || misaligned(out) || misaligned(out_bf16) || misaligned(acc_out) ||
        misaligned(ws))
        return HDQT_EALIGN;
    Orientation o;
    orient(kind, M, K, N, &o);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(ws);
    hdqt::QMeta* metaA = reinterpret_cast<hdqt::QMeta*>(base + L.scaleA);
    hdqt::QMeta* metaB = reinterpret_cast<hdqt::QMeta*>(base + L.scaleB);
    void* codesA = base + L.codesA;
    void* codesB = base + L.codesB;
    hdqt::GemmArgs g = plan_gemm(codesA, codesB, prm->A.b, prm->B.b, &metaA->scale, &metaB->scale,
                                 o.RA, o.RB, o.D, L.n_eff, prm->acc_bits, prm->s, out, acc_out, 1 + kind,
                                 out_bf16);
    if (mask_src && (misaligned(mask_src) || !out)) return out ? HDQT_EALIGN : HDQT_EINVAL_NULL;
    g.mask_src = mask_src;
    QuantSet set;
    set.add(make_quant_args(P, o.a_rows, o.a_cols, o.a_axis, L.n_eff, &prm->A, prm->seed, metaA, codesA, nullptr));
    set.add(make_quant_args(Q, o.b_rows, o.b_cols, o.b_axis, L.n_eff, &prm->B, prm->seed, metaB, codesB, nullptr));
    if ((rc = run_quantize_set(set, metaA, 2 * kMetaBytes, stream))) return rc;
    return run_planned_gemm(g, base + L.acc, ws_bytes - L.acc, stream);
}


// Workspace of hdqt_layer_step.  Offsets in bytes; the calibration records are
// contiguous from offset 0, so one launch clears them all.
enum { T_X1, T_X0, T_W0, T_W1, T_G1, T_G0, T_COUNT };
struct StepLayout {
    Lines lines;
    size_t meta[T_COUNT];
    size_t codes[T_COUNT];
    size_t acc[3];           // per matmul: slices of a split contraction
    size_t acc_bytes[3];
    int splits[3];
    int n_eff[3];
    size_t zero_bytes;
    size_t total;
};

int plan_step(int64_t M, int64_t K, int64_t N, const hdqt_params_t* const prm[3], bool with_dx,
              Lines lines, StepLayout* L)
{
    L->lines = lines;
    Orientation o[3];
    for (int k = 0; k < 3; ++k) {
        if (k == HDQT_GEMM_BWD_INPUT && !with_dx) continue;
        const int rc = check_gemm(k, M, K, N, prm[k], &o[k]);
        if (rc) return rc;
    }
    size_t off = 0;
    for (int t = 0; t < T_COUNT; ++t) { L->meta[t] = off; off += kMetaBytes; }
    for (int k = 0; k < 3; ++k) {
        L->acc[k] = off;
        L->acc_bytes[k] = 0;
        L->splits[k] = 1;
        L->n_eff[k] = 1;
        if (k == HDQT_GEMM_BWD_INPUT && !with_dx) continue;
        L->n_eff[k] = hdqt_n_eff(o[k].D, prm[k]->had_block);
        const int64_t D = lines.codes(o[k].D), s = lines.tile(o[k].D, prm[k]->s);
        L->splits[k] = choose_splits(o[k].RA, o[k].RB, D, (D + s - 1) / s);
    }
    L->zero_bytes = off;
    for (int k = 0; k < 3; ++k) {
        L->acc[k] = off;
        if (k == HDQT_GEMM_BWD_INPUT && !with_dx) continue;
        L->acc_bytes[k] = partial_bytes(o[k].RA, o[k].RB, lines.codes(o[k].D), lines.tile(o[k].D, prm[k]->s));
        off = align_up(off + L->acc_bytes[k], 256);
    }
    const hdqt_params_t *fwd = prm[0], *bwi = prm[1], *bww = prm[2];
    const size_t bytes[T_COUNT] = {
        (size_t)(M * lines.pitch(K, fwd->A.b)),                 // X along K
        (size_t)(K * lines.pitch(M, bww->A.b)),                 // X along M
        (size_t)(N * lines.pitch(K, fwd->B.b)),                 // W along K
        with_dx ? (size_t)(K * lines.pitch(N, bwi->B.b)) : 0,   // W along N
        with_dx ? (size_t)(M * lines.pitch(N, bwi->A.b)) : 0,   // G along N
        (size_t)(N * lines.pitch(M, bww->B.b)),                 // G along M
    };
    for (int t = 0; t < T_COUNT; ++t) {
        L->codes[t] = off;
        off = align_up(off + bytes[t], 256);
    }
    L->total = off;
    return HDQT_OK;
}


// ---- forward and backward halves of a layer's step, with X's codes along M handed over
constexpr size_t kSavedHeader = 256;     // the scale (one float) of the saved codes, then padding

struct FwdLayout {
    Lines lines;
    size_t metaX1, metaX0, metaW0;       // contiguous from offset 0
    size_t acc, acc_bytes;
    size_t codesX1, codesW0;
    size_t total;
    int n_fwd, n_bww;
};

int plan_fwd(int64_t M, int64_t K, int64_t N, const hdqt_params_t* fwd, const hdqt_params_t* bww,
             Lines lines, FwdLayout* L)
{
    L->lines = lines;
    Orientation o;
    int rc = check_gemm(HDQT_GEMM_FWD, M, K, N, fwd, &o);
    if (rc) return rc;
    L->n_fwd = hdqt_n_eff(K, fwd->had_block);
    L->n_bww = 1;
    if (bww) {
        Orientation ow;
        if ((rc = check_gemm(HDQT_GEMM_BWD_WEIGHT, M, K, N, bww, &ow))) return rc;
        L->n_bww = hdqt_n_eff(M, bww->had_block);
    }
    size_t off = 0;
    L->metaX1 = off; off += kMetaBytes;
    L->metaX0 = off; off += kMetaBytes;
    L->metaW0 = off; off += kMetaBytes;
    L->acc = off;
    L->acc_bytes = partial_bytes(M, N, lines.codes(K), lines.tile(K, fwd->s));
    off = align_up(off + L->acc_bytes, 256);
    L->codesX1 = off;
    off = align_up(off + (size_t)(M * lines.pitch(K, fwd->A.b)), 256);
    L->codesW0 = off;
    off = align_up(off + (size_t)(N * lines.pitch(K, fwd->B.b)), 256);
    L->total = off;
    return HDQT_OK;
}

struct BwdLayout {
    Lines lines;
    size_t metaG1, metaG0, metaW1;       // contiguous from offset 0
    size_t acc[2], acc_bytes[2];         // input gradient, weight gradient
    size_t codesG1, codesG0, codesW1;
    size_t total;
    int n_bwi, n_bww;
};

int plan_bwd(int64_t M, int64_t K, int64_t N, const hdqt_params_t* bwi, const hdqt_params_t* bww,
             Lines lines, BwdLayout* L)
{
    L->lines = lines;
    Orientation o;
    int rc = check_gemm(HDQT_GEMM_BWD_WEIGHT, M, K, N, bww, &o);
    if (rc) return rc;
    L->n_bww = hdqt_n_eff(M, bww->had_block);
    L->n_bwi = 1;
    if (bwi) {
        if ((rc = check_gemm(HDQT_GEMM_BWD_INPUT, M, K, N, bwi, &o))) return rc;
        L->n_bwi = hdqt_n_eff(N, bwi->had_block);
    }
    size_t off = 0;
    L->metaG1 = off; off += kMetaBytes;
    L->metaG0 = off; off += kMetaBytes;
    L->metaW1 = off; off += kMetaBytes;
    L->acc[0] = off;
    L->acc_bytes[0] = bwi ? partial_bytes(M, K, lines.codes(N), lines.tile(N, bwi->s)) : 0;
    off = align_up(off + L->acc_bytes[0], 256);
    L->acc[1] = off;
    L->acc_bytes[1] = partial_bytes(K, N, M, bww->s);
    off = align_up(off + L->acc_bytes[1], 256);
    L->codesG1 = off;
    off = align_up(off + (bwi ? (size_t)(M * lines.pitch(N, bwi->A.b)) : 0), 256);
    L->codesG0 = off;
    off = align_up(off + (size_t)(N * hdqt_codes_pitch(M, bww->B.b)), 256);
    L->codesW1 = off;
    off = align_up(off + (bwi ? (size_t)(K * lines.pitch(N, bwi->B.b)) : 0), 256);
    L->total = off;
    return HDQT_OK;
}

// ---- second reading of the low-bit accumulator (tiled quantization of the partial sums)

int check_requant(int64_t RA, int64_t RB, int64_t D, int64_t s, int acc_bits, int bA, int bB)
{
    if (s < 1) return HDQT_EINVAL_TILE;
    if (acc_bits < 2 || acc_bits > 24) return HDQT_EINVAL_ACC;
    const int64_t s_eff = s < D ? s : D;
    const int64_t max_prod = ((int64_t)1 << (bA - 1)) * ((int64_t)1 << (bB - 1));
    // a tile sum must be exact in binary32 ...
    if (s_eff > (((int64_t)1 << 24) - 1) / max_prod) return HDQT_EINVAL_TILE;
    // ... and the sum over tiles of code * maximum must stay inside int32
    const int64_t n_tiles = (D + s_eff - 1) / s_eff;
    const int64_t per_tile = ((int64_t)1 << (acc_bits - 1)) * s_eff * max_prod;
    if (n_tiles > (((int64_t)1 << 31) - 1) / per_tile) return HDQT_EINVAL_ACC;
    (void)RA; (void)RB;
    return HDQT_OK;
}

// workspace of the emulation: the maxima and every tile's sums ([n_tiles, RA, RB] int32)
size_t requant_bytes(int64_t RA, int64_t RB, int64_t D, int64_t s)
{
    const int64_t s_eff = s < D ? s : D;
    const int64_t n_tiles = (D + s_eff - 1) / s_eff;
    return align_up((size_t)n_tiles * sizeof(uint32_t), 256) +
           (size_t)n_tiles * (size_t)(RA * RB) * sizeof(int32_t);
}

hdqt::GemmArgs plan_requant(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                            const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff, int64_t s,
                            float* out, int32_t* acc_out)
{
    // (the tiles are what this reading quantizes: they stay as given)
    return plan_gemm(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, 32, s, out, acc_out, 0, nullptr, true);
}

// workspace of the path that will run: the two passes through the matrix-core kernel keep
// only the maxima (and, with a split contraction, one int32 slice per part)
size_t requant_bytes_for(int64_t RA, int64_t RB, int64_t D, int64_t s, int bA, int bB, int acc_bits)
{
    const hdqt::GemmArgs g = plan_requant(nullptr, nullptr, bA, bB, nullptr, nullptr, RA, RB, D, 1, s, nullptr, nullptr);
    if (!hdqt::gemm_requant_fast_eligible(g, acc_bits)) return requant_bytes(RA, RB, D, s);
    return align_up((size_t)g.n_tiles * sizeof(uint32_t), 256) +
           (g.splits > 1 ? (size_t)g.splits * (size_t)(RA * RB) * sizeof(int32_t) : 0);
}

int run_requant(const void* qA, const void* qB, int bA, int bB, const float* scaleA, const float* scaleB,
                int64_t RA, int64_t RB, int64_t D, int n_eff, int acc_bits, int64_t s, float* out,
                int32_t* acc_out, void* ws, size_t ws_bytes, hipStream_t stream)
{
    if (!ws || ws_bytes < requant_bytes_for(RA, RB, D, s, bA, bB, acc_bits)) return HDQT_EWORKSPACE;
    hdqt::GemmArgs g = plan_requant(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, s, out, acc_out);
    char* base = static_cast<char*>(ws);
    g.tile_max = reinterpret_cast<uint32_t*>(base);
    g.partial = reinterpret_cast<int32_t*>(base + align_up((size_t)g.n_tiles * sizeof(uint32_t), 256));
    hipError_t e = hdqt::launch_zero2(g.tile_max, g.n_tiles, nullptr, 0, stream);
    if (e != hipSuccess) return hip_fail(e);
    if (hdqt::gemm_requant_fast_eligible(g, acc_bits)) {
        // value = acc * 2^-(a-1) * (scaleA * scaleB) / n_eff: both trailing factors are powers of two
        g.inv_n = g.inv_n * ldexpf(1.0f, -(acc_bits - 1));
        e = hdqt::launch_gemm_requant_fast(g, acc_bits, 1, stream);
        if (e != hipSuccess) return hip_fail(e);
        e = hdqt::launch_gemm_requant_fast(g, acc_bits, 2, stream);
        if (e != hipSuccess) return hip_fail(e);
        if (g.splits > 1)
            e = hdqt::launch_reduce(g.partial, g.splits, g.RA * g.RB, g.scaleA, g.scaleB, g.inv_n, g.out, nullptr,
                                    g.acc_out, stream);
        return e == hipSuccess ? HDQT_OK : hip_fail(e);
    }
    e = hdqt::launch_gemm_requant(g, acc_bits, stream);
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

} // namespace

extern "C" {

int hdqt_n_eff(int64_t D, int had_block)
{
    if (D <= 0 || had_block < 1) return 1;
    int m = 1;
    while (m * 2 <= had_block && D % (m * 2) == 0) m *= 2;
    return m;
}

int64_t hdqt_codes_pitch(int64_t D, int b) { return b <= 4 ? (D + 1) / 2 : D; }

size_t hdqt_quantize_workspace_size(void) { return kMetaBytes; }

size_t hdqt_workspace_least(int gemm_kind, int64_t M, int64_t K, int64_t N, const hdqt_params_t* params)
{
    hdqt_ws_layout_t L;
    return hdqt_workspace_layout(gemm_kind, M, K, N, params, &L) == HDQT_OK ? least_bytes(L, params) : 0;
}

int hdqt_workspace_layout(int gemm_kind, int64_t M, int64_t K, int64_t N,
                          const hdqt_params_t* params, hdqt_ws_layout_t* layout)
{
    Orientation o;
    const int rc = check_gemm(gemm_kind, M, K, N, params, &o);
    if (rc) return rc;
    hdqt_ws_layout_t L;
    L.RA = o.RA; L.RB = o.RB; L.D = o.D;
    L.n_eff = hdqt_n_eff(o.D, params->had_block);
    size_t off = 0;
    // two calibration records, adjacent; `scale` is the first member of each
    L.scaleA = off;
    off += kMetaBytes;
    L.scaleB = off;
    off += kMetaBytes;
    L.codesA = off;
    off = align_up(off + (size_t)(o.RA * hdqt_codes_pitch(o.D, params->A.b)), 256);
    L.codesB = off;
    off = align_up(off + (size_t)(o.RB * hdqt_codes_pitch(o.D, params->B.b)), 256);
    L.acc = off;
    const size_t slices = partial_bytes(o.RA, o.RB, o.D, params->s);
    const size_t expanded = expanded_bytes(o.RA, o.RB, o.D, params->A.b, params->B.b, params->acc_bits, params->s);
    off = align_up(off + (slices > expanded ? slices : expanded) + 256, 256);
    L.total = off;
    if (layout) *layout = L;
    return HDQT_OK;
}

size_t hdqt_workspace_size(int gemm_kind, int64_t M, int64_t K, int64_t N,
                           const hdqt_params_t* params)
{
    hdqt_ws_layout_t L;
    return hdqt_workspace_layout(gemm_kind, M, K, N, params, &L) == HDQT_OK ? L.total : 0;
}

int hdqt_quantize(const float* T, int64_t rows, int64_t cols, int axis, int had_block,
                  const hdqt_operand_t* op, uint64_t seed, void* codes_out, float* scale_out,
                  void* workspace, size_t workspace_bytes, void* stream)
{
    if (!T || !codes_out || !scale_out || !op) return HDQT_EINVAL_NULL;
    int rc = check_dims2(rows, cols);
    if (rc) return rc;
    if (axis != 0 && axis != 1) return HDQT_EINVAL_AXIS;
    if ((rc = check_hadamard(had_block))) return rc;
    if ((rc = check_operand(op))) return rc;
    if (!workspace || workspace_bytes < hdqt_quantize_workspace_size()) return HDQT_EWORKSPACE;
    if (misaligned(T) || misaligned(codes_out) || misaligned(workspace)) return HDQT_EALIGN;
    if ((reinterpret_cast<uintptr_t>(scale_out) & 3u) != 0) return HDQT_EALIGN;
    const int64_t D = axis ? cols : rows;
    QuantSet set;
    set.add(make_quant_args(T, rows, cols, axis, hdqt_n_eff(D, had_block), op, seed,
                            static_cast<hdqt::QMeta*>(workspace), codes_out, scale_out));
    return run_quantize_set(set, workspace, kMetaBytes, static_cast<hipStream_t>(stream));
}

size_t hdqt_quantize_dual_workspace_size(void) { return 2 * kMetaBytes; }

int hdqt_quantize_dual(const float* T, int64_t rows, int64_t cols, int had_block,
                       const hdqt_operand_t* op_axis1, const hdqt_operand_t* op_axis0, uint64_t seed,
                       void* codes_axis1, float* scale_axis1, void* codes_axis0, float* scale_axis0,
                       void* workspace, size_t workspace_bytes, void* stream_v)
{
    if (!T || !op_axis1 || !op_axis0 || !codes_axis1 || !codes_axis0 || !scale_axis1 || !scale_axis0)
        return HDQT_EINVAL_NULL;
    int rc = check_dims2(rows, cols);
    if (rc) return rc;
    if ((rc = check_hadamard(had_block))) return rc;
    if ((rc = check_operand(op_axis1)) || (rc = check_operand(op_axis0))) return rc;
    if (!workspace || workspace_bytes < hdqt_quantize_dual_workspace_size()) return HDQT_EWORKSPACE;
    if (misaligned(T) || misaligned(codes_axis1) || misaligned(codes_axis0) || misaligned(workspace))
        return HDQT_EALIGN;
    if (((reinterpret_cast<uintptr_t>(scale_axis1) | reinterpret_cast<uintptr_t>(scale_axis0)) & 3u) != 0)
        return HDQT_EALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    hdqt::QMeta* meta1 = reinterpret_cast<hdqt::QMeta*>(base);
    hdqt::QMeta* meta0 = reinterpret_cast<hdqt::QMeta*>(base + kMetaBytes);
    QuantSet set;
    set.add(make_dual_args(T, rows, cols, hdqt_n_eff(cols, had_block), op_axis1, seed, hdqt_n_eff(rows, had_block),
                           op_axis0, seed, meta1, meta0, codes_axis1, codes_axis0, scale_axis1, scale_axis0, 0));
    return run_quantize_set(set, base, 2 * kMetaBytes, stream);
}

int hdqt_quantize_dual_im2col(const float* act, const hdqt_conv_t* geo, int had_block,
                              const hdqt_operand_t* op_axis1, const hdqt_operand_t* op_axis0,
                              uint64_t seed, void* codes_axis1, float* scale_axis1, void* codes_axis0,
                              float* scale_axis0, void* workspace, size_t workspace_bytes, void* stream_v)
{
    if (!act || !geo || !op_axis1 || !op_axis0 || !codes_axis1 || !codes_axis0 || !scale_axis1 ||
        !scale_axis0)
        return HDQT_EINVAL_NULL;
    int64_t rows, cols;
    if (!conv_matrix_shape(geo, &rows, &cols)) return HDQT_EINVAL_DIM;
    int rc;
    if ((rc = check_dims2(rows, cols)) || (rc = check_hadamard(had_block)) ||
        (rc = check_operand(op_axis1)) || (rc = check_operand(op_axis0)))
        return rc;
    if (!workspace || workspace_bytes < 2 * kMetaBytes) return HDQT_EWORKSPACE;
    if (misaligned(act) || misaligned(codes_axis1) || misaligned(codes_axis0) || misaligned(workspace))
        return HDQT_EALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    hdqt::QMeta* meta1 = reinterpret_cast<hdqt::QMeta*>(base);
    hdqt::QMeta* meta0 = reinterpret_cast<hdqt::QMeta*>(base + kMetaBytes);
    hdqt::DualArgs d = make_dual_args(act, rows, cols, hdqt_n_eff(cols, had_block), op_axis1, seed,
                                      hdqt_n_eff(rows, had_block), op_axis0, seed, meta1, meta0,
                                      codes_axis1, codes_axis0, scale_axis1, scale_axis0, 0);
    if (!set_conv_source(&d, geo) || !hdqt::quantize_dual_eligible(d)) return HDQT_EINVAL_GEOMETRY;
    QuantSet set;
    set.add(d);
    return run_quantize_set(set, base, 2 * kMetaBytes, stream);
}

} // extern "C"

namespace {
// the geometry shared by hdqt_im2col and hdqt_col2im; X and the activation are both of a size that
// the kernels index
int plan_unfold(int64_t batch, int channels, int height, int width, int kh, int kw, int stride, int pad_h, int pad_w,
                hdqt::Im2colArgs* a)
{
    if (batch < 1 || channels < 1 || height < 1 || width < 1 || kh < 1 || kw < 1 || stride < 1 || pad_h < 0 ||
        pad_w < 0 || kh > 255 || kw > 255 || height + 2 * pad_h < kh || width + 2 * pad_w < kw)
        return HDQT_EINVAL_DIM;
    const int Ho = (height + 2 * pad_h - kh) / stride + 1, Wo = (width + 2 * pad_w - kw) / stride + 1;
    const int64_t per_image = (int64_t)Ho * Wo, K = (int64_t)channels * kh * kw;
    if (batch > kMaxDim / per_image) return HDQT_EINVAL_DIM;
    const int64_t M = batch * per_image;
    const int rc = check_dims2(M, K);
    if (rc) return rc;
    if ((int64_t)channels * height * width >= ((int64_t)1 << 31) || (M + 3) / 4 >= ((int64_t)1 << 31))
        return HDQT_EINVAL_DIM;
    // (a stride longer than the padded image is as good as one of its length, and the kernels may add to it)
    const int longest = height + 2 * pad_h > width + 2 * pad_w ? height + 2 * pad_h : width + 2 * pad_w;
    if (stride > longest) stride = longest;
    *a = hdqt::Im2colArgs{nullptr, nullptr, M, channels, height, width, kh, kw, stride, pad_h, pad_w, Ho, Wo, nullptr};
    return HDQT_OK;
}
} // namespace

extern "C" {

int hdqt_im2col(const float* act, int64_t batch, int channels, int height, int width, int kh, int kw,
                int stride, int pad_h, int pad_w, float* X, void* stream)
{
    if (!act || !X) return HDQT_EINVAL_NULL;
    hdqt::Im2colArgs a;
    const int rc = plan_unfold(batch, channels, height, width, kh, kw, stride, pad_h, pad_w, &a);
    if (rc) return rc;
    if (misaligned(act) || misaligned(X)) return HDQT_EALIGN;
    a.act = act;
    a.X = X;
    const hipError_t e = hdqt::launch_im2col(a, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

int hdqt_col2im(const float* dX, int64_t batch, int channels, int height, int width, int kh, int kw,
                int stride, int pad_h, int pad_w, float* dAct, void* stream)
{
    if (!dX || !dAct) return HDQT_EINVAL_NULL;
    hdqt::Im2colArgs a;
    const int rc = plan_unfold(batch, channels, height, width, kh, kw, stride, pad_h, pad_w, &a);
    if (rc) return rc;
    // (the activation of a strided layer has many times the pixels that the matrix has rows)
    const int64_t hw = (int64_t)height * width;
    if (batch > kMaxElems / channels / hw) return HDQT_EINVAL_DIM;
    if (misaligned(dX) || misaligned(dAct)) return HDQT_EALIGN;
    a.X = const_cast<float*>(dX);
    a.M = batch * hw;
    a.out = dAct;
    const hipError_t e = hdqt::launch_col2im(a, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

int hdqt_transpose(const float* src, int64_t batch, int64_t rows, int64_t cols, float* dst, void* stream)
{
    if (!src || !dst) return HDQT_EINVAL_NULL;
    if (batch < 1 || batch > 65535) return HDQT_EINVAL_DIM;
    const int rc = check_dims2(rows, cols);
    if (rc) return rc;
    if (misaligned(src) || misaligned(dst)) return HDQT_EALIGN;
    const hipError_t e = hdqt::launch_transpose(src, dst, batch, rows, cols, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? HDQT_OK : hip_fail(e);
}

size_t hdqt_gemm_codes_workspace_size(int64_t RA, int64_t RB, int64_t D, int64_t s)
{
    if (RA <= 0 || RB <= 0 || D <= 0 || s < 1 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim) return 0;
    // (whatever the widths: for packed codes and an accumulator that the expanded form is for)
    const size_t slices = partial_bytes(RA, RB, D, s), clamped = expanded_bytes(RA, RB, D, 4, 4, 8, s),
                 plain = expanded_bytes(RA, RB, D, 4, 4, 32, s), expanded = clamped > plain ? clamped : plain;
    return slices > expanded ? slices : expanded;
}

size_t hdqt_gemm_codes_workspace_size_for(int64_t RA, int64_t RB, int64_t D, int64_t s, int bA, int bB, int acc_bits,
                                          int bf16)
{
    if (RA <= 0 || RB <= 0 || D <= 0 || s < 1 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim) return 0;
    if (bA < 2 || bA > 8 || bB < 2 || bB > 8 || check_accumulation(D, s, acc_bits, bA, bB)) return 0;
    const size_t slices = partial_bytes(RA, RB, D, s), expanded = bf16 ? 0 : expanded_bytes(RA, RB, D, bA, bB, acc_bits, s);
    return slices > expanded ? slices : expanded;
}

int hdqt_gemm_codes(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                    const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff,
                    int acc_bits, int64_t s, float* out, int32_t* acc_out, void* workspace,
                    size_t workspace_bytes, void* stream)
{
    return run_gemm_codes(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, acc_bits, s, out, nullptr,
                          acc_out, workspace, workspace_bytes, stream);
}

int hdqt_gemm_codes_bf16(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                         const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff,
                         int acc_bits, int64_t s, uint16_t* out, int32_t* acc_out, void* workspace,
                         size_t workspace_bytes, void* stream)
{
    return run_gemm_codes(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, acc_bits, s, nullptr, out,
                          acc_out, workspace, workspace_bytes, stream);
}

size_t hdqt_gemm_codes_requant_workspace_size(int64_t RA, int64_t RB, int64_t D, int64_t s)
{
    if (RA <= 0 || RB <= 0 || D <= 0 || s < 1 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim) return 0;
    return requant_bytes(RA, RB, D, s);
}

size_t hdqt_gemm_codes_requant_workspace_size_for(int64_t RA, int64_t RB, int64_t D, int64_t s, int bA,
                                                  int bB, int acc_bits)
{
    if (RA <= 0 || RB <= 0 || D <= 0 || s < 1 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim) return 0;
    if (bA < 2 || bA > 8 || bB < 2 || bB > 8) return 0;
    if (check_requant(RA, RB, D, s, acc_bits, bA, bB)) return 0;
    return requant_bytes_for(RA, RB, D, s, bA, bB, acc_bits);
}

int hdqt_gemm_codes_requant(const void* qA, const void* qB, int bA, int bB, const float* scaleA,
                            const float* scaleB, int64_t RA, int64_t RB, int64_t D, int n_eff,
                            int acc_bits, int64_t s, float* out, int32_t* acc_out, void* workspace,
                            size_t workspace_bytes, void* stream)
{
    if (!qA || !qB || !scaleA || !scaleB || (!out && !acc_out)) return HDQT_EINVAL_NULL;
    if (RA <= 0 || RB <= 0 || D <= 0 || RA >= kMaxDim || RB >= kMaxDim || D >= kMaxDim)
        return HDQT_EINVAL_DIM;
    int rc;
    if ((rc = check_dims2(RA, D)) || (rc = check_dims2(RB, D)) || (rc = check_dims2(RA, RB))) return rc;
    if (bA < 2 || bA > 8 || bB < 2 || bB > 8) return HDQT_EINVAL_BITS;
    if (!is_pow2(n_eff) || n_eff > hdqt::kMaxHadamard || D % n_eff != 0) return HDQT_EINVAL_HADAMARD;
    if ((rc = check_requant(RA, RB, D, s, acc_bits, bA, bB))) return rc;
    if (misaligned(qA) || misaligned(qB) || misaligned(out) || misaligned(acc_out) || misaligned(workspace))
        return HDQT_EALIGN;
    return run_requant(qA, qB, bA, bB, scaleA, scaleB, RA, RB, D, n_eff, acc_bits, s, out, acc_out,
                       workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

size_t hdqt_gemm_requant_workspace_size(int gemm_kind, int64_t M, int64_t K, int64_t N,
                                        const hdqt_params_t* params)
{
    hdqt_ws_layout_t L;
    if (hdqt_workspace_layout(gemm_kind, M, K, N, params, &L) != HDQT_OK) return 0;
    if (check_requant(L.RA, L.RB, L.D, params->s, params->acc_bits, params->A.b, params->B.b)) return 0;
    return L.acc + requant_bytes_for(L.RA, L.RB, L.D, params->s, params->A.b, params->B.b, params->acc_bits);
}

int hdqt_gemm_requant(int gemm_kind, const float* P, const float* Q, float* out, int64_t M, int64_t K,
                      int64_t N, const hdqt_params_t* params, int32_t* acc_out, void* workspace,
                      size_t workspace_bytes, void* stream_v)
{
    hdqt_ws_layout_t L;
    int rc = hdqt_workspace_layout(gemm_kind, M, K, N, params, &L);
    if (rc) return rc;
    if ((rc = check_requant(L.RA, L.RB, L.D, params->s, params->acc_bits, params->A.b, params->B.b)))
        return rc;
    if (!P || !Q || (!out && !acc_out)) return HDQT_EINVAL_NULL;
    if (!workspace || workspace_bytes < L.acc + requant_bytes_for(L.RA, L.RB, L.D, params->s, params->A.b,
                                                                  params->B.b, params->acc_bits))
        return HDQT_EWORKSPACE;
    if (misaligned(P) || misaligned(Q) || misaligned(out) || misaligned(acc_out) || misaligned(workspace))
        return HDQT_EALIGN;
    Orientation o;
    orient(gemm_kind, M, K, N, &o);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    hdqt::QMeta* metaA = reinterpret_cast<hdqt::QMeta*>(base + L.scaleA);
    hdqt::QMeta* metaB = reinterpret_cast<hdqt::QMeta*>(base + L.scaleB);
    QuantSet set;
    set.add(make_quant_args(P, o.a_rows, o.a_cols, o.a_axis, L.n_eff, &params->A, params->seed, metaA, base + L.codesA, nullptr));
    set.add(make_quant_args(Q, o.b_rows, o.b_cols, o.b_axis, L.n_eff, &params->B, params->seed, metaB, base + L.codesB, nullptr));
    if ((rc = run_quantize_set(set, metaA, 2 * kMetaBytes, stream))) return rc;
    return run_requant(base + L.codesA, base + L.codesB, params->A.b, params->B.b, &metaA->scale,
                       &metaB->scale, L.RA, L.RB, L.D, L.n_eff, params->acc_bits, params->s, out, acc_out,
                       base + L.acc, workspace_bytes - L.acc, stream);
}

size_t hdqt_layer_step_workspace_size(int64_t M, int64_t K, int64_t N, const hdqt_params_t* fwd,
                                      const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight)
{
    const hdqt_params_t* prm[3] = {fwd, bwd_input, bwd_weight};
    StepLayout L;
    return plan_step(M, K, N, prm, bwd_input != nullptr, {true}, &L) == HDQT_OK ? L.total : 0;
}

} // extern "C"

namespace {

// X is the [M, K] matrix, or, with `geo`, the activation whose im2col matrix it is.
int run_layer_step(const float* X, const hdqt_conv_t* geo, const float* W, const float* G, float* Z,
                   float* dX, float* dW, int64_t M, int64_t K, int64_t N, const hdqt_params_t* fwd,
                   const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight, void* workspace,
                   size_t workspace_bytes, void* stream_v)
{
    if (!X || !W || !G || !Z || !dW || !fwd || !bwd_weight) return HDQT_EINVAL_NULL;
    const bool with_dx = dX != nullptr;
    if (with_dx && !bwd_input) return HDQT_EINVAL_NULL;
    const hdqt_params_t* prm[3] = {fwd, bwd_input, bwd_weight};
    StepLayout L;
    int rc = plan_step(M, K, N, prm, with_dx, {true}, &L);
    if (!rc && workspace_bytes < L.total) rc = plan_step(M, K, N, prm, with_dx, kAsTheyAre, &L);
    if (rc) return rc;
    if (!workspace || workspace_bytes < L.total) return HDQT_EWORKSPACE;
    if (misaligned(X) || misaligned(W) || misaligned(G) || misaligned(Z) || misaligned(dX) ||
        misaligned(dW) || misaligned(workspace))
        return HDQT_EALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    auto meta = [&](int t) { return reinterpret_cast<hdqt::QMeta*>(base + L.meta[t]); };
    auto codes = [&](int t) { return static_cast<void*>(base + L.codes[t]); };
    auto acc = [&](int k) { return static_cast<void*>(base + L.acc[k]); };

    const int nF = L.n_eff[HDQT_GEMM_FWD], nI = L.n_eff[HDQT_GEMM_BWD_INPUT],
              nW = L.n_eff[HDQT_GEMM_BWD_WEIGHT];
    // X along K (forward) and along M (weight gradient); W along N (input gradient) and
    // along K (forward); G along N (input gradient) and along M (weight gradient)
    if (geo && !with_dx) return HDQT_EINVAL_GEOMETRY;       // (hdqt_conv_step asks for dXcol)
    QuantSet set;
    set.add(make_dual_args(X, M, K, nF, &fwd->A, fwd->seed, nW, &bwd_weight->A, bwd_weight->seed, meta(T_X1),
                           meta(T_X0), codes(T_X1), codes(T_X0), nullptr, nullptr, 1, L.lines, L.lines));
    if (with_dx) {
        set.add(make_dual_args(W, K, N, nI, &bwd_input->B, bwd_input->seed, nF, &fwd->B, fwd->seed, meta(T_W1),
                               meta(T_W0), codes(T_W1), codes(T_W0), nullptr, nullptr, 2, L.lines, L.lines));
        set.add(make_dual_args(G, M, N, nI, &bwd_input->A, bwd_input->seed, nW, &bwd_weight->B, bwd_weight->seed,
                               meta(T_G1), meta(T_G0), codes(T_G1), codes(T_G0), nullptr, nullptr, 3, L.lines, L.lines));
        // an activation source is read by the two-axis kernels only, and its layer's other tensors
        // are of a kind they take (nothing is launched before this is known)
        if (geo) {
            if (!set_conv_source(&set.both[0], geo)) return HDQT_EINVAL_GEOMETRY;
            for (int k = 0; k < 3; ++k)
                if (!hdqt::quantize_dual_eligible(set.both[k])) return HDQT_EINVAL_GEOMETRY;
        }
    } else {
        set.add(make_quant_args(W, K, N, 0, nF, &fwd->B, fwd->seed, meta(T_W0), codes(T_W0), nullptr, L.lines));
        set.add(make_quant_args(G, M, N, 0, nW, &bwd_weight->B, bwd_weight->seed, meta(T_G0), codes(T_G0), nullptr, L.lines));
    }
    if ((rc = run_quantize_set(set, base, L.zero_bytes, stream))) return rc;
    hdqt::GemmArgs g_fwd = plan_gemm(codes(T_X1), codes(T_W0), fwd->A.b, fwd->B.b, &meta(T_X1)->scale,
                                     &meta(T_W0)->scale, M, N, L.lines.codes(K), nF, fwd->acc_bits, L.lines.tile(K, fwd->s), Z, nullptr,
                                     1 + HDQT_GEMM_FWD);
    // Nobody can read Z before the two backward products of this call have run, and those move
    // several times the memory-side cache: from 16 MB on, Z is written with streaming stores
    // too, if its rows are whole half lines.  (Measured on the 65536 x 1152 x 128 layer, Z = 33.5 MB: left in the cache as dirty
    // lines it is written back under the kernels that follow -- forward 30.1 -> 28.1 us, and
    // the next call's pass over X 66.6 -> 60.8 us.)  The forward call on its own keeps the
    // 128 MB mark: its caller reads Z next.
    if (M * N * (int64_t)sizeof(float) >= ((int64_t)16 << 20) && N % 16 == 0) g_fwd.stream_out = 1;
    // The weight gradient goes before the input gradient: its operand, X's codes along M, is the
    // older data in the memory-side cache; the input gradient's large output comes last.
    PlannedGemm ps[3];
    int n = 0;
    ps[n++] = {g_fwd, acc(HDQT_GEMM_FWD), L.acc_bytes[HDQT_GEMM_FWD]};
    ps[n++] = {plan_gemm(codes(T_X0), codes(T_G0), bwd_weight->A.b, bwd_weight->B.b, &meta(T_X0)->scale,
                         &meta(T_G0)->scale, K, N, L.lines.codes(M), nW, bwd_weight->acc_bits, L.lines.tile(M, bwd_weight->s), dW, nullptr,
                         1 + HDQT_GEMM_BWD_WEIGHT),
               acc(HDQT_GEMM_BWD_WEIGHT), L.acc_bytes[HDQT_GEMM_BWD_WEIGHT]};
    if (with_dx)
        ps[n++] = {plan_gemm(codes(T_G1), codes(T_W1), bwd_input->A.b, bwd_input->B.b, &meta(T_G1)->scale,
                             &meta(T_W1)->scale, M, K, L.lines.codes(N), nI, bwd_input->acc_bits, L.lines.tile(N, bwd_input->s), dX, nullptr,
                             1 + HDQT_GEMM_BWD_INPUT),
                   acc(HDQT_GEMM_BWD_INPUT), L.acc_bytes[HDQT_GEMM_BWD_INPUT]};
    // dX in rows of whole half lines streams from the 128 MB mark on here, where a product on its own
    // does not: written normally it goes back to memory under the passes that follow (normal / streamed:
    // 65536 x 1136 x 128 422 / 398 us, 37816 x 1168 x 96 305 / 295, 32768 x 2320 x 256 475 / 447).
    if (with_dx && K % 16 == 0 && M * K * (int64_t)sizeof(float) >= ((int64_t)128 << 20)) ps[2].g.stream_out = 1;
    return run_planned_gemms(ps, n, stream);
}

} // namespace

extern "C" {

int hdqt_layer_step(const float* X, const float* W, const float* G, float* Z, float* dX, float* dW,
                    int64_t M, int64_t K, int64_t N, const hdqt_params_t* fwd,
                    const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight,
                    void* workspace, size_t workspace_bytes, void* stream)
{
    return run_layer_step(X, nullptr, W, G, Z, dX, dW, M, K, N, fwd, bwd_input, bwd_weight, workspace,
                          workspace_bytes, stream);
}

size_t hdqt_conv_step_workspace_size(const hdqt_conv_t* geo, int64_t N, const hdqt_params_t* fwd,
                                     const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight)
{
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K) || !bwd_input) return 0;
    hdqt::DualArgs d{};
    d.rows = M; d.cols = K;
    if (!set_conv_source(&d, geo)) return 0;
    return hdqt_layer_step_workspace_size(M, K, N, fwd, bwd_input, bwd_weight);
}

int hdqt_conv_step(const float* act, const hdqt_conv_t* geo, const float* W, const float* G, float* Z,
                   float* dXcol, float* dW, int64_t N, const hdqt_params_t* fwd,
                   const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight, void* workspace,
                   size_t workspace_bytes, void* stream)
{
    if (!geo || !dXcol || !bwd_input) return HDQT_EINVAL_NULL;
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K)) return HDQT_EINVAL_DIM;
    return run_layer_step(act, geo, W, G, Z, dXcol, dW, M, K, N, fwd, bwd_input, bwd_weight, workspace,
                          workspace_bytes, stream);
}

size_t hdqt_layer_saved_size(int64_t M, int64_t K, const hdqt_params_t* bwd_weight)
{
    if (!bwd_weight || check_dims2(M, K) || check_operand(&bwd_weight->A)) return 0;
    return kSavedHeader + align_up((size_t)(K * hdqt_codes_pitch(M, bwd_weight->A.b)), 256);
}

size_t hdqt_layer_fwd_workspace_size(int64_t M, int64_t K, int64_t N, const hdqt_params_t* fwd,
                                     const hdqt_params_t* bwd_weight)
{
    FwdLayout L;
    return plan_fwd(M, K, N, fwd, bwd_weight, {true}, &L) == HDQT_OK ? L.total : 0;
}

} // extern "C"

namespace {

// X is the [M, K] matrix, or, with `geo`, the activation whose im2col matrix it is.
int run_layer_fwd(const float* X, const hdqt_conv_t* geo, const float* W, float* Z, int64_t M, int64_t K,
                  int64_t N, const hdqt_params_t* fwd, const hdqt_params_t* bwd_weight, void* saved,
                  size_t saved_bytes, void* workspace, size_t workspace_bytes, void* stream_v)
{
    if (!X || !W || !Z || !fwd) return HDQT_EINVAL_NULL;
    if (bwd_weight && !saved) return HDQT_EINVAL_NULL;
    FwdLayout L;
    int rc = plan_fwd(M, K, N, fwd, bwd_weight, {true}, &L);
    if (!rc && workspace_bytes < L.total) rc = plan_fwd(M, K, N, fwd, bwd_weight, kAsTheyAre, &L);
    if (rc) return rc;
    if (!workspace || workspace_bytes < L.total) return HDQT_EWORKSPACE;
    if (bwd_weight && saved_bytes < hdqt_layer_saved_size(M, K, bwd_weight)) return HDQT_EWORKSPACE;
    if (misaligned(X) || misaligned(W) || misaligned(Z) || misaligned(saved) || misaligned(workspace))
        return HDQT_EALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    char* sv = static_cast<char*>(saved);
    auto meta = [&](size_t off) { return reinterpret_cast<hdqt::QMeta*>(base + off); };
    QuantSet set;
    if (bwd_weight)
        set.add(make_dual_args(X, M, K, L.n_fwd, &fwd->A, fwd->seed, L.n_bww, &bwd_weight->A, bwd_weight->seed,
                               meta(L.metaX1), meta(L.metaX0), base + L.codesX1, sv + kSavedHeader, nullptr,
                               reinterpret_cast<float*>(sv), 1, L.lines));
    else
        set.add(make_quant_args(X, M, K, 1, L.n_fwd, &fwd->A, fwd->seed, meta(L.metaX1), base + L.codesX1, nullptr, L.lines));
    if (geo) {
        // an activation source is read by the two-axis kernels only: both code sets are made,
        // and nothing is launched before the geometry is known to be taken
        if (!bwd_weight) return HDQT_EINVAL_NULL;
        if (!set_conv_source(&set.both[0], geo) || !hdqt::quantize_dual_eligible(set.both[0]))
            return HDQT_EINVAL_GEOMETRY;
    }
    set.add(make_quant_args(W, K, N, 0, L.n_fwd, &fwd->B, fwd->seed, meta(L.metaW0), base + L.codesW0, nullptr, L.lines));
    if ((rc = run_quantize_set(set, base, 3 * kMetaBytes, stream))) return rc;
    return run_planned_gemm(plan_gemm(base + L.codesX1, base + L.codesW0, fwd->A.b, fwd->B.b,
                                      &meta(L.metaX1)->scale, &meta(L.metaW0)->scale, M, N, L.lines.codes(K), L.n_fwd,
                                      fwd->acc_bits, L.lines.tile(K, fwd->s), Z, nullptr, 1 + HDQT_GEMM_FWD),
                            base + L.acc, L.acc_bytes, stream);
}

} // namespace

extern "C" {

int hdqt_layer_fwd(const float* X, const float* W, float* Z, int64_t M, int64_t K, int64_t N,
                   const hdqt_params_t* fwd, const hdqt_params_t* bwd_weight, void* saved,
                   size_t saved_bytes, void* workspace, size_t workspace_bytes, void* stream)
{
    return run_layer_fwd(X, nullptr, W, Z, M, K, N, fwd, bwd_weight, saved, saved_bytes, workspace,
                         workspace_bytes, stream);
}

int hdqt_conv_fwd(const float* act, const hdqt_conv_t* geo, const float* W, float* Z, int64_t N,
                  const hdqt_params_t* fwd, const hdqt_params_t* bwd_weight, void* saved,
                  size_t saved_bytes, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!geo) return HDQT_EINVAL_NULL;
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K)) return HDQT_EINVAL_DIM;
    return run_layer_fwd(act, geo, W, Z, M, K, N, fwd, bwd_weight, saved, saved_bytes, workspace,
                         workspace_bytes, stream);
}

size_t hdqt_layer_bwd_workspace_size(int64_t M, int64_t K, int64_t N, const hdqt_params_t* bwd_input,
                                     const hdqt_params_t* bwd_weight)
{
    BwdLayout L;
    return plan_bwd(M, K, N, bwd_input, bwd_weight, {true}, &L) == HDQT_OK ? L.total : 0;
}

} // extern "C"

namespace {

// dX is the gradient of the [M, K] matrix, or, with `geo`, of the activation it was unfolded from.
int run_layer_bwd(const float* G, const float* W, const void* saved, const hdqt_conv_t* geo, float* dX,
                  float* dW, int64_t M, int64_t K, int64_t N, const hdqt_params_t* bwd_input,
                  const hdqt_params_t* bwd_weight, void* workspace, size_t workspace_bytes,
                  void* stream_v, const float* mask_src = nullptr)
{
    if (!G || !saved || !dW || !bwd_weight) return HDQT_EINVAL_NULL;
    const bool with_dx = dX != nullptr;
    if (mask_src && !with_dx) return HDQT_EINVAL_NULL;
    if (misaligned(mask_src)) return HDQT_EALIGN;
    if (with_dx && (!bwd_input || !W)) return HDQT_EINVAL_NULL;
    BwdLayout L;
    // (A folded gradient is planned over the caller's contraction: which layers are refused is part of their results, and
    // padding an odd one to whole 32s would take it.)
    int rc = plan_bwd(M, K, N, with_dx ? bwd_input : nullptr, bwd_weight, {geo == nullptr}, &L);
    if (!rc && workspace_bytes < L.total) rc = plan_bwd(M, K, N, with_dx ? bwd_input : nullptr, bwd_weight, kAsTheyAre, &L);
    if (rc) return rc;
    if (!workspace || workspace_bytes < L.total) return HDQT_EWORKSPACE;
    if (misaligned(G) || misaligned(W) || misaligned(saved) || misaligned(dX) || misaligned(dW) ||
        misaligned(workspace))
        return HDQT_EALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    const char* sv = static_cast<const char*>(saved);
    auto meta = [&](size_t off) { return reinterpret_cast<hdqt::QMeta*>(base + off); };
    hdqt::GemmArgs g_dx{};
    if (with_dx) {
        g_dx = plan_gemm(base + L.codesG1, base + L.codesW1, bwd_input->A.b, bwd_input->B.b,
                         &meta(L.metaG1)->scale, &meta(L.metaW1)->scale, M, K, L.lines.codes(N), L.n_bwi,
                         bwd_input->acc_bits, L.lines.tile(N, bwd_input->s), dX, nullptr, 1 + HDQT_GEMM_BWD_INPUT);
        // (nothing is launched before the geometry is known to be taken)
        if (geo && !hdqt::gemm_fold_plan(&g_dx, geo->batch, geo->channels, geo->height, geo->width, geo->kh,
                                         geo->kw))
            return HDQT_EINVAL_GEOMETRY;
        g_dx.mask_src = mask_src;
        g_dx.padded = L.lines.codes(N) != N;
    } else if (geo) {
        return HDQT_EINVAL_NULL;
    }
    QuantSet set;
    if (with_dx) {
        set.add(make_dual_args(G, M, N, L.n_bwi, &bwd_input->A, bwd_input->seed, L.n_bww, &bwd_weight->B,
                               bwd_weight->seed, meta(L.metaG1), meta(L.metaG0), base + L.codesG1,
                               base + L.codesG0, nullptr, nullptr, 3, L.lines));
        set.add(make_quant_args(W, K, N, 1, L.n_bwi, &bwd_input->B, bwd_input->seed, meta(L.metaW1),
                                base + L.codesW1, nullptr, L.lines));
    } else {
        set.add(make_quant_args(G, M, N, 0, L.n_bww, &bwd_weight->B, bwd_weight->seed, meta(L.metaG0),
                                base + L.codesG0, nullptr));
    }
    if ((rc = run_quantize_set(set, base, 3 * kMetaBytes, stream))) return rc;
    PlannedGemm ps[2];
    int n = 0;
    ps[n++] = {plan_gemm(sv + kSavedHeader, base + L.codesG0, bwd_weight->A.b, bwd_weight->B.b,
                         reinterpret_cast<const float*>(sv), &meta(L.metaG0)->scale, K, N, M, L.n_bww,
                         bwd_weight->acc_bits, bwd_weight->s, dW, nullptr, 1 + HDQT_GEMM_BWD_WEIGHT),
               base + L.acc[1], L.acc_bytes[1]};
    if (with_dx) ps[n++] = {g_dx, base + L.acc[0], L.acc_bytes[0]};
    return run_planned_gemms(ps, n, stream);
}

} // namespace

extern "C" {

int hdqt_layer_bwd(const float* G, const float* W, const void* saved, float* dX, float* dW, int64_t M,
                   int64_t K, int64_t N, const hdqt_params_t* bwd_input,
                   const hdqt_params_t* bwd_weight, void* workspace, size_t workspace_bytes,
                   void* stream)
{
    return run_layer_bwd(G, W, saved, nullptr, dX, dW, M, K, N, bwd_input, bwd_weight, workspace,
                         workspace_bytes, stream);
}

int hdqt_conv_bwd(const float* G, const float* W, const void* saved, const hdqt_conv_t* geo, float* dAct,
                  float* dW, int64_t N, const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight,
                  void* workspace, size_t workspace_bytes, void* stream)
{
    if (!geo || !dAct) return HDQT_EINVAL_NULL;
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K)) return HDQT_EINVAL_DIM;
    return run_layer_bwd(G, W, saved, geo, dAct, dW, M, K, N, bwd_input, bwd_weight, workspace,
                         workspace_bytes, stream);
}

int hdqt_layer_bwd_masked(const float* G, const float* W, const void* saved, const float* x_mask,
                          float* dX, float* dW, int64_t M, int64_t K, int64_t N,
                          const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight, void* workspace,
                          size_t workspace_bytes, void* stream)
{
    if (!x_mask || !dX) return HDQT_EINVAL_NULL;
    return run_layer_bwd(G, W, saved, nullptr, dX, dW, M, K, N, bwd_input, bwd_weight, workspace,
                         workspace_bytes, stream, x_mask);
}

int hdqt_conv_bwd_masked(const float* G, const float* W, const void* saved, const hdqt_conv_t* geo,
                         const float* act_mask, float* dAct, float* dW, int64_t N,
                         const hdqt_params_t* bwd_input, const hdqt_params_t* bwd_weight, void* workspace,
                         size_t workspace_bytes, void* stream)
{
    if (!geo || !dAct || !act_mask) return HDQT_EINVAL_NULL;
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K)) return HDQT_EINVAL_DIM;
    return run_layer_bwd(G, W, saved, geo, dAct, dW, M, K, N, bwd_input, bwd_weight, workspace,
                         workspace_bytes, stream, act_mask);
}

int hdqt_gemm_bwd_input_masked(const float* G, const float* W, const float* x_mask, float* dX, int64_t M,
                               int64_t K, int64_t N, const hdqt_params_t* params, int32_t* acc_out,
                               void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x_mask || !dX) return HDQT_EINVAL_NULL;
    return run_gemm(HDQT_GEMM_BWD_INPUT, G, W, dX, M, K, N, params, acc_out, workspace, workspace_bytes,
                    stream, nullptr, x_mask);
}

int hdqt_gemm_codes_fold(const void* qG, const void* qW, int bG, int bW, const float* scaleG,
                         const float* scaleW, const hdqt_conv_t* geo, int64_t N, int n_eff, int acc_bits,
                         int64_t s, float* dAct, void* stream)
{
    if (!qG || !qW || !scaleG || !scaleW || !geo || !dAct) return HDQT_EINVAL_NULL;
    int64_t M, K;
    if (!conv_matrix_shape(geo, &M, &K) || N <= 0 || N >= kMaxDim) return HDQT_EINVAL_DIM;
    int rc;
    if ((rc = check_dims2(M, N)) || (rc = check_dims2(K, N)) || (rc = check_dims2(M, K))) return rc;
    if (bG < 2 || bG > 8 || bW < 2 || bW > 8) return HDQT_EINVAL_BITS;
    if (!is_pow2(n_eff) || n_eff > hdqt::kMaxHadamard || N % n_eff != 0) return HDQT_EINVAL_HADAMARD;
    if ((rc = check_accumulation(N, s, acc_bits, bG, bW))) return rc;
    if (misaligned(qG) || misaligned(qW) || misaligned(dAct)) return HDQT_EALIGN;
    hdqt::GemmArgs g = plan_gemm(qG, qW, bG, bW, scaleG, scaleW, M, K, N, n_eff, acc_bits, s, dAct, nullptr,
                                 1 + HDQT_GEMM_BWD_INPUT);
    if (!hdqt::gemm_fold_plan(&g, geo->batch, geo->channels, geo->height, geo->width, geo->kh, geo->kw))
        return HDQT_EINVAL_GEOMETRY;
    return run_planned_gemm(g, nullptr, 0, static_cast<hipStream_t>(stream));
}


int hdqt_gemm_fwd(const float* X, const float* W, float* Z, int64_t M, int64_t K, int64_t N,
                  const hdqt_params_t* params, int32_t* acc_out, void* workspace,
                  size_t workspace_bytes, void* stream)
{
    return run_gemm(HDQT_GEMM_FWD, X, W, Z, M, K, N, params, acc_out, workspace, workspace_bytes,
                    stream);
}

int hdqt_gemm_bwd_input(const float* G, const float* W, float* dX, int64_t M, int64_t K, int64_t N,
                        const hdqt_params_t* params, int32_t* acc_out, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    return run_gemm(HDQT_GEMM_BWD_INPUT, G, W, dX, M, K, N, params, acc_out, workspace,
                    workspace_bytes, stream);
}

int hdqt_gemm_bwd_input_bf16(const float* G, const float* W, uint16_t* dX, int64_t M, int64_t K,
                             int64_t N, const hdqt_params_t* params, int32_t* acc_out, void* workspace,
                             size_t workspace_bytes, void* stream)
{
    return run_gemm(HDQT_GEMM_BWD_INPUT, G, W, nullptr, M, K, N, params, acc_out, workspace,
                    workspace_bytes, stream, dX);
}

int hdqt_gemm_bwd_weight(const float* X, const float* G, float* dW, int64_t M, int64_t K,
                         int64_t N, const hdqt_params_t* params, int32_t* acc_out, void* workspace,
                         size_t workspace_bytes, void* stream)
{
    return run_gemm(HDQT_GEMM_BWD_WEIGHT, X, G, dW, M, K, N, params, acc_out, workspace,
                    workspace_bytes, stream);
}

// ---- hdqt_gemm_fwd without a workspace argument and without any allocation ----
//
// The calibration records and the codes of both operands, which hdqt_gemm_fwd keeps in the
// caller's workspace, live in a file-scope device array instead.  Every GPU the library runs
// on holds its own copy of the array at its own address: the address is asked for once per
// device (hipGetSymbolAddress with that device current) and only that pointer is ever handed
// to a kernel -- in host code the array's name is a stand-in, not a device address.
} // extern "C"

namespace {
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {nullptr};
std::mutex g_scratch_mu;

// device pointer of `scratch` on the current device; nullptr (and the HIP error recorded) on failure
void* static_scratch()
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        g_last_hip_error = (int)(e != hipSuccess ? e : hipErrorInvalidDevice);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            g_last_hip_error = (int)(e != hipSuccess ? e : hipErrorInvalidSymbol);
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
} // namespace

extern "C" {

size_t hdqt_gemm_fwd_static_max_bytes(void) { return kStaticScratchBytes; }

int hdqt_gemm_fwd_static(const float* X, const float* W, float* Z, int64_t M, int64_t K, int64_t N,
                         const hdqt_params_t* params, int32_t* acc_out, void* stream)
{
    hdqt_ws_layout_t L;
    const int rc = hdqt_workspace_layout(HDQT_GEMM_FWD, M, K, N, params, &L);
    if (rc) return rc;
    if (least_bytes(L, params) > kStaticScratchBytes) return HDQT_ESCRATCH;
    void* ptr = static_scratch();
    if (!ptr) return HDQT_EHIP;
    // run_gemm writes every word of the calibration records that it reads, or clears them with a
    // kernel first, and every code byte that the matmul reads: what an earlier call left behind in
    // the array is never seen.
    return run_gemm(HDQT_GEMM_FWD, X, W, Z, M, K, N, params, acc_out, ptr, kStaticScratchBytes, stream);
}

const char* hdqt_strerror(int code)
{
    switch (code) {
    case HDQT_OK: return "success";
    case HDQT_EINVAL_NULL: return "a required pointer is NULL";
    case HDQT_EINVAL_DIM: return "a dimension is not positive or is too large";
    case HDQT_EINVAL_HADAMARD: return "Hadamard block order must be a power of two in [1, 256]";
    case HDQT_EINVAL_BITS: return "code width b must be in [2, 8]";
    case HDQT_EINVAL_ACC: return "accumulator width must be in [2, 32] and the total must fit int32";
    case HDQT_EINVAL_TILE: return "tile length s must be >= 1 and a tile's sum must fit int32";
    case HDQT_EINVAL_CLIP: return "clip factor must be in (0, 1]";
    case HDQT_EINVAL_ROUND: return "unknown rounding mode";
    case HDQT_EINVAL_AXIS: return "axis must be 0 or 1 / unknown matmul kind";
    case HDQT_EWORKSPACE: return "workspace is NULL or too small";
    case HDQT_EALIGN: return "a pointer is not 16-byte aligned";
    case HDQT_EHIP: return "a HIP call failed (see hdqt_last_hip_error)";
    case HDQT_ESCRATCH: return "the shape needs more scratch than the library's fixed device array holds";
    case HDQT_EINVAL_GEOMETRY: return "convolution geometry or layer shape not taken by the activation-source kernels";
    default: return "unknown error code";
    }
}

int hdqt_last_hip_error(void) { return g_last_hip_error; }

} // extern "C"
