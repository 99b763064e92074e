// Matrix-core forward kernel of the local B-spline layer for short tables (up to 47 rows).
//
// y = sum over (input, table row) of basis(x) * table is a dense product whose left operand holds at most kMaxK + 1 values per
// input.  Sparse matrix instructions (two values of every four positions along the sum, v_smfmac_f32_32x32x32_bf16) skip half
// of the zeros: table row r of an input goes to group r mod G, position r / G of the G groups of four (mx_groups), so that the
// rows of a window fall into different groups; w_b, the last position of the last group, meets at most one row there.  Each group
// then has one row in slot 0 (positions 0..2) or slot 1 (position 3), and every index pair is (position, 3).
// The precision is that of fp32: every float is split into three bf16 parts (8 bits each, 24 in all), and six of the nine products of
// the parts are summed in fp32; the two left out that weigh most reach 2^-24.2 of the product together, and 2^-27.5 in the mean, beside
// the 2^-24 of a sum's rounding.  The parts have the exponent range of a float, and a common power of
// two keeps the lowest ones off its end.  Values that do not split (infinite, NaN, or too large for that) are found where they are
// split; the sums that read them, and those that come out infinite or NaN (two factors that split may have a product of parts
// that does not fit), are done in plain fp32 at the end.
//
// Error against fp64 (2-norm): 512 -> 512, G = 20 4.9e-7 (the LDS-staged kernel 9.0e-7); 256 -> 256, G = 28 1.3e-7 (6.4e-7);
// 75 -> 130, G = 12, k = 2 0.96e-7 (direct kernel 1.14e-7); 128 -> 128, G = 10 1.07e-7 (1.38e-7).
//
// What bounds it, 512 -> 512, G = 20, B = 16384, 602 us (the staged kernel, bound by its LDS reads: 914): the matrix instructions
// alone take 360 (by variants that leave a part out), evaluating the pairs 66 more, fetching the right operands from L2 63, reading
// the left ones from LDS 31; by counters the matrix cores are busy 45 % of the clocks, the rest of the VALU 27 %, LDS 26 %, and waves
// wait for memory or LDS 40 % of theirs and to issue 34 %.
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_matrix.hpp"
#include <cfloat>
#include <type_traits>

namespace KAN_NS {

using ::kan::MatrixTable;
using ::kan::kMxInputs;
using ::kan::kMxTile;
using ::kan::kMxSplits;

namespace {

typedef __bf16 Bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 Bf16 __attribute__((ext_vector_type(16)));
typedef __bf16 Bf2 __attribute__((ext_vector_type(2)));
typedef float F2 __attribute__((ext_vector_type(2)));
typedef float F16 __attribute__((ext_vector_type(16)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));
typedef unsigned U8 __attribute__((ext_vector_type(8)));

// Both operands are split times 2^24, which makes the lowest bit of the smallest float a bf16 number that is not subnormal; what
// is larger than kMxLargest then leaves the parts' range.
constexpr float kMxScale = 0x1p+24f, kMxLargest = 0x1p+96f;

// two floats rounded to bf16, low and high half
__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    F2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, Bf2));
}

// the three parts of two floats, each the pair's low and high half; the differences are exact
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&p)[kMxSplits])
{
#pragma unroll
    for (int s = 0; s < kMxSplits; ++s) {
        p[s] = bf16_pair(a, b);
        a -= __builtin_bit_cast(float, p[s] << 16);
        b -= __builtin_bit_cast(float, p[s] & 0xffff0000u);
    }
}

}  // namespace

// ---- the table: scale folded in, and split ----------------------------------------
// One workgroup per (step of four inputs, tile of 32 outputs), lane l of wave t <-> lane l of instruction t: column l % 32 and four
// of the instruction's eight groups, whose left operands are spread over both halves of the wave: with h = l / 32 groups
// 2 h, 2 h + 1, 4 + 2 h, 5 + 2 h, four table rows each.  Writes cf as fold_scale_kernel does and the operands
// of the forward kernel; rows past the table and columns past the layer are zero.  The first tile begins at output j0; cf: null
// if no folded table is wanted.
template <int NG>
__global__ __launch_bounds__(32 * NG) void matrix_table_kernel(const float *__restrict__ coef, const float *__restrict__ w_s,
                                                               const float *__restrict__ w_b, float *__restrict__ cf,
                                                               U4 *__restrict__ frag, int *__restrict__ odd, int n_in, int rows,
                                                               int n_out, int j0)
{
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6, step = blockIdx.x, tile = blockIdx.y;
    const int j = j0 + tile * kMxTile + (lane & 31), half = lane >> 5;
    float v[16];
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int grp = 8 * t + 4 * (e / 2) + 2 * half + e % 2, i = step * kMxInputs + grp / NG, g = grp % NG;
        const bool ok = i < n_in && j < n_out;
        const float s = ok ? w_s[(int64_t)i * n_out + j] : 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = g + NG * q;
            const bool base = row == 4 * NG - 1;
            float c = 0.0f;
            if (ok && (base || row < rows)) {
                if (!base) c = coef[((int64_t)i * rows + row) * n_out + j] * s;
                else if (w_b) c = w_b[(int64_t)i * n_out + j];
                if (cf) cf[((int64_t)i * (rows + 1) + (base ? rows : row)) * n_out + j] = c;
            }
            const bool fits = fabsf(c) < kMxLargest;
            bad |= !fits;
            v[4 * e + q] = fits ? c * kMxScale : 0.0f;
        }
    }
    unsigned p[8][kMxSplits];
#pragma unroll
    for (int e = 0; e < 8; ++e) split_pair(v[2 * e], v[2 * e + 1], p[e]);
    U4 *at = frag + ((((int64_t)tile * gridDim.x + step) * (NG / 2) + t) * kMxSplits) * 128 + lane;
#pragma unroll
    for (int s = 0; s < kMxSplits; ++s) {
        at[s * 128] = U4{p[0][s], p[1][s], p[2][s], p[3][s]};
        at[s * 128 + 64] = U4{p[4][s], p[5][s], p[6][s], p[7][s]};
    }
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0) odd[(int64_t)tile * gridDim.x + step] = any;
}

// ---- forward ----------------------------------------------------------------------
// A workgroup of WM x WN waves owns 32 * MT * WM samples and 32 * WN outputs; a wave MT tiles of 32 samples and one tile of
// outputs.  Per step of SI inputs all lanes evaluate the step's pairs and write the left operands (three parts, indices)
// to LDS for the step after; the right operands come from L2 straight into the registers that the instructions read, an
// instruction's worth ahead (prefetching them into L2 two steps ahead: 580 -> 653 us).  SI inputs a step: eight where a
// workgroup owns 64 samples, so that every lane has a pair (four, half of them idle: 75 -> 130, B = 6001 43 -> 37 us); 128
// samples have no room for eight in LDS.  FOLD: the products of the leading parts are folded into a second sum every other step
// (up to 64 inputs every step: 16 -> 256, G = 9, k = 5 error 0.86e-7, without 1.06e-7, the direct kernel's 0.92e-7), as exact as
// the two-level kernels that this one stands in for; the form with 128 samples, which has no registers for it, only takes layers
// whose other kernel has one level (forward_matrix_plan).
template <int NG, int SI>
struct MxArea {                              // left operands of one step of SI inputs in LDS, per sample
    // words of a sample's row of one part: 16-byte reads of eight samples fall into different banks
    static constexpr int kRow = SI * NG % 16 == 0 ? SI * NG + 4 : SI * NG;
    static constexpr int kIdx = SI * NG / 8;                                // words of a sample's indices
    template <int S> static constexpr int words() { return S * (kMxSplits * kRow + kIdx); }
};

template <int NG>
using IndexBits = std::conditional_t<(NG > 8), uint64_t, unsigned>;

// A pair's left operands: out[part][group], and the indices of its groups, four bits each.
template <int NG>
__device__ __forceinline__ void pair_operands(int row0, const float (&w)[kMaxK], float base, unsigned (&out)[kMxSplits][NG],
                                              IndexBits<NG> &index)
{
    const int q0 = row0 / NG, c0 = row0 - q0 * NG;
    unsigned part[(kMaxK + 1) / 2][kMxSplits], pb[kMxSplits];
#pragma unroll
    for (int s = 0; s < kMaxK; s += 2) split_pair(w[s], s + 1 < kMaxK ? w[s + 1] : 0.0f, part[s / 2]);
    split_pair(0.0f, base, pb);
    index = (IndexBits<NG>)0xCCCCCCCCCCCCCCCCull;
#pragma unroll
    for (int p = 0; p < kMxSplits; ++p)
#pragma unroll
        for (int g = 0; g < NG; ++g) out[p][g] = 0u;
#pragma unroll
    for (int s = 0; s < kMaxK; ++s) {
        const bool wrap = c0 + s >= NG;
        const int q = q0 + (wrap ? 1 : 0), g = c0 + s - (wrap ? NG : 0);
        const bool last = q == 3;
        index |= (IndexBits<NG>)(last ? 0u : (unsigned)q) << (4 * g);
#pragma unroll
        for (int p = 0; p < kMxSplits; ++p) {
            const unsigned v = part[s / 2][p], low = s % 2 ? v >> 16 : v & 0xffffu, high = s % 2 ? v & 0xffff0000u : v << 16;
            out[p][s] = last ? high : low;
        }
    }
    // rows 0 .. of the window stand at groups 0 ..: turn them to group c0
#pragma unroll
    for (int bit = 1; bit < NG; bit *= 2) {
        const bool on = (c0 & bit) != 0;
#pragma unroll
        for (int p = 0; p < kMxSplits; ++p) {
            unsigned t[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) t[g] = out[p][(g + NG - bit % NG) % NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) out[p][g] = on ? t[g] : out[p][g];
        }
    }
#pragma unroll
    for (int p = 0; p < kMxSplits; ++p) out[p][NG - 1] |= pb[p] & 0xffff0000u;      // (the zero in the low half may carry a sign)
}

template <int NG, int SI, int MT, int WM, int WN, bool FOLD, bool AHEAD>
__global__ __launch_bounds__(64 * WM * WN, WM * WN >= 16 ? 4 : 2) void forward_matrix_kernel(SplineGeom g, const float *__restrict__ x,
                                                                      const float *__restrict__ coef, const float *__restrict__ w_s,
                                                                      const float *__restrict__ w_b, const U4 *__restrict__ frag,
                                                                      const int *__restrict__ odd, float *__restrict__ y,
                                                                      int64_t B, int n_tiles, int j0, int fold_mask)
{
    constexpr int NT = 64 * WM * WN, S = 32 * MT * WM, EP = S * SI / NT, KS = SI * NG / 8;
    static_assert(S * SI % NT == 0 && SI % kMxInputs == 0, "");
    typedef MxArea<NG, SI> A;
    constexpr int kArea = A::template words<S>();
    extern __shared__ unsigned lds[];
    int *special = reinterpret_cast<int *>(lds + 2 * kArea);           // per sample: a value that does not split
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave / WN;
    const int tile = blockIdx.y * WN + wave % WN, tc = tile < n_tiles ? tile : n_tiles - 1;
    const int64_t b0 = (int64_t)blockIdx.x * S;
    const int n_steps = (g.n_in + SI - 1) / SI, n_parts = (g.n_in + kMxInputs - 1) / kMxInputs;      // of the table

    for (int s = tid; s < S; s += NT) special[s] = 0;

    // two sums: the products of the leading parts, and the others, whose roundings are 2^-8 of the former's
    F16 acc[MT], low[MT], tot[FOLD ? MT : 1];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[m][r] = low[m][r] = 0.0f; if (FOLD) tot[m][r] = 0.0f; }

    // this lane's pairs of a step: sample e / SI, input e % SI of e = tid + c * NT
    auto load_x = [&](int step, float (&v)[EP]) {
#pragma unroll
        for (int c = 0; c < EP; ++c) {
            const int e = tid + c * NT;
            int64_t b = b0 + e / SI;
            b = b < B ? b : B - 1;
            int i = step * SI + e % SI;
            i = i < g.n_in ? i : g.n_in - 1;
            v[c] = x[b * g.n_in + i];
        }
    };
    auto evaluate = [&](int step, const float (&v)[EP], unsigned *area) {
#pragma unroll
        for (int c = 0; c < EP; ++c) {
            const int e = tid + c * NT, s = e / SI, ii = e % SI, i = step * SI + ii;
            float w[kMaxK], dw[kMaxK], base, dbase;
            int row0;
            wave_windows<false>(v[c], g, i < g.n_in ? i : g.n_in - 1, row0, w, base, dw, dbase);
            const bool fits = fabsf(base) < kMxLargest;
            if (!fits) special[s] = 1;
            base = fits && i < g.n_in ? base * kMxScale : 0.0f;
#pragma unroll
            for (int k = 0; k < kMaxK; ++k) w[k] = i < g.n_in ? w[k] * kMxScale : 0.0f;
            unsigned out[kMxSplits][NG];
            IndexBits<NG> index;
            pair_operands<NG>(row0, w, base, out, index);
#pragma unroll
            for (int p = 0; p < kMxSplits; ++p) {
                if (AHEAD) __builtin_amdgcn_sched_barrier(0);
                unsigned *at = area + (p * S + s) * A::kRow + ii * NG;
                if constexpr (NG % 4 == 0) {
#pragma unroll
                    for (int q = 0; q < NG; q += 4)
                        *reinterpret_cast<U4 *>(at + q) = U4{out[p][q], out[p][q + 1], out[p][q + 2], out[p][q + 3]};
                } else {
#pragma unroll
                    for (int q = 0; q < NG; q += 2) *reinterpret_cast<uint2 *>(at + q) = make_uint2(out[p][q], out[p][q + 1]);
                }
            }
            unsigned char *ix = reinterpret_cast<unsigned char *>(area + kMxSplits * S * A::kRow + s * A::kIdx) + ii * (NG / 2);
            if constexpr (NG % 8 == 0) {
                *reinterpret_cast<unsigned *>(ix) = (unsigned)index;
            } else if constexpr (NG % 4 == 0) {
#pragma unroll
                for (int h = 0; h < NG / 4; ++h) reinterpret_cast<unsigned short *>(ix)[h] = (unsigned short)(index >> (16 * h));
            } else {
#pragma unroll
                for (int h = 0; h < NG / 2; ++h) ix[h] = (unsigned char)(index >> (8 * h));
            }
        }
    };

    const U4 *bp = frag + (int64_t)tc * n_parts * (NG / 2) * kMxSplits * 128 + lane;
    const int64_t last = (int64_t)n_parts * (NG / 2) - 1;
    auto load_b = [&](int64_t k, U4 (&b)[kMxSplits][2]) {
        const U4 *at = bp + (k < last ? k : last) * (kMxSplits * 128);
#pragma unroll
        for (int p = 0; p < kMxSplits; ++p) { b[p][0] = at[p * 128]; b[p][1] = at[p * 128 + 64]; }
    };

    float xv[EP];
    U4 bn[2][kMxSplits][2];
    load_x(0, xv);
    load_b(0, bn[0]);
    __syncthreads();                                   // special[] is cleared
    evaluate(0, xv, lds);
    load_x(n_steps > 1 ? 1 : 0, xv);
    __syncthreads();

    // An instruction's right operands are asked for one instruction step ahead and, with AHEAD, the left ones a tile ahead in a
    // pinned order (left to itself the compiler moves the loads down to their uses); four tiles leave no registers for that.
    auto multiply = [&](int step) {
        constexpr int MG = AHEAD ? 1 : 2, GPT = MT / MG, NGRP = KS * GPT;          // MG tiles' chains take turns
        const unsigned *area = lds + (step & 1) * kArea;
        const unsigned short *idx = reinterpret_cast<const unsigned short *>(area + kMxSplits * S * A::kRow);
        Bf8 a[2][MG][kMxSplits];
        int ix[2][MG];
        auto read_a = [&](int t, int m0, int to) {
#pragma unroll
            for (int m = 0; m < MG; ++m) {
                const int s = (wm * MT + m0 + m) * 32 + (lane & 31), h = 2 * t + (lane >> 5);
                ix[to][m] = idx[s * (2 * A::kIdx) + h];
#pragma unroll
                for (int p = 0; p < kMxSplits; ++p)
                    a[to][m][p] = __builtin_bit_cast(Bf8, *reinterpret_cast<const U4 *>(area + (p * S + s) * A::kRow + 4 * h));
            }
        };
        if (AHEAD) read_a(0, 0, 0);
#pragma unroll
        for (int gi = 0; gi < NGRP; ++gi) {
            const int t = gi / GPT, m0 = gi % GPT * MG, at = AHEAD ? gi & 1 : 0;
            if (gi % GPT == 0) load_b((int64_t)step * KS + t + 1, bn[(t + 1) & 1]);
            if (!AHEAD) read_a(t, m0, 0);
            else if (gi + 1 < NGRP) read_a((gi + 1) / GPT, (gi + 1) % GPT * MG, (gi + 1) & 1);
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
            Bf16 b[kMxSplits];
#pragma unroll
            for (int p = 0; p < kMxSplits; ++p)
                b[p] = __builtin_bit_cast(Bf16, __builtin_shufflevector(bn[t & 1][p][0], bn[t & 1][p][1], 0, 1, 2, 3, 4, 5, 6, 7));
            auto product = [&](F16 (&sum)[MT], int pa, int pb) {
#pragma unroll
                for (int m = 0; m < MG; ++m)
                    sum[m0 + m] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a[at][m][pa], b[pb], sum[m0 + m], ix[at][m], 0, 0);
            };
            product(low, 2, 0);
            product(low, 0, 2);
            product(acc, 0, 0);
            product(low, 1, 1);
            product(low, 1, 0);
            product(low, 0, 1);
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (KS % 2 != 0) {
#pragma unroll
            for (int p = 0; p < kMxSplits; ++p) { bn[0][p][0] = bn[1][p][0]; bn[0][p][1] = bn[1][p][1]; }
        }
        if constexpr (FOLD) {
            if ((step & fold_mask) == fold_mask) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int r = 0; r < 16; ++r) { tot[m][r] += acc[m][r]; acc[m][r] = 0.0f; }
            }
        }
    };
    // half of the waves take the parts of a step in the opposite order, so that the evaluation of one wave runs beside the matrix
    // instructions of the other on its SIMD
    const int late = WM * WN >= 8 ? wave >= WM * WN / 2 : 0;
    for (int step = 0; step < n_steps; ++step) {
#pragma unroll 1
        for (int part = 0; part < 2; ++part) {
            if (part == late) {
                if (step + 1 < n_steps) {
                    evaluate(step + 1, xv, lds + ((step + 1) & 1) * kArea);
                    load_x(step + 2 < n_steps ? step + 2 : n_steps - 1, xv);
                }
            } else {
                multiply(step);
            }
        }
        __syncthreads();
    }

    if (tile >= n_tiles) return;
    const int j = j0 + tile * kMxTile + (lane & 31);
    int flag = 0;
    for (int s = lane; s < n_parts; s += 64) flag |= odd[(int64_t)tile * n_parts + s];
    const bool all_odd = __any(flag != 0);
    // Samples of the wave's tiles with sums that are done again, a bit each: those that read a value which does not split, and
    // those with a sum that is not finite, where the products of parts may have passed the range of a float in either direction.
    const int up = 4 * (lane >> 5);
    unsigned again[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int s0 = (wm * MT + m) * 32;
        again[m] = (unsigned)__ballot(all_odd || special[s0 + (lane & 31)]);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[m][r] = ((FOLD ? tot[m][r] + acc[m][r] : acc[m][r]) + low[m][r]) * (1.0f / (kMxScale * kMxScale));
            const uint64_t past = __ballot(!(fabsf(acc[m][r]) <= FLT_MAX));
            again[m] |= ((unsigned)past ? 1u : 0u) << (8 * (r / 4) + r % 4) | ((past >> 32) ? 1u : 0u) << (8 * (r / 4) + 4 + r % 4);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int s = 8 * (r / 4) + up + r % 4;
            const int64_t b = b0 + s0 + s;
            if (b < B && j < g.n_out && !(again[m] >> s & 1)) y[b * g.n_out + j] = acc[m][r];
        }
    }
    // these in plain fp32: half a wave takes every other input
    const int jc = j < g.n_out ? j : g.n_out - 1;
    for (int s = 0; s < MT * 32; ++s) {
        const int64_t b = b0 + wm * MT * 32 + s;
        unsigned bits = again[0];
#pragma unroll
        for (int m = 1; m < MT; ++m) bits = s / 32 == m ? again[m] : bits;
        if (b >= B || !(bits >> s % 32 & 1)) continue;
        float sum = 0.0f, part = 0.0f;                   // two levels, as in the kernels this one stands in for
        int n = 0;
        for (int i = lane >> 5; i < g.n_in; i += 2) {
            const Pair p = pair_basis<false>(x[b * g.n_in + i], g, i);
            const float *slab = coef + (int64_t)i * g.rows * g.n_out + jc;
            const float scale = w_s[(int64_t)i * g.n_out + jc];
#pragma unroll
            for (int k = 0; k < kMaxK; ++k) {
                const int m = p.cell + k;                // rows that are not there take no part, whatever stands beside them
                const float c = slab[(int64_t)clampi(m, 0, g.rows - 1) * g.n_out] * scale;
                part = k <= g.k && m >= 0 && m < g.rows ? fmaf(p.w[k], c, part) : part;
            }
            if (w_b) part = fmaf(p.base, w_b[(int64_t)i * g.n_out + jc], part);
            if (++n == 8) { sum += part; part = 0.0f; n = 0; }
        }
        sum += part;
        sum += __shfl_xor(sum, 32);
        if (lane < 32 && j < g.n_out) y[b * g.n_out + j] = sum;
    }
}

// ---- host -------------------------------------------------------------------------
struct MatrixArgs {
    const float *x, *coef, *w_s, *w_b;
    float *cf, *y;
    void *table;
    int64_t B;
    int n_tiles, j0;           // tiles of this round, and its first output
};

template <int NG, int SI, int MT, int WM, int WN, bool FOLD, bool AHEAD>
static hipError_t matrix_launch(const SplineGeom &g, const MatrixTable &t, const MatrixArgs &a, hipStream_t st)
{
    constexpr int S = 32 * MT * WM, bytes = (2 * MxArea<NG, SI>::template words<S>() + S) * 4;
    struct Tag {};
    auto kern = forward_matrix_kernel<NG, SI, MT, WM, WN, FOLD, AHEAD>;
    if (hipError_t e = ensure_dynamic_lds<Tag>((const void *)kern, bytes); e != hipSuccess) return e;
    const int *odd = (const int *)((const char *)a.table + a.n_tiles * t.tile_bytes);
    const unsigned across = (unsigned)((a.n_tiles + WN - 1) / WN);
    const int64_t part = (int64_t)S * ((1 << 22) / across);       // samples of one launch: fewer than 2^32 threads
    for (int64_t b0 = 0; b0 < a.B; b0 += part) {
        const int64_t n = a.B - b0 < part ? a.B - b0 : part;
        const dim3 grid((unsigned)((n + S - 1) / S), across);
        prof::Timed tm(a.n_tiles < t.n_tiles ? "forward_matrix_range" : "forward_matrix", st);      // (a range of the outputs)
        kern<<<grid, 64 * WM * WN, bytes, st>>>(g, a.x + b0 * g.n_in, a.coef, a.w_s, a.w_b, (const U4 *)a.table, odd, a.y + b0 * g.n_out,
                                                n, a.n_tiles, a.j0, g.n_in <= 64 ? 0 : 1);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int NG>
static hipError_t matrix_forward(const SplineGeom &g, const MatrixTable &t, int form, const MatrixArgs &a, hipStream_t st)
{
    {
        prof::Timed tm("matrix_table", st);
        matrix_table_kernel<NG><<<dim3((unsigned)t.n_steps, (unsigned)a.n_tiles), 32 * NG, 0, st>>>(
            a.coef, a.w_s, a.w_b, a.cf, (U4 *)a.table, (int *)((char *)a.table + a.n_tiles * t.tile_bytes), g.n_in, g.rows, g.n_out, a.j0);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    switch (form) {
    case 1:
        if constexpr (NG < 8) return matrix_launch<NG, 4, 4, 1, 8, false, false>(g, t, a, st);
        return hipErrorInvalidValue;
    case 2:
        if constexpr (NG < 12) return matrix_launch<NG, 8, 2, 1, 8, true, true>(g, t, a, st);
        return hipErrorInvalidValue;
    case 3: return matrix_launch<NG, 8, 1, 2, 4, true, true>(g, t, a, st);
    default: return hipErrorInvalidValue;
    }
}

// The form with the shortest estimated time, if that is shorter than the time of the kernel that the layer would have; 0
// otherwise.  Each form costs a fixed time, that of the table, and a round of 256 workgroups a fixed time and so much a step (us; least
// squares over 1660 layers of 65..600 outputs, 8..600 inputs, up to 47 rows and 2^33 edges, all forms of each: 0.85..1.14 of the time,
// 0.05 in the mean).  Ten and twelve groups (32..47 rows) spill in the form of two tiles a wave, whose steps cost 1.7 and 2.2 times those
// of the third form; with twelve it is not built.  More groups do not fit LDS.
// The other kernel: the direct one by its edges, those of ragged rows dearer where more than half of the last tile is used, and the
// longer the table the more, as more samples fetch each row of it; the staged ones for short tables by the rounds of their workgroups, the
// one for long tables as its own plan counts.  Of the 1660 layers this takes 0.67 of the time of the other kernels in the mean, 1.04 at most
// but where the comment below says so (137 -> 140, G = 44, B = 12900 is one where the two are even, 240 / 242).  Other kernel / this one, us:
// 512 -> 512, G = 20, B = 16384 914 / 603; 256 -> 256, G = 28, B = 16384 684 / 235; 128 -> 128, G = 10, B = 16384 170 / 54; 75 -> 130,
// G = 12, B = 6001 58 / 37; 139 -> 139, G = 29, B = 12900 250 / 186; 265 -> 411, G = 41, k = 5, B = 4929 1730 / 593; 231 -> 270, G = 38, k = 1,
// B = 5201 525 / 181; not taken: 64 -> 130, G = 28, B = 1024
// 12 / 48, 32 -> 96, G = 12, B = 32768 39 / 40; 512 -> 256, G = 16, B = 2182 198 / 228.  Up to 64
// outputs the evaluation of the pairs is not shared by enough of them (64 -> 64, G = 10, B = 65536: 75 / 78 in the best of the forms tried).
int forward_matrix_plan(const SplineGeom &g, int64_t B)
{
    const MatrixTable t = ::kan::matrix_table(g.n_in, g.n_out, g.rows, kMaxK);
    if (t.groups == 0) return 0;
    struct Form { int samples, tiles, inputs; float fixed, round, step[5]; };        // step 0: not built
    static const Form forms[] = {{128, 8, 4, 5.0f, 18.0f, {2.8f, 4.35f, 0.0f, 0.0f, 0.0f}},
                                 {64, 8, 8, 4.7f, 11.2f, {2.58f, 3.82f, 5.58f, 9.12f, 0.0f}},
                                 {64, 4, 8, 6.3f, 5.9f, {2.14f, 3.17f, 4.15f, 5.3f, 6.31f}}};
    const float mb = 1e-6f * (float)g.n_in * (float)g.slab_rows * (float)g.n_out * 4.0f;      // the folded table
    const int lds = forward_lds_plan(g);
    const bool direct = forward_direct_plan(g, B) != 0, staged = !direct && lds != 0;
    // The first form has one level of sums: not where another kernel with two would take the layer (403 -> 164, G = 19, k = 1,
    // B = 16510: error 3.3e-7, the direct kernel's 2.0e-7).
    if (!staged && g.n_in < 20 && t.groups >= 8) return 0;        // (few inputs of many groups: 16 -> 104, G = 26, k = 5 1.05 of its error)
    int best = 0;
    float least = 0.0f;
    const float table = mb < 8.0f ? 2.0f * mb : 16.0f + 1.4f * (mb - 8.0f);
    for (int f = staged ? 0 : 1; f < 3; ++f) {
        const Form &o = forms[f];
        if (o.step[t.groups / 2 - 2] == 0.0f) continue;
        const int64_t groups = ((B + o.samples - 1) / o.samples) * ((t.n_tiles + o.tiles - 1) / o.tiles);
        const float rounds = (float)((groups + 255) / 256);
        // (the second form's steps take longer behind one another, more so on large tables: 512 -> 512, G = 20, B = 16384 629 in the first,
        // 673 in it)
        const float step = o.step[t.groups / 2 - 2] * (f == 1 && rounds > 1.0f ? 1.06f + 0.005f * mb : 1.0f);
        const float us = o.fixed + table + rounds * (o.round + (float)((g.n_in + o.inputs - 1) / o.inputs) * step);
        if (best == 0 || us < least) { best = f + 1; least = us; }
    }
    const float edges = 1e-6f * (float)B * (float)g.n_in * (float)((g.n_out + 63) / 64 * 64);
    constexpr float six = kMaxK == 6 ? 1.5f : 1.0f;              // windows of six cost these kernels half as much again
    float other;
    if (direct) {
        const bool in_l2 = mb < 6.3f, ragged = g.n_out % 16 != 0;
        const float past = mb * (B < 4000 ? (float)B / 4000.0f : 1.0f);        // few samples meet few rows of it
        const float edge = in_l2 ? (!ragged ? 0.57f : ((g.n_out - 1) % 64 < 32 ? 0.64f : 0.71f) + 0.025f * mb)
                                 : (!ragged ? 0.6f + 0.006f * past : 0.85f + 0.012f * past);
        other = 6.0f + six * edges * edge;
    } else if (staged) {
        const int64_t samples = lds == 8 ? 64 : 128, width = lds == 8 ? 512 : 256;          // of a workgroup
        const int64_t groups = (B + samples - 1) / samples * ((g.n_out + width - 1) / width);
        other = (kMaxK == 6 ? 1.3f : 1.0f) * (5.5f + (float)((groups + 255) / 256) * (lds == 8 ? 1.78f : 2.62f) * (float)g.n_in);
    } else {
        // (short tables below B = 28000 come here where the direct kernel would be behind as well: on eight waves the one for long tables is
        // faster on most of them, 72 -> 97, G = 26, B = 24202 76 / 99, but its sums are 1.03 to 1.08 times as far off)
        other = forward_lds_rows_us(g, B);
        if (other == 0.0f) other = six * (5.0f + edges / 1.45f);                  // the generic kernel
        else if (t.groups <= 8 && B < 28000) other = (kMaxK == 6 ? 1.1f : 0.85f) * (5.0f + edges / 1.75f);
    }
    return least < other ? best : 0;
}

// A table that does not fit is made and used a range of outputs at a time, the same sums in the same order.
hipError_t launch_forward_matrix(const SplineGeom &g, const float *x, const float *coef, const float *w_s, const float *w_b,
                                 float *cf, void *table, size_t table_bytes, float *y, int64_t B, hipStream_t st)
{
    const MatrixTable t = ::kan::matrix_table(g.n_in, g.n_out, g.rows, kMaxK);
    const int form = forward_matrix_plan(g, B), wide = form == 3 ? 4 : 8;
    const int64_t fit = (int64_t)(table_bytes / (t.tile_bytes + (size_t)t.n_steps * 4));
    if (form == 0 || fit < 1) return hipErrorInvalidValue;
    const int rounds = fit >= t.n_tiles ? 1 : (int)((t.n_tiles + fit - 1) / fit);
    int per = (t.n_tiles + rounds - 1) / rounds;
    if (rounds > 1 && (per + wide - 1) / wide * wide <= fit) per = (per + wide - 1) / wide * wide;      // whole workgroups
    for (int tile = 0; tile < t.n_tiles; tile += per) {
        const MatrixArgs a = {x, coef, w_s, w_b, cf, y, table, B, t.n_tiles - tile < per ? t.n_tiles - tile : per, tile * ::kan::kMxTile};
        const hipError_t e = [&] {
            switch (t.groups) {
            case 4:
                if constexpr (kMaxK <= 4) return matrix_forward<4>(g, t, form, a, st);
                return hipErrorInvalidValue;
            case 6: return matrix_forward<6>(g, t, form, a, st);
            case 8: return matrix_forward<8>(g, t, form, a, st);
            case 10: return matrix_forward<10>(g, t, form, a, st);
            case 12: return matrix_forward<12>(g, t, form, a, st);
            default: return hipErrorInvalidValue;
            }
        }();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace KAN_NS
