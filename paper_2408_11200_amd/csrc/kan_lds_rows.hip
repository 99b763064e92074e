// LDS-staged forward kernel for tables too long for forward_lds_kernel (a slab of a 256- or
// 512-wide output tile no longer fits LDS): hundreds of rows per input, as on large grids and on
// the generated tables of UKAN layers.
//
// Such layers used to gather their window rows straight from L2 (forward_generic_kernel), four
// 1 KB rows per (sample, input) pair, and ran at the rate at which a CU can pull lines out of L2.
// Here a workgroup takes a NARROW output tile (TJ = 64 or 32 outputs) and MANY samples
// (NW waves x SPW x S): the slab of the current input for that tile (slab_rows x TJ floats) is
// staged in LDS, double-buffered, and every row fetched from L2 once serves all the workgroup's
// samples, which cuts the L2 traffic by (samples x K) / slab_rows.
//
// Mapping inside a wave: the 64 lanes are SPW = 64 / LPS groups of LPS lanes; a group works on one
// sample at a time and its lanes hold four consecutive outputs each (LPS * 4 = TJ), so one 16-byte
// LDS read per lane fetches a window row for SPW samples at once (each group reads its own row).
// Every group handles S samples (slots), accumulators for all of them stay in registers
// (S x 4 per lane) while the workgroup walks over the inputs.  The per-pair quantities (K weights,
// base value, byte offsets of the window rows) go through a small per-wave area of LDS, written by the
// lane that evaluated the pair and read back by the group that owns the sample.
//
// Bound by the multiply-adds and the LDS reads of the window rows, both about 60 % busy; what was beside them and is gone:
//   - the multiply-adds waited for the evaluation of their pairs' x, and the copy for the multiply-adds: what a step reads from
//     memory is asked for a step or a round ahead (of windows of six rows half the waves take the parts the other way round);
//   - two groups' 128-byte rows of tiles of 32 met in a bank every other time, and pairs of groups eight samples apart always
//     (half of all LDS clocks): rows are read by parity, a group's samples are SPW apart;
//   - a step copied whole multiples of the workgroup, up to nine times its slab, and had a barrier for each input;
//   - x came one value a cache line, and its way from memory was waited for.
//   - a spill, or a use of an older load after a younger one was sent, waits for the copy under way.
// us, before / after: the wide layers of 128 -> 256 -> 256 -> 1, B = 32768, tables of 180 and 360 rows 1455 / 920 (the longer
// tables 500 on the old banks, 362 on these); 32 -> 32, G = 256, B = 131072 with its fold 76 / 57; 64 -> 64, G = 10, B = 65536
// 103 / 79.  Layers of two to twelve inputs, whose few steps do not hide the first copy: 0.88 of the time over all, 1.09 at most
// (3 -> 100, G = 64, B = 65536: 19.6 / 21.3).
// Windows of six rows (degrees 4 and 5, kan_lds_rows_k5.hip) against the direct and the row-stream kernel they had: 32 -> 32,
// G = 64, k = 5, B = 65536 with the fold 80 / 50; 600 calls of 8..128 inputs, 32..256 outputs: 0.69 of the time, 1.08 at most.
#include <type_traits>
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_wave.hpp"

namespace KAN_NS {

namespace {

// w[0..K), then two byte offsets of window rows and the base value; a tile of 64 has one offset and the base value
constexpr int kPairFloats = kMaxK == 4 ? 8 : 12;

}  // namespace

// A workgroup per (NW * SPW * S samples, TJ outputs), NW waves.  Needs rows >= kMaxK, n_out >= 4, for S = 8 four inputs.
// BASE: the table has slab_rows = rows + 1 rows per input, the last one the w_b row.  P (a power of two up to IPV): inputs a step;
// the sums are folded every `fold` inputs (a power of two).
template <int LPS, int S, int NW, int NQ, bool BASE>
__global__ __launch_bounds__(64 * NW) void forward_lds_rows_kernel(SplineGeom g, const float *__restrict__ x,
                                                                   const float *__restrict__ cf,
                                                                   float *__restrict__ y, int64_t B, int P, int fold,
                                                                   int n_tiles)
{
    constexpr int TJ = LPS * 4, SPW = 64 / LPS, NT = 64 * NW;
    constexpr int SMP = SPW * S;                        // samples per wave
    constexpr int IPV = 64 / SMP;                       // inputs one round of pair evaluations covers
    constexpr int slab_floats = NQ * NT * 4;            // padded slabs of a step
    static_assert(SMP <= 64 && 64 % SMP == 0, "the wave's samples must tile its lanes");
    extern __shared__ float lds[];                      // two steps' slabs, then NW areas of 64 pairs
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane / LPS, lj = lane % LPS;
    // Workgroups go to the 8 XCDs round-robin; an XCD takes neighbours in the order of the tiles, so that the workgroups that
    // copy the same slabs at the same time share an L2.  Not where a layer has few inputs: a last tile of a few outputs is then less
    // work than the others, and the XCDs that have only those wait (1 -> 65, G = 111, B = 116107: 23.4 us, 21.3 this way round).
    const int n_rows = (int)((B + NW * SMP - 1) / (NW * SMP));
    const int id = g.n_in < 8 ? (int)blockIdx.x : (int)(blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8);
    if (id >= n_rows * n_tiles) return;
    const int64_t b0 = ((int64_t)(id % n_rows) * NW + wave) * SMP;
    const int j0 = id / n_rows * TJ;
    const int j = j0 + lj * 4;
    float *pairs = lds + 2 * slab_floats + wave * (64 * kPairFloats);

    // two-level sum over the inputs (acc is folded into tot every 32 inputs, or more often where the plan says so): keeps the
    // rounding error of a sum over hundreds of inputs inside the forward tolerance
    float acc[S][4], tot[S][4];
#pragma unroll
    for (int q = 0; q < S; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) { acc[q][r] = 0.0f; tot[q][r] = 0.0f; }

    // slab copy: thread tid moves quads tid, tid + NT, ... of a step's rows (the table's rows follow each other over the
    // inputs).  Zeros are copied for rows and outputs that are not there.
    const int step_rows = P * g.slab_rows;
    int off[NQ];                                        // in bytes; past the end of every buffer for what is not there
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        const int e = tid + c * NT;
        const int row = e / LPS, jj = j0 + (e % LPS) * 4;
        off[c] = row < step_rows && jj < g.n_out ? (row * g.n_out + (jj + 4 > g.n_out ? g.n_out - 4 : jj)) * 4 : INT32_MIN;     // a row's last quad: n_out - 4 ..
    }
    const int copies = (step_rows * LPS - wave * 64 + NT - 1) / NT;      // of the wave; the others are padding only
    // shifts: a division by P costs a step of few multiply-adds as much as one of its LDS round trips (9 -> 40, G = 59, k = 2,
    // B = 25352 14.2 / 13.9 us, 1 -> 34, G = 74, B = 145799 18.3 / 17.1)
    const int log_p = __builtin_ctz(P), log_round = __builtin_ctz(IPV) - log_p;     // a round of evaluations: 1 << log_round steps
    const int n_steps = (g.n_in + P - 1) >> log_p;
    const int64_t step_floats = (int64_t)step_rows * g.n_out;
    f32x4 qd[NQ];
    auto fetch = [&](int t) {
        const int inputs = g.n_in - t * P < P ? g.n_in - t * P : P;      // loads past the table's end return zeros
        const i32x4 block = buffer_of(cf + (int64_t)t * step_floats, (unsigned)(inputs * g.slab_rows * g.n_out) * 4u);
#pragma unroll
        for (int c = 0; c < NQ; ++c)
            if (c < copies) qd[c] = buffer_load4(block, off[c], 0, 0);
    };
    auto stage = [&](float *slab) {
#pragma unroll
        for (int c = 0; c < NQ; ++c)
            if (c < copies) *reinterpret_cast<f32x4 *>(slab + (tid + c * NT) * 4) = qd[c];
    };

    // pair evaluation: lane <-> (input my_ii of the round, sample my_smp of the wave); what it reads is asked for a round
    // ahead, four inputs at a time where the lanes are all samples (a row of x is a cache line of its own)
    const int my_smp = lane % SMP;
    int my_ii = lane / SMP;
    asm("" : "+v"(my_ii));             // keeps cell_base's load a vector one, which does not hold up the waits for LDS
    const int64_t my_b = b0 + my_smp < B ? b0 + my_smp : B - 1;
    const float *__restrict__ xrow = x + my_b * g.n_in;
    float xv[IPV == 1 ? 4 : 1];
    int cell_base = 0;
    auto ask = [&](int round) {
        const int mi = round * IPV + my_ii;
        const int ic = mi < g.n_in ? mi : g.n_in - 1;
        if constexpr (IPV == 1) {
            if (round % 4 == 0) {
                const float4 v = load4u(xrow + (ic < g.n_in - 4 ? ic : g.n_in - 4));
                xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w;
            }
        } else {
            xv[0] = xrow[ic];
        }
        if (g.cell_base) cell_base = g.cell_base[ic];
    };
    auto evaluate = [&](int round) {
        float v = xv[0];
        if constexpr (IPV == 1) {
            const int first = round / 4 * 4;
            const int c = round - (first < g.n_in - 4 ? first : g.n_in - 4);
            v = c == 0 ? xv[0] : c == 1 ? xv[1] : c == 2 ? xv[2] : xv[3];
        }
        SplineGeom gi = g;
        gi.cell_base = &cell_base;
        gi.base_act = BASE ? 1 : 0;
        int row0;
        float w[kMaxK], dw[kMaxK], base, dbase;
        wave_windows<false>(v, gi, 0, row0, w, base, dw, dbase);
        row0 += (my_ii & (P - 1)) * g.slab_rows;
        // pair (input ii of the round, sample smp) sits at index ii * SMP + smp == the lane that evaluated it
        float *pair = pairs + lane * kPairFloats;
        if constexpr (kMaxK == 6) {
            const bool swap = LPS == 8 && ((row0 + my_smp) & 1);       // as below, rows 4 and 5 too
            *reinterpret_cast<float4 *>(pair) = make_float4(w[swap ? 1 : 0], w[swap ? 0 : 1], w[swap ? 3 : 2], w[swap ? 2 : 3]);
            *reinterpret_cast<float4 *>(pair + 4) =
                make_float4(w[swap ? kMaxK - 1 : kMaxK - 2], w[swap ? kMaxK - 2 : kMaxK - 1], __int_as_float((row0 + (swap ? 1 : 0)) * TJ * 4),
                            LPS == 16 ? base : __int_as_float((row0 + (swap ? 0 : 1)) * TJ * 4));
            if constexpr (LPS == 8 && BASE) pair[8] = base;
        } else if constexpr (LPS == 16) {
            *reinterpret_cast<float4 *>(pair) = make_float4(w[0], w[1], w[2], w[3]);
            *reinterpret_cast<float2 *>(pair + 4) = make_float2(__int_as_float(row0 * TJ * 4), base);
        } else {
            // A row is half the banks: neighbouring groups start with rows of different parity and swap rows 0 and 1, 2 and 3
            // of the window accordingly, so that their reads never meet in a bank.
            const bool swap = (row0 + my_smp) & 1;
            *reinterpret_cast<float4 *>(pair) = make_float4(swap ? w[1] : w[0], swap ? w[0] : w[1], swap ? w[3] : w[2], swap ? w[2] : w[3]);
            *reinterpret_cast<float4 *>(pair + 4) = make_float4(__int_as_float((row0 + (swap ? 1 : 0)) * TJ * 4),
                                                                __int_as_float((row0 + (swap ? 0 : 1)) * TJ * 4), base, 0.0f);
        }
    };

    // slots whose rows are in flight together: with more the kernel spills, and every spill waits for the copies on their way
    constexpr int kAtOnce = S == 8 ? (kMaxK == 4 && NQ + BASE < 4 ? 2 : 1) : NW == 8 || (kMaxK == 4 && NQ + BASE < 5) ? 4 : 2;
    auto compute = [&](int t) {
        const int i0 = t * P;
        const float *cur = lds + (t & 1) * slab_floats;
        if ((i0 & (fold - 1)) == 0) {
#pragma unroll
            for (int q = 0; q < S; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) { tot[q][r] += acc[q][r]; acc[q][r] = 0.0f; }
        }
        const int n_ii = g.n_in - i0 < P ? g.n_in - i0 : P;
#pragma clang loop unroll(disable)
        for (int ii = 0; ii < n_ii; ++ii) {
            float4 wb = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (BASE) wb = *reinterpret_cast<const float4 *>(cur + (ii * g.slab_rows + g.rows) * TJ + lj * 4);
            const float *pp = pairs + (((i0 + ii) % IPV) * SMP + grp) * kPairFloats;     // samples grp, grp + SPW, ...
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const float *pq = pp + q * (SPW * kPairFloats);
                float ws[kMaxK];
                float2 at;
                const float4 wa = *reinterpret_cast<const float4 *>(pq);
                ws[0] = wa.x; ws[1] = wa.y; ws[2] = wa.z; ws[3] = wa.w;
                if constexpr (kMaxK == 4) {
                    at = *reinterpret_cast<const float2 *>(pq + 4);
                } else {
                    const float4 wc = *reinterpret_cast<const float4 *>(pq + 4);
                    ws[4] = wc.x; ws[5] = wc.y;
                    at = make_float2(wc.z, wc.w);
                }
                const float base = !BASE ? 0.0f : LPS == 16 ? at.y : pq[kMaxK + 2];
                const char *win = reinterpret_cast<const char *>(cur + lj * 4);
                const float *w0 = reinterpret_cast<const float *>(win + __float_as_int(at.x));
                const float *w1 = LPS == 16 ? w0 + TJ : reinterpret_cast<const float *>(win + __float_as_int(at.y));
                float4 c[kMaxK];
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) c[s] = *reinterpret_cast<const float4 *>((s % 2 ? w1 : w0) + s / 2 * 2 * TJ);
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) {
                    acc[q][0] = fmaf(ws[s], c[s].x, acc[q][0]);
                    acc[q][1] = fmaf(ws[s], c[s].y, acc[q][1]);
                    acc[q][2] = fmaf(ws[s], c[s].z, acc[q][2]);
                    acc[q][3] = fmaf(ws[s], c[s].w, acc[q][3]);
                }
                if constexpr (BASE) {
                    acc[q][0] = fmaf(base, wb.x, acc[q][0]);
                    acc[q][1] = fmaf(base, wb.y, acc[q][1]);
                    acc[q][2] = fmaf(base, wb.z, acc[q][2]);
                    acc[q][3] = fmaf(base, wb.w, acc[q][3]);
                }
                if ((q + 1) % kAtOnce == 0) __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // A step's copy and pair evaluation come before its multiply-adds, or behind them for the next one; a wave's pairs are its own.
    // Windows of six rows with sixteen waves: two of a SIMD's four waves take the parts in the opposite order, so that LDS writes,
    // evaluation and multiply-adds of different waves overlap between two barriers.  Both orders together are twice the code, which
    // costs more than it gives elsewhere (us, mixed / before / behind:
    //   four rows              32 -> 32, G = 256, B = 131072 56.2 / 55.2 / 58.5; 256 -> 256, G = 176, B = 32768 558 / 553 / 571;
    //                          9 -> 40, G = 59, k = 2, B = 25352 14.4 / 13.2 / 13.3; 14 -> 40, G = 17, B = 9972 17.4 / 16.1 / 16.1
    //                          but 64 -> 64, G = 10, B = 65536, four inputs a step 81.7 / 84.7
    //   six rows, sixteen      32 -> 32, G = 64, B = 65536 39.7 / 41.6 / 40.4
    //             eight        46 -> 36, G = 131, B = 16813 63.6 / 58.4 / 55.7; 63 -> 32, G = 6, B = 33887 67.3 / 72.3 / 70.3)
    // Loads are waited for in order, so those for later come after the uses of the earlier ones.
    const bool early = kMaxK == 4 || (NW == 16 && ((wave >> 2) & 1));
    const int per_round = 1 << log_round;
    ask(0);
    fetch(0);
    if (!early) evaluate(0);
    stage(lds);
    if (n_steps > 1) fetch(1);
    if (!early && per_round < n_steps) ask(1);
    __syncthreads();
    // beside the multiply-adds of step t: the copy for t + 1, the wave's pairs of the round that begins with step `of`
    auto prepare = [&](int t, int of, bool early) {
        float *nxt = lds + ((t + 1) & 1) * slab_floats;
        const bool begins = (of & (per_round - 1)) == 0 && of < n_steps;
        if (early && begins) {
            evaluate(of >> log_round);
            wave_lds_sync();               // compute() reads what other lanes wrote, with no barrier in between
        }
        if (t + 1 < n_steps) stage(nxt);
        if (!early && begins) {
            wave_lds_sync();               // compute() has read what is overwritten here
            evaluate(of >> log_round);
        }
        if (t + 2 < n_steps) fetch(t + 2);
        if (begins && of + per_round < n_steps) ask((of >> log_round) + 1);
    };
    for (int t = 0; t < n_steps; ++t) {
        if (early) prepare(t, t, true);
        compute(t);
        if (!early) prepare(t, t + 1, false);
        __syncthreads();
    }

    if (j < g.n_out) {
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int64_t b = b0 + q * SPW + grp;
            if (b < B)
                store4u(y + b * g.n_out + (j + 4 > g.n_out ? g.n_out - 4 : j),
                        make_float4(tot[q][0] + acc[q][0], tot[q][1] + acc[q][1], tot[q][2] + acc[q][2], tot[q][3] + acc[q][3]));
        }
    }
}

namespace {

constexpr size_t kLdsBudget = 160 * 1024;

struct RowsPlan { int lps, slots, nw, nq, inputs, fold; };

// copies a thread makes of a step's slabs: what the kernel is built for, 0 if that is too few
int copies_of(int nw, int64_t quads)
{
    const int64_t need = (quads + 64 * nw - 1) / (64 * nw);
    if (nw == 16) return need <= 4 ? (int)need : 0;
    return need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : need <= 8 ? 8 : 0;
}

constexpr size_t lds_bytes(int nw, int nq) { return 2ull * nq * 64 * nw * 16 + (size_t)nw * 64 * kPairFloats * sizeof(float); }

// the variants that there are: the others would spill registers (eight samples a group), or need more LDS than a CU has
constexpr bool variant_built(int lps, int slots, int nw, int nq, bool base)
{
    return lds_bytes(nw, nq) <= kLdsBudget && (slots == 4 || (kMaxK == 4 ? lps == 16 || nq < 4 || !base : nq < (lps == 16 ? 3 : 2)));
}
int workgroups_a_cu(int nw, int nq) { return nw == 16 || 2 * lds_bytes(nw, nq) > kLdsBudget ? 1 : 2; }

// Clocks of an input on eight waves and several tiles: a step takes `row` a window row beside the copies at 64 bytes a clock, for
// each round of workgroups, and 1.4 times that where a CU works on two.
float eight_waves_clocks(int64_t wgs, int a_cu, int64_t quads, int row)
{
    const int64_t at_once = 256 * a_cu, full = (wgs - 1) / at_once;
    const float step = (float)(row * kMaxK) + (float)quads / 4;
    return ((float)full * (a_cu == 2 ? 1.4f : 1.0f) + (wgs - full * at_once > 256 ? 1.4f : 1.0f)) * step;
}

// Eight waves on several tiles against the kernels that gather (generic and direct), at 390 clocks a window row; the
// others take an edge of the padded width in 1.5e-6 us (windows of six: 2.2e-6), more on ragged rows and past L2.  Over 326
// layers of 65..512 outputs, 8..400 inputs, 31..251 rows and B = 2048..20000 the line takes 198 to 0.79 of their time in the mean
// (1.04 at most, where runs of one side differ by as much); of the other 128 those that it would slow reach 1.5 times.
// Other kernel / this one, us: 256 -> 256, G = 200, B = 8192 346 / 279; 400 -> 100, G = 60, B = 20000 1517 / 438; 256 -> 200, G = 80,
// B = 8192 522 / 212; left: 50 -> 256, G = 230, k = 1, B = 10000 (316 workgroups, one a CU: two rounds) 85 / 129; 32 -> 96, G = 230,
// B = 20000 62 / 87.  Not below a workgroup a CU: 512 -> 512, B = 2048, G = 200 597 / 617 (on sixteen waves), G = 400 755 / 1004.
// Tiles of 32 in place of the direct kernel, which the others (33..64 outputs) are well behind: 540 a row (windows of six: 440), and
// 1.07 times the direct kernel's time where its rows are not aligned (96 -> 44, G = 179, k = 1, B = 33091 145 / 158, 57 -> 48, G = 285,
// k = 2, B = 34176 77 / 150; 96 -> 40, G = 243, k = 5, B = 38374 222 / 266; taken: 98 -> 38, G = 202, B = 40000 168 / 156, k = 4,
// B = 51421 309 / 269; 283 -> 34, G = 165, B = 55796 658 / 441).
bool eight_waves_pay(int64_t wgs, int a_cu, int64_t quads, int64_t padded_edges, bool tiles_of_32, bool ragged)
{
    const int row = !tiles_of_32 ? 390 : kMaxK == 4 ? 540 : 440;
    const float edge = (kMaxK == 4 ? 1.0f : 1.5f) * (tiles_of_32 && ragged ? 1.07f : 1.0f) / 1.5e6f;
    return eight_waves_clocks(wgs, a_cu, quads, row) < 0.92f * 2200.0f * edge * (float)padded_edges;
}

// tile width, samples a group, workgroup size, copy depth and inputs a step for a layer (lps == 0: not applicable)
RowsPlan plan_of(const SplineGeom &g, int64_t B)
{
    RowsPlan none = {0, 0, 0, 0, 0, 0};
    if (g.rows < kMaxK || g.n_out < 32) return none;
    // Windows of six: layers of fewer than eight inputs, and of up to 16 with 33 .. 35 outputs, are left to the generic and the
    // row-stream kernel.  Not for speed: this one is the faster there, past short batches (us, k = 4, G = 30, as it is / here: 2 -> 32
    // B = 16384 9.9 / 8.8, 131072 31 / 12; 7 -> 32 20 / 15, 85 / 22; 7 -> 64 131072 86 / 32; 8 -> 33 16384 17.6 / 13.5, 131072 103 / 32;
    // 16 -> 33 65536 69 / 30).
    if (kMaxK == 6 && (g.n_in < 8 || (g.n_in <= 16 && g.n_out > 32 && g.n_out < 36))) return none;
    if (g.slab_rows != g.rows + 1 && (g.slab_rows != g.rows || g.base_act != 0)) return none;
    if ((int64_t)g.slab_rows * g.n_out >= 1ll << 29) return none;           // the copies' offsets have 31 bits
    const int lps_opts[] = {16, 8, 16, 8};
    for (int o = 0; o < 4; ++o) {
        const int lps = lps_opts[o], tj = lps * 4, spw = 64 / lps;
        if (lps == 16 && g.n_out <= 32) continue;
        const int64_t tiles = (g.n_out + tj - 1) / tj;
        // 16 waves when that still leaves about a workgroup per CU, else 8
        const int nw_opts[] = {16, 8};
        for (int nw : nw_opts) {
            const int64_t per_wg = (int64_t)nw * spw * 4;
            const int64_t wgs = (B + per_wg - 1) / per_wg * tiles;
            if (nw == 16 && wgs < 256) continue;
            // Eight waves (two per SIMD) on several tiles, of which each evaluates the pairs again: eight_waves_pay.  After all others,
            // with which that does not compare them (31 -> 276, G = 211, k = 5, B = 41404: 217 us on sixteen waves and tiles of 32, 340).
            const bool eight_tiled = nw == 8 && tiles > 1;
            if (eight_tiled != (o >= 2) || (eight_tiled && wgs < 256)) continue;
            const int64_t quads = (int64_t)g.slab_rows * lps;
            const int nq = copies_of(nw, quads);
            if (!nq || !variant_built(lps, 4, nw, nq, g.base_act != 0)) continue;
            // worth it only when a staged row serves many samples (the copy into LDS costs as much LDS
            // time per row as several reads of it): samples * K >= 4 * slab rows
            const bool direct = eight_tiled && forward_direct_beside_gathers(g, B) != 0;
            if (eight_tiled ? !eight_waves_pay(wgs, workgroups_a_cu(nw, nq), quads, B * ((g.n_out + 63) / 64 * 64), direct && lps == 8, g.n_out % 4 != 0)
                            : per_wg * kMaxK < 4 * (int64_t)g.slab_rows)
                continue;
            RowsPlan p = {lps, 4, nw, nq, 1, 32};
            if (direct) {
                // In place of the direct kernel, whose sixteen lane groups share the inputs: sums as short as its, chains and number
                // of partial sums in balance (25 -> 83, G = 5, B = 19696: its error 0.95e-7, folded every 32 inputs 1.9e-7, this
                // way 0.93e-7).  The generic and the row-stream kernel fold every 32 themselves.
                const int terms = g.k + 2;
                p.fold = g.n_in < 2 * terms ? 1 : g.n_in < 8 * terms ? 2 : g.n_in < 32 * terms ? 4 : 8;
            }
            // Eight samples a group halve the copies a sample (256 -> 256, 180 rows, B = 32768: 608 us, with four 756).  A CU
            // works through its workgroups in rounds of 256; a step of four samples a group takes about 2200 clocks beside
            // the copies, which go at 64 bytes a clock.
            if (nw == 16 && g.n_in >= 4 && variant_built(lps, 8, nw, nq, g.base_act != 0)) {
                const int64_t rounds4 = (wgs + 255) / 256, rounds8 = ((B + 2 * per_wg - 1) / (2 * per_wg) * tiles + 255) / 256;
                if (rounds8 * (1100 * kMaxK + quads / 4) < rounds4 * (550 * kMaxK + quads / 4)) p.slots = 8;
            }
            // several inputs a step where their slabs fit: one barrier for all of them.  The first step's copy is waited for, so
            // there have to be steps enough, or a copy of one quad a thread (8 -> 100, G = 120, B = 32768: 19 us an input a
            // step, 21 two)
            // (Nor where it costs the CU its second workgroup of eight waves and there is one: 21 -> 64, G = 79, k = 2, B = 37888, 296
            // workgroups: 45.6 us with two inputs a step, 33 with one.)
            const int most = 64 / (spw * p.slots);
            for (int n = 2; n <= most; n *= 2) {
                const int q = copies_of(nw, n * quads);
                if (q && (q == 1 || 8 * n <= g.n_in) && (wgs <= 256 || workgroups_a_cu(nw, q) == workgroups_a_cu(nw, nq)) &&
                    variant_built(lps, p.slots, nw, q, g.base_act != 0) && n * (int64_t)g.slab_rows * g.n_out < 1ll << 29) {
                    p.inputs = n;
                    p.nq = q;
                }
            }
            return p;
        }
    }
    return none;
}

template <int LPS, int S, int NW, int NQ, bool BASE>
hipError_t launch_variant(const SplineGeom &g, const float *x, const float *cf, float *y, int64_t B, const RowsPlan &p, hipStream_t st)
{
    constexpr int SPW = 64 / LPS;
    const size_t lds = lds_bytes(NW, NQ);
    auto kern = forward_lds_rows_kernel<LPS, S, NW, NQ, BASE>;
    struct Tag;
    hipError_t e = ensure_dynamic_lds<Tag>(reinterpret_cast<const void *>(kern), (int)lds);
    if (e != hipSuccess) return e;
    const int64_t per_wg = (int64_t)NW * SPW * S, n_tiles = (g.n_out + LPS * 4 - 1) / (LPS * 4);
    const int64_t wgs = (B + per_wg - 1) / per_wg * n_tiles;
    if ((wgs + 7) * (64 * NW) >= (1ll << 32)) return hipErrorInvalidValue;      // a launch takes fewer threads (512 GiB of x and y)
    prof::Timed tm("forward_lds_rows", st);
    kern<<<(unsigned)((wgs + 7) / 8 * 8), 64 * NW, lds, st>>>(g, x, cf, y, B, p.inputs, p.fold, (int)n_tiles);
    return hipGetLastError();
}

template <int LPS, int S, int NW>
hipError_t launch_by_quads(const RowsPlan &p, const SplineGeom &g, const float *x, const float *cf, float *y, int64_t B,
                           hipStream_t st)
{
    auto with = [&](auto n, auto base) {
        constexpr int NQ = decltype(n)::value;
        constexpr bool BASE = decltype(base)::value;
        if constexpr (variant_built(LPS, S, NW, NQ, BASE)) return launch_variant<LPS, S, NW, NQ, BASE>(g, x, cf, y, B, p, st);
        else return hipErrorInvalidValue;
    };
    auto by_base = [&](auto n) { return g.base_act != 0 ? with(n, std::true_type{}) : with(n, std::false_type{}); };
    switch (p.nq) {
    case 1: return by_base(std::integral_constant<int, 1>{});
    case 2: return by_base(std::integral_constant<int, 2>{});
    case 3: if constexpr (NW == 16) return by_base(std::integral_constant<int, 3>{}); break;
    case 4: return by_base(std::integral_constant<int, 4>{});
    case 8: if constexpr (NW == 8) return by_base(std::integral_constant<int, 8>{}); break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

int forward_lds_rows_plan(const SplineGeom &g, int64_t B) { return plan_of(g, B).lps; }

// (sixteen waves at a rate that they reach or pass on tables of up to 47 rows)
float forward_lds_rows_us(const SplineGeom &g, int64_t B)
{
    const RowsPlan p = plan_of(g, B);
    if (p.lps == 0) return 0.0f;
    const int64_t tj = p.lps * 4, per_wg = (int64_t)p.nw * (64 / p.lps) * p.slots, tiles = (g.n_out + tj - 1) / tj;
    if (p.nw == 8 && tiles > 1)
        return 3.0f + (float)g.n_in * eight_waves_clocks((B + per_wg - 1) / per_wg * tiles, workgroups_a_cu(p.nw, p.nq),
                                                         (int64_t)g.slab_rows * p.lps, 390) / 2200.0f;
    return (10.0f + (float)B * (float)g.n_in * (float)((g.n_out + 63) / 64 * 64) / 4.1e6f) * (kMaxK == 4 ? 1.0f : 1.3f);
}

int forward_lds_rows_rounds(const SplineGeom &g, int64_t B)
{
    const RowsPlan p = plan_of(g, B);
    if (p.lps == 0) return 0;
    const int64_t per_wg = (int64_t)p.nw * (64 / p.lps) * p.slots, tiles = (g.n_out + p.lps * 4 - 1) / (p.lps * 4);
    const int64_t at_once = 256 * workgroups_a_cu(p.nw, p.nq);
    return (int)(((B + per_wg - 1) / per_wg * tiles + at_once - 1) / at_once);
}

hipError_t launch_forward_lds_rows(const SplineGeom &g, const float *x, const float *cf, float *y, int64_t B,
                                   hipStream_t st)
{
    const RowsPlan p = plan_of(g, B);
    if (p.lps == 16 && p.slots == 8) return launch_by_quads<16, 8, 16>(p, g, x, cf, y, B, st);
    if (p.lps == 16 && p.nw == 16) return launch_by_quads<16, 4, 16>(p, g, x, cf, y, B, st);
    if (p.lps == 16 && p.nw == 8) return launch_by_quads<16, 4, 8>(p, g, x, cf, y, B, st);
    if (p.lps == 8 && p.slots == 8) return launch_by_quads<8, 8, 16>(p, g, x, cf, y, B, st);
    if (p.lps == 8 && p.nw == 16) return launch_by_quads<8, 4, 16>(p, g, x, cf, y, B, st);
    if (p.lps == 8 && p.nw == 8) return launch_by_quads<8, 4, 8>(p, g, x, cf, y, B, st);
    return hipErrorInvalidValue;
}

}  // namespace KAN_NS
