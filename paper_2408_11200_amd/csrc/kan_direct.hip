// Forward kernel for small batches, and for narrow and ragged layers: one launch from the parameters as they are.
//
// The large-batch kernels give a workgroup 64 .. 512 samples and let it walk over all the inputs, so a
// request of a few dozen samples occupies one or two of the 256 CUs and its time is that serial walk
// (64 -> 64, G = 10, B = 16: 48 us behind a 6 us fold of the scale into the table).  What bounds such a
// call is latency alone: the launches, and the chain x -> cell -> coefficient rows -> sum.  Here
//   - a workgroup owns NS = 1 or 4 samples and one output tile, and its waves split the INPUTS between
//     them: lane groups of LPS lanes (LPS * T outputs) take every NGRP-th input, so all the row loads of a
//     sample are in flight at once; the groups' partial sums meet in LDS and are added in group order;
//   - the scale is applied as the rows are read (one multiplication, rounded as the fold rounds it), so
//     the sums need no table; the table that the backward pass wants is written by extra workgroups of
//     the same launch (none of them when the caller keeps no table).
// Same shape: 54 -> 9.2 us per call, most of what is left being the launch.
// Large batches run the same kernel with 16-byte row reads (T = 4) and four samples a workgroup, at the L2 gather rate.
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_direct_slot.hpp"

namespace KAN_NS {

namespace {

// per pair: kMaxK weights, base value, first row of the window (8 floats: two quads)
constexpr int kDirectPairFloats = 8;
constexpr int kFoldPerThread = 8;        // table elements a thread of a fold workgroup writes

template <int T>
__device__ __forceinline__ void direct_load(const float *p, float (&v)[T])
{
    if constexpr (T == 4) {
        const float4 t = load4u(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        static_assert(T == 1, "one or four outputs per lane");
        v[0] = *p;
    }
}

}  // namespace

// grid: n_tiles * ceil(B / NS) workgroups of NW waves, then (cf != nullptr) fold workgroups.
// Any rows >= 1, n_in, n_out >= T (the lane of the last outputs is moved back inside the row); tables are coef[n_in][rows][n_out].  w_s == nullptr: coef is scaled
// already (a generated table); cf must then be null.
template <int LPS, int T, int NS, int NW>
__global__ __launch_bounds__(64 * NW) void forward_direct_kernel(SplineGeom g, const float *__restrict__ x,
                                                                 const float *__restrict__ coef,
                                                                 const float *__restrict__ w_s,
                                                                 const float *__restrict__ w_b,
                                                                 float *__restrict__ cf, float *__restrict__ y,
                                                                 int64_t B, int n_tiles, int64_t n_main)
{
    constexpr int NT = 64 * NW, NGRP = NT / LPS, TJ = LPS * T, IPR = NT / NS;
    static_assert(kMaxK <= 6, "a pair record is two quads");
    __shared__ float4 pairs[NT * (kDirectPairFloats / 4)];
    __shared__ float sums[NGRP * NS * TJ];
    const int tid = threadIdx.x;

    if ((int64_t)blockIdx.x >= n_main) {
        // fold: cf[i][m][j] = w_s[i][j] * coef[i][m][j], last row w_b (as fold_scale_kernel)
        const int64_t per_in = (int64_t)(g.rows + 1) * g.n_out, total = (int64_t)g.n_in * per_in;
        const int64_t p0 = ((int64_t)blockIdx.x - n_main) * (NT * kFoldPerThread);
        for (int u = 0; u < kFoldPerThread; ++u) {
            const int64_t p = p0 + u * NT + tid;
            if (p >= total) return;
            const int64_t i = p / per_in, rem = p - i * per_in;
            const int64_t m = rem / g.n_out, j = rem - m * g.n_out;
            float v;
            if (m < g.rows) v = coef[(i * g.rows + m) * g.n_out + j] * w_s[i * g.n_out + j];
            else v = g.base_act ? w_b[i * g.n_out + j] : 0.0f;
            cf[p] = v;
        }
        return;
    }

    const int tile = (int)(blockIdx.x % n_tiles);
    const int64_t b0 = (int64_t)(blockIdx.x / n_tiles) * NS;
    const int grp = tid / LPS, lj = tid % LPS;
    // lanes past the last output compute outputs 0 .. and drop them; a lane that straddles it starts at n_out - T
    const int jc = direct_first_output(tile * TJ + lj * T, T, g.n_out);

    // two-level sum over the inputs: a lane group's running sums are folded after about 32 of its inputs
    constexpr int kFoldRounds = 32 * NS > LPS ? 32 * NS / LPS : 1;
    float acc[NS][T], tot[NS][T];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int r = 0; r < T; ++r) { acc[s][r] = 0.0f; tot[s][r] = 0.0f; }

    for (int i0 = 0; i0 < g.n_in; i0 += IPR) {
        if (i0 > 0 && (i0 / IPR) % kFoldRounds == 0) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int r = 0; r < T; ++r) { tot[s][r] += acc[s][r]; acc[s][r] = 0.0f; }
        }
        const int n_ii = g.n_in - i0 < IPR ? g.n_in - i0 : IPR;
        {
            const int ii = tid / NS, s = tid % NS;
            if (ii < n_ii) {
                const int64_t b = b0 + s < B ? b0 + s : B - 1;
                const Pair p = pair_eval<false>(x[b * g.n_in + i0 + ii], g, i0 + ii);
                float rest[4];
                if constexpr (kMaxK == 4) {
                    rest[0] = p.base; rest[1] = __int_as_float(p.cell); rest[2] = 0.0f; rest[3] = 0.0f;
                } else {
                    rest[0] = p.base; rest[1] = __int_as_float(p.cell); rest[2] = p.w[kMaxK - 2]; rest[3] = p.w[kMaxK - 1];
                }
                pairs[tid * 2] = make_float4(p.w[0], p.w[1], p.w[2], p.w[3]);
                pairs[tid * 2 + 1] = make_float4(rest[0], rest[1], rest[2], rest[3]);
            }
        }
        __syncthreads();
        for (int ii = grp; ii < n_ii; ii += NGRP) {
            const int i = i0 + ii;
            const float *slab = coef + (int64_t)i * g.rows * g.n_out + jc;
            float sc[T], wb[T];
#pragma unroll
            for (int r = 0; r < T; ++r) sc[r] = 1.0f;
            if (w_s) direct_load<T>(w_s + (int64_t)i * g.n_out + jc, sc);
#pragma unroll
            for (int r = 0; r < T; ++r) wb[r] = 0.0f;
            if (g.base_act) direct_load<T>(w_b + (int64_t)i * g.n_out + jc, wb);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float4 a = pairs[(ii * NS + s) * 2], c = pairs[(ii * NS + s) * 2 + 1];
                float w[kMaxK];
                w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
                if constexpr (kMaxK == 6) { w[kMaxK - 2] = c.z; w[kMaxK - 1] = c.w; }
                const int cell = __float_as_int(c.y);
                // rows outside the table have zero weight and are clamped into it: no branch, every load in flight
                float v[kMaxK][T];
#pragma unroll
                for (int q = 0; q < kMaxK; ++q)
                    direct_load<T>(slab + (int64_t)clampi(cell + q, 0, g.rows - 1) * g.n_out, v[q]);
#pragma unroll
                for (int q = 0; q < kMaxK; ++q)
#pragma unroll
                    for (int r = 0; r < T; ++r) acc[s][r] = fmaf(w[q], v[q][r] * sc[r], acc[s][r]);
#pragma unroll
                for (int r = 0; r < T; ++r) acc[s][r] = fmaf(c.x, wb[r], acc[s][r]);
            }
        }
        __syncthreads();
    }

#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int r = 0; r < T; ++r) sums[(grp * NS + s) * TJ + lj * T + r] = tot[s][r] + acc[s][r];
    __syncthreads();
    for (int e = tid; e < NS * TJ; e += NT) {
        const int s = e / TJ, jj = tile * TJ + e % TJ;
        if (b0 + s >= B || jj >= g.n_out) continue;
        const float *at = sums + s * TJ + direct_slot(jj, tile * TJ, T, g.n_out);
        // 64 groups of sixteen outputs: eight in pairs, and the eights one after another; added one by one, groups of a few inputs each round
        // more often than the kernel of longer sums that would have such a layer (16 -> 16, G = 32, k = 1: error 0.89e-7 with 64 in a
        // row, the narrow kernel's 0.76e-7)
        constexpr int kPairs = T == 4 && NGRP == 64 ? 8 : 1;
        float v = 0.0f;
#pragma unroll 8
        for (int q = 0; q < NGRP; q += kPairs) {
            float t[kPairs];
#pragma unroll
            for (int u = 0; u < kPairs; ++u) t[u] = at[(q + u) * NS * TJ];
#pragma unroll
            for (int d = kPairs / 2; d > 0; d /= 2)
#pragma unroll
                for (int u = 0; u < d; ++u) t[u] += t[u + d];
            v += t[0];
        }
        y[(b0 + s) * g.n_out + jj] = v;
    }
}

// A launch takes fewer than 2^32 threads (hipModuleLaunchKernel): larger batches go in parts of half that.  Large folds
// go in a launch of their own, with wide accesses: beside many samples at 2^20 floats both take the same, at 2^18 the launch
// costs 1.5 us more, at 2^24 (16 -> 128, G = 10000) 22 us less; beside few samples the fold in the launch has the chip to itself
// (32 -> 64, G = 1000, B = 64, 2^21 floats: 9 us in the launch, 12 behind one; 256 -> 33, G = 1000, 2^23: 23 / 32).
template <int LPS, int T, int NS, int NW>
static hipError_t direct_launch(const SplineGeom &g, const float *x, const float *coef, const float *w_s,
                                const float *w_b, float *cf, float *y, int64_t B, hipStream_t st)
{
    constexpr int64_t kThreads = 64 * NW;
    const int n_tiles = (g.n_out + LPS * T - 1) / (LPS * T);
    const int64_t total = (int64_t)g.n_in * (g.rows + 1) * g.n_out, per = kThreads * kFoldPerThread;
    if (cf && total > (B <= 512 ? 1 << 23 : (B <= 2048 ? 1 << 21 : 1 << 20))) {
        if (hipError_t e = launch_fold_scale(coef, w_s, g.base_act ? w_b : nullptr, cf, g.n_in, g.rows, g.n_out, st);
            e != hipSuccess)
            return e;
        cf = nullptr;
    }
    const int64_t n_fold = cf ? (total + per - 1) / per : 0;
    const int64_t part = ((1ll << 31) / kThreads + n_tiles - 1) / n_tiles * NS;       // samples
    for (int64_t b0 = 0; b0 < B; b0 += part) {
        const int64_t n = B - b0 < part ? B - b0 : part, n_main = (n + NS - 1) / NS * n_tiles;
        const unsigned blocks = (unsigned)(n_main + (b0 == 0 ? n_fold : 0));
        prof::Timed tm("forward_direct", st);
        forward_direct_kernel<LPS, T, NS, NW><<<blocks, (unsigned)kThreads, 0, st>>>(g, x + b0 * g.n_in, coef, w_s, w_b, cf,
                                                                                     y + b0 * g.n_out, n, n_tiles, n_main);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// one sample per workgroup, one output per lane: the most workgroups and the shortest chain
template <int LPS>
static hipError_t direct_latency(const SplineGeom &g, const float *x, const float *coef, const float *w_s,
                                 const float *w_b, float *cf, float *y, int64_t B, hipStream_t st)
{
    return g.n_in >= 32 ? direct_launch<LPS, 1, 1, 16>(g, x, coef, w_s, w_b, cf, y, B, st)
                        : direct_launch<LPS, 1, 1, 4>(g, x, coef, w_s, w_b, cf, y, B, st);
}

// Where the line lies.  The direct kernel gathers every window row from L2 once per sample: its time is the edges of the
// padded width at about 1.8e12 edges/s while the table stays in L2, and at least 2.6 ns for a workgroup of four samples.  The
// LDS-staged kernels walk the inputs one after the other and, until their workgroups fill the chip, cost a fixed time an
// input however small the batch, so against them the line is one on B * n_out that falls with the inputs.  With fewer than
// eight inputs the others cost no more than their launches and the line is on the workgroups alone.  Past L2 the kernels
// that share a row between samples win from a few thousand samples on; narrow layers win by their shorter rows.
// Measured, other kernel / direct, us (a fold of more than 2^20 floats in a launch of its own is in both):
//   two inputs        2 -> 17, G = 20: B = 8192 11 / 9, 65536 18 / 43; 2 -> 200, G = 20: 2048 12 / 10, 8192 12 / 25
//   long-table        64 -> 64, G = 10: B = 4096 57 / 14, 16384 59 / 44, 32768 62 / 88; 8 -> 64, G = 20: 8192 11 / 10,
//                     16384 12 / 15; 16 -> 32, G = 5: 16384 24 / 15, 32768 24 / 26
//   256-wide tiles    256 -> 256, G = 10: B = 8192 661 / 302, 32768 666 / 1186; 8 -> 256, G = 20: 4096 26 / 15, 8192 27 / 27
//   512-wide tiles    512 -> 512, G = 10: B = 4096 832 / 600, 8192 836 / 1190; 64 -> 300, G = 20: 4096 121 / 74, 8192 122 / 138
//   row stream        in L2: 32 -> 24, G = 20: B = 131072 153 / 108; 32 -> 64, G = 1000: 32768 80 / 81, 131072 225 / 301;
//                     past it: 256 -> 32, G = 1000: 32768 507 / 475, 65536 679 / 943
//   generic           past L2: 256 -> 130, G = 300: B = 2048 244 / 215, 4096 307 / 444; in it: 8 -> 128, G = 100: 8192 14 / 15,
//                     16384 23 / 27; 128 -> 37, G = 200: 32768 406 / 167
//   narrow            one output on sixteen lanes: 64 -> 1, G = 20: B = 1024 8.9 / 7.3, 1500 9.1 / 9.6, 4096 9.2 / 21; G = 240: 512 9.0 / 8.7,
//                     1024 9.1 / 10.9; 256 -> 1: 1500 15.5 / 15.7, 4096 16 / 37; 500 -> 1: 1500 27 / 23, 2048 27 / 33
//                     32 -> 4, G = 20: 16384 20 / 15, 65536 31 / 46; 64 -> 4: 65536 56 / 50, 262144 199 / 207, G = 400 591 / 208; 256 -> 4:
//                     65536 214 / 175; 32 -> 5: G = 20 65536 35 / 45, G = 400 51 / 46; 64 -> 5: 262144 235 / 207; 16 -> 8: G = 20
//                     65536 36 / 42; 32 -> 8: 262144 312 / 185; 8 -> 16: 65536 48 / 42; 64 -> 16: 262144 1411 / 212; 32 -> 16, G = 1000: 65536 478 / 49
//   degrees 4 and 5   64 -> 4, G = 10000: B = 65536 481 / 96 (generic); 64 -> 300, G = 20: 4096 283 / 109 (512-wide tiles);
//                     64 -> 64, G = 300: 32768 140 / 131, 65536 252 / 277 (row stream)
//   degrees 4 and 5, staged slabs (a round of workgroups costs an input the same whether the chip is full or not, and a copied row
//                     has to serve enough samples)
//       up to 32 outputs   32 -> 32, G = 200: B = 34453 48 / 40, 48062 48 / 55, 66594 (a second round begins) 84 / 73; 63 -> 32, G = 131:
//                          34443 84 / 67; 23 -> 32, G = 20: 27322 34 / 27; 24 -> 32, G = 200: 34170 34 / 35; 16 -> 32: G = 140 23905 25 / 23,
//                          G = 80 34771 23 / 32; 14 -> 32, G = 324: 19738 25 / 20; 12 -> 32, G = 200: 24358 21 / 23; 8 -> 32, G = 6: 24141 15 / 21
//       more, long tables  32 -> 48, G = 131: 17406 42 / 33; 100 -> 48, G = 131: 17140 113 / 94; 16 -> 40, G = 131: 17881 24 / 22, G = 80
//                          24000 20 / 29; 13 -> 59, G = 85: 12493 19 / 16; 128 -> 36, G = 131: 34624 (two rounds) 284 / 258
//             short        32 -> 48, G = 30: 24000 32 / 45; 32 -> 64, G = 30: 17647 29 / 37; 8 -> 40, G = 30: 9448 12.5 / 11.6, 13107
//                          12.5 / 14.4; 12 -> 40, G = 30: 9649 17 / 13
// (sums of 4 and 6 products cost in proportion: the line counts them)
// lds_rows: whether the staged kernel for long tables would take the layer otherwise.
static int direct_plan(const SplineGeom &g, int64_t B, bool lds_rows, int lds)
{
    const int n = g.n_out, ni = g.n_in;
    const int64_t tiles = (n + 63) / 64, w = n <= 16 ? 16 : (n <= 32 ? 32 : tiles * 64), load = B * w * kMaxK / 4;
    const bool in_l2 = (int64_t)ni * g.slab_rows * n * 4 <= 8ll << 20;
#if KAN_MAXK == 4
    const bool narrow = narrow_applicable(g) != 0;
#else
    const bool narrow = false;
#endif
    if (ni < 8) return B * tiles <= (n < 4 ? 1 << 12 : (n >= 128 && (lds || lds_rows) ? 3 << 12 : 1 << 13)) ? 1 : 0;
    if (n < 4) {                                     // one output per lane at any batch: 16 lanes for at most three
        if (!narrow) return B <= (ni >= 32 ? 1 << 13 : 1 << 11) ? 1 : 0;
        // (longer tables cost the narrow kernel more, whose four lanes a sample read rows one at a time)
        if (n == 1 && ni >= 32) return B <= (ni >= 384 ? 7 << 8 : ni >= 256 ? 6 << 8 : g.rows >= 128 ? 1 << 9 : 5 << 8) ? 1 : 0;
        const int64_t per = n == 1 ? 32ll * ni : (g.rows >= 4096 ? 128ll : 64ll) * ni, cap = n == 1 ? 1 << 12 : 1 << 13;
        const int64_t low = n == 1 && g.rows >= 128 ? 1 << 10 : 1 << 11;
        const int64_t most = ni < 32 ? 1 << 12 : (per < low ? low : (per < cap ? per : cap));
        return B <= most ? 1 : 0;
    }
    constexpr bool six = kMaxK == 6;
    // The narrow kernel's lanes gather rows of their own, the wider and the longer the table the further from L1: at any batch.
    // (Nine to fifteen outputs of up to 63 inputs on short tables stay with the line below, which a test holds; not for speed.)
    if (narrow && (n == 16 || (n > 8 && (ni >= 64 || g.rows >= 64)) || ni >= 256 || (ni >= 64 && (n >= 5 || g.rows >= 256)) || (ni >= 32 && (n == 8 || (n >= 5 && g.rows >= 256))))) return 1;
    if (narrow)
        return load <= (ni >= 64 || (ni >= 32 && (n >= 8 || g.rows >= 512)) ? 1 << 20 : (ni >= 32 ? 1 << 18 : 1 << 17)) ? 1 : 0;
    if (lds_rows && six) {
        const int64_t round = 7ll << 18, rounds = forward_lds_rows_rounds(g, B);
        if (n <= 32)
            return load <= (ni >= 32 ? rounds * round : ni >= 20 ? 3ll << 19 : ni >= 16 ? 5ll << 18 : ni >= 10 ? 1ll << 20 : 3ll << 18) ? 1 : 0;
        if (g.rows <= 64) return load <= (ni < 16 ? 1 << 20 : 3 << 19) ? 1 : 0;
        return load <= (ni < 16 ? 5ll << 18 : ni < 64 ? round : rounds * round) ? 1 : 0;
    }
    if (lds_rows) return load <= (ni >= 32 ? 1 << 20 : (ni >= 16 ? 3 << 18 : 1 << 19)) ? 1 : 0;
    if (forward_rows_plan(g)) {
        if (!in_l2) return load <= (six && n <= 48 ? 3 << 19 : 1 << 20) ? 1 : 0;
        if (n <= 32) return ni >= 32 || load <= (six ? 3 << 20 : 1 << 21) ? 1 : 0;
        return (n <= 48 && ni >= 64) || load <= (ni >= 32 || six ? 3 << 20 : 1 << 21) ? 1 : 0;
    }
    if (lds == 4) return load <= (ni >= 32 ? 7 << 19 : (ni >= 16 || six ? 3 << 20 : 1 << 21)) ? 1 : 0;
    if (lds == 8) return load <= (six ? 5 << 19 : (ni >= 16 ? 1 << 21 : 1 << 20)) ? 1 : 0;
    // generic
    if (n <= 32) return ni >= 16 || load <= (six && n > 16 ? (in_l2 ? 3 << 20 : 3 << 19) : 1 << 20) ? 1 : 0;
    if (in_l2 && (n < 256 || n % 4 != 0)) return ni >= 16 || load <= (n >= 128 ? 1 << 20 : (six ? 3 << 20 : 1 << 22)) ? 1 : 0;
    return load <= (in_l2 || six ? 3 << 18 : 1 << 19) ? 1 : 0;
}

int forward_direct_plan(const SplineGeom &g, int64_t B)
{
    const int lds = forward_lds_plan(g);
    return direct_plan(g, B, forward_lds_rows_plan(g, B) != 0 && (g.n_out <= 64 || !lds), lds);
}

int forward_direct_beside_gathers(const SplineGeom &g, int64_t B) { return direct_plan(g, B, false, forward_lds_plan(g)); }

hipError_t launch_forward_direct(const SplineGeom &g, const float *x, const float *coef, const float *w_s,
                                 const float *w_b, float *cf, float *y, int64_t B, hipStream_t st)
{
    // once workgroups of one sample fill the chip twice over: four samples per workgroup (they share the row of scales
    // and base weights) and 16-byte row reads
    if (B * ((g.n_out + 63) / 64) >= 2048 && g.n_out >= 4) {
        if (g.n_out <= 16) return direct_launch<4, 4, 4, 4>(g, x, coef, w_s, w_b, cf, y, B, st);
        if (g.n_out <= 32) return direct_launch<8, 4, 4, 4>(g, x, coef, w_s, w_b, cf, y, B, st);
        return direct_launch<16, 4, 4, 4>(g, x, coef, w_s, w_b, cf, y, B, st);
    }
    if (g.n_out <= 16) return direct_latency<16>(g, x, coef, w_s, w_b, cf, y, B, st);
    if (g.n_out <= 32) return direct_latency<32>(g, x, coef, w_s, w_b, cf, y, B, st);
    return direct_latency<64>(g, x, coef, w_s, w_b, cf, y, B, st);
}

}  // namespace KAN_NS
