// Generic kernels of the local B-spline layer: they work for every shape the
// library accepts (any n_in, n_out, grid size, per-input cell offsets; degrees up to
// kMaxK - 1: 3 in the default build, 5 in the build of kan_generic_k5.hip) and are the
// fallback when no specialised kernel applies.
//
// Common mapping: lanes <-> outputs.  One wave owns T samples and a tile of
// 64*R outputs; the per-(sample, input) quantities (cell, window weights, base
// value) are wave-uniform, evaluated 64 pairs at a time with one pair per lane
// and then broadcast lane by lane into scalar registers, so the per-edge work is
// K multiply-adds whose coefficient operands are unit-stride across lanes.
#include "kan_device.hpp"
#include "kan_launch.hpp"

namespace KAN_NS {

// ---- helpers --------------------------------------------------------------

template <int R> struct VecOf;
template <> struct VecOf<1> { using type = float; };
template <> struct VecOf<2> { using type = float2; };
template <> struct VecOf<4> { using type = float4; };

template <int R>
__device__ __forceinline__ void load_vec(const float *p, float (&v)[R])
{
    if constexpr (R == 1) {
        v[0] = *p;
    } else if constexpr (R == 2) {
        float2 t = *reinterpret_cast<const float2 *>(p);
        v[0] = t.x; v[1] = t.y;
    } else {
        float4 t = *reinterpret_cast<const float4 *>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
}

template <int R>
__device__ __forceinline__ void store_vec(float *p, const float (&v)[R])
{
    if constexpr (R == 1) {
        *p = v[0];
    } else if constexpr (R == 2) {
        *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    } else {
        *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// ---- interval index export --------------------------------------------------

__global__ void interval_index_kernel(const float *__restrict__ x, int32_t *__restrict__ idx, int64_t n,
                                      float lo, float inv_h)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) {
        float t, d;
        idx[p] = interval_index(x[p], lo, inv_h, &t, &d);
    }
}

// ---- fold the per-edge spline scale into the coefficients -------------------
// cf[i][m][j] = w_s[i][j] * coef[i][m][j] for m < rows, and cf[i][rows][j] = w_b[i][j] (zero without
// a base term): afterwards the spline term costs K multiply-adds per edge with no separate scale,
// and one input's operands are one contiguous (rows + 1) x n_out block.
// grid (parts of an input's block, n_in), V floats a thread and access (V divides n_out).  Bound by the copy:
// 512 -> 512, G = 20: 20 -> 13 us against a flat index with two 64-bit divisions an element.
template <int V>
__global__ __launch_bounds__(256) void fold_scale_kernel(const float *__restrict__ coef, const float *__restrict__ w_s,
                                                         const float *__restrict__ w_b, float *__restrict__ cf, int rows,
                                                         int n_out)
{
    const unsigned i = blockIdx.y, per_row = (unsigned)n_out / V, total = (unsigned)(rows + 1) * per_row;
    const float *src = coef + (int64_t)i * rows * n_out, *sc = w_s + (int64_t)i * n_out;
    const float *wb = w_b ? w_b + (int64_t)i * n_out : nullptr;
    float *dst = cf + (int64_t)i * (rows + 1) * n_out;
    const unsigned e = blockIdx.x * 256u + threadIdx.x;
    if (e >= total) return;
    const unsigned m = e / per_row, j = (e - m * per_row) * V;
    if constexpr (V == 4) {
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (m < (unsigned)rows) {
            const float4 c = *reinterpret_cast<const float4 *>(src + (int64_t)e * 4), s = *reinterpret_cast<const float4 *>(sc + j);
            v = make_float4(c.x * s.x, c.y * s.y, c.z * s.z, c.w * s.w);
        } else if (wb) {
            v = *reinterpret_cast<const float4 *>(wb + j);
        }
        *reinterpret_cast<float4 *>(dst + (int64_t)e * 4) = v;
    } else {
        dst[e] = m < (unsigned)rows ? src[e] * sc[j] : (wb ? wb[j] : 0.0f);
    }
}

// ---- forward ---------------------------------------------------------------
// grid.x = batch tiles of 4*T samples, grid.y = output tiles of 64*R.
template <int R, int T>
__global__ __launch_bounds__(256) void forward_generic_kernel(SplineGeom g, const float *__restrict__ x,
                                                              const float *__restrict__ cf,
                                                              const float *__restrict__ w_b,
                                                              float *__restrict__ y, int64_t B)
{
    constexpr int IPV = kWave / T;      // inputs covered by one vector evaluation
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t b0 = ((int64_t)blockIdx.x * 4 + wave) * T;
    if (b0 >= B) return;                // whole wave out of range (uniform)
    const int j = blockIdx.y * (kWave * R) + lane * R;
    const bool j_ok = j < g.n_out;      // n_out is a multiple of R
    const int jc = j_ok ? j : 0;

    // two-level sum over the inputs: `acc` collects kFoldInputs inputs, then is folded into
    // `tot`; keeps the rounding error of a long fp32 sum well inside the tolerance
    constexpr int kFoldInputs = 32;
    float acc[T][R], tot[T][R];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < R; ++r) { acc[t][r] = 0.0f; tot[t][r] = 0.0f; }

    const int my_t = lane % T, my_ii = lane / T;
    const int64_t my_b = (b0 + my_t < B) ? b0 + my_t : B - 1;

    for (int i0 = 0; i0 < g.n_in; i0 += IPV) {
        if (i0 % kFoldInputs == 0 && i0 > 0) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < R; ++r) { tot[t][r] += acc[t][r]; acc[t][r] = 0.0f; }
        }
        const int my_i = i0 + my_ii;
        const bool i_ok = my_i < g.n_in;
        const int ic = i_ok ? my_i : g.n_in - 1;
        Pair p = pair_eval<false>(x[my_b * g.n_in + ic], g, ic);
        if (!i_ok) { p.cell = -kMaxK; p.base = 0.0f; }

        const int n_ii = (g.n_in - i0 < IPV) ? g.n_in - i0 : IPV;
        for (int ii = 0; ii < n_ii; ++ii) {
            const float *slab = cf + (int64_t)(i0 + ii) * g.slab_rows * g.n_out + jc;
            float wb[R];
#pragma unroll
            for (int r = 0; r < R; ++r) wb[r] = 0.0f;
            if (g.base_act) load_vec<R>(w_b + (int64_t)(i0 + ii) * g.n_out + jc, wb);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int src = ii * T + t;
                // no branch on "window outside the table": those weights are zero and the rows are
                // clamped, so the loads of all T samples can be in flight together
                const int cell = lane_i(p.cell, src);
                float c[kMaxK][R];
#pragma unroll
                for (int s = 0; s < kMaxK; ++s)
                    load_vec<R>(slab + (int64_t)clampi(cell + s, 0, g.rows - 1) * g.n_out, c[s]);
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) {
                    const float ws = lane_f(p.w[s], src);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[t][r] = fmaf(ws, c[s][r], acc[t][r]);
                }
                if (g.base_act) {
                    const float bs = lane_f(p.base, src);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[t][r] = fmaf(bs, wb[r], acc[t][r]);
                }
            }
        }
    }
    if (j_ok) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
#pragma unroll
            for (int r = 0; r < R; ++r) tot[t][r] += acc[t][r];
            if (b0 + t < B) store_vec<R>(y + (b0 + t) * g.n_out + j, tot[t]);
        }
    }
}

// ---- backward: dL/dx ---------------------------------------------------------
// One wave owns T samples and walks over every output tile; per pair it forms the
// per-lane partial  q = sum_r gy_r * (sum_s dw_s * cf_s[r] + dbase * w_b[r])  and the
// 64 partial vectors of one evaluation round are reduced together by a butterfly
// that ends with lane p holding the total of pair p, which is the lane that
// evaluated the pair and now stores gx for it.
template <int N>
__device__ __forceinline__ void butterfly_step(float (&q)[kWave], int lane)
{
    // q[0..2N) -> q[0..N): lanes with bit N clear keep the low half, the others the high half
    const bool up = (lane & N) != 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        float keep = up ? q[m + N] : q[m];
        float send = up ? q[m] : q[m + N];
        q[m] = keep + __shfl_xor(send, N, kWave);
    }
}

template <int R, int T>
__global__ __launch_bounds__(256) void dx_generic_kernel(SplineGeom g, const float *__restrict__ x,
                                                         const float *__restrict__ cf,
                                                         const float *__restrict__ w_b,
                                                         const float *__restrict__ gy,
                                                         float *__restrict__ gx, int64_t B)
{
    constexpr int IPV = kWave / T;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t b0 = ((int64_t)blockIdx.x * 4 + wave) * T;
    if (b0 >= B) return;
    const int my_t = lane % T, my_ii = lane / T;
    const int64_t my_b = (b0 + my_t < B) ? b0 + my_t : B - 1;
    const int n_jt = (g.n_out + kWave * R - 1) / (kWave * R);

    for (int i0 = 0; i0 < g.n_in; i0 += IPV) {
        const int my_i = i0 + my_ii;
        const bool i_ok = my_i < g.n_in;
        const int ic = i_ok ? my_i : g.n_in - 1;
        Pair p = pair_eval<true>(x[my_b * g.n_in + ic], g, ic);
        if (!i_ok) { p.cell = -kMaxK; p.dbase = 0.0f; }

        float q[kWave];
#pragma unroll
        for (int m = 0; m < kWave; ++m) q[m] = 0.0f;

        for (int jt = 0; jt < n_jt; ++jt) {
            const int j = jt * (kWave * R) + lane * R;
            const bool j_ok = j < g.n_out;
            const int jc = j_ok ? j : 0;
            float gyv[T][R];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int64_t b = (b0 + t < B) ? b0 + t : B - 1;
                load_vec<R>(gy + b * g.n_out + jc, gyv[t]);
                if (!j_ok) {
#pragma unroll
                    for (int r = 0; r < R; ++r) gyv[t][r] = 0.0f;
                }
            }
#pragma unroll
            for (int ii = 0; ii < IPV; ++ii) {
                if (i0 + ii < g.n_in) {
                    const float *slab = cf + (int64_t)(i0 + ii) * g.slab_rows * g.n_out + jc;
                    float wb[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) wb[r] = 0.0f;
                    if (g.base_act) load_vec<R>(w_b + (int64_t)(i0 + ii) * g.n_out + jc, wb);
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const int src = ii * T + t;
                        const int cell = lane_i(p.cell, src);
                        float d[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) d[r] = 0.0f;
                        if (cell > -kMaxK && cell < g.rows) {
                            float c[kMaxK][R];
#pragma unroll
                            for (int s = 0; s < kMaxK; ++s)
                                load_vec<R>(slab + (int64_t)clampi(cell + s, 0, g.rows - 1) * g.n_out, c[s]);
#pragma unroll
                            for (int s = 0; s < kMaxK; ++s) {
                                const float dws = lane_f(p.dw[s], src);
#pragma unroll
                                for (int r = 0; r < R; ++r) d[r] = fmaf(dws, c[s][r], d[r]);
                            }
                        }
                        if (g.base_act) {
                            const float dbs = lane_f(p.dbase, src);
#pragma unroll
                            for (int r = 0; r < R; ++r) d[r] = fmaf(dbs, wb[r], d[r]);
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) q[src] = fmaf(gyv[t][r], d[r], q[src]);
                    }
                }
            }
        }
        butterfly_step<32>(q, lane);
        butterfly_step<16>(q, lane);
        butterfly_step<8>(q, lane);
        butterfly_step<4>(q, lane);
        butterfly_step<2>(q, lane);
        butterfly_step<1>(q, lane);
        if (i_ok && b0 + my_t < B) gx[(b0 + my_t) * g.n_in + my_i] = q[0];
    }
}

// ---- backward: parameter gradients -------------------------------------------
// Stage 1.  One wave owns input i, a tile of 64*R outputs, one block of kRowBlock coefficient rows
// and one chunk of the batch, and keeps
//   acc[m][j] = sum_{b in chunk} gy[b][j] * N_{m - cell(b,i)}(u(b,i))      (m in its row block)
// in LDS that only this wave touches.  Samples are visited in index order and every row has exactly
// one owner, so the sum order is fixed.  Samples whose window misses the row block are skipped with
// a scalar test, which is what keeps large grids cheap: the LDS footprint per wave is a row block,
// not the whole slab, so many waves fit on a CU.  The raw sums go to part_c[chunk][i][m][j]; the
// base-term sums  sum_b gy[b][j] * silu(x[b][i])  are taken by the block that owns the sample's
// clamped cell and go to part_b[chunk * n_row_blocks + block][i][j].
constexpr int kRowBlock = 16;

template <int R>
__global__ __launch_bounds__(64) void dparam_generic_kernel(SplineGeom g, const float *__restrict__ x,
                                                            const float *__restrict__ gy,
                                                            float *__restrict__ part_c,
                                                            float *__restrict__ part_b, int64_t B,
                                                            int64_t chunk_len, int n_jt)
{
    constexpr int TJ = kWave * R;
    __shared__ float acc[kRowBlock * TJ];
    const int lane = threadIdx.x;
    // grid.x carries (row block, output tile): it may exceed the 65535 limit of grid.y for long tables
    const int i = blockIdx.y;
    const int jt = blockIdx.x % n_jt, rb = blockIdx.x / n_jt;
    const int n_rb = gridDim.x / n_jt;
    const int lo = rb * kRowBlock;
    const int hi = (lo + kRowBlock < g.rows) ? lo + kRowBlock : g.rows;
    const int j = jt * TJ + lane * R;
    const bool j_ok = j < g.n_out;
    const int jc = j_ok ? j : 0;
    const int64_t b_lo = (int64_t)blockIdx.z * chunk_len;
    const int64_t b_hi = (b_lo + chunk_len < B) ? b_lo + chunk_len : B;

    for (int m = 0; m < kRowBlock; ++m)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[m * TJ + lane * R + r] = 0.0f;
    // the base sums go in two levels (accb is folded into accb_hi every 256 samples) so that a chunk of a
    // thousand O(1) terms keeps fp32 accuracy
    float accb[R], accb_hi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { accb[r] = 0.0f; accb_hi[r] = 0.0f; }

    for (int64_t b0 = b_lo; b0 < b_hi; b0 += kWave) {
        if (((b0 - b_lo) & 255) == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) { accb_hi[r] += accb[r]; accb[r] = 0.0f; }
        }
        const int64_t my_b = (b0 + lane < b_hi) ? b0 + lane : b_hi - 1;
        Pair p = pair_eval<false>(x[my_b * g.n_in + i], g, i);
        const int n_b = (b_hi - b0 < kWave) ? (int)(b_hi - b0) : kWave;
        for (int t = 0; t < n_b; ++t) {
            const int cell = lane_i(p.cell, t);
            const int owner = clampi(cell, 0, g.rows - 1);
            const bool touches = cell + kMaxK > lo && cell < hi;
            const bool owns = owner >= lo && owner < hi;
            if (!(touches || (owns && part_b))) continue;          // uniform
            float gv[R];
            load_vec<R>(gy + (b0 + t) * g.n_out + jc, gv);
            if (touches) {
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) {
                    const int m = cell + s;
                    if (m >= lo && m < hi) {                        // uniform
                        const float ws = lane_f(p.w[s], t);
                        float *row = acc + (m - lo) * TJ + lane * R;
#pragma unroll
                        for (int r = 0; r < R; ++r) row[r] = fmaf(ws, gv[r], row[r]);
                    }
                }
            }
            if (owns && part_b) {
                const float bs = lane_f(p.base, t);
#pragma unroll
                for (int r = 0; r < R; ++r) accb[r] = fmaf(bs, gv[r], accb[r]);
            }
        }
    }
    if (!j_ok) return;
    float *pc = part_c + ((int64_t)blockIdx.z * g.n_in + i) * g.rows * g.n_out + j;
    for (int m = lo; m < hi; ++m) {
        float a[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = acc[(m - lo) * TJ + lane * R + r];
        store_vec<R>(pc + (int64_t)m * g.n_out, a);
    }
    if (part_b) {
#pragma unroll
        for (int r = 0; r < R; ++r) accb[r] += accb_hi[r];
        store_vec<R>(part_b + (((int64_t)blockIdx.z * n_rb + rb) * g.n_in + i) * g.n_out + j, accb);
    }
}

// Stage 2, the sum over the chunks, is kan_reduce.hip.

// ---- launchers -------------------------------------------------------------

static int pick_r(int n_out)
{
    if (n_out % 4 == 0 && n_out >= 256) return 4;
    if (n_out % 2 == 0 && n_out >= 128) return 2;
    return 1;
}

hipError_t launch_interval_index(const float *x, int32_t *idx, int64_t n, float lo, float inv_h,
                                 hipStream_t st)
{
    if (n == 0) return hipSuccess;
    unsigned blocks = (unsigned)((n + 255) / 256);
    prof::Timed tm("interval_index", st);
    interval_index_kernel<<<blocks, 256, 0, st>>>(x, idx, n, lo, inv_h);
    return hipGetLastError();
}

hipError_t launch_fold_scale(const float *coef, const float *w_s, const float *w_b, float *cf, int n_in, int rows,
                             int n_out, hipStream_t st)
{
    const int V = n_out % 4 == 0 ? 4 : 1;
    const int64_t per = (int64_t)(rows + 1) * (n_out / V);
    const dim3 grid((unsigned)((per + 255) / 256), (unsigned)n_in);
    prof::Timed tm("fold_scale", st);
    if (V == 4) fold_scale_kernel<4><<<grid, 256, 0, st>>>(coef, w_s, w_b, cf, rows, n_out);
    else fold_scale_kernel<1><<<grid, 256, 0, st>>>(coef, w_s, w_b, cf, rows, n_out);
    return hipGetLastError();
}

template <int R, int T>
static hipError_t forward_rt(const SplineGeom &g, const float *x, const float *cf, const float *w_b, float *y,
                             int64_t B, hipStream_t st)
{
    dim3 grid((unsigned)((B + 4 * T - 1) / (4 * T)), (unsigned)((g.n_out + 64 * R - 1) / (64 * R)));
    prof::Timed tm("forward_generic", st);
    forward_generic_kernel<R, T><<<grid, 256, 0, st>>>(g, x, cf, w_b, y, B);
    return hipGetLastError();
}

// samples per wave: as many as still leave the chip about four waves per SIMD (the kernel lives on
// loads in flight), between 2 and 8 (16 for the one- and two-output-per-lane variants)
template <int R>
static hipError_t forward_r(const SplineGeom &g, const float *x, const float *cf, const float *w_b, float *y,
                            int64_t B, hipStream_t st)
{
    const int64_t tiles = (g.n_out + 64 * R - 1) / (64 * R);
    auto waves = [&](int t) { return (B + t - 1) / t * tiles; };
    if constexpr (R != 4) {
        if (waves(16) >= 4096) return forward_rt<R, 16>(g, x, cf, w_b, y, B, st);
    }
    if (waves(8) >= 4096) return forward_rt<R, 8>(g, x, cf, w_b, y, B, st);
    if (waves(4) >= 4096) return forward_rt<R, 4>(g, x, cf, w_b, y, B, st);
    return forward_rt<R, 2>(g, x, cf, w_b, y, B, st);
}

hipError_t launch_forward_generic(const SplineGeom &g, const float *x, const float *cf, const float *w_b,
                                  float *y, int64_t B, hipStream_t st)
{
    switch (pick_r(g.n_out)) {
    case 4: return forward_r<4>(g, x, cf, w_b, y, B, st);
    case 2: return forward_r<2>(g, x, cf, w_b, y, B, st);
    default: return forward_r<1>(g, x, cf, w_b, y, B, st);
    }
}

template <int R>
static hipError_t dx_r(const SplineGeom &g, const float *x, const float *cf, const float *w_b, const float *gy,
                       float *gx, int64_t B, hipStream_t st)
{
    constexpr int T = 8;
    dim3 grid((unsigned)((B + 4 * T - 1) / (4 * T)));
    prof::Timed tm("dx_generic", st);
    dx_generic_kernel<R, T><<<grid, 256, 0, st>>>(g, x, cf, w_b, gy, gx, B);
    return hipGetLastError();
}

hipError_t launch_dx_generic(const SplineGeom &g, const float *x, const float *cf, const float *w_b,
                             const float *gy, float *gx, int64_t B, hipStream_t st)
{
    switch (pick_r(g.n_out)) {
    case 4: return dx_r<4>(g, x, cf, w_b, gy, gx, B, st);
    case 2: return dx_r<2>(g, x, cf, w_b, gy, gx, B, st);
    default: return dx_r<1>(g, x, cf, w_b, gy, gx, B, st);
    }
}

int dparam_generic_row_blocks(int rows) { return (rows + kRowBlock - 1) / kRowBlock; }

hipError_t launch_dparam_generic(const SplineGeom &g, const float *x, const float *gy, float *part_c,
                                 float *part_b, int64_t B, int n_chunks, int64_t chunk_len, hipStream_t st)
{
    const int R = pick_r(g.n_out);
    const int n_jt = (g.n_out + 64 * R - 1) / (64 * R);
    const int n_rb = dparam_generic_row_blocks(g.rows);
    if (g.n_in > 65535 || n_chunks > 65535) return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)(n_jt * n_rb), (unsigned)g.n_in, (unsigned)n_chunks);
    prof::Timed tm("dparam_generic", st);
    switch (R) {
    case 4: dparam_generic_kernel<4><<<grid, 64, 0, st>>>(g, x, gy, part_c, part_b, B, chunk_len, n_jt); break;
    case 2: dparam_generic_kernel<2><<<grid, 64, 0, st>>>(g, x, gy, part_c, part_b, B, chunk_len, n_jt); break;
    default: dparam_generic_kernel<1><<<grid, 64, 0, st>>>(g, x, gy, part_c, part_b, B, chunk_len, n_jt); break;
    }
    return hipGetLastError();
}

}  // namespace KAN_NS
