// Kernels for narrow layers (at most 16 outputs), e.g. the 5 -> 1 layer of a small KAN or the last
// layer of a regression stack.  With so few outputs the lanes <-> outputs mapping of the other
// kernels would leave most of a wave idle, so here lanes <-> samples (forward, dL/dx: every lane
// evaluates its own pair and gathers its own window; nothing is reduced across lanes).  The
// parameter gradients of narrow layers are taken by the chunk-sorted walk.
#include "kan_device.hpp"
#include "kan_launch.hpp"

namespace kan {

// ---- forward ------------------------------------------------------------------------------
// Q lanes per sample (four, or sixteen): lane q of the group takes inputs q, q + Q, ... and the partial sums are
// added across the group at the end (with one thread per sample a batch of a few ten thousand leaves
// most of the chip idle).
template <int NO, int Q>                         // Q = 16: NO = 1
__global__ __launch_bounds__(256) void forward_narrow_kernel(SplineGeom g, const float *__restrict__ x,
                                                             const float *__restrict__ cf,
                                                             const float *__restrict__ w_b, float *__restrict__ y,
                                                             int64_t B)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b = t / Q;
    const int q = (int)(t % Q);
    const int64_t bc = b < B ? b : B - 1;        // lanes past the batch recompute the last sample: groups stay whole
    float acc[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) acc[j] = 0.0f;
    float tot = 0.0f;                            // one output: folded every eight inputs, as the direct kernel's sums are short
    int n = 0;
    for (int i = q; i < g.n_in; i += Q) {
        Pair p = pair_basis<false>(x[bc * g.n_in + i], g, i);
        const float *slab = cf + (int64_t)i * g.slab_rows * g.n_out;
        // one output: a window is four neighbouring floats, one access (the lines looked up in L1 were the bound: 256 -> 1, 244 rows,
        // B = 32768 64 -> 49 us).  Where it hangs over an end of the table the access is moved back onto it and what it reads moved along,
        // so that other rows, whatever stands there, take no part (256 -> 1, G = 40, k = 1, B = 131072 101 us, row by row 145
        // and with four lanes a sample 121)
        if (NO == 1 && g.rows >= kMaxK) {
            const int c = clampi(p.cell, 0, g.rows - kMaxK), d = c - p.cell;
            const float4 r = load4u(slab + c);
            float v[kMaxK] = {r.x, r.y, r.z, r.w};
            if (!__all(d == 0)) {
                mask_pair<false>(p, g);
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) {
                    float t = 0.0f;
#pragma unroll
                    for (int u = 0; u < kMaxK; ++u) t = s - d == u ? (&r.x)[u] : t;
                    v[s] = t;
                }
            }
            acc[0] = fmaf(p.w[3], v[3], fmaf(p.w[2], v[2], fmaf(p.w[1], v[1], fmaf(p.w[0], v[0], acc[0]))));
        } else {
            mask_pair<false>(p, g);
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) {
                const float *row = slab + (int64_t)clampi(p.cell + s, 0, g.rows - 1) * g.n_out;
#pragma unroll
                for (int j = 0; j < NO; ++j)
                    if (j < g.n_out) acc[j] = fmaf(p.w[s], row[j], acc[j]);
            }
        }
        if (g.base_act) {
            const float *wb = w_b + (int64_t)i * g.n_out;
#pragma unroll
            for (int j = 0; j < NO; ++j)
                if (j < g.n_out) acc[j] = fmaf(p.base, wb[j], acc[j]);
        }
        if (NO == 1 && ++n == 8) { tot += acc[0]; acc[0] = 0.0f; n = 0; }
    }
    if (NO == 1) acc[0] += tot;
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        float v = acc[j];
#pragma unroll
        for (int d = 1; d < Q; d *= 2) v += __shfl_xor(v, d, 64);
        acc[j] = v;
    }
    if (q == 0 && b < B) {
#pragma unroll
        for (int j = 0; j < NO; ++j)
            if (j < g.n_out) y[b * g.n_out + j] = acc[j];
    }
}

// ---- backward: dL/dx ------------------------------------------------------------------------
template <int NO>
__global__ __launch_bounds__(256) void dx_narrow_kernel(SplineGeom g, const float *__restrict__ x,
                                                        const float *__restrict__ cf, const float *__restrict__ w_b,
                                                        const float *__restrict__ gy, float *__restrict__ gx,
                                                        int64_t B)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    float gv[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) gv[j] = (j < g.n_out) ? gy[b * g.n_out + j] : 0.0f;
    for (int i = 0; i < g.n_in; ++i) {
        const Pair p = pair_eval<true>(x[b * g.n_in + i], g, i);
        const float *slab = cf + (int64_t)i * g.slab_rows * g.n_out;
        float acc = 0.0f;
#pragma unroll
        for (int s = 0; s < kMaxK; ++s) {
            const float *row = slab + (int64_t)clampi(p.cell + s, 0, g.rows - 1) * g.n_out;
            float ts = 0.0f;
#pragma unroll
            for (int j = 0; j < NO; ++j)
                if (j < g.n_out) ts = fmaf(gv[j], row[j], ts);
            acc = fmaf(p.dw[s], ts, acc);
        }
        if (g.base_act) {
            const float *wb = w_b + (int64_t)i * g.n_out;
            float tb = 0.0f;
#pragma unroll
            for (int j = 0; j < NO; ++j)
                if (j < g.n_out) tb = fmaf(gv[j], wb[j], tb);
            acc = fmaf(p.dbase, tb, acc);
        }
        gx[b * g.n_in + i] = acc;
    }
}

// ---- launch -------------------------------------------------------------------------------------

int narrow_applicable(const SplineGeom &g) { return g.n_out <= 16 ? 1 : 0; }

#define KAN_NARROW_DISPATCH(n_out, CALL)        \
    if ((n_out) <= 1) { CALL(1); }               \
    else if ((n_out) <= 2) { CALL(2); }          \
    else if ((n_out) <= 4) { CALL(4); }          \
    else if ((n_out) <= 8) { CALL(8); }          \
    else { CALL(16); }

hipError_t launch_forward_narrow(const SplineGeom &g, const float *x, const float *cf, const float *w_b, float *y,
                                 int64_t B, hipStream_t st)
{
    prof::Timed tm("forward_narrow", st);
    // One output from 32 inputs on: sixteen lanes a sample, four times the waves and whole lines of x, until the batch fills the chip
    // either way (four / sixteen, G = 240, us: 256 -> 1, B = 32768 52 / 30; 128 -> 1, B = 5000 26 / 10; 32 -> 1, B = 65536 11.9 / 10.9,
    // 262144 27 / 30; 16 -> 1, B = 262144 16 / 20; 64 -> 2, B = 65536 41 / 71).  Degrees 1 and 2, where nearly every wave has a window over
    // the table's end: 34 -> 1, G = 40, k = 1, B = 65536 13.9 / 13.0, 108173 17.4 / 18.6, its third round of inputs almost empty;
    // 48 -> 1, B = 131072 25 / 23.
    const int64_t most = g.k < 3 && g.n_in > 32 && g.n_in < 48 ? 3 << 15 : 1 << 17;
    if (g.n_out == 1 && g.n_in >= 32 && B <= most) {
        forward_narrow_kernel<1, 16><<<(unsigned)((16 * B + 255) / 256), 256, 0, st>>>(g, x, cf, w_b, y, B);
        return hipGetLastError();
    }
    const unsigned blocks = (unsigned)((4 * B + 255) / 256);
#define CALL(N) forward_narrow_kernel<N, 4><<<blocks, 256, 0, st>>>(g, x, cf, w_b, y, B)
    KAN_NARROW_DISPATCH(g.n_out, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_dx_narrow(const SplineGeom &g, const float *x, const float *cf, const float *w_b, const float *gy,
                            float *gx, int64_t B, hipStream_t st)
{
    prof::Timed tm("dx_narrow", st);
    const unsigned blocks = (unsigned)((B + 255) / 256);
#define CALL(N) dx_narrow_kernel<N><<<blocks, 256, 0, st>>>(g, x, cf, w_b, gy, gx, B)
    KAN_NARROW_DISPATCH(g.n_out, CALL)
#undef CALL
    return hipGetLastError();
}

}  // namespace kan
