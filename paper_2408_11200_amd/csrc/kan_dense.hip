// Backward kernel for layers of few rows and outputs (small regression networks and their like): the whole pass
// between the launch and the reduction over the chunks in one kernel, as small dense products on the matrix cores.
//
// The chunk-sorted walk takes a transpose, a sort, the walk and a gather of carry rows before the reduction; on a
// layer like 16 -> 32 with 11 rows (B = 4096) those are launches and latency, and there is little for the sorting to save: the
// dense basis row of a sample (G + k weights and the base value) is barely longer than its window.  Here a workgroup
// takes one input and kSub samples at a time, writes their dense basis rows to LDS (P, one row per sample) beside
// their gy rows, and forms
//   parameter gradients:  P^T . gy           (rows x outputs, summed over the samples; the base row is gw_b's sum)
//   dL/dx:                dP : (gy . C^T)    (per sample the dot product of its derivative row with gy . C^T)
// with v_mfma_f32_16x16x4_f32, MT tiles of 16 rows by NTL tiles of 16 outputs.  The running sums stay in registers over
// the sub-chunks of a chunk; chunks are added by the reduction in fp64, so results are bit-reproducible.
#include "kan_device.hpp"
#include "kan_launch.hpp"

namespace kan {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSub = 256;               // samples a workgroup holds at a time, one per thread
constexpr int kPad = 4;                 // floats a LDS row is padded by: 16 rows x 4 columns then hit 64 banks

// What tells the rows of a sample from the others in its basis row is that their bits are not all zero: a zero weight inside
// the window is kept as -0.  Multiplied it stays zero, except by an infinity or NaN, which it must not hide.
__device__ __forceinline__ float in_window(float w) { return w == 0.0f ? -0.0f : w; }
__device__ __forceinline__ bool is_in_window(float w) { return __float_as_uint(w) != 0u; }

template <int MT, int NTL>
constexpr size_t dense_lds_bytes()
{
    return (size_t)(kSub * (16 * NTL + kPad) + kSub * (16 * MT + kPad) + 16 * MT * (16 * NTL + kPad)) * sizeof(float);
}

}  // namespace

// grid (n_in, n_chunks), 256 threads.  Chunk c covers samples c * chunk_len .. (chunk_len a multiple of kSub).
// coef[n_in][rows][n_out]; w_s may be null (coef is scaled already), w_b too (no base term).  Needs rows + 1 <= 16 * MT,
// n_out <= 16 * NTL.  Any of part_c, part_b, gx may be null.
template <int MT, int NTL>
__global__ __launch_bounds__(256) void backward_dense_kernel(SplineGeom g, const float *__restrict__ x,
                                                             const float *__restrict__ gy, const float *__restrict__ coef,
                                                             const float *__restrict__ w_s, const float *__restrict__ w_b,
                                                             float *__restrict__ part_c, float *__restrict__ part_b,
                                                             float *__restrict__ gx, int64_t B, int64_t chunk_len)
{
    constexpr int GS = 16 * NTL + kPad, PS = 16 * MT + kPad;
    extern __shared__ float lds[];
    float *gt = lds, *P = gt + kSub * GS, *C = P + kSub * PS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, l4 = lane >> 4;
    const int i = blockIdx.x;
    const int64_t c0 = (int64_t)blockIdx.y * chunk_len;
    const int64_t c1 = c0 + chunk_len < B ? c0 + chunk_len : B;

    for (int e = tid; e < kSub * GS; e += 256) gt[e] = 0.0f;           // columns past n_out stay zero
    for (int e = tid; e < kSub * PS; e += 256) P[e] = 0.0f;
    if (gx) {
        for (int e = tid; e < 16 * MT * GS; e += 256) {
            const int m = e / GS, j = e - m * GS;
            float v = 0.0f;
            if (j < g.n_out) {
                if (m < g.rows) {
                    v = coef[((int64_t)i * g.rows + m) * g.n_out + j];
                    if (w_s) v *= w_s[(int64_t)i * g.n_out + j];
                } else if (m == g.rows && g.base_act) {
                    v = w_b[(int64_t)i * g.n_out + j];
                }
            }
            C[e] = v;
        }
    }
    f32x4 acc[MT][NTL];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NTL; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int s_inc = 256 / g.n_out, j_inc = 256 - s_inc * g.n_out;
    float *mine = P + tid * PS;                                        // this thread's sample
    __syncthreads();

    for (int64_t b0 = c0; b0 < c1; b0 += kSub) {
        const int n_c = (int)(c1 - b0 < kSub ? c1 - b0 : kSub);
        bool finite = true;
        {
            int s = tid / g.n_out, j = tid - s * g.n_out;
            const float *src = gy + b0 * g.n_out;
            for (int e = tid; e < kSub * g.n_out; e += 256) {
                const float v = e < n_c * g.n_out ? src[e] : 0.0f;
                finite &= fabsf(v) <= 3.402823466e38f;
                gt[s * GS + j] = v;
                s += s_inc; j += j_inc;
                if (j >= g.n_out) { j -= g.n_out; ++s; }
            }
        }
        const bool live = tid < n_c;
        Pair p;
        if (live) {
            p = pair_eval<true>(x[(b0 + tid) * g.n_in + i], g, i);
#pragma unroll
            for (int q = 0; q < kMaxK; ++q)
                if (q <= g.k && p.cell + q >= 0 && p.cell + q < g.rows) mine[p.cell + q] = in_window(p.w[q]);
            if (g.base_act) mine[g.rows] = in_window(p.base);
        }
        // an infinite or NaN gradient must not reach the rows its sample does not touch: such a sub-chunk is summed
        // entry by entry below
        const bool all_finite = __syncthreads_and(finite ? 1 : 0) != 0;
        // each wave its own 64 samples
        const float *gw = gt + wave * 64 * GS, *Pw = P + wave * 64 * PS;
        if (part_c && !all_finite) {
            for (int s = 0; s < 64; ++s)
#pragma unroll
                for (int a = 0; a < MT; ++a)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float w = Pw[s * PS + 16 * a + 4 * l4 + v];
#pragma unroll
                        for (int b = 0; b < NTL; ++b)
                            if (is_in_window(w)) acc[a][b][v] = fmaf(w, gw[s * GS + 16 * b + l16], acc[a][b][v]);
                    }
        } else if (part_c) {
#pragma unroll 4
            for (int s = 0; s < 64; s += 4) {
                float av[MT], bv[NTL];
#pragma unroll
                for (int a = 0; a < MT; ++a) av[a] = Pw[(s + l4) * PS + 16 * a + l16];
#pragma unroll
                for (int b = 0; b < NTL; ++b) bv[b] = gw[(s + l4) * GS + 16 * b + l16];
#pragma unroll
                for (int a = 0; a < MT; ++a)
#pragma unroll
                    for (int b = 0; b < NTL; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
            }
        }
        __syncthreads();
        // the sample's row becomes its derivative row (the same entries), or zeros again
        if (live) {
#pragma unroll
            for (int q = 0; q < kMaxK; ++q)
                if (q <= g.k && p.cell + q >= 0 && p.cell + q < g.rows) mine[p.cell + q] = gx ? in_window(p.dw[q]) : 0.0f;
            if (g.base_act) mine[g.rows] = gx ? in_window(p.dbase) : 0.0f;
        }
        if (gx) {
            __syncthreads();
#pragma unroll
            for (int st = 0; st < 4; ++st) {            // tiles of 16 samples
                f32x4 h[MT];
#pragma unroll
                for (int a = 0; a < MT; ++a) h[a] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
                for (int j = 0; j < 16 * NTL; j += 4) {
                    const float av = gw[(16 * st + l16) * GS + j + l4];
#pragma unroll
                    for (int a = 0; a < MT; ++a)
                        h[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, C[(16 * a + l16) * GS + j + l4], h[a], 0, 0, 0);
                }
                // register v of the lane: sample 16 st + 4 l4 + v, row 16 a + l16
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int s = 16 * st + 4 * l4 + v;
                    float d = 0.0f;
#pragma unroll
                    for (int a = 0; a < MT; ++a) {
                        const float w = Pw[s * PS + 16 * a + l16];
                        d = is_in_window(w) ? fmaf(w, h[a][v], d) : d;        // rows outside the window: nothing, whatever they hold
                    }
                    d += __shfl_xor(d, 1, 64);
                    d += __shfl_xor(d, 2, 64);
                    d += __shfl_xor(d, 4, 64);
                    d += __shfl_xor(d, 8, 64);
                    const int64_t b = b0 + wave * 64 + s;
                    if (l16 == 0 && b < c1) gx[b * g.n_in + i] = d;
                }
            }
            __syncthreads();
            if (live) {
#pragma unroll
                for (int q = 0; q < kMaxK; ++q)
                    if (p.cell + q >= 0 && p.cell + q < g.rows) mine[p.cell + q] = 0.0f;
                mine[g.rows] = 0.0f;
            }
        }
    }

    if (!part_c) return;
    // the four waves' sums, added in wave order (the gy tile's space holds them: 4 * 256 * MT * NTL floats)
    __syncthreads();
    float *red = lds;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NTL; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[((wave * MT + a) * 16 + 4 * l4 + v) * (16 * NTL) + 16 * b + l16] = acc[a][b][v];
    __syncthreads();
    constexpr int kTile = 16 * MT * 16 * NTL;
    for (int e = tid; e < kTile; e += 256) {
        const int m = e / (16 * NTL), j = e % (16 * NTL);
        if (j >= g.n_out || m > g.rows) continue;
        const float v = ((red[e] + red[kTile + e]) + red[2 * kTile + e]) + red[3 * kTile + e];
        const int64_t ci = (int64_t)blockIdx.y * g.n_in + i;
        if (m < g.rows) part_c[(ci * g.rows + m) * g.n_out + j] = v;
        else if (part_b) part_b[ci * g.n_out + j] = v;
    }
}

namespace {
template <int MT, int NTL>
hipError_t dense_launch(const SplineGeom &g, const DensePlan &p, const float *x, const float *gy, const float *coef,
                        const float *w_s, const float *w_b, float *part_c, float *part_b, float *gx, int64_t B,
                        hipStream_t st)
{
    auto kern = backward_dense_kernel<MT, NTL>;
    struct Tag;
    if (hipError_t e = ensure_dynamic_lds<Tag>(reinterpret_cast<const void *>(kern), (int)dense_lds_bytes<MT, NTL>()); e != hipSuccess)
        return e;
    prof::Timed tm("backward_dense", st);
    kern<<<dim3((unsigned)g.n_in, (unsigned)p.n_chunks), 256, dense_lds_bytes<MT, NTL>(), st>>>(g, x, gy, coef, w_s, w_b, part_c,
                                                                                              part_b, gx, B, p.chunk_len);
    return hipGetLastError();
}
}  // namespace

// Where the line lies: on the pairs B * n_in, by the tiles a pair costs.  Backward pass with the reduction, walk / this,
// us:   2 -> 5, G = 10      B = 1024 32 / 17, 65536 87 / 20
//       16 -> 5, G = 10     B = 8192 37 / 20, 65536 85 / 72;       64 -> 5   B = 8192 44 / 40, 65536 159 / 238
//       16 -> 32, G = 10    B = 1024 34 / 22, 8192 41 / 25, 65536 100 / 149
//       64 -> 64, G = 10    B = 1024 39 / 31, 8192 60 / 228;       2 -> 64   B = 65536 138 / 80
//       16 -> 5, G = 55     B = 8192 43 / 36, 65536 87 / 164;      16 -> 32, G = 55   B = 1024 47 / 29, 8192 48 / 54
// (A line on the pairs alone leaves some to the walk that this kernel would do in less: with two inputs, as 2 -> 64 shows, the
// walk has few lists.)
DensePlan plan_dense(const SplineGeom &g, int64_t B)
{
    DensePlan p = {0, 0, 0};
    if (g.k >= kMaxK || g.n_out > 64 || g.rows + 1 > 64 || B < 1) return p;
    const bool short_rows = g.rows + 1 <= 32;
    const int64_t limit = g.n_out <= 16 ? (short_rows ? 1 << 20 : 1 << 17)
                          : g.n_out <= 32 ? (short_rows ? 1 << 18 : 1 << 16)
                                          : 1 << 16;
    if (B * g.n_in > limit) return p;
    // sub-chunks per chunk: as many as leave two workgroups per CU.  Within the limits above that is eight at most (running
    // sums of 512 samples a wave), or a chunk longer than the batch; the bound of 16 is not reached.
    int64_t sub = 1;
    const int64_t subs = (B + kSub - 1) / kSub;
    while (sub < 16 && (subs + 2 * sub - 1) / (2 * sub) * g.n_in >= 512) sub *= 2;
    p.chunk_len = sub * kSub;
    p.n_chunks = (int)((B + p.chunk_len - 1) / p.chunk_len);
    if (p.n_chunks > 65535) return p;
    p.ok = 1;
    return p;
}

hipError_t launch_backward_dense(const SplineGeom &g, const DensePlan &p, const float *x, const float *gy, const float *coef,
                                 const float *w_s, const float *w_b, float *part_c, float *part_b, float *gx, int64_t B,
                                 hipStream_t st)
{
    const int mt = (g.rows + 16) / 16, ntl = (g.n_out + 15) / 16;
#define KAN_DENSE(M, N) return dense_launch<M, N>(g, p, x, gy, coef, w_s, w_b, part_c, part_b, gx, B, st)
#define KAN_DENSE_ROW(M)                    \
    switch (ntl) {                          \
    case 1: KAN_DENSE(M, 1);                \
    case 2: KAN_DENSE(M, 2);                \
    default: KAN_DENSE(M, 4);               \
    }
    switch (mt) {
    case 1: KAN_DENSE_ROW(1)
    case 2: KAN_DENSE_ROW(2)
    default: KAN_DENSE_ROW(4)
    }
#undef KAN_DENSE_ROW
#undef KAN_DENSE
}

}  // namespace kan
