// Kernels of the UKAN-specific part: cell / group bookkeeping on the unbounded grid,
// the coefficient-generator (CG) MLP forward and backward.  The B-spline evaluation on
// the generated table is done by the same kernels as the bounded layer.
//
// The dense contractions of the CG run on the matrix cores in fp32
// (v_mfma_f32_32x32x2_f32); everything else here is small and bandwidth-bound.
#include <limits.h>
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "ukan_launch.hpp"

namespace kan {

// floor division by a positive K and the matching non-negative remainder
__device__ __forceinline__ int floordiv(int a, int K) { int q = a / K; return (a % K < 0) ? q - 1 : q; }

// ---- cell / group / offset export -------------------------------------------
__global__ void group_index_kernel(const float *__restrict__ x, int32_t *__restrict__ cell,
                                   int32_t *__restrict__ grp, int32_t *__restrict__ off, int64_t n,
                                   float inv_h, int K)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    float t, d;
    int32_t c = interval_index(x[p], 0.0f, inv_h, &t, &d);
    int32_t g = floordiv(c, K);
    if (cell) cell[p] = c;
    if (grp) grp[p] = g;
    if (off) off[p] = c - g * K;
}

// ---- per-input range of cells -------------------------------------------------
// Two kernels: strips of the batch write their partial minima and maxima, one workgroup combines them.  (Atomics on one
// pair per input needed a third kernel to set them up and kept a thread to one column: 28 -> 18 us at 33 MB, 256 inputs.)
constexpr int kRangeThreads = 1024;

// grid (strips, input tiles).  LR lanes x V inputs cover a tile of a row, the other threads take other rows of the strip.
template <int V>
__global__ __launch_bounds__(kRangeThreads) void range_kernel(const float *__restrict__ x, int32_t *__restrict__ part,
                                                              int64_t B, int n_in, float inv_h, int LR, int64_t strip)
{
    __shared__ int lo_s[kRangeThreads * V], hi_s[kRangeThreads * V];
    const int tid = threadIdx.x, col = tid % LR, rg = tid / LR, RP = kRangeThreads / LR;
    const int i = ((int)blockIdx.y * LR + col) * V;
    const int64_t b1 = ((int64_t)blockIdx.x + 1) * strip < B ? ((int64_t)blockIdx.x + 1) * strip : B;
    int lo[V], hi[V];
#pragma unroll
    for (int v = 0; v < V; ++v) { lo[v] = INT_MAX; hi[v] = INT_MIN; }
    if (i < n_in) {                                  // V divides n_in
        auto take = [&](const float (&q)[V]) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                float t, d;
                const int c = interval_index(q[v], 0.0f, inv_h, &t, &d);
                lo[v] = c < lo[v] ? c : lo[v];
                hi[v] = c > hi[v] ? c : hi[v];
            }
        };
        auto load = [&](int64_t b, float (&q)[V]) {
            if constexpr (V == 4) {
                const float4 t = *reinterpret_cast<const float4 *>(x + b * n_in + i);
                q[0] = t.x; q[1] = t.y; q[2] = t.z; q[3] = t.w;
            } else {
                q[0] = x[b * n_in + i];
            }
        };
        int64_t b = (int64_t)blockIdx.x * strip + rg;
        for (; b + 3 * RP < b1; b += 4 * RP) {       // four rows in flight
            float q[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) load(b + u * RP, q[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) take(q[u]);
        }
        for (; b < b1; b += RP) {
            float q[V];
            load(b, q);
            take(q);
        }
    }
    // rows of the workgroup, halving; columns stay
#pragma unroll
    for (int v = 0; v < V; ++v) { lo_s[tid * V + v] = lo[v]; hi_s[tid * V + v] = hi[v]; }
    for (int s = RP / 2; s > 0; s >>= 1) {
        __syncthreads();
        if (rg < s) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int o = (tid + s * LR) * V + v, m = tid * V + v;
                if (lo_s[o] < lo_s[m]) lo_s[m] = lo_s[o];
                if (hi_s[o] > hi_s[m]) hi_s[m] = hi_s[o];
            }
        }
    }
    if (rg == 0 && i < n_in) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            part[((int64_t)blockIdx.x * 2) * n_in + i + v] = lo_s[tid * V + v];
            part[((int64_t)blockIdx.x * 2 + 1) * n_in + i + v] = hi_s[tid * V + v];
        }
    }
}

// partial ranges -> first group held, relative-cell base; the widest span goes to summary[0].  overflow (may be null)
// receives 1 when the widest span exceeds `provided`, else 0.  One workgroup: LC lanes take the inputs of a tile, the
// other threads other strips of them.
__global__ __launch_bounds__(kRangeThreads) void range_finalize_kernel(const int32_t *__restrict__ part, int strips,
                                                                       int32_t *__restrict__ g_first,
                                                                       int32_t *__restrict__ cell_base,
                                                                       int32_t *__restrict__ summary, int n_in, int K,
                                                                       int LC, int provided, int32_t *__restrict__ overflow)
{
    __shared__ int lo_s[kRangeThreads], hi_s[kRangeThreads];
    const int tid = threadIdx.x, col = tid % LC, sg = tid / LC, SG = kRangeThreads / LC;
    int widest = 0;
    for (int i0 = 0; i0 < n_in; i0 += LC) {
        const int i = i0 + col;
        int lo = INT_MAX, hi = INT_MIN;
        if (i < n_in)
#pragma unroll 8
            for (int s = sg; s < strips; s += SG) {
                const int a = part[(int64_t)s * 2 * n_in + i], b = part[((int64_t)s * 2 + 1) * n_in + i];
                lo = a < lo ? a : lo;
                hi = b > hi ? b : hi;
            }
        __syncthreads();
        lo_s[tid] = lo; hi_s[tid] = hi;
        for (int s = SG / 2; s > 0; s >>= 1) {
            __syncthreads();
            if (sg < s) {
                const int o = tid + s * LC;
                if (lo_s[o] < lo_s[tid]) lo_s[tid] = lo_s[o];
                if (hi_s[o] > hi_s[tid]) hi_s[tid] = hi_s[o];
            }
        }
        if (sg == 0 && i < n_in) {
            const int gmin = floordiv(lo_s[tid], K), gmax = floordiv(hi_s[tid], K);
            const long long n = (long long)gmax - (long long)gmin + 2;      // groups gmin-1 .. gmax
            const int n32 = n > INT_MAX ? INT_MAX : (int)n;
            g_first[i] = gmin - 1;
            cell_base[i] = gmin * K;        // cell c reads table rows c - gmin*K .. + K-1
            widest = n32 > widest ? n32 : widest;
        }
    }
    __syncthreads();
    lo_s[tid] = widest;
    for (int s = kRangeThreads / 2; s > 0; s >>= 1) {
        __syncthreads();
        if (tid < s && lo_s[tid + s] > lo_s[tid]) lo_s[tid] = lo_s[tid + s];
    }
    if (tid == 0) {
        summary[0] = lo_s[0];
        if (overflow) overflow[0] = lo_s[0] > provided ? 1 : 0;
    }
}

// ---- CG input and hidden layer -------------------------------------------------
// Row (i, t) of the generator batch is group g_first[i] + t of input i: z = [E[i] ; PE(g)] (PE evaluated in fp64, rounded
// to fp32), pre = W1^T z + b1, hid = silu(pre).  A workgroup takes kHidRows consecutive rows, four threads a hidden unit
// and kHidRows / 4 rows a thread, with the z rows and W1 in LDS: a row a workgroup re-read W1 (16 KB at 64 x 64) per row
// and evaluated the frequencies anew.  What is left is mostly the sines in fp64 (48 000 rows in three launches: 84 -> 66 us;
// 1 400 rows, a load of W1 at a time behind the sines 15 us, eight before them 11, a row a workgroup 10).
constexpr int kHidRows = 16;
template <bool W1_LDS>
__global__ __launch_bounds__(256) void cg_hidden_kernel(const float *__restrict__ E, const float *__restrict__ W1,
                                                        const float *__restrict__ b1,
                                                        const int32_t *__restrict__ g_first, float *__restrict__ z,
                                                        float *__restrict__ pre, float *__restrict__ hid, int64_t rows,
                                                        int n_g, int d_pe, int d_feat, int d_hid, int per_block)
{
    extern __shared__ double freq[];                // d_pe / 2 frequencies, per_block x dz, W1
    const int dz = d_feat + d_pe, tid = threadIdx.x;
    float *zs = reinterpret_cast<float *>(freq + d_pe / 2), *w1 = zs + per_block * dz;
    const int64_t row0 = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * per_block;
    if (row0 >= rows) return;
    const int n = rows - row0 < per_block ? (int)(rows - row0) : per_block;
    if (W1_LDS) {                                   // first, and several loads in flight: nothing waits for them until the sums
#pragma unroll 8
        for (int e = tid; e < dz * d_hid; e += 256) w1[e] = W1[e];
    }
    // d_pe / 2 frequencies, once a workgroup
    const int half = d_pe / 2;
    for (int q = tid; q < half; q += 256) freq[q] = pow(10000.0, -2.0 * (double)q / (double)d_pe);
    for (int e = tid; e < n * d_feat; e += 256) {
        const int r = e / d_feat, c = e - r * d_feat;
        const float v = E[((row0 + r) / n_g) * d_feat + c];
        zs[r * dz + c] = v;
        if (z) z[(row0 + r) * dz + c] = v;
    }
    __syncthreads();
    for (int e = tid; e < n * half; e += 256) {
        const int r = e / half, q = e - r * half;
        const int64_t row = row0 + r;
        const int i = (int)(row / n_g), t = (int)(row - (int64_t)i * n_g);
        double sn, cs;
        sincos((double)(g_first[i] + t) * freq[q], &sn, &cs);
        const int c = d_feat + 2 * q;
        zs[r * dz + c] = (float)sn;
        zs[r * dz + c + 1] = (float)cs;
        if (z) { z[row * dz + c] = (float)sn; z[row * dz + c + 1] = (float)cs; }
    }
    __syncthreads();
    constexpr int PER = kHidRows / 4;
    for (int c = tid & 63; c < d_hid; c += 64) {
        const int r0 = (tid >> 6) * PER;
        // fp64 accumulation: this layer is tiny and its rounding error would otherwise be
        // amplified into every generated coefficient
        double sd[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) sd[u] = (double)b1[c];
        for (int p = 0; p < dz; ++p) {
            const double w = (double)(W1_LDS ? w1[p * d_hid + c] : W1[(int64_t)p * d_hid + c]);
#pragma unroll
            for (int u = 0; u < PER; ++u) sd[u] += (double)zs[(r0 + u < n ? r0 + u : n - 1) * dz + p] * w;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (r0 + u >= n) continue;
            const int64_t at = (row0 + r0 + u) * d_hid + c;
            if (pre) pre[at] = (float)sd[u];
            hid[at] = (float)(sd[u] / (1.0 + exp(-sd[u])));
        }
    }
}

// ---- matrix-core GEMM ------------------------------------------------------------
// C(m,n) = sum_k A(m,k) B(k,n), fp32 operands addressed through (row, column) strides so that
// transposed views need no copy.  One block = 4 waves = one BM x 64 tile of C; each wave owns a
// 32x32 quadrant of 64x64; K-slices are staged through LDS.  blockIdx.z selects a slice of K (split-K):
// slice z writes its own copy of C at C + z*c_slice.
//   ACC64 = false: v_mfma_f32_32x32x2_f32, fp32 accumulation folded every 64 terms (forward).
//   ACC64 = true : operands widened to fp64, v_mfma_f64_16x16x4_f64.  Used by the CG backward
//                  pass, whose long sums cancel heavily; the products are then exact and the
//                  only rounding is the final conversion to fp32.
//   BM = 32 : 32x64 tiles, a wave 32x16: twice the workgroups where all of K is one slice and N one tile (the hidden layer's
//             gradient, 13400 x 64 from 1024: 210 workgroups 75 us, 420 67, beside about 30 for the matrix instructions; a backward pass with
//             128 columns 782 -> 760, 256 268 -> 263, 512, where tiles of 64 fill the chip, 719 -> 720).
using f32x16 = __attribute__((__vector_size__(16 * sizeof(float)))) float;
using f64x4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;

template <int EPI, typename V>
__device__ __forceinline__ void gemm_store(const GemmArgs &a, float *C, int64_t m, int64_t n, V acc)
{
    if (m >= a.M || n >= a.N) return;
    if (EPI == EPI_PLAIN) {
        C[m * a.ldc + n] = (float)acc;
    } else if (EPI == EPI_CG_OUT) {
        // generator output: add b2, keep the raw value if asked, store the scale-folded one
        float val = (float)acc + a.bias[n];
        const int64_t i = m / a.rows_per_input;
        const float sc = a.scale[i * a.n_out + (n % a.n_out)];
        if (a.C2) a.C2[m * a.ldc + n] = val;
        C[m * a.ldc + n] = val * sc;
    } else {   // EPI_SILU_GRAD: multiply by silu'(pre), evaluated in fp64
        const double x = (double)a.aux[m * a.ldc + n];
        const double sg = 1.0 / (1.0 + exp(-x));
        C[m * a.ldc + n] = (float)((double)acc * (sg * (1.0 + x * (1.0 - sg))));
    }
}

template <int EPI, bool ACC64, int BM>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(GemmArgs a)
{
    static_assert(BM == 64 || (BM == 32 && ACC64), "");
    constexpr int BN = 64, BK = 16, PAD = 4, BJ = BM / 32;             // 16-column blocks of a wave
    // two LDS stages: the next K step is fetched into registers while the current one is multiplied,
    // then parked in the other stage; one barrier per step
    __shared__ float As[2][BK][BM + PAD];
    __shared__ float Bs[2][BK][BN + PAD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int64_t k_lo = (int64_t)blockIdx.z * a.k_slice;
    const int64_t k_hi = (k_lo + a.k_slice < a.K) ? k_lo + a.k_slice : a.K;
    const int wm = BM == 64 ? (wave >> 1) * 32 : 0, wn = BM == 64 ? (wave & 1) * 32 : wave * 16;

    f32x16 acc, tot;
    f64x4 dacc[2][BJ];
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[v] = 0.0f; tot[v] = 0.0f; }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
            for (int v = 0; v < 4; ++v) dacc[bi][bj][v] = 0.0;

    // A[BM x BK] and B[BK x BN] of one K step: four elements of each per thread; the thread -> element
    // map follows whichever stride is 1
    constexpr int PA = BM * BK / 256, PB = BN * BK / 256;
    float ra[PA], rb[PB];
    auto at_a = [&](int u, int &mm, int &kk) {
        const int e = tid + u * 256;
        if (a.a_cs == 1) { kk = e % BK; mm = e / BK; } else { mm = e % BM; kk = e / BM; }
    };
    auto at_b = [&](int u, int &nn, int &kk) {
        const int e = tid + u * 256;
        if (a.b_cs == 1) { nn = e % BN; kk = e / BN; } else { kk = e % BK; nn = e / BK; }
    };
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int u = 0; u < PA; ++u) {
            int mm, kk;
            at_a(u, mm, kk);
            const int64_t m = m0 + mm, k = k0 + kk;
            ra[u] = (m < a.M && k < k_hi) ? a.A[m * a.a_rs + k * a.a_cs] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            int nn, kk;
            at_b(u, nn, kk);
            const int64_t n = n0 + nn, kb = k0 + kk;
            rb[u] = (n < a.N && kb < k_hi) ? a.B[kb * a.b_rs + n * a.b_cs] : 0.0f;
        }
    };
    auto park = [&](int buf) {
        int mm, nn, kk;
#pragma unroll
        for (int u = 0; u < PA; ++u) { at_a(u, mm, kk); As[buf][kk][mm] = ra[u]; }
#pragma unroll
        for (int u = 0; u < PB; ++u) { at_b(u, nn, kk); Bs[buf][kk][nn] = rb[u]; }
    };

    // column sums of B (bias gradients) ride along in the first row of workgroups: thread -> (column, quarter of the K step)
    const bool sums = ACC64 && EPI == EPI_PLAIN && a.colsum && blockIdx.y == 0;
    double csum = 0.0;
    int step = 0, buf = 0;
    if (k_lo < k_hi) {
        fetch(k_lo);
        park(0);
    }
    __syncthreads();
    for (int64_t k0 = k_lo; k0 < k_hi; k0 += BK, ++step) {
        if (!ACC64 && (step & 3) == 0 && step > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) { tot[v] += acc[v]; acc[v] = 0.0f; }
        }
        const bool more = k0 + BK < k_hi;
        if (more) fetch(k0 + BK);
        if (sums) {
#pragma unroll
            for (int u = 0; u < 4; ++u) csum += (double)Bs[buf][wave * 4 + u][lane];
        }
        if constexpr (ACC64) {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 4) {
                const int kr = kk + (lane >> 4), c = lane & 15;
                const double a0 = (double)As[buf][kr][wm + c], a1 = (double)As[buf][kr][wm + 16 + c];
#pragma unroll
                for (int bj = 0; bj < BJ; ++bj) {
                    const double bv = (double)Bs[buf][kr][wn + 16 * bj + c];
                    dacc[0][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, bv, dacc[0][bj], 0, 0, 0);
                    dacc[1][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, bv, dacc[1][bj], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 2) {
                float av = As[buf][kk + (lane >> 5)][wm + (lane & 31)];
                float bv = Bs[buf][kk + (lane >> 5)][wn + (lane & 31)];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
            }
        }
        if (more) park(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }

    float *C = a.C + (int64_t)blockIdx.z * a.c_slice;
    if constexpr (ACC64 && EPI == EPI_PLAIN) {
        if (a.colsum) {                            // row M of the slice
            __shared__ double cs[4][64];
            cs[wave][lane] = csum;
            __syncthreads();
            if (sums && wave == 0 && n0 + lane < a.N)
                C[a.M * a.ldc + n0 + lane] = (float)(((cs[0][lane] + cs[1][lane]) + cs[2][lane]) + cs[3][lane]);
        }
    }
    if constexpr (ACC64) {
        // 16x16 block: register v of lane l is element (4*v + l/16, l%16)
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    gemm_store<EPI, double>(a, C, m0 + wm + 16 * bi + 4 * v + (lane >> 4),
                                            n0 + wn + 16 * bj + (lane & 15), dacc[bi][bj][v]);
    } else {
        // 32x32 block: register v of lane l is element (8*(v/4) + 4*(l/32) + v%4, l%32)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            gemm_store<EPI, float>(a, C, m0 + wm + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4),
                                   n0 + wn + (lane & 31), tot[v] + acc[v]);
    }
}

// The column sums of B alone (a bias gradient without its weights' gradient): row M of every slice as gemm_mfma_kernel
// writes it, term for term in its order.  grid (64 columns, slices); kSumSteps steps of 16 rows in flight.  128 -> 256, 16 groups,
// B = 256: 57 us with the product,
// 12 alone.
constexpr int kSumSteps = 8;
__global__ __launch_bounds__(256) void column_sums_kernel(GemmArgs a)
{
    __shared__ double cs[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n = (int64_t)blockIdx.x * 64 + lane;
    const int64_t k_lo = (int64_t)blockIdx.y * a.k_slice;
    const int64_t k_hi = (k_lo + a.k_slice < a.K) ? k_lo + a.k_slice : a.K;
    const float *col = a.B + (n < a.N ? n : 0) * a.b_cs;
    double sum = 0.0;
    for (int64_t k0 = k_lo + 4 * wave; k0 < k_hi; k0 += 16 * kSumSteps) {
        float v[4 * kSumSteps];
#pragma unroll
        for (int u = 0; u < 4 * kSumSteps; ++u) {
            const int64_t k = k0 + 16 * (u / 4) + u % 4;
            v[u] = col[(k < k_hi ? k : k_hi - 1) * a.b_rs];
        }
#pragma unroll
        for (int u = 0; u < 4 * kSumSteps; ++u) sum += k0 + 16 * (u / 4) + u % 4 < k_hi ? (double)v[u] : 0.0;
    }
    cs[wave][lane] = sum;
    __syncthreads();
    if (wave == 0 && n < a.N)
        a.C[(int64_t)blockIdx.y * a.c_slice + a.M * a.ldc + n] = (float)(((cs[0][lane] + cs[1][lane]) + cs[2][lane]) + cs[3][lane]);
}

// sum of split-K slices: element e of the result is sum_z part[z][e]; the first n of them are out (may be null), the
// n2 after those out2 (may be null).  Eight slices in flight, added in order.
__global__ __launch_bounds__(256) void slice_sum_kernel(const float *__restrict__ part, float *__restrict__ out,
                                                        int64_t n, float *__restrict__ out2, int64_t n2, int slices)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, total = n + n2;
    if (e >= total) return;
    float *dst = e < n ? (out ? out + e : nullptr) : (out2 ? out2 + (e - n) : nullptr);
    if (!dst) return;
    double s = 0.0;
    int z = 0;
    for (; z + 8 <= slices; z += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(z + u) * total + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (double)v[u];
    }
    for (; z < slices; ++z) s += (double)part[(int64_t)z * total + e];
    *dst = (float)s;
}

// gE[i][f] = sum_c W1[f][c] * S[i][c],  S[i][c] = sum_t gpre[(i,t)][c].  One block per input: its four waves share the
// rows of the column sums S (fp64, the shares added in wave order), then one thread per embedding feature.  The columns go
// in tiles, so that any d_hid fits; the sums over them run on in order.
constexpr int kEmbedCols = 512;
__global__ __launch_bounds__(256) void embed_grad_kernel(const float *__restrict__ W1, const float *__restrict__ gpre,
                                                         float *__restrict__ gE, int n_in, int n_g, int d_feat,
                                                         int d_hid)
{
    __shared__ double colsum[4][kEmbedCols];
    const int i = blockIdx.x, wave = threadIdx.x >> 6;
    const float *src = gpre + (int64_t)i * n_g * d_hid;
    for (int f0 = 0; f0 < d_feat; f0 += 256) {
        const int f = f0 + threadIdx.x;
        double e = 0.0;
        for (int c0 = 0; c0 < d_hid; c0 += kEmbedCols) {
            const int n_c = d_hid - c0 < kEmbedCols ? d_hid - c0 : kEmbedCols;
            if (f0 == 0 || d_hid > kEmbedCols) {            // one tile: its sums stay for the features after the first 256
                __syncthreads();
                for (int c = threadIdx.x & 63; c < n_c; c += 64) {
                    double s = 0.0;
                    int t = wave;
                    for (; t + 28 < n_g; t += 32) {         // eight rows in flight
                        float v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(t + 4 * u) * d_hid + c0 + c];
#pragma unroll
                        for (int u = 0; u < 8; ++u) s += (double)v[u];
                    }
                    for (; t < n_g; t += 4) s += (double)src[(int64_t)t * d_hid + c0 + c];
                    colsum[wave][c] = s;
                }
                __syncthreads();
                for (int c = threadIdx.x; c < n_c; c += 256)
                    colsum[0][c] = ((colsum[0][c] + colsum[1][c]) + colsum[2][c]) + colsum[3][c];
                __syncthreads();
            }
            if (f < d_feat)
#pragma unroll 8
                for (int c = 0; c < n_c; ++c) e += (double)W1[(int64_t)f * d_hid + c0 + c] * colsum[0][c];
        }
        if (f < d_feat) gE[(int64_t)i * d_feat + f] = (float)e;
    }
}

// UKAN -> KAN export: every input uses the same first group; coef[i][m][j] = table row (m + shift)
__global__ __launch_bounds__(256) void fill_int_kernel(int32_t *__restrict__ p, int32_t v, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ __launch_bounds__(256) void table_rows_kernel(const float *__restrict__ table, float *__restrict__ coef,
                                                         int n_in, int table_rows, int coef_rows, int shift, int n_out)
{
    const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (at >= (int64_t)n_in * coef_rows * n_out) return;
    const int j = (int)(at % n_out);
    const int m = (int)((at / n_out) % coef_rows);
    const int i = (int)(at / ((int64_t)n_out * coef_rows));
    coef[at] = table[((int64_t)i * table_rows + m + shift) * n_out + j];
}

// ---- launchers ----------------------------------------------------------------------

hipError_t launch_fill_int(int32_t *p, int32_t v, int n, hipStream_t st)
{
    fill_int_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, v, n);
    return hipGetLastError();
}

hipError_t launch_table_rows(const float *table, float *coef, int n_in, int table_rows, int coef_rows, int shift,
                             int n_out, hipStream_t st)
{
    const int64_t n = (int64_t)n_in * coef_rows * n_out;
    prof::Timed tm("ukan_table_rows", st);
    table_rows_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(table, coef, n_in, table_rows, coef_rows, shift, n_out);
    return hipGetLastError();
}

hipError_t launch_group_index(const float *x, int32_t *cell, int32_t *grp, int32_t *off, int64_t n, float inv_h,
                              int K, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    prof::Timed tm("group_index", st);
    group_index_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(x, cell, grp, off, n, inv_h, K);
    return hipGetLastError();
}

hipError_t launch_range(const float *x, int64_t B, int n_in, float inv_h, int K, int32_t *part, int32_t *g_first,
                        int32_t *cell_base, int32_t *summary, int32_t provided, int32_t *overflow, hipStream_t st)
{
    const int V = n_in % 4 == 0 ? 4 : 1;
    int LR = 1;
    while (LR < 64 && LR * V < n_in) LR *= 2;
    const int strips = range_strips(B);
    const int64_t strip = (B + strips - 1) / strips;
    const dim3 grid((unsigned)strips, (unsigned)((n_in + LR * V - 1) / (LR * V)));
    prof::Timed tm("ukan_range", st);
    if (V == 4) range_kernel<4><<<grid, kRangeThreads, 0, st>>>(x, part, B, n_in, inv_h, LR, strip);
    else range_kernel<1><<<grid, kRangeThreads, 0, st>>>(x, part, B, n_in, inv_h, LR, strip);
    int LC = 1;
    while (LC < 256 && LC < n_in) LC *= 2;
    range_finalize_kernel<<<1, kRangeThreads, 0, st>>>(part, strips, g_first, cell_base, summary, n_in, K, LC, provided, overflow);
    return hipGetLastError();
}

hipError_t launch_cg_hidden(const float *E, const float *W1, const float *b1, const int32_t *g_first, float *z,
                            float *pre, float *hid, int n_in, int n_g, int d_pe, int d_feat, int d_hid,
                            hipStream_t st)
{
    prof::Timed tm("cg_hidden", st);
    const int64_t rows = (int64_t)n_in * n_g;
    const size_t dz = (size_t)d_feat + d_pe, f_bytes = d_pe / 2 * sizeof(double), w_bytes = dz * d_hid * sizeof(float);
    const size_t all = f_bytes + kHidRows * dz * sizeof(float) + w_bytes;
    if (all <= 64 * 1024) {              // what every kernel may ask for
        cg_hidden_kernel<true><<<(unsigned)((rows + kHidRows - 1) / kHidRows), 256, all, st>>>(E, W1, b1, g_first, z, pre, hid,
                                                                                            rows, n_g, d_pe, d_feat, d_hid,
                                                                                            kHidRows);
    } else {
        // wide generators: W1 from L2, and one row a workgroup when sixteen do not fit either
        const int per = f_bytes + kHidRows * dz * sizeof(float) <= 64 * 1024 ? kHidRows : 1;
        const size_t lds = f_bytes + per * dz * sizeof(float);
        struct Tag;
        auto kern = cg_hidden_kernel<false>;
        if (lds > 64 * 1024)
            if (hipError_t e = ensure_dynamic_lds<Tag>(reinterpret_cast<const void *>(kern), (int)lds); e != hipSuccess) return e;
        // one dimension of a launch takes fewer than 2^32 threads: 2^20 workgroups a grid row
        const int64_t blocks = (rows + per - 1) / per, across = blocks < 1 << 20 ? blocks : 1 << 20;
        kern<<<dim3((unsigned)across, (unsigned)((blocks + across - 1) / across)), 256, lds, st>>>(E, W1, b1, g_first, z, pre, hid,
                                                                                                rows, n_g, d_pe, d_feat, d_hid,
                                                                                                per);
    }
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs &a, int epi, int slices, const char *family, hipStream_t st)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    prof::Timed tm(family, st);
    dim3 grid((unsigned)((a.N + 63) / 64), (unsigned)((a.M + 63) / 64), (unsigned)slices);
    switch (epi) {
    case EPI_PLAIN: gemm_mfma_kernel<EPI_PLAIN, true, 64><<<grid, 256, 0, st>>>(a); break;
    case EPI_CG_OUT: gemm_mfma_kernel<EPI_CG_OUT, false, 64><<<grid, 256, 0, st>>>(a); break;
    default: gemm_mfma_kernel<EPI_SILU_GRAD, true, 32><<<dim3(grid.x, (unsigned)((a.M + 31) / 32), grid.z), 256, 0, st>>>(a); break;
    }
    return hipGetLastError();
}

hipError_t launch_column_sums(const GemmArgs &a, int slices, hipStream_t st)
{
    prof::Timed tm("cg_colsum", st);
    column_sums_kernel<<<dim3((unsigned)((a.N + 63) / 64), (unsigned)slices), 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_slice_sum(const float *part, float *out, int64_t n, float *out2, int64_t n2, int slices, hipStream_t st)
{
    prof::Timed tm("cg_slice_sum", st);
    slice_sum_kernel<<<(unsigned)((n + n2 + 255) / 256), 256, 0, st>>>(part, out, n, out2, n2, slices);
    return hipGetLastError();
}

hipError_t launch_embed_grad(const float *W1, const float *gpre, float *gE, int n_in, int n_g, int d_feat,
                             int d_hid, hipStream_t st)
{
    prof::Timed tm("cg_embed_grad", st);
    embed_grad_kernel<<<n_in, 256, 0, st>>>(W1, gpre, gE, n_in, n_g, d_feat, d_hid);
    return hipGetLastError();
}

}  // namespace kan
