// Parameter gradients from the partial sums of the batch chunks: one pass over the partial tables.
//
// Bound by the read of the partial tables on wide layers and by latency on small ones.  The pass used to be three
// kernels (carry rows added to the tables; chunk sums, gcoef and the summed table; gw_s and gw_b from that and the
// coefficients), which read and wrote the summed table an extra time and, with few edges, ran one after the other
// on a fraction of the chip.  The three against this one (with the kernel that adds the slices of gw_s): 64 -> 64, G = 10,
// B = 65536 47 / 17 us; 32 -> 32, G = 1024, B = 131072 83 / 48 us; 32 -> 32, G = 64, k = 5, B = 65536 59 / 21 us;
// 16 -> 1, G = 2^18, B = 65536 285 / 119 us; 2 -> 200, G = 2^18, B = 65536 1416 / 1330 us; wide layers, bound by the read,
// 107 / 99 us (512 -> 512, G = 20, B = 16384: 4.3 TB/s, a large copy reaches 5.2).
//
// A workgroup takes one input, a tile of LJ lanes x T outputs and a slice of the table rows.  Its NT threads are
// LJ lanes x R rows x CS chunk shares (R * CS * LJ == NT, powers of two): with few rows the shares let every partial
// row of the tile be in flight at once.  All sums are fp64 in a fixed order.
#include <limits.h>
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_reduce.hpp"

namespace kan {

namespace {

constexpr int kSegStage = 2048;         // segment rows of one input kept in LDS
constexpr int kMarkBits = 4096;         // marks of the rows that have carry rows

template <int T>
__device__ __forceinline__ void reduce_load(const float *p, float (&v)[T])
{
    if constexpr (T == 4) {
        const float4 t = load4u(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        v[0] = *p;
    }
}
template <int T>
__device__ __forceinline__ void reduce_store(float *p, const float (&v)[T])
{
    if constexpr (T == 4) store4u(p, make_float4(v[0], v[1], v[2], v[3]));
    else *p = v[0];
}

// Sum over `n` (a power of two) threads that are `stride` apart of the T values each brought; the total is valid in the
// threads with index 0.  `at`: the thread's slot, `idx` its index among the n.  Every thread of the workgroup calls this.
template <int T>
__device__ __forceinline__ void tree_sum(double *lds, int at, int idx, int n, int stride, double (&v)[T])
{
    for (int s = n / 2; s > 0; s >>= 1) {
        __syncthreads();
        if (idx >= s && idx < 2 * s) {
#pragma unroll
            for (int r = 0; r < T; ++r) lds[at * T + r] = v[r];
        }
        __syncthreads();
        if (idx < s) {
#pragma unroll
            for (int r = 0; r < T; ++r) v[r] += lds[(at + s * stride) * T + r];
        }
    }
}

}  // namespace

// grid (n_in, output tiles, row slices).  slice_sums != nullptr: gw_s goes there, [slice][n_in][n_out] in fp64.
template <int T, int LJ, int NT>
__global__ __launch_bounds__(NT) void dparam_reduce_kernel(const float *__restrict__ part_c,
                                                           const float *__restrict__ part_b, CarryRows cr,
                                                           const float *__restrict__ coef, const float *__restrict__ w_s,
                                                           float *__restrict__ gcoef, float *__restrict__ gw_s,
                                                           float *__restrict__ gw_b, double *__restrict__ slice_sums,
                                                           int n_in, int rows, int n_out, int n_chunks, int n_slices_b,
                                                           int R, int CS)
{
    __shared__ double lds[NT * T];
    const int tid = threadIdx.x, lj = tid % LJ, grp = tid / LJ, row = grp % R, share = grp / R;
    const int i = blockIdx.x;
    const int jl = (blockIdx.y * LJ + lj) * T;
    const bool jok = jl < n_out;
    // the lane of the last outputs starts at n_out - T: what it shares with its neighbour comes out the same twice
    const int j = !jok ? 0 : (jl + T > n_out ? n_out - T : jl);
    const int per = (rows + gridDim.z - 1) / gridDim.z;
    const int m_lo = blockIdx.z * per, m_hi = m_lo + per < rows ? m_lo + per : rows;
    const int64_t slab = (int64_t)n_in * rows * n_out, edge = (int64_t)i * n_out + j;

    // the input's segment rows, staged: rows look through them; and marks for the rows of the slice (2^mark_shift to a
    // bit) that have carry rows at all: in a long table few do
    __shared__ int seg_lds[kSegStage];
    __shared__ unsigned marks[kMarkBits / 32];
    const bool staged = cr.n_seg > 1 && n_chunks * cr.n_seg <= kSegStage;
    int mark_shift = 0;
    if (cr.n_seg > 1) {
        while (((m_hi - m_lo) >> mark_shift) >= kMarkBits) ++mark_shift;
        for (int e = tid; e < kMarkBits / 32; e += NT) marks[e] = 0u;
        __syncthreads();
        for (int e = tid; e < n_chunks * cr.n_seg; e += NT) {
            const int c = e / cr.n_seg, k = e - c * cr.n_seg;
            const int first = cr.seg_row[((int64_t)c * n_in + i) * cr.n_seg + k];
            if (staged) seg_lds[e] = first;
            const int lo = first > m_lo ? first : m_lo, hi = first + cr.window < m_hi ? first + cr.window : m_hi;
            for (int m = lo; m < hi; ++m) {
                const int bit = (m - m_lo) >> mark_shift;
                if (k > 0) atomicOr(&marks[bit >> 5], 1u << (bit & 31));
            }
        }
        __syncthreads();
    }
    auto marked = [&](int m) {
        const int bit = (m - m_lo) >> mark_shift;
        return ((marks[bit >> 5] >> (bit & 31)) & 1u) != 0u;
    };
    auto seg_first = [&](int c, int k) {
        return staged ? seg_lds[c * cr.n_seg + k] : cr.seg_row[((int64_t)c * n_in + i) * cr.n_seg + k];
    };

    double gs[T];
#pragma unroll
    for (int r = 0; r < T; ++r) gs[r] = 0.0;
    if (gcoef || gw_s) {
        float ws[T];
        reduce_load<T>(w_s + edge, ws);
        for (int m0 = m_lo; m0 < m_hi; m0 += R) {
            const int m = m0 + row;
            const bool live = m < m_hi;
            const int64_t at = ((int64_t)i * rows + (live ? m : m_lo)) * n_out + j;
            float cv[T];
#pragma unroll
            for (int r = 0; r < T; ++r) cv[r] = 0.0f;
            if (gw_s && share == 0) reduce_load<T>(coef + at, cv);
            double a[T];
#pragma unroll
            for (int r = 0; r < T; ++r) a[r] = 0.0;
            int c = share;
            for (; c + 7 * CS < n_chunks; c += 8 * CS) {          // eight chunks in flight
                float v[8][T];
#pragma unroll
                for (int u = 0; u < 8; ++u) reduce_load<T>(part_c + (c + u * CS) * slab + at, v[u]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int r = 0; r < T; ++r) a[r] += (double)v[u][r];
            }
            for (; c < n_chunks; c += 4 * CS) {                   // and four of the last ones
                float v[4][T];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c + u * CS < n_chunks) reduce_load<T>(part_c + (c + u * CS) * slab + at, v[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c + u * CS < n_chunks) {
#pragma unroll
                        for (int r = 0; r < T; ++r) a[r] += (double)v[u][r];
                    }
            }
            if (cr.n_seg > 1 && live && marked(m)) {
                // carry rows: segment k's rows start at seg_row[k] (non-decreasing in k), so those of row m are
                // neighbours: the first is searched for, then four at a time are read
                for (int c = share; c < n_chunks; c += CS) {
                    const int64_t list = ((int64_t)c * n_in + i) * cr.n_seg;
                    int k = 1, hi = cr.n_seg;                         // segment 0 has no carry rows
                    while (k < hi) {
                        const int mid = (k + hi) >> 1;
                        if (seg_first(c, mid) < m - (cr.window - 1)) k = mid + 1;
                        else hi = mid;
                    }
                    for (int hits = 4; hits == 4; k += 4) {
                        hits = 0;
                        float v[4][T];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int first = k + u < cr.n_seg ? seg_first(c, k + u) : INT_MAX;
                            if (first > m) continue;
                            ++hits;
                            reduce_load<T>(cr.carry + ((list + k + u) * cr.window + (m - first)) * n_out + j, v[u]);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (u < hits) {
#pragma unroll
                                for (int r = 0; r < T; ++r) a[r] += (double)v[u][r];
                            }
                    }
                }
            }
            if (CS > 1) tree_sum<T>(lds, tid, share, CS, R * LJ, a);
            if (share == 0 && live) {
                if (gcoef && jok) {
                    float o[T];
#pragma unroll
                    for (int r = 0; r < T; ++r) o[r] = (float)((double)ws[r] * a[r]);
                    reduce_store<T>(gcoef + at, o);
                }
#pragma unroll
                for (int r = 0; r < T; ++r) gs[r] += (double)cv[r] * a[r];
            }
        }
    }
    if (gw_s) {
        tree_sum<T>(lds, tid, grp, R, LJ, gs);          // shares past the first hold zeros and do not take part
        if (grp == 0 && jok) {
            if (slice_sums) {
#pragma unroll
                for (int r = 0; r < T; ++r) slice_sums[(int64_t)blockIdx.z * n_in * n_out + edge + r] = gs[r];
            } else {
                float o[T];
#pragma unroll
                for (int r = 0; r < T; ++r) o[r] = (float)gs[r];
                reduce_store<T>(gw_s + edge, o);
            }
        }
    }
    if (gw_b && blockIdx.z == 0) {
        double b[T];
#pragma unroll
        for (int r = 0; r < T; ++r) b[r] = 0.0;
        if (part_b) {
            const int64_t slice = (int64_t)n_in * n_out;
            const int step = R * CS;
            int s = grp;
            for (; s + 3 * step < n_slices_b; s += 4 * step) {
                float v[4][T];
#pragma unroll
                for (int u = 0; u < 4; ++u) reduce_load<T>(part_b + (s + u * step) * slice + edge, v[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int r = 0; r < T; ++r) b[r] += (double)v[u][r];
            }
            for (; s < n_slices_b; s += step) {
                float v[T];
                reduce_load<T>(part_b + s * slice + edge, v);
#pragma unroll
                for (int r = 0; r < T; ++r) b[r] += (double)v[r];
            }
        }
        tree_sum<T>(lds, tid, grp, R * CS, LJ, b);
        if (grp == 0 && jok) {
            float o[T];
#pragma unroll
            for (int r = 0; r < T; ++r) o[r] = (float)b[r];
            reduce_store<T>(gw_b + edge, o);
        }
    }
}

__global__ __launch_bounds__(256) void dparam_reduce_slices_kernel(const double *__restrict__ slice_sums,
                                                                   float *__restrict__ gw_s, int64_t edges, int n_rs)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= edges) return;
    double s = 0.0;
    for (int r = 0; r < n_rs; r += 8) {                // eight in flight, added in order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = r + u < n_rs ? slice_sums[(int64_t)(r + u) * edges + e] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    gw_s[e] = (float)s;
}

namespace {
int lanes_of(int n_out) { return n_out > 32 ? 16 : (n_out > 16 ? 8 : 4); }
int tiles_of(int n_out) { const int w = n_out < 4 ? 4 : lanes_of(n_out) * 4; return (n_out + w - 1) / w; }
// Row slices: as many workgroups as four for a CU, in slices of a power of two of rows, at least 32 (below, the extra kernel
// that adds the slices of gw_s costs more than they give; so it does for tables of up to 64 rows).  A workgroup's rows are
// one chain of reads: 2 -> 512, G = 100, B = 65536: 163 us in one slice, 57 and 6 in four.
constexpr int kSliceRows = 32;
int most_slices(int n_in, int n_out)
{
    const int64_t blocks = (int64_t)n_in * tiles_of(n_out);
    return (int)(blocks > 1024 ? 1 : 1024 / blocks);
}
int row_slices(int n_in, int rows, int n_out)
{
    if (rows <= 2 * kSliceRows) return 1;
    const int most = most_slices(n_in, n_out);
    int per = kSliceRows;
    while (per < rows && (rows + per - 1) / per > most) per *= 2;
    return (rows + per - 1) / per;
}

template <int T, int LJ, int NT>
void launch_reduce(dim3 grid, const float *part_c, const float *part_b, const CarryRows &cr, const float *coef,
                   const float *w_s, float *gcoef, float *gw_s, float *gw_b, double *slices, int n_in, int rows, int n_out,
                   int n_chunks, int n_slices_b, hipStream_t st)
{
    const int per = (rows + (int)grid.z - 1) / (int)grid.z;
    int R = 1;
    while (R < per && R < NT / LJ) R *= 2;
    dparam_reduce_kernel<T, LJ, NT><<<grid, NT, 0, st>>>(part_c, part_b, cr, coef, w_s, gcoef, gw_s, gw_b, slices, n_in, rows,
                                                         n_out, n_chunks, n_slices_b, R, NT / LJ / R);
}
}  // namespace

size_t reduce_scratch_bytes(int n_in, int rows, int n_out)
{
    // not what row_slices says but its bound: that of a shorter table must fit the space of a longer one
    const int most = most_slices(n_in, n_out), n = rows / kSliceRows + 1 < most ? rows / kSliceRows + 1 : most;
    return n > 1 ? (size_t)n * n_in * n_out * sizeof(double) : 0;
}

hipError_t launch_dparam_reduce(const float *part_c, const float *part_b, const CarryRows &cr, const float *coef,
                                const float *w_s, float *gcoef, float *gw_s, float *gw_b, int n_in, int rows, int n_out,
                                int n_chunks, int n_slices_b, void *scratch, hipStream_t st)
{
    if (!gcoef && !gw_s && !gw_b) return hipSuccess;
    const int n_rs = gw_s && !scratch ? 1 : row_slices(n_in, rows, n_out);
    double *slices = gw_s && n_rs > 1 ? (double *)scratch : nullptr;
    const dim3 grid((unsigned)n_in, (unsigned)tiles_of(n_out), (unsigned)n_rs);
    // few workgroups: large ones, whose chunk shares keep more of the partial tables in flight
    const bool big = (int64_t)grid.x * grid.y * grid.z < 512;
#define KAN_REDUCE(T, LJ)                                                                                                     \
    (big ? launch_reduce<T, LJ, 1024>(grid, part_c, part_b, cr, coef, w_s, gcoef, gw_s, gw_b, slices, n_in, rows, n_out,       \
                                      n_chunks, n_slices_b, st)                                                               \
         : launch_reduce<T, LJ, 256>(grid, part_c, part_b, cr, coef, w_s, gcoef, gw_s, gw_b, slices, n_in, rows, n_out,        \
                                     n_chunks, n_slices_b, st))
    {
        prof::Timed tm("dparam_reduce", st);
        if (n_out == 1) KAN_REDUCE(1, 1);
        else if (n_out == 2) KAN_REDUCE(1, 2);
        else if (n_out == 3) KAN_REDUCE(1, 4);
        else if (lanes_of(n_out) == 4) KAN_REDUCE(4, 4);
        else if (lanes_of(n_out) == 8) KAN_REDUCE(4, 8);
        else KAN_REDUCE(4, 16);
    }
#undef KAN_REDUCE
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (slices) {
        const int64_t edges = (int64_t)n_in * n_out;
        prof::Timed tm("dparam_reduce_slices", st);
        dparam_reduce_slices_kernel<<<(unsigned)((edges + 255) / 256), 256, 0, st>>>(slices, gw_s, edges, n_rs);
    }
    return hipGetLastError();
}

}  // namespace kan
