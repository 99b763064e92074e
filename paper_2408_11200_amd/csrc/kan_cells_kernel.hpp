// Cell lists of the quad walk (kan_quads.hpp), for the window of the including translation unit.
//
// One workgroup orders the samples of one (chunk, input) by window row: one counting pass over the row field (kan_sort.hpp)
// whose slots start at a multiple of four for every row, so the runs come out filled up to quads; the values and sample
// indexes are placed in LDS and written out in order.  Bound by the LDS round trips of the counting and by the lists written, 6
// bytes an entry.
#pragma once
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_quads.hpp"
#include "kan_sort.hpp"

namespace KAN_NS {

namespace {

using ::kan::kQuadPad;
using ::kan::QuadWalkArgs;

// grid (n_chunks, n_in), NW waves; S / NW samples a wave, a multiple of 64
template <int NW>
__global__ __launch_bounds__(64 * NW) void cell_list_kernel(QuadWalkArgs p, const float *__restrict__ xT, int row_bits)
{
    constexpr int NT = 64 * NW;
    extern __shared__ unsigned lds_u[];
    __shared__ unsigned wave_total[NW];
    const int L = p.lists.L, bins = 1 << row_bits;
    float *xd = reinterpret_cast<float *>(lds_u);
    unsigned *counters = lds_u + L;
    uint16_t *sd = reinterpret_cast<uint16_t *>(counters + (NW / 2) * bins);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = blockIdx.x, i = blockIdx.y;
    const int64_t b0 = (int64_t)c * p.S;
    const int n_c = (int)((p.B - b0) < p.S ? (p.B - b0) : p.S);
    SplineGeom g;
    g.n_in = p.n_in; g.n_out = p.n_out; g.rows = p.rows; g.slab_rows = p.slab_rows; g.k = p.k; g.lo = p.lo; g.inv_h = p.inv_h;
    g.cell_base = p.cell_base; g.base_act = p.base_act;

    const int per_wave = p.S / NW, nb = per_wave / 64, half = (wave & 1) * 16;
    unsigned *mine = counters + (wave >> 1) * bins;
    float xv[kSortMaxBatches];
    unsigned row[kSortMaxBatches], off[kSortMaxBatches];
#pragma unroll
    for (int u = 0; u < kSortMaxBatches; ++u) {
        const int e = wave * per_wave + u * 64 + lane;
        xv[u] = u < nb && e < n_c ? xT[(int64_t)i * p.B + b0 + e] : 0.0f;
    }
    for (int e = tid; e < (NW / 2) * bins; e += NT) counters[e] = 0u;
    for (int e = tid; e < L; e += NT) { xd[e] = 0.0f; sd[e] = (uint16_t)kQuadPad; }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortMaxBatches; ++u)
        if (u < nb) {
            row[u] = (unsigned)window_row(xv[u], g, i);
            off[u] = count_digit(mine, half, row[u], row_bits, wave * per_wave + u * 64 + lane < n_c, lane);
        }
    __syncthreads();
    const int total = (int)slots_of_counts<NW, true>(counters, bins, wave_total);
#pragma unroll
    for (int u = 0; u < kSortMaxBatches; ++u) {
        const int e = wave * per_wave + u * 64 + lane;
        if (u < nb && e < n_c) {
            const unsigned at = ((mine[row[u]] >> half) & 0xffffu) + off[u];
            xd[at] = xv[u];
            sd[at] = (uint16_t)e;
        }
    }
    __syncthreads();
    const int64_t li = (int64_t)c * p.n_in + i;
    float *ox = p.lists.x + li * L;
    uint16_t *os = p.lists.sample + li * L;
    if (tid == 0) p.lists.n_quads[li] = total / 4;
    for (int e = tid * 4; e < total; e += NT * 4) {
        *reinterpret_cast<float4 *>(ox + e) = *reinterpret_cast<const float4 *>(xd + e);
        *reinterpret_cast<uint2 *>(os + e) = *reinterpret_cast<const uint2 *>(sd + e);
    }
}

template <int NW>
hipError_t launch_cell_list(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st)
{
    struct Tag;
    const size_t lds = (size_t)a.lists.L * 6 + ((size_t)(NW / 2) * 4 << row_bits);
    auto kern = cell_list_kernel<NW>;
    if (hipError_t e = ensure_dynamic_lds<Tag>(reinterpret_cast<const void *>(kern), (int)lds); e != hipSuccess) return e;
    const dim3 grid((unsigned)((a.B + a.S - 1) / a.S), (unsigned)a.n_in);
    prof::Timed tm("walk_cells", st);
    kern<<<grid, 64 * NW, lds, st>>>(a, xT, row_bits);
    return hipGetLastError();
}

// waves a list: 16 for chunks of 8192 samples, 8 for 4096, 4 below
hipError_t launch_cell_list_by_size(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st)
{
    return a.S >= 8192   ? launch_cell_list<16>(a, xT, row_bits, st)
           : a.S >= 4096 ? launch_cell_list<8>(a, xT, row_bits, st)
                         : launch_cell_list<4>(a, xT, row_bits, st);
}

}  // namespace

}  // namespace KAN_NS
