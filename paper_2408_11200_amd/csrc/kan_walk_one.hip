// Backward walk over cell lists (kan_quads.hpp) for layers of one output, windows of four rows.
//
// With one output the other walk's lanes <-> outputs mapping leaves fifteen lanes of sixteen idle.  Here lanes <-> quads: a
// workgroup takes the whole list of one (chunk, input), a lane the four entries of a quad, which share their window: its
// sums over the window's four rows need no other lane.  The quads of a cell stand in neighbouring lanes; a segmented sum over
// the wave leaves them in the cell's last lane, which adds them to the wave's own sums of that cell in LDS.  The waves' sums are
// combined in a fixed order, so the gradients are bit-reproducible.  The chunk's gy and the input's table sit in LDS.
//
// Bound by evaluating the pairs and, with dL/dx, by its scattered 4-byte stores: the inputs that share a line of gx are
// given to one XCD, whose L2 joins them.  256 -> 1, 244 rows, B = 32768: 204 -> 74 us (of it the stores of gx a third).
#include <type_traits>
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_quads.hpp"
#include "kan_wave.hpp"

namespace kan {

namespace {

constexpr int kOneInputs = 32;          // neighbouring inputs of one XCD: a 128-byte line of gx

template <bool DX, bool BASE>
__global__ __launch_bounds__(64 * kOneWaves) void walk_one_kernel(QuadWalkArgs p)
{
    constexpr int NT = 64 * kOneWaves;
    extern __shared__ float lds[];
    __shared__ float base_sum[kOneWaves];
    const int in_groups = (p.n_in + kOneInputs - 1) / kOneInputs;
    const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3, unit = k / kOneInputs * 8 + xcd, c = unit / in_groups;
    // (the groups of a chunk, if even in number, are turned each time they come round to the same XCDs, so that the last one, with fewer
    // inputs, does too)
    const int even = in_groups & -in_groups, turn = even == 1 ? 0 : c * (even < 8 ? even : 8) / 8;
    const int i = (unit + turn) % in_groups * kOneInputs + k % kOneInputs;
    if (c >= p.n_chunks || i >= p.n_in) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cells = p.rows - kMaxK + 1;
    float4 *sums = reinterpret_cast<float4 *>(lds);                    // [wave][cell]: over the window's rows
    float *gyl = lds + 4 * kOneWaves * cells, *tab = gyl + p.S;
    SplineGeom g;
    g.n_in = p.n_in; g.n_out = 1; g.rows = p.rows; g.slab_rows = p.slab_rows; g.k = p.k; g.lo = p.lo; g.inv_h = p.inv_h;
    g.cell_base = p.cell_base; g.base_act = BASE ? 1 : 0;
    const int64_t b0 = (int64_t)c * p.S;
    const int n_c = (int)((p.B - b0) < p.S ? (p.B - b0) : p.S);
    for (int e = tid; e < kOneWaves * cells; e += NT) sums[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int e = tid; e < n_c; e += NT) gyl[e] = p.gy[b0 + e];
    float wb = 0.0f;
    if constexpr (DX) {
        for (int m = tid; m < p.rows; m += NT) tab[m] = p.cf[(int64_t)i * p.slab_rows + m];
        if constexpr (BASE) wb = p.w_b[i];
    }
    __syncthreads();

    const int64_t li = (int64_t)c * p.n_in + i, list = li * p.lists.L;
    const int nq = p.lists.n_quads[li], per = ((nq + kOneWaves - 1) / kOneWaves + 63) / 64 * 64;
    const int q_end = (wave + 1) * per < nq ? (wave + 1) * per : nq;
    float4 *mine = sums + wave * cells;
    float ab = 0.0f;
    float4 xn;
    ushort4 sn;
    auto fetch = [&](int q0) {                                         // a round ahead
        const int64_t at = list + 4 * (int64_t)(q0 + lane < q_end ? q0 + lane : q_end - 1);
        xn = *reinterpret_cast<const float4 *>(p.lists.x + at);
        sn = *reinterpret_cast<const ushort4 *>(p.lists.sample + at);
    };
    if (wave * per < q_end) fetch(wave * per);
    for (int q0 = wave * per; q0 < q_end; q0 += 64) {
        const bool live = q0 + lane < q_end;
        const float4 xq = xn;
        const ushort4 sq = sn;
        if (q0 + 64 < q_end) fetch(q0 + 64);
        const float xs[4] = {xq.x, xq.y, xq.z, xq.w};
        const unsigned ss[4] = {sq.x, sq.y, sq.z, sq.w};
        float v[kMaxK] = {0.0f, 0.0f, 0.0f, 0.0f}, tv[kMaxK], bsum = 0.0f;
        int row = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = live && ss[u] != kQuadPad;                 // a quad's first entry is a sample's
            float w[kMaxK], dw[kMaxK], base, dbase;
            int row0;
            wave_windows<DX>(ss[u] != kQuadPad ? xs[u] : xs[0], g, i, row0, w, base, dw, dbase);
            if (u == 0) {
                row = row0;
                if constexpr (DX)
#pragma unroll
                    for (int s = 0; s < kMaxK; ++s) tv[s] = tab[row0 + s];
            }
            const float gv = ok ? gyl[ss[u]] : 0.0f;
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) v[s] = ok ? fmaf(w[s], gv, v[s]) : v[s];
            if constexpr (BASE) bsum = ok ? fmaf(base, gv, bsum) : bsum;
            if constexpr (DX) {
                float d = 0.0f;
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) d = fmaf(dw[s], tv[s], d);
                if constexpr (BASE) d = fmaf(dbase, wb, d);
                if (ok) p.gx[(b0 + ss[u]) * p.n_in + i] = gv * d;
            }
        }
        ab += bsum;
        if (!live) row = -1;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const bool same = __shfl_up(row, d) == row && lane >= d;
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) {
                const float t = __shfl_up(v[s], d);
                v[s] = same ? v[s] + t : v[s];
            }
        }
        const int after = __shfl_down(row, 1);
        if (live && (lane == 63 || after != row)) {
            const float4 o = mine[row];
            mine[row] = make_float4(o.x + v[0], o.y + v[1], o.z + v[2], o.w + v[3]);
        }
        wave_lds_sync();                   // the next round's lanes read what these wrote
    }
    if constexpr (BASE) {
#pragma unroll
        for (int d = 32; d > 0; d /= 2) ab += __shfl_xor(ab, d);
        if (lane == 0) base_sum[wave] = ab;
    }
    __syncthreads();
    if (p.part_c)
        for (int m = tid; m < p.rows; m += NT) {
            float t = 0.0f;
            for (int w = 0; w < kOneWaves; ++w)
#pragma unroll
                for (int s = 0; s < kMaxK; ++s) {
                    const int cell = m - s;
                    if (cell >= 0 && cell < cells) t += reinterpret_cast<const float *>(sums + w * cells + cell)[s];
                }
            p.part_c[li * p.rows + m] = t;
        }
    if (p.part_b && tid == 0) {
        float t = 0.0f;
        if constexpr (BASE)
            for (int w = 0; w < kOneWaves; ++w) t += base_sum[w];
        p.part_b[li] = t;
    }
}

}  // namespace

hipError_t walk_one(const QuadWalkArgs &a, hipStream_t st)
{
    const size_t bytes = walk_one_lds_bytes(a.rows, a.S);
    const int64_t units = (int64_t)a.n_chunks * ((a.n_in + kOneInputs - 1) / kOneInputs);
    const unsigned blocks = (unsigned)((units + 7) / 8 * 8 * kOneInputs);
    auto launch = [&](auto dx, auto base) {
        constexpr bool DX = decltype(dx)::value, BASE = decltype(base)::value;
        struct Tag {};
        if (hipError_t e = ensure_dynamic_lds<Tag>((const void *)walk_one_kernel<DX, BASE>, (int)bytes); e != hipSuccess) return e;
        walk_one_kernel<DX, BASE><<<blocks, 64 * kOneWaves, bytes, st>>>(a);
        return hipGetLastError();
    };
    auto by_base = [&](auto dx) { return a.base_act != 0 ? launch(dx, std::true_type{}) : launch(dx, std::false_type{}); };
    return a.gx ? by_base(std::true_type{}) : by_base(std::false_type{});
}

}  // namespace kan
