// The walk over cell lists padded to quads, and its launcher template.  Every (streams a wave, outputs a lane) variant is
// built in a translation unit of its own (kan_quads_s*t*.hip, kan_quads6_s*t*.hip for windows of six rows).
//
// Four consecutive entries of a list share their window rows, so a quad is the unit of work:
//   - one look at the window, one set of LDS reads and no per-record control flow;
//   - the parameter gradients are four rank-1 updates on the matrix cores (v_mfma_f32_4x4x1: A = the sample's weights,
//     B = the lane's gy), dL/dx one rank-1 update per window row for all four samples (A = their dw, B = the lane's table
//     entry) and four multiply-adds per output;
//   - the basis is evaluated here, one entry a lane and a batch of 64 entries a wave, and handed to the quads through a
//     small area of LDS owned by the wave, so a list is 6 bytes a pair instead of 44.
// A pad entry's gy row lies outside the buffer the gather names, which reads as zeros: nothing is fetched for it and no
// value of another sample takes part.
//
// Bound by the fp32 units: an instruction of 4x4x1 takes 10 clocks and does not overlap with another, a multiply-add beside it
// costs 1.5 more (their own rate: 3.5), but one between two of them about 5, so the loop has the two kinds in blocks.  With no
// gy read at all 512 -> 512 takes 1077 us of 1181.  Walk against the one over records, us: 512 -> 512, G = 20, B = 16384 1475 /
// 1149 (mixed instead of in blocks 1444), 256 -> 256, G = 200, B = 8192 285 / 210, 64 -> 64, G = 10, B = 65536 150 / 127,
// 32 -> 32, G = 1024, B = 131072 270 / 169, 32 -> 32, G = 64, k = 5, B = 65536 108 / 82, 128 -> 256 -> 256 -> 1 with tables of
// 360 rows, B = 32768 2000 / 1464; the lists (walk_cells) against the records of the sort: 90 / 29, 25 / 15, 53 / 22, 60 / 31,
// 76 / 15, 288 / 138.  An evaluation
// is 100 .. 200 instructions a batch of 64 entries, as much as the quads of a narrow layer: without masks and shifts inside the table
// (wave_windows) the whole pass went 181 -> 168 (32 -> 32, k = 5), 376 -> 371 (G = 1024), 626 -> 622 (256 -> 256).
#pragma once
#include <type_traits>
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_quads.hpp"
#include "kan_wave.hpp"

namespace KAN_NS {

namespace {

using ::kan::QuadWalkArgs;
using ::kan::kQuadPad;

constexpr int kWinRegs = (kMaxK + 3) / 4;          // accumulator quadruples of a window
constexpr int kWinSlots = 4 * kWinRegs;
// byte offsets past every chunk's gy, which is 2^30 bytes at most (plan_walk): of a pad entry's row, and of a lane without
// outputs; the sum of either with a real offset, or of both, lies outside too
constexpr unsigned kPadOffset = 0x80000000u, kIdleOffset = 0x40000000u;

template <int VT>
__device__ __forceinline__ void gather_vec(i32x4 rsrc, unsigned off, float *v)
{
    if constexpr (VT == 4) {
        const f32x4 t = buffer_load4(rsrc, (int)off, 0, 0);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else if constexpr (VT == 2) {
        const f32x2 t = buffer_load2(rsrc, (int)off, 0, 0);
        v[0] = t.x; v[1] = t.y;
    } else {
        static_assert(VT == 1, "one, two or four outputs");
        v[0] = buffer_load1(rsrc, (int)off, 0, 0);
    }
}

// A wave's evaluated batch: 64 entries, 16 quads.
template <int STREAMS, bool DX, bool BASE>
struct alignas(16) QuadArea {
    float w[16][kWinSlots][4];                     // [quad][window slot][sample of the quad]
    float dw[DX ? 64 : 1][kWinSlots];              // [entry][window slot]
    float base[BASE ? 64 : 4];
    float dbase[DX && BASE ? 64 : 4];
    unsigned off[STREAMS][64 / STREAMS + 4];       // byte offset of the sample's gy row in the chunk; a quad of pads follows
    unsigned sample[64];
    int row[16];                                   // first window row of the quad, -1 past the end
};

}  // namespace

// 4 waves a workgroup, STREAMS streams a wave (one (chunk, input, output tile, segment) each), T outputs a lane in groups of
// up to four neighbours.  FOLD: sums in two levels, folded every 256 entries, so that a long run of samples in one cell does
// not lose accuracy to sequential fp32 accumulation.  RAGGED: n_out is no multiple of the group; the lane of the last outputs
// is moved back to end with the row, its outputs are computed twice from the same operands and counted once in dL/dx.
template <int STREAMS, int T, bool DX, bool FOLD, bool RAGGED, bool BASE>
__global__ __launch_bounds__(256) void quad_walk_kernel(QuadWalkArgs p)
{
    constexpr int LPS = 64 / STREAMS, QPB = LPS / 4;           // lanes a stream; quads of a stream's batch
    constexpr int VT = T < 4 ? T : 4, NG = T / VT;
    __shared__ QuadArea<STREAMS, DX, BASE> areas[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane / LPS, q = lane % LPS, l4 = lane & 3;
    // Workgroups go to the 8 XCDs round-robin.  The XCDs form m = min(8, n_chunks) groups (m a power of two); chunk c is
    // handled by group c % m only, so that the gy rows a chunk's streams gather (every input re-reads them) stay in the
    // L2 of the XCDs of one group.
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int grp = xcd % p.xcd_groups, n_sub = 8 / p.xcd_groups, sub_x = xcd / p.xcd_groups;
    const int bpc_sub = (p.blocks_per_chunk + n_sub - 1) / n_sub;
    const int c_local = grp + p.xcd_groups * (slot / bpc_sub);
    const int c = p.chunk0 + c_local;
    const int blk = (slot % bpc_sub) * n_sub + sub_x;
    const int n_work = p.n_seg * p.n_jt * p.n_in;
    const int ws0 = (blk * 4 + wave) * STREAMS;
    if (c_local >= p.n_chunks || blk >= p.blocks_per_chunk || ws0 >= n_work) return;
    // streams past the last one repeat its work on an empty range and store nothing
    const bool real = ws0 + sub < n_work;
    const int ws = real ? ws0 + sub : n_work - 1;
    const int i = ws % p.n_in;
    const int jt = (ws / p.n_in) % p.n_jt;
    const int seg = ws / (p.n_in * p.n_jt);
    SplineGeom g;
    g.n_in = p.n_in; g.n_out = p.n_out; g.rows = p.rows; g.slab_rows = p.slab_rows; g.k = p.k; g.lo = p.lo; g.inv_h = p.inv_h;
    g.cell_base = p.cell_base; g.base_act = BASE ? 1 : 0;

    int jg[NG], skip[NG];                  // first output of a group; leading outputs that are the neighbour's too
    bool jok[NG];
#pragma unroll
    for (int v = 0; v < NG; ++v) {
        const int jl = jt * (LPS * T) + (v * LPS + q) * VT;
        jok[v] = real && jl < g.n_out;
        const int j = RAGGED && jl + VT > g.n_out ? g.n_out - VT : jl;
        skip[v] = RAGGED ? jl - j : 0;
        jg[v] = jok[v] ? j : 0;
    }
    const int64_t b0 = (int64_t)c * p.S;
    const int n_c = (int)((p.B - b0) < p.S ? (p.B - b0) : p.S);
    const unsigned row_bytes = (unsigned)g.n_out * 4u;
    const i32x4 gyr = buffer_of(p.gy + b0 * g.n_out, (unsigned)n_c * row_bytes);
    unsigned lane_off[NG];
#pragma unroll
    for (int v = 0; v < NG; ++v) lane_off[v] = jok[v] ? (unsigned)jg[v] * 4u : kIdleOffset;

    // the segment's entries: quads seg * nq / n_seg .. (seg + 1) * nq / n_seg of the list
    const int64_t li = (int64_t)c * g.n_in + i, list = li * p.lists.L;
    const int nq = p.lists.n_quads[li];
    const int e0 = (int)((int64_t)seg * nq / p.n_seg) * 4;
    const int e_next = (int)((int64_t)(seg + 1) * nq / p.n_seg) * 4;
    const int e1 = real ? e_next : e0;
    const float *lx = p.lists.x + list;
    const uint16_t *ls = p.lists.sample + list;
    // The segment owns the table rows from its first entry's row up to the next segment's first row; what its window holds
    // beyond that at the end goes to the next segment's carry rows.
    int cur = window_row(lx[e0], g, i);            // first row of the window the accumulators stand on
    const int r_next = seg + 1 < p.n_seg ? window_row(lx[e_next], g, i) : g.rows;
    if constexpr (STREAMS == 1) cur = __builtin_amdgcn_readfirstlane(cur);
    const bool want_c = real && p.part_c != nullptr;
    float *out = p.part_c + ((int64_t)c_local * g.n_in + i) * g.rows * g.n_out;
    // the table dL/dx reads: the input's slab where the wave has one input, else all of it (both 2^30 bytes at most, plan_walk)
    const int slab_bytes = g.slab_rows * g.n_out * 4;
    const i32x4 cfr = STREAMS == 1 ? buffer_of(p.cf + (int64_t)i * g.slab_rows * g.n_out, (unsigned)slab_bytes)
                                   : buffer_of(p.cf, (unsigned)(g.n_in * slab_bytes));
    const unsigned cf0 = STREAMS == 1 ? 0u : (unsigned)(i * slab_bytes);
    if (p.part_c != nullptr && real && p.n_seg > 1 && jt == 0 && q == 0) p.seg_row[li * p.n_seg + seg] = cur;

    // a[r]: running sums of output r over the window slots; hi: the second level
    constexpr int TH = FOLD ? T : 1;
    f32x4 a[T][kWinRegs], hi[TH][kWinRegs];
    float ab[T], abh[TH], zero[T];
#pragma unroll
    for (int r = 0; r < T; ++r) {
        ab[r] = 0.0f; zero[r] = 0.0f;
#pragma unroll
        for (int h = 0; h < kWinRegs; ++h) a[r][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int r = 0; r < TH; ++r) {
        abh[r] = 0.0f;
#pragma unroll
        for (int h = 0; h < kWinRegs; ++h) hi[r][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    auto store_row = [&](float *row, const float (&v)[T]) {
#pragma unroll
        for (int n = 0; n < NG; ++n)
            if (jok[n]) {
                if constexpr (VT == 4) store4u(row + jg[n], make_float4(v[4 * n], v[4 * n + 1], v[4 * n + 2], v[4 * n + 3]));
                else if constexpr (VT == 2) store2u(row + jg[n], make_float2(v[0], v[1]));
                else row[jg[n]] = v[0];
            }
    };
    auto load_row = [&](i32x4 rsrc, unsigned off, float (&v)[T]) {          // zero where an output is not the lane's own
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            gather_vec<VT>(rsrc, off + lane_off[n], &v[n * VT]);
            if constexpr (RAGGED) {
#pragma unroll
                for (int r = 0; r < VT; ++r) v[n * VT + r] = r < skip[n] ? 0.0f : v[n * VT + r];
            }
        }
    };
    if (want_c && !p.prezeroed && seg == 0)
        for (int m = 0; m < cur; ++m) store_row(out + (int64_t)m * g.n_out, zero);

    // dL/dx: table rows cur .. cur + K - 1 in their slots, the row that enters next, and the w_b row
    float cw[kWinSlots][T], nxt[T], wb[T];
    if constexpr (DX) {
#pragma unroll
        for (int r = 0; r < T; ++r) wb[r] = 0.0f;
        if constexpr (BASE) load_row(buffer_of(p.w_b, (unsigned)g.n_in * row_bytes), (unsigned)i * row_bytes, wb);
#pragma unroll
        for (int s = kMaxK; s < kWinSlots; ++s)
#pragma unroll
            for (int r = 0; r < T; ++r) cw[s][r] = 0.0f;
    }
    auto table_row = [&](int row, float (&v)[T]) { load_row(cfr, cf0 + (unsigned)row * row_bytes, v); };
    auto load_next = [&]() {               // row cur + K; clamped: unused past the end
        if constexpr (DX) table_row(cur + kMaxK < g.rows ? cur + kMaxK : g.rows - 1, nxt);
    };
    auto reload_window = [&]() {
        if constexpr (DX) {
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) table_row(cur + s, cw[s]);
            // waited for here: a load that may still be under way would make every quad wait for the gathers as well
#pragma unroll
            for (int s = 0; s < kMaxK; ++s)
#pragma unroll
                for (int r = 0; r < T; ++r) asm volatile("" : "+v"(cw[s][r]));
            load_next();
        }
    };
    auto put_row = [&](int row, const float (&v)[T]) {
        float *dst = out + (int64_t)row * g.n_out;
        if (p.shared) {
            // uniform.  Add to what earlier launches left in the row: within a launch this stream is the row's only
            // writer and launches follow each other on the stream, so the sum is the same every run; the hardware add
            // does not wait for the old value.
#pragma unroll
            for (int n = 0; n < NG; ++n)
                if (jok[n])
#pragma unroll
                    for (int r = 0; r < VT; ++r)
                        if (!RAGGED || r >= skip[n]) unsafeAtomicAdd(dst + jg[n] + r, v[n * VT + r]);
        } else {
            store_row(dst, v);
        }
    };
    // completes the first row of the window (store: writes it out, else it is left in `gone`) and lets the next one in
    float gone[T];
    auto retire = [&](bool store) {
#pragma unroll
        for (int r = 0; r < T; ++r) gone[r] = FOLD ? a[r][0][0] + hi[FOLD ? r : 0][0][0] : a[r][0][0];
        if (store && want_c) put_row(cur, gone);
#pragma unroll
        for (int s = 0; s < kMaxK; ++s)
#pragma unroll
            for (int r = 0; r < T; ++r) {
                constexpr int Z = kMaxK - 1;
                const int t = s < Z ? s + 1 : s;
                a[r][s / 4][s % 4] = s < Z ? a[r][t / 4][t % 4] : 0.0f;
                if constexpr (FOLD) hi[r][s / 4][s % 4] = s < Z ? hi[r][t / 4][t % 4] : 0.0f;
                if constexpr (DX) cw[s][r] = s < Z ? cw[t][r] : nxt[r];
            }
        ++cur;
        load_next();
    };
    // moves the window to `row`
    auto advance = [&](int row) {
        retire(true);                       // most often the next cell: of its own, it waits for an older load only
        const int flush = cur + kMaxK - 1;
#pragma clang loop unroll(disable)
        while (cur < row && cur < flush) retire(true);
        if (cur < row) {
            // clear of its old position; the rows in between are zero (stored here, or already zero)
            if (want_c && !p.prezeroed)
                for (int m = cur; m < row; ++m) store_row(out + (int64_t)m * g.n_out, zero);
            cur = row;
            reload_window();
        }
    };

    // entries of a batch: fetch() asks for the list's, evaluate() turns them into the quads' operands.  Returned: bit
    // sub * LPS + 4 b is set where quad b (b > 0) of the stream stands on another row than the quad before it.
    QuadArea<STREAMS, DX, BASE> &ar = areas[wave];
    float fx = 0.0f;
    unsigned fs = kQuadPad;
    int fe = 0;
    auto fetch = [&](int bi) {
        fe = e0 + bi * LPS + q;
        const int at = fe < e1 ? fe : e0;
        fx = lx[at];
        fs = ls[at];
    };
    auto evaluate = [&]() {
        const bool in = fe < e1, live = in && fs != kQuadPad;
        float w[kMaxK], dw[kMaxK], base, dbase;
        int row0;
        if constexpr (T < 8) {
            // A pad takes the x of its quad's first entry, which is none: stored as zero, one pad in a batch would put the whole wave
            // on the masked way wherever the table does not hold zero
            const float first = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, fx), 0, 0xF, 0xF, true));
            wave_windows<DX>(fs == kQuadPad ? first : fx, g, i, row0, w, base, dw, dbase);
        } else {                            // 512 outputs share an evaluation: two ways of it gain nothing (2158 .. 2295 us either way)
            const Pair pr = pair_eval<DX>(fx, g, i);
            window_of<false>(pr, g.rows, row0, w, base);
            if constexpr (DX) window_of<true>(pr, g.rows, row0, dw, dbase);
        }
#pragma unroll
        for (int s = 0; s < kWinSlots; ++s) ar.w[lane >> 2][s][l4] = s < kMaxK && live ? w[s < kMaxK ? s : 0] : 0.0f;
        if constexpr (DX) {
#pragma unroll
            for (int h = 0; h < kWinRegs; ++h) {
                float t[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) t[s] = 4 * h + s < kMaxK ? dw[4 * h + s < kMaxK ? 4 * h + s : 0] : 0.0f;
                *reinterpret_cast<float4 *>(&ar.dw[lane][4 * h]) = make_float4(t[0], t[1], t[2], t[3]);
            }
            if constexpr (BASE) ar.dbase[lane] = dbase;
        }
        if constexpr (BASE) ar.base[lane] = live ? base : 0.0f;
        ar.off[sub][q] = live ? fs * row_bytes : kPadOffset;
        ar.sample[lane] = live ? fs : kQuadPad;
        const int before = __shfl_up(row0, 4, 64);
        if (l4 == 0) ar.row[lane >> 2] = in ? row0 : -1;
        return __ballot(l4 == 0 && in && row0 != before);
    };
    auto gather = [&](uint4 o, float (&dst)[4][T]) {
        const unsigned ro[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int n = 0; n < NG; ++n) gather_vec<VT>(gyr, ro[u] + lane_off[n], &dst[u][n * VT]);
    };
    float res = 0.0f;                      // dL/dx of one entry of the batch (the lane's position says which)
    float gr[4][T];                        // gy rows of the quad, asked for a quad ahead
    auto work = [&](int b) {
        // the quad's operands: dw of sample l4, weights of slot l4 for the four samples
        const int qd = sub * QPB + b;
        const uint4 next = *reinterpret_cast<const uint4 *>(&ar.off[sub][(b + 1) * 4]);
        f32x4 wq[kWinRegs], dq[kWinRegs], bs = {0.0f, 0.0f, 0.0f, 0.0f}, qv[T];
        float db = 0.0f;
#pragma unroll
        for (int h = 0; h < kWinRegs; ++h) {
            if constexpr (DX) dq[h] = *reinterpret_cast<const f32x4 *>(&ar.dw[qd * 4 + l4][4 * h]);
            wq[h] = *reinterpret_cast<const f32x4 *>(&ar.w[qd][4 * h + l4][0]);
        }
        if constexpr (DX && BASE) db = ar.dbase[qd * 4 + l4];
        if constexpr (BASE) bs = *reinterpret_cast<const f32x4 *>(&ar.base[qd * 4]);
        // Matrix-core instructions first, then the multiply-adds: both run on the fp32 units and do not overlap, and a switch
        // between the two costs about five clocks
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (DX) {
#pragma unroll
            for (int r = 0; r < T; ++r) qv[r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < kMaxK; ++s)
#pragma unroll
                for (int r = 0; r < T; ++r)
                    qv[r] = __builtin_amdgcn_mfma_f32_4x4x1f32(dq[s / 4][s % 4], cw[s][r], qv[r], 0, 0, 0);
            if constexpr (BASE) {
#pragma unroll
                for (int r = 0; r < T; ++r) qv[r] = __builtin_amdgcn_mfma_f32_4x4x1f32(db, wb[r], qv[r], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int h = 0; h < kWinRegs; ++h)
#pragma unroll
                for (int r = 0; r < T; ++r)
                    a[r][h] = __builtin_amdgcn_mfma_f32_4x4x1f32(wq[h][u], gr[u][r], a[r][h], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (BASE) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int r = 0; r < T; ++r) ab[r] = fmaf(bs[u], gr[u][r], ab[r]);
        }
        float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (DX) {
#pragma unroll
            for (int r = 0; r < T; ++r)
#pragma unroll
                for (int u = 0; u < 4; ++u) dot[u] = fmaf(gr[u][r], qv[r][u], dot[u]);
        }
        // after the last use of gr (the sums are pinned above it), so that the next quad's rows come into the same registers
#pragma unroll
        for (int r = 0; r < T; ++r) asm volatile("" : "+v"(ab[r]));
#pragma unroll
        for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(dot[u]));
        __builtin_amdgcn_sched_barrier(0);
        gather(next, gr);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (DX) {
            // lanes of quarter n of the stream end up with sample n of the quad; the one at position b keeps it
            const float total = reduce_levels<LPS / 2, 4>(dot, lane);
            res = q % QPB == b ? total : res;
        }
    };

    // Quads of the longest of the wave's streams.  The last batch ends with them: short segments, whose pads make one batch into
    // a little more than one, walked 16 quads for the one or two left (backward pass, B = 3399, 66 -> 256, G = 14: 93 us,
    // 78 without them; records took 87)
    int n_quads = (e1 - e0) / 4;
#pragma unroll
    for (int d = LPS; d < 64; d *= 2) {
        const int o = __shfl_xor(n_quads, d, 64);
        n_quads = o > n_quads ? o : n_quads;
    }
    n_quads = __builtin_amdgcn_readfirstlane(n_quads);
    const int nb = (n_quads + QPB - 1) / QPB;
    unsigned long long streams = 0;        // bit 0 of every stream's lanes
#pragma unroll
    for (int s = 0; s < STREAMS; ++s) streams |= 1ull << (s * LPS);
    if (q < 4) ar.off[sub][LPS + q] = kPadOffset;
    reload_window();
    fetch(0);
    for (int bi = 0; bi < nb; ++bi) {
        const unsigned long long turns = evaluate();
        fetch(bi + 1);
        wave_lds_sync();
        gather(*reinterpret_cast<const uint4 *>(&ar.off[sub][0]), gr);
        // the quads between two moves of a window are a loop of their own, whose registers stay where they are
        const int here = n_quads - bi * QPB < QPB ? n_quads - bi * QPB : QPB;
        int b = 0;
        do {
            int row = ar.row[sub * QPB + b];
            if constexpr (STREAMS == 1) row = __builtin_amdgcn_readfirstlane(row);
            if (row > cur) advance(row);
#pragma clang loop unroll(disable)
            do work(b);
            while (++b < here && ((turns >> (4 * b)) & streams) == 0);
        } while (b < here);                 // (tested behind: the first quad is there, and a way past it costs the folded builds a copy of their sums)
        if constexpr (DX) {
            // lane -> entry 4 * (position in its quarter) + quarter of the stream's batch
            const unsigned smp = ar.sample[sub * LPS + (q % QPB) * 4 + q / QPB];
            float *gxo = p.gx + (int64_t)jt * p.B * g.n_in + b0 * g.n_in + i;
            if (smp != kQuadPad) gxo[(int64_t)smp * g.n_in] = res;
        }
        if constexpr (FOLD) {
            if ((bi + 1) % (256 / LPS) == 0) {
#pragma unroll
                for (int r = 0; r < T; ++r) {
#pragma unroll
                    for (int h = 0; h < kWinRegs; ++h) {
                        hi[r][h] += a[r][h];
                        a[r][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                    abh[r] += ab[r]; ab[r] = 0.0f;
                }
            }
        }
        wave_lds_sync();
    }

    if (!want_c) return;
    // what the window still holds: rows below r_next belong to this segment, the others to the next segment's carry rows
    // (carry row s2 stands for table row r_next + s2)
    float *cr = p.carry + ((li * p.n_seg + seg + 1) * kMaxK) * (int64_t)g.n_out;
    const int last = cur + kMaxK;            // one past the window
    for (int s = 0; s < kMaxK; ++s) {
        const int row = cur;
        retire(row < r_next);
        if (row >= r_next && seg + 1 < p.n_seg) store_row(cr + (int64_t)(row - r_next) * g.n_out, gone);
    }
    if (seg + 1 < p.n_seg)
        for (int s2 = (last > r_next ? last - r_next : 0); s2 < kMaxK; ++s2) store_row(cr + (int64_t)s2 * g.n_out, zero);
    if (!p.prezeroed)
        for (int m = last; m < r_next; ++m) store_row(out + (int64_t)m * g.n_out, zero);
    if (p.part_b) {
        float o[T];
#pragma unroll
        for (int r = 0; r < T; ++r) o[r] = FOLD ? ab[r] + abh[r < TH ? r : 0] : ab[r];
        store_row(p.part_b + (((int64_t)c * p.n_seg + seg) * g.n_in + i) * g.n_out, o);
    }
}

namespace {

template <int STREAMS, int T, bool DX, bool FOLD, bool RAGGED>
void quad_walk_by_base(const QuadWalkArgs &a, unsigned blocks, hipStream_t st)
{
    if (a.base_act != 0) quad_walk_kernel<STREAMS, T, DX, FOLD, RAGGED, true><<<blocks, 256, 0, st>>>(a);
    else quad_walk_kernel<STREAMS, T, DX, FOLD, RAGGED, false><<<blocks, 256, 0, st>>>(a);
}

template <int STREAMS, int T>
void quad_walk_launch(const QuadWalkArgs &a, unsigned blocks, hipStream_t st)
{
    const bool ragged = a.n_out % (T < 4 ? T : 4) != 0, fold = a.S > 1024, dx = a.gx != nullptr;
    auto by_fold = [&](auto rag, auto d) {
        constexpr bool R = decltype(rag)::value, D = decltype(d)::value;
        if (fold) quad_walk_by_base<STREAMS, T, D, true, R>(a, blocks, st);
        else quad_walk_by_base<STREAMS, T, D, false, R>(a, blocks, st);
    };
    auto by_dx = [&](auto rag) {
        if (dx) by_fold(rag, std::true_type{});
        else by_fold(rag, std::false_type{});
    };
    if (ragged) by_dx(std::integral_constant<bool, (T > 1)>{});
    else by_dx(std::false_type{});
}

}  // namespace

}  // namespace KAN_NS
