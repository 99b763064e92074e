// Planning and helper kernels of the backward walk, and its form built on pair records.  Where a chunk has a few samples for
// every cell the walk goes over lists of padded cells instead (kan_quads_kernel.hpp); what follows here describes the records.
//
// Pair records are sorted by window row over a whole chunk of the batch: the parameter gradients of every layer shape they cover, and dL/dx with them where
// that is the faster way.
//
// With many coefficient rows per input (G + k in the hundreds, or a generated UKAN table) a tile of
// 64 samples touches each row at most a few times, so any scheme that keeps "all rows of an input"
// or "a block of rows" in registers spends its time on rows that receive nothing.  Here the samples
// of one chunk (S = 256 .. 8192 samples) are sorted by the first row of their window, per input.  A
// stream then walks a sorted list once: the window rows of consecutive records never move
// backwards, so K accumulators per output follow the window along the rows; a row is written out
// the moment the window has passed it and rows that no sample touched are written as zeros on the
// way (or jumped over).  Work per stream is (records) x (K + 1) multiply-adds plus one 16-byte
// store per row -- independent of the grid size (section "Algorithm": cost of the local form does
// not grow with G).
//
//   1. transpose_kernel      x[B][n_in] -> xT[n_in][B], so that one input's samples are contiguous
//   2. cell_sort_kernel      per (chunk, input): stable LSD radix sort of the S samples by window row
//                            in LDS, then one record per sample in sorted order (structure of
//                            arrays: window row | sample, base value, the K weights)
//   3. backward_walk_kernel  the walk; partial sums per chunk, reduced by dparam_reduce (fp64,
//                            fixed order), so results are bit-reproducible
// When a list is cut into several segments (one stream each), what a segment's window holds past its last own row goes to
// four carry rows, which the reduction over the chunks adds to the next segment's rows.
//
// Lanes <-> outputs.  A wave holds 64 / LPS streams of LPS lanes each (LPS = 16, 32 or 64), so that
// narrow layers still fill the wave.  Records are loaded 16 at a time, one per lane of each DPP row
// of 16 lanes, and broadcast inside the row with row_newbcast; there is no scalar state, hence
// streams in one wave may diverge freely.
//
// The accumulation itself, acc[row s][output j] += w_s * gy[j] for the K = 4 window rows, is a
// rank-1 update, and runs on the matrix cores as v_mfma_f32_4x4x1 (16 blocks of 4x4 outer
// products): a lane's B operand is gy of its output, the A operand of every block is the weight
// quadruple of the current record, which the instruction itself broadcasts from the four lanes that
// hold it (cbsz / abid), so the weights of 16 records are one coalesced 256-byte load and cost no
// VALU work.  None of the 256 multiply-adds of an instruction is padding.
#include "kan_device.hpp"
#include "kan_launch.hpp"
#include "kan_highk.hpp"
#include "kan_quads.hpp"
#include "kan_sort.hpp"

namespace kan {

namespace {

// ---- 1. transpose --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void transpose_kernel(const float *__restrict__ x, float *__restrict__ xT,
                                                        int64_t B, int n_in)
{
    __shared__ float tile[64][65];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * 64;
    const int i0 = blockIdx.y * 64;
    for (int r = ty; r < 64; r += 4)
        tile[r][tx] = (b0 + r < B && i0 + tx < n_in) ? x[(b0 + r) * n_in + i0 + tx] : 0.0f;
    __syncthreads();
    for (int r = ty; r < 64; r += 4)
        if (i0 + r < n_in && b0 + tx < B) xT[(int64_t)(i0 + r) * B + b0 + tx] = tile[tx][r];
}

// ---- 2. sort + records ---------------------------------------------------------------------
// grid (n_chunks, n_in), NW waves.  key = window row << sbits | sample index in the chunk
// (sbits = log2 S): keys are distinct, and sorting them by the row digits with a stable counting
// sort keeps samples of equal row in batch order, which fixes the summation order downstream (kan_sort.hpp).
// Entries past the end of the batch get the largest row and end up behind every real record.
template <int NW>
__global__ __launch_bounds__(64 * NW) void cell_sort_kernel(SplineGeom g, const float *__restrict__ xT, int64_t B,
                                                            int S, int sbits, int row_bits, WalkRecords rec)
{
    constexpr int kSortThreads = 64 * NW;
    extern __shared__ unsigned lds_u[];
    unsigned *src = lds_u, *dst = lds_u + S;
    float *xs = reinterpret_cast<float *>(lds_u + 2 * S);
    unsigned *counters = lds_u + 2 * S + S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = blockIdx.x, i = blockIdx.y;
    const int64_t b0 = (int64_t)c * S;
    const int n_c = (int)((B - b0) < S ? (B - b0) : S);

    for (int e = tid; e < S; e += kSortThreads) {
        const bool live = e < n_c;
        const float xv = live ? xT[(int64_t)i * B + b0 + e] : 0.0f;
        xs[e] = xv;
        int row0 = g.rows - kMaxK;
        if (live) row0 = window_row(xv, g, i);
        src[e] = ((unsigned)row0 << sbits) | (unsigned)e;
    }
    __syncthreads();

    lds_sort<NW>(src, dst, counters, S, sbits, row_bits);

    const int64_t list = ((int64_t)c * g.n_in + i) * S;
    for (int p = tid; p < S; p += kSortThreads) {
        const int e = (int)(src[p] & (unsigned)(S - 1));
        const bool live = e < n_c;
        const Pair pr = rec.dw4 ? pair_eval<true>(xs[e], g, i) : pair_eval<false>(xs[e], g, i);
        float w[kMaxK], dw[kMaxK], base, dbase;
        int row0;
        window_of<false>(pr, g.rows, row0, w, base);
        window_of<true>(pr, g.rows, row0, dw, dbase);
        if (!live) {
            row0 = g.rows - kMaxK;
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) { w[s] = 0.0f; dw[s] = 0.0f; }
            base = 0.0f; dbase = 0.0f;
        }
        // The consumer keeps its K window rows in a ring indexed by (row mod K): store the weight of
        // window row row0 + s in position (row0 + s) mod K, so that it needs no shifting there.
        float wr[kMaxK], dwr[kMaxK];
#pragma unroll
        for (int q = 0; q < kMaxK; ++q) {
            float v = 0.0f, dv = 0.0f;
#pragma unroll
            for (int s = 0; s < kMaxK; ++s) {
                const bool hit = ((row0 + s) & (kMaxK - 1)) == q;
                v = hit ? w[s] : v;
                dv = hit ? dw[s] : dv;
            }
            wr[q] = v; dwr[q] = dv;
        }
        rec.rt[list + p] = row0 | ((live ? e : 0) << kRtRowBits);
        rec.base[list + p] = base;
        *reinterpret_cast<float4 *>(rec.w4 + (list + p) * 4) = make_float4(wr[0], wr[1], wr[2], wr[3]);
        if (rec.dw4) {
            rec.dbase[list + p] = dbase;
            *reinterpret_cast<float4 *>(rec.dw4 + (list + p) * 4) = make_float4(dwr[0], dwr[1], dwr[2], dwr[3]);
        }
    }
}

// Shared slabs: adds the carry rows of segments 1 .. n_seg-1 to the slabs, in segment order, after each round of chunks.
// One thread per (chunk, input, output).  (Slabs of their own: the reduction over the chunks adds the carry rows.)
__global__ __launch_bounds__(256) void walk_carry_kernel(SplineGeom g, const int *__restrict__ seg_row,
                                                         const float *__restrict__ carry, float *__restrict__ part_c,
                                                         int n_chunks, int n_seg, int chunk0, int window)
{
    // n_chunks chunks starting at chunk0 of the batch; the launch's chunk number l adds to slab l
    const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (at >= (int64_t)n_chunks * g.n_in * g.n_out) return;
    const int j = (int)(at % g.n_out);
    const int64_t ci = (int64_t)chunk0 * g.n_in + at / g.n_out;               // chunk * n_in + input
    float *slab = part_c + at / g.n_out * g.rows * g.n_out + j;
    for (int k = 1; k < n_seg; ++k) {
        const int rf = seg_row[ci * n_seg + k];
        const float *cr = carry + ((ci * n_seg + k) * window) * g.n_out + j;
        for (int s = 0; s < window; ++s)
            if (rf + s < g.rows) slab[(int64_t)(rf + s) * g.n_out] += cr[(int64_t)s * g.n_out];
    }
}

// plain zero fill (a kernel rather than a memset so that the call sequence can be captured in a graph)
__global__ __launch_bounds__(256) void fill_zero_kernel(float *__restrict__ p, int64_t n)
{
    const int64_t at = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (at + 3 < n) {
        *reinterpret_cast<float4 *>(p + at) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        for (int64_t e = at; e < n; ++e) p[e] = 0.0f;
    }
}

// gx = sum over the output tiles' partial gx
__global__ __launch_bounds__(256) void gx_sum_kernel(const float *__restrict__ part, float *__restrict__ gx, int64_t n,
                                                     int n_jt)
{
    const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (at >= n) return;
    float v = part[at];
    for (int t = 1; t < n_jt; ++t) v += part[(int64_t)t * n + at];
    gx[at] = v;
}

int log2_exact(int v) { int b = 0; while ((1 << b) < v) ++b; return b; }

}  // namespace

// ---- planning and launch ---------------------------------------------------------------------

namespace {

// quads: lists of padded cells where the shape allows (p.quads says), else one record a pair
WalkPlan plan_lists(const SplineGeom &g, int64_t B, bool allow_shared, bool high_degree, bool quads)
{
    WalkPlan p = {};
    if (g.rows < kMaxK || g.rows > kRtRowMask || B < 1) return p;
    if (high_degree && g.rows < 6) return p;          // a six-row window must fit the table
    const int64_t slab = (int64_t)g.n_in * g.rows * g.n_out * (int64_t)sizeof(float);
    const int s_max = high_degree && !quads ? 4096 : 8192;       // two records per pair: 2 S keys to sort, 12 bits for the sample
    auto pow2_floor = [s_max](int64_t v) { int64_t q = 256; while (q * 2 <= v && q < s_max) q *= 2; return (int)q; };
    // chunk length: a power of two between 256 and 8192 samples.  Every chunk writes a partial table that the reduction
    // reads back, so few long chunks are better, as long as
    //   - the gy rows of a chunk stay in cache (at most 8 MiB: twice an XCD's L2, the rest served by the memory-side
    //     cache.  128 -> 256 -> 256 -> 1 with tables of 360 rows, B = 32768, walk + sort + reduction: 4 MiB 2.73 ms, 8 MiB
    //     2.64 ms),
    //   - there is an eighth of the batch in a chunk at most (one chunk per XCD) or two workgroups per CU left to sort
    //     (256 -> 256, G = 200, B = 8192: eight chunks 538 us, four 422 us, two 368 us).
    // Raised further until the partial sums fit 2 GiB.  The parallelism of the walk comes from cutting each sorted list
    // into segments (below).
    int S = pow2_floor((8ll << 20) / ((int64_t)g.n_out * 4));
    int64_t share = B * g.n_in / 512 < B ? B * g.n_in / 512 : B;
    if (share < B / 8) share = B / 8;
    const int s_par = pow2_floor(share);
    S = S < s_par ? S : s_par;
    auto fit_sums = [&](int q) { while (q < s_max && ((B + q - 1) / q) * slab > (2ll << 30)) q *= 2; return q; };
    // Eight outputs per lane (one tile covers 512 outputs: the per-record work is shared by twice as many).  The quads take
    // them with chunks of 2048 samples (512 -> 512, G = 20, B = 16384, walk + reduction: 1024 samples 1181 + 99 us, 2048 1149 +
    // 52, 4096 1175 + 36 with gy past L2).  Records have registers
    // for single-level sums only, so chunks of at most 1024 samples: not where the partial sums ask for longer ones (two
    // levels spill: 256 -> 300, G = 1000, B = 8192 walk 15.4 ms against 1.2 with four).  Widths that are no multiple of
    // eight take it where it pays: many pairs of a short table, and a last tile more than half full (backward pass, four
    // outputs / eight: 16 -> 300, G = 20, B = 16384 107 / 97 us, 64 -> 300, G = 5, B = 16384 282 / 236; but 2 -> 300, G = 20,
    // B = 65536 101 / 137, 16 -> 300, G = 1000, B = 16384 214 / 317, 64 -> 515, G = 20, B = 4096 126 / 147).
    const int most8 = quads ? 2048 : 1024;
    const int s8 = fit_sums(S < most8 ? S : most8);
    const bool pays8 = g.n_out % 8 == 0 || (g.n_in >= 16 && B * g.n_in >= 1 << 17 && g.rows <= (B <= 16384 ? 320 : 128) &&
                                            (g.n_out - 1) % 512 >= 256);
    // Chunk c is walked by XCD c mod 8, and eight outputs a lane leave a SIMD two waves: chunks of 2048 samples may leave most of the
    // chip without work in the last round of waves, or of chunks.  The time of a pass with either length, us: a SIMD's waves two at
    // a time (a single one takes 0.65 of two), 0.2 an entry, and the partial tables written and read.  Full pass / parameter
    // gradients only, 1024 : 2048: 203 -> 260, G = 15, k = 1, B = 22307 0.68 / 0.65 (11 chunks, two for three XCDs), 58 -> 384, G = 21, B = 88501
    // 0.79 / 0.77; 512 -> 512, G = 20, B = 16384 1.03 / 1.05; 13 -> 512, G = 100, B = 63709 1.22 / 1.39.
    auto pass_us = [&](int q) {
        const int64_t chunks = (B + q - 1) / q, work = (int64_t)g.n_in * ((g.n_out + 511) / 512);
        int64_t groups = 1, segs = 1;
        while (groups * 2 <= 8 && groups * 2 <= chunks) groups *= 2;
        while (q / (segs * 2) >= 64 && chunks * segs * work < 2048) segs *= 2;
        const int64_t simds = 1024 / groups, deep = ((chunks + groups - 1) / groups * work * segs + simds - 1) / simds;
        return (deep / 2 + deep % 2 * 0.65) * (q / segs) * 0.2 + chunks * slab * 2 / 5e6;
    };
    // every width has a variant (widths that are no multiple of T run its ragged build)
    if (g.n_out > 256 && pays8 && s8 <= most8 && !(quads && high_degree)) {
        p.T = 8;
        p.streams = 1;
        // (of tables that leave the lists dense enough for quads, below)
        S = s8 == 2048 && g.rows - kMaxK + 1 <= 256 && fit_sums(1024) == 1024 && pass_us(1024) < pass_us(2048) ? 1024 : s8;
    } else {
        S = fit_sums(S);
        if (g.n_out > 32) {
            p.T = 4;
            p.streams = g.n_out > 128 ? 1 : (g.n_out > 64 ? 2 : 4);
        } else if (g.n_out > 16) {
            p.T = 2;        // 16 lanes x 2 outputs cover the layer: no idle lanes in a stream
            p.streams = 4;
        } else {
            p.T = g.n_out % 4 == 0 ? 4 : 1;
            p.streams = 4;
        }
    }
    const int tile = (64 / p.streams) * p.T;
    p.n_jt = (g.n_out + tile - 1) / tile;
    p.S = S;
    p.window = high_degree && quads ? 6 : kMaxK;
    p.hk = high_degree && !quads ? 1 : 0;
    p.L = p.hk ? 2 * S : S;
    p.sbits = log2_exact(S);
    p.n_chunks = (int)((B + S - 1) / S);
    // segments per list: enough for about 2048 waves, at least 64 records each
    int bits = 0;
    while ((1 << bits) < g.rows - p.window + 1) ++bits;
    p.row_bits = bits < 1 ? 1 : bits;
    p.ok = (int64_t)p.n_chunks * slab <= (4ll << 30) ? 1 : 0;
    p.shared = 0;
    p.n_slabs = p.n_chunks;
    auto plan_segments = [&](int chunks_per_launch) {
        p.n_seg = 1;
        while (p.L / (p.n_seg * 2) >= 64 &&
               (int64_t)chunks_per_launch * p.n_seg * p.n_jt * g.n_in < (int64_t)2048 * p.streams)
            p.n_seg *= 2;
    };
    plan_segments(p.n_chunks);
    // Tables too large for one partial slab per chunk: as many slabs as fit the budget (at least one),
    // the chunks walked in rounds of that many, one launch per round, chunk number l of a round adding its
    // sums to the rows it touches in slab l (the launches are ordered by the stream and every row of a slab
    // has one writer per launch, so the summation order is still fixed).
    if (!p.ok && allow_shared && slab <= (8ll << 30)) {
        p.ok = 1;
        p.shared = 1;
        const int64_t fit = (4ll << 30) / slab;
        p.n_slabs = (int)(fit < 1 ? 1 : (fit > p.n_chunks ? p.n_chunks : fit));
        plan_segments(p.n_slabs);
    }
    if (quads) {
        // One counting pass sorts a list; offsets of 30 bits into a chunk's gy and the table (with one stream a wave: an
        // input's); and samples a cell enough that the padding does not eat the gain.  Backward pass, records / quads, us, by
        // samples a cell:
        //   four outputs a lane, one stream   2: 64 -> 256, G = 1000, B = 8192 336 / 368 with 1, 247 / 210 with 20 (256 -> 256)
        //   eight outputs a lane              2: 256 -> 512, G = 1000, B = 8192 1428 / 1833; 47: 512 -> 512 1452 / 1148
        //   narrower                          1: 16 -> 32, G = 1000, 0.80 of the time, 8: 32 -> 32, G = 1024 274 / 169
        //   windows of six rows, one stream   2.6: 2 -> 130, G = 100, B = 1024 45 / 52; two streams 2.6: 51 / 54; 64: 0.6
        const int64_t most = 1ll << 28, slab_floats = (int64_t)g.slab_rows * g.n_out;
        const int per_cell = high_degree ? (p.streams == 1 ? 4 : p.streams == 2 ? 3 : 2)
                                         : (p.T == 8 ? 4 : p.streams == 1 ? 2 : 1);
        p.quads = p.row_bits <= 10 && S >= per_cell * (g.rows - p.window + 1) && (int64_t)S * g.n_out <= most &&
                  (p.streams == 1 ? 1 : g.n_in) * slab_floats <= most && (int64_t)g.n_in * g.n_out <= most ? 1 : 0;
        p.L = quad_list_entries(S, g.rows, p.window);
        // one output: a workgroup a list (kan_walk_one.hip), where there is one a CU (256 -> 1, B = 32768: 204 us / 74); fewer leave
        // CUs idle that segments of a list would fill.  Its sums and the chunk's gy have to fit LDS (and past 144 KB
        // it does not pay: 500 -> 1, G = 1000, B = 32768 672 / 698), its launch 2^32 threads.
        p.one = p.quads && g.n_out == 1 && !high_degree && !p.shared && (int64_t)p.n_chunks * g.n_in >= 256 &&
                (int64_t)p.n_chunks * g.n_in <= 1 << 22 && walk_one_lds_bytes(g.rows, S) <= 144 * 1024 ? 1 : 0;
        if (p.one) p.n_seg = 1;
    }
    return p;
}

}  // namespace

WalkPlan plan_walk(const SplineGeom &g, int64_t B, bool allow_shared, bool high_degree)
{
    const WalkPlan p = plan_lists(g, B, allow_shared, high_degree, true);
    return p.quads ? p : plan_lists(g, B, allow_shared, high_degree, false);
}

// one translation unit per kernel variant (kan_walk_s*t*.hip)
#define KAN_WALK_VARIANT(name)                                                                                      \
    void name(bool dx, unsigned blocks, hipStream_t st, const SplineGeom &g, const WalkRecords &rec, const float *gy, \
              const float *cf, const float *w_b, float *part_c, float *part_b, float *gx, int64_t B,              \
              const WalkPlan &p, int bpc, int m, int prezeroed, float *carry, int *seg_row, int chunk0, int n_chunks)
KAN_WALK_VARIANT(walk_launch_s1t8);
KAN_WALK_VARIANT(walk_launch_s1t4);
KAN_WALK_VARIANT(walk_launch_s2t4);
KAN_WALK_VARIANT(walk_launch_s4t4);
KAN_WALK_VARIANT(walk_launch_s4t2);
KAN_WALK_VARIANT(walk_launch_s4t1);
// n_out not a multiple of the outputs per lane
KAN_WALK_VARIANT(walk_launch_s1t8_ragged);
KAN_WALK_VARIANT(walk_launch_s1t4_ragged);
KAN_WALK_VARIANT(walk_launch_s2t4_ragged);
KAN_WALK_VARIANT(walk_launch_s4t4_ragged);
KAN_WALK_VARIANT(walk_launch_s4t2_ragged);
#undef KAN_WALK_VARIANT

namespace {
size_t up256(size_t v) { return (v + 255) / 256 * 256; }
}

// transposed x | records (row|sample, base, weights, derivative base, derivative weights) or cell lists |
// per-tile partial gx (layers wider than one tile) | carry rows of the list segments | first row of every segment
static size_t walk_carry_bytes(const WalkPlan &p, int n_in, int n_out)
{
    return up256((size_t)p.n_chunks * n_in * (p.n_seg + 1) * p.window * n_out * sizeof(float));
}
static size_t walk_seg_row_bytes(const WalkPlan &p, int n_in) { return up256((size_t)p.n_chunks * n_in * p.n_seg * sizeof(int)); }

size_t walk_scratch_bytes(const WalkPlan &p, int64_t B, int n_in, int n_out)
{
    const size_t n = (size_t)p.n_chunks * n_in * (p.window > kMaxK ? 2 * (size_t)p.S : p.quads ? (size_t)p.S : (size_t)p.L);
    const int n_part = p.n_jt * (p.hk ? 2 : 1);       // partial dL/dx results per (sample, input)
    const size_t gxp = n_part > 1 ? up256((size_t)n_part * B * n_in * sizeof(float)) : 0;
    // The records' size in either case (44 bytes a pair, 88 of degrees 4 and 5; lists of padded cells use 24 at most), so that this,
    // the largest part, does not jump where a batch or a table passes from one to the other.  What stands beside it follows the
    // plan: partial dL/dx, carry rows of four or six, chunks.
    const size_t lists = 3 * up256(n * 4) + 2 * up256(n * 16);
    return up256((size_t)B * n_in * sizeof(float)) + lists + gxp +
           walk_carry_bytes(p, n_in, n_out) + walk_seg_row_bytes(p, n_in);
}

// Per (chunk of S samples, input) the records in sorted order.  S: a power of two >= 256.
hipError_t launch_sorted_records(const SplineGeom &g, const float *xT, int64_t B, int S, int row_bits, const WalkRecords &rec,
                                 hipStream_t st)
{
    // waves per sort, measured: 16 for chunks of 8192 samples, 8 for 4096, 4 below
    const size_t lds = (size_t)S * 12 + sort_counter_bytes(S >= 8192 ? 16 : (S >= 4096 ? 8 : 4), row_bits);
    dim3 grid((unsigned)((B + S - 1) / S), (unsigned)g.n_in);
    prof::Timed tm("walk_sort", st);
    struct W16; struct W8; struct W4;
    hipError_t e;
    if (S >= 8192) {
        auto kern = cell_sort_kernel<16>;
        if ((e = ensure_dynamic_lds<W16>(reinterpret_cast<const void *>(kern), (int)lds)) != hipSuccess) return e;
        kern<<<grid, 1024, lds, st>>>(g, xT, B, S, log2_exact(S), row_bits, rec);
    } else if (S >= 4096) {
        auto kern = cell_sort_kernel<8>;
        if ((e = ensure_dynamic_lds<W8>(reinterpret_cast<const void *>(kern), (int)lds)) != hipSuccess) return e;
        kern<<<grid, 512, lds, st>>>(g, xT, B, S, log2_exact(S), row_bits, rec);
    } else {
        auto kern = cell_sort_kernel<4>;
        if ((e = ensure_dynamic_lds<W4>(reinterpret_cast<const void *>(kern), (int)lds)) != hipSuccess) return e;
        kern<<<grid, 256, lds, st>>>(g, xT, B, S, log2_exact(S), row_bits, rec);
    }
    return hipGetLastError();
}

// gx == nullptr: parameter gradients only.  part_c == nullptr: dL/dx only.  cf is the scale-folded
// table ([n_in][slab_rows][n_out]); w_b may be null when the layer has no base term.
hipError_t launch_backward_walk(const SplineGeom &g, const WalkPlan &p, const float *x, const float *gy,
                                const float *cf, const float *w_b, void *scratch, float *gx, float *part_c,
                                float *part_b, int64_t B, CarryRows *carry_rows, hipStream_t st)
{
    const size_t n = (size_t)p.n_chunks * g.n_in * p.L;
    const int n_part = p.n_jt * (p.hk ? 2 : 1);
    const bool dx = gx != nullptr;
    char *at = (char *)scratch;
    float *xT = (float *)at;            at += up256((size_t)B * g.n_in * sizeof(float));
    WalkRecords rec = {};
    QuadWalkArgs qa = {};
    if (p.quads) {
        qa.lists.x = (float *)at;           at += up256(n * 4);
        qa.lists.sample = (uint16_t *)at;   at += up256(n * 2);
        qa.lists.n_quads = (int *)at;       at += up256((size_t)p.n_chunks * g.n_in * 4);
        qa.lists.L = p.L;
    } else {
        rec.rt = (int *)at;                 at += up256(n * 4);
        rec.base = (float *)at;             at += up256(n * 4);
        rec.w4 = (float *)at;               at += up256(n * 16);
        rec.dbase = dx ? (float *)at : nullptr; at += up256(n * 4);
        rec.dw4 = dx ? (float *)at : nullptr;   at += up256(n * 16);
    }
    float *gx_part = (float *)at;       at += n_part > 1 ? up256((size_t)n_part * B * g.n_in * sizeof(float)) : 0;
    float *carry = (float *)at;         at += walk_carry_bytes(p, g.n_in, g.n_out);
    int *seg_row = (int *)at;
    // the chunks' carry rows are added by the reduction over the chunks; shared slabs take theirs below
    *carry_rows = CarryRows{seg_row, carry, p.shared ? 1 : p.n_seg, p.window};
    {
        dim3 grid((unsigned)((B + 63) / 64), (unsigned)((g.n_in + 63) / 64));
        prof::Timed tm("walk_transpose", st);
        transpose_kernel<<<grid, 256, 0, st>>>(x, xT, B, g.n_in);
    }
    if (p.quads) {
        qa.n_in = g.n_in; qa.n_out = g.n_out; qa.rows = g.rows; qa.slab_rows = g.slab_rows; qa.k = g.k; qa.lo = g.lo;
        qa.inv_h = g.inv_h; qa.cell_base = g.cell_base;
        qa.base_act = w_b != nullptr ? g.base_act : 0;
        qa.gy = gy; qa.cf = cf; qa.w_b = w_b; qa.part_c = part_c; qa.part_b = part_b;
        qa.carry = carry; qa.seg_row = seg_row; qa.B = B; qa.S = p.S; qa.n_seg = p.n_seg; qa.n_jt = p.n_jt;
        if (hipError_t e = p.window == 6 ? launch_cell_lists6(qa, xT, p.row_bits, st) : launch_cell_lists(qa, xT, p.row_bits, st);
            e != hipSuccess)
            return e;
    } else if (p.hk) {
        // degrees 4 and 5: the records come from the kernel built for a window of six rows
        HighKLayer l = {};
        l.n_in = g.n_in; l.n_out = g.n_out; l.rows = g.rows; l.k = g.k; l.lo = g.lo; l.inv_h = g.inv_h; l.base_act = g.base_act;
        l.slab_rows = g.slab_rows; l.cell_base = g.cell_base;
        if (hipError_t e = highk_sorted_records(l, xT, B, p.S, p.row_bits, rec.rt, rec.base, rec.w4, rec.dbase, rec.dw4, st);
            e != hipSuccess)
            return e;
    } else if (hipError_t e = launch_sorted_records(g, xT, B, p.S, p.row_bits, rec, st); e != hipSuccess) {
        return e;
    }
    const int bpc = (p.n_seg * p.n_jt * g.n_in + 4 * p.streams - 1) / (4 * p.streams);
    float *gx_out = dx ? (n_part > 1 ? gx_part : gx) : nullptr;
    // Sparse regime (far more rows than a chunk has samples): most rows of a chunk's partial slab
    // receive nothing.  The slab is zeroed with a streaming fill and the walk skips the gaps instead of
    // stepping through them row by row.  A shared slab is always used this way.
    const int prezeroed = (part_c != nullptr && (g.rows > 2 * p.S || p.shared)) ? 1 : 0;
    if (prezeroed) {
        const int64_t n4 = (int64_t)p.n_slabs * g.n_in * g.rows * g.n_out;
        prof::Timed tm("walk_zero_fill", st);
        fill_zero_kernel<<<(unsigned)((n4 + 1023) / 1024), 256, 0, st>>>(part_c, n4);
    }
    // one launch for all chunks, or (shared slabs) one launch per round of n_slabs chunks, each followed by
    // its carry rows
    const int per_launch = p.shared ? p.n_slabs : p.n_chunks;
    const int launches = (p.n_chunks + per_launch - 1) / per_launch;
    int m = 1;
    while (m * 2 <= 8 && m * 2 <= per_launch) m *= 2;
    const int bpc_sub = (bpc + 8 / m - 1) / (8 / m);
    const unsigned blocks = (unsigned)(8 * bpc_sub * ((per_launch + m - 1) / m));
    for (int l = 0; l < launches; ++l) {
        const int chunk0 = l * per_launch;
        const int here = p.n_chunks - chunk0 < per_launch ? p.n_chunks - chunk0 : per_launch;
        {
            prof::Timed tm(dx ? "backward_walk" : "dparam_walk", st);
            if (p.quads) {
                qa.gx = gx_out; qa.chunk0 = chunk0; qa.n_chunks = here; qa.blocks_per_chunk = bpc; qa.xcd_groups = m;
                qa.prezeroed = prezeroed;
                qa.shared = p.shared && chunk0 > 0 ? 1 : 0;       // the first round finds its slabs zero and stores
                if (p.one) {
                    if (hipError_t e = walk_one(qa, st); e != hipSuccess) return e;
                    continue;
                }
                auto walk = p.window == 6 ? (p.T == 2 ? quad_walk6_s4t2
                                             : p.T == 1 ? quad_walk6_s4t1
                                             : p.streams == 1 ? quad_walk6_s1t4
                                             : p.streams == 2 ? quad_walk6_s2t4 : quad_walk6_s4t4)
                            : p.T == 8 ? quad_walk_s1t8
                            : p.T == 2 ? quad_walk_s4t2
                            : p.T == 1 ? quad_walk_s4t1
                            : p.streams == 1 ? quad_walk_s1t4
                            : p.streams == 2 ? quad_walk_s2t4 : quad_walk_s4t4;
                walk(qa, blocks, st);
            } else {
                const bool ragged = g.n_out % p.T != 0;
                auto launch = p.T == 8 ? (ragged ? walk_launch_s1t8_ragged : walk_launch_s1t8)
                              : p.T == 2 ? (ragged ? walk_launch_s4t2_ragged : walk_launch_s4t2)
                              : p.T == 1 ? walk_launch_s4t1
                              : p.streams == 1 ? (ragged ? walk_launch_s1t4_ragged : walk_launch_s1t4)
                              : p.streams == 2 ? (ragged ? walk_launch_s2t4_ragged : walk_launch_s2t4)
                                               : (ragged ? walk_launch_s4t4_ragged : walk_launch_s4t4);
                launch(dx, blocks, st, g, rec, gy, cf, w_b, part_c, part_b, gx_out, B, p, bpc, m, prezeroed, carry, seg_row, chunk0, here);
            }
        }
        if (part_c != nullptr && p.n_seg > 1 && p.shared) {
            const int64_t nn = (int64_t)here * g.n_in * g.n_out;
            prof::Timed tm("walk_carry", st);
            walk_carry_kernel<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(g, seg_row, carry, part_c, here, p.n_seg, chunk0, p.window);
        }
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    if (dx && n_part > 1) {
        const int64_t nn = B * g.n_in;
        prof::Timed tm("walk_gx_sum", st);
        gx_sum_kernel<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(gx_part, gx, nn, n_part);
    }
    return hipGetLastError();
}

}  // namespace kan
