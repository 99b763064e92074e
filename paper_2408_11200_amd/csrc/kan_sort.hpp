// Stable LSD counting sort of one workgroup's keys in LDS, by a field of each key (the walk's row field).
//
// Bound by the chain of LDS round trips of a pass (one workgroup sorts one (chunk, input) list, and few fit a CU), so the
// digits are as wide as the counters leave room for: tables of up to 1024 rows (2048 for shorter lists) take one pass.
// A pass: every wave takes a contiguous share of the keys, 64 at a time; a key's rank among the wave's equal digits comes
// from ballots, one lane of each group of equal digits adds the group to the wave's counter, and rank and earlier count
// stay in registers; the counters are turned into first slots (prefix over digits, then over waves) by all threads; the
// keys are placed.  Nothing depends on timing.  Against 8-bit digits counted by one atomic a key and scanned by one wave:
// three layers of 360 rows, lists of 8192 (UKAN 128-256-256-1, B = 32768) 437 -> 288 us; 32 -> 32, G = 1024, B = 131072
// 76 -> 65; one-pass tables 57 -> 56 (64 -> 64, G = 10) and 88 -> 94 (512 -> 512, G = 20).  What is left is the records
// written, 44 bytes a pair.  Two waves share a 32-bit counter word (counts and slots fit 16 bits).
#pragma once
#include "kan_device.hpp"

namespace KAN_NS {

constexpr int kSortMaxBatches = 8;           // keys per wave / 64, at most

// digit width for a field: as few passes as digits of at most 10 (16 waves) or 11 bits allow, of equal width (the counters
// take LDS that a second workgroup on the CU could use: no wider than needed)
__host__ __device__ constexpr int sort_digit_bits(int NW, int field)
{
    const int most = NW >= 16 ? 10 : 11, n_pass = (field + most - 1) / most;
    return (field + n_pass - 1) / n_pass;
}
constexpr size_t sort_counter_bytes(int NW, int field) { return (size_t)(NW / 2) * 4 << sort_digit_bits(NW, field); }

// Place of a key with digit d among the keys its wave has counted so far, lanes before it included; counts the lanes' keys.
// mine: the wave's counter words, `half` the position of its 16 bits in them.  Lanes without a key take part with live ==
// false.  The last lane of a group of equal digits adds the group (LDS operations of one wave stay in order).
__device__ __forceinline__ unsigned count_digit(unsigned *mine, int half, unsigned d, int nbits, bool live, int lane)
{
    const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    unsigned long long same = __ballot(live);
    for (int bit = 0; bit < nbits; ++bit) {
        const bool set = ((d >> bit) & 1u) != 0u;
        const unsigned long long m = __ballot(set);
        same &= set ? m : ~m;
    }
    const unsigned off = ((mine[d] >> half) & 0xffffu) + (unsigned)__builtin_popcountll(same & below);
    if (live && (same >> lane) == 1ull) atomicAdd(&mine[d], (unsigned)__builtin_popcountll(same) << half);
    return off;
}

// Turns the counts of `bins` digits into first slots: digit by digit, within a digit wave by wave; PAD: every digit starts at
// a multiple of four.  Returns the slots in use.  Every thread calls this, between two barriers of its own.
template <int NW, bool PAD>
__device__ __forceinline__ unsigned slots_of_counts(unsigned *counters, int bins, unsigned *wave_total)
{
    constexpr int NT = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = bins > NT ? bins / NT : 1;
    const bool scans = tid * per < bins;
    unsigned sum = 0;
    if (scans)
        for (int d = tid * per; d < (tid + 1) * per; ++d) {
#pragma unroll
            for (int w = 0; w < NW / 2; ++w) {
                const unsigned v = counters[w * bins + d];
                sum += (v & 0xffffu) + (v >> 16);
            }
            if (PAD) sum = (sum + 3u) & ~3u;
        }
    unsigned inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
    }
    if (lane == 63) wave_total[wave] = inc;
    __syncthreads();
    unsigned at = inc - sum, total = 0;
    for (int w = 0; w < NW; ++w) {
        at += w < wave ? wave_total[w] : 0u;
        total += wave_total[w];
    }
    if (scans)
        for (int d = tid * per; d < (tid + 1) * per; ++d) {
#pragma unroll
            for (int w = 0; w < NW / 2; ++w) {
                const unsigned v = counters[w * bins + d];
                const unsigned a = at, b = at + (v & 0xffffu);
                at = b + (v >> 16);
                counters[w * bins + d] = a | (b << 16);
            }
            if (PAD) at = (at + 3u) & ~3u;
        }
    __syncthreads();
    return total;
}

// Sorts n keys (n / NW a multiple of 64, at most 512 a wave) by bits low .. low + field - 1; src and dst are n keys each
// and end up swapped so that src holds the result.  counters: sort_counter_bytes(NW, field) of LDS.
template <int NW>
__device__ __forceinline__ void lds_sort(unsigned *&src, unsigned *&dst, unsigned *counters, int n, int low, int field)
{
    constexpr int NT = 64 * NW;
    __shared__ unsigned wave_total[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bits = sort_digit_bits(NW, field), n_pass = (field + bits - 1) / bits, bins = 1 << bits;
    const int per_wave = n / NW, nb = per_wave / 64;
    const int half = (wave & 1) * 16;
    unsigned *mine = counters + (wave >> 1) * bins;
    for (int pass = 0; pass < n_pass; ++pass) {
        const int shift = low + bits * pass;
        const int nbits = field - bits * pass < bits ? field - bits * pass : bits;
        for (int e = tid; e < (NW / 2) * bins; e += NT) counters[e] = 0u;
        __syncthreads();
        unsigned key[kSortMaxBatches], off[kSortMaxBatches];
#pragma unroll
        for (int u = 0; u < kSortMaxBatches; ++u)
            if (u < nb) {
                key[u] = src[wave * per_wave + u * 64 + lane];
                const unsigned d = (key[u] >> shift) & (unsigned)(bins - 1);
                off[u] = count_digit(mine, half, d, nbits, true, lane);
            }
        __syncthreads();
        slots_of_counts<NW, false>(counters, bins, wave_total);
#pragma unroll
        for (int u = 0; u < kSortMaxBatches; ++u)
            if (u < nb) {
                const unsigned d = (key[u] >> shift) & (unsigned)(bins - 1);
                dst[((mine[d] >> half) & 0xffffu) + off[u]] = key[u];
            }
        __syncthreads();
        unsigned *t = src; src = dst; dst = t;
    }
}

}  // namespace KAN_NS
