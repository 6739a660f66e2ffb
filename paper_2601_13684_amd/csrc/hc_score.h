// hc_score.h -- the candidates' scores and the histogram of them that the lists are taken from: what the monitor's passes
// (hc_monitor.hip) and the combine pass of a decode step (hc_attn.hip), which makes them on the way, have in common.
#pragma once
#include "hc_internal.h"

namespace {

constexpr int SCORE_BLK = 256;                                     // threads of a workgroup that scores
constexpr int SCORE_PER_THREAD = HC_SEL_CHUNK / SCORE_BLK;         // candidates of a chunk per thread

// Score of candidate j from the G scaled logits of its row (rep_logits is [ctx][G] per pivot).
template <int G>
__device__ __forceinline__ void load_row(const float* __restrict__ lrow, int j, float (&l)[G])
{
    if (G == 1) {
        l[0] = lrow[j];
    } else if (G == 2) {
        const float2 v = reinterpret_cast<const float2*>(lrow)[j];
        l[0] = v.x; l[1] = v.y;
    } else {
#pragma unroll
        for (int q = 0; q < G / 4; ++q) {
            const float4 v = reinterpret_cast<const float4*>(lrow)[(size_t)j * (G / 4) + q];
            l[4 * q] = v.x; l[4 * q + 1] = v.y; l[4 * q + 2] = v.z; l[4 * q + 3] = v.w;
        }
    }
}
template <int G>
__device__ __forceinline__ float score_of(const float* __restrict__ lrow, int j, const float (&lse)[G], int agg)
{
    float l[G];
    load_row<G>(lrow, j, l);
    return hc_group_score<G>(l, lse, agg);
}

// ---- the histogram of a candidate range ----
//
// 2048 digits, narrow ones for where a list usually ends, wide ones on either side.  Probabilities (HC_AGG_PROB): 64 to an octave
// over [2^-23, 2^-7), each 1.1 to 1.6 % of a score wide, 16 over [2^-79, 2^-23) and [2^-7, 2); the lowest takes everything below (negative
// scores and what is no number among them), the highest everything above.  The digit in which a list ends then holds a
// hundred or so of 32K candidates (of the key's first 11 bits, four to an octave, thousands), unless scores are that close to
// each other; where sharp attention makes scores small they are far apart.  Mean logits (HC_AGG_LOGIT): digits of 1/64 over
// [-12, 12), of 1/8 from -44 to 44.
template <int MID, int LOW, int SHIFT>
struct Digits {                                      // x: number of a narrow digit, 0 .. MID - 1 the narrow ones
    static __device__ __forceinline__ uint32_t of(int x)
    {
        const int y = min(max(x, x >> SHIFT), (x + ((1 << SHIFT) - 1) * MID) >> SHIFT);      // (below 0 and above MID the flatter line)
        return (uint32_t)min(max(y + LOW, 0), HC_RADIX_BINS - 1);
    }
    static __device__ __forceinline__ int first(int digit) { return digit < LOW ? (digit - LOW) << SHIFT : digit < LOW + MID ? digit - LOW : MID + ((digit - LOW - MID) << SHIFT); }
};
typedef Digits<1024, 896, 2> FineDigits;
typedef Digits<1536, 256, 3> LinearDigits;
constexpr int FINE_BASE = (0x80000000u >> 17) + (104 << 6);     // the key of 2^-23, without its last 17 bits
// FineDigits::of the score's key, in a third of the instructions: negative scores and what is no number end in the lowest digit, as 0
// does, and the piecewise line is the middle one of three.
__device__ __forceinline__ uint32_t fine_digit(float s)
{
    const int x = (int)(__float_as_uint(fmaxf(s, 0.f)) >> 17) + (0x4000 - FINE_BASE + 896), y = (x >> 2) + (896 - 896 / 4);
    return (uint32_t)min(max(min(max(x, y), y + (1024 - 1024 / 4)), 0), HC_RADIX_BINS - 1);
}
__device__ __forceinline__ uint32_t linear_digit(float s) { return LinearDigits::of((int)fminf(fmaxf(floorf(s * 64.f), -4096.f), 4096.f) + 768); }

enum { HIST_KEYS = 0, HIST_FINE = 1, HIST_LINEAR = 2 };
// The scores x[i] of candidates first + i SCORE_BLK + t (those before hi) to the histogram in LDS, and to memory unless they came from there.
template <int HIST>
__device__ __forceinline__ void count_scores(uint32_t* sh, float* __restrict__ srow, int first, int hi, const float (&x)[SCORE_PER_THREAD])
{
#pragma unroll
    for (int i = 0; i < SCORE_PER_THREAD; ++i) {
        const int j = first + i * SCORE_BLK + (int)threadIdx.x;
        if (j < hi) {
            if (srow) srow[j] = x[i];
            atomicAdd(&sh[HIST == HIST_LINEAR ? linear_digit(x[i]) : HIST == HIST_FINE ? fine_digit(x[i]) : hc_score_key(x[i]) >> 21], 1u);
        }
    }
}
__device__ __forceinline__ void flush_counts(uint32_t* __restrict__ hist, const uint32_t* sh)
{
    for (int i = threadIdx.x; i < HC_RADIX_BINS; i += SCORE_BLK)
        if (sh[i]) atomicAdd(&hist[i], sh[i]);
}

}   // namespace
