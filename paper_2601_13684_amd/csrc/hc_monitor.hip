// hc_monitor.hip -- the pivot heads' drift monitor (Sec. 4.3, Eq. 9-10; Algorithm 1 stage 3):
// GQA-aggregated score (App. C.1), TopIndices_k for every needed set size, overlap with the
// baseline set, windowed-median retrieval signal, baseline update.
//
// Selection is exact: the k-th largest order-preserving 32-bit key of the fp32 scores is found, and ties at that
// threshold key are resolved by position (the equal-keyed candidates with the lowest indices are taken), which
// makes the result the unique first-k set under (score descending, index ascending).  Lists are emitted in
// ascending index order.
//
// The work is a few MB at most and bound by latency: what costs is the number of dependent launches (5-8 us each
// for one layer, several times that beside the attention pass) and of dependent memory round trips inside one.  So
// everything after the scores is ONE kernel, mon_select, with one workgroup per pivot and set size that keeps the keys
// of its items in LDS: threshold, ordered lists, |T ∩ baseline| through a bitmap in LDS, window, decision and
// baseline update.  What reaches it:
//   short candidate ranges   mon_direct scores the candidates itself: one launch
//   up to 64K candidates (beside the attention pass 32K, and for few lists 64K)
//                            mon_score_hist (scores and their histogram; many workgroups per pivot), mon_direct (the lists straight
//                            from the scores, no keys in LDS): two launches
//   longer ranges            mon_score_hist (scores, first-digit histogram; many workgroups per pivot), mon_compact (the
//                            candidates that can be in the longest list, and few more), mon_select over those (a few
//                            thousand): three launches
//   long lists               mon_score_hist, mon_hist twice, mon_count, mon_write, mon_decide: six launches of many workgroups
//   rows a filtering split pass kept
//                            mon_sparse_score (their scores, one dense run), mon_direct (mon_select beside the attention pass for
//                            lists of up to 4,096, and where mon_direct's LDS does not suffice, with the long ranges' first
//                            two in front of it where more rows are kept than it has room for): two launches, and behind them
//                            two that normally find nothing to do, for a pivot whose check failed: rep_logits_kernel
//                            (hc_attn.hip; all logits again, with their scores) and mon_select, which cuts the whole range
//                            down by itself (a launch more for that would cost every step 3 us), or the six of long lists
// (mon_prep clears the histograms and bitmaps, only after a call that failed midway; normally mon_select leaves
// them clear.)
//
// Measured on MI355X against a radix select in six launches over all candidates (score and histogram, two more
// histograms, counts, ordered write, decision): one 32K layer 19.8 instead of 51.5 us per call, eight sequences of 9K to
// 131K 33-36 instead of 81 us, the decode step of one 4K layer 23.3 instead of 49 us.
//
// Beside the attention pass (hc_decode_step's side stream) a workgroup has to find room on a compute unit that holds
// two attention workgroups, whose registers (at most 216 a lane) leave 80 per lane of a SIMD: 256 threads of at most 80
// registers, or 512 threads of at most 40 (the small forms of mon_select and mon_direct; no bound on waves per SIMD asks for so few, a
// test of the built kernels holds them to it).  In groups of eight heads the attention workgroups leave too little LDS for
// mon_select's keys: its large form runs there, on a compute unit of its own (measured with four layers of 229,376 and lists
// of 3,840: 266 us a step, 282 with the small form for as many as fit).  No local arrays (a kernel that needs scratch memory
// costs tens of us to launch), no device-wide fences.
#include <algorithm>
#include <cmath>

#include "hc_internal.h"
#include "hc_score.h"

namespace {

constexpr int BLK = SCORE_BLK;
constexpr int NWAVE = BLK / 64;

__device__ __forceinline__ float key_score(uint32_t key)      // inverse of hc_score_key
{
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// Workspace of one layer of a batch (rep: pivot).
struct Ws {
    uint32_t* hist;      // [HC_RADIX_BINS]: first-digit histogram of a long range, and behind it how many of mon_direct's
                         // workgroups are through with it (HC_HIST_WORDS in all)
    uint32_t* bitmap;    // [max_ctx / 32]: baseline set, where it does not fit in LDS
    // one piece of memory, `area` words per pivot, that a call uses either for survivors ...
    uint64_t* mask;      // [max_chunks][HC_SEL_CHUNK / 64]: which candidates survive
    int32_t* sv_pos;     // [sv_cap]: the survivors' positions
    // ... or for long lists
    uint32_t* h2;        // [HC_MAX_K_PER_REP][HC_RADIX_BINS]: second digits
    uint32_t* h3;        // [HC_MAX_K_PER_REP][HC_RADIX_BINS]: third digits
    uint32_t* sel;       // [HC_MAX_K_PER_REP][4]: first digits found / still needed, then two digits found / still needed
    uint32_t* cnt;       // [HC_MAX_K_PER_REP][max_chunks][2]: greater, equal
    uint32_t* hits;      // [max_chunks]: |T ∩ baseline| of every chunk
    int max_chunks, max_ctx, sv_cap;
    size_t area;
    __device__ Ws rep(int r) const
    {
        Ws w = *this;
        w.hist += (size_t)r * HC_HIST_WORDS;
        w.bitmap += (size_t)r * (max_ctx / 32);
        w.h2 += (size_t)r * area;
        w.h3 = w.h2 + HC_MAX_K_PER_REP * HC_RADIX_BINS;
        w.sel = w.h3 + HC_MAX_K_PER_REP * HC_RADIX_BINS;
        w.cnt = w.sel + HC_MAX_K_PER_REP * 4;
        w.hits = w.cnt + (size_t)HC_MAX_K_PER_REP * max_chunks * 2;
        w.mask = reinterpret_cast<uint64_t*>(w.h2);
        w.sv_pos = reinterpret_cast<int32_t*>(w.mask + (size_t)max_chunks * (HC_SEL_CHUNK / 64));
        return w;
    }
};

// One layer of a batched call: its workspace copy, its plan and the caller's buffers.  A launch handles
// up to HC_MAX_GROUP layers (blockIdx.z picks the layer), so that a group of layers costs the launches
// and the launch latencies of one.
struct MonItem {
    Ws ws;
    const RepDev* reps;
    const OutDev* outs;
    union {
        const float* rep_logits;
        float* copy_to;           // scores that the combine pass made: where the selection copies them (nullptr: they are the caller's already)
    };
    const float* lse;
    float* scores;
    int32_t* topk_idx;
    int32_t* base_idx;
    int32_t* ring;
    int32_t* inter;
    int32_t* flag;
    int n_reps;
    int store_slot;
    // A layer whose split pass filters the pivot logits: the selection runs over the kept rows only (reps = the
    // pivots as seen over those rows, pos_map = their positions), and a second, dense chain stands by for the
    // pivots whose check failed (need[rep] != 0).
    int need_sense;               // -1: unconditional; 0: run where need[rep] == 0; 1: run where need[rep] != 0
    int32_t* need;                // [n_reps]
    const RepDev* real_reps;      // the pivots by position (candidate range, table row); == reps unless filtered
    int32_t* pos_map;             // [n_reps][max_ctx] position of every kept row (written by mon_sparse_score), or
                                  // nullptr: a row is its position
    const HeadDev* heads;         // mon_sparse_score: where a pivot's segments are ...
    const SegDev* segs;           // ... which rows of the pivot's block they begin at ...
    const int32_t* seg_cnt;       // ... and how many rows each of them kept
    const int32_t* surv_pos;      // [n_reps][max_ctx] positions of the kept rows, by segment
    RepDev* vreps;                // written by mon_sparse_score
    RepFilter* filt;              // checked (this step's) and set (the next step's) when not nullptr
    uint32_t* counts;             // [n_reps][4] or nullptr
    int cap_rows;                 // filtered: more kept rows than this (or fewer than the largest list) go to the dense chain
    float margin;                 // filter for the next step: cut = smallest list threshold / margin
};
struct MonBatch {
    MonItem it[HC_MAX_GROUP];
};

// Scores of a pivot's candidates to the caller's buffer: part of `parts`, by a workgroup of NT threads.  (16 bytes to a lane; both
// rows begin at a multiple of 16 bytes.)
template <int NT>
__device__ __forceinline__ void copy_scores(const MonItem& it, int rep, int lo, int hi, int part, int parts)
{
    const float* __restrict__ from = it.scores + (size_t)rep * it.ws.max_ctx;
    float* __restrict__ to = it.copy_to + (size_t)rep * it.ws.max_ctx;
#pragma unroll 4
    for (int j = (lo & ~3) + (part * NT + (int)threadIdx.x) * 4; j < hi; j += parts * NT * 4) {
        const float4 v = *reinterpret_cast<const float4*>(from + j);
        if (j >= lo && j + 4 <= hi) {
            *reinterpret_cast<float4*>(to + j) = v;
        } else {
            const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (j + c >= lo && j + c < hi) to[j + c] = x[c];
        }
    }
}

__device__ __forceinline__ bool mon_skip(const MonItem& it, int rep)
{
    return it.need_sense >= 0 && ((it.need[rep] != 0) != (it.need_sense != 0));
}

// Cross-lane moves of the data-parallel primitives (no LDS traffic, unlike a shuffle).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t other, uint32_t v)       // lanes without a source get `other`
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)other, (int)v, CTRL, ROWS, 0xF, false);
}
constexpr int DPP_SHR1 = 0x111, DPP_SHR2 = 0x112, DPP_SHR4 = 0x114, DPP_SHR8 = 0x118;      // inside rows of 16 lanes
constexpr int DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;                                    // a row's last lane to the next row / half

__device__ __forceinline__ uint32_t lane_get(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }

__device__ __forceinline__ uint32_t wave_exscan(uint32_t v, uint32_t& total)
{
    uint32_t inc = v;
    inc += dpp<DPP_SHR1>(0u, inc);
    inc += dpp<DPP_SHR2>(0u, inc);
    inc += dpp<DPP_SHR4>(0u, inc);
    inc += dpp<DPP_SHR8>(0u, inc);
    inc += dpp<DPP_BCAST15, 0xA>(0u, inc);
    inc += dpp<DPP_BCAST31, 0xC>(0u, inc);
    total = lane_get(inc, 63);
    return inc - v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    uint32_t total;
    wave_exscan(v, total);
    return total;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max(v, dpp<DPP_SHR1>(v, v));
    v = max(v, dpp<DPP_SHR2>(v, v));
    v = max(v, dpp<DPP_SHR4>(v, v));
    v = max(v, dpp<DPP_SHR8>(v, v));
    v = max(v, dpp<DPP_BCAST15, 0xA>(v, v));
    v = max(v, dpp<DPP_BCAST31, 0xC>(v, v));
    return lane_get(v, 63);
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)      // set bits of mask below this lane
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t count_true(bool x) { return (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(x)); }

// In a histogram of HC_RADIX_BINS digit counts, walking from the highest digit down, find the digit in which the
// k-th largest element falls, how many of that digit's elements are still needed and how many there are.  Done by
// ONE wave (lane l owns 32 consecutive digits); result valid in all its lanes.  The lanes start their walks at
// different digits of their spans, so that in LDS they do not all hit the same bank.
__device__ __forceinline__ void find_digit(const uint32_t* hist, uint32_t k, uint32_t& digit, uint32_t& remaining, uint32_t& count)
{
    const int lane = threadIdx.x & 63;
    constexpr int per = HC_RADIX_BINS / 64;
    static_assert(per == 32, "a lane's span");
    const uint32_t* h = hist + (HC_RADIX_BINS - (lane + 1) * per);      // lane 0 owns the highest digits
    uint32_t local = 0;
#pragma unroll 8
    for (int i = 0; i < per; ++i) local += h[(i + lane) & (per - 1)];
    uint32_t tot;
    const uint32_t above = wave_exscan(local, tot);                     // elements in higher digits than this lane's
    const uint64_t who = __builtin_amdgcn_ballot_w64(above < k && k <= above + local);
    const int src = who ? __builtin_ctzll(who) : 0;
    const uint32_t base = lane_get(above, src);
    // the digits of that lane's span, one to a lane, from the highest down
    const uint32_t* hs = hist + (HC_RADIX_BINS - (src + 1) * per);
    const uint32_t c = lane < per ? hs[per - 1 - lane] : 0u;
    const uint32_t ab = base + wave_exscan(c, tot);
    const uint64_t hit = __builtin_amdgcn_ballot_w64(ab < k && k <= ab + c);
    const int at = hit ? __builtin_ctzll(hit) : 0;
    digit = (uint32_t)(HC_RADIX_BINS - (src + 1) * per + per - 1 - at);
    remaining = k - lane_get(ab, at);
    count = lane_get(c, at);
}

// The same by a workgroup of NW waves, the answer in every thread: a wave sums its part of the digits (wave 0 the highest), one
// barrier, then each finds part, lane and digit for itself, so that nothing has to be handed round.  (A wave by itself and
// a barrier to tell the others took 0.2 us longer.)  part: LDS for NW words.
template <int NW>
__device__ __forceinline__ void find_digit_all(const uint32_t* hist, uint32_t* part, uint32_t k, uint32_t& digit, uint32_t& remaining, uint32_t& count)
{
    constexpr int PER = HC_RADIX_BINS / (NW * 64);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    auto span = [&](int w) { return hist + (HC_RADIX_BINS - (w * 64 + lane + 1) * PER); };      // a lane's digits, lane 0 the highest
    uint32_t local = 0, tot;
#pragma unroll
    for (int i = 0; i < PER; ++i) local += span(wv)[i];
    tot = wave_sum(local);
    if (lane == 0) part[wv] = tot;
    __syncthreads();
    const uint32_t mine = lane < NW ? part[lane] : 0u;
    const uint32_t above = wave_exscan(mine, tot);
    const uint64_t who = __builtin_amdgcn_ballot_w64(above < k && k <= above + mine);
    const int w = who ? __builtin_ctzll(who) : 0;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += c[i] = span(w)[i];
    const uint32_t ab = lane_get(above, w) + wave_exscan(sum, tot);
    const uint64_t hit = __builtin_amdgcn_ballot_w64(ab < k && k <= ab + sum);
    const int src = hit ? __builtin_ctzll(hit) : 0;
    uint32_t before = lane_get(ab, src);
    digit = (uint32_t)(HC_RADIX_BINS - (w * 64 + src + 1) * PER);
    remaining = count = 0u;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
        const uint32_t here = lane_get(c[i], src);
        if (before < k && k <= before + here) {
            digit += (uint32_t)i;
            remaining = k - before;
            count = here;
        }
        before += here;
    }
}

__global__ __launch_bounds__(256) void mon_prep(Ws ws)
{
    const Ws w = ws.rep(blockIdx.y);
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < HC_HIST_WORDS; i += stride) w.hist[i] = 0u;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < (size_t)ws.max_ctx / 32; i += stride) w.bitmap[i] = 0u;
}

__device__ __forceinline__ uint32_t digit_low(uint32_t digit, bool linear)                // smallest key of a digit ...
{
    if (digit == 0u) return 0u;
    return linear ? hc_score_key((float)(LinearDigits::first((int)digit) - 768) / 64.f) : (uint32_t)(FineDigits::first((int)digit) + FINE_BASE) << 17;
}
__device__ __forceinline__ uint32_t digit_last(uint32_t digit, bool linear) { return digit == HC_RADIX_BINS - 1 ? 0xffffffffu : digit_low(digit + 1u, linear) - 1u; }      // ... and the largest

// ---- the survivors of a long range ----
//
// mon_select is one workgroup with room for some tens of thousands of items, so a long range is cut down first, by many.
// The histogram of the keys' first digits (11 bits) shows the digit in which the longest list ends: everything from that digit
// up survives.  At 229,376 candidates and a longest list of 7,872 these are 8,000 to 11,000 if the scores are spread out.  But a
// digit holds every score within 25 % of each other: where it would let more through than `limit`, the cut is estimated
// instead.  What comes before some item in the order (score descending, index ascending) survives then, and that item is
// taken from a sample of the range: one position out of each of HC_SAMPLES equal pieces, at a scattered place inside it.  Of k
// list entries t = k HC_SAMPLES / n are expected in the sample, with a spread of at most sqrt(t); the sample's item number
// t + 5 sqrt(t) + 8 lies beyond the k-th item of the range but for about one sample in a million, and then (mon_select counts)
// the whole range is selected from.  The order has no ties, so how the scores are distributed does not matter: about 11,700
// of the 229,376 survive, be they all within a per cent or all equal.  One call, three set sizes, lists of 7,872 and shorter:
// 34 us with spread-out scores, 52 with scores within 2 % of each other, 64 with equal ones (a cut at the digit alone, and
// one workgroup for what it lets through: 34, 352, 424; six launches over the whole range: 56, 60, 69).
__device__ __forceinline__ int sample_row(int i, int lo, int n)
{
    const uint32_t a = (uint32_t)(((uint64_t)i * (uint32_t)n) / HC_SAMPLES), b = (uint32_t)(((uint64_t)(i + 1) * (uint32_t)n) / HC_SAMPLES);
    return lo + (int)(a + (uint32_t)(((uint64_t)((uint32_t)i * 2654435761u) * (b - a)) >> 32));
}

// The last item that survives, for lists of up to k of the n items from lo on (the whole workgroup of NT threads calls it, with
// LDS for HC_RADIX_BINS and HC_SAMPLES / 32 words).
template <int NT, class ScoreAt>
__device__ __forceinline__ void sample_threshold(uint32_t* sm_hist, uint32_t* sm_tied, int lo, int n, int k, const ScoreAt& score_at, uint32_t& key_out, int& row_out)
{
    constexpr int PER = HC_SAMPLES / NT;
    const float t = (float)k * ((float)HC_SAMPLES / (float)n);
    const float place = t + 5.0f * sqrtf(t) + 8.0f;
    key_out = 0u;
    row_out = 0x7fffffff;
    if (place >= (float)HC_SAMPLES) return;          // everything survives (the same for every thread)
    uint32_t key[PER], rem = (uint32_t)place, prefix = 0, count;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        key[u] = hc_score_key(score_at(sample_row(u * NT + (int)threadIdx.x, lo, n)));
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);       // (four loads in flight: more only cost registers)
    }
#pragma unroll 1
    for (int shift = 21; shift >= 0; shift = shift == 21 ? 10 : shift - 10) {      // digits of 11, 11 and 10 bits
        const uint32_t known = shift == 21 ? 0u : shift == 10 ? 0xffe00000u : 0xfffffc00u, width = shift == 0 ? 1023u : 2047u;
        __syncthreads();
        for (int i = threadIdx.x; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const bool in = ((key[u] ^ prefix) & known) == 0u;
            const uint64_t m = __builtin_amdgcn_ballot_w64(in);
            const uint32_t digit = (key[u] >> shift) & width, one = m ? lane_get(digit, __builtin_ctzll(m)) : 0u;
            if (m == __builtin_amdgcn_ballot_w64(in && digit == one)) {      // (near-equal scores: one sum instead of 64 in turn)
                if (m && (threadIdx.x & 63) == 0) atomicAdd(&sm_hist[one], (uint32_t)__builtin_popcountll(m));
            } else if (in) {
                atomicAdd(&sm_hist[digit], 1u);
            }
        }
        __syncthreads();
        uint32_t digit;
        find_digit(sm_hist, rem, digit, rem, count);
        prefix |= digit << shift;
    }
    key_out = prefix;
    // of the sample's items with that key, the rem-th in position order
    for (int i = threadIdx.x; i < HC_SAMPLES / 32; i += NT) sm_tied[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (key[u] == prefix) atomicOr(&sm_tied[(u * NT + (int)threadIdx.x) >> 5], 1u << (threadIdx.x & 31));
    __syncthreads();
    const int lane = threadIdx.x & 63;
    static_assert(HC_SAMPLES / 32 == 128, "two words to a lane");
    const uint32_t w0 = sm_tied[2 * lane], w1 = sm_tied[2 * lane + 1], c0 = (uint32_t)__builtin_popcount(w0), c1 = (uint32_t)__builtin_popcount(w1);
    uint32_t tot;
    const uint32_t before = wave_exscan(c0 + c1, tot);
    const uint64_t who = __builtin_amdgcn_ballot_w64(before < rem && rem <= before + c0 + c1);
    const int src = who ? __builtin_ctzll(who) : 0;
    const uint32_t a0 = lane_get(w0, src), a1 = lane_get(w1, src);
    uint32_t left = rem - lane_get(before, src);     // 1 .. set bits of the two words
    uint64_t bits = ((uint64_t)a1 << 32) | a0;
    for (; left > 1u; --left) bits &= bits - 1;
    row_out = sample_row(src * 64 + (bits ? __builtin_ctzll(bits) : 0), lo, n);
}

// Scores and histogram of a long candidate range (over the first 11 bits of the keys, or the digits that mon_direct reads).  A workgroup takes `span` consecutive chunks of
// HC_SEL_CHUNK candidates: the histogram in LDS is cleared and flushed once for all of them.
// most: as many candidates as mon_direct will go through (a captured call may find more than when it was launched).
template <int G, int HIST>
__global__ __launch_bounds__(BLK) void mon_score_hist(MonBatch B, int scores_given, int agg, int span, int long_lists, int max_k, int most)
{
    __shared__ uint32_t sh[HC_RADIX_BINS];
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    RepDev rd = it.reps[rep];
    if (HIST != HIST_KEYS) rd.hi = min(rd.hi, rd.lo + most);
    const int c0 = blockIdx.x * span, c1 = min(c0 + span, rd.nchunk);
    if (c0 >= rd.nchunk) return;
    float* srow = it.scores + (size_t)rep * it.ws.max_ctx;
    const float* lrow = it.rep_logits ? it.rep_logits + (size_t)rep * G * it.ws.max_ctx : nullptr;
    float l[G];
#pragma unroll
    for (int g = 0; g < G; ++g) l[g] = (!scores_given && agg == HC_AGG_PROB) ? it.lse[(size_t)rd.bh * G + g] : 0.f;
    for (int i = threadIdx.x; i < HC_RADIX_BINS; i += BLK) sh[i] = 0u;
    if (HIST == HIST_KEYS && long_lists) {                       // a slice each: the later histograms cleared, the baseline list to its bitmap
        const Ws w = it.ws.rep(rep);
        const int first = blockIdx.x * BLK + threadIdx.x, step = (rd.nchunk + span - 1) / span * BLK;
        const int lo = it.real_reps[rep].lo, hi = it.real_reps[rep].hi;
        const int32_t* base = it.base_idx + (size_t)rd.bh * max_k;
        for (int i = first; i < 2 * HC_MAX_K_PER_REP * HC_RADIX_BINS; i += step) w.h2[i] = 0u;
        for (int i = first; i < rd.k[0]; i += step) {
            const int j = base[i] - lo;
            if (j >= 0 && j < hi - lo) atomicOr(&w.bitmap[j >> 5], 1u << (j & 31));
        }
    }
    __syncthreads();
    for (int ch = c0; ch < c1; ++ch) {
        const int first = rd.lo + ch * HC_SEL_CHUNK;
        float x[SCORE_PER_THREAD];
#pragma unroll
        for (int i = 0; i < SCORE_PER_THREAD; ++i) {       // candidate first + i*BLK + t: coalesced, loads independent
            const int j = first + i * BLK + threadIdx.x;
            x[i] = 0.f;
            if (j < rd.hi) x[i] = scores_given ? srow[j] : score_of<G>(lrow, j, l, agg);
        }
        count_scores<HIST>(sh, scores_given ? nullptr : srow, first, rd.hi, x);
    }
    __syncthreads();
    flush_counts(it.ws.rep(rep).hist, sh);
}

// The survivors are kept as one bit per candidate: nothing to reserve, little to write, few bits for mon_select to read.  A wave
// takes a chunk at a time, 64 candidates to a round.
constexpr int ROUNDS = HC_SEL_CHUNK / 64;
__device__ __forceinline__ void load_chunk(float (&s)[ROUNDS], const float* __restrict__ srow, int lo, int hi, int ch)
{
    const int first = lo + ch * HC_SEL_CHUNK + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) s[r] = srow[min(first + r * 64, hi - 1)];
}

// (Its first loads do not wait for the cut.)
__global__ __launch_bounds__(BLK, 8) void mon_compact(MonBatch B, int limit)
{
    __shared__ __attribute__((aligned(16))) uint32_t sm_hist[HC_RADIX_BINS];
    __shared__ uint32_t sm_tied[HC_SAMPLES / 32];
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    const RepDev rd = it.reps[rep];
    const int lane = threadIdx.x & 63, stride = gridDim.x * NWAVE;
    int ch = blockIdx.x * NWAVE + (threadIdx.x >> 6);
    if ((int)blockIdx.x * NWAVE >= rd.nchunk) return;
    const Ws w = it.ws.rep(rep);
    const float* srow = it.scores + (size_t)rep * it.ws.max_ctx;
    float s[ROUNDS];
    uint4 h[HC_RADIX_BINS / 4 / BLK];
#pragma unroll
    for (int i = 0; i < HC_RADIX_BINS / 4 / BLK; ++i) h[i] = reinterpret_cast<const uint4*>(w.hist)[i * BLK + threadIdx.x];
    load_chunk(s, srow, rd.lo, rd.hi, ch);
#pragma unroll
    for (int i = 0; i < HC_RADIX_BINS / 4 / BLK; ++i) reinterpret_cast<uint4*>(sm_hist)[i * BLK + threadIdx.x] = h[i];
    int row_max = 0x7fffffff, kmax = 1;
    for (int ks = 0; ks < rd.nk; ++ks) kmax = max(kmax, it.reps[rep].k[ks]);      // (indexing the register copy would spill it)
    __syncthreads();
    uint32_t digit, remaining, count;
    find_digit(sm_hist, (uint32_t)kmax, digit, remaining, count);
    uint32_t key_min = digit << 21;
    if ((uint32_t)kmax - remaining + count > (uint32_t)limit) {       // (the same for every thread)
        sample_threshold<BLK>(sm_hist, sm_tied, rd.lo, rd.hi - rd.lo, kmax, [&](int j) { return srow[j]; }, key_min, row_max);
        load_chunk(s, srow, rd.lo, rd.hi, ch);
    }
    for (; ch < rd.nchunk; ch += stride) {
        const int first = rd.lo + ch * HC_SEL_CHUNK + lane;
        uint32_t lo = 0, hi = 0;                     // lane r: round r's mask
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t key = hc_score_key(s[r]);
            const int j = first + r * 64;
            const uint64_t m = __builtin_amdgcn_ballot_w64(j < rd.hi && (key > key_min || (key == key_min && j <= row_max)));
            lo = lane == r ? (uint32_t)m : lo;
            hi = lane == r ? (uint32_t)(m >> 32) : hi;
        }
        if (lane < ROUNDS) w.mask[(size_t)ch * ROUNDS + lane] = ((uint64_t)hi << 32) | lo;
        if (ch + stride < rd.nchunk) load_chunk(s, srow, rd.lo, rd.hi, ch + stride);
    }
}

struct DriftCfg {
    int window, metric, tau_num, tau_den, max_k, tumbling, agg;
};

// ---- the decision ----

// What a decision needs of a pivot's ring row: how many values the window holds (the same in every lane), and value `lane`.
struct RingRow {
    int32_t count, value;
};
__device__ __forceinline__ RingRow ring_row(const MonItem& it, int bh, int window)
{
    const int32_t* rg = it.ring + (size_t)bh * (window + 1);
    const int lane = threadIdx.x & 63;
    RingRow r;
    r.value = lane < window ? rg[1 + lane] : 0;
    r.count = __builtin_amdgcn_readfirstlane(rg[0]);
    return r;
}

// Window update, decision, baseline update of a pivot, and the filter of the next step: by the whole workgroup (NT threads),
// after the lists are written.  inter: |T ∩ baseline|; tmin: the smallest list threshold, rows: how many rows the lists were
// taken from (both only for a filtering layer), lse: of query head `lane` of the group (likewise).  Every wave decides for
// itself, in registers (a window has at most 64 values, one to a lane), and the first writes it down: with the values and the
// verdict passed through LDS, five barriers, this took 0.5 us longer.
template <int NT>
__device__ __forceinline__ void decide(const MonItem& it, int rep, int bh, int rows, int k, const DriftCfg& cfg, int n_group, const RingRow& row,
                                       int32_t inter, uint32_t tmin, float lse)
{
    static_assert(HC_MAX_WINDOW <= 64, "a window's values, one to a lane");
    const int tid = threadIdx.x, lane = tid & 63;
    int32_t* rg = it.ring + (size_t)bh * (cfg.window + 1);
    if (it.store_slot == -2) return;                 // the lists were all that was wanted
    int cnt = row.count;
    if (cnt < 0 || cnt > cfg.window) cnt = 0;
    if (it.store_slot != -1) {
        // A buffered query of the window scored again at the test step (Algorithm 1): its overlap replaces
        // the one stored when the query was current.  Only while the ring is one short of full, i.e. the
        // monitor call that follows is the one that tests.
        if (tid == 0 && cnt == cfg.window - 1 && it.store_slot < cnt) rg[1 + it.store_slot] = inter;
        return;
    }
    const int drop = cnt == cfg.window ? 1 : 0;      // sliding window: the oldest value leaves
    const int m = cnt - drop + 1;                    // values in the window after the push
    int32_t value = drop ? __shfl_down(row.value, 1) : row.value;
    if (lane == m - 1) value = inter;
    int rank = 0;
    for (int j = 0; j < m; ++j) {                    // the lower median is found by ranking
        const int32_t o = (int32_t)lane_get((uint32_t)value, j);
        rank += o < value || (o == value && j < lane);
    }
    const uint64_t middle = __builtin_amdgcn_ballot_w64(lane < m && rank == (m - 1) / 2);
    const int32_t med = (int32_t)lane_get((uint32_t)value, middle ? __builtin_ctzll(middle) : 0);
    bool trig = false;
    if (m == cfg.window) {
        const long long kl = k;
        if (cfg.metric == HC_METRIC_OVERLAP)
            trig = (long long)med * cfg.tau_den < (long long)cfg.tau_num * kl;                     // med/k < tau
        else
            trig = (long long)med * cfg.tau_den < (long long)cfg.tau_num * (2 * kl - med);         // med/(2k-med) < tau
    }
    if (tid < 64) {
        if (lane < m) rg[1 + lane] = value;
        if (lane == 0) {
            // the window restarts after a retrieval; a tumbling window after every test
            rg[0] = (trig || (cfg.tumbling && m == cfg.window)) ? 0 : m;
            it.inter[bh] = inter;
            it.flag[bh] = trig;
            if (it.counts) {                         // (added without waiting for what was there)
                uint32_t* cn = it.counts + (size_t)rep * 4;
                atomicAdd(&cn[0], (uint32_t)(m == cfg.window));
                atomicAdd(&cn[1], (uint32_t)trig);
                atomicAdd(&cn[2], (uint32_t)(it.need_sense == 1));
                cn[3] = it.need_sense == 0 ? (uint32_t)rows : 0xffffffffu;
            }
        }
        if (it.filt) {
            // The filter of the next step's split pass: rows whose statistic, taken against this step's
            // log-sum-exp, stays below the smallest list threshold of this step divided by the margin are dropped.
            const float t = key_score(tmin);
            const float cutsum = (t > 0.f && t < 1.0e30f && it.margin >= 1.f) ? (float)n_group * t / it.margin : 0.f;
            RepFilter* f = it.filt + rep;
            if (lane < 8) f->ref[lane] = lane < n_group ? lse * 1.4426950408889634f : 0.f;
            if (lane == 8) f->cutsum = cutsum;
            if (lane == 9) f->armed = 1;
            if (lane < 6) f->pad[lane] = 0;
        }
    }
    if (trig) {                                      // K_base <- K_t
        __syncthreads();                             // (the list is written)
        const int32_t* src = it.topk_idx + (size_t)bh * cfg.max_k;
        int32_t* base = it.base_idx + (size_t)bh * cfg.max_k;
        for (int i = tid; i < k; i += NT) base[i] = src[i];
    }
}

// ---- the selection ----
//
// One workgroup per pivot and set size (blockIdx.y); the one of set size 0, the monitored list, also takes the
// decision.  Items are the pivot's candidates in position order: SRC_SCORES finds their scores in place (of the rows a
// filtering split pass kept, whose positions pos_map names, or of a short range), SRC_SURVIVORS takes what mon_compact left, SRC_RANGE cuts the range down itself.  Their keys are kept in LDS: `cap` of them;
// items beyond that are read again from the scores in every pass, so that any number of items is handled.  (Survivors
// that are fewer than the longest list or do not all fit, about one sample in a million, are given up for the range.)
//
// Threshold: the keys' range [smallest, largest] is cut into 2048 equal bins, so that the bins are evenly filled
// whatever the scores' scale is (a fixed top digit of the key would put most items into a handful of bins, whose
// LDS atomics then serialise).  The bin of the k-th key usually holds a few dozen items: they are collected and
// ranked by counting.  A bin with more (ties, extreme outliers) is cut again.
//
// The kernel is a chain of latencies and, with one wave per SIMD (beside the attention pass) or four (alone), of
// issue slots: every pass takes GROUP items a lane at a time, whose reads are issued together before the first is
// used, and set sizes go to workgroups of their own because the passes behind the histogram cost the same for each
// of them (one workgroup for all: 97 us for 16,700 rows and three set sizes with 256 threads; one each: 43; with 512
// threads of half the registers, two waves per SIMD: 28).
// (COPY: behind the `lists` rows of the grid that are set sizes there are workgroups that copy scores, see copy_scores.)
enum { SRC_SCORES = 1, SRC_SURVIVORS = 2, SRC_RANGE = 3 };
constexpr int SEL_LIST = 128;        // members of a threshold bin that are ranked by counting

constexpr int SEL_KEYS(int words) { return words / 264 * 256; }           // keys, with their masks, that fit in so many words (whole 256s)
constexpr int SEL_OUTS = 64;         // rows a list goes to that are kept at hand (in the lanes of a register)

// From memory to LDS without passing through registers, so that any number can be in flight: 4 or 16 bytes per lane,
// the lanes' pieces one behind the other in LDS.  dma_wait() before they are read.  (The wait is the builtin, which the
// compiler's own counting of outstanding accesses understands: after an opaque one it would wait again, for every
// store issued since, at each read of LDS.)
__device__ __forceinline__ void dma4(const void* src_of_lane, void* lds_of_wave)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src_of_lane,
                                     (__attribute__((address_space(3))) void*)lds_of_wave, 4, 0, 0);
}
__device__ __forceinline__ void dma16(const void* src_of_lane, void* lds_of_wave)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src_of_lane,
                                     (__attribute__((address_space(3))) void*)lds_of_wave, 16, 0, 0);
}
__device__ __forceinline__ void dma_wait()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// words[0, n) to lds[0, n rounded up to 256) by the waves first, first + step, ... of 256 words each; what is past the
// end repeats words before it.  (words + n rounded up to 4 must be readable where words is 16-byte aligned.)
__device__ __forceinline__ void dma_run(const void* words, uint32_t* lds, int n, int first, int step)
{
    const int lane = threadIdx.x & 63;
    const char* src = reinterpret_cast<const char*>(words);
    if (((uintptr_t)words & 15) == 0) {
        for (int b = first; b * 256 < n; b += step) dma16(src + (uint32_t)min(b * 256 + lane * 4, (n - 1) & ~3) * 4u, lds + b * 256);
    } else {
        for (int b = first; b * 64 < n; b += step) dma4(src + (uint32_t)min(b * 64 + lane, n - 1) * 4u, lds + b * 64);
    }
}

template <int NT, int SRC, bool COPY>
__global__ __launch_bounds__(NT) void mon_select(MonBatch B, DriftCfg cfg, int n_group, int lds_words, int lists)
{
    constexpr int NW = NT / 64, GROUP = NT == 512 ? 4 : 8;      // (four keep the small form within 40 registers)
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    __shared__ uint32_t sm_hist[HC_RADIX_BINS];
    __shared__ uint32_t sm_list[SEL_LIST];
    __shared__ uint32_t sm_lo, sm_shift, sm_rem, sm_cnt, sm_tau, sm_need, sm_ties, sm_nlist;
    __shared__ uint32_t sm_min[NW], sm_max[NW], sm_hits[NW], sm_gt[NW], sm_eq[NW];
    __shared__ uint32_t sm_wsum[NW];

    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.x, ks = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int max_ctx = it.ws.max_ctx;
    const RepDev rd = it.reps[rep];
    if (ks >= rd.nk) {
        if (COPY && ks >= lists) copy_scores<NT>(it, rep, rd.lo, rd.hi, ks - lists, (int)gridDim.y - lists);
        return;
    }
    const bool deciding = ks == 0;
    const Ws w = it.ws.rep(rep);
    const int32_t* pmap = it.pos_map ? it.pos_map + (size_t)rep * max_ctx : nullptr;
    float* srow = it.scores + (size_t)rep * max_ctx;
    const int k = it.reps[rep].k[ks];
    int k_longest = 1;
    for (int i = 0; i < rd.nk; ++i) k_longest = max(k_longest, it.reps[rep].k[i]);      // (indexing the register copy would spill it)
    const int real_lo = it.real_reps[rep].lo, real_hi = it.real_reps[rep].hi;   // the bitmap is indexed by position
    const int bw = deciding ? (real_hi - real_lo + 31) / 32 : 0;               // words of the baseline bitmap
    for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
    // what the decision needs from memory is asked for now
    RingRow ring{0, 0};
    if (deciding && it.store_slot != -2) ring = ring_row(it, rd.bh, cfg.window);
    const bool checks = deciding && it.need_sense == 0 && it.filt != nullptr;
    const float cutsum = checks ? it.filt[rep].cutsum : 0.f;
    float ref_minus_lse = -INFINITY, lse_of = 0.f;   // lane g: of query head g of the group, the first in log2 units
    if (deciding && it.filt && lane < n_group) lse_of = it.lse[(size_t)rd.bh * n_group + lane];
    if (checks && lane < n_group) ref_minus_lse = it.filt[rep].ref[lane] - lse_of * 1.4426950408889634f;
    // the rows this list goes to, one to a lane
    uint32_t v_row = 0;
    int n_rows = -1;                                 // -1: too many for the lanes, looked up when they are needed
    if (rd.out_count <= SEL_OUTS) {
        const OutDev od = it.outs[rd.out_begin + min(lane, rd.out_count - 1)];
        const bool mine = lane < rd.out_count && od.kslot == ks;
        uint64_t rows = __builtin_amdgcn_ballot_w64(mine);
        n_rows = __builtin_popcountll(rows);
        for (int i = 0; rows != 0; ++i, rows &= rows - 1) {
            const uint32_t row = lane_get((uint32_t)od.row, __builtin_ctzll(rows));
            v_row = lane == i ? row : v_row;
        }
    }

    int n = rd.hi - rd.lo;
    bool surv = false;                   // the items are survivors
    // survivors: a thread takes a run of the masks of 64 candidates, whose survivors are items first_item on
    const int rounds_all = rd.nchunk * (HC_SEL_CHUNK / 64), per_thread = (rounds_all + NT - 1) / NT;
    const int m_begin = min(tid * per_thread, rounds_all), m_end = min(m_begin + per_thread, rounds_all);
    uint32_t first_item = 0;
    if (SRC == SRC_RANGE) {
        static_assert(SEL_LIST >= HC_SAMPLES / 32, "the sample's ties");
        uint32_t key_min;
        int row_max;
        sample_threshold<NT>(sm_hist, sm_list, rd.lo, n, k_longest, [&](int j) { return srow[j]; }, key_min, row_max);
        // through LDS, as much of the range as there is room for at a time: all of its loads are in flight at once
        const int part = lds_words / HC_SEL_CHUNK * HC_SEL_CHUNK;
        for (int b = 0; b < n; b += part) {
            const int here = min(part, n - b);
            __syncthreads();
            dma_run(srow + rd.lo + b, dyn, here, wv, NW);
            dma_wait();
            __syncthreads();
            for (int r = wv; r * 64 < here; r += NW) {
                const uint32_t key = hc_score_key(__uint_as_float(dyn[r * 64 + lane]));
                const int i = r * 64 + lane;
                const uint64_t m = __builtin_amdgcn_ballot_w64(i < here && (key > key_min || (key == key_min && rd.lo + b + i <= row_max)));
                if (lane == 0) w.mask[b / 64 + r] = m;                 // (the same in every set size's workgroup)
            }
        }
        for (int r = (n + 63) / 64 + tid; r < rd.nchunk * ROUNDS; r += NT) w.mask[r] = 0u;
        __syncthreads();
        for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
    }
    if (SRC >= SRC_SURVIVORS) {
        uint32_t mine = 0, tot, all = 0;
#pragma unroll 4
        for (int m = m_begin; m < m_end; ++m) mine += (uint32_t)__builtin_popcountll(w.mask[m]);
        first_item = wave_exscan(mine, tot);
        if (lane == 0) sm_wsum[wv] = tot;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            first_item += i < wv ? sm_wsum[i] : 0u;
            all += sm_wsum[i];
        }
        surv = all >= (uint32_t)k_longest && all <= (uint32_t)min(w.sv_cap, SEL_KEYS(lds_words));
        if (surv) n = (int)all;
    }
    // Dynamic LDS: the keys (a multiple of 256 of them), a mask per 64 keys saying which are in the list, and the
    // baseline bitmap if it fits behind the items (otherwise the one in the workspace is used).
    const bool bm_lds = (bw <= lds_words && SEL_KEYS(lds_words - bw) >= n) || (bw <= lds_words / 2 && SEL_KEYS(lds_words) < n);
    const int cap = min(SEL_KEYS(lds_words - (bm_lds ? bw : 0)), (n + 255) & ~255);
    uint32_t* sm_key = dyn;
    uint64_t* sm_mask = reinterpret_cast<uint64_t*>(dyn + cap);
    uint32_t* sm_bm = dyn + cap + cap / 32;
    if (bm_lds)
        for (int i = tid; i < bw; i += NT) sm_bm[i] = 0u;
    __syncthreads();
    const bool fits = n <= cap;
    if (deciding) {                      // baseline list -> bitmap
        const int32_t* base = it.base_idx + (size_t)rd.bh * cfg.max_k;
        for (int i0 = tid; i0 < k; i0 += GROUP * NT) {
            int j[GROUP];
#pragma unroll
            for (int u = 0; u < GROUP; ++u) j[u] = i0 + u * NT < k ? base[i0 + u * NT] : -1;
#pragma unroll
            for (int u = 0; u < GROUP; ++u)
                if (j[u] >= real_lo && j[u] < real_hi) {
                    const int jj = j[u] - real_lo;
                    if (bm_lds) atomicOr(&sm_bm[jj >> 5], 1u << (jj & 31));
                    else atomicOr(&w.bitmap[jj >> 5], 1u << (jj & 31));
                }
        }
    }

    // ---- the items' keys, and their range ----
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    auto put = [&](int i, uint32_t key) {
        if (i < cap) sm_key[i] = key;
        kmin = min(kmin, key);
        kmax = max(kmax, key);
    };
    if (SRC >= SRC_SURVIVORS && surv) {
        // the survivors' rows of the range, then in their places their keys; the positions go to a table
        for (int m = m_begin; m < m_end; ++m)
            for (uint64_t bits = w.mask[m]; bits != 0; bits &= bits - 1) sm_key[first_item++] = (uint32_t)(m * 64 + __builtin_ctzll(bits));
        __syncthreads();
        constexpr int U = NT == 512 ? 4 : 8;
        for (int i0 = tid; i0 < n; i0 += U * NT) {
            float s[U];
            int row[U];
#pragma unroll
            for (int u = 0; u < U; ++u) row[u] = i0 + u * NT < n ? rd.lo + (int)sm_key[i0 + u * NT] : rd.lo;      // (its own items only: another's may be a key by now)
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] = srow[row[u]];
            if (pmap) {
#pragma unroll
                for (int u = 0; u < U; ++u) row[u] = pmap[row[u]];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * NT;
                if (i < n) {
                    put(i, hc_score_key(s[u]));
                    w.sv_pos[i] = row[u];
                }
            }
        }
    } else {
        // the scores that fit, 64 to a round, straight to LDS; then each turned into its key in place
        const int nd = min(n, cap);
        dma_run(srow + rd.lo, sm_key, nd, wv, NW);
        dma_wait();
        __syncthreads();
        constexpr int U = GROUP;
        for (int i0 = tid; i0 < nd; i0 += U * NT) {
            float s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] = __uint_as_float(sm_key[min(i0 + u * NT, nd - 1)]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < nd) put(i0 + u * NT, hc_score_key(s[u]));
        }
        for (int i = nd + tid; i < n; i += NT) put(i, hc_score_key(srow[rd.lo + i]));
    }
    kmin = ~wave_max(~kmin);
    kmax = wave_max(kmax);
    if (lane == 0) {
        sm_min[wv] = kmin;
        sm_max[wv] = kmax;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        kmin = min(kmin, sm_min[i]);
        kmax = max(kmax, sm_max[i]);
    }

    // GROUP keys of a lane: items first, first + step, ... (those past the end read some item's key)
    auto keys_of = [&](uint32_t (&key)[GROUP], int first, int step) {
        if (fits) {
#pragma unroll
            for (int u = 0; u < GROUP; ++u) key[u] = sm_key[min(first + u * step, n - 1)];
        } else {
#pragma unroll
            for (int u = 0; u < GROUP; ++u) key[u] = sm_key[min(first + u * step, cap - 1)];
            if (first + (GROUP - 1) * step >= cap) {
#pragma unroll
                for (int u = 0; u < GROUP; ++u)
                    if (first + u * step >= cap)
                        key[u] = hc_score_key(*reinterpret_cast<const float*>(reinterpret_cast<const char*>(srow) + (uint32_t)(rd.lo + min(first + u * step, n - 1)) * 4u));
            }
        }
    };

    // ---- threshold key, ties to take and ties there are, for a list of kt items; the answer in sm_tau / sm_need /
    // sm_ties (the whole workgroup calls it; sm_hist holds the histogram of all items over [kmin, kmax]) ----
    const uint32_t range = kmax - kmin;
    const uint32_t shift = range < HC_RADIX_BINS ? 0u : 21u - (uint32_t)__builtin_clz(range);       // range >> shift < 2048
    auto histogram = [&]() {
        if (range == 0u) return;                     // all equal
        for (int i0 = tid; i0 < n; i0 += GROUP * NT) {
            uint32_t key[GROUP];
            keys_of(key, i0, NT);
            if (i0 - tid + GROUP * NT <= n) {
#pragma unroll
                for (int u = 0; u < GROUP; ++u) atomicAdd(&sm_hist[(key[u] - kmin) >> shift], 1u);
            } else {
#pragma unroll
                for (int u = 0; u < GROUP; ++u)
                    if (i0 + u * NT < n) atomicAdd(&sm_hist[(key[u] - kmin) >> shift], 1u);
            }
        }
        __syncthreads();
    };
    auto threshold = [&](int kt) {
        if (wv == 0) {
            uint32_t digit = 0u, rem = (uint32_t)kt, count = (uint32_t)n;
            if (range != 0u) find_digit(sm_hist, (uint32_t)kt, digit, rem, count);
            if (lane == 0) {
                sm_lo = kmin + (digit << shift);
                sm_shift = shift;
                sm_rem = rem;
                sm_cnt = count;
                sm_nlist = 0u;
                sm_tau = 0xffffffffu;
                sm_need = sm_ties = 0u;
            }
        }
        __syncthreads();
        while (sm_cnt > SEL_LIST && sm_shift > 0u) {                     // (the same for every thread)
            const uint32_t lo = sm_lo, s = sm_shift, s2 = s > 11u ? s - 11u : 0u, k2 = sm_rem;
            __syncthreads();
            for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
            __syncthreads();
            for (int i0 = tid; i0 < n; i0 += GROUP * NT) {
                uint32_t key[GROUP];
                keys_of(key, i0, NT);
#pragma unroll
                for (int u = 0; u < GROUP; ++u)
                    if (i0 + u * NT < n && key[u] >= lo && ((key[u] - lo) >> s) == 0u) atomicAdd(&sm_hist[(key[u] - lo) >> s2], 1u);
            }
            __syncthreads();
            if (wv == 0) {
                uint32_t digit, rem, count;
                find_digit(sm_hist, k2, digit, rem, count);
                if (lane == 0) {
                    sm_lo = lo + (digit << s2);
                    sm_shift = s2;
                    sm_rem = rem;
                    sm_cnt = count;
                }
            }
            __syncthreads();
        }
        const uint32_t lo = sm_lo, s = sm_shift, rem = sm_rem;
        if (s == 0u) {                               // the bin is a single key
            if (tid == 0) {
                sm_tau = lo;
                sm_need = rem;
                sm_ties = sm_cnt;
            }
        } else {
            for (int i0 = tid; i0 < n; i0 += GROUP * NT) {
                uint32_t key[GROUP];
                keys_of(key, i0, NT);
#pragma unroll
                for (int u = 0; u < GROUP; ++u)
                    if (key[u] - lo < 1u << s && i0 + u * NT < n) {         // (lo + 2^s does not pass the largest 32-bit value)
                        const uint32_t at = atomicAdd(&sm_nlist, 1u);
                        if (at < SEL_LIST) sm_list[at] = key[u];
                    }
            }
            __syncthreads();
            if (wv == 0) {                           // one member to a lane (or two), compared with all of them
                const int m = (int)min(sm_nlist, (uint32_t)SEL_LIST);
                const uint32_t a = lane < m ? sm_list[lane] : 0u;
                uint32_t gt_a = 0, eq_a = 0;
                auto settle = [&](bool one, uint32_t key, uint32_t gt, uint32_t eq) {
                    if (one && gt < rem && rem <= gt + eq) {              // (equal keys write equal values)
                        sm_tau = key;
                        sm_need = rem - gt;
                        sm_ties = eq;
                    }
                };
                if (m <= 64) {
                    for (int i = 0; i < m; ++i) {
                        const uint32_t o = lane_get(a, i);
                        gt_a += o > a;
                        eq_a += o == a;
                    }
                } else {
                    const uint32_t b = lane + 64 < m ? sm_list[lane + 64] : 0u;
                    uint32_t gt_b = 0, eq_b = 0;
                    for (int i = 0; i < m; ++i) {
                        const uint32_t o = i < 64 ? lane_get(a, i) : lane_get(b, i - 64);
                        gt_a += o > a;
                        eq_a += o == a;
                        gt_b += o > b;
                        eq_b += o == b;
                    }
                    settle(lane + 64 < m, b, gt_b, eq_b);
                }
                settle(lane < m, a, gt_a, eq_a);
            }
        }
        __syncthreads();
    };
    uint32_t tmin = 0;                               // deciding, with a filter: the smallest list threshold
#pragma unroll 1
    for (bool longest = deciding && it.filt && k_longest != k;; longest = false) {
        histogram();
        threshold(longest ? k_longest : k);
        tmin = longest || k_longest == k ? sm_tau : tmin;
        if (!longest) break;
        __syncthreads();
        for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;       // (a bin may have been cut again)
        __syncthreads();
    }
    const uint32_t tau = sm_tau, need = sm_need;
    const bool all_ties = need == sm_ties;           // every item at the threshold is taken: the usual case

    bool decided_elsewhere = false;
    if (checks && cutsum > 0.f) {
        // The check of this step's filter.  The split pass dropped the rows whose statistic sum_g 2^(t_g - ref_g)
        // stayed below cutsum; with this step's own log-sum-exp such a row's score is below
        // (cutsum / G) max_g 2^(ref_g - lse_g).  If even the smallest list threshold found among the kept rows
        // reaches that bound (with room for the rounding of the statistic), no dropped row belongs to any list and
        // the lists are those of all rows.  Otherwise the dense chain redoes this pivot from all of its logits.
        // (Only the deciding workgroup looks and sets the filter: the others' lists are then written again.)
        const float d = exp2f(ref_minus_lse);
        float delta = 0.f;
        for (int g = 0; g < n_group; ++g) delta = fmaxf(delta, __uint_as_float(lane_get(__float_as_uint(d), g)));
        const float bound = cutsum / (float)n_group * delta * 1.0001f;
        if (!(key_score(tmin) >= bound)) {
            decided_elsewhere = true;
            if (tid == 0) it.need[rep] = 5;
        }
    }

    uint32_t hits = 0, lane_hits = 0;                // of the wave; of a lane
    if (!decided_elsewhere) {
        // The usual case: every round's choice is known now and kept as a mask; the keys are done with, and where the
        // positions come from a table, the run's part of it takes their place.
        const bool masked = fits && all_ties;
        const int32_t* table = SRC >= SRC_SURVIVORS && surv ? w.sv_pos : pmap ? pmap + rd.lo : nullptr;
        // A wave takes a run of the items, 64 to a round, GROUP rounds at a time.  First how many keys above (and at)
        // the threshold its run holds; then, from the runs before it, where its own entries go, and the list in
        // position order with |T ∩ baseline| of the monitored one.
        const int rounds = (n + 63) / 64;
        // (a table's run is copied 256 entries at a time)
        const int per = table && masked ? ((rounds + NW - 1) / NW + 3) & ~3 : (rounds + NW - 1) / NW;
        const int i_begin = min(wv * per * 64, n), i_end = min(i_begin + per * 64, n);
        const uint32_t floor_key = all_ties ? tau : tau + 1u;            // taken whatever its rank (tau is at most the key of +inf)
        uint32_t gt = 0, eq = 0;
        for (int i0 = i_begin; i0 < i_end; i0 += GROUP * 64) {
            uint32_t key[GROUP], mask_lo = 0, mask_hi = 0;
            keys_of(key, i0 + lane, 64);
#pragma unroll
            for (int u = 0; u < GROUP; ++u) {
                uint64_t m = __builtin_amdgcn_ballot_w64(key[u] >= floor_key);
                const int left = i_end - (i0 + u * 64);          // of this round's items
                if (left < 64) m = left > 0 ? m & ((1ull << left) - 1ull) : 0ull;
                gt += (uint32_t)__builtin_popcountll(m);
                mask_lo = lane == u ? (uint32_t)m : mask_lo;
                mask_hi = lane == u ? (uint32_t)(m >> 32) : mask_hi;
            }
            if (masked && lane < GROUP && i0 + lane * 64 < i_end) sm_mask[(i0 >> 6) + lane] = ((uint64_t)mask_hi << 32) | mask_lo;
            if (!all_ties) {
#pragma unroll
                for (int u = 0; u < GROUP; ++u) eq += count_true(i0 + u * 64 + lane < i_end && key[u] == tau);
            }
        }
        if (masked && table) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // (the run's keys are in no other wave's way)
            dma_run(table + i_begin, sm_key + i_begin, i_end - i_begin, 0, 1);
        }
        if (lane == 0) {
            sm_gt[wv] = gt;
            sm_eq[wv] = eq;
        }
        __syncthreads();
        uint32_t out = 0, eqb = 0;                   // entries before this run; ties before it, of which `need` are entries
        for (int i = 0; i < wv; ++i) {
            out += sm_gt[i] + min(sm_eq[i], need > eqb ? need - eqb : 0u);
            eqb += sm_eq[i];
        }
        out = (uint32_t)__builtin_amdgcn_readfirstlane((int)out);
        eqb = (uint32_t)__builtin_amdgcn_readfirstlane((int)eqb);
        dma_wait();
        if (masked && bm_lds && n_rows >= 0) {
            // (nothing but LDS is read here: a read of memory would wait for the stores before it)
            const uint32_t* bm = sm_bm;
            for (int i0 = i_begin; i0 < i_end; i0 += GROUP * 64) {
                const uint64_t masks = lane < GROUP && i0 + lane * 64 < i_end ? sm_mask[(i0 >> 6) + lane] : 0ull;       // lane u: round u
                int pos[GROUP];
                if (table) {
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) pos[u] = (int)sm_key[min(i0 + u * 64, cap - 64) + lane];
                } else {
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) pos[u] = rd.lo + i0 + u * 64 + lane;
                }
                uint64_t sel[GROUP];
                uint32_t dst[GROUP];                 // byte offset of the entry in its list
#pragma unroll
                for (int u = 0; u < GROUP; ++u) {
                    sel[u] = ((uint64_t)lane_get((uint32_t)(masks >> 32), u) << 32) | lane_get((uint32_t)masks, u);
                    dst[u] = min(out + lanes_below(sel[u]), (uint32_t)k - 1u) * 4u;      // (always below k; the limit keeps a corrupt state in bounds)
                    out += (uint32_t)__builtin_popcountll(sel[u]);
                }
                for (int o = 0; o < n_rows; ++o) {
                    char* list = reinterpret_cast<char*>(it.topk_idx + (size_t)lane_get(v_row, o) * cfg.max_k);
#pragma unroll
                    for (int u = 0; u < GROUP; ++u)
                        if (__builtin_amdgcn_inverse_ballot_w64(sel[u])) *reinterpret_cast<int32_t*>(list + dst[u]) = pos[u];
                }
                if (deciding) {
                    uint32_t word[GROUP];
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) {
                        pos[u] = __builtin_amdgcn_inverse_ballot_w64(sel[u]) ? pos[u] - real_lo : 0;
                        word[u] = bm[pos[u] >> 5];
                    }
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) hits += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((word[u] >> (pos[u] & 31)) & 1u) & sel[u]);
                }
            }
        } else {
#pragma unroll 1
            for (int i0 = i_begin; i0 < i_end; i0 += 64) {
                const int i = i0 + lane;
                const bool in = i < i_end;
                bool sel = false;
                int pos = 0;
                if (masked) {
                    sel = in && ((sm_mask[i0 >> 6] >> lane) & 1u);
                    pos = table ? (int)sm_key[min(i, cap - 1)] : rd.lo + i;
                } else {
                    const uint32_t key = !in ? 0u : i < cap ? sm_key[i] : hc_score_key(srow[rd.lo + i]);
                    pos = !in ? 0 : table ? table[i] : rd.lo + i;
                    const bool is_eq = in && key == tau;
                    const uint64_t eqm = __builtin_amdgcn_ballot_w64(is_eq);
                    sel = in && (key > tau || (is_eq && eqb + lanes_below(eqm) < need));
                    eqb += (uint32_t)__builtin_popcountll(eqm);
                }
                const uint64_t selm = __builtin_amdgcn_ballot_w64(sel);
                const uint32_t dst = min(out + lanes_below(selm), (uint32_t)k - 1u);
                out += (uint32_t)__builtin_popcountll(selm);
                if (!sel) continue;
                if (deciding) {
                    const int jj = pos - real_lo;
                    const uint32_t word = bm_lds ? sm_bm[jj >> 5] : __hip_atomic_load(&w.bitmap[jj >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    lane_hits += (word >> (jj & 31)) & 1u;
                }
                if (n_rows >= 0) {
                    for (int o = 0; o < n_rows; ++o) it.topk_idx[(size_t)lane_get(v_row, o) * cfg.max_k + dst] = pos;
                } else {
                    for (int o = 0; o < rd.out_count; ++o)
                        if (it.outs[rd.out_begin + o].kslot == ks) it.topk_idx[(size_t)it.outs[rd.out_begin + o].row * cfg.max_k + dst] = pos;
                }
            }
        }
    }
    if (!deciding) return;
    hits += wave_sum(lane_hits);
    if (lane == 0) sm_hits[wv] = hits;
    __syncthreads();

    // ---- the next call finds histogram and bitmap clear ----
    if (SRC == SRC_SURVIVORS)
        for (int i = tid; i < HC_RADIX_BINS; i += NT) w.hist[i] = 0u;
    if (!bm_lds)
        for (int i = tid; i < bw; i += NT) w.bitmap[i] = 0u;
    if (decided_elsewhere) return;

    // ---- window, decision, baseline ----
    int32_t inter = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) inter += (int32_t)sm_hits[i];
    decide<NT>(it, rep, rd.bh, rd.hi, k, cfg, n_group, ring, inter, tmin, lse_of);
}

// ---- the selection straight from the scores ----
//
// For up to 64 K candidates (beside the attention pass 32 K, for few lists 64 K), and for the rows a filtering split pass kept: one workgroup per
// pivot and set size, as mon_select, behind a launch that left the scores and their histogram (DIRECT_HIST), behind
// mon_sparse_score (DIRECT_MAP: kept rows), or by itself over a short range (DIRECT_LOGITS, or DIRECT_SCORES where the scores
// are given).  The histogram names the digit in which the list ends.  A wave then goes once through its run of the items, 1024 to a tile, 16 consecutive ones to a lane:
// what lies above that digit is in the list, a bit per item (a compare and an add with carry each); what lies in it, a hundred
// items or so, is ranked by counting in the order of the lists (score descending, index ascending), which leaves no ties to
// resolve; and the list is written from the bits.  No keys are made, kept or moved.  Where the digit holds more than BAND items it
// is cut again, over the scores.
//
// What bounds it is latency and issue: with 16 waves, an instruction that all of them execute takes 16 cycles of every SIMD.
// (With the items 64 to a round, one to a lane, and ballots, going through 32K of them took 4.3 us of the launch.)
// One pivot, three set sizes, us per call with the launch before it, and in brackets by mon_compact and mon_select (and
// mon_score_hist).  Given scores spread out / within 2 % of each other / equal: 10,000 candidates 15 / 19 / 19 (23 / 33 / 34), 32,768 19 /
// 24 / 25 (25 / 37 / 43), 65,000 25 / 33 / 37 (32 / 35 / 57).  Mean logits (HC_AGG_LOGIT) of any offset, spread out / within 0.1 %: 10,000
// 16 / 20 (24-27 / 27), 32,768 21 / 25-29 (27-40 / 40-43), 65,000 27-29 / 35-43 (35-49 / 48-53).  Given scores that are not what HC_AGG_PROB
// makes of logits, negative or above 2, end in a digit without an edge: 10,000 20 (23), 32,768 26-28 (25), 65,000 37-41 (32-34).  By
// itself, 4,096 candidates 12.2 / 12.3 / 12.0 (mon_select over keys 13.4 / 13.7 /
// 11.7), 8,192 15.4 / 15.2 / 14.3 (16.5 / 16.6 / 16.2).  Steps of four 32K layers with a drift at each, overlapped: 105 us (120).
constexpr int BAND = 512;                // items of the digit that can be ranked ...
constexpr int RANKED = 128;              // ... without a histogram of their own
constexpr int DIRECT_TILES = 4;          // of a wave: two words to a lane
static_assert(HC_SCORED_MOST + 3 == 1024 / 64 * DIRECT_TILES * HC_SEL_CHUNK, "what the large form goes through");

enum { DIRECT_HIST = 0, DIRECT_MAP = 1, DIRECT_SCORES = 2, DIRECT_LOGITS = 3 };
template <int NT, int SRC, int G, bool COPY>
__global__ __launch_bounds__(NT) void mon_direct(MonBatch B, DriftCfg cfg, int n_group, int bufs, int most, int bm_words, int lists)
{
    constexpr int NW = NT / 64, TILE = HC_SEL_CHUNK;
    constexpr bool MAP = SRC == DIRECT_MAP, HERE = SRC != DIRECT_HIST;   // HERE: the histogram is made by this workgroup
    static_assert(TILE == 1024, "16 items to a lane");
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];       // [bufs][NW][TILE] scores, a bit per item, the baseline bitmap
    __shared__ __attribute__((aligned(16))) uint32_t sm_hist[HC_RADIX_BINS];
    __shared__ uint64_t sm_band[BAND];
    __shared__ uint32_t sm_rank[RANKED], sm_part[NW], sm_count[NW], sm_eq[NW], sm_hits[NW], sm_nband, sm_nrank, sm_tau, sm_least, sm_most, sm_own[4];

    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.x, ks = blockIdx.y;
    if (rep >= it.n_reps) return;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const Ws w = it.ws.rep(rep);
    const RepDev rd = it.reps[rep];
    const int need_of = MAP ? it.need[rep] : 0;
    if (COPY && ks >= lists) {                       // (as in mon_select)
        copy_scores<NT>(it, rep, rd.lo, min(rd.hi, rd.lo + most), ks - lists, (int)gridDim.y - lists);
        return;
    }
    // (1 to 4: the pivot was handed on before it had a histogram; 5: by this launch's deciding workgroup)
    if (ks >= rd.nk || (need_of != 0 && need_of != 5)) return;
    const bool deciding = ks == 0;
    const int max_ctx = it.ws.max_ctx;
    // items are counted from a multiple of four positions (where they are read 16 bytes at a time), those from `first` to `end` - 1 are
    // candidates
    constexpr int ALIGN = SRC == DIRECT_LOGITS ? ~0 : ~3;
    const int lo4 = rd.lo & ALIGN, first = rd.lo - lo4, end = min(rd.hi - rd.lo, most) + first;     // (most: what the launch was sized for)
    float* srow = it.scores + (size_t)rep * max_ctx + lo4;
    const int tiles = (end + TILE - 1) / TILE, per = (tiles + NW - 1) / NW;      // (at most DIRECT_TILES: the launch sees to it)
    const int t0 = min(tiles, wv * per), t1 = min(tiles, t0 + per);

    // everything from memory is asked for now
    OutDev od{};
    if (rd.out_count <= SEL_OUTS) od = it.outs[rd.out_begin + min(lane, rd.out_count - 1)];
    int k = rd.k[0], k_longest = 1;
#pragma unroll
    for (int i = 0; i < HC_MAX_K_PER_REP; ++i) {     // (a loop over memory would be a chain of reads, a variable index would spill the copy)
        if (i == ks) k = rd.k[i];
        if (i < rd.nk) k_longest = max(k_longest, rd.k[i]);
    }
    const int real_lo = (MAP ? it.real_reps[rep].lo : rd.lo) & ALIGN, real_hi = min(MAP ? it.real_reps[rep].hi : rd.hi, real_lo + bm_words * 32);      // the bitmap is indexed by position
    const int bw = deciding ? (real_hi - real_lo + 31) / 32 : 0;
    const bool checks = MAP && deciding && it.need_sense == 0 && it.filt != nullptr;      // (a filter's rows come with a map)
    const float cutsum = checks ? it.filt[rep].cutsum : 0.f;
    float ref_of = -INFINITY, lse_of = 0.f;          // lane g: of query head g of the group
    if (checks && lane < n_group) lse_of = it.lse[(size_t)rd.bh * n_group + lane];
    if (checks && lane < n_group) ref_of = it.filt[rep].ref[lane];
    constexpr int HV = HC_RADIX_BINS / 4, HP = (HV + NT - 1) / NT;       // 16-byte pieces of the histogram, of a thread
    uint4 h[HP];
    if (!HERE) {
#pragma unroll
        for (int i = 0; i < HP; ++i) h[i] = reinterpret_cast<const uint4*>(w.hist)[min(i * NT + tid, HV - 1)];
    }
    RingRow ring{0, 0};
    if (deciding && it.store_slot != -2) ring = ring_row(it, rd.bh, cfg.window);
    // A tile goes straight to LDS, 16 bytes to a lane.  Lane o's items are pieces 4 o .. 4 o + 3 there, their order turned by o / 4, so
    // that 16 lanes reading theirs find 16 different groups of banks.
    auto buffer = [&](int t) { return dyn + ((t - t0) % bufs * NW + wv) * TILE; };
    auto fetch = [&](int t) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int piece = (16 * j + (lane >> 2)) * 4 + ((lane & 3) ^ ((lane >> 4) & 3));
            dma16(srow + min(t * TILE + piece * 4, (end - 1) & ~3), buffer(t) + j * 256);
        }
    };
    if (SRC != DIRECT_LOGITS)
        for (int t = t0; t < min(t1, t0 + bufs); ++t) fetch(t);
    // logits: item tid + u NT of each round of U NT (the first round's are asked for now)
    constexpr int U = SRC != DIRECT_LOGITS ? 1 : (NT == 512 ? 2 : 4) / (G >= 8 ? 2 : 1);
    const float* lrow = SRC == DIRECT_LOGITS ? it.rep_logits + ((size_t)rep * max_ctx + lo4) * G : nullptr;
    float row[U][G], lse_g[G];
    auto rows = [&](int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_row<G>(lrow, min(i0 + u * NT, end - 1), row[u]);
    };
    if (SRC == DIRECT_LOGITS) {
#pragma unroll
        for (int g = 0; g < G; ++g) lse_g[g] = cfg.agg == HC_AGG_PROB ? it.lse[(size_t)rd.bh * G + g] : 0.f;
        rows(tid);
    }
    // the rows this list goes to, one to a lane
    uint32_t v_row = 0;
    int n_rows = -1;                                 // -1: too many for the lanes, looked up when they are needed
    if (rd.out_count <= SEL_OUTS) {
        uint64_t rows = __builtin_amdgcn_ballot_w64(lane < rd.out_count && od.kslot == ks);
        n_rows = __builtin_popcountll(rows);
        for (int i = 0; rows != 0; ++i, rows &= rows - 1) {
            const uint32_t row = lane_get((uint32_t)od.row, __builtin_ctzll(rows));
            v_row = lane == i ? row : v_row;
        }
    }
    uint32_t* sm_bits = dyn + bufs * NW * TILE;      // [tiles * 32]: chosen items
    uint32_t* sm_bm = sm_bits + tiles * (TILE / 32);
    constexpr int GROUP = NT == 512 ? 4 : 8;
    const int32_t* base = it.base_idx + (size_t)rd.bh * cfg.max_k;
    int j_base[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) j_base[u] = deciding && tid + u * NT < k ? base[tid + u * NT] : -1;
    for (int i = tid; i < tiles * (TILE / 32) + bw; i += NT) sm_bits[i] = 0u;
    if (tid < RANKED) sm_rank[tid] = 0u;
    if (tid == 0) {
        sm_nband = sm_nrank = 0u;
        sm_least = 0xffffffffu;
        sm_most = 0u;
    }
    if (HERE) {
        for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
    } else {
#pragma unroll
        for (int i = 0; i < HP; ++i)
            if (i * NT + tid < HV) reinterpret_cast<uint4*>(sm_hist)[i * NT + tid] = h[i];
    }
    __syncthreads();
    uint32_t ticket = 0;                             // (through with the histogram in memory; looked at in the end)
    if (!HERE && tid == 0) ticket = atomicAdd(w.hist + HC_RADIX_BINS, 1u);
    if (deciding) {                                  // baseline list -> bitmap
        for (int i0 = tid;;) {
#pragma unroll
            for (int u = 0; u < GROUP; ++u)
                if (j_base[u] >= real_lo && j_base[u] < real_hi) atomicOr(&sm_bm[(j_base[u] - real_lo) >> 5], 1u << ((j_base[u] - real_lo) & 31));
            i0 += GROUP * NT;
            if (i0 - tid >= k) break;
#pragma unroll
            for (int u = 0; u < GROUP; ++u) j_base[u] = i0 + u * NT < k ? base[i0 + u * NT] : -1;
        }
    }
    // tile t is in LDS and the wave may read it; and it has been read: its place may take the one `bufs` further on
    auto arrived = [&](int t) {
        if (SRC == DIRECT_LOGITS) return;
        if (t == t0 || bufs == 1 || t >= t0 + bufs) dma_wait();          // (at first: for all that are in flight)
    };
    auto leave = [&](int t) {
        if (SRC != DIRECT_LOGITS && t + bufs < t1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
            fetch(t + bufs);
        }
    };
    const int turn = (lane >> 2) & 3;
    // Where the histogram is made of all candidates its digits are spread over what there is of keys, 2048 for [k_lo, k_hi].  (Digits
    // of fixed width took 4 us longer for scores within 2 % of each other: all items in one or two of them, then cut again.)
    uint32_t k_lo = 0, k_hi = 0, k_shift = 0;
    if (SRC == DIRECT_LOGITS || SRC == DIRECT_SCORES) {
        uint32_t least = 0xffffffffu, greatest = 0u;
        // (every tile is at its number's place: a tile to a wave)
        auto item_at = [&](int at) { return (at & ~15) | ((((at >> 2) & 3) ^ ((at >> 6) & 3)) << 2) | (at & 3); };
        if (SRC == DIRECT_LOGITS) {
            for (int i0 = tid; i0 < end; i0 += U * NT) {
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = hc_group_score<G>(row[u], lse_g, cfg.agg);
                if (i0 - tid + U * NT < end) rows(i0 + U * NT);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + u * NT;
                    if (i < end) {
                        const uint32_t key = hc_score_key(x[u]);
                        if (deciding) srow[i] = x[u];
                        dyn[item_at(i)] = __float_as_uint(x[u]);
                        least = min(least, key);
                        greatest = max(greatest, key);
                    }
                }
            }
        } else {
            if (t0 < t1) arrived(t0);
            __syncthreads();
            for (int at = tid; at < tiles * TILE; at += NT) {
                const int i = item_at(at);
                const uint32_t key = hc_score_key(__uint_as_float(dyn[at]));
                if (i >= first && i < end) {
                    least = min(least, key);
                    greatest = max(greatest, key);
                }
            }
        }
        least = ~wave_max(~least);
        greatest = wave_max(greatest);
        if (lane == 0) {
            atomicMin(&sm_least, least);
            atomicMax(&sm_most, greatest);
        }
        __syncthreads();
        k_lo = sm_least;
        k_hi = sm_most;
        const uint32_t range = k_hi - k_lo;
        k_shift = range < HC_RADIX_BINS ? 0u : 21u - (uint32_t)__builtin_clz(range);
        if (range != 0u)
            for (int at = tid; at < tiles * TILE; at += NT) {
                const int i = item_at(at);
                if (i >= first && i < end) atomicAdd(&sm_hist[(hc_score_key(__uint_as_float(dyn[at])) - k_lo) >> k_shift], 1u);
            }
        __syncthreads();
    } else if (HERE) {                               // few items, and digits of a few of them each: the histogram is made here
        // (issue bound: 12,700 rows took 4.7 us of the launch with key, digit and place of an item in 28 instructions; with 11 of them
        // 3.2, a step of four layers of 224K on one stream 255 -> 251 us)
        for (int t = t0; t < t1; ++t) {
            arrived(t);
            const float* tile = reinterpret_cast<const float*>(buffer(t));
            const int left = end - t * TILE;
            if (left >= TILE) {                      // (any order will do)
#pragma unroll 1
                for (int j = 0; j < 4; ++j) {
                    const float4 v = *reinterpret_cast<const float4*>(tile + (j * 64 + lane) * 4);
                    atomicAdd(&sm_hist[fine_digit(v.x)], 1u);
                    atomicAdd(&sm_hist[fine_digit(v.y)], 1u);
                    atomicAdd(&sm_hist[fine_digit(v.z)], 1u);
                    atomicAdd(&sm_hist[fine_digit(v.w)], 1u);
                }
            } else {
#pragma unroll 4
                for (int j = 0; j < 16; ++j) {
                    const int at = j * 64 + lane, i = (at & ~15) | ((((at >> 2) & 3) ^ ((at >> 6) & 3)) << 2) | (at & 3);
                    if (i < left) atomicAdd(&sm_hist[fine_digit(tile[at])], 1u);
                }
            }
            leave(t);
        }
        if (per > bufs)
            for (int t = t0; t < min(t1, t0 + bufs); ++t) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_s_waitcnt(0xC07F);
                fetch(t);
            }
        __syncthreads();
    }

    // ---- the digit in which the list ends: keys [lo, lo + wide], `count` items of which `rem` are in the list ----
    uint32_t digit, rem, count, tmin = 0u;
    const bool linear = SRC == DIRECT_HIST && cfg.agg == HC_AGG_LOGIT;
    auto find = [&](uint32_t k_of) {
        if ((SRC == DIRECT_LOGITS || SRC == DIRECT_SCORES) && k_lo == k_hi) {
            digit = 0u;
            rem = k_of;
            count = (uint32_t)(end - first);
        } else {
            find_digit_all<NW>(sm_hist, sm_part, k_of, digit, rem, count);
        }
        return SRC == DIRECT_LOGITS || SRC == DIRECT_SCORES ? k_lo + (digit << k_shift) : digit_low(digit, linear);
    };
    auto width = [&](uint32_t from) {                // (digits do not reach beyond what was counted in them)
        return SRC == DIRECT_LOGITS || SRC == DIRECT_SCORES ? min((1u << k_shift) - 1u, k_hi - from) : digit_last(digit, linear) - from;
    };
    uint32_t lo = find((uint32_t)k), wide = width(lo);
    // The filter's threshold is the smallest of all lists, to one part in 65,536: the edge of its digit would let more rows through,
    // and the lowest digit has no number at its edge, so that the check would fail at every step.
    bool for_filter = checks && k_longest != k;
    if (for_filter) {
        if (tid == 0) {                              // (this list's digit, meanwhile in LDS)
            sm_own[0] = lo;
            sm_own[1] = wide;
            sm_own[2] = rem;
            sm_own[3] = count;
        }
        __syncthreads();
        lo = find((uint32_t)k_longest);
        wide = width(lo);
    }
    // A digit with more items than can be ranked is cut again: its smallest and largest key are looked for first, then what
    // lies between is counted in 2048 parts.  (Counted in parts of the digit's width at once, equal ones summed over a wave because they
    // are in each other's way, an item to a lane: 32,768 items within 2 % of each other 27.8 us a call, equal 33.3; this way 23.6 and
    // 24.9.  65,800: 41.2 and 52.4; 32.6 and 36.9.)
    bool measured = false;
    for (;;) {                                       // (the same for every thread)
        if (for_filter ? wide < 128u : count <= BAND || wide == 0u) {
            if (!for_filter) break;
            for_filter = measured = false;
            tmin = lo;
            lo = sm_own[0];
            wide = sm_own[1];
            rem = sm_own[2];
            count = sm_own[3];
            continue;
        }
        const uint32_t shift = wide < HC_RADIX_BINS ? 0u : 21u - (uint32_t)__builtin_clz(wide);      // wide >> shift < 2048
        __syncthreads();
        if (measured) {
            for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
        } else if (tid == 0) {
            sm_least = 0xffffffffu;
            sm_most = 0u;
        }
        __syncthreads();
        uint32_t least = 0xffffffffu, greatest = 0u;
        // (positive numbers compare as their bits do; the tiles are still in LDS unless a wave has more of them than buffers; any order will do)
        auto pass = [&](auto raw, auto here) {
            constexpr bool RAW = decltype(raw)::value, LDS = decltype(here)::value;
            constexpr int R = SRC == DIRECT_LOGITS || NT == 512 ? (MAP ? 1 : 2) : 4;     // reads of a lane in flight
            const uint32_t from = RAW ? lo & 0x7fffffffu : lo;
#pragma unroll 1
            for (int t = t0; t < t1; ++t) {
                const bool whole = t * TILE >= first && (t + 1) * TILE <= end;
#pragma unroll 1
                for (int p0 = 4 * lane; p0 < TILE; p0 += 256 * R) {
                    float4 v[R];
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        if (LDS) v[u] = *reinterpret_cast<const float4*>(buffer(t) + p0 + 256 * u);
                        else v[u] = *reinterpret_cast<const float4*>(srow + min(t * TILE + p0 + 256 * u, (end - 1) & ~3));
                    }
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                        uint32_t d[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) d[c] = (RAW ? __float_as_uint(x[c]) : hc_score_key(x[c])) - from;
                        if (!whole) {
                            const int p = p0 + 256 * u, i = t * TILE + (LDS ? (p & ~15) | ((p ^ (p >> 4)) & 12) : p);
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                if (i + c < first || i + c >= end) d[c] = 0xffffffffu;       // (no candidate; wide is less)
                        }
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            if (measured) {
                                if (d[c] <= wide) atomicAdd(&sm_hist[d[c] >> shift], 1u);
                            } else {
                                least = min(least, d[c]);
                                greatest = d[c] <= wide ? max(greatest, d[c]) : greatest;
                            }
                        }
                    }
                }
            }
        };
        const bool raw = lo > 0x80000000u && lo + wide < 0xff800000u;
        if constexpr (SRC == DIRECT_LOGITS) {
            pass(std::false_type{}, std::true_type{});
        } else if constexpr (NT == 512) {            // (more forms would take registers)
            pass(std::false_type{}, std::false_type{});
        } else if (per <= bufs) {
            arrived(t0);
            if (raw) pass(std::true_type{}, std::true_type{});
            else pass(std::false_type{}, std::true_type{});
        } else {
            if (raw) pass(std::true_type{}, std::false_type{});
            else pass(std::false_type{}, std::false_type{});
        }
        if (!measured) {
            least = ~wave_max(~least);
            greatest = wave_max(greatest);
            if (lane == 0) {
                atomicMin(&sm_least, least);
                atomicMax(&sm_most, greatest);
            }
            __syncthreads();
            lo += sm_least;
            wide = sm_least <= sm_most ? sm_most - sm_least : 0u;        // (there is one, unless the histogram is not of these scores)
            measured = true;
        } else {
            __syncthreads();
            find_digit_all<NW>(sm_hist, sm_part, rem, digit, rem, count);
            wide = min((1u << shift) - 1u, wide - (digit << shift));
            lo += digit << shift;
            measured = false;
        }
    }

    // ---- above it, in it, below it ----
    uint32_t w0 = 0, w1 = 0;                         // a lane's items of tiles t0, t0 + 1 (16 bits each) and of t0 + 2, t0 + 3
    const bool tied = count > BAND;                  // one key, more items than can be ranked
    uint32_t e0 = 0, e1 = 0;                         // tied: the items with that key
    // As floats the scores compare as their keys do, but for what is no number (below everything either way, unless `lo` is).
    const bool plain = !tied && lo >= 0x80000000u && lo + wide < 0xff800000u;
    const float f_lo = key_score(lo), f_hi = key_score(lo + wide + 1u);
    for (int t = t0; t < t1; ++t) {
        arrived(t);
        const uint32_t* tile = buffer(t);
        const int i0 = t * TILE + 16 * lane;
        uint32_t above = 0, from = 0;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            const float4 v = *reinterpret_cast<const float4*>(tile + lane * 16 + (q ^ turn) * 4);
            const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int c = 3; c >= 0; --c) {
                if (plain) {
                    asm("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(above) : "s"(f_hi), "v"(x[c]) : "vcc");
                    asm("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(from) : "s"(f_lo), "v"(x[c]) : "vcc");
                } else {
                    const uint32_t key = hc_score_key(x[c]);
                    above = above + above + (key > lo + wide);
                    from = from + from + (key >= lo);
                }
            }
        }
        // (of the lane's items, the candidates)
        uint32_t valid = end - i0 >= 16 ? 0xffffu : end > i0 ? (1u << (end - i0)) - 1u : 0u;
        if (first > i0) valid &= 0xffffu << (first - i0);
        above &= valid;
        uint32_t band = from & valid & ~above;
        if (!tied) {
            const int o = lane * 16;
            for (; band != 0u; band &= band - 1u) {
                const int c = __builtin_ctz(band);
                const uint32_t at = atomicAdd(&sm_nband, 1u);
                if (at < BAND)
                    sm_band[at] = ((uint64_t)hc_score_key(__uint_as_float(tile[o + ((c >> 2) ^ turn) * 4 + (c & 3)])) << 32) | (uint32_t)~(i0 + c);
            }
        }
        const int at = (t - t0) & 1 ? 16 : 0;
        if (t - t0 < 2) {
            w0 |= above << at;
            e0 |= band << at;
        } else {
            w1 |= above << at;
            e1 |= band << at;
        }
        leave(t);
    }
    // counts of a word's two tiles, in 16 bits each
    auto counts = [](uint32_t x) { return (uint32_t)__builtin_popcount(x & 0xffffu) | (uint32_t)__builtin_popcount(x >> 16) << 16; };
    auto total = [&]() { return wave_sum((uint32_t)(__builtin_popcount(w0) + __builtin_popcount(w1))); };
    if (!tied) {
        const uint32_t mine = total();
        if (lane == 0) sm_count[wv] = mine;
        __syncthreads();
        auto choose = [&](uint64_t b) {
            const int i = (int)~(uint32_t)b;
            atomicOr(&sm_bits[i >> 5], 1u << (i & 31));
            atomicAdd(&sm_count[(i / TILE) / per], 1u);
        };
        int m = (int)min(sm_nband, (uint32_t)BAND);
        const uint64_t* list = sm_band;
        if (m > RANKED) {                            // a histogram over the digit first (the tiles are done with: their place takes the rest)
            uint64_t* rest = reinterpret_cast<uint64_t*>(dyn);
            const uint32_t shift = wide < HC_RADIX_BINS ? 0u : 21u - (uint32_t)__builtin_clz(wide);
            for (int i = tid; i < HC_RADIX_BINS; i += NT) sm_hist[i] = 0u;
            __syncthreads();
            const uint64_t b = sm_band[min(tid, m - 1)];
            const uint32_t d = ((uint32_t)(b >> 32) - lo) >> shift;
            if (tid < m) atomicAdd(&sm_hist[d], 1u);
            __syncthreads();
            find_digit_all<NW>(sm_hist, sm_part, rem, digit, rem, count);
            if (tid < m && d > digit) choose(b);
            if (tid < m && d == digit) rest[atomicAdd(&sm_nrank, 1u)] = b;
            __syncthreads();
            list = rest;
            m = (int)sm_nrank;
        }
        for (int m0 = 0; m0 < m; m0 += RANKED) {     // (once, unless hundreds are equal or nearly so)
            // rank of the items m0 on: NT threads for all pairs
            const int here = min(m - m0, RANKED), bits = here <= 1 ? 0 : 32 - __builtin_clz(here - 1);         // 2^bits >= here
            const int item = tid & ((1 << bits) - 1), parts = NT >> bits, each = (m + parts - 1) / parts;
            const int j0 = (tid >> bits) * each, j1 = min(m, j0 + each);
            const uint64_t own = list[m0 + min(item, here - 1)];
            uint32_t larger = 0;
#pragma unroll 4
            for (int j = j0; j < j1; ++j) larger += list[j] > own;
            if (item < here && larger) atomicAdd(&sm_rank[item], larger);
            __syncthreads();
            if (tid < here) {
                const uint64_t b = list[m0 + tid];
                const uint32_t rank = sm_rank[tid];
                if (rank < rem) choose(b);
                if (rank == rem - 1u) sm_tau = (uint32_t)(b >> 32);
                sm_rank[tid] = 0u;
            }
            __syncthreads();
        }
    } else {
        // of the items with that key the first `rem`
        uint32_t in0 = counts(e0), in1 = counts(e1), tot0, tot1;
        in0 = wave_exscan(in0, tot0);
        in1 = wave_exscan(in1, tot1);
        if (lane == 0) sm_eq[wv] = (tot0 & 0xffffu) + (tot0 >> 16) + (tot1 & 0xffffu) + (tot1 >> 16);
        __syncthreads();
        uint32_t before = 0;
        for (int i = 0; i < wv; ++i) before += sm_eq[i];
        auto first_of = [&](uint32_t e, uint32_t ahead) {                // those of e's items that are among the first `rem`
            const uint32_t take = rem > ahead ? rem - ahead : 0u;
            if (take == 0u) return 0u;
            while ((uint32_t)__builtin_popcount(e) > take) e &= ~(0x80000000u >> __builtin_clz(e));
            return e;
        };
        const uint32_t b1 = before + (tot0 & 0xffffu), b2 = b1 + (tot0 >> 16), b3 = b2 + (tot1 & 0xffffu);
        w0 |= first_of(e0 & 0xffffu, before + (in0 & 0xffffu)) | first_of(e0 & 0xffff0000u, b1 + (in0 >> 16));
        w1 |= first_of(e1 & 0xffffu, b2 + (in1 & 0xffffu)) | first_of(e1 & 0xffff0000u, b3 + (in1 >> 16));
        const uint32_t mine = total();
        if (lane == 0) sm_count[wv] = mine;
        if (tid == 0) sm_tau = lo;
        __syncthreads();
    }
    const uint32_t tau = sm_tau;
    if (k_longest == k) tmin = tau;

    bool decided_elsewhere = false;
    if (checks && cutsum > 0.f) {                    // the check of this step's filter: see mon_select
        const float d = exp2f(ref_of - lse_of * 1.4426950408889634f);
        float delta = 0.f;
        for (int g = 0; g < n_group; ++g) delta = fmaxf(delta, __uint_as_float(lane_get(__float_as_uint(d), g)));
        const float bound = cutsum / (float)n_group * delta * 1.0001f;
        if (!(key_score(tmin) >= bound)) {
            decided_elsewhere = true;
            if (tid == 0) it.need[rep] = 5;
        }
    }

    uint32_t hits = 0;
    if (!decided_elsewhere) {
        // ---- the list, and |T ∩ baseline|: item numbers to LDS (in the tiles' place), from there to the rows ----
        uint32_t out = 0;
        for (int i = 0; i < wv; ++i) out += sm_count[i];
        const uint16_t* half = reinterpret_cast<const uint16_t*>(sm_bits);           // a lane's items of tile t: half[64 t + lane]
        const int32_t* pmap = MAP ? it.pos_map + (size_t)rep * max_ctx + lo4 : nullptr;
        const uint32_t room = (uint32_t)(bufs * NW * TILE);
        for (uint32_t from = 0; from < (uint32_t)k; from += room) {      // (once, but for lists of more than 8,192 or 16,384)
            uint32_t before = out;
            for (int t = t0; t < t1; ++t) {
                const uint32_t x = t - t0 < 2 ? w0 : w1;
                uint32_t bits = ((t - t0) & 1 ? x >> 16 : x & 0xffffu) | half[t * 64 + lane], all;
                uint32_t at = before - from + wave_exscan((uint32_t)__builtin_popcount(bits), all);
                before += all;
                const int i0 = t * TILE + 16 * lane;
                if (!MAP && deciding && from == 0u)
                    hits += (uint32_t)__builtin_popcount(bits & (i0 < end ? sm_bm[i0 >> 5] >> (i0 & 16) : 0u));      // (an item's number is its bit of the bitmap)
                for (; bits != 0u; bits &= bits - 1u, ++at)
                    if (at < room) dyn[at] = (uint32_t)(i0 + __builtin_ctz(bits));
            }
            if (!MAP && deciding && from == 0u) {
                hits = wave_sum(hits);
                if (lane == 0) sm_hits[wv] = hits;
            }
            __syncthreads();
            const int n_out = (int)min((uint32_t)k - from, room);
            for (int i0 = tid; i0 < n_out; i0 += GROUP * NT) {
                int pos[GROUP];
#pragma unroll
                for (int u = 0; u < GROUP; ++u) pos[u] = min((int)dyn[min(i0 + u * NT, n_out - 1)], end - 1);        // (the limit keeps a corrupt state in bounds)
#pragma unroll
                for (int u = 0; u < GROUP; ++u) pos[u] = MAP ? pmap[pos[u]] : lo4 + pos[u];
                if (MAP && deciding) {
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) {
                        const int jj = min(max(pos[u], real_lo), real_hi - 1) - real_lo;
                        if (i0 + u * NT < n_out) hits += (sm_bm[jj >> 5] >> (jj & 31)) & 1u;
                    }
                }
                auto store = [&](int row) {
                    int32_t* list = it.topk_idx + (size_t)row * cfg.max_k + from;
#pragma unroll
                    for (int u = 0; u < GROUP; ++u)
                        if (i0 + u * NT < n_out) list[i0 + u * NT] = pos[u];
                };
                if (n_rows >= 0) {
                    for (int o = 0; o < n_rows; ++o) store((int)lane_get(v_row, o));
                } else {
                    for (int o = 0; o < rd.out_count; ++o)
                        if (it.outs[rd.out_begin + o].kslot == ks) store(it.outs[rd.out_begin + o].row);
                }
            }
            if (from + room < (uint32_t)k) __syncthreads();
        }
    }
    if (deciding && !decided_elsewhere) {
        if (MAP) {
            hits = wave_sum(hits);
            if (lane == 0) sm_hits[wv] = hits;
            __syncthreads();
        }
        int32_t inter = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) inter += (int32_t)sm_hits[i];
        decide<NT>(it, rep, rd.bh, rd.hi, k, cfg, n_group, ring, inter, tmin, lse_of);
    }
    // ---- the next call finds the histogram clear: the last of the pivot's workgroups to have read it sees to it ----
    if (!HERE && wv == 0 && __builtin_amdgcn_readfirstlane((int)ticket) == rd.nk - 1) {
        for (int i = lane; i < HV; i += 64) reinterpret_cast<uint4*>(w.hist)[i] = make_uint4(0u, 0u, 0u, 0u);
        if (lane == 0) w.hist[HC_RADIX_BINS] = 0u;
    }
}

// ---- long lists ----
//
// A workgroup per list is only as good as the lists are short (its time grows with them).  Lists of more than about 9,500
// entries are selected by many workgroups in six launches: mon_score_hist, two more digits of the keys (11 + 10 bits), counts per
// chunk, ordered write, decision.  229,376 candidates, a longest list of 40,000: 52 us with spread-out scores, 56 within 2 % of
// each other, 68 equal (by mon_select over the range: 408, 365, 472).

// The keys of four consecutive candidates, positions first4 .. first4 + 3 (first4 a multiple of 4: one 16-byte load), of which
// those inside [lo, hi) count.
__device__ __forceinline__ void load_keys(const float* __restrict__ srow, int first4, int lo, int hi, uint32_t (&key)[4], bool (&in)[4])
{
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (first4 < hi) v = *reinterpret_cast<const float4*>(srow + first4);     // (row stride a multiple of 64: in bounds)
    const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        in[i] = first4 + i >= lo && first4 + i < hi;
        key[i] = hc_score_key(f[i]);
    }
}

// dst[0, n) = src[0, n) by a workgroup of BLK threads (n a multiple of 4 BLK, both 16-byte aligned).
__device__ __forceinline__ void copy_words(uint32_t* dst, const uint32_t* __restrict__ src, int n)
{
#pragma unroll 4
    for (int i = threadIdx.x; i < n / 4; i += BLK) reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
}

// These passes work on chunks that start at a multiple of 4 positions, which can add one.
__device__ __forceinline__ int chunks_from_lo4(const RepDev& rd) { return (rd.hi - (rd.lo & ~3) + HC_SEL_CHUNK - 1) / HC_SEL_CHUNK; }

// PASS 2: second digits (bits 20..10) of the keys whose first digit matches; PASS 3: third digits (bits 9..0) of those whose
// upper 22 bits match.  A workgroup handles every set size of its pivot over `span` chunks.
template <int PASS>
__global__ __launch_bounds__(BLK, 8) void mon_hist(MonBatch B, int span)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];      // [nk][HC_RADIX_BINS]
    __shared__ uint32_t sm_prefix[HC_MAX_K_PER_REP];
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    const RepDev rd = it.reps[rep];
    const int lo4 = rd.lo & ~3, nchunk = chunks_from_lo4(rd);
    const int c0 = blockIdx.x * span, c1 = min(c0 + span, nchunk);
    if (c0 >= nchunk) return;
    const Ws w = it.ws.rep(rep);
    const uint32_t* before = PASS == 2 ? w.hist : w.h2;
    copy_words(dyn, before, (PASS == 2 ? 1 : rd.nk) * HC_RADIX_BINS);
    __syncthreads();
    for (int ks = threadIdx.x >> 6; ks < rd.nk; ks += NWAVE) {          // a wave per set size
        uint32_t digit, remaining, count;
        if (PASS == 2) {
            find_digit(dyn, (uint32_t)it.reps[rep].k[ks], digit, remaining, count);      // (indexing the register copy would spill it)
        } else {
            find_digit(dyn + ks * HC_RADIX_BINS, w.sel[ks * 4 + 1], digit, remaining, count);
            digit |= w.sel[ks * 4] << 11;
        }
        if ((threadIdx.x & 63) == 0) {
            sm_prefix[ks] = digit;
            if (blockIdx.x == 0) {       // for the next pass (every workgroup finds the same)
                w.sel[ks * 4 + (PASS == 2 ? 0 : 2)] = digit;
                w.sel[ks * 4 + (PASS == 2 ? 1 : 3)] = remaining;
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < rd.nk * HC_RADIX_BINS; i += BLK) dyn[i] = 0u;
    __syncthreads();
    const float* srow = it.scores + (size_t)rep * it.ws.max_ctx;
    for (int ch = c0; ch < c1; ch += 2) {            // two chunks' loads in flight
        uint32_t key[2][4];
        bool in[2][4];
        load_keys(srow, lo4 + ch * HC_SEL_CHUNK + threadIdx.x * 4, rd.lo, rd.hi, key[0], in[0]);
        load_keys(srow, lo4 + (ch + 1) * HC_SEL_CHUNK + threadIdx.x * 4, rd.lo, ch + 1 < c1 ? rd.hi : 0, key[1], in[1]);
        for (int ks = 0; ks < rd.nk; ++ks) {
            const uint32_t prefix = sm_prefix[ks];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (!in[u][i]) continue;
                    if (PASS == 2) {
                        if ((key[u][i] >> 21) == prefix) atomicAdd(&dyn[ks * HC_RADIX_BINS + ((key[u][i] >> 10) & 0x7ffu)], 1u);
                    } else {
                        if ((key[u][i] >> 10) == prefix) atomicAdd(&dyn[ks * HC_RADIX_BINS + (key[u][i] & 0x3ffu)], 1u);
                    }
                }
            }
        }
    }
    __syncthreads();
    uint32_t* out = PASS == 2 ? w.h2 : w.h3;
    for (int i = threadIdx.x; i < rd.nk * HC_RADIX_BINS; i += BLK)
        if (dyn[i]) atomicAdd(&out[i], dyn[i]);
}

// The threshold key of every set size, then per chunk the counts of greater and of equal keys: a wave takes a chunk, every
// fourth of the workgroup's span.  The check of a filtering layer (see mon_select) is made here.
__global__ __launch_bounds__(BLK) void mon_count(MonBatch B, int span, int n_group)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];      // [nk][HC_RADIX_BINS]
    __shared__ uint32_t sm_tau[HC_MAX_K_PER_REP];
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    const RepDev rd = it.reps[rep];
    const int lo4 = rd.lo & ~3, nchunk = chunks_from_lo4(rd);
    const int c0 = blockIdx.x * span, c1 = min(c0 + span, nchunk);
    if (c0 >= nchunk) return;
    const Ws w = it.ws.rep(rep);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    copy_words(dyn, w.h3, rd.nk * HC_RADIX_BINS);
    __syncthreads();
    for (int ks = wv; ks < rd.nk; ks += NWAVE) {
        uint32_t digit, need, count;
        find_digit(dyn + ks * HC_RADIX_BINS, w.sel[ks * 4 + 3], digit, need, count);
        const uint32_t tau = (w.sel[ks * 4 + 2] << 10) | digit;
        if (lane == 0) {
            sm_tau[ks] = tau;
            if (blockIdx.x == 0) {       // for mon_write (the other two words are still being read)
                w.sel[ks * 4] = tau;
                w.sel[ks * 4 + 1] = need;
            }
        }
    }
    __syncthreads();
    if (it.need_sense == 0 && it.filt && blockIdx.x == 0 && threadIdx.x == 0) {
        const RepFilter* f = it.filt + rep;
        if (f->cutsum > 0.f) {
            uint32_t tmin = sm_tau[0];
            for (int ks = 1; ks < rd.nk; ++ks) tmin = min(tmin, sm_tau[ks]);
            float delta = 0.f;
            for (int g = 0; g < n_group; ++g) delta = fmaxf(delta, exp2f(f->ref[g] - it.lse[(size_t)rd.bh * n_group + g] * 1.4426950408889634f));
            const float bound = f->cutsum / (float)n_group * delta * 1.0001f;
            if (!(key_score(tmin) >= bound)) it.need[rep] = 5;
        }
    }
    const float* srow = it.scores + (size_t)rep * it.ws.max_ctx;
    for (int ch = c0 + wv; ch < c1; ch += NWAVE) {
        uint32_t key[4][4];
        bool in[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) load_keys(srow, lo4 + ch * HC_SEL_CHUNK + q * 256 + lane * 4, rd.lo, rd.hi, key[q], in[q]);
        for (int ks = 0; ks < rd.nk; ++ks) {
            const uint32_t tau = sm_tau[ks];
            uint32_t gt = 0, eq = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gt += count_true(in[q][i] && key[q][i] > tau);
                    eq += count_true(in[q][i] && key[q][i] == tau);
                }
            }
            if (lane == 0) {
                uint32_t* cnt = w.cnt + ((size_t)ks * w.max_chunks + ch) * 2;
                cnt[0] = gt;
                cnt[1] = eq;
            }
        }
    }
}

// The lists of a pivot in ascending order, and |T ∩ baseline| of the monitored one.  A wave takes a chunk, in two halves
// of 512 candidates in position order (8 to a lane), and reads a half's keys once for all set sizes; what a set size
// carries from half to half (equal keys seen, entries emitted) lives in LDS: the kernel has to fit, in registers, beside
// the attention pass.
__global__ __launch_bounds__(BLK, 8) void mon_write(MonBatch B, DriftCfg cfg, int span)
{
    __shared__ uint32_t sm_carry[NWAVE][HC_MAX_K_PER_REP][2];
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps || mon_skip(it, rep)) return;
    const int max_ctx = it.ws.max_ctx;
    const int32_t* __restrict__ pmap = it.pos_map ? it.pos_map + (size_t)rep * max_ctx : nullptr;
    const RepDev rd = it.reps[rep];
    const int real_lo = it.real_reps[rep].lo, real_hi = it.real_reps[rep].hi;
    const int lo4 = rd.lo & ~3, nchunk = chunks_from_lo4(rd);
    const int c0 = blockIdx.x * span, c1 = min(c0 + span, nchunk);
    if (c0 >= nchunk) return;
    const Ws w = it.ws.rep(rep);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const float* srow = it.scores + (size_t)rep * max_ctx;
    for (int chunk = c0 + wv; chunk < c1; chunk += NWAVE) {
        for (int ks = 0; ks < rd.nk; ++ks) {
            const uint32_t need = w.sel[ks * 4 + 1];
            const uint32_t* cnt = w.cnt + (size_t)ks * w.max_chunks * 2;
            // over the chunks before this one: equal keys seen, and entries emitted (a chunk's greater keys plus as many
            // equal ones as are still needed)
            uint32_t eq_before = 0, emitted = 0;
            for (int b0 = 0; b0 < chunk; b0 += 64) {
                const int b = b0 + lane;
                const uint32_t g = b < chunk ? cnt[b * 2] : 0u, e = b < chunk ? cnt[b * 2 + 1] : 0u;
                uint32_t etot;
                const uint32_t eprev = eq_before + wave_exscan(e, etot);
                const uint32_t left = need > eprev ? need - eprev : 0u;
                emitted += wave_sum(g + min(e, left));
                eq_before += etot;
            }
            if (lane == 0) {
                sm_carry[wv][ks][0] = eq_before;
                sm_carry[wv][ks][1] = emitted;
            }
        }
        uint32_t hits = 0;
        for (int half = 0; half < 2; ++half) {
            uint32_t key[2][4];
            bool in[2][4];
            const int first8 = lo4 + chunk * HC_SEL_CHUNK + half * (HC_SEL_CHUNK / 2) + lane * 8;
            load_keys(srow, first8, rd.lo, rd.hi, key[0], in[0]);
            load_keys(srow, first8 + 4, rd.lo, rd.hi, key[1], in[1]);
            // the positions of the lane's 8 rows: themselves, or (rows a filtering split pass kept) what the map says
            int32_t jj[8];
            if (pmap) {
                int4 pa = make_int4(0, 0, 0, 0), pb = pa;
                if (first8 < rd.hi) pa = *reinterpret_cast<const int4*>(pmap + first8);          // (row stride a multiple of 64: in bounds)
                if (first8 + 4 < rd.hi) pb = *reinterpret_cast<const int4*>(pmap + first8 + 4);
                jj[0] = pa.x; jj[1] = pa.y; jj[2] = pa.z; jj[3] = pa.w;
                jj[4] = pb.x; jj[5] = pb.y; jj[6] = pb.z; jj[7] = pb.w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) jj[i] = first8 + i;
            }
            for (int ks = 0; ks < rd.nk; ++ks) {
                const uint32_t tau = w.sel[ks * 4], need = w.sel[ks * 4 + 1], k = (uint32_t)it.reps[rep].k[ks];
                const uint32_t eq_before = sm_carry[wv][ks][0], emitted = sm_carry[wv][ks][1];      // (written by this wave)
                uint32_t my_eq = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) my_eq += in[i / 4][i % 4] && key[i / 4][i % 4] == tau;
                uint32_t eq_tot, sel_tot, selmask = 0;
                uint32_t eq_rank = eq_before + wave_exscan(my_eq, eq_tot);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool at = in[i / 4][i % 4] && key[i / 4][i % 4] == tau;
                    const bool sel = at ? eq_rank < need : in[i / 4][i % 4] && key[i / 4][i % 4] > tau;
                    eq_rank += at;
                    selmask |= (uint32_t)sel << i;
                }
                const uint32_t pos0 = emitted + wave_exscan((uint32_t)__builtin_popcount(selmask), sel_tot);
                if (lane == 0) {
                    sm_carry[wv][ks][0] = eq_before + eq_tot;
                    sm_carry[wv][ks][1] = emitted + sel_tot;
                }
                if (ks == 0) {
                    // (all loads issued together; a row that is not selected reads word 0 and does not count)
                    uint32_t wd[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int j = (selmask >> i) & 1u ? min(max(jj[i], real_lo), real_hi - 1) - real_lo : 0;
                        wd[i] = (w.bitmap[j >> 5] >> (j & 31)) & (selmask >> i) & 1u;
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) hits += wd[i];
                }
                for (int o = rd.out_begin; o < rd.out_begin + rd.out_count; ++o) {      // the rows this list goes to
                    if (it.outs[o].kslot != ks) continue;
                    int32_t* dst = it.topk_idx + (size_t)it.outs[o].row * cfg.max_k;
                    uint32_t pos = pos0;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (selmask & (1u << i)) {
                            if (pos < k) dst[pos] = jj[i];      // (always; the guard keeps a corrupt state in bounds)
                            ++pos;
                        }
                    }
                }
            }
        }
        hits = wave_sum(hits);
        if (lane == 0) w.hits[chunk] = hits;
    }
}

// A workgroup per pivot, behind mon_write.
__global__ __launch_bounds__(BLK) void mon_decide(MonBatch B, DriftCfg cfg, int n_group)
{
    __shared__ uint32_t sm_hits[NWAVE];
    const MonItem& it = B.it[blockIdx.y];
    const int rep = blockIdx.x, tid = threadIdx.x;
    if (rep >= it.n_reps) return;
    if (it.need_sense == 1 && it.need[rep] == 0) return;         // decided over the kept rows
    const bool elsewhere = it.need_sense == 0 && it.need[rep] != 0;
    const RepDev rd = it.reps[rep];
    const Ws w = it.ws.rep(rep);
    RingRow ring{0, 0};
    if (it.store_slot != -2) ring = ring_row(it, rd.bh, cfg.window);
    const float lse_of = it.filt && (tid & 63) < n_group ? it.lse[(size_t)rd.bh * n_group + (tid & 63)] : 0.f;
    uint32_t h = 0;
    if (!elsewhere)
        for (int c = tid; c < chunks_from_lo4(rd); c += BLK) h += w.hits[c];
    h = wave_sum(h);
    if ((tid & 63) == 0) sm_hits[tid >> 6] = h;
    __syncthreads();
    // every other kernel of this call is done with histogram and bitmap: the next call finds them clear
    const int words = (it.real_reps[rep].hi - it.real_reps[rep].lo + 31) / 32;
    for (int i = tid; i < HC_RADIX_BINS; i += BLK) w.hist[i] = 0u;
    for (int i = tid; i < words; i += BLK) w.bitmap[i] = 0u;
    if (elsewhere) return;
    uint32_t tmin = 0xffffffffu;
    if (it.filt)
        for (int ks = 0; ks < rd.nk; ++ks) tmin = min(tmin, w.sel[ks * 4]);
    decide<BLK>(it, rep, rd.bh, rd.hi, rd.k[0], cfg, n_group, ring, (int32_t)(sm_hits[0] + sm_hits[1] + sm_hits[2] + sm_hits[3]), tmin, lse_of);
}

// Scores of the rows a filtering split pass kept.  They lie segment by segment in the pivot's block of rep_logits
// (positions in surv_pos, counts in seg_cnt); here they are scored with this step's log-sum-exp and laid out as one
// dense run in position order (scores[rep][0, n), pos_map[rep][0, n)), over which mon_select then works as over a
// short context.  Every workgroup makes the prefix sums of the pivot's segment counts itself (a few hundred numbers);
// then a wave takes a segment, whose rows are contiguous on both sides.
constexpr int MAX_FILTER_SEGS = 2048;
template <int G>
__global__ __launch_bounds__(BLK, 8) void mon_sparse_score(MonBatch B)
{
    __shared__ int sm_pref[MAX_FILTER_SEGS + 1];
    __shared__ int sm_row0[MAX_FILTER_SEGS];
    __shared__ int sm_wsum[NWAVE];
    __shared__ int sm_unknown;
    const MonItem& it = B.it[blockIdx.z];
    const int rep = blockIdx.y;
    if (rep >= it.n_reps) return;
    const int max_ctx = it.ws.max_ctx;
    const RepDev rd = it.real_reps[rep];
    const int part_begin = it.heads[rd.bh].part_begin, part_count = it.heads[rd.bh].part_count;
    const int nseg = min(part_count, MAX_FILTER_SEGS);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float l[G];
#pragma unroll
    for (int g = 0; g < G; ++g) l[g] = it.lse[(size_t)rd.bh * G + g];
    if (threadIdx.x == 0) sm_unknown = 0;
    __syncthreads();
    int carry = 0;
    for (int base = 0; base < nseg; base += BLK) {
        const int sidx = base + threadIdx.x;
        int c = 0;
        if (sidx < nseg) {
            const int row0 = it.segs[part_begin + sidx].row_begin, row1 = it.segs[part_begin + sidx].row_end;
            c = it.seg_cnt[part_begin + sidx];
            if (c < 0 || c > row1 - row0) {                    // not a count the split pass can have written
                sm_unknown = 1;
                c = 0;
            }
            sm_row0[sidx] = row0;
        }
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        if (lane == 63) sm_wsum[wv] = inc;
        __syncthreads();
        int before = carry;
        for (int k = 0; k < wv; ++k) before += sm_wsum[k];
        if (sidx < nseg) sm_pref[sidx] = before + inc - c;
        carry += sm_wsum[0] + sm_wsum[1] + sm_wsum[2] + sm_wsum[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) sm_pref[nseg] = carry;
    __syncthreads();
    const int n = carry;                                    // rows kept, all of them candidates
    int kmax = 0;
    for (int ks = 0; ks < rd.nk; ++ks) kmax = max(kmax, it.real_reps[rep].k[ks]);       // (indexing the register copy would spill it)
    // why a pivot goes to the dense chain: 1 more rows kept than the launch was sized for, 2 fewer than the longest
    // list needs, 3 a segment's count is out of range, 4 too many segments, (5: the check of mon_select failed)
    const int why = sm_unknown != 0 ? 3 : part_count > MAX_FILTER_SEGS ? 4 : n > it.cap_rows ? 1 : n < kmax ? 2 : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the pivot as mon_select sees it: a context of n rows, all of them candidates
        RepDev* v = it.vreps + rep;
        v->bh = rd.bh;
        v->lo = 0;
        v->hi = why ? 0 : n;
        v->nk = rd.nk;
        for (int ks = 0; ks < rd.nk; ++ks) v->k[ks] = it.real_reps[rep].k[ks];
        v->nchunk = why ? 0 : (n + HC_SEL_CHUNK - 1) / HC_SEL_CHUNK;
        v->out_begin = rd.out_begin;
        v->out_count = rd.out_count;
        it.need[rep] = why;
    }
    if (why) return;
    const float* lrow = it.rep_logits + (size_t)rep * G * max_ctx;
    const int32_t* prow = it.surv_pos + (size_t)rep * max_ctx;
    float* srow = it.scores + (size_t)rep * max_ctx;
    int32_t* drow = it.pos_map + (size_t)rep * max_ctx;
    for (int s = blockIdx.x * NWAVE + wv; s < nseg; s += gridDim.x * NWAVE) {
        const int row0 = sm_row0[s], d0 = sm_pref[s], cnt = sm_pref[s + 1] - d0;
        for (int i = lane; i < cnt; i += 64) {
            const float sc = score_of<G>(lrow, row0 + i, l, HC_AGG_PROB);
            const int32_t p = prow[row0 + i];
            srow[d0 + i] = sc;
            drow[d0 + i] = p;
        }
    }
}

}   // namespace

// mon_select's two forms.  Beside the attention pass the small one (512 threads of at most 40 registers) leaves room for two
// attention workgroups on its compute unit: 26 KB of LDS each with the pivot-logit filter, 41 KB without.  The large one
// (1024 threads) may take a whole compute unit, also beside the attention pass where the small one has no room for the
// items, and in groups of eight heads, two of whose attention workgroups leave no room for either.
constexpr int SELECT_STATIC = 10 * 1024;            // (what the kernel itself declares, rounded up)
template <int NT> static int select_room(const hc_ctx* ctx)
{
    return (NT == 1024 ? 152 * 1024 : ctx->side_pad_now ? 110 * 1024 : 76 * 1024) - SELECT_STATIC;
}
static bool select_small(const hc_ctx* ctx, int items)
{
    return ctx->beside_now && ctx->G < 8 && items <= SEL_KEYS(select_room<512>(ctx) / 4);
}

// mon_direct: up to as many items as its waves have bits for, if tiles and bitmaps fit in LDS beside what it declares.
constexpr int DIRECT_STATIC = 14 * 1024;
// Its two forms.  Beside the attention pass the small one fits next to two attention workgroups on a compute unit, but goes through
// 32 K candidates only.  For up to 64 K of an unfiltered layer the large one, which fits next to one of them (as long as it keeps
// one buffer of tiles), beats the survivors' three launches while lists are few.  Steps of four layers in groups of two, us by three launches / this way: one
// sequence (12 lists) of 36,000 114 / 101, 48K 124 / 108, 60,000 118 / 110, in groups of eight heads 36,000 160 / 143, 50,000 125 / 110; three (18 lists, a layer to a
// group) 111 / 109; two (24 lists) 106-120 / 111-113; four (48 lists, whose workgroups attention's then wait for) 174 / 187.  (For up to 32 K the small form and
// the large one take the same.)
struct DirectForm {
    int threads, room;           // room: dynamic LDS of a workgroup, bytes
};
static DirectForm direct_form(const hc_ctx* ctx, int mode, int items, int lists)
{
    if (!ctx->beside_now) return {1024, 156 * 1024 - DIRECT_STATIC};
    if (mode == 0 && !ctx->side_pad_now && items + 3 > 512 / 64 * DIRECT_TILES * HC_SEL_CHUNK && lists <= 20) return {1024, (ctx->G == 8 ? 106 : 116) * 1024 - DIRECT_STATIC};
    return {512, (ctx->G == 8 ? 56 : ctx->side_pad_now ? 110 : 76) * 1024 - DIRECT_STATIC};
}
// Candidates a launch goes through.  A captured call is replayed over contexts that have grown since, so a launch takes whole tiles:
// one to a wave, or up to the end of the last chunk that mon_score_hist takes (items are counted from a multiple of four
// positions, so that the last three may not fit).
static int direct_most(const DirectForm& f, int src, int items)
{
    const int tile_each = f.threads / 64 * HC_SEL_CHUNK;
    if (src == DIRECT_LOGITS) return tile_each;
    if (src == DIRECT_SCORES) return tile_each - 3;
    return std::min((items + HC_SEL_CHUNK - 1) / HC_SEL_CHUNK * HC_SEL_CHUNK, DIRECT_TILES * tile_each - 3);
}
static int direct_bytes(const DirectForm& f, int most, int bm_words, int bufs)
{
    const int tiles = (most + 3 + HC_SEL_CHUNK - 1) / HC_SEL_CHUNK;
    return 4 * (bufs * f.threads / 64 * HC_SEL_CHUNK + tiles * (HC_SEL_CHUNK / 32) + bm_words + 2);
}
static bool direct_fits(const DirectForm& f, int items, int bm_words)
{
    return items + 3 <= f.threads / 64 * DIRECT_TILES * HC_SEL_CHUNK && direct_bytes(f, direct_most(f, DIRECT_HIST, items), bm_words, 1) <= f.room;
}
// Lists that mon_direct writes in several pieces, going through its bits for each (a piece has 16,384 entries there, alone): whether
// the six launches of long lists take less.  One list, us by them / by mon_direct, scores spread out and within 2 % of each other: 32,000 of
// 40,000 candidates 54 54 / 45 51, 36,000 61 62 / 61 67; of 50,000 26,000 entries 46 45 / 45 46, 32,000 49 50 / 44 51, 36,000 51 51 / 54 61;
// of 58,000 16,000 40 41 / 31 38, 20,000 42 42 / 38 46, 26,000 43 43 / 49 51; of 65,480 16,000 40 40 / 31 39, 20,000 41 42 / 45 45, 60,000 62 63 /
// 98 106.  Each further list adds 5 us to the six and nothing to mon_direct: lists of 20,000, 10,000 and 5,000 of 65,480 54 54 / 44 45, of
// 36,000, 20,000 and 9,000 60 60 / 55 64, of 50,000 63 64 / 54 61.  (Beside the
// attention pass its ranges are shorter: steps of four layers of 31,000 with lists of 22,000 and 8,000 194 us by the six, 146.)
static bool direct_outlasted(const hc_ctx* ctx, int items, int max_k, int max_nk)
{
    return !ctx->beside_now && max_k > 16384 && !(max_nk >= 3 ? max_k <= 40960 : max_k <= 32768 && items <= 51200);
}
template <int SRC>
static hc_status launch_direct(hc_ctx* ctx, const DirectForm& f, const MonBatch& B, const DriftCfg& dc, const dim3& grid, int lists, int items, int bm_words, hipStream_t st)
{
    const int most = direct_most(f, SRC, items);
    bm_words = SRC == DIRECT_MAP ? bm_words + 1 : std::max(bm_words, (most + 3 + 31) / 32);      // (positions are counted from a multiple of four; a candidate's number is its bit)
    const int bufs = SRC < DIRECT_SCORES && items + 3 > f.threads / 64 * HC_SEL_CHUNK && direct_bytes(f, most, bm_words, 2) <= f.room ? 2 : 1;
    const unsigned lds = (unsigned)direct_bytes(f, most, bm_words, bufs);
#define HC_DIRECT_AS(NT, GG, COPY)                                                                                           \
    mon_direct<NT, SRC, GG, COPY><<<grid, dim3(NT), hc_side_lds(ctx, (const void*)mon_direct<NT, SRC, GG, COPY>, lds), st>>>(B, dc, ctx->G, bufs, most, bm_words, lists)
#define HC_DIRECT(NT, GG) HC_DIRECT_AS(NT, GG, false)
    const bool small = f.threads == 512;
    if constexpr (SRC == DIRECT_HIST)
        if ((int)grid.y > lists) {
            if (small) HC_DIRECT_AS(512, 1, true);
            else HC_DIRECT_AS(1024, 1, true);
            HC_HIP(ctx, hipGetLastError());
            return HC_OK;
        }
    if constexpr (SRC != DIRECT_LOGITS) {
        if (small) HC_DIRECT(512, 1);                                // (the group size only matters where logits are read)
        else HC_DIRECT(1024, 1);
    } else {
        switch (ctx->G * 2 + small) {
        case 2: HC_DIRECT(1024, 1); break;
        case 3: HC_DIRECT(512, 1); break;
        case 4: HC_DIRECT(1024, 2); break;
        case 5: HC_DIRECT(512, 2); break;
        case 8: HC_DIRECT(1024, 4); break;
        case 9: HC_DIRECT(512, 4); break;
        case 16: HC_DIRECT(1024, 8); break;
        default: HC_DIRECT(512, 8); break;
        }
    }
#undef HC_DIRECT
#undef HC_DIRECT_AS
    HC_HIP(ctx, hipGetLastError());
    return HC_OK;
}

// Launches mon_select over the batch, with LDS for want_keys items and a baseline bitmap of bm_words as far as it goes.
template <int NT, int SRC, bool COPY>
static hc_status launch_select_nt(hc_ctx* ctx, const MonBatch& B, const DriftCfg& dc, const dim3& grid, int lists, int want_keys, int bm_words, hipStream_t st)
{
    const unsigned lds = (unsigned)std::min((long long)select_room<NT>(ctx), ((long long)want_keys + 255) / 256 * 264 * 4 + bm_words * 4);
    mon_select<NT, SRC, COPY><<<grid, dim3(NT), hc_side_lds(ctx, (const void*)mon_select<NT, SRC, COPY>, lds), st>>>(B, dc, ctx->G, (int)(lds / 4), lists);
    HC_HIP(ctx, hipGetLastError());
    return HC_OK;
}

template <int SRC>
static hc_status launch_select(hc_ctx* ctx, const MonBatch& B, const DriftCfg& dc, const dim3& grid, int lists, int want_keys, int bm_words, bool small,
                               hipStream_t st)
{
    if constexpr (SRC == SRC_SURVIVORS)
        if ((int)grid.y > lists)
            return small ? launch_select_nt<512, SRC, true>(ctx, B, dc, grid, lists, want_keys, bm_words, st)
                         : launch_select_nt<1024, SRC, true>(ctx, B, dc, grid, lists, want_keys, bm_words, st);
    return small ? launch_select_nt<512, SRC, false>(ctx, B, dc, grid, lists, want_keys, bm_words, st)
                 : launch_select_nt<1024, SRC, false>(ctx, B, dc, grid, lists, want_keys, bm_words, st);
}

// Items that the sample lets through for a longest list of k out of n candidates: expected, and with room for its spread.
static void expected_survivors(long long k, long long n, int* mean, int* most)
{
    const double t = (double)k * HC_SAMPLES / (double)n, place = std::min((double)HC_SAMPLES, t + 5.0 * std::sqrt(t) + 8.0);
    *mean = (int)(place * (double)n / HC_SAMPLES);
    *most = (int)std::min((double)n, (place + 4.0 * std::sqrt(place)) * (double)n / HC_SAMPLES);
}

// The launches of long lists: see mon_hist.
static hc_status launch_long(hc_ctx* ctx, const MonBatch& B, const DriftCfg& dc, int n, int max_reps, int max_nk, int max_nchunk, int span, hipStream_t st)
{
    const dim3 grid((max_nchunk + 1 + span - 1) / span, max_reps, n);      // (chunks that start at a multiple of 4 can be one more)
    const unsigned lds = (unsigned)max_nk * HC_RADIX_BINS * 4;
    mon_hist<2><<<grid, dim3(BLK), hc_side_lds(ctx, (const void*)mon_hist<2>, lds), st>>>(B, span);
    HC_HIP(ctx, hipGetLastError());
    mon_hist<3><<<grid, dim3(BLK), hc_side_lds(ctx, (const void*)mon_hist<3>, lds), st>>>(B, span);
    HC_HIP(ctx, hipGetLastError());
    mon_count<<<grid, dim3(BLK), hc_side_lds(ctx, (const void*)mon_count, lds), st>>>(B, span, ctx->G);
    HC_HIP(ctx, hipGetLastError());
    // (the write pass has nothing to set up per workgroup: a chunk per wave)
    mon_write<<<dim3((max_nchunk + 1 + NWAVE - 1) / NWAVE, max_reps, n), dim3(BLK), hc_side_lds(ctx, (const void*)mon_write, 0), st>>>(B, dc, NWAVE);
    HC_HIP(ctx, hipGetLastError());
    mon_decide<<<dim3(max_reps, n), dim3(BLK), hc_side_lds(ctx, (const void*)mon_decide, 0), st>>>(B, dc, ctx->G);
    HC_HIP(ctx, hipGetLastError());
    return HC_OK;
}

// Candidates up to which one workgroup per pivot does everything, from the scores on.  What lies against more is that
// the exponentials of the scores are then made by one compute unit: at 32K candidates and a group of four this takes 18
// of 44 us, where two launches take 21 in all.  One launch and two, us: 12.2 and 14.5 at 4K, at 8K 15.3 and 15.3 with scores spread
// out, 15.2 and 21 within 2 % of each other.
constexpr int SELECT_DIRECT = 8192;
// Survivors (as the sample would let through) up to which one workgroup per list beats the six launches of long lists, with
// the sample in front of it where it is needed.  131,072 candidates, scores spread out / within 2 % / equal: a longest list of 8,192
// (11,000 expected) 37 / 48 / 58 us against 47 / 49 / 62; of 10,000 (13,100) 41 / 50 / 63 against 47 / 49 / 62.
// The prefill-time selection has one list per head and smoothed scores, so that it always needs the sample: at 131,072 positions
// and lists of 7,872 its line is lower (a whole hc_prefill_init without the offload 239 us with survivors, 224 with the six
// launches; at 32K, lists of 3,776, 129 and 141).
constexpr int SELECT_SURVIVORS = 13000, SELECT_SURVIVORS_PREFILL = 8000;

// How a chain selects from its candidates: one place for it, because the combine pass makes a histogram for a selection that follows a
// group later.
struct Choice {
    DirectForm form;
    bool direct;                 // mon_direct, from a histogram by its own digits
    bool long_lists;             // the six launches
    int survivors, most;         // of the sample: expected, and with room for its spread
    int hist;                    // what the histogram is over
};
// lists: workgroups that select; few: kept rows that fit in mon_select's LDS.
//
// mon_direct where it has room and the lists are not too long for it.  (candidates: of a filtering layer, what its launches are
// sized for.)  Beside the attention pass, where a read takes many times as long, not for the kept rows of short lists: few waves
// then have a tile, and the rows' positions are one read more behind the selection.  Steps of four layers, contexts of 66,000 to 123,000, a
// drift at every step, us by mon_select / mon_direct: longest list 1,728, three and six sequences 277 278 / 424 425; 3,776 297 314 /
// 459 480; 5,824 343 345 / 536 536; 7,872 478 467 / 596 594 (the kernel itself, 3,776, six sequences: 59 and 97).
static Choice choose(const hc_ctx* ctx, int mode, bool armed, bool few, bool prefill, int candidates, int lists, int nchunk, int max_k, int max_nk)
{
    Choice c;
    c.form = direct_form(ctx, mode, candidates, lists);
    c.direct = (mode == 0 ? candidates > SELECT_DIRECT : mode == 1 && armed) && direct_fits(c.form, candidates, nchunk * (HC_SEL_CHUNK / 32)) &&
               !(mode == 0 && direct_outlasted(ctx, candidates, max_k, max_nk)) && !(ctx->beside_now && few && max_k <= 4096);
    expected_survivors(max_k, candidates, &c.survivors, &c.most);
    c.long_lists = !c.direct && (c.survivors > (prefill ? SELECT_SURVIVORS_PREFILL : SELECT_SURVIVORS) || c.most > ctx->sv_cap);
    c.hist = !c.direct ? HIST_KEYS : ctx->cfg.agg == HC_AGG_LOGIT ? HIST_LINEAR : HIST_FINE;
    return c;
}

// The launches of one chain over a batch of layers.  mode 0: the plain chain (every pivot, all candidate positions).
// mode 1: the chain over the rows a filtering split pass kept.  mode 2: the chain that stands by behind
// mode 1, for the pivots whose check failed (their logits and scores are there already: see
// hc_launch_rep_logits).  ws_first: which workspace copy the first layer uses.
static hc_status run_chain(hc_ctx* ctx, int n, const hc_monitor_call* const* calls, int ws_first, int scores_given, int mode,
                           hipStream_t st)
{
    const hc_config& c = ctx->cfg;
    MonBatch B{};
    int max_reps = 0, max_nk = 1, max_nchunk = 0, max_real_chunk = 0, max_k = 1, candidates = 0, copiers = 0;
    bool armed = true;
    for (int i = 0; i < n; ++i) {
        const hc_monitor_call& x = *calls[i];
        hc_monitor_ws& m = ctx->ws[ws_first + i];
        MonItem& it = B.it[i];
        it.ws = Ws{m.hist, m.bitmap, nullptr, nullptr, m.area, nullptr, nullptr, nullptr, nullptr, ctx->max_chunks, c.max_ctx, ctx->sv_cap, ctx->area_words};
        it.reps = x.reps ? x.reps : x.L->reps;
        it.real_reps = it.reps;
        it.outs = x.reps ? x.outs : x.L->outs;
        it.rep_logits = x.rep_logits;
        it.lse = x.lse;
        it.scores = x.scores;
        it.topk_idx = x.topk_idx;
        it.base_idx = x.base_idx;
        it.ring = x.ring;
        it.inter = x.inter;
        it.flag = x.flag;
        it.n_reps = x.reps ? x.n_reps : x.L->n_reps;
        it.store_slot = x.store_slot;
        it.need_sense = -1;
        if (!x.reps && x.store_slot == -1) it.counts = x.L->mon_counts;
        int nchunk = x.reps ? x.max_nchunk : x.L->max_nchunk, cand = x.reps ? x.max_cand : x.L->max_cand;
        max_real_chunk = std::max(max_real_chunk, nchunk);
        if (mode != 0) {
            const hc_layer* L = x.L;
            it.need_sense = mode == 1 ? 0 : 1;
            it.need = L->need;
            it.filt = L->filt;
            it.counts = L->mon_counts;
            it.margin = ctx->filter_margin;
            if (mode == 1) {
                it.reps = L->vreps;
                it.pos_map = L->dense_pos;
                it.heads = L->heads;
                it.segs = L->segs;
                it.seg_cnt = L->seg_cnt;
                it.surv_pos = L->surv_pos;
                it.vreps = L->vreps;
                // Once the filter is set few rows are kept (about 1.6 times the longest list at the usual margin of
                // 1.25); a step that keeps more is handed to the dense chain.
                const int armed_cap = std::min(c.max_ctx, (ctx->filter_margin <= 1.5f ? 2 : 4) * L->max_k_any + 4096);
                it.cap_rows = L->filter_armed ? armed_cap : c.max_ctx;
                armed = armed && L->filter_armed;
                cand = std::min(cand, it.cap_rows);
                nchunk = std::min(nchunk, (it.cap_rows + HC_SEL_CHUNK - 1) / HC_SEL_CHUNK);
            }
        }
        max_reps = std::max(max_reps, it.n_reps);
        max_nchunk = std::max(max_nchunk, nchunk);
        candidates = std::max(candidates, cand);
        max_nk = std::max(max_nk, x.reps ? x.max_nk : x.L->max_nk);
        max_k = std::max(max_k, x.reps ? c.max_k : x.L->max_k_any);
        if (m.dirty && mode != 2) {     // a previous call that used this workspace copy did not run to its last kernel
            mon_prep<<<dim3(16, m.reps), dim3(256), 0, st>>>(it.ws);
            HC_HIP(ctx, hipGetLastError());
        }
        m.dirty = true;
        if (x.scored.hist >= 0) {
            it.ws.hist = x.L->score_hist;                // (not what is cleared above)
            it.copy_to = x.copy_to;
            if (x.copy_to) copiers = (max_real_chunk + 31) / 32;       // (a workgroup of its own to 32 K scores)
        }
    }
    if (max_reps == 0) return HC_OK;
    const DriftCfg dc{c.window, c.metric, c.tau_num, c.tau_den, c.max_k, c.window_mode != HC_WINDOW_SLIDING, c.agg};
    const dim3 gsel(max_reps, max_nk + copiers, n);
    const int bm_words = max_real_chunk * (HC_SEL_CHUNK / 32);
    const int pivots = max_reps * n;
    const bool scored = mode == 0 && calls[0]->scored.hist >= 0;       // (by all of the batch, or none)
    // One launch for what one workgroup per pivot handles by itself: short ranges, and the rows that a set filter keeps (at a
    // margin of 1.25 about 1.6 times the longest list) as far as their keys fit in LDS.
    const int kept = (ctx->filter_margin <= 1.5f ? 7 : 14) * ((max_k + 3) / 4);
    const bool few = mode == 1 && armed && (select_small(ctx, kept) || (!(ctx->beside_now && ctx->G < 8) && kept <= SEL_KEYS(select_room<1024>(ctx) / 4)));
    const Choice how = choose(ctx, mode, armed, few, calls[0]->store_slot == -2, candidates, pivots * max_nk, max_real_chunk, max_k, max_nk);
    const DirectForm& form = how.form;
    const bool direct = how.direct, long_lists = how.long_lists;
    const int survivors = how.survivors, most = how.most;
    for (int i = 0; i < n; ++i) {                        // a histogram is read as what it was made as
        const hc_score_plan& made = calls[i]->scored;
        if (scored ? made.hist != how.hist || long_lists || (direct && made.most != direct_most(form, DIRECT_HIST, candidates)) : made.hist >= 0)
            return hc_fail(ctx, HC_ESTATE, "internal: scores and histogram for another selection");
    }
    if (mode == 1) {
        if (direct)                                      // (more rows than it goes through, in a captured call: the dense chain's)
            for (int i = 0; i < n; ++i) B.it[i].cap_rows = std::min(B.it[i].cap_rows, direct_most(form, DIRECT_MAP, candidates));
        // enough waves for a segment each of a long context's few hundred, no more workgroups than compute units
        const dim3 g(std::max(4, std::min(armed ? 32 : 128, (armed ? 256 : 1024) / pivots)), max_reps, n);
        switch (ctx->G) {
        case 1: mon_sparse_score<1><<<g, dim3(BLK), hc_side_lds(ctx, (const void*)mon_sparse_score<1>, 0), st>>>(B); break;
        case 2: mon_sparse_score<2><<<g, dim3(BLK), hc_side_lds(ctx, (const void*)mon_sparse_score<2>, 0), st>>>(B); break;
        case 4: mon_sparse_score<4><<<g, dim3(BLK), hc_side_lds(ctx, (const void*)mon_sparse_score<4>, 0), st>>>(B); break;
        default: mon_sparse_score<8><<<g, dim3(BLK), hc_side_lds(ctx, (const void*)mon_sparse_score<8>, 0), st>>>(B); break;
        }
        HC_HIP(ctx, hipGetLastError());
    }
    if (scored && direct) return launch_direct<DIRECT_HIST>(ctx, form, B, dc, gsel, max_nk, candidates, bm_words, st);
    if (mode != 0) scores_given = 1;                     // they are there from here on
    if (mode == 1 && direct) return launch_direct<DIRECT_MAP>(ctx, form, B, dc, gsel, max_nk, candidates, bm_words, st);
    // (a tile to a wave; given scores are read from a multiple of four positions on)
    if (mode == 0 && candidates <= SELECT_DIRECT && (!scores_given || candidates + 3 <= form.threads / 64 * HC_SEL_CHUNK))
        return scores_given ? launch_direct<DIRECT_SCORES>(ctx, form, B, dc, gsel, max_nk, candidates, bm_words, st)
                            : launch_direct<DIRECT_LOGITS>(ctx, form, B, dc, gsel, max_nk, candidates, bm_words, st);
    if (few || candidates <= SELECT_DIRECT) {
        const bool small = few ? select_small(ctx, kept) : select_small(ctx, candidates);
        return launch_select<SRC_SCORES>(ctx, B, dc, gsel, max_nk, candidates, bm_words, small, st);
    }
    if (!scored && (mode != 2 || long_lists)) {
        // Chunks per workgroup, at most 8: about 2048 workgroups per launch (a call over eight sequences of 9K to 131K takes
        // 36 us with one chunk each, 37, 41, 50 with two, four, eight; one of 32K 28, 29, 32, 39), beside the attention pass
        // 512.  (The launches that stand by: few, long workgroups.)
        const int span = mode == 2 ? 32 : ctx->monitor_span > 0 ? ctx->monitor_span : std::max(1, std::min(8, (pivots * max_nchunk) / (ctx->beside_now ? 512 : 2048)));
        const dim3 g1((max_nchunk + span - 1) / span, max_reps, n);
#define HC_SCORE(GG, HIST)                                                                                                   \
    mon_score_hist<GG, HIST><<<g1, dim3(BLK), hc_side_lds(ctx, (const void*)mon_score_hist<GG, HIST>, 0), st>>>(B, scores_given, c.agg, span, long_lists, c.max_k, direct_most(form, DIRECT_HIST, candidates))
        switch (ctx->G * 4 + how.hist) {
        case 4: HC_SCORE(1, HIST_KEYS); break;
        case 5: HC_SCORE(1, HIST_FINE); break;
        case 6: HC_SCORE(1, HIST_LINEAR); break;
        case 8: HC_SCORE(2, HIST_KEYS); break;
        case 9: HC_SCORE(2, HIST_FINE); break;
        case 10: HC_SCORE(2, HIST_LINEAR); break;
        case 16: HC_SCORE(4, HIST_KEYS); break;
        case 17: HC_SCORE(4, HIST_FINE); break;
        case 18: HC_SCORE(4, HIST_LINEAR); break;
        case 32: HC_SCORE(8, HIST_KEYS); break;
        case 33: HC_SCORE(8, HIST_FINE); break;
        default: HC_SCORE(8, HIST_LINEAR); break;
        }
#undef HC_SCORE
        HC_HIP(ctx, hipGetLastError());
        if (direct) return launch_direct<DIRECT_HIST>(ctx, form, B, dc, gsel, max_nk, candidates, bm_words, st);
        if (long_lists) return launch_long(ctx, B, dc, n, max_reps, max_nk, max_nchunk, span, st);
    }
    // The small form where all that may survive fits, and what is expected fits with the baseline bitmap (without the bitmap in LDS
    // the lists are written a round at a time: 229,376 candidates, no filter, 53.2 us per layer-step with it, 51.9 with the large one).
    const bool small = select_small(ctx, std::max(most, survivors + (bm_words + 263) / 264 * 256));
    const int room = (small ? select_room<512>(ctx) : select_room<1024>(ctx)) / 4;
    const int fit = std::min(ctx->sv_cap, SEL_KEYS(bm_words <= room / 2 ? room - bm_words : room));
    // How many may survive by the first digit alone: the sample takes 11 us, mon_select as long for 10,000 more items (131,072
    // candidates, a longest list of 8,192: 34, 35, 35, 39, 41, 46 us with 0, 2,000, ... 10,000 more, 46 with the sample).
    const int limit = std::max(survivors, std::min(survivors + 10000, fit));
    if (mode == 2) return launch_select<SRC_RANGE>(ctx, B, dc, gsel, max_nk, std::max(most, 8192), bm_words, small, st);
    const int wg = std::max(1, std::min((max_nchunk + NWAVE - 1) / NWAVE, std::max(4, 1024 / pivots)));
    mon_compact<<<dim3(wg, max_reps, n), dim3(BLK), hc_side_lds(ctx, (const void*)mon_compact, 0), st>>>(B, limit);
    HC_HIP(ctx, hipGetLastError());
    return launch_select<SRC_SURVIVORS>(ctx, B, dc, gsel, max_nk, std::max(most, limit), bm_words, small, st);
}

// Whether the combine pass of a group's attention makes the scores and histograms of its unfiltered layers (with the context set as for the
// monitor call that follows: the same choice of what selects).  Up to 64 K candidates a step waits for its side chain (two
// groups of two 32K layers: the main stream by itself 49 us a step, the chains 85), which then begins with the selection: a launch and
// its reads less.  us per step, mon_score_hist on the side stream / with the combine pass: four layers 16K 85 / 79, 32K 99 / 85, 48K 106 / 98, 60,000 110-152 /
// 99-142, one of 10,000 33.2 / 28.5, of 32K 41.4 / 36.8; twelve sequences of 9,000 to 31,000, two layers 155 / 136.  Where mon_compact and mon_select take
// the lists (more than 20 of them) as long as the group's attention is short, here up to 1600 rows to a compute unit (36 us of
// reading): eight layers of 36,000 in groups of four 141 / 129, four sequences, a layer to a group 115 / 105; of 60,000, two and a half times the
// rows, 150 / 155.  Longer contexts wait for the attention.  (Of steps with a side stream the copy to the caller's buffer takes back 0.5 to 1 us, where
// mon_select takes the lists 2 to 3: eight layers of 36,000 128.5 / 131, four sequences 101 / 104.)
bool hc_monitor_reads_scores(const hc_ctx* ctx, int n, const hc_monitor_call* calls, hc_score_plan* plan)
{
    int m = 0, reps = 0, nk = 1, k = 1, nchunk = 0, candidates = 0;
    int64_t rows = 0;
    for (int i = 0; i < n; ++i) {
        const hc_layer* L = calls[i].L;
        rows += L->total_rows;
        if (hc_layer_filtered(ctx, L)) continue;
        ++m;
        reps = std::max(reps, L->n_reps);
        nk = std::max(nk, L->max_nk);
        k = std::max(k, L->max_k_any);
        nchunk = std::max(nchunk, L->max_nchunk);
        candidates = std::max(candidates, L->max_cand);
        if (!L->score_buf) return false;             // (made when its ranges were longer)
    }
    if (candidates <= SELECT_DIRECT || candidates > HC_SCORED_MOST) return false;
    const Choice how = choose(ctx, 0, false, false, false, candidates, reps * m * nk, nchunk, k, nk);
    if (how.long_lists || (!how.direct && rows > 1600 * (int64_t)ctx->n_cu)) return false;
    *plan = hc_score_plan{how.hist, how.direct ? direct_most(how.form, DIRECT_HIST, candidates) : HC_SCORED_MOST, nchunk};
    return true;
}

// The histograms of scores made with the combine pass, after a step that failed between that pass and the selection.
hc_status hc_launch_clear_hist(hc_ctx* ctx, const hc_layer* L, hipStream_t st)
{
    Ws ws{};                                             // (max_ctx 0: no bitmaps with these)
    ws.hist = L->score_hist;
    mon_prep<<<dim3(16, L->n_reps), dim3(256), 0, st>>>(ws);
    HC_HIP(ctx, hipGetLastError());
    return HC_OK;
}

hc_status hc_launch_monitor(hc_ctx* ctx, int n, const hc_monitor_call* calls, int scores_given, hipStream_t st)
{
    if (n < 1 || n > HC_MAX_GROUP) return hc_fail(ctx, HC_EINVAL, "monitor batch of %d layers", n);
    // Layers whose split pass filtered the pivot logits are handled over the kept rows, with the dense chain behind
    // them; all others (and every call that brings its own scores or logits: given scores, the window's re-scored
    // queries, the prefill-time selection) by the plain chain.
    const hc_monitor_call* plain[HC_MAX_GROUP];
    const hc_monitor_call* filt[HC_MAX_GROUP];
    int n_plain = 0, n_filt = 0;
    for (int i = 0; i < n; ++i) {
        const hc_monitor_call& x = calls[i];
        const bool f = !scores_given && x.store_slot == -1 && x.reps == nullptr && hc_layer_filtered(ctx, x.L);
        if (f && !(x.arena ? x.arena : x.L->last_arena))
            return hc_fail(ctx, HC_ESTATE, "monitor of a filtering layer before any attention call with pivot logits");
        (f ? filt[n_filt++] : plain[n_plain++]) = &x;
    }
    hc_status s = HC_OK;
    if (n_plain > 0) s = run_chain(ctx, n_plain, plain, 0, scores_given, 0, st);
    if (s == HC_OK && n_filt > 0) {
        s = run_chain(ctx, n_filt, filt, n_plain, 0, 1, st);
        // behind it, for the pivots whose check failed (decided on the device; normally none): all logits over
        // again with their scores, then the plain chain's rest over those
        if (s == HC_OK) {
            hc_rep_logits_call rl[HC_MAX_GROUP];
            for (int i = 0; i < n_filt; ++i) {
                const hc_monitor_call& x = *filt[i];
                rl[i] = hc_rep_logits_call{x.L, x.arena ? x.arena : x.L->last_arena, const_cast<float*>(x.rep_logits), x.lse, x.scores};
            }
            s = hc_launch_rep_logits(ctx, n_filt, rl, st);
        }
        if (s == HC_OK) s = run_chain(ctx, n_filt, filt, n_plain, 0, 2, st);
        if (s == HC_OK)
            for (int i = 0; i < n_filt; ++i) const_cast<hc_layer*>(filt[i]->L)->filter_armed = true;
    }
    if (s != HC_OK) return s;
    // everything enqueued: the workspace copies will be clear again when this call completes.  (Not so under
    // stream capture, where nothing has run yet and the graph may never be launched: they stay marked.)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) cap = hipStreamCaptureStatusActive;
    if (cap == hipStreamCaptureStatusNone)
        for (int i = 0; i < n; ++i) ctx->ws[i].dirty = false;
    return HC_OK;
}

hc_status hc_monitor_set_lds_limit()
{
    // mon_select takes most of a compute unit's LDS, and beside the attention pass every kernel here reserves more
    // than half of it (hc_side_lds)
    const void* fns[] = {(const void*)mon_direct<512, DIRECT_HIST, 1, false>, (const void*)mon_direct<512, DIRECT_MAP, 1, false>, (const void*)mon_direct<512, DIRECT_SCORES, 1, false>,
                         (const void*)mon_direct<512, DIRECT_LOGITS, 1, false>, (const void*)mon_direct<512, DIRECT_LOGITS, 2, false>, (const void*)mon_direct<512, DIRECT_LOGITS, 4, false>,
                         (const void*)mon_direct<512, DIRECT_LOGITS, 8, false>, (const void*)mon_direct<1024, DIRECT_HIST, 1, false>, (const void*)mon_direct<1024, DIRECT_MAP, 1, false>,
                         (const void*)mon_direct<1024, DIRECT_SCORES, 1, false>, (const void*)mon_direct<1024, DIRECT_LOGITS, 1, false>, (const void*)mon_direct<1024, DIRECT_LOGITS, 2, false>,
                         (const void*)mon_direct<1024, DIRECT_LOGITS, 4, false>, (const void*)mon_direct<1024, DIRECT_LOGITS, 8, false>, (const void*)mon_direct<512, DIRECT_HIST, 1, true>, (const void*)mon_direct<1024, DIRECT_HIST, 1, true>,
                         (const void*)mon_select<512, SRC_SURVIVORS, true>, (const void*)mon_select<1024, SRC_SURVIVORS, true>, (const void*)mon_hist<2>, (const void*)mon_hist<3>, (const void*)mon_count, (const void*)mon_write, (const void*)mon_decide,
                         (const void*)mon_compact, (const void*)mon_sparse_score<1>,
                         (const void*)mon_sparse_score<2>, (const void*)mon_sparse_score<4>, (const void*)mon_sparse_score<8>,
                         (const void*)mon_score_hist<1, HIST_KEYS>, (const void*)mon_score_hist<2, HIST_KEYS>, (const void*)mon_score_hist<4, HIST_KEYS>, (const void*)mon_score_hist<8, HIST_KEYS>,
                         (const void*)mon_score_hist<1, HIST_FINE>, (const void*)mon_score_hist<2, HIST_FINE>, (const void*)mon_score_hist<4, HIST_FINE>, (const void*)mon_score_hist<8, HIST_FINE>,
                         (const void*)mon_score_hist<1, HIST_LINEAR>, (const void*)mon_score_hist<2, HIST_LINEAR>, (const void*)mon_score_hist<4, HIST_LINEAR>, (const void*)mon_score_hist<8, HIST_LINEAR>,
                         (const void*)mon_select<512, SRC_SCORES, false>, (const void*)mon_select<512, SRC_SURVIVORS, false>, (const void*)mon_select<512, SRC_RANGE, false>,
                         (const void*)mon_select<1024, SRC_SCORES, false>, (const void*)mon_select<1024, SRC_SURVIVORS, false>, (const void*)mon_select<1024, SRC_RANGE, false>};
    for (const void* fn : fns)
        if (hc_allow_lds(fn) != hipSuccess) return HC_EHIP;
    return HC_OK;
}
