// hc_gather.hip -- AsyncUpdate of Algorithm 1 (Sec. 4.3): C_GPU^(s) <- C_CPU^(s)[I_s].
//
// The host tier is pinned host memory that the kernels read directly over the host link, 512
// contiguous bytes per retrieved position (its K row followed by its V row), so no host thread has
// to learn which pivots fired: the predicate (flag of the satellite's pivot) is read on the device
// and an untriggered call finds no rows to move.  32 lanes move one position: lanes 0-15
// the K row, lanes 16-31 the V row, 16 bytes each.
//
// The host link is the bound (about 55 GB/s against a refill of 10 MB per pivot), so with a slot map
// (slot_pos: which position every retrieved slot holds) only the difference moves: positions of the new
// list that are not resident go into the slots of resident positions that left the list.  The resident
// set afterwards is exactly the list; the order of the slots is not ascending any more, which attention
// does not care about.  gather_plan_bitmap_kernel finds the difference and moves its rows (for contexts whose bitmaps do
// not fit in LDS gather_plan_kernel finds it and gather_kernel moves the rows).
#include <algorithm>
#include <type_traits>

#include "hc_internal.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int GATHER_PASSES = 4;     // host reads a lane of gather_kernel has in flight
constexpr int PLAN_THREADS = 256;

// One layer of a batched call (gather_plan_kernel: blockIdx.z picks the layer; the others go through the satellites of all).
struct GatherItem {
    const SatDev* sats;
    const HeadDev* heads;
    const uint16_t* tier;
    const int32_t* topk_idx;
    const int32_t* flag;
    uint16_t* arena;
    int32_t* slot_pos;      // [B*Hkv][max_k] or nullptr: no slot map, the whole list is fetched in list order
    int32_t* pair_slot;     // [B*Hkv][max_k] workspace: the slots to overwrite ...
    int32_t* pair_pos;      // [B*Hkv][max_k]            ... and the positions that go there
    int32_t* npairs;        // [B*Hkv]
    int32_t* done;          // [B*Hkv] workgroups that are through with a satellite's slot map; zero between launches, which must not overlap
    int n_sats, pad;
};
struct GatherBatch {
    GatherItem it[HC_MAX_GROUP];
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }       // (kept in a scalar register)
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    return (int64_t)(((uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32) | (uint32_t)uniform((int)v));
}

// Index of v in the ascending list a[0, n), or -1.
__device__ __forceinline__ int find_sorted(const int32_t* a, int n, int32_t v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return (lo < n && a[lo] == v) ? lo : -1;
}

// Exclusive prefix sums of two per-thread counts over the workgroup (PLAN_THREADS threads); totals returned.
__device__ __forceinline__ void block_exscan2(uint32_t a, uint32_t b, uint32_t* sm, uint32_t& ex_a, uint32_t& ex_b,
                                              uint32_t& tot_a, uint32_t& tot_b)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t ia = a, ib = b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t ta = __shfl_up(ia, o), tb = __shfl_up(ib, o);
        if (lane >= o) {
            ia += ta;
            ib += tb;
        }
    }
    if (lane == 63) {
        sm[w * 2] = ia;
        sm[w * 2 + 1] = ib;
    }
    __syncthreads();
    uint32_t base_a = 0, base_b = 0;
    tot_a = tot_b = 0;
    for (int i = 0; i < PLAN_THREADS / 64; ++i) {
        if (i < w) {
            base_a += sm[i * 2];
            base_b += sm[i * 2 + 1];
        }
        tot_a += sm[i * 2];
        tot_b += sm[i * 2 + 1];
    }
    ex_a = base_a + ia - a;
    ex_b = base_b + ib - b;
}

// Rows to move of every satellite of a batch: entry e is satellite e % max_sats of item e / max_sats, count(item, satellite) its
// rows if its pivot fired.  Every wave goes through the entries for itself (each(e, rows), 64 to a call, lanes past the end
// with none), so that a launch that finds nothing to move, the usual case in a decode step, ends without a barrier.
constexpr int MAX_GATHER_SATS = 1024;     // satellites of a batch (layers x satellites per layer)
template <class Count, class Each>
__device__ __forceinline__ void entry_rows(const GatherBatch& B, int n_ent, int max_sats, const Count& count, const Each& each)
{
    const int lane = threadIdx.x & 63;
    auto chunks = [&](auto per, int base) {          // `per` times 64 entries, whose reads are in flight together
        constexpr int U = decltype(per)::value;
        const GatherItem* it[U];
        SatDev sd[U];
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * 64 + lane, sidx = e % max_sats;
            it[u] = &B.it[min(e / max_sats, HC_MAX_GROUP - 1)];
            sd[u].rep_bh = -1;
            if (e < n_ent && sidx < it[u]->n_sats) sd[u] = it[u]->sats[sidx];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = 0;
            if (sd[u].rep_bh >= 0) c[u] = it[u]->flag[sd[u].rep_bh];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c[u] != 0) c[u] = count(*it[u], sd[u]);
            each(base + u * 64 + lane, c[u]);
        }
    };
    if (n_ent <= 64) {
        chunks(std::integral_constant<int, 1>{}, 0);
    } else {
#pragma unroll 1
        for (int base = 0; base < n_ent; base += 256) chunks(std::integral_constant<int, 4>{}, base);
    }
}
__device__ __forceinline__ int wave_incl(int v)      // inclusive prefix sum over the wave
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o);
        if ((int)(threadIdx.x & 63) >= o) v += t;
    }
    return v;
}
constexpr int entry_words(int n_ent) { return (n_ent + 4) & ~3; }      // LDS for a count each and one more, a multiple of 16 bytes

// Moves pairs [begin, end) of a satellite: the row of position pos[k] from the tier into slot[k].  32 lanes move one position
// (lanes 0-15 its K row, 16-31 its V row, 16 bytes each), the first `movers` threads take part, PASSES positions each in flight:
// every host read of a pass is issued before the first store.
template <int PASSES>
__device__ __forceinline__ void move_rows(const GatherItem& it, const HeadDev& hd, int first_slot, int r, const int32_t* slot, const int32_t* pos, int begin,
                                          int end, int movers)
{
    int tid = threadIdx.x;
    asm("" : "+v"(tid));                 // (what follows from it is not kept in registers across the caller's loop)
    const int nsub = movers >> 5, sub = tid >> 5, is_v = (tid >> 4) & 1, chunk = tid & 15;
    if (tid >= movers) return;
    const u32x4* tier = reinterpret_cast<const u32x4*>(it.tier + uniform64(hd.tier_off));
    const long long to = (is_v ? uniform64(hd.v_off) : uniform64(hd.k_off)) / 8 + (long long)first_slot * 16 + chunk;
    u32x4* arena = reinterpret_cast<u32x4*>(it.arena);
    const int ctx = uniform(hd.ctx), piece = is_v * 16 + chunk;
#pragma unroll 1
    for (int k0 = begin + sub; k0 < end; k0 += nsub * PASSES) {
        u32x4 buf[PASSES];
        bool ok[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int j = pos[min(k0 + p * nsub, end - 1)];
            ok[p] = k0 + p * nsub < end && j >= 0 && j < ctx;        // a corrupt entry must not leave the tier block ...
            if (ok[p]) buf[p] = __builtin_nontemporal_load(tier + (size_t)j * 32 + piece);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int s = slot[min(k0 + p * nsub, end - 1)];
            if (ok[p] && s >= 0 && s < r) arena[to + (long long)s * 16] = buf[p];       // ... or the head's slots
        }
    }
}

// Pairs c0 .. c1 - 1 of a satellite's plan to slot[] and pos[]: a wave compacts its rounds r0 .. r1 - 1 of the masks, whose first free slot
// and fresh position are numbers at_free and at_fresh.  want: the list's entries of the first U rounds, read again if `again`.
template <int U, int NT>
__device__ __forceinline__ void write_pairs(int32_t* slot, int32_t* pos, int c0, int c1, const int32_t* list, uint32_t (&want)[U], bool again, bool over, int r,
                                            int r0, int r1, const uint64_t* free_mask, const uint64_t* fresh_mask, uint32_t at_free, uint32_t at_fresh)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t n = (uint32_t)(c1 - c0);
    if (over) {
#pragma unroll 1
        for (int i = tid; i < (int)n; i += NT) {
            slot[i] = c0 + i;
            pos[i] = list[c0 + i];
        }
        return;
    }
    at_free -= (uint32_t)c0;
    at_fresh -= (uint32_t)c0;
#pragma unroll 1
    for (int q0 = r0; q0 < r1; q0 += U) {
        if (again) {
#pragma unroll
            for (int u = 0; u < U; ++u) want[u] = (uint32_t)list[min((q0 + u) * 64 + lane, r - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (q0 + u >= r1) break;
            const uint64_t mf = free_mask[q0 + u], mn = fresh_mask[q0 + u], below = (1ull << lane) - 1ull;
            const uint32_t a = at_free + (uint32_t)__builtin_popcountll(mf & below), b = at_fresh + (uint32_t)__builtin_popcountll(mn & below);
            if (((mf >> lane) & 1u) && a < n) slot[a] = (q0 + u) * 64 + lane;
            if (((mn >> lane) & 1u) && b < n) pos[b] = (int32_t)want[u];
            at_free += (uint32_t)__builtin_popcountll(mf);
            at_fresh += (uint32_t)__builtin_popcountll(mn);
        }
    }
}

// Which slots of a satellite hold positions that left the list (free), which positions of the list are not resident (fresh);
// the k-th free slot takes the k-th fresh position.  And the move of those rows, in the same launch: the satellites that are to be
// refilled get workgroups in proportion to their lists (so that the time does not depend on how unequal these are, and a launch
// has as many workgroups as the host link needs, no more); each makes the plan and moves its share of the pairs.  Several
// workgroups then make the same plan, which costs no time (they would wait for it otherwise); the last of them to be
// through with the slot map brings it up to date.  (With the lists' rows dealt out in equal runs, some workgroups planned two
// satellites one after the other: six lists of 420 to 800 entries 19.5 us, this way 15.0; in two
// launches 16.3.)
//
// Two bitmaps over the context in LDS, of the listed positions and of those held by a slot, so that every slot and every
// list entry costs one LDS access; choices are kept as one mask per 64 entries, and a wave's run of them is compacted with
// ballots.  The plan is a chain of latencies: list and slot map are asked for together, at the start.
// Six lists of 704 to 7,872 entries, a quarter new, 2.6 MB over the link (45 us at its rate): 54 us, 66 in two launches (a plan
// by a workgroup per satellite, 11 us, then the rows, 54).  A launch that finds nothing to do takes 4 us.
// A workgroup's share of the pairs stays in LDS, in the place of the bitmaps: written to memory and read back (all pairs, by every
// workgroup of the satellite) they cost a round trip and a wait for the stores in front of the first row.  us, through memory / LDS: one list of
// 320 10.3 / 9.7, six of 420 to 640 15.1 / 13.8, 42 of 600 to 2,300 123 / 120.6, the six lists above 54.6 / 54.0.
// PLAN: the plan alone, a task to a satellite, whether its pivot fired or not; gather_kernel moves the rows.
template <int NT, bool PLAN>
__global__ __launch_bounds__(NT) void gather_plan_bitmap_kernel(GatherBatch B, int n_items, int max_sats, int max_k, int movers)
{
    constexpr int NW = NT / 64, U = NT == 512 ? 4 : 8;
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    __shared__ uint32_t sm_cnt[2][NW];
    __shared__ int sm_last;
    const int n_ent = n_items * max_sats, n_wgs = (int)gridDim.x;
    int* sm_first = reinterpret_cast<int*>(dyn);     // [n_ent + 1]
    uint32_t* sm_words = dyn + entry_words(n_ent);
    int total = 0, fired = 0;
    if (!PLAN) {
        entry_rows(B, n_ent, max_sats, [](const GatherItem&, const SatDev& sd) { return sd.r; }, [&](int e, int rows) {
            if (threadIdx.x < 64 && e < n_ent) sm_first[e] = rows;
            total += uniform(__builtin_amdgcn_readlane(wave_incl(rows), 63));
            fired += __builtin_popcountll(__builtin_amdgcn_ballot_w64(rows > 0));
        });
        if (total == 0) return;
    }
    const int tid = threadIdx.x, wv = uniform(tid >> 6), lane = tid & 63;
    // List rows to a task: where there are at least twice as many workgroups as satellites, such that every task has a workgroup of
    // its own; otherwise half a workgroup's, so that those who get two tasks or three are evenly busy, but 256 at least: a task makes its
    // satellite's whole plan, 7 us, about what 256 rows of a list take.  (Calls over satellites of 16,384, lists a quarter new, by 48
    // workgroups.  24, 27, 36, 42 satellites, lists of 80 to 140: 16, 17, 19, 21 us, without the lower bound 16, 26, 28, 28; of 310 to
    // 610: 37, 45, 49, 63, without 37, 44, 57, 59, with 512 37, 40, 49, 70.  Tasks of a workgroup's rows: 22, 22, 24, 25 and 45, 46, 56, 58.)
    const int by = 2 * fired <= n_wgs ? n_wgs - fired : 2 * n_wgs, share = max((total + by - 1) / by, 2 * fired <= n_wgs ? 1 : 256);
    if (!PLAN && wv == 0) {                     // rows -> first task (one for each of a satellite's workgroups)
        int before = 0;
#pragma unroll 1
        for (int base = 0; base < n_ent; base += 64) {
            const int mine = base + lane < n_ent ? (sm_first[base + lane] + share - 1) / share : 0, incl = before + wave_incl(mine);
            if (base + lane < n_ent) sm_first[base + lane] = incl - mine;
            before = __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) sm_first[n_ent] = before;
    }
    __syncthreads();
    const int tasks = PLAN ? n_ent : uniform(sm_first[n_ent]);
#pragma unroll 1
    for (int task = blockIdx.x; task < tasks; task += n_wgs) {           // (the same for the whole workgroup)
        int e = 0, part = 0, parts = 1;
        if (PLAN) {
            e = task;
        } else {
            for (int hi = n_ent; hi - e > 1;) {      // the last entry whose tasks begin at or before this one
                const int mid = (e + hi) >> 1;
                if (uniform(sm_first[mid]) <= task) e = mid;
                else hi = mid;
            }
            part = task - uniform(sm_first[e]);
            parts = uniform(sm_first[e + 1]) - uniform(sm_first[e]);
        }
        const GatherItem& it = B.it[e / max_sats];
        if (PLAN && (e % max_sats >= it.n_sats || it.flag[it.sats[e % max_sats].rep_bh] == 0)) continue;
        const int bh = uniform(it.sats[e % max_sats].bh), r = uniform(it.sats[e % max_sats].r), first_slot = uniform(it.sats[e % max_sats].first_slot);
        const HeadDev& hd = it.heads[bh];
        const uint32_t ctx = (uint32_t)uniform(hd.ctx);
        const int words = (int)(ctx + 31) / 32, rounds = (r + 63) / 64;
        uint32_t* listed = sm_words;
        uint32_t* held = sm_words + words;
        uint64_t* free_mask = reinterpret_cast<uint64_t*>(sm_words + ((2 * words + 3) & ~3));       // [rounds]: slots whose position left the list
        uint64_t* fresh_mask = free_mask + rounds;                                                   // [rounds]: list entries no slot holds
        const int32_t* list = it.topk_idx + (size_t)bh * max_k;
        int32_t* sp = it.slot_pos + (size_t)bh * max_k;
        // a wave takes a run of rounds of 64, U of them at a time; the first U stay in registers
        const int per = (rounds + NW - 1) / NW, r0 = min(rounds, wv * per), r1 = min(rounds, r0 + per);
        auto load = [&](uint32_t (&p)[U], const int32_t* src, int q0) {
#pragma unroll
            for (int u = 0; u < U; ++u) p[u] = q0 + u < r1 && (q0 + u) * 64 + lane < r ? (uint32_t)src[(q0 + u) * 64 + lane] : ctx;
        };
        uint32_t want[U], have[U];
        load(want, list, r0);
        load(have, sp, r0);
#pragma unroll 1
        for (int i = tid; i < 2 * words; i += NT) sm_words[i] = 0u;
        __syncthreads();
#pragma unroll 1
        for (int q0 = r0; q0 < r1; q0 += U) {
            if (q0 != r0) {
                load(want, list, q0);
                load(have, sp, q0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (want[u] < ctx) atomicOr(&listed[want[u] >> 5], 1u << (want[u] & 31));
                if (have[u] < ctx) atomicOr(&held[have[u] >> 5], 1u << (have[u] & 31));
            }
        }
        __syncthreads();
        uint32_t n_free = 0, n_fresh = 0;
#pragma unroll 1
        for (int q0 = r0; q0 < r1; q0 += U) {
            if (per > U) {                           // (registers hold the last rounds)
                load(want, list, q0);
                load(have, sp, q0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (q0 + u >= r1) break;
                const bool in = (q0 + u) * 64 + lane < r;
                const bool keep = have[u] < ctx && ((listed[min(have[u], ctx - 1) >> 5] >> (have[u] & 31)) & 1u);      // (a position held twice, a corrupt map, is caught by the count check below)
                const bool there = want[u] < ctx && ((held[min(want[u], ctx - 1) >> 5] >> (want[u] & 31)) & 1u);
                const uint64_t mf = __builtin_amdgcn_ballot_w64(in && !keep), mn = __builtin_amdgcn_ballot_w64(in && !there);
                if (lane == 0) {
                    free_mask[q0 + u] = mf;
                    fresh_mask[q0 + u] = mn;
                }
                n_free += (uint32_t)__builtin_popcountll(mf);
                n_fresh += (uint32_t)__builtin_popcountll(mn);
            }
        }
        if (lane == 0) {
            sm_cnt[0][wv] = n_free;
            sm_cnt[1][wv] = n_fresh;
        }
        __syncthreads();                             // (this workgroup has read the slot map)
        int ticket = 0;
        if (!PLAN && tid == 0 && parts > 1) ticket = atomicAdd(it.done + bh, 1);
        uint32_t at_free = 0, at_fresh = 0, tot_free = 0, tot_fresh = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            at_free += i < wv ? sm_cnt[0][i] : 0u;
            at_fresh += i < wv ? sm_cnt[1][i] : 0u;
            tot_free += sm_cnt[0][i];
            tot_fresh += sm_cnt[1][i];
        }
        at_free = (uint32_t)uniform((int)at_free);
        at_fresh = (uint32_t)uniform((int)at_fresh);
        tot_free = (uint32_t)uniform((int)tot_free);
        tot_fresh = (uint32_t)uniform((int)tot_fresh);
        const bool over = tot_free != tot_fresh;     // the slot map does not describe a set of r distinct positions: start over from the list
        const int pairs = over ? r : (int)tot_free;
        if constexpr (PLAN) {
            int32_t* pslot = it.pair_slot + (size_t)bh * max_k;
            int32_t* ppos = it.pair_pos + (size_t)bh * max_k;
            write_pairs<U, NT>(pslot, ppos, 0, pairs, list, want, per > U, over, r, r0, r1, free_mask, fresh_mask, at_free, at_fresh);
            __syncthreads();                         // the pairs are complete (and visible to the whole workgroup)
#pragma unroll 1
            for (int k = tid; k < pairs; k += NT) sp[pslot[k]] = ppos[k];
            if (tid == 0) it.npairs[bh] = pairs;
            __syncthreads();
        } else {
            // this workgroup's share of the pairs, in the bitmaps' place (as many at a time as there are words to a bitmap)
            int32_t* slot = reinterpret_cast<int32_t*>(sm_words);
            int32_t* pos = slot + words;
            const int k_begin = (int)((long long)pairs * part / parts), k_end = (int)((long long)pairs * (part + 1) / parts);
            auto own = [&](int c0, bool again) __attribute__((always_inline)) {
                write_pairs<U, NT>(slot, pos, c0, min(k_end, c0 + words), list, want, per > U || again, over, r, r0, r1, free_mask, fresh_mask, at_free, at_fresh);
            };
            own(k_begin, false);
            if (tid == 0) {
                sm_last = parts > 1 && ticket == parts - 1;
                if (sm_last) it.done[bh] = 0;
            }
            __syncthreads();
            if (sm_last) {                           // everyone has read the slot map: bring it up to date
#pragma unroll 1
                for (int c0 = 0; c0 < pairs; c0 += words) {
                    const int c1 = min(pairs, c0 + words);
                    write_pairs<U, NT>(slot, pos, c0, c1, list, want, true, over, r, r0, r1, free_mask, fresh_mask, at_free, at_fresh);
                    __syncthreads();
#pragma unroll 1
                    for (int k = tid; k < c1 - c0; k += NT) sp[slot[k]] = pos[k];
                    __syncthreads();
                }
                own(k_begin, true);
                __syncthreads();
            }
#pragma unroll 1
            for (int c0 = k_begin; c0 < k_end; c0 += words) {
                if (c0 != k_begin) {
                    own(c0, true);
                    __syncthreads();
                }
                const int n = min(k_end - c0, words);
                if (parts == 1)
#pragma unroll 1
                    for (int k = tid; k < n; k += NT) sp[slot[k]] = pos[k];
                move_rows<2>(it, hd, first_slot, r, slot, pos, 0, n, movers);
                __syncthreads();
            }
            __syncthreads();                         // (the next satellite takes over the LDS)
        }
    }
}

// The same for contexts whose bitmaps do not fit.  Dynamic LDS: the list (4 r bytes), found[r], keep[r].
__global__ __launch_bounds__(PLAN_THREADS) void gather_plan_kernel(GatherBatch B, int max_k)
{
    extern __shared__ int32_t sm_list[];
    __shared__ uint32_t sm_scan[2 * PLAN_THREADS / 64];
    const GatherItem& it = B.it[blockIdx.z];
    if ((int)blockIdx.y >= it.n_sats) return;
    const SatDev sd = it.sats[blockIdx.y];
    if (it.flag[sd.rep_bh] == 0) return;
    const int r = sd.r, tid = threadIdx.x;
    uint8_t* found = reinterpret_cast<uint8_t*>(sm_list + max_k);     // found[i]: list entry i is resident
    uint8_t* keep = found + max_k;                                     // keep[s]: slot s holds a listed position
    const int32_t* list = it.topk_idx + (size_t)sd.bh * max_k;
    int32_t* sp = it.slot_pos + (size_t)sd.bh * max_k;
    int32_t* pslot = it.pair_slot + (size_t)sd.bh * max_k;
    int32_t* ppos = it.pair_pos + (size_t)sd.bh * max_k;
    for (int i = tid; i < r; i += PLAN_THREADS) {
        sm_list[i] = list[i];
        found[i] = 0;
    }
    __syncthreads();
    for (int s = tid; s < r; s += PLAN_THREADS) {
        const int idx = find_sorted(sm_list, r, sp[s]);
        keep[s] = idx >= 0;
        if (idx >= 0) found[idx] = 1;       // a position held twice (a corrupt map) is caught by the count check below
    }
    __syncthreads();
    // each thread owns a contiguous run of slots / list entries, so that both compactions keep their order
    const int per = (r + PLAN_THREADS - 1) / PLAN_THREADS;
    const int e0 = min(r, tid * per), e1 = min(r, e0 + per);
    uint32_t n_free = 0, n_fresh = 0;
    for (int e = e0; e < e1; ++e) {
        n_free += !keep[e];
        n_fresh += !found[e];
    }
    uint32_t off_free, off_fresh, tot_free, tot_fresh;
    block_exscan2(n_free, n_fresh, sm_scan, off_free, off_fresh, tot_free, tot_fresh);
    if (tot_free != tot_fresh) {
        // the slot map does not describe a set of r distinct positions: start over from the list
        for (int i = tid; i < r; i += PLAN_THREADS) {
            pslot[i] = i;
            ppos[i] = sm_list[i];
            sp[i] = sm_list[i];
        }
        if (tid == 0) it.npairs[sd.bh] = r;
        return;
    }
    for (int e = e0; e < e1; ++e) {
        if (!keep[e]) pslot[off_free++] = e;
        if (!found[e]) ppos[off_fresh++] = sm_list[e];
    }
    __syncthreads();                        // the pairs are complete (and visible to the whole workgroup)
    for (int k = tid; k < (int)tot_free; k += PLAN_THREADS) sp[pslot[k]] = ppos[k];
    if (tid == 0) it.npairs[sd.bh] = (int32_t)tot_free;
}

// The refill where no bitmap plan moves the rows as well: whole lists (no slot map), and the pairs of gather_plan_kernel.  The rows
// of all satellites are numbered consecutively and dealt to the workgroups in equal runs.  A
// workgroup of T threads (64, 128 or 256) has T / 8 positions in flight.
__global__ __launch_bounds__(256, 8) void gather_kernel(GatherBatch B, int n_items, int max_sats, int max_k)
{
    __shared__ int sm_start[MAX_GATHER_SATS + 1];
    const int n_ent = n_items * max_sats;
    const int nthr = blockDim.x;            // 64, 128 or 256
    int total = 0;
    entry_rows(B, n_ent, max_sats, [](const GatherItem& it, const SatDev& sd) { return it.slot_pos ? min(max(it.npairs[sd.bh], 0), sd.r) : sd.r; },
               [&](int e, int rows) {
                   const int incl = total + wave_incl(rows);
                   if (threadIdx.x < 64 && e < n_ent) sm_start[e] = incl - rows;
                   total = __builtin_amdgcn_readlane(incl, 63);
               });
    if (total == 0) return;
    if (threadIdx.x == 0) sm_start[n_ent] = total;
    __syncthreads();
    const int per = ((total + (int)gridDim.x - 1) / (int)gridDim.x + 7) & ~7;
    const int g_begin = blockIdx.x * per, g_end = min(total, g_begin + per);
    const int nsub = nthr >> 5;                // positions of a sub-pass
    const int sub = threadIdx.x >> 5;          // which of them this half-wave moves
    const int l32 = threadIdx.x & 31;
    const int is_v = l32 >> 4;                 // lanes 16..31 move the V row
    const int chunk = l32 & 15;                // 16-byte chunk of the 256-byte row
    for (int row_first = g_begin; row_first < g_end; row_first += nsub * GATHER_PASSES) {
        u32x4 buf[GATHER_PASSES];
        u32x4* dst[GATHER_PASSES];
#pragma unroll
        for (int p = 0; p < GATHER_PASSES; ++p) {          // issue every host read first: they are latency-bound
            const int g = row_first + p * nsub + sub;
            dst[p] = nullptr;
            if (g < g_end) {
                int lo = 0, hi = n_ent;                    // the entry whose run holds row g
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (sm_start[mid] <= g) lo = mid;
                    else hi = mid;
                }
                const GatherItem& it = B.it[lo / max_sats];
                const SatDev sd = it.sats[lo % max_sats];
                const HeadDev hd = it.heads[sd.bh];
                const int i = g - sm_start[lo];
                const bool delta = it.slot_pos != nullptr;
                const int j = (delta ? it.pair_pos : it.topk_idx)[(size_t)sd.bh * max_k + i];
                const int sl = delta ? it.pair_slot[(size_t)sd.bh * max_k + i] : i;
                if (j >= 0 && j < hd.ctx && sl >= 0 && sl < sd.r) {     // a corrupt entry must not leave the tier block or the head's slots
                    const u32x4* src = reinterpret_cast<const u32x4*>(it.tier + hd.tier_off);
                    buf[p] = __builtin_nontemporal_load(src + (size_t)j * 32 + is_v * 16 + chunk);
                    dst[p] = reinterpret_cast<u32x4*>(it.arena + (is_v ? hd.v_off : hd.k_off)) + (size_t)(sd.first_slot + sl) * 16 + chunk;
                }
            }
        }
#pragma unroll
        for (int p = 0; p < GATHER_PASSES; ++p)
            if (dst[p]) *dst[p] = buf[p];
    }
}

}   // namespace

hc_status hc_launch_gather(hc_ctx* ctx, int n, const hc_gather_call* calls, bool may_overlap, hipStream_t st)
{
    if (n < 1 || n > HC_MAX_GROUP) return hc_fail(ctx, HC_EINVAL, "gather batch of %d layers", n);
    GatherBatch B{};
    int max_r = 0, max_sats = 0;
    bool any_delta = false;
    const int max_k = ctx->cfg.max_k;
    const size_t rows = (size_t)ctx->cfg.B * ctx->cfg.Hkv;
    for (int i = 0; i < n; ++i) {
        const hc_gather_call& x = calls[i];
        GatherItem& it = B.it[i];
        it = GatherItem{x.L->sats, x.L->heads, (const uint16_t*)x.tier, x.topk_idx, x.flag, (uint16_t*)x.arena, x.slot_pos,
                        ctx->pair_slot + i * rows * max_k, ctx->pair_pos + i * rows * max_k, ctx->npairs + i * rows,
                        ctx->gather_done + i * rows, x.L->n_sats, 0};
        any_delta |= x.slot_pos != nullptr;
        max_r = std::max(max_r, x.L->max_r);
        max_sats = std::max(max_sats, x.L->n_sats);
    }
    if (max_sats == 0 || max_r == 0) return HC_OK;
    if (n * max_sats > MAX_GATHER_SATS) return hc_fail(ctx, HC_ESHAPE, "hc_gather: more than %d satellites in a batch", MAX_GATHER_SATS);
    // A few dozen workgroups keep the host link busy.  More do not make the refill much faster, and every compute unit
    // that hosts gather waves has its memory pipeline filled with reads that take microseconds, behind which the
    // attention waves on the same unit queue (measured at the 224K shape with 16 workgroups per satellite in a
    // batch of 8 layers: the attention launch that ran beside a refill took 400 us instead of 45).  One refill of 2.6 MB by
    // itself with 32, 48, 64, 96, 160 workgroups: 60, 57, 57, 57, 54 us.  Beside the attention pass 48; but groups of up to four
    // layers with many satellites have little attention to hide a refill behind.  Steps with a drift at each, contexts of 66,000 to
    // 123,000, us with 48 / 96: groups of two layers, 36 satellites 290 282, 48 347 339, 72 590 575, 192 883 859; of four, 96 satellites 852
    // 857, whole-list jumps 947 914; of eight, 48 satellites (32 layers of 131,072) 34.4 and 35.9 a layer, of 229,376 47.5 and 48.2.
    long long rows_max = 0;
    for (int i = 0; i < n; ++i) rows_max += (long long)calls[i].L->n_sats * calls[i].L->max_r;
    const int thr = ctx->gather_threads, in_flight = thr / 32 * GATHER_PASSES;
    const int most = ctx->gather_workgroups > 0 ? ctx->gather_workgroups : ctx->beside_now && (n > 4 || 2 * n * max_sats <= 48) ? 48 : 96;
    const int nwg = (int)std::max<long long>(1, std::min<long long>(most, (rows_max + in_flight - 1) / in_flight));
    if (any_delta) {
        for (int i = 0; i < n; ++i)
            if (!calls[i].slot_pos) return hc_fail(ctx, HC_EINVAL, "hc_gather: in one batch either every layer has a slot map or none");
        const size_t lds = (size_t)max_k * (sizeof(int32_t) + 2);
        if (lds > 144 * 1024) return hc_fail(ctx, HC_ESHAPE, "hc_gather: max_k %d is too large for the slot-map path", max_k);
        // Where the bitmaps of the longest context, a mask per 64 entries and the satellites' first rows fit in LDS (beside the
        // attention pass: within what its workgroups leave of a compute unit's), one launch plans and moves; otherwise
        // a plan by binary search, a workgroup per satellite, and gather_kernel behind it (a list of 7,872: 43 us + 55).
        const unsigned maps = ((unsigned)ctx->cfg.max_ctx / 32 * 2 + 4) * 4 + (unsigned)((max_k + 63) / 64) * 16 + entry_words(n * max_sats) * 4;
        const unsigned room = (!ctx->beside_now ? 156 * 1024 : ctx->G == 8 ? 56 * 1024 : ctx->side_pad_now ? 110 * 1024 : 76 * 1024) - 256;
        // Many satellites, and perhaps another stream's attention pass on the GPU (a call by itself): the plan first, then gather_kernel,
        // whose workgroups are small enough to leave attention's their places.  By itself this takes the same from 48
        // satellites on; refills of whole lists of 66 / 96 satellites, 0.8 and 1.1 ms, made eight attention launches beside them 283 / 280 us
        // longer this way, 531 / 634 in one launch; of 48 265 and 361, but there one launch is 5 % faster, and of 24 161 and 187.
        const bool apart = may_overlap && n * max_sats > 48;
        if (maps <= room && apart) {
            gather_plan_bitmap_kernel<1024, true><<<dim3(std::min(n * max_sats, 256)), dim3(1024), maps, st>>>(B, n, max_sats, max_k, 0);
            HC_HIP(ctx, hipGetLastError());
        } else if (maps <= room) {
            if (ctx->beside_now)
                gather_plan_bitmap_kernel<512, false><<<dim3(nwg), dim3(512), hc_side_lds(ctx, (const void*)gather_plan_bitmap_kernel<512, false>, maps), st>>>(B, n, max_sats, max_k, thr);
            else
                gather_plan_bitmap_kernel<1024, false><<<dim3(nwg), dim3(1024), maps, st>>>(B, n, max_sats, max_k, 2 * thr);
            HC_HIP(ctx, hipGetLastError());
            return HC_OK;
        } else {
            gather_plan_kernel<<<dim3(1, max_sats, n), dim3(PLAN_THREADS), hc_side_lds(ctx, (const void*)gather_plan_kernel, (unsigned)lds), st>>>(B, max_k);
            HC_HIP(ctx, hipGetLastError());
        }
    }
    gather_kernel<<<dim3(nwg), dim3(thr), hc_side_lds(ctx, (const void*)gather_kernel, 0), st>>>(B, n, max_sats, max_k);
    HC_HIP(ctx, hipGetLastError());
    return HC_OK;
}

// the plan kernel may need more dynamic LDS than the default 64 KB limit, and beside the attention pass both kernels
// reserve more than half of a compute unit's LDS (hc_side_lds)
hc_status hc_gather_set_lds_limit()
{
    if (hc_allow_lds((const void*)gather_plan_bitmap_kernel<512, false>) != hipSuccess ||
        hc_allow_lds((const void*)gather_plan_bitmap_kernel<1024, false>) != hipSuccess ||
        hc_allow_lds((const void*)gather_plan_bitmap_kernel<1024, true>) != hipSuccess) return HC_EHIP;
    if (hc_allow_lds((const void*)gather_plan_kernel) != hipSuccess || hc_allow_lds((const void*)gather_kernel) != hipSuccess) return HC_EHIP;
    return HC_OK;
}
