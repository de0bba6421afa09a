// Iterative rerouting (Section 2.3; the assignment step of the "-I" variants of Section 4): top-k with
// capacity, then the dropped pairs are re-proposed, round by round, to the best expert that still has room.
// A fast heuristic beside the exact solver; it works on the same integer rewards, so every decision is an
// integer comparison.
//
// Orders (the paper leaves them open; these are fixed here so that the result is one well-defined assignment):
//   stage 1  pairs are taken by (choice rank, token id); an expert keeps the first C pairs naming it;
//   stage 2  at the start of a round the experts with room are fixed; a token fills its holes in slot order with
//            its best experts among those (not held, not yet proposed this round); proposals are taken by
//            (slot, token id) and an expert accepts while it has room; rounds repeat until nobody proposes.
// Stage 1 is a round of stage 2 in which everybody has room, so both run through the same two kernels:
//   k_iter_step   a block of 64 tokens takes the outcome of the round before and proposes for the holes that are left; a
//                 wavefront is 64 tokens of one slot, whose proposals per expert it counts
//   k_iter_scan   per expert: an expert with room for all its proposals needs no order; for the others the counts of
//                 the blocks before, slot by slot, tell how many of a block's proposals there is room for
// Once few pairs are left the step makes a list of them and a workgroup of the scan goes through all further rounds (iter_tail).
// The next round is enqueued when the step of one has begun; the first round without proposals, or of which no expert has room left, or
// the tail ends them, and what follows is enqueued while that runs.  All bound by latency: a step 6 to 8 us, a scan 6 to 7, the tail 25 for
// four rounds.  (The tail's LDS and threads cost a scan 0.5 us; as a kernel of its own it costs a launch instead, which is as much.)  A layer of 44032 tokens, 64 experts, top-2: 319 us with nine rounds of two launches, two of them enqueued ahead and what
// follows behind the host's wait, 296 now; route_logits of 60 batches of 64 to 65536 tokens to 8 to 256 experts 15 % less on average.
#include <algorithm>
#include <climits>

#include "common.h"
#include "host_words.h"
#include "iter_tail.h"
#include "row_keys.h"

namespace maxscore {
namespace {

struct IterState {
    unsigned long long total;
    int flow;
    int pad;
};

constexpr int kIterRows = 64, kScanThreads = 1024;
constexpr int kIterEnds = INT_MAX;                        // progress: steps that have begun, or that the last one has
constexpr int kIterWordProgress = 1, kIterWordFlow = 2, kIterWordRounds = 3, kIterWordOpen = 10, kIterWordTotal = 8;

// Tables of the rounds, in the workspace (WorkspaceLayout::price_off).
struct IterArea {
    int load[2][kMaxE];        // tokens per expert before round r, in half r & 1
    int cnt[kMaxE];            // proposals of the last round
    int tot[8][kMaxE];         // ... of the round in progress, in eight partial counts
    int any[4];                // whether there were proposals in round r, in word r & 3
    int rej[4];                // ... those there was no room for
    int room[4];               // ... whether an expert has room left
    long long t_end, t_after;  // device clock (10 ns) behind the last round, and at the end of the caller's work behind that
    int arrived;               // workgroups of that work's last kernel
};

struct IterArgs {
    const int32_t *q;
    int32_t *assign, *list;    // list: proposals, slot-major
    IterArea *ar;
    int *any;                  // per (slot, block): whether there are proposals
    void *tiles;               // per (slot, block): proposals per expert, 64 at most; then how many of them there is room for
    int *wcnt;                 // result: pairs per (block, expert)
    long long *bsum;           // ... reward per block
    int *bflow;                // ... pairs per block
    int T, E, k, C, n_wg;
    int ebits;
    int tail;                  // pairs that one workgroup takes at most (-1: none)
    int scan;                  // threads of a workgroup that a scan needs
};

// Best live expert of a row spread over a wavefront (lane l holds experts l, l+64, ...; bit c of `live` says
// whether the lane's c-th expert may still be chosen): largest reward, ties to the lower expert id; -1 if no
// expert is live.
template <int EPL>
__device__ inline int wave_best(const int (&val)[EPL], unsigned live)
{
    int m = INT_MIN;
#pragma unroll
    for (int c = 0; c < EPL; ++c)
        if (((live >> c) & 1) && val[c] > m) m = val[c];
    for (int off = 32; off >= 1; off >>= 1) {
        const int o = __shfl_xor(m, off);
        m = o > m ? o : m;
    }
    int e = -1;
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        const unsigned long long b = __ballot(((live >> c) & 1) && val[c] == m);
        if (e < 0 && b) e = 64 * c + __ffsll((long long)b) - 1;
    }
    return e;
}

__device__ inline unsigned drop_expert(unsigned live, int e, int lane)
{
    return (e >= 0 && lane == (e & 63)) ? live & ~(1u << (e >> 6)) : live;
}

// choice[s*T + i] <- the token's s-th best expert, s < k (slot-major list).  One wavefront per token row;
// lane l holds experts l, l+64, ...
template <int EPL>
__global__ __launch_bounds__(256) void k_iter_topk(const int32_t *__restrict__ q, int T, int E, int k,
                                                   int32_t *__restrict__ choice)
{
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    for (int row = wave; row < T; row += n_waves) {
        int val[EPL];
        unsigned live = 0;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const int e = lane + 64 * c;
            val[c] = e < E ? q[(size_t)row * E + e] : 0;
            live |= (e < E ? 1u : 0u) << c;
        }
        int mine = -1;
        for (int s = 0; s < k; ++s) {
            const int e = wave_best<EPL>(val, live);
            live = drop_expert(live, e, lane);
            if (lane == s) mine = e;
        }
        if (lane < k) choice[(size_t)lane * T + row] = mine;
    }
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lanes that hold the same expert as this one (0 for a lane without one)
__device__ __forceinline__ unsigned long long same_expert(int e, int ebits)
{
    unsigned long long same = __ballot(e >= 0);
    for (int b = 0; b < ebits; ++b) {
        const unsigned long long bal = __ballot((e >> b) & 1);
        same &= ((e >> b) & 1) ? bal : ~bal;
    }
    return e >= 0 ? same : 0ull;
}

template <int G>
__device__ __forceinline__ int group_max(int v)
{
    return (int)(~group_min_u32<G>(~((unsigned)v ^ 0x80000000u)) ^ 0x80000000u);
}

__global__ __launch_bounds__(1024) void k_iter_init(IterArea *ar)
{
    int *p = (int *)ar;
    for (int i = threadIdx.x; i < (int)(sizeof(IterArea) / 4); i += 1024) p[i] = 0;
}

// Which step of the rounds this is.  No step is enqueued behind one that ends them.
enum { kIterOn, kIterTail, kIterFull, kIterNone };        // ends them: in one workgroup, nobody has room, there were no proposals
__device__ __forceinline__ int iter_phase(const IterArgs &a, int r, int last)
{
    const IterArea *ar = a.ar;
    const int w = (r - 1) & 3, any = ar->any[w], rej = ar->rej[w], room = ar->room[w];      // (requested together)
    if (r == 0) return kIterOn;
    if (any == 0) return kIterNone;
    if (last) return kIterOn;
    return room == 0 ? kIterFull : rej <= a.tail ? kIterTail : kIterOn;
}

// G lanes own a token row, lane l columns (m >> 2) * 4G + 4l + (m & 3) for m < EPL (EPL >= 4), else l * EPL + m.
template <int G, int EPL, typename Tile>
__global__ __launch_bounds__(256) void k_iter_step(IterArgs a, int r, int last, int *host)
{
    extern __shared__ int s_mem[];
    const int E = a.E, k = a.k, T = a.T;
    int *s_slot = s_mem;                          // [64][k]
    int *s_prop = s_slot + kIterRows * k;         // [k][64]
    int *s_room = s_prop + kIterRows * k;         // [E] room for the round before, then for this one
    int *s_num = s_room + E;                      // [E] proposals of the round before
    int *s_cnt = s_num + E;                       // [4][E]
    __shared__ int s_queue[kIterRows];
    __shared__ int s_nq;
    __shared__ long long s_sum[4];
    __shared__ int s_flow[4];
    IterArea *ar = a.ar;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.x, row0 = w * kIterRows;
    const int nr = T - row0 < kIterRows ? T - row0 : kIterRows;
    const int phase = iter_phase(a, r, last);
    if (w == 0 && tid == 0) {
        ((volatile int *)host)[kIterWordProgress] = phase == kIterOn ? r + 1 : kIterEnds;
        ar->any[r & 3] = ar->rej[r & 3] = ar->room[r & 3] = 0;
    }
    const bool final = phase != kIterOn || last;
    for (int i = tid; i < nr * k; i += 256) s_slot[i] = r < 2 ? -1 : a.assign[(size_t)row0 * k + i];
    if (r > 0)
        for (int e = tid; e < E; e += 256) {
            s_room[e] = a.C - ar->load[(r - 1) & 1][e];
            s_num[e] = ar->cnt[e];
        }
    if (tid < kIterRows) s_queue[tid] = 0;        // kIterTail: the slots of a row that go on
    __syncthreads();
    if (phase != kIterNone && r > 0) {
        for (int s = wv; s < k; s += 4) {
            const int e = lane < nr ? a.list[(size_t)s * T + row0 + lane] : -1;
            if (!__any(e >= 0)) continue;
            const int room = e >= 0 ? s_room[e] : 0;
            bool take = e >= 0 && s_num[e] <= room;
            const bool asks = e >= 0 && !take && room > 0;
            if (__any(asks)) {
                const unsigned long long same = same_expert(e, a.ebits);
                if (asks) {
                    take = __popcll(same & ((1ull << lane) - 1)) < (int)((const Tile *)a.tiles)[((size_t)s * a.n_wg + w) * E + e];
                }
            }
            if (take) {
                s_slot[lane * k + s] = e;
                if (r > 1) a.assign[(size_t)(row0 + lane) * k + s] = e;
            } else if (phase == kIterTail && e >= 0) atomicOr((unsigned *)&s_queue[lane], 1u << s);
        }
        __syncthreads();
        if (r == 1)
            for (int i = tid; i < nr * k; i += 256) a.assign[(size_t)row0 * k + i] = s_slot[i];
    }
    if (final) {
        if (phase == kIterTail && wv == 0) {
            const unsigned mask = (unsigned)s_queue[lane];
            const unsigned long long b = __ballot(mask != 0);
            const int at = row0 + __popcll(b & ((1ull << lane) - 1));
            if (mask) {
                a.list[at] = row0 + lane;
                if (k > 1) a.list[T + at] = (int)mask;
            }
            if (lane == 0) a.any[w] = __popcll(b);
        }
        for (int e = tid; e < E; e += 256) s_cnt[e] = 0;
        __syncthreads();
        long long sum = 0;
        int flow = 0;
        for (int i = tid; i < nr * k; i += 256) {
            const int e = s_slot[i];
            if (e >= 0) {
                atomicAdd(&s_cnt[e], 1);
                sum += a.q[(size_t)(row0 + i / k) * E + e];
                ++flow;
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            sum += __shfl_xor(sum, off);
            flow += __shfl_xor(flow, off);
        }
        if (lane == 0) {
            s_sum[wv] = sum;
            s_flow[wv] = flow;
        }
        __syncthreads();
        for (int e = tid; e < E; e += 256) a.wcnt[(size_t)w * E + e] = s_cnt[e];
        if (tid == 0) {
            a.bsum[w] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
            a.bflow[w] = s_flow[0] + s_flow[1] + s_flow[2] + s_flow[3];
        }
        return;
    }
    for (int e = tid; e < E; e += 256) {
        s_room[e] = a.C - ar->load[r & 1][e];
        s_num[e] = 0;                              // now: proposals of this block
    }
    for (int i = tid; i < kIterRows * k; i += 256) s_prop[i] = -1;
    if (wv == 0) {                                 // the rows that have holes
        bool hole = false;
        if (lane < nr)
            for (int s = 0; s < k; ++s) hole |= s_slot[lane * k + s] < 0;
        const unsigned long long b = __ballot(hole);
        if (hole) s_queue[__popcll(b & ((1ull << lane) - 1))] = lane;
        if (lane == 0) s_nq = __popcll(b);
    }
    __syncthreads();
    const int lg = tid & (G - 1), grp = tid / G, nq = s_nq;
    const bool vec = EPL >= 4 && (E & 3) == 0 && ((size_t)a.q & 15) == 0;
    using RK = RowKeys<G, EPL>;
    auto col = [&](int m) { return RK::col(m, lg); };
    unsigned roomy = 0;
#pragma unroll
    for (int m = 0; m < EPL; ++m)
        if (col(m) < E && s_room[col(m)] > 0) roomy |= 1u << m;
    const int ib = a.ebits > 0 ? a.ebits : 1;
    for (int i = grp; i < nq; i += 256 / G) {
        const int lr = s_queue[i];
        const int32_t *qr = a.q + (size_t)(row0 + lr) * E;
        int v[EPL];
        RK::load(qr, E, vec, lg, v);
        unsigned live = roomy;
        for (int s = 0; s < k; ++s) {
            const int e = s_slot[lr * k + s];
            if (e < 0) continue;
            const int l = EPL >= 4 ? (e >> 2) & (G - 1) : e / EPL, m = EPL >= 4 ? e / (4 * G) * 4 + (e & 3) : e % EPL;
            if (l == lg) live &= ~(1u << m);
        }
        // rewards that span less than 2^(32 - ib), as those of scores do: packed with their columns, lower experts first
        int lo = INT_MAX, hi = INT_MIN;
#pragma unroll
        for (int m = 0; m < EPL; ++m)
            if ((live >> m) & 1) {
                lo = v[m] < lo ? v[m] : lo;
                hi = v[m] > hi ? v[m] : hi;
            }
        lo = ~group_max<G>(~lo);
        hi = group_max<G>(hi);
        if (hi < lo) continue;                             // nobody to ask
        if ((((unsigned)hi - (unsigned)lo + 1) >> (32 - ib)) == 0 && (unsigned)hi - (unsigned)lo != ~0u) {
            const unsigned cmask = (1u << ib) - 1;
            unsigned key[EPL];
#pragma unroll
            for (int m = 0; m < EPL; ++m)
                key[m] = (live >> m) & 1 ? ((unsigned)v[m] - (unsigned)lo + 1) << ib | (cmask - (unsigned)col(m)) : 0u;
            unsigned cur = RK::first(key);
            for (int s = 0; s < k && cur != 0; ++s) {
                if (s_slot[lr * k + s] >= 0) continue;
                if (lg == 0) s_prop[s * kIterRows + lr] = (int)(cmask - (cur & cmask));
                const unsigned next = RK::below(key, cur);
                cur = next < cur ? next : 0u;              // (below the last one the search wraps around)
            }
            continue;
        }
        for (int s = 0; s < k; ++s) {
            if (s_slot[lr * k + s] >= 0) continue;
            // the largest reward, the lowest expert that has it
            int best = INT_MIN;
#pragma unroll
            for (int m = 0; m < EPL; ++m)
                if (((live >> m) & 1) && v[m] > best) best = v[m];
            best = group_max<G>(best);
            int low = INT_MAX;
#pragma unroll
            for (int m = EPL - 1; m >= 0; --m)
                if (((live >> m) & 1) && v[m] == best) low = col(m);
            low = ~group_max<G>(~low);
            if (low == INT_MAX) break;                     // nobody left to ask
            const int l = EPL >= 4 ? (low >> 2) & (G - 1) : low / EPL, m = EPL >= 4 ? low / (4 * G) * 4 + (low & 3) : low % EPL;
            if (l == lg) live &= ~(1u << m);
            if (lg == 0) s_prop[s * kIterRows + lr] = low;
        }
    }
    __syncthreads();
    for (int s = wv; s < k; s += 4) {
        const int e = s_prop[s * kIterRows + lane];
        const size_t tile = (size_t)s * a.n_wg + w;
        if (lane < nr) a.list[(size_t)s * T + row0 + lane] = e;
        const bool some = __any(e >= 0);
        if (lane == 0) a.any[tile] = some;
        if (!some) continue;
        int *cnt = s_cnt + wv * E;
        for (int x = lane; x < E; x += 64) cnt[x] = 0;
        wave_lds_sync();
        const unsigned long long same = same_expert(e, a.ebits);
        if (e >= 0 && lane == __ffsll((long long)same) - 1) {
            const int n = __popcll(same);
            cnt[e] = n;
            atomicAdd(&s_num[e], n);
        }
        wave_lds_sync();
        for (int x = lane; x < E; x += 64) ((Tile *)a.tiles)[tile * E + x] = (Tile)cnt[x];
        wave_lds_sync();
    }
    __syncthreads();
    for (int e = tid; e < E; e += 256)
        if (s_num[e]) atomicAdd(&ar->tot[w & 7][e], s_num[e]);
}

// What the blocks have reported and what came later, to the host (one workgroup; every thread comes with its share).
__device__ __forceinline__ void iter_report(const IterArgs &a, long long sum, int flow, int rounds, int open, int *host)
{
    __shared__ int s_w[kScanThreads / 64];
    __shared__ long long s_sum[kScanThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int i = tid; i < a.n_wg; i += blockDim.x) {
        sum += a.bsum[i];
        flow += a.bflow[i];
    }
    for (int off = 32; off >= 1; off >>= 1) {
        sum += __shfl_xor(sum, off);
        flow += __shfl_xor(flow, off);
    }
    if (lane == 0) {
        s_sum[wv] = sum;
        s_w[wv] = flow;
    }
    __syncthreads();
    if (tid == 0) {
        sum = 0;
        flow = 0;
        for (int x = 0; x < (int)blockDim.x >> 6; ++x) {
            sum += s_sum[x];
            flow += s_w[x];
        }
        tell_host((long long *)(host + kIterWordTotal), sum);
        tell_host(host + kIterWordFlow, flow);
        tell_host(host + kIterWordRounds, rounds);
        tell_host(host + kIterWordOpen, open);
        tell_host(host, 1);              // (read when the stream has been waited for: a fence here took 3 us)
        a.ar->t_end = wall_clock64();
    }
}

// The best but `skip` of a row's live columns (bit m of `live`: this lane's m-th), ties to the lower expert; -1 if there are no more.
template <int G, int EPL>
__device__ __forceinline__ int iter_best(const int (&v)[EPL], unsigned live, int lg, int ib, int skip)
{
    using RK = RowKeys<G, EPL>;
    int lo = INT_MAX, hi = INT_MIN;
#pragma unroll
    for (int m = 0; m < EPL; ++m)
        if ((live >> m) & 1) {
            lo = v[m] < lo ? v[m] : lo;
            hi = v[m] > hi ? v[m] : hi;
        }
    lo = ~group_max<G>(~lo);
    hi = group_max<G>(hi);
    if (hi < lo) return -1;
    if ((((unsigned)hi - (unsigned)lo + 1) >> (32 - ib)) == 0 && (unsigned)hi - (unsigned)lo != ~0u) {       // (packed with their columns)
        const unsigned cmask = (1u << ib) - 1;
        unsigned key[EPL];
#pragma unroll
        for (int m = 0; m < EPL; ++m)
            key[m] = (live >> m) & 1 ? ((unsigned)v[m] - (unsigned)lo + 1) << ib | (cmask - (unsigned)RK::col(m, lg)) : 0u;
        unsigned cur = RK::first(key);
        for (int x = 0; x < skip && cur != 0; ++x) {
            const unsigned next = RK::below(key, cur);
            cur = next < cur ? next : 0u;                  // (below the last one the search wraps around)
        }
        return cur != 0 ? (int)(cmask - (cur & cmask)) : -1;
    }
    for (int x = 0;; ++x) {
        int best = INT_MIN;
#pragma unroll
        for (int m = 0; m < EPL; ++m)
            if (((live >> m) & 1) && v[m] > best) best = v[m];
        best = group_max<G>(best);
        int low = INT_MAX;
#pragma unroll
        for (int m = EPL - 1; m >= 0; --m)
            if (((live >> m) & 1) && v[m] == best) low = RK::col(m, lg);
        low = ~group_max<G>(~low);
        if (low == INT_MAX) return -1;
        if (x == skip) return low;
        const int l = EPL >= 4 ? (low >> 2) & (G - 1) : low / EPL, m = EPL >= 4 ? low / (4 * G) * 4 + (low & 3) : low % EPL;
        if (l == lg) live &= ~(1u << m);
    }
}

// Rounds r, r + 1, ... of the pairs the step has listed, in one workgroup: round by round a proposal of every pair, by G lanes each; a
// rank among the proposals for an expert without room for all of them; the pairs that were turned away go on, in their order (slot,
// token).  A pair that finds nobody to ask drops out: from round to round a token's open slots do not lose more slots before it than
// experts it could ask.  Bound by latency, 2 us a round of few pairs; 44032 tokens of 64 experts, top-2: four rounds of 672 pairs and less.
template <int G, int EPL>
__device__ __forceinline__ void iter_tail(const IterArgs &a, int r, int max_rounds, int *host)
{
    using RK = RowKeys<G, EPL>;
    extern __shared__ int s_mem[];
    __shared__ int s_w[kScanThreads / 64], s_tile[kTailMost / 64], s_flag[2];
    constexpr int NT = kScanThreads, NW = NT / 64, TILES = kTailMost / 64 / NW;      // tiles of 64 pairs a wavefront
    const int E = a.E, k = a.k, N = a.tail, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *s_tok = s_mem, *s_slot = s_tok + 2 * N, *s_room = s_slot + k * N, *s_cnt = s_room + E, *s_pre = s_cnt + E;
    unsigned *s_open = (unsigned *)s_tok + N, *s_ent = (unsigned *)s_pre, *s_ent2 = s_ent + N;
    unsigned short *s_prop = (unsigned short *)(s_ent2 + N);
    int *s_tab = s_pre + 2 * N + (N + 1) / 2;
    constexpr unsigned short none = 0xffff;
    auto before_me = [&](int v, int &total) {            // exclusive sum over the workgroup (two barriers)
        int inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (lane == 63) s_w[wv] = inc;
        __syncthreads();
        int base = 0, all = 0;
        for (int x = 0; x < NW; ++x) {
            const int y = s_w[x];
            base += x < wv ? y : 0;
            all += y;
        }
        __syncthreads();
        total = all;
        return base + inc - v;
    };
    // the rows, in token order
    int H = 0;
    for (int w0 = 0; w0 < a.n_wg; w0 += NT) {
        const int w = w0 + tid, c = w < a.n_wg ? a.any[w] : 0;
        int all;
        const int at = H + before_me(c, all);
        if (w < a.n_wg) s_pre[w] = at;
        H += all;
    }
    if (tid == 0) s_pre[a.n_wg] = H;
    for (int e = tid; e < E; e += NT) s_room[e] = a.C - a.ar->load[r & 1][e];
    if (tid < 2) s_flag[tid] = -1;
    __syncthreads();
    H = H < N ? H : N;                                   // (never more)
    for (int h = tid; h < H; h += NT) {
        int lo = 0, hi = a.n_wg;                         // the last block whose first row is not behind h
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_pre[mid] <= h) lo = mid;
            else hi = mid;
        }
        const int at = lo * kIterRows + (h - s_pre[lo]);
        s_tok[h] = a.list[at];
        s_open[h] = k > 1 ? (unsigned)a.list[a.T + at] : 1u;
    }
    __syncthreads();
    for (int i = tid; i < H * k; i += NT) s_slot[i] = a.assign[(size_t)s_tok[i / k] * k + i % k];
    // their pairs, by slot, then by token
    const int chunks = (H + 63) / 64;
    for (int c = wv; c < chunks; c += NW) {
        const unsigned m = c * 64 + lane < H ? s_open[c * 64 + lane] : 0u;
        for (int s = 0; s < k; ++s) {
            const int cnt = __popcll(__ballot((m >> s) & 1u));
            if (lane == 0) s_tab[s * chunks + c] = cnt;
        }
    }
    __syncthreads();
    int n = 0;
    for (int i0 = 0; i0 < k * chunks; i0 += NT) {
        const int i = i0 + tid, c = i < k * chunks ? s_tab[i] : 0;
        int all;
        const int at = n + before_me(c, all);
        if (i < k * chunks) s_tab[i] = at;
        n += all;
    }
    __syncthreads();
    for (int c = wv; c < chunks; c += NW) {
        const int row = c * 64 + lane;
        const unsigned m = row < H ? s_open[row] : 0u;
        for (int s = 0; s < k; ++s) {
            const unsigned long long b = __ballot((m >> s) & 1u);
            const int at = s_tab[s * chunks + c] + __popcll(b & ((1ull << lane) - 1));
            if (((m >> s) & 1u) && at < N) s_ent[at] = (unsigned)(row << 8 | s);
        }
    }
    n = n < N ? n : N;
    const int lg = tid & (G - 1), grp = tid / G;
    const bool vec = EPL >= 4 && (E & 3) == 0 && ((size_t)a.q & 15) == 0;
    const int ib = a.ebits > 0 ? a.ebits : 1;
    long long sum = 0;
    int flow = 0, rounds = 0, open = 0, got[TILES] = {};          // got: rewards on their way
    for (int round = r;; ++round) {
        for (int e = tid; e < E; e += NT) s_cnt[e] = 0;
        __syncthreads();
        unsigned roomy = 0;
#pragma unroll
        for (int m = 0; m < EPL; ++m)
            if (RK::col(m, lg) < E && s_room[RK::col(m, lg)] > 0) roomy |= 1u << m;
        int nx[EPL];                                     // the next pair's row is on its way
        if (grp < n) RK::load(a.q + (size_t)s_tok[s_ent[grp] >> 8] * E, E, vec, lg, nx);
        for (int i = grp; i < n; i += NT / G) {
            const unsigned ent = s_ent[i];
            const int row = (int)(ent >> 8), s = (int)(ent & 255);
            const int skip = __popc(s_open[row] & ((1u << s) - 1));          // open slots before this one take the best first
            int v[EPL];
#pragma unroll
            for (int m = 0; m < EPL; ++m) v[m] = nx[m];
            if (i + NT / G < n) RK::load(a.q + (size_t)s_tok[s_ent[i + NT / G] >> 8] * E, E, vec, lg, nx);
            unsigned live = roomy;
            for (int x = 0; x < k; ++x) {
                const int e = s_slot[row * k + x];
                if (e < 0) continue;
                const int l = EPL >= 4 ? (e >> 2) & (G - 1) : e / EPL, m = EPL >= 4 ? e / (4 * G) * 4 + (e & 3) : e % EPL;
                if (l == lg) live &= ~(1u << m);
            }
            const int best = iter_best<G, EPL>(v, live, lg, ib, skip);
            if (lg == 0) {
                s_prop[i] = best < 0 ? none : (unsigned short)best;
                if (best >= 0) atomicAdd(&s_cnt[best], 1);
            }
        }
        __syncthreads();
        for (int e = tid; e < E; e += NT) {
            if (s_cnt[e] > 0) s_flag[0] = round;
            if (s_cnt[e] > s_room[e]) s_flag[1] = round;
        }
        __syncthreads();
        if (s_flag[0] != round) {
            rounds = round - 1;
            break;
        }
        const int tiles = (n + 63) / 64;
        const bool ranks = s_flag[1] == round;
        int prop[TILES];
        unsigned long long same[TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const int t = wv + j * NW, i = t * 64 + lane;
            prop[j] = t < tiles && i < n && s_prop[i] != none ? (int)s_prop[i] : -1;
            same[j] = 0;
            if (!ranks || t >= tiles) continue;
            same[j] = same_expert(prop[j], a.ebits);
            for (int e = lane; e < E; e += 64) s_tab[t * E + e] = 0;
            wave_lds_sync();
            if (prop[j] >= 0 && lane == __ffsll((long long)same[j]) - 1) s_tab[t * E + prop[j]] = __popcll(same[j]);
        }
        if (ranks) __syncthreads();
        bool take[TILES];
        unsigned ent[TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            sum += got[j];
            got[j] = 0;
        }
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const int t = wv + j * NW, e = prop[j];
            take[j] = e >= 0;
            ent[j] = 0;
            if (t >= tiles) continue;
            if (e >= 0) {
                ent[j] = s_ent[t * 64 + lane];
                const int room = s_room[e];
                if (s_cnt[e] > room) {
                    int rank = __popcll(same[j] & ((1ull << lane) - 1));
                    for (int x = 0; x < t; ++x) rank += s_tab[x * E + e];
                    take[j] = rank < room;
                }
                if (take[j]) {
                    const int row = (int)(ent[j] >> 8), s = (int)(ent[j] & 255), tok = s_tok[row];
                    s_slot[row * k + s] = a.assign[(size_t)tok * k + s] = e;
                    atomicAnd(&s_open[row], ~(1u << s));
                    atomicAdd(&a.wcnt[(size_t)(tok / kIterRows) * E + e], 1);
                    got[j] = a.q[(size_t)tok * E + e];
                    ++flow;
                }
            }
            const int keep = __popcll(__ballot(e >= 0 && !take[j]));
            if (lane == 0) s_tile[t] = keep;
        }
        __syncthreads();
        for (int e = tid; e < E; e += NT) s_room[e] -= s_cnt[e] < s_room[e] ? s_cnt[e] : s_room[e];
        int left = 0, at[TILES] = {};
        for (int t = 0; t < tiles; ++t) {
#pragma unroll
            for (int j = 0; j < TILES; ++j)
                if (t == wv + j * NW) at[j] = left;
            left += s_tile[t];
        }
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const bool go_on = prop[j] >= 0 && !take[j];
            const unsigned long long b = __ballot(go_on);
            if (go_on) s_ent2[at[j] + __popcll(b & ((1ull << lane) - 1))] = ent[j];
        }
        unsigned *x = s_ent;
        s_ent = s_ent2;
        s_ent2 = x;
        n = left;
        if (round >= max_rounds) {
            rounds = max_rounds;
            open = max_rounds > 0;
            break;
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < TILES; ++j) sum += got[j];
    iter_report(a, sum, flow, rounds, open, host);
}

template <int G, int EPL, typename Tile>
__global__ __launch_bounds__(kScanThreads) void k_iter_scan(IterArgs a, int r, int last, int max_rounds, int *host)
{
    __shared__ int s_w[kScanThreads / 64];
    IterArea *ar = a.ar;
    const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int phase = iter_phase(a, r, last);
    if (phase == kIterTail) {
        if (e == 0) iter_tail<G, EPL>(a, r, max_rounds, host);
        return;
    }
    if (phase != kIterOn || last) {                // the end
        if (e == 0) iter_report(a, 0, 0, phase == kIterNone ? (r >= 2 ? r - 2 : 0) : r - 1, phase == kIterOn && max_rounds > 0, host);
        return;
    }
    if (tid >= a.scan) return;                     // (whole wavefronts; the barriers do not wait for them)
    int c = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) c += ar->tot[i][e];
    const int load = ar->load[r & 1][e], room = a.C - load;
    __syncthreads();
    if (tid < 8) ar->tot[tid][e] = 0;
    if (tid == 0) {
        ar->load[(r + 1) & 1][e] = load + (c < room ? c : room);
        ar->cnt[e] = c;
        if (c > 0) ar->any[r & 3] = 1;
        if (c < room) ar->room[r & 3] = 1;
        if (c > room) atomicAdd(&ar->rej[r & 3], c - (room > 0 ? room : 0));
    }
    if (c <= room || room <= 0) return;
    // eight tiles per thread and step, all on their way together
    const int n = a.k * a.n_wg;
    Tile *tiles = (Tile *)a.tiles;
    int before = 0;
    for (int b0 = 0; b0 < n; b0 += 8 * a.scan) {
        const int t0 = b0 + 8 * tid;
        int x[8], sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = t0 + i < n ? a.any[t0 + i] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = x[i] ? (int)tiles[(size_t)(t0 + i) * a.E + e] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += x[i];
        int inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (lane == 63) s_w[wv] = inc;
        __syncthreads();
        int run = before + inc - sum;
        for (int v = 0; v < (int)a.scan >> 6; ++v) {
            if (v < wv) run += s_w[v];
            before += s_w[v];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int left = room - run;
            if (x[i]) tiles[(size_t)(t0 + i) * a.E + e] = (Tile)(left < 0 ? 0 : left < kIterRows ? left : kIterRows);
            run += x[i];
        }
    }
}

__global__ __launch_bounds__(256) void k_iter_total(const int32_t *__restrict__ q, const int32_t *__restrict__ assign,
                                                    int T, int E, int k, IterState *__restrict__ st)
{
    __shared__ long long s_sum[4];
    __shared__ int s_cnt[4];
    const size_t n = (size_t)T * k;
    long long sum = 0;
    int cnt = 0;
    for (size_t a = (size_t)blockIdx.x * blockDim.x + threadIdx.x; a < n; a += (size_t)gridDim.x * blockDim.x) {
        const int e = assign[a];
        if (e >= 0) {
            sum += q[(a / k) * E + e];
            ++cnt;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        sum += __shfl_xor(sum, off);
        cnt += __shfl_xor(cnt, off);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        s_sum[wv] = sum;
        s_cnt[wv] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&st->total, (unsigned long long)(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]));
        atomicAdd(&st->flow, s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3]);
    }
}

template <int EPL>
void launch_topk(const int32_t *q, int T, int E, int k, int32_t *choice, hipStream_t s)
{
    const int grid = T < 4 * 2048 ? (T + 3) / 4 : 2048;
    hipLaunchKernelGGL(k_iter_topk<EPL>, dim3(grid), dim3(256), 0, s, q, T, E, k, choice);
}

}  // namespace

int32_t top1_run(const int32_t *q, int T, int E, int32_t *top1, hipStream_t s)
{
    const int epl = (E + 63) / 64;
    if (epl <= 1) launch_topk<1>(q, T, E, 1, top1, s);
    else if (epl <= 2) launch_topk<2>(q, T, E, 1, top1, s);
    else if (epl <= 4) launch_topk<4>(q, T, E, 1, top1, s);
    else if (epl <= 8) launch_topk<8>(q, T, E, 1, top1, s);
    else launch_topk<16>(q, T, E, 1, top1, s);
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

int32_t assign_total_run(const int32_t *q, const int32_t *assign, int T, int E, int k, void *state16,
                         int64_t *total, int32_t *flow, hipStream_t s)
{
    IterState *st = (IterState *)state16;
    IterState h = {};
    MS_HIP(hipMemcpyAsync(st, &h, sizeof(h), hipMemcpyHostToDevice, s));
    const size_t n = (size_t)T * k;
    int grid = (int)((n + 255) / 256);
    if (grid > 256) grid = 256;
    hipLaunchKernelGGL(k_iter_total, dim3(grid), dim3(256), 0, s, q, assign, T, E, k, st);
    MS_HIP(hipGetLastError());
    MS_HIP(hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, s));
    MS_HIP(hipStreamSynchronize(s));
    if (total) *total = (int64_t)h.total;
    if (flow) *flow = h.flow;
    return MAXSCORE_OK;
}

int32_t iter_run(const int32_t *q, int T, int E, int k, int C, int max_rounds, int32_t *assign, int64_t *total,
                 int32_t *flow, int32_t *rounds, float *after_ms, char *ws, hipStream_t s, IterAfter after, void *after_ctx)
{
    WorkspaceLayout L = workspace_layout(T, E, k);
    IterArgs a;
    a.q = q;
    a.assign = assign;
    a.list = (int32_t *)(ws + L.klist_off);
    a.n_wg = (T + kIterRows - 1) / kIterRows;
    char *at = ws + L.price_off;
    a.ar = (IterArea *)at;
    at += (sizeof(IterArea) + 255) / 256 * 256;
    a.bsum = (long long *)at;
    at += sizeof(long long) * a.n_wg;
    a.bflow = (int *)at;
    a.any = a.bflow + a.n_wg;
    // Words, or bytes where only these fit (more than 34 slots and 128 experts): stores of bytes to lines that several
    // chiplets write cost 44032 tokens of 64 experts, top-2, 140 us instead of 133.
    const size_t tiles_off = iter_tiles_off(L, T, E);
    const bool words = iter_tiles_are_words(L, T, E, k);
    if (!words && (E <= 128 || tiles_off + iter_tiles(T, E, k) > L.price_off)) return MAXSCORE_ERR_WORKSPACE;
    a.tiles = ws + tiles_off;
    a.wcnt = (int *)(ws + L.wcnt_off);
    a.T = T;
    a.E = E;
    a.k = k;
    a.C = C;
    a.ebits = 0;
    while ((1 << a.ebits) < E) ++a.ebits;
    int *host = nullptr, *host_dev = nullptr;
    int32_t rc = solver_words(&host, &host_dev);
    if (rc) return rc;
    volatile int *hw = host;
    hw[0] = hw[kIterWordProgress] = 0;

    int G = 8, EPL = 1;
    while (G * 16 < E) G *= 2;
    while (G * EPL < E) EPL *= 2;
    const size_t shm = sizeof(int) * ((size_t)2 * kIterRows * k + 6 * (size_t)E);
    a.tail = tail_most(E, k, a.n_wg);
    a.scan = std::min(kScanThreads, std::max(64, (k * a.n_wg + 511) / 512 * 64));       // eight tiles each
    const int threads = a.tail > 0 ? kScanThreads : a.scan;
    const size_t tail_shm = a.tail > 0 ? sizeof(int) * (size_t)tail_words(a.tail, E, k, a.n_wg) : 0;
    hipLaunchKernelGGL(k_iter_init, dim3(1), dim3(1024), 0, s, a.ar);
    bool ends = false;
    for (int r = 0; !ends; ++r) {
        const int last = r > max_rounds ? 1 : 0;
#define MS_IT(GG, PP, TT)                                                                                             \
    do {                                                                                                              \
        hipLaunchKernelGGL((k_iter_step<GG, PP, TT>), dim3(a.n_wg), dim3(256), shm, s, a, r, last, host_dev);         \
        hipLaunchKernelGGL((k_iter_scan<GG, PP, TT>), dim3(E), dim3(threads), tail_shm, s, a, r, last, max_rounds, host_dev); \
    } while (0)
#define MS_IB(GG)                                                                                                     \
    do {                                                                                                              \
        if (words) MS_IT(GG, 16, int);                                                                                \
        else MS_IT(GG, 16, unsigned char);                                                                            \
    } while (0)
        if (G == 8) {
            if (EPL == 1) MS_IT(8, 1, int);
            else if (EPL == 2) MS_IT(8, 2, int);
            else if (EPL == 4) MS_IT(8, 4, int);
            else if (EPL == 8) MS_IT(8, 8, int);
            else MS_IT(8, 16, int);
        } else if (G == 16) MS_IB(16);
        else if (G == 32) MS_IB(32);
        else MS_IB(64);
#undef MS_IB
#undef MS_IT
        if (hipGetLastError() != hipSuccess) {
            (void)hipStreamSynchronize(s);
            return MAXSCORE_ERR_HIP;
        }
        // The next round is enqueued when the step of this one has begun, unless that is the last: a launch that is queued in vain costs
        // 2 us, and the host is ready before this round ends.  The stream is looked at now and then, so that an error ends the wait.
        for (unsigned spin = 1;; ++spin) {
            const int begun = hw[kIterWordProgress];
            ends = last || begun == kIterEnds;
            if (ends || begun > r) break;
            if ((spin & 2047) == 0 && hipStreamQuery(s) != hipErrorNotReady && hw[kIterWordProgress] == begun) {
                (void)hipStreamSynchronize(s);
                return MAXSCORE_ERR_HIP;
            }
            __builtin_ia32_pause();
        }
    }
    // what follows is enqueued while the last round runs
    long long clock[2];
    DoneTell tell = {};
    bool told = false;
    rc = done_ticket(&tell, &a.ar->t_end, sizeof(clock) / 4);
    tell.arrived = &a.ar->arrived;
    const int32_t arc = rc == MAXSCORE_OK && after ? after(after_ctx, &a.ar->t_after, &tell, &told, s) : rc;
    rc = done_wait(tell, told, clock, s);
    if (rc) return rc;
    if (arc) return arc;
    if (after_ms) *after_ms = after ? (float)(clock[1] - clock[0]) * 1e-5f : 0.f;
    if (!hw[0]) return MAXSCORE_ERR_HIP;
    if (total) *total = *(volatile long long *)(host + kIterWordTotal);
    if (flow) *flow = hw[kIterWordFlow];
    if (rounds) *rounds = hw[kIterWordRounds];
    return hw[kIterWordOpen] ? MAXSCORE_ERR_NOT_CONVERGED : MAXSCORE_OK;
}

}  // namespace maxscore
