// Activation movement around the experts (Eq. 1; the capacity buffers of Section 2.3):
//   dispatch_tokens: expert input buffers [E, C, d] <- rows of x in dispatch order, zero padding
//   combine:         y[i, :] = sum_s gate[i, s] * expert_out[assign[i, s], token_pos[i, s], :]
// Both are permutations of rows of d values: HBM-bound, nothing to compute but the gate-weighted sum.
// A row is moved as 16-byte vectors by consecutive lanes, so every load and store of a wavefront is one
// contiguous kilobyte; the per-row indices are wavefront-uniform and read through the scalar path.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace maxscore {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <bool NT, typename V>
__device__ __forceinline__ void put(V v, V *p)
{
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <bool NT, typename V>
__device__ __forceinline__ V get(const V *p)
{
    return NT ? __builtin_nontemporal_load(p) : *p;
}

// One wavefront per destination row (slot r = j*C + s of the [E, C, d] buffer), grid-stride over rows.
// vec_per_row = d * elem_bytes / 16.
__global__ __launch_bounds__(256) void k_dispatch_tokens(const u32x4 *__restrict__ x,
                                                         const int32_t *__restrict__ offsets,
                                                         const int32_t *__restrict__ disp_token, int T, int E, int C,
                                                         int vec_per_row, u32x4 *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const long long n_rows = (long long)E * C;
    const long long wave0 = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const long long n_waves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long r = wave0; r < n_rows; r += n_waves) {
        const int j = (int)(r / C), s = (int)(r - (long long)j * C);
        const int o0 = offsets[j], cnt = offsets[j + 1] - o0;
        u32x4 *dst = out + r * vec_per_row;
        if (s < cnt) {
            const int tok = disp_token[o0 + s];
            const u32x4 *src = x + (size_t)(tok >= 0 && tok < T ? tok : 0) * vec_per_row;
            for (int c = lane; c < vec_per_row; c += 64) dst[c] = src[c];
        } else {
            for (int c = lane; c < vec_per_row; c += 64) dst[c] = u32x4{0u, 0u, 0u, 0u};
        }
    }
}

// The same by blocks of tokens: every list holds its tokens in ascending order, so the rows that want tokens
// [t0, t0 + tb) are one stretch of each list, found by bisection.  A workgroup turns its stretches into a list of rows
// per token, and a wavefront reads a token's row once and writes it to all of them.  A token in more than kTokenRows lists and
// lists in another order are served row by row.  In a list that is out of order the bisections of neighbouring workgroups can
// end far apart: of a descending list one workgroup gets everything.  So every workgroup looks at the same kListSamples entries
// first.  If these do not ascend, the stretches are equal shares of the list; if they do, they are the bisection's first steps.
// Either way the stretches cover every list exactly once, whatever its order: the samples and the same bisection with a
// larger key never end further left.  Workgroups from n_tb on zero the rows no token has.  These are neighbours, at the end of every
// list: a wavefront looks at rows that are as far apart as there are wavefronts, so that all of them get a share (a workgroup that took
// neighbouring rows could have nothing else: 7573 tokens of 1600 to 6 of 16 experts with room to spare 34 us, not 38; 65536 of 2048 to 6 of 8
// 400, not 436), and at another place between its neighbours each time (64 lists are as long as there are wavefronts, so that without
// it a wavefront would see the same place of every list: 10000 of 1024 to 1 of 64 with a tenth more room 9.0 us, 13.2 so, 9.9 with neighbouring rows).
// Bound by HBM: row by row in list order every row of x comes from memory k times once x is larger than the caches.
// 65536 tokens of 2048 to 8 of 128 experts: 683 to 441 us, 5.5 TB/s with x counted once (492 in a layer, behind the projection); 16384 to 8 of 64: 163 to 110 us.  The
// same in other orders: shuffled 632 us (2.8 ms without the samples), descending 640 (13.9), shuffled by eight 680 (785 with a
// list after the other instead of 64 together).
// LAST: the rows of x are read past the cache as well, which leaves it to what the projection has brought there.
constexpr int kBlockTokens = 32, kTokenRows = 16, kListMaxE = 2048, kListSamples = 8;

template <bool NT, bool LAST, int THREADS>
__global__ __launch_bounds__(THREADS) void k_dispatch_tokens_blocked(const u32x4 *__restrict__ x,
                                                                 const int32_t *__restrict__ offsets,
                                                                 const int32_t *__restrict__ disp_token, int T, int E,
                                                                 int C, int vec_per_row, int tb, int n_tb,
                                                                 u32x4 *__restrict__ out)
{
    extern __shared__ int s_mem[];
    int *s_first = s_mem, *s_n = s_mem + E;                // first entry of every list's stretch, and their number
    __shared__ unsigned s_row[kBlockTokens * kTokenRows];
    __shared__ int s_cnt[kBlockTokens];
    __shared__ int s_odd;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if ((int)blockIdx.x >= n_tb) {
        const long long n_rows = (long long)E * C;
        const unsigned n_waves = (gridDim.x - n_tb) * (THREADS / 64), w = (blockIdx.x - n_tb) * (THREADS / 64) + wv;
        // row `lane` of a turn's 64: one of every n_waves, moved on by 0.617 n_waves each time
        const unsigned mine = lane * n_waves + (w + lane * (unsigned)((unsigned long long)n_waves * 158 >> 8)) % n_waves;
        for (long long r0 = 0; r0 < n_rows; r0 += 64ll * n_waves) {
            const long long r = r0 + mine;
            bool pad = false;
            if (r < n_rows) {
                const int j = (int)(r / C), s = (int)(r - (long long)j * C);
                pad = s >= offsets[j + 1] - offsets[j];
            }
            for (unsigned long long m = __ballot(pad); m; m &= m - 1) {
                u32x4 *dst = out + (r0 + (unsigned)__builtin_amdgcn_readlane((int)mine, __ffsll((long long)m) - 1)) * vec_per_row;
                for (int c = lane; c < vec_per_row; c += 64) put<NT>(u32x4{0u, 0u, 0u, 0u}, dst + c);
            }
        }
        return;
    }
    const int t0 = blockIdx.x * tb, t1 = t0 + tb;
    if (tid < kBlockTokens) s_cnt[tid] = 0;
    if (tid == 0) s_odd = 0;
    __syncthreads();
    for (int j = tid; j < E; j += THREADS) {
        const int o0 = offsets[j];
        int cnt = offsets[j + 1] - o0;
        cnt = cnt < 0 ? 0 : cnt < C ? cnt : C;
        auto sample_at = [&](int i) { return i < 0 ? -1 : (int)((unsigned long long)cnt * i / kListSamples); };
        int v[kListSamples];
#pragma unroll
        for (int i = 0; i < kListSamples; ++i) v[i] = cnt > 0 ? disp_token[o0 + sample_at(i)] : 0;
        bool ascends = true;
        int na = 0, nb = 0;                               // samples below either end
#pragma unroll
        for (int i = 0; i < kListSamples; ++i) {
            if (i > 0 && sample_at(i) > sample_at(i - 1) && v[i] <= v[i - 1]) ascends = false;
            na += v[i] < t0 ? 1 : 0;
            nb += v[i] < t1 ? 1 : 0;
        }
        // both ends at once: the loads of a step are independent
        int a = cnt > 0 ? sample_at(na - 1) + 1 : 0, an = sample_at(na) - a, b = cnt > 0 ? sample_at(nb - 1) + 1 : 0, bn = sample_at(nb) - b;
        if (!ascends) an = bn = 0;
        while (an > 0 || bn > 0) {
            const int ah = an >> 1, bh = bn >> 1;
            const int va = an > 0 ? disp_token[o0 + a + ah] : 0, vb = bn > 0 ? disp_token[o0 + b + bh] : 0;
            if (an > 0) {
                if (va < t0) { a += ah + 1; an -= ah + 1; } else an = ah;
            }
            if (bn > 0) {
                if (vb < t1) { b += bh + 1; bn -= bh + 1; } else bn = bh;
            }
        }
        int lo = blockIdx.x == 0 ? 0 : a, hi = (int)blockIdx.x == n_tb - 1 ? cnt : b;
        if (!ascends) {
            lo = (int)((long long)cnt * blockIdx.x / n_tb);
            hi = (int)((long long)cnt * (blockIdx.x + 1) / n_tb);
            s_odd = 1;
        }
        s_first[j] = lo;
        s_n[j] = hi - lo;
        if (!ascends) continue;
        for (int s = lo; s < hi; ++s) {
            const int t = disp_token[o0 + s] - t0;
            if (t < 0 || t >= tb || t0 + t >= T) {
                s_odd = 1;
                break;
            }
            const int at = atomicAdd(&s_cnt[t], 1);
            if (at >= kTokenRows) {
                s_odd = 1;
                break;
            }
            s_row[t * kTokenRows + at] = (unsigned)j * (unsigned)C + (unsigned)s;
        }
    }
    __syncthreads();
    if (s_odd) {
        // the i-th rows of 64 stretches together, in turn to the wavefronts
        for (int j0 = 0, turn = wv; j0 < E; j0 += 64) {
            const int j = j0 + lane, n = j < E ? s_n[j] : 0, first = j < E ? s_first[j] : 0, at = j < E ? offsets[j] + first : 0;
            for (int i = 0; __any(i < n); ++i) {
                int tok = i < n ? disp_token[at + i] : 0;
                tok = tok >= 0 && tok < T ? tok : 0;
                for (unsigned long long m = __ballot(i < n); m; m &= m - 1, ++turn) {
                    if (turn % (THREADS / 64)) continue;
                    const int l = __ffsll((long long)m) - 1;
                    const u32x4 *src = x + (size_t)__builtin_amdgcn_readlane(tok, l) * vec_per_row;
                    u32x4 *dst = out + ((size_t)(j0 + l) * C + __builtin_amdgcn_readlane(first, l) + i) * vec_per_row;
                    for (int c = lane; c < vec_per_row; c += 64) put<NT>(src[c], dst + c);
                }
            }
        }
        return;
    }
    for (int t = wv; t < tb; t += THREADS / 64) {
        const int n = s_cnt[t];
        if (n == 0) continue;
        const unsigned mine = lane < n ? s_row[t * kTokenRows + lane] : 0u;
        const u32x4 *src = x + (size_t)(t0 + t) * vec_per_row;
        for (int c0 = lane; c0 < vec_per_row; c0 += 256) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = c0 + 64 * u < vec_per_row ? get<LAST>(src + c0 + 64 * u) : u32x4{0u, 0u, 0u, 0u};
            for (int i = 0; i < n; ++i) {
                u32x4 *dst = out + (size_t)(unsigned)__builtin_amdgcn_readlane((int)mine, i) * vec_per_row;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c0 + 64 * u < vec_per_row) put<NT>(v[u], dst + c0 + 64 * u);
            }
        }
    }
}

// Rows that are not a whole number of 16-byte vectors (or misaligned buffers): element by element.
template <typename TElem>
__global__ __launch_bounds__(256) void k_dispatch_tokens_elem(const TElem *__restrict__ x,
                                                              const int32_t *__restrict__ offsets,
                                                              const int32_t *__restrict__ disp_token, int T, int d,
                                                              int E, int C, TElem *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const long long n_rows = (long long)E * C;
    const long long wave0 = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const long long n_waves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long r = wave0; r < n_rows; r += n_waves) {
        const int j = (int)(r / C), s = (int)(r - (long long)j * C);
        const int o0 = offsets[j], cnt = offsets[j + 1] - o0;
        TElem *dst = out + r * d;
        if (s < cnt) {
            const int tok = disp_token[o0 + s];
            const TElem *src = x + (size_t)(tok >= 0 && tok < T ? tok : 0) * d;
            for (int c = lane; c < d; c += 64) dst[c] = src[c];
        } else {
            for (int c = lane; c < d; c += 64) dst[c] = (TElem)0;
        }
    }
}

__device__ __forceinline__ float bf16_to_f32(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

// A wavefront takes PIECES kilobytes of a token's row, its neighbours the next ones, and ends: the k gate-weighted pieces are accumulated
// in fp32, slot by slot, and written as fp32.  The indices of the slots (64 at most) are read by one lane each, and kCombineLoads pieces
// of them are on their way together.  A lane takes four columns at a time, its neighbours the next ones, so that a store is whole lines of
// fp32 (eight columns a lane, in one load of bf16, made every line of two stores: layers of 16384 tokens of 2048 to 8 of 64 experts 364 -> 357 us,
// 32768 612 -> 606, 65536 to 8 of 128 1246 -> 1236).  Bound by HBM beyond the last cache, which takes short-lived wavefronts in the order of the addresses
// best (a plain fill: 6.8 TB/s with 16 bytes a thread and no loop, 4.0 to 5.6 with loops over a fixed grid): 65536 tokens of 2048 from 8 of
// 128 experts 460 us (5.8 TB/s), 496 with whole rows and a loop over the tokens in every wavefront; 44032 of 1024 from 2 of 64 75 to 69.
constexpr int kCombineLoads = 4;

// AHEAD: the pieces of those slots are really on their way together.  A load under a condition is waited for before the next one (its register
// could hold something else), so a slot that is empty then reads what the one before it did, and a lane beyond the row its end; neither is used.
// QUADS: a lane's columns by four, PIECES kilobytes of the row, or half of one: rows of bf16 that are no longer.
template <bool BF16, bool NT, int QUADS, bool AHEAD>
__global__ __launch_bounds__(256) void k_combine(const void *__restrict__ buf_, const int32_t *__restrict__ assign,
                                                 const int32_t *__restrict__ token_pos,
                                                 const float *__restrict__ gates, int T, int d, int E, int k, int C,
                                                 int parts, float *__restrict__ y)
{
    using V = std::conditional_t<BF16, u32x2, u32x4>;        // four elements
    constexpr int PIECES = QUADS <= 2 && BF16 ? 1 : BF16 ? QUADS / 2 : QUADS, SLOTS = kCombineLoads / PIECES;
    const V *buf = (const V *)buf_;
    const int lane = threadIdx.x & 63, quads_per_row = d >> 2;
    const unsigned item = blockIdx.x * 4u + (threadIdx.x >> 6), i = __builtin_amdgcn_readfirstlane(item / (unsigned)parts);
    if (i >= (unsigned)T) return;
    const int c = (int)(item - i * (unsigned)parts) * (64 * QUADS) + lane;
    int e = -1, pos = 0;
    float g = 0.f;
    if (lane < k) {
        const size_t at = (size_t)i * k + lane;
        e = assign[at];
        pos = token_pos[at];
        g = gates[at];
        // an empty slot, or a place outside the expert's buffer (an assignment made with another capacity)
        if (e >= E || pos < 0 || pos >= C) e = -1;
    }
    f32x4 acc[QUADS];
#pragma unroll
    for (int u = 0; u < QUADS; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    int at[QUADS];
#pragma unroll
    for (int u = 0; u < QUADS; ++u) at[u] = c + 64 * u < quads_per_row ? c + 64 * u : quads_per_row - 1;
    const V *row = buf;
    for (int s = 0; s < k; s += SLOTS) {
        V vals[SLOTS][QUADS];
        bool have[SLOTS];
#pragma unroll
        for (int z = 0; z < SLOTS; ++z) {
            if (AHEAD) {
                const int sl = s + z < k ? s + z : k - 1, ea = __builtin_amdgcn_readlane(e, sl);
                have[z] = s + z < k && ea >= 0;
                row = ea >= 0 ? buf + ((size_t)ea * C + __builtin_amdgcn_readlane(pos, sl)) * quads_per_row : row;
#pragma unroll
                for (int u = 0; u < QUADS; ++u) vals[z][u] = get<NT>(row + at[u]);
                continue;
            }
            const int es = s + z < k ? __builtin_amdgcn_readlane(e, s + z) : -1;
            have[z] = es >= 0;
            if (!have[z]) continue;
            const V *src = buf + ((size_t)es * C + __builtin_amdgcn_readlane(pos, s + z)) * quads_per_row;
#pragma unroll
            for (int u = 0; u < QUADS; ++u) vals[z][u] = get<NT>(src + at[u]);
        }
#pragma unroll
        for (int z = 0; z < SLOTS; ++z) {
            if (!have[z]) continue;
            const float gs = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g), s + z));
#pragma unroll
            for (int u = 0; u < QUADS; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    float x;
                    if constexpr (BF16) x = __uint_as_float(w % 2 ? vals[z][u][w / 2] & 0xffff0000u : vals[z][u][w / 2] << 16);
                    else x = __uint_as_float(vals[z][u][w]);
                    acc[u][w] = fmaf(gs, x, acc[u][w]);
                }
        }
    }
    f32x4 *dst = (f32x4 *)(y + (size_t)i * d);
#pragma unroll
    for (int u = 0; u < QUADS; ++u)
        if (c + 64 * u < quads_per_row) put<NT>(acc[u], dst + c + 64 * u);
}

template <bool BF16>
__global__ __launch_bounds__(256) void k_combine_elem(const void *__restrict__ buf_, const int32_t *__restrict__ assign,
                                                      const int32_t *__restrict__ token_pos,
                                                      const float *__restrict__ gates, int T, int d, int E, int k,
                                                      int C, float *__restrict__ y)
{
    const size_t n = (size_t)T * d;
    for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < n; o += (size_t)gridDim.x * blockDim.x) {
        const size_t i = o / d, c = o - i * d;
        float acc = 0.f;
        for (int s = 0; s < k; ++s) {
            const int e = assign[i * k + s];
            if (e < 0) continue;
            const int pos = token_pos[i * k + s];
            if (e >= E || pos < 0 || pos >= C) continue;      // outside the expert's buffer: never read
            const size_t at = ((size_t)e * C + pos) * d + c;
            const float v = BF16 ? bf16_to_f32(((const unsigned short *)buf_)[at]) : ((const float *)buf_)[at];
            acc = fmaf(gates[i * k + s], v, acc);
        }
        y[o] = acc;
    }
}

}  // namespace

// What does not fit the 256 MiB of the last cache goes past it (non-temporal).  Rows out: buffers as large as that, or, with the rows they are
// read from and the results that come back, a third more: what is written then leaves the cache before it is read.  Buffers of 1024
// columns to 64 experts, the rerouting's layers, past the cache against through it: top-2 of 160 MiB (400 in all) 220 against 249 us, 200 (500)
// 258 and 280, top-4 of 200 (350) 217 and 231, top-6 of 240 (360) 235 and 243, fp32 top-1 of 120 (360) 226 and 236; but top-2 of 120 (300)
// 193 and 189, top-8 of 200 (275) 205 and 193 and of 240 (330) 224 and 225, 10007 of 1000 in fp32 to 6 of 96 (328) 318 and 312.
// So it is with two matrix products between rows out and rows back, which could find buffers of that size in the cache: what the first one
// loses, the rest of the layer gains.  Layers with experts of 256 to 1024 inner columns, past the cache against through it: 44032 of 1024 to 2 of 64 by rerouting 484
// and 490 us, 52000 586 and 600, 60000 of 768 to 2 of 32 597 and 616, of 512 to 4 of 64 640 and 661, 28000 of 1024 to 4 554 and 569, 20480 of 2048 to 3
// 776 and 787, 26000 to 2 604 and 613, 20000 of 1536 to 4 579 and 592, fp32 30000 of 1024 to 2 842 and 852; 12288 of 2048 to 5, 14336 to 4, 36000 of 1024
// in fp32 to 1 and 12000 to 5 within 1 %.  (Rows out and the first product alone, of x that the cache holds: 1 to 5 % slower.)
// Rows back: buffers and results of half of it (top-2 of 160 MiB in all 153 against 162 us, of 240 189 and 201, top-4 of 180 161 and 166,
// top-8 of 250 193 and 200; of 150 and less the same; with two matrix products before them and a sum that reads the results behind them 13 layers of
// 128 to 250 MiB take 0.98 to 1.005 of the time: 24000 of 1024 to 2 of 64 417 and 422, 44032 of 512 425 and 435, 10007 of 1000 in fp32 to 4 of 96 691 and 687).
static bool beyond_caches(size_t bytes) { return bytes >= (size_t)256 << 20; }
static bool out_past_caches(size_t x_bytes, size_t buf_bytes, size_t y_bytes)
{
    return beyond_caches(buf_bytes) || x_bytes + buf_bytes + y_bytes >= (size_t)336 << 20;
}
static bool back_past_caches(size_t bytes) { return bytes >= (size_t)128 << 20; }

int32_t dispatch_tokens_run(const void *x, int dtype, const int32_t *offsets, const int32_t *disp_token, int T, int d,
                            int E, int C, void *out, hipStream_t s)
{
    const int eb = dtype == MAXSCORE_DTYPE_BF16 ? 2 : 4;
    const long long n_rows = (long long)E * C;
    long long grid = (n_rows + 3) / 4;
    if (grid > 256 * 16) grid = 256 * 16;        // 16 workgroups of 4 wavefronts per compute unit, grid-stride
    if (grid < 1) grid = 1;
    const bool vec = ((size_t)d * eb) % 16 == 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)out % 16) == 0;
    // Blocks of tokens from 4096 tokens on (four blocks per compute unit; smaller batches are bound by latency, and their
    // rows of x stay in the caches), as long as the lists to search are not many more than the rows a block moves.
    // Where neither x nor the buffers fit the last cache, sixteen wavefronts to a workgroup and half as many tokens: fewer rows of x and
    // places of the lists are in use at a time.  In a layer, tight and with a quarter more room: 65536 tokens of 2048 to 8 of 128 experts
    // 512 -> 492 us, to 2 of 32 157 -> 138 and 187 -> 169, 33000 of 4096 to 4 of 32 262 -> 241 and 304 -> 285.  Of 128 to 192 MiB of x it
    // depends: 65536 of 1536 to 8 of 128 370 -> 340, to 4 of 64 167 -> 171.  A single expert a token: 117 -> 106 to 128, 92 -> 92 to 8.
    const size_t x_bytes = (size_t)T * d * eb, buf_bytes = (size_t)n_rows * d * eb;
    const bool nt = out_past_caches(x_bytes, buf_bytes, (size_t)T * d * 4);
    const bool wide = beyond_caches(buf_bytes) && T >= 16 * 1024 && E <= 128 * 16 && beyond_caches(x_bytes);
    const int tb = wide ? 16 : T >= 32 * 1024 ? 32 : T >= 16 * 1024 ? 16 : T >= 8 * 1024 ? 8 : 4;
    if (vec && T >= 4096 && E <= 128 * tb && E <= kListMaxE && n_rows < (1ll << 32)) {
        const int n_tb = (T + tb - 1) / tb, n_pad = (int)std::min<long long>((n_rows + 255) / 256, 1024);
#define MS_BLOCKED(NN, LL, TT)                                                                                              \
    hipLaunchKernelGGL((k_dispatch_tokens_blocked<NN, LL, TT>), dim3(n_tb + n_pad), dim3(TT), sizeof(int) * 2 * E, s, (const u32x4 *)x, \
                       offsets, disp_token, T, E, C, (int)((size_t)d * eb / 16), tb, n_tb, (u32x4 *)out)
        // Rows of x of 100 MiB and more are read past the cache (those that the projection has left in it are found there all the same; by themselves, the
        // same x again and again, they come from memory every time: 44032 tokens of 2048 to 2 of 64 86 and 119 us): layers with 64 and 96
        // MiB of them the same, 112 MiB (28672 tokens of 2048 to 4 of 128) 440 -> 421 us, 128 (65536 of 1024 to 4 of 64) 454 -> 412, 160
        // (40960 of 2048 to 8 of 64) 770 -> 731, 224 406 -> 403, 256 (65536 of 2048 to 8 of 128) 1234 -> 1207; 32768 with room to spare 606 -> 582.
        // (The projection's loads past the cache: 1234 -> 1226 there, but with both 1226, and 32768 606 -> 635.)
        const bool last = x_bytes >= (size_t)100 << 20;
        if (wide) MS_BLOCKED(true, true, 1024);
        else if (nt && last) MS_BLOCKED(true, true, 256);
        else if (nt) MS_BLOCKED(true, false, 256);
        else MS_BLOCKED(false, false, 256);
#undef MS_BLOCKED
    } else if (vec) {
        hipLaunchKernelGGL(k_dispatch_tokens, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4 *)x, offsets,
                           disp_token, T, E, C, (int)((size_t)d * eb / 16), (u32x4 *)out);
    } else if (eb == 2) {
        hipLaunchKernelGGL((k_dispatch_tokens_elem<unsigned short>), dim3((unsigned)grid), dim3(256), 0, s,
                           (const unsigned short *)x, offsets, disp_token, T, d, E, C, (unsigned short *)out);
    } else {
        hipLaunchKernelGGL((k_dispatch_tokens_elem<unsigned int>), dim3((unsigned)grid), dim3(256), 0, s,
                           (const unsigned int *)x, offsets, disp_token, T, d, E, C, (unsigned int *)out);
    }
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

int32_t combine_run(const void *buf, int dtype, const int32_t *assign, const int32_t *token_pos, const float *gates,
                    int T, int d, int E, int k, int C, float *y, hipStream_t s)
{
    const int eb = dtype == MAXSCORE_DTYPE_BF16 ? 2 : 4;
    const bool vec = ((size_t)d * eb) % 16 == 0 && ((uintptr_t)buf % 16) == 0 && ((uintptr_t)y % 16) == 0;
    if (vec) {
        const int vpr = (int)((size_t)d * eb / 16);
        const size_t traffic = (size_t)E * C * d * eb + (size_t)T * d * 4;
        const bool nt = back_past_caches(traffic);
        // Two kilobytes of a row to a wavefront where the rows come from the last cache: there a second wavefront on the same row costs more
        // than it brings (4361 tokens of 552 from 4 of 64 experts 7.2 us, 9.1 with one; 10007 of 1000 in fp32 from 6 of 96 56 and 59; 7988 of
        // 832 from 6 of 32 15.8 and 17.4).  Below some 24 MiB in all, or ten wavefronts to a compute unit, the chip is not full with half as
        // many (1024 of 1024 from 8 of 64 5.4 and 5.0), beyond some 448 MiB memory decides as above, and with one or two slots the result
        // does, which is written either way.  With three or four an odd number of pieces leaves too many lanes idle (21892 of 1536 from 4 of 32
        // 75 and 70).  Up to the same 448 MiB the loads of several slots go ahead of their use (10007 of 1000 in fp32 48.0 -> 43.2, 32768 of 1024
        // from 4 of 32 72.8 -> 65.8, 21892 of 1536 70.7 -> 65.3); from memory the rows come better one after the other (16384 of 2048 from 8
        // of 64 118 us, 122 with loads ahead, 65536 of 2048 470 and 473), and with two slots the rest would be read for nothing (4096 of 1024
        // 8.4 and 8.9).
        const int pieces = (vpr + 63) / 64;
        const bool ahead = k > 2 && traffic < (size_t)448 << 20;
        const bool two = ahead && vpr > 64 && (k > 4 || pieces % 2 == 0) && (long long)T * ((pieces + 1) / 2) >= 2560 &&
                         traffic >= (size_t)24 << 20;
        // Rows of bf16 of up to 256 columns: a lane takes four of them, not eight of which four are none (44032 of 256 from 8 of 64 experts
        // from memory 78.0 -> 75.5 us, of 64 49.4 -> 46.0, 16384 of 128 from 4 15.7 -> 14.8).
        const bool narrow = eb == 2 && vpr <= 32;
        const int piece = two ? 128 : 64, parts = (vpr + piece - 1) / piece;
        const int most = std::max(1, (1 << 24) / parts);            // tokens a launch (its threads are counted in 32 bits)
        for (int i0 = 0; i0 < T; i0 += most) {
            const int n = std::min(most, T - i0);
            const size_t at = (size_t)i0 * k;
#define MS_COMBINE(BB, NN, QQ, AA)                                                                                                   \
    hipLaunchKernelGGL((k_combine<BB, NN, QQ, AA>), dim3((unsigned)(((size_t)n * parts + 3) / 4)), dim3(256), 0, s, buf, assign + at, \
                       token_pos + at, gates + at, n, d, E, k, C, parts, y + (size_t)i0 * d)
#define MS_COMBINE_P(BB, NN)                         \
    do {                                             \
        constexpr int q = BB ? 2 : 1;                \
        if (two) MS_COMBINE(BB, NN, 2 * q, true);    \
        else if (BB && narrow && ahead) MS_COMBINE(BB, NN, 1, true); \
        else if (BB && narrow) MS_COMBINE(BB, NN, 1, false); \
        else if (ahead) MS_COMBINE(BB, NN, q, true); \
        else MS_COMBINE(BB, NN, q, false);           \
    } while (0)
            if (eb == 2) {
                if (nt) MS_COMBINE_P(true, true);
                else MS_COMBINE_P(true, false);
            } else if (nt) MS_COMBINE_P(false, true);
            else MS_COMBINE_P(false, false);
#undef MS_COMBINE_P
#undef MS_COMBINE
        }
    } else {
        size_t n = (size_t)T * d;
        long long grid = (long long)((n + 255) / 256);
        if (grid > 256 * 32) grid = 256 * 32;
        if (grid < 1) grid = 1;
        if (eb == 2)
            hipLaunchKernelGGL((k_combine_elem<true>), dim3((unsigned)grid), dim3(256), 0, s, buf, assign, token_pos,
                               gates, T, d, E, k, C, y);
        else
            hipLaunchKernelGGL((k_combine_elem<false>), dim3((unsigned)grid), dim3(256), 0, s, buf, assign,
                               token_pos, gates, T, d, E, k, C, y);
    }
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

}  // namespace maxscore
