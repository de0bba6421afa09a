// Algorithm 1 (Section 3.2) with its last step done the paper's way: Sinkhorn on the residual problem.
// The paper names the algorithm only; regulariser, iteration count and rounding are this library's reading:
//   top-1 per token (ties to the lower expert id), residual capacities caps_j = max(0, C - load_j), residual
//   affinities a' = scores with the top-1 entry set to 0;
//   K_ij = exp((a'_ij - max_j a'_ij) / tau) on experts with caps_j > 0, else 0 (the row shift is absorbed by u);
//   column targets m_j = caps_j * T / sum(caps);  v = 1;  n_iter times: u_i = 1 / sum_j K_ij v_j,
//   v_j = m_j / sum_i K_ij u_i;  plan_ij = u_i K_ij v_j;  second expert = arg-max_j plan_ij (ties to the lower
//   id; -1 when the row is all zero).
// Three ways to do it, by size; column sums are added in a fixed order everywhere, in double beyond one to four rows where one
// workgroup does it all, from the first on with eight lanes to a row; row sums are trees over the columns:
//   small    up to 65536 scores of up to 16 experts, half as many of up to 64: the whole call is one workgroup that keeps
//            K in registers, a thread owns whole rows.  An iteration takes 1.8 us (two barriers, 300 instructions of every
//            wavefront), two launches each 8.  The limit is that of the registers: 1024 threads of 64 entries, 512 beyond 16 columns.
//   medium   up to 64 experts: eight lanes per row, K recomputed from the scores; one launch per iteration, whose
//            workgroups begin by adding up the column sums of the iteration before
//   large    one wavefront per row, lane l holds experts l, l+64, ...; rows and columns are launches of their own
// 20 iterations, before and after the first two ways: 4096 tokens of 16 experts 228 and 67 us (4097, the first the medium way
// takes, 116), 16384 of 64 350 and 178 us.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "host_words.h"
#include "sums.h"

namespace maxscore {
namespace {

constexpr int kSkBlocksMax = 1024;

__device__ inline float sk_wave_max(float v)
{
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

__device__ inline float sk_wave_sum(float v)
{
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// first lane-major position holding the row maximum: expert with the largest value, ties to the lower id
template <int EPL>
__device__ inline int sk_argmax(const float (&x)[EPL], const bool (&in)[EPL], float mx)
{
    int e = -1;
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        const unsigned long long b = __ballot(in[c] && x[c] == mx);
        if (e < 0 && b) e = 64 * c + __ffsll((long long)b) - 1;
    }
    return e;
}

constexpr int kSkCopies = 8;                 // partial counts of the top-1 choices, one per chiplet

__global__ __launch_bounds__(1024) void k_sk_zero(int *counts)
{
    for (int i = threadIdx.x; i < kSkCopies * kMaxE; i += 1024) counts[i] = 0;
}

template <int EPL>
__global__ __launch_bounds__(256) void k_sk_top1(const float *__restrict__ scores, int T, int E,
                                                 int32_t *__restrict__ top1, int *__restrict__ counts)
{
    __shared__ int s_cnt[kMaxE];
    for (int e = threadIdx.x; e < E; e += 256) s_cnt[e] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    for (int row = wave; row < T; row += n_waves) {
        float x[EPL];
        bool in[EPL];
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const int e = lane + 64 * c;
            in[c] = e < E;
            x[c] = in[c] ? scores[(size_t)row * E + e] : -INFINITY;
            mx = fmaxf(mx, x[c]);
        }
        mx = sk_wave_max(mx);
        const int e = sk_argmax<EPL>(x, in, mx);
        if (lane == 0) {
            top1[row] = e;
            if (e >= 0) atomicAdd(&s_cnt[e], 1);
        }
    }
    __syncthreads();
    int *c = counts + (blockIdx.x % kSkCopies) * kMaxE;
    for (int e = threadIdx.x; e < E; e += 256)
        if (s_cnt[e]) atomicAdd(c + e, s_cnt[e]);
}

// caps, column targets and the starting v from the top-1 counts (one workgroup; thread j: expert j)
__device__ __forceinline__ void sk_targets(int count, int T, int E, int C, int &cap, float &target)
{
    __shared__ long long s_w[16];
    const int j = threadIdx.x;
    cap = 0;
    if (j < E) {
        const int left = C - count;
        cap = left > 0 ? left : 0;
    }
    long long sum = cap;
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if ((j & 63) == 0) s_w[j >> 6] = sum;
    __syncthreads();
    long long tot = 0;
    for (int w = 0; w < (int)blockDim.x >> 6; ++w) tot += s_w[w];
    target = tot > 0 ? (float)((double)cap * (double)T / (double)tot) : 0.f;
}

__global__ __launch_bounds__(1024) void k_sk_init(const int *__restrict__ counts, int T, int E, int C,
                                                  int32_t *__restrict__ caps, float *__restrict__ targets,
                                                  float *__restrict__ v)
{
    const int j = threadIdx.x;
    int n = 0, cap;
    float target;
    for (int c = 0; c < kSkCopies; ++c) n += j < E ? counts[c * kMaxE + j] : 0;
    sk_targets(n, T, E, C, cap, target);
    if (j < E) {
        if (caps) tell_host(caps + j, cap);
        targets[j] = target;
        v[j] = 1.f;
    }
}

__device__ __forceinline__ float sk_column(double sum, float m)
{
    return m > 0.f ? (float)((double)m / (sum > 1e-300 ? sum : 1e-300)) : 0.f;
}

// ---- small: everything in one workgroup ----

// Column sums over a wavefront: lanes exchange halves of their columns until every lane holds the sum of one of them (the
// last steps of EP < 64 add equal columns).  A thread comes with the sums of its own 64 / EP rows.  Up to four rows are added in
// fp32, sums of four rows in double; what lanes exchange for the first of these additions is still an fp32 number.
// (Values move between lanes by swaps and lane moves: shuffles through LDS were a third of an iteration.)
template <int OFF>
__device__ __forceinline__ int sk_move(int v)            // from the lane OFF away, within sixteen lanes
{
    static_assert(OFF <= 8, "within a row of lanes");
    if constexpr (OFF == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);                   // row_ror:8
    else if constexpr (OFF == 4) {
        const int from_above = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);                // row_shl:4, lanes 0-3 and 8-11
        return __builtin_amdgcn_update_dpp(from_above, v, 0x114, 0xf, 0xa, false);                       // row_shr:4, the others
    } else return __builtin_amdgcn_mov_dpp(v, OFF == 2 ? 0x4E : 0xB1, 0xf, 0xf, true);                   // quad_perm
}
template <int OFF>
__device__ __forceinline__ float sk_move(float v) { return __int_as_float(sk_move<OFF>(__float_as_int(v))); }
template <int OFF>
__device__ __forceinline__ double sk_move(double v)
{
    return __hiloint2double(sk_move<OFF>(__double2hiint(v)), sk_move<OFF>(__double2loint(v)));
}
// a of the lanes without bit OFF stays, that of the others goes to the lane OFF below; b the other way round
template <int OFF>
__device__ __forceinline__ void sk_swap(unsigned &a, unsigned &b)
{
    static_assert(OFF == 16 || OFF == 32, "rows of lanes");
    if constexpr (OFF == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <int OFF>
__device__ __forceinline__ void sk_swap(float &a, float &b)
{
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    sk_swap<OFF>(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int OFF>
__device__ __forceinline__ void sk_swap(double &a, double &b)
{
    unsigned x = (unsigned)__double2loint(a), y = (unsigned)__double2loint(b), z = (unsigned)__double2hiint(a), w = (unsigned)__double2hiint(b);
    sk_swap<OFF>(x, y);
    sk_swap<OFF>(z, w);
    a = __hiloint2double((int)z, (int)x);
    b = __hiloint2double((int)w, (int)y);
}

template <int HALF, int OFF, int N, typename V, typename W>
__device__ __forceinline__ void sk_exchange(const V (&f)[N], W (&sum)[HALF], int lane, int &column)
{
    const bool up = (lane & OFF) != 0;
    column |= up ? HALF : 0;
#pragma unroll
    for (int c = 0; c < HALF; ++c) {
        if constexpr (OFF >= 16) {
            V a = f[c], b = f[c + HALF];
            sk_swap<OFF>(a, b);
            sum[c] = (W)a + (W)b;
        } else {
            const V give = up ? f[c] : f[c + HALF], keep = up ? f[c + HALF] : f[c];
            sum[c] = (W)keep + (W)sk_move<OFF>(give);
        }
    }
}

template <int EP, int OFF, typename V>
__device__ __forceinline__ double sk_reduce_scatter(const V (&f)[EP], int lane, int &column)
{
    if constexpr (EP > 16) {                    // (one row so far with 64 columns, two with 32)
        V h[EP / 2];
        sk_exchange<EP / 2, OFF>(f, h, lane, column);
        return sk_reduce_scatter<EP / 2, OFF / 2>(h, lane, column);
    } else if constexpr (EP > 1) {
        double h[EP / 2];
        sk_exchange<EP / 2, OFF>(f, h, lane, column);
        return sk_reduce_scatter<EP / 2, OFF / 2>(h, lane, column);
    } else {
        double d = f[0];
        if constexpr (OFF >= 4) d += sk_move<4>(d);
        if constexpr (OFF >= 2) d += sk_move<2>(d);
        if constexpr (OFF >= 1) d += sk_move<1>(d);
        static_assert(OFF <= 4, "eight columns at least");
        return d;
    }
}

// 1 / x: the hardware's reciprocal and a Newton step, three instructions instead of ten.  1 - x * r is exact in the fused step, so that what is left
// of the reciprocal's error e is e^2, below the rounding of the last addition: the same bits as the division for every one of the 2^23 mantissas
// (compared at eleven exponents from 2^-99 to 2^91).
__device__ __forceinline__ float sk_reciprocal(float x)
{
    const float y = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, y, 1.f), y, y);
}

// Threads: as many as there are rows, up to a wavefront a SIMD; then as many as have their 64 / EP rows each, which wavefronts that share a SIMD
// would take in turn anyway, and a sum over the lanes for each.  Scores, choice and gates with a thread to a row, up to the 1024 there can be, and
// so: 700 tokens of 16 experts 60.4 -> 56.2 us, 1000 70.2 -> 57.7, 2048 78.2 -> 64.0, 3000 85.3 -> 76.1, 2048 of 8 72.6 -> 55.6, 300 of 16 and of 32 the
// same.
constexpr int kSkFewThreads = 256;
template <int EP>
constexpr int kSkSmallThreads = EP <= 16 ? 1024 : 512;

// GROUP: rows whose shares of a column sum are added in fp32 before they are widened: one up to 1024 tokens, two up to 3072 and four beyond (of 32
// experts one up to 512, else two), no more than with a thread to a row.  With four throughout 700 tokens of 16 experts took 52.9 us, 1000 54.3, 2048 62.0,
// and the plan's error against 64 bits went from 6.37e-8 to 6.45e-8 rms at 1000 (6.37e-8 so).
template <int EP, int GROUP>
__global__ __launch_bounds__(GROUP == 1 && EP < 64 ? kSkFewThreads : kSkSmallThreads<EP>) void k_sk_small(const float *__restrict__ scores, int T, int E, int C, float inv_tau,
                                                   int n_iter, int32_t *__restrict__ assign, float *__restrict__ plan,
                                                   int32_t *__restrict__ caps)          // (of the host, or null)
{
    constexpr int RR = 64 / EP;                 // rows per thread: r * nt + tid
    using Acc = std::conditional_t<(RR > GROUP), double, float>;
    static_assert(RR % GROUP == 0, "whole groups");
    __shared__ int s_cnt[EP];
    __shared__ float s_target[EP];
    __shared__ __attribute__((aligned(16))) float s_v[EP];
    __shared__ double s_red[16 * EP];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nt = blockDim.x, nw = nt >> 6;
    const bool vec = (E & 3) == 0 && ((size_t)scores & 15) == 0;
    if (tid < EP) s_cnt[tid] = 0;
    for (int i = tid; i < 16 * EP; i += nt) s_red[i] = 0.0;
    __syncthreads();
    float x[RR][EP], mx[RR], u[RR];
    int t1[RR];
#pragma unroll
    for (int r = 0; r < RR; ++r) {
        const int row = r * nt + tid;
        const float *p = scores + (size_t)(row < T ? row : 0) * E;
        if (vec) {
#pragma unroll
            for (int c = 0; c < EP; c += 4) {
                const float4 f = c < E ? *(const float4 *)(p + c) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                x[r][c] = f.x; x[r][c + 1] = f.y; x[r][c + 2] = f.z; x[r][c + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < EP; ++c) x[r][c] = c < E ? p[c] : -INFINITY;
        }
        float m = -INFINITY;
#pragma unroll
        for (int c = 0; c < EP; ++c) m = fmaxf(m, x[r][c]);
        t1[r] = -1;
#pragma unroll
        for (int c = EP - 1; c >= 0; --c)
            if (c < E && x[r][c] == m) t1[r] = c;
        if (row < T && t1[r] >= 0) atomicAdd(&s_cnt[t1[r]], 1);
        mx[r] = -INFINITY;
        u[r] = 1.f;
#pragma unroll
        for (int c = 0; c < EP; ++c) {
            if (c == t1[r]) x[r][c] = 0.f;
            if (c < E) mx[r] = fmaxf(mx[r], x[r][c]);
        }
    }
    __syncthreads();
    int cap;
    float target;
    sk_targets(tid < E ? s_cnt[tid] : 0, T, E, C, cap, target);
    if (tid < EP) {
        s_target[tid] = tid < E ? target : 0.f;
        s_v[tid] = tid < E && target > 0.f ? 1.f : 0.f;
        if (tid < E && caps) tell_host(caps + tid, cap);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int c = 0; c < EP; ++c) x[r][c] = s_target[c] > 0.f ? expf((x[r][c] - mx[r]) * inv_tau) : 0.f;     // K_ij
    const bool whole = (RR - 1) * nt + __builtin_amdgcn_readfirstlane(tid) < T;      // the wavefront has rows of every kind
    for (int it = 0; it < n_iter; ++it) {
        if (whole) {
            // (straight code, without the divisions: scores, choice and gates of 4096 tokens of 16 experts 84.6 -> 82.4 us)
            float z[RR], lo = 1.f, hi = 1.f;
#pragma unroll
            for (int r = 0; r < RR; ++r) z[r] = tree_dot<EP>(x[r], s_v);
#pragma unroll
            for (int r = 0; r < RR; ++r) {
                u[r] = sk_reciprocal(z[r]);
                lo = fminf(lo, z[r]);
                hi = fmaxf(hi, z[r]);
            }
            if (__builtin_expect(!(lo > 1e-30f && hi < 1e30f), 0)) {      // near the ends of the range
#pragma unroll
                for (int r = 0; r < RR; ++r) u[r] = 1.f / z[r];
            }
            u[RR - 1] = (RR - 1) * nt + tid < T ? u[RR - 1] : 0.f;
        } else {
#pragma unroll
            for (int r = 0; r < RR; ++r) u[r] = r * nt + tid < T ? 1.f / tree_dot<EP>(x[r], s_v) : 0.f;
        }
        Acc acc[EP];
#pragma unroll
        for (int c = 0; c < EP; ++c) {
#pragma unroll
            for (int r = 0; r < RR; r += GROUP) {
                float s = x[r][c] * u[r];       // of up to four rows, pairwise
                if constexpr (GROUP > 1) s += x[r + 1][c] * u[r + 1];
                if constexpr (GROUP > 2) s += x[r + 2][c] * u[r + 2] + x[r + 3][c] * u[r + 3];
                acc[c] = r ? acc[c] + (Acc)s : (Acc)s;
            }
        }
        int column = 0;
        const double sum = sk_reduce_scatter<EP, 32>(acc, lane, column);
        if (EP == 64 || lane % (64 / EP) == 0) s_red[wv * EP + column] = sum;
        __syncthreads();
        if (wv == 0) {
            // (of wavefronts that are not there zeros: all loads are on their way together; 82.4 -> 80.3 us)
            constexpr int N = kSkSmallThreads<EP> / 64 * EP / 64 > 0 ? kSkSmallThreads<EP> / 64 * EP / 64 : 1;
            double p[N], tot = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) p[i] = s_red[64 * i + lane];
#pragma unroll
            for (int i = 0; i < N; ++i) tot += p[i];
            if constexpr (EP <= 8) tot += sk_move<8>(tot);
            if constexpr (EP <= 16) {
                double o = tot;
                sk_swap<16>(tot, o);
                tot += o;
            }
            if constexpr (EP <= 32) {
                double o = tot;
                sk_swap<32>(tot, o);
                tot += o;
            }
            if (lane < E) s_v[lane] = sk_column(tot, s_target[lane]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RR; ++r) {
        const int row = r * nt + tid;
        if (row >= T) continue;
        float pm = -INFINITY;
#pragma unroll
        for (int c = 0; c < EP; ++c) {
            x[r][c] = c < E ? u[r] * x[r][c] * s_v[c] : -INFINITY;
            if (plan && c < E) plan[(size_t)row * E + c] = x[r][c];
            pm = fmaxf(pm, x[r][c]);
        }
        int second = -1;
        if (pm > 0.f) {
#pragma unroll
            for (int c = EP - 1; c >= 0; --c)
                if (c < E && x[r][c] == pm) second = c;
        }
        assign[2 * (size_t)row] = t1[r];
        assign[2 * (size_t)row + 1] = second;
    }
}

// ---- medium: eight lanes per row, lane l holds experts l * EPL .. ----

constexpr int kSkThreads = 1024, kSkBlocks = 128;

// The v of iteration `it` from the column sums of the one before; every workgroup does this for itself.
template <int EPL>
__device__ __forceinline__ void sk_columns(const float *__restrict__ part, int n_blocks, const float *__restrict__ targets,
                                           int E, int it, float *s_v, float *s_t)
{
    constexpr int EP = 8 * EPL, NG = kSkThreads / EP;
    __shared__ double s_red[16 * EP];
    const int tid = threadIdx.x, lane = tid & 63, j = tid % EP, g = tid / EP;
    double sum = 0.0;
    if (it > 0 && j < E) {
#pragma unroll 4
        for (int b = g; b < n_blocks; b += NG) sum += (double)part[(size_t)b * EP + j];
    }
    for (int off = EP; off < 64; off <<= 1) sum += __shfl_xor(sum, off);
    if (lane < EP) s_red[(tid >> 6) * EP + lane] = sum;
    __syncthreads();
    if (tid < EP) {
        double tot = 0.0;
#pragma unroll 4
        for (int h = 0; h < 16; ++h) tot += s_red[h * EP + tid];
        const float m = tid < E ? targets[tid] : 0.f;
        s_t[tid] = m;
        s_v[tid] = m > 0.f ? (it > 0 ? sk_column(tot, m) : 1.f) : 0.f;
    }
    __syncthreads();
}

template <int EPL>
__device__ __forceinline__ void sk_row_load(const float *__restrict__ p, int E, bool vec, int c0, float (&x)[EPL])
{
    if (EPL >= 4 && vec) {
#pragma unroll
        for (int c = 0; c < EPL; c += 4) {
            const float4 f = c0 + c < E ? *(const float4 *)(p + c0 + c) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            x[c] = f.x;
            if constexpr (EPL >= 4) { x[c + 1] = f.y; x[c + 2] = f.z; x[c + 3] = f.w; }
        }
    } else {
#pragma unroll
        for (int c = 0; c < EPL; ++c) x[c] = c0 + c < E ? p[c0 + c] : -INFINITY;
    }
}

// One iteration: u of every row, and the workgroup's part of the column sums.
template <int EPL>
__global__ __launch_bounds__(kSkThreads) void k_sk_iter(const float *__restrict__ scores, const int32_t *__restrict__ top1,
                                                        const float *__restrict__ targets, const float *__restrict__ part_in,
                                                        int it, int T, int E, float inv_tau, float *__restrict__ u,
                                                        float *__restrict__ part)
{
    constexpr int EP = 8 * EPL, NG = kSkThreads / 8;
    __shared__ float s_v[EP], s_t[EP];
    __shared__ double s_col[16 * EP];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c0 = (tid & 7) * EPL;
    const bool vec = (E & 3) == 0 && ((size_t)scores & 15) == 0;
    const int n_groups = gridDim.x * NG;
    int row = blockIdx.x * NG + (tid >> 3);
    float nx[EPL];
    sk_row_load<EPL>(scores + (size_t)(row < T ? row : T - 1) * E, E, vec, c0, nx);
    int nt = top1[row < T ? row : T - 1];
    sk_columns<EPL>(part_in, gridDim.x, targets, E, it, s_v, s_t);
    float vv[EPL];
    bool open[EPL];
    double acc[EPL];
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        vv[c] = s_v[c0 + c];
        open[c] = s_t[c0 + c] > 0.f;
        acc[c] = 0.0;
    }
    for (; row - (tid >> 3) < T; row += n_groups) {
        float x[EPL];
        const int t1 = nt;
#pragma unroll
        for (int c = 0; c < EPL; ++c) x[c] = nx[c];
        const int next = row + n_groups;
        if (next - (tid >> 3) < T) {
            sk_row_load<EPL>(scores + (size_t)(next < T ? next : T - 1) * E, E, vec, c0, nx);
            nt = top1[next < T ? next : T - 1];
        }
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            if (c0 + c == t1) x[c] = 0.f;
            if (c0 + c < E) mx = fmaxf(mx, x[c]);
        }
        for (int off = 1; off < 8; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
#pragma unroll
        for (int c = 0; c < EPL; ++c) x[c] = open[c] ? expf((x[c] - mx) * inv_tau) : 0.f;
        float s = tree_dot<EPL>(x, vv);
        for (int off = 1; off < 8; off <<= 1) s += __shfl_xor(s, off);
        const float ui = 1.f / s;
        if (row < T) {
            if ((tid & 7) == 0) u[row] = ui;
#pragma unroll
            for (int c = 0; c < EPL; ++c) acc[c] += (double)(x[c] * ui);
        }
    }
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        for (int off = 8; off < 64; off <<= 1) acc[c] += __shfl_xor(acc[c], off);
        if (lane < 8) s_col[wv * EP + c0 + c] = acc[c];
    }
    __syncthreads();
    if (tid < EP) {
        double tot = 0.0;
        for (int w = 0; w < 16; ++w) tot += s_col[w * EP + tid];
        part[(size_t)blockIdx.x * EP + tid] = (float)tot;
    }
}

// The plan's largest entry of every row, with the v of the last column update.
template <int EPL>
__global__ __launch_bounds__(kSkThreads) void k_sk_pick(const float *__restrict__ scores, const int32_t *__restrict__ top1,
                                                        const float *__restrict__ targets, const float *__restrict__ part,
                                                        int n_part, int n_iter, const float *__restrict__ u, int T, int E,
                                                        float inv_tau, int32_t *__restrict__ assign, float *__restrict__ plan)
{
    constexpr int EP = 8 * EPL, NG = kSkThreads / 8;
    __shared__ float s_v[EP], s_t[EP];
    const int tid = threadIdx.x, c0 = (tid & 7) * EPL;
    const bool vec = (E & 3) == 0 && ((size_t)scores & 15) == 0;
    sk_columns<EPL>(part, n_part, targets, E, n_iter, s_v, s_t);
    for (int row = blockIdx.x * NG + (tid >> 3); row < T; row += gridDim.x * NG) {
        const int t1 = top1[row];
        const float ui = n_iter > 0 ? u[row] : 1.f;
        float x[EPL];
        sk_row_load<EPL>(scores + (size_t)row * E, E, vec, c0, x);
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            if (c0 + c == t1) x[c] = 0.f;
            if (c0 + c < E) mx = fmaxf(mx, x[c]);
        }
        for (int off = 1; off < 8; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        float pm = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const float kij = s_t[c0 + c] > 0.f ? expf((x[c] - mx) * inv_tau) : 0.f;
            x[c] = c0 + c < E ? ui * kij * s_v[c0 + c] : -INFINITY;
            if (plan && c0 + c < E) plan[(size_t)row * E + c0 + c] = x[c];
            pm = fmaxf(pm, x[c]);
        }
        for (int off = 1; off < 8; off <<= 1) pm = fmaxf(pm, __shfl_xor(pm, off));
        int second = 0x7fffffff;
#pragma unroll
        for (int c = EPL - 1; c >= 0; --c)
            if (c0 + c < E && x[c] == pm) second = c0 + c;
        for (int off = 1; off < 8; off <<= 1) {
            const int o = __shfl_xor(second, off);
            second = o < second ? o : second;
        }
        if ((tid & 7) == 0) {
            assign[2 * (size_t)row] = t1;
            assign[2 * (size_t)row + 1] = pm > 0.f && second < E ? second : -1;
        }
    }
}

// ---- large ----

// u_i = 1 / sum_j K_ij v_j for the rows of this workgroup, and the workgroup's partial sums of K_ij u_i per
// column.  LAST: also the plan's arg-max (and the plan itself) with the v of the last column update.
template <int EPL>
__global__ __launch_bounds__(256) void k_sk_row(const float *__restrict__ scores, const int32_t *__restrict__ top1,
                                                const float *__restrict__ targets, const float *__restrict__ v,
                                                int T, int E, float inv_tau, float *__restrict__ u,
                                                float *__restrict__ part)
{
    extern __shared__ float s_sk[];        // [4][E] column partials of the four wavefronts
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    float vv[EPL], acc[EPL];
    bool in[EPL];
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        const int e = lane + 64 * c;
        in[c] = e < E;
        vv[c] = (in[c] && targets[e] > 0.f) ? v[e] : 0.f;      // closed experts: K = 0
        acc[c] = 0.f;
    }
    for (int row = wave; row < T; row += n_waves) {
        const int t1 = top1[row];
        float x[EPL];
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const int e = lane + 64 * c;
            x[c] = in[c] ? (e == t1 ? 0.f : scores[(size_t)row * E + e]) : -INFINITY;
            mx = fmaxf(mx, x[c]);
        }
        mx = sk_wave_max(mx);
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            x[c] = (in[c] && targets[lane + 64 * c] > 0.f) ? expf((x[c] - mx) * inv_tau) : 0.f;   // K_ij
            s += x[c] * vv[c];
        }
        s = sk_wave_sum(s);
        const float ui = 1.f / s;
        if (lane == 0) u[row] = ui;
#pragma unroll
        for (int c = 0; c < EPL; ++c) acc[c] += x[c] * ui;
    }
#pragma unroll
    for (int c = 0; c < EPL; ++c)
        if (in[c]) s_sk[wv * E + lane + 64 * c] = acc[c];
    __syncthreads();
    for (int j = threadIdx.x; j < E; j += 256)
        part[(size_t)blockIdx.x * E + j] = (s_sk[j] + s_sk[E + j]) + (s_sk[2 * E + j] + s_sk[3 * E + j]);
}

// v_j = targets_j / sum over workgroups of part[b][j] (one workgroup; partials added in a fixed order)
__global__ __launch_bounds__(1024) void k_sk_col(const float *__restrict__ part, int n_blocks,
                                                 const float *__restrict__ targets, int E, int epad,
                                                 float *__restrict__ v)
{
    __shared__ double s_red[1024];
    const int tid = threadIdx.x, groups = 1024 / epad;
    {
        const int j = tid % epad, g = tid / epad;
        double sum = 0.0;
        if (j < E) {
#pragma unroll 8
            for (int b = g; b < n_blocks; b += groups) sum += (double)part[(size_t)b * E + j];
        }
        s_red[g * epad + j] = sum;
    }
    __syncthreads();
    if (tid < E) {
        double sum = 0.0;
        for (int g = 0; g < groups; ++g) sum += s_red[g * epad + tid];
        const float m = targets[tid];
        v[tid] = sk_column(sum, m);
    }
}

template <int EPL>
__global__ __launch_bounds__(256) void k_sk_round(const float *__restrict__ scores, const int32_t *__restrict__ top1,
                                                  const float *__restrict__ targets, const float *__restrict__ v,
                                                  const float *__restrict__ u, int use_u, int T, int E,
                                                  float inv_tau, int32_t *__restrict__ assign,
                                                  float *__restrict__ plan)
{
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    float vv[EPL];
    bool in[EPL];
#pragma unroll
    for (int c = 0; c < EPL; ++c) {
        const int e = lane + 64 * c;
        in[c] = e < E;
        vv[c] = (in[c] && targets[e] > 0.f) ? v[e] : 0.f;
    }
    for (int row = wave; row < T; row += n_waves) {
        const int t1 = top1[row];
        const float ui = use_u ? u[row] : 1.f;
        float x[EPL];
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const int e = lane + 64 * c;
            x[c] = in[c] ? (e == t1 ? 0.f : scores[(size_t)row * E + e]) : -INFINITY;
            mx = fmaxf(mx, x[c]);
        }
        mx = sk_wave_max(mx);
        float pm = -INFINITY;
#pragma unroll
        for (int c = 0; c < EPL; ++c) {
            const float kij = (in[c] && targets[lane + 64 * c] > 0.f) ? expf((x[c] - mx) * inv_tau) : 0.f;
            x[c] = in[c] ? ui * kij * vv[c] : -INFINITY;
            if (plan && in[c]) plan[(size_t)row * E + lane + 64 * c] = x[c];
            pm = fmaxf(pm, x[c]);          // fmaxf ignores a NaN operand
        }
        pm = sk_wave_max(pm);
        int second = -1;
        if (pm > 0.f) second = sk_argmax<EPL>(x, in, pm);
        if (lane == 0) {
            assign[2 * (size_t)row] = t1;
            assign[2 * (size_t)row + 1] = second;
        }
    }
}

// The capacities go to pinned words of the calling thread (a copy of a few bytes is a kernel of its own, 4 us).
int32_t caps_words(int32_t *caps_host, int **words, int **words_dev)
{
    *words = *words_dev = nullptr;
    if (!caps_host) return MAXSCORE_OK;
    const int32_t rc = solver_words(words, words_dev);
    *words += kSolverWords;
    *words_dev += kSolverWords;
    return rc;
}
int32_t copy_caps(const int *words, int32_t *caps_host, int E, hipStream_t s)
{
    if (!caps_host) return MAXSCORE_OK;
    const int32_t rc = stream_done(s);
    if (rc) return rc;
    for (int e = 0; e < E; ++e) caps_host[e] = ((const volatile int *)words)[e];
    return MAXSCORE_OK;
}

template <int EPL>
int32_t run_epl(const float *scores, int T, int E, int C, float tau, int n_iter, int32_t *assign, float *plan,
                int32_t *caps_host, char *ws, hipStream_t s)
{
    WorkspaceLayout L = workspace_layout(T, E, 1);
    int32_t *top1 = (int32_t *)(ws + L.aux_off);
    int *counts = (int *)(ws + L.price_off);
    float *targets = (float *)(ws + L.gcount_off), *v = targets + kMaxE;
    int *words, *caps;
    const int32_t rc = caps_words(caps_host, &words, &caps);
    if (rc) return rc;
    float *u = (float *)(ws + L.klist_off);
    float *part = (float *)(ws + L.wcnt_off);
    int grid = T < 4 * kSkBlocksMax ? (T + 3) / 4 : kSkBlocksMax;
    if (grid > L.max_wg) grid = L.max_wg;
    const float inv_tau = 1.f / tau;
    int epad = 1;
    while (epad < E) epad <<= 1;

    hipLaunchKernelGGL(k_sk_zero, dim3(1), dim3(1024), 0, s, counts);
    hipLaunchKernelGGL(k_sk_top1<EPL>, dim3(grid), dim3(256), 0, s, scores, T, E, top1, counts);
    hipLaunchKernelGGL(k_sk_init, dim3(1), dim3(1024), 0, s, counts, T, E, C, caps, targets, v);
    if (EPL == 1) {
        const int blocks = (T + 127) / 128 < kSkBlocks ? (T + 127) / 128 : kSkBlocks;
        float *sums = (float *)(counts + kSkCopies * kMaxE);         // two halves: of this iteration and of the one before
        auto half = [&](int it) { return sums + (size_t)(it & 1) * kSkBlocks * 64; };
#define MS_SK(PP)                                                                                                          \
    do {                                                                                                                   \
        for (int it = 0; it < n_iter; ++it)                                                                                \
            hipLaunchKernelGGL(k_sk_iter<PP>, dim3(blocks), dim3(kSkThreads), 0, s, scores, top1, targets, half(it + 1), it, T, E, \
                               inv_tau, u, half(it));                                                                      \
        hipLaunchKernelGGL(k_sk_pick<PP>, dim3((T + 127) / 128 < 512 ? (T + 127) / 128 : 512), dim3(kSkThreads), 0, s,      \
                           scores, top1, targets, half(n_iter + 1), blocks, n_iter, u, T, E, inv_tau, assign, plan);       \
    } while (0)
        if (E <= 8) MS_SK(1);
        else if (E <= 16) MS_SK(2);
        else if (E <= 32) MS_SK(4);
        else MS_SK(8);
#undef MS_SK
        MS_HIP(hipGetLastError());
        return copy_caps(words, caps_host, E, s);
    }
    for (int it = 0; it < n_iter; ++it) {
        hipLaunchKernelGGL(k_sk_row<EPL>, dim3(grid), dim3(256), (size_t)4 * E * sizeof(float), s, scores, top1,
                           targets, v, T, E, inv_tau, u, part);
        hipLaunchKernelGGL(k_sk_col, dim3(1), dim3(1024), 0, s, part, grid, targets, E, epad, v);
    }
    hipLaunchKernelGGL(k_sk_round<EPL>, dim3(grid), dim3(256), 0, s, scores, top1, targets, v, u, n_iter > 0 ? 1 : 0,
                       T, E, inv_tau, assign, plan);
    MS_HIP(hipGetLastError());
    return copy_caps(words, caps_host, E, s);
}

}  // namespace

int32_t sinkhorn_run(const float *scores, int T, int E, int C, float tau, int n_iter, int32_t *assign, float *plan,
                     int32_t *caps_host, char *ws, hipStream_t s)
{
    const int epl = (E + 63) / 64;
    const int ep = E <= 8 ? 8 : E <= 16 ? 16 : E <= 32 ? 32 : 64;
    if (E <= 64 && T <= (ep <= 16 ? 1024 : 512) * (64 / ep)) {
        const int rows = 64 / ep, nt = (std::max((T + rows - 1) / rows, std::min(T, kSkFewThreads)) + 63) / 64 * 64;
        int *words, *caps;
        const int32_t rc = caps_words(caps_host, &words, &caps);
        if (rc) return rc;
        // (of threads with a row each, all but one row of a group are beyond the batch: zeros, which add nothing to round)
        const int most = ep <= 16 ? 1024 : 512, per = (T + most - 1) / most, group = T <= nt ? 4 : per == 1 ? 1 : per < 4 ? 2 : 4;
#define MS_SK(PP, GG) hipLaunchKernelGGL((k_sk_small<PP, GG>), dim3(1), dim3(nt), 0, s, scores, T, E, C, 1.f / tau, n_iter, assign, plan, caps)
#define MS_SKG(PP)                     \
    do {                               \
        if (group == 1) MS_SK(PP, 1);  \
        else if (group == 2) MS_SK(PP, 2); \
        else MS_SK(PP, 4);             \
    } while (0)
        if (ep == 8) MS_SKG(8);
        else if (ep == 16) MS_SKG(16);
        else if (ep == 32 && group == 1) MS_SK(32, 1);
        else if (ep == 32) MS_SK(32, 2);
        else MS_SK(64, 1);
#undef MS_SKG
#undef MS_SK
        MS_HIP(hipGetLastError());
        return copy_caps(words, caps_host, E, s);
    }
    if (epl <= 1) return run_epl<1>(scores, T, E, C, tau, n_iter, assign, plan, caps_host, ws, s);
    if (epl <= 2) return run_epl<2>(scores, T, E, C, tau, n_iter, assign, plan, caps_host, ws, s);
    if (epl <= 4) return run_epl<4>(scores, T, E, C, tau, n_iter, assign, plan, caps_host, ws, s);
    if (epl <= 8) return run_epl<8>(scores, T, E, C, tau, n_iter, assign, plan, caps_host, ws, s);
    return run_epl<16>(scores, T, E, C, tau, n_iter, assign, plan, caps_host, ws, s);
}

}  // namespace maxscore
