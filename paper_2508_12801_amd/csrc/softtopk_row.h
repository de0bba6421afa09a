// One token row of a2 + a3 (Eq. 6; softmax of Table 2 row 1), shared by the score kernel and by the projection
// kernel that computes the scores in its epilogue.  A group of G lanes owns the row; in the vector layout lane l
// owns the 4-column pieces l, l+G, l+2G, ... (columns (m >> 2) * 4G + 4l + (m & 3) for its m-th value), in the
// scalar layout the EPL consecutive columns l*EPL .. l*EPL+EPL-1.  Both kernels run the same instructions on the
// same values in the same lanes, so their scores and rewards are bit-equal.
#pragma once

#include "common.h"
#include "row_keys.h"

namespace maxscore {

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int off)
{
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    lo = __shfl_xor(lo, off);
    hi = __shfl_xor(hi, off);
    return ((unsigned long long)hi << 32) | lo;
}

// order-preserving map float -> uint32 (finite inputs)
__device__ __forceinline__ unsigned ord_f32(float x)
{
    unsigned u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// maximum and sum over a group of G lanes, left in all of them
template <int G>
__device__ __forceinline__ float max_of_group(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true)));     // quad_perm [1,0,3,2]
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true)));     // quad_perm [2,3,0,1]
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, true)));    // row_half_mirror
    if constexpr (G >= 16) v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, true)));   // row_mirror
    if constexpr (G >= 32) v = fmaxf(v, __shfl_xor(v, 16));
    if constexpr (G >= 64) v = fmaxf(v, __shfl_xor(v, 32));
    return v;
}
__device__ __forceinline__ int dpp_bits(float v) { return __float_as_int(v); }
__device__ __forceinline__ int dpp_bits(int v) { return v; }
template <typename V>
__device__ __forceinline__ V dpp_value(int v)
{
    if constexpr (sizeof(V) == 4 && V(0.5f) != V(0)) return __int_as_float(v);
    else return v;
}
// (adds the value of the lane G/2 away, then of the one G/4 away and so on: after a step all values repeat with its distance,
// and a rotation brings the same one as an exchange)
template <int G, typename V>
__device__ __forceinline__ V sum_of_group(V v)
{
    static_assert(G >= 8, "groups of 8 lanes at least");
    if constexpr (G >= 64) v += __shfl_xor(v, 32);
    if constexpr (G >= 32) v += __shfl_xor(v, 16);
    if constexpr (G >= 16) {
        v += dpp_value<V>(__builtin_amdgcn_mov_dpp(dpp_bits(v), 0x128, 0xf, 0xf, true));                 // row_ror:8
        v += dpp_value<V>(__builtin_amdgcn_mov_dpp(dpp_bits(v), 0x124, 0xf, 0xf, true));                 // row_ror:4
    } else {
        const int from_above = __builtin_amdgcn_update_dpp(0, dpp_bits(v), 0x104, 0xf, 0x5, false);      // row_shl:4, lanes 0-3 and 8-11
        v += dpp_value<V>(__builtin_amdgcn_update_dpp(from_above, dpp_bits(v), 0x114, 0xf, 0xa, false)); // row_shr:4, the others
    }
    v += dpp_value<V>(__builtin_amdgcn_mov_dpp(dpp_bits(v), 0x4E, 0xf, 0xf, true));                      // quad_perm [2,3,0,1]
    v += dpp_value<V>(__builtin_amdgcn_mov_dpp(dpp_bits(v), 0xB1, 0xf, 0xf, true));                      // quad_perm [1,0,3,2]
    return v;
}

// x: this lane's logits of the row (columns at or beyond E must hold -3.4e38f); sc, qq: its scores and rewards.
template <int G, int EPL, bool kVec>
__device__ __forceinline__ void softtopk_row(const float (&x)[EPL], int lg, int E, int k, float t, float qscale,
                                             int reading, float (&sc)[EPL], int (&qq)[EPL])
{
    auto colof = [&](int m) { return kVec ? ((m >> 2) * (4 * G) + lg * 4 + (m & 3)) : (lg * EPL + m); };
    float mx = -3.4e38f;
#pragma unroll
    for (int m = 0; m < EPL; ++m) mx = fmaxf(mx, x[m]);
    unsigned key[EPL];                 // order of the logits; columns the row does not have come last
#pragma unroll
    for (int m = 0; m < EPL; ++m) key[m] = colof(m) < E ? ord_f32(x[m]) : 0u;
    unsigned cur = RowKeys<G, EPL>::first(key);
    mx = max_of_group<G>(mx);
    float ex[EPL];
    float sum = 0.f;
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        // fast exponential (exp2 of the scaled argument): the argument is in [-87, 0], its scaling costs at most
        // |x| * 2^-24 of relative error, 1.5e-6 at x = -16, below which a probability is under 1e-7
        ex[m] = (colof(m) < E) ? __expf(x[m] - mx) : 0.f;
        sum += ex[m];
    }
    sum = sum_of_group<G>(sum);
    const float inv = 1.0f / sum;

    // Entries among the n_pick largest weigh by their rank, the others share the weight of the ranks beyond.  Where no two
    // of the largest are equal the rank is the number of values above: one subtraction and minimum per entry find the next
    // value, one comparison and addition count it.
    const int n_pick = (reading == MAXSCORE_SOFTTOPK_A1 || reading == MAXSCORE_SOFTTOPK_B) ? k : k - 1;
    float wv[EPL];
    float w_run = 0.f;                 // reading C: the weight of the rank being picked
    unsigned taken = 0;
    bool counted = false;
    if (t != 0.f && reading != MAXSCORE_SOFTTOPK_C) {
        int above[EPL];
#pragma unroll
        for (int m = 0; m < EPL; ++m) above[m] = 0;
        bool distinct = true;
        for (int r = 1; r <= n_pick; ++r) {
#pragma unroll
            for (int m = 0; m < EPL; ++m) above[m] += key[m] < cur ? 1 : 0;
            if (r < n_pick) {
                const unsigned next = RowKeys<G, EPL>::below(key, cur);
                distinct = distinct && next < cur && next != 0u;
                cur = next;
            }
        }
        int picked = 0;
#pragma unroll
        for (int m = 0; m < EPL; ++m) picked += above[m] < n_pick ? 1 : 0;
        picked = sum_of_group<G>(picked);
        counted = distinct && picked == n_pick;
        if (counted) {
#pragma unroll
            for (int m = 0; m < EPL; ++m) {
                wv[m] = reading == MAXSCORE_SOFTTOPK_B && above[m] < n_pick ? 0.f : (float)above[m];
                if (reading == MAXSCORE_SOFTTOPK_B && above[m] >= n_pick) wv[m] = (float)(k - 1);
            }
            taken = ~0u;
        }
    }
    // Equal logits among the largest (lower column first), and reading C: one by one.
    if (t != 0.f && !counted) {
        for (int r = 1; r <= n_pick; ++r) {
            unsigned bo = 0;
            int bm = -1;
#pragma unroll
            for (int m = 0; m < EPL; ++m) {
                const unsigned o = ord_f32(x[m]);
                const bool take = (colof(m) < E) && !((taken >> m) & 1u) && (bm < 0 || o > bo);
                bo = take ? o : bo;
                bm = take ? m : bm;
            }
            unsigned long long best =
                bm >= 0 ? (((unsigned long long)bo << 10) | (unsigned)(1023 - colof(bm))) : 0ull;
#pragma unroll
            for (int off = G / 2; off > 0; off >>= 1) {
                unsigned long long o = shfl_xor_u64(best, off);
                best = o > best ? o : best;
            }
            const int e = 1023 - (int)(best & 1023);
            const bool mine = kVec ? (((e >> 2) & (G - 1)) == lg) : (e / EPL == lg);
            if (mine) {
                const int m = kVec ? ((e / (4 * G)) * 4 + (e & 3)) : (e % EPL);
                const float w = reading == MAXSCORE_SOFTTOPK_B ? 0.f
                              : reading == MAXSCORE_SOFTTOPK_C ? w_run : (float)(r - 1);
#pragma unroll
                for (int mm = 0; mm < EPL; ++mm)
                    if (mm == m) wv[mm] = w;
                taken |= 1u << m;
            }
            if (reading == MAXSCORE_SOFTTOPK_C) {
                // mass outside the r largest, summed over what is left (no cancellation on peaked rows)
                float rest = 0.f;
#pragma unroll
                for (int m = 0; m < EPL; ++m) rest += ((taken >> m) & 1u) ? 0.f : ex[m];
#pragma unroll
                for (int off = G / 2; off > 0; off >>= 1) rest += __shfl_xor(rest, off);
                w_run += rest > 0.f ? 1.0f / (rest * inv) : 0.f;      // (nothing left: the entries beyond are 0 anyway)
            }
        }
    }
    const float w_rest = reading == MAXSCORE_SOFTTOPK_A1 ? (float)k
                       : reading == MAXSCORE_SOFTTOPK_C  ? w_run : (float)(k - 1);
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const float p = ex[m] * inv;
        const float w = ((taken >> m) & 1u) ? wv[m] : w_rest;
        sc[m] = p * (1.0f + t * w);
        qq[m] = __float2int_rn(sc[m] * qscale);
    }
}

}  // namespace maxscore
