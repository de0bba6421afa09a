// Rows as packed keys: the k best entries of a row in order, without sorting it.  Shared by the price solve and the iterative
// rerouting.
#pragma once

#include "common.h"

namespace maxscore {

// minimum over a group of G lanes, left in all of them
template <int G>
__device__ __forceinline__ unsigned group_min_u32(unsigned v)
{
    unsigned o;
    if constexpr (G >= 8) {
        o = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true); v = o < v ? o : v;    // quad_perm [1,0,3,2]
        o = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true); v = o < v ? o : v;    // quad_perm [2,3,0,1]
        o = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true); v = o < v ? o : v;   // row_half_mirror
    }
    if constexpr (G >= 16) {
        o = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, true); v = o < v ? o : v;   // row_mirror
    }
    if constexpr (G >= 32) { o = __shfl_xor(v, 16); v = o < v ? o : v; }
    if constexpr (G >= 64) { o = __shfl_xor(v, 32); v = o < v ? o : v; }
    return v;
}

// A group of G lanes owns a row; lane l owns columns (m >> 2) * 4G + 4l + (m & 3) for m < EPL (EPL >= 4: every load of
// the group covers whole lines), else l * EPL + m.  A value and its column are packed into one 32-bit key, so that the
// next best entry of a row is one subtract and one unsigned minimum per entry: the largest key below x is
// x - 1 - min over keys of (x - 1 - key), entries at or above x wrap around to large numbers.
template <int G, int EPL>
struct RowKeys {
    static __device__ __forceinline__ int col(int m, int lg)
    {
        return EPL >= 4 ? (m >> 2) * (4 * G) + lg * 4 + (m & 3) : lg * EPL + m;
    }
    static __device__ __forceinline__ void load(const int32_t *__restrict__ qr, int E, bool vec, int lg, int (&v)[EPL])
    {
        if (EPL >= 4 && vec) {
#pragma unroll
            for (int m = 0; m < EPL; m += 4) {
                const int c = col(m, lg);
                const int4 t4 = c < E ? *(const int4 *)(qr + c) : make_int4(0, 0, 0, 0);
                v[m] = t4.x;
                if constexpr (EPL >= 4) { v[m + 1] = t4.y; v[m + 2] = t4.z; v[m + 3] = t4.w; }
            }
        } else {
#pragma unroll
            for (int m = 0; m < EPL; ++m) v[m] = col(m, lg) < E ? qr[col(m, lg)] : 0;
        }
    }
    static __device__ __forceinline__ unsigned first(const unsigned (&key)[EPL])
    {
        unsigned d = ~key[0];
#pragma unroll
        for (int m = 1; m < EPL; ++m) d = ~key[m] < d ? ~key[m] : d;
        return ~group_min_u32<G>(d);
    }
    static __device__ __forceinline__ unsigned below(const unsigned (&key)[EPL], unsigned x)
    {
        const unsigned x1 = x - 1;
        unsigned d = x1 - key[0];
#pragma unroll
        for (int m = 1; m < EPL; ++m) {
            const unsigned dm = x1 - key[m];
            d = dm < d ? dm : d;
        }
        return x1 - group_min_u32<G>(d);
    }
};

}  // namespace maxscore
