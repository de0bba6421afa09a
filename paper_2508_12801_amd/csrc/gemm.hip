// a1: router projection  logits = x . W_g (+ bias)   (Eq. 2, Algorithm 1 step 2).
//
// bf16 inputs run on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation).  The output
// is only E <= 128 columns wide per workgroup, so the kernel is bound by streaming x from HBM:
// each workgroup owns 128 token rows, walks d in steps of 64, stages the x tile and the transposed
// W tile in LDS and prefetches the next tiles into registers while the matrix cores work.  The fast
// kernel (k_gemm_bf16_wtc) reads x with whole-line loads and restores the operand layout through LDS.
// Small batches, and fp32 throughout, run a kernel that splits d over the wavefronts of a workgroup (k_gemm_split).
#include <type_traits>

#include "common.h"
#include "softtopk_row.h"

namespace maxscore {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int BM = 128, BK = 64, LDP = BK + 8;   // LDS row pitch in bf16 elements (pad 16 B)

// 16-byte load of 8 bf16 starting at element (r, c) of a row-major [R, Ccols] matrix, zero outside.
template <bool ALIGNED>
__device__ __forceinline__ u32x4 load8(const unsigned short *__restrict__ p, int r, int c, int R, int Ccols)
{
    u32x4 out = {0u, 0u, 0u, 0u};
    if (r >= R || c >= Ccols) return out;
    const unsigned short *src = p + (size_t)r * Ccols + c;
    if (ALIGNED && c + 8 <= Ccols) {
        out = *(const u32x4 *)src;
    } else {
        unsigned short tmp[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) tmp[i] = (c + i < Ccols) ? src[i] : (unsigned short)0;
        out.x = tmp[0] | ((unsigned)tmp[1] << 16);
        out.y = tmp[2] | ((unsigned)tmp[3] << 16);
        out.z = tmp[4] | ((unsigned)tmp[5] << 16);
        out.w = tmp[6] | ((unsigned)tmp[7] << 16);
    }
    return out;
}

// NT = number of 32-column output tiles per workgroup (BN = 32*NT <= 128).
template <int NT, bool ALIGNED>
__global__ __launch_bounds__(256) void k_gemm_bf16(const unsigned short *__restrict__ x,
                                                   const unsigned short *__restrict__ W,
                                                   const float *__restrict__ bias, int T, int d, int E,
                                                   float *__restrict__ out)
{
    constexpr int BN = 32 * NT;
    __shared__ __attribute__((aligned(16))) unsigned short sA[BM * LDP];
    __shared__ __attribute__((aligned(16))) unsigned short sB[BN * LDP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int row0 = blockIdx.x * BM, col0 = blockIdx.y * 128;

    // global -> register staging: A tile 128 x 64 (4 x 16 B per thread), B tile 64 x BN
    const int a_r = tid >> 3, a_c = (tid & 7) * 8;              // + 32 rows per pass
    constexpr int B_VEC_PER_ROW = BN / 8;                        // 16-byte vectors per k-row
    constexpr int B_VECS = BK * B_VEC_PER_ROW;                   // per tile
    constexpr int B_PER_THREAD = (B_VECS + 255) / 256;
    u32x4 ra[4], rb[B_PER_THREAD];

    auto fetch = [&](int k0) {
#pragma unroll
        for (int p = 0; p < 4; ++p) ra[p] = load8<ALIGNED>(x, row0 + a_r + 32 * p, k0 + a_c, T, d);
#pragma unroll
        for (int p = 0; p < B_PER_THREAD; ++p) {
            int v = tid + 256 * p;
            int kr = v / B_VEC_PER_ROW, nc = (v % B_VEC_PER_ROW) * 8;
            rb[p] = (v < B_VECS) ? load8<ALIGNED>(W, k0 + kr, col0 + nc, d, E) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int p = 0; p < 4; ++p) *(u32x4 *)&sA[(a_r + 32 * p) * LDP + a_c] = ra[p];
#pragma unroll
        for (int p = 0; p < B_PER_THREAD; ++p) {
            int v = tid + 256 * p;
            if (v < B_VECS) {
                int kr = v / B_VEC_PER_ROW, nc = (v % B_VEC_PER_ROW) * 8;
                unsigned w4[4] = {rb[p].x, rb[p].y, rb[p].z, rb[p].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {      // transpose: sB[n][k]
                    sB[(nc + 2 * i) * LDP + kr] = (unsigned short)(w4[i] & 0xffffu);
                    sB[(nc + 2 * i + 1) * LDP + kr] = (unsigned short)(w4[i] >> 16);
                }
            }
        }
    };

    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nt][i] = 0.f;

    fetch(0);
    for (int k0 = 0; k0 < d; k0 += BK) {
        __syncthreads();            // previous tile fully consumed
        stash();
        __syncthreads();
        if (k0 + BK < d) fetch(k0 + BK);
        const int ar = wave * 32 + (lane & 31), kq = 8 * (lane >> 5);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            bf16x8 a = *(const bf16x8 *)&sA[ar * LDP + kk + kq];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                bf16x8 b = *(const bf16x8 *)&sB[(nt * 32 + (lane & 31)) * LDP + kk + kq];
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[nt], 0, 0, 0);
            }
        }
    }
    // epilogue: acc[nt][4*j + i] is row 8*j + 4*(lane/32) + i, column lane%32 of the 32 x 32 tile
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int col = col0 + nt * 32 + (lane & 31);
        if (col >= E) continue;
        const float bv = bias ? bias[col] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int row = row0 + wave * 32 + 8 * j + 4 * (lane >> 5) + i;
                if (row < T) out[(size_t)row * E + col] = acc[nt][4 * j + i] + bv;
            }
    }
}

// Transposed copy of the router weight: wt[E, d] <- W[d, E] (bf16 patterns), so that both MFMA
// operands are contiguous along the reduction index.
__global__ __launch_bounds__(256) void k_transpose_w(const unsigned short *__restrict__ W,
                                                     unsigned short *__restrict__ wt, int d, int E)
{
    __shared__ unsigned short tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // 32 x 8
    const int k0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
    for (int r = ty; r < 32; r += 8) {
        const int kk = k0 + r, n = n0 + tx;
        tile[r][tx] = (kk < d && n < E) ? W[(size_t)kk * E + n] : (unsigned short)0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int n = n0 + r, kk = k0 + tx;
        if (n < E && kk < d) wt[(size_t)n * d + kk] = tile[tx][r];
    }
}

// Main bf16 kernel (d % 8 == 0, 16-byte aligned x and wt).  Workgroup = 4 wavefronts = 128 token rows
// x (32*NT) experts; wavefront w owns rows 32w..32w+31.  Per 64-wide slab of d: the A fragments come
// straight from global memory into registers (each lane reads 16 bytes per MFMA step: row l%32,
// columns 8*(l/32).. of the step), the transposed-W slab goes through a double-buffered LDS tile shared
// by the four wavefronts.  The next slab of both is requested before the MFMAs of the current one.
template <int NT>
__global__ __launch_bounds__(256) void k_gemm_bf16_wt(const unsigned short *__restrict__ x,
                                                      const unsigned short *__restrict__ wt,
                                                      const float *__restrict__ bias, int T, int d, int E,
                                                      float *__restrict__ out)
{
    constexpr int BN = 32 * NT;
    __shared__ __attribute__((aligned(16))) unsigned short sB[2][BN * LDP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int row0 = blockIdx.x * BM, col0 = blockIdx.y * 128;
    const int arow = row0 + wave * 32 + (lane & 31), kq = 8 * (lane >> 5);
    const bool arow_ok = arow < T;
    const unsigned short *xrow = x + (size_t)(arow_ok ? arow : 0) * d;

    // B staging: BN rows x 64 columns = BN*8 16-byte vectors, B_PER per thread
    constexpr int B_VECS = BN * 8;
    constexpr int B_PER = (B_VECS + 255) / 256;
    // Two slabs of A are in flight per wavefront (x is the stream that has to come from HBM: with one
    // slab ahead the bytes in flight bound the kernel well below the memory rate); the transposed-W slab
    // comes from L2 and stays one ahead.
    u32x4 ra[2][4], rb[B_PER];
    auto fetch_a = [&](int k0, u32x4(&dst)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kk = k0 + 16 * j + kq;
            dst[j] = (arow_ok && kk < d) ? *(const u32x4 *)(xrow + kk) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto fetch_b = [&](int k0) {
#pragma unroll
        for (int p = 0; p < B_PER; ++p) {
            const int v = tid + 256 * p;
            const int n = v >> 3, kk = k0 + (v & 7) * 8;
            rb[p] = (v < B_VECS && col0 + n < E && kk < d) ? *(const u32x4 *)(wt + (size_t)(col0 + n) * d + kk)
                                                           : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto stash_b = [&](int buf) {
#pragma unroll
        for (int p = 0; p < B_PER; ++p) {
            const int v = tid + 256 * p;
            if (v < B_VECS) *(u32x4 *)&sB[buf][(v >> 3) * LDP + (v & 7) * 8] = rb[p];
        }
    };
    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nt][i] = 0.f;

    fetch_a(0, ra[0]);
    fetch_b(0);
    fetch_a(BK, ra[1]);
    stash_b(0);
    int buf = 0;
    auto step = [&](int k0, u32x4(&cur)[4]) {
        u32x4 a_cur[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) a_cur[j] = cur[j];
        __syncthreads();                         // sB[buf] is complete; sB[buf^1] is free again
        const bool more = k0 + BK < d;
        if (more) fetch_b(k0 + BK);
        if (k0 + 2 * BK < d) fetch_a(k0 + 2 * BK, cur);      // this register set is free again
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bf16x8 a = __builtin_bit_cast(bf16x8, a_cur[j]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                bf16x8 b = *(const bf16x8 *)&sB[buf][(nt * 32 + (lane & 31)) * LDP + 16 * j + kq];
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[nt], 0, 0, 0);
            }
        }
        if (more) stash_b(buf ^ 1);
        buf ^= 1;
    };
    for (int k0 = 0; k0 < d; k0 += 2 * BK) {
        step(k0, ra[0]);
        if (k0 + BK < d) step(k0 + BK, ra[1]);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int col = col0 + nt * 32 + (lane & 31);
        if (col >= E) continue;
        const float bv = bias ? bias[col] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int row = row0 + wave * 32 + 8 * j + 4 * (lane >> 5) + i;
                if (row < T) out[(size_t)row * E + col] = acc[nt][4 * j + i] + bv;
            }
    }
}

// Same tiling, but x reaches the matrix cores through a wavefront-private LDS tile: every global load
// instruction then reads whole 128-byte lines (8 rows x 128 B, 8 lanes per row) instead of 32 rows x 32 B in the
// MFMA operand layout, which is what the memory pipeline prefers; the operand layout is restored by the LDS
// read.  Needs d to be a multiple of 64.
//
// FUSE: the workgroup holds whole rows (E = 32 * NT columns, one workgroup column), so the SoftTopk scores and the
// integer rewards of Eq. 6 are computed here, from the accumulators, instead of writing the logits and reading
// them back in a second kernel: every wavefront passes its 32 rows through LDS, 16 at a time, into the layout of
// the score kernel (8 lanes per row, 16-byte pieces) and runs that kernel's row routine on them.  The logits are
// written only if the caller wants them.
template <int NT, int RB, int NS, bool FUSE>
__global__ __launch_bounds__(256) void k_gemm_bf16_wtc(const unsigned short *__restrict__ x,
                                                       const unsigned short *__restrict__ wt,
                                                       const float *__restrict__ bias, int T, int d, int E,
                                                       float *__restrict__ out, float *__restrict__ scores,
                                                       int32_t *__restrict__ q, int k, float t, float qscale)
{
    constexpr int BN = 32 * NT;
    constexpr int RW = 32 * RB;                  // rows per wavefront
    constexpr int NL = 4 * RB;                   // global loads per lane and slab
    __shared__ __attribute__((aligned(16))) unsigned short sB[2][BN * LDP];
    __shared__ __attribute__((aligned(16))) unsigned short sA[4][RW * LDP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int row0 = blockIdx.x * (4 * RW), col0 = blockIdx.y * 128;
    const int kq = 8 * (lane >> 5);
    const int lr = lane >> 3, lc = (lane & 7) * 8;          // loader: row inside a group of 8, column of the slab
    // Rows and columns beyond the matrix are computed from its last ones and dropped: a register that is either zeroed or loaded is waited
    // for around the load, and with it every slab on its way (65536 x 2048 to 32: 58.5 us before, 55.6 now; 32768 x 2048 to 128: 47.8, 45.5).
    const unsigned short *xp[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int r = row0 + wave * RW + 8 * i + lr;
        xp[i] = x + (size_t)(r < T ? r : T - 1) * d + lc;
    }
    constexpr int B_VECS = BN * 8;
    constexpr int B_PER = (B_VECS + 255) / 256;
    // NS slabs of x and W in flight per wavefront; three instead of two (and W one ahead): 16384 x 2048 to 128 experts 71 to
    // 60 us from HBM, 256 experts 80 to 70.  (Loads return in order: waiting for a slab of W requested after slabs of x
    // would wait for these as well, so both are requested equally far ahead.)
    u32x4 ra[NS][NL], rb[NS][B_PER];
    auto fetch_a = [&](int k0, u32x4(&dst)[NL]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) dst[i] = *(const u32x4 *)(xp[i] + k0);
    };
    static_assert(B_VECS % 256 == 0, "as many vectors to every thread");
    const unsigned short *wp[B_PER];
#pragma unroll
    for (int p = 0; p < B_PER; ++p) {
        const int v = tid + 256 * p, n = col0 + (v >> 3);
        wp[p] = wt + (size_t)(n < E ? n : E - 1) * d + (v & 7) * 8;
    }
    auto fetch_b = [&](int k0, u32x4(&dst)[B_PER]) {
#pragma unroll
        for (int p = 0; p < B_PER; ++p) dst[p] = *(const u32x4 *)(wp[p] + k0);
    };
    auto stash_b = [&](int buf, const u32x4(&src)[B_PER]) {
#pragma unroll
        for (int p = 0; p < B_PER; ++p) {
            const int v = tid + 256 * p;
            if (v < B_VECS) *(u32x4 *)&sB[buf][(v >> 3) * LDP + (v & 7) * 8] = src[p];
        }
    };
    f32x16 acc[RB][NT];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][nt][i] = 0.f;

    // Workgroups walk d in rotated orders: at any moment they read different column slabs of x, which spreads
    // the 2*d-byte row stride over the memory channels.
    const int nslab = d / BK;
    const int rot = (int)((blockIdx.x * 7u + (blockIdx.x >> 5)) % (unsigned)nslab);
    auto kof = [&](int i) {
        int sidx = i + rot;
        if (sidx >= nslab) sidx -= nslab;
        return sidx * BK;
    };
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (i < nslab) {
            fetch_b(kof(i), rb[i]);
            fetch_a(kof(i), ra[i]);
        }
    stash_b(0, rb[0]);
    int buf = 0;
    unsigned short *myA = sA[wave];
    auto step = [&](int it, u32x4(&cur)[NL], u32x4(&bcur)[B_PER], const u32x4(&bnext)[B_PER]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) *(u32x4 *)&myA[(8 * i + lr) * LDP + lc] = cur[i];
        __syncthreads();                         // sB[buf] and this wavefront's x tile are complete
        const bool more = it + 1 < nslab;
        if (it + NS < nslab) {
            fetch_b(kof(it + NS), bcur);
            fetch_a(kof(it + NS), cur);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bf16x8 a[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) a[b] = *(const bf16x8 *)&myA[(32 * b + (lane & 31)) * LDP + 16 * j + kq];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                bf16x8 bv = *(const bf16x8 *)&sB[buf][(nt * 32 + (lane & 31)) * LDP + 16 * j + kq];
#pragma unroll
                for (int b = 0; b < RB; ++b)
                    acc[b][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[b], bv, acc[b][nt], 0, 0, 0);
            }
        }
        if (more) stash_b(buf ^ 1, bnext);
        buf ^= 1;
    };
    for (int it = 0; it < nslab; it += NS) {
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (it + i < nslab) step(it + i, ra[i], rb[i], rb[(i + 1) % NS]);
    }
    if constexpr (FUSE) {
        static_assert(RB == 1, "the fused epilogue handles 32 rows per wavefront");
        constexpr int EPLS = BN / 8;                 // values per lane with 8 lanes per row
        constexpr int SP = BN + 4;                   // pitch of a staged row in floats
        static_assert(4 * 16 * SP * sizeof(float) <= sizeof(sB), "the staged rows reuse the W tiles");
        __syncthreads();                             // every wavefront is done with the W tiles
        float *stage = (float *)&sB[0][0] + wave * (16 * SP);
        float bvs[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bvs[nt] = bias ? bias[nt * 32 + (lane & 31)] : 0.f;
        const int lg = lane & 7, rl = lane >> 3;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        stage[(8 * jj + 4 * (lane >> 5) + i) * SP + nt * 32 + (lane & 31)] =
                            acc[0][nt][4 * (2 * half + jj) + i] + bvs[nt];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                const int r_local = 8 * pass + rl;
                const int row = row0 + wave * RW + 16 * half + r_local;
                if (row >= T) continue;          // (rows beyond the batch; 10 to 17 us at one that is no multiple of 128, while they were zeros and all ties)
                float xv[EPLS];
#pragma unroll
                for (int m = 0; m < EPLS; m += 4) {
                    const float4 v4 = *(const float4 *)&stage[r_local * SP + (m >> 2) * 32 + lg * 4];
                    xv[m] = v4.x; xv[m + 1] = v4.y; xv[m + 2] = v4.z; xv[m + 3] = v4.w;
                }
                float sc[EPLS];
                int qq[EPLS];
                softtopk_row<8, EPLS, true>(xv, lg, E, k, t, qscale, MAXSCORE_SOFTTOPK_A, sc, qq);
#pragma unroll
                for (int m = 0; m < EPLS; m += 4) {
                    const size_t o = (size_t)row * E + (m >> 2) * 32 + lg * 4;
                    if (out) *(float4 *)(out + o) = make_float4(xv[m], xv[m + 1], xv[m + 2], xv[m + 3]);
                    if (scores) *(float4 *)(scores + o) = make_float4(sc[m], sc[m + 1], sc[m + 2], sc[m + 3]);
                    if (q) *(int4 *)(q + o) = make_int4(qq[m], qq[m + 1], qq[m + 2], qq[m + 3]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();         // the next half overwrites the staged rows
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        return;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int col = col0 + nt * 32 + (lane & 31);
        if (col >= E) continue;
        const float bvs = bias ? bias[col] : 0.f;
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int row = row0 + wave * RW + 32 * b + 8 * j + 4 * (lane >> 5) + i;
                    if (row < T) out[(size_t)row * E + col] = acc[b][nt][4 * j + i] + bvs;
                }
    }
}

// The router weight in the order in which k_gemm_bf16_wide's lanes take it: 32 columns (fewer in the last block) after the other, of each
// 16 indices of d after the other, of these the lower 8 of every column, then the upper 8.  d is a multiple of 64.
__global__ __launch_bounds__(256) void k_operand_w(const unsigned short *__restrict__ W, unsigned short *__restrict__ wt, int d, int E)
{
    const int k0 = blockIdx.x * BK, n0 = blockIdx.y * 32, cols = E - n0 < 32 ? E - n0 : 32;
    const int j = threadIdx.x >> 6, h = (threadIdx.x >> 5) & 1, c = threadIdx.x & 31;
    if (c >= cols) return;
    const unsigned short *src = W + (size_t)(k0 + 16 * j + 8 * h) * E + n0 + c;
    unsigned v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = src[(size_t)i * E];
    *(u32x4 *)(wt + (size_t)n0 * d + ((size_t)(k0 / 8 + 2 * j + h) * cols + c) * 8) =
        u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
}

// 129 to 256 experts: a workgroup of eight wavefronts takes 64 whole rows, a wavefront 32 columns of them, so that the scores come from the
// sums as in k_gemm_bf16_wtc, in the layout of the score kernel for as many experts (16 lanes a row).  x goes through LDS in slabs that all
// wavefronts read; of W every wavefront has columns of its own, so that these come straight from L2, in operand order (k_operand_w: whole
// lines).  Three slabs of both are on their way.  The sums are those of k_gemm_bf16_wtc bit for bit: the same instructions in the same order
// of d.  Bound by the slabs: of x 8 KB from memory (3.4 TB/s on the whole chip), of W 32 KB from L2, and as many reads of LDS as matrix
// instructions, which take 0.6 us a slab together (0.2 each at their rates); and by the three arrays written at the end.  16384 x 2048 to 256
// 43.6 us, to 160 42.5; with two workgroups of 128 columns each, logits and the score kernel behind them 57.4 and 55.2 (W through LDS as
// well: 53 and 50).
template <bool VL>
__global__ __launch_bounds__(512) void k_gemm_bf16_wide(const unsigned short *__restrict__ x, const unsigned short *__restrict__ wt,
                                                        const float *__restrict__ bias, int T, int d, int E, float *__restrict__ out,
                                                        float *__restrict__ scores, int32_t *__restrict__ q, int k, float t, float qscale,
                                                        int quads)
{
    constexpr int BN = 256, RW = 64, NS = 4, NB = BK / 16;
    constexpr int SP = BN + 4;                   // pitch of a staged row in floats
    __shared__ __attribute__((aligned(16))) unsigned short sA[2][RW * LDP];
    __shared__ __attribute__((aligned(16))) float stage[RW * SP];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int row0 = blockIdx.x * RW, kq = 8 * (lane >> 5);
    const int lr = tid >> 3, lc = (tid & 7) * 8;             // loader: row, column of the slab
    const int col = wave * 32 + (lane & 31);
    // (rows and columns beyond the matrix are computed from others and dropped: a register that is zeroed or loaded is waited for around the
    // load, and with it every slab on its way)
    const int n0 = wave * 32 < E ? wave * 32 : 0, cols = E - n0 < 32 ? E - n0 : 32;
    const unsigned short *wp = wt + (size_t)n0 * d;
    const unsigned wo = ((lane >> 5) * cols + ((lane & 31) < cols ? (lane & 31) : cols - 1)) * 8;
    const unsigned short *xp = x + (size_t)(row0 + lr < T ? row0 + lr : T - 1) * d + lc;
    u32x4 ra[NS], rb[NS][NB];
    auto fetch_w = [&](int k0, u32x4(&b)[NB]) {
        const unsigned short *w0 = wp + (size_t)k0 * cols;
#pragma unroll
        for (int j = 0; j < NB; ++j) b[j] = *(const u32x4 *)(w0 + (16 * cols * j + wo));
    };
    auto fetch_x = [&](int k0, u32x4 &a) { a = *(const u32x4 *)(xp + k0); };
    // (d in the order of the workgroup of 128 rows that k_gemm_bf16_wtc would have)
    const int nslab = d / BK;
    const unsigned block = blockIdx.x / (BM / RW);
    const int rot = (int)((block * 7u + (block >> 5)) % (unsigned)nslab);
    auto kof = [&](int i) {
        int sidx = i + rot;
        if (sidx >= nslab) sidx -= nslab;
        return sidx * BK;
    };
    f32x16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (i < nslab) {
            fetch_x(kof(i), ra[i]);
            fetch_w(kof(i), rb[i]);
        }
    // The matrix instructions of a slab run while the operands of the next one come from LDS: straight behind each other they left the matrix
    // cores idle between the barriers.  W stays in the registers that it was loaded to until they have run, and x goes to LDS from its own: a
    // copy would be made early, and would wait for the load.
    bf16x8 av[2][2 * NB];
    auto put = [&](int it, auto part, auto cond) {
        constexpr int I = decltype(part)::value, P = I & 1;
        unsigned short *tA = sA[P];                          // (free: read two slabs ago, before the barrier of the last one)
        *(u32x4 *)&tA[lr * LDP + lc] = ra[I];
        __syncthreads();
        if (!decltype(cond)::value || it + NS < nslab) fetch_x(kof(it + NS), ra[I]);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 2; ++r) av[P][2 * j + r] = *(const bf16x8 *)&tA[(32 * r + (lane & 31)) * LDP + 16 * j + kq];
    };
    auto use = [&](int it, auto part, auto cond) {
        constexpr int I = decltype(part)::value, P = I & 1;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 2; ++r)
                acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[P][2 * j + r], __builtin_bit_cast(bf16x8, rb[I][j]), acc[r], 0, 0, 0);
        if (!decltype(cond)::value || it + NS < nslab) fetch_w(kof(it + NS), rb[I]);
    };
    static_assert(NS == 4, "four slabs a turn");
    constexpr std::integral_constant<int, 0> i0;
    constexpr std::integral_constant<int, 1> i1;
    constexpr std::integral_constant<int, 2> i2;
    constexpr std::integral_constant<int, 3> i3;
    auto turn = [&](int it, auto first, auto cond) {         // slabs it to it + 3 into registers, the products up to the last but one of them
        constexpr bool C = decltype(cond)::value;
        put(it, i0, cond);
        if (!decltype(first)::value) use(it - 1, i3, cond);
        if (!C || it + 1 < nslab) put(it + 1, i1, cond), use(it, i0, cond);
        if (!C || it + 2 < nslab) put(it + 2, i2, cond), use(it + 1, i1, cond);
        if (!C || it + 3 < nslab) put(it + 3, i3, cond), use(it + 2, i2, cond);
    };
    constexpr std::true_type yes;
    constexpr std::false_type no;
    int it = NS;
    if (nslab >= 2 * NS) turn(0, yes, no);       // (loads that may not be made are waited for early: only in the last two turns)
    else turn(0, yes, yes);
    for (; it + 2 * NS <= nslab; it += NS) turn(it, no, no);
    for (; it < nslab; it += NS) turn(it, no, yes);
    switch ((nslab - 1) % NS) {
    case 0: use(nslab - 1, i0, yes); break;
    case 1: use(nslab - 1, i1, yes); break;
    case 2: use(nslab - 1, i2, yes); break;
    default: use(nslab - 1, i3, yes);
    }
    const float bv = bias && col < E ? bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) stage[(32 * r + 8 * j + 4 * (lane >> 5) + i) * SP + col] = acc[r][4 * j + i] + bv;
    __syncthreads();
    const int lg = tid & 15;
    auto col_of = [&](int m) { return VL ? (m >> 2) * 64 + lg * 4 + (m & 3) : lg * 16 + m; };
    for (int r = tid >> 4; r < RW && row0 + r < T; r += 32) {
        float xv[16], sc[16];
        int qq[16];
#pragma unroll
        for (int m = 0; m < 16; m += 4) {
            const float4 v4 = *(const float4 *)&stage[r * SP + col_of(m)];
            const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) xv[m + i] = VL || col_of(m + i) < E ? v[i] : -3.4e38f;
        }
        softtopk_row<16, 16, VL>(xv, lg, E, k, t, qscale, MAXSCORE_SOFTTOPK_A, sc, qq);
        const size_t o0 = (size_t)(row0 + r) * E;
        if (VL || quads) {
#pragma unroll
            for (int m = 0; m < 16; m += 4) {
                if (!VL && col_of(m) >= E) continue;
                const size_t o = o0 + col_of(m);
                *(float4 *)(out + o) = make_float4(xv[m], xv[m + 1], xv[m + 2], xv[m + 3]);
                if (scores) *(float4 *)(scores + o) = make_float4(sc[m], sc[m + 1], sc[m + 2], sc[m + 3]);
                if (q) *(int4 *)(q + o) = make_int4(qq[m], qq[m + 1], qq[m + 2], qq[m + 3]);
            }
        } else {
#pragma unroll
            for (int m = 0; m < 16; ++m)
                if (col_of(m) < E) {
                    out[o0 + col_of(m)] = xv[m];
                    if (scores) scores[o0 + col_of(m)] = sc[m];
                    if (q) q[o0 + col_of(m)] = qq[m];
                }
        }
    }
}

// Split kernel: RT x 32 token rows per workgroup and up to 128 columns, d split over its KS wavefronts, whose parts are added up through
// LDS in a fixed order.  Operands come straight from global memory: within a step the matrix instruction may take its reduction
// indices in any order, so a lane reads 16 consecutive bytes of its row of x; and a tile may hold any 32 columns, so tile c takes the
// columns CT * j + c, and a lane reads its CT neighbouring columns of a row of W with one instruction.
// fp32 runs on v_mfma_f32_32x32x2_f32, four per step of 8 indices; bf16 on v_mfma_f32_32x32x16_bf16, one per step of 16.
// bf16 is bound by the latency of its loads and by the operands of W (from L2, once per 32 or 64 rows), fp32 by the matrix cores' fp32
// rate where its workgroups fill the chip (65536 rows: 101 TFLOP/s; the 157 workgroups of 10007 rows leave 99 of 256 compute units idle:
// 55).  With a load for every element of W and a wavefront to a column tile (so that x was read up to four times) bf16, scores
// in the projection, took 40.5 us at 16384 x 2048 to 64 experts (now 25.5), 15.5 at 256 x 2048 to 64 (11.6), 35 at 8192 x 2048 to 128 (23);
// fp32 47 us at 10007 x 1000 to 96 (34), 236 at 65536 x 1024 to 128 (171: 101 TFLOP/s).
// EPLS > 0: the tile holds whole rows of up to 8 * EPLS experts, and the scores and rewards are computed from it (as in k_gemm_bf16_wtc).
constexpr int kSplitPitch = 33;

template <int N>
struct __attribute__((packed, aligned(4))) Words {
    unsigned v[N];
};

template <bool BF16, bool XV, int EPLS, bool VL, int CT, int RT, int KS>
__global__ __launch_bounds__(64 * KS) void k_gemm_split(const void *__restrict__ x_, const void *__restrict__ W_,
                                                        const float *__restrict__ bias, int T, int d, int E,
                                                        float *__restrict__ out, float *__restrict__ scores,
                                                        int32_t *__restrict__ q, int k, float t, float qscale)
{
    using El = std::conditional_t<BF16, unsigned short, unsigned>;      // (fp32 as bits)
    constexpr int STEP = BF16 ? 16 : 8, LK = STEP / 2;       // reduction indices per step, per lane and step
    // Steps on their way: what the registers hold, of which a lane of sixteen wavefronts has 128.  Two row tiles there hold two steps, with
    // 17 to 32 experts' scores behind them three: logits of 16384 x 2048 to 16 22 us (30 with three, 19 registers spilled), scores 23 (29).
    constexpr int DEPTH = KS > 8 && RT > 1 ? (EPLS < 4 ? 2 : 3) : RT * CT > 4 || (KS > 8 && CT > 1 && EPLS == 0) ? 3 : 4;
    constexpr int NW = BF16 && CT > 1 ? CT / 2 : CT;         // words of a lane's columns
    constexpr int RS = KS * RT * CT * 32 * kSplitPitch * 4 <= 144 * 1024 ? RT : 1;       // row tiles added up at a time
    __shared__ __attribute__((aligned(16))) float s_part[KS * RS * CT * 32 * kSplitPitch];
    const int tid = threadIdx.x, lane = tid & 63, part = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * (32 * RT), col0 = blockIdx.y * (32 * CT);
    const int kl = LK * (lane >> 5);
    const El *xp[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int row = row0 + 32 * r + (lane & 31);
        xp[r] = (const El *)x_ + (size_t)(row < T ? row : T - 1) * d + kl;
    }
    const int col = col0 + CT * (lane & 31);                 // (columns beyond E are computed from others and dropped)
    const El *wp = (const El *)W_ + (size_t)kl * E;
    const int wc = col < E ? col : 0;
    struct Frag {
        u32x4 a[RT];
        unsigned b[LK][NW];
    };
    auto load = [&](int k0, Frag &f, bool whole) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (XV && whole) {
                f.a[r] = __builtin_bit_cast(u32x4, *(const Words<4> *)(xp[r] + k0));
            } else if (BF16) {
                unsigned v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = whole || k0 + kl + i < d ? xp[r][k0 + i] : 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) f.a[r][i] = v[2 * i] | (v[2 * i + 1] << 16);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) f.a[r][i] = whole || k0 + kl + i < d ? xp[r][k0 + i] : 0u;
            }
        }
#pragma unroll
        for (int i = 0; i < LK; ++i) {
            const El *w = wp + (size_t)(k0 + i) * E;
            const bool in = whole || k0 + kl + i < d;
            if constexpr (BF16 && CT == 1) {
                f.b[i][0] = in ? w[wc] : (El)0;
            } else {
                Words<NW> v = {};
                if (in) v = *(const Words<NW> *)(w + wc);
#pragma unroll
                for (int c = 0; c < NW; ++c) f.b[i][c] = v.v[c];
            }
        }
    };
    f32x16 acc[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][c][i] = 0.f;
    auto use = [&](const Frag &f) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if constexpr (BF16) {
                u32x4 b;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if constexpr (NW < CT) b[i] = __builtin_amdgcn_perm(f.b[2 * i + 1][c / 2], f.b[2 * i][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
                    else b[i] = f.b[2 * i][c] | (f.b[2 * i + 1][c] << 16);
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.a[r]), __builtin_bit_cast(bf16x8, b), acc[r][c], 0, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f.a[r][i]), __uint_as_float(f.b[i][c]), acc[r][c], 0, 0, 0);
            }
        }
    };
    // whole steps of this part, then (in the last part) what d leaves over
    const int steps = d / STEP, s0 = steps * part / KS, s1 = steps * (part + 1) / KS;
    Frag f[DEPTH];
    int s = s0;
    // (a part that is long enough enters its loop with all its loads made: behind loads that may not have been made the first steps of every
    // turn wait for all; 16384 x 1024 to 16 in fp32 22.2 -> 20.0 us, to 64 29.3 -> 28.1, 16384 x 2048 to 16 in bf16 21.3 -> 20.0)
    if (s + 2 * DEPTH <= s1) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load((s + i) * STEP, f[i], true);
        do {
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                const Frag cur = f[i];
                load((s + DEPTH + i) * STEP, f[i], true);
                use(cur);
            }
            s += DEPTH;
        } while (s + 2 * DEPTH <= s1);
    } else {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (s + i < s1) load((s + i) * STEP, f[i], true);
    }
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (s + i < s1) {
            const Frag cur = f[i];
            if (s + DEPTH + i < s1) load((s + DEPTH + i) * STEP, f[i], true);
            use(cur);
        }
    s += DEPTH;
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (s + i < s1) use(f[i]);
    if (part == KS - 1 && steps * STEP < d) {
        Frag g;
        load(steps * STEP, g, false);
        use(g);
    }
#pragma unroll
    for (int r0 = 0; r0 < RT; r0 += RS) {
        if (r0 > 0) __syncthreads();
        // acc[4 * j + i] is row 8 * j + 4 * (lane / 32) + i, column lane % 32 of the tile
#pragma unroll
        for (int r = 0; r < RS; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                float *mine = s_part + ((part * RS + r) * CT + c) * (32 * kSplitPitch);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mine[(8 * j + 4 * (lane >> 5) + i) * kSplitPitch + (lane & 31)] = acc[r0 + r][c][4 * j + i];
            }
        __syncthreads();
        auto total = [&](int r, int n) {                // of row r (of RS * 32) and column n
            const float *p0 = s_part + (((r >> 5) * CT + n % CT) * 32 + (r & 31)) * kSplitPitch + n / CT;
            float v = 0.f;
#pragma unroll
            for (int p = 0; p < KS; ++p) v += p0[p * (RS * CT * 32 * kSplitPitch)];
            return v;
        };
        const int row1 = row0 + 32 * r0;
        if constexpr (EPLS == 0) {
            for (int o = tid; o < RS * 32 * 32 * CT; o += 64 * KS) {
                const int r = o / (32 * CT), n = o - r * (32 * CT);
                if (row1 + r < T && col0 + n < E) out[(size_t)(row1 + r) * E + col0 + n] = total(r, n) + (bias ? bias[col0 + n] : 0.f);
            }
        } else {
            // eight lanes per row, in the layout of the score kernel for as many experts (its sums have to be the same)
            static_assert(RS * 256 <= 64 * KS, "a group of lanes per row");
            auto col_of = [](int m, int lg) { return VL ? (m >> 2) * 32 + lg * 4 + (m & 3) : lg * EPLS + m; };
            const bool quads = EPLS >= 4 && E % 4 == 0 && ((((uintptr_t)out) | ((uintptr_t)scores) | ((uintptr_t)q)) % 16) == 0;
            const int r = tid >> 3, lg = tid & 7;
            if (r < RS * 32 && row1 + r < T) {
                float xv[EPLS];
#pragma unroll
                for (int m = 0; m < EPLS; ++m) {
                    const int n = col_of(m, lg);
                    xv[m] = VL || n < E ? total(r, n) + (bias ? bias[n] : 0.f) : -3.4e38f;
                }
                float sc[EPLS];
                int qq[EPLS];
                softtopk_row<8, EPLS, VL>(xv, lg, E, k, t, qscale, MAXSCORE_SOFTTOPK_A, sc, qq);
                const size_t o0 = (size_t)(row1 + r) * E;
                if (VL || quads) {
#pragma unroll
                    for (int m = 0; m + 3 < EPLS; m += 4) {
                        const size_t o = o0 + col_of(m, lg);
                        if (!VL && col_of(m, lg) >= E) continue;
                        if (out) *(float4 *)(out + o) = make_float4(xv[m], xv[m + 1], xv[m + 2], xv[m + 3]);
                        if (scores) *(float4 *)(scores + o) = make_float4(sc[m], sc[m + 1], sc[m + 2], sc[m + 3]);
                        if (q) *(int4 *)(q + o) = make_int4(qq[m], qq[m + 1], qq[m + 2], qq[m + 3]);
                    }
                } else {
#pragma unroll
                    for (int m = 0; m < EPLS; ++m)
                        if (col_of(m, lg) < E) {
                            const size_t o = o0 + col_of(m, lg);
                            if (out) out[o] = xv[m];
                            if (scores) scores[o] = sc[m];
                            if (q) q[o] = qq[m];
                        }
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_copy16(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

}  // namespace

// The split kernel takes 32 rows to a workgroup while these fill the chip no more than once, and 64, which share the operands of W,
// beyond (up to 16384 tokens; 32 rows against 64, of 256, 1024 and 2048 in bf16, with scores): 64 experts, 8192 tokens 11.7 12.2 17.3
// against 11.5 12.5 20.8 us, 10007 tokens 14.3 19.8 31.4 against 11.6 13.0 22.6; 128 experts, 8192 tokens 11.9 15.6 23.3 against
// 16.0 22.6 33.7, 16384 tokens 19.0 29.8 45.4 against 18.1 26.7 39.2.
// fp32 has no such end.  From three column tiles on a workgroup has its compute unit to itself and one of 64 rows takes 1.6 to 1.8 times
// one of 32, so that 32 rows are the better ones wherever the fullest unit gets fewer than 1.7 times as many of them: 10007 tokens of
// 256, 1000 and 2048 to 256 experts 38 78 133 against 45 90 154 us, 20000 to 128 experts 37 83 139 against 45 92 156.
static int split_rows(int T, int E, bool own_unit)
{
    const long long cols = (E + 127) / 128, in32 = ((T + 31) / 32 * cols + 255) / 256, in64 = ((T + 63) / 64 * cols + 255) / 256;
    return in32 <= 1 || (own_unit && in32 * 10 < in64 * 17) ? 32 : 64;
}

// bf16: the split kernel as long as its workgroups of 64 rows fill the chip no more than once.  Tokens of 256, 512, 1024, 2048 and 4096,
// split against whole (with the transposition of W), scores in the projection: 64 experts, 16384 tokens 12 12 16 26 41 against 16 19 26
// 38 60 us, 20000 tokens 15 18 28 44 72 against 17 20 26 39 60; 128 experts, 16384 tokens 18 21 27 39 62 against 21 25 33 48 77, 20000
// tokens 30 35 47 70 112 against 23 26 35 49 79.  Logits: 96 experts, 16384 tokens 10 13 19 32 53 against 14 18 25 39 65, 20000 tokens 16 21
// 33 54 95 against 15 18 26 39 66; 256 experts, 8192 tokens 10 13 17 27 47 against 17 20 27 43 74, 12288 tokens 17 22 30 49 84 against 17 21
// 28 45 75 (scores below 12 us and logits below 8 are the host's time).
static bool split_is_better(int T, int E) { return (long long)((T + 31) / 32) * ((E + 127) / 128) <= 512; }

// Column tiles of a workgroup: neighbouring columns that a lane can read together, as many as there are tiles where that divides E (and
// the words of W have four bytes' alignment).
static int split_tiles(const void *W, bool bf16, int E)
{
    if (bf16 && (uintptr_t)W % 4 != 0) return 1;
    if (E <= 32) return 1;
    if (!bf16 && E > 64 && E <= 96 && E % 3 == 0) return 3;
    return E > 64 && E % 4 == 0 ? 4 : E % 2 == 0 ? 2 : 1;
}

// Whether a lane can read 16 bytes of its row of x at once (four bytes' alignment will do).
static bool split_xvec(const void *x, bool bf16, int d) { return !bf16 || (d % 2 == 0 && (uintptr_t)x % 4 == 0); }

template <bool BF16, int EPLS, bool VL, int CT>
static void split_launch(const void *x, const void *W, const float *bias, int T, int d, int E, float *logits, float *scores, int32_t *q, int k,
                         float t, float qscale, hipStream_t s)
{
    constexpr int KS1 = CT <= 2 ? 16 : 8, KS2 = CT == 1 ? 16 : 8;
    const bool xv = split_xvec(x, BF16, d);
    constexpr bool wide = BF16 || CT > 1;       // (fp32 up to 32 experts: 28 us with 32 rows, 30 with 64 at 16384 x 1024 to 16)
    const int rows = xv && wide ? split_rows(T, E, !BF16 && CT > 2) : 32;
    const dim3 g((T + rows - 1) / rows, (E + 32 * CT - 1) / (32 * CT));
#define MS_SPLIT(VV, RR, KK)                                                                                                       \
    hipLaunchKernelGGL((k_gemm_split<BF16, VV, EPLS, VL, CT, RR, KK>), g, dim3(64 * KK), 0, s, x, W, bias, T, d, E, logits, scores, q, k, t, qscale)
    if (rows == 64) {
        if constexpr (wide) MS_SPLIT(true, 2, KS2);
    } else if (xv) MS_SPLIT(true, 1, KS1);
    else if constexpr (BF16 && EPLS == 0) MS_SPLIT(false, 1, KS1);
#undef MS_SPLIT
}

// Scores in the projection: by the split kernel, if W allows whole rows in one workgroup.
static bool split_scores(const void *x, const void *W, int T, int d, int E)
{
    return split_is_better(T, E) && split_tiles(W, true, E) == E / 32 && split_xvec(x, true, d);
}

int32_t gemm_run(const void *x, const void *W, const float *bias, int dtype, int T, int d, int E, float *logits,
                 void *wt_scratch, hipStream_t s)
{
    const bool f32 = dtype == MAXSCORE_DTYPE_FP32;
    // (where the scores could come with the logits both have to come from the same kernel)
    const bool as_scores = gemm_softtopk_supported(dtype, d, E, x, wt_scratch);
    if (f32 || (as_scores ? split_scores(x, W, T, d, E) : split_is_better(T, E))) {
        const int ct = split_tiles(W, !f32, E);
#define MS_L(BB, CC) split_launch<BB, 0, false, CC>(x, W, bias, T, d, E, logits, nullptr, nullptr, 0, 0.f, 0.f, s)
        if (f32) {
            if (ct == 1) MS_L(false, 1);
            else if (ct == 2) MS_L(false, 2);
            else if (ct == 3) MS_L(false, 3);
            else MS_L(false, 4);
        } else if (ct == 1) MS_L(true, 1);
        else if (ct == 2) MS_L(true, 2);
        else MS_L(true, 4);
#undef MS_L
        MS_HIP(hipGetLastError());
        return MAXSCORE_OK;
    }
    const unsigned short *xb = (const unsigned short *)x, *wb = (const unsigned short *)W;
    dim3 grid((T + BM - 1) / BM, (E + 127) / 128);
    int et = E >= 128 ? 128 : E;
    int nt = (et + 31) / 32;
    if (wt_scratch && d % 8 == 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)wt_scratch % 16) == 0) {
        unsigned short *wt = (unsigned short *)wt_scratch;
        hipLaunchKernelGGL(k_transpose_w, dim3((d + 31) / 32, (E + 31) / 32), dim3(256), 0, s, wb, wt, d, E);
#define MS_GEMM3(NT_)                                                                                          \
    hipLaunchKernelGGL((k_gemm_bf16_wtc<NT_, 1, 3, false>), grid, dim3(256), 0, s, xb, wt, bias, T, d, E, logits, \
                       (float *)nullptr, (int32_t *)nullptr, 0, 0.f, 0.f)
        if (d % BK == 0) {
            if (nt == 1) MS_GEMM3(1);
            else if (nt == 2) MS_GEMM3(2);
            else if (nt == 3) MS_GEMM3(3);
            else MS_GEMM3(4);
            MS_HIP(hipGetLastError());
            return MAXSCORE_OK;
        }
#undef MS_GEMM3
#define MS_GEMM2(NT_) hipLaunchKernelGGL((k_gemm_bf16_wt<NT_>), grid, dim3(256), 0, s, xb, wt, bias, T, d, E, logits)
        if (nt == 1) MS_GEMM2(1);
        else if (nt == 2) MS_GEMM2(2);
        else if (nt == 3) MS_GEMM2(3);
        else MS_GEMM2(4);
#undef MS_GEMM2
        MS_HIP(hipGetLastError());
        return MAXSCORE_OK;
    }
    const bool aligned = (d % 8 == 0) && (E % 8 == 0) && (((uintptr_t)x | (uintptr_t)W) % 16 == 0);
#define MS_GEMM(NT_, AL_) \
    hipLaunchKernelGGL((k_gemm_bf16<NT_, AL_>), grid, dim3(256), 0, s, xb, wb, bias, T, d, E, logits)
    if (aligned) {
        if (nt == 1) MS_GEMM(1, true);
        else if (nt == 2) MS_GEMM(2, true);
        else if (nt == 3) MS_GEMM(3, true);
        else MS_GEMM(4, true);
    } else {
        if (nt == 1) MS_GEMM(1, false);
        else if (nt == 2) MS_GEMM(2, false);
        else if (nt == 3) MS_GEMM(3, false);
        else MS_GEMM(4, false);
    }
#undef MS_GEMM
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

bool gemm_softtopk_supported(int dtype, int d, int E, const void *x, const void *wt_scratch)
{
    return dtype == MAXSCORE_DTYPE_BF16 && (E == 32 || E == 64 || E == 128) && d >= BK && d % BK == 0 && wt_scratch &&
           ((uintptr_t)x % 16) == 0 && ((uintptr_t)wt_scratch % 16) == 0;
}

int32_t gemm_softtopk_run(const void *x, const void *W, const float *bias, int dtype, int T, int d, int E, int k,
                          float t, int shift, float *logits, float *scores, int32_t *q, void *wt_scratch,
                          hipStream_t s)
{
    if (!gemm_softtopk_supported(dtype, d, E, x, wt_scratch)) return MAXSCORE_ERR_SHAPE;
    if (((((uintptr_t)logits) | ((uintptr_t)scores) | ((uintptr_t)q)) % 16) != 0) return MAXSCORE_ERR_SHAPE;
    const unsigned short *xb = (const unsigned short *)x, *wb = (const unsigned short *)W;
    unsigned short *wt = (unsigned short *)wt_scratch;
    const float qscale = (float)(1 << shift);
    if (split_scores(x, W, T, d, E)) {
#define MS_LF(FF) split_launch<true, FF / 8, true, FF / 32>(x, W, bias, T, d, E, logits, scores, q, k, t, qscale, s)
        if (E == 32) MS_LF(32);
        else if (E == 64) MS_LF(64);
        else MS_LF(128);
#undef MS_LF
        MS_HIP(hipGetLastError());
        return MAXSCORE_OK;
    }
    hipLaunchKernelGGL(k_transpose_w, dim3((d + 31) / 32, (E + 31) / 32), dim3(256), 0, s, wb, wt, d, E);
    dim3 grid((T + BM - 1) / BM, 1);
#define MS_GEMMF(NT_)                                                                                         \
    hipLaunchKernelGGL((k_gemm_bf16_wtc<NT_, 1, 3, true>), grid, dim3(256), 0, s, xb, wt, bias, T, d, E, logits, \
                       scores, q, k, t, qscale)
    if (E == 32) MS_GEMMF(1);
    else if (E == 64) MS_GEMMF(2);
    else MS_GEMMF(4);
#undef MS_GEMMF
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

// Whole rows of up to 128 experts in a workgroup of the split kernel: the scores of other expert counts, and in fp32, from its sums.
// (In bf16 not of 32, 64 and 128 experts: where these do not come from gemm_softtopk_run, d is no multiple of 64 or there is no workspace,
// the score kernel runs behind the projection: 4096 x 1000 to 64 7.8 + 4.0 us, to 48 in one kernel 9.8.)
// With the score kernel behind the projection 4096 x 1024 to 16 took 14.2 us (now 11.5), 64 x 64 to 8 in fp32 14.0 (11.2), 20000 x 512 to 20
// 24.7 (20.7), 10007 x 1000 to 96 43.9 (43.1).  Beyond 64 experts and 16384 tokens the score kernel's wavefronts are the better ones
// (fp32, 65536 x 1024 to 128: 191, in the projection 195).
bool gemm_split_scores_supported(int dtype, int T, int d, int E, const void *x, const void *W)
{
    const bool bf16 = dtype == MAXSCORE_DTYPE_BF16;
    return E <= 128 && (E <= 64 || T <= 16384) && 32 * split_tiles(W, bf16, E) >= E && split_xvec(x, bf16, d) && (!bf16 || (split_is_better(T, E) && E != 32 && E != 64 && E != 128));
}

int32_t gemm_split_scores_run(const void *x, const void *W, const float *bias, int dtype, int T, int d, int E, int k, float t, int shift,
                              float *logits, float *scores, int32_t *q, hipStream_t s)
{
    if (!gemm_split_scores_supported(dtype, T, d, E, x, W)) return MAXSCORE_ERR_SHAPE;
    const float qscale = (float)(1 << shift);
    const bool bf16 = dtype == MAXSCORE_DTYPE_BF16;
    // (the score kernel reads whole rows in pieces of four columns where it can: the layouts have to agree)
    const bool vl = (E == 32 || E == 64 || E == 128) && ((((uintptr_t)logits) | ((uintptr_t)scores) | ((uintptr_t)q)) % 16) == 0;
    const int ct = split_tiles(W, bf16, E);
#define MS_LS(BB, PP, VV, CC) split_launch<BB, PP, VV, CC>(x, W, bias, T, d, E, logits, scores, q, k, t, qscale, s)
    if (bf16) {
        if (E <= 8) MS_LS(true, 1, false, 1);
        else if (E <= 16) MS_LS(true, 2, false, 1);
        else if (E < 32) MS_LS(true, 4, false, 1);
        else if (ct == 2) MS_LS(true, 8, false, 2);
        else MS_LS(true, 16, false, 4);
    } else if (ct == 1) {
        if (E <= 8) MS_LS(false, 1, false, 1);
        else if (E <= 16) MS_LS(false, 2, false, 1);
        else if (vl) MS_LS(false, 4, true, 1);
        else MS_LS(false, 4, false, 1);
    } else if (ct == 2) {
        if (vl) MS_LS(false, 8, true, 2);
        else MS_LS(false, 8, false, 2);
    } else if (ct == 3) MS_LS(false, 16, false, 3);
    else if (vl) MS_LS(false, 16, true, 4);
    else MS_LS(false, 16, false, 4);
#undef MS_LS
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

// Whether k_gemm_bf16_wide is the better one.  Of its workgroups each of the 256 compute units holds one at a time, so that a last set that
// leaves many units idle costs as much as a full one; the two kernels with their smaller workgroups lose less to it.  Against them, 2048 to
// 256: 9000 tokens 31.8 us to 48.2, 16384 43.6 to 57.4; then 20000 71.5 to 66.2 and 24576 75.2 to 73.0, 28672 75.2 to 75.5, 32768 75.2 to
// 79.6, 45056 115.7 to 127.8, 65536 155 to 180.  Hence one set, or sets that fill 7/8 of the places.
static bool wide_is_better(int T)
{
    const long long blocks = (T + 63) / 64, sets = (blocks + 255) / 256;
    return sets == 1 || blocks * 8 >= sets * 256 * 7;
}

// The scores of 129 to 256 experts in the projection, where gemm_run would take k_gemm_bf16_wtc.
bool gemm_wide_scores_supported(int dtype, int T, int d, int E, const void *x, const void *wt_scratch)
{
    return dtype == MAXSCORE_DTYPE_BF16 && E > 128 && E <= 256 && d >= BK && d % BK == 0 && wt_scratch && ((uintptr_t)x % 16) == 0 &&
           ((uintptr_t)wt_scratch % 16) == 0 && !split_is_better(T, E) && wide_is_better(T);
}

int32_t gemm_wide_scores_run(const void *x, const void *W, const float *bias, int dtype, int T, int d, int E, int k, float t, int shift,
                             float *logits, float *scores, int32_t *q, void *wt_scratch, hipStream_t s)
{
    if (!gemm_wide_scores_supported(dtype, T, d, E, x, wt_scratch)) return MAXSCORE_ERR_SHAPE;
    const unsigned short *xb = (const unsigned short *)x, *wb = (const unsigned short *)W;
    unsigned short *wt = (unsigned short *)wt_scratch;
    const float qscale = (float)(1 << shift);
    // (as the score kernel chooses: the layouts have to agree)
    const bool aligned = ((((uintptr_t)logits) | ((uintptr_t)scores) | ((uintptr_t)q)) % 16) == 0;
    hipLaunchKernelGGL(k_operand_w, dim3(d / BK, (E + 31) / 32), dim3(256), 0, s, wb, wt, d, E);
    if (E == 256 && aligned)
        hipLaunchKernelGGL(k_gemm_bf16_wide<true>, dim3((T + 63) / 64), dim3(512), 0, s, xb, wt, bias, T, d, E, logits, scores, q, k, t, qscale, 1);
    else
        hipLaunchKernelGGL(k_gemm_bf16_wide<false>, dim3((T + 63) / 64), dim3(512), 0, s, xb, wt, bias, T, d, E, logits, scores, q, k, t, qscale,
                           E % 4 == 0 && aligned ? 1 : 0);
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

int32_t copy_run(const void *src, void *dst, size_t bytes, hipStream_t s)
{
    size_t n = bytes / 16;
    int grid = (int)((n + 255) / 256);
    if (grid > 16384) grid = 16384;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(k_copy16, dim3(grid), dim3(256), 0, s, (const u32x4 *)src, (u32x4 *)dst, n);
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

}  // namespace maxscore
