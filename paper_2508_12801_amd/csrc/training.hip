// Training-side by-products of the routing path: the load-balance loss of Eq. 9 (Section 4.1) and the
// derivative of the gates (Eq. 2 with the SoftTopk scores of Eq. 6) with respect to the router logits.
//
// The rank multipliers of Eq. 6 are piecewise constant in the logits, so A_ij = m_ij * Softmax(L_i)_j gives
// dA_ij/dL_il = A_ij * (delta_jl - p_il): the backward pass needs the logits (for p) and the scores, not t or k.
#include "common.h"
#include "sums.h"

namespace maxscore {
namespace {

constexpr int kColBlocksMax = 256, kColRows = 16;

// part[b][j] <- sum of scores[row][j] over the rows of block b.  blockDim = 256 = cols x rowlanes; a thread owns
// VEC adjacent columns (VEC = 4 when E is a multiple of 4) and keeps kColRows row loads in flight.  Their sum is added in fp32,
// everything from there on in double: the mean of a column is good to kColRows roundings whatever the number of rows.
template <int VEC>
__global__ __launch_bounds__(256) void k_colsum(const float *__restrict__ scores, int T, int E, int cols,
                                                int rows_per_block, float *__restrict__ part)
{
    extern __shared__ double s_acc[];    // [rowlanes][E]
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    typedef double wide_t __attribute__((ext_vector_type(VEC)));
    const int rowlanes = 256 / cols, nvec = E / VEC;
    const int c = threadIdx.x % cols, rl = threadIdx.x / cols;
    const int r0 = blockIdx.x * rows_per_block;
    const int r1 = r0 + rows_per_block < T ? r0 + rows_per_block : T;
    const vec_t *src = reinterpret_cast<const vec_t *>(scores);
    for (int jv = c; jv < nvec; jv += cols) {
        wide_t acc = 0.0;
        for (int r = r0 + rl; r < r1; r += kColRows * rowlanes) {
            vec_t x[kColRows];
#pragma unroll
            for (int u = 0; u < kColRows; ++u) {
                const int ru = r + u * rowlanes;
                x[u] = src[(size_t)(ru < r1 ? ru : r1 - 1) * nvec + jv];
            }
            vec_t sum = x[0];
#pragma unroll
            for (int u = 1; u < kColRows; ++u) sum += r + u * rowlanes < r1 ? x[u] : (vec_t)0.f;
            acc += __builtin_convertvector(sum, wide_t);
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) s_acc[rl * E + jv * VEC + i] = acc[i];
    }
    __syncthreads();
    for (int j = threadIdx.x; j < E; j += 256) {
        double acc = 0.0;
        for (int l = 0; l < rowlanes; ++l) acc += s_acc[l * E + j];
        part[(size_t)blockIdx.x * E + j] = (float)acc;
    }
}

// One workgroup: column means, the loss and its derivative with respect to the scores of a column.  Thread
// (j, g) adds the partial sums g, g+groups, ... of column j, eight at a time; the groups that have any are then added in order.  Bound by
// latency: these loads, a barrier and that serial sum: 65536 tokens of 128 experts 4.8 us, 20000 of 128 4.7 (6.0 with the last ones of a
// thread one after the other), 65536 of 8 4.2, 256 of 8 2.5 (3.7 over all groups).  With four columns a thread the serial sum is four
// times as long: 5.4, 5.4, 8.0 and 7.9 us (5.3, 5.3, 5.3 and 2.4 over the groups that have any).
__global__ __launch_bounds__(1024) void k_aux_final(const float *__restrict__ part, int n_blocks,
                                                    const int32_t *__restrict__ offsets, int T, int E, int epad,
                                                    float lam, float *__restrict__ loss,
                                                    float *__restrict__ mean_scores, float *__restrict__ dscores_col)
{
    __shared__ double s_red[1024];
    __shared__ double s_w[16];
    const int tid = threadIdx.x, groups = 1024 / epad;
    {
        const int j = tid % epad, g = tid / epad;
        double sum = 0.0;
        if (j < E && g < n_blocks) {
            constexpr int L = 8;
            int b = g;
            for (; b + (L - 1) * groups < n_blocks; b += L * groups) {
                float x[L];
#pragma unroll
                for (int u = 0; u < L; ++u) x[u] = part[(size_t)(b + u * groups) * E + j];
#pragma unroll
                for (int u = 0; u < L; ++u) sum += (double)x[u];
            }
            // the rest, together as well
            if (b < n_blocks) {
                float x[L - 1];
#pragma unroll
                for (int u = 0; u < L - 1; ++u) x[u] = part[(size_t)(b + u * groups < n_blocks ? b + u * groups : b) * E + j];
#pragma unroll
                for (int u = 0; u < L - 1; ++u) sum += b + u * groups < n_blocks ? (double)x[u] : 0.0;
            }
        }
        s_red[g * epad + j] = sum;
    }
    __syncthreads();
    const int j = tid, filled = groups < n_blocks ? groups : n_blocks;
    double term = 0.0;
    if (j < E) {
        double sum = 0.0;
#pragma unroll 8
        for (int g = 0; g < filled; ++g) sum += s_red[g * epad + j];
        const double mean_a = sum / T;
        const double mean_p = (double)(offsets[j + 1] - offsets[j]) / T;
        term = mean_a * mean_p;
        if (mean_scores) mean_scores[j] = (float)mean_a;
        if (dscores_col) dscores_col[j] = (float)((double)lam / ((double)E * T) * mean_p);
    }
    for (int off = 32; off >= 1; off >>= 1) term += __shfl_xor(term, off);
    if ((j & 63) == 0) s_w[j >> 6] = term;
    __syncthreads();
    if (j == 0) {
        double tot = 0.0;
        for (int w = 0; w < 16; ++w) tot += s_w[w];
        *loss = (float)((double)lam * tot / E);
    }
}

// G lanes own a token row, lane l the 4-column pieces l, l+G, ... of it: a wavefront has 64 / G rows on their way, in whole
// lines.  The gradients of a row's gates are put in their columns through LDS, each read by one lane (read by all of them and compared
// with every column: 16 loads and 200 instructions a row).  Bound by HBM: 65536 rows of 128 experts 17.4 us (6.0 TB/s; 23.0 the other
// way), of 64 12.9 (14.2).
template <int G, int EPL>
__global__ __launch_bounds__(256) void k_gates_backward(const float *__restrict__ logits,
                                                        const float *__restrict__ scores,
                                                        const int32_t *__restrict__ assign,
                                                        const float *__restrict__ dgates,
                                                        const float *__restrict__ dscores_col, int T, int E, int k,
                                                        int vec, float *__restrict__ dlogits)
{
    constexpr int NG = 256 / G;
    __shared__ __attribute__((aligned(16))) float s_d[NG][G * EPL];      // gradients of a row's gates, at their experts
    const int lg = threadIdx.x & (G - 1);
    float *mine = s_d[threadIdx.x / G];
    auto col = [&](int m) { return (m >> 2) * (4 * G) + lg * 4 + (m & 3); };
    auto load = [&](const float *__restrict__ p, float fill, float(&x)[EPL]) {
#pragma unroll
        for (int m = 0; m < EPL; m += 4) {
            const int c = col(m);
            if (vec) {
                const float4 f = c < E ? *(const float4 *)(p + c) : make_float4(fill, fill, fill, fill);
                x[m] = f.x; x[m + 1] = f.y; x[m + 2] = f.z; x[m + 3] = f.w;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) x[m + i] = c + i < E ? p[c + i] : fill;
            }
        }
    };
    auto row_sync = [] {                     // (a row's lanes are of one wavefront)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int row = blockIdx.x * NG + threadIdx.x / G; row < T; row += gridDim.x * NG) {
        float l[EPL], a[EPL], g[EPL] = {};
        load(logits + (size_t)row * E, -INFINITY, l);
        load(scores + (size_t)row * E, 0.f, a);
        if (dscores_col) load(dscores_col, 0.f, g);
#pragma unroll
        for (int m = 0; m < EPL; m += 4) *(float4 *)(mine + col(m)) = make_float4(0.f, 0.f, 0.f, 0.f);
        row_sync();
        for (int s = lg; s < k; s += G) {
            const int e = assign[(size_t)row * k + s];
            if (e >= 0 && e < E) atomicAdd(mine + e, dgates[(size_t)row * k + s]);
        }
        row_sync();
#pragma unroll
        for (int m = 0; m < EPL; m += 4) {
            const float4 f = *(const float4 *)(mine + col(m));
            g[m] += f.x; g[m + 1] += f.y; g[m + 2] += f.z; g[m + 3] += f.w;
        }
        row_sync();
        float mx = -INFINITY;
#pragma unroll
        for (int m = 0; m < EPL; ++m) mx = fmaxf(mx, l[m]);
        for (int off = G / 2; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
#pragma unroll
        for (int m = 0; m < EPL; ++m) {
            l[m] = __expf(l[m] - mx);        // padded columns: exp(-inf) = 0
            g[m] *= a[m];                    // w_j = gA_j * A_j
        }
        float z = tree_sum<EPL>(l), w = tree_sum<EPL>(g);
        for (int off = G / 2; off >= 1; off >>= 1) {
            z += __shfl_xor(z, off);
            w += __shfl_xor(w, off);
        }
        const float scale = w / z;
        float *out = dlogits + (size_t)row * E;
#pragma unroll
        for (int m = 0; m < EPL; m += 4) {
            const int c = col(m);
            if (vec) {
                if (c < E) *(float4 *)(out + c) = make_float4(g[m] - l[m] * scale, g[m + 1] - l[m + 1] * scale,
                                                              g[m + 2] - l[m + 2] * scale, g[m + 3] - l[m + 3] * scale);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c + i < E) out[c + i] = g[m + i] - l[m + i] * scale;
            }
        }
    }
}

template <int G, int EPL>
void launch_bwd(const float *logits, const float *scores, const int32_t *assign, const float *dgates,
                const float *dcol, int T, int E, int k, float *dlogits, hipStream_t s)
{
    const int ng = 256 / G, grid = (T + ng - 1) / ng < 8192 ? (T + ng - 1) / ng : 8192;
    const int vec = E % 4 == 0 && (((uintptr_t)logits | (uintptr_t)scores | (uintptr_t)dlogits | (uintptr_t)dcol) % 16) == 0 ? 1 : 0;
    hipLaunchKernelGGL((k_gates_backward<G, EPL>), dim3(grid), dim3(256), 0, s, logits, scores, assign, dgates, dcol, T, E,
                       k, vec, dlogits);
}

}  // namespace

int32_t aux_loss_run(const float *scores, const int32_t *offsets, int T, int E, float lam, float *loss,
                     float *mean_scores, float *dscores_col, char *ws, hipStream_t s)
{
    WorkspaceLayout L = workspace_layout(T, E, 1);
    float *part = (float *)(ws + L.wcnt_off);          // n_blocks*E floats <= E*(T/4) ints
    const int vec = (E % 4 == 0 && ((uintptr_t)scores % 16) == 0) ? 4 : 1;
    int cols = 1;
    while (cols < E / vec && cols < 256) cols <<= 1;
    const int rowlanes = 256 / cols;
    int n_blocks = (T + 63) / 64;
    if (n_blocks > kColBlocksMax) n_blocks = kColBlocksMax;
    if (n_blocks > L.max_wg) n_blocks = L.max_wg;
    const int rows_per_block = (T + n_blocks - 1) / n_blocks;
    n_blocks = (T + rows_per_block - 1) / rows_per_block;
    const size_t shm = (size_t)rowlanes * E * sizeof(double);
    if (vec == 4)
        hipLaunchKernelGGL(k_colsum<4>, dim3(n_blocks), dim3(256), shm, s, scores, T, E, cols, rows_per_block, part);
    else
        hipLaunchKernelGGL(k_colsum<1>, dim3(n_blocks), dim3(256), shm, s, scores, T, E, cols, rows_per_block, part);
    int epad = 1;
    while (epad < E) epad <<= 1;
    hipLaunchKernelGGL(k_aux_final, dim3(1), dim3(1024), 0, s, part, n_blocks, offsets, T, E, epad, lam, loss, mean_scores, dscores_col);
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

int32_t gates_backward_run(const float *logits, const float *scores, const int32_t *assign, const float *dgates,
                           const float *dscores_col, int T, int E, int k, float *dlogits, hipStream_t s)
{
#define MS_BWD(GG, PP) launch_bwd<GG, PP>(logits, scores, assign, dgates, dscores_col, T, E, k, dlogits, s)
    if (E <= 32) MS_BWD(8, 4);
    else if (E <= 64) MS_BWD(16, 4);
    else if (E <= 128) MS_BWD(16, 8);
    else if (E <= 256) MS_BWD(32, 8);
    else if (E <= 512) MS_BWD(64, 8);
    else MS_BWD(64, 16);
#undef MS_BWD
    MS_HIP(hipGetLastError());
    return MAXSCORE_OK;
}

}  // namespace maxscore
