// FP64 products of the size of one molecule's matrices in the SCF step, where
// a 64 x 64-tiled GEMM has a few dozen workgroups that each walk the whole
// reduction (N = 270: 25 tiles, 15-20 us; N x n_occ blocks: 5 tiles).
#include "kernels.h"

#include <algorithm>
#include <climits>

namespace {

// C = alpha op(A) op(B) on 16 T x 16 T tiles, one per workgroup of 8 waves.
// Each wave takes every eighth block of 8 reduction indices over the whole
// tile, with operands read straight from memory two blocks ahead (a lane in
// group g takes indices 8 u + 2 g and + 1, so an operand whose rows run along
// the reduction is read 16 B at a time), and the eight partial tiles are summed
// through LDS in a fixed order.  Bound by latency: a tile is one chain of
// K / 64 blocks.  Buffer loads return zero past the end of a matrix; reduction
// indices past K and, for tri, past the triangle's edge are zeroed in both
// operands.  tri as for gemm_f64 (1 op(A) lower, 2 op(A) upper, 3 op(B) upper).
// T = 1 while its tiles fit two rounds of the 256 CUs, else T = 2 while they
// do.  Measured, N = 270, n_occ = 27: N x N x N 15.3 -> 5.1 us, the occupied
// blocks 15-20 -> 4 us.
template <bool TA, bool TB, int T>
__global__ __launch_bounds__(512) void gemm_split_kernel(int M, int N, int K, double alpha,
                                                         const double* __restrict__ A, int lda,
                                                         const double* __restrict__ B, int ldb,
                                                         double* __restrict__ C, int ldc, int tri) {
    constexpr int E = 16 * T;
    __shared__ double red[8][E][E + 1];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = E * blockIdx.y, n0 = E * blockIdx.x;
    int kbeg = 0, kend = K;
    if (tri == 1) kend = min(K, m0 + E);
    if (tri == 2) kbeg = m0 / 8 * 8;
    if (tri == 3) kend = min(K, n0 + E);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(A), (short)0, (TA ? (K - 1) * lda + M : (M - 1) * lda + K) * 8, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(B), (short)0, (TB ? (N - 1) * ldb + K : (K - 1) * ldb + N) * 8, 0x00020000);
    // two reduction indices k, k + 1 of one row of an operand
    auto get = [](__amdgpu_buffer_rsrc_t rs, bool along, int row, int k, int ld) {
        d2_t v;
        if (along) {
            v = __builtin_bit_cast(d2_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (row * ld + k) * 8, 0, 0));
        } else {
            v[0] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (k * ld + row) * 8, 0, 0));
            v[1] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, ((k + 1) * ld + row) * 8, 0, 0));
        }
        return v;
    };
    auto load = [&](int u, d2_t (&a)[T], d2_t (&b)[T]) {
        const int k = kbeg + 8 * u + 2 * g;
#pragma unroll
        for (int i = 0; i < T; ++i) {
            a[i] = get(ra, !TA, min(m0 + 16 * i + r, M - 1), k, lda);
            b[i] = get(rb, TB, min(n0 + 16 * i + r, N - 1), k, ldb);
        }
    };
    d4_t acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    const int nu = max(0, (kend - kbeg + 7) / 8);
    constexpr int D = 3;                           // blocks in flight
    d2_t a[D][T], b[D][T];
#pragma unroll
    for (int d = 0; d < D; ++d) load(wave + 8 * d, a[d], b[d]);
    for (int u0 = wave; u0 < nu; u0 += 8 * D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int u = u0 + 8 * d;
            if (u < nu) {
                const int k = kbeg + 8 * u + 2 * g;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool in = k + h < kend;
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            acc[i][j] = mfma_f64(in ? a[d][i][h] : 0.0, in ? b[d][j][h] : 0.0, acc[i][j]);
                }
                load(u + 8 * D, a[d], b[d]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) red[wave][16 * i + 4 * q + g][16 * j + r] = acc[i][j][q];
    __syncthreads();
    for (int e = tid; e < E * E; e += 512) {
        const int rr = e / E, cc = e % E;
        double v = red[0][rr][cc];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += red[w][rr][cc];
        if (m0 + rr < M && n0 + cc < N) C[(int64_t)(m0 + rr) * ldc + n0 + cc] = alpha * v;
    }
}

template <bool TA, bool TB>
void launch_split(int M, int N, int K, double alpha, const double* A, int lda, const double* B, int ldb, double* C,
                  int ldc, int tri, int T, hipStream_t s) {
    const dim3 grid((N + 16 * T - 1) / (16 * T), (M + 16 * T - 1) / (16 * T));
    if (T == 1) gemm_split_kernel<TA, TB, 1><<<grid, 512, 0, s>>>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri);
    else gemm_split_kernel<TA, TB, 2><<<grid, 512, 0, s>>>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri);
}

// Inverse of the Cholesky factor of an n x n Gram matrix, n <= 64, on one wave;
// a non-positive pivot's index is atomically min-ed into *bad.
__global__ __launch_bounds__(64) void chol_small_kernel(const double* __restrict__ A, int n, double* __restrict__ Linv,
                                                        int* __restrict__ bad) {
    __shared__ double S[64][65];
    const int lane = threadIdx.x;
    for (int r0 = 0; r0 < 64; r0 += 16) {
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = r0 + i;
            v[i] = (r < n && lane < n) ? A[(int64_t)r * n + lane] : (r == lane ? 1.0 : 0.0);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) S[r0 + i][lane] = v[i];
    }
    __syncthreads();
    chol_inv64_blocked(S, n, [&](int j) { atomicMin(bad, j); },
                       [&](int i, int c, double v) {
                           if (i < n && c < n) Linv[(int64_t)i * n + c] = v;
                       });
}

}  // namespace

namespace ri {

hipError_t gemm_scf(bool ta, bool tb, int M, int N, int K, double alpha, const double* A, int lda, const double* B,
                    int ldb, double* C, int ldc, int tri, hipStream_t s) {
    auto tiles = [&](int e) { return (int64_t)((M + e - 1) / e) * ((N + e - 1) / e); };
    const int64_t a = (int64_t)(ta ? K : M) * lda * 8, b = (int64_t)(tb ? N : K) * ldb * 8;
    const int T = tiles(16) <= 512 ? 1 : tiles(32) <= 512 ? 2 : 0;
    // the prefetch reaches 200 rows past the end: offsets must stay 32-bit
    if (T == 0 || a + 200ll * lda * 8 > INT_MAX || b + 200ll * ldb * 8 > INT_MAX)
        return gemm_f64(ta, tb, M, N, K, alpha, A, lda, 0, B, ldb, 0, 0.0, C, ldc, 0, 1, tri, 0, s);
    if (!ta && !tb) launch_split<false, false>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri, T, s);
    else if (!ta) launch_split<false, true>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri, T, s);
    else if (!tb) launch_split<true, false>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri, T, s);
    else launch_split<true, true>(M, N, K, alpha, A, lda, B, ldb, C, ldc, tri, T, s);
    return hipGetLastError();
}

hipError_t chol_small(const double* A, int n, double* Linv, int* bad, hipStream_t s) {
    if (n > 64) return hipErrorInvalidValue;
    chol_small_kernel<<<1, 64, 0, s>>>(A, n, Linv, bad);
    return hipGetLastError();
}

}  // namespace ri
