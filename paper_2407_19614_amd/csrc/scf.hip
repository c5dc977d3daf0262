// SCF helpers on the GPU: Fock assembly, the DIIS error F D S - S D F and
// extrapolation (Pulay), spectral bounds and trace-correcting purification
// (Niklasson's TC2) giving the projector onto the n_occ lowest orbitals of an
// orthogonalised Fock matrix, and the energy terms.
#include "kernels.h"

#include <algorithm>

namespace {

inline unsigned nb(int64_t n) { int64_t g = (n + 255) / 256; return (unsigned)(g > 1048576 ? 1048576 : g); }

__global__ void fock_kernel(const double* h, const double* J, const double* K, double* F, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        F[i] = h[i] + J[i] - K[i];
}

struct Ptrs { const double* p[8]; };

// Two-stage, deterministic reductions over N^2-element matrices: the workgroups
// of a first launch each reduce a fixed share into a partial row of `red`, then
// one workgroup combines the partials in order.
constexpr int RED_BLOCKS = 256;

// sum of v over the 256 threads of a workgroup (fixed order)
__device__ __forceinline__ double wg_sum(double v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

struct Slots { int s[8]; };
struct MutPtrs { double* p[8]; };

// Where `red` holds what between the launches of one step: RED_BLOCKS rows of
// the energies' partial sums, then one row per 32 x 32 upper tile of the error
// (8 inner products and the maximum).
constexpr int RE = 3 * RED_BLOCKS, ROW = 9;
__host__ __device__ inline int err_tiles(int N) {
    const int nt = (N + 31) / 32;
    return nt * (nt + 1) / 2;
}

// F = h + J - K; partial[b] = (D.h, D.J, D.K) over block b's share
__global__ __launch_bounds__(256) void fock_energy_kernel(const double* __restrict__ h, const double* __restrict__ J,
                                                          const double* __restrict__ K, const double* __restrict__ D,
                                                          double* __restrict__ F, int64_t n,
                                                          double* __restrict__ red) {
    __shared__ double sh[4];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double d = D[i], hi = h[i], j = J[i], k = K[i];
        F[i] = hi + j - k;
        a += d * hi;
        b += d * j;
        c += d * k;
    }
    a = wg_sum(a, sh);
    b = wg_sum(b, sh);
    c = wg_sum(c, sh);
    if (threadIdx.x == 0) {
        red[blockIdx.x * 3 + 0] = a;
        red[blockIdx.x * 3 + 1] = b;
        red[blockIdx.x * 3 + 2] = c;
    }
}

// One upper 32 x 32 tile of e = M - M^T with its mirror -e^T, both written to the
// ring with the same entries of F, and the tile pair's sums.
__global__ __launch_bounds__(256) void error_push_kernel(const double* __restrict__ M, const double* __restrict__ F,
                                                         MutPtrs dE, double* __restrict__ dFnew, int m, int N,
                                                         double* __restrict__ red) {
    __shared__ double t1[32][33], t2[32][33], sh[4];
    const int nt = (N + 31) / 32;
    int I = 0, rem = blockIdx.x;
    while (rem >= nt - I) {
        rem -= nt - I;
        ++I;
    }
    const int J = I + rem, c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int r = r0 + 8 * k;
        t1[r][c] = (32 * I + r < N && 32 * J + c < N) ? M[(int64_t)(32 * I + r) * N + 32 * J + c] : 0.0;
        t2[r][c] = (32 * J + r < N && 32 * I + c < N) ? M[(int64_t)(32 * J + r) * N + 32 * I + c] : 0.0;
    }
    __syncthreads();
    double dot[8], big = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) dot[k] = 0.0;
    double* en = dE.p[m - 1];
    auto put = [&](int row, int col, double e) {
        if (row >= N || col >= N) return;
        const int64_t i = (int64_t)row * N + col;
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (k < m - 1) dot[k] += dE.p[k][i] * e;
        en[i] = e;
        dFnew[i] = F[i];
        dot[7] += e * e;
        big = fmax(big, fabs(e));
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int r = r0 + 8 * k;
        put(32 * I + r, 32 * J + c, t1[r][c] - t2[c][r]);
        if (I != J) put(32 * J + r, 32 * I + c, t2[r][c] - t1[c][r]);
    }
    double* out = red + RE + (int64_t)blockIdx.x * ROW;
#pragma unroll
    for (int k = 0; k < 8; ++k) {                  // slot 7: <e, e>
        if (k < m - 1 || k == 7) {
            const double v = wg_sum(dot[k], sh);
            if (threadIdx.x == 0) out[k] = v;
        }
    }
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_down(big, o));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = big;
    __syncthreads();
    if (threadIdx.x == 0) out[8] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// LDS writes of this wave are seen by its later reads
__device__ __forceinline__ void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The sums of one step, the DIIS matrix (row and column of the new slot into the
// slot-indexed Bfull) and the solution of [B -1; -1 0] [c; l] = [0; -1] by
// Gaussian elimination with partial pivoting, on the first wave: the matrix lies
// in LDS, a lane per element of an update (one thread with the matrix in
// scratch memory took 38 us).
__global__ __launch_bounds__(256) void step_finish_kernel(const double* __restrict__ red,
                                                          const double* __restrict__ enuc, double* __restrict__ scal,
                                                          double* __restrict__ Bfull, Slots sl, int m, int tiles,
                                                          double* __restrict__ coef) {
    __shared__ double sh[4], row[8], a[9][11], x[9];
    const int tid = threadIdx.x;
    double e3[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) e3[k] = wg_sum(red[tid * 3 + k], sh);
    for (int k = 0; k < 8; ++k) {
        if (k >= m - 1 && k != 7) continue;
        double v = 0.0;
        for (int t = tid; t < tiles; t += 256) v += red[RE + (int64_t)t * ROW + k];
        v = wg_sum(v, sh);
        if (tid == 0) row[k == 7 ? m - 1 : k] = v;
    }
    double big = 0.0;
    for (int t = tid; t < tiles; t += 256) big = fmax(big, red[RE + (int64_t)t * ROW + 8]);
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_down(big, o));
    __syncthreads();
    if ((tid & 63) == 0) sh[tid >> 6] = big;
    __syncthreads();
    if (tid == 0) {
        const double en = *enuc;
        scal[0] = e3[0] + 0.5 * e3[1] - 0.5 * e3[2] + en;   // E_total
        scal[1] = en;
        scal[2] = e3[0];                                    // E_1e
        scal[3] = 0.5 * e3[1];                              // E_J
        scal[4] = -0.5 * e3[2];                             // E_K
        scal[5] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    }
    if (tid < m) {
        Bfull[sl.s[m - 1] * 8 + sl.s[tid]] = row[tid];
        Bfull[sl.s[tid] * 8 + sl.s[m - 1]] = row[tid];
    }
    __syncthreads();
    if (m < 2 || tid >= 64) return;
    const int n = m + 1;
    for (int e = tid; e < n * (n + 1); e += 64) {
        const int i = e / (n + 1), j = e % (n + 1);
        a[i][j] = i < m && j < m   ? Bfull[sl.s[i] * 8 + sl.s[j]]
                  : i < m          ? (j == m ? -1.0 : 0.0)
                  : (j == m ? 0.0 : -1.0);
    }
    lds_wave_sync();
    for (int c = 0; c < n; ++c) {
        int piv = c;
        for (int r = c + 1; r < n; ++r)
            if (fabs(a[r][c]) > fabs(a[piv][c])) piv = r;
        if (piv != c && tid <= n) {
            const double t = a[c][tid];
            a[c][tid] = a[piv][tid];
            a[piv][tid] = t;
        }
        lds_wave_sync();
        double d = a[c][c];
        if (d == 0.0) d = 1e-300;
        // rows below c, columns right of c; the factors' column is not read again
        const int w = n - c, cnt = (n - 1 - c) * w;
        for (int e = tid; e < cnt; e += 64) {
            const int r = c + 1 + e / w, k = c + 1 + e % w;
            a[r][k] -= a[r][c] / d * a[c][k];
        }
        lds_wave_sync();
    }
    if (tid == 0) {
        for (int r = n - 1; r >= 0; --r) {
            double s = a[r][n];
            for (int k = r + 1; k < n; ++k) s -= a[r][k] * x[k];
            x[r] = s / (a[r][r] == 0.0 ? 1e-300 : a[r][r]);
        }
        for (int i = 0; i < m; ++i) coef[i] = x[i];
    }
}

__global__ void combine_kernel(Ptrs Fs, const double* coef, int m, double* out, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int k = 0; k < m; ++k) s += coef[k] * Fs.p[k][i];
        out[i] = s;
    }
}

// Gershgorin interval of each row r (one wave per row): red[2r] = F_rr - sum
// |F_rc|, red[2r + 1] = F_rr + sum |F_rc| over c != r.
__global__ __launch_bounds__(256) void gersh_rows_kernel(const double* F, int N, double* red) {
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= N) return;
    const double* row = F + (int64_t)r * N;
    double off = 0.0;
    for (int c = lane; c < N; c += 64)
        if (c != r) off += fabs(row[c]);
    for (int o = 32; o > 0; o >>= 1) off += __shfl_down(off, o);
    if (lane == 0) {
        red[2 * r] = row[r] - off;
        red[2 * r + 1] = row[r] + off;
    }
}

// Counter-based pseudo-random values in [-1, 1) (a 32-bit integer hash of
// the element index); any full-rank block serves as a subspace start.
__global__ void hash_kernel(double* R, int64_t n, uint32_t seed) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t x = (uint32_t)i * 2654435761u ^ seed;
        x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
        R[i] = (double)x * (2.0 / 4294967296.0) - 1.0;
    }
}

// partial[b] = (D.h, D.J, D.K) over block b's share
__global__ __launch_bounds__(256) void energy_part_kernel(const double* D, const double* h, const double* J,
                                                          const double* K, int64_t n, double* red) {
    __shared__ double sh[4];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double d = D[i];
        a += d * h[i];
        b += d * J[i];
        c += d * K[i];
    }
    a = wg_sum(a, sh);
    b = wg_sum(b, sh);
    c = wg_sum(c, sh);
    if (threadIdx.x == 0) {
        red[blockIdx.x * 3 + 0] = a;
        red[blockIdx.x * 3 + 1] = b;
        red[blockIdx.x * 3 + 2] = c;
    }
}

__global__ __launch_bounds__(256) void energy_final_kernel(const double* red, const double* enuc, double* out) {
    __shared__ double sh[4];
    const bool in = threadIdx.x < RED_BLOCKS;
    const double a = wg_sum(in ? red[threadIdx.x * 3 + 0] : 0.0, sh);
    const double b = wg_sum(in ? red[threadIdx.x * 3 + 1] : 0.0, sh);
    const double c = wg_sum(in ? red[threadIdx.x * 3 + 2] : 0.0, sh);
    if (threadIdx.x == 0) {
        const double en = *enuc;
        out[0] = a + 0.5 * b - 0.5 * c + en;   // E_total
        out[1] = en;
        out[2] = a;                            // E_1e
        out[3] = 0.5 * b;                      // E_J
        out[4] = -0.5 * c;                     // E_K
    }
}

}  // namespace

namespace ri {

hipError_t fock_assemble(const double* h, const double* J, const double* K, double* F, int64_t n, hipStream_t st) {
    fock_kernel<<<nb(n), 256, 0, st>>>(h, J, K, F, n);
    return hipGetLastError();
}
hipError_t fock_energy(const double* h, const double* J, const double* K, const double* D, double* F, int64_t n,
                       double* red, hipStream_t st) {
    fock_energy_kernel<<<RED_BLOCKS, 256, 0, st>>>(h, J, K, D, F, n, red);
    return hipGetLastError();
}
hipError_t error_push(const double* M, const double* F, double* const* dE, double* dFnew, const int* slots, int m,
                      int N, double* red, hipStream_t st) {
    if (m < 1 || m > 8) return hipErrorInvalidValue;
    MutPtrs e{};
    for (int k = 0; k < m; ++k) e.p[k] = dE[slots[k]];
    error_push_kernel<<<err_tiles(N), 256, 0, st>>>(M, F, e, dFnew, m, N, red);
    return hipGetLastError();
}
hipError_t step_finish(double* red, const double* enuc, double* scal, double* Bfull, const int* slots, int m, int N,
                       double* coef, hipStream_t st) {
    if (m < 1 || m > 8) return hipErrorInvalidValue;
    Slots sl{};
    for (int k = 0; k < m; ++k) sl.s[k] = slots[k];
    step_finish_kernel<<<1, 256, 0, st>>>(red, enuc, scal, Bfull, sl, m, err_tiles(N), coef);
    return hipGetLastError();
}
hipError_t diis_combine(const double* const* Fs, const double* coef, int m, double* out, int64_t n, hipStream_t st) {
    Ptrs p{};
    for (int i = 0; i < m; ++i) p.p[i] = Fs[i];
    combine_kernel<<<nb(n), 256, 0, st>>>(p, coef, m, out, n);
    return hipGetLastError();
}
hipError_t gershgorin_rows(const double* F, int N, double* rows, hipStream_t st) {
    gersh_rows_kernel<<<(N + 3) / 4, 256, 0, st>>>(F, N, rows);
    return hipGetLastError();
}
hipError_t hash_matrix(double* R, int64_t n, uint32_t seed, hipStream_t st) {
    hash_kernel<<<nb(n), 256, 0, st>>>(R, n, seed);
    return hipGetLastError();
}
hipError_t energy_terms(const double* D, const double* h, const double* J, const double* K, int64_t n,
                        const double* enuc, double* out, double* red, hipStream_t st) {
    energy_part_kernel<<<RED_BLOCKS, 256, 0, st>>>(D, h, J, K, n, red);
    RI_TRY(hipGetLastError());
    energy_final_kernel<<<1, 256, 0, st>>>(red, enuc, out);
    return hipGetLastError();
}

int red_elems(int N) { return std::max(RE + ROW * err_tiles(N), 2 * N); }

}  // namespace ri
