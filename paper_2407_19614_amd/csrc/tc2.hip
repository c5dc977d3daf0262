// Trace-correcting purification (Niklasson's TC2) of an orthogonalised Fock
// matrix, one launch per step, for the single-molecule SCF.
//
// A step maps X to X^2 or 2X - X^2, whichever brings the trace closer to
// n_occ, and both need tr X and tr X^2 of the step's input.  X stays exactly
// symmetric (the start is symmetrised and every step forms X X^T, whose
// (i, j) and (j, i) entries are the same products summed in the same order),
// so tr X^2 = sum_ij X_ij^2 is known before the product is formed: each step
// writes, per output tile, the partial sums of tr Y and sum Y_ij^2 of its
// output Y, and every workgroup of the next step sums those partials in one
// fixed order, so all of them take the same branch and the same stopping
// decision.  The stopping rule is the one the batched SCF uses: once
// |tr X - tr X^2| < 1e-11 n_occ, this step and one more run, and later steps
// exit at once, so the host can launch steps in chunks and read the state
// once per chunk instead of once every few steps.  (Near convergence a step
// squares the eigenvalues' distance to 0 or 1 on one side and at most
// doubles it on the other, so the two steps take a summed distance of
// 1e-11 n_occ down to rounding.)
//
// Layout of a step: X^2 is symmetric, so only the upper output tiles are
// formed and each is written with its mirror, which keeps X exactly symmetric
// by construction.  The eight waves of a workgroup (two per SIMD) take the
// eighths of the reduction index; each wave owns the whole tile as T x T FP64
// MFMA tiles and reads its operands straight from X: the A operand of row tile
// i is X[k][m0 + 16 i + ..] (a row of X, by symmetry) and the B operand of
// column tile j is X[k][n0 + 16 j + ..], so the 16 lanes of each group read
// 16 consecutive doubles.  Buffer loads return zero past the end of X (rows
// k >= N), and the operands of the k-step four ahead are in flight while a
// step's MFMAs run.  The partial tiles are summed through LDS in one fixed
// order, then the update, the tile and mirror writes and the partial sums run
// in the epilogue.
// T: a step is a short chain of latencies (state, operands, MFMAs, LDS, writes),
// so a single molecule takes the smallest tile whose count still fits the 256
// CUs in one round: 16 up to N = 352, 32 up to N = 704, 48 beyond (N = 1000: 231
// tiles).  The state and the partial sums of the traces are read beside the
// operands: they decide only the update.  Measured, per step: N = 32 6.0 -> 3.9
// us, N = 270 11.8 -> 6.9, N = 400 14.8 -> 10.7, N = 1000 unchanged.
#include "kernels.h"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace {

constexpr int PD = 4;         // k-steps of operands in flight

__host__ __device__ inline int n_tiles_edge(int N, int T) { return (N + 16 * T - 1) / (16 * T); }

// upper tile t (row-major over I <= J) of an nt x nt tiling
__device__ inline void upper_tile(int t, int nt, int& I, int& J) {
    int i = 0, rem = t;
    while (rem >= nt - i) {
        rem -= nt - i;
        ++i;
    }
    I = i;
    J = i + rem;
}

// state fields (int[8] per parity buffer)
constexpr int S_CD = 0, S_DONE = 1, S_STEPS = 2, S_LAST = 3;

// sums of a and b over the NT threads of the workgroup, in a fixed order, in
// thread 0
template <int NT>
__device__ __forceinline__ void wg_sum2(double& a, double& b, double (*sh)[2]) {
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_down(a, o);
        b += __shfl_down(b, o);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6][0] = a;
        sh[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    a = b = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        a += sh[i][0];
        b += sh[i][1];
    }
}

// X0 = (hi I - (F + F^T)/2) / (hi - lo) on upper tile t (written with its
// mirror), with the tile's partial sums of tr X0 and sum X0_ij^2 over the
// entries it stands for, and (t = 0) the purification state reset.  rows: the
// Gershgorin interval of each row of F, combined here by every workgroup.
template <int T>
__device__ __forceinline__ void tc2_init_body(int t, const double* __restrict__ F, const double* __restrict__ rows,
                                              int N, double* __restrict__ X, double* __restrict__ part,
                                              int* __restrict__ st) {
    constexpr int TT = 16 * T;
    __shared__ double sh[4][2], bd[4][2];
    const int tid = threadIdx.x;
    double lo = 1e300, hi = -1e300;
    for (int r = tid; r < N; r += 256) {
        lo = fmin(lo, rows[2 * r]);
        hi = fmax(hi, rows[2 * r + 1]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o));
        hi = fmax(hi, __shfl_xor(hi, o));
    }
    if ((tid & 63) == 0) {
        bd[tid >> 6][0] = lo;
        bd[tid >> 6][1] = hi;
    }
    __syncthreads();
    lo = fmin(fmin(bd[0][0], bd[1][0]), fmin(bd[2][0], bd[3][0]));
    hi = fmax(fmax(bd[0][1], bd[1][1]), fmax(bd[2][1], bd[3][1]));
    const double s = 1.0 / (hi - lo);
    int I, J;
    upper_tile(t, n_tiles_edge(N, T), I, J);
    double f2 = 0.0, tr = 0.0;
    for (int e = tid; e < TT * TT; e += 256) {
        const int r = TT * I + e / TT, c = TT * J + e % TT;
        if (r < N && c < N) {
            const double fs = 0.5 * (F[(int64_t)r * N + c] + F[(int64_t)c * N + r]);
            const double x = ((r == c ? hi : 0.0) - fs) * s;
            X[(int64_t)r * N + c] = x;
            if (I != J) X[(int64_t)c * N + r] = x;
            f2 += (I == J ? 1.0 : 2.0) * x * x;
            if (r == c) tr += x;
        }
    }
    wg_sum2<256>(tr, f2, sh);
    if (tid == 0) {
        part[2 * t] = tr;
        part[2 * t + 1] = f2;
    }
    if (t == 0 && tid < 8) st[tid] = tid == S_CD ? -1 : 0;
}

// One step on upper tile t of `tiles`: Y = X^2 or 2X - X^2.
template <int T>
__device__ __forceinline__ void tc2_step_body(int t, int tiles, const double* __restrict__ X, double* __restrict__ Y,
                                              int N, int n_occ, const double* __restrict__ part_in,
                                              double* __restrict__ part_out, const int* __restrict__ st_in,
                                              int* __restrict__ st_out, int out_id) {
    constexpr int TT = 16 * T, LDT = TT + 1;
    constexpr int SLOTS = T < 3 ? 8 : 4;           // partial tiles in LDS: one a wave, or waves w and w + 4 in slot w
    __shared__ double sh[8][2];
    __shared__ double red[SLOTS][TT][LDT];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: the resource below is a scalar
    const int done = st_in[S_DONE], cd0 = st_in[S_CD];
    // tr X and tr X^2 from the previous step's partial sums: every wave sums them
    // in the same order
    double t1 = 0.0, t2 = 0.0;
    for (int i = lane; i < tiles; i += 64) {
        t1 += part_in[2 * i];
        t2 += part_in[2 * i + 1];
    }
    int I, J;
    upper_tile(t, n_tiles_edge(N, T), I, J);
    const int m0 = TT * I, n0 = TT * J;
    const bool diag = I == J;
    // this wave's eighth of the reduction index, in whole 4-deep k-steps
    const int Kq = ((N + 7) / 8 + 3) / 4 * 4;
    const int kbeg = wave * Kq, kend = min(N, kbeg + Kq), nks = max(0, (kend - kbeg + 3) / 4);
    // buffer loads over this wave's rows of X (and the prefetch past them) with the
    // whole offset in the lane's offset: rows k >= N read as zero (range check)
    const int krows = max(0, min(N - kbeg, Kq + 4 * PD));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(X + (int64_t)kbeg * N), (short)0, krows * N * 8, 0x00020000);
    int vA[T], vB[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        vA[i] = (g * N + m0 + 16 * i + r) * 8;
        vB[i] = (g * N + n0 + 16 * i + r) * 8;
    }
    const int step = 4 * N * 8;
    d4_t acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    // a diagonal tile's panels coincide; false: the purification has ended
    auto accumulate = [&](auto dg) {
        constexpr bool DIAG = decltype(dg)::value;
        auto ld = [&](int s, double (&pa)[T], double (&pb)[T]) {
#pragma unroll
            for (int i = 0; i < T; ++i)
                pa[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, vA[i] + s * step, 0, 0));
            if (!DIAG) {
#pragma unroll
                for (int i = 0; i < T; ++i)
                    pb[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, vB[i] + s * step, 0, 0));
            }
        };
        double pa[PD][T], pb[PD][T];
#pragma unroll
        for (int p = 0; p < PD; ++p) ld(p, pa[p], pb[p]);
        if (__builtin_amdgcn_readfirstlane(done)) return false;
        for (int s0 = 0; s0 < nks; s0 += PD) {
#pragma unroll
            for (int p = 0; p < PD; ++p) {
                if (s0 + p < nks) {
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            acc[i][j] = mfma_f64(pa[p][i], DIAG ? pa[p][j] : pb[p][j], acc[i][j]);
                    ld(s0 + p + PD, pa[p], pb[p]);
                }
            }
        }
        return true;
    };
    if (!(diag ? accumulate(std::true_type{}) : accumulate(std::false_type{}))) {
        if (t == 0 && tid < 8) st_out[tid] = st_in[tid];
        return;
    }
    // the entries of X of a 2X - X^2 update, from clamped addresses
    constexpr int EP = (TT * TT + 511) / 512;
    double xo[EP];
#pragma unroll
    for (int q = 0; q < EP; ++q) {
        const int e = min(tid + 512 * q, TT * TT - 1), gm = min(m0 + e / TT, N - 1), gn = min(n0 + e % TT, N - 1);
        xo[q] = X[(int64_t)gm * N + gn];
    }
    for (int o = 32; o > 0; o >>= 1) {
        t1 += __shfl_xor(t1, o);
        t2 += __shfl_xor(t2, o);
    }
    int cd = cd0;
    if (cd < 0) {
        if (fabs(t1 - t2) < 1e-11 * (double)max(1, n_occ)) cd = 1;
    } else if (cd > 0) {
        --cd;
    }
    const bool sq = fabs(t2 - n_occ) < fabs(2.0 * t1 - t2 - n_occ);
    if (t == 0 && tid == 0) {
        st_out[S_CD] = cd;
        st_out[S_DONE] = cd == 0;                 // this step's update is the last
        st_out[S_STEPS] = st_in[S_STEPS] + 1;
        st_out[S_LAST] = out_id;
        for (int k = 4; k < 8; ++k) st_out[k] = st_in[k];
    }
    // partial tiles to LDS: element q of lane (c, g) in MFMA tile (i, j) is
    // row 16 i + 4 q + g, column 16 j + c
    if (SLOTS == 8 || wave >= 4) {
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) red[wave % SLOTS][16 * i + 4 * q + g][16 * j + r] = acc[i][j][q];
    }
    __syncthreads();
    if (SLOTS == 4) {                              // waves 0-3 add theirs to the slots of 4-7
        if (wave < 4) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) red[wave % SLOTS][16 * i + 4 * q + g][16 * j + r] += acc[i][j][q];
        }
        __syncthreads();
    }
    // sum of the slots in one fixed order, the update, the tile's write
    // (diagonal tiles: the upper triangle) and the partial sums
    double f2 = 0.0, tr = 0.0;
#pragma unroll
    for (int q = 0; q < EP; ++q) {
        const int e = tid + 512 * q;
        if (e < TT * TT) {
            const int rr = e / TT, cc = e % TT, gm = m0 + rr, gn = n0 + cc;
            double v = 0.0;
            if (gm < N && gn < N && (!diag || rr <= cc)) {
                double x2 = red[0][rr][cc];
#pragma unroll
                for (int k = 1; k < SLOTS; ++k) x2 += red[k][rr][cc];
                v = sq ? x2 : 2.0 * xo[q] - x2;
                Y[(int64_t)gm * N + gn] = v;
                f2 += (gm == gn ? 1.0 : 2.0) * v * v;
                if (gm == gn) tr += v;
            }
            red[0][rr][cc] = v;   // each element is read and rewritten by one thread
        }
    }
    wg_sum2<512>(tr, f2, sh);                      // its barrier also covers red[0]
    if (tid == 0) {
        part_out[2 * t] = tr;
        part_out[2 * t + 1] = f2;
    }
    // mirror: Y[n][m] = Y[m][n], read transposed from LDS so that the writes
    // run along rows of Y
#pragma unroll
    for (int q = 0; q < EP; ++q) {
        const int e = tid + 512 * q;
        if (e < TT * TT) {
            const int cc = e / TT, rr = e % TT, gm = m0 + rr, gn = n0 + cc;
            if (gm < N && gn < N && (diag ? rr < cc : true)) Y[(int64_t)gn * N + gm] = red[0][rr][cc];
        }
    }
}

template <int T>
__global__ __launch_bounds__(256) void tc2f_init_kernel(const double* __restrict__ F, const double* __restrict__ rows,
                                                        int N, double* __restrict__ X, double* __restrict__ part,
                                                        int* __restrict__ st) {
    tc2_init_body<T>(blockIdx.x, F, rows, N, X, part, st);
}

template <int T>
__global__ __launch_bounds__(512) void tc2f_step_kernel(const double* __restrict__ X, double* __restrict__ Y, int N,
                                                        int n_occ, const double* __restrict__ part_in,
                                                        double* __restrict__ part_out, const int* __restrict__ st_in,
                                                        int* __restrict__ st_out, int out_id) {
    const int tiles = gridDim.x;
    tc2_step_body<T>(xcd_remap(blockIdx.x, tiles), tiles, X, Y, N, n_occ, part_in, part_out, st_in, st_out, out_id);
}

// The latest X is in Y when the last step that ran wrote there: copy it back.
__global__ void tc2f_final_kernel(double* X, const double* Y, int64_t n, const int* st) {
    if (st[S_LAST] != 1) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        X[i] = Y[i];
}

// tile edge of a single molecule's steps, in MFMA tiles (see the head of this file)
int tile_edge(int N) { return N <= 352 ? 1 : N <= 704 ? 2 : 3; }

int tiles(int N, int T) {
    const int nt = n_tiles_edge(N, T);
    return nt * (nt + 1) / 2;
}

}  // namespace

namespace ri {

int tc2f_tiles(int N) { return tiles(N, tile_edge(N)); }

hipError_t tc2f_init(const double* F, const double* rows, int N, double* X, double* part, int* state, hipStream_t st) {
    const int n = tc2f_tiles(N);
    switch (tile_edge(N)) {
        case 1: tc2f_init_kernel<1><<<n, 256, 0, st>>>(F, rows, N, X, part, state); break;
        case 2: tc2f_init_kernel<2><<<n, 256, 0, st>>>(F, rows, N, X, part, state); break;
        default: tc2f_init_kernel<3><<<n, 256, 0, st>>>(F, rows, N, X, part, state); break;
    }
    return hipGetLastError();
}

hipError_t tc2f_step(const double* X, double* Y, int N, int n_occ, const double* part_in, double* part_out,
                     const int* st_in, int* st_out, int out_id, hipStream_t st) {
    // buffer offsets into a wave's rows of X and the prefetch past them are 32-bit
    if ((int64_t)(N / 8 + 8 * PD + 12) * N * 8 > INT_MAX) return hipErrorInvalidValue;
    const int n = tc2f_tiles(N);
#define STEP(T) tc2f_step_kernel<T><<<n, 512, 0, st>>>(X, Y, N, n_occ, part_in, part_out, st_in, st_out, out_id)
    switch (tile_edge(N)) {
        case 1: STEP(1); break;
        case 2: STEP(2); break;
        default: STEP(3); break;
    }
#undef STEP
    return hipGetLastError();
}

hipError_t tc2f_final(double* X, const double* Y, int N, const int* state, hipStream_t st) {
    const int64_t n = (int64_t)N * N;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 4096);
    tc2f_final_kernel<<<(unsigned)g, 256, 0, st>>>(X, Y, n, state);
    return hipGetLastError();
}

}  // namespace ri
