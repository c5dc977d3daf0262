// Exchange from a density matrix alone (no occupied orbitals), as needed by
// a density start of the SCF: K = 1/2 sum_P B^P D B^P, the RI form of the
// exchange operator for any symmetric D.  By slabs of auxiliaries:
// (D B^P)[i][mu], rows (P, i), over each row's significant partners (the
// exchange half-transform with D in the place of the orbitals), the full
// square B^P unpacked as rows (P, sigma), and the lower tiles of the product
// of the two over all rows, in the SYRK's kernel.  The products are 2 N^2 N_aux
// times the mean number of partners plus N^3 N_aux flops, where two dense
// GEMMs took 4 N^3 N_aux; bound by FP64 MFMA throughput.  The second GEMM had
// only the tiles of one N x N matrix to run on.  Measured, whole build: N =
// 400, N_aux = 1200: 39.0 -> 5.1 ms (product 2.4, D B^P 1.4, unpacking 0.9); N
// = 130: 5.6 -> 0.38 ms.
#include "kernels.h"

#include <algorithm>

namespace {

// Bf[p][mu][nu] = B_c[p][pair(mu, nu)] or 0, rows of ld; and `tail` rows of zeros
// after the last one of Bf and of Y, which k_product reads
__global__ void unpack_full_kernel(const double* __restrict__ Bc, int64_t n_pairs, const int32_t* __restrict__ map,
                                   int N, int ld, int tail, double* __restrict__ Bf, double* __restrict__ Y) {
    const int nu = blockIdx.x * blockDim.x + threadIdx.x, mu = blockIdx.y, p = blockIdx.z;
    if (nu >= ld) return;
    if (p == 0)
        for (int64_t t = mu; t < tail; t += N) {
            const int64_t e = ((int64_t)gridDim.z * N + t) * ld + nu;
            Bf[e] = 0.0;
            Y[e] = 0.0;
        }
    const int32_t q = nu < N ? map[(int64_t)mu * N + nu] : -1;
    Bf[((int64_t)p * N + mu) * ld + nu] = q >= 0 ? Bc[(int64_t)p * n_pairs + q] : 0.0;
}

// Dp = (D + D^T) / 2, zero-padded to [rows][ld]
__global__ void pad_symmetric_kernel(const double* __restrict__ D, int N, int rows, int ld, double* __restrict__ Dp) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)rows * ld) return;
    const int r = (int)(e / ld), c = (int)(e % ld);
    Dp[e] = (r < N && c < N) ? 0.5 * (D[(int64_t)r * N + c] + D[(int64_t)c * N + r]) : 0.0;
}

}  // namespace

namespace ri {

// Auxiliaries a slab: whole blocks of 64, as many as keep the slab's B^P and
// D B^P at 512 MiB each, so that a slab's launches fill the chip at small N; above
// N = 1024 a block of 64, halved while it takes more than 1 GiB (32 from N =
// 1450 on, 8 from N = 2890 on).
int density_slab(int N, int n_aux) {
    const int64_t per = (int64_t)N * xt_ld(N) * 8;
    int64_t want = (int64_t(1) << 29) / (64 * per) * 64;
    if (want == 0)
        for (want = 64; want > DENSITY_SLAB_MIN && want * per > (int64_t(1) << 30);) want /= 2;
    return (int)std::min<int64_t>({want, n_aux, 32768});   // a grid dimension takes 65535
}

int density_slab_below(int slab) { return slab > 64 ? (slab - 1) / 64 * 64 : slab / 2; }

hipError_t k_density(const double* Bc, const int32_t* pairs, int64_t n_pairs, int N, int n_aux, const double* D,
                     const KDensity& w, double* K, hipStream_t st) {
    if (n_pairs == 0) return fill(K, 0.0, (int64_t)N * N, st);
    const int ld = xt_ld(N), cld = cpad_ld(N), rows = n_tiles_1d(N) * 64;
    RI_TRY(xs_lists(w.xs, pairs, n_pairs, N, st));
    pad_symmetric_kernel<<<(unsigned)(((int64_t)rows * cld + 255) / 256), 256, 0, st>>>(D, N, rows, cld, w.Dp);
    RI_TRY(hipGetLastError());
    int used = 0;
    for (int P0 = 0; P0 < n_aux; P0 += w.slab) {
        const int s = std::min(w.slab, n_aux - P0);
        const double* b = Bc + (int64_t)P0 * n_pairs;
        RI_TRY(xs_rows(w.xs, b, n_pairs, s, st));
        RI_TRY(xs_run(w.xs, N, s, N, w.Dp, w.Y, st));
        const int64_t rows_s = (int64_t)s * N;
        unpack_full_kernel<<<dim3((ld + 255) / 256, N, s), 256, 0, st>>>(b, n_pairs, w.xs.map, N, ld,
                                                                         (int)(xt_rows(s, N) - rows_s), w.Bf, w.Y);
        RI_TRY(hipGetLastError());
        // every slab has the same number of splits, so that each adds to what the first wrote
        int u = 0;
        RI_TRY(k_product(w.Bf, w.Y, rows_s, N, w.part, P0 == 0 ? w.ks : used, P0 > 0, &u, st));
        used = std::max(used, u);
    }
    return kreduce(w.part, used, N, 0.5, K, st);
}

}  // namespace ri
