// The FP64 half-transform X^P = B^P C_occ over significant pairs only.
//
// The packed tiles hold every (mu, nu), but only the pairs that passed the
// screening are not zero: 14 % of them at N = 1000, 26 % at N = 400.  The
// zeros lie too finely spread for whole tiles to be skipped (78 % of the
// 16 x 16 blocks of the N = 1000 workload hold a pair), so here each row mu
// runs over its own list of partners nu:
//     X^P[mu][i] = sum over partners nu of B_c[P][pair(mu, nu)] C[nu][i].
// For one mu that is a matrix product with the auxiliary index P as its
// columns: rows i, columns P, reduction over the partner list, four partners
// to an MFMA.  Its operands are gathered rows, C[nu][..] and the transposed
// fitted tensor BcT[pair][P], both contiguous over the 16 lanes of a group,
// so nothing is padded but the list (to a multiple of 4).
// Measured (FP64 build, N = 1000, N_aux = 3000, n_occ = 100, 67,000 pairs): X
// 9.8 -> 3.1 ms beside the Coulomb part, which reads the same transposed copy
// and no longer needs a capped grid; laying the copy out takes 0.63 ms, the
// whole build 14.8 -> 8.6 ms.  N = 370: X 288 -> 133 us, the build 488 -> 425.
// The multiplications of the pairs alone would take 1.1 ms at N = 1000: the
// MFMAs wait for the gathered operands (46 % busy at N = 600).
#include "kernels.h"

#include <algorithm>

namespace {
// map[mu][nu] = map[nu][mu] = pair index (the map is set to -1 before)
__global__ void pair_map_sym_kernel(const int32_t* __restrict__ pairs, int64_t n_pairs, int N,
                                    int32_t* __restrict__ map) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    const int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    map[(int64_t)mu * N + nu] = (int32_t)q;
    map[(int64_t)nu * N + mu] = (int32_t)q;
}

// Partner list of each row (one wave per row), in ascending nu: entries
// (nu, pair), then dummies (0, n_pairs) up to the next multiple of 64 and for
// the two chunks of 64 that the look-ahead reads past it; BcT's row n_pairs is
// zero.
__global__ __launch_bounds__(256) void row_list_kernel(const int32_t* __restrict__ map, int N, int n_pairs, int lmax,
                                                       int2* __restrict__ list, int* __restrict__ cnt) {
    const int mu = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (mu >= N) return;
    int2* out = list + (int64_t)mu * lmax;
    int n = 0;
    for (int c = 0; c < N; c += 64) {
        const int nu = c + lane;
        const int q = nu < N ? map[(int64_t)mu * N + nu] : -1;
        const unsigned long long m = __ballot(q >= 0);
        if (q >= 0) out[n + __popcll(m & ((1ull << lane) - 1))] = make_int2(nu, q);
        n += __popcll(m);
    }
    const int end = (n + 63) / 64 * 64 + 128;
    for (int k = n + lane; k < end; k += 64) out[k] = make_int2(0, n_pairs);
    if (lane == 0) cnt[mu] = n;
}

// BcT[P / 64][q][P % 64] = Bc[P][q], zero for P >= n_aux and in row n_pairs.
// 64 x 64 blocks through LDS: 512 B runs on both sides, so bound by memory
// (2 x 8 n_aux n_pairs bytes).  Blocks of 64 auxiliaries keep the pairs of a
// row, which are neighbours in q, next to each other in memory.
__global__ __launch_bounds__(256) void bc_transpose_kernel(const double* __restrict__ Bc, int n_aux, int64_t n_pairs,
                                                           double* __restrict__ BcT) {
    __shared__ double t[64][65];
    const int64_t q0 = (int64_t)blockIdx.x * 64;
    const int P0 = blockIdx.y * 64, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int P = P0 + 4 * r + w;
        v[r] = (P < n_aux && q0 + lane < n_pairs) ? Bc[(int64_t)P * n_pairs + q0 + lane] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) t[4 * r + w][lane] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t q = q0 + 4 * r + w;
        if (q <= n_pairs) BcT[(blockIdx.y * (n_pairs + 1) + q) * 64 + lane] = t[lane][4 * r + w];
    }
}

// Rows (P, i) of X^T for WV consecutive mu (one per wave) and 16 PT auxiliary
// indices.  Per step of 4 partners a wave issues MF PT 16x16x4 MFMAs and
// TQ PT 4x4x4 ones (the 4-row quads of an occupied count that is not a
// multiple of 16) on operands loaded XD steps ahead straight into registers.
// Lane (li, g) takes partner g of the step; a 16-byte load covers two
// occupied rows (tile pair: rows 32 m + 2 li + h) or two auxiliaries (column
// PT li + t of tile t), so a step costs 3-4 loads of C and PT / 2 of BcT.
// The waves meet only at the end, where each 16 x 16 result goes through
// LDS so that a row of X^T is written WV mu at a time.
template <int MF, int TQ, int PT, int XD, int WV>
__global__ __launch_bounds__(64 * WV, 2) void xs_kernel(const double* __restrict__ BcT, int64_t n_pairs,
                                                    const int2* __restrict__ list, const int* __restrict__ cnt,
                                                    int lmax, const double* __restrict__ Cp, int cld, int N,
                                                    int n_occ, int n_aux, int i0, double* __restrict__ Xt, int Npad) {
    constexpr int NA = MF + (TQ ? 1 : 0);
    static_assert(16 % XD == 0, "a chunk holds whole rounds");
    constexpr int LS = 16 * 17 + 4;                // one wave's 16 x 16 result in LDS
    __shared__ double Ls[2][WV * LS];
    const int no = (N + WV - 1) / WV;              // groups of WV rows
    const int L = xcd_remap(blockIdx.x, gridDim.x);
    const int mu0 = WV * (L % no), P0 = 16 * PT * (L / no);
    const int i1 = i0 + 128 * blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mu = mu0 + wave;
    d4_t acc[MF > 0 ? MF : 1][PT];
    double accq[TQ > 0 ? TQ : 1][PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
#pragma unroll
        for (int m = 0; m < MF; ++m) acc[m][t] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < TQ; ++q) accq[q][t] = 0.0;
    }
    if (mu < N) {
        const int2* ent = list + (int64_t)mu * lmax + lane;   // 64 entries, 16 steps, a chunk
        const double* bp = BcT + (int64_t)(P0 >> 6) * (n_pairs + 1) * 64 + (P0 & 63) + PT * li;
        const double* cp = Cp + i1;
        auto load = [&](int nu, int q, double (&a)[NA], double (&b)[PT]) {
            const double* c = cp + (int64_t)nu * cld;
            const double* r = bp + (int64_t)q * 64;
#pragma unroll
            for (int t = 0; t < PT; t += 2) {
                const d2_t v = *(const d2_t*)(r + t);
                b[t] = v[0];
                b[t + 1] = v[1];
            }
#pragma unroll
            for (int m = 0; m + 1 < MF; m += 2) {
                const d2_t v = *(const d2_t*)(c + 16 * m + 2 * li);
                a[m] = v[0];
                a[m + 1] = v[1];
            }
            if (MF & 1) a[MF - 1] = c[16 * (MF - 1) + li];
            if (TQ) a[NA - 1] = c[16 * MF + li];
        };
        auto mul = [&](const double (&a)[NA], const double (&b)[PT]) {
#pragma unroll
            for (int m = 0; m < MF; ++m)
#pragma unroll
                for (int t = 0; t < PT; ++t) acc[m][t] = mfma_f64(a[m], b[t], acc[m][t]);
            // a quad's A operand (row lane % 4) from the lanes that hold its rows
#pragma unroll
            for (int q = 0; q < TQ; ++q) {
                const double aq = __shfl(a[NA - 1], (lane & 48) + 4 * q + (lane & 3));
#pragma unroll
                for (int t = 0; t < PT; ++t)
                    accq[q][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(aq, b[t], accq[q][t], 0, 0, 0);
            }
        };
        const int nst = (__builtin_amdgcn_readfirstlane(cnt[mu]) + 3) / 4;
        double a[XD][NA], b[XD][PT];
        int2 e = ent[0], en = ent[64];
#pragma unroll
        for (int d = 0; d < XD; ++d) {
            load(__shfl(e.x, 4 * d + g), __shfl(e.y, 4 * d + g), a[d], b[d]);
            __builtin_amdgcn_sched_barrier(0);     // the loads stay in the order they are waited for
        }
        for (int s = 0; s < nst; s += XD) {
            if (((s + XD) & 15) == 0) {            // the steps loaded below start a new chunk
                e = en;
                en = ent[(s + XD) * 4 + 64];
            }
            const int k0 = 4 * ((s + XD) & 15) + g;
#pragma unroll
            for (int d = 0; d < XD; ++d) {
                if (s + d < nst) mul(a[d], b[d]);
                load(__shfl(e.x, k0 + 4 * d), __shfl(e.y, k0 + 4 * d), a[d], b[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // element q of lane (li, g) in tile m: row 4 q + g of the tile, column li
    auto put = [&](int buf, d4_t v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) Ls[buf][wave * LS + (4 * q + g) * 17 + li] = v[q];
    };
    // rows (P, i) of one result, WV mu each: i = ib + is * row, P = P0 + PT * p + t
    constexpr int LG = WV == 8 ? 3 : 2;
    const int u = tid & (WV - 1), row = (tid >> LG) & 15, p0 = tid >> (LG + 4);   // p = p0 + 4 k
    const bool in_mu = mu0 + u < N;
    auto get = [&](int buf, int rows, int ib, int is, int t) {
        double* out = Xt + ((int64_t)(P0 + t) * n_occ + ib) * Npad + mu0;
        const int i = ib + is * row;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int p = p0 + 4 * k;
            if (row < rows && i < n_occ && P0 + PT * p + t < n_aux && in_mu)
                out[(int64_t)(PT * p * n_occ + is * row) * Npad + u] = Ls[buf][u * LS + row * 17 + p];
        }
    };
    int buf = 0;
#pragma unroll
    for (int m = 0; m < MF; ++m) {
        const bool pair = m < MF / 2 * 2;
        const int ib = i1 + (pair ? 16 * (m & ~1) + (m & 1) : 16 * m);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            put(buf, acc[m][t]);
            __syncthreads();
            get(buf, 16, ib, pair ? 2 : 1, t);
            buf ^= 1;                              // the next result's barrier covers these reads
        }
    }
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            Ls[buf][wave * LS + g * 17 + li] = accq[q][t];
            __syncthreads();
            get(buf, 4, i1 + 16 * MF + 4 * q, 1, t);
            buf ^= 1;
        }
}

template <int MF, int TQ>
hipError_t xs_launch(const ri::XSparse& w, dim3 grid, const double* Cp, int cld, int N, int n_occ, int n_aux, int i0,
                     double* Xt, int Npad, hipStream_t st) {
    constexpr int PT = 2, XD = MF <= 2 ? 4 : 2, WV = 8;
    const unsigned blocks = (unsigned)((N + WV - 1) / WV) * (unsigned)((n_aux + 16 * PT - 1) / (16 * PT));
    xs_kernel<MF, TQ, PT, XD, WV><<<dim3(blocks, grid.y), 64 * WV, 0, st>>>(w.BcT, w.n_pairs, w.list, w.cnt, w.lmax, Cp, cld, N,
                                                                    n_occ, n_aux, i0, Xt, Npad);
    return hipGetLastError();
}

// gamma partials over a strip of pairs: gpart[strip][P] = sum_q dp[q] BcT[q][P],
// lanes along P.  One wave per (strip, 64 auxiliaries).
constexpr int GSTRIP = 256;
__global__ __launch_bounds__(256) void gamma_strip_kernel(const double* __restrict__ BcT, int64_t n_pairs, int nblk,
                                                          const double* __restrict__ dp, double* __restrict__ gpart) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int blk = blockIdx.x % nblk;
    const int64_t strip = blockIdx.x / nblk, q0 = strip * GSTRIP;
    __shared__ double sh[4][64];
    const int64_t a = q0 + wave * (GSTRIP / 4), z = min(n_pairs, a + GSTRIP / 4);
    const double* row = BcT + ((int64_t)blk * (n_pairs + 1) + a) * 64 + lane;
    double s = 0.0;
    int64_t q = a;
    for (; q + 8 <= z; q += 8, row += 512) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = row[64 * k];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += v[k] * dp[q + k];
    }
    for (; q < z; ++q, row += 64) s += *row * dp[q];
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0) gpart[strip * nblk * 64 + blk * 64 + lane] = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
}

// gamma[P] = sum of the strips in order, 16 auxiliaries per workgroup (16
// interleaved partial sums each); gpad is gamma zero-padded to whole blocks
__global__ __launch_bounds__(256) void gamma_sum_kernel(const double* __restrict__ gpart, int64_t strips, int ldp,
                                                        int n_aux, double* __restrict__ gamma,
                                                        double* __restrict__ gpad) {
    __shared__ double sh[16][17];
    const int p = threadIdx.x & 15, k = threadIdx.x >> 4, P = blockIdx.x * 16 + p;
    double s = 0.0;
    for (int64_t z = k; z < strips; z += 16) s += gpart[z * ldp + P];
    sh[k][p] = s;
    __syncthreads();
    if (k == 0) {
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) t += sh[j][p];
        gpad[P] = t;
        if (P < n_aux) gamma[P] = t;
    }
}

// J of a pair: sum_P gamma_P BcT[q][P], one wave per 16 pairs, lanes along P;
// written to both mirror positions.
constexpr int JQ = 16;
__global__ __launch_bounds__(256) void j_rows_kernel(const double* __restrict__ BcT, int64_t n_pairs, int nblk,
                                                     const double* __restrict__ gpad,
                                                     const int32_t* __restrict__ pairs, int N,
                                                     double* __restrict__ J) {
    const int lane = threadIdx.x & 63;
    const int64_t q0 = (blockIdx.x * 4ll + (threadIdx.x >> 6)) * JQ;
    if (q0 >= n_pairs) return;
    double s[JQ];
#pragma unroll
    for (int k = 0; k < JQ; ++k) s[k] = 0.0;
    for (int b = 0; b < nblk; ++b) {
        const double g = gpad[64 * b + lane];
        const double* row = BcT + ((int64_t)b * (n_pairs + 1) + q0) * 64 + lane;
#pragma unroll
        for (int k = 0; k < JQ; ++k) s[k] += g * row[64 * min((int64_t)k, n_pairs - q0)];   // row n_pairs is zero
    }
    double mine = 0.0;
#pragma unroll
    for (int k = 0; k < JQ; ++k) {
        double v = s[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        mine = lane == k ? v : mine;
    }
    if (lane < JQ && q0 + lane < n_pairs) {
        const int mu = pairs[2 * (q0 + lane)], nu = pairs[2 * (q0 + lane) + 1];
        J[(int64_t)mu * N + nu] = mine;
        J[(int64_t)nu * N + mu] = mine;
    }
}

}  // namespace

namespace ri {

bool xs_wanted(int N, int n_aux, int n_occ, int64_t n_pairs) {
    return n_pairs > 0 && (n_pairs + 1) * xs_ldp(n_aux) <= ((int64_t)1 << 33) && (double)(2 * n_pairs - N) <= 0.6 * (double)N * N &&
           xt_rows(n_aux, n_occ) * xt_ld(N) * 8 > (int64_t)RI_NOALLOC_SCRATCH_BYTES;
}

int xs_ldp(int n_aux) { return (n_aux + 63) / 64 * 64; }
int xs_lmax(int N) { return (N + 63) / 64 * 64 + 128; }

hipError_t xs_lists(const XSparse& w, const int32_t* pairs, int64_t n_pairs, int N, hipStream_t st) {
    RI_TRY(fill_i32(w.map, -1, (int64_t)N * N, st));
    pair_map_sym_kernel<<<(unsigned)((n_pairs + 255) / 256), 256, 0, st>>>(pairs, n_pairs, N, w.map);
    RI_TRY(hipGetLastError());
    row_list_kernel<<<(N + 3) / 4, 256, 0, st>>>(w.map, N, (int)n_pairs, w.lmax, w.list, w.cnt);
    return hipGetLastError();
}

hipError_t xs_rows(const XSparse& w, const double* Bc, int64_t n_pairs, int np, hipStream_t st) {
    bc_transpose_kernel<<<dim3((unsigned)(n_pairs / 64 + 1), xs_ldp(np) / 64), 256, 0, st>>>(Bc, np, n_pairs, w.BcT);
    return hipGetLastError();
}

hipError_t xs_prepare(const XSparse& w, const double* Bc, const int32_t* pairs, int64_t n_pairs, int N, int n_aux,
                      hipStream_t st) {
    RI_TRY(xs_lists(w, pairs, n_pairs, N, st));
    return xs_rows(w, Bc, n_pairs, n_aux, st);
}

int64_t xs_gpart(int n_aux, int64_t n_pairs) { return ((n_pairs + GSTRIP - 1) / GSTRIP + 1) * xs_ldp(n_aux); }

hipError_t xs_gamma_j(const XSparse& w, int N, int n_aux, const double* dpair, const int32_t* pairs, double* gamma,
                      double* J, hipStream_t st) {
    const int nblk = w.ldp / 64;
    const int64_t strips = (w.n_pairs + GSTRIP - 1) / GSTRIP;
    double* gpad = w.gpart + strips * w.ldp;
    gamma_strip_kernel<<<(unsigned)(strips * nblk), 256, 0, st>>>(w.BcT, w.n_pairs, nblk, dpair, w.gpart);
    RI_TRY(hipGetLastError());
    gamma_sum_kernel<<<w.ldp / 16, 256, 0, st>>>(w.gpart, strips, w.ldp, n_aux, gamma, gpad);
    RI_TRY(hipGetLastError());
    if (!J) return hipSuccess;
    RI_TRY(fill(J, 0.0, (int64_t)N * N, st));
    j_rows_kernel<<<(unsigned)((w.n_pairs + 4 * JQ - 1) / (4 * JQ)), 256, 0, st>>>(w.BcT, w.n_pairs, nblk, gpad, pairs,
                                                                                  N, J);
    return hipGetLastError();
}

hipError_t xs_transform(const XSparse& w, int N, int n_aux, int n_occ, const double* C, double* Cp, double* Xt,
                        hipStream_t st) {
    RI_TRY(cpad(C, N, n_occ, Cp, st));
    return xs_run(w, N, n_aux, n_occ, Cp, Xt, st);
}

hipError_t xs_run(const XSparse& w, int N, int n_aux, int n_occ, const double* Cp, double* Xt, hipStream_t st) {
    const int cld = cpad_ld(n_occ), Npad = xt_ld(N);
    // whole chunks of 128 occupied columns, then what is left: whole 16-row
    // tiles plus, when the last tile would hold 12 rows or fewer, 4-row quads
    const int full = n_occ / 128, left = n_occ % 128;
    if (full > 0) RI_TRY((xs_launch<8, 0>(w, dim3(1, full), Cp, cld, N, n_occ, n_aux, 0, Xt, Npad, st)));
    if (left == 0) return hipSuccess;
    const int mt = (left + 15) / 16, rem = left - 16 * (mt - 1);
    const int mf = rem <= 12 ? mt - 1 : mt, tq = rem <= 12 ? (rem + 3) / 4 : 0;
    switch (4 * mf + tq) {
#define XS(f, q) case 4 * f + q: return xs_launch<f, q>(w, dim3(1, 1), Cp, cld, N, n_occ, n_aux, 128 * full, Xt, Npad, st);
#define XSROW(f) XS(f, 1) XS(f, 2) XS(f, 3)
        XSROW(0) XSROW(1) XSROW(2) XSROW(3) XSROW(4) XSROW(5) XSROW(6) XSROW(7)
        XS(1, 0) XS(2, 0) XS(3, 0) XS(4, 0) XS(5, 0) XS(6, 0) XS(7, 0) XS(8, 0)
#undef XSROW
#undef XS
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ri
