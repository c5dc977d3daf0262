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

// Partner list of one row, by one wave, in ascending nu: entries (nu, pair),
// then dummies (0, n_pairs) up to the next multiple of 64 and for the two chunks
// of 64 that the look-ahead reads past it; BcT's row n_pairs is zero.
// SEG (the FP32 form): each block of 64 nu is padded to whole steps of 4 and
// bit 31 of the first entry of its last step says that the FP32 sum of the
// block ends there.  Returns the number of entries.
template <bool SEG>
__device__ __forceinline__ int row_list(const int32_t* __restrict__ map, int mu, int N, int n_pairs,
                                        int2* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    int n = 0;
    for (int c = 0; c < N; c += 64) {
        const int nu = c + lane;
        const int q = nu < N ? map[(int64_t)mu * N + nu] : -1;
        const unsigned long long m = __ballot(q >= 0);
        const int k = __popcll(m & ((1ull << lane) - 1)), all = __popcll(m);
        if (!SEG) {
            if (q >= 0) out[n + k] = make_int2(nu, q);
            n += all;
        } else if (all > 0) {
            const int pad = (all + 3) / 4 * 4, last = pad - 4;
            if (q >= 0) out[n + k] = make_int2(k == last ? nu | (int)0x80000000 : nu, q);
            if (lane >= all && lane < pad) out[n + lane] = make_int2(0, n_pairs);
            n += pad;
        }
    }
    const int end = (n + 63) / 64 * 64 + 128;
    for (int k = n + lane; k < end; k += 64) out[k] = make_int2(0, n_pairs);
    return n;
}

template <bool SEG>
__global__ __launch_bounds__(256) void row_list_kernel(const int32_t* __restrict__ map, int N, int n_pairs, int lmax,
                                                       int2* __restrict__ list, int* __restrict__ cnt) {
    const int mu = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (mu >= N) return;
    const int n = row_list<SEG>(map, mu, N, n_pairs, list + (int64_t)mu * lmax);
    if ((threadIdx.x & 63) == 0) cnt[mu] = n;
}

// BcT[P / 64][q][P % 64] = Bc[P][q], zero for P >= n_aux and in row n_pairs.
// 64 x 64 blocks through LDS: 512 B runs on both sides, so bound by memory
// (2 x 8 n_aux n_pairs bytes).  Blocks of 64 auxiliaries keep the pairs of a
// row, which are neighbours in q, next to each other in memory.
// TB float: the value rounded, as the FP32 packing does.
template <typename TB>
__global__ __launch_bounds__(256) void bc_transpose_kernel(const double* __restrict__ Bc, int n_aux, int64_t n_pairs,
                                                           TB* __restrict__ BcT) {
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
        if (q <= n_pairs) BcT[(blockIdx.y * (n_pairs + 1) + q) * 64 + lane] = (TB)t[lane][4 * r + w];
    }
}

// Writing the results.  The workgroup's 8 waves hold one mu each; every 16 x 16
// result (row r of a lane's element in `rows`, column li) goes through LDS so
// that a row (P, i) of X^T is written 8 mu at a time.
constexpr int WV = 8;                              // waves, and mu, per workgroup
constexpr int XLS = 16 * 17 + 4;                   // one wave's 16 x 16 result in LDS

template <typename T>
struct XStore {
    T* Ls;                                         // [2][WV * XLS]
    T* Xt;
    int mu0, P0, N, n_occ, n_aux, Npad, buf = 0;
    // rows (P, i): i = ib + is * row for row < rows, P = P0 + PT * p + t
    template <int PT>
    __device__ __forceinline__ void get(int rows, int ib, int is, int t) {
        __syncthreads();
        const int tid = threadIdx.x, u = tid & 7, row = (tid >> 3) & 15, p0 = tid >> 7;
        T* out = Xt + ((int64_t)(P0 + t) * n_occ + ib) * Npad + mu0;
        const int i = ib + is * row;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int p = p0 + 4 * k;
            if (row < rows && i < n_occ && P0 + PT * p + t < n_aux && mu0 + u < N)
                out[(int64_t)(PT * p * n_occ + is * row) * Npad + u] = Ls[buf * WV * XLS + u * XLS + row * 17 + p];
        }
        buf ^= 1;                                  // the next result's barrier covers these reads
    }
    __device__ __forceinline__ void put(int wave, int row, int col, T v) {
        Ls[buf * WV * XLS + wave * XLS + row * 17 + col] = v;
    }
};

// Rows (P, i) of X^T for 8 consecutive mu (one per wave) and 16 PT auxiliary
// indices.  Per step of 4 partners a wave issues MF PT 16x16x4 MFMAs and
// TQ PT 4x4x4 ones (the 4-row quads of an occupied count that is not a
// multiple of 16) on operands loaded XD steps ahead straight into registers.
// Lane (li, g) takes partner g of the step; a 16-byte load covers two
// occupied rows (tile pair: rows 32 m + 2 li + h) or two auxiliaries (column
// PT li + t of tile t), so a step costs 3-4 loads of C and PT / 2 of BcT.
// TB: the stored type of BcT, widened exactly.
template <int MF, int TQ, int PT, int XD, typename TB>
__device__ __forceinline__ void xs_body_f64(int mu0, int P0, int i1, const TB* __restrict__ BcT, int64_t n_pairs,
                                            const int2* __restrict__ list, const int* __restrict__ cnt, int lmax,
                                            const double* __restrict__ Cp, int cld, int N, int n_occ, int n_aux,
                                            double* __restrict__ Xt, int Npad) {
    constexpr int NA = MF + (TQ ? 1 : 0);
    static_assert(16 % XD == 0 && PT == 2, "a chunk holds whole rounds; two auxiliaries a load");
    typedef TB tb2_t __attribute__((ext_vector_type(2)));
    __shared__ double Ls[2 * WV * XLS];
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
        const TB* bp = BcT + (int64_t)(P0 >> 6) * (n_pairs + 1) * 64 + (P0 & 63) + PT * li;
        const double* cp = Cp + i1;
        auto load = [&](int nu, int q, double (&a)[NA], double (&b)[PT]) {
            const double* c = cp + (int64_t)(nu & 0x7fffffff) * cld;
            const tb2_t v = *(const tb2_t*)(bp + (int64_t)q * 64);
            b[0] = v[0];
            b[1] = v[1];
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
    XStore<double> x{Ls, Xt, mu0, P0, N, n_occ, n_aux, Npad};
    // element q of lane (li, g) in tile m: row 4 q + g of the tile, column li
#pragma unroll
    for (int m = 0; m < MF; ++m) {
        const bool pair = m < MF / 2 * 2;
        const int ib = i1 + (pair ? 16 * (m & ~1) + (m & 1) : 16 * m);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) x.put(wave, 4 * q + g, li, acc[m][t][q]);
            x.template get<PT>(16, ib, pair ? 2 : 1, t);
        }
    }
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            x.put(wave, g, li, accq[q][t]);
            x.template get<PT>(4, i1 + 16 * MF + 4 * q, 1, t);
        }
}

// FP32 measured: batched SCF of 60 molecules with N = 100-600, X for 49-64
// occupied rows 10.7 -> 4.6 ms a build (6.1 with one workgroup per CU), the whole
// call 620 -> 505 ms; N = 1000 build 10.0 -> 7.1 ms (X 6.5 -> 2.9).
// The same in FP32 arithmetic, bit for bit the dense FP32 kernel's sums: a
// 16x16x4 FP32 MFMA rounds as a chain of fused multiply-adds over its four k in
// order, so leaving out partners whose B is zero changes nothing as long as
// the others keep their order and each block of 64 nu is summed in FP32 from
// zero and then added in FP64.  Loads cover four occupied rows (rows
// 64 m + 4 li + h of four tiles) where there are four tiles.
template <int MF, int PT, int XD>
__device__ __forceinline__ void xs_body_f32(int mu0, int P0, int i1, const float* __restrict__ BcT, int64_t n_pairs,
                                            const int2* __restrict__ list, const int* __restrict__ cnt, int lmax,
                                            const float* __restrict__ Cp, int cld, int N, int n_occ, int n_aux,
                                            float* __restrict__ Xt, int Npad) {
    static_assert(16 % XD == 0 && XD < 16 && PT == 2, "a chunk holds whole rounds; two auxiliaries a load");
    typedef float f2_t __attribute__((ext_vector_type(2)));
    constexpr int M4 = MF / 4 * 4, M2 = MF / 2 * 2;   // tiles loaded by fours, then by twos
    __shared__ float Ls[2 * WV * XLS];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mu = mu0 + wave;
    d4_t sum[MF][PT];
#pragma unroll
    for (int m = 0; m < MF; ++m)
#pragma unroll
        for (int t = 0; t < PT; ++t) sum[m][t] = d4_t{0.0, 0.0, 0.0, 0.0};
    if (mu < N) {
        f4_t acc[MF][PT];
#pragma unroll
        for (int m = 0; m < MF; ++m)
#pragma unroll
            for (int t = 0; t < PT; ++t) acc[m][t] = f4_t{0.f, 0.f, 0.f, 0.f};
        const int2* ent = list + (int64_t)mu * lmax + lane;
        const float* bp = BcT + (int64_t)(P0 >> 6) * (n_pairs + 1) * 64 + (P0 & 63) + PT * li;
        const float* cp = Cp + i1;
        auto load = [&](int nu, int q, float (&a)[MF], float (&b)[PT]) {
            const float* c = cp + (int64_t)(nu & 0x7fffffff) * cld;
            const f2_t v = *(const f2_t*)(bp + (int64_t)q * 64);
            b[0] = v[0];
            b[1] = v[1];
#pragma unroll
            for (int m = 0; m < M4; m += 4) {
                const f4_t w = *(const f4_t*)(c + 16 * m + 4 * li);
#pragma unroll
                for (int h = 0; h < 4; ++h) a[m + h] = w[h];
            }
            if (M2 > M4) {
                const f2_t w = *(const f2_t*)(c + 16 * M4 + 2 * li);
                a[M4 < MF ? M4 : 0] = w[0];
                a[M4 + 1 < MF ? M4 + 1 : 0] = w[1];
            }
            if (MF > M2) a[MF - 1] = c[16 * M2 + li];
        };
        const int nst = (__builtin_amdgcn_readfirstlane(cnt[mu]) + 3) / 4;
        float a[XD][MF], b[XD][PT];
        int2 e = ent[0], en = ent[64];
#pragma unroll
        for (int d = 0; d < XD; ++d) {
            load(__shfl(e.x, 4 * d + g), __shfl(e.y, 4 * d + g), a[d], b[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
        unsigned long long ends = 0;               // bit 4 k: step k of the chunk ends a block of 64 nu
        for (int s = 0; s < nst; s += XD) {
            if ((s & 15) == 0) ends = __ballot(e.x < 0);
            if (((s + XD) & 15) == 0) {
                e = en;
                en = ent[(s + XD) * 4 + 64];
            }
            const int k0 = 4 * ((s + XD) & 15) + g;
#pragma unroll
            for (int d = 0; d < XD; ++d) {
                if (s + d < nst) {
#pragma unroll
                    for (int m = 0; m < MF; ++m)
#pragma unroll
                        for (int t = 0; t < PT; ++t)
                            acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][m], b[d][t], acc[m][t], 0, 0, 0);
                    if ((ends >> (4 * ((s & 15) + d))) & 1) {
#pragma unroll
                        for (int m = 0; m < MF; ++m)
#pragma unroll
                            for (int t = 0; t < PT; ++t)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    sum[m][t][r] += (double)acc[m][t][r];
                                    acc[m][t][r] = 0.0f;
                                }
                    }
                }
                load(__shfl(e.x, k0 + 4 * d), __shfl(e.y, k0 + 4 * d), a[d], b[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    XStore<float> x{Ls, Xt, mu0, P0, N, n_occ, n_aux, Npad};
    // element r of lane (li, g) in tile m: row 4 g + r of the tile, column li
#pragma unroll
    for (int m = 0; m < MF; ++m) {
        const int is = m < M4 ? 4 : m < M2 ? 2 : 1;
        const int ib = i1 + (m < M4 ? 16 * (m & ~3) + (m & 3) : m < M2 ? 16 * M4 + (m & 1) : 16 * m);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
#pragma unroll
            for (int r = 0; r < 4; ++r) x.put(wave, 4 * g + r, li, (float)sum[m][t][r]);
            x.template get<PT>(16, ib, is, t);
        }
    }
}

constexpr int XPT = 2;                             // 16-wide auxiliary tiles per workgroup
constexpr int xs_depth(int mf) { return mf <= 2 ? 4 : 2; }
// FP32: 4 tiles at depth 2 stay within the 128 registers that let two workgroups share a CU
constexpr int xs_depth32(int mf) { return mf == 4 ? 2 : 4; }
constexpr int xs_waves(int mf) { return mf <= 4 ? 4 : 2; }   // resident waves per SIMD asked for

template <int MF, int TQ, typename TB>
__global__ __launch_bounds__(64 * WV, 2) void xs_kernel(const TB* __restrict__ BcT, int64_t n_pairs,
                                                        const int2* __restrict__ list, const int* __restrict__ cnt,
                                                        int lmax, const double* __restrict__ Cp, int cld, int N,
                                                        int n_occ, int n_aux, int i0, double* __restrict__ Xt,
                                                        int Npad) {
    const int no = (N + WV - 1) / WV, L = xcd_remap(blockIdx.x, gridDim.x);
    xs_body_f64<MF, TQ, XPT, xs_depth(MF), TB>(WV * (L % no), 16 * XPT * (L / no), i0 + 128 * blockIdx.y, BcT, n_pairs,
                                               list, cnt, lmax, Cp, cld, N, n_occ, n_aux, Xt, Npad);
}

template <int MF>
__global__ __launch_bounds__(64 * WV, xs_waves(MF)) void xs32_kernel(const float* __restrict__ BcT, int64_t n_pairs,
                                                          const int2* __restrict__ list, const int* __restrict__ cnt,
                                                          int lmax, const float* __restrict__ Cp, int cld, int N,
                                                          int n_occ, int n_aux, int i0, float* __restrict__ Xt,
                                                          int Npad) {
    const int no = (N + WV - 1) / WV, L = xcd_remap(blockIdx.x, gridDim.x);
    xs_body_f32<MF, XPT, xs_depth32(MF)>(WV * (L % no), 16 * XPT * (L / no), i0 + 128 * blockIdx.y, BcT, n_pairs, list,
                                       cnt, lmax, Cp, cld, N, n_occ, n_aux, Xt, Npad);
}

dim3 xs_grid(int N, int n_aux, int chunks) {
    return dim3((unsigned)((N + WV - 1) / WV) * (unsigned)((n_aux + 16 * XPT - 1) / (16 * XPT)), (unsigned)chunks);
}

template <int MF, int TQ>
hipError_t xs_launch(const ri::XSparse& w, int chunks, const double* Cp, int cld, int N, int n_occ, int n_aux, int i0,
                     double* Xt, int Npad, hipStream_t st) {
    const dim3 grid = xs_grid(N, n_aux, chunks);
    if (w.BcT32)
        xs_kernel<MF, TQ, float><<<grid, 64 * WV, 0, st>>>(w.BcT32, w.n_pairs, w.list, w.cnt, w.lmax, Cp, cld, N, n_occ,
                                                           n_aux, i0, Xt, Npad);
    else
        xs_kernel<MF, TQ, double><<<grid, 64 * WV, 0, st>>>(w.BcT, w.n_pairs, w.list, w.cnt, w.lmax, Cp, cld, N, n_occ,
                                                            n_aux, i0, Xt, Npad);
    return hipGetLastError();
}

// The batched form: work items (8 mu, 32 auxiliaries) of the molecules whose
// shape is 4 MF + TQ (FP32: 4 MF); see x_transform_b.
template <int MF, int TQ, int PREC>
__global__ __launch_bounds__(64 * WV, 4) void xs_b_kernel(const ri::MolDesc* d, const int* prefix, int n_mol) {
    int mol, loc;
    ri::decode_item(prefix, n_mol, blockIdx.x, mol, loc);
    const ri::MolDesc& m = d[mol];
    if (!m.state[0] || m.xs != 4 * MF + TQ) return;
    const int no = (m.N + WV - 1) / WV, mu0 = WV * (loc % no), P0 = 16 * XPT * (loc / no);
    if constexpr (PREC == RI_FP64)
        xs_body_f64<MF, TQ, XPT, xs_depth(MF), double>(mu0, P0, 0, (const double*)m.BcT, m.n_pairs, m.plist, m.pcnt,
                                                       m.lmax, m.Cq, 64, m.N, m.n_occ, m.n_aux, (double*)m.Xt, m.npad);
    else if constexpr (PREC == ri::X_F64_B32)
        xs_body_f64<MF, TQ, XPT, xs_depth(MF), float>(mu0, P0, 0, (const float*)m.BcT, m.n_pairs, m.plist, m.pcnt,
                                                      m.lmax, m.Cq, 64, m.N, m.n_occ, m.n_aux, (double*)m.Xt, m.npad);
    else
        xs_body_f32<MF, XPT, xs_depth32(MF)>(mu0, P0, 0, (const float*)m.BcT, m.n_pairs, m.plist, m.pcnt, m.lmax,
                                           (const float*)m.Cq, 64, m.N, m.n_occ, m.n_aux, (float*)m.Xt, m.npad);
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

bool xs_sparse(int N, int n_aux, int64_t n_pairs) {
    return n_pairs > 0 && (n_pairs + 1) * xs_ldp(n_aux) <= ((int64_t)1 << 33) &&
           (double)(2 * n_pairs - N) <= 0.6 * (double)N * N;
}

bool xs_wanted(int N, int n_aux, int n_occ, int64_t n_pairs, int prec, bool once) {
    if ((prec != RI_FP64 && prec != RI_FP32) || !xs_sparse(N, n_aux, n_pairs)) return false;
    const int64_t xt = xt_rows(n_aux, n_occ) * xt_ld(N) * (prec == RI_FP64 ? 8 : 4);
    const double most = prec == RI_FP64 ? 0.42 : 0.34;
    return xt > (int64_t)RI_NOALLOC_SCRATCH_BYTES &&
           (!once || xt > ((int64_t)512 << 20) || (double)(2 * n_pairs - N) <= most * (double)N * N);
}

int64_t xs_most_pairs(int N, int n_aux) {
    int64_t n = std::min<int64_t>((int64_t)((0.6 * N * N + N) / 2), ((int64_t)1 << 33) / xs_ldp(n_aux) - 1) + 1;
    while (n > 0 && !xs_sparse(N, n_aux, n)) --n;
    return n;
}

int xs_ldp(int n_aux) { return (n_aux + 63) / 64 * 64; }
int xs_lmax(int N) { return (N + 63) / 64 * 64 + 128; }

hipError_t xs_lists(const XSparse& w, const int32_t* pairs, int64_t n_pairs, int N, hipStream_t st) {
    RI_TRY(fill_i32(w.map, -1, (int64_t)N * N, st));
    pair_map_sym_kernel<<<(unsigned)((n_pairs + 255) / 256), 256, 0, st>>>(pairs, n_pairs, N, w.map);
    RI_TRY(hipGetLastError());
    if (w.BcT32) row_list_kernel<true><<<(N + 3) / 4, 256, 0, st>>>(w.map, N, (int)n_pairs, w.lmax, w.list, w.cnt);
    else row_list_kernel<false><<<(N + 3) / 4, 256, 0, st>>>(w.map, N, (int)n_pairs, w.lmax, w.list, w.cnt);
    return hipGetLastError();
}

hipError_t xs_rows(const XSparse& w, const double* Bc, int64_t n_pairs, int np, hipStream_t st) {
    const dim3 grid((unsigned)(n_pairs / 64 + 1), xs_ldp(np) / 64);
    if (w.BcT32) bc_transpose_kernel<<<grid, 256, 0, st>>>(Bc, np, n_pairs, w.BcT32);
    else bc_transpose_kernel<<<grid, 256, 0, st>>>(Bc, np, n_pairs, w.BcT);
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
    if (full > 0) RI_TRY((xs_launch<8, 0>(w, full, Cp, cld, N, n_occ, n_aux, 0, Xt, Npad, st)));
    if (left == 0) return hipSuccess;
    const int mt = (left + 15) / 16, rem = left - 16 * (mt - 1);
    const int mf = rem <= 12 ? mt - 1 : mt, tq = rem <= 12 ? (rem + 3) / 4 : 0;
    switch (4 * mf + tq) {
#define XS(f, q) case 4 * f + q: return xs_launch<f, q>(w, 1, Cp, cld, N, n_occ, n_aux, 128 * full, Xt, Npad, st);
#define XSROW(f) XS(f, 1) XS(f, 2) XS(f, 3)
        XSROW(0) XSROW(1) XSROW(2) XSROW(3) XSROW(4) XSROW(5) XSROW(6) XSROW(7)
        XS(1, 0) XS(2, 0) XS(3, 0) XS(4, 0) XS(5, 0) XS(6, 0) XS(7, 0) XS(8, 0)
#undef XSROW
#undef XS
        default: return hipErrorInvalidValue;
    }
}

hipError_t xs_transform32(const XSparse& w, int N, int n_aux, int n_occ, const double* C, float* Cf, float* Xt,
                          hipStream_t st) {
    const int cld = cpad_ld(n_occ), Npad = xt_ld(N);
    RI_TRY(cpad_f32(C, N, n_occ, Cf, st));
    const int full = n_occ / 128, mt = (n_occ % 128 + 15) / 16;
#define XS32(f, ch, i0) xs32_kernel<f><<<xs_grid(N, n_aux, ch), 64 * WV, 0, st>>>(w.BcT32, w.n_pairs, w.list, w.cnt, \
                                                                w.lmax, Cf, cld, N, n_occ, n_aux, i0, Xt, Npad)
    if (full > 0) XS32(8, full, 0);
    RI_TRY(hipGetLastError());
    switch (mt) {
        case 0: return hipSuccess;
        case 1: XS32(1, 1, 128 * full); break;
        case 2: XS32(2, 1, 128 * full); break;
        case 3: XS32(3, 1, 128 * full); break;
        case 4: XS32(4, 1, 128 * full); break;
        case 5: XS32(5, 1, 128 * full); break;
        case 6: XS32(6, 1, 128 * full); break;
        case 7: XS32(7, 1, 128 * full); break;
        default: XS32(8, 1, 128 * full); break;
    }
#undef XS32
    return hipGetLastError();
}

int xs_items(int N, int n_aux) { return (int)xs_grid(N, n_aux, 1).x; }

hipError_t xs_transform_b(const MolDesc* d, const int* prefix, int n_mol, int total, int xs, int prec, hipStream_t st) {
    if (total <= 0) return hipSuccess;
    switch (prec == RI_FP32 ? 64 + xs : xs) {
#define XB(f, q)                                                                                              \
    case 4 * f + q:                                                                                           \
        if (prec == RI_FP64) xs_b_kernel<f, q, RI_FP64><<<total, 64 * WV, 0, st>>>(d, prefix, n_mol);         \
        else xs_b_kernel<f, q, X_F64_B32><<<total, 64 * WV, 0, st>>>(d, prefix, n_mol);                       \
        break;
        XB(0, 1) XB(0, 2) XB(0, 3) XB(1, 0) XB(1, 1) XB(1, 2) XB(1, 3) XB(2, 0)
        XB(2, 1) XB(2, 2) XB(2, 3) XB(3, 0) XB(3, 1) XB(3, 2) XB(3, 3) XB(4, 0)
#undef XB
#define XB(f) case 64 + 4 * f: xs_b_kernel<f, 0, RI_FP32><<<total, 64 * WV, 0, st>>>(d, prefix, n_mol); break;
        XB(1) XB(2) XB(3) XB(4)
#undef XB
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ri
