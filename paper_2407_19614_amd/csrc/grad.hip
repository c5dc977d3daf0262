// RI-HF analytic gradient contractions: one-electron (D h' - W S'),
// two-centre metric (-1/2 Z (P|Q)'), three-centre (Y (mu nu|P)') and the
// nuclear repulsion derivative.  Derivative integrals are evaluated on the
// fly and accumulated per atom: per-block LDS sums, one partial row per
// block, then a deterministic row reduction.
#include "kernels.h"

#include <algorithm>
#include <climits>

namespace {

constexpr double TWO_PI_52 = 34.98683665524972;   // 2 pi^{5/2}
constexpr int MAXC = 2048;                          // centres held in LDS

__device__ __forceinline__ void lds_add3(double* g, int atom, double x, double y, double z) {
    atomicAdd(&g[3 * atom + 0], x);
    atomicAdd(&g[3 * atom + 1], y);
    atomicAdd(&g[3 * atom + 2], z);
}

__device__ void flush(double* g, int nc3, double* part) {
    __syncthreads();
    double* row = part + (int64_t)blockIdx.x * nc3;
    for (int i = threadIdx.x; i < nc3; i += blockDim.x) row[i] = g[i];
}

// as flush, adding to the block's row (launches over several slabs)
__device__ void flush_add(double* g, int nc3, double* part) {
    __syncthreads();
    double* row = part + (int64_t)blockIdx.x * nc3;
    for (int i = threadIdx.x; i < nc3; i += blockDim.x) row[i] += g[i];
}

// F0(t) and F1(t) together.  Below t = 1, F1 from its Taylor series
// F1(t) = sum_k (-t)^k / (k! (2k + 3)), 19 terms (the first omitted term is
// below 3e-18), and F0 = 2t F1 + exp(-t) (the downward relation, all terms
// positive); above, F0 = (sqrt(pi)/2) erf(sqrt t) / sqrt t and
// F1 = (F0 - exp(-t)) / (2t).  From t = 40 on, erfc(sqrt t) < 1e-18 and
// exp(-t) < 5e-18 relative to F0, so both drop out: F0 = (sqrt(pi)/2) / sqrt t
// and F1 = F0 / (2t).
struct BoysTaylor {
    double c[19];
    constexpr BoysTaylor() : c() {
        double f = 1.0;   // (-1)^k / k!
        for (int k = 0; k < 19; ++k) {
            c[k] = f / (2 * k + 3);
            f = -f / (k + 1);
        }
    }
};
__device__ __forceinline__ void boys_f01(double t, double& f0, double& f1) {
    if (t < 1.0) {
        constexpr BoysTaylor B{};
        double s = B.c[18];
#pragma unroll
        for (int k = 17; k >= 0; --k) s = fma(s, t, B.c[k]);
        f1 = s;
        f0 = fma(2.0 * t, s, exp(-t));
    } else if (t < 40.0) {
        const double r = sqrt(t);
        f0 = 0.88622692545275801365 * erf(r) / r;
        f1 = (f0 - exp(-t)) / (2.0 * t);
    } else {
        f0 = 0.88622692545275801365 / sqrt(t);
        f1 = f0 / (2.0 * t);
    }
}

// F0(t) and F1(t) together, from a table of F_0 .. F_9 at multiples of 1/8 below
// t = 40: the Taylor expansions F_m(t) = sum_k F_{m+k}(t_j) (t_j - t)^k / k! to k = 8
// about the nearest point (|t_j - t| <= 1/16: the first omitted term is below
// 6e-18 of F_m); t >= 40 as above.  With the table rounded from double-double, F0
// is off by at most 2.0e-16 (rms 6e-17) and F1 by 2.1e-16 (7e-17), where the
// direct forms are off by 2.9e-16 (8e-17) and 4.9e-16 (1.1e-16).  The direct
// forms took most of the three-centre kernel's time (N = 1000: 3.5 -> 1.75 ms);
// the one-electron kernel keeps them: its blocks' copies of the table cost what
// they give (0.68 against 0.89 ms at N = 1000).
constexpr int BT_N = 322, BT_M = 11;               // points 0 .. 321; ten values in an odd row length

struct dd {
    double h, l;
};
__device__ __forceinline__ dd dd_fast(double h, double l) {
#pragma clang fp contract(off)
    const double s = h + l;
    return {s, l - (s - h)};
}
__device__ __forceinline__ dd dd_add(dd a, dd b) {
    const double s = a.h + b.h, v = s - a.h;
    return dd_fast(s, (a.h - (s - v)) + (b.h - v) + (a.l + b.l));
}
__device__ __forceinline__ dd dd_mul(dd a, dd b) {
#pragma clang fp contract(off)
    const double p = a.h * b.h;
    return dd_fast(p, fma(a.h, b.h, -p) + (a.h * b.l + a.l * b.h));
}
__device__ __forceinline__ dd dd_div(dd a, double c) {
#pragma clang fp contract(off)
    const double rc = 1.0 / c, q = a.h * rc;
    return dd_fast(q, (fma(-q, c, a.h) + a.l) * rc);
}

// Row j of the table, t = j / 8: F_9 from its series exp(-t) sum_k (2t)^k / (19 *
// 21 ... (2k + 19)), all terms positive, then the downward relation F_{m-1} =
// (2t F_m + exp(-t)) / (2m - 1), in double-double.
__device__ void boys_row(int j, double* T) {
    const dd x = {0.25 * j, 0.0};
    dd term = {1.0, 0.0}, sum, e = {1.0, 0.0}, b = {0x1.c3d6a24ed8222p-1, -0x1.e1e0a76cb0685p-55};   // b = exp(-1/8)
    for (int k = j; k > 0; k >>= 1) {
        if (k & 1) e = dd_mul(e, b);
        b = dd_mul(b, b);
    }
    term = dd_div(term, 19.0);
    sum = term;
    for (int k = 1; k < 200; ++k) {
        term = dd_div(dd_mul(term, x), 2.0 * k + 19.0);
        sum = dd_add(sum, term);
        if (term.h < 1e-22 * sum.h) break;
    }
    dd f = dd_mul(e, sum);
    T[9] = f.h;
    for (int m = 9; m > 0; --m) {
        f = dd_div(dd_add(dd_mul(x, f), e), 2.0 * m - 1.0);
        T[m - 1] = f.h;
    }
    T[10] = 0.0;
}

__device__ __forceinline__ void boys_f01(const double* T, double t, double& f0, double& f1) {
    const int j = (int)fma(fmin(t, 40.0), 8.0, 0.5);
    const double* f = T + j * BT_M;
    const double d = fma((double)j, 0.125, -t);
    double a = f[8], b = f[9];
#pragma unroll
    for (int k = 8; k > 0; --k) {
        const double x = d * (1.0 / k);
        a = fma(x, a, f[k - 1]);
        b = fma(x, b, f[k]);
    }
    f0 = a;
    f1 = b;
    if (t >= 40.0) {
        f0 = 0.88622692545275801365 / sqrt(t);
        f1 = f0 / (2.0 * t);
    }
}

// r = 1 / sqrt(x) and i = 1 / x to rounding: the hardware estimate, a Newton step,
// and one more on the exact residual 1 - x r^2
__device__ __forceinline__ void rsqrt_rcp(double x, double& r, double& i) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    const double h = x * y, l = fma(x, y, -h);
    r = fma(0.5 * y, fma(-l, y, fma(-h, y, 1.0)), y);
    const double z = r * r;
    i = fma(z, fma(-x, z, 1.0), z);
}

// Sum over the wave; every lane receives the total.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// sum over all (mu, nu) of D h'_mu_nu - W S'_mu_nu, taken over mu >= nu with
// weight 2 off the diagonal (h, S, D and W are symmetric).  One lower pair
// per thread; the nuclear-attraction loop over centres is uniform across the
// wave, so each centre's share is summed over the wave before one LDS add.
// g holds 3 * nc doubles of dynamic LDS.
__global__ __launch_bounds__(256) void g1e_kernel(const double* xyz, const double* Z, int nc, const int32_t* fc,
                                                  const double* fe, int N, const double* D, const double* W,
                                                  double* part) {
    extern __shared__ double g[];
    for (int i = threadIdx.x; i < 3 * nc; i += 256) g[i] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t total = (int64_t)N * (N + 1) / 2;
    const int64_t span = (int64_t)gridDim.x * 256;
    const int64_t rounds = (total + span - 1) / span;   // every wave runs the same count: shuffles stay uniform
    for (int64_t r = 0; r < rounds; ++r) {
        const int64_t e = r * span + blockIdx.x * 256ll + threadIdx.x;
        const bool in = e < total;
        int mu = 0, nu = 0;
        if (in) {
            mu = (int)((sqrt(8.0 * (double)e + 1.0) - 1.0) * 0.5);
            while ((int64_t)(mu + 1) * (mu + 2) / 2 <= e) ++mu;
            while ((int64_t)mu * (mu + 1) / 2 > e) --mu;
            nu = (int)(e - (int64_t)mu * (mu + 1) / 2);
        }
        const double wq = in ? (mu == nu ? 1.0 : 2.0) : 0.0;
        const double d = wq * D[(int64_t)mu * N + nu], w = wq * W[(int64_t)mu * N + nu];
        const double a = fe[mu], b = fe[nu];
        const int ca = fc[mu], cb = fc[nu];
        const double* A = xyz + 3 * ca;
        const double* B = xyz + 3 * cb;
        const double p = a + b, ip = 1.0 / p, m = a * b * ip;
        const double dx = A[0] - B[0], dy = A[1] - B[1], dz = A[2] - B[2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        const double kn = norm_s(a) * norm_s(b) * exp(-m * r2);
        // every term of this pair carries kn times D or W: below 1e-24 the pair
        // changes no gradient component by more than ~1e-20 (1e-14 over 1e6 pairs)
        const bool live = in && !(kn * (fabs(d) + fabs(w)) < 1e-24 * wq);
        if (__ballot(live) == 0) continue;
        const double s = kn * pow(RI_PI * ip, 1.5);
        const double t = m * (3.0 - 2.0 * m * r2) * s;
        // dS/dA = -2 m (A-B) S ; dT/dA = -2 m (A-B) (2 m S + T)
        const double fS = -2.0 * m * s, fT = -2.0 * m * (2.0 * m * s + t);
        const double coef = live ? d * fT - w * fS : 0.0;
        const double gx = coef * dx, gy = coef * dy, gz = coef * dz;   // to atom of mu; minus to atom of nu
        const double Px = (a * A[0] + b * B[0]) * ip, Py = (a * A[1] + b * B[1]) * ip, Pz = (a * A[2] + b * B[2]) * ip;
        const double dl = live ? d : 0.0;
        double ax = 0, ay = 0, az = 0, bx = 0, by = 0, bz = 0;
        const double pre0 = 2.0 * RI_PI * ip * kn;
        for (int c = 0; c < nc; ++c) {
            const double zc = Z[c];
            if (zc == 0.0) continue;
            const double* Cc = xyz + 3 * c;
            const double ex = Px - Cc[0], ey = Py - Cc[1], ez = Pz - Cc[2];
            const double x = p * (ex * ex + ey * ey + ez * ez);
            const double pre = zc * pre0;
            double F0, F1;
            boys_f01(x, F0, F1);
            const double V = -pre * F0;
            const double f1 = pre * F1;
            // dV/dA = V (-2 m (A-B)) + f1 2a (P-C);  dV/dB = V (2 m (A-B)) + f1 2b (P-C);  dV/dC = -f1 2p (P-C)
            const double va = -2.0 * m * V;
            ax += dl * (va * dx + f1 * 2.0 * a * ex);
            ay += dl * (va * dy + f1 * 2.0 * a * ey);
            az += dl * (va * dz + f1 * 2.0 * a * ez);
            bx += dl * (-va * dx + f1 * 2.0 * b * ex);
            by += dl * (-va * dy + f1 * 2.0 * b * ey);
            bz += dl * (-va * dz + f1 * 2.0 * b * ez);
            const double cc = -dl * f1 * 2.0 * p;
            const double sx = wave_sum(cc * ex), sy = wave_sum(cc * ey), sz = wave_sum(cc * ez);
            if (lane == 0) lds_add3(g, c, sx, sy, sz);
        }
        if (live) {
            lds_add3(g, ca, gx + ax, gy + ay, gz + az);
            lds_add3(g, cb, -gx + bx, -gy + by, -gz + bz);
        }
    }
    flush(g, 3 * nc, part);
}

// -1/2 sum_PQ Z_PQ (P|Q)' over the lower triangle (P > Q, weight 2);
// Z_PQ = c_P c_Q + Zx_PQ where Zx (lower) holds -2 sum_ij Xi Xi.
__global__ __launch_bounds__(256) void g2c_kernel(const double* xyz, const int32_t* ac, const double* ae, int na,
                                                  int nc, const double* Zx, const double* cv, double* part) {
    __shared__ double g[3 * MAXC];
    for (int i = threadIdx.x; i < 3 * nc; i += 256) g[i] = 0.0;
    __syncthreads();
    const int64_t total = (int64_t)na * na;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        int P = e / na, Q = e % na;
        if (Q >= P) continue;
        int cp = ac[P], cq = ac[Q];
        if (cp == cq) continue;
        double z = Zx[e] + cv[P] * cv[Q];
        double a = ae[P], b = ae[Q], s = a + b, w = a * b / s;
        const double* R = xyz + 3 * cp;
        const double* S = xyz + 3 * cq;
        double dx = R[0] - S[0], dy = R[1] - S[1], dz = R[2] - S[2];
        double c0 = norm_s(a) * norm_s(b) * TWO_PI_52 / (a * b * sqrt(s));
        double f = -c0 * boys_f1(w * (dx * dx + dy * dy + dz * dz)) * 2.0 * w;   // d(P|Q)/dR_P / (R_P - R_Q)
        double k = -z * f;   // -1/2 * 2 * Z * f
        lds_add3(g, cp, k * dx, k * dy, k * dz);
        lds_add3(g, cq, -k * dx, -k * dy, -k * dz);
    }
    flush(g, 3 * nc, part);
}

// Constants of pair q for the derivative integrals, as PC_N arrays over the pairs,
// and its two centres.
constexpr int PC_P = 0, PC_K = 1, PC_X = 2, PC_M = 5, PC_A = 6, PC_B = 7, PC_D = 8, PC_W = 11, PC_N = 12;

__device__ __forceinline__ void pair_consts(int64_t q, int mu, int nu, const double* __restrict__ xyz,
                                            const int32_t* __restrict__ fc, const double* __restrict__ fe,
                                            int64_t n_pairs, const double* __restrict__ D, int N,
                                            double* __restrict__ pc, int2* __restrict__ ctr) {
    const int ca = fc[mu], cb = fc[nu];
    const double a = fe[mu], b = fe[nu], p = a + b, ip = 1.0 / p, m = a * b * ip;
    const double* A = xyz + 3 * ca;
    const double* B = xyz + 3 * cb;
    const double dx = A[0] - B[0], dy = A[1] - B[1], dz = A[2] - B[2];
    auto put = [&](int k, double v) { pc[k * n_pairs + q] = v; };
    put(PC_P, p);
    put(PC_K, norm_s(a) * norm_s(b) * exp(-m * (dx * dx + dy * dy + dz * dz)) * TWO_PI_52 * ip);
    put(PC_X, (a * A[0] + b * B[0]) * ip);
    put(PC_X + 1, (a * A[1] + b * B[1]) * ip);
    put(PC_X + 2, (a * A[2] + b * B[2]) * ip);
    put(PC_M, m);
    put(PC_A, a * ip);
    put(PC_B, b * ip);
    put(PC_D, dx);
    put(PC_D + 1, dy);
    put(PC_D + 2, dz);
    put(PC_W, (mu == nu ? 1.0 : 2.0) * D[(int64_t)mu * N + nu]);
    ctr[q] = make_int2(mu == nu ? ~ca : ca, cb);   // the diagonal's weight is 1, the others' 2
}

// The first two blocks make the table T, the others a pair per thread.
__global__ __launch_bounds__(256) void pair_consts_kernel(const double* __restrict__ xyz,
                                                          const int32_t* __restrict__ fc,
                                                          const double* __restrict__ fe,
                                                          const int32_t* __restrict__ pairs, int64_t n_pairs,
                                                          const double* __restrict__ D, int N,
                                                          double* __restrict__ pc, int2* __restrict__ ctr,
                                                          double* __restrict__ T) {
    const int64_t q = (blockIdx.x - 2ll) * 256 + threadIdx.x;
    if (q < 0 && q + 512 < BT_N) boys_row((int)(q + 512), T + (q + 512) * BT_M);
    if (q < 0 || q >= n_pairs) return;
    pair_consts(q, pairs[2 * q], pairs[2 * q + 1], xyz, fc, fe, n_pairs, D, N, pc, ctr);
}

// sum_P sum_pairs w Y^P_mu_nu (mu nu|P)',  Y = c_P D_mu_nu - 2 (U^P C^T)_mu_nu, for
// auxiliary indices P0 .. P0 + np - 1 (WY[P - P0][q] = (U^P C^T)_mu_nu of pair q),
// into the block's partial row, or (P0 > 0) added to it.  Work items are (bpi blocks of 256 pairs,
// chunk of G3_PC auxiliaries), a pair per thread, the chunk's auxiliaries in
// turn (their constants staged in LDS).  With e = P - R_aux and g = 2 w c0 F1, an
// entry adds I y to s and g y e to G: the pair's centres take -2 m s (A - B) -
// (a/p) G and +2 m s (A - B) - (b/p) G at the end of the chunk, and the
// auxiliary's centre +G, kept in registers over the item's pairs and summed over
// the wave once (a wave sum per entry cost 36 lane exchanges of the some 100
// instructions that an entry takes).  Bound by FP64 throughput and the table's
// LDS reads; an entry at a time keeps to the registers (all eight
// unrolled together: 91 spilled, 3.05 ms; 1.75 ms so, and 220 -> 153 us at N = 300).  g holds 3 * nc
// doubles of dynamic LDS.
constexpr int G3_PC = 8;

__global__ __launch_bounds__(256, 2) void g3c_kernel(const double* __restrict__ xyz, const int32_t* __restrict__ ac,
                                                     const double* __restrict__ ae, int P0, int np, int nc,
                                                     int64_t n_pairs, int bpi, const double* __restrict__ pc,
                                                     const int2* __restrict__ ctr, const double* __restrict__ WY,
                                                     const double* __restrict__ cv, const double* __restrict__ bt, double* __restrict__ part) {
    extern __shared__ double g[];
    __shared__ double T[BT_N * BT_M];
    __shared__ double sp[G3_PC][6];   // alpha, norm(alpha) / alpha, centre (3), c_P
    __shared__ int sc[G3_PC];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < 3 * nc; i += 256) g[i] = 0.0;
    for (int i = tid; i < BT_N * BT_M; i += 256) T[i] = bt[i];
    const int64_t pb = (n_pairs + 256ll * bpi - 1) / (256ll * bpi);
    const int64_t items = pb * ((np + G3_PC - 1) / G3_PC);
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int pc0 = (int)(it / pb) * G3_PC, pcn = min(G3_PC, np - pc0);
        __syncthreads();   // the previous item's reads of sp are done (g and T ready before the first)
        if (tid < G3_PC) {
            // past the last auxiliary: its own values again, with zero weight
            const int P = P0 + min(pc0 + tid, np - 1), c = ac[P];
            const double al = ae[P];
            sp[tid][0] = al;
            sp[tid][1] = tid < pcn ? norm_s(al) / al : 0.0;
            sp[tid][2] = xyz[3 * c];
            sp[tid][3] = xyz[3 * c + 1];
            sp[tid][4] = xyz[3 * c + 2];
            sp[tid][5] = cv[P];
            sc[tid] = c;
        }
        __syncthreads();
        double ga[G3_PC][3];
#pragma unroll
        for (int k = 0; k < G3_PC; ++k) ga[k][0] = ga[k][1] = ga[k][2] = 0.0;
        for (int blk = 0; blk < bpi; ++blk) {
            const int64_t qq = ((it % pb) * bpi + blk) * 256 + tid;
            if (((it % pb) * bpi + blk) * 256 >= n_pairs) break;
            const bool live = qq < n_pairs;
            const int64_t q = live ? qq : n_pairs - 1;
            auto con = [&](int k) { return pc[k * n_pairs + q]; };
            const int2 cc = ctr[q];
            const double p = con(PC_P), kp = live ? con(PC_K) : 0.0;   // lanes past the pairs add zeros
            const double Px = con(PC_X), Py = con(PC_X + 1), Pz = con(PC_X + 2), dw = con(PC_W);
            const double w2 = cc.x < 0 ? 2.0 : 4.0;
            const double* wy = WY + (int64_t)pc0 * n_pairs + q;
            double s = 0.0, gx = 0.0, gy = 0.0, gz = 0.0, yc[G3_PC];
#pragma unroll
            for (int k = 0; k < G3_PC; ++k) yc[k] = wy[(int64_t)min(k, pcn - 1) * n_pairs];
#pragma unroll
            for (int k = 0; k < G3_PC; ++k) {
                __builtin_amdgcn_sched_barrier(0);   // an entry at a time, to stay in registers
                const double al = sp[k][0];
                const double y = fma(sp[k][5], dw, -w2 * yc[k]);
                double r, isa;
                rsqrt_rcp(p + al, r, isa);
                const double w = p * al * isa;
                const double ex = Px - sp[k][2], ey = Py - sp[k][3], ez = Pz - sp[k][4];
                double F0, F1;
                boys_f01(T, w * (ex * ex + ey * ey + ez * ez), F0, F1);
                const double c0 = kp * sp[k][1] * r * y;
                s = fma(c0, F0, s);
                const double gg = 2.0 * w * c0 * F1;
                const double vx = gg * ex, vy = gg * ey, vz = gg * ez;
                gx += vx; gy += vy; gz += vz;
                ga[k][0] += vx; ga[k][1] += vy; ga[k][2] += vz;
            }
            if (live) {
                const double f = 2.0 * con(PC_M) * s, ap = con(PC_A), bp = con(PC_B);
                const double fx = f * con(PC_D), fy = f * con(PC_D + 1), fz = f * con(PC_D + 2);
                lds_add3(g, cc.x < 0 ? ~cc.x : cc.x, -fx - ap * gx, -fy - ap * gy, -fz - ap * gz);
                lds_add3(g, cc.y, fx - bp * gx, fy - bp * gy, fz - bp * gz);
            }
        }
#pragma unroll
        for (int k = 0; k < G3_PC; ++k) {
            const double sx = wave_sum(ga[k][0]), sy = wave_sum(ga[k][1]), sz = wave_sum(ga[k][2]);
            if (lane == 0) lds_add3(g, sc[k], sx, sy, sz);
        }
    }
    if (P0 == 0) flush(g, 3 * nc, part);
    else flush_add(g, 3 * nc, part);
}

// The pairs by rows: sp, a copy of the pairs, and rows, the first of each mu in it
// (rows[N] = n_pairs).  Pairs that are not sorted by mu set rows[N + 1], which is 0
// before, and are sorted by pair_sort_kernel.
struct Pair {   // aligned as the caller's ints
    int32_t x, y;
};

__global__ __launch_bounds__(256) void pair_rows_kernel(const Pair* __restrict__ pairs, int64_t n_pairs, int N,
                                                        int32_t* __restrict__ rows, Pair* __restrict__ sp) {
    const int64_t t = blockIdx.x * 256ll + threadIdx.x;
    if (t < n_pairs) {
        sp[t] = pairs[t];
        if (t + 1 < n_pairs && pairs[t].x > pairs[t + 1].x) rows[N + 1] = 1;
    }
    if (t > N) return;
    int64_t lo = 0, hi = n_pairs;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (pairs[mid].x < t) lo = mid + 1;
        else hi = mid;
    }
    rows[t] = (int32_t)lo;
}

// Row mu of the pairs in any order, by one workgroup: counts the pairs of the rows
// before it (rows[mu]) and its own, a quarter of the list per wave, then places its
// own in the order that they have.  Returns their first place and count.
__device__ __forceinline__ int2 sort_row(const Pair* __restrict__ pairs, int64_t n_pairs, int mu, int32_t* rows,
                                         Pair* __restrict__ sp) {
    constexpr int D = 8;                           // steps of 64 pairs in flight
    __shared__ int32_t before[4], own[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t per = (n_pairs + 255) / 256 * 64, a = wave * per, z = min(n_pairs, a + per);
    int32_t less = 0, mine = 0, at = 0, first = 0, all = 0;
    for (int pass = 0; pass < 2; ++pass) {         // count, then place
        for (int64_t q0 = a; q0 < z; q0 += 64 * D) {
            Pair v[D];
#pragma unroll
            for (int d = 0; d < D; ++d) v[d] = pairs[min(q0 + 64 * d + lane, n_pairs - 1)];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const bool in = q0 + 64 * d + lane < z;
                const unsigned long long m = __ballot(in && v[d].x == mu);
                if (pass == 0) {
                    less += __popcll(__ballot(in && v[d].x < mu));
                    mine += __popcll(m);
                } else if (m) {
                    if ((m >> lane) & 1) sp[at + __popcll(m & ((1ull << lane) - 1))] = v[d];
                    at += __popcll(m);
                }
            }
        }
        if (pass == 0) {
            if (lane == 0) {
                before[wave] = less;
                own[wave] = mine;
            }
            __syncthreads();
            first = before[0] + before[1] + before[2] + before[3];
            all = own[0] + own[1] + own[2] + own[3];
            if (threadIdx.x == 0) rows[mu] = first;
            at = first;
            for (int w = 0; w < wave; ++w) at += own[w];
        }
    }
    return make_int2(first, all);
}

// Pairs that pair_rows_kernel found in another order, a workgroup per row (the last:
// the end).  Bound by the reads of the list through L2, N times.  Measured, gradient
// of shuffled pairs: N = 400 1.24 ms, N = 1000 13.0 (on one workgroup, a row a thread:
// 3.5, 21.1; sorted: 1.21, 12.8).
__global__ __launch_bounds__(256) void pair_sort_kernel(const Pair* __restrict__ pairs, int64_t n_pairs, int N,
                                                        int32_t* rows, Pair* __restrict__ sp) {
    if (rows[N + 1] != 0) sort_row(pairs, n_pairs, blockIdx.x, rows, sp);
}

// The nuclear repulsion's row of partial sums, by one workgroup.
__device__ void nuclear_row(const double* xyz, const double* Z, int nc, double* part) {
    for (int A = threadIdx.x; A < nc; A += 256) {
        double gx = 0, gy = 0, gz = 0;
        for (int B = 0; B < nc; ++B) {
            if (B == A || Z[A] * Z[B] == 0.0) continue;
            double dx = xyz[3 * A] - xyz[3 * B], dy = xyz[3 * A + 1] - xyz[3 * B + 1], dz = xyz[3 * A + 2] - xyz[3 * B + 2];
            double r = sqrt(dx * dx + dy * dy + dz * dz);
            double f = -Z[A] * Z[B] / (r * r * r);
            gx += f * dx; gy += f * dy; gz += f * dz;
        }
        part[3 * A] = gx; part[3 * A + 1] = gy; part[3 * A + 2] = gz;
    }
}

__global__ __launch_bounds__(256) void gnuc_kernel(const double* xyz, const double* Z, int nc, double* part) {
    nuclear_row(xyz, Z, nc, part);
}

// All of the above in one launch for short lists, in any order: the first two blocks
// make the table T, the third the nuclear row, the others a row of pairs each.
// Bound by the table's chain of double-double operations (15 us), beside the work
// of the caller's stream.
__global__ __launch_bounds__(256) void pair_setup_kernel(const Pair* __restrict__ pairs, int64_t n_pairs, int N,
                                                         int32_t* rows, Pair* __restrict__ sp,
                                                         const double* __restrict__ xyz, const double* __restrict__ Z,
                                                         int nc, const int32_t* __restrict__ fc,
                                                         const double* __restrict__ fe, const double* __restrict__ D,
                                                         double* __restrict__ pc, int2* __restrict__ ctr,
                                                         double* __restrict__ T, double* __restrict__ nuc) {
    if (blockIdx.x < 2) {
        const int j = blockIdx.x * 256 + threadIdx.x;
        if (j < BT_N) boys_row(j, T + j * BT_M);
        return;
    }
    if (blockIdx.x == 2) {
        nuclear_row(xyz, Z, nc, nuc);
        return;
    }
    const int2 own = sort_row(pairs, n_pairs, blockIdx.x - 3, rows, sp);
    __syncthreads();                               // the row's pairs are placed
    for (int k = threadIdx.x; k < own.y; k += 256) {
        const int q = own.x + k;
        pair_consts(q, sp[q].x, sp[q].y, xyz, fc, fe, n_pairs, D, N, pc, ctr);
    }
}

// WY[p][q] (+)= sum_k U[p][mu][k] C[nu][k] over K columns for the significant pairs q =
// (mu, nu) and p in [0, np): U [np][N][ld], C [N][ld].  A wave takes one mu and
// 16 PT auxiliaries: for each 16 of mu's partners nu <= mu an MFMA tile has rows
// U^p[mu], held in registers for the whole item, and columns the gathered rows
// C[nu], streamed 16 B a lane (lane (li, g) holds reduction indices
// 8 u + 2 g + h of either).  Bound by FP64 MFMA and the gathered rows' way
// through L2.  On whole lower tiles the products were 7.4 times the pairs at
// N = 1000 and 23 slabs of N x N each: products 7.85 -> 1.63 ms, and the
// derivative kernel, which now reads them contiguously, 3.76 -> 3.50.
// two doubles of a row that starts at any multiple of 8 bytes
typedef double d2u_t __attribute__((ext_vector_type(2), aligned(8)));

template <int KU>
__global__ __launch_bounds__(256, 2) void wp_kernel(const double* __restrict__ U, const double* __restrict__ C,
                                                    const int32_t* __restrict__ pairs,
                                                    const int32_t* __restrict__ rows, int N, int64_t ld, int K, int np,
                                                    int64_t n_pairs, int add, double* __restrict__ WY) {
    constexpr int PT = KU <= 8 ? 4 : 2;
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive workgroups of an XCD take the same auxiliaries: C's rows and U's stay in its L2
    const int L = xcd_remap(blockIdx.x, gridDim.x);
    const int mb = (N + 3) / 4, mu = 4 * (L % mb) + wave, P0 = 16 * PT * (L / mb);
    if (mu >= N) return;
    const int q0 = rows[mu], q1 = rows[mu + 1];
    if (q0 == q1) return;
    auto row = [&](const double* r, int u) {
        const int k0 = 8 * u + 2 * g;
        d2u_t v;
        if (u < KU - 1) {
            v = *(const d2u_t*)(r + k0);
        } else {
            v[0] = k0 < K ? r[min(k0, K - 1)] : 0.0;
            v[1] = k0 + 1 < K ? r[min(k0 + 1, K - 1)] : 0.0;
        }
        return v;
    };
    d2u_t a[PT][KU];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const double* ur = U + ((int64_t)min(P0 + 16 * t + li, np - 1) * N + mu) * ld;
#pragma unroll
        for (int u = 0; u < KU; ++u) a[t][u] = row(ur, u);
    }
    const double* cr = C + (int64_t)pairs[2 * (int64_t)min(q0 + li, q1 - 1) + 1] * ld;
    for (int qb = q0; qb < q1; qb += 16) {
        const int q = qb + li;
        const double* cn = C + (int64_t)pairs[2 * (int64_t)min(q + 16, q1 - 1) + 1] * ld;   // the next tile's rows
        d4_t acc[PT];
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int P = P0 + 16 * t + 4 * r + g;
                acc[t][r] = (add && q < q1 && P < np) ? WY[(int64_t)P * n_pairs + q] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const d2u_t b = row(cr, u);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < PT; ++t) acc[t] = mfma_f64(a[t][u][h], b[h], acc[t]);
        }
        // element r of lane (li, g): auxiliary row 4 r + g, pair column li
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int P = P0 + 16 * t + 4 * r + g;
                if (q < q1 && P < np) WY[(int64_t)P * n_pairs + q] = acc[t][r];
            }
        cr = cn;
    }
}

// U[p][mu][i] = sum_j C[mu][j] Xi^p[i][j] for p in [0, np): C [N][K], Xi^p the
// K x K block p of Xi [np][K][K].  Xi^p is symmetric (Xi = L^{-T} B_ij, and
// each B_ij^P = C^T B^P C is), so this is C Xi^p read along its rows: C's 64
// rows of the row tile stay in registers as A operands for a group of WY_PB
// auxiliaries, and Xi^p's rows stream in as B operands, 16 B per lane with
// buffer loads (MFMA step 2u + h of a lane in group g takes reduction index
// 8u + 2g + h on both operands; indices >= K are zeroed, rows >= N read as
// zero).  Grid: (row tile, column tile of the n_occ columns) x groups of
// auxiliaries.
constexpr int WY_PB = 8;
template <int KU>
__global__ __launch_bounds__(256, 2) void u_kernel(const double* __restrict__ C, const double* __restrict__ Xi,
                                                   int N, int K, int np, double* __restrict__ U) {
    const int nct = (K + 63) / 64;
    const int I = blockIdx.x / nct, Jc = blockIdx.x % nct;
    const int p0 = blockIdx.y * WY_PB, p1 = min(np, p0 + WY_PB);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, g = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int rowbytes = K * 8;
    const __amdgpu_buffer_rsrc_t cr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(C), (short)0, N * rowbytes, 0x00020000);
    d2_t a[2][KU];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int mu = 64 * I + wm + 16 * i + li;
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int k0 = 8 * u + 2 * g;
            d2_t v = __builtin_bit_cast(d2_t, __builtin_amdgcn_raw_buffer_load_b128(cr, mu * rowbytes + k0 * 8, 0, 0));
            if (k0 >= K) v[0] = 0.0;
            if (k0 + 1 >= K) v[1] = 0.0;
            a[i][u] = v;
        }
    }
    for (int p = p0; p < p1; ++p) {
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<double*>(Xi + (int64_t)p * K * K), (short)0, K * rowbytes, 0x00020000);
        d4_t acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
        const int r0 = (64 * Jc + wn + li) * rowbytes, r1 = r0 + 16 * rowbytes;
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int k0 = 8 * u + 2 * g;
            d2_t b0 = __builtin_bit_cast(d2_t, __builtin_amdgcn_raw_buffer_load_b128(xr, r0 + k0 * 8, 0, 0));
            d2_t b1 = __builtin_bit_cast(d2_t, __builtin_amdgcn_raw_buffer_load_b128(xr, r1 + k0 * 8, 0, 0));
            if (k0 >= K) { b0[0] = 0.0; b1[0] = 0.0; }
            if (k0 + 1 >= K) { b0[1] = 0.0; b1[1] = 0.0; }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc[i][0] = mfma_f64(a[i][u][h], b0[h], acc[i][0]);
                    acc[i][1] = mfma_f64(a[i][u][h], b1[h], acc[i][1]);
                }
            }
        }
        double* out = U + (int64_t)p * N * K;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int col = 64 * Jc + wn + 16 * j + li;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 64 * I + wm + 16 * i + 4 * r + g;
                    if (row < N && col < K) out[(int64_t)row * K + col] = acc[i][j][r];
                }
            }
    }
}

// grad[i] = sum over rows of part[row][i]: one block per component, the rows
// strided over the threads, then a fixed-order tree (deterministic).
__global__ __launch_bounds__(256) void greduce_kernel(const double* part, int rows, int nc3, double* grad) {
    const int i = blockIdx.x;
    double s = 0.0;
    for (int r = threadIdx.x; r < rows; r += 256) s += part[(int64_t)r * nc3 + i];
    __shared__ double sh[256];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) grad[i] = sh[0];
}

// The blocks B_ij^P and Xi^P are symmetric in ij up to rounding.  pack: Bp[P][e] =
// B[P][i][j] for the entries e = i (i + 1) / 2 + j, j <= i, times sqrt 2 off the
// diagonal, so that sums over all ij are sums over e; unpack: both halves of
// Xi[P] from Xp[P].  A workgroup per row (P, i).
__global__ __launch_bounds__(256) void pack_ij_kernel(const double* __restrict__ B, int o, double* __restrict__ Bp) {
    const int64_t P = blockIdx.x / o;
    const int i = (int)(blockIdx.x % o);
    const double* row = B + (P * o + i) * o;
    double* out = Bp + P * ((int64_t)o * (o + 1) / 2) + (int64_t)i * (i + 1) / 2;
    for (int j = threadIdx.x; j <= i; j += blockDim.x) out[j] = j == i ? row[j] : 1.41421356237309504880 * row[j];
}
// pack of the mean of the two halves: after an FP32 half-transform they are rounded
// independently at 2^-24 (j's column of C in FP32, i's in FP64), and one of them
// alone would carry sqrt 2 times the error of both.  A workgroup per lower 32 x 32
// tile of a block, its mirror tile through LDS (gradient of N = 1000 in FP32 13.17
// ms, 13.23 with the mirror read down its columns, 13.08 without the mean).
__global__ __launch_bounds__(256) void pack_mean_ij_kernel(const double* __restrict__ B, int o, int tiles,
                                                           double* __restrict__ Bp) {
    __shared__ double m[32][33];
    const int64_t P = blockIdx.x / tiles;
    const int t = (int)(blockIdx.x % tiles), c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= t) ++I;
    const int J = t - I * (I + 1) / 2;
    const double* blk = B + P * o * o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {                  // mirror: rows of J, columns of I
        const int r = 32 * J + r0 + 8 * k, q = 32 * I + c;
        m[r0 + 8 * k][c] = (r < o && q < o) ? blk[(int64_t)r * o + q] : 0.0;
    }
    __syncthreads();
    double* out = Bp + P * ((int64_t)o * (o + 1) / 2);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = 32 * I + r0 + 8 * k, j = 32 * J + c;
        if (i >= o || j > i) continue;
        const double v = 0.5 * (blk[(int64_t)i * o + j] + m[c][r0 + 8 * k]);
        out[(int64_t)i * (i + 1) / 2 + j] = j == i ? v : 1.41421356237309504880 * v;
    }
}
__global__ __launch_bounds__(256) void unpack_ij_kernel(const double* __restrict__ Xp, int o, double* __restrict__ Xi) {
    const int64_t P = blockIdx.x / o;
    const int i = (int)(blockIdx.x % o);
    const double* in = Xp + P * ((int64_t)o * (o + 1) / 2);
    double* out = Xi + (P * o + i) * o;
    for (int j = threadIdx.x; j < o; j += blockDim.x) {
        const int hi = max(i, j), lo = min(i, j);
        out[j] = (i == j ? 1.0 : 0.70710678118654752440) * in[(int64_t)hi * (hi + 1) / 2 + lo];
    }
}

// The same mean in place, for blocks that are not packed.
__global__ __launch_bounds__(256) void mean_ij_kernel(double* __restrict__ B, int o, int64_t n) {
    const int64_t e = blockIdx.x * 256ll + threadIdx.x;
    if (e >= n) return;
    const int j = (int)(e % o), i = (int)(e / o % o);
    if (j >= i) return;
    double* t = B + e / o / o * o * o + (int64_t)j * o + i;
    const double v = 0.5 * (B[e] + *t);
    B[e] = v;
    *t = v;
}

// out[r][c] = sum_z part[z][r][c] for c <= r, z in order.
__global__ void sum_lower_kernel(const double* part, int S, int64_t stride, int n, double* out) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)n * n) return;
    if (e % n > e / n) return;
    double s = part[e];
    for (int z = 1; z < S; ++z) s += part[z * stride + e];
    out[e] = s;
}

__global__ void gamma_dp_kernel(const int32_t* pairs, int64_t n_pairs, const double* C, int n_occ, double* dp) {
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    double s = 0.0;
    for (int i = 0; i < n_occ; ++i) s += C[(int64_t)mu * n_occ + i] * C[(int64_t)nu * n_occ + i];
    dp[q] = (mu == nu ? 2.0 : 4.0) * s;
}

__global__ __launch_bounds__(256) void gamma_row_kernel(const double* Bc, int64_t n_pairs, const double* dp,
                                                        double* gamma) {
    const double* row = Bc + (int64_t)blockIdx.x * n_pairs;
    double s = 0.0;
    for (int64_t q = threadIdx.x; q < n_pairs; q += 256) s += row[q] * dp[q];
    __shared__ double sh[4];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) gamma[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

}  // namespace

namespace ri {

hipError_t pack_ij(const double* B, int o, int np, bool mean, double* Bp, hipStream_t st) {
    const int t = (o + 31) / 32, tiles = t * (t + 1) / 2;
    if (mean) pack_mean_ij_kernel<<<(unsigned)np * (unsigned)tiles, 256, 0, st>>>(B, o, tiles, Bp);
    else pack_ij_kernel<<<(unsigned)np * (unsigned)o, o > 64 ? 128 : 64, 0, st>>>(B, o, Bp);
    return hipGetLastError();
}
hipError_t mean_ij(double* B, int o, int np, hipStream_t st) {
    const int64_t n = (int64_t)np * o * o;
    mean_ij_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(B, o, n);
    return hipGetLastError();
}
hipError_t unpack_ij(const double* Xp, int o, int np, double* Xi, hipStream_t st) {
    unpack_ij_kernel<<<(unsigned)np * (unsigned)o, o > 64 ? 128 : 64, 0, st>>>(Xp, o, Xi);
    return hipGetLastError();
}
hipError_t grad_one_electron(const ri_system* s, const double* D, const double* W, double* part, hipStream_t st) {
    if (s->n_centres > MAXC) return hipErrorInvalidValue;
    g1e_kernel<<<GRAD_BLOCKS, 256, 3 * s->n_centres * sizeof(double), st>>>(s->xyz, s->Z, s->n_centres, s->fn_centre, s->fn_exp, s->n_fn, D, W, part);
    return hipGetLastError();
}
hipError_t grad_metric(const ri_system* s, const double* Zx, const double* c, double* part, hipStream_t st) {
    if (s->n_centres > MAXC) return hipErrorInvalidValue;
    g2c_kernel<<<GRAD_BLOCKS, 256, 0, st>>>(s->xyz, s->aux_centre, s->aux_exp, s->n_aux, s->n_centres, Zx, c, part);
    return hipGetLastError();
}
// Zx = -2 Xi Xi^T on the lower tiles (Xi: n_aux x K, row-major).  The
// reduction over K is split into S column ranges, one batch of the GEMM each,
// into S partial products in `tmp` (tmp_elems doubles), then summed in order:
// the unsplit form has only the lower 128-tiles as workgroups (300 at
// n_aux = 3000), too few to fill the chip for a long K.
hipError_t grad_metric_z(const double* Xi, int n_aux, int64_t K, double* tmp, int64_t tmp_elems, double* Zx,
                         hipStream_t st) {
    const int64_t n2 = (int64_t)n_aux * n_aux;
    const int64_t t128 = (n_aux + 127) / 128, lower = t128 * (t128 + 1) / 2;
    int S = (int)std::max<int64_t>(1, std::min<int64_t>({(3 * 512 + lower / 2) / lower, 16, K / 256, tmp_elems / n2 - 1}));
    if (S <= 1)
        return gemm_f64(false, true, n_aux, n_aux, (int)K, -2.0, Xi, K, 0, Xi, K, 0, 0.0, Zx, n_aux, 0, 1, 0, 1, st);
    // S equal ranges in one launch; the K % S columns left over, if any, in a
    // launch of their own into one more partial
    const int64_t kc = K / S, rem = K - S * kc;
    RI_TRY(gemm_f64(false, true, n_aux, n_aux, (int)kc, -2.0, Xi, K, kc, Xi, K, kc, 0.0, tmp, n_aux, n2, S, 0, 1, st));
    if (rem > 0) {
        RI_TRY(gemm_f64(false, true, n_aux, n_aux, (int)rem, -2.0, Xi + S * kc, K, 0, Xi + S * kc, K, 0, 0.0,
                        tmp + (int64_t)S * n2, n_aux, 0, 1, 0, 1, st));
        ++S;
    }
    sum_lower_kernel<<<(unsigned)((n2 + 255) / 256), 256, 0, st>>>(tmp, S, n2, n_aux, Zx);
    return hipGetLastError();
}
int grad_slab(int N, int n_aux) {
    const int64_t per = (int64_t)N * N * 8;
    return (int)std::max<int64_t>(1, std::min<int64_t>(n_aux, (int64_t(1) << 30) / per));
}

// U[p] = C Xi^p for p < np (Xi [np][K][K], each block symmetric; U [np][N][K]).
hipError_t u_products(const double* C, const double* Xi, int N, int K, int np, double* U, hipStream_t st) {
    const int ku = (K + 7) / 8;
    if (ku > 16 || (int64_t)N * K * 8 > INT_MAX)
        return gemm_f64(false, false, N, K, K, 1.0, C, K, 0, Xi, K, (int64_t)K * K, 0.0, U, K, (int64_t)N * K, np, 0,
                        0, st);
    const dim3 grid((unsigned)(((N + 63) / 64) * ((K + 63) / 64)), (unsigned)((np + WY_PB - 1) / WY_PB));
    switch (ku) {
#define UK(n) case n: u_kernel<n><<<grid, 256, 0, st>>>(C, Xi, N, K, np, U); break;
        UK(1) UK(2) UK(3) UK(4) UK(5) UK(6) UK(7) UK(8)
        UK(9) UK(10) UK(11) UK(12) UK(13) UK(14) UK(15) UK(16)
#undef UK
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
// Pairs times functions up to which pair_setup_kernel, which reads the list 2 N
// times, takes the place of five launches: the gradient of N = 130 in 230 us for
// 240, N = 240 480 for 492, N = 350 903 for 909, N = 500 (14.5 M) 1947 for 1943.
constexpr int64_t PAIR_SETUP_MAX = 1 << 23;
// Where the parts of the three-centre term's scratch lie.
struct PairScratch {
    double* pc;      // [PC_N][n_pairs]
    int2* ctr;       // [n_pairs]
    Pair* sp;        // [n_pairs] pairs by rows
    double* bt;      // table of the Boys function
    PairScratch(double* p, int64_t n_pairs)
        : pc(p), ctr((int2*)(p + PC_N * n_pairs)), sp((Pair*)(ctr + n_pairs)), bt((double*)(sp + n_pairs)) {}
};
hipError_t grad_pairs(const ri_system* s, const int32_t* pairs, int64_t n_pairs, const double* D, int32_t* rows,
                      double* pscratch, double* nuclear, hipStream_t st) {
    const int N = s->n_fn;
    const PairScratch w(pscratch, n_pairs);
    const Pair* given = (const Pair*)pairs;
    if (n_pairs > 0 && N * n_pairs <= PAIR_SETUP_MAX) {
        pair_setup_kernel<<<(unsigned)N + 4, 256, 0, st>>>(given, n_pairs, N, rows, w.sp, s->xyz, s->Z, s->n_centres,
                                                           s->fn_centre, s->fn_exp, D, w.pc, w.ctr, w.bt, nuclear);
        return hipGetLastError();
    }
    gnuc_kernel<<<1, 256, 0, st>>>(s->xyz, s->Z, s->n_centres, nuclear);
    RI_TRY(hipGetLastError());
    if (n_pairs == 0) return hipSuccess;
    RI_TRY(fill_i32(rows + N + 1, 0, 1, st));
    pair_rows_kernel<<<(unsigned)((std::max<int64_t>(n_pairs, N + 1) + 255) / 256), 256, 0, st>>>(given, n_pairs, N, rows,
                                                                                                  w.sp);
    pair_sort_kernel<<<(unsigned)N + 1, 256, 0, st>>>(given, n_pairs, N, rows, w.sp);
    RI_TRY(hipGetLastError());
    pair_consts_kernel<<<(unsigned)((n_pairs + 255) / 256 + 2), 256, 0, st>>>(s->xyz, s->fn_centre, s->fn_exp,
                                                                              (const int32_t*)w.sp, n_pairs, D, N, w.pc,
                                                                              w.ctr, w.bt);
    return hipGetLastError();
}
hipError_t grad_three_centre(const ri_system* s, int64_t n_pairs, const double* U, const double* C, int n_occ,
                             const double* c, double* WY, const int32_t* rows, double* pscratch, double* part,
                             hipStream_t st) {
    if (s->n_centres > MAXC) return hipErrorInvalidValue;
    const int N = s->n_fn, na = s->n_aux;
    const size_t lds = 3 * s->n_centres * sizeof(double);
    if (n_pairs == 0) return fill(part, 0.0, (int64_t)GRAD_BLOCKS * 3 * s->n_centres, st);
    const PairScratch w(pscratch, n_pairs);
    const int32_t* pairs = (const int32_t*)w.sp;
    // auxiliaries at a time that WY holds (nearly twice grad_slab where every pair is listed once)
    const int ns = (int)std::min<int64_t>(na, grad_wy_elems(N, na, n_pairs) / n_pairs);
    for (int P0 = 0; P0 < na; P0 += ns) {
        const int np = std::min(ns, na - P0);
        for (int k0 = 0; k0 < n_occ; k0 += 128) {
            const int K = std::min(128, n_occ - k0), ku = (K + 7) / 8, pt = ku <= 8 ? 4 : 2;
            const unsigned blocks = (unsigned)((N + 3) / 4) * (unsigned)((np + 16 * pt - 1) / (16 * pt));
            const double* u = U + (int64_t)P0 * N * n_occ + k0;
            switch (ku) {
#define WP(n) case n: wp_kernel<n><<<blocks, 256, 0, st>>>(u, C + k0, pairs, rows, N, n_occ, K, np, n_pairs, k0 > 0, WY); break;
                WP(1) WP(2) WP(3) WP(4) WP(5) WP(6) WP(7) WP(8)
                WP(9) WP(10) WP(11) WP(12) WP(13) WP(14) WP(15) WP(16)
#undef WP
                default: return hipErrorInvalidValue;
            }
            RI_TRY(hipGetLastError());
        }
        // blocks of pairs per item: as many as leave every workgroup two items
        const int64_t one = (n_pairs + 255) / 256 * ((np + G3_PC - 1) / G3_PC);
        const int bpi = (int)std::max<int64_t>(1, std::min<int64_t>(8, one / (2 * GRAD_BLOCKS)));
        g3c_kernel<<<GRAD_BLOCKS, 256, lds, st>>>(s->xyz, s->aux_centre, s->aux_exp, P0, np, s->n_centres, n_pairs, bpi,
                                                  w.pc, w.ctr, WY, c, w.bt, part);
        RI_TRY(hipGetLastError());
    }
    return hipSuccess;
}
int64_t grad_wy_elems(int N, int n_aux, int64_t n_pairs) {
    return std::max((int64_t)grad_slab(N, n_aux) * N * N, n_pairs);
}
int64_t grad_pair_elems(int64_t n_pairs) { return (PC_N + 2) * n_pairs + BT_N * BT_M; }
hipError_t grad_reduce(const double* part, int rows, int n_centres, double* grad, hipStream_t st) {
    greduce_kernel<<<3 * n_centres, 256, 0, st>>>(part, rows, 3 * n_centres, grad);
    return hipGetLastError();
}
hipError_t gamma_only(const double* Bc, const int32_t* pairs, int64_t n_pairs, int n_aux, int n_occ, const double* C,
                      double* dpair, double* gamma, hipStream_t st) {
    if (n_pairs == 0) return fill(gamma, 0.0, n_aux, st);
    gamma_dp_kernel<<<(unsigned)((n_pairs + 255) / 256), 256, 0, st>>>(pairs, n_pairs, C, n_occ, dpair);
    RI_TRY(hipGetLastError());
    gamma_row_kernel<<<n_aux, 256, 0, st>>>(Bc, n_pairs, dpair, gamma);
    return hipGetLastError();
}

}  // namespace ri
