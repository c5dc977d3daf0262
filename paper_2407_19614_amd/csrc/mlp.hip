// Learned SCF start (project extension): per-pair features, a 3-layer MLP
// (width 256, SiLU) trained in FP32 with its own forward, backward and Adam
// kernels, BF16 inference for the 256 x 256 layer, and the scatter of
// predicted pair densities into a dense symmetric matrix.
#include "kernels.h"
#include "mlp_split.h"

#include <algorithm>

namespace {

constexpr int NF = RI_MLP_NFEAT;
constexpr int W = RI_MLP_WIDTH;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float silu(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
    float s = 1.0f / (1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}
__device__ __forceinline__ f4_t mfma_f32x4(float a, float b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// f0 |A-B|, f1 ln max(a,b), f2 ln min(a,b), f3 same centre, f4 exp(-(ab/(a+b))|A-B|^2),
// f5/f6 max/min coordination sum_{C != X} exp(-|R_X - R_C|^2 / 8),
// f7 sum_C exp(-|P - R_C|^2 / 4) at the Gaussian product centre P.
// Bound by the exponentials.  The coordination depends on the centre only, so
// each workgroup forms it once for all centres (8 partial sums each, in
// dynamic LDS: 9 nc doubles) where COORD is set; the pair then needs one
// exponential per centre instead of three.
template <bool COORD>
__global__ __launch_bounds__(256) void features_kernel(const double* __restrict__ xyz, int nc,
                                                       const int32_t* __restrict__ fc,
                                                       const double* __restrict__ fe,
                                                       const int32_t* __restrict__ pairs, int64_t n_pairs,
                                                       float* __restrict__ feat) {
    extern __shared__ double cs[];   // [nc] coordination, then [nc][8] partial sums
    if (COORD) {
        for (int e = threadIdx.x; e < 8 * nc; e += 256) {
            const int X = e >> 3;
            const double x = xyz[3 * X], y = xyz[3 * X + 1], z = xyz[3 * X + 2];
            double v = 0.0;
            for (int c = e & 7; c < nc; c += 8) {
                const double dx = x - xyz[3 * c], dy = y - xyz[3 * c + 1], dz = z - xyz[3 * c + 2];
                if (c != X) v += exp(-(dx * dx + dy * dy + dz * dz) / 8.0);
            }
            cs[nc + e] = v;
        }
        __syncthreads();
        for (int X = threadIdx.x; X < nc; X += 256) {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) v += cs[nc + 8 * X + k];
            cs[X] = v;
        }
        __syncthreads();
    }
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    int ca = fc[mu], cb = fc[nu];
    double a = fe[mu], b = fe[nu];
    const double* A = xyz + 3 * ca;
    const double* B = xyz + 3 * cb;
    double dx = A[0] - B[0], dy = A[1] - B[1], dz = A[2] - B[2];
    double r2 = dx * dx + dy * dy + dz * dz;
    double Px = (a * A[0] + b * B[0]) / (a + b), Py = (a * A[1] + b * B[1]) / (a + b),
           Pz = (a * A[2] + b * B[2]) / (a + b);
    double cA = COORD ? cs[ca] : 0.0, cB = COORD ? cs[cb] : 0.0, md = 0.0;
    for (int c = 0; c < nc; ++c) {
        const double* C = xyz + 3 * c;
        double px = Px - C[0], py = Py - C[1], pz = Pz - C[2];
        md += exp(-(px * px + py * py + pz * pz) / 4.0);
        if (!COORD) {
            double ax = A[0] - C[0], ay = A[1] - C[1], az = A[2] - C[2];
            double bx = B[0] - C[0], by = B[1] - C[1], bz = B[2] - C[2];
            if (c != ca) cA += exp(-(ax * ax + ay * ay + az * az) / 8.0);
            if (c != cb) cB += exp(-(bx * bx + by * by + bz * bz) / 8.0);
        }
    }
    float* f = feat + q * NF;
    f[0] = (float)sqrt(r2);
    f[1] = (float)log(fmax(a, b));
    f[2] = (float)log(fmin(a, b));
    f[3] = ca == cb ? 1.0f : 0.0f;
    f[4] = (float)exp(-(a * b / (a + b)) * r2);
    f[5] = (float)fmax(cA, cB);
    f[6] = (float)fmin(cA, cB);
    f[7] = (float)md;
}

// Layout of one block's partial sums in a training step (columns of `part`)
constexpr int PW1 = 0, PB1 = PW1 + NF * W, PB2 = PB1 + W, PW3 = PB2 + W, PB3 = PW3 + W, PLOSS = PB3 + 1, PCOLS = PLOSS + 1;

// The network on 32 MT rows, all three layers in one launch, and with TRAIN
// the loss and the backward pass of the same rows down to the partial sums of
// every gradient but W2's, so that the activations never leave the chip
// except for h1 and dz2, the operands of that one product.
// The 256 x 256 layer runs on MFMA: 8 waves, each 16 MT rows x 64 columns
// (MT x 4 tiles); its A operand comes from the block's activations in LDS
// (rows padded by 4 floats or 8 bfloat16: conflict-free), its B operand
// straight from W2 in 16-byte loads, since 256 KB of weights do not fit beside
// them and are shared by every block through L2.
//   forward FP32: columns 4 li + t of tile t, one load for four tiles;
//   forward BF16: columns 16 t + li from W2^T in bfloat16, 32-deep MFMAs;
//   backward: output columns 16 t + li are rows of W2, one load for four
//   k-steps (k = 16 u + 4 g + h on both operands).
// Bound by MFMA throughput (the FP32 step's 4.3 GFLOP of this kernel take 27
// us at peak) and the latency of the weight loads.  Before, each layer,
// elementwise step and column sum was a launch of its own over the activations
// in memory.  Measured, training step of 16384 rows: 5171 -> 98 us (this kernel
// 73, g_W2 25, the update 11; g_W2 and g_W1 alone took 4761 on 20 workgroups);
// BF16 inference with the features of 22,000 pairs: 99 -> 36 us.
template <bool BF16, bool TRAIN, int MT>
__global__ __launch_bounds__(512, 2) void mlp_kernel(const float* __restrict__ feat, int64_t n,
                                                     const float* __restrict__ mu, const float* __restrict__ sg,
                                                     const float* __restrict__ P, const __bf16* __restrict__ W2t,
                                                     float* __restrict__ y_out, const float* __restrict__ target,
                                                     float* __restrict__ h1g, float* __restrict__ dz2g,
                                                     float* __restrict__ part) {
    constexpr int RB = 32 * MT;
    constexpr int LDF = W + 4, LDB = W + 8;
    __shared__ __align__(16) float H[BF16 ? RB * LDB / 2 : RB * LDF];   // h1, then dz2
    __shared__ float X[RB][NF];
    __shared__ float ys[4][RB], dyv[RB];
    const float* W1 = P + RI_MLP_OFF_W1;
    const float* W2 = P + RI_MLP_OFF_W2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * RB;
    for (int e = tid; e < RB * NF; e += 512) {
        const int r = e / NF, k = e % NF;
        X[r][k] = r0 + r < n ? (feat[(r0 + r) * NF + k] - mu[k]) / sg[k] : 0.0f;
    }
    __syncthreads();
    {
        const int c = tid & (W - 1);
        float w[NF];
#pragma unroll
        for (int k = 0; k < NF; ++k) w[k] = W1[k * W + c];
        const float b = P[RI_MLP_OFF_B1 + c];
        for (int r = tid >> 8; r < RB; r += 2) {
            float z = b;
#pragma unroll
            for (int k = 0; k < NF; ++k) z += X[r][k] * w[k];
            const float h = silu(z);
            if constexpr (BF16) ((__bf16*)H)[r * LDB + c] = (__bf16)h;
            else H[r * LDF + c] = h;
            if (TRAIN) h1g[(r0 + r) * W + c] = h;
        }
    }
    __syncthreads();
    const int wr = (wave >> 2) * 16 * MT, cq = (wave & 3) * 64;
    auto col = [&](int t) { return cq + (BF16 ? 16 * t + li : 4 * li + t); };
    f4_t acc[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i][t] = f4_t{0, 0, 0, 0};
    if constexpr (BF16) {
        const __bf16* Hb = (const __bf16*)H;
#pragma unroll
        for (int k0 = 0; k0 < W; k0 += 32) {
            bf16x8_t b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t] = *(const bf16x8_t*)(W2t + (int64_t)(cq + 16 * t + li) * W + k0 + 8 * lk);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const bf16x8_t a = *(const bf16x8_t*)(Hb + (wr + 16 * i + li) * LDB + k0 + 8 * lk);
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[t], acc[i][t], 0, 0, 0);
            }
        }
    } else {
        const float* bp = W2 + lk * W + cq + 4 * li;
        constexpr int D = 8;                       // k-steps of weights in flight
        f4_t b[D];
#pragma unroll
        for (int d = 0; d < D; ++d) b[d] = *(const f4_t*)(bp + 4 * d * W);
        for (int s0 = 0; s0 < W / 4; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int s = s0 + d;
                float a[MT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = H[(wr + 16 * i + li) * LDF + 4 * s + lk];
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[i][t] = mfma_f32x4(a[i], b[d][t], acc[i][t]);
                b[d] = *(const f4_t*)(bp + 4 * min(s + D, W / 4 - 1) * W);
            }
        }
    }
    // element q of lane (li, lk) in tile (i, t): row wr + 16 i + 4 lk + q, column col(t)
    float w3[4], b2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        w3[t] = P[RI_MLP_OFF_W3 + col(t)];
        b2[t] = P[RI_MLP_OFF_B2 + col(t)];
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v = 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                acc[i][t][q] += b2[t];             // z2
                v += silu(acc[i][t][q]) * w3[t];
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (li == 0) ys[wave & 3][wr + 16 * i + 4 * lk + q] = v;
        }
    __syncthreads();                               // also: every wave has read h1
    if (tid < RB) {
        const float y = ys[0][tid] + ys[1][tid] + ys[2][tid] + ys[3][tid] + P[RI_MLP_OFF_B3];
        const bool in = r0 + tid < n;
        if (!TRAIN && in) y_out[r0 + tid] = y;
        if (TRAIN) {
            const float r = in ? y - target[r0 + tid] : 0.0f;
            dyv[tid] = 2.0f * r / (float)n;
            ys[0][tid] = r * r;
        }
    }
    if constexpr (TRAIN) {
        static_assert(!BF16, "training is FP32");
        __syncthreads();
        float* pp = part + (int64_t)blockIdx.x * PCOLS;
        if (tid == 0) {
            float l = 0.0f, d = 0.0f;
            for (int r = 0; r < RB; ++r) {
                l += ys[0][r];
                d += dyv[r];
            }
            pp[PLOSS] = l;
            pp[PB3] = d;
        }
        float g3[4], gb[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) g3[t] = gb[t] = 0.0f;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = wr + 16 * i + 4 * lk + q;
                const float dy = dyv[row];
                f4_t o;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float z = acc[i][t][q];
                    g3[t] += silu(z) * dy;
                    o[t] = dy * w3[t] * dsilu(z);
                    gb[t] += o[t];
                }
                *(f4_t*)(H + row * LDF + cq + 4 * li) = o;
                *(f4_t*)(dz2g + (r0 + row) * W + cq + 4 * li) = o;
            }
        __shared__ float red[PB3];                 // the upper rows' share of the column sums
        auto colsum = [&](float v, int at, bool low) {
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (lk == 0) {
                if (low) pp[at] = v + red[at];
                else red[at] = v;
            }
        };
        const bool low = wave < 4;
        if (!low)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                colsum(g3[t], PW3 + col(t), false);
                colsum(gb[t], PB2 + col(t), false);
            }
        __syncthreads();
        if (low)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                colsum(g3[t], PW3 + col(t), true);
                colsum(gb[t], PB2 + col(t), true);
            }
        // dh1 = dz2 W2^T
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[i][t] = f4_t{0, 0, 0, 0};
        f4_t b[2][4];
        const float* bp = W2 + (int64_t)(cq + li) * W + 4 * lk;
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int t = 0; t < 4; ++t) b[d][t] = *(const f4_t*)(bp + 16 * t * W + 16 * d);
        for (int u0 = 0; u0 < W / 16; u0 += 2) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int u = u0 + d;
                f4_t a[MT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = *(const f4_t*)(H + (wr + 16 * i + li) * LDF + 16 * u + 4 * lk);
#pragma unroll
                for (int h = 0; h < 4; ++h)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[i][t] = mfma_f32x4(a[i][h], b[d][t][h], acc[i][t]);
#pragma unroll
                for (int t = 0; t < 4; ++t) b[d][t] = *(const f4_t*)(bp + 16 * t * W + 16 * min(u + 2, W / 16 - 1));
            }
        }
        // dz1 = dh1 silu'(z1) with z1 formed again, and its sums; columns 16 t + li
        float hold[4][NF + 1];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int c = cq + 16 * t + li;
            float w[NF], g[NF], s = 0.0f;
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                w[k] = W1[k * W + c];
                g[k] = 0.0f;
            }
            const float b1 = P[RI_MLP_OFF_B1 + c];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float* x = X[wr + 16 * i + 4 * lk + q];
                    float z = b1;
#pragma unroll
                    for (int k = 0; k < NF; ++k) z += x[k] * w[k];
                    const float d = acc[i][t][q] * dsilu(z);
                    s += d;
#pragma unroll
                    for (int k = 0; k < NF; ++k) g[k] += x[k] * d;
                }
            if (!low) {
                colsum(s, PB1 + c, false);
#pragma unroll
                for (int k = 0; k < NF; ++k) colsum(g[k], PW1 + k * W + c, false);
            } else {
                hold[t][0] = s;
#pragma unroll
                for (int k = 0; k < NF; ++k) hold[t][k + 1] = g[k];
            }
        }
        __syncthreads();
        if (low)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = cq + 16 * t + li;
                colsum(hold[t][0], PB1 + c, true);
#pragma unroll
                for (int k = 0; k < NF; ++k) colsum(hold[t][k + 1], PW1 + k * W + c, true);
            }
    }
}

// g_W2 partials: rows r of one split of h1^T dz2 (both [rows][256], rows a
// multiple of 32).  One 64 x 64 tile per workgroup; each of its 4 waves takes
// a quarter of the split's rows over the whole tile, its operands straight
// from memory (16 bytes per lane: rows m = 4 li + i, columns 4 li + j of tile
// (i, j)), and the four sums meet in LDS.  The product has 16 tiles only, so
// the reduction over the rows is split to fill the chip; without that it ran
// on 16 workgroups (2.4 ms for 16384 rows).
__global__ __launch_bounds__(256, 2) void gw2_kernel(const float* __restrict__ h1, const float* __restrict__ dz2,
                                                     int64_t rows, int64_t per, float* __restrict__ part) {
    __shared__ f4_t sh[3][64][17];
    const int tile = blockIdx.x & 15, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t z = blockIdx.x >> 4;
    const int m0 = (tile >> 2) * 64, n0 = (tile & 3) * 64;
    const int64_t a0 = (4 * z + wave) * per, a1 = min(rows, a0 + per);
    f4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f4_t{0, 0, 0, 0};
    const float* ap = h1 + (a0 + lk) * W + m0 + 4 * li;
    const float* bp = dz2 + (a0 + lk) * W + n0 + 4 * li;
    const int steps = a1 > a0 ? (int)((a1 - a0) / 4) : 0;
    constexpr int D = 4;
    if (steps > 0) {                               // per and rows are multiples of 16: steps of D
        f4_t a[D], b[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            a[d] = *(const f4_t*)(ap + (int64_t)d * 4 * W);
            b[d] = *(const f4_t*)(bp + (int64_t)d * 4 * W);
        }
        for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f32x4(a[d][i], b[d][j], acc[i][j]);
                const int64_t nx = (int64_t)min(s0 + d + D, steps - 1) * 4 * W;
                a[d] = *(const f4_t*)(ap + nx);
                b[d] = *(const f4_t*)(bp + nx);
            }
        }
    }
    if (wave > 0)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) sh[wave - 1][lane][4 * i + j] = acc[i][j];
    __syncthreads();
    if (wave > 0) return;
    float* out = part + z * (W * W);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int w = 0; w < 3; ++w) acc[i][j] += sh[w][lane][4 * i + j];
        }
    // element q of tile (i, j): row m0 + 4 (4 lk + q) + i, columns n0 + 4 li + j
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4_t v = f4_t{acc[i][0][q], acc[i][1][q], acc[i][2][q], acc[i][3][q]};
            *(f4_t*)(out + (m0 + 4 * (4 * lk + q) + i) * W + n0 + 4 * li) = v;
        }
}

// The gradient from its partial sums (W2's splits in pw2, everything else and
// the loss in pr, one row per block), and the Adam update.  Blocks
// 0 .. 255 take W2's rows, the others 32 further columns each (8 threads per
// column over the rows, summed in one fixed order).
__global__ __launch_bounds__(256) void grad_adam_kernel(const float* __restrict__ pw2, int splits,
                                                        const float* __restrict__ pr, int nrow, float inv_n,
                                                        float* __restrict__ p, float* __restrict__ g_out,
                                                        float* __restrict__ m, float* __restrict__ v,
                                                        float* __restrict__ loss, float lr, float b1, float b2,
                                                        float eps, float c1, float c2) {
    __shared__ float sh[8][33];
    int i = -1;
    float gi = 0.0f;
    if (blockIdx.x < W) {
        const int e = blockIdx.x * W + threadIdx.x;
        for (int z = 0; z < splits; ++z) gi += pw2[(int64_t)z * (W * W) + e];
        i = RI_MLP_OFF_W2 + e;
    } else {
        const int c = threadIdx.x & 31, k = threadIdx.x >> 5, e = (blockIdx.x - W) * 32 + c;
        float s = 0.0f;
        if (e < PCOLS)
            for (int r = k; r < nrow; r += 8) s += pr[(int64_t)r * PCOLS + e];
        sh[k][c] = s;
        __syncthreads();
        if (k != 0 || e >= PCOLS) return;
#pragma unroll
        for (int j = 0; j < 8; ++j) gi += sh[j][c];
        if (e == PLOSS) {
            *loss = gi * inv_n;
            return;
        }
        i = e < PB1 ? RI_MLP_OFF_W1 + e : e < PB2 ? RI_MLP_OFF_B1 + e - PB1 : e < PW3 ? RI_MLP_OFF_B2 + e - PB2
            : e < PB3 ? RI_MLP_OFF_W3 + e - PW3 : RI_MLP_OFF_B3;
    }
    if (g_out) g_out[i] = gi;
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void transpose_bf16_kernel(const float* W2, __bf16* W2t) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= W * W) return;
    int k = e / W, c = e % W;
    W2t[c * W + k] = (__bf16)W2[e];
}

__global__ void scatter_density_kernel(const int32_t* pairs, int64_t n_pairs, const float* d, int N, double* D) {
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    double v = d[q];
    D[(int64_t)mu * N + nu] = v;
    D[(int64_t)nu * N + mu] = v;
}

__global__ void gather_density_kernel(const int32_t* pairs, int64_t n_pairs, const double* D, int N, float* d) {
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    d[q] = (float)D[(int64_t)pairs[2 * q] * N + pairs[2 * q + 1]];
}

// Distance^2 of the pair's centres, the coordination sum c_A + c_B and the
// Gaussian-product-centre density (f7 above) of one geometry.
__device__ __forceinline__ void pair_geometry(const double* xyz, int nc, int ca, int cb, double a, double b,
                                              double& r2, double& csum, double& md) {
    const double* A = xyz + 3 * ca;
    const double* B = xyz + 3 * cb;
    const double dx = A[0] - B[0], dy = A[1] - B[1], dz = A[2] - B[2];
    r2 = dx * dx + dy * dy + dz * dz;
    const double Px = (a * A[0] + b * B[0]) / (a + b), Py = (a * A[1] + b * B[1]) / (a + b),
                 Pz = (a * A[2] + b * B[2]) / (a + b);
    double cA = 0.0, cB = 0.0, m = 0.0;
    for (int c = 0; c < nc; ++c) {
        const double* C = xyz + 3 * c;
        const double ax = A[0] - C[0], ay = A[1] - C[1], az = A[2] - C[2];
        const double bx = B[0] - C[0], by = B[1] - C[1], bz = B[2] - C[2];
        const double px = Px - C[0], py = Py - C[1], pz = Pz - C[2];
        if (c != ca) cA += exp(-(ax * ax + ay * ay + az * az) / 8.0);
        if (c != cb) cB += exp(-(bx * bx + by * by + bz * bz) / 8.0);
        m += exp(-(px * px + py * py + pz * pz) / 4.0);
    }
    csum = cA + cB;
    md = m;
}

// Features of a pair for the density change between the previous geometry
// (xyz0, converged density Dp) and the new one (xyz): g0 = Dp[mu][nu],
// g1 = change of |A - B|, g2 = change of exp(-(ab/(a+b))|A-B|^2), g3/g4 =
// ln max/min(a, b), g5 = same centre, g6 = change of c_A + c_B, g7 = change of
// the product-centre density.
__global__ void delta_features_kernel(const double* xyz, const double* xyz0, int nc, const int32_t* fc,
                                      const double* fe, const int32_t* pairs, int64_t n_pairs, const double* Dp,
                                      int N, float* feat) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    const int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    const int ca = fc[mu], cb = fc[nu];
    const double a = fe[mu], b = fe[nu], e = a * b / (a + b);
    double r2, cs, md, r20, cs0, md0;
    pair_geometry(xyz, nc, ca, cb, a, b, r2, cs, md);
    pair_geometry(xyz0, nc, ca, cb, a, b, r20, cs0, md0);
    float* f = feat + q * NF;
    f[0] = (float)Dp[(int64_t)mu * N + nu];
    f[1] = (float)(sqrt(r2) - sqrt(r20));
    f[2] = (float)(exp(-e * r2) - exp(-e * r20));
    f[3] = (float)log(fmax(a, b));
    f[4] = (float)log(fmin(a, b));
    f[5] = ca == cb ? 1.0f : 0.0f;
    f[6] = (float)(cs - cs0);
    f[7] = (float)(md - md0);
}

// d[q] = scale (Dn - Dp)[mu][nu] on the listed pairs
__global__ void density_change_kernel(const int32_t* pairs, int64_t n_pairs, const double* Dn, const double* Dp,
                                      int N, float scale, float* d) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    const int64_t i = (int64_t)pairs[2 * q] * N + pairs[2 * q + 1];
    d[q] = (float)((double)scale * (Dn[i] - Dp[i]));
}

// Dout[mu][nu] = Dout[nu][mu] = Dp[mu][nu] + scale d[q] on the listed pairs
// (Dout holds a copy of Dp elsewhere)
__global__ void density_add_kernel(const int32_t* pairs, int64_t n_pairs, const float* d, double scale,
                                   const double* Dp, int N, double* Dout) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    const int mu = pairs[2 * q], nu = pairs[2 * q + 1];
    const double v = Dp[(int64_t)mu * N + nu] + scale * (double)d[q];
    Dout[(int64_t)mu * N + nu] = v;
    Dout[(int64_t)nu * N + mu] = v;
}

// Rows per workgroup: 64, or 32 where 64 would leave most of the 256 CUs idle.
int block_rows(int64_t n) { return n > 64 * 256 / 2 ? 64 : 32; }

inline unsigned g1(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

}  // namespace

namespace ri {

hipError_t pair_features(const ri_system* s, const int32_t* pairs, int64_t n_pairs, float* feat, hipStream_t st) {
    if (n_pairs == 0) return hipSuccess;
    const size_t lds = 9 * sizeof(double) * (size_t)s->n_centres;
    if (lds <= 32768)   // 455 centres; beyond, the sums no longer leave room for several workgroups per CU
        features_kernel<true><<<g1(n_pairs), 256, lds, st>>>(s->xyz, s->n_centres, s->fn_centre, s->fn_exp, pairs,
                                                             n_pairs, feat);
    else
        features_kernel<false><<<g1(n_pairs), 256, 0, st>>>(s->xyz, s->n_centres, s->fn_centre, s->fn_exp, pairs,
                                                            n_pairs, feat);
    return hipGetLastError();
}

MlpWS carve_mlp(char* base, size_t cap, size_t& off, int64_t n) {
    auto take = [&](int64_t cnt, size_t esz) {
        size_t b = ((size_t)cnt * esz + 255) & ~(size_t)255;
        size_t o = off;
        off += b;
        return base ? (void*)(base + o) : nullptr;
    };
    MlpWS w;
    const int64_t rows = (n + 63) / 64 * 64;
    w.h1 = (float*)take(rows * W, 4);
    w.dz2 = (float*)take(rows * W, 4);
    w.part = (float*)take((rows / 32) * PCOLS, 4);
    w.pw2 = (float*)take((int64_t)GW2_SPLITS * W * W, 4);
    w.W2t = (__bf16*)take(W * W, 2);
    (void)cap;
    return w;
}

hipError_t mlp_forward(const ri_mlp* net, const float* feat, int64_t n, float* y, int prec, const MlpWS& w,
                       hipStream_t st) {
    const float* P = net->params;
    const int rb = block_rows(n);
    if (prec == RI_MLP_BF16) {
        transpose_bf16_kernel<<<g1(W * W), 256, 0, st>>>(P + RI_MLP_OFF_W2, w.W2t);
        RI_TRY(hipGetLastError());
    }
#define FWD(B, M) mlp_kernel<B, false, M><<<g1(n, rb), 512, 0, st>>>(feat, n, net->mu, net->sigma, P, w.W2t, y, \
                                                                     nullptr, nullptr, nullptr, nullptr)
    if (prec == RI_MLP_BF16) {
        if (rb == 64) FWD(true, 2); else FWD(true, 1);
    } else {
        if (rb == 64) FWD(false, 2); else FWD(false, 1);
    }
#undef FWD
    return hipGetLastError();
}

hipError_t mlp_train_step(const ri_mlp* net, float* m, float* v, int step, float lr, const float* feat,
                          const float* target, int64_t n, float* loss, float* grad, const MlpWS& w, hipStream_t st) {
    float* P = net->params;
    const int rb = block_rows(n), nblk = (int)g1(n, rb);
    if (rb == 64)
        mlp_kernel<false, true, 2><<<nblk, 512, 0, st>>>(feat, n, net->mu, net->sigma, P, nullptr, nullptr, target,
                                                         w.h1, w.dz2, w.part);
    else
        mlp_kernel<false, true, 1><<<nblk, 512, 0, st>>>(feat, n, net->mu, net->sigma, P, nullptr, nullptr, target,
                                                         w.h1, w.dz2, w.part);
    RI_TRY(hipGetLastError());
    const int64_t rows = (int64_t)nblk * rb;
    const auto [per, splits] = gw2_split(rows);
    if (splits > GW2_SPLITS) return hipErrorInvalidValue;
    gw2_kernel<<<16 * splits, 256, 0, st>>>(w.h1, w.dz2, rows, per, w.pw2);
    RI_TRY(hipGetLastError());
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    grad_adam_kernel<<<W + (PCOLS + 31) / 32, 256, 0, st>>>(w.pw2, splits, w.part, nblk, 1.0f / (float)n, P, grad, m, v,
                                                            loss, lr, b1, b2, 1e-8f, c1, c2);
    return hipGetLastError();
}

hipError_t scatter_density(int N, const int32_t* pairs, int64_t n_pairs, const float* d, double* D, hipStream_t st) {
    RI_TRY(fill(D, 0.0, (int64_t)N * N, st));
    if (n_pairs == 0) return hipSuccess;
    scatter_density_kernel<<<g1(n_pairs), 256, 0, st>>>(pairs, n_pairs, d, N, D);
    return hipGetLastError();
}

hipError_t pair_delta_features(const ri_system* s, const double* xyz_prev, const int32_t* pairs, int64_t n_pairs,
                               const double* D_prev, float* feat, hipStream_t st) {
    if (n_pairs == 0) return hipSuccess;
    delta_features_kernel<<<g1(n_pairs), 256, 0, st>>>(s->xyz, xyz_prev, s->n_centres, s->fn_centre, s->fn_exp,
                                                        pairs, n_pairs, D_prev, s->n_fn, feat);
    return hipGetLastError();
}

hipError_t density_change(int N, const int32_t* pairs, int64_t n_pairs, const double* Dn, const double* Dp,
                          float scale, float* d, hipStream_t st) {
    if (n_pairs == 0) return hipSuccess;
    density_change_kernel<<<g1(n_pairs), 256, 0, st>>>(pairs, n_pairs, Dn, Dp, N, scale, d);
    return hipGetLastError();
}

hipError_t density_add(int N, const int32_t* pairs, int64_t n_pairs, const float* d, double scale, const double* Dp,
                       double* Dout, hipStream_t st) {
    RI_TRY(copy(Dout, Dp, (int64_t)N * N, st));
    if (n_pairs == 0) return hipSuccess;
    density_add_kernel<<<g1(n_pairs), 256, 0, st>>>(pairs, n_pairs, d, scale, Dp, N, Dout);
    return hipGetLastError();
}

hipError_t gather_density(int N, const int32_t* pairs, int64_t n_pairs, const double* D, float* d, hipStream_t st) {
    if (n_pairs == 0) return hipSuccess;
    gather_density_kernel<<<g1(n_pairs), 256, 0, st>>>(pairs, n_pairs, D, N, d);
    return hipGetLastError();
}

}  // namespace ri
