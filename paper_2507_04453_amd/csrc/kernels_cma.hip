// Ranking and the rank-weighted update of (m, sigma, C)  (paper: Algorithm 1, "each worker
// reconstructs the same population and performs one CMA-ES update").  Equations follow Hansen's
// tutorial (arXiv:1604.00772).  All reductions run in a fixed order without atomics, so replicated
// workers stay bit-identical.
#include "essa_internal.h"

namespace {

// order[#candidates that beat i] = i.  j beats i when F_j > F_i, or F_j == F_i and j < i.  NaN -> -inf.
__global__ __launch_bounds__(1024) void rank_kernel(const float* __restrict__ F, int K, int32_t* __restrict__ order) {
    __shared__ float key[1024];
    const int i = threadIdx.x;
    if (i < K) {
        const float f = F[i];
        key[i] = (f != f) ? -INFINITY : f;
    }
    __syncthreads();
    if (i < K) {
        const float mine = key[i];
        int better = 0;
        for (int j = 0; j < K; ++j) {
            const float o = key[j];
            better += (o > mine) || (o == mine && j < i);
        }
        order[better] = i;
    }
}

// z_w[l] = sum_i w[i] Z[i, l], summed for i = 0..mu-1 in fp64;  out_z = z_w,  out_dz = D * z_w.  Latency: a wave per workgroup, so
// that n in the thousands reaches many CUs, and the loads of eight rows asked for together (n = 3584, 16 rows: 5.7 -> 4.6 us).
// The two rows go where `at` says: rows of n, or the operand tiles of the product with the basis (columns past n zero there).
template <bool TILED>
__global__ void weighted_rowsum_kernel(const float* __restrict__ Z, const float* __restrict__ w, const float* __restrict__ D, int mu,
                                       int n, int ny, float* __restrict__ S) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    auto at = [&](int j) { return TILED ? essa_k::tiled_rows_at(j, l, ny + 2, n) : (size_t)j * n + l; };
    if (l >= n) {
        if (TILED && l < (n + 15) / 16 * 16) S[at(ny)] = S[at(ny + 1)] = 0.f;
        return;
    }
    const float dl = D[l];
    double acc = 0.0;
    int i = 0;
    for (; i + 8 <= mu; i += 8) {
        float z[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = Z[(size_t)(i + e) * n + l];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += (double)w[i + e] * (double)z[e];
    }
    for (; i < mu; ++i) acc += (double)w[i] * (double)Z[(size_t)i * n + l];
    const float zw = (float)acc;
    S[at(ny)] = zw;
    S[at(ny + 1)] = dl * zw;
}

__device__ __forceinline__ double block_sum_1024(double v, double* sh) {
    // fixed binary tree over 1024 slots, halves added together: the upper levels from LDS in registers, the last six across
    // the lanes; every wave does the whole of it, so there is no barrier between the levels
    sh[threadIdx.x] = v;
    __syncthreads();
    double r[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) r[k] = sh[64 * k + (threadIdx.x & 63)];
#pragma unroll
    for (int s = 8; s > 0; s >>= 1)
#pragma unroll
        for (int k = 0; k < s; ++k) r[k] += r[k + s];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) r[0] += __shfl_xor(r[0], s, 64);
    __syncthreads();
    return r[0];
}

// One workgroup.  BY rows 0..ny-1 are y_{i:lambda} = B D z_{i:lambda}, row ny is B z_w, row ny+1 is y_w = B D z_w
// (the weighted mean of the mu best y_i, taken before the product with B because that product is linear).
// The ranking leaves for the caller here, behind every launch that reads seeds or rewards: order_out may be either of them.
constexpr int HELD = 4;
__global__ __launch_bounds__(1024) void cma_vectors_kernel(essa_k::cma_consts c, const float* __restrict__ w, const float* __restrict__ BY,
                                                          float* __restrict__ m, float* __restrict__ p_sigma, float* __restrict__ p_c,
                                                          essa_cma_scalars* __restrict__ sc, const int32_t* __restrict__ order, int32_t* __restrict__ order_out) {
    __shared__ double sh[1024];
    const int n = c.n, mu = c.ny;
    const int rank = order_out ? order[min((int)threadIdx.x, c.K - 1)] : 0;
    const float sigma = sc->sigma;
    const int t = sc->t;
    const double cs = c.c_sigma, cc = c.c_c, mueff = c.mu_eff;
    const float ps_coef = (float)sqrt(cs * (2.0 - cs) * mueff);
    // Latency: of the first 4096 elements everything is asked for in front of the reduction, and what does not hang on it is done
    // there.  n = 3584: 7.9 -> 6.1 us.
    float ps0[HELD], bz[HELD], yw0[HELD], m0[HELD], pc0[HELD];
#pragma unroll
    for (int e = 0; e < HELD; ++e) {
        const int l = min((int)threadIdx.x + 1024 * e, n - 1);
        ps0[e] = p_sigma[l];
        bz[e] = BY[(size_t)mu * n + l];
        yw0[e] = BY[(size_t)(mu + 1) * n + l];
        m0[e] = m[l];
        pc0[e] = p_c[l];
    }
    const double denom = sqrt(1.0 - pow(1.0 - cs, 2.0 * (double)(t + 1)));
    if (order_out && (int)threadIdx.x < c.K) order_out[threadIdx.x] = rank;      // K <= 1024
    double part = 0.0;
#pragma unroll
    for (int e = 0; e < HELD; ++e) {
        const int l = threadIdx.x + 1024 * e;
        if (l < n) {
            const float ps = (1.0f - c.c_sigma) * ps0[e] + ps_coef * bz[e];
            p_sigma[l] = ps;
            part += (double)ps * (double)ps;
        }
    }
    for (int l = threadIdx.x + 1024 * HELD; l < n; l += 1024) {
        const float ps = (1.0f - c.c_sigma) * p_sigma[l] + ps_coef * BY[(size_t)mu * n + l];
        p_sigma[l] = ps;
        part += (double)ps * (double)ps;
    }
    const double ps_norm = sqrt(block_sum_1024(part, sh));
    const float h_sigma = (ps_norm / denom < (1.4 + 2.0 / ((double)n + 1.0)) * (double)c.chi_n) ? 1.0f : 0.0f;
    const float pc_coef = h_sigma * (float)sqrt(cc * (2.0 - cc) * mueff);
#pragma unroll
    for (int e = 0; e < HELD; ++e) {
        const int l = threadIdx.x + 1024 * e;
        if (l < n) {
            m[l] = m0[e] + sigma * yw0[e];
            p_c[l] = fmaf(pc_coef, yw0[e], (1.0f - c.c_c) * pc0[e]);
        }
    }
    for (int l = threadIdx.x + 1024 * HELD; l < n; l += 1024) {
        const float yw = BY[(size_t)(mu + 1) * n + l];
        m[l] += sigma * yw;
        p_c[l] = fmaf(pc_coef, yw, (1.0f - c.c_c) * p_c[l]);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sc->sigma = (float)((double)sigma * exp((cs / (double)c.d_sigma) * (ps_norm / (double)c.chi_n - 1.0)));
        sc->t = t + 1;
        sc->h_sigma = h_sigma;
        sc->ps_norm = (float)ps_norm;
    }
}

// C <- a C + c_1 p_c p_c^T + c_mu sum_i w_i y_i y_i^T on one 64x64 tile per workgroup, 16 rows a wave, the terms four at a time on the fp32 MFMA
// 16x16x4, operands straight from memory (they are in the L2; through LDS, a tile's terms cost as long as its bytes).  The MFMA's row dimension
// runs along C's columns, so that a lane's four results are four neighbours of a row of C.
// Every rank-one term enters as (s sqrt|coef| v)(sqrt|coef| v)^T, s the sign of its weight, so that C stays exactly
// symmetric.  A negative weight (tutorial, Eq. 46-47) is first rescaled by n / |C^-1/2 y|^2 = n / |z|^2.
// HBM binds: C read and written.  A tile above the diagonal that mirrors the one below is read alone and leaves a second time, turned over
// through LDS: three quarters of the bytes, half the sums (n = 3584, 17 terms, C from HBM: 27.2 -> 23.1 us, with the order of tiles below 19.9).
// The tiles above the diagonal come first, so that those with work to do go evenly over the CUs: row by row, with the idle ones between them, a CU could have twice
// its share, and at n = 2688 an update of 24 candidates took 41.3 us where reading all of C took 39.1; this takes 37.5 (1792: 30.7, 30.6, 29.1; 5120: 103.4, 103, 96.2; 3584: 50.3,
// 53.4, 47.6; C and B from HBM).
// 72 registers let 7 workgroups share a CU: at n = 3584 all 1596 are there at once (5 of them: 24.2 us; 8, with operands spilled: no faster).  A pair of tiles that a blob brought with
// different bits keeps them: both are read.  With no pair alike an update of 12 candidates takes 33.0 us at n = 2688 and 140 at
// 5998, 4 and 8 % more than with terms through LDS.
constexpr int CV_T = 64, CV_P = CV_T + 4;
typedef float quad __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256, 7) void cma_cov_kernel(essa_k::cma_consts c, const float* __restrict__ w, const float* __restrict__ BY,
                                                     const float* __restrict__ p_c, const essa_cma_scalars* __restrict__ sc,
                                                     const float* __restrict__ zn2, const int32_t* __restrict__ turns, float* __restrict__ C) {
    __shared__ __attribute__((aligned(16))) float turned[CV_T * CV_P];
    const int n = c.n, mu = c.ny, nt = (n + CV_T - 1) / CV_T;
    const essa_k::tile_at tile = essa_k::upper_first_tile(blockIdx.x, blockIdx.y, nt);
    if (tile.row < 0) return;
    const bool both = turns[min(tile.row, tile.col) * nt + max(tile.row, tile.col)] != 0, turn = both && tile.row < tile.col;
    if (both && tile.row > tile.col) return;
    const int i0 = tile.row * CV_T, j0 = tile.col * CV_T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int i = i0 + 16 * wave + l16, ic = min(i, n - 1);
    // the tile of C is asked for first: it comes from HBM while the rank-one terms are added up
    quad cold[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int j = j0 + 16 * b + 4 * kq;                // 16-byte accesses need 4-byte alignment only: any n
        cold[b] = quad{0.f, 0.f, 0.f, 0.f};
        if (j + 3 < n) cold[b] = *reinterpret_cast<const quad*>(C + (size_t)ic * n + j);
    }
    f32x4 acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
    int cj[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) cj[b] = min(j0 + 16 * b + l16, n - 1);
    auto add = [&](float coef, float sign, float ti, const float (&tj)[4]) {
        const float a = sign * (coef * ti);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(coef * tj[b], a, acc[b], 0, 0, 0);
    };
    constexpr int AT_ONCE = 2;                             // steps of four terms whose operands are asked for together
    for (int v0 = 0; v0 < mu; v0 += 4 * AT_ONCE) {
        float wv[AT_ONCE], zz[AT_ONCE], ti[AT_ONCE], tj[AT_ONCE][4];
#pragma unroll
        for (int s = 0; s < AT_ONCE; ++s) {
            const int v = min(v0 + 4 * s + kq, mu - 1), row = v * n;      // at most 1024 rows of 16384
            wv[s] = w[v];
            zz[s] = zn2 ? zn2[v] : 1.f;
            ti[s] = BY[row + ic];
#pragma unroll
            for (int b = 0; b < 4; ++b) tj[s][b] = BY[row + cj[b]];
        }
#pragma unroll
        for (int s = 0; s < AT_ONCE; ++s) {
            const bool live = v0 + 4 * s + kq < mu;        // past the last term: zeros, whatever its elements are
            const float weight = wv[s] < 0.f ? wv[s] * (float)n / zz[s] : wv[s], sign = weight < 0.f ? -1.f : 1.f;
            float t[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) t[b] = live ? tj[s][b] : 0.f;
            add(live ? sqrtf(c.c_mu * fabsf(weight)) : 0.f, sign, live ? ti[s] : 0.f, t);
        }
    }
    {
        float t[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) t[b] = kq == 0 ? p_c[cj[b]] : 0.f;
        add(sqrtf(c.c_1), 1.f, kq == 0 ? p_c[ic] : 0.f, t);
    }
    const float hs = sc->h_sigma;
    const float decay = 1.0f - c.c_1 - c.c_mu * c.w_sum + (1.0f - hs) * c.c_1 * c.c_c * (2.0f - c.c_c);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int j = j0 + 16 * b + 4 * kq;
        float* at = C + (size_t)ic * n + j;
        if (i < n && j + 3 < n) {
            quad cv = cold[b];
#pragma unroll
            for (int q = 0; q < 4; ++q) cv[q] = decay * cv[q] + acc[b][q];
            *reinterpret_cast<quad*>(at) = cv;
            if (turn) {
#pragma unroll
                for (int q = 0; q < 4; ++q) turned[(16 * b + 4 * kq + q) * CV_P + 16 * wave + l16] = cv[q];
            }
        } else if (i < n) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + q < n) {
                    const float cv = decay * at[q] + acc[b][q];
                    at[q] = cv;
                    if (turn) turned[(16 * b + 4 * kq + q) * CV_P + 16 * wave + l16] = cv;
                }
        }
    }
    if (!turn) return;                                     // the same for the whole workgroup
    __syncthreads();
    // row j0 + r of the turned tile: 64 columns from i0 on, all of them below n since i0 < j0
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int r = (threadIdx.x >> 4) + 16 * t, at = (threadIdx.x & 15) * 4;
        if (j0 + r < n) *reinterpret_cast<quad*>(C + (size_t)(j0 + r) * n + i0 + at) = *reinterpret_cast<const f32x4*>(turned + r * CV_P + at);
    }
}

// Bits, so that a NaN or a signed zero decides too.
__global__ __launch_bounds__(256) void cma_look_symmetric_kernel(const uint32_t* __restrict__ C, int n, int32_t* __restrict__ turns) {
    __shared__ uint32_t T[64][65];
    if (blockIdx.x < blockIdx.y) return;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    for (int e = threadIdx.x; e < 4096; e += 256)
        if (j0 + (e >> 6) < n && i0 + (e & 63) < n) T[e >> 6][e & 63] = C[(size_t)(j0 + (e >> 6)) * n + i0 + (e & 63)];
    __syncthreads();
    int differ = 0;
    for (int e = threadIdx.x; e < 4096; e += 256)
        if (i0 + (e >> 6) < n && j0 + (e & 63) < n) differ |= C[(size_t)(i0 + (e >> 6)) * n + j0 + (e & 63)] != T[e & 63][e >> 6];
    differ = __syncthreads_or(differ);
    if (threadIdx.x == 0) turns[blockIdx.y * gridDim.x + blockIdx.x] = !differ;
}

// out[j] = |Z[j, :]|^2.  One workgroup per row, fp64, fixed tree.
__global__ __launch_bounds__(1024) void row_norms2_kernel(const float* __restrict__ Z, int n, float* __restrict__ out) {
    __shared__ double sh[1024];
    const float* z = Z + (size_t)blockIdx.x * n;
    double part = 0.0;
    for (int l = threadIdx.x; l < n; l += 1024) part += (double)z[l] * (double)z[l];
    const double tot = block_sum_1024(part, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = (float)tot;
}

// Separable CMA-ES (Ros & Hansen 2008): the covariance update read on the diagonal, with its own learning rates
// (already in c.c_1, c.c_mu), and the axis lengths that the next generation samples with.
__global__ void sep_cov_kernel(essa_k::cma_consts c, const float* __restrict__ w, const float* __restrict__ Y, const float* __restrict__ p_c,
                               const essa_cma_scalars* __restrict__ sc, float* __restrict__ Cd, float* __restrict__ D) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= c.n) return;
    double acc = 0.0;
    for (int i = 0; i < c.mu; ++i) {
        const double y = (double)Y[(size_t)i * c.n + l];
        acc += (double)w[i] * y * y;
    }
    const float hs = sc->h_sigma;
    const float decay = 1.0f - c.c_1 - c.c_mu + (1.0f - hs) * c.c_1 * c.c_c * (2.0f - c.c_c);
    const float pc = p_c[l];
    const float v = decay * Cd[l] + c.c_1 * pc * pc + c.c_mu * (float)acc;
    Cd[l] = v;
    D[l] = sqrtf(fmaxf(v, 0.f));
}

// m[l] += scale * sum_j coef_j Z[j, l]; generation counter bumped by the first thread.
__global__ void mean_step_kernel(const float* __restrict__ Z, const float* __restrict__ coef, double uniform, int J, int n,
                                 essa_cma_scalars* __restrict__ sc, int use_sigma, float* __restrict__ m) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l < n) {
        double acc = 0.0;
        for (int j = 0; j < J; ++j) acc += (coef ? (double)coef[j] : uniform) * (double)Z[(size_t)j * n + l];
        const double scale = use_sigma ? (double)sc->sigma : 1.0;
        m[l] = (float)((double)m[l] + scale * acc);
    }
    if (l == 0) sc->t = sc->t + 1;
}

// ARS (Mania, Guy & Recht 2018, Algorithm 1): directions ordered by max(r+, r-), the step's coefficients for the b best.
__global__ __launch_bounds__(1024) void ars_prepare_kernel(const float* __restrict__ r, int N, int b, float alpha, int32_t* __restrict__ order,
                                                          float* __restrict__ coef) {
    __shared__ float key[1024];
    __shared__ int ord[1024];
    __shared__ double sh[1024];
    const int j = threadIdx.x;
    float rp = 0.f, rm = 0.f;
    if (j < N) {
        rp = r[2 * j];
        rm = r[2 * j + 1];
        if (rp != rp) rp = -INFINITY;
        if (rm != rm) rm = -INFINITY;
        key[j] = fmaxf(rp, rm);
    }
    __syncthreads();
    if (j < N) {
        const float mine = key[j];
        int better = 0;
        for (int o = 0; o < N; ++o) better += (key[o] > mine) || (key[o] == mine && o < j);
        ord[better] = j;
        order[better] = j;
    }
    __syncthreads();
    // thread i < b owns direction ord[i]
    double a = 0.0, d = 0.0;
    int bad = 0;
    if (j < b) {
        const int dir = ord[j];
        float p = r[2 * dir], q = r[2 * dir + 1];
        if (p != p) p = -INFINITY;
        if (q != q) q = -INFINITY;
        bad = !(isfinite(p) && isfinite(q));
        a = bad ? 0.0 : (double)p + (double)q;
        d = bad ? 0.0 : (double)p - (double)q;
    }
    const double nbad = block_sum_1024((double)bad, sh);
    const double mean = block_sum_1024(a, sh) / (2.0 * b);
    double dev = 0.0;
    if (j < b && !bad) {
        const int dir = ord[j];
        const double p = (double)r[2 * dir] - mean, q = (double)r[2 * dir + 1] - mean;
        dev = p * p + q * q;
    }
    const double var = block_sum_1024(dev, sh) / (2.0 * b);
    const double sR = sqrt(var);
    if (j < b) coef[j] = (nbad > 0.0 || !(sR > 0.0)) ? 0.f : (float)((double)alpha * d / ((double)b * sR));
}

}  // namespace

namespace essa_k {

hipError_t rank_rewards(hipStream_t st, const float* F, int K, int32_t* order) {
    hipLaunchKernelGGL(rank_kernel, dim3(1), dim3(1024), 0, st, F, K, order);
    return hipGetLastError();
}

hipError_t cma_build_rhs(hipStream_t st, const uint32_t* seeds, int32_t* order, const float* rewards, const float* w, const cma_consts& c,
                         const float* D, float* S, float* Z, bool tiled, bool want_z) {
    const int32_t* sel = rewards ? nullptr : order;
    if (tiled && c.ny <= 64) return update_rhs(st, seeds, sel, c.ny, c.mu, c.n, w, D, S, want_z ? Z : nullptr, rewards, c.K, order);
    hipError_t e = tiled ? normals_tiled(st, seeds, sel, c.ny, c.ny + 2, c.n, D, S, Z, rewards, c.K, order)
                         : normals_scaled(st, seeds, sel, c.ny, c.n, D, S, Z, rewards, c.K, order);
    if (e != hipSuccess) return e;
    if (tiled) hipLaunchKernelGGL(weighted_rowsum_kernel<true>, dim3((c.n + 63) / 64), dim3(64), 0, st, Z, w, D, c.mu, c.n, c.ny, S);
    else hipLaunchKernelGGL(weighted_rowsum_kernel<false>, dim3((c.n + 63) / 64), dim3(64), 0, st, Z, w, D, c.mu, c.n, c.ny, S);
    return hipGetLastError();
}

hipError_t cma_vectors(hipStream_t st, const cma_consts& c, const float* w, const float* BY, float* m, float* p_sigma,
                       float* p_c, essa_cma_scalars* sc, const int32_t* order, int32_t* order_out) {
    hipLaunchKernelGGL(cma_vectors_kernel, dim3(1), dim3(1024), 0, st, c, w, BY, m, p_sigma, p_c, sc, order, order_out);
    return hipGetLastError();
}

hipError_t cma_covariance(hipStream_t st, const cma_consts& c, const float* w, const float* BY, const float* p_c,
                          const essa_cma_scalars* sc, const float* zn2, const int32_t* turn, float* C) {
    const int nt = (c.n + CV_T - 1) / CV_T;
    hipLaunchKernelGGL(cma_cov_kernel, dim3(essa_k::upper_first_width(nt), nt), dim3(256), 0, st, c, w, BY, p_c, sc, zn2, turn, C);
    return hipGetLastError();
}

hipError_t cma_look_symmetric(hipStream_t st, const float* C, int n, int32_t* turn) {
    dim3 grid((n + 63) / 64, (n + 63) / 64);
    hipLaunchKernelGGL(cma_look_symmetric_kernel, grid, dim3(256), 0, st, reinterpret_cast<const uint32_t*>(C), n, turn);
    return hipGetLastError();
}

hipError_t row_norms2(hipStream_t st, const float* Z, int J, int n, float* out) {
    hipLaunchKernelGGL(row_norms2_kernel, dim3(J), dim3(1024), 0, st, Z, n, out);
    return hipGetLastError();
}

hipError_t sep_covariance(hipStream_t st, const cma_consts& c, const float* w, const float* Y, const float* p_c,
                          const essa_cma_scalars* sc, float* Cd, float* D) {
    hipLaunchKernelGGL(sep_cov_kernel, dim3((c.n + 255) / 256), dim3(256), 0, st, c, w, Y, p_c, sc, Cd, D);
    return hipGetLastError();
}

hipError_t mean_step(hipStream_t st, const float* Z, const float* coef, double uniform, int J, int n, essa_cma_scalars* sc,
                     int use_sigma, float* m) {
    hipLaunchKernelGGL(mean_step_kernel, dim3((n + 255) / 256), dim3(256), 0, st, Z, coef, uniform, J, n, sc, use_sigma, m);
    return hipGetLastError();
}

hipError_t ars_prepare(hipStream_t st, const float* rewards, int N, int b, float alpha, int32_t* order, float* coef) {
    hipLaunchKernelGGL(ars_prepare_kernel, dim3(1), dim3(1024), 0, st, rewards, N, b, alpha, order, coef);
    return hipGetLastError();
}

}  // namespace essa_k
