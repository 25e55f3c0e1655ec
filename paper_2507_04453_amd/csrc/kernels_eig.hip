// Eigendecomposition of the search covariance on the device: C = B diag(D^2) B^T
// (decomposition step of the (mu/mu_w, lambda)-CMA-ES, Hansen's tutorial arXiv:1604.00772 Sec. B.2; the paper's
// Algorithm 1 keeps (m, sigma, C) and samples through this factorisation).
//
// Method: one-sided block Jacobi in fp64.  A = C V is kept column by column (At[c][:] = column c of A), V starts as the
// identity.  Columns are grouped in blocks of 32; a sweep visits every pair of blocks once (round-robin tournament,
// nblk/2 disjoint pairs per round, nblk-1 rounds).  For a pair the 64 x 64 Gram matrix G = P^T P of its 64-column
// panel P is formed, diagonalised by a small two-sided Jacobi solver in LDS (G -> Q^T G Q), and the panel of A and of
// V is multiplied by Q.  When all columns of A are orthogonal, they are lambda_c v_c: V holds the eigenvectors and
// lambda_c = v_c^T a_c.  Every sum runs in a fixed order, so the result is the same bits on every run.
//
// A sweep is a chain of nblk - 1 rounds whose 64 x 64 solver keeps a few workgroups busy, so once V is close to the
// eigenvectors (a refresh after some generations, the last sweeps of a cold start) the iteration goes on by simultaneous
// first-order corrections instead: V <- V + V E with E from S = V^T C V and R = I - V^T V (Ogita and Aishima, "Iterative
// refinement for symmetric eigenvalue decomposition", 2018).  It converges quadratically like Jacobi's last sweeps and a
// step is four products of n x n matrices that fill the chip.  Columns keep their places and signs either way.
// Measured, n = 896: a sweep takes 3 ms, a step 0.11 to 0.13 ms (the products' fp64 MFMA time alone is 0.07); the refresh after
// 8 generations of 36 candidates 12.3 -> 0.45 ms (3 or 4 steps in place of 4 sweeps), n = 3584 with nothing to do 15 -> 3.1 ms.
#include "forward_device.h"
#include <cmath>
#include <cstring>
#include <utility>

namespace {

constexpr int EB = 32;             // columns per block
constexpr int EP = 2 * EB;         // columns per panel
constexpr int ER = 64;             // rows per LDS chunk
constexpr int EPITCH = ER + 1;     // LDS pitch (doubles)
typedef __attribute__((ext_vector_type(4))) double f64x4;

// round-robin tournament over nblk players (nblk even): the p-th pair of round `round`
__device__ __forceinline__ void pair_of(int nblk, int round, int p, int& I, int& J) {
    const int m = nblk - 1;
    if (p == 0) { I = m; J = round % m; }
    else { I = (round + p) % m; J = (round - p + m) % m; }
    if (I > J) { const int t = I; I = J; J = t; }
}

__device__ __forceinline__ int panel_col(int I, int J, int c) { return c < EB ? I * EB + c : J * EB + (c - EB); }

// 1 / sqrt(x) for a normal x: the hardware's estimate and two Newton steps y <- y (3/2 - x/2 y^2)
__device__ __forceinline__ double rsqrt_newton(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    y = y * fma(-hx * y, y, 1.5);
    y = y * fma(-hx * y, y, 1.5);
    return y;
}

// Cs[c][r] = (C[c][r] + C[r][c]) / 2 in fp64, zero beyond n; on a cold start also Vt = identity
__global__ __launch_bounds__(256) void eig_init_kernel(const float* __restrict__ C, int n, int ld, double* __restrict__ Cs, double* __restrict__ Vt,
                                                      int cold) {
    const int c = blockIdx.x;
    for (int r = threadIdx.x; r < ld; r += 256) {
        double a = 0.0;
        if (c < n && r < n) a = 0.5 * ((double)C[(size_t)c * n + r] + (double)C[(size_t)r * n + c]);
        Cs[(size_t)c * ld + r] = a;
        if (cold) Vt[(size_t)c * ld + r] = (r == c) ? 1.0 : 0.0;
    }
}

// ---- products of whole matrices -----------------------------------------------------------------------------------
// One 64 x 64 tile of X Y^T (NT: Y's row j is output column j) or X Y (NN) per workgroup of 8 waves, on the fp64 MFMA
// 16x16x4: a wave owns a 32 x 32 patch for one half of every K chunk of 32, the halves are added through LDS at the end.  The
// MFMA rate binds (64 cycles per MFMA, 128 flops per clock and CU; a chunk brings 32 KB in for 2048 of those cycles: 26 us at n = 896, where
// a CU has one tile), so everything else has to stay out of its way.  Chunks go from memory into LDS without passing through registers (a
// ds_write of the same bytes costs 5 us a product), two stages, two workgroups a CU where there are enough tiles (three or four stages and one
// workgroup: no faster at n = 896, 6 % slower at 1792).  An operand row of a chunk is 16 pieces of 16 bytes, piece p of row r at p ^ (r & 7): eight
// lanes of a fragment read meet eight different pieces of the banks' 128 bytes (rows 36 doubles apart: 16 clocks for 512 bytes in place of
// 4, as long as the MFMAs).  A piece is two k, so the MFMAs of a sub-step of 8 k take the even and the odd ones in turn, on both sides.  The
// fragments of a sub-step are read under the MFMAs of the one before; the one barrier of a chunk sits between its two sub-steps.
// Product, us (through registers, two barriers a chunk / this): n = 448 23.1 / 17.0, 896 45.9 / 33.9, 1792 264 / 214.
constexpr int MK = 32, MS = 2, MNT = 512;
constexpr uint32_t MSTAGE = 2 * 64 * MK * sizeof(double);
constexpr size_t MM_SMEM = MS * (size_t)MSTAGE;
static_assert((size_t)4 * 1024 * sizeof(double) <= MM_SMEM, "the wave halves fit");

// acc: this wave's patch; complete (both K halves) in waves 0..3 only.  Element v of acc[a][b]: row 32 wr + 16 a + 4 v + lane / 16,
// column 32 wc + 16 b + lane % 16, wr = (wave >> 1) & 1, wc = wave & 1.
template <bool NN>
__device__ __forceinline__ void tile_product(const double* __restrict__ X, const double* __restrict__ Y, int ld, int i0, int j0, double* lds, f64x4 (&acc)[2][2]) {
    typedef __attribute__((ext_vector_type(2))) double f64x2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kq = lane >> 4;
    const int wr = (wave >> 1) & 1, wc = wave & 1, kh = wave >> 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)lds;
    unsigned char* smem = reinterpret_cast<unsigned char*>(lds);
    // A wave moves four kilobytes of a chunk: 4 rows x 256 bytes of X, twice, and as much of Y (NN: 2 rows x 512 bytes, twice)
    const int chunks = ld / MK, last = chunks - 1;         // at least MS, as many as are asked for up front: ld is a multiple of 64
    const i32x4 xres = buffer_words(X + (size_t)i0 * ld);
    uint32_t off[2], yoff[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int row = (wave * 2 + e) * 4 + (lane >> 4), at = (lane & 15) ^ (row & 7);
        off[e] = (uint32_t)row * (uint32_t)ld * 8u + at * 16;
        yoff[e] = NN ? (uint32_t)((wave * 2 + e) * 2 + (lane >> 5)) * (uint32_t)ld * 8u + (lane & 31) * 16 : off[e];
    }
    const i32x4 yres0 = buffer_words(Y + (size_t)j0 * ld);
    auto fetch = [&](int chunk, uint32_t stage) {
        const int c = min(chunk, last);
        const i32x4 yres = NN ? buffer_words(Y + (size_t)c * MK * ld + j0) : yres0;
#pragma unroll
        for (int e = 0; e < 2; ++e) load_lds16(lds0 + stage + (wave * 2 + e) * 1024, off[e], xres, (uint32_t)c * (MK * 8u));
#pragma unroll
        for (int e = 0; e < 2; ++e) load_lds16(lds0 + stage + 16384 + (wave * 2 + e) * 1024, yoff[e], yres, NN ? 0u : (uint32_t)c * (MK * 8u));
    };
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = (f64x4){0.0, 0.0, 0.0, 0.0};
    // lane's pieces of a sub-step of 8 k: k = 2 kq, 2 kq + 1 of it (both operands alike)
    uint32_t xat[2], yat[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint32_t at = (uint32_t)((8 * kh + 4 * u + kq) ^ (l16 & 7)) * 16;
        xat[u] = (32 * wr + l16) * 256 + at;
        yat[u] = 16384 + (NN ? (16 * kh + 8 * u + 2 * kq) * 512 + (32 * wc + l16) * 8 : (32 * wc + l16) * 256 + at);
    }
    f64x2 fx[2][2], fy[2][2];
    auto read = [&](uint32_t stage, int u) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            fx[u][a] = *reinterpret_cast<const f64x2*>(smem + stage + xat[u] + a * 4096);
            if (NN) {
                fy[u][a][0] = *reinterpret_cast<const double*>(smem + stage + yat[u] + a * 128);
                fy[u][a][1] = *reinterpret_cast<const double*>(smem + stage + yat[u] + a * 128 + 512);
            } else fy[u][a] = *reinterpret_cast<const f64x2*>(smem + stage + yat[u] + a * 4096);
        }
    };
    auto multiply = [&](int u, int e) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fx[u][a][e], fy[u][b][e], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    uint32_t cur = 0, nxt = MSTAGE;
#pragma unroll
    for (int i = 0; i < MS; ++i) fetch(i, i * MSTAGE);
    wait_loads_and_meet<(MS - 1) * 4>();
    read(0, 0);
    for (int i = 0; i < chunks; ++i) {
        read(cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, 0);
        multiply(0, 1);
        wait_loads_and_meet<(MS - 2) * 4>();               // chunk i + 1 is there, and everybody has read chunk i
        __builtin_amdgcn_sched_barrier(0);
        read(nxt, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1, 0);
        fetch(i + MS, cur);                                // past the end the last chunk again, for nobody
        __builtin_amdgcn_sched_barrier(0);
        multiply(1, 1);
        cur = nxt;
        nxt = nxt == (MS - 1) * MSTAGE ? 0 : nxt + MSTAGE;
    }
    wait_loads_and_meet<0>();                              // what was asked for past the end has landed
    // the second K halves join the first
    double* half = lds + (size_t)(wave & 3) * 1024 + lane;
    if (kh == 1) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) half[((a * 2 + b) * 4 + v) * 64] = acc[a][b][v];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[a][b][v] += half[((a * 2 + b) * 4 + v) * 64];
    }
}

template <class F>
__device__ __forceinline__ void each_element(const f64x4 (&acc)[2][2], F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    if (wave >= 4) return;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) f(32 * (wave >> 1) + 16 * a + 4 * v + kq, 32 * (wave & 1) + 16 * b + l16, acc[a][b][v]);
}

// Out = Vt Cs: row c of Out = column c of C V (C symmetric, so its rows serve as columns)
__global__ __launch_bounds__(MNT) void eig_matmul_kernel(const double* __restrict__ Vt, const double* __restrict__ Cs, int ld, double* __restrict__ Out) {
    extern __shared__ __attribute__((aligned(16))) double dyn_mm[];
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    f64x4 acc[2][2];
    tile_product<false>(Vt, Cs, ld, i0, j0, dyn_mm, acc);
    each_element(acc, [&](int r, int c, double v) { Out[(size_t)(i0 + r) * ld + j0 + c] = v; });
}

// The tile pair (I <= J) that a workgroup of a triangular grid takes
__device__ __forceinline__ void tri_pair(int t, int& I, int& J) {
    J = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((J + 1) * (J + 2) / 2 <= t) ++J;
    while (J * (J + 1) / 2 > t) --J;
    I = t - J * (J + 1) / 2;
}

// S = V^T C V (blockIdx.y = 0) into the tiles (I, J) of M with I <= J, R = I - V^T V (blockIdx.y = 1) into the tiles (J, I)
// below, its diagonal tiles into Rd; the diagonals of both also as vectors
__global__ __launch_bounds__(MNT) void eig_residual_kernel(const double* __restrict__ Vt, const double* __restrict__ At, int ld, double* __restrict__ M,
                                                           double* __restrict__ Rd, double* __restrict__ diagS, double* __restrict__ diagR) {
    extern __shared__ __attribute__((aligned(16))) double dyn_mm[];
    int I, J;
    tri_pair(blockIdx.x, I, J);
    f64x4 acc[2][2];
    if (blockIdx.y == 0) {
        tile_product<false>(Vt, At, ld, I * 64, J * 64, dyn_mm, acc);
        each_element(acc, [&](int r, int c, double v) {
            M[(size_t)(I * 64 + r) * ld + J * 64 + c] = v;
            if (I == J && r == c) diagS[I * 64 + r] = v;
        });
    } else {
        tile_product<false>(Vt, Vt, ld, J * 64, I * 64, dyn_mm, acc);
        each_element(acc, [&](int r, int c, double v) {
            v = (I == J && r == c ? 1.0 : 0.0) - v;
            if (I == J) Rd[((size_t)I * 64 + r) * 64 + c] = v;
            else M[(size_t)(J * 64 + r) * ld + I * 64 + c] = v;
            if (I == J && r == c) diagR[I * 64 + r] = v;
        });
    }
}

// E from S and R, in their place and transposed (row c of M becomes column c of E).  With lambda_i = S_ii / (1 - R_ii) and
// s = S_ij + R_ij (lambda_i + lambda_j) / 2, the off-diagonal element seen from orthonormal columns:
//   E_ij = R_ij / 2 + t,  E_ji = R_ij / 2 - t,  t = s / (lambda_j - lambda_i)
// and t = 0 for pairs whose cosine |s| (lambda_i + lambda_j) / (lambda_i lambda_j) (the measure of the sweeps: columns of C V are
// compared) is already below `leave`, and for pairs too close together for a first-order angle (|t| > STRONG): these are
// turned exactly, one partner per column and step (eig_pair_kernel).  The largest cosine goes to offmax; per row and tile
// the sum of |E| goes to part and the strongest such pair to the st_ arrays (all [tile][row]).
constexpr double STRONG = 0.25;
// Latency, three fp64 divisions per pair: 1024 threads a tile take 12 us at n = 896 where 256 took 27.
constexpr int EC_NT = 1024;
__global__ __launch_bounds__(EC_NT) void eig_correction_kernel(double* __restrict__ M, const double* __restrict__ Rd, const double* __restrict__ diagS,
                                                             const double* __restrict__ diagR, int ld, int n, int with_t, double leave,
                                                             double* __restrict__ part, double* __restrict__ st_s, float* __restrict__ st_t,
                                                             int* __restrict__ st_j, unsigned* __restrict__ offmax) {
    __shared__ double Rt[64][65], Ab[64][65], lam[2][64];
    __shared__ unsigned mx;
    int I, J;
    tri_pair(blockIdx.x, I, J);
    const int tid = threadIdx.x;
    if (tid == 0) mx = 0u;
    if (tid < 128) {
        const int k = (tid < 64 ? I : J) * 64 + (tid & 63);
        lam[tid >> 6][tid & 63] = diagS[k] / (1.0 - diagR[k]);
    }
    for (int e = tid; e < 4096; e += EC_NT) {
        const int r = e >> 6, c = e & 63;                  // R_ji, j = row: Rt[i][j]
        Rt[c][r] = I == J ? Rd[((size_t)I * 64 + r) * 64 + c] : M[(size_t)(J * 64 + r) * ld + I * 64 + c];
    }
    __syncthreads();
    unsigned best = 0u;
    for (int e = tid; e < 4096; e += EC_NT) {
        const int a = e >> 6, b = e & 63;
        const bool live = I * 64 + a < n && J * 64 + b < n;
        double r = live ? Rt[a][b] : 0.0, t = 0.0;
        if (with_t && live && (I < J || a < b)) {
            const double la = lam[0][a], lb = lam[1][b], s = M[(size_t)(I * 64 + a) * ld + J * 64 + b] + 0.5 * r * (la + lb);
            const float cosine = (float)(fabs(s) * (la + lb) / (la * lb));
            best = max(best, __float_as_uint(cosine) & 0x7fffffffu);      // a NaN's bits are larger than any number's
            if (!(cosine <= (float)leave)) t = s / (lb - la);
        }
        Ab[a][b] = t;
    }
    atomicMax(&mx, best);
    __syncthreads();
    auto weak = [](double t) { return fabs(t) > STRONG ? 0.0 : t; };
    // The share of this tile in a column's sum and its strongest pair: 8 lanes per column, 8 elements each, the lanes joined in ascending
    // order (threads 0 .. 511 the columns of tile I, the others those of tile J).
    double sum = 0.0, top_s = 0.0;
    float top_t = 0.f;
    int top_j = -1;
    auto look = [&](double r, double t, int i, int j, int col) {       // pair (i of tile I, j of tile J) seen from the other column
        sum += 0.5 * fabs(r) + fabs(weak(t));
        if (fabs(t) > STRONG && fmin(fabs(t), 1e30) > (double)top_t) {
            top_t = (float)fmin(fabs(t), 1e30);
            top_j = col;
            top_s = M[(size_t)(I * 64 + i) * ld + J * 64 + j] + 0.5 * r * (lam[0][i] + lam[1][j]);
        }
    };
    const int seg = (tid & 7) * 8, own = (tid >> 3) & 63;
    if (tid < 512) {
        for (int b = seg; b < seg + 8; ++b) look(Rt[own][b], Ab[own][b], own, b, J * 64 + b);
        if (I == J)
            for (int a = seg; a < seg + 8; ++a) look(0.0, Ab[a][own], a, own, I * 64 + a);
    } else if (I < J) {
        for (int a = seg; a < seg + 8; ++a) look(Rt[a][own], Ab[a][own], a, own, I * 64 + a);
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) {                // a lane takes over what lies behind its own; the first wins a tie
        const double s2 = __shfl_down(sum, off, 8), ts = __shfl_down(top_s, off, 8);
        const float tt = __shfl_down(top_t, off, 8);
        const int tj = __shfl_down(top_j, off, 8);
        sum += s2;
        if (tt > top_t) {
            top_t = tt;
            top_s = ts;
            top_j = tj;
        }
    }
    if (seg == 0 && (tid < 512 || I < J)) {
        const size_t at = tid < 512 ? (size_t)J * ld + I * 64 + own : (size_t)I * ld + J * 64 + own;
        part[at] = sum;
        st_s[at] = top_s;
        st_t[at] = top_t;
        st_j[at] = top_j;
    }
    __syncthreads();                                       // S is read above
    if (I < J) {
        // Ab: t of (i, j); E_ji lies in row i of the transposed matrix, E_ij in row j
        for (int e = tid; e < 4096; e += EC_NT) {
            const int a = e >> 6, b = e & 63;
            M[(size_t)(I * 64 + a) * ld + J * 64 + b] = 0.5 * Rt[a][b] - weak(Ab[a][b]);
            M[(size_t)(J * 64 + a) * ld + I * 64 + b] = 0.5 * Rt[b][a] + weak(Ab[b][a]);
        }
    } else {
        for (int e = tid; e < 4096; e += EC_NT) {
            const int a = e >> 6, b = e & 63;
            M[(size_t)(I * 64 + a) * ld + I * 64 + b] = 0.5 * Rt[a][b] + (a > b ? weak(Ab[b][a]) : -weak(Ab[a][b]));
        }
    }
    if (tid == 0) atomicMax(offmax, mx);
}

// What the host decides by: the largest cosine, the largest row sum of |E| (a bound on |E|_2), the range of the eigenvalues, the
// number of columns with a strong partner; lambda itself for the case that this was the last step, and each column's
// strongest partner.  One workgroup; offmax is left cleared for the next step.
// A step is taken while the corrections are small: |E|_2 <= max row sum <= 1/2 keeps |I - V^T V| <= 1/3 afterwards, which the
// R / 2 part of the next steps removes quadratically whatever happens to the angles.  Eigenvalues a millionth of the
// largest and below are left to the sweeps, whose column cosines resolve them better than S does.
constexpr float STEP_MAX = 0.5f, LAST_STEP = 1e-5f, NO_STEP = 1e-9f, RANGE = 1e-6f;
struct eig_stats { float off, esum, lmin, lmax; int strong, fits, go; };    // fits: a step may be taken; go: and there is something to correct
__global__ __launch_bounds__(1024) void eig_stats_kernel(const double* __restrict__ part, const double* __restrict__ st_s, const float* __restrict__ st_t,
                                                         const int* __restrict__ st_j, const double* __restrict__ diagS, const double* __restrict__ diagR,
                                                         int ld, int n, unsigned* __restrict__ offmax, double* __restrict__ lam,
                                                         double* __restrict__ pair_s, int* __restrict__ partner, eig_stats* __restrict__ out,
                                                         eig_stats* __restrict__ out_host) {
    __shared__ float es[1024], lo[1024], hi[1024];
    __shared__ int strong;
    const int tid = threadIdx.x, nt = ld / 64;
    if (tid == 0) strong = 0;
    __syncthreads();
    float e = 0.f, l = INFINITY, h = -INFINITY;
    for (int i = tid; i < n; i += 1024) {
        double s = 0.0;
        float top = 0.f;
        int at = -1;
        for (int t = 0; t < nt; ++t) {
            s += part[(size_t)t * ld + i];
            const float x = st_t[(size_t)t * ld + i];
            if (x > top) { top = x; at = t; }
        }
        partner[i] = at >= 0 ? st_j[(size_t)at * ld + i] : -1;
        if (at >= 0) {
            pair_s[i] = st_s[(size_t)at * ld + i];
            atomicAdd(&strong, 1);
        }
        const double v = diagS[i] / (1.0 - diagR[i]);
        lam[i] = v;
        e = (float)s <= e ? e : (float)s;                  // a NaN wins and stays
        if (e != e) e = INFINITY;
        l = (float)v >= l ? l : (float)v;
        h = (float)v <= h ? h : (float)v;
    }
    es[tid] = e; lo[tid] = l; hi[tid] = h;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if (tid < st) {
            es[tid] = fmaxf(es[tid], es[tid + st]);
            lo[tid] = fminf(lo[tid], lo[tid + st]);
            hi[tid] = fmaxf(hi[tid], hi[tid + st]);
        }
        __syncthreads();
    }
    if (tid == 0) {
        eig_stats r;
        r.off = __uint_as_float(*offmax);
        r.esum = es[0]; r.lmin = lo[0]; r.lmax = hi[0];
        r.strong = strong;
        r.fits = r.esum <= STEP_MAX && r.lmin > RANGE * r.lmax && r.lmax < INFINITY;
        r.go = r.fits && (r.esum > NO_STEP || strong > 0);
        *out = r;
        if (out_host) *out_host = r;
        *offmax = 0u;
    }
}

// The exact turn J of the columns that are each other's strongest partner, put behind the correction: I + E becomes (I + E) J.
// One workgroup per column; rows of M are columns of E.
__global__ __launch_bounds__(256) void eig_pair_kernel(double* __restrict__ M, const double* __restrict__ pair_s, const double* __restrict__ lam,
                                                       const int* __restrict__ partner, int ld, const eig_stats* __restrict__ when) {
    const int i = blockIdx.x, j = partner[i];
    if (!when->go || j <= i || partner[j] != i) return;
    const double a = lam[j] - lam[i], b = 2.0 * pair_s[i];
    const double t = (a >= 0.0 ? b : -b) / (fabs(a) + sqrt(a * a + b * b));
    const double c = 1.0 / sqrt(1.0 + t * t), s = t * c;
    for (int k = threadIdx.x; k < ld; k += 256) {
        const double ei = k == i ? 1.0 : 0.0, ej = k == j ? 1.0 : 0.0;
        const double x = M[(size_t)i * ld + k] + ei, y = M[(size_t)j * ld + k] + ej;
        M[(size_t)i * ld + k] = (c * x - s * y) - ei;
        M[(size_t)j * ld + k] = (s * x + c * y) - ej;
    }
}

// Vn = Vt + E^T Vt (rows are columns of V; Et = E transposed as the correction kernel left it); when: null, or whether to
__global__ __launch_bounds__(MNT) void eig_apply_kernel(const double* __restrict__ Et, const double* __restrict__ Vt, int ld, double* __restrict__ Vn,
                                                        const eig_stats* __restrict__ when) {
    extern __shared__ __attribute__((aligned(16))) double dyn_mm[];
    if (when && !when->go) return;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    f64x4 acc[2][2];
    tile_product<true>(Et, Vt, ld, i0, j0, dyn_mm, acc);
    each_element(acc, [&](int r, int c, double v) {
        const size_t at = (size_t)(i0 + r) * ld + j0 + c;
        Vn[at] = Vt[at] + v;
    });
}

// Gram matrix of a panel over one slice of the rows: Gpart[pair][slice][a][b] = sum_r P[r][a] P[r][b]
__global__ __launch_bounds__(256) void eig_gram_kernel(const double* __restrict__ At, int ld, int n, int nblk, int round, int chunks_per_slice,
                                                      double* __restrict__ Gpart) {
    __shared__ double T[EP][EPITCH];
    const int pair = blockIdx.x, slice = blockIdx.y, S = gridDim.y, tid = threadIdx.x;
    int I, J;
    pair_of(nblk, round, pair, I, J);
    // fp64 MFMA 16x16x4: wave w owns rows 16w .. 16w+15 of G (all four 16-column blocks).  Operand element (i, k) and (k, j)
    // sit in lane i + 16 k resp. j + 16 k; with A[i][k] = P[r0 + k][16w + i] and B[k][j] = P[r0 + k][16jb + j] both operands
    // are T[column][row] read at [16 x + lane % 16][rr + lane / 16].  Accumulator element v of a lane is G[16w + 4 v +
    // lane / 16][16jb + lane % 16] (the fp64 form's own order: not that of the fp32 16x16x4).  (The vector and the matrix unit have the same fp64 rate on this chip; the MFMA needs a sixth of
    // the LDS reads per product.)
    const int wave = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    f64x4 acc[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) acc[jb] = (f64x4){0.0, 0.0, 0.0, 0.0};
    for (int ch = 0; ch < chunks_per_slice; ++ch) {
        const int r0 = (slice * chunks_per_slice + ch) * ER;
        if (r0 >= n) break;                                    // uniform for the workgroup
        for (int idx = tid; idx < EP * ER; idx += 256) {
            const int c = idx >> 6, rr = idx & 63, row = r0 + rr;
            T[c][rr] = row < n ? At[(size_t)panel_col(I, J, c) * ld + row] : 0.0;
        }
        __syncthreads();
#pragma unroll 4
        for (int rr = 0; rr < ER; rr += 4) {
            double f[4];
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) f[jb] = T[16 * jb + l16][rr + kq];
            const double a = T[16 * wave + l16][rr + kq];      // (one of the four above; read again rather than selected)
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) acc[jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, f[jb], acc[jb], 0, 0, 0);
        }
        __syncthreads();
    }
    double* out = Gpart + ((size_t)pair * S + slice) * EP * EP;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int v = 0; v < 4; ++v) out[(16 * wave + 4 * v + kq) * EP + 16 * jb + l16] = acc[jb][v];
}

// Diagonalises the 64 x 64 Gram matrix of every panel: cyclic two-sided Jacobi in LDS, 32 disjoint rotations per step
// (round-robin over the 64 indices), 63 steps per sweep.  With the 32 rotations J_k of a step known, the 2 x 2 block of G
// at (rows of pair k, columns of pair l) becomes J_k^T block J_l independently of all other blocks: one thread per block
// (1024 threads), two barriers per step.  Q (the product of the rotations) goes to Qout; the largest
// |G[a][b]| / sqrt(G[a][a] G[b][b]) met before rotating goes to offmax (as the bits of a non-negative float, so that an
// integer maximum orders them).
constexpr int SMALL_NT = 1024;
__global__ __launch_bounds__(SMALL_NT) void eig_small_kernel(const double* __restrict__ Gpart, int S, double* __restrict__ Qout,
                                                            unsigned* __restrict__ offmax, unsigned* __restrict__ rotated, int max_inner,
                                                            double inner_tol) {
    extern __shared__ __attribute__((aligned(16))) double dyn_small[];       // two 64 x 65 matrices: more than the static limit
    double (*G)[EPITCH] = reinterpret_cast<double (*)[EPITCH]>(dyn_small);
    double (*Q)[EPITCH] = reinterpret_cast<double (*)[EPITCH]>(dyn_small + EP * EPITCH);
    __shared__ double cs[EB][2];
    __shared__ int pq[EB][2];
    __shared__ double red[SMALL_NT / 64];
    __shared__ int again, did;                                 // did: some rotation of this panel was not the identity
    const int pair = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) did = 0;
    const double* src = Gpart + (size_t)pair * S * EP * EP;
    for (int idx = tid; idx < EP * EP; idx += SMALL_NT) {
        double g = src[idx];
        for (int s = 1; s < S; ++s) g += src[(size_t)s * EP * EP + idx];
        G[idx >> 6][idx & 63] = g;
        Q[idx >> 6][idx & 63] = (idx >> 6) == (idx & 63) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < max_inner; ++sweep) {
        // how far from diagonal (relative); the first measure is the panel's contribution to the outer test
        double m = 0.0;
        for (int idx = tid; idx < EP * EP; idx += SMALL_NT) {
            const int a = idx >> 6, b = idx & 63;
            if (a < b) {
                const double d = G[a][a] * G[b][b];
                if (d > 0.0) m = fmax(m, fabs(G[a][b]) / sqrt(d));
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
        if (lane == 0) red[wave] = m;
        __syncthreads();
        if (tid == 0) {
            double t = red[0];
            for (int w = 1; w < SMALL_NT / 64; ++w) t = fmax(t, red[w]);
            if (sweep == 0) atomicMax(offmax, __float_as_uint((float)t));
            again = t > inner_tol;
        }
        __syncthreads();
        if (!again) break;
        for (int step = 0; step < EP - 1; ++step) {
            if (tid < EB) {
                int p, q;
                pair_of(EP, step, tid, p, q);
                const double gpq = G[p][q], gpp = G[p][p], gqq = G[q][q];
                double c = 1.0, s = 0.0;
                if (fabs(gpq) > 1e-300 && gpq * gpq > (inner_tol * inner_tol) * fabs(gpp * gqq)) {
                    // t = tan(phi) = sign(a) b / (|a| + sqrt(a^2 + b^2)) with a = gqq - gpp, b = 2 gpq (the tutorial form with
                    // theta = a / b, multiplied through by |b|), c = 1 / sqrt(1 + t^2), s = t c.  These 32 threads are the
                    // critical path of a step, so the square roots and the division are the hardware's reciprocal (square
                    // root) estimates with Newton steps: c to full precision (c^2 + s^2 = c^2 (1 + t^2) = 1 to rounding whatever
                    // t is, which is what keeps Q orthogonal); an error in t only moves the angle by its relative size.
                    const double a = gqq - gpp, b = 2.0 * gpq, h2 = a * a + b * b;
                    double t;
                    if (h2 > 1e-280 && h2 < 1e280) {
                        const double den = fabs(a) + h2 * rsqrt_newton(h2);
                        double r = __builtin_amdgcn_rcp(den);
                        r = fma(fma(-den, r, 1.0), r, r);
                        r = fma(fma(-den, r, 1.0), r, r);
                        t = (a >= 0.0 ? b : -b) * r;
                    } else {
                        const double theta = a / b;
                        t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                    }
                    c = rsqrt_newton(fma(t, t, 1.0));
                    s = t * c;
                    if (s != 0.0) did = 1;
                }
                pq[tid][0] = p; pq[tid][1] = q;
                cs[tid][0] = c; cs[tid][1] = s;
            }
            __syncthreads();
            {
                // block (k, l) of G: rows (p_k, q_k), columns (p_l, q_l)
                const int k = tid >> 5, l = tid & 31;
                const int pk = pq[k][0], qk = pq[k][1], pl = pq[l][0], ql = pq[l][1];
                const double ck = cs[k][0], sk = cs[k][1], cl = cs[l][0], sl = cs[l][1];
                const double a = G[pk][pl], b = G[pk][ql], c = G[qk][pl], d = G[qk][ql];
                const double a1 = cl * a - sl * b, b1 = sl * a + cl * b, c1 = cl * c - sl * d, d1 = sl * c + cl * d;
                G[pk][pl] = ck * a1 - sk * c1;
                G[qk][pl] = sk * a1 + ck * c1;
                G[pk][ql] = ck * b1 - sk * d1;
                G[qk][ql] = sk * b1 + ck * d1;
                // columns (p_l, q_l) of Q, rows 2k and 2k + 1
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * k + e;
                    const double qp = Q[i][pl], qq = Q[i][ql];
                    Q[i][pl] = cl * qp - sl * qq;
                    Q[i][ql] = sl * qp + cl * qq;
                }
            }
            __syncthreads();
        }
    }
    // a panel that needed no rotation has Q = I exactly: the update kernel skips it (no traffic at all for its columns)
    if (tid == 0) rotated[pair] = (unsigned)did;
    if (!did) return;                                          // uniform: did was last written before the last barrier
    double* out = Qout + (size_t)pair * EP * EP;
    for (int idx = tid; idx < EP * EP; idx += SMALL_NT) out[idx] = Q[idx >> 6][idx & 63];
}

// panel <- panel * Q for A (blockIdx.z = 0) and V (blockIdx.z = 1); a workgroup loads Q once and takes UCH chunks of 64 rows
constexpr int UCH = 4;
__global__ __launch_bounds__(256) void eig_update_kernel(double* __restrict__ At, double* __restrict__ Vt, int ld, int n, int nblk, int round,
                                                        const double* __restrict__ Qin, const unsigned* __restrict__ rotated) {
    extern __shared__ __attribute__((aligned(16))) double dyn_upd[];
    double (*T)[EPITCH] = reinterpret_cast<double (*)[EPITCH]>(dyn_upd);
    double (*Qs)[EPITCH] = reinterpret_cast<double (*)[EPITCH]>(dyn_upd + EP * EPITCH);
    const int pair = blockIdx.x, tid = threadIdx.x;
    if (rotated[pair] == 0) return;                            // Q = I: nothing to do (uniform for the workgroup)
    double* M = blockIdx.z == 0 ? At : Vt;
    int I, J;
    pair_of(nblk, round, pair, I, J);
    const double* qsrc = Qin + (size_t)pair * EP * EP;
    for (int idx = tid; idx < EP * EP; idx += 256) Qs[idx >> 6][idx & 63] = qsrc[idx];      // Qs[c][c'] = Q[c][c']
    // fp64 MFMA 16x16x4: wave w owns rows 16w .. 16w+15 of the chunk for all 64 new columns.  out[c'][row] = sum_c Q[c][c']
    // T[c][row]: A[i][k] = Q[kk + k][16ib + i], B[k][j] = T[kk + k][16w + j]; accumulator element v of a lane is new column
    // 16ib + 4 v + lane / 16 at row 16w + lane % 16.
    const int wave = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    for (int ch = 0; ch < UCH; ++ch) {
        const int r0 = (blockIdx.y * UCH + ch) * ER;
        if (r0 >= n) break;                                    // uniform for the workgroup
        __syncthreads();                                       // Q is in place / the previous chunk's tile has been read
        for (int idx = tid; idx < EP * ER; idx += 256) {
            const int c = idx >> 6, rr = idx & 63, row = r0 + rr;
            T[c][rr] = row < n ? M[(size_t)panel_col(I, J, c) * ld + row] : 0.0;
        }
        __syncthreads();
        f64x4 acc[4];
#pragma unroll
        for (int ib = 0; ib < 4; ++ib) acc[ib] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int kk = 0; kk < EP; kk += 4) {
            const double b = T[kk + kq][16 * wave + l16];
#pragma unroll
            for (int ib = 0; ib < 4; ++ib) acc[ib] = __builtin_amdgcn_mfma_f64_16x16x4f64(Qs[kk + kq][16 * ib + l16], b, acc[ib], 0, 0, 0);
        }
        const int row = r0 + 16 * wave + l16;
        if (row < n) {
#pragma unroll
            for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                for (int v = 0; v < 4; ++v) M[(size_t)panel_col(I, J, 16 * ib + 4 * v + kq) * ld + row] = acc[ib][v];
        }
    }
}

// lambda_c = v_c^T a_c (A = C V)
__global__ __launch_bounds__(256) void eig_lambda_kernel(const double* __restrict__ At, const double* __restrict__ Vt, int ld, int n, double* __restrict__ lam) {
    __shared__ double red[256];
    const int c = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    for (int r = tid; r < n; r += 256) s = fma(Vt[(size_t)c * ld + r], At[(size_t)c * ld + r], s);
    red[tid] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) lam[c] = red[0];
}

// B[r][c] = V[r][c] (through LDS: V is kept by columns, B by rows), D_c = sqrt(max(lambda_c, 0))
__global__ __launch_bounds__(256) void eig_finish_kernel(const double* __restrict__ Vt, const double* __restrict__ lam, int ld, int n,
                                                        float* __restrict__ B, float* __restrict__ D) {
    __shared__ float T[64][65];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64, tid = threadIdx.x;
    for (int e = tid; e < 4096; e += 256) T[e >> 6][e & 63] = (float)Vt[(size_t)(c0 + (e >> 6)) * ld + r0 + (e & 63)];
    __syncthreads();
    for (int e = tid; e < 4096; e += 256) {
        const int r = r0 + (e >> 6), c = c0 + (e & 63);
        if (r < n && c < n) B[(size_t)r * n + c] = T[e & 63][e >> 6];
    }
    if (blockIdx.y == 0 && tid < 64 && c0 + tid < n) D[c0 + tid] = (float)sqrt(fmax(lam[c0 + tid], 0.0));
}

__global__ void eig_clear_kernel(unsigned* flag) { *flag = 0u; }

}  // namespace

namespace essa_k {

size_t eig_basis_bytes(int n) {
    const size_t npad = (size_t)(n + EP - 1) / EP * EP;
    return npad * npad * sizeof(double);
}

// the matrices and vectors that the correction steps need on top of the sweeps' own
static size_t eig_refine_doubles(int n) {
    const size_t npad = (size_t)(n + EP - 1) / EP * EP;
    return npad * npad + npad * 64 + 3 * npad * (npad / 64) + 2 * npad;
}

size_t eig_workspace_bytes(int n, bool refine) {
    const size_t npad = (size_t)(n + EP - 1) / EP * EP, ld = npad, npairs = npad / EP;
    const size_t S = 8;
    return 2 * npad * ld * sizeof(double) + npairs * S * EP * EP * sizeof(double) + npairs * EP * EP * sizeof(double) + 3 * npad * sizeof(double) + 256 +
           npairs * sizeof(unsigned) + 256 + (refine ? eig_refine_doubles(n) * sizeof(double) : 0);
}

hipError_t eig_refresh(hipStream_t st, const float* C, int n, void* ws, bool refine, double* Vt, int warm, int max_sweeps, float tol, float* B, float* D,
                       void* host, hipEvent_t told, int* sweeps_done, float* off_final) {
    const int npad = (n + EP - 1) / EP * EP, ld = npad, nblk = npad / EB, npairs = nblk / 2, nt = npad / 64, ntri = nt * (nt + 1) / 2;
    const int chunks = (n + ER - 1) / ER;
    const int S = 8, chunks_per_slice = (chunks + S - 1) / S;
    double* At = (double*)ws;
    double* Cs = At + (size_t)npad * ld;
    double* Gpart = Cs + (size_t)npad * ld;
    double* Q = Gpart + (size_t)npairs * S * EP * EP;
    double* lam = Q + (size_t)npairs * EP * EP;
    double* diagS = lam + npad;
    double* diagR = diagS + npad;
    unsigned* flag = (unsigned*)(diagR + npad);
    eig_stats* stats_dev = (eig_stats*)(flag + 16);
    unsigned* rotated = flag + 64;                             // [npairs], behind the 256 bytes of the flag
    double* M = (double*)(((uintptr_t)(rotated + npairs) + 255) & ~(uintptr_t)255);     // correction steps only, as what follows
    double* Rd = M + (size_t)npad * ld;
    double* part = Rd + (size_t)npad * 64;
    double* st_s = part + (size_t)npad * nt;
    float* st_t = (float*)(st_s + (size_t)npad * nt);
    int* st_j = (int*)(st_t + (size_t)npad * nt);
    double* pair_s = (double*)(st_j + (size_t)npad * nt);
    int* partner = (int*)(pair_s + npad);
    constexpr size_t two_mats = (size_t)2 * EP * EPITCH * sizeof(double);
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipSuccess;
        auto allow = [&](const void* k, size_t bytes) {
            if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        };
        allow(reinterpret_cast<const void*>(eig_small_kernel), two_mats);
        allow(reinterpret_cast<const void*>(eig_update_kernel), two_mats);
        allow(reinterpret_cast<const void*>(eig_matmul_kernel), MM_SMEM);
        allow(reinterpret_cast<const void*>(eig_residual_kernel), MM_SMEM);
        allow(reinterpret_cast<const void*>(eig_apply_kernel), MM_SMEM);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
    // V and A = C V; a correction step writes the new V where A was, and the two buffers change places
    double *V = Vt, *A = At;
    const dim3 tiles(nt, nt);
    auto multiply = [&]() { hipLaunchKernelGGL(eig_matmul_kernel, tiles, dim3(MNT), MM_SMEM, st, V, Cs, ld, A); };
    // with the basis of the last refresh (kept in fp64) the columns of A start out nearly orthogonal; on a cold start V = I
    hipLaunchKernelGGL(eig_init_kernel, dim3(npad), dim3(256), 0, st, C, n, ld, Cs, Vt, warm ? 0 : 1);
    hipLaunchKernelGGL(eig_clear_kernel, dim3(1), dim3(1), 0, st, flag);
    multiply();
    // a pair of columns whose cosine is a hundredth of the caller's tolerance or less is left alone (and a panel with only such
    // pairs costs no update): the outer test cannot tell the difference, and an unchanged C costs one pass of Gram matrices
    const double inner_tol = tol > 1e-13f ? 0.01 * (double)tol : 1e-15;
    auto read_back = [&](void* dst, const void* src, size_t bytes) {
        hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
        return e != hipSuccess ? e : hipStreamSynchronize(st);
    };
    // A step's numbers go to host memory with an event behind them, and the step itself follows at once, deciding by the same numbers on the
    // device: the host learns of it while it runs (four updates and a refresh, n = 896: 677 -> 601 us, 300: 523 -> 398).  In a single tile the
    // products are too short to cover launches for nothing, 2 us each: there, after a step has been refused, the next ones wait for the host (four updates of 36 candidates and a
    // refresh that is mostly sweeps, n = 64: 447 -> 436 us, 16: 522 -> 509; n = 200 the other way 2077 -> 2086).  A refresh with nothing to do pays for them up to 128
    // dimensions: with copies 64 us at 64 dimensions, this 68; 83 and 83 at 200, 151 and 132 at 896.
    // Without such memory the host asks for a copy and waits for the step.
    eig_stats* const told_at = (eig_stats*)host;
    auto measure = [&](int with_t) {                           // E is in M afterwards
        hipLaunchKernelGGL(eig_residual_kernel, dim3(ntri, 2), dim3(MNT), MM_SMEM, st, V, A, ld, M, Rd, diagS, diagR);
        hipLaunchKernelGGL(eig_correction_kernel, dim3(ntri), dim3(EC_NT), 0, st, M, Rd, diagS, diagR, ld, n, with_t, inner_tol, part, st_s, st_t, st_j, flag);
        hipLaunchKernelGGL(eig_stats_kernel, dim3(1), dim3(1024), 0, st, part, st_s, st_t, st_j, diagS, diagR, ld, n, flag, lam, pair_s, partner, stats_dev,
                           told_at);
        return told_at ? hipEventRecord(told, st) : hipSuccess;
    };
    auto learn = [&](eig_stats& s) {
        if (!told_at) return read_back(&s, stats_dev, sizeof s);
        hipError_t e = hipEventSynchronize(told);
        std::memcpy(&s, told_at, sizeof s);
        return e;
    };
    auto apply = [&](const eig_stats* when) { hipLaunchKernelGGL(eig_apply_kernel, tiles, dim3(MNT), MM_SMEM, st, M, V, ld, A, when); };
    constexpr int STEPS_MAX = 12;                              // four or five at most are needed to go from 1/2 to rounding
    int sweeps = 0, steps = 0, all_steps = 0;
    float off = 0.f;
    bool done = false, try_steps = refine, ahead = true;
    while (!done) {
        bool moved = false;
        while (try_steps && steps < STEPS_MAX) {
            eig_stats s;
            hipError_t e = measure(1);
            if (e != hipSuccess) return e;
            const auto step = [&]() {
                hipLaunchKernelGGL(eig_pair_kernel, dim3(n), dim3(256), 0, st, M, pair_s, lam, partner, ld, stats_dev);
                apply(stats_dev);
            };
            if (ahead) step();
            e = learn(s);
            if (e != hipSuccess) return e;
            if (!s.fits) { ahead = nt > 1; break; }
            if (!ahead && s.go) step();
            ++steps, ++all_steps;
            off = s.off;
            done = s.off <= tol && s.esum <= LAST_STEP && s.strong == 0;      // the step's error is of the order of |E|^2: 1e-10
            if (s.go) {
                std::swap(V, A);
                moved = true;
                if (!done) multiply();
            }
            if (done) break;
        }
        if (done) break;
        // back to rotations, which need orthonormal columns
        for (int i = 0; moved && i < STEPS_MAX; ++i) {
            eig_stats s;
            hipError_t e = measure(0);
            if (e == hipSuccess) e = learn(s);
            if (e != hipSuccess) return e;
            moved = s.esum > 1e-13f * (float)npad;
            if (!moved) break;
            apply(nullptr);
            std::swap(V, A);
            multiply();
        }
        if (sweeps == max_sweeps) break;
        for (int round = 0; round < nblk - 1; ++round) {
            hipLaunchKernelGGL(eig_gram_kernel, dim3(npairs, S), dim3(256), 0, st, A, ld, n, nblk, round, chunks_per_slice, Gpart);
            hipLaunchKernelGGL(eig_small_kernel, dim3(npairs), dim3(SMALL_NT), two_mats, st, Gpart, S, Q, flag, rotated, 4, inner_tol);
            hipLaunchKernelGGL(eig_update_kernel, dim3(npairs, (chunks + UCH - 1) / UCH, 2), dim3(256), two_mats, st, A, V, ld, n, nblk, round, Q, rotated);
        }
        ++sweeps;
        unsigned bits = 0;
        hipError_t e = read_back(&bits, flag, sizeof bits);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(eig_clear_kernel, dim3(1), dim3(1), 0, st, flag);
        std::memcpy(&off, &bits, sizeof off);
        if (off <= tol) {                                      // the sweep that measured `off` has also rotated: it counts
            hipLaunchKernelGGL(eig_lambda_kernel, dim3(n), dim3(256), 0, st, A, V, ld, n, lam);
            done = true;
        }
        try_steps = refine && off < 0.1f;                      // far from diagonal a step cannot be taken: not worth the products
        steps = 0;
    }
    if (!done) hipLaunchKernelGGL(eig_lambda_kernel, dim3(n), dim3(256), 0, st, A, V, ld, n, lam);
    if (V != Vt) {
        hipError_t e = hipMemcpyAsync(Vt, V, (size_t)npad * ld * sizeof(double), hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(eig_finish_kernel, tiles, dim3(256), 0, st, V, lam, ld, n, B, D);
    if (sweeps_done) *sweeps_done = sweeps + all_steps;
    if (off_final) *off_final = off;
    return hipGetLastError();
}

}  // namespace essa_k
