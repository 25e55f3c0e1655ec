// Seed -> candidate sampling kernels (paper: Method, "Evolutionary optimization"; Algorithm 1,
// "sample candidate offsets from shared seeds"), the theta -> singular-value scatter, and the skinny
// fp32 product with the covariance basis that both the sampler and the update use.
#include "essa_internal.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;

namespace {

// Philox4x32-10 of Salmon et al. (SC'11): ten rounds of two 32x32->64 multiplies and xors, the key
// bumped by the Weyl constants between rounds.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint2 k) {
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int rnd = 0; rnd < 10; ++rnd) {
        if (rnd > 0) { k.x += W0; k.y += W1; }
        const uint32_t hi0 = __umulhi(M0, c.x), lo0 = M0 * c.x;
        const uint32_t hi1 = __umulhi(M1, c.z), lo1 = M1 * c.z;
        c = make_uint4(hi1 ^ c.y ^ k.x, lo1, hi0 ^ c.w ^ k.y, lo0);
    }
    return c;
}

// Box-Muller on 24-bit uniforms, evaluated in fp64 and rounded once to fp32 so that the value does
// not depend on the accuracy of fp32 log / sincos near u = 1.
__device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb, float& za, float& zb) {
    const double ua = ((double)(wa >> 8) + 0.5) * 0x1p-24;
    const double ub = ((double)(wb >> 8) + 0.5) * 0x1p-24;
    const double rho = sqrt(-2.0 * log(ua));
    double s, c;
    sincospi(2.0 * ub, &s, &c);
    za = (float)(rho * c);
    zb = (float)(rho * s);
}

__global__ void philox_words_kernel(const uint32_t* __restrict__ seeds, int K, int n_blocks, uint32_t* __restrict__ out) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)K * n_blocks) return;
    const int k = (int)(idx / n_blocks), c = (int)(idx % n_blocks);
    const uint4 w = philox4x32_10(make_uint4((uint32_t)c, 0u, 0u, 0u), make_uint2(seeds[k], 0u));
    reinterpret_cast<uint4*>(out)[idx] = w;
}

using essa_k::tiled_rows_at;

// The ranking of K <= 256 rewards (larger first, ties by index, NaN last), worked out by the whole workgroup in LDS -- a few hundred
// comparisons instead of a kernel launch of its own; the first workgroup also writes it to rank_order.
__device__ __forceinline__ void rank_in_lds(const float* rank_F, int rank_K, int32_t* rank_order, float* key, int* ord) {
    const int i = threadIdx.x;
    if (i < rank_K) {
        const float f = rank_F[i];
        key[i] = (f != f) ? -INFINITY : f;
    }
    __syncthreads();
    if (i < rank_K) {
        const float mine = key[i];
        int better = 0;
        for (int j = 0; j < rank_K; ++j) {
            const float o = key[j];
            better += (o > mine) || (o == mine && j < i);
        }
        ord[better] = i;
        if (blockIdx.x == 0 && rank_order) rank_order[better] = i;
    }
    __syncthreads();
}

// S[j, l] = D[l] * z_{cand(j)}[l],  cand(j) = sel ? sel[j] : j ; optional copy of z itself.  With rank_F the selection is the ranking of
// rank_K <= 256 rewards.  TILED: S in the tiles above, of a matrix of `rows` rows, else in rows.
template <bool TILED>
__global__ __launch_bounds__(256) void normals_scaled_kernel(const uint32_t* __restrict__ seeds, const int32_t* __restrict__ sel, int J, int rows, int n,
                                                            const float* __restrict__ D, float* __restrict__ S, float* __restrict__ z_out,
                                                            const float* __restrict__ rank_F, int rank_K, int32_t* __restrict__ rank_order) {
    __shared__ float key[256];
    __shared__ int ord[256];
    if (rank_F) rank_in_lds(rank_F, rank_K, rank_order, key, ord);
    const int nb = TILED ? (n + 15) / 16 * 4 : (n + 3) / 4;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)J * nb) return;
    const int j = (int)(idx / nb), c = (int)(idx % nb);
    const int cand = rank_F ? ord[j] : (sel ? sel[j] : j);
    const uint4 w = philox4x32_10(make_uint4((uint32_t)c, 0u, 0u, 0u), make_uint2(seeds[cand], 0u));
    float z[4];
    box_muller(w.x, w.y, z[0], z[1]);
    box_muller(w.z, w.w, z[2], z[3]);
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int l = 4 * c + e;
        v[e] = l < n ? (D ? D[l] * z[e] : z[e]) : 0.f;
        if (l < n) {
            if (!TILED) S[(size_t)j * n + l] = v[e];
            if (z_out) z_out[(size_t)j * n + l] = z[e];
        }
    }
    if (TILED) *reinterpret_cast<float4*>(S + tiled_rows_at(j, 4 * c, rows, n)) = make_float4(v[0], v[1], v[2], v[3]);
}

// The right-hand sides of an update in one launch: rows i < ny the selected D * z_i, row ny z_w = sum_{i < mu} w[i] z_i (fp64, i ascending),
// row ny + 1 D * z_w; z_i itself to Z when asked for.  A workgroup takes 16 blocks of four columns and 32 candidates at a time, whose normals
// meet in LDS.  Latency: one launch in place of two (n = 3584, 16 of 32 candidates: 5.3 + 4.0 -> 6 us); beyond 64 candidates the
// passes in a row take longer than the launch saved, and the kernels below do it.
constexpr int RHS_C = 32, RHS_B = 16;
__global__ __launch_bounds__(RHS_C * RHS_B) void update_rhs_kernel(const uint32_t* __restrict__ seeds, const int32_t* __restrict__ sel, int ny, int mu, int n,
                                                                  const float* __restrict__ w, const float* __restrict__ D, float* __restrict__ S, float* __restrict__ Z,
                                                                  const float* __restrict__ rank_F, int rank_K, int32_t* __restrict__ rank_order) {
    __shared__ float key[256];
    __shared__ int ord[256];
    __shared__ float zs[RHS_C][RHS_B * 4 + 1];
    if (rank_F) rank_in_lds(rank_F, rank_K, rank_order, key, ord);
    const int cb = threadIdx.x % RHS_B, ci = threadIdx.x / RHS_B, c = blockIdx.x * RHS_B + cb, l0 = blockIdx.x * RHS_B * 4;
    const bool in = c < (n + 15) / 16 * 4;
    float d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = 4 * c + e < n ? D[4 * c + e] : 0.f;
    double acc = 0.0;                                      // threads 0 .. 63: column l0 + thread
    for (int i0 = 0; i0 < ny; i0 += RHS_C) {
        const int i = i0 + ci;
        float z[4] = {0.f, 0.f, 0.f, 0.f};
        if (i < ny && in) {
            const uint4 p = philox4x32_10(make_uint4((uint32_t)c, 0u, 0u, 0u), make_uint2(seeds[rank_F ? ord[i] : sel[i]], 0u));
            box_muller(p.x, p.y, z[0], z[1]);
            box_muller(p.z, p.w, z[2], z[3]);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = 4 * c + e < n ? d[e] * z[e] : 0.f;
                if (Z && 4 * c + e < n) Z[(size_t)i * n + 4 * c + e] = z[e];
            }
            *reinterpret_cast<float4*>(S + tiled_rows_at(i, 4 * c, ny + 2, n)) = make_float4(v[0], v[1], v[2], v[3]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) zs[ci][cb * 4 + e] = z[e];
        __syncthreads();
        if (threadIdx.x < RHS_B * 4)
            for (int k = 0; k < RHS_C && i0 + k < mu; ++k) acc += (double)w[i0 + k] * (double)zs[k][threadIdx.x];
        __syncthreads();
    }
    const int l = l0 + threadIdx.x;
    if (threadIdx.x < RHS_B * 4 && l < (n + 15) / 16 * 16) {
        const float zw = l < n ? (float)acc : 0.f;
        S[tiled_rows_at(ny, l, ny + 2, n)] = zw;
        S[tiled_rows_at(ny + 1, l, ny + 2, n)] = l < n ? D[l] * zw : 0.f;
    }
}

// theta[k, i] = m[i] + sigma sum_l B[i, l] D[l] z_k[l] in one launch for a search of at most 64 dimensions: a few candidates a
// workgroup, their normals and B in LDS.  Latency binds: the products of a thread's outputs come one after the other (n = 64, 0.8 us each), and code is fetched
// anew for every launch (four outputs of a thread side by side, in longer code: 7.6 -> 10 us at 32 candidates).
constexpr int SMALL_N = 64, SMALL_K = 16;
__global__ __launch_bounds__(256) void sample_small_kernel(const uint32_t* __restrict__ seeds, int K, int per, int n, const float* __restrict__ m, const float* __restrict__ B,
                                                          const float* __restrict__ D, const essa_cma_scalars* __restrict__ sc, float* __restrict__ theta,
                                                          float* __restrict__ z_out) {
    __shared__ float Bs[SMALL_N][SMALL_N + 1], S[SMALL_K][SMALL_N + 1];
    const int tid = threadIdx.x, c = tid & 15, k = tid >> 4, k0 = blockIdx.x * per;
    for (int e = tid; e < n * n; e += 256) Bs[e / n][e % n] = B[e];
    const float sigma = sc->sigma;
    if (k < per && k0 + k < K && 4 * c < n) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)c, 0u, 0u, 0u), make_uint2(seeds[k0 + k], 0u));
        float z[4];
        box_muller(w.x, w.y, z[0], z[1]);
        box_muller(w.z, w.w, z[2], z[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int l = 4 * c + e;
            if (l < n) {
                S[k][l] = D[l] * z[e];
                if (z_out) z_out[(size_t)(k0 + k) * n + l] = z[e];
            }
        }
    }
    __syncthreads();
    for (int o = tid; o < per * n; o += 256) {
        const int kk = o / n, i = o % n;
        if (k0 + kk >= K) break;
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        int l = 0;
        for (; l + 4 <= n; l += 4)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = fmaf(S[kk][l + e], Bs[i][l + e], a[e]);
        for (; l < n; ++l) a[0] = fmaf(S[kk][l], Bs[i][l], a[0]);
        theta[(size_t)(k0 + kk) * n + i] = m[i] + sigma * ((a[0] + a[1]) + (a[2] + a[3]));
    }
}

// Distributions with a diagonal covariance: theta[k, l] = m[l] + s_k sigma d[l] z[l] (d = 1 without D).  With
// pairs, candidates 2j and 2j + 1 mirror each other around m on the direction of seed j (ARS, Algorithm 1).
__global__ void sample_diag_kernel(const uint32_t* __restrict__ seeds, int K, int n, const float* __restrict__ m,
                                   const float* __restrict__ D, const essa_cma_scalars* __restrict__ sc, int pairs,
                                   float* __restrict__ theta, float* __restrict__ z_out) {
    const int nb = (n + 3) / 4;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)K * nb) return;
    const int k = (int)(idx / nb), c = (int)(idx % nb);
    const uint32_t seed = pairs ? seeds[k >> 1] : seeds[k];
    const float sgn = (pairs && (k & 1)) ? -1.0f : 1.0f;
    const uint4 w = philox4x32_10(make_uint4((uint32_t)c, 0u, 0u, 0u), make_uint2(seed, 0u));
    float z[4];
    box_muller(w.x, w.y, z[0], z[1]);
    box_muller(w.z, w.w, z[2], z[3]);
    const float sigma = sc->sigma;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int l = 4 * c + e;
        if (l < n) {
            const float zs = sgn * z[e];
            theta[(size_t)k * n + l] = m[l] + (D ? sigma * D[l] : sigma) * zs;
            if (z_out) z_out[(size_t)k * n + l] = zs;
        }
    }
}

__global__ void theta_to_sigma_kernel(int P, int r, int n_top, const float* __restrict__ sftA, const float* __restrict__ sftB,
                                      const float* __restrict__ theta, int K, float* __restrict__ sA, float* __restrict__ sB) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)K * P * r;
    if (idx >= total) return;
    const int j = (int)(idx % r), p = (int)((idx / r) % P), k = (int)(idx / ((long long)r * P));
    const size_t n = (size_t)P * 2 * n_top;
    float a = sftA[p * r + j], b = sftB[p * r + j];
    if (j < n_top) {
        a += theta[k * n + (size_t)p * 2 * n_top + j];
        b += theta[k * n + (size_t)p * 2 * n_top + n_top + j];
    }
    sA[idx] = a;
    sB[idx] = b;
}

// Out[j, i] = bias[i] + scale * sum_l S[j,l] * B[i,l]        (fp32 MFMA 16x16x4; S in operand tiles)
// One workgroup = 16 rows of B x (16 * JB) rows of S.  Its 8 waves interleave over chunks of 16 columns (a lane
// loads four consecutive floats of its row, which feed four MFMA steps) and their partial tiles are summed
// through LDS in a fixed order (bit-reproducible).  B is read exactly once when J <= 16 * JB.
constexpr int SG_WAVES = 8;
constexpr int SG_BUNCH = 2;          // chunks a wave asks for at once; two bunches in turn
typedef __attribute__((ext_vector_type(4))) float f32x4;
template <bool TAIL, int JB>
__global__ __launch_bounds__(SG_WAVES * 64) void skinny_gemm_nt_kernel(const float* __restrict__ S, int J, const float* __restrict__ B,
                                                                      int n, const float* __restrict__ bias,
                                                                      const essa_cma_scalars* __restrict__ sc, int use_sigma,
                                                                      float* __restrict__ Out) {
    __shared__ __attribute__((aligned(16))) float red[SG_WAVES][JB][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = blockIdx.x * 16, j0 = blockIdx.y * 16 * JB;
    const int l16 = lane & 15, kq = lane >> 4;
    const int i = i0 + l16;
    f32x4 acc[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) acc[jb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int nchunks = (n + 15) / 16;
    // A wave walks its chunks (wave, wave + 8, ...) in ascending order.
    {
        // Buffer loads: a row or a chunk past the end is an offset outside the descriptor and comes back as zeros, so there
        // is no branch around any load and the compiler can count them.  What bounds it is what the loads cost the CU's address path:
        // 16 rows x 64 bytes of B take it 55 cycles, a contiguous kilobyte of S 16 (S in rows cost as much as B, twice over).  A wave asks
        // for two chunks of both, and for the next two in front of the MFMAs of these: deeper bunches (14 of B, S behind them)
        // queue everybody's B in front of everybody's S.  Product / update and next candidates, us, S in rows and bunches of 14 against this:
        // n = 3584, 32 candidates 21.3 / 15.5 and 82 / 65; 64 candidates at n = 5121 303 / 191 (both); 896, 36 candidates 45 / 35 (both).
        // (n <= 16384: B stays below the descriptor's 2 GB.  S need not: its descriptor begins at this workgroup's tiles.)
        // The loads need 4-byte alignment only, so any n takes this path.  TAIL: n is not a multiple of 4, and the quad that
        // crosses the end of a row is the row's last four elements, moved into place.
        typedef __amdgpu_buffer_rsrc_t rsrc_t;
        constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
        const rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B), 0, (uint32_t)n * (uint32_t)n * 4u, 0x00020000);
        const int sshift = essa_k::tiled_rows_shift(J);
        const uint32_t tile = (uint32_t)nchunks << (sshift + 6);
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(S + tiled_rows_at(j0, 0, J, n)), 0, JB * tile, 0x00020000);
        uint32_t scol[JB];                                  // columns past J are not asked for
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) scol[jb] = j0 + 16 * jb + l16 < J ? (uint32_t)jb * tile + (uint32_t)((kq << sshift) + l16) * 16u : OUT_OF_RANGE;
        const uint32_t brow = (uint32_t)i * (uint32_t)n * 4u;                    // i >= n: beyond the descriptor
        auto ld_s = [&](int jb, int chunk) {               // a contiguous kilobyte
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, chunk < nchunks ? scol[jb] + ((uint32_t)chunk << (sshift + 6)) : OUT_OF_RANGE, 0, 0);
            f32x4 f;
            __builtin_memcpy(&f, &v, 16);
            return f;
        };
        auto ld = [&](rsrc_t r, uint32_t row_off, int chunk) {
            const int l = chunk * 16 + 4 * kq;
            f32x4 f;
            if (TAIL && n < 4) {                            // a row shorter than one load
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    f[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, l + e < n ? row_off + (uint32_t)(l + e) * 4u : OUT_OF_RANGE, 0, 0));
                return f;
            }
            const uint32_t off = l < n ? row_off + (uint32_t)(TAIL ? min(l, n - 4) : l) * 4u : OUT_OF_RANGE;
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
            __builtin_memcpy(&f, &v, 16);
            return f;
        };
        const int over = 4 - (n & 3);                       // TAIL: elements by which a row's last quad starts early
        auto place = [&](const f32x4& f, int chunk) {
            if (!TAIL) return f;
            const int l = chunk * 16 + 4 * kq;
            const bool cross = n >= 4 && l < n && l + 4 > n;
            f32x4 v;
            v[0] = cross ? (over == 3 ? f[3] : over == 2 ? f[2] : f[1]) : f[0];
            v[1] = cross ? (over == 3 ? 0.f : over == 2 ? f[3] : f[2]) : f[1];
            v[2] = cross ? (over == 1 ? f[3] : 0.f) : f[2];
            v[3] = cross ? 0.f : f[3];
            return v;
        };
        f32x4 a[2][SG_BUNCH], sv[2][SG_BUNCH][JB];
        auto ask = [&](int base, int set) {
#pragma unroll
            for (int u = 0; u < SG_BUNCH; ++u) a[set][u] = ld(rb, brow, base + u * SG_WAVES);
            __builtin_amdgcn_sched_barrier(0);              // left alone, the compiler moves every load down to its first use
#pragma unroll
            for (int u = 0; u < SG_BUNCH; ++u)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) sv[set][u][jb] = ld_s(jb, base + u * SG_WAVES);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply = [&](int base, int set) {
#pragma unroll
            for (int u = 0; u < SG_BUNCH; ++u) {
                const f32x4 au = place(a[set][u], base + u * SG_WAVES);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb) acc[jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(au[e], sv[set][u][jb][e], acc[jb], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr int STEP = SG_BUNCH * SG_WAVES;
        ask(wave, 0);
        for (int base = wave; base < nchunks; base += 2 * STEP) {
            ask(base + STEP, 1);
            multiply(base, 0);
            ask(base + 2 * STEP, 0);
            multiply(base + STEP, 1);
        }
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][jb][q][lane] = acc[jb][q];
    __syncthreads();
    const float scale = use_sigma ? sc->sigma : 1.0f;
    for (int idx = threadIdx.x; idx < JB * 4 * 64; idx += SG_WAVES * 64) {
        const int ln = idx & 63, q = (idx >> 6) & 3, jb = idx >> 8;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < SG_WAVES; ++w) sum += red[w][jb][q][ln];
        // accumulator element q of lane ln: row (of B) 4*(ln/16) + q, column (of S) ln%16
        const int ii = i0 + 4 * (ln >> 4) + q;
        const int jj = j0 + 16 * jb + (ln & 15);
        if (ii < n && jj < J) Out[(size_t)jj * n + ii] = (bias ? bias[ii] : 0.f) + scale * sum;
    }
}

}  // namespace

namespace essa_k {

hipError_t philox_words(hipStream_t st, const uint32_t* seeds, int K, int n_blocks, uint32_t* out) {
    const long long total = (long long)K * n_blocks;
    hipLaunchKernelGGL(philox_words_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, seeds, K, n_blocks, out);
    return hipGetLastError();
}

hipError_t normals_scaled(hipStream_t st, const uint32_t* seeds, const int32_t* sel, int J, int n, const float* D, float* S,
                          float* z_out, const float* rank_F, int rank_K, int32_t* rank_order) {
    const long long total = (long long)J * ((n + 3) / 4);
    hipLaunchKernelGGL(normals_scaled_kernel<false>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, seeds, sel, J, J, n, D, S, z_out, rank_F,
                       rank_K, rank_order);
    return hipGetLastError();
}

hipError_t normals_tiled(hipStream_t st, const uint32_t* seeds, const int32_t* sel, int J, int rows, int n, const float* D, float* S,
                         float* z_out, const float* rank_F, int rank_K, int32_t* rank_order) {
    const long long total = (long long)J * ((n + 15) / 16 * 4);
    hipLaunchKernelGGL(normals_scaled_kernel<true>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, seeds, sel, J, rows, n, D, S, z_out, rank_F,
                       rank_K, rank_order);
    return hipGetLastError();
}

hipError_t update_rhs(hipStream_t st, const uint32_t* seeds, const int32_t* sel, int ny, int mu, int n, const float* w, const float* D, float* S,
                      float* Z, const float* rank_F, int rank_K, int32_t* rank_order) {
    const int blocks = (n + 15) / 16 * 4;
    hipLaunchKernelGGL(update_rhs_kernel, dim3((blocks + RHS_B - 1) / RHS_B), dim3(RHS_C * RHS_B), 0, st, seeds, sel, ny, mu, n, w, D, S, Z, rank_F, rank_K,
                       rank_order);
    return hipGetLastError();
}

bool sample_small(hipStream_t st, const uint32_t* seeds, int K, int n, const float* m, const float* B, const float* D, const essa_cma_scalars* sc, float* theta,
                  float* z_out) {
    // B and the normals of 16 candidates are kept for at most 64 dimensions.  us in a replayed graph, two launches / one: 16 dimensions 4.9 / 3.4 at 4 candidates, 8.7 / 8.5
    // at 24576, 9.0 / 10.4 at 32768 (mostly idle threads, so they go in two); 64 dimensions 5.4 / 5.5 at 4, 57.5 / 42.3 at 65536.  A caller who does not record is
    // spared 3 us a call besides.
    if (n > SMALL_N || (n <= 16 && K > 24576)) return false;
    // An output a thread, while there are not so many workgroups that their copies of B take longer: 64 dimensions, 16 candidates a workgroup / 4: 7.9 / 5.7 at 32,
    // 8.2 / 6.0 at 1024, 8.8 / 8.2 at 4096 (two launches 6.4, 7.9, 9.1); 32 dimensions, 16 / 8: 4.7 / 4.1 at 32
    int per = n <= 16 ? 16 : n <= 32 ? 8 : 4;
    if (K > 1024 * per) per = SMALL_K;
    hipLaunchKernelGGL(sample_small_kernel, dim3((K + per - 1) / per), dim3(256), 0, st, seeds, K, per, n, m, B, D, sc, theta, z_out);
    return true;
}

hipError_t sample_diag(hipStream_t st, const uint32_t* seeds, int K, int n, const float* m, const float* D,
                       const essa_cma_scalars* sc, int pairs, float* theta, float* z_out) {
    const long long total = (long long)K * ((n + 3) / 4);
    hipLaunchKernelGGL(sample_diag_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, seeds, K, n, m, D, sc, pairs, theta,
                       z_out);
    return hipGetLastError();
}

template <int JB>
static void launch_skinny(hipStream_t st, const float* S, int J, const float* B, int n, const float* bias, const essa_cma_scalars* sc,
                          int use_sigma, float* Out) {
    dim3 grid((n + 15) / 16, (J + 16 * JB - 1) / (16 * JB));
    if (n % 4 != 0)
        hipLaunchKernelGGL((skinny_gemm_nt_kernel<true, JB>), grid, dim3(SG_WAVES * 64), 0, st, S, J, B, n, bias, sc, use_sigma, Out);
    else
        hipLaunchKernelGGL((skinny_gemm_nt_kernel<false, JB>), grid, dim3(SG_WAVES * 64), 0, st, S, J, B, n, bias, sc, use_sigma, Out);
}

hipError_t skinny_gemm_nt(hipStream_t st, const float* S, int J, const float* B, int n, const float* bias,
                          const essa_cma_scalars* sc, int use_sigma, float* Out) {
    // as few passes over B as 64 columns each allow, their blocks of 16 columns spread evenly: a block of padding costs what a full one does
    // (candidates at n = 3584, us, two widths of 32 and 64 columns / this: 36 of them 31.5 / 29.4, 70 58 / 51, 96 62.6 / 59.4)
    const int blocks = (J + 15) / 16, passes = (blocks + 3) / 4;
    switch ((blocks + passes - 1) / passes) {
        case 1: launch_skinny<1>(st, S, J, B, n, bias, sc, use_sigma, Out); break;
        case 2: launch_skinny<2>(st, S, J, B, n, bias, sc, use_sigma, Out); break;
        case 3: launch_skinny<3>(st, S, J, B, n, bias, sc, use_sigma, Out); break;
        default: launch_skinny<4>(st, S, J, B, n, bias, sc, use_sigma, Out);
    }
    return hipGetLastError();
}

hipError_t theta_to_sigma(hipStream_t st, int P, int r, int n_top, const float* sftA, const float* sftB, const float* theta,
                          int K, float* sA, float* sB) {
    const long long total = (long long)K * P * r;
    hipLaunchKernelGGL(theta_to_sigma_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, P, r, n_top, sftA, sftB, theta,
                       K, sA, sB);
    return hipGetLastError();
}

}  // namespace essa_k
