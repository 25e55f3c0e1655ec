// Population-batched forward of SVD-parameterised LoRA projections on a shared quantised base weight
// (paper: Algorithm 1, reconstruction step W' = W + B'A', A' = U_A diag(sA) V_A^T, B' = U_B diag(sB) V_B^T,
// followed by the inference pass).  The candidate's dense W' is never formed:
//     y_i = W_deq x_i + U_B ( sB_c * ( (V_B^T U_A) ( sA_c * (V_A^T x_i) ) ) ),   c = row2cand[i].
//
// Launch sequence of one grouped call:
//   1. prologue: per row, the rank-space vector u_i = sB_c * (M (sA_c * V_A^T x_i)) (and, where the
//      format needs them, per-group sums of x or the row's int8 quantisation);
//   2. GEMM: Y = X W_q^T with the dequantisation fused (weights converted in registers on their way
//      into LDS, scales applied to the fp32 accumulators), and the rank-r term U_B u_i added by one or
//      two more MFMA steps in the epilogue.
#include <type_traits>

#include "essa_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;

namespace {

struct fwd_args {
    essa_k::fwd_item it[ESSA_MAX_GROUP];
    int tile_start[ESSA_MAX_GROUP + 1];   // prefix sums of GEMM tiles per item
    int n_items;
    unsigned flags;
};

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    // round to nearest even in one instruction (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}
// exact for integers of at most 8 significant bits
__device__ __forceinline__ uint32_t pack_bf16_trunc(float lo, float hi) {
    return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
}

// ------------------------------------------------------------------------------------------------
// 1. prologue: one workgroup per row
// ------------------------------------------------------------------------------------------------
template <int RP, bool XBF16>
__global__ __launch_bounds__(256) void prologue_kernel(fwd_args a) {
    const essa_k::fwd_item& it = a.it[blockIdx.y];
    const int i = blockIdx.x;
    if (i >= it.R) return;
    __shared__ float part[4][RP];
    __shared__ float tvec[RP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int din = it.d_in;
    // what stands behind the reduction is on its way from here: the row's singular values and this thread's row of M
    const int c = it.row2cand[i], jr = min(tid, it.r - 1);
    const float sa = it.sigmaA[(size_t)c * it.sigma_stride + jr], sb = it.sigmaB[(size_t)c * it.sigma_stride + jr];
    f32x4 mrow[RP / 4];
#pragma unroll
    for (int q = 0; q < RP / 4; ++q) mrow[q] = *reinterpret_cast<const f32x4*>(it.M + min(tid, RP - 1) * RP + 4 * q);
    float acc[RP];
#pragma unroll
    for (int j = 0; j < RP; ++j) acc[j] = 0.f;
    for (int l = tid; l < din; l += 256) {
        const float x = XBF16 ? bf16_bits_to_f32(((const uint16_t*)it.X)[(size_t)i * din + l]) : ((const float*)it.X)[(size_t)i * din + l];
        const float4* v = reinterpret_cast<const float4*>(it.VA32 + (size_t)l * RP);
#pragma unroll
        for (int j4 = 0; j4 < RP / 4; ++j4) {
            const float4 vv = v[j4];
            acc[4 * j4 + 0] = fmaf(x, vv.x, acc[4 * j4 + 0]);
            acc[4 * j4 + 1] = fmaf(x, vv.y, acc[4 * j4 + 1]);
            acc[4 * j4 + 2] = fmaf(x, vv.z, acc[4 * j4 + 2]);
            acc[4 * j4 + 3] = fmaf(x, vv.w, acc[4 * j4 + 3]);
        }
    }
#pragma unroll
    for (int j = 0; j < RP; ++j) {
        float v = acc[j];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) part[wave][j] = v;
    }
    __syncthreads();
    if (tid < RP) {
        const float t = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
        tvec[tid] = tid < it.r ? sa * t : 0.f;             // M is zero there as well
    }
    __syncthreads();
    if (tid < RP) {
        float u = 0.f;
        if (tid < it.r && !(a.flags & ESSA_BASE_ONLY)) {
#pragma unroll
            for (int l = 0; l < RP; ++l) u = fmaf(mrow[l >> 2][l & 3], tvec[l], u);
            u *= sb;
        }
        it.U32[(size_t)i * RP + tid] = u;
        // bf16 head and tail: u = hi + lo to about 2^-17, so that the MFMA epilogue loses nothing
        const uint16_t hi = f32_to_bf16_bits(u);
        it.U16[(size_t)i * 2 * RP + tid] = hi;
        it.U16[(size_t)i * 2 * RP + RP + tid] = f32_to_bf16_bits(u - bf16_bits_to_f32(hi));
    }
    if (it.groups > 0) {   // group sums of x for the asymmetric 4-bit format
        for (int g = wave; g < it.groups; g += 4) {
            const int l = g * 128 + 2 * lane;
            float s;
            if (XBF16) {
                const uint32_t two = *reinterpret_cast<const uint32_t*>((const uint16_t*)it.X + (size_t)i * din + l);
                s = __uint_as_float(two << 16) + __uint_as_float(two & 0xffff0000u);
            } else {
                const float2 two = *reinterpret_cast<const float2*>((const float*)it.X + (size_t)i * din + l);
                s = two.x + two.y;
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (lane == 0) it.xsum[(size_t)i * it.groups + g] = s;
        }
    }
}

// per-row dynamic int8 quantisation of bf16 activations (W8A8 mode); the decisions are taken in fp32:
// amax = max|x|, inv = 127/amax, q = rint(x*inv) (ties to even), scale = amax/127.
__global__ __launch_bounds__(256) void rowquant_kernel(fwd_args a) {
    const essa_k::fwd_item& it = a.it[blockIdx.y];
    const int i = blockIdx.x;
    if (i >= it.R) return;
    __shared__ float wmax[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint16_t* x = (const uint16_t*)it.X + (size_t)i * it.d_in;
    float m = 0.f;
    for (int l = tid; l < it.d_in; l += 256) m = fmaxf(m, fabsf(bf16_bits_to_f32(x[l])));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if (lane == 0) wmax[wave] = m;
    __syncthreads();
    const float amax = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    const float inv = amax > 0.f ? 127.0f / amax : 0.f;
    for (int l = tid; l < it.d_in; l += 256) {
        float q = rintf(bf16_bits_to_f32(x[l]) * inv);
        q = fminf(fmaxf(q, -127.f), 127.f);
        it.Xq[(size_t)i * it.d_in + l] = (int8_t)(int)q;
    }
    if (tid == 0) it.xscale[i] = amax > 0.f ? amax / 127.0f : 0.f;
}

// ------------------------------------------------------------------------------------------------
// 2a. generic fp32 GEMM (fp32 activations, or shapes the MFMA kernels do not take)
// ------------------------------------------------------------------------------------------------
// Four consecutive columns k .. k + 3 of an activation row and of a row of int8 weights as fp32, for any alignment; columns past
// d_in and rows past the last are zeros.
template <bool XBF16>
__device__ __forceinline__ f32x4 x_quad(const essa_k::fwd_item& it, int i, int k) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (i >= it.R) return v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (k + e < it.d_in) {
            const size_t at = (size_t)i * it.d_in + k + e;
            v[e] = XBF16 ? bf16_bits_to_f32(((const uint16_t*)it.X)[at]) : ((const float*)it.X)[at];
        }
    return v;
}
__device__ __forceinline__ f32x4 w_quad(const essa_k::fwd_item& it, int o, int k) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (o >= it.d_out || k >= it.d_in) return v;
    const size_t at = (size_t)o * it.d_in + k;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (k + e < it.d_in) v[e] = (float)((const int8_t*)it.Wq)[at + e];
    return v;
}

// fp32 products on the 16 x 16 x 4 MFMA.  Tile = 16 MT rows x 16 MT channels, its 8 waves split K (wave w takes the 16-column
// steps w, w + 8, ...) and their sums meet in LDS, added in wave order.  Operands go memory -> registers: lane (l16, kg) holds
// four consecutive columns 4 kg .. of its row, and MFMA j multiplies column 4 kg + j of both sides.  A single small matrix
// is all latency: many workgroups, a short K chain in each, no barrier before the end.
// us per call (prologue included), 64 x 64 tiles of 4 x 4 outputs per thread on the vector ALU / this: one int8 matrix of 512 x 512 at
// 64 rows 73 / 12, 1024 x 1024 at 256 118 / 21 and at 4096 222 / 168, 4096 x 4096 at 16 372 / 32 and at 2048 1168 / 979 (70 TFLOP/s);
// rows of no whole quads, 1021 x 1021 at 200, 119 / 49; 4-bit, 1024 x 1024 at 64, 120 / 15, 4096 x 4096 at 1024, 667 / 550.
template <bool XBF16, bool YBF16, int MT>
__global__ __launch_bounds__(512) void gemm_f32_kernel(fwd_args a) {
    constexpr int BM = 16 * MT;
    __shared__ float red[8][MT * MT][256];
    int g = 0;
    while (g + 1 < a.n_items && (int)blockIdx.x >= a.tile_start[g + 1]) ++g;
    const essa_k::fwd_item& it = a.it[g];
    const int tile = blockIdx.x - a.tile_start[g];
    const int tiles_m = (it.R + BM - 1) / BM;
    const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BM;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kg = lane >> 4;
    const int din = it.d_in, dout = it.d_out;
    f32x4 acc[MT][MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < MT; ++n) acc[m][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
    constexpr int U = 4;                                   // steps whose loads are asked for together
    // FAST: int8 weights and rows of whole quads; addresses are clamped and the columns past d_in zeroed in the registers, so that
    // there is no branch between the loads.  Rows past the last one are never stored.
    auto loop = [&](auto fast_c) {
        constexpr bool FAST = decltype(fast_c)::value;
        size_t xrow[MT], wrow[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            xrow[m] = (size_t)min(m0 + 16 * m + l16, it.R - 1) * din;
            wrow[m] = (size_t)min(n0 + 16 * m + l16, dout - 1) * din;
        }
        for (int k0 = wave * 16; k0 < din; k0 += 128 * U) {
            f32x4 xv[U][MT], wv[U][MT];
            if constexpr (FAST) {
                uint2 xb[U][MT];
                uint32_t wb[U][MT];
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    const int k = min(k0 + 128 * s + 4 * kg, din - 4);
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        if (XBF16) xb[s][m] = *reinterpret_cast<const uint2*>((const uint16_t*)it.X + xrow[m] + k);
                        else xv[s][m] = *reinterpret_cast<const f32x4*>((const float*)it.X + xrow[m] + k);
                        wb[s][m] = *reinterpret_cast<const uint32_t*>((const int8_t*)it.Wq + wrow[m] + k);
                    }
                }
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    const bool in = k0 + 128 * s + 4 * kg < din;
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        if (XBF16)
                            xv[s][m] = (f32x4){__uint_as_float(xb[s][m].x << 16), __uint_as_float(xb[s][m].x & 0xffff0000u), __uint_as_float(xb[s][m].y << 16),
                                               __uint_as_float(xb[s][m].y & 0xffff0000u)};
                        const uint32_t w = wb[s][m];
                        wv[s][m] = (f32x4){(float)(int8_t)(w & 0xff), (float)(int8_t)((w >> 8) & 0xff), (float)(int8_t)((w >> 16) & 0xff), (float)(int8_t)(w >> 24)};
#pragma unroll
                        for (int e = 0; e < 4; ++e) xv[s][m][e] = in ? xv[s][m][e] : 0.f;
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    const int k = k0 + 128 * s + 4 * kg;
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        xv[s][m] = x_quad<XBF16>(it, m0 + 16 * m + l16, k);
                        wv[s][m] = w_quad(it, n0 + 16 * m + l16, k);
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < U; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
#pragma unroll
                        for (int n = 0; n < MT; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s][m][j], wv[s][n][j], acc[m][n], 0, 0, 0);
        }
    };
    // 4-bit weights: a wave takes whole groups of 128 columns, so that their scales and zeros are fetched once.  The order of the sums
    // is the same whether the rows can be loaded 16 bytes at a time (FAST) or not.
    auto loop_q4 = [&](auto fast_c) {
        constexpr bool FAST = decltype(fast_c)::value;
        size_t xrow[MT], wrow[MT];
        int o[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            o[m] = min(n0 + 16 * m + l16, dout - 1);
            xrow[m] = (size_t)min(m0 + 16 * m + l16, it.R - 1) * din;
            wrow[m] = (size_t)o[m] * din;
        }
        for (int grp = wave; grp < it.groups; grp += 8) {
            float sc[MT], z[MT];
#pragma unroll
            for (int n = 0; n < MT; ++n) {
                sc[n] = it.scale[(size_t)o[n] * it.groups + grp];
                z[n] = it.zero[(size_t)o[n] * it.groups + grp];
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                f32x4 xv[U][MT];
                uint32_t wb[U][MT];
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    const int k = grp * 128 + half * 64 + 16 * s + 4 * kg;
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        if (!FAST) {
                            xv[s][m] = x_quad<XBF16>(it, m0 + 16 * m + l16, k);
                        } else if (XBF16) {
                            const uint2 b = *reinterpret_cast<const uint2*>((const uint16_t*)it.X + xrow[m] + k);
                            xv[s][m] = (f32x4){__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
                        } else {
                            xv[s][m] = *reinterpret_cast<const f32x4*>((const float*)it.X + xrow[m] + k);
                        }
                        wb[s][m] = *reinterpret_cast<const uint16_t*>((const uint8_t*)it.Wq + ((wrow[m] + k) >> 1));
                    }
                }
#pragma unroll
                for (int s = 0; s < U; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float w[MT];
#pragma unroll
                        for (int n = 0; n < MT; ++n) w[n] = sc[n] * ((float)((wb[s][n] >> (4 * j)) & 15u) - z[n]);
#pragma unroll
                        for (int m = 0; m < MT; ++m)
#pragma unroll
                            for (int n = 0; n < MT; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s][m][j], w[n], acc[m][n], 0, 0, 0);
                    }
            }
        }
    };
    const bool x_quads = din % 4 == 0 && ((uintptr_t)it.X & (XBF16 ? 7 : 15)) == 0;
    if (it.quant == ESSA_QUANT_INT8_PERCH) {
        if (x_quads) loop(std::true_type{});
        else loop(std::false_type{});
    } else if (x_quads) loop_q4(std::true_type{});
    else loop_q4(std::false_type{});
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < MT; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave][m * MT + n][(4 * kg + e) * 16 + l16] = acc[m][n][e];
    __syncthreads();
    for (int q = tid; q < MT * MT * 256; q += 512) {
        const int blk = q >> 8, i = m0 + 16 * (blk / MT) + ((q >> 4) & 15), o = n0 + 16 * (blk % MT) + (q & 15);
        if (i >= it.R || o >= dout) continue;
        float l = 0.f;
        if (!(a.flags & ESSA_BASE_ONLY)) {                 // columns r .. rp - 1 of both are zero
            const f32x4* u = reinterpret_cast<const f32x4*>(it.U32 + (size_t)i * it.rp);
            const f32x4* ub = reinterpret_cast<const f32x4*>(it.UB32 + (size_t)o * it.rp);
            for (int j0 = 0; j0 < it.rp; j0 += 16) {
                f32x4 uv[4], bv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { uv[e] = u[j0 / 4 + e]; bv[e] = ub[j0 / 4 + e]; }
#pragma unroll
                for (int e = 0; e < 16; ++e) l = fmaf(uv[e >> 2][e & 3], bv[e >> 2][e & 3], l);
            }
        }
        const float sc = it.quant == ESSA_QUANT_INT8_PERCH ? it.scale[o] : 1.f;
        float v = red[0][blk][q & 255];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += red[w][blk][q & 255];
        v *= sc;
        if (a.flags & ESSA_LORA_ONLY) v = 0.f;
        if (!(a.flags & ESSA_BASE_ONLY)) v += l;
        if (YBF16) ((uint16_t*)it.Y)[(size_t)i * dout + o] = f32_to_bf16_bits(v);
        else ((float*)it.Y)[(size_t)i * dout + o] = v;
    }
}

// ------------------------------------------------------------------------------------------------
// 2b. MFMA GEMM with fused dequantisation.  MODE 0: int8 weights x bf16 activations (bf16 MFMA);
// MODE 1: 4-bit group-128 weights x bf16 activations (bf16 MFMA, per-group fp32 rescale);
// MODE 2: int8 weights x int8 activations (int8 MFMA, exact int32 accumulation).
// 256 threads = 2 x 2 waves, each wave owns a (BM/2) x (BN/2) tile made of 32x32 MFMA blocks.
// ------------------------------------------------------------------------------------------------
constexpr int BK = 64;

template <int BM, int BN, int MODE, bool YBF16, bool DUMP_I32>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(fwd_args a, int32_t* __restrict__ acc_out) {
    constexpr int MI = BM / 64, NI = BN / 64;
    constexpr int ESZ = MODE == 2 ? 1 : 2;                 // bytes per LDS element
    constexpr int LDA = (BK + (MODE == 2 ? 16 : 8));       // elements per LDS row (padded)
    __shared__ __attribute__((aligned(16))) unsigned char As[BM * LDA * ESZ];
    __shared__ __attribute__((aligned(16))) unsigned char Bs[BN * LDA * ESZ];

    int g = 0;
    while (g + 1 < a.n_items && (int)blockIdx.x >= a.tile_start[g + 1]) ++g;
    const essa_k::fwd_item& it = a.it[g];
    const int tile = blockIdx.x - a.tile_start[g];
    const int tiles_m = (it.R + BM - 1) / BM;
    const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, h = lane >> 5;
    const int din = it.d_in, dout = it.d_out, R = it.R, G = it.groups;

    // ---- global -> register staging -------------------------------------------------------------
    // X tile: BM rows x 64 elements; chunks of 16 bytes (8 bf16 or 16 int8)
    constexpr int XCH_ROW = MODE == 2 ? 4 : 8;                       // chunks per row
    constexpr int XCH = (BM * XCH_ROW + 255) / 256;                  // chunks per thread
    // W tile: BN rows x 64 elements; int8 -> 4 chunks per row, 4-bit -> 2 chunks per row
    constexpr int WCH_ROW = MODE == 1 ? 2 : 4;
    constexpr int WCH = (BN * WCH_ROW + 255) / 256;
    uint4 xr[XCH], wr[WCH];
    const unsigned char* Xb = MODE == 2 ? (const unsigned char*)it.Xq : (const unsigned char*)it.X;
    const size_t x_row_bytes = (size_t)din * ESZ;
    const size_t w_row_bytes = MODE == 1 ? (size_t)din / 2 : (size_t)din;
    const int nk = (din + BK - 1) / BK;

    auto load_tiles = [&](int kt) {
#pragma unroll
        for (int e = 0; e < XCH; ++e) {
            const int ch = tid + 256 * e, row = ch / XCH_ROW, part = ch % XCH_ROW;
            const int k = kt * BK + part * (16 / ESZ);
            xr[e] = make_uint4(0, 0, 0, 0);
            if (ch < BM * XCH_ROW && m0 + row < R && k < din)
                xr[e] = *reinterpret_cast<const uint4*>(Xb + (size_t)(m0 + row) * x_row_bytes + (size_t)k * ESZ);
        }
#pragma unroll
        for (int e = 0; e < WCH; ++e) {
            const int ch = tid + 256 * e, row = ch / WCH_ROW, part = ch % WCH_ROW;
            const int k = kt * BK + part * (MODE == 1 ? 32 : 16);
            wr[e] = make_uint4(0, 0, 0, 0);
            if (ch < BN * WCH_ROW && n0 + row < dout && k < din)
                wr[e] = *reinterpret_cast<const uint4*>((const unsigned char*)it.Wq + (size_t)(n0 + row) * w_row_bytes +
                                                        (MODE == 1 ? (size_t)k / 2 : (size_t)k));
        }
    };
    auto store_tiles = [&]() {
#pragma unroll
        for (int e = 0; e < XCH; ++e) {
            const int ch = tid + 256 * e, row = ch / XCH_ROW, part = ch % XCH_ROW;
            if (ch < BM * XCH_ROW) *reinterpret_cast<uint4*>(As + ((size_t)row * LDA + part * (16 / ESZ)) * ESZ) = xr[e];
        }
#pragma unroll
        for (int e = 0; e < WCH; ++e) {
            const int ch = tid + 256 * e, row = ch / WCH_ROW, part = ch % WCH_ROW;
            if (ch >= BN * WCH_ROW) continue;
            if (MODE == 2) {
                *reinterpret_cast<uint4*>(Bs + (size_t)row * LDA + part * 16) = wr[e];
            } else if (MODE == 0) {
                // 16 int8 -> 16 bf16 (exact)
                const uint32_t w4[4] = {wr[e].x, wr[e].y, wr[e].z, wr[e].w};
                uint32_t o[8];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int v = (int)w4[d];
                    const float f0 = (float)((v << 24) >> 24), f1 = (float)((v << 16) >> 24);
                    const float f2 = (float)((v << 8) >> 24), f3 = (float)(v >> 24);
                    o[2 * d] = pack_bf16_trunc(f0, f1);
                    o[2 * d + 1] = pack_bf16_trunc(f2, f3);
                }
                uint4* dst = reinterpret_cast<uint4*>(Bs + ((size_t)row * LDA + part * 16) * 2);
                dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
                dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
            } else {
                // 16 bytes = 32 nibbles -> 32 bf16 (exact): column 2j in the low nibble
                const uint32_t w4[4] = {wr[e].x, wr[e].y, wr[e].z, wr[e].w};
                uint4* dst = reinterpret_cast<uint4*>(Bs + ((size_t)row * LDA + part * 32) * 2);
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t o[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const uint32_t byte = (w4[d] >> (8 * b)) & 0xffu;
                        o[b] = pack_bf16_trunc((float)(byte & 15u), (float)(byte >> 4));
                    }
                    dst[d] = make_uint4(o[0], o[1], o[2], o[3]);
                }
            }
        }
    };

    using acc_t = typename std::conditional<MODE == 2, i32x16, f32x16>::type;
    acc_t acc[MI][NI];
    f32x16 tot[MODE == 1 ? MI : 1][MODE == 1 ? NI : 1];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[mi][ni][q] = 0;
            if (MODE == 1)
#pragma unroll
                for (int q = 0; q < 16; ++q) tot[mi][ni][q] = 0.f;
        }

    load_tiles(0);
    for (int kt = 0; kt < nk; ++kt) {
        store_tiles();
        __syncthreads();
        if (kt + 1 < nk) load_tiles(kt + 1);
        if constexpr (MODE == 2) {
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks) {
                i32x4 av[MI], bv[NI];
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
                    av[mi] = *reinterpret_cast<const i32x4*>(As + (size_t)(wm * (BM / 2) + mi * 32 + l32) * LDA + ks * 32 + 16 * h);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    bv[ni] = *reinterpret_cast<const i32x4*>(Bs + (size_t)(wn * (BN / 2) + ni * 32 + l32) * LDA + ks * 32 + 16 * h);
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc[mi][ni] = (acc_t)__builtin_amdgcn_mfma_i32_32x32x32_i8(av[mi], bv[ni], (i32x16)acc[mi][ni], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < BK / 16; ++ks) {
                bf16x8 av[MI], bv[NI];
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
                    av[mi] = *reinterpret_cast<const bf16x8*>(As + ((size_t)(wm * (BM / 2) + mi * 32 + l32) * LDA + ks * 16 + 8 * h) * 2);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    bv[ni] = *reinterpret_cast<const bf16x8*>(Bs + ((size_t)(wn * (BN / 2) + ni * 32 + l32) * LDA + ks * 16 + 8 * h) * 2);
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc[mi][ni] = (acc_t)__builtin_amdgcn_mfma_f32_32x32x16_bf16(av[mi], bv[ni], (f32x16)acc[mi][ni], 0, 0, 0);
            }
            if constexpr (MODE == 1) if (kt & 1) {
                // end of a 128-column group: tot += s * (acc - z * sum_group(x)), then restart acc
                const int grp = kt >> 1;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const int o = min(n0 + wn * (BN / 2) + ni * 32 + l32, dout - 1);
                    const float s = it.scale[(size_t)o * G + grp], z = it.zero[(size_t)o * G + grp];
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int q = 0; q < 16; ++q) {
                            const int i = min(m0 + wm * (BM / 2) + mi * 32 + 8 * (q >> 2) + 4 * h + (q & 3), R - 1);
                            const float xs = it.xsum[(size_t)i * G + grp];
                            tot[mi][ni][q] = fmaf(s, fmaf(-z, xs, acc[mi][ni][q]), tot[mi][ni][q]);
                            acc[mi][ni][q] = 0;
                        }
                }
            }
        }
        __syncthreads();
    }

    // ---- epilogue ----------------------------------------------------------------------------------
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int o = n0 + wn * (BN / 2) + ni * 32 + l32;
        const int oc = min(o, dout - 1);
        const float wscale = MODE == 1 ? 1.f : it.scale[oc];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int rbase = m0 + wm * (BM / 2) + mi * 32;
            if (DUMP_I32) {
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int i = rbase + 8 * (q >> 2) + 4 * h + (q & 3);
                    if (i < R && o < dout) acc_out[(size_t)i * dout + o] = (int)acc[mi][ni][q];
                }
                continue;
            }
            f32x16 v;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                if (MODE == 2) {
                    const int i = min(rbase + 8 * (q >> 2) + 4 * h + (q & 3), R - 1);
                    v[q] = (float)acc[mi][ni][q] * (it.xscale[i] * wscale);   // one rounding in the product of scales
                } else if (MODE == 1) {
                    v[q] = tot[mi][ni][q];
                } else {
                    v[q] = (float)acc[mi][ni][q] * wscale;
                }
                if (a.flags & ESSA_LORA_ONLY) v[q] = 0.f;
            }
            if (!(a.flags & ESSA_BASE_ONLY)) {
                // rank-r term U_B u_i by MFMA steps of 16 rank columns.  Both operands are stored as a bf16
                // head and tail (x = hi + lo); hi*hi + hi*lo + lo*hi keeps the term at fp32-like accuracy.
                const int ur = min(rbase + l32, R - 1);
                const uint16_t* up = it.U16 + (size_t)ur * 2 * it.rp + 8 * h;
                const uint16_t* bp = it.UB16 + (size_t)oc * 2 * it.rp + 8 * h;
                for (int ks = 0; ks < it.rp / 16; ++ks) {
                    const bf16x8 ua_hi = *reinterpret_cast<const bf16x8*>(up + ks * 16);
                    const bf16x8 ua_lo = *reinterpret_cast<const bf16x8*>(up + it.rp + ks * 16);
                    const bf16x8 ub_hi = *reinterpret_cast<const bf16x8*>(bp + ks * 16);
                    const bf16x8 ub_lo = *reinterpret_cast<const bf16x8*>(bp + it.rp + ks * 16);
                    v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ua_lo, ub_hi, v, 0, 0, 0);
                    v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ua_hi, ub_lo, v, 0, 0, 0);
                    v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ua_hi, ub_hi, v, 0, 0, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int i = rbase + 8 * (q >> 2) + 4 * h + (q & 3);
                if (i < R && o < dout) {
                    if (YBF16) ((uint16_t*)it.Y)[(size_t)i * dout + o] = f32_to_bf16_bits(v[q]);
                    else ((float*)it.Y)[(size_t)i * dout + o] = v[q];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// synthetic reward
// ------------------------------------------------------------------------------------------------
struct reward_args {
    const void* Y[ESSA_MAX_GROUP];
    const float* v[ESSA_MAX_GROUP];
    int d_out[ESSA_MAX_GROUP];
    int n_items, R;
};

// rowdot[i] = sum over the items (in order) of <Y_item[i, :], v_item>.  One workgroup per row; wave w takes the
// items g = w, w+4, ...; 16-byte loads when VEC.  The per-item sums meet in LDS and are added in item order.
template <bool YBF16, bool VEC>
__global__ __launch_bounds__(256) void rowdot_kernel(reward_args a, float* __restrict__ rowdot) {
    __shared__ float dots[ESSA_MAX_GROUP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = blockIdx.x;
    for (int g = wave; g < a.n_items; g += 4) {
        const int d = a.d_out[g];
        const float* __restrict__ v = a.v[g];
        float s = 0.f;
        if (VEC && YBF16) {
            const uint4* y = reinterpret_cast<const uint4*>((const uint16_t*)a.Y[g] + (size_t)row * d);
            for (int c = lane; c < d / 8; c += 64) {
                const uint4 w = y[c];
                const float4 v0 = *reinterpret_cast<const float4*>(v + c * 8), v1 = *reinterpret_cast<const float4*>(v + c * 8 + 4);
                s = fmaf(__uint_as_float(w.x << 16), v0.x, s);
                s = fmaf(__uint_as_float(w.x & 0xffff0000u), v0.y, s);
                s = fmaf(__uint_as_float(w.y << 16), v0.z, s);
                s = fmaf(__uint_as_float(w.y & 0xffff0000u), v0.w, s);
                s = fmaf(__uint_as_float(w.z << 16), v1.x, s);
                s = fmaf(__uint_as_float(w.z & 0xffff0000u), v1.y, s);
                s = fmaf(__uint_as_float(w.w << 16), v1.z, s);
                s = fmaf(__uint_as_float(w.w & 0xffff0000u), v1.w, s);
            }
        } else if (VEC) {
            const float4* y = reinterpret_cast<const float4*>((const float*)a.Y[g] + (size_t)row * d);
            for (int c = lane; c < d / 4; c += 64) {
                const float4 w = y[c], vv = *reinterpret_cast<const float4*>(v + c * 4);
                s = fmaf(w.x, vv.x, s);
                s = fmaf(w.y, vv.y, s);
                s = fmaf(w.z, vv.z, s);
                s = fmaf(w.w, vv.w, s);
            }
        } else {
            for (int o = lane; o < d; o += 64) {
                const float y = YBF16 ? bf16_bits_to_f32(((const uint16_t*)a.Y[g])[(size_t)row * d + o]) : ((const float*)a.Y[g])[(size_t)row * d + o];
                s = fmaf(y, v[o], s);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) dots[g] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float total = 0.f;
        for (int g = 0; g < a.n_items; ++g) total += dots[g];
        rowdot[row] = total;
    }
}

// F[k] += (sum of rowdot over the rows of candidate k) / (their number); fixed-order tree, 0/0 = NaN.
__global__ __launch_bounds__(256) void cand_mean_kernel(const float* __restrict__ rowdot, const int32_t* __restrict__ row2cand, int R,
                                                       float* __restrict__ F) {
    __shared__ double ssum[256];
    __shared__ int scnt[256];
    const int k = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    int cnt = 0;
    for (int i = tid; i < R; i += 256)
        if (row2cand[i] == k) { s += (double)rowdot[i]; ++cnt; }
    ssum[tid] = s;
    scnt[tid] = cnt;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) { ssum[tid] += ssum[tid + st]; scnt[tid] += scnt[tid + st]; }
        __syncthreads();
    }
    if (tid == 0) F[k] += (float)(ssum[0] / (double)scnt[0]);
}

// The generic-path twin of the reward partials that the int8-limb GEMM writes in its epilogue: for every item and every
// block b of 128 output channels, rowpart[b][row] = <Y[row, 128 b ..], v[128 b ..]>.  One wave per row and block; all of it is
// latency, so at few rows every (row, block) gets a wave of its own instead of a share of a row's workgroup (7B-shaped layers
// with int8 weights and reward, whole call: 29.4 -> 17.5 us a layer at 8 rows, 34.2 -> 23.5 at 64).
struct rowblock_args {
    const void* Y[ESSA_MAX_GROUP];
    const float* v[ESSA_MAX_GROUP];
    float* rowpart[ESSA_MAX_GROUP];
    int d_out[ESSA_MAX_GROUP];
    int block_start[ESSA_MAX_GROUP + 1];   // blocks per item (prefix sums)
    int n_items, R;
};
template <bool YBF16>
__global__ __launch_bounds__(256) void rowdot_blocks_kernel(rowblock_args a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = blockIdx.x;
    for (int q = blockIdx.y * 4 + wave; q < a.block_start[ESSA_MAX_GROUP]; q += 4 * gridDim.y) {
        int g = 0;
#pragma unroll
        for (int i = 1; i < ESSA_MAX_GROUP; ++i) g += (i < a.n_items && q >= a.block_start[i]) ? 1 : 0;
        const int d = a.d_out[g], b = q - a.block_start[g];
        const float* __restrict__ v = a.v[g];
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int o = b * 128 + 2 * lane + e;
            if (o < d) {
                const float y = YBF16 ? bf16_bits_to_f32(((const uint16_t*)a.Y[g])[(size_t)row * d + o]) : ((const float*)a.Y[g])[(size_t)row * d + o];
                s = fmaf(y, v[o], s);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) a.rowpart[g][(size_t)b * a.R + row] = s;
    }
}

// rowsum[g][i] = sum of rowpart[b][i] over the blocks b = 16 (g + G q) + sl, q = 0, 1, ..., first along q inside a
// thread, then over the 16 interleaved slices sl in ascending order: a fixed order, whatever the launch timing
__global__ __launch_bounds__(1024) void rowpart_sum_kernel(const float* __restrict__ rowpart, int n_blocks, int R, double* __restrict__ rowsum) {
    __shared__ double part[16][64];
    const int c = threadIdx.x & 63, sl = threadIdx.x >> 6, i = blockIdx.x * 64 + c;
    const int g = blockIdx.y, G = gridDim.y;
    double s = 0.0;
    if (i < R)
        for (int b = 16 * g + sl; b < n_blocks; b += 16 * G) s += (double)rowpart[(size_t)b * R + i];
    part[sl][c] = s;
    __syncthreads();
    if (sl == 0 && i < R) {
        double t = part[0][c];
#pragma unroll
        for (int q = 1; q < 16; ++q) t += part[q][c];
        rowsum[(size_t)g * R + i] = t;
    }
}

// F[k] += (sum over the rows of candidate k, and over the G slices of each row in ascending order) / (number of rows)
// PARTS > 0: the rows' sums are taken here, over at most PARTS blocks (G of them), in the order and with the bits of rowpart_sum_kernel.
// A candidate's rows are one workgroup's work, so latency is what there is to pay: the map is read four places at a time and a row's partials together.
// One after the other, 16 blocks of 32768 rows took 205 us with one candidate, 67 with 4 and 22 with 64 (in two launches 60, 31 and 22); this takes 46, 19
// and 10, and 64 rows of 4 candidates 4.1 -> 3.1 (in two launches 4.5).
template <int PARTS>
__global__ __launch_bounds__(256) void cand_mean_sliced_kernel(const double* __restrict__ rowsum, const float* __restrict__ rowpart, int G,
                                                              const int32_t* __restrict__ row2cand, int R, float* __restrict__ F) {
    constexpr int SCAN = 4;                                // places of the map asked for together
    __shared__ double ssum[256];
    __shared__ int scnt[256];
    const int k = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    int cnt = 0;
    for (uint32_t i0 = tid; i0 < (uint32_t)R; i0 += SCAN * 256) {
        int32_t cand[SCAN];
#pragma unroll
        for (int q = 0; q < SCAN; ++q) cand[q] = row2cand[min(i0 + 256 * q, (uint32_t)R - 1)];
        uint32_t mine = 0;
#pragma unroll
        for (int q = 0; q < SCAN; ++q) mine |= cand[q] == k && i0 + 256 * q < (uint32_t)R ? 1u << q : 0u;
        for (; mine; mine &= mine - 1) {                   // in ascending order
            const uint32_t i = i0 + 256 * __builtin_ctz(mine);
            double t;
            if constexpr (PARTS > 0) {
                float p[PARTS];
#pragma unroll
                for (int g = 0; g < PARTS; ++g) p[g] = (rowpart + (size_t)min(g, G - 1) * R)[i];
                t = 0.0 + (double)p[0];
#pragma unroll
                for (int g = 1; g < PARTS; ++g)
                    if (g < G) t += (double)p[g];
            } else {
                t = rowsum[i];
                for (int g = 1; g < G; ++g) t += rowsum[(size_t)g * R + i];
            }
            s += t;
            ++cnt;
        }
    }
    ssum[tid] = s;
    scnt[tid] = cnt;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) { ssum[tid] += ssum[tid + st]; scnt[tid] += scnt[tid + st]; }
        __syncthreads();
    }
    if (tid == 0) F[k] += (float)(ssum[0] / (double)scnt[0]);
}

}  // namespace

namespace essa_k {

static bool mfma_shape_ok(const fwd_item& it) { return it.d_in % 16 == 0; }

template <int BM, int BN>
static void launch_mfma(hipStream_t st, fwd_args& a, int n_items, int mode, int y_dtype) {
    int total = 0;
    for (int g = 0; g < n_items; ++g) {
        a.tile_start[g] = total;
        total += ((a.it[g].R + BM - 1) / BM) * ((a.it[g].d_out + BN - 1) / BN);
    }
    a.tile_start[n_items] = total;
    const bool yb = y_dtype == ESSA_BF16;
#define ESSA_LAUNCH(MODE_)                                                                                        \
    if (yb) hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, MODE_, true, false>), dim3(total), dim3(256), 0, st, a, nullptr); \
    else hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, MODE_, false, false>), dim3(total), dim3(256), 0, st, a, nullptr)
    if (mode == 0) { ESSA_LAUNCH(0); }
    else if (mode == 1) { ESSA_LAUNCH(1); }
    else { ESSA_LAUNCH(2); }
#undef ESSA_LAUNCH
}

hipError_t forward_group(hipStream_t st, const fwd_item* items, int n_items, int x_dtype, int y_dtype, unsigned flags,
                         hipEvent_t ev_start, hipEvent_t ev_stop) {
    // items are grouped by the kernel family that takes them; within a family they share one launch
    fwd_args a{};
    a.flags = flags;
    int maxR = 0;
    for (int g = 0; g < n_items; ++g) { a.it[g] = items[g]; maxR = items[g].R > maxR ? items[g].R : maxR; }
    a.n_items = n_items;
    const bool xb = x_dtype == ESSA_BF16;

    // prologue (the rank padding is the same for every item of a launch; split by rp)
    for (int rp : {16, 32}) {
        fwd_args p{};
        p.flags = flags;
        int cnt = 0, mr = 0;
        for (int g = 0; g < n_items; ++g)
            if (items[g].rp == rp) { p.it[cnt++] = items[g]; mr = items[g].R > mr ? items[g].R : mr; }
        if (!cnt) continue;
        p.n_items = cnt;
        dim3 grid(mr, cnt);
        if (rp == 16) {
            if (xb) hipLaunchKernelGGL((prologue_kernel<16, true>), grid, dim3(256), 0, st, p);
            else hipLaunchKernelGGL((prologue_kernel<16, false>), grid, dim3(256), 0, st, p);
        } else {
            if (xb) hipLaunchKernelGGL((prologue_kernel<32, true>), grid, dim3(256), 0, st, p);
            else hipLaunchKernelGGL((prologue_kernel<32, false>), grid, dim3(256), 0, st, p);
        }
    }
    if (flags & ESSA_COMPUTE_W8A8) hipLaunchKernelGGL(rowquant_kernel, dim3(maxR, n_items), dim3(256), 0, st, a);

    // split the items between the MFMA family (bf16 activations, d_in % 16 == 0) and the generic one
    fwd_args am{}, ag{};
    am.flags = ag.flags = flags;
    int mode = -1;
    for (int g = 0; g < n_items; ++g) {
        const int want = (flags & ESSA_COMPUTE_W8A8) ? 2 : (items[g].quant == ESSA_QUANT_INT4_G128 ? 1 : 0);
        if (xb && mfma_shape_ok(items[g]) && (mode < 0 || mode == want)) { am.it[am.n_items++] = items[g]; mode = want; }
        else if (xb && mfma_shape_ok(items[g])) {   // a second format in one group: its own launch
            fwd_args one{};
            one.flags = flags;
            one.it[0] = items[g];
            one.n_items = 1;
            launch_mfma<64, 64>(st, one, 1, want, y_dtype);
        } else ag.it[ag.n_items++] = items[g];
    }
    if (am.n_items) {
        if (ev_start) (void)hipEventRecord(ev_start, st);
        long long tiles128 = 0;
        for (int g = 0; g < am.n_items; ++g) tiles128 += (long long)((am.it[g].R + 127) / 128) * ((am.it[g].d_out + 127) / 128);
        if (tiles128 >= 512) launch_mfma<128, 128>(st, am, am.n_items, mode, y_dtype);
        else launch_mfma<64, 64>(st, am, am.n_items, mode, y_dtype);
        if (ev_stop) (void)hipEventRecord(ev_stop, st);
    }
    if (ag.n_items) {
        const bool time_this = !am.n_items;               // a call's one pair of events brackets its first GEMM launch
        if (time_this && ev_start) (void)hipEventRecord(ev_start, st);
        // 32 x 32 tiles, which load each operand half as often, once there is one per CU; below that CUs would stay idle, and there
        // are four times as many 16 x 16 ones (1024 x 1024 at 256 rows, 256 large or 1024 small tiles: 20.7 / 26.7 us)
        auto tiles = [&](const fwd_item& it, int bm) { return ((it.R + bm - 1) / bm) * ((it.d_out + bm - 1) / bm); };
        long long big = 0;
        for (int g = 0; g < ag.n_items; ++g) big += tiles(ag.it[g], 32);
        const int bm = big >= 256 ? 32 : 16;
        int total = 0;
        for (int g = 0; g < ag.n_items; ++g) {
            ag.tile_start[g] = total;
            total += tiles(ag.it[g], bm);
        }
        ag.tile_start[ag.n_items] = total;
        const bool yb = y_dtype == ESSA_BF16;
        auto launch = [&](auto mt) {
            constexpr int MT = decltype(mt)::value;
            if (xb && yb) hipLaunchKernelGGL((gemm_f32_kernel<true, true, MT>), dim3(total), dim3(512), 0, st, ag);
            else if (xb) hipLaunchKernelGGL((gemm_f32_kernel<true, false, MT>), dim3(total), dim3(512), 0, st, ag);
            else if (yb) hipLaunchKernelGGL((gemm_f32_kernel<false, true, MT>), dim3(total), dim3(512), 0, st, ag);
            else hipLaunchKernelGGL((gemm_f32_kernel<false, false, MT>), dim3(total), dim3(512), 0, st, ag);
        };
        if (bm == 32) launch(std::integral_constant<int, 2>{});
        else launch(std::integral_constant<int, 1>{});
        if (time_this && ev_stop) (void)hipEventRecord(ev_stop, st);
    }
    return hipGetLastError();
}

hipError_t w8a8_accumulators(hipStream_t st, const fwd_item& it, int x_dtype, int32_t* acc_out) {
    (void)x_dtype;
    fwd_args a{};
    a.it[0] = it;
    a.n_items = 1;
    hipLaunchKernelGGL(rowquant_kernel, dim3(it.R, 1), dim3(256), 0, st, a);
    a.tile_start[0] = 0;
    const int total = ((it.R + 63) / 64) * ((it.d_out + 63) / 64);
    a.tile_start[1] = total;
    hipLaunchKernelGGL((gemm_mfma_kernel<64, 64, 2, false, true>), dim3(total), dim3(256), 0, st, a, acc_out);
    return hipGetLastError();
}

hipError_t reward_accumulate(hipStream_t st, int n_items, const void* const* Y, const int* d_out, const float* const* v, int y_dtype,
                             int R, const int32_t* row2cand, int K, float* rowdot, float* F) {
    reward_args a{};
    a.n_items = n_items;
    a.R = R;
    bool vec = true;
    const int epv = y_dtype == ESSA_BF16 ? 8 : 4;
    for (int g = 0; g < n_items; ++g) {
        a.Y[g] = Y[g];
        a.v[g] = v[g];
        a.d_out[g] = d_out[g];
        vec = vec && d_out[g] % epv == 0 && ((uintptr_t)Y[g] & 15) == 0 && ((uintptr_t)v[g] & 15) == 0;
    }
    const dim3 grid(R);
    if (y_dtype == ESSA_BF16) {
        if (vec) hipLaunchKernelGGL((rowdot_kernel<true, true>), grid, dim3(256), 0, st, a, rowdot);
        else hipLaunchKernelGGL((rowdot_kernel<true, false>), grid, dim3(256), 0, st, a, rowdot);
    } else {
        if (vec) hipLaunchKernelGGL((rowdot_kernel<false, true>), grid, dim3(256), 0, st, a, rowdot);
        else hipLaunchKernelGGL((rowdot_kernel<false, false>), grid, dim3(256), 0, st, a, rowdot);
    }
    hipLaunchKernelGGL(cand_mean_kernel, dim3(K), dim3(256), 0, st, rowdot, row2cand, R, F);
    return hipGetLastError();
}

hipError_t rowdot_blocks(hipStream_t st, const fwd_item* items, int n_items, int y_dtype) {
    rowblock_args a{};
    int blocks = 0;
    for (int g = 0; g < n_items; ++g) {
        if (!items[g].rv) continue;
        a.Y[a.n_items] = items[g].Y;
        a.v[a.n_items] = items[g].rv;
        a.rowpart[a.n_items] = items[g].rowpart;
        a.d_out[a.n_items] = items[g].d_out;
        a.R = items[g].R;
        a.block_start[a.n_items] = blocks;
        blocks += (items[g].d_out + 127) / 128;
        ++a.n_items;
    }
    if (a.n_items == 0) return hipSuccess;
    for (int g = a.n_items; g <= ESSA_MAX_GROUP; ++g) a.block_start[g] = blocks;
    const dim3 grid(a.R, std::max(1, std::min((blocks + 3) / 4, 2048 / a.R)));     // about one round of workgroups at most
    if (y_dtype == ESSA_BF16) hipLaunchKernelGGL((rowdot_blocks_kernel<true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((rowdot_blocks_kernel<false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

int reward_slices(int n_blocks) { return n_blocks >= 256 ? 16 : (n_blocks + 15) / 16; }

hipError_t reward_finish(hipStream_t st, const float* rowpart, int n_blocks, int R, const int32_t* row2cand, int K,
                         double* rowsum, float* F) {
    // one block a slice of rowpart_sum_kernel: its launch and a gap are more than what reading the partials in the second one adds, at any number of rows and
    // candidates (us, one launch / two; 1 block and 64 rows of 4 candidates 2.8 / 4.4, 16 blocks and 8192 rows of one candidate 13.6 / 17.6)
    if (n_blocks <= 16) {
        const auto kernel = n_blocks == 1 ? cand_mean_sliced_kernel<1> : n_blocks <= 4 ? cand_mean_sliced_kernel<4> : n_blocks <= 8 ? cand_mean_sliced_kernel<8>
                                                                                                                           : cand_mean_sliced_kernel<16>;
        hipLaunchKernelGGL(kernel, dim3(K), dim3(256), 0, st, nullptr, rowpart, n_blocks, row2cand, R, F);
        return hipGetLastError();
    }
    const int G = reward_slices(n_blocks);
    hipLaunchKernelGGL(rowpart_sum_kernel, dim3((R + 63) / 64, G), dim3(1024), 0, st, rowpart, n_blocks, R, rowsum);
    hipLaunchKernelGGL(cand_mean_sliced_kernel<0>, dim3(K), dim3(256), 0, st, rowsum, nullptr, G, row2cand, R, F);
    return hipGetLastError();
}

}  // namespace essa_k
