// Forward for int8 base weights and bf16 activations at prompt-sized row counts: exact bf16 products on the bf16 MFMA.
//
// An int8 weight is exact in bf16, with any power of two, so W_deq x_i = m_o <2^e_o q_o, x_i> needs no quantised activations at all
// when the products run on the bf16 MFMA with fp32 accumulation.  One bf16 pass costs the matrix cores what the two int8 passes of the
// fixed-point limbs cost, and everything around the product gets cheaper: no pass that re-expresses the rows, one
// accumulator per output instead of two (which is what lets a wave own a 128 x 128 patch), and x is read as it is.
// The projection keeps a bf16 copy of its weights in MFMA-operand tiles for this.
//
// Three launches: rank_down (t = V_A^T x, K split over workgroups), rank_finish (u = sB_c * (M (sA_c * t)) as bf16 head and
// tail; the 64-row tiles, and the 4-bit ones of 128 channels, do this themselves), gemm_bf16 (base product, scale, U_B u, output tile, reward partials).
#include "forward_device.h"
#include <hip/hip_ext.h>
#include <algorithm>
#include <utility>

namespace {

struct prefill_item {                      // the fields of one projection that these kernels use
    const uint16_t *X, *W16, *US16, *VAp, *VA3p;
    const float *scale16, *M, *sigmaA, *sigmaB, *rv;
    const int32_t* row2cand;
    void* Y;
    uint16_t* U16;
    float *Tpart, *rowpart;
    long long sigma_stride;
    int R, d_in, d_out, r, rp, n_blocks;
};

struct prefill_args {
    prefill_item it[ESSA_MAX_GROUP];
    int tile_start[ESSA_MAX_GROUP + 1];    // workgroups per item (prefix sums)
    int n_items;
    unsigned flags;
    int ksplit[ESSA_MAX_GROUP];            // rank_down: the item's K is cut in this many parts (at most 8)
    float u_scale;                         // rank_finish leaves u times this power of two
    uint16_t* XS16[ESSA_MAX_GROUP];        // 4-bit weights: where rank_down leaves the sums of x over groups of 128 columns (null: another item of this X does)
    int Gn[ESSA_MAX_GROUP];                // groups rounded up to 32
};

// f(0), f(1), ... f(N - 1) with the index as a compile-time constant: the K loops are one straight-line schedule
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_seq(f, std::make_integer_sequence<int, N>{}); }

// Workgroups go round-robin over the 8 XCDs: XCD x takes a contiguous range of the T tiles.
__device__ __forceinline__ int xcd_contiguous(int b, int T) {
    const int x = b & 7, q = T >> 3, rem = T & 7;
    return x * q + min(x, rem) + (b >> 3);
}

// ------------------------------------------------------------------------------------------------
// t = V_A^T x: one workgroup per item, 128 rows and K part; each of its 4 waves owns 32 rows for all columns.  x tiles
// (128 bytes of each row per step, the 16-byte parts of row r at part ^ ((r >> 1) & 7)) and the operand tiles of V_A
// (bf16 head and tail; THIRD: and what they leave of the fp32 value, so that every product has all of V_A's bits) go through
// LDS, three steps deep.
// ------------------------------------------------------------------------------------------------
constexpr int RD_ROWS = 128;

// SUMS (4-bit weights): the sums of x over groups of 128 columns as well, 2^-7 of them as three bf16 (all of an fp32 number), in
// the operand tiles of the product that wants them, [16 rows][32 groups][part][8 groups][row][group].  They come from
// the x fragments that are in registers anyway, times an operand that is 2^-7 in the column of the group and zero elsewhere; 32 groups
// fill an accumulator.  K parts then end between groups.  An Inf or a NaN reaches every sum of its row, and makes it NaN.
template <int RP, bool THIRD, bool SUMS = false>
__global__ __launch_bounds__(256, THIRD && RP == 32 ? 1 : 2) void rank_down_kernel(prefill_args a) {
    constexpr int NBH = RP / 16, NBV = NBH + (THIRD ? 1 : 0);   // 32-column blocks of [heads | tails], of the third parts
    constexpr int XST = RD_ROWS * 128, VST = 4 * NBV * 1024, ST = XST + VST;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[3 * ST];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    int g = 0;
#pragma unroll
    for (int i = 1; i < ESSA_MAX_GROUP; ++i) g += (i < a.n_items && (int)blockIdx.x >= a.tile_start[i]) ? 1 : 0;
    const prefill_item it = fetch_item(a.it[g]);
    if (it.rp != RP || (it.VA3p != nullptr) != THIRD) return;
    const int ksplit = a.ksplit[g], rel = blockIdx.x - a.tile_start[g], part = rel % ksplit;
    const int m0 = (rel / ksplit) * RD_ROWS;
    const int R = it.R, din = it.d_in;
    const int nk_all = (din + 63) / 64;
    constexpr int UNIT = SUMS ? 2 : 1;
    const int k_lo = (int)((long long)(nk_all / UNIT) * part / ksplit) * UNIT, k_hi = (int)((long long)(nk_all / UNIT) * (part + 1) / ksplit) * UNIT;
    const int ksteps = din / 16;
    const bool sums = SUMS && a.XS16[g] != nullptr;

    const i32x4 xres = buffer_words(it.X + (size_t)m0 * din);
    const i32x4 vres = buffer_words(it.VAp), vres3 = buffer_words(THIRD ? it.VA3p : it.VAp);
    uint32_t xoff[4];
    int xpart[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = wave * 32 + e * 8 + (lane >> 3);
        xpart[e] = (lane & 7) ^ ((row >> 1) & 7);
        xoff[e] = (uint32_t)min(row, R - 1 - m0) * (uint32_t)(din * 2) + xpart[e] * 16;
    }
    auto issue = [&](int kt, int stage) {
        const int k = min(kt, k_hi - 1);
        const uint32_t sx = lds0 + stage * ST + wave * 4096, sv = lds0 + stage * ST + XST;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // columns past the row read the row's last 16 bytes instead: V_A's tiles are zeroed there
            const int over = max(0, k * 64 + xpart[e] * 8 + 8 - din);
            load_lds16(sx + e * 1024, xoff[e] - over * 2, xres, (uint32_t)k * 128);
        }
#pragma unroll
        for (int e = 0; e < NBV; ++e) {
            const int q = wave * NBV + e, ks = min(4 * k + wave, ksteps - 1);
            if (e < NBH) load_lds16(sv + q * 1024, lane * 16, vres, (uint32_t)((ks * NBH + e) * 1024));
            else load_lds16(sv + q * 1024, lane * 16, vres3, (uint32_t)ks * 1024);
        }
    };
    f32x16 acc[NBV];
#pragma unroll
    for (int b = 0; b < NBV; ++b)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[b][q] = 0.f;
    f32x16 acc_s;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc_s[q] = 0.f;
    auto put_sums = [&](int g_end) {                       // the window of 32 groups that g_end - 1 lies in, up to g_end
        const int Gn = a.Gn[g], gr = ((g_end - 1) & ~31) + l32;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int row = m0 + wave * 32 + 8 * (q >> 2) + 4 * h + (q & 3);
            float v = acc_s[q];
            if (row < R && gr >= k_lo / 2 && gr < g_end) {
                const gptr<uint16_t> dst = as_global_w(a.XS16[g]) + ((size_t)(row >> 4) * (Gn >> 5) + (gr >> 5)) * 1536 + (gr >> 3 & 3) * 128 + (row & 15) * 8 + (gr & 7);
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const uint16_t bits = f32_to_bf16_bits(v);
                    dst[512 * e] = bits;
                    v -= bf16_bits_to_f32(bits);
                }
            }
            acc_s[q] = 0.f;
        }
    };
    if (k_lo < k_hi) {
        issue(k_lo, 0);
        issue(k_lo + 1, 1);
        int st = 0;
        const uint32_t xrow = wave * 4096 + l32 * 128, sw = (l32 >> 1) & 7;
        for (int kt = k_lo; kt < k_hi; ++kt) {
            wait_loads_and_meet<4 + NBV>();
            issue(kt + 2, st == 0 ? 2 : st - 1);
            const unsigned char* sx = smem + st * ST;
            const uint32_t one = l32 == ((kt >> 1) & 31) ? 0x3c003c00u : 0u;   // 2^-7 twice
            const bf16x8 pick = __builtin_bit_cast(bf16x8, (u32x4){one, one, one, one});
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool live = 4 * kt + j < ksteps;      // steps past the row multiply by zeros
                const bf16x8 xf = *reinterpret_cast<const bf16x8*>(sx + xrow + (((2 * j + h) ^ sw) * 16));
#pragma unroll
                for (int b = 0; b < NBV; ++b) {
                    u32x4 vf = *reinterpret_cast<const u32x4*>(sx + XST + (j * NBV + b) * 1024 + lane * 16);
                    if (!live) vf = (u32x4){0, 0, 0, 0};
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, __builtin_bit_cast(bf16x8, vf), acc[b], 0, 0, 0);
                }
                if (SUMS && sums) acc_s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, pick, acc_s, 0, 0, 0);
            }
            if (SUMS && sums && (kt & 63) == 63 && kt + 1 < k_hi) put_sums((kt + 1) / 2);
            st = st == 2 ? 0 : st + 1;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // the last part also clears the rest of its eight groups, whose columns no group has touched
        if (SUMS && sums) put_sums(k_hi == nk_all ? (nk_all / 2 + 7) / 8 * 8 : k_hi / 2);
    }
    const gptr<float> out = as_global_w(it.Tpart) + ((size_t)part * R + m0) * RP;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int row = wave * 32 + 8 * (q >> 2) + 4 * h + (q & 3);
        float t = RP == 32 ? acc[NBH - 1][q] : __shfl_xor(acc[0][q], 16, 64);   // rank 16: columns j and 16 + j hold head and tail of V_A's column j
        if (THIRD) t += acc[NBV - 1][q];
        t = acc[0][q] + t;
        if (m0 + row < R && l32 < RP) out[(size_t)row * RP + l32] = t;
    }
}

// u = scale sB_c * (M (sA_c * t)) of ROWS rows from i0 on by 256 threads (scale: a power of two), the K parts of t added in ascending order; put(row, j, head, tail)
// gets every element as two bf16.  With several elements a thread the parts are asked for without a branch between them (26.8 -> 25.5 us,
// 3584 -> 512 at 512 rows); with one, and rows in the thousands, no more of them than there are.  tv: ROWS x (RP + 4) floats of LDS, Ms: RP x (RP + 4).
template <int RP, int ROWS, class ITEM, class F>
__device__ __forceinline__ void rank_rows(const ITEM& it, int ksplit, float scale, int i0, float* tv, float* Ms, F&& put) {
    constexpr int P = RP + 4, EU = ROWS * RP / 256;
    const int tid = threadIdx.x, j = tid % RP, R = it.R;
    const gptr<const float> tp = as_global(it.Tpart);
    float part[EU][8], sa[EU], sb[EU], m[(RP * RP + 255) / 256];
#pragma unroll
    for (int k = 0; k < EU; ++k) {
        const int ic = min(i0 + (tid + 256 * k) / RP, R - 1);
        const size_t at = (size_t)as_global(it.row2cand)[ic] * it.sigma_stride + min(j, it.r - 1);
        sa[k] = as_global(it.sigmaA)[at];
        sb[k] = as_global(it.sigmaB)[at];
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (EU > 1 || s < ksplit) part[k][s] = tp[((size_t)min(s, ksplit - 1) * R + ic) * RP + j];
    }
#pragma unroll
    for (int k = 0; k < (RP * RP + 255) / 256; ++k) m[k] = as_global(it.M)[tid + 256 * k];
#pragma unroll
    for (int k = 0; k < (RP * RP + 255) / 256; ++k) Ms[(tid + 256 * k) / RP * P + j] = m[k];
#pragma unroll
    for (int k = 0; k < EU; ++k) {
        float t = part[k][0];
#pragma unroll
        for (int s = 1; s < 8; ++s)
            if (s < ksplit) t += part[k][s];
        tv[(tid + 256 * k) / RP * P + j] = (j < it.r ? sa[k] : 0.f) * t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < EU; ++k) {
        const int lr = (tid + 256 * k) / RP;
        float u = 0.f;
#pragma unroll
        for (int l = 0; l < RP; ++l) u = fmaf(Ms[j * P + l], tv[lr * P + l], u);
        u *= j < it.r ? sb[k] * scale : 0.f;
        const uint16_t hi = f32_to_bf16_bits(u);
        put(lr, j, hi, f32_to_bf16_bits(u - bf16_bits_to_f32(hi)));
    }
}

// The rows' u for the tiles that do not form it themselves.  Latency and a few bytes per row: one thread per element.
template <int RP>
__global__ __launch_bounds__(256) void rank_finish_kernel(prefill_args a) {
    constexpr int ROWS = 256 / RP, P = RP + 4;
    __shared__ float tv[ROWS * P], Ms[RP * P];
    const prefill_item& it = a.it[blockIdx.y];
    const int i0 = blockIdx.x * ROWS;
    if (it.rp != RP || i0 >= it.R) return;
    rank_rows<RP, ROWS>(it, a.ksplit[blockIdx.y], a.u_scale, i0, tv, Ms, [&](int lr, int j, uint16_t hi, uint16_t lo) {
        if (i0 + lr >= it.R) return;
        const gptr<uint16_t> ur = as_global_w(it.U16) + (size_t)(i0 + lr) * 2 * RP;
        ur[j] = hi;
        ur[RP + j] = lo;
    });
}

// The base term alone: u = 0, and NaN for a row that holds an Inf or a NaN, which makes its whole output row NaN as in the full
// forward (there V_A^T x is non-finite for such a row).  One wave per row.
__global__ __launch_bounds__(256) void rank_none_kernel(prefill_args a) {
    const prefill_item& it = a.it[blockIdx.y];
    const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= it.R) return;
    const gptr<const u32x4> x = as_global(reinterpret_cast<const u32x4*>(it.X + (size_t)i * it.d_in));
    uint32_t top = 0;                                      // sign gone, bf16 bits order like the values; Inf and NaN lie above
    for (int k = lane; k < it.d_in / 8; k += 64) {
        const u32x4 v = x[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) top = max(top, max(v[e] & 0x7fff0000u, v[e] << 17 >> 1));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off, 64));
    if (lane < it.rp) reinterpret_cast<gptr<uint32_t>>(as_global_w(it.U16))[(size_t)i * it.rp + lane] = top < 0x7f800000u ? 0u : 0x7fc07fc0u;
}

// ------------------------------------------------------------------------------------------------
// Base product on the bf16 MFMA.  256 threads = 4 waves in a 2 x 2 grid, tile = 32 NR rows x 64 NB channels, a wave owns a
// patch of 16 NR rows x 32 NB channels (128 x 128 at NR = 8, NB = 4: 256 accumulator registers, one wave per SIMD).  The weights
// are the MFMA's row operand and the activations its column operand, so a lane's accumulators run along the channels and
// the output tile is written 8 or 16 bytes at a time.
//
// K advances in steps of 64, two sub-steps of 32.  Both operands go memory -> LDS directly; weights keep their operand tiles
// (1 KB per 16 channels x 32 columns, read back contiguously), an activation row is 128 bytes with its 16-byte parts swizzled.
// XS activation and WS weight stages; one step (kt):
//   sub-step 0: MFMAs; fragments of sub-step 1; the activations of step kt + XS - 1
//   meet: step kt + 1 is complete in LDS, nobody reads step kt any more
//   sub-step 1: MFMAs; fragments of sub-step 0 of step kt + 1; the weights of step kt + WS
// with the reads and loads spread between the MFMAs (the four or eight MFMAs of a 64-row tile's sub-step are over before an LDS
// read comes back, so they ask for everything in front of them: 28.4 against 29.5 us, 3584 -> 512 at 512 rows, 64 x 128).  The 16 x 16 x 32 form of the MFMA, not 32 x 32 x 16: same rate on
// paper, but the chip runs these kernels at its power limit and the smaller form does more per watt (MFMAs alone, operands
// in registers, all CUs: 2026 against 1714 TFLOP/s; this kernel on 32768 x 5120 x 12288: 3.13 against 3.39 ms).
//
// Measured (256 x 256 tile, 32768 rows, 5120 -> 12288, one MI355X): 3.13 ms with its rank kernels, 1.32 PFLOP/s; the int8-limb
// tile it replaces took 3.99 + 0.65 ms.  A tile of K = 3584 spends 70 us in its loop (135.8 k cycles at 1.94 GHz, 114.7 k of
// them MFMA; the direct-to-LDS loads block the wave's issue for about 15 cycles each), 2 us before and 7 us after it.
// ------------------------------------------------------------------------------------------------
thread_local hipEvent_t tl_pre_start = nullptr, tl_pre_stop = nullptr;   // events of the GEMM launch being timed

// A 64-row tile forms the u of its rows itself, in LDS behind its stages: the rows (head and tail), M, sA t.
constexpr size_t OWN_UROW = 144, OWN_MS = 64 * OWN_UROW, OWN_TV = OWN_MS + 32 * 36 * 4, OWN_BYTES = OWN_TV + 64 * 36 * 4;

template <int NR, int NB, int XS, int WS>
constexpr size_t bf16_smem_bytes(bool ybf16) {
    constexpr size_t BM = 32 * NR, BN = 64 * NB;
    const size_t stages = XS * BM * 128 + WS * BN * 128 + (NR == 2 ? OWN_BYTES : 0);
    const size_t ctile = ybf16 ? BM * (BN * 2 + 16) : BM * ((NB == 1 ? BN : BN / 2) * 4 + 16);
    return stages > ctile ? stages : ctile;
}

// An output tile on its way from LDS to memory: BM rows of BN channels from o0 on.  In two halves: of every 64 channels the first 32, then the others,
// whatever the tile, so that a reward partial is added up in one order.
template <int BM, int BN, int HALVES, bool YBF16, class ITEM>
__device__ __forceinline__ void store_rows(const unsigned char* smem, const ITEM& it, int m0, int o0, int half) {
    constexpr int ESZ = YBF16 ? 2 : 4, EPV = 16 / ESZ, CW = BN / HALVES, CROW = CW * ESZ + 16, PPR = CW / EPV;
    const int tid = threadIdx.x, R = it.R, dout = it.d_out;
    const bool with_reward = it.rv != nullptr;
    const bool vec_ok = (dout % EPV == 0) && ((reinterpret_cast<uintptr_t>(it.Y) & 15) == 0);
    const gptr<unsigned char> Yb = as_global_w(reinterpret_cast<unsigned char*>(it.Y));
    // full rows, 16 bytes per thread; with a reward vector the row's share over each 128-channel block goes to rowpart
    const int piece = tid % PPR, c0 = piece * EPV;
    const int o = o0 + (HALVES == 1 ? c0 : c0 / 32 * 64 + 32 * half + c0 % 32);
    float rvp[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) rvp[e] = (with_reward && o + e < dout) ? as_global(it.rv)[o + e] : 0.f;
    static_assert(256 % PPR == 0 && (BM * PPR) % 256 == 0, "a thread keeps its piece from row to row");
#pragma unroll 8
    for (int p0 = 0; p0 < BM * PPR; p0 += 256) {
        const int row = (p0 + tid) / PPR, i = m0 + row;
        const bool valid = i < R && o < dout;
        const u32x4 val = *reinterpret_cast<const u32x4*>(smem + (size_t)row * CROW + piece * 16);
        if (valid) {
            if (vec_ok && o + EPV <= dout) {
                __builtin_nontemporal_store(val, reinterpret_cast<gptr<u32x4>>(Yb + ((size_t)i * dout + o) * ESZ));
            } else {
                for (int e = 0; e < EPV && o + e < dout; ++e) {
                    if (YBF16) reinterpret_cast<gptr<uint16_t>>(Yb)[(size_t)i * dout + o + e] = (uint16_t)(val[e >> 1] >> (16 * (e & 1)));
                    else reinterpret_cast<gptr<uint32_t>>(Yb)[(size_t)i * dout + o + e] = val[e];
                }
            }
        }
        if (with_reward) {
            constexpr int LPB = 128 / HALVES / EPV;    // lanes per 128-channel block
            float s = 0.f;
            if (valid) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float y = YBF16 ? __uint_as_float((e & 1) ? (val[e >> 1] & 0xffff0000u) : (val[e >> 1] << 16)) : __uint_as_float(val[e]);
                    s = fmaf(o + e < dout ? y : 0.f, rvp[e], s);
                }
            }
#pragma unroll
            for (int off = LPB / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (piece % LPB == 0 && valid) {
                const gptr<float> dst = as_global_w(it.rowpart) + (size_t)(o >> 7) * R + i;
                *dst = half == 0 ? s : *dst + s;       // the second half of the block's channels: this thread wrote the first
            }
        }
    }
}

// acc += A B with the accumulator pinned to the accumulation registers.  Left to choose, the register allocator moves some of
// a 128 x 128 patch's accumulators to and fro inside the loop (48 moves per step: 145 k cycles for a 56-step loop, 135 k
// without; the smaller patches likewise), so the instruction is written out.
__device__ __forceinline__ void mfma_pinned(const bf16x8& A, const bf16x8& B, f32x4& acc) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(A), "v"(B));
}

// block k of a half is the wave's 16-channel block half_block(half, k)
template <int HALVES> __device__ __forceinline__ constexpr int half_block(int half, int k) { return HALVES == 1 ? k : 4 * (k >> 1) + 2 * half + (k & 1); }

template <int NR, int NB, int XS, int WS, bool YBF16>
__global__ __launch_bounds__(256, (bf16_smem_bytes<NR, NB, XS, WS>(true) > 80 * 1024 ? 1 : 2)) void gemm_bf16_kernel(prefill_args a) {
    constexpr int BM = 32 * NR, BN = 64 * NB, NBT = BN / 32;
    constexpr uint32_t XST = BM * 128, WST = BN * 128, W0 = XS * XST, U0 = W0 + WS * WST;
    constexpr bool OWN_U = NR == 2;
    constexpr int NC = 2 * NB;                             // 16-row (NR) and 16-channel (NC) blocks of a wave
    constexpr int NMF = NR * NC, NRD = NR + NC, XL = NR, WL = 2 * NB;     // per wave: MFMAs and fragment reads of a sub-step, loads of a step
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1, l16 = lane & 15, kg = lane >> 4;

    const int b = xcd_contiguous(blockIdx.x, a.tile_start[ESSA_MAX_GROUP]);
    int g = 0;
#pragma unroll
    for (int i = 1; i < ESSA_MAX_GROUP; ++i) g += (i < a.n_items && b >= a.tile_start[i]) ? 1 : 0;
    const prefill_item it = fetch_item(a.it[g]);
    const int R = it.R, dout = it.d_out, din = it.d_in, rp = it.rp;
    const int tiles_m = (R + BM - 1) / BM, tiles_n = (it.n_blocks + NBT - 1) / NBT;
    int tm, tn;
    {   // patches of 4 row tiles x all column tiles, rows fastest: the 32 tiles an XCD runs at a time are about 4 x 8
        const int tile = b - a.tile_start[g], per = 4 * tiles_n, grp = tile / per, rem = tile % per;
        const int rows = min(4, tiles_m - 4 * grp);
        tn = rem / rows;
        tm = 4 * grp + rem % rows;
    }
    const int m0 = tm * BM, nb0 = tn * NBT;
    const int nk = (din + 63) / 64;

    const i32x4 xres = buffer_words(it.X + (size_t)m0 * din);
    const i32x4 wres = buffer_words(it.W16);
    uint32_t xoff[XL];
#pragma unroll
    for (int e = 0; e < XL; ++e) {
        const int row = (wave * XL + e) * 8 + (lane >> 3);
        xoff[e] = (uint32_t)min(row, R - 1 - m0) * (uint32_t)(din * 2) + (((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
    // in the last step of a row that is not a multiple of 64 wide, lanes past its end read its last 16 bytes (the weights
    // are zero there); even and odd loads of a wave differ in their swizzle
    uint32_t back[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int part = (lane & 7) ^ ((((wave * XL + e) * 8 + (lane >> 3)) >> 1) & 7);
        back[e] = (uint32_t)max(0, (nk - 1) * 64 + part * 8 + 8 - din) * 2u;
    }
    uint32_t wsoff[WL];                                    // scalar: where load e's kilobyte starts inside a K step
#pragma unroll
    for (int e = 0; e < WL; ++e) {
        const int q = wave * WL + e;
        wsoff[e] = (uint32_t)(min(nb0 + (q >> 2), it.n_blocks - 1) * 4 + (q & 3)) * 1024u;
    }
    const uint32_t wstep = (uint32_t)it.n_blocks * 4096u, lane16 = lane * 16;
    auto load_x = [&](int e, int kt, uint32_t stage) {
        const int k = min(kt, nk - 1);
        const uint32_t off = xoff[e] - (back[e & 1] & (uint32_t)(k < nk - 1 ? 0 : -1));
        load_lds16(lds0 + stage + (wave * XL + e) * 1024, off, xres, (uint32_t)k * 128u);
    };
    auto load_w = [&](int e, int kt, uint32_t stage) {
        load_lds16(lds0 + stage + (wave * WL + e) * 1024, lane16, wres, (uint32_t)min(kt, nk - 1) * wstep + wsoff[e]);
    };

    f32x4 acc[NC][NR];
#pragma unroll
    for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int m = 0; m < NR; ++m) acc[n][m] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // the steps the loop finds on their way, in the order its own iterations would have asked for them
    static_for<(XS > WS ? XS : WS)>([&](auto tc) {
        constexpr int t = decltype(tc)::value - (XS > WS ? XS : WS), x = t + XS - 1, w = t + WS;
        if constexpr (x >= 0) {
#pragma unroll
            for (int e = 0; e < XL; ++e) load_x(e, x, x * XST);
        }
        if constexpr (w >= 0) {
#pragma unroll
            for (int e = 0; e < WL; ++e) load_w(e, w, W0 + w * WST);
        }
    });
    // loads still on their way when step 0 has to be there, and when step kt + 1 has to be there in the middle of step kt
    constexpr int FIRST = (XS > WS ? (WS - 1) * XL + (WS - 1) * WL : (XS - 2) * XL + (XS - 1) * WL);
    constexpr int AHEAD_X = (XS - 2) * (XL + WL), AHEAD_W = (WS - 1) * XL + (WS - 2) * WL, AHEAD = AHEAD_X < AHEAD_W ? AHEAD_X : AHEAD_W;
    static_assert(FIRST < 64 && AHEAD < 64, "the load counter has six bits");

    if constexpr (OWN_U) {                                 // u of the tile's rows, while the first steps are on their way
        static_assert(bf16_smem_bytes<NR, NB, XS, WS>(true) == U0 + OWN_BYTES && BM * (BN * 2 + 16) <= U0, "behind the stages and the output tile");
        const auto own = [&](int row, int j, uint16_t hi, uint16_t lo) {
            uint16_t* ur = reinterpret_cast<uint16_t*>(smem + U0 + (size_t)row * OWN_UROW);
            ur[j] = hi;
            ur[rp + j] = lo;
        };
        float *tv = reinterpret_cast<float*>(smem + U0 + OWN_TV), *Ms = reinterpret_cast<float*>(smem + U0 + OWN_MS);
        if (a.flags & ESSA_BASE_ONLY) {                    // zeros, or NaN for a row that is not finite
            for (int e = tid; e < BM * rp; e += 256) {
                const gptr<const uint16_t> ur = as_global(it.U16) + (size_t)min(m0 + e / rp, R - 1) * 2 * rp + e % rp;
                own(e / rp, e % rp, ur[0], ur[rp]);
            }
        } else if (rp == 16) rank_rows<16, BM>(it, a.ksplit[g], 1.f, m0, tv, Ms, own);
        else rank_rows<32, BM>(it, a.ksplit[g], 1.f, m0, tv, Ms, own);
    }

    uint32_t xr[2];                                        // this lane's fragment of sub-step j inside an activation stage
#pragma unroll
    for (int j = 0; j < 2; ++j) xr[j] = (wr * 16 * NR + l16) * 128 + (((4 * j + kg) ^ ((l16 >> 1) & 7)) * 16);
    const uint32_t wfr = W0 + wc * NB * 4096 + lane16;
    bf16x8 fx[2][NR], fw[2][NC];
    auto read_frag = [&](int set, int i, uint32_t xs, uint32_t ws, int j) {
        // in the order the MFMAs want them: weights 0, the activations, the other weights
        if (i == 0 || i > NR) fw[set][i == 0 ? 0 : i - NR] = *reinterpret_cast<const bf16x8*>(smem + ws + wfr + (i == 0 ? 0 : i - NR) * 2048 + j * 1024);
        else fx[set][i - 1] = *reinterpret_cast<const bf16x8*>(smem + xs + xr[j] + (i - 1) * 2048);
    };
    wait_loads_and_meet<FIRST>();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NRD; ++i) read_frag(0, i, 0, 0, 0);

    uint32_t x_cur = 0, x_nxt = XST, x_far = (XS - 1) * XST, w_cur = 0, w_nxt = WST;
    for (int kt = 0; kt < nk; ++kt) {
        static_for<2>([&](auto jc) {
            constexpr int j = jc;
            if constexpr (j == 1) {
                __builtin_amdgcn_sched_barrier(0);
                wait_loads_and_meet<AHEAD>();
                __builtin_amdgcn_sched_barrier(0);
            }
            static_for<NMF>([&](auto ic) {
                constexpr int i = ic;
                mfma_pinned(fw[j][i / NR], fx[j][i % NR], acc[i / NR][i % NR]);
                static_for<NRD>([&](auto rc) {
                    constexpr int r = rc;
                    if constexpr ((NR == 2 ? r / 2 : r * NMF / NRD) == i) read_frag(j ^ 1, r, j == 1 ? x_nxt : x_cur, j == 1 ? w_nxt : w_cur, j ^ 1);
                });
                // one load every few MFMAs, never a burst; the weights, which have the shorter way to go, as early as they can
                if constexpr (j == 1) {
                    static_for<WL>([&](auto ec) {
                        constexpr int e = ec;
                        if constexpr (e * NMF / (2 * WL) + 1 == i) load_w(e, kt + WS, W0 + w_cur);
                    });
                } else {
                    static_for<XL>([&](auto ec) {
                        constexpr int e = ec;
                        if constexpr (e * NMF / XL + 1 == i) load_x(e, kt + XS - 1, x_far);
                    });
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        x_far = x_cur;                                     // its last reader was this step
        x_cur = x_nxt;
        x_nxt = x_nxt == (XS - 1) * XST ? 0 : x_nxt + XST;
        w_cur = w_nxt;
        w_nxt = w_nxt == (WS - 1) * WST ? 0 : w_nxt + WST;
    }
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // the pinned MFMAs' results are not tracked by the compiler
    // ---- epilogue: rank-r term, scale, LDS tile, rows out.  Y = m_o (<2^e_o q_o, x> + (U_B / m_o) u): with U_B divided by the channel
    // scale beforehand the rank-r term (bf16 head+tail: lo*hi + hi*lo + hi*hi per 16 rank columns) is three more MFMAs on the
    // accumulators where they are, and one multiplication per output is all the vector ALU has to do.
    // What it reads from memory is asked for in one batch; rank 16 and 32 are separate straight-line code, so that the
    // blocks' MFMA chains, conversions and LDS writes overlap.
    constexpr int HALVES = YBF16 || NB == 1 ? 1 : 2, ESZ = YBF16 ? 2 : 4, CROW = BN / HALVES * ESZ + 16, NH = NC / HALVES;
    // An fp32 tile leaves in two halves (64 channels wide: at once): of every 128 channels 0..31 and 64..95, then the others, on
    // either tile width, so that a reward partial is added up in one order whatever tile its group got.
    auto to_tile = [&](int k, int m, const f32x4& v) {     // k: the block's place in the half
        unsigned char* dst = smem + (size_t)((wr * NR + m) * 16 + l16) * CROW + (size_t)((wc * NH + k) * 16 + 4 * kg) * ESZ;
        if (YBF16) {
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            *reinterpret_cast<bf16x4*>(dst) = __builtin_convertvector(v, bf16x4);
        } else {
            *reinterpret_cast<f32x4*>(dst) = v;
        }
    };
    // the rank columns as the K of 16 x 16 x 32 products: at rank 16 head and tail of U_B sit side by side in one fragment
    // and meet the head of u, then its tail; at rank 32 each is a fragment of its own and lo*lo is left out
    auto finish = [&](auto ks_count, auto half_index) {
        constexpr int KS = decltype(ks_count)::value, HALF = decltype(half_index)::value;
        bf16x8 uu[NR][2], ub[2][KS];                       // head and tail of u; U_B and scales one block ahead
        f32x4 sc[2];
        auto ask = [&](int k) {
            const int n = half_block<HALVES>(HALF, k);
            const int o = min((nb0 + wc * NB) * 32 + n * 16 + l16, dout - 1);
            const gptr<const uint16_t> bp = as_global(it.US16) + (size_t)o * (32 * KS) + 8 * kg;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ub[k & 1][ks] = *reinterpret_cast<gptr<const bf16x8>>(bp + 32 * ks);
            // the slack behind the array covers a last block that is not full
            sc[k & 1] = *as_global(reinterpret_cast<const f32x4*>(it.scale16 + min((nb0 + wc * NB) * 32 + n * 16, it.n_blocks * 32 - 16) + 4 * kg));
        };
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const int row = (wr * NR + m) * 16 + l16, at = 8 * (KS == 1 ? kg & 1 : kg);
            const gptr<const uint16_t> up = as_global(it.U16) + (size_t)min(m0 + row, R - 1) * (32 * KS) + at;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if constexpr (OWN_U) uu[m][e] = *reinterpret_cast<const bf16x8*>(smem + U0 + (size_t)row * OWN_UROW + 2 * (at + e * 16 * KS));
                else uu[m][e] = *reinterpret_cast<gptr<const bf16x8>>(up + e * 16 * KS);
            }
        }
        ask(0);
        if constexpr (HALF == 0) wait_loads_and_meet<0>();   // the stages become the output tile
#pragma unroll
        for (int k = 0; k < NH; ++k) {
            const int n = half_block<HALVES>(HALF, k);
            __builtin_amdgcn_sched_barrier(0);
            if (k + 1 < NH) ask(k + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NR; ++m) {
                acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[k & 1][0], uu[m][1], acc[n][m], 0, 0, 0);
                if (KS == 2) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[k & 1][KS - 1], uu[m][0], acc[n][m], 0, 0, 0);
                acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[k & 1][0], uu[m][0], acc[n][m], 0, 0, 0);
            }
#pragma unroll
            for (int m = 0; m < NR; ++m) to_tile(k, m, acc[n][m] * sc[k & 1]);
        }
    };
    if (a.flags & ESSA_LORA_ONLY) {
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int m = 0; m < NR; ++m) acc[n][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    static_for<HALVES>([&](auto half_c) {
        constexpr int half = half_c;
        if (rp == 16) finish(std::integral_constant<int, 1>{}, half_c);
        else finish(std::integral_constant<int, 2>{}, half_c);
        __syncthreads();
        store_rows<BM, BN, HALVES, YBF16>(smem, it, m0, nb0 * 32, half);
        if constexpr (half + 1 < HALVES) __syncthreads();
    });
}

template <int NR, int NB, int XS, int WS, bool YBF16>
hipError_t launch_bf16(hipStream_t st, prefill_args& a) {
    int total = 0;
    for (int g = 0; g < a.n_items; ++g) {
        a.tile_start[g] = total;
        total += ((a.it[g].R + 32 * NR - 1) / (32 * NR)) * ((a.it[g].n_blocks + 2 * NB - 1) / (2 * NB));
    }
    for (int g = a.n_items; g <= ESSA_MAX_GROUP; ++g) a.tile_start[g] = total;
    constexpr size_t smem = bf16_smem_bytes<NR, NB, XS, WS>(YBF16);
    static_assert(smem <= 160 * 1024, "tile does not fit the LDS of a CU");
    auto kern = gemm_bf16_kernel<NR, NB, XS, WS, YBF16>;
    static bool attr_done = false;   // one flag per instantiation
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
    if (tl_pre_start) hipExtLaunchKernelGGL(kern, dim3(total), dim3(256), (uint32_t)smem, st, tl_pre_start, tl_pre_stop, 0, a);
    else hipLaunchKernelGGL(kern, dim3(total), dim3(256), smem, st, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Base product for 4-bit weights on the bf16 MFMA, activations as they are.  With q the 4-bit code, (16 + q) 2^-12 is a bf16
// number whose bits are a constant with q put into its mantissa: one shift and one and-or make two weights.  A group's sum
// g = <(16 + q) 2^-12, x> over its 128 columns meets its scale in one fp32 FMA, and the zero points and the 16 come back as a product
// over the groups, - s (z + 16) 2^-12 times the group's sum of x (rank_down's).  Both as three bf16, the six products that reach 2^-24 of
// it: rows whose entries have a mean make it many times larger than the output (head and tail alone: 8e-5 rms for 1 + N(0, 1), 7e-5 for |N(0, 1)|).
//   Y = 2^12 (sum_g s_g g_g - sum_g s_g (z_g + 16) 2^-12 X_g + U_B 2^-12 u)
// The 2^-12 keeps every partial sum below the output that it grows into: nothing overflows that the output does not.
//
// What bounds it is vector-instruction issue next to the MFMAs: per 16 x 16 x 32 product one FMA, and 7 / NR instructions of
// unpacking, since a wave of 16 NR rows x 64 channels unpacks a fragment once for NR products (the int8-limb tile needs 16 per pair
// of its MFMAs).  256 threads = 4 waves side by side, 16 NR rows x 256 channels (128 for calls of few tiles), so no
// weight is unpacked twice in a workgroup; two workgroups a CU, whose unpacking, MFMAs and waits overlap.
//
// A step is one group.  Activations (D stages: rows of 128 bytes per half group, 16-byte parts swizzled as above), weights (D - 1,
// a wave's own: a place is free once its codes are in registers) and scales go memory -> LDS directly, D - 1 steps ahead.
//
// Measured (6000 rows, q, k, v, o of 3584 columns): 260 us, 1.37 PFLOP/s at 2.0 GHz, against 376 us on the int8-limb tiles; with the launches
// around it 298 against 456.  MFMAs are 55 % of its cycles; in copies without the unpacking and folding, or without the loads, the cycles fall by an
// eighth or less and the clock with them: the chip is at its power limit here as in the kernel above.
// ------------------------------------------------------------------------------------------------
struct q4_item {
    const uint16_t *X, *UB16, *U16, *SZn, *XS16;
    const uint8_t* Wn;
    const float *St, *rv;
    void* Y;
    float* rowpart;
    int R, d_in, d_out, rp, n_blocks, Gn;
};
struct q4_rank {                           // what tiles that form u themselves want beside it
    const float *Tpart, *M, *sigmaA, *sigmaB;
    const int32_t* row2cand;
    long long sigma_stride;
    int R, r, rp, ksplit;
};
struct q4_args {
    q4_item it[ESSA_MAX_GROUP];
    q4_rank rk[ESSA_MAX_GROUP];
    int tile_start[ESSA_MAX_GROUP + 1];
    int n_items;
};

template <int NR, int NC>
constexpr size_t q4_own_bytes() { return NC == 2 ? 16 * NR * OWN_UROW + 32 * 36 * 4 + 16 * NR * 36 * 4 : 0; }

template <int NR, int NC, int D>
constexpr size_t q4_smem_bytes() {
    constexpr size_t BM = 16 * NR, stages = D * BM * 256 + (D - 1) * NC * 4096 + D * 1024, ctile = BM * (NC * 128 + 16);
    return (stages > ctile ? stages : ctile) + q4_own_bytes<NR, NC>();
}

template <int NR, int NC, int D, bool YBF16>
__global__ __launch_bounds__(256, 2) void gemm_q4_exact_kernel(q4_args a) {
    constexpr int BM = 16 * NR, BN = 64 * NC, NBT = BN / 32, PATCH = 8, LOADS = NR + NC + 1;   // LOADS: of a wave and step
    constexpr uint32_t XST = BM * 256, XH = BM * 128, WST = NC * 4096, W0 = D * XST, S0 = W0 + (D - 1) * WST;
    static_assert(NR >= 2 && (NC == 2 || NC == 4) && (NR > 3 || NR + 1 <= 4 * (NR - 1)), "every load of a step has its place in row blocks 1 and 2");
    static_assert((D - 2) * LOADS < 64, "the load counter has six bits");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;

    const int b = xcd_contiguous(blockIdx.x, a.tile_start[ESSA_MAX_GROUP]);
    int gi = 0;
#pragma unroll
    for (int i = 1; i < ESSA_MAX_GROUP; ++i) gi += (i < a.n_items && b >= a.tile_start[i]) ? 1 : 0;
    const q4_item it = fetch_item(a.it[gi]);
    const int R = it.R, dout = it.d_out, din = it.d_in, rp = it.rp, ng = din / 128, nb16 = it.n_blocks * 2;
    const int tiles_m = (R + BM - 1) / BM, tiles_n = (it.n_blocks + NBT - 1) / NBT;
    int tm, tn;
    {   // patches of 8 row tiles x all column tiles, rows fastest: the 64 tiles an XCD runs at a time are about 8 x 8
        const int tile = b - a.tile_start[gi], per = PATCH * tiles_n, grp = tile / per, rem = tile % per;
        const int rows = min(PATCH, tiles_m - PATCH * grp);
        tn = rem / rows;
        tm = PATCH * grp + rem % rows;
    }
    const int m0 = tm * BM, nb0 = tn * NBT;

    const i32x4 xres = buffer_words(it.X + (size_t)m0 * din), wres = buffer_words(it.Wn), sres = buffer_words(it.St);
    // load q = wave NR + e of the 4 NR of a step: half group q / (2 NR), 8 rows; its swizzle hangs on the parity of q
    const uint32_t xlim = essa_k::last_row_offset(R, m0, BM, din * 2), xrow = (uint32_t)(lane >> 3) * (uint32_t)(din * 2);
    uint32_t xpart[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) xpart[e] = ((lane & 7) ^ ((4 * (wave * NR + e) + (lane >> 4)) & 7)) * 16;
    const uint32_t lane16 = lane * 16;
    const uint32_t soff = (uint32_t)min(nb0 * 32 + wave * (16 * NC) + lane, it.n_blocks * 32 - 1) * 4u, sstep = (uint32_t)it.n_blocks * 128u;
    uint32_t woff[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) woff[n] = (uint32_t)min(nb0 * 2 + wave * NC + n, nb16 - 1) * 1024u;
    auto load_x = [&](int e, int g, uint32_t stage) {
        const int q = wave * NR + e, half = q >= 2 * NR ? 1 : 0;
        load_lds16(lds0 + stage + q * 1024, min(xrow + (uint32_t)(q - half * 2 * NR) * 8u * (uint32_t)(din * 2), xlim) + xpart[e & 1], xres, (uint32_t)(g * 256 + half * 128));
    };
    auto load_w = [&](int n, int g, uint32_t stage) { load_lds16(lds0 + W0 + stage + (wave * NC + n) * 1024, lane16, wres, (uint32_t)g * (uint32_t)nb16 * 1024u + woff[n]); };
    auto load_s = [&](int g, uint32_t stage) { load_lds4(lds0 + S0 + stage + wave * 256, soff, sres, (uint32_t)g * sstep); };
    // the totals start with the zero points' and the rank-r term, whose operands are asked for in front of the first step's
    f32x4 tot[NC][NR];
#pragma unroll
    for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int m = 0; m < NR; ++m) tot[n][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
    {
        const int ch0 = nb0 * 32 + wave * (16 * NC) + l16, nc = it.Gn / 32;
        // 32 groups, a place for every part, so that all are on their way before the steps' first loads: with the second and the third part in one place
        // the second is another round trip a tile (q, k, v, o, two places / three: 1152 columns, 15442 rows 183.8 / 179.3 us; 3584, 6000 rows 326 / 324)
        bf16x8 z[3][NC], xs[3][NR];
        const rsrc_t zres = make_rsrc(it.SZn), sumres = make_rsrc(it.XS16 + (size_t)(m0 / 16) * nc * 1536);
        uint32_t zoff[NC], sumoff[NR];                     // operand tiles of 16 channels or rows and 32 groups: a kilobyte per part
#pragma unroll
        for (int n = 0; n < NC; ++n) zoff[n] = (uint32_t)min(nb0 * 2 + wave * NC + n, nb16 - 1) * (uint32_t)nc * 3072u;
#pragma unroll
        for (int m = 0; m < NR; ++m) sumoff[m] = (uint32_t)min(m, (R - 1 - m0) / 16) * (uint32_t)nc * 3072u;
        auto ask_z = [&](int c, int p) {
#pragma unroll
            for (int n = 0; n < NC; ++n) z[p][n] = __builtin_bit_cast(bf16x8, load16(zres, lane16, zoff[n] + c * 3072 + p * 1024));
        };
        auto ask_x = [&](int c, int p) {                   // eights past the last group: beyond the descriptor, zeros
            const uint32_t xlane = c * 32 + kg * 8 < ng ? lane16 : 0x80000000u;
#pragma unroll
            for (int m = 0; m < NR; ++m) xs[p][m] = __builtin_bit_cast(bf16x8, load16(sumres, xlane, sumoff[m] + c * 3072 + p * 1024));
        };
        auto multiply = [&](int pz, int px) {
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int m = 0; m < NR; ++m) tot[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(z[pz][n], xs[px][m], tot[n][m], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto chunk = [&](int c, auto last) {               // no branch around a load: the compiler has to count them
            multiply(0, 2);
            if constexpr (!last) ask_x(c + 1, 2);
            multiply(2, 0);
            if constexpr (!last) ask_z(c + 1, 2);
            multiply(0, 0);
            multiply(0, 1);
            if constexpr (!last) ask_z(c + 1, 0);
            multiply(1, 0);
            if constexpr (!last) ask_x(c + 1, 0);
            multiply(1, 1);
            if constexpr (!last) ask_x(c + 1, 1), ask_z(c + 1, 1);
            __builtin_amdgcn_sched_barrier(0);
        };
        ask_z(0, 0), ask_x(0, 2), ask_z(0, 2), ask_x(0, 0), ask_x(0, 1), ask_z(0, 1);
        __builtin_amdgcn_sched_barrier(0);
        static_for<D - 1>([&](auto tc) {
            constexpr int t = tc;
#pragma unroll
            for (int n = 0; n < NC; ++n) load_w(n, min(t, ng - 1), t * WST);
#pragma unroll
            for (int e = 0; e < NR; ++e) load_x(e, min(t, ng - 1), t * XST);
            load_s(min(t, ng - 1), t * 1024);
        });
        for (int c = 0; c < nc - 1; ++c) chunk(c, std::false_type{});
        chunk(nc - 1, std::true_type{});
        // a tile of 128 channels forms u itself, in LDS behind the stages: the rows (head and tail), M, sA t
        constexpr bool OWN_U = NC == 2;
        constexpr size_t U0 = q4_smem_bytes<NR, NC, D>() - q4_own_bytes<NR, NC>();
        static_assert(!OWN_U || U0 >= S0 + D * 1024, "behind the stages");
        if constexpr (OWN_U) {
            const auto own = [&](int row, int j, uint16_t hi, uint16_t lo) {
                uint16_t* ur = reinterpret_cast<uint16_t*>(smem + U0 + (size_t)row * OWN_UROW);
                ur[j] = hi;
                ur[rp + j] = lo;
            };
            float *Ms = reinterpret_cast<float*>(smem + U0 + BM * OWN_UROW), *tv = Ms + 32 * 36;
            const q4_rank rk = fetch_item(a.rk[gi]);
            if (rp == 16) rank_rows<16, BM>(rk, rk.ksplit, 0x1p-12f, m0, tv, Ms, own);
            else rank_rows<32, BM>(rk, rk.ksplit, 0x1p-12f, m0, tv, Ms, own);
            __syncthreads();
        }
        auto rank_term = [&](auto ks_count) {              // as in the kernel above, for u 2^-12
            constexpr int KS = decltype(ks_count)::value;
            bf16x8 ub[NC][KS], uu[NR][2];
            const rsrc_t bres = make_rsrc(it.UB16), ures = make_rsrc(it.U16 + (size_t)m0 * (32 * KS));
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) ub[n][ks] = __builtin_bit_cast(bf16x8, load16(bres, (uint32_t)min(ch0 + n * 16, dout - 1) * (64 * KS) + 16 * kg, 64 * ks));
#pragma unroll
            for (int m = 0; m < NR; ++m)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int at = 16 * (KS == 1 ? kg & 1 : kg) + e * 32 * KS;
                    if constexpr (OWN_U) uu[m][e] = *reinterpret_cast<const bf16x8*>(smem + U0 + (size_t)(m * 16 + l16) * OWN_UROW + at);
                    else uu[m][e] = __builtin_bit_cast(bf16x8, load16(ures, (uint32_t)min(m * 16 + l16, R - 1 - m0) * (64 * KS) + at, 0));
                }
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    tot[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[n][0], uu[m][1], tot[n][m], 0, 0, 0);
                    if (KS == 2) tot[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[n][KS - 1], uu[m][0], tot[n][m], 0, 0, 0);
                    tot[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[n][0], uu[m][0], tot[n][m], 0, 0, 0);
                }
        };
        if (rp == 16) rank_term(std::integral_constant<int, 1>{});
        else rank_term(std::integral_constant<int, 2>{});
    }

    uint32_t xr[2];                                        // this lane's fragment of the even and odd 32 columns of a half group
#pragma unroll
    for (int j = 0; j < 2; ++j) xr[j] = l16 * 128 + (((4 * j + kg) ^ ((l16 >> 1) & 7)) * 16);
    const uint32_t mask = 0x00780078u;
    uint32_t tag = 0x3b803b80u;
    asm("" : "+v"(tag));                                   // in a vector register: one instruction takes one constant from elsewhere
    uint32_t cur = 0, far = (D - 1) * XST, w_cur = 0, s_cur = 0, s_far = (D - 1) * 1024;
    for (int g = 0; g < ng; ++g) {
        wait_loads_and_meet<(D - 2) * LOADS>();            // step g is in LDS, nobody reads step g - 1 any more
        u32x4 raw[NC];
        f32x4 sc[NC], sum[2][NC];
        bf16x8 xa[4], w[NC][4];
        auto frag = [&](int m, int k) { return *reinterpret_cast<const bf16x8*>(smem + cur + (k >> 1) * XH + m * 2048 + xr[k & 1]); };
#pragma unroll
        for (int n = 0; n < NC; ++n) raw[n] = *reinterpret_cast<const u32x4*>(smem + W0 + w_cur + (wave * NC + n) * 1024 + lane16);
#pragma unroll
        for (int k = 0; k < 4; ++k) xa[k] = frag(0, k);
#pragma unroll
        for (int n = 0; n < NC; ++n) sc[n] = *reinterpret_cast<const f32x4*>(smem + S0 + s_cur + (wave * 64 + n * 16 + 4 * kg) * 4);
        const int gn = min(g + D - 1, ng - 1);             // past the end the last step is fetched again, and never read
        auto fold = [&](int m, int i) {                    // element i of row block m's group sums, times its scale
            tot[i >> 2][m][i & 3] = fmaf(sc[i >> 2][i & 3], sum[m & 1][i >> 2][i & 3], tot[i >> 2][m][i & 3]);
        };
        __builtin_amdgcn_sched_barrier(0);
        static_for<NR>([&](auto mc) {
            constexpr int m = mc;
            static_for<4>([&](auto kc) {
                constexpr int k = kc;
                static_for<NC>([&](auto nc) {
                    constexpr int n = nc, at = k * NC + n;
                    if constexpr (m == 0) {
                        // eight codes: pair i of the fragment has its codes at bits 3 + 4 i and 19 + 4 i (mod 32)
                        const uint32_t r = raw[n][k];
                        const u32x4 f = {(r & mask) | tag, ((r >> 4) & mask) | tag, ((r >> 8) & mask) | tag, (__builtin_amdgcn_alignbit(r, r, 12) & mask) | tag};
                        w[n][k] = __builtin_bit_cast(bf16x8, f);
                    }
                    const f32x4 c = k == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : sum[m & 1][n];
                    sum[m & 1][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[n][k], xa[k], c, 0, 0, 0);
                    if constexpr (m > 0) fold(m - 1, at);
                    // the codes are all in registers by row block 1: their place is free
                    if constexpr (m == 1 && at % 4 == 1) load_w(at / 4, gn, w_cur);
                    if constexpr (m >= 1 && m <= 2 && n == NC - 1) {
                        constexpr int e = (m - 1) * 4 + k;
                        if constexpr (e < NR) load_x(e, gn, far);
                        if constexpr (e == NR) load_s(gn, s_far);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (m + 1 < NR) xa[k] = frag(m + 1, k);
            });
        });
#pragma unroll
        for (int i = 0; i < 4 * NC; ++i) fold(NR - 1, i);
        far = cur;                                         // its last reader was this step
        cur = cur == (D - 1) * XST ? 0 : cur + XST;
        s_far = s_cur;
        s_cur = s_cur == (D - 1) * 1024 ? 0 : s_cur + 1024;
        w_cur = w_cur == (D - 2) * WST ? 0 : w_cur + WST;
    }
    wait_loads_and_meet<0>();                              // the stages become the output tile
    constexpr int HALVES = YBF16 ? 1 : 2, ESZ = YBF16 ? 2 : 4, CROW = BN / HALVES * ESZ + 16;
    static_for<HALVES>([&](auto half_c) {
        constexpr int half = half_c;
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int m = 0; m < NR; ++m) {
                const f32x4 v = tot[n][m] * 0x1p12f;
                const int c = (wave * NC + n) * 16 + 4 * kg;   // of the tile; of the half it lies in: every second 32 left out
                if (YBF16) {
                    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
                    *reinterpret_cast<bf16x4*>(smem + (size_t)(m * 16 + l16) * CROW + c * ESZ) = __builtin_convertvector(v, bf16x4);
                } else if ((c >> 5 & 1) == half) {
                    *reinterpret_cast<f32x4*>(smem + (size_t)(m * 16 + l16) * CROW + (c / 64 * 32 + c % 32) * ESZ) = v;
                }
            }
        __syncthreads();
        store_rows<BM, BN, HALVES, YBF16>(smem, it, m0, nb0 * 32, half);
        if constexpr (half + 1 < HALVES) __syncthreads();
    });
}

template <int NR, int NC, int D, bool YBF16>
hipError_t launch_q4(hipStream_t st, q4_args& a) {
    int total = 0;
    for (int g = 0; g < a.n_items; ++g) {
        a.tile_start[g] = total;
        total += ((a.it[g].R + 16 * NR - 1) / (16 * NR)) * ((a.it[g].n_blocks + 2 * NC - 1) / (2 * NC));
    }
    for (int g = a.n_items; g <= ESSA_MAX_GROUP; ++g) a.tile_start[g] = total;
    constexpr size_t smem = q4_smem_bytes<NR, NC, D>();
    static_assert(smem <= 160 * 1024, "tile does not fit the LDS of a CU");
    auto kern = gemm_q4_exact_kernel<NR, NC, D, YBF16>;
    static bool attr_done = false;   // one flag per instantiation
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
    if (tl_pre_start) hipExtLaunchKernelGGL(kern, dim3(total), dim3(256), (uint32_t)smem, st, tl_pre_start, tl_pre_stop, 0, a);
    else hipLaunchKernelGGL(kern, dim3(total), dim3(256), smem, st, a);
    return hipGetLastError();
}

// What a group takes on one kind of tile.  Tiles go to the 256 CUs in rounds (two at a time on a CU where slots is 512): what does not depend on K,
// per call and per round, plus (K steps) x (time of a step) for every full round and the last one, which runs faster the
// emptier it is (one CU in two or fewer: no faster than that; the clock falls as the chip fills), plus shares of the weights' way from HBM and of
// the outputs' way there:
//   us = call + rounds * round + steps * (full rounds * hi + last round's lo .. hi) + per_wmb * (MB of weights) + per_ymb * (MB of outputs)
struct tile_cost { int rows, channels, slots; double call, round, lo, mid, hi, per_wmb, per_ymb; };
template <class ITEM>
long long count_tiles(const tile_cost& c, const ITEM* items, int n_items) {
    long long t = 0;
    for (int g = 0; g < n_items; ++g) t += (long long)((items[g].R + c.rows - 1) / c.rows) * ((items[g].n_blocks * 32 + c.channels - 1) / c.channels);
    return t;
}
double tile_us(const tile_cost& c, long long tiles, int steps, double w_mb, double y_mb) {
    const long long full = tiles / c.slots, rest = tiles % c.slots;
    const double over = std::max(0.0, 2.0 * rest / c.slots - 1.0);   // how far the last round is beyond half full
    double last = 0;
    // two workgroups a CU: up to half full a CU has one, beyond that some have two
    if (rest) last = c.slots == 512 ? (over == 0 ? c.lo : c.mid + (c.hi - c.mid) * over) : c.lo + (c.hi - c.lo) * over * over;
    return c.call + c.round * (full + (rest ? 1 : 0)) + steps * (full * c.hi + last) + c.per_wmb * w_mb + c.per_ymb * y_mb;
}

// Which tile takes a group of 4-bit projections: the formula fitted to 331 groups and single projections of 512 to 8192 columns, every tile forced;
// 0.2 % on average from the fastest tile, 5 % at worst.  The tallest tile unpacks least per product, and a last round that is not full costs what
// it costs whatever its tiles; 128 channels are for calls of few tiles, a projection alone above all, and form u themselves (2 to 4 us of a call,
// even where there are several rounds); they have to be 2 % ahead, which is what the formula is off by.  All run two to a CU.  us by tile (int8-limb tiles):
//                               64 x 256   80 x 256   96 x 256   32 x 128   48 x 128   64 x 128
//   q, k, v, o  8192   512   rows   210        156        164        214        199        218     (186)
//               8192  1187   rows   341        335        314        480        406        393     (408)
//               3584   640   rows    61         51         56         65         62         66     (71)
//               3584  6000   rows   333        324        308        488        424        395     (442)
//   q alone     8192   257   rows    85         91        101         85         66         73     (80)
//               3584   512   rows    47         51         53         33         37         38     (36)
//   k alone     8192   512   rows    87         91         99         48         52         67     (60)
//               3584  1024   rows    47         49         54         28         30         37     (38)
//               1024  1024   rows    25         27         28         17         18         19     (18)
enum q4_tile { Q4_64x256, Q4_80x256, Q4_96x256, Q4_32x128, Q4_48x128, Q4_64x128 };
constexpr tile_cost Q4_COST[] = {{64, 256, 512, 16.6, 1.5, 0.913, 1.389, 1.435, 0.18, 0.46}, {80, 256, 512, 17.0, 1.6, 0.972, 1.612, 1.677, 0.19, 0.45},
                                 {96, 256, 512, 17.5, 1.9, 1.078, 1.830, 1.922, 0.20, 0.48}, {32, 128, 512, 12.4, 2.2, 0.358, 0.518, 0.543, 0.22, 0.62},
                                 {48, 128, 512, 12.7, 2.3, 0.407, 0.651, 0.684, 0.20, 0.54}, {64, 128, 512, 12.8, 1.9, 0.646, 0.743, 0.851, 0.24, 0.60}};
q4_tile pick_q4_tile(const q4_args& a, int y_size) {
    int best = 0, ng = 1;
    double best_us = 0, w_mb = 0, y_mb = 0;
    for (int g = 0; g < a.n_items; ++g) {
        ng = std::max(ng, a.it[g].d_in / 128);
        w_mb += 0.5e-6 * a.it[g].d_in * a.it[g].d_out;
        y_mb += 1e-6 * y_size * a.it[g].R * a.it[g].d_out;
    }
    for (int i = 0; i < (int)(sizeof(Q4_COST) / sizeof(Q4_COST[0])); ++i) {
        const double us = tile_us(Q4_COST[i], count_tiles(Q4_COST[i], a.it, a.n_items), ng, w_mb, y_mb) * (i >= Q4_32x128 ? 1.02 : 1.0);
        if (i == 0 || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    return (q4_tile)best;
}

// Which tile takes a group of int8 projections.  Fitted to whole calls, each with every tile forced: 284 groups and single projections of 256 to
// 14336 columns, k and v from an eighth of q to as wide, 1 to 24000 rows, bf16 and fp32 outputs, weights from HBM.  The tile it names is within 0.3 %
// of the fastest on average there, 10 % at worst.  Another tile than 256 x 256 has to be 2 % ahead: it is what runs best for long, and the
// formula is a few per cent off.  Two rounds of a low tile often beat
// one and a bit of the high one, or a round that is two thirds full (q, k, v, o of 3584 columns, k and v with 512 channels, us):
//   rows       256 x 256   224 x 256   192 x 256   160 x 256   256 x 128   160 x 128   128 x 128, two a CU   128 x 128, five stages
//     300            81          77          75          67          56          51          57                  42
//     700            81          77          74          64          58          78          65                  73
//    1187            84          83          79          76         106          86         100                 102
//    1536            91          88          85         121         111         116         108                 116
//    2560           172         159         151         144         163         171         167                 183
//    4096           193         236         219         241         222         262         229                 268
//   20000           987        1003        1023        1049        1124        1239        1141                1334
// and with few rows one round of the lowest tiles (8192 columns, 8 rows: 64 x 128 67 us, 128 x 128 74; 3584 columns, 200 rows 35 and 45).
// The 64-row tiles form u themselves (the launch of rank_finish and its wait that they save are 3 us); 64 x 64 is half of a reward
// partial wide, so it is for calls without reward vectors (3584 -> 512 at 512 rows 21 us, 64 x 128 25.6).  Both are for calls that they finish
// in one round; a CU's load path takes 24 KB of operands in 0.3 us, and weights straight into registers took as long.
enum bf16_tile { TILE_256x256, TILE_224x256, TILE_192x256, TILE_160x256, TILE_256x128, TILE_160x128, TILE_128x128, TILE_128x128_DEEP, TILE_64x128, TILE_64x64 };
constexpr tile_cost TILE_COST[] = {
    {256, 256, 256, 9.2, 8.4, 0.903, 0, 1.016, 0.071, 0.58}, {224, 256, 256, 10.6, 6.6, 0.834, 0, 0.918, 0.080, 0.58},
    {192, 256, 256, 9.5, 6.4, 0.775, 0, 0.805, 0.093, 0.57}, {160, 256, 256, 10.2, 5.4, 0.661, 0, 0.721, 0.074, 0.58},
    {256, 128, 256, 9.8, 5.0, 0.560, 0, 0.621, 0.080, 0.57}, {160, 128, 256, 10.3, 3.4, 0.420, 0, 0.461, 0.078, 0.54},
    {128, 128, 512, 10.0, 1.8, 0.459, 0.614, 0.690, 0.125, 0.61}, {128, 128, 256, 10.2, 2.7, 0.368, 0, 0.388, 0.095, 0.64},
    {64, 128, 256, 5.7, 4.9, 0.285, 0, 0.274, 0.120, 0.10}, {64, 64, 256, 5.9, 4.1, 0.209, 0, 0.253, 0.079, 0.03}};
bf16_tile pick_tile(const prefill_item* items, int n_items, int y_size) {
    int nk = 1;
    double w_mb = 0, y_mb = 0;
    bool rewards = false;
    for (int g = 0; g < n_items; ++g) {
        nk = std::max(nk, (items[g].d_in + 63) / 64);
        w_mb += 2e-6 * items[g].d_in * items[g].d_out;
        y_mb += 1e-6 * y_size * items[g].R * items[g].d_out;
        rewards = rewards || items[g].rv;
    }
    int best = 0;
    double best_us = 0;
    for (int i = 0; i < (int)(sizeof(TILE_COST) / sizeof(TILE_COST[0])); ++i) {
        const tile_cost& c = TILE_COST[i];
        const long long tiles = count_tiles(c, items, n_items);
        if ((i >= TILE_64x128 && tiles > c.slots) || (i == TILE_64x64 && rewards)) continue;
        const double us = tile_us(c, tiles, nk, w_mb, y_mb) * (i == TILE_256x256 ? 0.98 : 1.0);
        if (i == 0 || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    return (bf16_tile)best;
}

// the rank-space vectors of every row
hipError_t launch_rank(hipStream_t st, prefill_args& a, bool finish) {
    int total = 0, maxR = 0;
    bool has16[2] = {false, false}, has32[2] = {false, false};   // [V_A with all its bits]
    const bool sums = a.Gn[0] > 0;         // 4-bit weights throughout
    for (int g = 0; g < a.n_items; ++g) {
        // K parts: enough workgroups for two per CU in a group of four projections, no part shorter than four steps; by the
        // item's own size only, so that an item's sums do not depend on what it is grouped with
        const int blocks = (a.it[g].R + RD_ROWS - 1) / RD_ROWS, nk = (a.it[g].d_in + 63) / 64;
        a.ksplit[g] = std::max(1, std::min({8, nk / 4, (128 + blocks - 1) / blocks}));
        a.tile_start[g] = total;
        total += blocks * a.ksplit[g];
        maxR = std::max(maxR, a.it[g].R);
        (a.it[g].rp == 16 ? has16 : has32)[a.it[g].VA3p != nullptr] = true;
    }
    for (int g = a.n_items; g <= ESSA_MAX_GROUP; ++g) a.tile_start[g] = total;
    if (sums) {
        if (has16[0]) hipLaunchKernelGGL((rank_down_kernel<16, false, true>), dim3(total), dim3(256), 0, st, a);
        if (has32[0]) hipLaunchKernelGGL((rank_down_kernel<32, false, true>), dim3(total), dim3(256), 0, st, a);
    } else if (has16[0]) hipLaunchKernelGGL((rank_down_kernel<16, false>), dim3(total), dim3(256), 0, st, a);
    if (has16[1]) hipLaunchKernelGGL((rank_down_kernel<16, true>), dim3(total), dim3(256), 0, st, a);
    if (has32[0] && !sums) hipLaunchKernelGGL((rank_down_kernel<32, false>), dim3(total), dim3(256), 0, st, a);
    if (has32[1]) hipLaunchKernelGGL((rank_down_kernel<32, true>), dim3(total), dim3(256), 0, st, a);
    if (!finish) return hipGetLastError();
    if (has16[0] || has16[1]) hipLaunchKernelGGL(rank_finish_kernel<16>, dim3((maxR + 15) / 16, a.n_items), dim3(256), 0, st, a);
    if (has32[0] || has32[1]) hipLaunchKernelGGL(rank_finish_kernel<32>, dim3((maxR + 7) / 8, a.n_items), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace

namespace essa_k {

__global__ __launch_bounds__(256) void expand_weights_kernel(const int8_t* __restrict__ Wt, const float* __restrict__ scale, int dout, int n_blocks,
                                                             long long pieces, uint16_t* __restrict__ W16) {
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < pieces; p += (long long)gridDim.x * 256) {
        const int lane = (int)(p & 63), j = (int)(p >> 6) & 1, half = (int)(p >> 7) & 1, kg = lane >> 4, l = 16 * half + (lane & 15);
        const long long blk = p >> 8, kt = blk / n_blocks, nb = blk % n_blocks;
        // columns 64 kt + 32 j + 8 kg .. + 7 of channel 32 nb + l
        const int8_t* src = Wt + ((2 * kt + j) * n_blocks + nb) * 1024 + ((kg >> 1) * 32 + l) * 16 + 8 * (kg & 1);
        const int o = (int)nb * 32 + l;
        const float s = o < dout ? scale[o] : 0.f;         // a channel of scale 0 contributes nothing
        const float two = s != 0.f ? ldexpf(1.f, ilogbf(s) - 8) : 0.f;
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = f32_to_bf16_bits((float)src[e] * two);
        __builtin_memcpy(W16 + p * 8, v, 16);
    }
}

hipError_t expand_weights(hipStream_t st, const int8_t* Wt, const float* scale, int dout, int n_blocks, int nk, uint16_t* W16) {
    const long long pieces = (long long)nk * n_blocks * 256;
    hipLaunchKernelGGL(expand_weights_kernel, dim3((unsigned)std::min<long long>((pieces + 255) / 256, 4096)), dim3(256), 0, st, Wt, scale, dout, n_blocks, pieces, W16);
    return hipGetLastError();
}

// One thread per word of eight codes: block (g, 16 channels), lane (kg, l16), word j = columns 128 g + 32 j + 8 kg .. + 7 of channel l16
__global__ __launch_bounds__(256) void repack_nibbles_kernel(const int8_t* __restrict__ Wt, int n_blocks, long long words, uint32_t* __restrict__ Wn) {
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < words; p += (long long)gridDim.x * 256) {
        const int j = (int)(p & 3), lane = (int)(p >> 2) & 63, kg = lane >> 4;
        const long long blk = p >> 8, g = blk / (2 * n_blocks);
        const int ch = (int)(blk % (2 * n_blocks)) * 16 + (lane & 15);
        // the int8 operand tile: pair of 32-column chunks 2 g + j / 2, low nibbles the even chunk's, high ones the odd one's
        const int8_t* src = Wt + ((2 * g + (j >> 1)) * n_blocks + ch / 32) * 1024 + ((kg >> 1) * 32 + ch % 32) * 16 + 8 * (kg & 1);
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t q = ((uint8_t)src[e] >> (4 * (j & 1))) & 15u;
            const int at = 3 + 4 * (e >> 1) + 16 * (e & 1);
            w |= (q << (at & 31)) | (at > 28 ? q >> (32 - at) : 0u);
        }
        Wn[p] = w;
    }
}

hipError_t repack_nibbles(hipStream_t st, const int8_t* Wt, int groups, int n_blocks, uint8_t* Wn) {
    const long long words = (long long)groups * n_blocks * 512;
    hipLaunchKernelGGL(repack_nibbles_kernel, dim3((unsigned)std::min<long long>((words + 255) / 256, 4096)), dim3(256), 0, st, Wt, n_blocks, words, (uint32_t*)Wn);
    return hipGetLastError();
}

hipError_t forward_prefill_q4(hipStream_t st, const fwd_item* items, int n_items, int y_dtype, hipEvent_t ev_start, hipEvent_t ev_stop) {
    prefill_args r{};
    q4_args a{};
    for (int g = 0; g < n_items; ++g) {
        const fwd_item& k = items[g];
        r.it[g] = prefill_item{(const uint16_t*)k.X, nullptr, nullptr, k.VAp, nullptr, nullptr, k.M, k.sigmaA, k.sigmaB, nullptr, k.row2cand, nullptr,
                               k.U16, k.Tpart, nullptr, k.sigma_stride, k.R, k.d_in, k.d_out, k.r, k.rp, k.n_blocks};
        uint16_t* sums = (uint16_t*)k.Xh;                  // 192 bytes a row and 32 groups, where the limb kernels keep at least 512
        r.XS16[g] = k.x_owner ? sums : nullptr;
        r.Gn[g] = (k.groups + 31) / 32 * 32;
        a.it[g] = q4_item{(const uint16_t*)k.X, k.UB16, k.U16, k.SZn, sums, k.Wn, k.St, k.rv, k.Y, k.rowpart, k.R, k.d_in, k.d_out, k.rp, k.n_blocks, r.Gn[g]};
    }
    r.n_items = a.n_items = n_items;
    r.u_scale = 0x1p-12f;
    const bool yb = y_dtype == ESSA_BF16;
    const q4_tile tile = pick_q4_tile(a, yb ? 2 : 4);
    hipError_t e = launch_rank(st, r, tile < Q4_32x128);
    if (e != hipSuccess) return e;
    for (int g = 0; g < n_items; ++g)
        a.rk[g] = q4_rank{items[g].Tpart, items[g].M, items[g].sigmaA, items[g].sigmaB, items[g].row2cand, items[g].sigma_stride, items[g].R, items[g].r, items[g].rp, r.ksplit[g]};
    tl_pre_start = ev_start;
    tl_pre_stop = ev_stop;
    switch (tile) {
        case Q4_64x256: e = yb ? launch_q4<4, 4, 2, true>(st, a) : launch_q4<4, 4, 2, false>(st, a); break;
        case Q4_80x256: e = yb ? launch_q4<5, 4, 2, true>(st, a) : launch_q4<5, 4, 2, false>(st, a); break;
        case Q4_96x256: e = yb ? launch_q4<6, 4, 2, true>(st, a) : launch_q4<6, 4, 2, false>(st, a); break;
        case Q4_32x128: e = yb ? launch_q4<2, 2, 4, true>(st, a) : launch_q4<2, 2, 4, false>(st, a); break;
        case Q4_48x128: e = yb ? launch_q4<3, 2, 3, true>(st, a) : launch_q4<3, 2, 3, false>(st, a); break;
        default: e = yb ? launch_q4<4, 2, 2, true>(st, a) : launch_q4<4, 2, 2, false>(st, a); break;
    }
    tl_pre_start = tl_pre_stop = nullptr;
    return e;
}

bool prefill_takes(const fwd_item& it) {
    return it.quant == ESSA_QUANT_INT8_PERCH && it.W16 && it.d_in % 16 == 0 && ((uintptr_t)it.X & 15) == 0;
}

hipError_t forward_prefill(hipStream_t st, const fwd_item* items, int n_items, int y_dtype, unsigned flags, hipEvent_t ev_start,
                           hipEvent_t ev_stop) {
    prefill_args a{};
    for (int g = 0; g < n_items; ++g) {
        const fwd_item& k = items[g];
        a.it[g] = prefill_item{(const uint16_t*)k.X, k.W16, k.US16, k.VAp, k.VA3p, k.scale16, k.M, k.sigmaA, k.sigmaB, k.rv, k.row2cand, k.Y,
                               k.U16, k.Tpart, k.rowpart, k.sigma_stride, k.R, k.d_in, k.d_out, k.r, k.rp, k.n_blocks};
    }
    a.n_items = n_items;
    a.flags = flags;
    a.u_scale = 1.f;
    const bf16_tile tile = pick_tile(a.it, n_items, y_dtype == ESSA_BF16 ? 2 : 4);
    if (flags & ESSA_BASE_ONLY) {
        int maxR = 0;
        for (int g = 0; g < n_items; ++g) maxR = std::max(maxR, a.it[g].R);
        hipLaunchKernelGGL(rank_none_kernel, dim3((maxR + 3) / 4, n_items), dim3(256), 0, st, a);
    } else {
        hipError_t e = launch_rank(st, a, tile < TILE_64x128);
        if (e != hipSuccess) return e;
    }
    tl_pre_start = ev_start;
    tl_pre_stop = ev_stop;
    const bool yb = y_dtype == ESSA_BF16;
    hipError_t e;
    switch (tile) {
        case TILE_256x256: e = yb ? launch_bf16<8, 4, 3, 2, true>(st, a) : launch_bf16<8, 4, 3, 2, false>(st, a); break;
        case TILE_224x256: e = yb ? launch_bf16<7, 4, 3, 2, true>(st, a) : launch_bf16<7, 4, 3, 2, false>(st, a); break;
        case TILE_192x256: e = yb ? launch_bf16<6, 4, 3, 2, true>(st, a) : launch_bf16<6, 4, 3, 2, false>(st, a); break;
        case TILE_160x256: e = yb ? launch_bf16<5, 4, 3, 3, true>(st, a) : launch_bf16<5, 4, 3, 3, false>(st, a); break;
        case TILE_160x128: e = yb ? launch_bf16<5, 2, 4, 4, true>(st, a) : launch_bf16<5, 2, 4, 4, false>(st, a); break;
        case TILE_256x128: e = yb ? launch_bf16<8, 2, 3, 4, true>(st, a) : launch_bf16<8, 2, 3, 4, false>(st, a); break;
        case TILE_128x128: e = yb ? launch_bf16<4, 2, 3, 2, true>(st, a) : launch_bf16<4, 2, 3, 2, false>(st, a); break;
        case TILE_128x128_DEEP: e = yb ? launch_bf16<4, 2, 5, 5, true>(st, a) : launch_bf16<4, 2, 5, 5, false>(st, a); break;
        case TILE_64x128: e = yb ? launch_bf16<2, 2, 5, 4, true>(st, a) : launch_bf16<2, 2, 5, 4, false>(st, a); break;
        default: e = yb ? launch_bf16<2, 1, 5, 4, true>(st, a) : launch_bf16<2, 1, 5, 4, false>(st, a); break;
    }
    tl_pre_start = tl_pre_stop = nullptr;
    return e;
}

}  // namespace essa_k
