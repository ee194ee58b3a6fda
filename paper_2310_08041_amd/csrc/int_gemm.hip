// Integer GEMM on the gfx950 int8 matrix cores with a dequantising epilogue.
//
//   acc[n, o] = sum_k a[n, k] * w[o, k]          (Eq. 1 on the codes of Eq. 2; exact int32)
//   Y[n, o]   = ((float)(acc - bx[n]*cs[o] - bw[o]*rs[n] + K*bx[n]*bw[o]) * ax[n]) * aw[o]
//
// Both operands arrive as packed 4/6/8-bit codes, K contiguous.  A workgroup of 256 lanes (4 waves,
// 2 x 2) owns a 128 x 128 tile of Y.  Per K-tile of 256 codes every lane fetches 64-code units of
// the packed rows from HBM into registers (16-byte loads), expands them to one byte per code and
// stores them into LDS (16-byte chunks, XOR-swizzled by row so that the matrix-core operand reads
// are bank-conflict free); the loads of the next K-tile are in flight while the current one is
// multiplied.  Each wave multiplies 64 x 64 with v_mfma_i32_16x16x64_i8 (16 accumulator tiles).
//
// 8-bit codes do not fit a signed byte: they are stored as code-128 and the accumulator is corrected
// with the row / column sums the epilogue already has.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <mutex>
#include <type_traits>
#include <vector>

#include "qllm.h"
#include "qllm_probes.h"
#include "fused_common.h"
#include "lds_copy.h"

extern "C" void qllm_note_hip_error(const char *step, const char *name);

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, KT = 256; // block tile; KT codes per LDS stage
constexpr int THREADS = 256;
constexpr int UNIT = 64;                    // codes per fetch unit = K of one MFMA
constexpr int ROW_LDS = KT;                 // bytes per tile row in LDS (one byte per code)

struct GemmArgs {
    const uint8_t *a_codes, *w_codes;
    int64_t a_row_bytes, w_row_bytes;
    const float *ax, *aw;
    const int32_t *bx, *bw, *rs, *cs;
    int32_t N, O, K, Kpad;
    int32_t small_zero; // zero-points below this (in magnitude) keep every epilogue term inside 24 / 32 bits; 0: never
    void *y;
    int64_t ldy;
    int32_t *acc_dump;
    int32_t *partial; // [splits][N][O] raw accumulators when K is split over workgroups, else unused
    int32_t splits;
    const uint8_t *a_tiles, *w_tiles; // both operands as 6-bit fields in matrix-core order (see TILES6 below), or null
    const uint8_t *a_tiles8, *w_tiles8; // both operands as bytes in matrix-core order (see TILES8 below), or null
    bool a_laid; // a_tiles (a_tiles8) holds the activations already
    // A launch of the FP6 or the byte-operand kernel may cover the output features o_first .. O - 1 only (the call is
    // then two launches with different tiles, each with its own O); never together with acc_dump, whose rows are O long.
    int32_t o_first;
    int32_t lds_epilogue; // 1: K allows finish_from_lds and nobody asked for the raw accumulators
};

template <int BITS>
struct Unit {
    uint4 r[BITS / 2]; // 64 codes: 32 / 48 / 64 bytes
};

// unit number `unit` (64 codes each) of a packed row
template <int BITS>
__device__ __forceinline__ void load_unit(Unit<BITS> &u, const uint8_t *row, int unit)
{
    const uint4 *p = reinterpret_cast<const uint4 *>(row + (int64_t)unit * (UNIT * BITS / 8));
#pragma unroll
    for (int i = 0; i < BITS / 2; ++i) u.r[i] = p[i];
}

// 8 nibbles of w -> 8 bytes in channel order
__device__ __forceinline__ void expand4(uint32_t w, uint32_t &d0, uint32_t &d1)
{
    const uint32_t lo = w & 0x0f0f0f0fu;        // codes 0 2 4 6
    const uint32_t hi = (w >> 4) & 0x0f0f0f0fu; // codes 1 3 5 7
    d0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u); // lo.b0 hi.b0 lo.b1 hi.b1
    d1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u); // lo.b2 hi.b2 lo.b3 hi.b3
}

// four 6-bit codes in the low 24 bits of t (higher bits are ignored) -> four bytes
__device__ __forceinline__ uint32_t spread6(uint32_t t)
{
    const uint32_t x = (t & 0xfffu) | ((t << 4) & 0x0fff0000u);      // codes 0,1 in the low half, 2,3 in the high half
    return (x & 0x003f003fu) | ((x << 2) & 0x3f003f00u);
}

// One unit (64 packed codes) -> 64 bytes, as 16 dwords.  PERM: both operands are 4-bit, so the order of
// the codes inside a unit is free as long as both sides use the same one; even codes then odd codes of
// each dword is the cheapest (two masks and a shift instead of two more byte permutes).  8-bit codes
// become code - 128, a signed byte (the epilogue adds the difference back).
template <int BITS, bool PERM>
__device__ __forceinline__ void expand_unit(const Unit<BITS> &u, uint32_t (&d)[16])
{
    if constexpr (BITS == 4) {
        const uint32_t w[8] = {u.r[0].x, u.r[0].y, u.r[0].z, u.r[0].w, u.r[1].x, u.r[1].y, u.r[1].z, u.r[1].w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (PERM) {
                d[2 * i] = w[i] & 0x0f0f0f0fu;
                d[2 * i + 1] = (w[i] >> 4) & 0x0f0f0f0fu;
            } else {
                expand4(w[i], d[2 * i], d[2 * i + 1]);
            }
        }
    } else if constexpr (BITS == 6) {
        const uint32_t w[12] = {u.r[0].x, u.r[0].y, u.r[0].z, u.r[0].w, u.r[1].x, u.r[1].y,
                                u.r[1].z, u.r[1].w, u.r[2].x, u.r[2].y, u.r[2].z, u.r[2].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) { // 3 dwords = 4 groups of 24 bits
            const uint32_t w0 = w[3 * i], w1 = w[3 * i + 1], w2 = w[3 * i + 2];
            d[4 * i + 0] = spread6(w0);
            d[4 * i + 1] = spread6(__builtin_amdgcn_alignbit(w1, w0, 24));
            d[4 * i + 2] = spread6(__builtin_amdgcn_alignbit(w2, w1, 16));
            d[4 * i + 3] = spread6(w2 >> 8);
        }
    } else {
        const uint32_t w[16] = {u.r[0].x, u.r[0].y, u.r[0].z, u.r[0].w, u.r[1].x, u.r[1].y, u.r[1].z, u.r[1].w,
                                u.r[2].x, u.r[2].y, u.r[2].z, u.r[2].w, u.r[3].x, u.r[3].y, u.r[3].z, u.r[3].w};
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = w[i] ^ 0x80808080u; // code - 128 as a signed byte
    }
}

// Expands one unit and stores it as four 16-byte chunks of LDS row `row` (ROWB bytes per row, chunks
// XOR-swizzled by row).
template <int BITS, int ROWB, bool PERM>
__device__ __forceinline__ void store_unit(const Unit<BITS> &u, uint8_t *tile, int row, int ku)
{
    uint32_t d[16];
    expand_unit<BITS, PERM>(u, d);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int chunk = (ku * 4 + c) ^ (row & 7);
        *reinterpret_cast<uint4 *>(tile + row * ROWB + chunk * 16) =
            make_uint4(d[4 * c], d[4 * c + 1], d[4 * c + 2], d[4 * c + 3]);
    }
}

// Chunk c (16 codes -> 16 bytes) of one unit, expanded and stored; c is a constant where this is
// called, so only that chunk's share of the expansion is left of expand_unit.
template <int BITS, int ROWB, bool PERM>
__device__ __forceinline__ void store_chunk(const Unit<BITS> &u, uint8_t *tile, int row, int ku, int c)
{
    uint32_t d[16];
    expand_unit<BITS, PERM>(u, d);
    const int chunk = (ku * 4 + c) ^ (row & 7);
    *reinterpret_cast<uint4 *>(tile + row * ROWB + chunk * 16) = make_uint4(d[4 * c], d[4 * c + 1], d[4 * c + 2], d[4 * c + 3]);
}

template <int ROWB>
__device__ __forceinline__ v4i load_frag(const uint8_t *tile, int row, int chunk)
{
    return *reinterpret_cast<const v4i *>(tile + row * ROWB + ((chunk ^ (row & 7)) * 16));
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Two floats -> two bfloat16 in one dword, round to nearest even: the hardware's packed conversion
// (v_cvt_pk_bf16_f32), one instruction where the integer form above takes about ten for the pair.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32x2_to_bf16x2_rne(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Stores 4 consecutive output features of one token (16 bytes per lane for fp32, 8 for bf16) and,
// if asked for, the raw accumulators.
template <typename YT>
__device__ __forceinline__ void store4(const GemmArgs &g, const float *out, const int32_t *raw, int n, int ob)
{
    if (ob + 3 < g.O) {
        if constexpr (sizeof(YT) == 4) {
            float *yp = reinterpret_cast<float *>(g.y) + (int64_t)n * g.ldy + ob;
            if ((reinterpret_cast<uintptr_t>(yp) & 15u) == 0) {
                *reinterpret_cast<float4 *>(yp) = make_float4(out[0], out[1], out[2], out[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) yp[r] = out[r];
            }
        } else {
            uint16_t *yp = reinterpret_cast<uint16_t *>(g.y) + (int64_t)n * g.ldy + ob;
            const uint32_t p0 = f32x2_to_bf16x2_rne(out[0], out[1]), p1 = f32x2_to_bf16x2_rne(out[2], out[3]);
            if ((reinterpret_cast<uintptr_t>(yp) & 7u) == 0) {
                *reinterpret_cast<uint2 *>(yp) = make_uint2(p0, p1);
            } else {
                yp[0] = (uint16_t)p0; yp[1] = (uint16_t)(p0 >> 16);
                yp[2] = (uint16_t)p1; yp[3] = (uint16_t)(p1 >> 16);
            }
        }
        if (g.acc_dump) {
#pragma unroll
            for (int r = 0; r < 4; ++r) g.acc_dump[(int64_t)n * g.O + ob + r] = raw[r];
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (ob + r < g.O) {
                if constexpr (sizeof(YT) == 4)
                    reinterpret_cast<float *>(g.y)[(int64_t)n * g.ldy + ob + r] = out[r];
                else
                    reinterpret_cast<uint16_t *>(g.y)[(int64_t)n * g.ldy + ob + r] = f32_to_bf16_rne(out[r]);
                if (g.acc_dump) g.acc_dump[(int64_t)n * g.O + ob + r] = raw[r];
            }
    }
}

// Dequantising epilogue of one wave tile: NI x NJ matrix-core tiles of 16 x 16; the lane holds, for
// tile (i, j), token n_base + 16 i + (lane & 15) and features o_base + 16 j + 4 (lane >> 4) + 0..3.
//   bracket = acc - bx*cs - bw*rs + K*bx*bw       (exact integer)
//   Y       = ((float)bracket * ax) * aw
// When both zero-points are small (the usual case: |beta| < g.small_zero, a bound the launcher derives
// from K and the bit widths) every factor fits 24 bits and every sum 32 bits, and the bracket costs
// three full-rate multiply-adds; otherwise it is formed in 64-bit arithmetic.
// An accumulator as the integer it stands for: the int8 matrix cores' own, or 64 x the FP6 path's float (exact).
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int32_t acc_int(const v4i &a, int r) { return a[r]; }
__device__ __forceinline__ int32_t acc_int(const v4f &a, int r) { return (int32_t)(a[r] * 64.0f); }

template <int ABITS, int WBITS, typename YT, int NI, int NJ, typename ACC>
__device__ __forceinline__ void finish_wave_tile(const GemmArgs &g, const ACC (&acc)[NI][NJ], int n_base, int o_base,
                                                 int lane, int32_t k_biased = -1)
{
    constexpr int SA = ABITS == 8 ? 1 : 0, SW = WBITS == 8 ? 1 : 0;
    int32_t cs[NJ][4], bw[NJ][4];
    float aw[NJ][4];
    bool cols_small = true;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = min(o_base + j * 16 + 4 * (lane >> 4) + r, g.O - 1);
            cs[j][r] = g.cs[o];
            bw[j][r] = g.bw[o];
            aw[j][r] = g.aw[o];
            cols_small = cols_small && abs(bw[j][r]) < g.small_zero;
        }
    // 8-bit codes went into the matrix cores as code - 128; where both sides did, every place of K that held such a
    // pair adds 128 * 128: the padded row length, unless the kernel says how many places it summed that way
    const int32_t k_off = 16384 * SA * SW * (k_biased >= 0 ? k_biased : g.Kpad);

    // The usual case, decided once for the wave: the tile lies inside Y, Y's rows are aligned for whole stores, nobody
    // asked for the raw accumulators, and every zero-point of the tile is small.  Then the tile is straight-line
    // code: three 24-bit multiply-adds, a conversion and two multiplications per output, one store per four.
    {
        const bool inside = n_base + 16 * NI <= g.N && o_base + 16 * NJ <= g.O;
        const bool aligned = (reinterpret_cast<uintptr_t>(g.y) & (sizeof(YT) == 4 ? 15u : 7u)) == 0 && (g.ldy & 3) == 0;
        if (inside && aligned && !g.acc_dump) { // wave-uniform so far: the loads below are in bounds
            int32_t bxs[NI], rss[NI];
            float axs[NI];
            bool small = cols_small;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int n = n_base + i * 16 + (lane & 15);
                bxs[i] = g.bx[n];
                rss[i] = g.rs[n];
                axs[i] = g.ax[n];
                small = small && abs(bxs[i]) < g.small_zero;
            }
            if (__all(small)) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int n = n_base + i * 16 + (lane & 15);
                    const int32_t kbx = g.K * bxs[i];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        float out[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            int32_t t = acc_int(acc[i][j], r) + 128 * SW * rss[i] + 128 * SA * cs[j][r] - k_off;
                            t -= __mul24(bxs[i], cs[j][r]);
                            t -= __mul24(bw[j][r], rss[i]);
                            t += __mul24(kbx, bw[j][r]);
                            float v = (float)t;
                            v = v * axs[i];
                            v = v * aw[j][r];
                            out[r] = v;
                        }
                        const int64_t at = (int64_t)n * g.ldy + o_base + j * 16 + 4 * (lane >> 4);
                        if constexpr (sizeof(YT) == 4)
                            *reinterpret_cast<float4 *>(reinterpret_cast<float *>(g.y) + at) = make_float4(out[0], out[1], out[2], out[3]);
                        else
                            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(g.y) + at) =
                                make_uint2(f32x2_to_bf16x2_rne(out[0], out[1]), f32x2_to_bf16x2_rne(out[2], out[3]));
                    }
                }
                return;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int n = n_base + i * 16 + (lane & 15);
        if (n >= g.N) continue;
        const int32_t bx = g.bx[n], rs = g.rs[n];
        const float ax = g.ax[n];
        const bool small = cols_small && abs(bx) < g.small_zero;
        const int32_t kbx = g.K * bx; // only used when small
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            float out[4];
            int32_t raw[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // the true accumulator fits int32 (checked by the launcher), so wrapping sums are exact
                raw[r] = acc_int(acc[i][j], r) + 128 * SW * rs + 128 * SA * cs[j][r] - k_off;
                float v;
                if (small) {
                    int32_t t = raw[r] - __mul24(bx, cs[j][r]);
                    t -= __mul24(bw[j][r], rs);
                    t += __mul24(kbx, bw[j][r]);
                    v = (float)t;
                } else {
                    const int64_t t = (int64_t)raw[r] - (int64_t)bx * cs[j][r] - (int64_t)bw[j][r] * rs +
                                      (int64_t)g.K * bx * bw[j][r];
                    v = (float)t;
                }
                v = v * ax;
                v = v * aw[j][r];
                out[r] = v;
            }
            store4<YT>(g, out, raw, n, o_base + j * 16 + 4 * (lane >> 4));
        }
    }
}

template <int ABITS, int WBITS, typename YT>
__global__ __launch_bounds__(THREADS) void int_gemm_kernel(const GemmArgs g)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds_a[BM * ROW_LDS];
    __shared__ __attribute__((aligned(16))) uint8_t lds_w[BN * ROW_LDS];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1; // wave position in the 2 x 2 arrangement
    const int n0 = blockIdx.y * BM, o0 = blockIdx.x * BN;

    // fetch assignment: units tid and tid + 256 of each operand tile (unit = row * 4 + ku)
    const int f_row = tid >> 2, f_ku = tid & 3;
    const uint8_t *a_row[2], *w_row[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int rn = min(n0 + f_row + 64 * h, g.N - 1); // rows past the edge re-read the last row
        const int ro = min(o0 + f_row + 64 * h, g.O - 1);
        a_row[h] = g.a_codes + (int64_t)rn * g.a_row_bytes;
        w_row[h] = g.w_codes + (int64_t)ro * g.w_row_bytes;
    }

    v4i acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    Unit<ABITS> ua[2];
    Unit<WBITS> uw[2];
    const int n_kt = g.Kpad / KT;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        load_unit<ABITS>(ua[h], a_row[h], f_ku);
        load_unit<WBITS>(uw[h], w_row[h], f_ku);
    }

    for (int kt = 0; kt < n_kt; ++kt) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            store_unit<ABITS, ROW_LDS, ABITS == 4 && WBITS == 4>(ua[h], lds_a, f_row + 64 * h, f_ku);
            store_unit<WBITS, ROW_LDS, ABITS == 4 && WBITS == 4>(uw[h], lds_w, f_row + 64 * h, f_ku);
        }
        __syncthreads();
        if (kt + 1 < n_kt) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                load_unit<ABITS>(ua[h], a_row[h], (kt + 1) * (KT / UNIT) + f_ku);
                load_unit<WBITS>(uw[h], w_row[h], (kt + 1) * (KT / UNIT) + f_ku);
            }
        }
#pragma unroll
        for (int ks = 0; ks < KT / UNIT; ++ks) {
            const int chunk = ks * 4 + (lane >> 4);
            v4i fa[4], fw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) fa[i] = load_frag<ROW_LDS>(lds_a, wm * 64 + i * 16 + (lane & 15), chunk);
#pragma unroll
            for (int j = 0; j < 4; ++j) fw[j] = load_frag<ROW_LDS>(lds_w, wn * 64 + j * 16 + (lane & 15), chunk);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    // operand order (w, a): the lane then holds 4 consecutive OUTPUT features of one
                    // token, so the stores below write 16 bytes per lane
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[j], fa[i], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    // ---- epilogue.  acc[i][j][r]: token n0 + wm*64 + i*16 + (lane & 15),
    //                               feature o0 + wn*64 + j*16 + 4*(lane >> 4) + r
    finish_wave_tile<ABITS, WBITS, YT, 4, 4>(g, acc, n0 + wm * 64, o0 + wn * 64, lane);
}

// ---- the large-tile kernel for bit pairs other than 4/4: 512 lanes (8 waves, 2 x 4), a 256 x 256 tile
// of Y, K-tiles of 128 codes, one byte per code in two LDS buffers.  While the matrix cores work
// through buffer `cur`, the lanes expand the next K-tile (fetched one iteration earlier) into the other
// buffer, one 16-byte chunk per group of four matrix-core operations, and fetch the one after it: one
// barrier per K-tile.
constexpr int LBM = 256, LBN = 256, LKT = 128, LTHREADS = 512, LROWB = LKT; // one byte per code in LDS
constexpr int LBUF = (LBM + LBN) * LROWB;                                   // 64 KB per buffer

template <int ABITS, int WBITS, typename YT>
__global__ __launch_bounds__(LTHREADS) void int_gemm_big_kernel(const GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr bool PERM = ABITS == 4 && WBITS == 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3; // wave tile: 128 tokens x 64 features
    const int n0 = blockIdx.y * LBM, o0 = blockIdx.x * LBN;

    // fetch assignment: one unit of each operand per lane and K-tile (unit = row * 2 + ku)
    const int f_row = tid >> 1, f_ku = tid & 1;
    const uint8_t *a_row = g.a_codes + (int64_t)min(n0 + f_row, g.N - 1) * g.a_row_bytes; // past the edge:
    const uint8_t *w_row = g.w_codes + (int64_t)min(o0 + f_row, g.O - 1) * g.w_row_bytes; // re-read the last row

    v4i acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    Unit<ABITS> ua;
    Unit<WBITS> uw;
    const int n_kt = g.Kpad / LKT;
    load_unit<ABITS>(ua, a_row, f_ku);
    load_unit<WBITS>(uw, w_row, f_ku);
    store_unit<ABITS, LROWB, PERM>(ua, lds, f_row, f_ku);
    store_unit<WBITS, LROWB, PERM>(uw, lds + LBM * LROWB, f_row, f_ku);
    load_unit<ABITS>(ua, a_row, min(1, n_kt - 1) * 2 + f_ku);
    load_unit<WBITS>(uw, w_row, min(1, n_kt - 1) * 2 + f_ku);
    __syncthreads();

    // One K-tile = 16 groups of four matrix-core operations: group s multiplies the token-side
    // fragment s (rows 16 (s & 7) .. of the wave's 128, half s >> 3 of the K-tile) with the four
    // feature-side fragments of that half.  Everything else is spread over the groups, in an order
    // fixed by scheduling fences, so that the matrix cores never wait for it:
    //   * token-side fragment s + DIST is requested in group s (a ring of RING registers), also
    //     across the K-tile boundary; the feature-side fragments of the second half in groups 0..3,
    //     those of the next K-tile's first half in the last two groups;
    //   * the refill of the other buffer (expand one 16-byte chunk of the unit fetched a K-tile
    //     ago, store it) takes groups 4..11, one chunk each; the fetch of the K-tile after that
    //     follows in group 12;
    //   * the one barrier per K-tile sits after group 15 - DIST: every refill store precedes it and
    //     every read of the next K-tile follows it; every read of this K-tile precedes it and the
    //     stores that will overwrite this buffer follow the next one.
    // The last K-tile refills and prefetches like the others (a re-read of the last K-tile into the
    // buffer nobody reads any more), which keeps the loop body free of branches.
    constexpr int DIST = 2, RING = 4, GROUPS = 8 * (LKT / UNIT), REFILL0 = 4;
    static_assert(GROUPS == 16 && GROUPS % RING == 0 && DIST < RING && REFILL0 + 8 < GROUPS - DIST, "group plan");
    // The loop is rotated by DIST groups: an iteration starts, right after the barrier, with the last
    // DIST groups of the previous K-tile (which request the first fragments of this one) and ends
    // with the barrier, so that no LDS request is pending across the loop's back edge.  Before the
    // first K-tile those groups multiply zeros; after the last one they run once more on their own.
    v4i fw[2][4], fa[RING];
#pragma unroll
    for (int j = 0; j < 4; ++j) fw[1][j] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int s = GROUPS - DIST; s < GROUPS; ++s) fa[s % RING] = v4i{0, 0, 0, 0};
    const int frow = lane & 15, fchunk = lane >> 4;

    for (int kt = 0; kt < n_kt; ++kt) {
        uint8_t *cur = lds + (kt & 1) * LBUF, *nxt = lds + ((kt + 1) & 1) * LBUF;
        const int kt2 = min(kt + 2, n_kt - 1);
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            const int s = (u + GROUPS - DIST) % GROUPS, ks = s >> 3, t = (s + DIST) % GROUPS;
            auto multiply = [&] {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[s & 7][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[ks][j], fa[s % RING], acc[s & 7][j], 0, 0, 0);
            };
            // group 0 is the first to use what the two groups before it asked for: its own requests
            // come after its operations, so that it waits for nothing newer than it needs
            if (s == 0) {
                multiply();
                __builtin_amdgcn_sched_barrier(0);
            }
            // fragment requests (all from this iteration's K-tile)
            fa[t % RING] = load_frag<LROWB>(cur, wm * 128 + (t & 7) * 16 + frow, (t >> 3) * 4 + fchunk);
            if (s < 4) fw[1][s] = load_frag<LROWB>(cur + LBM * LROWB, wn * 64 + s * 16 + frow, 4 + fchunk);
            if (s >= GROUPS - 2) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int j = (s - (GROUPS - 2)) * 2 + h;
                    fw[0][j] = load_frag<LROWB>(cur + LBM * LROWB, wn * 64 + j * 16 + frow, fchunk);
                }
            }
            // refill of the other buffer, fetch of the K-tile after it
            if (s >= REFILL0 && s < REFILL0 + 4) store_chunk<ABITS, LROWB, PERM>(ua, nxt, f_row, f_ku, s - REFILL0);
            if (s >= REFILL0 + 4 && s < REFILL0 + 8) store_chunk<WBITS, LROWB, PERM>(uw, nxt + LBM * LROWB, f_row, f_ku, s - REFILL0 - 4);
            if (s == REFILL0 + 8) {
                load_unit<ABITS>(ua, a_row, kt2 * 2 + f_ku);
                load_unit<WBITS>(uw, w_row, kt2 * 2 + f_ku);
            }
            if (s != 0) multiply();
            if (u == GROUPS - 1) __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = GROUPS - DIST; s < GROUPS; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[s & 7][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[1][j], fa[s % RING], acc[s & 7][j], 0, 0, 0);

    finish_wave_tile<ABITS, WBITS, YT, 8, 4>(g, acc, n0 + wm * 128, o0 + wn * 64, lane);
}

// ---- 4-bit codes on both sides, many tokens: the same 256 x 256 tile and 2 x 4 waves, but the codes
// stay packed (two per byte) in LDS and are split into bytes in registers, after the operand read.
// That halves the LDS traffic of the kernel above, which was what held it back: per K-tile of 128
// codes its expanded stores and operand reads kept LDS busy as long as the matrix cores were.
//   * LDS row = the 64 packed bytes of a K-tile; a lane (r, q) of an operand read takes the 16 bytes
//     q of row r: the low nibbles are its 16 codes for one matrix-core operation (m = 0), the high
//     nibbles those for a second one (m = 1).  Which 64 codes of the K-tile an operation sums is free
//     as long as both operands agree, and they do: same read, same split.
//   * Where a row's four 16-byte pieces sit in LDS is chosen for the banks.  Within a block of 16
//     rows, row r is stored as row place16(r) and its piece q at position q ^ (r & 3): a read by
//     lanes (r, q) then covers the block's 1 KB exactly once and each lane falls on the same banks
//     as in the byte-per-code layout of the kernel above (measured free of conflicts; rows kept in
//     order with any XOR of the piece index cost two passes per read).  The stores go the other way
//     round: lane t writes the t-th 16 bytes of the buffer half and fetches whichever row and piece
//     belong there, still four lanes per row.
//   * One K-tile = 16 groups of four matrix-core operations, (i, m) = (s >> 1, s & 1): token rows
//     16 i .. of the wave's 128, nibble m, times the wave's four feature-side operands of nibble m.
//     The eight feature-side operands of a K-tile stay split in registers; the token side streams:
//     packed read two row blocks ahead (a ring of four), split one group ahead.
//   * As above the order is fixed by scheduling fences, the loop is rotated by four groups (it
//     starts, after the barrier, with the last four groups of the previous K-tile, which request
//     the first operands of this one and multiply zeros the first time round) and refills without
//     branches.
constexpr int PROWB = 64;                       // packed bytes per LDS row and K-tile
constexpr int PBUF = (LBM + LBN) * PROWB;       // 32 KB per buffer
constexpr int PKT = 128;                        // codes per K-tile
constexpr int NBUF = 4;                         // ring of LDS buffers
constexpr int WAIT_VM8 = 8 | (7 << 4) | (15 << 8);       // s_waitcnt vmcnt(8) and nothing else
constexpr int WAIT_VM0 = 0 | (7 << 4) | (15 << 8);       // s_waitcnt vmcnt(0) and nothing else
constexpr int WAIT_VM8_LGKM0 = 8 | (7 << 4) | (0 << 8);  // s_waitcnt vmcnt(8) lgkmcnt(0)

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4i nib_lo(v4u p) { return (v4i)(p & 0x0f0f0f0fu); }
__device__ __forceinline__ v4i nib_hi(v4u p) { return (v4i)((p >> 4) & 0x0f0f0f0fu); }
// place of row r (0..15) inside its block of 16 rows, and the row stored at place p
__device__ __forceinline__ int place16(int r) { return ((r & 2) << 2) | ((r & 8) >> 1) | ((r & 1) << 1) | ((r & 4) >> 2); }
__device__ __forceinline__ int row_at16(int p) { return ((p & 2) >> 1) | ((p & 8) >> 2) | ((p & 1) << 2) | ((p & 4) << 1); }

// MI x NJ matrix-core tiles per wave: 8 x 4 (a 256 x 256 tile of Y per workgroup, the shape for many
// tokens) or 4 x 2 (128 x 128: four times as many workgroups, two of which share a CU, for shapes
// whose 256 x 256 tiles would leave most of the chip idle).
// SPLIT: K is dealt out to gridDim.z workgroups per tile of Y (shapes with so few tiles that most CUs
// would idle through a long K loop); each writes its raw accumulators to g.partial and
// splitk_finish_kernel adds them up and does the epilogue.
template <typename YT, int MI, int NJ, bool SPLIT = false>
__global__ __launch_bounds__(LTHREADS, MI == 8 ? 1 : 2) void int_gemm_w4a4_kernel(const GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int TM = 2 * MI * 16, TN = 4 * NJ * 16;     // the workgroup's tile of Y: 2 x 4 waves
    constexpr int STAGE = (TM + TN) * PROWB;              // bytes of one buffer of the ring
    constexpr int BLOCKS = (TM + TN) / 16, NLOAD = BLOCKS / 8; // 16-row blocks per K-tile; loads per wave and K-tile
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3; // wave tile: 16 MI tokens x 16 NJ features
    const int n0 = blockIdx.y * TM, o0 = blockIdx.x * TN;

    // fetch assignment: wave w brings in the 16-row blocks w, w + 8, .. of the buffer (the tile's token
    // rows first, then its feature rows); lane l fills the l-th 16 bytes of a block, that is piece
    // f_piece of the block's row f_row
    const int f_row = row_at16(lane >> 2), f_piece = (lane & 3) ^ (f_row & 3);
    const uint8_t *src[NLOAD];
#pragma unroll
    for (int t = 0; t < NLOAD; ++t) { // past the edge: re-read the last row
        const int blk = wave + 8 * t;
        src[t] = blk < TM / 16
                     ? g.a_codes + (int64_t)min(n0 + blk * 16 + f_row, g.N - 1) * g.a_row_bytes + f_piece * 16
                     : g.w_codes + (int64_t)min(o0 + (blk - TM / 16) * 16 + f_row, g.O - 1) * g.w_row_bytes + f_piece * 16;
    }

    // operand reads: lane (r, q) takes piece q of row r of a block of 16 rows
    const int r = lane & 15, q = lane >> 4;
    const int a_off = (wm * 16 * MI + place16(r)) * PROWB + ((q ^ (r & 3)) << 4);      // + i * 16 rows
    const int w_off = (TM + wn * 16 * NJ + place16(r)) * PROWB + ((q ^ (r & 3)) << 4); // + j * 16 rows

    v4i acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // Refill: 16-byte global loads that write LDS directly (lane l of a wave lands at the wave's LDS
    // base + 16 l, which is why a block's order above is the lanes' order): no staging registers, no
    // LDS store instructions; NLOAD loads per wave and K-tile, issued three K-tiles ahead into a ring
    // of four buffers.  Loads complete in order, so "at most 2 NLOAD outstanding" before the barrier
    // means the next K-tile has landed.
    constexpr int WAIT_LANDED = 2 * NLOAD | (7 << 4) | (15 << 8);    // s_waitcnt vmcnt(2 NLOAD)
    constexpr int WAIT_LANDED_LGKM0 = 2 * NLOAD | (7 << 4) | (0 << 8); // ... and lgkmcnt(0)
    const int all_kt = g.Kpad / PKT;
    const int kt_first = SPLIT ? (int)((int64_t)all_kt * blockIdx.z / gridDim.z) : 0;
    const int n_kt = (SPLIT ? (int)((int64_t)all_kt * (blockIdx.z + 1) / gridDim.z) : all_kt) - kt_first; // this workgroup's K-tiles
    auto fetch = [&](int kt) { // its K-tile kt (clamped to the last one) -> buffer kt & 3
        const int ktc = kt_first + min(kt, n_kt - 1);
        uint8_t *dst = lds + (kt & (NBUF - 1)) * STAGE + wave * 16 * PROWB;
#pragma unroll
        for (int t = 0; t < NLOAD; ++t)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[t] + (int64_t)ktc * PROWB),
                                             (__attribute__((address_space(3))) void *)(dst + t * 8 * 16 * PROWB), 16, 0, 0);
    };
    fetch(0);
    fetch(1);
    fetch(2);
    __builtin_amdgcn_s_waitcnt(WAIT_LANDED);
    __syncthreads();

    constexpr int GROUPS = 2 * MI, ROT = 5, RING = 4, AHEAD = 3;
    static_assert(MI % RING == 0 && ROT == 2 * AHEAD - 1 && ROT < GROUPS && NJ % 2 == 0, "group plan");
    v4u ap[RING], wp[NJ];
    v4i fa[2], fw[2][NJ];
#pragma unroll
    for (int k = 0; k < RING; ++k) ap[k] = v4u{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NJ; ++j) fw[0][j] = fw[1][j] = v4i{0, 0, 0, 0};
    fa[0] = fa[1] = v4i{0, 0, 0, 0};

    for (int kt = 0; kt < n_kt; ++kt) {
        const uint8_t *cur = lds + (kt & (NBUF - 1)) * STAGE;
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            const int s = (u + GROUPS - ROT) % GROUPS, i = s >> 1, m = s & 1;
            // the K-tile three ahead, into the buffer whose last reader passed the previous barrier
            if (s == 0) fetch(kt + 3);
            // the group's operations
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[m][j], fa[m], acc[i][j], 0, 0, 0);
            // splits for the next group: the other nibble of this row block, or the next block's low one
            if (m == 0) fa[1] = nib_hi(ap[i % RING]);
            else fa[0] = nib_lo(ap[(i + 1) % RING]);
            // feature side of the new K-tile: low nibbles once the last low group of the old one is
            // through (the last but one), high nibbles after its last high group (the last)
            if (s == GROUPS - 1) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) fw[0][j] = nib_lo(wp[j]);
            }
            if (s == 0) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) fw[1][j] = nib_hi(wp[j]);
            }
            if (u == GROUPS - 1) {
                // next K-tile landed (this wave's share; the barrier adds the others'), own reads done
                __builtin_amdgcn_s_waitcnt(WAIT_LANDED_LGKM0);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            // requests come after the split that had to wait for an earlier one, so that the wait
            // does not cover them: token rows three blocks ahead (after a high-nibble group), the
            // feature rows of this iteration's K-tile in its first two groups.  All of them read
            // this iteration's K-tile: the first group of the iteration is the first to look ahead.
            __builtin_amdgcn_sched_barrier(0);
            if (m == 1) ap[(i + AHEAD) % RING] = *reinterpret_cast<const v4u *>(cur + a_off + ((i + AHEAD) % MI) * 16 * PROWB);
            if (u < 2) {
#pragma unroll
                for (int h = 0; h < NJ / 2; ++h)
                    wp[(NJ / 2) * u + h] = *reinterpret_cast<const v4u *>(cur + w_off + ((NJ / 2) * u + h) * 16 * PROWB);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the loads past the last K-tile went to buffers nobody reads; they must not outlive the workgroup
    __builtin_amdgcn_s_waitcnt(WAIT_VM0);
    // the last groups of the last K-tile
#pragma unroll
    for (int s = GROUPS - ROT; s < GROUPS; ++s) {
        const int i = s >> 1, m = s & 1;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[m][j], fa[m], acc[i][j], 0, 0, 0);
        if (m == 0) fa[1] = nib_hi(ap[i % RING]);
        else if (i < MI - 1) fa[0] = nib_lo(ap[(i + 1) % RING]);
    }

    if constexpr (SPLIT) {
        // raw accumulators of this part of K: token n, four consecutive features per lane and tile
        int32_t *part = g.partial + (int64_t)blockIdx.z * g.N * g.O;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int n = n0 + wm * 16 * MI + i * 16 + (lane & 15);
            if (n >= g.N) continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int o = o0 + wn * 16 * NJ + j * 16 + 4 * (lane >> 4);
                int32_t *p = part + (int64_t)n * g.O + o;
                if (o + 3 < g.O && (g.O & 3) == 0) {
                    *reinterpret_cast<v4i *>(p) = acc[i][j];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o + e < g.O) p[e] = acc[i][j][e];
                }
            }
        }
    } else {
        finish_wave_tile<4, 4, YT, MI, NJ>(g, acc, n0 + wm * 16 * MI, o0 + wn * 16 * NJ, lane);
    }
}

// ---- epilogue of the kernels that leave room for its constants in LDS (EPI_BYTES behind the ring).  A wave that
// fetches them from global memory after its last K-tile waits for memory with nothing left to multiply, and the
// bracket written out term by term is three 24-bit multiply-adds per output; both count where K is short.
// With a' = a - 128 for 8-bit codes (else a), the same for w, and primed zero-points and sums to match,
//   bracket = sum (a' - bx')(w' - bw') = acc - bx' * cs' - bw' * (rs - K bx),     rs - K bx = sum (a - bx),
// two multiply-adds.  Taken when every zero-point of the tile lies among the codes, 0 <= beta <= qmax (a row or column
// that spans zero): then |rs - K bx| and |cs'| <= qmax K < 2^23 and the bracket is below qmax_a qmax_w K < 2^31, so
// 24-bit multiply-adds with wrapping 32-bit sums are exact.  Stores are 16 bytes per lane, 64 bytes of 16 rows each:
// with 8 bytes per lane (32 of 16 rows) the same tiles leave at 3.65 instead of 4.9 TB/s, which a short K does not hide
// (4096 x 5120 -> 27648: 318 -> 286 us; 2048 x 4096 -> 8192: 42.5 -> 39.2; odd widths, 777 x 5000 -> 4999 fp32: 41 -> 36).  On the FP6 path the same in floats: acc holds 1/64 of the
// accumulator, bx * cs / 64 and bw * (rs - K bx) / 64 are multiples of 1/64 below 225 K / 64 and every partial sum of
// the three terms, in the order they are added, is below 225 K / 64 < 2^24 / 64, hence exact; 64 goes into ax.
template <int TM, int TN>
constexpr int EPI_BYTES = TM * 16 + 3 * TN * 4 + 8 * 4;

// 16-byte stores at whatever alignment Y's rows have (any width and stride): one instruction, dword- or half-word-aligned
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int v4u_any __attribute__((ext_vector_type(4), aligned(2)));

// The constants on their way to LDS, one token's or one feature's per lane (at least TM + TN lanes, 4 or 8 waves).
struct EpiRegs {
    int32_t zero, sum;
    float scale;
};
template <int TM, int TN>
__device__ __forceinline__ EpiRegs load_epilogue(const GemmArgs &g, int n0, int o0, int tid)
{
    EpiRegs e{0, 0, 0.0f};
    if (tid < TM) {
        const int n = min(n0 + tid, g.N - 1);
        e.zero = g.bx[n]; e.sum = g.rs[n]; e.scale = g.ax[n];
    } else if (tid < TM + TN) {
        const int o = min(o0 + tid - TM, g.O - 1);
        e.zero = g.bw[o]; e.sum = g.cs[o]; e.scale = g.aw[o];
    }
    return e;
}

// A barrier must follow before finish_from_lds.
template <int ABITS, int WBITS, int TM, int TN, bool FP, int WAVES>
__device__ __forceinline__ void store_epilogue(const GemmArgs &g, const EpiRegs &e, uint8_t *epi, int tid)
{
    constexpr int QA = (1 << ABITS) - 1, QW = (1 << WBITS) - 1, SA = ABITS == 8 ? 128 : 0, SW = WBITS == 8 ? 128 : 0;
    uint32_t *tok = reinterpret_cast<uint32_t *>(epi), *feat = reinterpret_cast<uint32_t *>(epi + TM * 16);
    bool ok = g.lds_epilogue != 0;
    if (tid < TM) {
        ok = ok && e.zero >= 0 && e.zero <= QA && (!FP || e.scale < 1e30f);
        const int32_t rsk = e.sum - g.K * e.zero;
        v4i v{SA - e.zero, rsk, 0, 0};
        if constexpr (FP) v = v4i{__builtin_bit_cast(int, -(float)e.zero), __builtin_bit_cast(int, (float)rsk * (1.0f / 64.0f)), 0, 0};
        v[2] = __builtin_bit_cast(int, FP ? e.scale * 64.0f : e.scale);
        *reinterpret_cast<v4i *>(tok + 4 * tid) = v;
    } else if (tid < TM + TN) {
        const int f = tid - TM;
        const int32_t cs = e.sum - SW * g.K;
        ok = ok && e.zero >= 0 && e.zero <= QW;
        feat[f] = FP ? __float_as_uint((float)cs * (1.0f / 64.0f)) : (uint32_t)cs;
        feat[TN + f] = FP ? __float_as_uint(-(float)e.zero) : (uint32_t)(SW - e.zero);
        feat[2 * TN + f] = __float_as_uint(e.scale);
    }
    const bool all = __all(ok);
    if ((tid & 63) == 0)
#pragma unroll
        for (int k = 0; k < 8; k += WAVES) reinterpret_cast<int32_t *>(epi + TM * 16 + 3 * TN * 4)[k + (tid >> 6)] = all; // eight flags
}

// One wave tile from the constants in LDS; false: not taken (the caller falls back to finish_wave_tile).
// nl, ol: the wave's first token and feature inside the workgroup's tile.
template <typename YT, int TM, int TN, int NI, int NJ, typename ACC>
__device__ __forceinline__ bool finish_from_lds(const GemmArgs &g, const ACC (&acc)[NI][NJ], const uint8_t *epi, int n0, int o0,
                                                int nl, int ol, int lane)
{
    constexpr bool FP = std::is_same<ACC, v4f>::value;
    const v4i *flags = reinterpret_cast<const v4i *>(epi + TM * 16 + 3 * TN * 4);
    const v4i f0 = flags[0], f1 = flags[1];
    if (!__builtin_amdgcn_readfirstlane(f0[0] & f0[1] & f0[2] & f0[3] & f1[0] & f1[1] & f1[2] & f1[3])) return false;
    typedef typename std::conditional<FP, v4f, v4i>::type V;
    const uint8_t *feat = epi + TM * 16;
    const int oq = 4 * (lane >> 4);
    V cs[NJ], nbw[NJ];
    v4f aw[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        cs[j] = *reinterpret_cast<const V *>(feat + 4 * (ol + 16 * j + oq));
        nbw[j] = *reinterpret_cast<const V *>(feat + 4 * (TN + ol + 16 * j + oq));
        aw[j] = *reinterpret_cast<const v4f *>(feat + 4 * (2 * TN + ol + 16 * j + oq));
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int nt = nl + 16 * i + (lane & 15), n = n0 + nt;
        const V c = *reinterpret_cast<const V *>(epi + 16 * nt);
        const auto third = c[2]; // a value of its own: the compiler's bit cast of a vector's element takes the first one
        const float ax = __builtin_bit_cast(float, third);
        const bool row = n < g.N;
        auto value = [&](int j, int r) {
            float v;
            if constexpr (FP) {
                v = __builtin_fmaf(c[0], cs[j][r], acc[i][j][r]);
                v = __builtin_fmaf(c[1], nbw[j][r], v);
            } else {
                int32_t s = acc[i][j][r] + __mul24(c[0], cs[j][r]);
                s += __mul24(c[1], nbw[j][r]);
                v = (float)s;
            }
            return (v * ax) * aw[j][r];
        };
        if constexpr (sizeof(YT) == 4) {
            const int64_t at = (int64_t)n * g.ldy + o0 + ol + oq;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const v4f out{value(j, 0), value(j, 1), value(j, 2), value(j, 3)};
                float *const yp = reinterpret_cast<float *>(g.y) + at + 16 * j;
                const int left = row ? g.O - (o0 + ol + 16 * j + oq) : 0;
                if (left >= 4) {
                    *reinterpret_cast<v4f_any *>(yp) = out;
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (e < left) yp[e] = out[e];
                }
            }
        } else {
            // a lane's four features of tile j and of tile j + 1 are 8 bytes each; rows of 16 lanes trade them so that
            // every lane stores 8 neighbouring features of one tile
            const int q = lane >> 4, half = 16 * (q & 1) + 8 * (q >> 1);
            const int64_t at = (int64_t)n * g.ldy + o0 + ol + half;
#pragma unroll
            for (int j = 0; j < NJ; j += 2) {
                const auto lo = __builtin_amdgcn_permlane16_swap(f32x2_to_bf16x2_rne(value(j, 0), value(j, 1)),
                                                                 f32x2_to_bf16x2_rne(value(j + 1, 0), value(j + 1, 1)), false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(f32x2_to_bf16x2_rne(value(j, 2), value(j, 3)),
                                                                 f32x2_to_bf16x2_rne(value(j + 1, 2), value(j + 1, 3)), false, false);
                const uint32_t out[4] = {lo[0], hi[0], lo[1], hi[1]};
                uint16_t *const yp = reinterpret_cast<uint16_t *>(g.y) + at + 16 * j;
                const int left = row ? g.O - (o0 + ol + 16 * j + half) : 0;
                if (left >= 8) {
                    *reinterpret_cast<v4u_any *>(yp) = v4u{out[0], out[1], out[2], out[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 7; ++e)
                        if (e < left) yp[e] = (uint16_t)(out[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
    }
    return true;
}

// Which tile of Y a workgroup of a large product takes.  Workgroups go to the eight XCDs in turn by their number, and
// an XCD's workgroups share its L2: tiles are handed out so that each XCD walks a run of neighbouring tiles, down
// bands of up to eight tiles of tokens and then along the features, and its 32 resident workgroups share
// 8 + 4 operand streams whatever the grid's width is (4096 x 5120 -> 27648, 108 tiles wide: up to 30 streams in row
// order, 335 us; 318 so).  Large tiles only: 128 x 128 tiles, two workgroups per CU, lost by it (777 x 5000 -> 4999 with
// 8-bit activations 41.5 -> 45.3 us, 2048 x 4096 -> 4096 30.8 -> 32.1).
struct TileAt {
    int n, o;
};
__device__ __forceinline__ TileAt tile_at(int nb, int ob)
{
    const uint32_t b = blockIdx.y * gridDim.x + blockIdx.x, total = (uint32_t)nb * (uint32_t)ob, xcd = b & 7u;
    const uint32_t t = xcd * (total >> 3) + min(xcd, total & 7u) + (b >> 3);
    const uint32_t bands = ((uint32_t)nb + 7u) >> 3, height = ((uint32_t)nb + bands - 1u) / bands;
    const uint32_t band = t / (height * (uint32_t)ob), r = t - band * height * (uint32_t)ob, first = band * height;
    const uint32_t h = min(height, (uint32_t)nb - first), o = r / h;
    return TileAt{__builtin_amdgcn_readfirstlane((int)(first + r - o * h)), __builtin_amdgcn_readfirstlane((int)o)};
}

// ---- 4-bit codes on both sides on the FP6 matrix cores.
// gfx950 multiplies 6-bit floating-point operands (E2M3: sign, 2 exponent bits, 3 mantissa bits, no
// infinities or NaNs) at twice the rate of int8, 128 values of K per operation.  The 6-bit pattern
// 00cccc, a 4-bit code c zero-extended, IS the E2M3 number c / 8 (exponent field 0: c / 8 for c < 8;
// exponent field 1: (8 + (c - 8)) / 8), so the product of two codes is a * w / 64 exactly, and the
// fp32 accumulation is exact as well: every partial sum, whatever the order and grouping the hardware
// adds in, is a multiple of 1/64 below 225 K / 64 < 2^24 / 64 (K < 74565; the entry point allows
// 32768), hence a representable fp32 number, so no addition ever rounds.  64 acc is the int32
// accumulator of Eq. (1), bit for bit.
//
// TILES6, the operand format (made once per weight by qllm_pack_tiles6, per call for the activations, whose blocks hold
// the same bytes in another order, see tiles6_x in fused_common.h):
// rows in blocks of 16, K in tiles of 128 codes; block b, K-tile t is the 1536 bytes at
// (b * tiles + t) * 1536 and holds what the 64 lanes of one operand read need, lane l = 16 q + r having
// row 16 b + r and codes 128 t + 32 q + e, e = 0..31, code e in bits 6 e .. 6 e + 3 of a 192-bit
// little-endian number: its first 16 bytes at 16 l, its last 8 at 1024 + 8 l.  Rows past the matrix
// are zero codes.  A stage of LDS is such blocks one after the other exactly as they lie in memory,
// so the refill is a plain copy (16-byte loads that write LDS directly) and both operand reads
// (ds_read_b128 of 1 KB, ds_read_b64 of 512 bytes per wave) are contiguous: no bank conflicts, and no
// vector instruction between LDS and the matrix cores.
//
// Same tiling as the int8 kernel above (2 x 4 waves, MI x NJ operations of 16 x 16 per wave and
// K-tile), a ring of three stages (48 KB each for the 256 x 256 tile), fetches two K-tiles ahead.
// One K-tile = MI groups of NJ operations (group i: token rows 16 i ..); the loop is rotated by AHEAD groups (an
// iteration starts with the last groups of the K-tile before, zeros the first time) and unrolled by two, so
// that the alternation of the two feature-side register sets is static; KTilePlan has the order of reads and loads.
typedef int v8i __attribute__((ext_vector_type(8)));
constexpr int T6_BLOCK = qllm_detail::TILES6_BLOCK, T6_X = qllm_detail::TILES6_X, T6_KT = 128, T6_STAGES = 3;

typedef int v2i __attribute__((ext_vector_type(2)));
struct Frag6 {
    v4i x;
    v2i y;
};
__device__ __forceinline__ v8i operand6(const Frag6 &f) { return v8i{f.x[0], f.x[1], f.x[2], f.x[3], f.y[0], f.y[1], 0, 0}; }
__device__ __forceinline__ Frag6 read6(const uint8_t *block, int x, int y)
{
    Frag6 f;
    f.x = *reinterpret_cast<const v4i *>(block + x);
    f.y = *reinterpret_cast<const v2i *>(block + y);
    return f;
}

// What a wave issues behind which of a K-tile's MI * NJ matrix-core operations, in gemm_w4a4_fp6_kernel and gemm_tiles8_kernel.
// The first AHEAD groups of NJ finish the K-tile before, so they need nothing of this one: its operands are read behind
// them, one block behind an operation, the feature side first, and the matrix cores run from the barrier on.  (All
// reads of a K-tile's first groups in front of the first operation: eight waves' reads keep the LDS busy for some 300 of
// the K-tile's 1500 clocks before any of them multiplies.)  The large tile reads a token-side block behind every other
// operation and loads behind every third from the middle on (a load the CU's address unit has not accepted yet holds its
// wave up).  With the copies of lds_copy.h, kernel traces on one card, us, before both : now: FP6 2048 x 28672 -> 8192 185.4 : 181.3,
// 4096 x 5120 -> 27648 283.4 : 278.1, 2048 x 4096 -> 8192 of 12288 39.8 : 39.9; bytes, 6-bit 2048 x 28672 -> 8192 302 : 281, small tiles
// 777 x 5000 -> 4999 37.4 : 35.0, with K split 200 x 13824 -> 5120 26.7 : 26.2; qllm_int_gemm, small tiles of 300-2048 tokens, 4096-28672
// channels: bytes 3-16 % faster, FP6 within 2 % either way.  Where the token-side reads go (every operation, second, third)
// changes nothing any more: in clocks the large tiles are at 0.78 (FP6) and 0.88 (int8) of the same loop without reads and
// loads; the clock under this load is 1.96-2.05 GHz (2.45 on operands of zeros).
template <int MI, int NJ>
struct KTilePlan {
    static constexpr int AHEAD = 2, STEPS = MI * NJ;
    static constexpr int READ_STEP = MI == 8 ? 2 : 1, FIRST_LOAD = MI == 8 ? 14 : NJ - 1, LOAD_STEP = MI == 8 ? 3 : NJ;
    static constexpr int MOST_LOADS = (STEPS - 1 - FIRST_LOAD) / LOAD_STEP + 1;
    // a block's registers are free once the operations on the K-tile before that read them are behind: the last
    // AHEAD blocks are read after step AHEAD * NJ, and every one before its own first use (step (AHEAD + b) * NJ)
    static_assert(NJ + (MI - AHEAD) * READ_STEP >= AHEAD * NJ - 1 && NJ <= AHEAD * NJ && NJ + (MI - 1) * READ_STEP < STEPS, "order of reads");
    static constexpr int feature_read(int s) { return s < NJ ? s : -1; }
    static constexpr int token_read(int s) { return s >= NJ && (s - NJ) % READ_STEP == 0 && (s - NJ) / READ_STEP < MI ? (s - NJ) / READ_STEP : -1; }
    static constexpr int load(int s, int n) { return s >= FIRST_LOAD && (s - FIRST_LOAD) % LOAD_STEP == 0 && (s - FIRST_LOAD) / LOAD_STEP < n ? (s - FIRST_LOAD) / LOAD_STEP : -1; }
};

// SPLIT: K is dealt out to gridDim.z workgroups per tile of Y, as in int_gemm_w4a4_kernel; the parts' sums leave as
// the integers they stand for.
template <typename YT, int MI, int NJ, bool SPLIT = false>
__global__ __launch_bounds__(LTHREADS, MI == 8 ? 1 : 2) void gemm_w4a4_fp6_kernel(const GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int TM = 2 * MI * 16, TN = 4 * NJ * 16;
    constexpr int BLOCKS = (TM + TN) / 16, STAGE = BLOCKS * T6_BLOCK, NLOAD = STAGE / (8 * 1024);
    static_assert(STAGE % (8 * 1024) == 0, "a stage is a whole number of 1 KB loads per wave");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const TileAt at = MI < 8 ? TileAt{(int)blockIdx.y, (int)blockIdx.x} : tile_at((int)gridDim.y, (int)gridDim.x);
    const int n0 = at.n * TM, o0 = g.o_first + at.o * TN;
    const int all_kt = g.Kpad / T6_KT;
    const int a_blocks = (g.N + 15) / 16, w_blocks = (g.O + 15) / 16;

    // fetch assignment: load t of wave w fills bytes 1024 (NLOAD w + t) .. of the stage, lane l its l-th 16.  The
    // token side of a stage is a whole number of such loads, so a load is all token side or all feature side: one
    // base for the wave, a 32-bit offset per lane that never changes (the K-tile moves the base).
    uint32_t src_off[NLOAD];
#pragma unroll
    for (int t = 0; t < NLOAD; ++t) {
        const int off = (wave * NLOAD + t) * 1024 + lane * 16, blk = off / T6_BLOCK, within = off % T6_BLOCK;
        const bool token = blk < TM / 16; // past the edge: the last block again (its results are not stored)
        const int rb = token ? min(n0 / 16 + blk, a_blocks - 1) : min(o0 / 16 + blk - TM / 16, w_blocks - 1);
        src_off[t] = (uint32_t)rb * (uint32_t)all_kt * T6_BLOCK + within;
    }
    static_assert((TM / 16 * T6_BLOCK) % 1024 == 0, "token side = whole loads");
    // load t of K-tile kt (clamped to the last one) -> that stage of the ring
    auto fetch_one = [&](int kt, int stage, int t) {
        const int ktc = min(kt, all_kt - 1);
        const bool token = (wave * NLOAD + t) * 1024 < TM / 16 * T6_BLOCK;
        qllm_detail::copy_1k_to_lds(token ? g.a_tiles : g.w_tiles, (uint32_t)(token ? a_blocks : w_blocks) * (uint32_t)all_kt * T6_BLOCK,
                                    src_off[t], (uint32_t)ktc * T6_BLOCK, lds + stage * STAGE + (wave * NLOAD + t) * 1024);
    };
    auto fetch = [&](int kt, int stage) {
#pragma unroll
        for (int t = 0; t < NLOAD; ++t) fetch_one(kt, stage, t);
    };
    constexpr int WAIT_LANDED = NLOAD | (7 << 4) | (15 << 8);       // s_waitcnt vmcnt(NLOAD): all but the newest fetch
    constexpr int WAIT_LANDED_LGKM0 = NLOAD | (7 << 4) | (0 << 8);  // ... and lgkmcnt(0)

    v4f acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // this workgroup's K-tiles (fetches past them, up to the last K-tile of the row, go to stages nobody reads)
    const int kt_first = SPLIT ? (int)((int64_t)all_kt * blockIdx.z / gridDim.z) : 0;
    const int kt_end = SPLIT ? (int)((int64_t)all_kt * (blockIdx.z + 1) / gridDim.z) : all_kt;
    uint8_t *const epi = lds + T6_STAGES * STAGE; // the epilogue's constants, behind the ring
    if constexpr (!SPLIT) store_epilogue<4, 4, TM, TN, true, 8>(g, load_epilogue<TM, TN>(g, n0, o0, tid), epi, tid);
    fetch(kt_first, 0);
    fetch(kt_first + 1, 1);
    __builtin_amdgcn_s_waitcnt(WAIT_LANDED);
    __syncthreads();

    // Token-side operands: all MI blocks of a K-tile have registers of their own.
    typedef KTilePlan<MI, NJ> Plan;
    constexpr int AHEAD = Plan::AHEAD;
    static_assert(NLOAD <= Plan::MOST_LOADS, "every load of a K-tile has its place");
    Frag6 ar[MI], wr[2][NJ];
#pragma unroll
    for (int k = 0; k < MI; ++k) ar[k] = Frag6{v4i{0, 0, 0, 0}, v2i{0, 0}};
#pragma unroll
    for (int j = 0; j < NJ; ++j) wr[0][j] = wr[1][j] = Frag6{v4i{0, 0, 0, 0}, v2i{0, 0}};

    const int a_blk0 = wm * MI, w_blk0 = TM / 16 + wn * NJ; // the wave's first token-side and feature-side block of a stage
    const int a_x = qllm_detail::tiles6_x(lane & 15, lane >> 4), a_y = qllm_detail::tiles6_y(lane & 15, lane >> 4);
    int stage = 0, fetch_stage = 2;
    // one K-tile, P = which feature-side register set it reads into (the other one still serves the
    // AHEAD groups left of the K-tile before)
    auto k_tile = [&](auto parity, int kt) {
        constexpr int P = decltype(parity)::value;
        const uint8_t *cur = lds + stage * STAGE;
#pragma unroll
        for (int u = 0; u < MI; ++u) {
            const bool old = u < AHEAD;
            const int i = old ? MI - AHEAD + u : u - AHEAD;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int s = u * NJ + j;
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand6(wr[old ? 1 - P : P][j]), operand6(ar[i]),
                                                                             acc[i][j], 2, 2, 0, 0, 0, 0);
                if (Plan::feature_read(s) >= 0) wr[P][Plan::feature_read(s)] = read6(cur + (w_blk0 + Plan::feature_read(s)) * T6_BLOCK, 16 * lane, T6_X + 8 * lane);
                if (Plan::token_read(s) >= 0) ar[Plan::token_read(s)] = read6(cur + (a_blk0 + Plan::token_read(s)) * T6_BLOCK, a_x, a_y);
                // the K-tile two ahead, into the stage whose last reader passed the previous barrier
                if (Plan::load(s, NLOAD) >= 0) fetch_one(kt + 2, fetch_stage, Plan::load(s, NLOAD));
                __builtin_amdgcn_sched_barrier(0); // this order is the order issued; also keeps the 8-byte reads of neighbouring blocks apart
            }
        }
        // the next K-tile has landed (this wave's share; the barrier adds the others'), own reads done
        __builtin_amdgcn_s_waitcnt(WAIT_LANDED_LGKM0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch_stage = stage;
        stage = stage == T6_STAGES - 1 ? 0 : stage + 1;
    };
    int kt = kt_first;
    for (; kt + 1 < kt_end; kt += 2) {
        k_tile(std::integral_constant<int, 0>{}, kt);
        k_tile(std::integral_constant<int, 1>{}, kt + 1);
    }
    if (kt < kt_end) k_tile(std::integral_constant<int, 0>{}, kt);
    // the loads past the last K-tile went to stages nobody reads; they must not outlive the workgroup
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
    // the last groups of the last K-tile
    auto last_groups = [&](auto parity) {
        constexpr int P = decltype(parity)::value;
#pragma unroll
        for (int i = MI - AHEAD; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand6(wr[P][j]), operand6(ar[i]), acc[i][j], 2, 2,
                                                                             0, 0, 0, 0);
    };
    if ((kt_end - kt_first) & 1) last_groups(std::integral_constant<int, 0>{});
    else last_groups(std::integral_constant<int, 1>{});

    if constexpr (SPLIT) {
        // this part's sums as integers (64 acc, exactly): token n, four consecutive features per lane and tile
        int32_t *part = g.partial + (int64_t)blockIdx.z * g.N * g.O;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int n = n0 + wm * 16 * MI + i * 16 + (lane & 15);
            if (n >= g.N) continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int o = o0 + wn * 16 * NJ + j * 16 + 4 * (lane >> 4);
                int32_t *p = part + (int64_t)n * g.O + o;
                const v4i v{acc_int(acc[i][j], 0), acc_int(acc[i][j], 1), acc_int(acc[i][j], 2), acc_int(acc[i][j], 3)};
                if (o + 3 < g.O && (g.O & 3) == 0) {
                    *reinterpret_cast<v4i *>(p) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o + e < g.O) p[e] = v[e];
                }
            }
        }
    } else {
        if (finish_from_lds<YT, TM, TN>(g, acc, epi, n0, o0, wm * 16 * MI, wn * 16 * NJ, lane)) return;
        finish_wave_tile<4, 4, YT, MI, NJ>(g, acc, n0 + wm * 16 * MI, o0 + wn * 16 * NJ, lane); // 64 acc: the integer accumulators, exactly
    }
}

// Packed 4-bit rows -> TILES6; one lane per (block, K-tile, lane of the operand read).  BY_ROW: as activations lie.
template <bool BY_ROW>
__global__ __launch_bounds__(256) void tiles6_kernel(const uint8_t *codes, int64_t row_bytes, int32_t rows, int32_t n_kt,
                                                    uint8_t *tiles, int64_t n_items)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_items) return;
    const int l = (int)(idx & 63), r = l & 15, q = l >> 4;
    const int64_t bk = idx >> 6, b = bk / n_kt;
    const int kt = (int)(bk - b * n_kt);
    const int64_t row = b * 16 + r;
    uint4 p = make_uint4(0u, 0u, 0u, 0u);
    if (row < rows) p = *reinterpret_cast<const uint4 *>(codes + row * row_bytes + kt * (T6_KT / 2) + q * 16);
    const qllm_detail::Lane6 v = qllm_detail::lane6(p);
    uint8_t *blk = tiles + bk * T6_BLOCK;
    *reinterpret_cast<uint4 *>(blk + (BY_ROW ? qllm_detail::tiles6_x(r, q) : 16 * l)) = v.x;
    *reinterpret_cast<uint2 *>(blk + (BY_ROW ? qllm_detail::tiles6_y(r, q) : T6_X + 8 * l)) = v.y;
}

// ---- 6- and 8-bit codes (and 8-bit activations on 4-bit weights) straight from LDS into the int8 matrix cores.
// TILES8, the operand format (made once per weight by qllm_pack_tiles8, per call for the activations): one byte
// per code, rows in blocks of 16, K in tiles of 64 codes; block b, K-tile t is the 1024 bytes at
// (b * tiles + t) * 1024 and holds what the 64 lanes of one operand read need: lane l = 16 q + r has row
// 16 b + r and codes 64 t + 16 q + e, e = 0..15, at byte 16 l + e.  A 4- or 6-bit code is its own value; an 8-bit
// code c is stored as c ^ 0x80, the signed byte c - 128 (the epilogue adds the difference back).  Rows past the
// matrix and places past K are zero bytes: they add nothing.  As with TILES6 a stage of LDS is such blocks as
// they lie in memory, the refill a plain copy by 16-byte loads that write LDS directly, an operand read one
// contiguous ds_read_b128 per wave, and there is no vector instruction between LDS and the matrix cores (the
// kernels that expand packed codes at refill time spend most of their issue slots on that).
// Tiling, ring, group plan and loop rotation are those of gemm_w4a4_fp6_kernel; one K-tile here is 64 codes,
// which takes the int8 matrix cores as long as 128 codes take the FP6 ones.
constexpr int T8_BLOCK = 1024, T8_KT = 64;


// SPLIT: K is dealt out to gridDim.z workgroups per tile of Y (so few tiles that most CUs would idle); each writes
// its raw accumulators to g.partial and splitk_finish_kernel adds them up and does the epilogue.
// STAGES of the ring: three; four for the small tile where there is at most one workgroup per CU, which then waits for
// memory (200 tokens, 13824 -> 5120 6 / 6 with K split in three: 32.7 -> 27.2 us; six change nothing more).  With two
// workgroups per CU the fourth costs (2171 x 8832 -> 3712: 135 -> 144), for the large tile it changes nothing.
template <int ABITS, int WBITS, typename YT, int MI, int NJ, int STAGES, bool SPLIT = false>
__global__ __launch_bounds__(LTHREADS, MI == 8 ? 1 : 2) void gemm_tiles8_kernel(const GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int TM = 2 * MI * 16, TN = 4 * NJ * 16;
    constexpr int BLOCKS = (TM + TN) / 16, STAGE = BLOCKS * T8_BLOCK, NLOAD = STAGE / (8 * 1024);
    static_assert(STAGE % (8 * 1024) == 0 && NLOAD <= MI, "a stage is a whole number of 1 KB loads per wave, one per group");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const TileAt at = MI < 8 ? TileAt{(int)blockIdx.y, (int)blockIdx.x} : tile_at((int)gridDim.y, (int)gridDim.x);
    const int n0 = at.n * TM, o0 = g.o_first + at.o * TN;
    const int all_kt = (g.K + T8_KT - 1) / T8_KT;
    const int a_blocks = (g.N + 15) / 16, w_blocks = (g.O + 15) / 16;

    // fetch assignment: load t of wave w fills block NLOAD w + t of the stage, lane l its l-th 16 bytes; a load is
    // all token side or all feature side: one base for the wave, a 32-bit offset per lane that never changes
    uint32_t src_off[NLOAD];
#pragma unroll
    for (int t = 0; t < NLOAD; ++t) {
        const int blk = wave * NLOAD + t;
        const bool token = blk < TM / 16; // past the edge: the last block again (its results are not stored)
        const int rb = token ? min(n0 / 16 + blk, a_blocks - 1) : min(o0 / 16 + blk - TM / 16, w_blocks - 1);
        src_off[t] = (uint32_t)rb * (uint32_t)all_kt * T8_BLOCK + lane * 16;
    }
    auto fetch_one = [&](int kt, int stage, int t) { // load t of K-tile kt (clamped to the last one) -> that stage
        const int ktc = min(kt, all_kt - 1);
        const bool token = wave * NLOAD + t < TM / 16;
        qllm_detail::copy_1k_to_lds(token ? g.a_tiles8 : g.w_tiles8, (uint32_t)(token ? a_blocks : w_blocks) * (uint32_t)all_kt * T8_BLOCK,
                                    src_off[t], (uint32_t)ktc * T8_BLOCK, lds + stage * STAGE + (wave * NLOAD + t) * 1024);
    };
    auto fetch = [&](int kt, int stage) {
#pragma unroll
        for (int t = 0; t < NLOAD; ++t) fetch_one(kt, stage, t);
    };
    constexpr int IN_FLIGHT = (STAGES - 2) * NLOAD; // loads of the K-tiles after the next one
    constexpr int WAIT_LANDED = IN_FLIGHT | (7 << 4) | (15 << 8);       // s_waitcnt vmcnt(IN_FLIGHT): the next K-tile has landed
    constexpr int WAIT_LANDED_LGKM0 = IN_FLIGHT | (7 << 4) | (0 << 8);  // ... and lgkmcnt(0)
    static_assert(IN_FLIGHT < 16, "the low four bits of vmcnt");

    v4i acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // this workgroup's K-tiles (fetches past them, up to the last K-tile of the row, go to stages nobody reads)
    const int kt_first = SPLIT ? (int)((int64_t)all_kt * blockIdx.z / gridDim.z) : 0;
    const int kt_end = SPLIT ? (int)((int64_t)all_kt * (blockIdx.z + 1) / gridDim.z) : all_kt;
    uint8_t *const epi = lds + STAGES * STAGE; // the epilogue's constants, behind the ring
    if constexpr (!SPLIT) store_epilogue<ABITS, WBITS, TM, TN, false, 8>(g, load_epilogue<TM, TN>(g, n0, o0, tid), epi, tid);
    fetch(kt_first, 0);
#pragma unroll
    for (int s = 1; s < STAGES - 1; ++s) fetch(kt_first + s, s);
    __builtin_amdgcn_s_waitcnt(WAIT_LANDED);
    __syncthreads();

    typedef KTilePlan<MI, NJ> Plan;
    constexpr int AHEAD = Plan::AHEAD;
    static_assert(NLOAD <= Plan::MOST_LOADS, "every load of a K-tile has its place");
    v4i ar[MI], wr[2][NJ];
#pragma unroll
    for (int k = 0; k < MI; ++k) ar[k] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NJ; ++j) wr[0][j] = wr[1][j] = v4i{0, 0, 0, 0};

    const int a_blk0 = wm * MI, w_blk0 = TM / 16 + wn * NJ; // the wave's first token-side and feature-side block of a stage
    int stage = 0, fetch_stage = STAGES - 1;
    auto k_tile = [&](auto parity, int kt) {
        constexpr int P = decltype(parity)::value;
        const uint8_t *cur = lds + stage * STAGE;
        auto operand = [&](int blk) { return *reinterpret_cast<const v4i *>(cur + blk * T8_BLOCK + 16 * lane); };
#pragma unroll
        for (int u = 0; u < MI; ++u) {
            const bool old = u < AHEAD;
            const int i = old ? MI - AHEAD + u : u - AHEAD;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int s = u * NJ + j;
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[old ? 1 - P : P][j], ar[i], acc[i][j], 0, 0, 0);
                if (Plan::feature_read(s) >= 0) wr[P][Plan::feature_read(s)] = operand(w_blk0 + Plan::feature_read(s));
                if (Plan::token_read(s) >= 0) ar[Plan::token_read(s)] = operand(a_blk0 + Plan::token_read(s));
                if (Plan::load(s, NLOAD) >= 0) fetch_one(kt + STAGES - 1, fetch_stage, Plan::load(s, NLOAD));
                __builtin_amdgcn_sched_barrier(0); // this order is the order issued
            }
        }
        // the next K-tile has landed (this wave's share; the barrier adds the others'), own reads done
        __builtin_amdgcn_s_waitcnt(WAIT_LANDED_LGKM0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch_stage = stage;
        stage = stage == STAGES - 1 ? 0 : stage + 1;
    };
    int kt = kt_first;
    for (; kt + 1 < kt_end; kt += 2) {
        k_tile(std::integral_constant<int, 0>{}, kt);
        k_tile(std::integral_constant<int, 1>{}, kt + 1);
    }
    if (kt < kt_end) k_tile(std::integral_constant<int, 0>{}, kt);
    // the loads past the last K-tile went to stages nobody reads; they must not outlive the workgroup
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
    auto last_groups = [&](auto parity) { // the last groups of the last K-tile
        constexpr int P = decltype(parity)::value;
#pragma unroll
        for (int i = MI - AHEAD; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[P][j], ar[i], acc[i][j], 0, 0, 0);
    };
    if ((kt_end - kt_first) & 1) last_groups(std::integral_constant<int, 0>{});
    else last_groups(std::integral_constant<int, 1>{});

    if constexpr (SPLIT) {
        // raw accumulators of this part of K: token n, four consecutive features per lane and tile
        int32_t *part = g.partial + (int64_t)blockIdx.z * g.N * g.O;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int n = n0 + wm * 16 * MI + i * 16 + (lane & 15);
            if (n >= g.N) continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int o = o0 + wn * 16 * NJ + j * 16 + 4 * (lane >> 4);
                int32_t *p = part + (int64_t)n * g.O + o;
                if (o + 3 < g.O && (g.O & 3) == 0) {
                    *reinterpret_cast<v4i *>(p) = acc[i][j];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o + e < g.O) p[e] = acc[i][j][e];
                }
            }
        }
    } else {
        // places past K are zero bytes on both sides, so only the K real places carry the two offsets of 128
        if (finish_from_lds<YT, TM, TN>(g, acc, epi, n0, o0, wm * 16 * MI, wn * 16 * NJ, lane)) return;
        finish_wave_tile<ABITS, WBITS, YT, MI, NJ>(g, acc, n0 + wm * 16 * MI, o0 + wn * 16 * NJ, lane, g.K);
    }
}

// ---- mid-size batches: one round of workgroups, each with two halves that sum alternate K-tiles.
// Tiles of 32 MI tokens x 32 NJ features of Y, so that a product too large for the streaming kernel and too small to fill
// rounds of the tiles above is one workgroup per CU (plan_mid6, plan_mid8).  Waves 0..3 (2 x 2, 16 MI x 16 NJ each) work on the
// first K-tile of a step and waves 4..7 on the second; at the end each half finishes half of the tile's tokens and gets the other
// half's sums of them through LDS.  Against one K-tile per barrier and eight waves over the tile this halves the barriers and takes
// a third off the operand reads; against K split over workgroups it writes no partial sums and needs no second launch.
// What bounds it is the way of the operands into LDS: loads alone take 0.9 to 1.0 of its time.  Copies of it with parts of the loop left out,
// us: all; without loads; without operand reads; without either; loads alone (/: weights out of every cache, else three sets in turn):
//   256 x 8192 -> 8192 8/4 22.3; 17.2; 21.5; 13.1; 21.4 / 31.5; 17.9; 31.2; 13.9; 31.2     600 x 28672 -> 8192 8/8 143; 108; 140; 77; 139
//   200 x 5120 -> 5120 4/4 12.1; 9.9; 11.8; 7.9; 11.6 / 16.2; 10.5; 15.9; 8.5; 15.8        400 x 28672 -> 8192 4/4 75; 46; 72; 33; 72
// At the first shape that is 74 / 50 GB/s into the LDS of a CU, each line counted for every CU that asks for it (3.2 / 2.2 TB/s of
// different bytes over the chip).  A ring deeper than four stages changes nothing, and lines asked for ahead hold up the loads
// behind them.
// Operands are read a step ahead of their operations: two sets of registers, a step reads one and multiplies the other.
struct MidBytes { // TILES8 on both sides, int8 matrix cores
    typedef v4i Acc;
    typedef v4i Frag;
    static constexpr int KT = T8_KT, BLOCK = T8_BLOCK;
    static constexpr bool FP = false;
    static __device__ __forceinline__ Frag zero() { return v4i{0, 0, 0, 0}; }
    static __device__ __forceinline__ const uint8_t *tokens(const GemmArgs &g) { return g.a_tiles8; }
    static __device__ __forceinline__ const uint8_t *features(const GemmArgs &g) { return g.w_tiles8; }
    static __device__ __forceinline__ int k_tiles(const GemmArgs &g) { return (g.K + KT - 1) / KT; }
    static __device__ __forceinline__ Frag token(const uint8_t *block, int lane) { return *reinterpret_cast<const v4i *>(block + 16 * lane); }
    static __device__ __forceinline__ Frag feature(const uint8_t *block, int lane) { return token(block, lane); }
    static __device__ __forceinline__ Acc multiply(const Frag &w, const Frag &a, const Acc &c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(w, a, c, 0, 0, 0); }
};

struct MidFp6 { // TILES6 on both sides, FP6 matrix cores
    typedef v4f Acc;
    typedef Frag6 Frag;
    static constexpr int KT = T6_KT, BLOCK = T6_BLOCK;
    static constexpr bool FP = true;
    static __device__ __forceinline__ Frag zero() { return Frag6{v4i{0, 0, 0, 0}, v2i{0, 0}}; }
    static __device__ __forceinline__ const uint8_t *tokens(const GemmArgs &g) { return g.a_tiles; }
    static __device__ __forceinline__ const uint8_t *features(const GemmArgs &g) { return g.w_tiles; }
    static __device__ __forceinline__ int k_tiles(const GemmArgs &g) { return g.Kpad / KT; }
    static __device__ __forceinline__ Frag token(const uint8_t *block, int lane)
    {
        return read6(block, qllm_detail::tiles6_x(lane & 15, lane >> 4), qllm_detail::tiles6_y(lane & 15, lane >> 4));
    }
    static __device__ __forceinline__ Frag feature(const uint8_t *block, int lane) { return read6(block, 16 * lane, T6_X + 8 * lane); }
    static __device__ __forceinline__ Acc multiply(const Frag &w, const Frag &a, const Acc &c)
    {
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand6(w), operand6(a), c, 2, 2, 0, 0, 0, 0);
    }
};

template <class OP, int MI, int NJ, int STAGES>
constexpr size_t mid_lds()
{
    constexpr int ring = STAGES * 2 * 2 * (MI + NJ) * OP::BLOCK, sums = 8 * ((MI + 1) / 2) * NJ * 1024;
    return (size_t)(ring > sums ? ring : sums) + EPI_BYTES<32 * MI, 32 * NJ>;
}

template <class OP, int ABITS, int WBITS, typename YT, int MI, int NJ, int STAGES>
__global__ __launch_bounds__(LTHREADS, 1) void gemm_mid_kernel(const GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    typedef typename OP::Acc Acc;
    constexpr int TM = 32 * MI, TN = 32 * NJ, BLOCKS = 2 * (MI + NJ);
    constexpr int HALF = BLOCKS * OP::BLOCK, STAGE = 2 * HALF, UNITS = HALF / 1024, NLOAD = (UNITS + 3) / 4;
    static_assert(HALF % 1024 == 0 && 2 * MI * OP::BLOCK % 1024 == 0, "a load of 1 KB is all token side or all feature side");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    // gridDim.x is a multiple of eight, so that the tiles of the same features run on one XCD; 64-feature tiles go there in
    // pairs, as the 128-feature columns do whose weights the layer call reads ahead
    const int x = blockIdx.x, n0 = blockIdx.y * TM, o0 = (NJ == 2 ? 2 * (8 * (x >> 4) + (x & 7)) + (x >> 3 & 1) : x) * TN;
    if (o0 >= g.O) return;
    const int all_kt = OP::k_tiles(g), steps = (all_kt + 1) / 2;
    const int a_blocks = (g.N + 15) / 16, w_blocks = (g.O + 15) / 16;

    // fetch assignment: the four waves of a half bring in its K-tile, load t of wave w its KB NLOAD (w & 3) + t (the last KB
    // again where the waves have more loads than there are), lane l the l-th 16 bytes of it
    uint32_t src_off[NLOAD];
#pragma unroll
    for (int t = 0; t < NLOAD; ++t) {
        const int off = min((wave & 3) * NLOAD + t, UNITS - 1) * 1024 + lane * 16, blk = off / OP::BLOCK, within = off % OP::BLOCK;
        const int rb = blk < 2 * MI ? min(n0 / 16 + blk, a_blocks - 1) : min(o0 / 16 + blk - 2 * MI, w_blocks - 1); // past the edge: the last block
        src_off[t] = (uint32_t)rb * (uint32_t)all_kt * OP::BLOCK + within;
    }
    auto fetch_one = [&](int step, int stage, int t) { // past the last K-tile (of an odd number, or of the ring's end): zeros
        const int unit = min((wave & 3) * NLOAD + t, UNITS - 1), kt = 2 * step + half;
        const bool token = unit * 1024 < 2 * MI * OP::BLOCK;
        const uint32_t bytes = kt < all_kt ? (uint32_t)(token ? a_blocks : w_blocks) * (uint32_t)all_kt * OP::BLOCK : 0u;
        qllm_detail::copy_1k_to_lds(token ? OP::tokens(g) : OP::features(g), bytes, src_off[t], (uint32_t)kt * OP::BLOCK,
                                    lds + stage * STAGE + half * HALF + unit * 1024);
    };
    constexpr int IN_FLIGHT = (STAGES - 2) * NLOAD; // loads of the steps after the next one
    constexpr int WAIT_LANDED = IN_FLIGHT | (7 << 4) | (15 << 8);      // s_waitcnt vmcnt(IN_FLIGHT): the next step has landed
    constexpr int WAIT_LANDED_LGKM0 = IN_FLIGHT | (7 << 4) | (0 << 8); // ... and lgkmcnt(0)
    static_assert(IN_FLIGHT < 16, "the low four bits of vmcnt");

    Acc acc[MI][NJ];
    typename OP::Frag ar[2][MI], wr[2][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i) ar[i / MI][i % MI] = OP::zero();
#pragma unroll
    for (int j = 0; j < 2 * NJ; ++j) wr[j / NJ][j % NJ] = OP::zero();

    uint8_t *const epi = lds + (mid_lds<OP, MI, NJ, STAGES>() - EPI_BYTES<TM, TN>);
    store_epilogue<ABITS, WBITS, TM, TN, OP::FP, 8>(g, load_epilogue<TM, TN>(g, n0, o0, tid), epi, tid);
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
#pragma unroll
        for (int t = 0; t < NLOAD; ++t) fetch_one(s, s, t);
    __builtin_amdgcn_s_waitcnt(WAIT_LANDED);
    __syncthreads();

    int stage = 0, fetch_stage = STAGES - 1;
    // reads this step's operands into set P and multiplies the step's before (the first time zeros) from the other one
    auto k_step = [&](auto parity, int step) {
        constexpr int P = decltype(parity)::value;
        constexpr int LOAD_STEP = 2 * NLOAD <= MI * NJ + 1 ? 2 : 1;
        static_assert(NJ + MI <= MI * NJ && NLOAD <= MI * NJ, "every read and load has its place behind an operation");
        const uint8_t *const tokens = lds + stage * STAGE + half * HALF + wm * MI * OP::BLOCK;
        const uint8_t *const features = lds + stage * STAGE + half * HALF + (2 * MI + wn * NJ) * OP::BLOCK;
#pragma unroll
        for (int s = 0; s < MI * NJ; ++s) {
            acc[s / NJ][s % NJ] = OP::multiply(wr[1 - P][s % NJ], ar[1 - P][s / NJ], acc[s / NJ][s % NJ]);
            if (s < NJ) wr[P][s] = OP::feature(features + s * OP::BLOCK, lane);
            else if (s < NJ + MI) ar[P][s - NJ] = OP::token(tokens + (s - NJ) * OP::BLOCK, lane);
            if (s % LOAD_STEP == 0 && s / LOAD_STEP < NLOAD) fetch_one(step + STAGES - 1, fetch_stage, s / LOAD_STEP); // into the stage whose last reader passed the barrier
            __builtin_amdgcn_sched_barrier(0); // this order is the order issued
        }
        // the next step has landed (this wave's share; the barrier adds the others'), own reads done
        __builtin_amdgcn_s_waitcnt(WAIT_LANDED_LGKM0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch_stage = stage;
        stage = stage == STAGES - 1 ? 0 : stage + 1;
    };
    int step = 0;
    for (; step + 1 < steps; step += 2) {
        k_step(std::integral_constant<int, 0>{}, step);
        k_step(std::integral_constant<int, 1>{}, step + 1);
    }
    if (step < steps) k_step(std::integral_constant<int, 0>{}, step);
    auto last_step = [&](auto parity) {
        constexpr int P = decltype(parity)::value;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = OP::multiply(wr[P][j], ar[P][i], acc[i][j]);
    };
    if (steps & 1) last_step(std::integral_constant<int, 0>{});
    else last_step(std::integral_constant<int, 1>{});
    // the loads past the last step went to stages nobody reads; the sums below take their place in LDS
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
    __syncthreads();

    constexpr int FIRST = (MI + 1) / 2; // the first half finishes its waves' first FIRST blocks of tokens, the second the others
    Acc *const sums = reinterpret_cast<Acc *>(lds) + (wave & 3) * FIRST * NJ * 64 + lane;
    constexpr int OTHER = 4 * FIRST * NJ * 64; // from the sums that the first half leaves to the second's
    auto leave = [&](auto from, auto to) {
#pragma unroll
        for (int i = decltype(from)::value; i < decltype(to)::value; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) sums[half * OTHER + ((i - decltype(from)::value) * NJ + j) * 64] = acc[i][j];
    };
    auto finish = [&](auto from, auto to) {
        constexpr int F = decltype(from)::value, COUNT = decltype(to)::value - F;
        Acc sum[COUNT][NJ];
#pragma unroll
        for (int i = 0; i < COUNT; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) sum[i][j] = acc[F + i][j] + sums[(1 - half) * OTHER + (i * NJ + j) * 64];
        const int nl = wm * 16 * MI + 16 * F, ol = wn * 16 * NJ;
        if (finish_from_lds<YT, TM, TN>(g, sum, epi, n0, o0, nl, ol, lane)) return;
        finish_wave_tile<ABITS, WBITS, YT, COUNT, NJ>(g, sum, n0 + nl, o0 + ol, lane, g.K);
    };
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, FIRST> some{};
    constexpr std::integral_constant<int, MI> all{};
    if (half == 0) leave(some, all);
    else leave(none, some);
    __syncthreads();
    if (half == 0) finish(none, some);
    else finish(some, all);
}

// Packed rows -> TILES8; one lane per (block, K-tile, lane of the operand read): 16 codes of one row.
template <int BITS>
__global__ __launch_bounds__(256) void tiles8_kernel(const uint8_t *codes, int64_t row_bytes, int32_t rows, int32_t K, int32_t n_kt,
                                                    uint8_t *tiles, int64_t n_items)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_items) return;
    const int l = (int)(idx & 63), r = l & 15, q = l >> 4;
    const int64_t bk = idx >> 6, b = bk / n_kt;
    const int kt = (int)(bk - b * n_kt);
    const int64_t row = b * 16 + r;
    const int k0 = kt * T8_KT + 16 * q; // the lane's first code
    uint32_t d[4] = {0u, 0u, 0u, 0u};
    if (row < rows && k0 < K) {
        // the lane's 2 * BITS bytes of the packed row, dword by dword; what lies past the row's end reads as zero codes
        const int64_t at = (int64_t)k0 * BITS / 8; // a multiple of 4
        const uint8_t *src = codes + row * row_bytes + at;
        uint32_t w[BITS / 2];
#pragma unroll
        for (int i = 0; i < BITS / 2; ++i) w[i] = at + 4 * i < row_bytes ? reinterpret_cast<const uint32_t *>(src)[i] : 0u;
        if constexpr (BITS == 4) {
            expand4(w[0], d[0], d[1]);
            expand4(w[1], d[2], d[3]);
        } else if constexpr (BITS == 6) {
            d[0] = spread6(w[0]);
            d[1] = spread6(__builtin_amdgcn_alignbit(w[1], w[0], 24));
            d[2] = spread6(__builtin_amdgcn_alignbit(w[2], w[1], 16));
            d[3] = spread6(w[2] >> 8);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // code - 128 as a signed byte, in the places that hold a code
                const int left = K - (k0 + 4 * i);
                const uint32_t live = left >= 4 ? 0xffffffffu : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
                d[i] = (w[i] ^ 0x80808080u) & live;
            }
        }
    }
    *reinterpret_cast<uint4 *>(tiles + bk * T8_BLOCK + 16 * l) = make_uint4(d[0], d[1], d[2], d[3]);
}

// Sum of the parts of a split K and the dequantising epilogue, four neighbouring outputs of a token per lane (one where
// O is no multiple of four: V = 1); the bracket in 64-bit arithmetic, which gives the same float as the narrow form.
// SA / SW: that side's codes are 8-bit and went into the matrix cores as code - 128 in every one of the K places (the
// byte-operand path), which is added back here.  Bound by the parts it reads: 16-byte loads where one output per lane had
// 4-byte ones (three parts of 200 x 5120: 5.4 -> 4.8 us).
constexpr int MAX_SPLITS = 8; // t8_splits; k_splits stays at four, its parts are part of the workspace's floor
template <typename YT, int SA, int SW, int V>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const GemmArgs g)
{
    typedef int vi __attribute__((ext_vector_type(V)));
    const int n = blockIdx.y, o = (int)(blockIdx.x * 256 + threadIdx.x) * V;
    if (o >= g.O) return;
    const int64_t idx = (int64_t)n * g.O + o;
    vi raw = vi(0); // the true accumulator fits int32 (checked by the launcher), so wrapping sums are exact
    for (int z0 = 0; z0 < g.splits; z0 += 4) { // four parts asked for at once; past the last part the last one again
        vi part[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) part[z] = *reinterpret_cast<const vi *>(g.partial + (int64_t)min(z0 + z, g.splits - 1) * g.N * g.O + idx);
#pragma unroll
        for (int z = 0; z < 4; ++z) raw += z0 + z < g.splits ? part[z] : vi(0);
    }
    const int32_t rs = g.rs[n];
    const int64_t bx = g.bx[n];
    const float ax = g.ax[n];
    float out[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int32_t cs = g.cs[o + e];
        const int64_t bw = g.bw[o + e];
        raw[e] += 128 * SW * rs + 128 * SA * cs - 16384 * SA * SW * g.K;
        const int64_t t = (int64_t)raw[e] - bx * cs - bw * rs + (int64_t)g.K * bx * bw;
        out[e] = ((float)t * ax) * g.aw[o + e];
    }
    const int64_t at = (int64_t)n * g.ldy + o;
    if constexpr (V == 1) {
        if constexpr (sizeof(YT) == 4) reinterpret_cast<float *>(g.y)[at] = out[0];
        else reinterpret_cast<uint16_t *>(g.y)[at] = f32_to_bf16_rne(out[0]);
    } else if constexpr (sizeof(YT) == 4) {
        *reinterpret_cast<v4f_any *>(reinterpret_cast<float *>(g.y) + at) = v4f{out[0], out[1], out[2], out[3]};
    } else {
        typedef unsigned int v2u_any __attribute__((ext_vector_type(2), aligned(2)));
        *reinterpret_cast<v2u_any *>(reinterpret_cast<uint16_t *>(g.y) + at) = v2u_any{f32x2_to_bf16x2_rne(out[0], out[1]), f32x2_to_bf16x2_rne(out[2], out[3])};
    }
    if (g.acc_dump) {
#pragma unroll
        for (int e = 0; e < V; ++e) g.acc_dump[idx + e] = raw[e];
    }
}

// ---- few tokens (decode, small batches): the weights are read once from HBM and that is the whole cost.  A
// workgroup owns 16 RT output features and 16 NT tokens; its WAVES waves split K:
// each takes a run of steps of STEP codes and works on its own, without barriers, until the partial tiles are added up
// at the end.
//   * Global loads are laid out for the memory pipeline, not for the matrix cores: consecutive lanes
//     take consecutive 16-byte pieces of a row's STEP codes, so one load instruction touches whole
//     (half) cache lines (a lane per matrix-core operand row would touch three to four times as many lines,
//     and the address unit, one line per cycle, would be the limit).  Two steps' loads are in flight.
//   * The pieces pass through a wave-private strip of LDS, still packed, and come back as a quarter of the step's
//     codes of row r, the c-th, for lane (r, c), are expanded in registers and feed STEP / 64 matrix-core
//     operations, the m-th on codes 16 m .. 16 m + 15 of every lane's quarter: which 64 codes
//     of the step one operation sums is free as long as both operands agree.
template <int BITS, int STEP>
constexpr int SK_ROW = STEP * BITS / 8 + 16; // bytes of LDS per row and step: the packed codes and a pad against bank conflicts

template <int ABITS, int WBITS, int NT, int RT, int STEP>
constexpr int SK_STRIP = 16 * RT * SK_ROW<WBITS, STEP> + 16 * NT * SK_ROW<ABITS, STEP>; // LDS bytes per wave

template <int ABITS, int WBITS, int NT, int RT, int WAVES, int STEP>
constexpr size_t skinny_lds()
{
    const size_t strips = (size_t)WAVES * SK_STRIP<ABITS, WBITS, NT, RT, STEP>;
    const size_t red = (size_t)WAVES * NT * RT * 64 * sizeof(v4i);
    return (strips > red ? strips : red) + EPI_BYTES<16 * NT, 16 * RT>;
}

// CODES codes of one row (packed, in DW dwords) -> one byte per code; the orders of expand_unit
template <int BITS, int CODES, bool PERM>
__device__ __forceinline__ void expand_codes(const uint32_t (&w)[CODES * BITS / 32], uint32_t (&d)[CODES / 4])
{
    if constexpr (BITS == 4) {
#pragma unroll
        for (int i = 0; i < CODES / 8; ++i) {
            if constexpr (PERM) {
                d[2 * i] = w[i] & 0x0f0f0f0fu;
                d[2 * i + 1] = (w[i] >> 4) & 0x0f0f0f0fu;
            } else {
                expand4(w[i], d[2 * i], d[2 * i + 1]);
            }
        }
    } else if constexpr (BITS == 6) {
#pragma unroll
        for (int i = 0; i < CODES / 16; ++i) { // 3 dwords = 4 groups of 24 bits
            const uint32_t w0 = w[3 * i], w1 = w[3 * i + 1], w2 = w[3 * i + 2];
            d[4 * i + 0] = spread6(w0);
            d[4 * i + 1] = spread6(__builtin_amdgcn_alignbit(w1, w0, 24));
            d[4 * i + 2] = spread6(__builtin_amdgcn_alignbit(w2, w1, 16));
            d[4 * i + 3] = spread6(w2 >> 8);
        }
    } else {
#pragma unroll
        for (int i = 0; i < CODES / 4; ++i) d[i] = w[i] ^ 0x80808080u; // code - 128 as a signed byte
    }
}

// Registers for two workgroups of eight waves per CU where the loop fits in them (with one workgroup 27648 x 5120 6-bit
// weights and 16 tokens take 34 instead of 29 us, and 4-bit weights and 32 tokens 23.6 instead of 20.9).
template <int ABITS, int WBITS, int NT>
constexpr int SK_WAVES_PER_SIMD = NT == 1 || (NT == 2 && ABITS == 4 && WBITS == 4) ? 4 : 2;

template <int ABITS, int WBITS, typename YT, int NT, int RT, int WAVES, int STEP>
__global__ __launch_bounds__(64 * WAVES, (SK_WAVES_PER_SIMD<ABITS, WBITS, NT>)) void int_gemm_skinny_kernel(const GemmArgs g)
{
    // [WAVES] strips; afterwards reused as [WAVES][NT * RT][64] v4i for the final sum
    extern __shared__ __align__(16) uint8_t sk_lds[];
    constexpr bool PERM = ABITS == 4 && WBITS == 4;
    constexpr int CODES = STEP / 4;                                                    // a lane's codes of one row and step
    constexpr int WB = STEP * WBITS / 8, AB = STEP * ABITS / 8;                        // bytes per row and step
    constexpr int WPIECES = WB / 16, APIECES = AB / 16;                                // 16-byte pieces per row and step
    constexpr int WLOADS = 16 * RT * WPIECES / 64, ALOADS = 16 * NT * APIECES / 64; // load instructions per step
    static_assert(16 * RT * WPIECES % 64 == 0 && 16 * NT * APIECES % 64 == 0, "whole load instructions");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, c = lane >> 4;
    const int o0 = blockIdx.x * (16 * RT), n0 = blockIdx.y * (16 * NT);
    uint8_t *w_strip = sk_lds + wave * SK_STRIP<ABITS, WBITS, NT, RT, STEP>, *a_strip = w_strip + 16 * RT * SK_ROW<WBITS, STEP>;

    // piece lane + 64 t of a step: where it comes from (from the operand's first row and the step's first byte on; past
    // the edge the last row again) and where it goes
    const uint8_t *const w_base = g.w_codes + (int64_t)o0 * g.w_row_bytes, *const a_base = g.a_codes + (int64_t)n0 * g.a_row_bytes;
    uint32_t w_src[WLOADS], a_src[ALOADS];
    int w_dst[WLOADS], a_dst[ALOADS];
#pragma unroll
    for (int t = 0; t < WLOADS; ++t) {
        const int q = lane + 64 * t, row = q / WPIECES, piece = q % WPIECES;
        w_src[t] = (uint32_t)min(row, g.O - 1 - o0) * (uint32_t)g.w_row_bytes + 16 * piece;
        w_dst[t] = row * SK_ROW<WBITS, STEP> + 16 * piece;
    }
#pragma unroll
    for (int t = 0; t < ALOADS; ++t) {
        const int q = lane + 64 * t, row = q / APIECES, piece = q % APIECES;
        a_src[t] = (uint32_t)min(row, g.N - 1 - n0) * (uint32_t)g.a_row_bytes + 16 * piece;
        a_dst[t] = row * SK_ROW<ABITS, STEP> + 16 * piece;
    }

    constexpr size_t EPI_AT = skinny_lds<ABITS, WBITS, NT, RT, WAVES, STEP>() - EPI_BYTES<16 * NT, 16 * RT>;
    uint8_t *const epi = sk_lds + EPI_AT; // the epilogue's constants, behind strips and partial tiles
    const EpiRegs epi_regs = load_epilogue<16 * NT, 16 * RT>(g, n0, o0, tid);

    v4i acc[NT][RT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    v4i w0[WLOADS], a0[ALOADS], w1[WLOADS], a1[ALOADS]; // two register stages
    auto fetch = [&](v4i (&tw)[WLOADS], v4i (&ta)[ALOADS], int s) {
        const uint8_t *wp = w_base + (int64_t)s * WB, *ap = a_base + (int64_t)s * AB;
#pragma unroll
        for (int k = 0; k < WLOADS; ++k) tw[k] = *reinterpret_cast<const v4i *>(wp + w_src[k]);
#pragma unroll
        for (int k = 0; k < ALOADS; ++k) ta[k] = *reinterpret_cast<const v4i *>(ap + a_src[k]);
    };
    auto work = [&](const v4i (&tw)[WLOADS], const v4i (&ta)[ALOADS]) {
        // a wave's LDS operations complete in order: these writes follow the previous step's reads
#pragma unroll
        for (int k = 0; k < WLOADS; ++k) *reinterpret_cast<v4i *>(w_strip + w_dst[k]) = tw[k];
#pragma unroll
        for (int k = 0; k < ALOADS; ++k) *reinterpret_cast<v4i *>(a_strip + a_dst[k]) = ta[k];
        auto quarter = [&](const uint8_t *strip_row, auto bits, uint32_t (&d)[CODES / 4]) { // lane (r, c)'s codes of a row
            constexpr int BITS = decltype(bits)::value, DW = CODES * BITS / 32;
            uint32_t u[DW];
            const uint8_t *p = strip_row + c * (4 * DW);
            if constexpr (DW % 4 == 0) {
#pragma unroll
                for (int k = 0; k < DW / 4; ++k) {
                    const v4i v = reinterpret_cast<const v4i *>(p)[k];
                    u[4 * k] = (uint32_t)v[0]; u[4 * k + 1] = (uint32_t)v[1]; u[4 * k + 2] = (uint32_t)v[2]; u[4 * k + 3] = (uint32_t)v[3];
                }
            } else {
#pragma unroll
                for (int k = 0; k < DW / 2; ++k) {
                    const v2i v = reinterpret_cast<const v2i *>(p)[k];
                    u[2 * k] = (uint32_t)v[0]; u[2 * k + 1] = (uint32_t)v[1];
                }
            }
            expand_codes<BITS, CODES, PERM>(u, d);
        };
        uint32_t dw[RT][CODES / 4];
#pragma unroll
        for (int j = 0; j < RT; ++j)
            quarter(w_strip + (16 * j + r) * SK_ROW<WBITS, STEP>, std::integral_constant<int, WBITS>{}, dw[j]);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            uint32_t da[CODES / 4];
            quarter(a_strip + (16 * i + r) * SK_ROW<ABITS, STEP>, std::integral_constant<int, ABITS>{}, da);
#pragma unroll
            for (int m = 0; m < CODES / 16; ++m)
#pragma unroll
                for (int j = 0; j < RT; ++j) {
                    const v4i fw = {(int)dw[j][4 * m], (int)dw[j][4 * m + 1], (int)dw[j][4 * m + 2], (int)dw[j][4 * m + 3]};
                    const v4i fa = {(int)da[4 * m], (int)da[4 * m + 1], (int)da[4 * m + 2], (int)da[4 * m + 3]};
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw, fa, acc[i][j], 0, 0, 0);
                }
        }
    };

    const int n_steps = g.Kpad / STEP; // rows are padded to a multiple of 256 codes
    if constexpr ((NT == 4 || NT == 6) && (ABITS == 4 || (WBITS == 4 && RT == 2))) {
        // Two steps at a time, each asking for the one after the next.  The last two of an even number ask for nothing, an odd number
        // still asks for the wave's first step again, once where the other form does so twice.  It is a copy of the step more in the
        // code, which costs what it gains with one or two tiles of tokens, with 6-bit codes, with 8-bit weights and, under 8-bit
        // activations, with 64 features; with eight tiles the registers run out (128 x 8192 -> 8192 18 : 63).  us, other form : this one:
        //   product: 33 x 5120 -> 27648 4 / 4 21.3 : 18.7, 96 x 4096 -> 4096 4 / 4 9.3 : 8.3, 50 x 4096 -> 4096 8 / 4 9.8 : 8.7, 64 x 28672 ->
        //     8192 4 / 4 44.3 : 44.2; 32 x 8192 -> 8192 6 / 6 15.2 : 15.8, 24 x 5120 -> 13824 4 / 4 10.1 : 10.3
        //   layer call, weights in cache / out of every cache: 38 x 3712 -> 25472 4 / 4 23.8 : 22.1 / 26.3 : 25.7, 50 x 3200 -> 640 8 / 4 14.2 :
        //     12.9 / 15.8 : 14.6; 62 x 4544 -> 4583 8 / 8 17.7 : 18.3 / 21.6 : 22.5, 70 x 1536 -> 1408 8 / 8 12.1 : 12.4 / 14.4 : 14.2; 64 features: 59 x 8320 ->
        //     8320 8 / 4 28.0 : 27.3 / 32.5 : 34.1, 46 x 3840 -> 17152 24.4 : 24.2 / 28.7 : 29.8
        const int mine = wave < n_steps ? (n_steps - wave + WAVES - 1) / WAVES : 0; // this wave's steps: wave, wave + WAVES, ..
        auto step = [&](int k) { return k < mine ? wave + k * WAVES : wave; };
        if (mine > 0) {
            fetch(w0, a0, step(0));
            fetch(w1, a1, step(1));
            int k = 0;
            for (; k + 2 < mine; k += 2) {
                work(w0, a0);
                fetch(w0, a0, step(k + 2));
                work(w1, a1);
                fetch(w1, a1, step(k + 3));
            }
            work(w0, a0);
            if (k + 1 < mine) work(w1, a1);
        }
    } else {
        // Every fetch is unconditional (past the end a wave re-reads its first step, from cache), so that
        // the number of loads in flight at each wait is known when the code is compiled.
        int s = wave;
        if (s < n_steps) {
            fetch(w0, a0, s);
            fetch(w1, a1, s + WAVES < n_steps ? s + WAVES : wave);
            while (true) { // two steps per turn: the register stages alternate without being indexed
                work(w0, a0);
                fetch(w0, a0, s + 2 * WAVES < n_steps ? s + 2 * WAVES : wave);
                s += WAVES;
                if (s >= n_steps) break;
                work(w1, a1);
                fetch(w1, a1, s + 2 * WAVES < n_steps ? s + 2 * WAVES : wave);
                s += WAVES;
                if (s >= n_steps) break;
            }
        }
    }

    // ---- add the waves' partial tiles up; wave t finishes token tiles t, t + WAVES, ..
    store_epilogue<ABITS, WBITS, 16 * NT, 16 * RT, false, WAVES>(g, epi_regs, epi, tid);
    __syncthreads(); // the strips are no longer read
    v4i *red = reinterpret_cast<v4i *>(sk_lds);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) red[(wave * (NT * RT) + i * RT + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    for (int i = wave; i < NT; i += WAVES) {
        v4i sum[1][RT];
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            sum[0][j] = red[(i * RT + j) * 64 + lane];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) sum[0][j] += red[(w * (NT * RT) + i * RT + j) * 64 + lane];
            // 8-bit codes on both sides: places past K were zero codes, -128 times -128 each
            if constexpr (ABITS == 8 && WBITS == 8) sum[0][j] -= 16384 * (g.Kpad - g.K);
        }
        if (finish_from_lds<YT, 16 * NT, 16 * RT>(g, sum, epi, n0, o0, 16 * i, 0, lane)) continue;
        finish_wave_tile<ABITS, WBITS, YT, 1, RT>(g, sum, n0 + 16 * i, o0, lane, g.K);
    }
}

// kernels whose LDS limit has been raised (once each: every kernel here always asks for the same amount,
// and no runtime call then sits between a caller's stream capture and the launch)
std::mutex raised_lock;
std::vector<const void *> raised;

template <typename K>
int32_t launch_kernel(K kernel, dim3 grid, dim3 block, size_t lds, const GemmArgs &g, hipStream_t stream)
{
    if (lds > 48 * 1024) {
        const void *fn = reinterpret_cast<const void *>(kernel);
        std::lock_guard<std::mutex> hold(raised_lock);
        bool done = false;
        for (const void *k : raised) done = done || k == fn;
        if (!done) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                qllm_note_hip_error("int gemm: raising the LDS limit", hipGetErrorName(e));
                return QLLM_ERR_HIP;
            }
            raised.push_back(fn);
        }
    }
    (void)hipGetLastError(); // drop any stale error of the calling thread: only this launch is judged
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        qllm_note_hip_error("int gemm: launch", hipGetErrorName(e));
        return QLLM_ERR_HIP;
    }
    return QLLM_OK;
}

template <int SA, int SW>
int32_t launch_finish(const GemmArgs &g, int32_t y_dtype, hipStream_t stream)
{
    if ((g.O & 3) == 0 && (reinterpret_cast<uintptr_t>(g.partial) & 15u) == 0) {
        const dim3 grid((unsigned)((g.O / 4 + 255) / 256), (unsigned)g.N);
        if (y_dtype == QLLM_F32) return launch_kernel(splitk_finish_kernel<float, SA, SW, 4>, grid, dim3(256), 0, g, stream);
        return launch_kernel(splitk_finish_kernel<uint16_t, SA, SW, 4>, grid, dim3(256), 0, g, stream);
    }
    const dim3 grid((unsigned)((g.O + 255) / 256), (unsigned)g.N); // at most 128 tiles of 128 x 128: N <= 16384
    if (y_dtype == QLLM_F32) return launch_kernel(splitk_finish_kernel<float, SA, SW, 1>, grid, dim3(256), 0, g, stream);
    return launch_kernel(splitk_finish_kernel<uint16_t, SA, SW, 1>, grid, dim3(256), 0, g, stream);
}

// How a product with 256 x 256 or 128 x 128 tiles is laid over the chip.  A round of 256 large tiles (one per CU)
// takes one unit of time, a round of 512 small ones (two per CU; half the outputs at about three quarters of the
// rate) 0.65.  Large tiles throughout, small tiles throughout, or -- when the large tiles fill whole rounds and
// leave a rest -- large tiles for the output features of the whole rounds and small tiles for the others, as two
// launches (7B q/k/v: 384 large tiles are two rounds, 1536 small ones three; 256 large + 512 small are 1.65).
struct TilePlan {
    bool small;      // 128 x 128 tiles for everything (or for everything from o_split on)
    int32_t o_split; // > 0: large tiles for features below o_split, small tiles from there on
};
TilePlan plan_tiles(int64_t N, int64_t O, bool may_split_launch)
{
    const int64_t nb = (N + LBM - 1) / LBM, ob = (O + LBN - 1) / LBN, big_tiles = nb * ob;
    const int64_t small_tiles = ((O + 127) / 128) * ((N + 127) / 128);
    const double cost_big = (double)((big_tiles + 255) / 256), cost_small = 0.65 * (double)((small_tiles + 511) / 512);
    if (N <= 128) return TilePlan{true, 0};
    TilePlan best{cost_small < cost_big, 0};
    double best_cost = cost_small < cost_big ? cost_small : cost_big;
    const int64_t whole = big_tiles / 256, ca = whole * 256 / nb; // feature blocks that whole rounds of large tiles cover
    if (may_split_launch && whole >= 1 && ca > 0 && ca < ob) {
        const int64_t rest_small = ((O - ca * LBN + 127) / 128) * ((N + 127) / 128);
        const double cost = (double)((ca * nb + 255) / 256) + 0.65 * (double)((rest_small + 511) / 512);
        if (cost < best_cost - 0.05) best = TilePlan{false, (int32_t)(ca * LBN)};
    }
    return best;
}

// Packed 4-bit rows (device) -> TILES6 (device).
template <bool BY_ROW>
int32_t launch_tiles6(const uint8_t *codes, int64_t row_bytes, int64_t rows, int64_t Kpad, uint8_t *tiles, hipStream_t stream)
{
    const int64_t n_kt = Kpad / T6_KT, n_items = (rows + 15) / 16 * n_kt * 64;
    (void)hipGetLastError();
    hipLaunchKernelGGL(tiles6_kernel<BY_ROW>, dim3((unsigned)((n_items + 255) / 256)), dim3(256), 0, stream, codes, row_bytes, (int32_t)rows,
                       (int32_t)n_kt, tiles, n_items);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        qllm_note_hip_error("tiles6: launch", hipGetErrorName(e));
        return QLLM_ERR_HIP;
    }
    return QLLM_OK;
}

// The tile of gemm_mid_kernel that a product takes, in units of 32 tokens and 32 features; none: another kernel.
struct MidPlan {
    int mi, nj;
};
// Whether its launch is one round: columns of 128 features go to the eight XCDs in turn, so that what counts is the XCD with the
// most of them, 32 workgroups each (2346 x 17792 -> 1280 4 / 4, ten columns, four tiles of 64 features by 15 of tokens on the 32 CUs
// of an XCD: 145 -> 178 us; 1075 x 896 -> 1536 8 / 4 14.3 -> 18.4).
int64_t mid_columns(int64_t O) { return ((O + 127) / 128 + 7) / 8 * 8; }
bool mid_fits(const MidPlan &p, int64_t N, int64_t O) { return mid_columns(O) * (4 / p.nj) * ((N + 32 * p.mi - 1) / (32 * p.mi)) <= 256; }

template <class OP, int ABITS, int WBITS, int MI, int NJ, int STAGES>
int32_t launch_mid(const GemmArgs &g, int32_t y_dtype, hipStream_t stream)
{
    static_assert(NJ == 2 || NJ == 4, "columns of 128 features, or their halves");
    const dim3 grid((unsigned)mid_columns(g.O) * (4 / NJ), (unsigned)((g.N + 32 * MI - 1) / (32 * MI)));
    constexpr size_t lds = mid_lds<OP, MI, NJ, STAGES>();
    if (y_dtype == QLLM_F32) return launch_kernel(gemm_mid_kernel<OP, ABITS, WBITS, float, MI, NJ, STAGES>, grid, dim3(LTHREADS), lds, g, stream);
    return launch_kernel(gemm_mid_kernel<OP, ABITS, WBITS, uint16_t, MI, NJ, STAGES>, grid, dim3(LTHREADS), lds, g, stream);
}

// 4-bit codes on both sides, more than 32 tokens, on the FP6 matrix cores: the activations are re-laid
// into g.a_tiles first, unless they are there already.
int32_t launch_fp6(const GemmArgs &g, const TilePlan &plan, const MidPlan &mid, int32_t y_dtype, hipStream_t stream)
{
    if (mid.mi == 5) return launch_mid<MidFp6, 4, 4, 5, 2, 3>(g, y_dtype, stream); // only where the activations are laid out
    if (mid.mi == 4 && mid.nj == 2) return launch_mid<MidFp6, 4, 4, 4, 2, 4>(g, y_dtype, stream);
    if (mid.mi == 4) return launch_mid<MidFp6, 4, 4, 4, 4, 3>(g, y_dtype, stream);
    if (!g.a_laid) {
        const int32_t st = launch_tiles6<true>(g.a_codes, g.a_row_bytes, g.N, g.Kpad, const_cast<uint8_t *>(g.a_tiles), stream);
        if (st != QLLM_OK) return st;
    }
    auto launch_small = [&](const GemmArgs &ga) -> int32_t {
        const dim3 grid((unsigned)((ga.O - ga.o_first + 127) / 128), (unsigned)((ga.N + 127) / 128), (unsigned)(ga.splits > 1 ? ga.splits : 1));
        constexpr size_t lds = (size_t)T6_STAGES * 16 * T6_BLOCK + EPI_BYTES<128, 128>;
        if (ga.splits > 1) {
            const int32_t sp = launch_kernel(gemm_w4a4_fp6_kernel<float, 4, 2, true>, grid, dim3(LTHREADS), lds, ga, stream);
            if (sp != QLLM_OK) return sp;
            return launch_finish<0, 0>(ga, y_dtype, stream);
        }
        if (y_dtype == QLLM_F32) return launch_kernel(gemm_w4a4_fp6_kernel<float, 4, 2>, grid, dim3(LTHREADS), lds, ga, stream);
        return launch_kernel(gemm_w4a4_fp6_kernel<uint16_t, 4, 2>, grid, dim3(LTHREADS), lds, ga, stream);
    };
    auto launch_big = [&](const GemmArgs &ga) -> int32_t {
        const dim3 grid((unsigned)((ga.O - ga.o_first + LBN - 1) / LBN), (unsigned)((ga.N + LBM - 1) / LBM));
        constexpr size_t lds = (size_t)T6_STAGES * 32 * T6_BLOCK + EPI_BYTES<256, 256>;
        if (y_dtype == QLLM_F32) return launch_kernel(gemm_w4a4_fp6_kernel<float, 8, 4>, grid, dim3(LTHREADS), lds, ga, stream);
        return launch_kernel(gemm_w4a4_fp6_kernel<uint16_t, 8, 4>, grid, dim3(LTHREADS), lds, ga, stream);
    };
    if (g.splits > 1) return launch_small(g); // K is only split where the small tile is the choice
    if (plan.o_split > 0) { // whole rounds of large tiles, then the other output features with small ones
        GemmArgs first = g, rest = g;
        first.O = plan.o_split;
        rest.o_first = plan.o_split;
        const int32_t rc = launch_big(first);
        return rc != QLLM_OK ? rc : launch_small(rest);
    }
    return plan.small ? launch_small(g) : launch_big(g);
}

// Packed rows (device) -> TILES8 (device).
int32_t launch_tiles8(const uint8_t *codes, int32_t bits, int64_t rows, int64_t K, uint8_t *tiles, hipStream_t stream)
{
    const int64_t n_kt = (K + T8_KT - 1) / T8_KT, n_items = (rows + 15) / 16 * n_kt * 64;
    const dim3 grid((unsigned)((n_items + 255) / 256));
    const int64_t row_bytes = qllm_packed_row_bytes(K, bits);
    (void)hipGetLastError();
    if (bits == 4) hipLaunchKernelGGL(tiles8_kernel<4>, grid, dim3(256), 0, stream, codes, row_bytes, (int32_t)rows, (int32_t)K, (int32_t)n_kt, tiles, n_items);
    else if (bits == 6) hipLaunchKernelGGL(tiles8_kernel<6>, grid, dim3(256), 0, stream, codes, row_bytes, (int32_t)rows, (int32_t)K, (int32_t)n_kt, tiles, n_items);
    else hipLaunchKernelGGL(tiles8_kernel<8>, grid, dim3(256), 0, stream, codes, row_bytes, (int32_t)rows, (int32_t)K, (int32_t)n_kt, tiles, n_items);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        qllm_note_hip_error("tiles8: launch", hipGetErrorName(e));
        return QLLM_ERR_HIP;
    }
    return QLLM_OK;
}

// The byte-operand path's tile where K may be split: 128 x 128 (two workgroups per CU) where that is the plan
// for the whole product, as on the FP6 path, and for up to 128 tokens.
bool t8_small_tile(int64_t N, int64_t O) { return plan_tiles(N, O, false).small; }

// Into how many parts the byte-operand path splits K when it has room for the parts' accumulators: as on the
// 4-bit path, only where 128 x 128 tiles leave most CUs without a workgroup, every part at least eight K-tiles; up to
// eight parts (16384 -> 1024, 128 tokens: 26.7 us with four, 21 with eight; 28672 -> 2048: 37.6, 29), one workgroup per CU
// (two: 8192 x 8192, 200 tokens 34 -> 40).
int32_t t8_splits(int64_t N, int64_t K, int64_t O)
{
    if (N <= 32 || !t8_small_tile(N, O)) return 1;
    const int64_t tiles = ((O + 127) / 128) * ((N + 127) / 128), n_kt = (K + T8_KT - 1) / T8_KT;
    if (tiles > 128) return 1;
    int64_t s = 256 / tiles;
    if (s > MAX_SPLITS) s = MAX_SPLITS;
    if (s > n_kt / 8) s = n_kt / 8;
    return s < 2 ? 1 : (int32_t)s;
}

// gemm_mid_kernel on byte operands.
// Layer call, us, other kernel : this one, three sets of weights in turn / weights out of every cache:
//   128 x 64 in place of 128 x 128 tiles with K split (or of half a round of them), where these tiles are one round:
//     256 x 8192 -> 8192 8/4 36.1 : 30.9 / 42.2 : 40.2, 100 x 4096 -> 16384 6/6 30.4 : 24.3 / 33.8 : 29.2, 553 x 1024 -> 2944 6/6
//     24.1 : 14.7 / 24.4 : 15.2, 250 x 3000 -> 5000 8/4 21.1 : 16.7
//   A workgroup loads the whole K of 192 rows where one of the other kernel's loads its part of 256 rows.  From some 640 thousand codes
//   more on that costs what finish and sums in memory save, first where the weights come from HBM: 822 x 9984 -> 1664 8/8 (two
//     parts) 54.8 : 44.1 / 54.2 : 47.8, 230 x 5888 -> 5120 8/4 (three) 26.3 : 24.3 / 29.3 : 30.9; 2048 x 7000 -> 512 8/8 (four) 48.6 : 47.3 /
//     48.4 : 52.1, 362 x 5760 -> 2048 6/6 (five) 26.8 : 26.9 / 27.9 : 32.6.  Sooner up to 128 tokens, for which the layer call reads weights ahead
//     of parts: 73 x 3584 -> 12160 6/6 21.4 : 18.0 / 24.5 : 22.8, 83 x 4352 -> 9600 8/4 22.2 : 20.4 / 24.3 : 25.9.  Later where the
//     features are no multiple of four, which the finish takes one by one: 108 x 4800 -> 5534 8/8 28.0 : 20.9 / 30.1 : 25.8, 985 x
//     5376 -> 975 39.8 : 29.6 / 39.9 : 33.9
//   Where the other kernel has K whole too, up to 512 channels are mostly start and end and half as many features per workgroup lose out
//     of cache (487 x 384 -> 2176 8/4 11.6 : 11.4 / 11.7 : 12.6, 235 x 512 -> 3584 6/6 11.6 : 11.3 / 12.5 : 12.9; 240 layers 1.03 / 0.995 of the
//     other's rate), but for features that are no multiple of four (328 x 384 -> 3985 6/6 13.0 : 12.2 / 13.9 : 13.4); and up to six
//     columns of 128 features leave two XCDs without work (1987 x 384 -> 640 6/6 13.5 : 13.7 / 13.2 : 13.6)
//   Up to 128 tokens 6-bit codes with fewer than 184 such tiles stay with the parts of K, for which the layer call reads weights ahead
//     (100 x 5120 -> 9216 23.4 : 20.9 all the same).
//   160 x 128, where 128 x 128 tiles are more than one round of workgroups and these are not: 777 x 5000 -> 4999 8/4 31.9 : 24.7 (the
//     product), 600 x 28672 -> 8192 8/8 207 : 172 / 207 : 173, 777 x 5120 -> 5120 8/8 43.8 : 36.5, 300 x 4096 -> 12288 8/4 34.1 : 29.0 / 36.9 :
//     35.6; one row of tiles, 129 to 160 tokens, is up to 4 % behind out of cache at a short K (136 x 2432 -> 20480 8/4 25.3 : 22.5 / 28.3 :
//     29.3; 139 x 2304 -> 27029 31.8 : 24.7 / 33.4 : 31.3).  With no more 128 x 128 tiles than CUs they lose (600 x 5120 -> 5120 8/4 29.5 :
//     31.5, 400 x 8192 -> 8192 51 : 53), and a short K gains nothing (600 x 2048 -> 8192 8/4 22.9 : 21.2; 640 x 1024 -> 8192 6/6 17.5 :
//     17.5 / 21.7 : 23.0)
MidPlan plan_mid8(int64_t N, int64_t K, int64_t O, int a_bits)
{
    auto groups = [&](int64_t tm, int64_t tn) { return ((N + tm - 1) / tm) * ((O + tn - 1) / tn); };
    const int64_t half_tiles = groups(128, 64), fewest = a_bits == 6 && N <= 128 ? 184 : 80, parts = t8_splits(N, K, O);
    const bool gains = parts > 1 ? 192 * K - 256 * K / parts <= (O % 4 ? 745000 : N > 128 ? 640000 : 450000) : O > 6 * 128 && (K > 512 || O % 4);
    if (half_tiles >= fewest && mid_fits(MidPlan{4, 2}, N, O) && K <= 12288 && gains) return MidPlan{4, 2};
    if (groups(128, 128) > 256 && mid_fits(MidPlan{5, 4}, N, O) && K >= 2048) return MidPlan{5, 4};
    return MidPlan{0, 0};
}

// 6- or 8-bit activations, more than 32 tokens, byte operands straight into the int8 matrix cores: the
// activations are re-laid into the workspace, then the product, laid over the chip as on the FP6 path.
template <int ABITS, int WBITS>
int32_t launch_t8(const GemmArgs &g, const TilePlan &plan, const MidPlan &mid, int32_t y_dtype, hipStream_t stream)
{
    if (!g.a_laid) {
        const int32_t st = launch_tiles8(g.a_codes, ABITS, g.N, g.K, const_cast<uint8_t *>(g.a_tiles8), stream);
        if (st != QLLM_OK) return st;
    }
    auto launch_small = [&](const GemmArgs &ga) -> int32_t {
        const dim3 grid((unsigned)((ga.O - ga.o_first + 127) / 128), (unsigned)((ga.N + 127) / 128), (unsigned)(ga.splits > 1 ? ga.splits : 1));
        constexpr size_t lds3 = (size_t)3 * 16 * T8_BLOCK + EPI_BYTES<128, 128>, lds4 = (size_t)4 * 16 * T8_BLOCK + EPI_BYTES<128, 128>;
        if (ga.splits > 1) { // at most 256 workgroups
            const int32_t sp = launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, float, 4, 2, 4, true>, grid, dim3(LTHREADS), lds4, ga, stream);
            if (sp != QLLM_OK) return sp;
            constexpr int SA = ABITS == 8 ? 1 : 0, SW = WBITS == 8 ? 1 : 0;
            return launch_finish<SA, SW>(ga, y_dtype, stream);
        }
        if ((int64_t)grid.x * grid.y <= 256) {
            if (y_dtype == QLLM_F32) return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, float, 4, 2, 4>, grid, dim3(LTHREADS), lds4, ga, stream);
            return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, uint16_t, 4, 2, 4>, grid, dim3(LTHREADS), lds4, ga, stream);
        }
        if (y_dtype == QLLM_F32) return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, float, 4, 2, 3>, grid, dim3(LTHREADS), lds3, ga, stream);
        return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, uint16_t, 4, 2, 3>, grid, dim3(LTHREADS), lds3, ga, stream);
    };
    auto launch_big = [&](const GemmArgs &ga) -> int32_t {
        const dim3 grid((unsigned)((ga.O - ga.o_first + LBN - 1) / LBN), (unsigned)((ga.N + LBM - 1) / LBM));
        constexpr size_t lds = (size_t)3 * 32 * T8_BLOCK + EPI_BYTES<256, 256>;
        if (y_dtype == QLLM_F32) return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, float, 8, 4, 3>, grid, dim3(LTHREADS), lds, ga, stream);
        return launch_kernel(gemm_tiles8_kernel<ABITS, WBITS, uint16_t, 8, 4, 3>, grid, dim3(LTHREADS), lds, ga, stream);
    };
    if (mid.mi == 4) return launch_mid<MidBytes, ABITS, WBITS, 4, 2, 4>(g, y_dtype, stream);
    if (mid.mi == 5) return launch_mid<MidBytes, ABITS, WBITS, 5, 4, 4>(g, y_dtype, stream);
    if (g.splits > 1) return launch_small(g); // K is only split where the small tile is the choice
    if (plan.o_split > 0) { // whole rounds of large tiles, then the other output features with small ones
        GemmArgs first = g, rest = g;
        first.O = plan.o_split;
        rest.o_first = plan.o_split;
        const int32_t rc = launch_big(first);
        return rc != QLLM_OK ? rc : launch_small(rest);
    }
    return plan.small ? launch_small(g) : launch_big(g);
}

template <int ABITS, int WBITS, int NT, int RT, int WAVES, int STEP>
int32_t launch_skinny(const GemmArgs &g, int32_t y_dtype, hipStream_t stream)
{
    static_assert(16 * NT + 16 * RT <= 64 * WAVES, "a lane stages one token's or one feature's constants");
    const dim3 grid((unsigned)((g.O + 16 * RT - 1) / (16 * RT)), (unsigned)((g.N + 16 * NT - 1) / (16 * NT)));
    constexpr size_t lds = skinny_lds<ABITS, WBITS, NT, RT, WAVES, STEP>();
    if (y_dtype == QLLM_F32) return launch_kernel(int_gemm_skinny_kernel<ABITS, WBITS, float, NT, RT, WAVES, STEP>, grid, dim3(64 * WAVES), lds, g, stream);
    return launch_kernel(int_gemm_skinny_kernel<ABITS, WBITS, uint16_t, NT, RT, WAVES, STEP>, grid, dim3(64 * WAVES), lds, g, stream);
}

// Whether the weight-streaming kernel takes a product, and how.  Up to 32 tokens always, and 4-bit codes up to 64.
// Beyond, every workgroup passes its token tiles' packed codes through LDS and the vector unit for 32 or 64 features
// only, so its cost grows with K, the tiles per workgroup and their number in whole rounds of one per CU ("cost" = K nt
// ceil(groups / 256)); what the tiled kernels cost beside it are up to three launches (re-laying, product, finish) and
// weights of 6 or 8 bits per code.  So it takes products of few workgroups, one or two per CU, whatever the tokens and
// features are that make them, below a line of cost.  Both sides were timed on 14000 products (33-8192 tokens, K 256-16384,
// 128-27648 features; weights in cache and not) when the tiled side had no mid-size tiles, which only 4-bit layers ask for first
// (layer_streams); the others' lines have not been drawn again since: tiled / stream of the layer call, geometric mean, is 1.23 (4 / 4), 1.11
// (6 / 6), 1.12 (8 / 8) and 1.16 (8 / 4) where the rule streams, the worst 0.84, and 0.72-0.86 where it does not.  Around
// the lines (us of the layer call, stream : tiled):
//   4 / 4  two workgroups per CU: 128 tokens, 2048 -> 16384 17.5 : 24.0 (512 workgroups); 256, 1024 -> 12288 17.6 : 14.3
//          (768); 4096, 256 -> 4096 41.5 : 22.6 (4096); 90000, 50000 up to 32 workgroups (four parts of K in the tiled
//          kernels): 1024, 2048 -> 1024 15.7 : 25.3 (16k); 2048, 8192 -> 512 36 : 43 (66k); 247, 8448 -> 256 24.1 : 23.0 (68k, 16)
//   6 / 6, 8 / 8, 8 / 4  one workgroup per CU, two where the tiled kernels would split K and finish in a launch of its own:
//          256 tokens, 1024 -> 12288 6 / 6 27.4 : 14.2 (1152, K whole), 8 / 8 21.3 : 14.2 (768, K whole); 512, 1024 -> 2048 8 / 8
//          13.7 : 23.9 (256, split); 1024, 512 -> 2048 8 / 8 13.8 : 12.1 (512, K whole); lines, up to 64 workgroups (eight
//          parts of K) and beyond: 6 / 6 16000 / 28000, 8 / 8 20000 / 33000, 8 / 4 20000 / 40000 (96 tokens, 4096 -> 4096
//          8 / 4, 128 workgroups: 18 : 21 at 25k; 48, 4096 -> 256, 8: 15.0 : 13.7 at 16k)
//          in qllm_int_gemm, where the tiled path re-lays the activations in a launch of its own (4-6 us), two
//          workgroups per CU either way and 6 / 6 20000 / 33000, 8 / 8 28000 / 45000, 8 / 4 33000 / 70000
//          8 / 4 up to 64 tokens and more than 256 workgroups, which are half as many of 64 features, two per CU either way:
//          80000 up to 512, where the second round that is charged is not there, and beyond it or alone 100000 (64 tokens,
//          8960 -> 14336 30.7 : 34.9, weights not in cache 45 : 67; 33, 12288 -> 10240 33.9 : 32.8, alone 27.5 : 28.9; 33,
//          6144 -> 27648 34.2 : 36.2, alone 29.1 : 33.7).  6 / 6 and 8 / 8 lose there (64, 6144 -> 10240 28.6 : 24.8, 27.4 : 24.6)
// Where the weight came without its re-laid copy the tiled kernels expand packed codes (54-130 us up to 128 tokens): five
// workgroups per CU (512 tokens, 512 -> 6144 6 / 6 21 : 26 at 1152; 4096, 256 -> 1024 25 : 25 at 1376), 100000.
struct StreamPlan {
    bool take;
    int nt;         // 16-token tiles per workgroup
    int64_t groups; // workgroups, at 32 features each
};
StreamPlan plan_stream(int64_t N, int64_t K, int64_t O, int a_bits, int w_bits, bool relaid, bool relays_codes)
{
    const int64_t og = (O + 31) / 32;
    if (N <= 32) return StreamPlan{true, N <= 16 ? 1 : 2, og};
    const int64_t most = a_bits == 6 ? 6 : 8; // six-bit codes: registers for six tiles
    const int64_t tiles = (N + 15) / 16, blocks = (tiles + most - 1) / most, each = (tiles + blocks - 1) / blocks;
    const int nt = each <= 4 ? 4 : each <= 6 ? 6 : 8;
    const int64_t groups = og * blocks, cost = K * nt * ((groups + 255) / 256);
    const int64_t launched = nt == 4 && groups > 256 ? (groups + 1) / 2 : groups; // 64 features each, see launch_stream
    const bool few = groups <= 64;
    int64_t most_groups, line;
    if (a_bits == 4) {
        most_groups = 512, line = groups <= 32 ? 50000 : 90000;
    } else if (!relaid) {
        most_groups = 1280, line = 100000;
    } else if (relays_codes) {
        most_groups = 512, line = a_bits == 6 ? (few ? 20000 : 33000) : w_bits == 8 ? (few ? 28000 : 45000) : few ? 33000 : 70000;
    } else {
        most_groups = t8_splits(N, K, O) > 1 ? 512 : 256, line = a_bits == 6 ? (few ? 16000 : 28000) : few ? 20000 : w_bits == 8 ? 33000 : 40000;
    }
    if (relaid && a_bits == 8 && w_bits == 4 && nt == 4 && groups > 256) most_groups = 512, line = relays_codes || groups > 512 ? 100000 : 80000;
    const bool take = (a_bits == 4 && N <= 64) || (launched <= most_groups && cost <= line);
    return StreamPlan{take && blocks <= 65535, nt, groups};
}

template <int ABITS, int WBITS>
int32_t launch_stream(const GemmArgs &g, const StreamPlan &plan, int32_t y_dtype, hipStream_t stream)
{
    constexpr int STEP = ABITS == 8 ? 64 : 128; // 64-byte (6 bits: 96-byte) rows of LDS where there are many
    // more workgroups than CUs: smaller ones, several to a CU (16 tokens, 5120 -> 27648 4 / 4: 16.4 : 17.7 us)
    const bool wide = plan.groups > 256;
    if (plan.nt == 1) {
        if (wide) return launch_skinny<ABITS, WBITS, 1, 2, 4, 256>(g, y_dtype, stream);
        return launch_skinny<ABITS, WBITS, 1, 2, 8, 256>(g, y_dtype, stream);
    }
    if (plan.nt == 2) {
        if constexpr (ABITS == 8 && WBITS == 4) { // 5120 -> 27648: 27.3 : 31.7 us, 4096 -> 12288: 9.7 : 13.5
            if (wide) return launch_skinny<ABITS, WBITS, 2, 4, 8, STEP>(g, y_dtype, stream);
        } else if constexpr (ABITS == 6) { // 36.2 : 40, 13.8 : 16.8
            if (wide) return launch_skinny<ABITS, WBITS, 2, 2, 8, STEP>(g, y_dtype, stream);
        }
        return launch_skinny<ABITS, WBITS, 2, 2, 8, 256>(g, y_dtype, stream);
    }
    if (plan.nt == 4) {
        if (plan.groups > 512) return launch_skinny<ABITS, WBITS, 4, 4, 4, STEP>(g, y_dtype, stream); // 5120 -> 27648: 26.7 : 29.3 us with 8 waves
        if (wide) return launch_skinny<ABITS, WBITS, 4, 4, 8, STEP>(g, y_dtype, stream);              // 4096 -> 12288 6 / 6: 16.6 : 19 with 4 waves
        return launch_skinny<ABITS, WBITS, 4, 2, 8, STEP>(g, y_dtype, stream);
    }
    if (plan.nt == 6) {
        if (wide) return launch_skinny<ABITS, WBITS, 6, 2, 4, STEP>(g, y_dtype, stream);
        return launch_skinny<ABITS, WBITS, 6, 2, 8, STEP>(g, y_dtype, stream);
    }
    if constexpr (ABITS == 6) return QLLM_ERR_SHAPE; // not reached: at most six tiles
    else {
        if (wide) return launch_skinny<ABITS, WBITS, 8, 2, 4, STEP>(g, y_dtype, stream);
        return launch_skinny<ABITS, WBITS, 8, 2, 8, STEP>(g, y_dtype, stream);
    }
}

// Into how many parts K is split (1: not at all).  Only 4-bit codes with 128 x 128 tiles that leave
// most CUs without a workgroup (up to 64 tiles: four parts, up to 128: two; beyond that the parts'
// accumulators, written and read back, cost what the shorter K loop gains); every part keeps at least
// eight K-tiles.
int32_t k_splits(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    if (a_bits != 4 || N <= 64) return 1; // up to 64 tokens the weight-streaming kernel runs
    const int64_t tiles = ((O + 127) / 128) * ((N + 127) / 128);
    const int64_t n_kt = (K + QLLM_K_PAD - 1) / QLLM_K_PAD * QLLM_K_PAD / PKT;
    if (tiles > 128) return 1;
    int64_t s = 256 / tiles;
    if (s > 4) s = 4;
    if (s > n_kt / 8) s = n_kt / 8;
    return s < 2 ? 1 : (int32_t)s;
}

// gemm_mid_kernel on the FP6 matrix cores: in the layer call only, where the activations are laid out at no cost (qllm_int_gemm
// re-lays them in a launch of its own, which is what the streaming kernel and packed rows save).  Layer call, three sets of weights
// in turn, us, other kernel : this one:
//   128 x 64 in place of the streaming kernel or of K split, where these tiles are more than half a round:
//     100 x 4096 -> 12288 22.1 : 17.4, 66 x 5120 -> 9216 23.0 : 18.0, 128 x 6144 -> 16384 32.8 : 25.0, 200 x 5120 -> 5120 24.8 : 18.8,
//     256 x 8192 -> 8192 30.6 : 25.2, 512 x 4096 -> 4096 23.8 : 18.7, 1000 x 8192 -> 2048 38.2 : 33.0, 512 x 11008 -> 4096 38.1 : 33.3;
//     128 tiles are about even (100 x 8192 -> 8192 24.0 : 23.5, 66 x 4096 -> 8192 15.1 : 16.2), and so is a long K (160 x 28672 -> 8192
//     81.8 : 79.7, 256 tokens 88.6 : 95.3; 128 x 11008 -> 12288 45.5 : 45.5 / 47.0 : 46.8), where the streaming kernel's 4 bits per weight
//     are the fewer from HBM up to 128 tokens (/: out of every cache; 66 x 7680 -> 9216 24.1 : 23.2 / 27.1 : 29.1, 80 x 8192 -> 10240 26.8 : 24.5 / 29.2 :
//     30.0; 66 x 5120 -> 9216 22.2 : 18.6 / 26.4 : 23.1); more tokens lose up to 4 % there with three parts of K (1136 x 8448 -> 1024 39.5 : 36.1 /
//     40.0 : 41.6, 188 x 4096 -> 4864 19.3 : 17.5 / 19.4 : 19.8).  A short K stays with the streaming kernel: its
//     4 bits per weight are fewer from memory (250 x 1024 -> 6144 12.9 : 11.5, out of cache 16.6 : 17.8; 140 x 512 -> 8192 10.3 : 10.3 and 14.0 : 15.1;
//     160 x 2048 -> 8192 15.5 : 13.8 and 19.7 : 19.1)
//   160 x 64 where 128 x 128 tiles are more than half a round and these are one: 600 x 11008 -> 4096 41.1 : 37.1, 300 x 8192 -> 8192
//     33.1 : 30.9, 400 x 5120 -> 5120 23.7 : 22.5, 160 x 4096 -> 16384 20.8 : 19.8; 300 x 2048 -> 8192 15.6 : 15.7, 700 x 3000 -> 3000 19.6 : 19.0
//   128 x 128, as many of them: 400 x 28672 -> 8192 114.5 : 96.7, 1024 x 11008 -> 4096 47.3 : 45.7, 777 tokens 45.0 : 42.9; 400 x 8192
//     -> 8192 35.0 : 36.1.  Up to six columns of 128 features leave two XCDs without work: 3917 x 12864 -> 566 91.8 : 103.1, 3111 x 11264
//     -> 768 68.8 : 73.3 (eight, 3263 x 12416 -> 1024 82.9 : 84.4 / 91.0 : 87.5)
MidPlan plan_mid6(int64_t N, int64_t K, int64_t O)
{
    auto groups = [&](int64_t tm, int64_t tn) { return ((N + tm - 1) / tm) * ((O + tn - 1) / tn); };
    const int64_t half_tiles = groups(128, 64), tiles = groups(128, 128);
    if (half_tiles >= 144 && mid_fits(MidPlan{4, 2}, N, O) && K >= (N > 128 ? 2048 : 2304) && K <= 12288 && K * k_splits(N, K, O, 4) <= (N > 128 ? 30000 : 22000)) return MidPlan{4, 2};
    if (tiles > 128 && mid_fits(MidPlan{5, 2}, N, O) && K >= 3072) return MidPlan{5, 2};
    if (tiles > 128 && O > 6 * 128 && mid_fits(MidPlan{4, 4}, N, O) && K >= 10240) return MidPlan{4, 4};
    return MidPlan{0, 0};
}

// The kernel, tiles and parts of K of a product.
struct Route {
    int32_t kernel;    // QLLM_GEMM_*
    int32_t splits;    // parts of K
    TilePlan tiles;    // not for the streaming kernel
    MidPlan mid;       // operands in matrix-core order, K not split
    StreamPlan stream; // the streaming kernel only
};

// tiles6, tiles8: that path has its two operands (the weight's copy and room for the activations').  parts8: parts of a
// split K that the workspace holds on the byte-operand path.  a_laid: the activations are in tiles6 / tiles8 form already and
// nowhere else.  one_launch: nothing that takes two.
Route plan_route(int64_t N, int64_t K, int64_t O, int a_bits, int w_bits, bool tiles6, bool tiles8, int64_t parts8, bool a_laid, bool one_launch)
{
    const bool both4 = a_bits == 4 && w_bits == 4;
    Route r{QLLM_GEMM_EXPANDS, 1, TilePlan{true, 0}, MidPlan{0, 0}, plan_stream(N, K, O, a_bits, w_bits, both4 ? tiles6 : tiles8, true)};
    if (r.stream.take && !a_laid) {
        r.kernel = QLLM_GEMM_STREAMS;
    } else if (both4) {
        r.splits = k_splits(N, K, O, 4);
        if (tiles6) {
            r.kernel = QLLM_GEMM_FP6;
            if (a_laid) r.mid = plan_mid6(N, K, O);
            if (r.mid.mi) r.splits = 1;
            else if (r.splits == 1) r.tiles = plan_tiles(N, O, !one_launch);
        } else {
            // 256 x 256 tiles run one workgroup per CU, 128 x 128 tiles two, at about three quarters of the large tile's
            // rate per matrix-core operation: the small tile is taken where it fills the chip's rounds that much
            // better (few tiles, or a last round that is mostly empty: 384 large tiles are 1.5 rounds, 1536 small ones 3).
            const int64_t big_tiles = ((O + LBN - 1) / LBN) * ((N + LBM - 1) / LBM), small_tiles = ((O + 127) / 128) * ((N + 127) / 128);
            const double big_fill = (double)big_tiles / (double)(256 * ((big_tiles + 255) / 256));
            const double small_fill = (double)small_tiles / (double)(512 * ((small_tiles + 511) / 512));
            r.tiles.small = N <= 128 || big_fill < 0.78 * small_fill;
            if (!r.tiles.small) r.splits = 1;
        }
    } else if (tiles8) {
        r.kernel = QLLM_GEMM_BYTES;
        const int64_t s = t8_splits(N, K, O);
        r.mid = plan_mid8(N, K, O, a_bits);
        if (r.mid.mi) return r;
        if (s > 1 && parts8 > 1) r.splits = (int32_t)(parts8 < s ? parts8 : s);
        else r.tiles = plan_tiles(N, O, !one_launch);
    } else {
        r.tiles.small = N <= 128;
    }
    return r;
}

template <int ABITS, int WBITS>
int32_t launch(const GemmArgs &g, const Route &route, int32_t y_dtype, hipStream_t stream)
{
    if (route.kernel == QLLM_GEMM_STREAMS) return launch_stream<ABITS, WBITS>(g, route.stream, y_dtype, stream);
    const bool small = route.tiles.small;
    const dim3 big_grid((unsigned)((g.O + LBN - 1) / LBN), (unsigned)((g.N + LBM - 1) / LBM));
    if constexpr (ABITS == 4 && WBITS == 4) {
        if (route.kernel == QLLM_GEMM_FP6) return launch_fp6(g, route.tiles, route.mid, y_dtype, stream);
        if (small) {
            const dim3 grid((unsigned)((g.O + 127) / 128), (unsigned)((g.N + 127) / 128), (unsigned)(g.splits > 1 ? g.splits : 1));
            constexpr size_t lds = (size_t)NBUF * 256 * PROWB;
            if (g.splits > 1) {
                const int32_t st = launch_kernel(int_gemm_w4a4_kernel<float, 4, 2, true>, grid, dim3(LTHREADS), lds, g, stream);
                if (st != QLLM_OK) return st;
                return launch_finish<0, 0>(g, y_dtype, stream);
            }
            if (y_dtype == QLLM_F32) return launch_kernel(int_gemm_w4a4_kernel<float, 4, 2>, grid, dim3(LTHREADS), lds, g, stream);
            return launch_kernel(int_gemm_w4a4_kernel<uint16_t, 4, 2>, grid, dim3(LTHREADS), lds, g, stream);
        }
        if (y_dtype == QLLM_F32) return launch_kernel(int_gemm_w4a4_kernel<float, 8, 4>, big_grid, dim3(LTHREADS), NBUF * PBUF, g, stream);
        return launch_kernel(int_gemm_w4a4_kernel<uint16_t, 8, 4>, big_grid, dim3(LTHREADS), NBUF * PBUF, g, stream);
    } else {
        if (route.kernel == QLLM_GEMM_BYTES) return launch_t8<ABITS, WBITS>(g, route.tiles, route.mid, y_dtype, stream);
        if (small) { // 33..128 tokens
            const dim3 grid((unsigned)((g.O + BN - 1) / BN), (unsigned)((g.N + BM - 1) / BM));
            if (y_dtype == QLLM_F32) return launch_kernel(int_gemm_kernel<ABITS, WBITS, float>, grid, dim3(THREADS), 0, g, stream);
            return launch_kernel(int_gemm_kernel<ABITS, WBITS, uint16_t>, grid, dim3(THREADS), 0, g, stream);
        }
        if (y_dtype == QLLM_F32) return launch_kernel(int_gemm_big_kernel<ABITS, WBITS, float>, big_grid, dim3(LTHREADS), 2 * LBUF, g, stream);
        return launch_kernel(int_gemm_big_kernel<ABITS, WBITS, uint16_t>, big_grid, dim3(LTHREADS), 2 * LBUF, g, stream);
    }
}

// Largest L such that |beta_x| < L and |beta_w| < L keep the epilogue inside narrow integers: row and column
// sums and K * beta_x below 2^23 (24-bit multiplies), and the accumulator together with the three correction
// terms -- in whatever order they are added -- below 2^31 in magnitude:
//     K * (qa * qw + (qa + qw) * L + L * L)  <  2^31,
// the largest value sum((a - beta_x) * (w - beta_w)) and each of its partial sums can take.
int32_t small_zero_bound(int64_t K, int32_t a_bits, int32_t w_bits)
{
    const int64_t qa = (1 << a_bits) - 1, qw = (1 << w_bits) - 1, qm = qa > qw ? qa : qw;
    if (qm * K >= (1 << 23) || qa * qw * K >= (1ll << 31)) return 0;
    int64_t L = 1 << 20;
    while (L > 0 && (K * L >= (1 << 23) || K * (qa * qw + (qa + qw) * L + L * L) >= (1ll << 31))) L /= 2;
    return (int32_t)L;
}

} // namespace

extern "C" int64_t qllm_gemm_workspace_floor_bytes(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    if (a_bits != 4 && a_bits != 6 && a_bits != 8) return QLLM_ERR_BITS;
    if (N < 0 || K <= 0 || O <= 0) return QLLM_ERR_SHAPE;
    const int32_t s = k_splits(N, K, O, a_bits);
    return s > 1 ? (int64_t)s * N * O * (int64_t)sizeof(int32_t) : 0;
}

extern "C" int64_t qllm_gemm_workspace_bytes(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    const int64_t floor_bytes = qllm_gemm_workspace_floor_bytes(N, K, O, a_bits);
    if (floor_bytes < 0) return floor_bytes;
    if (N <= 32 || (a_bits == 4 && N <= 64)) return floor_bytes; // the weight-streaming kernel needs none
    // 4-bit codes: the parts' accumulators where K is split (the floor), then the activations' tiles for the FP6 path
    if (a_bits == 4) return 225 * K < (1 << 24) ? (floor_bytes + 255) / 256 * 256 + qllm_tiles6_bytes(N, K) : floor_bytes;
    // the byte-operand path: the activations' bytes, then the parts' accumulators where it splits K
    const int32_t s8 = t8_splits(N, K, O);
    return (qllm_tiles8_bytes(N, K) + 255) / 256 * 256 + (s8 > 1 ? (int64_t)s8 * N * O * (int64_t)sizeof(int32_t) : 0);
}

namespace {

// The byte-operand path of the other bit pairs: more than 32 tokens, the weight's tiles at hand and room for the
// activations' in the workspace.
bool has_room_for_tiles8(int64_t N, const qllm_weight *w, int32_t a_bits, const void *workspace, int64_t workspace_bytes)
{
    return !(a_bits == 4 && w->bits == 4) && w->tiles8 && N > 32 && workspace && workspace_bytes >= qllm_tiles8_bytes(N, w->K) &&
           qllm_tiles8_bytes(N, w->K) < (1ll << 32) && qllm_tiles8_bytes(w->O, w->K) < (1ll << 32);
}

// Where the FP6 path's activations go in the workspace: behind the parts of a split K, whether the sum is split or streamed.
int64_t tiles6_at(int64_t N, int64_t K, int64_t O)
{
    return (qllm_gemm_workspace_floor_bytes(N, K, O, 4) + 255) / 256 * 256;
}

// The FP6 path: 4-bit codes, more than 64 tokens, the weight's tiles at hand and room for the activations'.  The kernel
// addresses either operand with 32-bit offsets.
bool has_room_for_tiles6(int64_t N, const qllm_weight *w, int32_t a_bits, const void *workspace, int64_t workspace_bytes)
{
    return a_bits == 4 && w->bits == 4 && w->tiles6 && N > 64 && workspace && 225 * w->K < (1 << 24) &&
           workspace_bytes >= tiles6_at(N, w->K, w->O) + qllm_tiles6_bytes(N, w->K) && qllm_tiles6_bytes(N, w->K) < (1ll << 32) &&
           qllm_tiles6_bytes(w->O, w->K) < (1ll << 32);
}

// Whether the layer call's product takes packed rows from the fused kernel because the streaming kernel is the cheaper way.
bool layer_streams(int64_t N, const qllm_weight *w, int32_t a_bits, bool tiles6)
{
    return plan_stream(N, w->K, w->O, a_bits, w->bits, true, false).take && !(tiles6 && plan_mid6(N, w->K, w->O).mi);
}

// The byte-operand path's workspace: the activations, then as many parts of a split K as fit behind them.
int64_t parts8_at(int64_t N, int64_t K) { return (qllm_tiles8_bytes(N, K) + 255) / 256 * 256; }
int64_t parts8_that_fit(int64_t N, int64_t K, int64_t O, int64_t workspace_bytes)
{
    return (workspace_bytes - parts8_at(N, K)) / (N * O * (int64_t)sizeof(int32_t));
}

// The arguments of qllm_int_gemm.
int32_t check_product(const qllm_qact *a, int32_t a_bits, int64_t N, const qllm_weight *w, const void *y, int32_t y_dtype, int64_t ldy,
                      const void *workspace, int64_t workspace_bytes)
{
    if (!a || !w || !y) return QLLM_ERR_NULL;
    if (!a->codes || !a->scale || !a->zero || !a->rowsum) return QLLM_ERR_NULL;
    if (!w->codes || !w->scale || !w->zero || !w->colsum) return QLLM_ERR_NULL;
    if (y_dtype != QLLM_F32 && y_dtype != QLLM_BF16) return QLLM_ERR_DTYPE;
    const int32_t wb = w->bits;
    const bool pair_ok = (a_bits == wb && (wb == 4 || wb == 6 || wb == 8)) || (a_bits == 8 && wb == 4);
    if (!pair_ok) return QLLM_ERR_BITS;
    if (N < 0 || N > INT32_MAX || w->O <= 0 || w->O > INT32_MAX || w->K <= 0 || w->K > (1 << 24) || ldy < w->O)
        return QLLM_ERR_SHAPE;
    // the largest possible sum of products must stay inside int32
    const int64_t qa = (1 << a_bits) - 1, qw = (1 << wb) - 1;
    if (qa * qw * w->K > INT32_MAX) return QLLM_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(a->codes) & 15u) || (reinterpret_cast<uintptr_t>(w->codes) & 15u))
        return QLLM_ERR_ALIGN;
    if (workspace_bytes < qllm_gemm_workspace_floor_bytes(N, w->K, w->O, a_bits)) return QLLM_ERR_WORKSPACE;
    if (N == 0) return QLLM_OK;
    const bool ws_aligned = (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0;
    if (wb == 4 && k_splits(N, w->K, w->O, a_bits) > 1 && (!workspace || !ws_aligned)) return workspace ? QLLM_ERR_ALIGN : QLLM_ERR_WORKSPACE;
    if (has_room_for_tiles6(N, w, a_bits, workspace, workspace_bytes) && (!ws_aligned || (reinterpret_cast<uintptr_t>(w->tiles6) & 15u)))
        return QLLM_ERR_ALIGN;
    if (has_room_for_tiles8(N, w, a_bits, workspace, workspace_bytes) && (!ws_aligned || (reinterpret_cast<uintptr_t>(w->tiles8) & 15u)))
        return QLLM_ERR_ALIGN;
    return QLLM_OK;
}

// qllm_int_gemm; a_laid: the activations already lie where the workspace has them in tiles6 or tiles8 layout, and the
// path that reads them there is the one that runs.
int32_t int_gemm(const qllm_qact *a, int32_t a_bits, int64_t N, const qllm_weight *w, void *y, int32_t y_dtype, int64_t ldy,
                 int32_t *acc_dump, void *workspace, int64_t workspace_bytes, bool a_laid, void *hip_stream)
{
    const int32_t rc = check_product(a, a_bits, N, w, y, y_dtype, ldy, workspace, workspace_bytes);
    if (rc != QLLM_OK || N == 0) return rc;
    const int32_t wb = w->bits;

    GemmArgs g{};
    g.a_codes = a->codes;
    g.w_codes = w->codes;
    g.a_row_bytes = qllm_packed_row_bytes(w->K, a_bits);
    g.w_row_bytes = qllm_packed_row_bytes(w->K, wb);
    g.ax = a->scale; g.bx = a->zero; g.rs = a->rowsum;
    g.aw = w->scale; g.bw = w->zero; g.cs = w->colsum;
    g.N = (int32_t)N; g.O = (int32_t)w->O; g.K = (int32_t)w->K;
    g.Kpad = (int32_t)((w->K + QLLM_K_PAD - 1) / QLLM_K_PAD * QLLM_K_PAD);
    g.y = y; g.ldy = ldy; g.acc_dump = acc_dump;
    const bool tiles6 = has_room_for_tiles6(N, w, a_bits, workspace, workspace_bytes);
    const bool tiles8 = has_room_for_tiles8(N, w, a_bits, workspace, workspace_bytes);
    const Route route = plan_route(N, w->K, w->O, a_bits, wb, tiles6, tiles8, tiles8 ? parts8_that_fit(N, w->K, w->O, workspace_bytes) : 0,
                                   a_laid, acc_dump != nullptr);
    g.splits = route.splits;
    g.partial = static_cast<int32_t *>(workspace);
    if (tiles6) {
        g.a_tiles = static_cast<const uint8_t *>(workspace) + tiles6_at(N, w->K, w->O);
        g.w_tiles = w->tiles6;
    }
    g.a_laid = a_laid;
    if (tiles8) {
        g.a_tiles8 = static_cast<const uint8_t *>(workspace);
        g.w_tiles8 = w->tiles8;
        g.partial = reinterpret_cast<int32_t *>(static_cast<uint8_t *>(workspace) + parts8_at(N, w->K));
    }
    g.small_zero = small_zero_bound(w->K, a_bits, wb);
    // finish_from_lds: sums that fit 24 bits (see there), no raw accumulators
    const int64_t q_most = (1 << (a_bits > wb ? a_bits : wb)) - 1;
    g.lds_epilogue = !acc_dump && q_most * w->K < (1 << 23) &&
                     (a_bits != 4 || wb != 4 || 225 * w->K < (1 << 24));
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    if (a_bits == 4) return launch<4, 4>(g, route, y_dtype, stream);
    if (a_bits == 6) return launch<6, 6>(g, route, y_dtype, stream);
    if (wb == 8) return launch<8, 8>(g, route, y_dtype, stream);
    return launch<8, 4>(g, route, y_dtype, stream);
}

} // namespace

extern "C" int32_t qllm_int_gemm(const qllm_qact *a, int32_t a_bits, int64_t N, const qllm_weight *w, void *y,
                                 int32_t y_dtype, int64_t ldy, int32_t *acc_dump, void *workspace,
                                 int64_t workspace_bytes, void *hip_stream)
{
    return int_gemm(a, a_bits, N, w, y, y_dtype, ldy, acc_dump, workspace, workspace_bytes, false, hip_stream);
}

namespace {

// The route of qllm_int_gemm, or of the layer call's product, without a launch.
int32_t describe_route(const qllm_weight *w, int32_t a_bits, int64_t N, int64_t workspace_bytes, int32_t in_layer, Route *r)
{
    const int32_t wb = w->bits;
    if (!((a_bits == wb && (wb == 4 || wb == 6 || wb == 8)) || (a_bits == 8 && wb == 4))) return QLLM_ERR_BITS;
    if (N <= 0 || N > INT32_MAX || w->O <= 0 || w->O > INT32_MAX || w->K <= 0 || w->K > (1 << 24)) return QLLM_ERR_SHAPE;
    if (workspace_bytes < qllm_gemm_workspace_floor_bytes(N, w->K, w->O, a_bits)) return QLLM_ERR_WORKSPACE;
    const void *some = w; // any address: only whether there is a workspace counts
    const bool tiles8 = has_room_for_tiles8(N, w, a_bits, some, workspace_bytes);
    const bool tiles6 = has_room_for_tiles6(N, w, a_bits, some, workspace_bytes);
    *r = plan_route(N, w->K, w->O, a_bits, wb, tiles6, tiles8, tiles8 ? parts8_that_fit(N, w->K, w->O, workspace_bytes) : 0,
                    in_layer && (tiles6 || tiles8) && !layer_streams(N, w, a_bits, tiles6), false);
    return QLLM_OK;
}

} // namespace

extern "C" int32_t qllm_gemm_kernel_choice(const qllm_weight *w, int32_t a_bits, int64_t N, int64_t workspace_bytes, int32_t in_layer,
                                           int32_t *tile, int32_t *parts)
{
    if (!w || !tile || !parts) return QLLM_ERR_NULL;
    Route r;
    const int32_t rc = describe_route(w, a_bits, N, workspace_bytes, in_layer, &r);
    if (rc != QLLM_OK) return rc;
    *parts = r.splits;
    *tile = r.kernel == QLLM_GEMM_STREAMS ? 0 : r.tiles.o_split > 0 ? 256 + 128 : r.tiles.small ? 128 : 256;
    return r.kernel;
}

extern "C" int32_t qllm_probe_mid_tile(const qllm_weight *w, int32_t a_bits, int64_t N, int64_t workspace_bytes, int32_t in_layer,
                                       int32_t *tokens, int32_t *features)
{
    if (!w || !tokens || !features) return QLLM_ERR_NULL;
    Route r;
    const int32_t rc = describe_route(w, a_bits, N, workspace_bytes, in_layer, &r);
    if (rc != QLLM_OK) return rc;
    *tokens = 32 * r.mid.mi;
    *features = 32 * r.mid.nj;
    return QLLM_OK;
}

extern "C" int64_t qllm_tiles6_bytes(int64_t rows, int64_t K)
{
    if (rows < 0 || K <= 0) return QLLM_ERR_SHAPE;
    const int64_t Kpad = (K + QLLM_K_PAD - 1) / QLLM_K_PAD * QLLM_K_PAD;
    return (rows + 15) / 16 * (Kpad / T6_KT) * T6_BLOCK;
}

extern "C" int32_t qllm_pack_tiles6(const uint8_t *codes, int64_t rows, int64_t K, uint8_t *tiles, void *hip_stream)
{
    if (!codes || !tiles) return QLLM_ERR_NULL;
    if (rows < 0 || rows > INT32_MAX || K <= 0 || K > (1 << 24)) return QLLM_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(codes) & 15u) || (reinterpret_cast<uintptr_t>(tiles) & 15u)) return QLLM_ERR_ALIGN;
    if (rows == 0) return QLLM_OK;
    const int64_t Kpad = (K + QLLM_K_PAD - 1) / QLLM_K_PAD * QLLM_K_PAD;
    return launch_tiles6<false>(codes, qllm_packed_row_bytes(K, 4), rows, Kpad, tiles, reinterpret_cast<hipStream_t>(hip_stream));
}

extern "C" int64_t qllm_tiles8_bytes(int64_t rows, int64_t K)
{
    if (rows < 0 || K <= 0) return QLLM_ERR_SHAPE;
    return (rows + 15) / 16 * ((K + T8_KT - 1) / T8_KT) * T8_BLOCK;
}

extern "C" int32_t qllm_pack_tiles8(const uint8_t *codes, int32_t bits, int64_t rows, int64_t K, uint8_t *tiles, void *hip_stream)
{
    if (!codes || !tiles) return QLLM_ERR_NULL;
    if (bits != 4 && bits != 6 && bits != 8) return QLLM_ERR_BITS;
    if (rows < 0 || rows > INT32_MAX || K <= 0 || K > (1 << 24)) return QLLM_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(codes) & 15u) || (reinterpret_cast<uintptr_t>(tiles) & 15u)) return QLLM_ERR_ALIGN;
    if (rows == 0) return QLLM_OK;
    return launch_tiles8(codes, bits, rows, K, tiles, reinterpret_cast<hipStream_t>(hip_stream));
}

namespace {

// What the layer needs at least (quantized activations + what the GEMM needs whatever path it takes), and the
// room that lets the GEMM take its FP6 path when the weight comes with tiles.
int64_t layer_workspace_floor(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    const int64_t gw = qllm_gemm_workspace_floor_bytes(N, K, O, a_bits);
    if (gw < 0) return gw;
    const int64_t rb = qllm_packed_row_bytes(K, a_bits);
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    return up(N * rb) + 3 * up(N * 4) + up(gw);
}

// What the product of a layer call is going to read of its weights, workgroup by workgroup: the small tiles of up to 128
// tokens, which are numbered along the features.  Not for the streaming kernel, which loses as often as it gains by it
// (layer, us, without : with: 16 tokens 8192 -> 28672 4 / 4 33.5 : 32.6, 28672 -> 8192 6 / 6 57.2 : 58.0, 90 tokens 13824 -> 5120
// 28.8 : 30.0: unpacking bounds it, not the weights' way).
WeightsAhead weights_ahead(int64_t N, const qllm_weight *w, bool tiles6, int32_t splits)
{
    if (N > 128) return WeightsAhead{nullptr, 0, 0, 0, 0, 0};
    const int32_t cols = (int32_t)((w->O + 127) / 128);
    if (tiles6) return WeightsAhead{w->tiles6, qllm_tiles6_bytes(w->O, w->K), (int32_t)qllm_tiles6_bytes(16, w->K), T6_BLOCK, cols, splits};
    return WeightsAhead{w->tiles8, qllm_tiles8_bytes(w->O, w->K), (int32_t)qllm_tiles8_bytes(16, w->K), T8_BLOCK, cols, splits};
}

// What the layer call asks of the fused kernel beyond packed rows: where the product is going to read its activations in
// matrix-core order, the fused kernel writes them so (one launch and a pass over the codes less), and with few tokens reads
// the product's weights ahead.  p, left: the workspace behind the packed rows.
struct LayerAsks {
    uint8_t *tiles; // null: packed rows
    WeightsAhead ahead;
};
LayerAsks layer_asks(int64_t N, const qllm_weight *w, int32_t a_bits, uint8_t *p, int64_t left)
{
    LayerAsks l{nullptr, {nullptr, 0, 0, 0, 0, 0}};
    const bool tiles6 = has_room_for_tiles6(N, w, a_bits, p, left);
    if (layer_streams(N, w, a_bits, tiles6)) return l;
    if (tiles6) l.tiles = p + tiles6_at(N, w->K, w->O);
    else if (has_room_for_tiles8(N, w, a_bits, p, left)) l.tiles = p;
    const int64_t parts8 = l.tiles && !tiles6 ? parts8_that_fit(N, w->K, w->O, left) : 0;
    if (l.tiles) l.ahead = weights_ahead(N, w, tiles6, plan_route(N, w->K, w->O, a_bits, w->bits, tiles6, !tiles6, parts8, true, false).splits);
    return l;
}

} // namespace

extern "C" int64_t qllm_workspace_floor_bytes(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    return layer_workspace_floor(N, K, O, a_bits);
}

extern "C" int64_t qllm_workspace_bytes(int64_t N, int64_t K, int64_t O, int32_t a_bits)
{
    const int64_t floor_bytes = layer_workspace_floor(N, K, O, a_bits);
    if (floor_bytes < 0) return floor_bytes;
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    return floor_bytes - up(qllm_gemm_workspace_floor_bytes(N, K, O, a_bits)) + up(qllm_gemm_workspace_bytes(N, K, O, a_bits));
}

namespace {

// halves: 1 the fused kernel, 2 the product on what it left in the workspace, 3 both
int32_t layer_call(int halves, const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx, int32_t norm, const float *gamma,
                   const float *beta, float eps, const qllm_map *map, int32_t a_bits, const qllm_weight *w, void *y, int32_t y_dtype,
                   int64_t ldy, void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    if (!map || !w) return QLLM_ERR_NULL;
    if (w->K != map->C_out) return QLLM_ERR_SHAPE;
    if (N < 0) return QLLM_ERR_SHAPE;
    const int64_t need = layer_workspace_floor(N, map->C_out, w->O, a_bits); // more lets the GEMM take its FP6 path
    if (need < 0) return (int32_t)need;
    if (N == 0) return QLLM_OK; // nothing to do, whatever the workspace
    if (!workspace || workspace_bytes < need) return QLLM_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return QLLM_ERR_ALIGN;
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    uint8_t *p = static_cast<uint8_t *>(workspace);
    qllm_qact q;
    q.codes = p;
    p += up(N * qllm_packed_row_bytes(map->C_out, a_bits));
    q.scale = reinterpret_cast<float *>(p);
    p += up(N * 4);
    q.zero = reinterpret_cast<int32_t *>(p);
    p += up(N * 4);
    q.rowsum = reinterpret_cast<int32_t *>(p);
    p += up(N * 4);
    const int64_t left = workspace_bytes - (p - static_cast<uint8_t *>(workspace));
    // both halves' arguments before either is launched: a call that is refused touches nothing, the weights neither
    qllm_detail::FusedArgs fused{};
    int32_t rc = qllm_fused_prepare(x, x_dtype, N, C, ldx, norm, gamma, beta, eps, map, a_bits, &q, &fused);
    if (rc != QLLM_OK) return rc;
    rc = check_product(&q, a_bits, N, w, y, y_dtype, ldy, p, left);
    if (rc != QLLM_OK) return rc;
    const LayerAsks ask = layer_asks(N, w, a_bits, p, left);
    bool laid = qllm_fused_lays(fused, x_dtype, a_bits, ask.tiles);
    if (halves & 1) rc = qllm_fused_run(fused, x_dtype, a_bits, ask.tiles, &laid, ask.ahead.base ? &ask.ahead : nullptr, hip_stream);
    if (rc != QLLM_OK || !(halves & 2)) return rc;
    return int_gemm(&q, a_bits, N, w, y, y_dtype, ldy, nullptr, p, left, laid, hip_stream);
}

} // namespace

extern "C" int32_t qllm_reassembled_linear(const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx,
                                           int32_t norm, const float *gamma, const float *beta, float eps,
                                           const qllm_map *map, int32_t a_bits, const qllm_weight *w, void *y,
                                           int32_t y_dtype, int64_t ldy, void *workspace, int64_t workspace_bytes,
                                           void *hip_stream)
{
    return layer_call(3, x, x_dtype, N, C, ldx, norm, gamma, beta, eps, map, a_bits, w, y, y_dtype, ldy, workspace, workspace_bytes, hip_stream);
}

extern "C" int32_t qllm_probe_layer_half(int32_t half, const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx, int32_t norm,
                                         const float *gamma, const float *beta, float eps, const qllm_map *map, int32_t a_bits,
                                         const qllm_weight *w, void *y, int32_t y_dtype, int64_t ldy, void *workspace,
                                         int64_t workspace_bytes, void *hip_stream)
{
    if (half != 1 && half != 2) return QLLM_ERR_SHAPE;
    return layer_call(half, x, x_dtype, N, C, ldx, norm, gamma, beta, eps, map, a_bits, w, y, y_dtype, ldy, workspace, workspace_bytes, hip_stream);
}

extern "C" int32_t qllm_probe_layer_launch(const qllm_map *map, int32_t x_dtype, int64_t N, int64_t ldx, int32_t norm, int32_t has_beta,
                                           int32_t a_bits, const qllm_weight *w, int64_t workspace_bytes, qllm_layer_launch *out)
{
    if (!map || !w || !out) return QLLM_ERR_NULL;
    if (w->K != map->C_out || N <= 0) return QLLM_ERR_SHAPE;
    const int64_t need = layer_workspace_floor(N, map->C_out, w->O, a_bits);
    if (need < 0) return (int32_t)need;
    if (workspace_bytes < need) return QLLM_ERR_WORKSPACE;
    qllm_detail::FusedArgs fused{};
    const int32_t rc = qllm_fused_describe(map, x_dtype, N, ldx, norm, has_beta, a_bits, &fused);
    if (rc != QLLM_OK) return rc;
    uint8_t *const some = reinterpret_cast<uint8_t *>(4096); // any address: only whether there is a workspace counts
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    const LayerAsks ask = layer_asks(N, w, a_bits, some, workspace_bytes - up(N * qllm_packed_row_bytes(w->K, a_bits)) - 3 * up(N * 4));
    return qllm_fused_launch_facts(fused, x_dtype, a_bits, ask.tiles, ask.ahead.base ? &ask.ahead : nullptr, out);
}

// ---- the layer for callers that cannot allocate: its workspace is a device array of this library

namespace {

// Device memory beyond the inputs and outputs of the layer: the quantized activations between the two kernels
// and, where the sum over K is split over workgroups, their partial accumulators.  One copy per GPU, held from
// the moment the code object is loaded on it until the process ends.  In host code this name is only a handle:
// the address on the current device comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[QLLM_STATIC_WORKSPACE_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex scratch_lock;
void *scratch_at[MAX_DEVICES]; // the array's address on each device, asked for once

int32_t scratch_pointer(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        qllm_note_hip_error("static workspace: current device", e != hipSuccess ? hipGetErrorName(e) : "device number out of range");
        return QLLM_ERR_HIP;
    }
    std::lock_guard<std::mutex> hold(scratch_lock);
    if (!scratch_at[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            qllm_note_hip_error("static workspace: address of the device array", e != hipSuccess ? hipGetErrorName(e) : "null address");
            return QLLM_ERR_HIP;
        }
        scratch_at[dev] = p;
    }
    *out = scratch_at[dev];
    return QLLM_OK;
}

} // namespace

extern "C" int32_t qllm_reassembled_linear_static(const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx,
                                                  int32_t norm, const float *gamma, const float *beta, float eps,
                                                  const qllm_map *map, int32_t a_bits, const qllm_weight *w, void *y,
                                                  int32_t y_dtype, int64_t ldy, void *hip_stream)
{
    if (!map || !w) return QLLM_ERR_NULL;
    if (w->K != map->C_out) return QLLM_ERR_SHAPE;
    if (N < 0) return QLLM_ERR_SHAPE;
    const int64_t need = layer_workspace_floor(N, map->C_out, w->O, a_bits);
    if (need < 0) return (int32_t)need;
    if (need > (int64_t)QLLM_STATIC_WORKSPACE_BYTES) return QLLM_ERR_WORKSPACE; // too large a batch for the built-in workspace
    if (N == 0) return QLLM_OK;
    void *ws = nullptr;
    const int32_t rc = scratch_pointer(&ws);
    if (rc != QLLM_OK) return rc;
    return qllm_reassembled_linear(x, x_dtype, N, C, ldx, norm, gamma, beta, eps, map, a_bits, w, y, y_dtype, ldy, ws,
                                   (int64_t)QLLM_STATIC_WORKSPACE_BYTES, hip_stream);
}
