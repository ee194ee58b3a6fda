// Internal to libqllm: what the two fused-kernel translation units share.
#ifndef QLLM_FUSED_COMMON_H
#define QLLM_FUSED_COMMON_H

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "qllm.h"
#include "qllm_probes.h"

extern "C" void qllm_note_hip_error(const char *step, const char *name);

namespace qllm_detail {

constexpr int GROUP = QLLM_MAP_GROUP; // 8 channels per lane and step
constexpr float MAGIC = 12582912.0f;  // 1.5 * 2^23: x + MAGIC rounds x to an integer, ties to even
constexpr int32_t MAGIC_BITS = 0x4B400000;
constexpr float FAST_LIMIT = 2097152.0f; // 2^21: below it the MAGIC trick is exact

// x / d by one multiplication, exact for x d < 2^32: x ceil(2^32 / d) / 2^32 is less than x d / 2^32 / d too large
struct QuotientBy {
    uint32_t d, m;
    __device__ __forceinline__ uint32_t divide(uint32_t x) const { return d == 1u ? x : __umulhi(x, m); }
};
inline QuotientBy quotient_by(uint32_t d) { return QuotientBy{d, d > 1u ? 0xffffffffu / d + 1u : 0u}; }

struct FusedArgs {
    const void *x;
    int64_t ldx;
    int32_t N, C, norm, vec_ok;
    const float *gamma, *beta;
    float eps;
    double inv_C; // 1 / C
    const int32_t *row_ptr, *src, *desc;
    const float *scale;
    const int32_t *work, *chunks, *spec, *dest, *longs, *segs, *recs, *xlrows, *xlent; // the parts of the plan (see qllm_plan_map_host)
    int32_t n_comp, n_long, n_pub, n_work, n_chunks, n_spec, n_dest, n_segw, n_xl;
    int32_t C_out, n_groups, n_groups_pad, S;
    uint8_t *codes;
    int64_t row_bytes;
    float *alpha;
    int32_t *zero, *rowsum;
    uint8_t *tiles; // not null: the codes leave as the product reads them, TILES6 in the activations' order (4 bits, see tiles6_x) or TILES8
    int32_t tiles_kt; // its K-tiles per row
    int32_t row_at; // 4 bits: where in LDS (dwords) the row is put together before it leaves
    int32_t row_groups; // workgroups that have rows
    // calibration variant
    float *absmax, *y_dump;
    int32_t n_dump;
    // Workgroups beyond the rows' read weights that the product after this kernel is going to need (see read_ahead)
    const uint8_t *ahead;
    int64_t ahead_total;    // bytes of the weights; 0: none of this
    int32_t ahead_block;    // of a block of 16 features
    uint32_t ahead_tile, ahead_kt;      // of one of its K-tiles; their number
    QuotientBy ahead_cols, ahead_splits; // the product's workgroups: 8 blocks each, one after the other, times parts of K
    int32_t ahead_each;     // bytes to read for every workgroup: its first blocks
    QuotientBy ahead_pieces, ahead_of_block; // the same in KB; KB of a block's part of K
};

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// ---- Eq. (2) for one value; the row's parameters are uniform over the workgroup
// rne(x*inv) on the exact product.  Fast form: one fused multiply-add against MAGIC, whose single
// rounding lands on the integer grid.  Slow form (huge quotients): the product is exact in fp64.
__device__ __forceinline__ int32_t rne_product_fast(float x, float inv)
{
    return __float_as_int(__builtin_fmaf(x, inv, MAGIC)) - MAGIC_BITS;
}

__device__ __forceinline__ double rne_product_slow(float x, float inv)
{
    return rint((double)x * (double)inv);
}

template <int QMAX>
__device__ __forceinline__ int32_t quant_code(float x, float inv, int32_t beta, int32_t fast)
{
    if (fast) {
        const int32_t q = rne_product_fast(x, inv) + beta; // both below 2^22 in magnitude
        return q < 0 ? 0 : (q > QMAX ? QMAX : q);
    }
    const double q = rne_product_slow(x, inv) + (double)beta;
    return (int32_t)fmin(fmax(q, 0.0), (double)QMAX);
}

// ---- TILES6, the operand layout of the FP6 path (see qllm_pack_tiles6): 32 packed 4-bit codes of a row -> what one lane of a
// matrix-core operand read finds, its first 16 bytes and its last 8
constexpr int TILES6_BLOCK = 1536, TILES6_X = 1024; // bytes per block of 16 rows and K-tile of 128 codes; where the last 8 bytes lie
// Where they lie in the block for codes 32 q .. of row r.  Weights: in the order of the lanes, 16 q + r.  Activations are
// written a row at a time, so there a row's bytes are neighbours, 64 and 32 of them, one request each to the caches
// where the lanes' order makes four; the pieces of a row are swapped by its number so that an operand read from LDS
// finds every lane on banks of its own (4.3 clocks per 16-byte read, 8.1 in plain order).
__device__ __forceinline__ int tiles6_x(int r, int q) { return 64 * r + 16 * (q ^ (r >> 1 & 3)); }
__device__ __forceinline__ int tiles6_y(int r, int q) { return TILES6_X + 32 * r + 8 * (q ^ (r >> 2)); }

// 4 nibbles in bits 0..15 -> four 6-bit fields in bits 0..23
__device__ __forceinline__ uint32_t spread4(uint32_t x)
{
    const uint32_t y = (x & 0xffu) | ((x & 0xff00u) << 4); // nibbles 0, 1 in bits 0..7; 2, 3 in bits 12..19
    return (y & 0x00f00fu) | ((y & 0x0f00f0u) << 2);       // nibble k in bits 6 k .. 6 k + 3
}

struct Lane6 {
    uint4 x;
    uint2 y;
};
__device__ __forceinline__ Lane6 lane6(const uint4 &codes)
{
    const uint32_t w[4] = {codes.x, codes.y, codes.z, codes.w};
    uint32_t s[8]; // eight pieces of 24 bits
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s[2 * i] = spread4(w[i] & 0xffffu);
        s[2 * i + 1] = spread4(w[i] >> 16);
    }
    return Lane6{make_uint4(s[0] | (s[1] << 24), (s[1] >> 8) | (s[2] << 16), (s[2] >> 16) | (s[3] << 8), s[4] | (s[5] << 24)),
                 make_uint2((s[5] >> 8) | (s[6] << 16), (s[6] >> 16) | (s[7] << 8))};
}

} // namespace qllm_detail

// Launches the planned kernel (fused_planned.hip).  Returns QLLM_ERR_WORKSPACE if the shape or the
// general groups are more than it holds on chip: the caller then takes the plain kernel.
int32_t qllm_launch_fused_planned(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits, hipStream_t stream);
// The same with the codes written to a.tiles (fused_planned_tiles.hip), where they fit (else the caller takes packed rows).
bool qllm_fused_tiles_fit(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits);
int32_t qllm_launch_fused_tiles(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits, hipStream_t stream);
// The shape of the planned kernel's launch, whether it begins with an empty output pass, and the bytes of a.ahead that it reads
int64_t qllm_fused_ahead(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits, int32_t *chunks_per_lane, int32_t *lanes, int32_t *empty_pass);
// QLLM_FUSED_*: the form of the fused kernel that qllm_launch_fused_planned would run for these arguments
int32_t qllm_choose_fused_planned(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits);

// Weights of the product that follows, in blocks of 16 features, `block` bytes each, made of K-tiles of `tile` bytes.  Workgroup
// c of it goes to XCD c % 8 and reads 8 blocks from 8 (c % cols) on, part c / cols of `splits` of their K-tiles.
struct WeightsAhead {
    const uint8_t *base;
    int64_t total;
    int32_t block, tile, cols, splits;
};

// qllm_norm_reassemble_quant in two halves, so that the layer call has checked all of its arguments before it launches anything.
// The checks, and the arguments of the kernel (N == 0: none, nothing is to be launched).
int32_t qllm_fused_prepare(const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx, int32_t norm, const float *gamma,
                           const float *beta, float eps, const qllm_map *map, int32_t bits, const qllm_qact *out,
                           qllm_detail::FusedArgs *args);
// The launch, with the choice of layout: tiles not null asks for the codes as the product reads them, TILES6 in the activations'
// order (4 bits; not what qllm_pack_tiles6 makes of weights) or TILES8, in place of out->codes (rows past N in the last
// block of 16 are left as they are: the product of such a row is dropped);
// *wrote_tiles says whether the kernel that runs does that (the planned one); if not, out->codes holds the packed rows as
// ever.  ahead: not null where the product's weights may be read into the caches on the side.
int32_t qllm_fused_run(const qllm_detail::FusedArgs &prepared, int32_t x_dtype, int32_t bits, uint8_t *tiles, bool *wrote_tiles,
                       const WeightsAhead *ahead, void *hip_stream);
// Whether qllm_fused_run lays the codes out where it is asked to.
bool qllm_fused_lays(const qllm_detail::FusedArgs &a, int32_t x_dtype, int32_t bits, const uint8_t *tiles);
// As much of the arguments as the choice of a launch depends on, and that choice.
int32_t qllm_fused_describe(const qllm_map *map, int32_t x_dtype, int64_t N, int64_t ldx, int32_t norm, int32_t has_beta, int32_t bits,
                            qllm_detail::FusedArgs *args);
int32_t qllm_fused_launch_facts(const qllm_detail::FusedArgs &described, int32_t x_dtype, int32_t bits, uint8_t *tiles,
                                const WeightsAhead *ahead, qllm_layer_launch *out);

#endif
