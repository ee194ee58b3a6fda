// Launch shape and LDS need of the planned fused kernel: shared by the launcher (which form of the kernel fits) and the
// plan builder (whether to stage only the chunks that hold sources, or all of them).  Plain C++, no HIP.
#ifndef QLLM_PLAN_BUDGET_H
#define QLLM_PLAN_BUDGET_H

#include <cstdint>

namespace qllm_detail {

// dynamic LDS a launch may ask for: 160 KB per CU, less the kernel's static reduction slots
constexpr int64_t FUSED_MAX_LDS = 159 * 1024;

struct PlanCounts {
    int64_t n_comp, n_long, n_pub, n_chunks, n_spec, n_dest, n_segw;
};

// words_per_chunk: LDS dwords per packed chunk of 8 codes (1 for 4-bit, 2 for 6- and 8-bit codes);
// staging_sets: x alone, with gamma, with gamma and beta (1..3); slots: chunks per lane x lanes of the launch
// (one word per slot for its chunk, two for its output group).
inline int64_t fused_lists_lds_bytes(const PlanCounts &p, int64_t words_per_chunk, int64_t staging_sets, int64_t slots)
{
    const int64_t w = words_per_chunk, n_stage = 8 * p.n_pub + 4, n_dest4 = (p.n_dest + 3) / 4 * 4;
    return (staging_sets * n_stage + n_dest4) * 4 + p.n_long * 16 + p.n_comp * 32 + p.n_spec * 8 +
           (p.n_comp * w + w + (p.n_chunks + 1) * w) * 4 + (p.n_dest + p.n_segw + 3 * slots + 1) * 4; // + 1: the two-word slots start at an even word
}

// The same with the lists left in global memory and the whole row staged in the input's own type.  How many chunks the
// plan gives a staging number makes no difference to it, so that numbering few of them takes this form from no map.
inline int64_t fused_streamed_lds_bytes(const PlanCounts &p, int64_t words_per_chunk, int64_t C, int64_t elem_bytes, int64_t slots)
{
    const int64_t w = words_per_chunk, n_dest4 = (p.n_dest + 3) / 4 * 4;
    return ((C + 8) * elem_bytes + 15) / 16 * 16 + n_dest4 * 4 + (p.n_comp * w + w + (p.n_chunks + 1) * w) * 4 + (3 * slots + 1) * 4;
}

struct Shape {
    int iters, nt; // chunks per lane, lanes
};

// Chunks (or output groups) per lane and the workgroup size for rows of `units` of them.  A workgroup's
// waves go to the CU's four SIMDs in turn, so the SIMD with the most of them, ceil(waves / 4), sets the pace:
// the cost of a row is that count times (chunks per lane + the fixed work of a wave and row, about one
// chunk's worth).  With fewer rows than CUs every workgroup has one row and the fewest chunks per lane win.
// The irregular part of the plan (long-row entries, computed channels, composite groups) is dealt out over the
// lanes, and every further pass over one of its lists is a chain of dependent LDS reads that nothing overlaps:
// if some shape has enough lanes for the longest of the three lists (`irregular`), only such shapes are
// considered; if none has, the one with the most lanes.  (Measured at the 5120- and 4096-channel shapes over maps
// from 1 % to 25 % of the channels merged: the best of the shapes in nine cases of ten, and up to 1.8 times
// faster than the shape the regular part alone would pick.)
inline Shape pick_shape(int64_t units, bool more_rows_than_cus, bool layer_norm, int64_t irregular)
{
    Shape best{0, 0};
    int best_cost = 0;
    bool best_covers = false;
    for (int iters = 1; iters <= (layer_norm ? 4 : 5); ++iters) { // LayerNorm at five chunks per lane spills
        const int nt = (int)(((units + iters - 1) / iters + 63) / 64 * 64);
        if (nt > (iters == 5 ? 768 : 1024)) continue; // five chunks per lane need the registers of three waves per SIMD
        const int waves = nt / 64;
        const int cost = more_rows_than_cus ? (waves + 3) / 4 * (iters + 1) : iters;
        const bool covers = nt >= irregular;
        // a shape that covers beats one that does not; among equals the cheaper one; the first feasible shape has
        // the most lanes and stays if nothing covers
        const bool better = best.iters == 0 || (covers && !best_covers) || (covers == best_covers && covers && cost < best_cost);
        if (better) {
            best = {iters, nt};
            best_cost = cost;
            best_covers = covers;
        }
    }
    return best;
}

// Whether the planned kernel begins with an output pass over whatever LDS holds, so that its row loop need not ask whether a
// row is waiting to be put out.  In a launch of one row per workgroup that pass is a tenth of the kernel (fused kernel, us, with
// it : asked: 200 x 13824 6-bit 10.0 : 8.6, 100 x 5120 4-bit 7.4 : 6.8, 1 x 4096 4.96 : 4.56, 777 x 5000 fp32 8-bit 22.3 : 20.2,
// 4096 x 5120 29.8 : 28.8).  It stays where the branches cost the scheduler more, which goes by registers and not by the
// row's length:
//   lists streamed;
//   five chunks per lane of two words (2048 x 28672 6-bit 57.4 : 58.9; 4-bit 61.9 : 60.8);
//   4-bit codes of fp32 rows with LayerNorm at three chunks per lane (packed rows, 2048 tokens: 5120 channels 24.0 : 24.4, 9216
//   33.4 : 35.0, 11264 42.2 : 46.7, 17408 66.5 : 77.6) and at four that fit exactly with more than two rows per workgroup (see
//   below); not at four with bounds, whose registers spill either way (7168 51.5 : 46.7, 13312 85.4 : 81.5, 23552 159.8 : 152.7), nor where
//   the codes are laid out for the product (8192, layer 88.6 : 84.8).
constexpr bool fused_empty_pass(bool tiles, bool f32, bool layer_norm, int bits, int iters, bool exact_fit, bool streams)
{
    if (streams || (iters == 5 && bits != 4)) return true;
    return f32 && layer_norm && bits == 4 && (iters == 3 || (iters == 4 && exact_fit && !tiles));
}
// Up to two rows per resident workgroup (128 registers: 16 wavefronts per CU): packed rows of 512 lanes and four chunks, us, with
// it : asked, 400 tokens 26.2 : 25.4, 512 27.8 : 27.5, 1536 62.9 : 66.8; 448 lanes 400 22.5 : 19.3, 1024 37.7 : 36.8, 1536 49.6 : 50.6; 768
// lanes 512 36.6 : 35.1, 1024 62.0 : 63.5, 2048 108 : 117; 256 lanes 2048 39.9 : 38.8, 4096 65.3 : 68.2.
inline bool fused_few_rows(int64_t rows, int lanes, int cus) { return rows <= 2 * (int64_t)cus * (1024 / lanes); }

// How many bytes of every chunk of the product's weights the idle CUs of the fused launch read ahead (a chunk per workgroup of
// the product).  24 MB of the L2s' 32, and no more than four times what the reading wavefronts have in flight at once (4 KB each):
// they have the lanes of a row's workgroup, and a short row is done in the time of some four trips to memory; what is still
// being read then holds the product up.  Layer, us, no reading : 24 MB whatever the row : four trips (weights in the cache
// behind the L2s / not):
//   512 -> 27648, 128 tokens 8 / 8       13.1 : 21.3 : 12.7    14.0 : 26.5 : 13.7     (64 lanes)
//   1024 -> 27648, 128 tokens 6 / 6      15.8 : 22.5 : 15.4    16.9 : 28.3 : 16.5
//   5120 -> 11008, 100 tokens 6 / 6      26.1 : 26.1 : 25.6    32.9 : 30.6 : 29.9     (K in two parts, 86 columns of tiles)
//   4096 -> 20500, 100 tokens 4 / 4      22.1 : 21.3 : 21.2    27.8 : 27.2 : 27.0
//   13824 -> 8192, 40 tokens 8 / 4       32.8 : 34.2 : 34.0    (the worst of 351 shapes in cache; none loses more than 2 % out of it)
// Geometric mean over 351 shapes (33-128 tokens, 512-16384 channels, 4096-28672 features): 1.019 and 1.040 of no reading.  Where
// K is split and the columns of tiles are not a multiple of 8, most workgroups of the product find their weights on another
// XCD, and still gain: 1.016 and 1.045 over 32 of those shapes.  With fewer idle CUs than rows the reading takes longer than
// the rows (160 x 5120 -> 13824 25.4 : 25.9, 200 x 4096 -> 12288 19.2 : 22.5): there is none.
constexpr int64_t READ_AHEAD_BYTES = 24000000, READ_AHEAD_TRIPS = 4, READ_AHEAD_IN_FLIGHT = 4096;
inline int64_t read_ahead_each(int64_t total, int64_t chunk, int64_t waves)
{
    const int64_t chunks = (total + chunk - 1) / chunk, trips = READ_AHEAD_TRIPS * READ_AHEAD_IN_FLIGHT * waves;
    const int64_t each = (trips < READ_AHEAD_BYTES ? trips : READ_AHEAD_BYTES) / chunks;
    return (each < chunk ? each : chunk) / 1024 * 1024;
}

} // namespace qllm_detail

#endif
