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

// The planned kernel begins with an output pass over whatever LDS holds where there are more rows per resident workgroup than
// this (0: always), and its row loop need not ask then whether a row is waiting to be put out.  In a launch of one row per
// workgroup that pass is a tenth of the kernel (fused kernel, us, with it : asked: 200 x 13824 6-bit 10.0 : 8.6, 100 x 5120 4-bit
// 7.4 : 6.8, 1 x 4096 4.96 : 4.56, 777 x 5000 fp32 8-bit 22.3 : 20.2, 4096 x 5120 29.8 : 28.8).  Over many rows the branches cost more
// where the registers are short: both kernels of every kind, 1254 launches of 300-4096 rows, geometric means of with : asked (packed
// rows; layer with the codes laid out for the product), at most one row per workgroup / more than four:
//   lists streamed                                            1.00, no difference
//   four chunks per lane that fit exactly, no LayerNorm:
//     bf16 RMS 4-bit 1.00 / 1.05 (1.00 / 1.01), 6-bit 0.98 / 1.11 (0.99 / 1.04), 8-bit 1.00 / 1.15 (1.01 / 1.08)
//     bf16 without a norm 6-bit 1.02 / 1.12 (0.98 / 1.05), 8-bit 0.96 / 1.18 (0.95 / 1.03); fp32 RMS 6-bit 1.00 / 1.05 (0.99 / 1.03)
//     the others of this shape                                0.90-0.98 / 0.97-1.00
//   four with bounds, 6-bit, laid out                         (0.86-0.95 / 1.02-1.11; packed rows 0.88-0.91 / 0.93-0.98)
//     8-bit without a norm                                    (0.92-0.96, 1.01-1.04 from two rows; packed 0.80-0.87 / 0.87-0.94)
//   LayerNorm, three chunks, fp32 4-bit                       0.99-1.05 / 1.08-1.10 (1.00-1.01 from two rows)
//     bf16 4-bit 0.96 / 1.03-1.05 (exact fit 0.96 / 1.02, with bounds 0.96 at every size), fp32 6-bit 0.87 / 1.01 (0.95 / 1.03),
//     8-bit exact fit 0.93 / 1.04 (0.97 / 1.05), 1.02 (1.01) from two rows
//   LayerNorm, four that fit exactly, fp32 4-bit, packed      0.90 / 1.08, 1.03 from two rows
//   RMS, two chunks, 4-bit, packed: 0.94-0.96 / 1.01-1.07, where asking takes a register more than five workgroups per CU
//     leave (bf16 2048 x 4096 11.2 : 11.7, 4096 x 2560 14.8 : 15.7; at most one row 0.95)
//   five chunks of two words                                  0.89-0.98 / 0.95-1.05 (0.95-1.01 / 1.00-1.05)
//   all others                                                0.80-0.97 / 0.87-0.99 (the worst single launches, packed fp32 4-bit of 256
//     lanes at exactly two rows: 2048 x 8192 RMS 19.4 : 20.4, 2048 x 7168 without a norm 16.4 : 18.0)
constexpr int EMPTY_PASS_NEVER = 1 << 20;
enum { EMPTY_PASS_NO_NORM, EMPTY_PASS_LAYER, EMPTY_PASS_RMS };
constexpr int empty_pass_rows(bool tiles, bool f32, int norm, int bits, int iters, bool exact_fit, bool streams)
{
    const bool layer = norm == EMPTY_PASS_LAYER, two_words = bits != 4;
    if (streams || (iters == 5 && two_words)) return 0;
    if (layer && iters == 3 && f32 && !two_words) return 0;
    if (layer && iters == 3 && (f32 ? exact_fit || (tiles && bits == 6) : !two_words && (exact_fit || !tiles))) return bits == 8 ? 2 : 4;
    if (layer && iters == 4 && f32 && !two_words && exact_fit && !tiles) return 2;
    if (!layer && iters == 4 && exact_fit && (f32 ? norm == EMPTY_PASS_RMS && bits == 6 : norm == EMPTY_PASS_RMS || two_words)) return 0;
    if (!layer && iters == 4 && !exact_fit && tiles && two_words && (bits == 6 || norm == EMPTY_PASS_NO_NORM)) return bits == 8 ? 2 : 4;
    if (norm == EMPTY_PASS_RMS && iters == 2 && !two_words && !tiles && !(f32 && exact_fit)) return exact_fit ? 1 : 2;
    return EMPTY_PASS_NEVER;
}
// Most of these kernels take 97 to 128 registers: 16 wavefronts per CU.
inline bool begins_with_empty_pass(int rows, int64_t N, int lanes, int cus) { return N > rows * (int64_t)cus * (lanes < 1024 ? 1024 / lanes : 1); }

// How many bytes of its weights the idle CUs of the fused launch read ahead for every workgroup of the product: its first blocks,
// whole (the first K-tiles of all of them leave the memory idle first and the matrix cores after that).  24 MB of the L2s' 32,
// and no more than four times what the reading wavefronts have in flight at once (4 KB each), twice where the row has no norm:
// they have the lanes of a row's workgroup, and a short row is done in the time of some four trips to memory; what is still
// being read then holds the product up.  Layer, us, no reading : 24 MB whatever the row and the split of K : now, three sets of
// weights in turn (in the cache behind the L2s; out of it, with 5 for the measurement itself):
//   512 -> 27648, 128 tokens 8 / 8       12.5 : 21.0 : 12.2    18.2 : 31.0 : 18.1     (64 lanes)
//   1024 -> 27648, 128 tokens 6 / 6      15.3 : 22.8 : 14.8    23.3 : 33.9 : 22.2
//   5120 -> 27648, 100 tokens 4 / 4      36.6 : 34.9 : 34.9    54.9 : 51.6 : 51.8
//   5120 -> 11008, 100 tokens 6 / 6      25.1 : 25.0 : 24.6    42.0 : 40.7 : 41.2     (K in two parts, 86 columns of tiles)
//   13824 -> 8192, 40 tokens 8 / 4       38.5 : 39.0 : 37.4    62.7 : 58.4 : 57.3     (three parts, 64 columns)
//   10752 -> 3968, 53 tokens 8 / 8       22.8 : 24.2 : 21.3    37.5 : 33.3 : 33.8     (eight parts, 31 columns)
//   23040 -> 1664, 68 tokens 8 / 8       27.9 : 30.0 : 27.6    42.5 : 44.2 : 42.9
// Geometric mean over 96 shapes that read (33-128 tokens, 512-28672 channels, 256-27648 features): 1.010 and 1.041 of no reading, 24 MB
// 0.970 and 1.021; the worst, lists streamed, 23168 -> 2304, 60 tokens 38.6 : 40.9 : 40.1.  Streamed lists come through
// the same L2s; where these still hold the weights from the last call their rows wait for nothing gained: 5 % merged, weights of
// 6-12 MB 0.977 of no reading (41 x 16128 -> 640 8 / 8 32.2 : 34.8), but 1.045 out of cache, where a model's weights are.  With fewer idle CUs than rows the reading
// takes longer than the rows (160 x 5120 -> 13824 25.4 : 25.9, 200 x 4096 -> 12288 19.2 : 22.5): there is none.
constexpr int64_t READ_AHEAD_BYTES = 24000000, READ_AHEAD_TRIPS = 4, READ_AHEAD_IN_FLIGHT = 4096;
inline int64_t read_ahead_each(int64_t block, int64_t tile, int64_t cols, int64_t splits, int64_t waves, bool norm)
{
    const int64_t trips = (norm ? READ_AHEAD_TRIPS : READ_AHEAD_TRIPS / 2) * READ_AHEAD_IN_FLIGHT * waves, part = block / tile / splits * tile; // of a block, per part of K
    const int64_t each = (trips < READ_AHEAD_BYTES ? trips : READ_AHEAD_BYTES) / (cols * splits), most = 8 * (part / 1024) * 1024;
    return each < most ? each / 1024 * 1024 : most;
}

} // namespace qllm_detail

#endif
