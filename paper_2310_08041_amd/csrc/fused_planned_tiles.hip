// The planned fused kernels that write the codes as the GEMM reads them (qllm_pack_tiles6 for 4-bit codes, qllm_pack_tiles8
// for 6- and 8-bit ones) instead of packed rows: fused_planned.hip once more, so that the two sets of kernels compile side
// by side.
#define QLLM_FUSED_TILES 1
#include "fused_planned.hip"
