// The planned fused kernels of 6- and 8-bit codes that write the byte layout of the GEMM (qllm_pack_tiles8) instead of
// packed rows: fused_planned.hip once more, so that the two sets of kernels compile side by side.
#define QLLM_FUSED_TILES8 1
#include "fused_planned.hip"
