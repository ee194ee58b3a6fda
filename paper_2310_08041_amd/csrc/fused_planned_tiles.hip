// The planned fused kernels that write the codes as the GEMM reads them (4-bit codes as TILES6 in the activations' order, 6- and
// 8-bit ones as TILES8) instead of packed rows: fused_planned.hip once more, so that the two sets of kernels compile side
// by side.
#define QLLM_FUSED_TILES 1
#include "fused_planned.hip"
