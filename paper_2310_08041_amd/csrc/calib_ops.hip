// Two small device operations of the offline search for theta (Algorithm 1): the full-precision output
// of the layer that the quantized layer is scored against, and the squared error between the two.
// Neither is on the hot path; both are deterministic fp64 kernels.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "qllm.h"

extern "C" void qllm_note_hip_error(const char *step, const char *name);

namespace {

constexpr int THREADS = 256, TK = 32;
typedef double v4d __attribute__((ext_vector_type(4)));

// out[n, o] = sum_c y[n, c] * W[c, o], every product and sum in double (fp32 inputs widened exactly), in steps of four c
// in ascending order, on the fp64 matrix cores.  A workgroup (2 x 2 waves) owns MI * 32 tokens x NJ * 32 features, a wave
// MI x NJ tiles of 16 x 16.  K-steps of 32 pass through LDS as fp32 (the next one's loads are in flight in registers
// while this one is multiplied) and are widened when they are read: per four c a wave reads MI + NJ values for MI * NJ
// operations of 64 clocks each, so that the matrix cores are what bounds it.  Rows of the y tile are 36 floats apart and
// those of the W tile 16 past a multiple of 32: the 64 lanes of an operand read (16 rows x 4 c) fall on 64 banks.
// 1024 x 4096 x 4096: 1715 us with one multiply-add per lane and clock from fp64 tiles, now 590 (58 TFLOP/s; a large
// library product reaches 68 on the same card).
template <int MI, int NJ>
__global__ __launch_bounds__(THREADS) void linear_f64_kernel(const float *y, int64_t N, int64_t C, int64_t ldy, const float *W,
                                                             int64_t O, int64_t ldw, double *out, int64_t ldo, int32_t vec_ok)
{
    constexpr int TM = 32 * MI, TN = 32 * NJ, YS = TK + 4, WS = TN + 16, YL = TM * TK / 4 / THREADS, WL = TN * TK / 4 / THREADS;
    static_assert(WS % 32 == 16, "four rows of W apart, 16 banks apart");
    __shared__ __attribute__((aligned(16))) float ys[TM * YS], ws[TK * WS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, q = lane >> 4;
    const int wm = (wave >> 1) * 16 * MI, wn = (wave & 1) * 16 * NJ;
    const int64_t n0 = (int64_t)blockIdx.y * TM, o0 = (int64_t)blockIdx.x * TN;
    float4 yr[YL], wr[WL];
    // four neighbouring values of a row, zero past its end or past the last row
    auto four = [&](const float *base, int64_t ld, int64_t row, int64_t rows, int64_t col, int64_t cols) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row >= rows || col >= cols) return v;
        const float *p = base + row * ld + col;
        if (vec_ok && col + 4 <= cols) return *reinterpret_cast<const float4 *>(p);
        v.x = p[0];
        if (col + 1 < cols) v.y = p[1];
        if (col + 2 < cols) v.z = p[2];
        if (col + 3 < cols) v.w = p[3];
        return v;
    };
    auto fetch = [&](int64_t c0) {
#pragma unroll
        for (int t = 0; t < YL; ++t) {
            const int e = tid + t * THREADS;
            yr[t] = four(y, ldy, n0 + e / (TK / 4), N, c0 + 4 * (e % (TK / 4)), C);
        }
#pragma unroll
        for (int t = 0; t < WL; ++t) {
            const int e = tid + t * THREADS;
            wr[t] = four(W, ldw, c0 + e / (TN / 4), C, o0 + 4 * (e % (TN / 4)), O);
        }
    };
    v4d acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    fetch(0);
    for (int64_t c0 = 0; c0 < C; c0 += TK) {
        __syncthreads(); // the previous step has been read
#pragma unroll
        for (int t = 0; t < YL; ++t) {
            const int e = tid + t * THREADS;
            *reinterpret_cast<float4 *>(ys + e / (TK / 4) * YS + 4 * (e % (TK / 4))) = yr[t];
        }
#pragma unroll
        for (int t = 0; t < WL; ++t) {
            const int e = tid + t * THREADS;
            *reinterpret_cast<float4 *>(ws + e / (TN / 4) * WS + 4 * (e % (TN / 4))) = wr[t];
        }
        __syncthreads();
        if (c0 + TK < C) fetch(c0 + TK);
#pragma unroll
        for (int k = 0; k < TK; k += 4) {
            double a[MI], b[NJ];
#pragma unroll
            for (int i = 0; i < MI; ++i) a[i] = (double)ys[(wm + 16 * i + r) * YS + k + q];
#pragma unroll
            for (int j = 0; j < NJ; ++j) b[j] = (double)ws[(k + q) * WS + wn + 16 * j + r];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    // element e of an accumulator: token (lane >> 4) + 4 e, feature lane & 15
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t n = n0 + wm + 16 * i + q + 4 * e, o = o0 + wn + 16 * j + r;
                if (n < N && o < O) out[n * ldo + o] = acc[i][j][e];
            }
}

__device__ __forceinline__ double widen_out(const void *p, int32_t dtype, int64_t at)
{
    if (dtype == QLLM_BF16) return (double)__uint_as_float((uint32_t)static_cast<const uint16_t *>(p)[at] << 16);
    return (double)static_cast<const float *>(p)[at];
}

// One partial sum per row: sum_o (got[n, o] - ref[n, o])^2 in double, o ascending within a lane, lanes and waves
// combined in a fixed order.
__global__ __launch_bounds__(THREADS) void sq_error_rows_kernel(const void *got, int32_t dtype, int64_t O, int64_t ldg,
                                                                const double *ref, int64_t ldr, double *partial)
{
    __shared__ double red[THREADS / 64];
    const int64_t n = blockIdx.x;
    double s = 0.0;
    for (int64_t o = threadIdx.x; o < O; o += THREADS) {
        const double d = widen_out(got, dtype, n * ldg + o) - ref[n * ldr + o];
        s = __builtin_fma(d, d, s);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[n] = (red[0] + red[1]) + (red[2] + red[3]);
}

// The rows' partial sums added up by one workgroup, in a fixed order.
__global__ __launch_bounds__(THREADS) void sq_error_total_kernel(const double *partial, int64_t N, double *result)
{
    __shared__ double red[THREADS];
    double s = 0.0;
    for (int64_t n = threadIdx.x; n < N; n += THREADS) s += partial[n];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = THREADS / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *result = red[0];
}

int32_t launched(const char *what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        qllm_note_hip_error(what, hipGetErrorName(e));
        return QLLM_ERR_HIP;
    }
    return QLLM_OK;
}

} // namespace

extern "C" int32_t qllm_linear_f64(const float *y, int64_t N, int64_t C, int64_t ldy, const float *W, int64_t O, int64_t ldw,
                                   double *out, int64_t ldo, void *hip_stream)
{
    if (!y || !W || !out) return QLLM_ERR_NULL;
    if (N < 0 || C <= 0 || O <= 0 || ldy < C || ldw < O || ldo < O) return QLLM_ERR_SHAPE;
    if ((N + 63) / 64 > 65535) return QLLM_ERR_SHAPE;
    if (N == 0) return QLLM_OK;
    const int32_t vec_ok = (ldy & 3) == 0 && (ldw & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0 &&
                           (reinterpret_cast<uintptr_t>(W) & 15u) == 0;
    // 128 x 64 tiles where they give every CU at least one, else 32 x 32 ones: eight times as many workgroups
    const int64_t big = ((N + 127) / 128) * ((O + 63) / 64);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    (void)hipGetLastError();
    if (big >= 256 || (N + 31) / 32 > 65535)
        hipLaunchKernelGGL((linear_f64_kernel<4, 2>), dim3((unsigned)((O + 63) / 64), (unsigned)((N + 127) / 128)), dim3(THREADS), 0,
                           stream, y, N, C, ldy, W, O, ldw, out, ldo, vec_ok);
    else
        hipLaunchKernelGGL((linear_f64_kernel<1, 1>), dim3((unsigned)((O + 31) / 32), (unsigned)((N + 31) / 32)), dim3(THREADS), 0,
                           stream, y, N, C, ldy, W, O, ldw, out, ldo, vec_ok);
    return launched("full-precision layer output: launch");
}

extern "C" int64_t qllm_sq_error_workspace_bytes(int64_t N)
{
    return N < 0 ? (int64_t)QLLM_ERR_SHAPE : N * (int64_t)sizeof(double);
}

extern "C" int32_t qllm_sq_error(const void *got, int32_t got_dtype, int64_t N, int64_t O, int64_t ldg, const double *ref,
                                 int64_t ldr, double *result, void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    if (!got || !ref || !result) return QLLM_ERR_NULL;
    if (got_dtype != QLLM_F32 && got_dtype != QLLM_BF16) return QLLM_ERR_DTYPE;
    if (N <= 0 || O <= 0 || ldg < O || ldr < O || N > INT32_MAX) return QLLM_ERR_SHAPE;
    if (!workspace || workspace_bytes < qllm_sq_error_workspace_bytes(N)) return QLLM_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 7u) return QLLM_ERR_ALIGN;
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    double *partial = static_cast<double *>(workspace);
    (void)hipGetLastError();
    hipLaunchKernelGGL(sq_error_rows_kernel, dim3((unsigned)N), dim3(THREADS), 0, stream, got, got_dtype, O, ldg, ref, ldr, partial);
    int32_t rc = launched("squared output error: rows");
    if (rc != QLLM_OK) return rc;
    hipLaunchKernelGGL(sq_error_total_kernel, dim3(1), dim3(THREADS), 0, stream, partial, N, result);
    return launched("squared output error: total");
}
