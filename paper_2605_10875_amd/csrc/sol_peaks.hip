// Microbenchmarks that measure what this GPU actually reaches on the two rooflines the path is priced against:
// register-only bf16 MFMA loops (no memory traffic at all) and a plain device-to-device copy. The benchmark prints
// them beside the published peaks; nothing on the product path calls them.
#include "../../include/sol.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Every wave issues `iters` rounds of eight independent 32x32x16 bf16 MFMAs on registers (eight accumulators, so a
// result is never waited for); the sums are stored once at the end so the loop cannot be dropped.
__global__ __launch_bounds__(256) void k_peak_mfma(float *out, int iters)
{
    const uint32_t lane = threadIdx.x;
    const u32x4_t au = {0x3f803f80u + lane, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};      // bf16 ones (and a lane mark)
    const u32x4_t bu = {0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u};
    const bf16x8_t a = __builtin_bit_cast(bf16x8_t, au), b = __builtin_bit_cast(bf16x8_t, bu);
    f32x16_t acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[j], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[j][r];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// 16 fragments of 8 bf16 for every lane of a wave: normally distributed values (Box and Muller's transform of a hashed index), or ones
__global__ __launch_bounds__(256) void k_peak_operands(uint32_t *__restrict__ out, bool normal)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;       // two bf16
    auto hash = [](uint32_t x) { x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; return x ^ (x >> 16); };
    const float u = ((float)(hash(2 * i) >> 8) + 0.5f) * 0x1p-24f, v = (float)(hash(2 * i + 1) >> 8) * 0x1p-24f;
    const float r = sqrtf(-2.0f * logf(u));
    const __bf16 a = (__bf16)(normal ? r * cosf(6.2831853f * v) : 1.0f), b = (__bf16)(normal ? r * sinf(6.2831853f * v) : 1.0f);
    out[i] = (uint32_t)__builtin_bit_cast(uint16_t, a) | (uint32_t)__builtin_bit_cast(uint16_t, b) << 16;
}
// What the matrix cores reach depends on the instruction and on the data, through the power that both take: the products of a
// 128 x 128 wave tile from operands that are loaded once (256 accumulator registers, one wave per SIMD, as in the large GEMM).
__global__ __launch_bounds__(256, 1) void k_peak_data32(const bf16x8_t *__restrict__ in, float *__restrict__ out, int iters)
{
    const int lane = threadIdx.x & 63;
    bf16x8_t a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { a[i] = in[i * 64 + lane]; b[i] = in[(8 + i) * 64 + lane]; }
    f32x16_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int t = 0; t < iters; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) s += acc[i][j][r];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}
__global__ __launch_bounds__(256, 1) void k_peak_data16(const bf16x8_t *__restrict__ in, float *__restrict__ out, int iters)
{
    const int lane = threadIdx.x & 63;
    bf16x8_t a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { a[i] = in[i * 64 + lane]; b[i] = in[(8 + i) * 64 + lane]; }
    f32x4_t acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < iters; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) s += acc[i][j][r];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// dst[i] = src[i], 16 bytes per lane and step, grid-stride
__global__ __launch_bounds__(256) void k_peak_copy(const u32x4_t *__restrict__ src, u32x4_t *__restrict__ dst, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        dst[i] = __builtin_nontemporal_load(src + i);
}

// read-only: four independent 16-byte loads per lane and step, folded into one word that is stored at the end
__global__ __launch_bounds__(256) void k_peak_read(const u32x4_t *__restrict__ src, uint32_t *__restrict__ out, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t n4 = n16 / (4 * stride) * (4 * stride);
    u32x4_t acc = {0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += 4 * stride) {
        const u32x4_t a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + stride);
        const u32x4_t c = __builtin_nontemporal_load(src + i + 2 * stride), d = __builtin_nontemporal_load(src + i + 3 * stride);
        acc ^= a ^ b ^ c ^ d;
    }
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = acc.x ^ acc.y ^ acc.z ^ acc.w;
}

}  // namespace

extern "C" int sol_measure_peaks(void *scratch, size_t scratch_bytes, int reps, float *mfma_tflops_out, float *copy_gbs_out,
                                 float *read_gbs_out, void *stream)
{
    if (!scratch || !mfma_tflops_out || !copy_gbs_out || !read_gbs_out || reps <= 0) return SOL_ERR_INVALID_ARG;
    if (scratch_bytes < ((size_t)64 << 20)) return SOL_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return SOL_ERR_HIP;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return SOL_ERR_HIP;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return SOL_ERR_HIP; }
    int rc = SOL_OK;
    float ms = 0.f;
    // MFMA: two workgroups of four waves per CU (two waves per SIMD), 4096 rounds of 8 MFMAs of 32 * 32 * 16 * 2 flops
    const int blocks = 2 * cus, iters = 4096;
    hipLaunchKernelGGL(k_peak_mfma, dim3(blocks), dim3(256), 0, st, (float *)scratch, 64);      // warm-up
    (void)hipEventRecord(e0, st);
    for (int r = 0; r < reps; ++r) hipLaunchKernelGGL(k_peak_mfma, dim3(blocks), dim3(256), 0, st, (float *)scratch, iters);
    (void)hipEventRecord(e1, st);
    if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = SOL_ERR_HIP;
    const double flops = (double)reps * blocks * 4.0 * iters * 8.0 * (32.0 * 32.0 * 16.0 * 2.0);
    *mfma_tflops_out = rc ? 0.f : (float)(flops / (ms * 1e-3) / 1e12);
    // copy: half of the scratch into the other half (read + written bytes counted)
    const size_t half = (scratch_bytes / 2) & ~(size_t)255, n16 = half / 16;
    const u32x4_t *src = (const u32x4_t *)scratch;
    u32x4_t *dst = (u32x4_t *)((char *)scratch + half);
    const int cblocks = cus * 16;
    hipLaunchKernelGGL(k_peak_copy, dim3(cblocks), dim3(256), 0, st, src, dst, n16);            // warm-up
    (void)hipEventRecord(e0, st);
    for (int r = 0; r < reps; ++r) hipLaunchKernelGGL(k_peak_copy, dim3(cblocks), dim3(256), 0, st, src, dst, n16);
    (void)hipEventRecord(e1, st);
    if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = SOL_ERR_HIP;
    *copy_gbs_out = rc ? 0.f : (float)(2.0 * half * reps / (ms * 1e-3) / 1e9);
    // read: the first half of the scratch, results into the start of the second half
    const int rblocks = cus * 8;
    const size_t rstride = (size_t)rblocks * 256, rbytes = n16 / (4 * rstride) * (4 * rstride) * 16;
    hipLaunchKernelGGL(k_peak_read, dim3(rblocks), dim3(256), 0, st, src, (uint32_t *)dst, n16);   // warm-up
    (void)hipEventRecord(e0, st);
    for (int r = 0; r < reps; ++r) hipLaunchKernelGGL(k_peak_read, dim3(rblocks), dim3(256), 0, st, src, (uint32_t *)dst, n16);
    (void)hipEventRecord(e1, st);
    if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = SOL_ERR_HIP;
    *read_gbs_out = rc ? 0.f : (float)((double)rbytes * reps / (ms * 1e-3) / 1e9);
    if (hipGetLastError() != hipSuccess) rc = SOL_ERR_HIP;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

extern "C" int sol_measure_mfma(void *scratch, size_t scratch_bytes, int reps, float *tflops_out, void *stream)
{
    if (!scratch || !tflops_out || reps <= 0) return SOL_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return SOL_ERR_HIP;
    constexpr size_t OPERANDS = 16 * 64 * 16;                // bytes
    if (scratch_bytes < OPERANDS + (size_t)cus * 256 * sizeof(float)) return SOL_ERR_WORKSPACE;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return SOL_ERR_HIP;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return SOL_ERR_HIP; }
    const bf16x8_t *in = (const bf16x8_t *)scratch;
    float *out = (float *)((char *)scratch + OPERANDS);
    int rc = SOL_OK;
    for (int v = 0; v < 4 && rc == SOL_OK; ++v) {            // 32x32x16 on ones, on normal data; 16x16x32 likewise
        const bool wide = v < 2;
        const int iters = wide ? 8192 : 4096;                // 1.8 to 2.5 ms per launch
        auto *const kern = wide ? k_peak_data32 : k_peak_data16;
        hipLaunchKernelGGL(k_peak_operands, dim3((unsigned)(OPERANDS / 4 / 256)), dim3(256), 0, st, (uint32_t *)scratch, (v & 1) != 0);
        hipLaunchKernelGGL(kern, dim3(cus), dim3(256), 0, st, in, out, iters);                   // warm-up
        (void)hipEventRecord(e0, st);
        for (int r = 0; r < reps; ++r) hipLaunchKernelGGL(kern, dim3(cus), dim3(256), 0, st, in, out, iters);
        (void)hipEventRecord(e1, st);
        float ms = 0.f;
        if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = SOL_ERR_HIP;
        const double flops = (double)reps * cus * 4.0 * iters * (wide ? 16.0 * 32 * 32 * 16 * 2 : 64.0 * 16 * 16 * 32 * 2);
        tflops_out[v] = rc ? 0.f : (float)(flops / (ms * 1e-3) / 1e12);
    }
    if (hipGetLastError() != hipSuccess) rc = SOL_ERR_HIP;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}
