// GEMMs  C[M][N] = A[M][K] * W[N][K]^T  (both operands K-contiguous).
//   launch_gemm_f32rows : fp32 operands on the fp32 matrix instructions, up to three stacked weight matrices.
//   launch_gemm_generic : any shape / dtype, fp32 FMA on LDS tiles, fp32 output: what the MFMA kernels do not cover.
#include "sol_internal.h"

namespace sol {

constexpr int GT = 64;    // tile M = tile N
constexpr int GK = 16;    // tile K

template <typename TA, typename TW>
__global__ void __launch_bounds__(256)
k_gemm_generic(const TA *__restrict__ A, int64_t lda, const TW *__restrict__ W, int64_t ldw, float *__restrict__ C,
               int64_t ldc, int64_t M, int N, int K)
{
    __shared__ float As[GK][GT + 4];
    __shared__ float Ws[GK][GT + 4];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;          // 16 x 16 threads, 4 x 4 outputs each
    const int64_t m0 = (int64_t)blockIdx.y * GT;
    const int n0 = blockIdx.x * GT;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += GK) {
        // each thread loads 4 elements of A and of W: element (row = tid/4 + 0.., k = (tid%4)*4 ..)
        {
            const int rr = tid >> 2, kk = (tid & 3) * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + kk + e;
                const int64_t ar = m0 + rr;
                const int wr = n0 + rr;
                As[kk + e][rr] = (ar < M && k < K) ? ld(A + ar * lda + k) : 0.f;
                Ws[kk + e][rr] = (wr < N && k < K) ? ld(W + (int64_t)wr * ldw + k) : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < GK; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = Ws[k][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t r = m0 + ty * 4 + i;
        if (r >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = n0 + tx * 4 + j;
            if (c < N) C[r * ldc + c] = acc[i][j];
        }
    }
}

// ------------------------------------------------------------------------------------------------
// fp32 operands on v_mfma_f32_32x32x2_f32. The instruction is an fmaf chain over its two k in ascending order
// (subnormals included), so with k walked in order every output is the fmaf chain of k_gemm_generic, bit for bit, at
// twice the vector pipes' rate and without their LDS reads per product. Bound: the fp32 matrix rate (256 flops per
// clock and CU): a slice of 32 k takes a 64 x 64 wave tile 4096 clocks against 48 KB of loads and LDS reads, so plain
// double buffering hides everything else. 1018 rows x 3072 / 2048 / 16384 / 2048 columns of the 1B layer:
// 4.53 ms with fmaf -> see the dispatch below.
// ------------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef float f32x4v_t __attribute__((ext_vector_type(4)));

struct FMap {                        // output column -> weight row of up to three stacked matrices [n][ldw]
    const float *base[3];
    int end[3];
    int64_t ldw;
    __device__ __forceinline__ const float *row(int v) const
    {
        if (v < end[0]) return base[0] + (int64_t)v * ldw;
        if (v < end[1]) return base[1] + (int64_t)(v - end[0]) * ldw;
        return base[2] + (int64_t)(v - end[1]) * ldw;
    }
};

// 16 bytes per lane straight into LDS: lane l's piece lands at lds_addr + 16 * l (wave-uniform)
__device__ __forceinline__ void lds_load16(const float *src, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}

template <int BM, int BN, int WM, int WN>
__global__ void __launch_bounds__(256, 2)
k_gemm_f32mfma(const float *__restrict__ A, int64_t lda, FMap map, float *__restrict__ C, int64_t ldc, int64_t M, int N, int K,
               int tiles_m, int tiles_n)
{
    static_assert((BM / WM) * (BN / WN) == 4, "four waves");
    constexpr int NWN = BN / WN, TM = WM / 32, TN = WN / 32, AP = BM / 32, BP = BN / 32, ST = 3;
    constexpr uint32_t SB = (BM + BN) * 128;                 // a stage: rows of 32 floats, 16-byte chunks XOR-swizzled
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / NWN, wn = wave - wm * NWN;
    // workgroup b runs on XCD b % 8; an XCD owns a contiguous band of the tiles, column by column
    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= n_tiles) return;
    const int64_t m0 = (int64_t)(lin % tiles_m) * BM;
    const int n0 = (lin / tiles_m) * BN;

    const int chunk = tid & 7, rip = tid >> 3;               // 8 lanes x 16 bytes per row, 32 rows per pass
    const int sw = (chunk ^ ((rip >> 1) & 7)) * 4;
    const float *ap[AP], *bp[BP];                            // rows past the end: the last row again, never stored
#pragma unroll
    for (int p = 0; p < AP; ++p) {
        const int64_t r = m0 + p * 32 + rip;
        ap[p] = A + (r < M ? r : M - 1) * lda + sw;
    }
#pragma unroll
    for (int p = 0; p < BP; ++p) {
        const int v = n0 + p * 32 + rip;
        bp[p] = map.row(v < N ? v : N - 1) + sw;
    }
    const int KT = K / 32;
    auto request = [&](int kt, uint32_t stage) {
        const int koff = (kt < KT ? kt : KT - 1) * 32;
#pragma unroll
        for (int p = 0; p < AP; ++p) lds_load16(ap[p] + koff, stage + (uint32_t)(p * 4096 + wave * 1024));
#pragma unroll
        for (int p = 0; p < BP; ++p) lds_load16(bp[p] + koff, stage + (uint32_t)((AP + p) * 4096 + wave * 1024));
    };
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int frow = lane & 31, fsw = (frow >> 1) & 7;
    const bool hi = lane >= 32;                              // lanes 0..31 supply the even k of a pair, 32..63 the odd one
    const int a_frag = (wm * WM + frow) * 128, b_frag = (BM + wn * WN + frow) * 128;

    request(0, 0);
    request(1, SB);
    uint32_t cur = 0, fre = 2 * SB;
    for (int kt = 0; kt < KT; ++kt) {
        // slice kt has landed (the youngest slice may be in flight), the stage of slice kt - 1 is read out; for all waves
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(AP + BP) : "memory");
        request(kt + 2, fre);
        const unsigned char *const st = lds + cur;
#pragma unroll
        for (int c = 0; c < 8; ++c) {                        // four k
            const int coff = (c ^ fsw) << 4;
            f32x4v_t a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const f32x4v_t *>(st + a_frag + i * 4096 + coff);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const f32x4v_t *>(st + b_frag + j * 4096 + coff);
#pragma unroll
            for (int e = 0; e < 4; e += 2)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(hi ? a[i][e + 1] : a[i][e], hi ? b[j][e + 1] : b[j][e], acc[i][j], 0, 0, 0);
        }
        fre = cur;
        cur = cur + SB == ST * SB ? 0 : cur + SB;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // no LDS-direct load outlives its workgroup
    const int col0 = n0 + wn * WN + frow;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t row = m0 + wm * WM + i * 32 + 8 * (r >> 2) + (r & 3) + (hi ? 4 : 0);
            if (row >= M) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (col0 + 32 * j < N) C[row * ldc + col0 + 32 * j] = acc[i][j][r];
        }
}

template <int BM, int BN, int WM, int WN>
static bool launch_f32mfma(const float *A, int64_t lda, const FMap &map, float *C, int64_t ldc, int64_t M, int N, int K, hipStream_t st)
{
    constexpr size_t lds = 3 * (size_t)(BM + BN) * 128;
    auto kern = k_gemm_f32mfma<BM, BN, WM, WN>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return false;
        attr_done = true;
    }
    const int tm = (int)((M + BM - 1) / BM), tn = (N + BN - 1) / BN, per_xcd = (tm * tn + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256), lds, st, A, lda, map, C, ldc, M, N, K, tm, tn);
    return true;
}

// The matrix rate bounds every tile, so the tile is the one whose rounds over the CUs compute the least: a 64 x 64 tile
// reads twice the operands per product of a 128 x 128 tile and is charged a tenth more.
bool launch_gemm_f32rows(const float *A, int64_t lda, const float *w0, int n0, const float *w1, int n1, const float *w2, int n2,
                         int64_t ldw, float *C, int64_t ldc, int64_t M, int K, hipStream_t st)
{
    const int64_t N = (int64_t)n0 + n1 + n2;
    auto aligned = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    if (K < 32 || K % 32 || lda % 4 || ldw % 4 || !aligned(A) || !aligned(w0) || !aligned(w1) || !aligned(w2) ||
        M > (1ll << 30) || N > (1ll << 30))
        return false;                                        // 16-byte loads of whole slices
    if (M <= 0 || N <= 0) return true;
    FMap map{{w0, w1, w2}, {n0, n0 + n1, n0 + n1 + n2}, ldw};
    const int cus = device_cus() > 0 ? device_cus() : 256;
    auto cost = [&](int bm, int bn, double per) {
        const int64_t tiles = (M + bm - 1) / bm * ((N + bn - 1) / bn);
        return (double)((tiles + cus - 1) / cus) * bm * bn * per;
    };
    const double c0 = cost(128, 128, 1.0), c1 = cost(64, 128, 1.05), c2 = cost(64, 64, 1.1);
    if ((M + 63) / 64 * ((N + 63) / 64) > (1ll << 30)) return false;
    if (c0 <= c1 && c0 <= c2) return launch_f32mfma<128, 128, 64, 64>(A, lda, map, C, ldc, M, (int)N, K, st);
    if (c1 <= c2) return launch_f32mfma<64, 128, 32, 64>(A, lda, map, C, ldc, M, (int)N, K, st);
    return launch_f32mfma<64, 64, 32, 32>(A, lda, map, C, ldc, M, (int)N, K, st);
}

void launch_gemm_generic(const void *A, int a_dtype, int64_t lda, const void *W, int w_dtype, int64_t ldw, float *C,
                         int64_t ldc, int64_t M, int N, int K, hipStream_t st)
{
    if (M <= 0 || N <= 0) return;
    if (a_dtype == 0 && w_dtype == 0 &&
        launch_gemm_f32rows((const float *)A, lda, (const float *)W, N, nullptr, 0, nullptr, 0, ldw, C, ldc, M, K, st))
        return;
    const dim3 grid((unsigned)((N + GT - 1) / GT), (unsigned)((M + GT - 1) / GT));
    if (a_dtype == 0 && w_dtype == 0)
        hipLaunchKernelGGL((k_gemm_generic<float, float>), grid, dim3(256), 0, st, (const float *)A, lda,
                           (const float *)W, ldw, C, ldc, M, N, K);
    else if (a_dtype == 1 && w_dtype == 1)
        hipLaunchKernelGGL((k_gemm_generic<bf16_t, bf16_t>), grid, dim3(256), 0, st, (const bf16_t *)A, lda,
                           (const bf16_t *)W, ldw, C, ldc, M, N, K);
}

}  // namespace sol
