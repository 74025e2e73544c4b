// GEMMs  C[M][N] = A[M][K] * W[N][K]^T  (both operands K-contiguous).
//   launch_gemm_f32*    : fp32 operands on the fp32 matrix instructions, also with what follows the product in a layer.
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
// fp32 operands on the fp32 matrix instructions. v_mfma_f32_16x16x4_f32 is an fmaf chain over its k in ascending order
// (subnormals included), so with k walked in order every output is the fmaf chain of k_gemm_generic, bit for bit,
// at twice the vector pipes' rate and without their LDS reads per product. Bound: the fp32 matrix rate (155 TFLOP/s measured, 124
// reached) for large products; the chain over k, 32 clocks per 4 k, for small ones. k_gemm_generic -> here, us: 1018 x 16384 x 2048
// 2470 -> 551 (with SiLU * up at its end), 1018 x 2048 x 8192 1310 -> 296 (with the residual), 512 x 256 x 256 30 -> 4.8, 512 x 256 x 1024
// 108 -> 12.
// ------------------------------------------------------------------------------------------------
typedef float f32x4v_t __attribute__((ext_vector_type(4)));

enum { FMAP_STACKED, FMAP_PAIRS, FMAP_ROPE };
struct FMap {                        // output column -> weight row of up to three matrices [n][ldw]
    const float *base[3];
    int end[3];
    int64_t ldw;
    int mode, dh;                    // stacked; pairs: column 2 c of base[0]'s row c, 2 c + 1 of base[1]'s; rope: stacked heads of dh
                                     // rows, columns 2 c and 2 c + 1 of a head its rows c and c + dh / 2
    __device__ __forceinline__ const float *row(int v) const
    {
        if (mode == FMAP_PAIRS) return base[v & 1] + (int64_t)(v >> 1) * ldw;
        const int seg = v < end[0] ? 0 : (v < end[1] ? 1 : 2);
        v -= seg == 0 ? 0 : end[seg - 1];
        if (mode == FMAP_ROPE) {
            const int head = v / dh, i = v - head * dh;
            v = head * dh + (i & 1) * (dh >> 1) + (i >> 1);
        }
        return base[seg] + (int64_t)v * ldw;
    }
};

// What becomes of a product. A lane of the accumulators holds one column of several rows; column(v) is what it needs to know
// of it, early(row, ..) reads what it needs of memory (ahead of the K loop where a tile is small), put(row, .., x, y) gets the
// product x and, if `pairs`, the neighbouring column's y (lane ^ 1: the columns 2 c and 2 c + 1 that FMAP_PAIRS and FMAP_ROPE
// put side by side). The values are those of the separate kernels (k_silu_mul, k_rope_store, k_resid_out), whose passes over
// the product these save. Measured: a one-layer model's call over 4 x 128 tokens, 95.0 -> 88.5 us (a launch of about 4 us each);
// a 1B layer over 2 x 509 tokens, 1311 -> 1303 us (the three kernels took 45 us; their work now ends the product's tiles, and
// the gate / up weights arrive from two matrices). (0 + x: their sum over one split.)
struct F32Store {
    static constexpr bool pairs = false;
    float *C; int64_t ldc;
    struct Col { float *p; };
    __device__ __forceinline__ Col column(int v) const { return Col{C + v}; }
    struct Early {};
    __device__ __forceinline__ Early early(int64_t, const Col &) const { return Early(); }
    __device__ __forceinline__ void put(int64_t row, const Col &c, const Early &, float x, float) const { c.p[row * ldc] = x; }
};
struct F32Resid {                    // out = x2 + product
    static constexpr bool pairs = false;
    const float *x2; float *out; int64_t ldc;
    struct Col { int v; };
    __device__ __forceinline__ Col column(int v) const { return Col{v}; }
    struct Early { float x2; };
    __device__ __forceinline__ Early early(int64_t row, const Col &c) const { return Early{x2[row * ldc + c.v]}; }
    __device__ __forceinline__ void put(int64_t row, const Col &c, const Early &e, float x, float) const
    {
        out[row * ldc + c.v] = e.x2 + (0.f + x);
    }
};
struct F32Silu {                     // a = silu(gate) * up; FMAP_PAIRS of gate and up
    static constexpr bool pairs = true;
    float *a; int64_t ldc;
    struct Col { int v; };
    __device__ __forceinline__ Col column(int v) const { return Col{v}; }
    struct Early {};
    __device__ __forceinline__ Early early(int64_t, const Col &) const { return Early(); }
    __device__ __forceinline__ void put(int64_t row, const Col &c, const Early &, float x, float y) const
    {
        if ((c.v & 1) == 0) a[row * ldc + (c.v >> 1)] = silu_mul(0.f + x, 0.f + y);
    }
};
struct F32Qkv {                      // rotary on q and k heads, q -> [M][nq], K / V -> caches; FMAP_ROPE of q, k and v
    static constexpr bool pairs = true;
    float *q, *kc, *vc;
    const float2 *rope; const int32_t *pos0;
    int Tn, L_max, crows, Hq, Hkv, dh;
    int *flags;
    struct Col { int slot, c; bool odd, first; };
    __device__ __forceinline__ Col column(int v) const
    {
        const int slot = v / dh, i = v - slot * dh;
        return Col{slot, i >> 1, (i & 1) != 0, v == 0};
    }
    struct Early { uint32_t s; int pos; float2 cs; };        // sequence; position, -1 where the sequence does not fit its cache
    __device__ __forceinline__ Early early(int64_t row, const Col &c) const
    {
        const uint32_t r = (uint32_t)row, s = r / (uint32_t)Tn;
        const int p0 = pos0 ? pos0[s] : 0;
        Early e{s, p0 < 0 || p0 + Tn > L_max ? -1 : p0 + (int)(r - s * (uint32_t)Tn), {1.f, 0.f}};
        if (e.pos >= 0 && c.slot < Hq + Hkv) e.cs = rope[(int64_t)e.pos * (dh >> 1) + c.c];
        return e;
    }
    __device__ __forceinline__ void put(int64_t row, const Col &c, const Early &e, float x, float y) const
    {
        if (e.pos < 0) {                                     // skipped
            if (c.first) atomicOr(flags, FLAG_CACHE_OVERFLOW);
            return;
        }
        const int pos = e.pos, half = dh >> 1;
        const int64_t s = e.s;
        x = 0.f + x, y = 0.f + y;
        if (c.slot < Hq + Hkv) {
            const float2 z = rotate_pair(c.odd ? y : x, c.odd ? x : y, e.cs);
            x = c.odd ? z.y : z.x;
        }
        float *const dst = c.slot < Hq ? q + row * (int64_t)(Hq * dh) + c.slot * dh
                         : (c.slot < Hq + Hkv ? kc + ((s * Hkv + (c.slot - Hq)) * crows + pos) * dh
                                              : vc + ((s * Hkv + (c.slot - Hq - Hkv)) * crows + pos) * dh);
        dst[c.c + (c.odd ? half : 0)] = x;
    }
};
template <class Epi>
__device__ __forceinline__ void f32_put(const Epi &epi, int64_t row, const typename Epi::Col &c, const typename Epi::Early &e, float x)
{
    float y = 0.f;
    if constexpr (Epi::pairs) y = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));   // lane ^ 1
    epi.put(row, c, e, x, y);
}

// 16 bytes per lane straight into LDS: lane l's piece lands at lds_addr + 16 * l (wave-uniform)
__device__ __forceinline__ void lds_load16(const float *src, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}

// ST stages of U slices of 32 k, one barrier per stage. The waves' fragments are read 4 bytes per lane (16 rows' chunks fill the 64
// banks), CG times 4 k ahead of the matrix instructions that take them, and requests go out behind those; the order is fixed, since left
// to the compiler the reads sink to their uses. (The kernel before this one read 16 bytes per lane for 32x32x2 instructions and
// picked each lane half's k by two selects per instruction, behind the reads' full latency.) Bound: the fp32 matrix rate (155
// TFLOP/s measured, no less on normal data than on zeros); 1018 rows of the 1B shape, us: gate / up 631 -> 551 (124 TFLOP/s), q/k/v
// 135 -> 124, down 350 -> 296, o 92 -> 78. Two stages of 128 x 128 tiles: two workgroups share a CU and hide each other's barriers.
// 64 x 64 tiles: two per CU take two slices per barrier (down 321 -> 296); three per CU, which these would not let in, three
// stages of one (q/k/v: 124 against 157).
template <int BM, int BN, int WM, int WN, int ST, int U, int CG, class Epi>
__global__ void __launch_bounds__(256, 2)
k_gemm_f32mfma(const float *__restrict__ A, int64_t lda, FMap map, Epi epi, int64_t M, int N, int K, int tiles_m, int tiles_n)
{
    static_assert((BM / WM) * (BN / WN) == 4, "four waves");
    constexpr int NWN = BN / WN, TM = WM / 16, TN = WN / 16, AP = BM / 32, BP = BN / 32;
    constexpr int PP = AP + BP, NG = 8 * U / CG, NM = CG * TM * TN, NR = CG * (TM + TN);   // groups of CG * 4 k, their matrix instructions and reads
    constexpr uint32_t LB = (BM + BN) * 128, SB = U * LB;     // a slice: rows of 32 floats, 16-byte chunks XOR-swizzled; a stage: U slices
    static_assert(8 * U % CG == 0 && NR <= NM && NG * NM % (U * PP) == 0, "whole groups; a group's instructions cover the next one's reads, all of them the requests");
    static_assert(ST >= 2 && U * PP * (ST - 2) < 64 && ST * SB <= 163840, "vmcnt counts the loads in flight; the LDS holds them");
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
    const int KT = K / (32 * U);
    auto request = [&](auto p_, int koff, uint32_t stage) {
        constexpr int u = p_ / PP, p = p_ % PP;
        const uint32_t to = stage + u * LB + (uint32_t)(p * 4096 + wave * 1024);
        if constexpr (p < AP) lds_load16(ap[p] + koff + 32 * u, to);
        else lds_load16(bp[p - AP] + koff + 32 * u, to);
    };
    f32x4v_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4v_t{0.f, 0.f, 0.f, 0.f};
    const int r16 = lane & 15, g = lane >> 4, fsw = (r16 >> 1) & 7;       // this lane supplies k = 4c + g of row r16 of each 16
    const int a_frag = (wm * WM + r16) * 128 + g * 4, b_frag = (BM + wn * WN + r16) * 128 + g * 4;
    struct Frags { float a[CG][TM], b[CG][TN]; } f[2];
    auto read = [&](auto r_, Frags &x, int grp, uint32_t stage) {
        constexpr int R = r_, c = R / (TM + TN), i = R % (TM + TN);
        const unsigned char *const st = lds + stage + ((grp * CG + c) >> 3) * LB;
        const int coff = (((grp * CG + c) & 7) ^ fsw) << 4;
        if constexpr (i < TM) x.a[c][i] = *reinterpret_cast<const float *>(st + a_frag + i * 2048 + coff);
        else x.b[c][i - TM] = *reinterpret_cast<const float *>(st + b_frag + (i - TM) * 2048 + coff);
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) static_for<U * PP>([&](auto p) { request(p, (s < KT ? s : KT - 1) * 32 * U, s * SB); });
    uint32_t cur = 0, fre = (ST - 1) * SB;
    for (int kt = 0; kt < KT; ++kt) {
        // slice kt has landed (the ST - 2 younger ones may be in flight), the stage of slice kt - 1 is read out; for all waves
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(U * PP * (ST - 2)) : "memory");
        const int koff = (kt + ST - 1 < KT ? kt + ST - 1 : KT - 1) * 32 * U;
        static_for<NR>([&](auto r) { read(r, f[0], 0, cur); });
        static_for<NG>([&](auto g_) {
            constexpr int grp = g_;
            static_for<NM>([&](auto m_) {
                constexpr int m = m_, c = m / (TM * TN), i = m / TN % TM, j = (i & 1) ? TN - 1 - m % TN : m % TN;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[grp & 1].a[c][i], f[grp & 1].b[c][j], acc[i][j], 0, 0, 0);
                if constexpr (grp + 1 < NG && m < NR) read(m_, f[1 - (grp & 1)], grp + 1, cur);
                constexpr int q = grp * NM + m;               // the requests: one behind every MPR-th instruction
                constexpr int MPR = NG * NM / (U * PP);
                if constexpr (q % MPR == MPR / 2) request(std::integral_constant<int, q / MPR>{}, koff, fre);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        fre = cur;
        cur = cur + SB == ST * SB ? 0 : cur + SB;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // no LDS-direct load outlives its workgroup
    const int col0 = n0 + wn * WN + r16;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if (col0 + 16 * j >= N) continue;                    // (N is even where columns come in pairs)
        const typename Epi::Col cj = epi.column(col0 + 16 * j);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = m0 + wm * WM + i * 16 + 4 * g + r;
                if (row < M) f32_put(epi, row, cj, epi.early(row, cj), acc[i][j][r]);
            }
    }
}

// 32 x 32 tiles of four waves, one 16x16 tile each: a quarter of the tile and of the chain's time per k, for products too
// small to give every CU a 64 x 64 tile. Pipeline as in k_gemm_tile: four slices of 32 k in flight, the fragments of
// slice kt + 1 read (4 bytes per lane, conflict-free: 16 rows' chunks fill the 64 banks) while slice kt is multiplied.
constexpr int F32SMALL_STAGES = 4;
template <class Epi>
__global__ void __launch_bounds__(256)
k_gemm_f32small(const float *__restrict__ A, int64_t lda, FMap map, Epi epi, int64_t M, int N, int K, int tiles_m, int tiles_n)
{
    constexpr int ST = F32SMALL_STAGES;
    constexpr uint32_t SB = 64 * 128;
    extern __shared__ __align__(16) unsigned char lds[];     // (a static array that only the loads' asm writes would count as unwritten)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= n_tiles) return;
    const int64_t m0 = (int64_t)(lin % tiles_m) * 32;
    const int n0 = (lin / tiles_m) * 32;
    const int chunk = tid & 7, rip = tid >> 3;               // 8 lanes x 16 bytes per row
    const int sw = (chunk ^ ((rip >> 1) & 7)) * 4;
    const float *const ap = A + (m0 + rip < M ? m0 + rip : M - 1) * lda + sw;
    const float *const bp = map.row(n0 + rip < N ? n0 + rip : N - 1) + sw;
    const int KT = K / 32;
    auto request = [&](int kt, uint32_t stage) {
        const int koff = (kt < KT ? kt : KT - 1) * 32;       // past the end: the last slice again, never multiplied
        lds_load16(ap + koff, stage + (uint32_t)(wave * 1024));
        lds_load16(bp + koff, stage + (uint32_t)(4096 + wave * 1024));
    };
    f32x4v_t acc = {0.f, 0.f, 0.f, 0.f};
    const int r16 = lane & 15, g = lane >> 4;                // this lane supplies k = 4c + g of row r16 of its wave's tile
    const int col = n0 + (wave & 1) * 16 + r16;              // and gets rows row0 .. row0 + 3 of this column
    const int64_t row0 = m0 + (wave >> 1) * 16 + 4 * g;
    const bool there = col < N;
    const int ar = (wave >> 1) * 16 + r16, br = (wave & 1) * 16 + r16;
    const int a_frag = ar * 128 + g * 4, b_frag = 4096 + br * 128 + g * 4, asw = (ar >> 1) & 7, bsw = (br >> 1) & 7;
    float a0[8], b0[8], a1[8], b1[8];
    auto fragments = [&](float (&a)[8], float (&b)[8], uint32_t stage) {
        const unsigned char *const st = lds + stage;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            a[c] = *reinterpret_cast<const float *>(st + a_frag + ((c ^ asw) << 4));
            b[c] = *reinterpret_cast<const float *>(st + b_frag + ((c ^ bsw) << 4));
        }
    };
    auto multiply = [&](const float (&a)[8], const float (&b)[8]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], b[c], acc, 0, 0, 0);
    };
    // (ahead of the LDS-direct loads, whose count the waits below know)
    const typename Epi::Col c = epi.column(there ? col : 0);
    typename Epi::Early early[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) early[r] = epi.early(row0 + r < M ? row0 + r : M - 1, c);
#pragma unroll
    for (int s = 0; s < ST; ++s) request(s, s * SB);
    uint32_t cur = 0, nxt = SB;                              // the stages of slices kt and kt + 1
#define SOL_F32_SYNC(N) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(2 * (N)) : "memory")
    SOL_F32_SYNC(ST - 1);
    fragments(a0, b0, 0);
    for (int kt = 0; kt < KT; kt += 2) {
        SOL_F32_SYNC(ST - 2);                                // slice kt + 1 is there, the stage of slice kt is read out
        request(kt + ST, cur);
        fragments(a1, b1, nxt);
        multiply(a0, b0);
        cur = nxt; nxt = nxt + SB == ST * SB ? 0 : nxt + SB;
        if (kt + 1 >= KT) break;
        SOL_F32_SYNC(ST - 2);
        request(kt + 1 + ST, cur);
        fragments(a0, b0, nxt);
        multiply(a1, b1);
        cur = nxt; nxt = nxt + SB == ST * SB ? 0 : nxt + SB;
    }
#undef SOL_F32_SYNC
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // no LDS-direct load outlives its workgroup
    if (!there) return;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (row0 + r < M) f32_put(epi, row0 + r, c, early[r], acc[r]);
}

template <int BM, int BN, int WM, int WN, int ST, int U, int CG, class Epi>
static bool launch_f32mfma(const float *A, int64_t lda, const FMap &map, const Epi &epi, int64_t M, int N, int K, hipStream_t st)
{
    constexpr size_t lds = (size_t)ST * U * (BM + BN) * 128;
    auto kern = k_gemm_f32mfma<BM, BN, WM, WN, ST, U, CG, Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return false;
        attr_done = true;
    }
    const int tm = (int)((M + BM - 1) / BM), tn = (N + BN - 1) / BN, per_xcd = (tm * tn + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256), lds, st, A, lda, map, epi, M, N, K, tm, tn);
    return true;
}

// The tile is the one that ends soonest by what was measured at K = 2048 and 8192 (r: rounds of one tile on every CU; us at K = 2048, 32 to 3000
// rows of 2048, 3072 and 16384 columns):
//   32 x 32: 10 + 11.6 r        21 at one round, 33, 43, 54, 68, 80, 91, 103, 118; 195 at 16
//   64 x 64: 47; 2 + 35 r       46, 72, 106, 138, 178, 208, 249, 282, 384 at 11. Two workgroups of two slices per stage share a CU, or three of
//                               one: 72 against 75 at two rounds, 138 - 147 at four; 48 - 46 at one (202 - 175 at K = 8192), 120 - 106 at
//                               three, level from five on. So two slices at two and four rounds, where K is whole pairs of slices.
//                               One and two rounds are worth 10 less where K is short or columns come in pairs: alone 9.1 us against 9.9 of
//                               four rounds of 32 x 32 at K = 256, but with SiLU * up at its end 12.9 either way, and the quantiser after it
//                               4.6 - 3.7 (4 x 128 tokens of a one-layer model); q/k/v of 300 rows alone 48 - 55, with the rotation
//                               56.8 - 55.2; gate / up of 70 rows alone 70 - 79, with SiLU * up 78 - 80 and the layer level
//   128 x 128: 147; 126 r       for an even r, as long for the odd one before it (two share a CU): 250 at two, 498 at three, 508 at four
// So: 32 x 32 for up to three rounds of it (and five: 68 against 72), 64 x 64 up to four of its own and wherever its share of the last
// round is smaller, 128 x 128 where it fills pairs of rounds: within 3 % of the best of the four at 146 sizes of K = 64 to 14336, one and
// two rounds of the latter aside. 1018 rows of the 1B shape: o and down two rounds of 64 x 64, q/k/v three, gate / up four of 128 x 128. Before this
// was measured for the present kernels 64 x 64 was priced 21 + 36 r: 800 rows by 2048 columns took 90 us where two rounds take 72, 1400
// rows 144 where three take 107, 700 rows by 16384 columns 498 (128 x 128) where eleven take 384.
template <class Epi>
static bool launch_f32_product(const float *A, int64_t lda, const FMap &map, const Epi &epi, int64_t M, int64_t N, int K, hipStream_t st)
{
    auto aligned = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    if (K < 32 || K % 32 || lda % 4 || map.ldw % 4 || !aligned(A) || !aligned(map.base[0]) || !aligned(map.base[1]) ||
        !aligned(map.base[2]) || M > (1ll << 30) || N > (1ll << 30))
        return false;                                        // 16-byte loads of whole slices
    if (M <= 0 || N <= 0) return true;
    const int cus = device_cus() > 0 ? device_cus() : 256;
    auto rounds = [&](int b) { return ((M + b - 1) / b * ((N + b - 1) / b) + cus - 1) / cus; };
    if ((M + 31) / 32 * ((N + 31) / 32) > (1ll << 30)) return false;
    const int64_t r64 = rounds(64), r128 = rounds(128);
    const double c32 = 10 + 11.6 * (double)rounds(32), c128 = r128 == 1 ? 147 : 126 * (double)(r128 + r128 % 2);
    const double c64 = (r64 == 1 ? 47 : 2 + 35 * (double)r64) + (r64 <= 2 && (Epi::pairs || K < 1024) ? 10 : 0);
    if (c128 <= c64 && c128 <= c32) return launch_f32mfma<128, 128, 64, 64, 2, 1, 1>(A, lda, map, epi, M, (int)N, K, st);
    if (c64 <= c32)
        return (r64 == 2 || r64 == 4) && K % 64 == 0 ? launch_f32mfma<64, 64, 32, 32, 2, 2, 2>(A, lda, map, epi, M, (int)N, K, st)
                                                     : launch_f32mfma<64, 64, 32, 32, 3, 1, 2>(A, lda, map, epi, M, (int)N, K, st);
    const int tm = (int)((M + 31) / 32), tn = (int)((N + 31) / 32);
    hipLaunchKernelGGL(k_gemm_f32small<Epi>, dim3((tm * tn + 7) / 8 * 8), dim3(256), F32SMALL_STAGES * 64 * 128, st, A, lda, map, epi, M, (int)N, K, tm, tn);
    return true;
}

bool launch_gemm_f32rows(const float *A, int64_t lda, const float *w, int N, int64_t ldw, float *C, int64_t ldc, int64_t M, int K,
                         hipStream_t st)
{
    const FMap map{{w, w, w}, {N, N, N}, ldw, FMAP_STACKED, 0};
    return launch_f32_product(A, lda, map, F32Store{C, ldc}, M, N, K, st);
}

// out = x2 + A w^T
bool launch_gemm_f32_resid(const float *A, const float *w, const float *x2, float *out, int64_t M, int N, int K, hipStream_t st)
{
    const FMap map{{w, w, w}, {N, N, N}, K, FMAP_STACKED, 0};
    return launch_f32_product(A, K, map, F32Resid{x2, out, N}, M, N, K, st);
}

// a = silu(A wg^T) * (A wu^T)
bool launch_gemm_f32_silu(const float *A, const float *wg, const float *wu, float *a, int64_t M, int dff, int K, hipStream_t st)
{
    const FMap map{{wg, wu, wu}, {0, 0, 0}, K, FMAP_PAIRS, 0};
    return launch_f32_product(A, K, map, F32Silu{a, dff}, M, 2 * (int64_t)dff, K, st);
}

// q / k / v, rotary embedding, cache write (cache_rows as for launch_rope_store)
bool launch_gemm_f32_qkv(const float *A, const float *wq, const float *wk, const float *wv, float *q, float *kc, float *vc,
                         const float2 *rope, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh, int K,
                         int *flags, hipStream_t st, int cache_rows)
{
    const int64_t M = (int64_t)n_seq * T;
    const int nq = Hq * dh, nkv = Hkv * dh;
    if (dh % 2) return false;
    const FMap map{{wq, wk, wv}, {nq, nq + nkv, nq + 2 * nkv}, K, FMAP_ROPE, dh};
    const F32Qkv epi{q, kc, vc, rope, pos0, T, L_max, cache_rows > 0 ? cache_rows : L_max, Hq, Hkv, dh, flags};
    return launch_f32_product(A, K, map, epi, M, (int64_t)nq + 2 * nkv, K, st);
}

void launch_gemm_generic(const void *A, int a_dtype, int64_t lda, const void *W, int w_dtype, int64_t ldw, float *C,
                         int64_t ldc, int64_t M, int N, int K, hipStream_t st)
{
    if (M <= 0 || N <= 0) return;
    if (a_dtype == 0 && w_dtype == 0 &&
        launch_gemm_f32rows((const float *)A, lda, (const float *)W, N, ldw, C, ldc, M, K, st))
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
