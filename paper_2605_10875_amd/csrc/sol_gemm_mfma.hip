// bf16 MFMA GEMMs for gfx950 with fused epilogues:  C[M][Nv] = A[M][K] * Wv[Nv][K]^T, fp32 accumulate.
//
// Both operands are K-contiguous, which is the layout the matrix instructions want for A and B
// alike (each lane supplies 8 consecutive k of one row / one column). "Nv" is a virtual column
// space: a column maps to a row of one of up to three weight matrices (q|k|v stacked, or gate and
// up interleaved in pieces of 32 columns so that SiLU(gate)*up is formed inside one wave tile).
//
// k_gemm_mfma: 256 x 256 tiles for whole rounds of the chip; k_gemm_tile: smaller tiles for few rows. A and B K-slices
// of 64 go from global memory straight into LDS (LDS-direct loads, XOR-swizzled 16-byte chunks so that the 128-bit fragment
// reads are bank-conflict free). Workgroups are mapped to tiles
// XCD-aware: each of the 8 XCDs walks its own contiguous band of the tile grid in groups of
// GROUP_M tile rows, so the tiles resident on an XCD at any time share A rows and B columns in
// that XCD's L2.
#include "sol_internal.h"

namespace sol {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // native 16-byte vector (stays in registers)
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 64;               // K step (bf16 elements); one LDS row = 128 bytes = 8 chunks of 16 B
constexpr int GROUP_M = 4;           // tile rows walked together by an XCD: its 32 CUs then hold 4 x 8 tiles (measured on the
                                     // 16 x 2048-token stack: 2, 4 within 1 %; 8: 2 - 4 % slower; 16: 4 - 8 % slower)
// LDS has 64 banks of 4 bytes: two 128-byte rows share one bank row, and the 16-byte chunk index is XOR-ed with bits of the row so
// that the 16 rows of a fragment lie in different banks: 16 consecutive token rows; weight rows 8a + b (+ 4), a and b = 0 .. 3.
__device__ __forceinline__ uint32_t x_swizzle(int r) { return (uint32_t)((r >> 1) & 7); }
__device__ __forceinline__ uint32_t w_swizzle(int r) { return (uint32_t)(((r >> 1) & 1) | (((r >> 3) & 3) << 1)); }

struct BMap {                        // virtual column -> weight row
    const bf16_t *base[3];
    int seg_end[3];                  // mode 0: virtual columns [seg_end[i-1], seg_end[i]) belong to base[i]
    int mode;                        // 0 = stacked segments, 1 = gate/up interleaved in halves of `half`
    int half;
    int64_t ld;
    __device__ __forceinline__ const bf16_t *row(int v) const
    {
        if (mode == 0) {
            if (v < seg_end[0]) return base[0] + (int64_t)v * ld;
            if (v < seg_end[1]) return base[1] + (int64_t)(v - seg_end[0]) * ld;
            return base[2] + (int64_t)(v - seg_end[1]) * ld;
        }
        const int blk = v / (2 * half), w = v - blk * 2 * half;
        const int r = blk * half + (w < half ? w : w - half);
        return (w < half ? base[0] : base[1]) + (int64_t)r * ld;
    }
};

// own * cos -+ partner * sin (lower / upper half of the head). Which of the two products is rounded before the sum (the sine's in
// the lower half, the cosine's in the upper) is spelled out: left to the compiler, it differed between the epilogues, and the last
// bit of a row's q and K with the tiles that its call was dealt to.
__device__ __forceinline__ float rotated(float own, float partner, float2 cs, bool lo)
{
    return lo ? __builtin_fmaf(own, cs.x, -(partner * cs.y)) : __builtin_fmaf(partner, cs.y, own * cs.x);
}

// LM head with the logits never written: per (token, tile of 128 vocabulary entries) the maximum and the sum of
// exp(logit - maximum); k_nll_finish_cols folds the tiles of a token into  logsumexp(logits) - logits[target]
// (Method, Eq. 1, negated), the target's logit coming from k_target_logit.
// target token of every row (teacher-forced rows (b, g, t) share the targets of input b when broadcast_g)
// and clears the n_pad pieces of 16 bytes behind the hidden states' last row (a launch less for every call whose rows are no whole tiles)
__global__ void __launch_bounds__(256)
k_row_targets(const int32_t *__restrict__ targets, int64_t M, int G, int Tn, int broadcast_g, int V, int32_t *__restrict__ row_tgt,
              int *__restrict__ flags, u32x4_t *__restrict__ pad, int64_t n_pad)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = r; i < n_pad; i += (int64_t)gridDim.x * 256) pad[i] = u32x4_t{0u, 0u, 0u, 0u};
    if (r >= M) return;
    const int64_t ti = broadcast_g ? (r / ((int64_t)G * Tn)) * Tn + (r % Tn) : r;
    int tg = targets[ti];
    if (tg < 0 || tg >= V) {                       // outside the vocabulary: clamped, and reported through the sticky flag
        atomicOr(flags, FLAG_BAD_TOKEN);
        tg = tg < 0 ? 0 : V - 1;
    }
    row_tgt[r] = tg;
}

// logit of each row's target: one wave per row, hf[r] . lm_head[target(r)] in fp32
__global__ void __launch_bounds__(256)
k_target_logit(const bf16_t *__restrict__ hf, const bf16_t *__restrict__ lm_head, const int32_t *__restrict__ row_tgt, int64_t M,
               int K, float *__restrict__ tgt_logit)
{
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    const bf16_t *a = hf + r * K, *b = lm_head + (int64_t)row_tgt[r] * K;
    float acc = 0.f;
    for (int k = lane * 8; k < K; k += 512) {
        const uint4 x = *reinterpret_cast<const uint4 *>(a + k), y = *reinterpret_cast<const uint4 *>(b + k);
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc = __builtin_fmaf(__uint_as_float(xs[e] << 16), __uint_as_float(ys[e] << 16), acc);
            acc = __builtin_fmaf(__uint_as_float(xs[e] & 0xFFFF0000u), __uint_as_float(ys[e] & 0xFFFF0000u), acc);
        }
    }
    acc = wave_sum_dpp(acc);
    if (lane == 0) tgt_logit[r] = acc;
}

// nll = max + log(sum_t s_t * exp(m_t - max)) - target logit over part [n_wt][Mp]. A workgroup takes 32 rows; half wave q
// of its 32 takes the tiles t = q, q + 32, ... of these rows (it reads 32 consecutive entries of a tile), keeps the first
// 32 of them in registers (all of them up to 1024 tiles; the others are read twice), and adds them up under the row's
// maximum; the 32 sums of a row are added by one thread: the same sequence of operations for every row, whatever the batch.
// All sums are trees: 4e-8 (rms, of the sum) from 64 bits at 1002 tiles, where a running maximum and sum is 7e-8 off and a
// chain of 32 and 32 additions 9e-8.
// Bound: latency for few rows (one load and one exchange each for maximum and sum; a running maximum was a chain of a load
// and two exponentials per tile: 28 us for 64 rows of 1002 tiles, now 8.5), HBM for many (4.3 TB/s at 32768).
constexpr int NLL_FIN_TILES = 32;                              // per half wave in registers
template <int N> __device__ __forceinline__ float tree_sum(float (&v)[N])
{
#pragma unroll
    for (int w = N / 2; w >= 1; w >>= 1)
#pragma unroll
        for (int u = 0; u < w; ++u) v[u] += v[u + w];
    return v[0];
}
__global__ void __launch_bounds__(1024)
k_nll_finish_cols(const float2 *__restrict__ part, const float *__restrict__ tgt_logit, int n_wt, int64_t M, int64_t Mp,
                  float *__restrict__ nll)
{
    __shared__ float fold[32][33];
    const int rl = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int64_t r = (int64_t)blockIdx.x * 32 + rl;           // r < Mp: the grid covers ceil(M / 32) * 32 <= Mp rows
    const int t_more = 32 * NLL_FIN_TILES;                     // tiles from here on are read twice, 8 per step and half wave
    float2 v[NLL_FIN_TILES];
#pragma unroll
    for (int u = 0; u < NLL_FIN_TILES; ++u) {
        const int t = q + 32 * u;
        v[u] = make_float2(-INFINITY, 0.f);
        if (t < n_wt) v[u] = part[(int64_t)t * Mp + r];
    }
    float mx = v[0].x;
#pragma unroll
    for (int u = 1; u < NLL_FIN_TILES; ++u) mx = fmaxf(mx, v[u].x);
    for (int t = q + t_more; t < n_wt; t += 32) mx = fmaxf(mx, part[(int64_t)t * Mp + r].x);
    fold[q][rl] = mx;
    __syncthreads();
#pragma unroll 8
    for (int i = 0; i < 32; ++i) mx = fmaxf(mx, fold[i][rl]);
    __syncthreads();
    float s[NLL_FIN_TILES];
#pragma unroll
    for (int u = 0; u < NLL_FIN_TILES; ++u) s[u] = v[u].y * expf(v[u].x - mx);
    float se = tree_sum(s);
    for (int t0 = q + t_more; t0 < n_wt; t0 += 8 * 32) {
        float m[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = t0 + 32 * u;
            const float2 w = t < n_wt ? part[(int64_t)t * Mp + r] : make_float2(-INFINITY, 0.f);
            m[u] = w.y * expf(w.x - mx);
        }
        se += tree_sum(m);
    }
    fold[q][rl] = se;
    __syncthreads();
    if (q != 0 || r >= M) return;
#pragma unroll
    for (int i = 0; i < 32; ++i) s[i] = fold[i][rl];
    nll[r] = (mx + logf(tree_sum(s))) - tgt_logit[r];
}

// 16 bytes per lane from global memory (wave-uniform base + 32-bit byte offset per lane) straight into LDS: lane l's
// piece lands at lds_base + C + 16 * l (M0 holds the wave's LDS byte address, a base and a constant so that the compiler keeps no 32 sums
// of them in scalar registers; one wait state between writing M0 and the load). Written as inline assembly because the
// compiler, which sees an LDS write it cannot place, would wait for the load before the next LDS read of any stage. The kernel
// therefore owns the waits: before the barrier that publishes a stage, and before a workgroup ends. The kernel must have
// no static LDS (the dynamic segment then starts at LDS address 0).
template <int C> __device__ __forceinline__ void dtl16c(const bf16_t *base, uint32_t byte_off, uint32_t lds_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_base), "n"(C) : "memory", "m0", "scc");
}
// s_waitcnt vmcnt(N) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, the expcnt and lgkmcnt fields at "no wait")
template <int N> __device__ __forceinline__ void vm_wait()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt(((N >> 4) << 14) | 0x0F70 | (N & 15));
}

// ------------------------------------------------------------------------------------------------
// 256 x 256 tiles: 4 waves, one per SIMD, each with 128 weight rows x 128 tokens of the product on v_mfma_f32_16x16x32_bf16
// (its sums are those of two 32x32x16 instructions bit for bit, so the tile does not show in the results). The weights are the
// instruction's first operand: a lane's four results are then consecutive columns of one token's output row.
//
// Bound: for the most part the power the chip grants its matrix cores. With normally distributed operands a loop of nothing but
// 32x32x16 instructions reaches 1.78 PFLOP/s (2.4 on ones), of 16x16x32 2.05: they move fewer accumulator bits per product
// (sol_measure_mfma measures all four). This kernel without an epilogue reaches 1.67 of the 2.05.
// A step (64 of K) goes through the four quadrants of the wave tile: (top, left), (top, right), (bottom, right), (bottom,
// left), each 32 instructions, and reads one half of an operand from the LDS per quadrant, for the next one. So every half
// of a slice is read out during ONE quadrant, and the LDS-direct requests of slice kt + 2 go into it from the barrier that
// follows, two barriers per step: a request has 1 to 1.5 steps to arrive, where the whole-slice order of the kernel before this
// one (fragments two k-groups ahead, one barrier) left it 0.5 to 1.
// 32768 rows, epilogue included, us, that kernel -> this one, normal data: 1B shape gate / up 1627 -> 1437, down 823 -> 738, o 264 -> 245,
// q/k/v 371 -> 334, head 12300 -> 11665; 8B shape gate / up 5441 -> 4877, down 2930 -> 2504. Without an epilogue gate / up is 1320 (1.67
// PFLOP/s; 980 us, 2.24 PFLOP/s, on zeros): SiLU and the head's exponentials cost what they take to issue (3.7 and 4.1 us per tile
// of 42), the residual epilogues what a round's 98 MB take at the rate of a copy (all CUs store at once; letting the stores
// drain behind another step changes nothing).
//
// The 256 accumulator registers of a lane are a[0:255], named in the instructions' text: left to the register allocator, 64
// groups of four that fill the file exactly are moved about between steps (0.8 PFLOP/s). The compiler must not use that
// half of the register file in this kernel for anything else. SOL_ACC_ALL among the clobbers of every barrier, of acc_settle and
// before each token of the epilogue keeps it from values that live longer than that; for the others the build looks in the machine
// code and fails on any other use (isa.py). Wait states between the last matrix instruction and the first read of its result are
// the kernel's own business too (acc_settle).
// ------------------------------------------------------------------------------------------------
#define SOL_A4(x) "a" #x "0", "a" #x "1", "a" #x "2", "a" #x "3", "a" #x "4", "a" #x "5", "a" #x "6", "a" #x "7", "a" #x "8", "a" #x "9"
#define SOL_ACC_ALL                                                                                                             \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", SOL_A4(1), SOL_A4(2), SOL_A4(3), SOL_A4(4), SOL_A4(5), SOL_A4(6),   \
    SOL_A4(7), SOL_A4(8), SOL_A4(9), SOL_A4(10), SOL_A4(11), SOL_A4(12), SOL_A4(13), SOL_A4(14), SOL_A4(15), SOL_A4(16), SOL_A4(17), \
    SOL_A4(18), SOL_A4(19), SOL_A4(20), SOL_A4(21), SOL_A4(22), SOL_A4(23), SOL_A4(24), "a250", "a251", "a252", "a253", "a254", "a255"

// accumulator tile at a[R:R+3] = (FIRST ? 0 : itself) + x * y
template <int R, bool FIRST> __device__ __forceinline__ void acc_mma(const bf16x8_t &x, const bf16x8_t &y)
{
    if constexpr (FIRST) asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, 0" ::"v"(x), "v"(y), "n"(R), "n"(R + 3));
    else asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(x), "v"(y), "n"(R), "n"(R + 3));
}
// the last matrix instruction's results may be read (18 wait states at most)
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory", SOL_ACC_ALL); }
template <int R> __device__ __forceinline__ f32x4_t acc_read()
{
    float a, b, c, d;
    asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]"
                 : "=v"(a), "=v"(b), "=v"(c), "=v"(d) : "n"(R), "n"(R + 1), "n"(R + 2), "n"(R + 3));
    return f32x4_t{a, b, c, d};
}

// ------------------------------------------------------------------------------------------------
// Epilogues. A lane holds, for token 16 t + lane % 16 of its wave tile (t < TX) and g = lane / 16, the columns
// 32 p + 8 g .. + 7 (p < NP) of the wave tile: 16 bytes of a bf16 row. Parts of an epilogue (row: an existing token, col0:
// the wave tile's first virtual column):
//   place(row[TX], p)              what is known of the lane's tokens before anything else
//   fetch(row, p, col0, g, aux)    reads what a token's piece needs, AHEAD tokens ahead of
//   put(row, ok, p, col0, g, v, aux)   which combines and stores it (ok: the token exists)
// The pieces lie in the caller's tensors, which are aligned to their elements only: AnyU4, AnyF4.
// ------------------------------------------------------------------------------------------------
typedef u32x4_t AnyU4 __attribute__((aligned(2)));
typedef f32x4_t AnyF4 __attribute__((aligned(4)));
struct NoPlace {};
struct EpiTokens {                                          // what most epilogues have in common
    static constexpr bool weight_rows = false;              // tiles are walked in bands of tokens (or of weight rows)
    static constexpr int AHEAD = 2;
    typedef NoPlace Place;
    template <int NP> struct Aux {};
    template <int TX> __device__ __forceinline__ void place(const uint32_t (&)[TX], NoPlace (&)[TX]) const {}
    template <class A> __device__ __forceinline__ void fetch(uint32_t, const NoPlace &, int, int, A &) const {}
};
__device__ __forceinline__ u32x4_t pack8(const float (&v)[8])
{
    return u32x4_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

struct EpiStoreF32x8 : EpiTokens {
    float *C; int64_t ldc;
    EpiStoreF32x8(float *c, int64_t l) : C(c), ldc(l) {}
    template <int NP> __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[NP][8], const Aux<NP> &) const
    {
        float *const o = C + row * ldc + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<AnyF4 *>(o + 32 * p + 4 * h) = f32x4_t{v[p][4 * h], v[p][4 * h + 1], v[p][4 * h + 2], v[p][4 * h + 3]};
    }
};

// x2 = resid + acc (fp32 out), resid in bf16
struct EpiResidF32x8 : EpiTokens {
    const bf16_t *resid; float *out; int64_t ld;
    EpiResidF32x8(const bf16_t *r, float *o, int64_t l) : resid(r), out(o), ld(l) {}
    template <int NP> struct Aux { u32x4_t r[NP]; };
    template <int NP> __device__ __forceinline__ void fetch(uint32_t row, const NoPlace &, int col0, int g, Aux<NP> &x) const
    {
        const bf16_t *const r = resid + row * ld + col0 + 8 * g;
#pragma unroll
        for (int p = 0; p < NP; ++p) x.r[p] = *reinterpret_cast<const AnyU4 *>(r + 32 * p);
    }
    template <int NP> __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[NP][8], const Aux<NP> &x) const
    {
        float *const o = out + row * ld + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4_t y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t w = x.r[p][2 * h + (e >> 1)];
                    y[e] = v[p][4 * h + e] + __uint_as_float((e & 1) ? w & 0xFFFF0000u : w << 16);
                }
                *reinterpret_cast<f32x4_t *>(o + 32 * p + 4 * h) = y;
            }
    }
};

// out = bf16(x2 + acc), x2 in fp32
struct EpiResidOut8 : EpiTokens {
    const float *x2; bf16_t *out; int64_t ld;
    EpiResidOut8(const float *x, bf16_t *o, int64_t l) : x2(x), out(o), ld(l) {}
    template <int NP> struct Aux { f32x4_t r[NP][2]; };
    template <int NP> __device__ __forceinline__ void fetch(uint32_t row, const NoPlace &, int col0, int g, Aux<NP> &x) const
    {
        const float *const r = x2 + row * ld + col0 + 8 * g;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) x.r[p][h] = *reinterpret_cast<const AnyF4 *>(r + 32 * p + 4 * h);
    }
    template <int NP> __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[NP][8], const Aux<NP> &x) const
    {
        bf16_t *const o = out + row * ld + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = v[p][e] + x.r[p][e >> 2][e & 3];
            *reinterpret_cast<AnyU4 *>(o + 32 * p) = pack8(y);
        }
    }
};

// a = bf16(silu(gate) * up); gate in the wave tile's even pieces, up in the odd ones
struct EpiSiluMul8 : EpiTokens {
    bf16_t *a; int64_t ld;
    EpiSiluMul8(bf16_t *a_, int64_t l) : a(a_), ld(l) {}
    static __device__ __forceinline__ float silu_mul(float g, float u)
    {
        // g * sigmoid(g) * u with the hardware exp2 / reciprocal instructions (about 1 ulp each, far below the
        // bf16 rounding that follows). v_rcp_f32 itself: a correctly rounded reciprocal is an eleven-instruction
        // division sequence, a third of this epilogue's vector instructions.
        return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
    }
    template <int NP> __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[NP][8], const Aux<NP> &) const
    {
        bf16_t *const o = a + row * ld + col0 / 2 + 8 * g;
        u32x4_t y[NP / 2];
#pragma unroll
        for (int p = 0; p < NP / 2; ++p) {
            float z[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = silu_mul(v[2 * p][e], v[2 * p + 1][e]);
            y[p] = pack8(z);
        }
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < NP / 2; ++p) *reinterpret_cast<u32x4_t *>(o + 32 * p) = y[p];
    }
};

// Rotary embedding on q and k heads (pairs (c, c + dh/2)), q -> [M][nq], k/v -> caches, positions by arithmetic. A row whose sequence
// does not fit its cache is flagged and not stored.
template <int DHT>
struct EpiQkvRope8 : EpiTokens {
    static constexpr int ND = DHT / 64;                     // pieces of cos / sin that a token needs
    static constexpr int AHEAD = DHT == 64 ? 2 : 1;         // (three sets of two pieces spill)
    bf16_t *q, *kc, *vc;
    const float2 *rope; const int32_t *pos0;
    int Tn, L_max, crows, Hq, Hkv;                          // crows: rows of a cache slab
    int *flags;
    EpiQkvRope8(bf16_t *q_, bf16_t *k, bf16_t *v, const float2 *r, const int32_t *p0, int T, int L, int c, int hq, int hkv, int *f)
        : q(q_), kc(k), vc(v), rope(r), pos0(p0), Tn(T), L_max(L), crows(c), Hq(hq), Hkv(hkv), flags(f) {}
    struct Place { int s, pos; };                           // pos < 0: not stored
    template <int NP> struct Aux { f32x4_t cs[ND][4]; };
    template <int TX> __device__ __forceinline__ void place(const uint32_t (&row)[TX], Place (&pl)[TX]) const
    {
        int p0[TX];
#pragma unroll
        for (int t = 0; t < TX; ++t) {
            pl[t].s = (int)(row[t] / (uint32_t)Tn);
            p0[t] = pos0 ? pos0[pl[t].s] : 0;
        }
#pragma unroll
        for (int t = 0; t < TX; ++t) {
            const bool bad = p0[t] < 0 || p0[t] + Tn > L_max;
            if (bad) atomicOr(flags, FLAG_CACHE_OVERFLOW);
            pl[t].pos = bad ? -1 : p0[t] + (int)(row[t] - (uint32_t)pl[t].s * (uint32_t)Tn);
        }
    }
    template <int NP> __device__ __forceinline__ void fetch(uint32_t, const Place &pl, int col0, int g, Aux<NP> &x) const
    {
        if (col0 >= (Hq + Hkv) * DHT) return;               // v
        const float *const r = reinterpret_cast<const float *>(rope + (int64_t)(pl.pos < 0 ? 0 : pl.pos) * (DHT / 2)) + 16 * g;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int h = 0; h < 4; ++h) x.cs[d][h] = *reinterpret_cast<const f32x4_t *>(r + 64 * d + 4 * h);
    }
    template <int NP> __device__ __forceinline__ void put(uint32_t row, bool ok, const Place &pl, int col0, int g, const float (&v)[NP][8], const Aux<NP> &x) const
    {
        static_assert(NP % (2 * ND) == 0, "whole heads");
        constexpr int dh = DHT;
        const int nq = Hq * dh, nkv = Hkv * dh;
        const int seg = col0 < nq ? 0 : (col0 < nq + nkv ? 1 : 2);            // the wave tile lies inside one of q / k / v
        const int w0 = col0 - (seg == 0 ? 0 : (seg == 1 ? nq : nq + nkv));
        bf16_t *d;                                          // piece 0's destination
        int64_t up;                                         // elements from pieces 0, 1 to 2, 3
        if (seg == 0) { d = q + row * (int64_t)nq + w0; up = 64; }
        else {
            d = (seg == 1 ? kc : vc) + (((int64_t)pl.s * Hkv + w0 / dh) * crows + pl.pos) * dh;
            up = dh == 64 ? (int64_t)crows * 64 : 64;
        }
        d += 8 * g;
        u32x4_t y[NP];
        if (seg == 2) {
#pragma unroll
            for (int p = 0; p < NP; ++p) y[p] = pack8(v[p]);
        } else {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const bool lo = (p & ND) == 0;              // lower half of its head; the partner is ND pieces on
                const int cd = p & (ND - 1);
                float z[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    z[e] = rotated(v[p][e], v[p ^ ND][e], make_float2(x.cs[cd][e >> 1][2 * (e & 1)], x.cs[cd][e >> 1][2 * (e & 1) + 1]), lo);
                y[p] = pack8(z);
            }
        }
        if (!ok || pl.pos < 0) return;
#pragma unroll
        for (int p = 0; p < NP; ++p) *reinterpret_cast<AnyU4 *>(d + (p >> 1) * up + 32 * (p & 1)) = y[p];
    }
};

// LM head with the logits never written: per (token, tile of 128 vocabulary entries) the maximum and the sum of exp(logit - maximum). A
// lane holds 32 logits of a token (rows 8g .. 8g + 7 of every 32), so both are sums over its registers plus two exchanges. The tiles
// are walked in bands of vocabulary entries: the big operand (525 MB of weights at the Llama vocabulary) is the one that each XCD streams
// once, and the hidden states, which the memory-side cache holds, are the ones read again. part: [V / 128][Mp] (token fastest; Mp =
// padded token count). What a token gets does not depend on the other tokens of the call.
struct EpiNllCols8 {
    static constexpr bool weight_rows = true;
    float2 *part;                                           // [V / 128][Mp]
    int64_t Mp;
};
__device__ __forceinline__ float lane_xor(float v, int lane, int x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ x) << 2, __builtin_bit_cast(int, v)));
}

// acc(i, t): accumulator of weight tile i (two per 32 columns) and token tile t, both integral constants
template <int TW, int TX, class Epi, class Acc>
__device__ __forceinline__ void tile_epilogue(const Epi &epi, Acc acc, int64_t m_w, int64_t M, int col0, int lane)
{
    constexpr int NP = TW / 2, AHEAD = Epi::AHEAD < TX ? Epi::AHEAD : TX;
    const int g = lane >> 4;
    uint32_t row[TX];
    bool ok[TX];
    typename Epi::Place pl[TX];
#pragma unroll
    for (int t = 0; t < TX; ++t) {
        const int64_t r = m_w + 16 * t + (lane & 15);
        ok[t] = r < M;
        row[t] = (uint32_t)(ok[t] ? r : M - 1);
    }
    epi.place(row, pl);
    typename Epi::template Aux<NP> aux[AHEAD + 1];
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) epi.fetch(row[t], pl[t], col0, g, aux[t]);
    static_for<TX>([&](auto t_) {
        constexpr int t = t_;
        if constexpr (t + AHEAD < TX) epi.fetch(row[t + AHEAD], pl[t + AHEAD], col0, g, aux[(t + AHEAD) % (AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
        float v[NP][8];
        static_for<TW>([&](auto i_) {
            constexpr int i = i_;
            const f32x4_t a = acc(i_, t_);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i >> 1][4 * (i & 1) + e] = a[e];
        });
        epi.put(row[t], ok[t], pl[t], col0, g, v, aux[t % (AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
    });
}
template <int TW, int TX, class Acc>
__device__ __forceinline__ void tile_epilogue(const EpiNllCols8 &epi, Acc acc, int64_t m_w, int64_t, int col0, int lane)
{
    static_assert(TW == 8, "tiles of 128 vocabulary entries");
    constexpr float LOG2E = 1.44269504088896341f;
    float2 *const dst = epi.part + (int64_t)(col0 / 128) * epi.Mp + m_w + (lane & 15);
    static_for<TX>([&](auto t_) {
        constexpr int t = t_;
        f32x4_t v[8];
        static_for<8>([&](auto i_) { v[i_] = acc(i_, t_); });
        float m = v[0][0];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) m = fmaxf(m, v[i][e]);
        m = fmaxf(m, lane_xor(m, lane, 16));
        m = fmaxf(m, lane_xor(m, lane, 32));
        const float ml = m * LOG2E;
        float h[2];                                         // rows with bit 2 clear, set
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int i = b; i < 8; i += 2)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    s0 += __builtin_amdgcn_exp2f(__builtin_fmaf(v[i][e], LOG2E, -ml));
                    s1 += __builtin_amdgcn_exp2f(__builtin_fmaf(v[i][e + 1], LOG2E, -ml));
                }
            h[b] = s0 + s1;
        }
        float se = h[0] + h[1];
        se += lane_xor(se, lane, 16);
        se += lane_xor(se, lane, 32);
        if (lane < 16) dst[16 * t] = make_float2(m, se);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// XT: token tiles of 16 per wave, 8 (256 x 256 tiles) or 4 (128 tokens x 256 weight rows: one tile per workgroup, for fewer rows;
// three LDS stages; 8B shape, 2048 rows, against 32x32x16 instructions in that tile, us: down 217 -> 197, o 56 -> 50). ST: LDS stages.
template <int XT, int ST, class Epi>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_gemm_mfma(const bf16_t *__restrict__ X, BMap bmap, int64_t m_first, int64_t M, int K, int tiles_r, int tiles_c, Epi epi)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr bool WALK = XT == 8;                          // several tiles per workgroup
    constexpr int BT = 32 * XT;                             // tokens of a tile
    constexpr int SB = (256 + BT) * 128;                    // a stage: 256 weight rows, BT token rows of 128 bytes
    constexpr int XQ = XT / 2;                              // requests per half of the tokens
    constexpr int IN_FLIGHT = (8 + XT) * (ST - 1);          // requests younger than what a half step reads
    static_assert((XT == 8 || XT == 4) && ST * SB <= 163840 && (!WALK || ST == 2), "tile");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ww = wave >> 1, wt = wave & 1;                // this wave's half of the weight rows, of the tokens

    // ---- XCD-aware tile mapping: workgroup b runs on XCD b % 8; XCD x owns a contiguous band ----
    const int n_tiles = tiles_r * tiles_c, per_xcd = (n_tiles + 7) / 8;
    const int band_end = ((int)(blockIdx.x & 7) + 1) * per_xcd < n_tiles ? ((int)(blockIdx.x & 7) + 1) * per_xcd : n_tiles;
    const int lin_step = (int)(gridDim.x >> 3);
    int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= band_end) return;
    const int group_sz = GROUP_M * tiles_c;

    // ---- sources of the staged K slices: uniform bases, per-lane byte offsets ----
    const int64_t ld = bmap.ld;                             // of weights and tokens alike
    const int64_t w_mid = (bmap.mode == 0 ? 64 : 32) * ld;  // rows of piece p + 2 behind piece p
    const int chunk = tid & 7, rip = tid >> 3;              // this thread's 16-byte piece and row of a pass of 32 rows
    const uint32_t w_off0 = ((uint32_t)rip * (uint32_t)ld + (uint32_t)((chunk ^ w_swizzle(rip)) * 8)) * 2u;
    const uint32_t w_off1 = w_off0 + (uint32_t)(2 * w_mid) * 2u;
    const uint32_t x_chunk = (uint32_t)((chunk ^ x_swizzle(rip)) * 8);
    uint32_t x_off[XT];
    const bf16_t *we, *wo, *we2, *wo2, *xb;                 // of the slice being requested: pieces 0, 1, 2, 3 (4 .. 7 at w_off1), tokens
    int64_t m0, m0_next;
    int n0, n0_next;
    auto tile_src = [&](int l, int64_t &m, int &n) {
        const int grp = l / group_sz, in_grp = l - grp * group_sz;
        const int rows_here = (tiles_r - grp * GROUP_M) < GROUP_M ? (tiles_r - grp * GROUP_M) : GROUP_M;
        const int tr = grp * GROUP_M + in_grp % rows_here, tc = in_grp / rows_here;
        m = m_first + (int64_t)(Epi::weight_rows ? tc : tr) * BT;
        n = (Epi::weight_rows ? tr : tc) * 256;
        we = bmap.row(n);
        wo = bmap.row(n + 32);
        we2 = we + w_mid;
        wo2 = wo + w_mid;
        xb = X + m * ld;
#pragma unroll
        for (int p = 0; p < XT; ++p) {
            int64_t r = p * 32 + rip;
            if (m + r >= M) r = M - 1 - m;                  // ragged last tile: re-read the last row, never stored
            x_off[p] = ((uint32_t)(r * ld) + x_chunk) * 2u;
        }
    };
    // request R of a slice into the stage at byte stg: 0..3 the weights' top halves (rows 0..63 of each wave's 128), then XQ of the
    // tokens' left halves, XQ of the right ones, 4 of the weights' bottom halves
    const uint32_t wave_lds = (uint32_t)wave * 1024u;
    auto request = [&](auto r_, int stg) {
        constexpr int R = r_;
        const uint32_t at = wave_lds + (uint32_t)stg;
        if constexpr (R < 4 || R >= 4 + 2 * XQ) {
            constexpr bool low = R >= 4;
            constexpr int q = (low ? R - 2 * XQ : R) & 3, p = (q & 1) + 4 * (q >> 1) + (low ? 2 : 0);
            dtl16c<p * 4096>(q & 1 ? (low ? wo2 : wo) : (low ? we2 : we), q >> 1 ? w_off1 : w_off0, at);
        } else {
            constexpr int q = (R - 4) % XQ, h = (R - 4) / XQ;       // XT 8: a wave's halves are 64 rows, two pieces each; 4: 32, one
            constexpr int p = XT == 8 ? (q & 1) + 4 * (q >> 1) + 2 * h : 2 * q + h;
            dtl16c<32768 + p * 4096>(xb, x_off[p], at);
        }
    };
    auto next_slice = [&] { we += BK; wo += BK; we2 += BK; wo2 += BK; xb += BK; };

    // ---- fragments. Weight rows are dealt to the 16 rows of instruction tiles 2p and 2p + 1 so that a lane's results of the
    // two are eight consecutive columns: lane (m, g) reads row 32p + 8 (m / 4) + 4 e + m % 4 of tile 2p + e ----
    const int m16 = lane & 15, g = lane >> 4;
    const uint32_t w_row = (uint32_t)(ww * 128 + 8 * (m16 >> 2) + (m16 & 3)) * 128, w_swz = w_swizzle(8 * (m16 >> 2) + (m16 & 3));
    const uint32_t x_row = (uint32_t)(256 + wt * 16 * XT + m16) * 128, x_swz = x_swizzle(m16);
    const uint32_t w_at[2] = {w_row + (((uint32_t)g ^ w_swz) << 4), w_row + (((uint32_t)(g + 4) ^ w_swz) << 4)};
    const uint32_t x_at[2] = {x_row + (((uint32_t)g ^ x_swz) << 4), x_row + (((uint32_t)(g + 4) ^ x_swz) << 4)};
    typedef bf16x8_t HalfW[2][4], HalfX[2][XQ];             // half an operand of a step: [32 of K][16 rows]
    auto read_w = [&](HalfW &d, auto f_, int half, int stg) {
        constexpr int f = f_;
        d[f >> 2][f & 3] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(
                                                            lds + stg + w_at[f >> 2] + (half * 64 + ((f & 3) >> 1) * 32 + (f & 1) * 4) * 128));
    };
    auto read_x = [&](HalfX &d, auto f_, int half, int stg) {
        constexpr int f = f_, k = f / XQ, j = f % XQ;
        if constexpr (f < 2 * XQ)
            d[k][j] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(lds + stg + x_at[k] + (half * XQ + j) * 16 * 128));
    };
    // One quadrant: 32 (16) instructions in the order that changes one operand at a time; behind the first 16, 8 (or 4) fragment
    // reads, and spread over all the NREQ_ requests from REQ0_ on.
#define SOL_QUAD(FIRST_, W_, X_, HW_, HX_, READ_, RD_, RHALF_, RSTG_, REQ0_, NREQ_, STG_)                                         \
    static_for<8 * XQ>([&](auto m_) {                                                                                          \
        constexpr int m = m_, kg = m / (4 * XQ), i = (m / XQ) & 3, j = (i & 1) ? XQ - 1 - m % XQ : m % XQ;                       \
        acc_mma<4 * (XT * (HW_ * 4 + i) + HX_ * XQ + j), FIRST_ && kg == 0>(W_[kg][i], X_[kg][j]);                              \
        if constexpr ((m & 1) == 0 && m < 16) READ_(RD_, std::integral_constant<int, m / 2>{}, RHALF_, RSTG_);                   \
        if constexpr (m % (8 * XQ / NREQ_) == 1) request(std::integral_constant<int, REQ0_ + m / (8 * XQ / NREQ_)>{}, STG_);     \
        __builtin_amdgcn_sched_barrier(0);                                                                                     \
    });
    // The youngest requests are those of the last 2 (ST - 1) half steps: what the half step after the barrier reads has landed. The
    // wave's own reads of the halves that will be overwritten are over (lgkmcnt).
#define SOL_SYNC                                                                                                               \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(IN_FLIGHT) : "memory", SOL_ACC_ALL);                                      \
    __builtin_amdgcn_sched_barrier(0);
    // One step of the slice in stage CS_, the next in NS_; XL_ holds its left tokens, XR_ is free. Requests: slice + ST into CS_.
#define SOL_STEP(FIRST_, XL_, XR_, CS_, NS_)                                                                                    \
    SOL_QUAD(FIRST_, wtop, XL_, 0, 0, read_x, XR_, 1, CS_, 0, 4, CS_)                                                           \
    SOL_QUAD(FIRST_, wtop, XR_, 0, 1, read_w, wbot, 1, CS_, 4, XQ, CS_)                                                         \
    SOL_SYNC                                                                                                                   \
    SOL_QUAD(FIRST_, wbot, XR_, 1, 1, read_w, wtop, 0, NS_, 4 + XQ, XQ, CS_)                                                    \
    SOL_QUAD(FIRST_, wbot, XL_, 1, 0, read_x, XR_, 0, NS_, 4 + 2 * XQ, 4, CS_)                                                  \
    SOL_SYNC
    // Two steps. WALK: the requests of a tile's last two are the first two slices of the next tile (of this one again after the last
    // tile: never used), so only a workgroup's first tile starts cold. Otherwise requests past the end are the last slice again.
#define SOL_PAIR(FIRST_, KT_)                                                                                                  \
    {                                                                                                                          \
        if constexpr (WALK) {                                                                                                  \
            if ((KT_) == KT - 2) tile_src(more ? lin + lin_step : lin, m0_next, n0_next);                                       \
            else next_slice();                                                                                                 \
            SOL_STEP(FIRST_, xa, xc, 0, SB)                                                                                     \
            next_slice();                                                                                                      \
            SOL_STEP(false, xc, xa, SB, 0)                                                                                      \
        } else {                                                                                                               \
            if ((KT_) + ST < KT) next_slice();                                                                                 \
            SOL_STEP(FIRST_, xa, xc, cs, ns)                                                                                    \
            cs = ns; ns = ns + SB == ST * SB ? 0 : ns + SB;                                                                    \
            if ((KT_) + 1 + ST < KT) next_slice();                                                                             \
            SOL_STEP(false, xc, xa, cs, ns)                                                                                     \
            cs = ns; ns = ns + SB == ST * SB ? 0 : ns + SB;                                                                    \
        }                                                                                                                      \
    }
    HalfW wtop, wbot;
    HalfX xa, xc;
    const int KT = K / BK;                                  // even (K is a multiple of 128)
    tile_src(lin, m0, n0);
    for (int s = 0; s < ST; ++s) {
        if (s > 0 && s < KT) next_slice();
        static_for<8 + XT>([&](auto r) { request(r, s * SB); });
    }
    SOL_SYNC
    static_for<8>([&](auto f) { read_w(wtop, f, 0, 0); read_x(xa, f, 0, 0); });
    SOL_SYNC
    [[maybe_unused]] int cs = 0, ns = SB;
    for (;;) {
        [[maybe_unused]] const bool more = WALK && lin + lin_step < band_end;
        SOL_PAIR(true, 0)
        for (int kt = 2; kt < KT; kt += 2) SOL_PAIR(false, kt)
        acc_settle();
        tile_epilogue<8, XT>(epi, [](auto i, auto t) {
            if constexpr (i == 0) asm volatile("" ::: SOL_ACC_ALL);                 // a token's piece of the epilogue
            return acc_read<4 * (XT * i + t)>();
        }, m0 + wt * 16 * XT, M, n0 + ww * 128, lane);
        if (!more) break;
        lin += lin_step; m0 = m0_next; n0 = n0_next;
    }
#undef SOL_PAIR
#undef SOL_STEP
#undef SOL_SYNC
#undef SOL_QUAD
    vm_wait<0>();                                           // no LDS-direct load outlives its workgroup
}

// ------------------------------------------------------------------------------------------------
// The same product with smaller tiles, for row counts whose 256 x 256 tiles would leave CUs idle; plan_gemm gives a CU at
// most one workgroup. G LDS groups of U slices each are filled by LDS-direct loads: while a group is multiplied from
// registers, the fragments of the next are read and the groups after those are on their way; one barrier per group. The last
// groups are unrolled: no request past the end, no wait that depends on a counter (either costs a tenth of a K of 2048).
// Bound: a CU's rate of L2 misses. 64 x 64 tiles take 0.18 us per slice of 16 KB (90 GB/s), 128 x 64 0.3, 128 x 128 0.5,
// whatever U and G are from (2, 4) to (1, 10); from the L2 alone the loads would reach 130 GB/s.
// 128 x 64 and 128 x 128 tiles have eight waves, two per SIMD, so that one's instructions cover the other's barrier and reads. Four
// waves (32 x 64, 64 x 64) -> eight, us: down of the 1B shape, 600 rows 35.6 -> 34.6, 1300 56.9 -> 52.7; of the 8B shape, 260 rows
// 62.5 -> 60.2, 700 111.8 -> 106.4; o 8B 700 32.7 -> 31.0; q/k/v 1B 400 rows 12.5 -> 11.8, 700 19.3 -> 17.8. With six or five
// slices in flight, or groups of two: no better, or worse. Heads of 128 in 128 x 128 tiles: level, four waves there.
// Against the kernel before this one (32x32x16 instructions, eight waves, 4-byte stores, requests past the end), us: q/k/v of the 1B
// shape 70 rows 14.1 -> 9.0, 400 rows 16.4 -> 11.8, of the 8B shape 36.0 -> 21.3 and 41.8 -> 32.9; down 1B 24.9 -> 22.8 (140 rows) and
// 42.7 -> 40.4 (1024), 8B 62.9 -> 60.2 (260); 1B o at 512, 1200 and 1300 rows, the one map that is not faster: 9.2 -> 9.3, 17.9 -> 18.1,
// 18.5 -> 18.6.
// The sums are k_gemm_mfma's (the same instructions over k), so the tile does not show in the results.
// ------------------------------------------------------------------------------------------------
template <int BT, int BW, int WT, int WW, int U, int G, class Epi>
__global__ void __launch_bounds__((BT / WT) * (BW / WW) * 64, 1)
k_gemm_tile(const bf16_t *__restrict__ X, BMap bmap, int64_t m_first, int64_t M, int K, int tiles_m, int tiles_n, Epi epi)
{
    constexpr int NWT = BT / WT, NT = NWT * (BW / WW) * 64;
    constexpr int TW = WW / 16, TX = WT / 16;
    constexpr int RPP = NT / 8, WP = BW / RPP, XP = BT / RPP;      // rows per pass of the workgroup's loads, passes
    constexpr uint32_t SB = (BW + BT) * 128, GB = U * SB;          // bytes of a slice, of a group
    constexpr int PER = U * (WP + XP);                             // a wave's requests per group
    static_assert(BW % RPP == 0 && BT % RPP == 0 && RPP % 16 == 0 && WW % 32 == 0, "tile / thread mismatch");
    static_assert(G >= 2 && PER * (G - 1) < 64 && GB * G <= 163840, "vmcnt counts the loads in flight; the LDS holds them");
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ww = wave / NWT, wt = wave - ww * NWT;
    // XCD-aware tile mapping as in k_gemm_mfma
    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= n_tiles) return;
    const int group_sz = GROUP_M * tiles_n, grp = lin / group_sz, in_grp = lin - grp * group_sz;
    const int rows_here = (tiles_m - grp * GROUP_M) < GROUP_M ? (tiles_m - grp * GROUP_M) : GROUP_M;
    const int64_t m0 = m_first + (int64_t)(grp * GROUP_M + in_grp % rows_here) * BT;
    const int n0 = (in_grp / rows_here) * BW;

    const int64_t ld = bmap.ld;                            // of weights and tokens alike
    const int chunk = tid & 7, rip = tid >> 3;
    const bf16_t *x_base = X + m0 * ld;
    uint32_t x_off[XP];
#pragma unroll
    for (int p = 0; p < XP; ++p) {
        int64_t r = p * RPP + rip;
        if (m0 + r >= M) r = M - 1 - m0;                   // ragged last tile: re-read the last row, never stored
        x_off[p] = ((uint32_t)(r * ld) + (uint32_t)((chunk ^ x_swizzle(rip)) * 8)) * 2u;
    }
    const bf16_t *w_base[WP];
    uint32_t w_off[RPP % 32 ? 2 : 1];                      // (the weights' swizzle repeats after 32 rows)
#pragma unroll
    for (int p = 0; p < WP; ++p) w_base[p] = bmap.row(n0 + p * RPP + wave * 8);   // a wave's 8 rows lie in one weight matrix
#pragma unroll
    for (int p = 0; p < (RPP % 32 ? 2 : 1); ++p)
        w_off[p] = ((uint32_t)(rip & 7) * (uint32_t)ld + (uint32_t)((chunk ^ w_swizzle(p * RPP + rip)) * 8)) * 2u;

    const int KT = K / BK, KG = KT / U;                    // KT is even (K is a multiple of 128)
    static_assert(U == 1 || U == 2, "whole groups");
    // request R (of PER) of group kg into the group at byte `at`
    auto request = [&](auto r_, int kg, uint32_t at) {
        constexpr int R = r_, u = R / (WP + XP), p = R % (WP + XP);
        const int koff = (kg * U + u) * BK;
        const uint32_t to = at + (uint32_t)wave * 1024u;
        if constexpr (p < WP) dtl16c<u * (int)SB + p * RPP * 128>(w_base[p] + koff, w_off[RPP % 32 ? p & 1 : 0], to);
        else dtl16c<u * (int)SB + (BW + (p - WP) * RPP) * 128>(x_base + koff, x_off[p - WP], to);
    };
    const int m16 = lane & 15, g = lane >> 4;
    const uint32_t w_row = (uint32_t)(ww * WW + 8 * (m16 >> 2) + (m16 & 3)) * 128, x_row = (uint32_t)(BW + wt * WT + m16) * 128;
    const uint32_t w_swz = w_swizzle(8 * (m16 >> 2) + (m16 & 3)), x_swz = x_swizzle(m16);
    struct Frags { bf16x8_t w[2 * U][TW], x[2 * U][TX]; };
    constexpr int NR = 2 * U * (TW + TX), NM = 2 * U * TW * TX;    // fragment reads, matrix instructions of a group
    auto fragment = [&](auto r_, Frags &f, uint32_t at) {
        constexpr int R = r_, k = R / (TW + TX), i = R % (TW + TX);
        const unsigned char *const st = lds + at + (k >> 1) * SB;
        const uint32_t c = (uint32_t)(g + 4 * (k & 1));
        if constexpr (i < TW)
            f.w[k][i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(
                                                         st + w_row + ((c ^ w_swz) << 4) + ((i >> 1) * 32 + (i & 1) * 4) * 128));
        else f.x[k][i - TW] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(st + x_row + ((c ^ x_swz) << 4) + (i - TW) * 16 * 128));
    };
    f32x4_t acc[TW][TX];
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int j = 0; j < TX; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // A group: its matrix instructions, behind the first of them the reads of the next group (RPM each), then the requests.
    constexpr int RPM = 2 * NR > NM ? (2 * NR + NM - 1) / NM : 1, QM = (NR + RPM - 1) / RPM;
    constexpr int QPM = NM > QM ? (PER + NM - QM - 1) / (NM - QM) : PER;
    auto group = [&](auto more_, const Frags &f, Frags &next, uint32_t at_next, int kg_load, uint32_t at_load) {
        static_for<NM>([&](auto m_) {
            constexpr int m = m_, k = m / (TW * TX), i = m / TX % TW, j = (i & 1) ? TX - 1 - m % TX : m % TX;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[k][i], f.x[k][j], acc[i][j], 0, 0, 0);
            static_for<RPM>([&](auto r) { if constexpr (m * RPM + r < NR) fragment(std::integral_constant<int, m * RPM + r>{}, next, at_next); });
            static_for<QPM>([&](auto r) {
                constexpr int q = NM > QM ? (m - QM) * QPM + r : (m == NM - 1 ? (int)r : PER);
                if constexpr (more_ && q >= 0 && q < PER) request(std::integral_constant<int, q>{}, kg_load, at_load);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // all but the N youngest groups that this wave requested have landed and its fragment reads are over; so for all waves
#define SOL_TILE_SYNC(N) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PER * ((N) > 0 ? (N) : 0)) : "memory")
    for (int s = 0; s < G; ++s)
        if (s < KG) static_for<PER>([&](auto r) { request(r, s, s * GB); });
    Frags f[2];
    uint32_t cur = 0, nxt = GB;                            // groups kg and kg + 1
    auto turn = [&] { cur = nxt; nxt = nxt + GB == G * GB ? 0 : nxt + GB; };
    if (KG >= G) {
        SOL_TILE_SYNC(G - 1);
        static_for<NR>([&](auto r) { fragment(r, f[0], 0); });
        int kg = 0;
        for (; kg + G + 1 < KG; kg += 2) {
            SOL_TILE_SYNC(G - 2);                          // group kg + 1 is there, group kg is read out
            group(std::true_type{}, f[0], f[1], nxt, kg + G, cur);
            turn();
            SOL_TILE_SYNC(G - 2);
            group(std::true_type{}, f[1], f[0], nxt, kg + 1 + G, cur);
            turn();
        }
        // the last G or G + 1 groups, nothing left to request but the one group of the latter
        auto tail = [&](auto n_) {
            constexpr int N = n_;
            static_for<N>([&](auto i_) {
                constexpr int i = i_;
                SOL_TILE_SYNC(N - 2 - i < G - 2 ? N - 2 - i : G - 2);
                group(std::integral_constant<bool, (i + G < N)>{}, f[i & 1], f[1 - (i & 1)], nxt, kg + i + G, cur);
                turn();
            });
        };
        if (KG - kg == G) tail(std::integral_constant<int, G>{});
        else tail(std::integral_constant<int, G + 1>{});
    } else {                                               // short K: all of it is in the LDS
        SOL_TILE_SYNC(0);
        for (int kg = 0; kg < KG; ++kg) {
            static_for<NR>([&](auto r) { fragment(r, f[0], (uint32_t)kg * GB); });
            group(std::false_type{}, f[0], f[1], (uint32_t)kg * GB, 0, 0);
        }
    }
#undef SOL_TILE_SYNC
    tile_epilogue<TW, TX>(epi, [&](auto i, auto t) { return acc[i][t]; }, m0 + wt * WT, M, n0 + ww * WW, lane);
}

// ------------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------------
// compute units of the current device (one persistent workgroup each), 0 if the query fails
int device_cus()
{
    static int cus[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (!cus[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cus[dev] = n;
    }
    return cus[dev];
}

// M tokens [M][K] times the weight rows of bmap, 256 x 256 tiles: one workgroup per CU (CUs / 8 per XCD) walks its share
template <class Epi>
static bool launch_mfma(const bf16_t *X, const BMap &bmap, int64_t M, int Nv, int K, const Epi &epi, hipStream_t st)
{
    if (M <= 0) return true;
    if (Nv % 256 || K % (2 * BK) || K < 2 * BK || bmap.ld != K || (bmap.mode == 1 && bmap.half != 32)) return false;
    constexpr size_t lds = 131072;
    const int tiles_x = (int)((M + 255) / 256), tiles_w = Nv / 256;
    const int per_xcd = (tiles_x * tiles_w + 7) / 8, wg_xcd = device_cus() / 8;
    auto kern = k_gemm_mfma<8, 2, Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess) return false;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3((wg_xcd > 0 && wg_xcd < per_xcd ? wg_xcd : per_xcd) * 8), dim3(256), lds, st, X, bmap, (int64_t)0, M, K,
                       Epi::weight_rows ? tiles_w : tiles_x, Epi::weight_rows ? tiles_x : tiles_w, epi);
    return true;
}

constexpr int SOL_WN = 128;                                // vocabulary entries of a partial sum of the head

// How the rows of a product are dealt to tiles. A grid of at most one smaller tile per CU takes, in rounds of one 256 x 256 tile on every
// CU (183 us at K = 8192; what a grid takes hardly depends on how many CUs it fills): 64 x 64 0.14, 128 x 64 0.22, 128 x 128 0.35,
// 128 x 256 0.56 (25.6, 40, 64 and 102 us: down projection of the 1B shape, 512, 1024, 2048 and 4096 rows). So a call takes the smallest
// tile of which every CU gets at most one; with more rows than that, whole rounds of 256 x 256 tiles (or whole tile rows) first and the
// smaller tile for the rest, where that ends sooner than a last round that is nearly empty. Any smaller tile ends sooner than a round and
// later than none, and rows that fit one tile take the smallest that they fit: no more than that is asked here (REST: with costs of 0.1 to
// 0.7 in its place, one for each tile, every plan of 1 to 20000 rows and 256 to 32768 columns stays the same). The q/k/v map with
// heads of 128 has 64 x 128 tiles in place of both 64-column ones (one per CU as well). The tile does not show in the results.
struct GemmPlan {
    int64_t big;                 // rows [0, big) in 256 x 256 tiles (all rows, or a multiple of 256)
    int small;                   // the others: 0 = 64 x 64, 1 = 128 x 64, 2 = 128 x 128, 3 = 128 x 256
};
// the smallest tile of which every CU gets at most one, -1 if there is none
static int small_tile(int64_t rows, int N, int cus)
{
    static const int bm[4] = {64, 128, 128, 128}, bn[4] = {64, 64, 128, 256};
    for (int cfg = 0; cfg < 4; ++cfg)
        if ((rows + bm[cfg] - 1) / bm[cfg] * (N / bn[cfg]) <= cus) return cfg;
    return -1;
}
static GemmPlan plan_gemm(int64_t M, int N)
{
    const int cus = device_cus() > 0 ? device_cus() : 256;
    const int64_t tn = N / 256, whole = M / 256;           // tile columns, whole tile rows
    const double REST = 0.5;                               // rounds
    GemmPlan best{M, 0};
    double best_cost = (double)(((M + 255) / 256 * tn + cus - 1) / cus);
    const int64_t rounds = whole * tn / cus;               // whole rounds of whole tiles
    const int64_t cand[3] = {0, rounds > 0 ? rounds * cus / tn : 0, whole};
    for (int64_t r : cand) {
        if (r * 256 >= M) continue;
        const int cfg = small_tile(M - r * 256, N, cus);
        const double c = (double)((r * tn + cus - 1) / cus) + REST;
        if (cfg >= 0 && c < best_cost) { best_cost = c; best = GemmPlan{r * 256, cfg}; }
    }
    return best;
}

template <int BT, int BW, int WT, int WW, int U, int G, class Epi>
static bool launch_tile(const bf16_t *X, const BMap &bmap, int64_t m_first, int64_t M, int Nv, int K, const Epi &epi, hipStream_t st)
{
    constexpr size_t lds = (size_t)U * G * (BW + BT) * 128;
    auto kern = k_gemm_tile<BT, BW, WT, WW, U, G, Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess) return false;
        attr_done = true;
    }
    const int tiles_m = (int)((M - m_first + BT - 1) / BT), tiles_n = Nv / BW, per_xcd = (tiles_m * tiles_n + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3((BT / WT) * (BW / WW) * 64), lds, st, X, bmap, m_first, M, K, tiles_m, tiles_n, epi);
    return true;
}
// 128 tokens x 256 weight rows
template <class Epi>
static bool launch_half(const bf16_t *X, const BMap &bmap, int64_t m_first, int64_t M, int Nv, int K, const Epi &epi, hipStream_t st)
{
    constexpr size_t lds = 3 * (256 + 128) * 128;
    auto kern = k_gemm_mfma<4, 3, Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess) return false;
        attr_done = true;
    }
    const int tiles_m = (int)((M - m_first + 127) / 128), tiles_n = Nv / 256, per_xcd = (tiles_m * tiles_n + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256), lds, st, X, bmap, m_first, M, K, tiles_m, tiles_n, epi);
    return true;
}

// Rows [m_first, M) in tiles of configuration cfg (GemmPlan::small). WN: columns an epilogue needs in one wave tile.
template <int WN, class Epi>
static bool launch_small(int cfg, const bf16_t *X, const BMap &bmap, int64_t m_first, int64_t M, int Nv, int K, const Epi &epi, hipStream_t st)
{
    if (Nv % 256 || K % (2 * BK) || K < 2 * BK || bmap.ld != K || (bmap.mode == 1 && bmap.half != 32)) return false;
    if (cfg == 3) return launch_half(X, bmap, m_first, M, Nv, K, epi, st);
    if constexpr (WN == 128) {                               // a head of 128 in one wave tile: no 64-column tiles
        if (cfg <= 1) return launch_tile<64, 128, 16, 128, 1, 4>(X, bmap, m_first, M, Nv, K, epi, st);
        return launch_tile<128, 128, 32, 128, 1, 4>(X, bmap, m_first, M, Nv, K, epi, st);
    } else {
        if (cfg == 0) {
            if constexpr (WN == 32) return launch_tile<64, 64, 32, 32, 2, 4>(X, bmap, m_first, M, Nv, K, epi, st);
            else return launch_tile<64, 64, 16, 64, 2, 4>(X, bmap, m_first, M, Nv, K, epi, st);
        }
        if (cfg == 1) {
            if constexpr (WN == 32) return launch_tile<128, 64, 32, 32, 1, 4>(X, bmap, m_first, M, Nv, K, epi, st);
            else return launch_tile<128, 64, 16, 64, 1, 4>(X, bmap, m_first, M, Nv, K, epi, st);
        }
        return launch_tile<128, 128, 32, 64, 1, 4>(X, bmap, m_first, M, Nv, K, epi, st);
    }
}

template <int DHT>
static bool launch_qkv_rope(const bf16_t *h, const BMap &bm, bf16_t *q, bf16_t *kc, bf16_t *vc, const float2 *rope,
                            const int32_t *pos0, int n_seq, int T, int L_max, int crows, int Hq, int Hkv, int d, int *flags, hipStream_t st)
{
    const int64_t M = (int64_t)n_seq * T;
    const int N = (Hq + 2 * Hkv) * DHT;
    if (M >= (1ll << 31)) return false;
    const GemmPlan plan = plan_gemm(M, N);
    const EpiQkvRope8<DHT> epi{q, kc, vc, rope, pos0, T, L_max, crows, Hq, Hkv, flags};
    if (plan.big > 0 && !launch_mfma(h, bm, plan.big, N, d, epi, st)) return false;
    return plan.big == M || launch_small<DHT>(plan.small, h, bm, plan.big, M, N, d, epi, st);
}

bool launch_gemm_qkv_rope(const void *h, const void *wq, const void *wk, const void *wv, void *q, void *kc, void *vc,
                          const float2 *rope, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh,
                          int d, int *flags, hipStream_t st, int cache_rows)
{
    const int nq = Hq * dh, nkv = Hkv * dh;
    if ((dh != 64 && dh != 128) || nq % 256 || nkv % 256) return false;      // heads must not straddle wave tiles
    if ((int64_t)n_seq * T <= 0) return true;
    if (d % (2 * BK) || d < 2 * BK) return false;
    const int crows = cache_rows > 0 ? cache_rows : L_max;                    // rows of a (sequence, KV head) in the caches
    BMap bm{};
    bm.base[0] = (const bf16_t *)wq; bm.base[1] = (const bf16_t *)wk; bm.base[2] = (const bf16_t *)wv;
    bm.seg_end[0] = nq; bm.seg_end[1] = nq + nkv; bm.seg_end[2] = nq + 2 * nkv;
    bm.mode = 0; bm.half = 0; bm.ld = d;
    auto *const go = dh == 64 ? launch_qkv_rope<64> : launch_qkv_rope<128>;
    return go((const bf16_t *)h, bm, (bf16_t *)q, (bf16_t *)kc, (bf16_t *)vc, rope, pos0, n_seq, T, L_max, crows, Hq, Hkv, d,
              flags, st);
}

static BMap plain_map(const void *w, int N, int K)
{
    BMap bm{};
    bm.base[0] = (const bf16_t *)w; bm.seg_end[0] = bm.seg_end[1] = bm.seg_end[2] = N; bm.mode = 0; bm.ld = K;
    return bm;
}

template <int WN, class Epi>
static bool launch_planned(const void *a, const BMap &bm, int64_t M, int N, int K, const Epi &epi, hipStream_t st)
{
    if (M <= 0) return true;
    if (N % 256 || K % (2 * BK) || K < 2 * BK) return false;
    const GemmPlan plan = plan_gemm(M, N);
    if (plan.big > 0 && !launch_mfma((const bf16_t *)a, bm, plan.big, N, K, epi, st)) return false;
    return plan.big == M || launch_small<WN>(plan.small, (const bf16_t *)a, bm, plan.big, M, N, K, epi, st);
}

bool launch_gemm_resid_f32(const void *a, const void *w, const void *resid, float *out, int64_t M, int N, int K,
                           hipStream_t st)
{
    return launch_planned<32>(a, plain_map(w, N, K), M, N, K, EpiResidF32x8{(const bf16_t *)resid, out, N}, st);
}

bool launch_gemm_gateup_silu(const void *h, const void *wg, const void *wu, void *a, int64_t M, int dff, int d,
                             hipStream_t st)
{
    if (M <= 0) return true;
    if (dff % 64) return false;
    BMap bm{};
    bm.base[0] = (const bf16_t *)wg; bm.base[1] = (const bf16_t *)wu; bm.mode = 1; bm.ld = d;
    bm.half = 32;                                             // gate / up interleaved in pieces of 32 columns
    return launch_planned<64>(h, bm, M, 2 * dff, d, EpiSiluMul8{(bf16_t *)a, dff}, st);
}

bool launch_gemm_resid_out(const void *a, const void *w, const float *x2, void *out, int64_t M, int N, int K,
                           hipStream_t st)
{
    return launch_planned<32>(a, plain_map(w, N, K), M, N, K, EpiResidOut8{x2, (bf16_t *)out, N}, st);
}

bool launch_gemm_f32(const void *a, const void *w, float *C, int64_t ldc, int64_t M, int N, int K, hipStream_t st)
{
    return launch_planned<32>(a, plain_map(w, N, K), M, N, K, EpiStoreF32x8{C, ldc}, st);
}

static int64_t nll_pad_rows(int64_t M) { return (M + 255) / 256 * 256; }
int64_t gemm_nll_hf_rows(int64_t M) { return nll_pad_rows(M); }
size_t gemm_nll_scratch_bytes(int64_t M, int V) { return (size_t)nll_pad_rows(M) * ((size_t)(V / SOL_WN) * sizeof(float2) + 8); }

// nll[r] = logsumexp(hf[r] . lm_head^T) - (hf[r] . lm_head[target(r)]) without materialising the logits.
// hf: [gemm_nll_hf_rows(M)][K], the first M rows filled (the padding rows are cleared here); scratch:
// gemm_nll_scratch_bytes(M, V) bytes. Returns false (nothing launched) if the shape does not tile.
bool launch_gemm_nll(void *hf, const void *lm_head, const int32_t *targets, int G, int T, bool broadcast_g,
                     float *nll, void *scratch, int64_t M, int V, int K, int *flags, hipStream_t st)
{
    if (M <= 0) return true;
    // A decode step's few tokens take tiles of 32 or 64 tokens: with 256 columns of padding the matrix cores need as long as HBM. The
    // partial results are those of the large tiles bit for bit. 128256 entries of 2048, all four launches: 1 to 64 tokens 134 us (120
    // of it the product, 4.4 TB/s; two workgroups per CU with half of the stages: 137), 100 tokens (256 columns) 147.
    const int64_t Mp = M <= 32 ? 32 : M <= 64 ? 64 : nll_pad_rows(M);
    if (V % 256 || K % (2 * BK) || K < 2 * BK || Mp >= (1ll << 31)) return false;
    const int n_wt = V / SOL_WN;
    float2 *part = (float2 *)scratch;
    float *tgt_logit = (float *)(part + (size_t)Mp * n_wt);
    int32_t *row_tgt = (int32_t *)(tgt_logit + Mp);
    const int64_t n_pad = (Mp - M) * K / 8, row_wgs = (M + 255) / 256, pad_wgs = (n_pad + 255) / 256;
    hipLaunchKernelGGL(k_row_targets, dim3((unsigned)(row_wgs > pad_wgs ? row_wgs : pad_wgs)), dim3(256), 0, st, targets, M, G, T,
                       broadcast_g ? 1 : 0, V, row_tgt, flags, (u32x4_t *)((bf16_t *)hf + M * K), n_pad);
    const BMap bm = plain_map(lm_head, V, K);
    const EpiNllCols8 epi{part, Mp};
    const bf16_t *const x = (const bf16_t *)hf;
    if (!(Mp == 32 ? launch_tile<32, 256, 32, 128, 1, 4>(x, bm, 0, Mp, V, K, epi, st)
          : Mp == 64 ? launch_tile<64, 256, 32, 128, 1, 4>(x, bm, 0, Mp, V, K, epi, st)
                     : launch_mfma(x, bm, Mp, V, K, epi, st)))
        return false;
    hipLaunchKernelGGL(k_target_logit, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, st, (const bf16_t *)hf,
                       (const bf16_t *)lm_head, row_tgt, M, K, tgt_logit);
    hipLaunchKernelGGL(k_nll_finish_cols, dim3((unsigned)((M + 31) / 32)), dim3(1024), 0, st, part, tgt_logit, n_wt,
                       M, Mp, nll);
    return true;
}

// =================================================================================================
// Skinny GEMM for the decode step: out[M][Nv] = x[M][K] * Wv[Nv][K]^T with M <= 64 tokens.
// HBM-bound: every weight byte is read exactly once, by exactly one wave. A wave owns 32 weight
// rows (they are the MFMA's "A" rows) and streams them straight from global memory in 128-byte
// pieces (lane (r, h) takes the 64 contiguous bytes of half h of row r, so every fetched line is
// fully used); the activations are the "B" operand, staged per workgroup in LDS in K chunks of 512.
// Since the same k-to-lane assignment is used for A and B the MFMA sum is exact. The K range may be
// split over gridDim.y workgroups; partial sums go to fp32 partial[split][M][Nv] and are folded by
// the consumer kernel in split order (fixed split count per shape => deterministic).
// =================================================================================================
constexpr int SK_KC = 512;                 // K chunk staged in LDS
constexpr int SK_XROW = SK_KC * 2 + 16;    // padded LDS row of activations (bytes): rows shift 4 banks

template <int MT>                           // MT tiles of 32 tokens (1: M <= 32, 2: M <= 64)
__global__ void __launch_bounds__(256)
k_gemm_skinny(const bf16_t *__restrict__ x, int64_t ldx, BMap bmap, int M, int Nv, int K, int k_per_split,
              float *__restrict__ partial, int xrow)
{
    extern __shared__ __align__(16) unsigned char xs[];      // [MT*32][xrow]: xrow = padded bytes of a staged row (the
                                                             // chunk is no longer than a split: short splits leave room
                                                             // for more workgroups per CU)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (blockIdx.x * 4 + wave) * 32;
    const int split = blockIdx.y;
    const int k_begin = split * k_per_split;
    const int k_end = (k_begin + k_per_split < K) ? k_begin + k_per_split : K;
    const int r = lane & 31, h = lane >> 5;
    const bool live = n0 < Nv;                                // whole wave
    int nrow = n0 + r;
    if (nrow >= Nv) nrow = Nv - 1;
    const bf16_t *wrow = bmap.row(nrow) + h * 32;             // this lane's 64-byte half of each 128-byte piece
    floatx16_t acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

    // The split's K range is walked in 64-wide blocks, UK blocks per batch, two batches per LDS chunk of
    // activations. Weight loads run one batch ahead of the MFMAs (two register sets), and the first batch
    // of a chunk is already in flight while the chunk's activations are staged, so a workgroup pays the
    // global-memory latency about once instead of once per batch.
    constexpr int UK = 4;                                             // 64-wide K blocks per batch
    static_assert(SK_KC == 2 * UK * 64, "two batches per staged chunk");
    const int nblk = (k_end - k_begin) / 64;
    u32x4_t wa0[UK][4], wa1[UK][4];
#define SOL_SK_LOADW(WA, B0_)                                                                              \
    _Pragma("unroll") for (int u = 0; u < UK; ++u) {                                                       \
        const int blk_ = ((B0_) + u < nblk) ? (B0_) + u : nblk - 1;     /* ragged tail: re-read, not used */ \
        _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                      \
            WA[u][j] = *reinterpret_cast<const u32x4_t *>(wrow + k_begin + blk_ * 64 + j * 8);             \
    }
#define SOL_SK_MMA(WA, B0_, KOFF_)          /* KOFF_: offset of the batch inside the staged chunk */          \
    _Pragma("unroll") for (int u = 0; u < UK; ++u) {                                                       \
        if ((B0_) + u < nblk) {                                                                            \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                \
                const bf16x8_t af = __builtin_bit_cast(bf16x8_t, WA[u][j]);                                \
                _Pragma("unroll") for (int t = 0; t < MT; ++t) {                                           \
                    const unsigned char *xp = xs + (t * 32 + r) * xrow + ((KOFF_) + u * 64 + h * 32 + j * 8) * 2; \
                    const bf16x8_t bfr = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(xp)); \
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc[t], 0, 0, 0);            \
                }                                                                                          \
            }                                                                                              \
        }                                                                                                  \
    }
    if (live) SOL_SK_LOADW(wa0, 0);
    for (int b0 = 0; b0 < nblk; b0 += 2 * UK) {
        const int kc = k_begin + b0 * 64;
        const int kw = (k_end - kc < SK_KC) ? (k_end - kc) : SK_KC;   // multiple of 64
        __syncthreads();                                              // previous chunk fully consumed
        // stage x[0..MT*32)[kc .. kc+kw) into LDS, 16 bytes per thread per step (rows >= M: zeros)
        const int pieces = kw / 8;
        for (int idx = tid; idx < MT * 32 * pieces; idx += 256) {
            const int m = idx / pieces, p = idx - m * pieces;
            u32x4_t v = {0u, 0u, 0u, 0u};
            if (m < M) v = *reinterpret_cast<const u32x4_t *>(x + (int64_t)m * ldx + kc + p * 8);
            *reinterpret_cast<u32x4_t *>(xs + m * xrow + p * 16) = v;
        }
        __syncthreads();
        if (live) {
            if (b0 + UK < nblk) SOL_SK_LOADW(wa1, b0 + UK);
            SOL_SK_MMA(wa0, b0, 0);
            if (b0 + 2 * UK < nblk) SOL_SK_LOADW(wa0, b0 + 2 * UK);
            if (b0 + UK < nblk) SOL_SK_MMA(wa1, b0 + UK, UK * 64);
        }
    }
#undef SOL_SK_LOADW
#undef SOL_SK_MMA
    if (!live) return;
    // acc[t][i]: weight row n0 + 8*(i/4) + 4*h + (i%4), token t*32 + r
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int m = t * 32 + r;
        if (m < M) {
            float *dst = partial + ((int64_t)split * M + m) * Nv + n0 + 4 * h;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (n0 + 8 * g + 4 * h + 3 < Nv) {
                    const float4 v = make_float4(acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]);
                    *reinterpret_cast<float4 *>(dst + 8 * g) = v;
                }
            }
        }
    }
}

// Number of K splits for the skinny kernel: enough waves to cover the chip, partial-sum traffic kept
// below about a quarter of the weight traffic.
int skinny_splits(int M, int Nv, int K)
{
    const int tiles = (Nv + 31) / 32;
    int want = (2048 + tiles - 1) / tiles;
    int cap = K / (4 * (M > 0 ? M : 1));
    if (cap < 1) cap = 1;
    int s = want < cap ? want : cap;
    if (s < 1) s = 1;
    while (s > 1 && (K / 64) % s != 0) --s;                 // every split gets a whole number of 64-wide blocks
    return s;
}

static bool launch_skinny(const bf16_t *x, int64_t ldx, const BMap &bm, int M, int Nv, int K, float *partial, int nsplit,
                          hipStream_t st)
{
    if (M <= 0) return true;
    if (M > 64 || Nv % 4 || K % 64) return false;
    const int k_per_split = K / nsplit;
    if (k_per_split % 64) return false;
    const dim3 grid((Nv + 127) / 128, nsplit);
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(k_gemm_skinny<2>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)((size_t)64 * SK_XROW)) != hipSuccess) return false;
        attr_done = true;
    }
    const int xrow = (k_per_split < SK_KC ? k_per_split : SK_KC) * 2 + 16;
    if (M <= 32)
        hipLaunchKernelGGL((k_gemm_skinny<1>), grid, dim3(256), (size_t)32 * xrow, st, x, ldx, bm, M, Nv, K, k_per_split, partial, xrow);
    else
        hipLaunchKernelGGL((k_gemm_skinny<2>), grid, dim3(256), (size_t)64 * xrow, st, x, ldx, bm, M, Nv, K, k_per_split, partial, xrow);
    return true;
}

// partial[nsplit][M][N] = x * [w0; w1; w2]^T  (rows of up to three stacked weight matrices)
bool launch_gemm_skinny(const void *x, int64_t ldx, const void *w0, int n0, const void *w1, int n1, const void *w2,
                        int n2, int M, int K, float *partial, int nsplit, hipStream_t st)
{
    BMap bm{};
    bm.base[0] = (const bf16_t *)w0; bm.base[1] = (const bf16_t *)w1; bm.base[2] = (const bf16_t *)w2;
    bm.seg_end[0] = n0; bm.seg_end[1] = n0 + n1; bm.seg_end[2] = n0 + n1 + n2;
    bm.mode = 0; bm.half = 0; bm.ld = K;
    return launch_skinny((const bf16_t *)x, ldx, bm, M, n0 + n1 + n2, K, partial, nsplit, st);
}

}  // namespace sol
