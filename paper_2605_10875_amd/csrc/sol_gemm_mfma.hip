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

#include <type_traits>
#include <utility>

namespace sol {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // native 16-byte vector (stays in registers)
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 64;               // K step (bf16 elements); one LDS row = 128 bytes = 8 chunks of 16 B
constexpr int GROUP_M = 4;           // tile rows walked together by an XCD: its 32 CUs then hold 4 x 8 tiles (measured on the
                                     // 16 x 2048-token stack: 2, 4 within 1 %; 8: 2 - 4 % slower; 16: 4 - 8 % slower)
// LDS has 64 banks of 4 bytes (256 B per clock): two 128-byte rows share one bank row, so the
// 16-byte chunk index is XOR-ed with bits 1..3 of the row. Measured SQ_LDS_BANK_CONFLICT drops 32x
// against swizzling with bits 0..2.
#ifndef SOL_SWZ
#define SOL_SWZ(r) (((r) >> 1) & 7)
#endif

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

// ------------------------------------------------------------------------------------------------
// Epilogues work on the accumulator layout of v_mfma_f32_32x32x16 directly: for one (row-tile, register
// pair) a lane holds, for two consecutive rows, the TN values at columns  c + 32*j  (c = lane % 32) of
// the wave tile. An epilogue has two halves so that the kernel can issue every global read of a 32-row
// tile before the first store (the compiler must assume that stores alias later loads):
//   preload(row0, row1, ok0, ok1, vcol0, c, aux)      reads what the row pair needs from memory into aux
//                                                     (row0 / row1 clamped to existing rows: no branches)
//   rows2(row0, ok0, ok1, vcol0, c, v0, v1, aux)      combines and stores
// row0 / row0 + 1 are the global rows, ok0 / ok1 say whether they exist (every lane still runs the code:
// bf16 outputs exchange values between neighbouring lanes), vcol0 is the wave tile's first virtual column.
// ------------------------------------------------------------------------------------------------

// Two rows of bf16 outputs at column c: neighbouring lanes pair up so that every lane stores one 4-byte
// pair: even lanes (row0, columns c, c+1), odd lanes (row1, columns c-1, c).
__device__ __forceinline__ void store_bf16_rows2(bf16_t *p0, bf16_t *p1, bool ok0, bool ok1, int c, float x0, float x1)
{
    const float t0 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x0), 0xB1, 0xF, 0xF, false));
    const float t1 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x1), 0xB1, 0xF, 0xF, false));
    const bool even = (c & 1) == 0;
    const uint32_t pk = even ? pack_bf16x2(x0, t0) : pack_bf16x2(t1, x1);
    bf16_t *dst = even ? p0 + c : p1 + (c - 1);
    if (even ? ok0 : ok1) *reinterpret_cast<uint32_t *>(dst) = pk;
}

struct NoAux {};

struct EpiStoreF32 {
    float *C; int64_t ldc;
    template <int TN> using Aux = NoAux;
    template <int TN> __device__ __forceinline__ void preload0(int64_t, int64_t, NoAux &) const {}
    template <int TN> __device__ __forceinline__ void preload(int64_t, int64_t, bool, bool, int, int, NoAux &) const {}
    template <int TN>
    __device__ __forceinline__ void rows2(int64_t row0, bool ok0, bool ok1, int vcol0, int c, const float (&v0)[TN],
                                          const float (&v1)[TN], const NoAux &) const
    {
        float *p0 = C + row0 * ldc + vcol0 + c, *p1 = p0 + ldc;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (ok0) p0[32 * j] = v0[j];
            if (ok1) p1[32 * j] = v1[j];
        }
    }
};

template <int TN> struct AuxRows { float a0[TN], a1[TN]; };

// x2 = resid + acc  (fp32 out), resid in bf16
struct EpiResidF32 {
    const bf16_t *resid; float *out; int64_t ld;
    template <int TN> using Aux = AuxRows<TN>;
    template <int TN> __device__ __forceinline__ void preload0(int64_t, int64_t, AuxRows<TN> &) const {}
    template <int TN>
    __device__ __forceinline__ void preload(int64_t row0, int64_t row1, bool, bool, int vcol0, int c, AuxRows<TN> &x) const
    {
        const int64_t o0 = row0 * ld + vcol0 + c, o1 = row1 * ld + vcol0 + c;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            x.a0[j] = bf16_to_f32(resid[o0 + 32 * j]);
            x.a1[j] = bf16_to_f32(resid[o1 + 32 * j]);
        }
    }
    template <int TN>
    __device__ __forceinline__ void rows2(int64_t row0, bool ok0, bool ok1, int vcol0, int c, const float (&v0)[TN],
                                          const float (&v1)[TN], const AuxRows<TN> &x) const
    {
        const int64_t o0 = row0 * ld + vcol0 + c, o1 = o0 + ld;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (ok0) out[o0 + 32 * j] = v0[j] + x.a0[j];
            if (ok1) out[o1 + 32 * j] = v1[j] + x.a1[j];
        }
    }
};

// out = bf16(x2 + acc), x2 in fp32
struct EpiResidOut {
    const float *x2; bf16_t *out; int64_t ld;
    template <int TN> using Aux = AuxRows<TN>;
    template <int TN> __device__ __forceinline__ void preload0(int64_t, int64_t, AuxRows<TN> &) const {}
    template <int TN>
    __device__ __forceinline__ void preload(int64_t row0, int64_t row1, bool, bool, int vcol0, int c, AuxRows<TN> &x) const
    {
        const int64_t o0 = row0 * ld + vcol0 + c, o1 = row1 * ld + vcol0 + c;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            x.a0[j] = x2[o0 + 32 * j];
            x.a1[j] = x2[o1 + 32 * j];
        }
    }
    template <int TN>
    __device__ __forceinline__ void rows2(int64_t row0, bool ok0, bool ok1, int vcol0, int c, const float (&v0)[TN],
                                          const float (&v1)[TN], const AuxRows<TN> &x) const
    {
        const int64_t o0 = row0 * ld + vcol0, o1 = o0 + ld;
#pragma unroll
        for (int j = 0; j < TN; ++j)
            store_bf16_rows2(out + o0 + 32 * j, out + o1 + 32 * j, ok0, ok1, c, v0[j] + x.a0[j], v1[j] + x.a1[j]);
    }
};

// a = bf16(silu(gate) * up); the wave tile's first WN/2 columns are gate, the rest the matching up
struct EpiSiluMul {
    bf16_t *a; int64_t ld;   // [M][d_ff]
    template <int TN> using Aux = NoAux;
    template <int TN> __device__ __forceinline__ void preload0(int64_t, int64_t, NoAux &) const {}
    template <int TN> __device__ __forceinline__ void preload(int64_t, int64_t, bool, bool, int, int, NoAux &) const {}
    static __device__ __forceinline__ float silu_mul(float g, float u)
    {
        // g * sigmoid(g) * u with the hardware exp2 / reciprocal instructions (about 1 ulp each, far below the
        // bf16 rounding that follows). v_rcp_f32 itself: a correctly rounded reciprocal is an eleven-instruction
        // division sequence, a third of this epilogue's vector instructions.
        return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
    }
    template <int TN>
    __device__ __forceinline__ void rows2(int64_t row0, bool ok0, bool ok1, int vcol0, int c, const float (&v0)[TN],
                                          const float (&v1)[TN], const NoAux &) const
    {
        constexpr int WN = TN * 32;
        bf16_t *p0 = a + row0 * ld + (vcol0 / WN) * (WN / 2), *p1 = p0 + ld;
#pragma unroll
        for (int j = 0; j < TN / 2; ++j)
            store_bf16_rows2(p0 + 32 * j, p1 + 32 * j, ok0, ok1, c, silu_mul(v0[j], v0[j + TN / 2]),
                             silu_mul(v1[j], v1[j + TN / 2]));
    }
};

// rotary embedding on q and k heads (pairs (c, c + dh/2)), q -> [M][nq], k/v -> caches.
// row_sp[row] = (sequence, absolute position) of the row, position -1 if its sequence does not fit the
// cache (written by k_row_positions before the GEMM).
// own * cos -+ partner * sin (lower / upper half of the head). Which of the two products is rounded before the sum (the sine's in
// the lower half, the cosine's in the upper) is spelled out: left to the compiler, it differed between the epilogues, and the last
// bit of a row's q and K with the tiles that its call was dealt to.
__device__ __forceinline__ float rotated(float own, float partner, float2 cs, bool lo)
{
    return lo ? __builtin_fmaf(own, cs.x, -(partner * cs.y)) : __builtin_fmaf(partner, cs.y, own * cs.x);
}
template <int TN> struct AuxRope { float2 t0[TN], t1[TN]; int2 sp0, sp1; };

template <int DHT>                                      // head size: 64 or 128
struct EpiQkvRope {
    bf16_t *q, *kc, *vc;
    const float2 *rope; const int2 *row_sp;
    int L_max, Hq, Hkv;
    template <int TN> using Aux = AuxRope<TN>;
    template <int TN> __device__ __forceinline__ void preload0(int64_t row0, int64_t row1, AuxRope<TN> &x) const
    {
        x.sp0 = row_sp[row0];
        x.sp1 = row_sp[row1];
    }
    template <int TN>
    __device__ __forceinline__ void preload(int64_t, int64_t, bool, bool, int vcol0, int c, AuxRope<TN> &x) const
    {
        constexpr int dh = DHT, half = DHT / 2;
        if (vcol0 < (Hq + Hkv) * dh) {                   // q or k: cos / sin of the two positions
            const int pa = x.sp0.y < 0 ? 0 : x.sp0.y, pb = x.sp1.y < 0 ? 0 : x.sp1.y;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int cj = (32 * j + c) & (dh - 1);  // position inside the head
                const int ci = cj < half ? cj : cj - half;
                x.t0[j] = rope[(int64_t)pa * half + ci];
                x.t1[j] = rope[(int64_t)pb * half + ci];
            }
        }
    }
    template <int TN>
    __device__ __forceinline__ void rows2(int64_t row0, bool ok0, bool ok1, int vcol0, int c, const float (&v0)[TN],
                                          const float (&v1)[TN], const AuxRope<TN> &x) const
    {
        constexpr int dh = DHT, half = DHT / 2;
        const int nq = Hq * dh, nkv = Hkv * dh;
        ok0 = ok0 && x.sp0.y >= 0;
        ok1 = ok1 && x.sp1.y >= 0;
        // the wave tile (128 columns, heads of 64 or 128) lies inside one of q / k / v
        const int seg = vcol0 < nq ? 0 : (vcol0 < nq + nkv ? 1 : 2);
        const int w0 = vcol0 - (seg == 0 ? 0 : (seg == 1 ? nq : nq + nkv));   // column inside the segment
        bf16_t *d0, *d1;                                 // destination of the wave tile's first column, rows 0 / 1
        if (seg == 0) { d0 = q + row0 * (int64_t)nq + w0; d1 = d0 + nq; }
        else {
            bf16_t *cache = seg == 1 ? kc : vc;
            const int hd = w0 / dh, wi = w0 - hd * dh;
            d0 = cache + (((int64_t)x.sp0.x * Hkv + hd) * L_max + x.sp0.y) * dh + wi;
            d1 = cache + (((int64_t)x.sp1.x * Hkv + hd) * L_max + x.sp1.y) * dh + wi;
        }
        const int hstep = (seg == 0 || dh >= TN * 32) ? 0 : (int)((int64_t)L_max * dh) - dh;   // next head inside the tile (dh = 64)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float o0 = v0[j], o1 = v1[j];
            if (seg < 2) {                               // q or k: rotate
                const bool lo = ((32 * j) & (dh - 1)) < half;                 // the same for every c < 32
                const int jp = lo ? j + half / 32 : j - half / 32;            // tile of the partner column
                const float y0 = v0[jp], y1 = v1[jp];
                o0 = rotated(o0, y0, x.t0[j], lo);
                o1 = rotated(o1, y1, x.t1[j], lo);
            }
            const int hj = (32 * j) / dh;                // head inside the tile of column 32*j + c
            const int64_t off = (seg == 0) ? 32 * j : (int64_t)hj * hstep + 32 * j;
            store_bf16_rows2(d0 + off, d1 + off, ok0, ok1, c, o0, o1);
        }
    }
};

// row -> (sequence, absolute position), position -1 (and the overflow flag) if the sequence does not fit
__global__ void __launch_bounds__(256)
k_row_positions(const int32_t *__restrict__ pos0, int64_t M, int Tn, int L_max, int2 *__restrict__ row_sp, int *flags)
{
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= M) return;
    const int s = (int)(row / Tn), i = (int)(row - (int64_t)s * Tn);
    const int p0 = pos0 ? pos0[s] : 0;
    const bool bad = p0 < 0 || p0 + Tn > L_max;
    if (bad && i == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
    row_sp[row] = make_int2(s, bad ? -1 : p0 + i);
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

// The product's rows are the vocabulary entries (A = the head's weights), its columns the tokens (B = the hidden
// states, padded with zero rows to a multiple of the tile). A lane of the
// accumulator layout then holds, for each of its TN tokens, 16 * TM logits of that token (the wave tile's 128 vocabulary
// rows are split between the two halves of the wave), so the maximum and the sum of exponentials per (token, tile) are
// sums over the lane's own registers plus ONE exchange with lane ^ 32 (with tokens as rows a lane holds one column
// and every row costs two five-step butterflies), and the big operand (525 MB of weights at the Llama vocabulary) is
// the one that each XCD streams once, while the hidden states, which the memory-side cache holds, are the ones read
// again. part: [V / 128][Mp] (token fastest: a half-wave stores 32 consecutive entries; Mp = padded token count).
// What a token gets does not depend on the other tokens of the call. The target's logit comes from k_target_logit,
// since a lane would have to search its registers for it.
__device__ __forceinline__ float swap_halves(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, __builtin_bit_cast(int, v)));
}
struct EpiNllCols {
    static constexpr bool whole_tile = true;
    float2 *part;               // [V / 128][Mp]
    int64_t M;                  // Mp: tokens, padded to the tile
    template <int TM, int TN>
    __device__ __forceinline__ void tile(const floatx16_t (&acc)[TM][TN], int64_t vrow_w, int tcol_w, int lane) const
    {
        constexpr float LOG2E = 1.44269504088896341f;
        float2 *dst = part + (vrow_w / (TM * 32)) * M + tcol_w + (lane & 31);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float m = acc[0][j][0];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) m = fmaxf(m, acc[i][j][r]);
            m = fmaxf(m, swap_halves(m, lane));
            const float ml = m * LOG2E;
            float q4[4];                                          // rows 8q .. 8q + 7 of every 32: this lane's half, then both
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float s0 = 0.f, s1 = 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 4 * q; r < 4 * q + 4; r += 2) {
                        s0 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][r], LOG2E, -ml));
                        s1 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][r + 1], LOG2E, -ml));
                    }
                const float own = s0 + s1;
                q4[q] = own + swap_halves(own, lane);
            }
            const float se = (q4[0] + q4[1]) + (q4[2] + q4[3]);
            if (lane < 32) dst[32 * j] = make_float2(m, se);
        }
    }
};

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

// Register r of accumulator tile (i, j) is row 32*i + 8*(r/4) + 4*(lane/32) + r%4, column 32*j + lane%32
// of the wave tile (row_w already holds the wave tile's first row + 4*(lane/32)). Per 32-row tile all
// global reads of the epilogue are issued first, then the row pairs are combined and stored.
template <class E, class = void> struct epi_whole_tile { static constexpr bool value = false; };
template <class E> struct epi_whole_tile<E, decltype((void)E::whole_tile)> { static constexpr bool value = E::whole_tile; };

template <bool FULL, int TM, int TN, class Epi>
__device__ __forceinline__ void gemm_epilogue(const floatx16_t (&acc)[TM][TN], const Epi &epi, int64_t row_w, int64_t M,
                                              int vcol0, int c)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        typename Epi::template Aux<TN> aux[8];
#pragma unroll
        for (int rp = 0; rp < 8; ++rp) {
            const int64_t row0 = row_w + i * 32 + 8 * (rp >> 1) + 2 * (rp & 1);
            const bool ok0 = FULL || row0 < M, ok1 = FULL || row0 + 1 < M;
            epi.template preload0<TN>(ok0 ? row0 : M - 1, ok1 ? row0 + 1 : M - 1, aux[rp]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rp = 0; rp < 8; ++rp) {
            const int64_t row0 = row_w + i * 32 + 8 * (rp >> 1) + 2 * (rp & 1);
            const bool ok0 = FULL || row0 < M, ok1 = FULL || row0 + 1 < M;
            epi.template preload<TN>(ok0 ? row0 : M - 1, ok1 ? row0 + 1 : M - 1, ok0, ok1, vcol0, c, aux[rp]);
        }
        __builtin_amdgcn_sched_barrier(0);                // keep the reads up here: sunk next to their uses they serialise
#pragma unroll
        for (int rp = 0; rp < 8; ++rp) {
            const int r = 2 * rp;                         // registers r, r + 1: two consecutive rows
            const int64_t row0 = row_w + i * 32 + 8 * (r >> 2) + (r & 3);
            float v0[TN], v1[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) { v0[j] = acc[i][j][r]; v1[j] = acc[i][j][r + 1]; }
            epi.template rows2<TN>(row0, FULL || row0 < M, FULL || row0 + 1 < M, vcol0, c, v0, v1, aux[rp]);
        }
    }
}

// 16 bytes per lane from global memory (wave-uniform base + 32-bit byte offset per lane) straight into LDS: lane l's
// piece lands at lds_addr + 16 * l (M0 holds the wave's LDS byte address; one wait state between writing M0 and the
// load). Written as inline assembly because the compiler, which sees an LDS write it cannot place, would wait for
// the load before the next LDS read of any stage. The kernel therefore owns the waits: vm_wait<0>() before the
// barrier that publishes a stage, and before a workgroup ends. The kernel must have no static LDS (the dynamic
// segment then starts at LDS address 0).
__device__ __forceinline__ void dtl16(const bf16_t *base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// the same with the LDS address as a base and a constant: nothing for the compiler to keep 32 sums of in scalar registers
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
// Bound: the power the chip grants its matrix cores. With normally distributed operands a loop of nothing but 32x32x16
// instructions reaches 1.78 PFLOP/s (2.46 on zeros), of 16x16x32 2.06: they move fewer accumulator bits per product.
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
// half of the register file in this kernel for anything else; ACC_ALL among the clobbers of every barrier keeps it from values that live
// long, and tests/test_isa_waits.py looks for any other use in the disassembly. Wait states between the last matrix instruction and the first
// read of its result are the kernel's own business too (acc_settle).
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
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
template <int R> __device__ __forceinline__ f32x4_t acc_read()
{
    float a, b, c, d;
    asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]"
                 : "=v"(a), "=v"(b), "=v"(c), "=v"(d) : "n"(R), "n"(R + 1), "n"(R + 2), "n"(R + 3));
    return f32x4_t{a, b, c, d};
}
template <int... I, class F> __device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_(std::make_integer_sequence<int, N>{}, f); }

// ------------------------------------------------------------------------------------------------
// Epilogues of k_gemm_mfma. A lane holds, for token 16 t + lane % 16 of its wave tile's 128 (t < 8) and g = lane / 16, the columns
// 32 p + 8 g .. + 7 (p < 4) of the wave tile's 128: 16 bytes of a bf16 row. Parts of an epilogue (row: an existing token, col0:
// the wave tile's first virtual column):
//   place(row[8], p)               what is known of the lane's eight tokens before anything else
//   fetch(row, p, col0, g, aux)    reads what a token's piece needs, AHEAD tokens ahead of
//   put(row, ok, p, col0, g, v, aux)   which combines and stores it (ok: the token exists)
// The pieces lie in the caller's tensors, which are aligned to their elements only: AnyVec.
// ------------------------------------------------------------------------------------------------
typedef u32x4_t AnyU4 __attribute__((aligned(2)));
typedef f32x4_t AnyF4 __attribute__((aligned(4)));
struct NoPlace {};
struct EpiTokens {                                          // what most epilogues have in common
    static constexpr bool weight_rows = false;              // tiles are walked in bands of tokens (or of weight rows)
    static constexpr int AHEAD = 2;
    typedef NoPlace Place;
    struct Aux {};
    __device__ __forceinline__ void place(const uint32_t (&)[8], NoPlace (&)[8]) const {}
    template <class A> __device__ __forceinline__ void fetch(uint32_t, const NoPlace &, int, int, A &) const {}
};
__device__ __forceinline__ u32x4_t pack8(const float (&v)[8])
{
    return u32x4_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

struct EpiStoreF32x8 : EpiTokens {
    float *C; int64_t ldc;
    EpiStoreF32x8(float *c, int64_t l) : C(c), ldc(l) {}
    __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[4][8], const Aux &) const
    {
        float *const o = C + row * ldc + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<AnyF4 *>(o + 32 * p + 4 * h) = f32x4_t{v[p][4 * h], v[p][4 * h + 1], v[p][4 * h + 2], v[p][4 * h + 3]};
    }
};

struct EpiResidF32x8 : EpiTokens {                          // EpiResidF32
    const bf16_t *resid; float *out; int64_t ld;
    EpiResidF32x8(const bf16_t *r, float *o, int64_t l) : resid(r), out(o), ld(l) {}
    struct Aux { u32x4_t r[4]; };
    __device__ __forceinline__ void fetch(uint32_t row, const NoPlace &, int col0, int g, Aux &x) const
    {
        const bf16_t *const r = resid + row * ld + col0 + 8 * g;
#pragma unroll
        for (int p = 0; p < 4; ++p) x.r[p] = *reinterpret_cast<const AnyU4 *>(r + 32 * p);
    }
    __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[4][8], const Aux &x) const
    {
        float *const o = out + row * ld + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < 4; ++p)
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

struct EpiResidOut8 : EpiTokens {                           // EpiResidOut
    const float *x2; bf16_t *out; int64_t ld;
    EpiResidOut8(const float *x, bf16_t *o, int64_t l) : x2(x), out(o), ld(l) {}
    struct Aux { f32x4_t r[4][2]; };
    __device__ __forceinline__ void fetch(uint32_t row, const NoPlace &, int col0, int g, Aux &x) const
    {
        const float *const r = x2 + row * ld + col0 + 8 * g;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) x.r[p][h] = *reinterpret_cast<const AnyF4 *>(r + 32 * p + 4 * h);
    }
    __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[4][8], const Aux &x) const
    {
        bf16_t *const o = out + row * ld + col0 + 8 * g;
        if (!ok) return;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = v[p][e] + x.r[p][e >> 2][e & 3];
            *reinterpret_cast<AnyU4 *>(o + 32 * p) = pack8(y);
        }
    }
};

struct EpiSiluMul8 : EpiTokens {                            // EpiSiluMul; gate in pieces 0 and 2, up in 1 and 3
    bf16_t *a; int64_t ld;
    EpiSiluMul8(bf16_t *a_, int64_t l) : a(a_), ld(l) {}
    __device__ __forceinline__ void put(uint32_t row, bool ok, const NoPlace &, int col0, int g, const float (&v)[4][8], const Aux &) const
    {
        bf16_t *const o = a + row * ld + col0 / 2 + 8 * g;
        u32x4_t y[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            float z[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = EpiSiluMul::silu_mul(v[2 * p][e], v[2 * p + 1][e]);
            y[p] = pack8(z);
        }
        if (!ok) return;
        *reinterpret_cast<u32x4_t *>(o) = y[0];
        *reinterpret_cast<u32x4_t *>(o + 32) = y[1];
    }
};

// EpiQkvRope with the rows' positions by arithmetic: a row's sequence that does not fit its cache is flagged and not stored.
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
    struct Aux { f32x4_t cs[ND][4]; };
    __device__ __forceinline__ void place(const uint32_t (&row)[8], Place (&pl)[8]) const
    {
        int p0[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            pl[t].s = (int)(row[t] / (uint32_t)Tn);
            p0[t] = pos0 ? pos0[pl[t].s] : 0;
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bool bad = p0[t] < 0 || p0[t] + Tn > L_max;
            if (bad) atomicOr(flags, FLAG_CACHE_OVERFLOW);
            pl[t].pos = bad ? -1 : p0[t] + (int)(row[t] - (uint32_t)pl[t].s * (uint32_t)Tn);
        }
    }
    __device__ __forceinline__ void fetch(uint32_t, const Place &pl, int col0, int g, Aux &x) const
    {
        if (col0 >= (Hq + Hkv) * DHT) return;               // v
        const float *const r = reinterpret_cast<const float *>(rope + (int64_t)(pl.pos < 0 ? 0 : pl.pos) * (DHT / 2)) + 16 * g;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int h = 0; h < 4; ++h) x.cs[d][h] = *reinterpret_cast<const f32x4_t *>(r + 64 * d + 4 * h);
    }
    __device__ __forceinline__ void put(uint32_t row, bool ok, const Place &pl, int col0, int g, const float (&v)[4][8], const Aux &x) const
    {
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
        u32x4_t y[4];
        if (seg == 2) {
#pragma unroll
            for (int p = 0; p < 4; ++p) y[p] = pack8(v[p]);
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
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
        for (int p = 0; p < 4; ++p) *reinterpret_cast<AnyU4 *>(d + (p >> 1) * up + 32 * (p & 1)) = y[p];
    }
};

// EpiNllCols: the partial results of the wave tile's 128 vocabulary entries. A lane holds rows 8g .. 8g + 7 of every 32; the sums
// run in that epilogue's order.
struct EpiNllCols8 {
    static constexpr bool weight_rows = true;
    float2 *part;                                           // [V / 128][Mp]
    int64_t Mp;
};
__device__ __forceinline__ float lane_xor(float v, int lane, int x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ x) << 2, __builtin_bit_cast(int, v)));
}

template <class Epi>
__device__ __forceinline__ void tile_epilogue(const Epi &epi, int64_t m_w, int64_t M, int col0, int lane)
{
    const int g = lane >> 4;
    uint32_t row[8];
    bool ok[8];
    typename Epi::Place pl[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int64_t r = m_w + 16 * t + (lane & 15);
        ok[t] = r < M;
        row[t] = (uint32_t)(ok[t] ? r : M - 1);
    }
    epi.place(row, pl);
    typename Epi::Aux aux[Epi::AHEAD + 1];
#pragma unroll
    for (int t = 0; t < Epi::AHEAD; ++t) epi.fetch(row[t], pl[t], col0, g, aux[t]);
    static_for<8>([&](auto t_) {
        constexpr int t = t_;
        if constexpr (t + Epi::AHEAD < 8) epi.fetch(row[t + Epi::AHEAD], pl[t + Epi::AHEAD], col0, g, aux[(t + Epi::AHEAD) % (Epi::AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
        float v[4][8];
        static_for<8>([&](auto i_) {
            constexpr int i = i_;
            const f32x4_t a = acc_read<4 * (8 * i + t)>();
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i >> 1][4 * (i & 1) + e] = a[e];
        });
        epi.put(row[t], ok[t], pl[t], col0, g, v, aux[t % (Epi::AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
    });
}
__device__ __forceinline__ void tile_epilogue(const EpiNllCols8 &epi, int64_t m_w, int64_t, int col0, int lane)
{
    constexpr float LOG2E = 1.44269504088896341f;
    float2 *const dst = epi.part + (int64_t)(col0 / 128) * epi.Mp + m_w + (lane & 15);
    static_for<8>([&](auto t_) {
        constexpr int t = t_;
        f32x4_t v[8];
        static_for<8>([&](auto i_) { v[i_] = acc_read<4 * (8 * i_ + t)>(); });
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

template <class Epi>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_gemm_mfma(const bf16_t *__restrict__ X, BMap bmap, int64_t M, int K, int tiles_r, int tiles_c, Epi epi)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int SB = 65536;                               // a stage: 256 weight rows, 256 token rows of 128 bytes
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
    const uint32_t w_off0 = ((uint32_t)rip * (uint32_t)ld + (uint32_t)((chunk ^ (((rip >> 1) & 1) | ((rip >> 3) << 1))) * 8)) * 2u;
    const uint32_t w_off1 = w_off0 + (uint32_t)(2 * w_mid) * 2u;
    const uint32_t x_chunk = (uint32_t)((chunk ^ ((rip >> 1) & 7)) * 8);
    uint32_t x_off[8];
    const bf16_t *we, *wo, *we2, *wo2, *xb;                 // of the slice being requested: pieces 0, 1, 2, 3 (4 .. 7 at w_off1), tokens
    int64_t m0, m0_next;
    int n0, n0_next;
    auto tile_src = [&](int l, int64_t &m, int &n) {
        const int grp = l / group_sz, in_grp = l - grp * group_sz;
        const int rows_here = (tiles_r - grp * GROUP_M) < GROUP_M ? (tiles_r - grp * GROUP_M) : GROUP_M;
        const int tr = grp * GROUP_M + in_grp % rows_here, tc = in_grp / rows_here;
        m = (int64_t)(Epi::weight_rows ? tc : tr) * 256;
        n = (Epi::weight_rows ? tr : tc) * 256;
        we = bmap.row(n);
        wo = bmap.row(n + 32);
        we2 = we + w_mid;
        wo2 = wo + w_mid;
        xb = X + m * ld;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            int64_t r = p * 32 + rip;
            if (m + r >= M) r = M - 1 - m;                  // ragged last tile: re-read the last row, never stored
            x_off[p] = ((uint32_t)(r * ld) + x_chunk) * 2u;
        }
    };
    // request R of a slice into stage STG: 0..3 the weights' top halves (rows 0..63 of each wave's 128), 4..7 the tokens' left
    // halves, 8..11 right, 12..15 bottom
    const uint32_t wave_lds = (uint32_t)wave * 1024u;
    auto request = [&](auto r_, auto stg_) {
        constexpr int R = r_, q = R & 3, p = (q & 1) + 4 * (q >> 1) + (R >= 8 ? 2 : 0), at = (int)stg_ + p * 4096;
        if constexpr (R < 4) dtl16c<at>(q & 1 ? wo : we, q >> 1 ? w_off1 : w_off0, wave_lds);
        else if constexpr (R >= 12) dtl16c<at>(q & 1 ? wo2 : we2, q >> 1 ? w_off1 : w_off0, wave_lds);
        else dtl16c<at + 32768>(xb, x_off[p], wave_lds);
    };
    auto next_slice = [&] { we += BK; wo += BK; we2 += BK; wo2 += BK; xb += BK; };

    // ---- fragments. Weight rows are dealt to the 16 rows of instruction tiles 2p and 2p + 1 so that a lane's results of the
    // two are eight consecutive columns: lane (m, g) reads row 32p + 8 (m / 4) + 4 e + m % 4 of tile 2p + e ----
    const int m16 = lane & 15, g = lane >> 4;
    const uint32_t w_row = (uint32_t)(ww * 128 + 8 * (m16 >> 2) + (m16 & 3)) * 128, w_swz = (uint32_t)(((m16 >> 1) & 1) | ((m16 >> 2) << 1));
    const uint32_t x_row = (uint32_t)(256 + wt * 128 + m16) * 128, x_swz = (uint32_t)((m16 >> 1) & 7);
    const uint32_t w_at[2] = {w_row + (((uint32_t)g ^ w_swz) << 4), w_row + (((uint32_t)(g + 4) ^ w_swz) << 4)};
    const uint32_t x_at[2] = {x_row + (((uint32_t)g ^ x_swz) << 4), x_row + (((uint32_t)(g + 4) ^ x_swz) << 4)};
    typedef bf16x8_t Half[2][4];                            // half an operand of a step: [32 of K][16 rows]
    auto read_w = [&](Half &d, auto f_, int half, int stg) {
        constexpr int f = f_;
        d[f >> 2][f & 3] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(
                                                            lds + stg + w_at[f >> 2] + (half * 64 + ((f & 3) >> 1) * 32 + (f & 1) * 4) * 128));
    };
    auto read_x = [&](Half &d, auto f_, int half, int stg) {
        constexpr int f = f_;
        d[f >> 2][f & 3] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(lds + stg + x_at[f >> 2] + (half * 64 + (f & 3) * 16) * 128));
    };
    // One quadrant: 32 instructions in the order that changes one operand at a time; behind them 8 fragment reads (the first
    // 16) and 4 requests.
#define SOL_QUAD(FIRST_, W_, X_, HW_, HX_, READ_, RD_, RHALF_, RSTG_, REQ0_, STG_)                                        \
    static_for<32>([&](auto m_) {                                                                                              \
        constexpr int m = m_, kg = m >> 4, i = (m >> 2) & 3, j = (i & 1) ? 3 - (m & 3) : (m & 3);                                \
        acc_mma<4 * (8 * (HW_ * 4 + i) + HX_ * 4 + j), FIRST_ && kg == 0>(W_[kg][i], X_[kg][j]);                                 \
        if constexpr ((m & 1) == 0 && m < 16) READ_(RD_, std::integral_constant<int, m / 2>{}, RHALF_, RSTG_);                   \
        if constexpr ((m & 7) == 1) request(std::integral_constant<int, REQ0_ + m / 8>{}, std::integral_constant<int, STG_>{});                          \
        __builtin_amdgcn_sched_barrier(0);                                                                                     \
    });
    // The 16 youngest requests are those of the last two half steps: what the half step after the barrier reads has landed. The
    // wave's own reads of the halves that will be overwritten are over (lgkmcnt).
#define SOL_SYNC                                                                                                               \
    asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory", SOL_ACC_ALL);                                      \
    __builtin_amdgcn_sched_barrier(0);
    // One step of the slice in stage CS_, the next in NS_; XL_ holds its left tokens, XR_ is free. Requests: slice + 2 into CS_.
#define SOL_STEP(FIRST_, XL_, XR_, CS_, NS_)                                                                             \
    SOL_QUAD(FIRST_, wtop, XL_, 0, 0, read_x, XR_, 1, CS_, 0, CS_)                                                       \
    SOL_QUAD(FIRST_, wtop, XR_, 0, 1, read_w, wbot, 1, CS_, 4, CS_)                                                      \
    SOL_SYNC                                                                                                                   \
    SOL_QUAD(FIRST_, wbot, XR_, 1, 1, read_w, wtop, 0, NS_, 8, CS_)                                                      \
    SOL_QUAD(FIRST_, wbot, XL_, 1, 0, read_x, XR_, 0, NS_, 12, CS_)                                                      \
    SOL_SYNC
    // Two steps; the requests of a tile's last two are the first two slices of the next tile (of this one again after the last
    // tile: never used), so only a workgroup's first tile starts cold.
#define SOL_PAIR(FIRST_, KT_)                                                                                                  \
    {                                                                                                                          \
        if ((KT_) == KT - 2) tile_src(more ? lin + lin_step : lin, m0_next, n0_next);                                           \
        else next_slice();                                                                                                     \
        SOL_STEP(FIRST_, xa, xc, 0, SB)                                                                                         \
        next_slice();                                                                                                          \
        SOL_STEP(false, xc, xa, SB, 0)                                                                                          \
    }
    Half wtop, wbot, xa, xc;
    const int KT = K / BK;                                  // even (K is a multiple of 128)
    tile_src(lin, m0, n0);
    static_for<16>([&](auto r) { request(r, std::integral_constant<int, 0>{}); });
    next_slice();
    static_for<16>([&](auto r) { request(r, std::integral_constant<int, SB>{}); });
    SOL_SYNC
    static_for<8>([&](auto f) { read_w(wtop, f, 0, 0); read_x(xa, f, 0, 0); });
    SOL_SYNC
    for (;;) {
        const bool more = lin + lin_step < band_end;
        SOL_PAIR(true, 0)
        for (int kt = 2; kt < KT; kt += 2) SOL_PAIR(false, kt)
        acc_settle();
        tile_epilogue(epi, m0 + wt * 128, M, n0 + ww * 128, lane);
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
// most one workgroup. ST LDS stages filled by LDS-direct loads, so that ST slices are in flight. A step reads the fragments
// of slice kt + 1 and multiplies slice kt; their order is the compiler's, which keeps only part of the next slice's fragments
// in registers (61 to 91 for the 32 x 32 and 32 x 64 wave tiles). Bound: a step's time goes with its bytes, 0.19 us per slice
// of a 64 x 64 tile (16 KB) and 0.39 us of 128 x 128 (32 KB), about 85 GB/s for one CU alone. Every output is a
// chain of 32x32x16 MFMAs over k, two of which are one 16x16x32 of k_gemm_mfma bit for bit: the tile does not show in the results.
// ------------------------------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, int ST, class Epi>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64, 2)
k_gemm_tile(const bf16_t *__restrict__ A, int64_t lda, BMap bmap, int64_t m_first, int64_t M, int Nv, int K, int tiles_m,
            int tiles_n, Epi epi)
{
    constexpr int NWN = BN / WN, NT = (BM / WM) * NWN * 64;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int RPP = NT / 8, AP = BM / RPP, BP = BN / RPP;      // rows per pass of the workgroup's loads, passes
    constexpr uint32_t SB = (BM + BN) * 128;                       // bytes of a stage
    static_assert(BM % RPP == 0 && BN % RPP == 0 && RPP % 16 == 0, "tile / thread mismatch");
    static_assert(ST >= 2 && (AP + BP) * (ST - 1) < 64, "vmcnt counts the loads in flight");
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / NWN, wn = wave - wm * NWN;
    // XCD-aware tile mapping as in k_gemm_mfma
    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= n_tiles) return;
    const int group_sz = GROUP_M * tiles_n, grp = lin / group_sz, in_grp = lin - grp * group_sz;
    const int rows_here = (tiles_m - grp * GROUP_M) < GROUP_M ? (tiles_m - grp * GROUP_M) : GROUP_M;
    const int64_t m0 = m_first + (int64_t)(grp * GROUP_M + in_grp % rows_here) * BM;
    const int n0 = (in_grp / rows_here) * BN;

    const int chunk = tid & 7, rip = tid >> 3;
    const uint32_t sw = (uint32_t)((chunk ^ SOL_SWZ(rip)) * 8);
    const bf16_t *a_base = A + m0 * lda;
    uint32_t a_off[AP];
#pragma unroll
    for (int p = 0; p < AP; ++p) {
        int64_t rl = p * RPP + rip;
        if (m0 + rl >= M) rl = M - 1 - m0;                 // ragged last tile: re-read the last row, never stored
        a_off[p] = ((uint32_t)(rl * lda) + sw) * 2u;
    }
    const bf16_t *b_base[BP];
#pragma unroll
    for (int p = 0; p < BP; ++p) b_base[p] = bmap.row(n0 + p * RPP + wave * 8);   // a wave's 8 rows lie in one weight matrix
    const uint32_t b_off = ((uint32_t)(rip & 7) * (uint32_t)bmap.ld + sw) * 2u;

    const int KT = K / BK;                                 // even (K is a multiple of 128)
    auto request = [&](int kt, uint32_t stage) {
        const int koff = (kt < KT ? kt : KT - 1) * BK;     // past the end: the last slice again, never multiplied
#pragma unroll
        for (int p = 0; p < AP; ++p) dtl16(a_base + koff, a_off[p], stage + (uint32_t)(p * RPP * 128 + wave * 1024));
#pragma unroll
        for (int p = 0; p < BP; ++p) dtl16(b_base[p] + koff, b_off, stage + (uint32_t)((BM + p * RPP) * 128 + wave * 1024));
    };
    const int frow = lane & 31, fk = lane >> 5, fsw = SOL_SWZ(frow);
    const int a_frag = (wm * WM + frow) * 128, b_frag = (BM + wn * WN + frow) * 128;
    auto fragments = [&](bf16x8_t (&fa)[4][TM], bf16x8_t (&fb)[4][TN], uint32_t stage) {
        const unsigned char *const st = lds + stage;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int coff = ((kk * 2 + fk) ^ fsw) << 4;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[kk][i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(st + a_frag + i * 32 * 128 + coff));
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[kk][j] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(st + b_frag + j * 32 * 128 + coff));
        }
    };
    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    auto multiply = [&](const bf16x8_t (&fa)[4][TM], const bf16x8_t (&fb)[4][TN]) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i], fb[kk][j], acc[i][j], 0, 0, 0);
    };
    // All but the N youngest slices that this wave requested have landed and its fragment reads are over; so for all waves.
#define SOL_TILE_SYNC(N) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"((AP + BP) * (N)) : "memory")
#pragma unroll
    for (int s = 0; s < ST; ++s) request(s, s * SB);
    bf16x8_t fa0[4][TM], fb0[4][TN], fa1[4][TM], fb1[4][TN];
    uint32_t cur = 0, nxt = SB;                            // the stages of slices kt and kt + 1
    SOL_TILE_SYNC(ST - 1);
    fragments(fa0, fb0, 0);
    for (int kt = 0; kt < KT; kt += 2) {
        SOL_TILE_SYNC(ST - 2);                             // slice kt + 1 is there, the stage of slice kt is read out
        request(kt + ST, cur);
        fragments(fa1, fb1, nxt);
        multiply(fa0, fb0);
        cur = nxt; nxt = nxt + SB == ST * SB ? 0 : nxt + SB;
        SOL_TILE_SYNC(ST - 2);
        request(kt + 1 + ST, cur);
        fragments(fa0, fb0, nxt);
        multiply(fa1, fb1);
        cur = nxt; nxt = nxt + SB == ST * SB ? 0 : nxt + SB;
    }
#undef SOL_TILE_SYNC
    vm_wait<0>();                                           // no LDS-direct load outlives its workgroup
    if constexpr (epi_whole_tile<Epi>::value) {             // (the launcher admits whole tiles only)
        epi.template tile<TM, TN>(acc, m0 + wm * WM, n0 + wn * WN, lane);
    } else {
        const int64_t row_w = m0 + wm * WM + 4 * (lane >> 5);
        if (m0 + BM <= M) gemm_epilogue<true, TM, TN>(acc, epi, row_w, M, n0 + wn * WN, lane & 31);
        else gemm_epilogue<false, TM, TN>(acc, epi, row_w, M, n0 + wn * WN, lane & 31);
    }
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
    auto kern = k_gemm_mfma<Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess) return false;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3((wg_xcd > 0 && wg_xcd < per_xcd ? wg_xcd : per_xcd) * 8), dim3(256), lds, st, X, bmap, M, K,
                       Epi::weight_rows ? tiles_w : tiles_x, Epi::weight_rows ? tiles_x : tiles_w, epi);
    return true;
}

constexpr int SOL_WN = 128;                                // vocabulary entries of a partial sum of the head

// How the rows of a product are dealt to tiles. Per round of one workgroup on every CU, a 256 x 256 tile per CU costs
// 1; a grid of one smaller tile per CU at most costs, relative to that (K = 2048 .. 14336, 80 .. 2048 rows, the
// projections of the 1B and 8B shapes; what a round takes hardly depends on how many CUs it fills):
//   64 x 64: 0.23   128 x 64: 0.36   128 x 128: 0.5   128 x 256: 0.75
// (down projection of the 1B shape, 256 x 256 -> rule: 333 rows 122 -> 28 us, 1024 rows 123 -> 43, 2048 rows 125 -> 69.)
// The q/k/v map with heads of 128 has 64 x 128 tiles in place of both 64-column ones, and goes by the same costs: 8B shape, 80
// rows 80 -> 36 us, 333 rows 86 -> 44, 512 rows 77 -> 45, 1024 rows 82 -> 65, from 1500 rows on 256 x 256 tiles.
// So a call takes the smallest tile of which every CU gets at most one; with more rows than that, whole rounds of
// 256 x 256 tiles first and the smaller tile for the rest where that ends sooner than a last round that is nearly
// empty. The tile does not show in the results.
struct GemmPlan {
    int64_t big;                 // rows [0, big) in 256 x 256 tiles (all rows, or a multiple of 256)
    int small;                   // the others: 0 = 64 x 64, 1 = 128 x 64, 2 = 128 x 128, 3 = 128 x 256
};
static double small_tile_cost(int64_t rows, int N, int cus, int &cfg)
{
    static const int bm[4] = {64, 128, 128, 128}, bn[4] = {64, 64, 128, 256};
    static const double cost[4] = {0.23, 0.36, 0.5, 0.75};
    for (cfg = 0; cfg < 4; ++cfg)
        if ((rows + bm[cfg] - 1) / bm[cfg] * (N / bn[cfg]) <= cus) return cost[cfg];
    return 1e9;
}
static GemmPlan plan_gemm(int64_t M, int N)
{
    const int cus = device_cus() > 0 ? device_cus() : 256;
    const int64_t tn = N / 256, whole = M / 256;           // tile columns, whole tile rows
    const double launch = 0.05;                            // one more kernel
    GemmPlan best{M, 0};
    double best_cost = (double)(((M + 255) / 256 * tn + cus - 1) / cus);
    const int64_t rounds = whole * tn / cus;               // whole rounds of whole tiles
    const int64_t cand[3] = {0, rounds > 0 ? rounds * cus / tn : 0, whole};
    for (int64_t r : cand) {
        if (r * 256 >= M) continue;
        int cfg;
        const double c = (double)((r * tn + cus - 1) / cus) + small_tile_cost(M - r * 256, N, cus, cfg) + (r > 0 ? launch : 0.0);
        if (c < best_cost) { best_cost = c; best = GemmPlan{r * 256, cfg}; }
    }
    return best;
}

template <int BM, int BN, int WM, int WN, int ST, class Epi>
static bool launch_tile(const bf16_t *A, int64_t lda, const BMap &bmap, int64_t m_first, int64_t M, int Nv, int K,
                        const Epi &epi, hipStream_t st)
{
    constexpr size_t lds = (size_t)ST * (BM + BN) * 128;
    auto kern = k_gemm_tile<BM, BN, WM, WN, ST, Epi>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess) return false;
        attr_done = true;
    }
    const int tiles_m = (int)((M - m_first + BM - 1) / BM), tiles_n = Nv / BN, per_xcd = (tiles_m * tiles_n + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3((BM / WM) * (BN / WN) * 64), lds, st, A, lda, bmap, m_first, M, Nv, K,
                       tiles_m, tiles_n, epi);
    return true;
}

// Rows [m_first, M) in tiles of configuration cfg (GemmPlan::small). WN: columns an epilogue needs in one wave tile.
template <int WN, class Epi>
static bool launch_small(int cfg, const bf16_t *A, int64_t lda, const BMap &bmap, int64_t m_first, int64_t M, int Nv, int K,
                         const Epi &epi, hipStream_t st)
{
    if (Nv % 256 || K % (2 * BK) || K < 2 * BK) return false;
    if constexpr (WN == 128) {                               // a head of 128 in one wave tile: no 64-column tiles
        if (cfg <= 1) return launch_tile<64, 128, 32, 128, 6>(A, lda, bmap, m_first, M, Nv, K, epi, st);
        if (cfg == 2) return launch_tile<128, 128, 32, 128, 3>(A, lda, bmap, m_first, M, Nv, K, epi, st);
        return launch_tile<128, 256, 32, 128, 3>(A, lda, bmap, m_first, M, Nv, K, epi, st);
    } else {
        // slices in flight: at 24 KB each the 64 x 128 and 128 x 64 tiles gain from six (down projection of the 8B shape, 333 rows:
        // three 94 us, six 85; 1B shape, 1024 rows: 52.5, 49.5); 64 x 64 with eight and 128 x 128 with five measure as here
        if (cfg == 0) return launch_tile<64, 64, 32, WN, 4>(A, lda, bmap, m_first, M, Nv, K, epi, st);
        if (cfg == 1) return launch_tile<128, 64, 32, WN, 6>(A, lda, bmap, m_first, M, Nv, K, epi, st);
        if (cfg == 2) return launch_tile<128, 128, 32, 64, 4>(A, lda, bmap, m_first, M, Nv, K, epi, st);
        return launch_tile<128, 256, 64, 64, 3>(A, lda, bmap, m_first, M, Nv, K, epi, st);
    }
}

template <int DHT>
static bool launch_qkv_rope(const bf16_t *h, const BMap &bm, bf16_t *q, bf16_t *kc, bf16_t *vc, const float2 *rope,
                            const int32_t *pos0, int n_seq, int T, int L_max, int crows, int Hq, int Hkv, int d, int *flags,
                            int2 *row_sp, hipStream_t st)
{
    const int64_t M = (int64_t)n_seq * T;
    const int N = (Hq + 2 * Hkv) * DHT;
    if (M >= (1ll << 31)) return false;
    const GemmPlan plan = plan_gemm(M, N);
    if (plan.big > 0 &&
        !launch_mfma(h, bm, plan.big, N, d, EpiQkvRope8<DHT>{q, kc, vc, rope, pos0, T, L_max, crows, Hq, Hkv, flags}, st))
        return false;
    if (plan.big == M) return true;
    // the small tiles' table of the rows' (sequence, position), and the flags
    hipLaunchKernelGGL(k_row_positions, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, st, pos0, M, T, L_max, row_sp, flags);
    EpiQkvRope<DHT> epi{q, kc, vc, rope, row_sp, crows, Hq, Hkv};
    return launch_small<DHT>(plan.small, h, d, bm, plan.big, M, N, d, epi, st);
}

bool launch_gemm_qkv_rope(const void *h, const void *wq, const void *wk, const void *wv, void *q, void *kc, void *vc,
                          const float2 *rope, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh,
                          int d, int *flags, void *row_sp_ws, hipStream_t st, int cache_rows)
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
              flags, (int2 *)row_sp_ws, st);
}

static BMap plain_map(const void *w, int N, int K)
{
    BMap bm{};
    bm.base[0] = (const bf16_t *)w; bm.seg_end[0] = bm.seg_end[1] = bm.seg_end[2] = N; bm.mode = 0; bm.ld = K;
    return bm;
}

// A product over plain weight rows: `big` of the plan with epilogue eb, the others with e.
template <class EpiBig, class Epi>
static bool launch_planned(const void *a, const void *w, int64_t M, int N, int K, const EpiBig &eb, const Epi &e, hipStream_t st)
{
    if (M <= 0) return true;
    if (N % 256 || K % (2 * BK) || K < 2 * BK) return false;
    const BMap bm = plain_map(w, N, K);
    const GemmPlan plan = plan_gemm(M, N);
    if (plan.big > 0 && !launch_mfma((const bf16_t *)a, bm, plan.big, N, K, eb, st)) return false;
    return plan.big == M || launch_small<32>(plan.small, (const bf16_t *)a, K, bm, plan.big, M, N, K, e, st);
}

bool launch_gemm_resid_f32(const void *a, const void *w, const void *resid, float *out, int64_t M, int N, int K,
                           hipStream_t st)
{
    return launch_planned(a, w, M, N, K, EpiResidF32x8{(const bf16_t *)resid, out, N}, EpiResidF32{(const bf16_t *)resid, out, N}, st);
}

bool launch_gemm_gateup_silu(const void *h, const void *wg, const void *wu, void *a, int64_t M, int dff, int d,
                             hipStream_t st)
{
    const int N = 2 * dff;
    if (M <= 0) return true;
    if (dff % 64 || N % 256 || d % (2 * BK) || d < 2 * BK) return false;
    BMap bm{};
    bm.base[0] = (const bf16_t *)wg; bm.base[1] = (const bf16_t *)wu; bm.mode = 1; bm.ld = d;
    bm.half = 32;                                             // gate / up interleaved in pieces of 32 columns
    const GemmPlan plan = plan_gemm(M, N);
    if (plan.big > 0 && !launch_mfma((const bf16_t *)h, bm, plan.big, N, d, EpiSiluMul8{(bf16_t *)a, dff}, st)) return false;
    return plan.big == M || launch_small<64>(plan.small, (const bf16_t *)h, d, bm, plan.big, M, N, d, EpiSiluMul{(bf16_t *)a, dff}, st);
}

bool launch_gemm_resid_out(const void *a, const void *w, const float *x2, void *out, int64_t M, int N, int K,
                           hipStream_t st)
{
    return launch_planned(a, w, M, N, K, EpiResidOut8{x2, (bf16_t *)out, N}, EpiResidOut{x2, (bf16_t *)out, N}, st);
}

bool launch_gemm_f32(const void *a, const void *w, float *C, int64_t ldc, int64_t M, int N, int K, hipStream_t st)
{
    return launch_planned(a, w, M, N, K, EpiStoreF32x8{C, ldc}, EpiStoreF32{C, ldc}, st);
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
    // A decode step's few tokens take tiles of 32 or 64 columns, two workgroups per CU: with 256 columns of padding the matrix
    // cores need as long as HBM. The partial results are those of the large tiles bit for bit.
    // 128256 entries of 2048, one token: 133 -> 109 .. 123 us on two cards; a 1B decode step of 1 sequence 1198 -> 1165, of 64
    // 4599 -> 4553.
    const int64_t Mp = M <= 32 ? 32 : M <= 64 ? 64 : nll_pad_rows(M);
    if (V % 256 || K % (2 * BK) || K < 2 * BK || Mp >= (1ll << 31)) return false;
    const int n_wt = V / SOL_WN;
    float2 *part = (float2 *)scratch;
    float *tgt_logit = (float *)(part + (size_t)Mp * n_wt);
    int32_t *row_tgt = (int32_t *)(tgt_logit + Mp);
    const int64_t n_pad = (Mp - M) * K / 8, row_wgs = (M + 255) / 256, pad_wgs = (n_pad + 255) / 256;
    hipLaunchKernelGGL(k_row_targets, dim3((unsigned)(row_wgs > pad_wgs ? row_wgs : pad_wgs)), dim3(256), 0, st, targets, M, G, T,
                       broadcast_g ? 1 : 0, V, row_tgt, flags, (u32x4_t *)((bf16_t *)hf + M * K), n_pad);
    const BMap bt = plain_map(hf, (int)Mp, K);
    const EpiNllCols epc{part, Mp};
    const bf16_t *const head = (const bf16_t *)lm_head;
    if (!(Mp == 32 ? launch_tile<256, 32, 128, 32, 2>(head, K, bt, 0, V, (int)Mp, K, epc, st)
          : Mp == 64 ? launch_tile<256, 64, 128, 32, 2>(head, K, bt, 0, V, (int)Mp, K, epc, st)
                     : launch_mfma((const bf16_t *)hf, plain_map(lm_head, V, K), Mp, V, K, EpiNllCols8{part, Mp}, st)))
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
