// Linear maps of a decode step with one row. A wave ends with finished outputs, so that what follows the product (rotary
// embedding and cache write, residual, SiLU(gate)*up) is done where the sum is, and the norms where their result is read: no
// partial sums in memory and six launches per layer less than with the K-split kernel (k_gemm_skinny, sol_gemm_mfma.hip), whose
// epilogues are kernels of their own.
// The sums are those of that kernel, bit for bit: K is cut into the same splits, a split is the same chain of MFMAs, and the
// splits are added in order, so that a sequence decoded alone has the results it has among others.
// Bound: HBM (weights once) for the wide maps, launch and load latency for the narrow ones. A layer of a graph-replayed decode
// step with a cache of 300 keys (us, K-split kernel -> here): 1B shape 80.2 -> 60.7, 8B shape 133.9 -> 117.6, both before the
// norms came here (3 to 4 less); gate / up of the 1B shape: 14.8 us, 4.5 TB/s, 15.5 with its norm. (One fmaf chain per row took
// 58.7 and 113.3, but then a row rounded unlike the same row in a batch. Four blocks in registers in place of two or three: 1120 ->
// 1129 us for the 1B step.) More rows stay with the K-split kernel.
#include "sol_internal.h"

namespace sol {

typedef uint32_t u32x4_v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_v __attribute__((ext_vector_type(8)));
typedef float f32x16_v __attribute__((ext_vector_type(16)));

enum GemvMode {
    GV_QKV,        // q / k / v: rotary on q and k heads, q -> out, K / V -> caches
    GV_RESID_F32,  // out (fp32) = aux (bf16) + product
    GV_SILU,       // out (bf16) = silu(w0 product) * (w1 product)
    GV_RESID_OUT,  // out (bf16) = aux (fp32) + product
    GV_F32         // out (fp32) = product
};

struct GemvArgs {
    const bf16_t *x;               // [K]
    int K;
    const bf16_t *w0, *w1, *w2;
    void *out;
    const void *aux;
    int units;                     // pairs of weight rows
    int splits, kps;               // of K, and k per split (a multiple of 64)
    bf16_t *kc, *vc;               // GV_QKV only from here on
    const float2 *rope;
    const int32_t *pos0;
    int L_max, crows, Hq, Hkv, dh;
    int *flags;
    NormIn norm;                   // norm.x set: x is the RMS norm, quantised, of that row
};

// The matrix of a 32x32x16 MFMA holds 32 (weight row, split) pairs as its rows and the activations of the pairs' splits as
// its columns: the diagonal is the 32 partial sums, each the chain that k_gemm_skinny runs for it (k 32 h + 8 j .. + 7 of a
// 64-wide block in step j from lane half h). The other elements are not used: the matrix cores have 12 times the rate that
// the weights come at. SP: the splits, rounded up to a power of two (the surplus pairs repeat the last split and count as 0).
// A unit is two rows: the two of a rotary pair, gate and up of a channel, or two neighbouring outputs; a wave takes 16 / SP of
// them, or one in two matrices. Two blocks' loads (one with two matrices) are in flight while one is multiplied: 15.5 -> 14.8 us
// for gate / up of the 1B shape against one block. More units per wave (two matrices for every SP) took 16.0 us there, and
// activations from memory for every SP 18.3.
// NCH > 0: the activations are the RMS norm (and fake-quantiser) of a row of NCH * 512, bf16 for q / k / v and fp32 for gate /
// up. Every wave normalises the whole row, in the order of k_rmsnorm_fq_wave and with its bits, and brings every nw-th chunk
// of it to the LDS. The row is requested before the weights (loads return in order), whose first blocks arrive meanwhile.
// The norm's own kernels took 2.5 and 3.1 us per layer for a row of 2048: a decode step of the 1B model, 1307 -> 1252 us.
template <int MODE, int SP, int NCH>
__global__ void __launch_bounds__(256)
k_gemv(GemvArgs a)
{
    constexpr int NC = NCH > 0 ? NCH : 1, NP = MODE == GV_SILU ? 2 : 1;      // 16-byte pieces of the row per chunk and lane
    static_assert(NCH == 0 || (SP < 32 && (MODE == GV_QKV || MODE == GV_SILU)), "the normalised row goes through the LDS");
    constexpr bool XD = SP == 32;                            // activations straight from memory, each piece once per wave
    constexpr int NT = XD ? 2 : 1, UW = 16 * NT / SP;        // matrices and units of a wave
    constexpr int ND = XD ? 2 : 3;                           // blocks in registers
    extern __shared__ __align__(16) unsigned char xs[];      // activations, [block][j][h][SP] pieces of 8: a step's columns together
    __shared__ __align__(16) float fold[4][NT * 32];         // [unit][row of the pair][SP]
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int u0 = ((int)blockIdx.x * nw + w) * UW, half = a.dh >> 1;
    const int uq = MODE == GV_QKV ? a.Hq * half : 0, uk = MODE == GV_QKV ? a.Hkv * half : 0;
    const bf16_t *row[NT];                                   // this lane's weight rows from its split and half on
    {
        const int sp = r % SP, off = (sp < a.splits ? sp : a.splits - 1) * a.kps + h * 32;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int q = (t * 32 + r) / SP, which = q & 1;
            int u = u0 + (q >> 1);
            if (u >= a.units) u = a.units - 1;               // past the end: the last unit again, never stored
            if (MODE == GV_QKV) {                            // the pair (c, c + half) of a head of q, k or v
                const bf16_t *m = u < uq ? a.w0 : (u < uq + uk ? a.w1 : a.w2);
                const int v = u < uq ? u : (u < uq + uk ? u - uq : u - uq - uk), head = v / half;
                row[t] = m + ((int64_t)head * a.dh + (v - head * half) + which * half) * a.K;
            } else if (MODE == GV_SILU) {
                row[t] = (which ? a.w1 : a.w0) + (int64_t)u * a.K;
            } else {
                row[t] = a.w0 + (2 * (int64_t)u + which) * a.K;
            }
            row[t] += off;
        }
    }
    u32x4_w nx[NC * NP], nwt[NC];                            // the row to normalise, raw, and the norm's weights
    int nbits = 16;
    if constexpr (NCH > 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
                nx[c * NP + p] = *reinterpret_cast<const u32x4_w *>((const unsigned char *)a.norm.x + (size_t)(c * 64 + lane) * 16 * NP + p * 16);
            nwt[c] = *reinterpret_cast<const u32x4_w *>((const bf16_t *)a.norm.w + c * 512 + lane * 8);
        }
        if (a.norm.ra) nbits = a.norm.ra[0].bits;
        __builtin_amdgcn_sched_barrier(0);
    }
    const int nblk = a.kps / 64;
    struct Set { u32x4_v w[NT][4], x[XD ? 4 : 1]; } set[ND];         // blocks in flight
    const bf16_t *const xg = a.x + (r % SP < a.splits ? r % SP : a.splits - 1) * a.kps + h * 32;
    auto load = [&](int blk, Set &s) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int t = 0; t < NT; ++t) s.w[t][j] = *reinterpret_cast<const u32x4_v *>(row[t] + blk * 64 + j * 8);
            if (XD) s.x[j] = *reinterpret_cast<const u32x4_v *>(xg + blk * 64 + j * 8);
        }
    };
#pragma unroll
    for (int d = 0; d + 1 < ND; ++d)
        if (d < nblk) load(d, set[d]);
    if constexpr (NCH > 0) __builtin_amdgcn_sched_barrier(0);
    // what the outputs of this lane's unit will need
    const int u = u0 + lane;
    const bool mine = lane < UW && u < a.units;
    int pos = 0, head = 0, c = 0, seg = 0;
    float2 cs = {1.f, 0.f}, res = {0.f, 0.f};
    if (MODE == GV_QKV) {
        pos = a.pos0 ? a.pos0[0] : 0;
        const int uu = mine ? u : 0;
        seg = uu < uq ? 0 : (uu < uq + uk ? 1 : 2);
        const int v = seg == 0 ? uu : (seg == 1 ? uu - uq : uu - uq - uk);
        head = v / half;
        c = v - head * half;
        if (pos < 0 || pos + 1 > a.L_max) {                  // the sequence does not fit its cache: skipped, by all waves alike
            if (u == 0) atomicOr(a.flags, FLAG_CACHE_OVERFLOW);
            return;
        }
        cs = a.rope[(int64_t)pos * half + c];
    } else if (MODE == GV_RESID_F32) {
        const uint32_t x = mine ? *reinterpret_cast<const uint32_t *>((const bf16_t *)a.aux + 2 * u) : 0u;
        res = make_float2(__uint_as_float(x << 16), __uint_as_float(x & 0xFFFF0000u));
    } else if (MODE == GV_RESID_OUT) {
        if (mine) res = *reinterpret_cast<const float2 *>((const float *)a.aux + 2 * u);
    }
    if (!XD) {
        const int pps = a.kps / 8;                           // pieces per split
        auto slot = [&](int i) {                             // of piece i in the LDS
            const int sp = i / pps, p = i - sp * pps;        // p = block * 8 + h * 4 + j
            return reinterpret_cast<u32x4_v *>(xs + (size_t)((((p >> 3) * 4 + (p & 3)) * 2 + ((p >> 2) & 1)) * SP + sp) * 16);
        };
        if constexpr (NCH > 0) {
            float v[NC][8];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (NP == 2) v[c][e] = __uint_as_float(nx[c * NP + (e >> 2)][e & 3]);
                    else v[c][e] = __uint_as_float(e & 1 ? nx[c][e >> 1] & 0xFFFF0000u : nx[c][e >> 1] << 16);
                }
            const float amax = wave_norm_row<NC>(v, [&](int c) { return nwt[c]; }, a.norm.eps);
            wave_fq_row<NC>(v, amax, nbits);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (c % nw != w) continue;
                u32x4_v o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = pack_bf16x2(v[c][2 * e], v[c][2 * e + 1]);
                *slot(c * 64 + lane) = o;
            }
        } else {
            for (int i = tid; i < a.K / 8; i += blockDim.x) *slot(i) = *reinterpret_cast<const u32x4_v *>(a.x + (int64_t)i * 8);
        }
        __syncthreads();
    }
    f32x16_v acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    const unsigned char *const xl = xs + (h * SP + r % SP) * 16;
    auto multiply = [&](int blk, const Set &s) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32x4_v xv = XD ? s.x[XD ? j : 0] : *reinterpret_cast<const u32x4_v *>(xl + (size_t)(blk * 4 + j) * 2 * SP * 16);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_v, s.w[t][j]), __builtin_bit_cast(bf16x8_v, xv), acc[t], 0, 0, 0);
        }
    };
    for (int b0 = 0; b0 < nblk; b0 += ND) {
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            const int blk = b0 + d;
            if (blk + ND - 1 < nblk) load(blk + ND - 1, set[(d + ND - 1) % ND]);
            if (blk < nblk) multiply(blk, set[d]);
        }
    }
    // the diagonal: element (r, r) is element 4 * (r / 8) + r % 4 of lane (r, h = (r / 4) % 2)
    if (h == ((r >> 2) & 1)) {
        const int at = 4 * (r >> 3) + (r & 3);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float v = acc[t][0];
#pragma unroll
            for (int i = 1; i < 16; ++i) v = at == i ? acc[t][i] : v;
            fold[w][t * 32 + r] = r % SP < a.splits ? v : 0.f;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read by this wave only
    if (!mine) return;
    float y[2];                                              // the splits in order, from 0 on, as the K-split kernel's consumers add them
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float *f = &fold[w][(lane * 2 + t) * SP];
        float v = 0.f;
#pragma unroll
        for (int sp = 0; sp < SP; ++sp) v += f[sp];
        y[t] = v;
    }
    if (MODE == GV_QKV) {
        bf16_t *dst = seg == 0 ? (bf16_t *)a.out + head * a.dh : (seg == 1 ? a.kc : a.vc) + ((int64_t)head * a.crows + pos) * a.dh;
        if (seg < 2) {
            const float2 z = rotate_pair(y[0], y[1], cs);
            y[0] = z.x; y[1] = z.y;
        }
        st(dst + c, y[0]);
        st(dst + c + half, y[1]);
    } else if (MODE == GV_SILU) {
        st((bf16_t *)a.out + u, silu_mul(y[0], y[1]));
    } else if (MODE == GV_RESID_OUT) {
        *reinterpret_cast<uint32_t *>((bf16_t *)a.out + 2 * u) = pack_bf16x2(res.x + y[0], res.y + y[1]);
    } else {                                                 // (GV_F32: the products themselves)
        if (MODE == GV_RESID_F32) { y[0] = res.x + y[0]; y[1] = res.y + y[1]; }
        *reinterpret_cast<float2 *>((float *)a.out + 2 * u) = make_float2(y[0], y[1]);
    }
}

template <int MODE, int SP, int NCH>
static bool launch_gemv_sp(const GemvArgs &a, hipStream_t st)
{
    const size_t lds = SP == 32 ? 0 : 2 * (size_t)a.kps * SP;
    if (lds > (62u << 10)) return false;
    constexpr int UW = SP == 32 ? 1 : 16 / SP;               // as in the kernel
    const int waves = (a.units + UW - 1) / UW, cus = device_cus() > 0 ? device_cus() : 256;
    const int nw = waves >= 4 * cus ? 4 : (waves + cus - 1) / cus;   // up to four waves in a workgroup, all CUs first
    hipLaunchKernelGGL((k_gemv<MODE, SP, NCH>), dim3((unsigned)((waves + nw - 1) / nw)), dim3(64 * nw), lds, st, a);
    return true;
}

// Nv: the width that the K-split kernel would be called with (all stacked maps)
template <int MODE, int NCH>
static bool launch_gemv_ch(GemvArgs a, int Nv, hipStream_t st)
{
    if (Nv <= 0 || Nv % 4 || a.K < 64 || a.K % 64) return false;
    a.units = Nv / 2;
    a.splits = skinny_splits(1, Nv, a.K);
    if (a.K % a.splits) return false;
    a.kps = a.K / a.splits;
    if (a.kps % 64) return false;
    if (a.splits <= 2) return launch_gemv_sp<MODE, 2, NCH>(a, st);
    if (a.splits <= 4) return launch_gemv_sp<MODE, 4, NCH>(a, st);
    if (a.splits <= 8) return launch_gemv_sp<MODE, 8, NCH>(a, st);
    if (a.splits <= 16) return launch_gemv_sp<MODE, 16, NCH>(a, st);
    if constexpr (NCH == 0) return a.splits <= 32 && launch_gemv_sp<MODE, 32, 0>(a, st);
    return false;                                            // (32 splits take the activations from memory)
}

template <int MODE>
static bool launch_gemv(const GemvArgs &a, int Nv, hipStream_t st)
{
    if (!a.norm.x) return launch_gemv_ch<MODE, 0>(a, Nv, st);
    if constexpr (MODE == GV_QKV || MODE == GV_SILU) {       // the widths of k_rmsnorm_fq_wave
        if (a.K == 2048) return launch_gemv_ch<MODE, 4>(a, Nv, st);
        if (a.K == 4096) return launch_gemv_ch<MODE, 8>(a, Nv, st);
    }
    return false;
}

bool launch_gemv_qkv_rope(const void *h, const void *wq, const void *wk, const void *wv, void *q, void *kc, void *vc,
                          const float2 *rope, const int32_t *pos0, int L_max, int Hq, int Hkv, int dh, int d,
                          int *flags, hipStream_t st, int cache_rows, const NormIn *norm)
{
    const GemvArgs a{(const bf16_t *)h, d, (const bf16_t *)wq, (const bf16_t *)wk, (const bf16_t *)wv, q, nullptr, 0, 0, 0,
                     (bf16_t *)kc, (bf16_t *)vc, rope, pos0, L_max, cache_rows > 0 ? cache_rows : L_max, Hq, Hkv, dh, flags,
                     norm ? *norm : NormIn{}};
    return dh % 2 == 0 && launch_gemv<GV_QKV>(a, (Hq + 2 * Hkv) * dh, st);
}

static GemvArgs plain_args(const void *x, int K, const void *w0, const void *w1, void *out, const void *aux)
{
    return GemvArgs{(const bf16_t *)x, K, (const bf16_t *)w0, (const bf16_t *)w1, nullptr, out, aux, 0, 0, 0,
                    nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0, 0, nullptr, NormIn{}};
}

bool launch_gemv_resid_f32(const void *a, const void *w, const void *resid, float *out, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_RESID_F32>(plain_args(a, K, w, nullptr, out, resid), N, st);
}

bool launch_gemv_gateup_silu(const void *h, const void *wg, const void *wu, void *a, int dff, int d, hipStream_t st, const NormIn *norm)
{
    GemvArgs g = plain_args(h, d, wg, wu, a, nullptr);
    if (norm) g.norm = *norm;
    return launch_gemv<GV_SILU>(g, 2 * dff, st);
}

bool launch_gemv_resid_out(const void *a, const void *w, const float *x2, void *out, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_RESID_OUT>(plain_args(a, K, w, nullptr, out, x2), N, st);
}

bool launch_gemv_f32(const void *a, const void *w, float *C, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_F32>(plain_args(a, K, w, nullptr, C, nullptr), N, st);
}

}  // namespace sol
