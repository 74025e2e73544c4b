// Linear maps of a decode step with one row: every weight row is read once, by one wave, over the whole of K, so that
// a wave ends with finished outputs and what follows the product (rotary embedding and cache write, residual, SiLU(gate)*up)
// is done where the sum is: no partial sums in memory and four launches per layer less than with the K-split MFMA kernel
// (k_gemm_skinny, sol_gemm_mfma.hip), whose epilogues are kernels of their own.
// Bound: HBM (weights once) for the wide maps, launch and load latency for the narrow ones. A layer of a graph-replayed
// decode step with a cache of 300 keys (us, K-split MFMA kernel -> here): 1B shape 87.9 -> 66.7, 8B shape 144.5 -> 119.7;
// gate / up of the 1B shape: 12.6 us, 5.3 TB/s. More rows stay with the K-split kernel: with a template over rows this one
// was faster up to four (4 rows, 1B: 90.8 -> 81.9; 5: 92.1 -> 96.9), but batches of two to four then rounded unlike larger ones.
#include "sol_internal.h"

namespace sol {

typedef uint32_t u32x4_v __attribute__((ext_vector_type(4)));

enum GemvMode {
    GV_QKV,        // q / k / v: rotary on q and k heads, q -> out, K / V -> caches
    GV_RESID_F32,  // out (fp32) = aux (bf16) + product
    GV_SILU,       // out (bf16) = silu(w0 product) * (w1 product)
    GV_RESID_OUT,  // out (bf16) = aux (fp32) + product
    GV_F32         // out (fp32) = product
};

struct GemvArgs {
    const bf16_t *x;               // [K]
    int K, N;                      // N: outputs (GV_SILU: of one of the two maps)
    const bf16_t *w0, *w1, *w2;
    void *out;
    const void *aux;
    bf16_t *kc, *vc;               // GV_QKV only from here on
    const float2 *rope;
    const int32_t *pos0;
    int L_max, crows, Hq, Hkv, dh;
    int *flags;
};

constexpr int GV_KC = 2048;        // K chunk of the activations in LDS

// A wave takes two weight rows: the two of a rotary pair, gate and up of a channel, or two neighbouring outputs. Lane l
// holds k = 8 l .. 8 l + 7 of each 512-wide piece (1 KB of a row per load); the next chunk's eight loads are in flight
// while this one's are multiplied.
template <int MODE>
__global__ void __launch_bounds__(256)
k_gemv(GemvArgs a)
{
    __shared__ __align__(16) bf16_t xs[GV_KC];
    const int tid = threadIdx.x, lane = tid & 63;
    const int u = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (tid >> 6)));
    const int half = a.dh >> 1;
    // this wave's two rows
    const bf16_t *r0, *r1;
    int seg = 0, head = 0, c = 0;
    bool live;
    if (MODE == GV_QKV) {
        const int uq = a.Hq * half, uk = a.Hkv * half;
        live = u < uq + 2 * uk;
        seg = u < uq ? 0 : (u < uq + uk ? 1 : 2);
        const int v = live ? u - (seg == 0 ? 0 : (seg == 1 ? uq : uq + uk)) : 0;
        if (!live) seg = 0;
        const bf16_t *w = seg == 0 ? a.w0 : (seg == 1 ? a.w1 : a.w2);
        head = v / half;
        c = v - head * half;
        r0 = w + ((int64_t)head * a.dh + c) * a.K;
        r1 = r0 + (int64_t)half * a.K;
    } else {
        const int units = MODE == GV_SILU ? a.N : a.N / 2;
        live = u < units;
        const int v = live ? u : 0;
        r0 = a.w0 + (MODE == GV_SILU ? (int64_t)v : 2 * (int64_t)v) * a.K;
        r1 = MODE == GV_SILU ? a.w1 + (int64_t)v * a.K : r0 + a.K;
    }
    float s0 = 0.f, s1 = 0.f;
    u32x4_v wa[4], wb[4], na[4], nb[4];
    auto load = [&](int k0, u32x4_v (&p)[4], u32x4_v (&q)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int k = k0 + i * 512;
            if (k >= a.K) k = a.K - 512;                     // past the end: re-read, not multiplied
            p[i] = *reinterpret_cast<const u32x4_v *>(r0 + k + lane * 8);
            q[i] = *reinterpret_cast<const u32x4_v *>(r1 + k + lane * 8);
        }
    };
    load(0, wa, wb);
    for (int k0 = 0; k0 < a.K; k0 += GV_KC) {
        const int kw = a.K - k0 < GV_KC ? a.K - k0 : GV_KC;  // a multiple of 512
        __syncthreads();
        if (tid * 8 < kw) *reinterpret_cast<u32x4_v *>(&xs[tid * 8]) = *reinterpret_cast<const u32x4_v *>(a.x + k0 + tid * 8);
        if (k0 + GV_KC < a.K) load(k0 + GV_KC, na, nb);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i * 512 < kw) {
                const u32x4_v xv = *reinterpret_cast<const u32x4_v *>(&xs[i * 512 + lane * 8]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a0 = __uint_as_float(wa[i][e] << 16), a1 = __uint_as_float(wa[i][e] & 0xFFFF0000u);
                    const float b0 = __uint_as_float(wb[i][e] << 16), b1 = __uint_as_float(wb[i][e] & 0xFFFF0000u);
                    const float x0 = __uint_as_float(xv[e] << 16), x1 = __uint_as_float(xv[e] & 0xFFFF0000u);
                    s0 = __builtin_fmaf(a1, x1, __builtin_fmaf(a0, x0, s0));
                    s1 = __builtin_fmaf(b1, x1, __builtin_fmaf(b0, x0, s1));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) { wa[i] = na[i]; wb[i] = nb[i]; }
    }
    s0 = wave_sum_dpp(s0);
    s1 = wave_sum_dpp(s1);
    if (!live || lane != 0) return;
    if (MODE == GV_QKV) {
        const int pos = a.pos0 ? a.pos0[0] : 0;
        if (pos < 0 || pos + 1 > a.L_max) {                  // the sequence does not fit its cache: skipped
            if (u == 0) atomicOr(a.flags, FLAG_CACHE_OVERFLOW);
            return;
        }
        bf16_t *dst = seg == 0 ? (bf16_t *)a.out + head * a.dh : (seg == 1 ? a.kc : a.vc) + ((int64_t)head * a.crows + pos) * a.dh;
        if (seg < 2) {
            const float2 t = a.rope[(int64_t)pos * half + c];
            const float y0 = __builtin_fmaf(s0, t.x, -(s1 * t.y)), y1 = __builtin_fmaf(s1, t.x, s0 * t.y);
            s0 = y0; s1 = y1;
        }
        st(dst + c, s0);
        st(dst + c + half, s1);
    } else if (MODE == GV_SILU) {
        st((bf16_t *)a.out + u, (s0 / (1.0f + expf(-s0))) * s1);
    } else {
        const int o = 2 * u;
        if (MODE == GV_RESID_F32) {
            const uint32_t r = *reinterpret_cast<const uint32_t *>((const bf16_t *)a.aux + o);
            *reinterpret_cast<float2 *>((float *)a.out + o) = make_float2(__uint_as_float(r << 16) + s0, __uint_as_float(r & 0xFFFF0000u) + s1);
        } else if (MODE == GV_RESID_OUT) {
            const float2 r = *reinterpret_cast<const float2 *>((const float *)a.aux + o);
            *reinterpret_cast<uint32_t *>((bf16_t *)a.out + o) = pack_bf16x2(r.x + s0, r.y + s1);
        } else {
            *reinterpret_cast<float2 *>((float *)a.out + o) = make_float2(s0, s1);
        }
    }
}

template <int MODE>
static bool launch_gemv(const GemvArgs &a, int N, int units, hipStream_t st)
{
    if (a.K < 512 || a.K % 512 != 0 || N % 2 != 0) return false;
    hipLaunchKernelGGL(k_gemv<MODE>, dim3((unsigned)((units + 3) / 4)), dim3(256), 0, st, a);
    return true;
}

bool launch_gemv_qkv_rope(const void *h, const void *wq, const void *wk, const void *wv, void *q, void *kc, void *vc,
                          const float2 *rope, const int32_t *pos0, int L_max, int Hq, int Hkv, int dh, int d,
                          int *flags, hipStream_t st, int cache_rows)
{
    const GemvArgs a{(const bf16_t *)h, d, 0, (const bf16_t *)wq, (const bf16_t *)wk, (const bf16_t *)wv, q, nullptr,
                     (bf16_t *)kc, (bf16_t *)vc, rope, pos0, L_max, cache_rows > 0 ? cache_rows : L_max, Hq, Hkv, dh, flags};
    return launch_gemv<GV_QKV>(a, dh, (Hq + 2 * Hkv) * (dh / 2), st);
}

static GemvArgs plain_args(const void *x, int N, int K, const void *w0, const void *w1, void *out, const void *aux)
{
    return GemvArgs{(const bf16_t *)x, K, N, (const bf16_t *)w0, (const bf16_t *)w1, nullptr, out, aux,
                    nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0, 0, nullptr};
}

bool launch_gemv_resid_f32(const void *a, const void *w, const void *resid, float *out, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_RESID_F32>(plain_args(a, N, K, w, nullptr, out, resid), N, N / 2, st);
}

bool launch_gemv_gateup_silu(const void *h, const void *wg, const void *wu, void *a, int dff, int d, hipStream_t st)
{
    return launch_gemv<GV_SILU>(plain_args(h, dff, d, wg, wu, a, nullptr), dff, dff, st);
}

bool launch_gemv_resid_out(const void *a, const void *w, const float *x2, void *out, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_RESID_OUT>(plain_args(a, N, K, w, nullptr, out, x2), N, N / 2, st);
}

bool launch_gemv_f32(const void *a, const void *w, float *C, int N, int K, hipStream_t st)
{
    return launch_gemv<GV_F32>(plain_args(a, N, K, w, nullptr, C, nullptr), N, N / 2, st);
}

}  // namespace sol
