// Linear maps of a decode step with very few rows: every weight row is read once, by one wave, over the whole of K, so that
// a wave ends with finished outputs and what follows the product (rotary embedding and cache write, residual, SiLU(gate)*up)
// is done where the sum is: no partial sums in memory and four launches per layer less than with the K-split MFMA kernel
// (k_gemm_skinny, sol_gemm_mfma.hip), whose epilogues are kernels of their own.
// Bound: HBM (weights once) for the wide maps, launch and load latency for the narrow ones; the vector pipes spend
// 1 + rows instructions per weight, which is what limits the row count (see gemv_rows_ok).
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
    const bf16_t *x;               // [M][K]
    int M, K, N;                   // N: outputs per row (GV_SILU: of one of the two maps)
    const bf16_t *w0, *w1, *w2;
    void *out;
    const void *aux;
    bf16_t *kc, *vc;               // GV_QKV only from here on
    const float2 *rope;
    const int32_t *pos0;
    int T, L_max, crows, Hq, Hkv, dh;
    int *flags;
};

constexpr int GV_KC = 2048;        // K chunk of the activations in LDS

// A wave takes two weight rows: the two of a rotary pair, gate and up of a channel, or two neighbouring outputs. Lane l
// holds k = 8 l .. 8 l + 7 of each 512-wide piece (1 KB of a row per load); the next chunk's eight loads are in flight
// while this one's are multiplied.
template <int MB, int MODE>
__global__ void __launch_bounds__(256)
k_gemv(GemvArgs a)
{
    __shared__ __align__(16) bf16_t xs[MB][GV_KC];
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
    float acc0[MB], acc1[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) acc0[m] = acc1[m] = 0.f;
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
#pragma unroll
        for (int m = 0; m < MB; ++m)
            if (tid * 8 < kw) {
                u32x4_v v = {0u, 0u, 0u, 0u};
                if (m < a.M) v = *reinterpret_cast<const u32x4_v *>(a.x + (int64_t)m * a.K + k0 + tid * 8);
                *reinterpret_cast<u32x4_v *>(&xs[m][tid * 8]) = v;
            }
        if (k0 + GV_KC < a.K) load(k0 + GV_KC, na, nb);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i * 512 < kw) {
                u32x4_v xv[MB];
#pragma unroll
                for (int m = 0; m < MB; ++m) xv[m] = *reinterpret_cast<const u32x4_v *>(&xs[m][i * 512 + lane * 8]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a0 = __uint_as_float(wa[i][e] << 16), a1 = __uint_as_float(wa[i][e] & 0xFFFF0000u);
                    const float b0 = __uint_as_float(wb[i][e] << 16), b1 = __uint_as_float(wb[i][e] & 0xFFFF0000u);
#pragma unroll
                    for (int m = 0; m < MB; ++m) {
                        const float x0 = __uint_as_float(xv[m][e] << 16), x1 = __uint_as_float(xv[m][e] & 0xFFFF0000u);
                        acc0[m] = __builtin_fmaf(a1, x1, __builtin_fmaf(a0, x0, acc0[m]));
                        acc1[m] = __builtin_fmaf(b1, x1, __builtin_fmaf(b0, x0, acc1[m]));
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) { wa[i] = na[i]; wb[i] = nb[i]; }
    }
    // lane m keeps row m's two sums
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const float t0 = wave_sum_dpp(acc0[m]), t1 = wave_sum_dpp(acc1[m]);
        if (lane == m) { s0 = t0; s1 = t1; }
    }
    const int m = lane;
    if (!live || m >= a.M) return;
    if (MODE == GV_QKV) {
        const int s = m / a.T, i = m - s * a.T;
        const int p0 = a.pos0 ? a.pos0[s] : 0;
        if (p0 < 0 || p0 + a.T > a.L_max) {                  // the sequence does not fit its cache: skipped
            if (u == 0) atomicOr(a.flags, FLAG_CACHE_OVERFLOW);
            return;
        }
        const int pos = p0 + i;
        bf16_t *dst = seg == 0 ? (bf16_t *)a.out + (int64_t)m * a.Hq * a.dh + head * a.dh
                               : (seg == 1 ? a.kc : a.vc) + (((int64_t)s * a.Hkv + head) * a.crows + pos) * a.dh;
        if (seg < 2) {
            const float2 t = a.rope[(int64_t)pos * half + c];
            const float y0 = __builtin_fmaf(s0, t.x, -(s1 * t.y)), y1 = __builtin_fmaf(s1, t.x, s0 * t.y);
            s0 = y0; s1 = y1;
        }
        st(dst + c, s0);
        st(dst + c + half, s1);
    } else if (MODE == GV_SILU) {
        st((bf16_t *)a.out + (int64_t)m * a.N + u, (s0 / (1.0f + expf(-s0))) * s1);
    } else {
        const int64_t o = (int64_t)m * a.N + 2 * u;
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
static void launch_gemv(const GemvArgs &a, int units, hipStream_t st)
{
    const dim3 grid((unsigned)((units + 3) / 4));
    if (a.M == 1) hipLaunchKernelGGL((k_gemv<1, MODE>), grid, dim3(256), 0, st, a);
    else if (a.M == 2) hipLaunchKernelGGL((k_gemv<2, MODE>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_gemv<4, MODE>), grid, dim3(256), 0, st, a);
}

// A layer of a graph-replayed decode step with caches of 300 keys (us), K-split MFMA kernel -> here: 1B shape, 1 row
// 87.9 -> 66.7, 2 rows 90.0 -> 70.7, 3: 90.6 -> 79.9, 4: 90.8 -> 81.9, 5: 92.1 -> 96.9, 8: 92.6 -> 103; 8B shape, 1 row 144.5 ->
// 119.7, 4: 153.4 -> 149.6, 5: 158.7 -> 174.4. Gate / up of the 1B shape, one row: 12.6 us, 5.3 TB/s.
bool gemv_rows_ok(int64_t M) { return M >= 1 && M <= GEMV_MAX_ROWS; }

static bool gemv_shape_ok(int64_t M, int N, int K) { return gemv_rows_ok(M) && K >= 512 && K % 512 == 0 && N % 2 == 0; }

bool launch_gemv_qkv_rope(const void *h, const void *wq, const void *wk, const void *wv, void *q, void *kc, void *vc,
                          const float2 *rope, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh, int d,
                          int *flags, hipStream_t st, int cache_rows)
{
    const int64_t M = (int64_t)n_seq * T;
    if (!gemv_shape_ok(M, dh, d)) return false;
    GemvArgs a{(const bf16_t *)h, (int)M, d, 0, (const bf16_t *)wq, (const bf16_t *)wk, (const bf16_t *)wv, q, nullptr,
               (bf16_t *)kc, (bf16_t *)vc, rope, pos0, T, L_max, cache_rows > 0 ? cache_rows : L_max, Hq, Hkv, dh, flags};
    launch_gemv<GV_QKV>(a, (Hq + 2 * Hkv) * (dh / 2), st);
    return true;
}

static GemvArgs plain_args(const void *x, int64_t M, int N, int K, const void *w0, const void *w1, void *out, const void *aux)
{
    return GemvArgs{(const bf16_t *)x, (int)M, K, N, (const bf16_t *)w0, (const bf16_t *)w1, nullptr, out, aux,
                    nullptr, nullptr, nullptr, nullptr, 1, 0, 0, 0, 0, 0, nullptr};
}

bool launch_gemv_resid_f32(const void *a, const void *w, const void *resid, float *out, int64_t M, int N, int K, hipStream_t st)
{
    if (!gemv_shape_ok(M, N, K)) return false;
    launch_gemv<GV_RESID_F32>(plain_args(a, M, N, K, w, nullptr, out, resid), N / 2, st);
    return true;
}

bool launch_gemv_gateup_silu(const void *h, const void *wg, const void *wu, void *a, int64_t M, int dff, int d, hipStream_t st)
{
    if (!gemv_shape_ok(M, dff, d)) return false;
    launch_gemv<GV_SILU>(plain_args(h, M, dff, d, wg, wu, a, nullptr), dff, st);
    return true;
}

bool launch_gemv_resid_out(const void *a, const void *w, const float *x2, void *out, int64_t M, int N, int K, hipStream_t st)
{
    if (!gemv_shape_ok(M, N, K)) return false;
    launch_gemv<GV_RESID_OUT>(plain_args(a, M, N, K, w, nullptr, out, x2), N / 2, st);
    return true;
}

bool launch_gemv_f32(const void *a, const void *w, float *C, int64_t M, int N, int K, hipStream_t st)
{
    if (!gemv_shape_ok(M, N, K)) return false;
    launch_gemv<GV_F32>(plain_args(a, M, N, K, w, nullptr, C, nullptr), N / 2, st);
    return true;
}

}  // namespace sol
