// Reward reduction after the teacher-forced pass (Method, "Actions and controlled compute", Eqs. 2-5, and
// "GRPO with per-sequence budget sampling"): from the NLL tensor [B][K][T] and the action ids to
//   - the realised compute averages of each schedule over its effective steps, the squared-hinge penalty,
//   - the discounted return-to-go of the task reward r_t = -nll_t, the signal r_t = G_t - C,
//   - advantages: mean-centred over the K schedules of an input at fixed t, whitened over the batch.
// Tiny and latency-bound: three short kernels, sums that decide the whitening and the return-to-go in fp64 and in a fixed order.
#include "sol_internal.h"

namespace sol {

constexpr int RW_BLOCK = 256;

__device__ __forceinline__ double block_sum_f64(double v, double *red)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < RW_BLOCK / 64; ++i) t += red[i];
    __syncthreads();
    return t;
}

// the same for four values behind one pair of barriers; red: [RW_BLOCK / 64][4]
__device__ __forceinline__ void block_sum4_f64(double (&v)[4], double *red)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], o, 64);
    if (lane == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[4 * w + e] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = 0.0;
#pragma unroll
        for (int i = 0; i < RW_BLOCK / 64; ++i) v[e] += red[4 * i + e];
    }
    __syncthreads();
}

// One workgroup per schedule (b, k), RW_TILE steps at a time from the last to the first. Return-to-go of a tile: a thread sums
// its RW_STEPS consecutive steps backwards, the threads' sums are folded by a suffix scan over the wave's lanes (a lane's
// distance is a constant number of steps, so the weights are powers of gamma) and over the four waves, then every thread
// runs its steps again from the carry of the steps behind them. All in fp64: one rounding per return.
// Bound: latency (loads, two scans, stores of one workgroup). The scan through one thread's 256 carries and three fp64 divisions
// per step took 15.7 us for rows of 2048 steps, this 8.6; the three kernels of 2 x 8 x 2048 steps 25 -> 16 us.
constexpr int RW_STEPS = 8, RW_TILE = RW_BLOCK * RW_STEPS;
constexpr int RW_TABLE = 512;                                       // actions whose rates fit the LDS (12 KB)
__global__ void __launch_bounds__(RW_BLOCK)
k_reward_rows(const float *__restrict__ nll, const int32_t *__restrict__ ids, const ActionDev *__restrict__ table,
              int n_actions, const int32_t *__restrict__ eff, const float *__restrict__ targets, RewardCfg rc, int K, int T,
              float *__restrict__ avg_out, float *__restrict__ pen_out, float *__restrict__ ret_out,
              float *__restrict__ signal, int *flags)
{
    __shared__ double red[RW_BLOCK / 64 * 4], s_rate[RW_TABLE * 3], s_wave[RW_BLOCK / 64];
    __shared__ float s_x[RW_TILE + RW_TILE / RW_STEPS];             // step i of the tile at i + i / RW_STEPS: no bank conflicts
    const int k = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t row = ((int64_t)b * K + k) * T;
    auto rate = [&](const ActionDev &a, int e) {
        return e == 0 ? (double)a.keep_num / (double)a.keep_den : e == 1 ? (double)a.mlp_keep_num / (double)a.mlp_keep_den
                                                                        : (double)(a.bits < 16u ? a.bits : 16u) / 16.0;
    };
    const int n_tiles = (T + RW_TILE - 1) / RW_TILE;
    float x[RW_STEPS];                                              // the last tile's values, requested first of all
    auto load_tile = [&](int tile) {
#pragma unroll
        for (int i = 0; i < RW_STEPS; ++i) {
            const int t = tile * RW_TILE + i * RW_BLOCK + tid;
            x[i] = t < T ? nll[row + t] : 0.f;
        }
    };
    load_tile(n_tiles - 1);
    const bool in_lds = n_actions <= RW_TABLE;
    if (in_lds) {
        for (int i = tid; i < n_actions; i += RW_BLOCK) {
            const ActionDev a = table[i];
#pragma unroll
            for (int e = 0; e < 3; ++e) s_rate[3 * i + e] = rate(a, e);
        }
        __syncthreads();
    }
    // ---- realised averages over the effective steps, penalty -------------------------------------
    double sum[4] = {0.0, 0.0, 0.0, 0.0};                           // keep rate, MLP keep rate, bits, steps
    bool bad = false;
#pragma unroll 8
    for (int t = tid; t < T; t += RW_BLOCK) {
        const int e = eff ? (eff[(int64_t)b * T + t] != 0) : 1;
        int id = ids[row + t];
        if (id < 0 || id >= n_actions) { bad = true; id = 0; }
        if (e) {
            if (in_lds) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sum[c] += s_rate[3 * id + c];
            } else {
                const ActionDev a = table[id];
#pragma unroll
                for (int c = 0; c < 3; ++c) sum[c] += rate(a, c);
            }
            sum[3] += 1.0;
        }
    }
    if (bad) atomicOr(flags, FLAG_BAD_ACTION);
    block_sum4_f64(sum, red);
    const double sn = sum[3];
    const float ck = targets[b * 3 + 0], cr = targets[b * 3 + 1], ce = targets[b * 3 + 2];
    const float ak = sn > 0.0 ? (float)(sum[0] / sn) : ck, ar = sn > 0.0 ? (float)(sum[1] / sn) : cr, ae = sn > 0.0 ? (float)(sum[2] / sn) : ce;
    auto psi = [&](float d) { const float v = fmaxf(0.f, fabsf(d) - rc.tau); return v * v; };
    const float pen = rc.alpha_kappa * psi(ak - ck) + rc.alpha_rho * psi(ar - cr) + rc.alpha_eta * psi(ae - ce);
    if (tid == 0) {
        if (avg_out) { float *o = avg_out + ((int64_t)b * K + k) * 3; o[0] = ak; o[1] = ar; o[2] = ae; }
        if (pen_out) pen_out[(int64_t)b * K + k] = pen;
    }
    // ---- return-to-go ---------------------------------------------------------------------------
    // weights stay above zero (gamma is, gamma^512 need not be): an infinite NLL makes every return before it infinite, and
    // what a weight of 2^-1022 adds to a finite one is far below its last place
    constexpr double W_MIN = 0x1p-1022;
    double gp[7];                                                   // gamma^(RW_STEPS * 2^i)
    {
        double g = (double)rc.gamma;
        for (int i = 1; i < RW_STEPS; i <<= 1) g *= g;
#pragma unroll
        for (int i = 0; i < 7; ++i) { gp[i] = fmax(g, W_MIN); g *= g; }
    }
    double tail = 1.0;                                              // gamma^(steps of the lanes behind this one)
#pragma unroll
    for (int i = 0; i < 6; ++i) tail *= ((63 - lane) >> i) & 1 ? gp[i] : 1.0;
    tail = fmax(tail, W_MIN);
    double behind = 0.0;                                            // return-to-go at the first step behind the tile
    for (int tile = n_tiles - 1; tile >= 0; --tile) {
        if (tile < n_tiles - 1) load_tile(tile);
#pragma unroll
        for (int i = 0; i < RW_STEPS; ++i) {
            const int c = i * RW_BLOCK + tid;
            s_x[c + c / RW_STEPS] = x[i];
        }
        __syncthreads();
        float *const mine = s_x + tid * (RW_STEPS + 1);
        double v = 0.0;
#pragma unroll
        for (int i = RW_STEPS - 1; i >= 0; --i) v = (double)rc.gamma * v - (double)mine[i];
#pragma unroll
        for (int i = 0; i < 6; ++i) {                               // v: the steps from this lane's first to the wave's last
            const double u = __shfl_down(v, 1 << i, 64);
            if (lane + (1 << i) < 64) v += gp[i] * u;
        }
        if (lane == 0) s_wave[w] = v;
        double g = __shfl_down(v, 1, 64);
        if (lane == 63) g = 0.0;
        __syncthreads();
        double c = behind;                                          // return-to-go at the first step behind the wave
#pragma unroll
        for (int i = RW_BLOCK / 64 - 1; i >= 0; --i) {
            if (i == w) g += tail * c;
            c = s_wave[i] + gp[6] * c;
        }
        behind = c;                                                 // of the tile
#pragma unroll
        for (int i = RW_STEPS - 1; i >= 0; --i) {
            g = (double)rc.gamma * g - (double)mine[i];
            mine[i] = (float)g;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RW_STEPS; ++i) {
            const int l = i * RW_BLOCK + tid, t = tile * RW_TILE + l;
            const float G = s_x[l + l / RW_STEPS];
            if (t < T) {
                if (ret_out) ret_out[row + t] = G;
                signal[row + t] = G - pen;
            }
        }
        __syncthreads();                                            // s_x and s_wave are free for the tile before
    }
}

// mean over the K schedules of an input at fixed t; writes the centred signal and per-workgroup partial sums
__global__ void __launch_bounds__(RW_BLOCK)
k_reward_center(const float *__restrict__ signal, int K, int T, float *__restrict__ adv, double *__restrict__ partial)
{
    __shared__ double red[RW_BLOCK / 64];
    const int b = blockIdx.y, t = blockIdx.x * RW_BLOCK + threadIdx.x;
    double s1 = 0.0, s2 = 0.0;
    if (t < T) {
        const float *p = signal + (int64_t)b * K * T + t;
        double m = 0.0;
#pragma unroll 8
        for (int k = 0; k < K; ++k) m += (double)p[(int64_t)k * T];
        m /= (double)K;
#pragma unroll 8
        for (int k = 0; k < K; ++k) {
            const double c = (double)p[(int64_t)k * T] - m;
            adv[(int64_t)b * K * T + (int64_t)k * T + t] = (float)c;
            s1 += c; s2 += c * c;
        }
    }
    s1 = block_sum_f64(s1, red); s2 = block_sum_f64(s2, red);
    if (threadIdx.x == 0) {
        double *o = partial + 2 * ((int64_t)blockIdx.y * gridDim.x + blockIdx.x);
        o[0] = s1; o[1] = s2;
    }
}

// every workgroup folds the partial sums in the same fixed order, then whitens its share
__global__ void __launch_bounds__(RW_BLOCK)
k_reward_whiten(float *__restrict__ adv, const double *__restrict__ partial, int n_partial, int64_t n, float eps)
{
    __shared__ double red[RW_BLOCK / 64];
    double s1 = 0.0, s2 = 0.0;
    for (int i = threadIdx.x; i < n_partial; i += RW_BLOCK) { s1 += partial[2 * i]; s2 += partial[2 * i + 1]; }
    s1 = block_sum_f64(s1, red); s2 = block_sum_f64(s2, red);
    const double mean = s1 / (double)n;
    double var = s2 / (double)n - mean * mean;
    var = var > 0.0 ? var : 0.0;
    const float mu = (float)mean, inv = (float)(1.0 / (sqrt(var) + (double)eps));
    for (int64_t i = (int64_t)blockIdx.x * RW_BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * RW_BLOCK)
        adv[i] = (adv[i] - mu) * inv;
}

size_t reward_scratch_bytes(int B, int T) { return (size_t)B * ((T + RW_BLOCK - 1) / RW_BLOCK) * 2 * sizeof(double) + 64; }

void launch_reward(const float *nll, const int32_t *ids, const ActionDev *table, int n_actions, const int32_t *eff,
                   const float *targets, const RewardCfg &rc, int B, int K, int T, float *avg_out, float *pen_out,
                   float *ret_out, float *signal, float *adv, void *scratch, int *flags, hipStream_t st)
{
    if ((int64_t)B * K * T <= 0) return;
    double *partial = (double *)scratch;
    const int tb = (T + RW_BLOCK - 1) / RW_BLOCK;
    hipLaunchKernelGGL(k_reward_rows, dim3(K, B), dim3(RW_BLOCK), 0, st, nll, ids, table, n_actions, eff, targets, rc, K, T,
                       avg_out, pen_out, ret_out, signal, flags);
    hipLaunchKernelGGL(k_reward_center, dim3(tb, B), dim3(RW_BLOCK), 0, st, signal, K, T, adv, partial);
    const int64_t n = (int64_t)B * K * T;
    int grid = (int)((n + RW_BLOCK * 4 - 1) / (RW_BLOCK * 4));
    grid = grid < 1 ? 1 : (grid > 1024 ? 1024 : grid);
    hipLaunchKernelGGL(k_reward_whiten, dim3(grid), dim3(RW_BLOCK), 0, st, adv, partial, tb * B, n, rc.eps);
}

}  // namespace sol
