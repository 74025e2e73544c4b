// Attention with per-query budgeted key selection.
//
// k_attn_rows: one workgroup per (query row, group of HPB query heads that share a KV head).
//   1. scores s_j = (q . k_j) / sqrt(dh) over the allowed cache positions j in [0, pos]   -> LDS (fp32)
//   2. budget b = ceil(kappa * n); b < n: exact b-th largest score by radix select, ties to the
//      lower position; b = n: dense
//   3. softmax over the kept keys (dropped keys contribute exp(-inf) = 0)
//   4. o = sum_j p_j v_j, reading only V rows kept by at least one of the HPB heads
// K is streamed once per workgroup (HPB heads share it), V rows are gathered. This is the any-shape /
// fp32 path, and the only one that knows the other key-selection rules of the method (Appendix "Quest
// masking"):
//   - sink / window keys: the first n_sink and the last n_window allowed keys are always kept and
//     count against the budget (the selection sees them with the largest possible key);
//   - pages of S > 1 contiguous keys: a page's score is the upper bound sum_c max(q_c max_c, q_c min_c)
//     over the channel-wise extremes of its allowed keys; the top ceil(b / S) pages are kept whole
//     (ties to the lower page) together with the forced keys.
#include <type_traits>
#include "sol_internal.h"

namespace sol {

struct ScoreKeyLds {
    const float *row;
    __device__ __forceinline__ uint32_t operator()(int i) const { return score_key(row[i]); }
};

// selection key of key j when keys [0, sink_end) and [win_begin, n) are forced
struct ForcedKeyLds {
    const float *row;
    int sink_end, win_begin;
    __device__ __forceinline__ uint32_t operator()(int i) const
    {
        return (i < sink_end || i >= win_begin) ? 0xFFFFFFFFu : score_key(row[i]);
    }
};

template <typename T, int HPB, int BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_attn_rows(const T *__restrict__ q, const T *__restrict__ kc, const T *__restrict__ vc, float *__restrict__ o32,
            const RowAct *__restrict__ ra, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hq, int Hkv,
            int dh, int lpad, float scale, int *flags, AttnOpts opt, int ppad)
{
    constexpr int VEC = Vec16<T>::N;
    constexpr int NW = BLOCK / 64;
    extern __shared__ float smem[];
    float *sc = smem;                               // [HPB][lpad]
    float *ored = smem + (size_t)HPB * lpad;        // [NW][HPB][dh]
    float *pgs = ored + (size_t)NW * HPB * dh;      // [HPB][ppad] page scores (page size > 1 only)
    __shared__ int hist[256];
    __shared__ int sh[4];
    __shared__ int wcnt[NW];
    __shared__ float red[NW];

    const int tid = threadIdx.x;
    const int64_t r = blockIdx.y;
    const int s = (int)(r / Tn), i = (int)(r % Tn);
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) {               // the sequence does not fit its cache: skipped
        if (tid == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
        return;
    }
    const int n = p0 + i + 1;                       // allowed keys 0..pos, self included
    const int h0 = blockIdx.x * HPB;
    const int kvh = h0 / (Hq / Hkv);
    const T *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * dh;
    const T *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * dh;
    const int lpk = dh / VEC;                       // lanes per key (power of two, <= 64)
    const int kpi = BLOCK / lpk;                    // keys per block iteration
    const int ks = tid / lpk, cs = tid - ks * lpk;

    // ---- 1. scores -------------------------------------------------------------------------
    float qf[HPB][VEC];
#pragma unroll
    for (int h = 0; h < HPB; ++h) {
        Vec16<T> v;
        v.load(q + r * (int64_t)(Hq * dh) + (int64_t)(h0 + h) * dh + cs * VEC);
        v.unpack(qf[h]);
    }
    for (int j0 = 0; j0 < n; j0 += kpi) {
        const int j = j0 + ks;
        float part[HPB];
#pragma unroll
        for (int h = 0; h < HPB; ++h) part[h] = 0.f;
        if (j < n) {
            Vec16<T> kv;
            kv.load(kbase + (int64_t)j * dh + cs * VEC);
            float kf[VEC];
            kv.unpack(kf);
#pragma unroll
            for (int h = 0; h < HPB; ++h)
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[h] = fmaf(qf[h][e], kf[e], part[h]);
        }
        for (int o = lpk >> 1; o > 0; o >>= 1)
#pragma unroll
            for (int h = 0; h < HPB; ++h) part[h] += __shfl_xor(part[h], o, 64);
        if (cs == 0 && j < n)
#pragma unroll
            for (int h = 0; h < HPB; ++h) sc[h * lpad + j] = part[h] * scale;
    }
    const RowAct act = ra[r];
    const int b = budget_ceil(act.keep_num, act.keep_den, n);
    const int S = opt.page;
    const int n_pages = (n + S - 1) / S;
    if (S > 1 && b < n) {
        // ---- 1b. page bounds: a group of lpk lanes walks the allowed keys of one page --------------
        for (int u0 = 0; u0 < n_pages; u0 += kpi) {
            const int u = u0 + ks;
            float part[HPB];
#pragma unroll
            for (int h = 0; h < HPB; ++h) part[h] = 0.f;
            if (u < n_pages) {
                const int j0 = u * S, j1 = (j0 + S < n) ? j0 + S : n;
                float kmx[VEC], kmn[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) { kmx[e] = -INFINITY; kmn[e] = INFINITY; }
                for (int j = j0; j < j1; ++j) {
                    Vec16<T> kv;
                    kv.load(kbase + (int64_t)j * dh + cs * VEC);
                    float kf[VEC];
                    kv.unpack(kf);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) { kmx[e] = fmaxf(kmx[e], kf[e]); kmn[e] = fminf(kmn[e], kf[e]); }
                }
#pragma unroll
                for (int h = 0; h < HPB; ++h)
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        part[h] = fmaf(qf[h][e], qf[h][e] >= 0.f ? kmx[e] : kmn[e], part[h]);
            }
            for (int o = lpk >> 1; o > 0; o >>= 1)
#pragma unroll
                for (int h = 0; h < HPB; ++h) part[h] += __shfl_xor(part[h], o, 64);
            if (cs == 0 && u < n_pages)
#pragma unroll
                for (int h = 0; h < HPB; ++h) pgs[h * ppad + u] = part[h];
        }
    }
    __syncthreads();

    // ---- 2 + 3. selection and softmax numerators, head by head ------------------------------
    // forced keys: [0, sink_end) and [win_begin, n)
    const int sink_end = opt.n_sink < n ? opt.n_sink : n;
    int win_begin = n - opt.n_window;
    win_begin = win_begin < sink_end ? sink_end : win_begin;
    const int forced = sink_end + (n - win_begin);
    float inv_den[HPB];
#pragma unroll
    for (int h = 0; h < HPB; ++h) {
        float *row = sc + h * lpad;
        uint32_t thr = 0u; int J = n;                // by key (S = 1) or by page (S > 1): kept if above thr, or tied and <= J
        if (b < n) {
            int quota, n_eq;
            if (S > 1) {
                ScoreKeyLds kf{pgs + h * ppad};
                int np = (b + S - 1) / S;
                np = np < n_pages ? np : n_pages;
                J = n_pages;
                if (np < n_pages) {
                    block_radix_select<BLOCK>(kf, n_pages, np, hist, sh, thr, quota, n_eq);
                    if (quota < n_eq) J = block_tie_cutoff<BLOCK>(kf, n_pages, thr, quota, wcnt, sh);
                }
            } else if (forced == 0) {
                ScoreKeyLds kf{row};
                block_radix_select<BLOCK>(kf, n, b, hist, sh, thr, quota, n_eq);
                if (quota < n_eq) J = block_tie_cutoff<BLOCK>(kf, n, thr, quota, wcnt, sh);
            } else if (forced < n) {                 // forced keys rank first; the rest of the budget goes by score
                ForcedKeyLds kf{row, sink_end, win_begin};
                const int bb = b > forced ? b : forced;
                block_radix_select<BLOCK>(kf, n, bb, hist, sh, thr, quota, n_eq);
                if (quota < n_eq) J = block_tie_cutoff<BLOCK>(kf, n, thr, quota, wcnt, sh);
            }
        }
        auto kept = [&](int j, float sv) -> bool {
            if (b >= n) return true;
            const bool f = j < sink_end || j >= win_begin;
            if (S > 1) {
                const int u = j / S;
                const uint32_t key = score_key(pgs[h * ppad + u]);
                return f || key > thr || (key == thr && u <= J);
            }
            const uint32_t key = f ? 0xFFFFFFFFu : score_key(sv);
            return key > thr || (key == thr && j <= J);
        };
        float mx = -INFINITY;                        // over the kept keys (the best key may be dropped with its page)
        for (int j = tid; j < n; j += BLOCK) {
            const float sv = row[j];
            if (kept(j, sv)) mx = fmaxf(mx, sv);
        }
        mx = block_max<BLOCK>(mx, red);
        float den = 0.f;
        for (int j = tid; j < n; j += BLOCK) {
            const float sv = row[j];
            const float p = kept(j, sv) ? expf(sv - mx) : 0.f;
            row[j] = p;
            den += p;
        }
        den = block_sum<BLOCK>(den, red);
        inv_den[h] = 1.0f / den;
    }
    __syncthreads();

    // ---- 4. o = sum p_j v_j over rows any head kept --------------------------------------------
    float acc[HPB][VEC];
#pragma unroll
    for (int h = 0; h < HPB; ++h)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[h][e] = 0.f;
    for (int j = ks; j < n; j += kpi) {
        float p[HPB];
        bool any = false;
#pragma unroll
        for (int h = 0; h < HPB; ++h) { p[h] = sc[h * lpad + j]; any |= (p[h] != 0.f); }
        if (!any) continue;
        Vec16<T> vv;
        vv.load(vbase + (int64_t)j * dh + cs * VEC);
        float vf[VEC];
        vv.unpack(vf);
#pragma unroll
        for (int h = 0; h < HPB; ++h)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[h][e] = fmaf(p[h], vf[e], acc[h][e]);
    }
    // reduce over the key slots of a wave (lanes with equal cs), then across waves in fixed order
    for (int o = lpk; o < 64; o <<= 1)
#pragma unroll
        for (int h = 0; h < HPB; ++h)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[h][e] += __shfl_xor(acc[h][e], o, 64);
    const int w = tid >> 6, lane = tid & 63;
    if (lane < lpk) {
#pragma unroll
        for (int h = 0; h < HPB; ++h)
#pragma unroll
            for (int e = 0; e < VEC; ++e) ored[((size_t)w * HPB + h) * dh + lane * VEC + e] = acc[h][e];
    }
    __syncthreads();
    for (int idx = tid; idx < HPB * dh; idx += BLOCK) {
        const int h = idx / dh;
        float t = 0.f;
        for (int ww = 0; ww < NW; ++ww) t += ored[(size_t)ww * HPB * dh + idx];
        float id = inv_den[0];
#pragma unroll
        for (int hh = 1; hh < HPB; ++hh) if (h == hh) id = inv_den[hh];
        o32[r * (int64_t)(Hq * dh) + (int64_t)h0 * dh + idx] = t * id;
    }
}

template <typename T, int HPB, int BLOCK>
static bool launch_attn_rows_t(const void *q, const void *kc, const void *vc, float *o32, const RowAct *ra,
                               const int32_t *pos0, int n_seq, int Tn, int L_max, int Hq, int Hkv, int dh, int lpad,
                               size_t lds, int *flags, AttnOpts opt, int ppad, hipStream_t st)
{
    auto kern = k_attn_rows<T, HPB, BLOCK>;
    if (lds > 48 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return false;
    }
    const float scale = 1.0f / sqrtf((float)dh);
    hipLaunchKernelGGL(kern, dim3(Hq / HPB, (unsigned)((int64_t)n_seq * Tn)), dim3(BLOCK), lds, st, (const T *)q,
                       (const T *)kc, (const T *)vc, o32, ra, pos0, Tn, L_max, Hq, Hkv, dh, lpad, scale, flags, opt, ppad);
    return true;
}

static bool launch_attn_f32(const float *q, const float *kc, const float *vc, float *o32, const RowAct *ra, const int32_t *pos0,
                            int n_seq, int T, int L_max, int Hq, int Hkv, int dh, int *flags, hipStream_t st);

bool launch_attn_rows(const void *q, const void *k_cache, const void *v_cache, int dtype, float *o32,
                      const RowAct *ra, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh,
                      int *flags, hipStream_t st, AttnOpts opt)
{
    if ((int64_t)n_seq * T <= 0) return true;
    if (opt.page < 1 || opt.n_sink < 0 || opt.n_window < 0) return false;
    if (dtype == 0 && opt.plain() &&
        launch_attn_f32((const float *)q, (const float *)k_cache, (const float *)v_cache, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, dh, flags, st))
        return true;
    const int vec = dtype == 0 ? 4 : 8;
    if (dh % vec) return false;
    const int lpk = dh / vec;
    if (lpk > 64 || (lpk & (lpk - 1))) return false;
    const int g = Hq / Hkv;
    const int lpad = (L_max + 63) & ~63;
    // long caches (decode) get 1024-thread workgroups: more loads in flight per CU
    const int block = (L_max >= 2048) ? 1024 : 256;
    const size_t budget = 150 * 1024;
    const int ppad = opt.page > 1 ? (L_max + opt.page - 1) / opt.page : 0;
    int hpb = 4;
    while (hpb > 1 && (g % hpb != 0 ||
                       (size_t)hpb * (lpad + ppad) * 4 + (size_t)(block / 64) * hpb * dh * 4 > budget)) hpb >>= 1;
    const size_t lds = (size_t)hpb * (lpad + ppad) * 4 + (size_t)(block / 64) * hpb * dh * 4;
    if (lds > budget) return false;
#define SOL_ATTN_CASE(TT, H, B)                                                                                     \
    return launch_attn_rows_t<TT, H, B>(q, k_cache, v_cache, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, dh, lpad, lds, \
                                        flags, opt, ppad, st)
    if (dtype == 0) {
        if (block == 256) { if (hpb == 4) SOL_ATTN_CASE(float, 4, 256); if (hpb == 2) SOL_ATTN_CASE(float, 2, 256); SOL_ATTN_CASE(float, 1, 256); }
        else { if (hpb == 4) SOL_ATTN_CASE(float, 4, 1024); if (hpb == 2) SOL_ATTN_CASE(float, 2, 1024); SOL_ATTN_CASE(float, 1, 1024); }
    } else {
        if (block == 256) { if (hpb == 4) SOL_ATTN_CASE(bf16_t, 4, 256); if (hpb == 2) SOL_ATTN_CASE(bf16_t, 2, 256); SOL_ATTN_CASE(bf16_t, 1, 256); }
        else { if (hpb == 4) SOL_ATTN_CASE(bf16_t, 4, 1024); if (hpb == 2) SOL_ATTN_CASE(bf16_t, 2, 1024); SOL_ATTN_CASE(bf16_t, 1, 1024); }
    }
#undef SOL_ATTN_CASE
    return false;
}


typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_a;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_a;
typedef uint32_t u32x4_a __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_a __attribute__((ext_vector_type(2)));
typedef float f32x4_a __attribute__((ext_vector_type(4)));

// =================================================================================================
// Batched bf16 attention in two kernels.
//
//   k_attn_select   per (sequence, query head, 16 or 32 query rows): all causal scores of the rows by MFMA
//                   through LDS into registers as fp32, then per row the row maximum and -- when the budget is
//                   below the row length -- the exact threshold of the b largest scores (two or four rows per wave).
//                   Output per (row, head): { thr, max, jstar }: a key is kept iff
//                   s > thr  or  (s == thr and key index <= jstar).
//   k_attn_pv       per (sequence, KV head, 16 or 32 query rows), one wave per query head of the group: streams
//                   K and V^T chunks through LDS once for all heads of the group, recomputes the scores
//                   with the same MFMA sequence (bit-identical to the first kernel's), applies the
//                   threshold, and accumulates softmax numerators times V flash-style with scores and
//                   probabilities never leaving registers (the row maximum is already known, so there
//                   is no running rescale).
// Both compute a score tile as S^T = K Q^T, so a lane owns one query and four keys per tile; in
// k_attn_pv the keys of a 32-key chunk are assigned to MFMA rows such that each lane group ends up
// with 8 consecutive keys, which is exactly the A operand of the P V product.
// =================================================================================================
struct __align__(16) SelRow { float thr, mx; int jstar; int pad; };
__host__ __device__ __forceinline__ int attn_lpad64(int L_max) { return (L_max + 63) & ~63; }

// column (256*j + 4*lane + e order) of the quota-th key equal to thr; quota >= 1 and at most the
// number of such keys
template <int SLOTS>
__device__ __forceinline__ int wave_tie_last(const float (&key)[SLOTS], int n, float thr, int quota, int lane)
{
    int result = 0x7FFFFFFF;
    bool found = false;
#pragma unroll
    for (int j = 0; j < SLOTS / 4; ++j) {
        if (256 * j < n && !found) {
            int below = 0, here = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned long long bal = __ballot(key[4 * j + e] == thr);
                below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, below));
                here += __popcll(bal);
            }
            if (quota <= here) {                         // the quota-th tie sits in this group of 256 columns
                int mine = 0, col = -1;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool tie = key[4 * j + e] == thr;
                    if (tie && below + mine == quota - 1) col = 256 * j + 4 * lane + e;
                    mine += tie;
                }
                const unsigned long long who = __ballot(col >= 0);          // exactly one lane
                result = __builtin_amdgcn_readlane(col, (int)__builtin_ctzll(who));
                found = true;
            } else {
                quota -= here;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    return result;
}

// ---- R rows of one wave searched together ----------------------------------------------------------------------------
// The row a lane group (64 / R lanes) keeps the search state of: lanes [r * 64 / R, (r + 1) * 64 / R) hold row r's, so the
// interpolation and the bracket updates, ~35 vector instructions per step, are done once for all R rows; only the counts
// (two vector instructions per 64 scores) are per row. A pivot goes to its row's compares through a scalar register
// (readlane); the lanes' counts of all rows are summed by one exchange that leaves each row's in its group.
template <class T> __device__ __forceinline__ void swap_lanes32(T &a, T &b)     // upper half of a <-> lower half of b
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]), b = __builtin_bit_cast(T, (uint32_t)r[1]);
}
template <class T> __device__ __forceinline__ void swap_lanes16(T &a, T &b)     // odd rows of 16 lanes of a <-> even rows of b
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]), b = __builtin_bit_cast(T, (uint32_t)r[1]);
}
struct OpMaxF { __device__ __forceinline__ float operator()(float a, float b) const { return __builtin_fmaxf(a, b); } };
struct OpMinF { __device__ __forceinline__ float operator()(float a, float b) const { return __builtin_fminf(a, b); } };
struct OpAddI { __device__ __forceinline__ int operator()(int a, int b) const { return a + b; } };
// every lane of a row of 16 has a source under these controls: bound_ctrl lets the compiler fold the move into the operation
template <int CTRL, class T> __device__ __forceinline__ T dpp_of(T v)
{
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// x[r]: the lanes' parts of row r; result: in the lanes of group r the whole of row r
template <int R, class T, class Op> __device__ __forceinline__ T group_reduce(const T (&x)[R], Op op)
{
    static_assert(R == 2 || R == 4, "two or four rows per wave");
    T v, a = x[0], b = x[R / 2];
    swap_lanes32(a, b);
    v = op(a, b);
    if constexpr (R == 4) {
        T c = x[1], d = x[3];
        swap_lanes32(c, d);
        T e = op(c, d);
        swap_lanes16(v, e);
        v = op(v, e);
    }
    v = op(v, dpp_of<0xB1>(v));                          // quad_perm [1,0,3,2]
    v = op(v, dpp_of<0x4E>(v));                          // quad_perm [2,3,0,1]
    v = op(v, dpp_of<0x141>(v));                         // row_half_mirror
    v = op(v, dpp_of<0x140>(v));                         // row_mirror
    if constexpr (R == 2) {
        T w = v;
        swap_lanes16(v, w);
        v = op(v, w);
    }
    return v;
}

// What a wave gathers from its rows' scores while they come in: extremes over all of them, sum and sum of squares over
// the first two of every four columns (they only place the first pivot)
template <int R> struct RowStats {
    float mx[R], mn[R], s1[R], s2[R];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int r = 0; r < R; ++r) mx[r] = -__builtin_inff(), mn[r] = __builtin_inff(), s1[r] = 0.f, s2[r] = 0.f;
    }
};
// columns col0 + 4 * lane + e (e < 4) of row r (n valid columns) into four registers; -inf past the row's end
template <int R>
__device__ __forceinline__ void row_take4(RowStats<R> &st, int r, f32x4_a v, int col0, int n, int lane, float &k0, float &k1,
                                          float &k2, float &k3)
{
    if (col0 + 256 <= n) {
        k0 = v[0], k1 = v[1], k2 = v[2], k3 = v[3];
        st.mx[r] = __builtin_fmaxf(__builtin_fmaxf(st.mx[r], v[0]), v[1]);
        st.mx[r] = __builtin_fmaxf(__builtin_fmaxf(st.mx[r], v[2]), v[3]);
        st.mn[r] = __builtin_fminf(__builtin_fminf(st.mn[r], v[0]), v[1]);
        st.mn[r] = __builtin_fminf(__builtin_fminf(st.mn[r], v[2]), v[3]);
        st.s1[r] += v[0];
        st.s1[r] += v[1];
        st.s2[r] = __builtin_fmaf(v[0], v[0], st.s2[r]);
        st.s2[r] = __builtin_fmaf(v[1], v[1], st.s2[r]);
    } else {
        float k[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool valid = col0 + 4 * lane + e < n;
            k[e] = valid ? v[e] : -__builtin_inff();
            st.mx[r] = __builtin_fmaxf(st.mx[r], k[e]);
            st.mn[r] = valid ? __builtin_fminf(st.mn[r], v[e]) : st.mn[r];
            if (e < 2) {
                const float x = valid ? v[e] : 0.f;
                st.s1[r] += x;
                st.s2[r] = __builtin_fmaf(x, x, st.s2[r]);
            }
        }
        k0 = k[0], k1 = k[1], k2 = k[2], k3 = k[3];
    }
}

// number of this lane's scores >= pivot (uniform) in the first ng groups of 256 columns: a compare and an add with carry
// per 64 scores. One dispatch, then straight-line code. Rows shorter than the variant's class (the first rows of a wave at
// the class's edge) count every group of the class.
template <int SLOTS, int NG> __device__ __forceinline__ int wave_count_ge_n(const float (&key)[SLOTS], float pivot)
{
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < 4 * NG; ++j) cnt += key[j] >= pivot ? 1 : 0;
    return cnt;
}
template <int SLOTS>
__device__ __forceinline__ int wave_count_ge_s(const float (&key)[SLOTS], int ng, float pivot)
{
    if constexpr (SLOTS == 4) {
        return wave_count_ge_n<SLOTS, 1>(key, pivot);
    } else if constexpr (SLOTS == 16) {
        if (ng <= 2) return ng == 1 ? wave_count_ge_n<SLOTS, 1>(key, pivot) : wave_count_ge_n<SLOTS, 2>(key, pivot);
        return ng == 3 ? wave_count_ge_n<SLOTS, 3>(key, pivot) : wave_count_ge_n<SLOTS, 4>(key, pivot);
    } else if constexpr (SLOTS == 20) {
        return wave_count_ge_n<SLOTS, 5>(key, pivot);
    } else if constexpr (SLOTS == 32) {
        if (ng <= 6) return ng <= 5 ? wave_count_ge_n<SLOTS, 5>(key, pivot) : wave_count_ge_n<SLOTS, 6>(key, pivot);
        return ng == 7 ? wave_count_ge_n<SLOTS, 7>(key, pivot) : wave_count_ge_n<SLOTS, 8>(key, pivot);
    } else {
        static_assert(SLOTS == 64, "variants of the threshold kernel");
        if (ng <= 12) {
            if (ng <= 10) return ng <= 9 ? wave_count_ge_n<SLOTS, 9>(key, pivot) : wave_count_ge_n<SLOTS, 10>(key, pivot);
            return ng == 11 ? wave_count_ge_n<SLOTS, 11>(key, pivot) : wave_count_ge_n<SLOTS, 12>(key, pivot);
        }
        if (ng <= 14) return ng == 13 ? wave_count_ge_n<SLOTS, 13>(key, pivot) : wave_count_ge_n<SLOTS, 14>(key, pivot);
        return ng == 15 ? wave_count_ge_n<SLOTS, 15>(key, pivot) : wave_count_ge_n<SLOTS, 16>(key, pivot);
    }
}

// The search itself. In lane group r: n and b of row r (open: b < n, the row is there), fmx / fmn its extremes, s1 / s2 the
// sums of RowStats. Returns row r's threshold in its group's first lane (-inf where not open) and the index of the last kept key
// among those equal to it (INT_MAX when all of them are kept).
// The threshold is a pivot with exactly b scores at or above it, or the b-th largest score itself where ties leave no such
// pivot. The first pivot is the quantile of a normal distribution with the row's mean and variance (Abramowitz & Stegun
// 26.2.23), the second a Newton step with that distribution's density; then regula falsi between the ends of the bracket,
// whose weights are the counts' log-odds, log2((c + 1/2) / (n - c + 1/2)) (close to linear in the score for bell-shaped
// rows), with the Illinois correction (an end that stays put is scaled by a half), and from the 13th step on the middle
// of the bracket in key space, which bounds the worst case. Every pivot is clamped into the open bracket, so every step
// shrinks it. In a simulation 4.5 steps on normal rows of 512 .. 3072 scores, 6 on heavy-tailed ones, where regula falsi
// from the row's extremes takes 6.4 and 7.5. The attention stage on other rows, against that on normal ones (4 x 4096 tokens,
// head size 64, 1802 us): a common shift 1.01, keys that grow with the position 1.07, four keys 20 times the others 1.09, a
// third of them shifted along the query 1.08, norms spread by e 1.17, 16 clusters 1.44, 64 distinct keys (all ties) 2.37; with regula
// falsi from the extremes 1.01, 1.08, 1.13, 1.00, 1.16, 1.38, 2.23 (of 2719 us).
template <int R, int SLOTS>
__device__ __forceinline__ float wave_search_rows(const float (&key)[R][SLOTS], int ng, int n, int b, bool open, float fmx,
                                                  float fmn, float s1, float s2, int lane, int &jstar)
{
    constexpr int W = 64 / R;
    ng = __builtin_amdgcn_readfirstlane(ng);
    unsigned long long first = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) first |= 1ull << (r * W);
    auto to_key = [](float v) {
        const uint32_t u = __float_as_uint(v);
        return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    };
    uint32_t lo = to_key(fmn + 0.0f), hi = to_key(fmx + 0.0f);       // -0 + 0 = +0
    hi = open ? hi : lo;
    const float nf = (float)n, bf = (float)b, nh = nf + 0.5f;
    const float t_b = __builtin_amdgcn_logf(bf * __builtin_amdgcn_rcpf((nf - bf) + 1.0f));
    float flo = fmn, fhi = fmx;
    const float t_n = __builtin_amdgcn_logf(nh * 2.0f);
    float glo = t_n - t_b, ghi = -t_n - t_b;
    float w_up = 1.0f, w_dn = 1.0f;
    float fp, slope;
    {
        const float inv = __builtin_amdgcn_rcpf((float)((n >> 2) * 2 + ((n & 3) < 2 ? (n & 3) : 2)));
        const float mean = s1 * inv;
        const float sd = __builtin_amdgcn_sqrtf(__builtin_fmaxf(__builtin_fmaf(s2, inv, -mean * mean), 0.f));
        const float p = (bf - 0.5f) * __builtin_amdgcn_rcpf(nf);     // upper tail at the threshold
        const float t = __builtin_amdgcn_sqrtf(-1.3862943611f * __builtin_amdgcn_logf(__builtin_fminf(p, 1.0f - p)));
        const float num = __builtin_fmaf(__builtin_fmaf(0.010328f, t, 0.802853f), t, 2.515517f);
        const float den = __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(0.001308f, t, 0.189269f), t, 1.432788f), t, 1.0f);
        const float z = t - num * __builtin_amdgcn_rcpf(den);
        fp = __builtin_fmaf(sd, p < 0.5f ? z : -z, mean);
        // one count more or less moves the pivot by sd / (n * density)
        slope = sd * 2.5066283f * __builtin_amdgcn_exp2f(0.72134752f * z * z) * __builtin_amdgcn_rcpf(nf);
    }
    unsigned long long exact = 0;
    for (int it = 0;; ++it) {
        asm volatile("" : "+s"(it));                     // no peeled copies of the loop: the counts are most of the code
        const bool act = lo < hi;
        const unsigned long long todo = __ballot(act) & first;
        if (todo == 0) break;
        uint32_t mid = to_key(fp);
        mid = __builtin_elementwise_max(mid, lo + 1u);
        mid = __builtin_elementwise_min(mid, hi);
        if (it >= 12) mid = lo + ((hi - lo + 1u) >> 1);
        int32_t sgn = (int32_t)mid >> 31;
        asm("" : "+v"(sgn));                             // or the compiler makes a compare and a select of it
        const float fmid = __uint_as_float(mid ^ (~(uint32_t)sgn | 0x80000000u));
        int part[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            part[r] = 0;
            if (todo & (1ull << (r * W)))
                part[r] = wave_count_ge_s<SLOTS>(key[r], ng, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fmid), r * W)));
        }
        const int cnt = group_reduce<R>(part, OpAddI());
        const float cf = (float)cnt;
        const float g = __builtin_amdgcn_logf((cf + 0.5f) * __builtin_amdgcn_rcpf(nh - cf)) - t_b;
        const bool eq = act && cnt == b, up = act && cnt > b, dn = act && cnt < b;
        exact |= __ballot(eq);
        lo = eq || up ? mid : lo;
        hi = eq ? mid : (dn ? mid - 1u : hi);
        flo = up ? fmid : flo;
        fhi = up ? fhi : fmid;
        const float glo_w = glo * w_dn, ghi_w = ghi * w_up;
        glo = up ? g : glo_w;
        ghi = up ? ghi_w : g;
        w_up = up ? 0.5f : 1.0f;
        w_dn = up ? 1.0f : 0.5f;
        if (it == 0) fp = __builtin_fmaf(cf - bf, slope, fmid);
        else fp = __builtin_fmaf(fhi - flo, glo * __builtin_amdgcn_rcpf(glo - ghi), flo);
    }
    jstar = 0x7FFFFFFF;
    const float thr = score_unkey(lo);
    const unsigned long long closed = __ballot(open) & first & ~exact;      // the bracket closed on a score
    if (closed) {
        const float next = score_unkey(lo + 1u);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (closed & (1ull << (r * W))) {
                const float ft = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr), r * W));
                const float fn = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(next), r * W));
                const int nr = __builtin_amdgcn_readlane(n, r * W), br = __builtin_amdgcn_readlane(b, r * W);
                const float n_ge = wave_sum_dpp((float)wave_count_ge_s<SLOTS>(key[r], ng, ft));
                if (n_ge > (float)br) {                  // more scores equal to the threshold than the budget takes
                    const int n_gt = (int)wave_sum_dpp((float)wave_count_ge_s<SLOTS>(key[r], ng, fn));
                    const int js = wave_tie_last<SLOTS>(key[r], nr, ft, br - n_gt, lane);
                    jstar = lane == r * W ? js : jstar;
                }
            }
    }
    return open ? thr : -__builtin_inff();
}

// Thresholds: one workgroup of 8 waves takes blocks of 8 * R query rows of one (sequence, head). The scores of a block are
// made in parts of SC keys: the waves stream the part's key tiles (two register sets in flight where they fit) and multiply
// them into the LDS, and after a barrier every wave takes its R rows' piece of the part into registers, so that the LDS
// holds a part of a row instead of the whole and does not bound the rows per block. When the last part is in, a wave
// searches its R rows together (wave_search_rows) and goes straight on to the first part of the next block, whose first
// tiles were requested ahead of the search: waves whose search is short stream keys while the others still search.
// Blocks of 16 rows fill the 16 query columns of the MFMA, and all causal K passes through the CU's L1 once per block: with
// whole rows in the LDS only 8 rows of 4096 keys fit, half the columns were multiplied for nothing and the K stream was twice
// as long. Two rows per wave share the search's bookkeeping (see wave_search_rows). Measured per launch, before and after:
// rows of 2049 .. 4096 keys at head size 128 (8 x 4096 tokens) 3.88 -> 2.24 ms, of 1025 .. 2048 keys 0.75 -> 0.51 ms there
// and 1.19 -> 0.79 ms at head size 64 (16 x 2048 tokens), up to 1024 keys 0.51 -> 0.38 ms.
// Bound (2049 .. 4096 keys, of 2.24 ms, by builds with pieces taken out): K stream 0.75 (at the 57 bytes per clock that an L2
// feeds a CU), products and LDS writes 0.3, taking the rows out of the LDS 0.45, search 0.75; a second buffer, so that half
// of the waves do their scores while the others take rows or search, was slower (2.43: smaller parts, more barriers), and so
// were parts of 256 keys behind a barrier each (2.49).
// PRE: keys [0, pv.P) of sequence s are read from the prefix cache of input s / pv.K (shared by the pv.K schedules
// of that input), keys from pv.P on from the sequence's own cache kc, which holds positions pv.P.. only
// ([n_seq][Hkv][crows][DH]); pv.P is a multiple of 64 and the two caches lie less than 2^31 elements apart.
// KF: kc (with PRE: pv.kf, for the prefix keys) is the copy of the K cache in MFMA operand order written by k_frag_k,
// in which the 16 bytes a lane feeds to one MFMA are contiguous over the lanes: a fragment load reads 1 KB in a row
// (8 full cache lines) where the same load from the cache itself picks 64-byte pieces out of 16 rows. The values in
// the registers are the same either way. With PRE the sequence's own keys (positions pv.P..) still come from its cache.
// Blocks are dealt to the nb workgroups of a (sequence, head) in zigzag order (k-th visit: block nb*k + bi for even k,
// nb*k + nb-1-bi for odd k), which gives every workgroup the same number of causal keys.
template <int SLOTS, int DH, int R, int U, int NS, int SC> struct SelShape {
    static constexpr int NW = 8, BQ = NW * R, RT = (BQ + 15) / 16, KK = DH / 32, PARTS = (SLOTS * 64 + SC - 1) / SC;
    static constexpr int GT = NW * U;                      // key tiles of a group: U per wave
    static constexpr int LS = SC + 4;                      // row stride = 4 mod 64 floats: the 16 query rows of a 128-bit
                                                           // store hit 16 different bank groups
    static constexpr int LDS = BQ * LS * 4;
    static_assert(SC % 256 == 0 && SC % (GT * NS * 16) == 0 && BQ % 16 == 0, "parts of whole 256-column groups and whole rounds of the register sets");
};
template <int SLOTS, int DH, int R, int U, int NS, int SC, bool PRE, bool KF>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(SLOTS <= 32 ? 4 : 2, 8)))
k_attn_select(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, SelRow *__restrict__ sel,
                   const RowAct *__restrict__ ra, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hq, int Hkv,
                   float scale, int nb, PrefixView pv, int n_lo, int n_hi)
{
    using Sh = SelShape<SLOTS, DH, R, U, NS, SC>;
    constexpr int NW = Sh::NW, BQ = Sh::BQ, RT = Sh::RT, KK = Sh::KK, GT = Sh::GT, LS = Sh::LS, W = 64 / R;
    extern __shared__ __align__(16) float sc[];            // [BQ][LS]

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bi = blockIdx.x, h = blockIdx.y, s = blockIdx.z, kvh = h / (Hq / Hkv);
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) return;                 // flagged by the projection kernel; sequence skipped
    // this launch takes the rows whose key count n = p0 + row + 1 lies in (n_lo, n_hi]: rows [q_lo, q_hi) of the sequence
    // (long sequences are split by row length over the kernel's variants; the blocks of BQ rows count from q_lo)
    const int q_lo = n_lo - p0 < 0 ? 0 : (n_lo - p0 > Tn ? Tn : n_lo - p0);
    const int q_hi = n_hi - p0 < 0 ? 0 : (n_hi - p0 > Tn ? Tn : n_hi - p0);
    if (q_hi <= q_lo) return;                              // whole workgroup, before any barrier
    const int n_qb = (q_hi - q_lo + BQ - 1) / BQ;
    // wave-uniform bases + 32-bit per-lane offsets: one address register per load instead of two
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)(KF ? attn_lpad64(L_max) : L_max) * DH;
    uint32_t kdelta = 0u;                                  // PRE: offset of the own cache (minus P rows) from the prefix cache
    if constexpr (PRE) {
        const bf16_t *own = kc + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * DH - (int64_t)pv.P * DH;
        kbase = (KF ? pv.kf : pv.k) + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * DH;
        kdelta = (uint32_t)__builtin_amdgcn_readfirstlane((int)(own - kbase));
    }
    const char *const kb = reinterpret_cast<const char *>(kbase);
    const char *const qb0 = reinterpret_cast<const char *>(q + (int64_t)s * Tn * (int64_t)(Hq * DH) + (int64_t)h * DH);
    const int l16 = lane & 15, lg = lane >> 4;

    // q fragments ahead of the search too, where the registers leave room
    constexpr bool Q_AHEAD = SLOTS > 32 || R * SLOTS + (RT + NS * U) * KK * 4 <= 88;
    // of the next block's first group, the tiles that are requested ahead of the search (the others behind it)
    constexpr int U_AHEAD = (NS == 1 && SLOTS <= 32 && R * SLOTS + U * KK * 4 > 88) ? U / 2 : U;
    bf16x8_a qf[RT][KK], kf[NS][U][KK];                    // group g's key tiles in set g % NS

    auto load_q = [&](int q0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            int qr = q0 + rt * 16 + l16;
            if (qr >= Tn) qr = Tn - 1;
            const uint32_t qo = ((uint32_t)qr * (uint32_t)(Hq * DH) + (uint32_t)(lg * 8)) * 2u;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) qf[rt][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(qb0 + qo + kk * 64));
        }
    };
    // this wave's key tiles t0 + w, t0 + NW + w, .. into a set (none from the block's n_keys-th key on): lane (l16, lg) gets
    // 8 channels at 8 * lg of key 16 * tile + l16 for every 32-channel piece
    auto load_k = [&](bf16x8_a (&set)[U][KK], int t0, int n_keys, int u0, int u1) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kt = t0 + u * NW + w;
            if (u < u0 || u >= u1 || kt * 16 >= n_keys) continue;
            const char *base;                              // uniform: the lanes' own part is one 32-bit offset
            uint32_t off;
            int step;
            if constexpr (KF) {
                base = kb + (uint32_t)kt * (uint32_t)(KK * 1024), off = (uint32_t)lane * 16u, step = 1024;
            }
            if (!KF || (PRE && kt * 16 >= pv.P)) {         // from the cache itself (with KF: the sequence's own keys)
                int key_i = kt * 16 + l16;
                if (key_i >= n_keys) key_i = n_keys - 1;
                base = kb + ((PRE && kt * 16 >= pv.P) ? (uint64_t)kdelta * 2u : 0u);
                off = ((uint32_t)key_i * (uint32_t)DH + (uint32_t)(lg * 8)) * 2u, step = 64;
            }
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) set[u][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(base + off + kk * step));
        }
    };

    // S^T tile = K tile (rows) x Q^T (columns): lane (l16, lg) gets keys 4 * lg .. 4 * lg + 3 of query l16. The group's
    // tiles t0 + w .. of a block of n_kt tiles into the LDS; t_part: the part's first tile
    auto score_group = [&](const bf16x8_a (&set)[U][KK], int t0, int t_part, int n_kt) {
        float *const dst = sc + l16 * LS + (t0 - t_part + w) * 16 + 4 * lg;
        floatx4_a acc[U][RT];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[u][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(set[u][kk], qf[rt][kk], kk ? acc[u][rt] : floatx4_a{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)                // a tile past the last one: the set's old values, in columns that nobody reads
                *reinterpret_cast<f32x4_a *>(dst + rt * 16 * LS + u * NW * 16) =
                    f32x4_a{acc[u][rt][0] * scale, acc[u][rt][1] * scale, acc[u][rt][2] * scale, acc[u][rt][3] * scale};
    };

    int visit = 0, qb = bi;
    if (qb >= n_qb) return;
#pragma unroll
    for (int i = 0; i < NS; ++i)                           // a set may be multiplied before it was ever loaded (see score_group)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kf[i][u][kk] = __builtin_bit_cast(bf16x8_a, u32x4_a{0u, 0u, 0u, 0u});
    {
        const int q0 = q_lo + qb * BQ, n_max = p0 + (q_hi < q0 + BQ ? q_hi : q0 + BQ);
        if (Q_AHEAD) load_q(q0);
#pragma unroll
        for (int i = 0; i < NS; ++i) load_k(kf[i], i * GT, n_max, 0, U_AHEAD);
    }
    // the barriers wait for LDS only: global loads and the result's store stay in flight
#define SOL_SEL_BARRIER asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")
    while (true) {
        const int q0 = q_lo + qb * BQ;
        const int rows = (q_hi - q0 < BQ) ? (q_hi - q0) : BQ;
        const int n_max = p0 + q0 + rows, n_kt = (n_max + 15) >> 4;
        const int n_first = p0 + q0 + w * R + 1;           // keys of the wave's first row
        if (!Q_AHEAD) load_q(q0);
        if (U_AHEAD < U) load_k(kf[0], 0, n_max, U_AHEAD, U);
        float key[R][SLOTS];
        RowStats<R> st;
        st.clear();
        // rows' actions: lane group r takes row r's
        const int my_row = w * R + lane / W;
        RowAct act = RowAct();
        if (my_row < rows) act = ra[(int64_t)s * Tn + q0 + my_row];
        const int n = p0 + q0 + my_row + 1;
        const int b = my_row < rows ? budget_ceil(act.keep_num, act.keep_den, n) : n;
#pragma unroll
        for (int part = 0; part < Sh::PARTS; ++part) {
            constexpr int PT = SC / 16;                    // tiles of a part
            if (part * SC < n_max) {
                const int t_end = n_kt < (part + 1) * PT ? n_kt : (part + 1) * PT;
                for (int t0 = part * PT; t0 < t_end; t0 += NS * GT) {
#pragma unroll
                    for (int i = 0; i < NS; ++i)
                        if (t0 + i * GT < t_end) {
                            score_group(kf[i], t0 + i * GT, part * PT, n_kt);
                            if (t0 + (i + NS) * GT < n_kt) load_k(kf[i], t0 + (i + NS) * GT, n_max, 0, U);
                        }
                }
                SOL_SEL_BARRIER;                           // the part is complete
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int g = 0; g < SC / 256; ++g) {
                        const int j = part * (SC / 256) + g;
                        if (4 * j >= SLOTS) continue;
                        if (256 * j < n_max)
                            row_take4<R>(st, r, *reinterpret_cast<const f32x4_a *>(sc + (w * R + r) * LS + 256 * g + 4 * lane), 256 * j,
                                         n_first + r, lane, key[r][4 * j], key[r][4 * j + 1], key[r][4 * j + 2], key[r][4 * j + 3]);
                        else key[r][4 * j] = key[r][4 * j + 1] = key[r][4 * j + 2] = key[r][4 * j + 3] = -__builtin_inff();
                    }
                SOL_SEL_BARRIER;                           // every wave has its rows' pieces: the next part may be written
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int j = part * (SC / 64); j < (part + 1) * (SC / 64) && j < SLOTS; ++j) key[r][j] = -__builtin_inff();
            }
        }
        ++visit;
        const int qb_next = nb * visit + ((visit & 1) ? nb - 1 - bi : bi);
        const bool more = qb_next < n_qb;
        if (more) {
            const int q0n = q_lo + qb_next * BQ;
            if (Q_AHEAD) load_q(q0n);
#pragma unroll
            for (int i = 0; i < NS; ++i) load_k(kf[i], i * GT, p0 + (q_hi < q0n + BQ ? q_hi : q0n + BQ), 0, U_AHEAD);
        }
        const float fmx = group_reduce<R>(st.mx, OpMaxF()), fmn = group_reduce<R>(st.mn, OpMinF());
        const float s1 = group_reduce<R>(st.s1, OpAddF()), s2 = group_reduce<R>(st.s2, OpAddF());
        int js;
        const float thr = wave_search_rows<R, SLOTS>(key, (n_first + R - 1 + 255) >> 8, n, b, b < n, fmx, fmn, s1, s2, lane, js);
        if (lane % W == 0 && my_row < rows) sel[((int64_t)s * Tn + q0 + my_row) * Hq + h] = SelRow{thr, fmx + 0.0f, js, 0};
        if (!more) break;
        qb = qb_next;
    }
#undef SOL_SEL_BARRIER
}

// Unit hook: the row stage of k_attn_select (scores of R rows into registers, threshold search, tie index) on caller
// rows, R per wave; keep[r][j] = 1 for the kept columns, by the same rule k_attn_pv applies to {thr, jstar}.
template <int SLOTS, int R>
__global__ void __launch_bounds__(64) k_test_select_rows(const float *__restrict__ scores, int rows, int n_cols,
                                                         const int32_t *__restrict__ n_valid, const int32_t *__restrict__ kk,
                                                         uint8_t *__restrict__ keep)
{
    extern __shared__ __align__(16) float sc[];              // [R][SLOTS * 64]
    constexpr int W = 64 / R, LP = SLOTS * 64;
    const int lane = threadIdx.x, r0 = blockIdx.x * R;
    float key[R][SLOTS];
    RowStats<R> st;
    st.clear();
    int n_top = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool there = r0 + r < rows;
        const int n = there ? n_valid[r0 + r] : 1;
        n_top = n > n_top ? n : n_top;
        for (int j = lane; j < LP; j += 64) sc[r * LP + j] = (there && j < n) ? scores[(int64_t)(r0 + r) * n_cols + j] : 0.f;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SLOTS / 4; ++j)
            row_take4<R>(st, r, *reinterpret_cast<const f32x4_a *>(sc + r * LP + 256 * j + 4 * lane), 256 * j, n, lane,
                         key[r][4 * j], key[r][4 * j + 1], key[r][4 * j + 2], key[r][4 * j + 3]);
    }
    const float fmx = group_reduce<R>(st.mx, OpMaxF()), fmn = group_reduce<R>(st.mn, OpMinF());
    const float s1 = group_reduce<R>(st.s1, OpAddF()), s2 = group_reduce<R>(st.s2, OpAddF());
    const int mine = r0 + lane / W;
    const int n = mine < rows ? n_valid[mine] : 1, b = mine < rows ? kk[mine] : 1;
    int js;
    const float thr = wave_search_rows<R, SLOTS>(key, (n_top + 255) >> 8, n, b, b < n, fmx, fmn, s1, s2, lane, js);
    for (int r = 0; r < R && r0 + r < rows; ++r) {
        const float fthr = __shfl(thr, r * W, 64);
        const int jr = __shfl(js, r * W, 64), nr = n_valid[r0 + r];
        for (int j = lane; j < n_cols; j += 64) {
            const float sv = j < nr ? sc[r * LP + j] : 0.f;
            keep[(int64_t)(r0 + r) * n_cols + j] = (j < nr && (sv > fthr || (sv == fthr && j <= jr))) ? 1 : 0;
        }
    }
}

bool launch_test_attn_threshold(const float *scores, int rows, int n_cols, const int32_t *n_valid, const int32_t *k,
                                uint8_t *keep_out, hipStream_t st)
{
    if (n_cols > 4096) return false;
    // the variants of k_attn_select, by columns; up to 1024 both widths of a wave, four rows for the first half of the rows
    const int half = n_cols <= 1024 ? (rows + 1) / 2 : 0;
#define SOL_TSEL(SL, R_, R0, COUNT)                                                                                  \
    if ((COUNT) > 0)                                                                                                 \
        hipLaunchKernelGGL((k_test_select_rows<SL, R_>), dim3(((COUNT) + R_ - 1) / R_), dim3(64), (size_t)(R_) * (SL) * 64 * 4, st, \
                           scores + (int64_t)(R0) * n_cols, COUNT, n_cols, n_valid + (R0), k + (R0), keep_out + (int64_t)(R0) * n_cols)
    if (n_cols <= 256) { SOL_TSEL(4, 4, 0, half); SOL_TSEL(4, 2, half, rows - half); }
    else if (n_cols <= 1024) { SOL_TSEL(16, 4, 0, half); SOL_TSEL(16, 2, half, rows - half); }
    else if (n_cols <= 1280) { SOL_TSEL(20, 2, 0, rows); }
    else if (n_cols <= 2048) { SOL_TSEL(32, 2, 0, rows); }
    else { SOL_TSEL(64, 2, 0, rows); }
#undef SOL_TSEL
    return true;
}

// ---- fp32 attention of batched passes, plain top-k rule --------------------------------------------------------------
// One workgroup of four waves per (sequence, head, 16 query rows), rows of at most 1024 keys: scores by the fp32 matrix
// instruction into the LDS, four rows per wave searched as in k_attn_select, numerators back into the LDS, P V by the fp32
// matrix instruction. Every sum is made in the order of k_attn_rows with 256 threads, so that the results are its bits (a score
// that rounds otherwise swaps kept keys here and there):
//   - a score: groups of four channels, each one instruction from zero (k adds in order, as a chain of fma), then the tree
//     over the groups c, c ^ DH/8, .., c ^ 1 that its lanes' exchanges make. A lane loads 16 bytes, a group's four channels;
//     lane group lg wants channel lg of every group: a 4 x 4 transposition of registers and lane groups (transpose4).
//   - the denominator: chains over columns 256 apart, then lanes 32, 16, 8, 4, 2, 1 apart, then groups of 64 in order.
//   - an output: a chain over the keys KPI apart for every slot (key mod KPI), so that the k of an instruction is four
//     consecutive keys of a slot; slots of a wave as a tree, waves in order.
// A NaN or an infinity in a V row that a query does not keep would reach it through a product with 0: results that are not
// finite are made again over the kept keys alone.
// Bound: vector instructions (search, exponentials, the trees) and latency. k_attn_rows, a workgroup per row with a radix
// select in the LDS, took 250 us for 2 x 509 rows of 32 heads of 64, this 98; 19.0 us for 4 x 128 rows of 4 heads, this 16.5.
__device__ __forceinline__ void transpose4(f32x4_a &v)        // [element][lane group] -> [lane group][element]
{
    float a = v[0], b = v[1], c = v[2], d = v[3];
    swap_lanes32(a, c);
    swap_lanes32(b, d);
    swap_lanes16(a, b);
    swap_lanes16(c, d);
    v = f32x4_a{a, b, c, d};
}
template <int DH>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_attn_f32(const float *__restrict__ q, const float *__restrict__ kc, const float *__restrict__ vc, float *__restrict__ o32,
           const RowAct *__restrict__ ra, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hq, int Hkv, float scale,
           int LS, int *flags)
{
    constexpr int NW = 4, R = 4, SLOTS = 16, W = 16, NI = DH / 16, NC = DH / 64;
    constexpr int KPI = 1024 / DH, SPW = KPI / NW;         // key slots, and slots of a wave
    extern __shared__ __align__(16) float sc[];            // [16][LS] scores, then numerators; [NW][16][DH] the waves' outputs
    __shared__ float s_inv[16];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.y, s = blockIdx.z, kvh = h / (Hq / Hkv), q0 = blockIdx.x * 16;
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) {                       // the sequence does not fit its cache: skipped
        if (tid == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
        return;
    }
    const int rows = Tn - q0 < 16 ? Tn - q0 : 16;
    const int n_max = p0 + q0 + rows, n_kt = (n_max + 15) >> 4;
    const float *const kb = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const float *const vb = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const int64_t row0 = (int64_t)s * Tn + q0;

    // ---- scores: the waves take key tiles of 16 in turn -------------------------------------------
    f32x4_a qf[NI], kf[2][NI];                             // channels 16 i + 4 lg .. + 3; transposed: channel lg of groups 4 i .. 4 i + 3
    {
        const int qr = l16 < rows ? l16 : rows - 1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            qf[i] = *reinterpret_cast<const f32x4_a *>(q + (row0 + qr) * (int64_t)(Hq * DH) + (int64_t)h * DH + 16 * i + 4 * lg);
            transpose4(qf[i]);
        }
    }
    auto load_k = [&](int kt, f32x4_a (&k)[NI]) {
        int key = kt * 16 + l16;
        key = key < n_max ? key : n_max - 1;
#pragma unroll
        for (int i = 0; i < NI; ++i) k[i] = *reinterpret_cast<const f32x4_a *>(kb + (int64_t)key * DH + 16 * i + 4 * lg);
    };
    auto score = [&](int kt, f32x4_a (&k)[NI]) {           // lane (l16, lg): keys 4 lg .. 4 lg + 3 of query l16
#pragma unroll
        for (int i = 0; i < NI; ++i) transpose4(k[i]);
        const floatx4_a zero = {0.f, 0.f, 0.f, 0.f};
        floatx4_a t[2 * NI];
#pragma unroll
        for (int c = 0; c < 2 * NI; ++c) {                 // groups c and c + DH / 8
            const int d = c + 2 * NI;
            t[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c / 4][c % 4], qf[c / 4][c % 4], zero, 0, 0, 0) +
                   __builtin_amdgcn_mfma_f32_16x16x4f32(k[d / 4][d % 4], qf[d / 4][d % 4], zero, 0, 0, 0);
        }
#pragma unroll
        for (int o = NI; o > 0; o >>= 1)
#pragma unroll
            for (int c = 0; c < o; ++c) t[c] = t[c] + t[c + o];
        *reinterpret_cast<f32x4_a *>(sc + l16 * LS + kt * 16 + 4 * lg) =
            f32x4_a{t[0][0] * scale, t[0][1] * scale, t[0][2] * scale, t[0][3] * scale};
    };
    if (w < n_kt) load_k(w, kf[0]);
    for (int kt = w; kt < n_kt; kt += 2 * NW) {
        if (kt + NW < n_kt) load_k(kt + NW, kf[1]);
        score(kt, kf[0]);
        if (kt + 2 * NW < n_kt) load_k(kt + 2 * NW, kf[0]);
        if (kt + NW < n_kt) score(kt + NW, kf[1]);
    }
    const int my_row = w * R + lane / W;                   // lane group r: row w * R + r
    RowAct act = RowAct();
    if (my_row < rows) act = ra[row0 + my_row];
    const int n = p0 + q0 + my_row + 1;
    const int b = my_row < rows ? budget_ceil(act.keep_num, act.keep_den, n) : n;
    __syncthreads();

    // ---- thresholds, numerators -----------------------------------------------------------------
    {
        const int n_first = p0 + q0 + w * R + 1;
        float key[R][SLOTS];
        RowStats<R> st;
        st.clear();
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < SLOTS / 4; ++j) {
                if (256 * j < n_max)                       // LS covers whole groups of 256 columns
                    row_take4<R>(st, r, *reinterpret_cast<const f32x4_a *>(sc + (w * R + r) * LS + 256 * j + 4 * lane), 256 * j, n_first + r,
                                 lane, key[r][4 * j], key[r][4 * j + 1], key[r][4 * j + 2], key[r][4 * j + 3]);
                else key[r][4 * j] = key[r][4 * j + 1] = key[r][4 * j + 2] = key[r][4 * j + 3] = -__builtin_inff();
            }
        const float fmx = group_reduce<R>(st.mx, OpMaxF()), fmn = group_reduce<R>(st.mn, OpMinF());
        const float s1 = group_reduce<R>(st.s1, OpAddF()), s2 = group_reduce<R>(st.s2, OpAddF());
        int js;
        const float thr = wave_search_rows<R, SLOTS>(key, (n_first + R - 1 + 255) >> 8, n, b, b < n, fmx, fmn, s1, s2, lane, js);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float rt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr), r * W));
            const float rm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fmx), r * W));
            const int rj = __builtin_amdgcn_readlane(js, r * W);
            f32x4_a den = {0.f, 0.f, 0.f, 0.f};            // of columns 4 * lane + e, 256 + 4 * lane + e, ..
#pragma unroll
            for (int j = 0; j < SLOTS / 4; ++j)
                if (256 * j < n_max) {
                    f32x4_a pr;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float sv = key[r][4 * j + e];  // dropped: below the threshold, or a tie that loses (a NaN is kept)
                        const bool drop = sv < rt || (sv == rt && 256 * j + 4 * lane + e > rj);
                        pr[e] = drop ? 0.f : expf(sv - rm);
                        den[e] += pr[e];
                    }
                    *reinterpret_cast<f32x4_a *>(sc + (w * R + r) * LS + 256 * j + 4 * lane) = pr;
                }
            // columns 32, 16, 8, 4 apart: lanes 8, 4, 2, 1 apart in a row of 16 (rotations: what they meet has that period)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                den[e] += dpp_of<0x128>(den[e]);           // row_ror:8
                den[e] += dpp_of<0x124>(den[e]);           // row_ror:4
                den[e] += dpp_of<0x122>(den[e]);           // row_ror:2
                den[e] += dpp_of<0x121>(den[e]);           // row_ror:1
            }
            const float d64 = (den[0] + den[2]) + (den[1] + den[3]);
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) d += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d64), 16 * i));
            if (lane == 0) s_inv[w * R + r] = 1.0f / d;
        }
    }
    __syncthreads();

    // ---- P V: slots SPW * w .. of KPI, four keys of a slot per instruction -----------------------------
    constexpr int KCH = 4 * KPI;
    floatx4_a acc[SPW][NC][4];                             // [slot][64 channels][channel 4 l16 + e]
#pragma unroll
    for (int a = 0; a < SPW; ++a)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[a][c][e] = floatx4_a{0.f, 0.f, 0.f, 0.f};
    f32x4_a vf[2][SPW][NC];
    auto load_v = [&](int k0, f32x4_a (&v)[SPW][NC]) {
#pragma unroll
        for (int a = 0; a < SPW; ++a) {
            int k = k0 + KPI * lg + SPW * w + a;
            k = k < n_max ? k : n_max - 1;                 // its numerators are 0
#pragma unroll
            for (int c = 0; c < NC; ++c) v[a][c] = *reinterpret_cast<const f32x4_a *>(vb + (int64_t)k * DH + 64 * c + 4 * l16);
        }
    };
    auto product = [&](int k0, const f32x4_a (&v)[SPW][NC]) {
        const float *const pr = sc + l16 * LS + k0 + KPI * lg + SPW * w;
        float pa[SPW];
#pragma unroll
        for (int a = 0; a < SPW; ++a) pa[a] = pr[a];
#pragma unroll
        for (int a = 0; a < SPW; ++a)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[a][c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[a], v[a][c][e], acc[a][c][e], 0, 0, 0);
    };
    load_v(0, vf[0]);
    for (int k0 = 0; k0 < n_max; k0 += 2 * KCH) {
        if (k0 + KCH < n_max) load_v(k0 + KCH, vf[1]);
        product(k0, vf[0]);
        if (k0 + 2 * KCH < n_max) load_v(k0 + 2 * KCH, vf[0]);
        if (k0 + KCH < n_max) product(k0 + KCH, vf[1]);
    }
    // lane (l16, lg) register r is query 4 lg + r, channels 64 c + 4 l16 + e; the waves' parts meet in the LDS
    float *const red = sc + 16 * LS;                       // [NW][16][DH]
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4_a t;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t[e] = acc[0][c][e][r] + acc[1][c][e][r];
                if constexpr (SPW == 4) t[e] += acc[2][c][e][r] + acc[3][c][e][r];
            }
            *reinterpret_cast<f32x4_a *>(red + (w * 16 + 4 * lg + r) * DH + 64 * c + 4 * l16) = t;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int el = (i * 256 + tid) * 4, r = el / DH, ch = el - r * DH;
        if (r >= rows) continue;
        f32x4_a y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < NW; ++a) y += *reinterpret_cast<const f32x4_a *>(red + a * 16 * DH + el);
        y *= s_inv[r];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (!(__builtin_fabsf(y[e]) < __builtin_inff())) {
                float z = 0.f;
                for (int j = 0; j < p0 + q0 + r + 1; ++j) {
                    const float pj = sc[r * LS + j];
                    if (pj != 0.f) z = __builtin_fmaf(pj, vb[(int64_t)j * DH + ch + e], z);
                }
                y[e] = z * s_inv[r];
            }
        *reinterpret_cast<f32x4_a *>(o32 + (row0 + r) * (int64_t)(Hq * DH) + (int64_t)h * DH + ch) = y;
    }
}

// Passes of 16 rows per sequence or more on caches of at most 1024 positions: fewer rows leave most of a block's 16 columns
// empty, longer rows do not fit the search's registers (and what a row holds is not known here, only what its cache can hold);
// both stay with k_attn_rows. So do small passes of models with fewer than four heads per group, whose workgroups there have one or two
// short rows each and fit the chip together: a layer's call over one sequence of 4 heads of 64, us, k_attn_rows / here, 16 rows
// 57 / 62, 128 rows 64 / 68, 250 rows 73 / 72, 16 rows behind 368 keys 72 / 71; 4 x 128 rows 81 / 79; 32 x 16 rows 75 / 76, 128 x 16
// rows 137 / 122; 16 heads, 64 rows 69 / 73, 2 x 128 rows 93 / 85; 4 heads in 2 groups of 128, 16 rows 64 / 66, 128 rows 77 / 72. With
// four heads per group (32 heads of 64) 16 rows 86 / 82, 16 rows behind 900 keys 141 / 103.
static bool launch_attn_f32(const float *q, const float *kc, const float *vc, float *o32, const RowAct *ra, const int32_t *pos0,
                            int n_seq, int T, int L_max, int Hq, int Hkv, int dh, int *flags, hipStream_t st)
{
    if ((dh != 64 && dh != 128) || T < 16 || L_max > 1024 || Hkv <= 0 || Hq % Hkv || Hq > 65535 || n_seq > 65535) return false;
    const int heads = Hq / Hkv % 4 == 0 ? 4 : Hq / Hkv % 2 == 0 ? 2 : 1, keys = pos0 ? L_max : T;   // k_attn_rows: heads per workgroup
    const int64_t rows = (int64_t)n_seq * T * Hq;
    if (heads < 4 && keys * heads * dh <= 24576 && rows <= 2048 && rows * keys * heads <= 163840) return false;
    const int LS = (L_max + 255) / 256 * 256 + 4;          // row stride = 4 mod 64 floats
    const size_t lds = ((size_t)16 * LS + 4 * 16 * dh) * 4;
    auto kern = dh == 64 ? k_attn_f32<64> : k_attn_f32<128>;
    if (lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 104 * 1024) != hipSuccess)
        return false;
    hipLaunchKernelGGL(kern, dim3((T + 15) / 16, Hq, n_seq), dim3(256), lds, st, q, kc, vc, o32, ra, pos0, T, L_max, Hq, Hkv,
                       1.0f / sqrtf((float)dh), LS, flags);
    return true;
}

// ---- k_attn_pv -------------------------------------------------------------------------------------
// LDS chunk layouts (bf16, 16-byte pieces XOR-swizzled so that the 128-bit fragment reads of 16 lanes
// hit 16 different bank groups):
//   K chunk   [64 keys][DH]      piece' = piece ^ swzK(key row)
//   V^T chunk [DH][64 keys]      piece' = piece ^ ((d >> 1) & 7)
template <int DH> __device__ __forceinline__ int pv_swz_k(int row)
{
    if constexpr (DH == 64) return ((row >> 1) & 1) | (((row >> 3) & 3) << 1);   // rows {0-3, 8-11, 16-19, 24-27} (+4)
    else return (row & 3) | (((row >> 3) & 3) << 2);
}
// The transposing read takes, per group of 16 lanes, 4 keys (lanes 4 j .. 4 j + 3: key j) x 16 channels (4 per lane) and
// hands lane i the 4 keys of channel i. The 64 lanes of a read touch 32 bytes each of 16 rows: the 32-byte windows of a row
// are XOR-ed with row bits so that 8 of these rows fill the 64 banks (rows 4 apart, the second read, swizzle alike).
template <int DH> __device__ __forceinline__ int pv_swz_v(int row)
{
    return DH == 64 ? (row & 2) | ((row >> 1) & 4) : ((row & 3) << 1) | (row & 8);
}
typedef short s16x4_a __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_a lds_s16x4;
// keys key0 .. key0 + 7 (key0: this lane group's, a multiple of 8) of channel 16 * dt + l16
template <int DH> __device__ __forceinline__ bf16x8_a pv_read_v(const unsigned char *vb, int key0, int dt, int l16)
{
    const int row = key0 + (l16 >> 2);
    const unsigned char *p = vb + row * (DH * 2) + (((dt * 2) ^ pv_swz_v<DH>(row)) << 4) + (l16 & 3) * 8;
    const s16x4_a a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4_a b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * DH * 2));
    return __builtin_bit_cast(bf16x8_a, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// softmax numerators of one 32-key sub-chunk for one query tile, as the A operand (hi and lo bf16
// halves) of the P V product. st[kt][r] is the score of key  kbase + 8*lg + 4*kt + r.
template <bool MASK, bool TIES>
__device__ __forceinline__ void pv_probs(const floatx4_a (&st)[2], float scale, float thr, float mxl, int jstar, int pos,
                                         int kfirst, float &den, bf16x8_a &phi, bf16x8_a &plo)
{
    float p[8];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float sv = st[kt][r] * scale;
            const int j = kfirst + 4 * kt + r;
            bool keep = sv >= thr;
            if (TIES) keep = sv > thr || (sv == thr && j <= jstar);
            if (MASK) keep = keep && j <= pos;
            const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(sv, 1.44269504088896341f, -mxl));
            p[4 * kt + r] = keep ? e : 0.f;
            den += p[4 * kt + r];
        }
    u32x4_a hi, lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hi[i] = pack_bf16x2(p[2 * i], p[2 * i + 1]);
        lo[i] = pack_bf16x2(p[2 * i] - __uint_as_float(hi[i] << 16), p[2 * i + 1] - __uint_as_float(hi[i] & 0xFFFF0000u));
    }
    phi = __builtin_bit_cast(bf16x8_a, hi);
    plo = __builtin_bit_cast(bf16x8_a, lo);
}

// V chunks are staged as they lie in the cache, rows of DH channels, and read with the transposing LDS load into the B
// operand of P V (8 consecutive keys of a channel per lane); a transposed copy in memory was a pass over the whole V cache
// per layer (85 of 396 us for a refresh of 64 x 4096 keys).
// PRE: as in k_attn_select; kc and vc then hold the sequence's own positions, from pv.P on, pv.k and pv.v the prefix;
// 64-key chunks never straddle pv.P.
// NQT: query tiles of 16 rows per workgroup and block (see pv_split).
// Occupancy floors (4+ heads per group): four waves per SIMD at head size 64 (128 registers; the 18 values that do not
// fit are spilled outside the chunk loop), two at head size 128 (256 registers, no spills). Left alone the compiler takes
// 186 and 328 registers, and with one wave per SIMD the softmax's exp / pack chains and the MFMAs have nothing to
// overlap with: 2.90 -> 1.81 ms per launch at the 8B shape with 4096-token sequences.
template <int DH, int G, bool PRE, int NQT>
__global__ void __launch_bounds__(G * 64) __attribute__((amdgpu_waves_per_eu(DH == 64 && G >= 4 ? 4 : (DH == 128 && G >= 4 ? 2 : 1), 8)))
k_attn_pv(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, const bf16_t *__restrict__ vc,
          const SelRow *__restrict__ sel, float *__restrict__ o32, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hq,
          int Hkv, float scale, PrefixView pv)
{
    constexpr int NT = G * 64, KK = DH / 32, DT = DH / 16, KC = 64, QT = 16 * NQT;
    constexpr int KP = DH / 8;                              // 16-byte pieces per K row
    constexpr int PIECES = KC * KP / NT;                     // of K and of V, per thread and chunk
    constexpr int K_BYTES = KC * DH * 2, STAGE = 2 * K_BYTES;
    static_assert(KC * KP % NT == 0, "chunk / thread mismatch");
    extern __shared__ __align__(16) unsigned char pvl[];   // 2 stages of { K chunk, V chunk }

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the 8 XCDs round-robin in launch order; the gridDim.x workgroups of a (sequence, KV head) read the
    // same K and V, so they are renumbered to share an XCD (and its L2): of 8 * gridDim.x consecutive workgroups, those
    // with the same launch index modulo 8 form one group.
    int bx = blockIdx.x, kvh = blockIdx.y, s = blockIdx.z;
    {
        const int nbx = gridDim.x, n_grp = (int)(gridDim.y * gridDim.z);
        if (n_grp % 8 == 0) {
            const int id = bx + nbx * (kvh + (int)gridDim.y * s), chunk = id / (8 * nbx), within = id - chunk * (8 * nbx);
            const int g = chunk * 8 + (within & 7);
            bx = within >> 3;
            kvh = g % (int)gridDim.y;
            s = g / (int)gridDim.y;
        }
    }
    const int h = kvh * G + w;
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) return;
    // A workgroup takes query blocks n_qb - 1 - x and x: every workgroup streams the same number of causal keys.
    // With one block per workgroup the lifetimes differ by a factor of up to n_qb, and slots freed by the short
    // workgroups of a launch were seen to stay empty until the long ones around them had ended.
    // A grid of one workgroup per block: no partners (all of them are resident at once, see pv_split).
    const int n_qb = (Tn + QT - 1) / QT;
    const bool alone = (int)gridDim.x >= n_qb;
    for (int pass = 0; pass < 2; ++pass) {
    const int qb = pass == 0 ? n_qb - 1 - bx : bx;
    if (pass == 1 && (alone || qb >= n_qb - 1 - bx)) break; // the middle block of an odd count is its own partner
    const int q0 = qb * QT;
    const int rows = (Tn - q0 < QT) ? (Tn - q0) : QT;
    const int n_max = p0 + q0 + rows;                      // keys seen by the block's last live row
    const int n_chunks = (n_max + KC - 1) / KC;
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *kpre = nullptr, *vpre = nullptr;
    if constexpr (PRE) {                                    // own segment addressed by absolute key: bases minus P keys
        kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * DH - (int64_t)pv.P * DH;
        vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * DH - (int64_t)pv.P * DH;
        kpre = pv.k + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * DH;
        vpre = pv.v + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * DH;
    }

    // per-lane query state: lane l16 of every lane group owns query q0 + 16*qt + l16
    bf16x8_a qf[NQT][KK];
    float thr[NQT], mxl[NQT], den[NQT];
    int jstar[NQT], pos[NQT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        den[qt] = 0.f;
        const int qi = q0 + 16 * qt + l16;
        const bool live = qi < Tn;
        const int qr = live ? qi : Tn - 1;
        const bf16_t *qp = q + ((int64_t)s * Tn + qr) * (int64_t)(Hq * DH) + (int64_t)h * DH + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            qf[qt][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(qp + kk * 32));
        const SelRow sr = sel[((int64_t)s * Tn + qr) * Hq + h];
        thr[qt] = live ? sr.thr : __builtin_inff();        // dead rows of a ragged block keep nothing
        mxl[qt] = sr.mx * 1.44269504088896341f;
        jstar[qt] = sr.jstar;
        pos[qt] = p0 + qi;
    }
    const bool any_ties = __ballot(jstar[0] != 0x7FFFFFFF || jstar[NQT - 1] != 0x7FFFFFFF) != 0ull;

    floatx4_a oacc[NQT][DT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] = floatx4_a{0.f, 0.f, 0.f, 0.f};

    // staging: global -> registers -> LDS, one chunk ahead
    u32x4_a kreg0[PIECES], vreg0[PIECES];
#define SOL_PV_GLOAD(KR, VR, CH_)                                                                                  \
    {                                                                                                      \
        const int key0_ = (CH_) * KC;                                                                      \
        const bool pre_ = PRE && key0_ < pv.P;              /* chunk-uniform: P is a multiple of the chunk */ \
        const bf16_t *kb_ = pre_ ? kpre : kbase, *vb_ = pre_ ? vpre : vbase;                               \
        _Pragma("unroll") for (int i = 0; i < PIECES; ++i) {                                             \
            const int pc = i * NT + tid, row = pc / KP, piece = pc - row * KP;                             \
            int key = key0_ + row;                                                                         \
            if (key >= n_max) key = n_max - 1;              /* never used unmasked: beyond every row */     \
            KR[i] = *reinterpret_cast<const u32x4_a *>(kb_ + (int64_t)key * DH + piece * 8);               \
            VR[i] = *reinterpret_cast<const u32x4_a *>(vb_ + (int64_t)key * DH + piece * 8);               \
        }                                                                                                  \
    }
#define SOL_PV_LSTORE(KR, VR, STG_)                                                                                \
    {                                                                                                      \
        unsigned char *kb_ = pvl + (STG_) * STAGE, *vb_ = kb_ + K_BYTES;                                   \
        _Pragma("unroll") for (int i = 0; i < PIECES; ++i) {                                             \
            const int pc = i * NT + tid, row = pc / KP, piece = pc - row * KP;                             \
            *reinterpret_cast<u32x4_a *>(kb_ + row * (DH * 2) + ((piece ^ pv_swz_k<DH>(row)) << 4)) = KR[i]; \
            *reinterpret_cast<u32x4_a *>(vb_ + row * (DH * 2) + ((piece ^ pv_swz_v<DH>(row)) << 4)) = VR[i]; \
        }                                                                                                  \
    }

    // chunk ch is multiplied out of LDS stage ch % 2 while chunk ch + 1 (fetched one iteration ago) moves from
    // registers into the other stage and chunk ch + 2 is fetched: global latency has a whole iteration to hide in
    SOL_PV_GLOAD(kreg0, vreg0, 0);
    SOL_PV_LSTORE(kreg0, vreg0, 0);
    if (1 < n_chunks) SOL_PV_GLOAD(kreg0, vreg0, 1);
    __syncthreads();
    for (int ch = 0; ch < n_chunks; ++ch) {
        const int stg = ch & 1;
        // one register set: what was fetched an iteration ago goes to LDS, then the set is requested again
        if (ch + 1 < n_chunks) SOL_PV_LSTORE(kreg0, vreg0, stg ^ 1);
        if (ch + 2 < n_chunks) SOL_PV_GLOAD(kreg0, vreg0, ch + 2);
        const unsigned char *kb = pvl + stg * STAGE, *vb = kb + K_BYTES;
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            const int kb32 = ch * KC + cc * 32;             // first key of this 32-key sub-chunk
            if (kb32 < n_max) {
                // scores: MFMA row m of tile kt is key  kb32 + 8*(m >> 2) + 4*kt + (m & 3)
                floatx4_a st[NQT][2];                         // [qt][kt]
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    const int krow = cc * 32 + 8 * (l16 >> 2) + 4 * kt + (l16 & 3);
                    bf16x8_a kf[KK];
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
                        kf[kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(
                            kb + krow * (DH * 2) + (((kk * 4 + lg) ^ pv_swz_k<DH>(krow)) << 4)));
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt) {
                        floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk)
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kk], qf[qt][kk], acc, 0, 0, 0);
                        st[qt][kt] = acc;
                    }
                }
                bf16x8_a phi[NQT], plo[NQT];
                const int kfirst = kb32 + 8 * lg;
                const bool diag = kb32 + 31 > p0 + q0;      // some key of the sub-chunk is beyond some query
#pragma unroll
                for (int qt = 0; qt < NQT; ++qt) {
                    if (any_ties) pv_probs<true, true>(st[qt], scale, thr[qt], mxl[qt], jstar[qt], pos[qt], kfirst, den[qt], phi[qt], plo[qt]);
                    else if (diag) pv_probs<true, false>(st[qt], scale, thr[qt], mxl[qt], jstar[qt], pos[qt], kfirst, den[qt], phi[qt], plo[qt]);
                    else pv_probs<false, false>(st[qt], scale, thr[qt], mxl[qt], jstar[qt], pos[qt], kfirst, den[qt], phi[qt], plo[qt]);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const bf16x8_a vf = pv_read_v<DH>(vb, cc * 32 + 8 * lg, dt, l16);
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt) {
                        oacc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo[qt], vf, oacc[qt][dt], 0, 0, 0);
                        oacc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi[qt], vf, oacc[qt][dt], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();                                   // also frees both stages for the workgroup's next block
    }
#undef SOL_PV_GLOAD
#undef SOL_PV_LSTORE

    // ---- normalise and store: accumulator lane (l16, lg) register r is query 4*lg + r, column 16*dt + l16 ----
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        float dsum = den[qt];
        dsum += __shfl_xor(dsum, 16);
        dsum += __shfl_xor(dsum, 32);
        const float inv = dsum > 0.f ? 1.0f / dsum : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float iv = __shfl(inv, 4 * lg + r);
            const int qi = q0 + 16 * qt + 4 * lg + r;
            if (qi < Tn) {
                float *op = o32 + ((int64_t)s * Tn + qi) * (int64_t)(Hq * DH) + (int64_t)h * DH + l16;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) op[dt * 16] = oacc[qt][dt][r] * iv;
            }
        }
    }
    }   // pass
}

// The search for a decode row's threshold: wave_search_rows for one row whose columns several waves hold, which count between
// barriers and all run this on the same numbers. Done when exactly b of the n keys are >= thr, or, where ties leave no such
// pivot, when the bracket has closed on the b-th largest (exact = false). Invariant: count(key >= lo) >= b, count(key >= hi + 1) < b.
// m1, m2: mean and mean square of a sample of the row. The first pivot is the normal quantile (Abramowitz and Stegun 26.2.23) of the kept
// share. On normal rows 4.5 rounds where regula falsi on the counts from the row's extremes takes 6.4; but the last of them close
// in on one key, and the slowest of a launch's 32 rows takes 11. So once the bracket holds FEW keys they are gathered in the LDS
// and ranked there: 2.6 rounds, 4 for the slowest of 32. (Ranked by every wave for itself the 64 comparisons cost as much as
// the rounds they save: 16 waves share four SIMDs.) Skewed rows and rows with outliers take 4 to 8 where that regula falsi took 8 to 21,
// clusters and magnitudes over a hundred powers of two 15 to 29.
// us per layer of a replayed 1B step, that search -> this one, at kept shares 1/16, 1/8, 1/4, 1/2 and 1: one sequence of 4096 keys 68.5,
// 67.1, 66.4, 66.2, 57.3 -> 61.3, 61.6, 61.7, 61.8, 57.5; 8 of 2048 keys 101, 101, 100, 99, 88 -> 93, 93, 94, 94, 88; 64 of 8192 keys 278,
// 277, 280, 290, 269 -> 256, 258, 266, 279, 268. k_dec_select alone, one sequence of 4096 keys: 12.8 -> 8.6.
struct PivotSearch {
    static constexpr int FEW = 64;
    uint32_t lo, hi, thr = 0u;
    bool done = false, exact = true;
    float flo, fhi, glo, ghi, w_up = 1.0f, w_dn = 1.0f, fp, slope, t_b, nh, bf;
    int b, clo, chi = 0;                                     // count(key >= lo), count(key > hi)
    __device__ __forceinline__ PivotSearch(int n, int b_, uint32_t lo_, uint32_t hi_, float m1, float m2)
        : lo(lo_), hi(hi_), b(b_), clo(n)
    {
        const float nf = (float)n;
        bf = (float)b;
        nh = nf + 0.5f;
        t_b = __builtin_amdgcn_logf(bf * __builtin_amdgcn_rcpf((nf - bf) + 1.0f));
        flo = score_unkey(lo);
        fhi = score_unkey(hi);
        const float t_n = __builtin_amdgcn_logf(nh * 2.0f);
        glo = t_n - t_b;
        ghi = -t_n - t_b;
        const float sd = __builtin_amdgcn_sqrtf(__builtin_fmaxf(__builtin_fmaf(-m1, m1, m2), 0.f));
        const float p = (bf - 0.5f) * __builtin_amdgcn_rcpf(nf);     // upper tail at the threshold
        const float t = __builtin_amdgcn_sqrtf(-1.3862943611f * __builtin_amdgcn_logf(__builtin_fminf(p, 1.0f - p)));
        const float num = __builtin_fmaf(__builtin_fmaf(0.010328f, t, 0.802853f), t, 2.515517f);
        const float den = __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(0.001308f, t, 0.189269f), t, 1.432788f), t, 1.0f);
        const float z = t - num * __builtin_amdgcn_rcpf(den);
        fp = __builtin_fmaf(sd, p < 0.5f ? z : -z, m1);
        slope = sd * 2.5066283f * __builtin_amdgcn_exp2f(0.72134752f * z * z) * __builtin_amdgcn_rcpf(nf);
    }
    __device__ __forceinline__ uint32_t pivot(int it) const      // of (lo, hi]
    {
        uint32_t mid = score_key(fp);
        mid = __builtin_elementwise_min(__builtin_elementwise_max(mid, lo + 1u), hi);
        if (it >= 12) mid = lo + ((hi - lo + 1u) >> 1);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)mid);
    }
    __device__ __forceinline__ void count(int it, uint32_t mid, int cnt)
    {
        const float cf = (float)cnt, fmid = score_unkey(mid);
        const float g = __builtin_amdgcn_logf((cf + 0.5f) * __builtin_amdgcn_rcpf(nh - cf)) - t_b;
        if (cnt == b) { thr = mid; done = true; }
        else if (cnt > b) {
            lo = mid; clo = cnt; flo = fmid; glo = g;
            ghi *= w_up;
            w_up = 0.5f; w_dn = 1.0f;
        } else {
            hi = mid - 1u; chi = cnt; fhi = fmid; ghi = g;
            glo *= w_dn;
            w_up = 1.0f; w_dn = 0.5f;
        }
        fp = it == 0 ? __builtin_fmaf(cf - bf, slope, fmid) : __builtin_fmaf(fhi - flo, glo * __builtin_amdgcn_rcpf(glo - ghi), flo);
    }
    __device__ __forceinline__ bool few() const { return !done && clo - chi <= FEW; }
    __device__ __forceinline__ bool open() const { return !done && lo < hi && clo - chi > FEW; }
};
// The keys of a bracket that holds few of them, in any order: n_few is 0 before, a barrier follows.
template <int SLOTS>
__device__ __forceinline__ void gather_few(const PivotSearch &find, const uint32_t (&key)[SLOTS], uint32_t *cand, int *n_few)
{
#pragma unroll
    for (int i = 0; i < SLOTS; ++i)
        if (key[i] - find.lo <= find.hi - find.lo) {
            const int at = atomicAdd(n_few, 1);
            if (at < PivotSearch::FEW) cand[at] = key[i];
        }
}
// The (b - count above the bracket)-th largest of them, and whether it is the last of its value; one wave, cand 0 behind the keys.
__device__ __forceinline__ uint2 rank_few(const PivotSearch &find, const uint32_t *cand, int lane)
{
    const int m = find.clo - find.chi, k = find.b - find.chi;
    const uint32_t own = cand[lane];
    int gt = 0;
    for (int i = 0; i < m; i += 8) {
        const uint4 c = *reinterpret_cast<const uint4 *>(cand + i), d = *reinterpret_cast<const uint4 *>(cand + i + 4);
        gt += (c.x > own) + (c.y > own) + (c.z > own) + (c.w > own) + (d.x > own) + (d.y > own) + (d.z > own) + (d.w > own);
    }
    const uint32_t thr = wave_min_u32(lane < m && gt < k ? own : 0xFFFFFFFFu);
    return make_uint2(thr, __popcll(__ballot(lane < m && own >= thr)) == k);
}

// =================================================================================================
// Decode attention (one query per sequence, bf16, HBM-bound): one workgroup of 16 waves per
// (sequence, KV head) serves the HPB = 4 query heads that share that KV head, so K is streamed from
// HBM once and V rows are fetched once if any of the four heads kept them.
//   1. scores on MFMA: A = a tile of 16 keys (each lane loads 16 contiguous bytes of a K row straight
//      from global memory, four tiles in flight per wave), B = the query heads as columns; fp32 scores
//      of all four heads go to LDS.
//   2. selection: the 4 waves of a head hold a quarter of the row each in registers and search the
//      key range together, exchanging their ballot counts through LDS once per step.
//   3. softmax numerators back to LDS, 4. V rows gathered where any head kept the key.
// =================================================================================================
constexpr int DEC_WAVES = 16, DEC_BLOCK = DEC_WAVES * 64, DEC_HPB = 4, DEC_GW = DEC_WAVES / DEC_HPB;
// The halving steps lane ^ O, lane ^ 2 O, .. lane ^ 32, with every index a constant (as one loop over an array they end in
// compare / select chains of thousands of instructions wherever the loop is unrolled too late).
template <int N> struct DecVals { float v[N]; };
template <int O, int N>
__device__ __forceinline__ auto dec_halve(const DecVals<N> &a, int lane, int &fbase)
{
    DecVals<N / 2> r;
    const bool up = (lane & O) != 0;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const float keep = up ? a.v[i + N / 2] : a.v[i], send = up ? a.v[i] : a.v[i + N / 2];
        r.v[i] = keep + __shfl_xor(send, O, 64);
    }
    fbase += up ? N / 2 : 0;
    if constexpr (O < 32) return dec_halve<2 * O>(r, lane, fbase);
    else return r;
}

// The last phases of the decode kernels: sc holds the softmax numerators of the HPB heads ([HPB][lpad], 0 for
// dropped keys), den(head) the denominators (called after a barrier); o_row receives HPB * DH outputs. NW waves.
//   4. o = sum_j p_j v_j, reading only V rows kept by at least one head; 5. reduction over lanes and waves.
template <int DH, int NW, class Den>
__device__ __forceinline__ void decode_pv_tail(float *sc, int lpad, int n, const bf16_t *__restrict__ vbase,
                                               Den den, float *__restrict__ o_row)
{
    constexpr int VEC = 8, LPK = DH / VEC, KPI = NW * 64 / LPK;
    const int tid = threadIdx.x;
    // ---- 4. o = sum p_j v_j over rows any head kept ---------------------------------------------------
    const int ks = tid / LPK, cs = tid - ks * LPK;
    float acc[DEC_HPB][VEC];
#pragma unroll
    for (int hh = 0; hh < DEC_HPB; ++hh)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[hh][e] = 0.f;
    constexpr int UV = 4;
    for (int j0 = ks; j0 < n; j0 += KPI * UV) {
        float p[UV][DEC_HPB];
        u32x4_a vv[UV];
        bool any[UV];
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            const int j = j0 + u * KPI;
            any[u] = false;
#pragma unroll
            for (int hh = 0; hh < DEC_HPB; ++hh) {
                p[u][hh] = (j < n) ? sc[hh * lpad + j] : 0.f;
                any[u] |= p[u][hh] != 0.f;
            }
            vv[u] = u32x4_a{0u, 0u, 0u, 0u};
            if (any[u]) vv[u] = *reinterpret_cast<const u32x4_a *>(vbase + (int64_t)j * DH + cs * VEC);
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            if (any[u]) {
#pragma unroll
                for (int wi = 0; wi < 4; ++wi) {
                    const float v0 = __uint_as_float(vv[u][wi] << 16), v1 = __uint_as_float(vv[u][wi] & 0xFFFF0000u);
#pragma unroll
                    for (int hh = 0; hh < DEC_HPB; ++hh) {
                        acc[hh][2 * wi] = fmaf(p[u][hh], v0, acc[hh][2 * wi]);
                        acc[hh][2 * wi + 1] = fmaf(p[u][hh], v1, acc[hh][2 * wi + 1]);
                    }
                }
            }
        }
    }
    // ---- 5. reduction --------------------------------------------------------------------------------
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Reduce over the key slots of a wave (lanes with equal cs) by halving butterflies: at each step a lane
    // keeps one half of its values and hands the other half to its partner, so the 4 * VEC values per lane
    // end as 4 * VEC * LPK / 64 fully reduced ones; then across waves in fixed order.
    DecVals<DEC_HPB * VEC> flat;
#pragma unroll
    for (int i = 0; i < DEC_HPB * VEC; ++i) flat.v[i] = acc[i / VEC][i % VEC];
    int fbase = 0;                                             // first flattened (head, element) index this lane keeps
    const auto kept = dec_halve<LPK>(flat, lane, fbase);
    const float *accf = kept.v;
    constexpr int NKEEP = DEC_HPB * VEC * LPK / 64;            // 4 (head_dim 64) or 8 (head_dim 128)
    __syncthreads();                                           // all reads of the numerators are done
    float *ored = sc;                                          // [NW][HPB][DH]
    {
        const int hh = fbase / VEC, e0 = fbase - hh * VEC;     // NKEEP values of one head, elements e0..e0+NKEEP-1
        float *dst = ored + ((size_t)w * DEC_HPB + hh) * DH + (lane & (LPK - 1)) * VEC + e0;
#pragma unroll
        for (int i = 0; i < NKEEP; i += 4)
            *reinterpret_cast<f32x4_a *>(dst + i) = f32x4_a{accf[i], accf[i + 1], accf[i + 2], accf[i + 3]};
    }
    __syncthreads();
    for (int idx = tid; idx < DEC_HPB * DH; idx += NW * 64) {
        const int hh = idx / DH;
        float t = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) t += ored[(size_t)ww * DEC_HPB * DH + idx];
        o_row[idx] = t / den(hh);
    }
}

template <int DH, int SLOTS>
__global__ void __launch_bounds__(DEC_BLOCK)
k_attn_decode(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, const bf16_t *__restrict__ vc,
              float *__restrict__ o32, const RowAct *__restrict__ ra, const int32_t *__restrict__ cache_len,
              const int32_t *__restrict__ seq_order, int L_max, int Hq, int Hkv, float scale, int *flags)
{
    constexpr int KK = DH / 32, SLICE = SLOTS * 64, LPAD = SLICE * DEC_GW, NJ = SLOTS / 4;
    extern __shared__ __align__(16) float sc[];               // [DEC_HPB][LPAD]; later partial O [DEC_WAVES][HPB][DH]
    __shared__ int s_cnt[2][DEC_WAVES];
    __shared__ uint32_t s_min[DEC_WAVES], s_max[DEC_WAVES];
    __shared__ float s_s1[DEC_WAVES], s_s2[DEC_WAVES];
    __shared__ __align__(16) uint32_t s_cand[DEC_HPB][PivotSearch::FEW];
    __shared__ int s_few[DEC_HPB];
    __shared__ uint2 s_rank[DEC_HPB];
    __shared__ int s_done[2][DEC_HPB];
    __shared__ int s_gt[DEC_WAVES];
    __shared__ float s_den[DEC_WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = blockIdx.x;
    // Longest sequences first: workgroups are handed to compute units in launch order, one per CU, so with
    // mixed cache lengths the last round would otherwise wait for a long row that started late. seq_order
    // (k_seq_order, once per decode step) lists the sequences by decreasing cache length.
    int s = seq_order ? seq_order[blockIdx.y] : (int)blockIdx.y;
    s = __builtin_amdgcn_readfirstlane(s);
    const int p0 = __builtin_amdgcn_readfirstlane(cache_len[s]);
    if (p0 < 0 || p0 + 1 > L_max) {
        if (tid == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
        return;
    }
    const int n = p0 + 1;                                      // keys 0..p0 (the new token's key included)
    const RowAct act = ra[s];
    const int b = __builtin_amdgcn_readfirstlane(budget_ceil(act.keep_num, act.keep_den, n));   // 64-bit divide runs on the VALU
    const int h0 = kvh * DEC_HPB;
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const int l16 = lane & 15, lg = lane >> 4;

    // ---- 1. scores -----------------------------------------------------------------------------
    {
        bf16x8_a qf[KK];                                       // B operand: column = head (l16 < HPB), zero elsewhere
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            u32x4_a v = {0u, 0u, 0u, 0u};
            if (l16 < DEC_HPB)
                v = *reinterpret_cast<const u32x4_a *>(q + (int64_t)s * (Hq * DH) + (int64_t)(h0 + l16) * DH + kk * 32 + lg * 8);
            qf[kk] = __builtin_bit_cast(bf16x8_a, v);
        }
        const int n_kt = (n + 15) >> 4;
        // two register sets of key tiles: the loads of the next group are in flight while this group is multiplied
        constexpr int U = DH == 64 ? 4 : 2, STEP = DEC_WAVES * U;
        bf16x8_a kfa[U][KK], kfb[U][KK];
#define SOL_DEC_LOADK(KF, KT0_)                                                                            \
    _Pragma("unroll") for (int u = 0; u < U; ++u) {                                                        \
        int key = ((KT0_) + u * DEC_WAVES) * 16 + l16;                                                     \
        if (key >= n) key = n - 1;                                                                         \
        const bf16_t *kp = kbase + (int64_t)key * DH + lg * 8;                                             \
        _Pragma("unroll") for (int kk = 0; kk < KK; ++kk)                                                  \
            KF[u][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(kp + kk * 32));    \
    }
#define SOL_DEC_MMAK(KF, KT0_)                                                                             \
    _Pragma("unroll") for (int u = 0; u < U; ++u) {                                                        \
        const int kt = (KT0_) + u * DEC_WAVES;                                                             \
        if (kt < n_kt) {                                                                                   \
            floatx4_a acc = {0.f, 0.f, 0.f, 0.f};                                                          \
            _Pragma("unroll") for (int kk = 0; kk < KK; ++kk)                                              \
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(KF[u][kk], qf[kk], acc, 0, 0, 0);            \
            if (l16 < DEC_HPB) {                                                                           \
                _Pragma("unroll") for (int r = 0; r < 4; ++r) sc[l16 * LPAD + kt * 16 + lg * 4 + r] = acc[r] * scale; \
            }                                                                                              \
        }                                                                                                  \
    }
        int kt0 = w;
        if (kt0 < n_kt) SOL_DEC_LOADK(kfa, kt0);
        for (; kt0 < n_kt; kt0 += 2 * STEP) {
            if (kt0 + STEP < n_kt) SOL_DEC_LOADK(kfb, kt0 + STEP);
            SOL_DEC_MMAK(kfa, kt0);
            if (kt0 + 2 * STEP < n_kt) SOL_DEC_LOADK(kfa, kt0 + 2 * STEP);
            if (kt0 + STEP < n_kt) SOL_DEC_MMAK(kfb, kt0 + STEP);
        }
#undef SOL_DEC_LOADK
#undef SOL_DEC_MMAK
    }
    __syncthreads();

    // ---- 2. selection: DEC_GW waves per head, each with SLICE columns in registers --------------
    const int head = w / DEC_GW, wg = w - head * DEC_GW;
    const int base = wg * SLICE;
    int n_loc = n - base;
    n_loc = n_loc < 0 ? 0 : (n_loc > SLICE ? SLICE : n_loc);   // valid columns held by this wave
    float *row = sc + head * LPAD + base;
    uint32_t key[SLOTS];                                        // the score itself is recovered from its key
    uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
    float s1 = 0.f, s2 = 0.f;                                  // over every fourth column
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (256 * j < n_loc) {
            const f32x4_a v = *reinterpret_cast<const f32x4_a *>(row + 256 * j + 4 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool valid = 256 * j + 4 * lane + e < n_loc;
                const uint32_t kv = valid ? score_key(v[e]) : 0u;
                key[4 * j + e] = kv;
                kmax = kv > kmax ? kv : kmax;
                kmin = (valid && kv < kmin) ? kv : kmin;
                if (e == 0 && valid) { s1 += v[0]; s2 = __builtin_fmaf(v[0], v[0], s2); }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) key[4 * j + e] = 0u;
        }
    }
    kmax = wave_max_u32(kmax);
    kmin = wave_min_u32(kmin);
    if (b < n) {
        s1 = wave_sum_dpp(s1);
        s2 = wave_sum_dpp(s2);
    }
    if (tid < DEC_HPB) s_few[tid] = 0;
    if (tid < DEC_HPB * PivotSearch::FEW) s_cand[tid / PivotSearch::FEW][tid % PivotSearch::FEW] = 0u;
    if (lane == 0) { s_max[w] = kmax; s_min[w] = kmin; s_s1[w] = s1; s_s2[w] = s2; }
    __syncthreads();
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    s1 = s2 = 0.f;
#pragma unroll
    for (int i = 0; i < DEC_GW; ++i) {
        const uint32_t a = s_min[head * DEC_GW + i], c = s_max[head * DEC_GW + i];
        lo = a < lo ? a : lo;
        hi = c > hi ? c : hi;
        s1 += s_s1[head * DEC_GW + i];
        s2 += s_s2[head * DEC_GW + i];
    }
    // values read back from LDS are wave-uniform: move them to scalar registers so that the search
    // below is scalar control flow
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
    const float mx = score_unkey(hi);                          // the head's best score, always kept
    uint32_t thr = 1u;                                         // budget keeps all: every valid key passes
    bool exact = true;
    if (b < n) {                                               // the same for the four heads
        const float inv = 1.0f / (float)((n + 3) >> 2);
        PivotSearch find(n, b, lo, hi, s1 * inv, s2 * inv);
        for (int it = 0; it < 48; ++it) {
            const int par = it & 1;
            uint32_t mid = 0u;
            const bool go = find.open();
            if (go) {
                mid = find.pivot(it);
                const int c = wave_count_ge<SLOTS>(key, n_loc, mid);
                if (lane == 0) s_cnt[par][w] = c;
            }
            if (wg == 0 && lane == 0) s_done[par][head] = !go;
            __syncthreads();
            if (go) {
                int cnt = 0;
#pragma unroll
                for (int i = 0; i < DEC_GW; ++i) cnt += s_cnt[par][head * DEC_GW + i];
                find.count(it, mid, __builtin_amdgcn_readfirstlane(cnt));
            }
            const bool all_done =
                __builtin_amdgcn_readfirstlane(s_done[par][0] & s_done[par][1] & s_done[par][2] & s_done[par][3]) != 0;
            if (all_done) break;                                   // uniform: every wave reads the same flags
        }
        const bool few = find.few();
        if (few) gather_few<SLOTS>(find, key, s_cand[head], &s_few[head]);
        __syncthreads();
        if (few && wg == head) {                                   // (these four waves run on different SIMDs)
            const uint2 r = rank_few(find, s_cand[head], lane);
            if (lane == 0) s_rank[head] = r;
        }
        __syncthreads();
        if (few) { find.thr = s_rank[head].x; find.exact = s_rank[head].y != 0; }
        else if (!find.done) { find.thr = find.lo; find.exact = false; }      // the bracket has closed on many equal keys
        thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)find.thr);
        exact = __builtin_amdgcn_readfirstlane((int)find.exact) != 0;
    }
    // Ties at the threshold go to the lower columns. Rare for fp32 scores, so the fix-up is a plain
    // loop by the first wave of the head over the row in LDS: tied keys beyond the quota get -inf.
    {
        const bool need = (b < n) && !exact;
        int gt = 0;
        if (need) {
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) gt += __popcll(__ballot(key[i] > thr));
        }
        if (lane == 0) s_gt[w] = gt;
        __syncthreads();
        if (need && wg == 0) {
            int quota = b;
#pragma unroll
            for (int i = 0; i < DEC_GW; ++i) quota -= s_gt[head * DEC_GW + i];
            quota = __builtin_amdgcn_readfirstlane(quota);      // >= 1 tied keys stay
            float *hrow = sc + head * LPAD;
            int taken = 0;
            for (int c0 = 0; c0 < n; c0 += 64) {
                const int col = c0 + lane;
                const bool tie = col < n && score_key(hrow[col]) == thr;
                const unsigned long long bal = __ballot(tie);
                const int rank = taken + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
                if (tie && rank >= quota) hrow[col] = -INFINITY;
                taken += __popcll(bal);
            }
        }
        __syncthreads();
    }

    // ---- 3. softmax numerators back to LDS ----------------------------------------------------------
    // The scores are still in registers (as keys); only a row the tie fix-up rewrote is read back.
    float den = 0.f;
    const bool reread = (b < n) && !exact;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (256 * j < n_loc) {
            f32x4_a v = {0.f, 0.f, 0.f, 0.f};
            if (reread) v = *reinterpret_cast<const f32x4_a *>(row + 256 * j + 4 * lane);
            f32x4_a p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t kv = reread ? score_key(v[e]) : key[4 * j + e];
                const float sv = reread ? v[e] : score_unkey(key[4 * j + e]);
                const bool on = (256 * j + 4 * lane + e < n_loc) && kv >= thr;
                p[e] = on ? __expf(sv - mx) : 0.f;
                den += p[e];
            }
            *reinterpret_cast<f32x4_a *>(row + 256 * j + 4 * lane) = p;
        }
    }
    den = wave_sum_dpp(den);
    if (lane == 0) s_den[w] = den;
    __syncthreads();

    decode_pv_tail<DH, DEC_WAVES>(sc, LPAD, n, vbase, [&](int hh) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < DEC_GW; ++i) d += s_den[hh * DEC_GW + i];
        return d;
    }, o32 + (int64_t)s * (Hq * DH) + (int64_t)h0 * DH);
}

template <int DH, int SLOTS>
static bool launch_attn_decode_t(const void *q, const void *kc, const void *vc, float *o32, const RowAct *ra,
                                 const int32_t *cache_len, const int32_t *seq_order, int B, int L_max, int Hq, int Hkv,
                                 int *flags, hipStream_t st)
{
    auto kern = k_attn_decode<DH, SLOTS>;
    const size_t lds = (size_t)DEC_HPB * SLOTS * 64 * DEC_GW * 4;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return false;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3(Hkv, B), dim3(DEC_BLOCK), lds, st, (const bf16_t *)q, (const bf16_t *)kc,
                       (const bf16_t *)vc, o32, ra, cache_len, seq_order, L_max, Hq, Hkv, 1.0f / sqrtf((float)DH), flags);
    return true;
}

// =================================================================================================
// The same attention for few sequences: with B * Hkv items for 256 CUs the one-workgroup-per-item kernel leaves most of
// the chip idle and takes an item's whole latency (39 us at 4096 keys for any B up to 32). Here an item's keys are
// spread over workgroups, in three launches (4.4 + 8.6 + 7.7 us there, 4.3 + 4.3 + 6.8 where the budget keeps all) with the scores between them in global memory (16
// bytes per key and KV head against the key's 128 or 256 bytes of K; they stay in the caches). Every sum is made in the
// order of that kernel, so that a sequence's result does not depend on how many others there are:
//   k_dec_scores  : scores of DSP_KEYS keys for the 4 heads of a KV group (the MFMA sequence of k_attn_decode)
//   k_dec_select  : per head, 16 waves: the exact threshold of the budget, the last kept tie, the maximum and denominator
//   k_dec_values  : softmax numerators of a sixteenth of the keys and their sum over the V rows -> partial outputs, which
//                   the row quantiser sums in order and divides
// Bound: launch latencies for one or two sequences, HBM (V rows of dropped keys included) above.
// =================================================================================================
constexpr int DSP_KEYS = 256;                                // keys of a k_dec_scores workgroup: four tiles of 16 per wave
constexpr int DSP_MAX_L = 9216;

template <int DH>
__global__ void __launch_bounds__(256)
k_dec_scores(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, float *__restrict__ scores,
             const int32_t *__restrict__ cache_len, int L_max, int Hq, int Hkv, int lpad, float scale, int *flags)
{
    constexpr int KK = DH / 32, U = DSP_KEYS / 64;           // key tiles of a wave, all in flight
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int kvh = blockIdx.y, s = blockIdx.z, h0 = kvh * DEC_HPB;
    const int p0 = __builtin_amdgcn_readfirstlane(cache_len[s]);
    if (p0 < 0 || p0 + 1 > L_max) {
        if (threadIdx.x == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
        return;
    }
    const int n = p0 + 1, kt0 = (int)blockIdx.x * (DSP_KEYS / 16) + w * U;
    if (kt0 * 16 >= n) return;
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    bf16x8_a qf[KK], kf[U][KK];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int key = (kt0 + u) * 16 + l16;
        if (key >= n) key = n - 1;
        const bf16_t *kp = kbase + (int64_t)key * DH + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) kf[u][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(kp + kk * 32));
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        u32x4_a v = {0u, 0u, 0u, 0u};
        if (l16 < DEC_HPB)
            v = *reinterpret_cast<const u32x4_a *>(q + (int64_t)s * (Hq * DH) + (int64_t)(h0 + l16) * DH + kk * 32 + lg * 8);
        qf[kk] = __builtin_bit_cast(bf16x8_a, v);
    }
    float *row = scores + ((int64_t)s * Hq + h0 + l16) * lpad;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][kk], qf[kk], acc, 0, 0, 0);
        const int j = (kt0 + u) * 16 + lg * 4;               // entries from n on are never read (lpad is a multiple of 64)
        if (l16 < DEC_HPB && j < n)
            *reinterpret_cast<f32x4_a *>(row + j) = f32x4_a{acc[0] * scale, acc[1] * scale, acc[2] * scale, acc[3] * scale};
    }
}

constexpr int DSEL_WAVES = 16;                               // of one head: a round of the search counts SLOTS columns per lane
// NJU: SLOTS / 4 of k_attn_decode for the same L_max, which says how its denominator is summed
template <int SLOTS, int NJU>
__global__ void __launch_bounds__(DSEL_WAVES * 64)
k_dec_select(const float *__restrict__ scores, DecSel *__restrict__ sel, const RowAct *__restrict__ ra,
             const int32_t *__restrict__ cache_len, int L_max, int Hq, int lpad)
{
    constexpr int SLICE = SLOTS * 64, NJ = SLOTS / 4;
    __shared__ int s_cnt[2][DSEL_WAVES], s_gt[DSEL_WAVES], s_tie[DSEL_WAVES], s_last;
    __shared__ uint32_t s_min[DSEL_WAVES], s_max[DSEL_WAVES];
    __shared__ float s_s1[DSEL_WAVES], s_s2[DSEL_WAVES];
    __shared__ __align__(16) uint32_t s_cand[PivotSearch::FEW];
    __shared__ int s_few;
    __shared__ uint2 s_rank;
    __shared__ float s_den[DEC_GW];
    __shared__ __align__(16) float s_p[DSEL_WAVES * SLICE];
    static_assert(DEC_GW * NJU * 256 <= DSEL_WAVES * SLICE, "");
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int head = blockIdx.x, s = blockIdx.y;
    const int p0 = __builtin_amdgcn_readfirstlane(cache_len[s]);
    if (p0 < 0 || p0 + 1 > L_max) return;
    const int n = p0 + 1, base = w * SLICE;
    int n_loc = n - base;
    n_loc = n_loc < 0 ? 0 : (n_loc > SLICE ? SLICE : n_loc); // columns held by this wave
    const RowAct act = ra[s];
    const int b = __builtin_amdgcn_readfirstlane(budget_ceil(act.keep_num, act.keep_den, n));
    const float *row = scores + ((int64_t)s * Hq + head) * lpad + base;
    uint32_t key[SLOTS];
    uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
    float s1 = 0.f, s2 = 0.f;                                // over every fourth column
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = 256 * j + 4 * lane;
        f32x4_a v = {0.f, 0.f, 0.f, 0.f};
        if (c < n_loc) v = *reinterpret_cast<const f32x4_a *>(row + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool valid = c + e < n_loc;
            const uint32_t kv = valid ? score_key(v[e]) : 0u;
            key[4 * j + e] = kv;
            kmax = kv > kmax ? kv : kmax;
            kmin = (valid && kv < kmin) ? kv : kmin;
            if (e == 0 && valid) { s1 += v[0]; s2 = __builtin_fmaf(v[0], v[0], s2); }
        }
    }
    kmax = wave_max_u32(kmax);
    kmin = wave_min_u32(kmin);
    if (b < n) {
        s1 = wave_sum_dpp(s1);
        s2 = wave_sum_dpp(s2);
    }
    if (threadIdx.x == 0) s_few = 0;
    if (threadIdx.x < PivotSearch::FEW) s_cand[threadIdx.x] = 0u;
    if (lane == 0) { s_max[w] = kmax; s_min[w] = kmin; s_s1[w] = s1; s_s2[w] = s2; }
    __syncthreads();
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    s1 = s2 = 0.f;
#pragma unroll
    for (int i = 0; i < DSEL_WAVES; ++i) {
        lo = s_min[i] < lo ? s_min[i] : lo;
        hi = s_max[i] > hi ? s_max[i] : hi;
        s1 += s_s1[i];
        s2 += s_s2[i];
    }
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
    const float mx = score_unkey(hi);                        // the head's best score, always kept
    uint32_t thr = 1u;                                       // budget keeps all: every valid key passes
    bool exact = true;
    if (b < n) {                                             // every wave runs the same steps
        const float inv = 1.0f / (float)((n + 3) >> 2);
        PivotSearch find(n, b, lo, hi, s1 * inv, s2 * inv);
        for (int it = 0; it < 48 && find.open(); ++it) {
            const uint32_t mid = find.pivot(it);
            const int c = wave_count_ge<SLOTS>(key, n_loc, mid);
            if (lane == 0) s_cnt[it & 1][w] = c;
            __syncthreads();
            int cnt = 0;
#pragma unroll
            for (int i = 0; i < DSEL_WAVES; ++i) cnt += s_cnt[it & 1][i];
            find.count(it, mid, __builtin_amdgcn_readfirstlane(cnt));
        }
        if (find.few()) {
            gather_few<SLOTS>(find, key, s_cand, &s_few);
            __syncthreads();
            if (w == 0) {
                const uint2 r = rank_few(find, s_cand, lane);
                if (lane == 0) s_rank = r;
            }
            __syncthreads();
            find.thr = s_rank.x;
            find.exact = s_rank.y != 0;
        } else if (!find.done) { find.thr = find.lo; find.exact = false; }     // the bracket has closed on many equal keys
        thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)find.thr);
        exact = __builtin_amdgcn_readfirstlane((int)find.exact) != 0;
    }
    // ties at the threshold go to the lower columns: the last one kept
    int jstar = 0x7FFFFFFF;
    if (b < n && !exact) {                                   // the same for all waves
        int gt = 0, eq = 0;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            gt += __popcll(__ballot(key[i] > thr));
            eq += __popcll(__ballot(key[i] == thr));
        }
        if (lane == 0) { s_gt[w] = gt; s_tie[w] = eq; }
        if (threadIdx.x == 0) s_last = 0x7FFFFFFF;
        __syncthreads();
        int quota = b;
#pragma unroll
        for (int i = 0; i < DSEL_WAVES; ++i) quota -= s_gt[i];
        for (int i = 0; i < w; ++i) quota -= s_tie[i];       // ties left for this wave's columns
        quota = __builtin_amdgcn_readfirstlane(quota);
        if (quota >= 1 && quota <= eq) {                     // exactly one wave holds the quota-th tie
            int taken = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                int below = 0, here = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned long long bal = __ballot(key[4 * j + e] == thr);
                    below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, below));
                    here += __popcll(bal);
                }
                int rank = taken + below;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (key[4 * j + e] == thr && rank++ == quota - 1) s_last = base + 256 * j + 4 * lane + e;
                taken += here;
            }
        }
        __syncthreads();
        jstar = s_last;
    }
    // the denominator, in the order of k_attn_decode: DEC_GW waves with NJU blocks of 256 columns each
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = 256 * j + 4 * lane;
        f32x4_a p;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t kv = key[4 * j + e];
            const bool kept = c + e < n_loc && (kv > thr || (kv == thr && base + c + e <= jstar));
            p[e] = kept ? __expf(score_unkey(kv) - mx) : 0.f;
        }
        *reinterpret_cast<f32x4_a *>(s_p + base + c) = p;
    }
    __syncthreads();
    if (w < DEC_GW) {
        float den = 0.f;
#pragma unroll
        for (int j = 0; j < NJU; ++j) {
            const f32x4_a p = *reinterpret_cast<const f32x4_a *>(s_p + (w * NJU + j) * 256 + 4 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) den += p[e];
        }
        den = wave_sum_dpp(den);
        if (lane == 0) s_den[w] = den;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < DEC_GW; ++i) d += s_den[i];
        sel[(int64_t)s * Hq + head] = DecSel{thr, mx, d, jstar};
    }
}

// grid (16, Hkv, B): workgroup ww does what wave ww of k_attn_decode does, its key slots and its order of sums, and wave h
// one of the KV head's four query heads: part [16][B][Hq * DH], which the row quantiser sums and divides as that kernel
// does. All V rows of the slots (kept or not) go straight to LDS, up to DSV_STEPS steps at once, so that a workgroup waits
// for memory once and the four waves read each row from there. The loops stay rolled on purpose: a launch this short is
// bound by latencies, instruction fetches among them (unrolled, with V in registers: 11.3 us at one sequence of the 1B
// shape and 4096 keys).
constexpr int DSV_STEPS = 48;                                // 1 KB of V each
template <int DH>
__global__ void __launch_bounds__(256)
k_dec_values(const float *__restrict__ scores, const DecSel *__restrict__ sel, const bf16_t *__restrict__ vc,
             float *__restrict__ part, const int32_t *__restrict__ cache_len, int L_max, int Hq, int Hkv, int lpad, int cap)
{
    constexpr int LPK = DH / 8, SPW = 64 / LPK, KPI = DEC_WAVES * SPW;
    extern __shared__ __align__(16) unsigned char dvl[];     // [cap][64 lanes][8] bf16, then numerators [4][steps * SPW]
    const int lane = threadIdx.x & 63, slot = lane / LPK, cs = lane - slot * LPK;
    const int h = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int kvh = blockIdx.y, s = blockIdx.z, head = kvh * DEC_HPB + h, first = (int)blockIdx.x * SPW;
    const int p0 = __builtin_amdgcn_readfirstlane(cache_len[s]);
    if (p0 < 0 || p0 + 1 > L_max) return;
    const int n = p0 + 1, nit = (n + KPI - 1) / KPI;
    const bf16_t *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH + cs * 8;
    const DecSel d = sel[(int64_t)s * Hq + head];
    const float *srow = scores + ((int64_t)s * Hq + head) * lpad;
    float *my = reinterpret_cast<float *>(dvl + (size_t)cap * 1024) + h * ((L_max + KPI - 1) / KPI) * SPW;
    DecVals<8> acc;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc.v[e] = 0.f;
    for (int c0 = 0; c0 < nit; c0 += cap) {
        const int c1 = c0 + cap < nit ? c0 + cap : nit;
        if (c0) __syncthreads();                             // the previous steps' rows have been read
        for (int i = c0 + h; i < c1; i += DEC_HPB) {
            int j = i * KPI + first + slot;
            if (j >= n) j = n - 1;                           // weight 0
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                         ::"v"(vbase + (int64_t)j * DH), "s"((i - c0) * 1024) : "memory", "m0");
        }
        if (c0 == 0) {
#pragma unroll 4
            for (int i = lane; i < nit * SPW; i += 64) {     // this wave's numerators, the slots of a step together
                const int j = i / SPW * KPI + first + i % SPW;
                const float v = srow[j < n ? j : n - 1];
                const uint32_t kv = score_key(v);
                const bool kept = j < n && (kv > d.thr || (kv == d.thr && j <= d.jstar));
                my[i] = kept ? __expf(v - d.mx) : 0.f;
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll 4
        for (int i = c0; i < c1; ++i) {
            const u32x4_a v = *reinterpret_cast<const u32x4_a *>(dvl + (i - c0) * 1024 + lane * 16);
            const float p = my[i * SPW + slot];
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) {
                const uint32_t x = p != 0.f ? v[wi] : 0u;    // a row that the head dropped may hold anything
                acc.v[2 * wi] = fmaf(p, __uint_as_float(x << 16), acc.v[2 * wi]);
                acc.v[2 * wi + 1] = fmaf(p, __uint_as_float(x & 0xFFFF0000u), acc.v[2 * wi + 1]);
            }
        }
    }
    int fbase = 0;
    const auto kept = dec_halve<LPK>(acc, lane, fbase);
    float *dst = part + (((int64_t)blockIdx.x * gridDim.z + s) * Hq + head) * DH + cs * 8 + fbase;
#pragma unroll
    for (int i = 0; i < LPK / 8; ++i) dst[i] = kept.v[i];
}

// Scratch of the split path for B sequences: scores, selection rows and partial outputs. 0: the shape, or B, is not its.
// It pays while few items leave most CUs of the one-workgroup-per-item kernel idle and their rows are long enough for that
// kernel's latency to show. What a row holds is not known here, only what its cache can hold: rows of few keys pay for the two
// launches more and the wider fold. Per layer of a graph-replayed step, caches of 8184 positions (us, one workgroup per item ->
// split, at 300 / 1000 / 2000 / 8000 keys): 1B shape, B = 1: 63 -> 64, 69 -> 65, 79 -> 66, 115 -> 75; B = 4: 88 -> 93, 94 -> 94, 105 -> 95,
// 142 -> 107; 8B shape, B = 1: 123 -> 128, 128 -> 124, 145 -> 126, 220 -> 139; B = 4: 157 -> 166, 162 -> 165, 179 -> 169, 256 -> 188. Not
// taken: 1B, B = 8: 92 -> 101, 97 -> 102, 107 -> 105, 145 -> 124; B = 12: 94 -> 109, 98 -> 110, 109 -> 115, 149 -> 142; 8B, B = 8: 156 ->
// 174, 162 -> 173, 180 -> 180, 258 -> 218. Both take the same time at 500 and 1000 keys at 8 and 32 items of the 1B shape, at 700 and 1200
// of the 8B shape: so the line is drawn at 32 items, and at about twice those keys. (At 64 items they meet at 2000 keys and the split loses
// a tenth on short rows.) Rows of more
// than 4096 outputs are outside k_fold_fq_rows, and the general quantiser reads the sixteen parts with one workgroup: 64 query
// heads of 128, 2000 keys, 251 -> 332. (A split by ranges of 256 keys, its partial outputs divided by the denominator, took 2 to
// 9 us less per layer, but then a step's rounding changed with B.)
static int dsp_lpad(int L_max) { return (L_max + DSP_KEYS - 1) / DSP_KEYS * DSP_KEYS; }
size_t attn_decode_split_bytes(int B, int L_max, int Hq, int Hkv, int dh)
{
    if (B <= 0 || Hq != DEC_HPB * Hkv || (dh != 64 && dh != 128) || Hq * dh > 4096 || L_max > DSP_MAX_L || L_max < 1) return 0;
    const int64_t items = (int64_t)B * Hkv;
    static_assert(DECODE_SPLIT_MAX_B >= 32, "");
    if (items > 32 || L_max < 1536 || L_max < 64 * items) return 0;
    return (size_t)B * Hq * ((size_t)dsp_lpad(L_max) * 4 + sizeof(DecSel) + (size_t)DEC_WAVES * dh * 4);
}

// B sequences as launch_attn_decode, in three launches; writes nsplit partial outputs [nsplit][B][Hq * dh] at *part,
// to be summed in that order and divided by (*sel)[B][Hq].den: then the bits are launch_attn_decode's.
bool launch_attn_decode_split(const void *q, const void *k_cache, const void *v_cache, void *ws, const RowAct *ra,
                              const int32_t *cache_len, int B, int L_max, int Hq, int Hkv, int dh, int *flags, hipStream_t st,
                              const float **part_out, const DecSel **sel_out, int *nsplit_out)
{
    if (!cache_len || !attn_decode_split_bytes(B, L_max, Hq, Hkv, dh)) return false;
    const int lpad = dsp_lpad(L_max);
    float *scores = (float *)ws;
    DecSel *sel = (DecSel *)(scores + (size_t)B * Hq * lpad);
    float *part = (float *)(sel + (size_t)B * Hq);
    const float scale = 1.0f / sqrtf((float)dh);
    const dim3 g1(lpad / DSP_KEYS, Hkv, B), g2(Hq, B), g3(DEC_WAVES, Hkv, B);
    if (dh == 64) hipLaunchKernelGGL(k_dec_scores<64>, g1, dim3(256), 0, st, (const bf16_t *)q, (const bf16_t *)k_cache, scores, cache_len, L_max, Hq, Hkv, lpad, scale, flags);
    else hipLaunchKernelGGL(k_dec_scores<128>, g1, dim3(256), 0, st, (const bf16_t *)q, (const bf16_t *)k_cache, scores, cache_len, L_max, Hq, Hkv, lpad, scale, flags);
#define SOL_DEC_SEL(SL, NJU) hipLaunchKernelGGL((k_dec_select<SL, NJU>), g2, dim3(DSEL_WAVES * 64), 0, st, scores, sel, ra, cache_len, L_max, Hq, lpad)
    if (L_max <= 2048) SOL_DEC_SEL(4, 2);
    else if (L_max <= 4096) SOL_DEC_SEL(4, 4);
    else if (L_max <= 8192) SOL_DEC_SEL(8, 8);
    else SOL_DEC_SEL(12, 9);
#undef SOL_DEC_SEL
    const int steps = (L_max + 8192 / dh - 1) / (8192 / dh), rounds = (steps + DSV_STEPS - 1) / DSV_STEPS, cap = (steps + rounds - 1) / rounds;
    const size_t lds = (size_t)cap * 1024 + (size_t)DEC_HPB * steps * (512 / dh) * 4;   // at most 57 KB
    if (dh == 64) hipLaunchKernelGGL(k_dec_values<64>, g3, dim3(256), lds, st, scores, sel, (const bf16_t *)v_cache, part, cache_len, L_max, Hq, Hkv, lpad, cap);
    else hipLaunchKernelGGL(k_dec_values<128>, g3, dim3(256), lds, st, scores, sel, (const bf16_t *)v_cache, part, cache_len, L_max, Hq, Hkv, lpad, cap);
    *part_out = part;
    *sel_out = sel;
    *nsplit_out = DEC_WAVES;
    return true;
}

// order[r] = the sequence with the r-th longest cache (equal lengths in index order); identity beyond 1024
// sequences. One workgroup; the lengths are the same for every layer of a decode step.
__global__ void __launch_bounds__(1024)
k_seq_order(const int32_t *__restrict__ len, int n, int32_t *__restrict__ order)
{
    __shared__ int s_len[1024];
    const int tid = threadIdx.x;
    if (n > 1024) {
        for (int i = tid; i < n; i += 1024) order[i] = i;
        return;
    }
    const int my_len = tid < n ? len[tid] : 0;
    s_len[tid] = my_len;
    __syncthreads();
    if (tid < n) {
        int rank = 0;
        for (int j = 0; j < n; ++j) {
            const int lj = s_len[j];
            rank += (lj > my_len || (lj == my_len && j < tid)) ? 1 : 0;
        }
        order[rank] = tid;
    }
}

void launch_seq_order(const int32_t *cache_len, int B, int32_t *order, hipStream_t st)
{
    if (B > 0) hipLaunchKernelGGL(k_seq_order, dim3(1), dim3(1024), 0, st, cache_len, B, order);
}

// One query per sequence (T = 1), bf16, 4 query heads per KV head, head_dim 64 / 128, L_max <= 9216.
// seq_order: sequences by decreasing cache length (launch_seq_order), or null for launch order.
bool launch_attn_decode(const void *q, const void *k_cache, const void *v_cache, float *o32, const RowAct *ra,
                        const int32_t *cache_len, const int32_t *seq_order, int B, int L_max, int Hq, int Hkv, int dh,
                        int *flags, hipStream_t st)
{
    if (B <= 0) return true;
    if (!cache_len || Hq != DEC_HPB * Hkv || (dh != 64 && dh != 128) || L_max > 9216) return false;
    const size_t red = (size_t)DEC_WAVES * DEC_HPB * dh * 4;
#define SOL_DEC(SL)                                                                                             \
    if ((size_t)DEC_HPB * SL * 64 * DEC_GW * 4 >= red)                                                           \
        return dh == 64 ? launch_attn_decode_t<64, SL>(q, k_cache, v_cache, o32, ra, cache_len, seq_order, B, L_max, Hq, Hkv, flags, st) \
                        : launch_attn_decode_t<128, SL>(q, k_cache, v_cache, o32, ra, cache_len, seq_order, B, L_max, Hq, Hkv, flags, st)
    if (L_max <= 1024) { SOL_DEC(4); }
    if (L_max <= 2048) { SOL_DEC(8); }
    if (L_max <= 4096) { SOL_DEC(16); }
    if (L_max <= 8192) { SOL_DEC(32); }
    SOL_DEC(36);                                   // 9216 columns: an 8192-token cache plus the tokens being decoded
#undef SOL_DEC
    return false;
}

// =================================================================================================
// Decode attention under the page rule (Appendix "Quest masking", page size S > 1), bf16.
//
// Page metadata: for every page of S contiguous keys of a (sequence, KV head) one row of 2 * dh bf16 values,
// [channel-wise maximum | channel-wise minimum] over the keys of the page written so far. The caller owns
// the buffer ([n_seq][Hkv][ceil(L_max / S)][2 * dh]); k_page_meta_build fills it from a cache,
// k_page_meta_update folds in the key a decode step has just written. With it the page bound
//   sum_c max(q_c max_c, q_c min_c) = [max(q, 0) | min(q, 0)] . [max | min]
// is a dot product of length 2 * dh, i.e. the score kernel's MFMA loop run over metadata rows, and a decode
// step reads 2 / S of K for the bounds plus the K and V rows of the pages it keeps, not all of K.
// =================================================================================================
template <int DH>
__global__ void __launch_bounds__(256)
k_page_meta_build(const bf16_t *__restrict__ kc, const int32_t *__restrict__ len, bf16_t *__restrict__ meta, int S,
                  int L_max, int P_max, int Hkv, const int32_t *__restrict__ first, int extra)
{
    constexpr int LPK = DH / 8, PPB = 256 / LPK;               // lanes per page row, pages per workgroup
    const int s = blockIdx.z, kvh = blockIdx.y;
    const int u = blockIdx.x * PPB + threadIdx.x / LPK, cs = threadIdx.x % LPK;
    int n = len[s] + extra;
    n = n < 0 ? 0 : (n > L_max ? L_max : n);
    const int j0 = u * S;
    if (u >= P_max || j0 >= n) return;
    if (first && j0 + S <= first[s]) return;                   // page wholly before the rewritten keys
    const int j1 = j0 + S < n ? j0 + S : n;
    const bf16_t *kb = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH + cs * 8;
    float mx[8], mn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { mx[e] = -INFINITY; mn[e] = INFINITY; }
    for (int j = j0; j < j1; ++j) {
        const u32x4_a v = *reinterpret_cast<const u32x4_a *>(kb + (int64_t)j * DH);
#pragma unroll
        for (int wi = 0; wi < 4; ++wi) {
            const float a = __uint_as_float(v[wi] << 16), b = __uint_as_float(v[wi] & 0xFFFF0000u);
            mx[2 * wi] = fmaxf(mx[2 * wi], a); mn[2 * wi] = fminf(mn[2 * wi], a);
            mx[2 * wi + 1] = fmaxf(mx[2 * wi + 1], b); mn[2 * wi + 1] = fminf(mn[2 * wi + 1], b);
        }
    }
    bf16_t *mrow = meta + (((int64_t)s * Hkv + kvh) * P_max + u) * (2 * DH) + cs * 8;
    u32x4_a omx, omn;                                          // extremes of bf16 values are bf16 values: exact
#pragma unroll
    for (int wi = 0; wi < 4; ++wi) {
        omx[wi] = (__float_as_uint(mx[2 * wi]) >> 16) | (__float_as_uint(mx[2 * wi + 1]) & 0xFFFF0000u);
        omn[wi] = (__float_as_uint(mn[2 * wi]) >> 16) | (__float_as_uint(mn[2 * wi + 1]) & 0xFFFF0000u);
    }
    *reinterpret_cast<u32x4_a *>(mrow) = omx;
    *reinterpret_cast<u32x4_a *>(mrow + DH) = omn;
}

// the key at position pos[s] (just written) joins its page: first key of a page initialises the row
template <int DH>
__global__ void __launch_bounds__(64)
k_page_meta_update(const bf16_t *__restrict__ kc, const int32_t *__restrict__ pos, bf16_t *__restrict__ meta, int S,
                   int L_max, int P_max, int Hkv)
{
    constexpr int LPK = DH / 8;
    const int s = blockIdx.y, kvh = blockIdx.x, cs = threadIdx.x;
    const int p = pos[s];
    if (cs >= LPK || p < 0 || p >= L_max) return;
    const int u = p / S;
    const u32x4_a v = *reinterpret_cast<const u32x4_a *>(kc + (((int64_t)s * Hkv + kvh) * L_max + p) * DH + cs * 8);
    bf16_t *mrow = meta + (((int64_t)s * Hkv + kvh) * P_max + u) * (2 * DH) + cs * 8;
    u32x4_a omx = v, omn = v;
    if (p != u * S) {
        const u32x4_a amx = *reinterpret_cast<const u32x4_a *>(mrow), amn = *reinterpret_cast<const u32x4_a *>(mrow + DH);
#pragma unroll
        for (int wi = 0; wi < 4; ++wi) {
            const float a = __uint_as_float(v[wi] << 16), b = __uint_as_float(v[wi] & 0xFFFF0000u);
            const float xa = fmaxf(a, __uint_as_float(amx[wi] << 16)), xb = fmaxf(b, __uint_as_float(amx[wi] & 0xFFFF0000u));
            const float na = fminf(a, __uint_as_float(amn[wi] << 16)), nb = fminf(b, __uint_as_float(amn[wi] & 0xFFFF0000u));
            omx[wi] = (__float_as_uint(xa) >> 16) | (__float_as_uint(xb) & 0xFFFF0000u);
            omn[wi] = (__float_as_uint(na) >> 16) | (__float_as_uint(nb) & 0xFFFF0000u);
        }
    }
    *reinterpret_cast<u32x4_a *>(mrow) = omx;
    *reinterpret_cast<u32x4_a *>(mrow + DH) = omn;
}

bool launch_page_meta_build(const void *k_cache, const int32_t *len, void *meta, int n_seq, int L_max, int Hkv, int dh,
                            int S, hipStream_t st, const int32_t *first, int extra)
{
    if (n_seq <= 0) return true;
    if (S < 2 || (dh != 64 && dh != 128)) return false;
    const int P_max = (L_max + S - 1) / S;
    const int ppb = 256 / (dh / 8);
    const dim3 grid((unsigned)((P_max + ppb - 1) / ppb), Hkv, n_seq);
    if (dh == 64) hipLaunchKernelGGL(k_page_meta_build<64>, grid, dim3(256), 0, st, (const bf16_t *)k_cache, len, (bf16_t *)meta, S, L_max, P_max, Hkv, first, extra);
    else hipLaunchKernelGGL(k_page_meta_build<128>, grid, dim3(256), 0, st, (const bf16_t *)k_cache, len, (bf16_t *)meta, S, L_max, P_max, Hkv, first, extra);
    return true;
}

bool launch_page_meta_update(const void *k_cache, const int32_t *pos, void *meta, int n_seq, int L_max, int Hkv, int dh,
                             int S, hipStream_t st)
{
    if (n_seq <= 0) return true;
    if (S < 2 || (dh != 64 && dh != 128)) return false;
    const int P_max = (L_max + S - 1) / S;
    if (dh == 64) hipLaunchKernelGGL(k_page_meta_update<64>, dim3(Hkv, n_seq), dim3(64), 0, st, (const bf16_t *)k_cache, pos, (bf16_t *)meta, S, L_max, P_max, Hkv);
    else hipLaunchKernelGGL(k_page_meta_update<128>, dim3(Hkv, n_seq), dim3(64), 0, st, (const bf16_t *)k_cache, pos, (bf16_t *)meta, S, L_max, P_max, Hkv);
    return true;
}

// [max(q, 0) | min(q, 0)] of a pair of packed bf16 values: element e of the doubled query row
__device__ __forceinline__ uint32_t q_split_pair(uint32_t x, bool neg_half)
{
    const bool nlo = (x & 0x8000u) != 0u, nhi = (x & 0x80000000u) != 0u;
    const uint32_t lo = (nlo == neg_half) ? (x & 0xFFFFu) : 0u;
    const uint32_t hi = (nhi == neg_half) ? (x & 0xFFFF0000u) : 0u;
    return lo | hi;
}

// One workgroup of 16 waves per (sequence, KV head), the 4 query heads of the group together:
//   1. page bounds on MFMA from the metadata rows (fp32, to LDS);
//   2. per head, the threshold of the top ceil(b / S) bounds (same joint search as the per-key kernel, over
//      pages), ties to the lower page; the kept pages of the 4 heads as bit flags in LDS;
//   3. scores of the keys of kept pages and of the sink / window keys (K tiles no head needs are skipped),
//      -inf elsewhere;  4. softmax numerators;  5. V rows gathered where any head kept the key.
template <int DH, int SLOTS>
__global__ void __launch_bounds__(DEC_BLOCK)
k_attn_decode_paged(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, const bf16_t *__restrict__ vc,
                    const bf16_t *__restrict__ meta, float *__restrict__ o32, const RowAct *__restrict__ ra,
                    const int32_t *__restrict__ cache_len, const int32_t *__restrict__ seq_order, int L_max, int P_max,
                    int lpad, int Hq, int Hkv, float scale, AttnOpts opt, int *flags)
{
    constexpr int KK = DH / 32, KK2 = 2 * KK, SLICE = SLOTS * 64, PPAD = SLICE * DEC_GW, NJ = SLOTS / 4;
    extern __shared__ __align__(16) float sc[];               // page bounds [HPB][PPAD], then scores [HPB][lpad], then partial O
    __shared__ int s_pk[PPAD];                                 // bit h: head h keeps the page
    __shared__ int s_cnt[2][DEC_WAVES];
    __shared__ uint32_t s_min[DEC_WAVES], s_max[DEC_WAVES];
    __shared__ int s_done[2][DEC_HPB];
    __shared__ int s_gt[DEC_WAVES];
    __shared__ float s_den[DEC_WAVES], s_mx[DEC_WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = blockIdx.x;
    const int s = __builtin_amdgcn_readfirstlane(seq_order ? seq_order[blockIdx.y] : (int)blockIdx.y);
    const int p0 = __builtin_amdgcn_readfirstlane(cache_len[s]);
    if (p0 < 0 || p0 + 1 > L_max) {
        if (tid == 0) atomicOr(flags, FLAG_CACHE_OVERFLOW);
        return;
    }
    const int n = p0 + 1;
    const int S = opt.page;
    const int n_pages = (n + S - 1) / S;
    const int h0 = kvh * DEC_HPB;
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *mbase = meta + ((int64_t)s * Hkv + kvh) * (int64_t)P_max * (2 * DH);
    const int l16 = lane & 15, lg = lane >> 4;
    const RowAct act = ra[s];
    const int b = __builtin_amdgcn_readfirstlane(budget_ceil(act.keep_num, act.keep_den, n));
    int np = (b + S - 1) / S;
    np = np < n_pages ? np : n_pages;
    const bool all_pages = b >= n || np >= n_pages;            // every page (or, b >= n, every key) is kept
    const bool dense = b >= n;
    const int head = w / DEC_GW, wg = w - head * DEC_GW;

    for (int u = tid; u < PPAD; u += DEC_BLOCK) s_pk[u] = 0;

    // the query heads as MFMA B operand (column = head)
    u32x4_a qraw[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        qraw[kk] = u32x4_a{0u, 0u, 0u, 0u};
        if (l16 < DEC_HPB)
            qraw[kk] = *reinterpret_cast<const u32x4_a *>(q + (int64_t)s * (Hq * DH) + (int64_t)(h0 + l16) * DH + kk * 32 + lg * 8);
    }

    if (!all_pages) {
        // ---- 1. page bounds ---------------------------------------------------------------------
        bf16x8_a qq[KK2];                                      // [max(q, 0) | min(q, 0)], 2 * DH long
#pragma unroll
        for (int kk = 0; kk < KK2; ++kk) {
            u32x4_a v;
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) v[wi] = q_split_pair(qraw[kk % KK][wi], kk >= KK);
            qq[kk] = __builtin_bit_cast(bf16x8_a, v);
        }
        const int n_pt = (n_pages + 15) >> 4;
        constexpr int U = 2;
        for (int pt0 = w; pt0 < n_pt; pt0 += DEC_WAVES * U) {
            bf16x8_a mf[U][KK2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int pg = (pt0 + u * DEC_WAVES) * 16 + l16;
                if (pg >= n_pages) pg = n_pages - 1;
                const bf16_t *mp = mbase + (int64_t)pg * (2 * DH) + lg * 8;
#pragma unroll
                for (int kk = 0; kk < KK2; ++kk)
                    mf[u][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(mp + kk * 32));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int pt = pt0 + u * DEC_WAVES;
                if (pt < n_pt) {
                    floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kk = 0; kk < KK2; ++kk)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mf[u][kk], qq[kk], acc, 0, 0, 0);
                    if (l16 < DEC_HPB) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) sc[l16 * PPAD + pt * 16 + lg * 4 + r] = acc[r];
                    }
                }
            }
        }
        __syncthreads();

        // ---- 2. the np best pages of each head ------------------------------------------------------
        const int base = wg * SLICE;
        int n_loc = n_pages - base;
        n_loc = n_loc < 0 ? 0 : (n_loc > SLICE ? SLICE : n_loc);
        float *row = sc + head * PPAD + base;
        uint32_t key[SLOTS];
        uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (256 * j < n_loc) {
                const f32x4_a v = *reinterpret_cast<const f32x4_a *>(row + 256 * j + 4 * lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool valid = 256 * j + 4 * lane + e < n_loc;
                    const uint32_t kv = valid ? score_key(v[e]) : 0u;
                    key[4 * j + e] = kv;
                    kmax = kv > kmax ? kv : kmax;
                    kmin = (valid && kv < kmin) ? kv : kmin;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) key[4 * j + e] = 0u;
            }
        }
        kmax = wave_max_u32(kmax);
        kmin = wave_min_u32(kmin);
        if (lane == 0) { s_max[w] = kmax; s_min[w] = kmin; }
        __syncthreads();
        uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
        for (int i = 0; i < DEC_GW; ++i) {
            const uint32_t a = s_min[head * DEC_GW + i], c = s_max[head * DEC_GW + i];
            lo = a < lo ? a : lo;
            hi = c > hi ? c : hi;
        }
        lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
        hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
        uint32_t thr = 1u;
        bool done = false, exact = true;
        // invariant: count(key >= lo) >= np, count(key >= hi + 1) < np; regula falsi with the Illinois correction
        // on g(x) = count(key >= x) - np + 1/2, the midpoint of the key range after 12 rounds or a bad guess
        float flo = score_unkey(lo), fhi = score_unkey(hi), glo = (float)(n_pages - np) + 0.5f, ghi = 0.5f - (float)np;
        int side = 0;
        for (int it = 0; it < 48; ++it) {
            const int par = it & 1;
            uint32_t mid = 0u;
            if (!done) {
                const float fp = __builtin_fmaf(fhi - flo, glo * __builtin_amdgcn_rcpf(glo - ghi), flo);
                mid = (uint32_t)__builtin_amdgcn_readfirstlane((int)score_key(fp));
                if (it >= 12 || !(mid > lo && mid <= hi)) mid = lo + ((hi - lo + 1u) >> 1);
                const int c = lo < hi ? wave_count_ge<SLOTS>(key, n_loc, mid) : 0;
                if (lane == 0) s_cnt[par][w] = c;
            }
            if (wg == 0 && lane == 0) s_done[par][head] = done || lo >= hi;
            __syncthreads();
            if (!done) {
                if (lo >= hi) { thr = lo; exact = false; done = true; }
                else {
                    int cnt = 0;
#pragma unroll
                    for (int i = 0; i < DEC_GW; ++i) cnt += s_cnt[par][head * DEC_GW + i];
                    cnt = __builtin_amdgcn_readfirstlane(cnt);
                    const float g = (float)(cnt - np) + 0.5f;
                    if (cnt == np) { thr = mid; done = true; }
                    else if (cnt > np) {
                        lo = mid; flo = score_unkey(mid); glo = g;
                        if (side > 0) ghi *= 0.5f;
                        side = 1;
                    } else {
                        hi = mid - 1u; fhi = score_unkey(hi); ghi = g;
                        if (side < 0) glo *= 0.5f;
                        side = -1;
                    }
                }
            }
            const bool all_done =
                __builtin_amdgcn_readfirstlane(s_done[par][0] & s_done[par][1] & s_done[par][2] & s_done[par][3]) != 0;
            if (all_done) break;
        }
        // ties at the threshold go to the lower pages: the first wave of the head walks the row
        {
            const bool need = !exact;
            int gt = 0;
            if (need) {
#pragma unroll
                for (int i = 0; i < SLOTS; ++i) gt += __popcll(__ballot(key[i] > thr));
            }
            if (lane == 0) s_gt[w] = gt;
            __syncthreads();
            if (need && wg == 0) {
                int quota = np;
#pragma unroll
                for (int i = 0; i < DEC_GW; ++i) quota -= s_gt[head * DEC_GW + i];
                quota = __builtin_amdgcn_readfirstlane(quota);
                float *hrow = sc + head * PPAD;
                int taken = 0;
                for (int c0 = 0; c0 < n_pages; c0 += 64) {
                    const int col = c0 + lane;
                    const bool tie = col < n_pages && score_key(hrow[col]) == thr;
                    const unsigned long long bal = __ballot(tie);
                    const int rank = taken + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
                    if (tie && rank >= quota) hrow[col] = -INFINITY;
                    taken += __popcll(bal);
                }
            }
            __syncthreads();
        }
        // kept pages of this head -> flags
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (256 * j < n_loc) {
                const f32x4_a v = *reinterpret_cast<const f32x4_a *>(row + 256 * j + 4 * lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int u = 256 * j + 4 * lane + e;
                    if (u < n_loc && score_key(v[e]) >= thr) atomicOr(&s_pk[base + u], 1 << head);
                }
            }
        }
    }
    __syncthreads();                                           // flags complete; the page bounds in sc are dead

    // ---- 3. scores of the kept keys ---------------------------------------------------------------
    const int sink_end = opt.n_sink < n ? opt.n_sink : n;
    int win_begin = n - opt.n_window;
    win_begin = win_begin < sink_end ? sink_end : win_begin;
    {
        bf16x8_a qf[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qf[kk] = __builtin_bit_cast(bf16x8_a, qraw[kk]);
        const int n_kt = (n + 15) >> 4;
        constexpr int U = 4;
        for (int kt0 = w; kt0 < n_kt; kt0 += DEC_WAVES * U) {
            bf16x8_a kf[U][KK];
            bool need[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kt = kt0 + u * DEC_WAVES;
                const int j0 = kt * 16, j1 = j0 + 15 < n - 1 ? j0 + 15 : n - 1;
                bool nd = false;
                if (kt < n_kt) {
                    nd = all_pages || j0 < sink_end || j1 >= win_begin;
                    if (!nd)
                        for (int pg = j0 / S; pg <= j1 / S; ++pg) nd |= s_pk[pg] != 0;
                }
                need[u] = __builtin_amdgcn_readfirstlane((int)nd) != 0;
                if (need[u]) {
                    int key = j0 + l16;
                    if (key >= n) key = n - 1;
                    const bf16_t *kp = kbase + (int64_t)key * DH + lg * 8;
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
                        kf[u][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(kp + kk * 32));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kt = kt0 + u * DEC_WAVES;
                if (kt < n_kt) {
                    floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
                    if (need[u]) {
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk)
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][kk], qf[kk], acc, 0, 0, 0);
                    }
                    if (l16 < DEC_HPB) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int j = kt * 16 + lg * 4 + r;
                            bool kept = false;
                            if (need[u] && j < n)
                                kept = dense || j < sink_end || j >= win_begin || all_pages || ((s_pk[j / S] >> l16) & 1) != 0;
                            sc[l16 * lpad + j] = kept ? acc[r] * scale : -INFINITY;
                        }
                    }
                }
            }
        }
    }
    __syncthreads();

    // ---- 4. softmax numerators over the kept keys ---------------------------------------------------
    {
        float *row = sc + head * lpad;
        float mx = -INFINITY;
        for (int j0 = wg * 256; j0 < n; j0 += DEC_GW * 256) {
            const f32x4_a v = *reinterpret_cast<const f32x4_a *>(row + j0 + 4 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = (j0 + 4 * lane + e < n) ? fmaxf(mx, v[e]) : mx;
        }
        mx = wave_reduce_dpp<float>(mx, -INFINITY, [](float x, float y) { return fmaxf(x, y); });
        if (lane == 0) s_mx[w] = mx;
        __syncthreads();
        mx = s_mx[head * DEC_GW];
#pragma unroll
        for (int i = 1; i < DEC_GW; ++i) mx = fmaxf(mx, s_mx[head * DEC_GW + i]);
        float den = 0.f;
        for (int j0 = wg * 256; j0 < n; j0 += DEC_GW * 256) {
            const f32x4_a v = *reinterpret_cast<const f32x4_a *>(row + j0 + 4 * lane);
            f32x4_a p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[e] = (j0 + 4 * lane + e < n) ? __expf(v[e] - mx) : 0.f;     // exp(-inf) = 0 for dropped keys
                den += p[e];
            }
            *reinterpret_cast<f32x4_a *>(row + j0 + 4 * lane) = p;
        }
        den = wave_sum_dpp(den);
        if (lane == 0) s_den[w] = den;
        __syncthreads();
    }
    decode_pv_tail<DH, DEC_WAVES>(sc, lpad, n, vbase, [&](int hh) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < DEC_GW; ++i) d += s_den[hh * DEC_GW + i];
        return d;
    }, o32 + (int64_t)s * (Hq * DH) + (int64_t)h0 * DH);
}

template <int DH, int SLOTS>
static bool launch_attn_decode_paged_t(const void *q, const void *kc, const void *vc, const void *meta, float *o32,
                                       const RowAct *ra, const int32_t *cache_len, const int32_t *seq_order, int B,
                                       int L_max, int P_max, int lpad, int Hq, int Hkv, AttnOpts opt, int *flags,
                                       hipStream_t st)
{
    auto kern = k_attn_decode_paged<DH, SLOTS>;
    size_t lds = (size_t)DEC_HPB * lpad * 4;
    const size_t pg = (size_t)DEC_HPB * SLOTS * 64 * DEC_GW * 4, red = (size_t)DEC_WAVES * DEC_HPB * DH * 4;
    lds = lds < pg ? pg : lds;
    lds = lds < red ? red : lds;
    if (lds + (size_t)SLOTS * 64 * DEC_GW * 4 + 1024 > 160 * 1024) return false;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                150 * 1024) != hipSuccess)
            return false;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3(Hkv, B), dim3(DEC_BLOCK), lds, st, (const bf16_t *)q, (const bf16_t *)kc,
                       (const bf16_t *)vc, (const bf16_t *)meta, o32, ra, cache_len, seq_order, L_max, P_max, lpad, Hq, Hkv,
                       1.0f / sqrtf((float)DH), opt, flags);
    return true;
}

// One query per sequence under the page rule, with caller-kept page metadata (page_meta_build / _update).
// bf16, 4 query heads per KV head, head_dim 64 / 128, at most 3072 pages and about 9000 keys.
bool launch_attn_decode_paged(const void *q, const void *k_cache, const void *v_cache, const void *meta, float *o32,
                              const RowAct *ra, const int32_t *cache_len, const int32_t *seq_order, int B, int L_max, int Hq,
                              int Hkv, int dh, AttnOpts opt, int *flags, hipStream_t st)
{
    if (B <= 0) return true;
    if (!cache_len || !meta || opt.page < 2 || Hq != DEC_HPB * Hkv || (dh != 64 && dh != 128)) return false;
    const int P_max = (L_max + opt.page - 1) / opt.page;
    const int lpad = (L_max + 1023) & ~1023;                   // rows are walked in steps of 4 waves x 256 columns
    if ((size_t)DEC_HPB * lpad * 4 > 148 * 1024) return false;
#define SOL_DECP(SL)                                                                                            \
    if (P_max <= SL * 64 * DEC_GW)                                                                              \
        return dh == 64 ? launch_attn_decode_paged_t<64, SL>(q, k_cache, v_cache, meta, o32, ra, cache_len, seq_order, B, \
                                                             L_max, P_max, lpad, Hq, Hkv, opt, flags, st)       \
                        : launch_attn_decode_paged_t<128, SL>(q, k_cache, v_cache, meta, o32, ra, cache_len, seq_order, B, \
                                                              L_max, P_max, lpad, Hq, Hkv, opt, flags, st)
    SOL_DECP(4);
    SOL_DECP(8);
    SOL_DECP(12);
#undef SOL_DECP
    return false;
}

// K cache [s][kvh][key][dh] -> kfr [s][kvh][tile of 16 keys][dh / 32][64 lanes][8]: lane (l16, lg) of piece kk holds
// channels 32*kk + 8*lg .. + 7 of key 16*tile + l16, the A operand of mfma_f32_16x16x32_bf16 for that tile; keys from
// pos0[s] + Tn on are zero. attn_lpad64(L_max) keys per (s, kvh).
template <int DH>
__global__ void __launch_bounds__(256)
k_frag_k(const bf16_t *__restrict__ kc, bf16_t *__restrict__ kfr, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hkv,
         int lpad)
{
    constexpr int KP = DH / 8, KK = DH / 32;                // 16-byte pieces per key
    const int kb = blockIdx.x * 64, kvh = blockIdx.y, s = blockIdx.z;
    const int p0 = pos0 ? pos0[s] : 0;
    int len = p0 + Tn;
    if (p0 < 0 || len > L_max) len = 0;
    const bf16_t *src = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    bf16_t *dst = kfr + ((int64_t)s * Hkv + kvh) * (int64_t)lpad * DH;
    for (int idx = threadIdx.x; idx < 64 * KP; idx += 256) {
        const int key = kb + idx / KP, p = idx % KP;
        if (key >= lpad) break;
        u32x4_a v = {0u, 0u, 0u, 0u};
        if (key < len) v = *reinterpret_cast<const u32x4_a *>(src + (int64_t)key * DH + p * 8);
        const int tile = key >> 4, l16 = key & 15, kk = p >> 2, lg = p & 3;
        *reinterpret_cast<u32x4_a *>(dst + ((int64_t)(tile * KK + kk) * 64 + lg * 16 + l16) * 8) = v;
    }
}

// rows whose key count lies in (n_lo, n_hi] (all rows by default); SLOTS * 64 >= min(n_hi, L_max) is the caller's business
template <int SLOTS, int DH, int R, int U, int NS, int SC, bool PRE, bool KF>
static bool launch_attn_select_t(const void *q, const void *kc, SelRow *sel, const RowAct *ra, const int32_t *pos0,
                                 int n_seq, int Tn, int L_max, int Hq, int Hkv, hipStream_t st, PrefixView pv = PrefixView(),
                                 int n_lo = 0, int n_hi = 1 << 30)
{
    using Sh = SelShape<SLOTS, DH, R, U, NS, SC>;
    constexpr int BQ = Sh::BQ;
    auto kern = k_attn_select<SLOTS, DH, R, U, NS, SC, PRE, KF>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Sh::LDS) != hipSuccess)
            return false;
        attr_done = true;
    }
    // workgroups per (sequence, head): enough to fill the chip about eight times over, at most one per block
    int t_range = (n_hi < L_max ? n_hi : L_max) - n_lo;     // no sequence has more rows than that in the range
    if (t_range > Tn) t_range = Tn;
    if (t_range <= 0) return true;
    const int n_qb = (t_range + BQ - 1) / BQ;
    int nb = (int)((4096 + (int64_t)Hq * n_seq - 1) / ((int64_t)Hq * n_seq));
    if (nb > n_qb) nb = n_qb;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(kern, dim3(nb, Hq, n_seq), dim3(512), Sh::LDS, st, (const bf16_t *)q, (const bf16_t *)kc, sel, ra,
                       pos0, Tn, L_max, Hq, Hkv, 1.0f / sqrtf((float)DH), nb, pv, n_lo, n_hi);
    return true;
}

// How the softmax V kernels deal a sequence's query rows to workgroups: tiles of 16 rows per workgroup and block, workgroups
// per (sequence, KV head). A block of two tiles reads K and V once for 32 rows, and a workgroup that takes a late and an early
// block lasts as long as the others: the better one as soon as such workgroups take 3/5 of the chip's slots (all of them where
// no keys lie before the rows and the head size is 64: an early block then costs little). Fewer leave CUs without work; so
// blocks of one tile, one per workgroup while all of these are resident at once, else a late and an early one, unless that is no
// larger a grid than two tiles make (17 .. 32 rows: two sweeps of the keys instead of one, and nothing for it). Slots: resident
// workgroups of one-tile blocks. Timed for 3430 layers of 1 .. 128 sequences, 17 .. 1000 rows, 0 .. 3000 keys before them, 1 .. 8
// heads per group, both rules and dense: 9 % less than with two tiles always (geometric mean of the calls), 10 slower by
// 1 to 3 %. With the line at all slots throughout, 196 were slower, by up to 9 %. A layer under the page rule, 64 x 32 rows behind 3000
// keys, 1B shape, us: two tiles 622, pairs of one 667, one per workgroup (more than the slots) 611.
// 1B shape, us of the kernel, pairs of two tiles / pairs of one / one: 333 rows 21 / 12 / 10; 2 x 700 rows 32 / 24 / 22; 8 x 250
// rows 20 / 14 / 16; page rule, 14 x 437 rows 63 / 53 / 55; 16 x 2048 rows 560 / 640 / 660; refresh of 8 x 64 rows 129 / 83 / 47; 8B
// shape: 333 rows 21 / 17 / 14, page rule, 3 x 1777 rows 260 / 283 / 307.
struct PvSplit { int tiles, grid; };
static PvSplit pv_split(int T, int L_max, int64_t groups, int dh, int G)
{
    if (T <= 16) return PvSplit{1, 1};
    const int cus = device_cus() > 0 ? device_cus() : 256;
    const int64_t slots = (int64_t)cus * (dh == 64 ? 4 : 2) / (G == 8 ? 2 : 1);      // (registers, LDS)
    const int pairs = ((T + 31) / 32 + 1) / 2, blocks = (T + 15) / 16, halves = (blocks + 1) / 2;
    if (blocks * groups < slots) return PvSplit{1, blocks};
    const int64_t line = L_max <= T && dh == 64 ? slots : slots * 3 / 5;
    return pairs * groups >= line || halves <= pairs ? PvSplit{2, pairs} : PvSplit{1, halves};
}

template <int DH, int G, bool PRE = false>
static bool launch_attn_pv_t(const void *q, const void *kc, const void *vc, const SelRow *sel, float *o32,
                             const int32_t *pos0, int n_seq, int Tn, int L_max, int Hq, int Hkv, hipStream_t st,
                             PrefixView pv = PrefixView())
{
    const size_t lds = 4 * (size_t)64 * DH * 2;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(k_attn_pv<DH, G, PRE, 1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void *>(k_attn_pv<DH, G, PRE, 2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return false;
        attr_done = true;
    }
    const PvSplit sp = pv_split(Tn, L_max, (int64_t)n_seq * Hkv, DH, G);
    if (sp.tiles == 1)                                       // one tile of 16 query rows per workgroup
        hipLaunchKernelGGL((k_attn_pv<DH, G, PRE, 1>), dim3(sp.grid, Hkv, n_seq), dim3(G * 64), lds, st, (const bf16_t *)q,
                           (const bf16_t *)kc, (const bf16_t *)vc, sel, o32, pos0, Tn, L_max, Hq, Hkv,
                           1.0f / sqrtf((float)DH), pv);
    else
        hipLaunchKernelGGL((k_attn_pv<DH, G, PRE, 2>), dim3(sp.grid, Hkv, n_seq), dim3(G * 64), lds, st,
                           (const bf16_t *)q, (const bf16_t *)kc, (const bf16_t *)vc, sel, o32, pos0, Tn, L_max, Hq, Hkv,
                           1.0f / sqrtf((float)DH), pv);
    return true;
}

// =================================================================================================
// Batched bf16 attention under the page rule (page size S a power of two, 4 <= S <= 64), sink / window keys.
//   k_page_prefix_meta : pm[j] = channel-wise [max | min] over the keys of j's page up to j (2 * dh values per key).
//                        The last key of a full page carries the page's extremes; row p is the partial page of the
//                        query at position p.
//   k_attn_select_pages: per (16 query rows, head): page bounds [max(q,0) | min(q,0)] . pm on MFMA (full pages as one
//                        tile product, the partial page of every query as the diagonal of one more tile), then per
//                        row the top ceil(b / S) bounds, ties to the lower page -> a bit mask of kept pages.
//   k_attn_pv_pages    : k_attn_pv with the mask (and the forced keys) as keep rule and a running maximum, since the
//                        largest kept score is not known beforehand.
// =================================================================================================
template <int DH>
__global__ void __launch_bounds__(256)
k_page_prefix_meta(const bf16_t *__restrict__ kc, const int32_t *__restrict__ pos0, bf16_t *__restrict__ pm, int Tn, int S,
                   int L_max, int Hkv)
{
    constexpr int LPK = DH / 8, PPB = 256 / LPK;
    const int s = blockIdx.z, kvh = blockIdx.y;
    const int u = blockIdx.x * PPB + threadIdx.x / LPK, cs = threadIdx.x % LPK;
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) return;
    const int n = p0 + Tn, j0 = u * S;
    if (j0 >= n) return;
    const int j1 = j0 + S < n ? j0 + S : n;
    const bf16_t *kb = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH + cs * 8;
    bf16_t *pb = pm + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * (2 * DH) + cs * 8;
    float mx[8], mn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { mx[e] = -INFINITY; mn[e] = INFINITY; }
    for (int j = j0; j < j1; ++j) {
        const u32x4_a v = *reinterpret_cast<const u32x4_a *>(kb + (int64_t)j * DH);
        u32x4_a omx, omn;
#pragma unroll
        for (int wi = 0; wi < 4; ++wi) {
            const float a = __uint_as_float(v[wi] << 16), b = __uint_as_float(v[wi] & 0xFFFF0000u);
            mx[2 * wi] = fmaxf(mx[2 * wi], a); mn[2 * wi] = fminf(mn[2 * wi], a);
            mx[2 * wi + 1] = fmaxf(mx[2 * wi + 1], b); mn[2 * wi + 1] = fminf(mn[2 * wi + 1], b);
            omx[wi] = (__float_as_uint(mx[2 * wi]) >> 16) | (__float_as_uint(mx[2 * wi + 1]) & 0xFFFF0000u);
            omn[wi] = (__float_as_uint(mn[2 * wi]) >> 16) | (__float_as_uint(mn[2 * wi + 1]) & 0xFFFF0000u);
        }
        *reinterpret_cast<u32x4_a *>(pb + (int64_t)j * (2 * DH)) = omx;
        *reinterpret_cast<u32x4_a *>(pb + (int64_t)j * (2 * DH) + DH) = omn;
    }
}

// PRE (shared prefix, as in k_attn_select): pm holds the metadata rows of the sequence's own keys (positions pv.P..,
// [n_seq][Hkv][pv.crows][2 * DH]), pv.pm those of the prefix keys of input s / pv.K ([inputs][Hkv][pv.P][2 * DH]);
// pv.P is a multiple of 16 pages, so a tile of 16 pages lies on one side.
template <int DH, int W, bool PRE>
__global__ void __launch_bounds__(256)
k_attn_select_pages(const bf16_t *__restrict__ q, const bf16_t *__restrict__ pm, unsigned long long *__restrict__ selp,
                    const RowAct *__restrict__ ra, const int32_t *__restrict__ pos0, int Tn, int L_max, int Hq, int Hkv,
                    int log2S, PrefixView pv)
{
    constexpr int KK = DH / 32, KK2 = 2 * KK, PS = 64 * W + 4, BQ = 16;
    __shared__ float sb[BQ][PS];                             // bounds of the full pages, [query][page]
    __shared__ float sd[BQ];                                 // bound of each query's own (partial) page
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q0 = blockIdx.x * BQ, h = blockIdx.y, s = blockIdx.z;
    const int kvh = h / (Hq / Hkv);
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) return;
    const int S = 1 << log2S;
    const int q_last = (q0 + BQ - 1 < Tn ? q0 + BQ - 1 : Tn - 1);
    const int u_max = (p0 + q_last) >> log2S;                // last page any query of the block touches
    const bf16_t *pmb = pm + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * (2 * DH);
    const bf16_t *pmb_pre = nullptr;
    if constexpr (PRE) {                                     // own rows addressed by absolute key: base minus P rows
        pmb = pm + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * (2 * DH) - (int64_t)pv.P * (2 * DH);
        pmb_pre = pv.pm + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * (2 * DH);
    }

    // queries as MFMA B operand: column l16 = query q0 + l16, doubled row [max(q, 0) | min(q, 0)]
    bf16x8_a qq[KK2];
    {
        const int qi = q0 + l16 < Tn ? q0 + l16 : Tn - 1;
        const bf16_t *qp = q + ((int64_t)s * Tn + qi) * (int64_t)(Hq * DH) + (int64_t)h * DH + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const u32x4_a raw = *reinterpret_cast<const u32x4_a *>(qp + kk * 32);
            u32x4_a a, b;
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) { a[wi] = q_split_pair(raw[wi], false); b[wi] = q_split_pair(raw[wi], true); }
            qq[kk] = __builtin_bit_cast(bf16x8_a, a);
            qq[KK + kk] = __builtin_bit_cast(bf16x8_a, b);
        }
    }
    // full pages: tile pt holds pages 16 pt .. 16 pt + 15; page u is read from the row of its last key
    const int n_pt = (u_max + 16) >> 4;
    for (int pt = w; pt < n_pt; pt += 4) {
        int j = (((pt * 16 + l16) + 1) << log2S) - 1;
        j = j < L_max ? j : L_max - 1;                       // pages past the live keys are masked below
        const bf16_t *mp = ((PRE && ((pt * 16) << log2S) < pv.P) ? pmb_pre : pmb) + (int64_t)j * (2 * DH) + lg * 8;
        floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK2; ++kk) {
            const bf16x8_a mf = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(mp + kk * 32));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mf, qq[kk], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) sb[l16][pt * 16 + lg * 4 + r] = acc[r];
    }
    if (w == 3) {                                            // the queries' own pages: row m = the key of query m; diagonal
        int j = p0 + q0 + l16;
        j = j < p0 + Tn ? j : p0 + Tn - 1;
        const bf16_t *mp = pmb + (int64_t)j * (2 * DH) + lg * 8;
        floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK2; ++kk) {
            const bf16x8_a mf = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(mp + kk * 32));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mf, qq[kk], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (lg * 4 + r == l16) sd[l16] = acc[r];
    }
    __syncthreads();

    // ---- per query row: the top ceil(b / S) pages ------------------------------------------------
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (int i = 4 * w; i < 4 * w + 4; ++i) {
        const int qi = q0 + i;
        if (qi >= Tn) break;                                 // uniform
        const int p = p0 + qi, n = p + 1, u_p = p >> log2S, npg = u_p + 1;
        const RowAct act = ra[(int64_t)s * Tn + qi];
        const int b = __builtin_amdgcn_readfirstlane(budget_ceil(act.keep_num, act.keep_den, n));
        int np = (b + S - 1) >> log2S;
        np = np < npg ? np : npg;
        unsigned long long mask[W];
        if (b >= n || np >= npg) {
#pragma unroll
            for (int ww = 0; ww < W; ++ww) mask[ww] = ~0ull;
        } else {
            uint32_t key[W];
            uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
#pragma unroll
            for (int ww = 0; ww < W; ++ww) {
                const int u = 64 * ww + lane;
                const float v = u < u_p ? sb[i][u] : sd[i];
                key[ww] = u <= u_p ? score_key(v) : 0u;
                if (u <= u_p) { kmax = key[ww] > kmax ? key[ww] : kmax; kmin = key[ww] < kmin ? key[ww] : kmin; }
            }
            uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_min_u32(kmin));
            uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(kmax));
            auto count_ge = [&](uint32_t t) -> int {
                int c = 0;
#pragma unroll
                for (int ww = 0; ww < W; ++ww) c += __popcll(__ballot(key[ww] >= t));
                return c;
            };
            bool exact = false;                              // invariant: count(key >= lo) >= np, count(key >= hi + 1) < np
            while (lo < hi) {
                const uint32_t mid = lo + ((hi - lo + 1u) >> 1);
                const int c = count_ge(mid);
                if (c == np) { lo = mid; exact = true; break; }
                if (c > np) lo = mid; else hi = mid - 1u;
            }
            const uint32_t thr = lo;
            int quota = 64 * W;                              // tied pages kept, lowest pages first
            if (!exact) {
                const int n_ge = count_ge(thr);
                if (n_ge > np) quota = np - (thr == 0xFFFFFFFFu ? 0 : count_ge(thr + 1u));
            }
#pragma unroll
            for (int ww = 0; ww < W; ++ww) {
                const bool tie = key[ww] == thr && 64 * ww + lane <= u_p;
                const unsigned long long bal = __ballot(tie);
                const bool keep = key[ww] > thr || (tie && __popcll(bal & lt_mask) < quota);
                mask[ww] = __ballot(keep);
                const int total = __popcll(bal);
                quota = quota > total ? quota - total : 0;
            }
        }
        if (lane == 0) {
            unsigned long long *o = selp + (((int64_t)s * Tn + qi) * Hq + h) * W;
#pragma unroll
            for (int ww = 0; ww < W; ++ww) o[ww] = mask[ww];
        }
    }
}

// maximum over the four lanes l16, l16 + 16, l16 + 32, l16 + 48 with the gfx950 lane-swap instructions (vector ALU
// only: v_permlane32_swap exchanges the upper half of one operand with the lower half of the other,
// v_permlane16_swap the odd rows of 16 lanes of one with the even rows of the other)
typedef uint32_t u32x2_a __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float max_over_lane_groups(float v)
{
    const u32x2_a a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const u32x2_a b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// PRE: two-segment addressing as in k_attn_pv. NQT: query tiles of 16 rows per workgroup and block (see pv_split).
template <int DH, int G, int W, bool PRE, int NQT>
// (4+ heads per group. Head size 64: a floor of 3 / 4 waves per SIMD caps the registers at 168 / 128; left alone the compiler
// takes 218 and 138 and the exp / pack chains of the softmax have nothing to overlap with: 0.94 -> 0.74 ms at C2 under the paper's
// configuration; head size 128: 2 waves per SIMD, 256 registers instead of 410, 4.51 -> 2.44 ms at the 8B shape with 4096-token
// sequences. 1 or 2 heads per group: a wave holds 4 or 2 times as much of a staged chunk, five workgroups of 1 or 2 waves fill the
// LDS anyway, and the floor's cap only spilled: head size 64, 32 heads, 2 x 2048 tokens, 1 per group 623 -> 194 us (498 with the
// transposed copy of V), 2 per group 138 -> 110)
__global__ void __launch_bounds__(G * 64) __attribute__((amdgpu_waves_per_eu(G == 1 ? 1 : (G == 2 ? (DH == 64 ? 2 : 1) : (DH == 64 ? (NQT == 1 ? 4 : 3) : 2)), 8)))
k_attn_pv_pages(const bf16_t *__restrict__ q, const bf16_t *__restrict__ kc, const bf16_t *__restrict__ vc,
                const unsigned long long *__restrict__ selp, float *__restrict__ o32, const int32_t *__restrict__ pos0, int Tn,
                int L_max, int Hq, int Hkv, float scale, int log2S, int n_sink, int n_window, PrefixView pv)
{
    constexpr int NT = G * 64, KK = DH / 32, DT = DH / 16, KC = 64, QT = 16 * NQT;
    constexpr int KP = DH / 8;
    constexpr int PIECES = KC * KP / NT;                     // of K and of V, per thread and chunk
    constexpr int K_BYTES = KC * DH * 2, STAGE = 2 * K_BYTES;
    static_assert(KC * KP % NT == 0, "chunk / thread mismatch");
    extern __shared__ __align__(16) unsigned char pvl[];

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = blockIdx.y, s = blockIdx.z, h = kvh * G + w;
    const int p0 = pos0 ? pos0[s] : 0;
    if (p0 < 0 || p0 + Tn > L_max) return;
    const int n_qb = (Tn + QT - 1) / QT;
    const bool alone = (int)gridDim.x >= n_qb;
    for (int pass = 0; pass < 2; ++pass) {                  // query blocks n_qb - 1 - x and x, as in k_attn_pv
    const int qb = pass == 0 ? n_qb - 1 - (int)blockIdx.x : (int)blockIdx.x;
    if (pass == 1 && (alone || qb >= n_qb - 1 - (int)blockIdx.x)) break;
    const int q0 = qb * QT;
    const int rows = (Tn - q0 < QT) ? (Tn - q0) : QT;
    const int n_max = p0 + q0 + rows;
    const int n_chunks = (n_max + KC - 1) / KC;
    const bf16_t *kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)L_max * DH;
    const bf16_t *kpre = nullptr, *vpre = nullptr;
    if constexpr (PRE) {                                    // own segment addressed by absolute key: bases minus P keys
        kbase = kc + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * DH - (int64_t)pv.P * DH;
        vbase = vc + ((int64_t)s * Hkv + kvh) * (int64_t)pv.crows * DH - (int64_t)pv.P * DH;
        kpre = pv.k + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * DH;
        vpre = pv.v + ((int64_t)(s / pv.K) * Hkv + kvh) * (int64_t)pv.P * DH;
    }
    const float sl2 = scale * 1.44269504088896341f;          // scores in the log2 domain

    bf16x8_a qf[NQT][KK];
    unsigned long long mask[NQT][W];
    float m_run[NQT], den[NQT];
    int pos[NQT], sink_end[NQT], win_begin[NQT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        m_run[qt] = -INFINITY;
        den[qt] = 0.f;
        const int qi = q0 + 16 * qt + l16;
        const bool live = qi < Tn;
        const int qr = live ? qi : Tn - 1;
        const bf16_t *qp = q + ((int64_t)s * Tn + qr) * (int64_t)(Hq * DH) + (int64_t)h * DH + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            qf[qt][kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(qp + kk * 32));
#pragma unroll
        for (int ww = 0; ww < W; ++ww)                      // no masks at all: every page of every row is kept
            mask[qt][ww] = selp ? selp[(((int64_t)s * Tn + qr) * Hq + h) * W + ww] : ~0ull;
        pos[qt] = live ? p0 + qi : -1;                      // dead rows of a ragged block keep nothing
        const int n = p0 + qi + 1;
        sink_end[qt] = n_sink < n ? n_sink : n;
        win_begin[qt] = n - n_window > sink_end[qt] ? n - n_window : sink_end[qt];
    }

    floatx4_a oacc[NQT][DT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] = floatx4_a{0.f, 0.f, 0.f, 0.f};

    u32x4_a kreg0[PIECES], vreg0[PIECES];
#define SOL_PV_GLOAD(KR, VR, CH_)                                                                                  \
    {                                                                                                      \
        const int key0_ = (CH_) * KC;                                                                      \
        const bool pre_ = PRE && key0_ < pv.P;              /* chunk-uniform: P is a multiple of the chunk */ \
        const bf16_t *kb_ = pre_ ? kpre : kbase, *vb_ = pre_ ? vpre : vbase;                               \
        _Pragma("unroll") for (int i = 0; i < PIECES; ++i) {                                             \
            const int pc = i * NT + tid, row = pc / KP, piece = pc - row * KP;                             \
            int key = key0_ + row;                                                                         \
            if (key >= n_max) key = n_max - 1;                                                             \
            KR[i] = *reinterpret_cast<const u32x4_a *>(kb_ + (int64_t)key * DH + piece * 8);               \
            VR[i] = *reinterpret_cast<const u32x4_a *>(vb_ + (int64_t)key * DH + piece * 8);               \
        }                                                                                                  \
    }
#define SOL_PV_LSTORE(KR, VR, STG_)                                                                                \
    {                                                                                                      \
        unsigned char *kb_ = pvl + (STG_) * STAGE, *vb_ = kb_ + K_BYTES;                                   \
        _Pragma("unroll") for (int i = 0; i < PIECES; ++i) {                                             \
            const int pc = i * NT + tid, row = pc / KP, piece = pc - row * KP;                             \
            *reinterpret_cast<u32x4_a *>(kb_ + row * (DH * 2) + ((piece ^ pv_swz_k<DH>(row)) << 4)) = KR[i]; \
            *reinterpret_cast<u32x4_a *>(vb_ + row * (DH * 2) + ((piece ^ pv_swz_v<DH>(row)) << 4)) = VR[i]; \
        }                                                                                                  \
    }
    SOL_PV_GLOAD(kreg0, vreg0, 0);
    SOL_PV_LSTORE(kreg0, vreg0, 0);
    if (1 < n_chunks) SOL_PV_GLOAD(kreg0, vreg0, 1);
    __syncthreads();
    for (int ch = 0; ch < n_chunks; ++ch) {
        const int stg = ch & 1;
        // one register set: what was fetched an iteration ago goes to LDS, then the set is requested again
        if (ch + 1 < n_chunks) SOL_PV_LSTORE(kreg0, vreg0, stg ^ 1);
        if (ch + 2 < n_chunks) SOL_PV_GLOAD(kreg0, vreg0, ch + 2);
        const unsigned char *kb = pvl + stg * STAGE, *vb = kb + K_BYTES;
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            const int kb32 = ch * KC + cc * 32;
            if (kb32 < n_max) {
                floatx4_a st[NQT][2];
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    const int krow = cc * 32 + 8 * (l16 >> 2) + 4 * kt + (l16 & 3);
                    bf16x8_a kf[KK];
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
                        kf[kk] = __builtin_bit_cast(bf16x8_a, *reinterpret_cast<const u32x4_a *>(
                            kb + krow * (DH * 2) + (((kk * 4 + lg) ^ pv_swz_k<DH>(krow)) << 4)));
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt) {
                        floatx4_a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk)
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kk], qf[qt][kk], acc, 0, 0, 0);
                        st[qt][kt] = acc;
                    }
                }
                // keep rule, running maximum (log2 domain), numerators as hi + lo bf16 pairs
                bf16x8_a phi[NQT], plo[NQT];                    // numerators as hi + lo bf16 pairs (single bf16 numerators cost
                float fac[NQT];                               // ~1e-2 of a short row: measured, not taken)
                bool grew = false;
                const int kfirst = kb32 + 8 * lg;
                // sub-chunks wholly before every query of the block and free of sink / window keys need the page
                // bit only (one test per 4 keys, folded into the scaling as an additive 0 / -inf)
                const bool plain = kb32 + 31 <= p0 + q0 && kb32 >= n_sink && kb32 + 31 < p0 + q0 + 1 - n_window;
#pragma unroll
                for (int qt = 0; qt < NQT; ++qt) {
                    float x[8];
                    float m_loc = -INFINITY;
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        const int j0 = kfirst + 4 * kt;      // 4 consecutive keys of one page (S >= 4)
                        const int u = j0 >> log2S;
                        unsigned long long word = mask[qt][0];
#pragma unroll
                        for (int ww = 1; ww < W; ++ww) word = (u >> 6) == ww ? mask[qt][ww] : word;
                        const bool bit = ((word >> (u & 63)) & 1ull) != 0ull;
                        if (plain) {
                            const float off = bit ? 0.f : -INFINITY;
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                x[4 * kt + r] = __builtin_fmaf(st[qt][kt][r], sl2, off);
                                m_loc = fmaxf(m_loc, x[4 * kt + r]);
                            }
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int j = j0 + r;
                                const bool keep = (bit || j < sink_end[qt] || j >= win_begin[qt]) && j <= pos[qt];
                                x[4 * kt + r] = keep ? st[qt][kt][r] * sl2 : -INFINITY;
                                m_loc = fmaxf(m_loc, x[4 * kt + r]);
                            }
                        }
                    }
                    m_loc = max_over_lane_groups(m_loc);
                    const float m_new = fmaxf(m_run[qt], m_loc);
                    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
                    grew |= m_new > m_run[qt];
                    fac[qt] = __builtin_amdgcn_exp2f(m_run[qt] - m_safe);     // exp2(-inf) = 0 before the first kept key
                    m_run[qt] = m_new;
                    float p[8], psum = 0.f;
#pragma unroll
                    for (int i = 0; i < 8; ++i) { p[i] = __builtin_amdgcn_exp2f(x[i] - m_safe); psum += p[i]; }
                    den[qt] = den[qt] * fac[qt] + psum;
                    u32x4_a hi, lo;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        hi[i] = pack_bf16x2(p[2 * i], p[2 * i + 1]);
                        lo[i] = pack_bf16x2(p[2 * i] - __uint_as_float(hi[i] << 16), p[2 * i + 1] - __uint_as_float(hi[i] & 0xFFFF0000u));
                    }
                    phi[qt] = __builtin_bit_cast(bf16x8_a, hi);
                    plo[qt] = __builtin_bit_cast(bf16x8_a, lo);
                }
                if (__ballot(grew) != 0ull) {                // some row's maximum moved: rescale what is accumulated
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float fo = __shfl(fac[qt], 4 * lg + r);    // accumulator register r is query 4 lg + r
#pragma unroll
                            for (int dt = 0; dt < DT; ++dt) oacc[qt][dt][r] *= fo;
                        }
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const bf16x8_a vf = pv_read_v<DH>(vb, cc * 32 + 8 * lg, dt, l16);
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt) {
                        oacc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo[qt], vf, oacc[qt][dt], 0, 0, 0);
                        oacc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi[qt], vf, oacc[qt][dt], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();
    }
#undef SOL_PV_GLOAD
#undef SOL_PV_LSTORE
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        float dsum = den[qt];
        dsum += __shfl_xor(dsum, 16);
        dsum += __shfl_xor(dsum, 32);
        const float inv = dsum > 0.f ? 1.0f / dsum : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float iv = __shfl(inv, 4 * lg + r);
            const int qi = q0 + 16 * qt + 4 * lg + r;
            if (qi < Tn) {
                float *op = o32 + ((int64_t)s * Tn + qi) * (int64_t)(Hq * DH) + (int64_t)h * DH + l16;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) op[dt * 16] = oacc[qt][dt][r] * iv;
            }
        }
    }
    }   // pass
}

int attn_tile_lpad(int L_max) { return attn_lpad64(L_max); }
size_t attn_tile_sel_bytes(int64_t rows, int Hq) { return (size_t)rows * Hq * sizeof(SelRow); }

bool launch_attn_frag_k(const void *k_cache, void *kfr, const int32_t *pos0, int n_seq, int T, int L_max, int Hkv, int dh,
                        hipStream_t st)
{
    if ((dh != 64 && dh != 128) || n_seq <= 0 || T <= 0 || L_max <= 0) return false;
    const int lpad = attn_lpad64(L_max);
    const dim3 tg(lpad / 64, Hkv, n_seq);
    if (dh == 64)
        hipLaunchKernelGGL((k_frag_k<64>), tg, dim3(256), 0, st, (const bf16_t *)k_cache, (bf16_t *)kfr, pos0, T, L_max, Hkv, lpad);
    else
        hipLaunchKernelGGL((k_frag_k<128>), tg, dim3(256), 0, st, (const bf16_t *)k_cache, (bf16_t *)kfr, pos0, T, L_max, Hkv, lpad);
    return true;
}

bool launch_attn_tile(const void *q, const void *k_cache, const void *v_cache, void *kfr, void *sel_ws, float *o32,
                      const RowAct *ra, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh,
                      hipStream_t st)
{
    if ((int64_t)n_seq * T <= 0) return true;
    const int G = Hkv > 0 ? Hq / Hkv : 0;
    if ((dh != 64 && dh != 128) || L_max > 4096 || T < 16 || G * Hkv != Hq || (G != 1 && G != 2 && G != 4 && G != 8))
        return false;
    SelRow *sel = (SelRow *)sel_ws;
    // K in MFMA operand order for the threshold kernel, which reads all causal keys once per block of 16 or 32 query rows
    // (up to 256 keys the copy does not pay)
    const bool frag = L_max > 256;
    if (frag && !launch_attn_frag_k(k_cache, kfr, pos0, n_seq, T, L_max, Hkv, dh, st)) return false;
    // A launch per class of row lengths: the rows of a long sequence that see at most 1024 (2048) keys go to the variant for
    // that length, whose rows take fewer registers, not to the one the sequence's last row needs.
    bool ok;
#define SOL_SEL2(SL, DH_, R, U, NS, SC, KF, LO, HI)                                                                  \
    launch_attn_select_t<SL, DH_, R, U, NS, SC, false, KF>(q, KF ? kfr : k_cache, sel, ra, pos0, n_seq, T, L_max, Hq, Hkv, st, PrefixView(), LO, HI)
#define SOL_SEL(SL, R64, U64, NS64, SC64, R128, U128, NS128, SC128, KF, LO, HI)                                      \
    ok = dh == 64 ? SOL_SEL2(SL, 64, R64, U64, NS64, SC64, KF, LO, HI) : SOL_SEL2(SL, 128, R128, U128, NS128, SC128, KF, LO, HI)
    // Rows per wave, key tiles and register sets in flight, keys per part. Four rows per wave where they fit 128 registers (up to
    // 1024 keys at head size 64: 0.38 against 0.49 ms with two); parts so that two workgroups share a CU's LDS; in the longest
    // class the registers hold one workgroup per CU, so a part takes most of the LDS.
    constexpr int ALL = 1 << 30;
    if (L_max <= 256) { SOL_SEL(4, 4, 2, 1, 256, 4, 2, 1, 256, false, 0, ALL); }
    else {
        SOL_SEL(16, 4, 2, 1, 512, 2, 2, 1, 1024, true, 0, 1024);
        if (ok && L_max > 1024) { SOL_SEL(32, 2, 2, 1, 1024, 2, 2, 1, 1024, true, 1024, 2048); }
        if (ok && L_max > 2048) { SOL_SEL(64, 2, 4, 1, 2048, 2, 4, 1, 2048, true, 2048, ALL); }
    }
#undef SOL_SEL2
#undef SOL_SEL
    if (!ok) return false;
#define SOL_PV(G_)                                                                                                   \
    return dh == 64 ? launch_attn_pv_t<64, G_>(q, k_cache, v_cache, sel, o32, pos0, n_seq, T, L_max, Hq, Hkv, st)  \
                    : launch_attn_pv_t<128, G_>(q, k_cache, v_cache, sel, o32, pos0, n_seq, T, L_max, Hq, Hkv, st)
    if (G == 1) { SOL_PV(1); }
    if (G == 2) { SOL_PV(2); }
    if (G == 4) { SOL_PV(4); }
    SOL_PV(8);
#undef SOL_PV
}

// launch_attn_tile for sequences that share prefix caches (PrefixView): k_cache / v_cache hold positions pv.P.. only
// ([n_seq][Hkv][pv.crows][dh]);
// every sequence's T rows sit at positions pv.P .. pv.P + T - 1. Returns false (nothing launched) outside the shapes
// of launch_attn_tile, if pv.P is not a multiple of 64 or the caches lie 2^31 elements or more apart.
// shape and address limits of launch_attn_tile_prefix (only differences of the pointers are looked at)
bool attn_tile_prefix_ok(const void *k_cache, int n_seq, int T, int Hq, int Hkv, int dh, const PrefixView &pv)
{
    const int G = Hkv > 0 ? Hq / Hkv : 0, L_max = pv.P + T;
    if ((dh != 64 && dh != 128) || L_max > 4096 || T < 16 || G * Hkv != Hq || (G != 1 && G != 2 && G != 4 && G != 8))
        return false;
    if (pv.P <= 0 || pv.P % 64 || pv.K < 1 || T > pv.crows) return false;
    // the threshold kernel reaches a sequence's own keys as a 32-bit element offset from its input's prefix cache:
    // (own cache of (s, kvh), minus P rows) - (prefix cache of (s / K, kvh)) must lie in [0, 2^31 - a row span) for
    // every (s, kvh); the difference is linear in input, schedule and head, so the corners decide
    if (n_seq % pv.K) return false;
    // (the same from the prefix's copy in operand order, when the view has one: same shape, same strides)
    for (const bf16_t *pre : {pv.k, pv.kf}) {
        if (!pre) continue;
        const int64_t base = (const bf16_t *)k_cache - pre - (int64_t)pv.P * dh;
        for (int c = 0; c < 8; ++c) {
            const int64_t b = (c & 1) ? n_seq / pv.K - 1 : 0, k = (c & 2) ? pv.K - 1 : 0, kv = (c & 4) ? Hkv - 1 : 0;
            const int64_t diff = base + ((b * pv.K + k) * Hkv + kv) * (int64_t)pv.crows * dh - (b * Hkv + kv) * (int64_t)pv.P * dh;
            if (diff < 0 || diff >= (1ll << 31) - (int64_t)(L_max + 1) * dh) return false;
        }
    }
    return true;
}

bool launch_attn_tile_prefix(const void *q, const void *k_cache, const void *v_cache, void *sel_ws, float *o32,
                             const RowAct *ra, const int32_t *pos0, int n_seq, int T, int Hq, int Hkv, int dh, PrefixView pv,
                             hipStream_t st)
{
    if ((int64_t)n_seq * T <= 0) return true;
    if (pv.kf && !attn_tile_prefix_ok(k_cache, n_seq, T, Hq, Hkv, dh, pv)) pv.kf = nullptr;   // copy out of reach: do without
    if (!pv.k || !pv.v || !attn_tile_prefix_ok(k_cache, n_seq, T, Hq, Hkv, dh, pv)) return false;
    const int G = Hq / Hkv, L_max = pv.P + T;
    SelRow *sel = (SelRow *)sel_ws;
    bool ok;
    // rows longer than 1024 keys read the prefix keys from their copy in operand order, if the view has one
#define SOL_SEL2(SL, DH_, U, NS, SC, KF) launch_attn_select_t<SL, DH_, 2, U, NS, SC, true, KF>(q, k_cache, sel, ra, pos0, n_seq, T, L_max, Hq, Hkv, st, pv)
#define SOL_SEL(SL, U64, NS64, U128, NS128, SC, KF) ok = dh == 64 ? SOL_SEL2(SL, 64, U64, NS64, SC, KF) : SOL_SEL2(SL, 128, U128, NS128, SC, KF)
    if (L_max <= 256) { SOL_SEL(4, 2, 1, 2, 1, 256, false); }
    else if (L_max <= 1024) { SOL_SEL(16, 2, 1, 2, 1, 1024, false); }
    else if (L_max <= 1280) {
        if (pv.kf) { SOL_SEL(20, 2, 1, 2, 1, 768, true); } else { SOL_SEL(20, 2, 1, 2, 1, 768, false); }
    } else if (L_max <= 2048) {
        if (pv.kf) { SOL_SEL(32, 2, 1, 2, 1, 1024, true); } else { SOL_SEL(32, 2, 1, 2, 1, 1024, false); }
    } else {
        if (pv.kf) { SOL_SEL(64, 4, 2, 2, 2, 2048, true); } else { SOL_SEL(64, 4, 2, 2, 2, 2048, false); }
    }
#undef SOL_SEL2
#undef SOL_SEL
    if (!ok) return false;
#define SOL_PV(G_)                                                                                                   \
    return dh == 64 ? launch_attn_pv_t<64, G_, true>(q, k_cache, v_cache, sel, o32, pos0, n_seq, T, L_max, Hq, Hkv, st, pv)  \
                    : launch_attn_pv_t<128, G_, true>(q, k_cache, v_cache, sel, o32, pos0, n_seq, T, L_max, Hq, Hkv, st, pv)
    if (G == 1) { SOL_PV(1); }
    if (G == 2) { SOL_PV(2); }
    if (G == 4) { SOL_PV(4); }
    SOL_PV(8);
#undef SOL_PV
}

// PRE: kc / vc / pm belong to the sequences' own keys (pv.crows rows each, positions pv.P..), L_max = pv.P + T.
template <int DH, int W, bool PRE = false>
static bool launch_attn_tile_pages_t(const void *q, const void *kc, const void *vc, void *pm, void *selp, float *o32,
                                     const RowAct *ra, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv,
                                     int log2S, AttnOpts opt, hipStream_t st, PrefixView pv = PrefixView())
{
    const int S = 1 << log2S, G = Hq / Hkv;
    constexpr int ppb = 256 / (DH / 8);
    if (PRE)   // metadata of the own keys, by local row (pages do not straddle pv.P)
        hipLaunchKernelGGL(k_page_prefix_meta<DH>, dim3(((pv.crows + S - 1) / S + ppb - 1) / ppb, Hkv, n_seq), dim3(256), 0,
                           st, (const bf16_t *)kc, (const int32_t *)nullptr, (bf16_t *)pm, T, S, pv.crows, Hkv);
    else
        hipLaunchKernelGGL(k_page_prefix_meta<DH>, dim3(((L_max + S - 1) / S + ppb - 1) / ppb, Hkv, n_seq), dim3(256), 0, st,
                           (const bf16_t *)kc, pos0, (bf16_t *)pm, T, S, L_max, Hkv);
    hipLaunchKernelGGL((k_attn_select_pages<DH, W, PRE>), dim3((T + 15) / 16, Hq, n_seq), dim3(256), 0, st, (const bf16_t *)q,
                       (const bf16_t *)pm, (unsigned long long *)selp, ra, pos0, T, L_max, Hq, Hkv, log2S, pv);
    const size_t lds = 4 * (size_t)64 * DH * 2;
    const float scale = 1.0f / sqrtf((float)DH);
#define SOL_PVP(G_, NQT_)                                                                                            \
    {                                                                                                                \
        auto kern = k_attn_pv_pages<DH, G_, W, PRE, NQT_>;                                                           \
        static bool attr_done = false;                                                                               \
        if (!attr_done) {                                                                                            \
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                    (int)lds) != hipSuccess)                                                         \
                return false;                                                                                        \
            attr_done = true;                                                                                        \
        }                                                                                                            \
        hipLaunchKernelGGL(kern, dim3(sp.grid, Hkv, n_seq), dim3(G_ * 64), lds, st, (const bf16_t *)q, \
                           (const bf16_t *)kc, (const bf16_t *)vc, (const unsigned long long *)selp, o32, pos0, T, L_max, Hq, \
                           Hkv, scale, log2S, opt.n_sink, opt.n_window, pv);                                  \
        return true;                                                                                                 \
    }
    const PvSplit sp = pv_split(T, L_max, (int64_t)n_seq * Hkv, DH, G);
    if (sp.tiles == 1) {                                     // one tile of 16 query rows per workgroup
        if (G == 1) SOL_PVP(1, 1)
        if (G == 2) SOL_PVP(2, 1)
        if (G == 4) SOL_PVP(4, 1)
        SOL_PVP(8, 1)
    }
    if (G == 1) SOL_PVP(1, 2)
    if (G == 2) SOL_PVP(2, 2)
    if (G == 4) SOL_PVP(4, 2)
    SOL_PVP(8, 2)
#undef SOL_PVP
}

// Dense causal attention for rows that keep every key (prefill, cache refresh): the flash-style kernel alone, with
// its running maximum, no threshold pass. Shapes of launch_attn_tile.
bool launch_attn_tile_dense(const void *q, const void *k_cache, const void *v_cache, float *o32,
                            const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv, int dh, hipStream_t st)
{
    if ((int64_t)n_seq * T <= 0) return true;
    const int G = Hkv > 0 ? Hq / Hkv : 0;
    if ((dh != 64 && dh != 128) || L_max > 4096 || T < 16 || G * Hkv != Hq || (G != 1 && G != 2 && G != 4 && G != 8))
        return false;
    const size_t lds = 4 * (size_t)64 * dh * 2;
    const float scale = 1.0f / sqrtf((float)dh);
#define SOL_PVD2(DH_, G_, NQT_)                                                                                      \
    {                                                                                                                \
        auto kern = k_attn_pv_pages<DH_, G_, 1, false, NQT_>;                                                        \
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,    \
                                (int)lds) != hipSuccess)                                                             \
            return false;                                                                                            \
        hipLaunchKernelGGL(kern, dim3(sp.grid, Hkv, n_seq), dim3(G_ * 64), lds, st, (const bf16_t *)q, \
                           (const bf16_t *)k_cache, (const bf16_t *)v_cache, (const unsigned long long *)nullptr, o32, pos0, T, \
                           L_max, Hq, Hkv, scale, 6, 0, 0, PrefixView());                                     \
        return true;                                                                                                 \
    }
    const PvSplit sp = pv_split(T, L_max, (int64_t)n_seq * Hkv, dh, G);
#define SOL_PVD(DH_, G_) { if (sp.tiles == 1) SOL_PVD2(DH_, G_, 1) SOL_PVD2(DH_, G_, 2) }
    if (dh == 64) {
        if (G == 1) SOL_PVD(64, 1)
        if (G == 2) SOL_PVD(64, 2)
        if (G == 4) SOL_PVD(64, 4)
        SOL_PVD(64, 8)
    }
    if (G == 1) SOL_PVD(128, 1)
    if (G == 2) SOL_PVD(128, 2)
    if (G == 4) SOL_PVD(128, 4)
    SOL_PVD(128, 8)
#undef SOL_PVD
#undef SOL_PVD2
}

size_t attn_tile_pages_meta_bytes(int64_t n_seq, int Hkv, int L_max, int dh) { return (size_t)n_seq * Hkv * L_max * 2 * dh * 2; }
size_t attn_tile_pages_sel_bytes(int64_t rows, int Hq, int L_max, int S) { return (size_t)rows * Hq * (((L_max + S - 1) / S + 63) / 64) * 8; }

// Batched bf16 attention under the page rule: page size a power of two in [4, 64], at most 256 pages, the limits of
// launch_attn_tile otherwise. pm: attn_tile_pages_meta_bytes of scratch, selp: attn_tile_pages_sel_bytes.
bool launch_attn_tile_pages(const void *q, const void *k_cache, const void *v_cache, void *pm, void *selp,
                            float *o32, const RowAct *ra, const int32_t *pos0, int n_seq, int T, int L_max, int Hq, int Hkv,
                            int dh, AttnOpts opt, hipStream_t st)
{
    if ((int64_t)n_seq * T <= 0) return true;
    const int G = Hkv > 0 ? Hq / Hkv : 0, S = opt.page;
    if ((dh != 64 && dh != 128) || L_max > 4096 || T < 16 || G * Hkv != Hq || (G != 1 && G != 2 && G != 4 && G != 8))
        return false;
    if (S < 4 || S > 64 || (S & (S - 1)) || !pm) return false;
    int log2S = 0;
    while ((1 << log2S) < S) ++log2S;
    const int n_words = ((L_max + S - 1) / S + 63) / 64;
    if (n_words > 4) return false;
#define SOL_TP(W_)                                                                                                   \
    return dh == 64 ? launch_attn_tile_pages_t<64, W_>(q, k_cache, v_cache, pm, selp, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, log2S, opt, st) \
                    : launch_attn_tile_pages_t<128, W_>(q, k_cache, v_cache, pm, selp, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, log2S, opt, st)
    if (n_words == 1) { SOL_TP(1); }
    if (n_words == 2) { SOL_TP(2); }
    SOL_TP(4);
#undef SOL_TP
}

// Prefix side of the shared-prefix variant: the metadata rows of the prefix keys, once per input and layer.
bool launch_page_prefix_meta(const void *k_cache, void *pm, int n_seq, int P, int Hkv, int dh, int S, hipStream_t st)
{
    if ((int64_t)n_seq * P <= 0) return true;
    if ((dh != 64 && dh != 128) || S < 4 || S > 64 || (S & (S - 1)) || !pm) return false;
    const int ppb = 256 / (dh / 8);
    const dim3 grid(((P + S - 1) / S + ppb - 1) / ppb, Hkv, n_seq);
    if (dh == 64)
        hipLaunchKernelGGL(k_page_prefix_meta<64>, grid, dim3(256), 0, st, (const bf16_t *)k_cache, (const int32_t *)nullptr,
                           (bf16_t *)pm, P, S, P, Hkv);
    else
        hipLaunchKernelGGL(k_page_prefix_meta<128>, grid, dim3(256), 0, st, (const bf16_t *)k_cache, (const int32_t *)nullptr,
                           (bf16_t *)pm, P, S, P, Hkv);
    return true;
}

// shapes launch_attn_tile_pages_prefix takes
bool attn_tile_pages_prefix_ok(int n_seq, int T, int Hq, int Hkv, int dh, int S, const PrefixView &pv)
{
    const int G = Hkv > 0 ? Hq / Hkv : 0, L_max = pv.P + T;
    if ((dh != 64 && dh != 128) || L_max > 4096 || T < 16 || G * Hkv != Hq || (G != 1 && G != 2 && G != 4 && G != 8))
        return false;
    if (S < 4 || S > 64 || (S & (S - 1)) || ((L_max + S - 1) / S + 63) / 64 > 4) return false;
    // chunks of 64 keys and tiles of 16 pages must lie on one side of the prefix boundary
    return pv.P > 0 && pv.P % 64 == 0 && pv.P % (16 * S) == 0 && pv.K >= 1 && n_seq % pv.K == 0 && T <= pv.crows;
}

// launch_attn_tile_pages for sequences that share prefix caches (PrefixView: pv.k, pv.v and pv.pm of the input's
// prefix, written by the prefix pass and launch_page_prefix_meta); k_cache / v_cache / pm hold the sequences'
// own pv.crows positions from pv.P on.
bool launch_attn_tile_pages_prefix(const void *q, const void *k_cache, const void *v_cache, void *pm, void *selp,
                                   float *o32, const RowAct *ra, const int32_t *pos0, int n_seq, int T, int Hq, int Hkv,
                                   int dh, AttnOpts opt, PrefixView pv, hipStream_t st)
{
    if ((int64_t)n_seq * T <= 0) return true;
    const int S = opt.page;
    if (!pv.k || !pv.v || !pv.pm || !pm || !attn_tile_pages_prefix_ok(n_seq, T, Hq, Hkv, dh, S, pv)) return false;
    const int L_max = pv.P + T;
    int log2S = 0;
    while ((1 << log2S) < S) ++log2S;
    const int n_words = ((L_max + S - 1) / S + 63) / 64;
#define SOL_TPP(W_)                                                                                                  \
    return dh == 64 ? launch_attn_tile_pages_t<64, W_, true>(q, k_cache, v_cache, pm, selp, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, log2S, opt, st, pv) \
                    : launch_attn_tile_pages_t<128, W_, true>(q, k_cache, v_cache, pm, selp, o32, ra, pos0, n_seq, T, L_max, Hq, Hkv, log2S, opt, st, pv)
    if (n_words == 1) { SOL_TPP(1); }
    if (n_words == 2) { SOL_TPP(2); }
    SOL_TPP(4);
#undef SOL_TPP
}

}  // namespace sol
