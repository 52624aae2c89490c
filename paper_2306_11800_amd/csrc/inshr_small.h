// The search for small tensors (at most SMALL_MAX values): one workgroup sorts the tensor's keys in
// LDS and reads everything the search is after from the sorted array -- thresholds, boundaries, the
// numbers of pruned / protected values, the bins' populations and sums, centres, errors, choice.
//
// The sweeps of the general path (two histograms, threshold select, gather, group sort) are about
// twenty launches with tables of 32768 bins per tensor behind them, whatever the tensor's size: a
// step of a 4096-value tensor took 0.52 ms (0.14 so), and in a checkpoint with hundreds of norm weights
// and biases the per-tensor kernels ran over all of them in several rounds of workgroups.  Sorting 4096
// keys takes 15 us.  What it leaves behind for later calls (thresholds, class counts, boundary keys, centres,
// a key -> bin table of eight bins per key prefix) has the form of the general path.
//
// Bound by latency: about 70 barriers and LDS round trips of one workgroup, and walks of at most 129 values
// per lane and bin (sum_range).  15 pairs, 90 configurations, one tensor / 300 tensors at once, us: 4096
// Gaussian values 84 / 95, 16384 100 / 199; 16384 values of one 69 / 132 and 90 % of zero 138 / 269
// (with every bin walked value by value 6600 / 12400 and 4300 / 7400).
#pragma once
#include "inshr_launch.h"

namespace inshr {

__device__ __forceinline__ u32 lower_bound_key(const u32 *keys, u32 n, u32 key) // keys below
{
    u32 lo = 0u, hi = n;
    while (lo < hi) {
        const u32 mid = (lo + hi) >> 1;
        if (keys[mid] < key)
            lo = mid + 1u;
        else
            hi = mid;
    }
    return lo;
}
__device__ __forceinline__ u32 upper_bound_key(const u32 *keys, u32 n, u32 key) // keys at or below
{
    u32 lo = 0u, hi = n;
    while (lo < hi) {
        const u32 mid = (lo + hi) >> 1;
        if (keys[mid] <= key)
            lo = mid + 1u;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ double value_of_key(u32 k) { return (double)__uint_as_float(bits_of_key(k)); }

// Sum of the values of sorted positions [a, b), which lie in one 8-bit bin (or in a bin of fewer than 256
// values); the walk starts at a lane's own offset, so that the lanes of a wave, whose ranges are equally
// long, do not read the same LDS bank step after step.  A bin holds at most n_kept / 256 + 1 values, 65
// here, unless one value is repeated: all boundaries that fall among equal keys lie at the first of
// them, so that one bin starts with the whole run (of a constant or mostly zero tensor, nearly
// everything).  The run is taken at once: count times value, which is exact (14 + 24 bits).
__device__ __forceinline__ double sum_range(const u32 *keys, u32 a, u32 b)
{
    if (a >= b) return 0.0;
    double s = 0.0;
    if (b - a > 2u * SMALL_MAX / 256u) {
        const u32 first = keys[a], run = upper_bound_key(keys + a, b - a, first);
        s = (double)run * value_of_key(first);
        a += run;
        if (a >= b) return s;
    }
    const u32 len = b - a;
    u32 i = a + (threadIdx.x & 63u) % len;
    for (u32 j = 0; j < len; j++) {
        s += value_of_key(keys[i]);
        i = i + 1u < b ? i + 1u : a;
    }
    return s;
}

constexpr u32 LBS = NBT + 1; // per-pair stride of the boundary positions

// What a workgroup of NT threads needs for at most NT * ROWS keys.
template <int NT, int ROWS> struct SmallShared {
    static constexpr int NW = NT / 64;
    double S8[MAX_PAIRS * 256];              // sums of the 8-bit bins
    u32 keys[NT * ROWS];
    u32 wcount[NW * 256];                    // digit counters of the sort
    u16 LB[MAX_PAIRS * LBS];                 // keys below each boundary
    u32 s_or, s_and, wsum[4];
    u32 s_nneg, s_npos0;                     // negative keys; keys at or below zero
    u32 s_thr[MAX_THR], s_cnt[MAX_THR][4];   // magnitude; below (neg, pos), above (neg, pos)
    u32 s_A[MAX_PAIRS], s_Ap[MAX_PAIRS], s_gl[MAX_PAIRS], s_gr[MAX_PAIRS], s_Mn[MAX_PAIRS], s_M[MAX_PAIRS];
    double s_red[NW][MAX_FRAC + 1], s_sq[MAX_FRAC + 1]; // sums of squares: all, protected per fraction
    __attribute__((aligned(4))) u16 s_cfg[MAX_PAIRS][K_SLOTS]; // first grid entry of (pair, log2 K | 9 + i: 3, 6, 12 bins)
    double s_acc[MAX_PAIRS][K_SLOTS];
    double s_sse[MAX_CFG];
    u64 s_cost[MAX_CFG];
};

// ORDERED: as in the group sort (k_bucket).
template <int NT, int ROWS, bool ORDERED>
__device__ __forceinline__ void search_small(SmallShared<NT, ROWS> &sh, int t, const TDesc *__restrict__ td,
                                             const GridDesc *__restrict__ gd, const Bufs &B)
{
    constexpr u32 NW = NT / 64;
    double *const S8 = sh.S8;
    u32 *const keys = sh.keys, *const wcount = sh.wcount, *const wsum = sh.wsum, *const s_thr = sh.s_thr;
    u16 *const LB = sh.LB;
    u32 &s_or = sh.s_or, &s_and = sh.s_and, &s_nneg = sh.s_nneg, &s_npos0 = sh.s_npos0;
    auto &s_cnt = sh.s_cnt;
    u32 *const s_A = sh.s_A, *const s_Ap = sh.s_Ap, *const s_gl = sh.s_gl, *const s_gr = sh.s_gr, *const s_Mn = sh.s_Mn, *const s_M = sh.s_M;
    auto &s_red = sh.s_red;
    double *const s_sq = sh.s_sq, *const s_sse = sh.s_sse;
    u64 *const s_cost = sh.s_cost;
    auto &s_cfg = sh.s_cfg;
    auto &s_acc = sh.s_acc;

    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TDesc d = td[t];
    const u32 n = (u32)d.n;
    TState *st = B.ts + t;
    const u32 n_pairs = gd->n_pairs, n_p = gd->n_p, n_o = gd->n_o, n_thr = n_p + n_o, n_cfg = gd->n_cfg;
    if (tid == 0u) {
        s_or = 0u;
        s_and = 0xFFFFFFFFu;
    }
    for (u32 i = tid; i < (u32)MAX_PAIRS * (u32)K_SLOTS; i += NT) (&s_cfg[0][0])[i] = 0xFFFFu;
    // eight bins per key prefix (for kernels that want a key -> bin table)
    u32 *tab = B.table2 + (size_t)t * COARSE;
    for (u32 i = tid; i < (u32)COARSE; i += NT) tab[i] = (8u * i) << 5 | 3u;
    __syncthreads();

    // ---- sort (least significant digit first, equal digits over the bits that differ) ------------
    const u32 rows = (n + NT - 1u) / NT, chunk = rows * 64u;
    u32 kreg[ROWS], rreg[ROWS];
    {
        const GLOBAL_AS float *src = gptr(d.data);
        float x[ROWS];
        u32 vo = 0u, va = 0xFFFFFFFFu;
        double q = 0.0;
#pragma unroll
        for (u32 r = 0; r < (u32)ROWS; r++) {
            const u32 i = wave * chunk + r * 64u + lane;
            x[r] = (r < rows && i < n) ? src[i] : 0.0f;
        }
#pragma unroll
        for (u32 r = 0; r < (u32)ROWS; r++) {
            const u32 i = wave * chunk + r * 64u + lane;
            kreg[r] = key_of_float(x[r]);
            q = fma((double)x[r], (double)x[r], q);
            if (r < rows && i < n) {
                vo |= kreg[r];
                va &= kreg[r];
            }
        }
        vo = wave_or(vo);
        va = wave_and(va);
        q = wave_sum_f64(q);
        if (lane == 0u) {
            atomicOr(&s_or, vo);
            atomicAnd(&s_and, va);
            s_red[wave][0] = q;
        }
        u32 *wc0 = wcount + wave * 256u;
        if (ORDERED && ((u32)t & 15u) == 0u) { // cross-check of the ordered ranking, as in the group sort
            for (u32 i = lane; i < 256u; i += 64u) wc0[i] = 0u;
            const bool valid = wave * chunk + lane < n;
            const u32 digit = valid ? (kreg[0] & 255u) : 0u;
            u32 got = 0u;
            if (valid) got = atomicAdd(&wc0[digit], 1u);
            u64 peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const bool bit = (digit >> b) & 1u;
                const u64 m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            if (valid && got != (u32)__popcll(peers & ((1ull << lane) - 1ull)))
                atomicOr(&st->internal_err, 1024u);
        }
    }
    __syncthreads();
    const u32 dbits = n > 1u ? s_or ^ s_and : 0u;
    const u32 b_lo = dbits ? (u32)__ffs((int)dbits) - 1u : 0u;
    const u32 n_bits = dbits ? 32u - (u32)__clz((int)dbits) - b_lo : 0u;
    const u32 n_pass = (n_bits + 7u) >> 3;
    const u32 dwidth = n_pass ? (n_bits + n_pass - 1u) / n_pass : 0u;
    const u32 dmask = (1u << dwidth) - 1u;
    u32 *wcnt = wcount + wave * 256u;
    if (n_pass == 0u) {
#pragma unroll
        for (u32 r = 0; r < (u32)ROWS; r++) {
            const u32 i = wave * chunk + r * 64u + lane;
            if (r < rows && i < n) keys[i] = kreg[r];
        }
        __syncthreads();
    }
    for (u32 pass = 0; pass < n_pass; pass++) {
        const u32 shift = b_lo + pass * dwidth;
        for (u32 i = lane; i < 256u; i += 64u) wcnt[i] = 0u; // (a wave's own counters: its operations stay in order)
#pragma unroll
        for (u32 r = 0; r < (u32)ROWS; r++) {
            rreg[r] = 0u;
            if (r < rows) {
                const u32 i = wave * chunk + r * 64u + lane;
                if (pass) kreg[r] = i < n ? keys[i] : 0u;
                rreg[r] = digit_rank<ORDERED>(wcnt, (kreg[r] >> shift) & dmask, i < n);
            }
        }
        __syncthreads();
        u32 tot = 0u, excl = 0u, cw[NW];
        if (tid < 256u) {
#pragma unroll
            for (u32 w = 0; w < NW; w++) cw[w] = wcount[w * 256u + tid];
#pragma unroll
            for (u32 w = 0; w < NW; w++) tot += cw[w];
            const u32 inc = wave_incl_scan(tot);
            excl = inc - tot;
            if (lane == 63u) wsum[wave] = inc;
        }
        __syncthreads();
        if (tid < 256u) {
            u32 run = excl;
#pragma unroll
            for (u32 w = 0; w < 3u; w++) run += w < wave ? wsum[w] : 0u; // (waves 0..3 scan)
#pragma unroll
            for (u32 w = 0; w < NW; w++) {
                wcount[w * 256u + tid] = run;
                run += cw[w];
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 r = 0; r < (u32)ROWS; r++) { // (all keys are in registers: the array is overwritten)
            const u32 i = wave * chunk + r * 64u + lane;
            if (r < rows && i < n) keys[wcnt[(kreg[r] >> shift) & dmask] + rreg[r]] = kreg[r];
        }
        __syncthreads();
    }

    // ---- thresholds and class counts --------------------------------------------------------------
    if (tid == 0u) s_nneg = lower_bound_key(keys, n, ZERO_KEY);
    if (tid == 64u) s_npos0 = upper_bound_key(keys, n, ZERO_KEY);
    if (tid < n_cfg) {
        enter_config(s_cfg, tid, gd->cfg_pair[tid], gd->cfg_K[tid]);
    }
    __syncthreads();
    const u32 n_neg = s_nneg, n_nonpos = s_npos0;
    if (tid < n_thr) {
        // the k-th smallest magnitude: negative keys downwards and the others upwards are two sorted
        // lists; i of the k smaller ones come from the latter
        const u32 ppm = tid < n_p ? gd->p_ppm[tid] : gd->o_ppm[tid - n_p];
        const u32 c = (u32)((u64)n * ppm / 1000000ull);
        const u32 k = tid < n_p ? c : n - 1u - c;
        const u32 len_p = n - n_neg, len_n = n_neg;
        u32 lo = k > len_n ? k - len_n : 0u, hi = k < len_p ? k : len_p;
        while (lo < hi) {
            const u32 i = (lo + hi) >> 1, j = k - i; // (i < len_p and j > 0 here)
            if (mag_of_key(keys[n_neg + i]) < mag_of_key(keys[n_neg - j]))
                lo = i + 1u;
            else
                hi = i;
        }
        const u32 j = k - lo;
        const u32 mp = lo < len_p ? mag_of_key(keys[n_neg + lo]) : 0xFFFFFFFFu;
        const u32 mn = j < len_n ? mag_of_key(keys[n_neg - 1u - j]) : 0xFFFFFFFFu;
        s_thr[tid] = mp < mn ? mp : mn;
    }
    __syncthreads();
    for (u32 i = tid; i < 4u * n_thr; i += NT) {
        const u32 tau = s_thr[i >> 2];
        u32 c;
        switch (i & 3u) {
        case 0: c = n_neg - upper_bound_key(keys, n, key_neg(tau)); break;
        case 1: c = lower_bound_key(keys, n, key_pos(tau)) - n_neg; break;
        case 2: c = lower_bound_key(keys, n, key_neg(tau)); break;
        default: c = n - upper_bound_key(keys, n, key_pos(tau)); break;
        }
        s_cnt[i >> 2][i & 3u] = c;
    }
    __syncthreads();
    if (tid < n_pairs) {
        const u32 tp = gd->pair_p[tid], to = n_p + gd->pair_o[tid];
        const u32 Pn = s_cnt[tp][0], Pp = s_cnt[tp][1], An = s_cnt[to][2], Ap = s_cnt[to][3];
        const u32 Mn = n_neg - An - Pn, Mp = n - n_neg - Ap - Pp;
        s_A[tid] = An;
        s_Ap[tid] = n - Ap;
        s_gl[tid] = n_neg - Pn; // the pruned values are the sorted positions [s_gl, s_gr)
        s_gr[tid] = n_neg + Pp;
        s_Mn[tid] = Mn;
        s_M[tid] = Mn + Mp;
        st->pair_An[tid] = An;
        st->pair_Ap[tid] = Ap;
        st->pair_Pn[tid] = Pn;
        st->pair_Pp[tid] = Pp;
        st->pair_Mn[tid] = Mn;
        st->pair_M[tid] = Mn + Mp;
        if (Mn + Mp == 0u || Mn > n || Mp > n) atomicOr(&st->internal_err, 32u);
    }
    if (tid < n_thr) st->thr_mag[tid] = s_thr[tid];
    if (tid == 0u) {
        st->n_neg = n_neg;
        st->n_zero = n_nonpos - n_neg;
        st->n_thr = n_thr;
        st->nb2 = 8u * (u32)COARSE;
        st->zbin = ZERO_KEY >> L1_SHIFT;
        if (mag_of_key(keys[0]) >= 0x7f800000u || mag_of_key(keys[n - 1u]) >= 0x7f800000u) st->nonfinite = 1u;
    }
    // sums of squares of the protected values
    for (u32 o = 0; o < n_o; o++) {
        const u32 a = s_cnt[n_p + o][2], c = a + s_cnt[n_p + o][3], skip = n - c;
        double q = 0.0;
        for (u32 i = tid; i < c; i += NT) {
            const double x = value_of_key(keys[i < a ? i : i + skip]);
            q = fma(x, x, q);
        }
        if (c) q = wave_sum_f64(q); // (the same for all)
        if (lane == 0u) s_red[wave][1u + o] = q;
    }
    __syncthreads();
    if (tid <= n_o) {
        double s = 0.0;
        for (u32 w = 0; w < NW; w++) s += s_red[w][tid];
        s_sq[tid] = s;
        if (tid == 0u)
            st->sumsq = s;
        else
            st->thr_sumsq[n_p + tid - 1u] = s;
    }

    // ---- boundaries --------------------------------------------------------------------------------
    const u32 n_bnd = gd->n_all; // (all of them: the sums start from 256 bins)
    u32 *tk = B.tgt_key + (size_t)t * TGT_STRIDE;
    for (u32 w = tid; w < n_pairs * n_bnd; w += NT) {
        const u32 q = w / n_bnd, i = w % n_bnd;
        u32 num, den;
        bnd_fraction(i, num, den);
        const u32 k = num * s_M[q] / den; // (below 2^14 * 256)
        u32 r = k < s_Mn[q] ? s_A[q] + k : s_A[q] + (s_gr[q] - s_gl[q]) + k;
        if (r >= n) { // (only without quantized values, which is reported)
            r = n - 1u;
            atomicOr(&st->internal_err, 64u);
        }
        const u32 key = keys[r];
        tk[q * NBT + i] = key;
        LB[q * LBS + i] = (u16)((r && keys[r - 1u] == key) ? lower_bound_key(keys, r, key) : r);
    }
    __syncthreads();
    // ---- sums of the 8-bit bins of every pair ------------------------------------------------------
    // positions of bin k of K bins, boundaries lo and hi apart, without the pruned gap
    auto bin_lo = [&](u32 q, u32 K, u32 k) -> u32 { return k == 0u ? s_A[q] : (u32)LB[q * LBS + bnd_index(K, k)]; };
    auto bin_hi = [&](u32 q, u32 K, u32 k) -> u32 {
        return k == K - 1u ? s_Ap[q] : (u32)LB[q * LBS + bnd_index(K, k + 1u)];
    };
    auto bin_count = [&](u32 q, u32 a, u32 b) -> u32 {
        const u32 x = a > s_gl[q] ? a : s_gl[q], y = b < s_gr[q] ? b : s_gr[q];
        return b - a - (x < y ? y - x : 0u);
    };
    auto range_sum = [&](u32 q, u32 a, u32 b) -> double {
        const u32 gl = s_gl[q], gr = s_gr[q];
        return sum_range(keys, a, b < gl ? b : gl) + sum_range(keys, a > gr ? a : gr, b);
    };
    for (u32 w = tid; w < n_pairs * 256u; w += NT) {
        const u32 q = w >> 8, k = w & 255u;
        S8[w] = range_sum(q, bin_lo(q, 256u, k), bin_hi(q, 256u, k));
    }
    __syncthreads();
    // ---- centres and errors, 256 bins first, then 128, ... 2 (sums of neighbours) ------------------
    float *cb = B.codebook + (size_t)t * n_cfg * CB_STRIDE;
    auto centre = [&](u32 q, u32 K, u32 k, u32 g, double sk) -> double { // returns 2 c S - n c^2
        const u32 nk = bin_count(q, bin_lo(q, K, k), bin_hi(q, K, k));
        const float c = nk ? (float)(sk / (double)nk) // (an empty bin: its lower boundary)
                           : __uint_as_float(bits_of_key(keys[LB[q * LBS + bnd_index(K, k == 0u ? 1u : k)]]));
        cb[g * CB_STRIDE + k] = c;
        const double cd = (double)c;
        return 2.0 * cd * sk - (double)nk * cd * cd;
    };
    for (u32 q = wave; q < n_pairs; q += NW) { // 3, 6 and 12 bins: whole 8-bit bins and the pieces at either end
        for (u32 s = 9u; s < 12u; s++) {
            const u32 g = s_cfg[q][s];
            if (g == 0xFFFFu) continue;
            const u32 K = 3u << (s - 9u);
            double acc = 0.0;
            if (lane < K) {
                const u32 a = bin_lo(q, K, lane), b = bin_hi(q, K, lane);
                u32 lo = 0u, hi = 256u; // first 8-bit bin that starts at or after a
                while (lo < hi) {
                    const u32 mid = (lo + hi) >> 1;
                    if (bin_lo(q, 256u, mid) < a)
                        lo = mid + 1u;
                    else
                        hi = mid;
                }
                u32 e = lo; // one past the last that ends at or before b
                for (u32 step = 128u; step > 0u; step >>= 1)
                    if (e + step <= 256u && bin_hi(q, 256u, e + step - 1u) <= b) e += step;
                double sk = 0.0;
                if (e > lo) {
                    for (u32 k = lo; k < e; k++) sk += S8[q * 256u + k];
                    sk += range_sum(q, a, bin_lo(q, 256u, lo)) + range_sum(q, bin_hi(q, 256u, e - 1u), b);
                } else {
                    sk = range_sum(q, a, b);
                }
                acc = centre(q, K, lane, g, sk);
            }
            acc = wave_sum_f64(acc);
            if (lane == 0u) s_acc[q][s] = acc;
        }
    }
    for (u32 lg = 8u; lg >= 1u; lg--) {
        const u32 K = 1u << lg;
        for (u32 q = wave; q < n_pairs; q += NW) {
            const u32 g = s_cfg[q][lg];
            if (g == 0xFFFFu) continue;
            double acc = 0.0;
            for (u32 k = lane; k < K; k += 64u) acc += centre(q, K, k, g, S8[q * 256u + k]);
            acc = wave_sum_f64(acc);
            if (lane == 0u) s_acc[q][lg] = acc;
        }
        if (lg == 1u) break;
        // (a pair's sums are folded by the wave that reads them: no barrier, a wave's LDS operations
        // stay in order)
        asm volatile("" ::: "memory");
        for (u32 q = wave; q < n_pairs; q += NW) {
            double f[2];
#pragma unroll
            for (u32 j = 0; j < 2u; j++) {
                const u32 k = lane + 64u * j;
                f[j] = k < K / 2u ? S8[q * 256u + 2u * k] + S8[q * 256u + 2u * k + 1u] : 0.0;
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (u32 j = 0; j < 2u; j++) {
                const u32 k = lane + 64u * j;
                if (k < K / 2u) S8[q * 256u + k] = f[j];
            }
        }
        asm volatile("" ::: "memory");
    }
    __syncthreads();
    // ---- scores and choice -------------------------------------------------------------------------
    Score *sc = B.scores + (size_t)t * n_cfg;
    for (u32 g = tid; g < n_cfg; g += NT) {
        const u32 K = gd->cfg_K[g], q = gd->cfg_pair[g];
        double sse = s_sq[0] - s_sq[1u + gd->pair_o[q]] - s_acc[q][k_slot(K)];
        if (sse < 0.0) sse = 0.0;
        Score r;
        r.sse = sse;
        r.sumsq = s_sq[0];
        r.n_outlier = s_A[q] + (n - s_Ap[q]);
        r.n_kept = s_M[q];
        r.n_pruned = s_gr[q] - s_gl[q];
        r.cost_bits = payload_bits(r.n_kept, r.n_outlier, K, gd->cfg_l16[g]);
        sc[g] = r;
        s_sse[g] = sse;
        s_cost[g] = r.cost_bits;
        if (r.n_pruned + r.n_outlier + r.n_kept != d.n) atomicOr(&st->internal_err, 256u);
    }
    __syncthreads();
    if (wave == 0u) {
        const Choice c = choose_config(s_sse, s_cost, n_cfg, gd->eps, s_sq[0]);
        if (lane == 0u) {
            st->best = c.best;
            st->feasible = c.feasible;
            store_result(st, B.res + t);
        }
    }
}

// The small tensor at position t by a workgroup of 1024 threads; sm: SMALL_LDS bytes.
constexpr int SMALL_LDS = (int)sizeof(SmallShared<BLOCK, SMALL_MAX / BLOCK>);
template <bool ORDERED>
__device__ __forceinline__ void small_beside(void *sm, const TDesc *td, const GridDesc *gd, const Bufs &B, int t, bool large)
{
    if (large)
        search_small<BLOCK, SMALL_MAX / BLOCK, ORDERED>(*reinterpret_cast<SmallShared<BLOCK, SMALL_MAX / BLOCK> *>(sm), t, td, gd, B);
    else
        search_small<BLOCK, SMALL_TINY / BLOCK, ORDERED>(*reinterpret_cast<SmallShared<BLOCK, SMALL_TINY / BLOCK> *>(sm), t, td, gd, B);
}
// Tensors of up to SMALL_TINY values go by 1024 threads beside the launch's others while all its workgroups are resident
// together (47 us for one of 4096 values), else by 512 threads, two workgroups to a CU, in a launch of their own (53 us;
// 300 of them 71 us instead of 92).
inline bool small_crowd(const Batch &bt, int others) { return others + bt.nS1 + bt.nS0 > bt.n_cu; }

} // namespace inshr
