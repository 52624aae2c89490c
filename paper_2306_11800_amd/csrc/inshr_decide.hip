// The choice of a search (Sec. 5) from the second histogram alone, where bounds of the errors settle it.
//
// A search that is not asked for its score table has one answer per tensor: the cheapest configuration
// within eps.  What a configuration costs follows from the exact class counts; its error is known within a
// few percent from the equal-population bins of sweep 2, and that is nearly always enough.  Boundaries and
// centres are then worked out for the chosen configuration alone, by the quantizer, instead of for every
// pair of the grid: of 32768 bins 259 hold an edge instead of up to 3885, the gathered keys of which took sweep 3,
// the split and the group sort two thirds of a search (6.7 G values, 105 configurations: 16.8 of 25.0 ms;
// k_decide in their place: 0.07 ms.  Search and quantizing together 33.4 -> 20.0 ms).
// Where one configuration's bounds leave the choice open, its exact error is worked out (launch_resolve with that
// configuration in view) and settles it; a tensor with more of them is scored exactly, the whole grid.
//
// The bounds.  Let x^ be the sorted values with every value replaced by the middle of its bin's key range
// (the order stays), F_P(y) = sum over the clusters of partition P of (y - mean)^2 + sum of the pruned y^2.
//   - sqrt F_P is a distance from a linear space: |sqrt F_P(x) - sqrt F_P(x^)| <= |x - x^|, and the right
//     side is at most sqrt V, V = sum over the values not protected of (half their bin's width)^2.
//   - The clusters start at values of given ranks; a run of equal values goes to the upper cluster as a
//     whole.  The true partition P' therefore differs from the partition by rank P in that at most r_j
//     values of boundary j's bin (its values below the rank) move up from cluster j - 1 to j.  They have the
//     same x^ = m_j.  With the means c of P: F_P'(x^) <= F_P(x^) + sum r_j max(0, (m_j - c_j)^2 - (m_j -
//     c_(j-1))^2); with the means c' of P', which lie between c and the mean that every possible move
//     together would give, F_P'(x^) >= F_P(x^) - sum r_j max(0, (m_j - c'_(j-1))^2 - (m_j - c'_j)^2).
// The sums over ranks are taken in fp64, in units of a power of two near the tensor's root mean square, and so
// are means and the lowest means c'.  What is rounded to fp32 (u = 2^-24):
//   - the middles, by u of their size each; any number may stand for a bin's middle as long as its distance to
//     the values is counted, so |x - x^| grows by at most u |x|: 2 u of the sum of squares in F
//   - V's terms and their sums over 32 bins, 34 u of V up to the rank; 1e-5 of it (168 u) is added
//   - the distances in U and L, differences of squares that may cancel: at most 13 u (m^2 + mean^2) per square,
//     26 u (1.6e-6) of the three squares together; 4e-6 of them is added to each difference
//   - F and the pruned squares when they are added up, the roots and their squares: a few u of the sum of squares
//     where a bound is near eps or a lower one.  1e-5 (168 u) of the sum of squares is added on either side.
//
// One workgroup per tensor (its LDS leaves room for one on a CU), bound by the latency of its steps: 39 us for one tensor
// (k_plan2, the first of those it takes the place of, 36 us), 128 us for 294 tensors and 105 configurations.
#include "inshr_small.h"

namespace inshr {

constexpr int D_EDGES = (MAX_PAIRS * EPP + 7) & ~7; // edges (boundaries and class edges of all pairs) at most
constexpr int D_PER = (D_EDGES + BLOCK - 1) / BLOCK; // per thread
struct DecideMarks {                     // per bin with an edge: sums over the bins before it
    double s1[D_EDGES], s2[D_EDGES];
    float v[D_EDGES], mid[D_EDGES], rad[D_EDGES];
};
struct DecideEdges {                     // per edge: sums over the ranks before it
    double s1[D_EDGES], s2[D_EDGES];
    float mid[D_EDGES];                  // middle of its bin
    u32 rank[D_EDGES], res[D_EDGES];     // its rank, the values of its bin below it
};
struct DecideShared {
    union {
        DecideMarks m;
        DecideEdges e;
    };
    u32 T[COARSE];                       // key prefix -> bins
    u32 pre8[L2_BINS / 8];               // keys in the bins before every eighth
    u32 act[L2_BINS / 32];               // bins with an edge
    u32 before[L2_BINS / 32];            // ... in the words before
    double w_s[3][BLOCK / 64];
    float v[MAX_PAIRS][2];               // V up to the first and the last class edge
    float lo[MAX_CFG], hi[MAX_CFG];
    u64 cost[MAX_CFG];
    u64 rk[MAX_PAIRS][4], M[MAX_PAIRS], Mn[MAX_PAIRS]; // ranks of the class edges; quantized values
    double sumsq;
    u32 tmp[BLOCK / 64], tmp2[BLOCK / 64];
};

__device__ __forceinline__ void decide(DecideShared &sh, int t, const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                       const u32 *__restrict__ t_fu_off, const Bufs &B)
{
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u64 n = td[t].n;
    TState *st = B.ts + t;
    const u32 n_pairs = gd->n_pairs, n_cfg = gd->n_cfg, n_bnd = gd->n_bnd, per_pair = n_bnd + 4u;
    const u32 n_edges = n_pairs * per_pair;
    const u32 *h2 = B.hist2 + (size_t)t * L2_BINS;
    const u32 *tab = B.table2 + (size_t)t * COARSE;
    typedef u32 u4 __attribute__((ext_vector_type(4)));

    // ---- the thread's 32 bins (those past the last one are empty) ------------------------------------
    u4 c[8];
#pragma unroll
    for (u32 i = 0; i < 8u; i++) c[i] = ((const GLOBAL_AS u4 *)gptr(h2))[tid * 8u + i];
    for (u32 i = tid; i < (u32)COARSE; i += BLOCK) sh.T[i] = tab[i];
    sh.act[tid] = 0u;
    static_assert(L2_BINS / 32 == BLOCK, "one word of the marked bins per thread");
    store_pairs(st, gd, n);
    if (tid < n_pairs) { // (its own stores)
        const u64 n_neg = st->n_neg;
        sh.rk[tid][0] = st->pair_An[tid];
        sh.rk[tid][1] = n_neg - st->pair_Pn[tid];
        sh.rk[tid][2] = n_neg + st->pair_Pp[tid];
        sh.rk[tid][3] = n - st->pair_Ap[tid];
        sh.M[tid] = st->pair_M[tid];
        sh.Mn[tid] = st->pair_Mn[tid];
    }
    if (wave == BLOCK / 64 - 1u) { // the units' parts of the sum of squares, in a fixed order
        double s = 0.0;
        for (u32 u = t_fu_off[t] + lane; u < t_fu_off[t + 1]; u += 64u) s += B.sq_part[(size_t)u * SQ_STRIDE];
        s = wave_sum_f64(s);
        if (lane == 0u) {
            sh.sumsq = s;
            st->sumsq = s;
        }
    }
    u32 part[4];
    u32 mine = 0u;
#pragma unroll
    for (u32 i = 0; i < 8u; i++) {
        if ((i & 1u) == 0u) part[i >> 1] = mine;
        mine += c[i].x + c[i].y + c[i].z + c[i].w;
    }
    const u32 inc_n = wave_incl_scan(mine);
    if (lane == 63u) sh.tmp[wave] = inc_n;
    __syncthreads();
    u32 before = inc_n - mine, total = 0u;
    for (u32 w = 0; w < BLOCK / 64; w++) {
        const u32 x = sh.tmp[w];
        before += w < wave ? x : 0u;
        total += x;
    }
#pragma unroll
    for (u32 i = 0; i < 4u; i++) sh.pre8[4u * tid + i] = before + part[i];
    if (tid == 0 && (u64)total != n) atomicOr(&st->internal_err, 16u);
    // unit of all values below: a power of two near the root mean square
    const double ms = sh.sumsq / (double)n;
    int ex = ms > 0.0 && ms < 1e300 ? ilogb(ms) / 2 : 0;
    ex = ex < -120 ? -120 : ex > 120 ? 120 : ex;
    const float unit = ldexpf(1.0f, -ex);
    const float sumsq = (float)ldexp(sh.sumsq, -2 * ex);
    __syncthreads();

    // ---- bin of every edge's rank, and the values of that bin below the rank ------------------------
    u32 e_rank[D_PER], e_bin[D_PER], e_res[D_PER];
#pragma unroll
    for (int k = 0; k < D_PER; k++) {
        const u32 i = tid + (u32)(k * BLOCK);
        e_rank[k] = e_bin[k] = e_res[k] = 0u;
        if (i >= n_edges) continue;
        const u32 q = i / per_pair, j = i % per_pair;
        u64 r;
        if (j < n_bnd) {
            u32 num, den;
            bnd_fraction(gd->bnd[j], num, den);
            const u64 x = (u64)num * sh.M[q], kk = den == 256u ? x >> 8 : x / 12ull;
            r = sh.rk[q][0] + kk + (kk < sh.Mn[q] ? 0ull : sh.rk[q][2] - sh.rk[q][1]);
        } else {
            r = sh.rk[q][j - n_bnd];
        }
        e_rank[k] = r < n ? (u32)r : (u32)n;
    }
#pragma unroll
    for (int k = 0; k < D_PER; k++) { // last group of eight bins that starts at or before the rank
        u32 b = 0u;
#pragma unroll
        for (u32 step = L2_BINS / 16; step > 0u; step >>= 1)
            if (sh.pre8[b + step] <= e_rank[k]) b += step;
        e_bin[k] = b;
    }
#pragma unroll
    for (int k = 0; k < D_PER; k++) {
        if (tid + (u32)(k * BLOCK) >= n_edges) continue;
        u32 run = sh.pre8[e_bin[k]], bin = 8u * e_bin[k], res = e_rank[k] - run;
        const u4 x = ((const GLOBAL_AS u4 *)gptr(h2))[2u * e_bin[k]], y = ((const GLOBAL_AS u4 *)gptr(h2))[2u * e_bin[k] + 1u];
        const u32 f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
        for (u32 i = 1; i < 8u; i++) { // last bin that starts at or before the rank
            run += f[i - 1u];
            if (run <= e_rank[k]) {
                bin = 8u * e_bin[k] + i;
                res = e_rank[k] - run;
            }
        }
        e_bin[k] = bin;
        e_res[k] = res;
        atomicOr(&sh.act[bin >> 5], 1u << (bin & 31u));
    }
    // ---- every thread sums up its 32 bins ------------------------------------------------------------
    u32 p0 = 0u; // key prefix of the first one
#pragma unroll
    for (u32 step = COARSE / 2; step > 0u; step >>= 1)
        if (((sh.T[p0 + step] >> 5) & 0x7fffu) <= 32u * tid) p0 += step;
    auto walk = [&](auto &&f) { // f(i, keys, middle, half the width) of the thread's bins in order
        u32 p = p0, e = sh.T[p0], sub = 32u * tid - ((e >> 5) & 0x7fffu);
        u4 next = ((const GLOBAL_AS u4 *)gptr(h2))[tid * 8u];
#pragma unroll 1
        for (u32 i4 = 0; i4 < 8u; i4++) { // (four at a time, read again: 32 in registers, in fp64 too, would spill)
            const u4 now = next;
            if (i4 < 7u) next = ((const GLOBAL_AS u4 *)gptr(h2))[tid * 8u + i4 + 1u];
#pragma unroll
            for (u32 j = 0; j < 4u; j++) {
                const u32 k = now[j], d = e & 31u;
                float m = 0.0f, r = 0.0f;
                if (k) { // (finite values only: no bin of infinities)
                    const u32 first = (p << COARSE_SHIFT) | (sub << (COARSE_SHIFT - d));
                    const float a = __uint_as_float(bits_of_key(first)) * unit;
                    const float b = __uint_as_float(bits_of_key(first + ((1u << (COARSE_SHIFT - d)) - 1u))) * unit;
                    m = 0.5f * (a + b);
                    r = 0.5f * (b - a);
                }
                f(4u * i4 + j, k, m, r);
                if (++sub >> d) {
                    sub = 0u;
                    p = p + 1u < (u32)COARSE ? p + 1u : p;
                    e = sh.T[p];
                }
            }
        }
    };
    double s1 = 0.0, s2 = 0.0;
    float v = 0.0f;
    auto add = [&](u32 k, float m, float r) {
        const double km = (double)k * (double)m;
        s1 += km;
        s2 += km * (double)m;
        v += (float)k * r * r;
    };
    walk([&](u32, u32 k, float m, float r) { add(k, m, r); });
    auto scan = [&](double x, int which) { // exclusive over the lanes; the waves' totals to LDS
        double y = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double z = __shfl_up(y, o);
            if ((int)lane >= o) y += z;
        }
        if (lane == 63u) sh.w_s[which][wave] = y;
        return y - x;
    };
    double b1 = scan(s1, 0), b2 = scan(s2, 1), bv = scan((double)v, 2);
    __syncthreads(); // (all edges are marked)
    const u32 word = sh.act[tid], n_marks = (u32)__popc(word);
    const u32 inc = wave_incl_scan(n_marks);
    if (lane == 63u) sh.tmp2[wave] = inc;
    __syncthreads();
    u32 at = inc - n_marks;
    for (u32 w = 0; w < wave; w++) {
        b1 += sh.w_s[0][w];
        b2 += sh.w_s[1][w];
        bv += sh.w_s[2][w];
        at += sh.tmp2[w];
    }
    sh.before[tid] = at;
    if (word) {
        s1 = s2 = 0.0;
        v = 0.0f;
        walk([&](u32 i, u32 k, float m, float r) {
            if ((word >> i) & 1u) {
                sh.m.s1[at] = b1 + s1;
                sh.m.s2[at] = b2 + s2;
                sh.m.v[at] = (float)(bv + (double)v);
                sh.m.mid[at] = m;
                sh.m.rad[at] = r;
                at++;
            }
            add(k, m, r);
        });
    }
    __syncthreads();
    // ---- sums over the ranks before every edge -------------------------------------------------------
    double e1[D_PER], e2[D_PER];
    float em[D_PER];
#pragma unroll
    for (int k = 0; k < D_PER; k++) {
        const u32 i = tid + (u32)(k * BLOCK);
        e1[k] = e2[k] = 0.0;
        em[k] = 0.0f;
        if (i >= n_edges) continue;
        const u32 w = e_bin[k] >> 5;
        const u32 x = sh.before[w] + (u32)__popc(sh.act[w] & ((1u << (e_bin[k] & 31u)) - 1u));
        const float r = (float)e_res[k], h = sh.m.rad[x];
        em[k] = sh.m.mid[x];
        e1[k] = sh.m.s1[x] + (double)e_res[k] * (double)em[k];
        e2[k] = sh.m.s2[x] + (double)e_res[k] * ((double)em[k] * (double)em[k]);
        const u32 q = i / per_pair, j = i % per_pair;
        if (j == n_bnd || j == n_bnd + 3u) sh.v[q][j == n_bnd ? 0 : 1] = sh.m.v[x] + r * h * h;
    }
    __syncthreads();
    // (edges of pair q: boundary index b at q * EPP + b, class edges at q * EPP + NBT ..)
#pragma unroll
    for (int k = 0; k < D_PER; k++) {
        const u32 i = tid + (u32)(k * BLOCK);
        if (i >= n_edges) continue;
        const u32 q = i / per_pair, j = i % per_pair;
        const u32 to = q * (u32)EPP + (j < n_bnd ? (u32)gd->bnd[j] : (u32)NBT + (j - n_bnd));
        sh.e.s1[to] = e1[k];
        sh.e.s2[to] = e2[k];
        sh.e.mid[to] = em[k];
        sh.e.rank[to] = e_rank[k];
        sh.e.res[to] = e_res[k];
    }
    __syncthreads();
    // ---- bounds of every configuration: a wave each, a run of bins per lane --------------------------
    const float slack = 1e-5f * sumsq;
    for (u32 g = wave; g < n_cfg; g += BLOCK / 64) {
        const u32 K = gd->cfg_K[g], q = gd->cfg_pair[g], e0 = q * (u32)EPP;
        const u32 per = K > 64u ? K / 64u : 1u; // 1, 2 or 4
        const u32 g1 = e0 + (u32)NBT + 1u, g2 = e0 + (u32)NBT + 2u; // the pruned gap
        const u32 rg1 = sh.e.rank[g1], rg2 = sh.e.rank[g2];
        const double gS = sh.e.s1[g2] - sh.e.s1[g1], gQ = sh.e.s2[g2] - sh.e.s2[g1];
        double F = 0.0;
        float U = 0.0f, L = 0.0f;
        bool empty = false;
        // the bin before the lane's first is recomputed for the boundary between them
        float c_prev = 0.0f, l_prev = 0.0f;
        if (lane * per < K) {
            for (u32 j = lane ? 0u : 1u; j <= per; j++) {
                const u32 b = lane * per + j - 1u;
                const u32 lo = b ? e0 + bnd_index(K, b) : e0 + (u32)NBT;
                const u32 up = b + 1u < K ? e0 + bnd_index(K, b + 1u) : e0 + (u32)NBT + 3u;
                const u32 rl = sh.e.rank[lo], ru = sh.e.rank[up];
                const float ml = sh.e.mid[lo], mu = sh.e.mid[up];
                u32 nk = ru - rl;
                double S = sh.e.s1[up] - sh.e.s1[lo], Q = sh.e.s2[up] - sh.e.s2[lo];
                if (rl < rg2 && ru > rg1) { // the bin lies around the gap
                    nk -= rg2 - rg1;
                    S -= gS;
                    Q -= gQ;
                }
                if (nk == 0u || nk > 0x7fffffffu || (float)n > 1e4f * (float)nk) empty = true; // (no bound)
                nk = nk ? nk : 1u;
                const double mean_d = S / (double)nk;
                const float mean = (float)mean_d;
                const u32 xu = b + 1u < K ? sh.e.res[up] : 0u, xl = b ? sh.e.res[lo] : 0u;
                float low = ml; // the lowest mean that the moves can give
                if (nk > xu) { // (the counts are exact)
                    low = (float)((S - (double)xu * (double)mu + (double)xl * (double)ml) / ((double)(nk - xu) + (double)xl));
                    low = fminf(fmaxf(low, ml), mean);
                }
                if (j) F += fmax(Q - S * mean_d, 0.0);
                if (b && j) { // boundary b, between bins b - 1 and b
                    const float x = ml - mean, y = ml - c_prev, z = ml - l_prev, w = fmaxf(low - ml, 0.0f);
                    U += (float)xl * fmaxf(x * x - y * y + 4e-6f * (ml * ml + mean * mean + c_prev * c_prev), 0.0f);
                    L += (float)xl * fmaxf(z * z - w * w + 4e-6f * (ml * ml + low * low + l_prev * l_prev), 0.0f);
                }
                c_prev = mean;
                l_prev = low;
            }
        }
        F = wave_sum_f64(F);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            U += __shfl_xor(U, o);
            L += __shfl_xor(L, o);
        }
        const bool open = __ballot(empty) != 0ull;
        if (lane == 0u) {
            const float V = fmaxf(sh.v[q][1] - sh.v[q][0], 0.0f) + 1e-5f * sh.v[q][1];
            const float rv = sqrtf(V), f = (float)F, pruned = fmaxf((float)gQ, 0.0f);
            const float a = sqrtf(fmaxf(f - L, 0.0f) + pruned) - rv, z = sqrtf(f + U + pruned) + rv;
            sh.lo[g] = open ? -1.0f : (a > 0.0f ? a * a : 0.0f) - slack;
            sh.hi[g] = open ? __uint_as_float(0x7f800000u) : z * z + slack;
            sh.cost[g] = payload_bits(sh.M[q], sh.rk[q][0] + (n - sh.rk[q][3]), K, gd->cfg_l16[g]);
        }
    }
    __syncthreads();
    // ---- the choice: the cheapest configuration that is surely within eps, unless one that may be is cheaper
    if (wave == 0u) {
        // (a bound on eps of this size settles nothing; the products keep two digits more than the slack)
        const bool usable = gd->eps >= 0.0 && gd->eps < 1e6;
        const float lim = (float)gd->eps * sumsq;
        u64 bc = ~0ull;
        u32 bg = 0xFFFFFFFFu;
        for (u32 g = lane; g < n_cfg; g += 64u)
            if (sh.hi[g] <= lim && (bg == 0xFFFFFFFFu || sh.cost[g] < bc)) {
                bc = sh.cost[g];
                bg = g;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const u64 c2 = __shfl_xor(bc, o);
            const u32 g2 = __shfl_xor(bg, o);
            if (g2 != 0xFFFFFFFFu && (bg == 0xFFFFFFFFu || c2 < bc || (c2 == bc && g2 < bg))) {
                bc = c2;
                bg = g2;
            }
        }
        // One configuration whose bounds leave it open, and nothing else: the choice hangs on its error alone, and
        // what it is if that configuration is out is known.  (Of the tensors that stay open none has been seen with
        // more: the bounds are a few tenths of a percent apart, the errors of neighbouring configurations far more.)
        const bool any_sure = bg != 0xFFFFFFFFu;
        u32 n_open = usable ? 0u : 2u, og = 0u;
        bool undecided = false;
        if (any_sure) {
            for (u32 g = lane; g < n_cfg; g += 64u)
                if (!(sh.hi[g] <= lim) && !(sh.lo[g] > lim) && (sh.cost[g] < bc || (sh.cost[g] == bc && g < bg))) {
                    n_open++;
                    og = g;
                }
        } else { // none surely within: settled where all are surely beyond and one is surely the most accurate
            float bh = __uint_as_float(0x7f800000u);
            for (u32 g = lane; g < n_cfg; g += 64u)
                if (bg == 0xFFFFFFFFu || sh.hi[g] < bh) {
                    bh = sh.hi[g];
                    bg = g;
                }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float h2x = __shfl_xor(bh, o);
                const u32 g2 = __shfl_xor(bg, o);
                if (g2 != 0xFFFFFFFFu && (bg == 0xFFFFFFFFu || h2x < bh || (h2x == bh && g2 < bg))) {
                    bh = h2x;
                    bg = g2;
                }
            }
            for (u32 g = lane; g < n_cfg; g += 64u) {
                if (!(sh.lo[g] > lim)) {
                    n_open++;
                    og = g;
                }
                undecided |= g != bg && !(sh.lo[g] > bh);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const u32 g2 = __shfl_xor(og, o);
            og = og > g2 ? og : g2; // (the only one, or of no account)
        }
        const u32 opens = wave_sum(n_open);
        const bool open = opens > 1u || __ballot(undecided) != 0ull;
        if (lane == 0u) {
            st->best = open ? VIEW_NONE : opens ? CHOICE_IF | og : bg;
            st->feasible = st->feasible_else = any_sure ? 1u : 0u;
            st->best_else = bg;
            store_result(st, B.res + t);
        }
    }
}

// The small tensors' searches in the first n_small workgroups (n16 of the larger kind first), which take as long as a
// decision: 70 us, 60 us here and two launches of small ones before them were 70 + 50 + 60 us for a checkpoint of all
// three kinds.
template <bool ORDERED>
__global__ __launch_bounds__(BLOCK) void k_decide(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                  const u32 *__restrict__ t_fu_off, Bufs B, int nB, int n16, int n_small)
{
    extern __shared__ double sm_decide[];
    const int b = blockIdx.x;
    if (b < n_small)
        small_beside<ORDERED>(sm_decide, td, gd, B, nB + b, b < n16);
    else
        decide(*reinterpret_cast<DecideShared *>(sm_decide), b - n_small, td, gd, t_fu_off, B);
}

hipError_t launch_decide(const Batch &bt, hipStream_t s)
{
    constexpr int lds = (int)sizeof(DecideShared) > SMALL_LDS ? (int)sizeof(DecideShared) : SMALL_LDS;
    static bool attr = false;
    hipError_t e;
    if (!attr) {
        if ((e = hipFuncSetAttribute((const void *)k_decide<true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds))) return e;
        if ((e = hipFuncSetAttribute((const void *)k_decide<false>, hipFuncAttributeMaxDynamicSharedMemorySize, lds))) return e;
        attr = true;
    }
    if (bt.nB == 0) return launch_small(bt, s);
    const bool crowd = small_crowd(bt, bt.nB);
    if (crowd && bt.nS0 && (e = launch_small_many(bt, s))) return e;
    const int n_small = bt.nS1 + (crowd ? 0 : bt.nS0);
    if (bt.lds_ordered)
        PROF("k_decide", s, k_decide<true><<<n_small + bt.nB, BLOCK, lds, s>>>(bt.td, bt.gd, bt.t_fu_off, bt.bufs, bt.nB, bt.nS1, n_small));
    else
        PROF("k_decide", s, k_decide<false><<<n_small + bt.nB, BLOCK, lds, s>>>(bt.td, bt.gd, bt.t_fu_off, bt.bufs, bt.nB, bt.nS1, n_small));
    return hipGetLastError();
}

} // namespace inshr
