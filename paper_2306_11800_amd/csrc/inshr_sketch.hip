// Boundaries from the log-space sketch and weighted K-Means on its buckets (Sec. 4.3 / Algorithm 1,
// Sec. 4.4 / Algorithms 2 and 3), as an alternative to the equal-population bins of the search: the
// values between the two thresholds are counted per bucket (sign, ceil(log_gamma |x|)), the
// buckets are clustered with sample weights sigma * frequency + (1 - sigma) * magnitude (both
// divided by their largest entry), and the cluster centres become the codebook; the quantizer then
// runs with the midpoints of neighbouring centres as boundaries.
//
//   k_sketch_hist    one more sweep over the tensors (4 bytes per element, like the search's
//                    sweeps): a table in LDS maps the magnitude's top 14 bits to the first bucket
//                    that its 2^17 magnitudes touch and the largest magnitude of that bucket (a
//                    range of 2^(1/64) never touches more than two buckets for alpha >= 0.01), so
//                    the bucket is one LDS read, an add and a shift; the counts go to an LDS
//                    histogram (positive buckets, negative buckets, zeros).  Zeros and denormals,
//                    whose ranges are wider, are set aside and search the bucket list.
//   k_sketch_kmeans  one workgroup per tensor: compacts the non-empty buckets, draws the K
//                    starting centres (one wave with the buckets in its registers: running sums by a
//                    scan), then Lloyd rounds on the sorted list by a wave per set of centres — a
//                    cluster is a contiguous run of buckets, found by bisection on the midpoints
//                    and summed in index order by one lane — until the runs repeat.
//                    All arithmetic is fp64 without contraction (products and sums rounded
//                    separately).  For the search over the bit width (Sec. 5 restricted to the
//                    number of bins) the draws are made once for 256 clusters and the rounds run
//                    for 4, 8, ..., 256 clusters from the first 4, 8, ... draws.
//   k_sketch_score   the search's sweep: all boundaries of the seven sets, sorted, cut the key axis
//                    into at most 502 slots; the slot of a key comes from the equal-population
//                    bins of the threshold search (a table gives the slot of every bin without a
//                    boundary; in the few bins with one the key is compared with the boundaries
//                    from the bin's first one on); count and sum per slot in LDS, added to the
//                    tensor's arrays in global memory.
//   k_sketch_choose  per tensor: the error of every set from the slot moments, the fewest bits
//                    within the bound, and that set's keys and centres for the quantizer.
#include "inshr_sketch.h"

#include <type_traits>

// The clustering follows its definition operation by operation: no product may be fused into the
// sum that takes it.  The __dmul_rn / __dadd_rn of the HIP headers are plain operators compiled with
// the headers' own contraction setting, so the operations are written here, with contraction off.
#pragma clang fp contract(off)

namespace inshr {

__device__ __forceinline__ double mul_rn(double a, double b) { return a * b; }
__device__ __forceinline__ double add_rn(double a, double b) { return a + b; }
__device__ __forceinline__ double sub_rn(double a, double b) { return a - b; }
__device__ __forceinline__ double div_rn(double a, double b) { return a / b; }

// Histogram layout: positive bucket b at b, negative bucket b at SK_MAX_IDX + b, zeros at
// 2 * SK_MAX_IDX.  Bucket of a denormal or zero magnitude (rare): search of the bucket list.
__device__ __noinline__ u32 sketch_slot_small(u32 bits, const SketchParams &P)
{
    const u32 mag = bits & 0x7fffffffu;
    if (mag == 0u) return 2u * (u32)SK_MAX_IDX;
    u32 lo = 0u, hi = P.n_idx - 1u;
    while (lo < hi) { // first bucket whose largest magnitude reaches mag
        const u32 mid = (lo + hi) >> 1;
        if (P.tops[mid] >= mag)
            hi = mid;
        else
            lo = mid + 1u;
    }
    return lo + (bits >> 31) * (u32)SK_MAX_IDX;
}

// LIGHT: also the protected values of the tile (wave-uniform count) and their squares.
template <bool FULL, bool LIGHT>
__device__ __forceinline__ void sketch_tile(const float (&v)[16], u32 mask, u32 tau_p, u32 tau_o,
                                            const u32 *cell, u32 *h, const SketchParams &P, u32 &n_prot,
                                            double &q_prot)
{
    u32 small = 0u; // elements between the thresholds whose magnitude is zero or denormal
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const u32 bits = __float_as_uint(v[i]);
        const u32 mag = bits & 0x7fffffffu;
        bool take = mag >= tau_p && mag <= tau_o;
        if (!FULL) take = take && ((mask >> i) & 1u);
        if (LIGHT) {
            const bool prot = mag > tau_o && (FULL || ((mask >> i) & 1u));
            const u64 pm = __ballot(prot);
            if (pm) {
                n_prot += (u32)__popcll(pm);
                if (prot) q_prot = fma((double)v[i], (double)v[i], q_prot);
            }
        }
        if (take && mag < 0x00800000u) small |= 1u << i;
        if (take && mag >= 0x00800000u) {
            // entry = first bucket of the cell << 17 | (2^17 - 1 - low bits of that bucket's largest
            // magnitude): the sum carries into the bucket field when the magnitude lies above it
            const u32 b = (cell[mag >> 17] + (mag & 0x1FFFFu)) >> 17;
            atomicAdd(&h[b + (bits >> 31) * (u32)SK_MAX_IDX], 1u);
        }
    }
    if (__ballot(small != 0u)) {
#pragma unroll 1
        for (int i = 0; i < 16; i++)
            if ((small >> i) & 1u) atomicAdd(&h[sketch_slot_small(__float_as_uint(v[i]), P)], 1u);
    }
}

template <bool LIGHT>
__global__ __launch_bounds__(BLOCK) void k_sketch_hist(const TDesc *__restrict__ td, int nT,
                                                       const u64 *__restrict__ wg_tile0,
                                                       const u32 *__restrict__ wg_fu0,
                                                       const GridDesc *__restrict__ gd,
                                                       const SketchDesc *__restrict__ sd,
                                                       SketchParams P, Bufs B)
{
    // one static array (it starts at LDS address 0, so offsets fold into the LDS instructions)
    __shared__ u32 smem[SK_CELLS + SK_HIST];
    u32 *cell = smem;
    u32 *h = smem + SK_CELLS;
    __shared__ double s_q[BLOCK / 64];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u64 tile_lo = wg_tile0[blockIdx.x], tile_hi = wg_tile0[blockIdx.x + 1];
    if (tile_lo >= tile_hi) return;
    for (int i = tid; i < SK_CELLS; i += BLOCK) cell[i] = P.cell[i];
    for (int i = tid; i < SK_HIST; i += BLOCK) h[i] = 0u;
    int t = find_tensor(td, nT, tile_lo);
    const int t_first = t;
    u64 tile = tile_lo;
    while (tile < tile_hi) {
        const TDesc d = td[t];
        const u64 n_tiles_t = (d.n + TILE - 1) / TILE;
        const u64 t_end = d.tile0 + n_tiles_t;
        const u64 stop = t_end < tile_hi ? t_end : tile_hi;
        const SketchDesc s = sd[t];
        if (!s.active) {
            tile = stop;
            t++;
            continue;
        }
        const TState *st = B.ts + t;
        const u32 pair = gd->cfg_pair[s.cfg];
        const u32 o = gd->pair_o[pair];
        const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + o];
        double q_prot = 0.0; // squares of this thread's protected values
        __syncthreads();
        for (; tile < stop; tile++) {
            const u64 e0 = (tile - d.tile0) * (u64)TILE;
            const u64 rem = d.n - e0;
            const u32 cnt = tile_len(rem, (u32)TILE);
            float v[16];
            const u32 mask = load_tile(d, e0, cnt, v);
            u32 n_prot = 0u; // protected values of this wave in the tile (wave-uniform)
            if (cnt == (u32)TILE)
                sketch_tile<true, LIGHT>(v, mask, tau_p, tau_o, cell, h, P, n_prot, q_prot);
            else
                sketch_tile<false, LIGHT>(v, mask, tau_p, tau_o, cell, h, P, n_prot, q_prot);
            if (LIGHT && lane == 0u && n_prot) atomicAdd(&B.tile_out[tile * MAX_FRAC + o], n_prot);
        }
        if (LIGHT) { // this unit's sum of squares of the protected values, in a fixed order
            q_prot = wave_sum_f64(q_prot);
            if (lane == 0u) s_q[wave] = q_prot;
        }
        __syncthreads();
        if (LIGHT && tid == 0) {
            double sum = 0.0;
            for (int w = 0; w < BLOCK / 64; w++) sum += s_q[w];
            B.sq_part[(size_t)(wg_fu0[blockIdx.x] + (u32)(t - t_first)) * SQ_STRIDE + 1u + o] = sum;
        }
        u32 *gh = P.hist + (size_t)t * SK_HIST;
        for (int i = tid; i < SK_HIST; i += BLOCK) {
            const u32 c = h[i];
            if (c) {
                atomicAdd(&gh[i], c);
                h[i] = 0u;
            }
        }
        t++;
    }
}

// histogram slot of position v in value order: negative buckets descending, zeros, positive ascending
__device__ __forceinline__ u32 slot_in_value_order(u32 v)
{
    if (v < (u32)SK_MAX_IDX) return 2u * (u32)SK_MAX_IDX - 1u - v;
    if (v == (u32)SK_MAX_IDX) return 2u * (u32)SK_MAX_IDX;
    return v - (u32)SK_MAX_IDX - 1u;
}
// value of the bucket at position slot of the histogram
__device__ __forceinline__ double slot_value(u32 slot, const SketchParams &P)
{
    if (slot == 2u * (u32)SK_MAX_IDX) return 0.0;
    if (slot < (u32)SK_MAX_IDX) return P.rep[slot];
    return -P.rep[slot - (u32)SK_MAX_IDX];
}

// Inclusive prefix sum of non-negative numbers over the 64 lanes, with data-parallel-primitive moves as in
// wave_incl_scan, and the value of the lane below (0 in lane 0).
template <int CTRL, int ROWS> __device__ __forceinline__ double moved(double x)
{
    const u64 b = (u64)__double_as_longlong(x);
    const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)b, CTRL, ROWS, 0xf, ROWS == 0xf);
    const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(b >> 32), CTRL, ROWS, 0xf, ROWS == 0xf);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
__device__ __forceinline__ double wave_incl_sum(double x)
{
    x = add_rn(x, moved<0x111, 0xf>(x));
    x = add_rn(x, moved<0x112, 0xf>(x));
    x = add_rn(x, moved<0x114, 0xf>(x));
    x = add_rn(x, moved<0x118, 0xf>(x));
    x = add_rn(x, moved<0x142, 0xa>(x));
    return add_rn(x, moved<0x143, 0xc>(x));
}
__device__ __forceinline__ double lane_below(double x) { return moved<0x138, 0xf>(x); }
__device__ __forceinline__ double lane_value(double x, u32 lane)
{
    const u64 b = (u64)__double_as_longlong(x);
    const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)b, (int)lane);
    const u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(b >> 32), (int)lane);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}

constexpr int KM_BLOCK = 512; // threads of a clustering workgroup (256 registers each: see draw_centres)
typedef double d2 __attribute__((ext_vector_type(2)));

// Weighted K-Means++ draws (Algorithm 3) by one wave, from a list of at most 64 * PER buckets of which a lane keeps PER,
// value, weight and distance, in registers: a draw waits for nobody.  Per draw a lane adds the probabilities of its
// buckets up, a scan gives the running sums of the lanes, and the first lane whose running sum exceeds the target
// finds its bucket (every lane looks, one is asked).  Bound by the chain of dependent fp64 operations: 256 draws
// from up to 256 / 384 / 1024 / 1536 buckets 65 / 89 / 152 / 200 us (by all waves, two barriers a draw and three from more than
// 1024 buckets: 200 us and more).  xw: weights in x.
template <u32 PER, class T, class D>
__device__ __forceinline__ void draw_centres(const T *xq, const D *xw, u32 m, u32 K, const double *uni, double *craw)
{
    const u32 lane = threadIdx.x & 63u, lo = lane * PER;
    double x[PER], v[PER], d[PER];
#pragma unroll
    for (u32 q = 0; q < PER; q++) {
        const u32 i = lo + q < m ? lo + q : m - 1u;
        x[q] = xq[i];
        v[q] = lo + q < m ? xw[i].x : 0.0;
        d[q] = 1.0; // (the first draw's probabilities are the weights)
    }
    double xj = 0.0;
    for (u32 r = 0; r < K; r++) {
        double upto[PER];
        upto[0] = mul_rn(d[0], v[0]);
#pragma unroll
        for (u32 q = 1; q < PER; q++) upto[q] = add_rn(upto[q - 1u], mul_rn(d[q], v[q]));
        const double inc = wave_incl_sum(upto[PER - 1u]), before = lane_below(inc), total = lane_value(inc, 63u);
        if (r == 0u || total > 0.0) { // (else every bucket is a centre already: the last one again)
            const double target = mul_rn(uni[r], total);
            // (a lane that has something to draw from: the tree's sums need not ascend, one that adds nothing may end an ulp
            // above the lane below it)
            const double whole = upto[PER - 1u];
            const u64 above = __ballot(whole > 0.0 && inc > target);
            if (above) {
                // (where rounding leaves no sum of the lane above: its last bucket that can be drawn)
                double rest = sub_rn(target, before);
                rest = rest > 0.0 ? rest : 0.0;
                rest = whole > rest ? rest : __longlong_as_double(__double_as_longlong(whole) - 1ll);
                double pick = x[PER - 1u];
#pragma unroll
                for (u32 q = PER - 1u; q-- > 0u;) pick = upto[q] > rest ? x[q] : pick;
                xj = lane_value(pick, (u32)__builtin_ctzll(above));
            } else { // no running sum exceeds the target (rounding): the last bucket that can be drawn
                double pick = x[0];
                bool some = false;
#pragma unroll
                for (u32 q = 0; q < PER; q++) {
                    const bool is = mul_rn(d[q], v[q]) > 0.0;
                    pick = is ? x[q] : pick;
                    some |= is;
                }
                const u64 can = __ballot(some);
                xj = lane_value(pick, can ? 63u - (u32)__builtin_clzll(can) : 0u);
            }
        }
        if (lane == 0u) craw[r] = xj;
#pragma unroll
        for (u32 q = 0; q < PER; q++) {
            const double df = sub_rn(x[q], xj), d2 = mul_rn(df, df);
            d[q] = (r == 0u || d2 < d[q]) ? d2 : d[q];
        }
    }
}
// The same from longer lists, by all threads; the distances in y of xw.
template <class T, class D>
__device__ __forceinline__ void draw_centres_long(const T *xq, D *xw, u32 m, u32 K, const double *uni, double *craw,
                                                  double *s_red, u32 *s_pick, u32 *s_last, u32 &s_chosen)
{
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 per = (m + KM_BLOCK - 1u) / KM_BLOCK;
    const u32 lo = tid * per < m ? tid * per : m, hi = lo + per < m ? lo + per : m;
    if (tid < 2u) {
        s_pick[tid] = 0xFFFFFFFFu;
        s_last[tid] = 0u;
    }
    __syncthreads();
    // Per draw: (1) every thread sums the probabilities of its share, a scan gives the running
    // sums inside the wave, the wave totals go to LDS; (2) every thread adds the totals of the
    // waves before its own (in wave order) and the first thread that has something to draw from and whose
    // running sum exceeds the target announces itself; (3) that thread walks its share.  The LDS cells alternate between two copies
    // from draw to draw, so that a draw never waits for the cells of the one before to be read.
    for (u32 r = 0; r < K; r++) {
        const u32 cp = r & 1u;
        double inc = 0.0;
        u32 last_pos = 0u; // last bucket of the share that could be drawn, + 1
        for (u32 i = lo; i < hi; i++) {
            const d2 b = xw[i];
            const double p = r ? mul_rn(b.y, b.x) : b.x;
            inc = add_rn(inc, p);
            if (p > 0.0) last_pos = i + 1u;
        }
        inc = wave_incl_sum(inc);
        const double before = lane_below(inc);
        if (lane == 63u) s_red[cp * (KM_BLOCK / 64) + wave] = inc;
        __syncthreads();
        double wbase = 0.0, total = 0.0;
        for (u32 wv = 0; wv < KM_BLOCK / 64; wv++) {
            if (wv == wave) wbase = total;
            total = add_rn(total, s_red[cp * (KM_BLOCK / 64) + wv]);
        }
        if (r > 0u && !(total > 0.0)) { // every bucket is a centre already: repeat the last one
            if (tid == 0) craw[r] = craw[r - 1u];
            continue; // (nothing of this draw's cells is used again before two more barriers)
        }
        const double target = mul_rn(uni[r], total);
        const double excl = add_rn(wbase, before), incl = add_rn(wbase, inc);
        // one atomic per wave: its first lane above the target, its last lane with a drawable bucket
        const u64 above = __ballot(incl > target && last_pos != 0u), drawable = __ballot(last_pos != 0u);
        if (above && lane == (u32)__builtin_ctzll(above)) atomicMin(&s_pick[cp], tid);
        if (drawable && lane == 63u - (u32)__builtin_clzll(drawable)) atomicMax(&s_last[cp], last_pos);
        __syncthreads();
        const u32 pick = s_pick[cp];
        if (tid == (pick == 0xFFFFFFFFu ? 0u : pick)) {
            // no running sum exceeds the target (rounding): the last bucket that could be drawn
            u32 jj = s_last[cp] ? s_last[cp] - 1u : 0u;
            if (pick != 0xFFFFFFFFu) {
                double run = excl; // the running sum at the start of this thread's share
                jj = last_pos - 1u;
                for (u32 i = lo; i < hi; i++) {
                    const d2 b = xw[i];
                    const double p = r ? mul_rn(b.y, b.x) : b.x;
                    run = add_rn(run, p);
                    if (p > 0.0 && run > target) {
                        jj = i;
                        break;
                    }
                }
            }
            s_chosen = jj;
            craw[r] = xq[jj];
            s_pick[cp ^ 1u] = 0xFFFFFFFFu;
            s_last[cp ^ 1u] = 0u;
        }
        __syncthreads();
        const double cj = xq[s_chosen];
        for (u32 i = lo; i < hi; i++) {
            const double df = sub_rn(xq[i], cj), dd = mul_rn(df, df), old = xw[i].y;
            xw[i].y = (r == 0u || dd < old) ? dd : old;
        }
    }
}

// Weights and products of the run [i, e) of a list, each added up in index order.  15 entries may be read past the list's
// end (LDS has room for them; behind a scratch row lies more of the same allocation): eight entries are asked for before the
// eight before them are added: about 14 ns a bucket in LDS, 25 with eight reads and the sums of what they bring in turn.
// (Lists in device memory, 16 of 6000 buckets, all widths / 256 / 16 centres: one entry at a time 16.3 / 8.8 / 5.8 ms, so 8.0 /
// 4.7 / 1.6.)
template <class D> __device__ __forceinline__ d2 run_sum(const D *xw, u32 i, u32 e)
{
    double sw = 0.0, sx = 0.0;
    constexpr u32 N = 8;
    d2 a[N], b[N];
    auto ask = [&](d2 (&to)[N]) {
#pragma unroll
        for (u32 j = 0; j < N; j++) to[j] = xw[i + j];
    };
    auto add = [&](const d2 (&from)[N]) {
#pragma unroll
        for (u32 j = 0; j < N; j++) {
            sw = add_rn(sw, from[j].x);
            sx = add_rn(sx, from[j].y);
        }
    };
    auto add_rest = [&](const d2 (&from)[N]) { // (a sum that starts at +0.0 does not change by another +0.0)
#pragma unroll
        for (u32 j = 0; j < N; j++) {
            sw = add_rn(sw, i + j < e ? from[j].x : 0.0);
            sx = add_rn(sx, i + j < e ? from[j].y : 0.0);
        }
    };
    if (i >= e) return d2{0.0, 0.0};
    ask(a);
    while (e - i > 2u * N) {
        i += N;
        ask(b);
        add(a);
        i += N;
        ask(a);
        add(b);
    }
    if (e - i > N) {
        i += N;
        ask(b);
        add(a);
        add_rest(b);
    } else {
        add_rest(a);
    }
    return d2{sw, sx};
}

// Weighted Lloyd rounds of one set of Kb centres by one wave, from the sorted centres c_set, which it leaves the last
// ones in; the number of rounds is returned.  Cluster k = the buckets in (midpoint k-1, midpoint k], a run of the
// sorted list, belongs to lane k % 64.  No wave waits for another set's rounds, and a cluster whose run is the one of
// the round before keeps its centre.  Bound by the longest run that changed: a cluster around zero can hold
// half of the buckets.
template <u32 Q, class T, class D>
__device__ __forceinline__ u32 lloyd_rounds(const T *xq, const D *xw, u32 m, u32 Kb, double *c_set, u32 max_iter)
{
    const u32 lane = threadIdx.x & 63u;
    double c[Q];
    u32 first[Q], end[Q], steps = 1u; // steps: a power of two above m
    while (steps <= m) steps <<= 1;
#pragma unroll
    for (u32 q = 0; q < Q; q++) {
        c[q] = q * 64u + lane < Kb ? c_set[q * 64u + lane] : 0.0;
        first[q] = end[q] = 0xFFFFFFFFu;
    }
    u32 rounds = 0u;
    for (u32 it = 0; it < max_iter; it++) {
        double mid[Q];
        u32 a[Q];
#pragma unroll
        for (u32 q = 0; q < Q; q++) {
            double below = lane_below(c[q]);
            const double across = lane_value(c[q > 0u ? q - 1u : 0u], 63u);
            if (q > 0u) below = lane == 0u ? across : below;
            mid[q] = mul_rn(add_rn(below, c[q]), 0.5);
            a[q] = 0u;
        }
        for (u32 step = steps >> 1; step > 0u; step >>= 1) { // buckets up to the midpoint
#pragma unroll
            for (u32 q = 0; q < Q; q++) {
                const u32 to = a[q] + step;
                const double x = xq[(to < m ? to : m) - 1u];
                a[q] = to <= m && !(x > mid[q]) ? to : a[q];
            }
        }
        bool again[Q], other = false;
#pragma unroll
        for (u32 q = 0; q < Q; q++) {
            const u32 k = q * 64u + lane;
            a[q] = k == 0u ? 0u : k < Kb ? a[q] : m;
        }
#pragma unroll
        for (u32 q = 0; q < Q; q++) {
            const u32 next = q + 1u < Q ? (u32)__builtin_amdgcn_readlane((int)a[q + 1u < Q ? q + 1u : q], 0) : m;
            const u32 up = __shfl_down(a[q], 1), e = lane == 63u ? next : up;
            other |= a[q] != first[q];
            again[q] = a[q] != first[q] || e != end[q];
            first[q] = a[q];
            end[q] = e;
        }
        if (__ballot(other) == 0ull) break;
#pragma unroll
        for (u32 q = 0; q < Q; q++) {
            if (!again[q]) continue;
            const d2 s = run_sum(xw, first[q], end[q]);
            if (s.x > 0.0) c[q] = div_rn(s.y, s.x);
        }
        rounds++;
    }
#pragma unroll
    for (u32 q = 0; q < Q; q++)
        if (q * 64u + lane < Kb) c_set[q * 64u + lane] = c[q];
    return rounds;
}

// One workgroup per tensor, bound by the latency of one wave's draws and Lloyd rounds.  74 tensors of 390 buckets:
// 0.62 ms -> 0.31; 17 of up to 300 buckets: 0.36 -> 0.15; 33 of about 1000: 2.1 -> 0.8 ms (before: a bucket per thread, all
// sets' rounds in step, every cluster added up in every round).
__global__ __launch_bounds__(KM_BLOCK) void k_sketch_kmeans(const GridDesc *__restrict__ gd,
                                                            const SketchDesc *__restrict__ sd,
                                                            SketchParams P)
{
    constexpr u32 WAVES = KM_BLOCK / 64;
    __shared__ u32 s_n[WAVES], s_max[WAVES], s_pick[2], s_last[2], s_rounds[SK_SETS], s_chosen;
    __shared__ double s_red[2 * WAVES];
    __shared__ double cen[512], craw[256]; // the sorted centres of every set, those of 2 << (set + 1) from 4 * (2 ^ set - 1)
    const int t = blockIdx.x;
    const SketchDesc s = sd[t];
    if (!s.active) return;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // one set of centres for the configuration's bits, or (P.multi) one for each of 2 .. 8 bits: the
    // draws of a narrower set are the first draws of the widest
    const u32 K = P.multi ? 256u : 1u << gd->cfg_bits[s.cfg];
    const u32 n_sets = P.multi ? (u32)SK_SETS : 1u;
    const u32 *h = P.hist + (size_t)t * SK_HIST;
    // bucket values; weights and, in turn, squared distances or products: in LDS when the list is short enough (a few
    // hundred to a few thousand buckets is the rule), else in the tensor's scratch rows
    __shared__ double l_x[SK_LDS];
    __shared__ d2 l_w[SK_LDS + 16];

    // ---- the non-empty buckets in value order (Algorithm 1: unique with counts); a wave has whole rows of 64 ----
    constexpr u32 ROWS = (SK_HIST + KM_BLOCK - 1) / KM_BLOCK;
    u32 cnt[ROWS], mine = 0u, cmax = 0u;
#pragma unroll
    for (u32 i = 0; i < ROWS; i++) {
        const u32 v = (wave * ROWS + i) * 64u + lane;
        cnt[i] = v < (u32)SK_HIST ? h[slot_in_value_order(v)] : 0u;
    }
#pragma unroll
    for (u32 i = 0; i < ROWS; i++) {
        mine += (u32)__popcll(__ballot(cnt[i] != 0u));
        cmax = cnt[i] > cmax ? cnt[i] : cmax;
    }
    cmax = (u32)__builtin_amdgcn_readlane((int)wave_incl_max(cmax), 63);
    if (lane == 0u) {
        s_n[wave] = mine;
        s_max[wave] = cmax;
    }
    __syncthreads();
    u32 base = 0u, m = 0u, maxc = 0u;
    for (u32 wv = 0; wv < WAVES; wv++) {
        const u32 y = s_n[wv];
        if (wv < wave) base += y;
        m += y;
        maxc = s_max[wv] > maxc ? s_max[wv] : maxc;
    }
    // the rest, for bucket lists in LDS or in device memory
    auto cluster = [&](auto *xq, auto *xw, auto in_lds) {
        constexpr bool LDS = decltype(in_lds)::value;
        u32 pos = base;
#pragma unroll
        for (u32 i = 0; i < ROWS; i++) {
            const u64 some = __ballot(cnt[i] != 0u);
            if (cnt[i]) {
                const u32 at = pos + __builtin_amdgcn_mbcnt_hi((u32)(some >> 32), __builtin_amdgcn_mbcnt_lo((u32)some, 0u));
                xq[at] = slot_value(slot_in_value_order((wave * ROWS + i) * 64u + lane), P);
                xw[at].x = (double)cnt[i]; // the count, replaced by the weight below
            }
            pos += (u32)__popcll(some);
        }
        if (m == 0u) { // (cannot happen: at least one value lies between the thresholds)
            if (tid == 0) {
                P.info[t].n_buckets = 0u;
                P.info[t].rounds = 0u;
            }
            return;
        }
        double *uni = cen; // the draws' random numbers (the sorted centres take this array afterwards)
        if (tid < 256u) uni[tid] = P.uniforms[(size_t)t * 256 + tid];
        __syncthreads();
        // ---- sample weights (Algorithm 2): sigma * C / max C + (1 - sigma) * |X| / max |X| ----
        const double x_first = fabs(xq[0]), x_last = fabs(xq[m - 1u]);
        const double mx = x_first > x_last ? x_first : x_last;
        const double one_minus = sub_rn(1.0, P.sigma);
        for (u32 i = tid; i < m; i += KM_BLOCK) {
            const double c_hat = div_rn(xw[i].x, (double)maxc);
            const double x_hat = mx > 0.0 ? div_rn(fabs(xq[i]), mx) : 0.0;
            xw[i].x = add_rn(mul_rn(P.sigma, c_hat), mul_rn(one_minus, x_hat));
        }
        __syncthreads();
        // ---- weighted K-Means++ draws ----
        if (!LDS || m > 24u * 64u)
            draw_centres_long(xq, xw, m, K, uni, craw, s_red, s_pick, s_last, s_chosen);
        else if (wave == 0u) {
            if (m <= 4u * 64u)
                draw_centres<4>(xq, xw, m, K, uni, craw);
            else if (m <= 6u * 64u)
                draw_centres<6>(xq, xw, m, K, uni, craw);
            else if (m <= 8u * 64u)
                draw_centres<8>(xq, xw, m, K, uni, craw);
            else if (m <= 12u * 64u)
                draw_centres<12>(xq, xw, m, K, uni, craw);
            else if (m <= 16u * 64u)
                draw_centres<16>(xq, xw, m, K, uni, craw);
            else
                draw_centres<24>(xq, xw, m, K, uni, craw);
        }
        __syncthreads();
        // ---- every set's first centres, sorted, by a thread per centre (the random numbers in their place have been
        // used); the products (the distances are done with) ----
        auto each_centre = [&](auto &&f) { // f(set, number of its centres, centre)
            for (u32 j = tid; j < (P.multi ? 508u : K); j += KM_BLOCK) {
                const u32 set = P.multi ? 29u - (u32)__builtin_clz(j + 4u) : 0u; // (centres of narrower sets before: (4 << set) - 4)
                f(set, P.multi ? 4u << set : K, P.multi ? j + 4u - (4u << set) : j);
            }
        };
        each_centre([&](u32 set, u32 Kb, u32 k) {
            const double c_raw = craw[k];
            u32 rank = 0u;
            for (u32 i = 0; i < Kb; i++) {
                const double y = craw[i];
                rank += (y < c_raw || (y == c_raw && i < k)) ? 1u : 0u;
            }
            cen[(P.multi ? (4u << set) - 4u : 0u) + rank] = c_raw;
        });
        for (u32 i = tid; i < m; i += KM_BLOCK) xw[i].y = mul_rn(xw[i].x, xq[i]);
        __syncthreads();
        // ---- Lloyd rounds, a wave per set ----
        static_assert(SK_SETS <= WAVES, "a wave per set");
        if (wave < n_sets) {
            const u32 Ks = P.multi ? 4u << wave : K;
            double *c_set = cen + (P.multi ? Ks - 4u : 0u);
            const u32 r = Ks <= 64u    ? lloyd_rounds<1>(xq, xw, m, Ks, c_set, P.max_iter)
                          : Ks <= 128u ? lloyd_rounds<2>(xq, xw, m, Ks, c_set, P.max_iter)
                                       : lloyd_rounds<4>(xq, xw, m, Ks, c_set, P.max_iter);
            if (lane == 0u) s_rounds[wave] = r;
        }
        // ---- codebooks and boundaries ----
        u32 *ak = P.alt_key + (size_t)t * n_sets * 256;
        float *acb = P.alt_cb + (size_t)t * n_sets * 256;
        for (u32 i = tid; i < n_sets * 256u; i += KM_BLOCK) {
            ak[i] = 0u;
            acb[i] = 0.0f;
        }
        __syncthreads();
        each_centre([&](u32 set, u32 Kb, u32 k) {
            const double *c_set = cen + (P.multi ? Kb - 4u : 0u);
            acb[set * 256u + k] = __double2float_rn(c_set[k]);
            if (k + 1u < Kb) {
                const double lo = (double)__double2float_rn(c_set[k]), hi = (double)__double2float_rn(c_set[k + 1u]);
                const double mid = mul_rn(add_rn(lo, hi), 0.5);
                // a value goes to the upper centre when it lies strictly above the midpoint: the
                // boundary is the smallest fp32 number above it
                ak[set * 256u + (k + 1u) * (256u / Kb) - 1u] = key_of_float(__double2float_rd(mid)) + 1u;
            }
        });
        if (P.multi && tid < n_sets) P.set_rounds[(size_t)t * SK_SETS + tid] = s_rounds[tid];
        if (tid == 0) { // (of the widest set)
            P.info[t].n_buckets = m;
            P.info[t].rounds = s_rounds[n_sets - 1u];
        }
    };
    if (m <= (u32)SK_LDS)
        cluster(l_x, l_w, std::true_type());
    else
        cluster(gptr(P.xq) + (size_t)t * SK_HIST, gptr((d2 *)P.wd) + (size_t)t * SK_HIST, std::false_type());
}

// ------------------------------------------------------------------------------------------
// exact error of every set of centres (Sec. 5 restricted to the number of bins)
// ------------------------------------------------------------------------------------------
// All boundaries of a tensor's SK_SETS sets, sorted, cut the key axis into at most SK_EDGES + 1
// slots; a slot lies inside one cluster of every set, so count and sum per slot give the error of
// every set: (sum_all - sum_protected) x^2 - sum over slots of (2 c sx - n c^2), c the slot's centre.
__device__ __forceinline__ u32 n_boundaries_before(u32 set) { return (4u << set) - 4u - set; } // sum of 2^b - 1, b = 2 .. set + 1

__global__ __launch_bounds__(BLOCK) void k_sketch_score(const TDesc *__restrict__ td, int nT,
                                                        const u64 *__restrict__ wg_tile0,
                                                        const GridDesc *__restrict__ gd,
                                                        const SketchDesc *__restrict__ sd,
                                                        SketchParams P, Bufs B)
{
    // The slot of a key = the boundaries at or below it.  The search's equal-population bins (up to
    // 32768 per tensor, found through the key-prefix table) are far finer than the 502 slots: a table
    // gives the slot of every bin that holds no boundary, and for the few bins that do, the first
    // boundary to compare the key with.
    struct ScoreShared {
        u32 T[COARSE];                        // key prefix -> bins
        u16 stab[L2_BINS];                    // slot, or 0x8000 | boundaries below the bin
        u32 raw[SK_EDGES], edge[SK_EDGES + 1];
        // (four copies of the slot moments, one per lane modulo 4: the slots are few and the lanes
        // of a wave that hit the same address are served one after the other)
        u32 cnt[SK_COPIES * SK_SLOTS];
        double sx[SK_COPIES * SK_SLOTS];
    };
    __shared__ ScoreShared sh;
    const u32 tid = threadIdx.x, copy = (tid & (u32)(SK_COPIES - 1)) * (u32)SK_SLOTS;
    const u64 tile_lo = wg_tile0[blockIdx.x], tile_hi = wg_tile0[blockIdx.x + 1];
    if (tile_lo >= tile_hi) return;
    int t = find_tensor(td, nT, tile_lo);
    u64 tile = tile_lo;
    while (tile < tile_hi) {
        const TDesc d = td[t];
        const u64 n_tiles_t = (d.n + TILE - 1) / TILE;
        const u64 t_end = d.tile0 + n_tiles_t;
        const u64 stop = t_end < tile_hi ? t_end : tile_hi;
        const SketchDesc s = sd[t];
        if (!s.active) {
            tile = stop;
            t++;
            continue;
        }
        const TState *st = B.ts + t;
        const u32 pair = gd->cfg_pair[s.cfg];
        const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + gd->pair_o[pair]];
        const u32 nb2 = st->nb2;
        __syncthreads();
        for (u32 i = tid; i < (u32)COARSE; i += BLOCK) sh.T[i] = entry_for_u16(B.table2[(size_t)t * COARSE + i]);
        if (tid < (u32)SK_EDGES) { // boundary j of set b sits at ((j + 1) << (8 - bits)) - 1 of its row
            u32 set = 0u;
            while (set + 1u < (u32)SK_SETS && tid >= n_boundaries_before(set + 1u)) set++;
            const u32 j = tid - n_boundaries_before(set), bits = 2u + set;
            sh.raw[tid] = P.alt_key[((size_t)t * SK_SETS + set) * 256 + (((j + 1u) << (8u - bits)) - 1u)];
        }
        for (u32 i = tid; i < (u32)(SK_COPIES * SK_SLOTS); i += BLOCK) {
            sh.cnt[i] = 0u;
            sh.sx[i] = 0.0;
        }
        __syncthreads();
        if (tid < (u32)SK_EDGES) { // sort by counting the smaller ones
            const u32 x = sh.raw[tid];
            u32 r = 0u;
            for (u32 i = 0; i < (u32)SK_EDGES; i++) {
                const u32 y = sh.raw[i];
                r += (y < x || (y == x && i < tid)) ? 1u : 0u;
            }
            sh.edge[r] = x;
        }
        if (tid == 0) sh.edge[SK_EDGES] = 0xFFFFFFFFu;
        __syncthreads();
        for (u32 b = tid; b < nb2; b += BLOCK) { // slot of every bin, or its first boundary
            u32 lo = 0u, hi = COARSE - 1u; // key prefix of the bin: last one that starts at or below it
            while (lo < hi) {
                const u32 mid = (lo + hi + 1u) >> 1;
                if ((sh.T[mid] >> 6) <= b)
                    lo = mid;
                else
                    hi = mid - 1u;
            }
            const u32 e = sh.T[lo], dd = e & 31u, sub = b - (e >> 6);
            const u32 first = (lo << COARSE_SHIFT) | (sub << (COARSE_SHIFT - dd));
            const u32 last = first + ((1u << (COARSE_SHIFT - dd)) - 1u);
            u32 below = 0u, upto = 0u; // boundaries < first, boundaries <= last
#pragma unroll
            for (u32 step = 256u; step > 0u; step >>= 1) {
                if (below + step <= (u32)SK_EDGES && sh.edge[below + step - 1u] < first) below += step;
                if (upto + step <= (u32)SK_EDGES && sh.edge[upto + step - 1u] <= last) upto += step;
            }
            sh.stab[b] = (u16)((below == upto) ? below : (0x8000u | below));
        }
        __syncthreads();
        for (; tile < stop; tile++) {
            const u64 e0 = (tile - d.tile0) * (u64)TILE;
            const u64 rem = d.n - e0;
            const u32 c = tile_len(rem, (u32)TILE);
            float v[16];
            const u32 mask = load_tile(d, e0, c, v);
#pragma unroll 4
            for (int i = 0; i < 16; i++) {
                const u32 key = key_of_float(v[i]);
                const u32 mag = mag_of_key(key);
                if (!((mask >> i) & 1u) || mag < tau_p || mag > tau_o) continue;
                u32 slot = lookup_u16(sh.stab, key, sh.T[key >> COARSE_SHIFT]);
                if (slot & 0x8000u) {
                    slot &= 0x7fffu;
                    while (sh.edge[slot] <= key) slot++; // (the list ends with 0xFFFFFFFF, above every finite key)
                }
                atomicAdd(&sh.cnt[copy + slot], 1u);
                atomicAdd(&sh.sx[copy + slot], (double)v[i]);
            }
        }
        __syncthreads();
        // this unit's part of the tensor's slot moments
        u32 *gc = P.slot_cnt + (size_t)t * SK_SLOTS;
        double *gx = P.slot_sx + (size_t)t * SK_SLOTS;
        for (u32 i = tid; i <= (u32)SK_EDGES; i += BLOCK) {
            u32 n = 0u;
            double sum = 0.0;
            for (u32 k = 0; k < (u32)SK_COPIES; k++) {
                n += sh.cnt[k * SK_SLOTS + i];
                sum += sh.sx[k * SK_SLOTS + i];
            }
            if (n) {
                atomicAdd(&gc[i], n);
                atomicAdd(&gx[i], sum);
            }
        }
        if (tid < (u32)SK_EDGES) P.slot_edge[(size_t)t * SK_SLOTS + tid] = sh.edge[tid]; // (the same from every unit)
        t++;
    }
}

// (bound by latency: the slots' shares by all threads, then added in slot order by a thread per set from LDS; a
// thread per set that walked the slots in device memory took 0.25 ms, 0.02 ms so)
// per tensor: error of every set, the fewest bits within eps, and that set's keys and centres
// where the quantizer looks for them
__global__ __launch_bounds__(256) void k_sketch_choose(const TDesc *__restrict__ td,
                                                       const u32 *__restrict__ t_fu_off,
                                                       const GridDesc *__restrict__ gd,
                                                       const SketchDesc *__restrict__ sd,
                                                       SketchParams P, Bufs B)
{
    constexpr int N = SK_EDGES + 1;
    __shared__ double s_sse[SK_SETS], s_sq[256], s_prot[256];
    __shared__ double term[SK_SETS][N]; // what a slot takes off a set's error
    __shared__ u32 top[SK_SETS][256];   // largest of a set's boundaries up to each
    __shared__ u32 s_best;
    const int t = blockIdx.x;
    const SketchDesc s = sd[t];
    if (!s.active) return;
    const u32 tid = threadIdx.x;
    const TState *st = B.ts + t;
    const u32 pair = gd->cfg_pair[s.cfg];
    // sum_pruned x^2 + sum_quantized (x - c)^2 = (sum_all - sum_protected) x^2 - sum_quantized (2 c x - c^2)
    double sumsq = st->sumsq, protsq = st->thr_sumsq[gd->n_p + gd->pair_o[pair]];
    if (P.light) { // no scoring kernel has added the units' parts up
        sumsq = 0.0;
        protsq = 0.0;
        for (u32 u0 = t_fu_off[t], u1 = t_fu_off[t + 1]; u0 < u1; u0 += 256u) { // 256 read together, added in order
            const u32 k = u1 - u0 < 256u ? u1 - u0 : 256u;
            if (tid < k) {
                s_sq[tid] = B.sq_part[(size_t)(u0 + tid) * SQ_STRIDE];
                s_prot[tid] = B.sq_part[(size_t)(u0 + tid) * SQ_STRIDE + 1u + gd->pair_o[pair]];
            }
            __syncthreads();
            for (u32 i = 0; i < k; i++) {
                sumsq += s_sq[i];
                protsq += s_prot[i];
            }
            __syncthreads();
        }
    }
    const double not_protected = sumsq - protsq;
    const u32 *gc = P.slot_cnt + (size_t)t * SK_SLOTS;
    const double *gx = P.slot_sx + (size_t)t * SK_SLOTS;
    const u32 *edge = P.slot_edge + (size_t)t * SK_SLOTS;
    const u32 lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (u32 set = wave; set < (u32)SK_SETS; set += 4u) { // a wave per set
        const u32 Kb = 4u << set, sh = 6u - set;
        const u32 *ak = P.alt_key + ((size_t)t * SK_SETS + set) * 256;
        u32 before = 0u;
        for (u32 k = lane; k - lane < Kb; k += 64u) {
            const u32 y = wave_incl_max(k > 0u && k < Kb ? ak[(k << sh) - 1u] : 0u);
            const u32 m = y > before ? y : before;
            if (k < Kb) top[set][k] = m;
            before = (u32)__builtin_amdgcn_readlane((int)m, 63);
        }
    }
    __syncthreads();
    for (u32 slot = tid; slot < (u32)N; slot += 256u) {
        const u32 n = gc[slot], first = slot ? edge[slot - 1u] : 0u; // the slot starts at edge[slot - 1]
        const double x = gx[slot];
#pragma unroll
        for (u32 set = 0; set < (u32)SK_SETS; set++) {
            const float *acb = P.alt_cb + ((size_t)t * SK_SETS + set) * 256;
            u32 cluster = 0u; // of the slot: boundaries of this set at or below the slot's keys
            if (slot)
#pragma unroll
                for (u32 step = 2u << set; step > 0u; step >>= 1)
                    if (top[set][cluster + step] <= first) cluster += step;
            const double c = (double)acb[cluster];
            term[set][slot] = n ? 2.0 * c * x - (double)n * c * c : 0.0;
        }
    }
    __syncthreads();
    if (tid < (u32)SK_SETS) {
        double gain = 0.0;
#pragma unroll 8
        for (int slot = 0; slot < N; slot++) gain += term[tid][slot];
        const double sse = not_protected - gain;
        s_sse[tid] = sse > 0.0 ? sse : 0.0;
    }
    __syncthreads();
    if (tid == 0) {
        const double bound = P.eps * sumsq;
        u32 best = SK_SETS - 1u, feasible = 0u;
        for (u32 set = 0; set < (u32)SK_SETS; set++)
            if (s_sse[set] <= bound) {
                best = set;
                feasible = 1u;
                break;
            }
        s_best = best;
        SketchChoice r;
        for (u32 set = 0; set < (u32)SK_SETS; set++) {
            r.sse[set] = s_sse[set];
            r.rounds[set] = P.set_rounds[(size_t)t * SK_SETS + set];
        }
        r.sumsq = sumsq;
        r.best_bits = 2u + best;
        r.feasible = feasible;
        P.choice[t] = r;
    }
    __syncthreads();
    const u32 best = s_best;
    P.final_key[(size_t)t * 256 + tid] = P.alt_key[((size_t)t * SK_SETS + best) * 256 + tid];
    P.final_cb[(size_t)t * 256 + tid] = P.alt_cb[((size_t)t * SK_SETS + best) * 256 + tid];
}

// ------------------------------------------------------------------------------------------
// The sketch as the quantile estimator (Sec. 4.3, Algorithm 1): one sweep counts the magnitudes of
// a tensor per bucket; the estimate of the magnitude of a rank is the value of the bucket in which
// the running count passes the rank (relative error alpha).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_sketch_maghist(const MagDesc *__restrict__ md, int nT, u64 n_chunks,
                                                          const u32 *__restrict__ gcell,
                                                          const u32 *__restrict__ tops, u32 n_idx,
                                                          u32 *__restrict__ hist, u32 *__restrict__ nonfinite)
{
    __shared__ u32 smem[SK_CELLS + SK_MAG_HIST];
    u32 *cell = smem, *h = smem + SK_CELLS;
    const u32 tid = threadIdx.x;
    // every workgroup takes an equal share of the chunks, in order; its counts go to a tensor's
    // histogram when the share moves on to the next tensor
    const u64 c_lo = n_chunks * (u64)blockIdx.x / gridDim.x, c_hi = n_chunks * ((u64)blockIdx.x + 1u) / gridDim.x;
    if (c_lo >= c_hi) return;
    int t = 0, hi = nT - 1; // last tensor whose first chunk is <= c_lo
    while (t < hi) {
        const int mid = (t + hi + 1) >> 1;
        if (md[mid].chunk0 <= c_lo)
            t = mid;
        else
            hi = mid - 1;
    }
    for (int i = tid; i < SK_CELLS; i += BLOCK) cell[i] = gcell[i];
    for (int i = tid; i < SK_MAG_HIST; i += BLOCK) h[i] = 0u;
    __syncthreads();
    bool bad = false;
    u64 c = c_lo;
    while (c < c_hi) {
        const MagDesc d = md[t];
        const u64 t_end = d.chunk0 + (d.n + SK_MAG_CHUNK - 1) / SK_MAG_CHUNK;
        const u64 stop = t_end < c_hi ? t_end : c_hi;
        for (; c < stop; c++) {
            TDesc td1; // (for the tile loader of the sweeps)
            td1.data = d.x;
            td1.n = d.n;
#pragma unroll 1
            for (u32 tl = 0; tl < (u32)SK_MAG_CHUNK / TILE; tl++) {
                const u64 e0 = (c - d.chunk0) * (u64)SK_MAG_CHUNK + (u64)tl * TILE;
                if (e0 >= d.n) break;
                const u64 rem = d.n - e0;
                const u32 cnt = tile_len(rem, (u32)TILE);
                float v[16];
                const u32 mask = load_tile(td1, e0, cnt, v);
#pragma unroll
                for (int j = 0; j < 16; j++) {
                    if (!((mask >> j) & 1u)) continue; // past the end
                    const u32 mag = __float_as_uint(v[j]) & 0x7fffffffu;
                    if (mag >= 0x7f800000u) {
                        bad = true;
                    } else if (mag >= 0x00800000u) {
                        // entry = first bucket of the cell << 17 | (2^17 - 1 - low bits of that bucket's
                        // largest magnitude): the sum carries into the bucket field when the magnitude
                        // lies above it
                        atomicAdd(&h[1u + ((cell[mag >> 17] + (mag & 0x1FFFFu)) >> 17)], 1u);
                    } else if (mag == 0u) {
                        atomicAdd(&h[0], 1u);
                    } else { // a denormal: first bucket whose largest magnitude reaches it
                        u32 a = 0u, b = n_idx - 1u;
                        while (a < b) {
                            const u32 mid = (a + b) >> 1;
                            if (tops[mid] >= mag)
                                b = mid;
                            else
                                a = mid + 1u;
                        }
                        atomicAdd(&h[1u + a], 1u);
                    }
                }
            }
        }
        __syncthreads();
        u32 *gh = hist + (size_t)t * SK_MAG_HIST;
        for (int i = tid; i < SK_MAG_HIST; i += BLOCK) {
            const u32 v = h[i];
            if (v) {
                atomicAdd(&gh[i], v);
                h[i] = 0u;
            }
        }
        __syncthreads();
        t++;
    }
    if (bad) atomicOr(nonfinite, 1u);
}

__global__ __launch_bounds__(256) void k_sketch_quantile_pick(const MagDesc *__restrict__ md,
                                                              const u32 *__restrict__ hist,
                                                              const double *__restrict__ rep, u32 n_idx,
                                                              const u64 *__restrict__ ranks, u32 n_q,
                                                              double *__restrict__ est)
{
    __shared__ u32 cum[SK_MAG_HIST + 1]; // keys in the buckets before each one (n < 2^32)
    const int t = blockIdx.x;
    const u32 *gh = hist + (size_t)t * SK_MAG_HIST;
    if (threadIdx.x == 0) {
        u32 run = 0u;
        for (u32 i = 0; i <= n_idx; i++) {
            cum[i] = run;
            run += gh[i];
        }
        cum[n_idx + 1u] = run;
    }
    __syncthreads();
    for (u32 k = threadIdx.x; k < n_q; k += 256u) {
        const u64 rank = ranks[(size_t)t * n_q + k];
        u32 lo = 0u, hi = n_idx; // first bucket (in magnitude order, zeros first) whose running count passes the rank
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if ((u64)cum[mid + 1u] > rank)
                hi = mid;
            else
                lo = mid + 1u;
        }
        est[(size_t)t * n_q + k] = lo == 0u ? 0.0 : rep[lo - 1u];
    }
    (void)md;
}

hipError_t launch_sketch_quantiles(const MagDesc *md, int nT, u64 n_chunks, int n_wg, const u32 *cell, const u32 *tops,
                                   const double *rep, u32 n_idx, u32 *hist, u32 *nonfinite,
                                   const u64 *ranks, u32 n_q, double *est, hipStream_t s)
{
    const unsigned grid = (unsigned)(n_chunks < (u64)n_wg ? n_chunks : (u64)n_wg);
    PROF("k_sketch_maghist", s, k_sketch_maghist<<<grid, BLOCK, 0, s>>>(md, nT, n_chunks, cell, tops, n_idx, hist, nonfinite));
    PROF("k_sketch_quantile_pick", s, k_sketch_quantile_pick<<<nT, 256, 0, s>>>(md, hist, rep, n_idx, ranks, n_q, est));
    return hipGetLastError();
}

hipError_t launch_sketch(const Batch &bt, const SketchDesc *sd, const SketchParams &P, hipStream_t s)
{
    if (P.light)
        PROF("k_sketch_hist", s, k_sketch_hist<true><<<bt.n_wg, BLOCK, 0, s>>>(bt.td, bt.nT, bt.wg_tile0, bt.wg_fu0,
                                                                              bt.gd, sd, P, bt.bufs));
    else
        PROF("k_sketch_hist", s, k_sketch_hist<false><<<bt.n_wg_all, BLOCK, 0, s>>>(bt.td, bt.nT, bt.wg_tile0_all, nullptr,
                                                                               bt.gd, sd, P, bt.bufs));
    PROF("k_sketch_kmeans", s, k_sketch_kmeans<<<bt.nT, KM_BLOCK, 0, s>>>(bt.gd, sd, P));
    if (P.multi) {
        PROF("k_sketch_score", s,
             k_sketch_score<<<bt.n_wg_all, BLOCK, 0, s>>>(bt.td, bt.nT, bt.wg_tile0_all, bt.gd, sd, P, bt.bufs));
        PROF("k_sketch_choose", s,
             k_sketch_choose<<<bt.nT, 256, 0, s>>>(bt.td, bt.t_fu_off, bt.gd, sd, P, bt.bufs));
    }
    return hipGetLastError();
}

} // namespace inshr
