// Scoring of every grid configuration from one pass over the data (Sec. 5: the search evaluates a
// grid of configurations; here all of them share the sweeps).
//
// All boundaries and class edges of all (prune, protect) pairs form one list of "edges" ordered by
// key; slot s holds the keys with exactly s edges at or below them, and a slot fixes class and bin
// under every configuration, because the boundaries for fewer bits are a subset of those for
// 8 bits (floor(j*M/2^b) = floor(j*2^(8-b)*M/2^8)).  The order of the list is known before any
// boundary key is: a boundary is the key of a given rank, a class edge has a known number of keys
// below it, and rank order is key order (a class edge goes before a boundary of equal rank).
// Per slot the sweeps provide (count, sum x); a small kernel turns slots into per-bin centres
// (Sec. 4.4, one centre update) and errors:
//   sse = sum_all x^2 - sum_protected x^2 - sum_bins (2 c S - n c^2)        (c rounded to fp32)
// (a pruned element's error x^2 is its own share of sum_all x^2).
#include "inshr_launch.h"

namespace inshr {

// ------------------------------------------------------------------------------------------
// edge order; for every bin without an edge its slot, and the keys per slot in such bins
// ------------------------------------------------------------------------------------------
// One workgroup per tensor, bound by the latency of its steps.  The edges are put in order by a
// radix sort of their ranks (a bitonic sort of 4096 words, lane exchanges and all, took two thirds of
// the kernel), slots and sub-slots of the bins come from scans over the bins (two bisections per bin
// took the rest): 1 Mi values, 6 pairs: 200 -> 40 us.
constexpr int EROWS = MAX_EDGES / BLOCK; // edges per thread
struct EdgeShared {
    u32 below[MAX_EDGES];                // sort: keys below the edge; afterwards the bin of each edge, in order
    u16 item[MAX_EDGES];                 // sort: edge item; afterwards the group of each edge's bin
    u32 wcount[(BLOCK / 64) * 256];      // sort: digit counters
    u16 mark[L2_BINS + 64];              // per bin: edges in lower bins + 1 where that changes | 0x8000 where
                                         // the exponent changes
    u32 segc[MAX_EDGES];                 // keys per slot in bins without an edge
    u32 subc[MAX_SUB];                   // ... per sub-slot
};

template <bool ORDERED>
__global__ __launch_bounds__(BLOCK) void k_edges(const TDesc *__restrict__ td,
                                                 const GridDesc *__restrict__ gd, Bufs B, u32 *__restrict__ grp_list,
                                                 u32 *__restrict__ n_grp_total)
{
    extern __shared__ double sm_edges[];
    EdgeShared &sh = *reinterpret_cast<EdgeShared *>(sm_edges);
    __shared__ u32 ckey[MAX_PAIRS * 4], wsum[4], s_at, s_err;
    __shared__ u32 w_E[BLOCK / 64], w_X[BLOCK / 64], w_P[BLOCK / 64];

    const int t = blockIdx.x;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TState *st = B.ts + t;
    if (B.view[t] == VIEW_NONE) return;
    const View vw = view_of(gd, B.view[t]);
    const u64 n = td[t].n, n_neg = st->n_neg;
    const u32 n_p = gd->n_p;
    // edge items: pair q has the boundaries q * EPP + (index) and the class edges q * EPP + NBT ..
    // NBT + 3; the list holds n_e = (pairs in view) * (n_bnd + 4) of them
    const u32 n_bnd = vw.n_bnd, n_c = 4u * vw.n_pairs;
    const u32 n_e = vw.n_pairs * n_bnd + n_c;
    const u32 nb2 = st->nb2, zbin = st->zbin;
    const u32 G = st->pool_overflow ? 0u : st->n_groups; // (overflow: nothing valid to sort)
    const u32 *tb = B.tgt_bin + (size_t)t * TGT_STRIDE;
    const u32 *trank = B.tgt_rank + (size_t)t * TGT_STRIDE;
    const u32 *tab = B.table2 + (size_t)t * COARSE;
    const u32 *binfo = B.binfo + (size_t)t * L2_BINS;
    const u32 *h2 = B.hist2 + (size_t)t * L2_BINS;
    const u16 *gtab = B.bin_group + (size_t)t * L2_BINS;
    u32 *elo = B.grp_elo + (size_t)t * MAX_GROUPS;
    u32 *ehi = B.grp_ehi + (size_t)t * MAX_GROUPS;
    u32 *sub_code = B.sub_code + (size_t)t * MAX_SUB;

    if (tid < n_c)
        ckey[tid] = class_edge_key(tid & 3u, st->thr_mag[gd->pair_p[vw.q0 + (tid >> 2)]],
                                   st->thr_mag[n_p + gd->pair_o[vw.q0 + (tid >> 2)]]);
    if (tid == 0u) {
        s_err = 0u;
        if (G) s_at = atomicAdd(n_grp_total, G);
    }
    for (u32 g = tid; g < st->n_groups; g += BLOCK) {
        elo[g] = 0xFFFFFFFFu;
        ehi[g] = 0u;
    }
    for (u32 i = tid; i < (L2_BINS + 64u) / 2u; i += BLOCK) reinterpret_cast<u32 *>(sh.mark)[i] = 0u;
    for (u32 i = tid; i < (u32)MAX_EDGES; i += BLOCK) sh.segc[i] = 0u;
    for (u32 i = tid; i < (u32)MAX_SUB; i += BLOCK) {
        sh.subc[i] = 0u;
        sub_code[i] = 0xFFFFFFFFu; // no bin has this sub-slot
    }
    __syncthreads();
    // work list of the group sort: (tensor, group), in any order
    for (u32 g = tid; g < G; g += BLOCK) grp_list[s_at + g] = ((u32)t << 13) | g;
    // The class edges go first, in key order (several may have the same number of keys below them and
    // still lie in different bins), then the boundaries; a stable sort by the number of keys below
    // keeps a class edge before a boundary of equal rank.
    if (tid < n_c) {
        const u32 q = vw.q0 + (tid >> 2), key = ckey[tid];
        u32 order = 0u;
        for (u32 j = 0; j < n_c; j++) order += (ckey[j] < key || (ckey[j] == key && j < tid)) ? 1u : 0u;
        u64 below;
        switch (tid & 3u) {
        case 0: below = st->pair_An[q]; break;                 // keys < first quantized negative
        case 1: below = n_neg - st->pair_Pn[q]; break;         // keys < first pruned
        case 2: below = n_neg + st->pair_Pp[q]; break;         // keys < first quantized positive
        default: below = n - st->pair_Ap[q]; break;            // keys < first protected positive
        }
        sh.below[order] = (u32)below;
        sh.item[order] = (u16)(q * EPP + (u32)NBT + (tid & 3u));
    }
    for (u32 w = tid; w < vw.n_pairs * n_bnd; w += BLOCK) {
        const u32 q = vw.q0 + w / n_bnd, e = view_bnd(gd, vw, w % n_bnd);
        sh.below[n_c + w] = trank[q * NBT + e];
        sh.item[n_c + w] = (u16)(q * EPP + e);
    }
    __syncthreads();
    {
        const u32 n_bits = 64u - (u32)__clzll((long long)n); // (keys below an edge: at most n < 2^32)
        const u32 n_pass = (n_bits + 7u) >> 3;
        const u32 dwidth = (n_bits + n_pass - 1u) / n_pass, dmask = (1u << dwidth) - 1u;
        const u32 rows = (n_e + BLOCK - 1u) / BLOCK, chunk = rows * 64u;
        u32 *wcnt = sh.wcount + wave * 256u;
        for (u32 pass = 0; pass < n_pass; pass++) {
            const u32 shift = pass * dwidth;
            u32 kreg[EROWS], rreg[EROWS];
            u16 ireg[EROWS];
            for (u32 i = lane; i < 256u; i += 64u) wcnt[i] = 0u; // (a wave's own row: its operations stay in order)
#pragma unroll
            for (u32 r = 0; r < (u32)EROWS; r++) {
                kreg[r] = rreg[r] = 0u;
                ireg[r] = 0;
                if (r < rows) {
                    const u32 i = wave * chunk + r * 64u + lane;
                    const bool valid = i < n_e;
                    if (valid) {
                        kreg[r] = sh.below[i];
                        ireg[r] = sh.item[i];
                    }
                    rreg[r] = digit_rank<ORDERED>(wcnt, (kreg[r] >> shift) & dmask, valid);
                }
            }
            __syncthreads();
            u32 tot = 0u, excl = 0u, cw[BLOCK / 64];
            if (tid < 256u) {
#pragma unroll
                for (u32 w = 0; w < (u32)(BLOCK / 64); w++) cw[w] = sh.wcount[w * 256u + tid];
#pragma unroll
                for (u32 w = 0; w < (u32)(BLOCK / 64); w++) tot += cw[w];
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
                for (u32 w = 0; w < (u32)(BLOCK / 64); w++) {
                    sh.wcount[w * 256u + tid] = run;
                    run += cw[w];
                }
            }
            __syncthreads();
#pragma unroll
            for (u32 r = 0; r < (u32)EROWS; r++) { // (everything is in registers: the arrays are overwritten)
                const u32 i = wave * chunk + r * 64u + lane;
                if (r < rows && i < n_e) {
                    const u32 at = wcnt[(kreg[r] >> shift) & dmask] + rreg[r];
                    sh.below[at] = kreg[r];
                    sh.item[at] = ireg[r];
                }
            }
            __syncthreads();
        }
    }
    u32 *E = B.edges + (size_t)t * MAX_EDGES;
    u32 *eb = B.edge_bin + (size_t)t * MAX_EDGES;
    u16 *ei = B.edge_item + (size_t)t * MAX_EDGES;
    u16 *pe = B.pair_eidx + (size_t)t * MAX_PAIRS * EIDX_STRIDE;
    for (u32 pos = tid; pos < n_e; pos += BLOCK) { // (each thread replaces the entries it has read)
        const u32 item = sh.item[pos];
        const u32 q = item / EPP, e = item % EPP;
        u32 key = 0u, bin; // (a boundary's key is found later, from the gathered keys)
        if (e < (u32)NBT) {
            bin = tb[q * NBT + e];
            if (bin == RESOLVED) {
                bin = zbin;
                key = ZERO_KEY;
            }
        } else {
            key = ckey[(q - vw.q0) * 4u + (e - NBT)];
            bin = l2_bin(key, tab[key >> COARSE_SHIFT]);
        }
        E[pos] = key;
        eb[pos] = bin;
        ei[pos] = (u16)item;
        pe[q * EIDX_STRIDE + e] = (u16)pos;
        sh.below[pos] = bin;
        sh.item[pos] = bin < nb2 ? gtab[bin] : (u16)0xFFFFu;
    }
    // where the sign and exponent of the bins change (a table prefix is sign, exponent and three
    // mantissa bits; every prefix has a bin of its own)
    for (u32 k = 1u + tid; k < 512u; k += BLOCK) sh.mark[(tab[8u * k] >> 5) & 0x7fffu] = 0x8000u;
    __syncthreads();
    for (u32 pos = tid; pos < n_e; pos += BLOCK) {
        const u32 bin = sh.below[pos], g = sh.item[pos];
        const bool last = pos + 1u == n_e;
        const u32 nbin = last ? 0xFFFFFFFFu : sh.below[pos + 1u];
        if (nbin < bin || g >= (u32)MAX_GROUPS) s_err = 1u;
        // the bins behind this one have pos + 1 edges in lower bins
        if (nbin != bin && bin + 1u < nb2) sh.mark[bin + 1u] = (u16)((sh.mark[bin + 1u] & 0x8000u) | (pos + 1u));
        // groups are runs of bins, so their edges are runs of the list
        if (g < (u32)MAX_GROUPS) {
            if (pos == 0u || sh.item[pos - 1u] != g) elo[g] = pos;
            if (last || sh.item[pos + 1u] != g) ehi[g] = pos + 1u;
        }
    }
    __syncthreads();
    // Slot and sub-slot of every bin.  A bin without an edge lies inside one slot; sweep 3 adds the
    // mantissas of its keys as integers, which is exact and linear in the value only among keys of
    // one sign and exponent, so a slot is cut further wherever the exponent changes: sub-slot =
    // (edges in lower bins) + (key >> 23 of the bin).  Both terms grow with the bin, so the sum
    // names the pair; it stays below n_e + 512.
    // Every wave walks a run of bins in rows of 64: edges in lower bins = largest mark so far,
    // exponent = exponent marks so far, P = keys of the bins without an edge so far.  Where a slot
    // (a sub-slot) begins, P is taken from its count and added to the one before.
    constexpr u32 ROWS = L2_BINS / BLOCK;
    const u32 rows = (nb2 + BLOCK - 1u) / BLOCK;
    u32 pop[ROWS], actm = 0u; // keys of this lane's bins without an edge; its bins with one
    u32 tE = 0u, tX = 0u, tP = 0u;
#pragma unroll
    for (u32 r = 0; r < ROWS; r++) {
        pop[r] = 0u;
        const u32 b = (wave * rows + r) * 64u + lane;
        if (r < rows && b < nb2) {
            const bool act = binfo[b] != INACTIVE;
            const u32 c = h2[b];
            pop[r] = act ? 0u : c;
            actm |= (act ? 1u : 0u) << r;
        }
    }
    for (u32 r = 0; r < rows; r++) {
        const u32 b = (wave * rows + r) * 64u + lane;
        const u32 m = b < nb2 ? (u32)sh.mark[b] : 0u;
        tE = max(tE, m & 0x7fffu);
        tX += (u32)__popcll(__ballot(m >> 15));
    }
#pragma unroll
    for (u32 r = 0; r < ROWS; r++) tP += pop[r];
    tE = wave_incl_max(tE);
    tP = wave_incl_scan(tP);
    if (lane == 63u) {
        w_E[wave] = tE;
        w_X[wave] = tX;
        w_P[wave] = tP;
    }
    __syncthreads();
    u32 cE = 0u, cX = 0u, cP = 0u; // up to the bin before the row's first
    for (u32 w = 0; w < wave; w++) {
        cE = max(cE, w_E[w]);
        cX += w_X[w];
        cP += w_P[w];
    }
    u16 *sl = B.sl + (size_t)t * (L2_BINS + 64);
#pragma unroll
    for (u32 r = 0; r < ROWS; r++) {
        if (r >= rows) continue;
        const u32 b = (wave * rows + r) * 64u + lane;
        const bool in = b < nb2;
        const u32 m = in ? (u32)sh.mark[b] : 0u;
        const u64 xm = __ballot(m >> 15);
        const u32 eM = max(wave_incl_max(m & 0x7fffu), cE);
        const u32 xM = __builtin_amdgcn_mbcnt_hi((u32)(xm >> 32), __builtin_amdgcn_mbcnt_lo((u32)xm, cX)) + (m >> 15);
        const u32 pI = wave_incl_scan(pop[r]) + cP, pE = pI - pop[r];
        u32 ePrev = (u32)__shfl_up((int)eM, 1), xPrev = (u32)__shfl_up((int)xM, 1);
        if (lane == 0u) {
            ePrev = cE;
            xPrev = cX;
        }
        const u32 ss = eM + xM, ssPrev = ePrev + xPrev;
        if (in) {
            const bool first = b == 0u;
            if (ss >= (u32)MAX_SUB) {
                s_err = 1u;
                sl[b] = 0xFFFFu;
            } else {
                sl[b] = ((actm >> r) & 1u) ? (u16)0xFFFFu : (u16)ss;
                if (first || ss != ssPrev) {
                    atomicAdd(&sh.subc[ss], 0u - pE);
                    if (!first) atomicAdd(&sh.subc[ssPrev], pE);
                    sub_code[ss] = (eM << 9) | xM;
                }
                if (first || eM != ePrev) {
                    atomicAdd(&sh.segc[eM], 0u - pE);
                    if (!first) atomicAdd(&sh.segc[ePrev], pE);
                }
                if (b + 1u == nb2) {
                    atomicAdd(&sh.subc[ss], pI);
                    atomicAdd(&sh.segc[eM], pI);
                }
            }
        }
        cE = (u32)__builtin_amdgcn_readlane((int)eM, 63);
        cX += (u32)__popcll(xm);
        cP = (u32)__builtin_amdgcn_readlane((int)pI, 63);
    }
    __syncthreads();
    if (tid == 0 && s_err) atomicOr(&st->internal_err, 512u);
    u32 *sc = B.seg_cnt + (size_t)t * MAX_EDGES;
    for (u32 i = tid; i <= n_e; i += BLOCK) sc[i] = sh.segc[i];
    u32 *sub_cnt = B.sub_cnt + (size_t)t * MAX_SUB;
    for (u32 i = tid; i < (u32)MAX_SUB; i += BLOCK) sub_cnt[i] = sh.subc[i];
    if (tid == 0) {
        st->n_sub = min(n_e + 512u, (u32)MAX_SUB);
        st->n_edges = n_e;
    }
}

// ------------------------------------------------------------------------------------------
// slots -> bins -> centres, errors, choice
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float float_of_key(u32 k) { return __uint_as_float(bits_of_key(k)); }

__global__ __launch_bounds__(BLOCK) void k_final(const TDesc *__restrict__ td,
                                                 const GridDesc *__restrict__ gd,
                                                 const u32 *__restrict__ t_fu_off,
                                                 const u32 *__restrict__ t_gu_off, Bufs B)
{
    extern __shared__ u32 smem[];
    double *V = reinterpret_cast<double *>(smem);              // [4096] sum of each slot
    u64 *C = reinterpret_cast<u64 *>(smem + 2 * MAX_EDGES);    // [4096] keys in slots 0..s
    double *S8 = reinterpret_cast<double *>(smem + 4 * MAX_EDGES); // [MAX_PAIRS][256] sums of a pair's bins
    double *SV = S8 + MAX_PAIRS * 256;                         // [MAX_SUB] sum of each sub-slot
    __shared__ double s_qout[MAX_FRAC];
    __shared__ double s_sumsq;
    __shared__ __attribute__((aligned(4))) u16 s_cfg[MAX_PAIRS][K_SLOTS]; // first grid entry of (pair, K)
    __shared__ double s_acc[MAX_PAIRS][K_SLOTS];

    const int t = blockIdx.x;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TState *st = B.ts + t;
    if (B.view[t] == VIEW_NONE) return;
    const View vw = view_of(gd, B.view[t]);
    const u64 n = td[t].n;
    const u32 m = st->n_edges;
    const u32 n_cfg = gd->n_cfg, n_p = gd->n_p, n_o = gd->n_o;

    const u32 *segc = B.seg_cnt + (size_t)t * MAX_EDGES;
    const u32 *gc = B.grp_cnt + (size_t)t * 2 * MAX_EDGES;
    const double *gs = B.grp_sx + (size_t)t * 2 * MAX_EDGES;
    for (u32 i = tid; i < (u32)MAX_PAIRS * (u32)K_SLOTS; i += BLOCK) (&s_cfg[0][0])[i] = 0xFFFFu;
    // Per slot: count and sum.  The counts are kept as inclusive prefixes over the slots (a bin is
    // a run of consecutive slots, so its count is a difference): every thread owns four consecutive
    // slots, the running totals of the threads before it come from a scan.  The sums are kept per
    // slot and added bin by bin: a difference of prefix sums would lose a bin of small values next
    // to large ones (fp64 carries 16 digits, fp32 values span 83).
    __shared__ u64 w_c[BLOCK / 64];
    // Keys of bins without an edge: sweep 3 left, per sub-slot, the sum of their 23 mantissa bits.
    // All keys of a sub-slot share sign and exponent E, so their values add up to
    // +-2^(E-150) (2^23 count + sum of mantissas), or +-2^-149 (sum) for E = 0.  The integer is below
    // 2^24 count: converted exactly for a sub-slot of up to 2^29 keys (a bin holds n_kept / K keys, K the
    // grid's largest), and rounded once, like any sum in 64 bits, where a larger tensor and a grid of
    // few bins put more into one.
    const u32 n_sub = st->n_sub;
    const u32 *sub_code = B.sub_code + (size_t)t * MAX_SUB;
    const u32 *sub_cnt = B.sub_cnt + (size_t)t * MAX_SUB;
    const u64 *mom = B.mom_sx + (size_t)t * MAX_SUB;
    // (first and last sub-slot of every slot: kept where the slot's sum goes afterwards)
    u32 *ss_lo = reinterpret_cast<u32 *>(V), *ss_hi = ss_lo + 1; // [2 * slot]
    for (u32 i = tid; i <= m; i += BLOCK) {
        ss_lo[2u * i] = 0xFFFFFFFFu;
        ss_hi[2u * i] = 0u;
    }
    __syncthreads();
    if (vw.K) {
        if (tid == 0u) enter_config(s_cfg, vw.cfg, vw.q0, vw.K);
    } else {
        for (u32 g = tid; g < n_cfg; g += BLOCK) enter_config(s_cfg, g, gd->cfg_pair[g], gd->cfg_K[g]);
    }
    for (u32 ss = tid; ss < n_sub; ss += BLOCK) {
        const u32 code = sub_code[ss];
        double val = 0.0;
        if (code != 0xFFFFFFFFu) {
            const u64 tot = mom[ss];
            const u32 bx = code & 511u; // key >> 23: the top bit is set for values >= 0, else all bits are flipped
            const bool neg = (bx & 256u) == 0u;
            const int E = (int)((neg ? ~bx : bx) & 255u);
            if (E)
                val = ldexp((double)(((u64)sub_cnt[ss] << 23) + tot), E - 150);
            else
                val = ldexp((double)tot, -149);
            if (neg) val = -val;
            const u32 slot = code >> 9;
            if (slot <= m) {
                atomicMin(&ss_lo[2u * slot], ss);
                atomicMax(&ss_hi[2u * slot], ss);
            }
        }
        SV[ss] = val;
    }
    __syncthreads();
    {
        u64 pc[4];
        u64 run_c = 0;
        // a slot's sub-slots in ascending order (those in between that no bin has hold 0.0)
        double su[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const u32 i = 4u * tid + (u32)r;
            if (i <= m) {
                const u32 a = ss_lo[2u * i], b = ss_hi[2u * i];
                for (u32 ss = a; ss <= b && a != 0xFFFFFFFFu; ss++) su[r] += SV[ss];
            }
        }
        __syncthreads(); // V is written next
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const u32 i = 4u * tid + r;
            double sv = 0.0;
            u64 c = 0;
            if (i <= m) {
                // then the gathered keys from the group of the slot's lower edge and from the
                // group of its upper edge
                sv = su[r];
                sv += gs[i];
                sv += gs[MAX_EDGES + i];
                c = (u64)segc[i] + gc[i] + gc[MAX_EDGES + i];
            }
            V[i] = sv;
            run_c += c;
            pc[r] = run_c;
        }
        u64 inc_c = run_c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const u64 b = __shfl_up(inc_c, o);
            if ((int)lane >= o) inc_c += b;
        }
        if (lane == 63u) w_c[wave] = inc_c;
        __syncthreads();
        u64 base_c = inc_c - run_c;
        for (u32 w = 0; w < wave; w++) base_c += w_c[w];
#pragma unroll
        for (int r = 0; r < 4; r++) C[4u * tid + r] = base_c + pc[r];
    }
    // sums of squares: wave 0 the tensor's, wave 1 + o the protected values' of fraction o; the units'
    // parts in a fixed order
    if (wave <= n_o) {
        double s = 0.0;
        if (wave == 0u)
            for (u32 u = t_fu_off[t] + lane; u < t_fu_off[t + 1]; u += 64u) s += B.sq_part[(size_t)u * SQ_STRIDE];
        else
            for (u32 u = t_gu_off[t] + lane; u < t_gu_off[t + 1]; u += 64u) s += B.sq_prot[(size_t)u * MAX_FRAC + wave - 1u];
        s = wave_sum_f64(s);
        if (lane == 0u) {
            if (wave == 0u) {
                s_sumsq = s;
                st->sumsq = s;
            } else {
                s_qout[wave - 1u] = s;
                st->thr_sumsq[n_p + wave - 1u] = s;
            }
        }
    }
    __syncthreads();

    const u16 *pe = B.pair_eidx + (size_t)t * MAX_PAIRS * EIDX_STRIDE;
    // bin k of K: slots lo + 1 .. hi without those of the pruned gap (g_lo, g_hi]
    struct Span {
        u32 lo, hi, g_lo, g_hi;
    };
    auto span = [&](u32 q, u32 K, u32 k) -> Span {
        const u16 *e = pe + q * EIDX_STRIDE;
        Span x;
        x.lo = (k == 0u) ? e[NBT + 0] : e[bnd_index(K, k)];
        x.hi = (k == K - 1u) ? e[NBT + 3] : e[bnd_index(K, k + 1u)];
        x.g_lo = e[NBT + 1];
        x.g_hi = e[NBT + 2];
        return x;
    };
    auto slot_sum = [&](const Span &x) -> double {
        double sk = 0.0;
        for (u32 i = x.lo + 1u; i <= min(x.hi, x.g_lo); i++) sk += V[i];
        for (u32 i = max(x.lo, x.g_hi) + 1u; i <= x.hi; i++) sk += V[i];
        return sk;
    };
    // sums of the finest bins of every pair, slot by slot; the bins for fewer bits are unions of them
    const u32 K_top = !vw.K ? gd->K_top : (vw.K & (vw.K - 1u)) ? 1u : vw.K;
    for (u32 w = tid; w < vw.n_pairs * K_top; w += BLOCK) {
        const u32 q = vw.q0 + w / K_top, k = w % K_top;
        if (K_top > 1u) S8[q * 256u + k] = slot_sum(span(q, K_top, k));
    }
    __syncthreads();
    const u32 *tk = B.tgt_key + (size_t)t * TGT_STRIDE;
    float *cb = B.codebook + (size_t)t * n_cfg * CB_STRIDE;
    auto centre = [&](u32 q, u32 K, u32 k, u32 g, const Span &x, double sk) -> double { // returns 2 c S - n c^2
        u64 nk = C[x.hi] - C[x.lo];
        const u32 a = max(x.lo, x.g_lo), b = min(x.hi, x.g_hi);
        if (a < b) nk -= C[b] - C[a];
        const float c = nk ? (float)(sk / (double)nk) : float_of_key(tk[q * NBT + bnd_index(K, k == 0u ? 1u : k)]);
        cb[g * CB_STRIDE + k] = c;
        const double cd = (double)c;
        return 2.0 * cd * sk - (double)nk * cd * cd;
    };
    // One wave per pair: 3, 6 and 12 bins first (the lanes of a bin share its slots), then K_top bins,
    // half as many, ... 2: the sums of neighbours are added in place by the wave that reads them.
    for (u32 q = vw.q0 + wave; q < vw.q0 + vw.n_pairs; q += BLOCK / 64) {
        for (u32 s = 9u; s < 12u; s++) {
            const u32 g = s_cfg[q][s];
            if (g == 0xFFFFu) continue;
            const u32 K = 3u << (s - 9u), per = 64u / K; // lanes per bin
            const u32 k = lane / per, part = lane % per;
            double sk = 0.0, acc = 0.0;
            Span x = {0u, 0u, 0u, 0u};
            if (k < K) {
                x = span(q, K, k);
                for (u32 i = x.lo + 1u + part; i <= x.hi; i += per)
                    if (i <= x.g_lo || i > x.g_hi) sk += V[i];
            }
            double tot = 0.0; // (a bin's lanes in a fixed order)
            for (u32 j = 0; j < per; j++) tot += __shfl(sk, (int)min(k * per + j, 63u));
            if (k < K && part == 0u) acc = centre(q, K, k, g, x, tot);
            acc = wave_sum_f64(acc);
            if (lane == 0u) s_acc[q][s] = acc;
        }
        for (u32 K = K_top; K >= 2u; K >>= 1) {
            const u32 s = k_slot(K), g = s_cfg[q][s];
            if (g != 0xFFFFu) {
                double acc = 0.0;
                for (u32 k = lane; k < K; k += 64u) acc += centre(q, K, k, g, span(q, K, k), S8[q * 256u + k]);
                acc = wave_sum_f64(acc);
                if (lane == 0u) s_acc[q][s] = acc;
            }
            if (vw.K) break;
            asm volatile("" ::: "memory");
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
            asm volatile("" ::: "memory");
        }
    }
    __syncthreads();
    Score *sc = B.scores + (size_t)t * n_cfg;
    __shared__ double s_sse[MAX_CFG];
    __shared__ u64 s_cost[MAX_CFG];
    for (u32 g = tid; g < n_cfg; g += BLOCK) {
        if (vw.K && g != vw.cfg) continue;
        const u32 K = gd->cfg_K[g], q = gd->cfg_pair[g];
        double sse = s_sumsq - s_qout[gd->pair_o[q]] - s_acc[q][k_slot(K)];
        if (sse < 0.0) sse = 0.0;
        Score r;
        r.sse = sse;
        r.sumsq = s_sumsq;
        r.n_pruned = st->pair_Pn[q] + st->pair_Pp[q];
        r.n_outlier = st->pair_An[q] + st->pair_Ap[q];
        r.n_kept = st->pair_M[q];
        r.cost_bits = payload_bits(r.n_kept, r.n_outlier, K, gd->cfg_l16[g]);
        sc[g] = r;
        s_sse[g] = sse;
        s_cost[g] = r.cost_bits;
        if (r.n_pruned + r.n_outlier + r.n_kept != n) atomicOr(&st->internal_err, 256u);
    }
    __syncthreads();
    if (wave == 0u) {
        if (vw.K) {
            if (lane == 0u) settle_choice(st, vw.cfg, s_sse[vw.cfg], s_sumsq, gd->eps);
        } else {
            const Choice c = choose_config(s_sse, s_cost, n_cfg, gd->eps, s_sumsq);
            if (lane == 0u) {
                st->best = c.best;
                st->feasible = c.feasible;
            }
        }
        if (lane == 0u) store_result(st, B.res + t);
    }
}

constexpr int SM_EDGES = (int)sizeof(EdgeShared);
constexpr int SM_FINAL = (2 * MAX_EDGES + 2 * MAX_EDGES) * 4 + MAX_PAIRS * 256 * 8 + MAX_SUB * 8;

static bool g_attr_done = false;
static hipError_t set_attrs()
{
    if (g_attr_done) return hipSuccess;
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void *)k_edges<true>, hipFuncAttributeMaxDynamicSharedMemorySize, SM_EDGES))) return e;
    if ((e = hipFuncSetAttribute((const void *)k_edges<false>, hipFuncAttributeMaxDynamicSharedMemorySize, SM_EDGES))) return e;
    if ((e = hipFuncSetAttribute((const void *)k_final, hipFuncAttributeMaxDynamicSharedMemorySize, SM_FINAL))) return e;
    g_attr_done = true;
    return hipSuccess;
}

hipError_t launch_edges(const Batch &bt, hipStream_t s)
{
    hipError_t e = set_attrs();
    if (e) return e;
    if (bt.lds_ordered)
        PROF("k_edges", s, k_edges<true><<<bt.nB, BLOCK, SM_EDGES, s>>>(bt.td, bt.gd, bt.bufs, bt.grp_list, bt.n_grp_total));
    else
        PROF("k_edges", s, k_edges<false><<<bt.nB, BLOCK, SM_EDGES, s>>>(bt.td, bt.gd, bt.bufs, bt.grp_list, bt.n_grp_total));
    return hipGetLastError();
}

hipError_t launch_score(const Batch &bt, hipStream_t s)
{
    if (bt.nB == 0) return hipSuccess;
    hipError_t e = set_attrs();
    if (e) return e;
    PROF("k_final", s, k_final<<<bt.nB, BLOCK, SM_FINAL, s>>>(bt.td, bt.gd, bt.t_fu_off, bt.t_gu_off, bt.bufs));
    return hipGetLastError();
}

} // namespace inshr
