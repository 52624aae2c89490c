// Quantizing with one given configuration per tensor from the thresholds and the second histogram of a
// search, when boundaries and centres have not been worked out yet: one sweep instead of two.
//
// The exact ranks of a configuration's K - 1 boundaries (Sec. 4.4) name the search's bins they fall into;
// every other bin lies between two breakpoints and has one symbol.  The sweep writes the symbols and adds the
// values to their symbol's sum; for the few values inside these bins (of 32768 bins at most 255 hold a
// boundary of unknown key) it takes the boundary to lie where its rank would put it if the bin's values were
// evenly spread, and lists them.  The exact boundaries are read off at their ranks in the lists, and what the
// guess got wrong (a few percent of the listed values) is put right in the stream and in the sums.
//
//   k_fplan    per tensor: breakpoints in order of rank, symbol of every bin of the search (a table of
//              64 KB that the sweep loads), the bins with a boundary of unknown key ("open")
//   k_fuse     the sweep
//   k_fsplit   listed values -> their bins
//   k_fsel     one wave per boundary: the key of its rank inside its bin
//   k_fpatch   listed values whose symbol the guess got wrong
//   k_fprot    protected values: the sweep's lists, one per wave -> the tensor's list in index order
//   k_fhead    per tensor: centres, boundaries, class counts
//
// 6.7 G values, symbols of 9 bits: k_fuse 9.5 ms (27.0 GB read, 9.3 GB written: 3.8 TB/s; bound by vector issue and the
// LDS pipe, half of whose time are bank conflicts of the table reads; one workgroup of 16 waves fits a CU.  11.0 when
// a tile's words were OR-ed together in LDS behind a barrier), k_fsplit 0.34, k_fsel 0.22, k_fpatch 0.41, k_fprot 0.37; boundaries, centres and
// k_quant for one configuration took 8.7 (k_gather) + 0.6 + 8.9 (k_quant).  100 M values in 48 tensors: 0.25 ms where
// k_plan2 .. k_quant took 0.70.
//
// Without output buffers (QDesc::packed is NULL) the same kernels work out boundaries, centres and the exact error of the
// configuration and settle a choice that hangs on it: 1 Mi values 67 us where k_plan2 .. k_final took 130, 162 M
// compacted values 0.22 ms instead of 0.38.
//
// A tensor that these means do not hold (a bin with more values than one wave should read, lists that
// overflow) is marked (TState::fuse_bad); the host sends it through launch_resolve and launch_quantize.
#include "inshr_quant.h"

namespace inshr {

// Table entries: a symbol (0, 2 .. K + 1), or
constexpr u32 F_PROT = 0x2000u;  // every value of the bin is protected
constexpr u32 F_OPEN = 0x4000u;  // the bin holds breakpoints, boundaries whose key is not known among them:
                                 // | the first breakpoint of the bin
constexpr u32 F_EDGES = 0x8000u; // the bin holds known breakpoints only: | the first of them
// Sums: the values of one symbol, sign and exponent share a cell, where their number and the sum of their 23
// mantissa bits are counted together (the value is linear in the mantissa; integers: any order, exact).
// Cell = symbol + (key >> 23): both grow with the key, so no two pairs of them meet in a cell.
constexpr u32 F_CELLS = 776;     // 257 + 511 + 1, padded
constexpr u32 F_COPIES = 4;      // by lane modulo 4: a bin of the quantizer takes many of a wave's lanes
constexpr u32 F_CNT = 43;        // a cell's count starts at this bit; below it the sum of up to 2^20 mantissas
constexpr u32 F_FLUSH = 64;      // tiles after which the cells are emptied: 2^20 values
static_assert((u64)F_FLUSH * TILE == 1ull << (F_CNT - 23), "the sum of the mantissas stays below the count");
constexpr u32 F_MAXBIN = 65536;  // most values of an open bin
constexpr u32 F_TILEW = 32;      // words per tile in front of a unit's protected lists: 16 waves x 4 u16 counts

// A unit's protected lists lie in the first half of the tensor's span of the first pool (the second half
// takes the listed values, bin by bin).
struct ProtLists {
    u64 counts, list; // counts per tile; list of wave w from list + w * cap on
    u32 cap;
};
__device__ __forceinline__ ProtLists prot_lists(const Unit &un, u64 span)
{
    ProtLists p;
    const u64 tiles = un.tile1 - un.tile0;
    p.counts = span + (un.off() - span) / 2u;
    p.list = p.counts + tiles * F_TILEW;
    p.cap = (u32)((8ull * un.capw - tiles * F_TILEW) / 16u); // (a share has room for 32 keys per tile and 1024 more, or for all: at least 510, and 14 per tile)
    return p;
}
// Values listed by wave w of a unit: keys and indices, each in one half of its share of the second pool.
__device__ __forceinline__ u32 *open_keys(const Bufs &B, const Unit &un, u32 w) { return B.pool2 + un.off() + (u64)w * un.capw; }
__device__ __forceinline__ u32 open_cap(const Unit &un) { return un.capw / 2u; }

// ------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_fplan(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                 const QDesc *__restrict__ qd, Bufs B)
{
    __shared__ u32 T[COARSE];
    __shared__ u32 pre8[L2_BINS / 8];                     // keys in the bins before every eighth
    __shared__ u32 tmp[BLOCK / 64], n_at[L2_BINS / 32];   // breakpoints in every 32 bins
    __shared__ u32 b_rank[256], b_bin[256], c_rank[4], c_pos[4];
    __shared__ u32 bp[QBP + 8], bp_bin[QBP + 8];          // breakpoints in order
    __shared__ u16 symtab[QBP];
    __shared__ u32 has[L2_BINS / 32], open[L2_BINS / 32]; // bins with a breakpoint, with one of unknown key
    __shared__ u32 w_new[4], w_pop[4];
    __shared__ u32 s_bad;

    const int t = blockIdx.x;
    const QDesc q = qd[t];
    if (!q.fused) return;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u64 n = td[t].n;
    TState *st = B.ts + t;
    const u32 pair = gd->cfg_pair[q.cfg], K = gd->cfg_K[q.cfg], n_bnd = K - 1u, n_bp = n_bnd + 4u;
    const u32 zbin = st->zbin, n_zero = (u32)st->n_zero;
    const u32 *h2 = B.hist2 + (size_t)t * L2_BINS;
    const u32 *tab = B.table2 + (size_t)t * COARSE;
    u32 *tk = B.tgt_key + (size_t)t * TGT_STRIDE + pair * NBT;
    u32 *goff = B.grp_off + (size_t)t * MAX_GROUPS, *gcur = B.grp_cur + (size_t)t * MAX_GROUPS;

    typedef u32 u4 __attribute__((ext_vector_type(4)));
    u32 part[4], mine = 0u; // keys of the thread's 32 bins (those past the last one are empty)
    {
        u4 c[8];
#pragma unroll
        for (u32 i = 0; i < 8u; i++) c[i] = ((const GLOBAL_AS u4 *)gptr(h2))[tid * 8u + i];
#pragma unroll
        for (u32 i = 0; i < 8u; i++) {
            if ((i & 1u) == 0u) part[i >> 1] = mine;
            mine += c[i].x + c[i].y + c[i].z + c[i].w;
        }
    }
    for (u32 i = tid; i < (u32)COARSE; i += BLOCK) T[i] = tab[i];
    has[tid] = open[tid] = n_at[tid] = 0u;
    static_assert(L2_BINS / 32 == BLOCK, "one word of the bins' bits per thread");
    if (tid == 0u) s_bad = 0u;
    for (u32 i = tid; i < 2u * F_CELLS; i += BLOCK) B.mom_sx[(size_t)t * MAX_SUB + i] = 0ull;
    const u32 inc_n = wave_incl_scan(mine);
    if (lane == 63u) tmp[wave] = inc_n;
    __syncthreads();
    u32 before = inc_n - mine, total = 0u;
    for (u32 w = 0; w < BLOCK / 64; w++) {
        const u32 x = tmp[w];
        before += w < wave ? x : 0u;
        total += x;
    }
#pragma unroll
    for (u32 i = 0; i < 4u; i++) pre8[4u * tid + i] = before + part[i];
    if (tid == 0u && (u64)total != n) atomicOr(&st->internal_err, 16u);
    __syncthreads();
    const u64 An = st->pair_An[pair], Mn = st->pair_Mn[pair], M = st->pair_M[pair];
    const u64 PP = st->pair_Pn[pair] + st->pair_Pp[pair];
    const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + gd->pair_o[pair]];

    // ---- boundaries: rank, bin, values of the bin below the rank; class edges ------------------------
    u32 bin = 0u, res = 0u, klo = 0u, guess = 0u, bits = 0u, pop = 0u, rank = 0u;
    bool known = true; // the boundary is the zero key
    const bool is_edge = tid >= 256u && tid < 260u;
    u32 edge = 0u;
    if (tid < n_bnd) {
        u32 num, den;
        bnd_fraction(bnd_index(K, tid + 1u), num, den);
        const u64 x = (u64)num * M, k = den == 256u ? x >> 8 : x / 12ull;
        const u64 r = An + k + (k < Mn ? 0ull : PP);
        if (r >= n) atomicOr(&s_bad, 1u); // (only without quantized values, which is reported)
        rank = (u32)(r < n ? r : n - 1ull);
        u32 g = 0u; // last group of eight bins that starts at or before the rank, the last such bin of it
#pragma unroll
        for (u32 step = L2_BINS / 16; step > 0u; step >>= 1)
            if (pre8[g + step] <= rank) g += step;
        const u4 y0 = ((const GLOBAL_AS u4 *)gptr(h2))[2u * g], y1 = ((const GLOBAL_AS u4 *)gptr(h2))[2u * g + 1u];
        const u32 f[8] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w};
        u32 run = pre8[g];
        bin = 8u * g;
        res = rank - run;
        pop = f[0];
#pragma unroll
        for (u32 i = 1; i < 8u; i++) {
            run += f[i - 1u];
            if (run <= rank) {
                bin = 8u * g + i;
                res = rank - run;
                pop = f[i];
            }
        }
        u32 lo, hi;
        known = bin == zbin && res < n_zero; // exact zeros come first in their bin and are never put aside
        if (bin == zbin) {
            res -= known ? 0u : n_zero;
            pop -= n_zero;
        }
        lo = 0u;
        hi = COARSE - 1u; // key prefix of the bin: the last one that starts at or below it
        while (lo < hi) {
            const u32 mid = (lo + hi + 1u) >> 1;
            if (((T[mid] >> 5) & 0x7fffu) <= bin)
                lo = mid;
            else
                hi = mid - 1u;
        }
        const u32 e = T[lo];
        bits = (u32)COARSE_SHIFT - (e & 31u);
        klo = (lo << COARSE_SHIFT) | ((bin - ((e >> 5) & 0x7fffu)) << bits);
        b_rank[tid] = rank;
        b_bin[tid] = known ? RESOLVED : bin;
        guess = klo + (u32)(((u64)res << bits) / (pop ? pop : 1u)); // (below the next bin: res < pop)
        if (known) klo = guess = ZERO_KEY;
    } else if (is_edge) {
        edge = tid - 256u;
        guess = class_edge_key(edge, tau_p, tau_o);
        bin = l2_bin(guess, T[guess >> COARSE_SHIFT]);
        c_rank[edge] = (u32)(edge == 0u ? An : edge == 1u ? An + Mn : edge == 2u ? An + Mn + PP : An + M + PP);
    }
    __syncthreads();
    // ---- all breakpoints in order of rank, a class edge before a boundary of equal rank --------------
    u32 pos = 0u;
    if (tid < n_bnd) {
        pos = tid;
#pragma unroll
        for (u32 e = 0; e < 4u; e++) pos += c_rank[e] <= rank ? 1u : 0u;
    } else if (is_edge) {
        u32 lo = 0u, hi = n_bnd; // boundaries of lower rank
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if (b_rank[mid] < c_rank[edge])
                lo = mid + 1u;
            else
                hi = mid;
        }
        pos = c_pos[edge] = lo + edge;
    }
    if (tid < n_bnd || is_edge) {
        bp[pos] = guess;
        bp_bin[pos] = bin;
        atomicOr(&has[bin >> 5], 1u << (bin & 31u));
        atomicAdd(&n_at[bin >> 5], 1u);
        if (!known) atomicOr(&open[bin >> 5], 1u << (bin & 31u));
    }
    if (tid >= n_bp && tid < (u32)QBP + 8u) bp[tid] = 0xFFFFFFFFu; // (n_bp <= 259: places that nothing else writes)
    // ---- the open bins in order (the boundaries ascend), room for their values -----------------------
    const bool fresh = !known && !(tid && b_bin[tid - 1u] == bin);
    u32 u_in = 0u, p_in = 0u;
    if (tid < 256u) {
        u_in = wave_incl_scan(fresh ? 1u : 0u);
        p_in = wave_incl_scan(fresh ? pop : 0u);
        if (lane == 63u) {
            w_new[wave] = u_in;
            w_pop[wave] = p_in;
        }
        if (fresh && pop > F_MAXBIN) atomicOr(&s_bad, 1u);
    }
    __syncthreads();
    if (tid < n_bnd) {
        for (u32 w = 0; w < wave; w++) {
            u_in += w_new[w];
            p_in += w_pop[w];
        }
        u32 *row = B.tgt_bin + (size_t)t * TGT_STRIDE;
        row[tid] = known ? RESOLVED : u_in - 1u;
        B.tgt_res[(size_t)t * TGT_STRIDE + tid] = res;
        tk[bnd_index(K, tid + 1u)] = known ? ZERO_KEY : 0u;
        if (fresh) {
            B.tgt_klo[(size_t)t * TGT_STRIDE + u_in - 1u] = klo;
            B.tgt_khi[(size_t)t * TGT_STRIDE + u_in - 1u] = bits;
            goff[u_in - 1u] = p_in - pop;
            gcur[u_in - 1u] = 0u;
        }
    }
    if (tid == 0u) {
        const u32 U = w_new[0] + w_new[1] + w_new[2] + w_new[3];
        const u64 all = (u64)w_pop[0] + w_pop[1] + w_pop[2] + w_pop[3];
        goff[U] = (u32)all;
        st->n_groups = U;
        st->fuse_bad = (s_bad || all > q.span_len / 2u || M == 0ull) ? 1u : 0u;
    }
    if (tid <= n_bp) { // symbol behind tid breakpoints
        u32 ce = 0u;
#pragma unroll
        for (u32 e = 0; e < 4u; e++) ce += c_pos[e] < tid ? 1u : 0u;
        symtab[tid] = (u16)(ce == 0u || ce == 4u ? 1u : ce == 2u ? 0u : 2u + tid - ce);
    }
    const u32 here = n_at[tid], inc_b = wave_incl_scan(here);
    if (lane == 63u) tmp[wave] = inc_b;
    __syncthreads();
    // breakpoints and symbols for the sweep.  The guesses of a bin's boundaries and the class edges among them
    // need not be in order: a running maximum (it changes nothing in a bin whose breakpoints are all known,
    // lower ones lie in lower bins)
    u32 *gbp = B.edges + (size_t)t * MAX_EDGES;
    u16 *gsym = B.edge_item + (size_t)t * MAX_EDGES;
    static_assert((QBP + 8 + 63) / 64 <= 5, "five waves hold the breakpoints");
    if (wave < 5u) {
        u32 top = 0u; // the largest of the waves before
        for (u32 w = 0; w < wave; w++) top = max(top, (u32)__builtin_amdgcn_readlane((int)wave_incl_max(bp[w * 64u + lane]), 63));
        const u32 x = tid < (u32)QBP + 8u ? bp[tid] : 0u;
        const u32 y = max(wave_incl_max(x), top);
        if (tid < (u32)QBP + 8u) gbp[tid] = y;
    }
    if (tid <= n_bp) gsym[tid] = symtab[tid];
    if (tid == 0u) { // symbol of the zero key: quantized values are at most as many boundaries above
        u32 ce = 0u, nb = 0u;
        for (u32 e = 0; e < 4u; e++) ce += class_edge_key(e, tau_p, tau_o) <= ZERO_KEY ? 1u : 0u;
        u32 lo = 0u, hi = n_bnd; // boundaries in lower bins, and those that are the zero key
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if (b_bin[mid] == RESOLVED || b_bin[mid] < zbin)
                lo = mid + 1u;
            else
                hi = mid;
        }
        nb = lo;
        gsym[QBP] = (u16)(ce == 0u || ce == 4u ? 1u : ce == 2u ? 0u : 2u + nb);
    }
    // ---- table of the thread's 32 bins ---------------------------------------------------------------
    u32 s = inc_b - here; // breakpoints in lower bins
    for (u32 w = 0; w < wave; w++) s += tmp[w];
    auto code = [&](u32 slot) { return symtab[slot] == 1u ? F_PROT : (u32)symtab[slot]; };
    u32 e = code(s);
    const u32 word = has[tid], wopen = open[tid];
    u4 row[4];
#pragma unroll
    for (u32 i = 0; i < 16u; i++) row[i >> 2][i & 3u] = e | (e << 16);
    if (word) {
#pragma unroll
        for (u32 i = 0; i < 32u; i++) {
            u32 v = e;
            if ((word >> i) & 1u) {
                v = ((wopen >> i) & 1u ? F_OPEN : F_EDGES) | s;
                while (s < n_bp && bp_bin[s] == 32u * tid + i) s++;
                e = code(s);
            }
            const u32 j = i >> 1;
            row[j >> 2][j & 3u] = (i & 1u) ? (row[j >> 2][j & 3u] & 0xFFFFu) | (v << 16) : v;
        }
    }
    // (rows of the table start at multiples of 128 bytes)
    GLOBAL_AS u4 *sl = (GLOBAL_AS u4 *)gptr((u32 *)(B.sl + (size_t)t * (L2_BINS + 64)));
#pragma unroll
    for (u32 i = 0; i < 4u; i++) sl[4u * tid + i] = row[i];
}

// ------------------------------------------------------------------------------------------
// the sweep
// ------------------------------------------------------------------------------------------
struct FuseShared {
    u32 T[COARSE];                   // key prefix -> bins
    u16 symt[L2_BINS];               // table of the bins
    unsigned long long piece[4 * BLOCK]; // a tile's symbols, joined as WavePack does: 64 words for every wave and quarter
    unsigned long long queue[BLOCK];     // per wave: values whose symbol the table of the bins does not say
    unsigned long long cell[F_CELLS * F_COPIES];
    u32 bp[QBP + 8];
    u16 symtab[QBP + 8];
};
struct FuseOut { // where a wave's lists go
    GLOBAL_AS u32 *key, *idx, *prot;
    u32 cap, pcap;       // entries of the lists
    u32 n, np;           // ... in use (wave-uniform)
    u32 nq;              // values in the wave's queue, at most 64
    bool overflow;
};

// The symbol that the sweep gives a listed value: what the guessed breakpoints say, but protected values are
// known exactly (they are listed at once).
__device__ __forceinline__ u32 listed_symbol(u32 guess, u32 key, u32 tau_o)
{
    return mag_of_key(key) > tau_o ? 1u : guess == 1u ? 0u : guess;
}

__device__ __forceinline__ void add_value(FuseShared &fs, u32 sym, u32 key, float x, u32 copy)
{
    atomicAdd(&fs.cell[(sym + (key >> 23)) * F_COPIES + copy],
              (unsigned long long)(__float_as_uint(x) & 0x7fffffu) | (1ull << F_CNT));
}

// Of 1024 values that a wave takes of a tile some twenty lie in bins that hold a breakpoint or are protected: few enough
// for one pass over all of them, and in every quarter of them there are some.  So they queue up, and the wave works
// on them together, a lane each, when the tile is through or the queue is full.  (A pass per quarter, or several if two
// of a lane's four were among them: 6.7 G values 10.3 ms, 9.5 so; GPT-2 medium with Adam state 1.46 and 1.41.)
// An entry: the key, and above it the table's entry and the value's place in the tile: quarter << 8 | lane << 2 | which of four.
__device__ __forceinline__ unsigned long long queue_entry(u32 key, u32 e, u32 place) { return (u64)(place << 16 | e) << 32 | key; }

struct FuseTile { // what the wave knows of the tile
    u32 e0, n_bp, tau_o;
    u32 zero_sym; // symbol of the zeros, if their bin holds breakpoints; F_PROT or above if the table says it
};

// DRY: nothing is written but the lists (no output buffers).
// pc[j]: protected values of the wave's quarter j so far.
template <bool DRY>
__device__ __forceinline__ void fuse_queue(FuseShared &fs, u32 lane, const FuseTile &ft, const WavePack &wp, FuseOut &o, u32 (&pc)[4])
{
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool aside = false, prot = false;
    u32 k = 0u, place = 0u, index = 0u;
    asm volatile("" ::: "memory"); // (a wave's LDS operations complete in order)
    if (lane < o.nq) {
        const unsigned long long entry = fs.queue[wave * 64u + lane];
        k = (u32)entry;
        const u32 x = (u32)(entry >> 32) & 0xFFFFu;
        place = (u32)(entry >> 48);
        index = ft.e0 + 4096u * (place >> 8) + 256u * wave + (place & 255u);
        u32 sym = 1u;
        if (x != F_PROT) {
            u32 s = x & 511u; // breakpoints at or below the key, from the bin's first one on
            if (fs.bp[s] <= k) {
                s++;
                if (fs.bp[s] <= k) s = slot_of_key(fs.bp, ft.n_bp, k);
            }
            sym = fs.symtab[s];
            if (x & F_OPEN) {
                aside = true;
                sym = listed_symbol(sym, k, ft.tau_o);
            }
        }
        prot = sym == 1u;
        if (!DRY) wp.add(fs.piece + (place >> 8) * BLOCK + wave * 64u, (place >> 2) & 63u, place & 3u, sym);
        if (sym >= 2u) add_value(fs, sym, k, __uint_as_float(bits_of_key(k)), lane & (F_COPIES - 1u));
    }
    o.nq = 0u;
    const u64 am = __ballot(aside);
    if (am) {
        const u32 m = (u32)__popcll(am);
        if (o.n + m > o.cap) {
            o.overflow = true;
        } else {
            if (aside) {
                const u32 at = __builtin_amdgcn_mbcnt_hi((u32)(am >> 32), __builtin_amdgcn_mbcnt_lo((u32)am, o.n));
                o.key[at] = k;
                if (!DRY) o.idx[at] = index;
            }
            o.n += m;
        }
    }
    const u64 pm = __ballot(prot);
    if (pm) { // listed in index order, as they queued up
        const u32 m = (u32)__popcll(pm);
        if (o.np + m > o.pcap) {
            o.overflow = true;
        } else {
            if (prot) o.prot[__builtin_amdgcn_mbcnt_hi((u32)(pm >> 32), __builtin_amdgcn_mbcnt_lo((u32)pm, o.np))] = index;
            o.np += m;
#pragma unroll
            for (u32 j = 0; j < 4u; j++) pc[j] += (u32)__popcll(__ballot(prot && place >> 8 == j));
        }
    }
    asm volatile("" ::: "memory");
}

template <bool FULL, bool DRY>
__device__ __forceinline__ void fuse_tile(FuseShared &fs, u32 lane, const float (&v)[16], u32 mask, const FuseTile &ft, u32 w,
                                          GLOBAL_AS unsigned long long *dst, u32 n_words, FuseOut &o, u32 (&pc)[4])
{
    const u32 copy = lane & (F_COPIES - 1u), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WavePack wp(w, lane);
    pc[0] = pc[1] = pc[2] = pc[3] = 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        u32 e[4], key[4];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            key[c] = key_of_float(v[4 * j + c]);
            e[c] = fs.T[key[c] >> COARSE_SHIFT];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) {
            e[c] = lookup_u16(fs.symt, key[c], e[c]);
            if (!FULL && !((mask >> (4 * j + c)) & 1u)) e[c] = 0u;
        }
        if (ft.zero_sym < F_PROT) // (they may be most of a tensor)
#pragma unroll
            for (int c = 0; c < 4; c++) e[c] = key[c] == ZERO_KEY && e[c] >= F_PROT ? ft.zero_sym : e[c];
        u32 lo32 = 0u, s3 = 0u;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const u32 sym = e[c] < F_PROT ? e[c] : 0u;
            if (c < 3)
                lo32 |= sym << (c * w);
            else
                s3 = sym;
            if (sym >= 2u) add_value(fs, sym, key[c], v[4 * j + c], copy);
        }
        if (!DRY) wp.put((unsigned long long)lo32 | ((unsigned long long)s3 << (3u * w)), fs.piece + j * BLOCK + wave * 64u, lane);
        if (__ballot((e[0] | e[1] | e[2] | e[3]) >= F_PROT)) { // (the same for the whole wave)
            u32 n = 0u, below;
#pragma unroll
            for (int c = 0; c < 4; c++) n += e[c] >= F_PROT ? 1u : 0u;
            const u32 all = rank_counts(n, below);
            // (more than 64 of a quarter: 16 lanes at a time)
            for (u32 part = 0u; part < 4u; part += all > 64u ? 1u : 4u) {
                const bool now = all <= 64u || lane >> 4 == part;
                u32 m = all;
                if (all > 64u) m = rank_counts(now ? n : 0u, below);
                if (o.nq + m > 64u) fuse_queue<DRY>(fs, lane, ft, wp, o, pc);
                u32 at = wave * 64u + o.nq + below;
#pragma unroll
                for (int c = 0; c < 4; c++)
                    if (now && e[c] >= F_PROT) fs.queue[at++] = queue_entry(key[c], e[c], (u32)j << 8 | lane << 2 | (u32)c);
                o.nq += m;
            }
        }
    }
    if (o.nq) fuse_queue<DRY>(fs, lane, ft, wp, o, pc);
    if (!DRY) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const unsigned long long x = wp.word(fs.piece + j * BLOCK + wave * 64u, lane);
            const u32 at = ((u32)j * (BLOCK / 64) + wave) * 4u * w + lane;
            if (lane < 4u * w && (FULL || at < n_words)) dst[at] = x;
        }
        asm volatile("" ::: "memory");
    }
}

template <bool DRY>
__global__ __launch_bounds__(BLOCK) void k_fuse(const TDesc *__restrict__ td, const u32 *__restrict__ wg_gu0,
                                                const GridDesc *__restrict__ gd, const QDesc *__restrict__ qd, Bufs B)
{
    __shared__ FuseShared fs; // (one static object: it starts at LDS address 0, offsets fold into the instructions)
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (u32 k = threadIdx.x; k < F_CELLS * F_COPIES; k += BLOCK) fs.cell[k] = 0ull;
    for (u32 gu = wg_gu0[blockIdx.x]; gu < wg_gu0[blockIdx.x + 1]; gu++) {
        u32 tid = threadIdx.x;
        asm volatile("" : "+v"(tid)); // (what is derived from it is cheap: worked out per unit it is not kept in scratch)
        const u32 lane = tid & 63u;
        const Unit un = B.gunits[gu];
        const int t = (int)un.tensor;
        TState *st = B.ts + t;
        const QDesc q = qd[t];
        if (st->fuse_bad & 1u) continue; // (as k_fplan found; the same for the whole workgroup)
        const TDesc d = td[t];
        const u32 K = gd->cfg_K[q.cfg], w = symbol_bits(K), n_bp = K + 3u;
        __syncthreads(); // (the tables of the unit before are not read any more)
        for (u32 i = tid; i < (u32)COARSE; i += BLOCK) fs.T[i] = entry_for_u16(B.table2[(size_t)t * COARSE + i]);
        {
            const u32 *gseg = reinterpret_cast<const u32 *>(B.sl + (size_t)t * (L2_BINS + 64));
            u32 *seg32 = reinterpret_cast<u32 *>(fs.symt);
#pragma unroll 4
            for (u32 i = tid; i < (u32)L2_BINS / 2u; i += BLOCK) seg32[i] = gseg[i];
        }
        if (tid < (u32)QBP + 8u) {
            fs.bp[tid] = B.edges[(size_t)t * MAX_EDGES + tid];
            fs.symtab[tid] = B.edge_item[(size_t)t * MAX_EDGES + tid];
        }
        __syncthreads();
        const u32 zero_e = lookup_u16(fs.symt, ZERO_KEY, fs.T[ZERO_KEY >> COARSE_SHIFT]);
        const u32 zero_sym = __builtin_amdgcn_readfirstlane(zero_e >= F_PROT ? (u32)fs.symtab[QBP] : F_PROT);
        const u32 tau_o = __builtin_amdgcn_readfirstlane(st->thr_mag[gd->n_p + gd->pair_o[gd->cfg_pair[q.cfg]]]);
        GLOBAL_AS unsigned long long *packed = gptr(q.packed);
        const ProtLists pl = prot_lists(un, q.span);
        FuseOut o;
        o.key = gptr(open_keys(B, un, wave));
        o.cap = open_cap(un);
        o.idx = o.key + o.cap;
        o.prot = gptr(B.pool) + pl.list + (u64)wave * pl.cap;
        o.pcap = pl.cap;
        o.n = o.np = o.nq = 0u;
        o.overflow = false;
        u64 sum_m = 0ull; // cell tid of the unit so far
        u32 sum_c = 0u;
        auto tile_cnt = [&](u64 tl) -> u32 {
            const u64 rem = d.n - (tl - d.tile0) * (u64)TILE;
            return tile_len(rem, (u32)TILE);
        };
        auto flush = [&] { // the cells are emptied, by all threads together
            if (tid < F_CELLS) {
#pragma unroll
                for (u32 k = 0; k < F_COPIES; k++) {
                    const unsigned long long x = fs.cell[tid * F_COPIES + k];
                    sum_m += x & ((1ull << F_CNT) - 1ull);
                    sum_c += (u32)(x >> F_CNT);
                    fs.cell[tid * F_COPIES + k] = 0ull;
                }
            }
        };
        // The waves drift apart freely: a wave's symbols are whole words of their own, which it packs and stores.  A tile's
        // values are asked for during the tile before.
        float vn[16];
        bool ahead = false;
        for (u64 tile = un.tile0; tile < un.tile1; tile++) {
            const u64 e0 = (tile - d.tile0) * (u64)TILE;
            const u32 cnt = tile_cnt(tile);
            float v[16];
            u32 mask = 0xFFFFu;
            if (ahead) {
#pragma unroll
                for (int i = 0; i < 16; i++) v[i] = vn[i];
            } else {
                mask = load_tile(d, e0, cnt, v);
            }
#pragma unroll
            for (int i = 0; i < 16; i++)
                asm volatile("" : "+v"(v[i])); // the values are taken here, before any store below
            ahead = tile + 1 < un.tile1 && tile_cnt(tile + 1) == (u32)TILE;
            if (ahead) load_tile_ahead(d, e0 + TILE, vn);
            u32 pc[4];
            GLOBAL_AS unsigned long long *dst = packed + (tile - d.tile0) * (u64)(256u * w);
            const u32 n_words = (cnt * w + 63u) >> 6;
            // (whole tile or not is the same for every lane: the tile code uses ballots)
            const FuseTile ft = {(u32)e0, n_bp, tau_o, zero_sym};
            if (cnt == (u32)TILE)
                fuse_tile<true, DRY>(fs, lane, v, mask, ft, w, dst, n_words, o, pc);
            else
                fuse_tile<false, DRY>(fs, lane, v, mask, ft, w, dst, n_words, o, pc);
            if (lane == 0u) {
                typedef u32 u2 __attribute__((ext_vector_type(2)));
                const u2 x = {pc[0] | (pc[1] << 16), pc[2] | (pc[3] << 16)};
                *(GLOBAL_AS u2 *)(gptr(B.pool) + pl.counts + (tile - un.tile0) * F_TILEW + 2u * wave) = x;
            }
            if ((tile + 1 - un.tile0) % F_FLUSH == 0 && tile + 1 < un.tile1) {
                __syncthreads();
                flush();
                __syncthreads();
            }
        }
        __syncthreads();
        flush();
        if (tid < F_CELLS && sum_c) {
            unsigned long long *gm = (unsigned long long *)B.mom_sx + (size_t)t * MAX_SUB;
            if (sum_m) atomicAdd(&gm[tid], (unsigned long long)sum_m);
            atomicAdd(&gm[F_CELLS + tid], (unsigned long long)sum_c);
        }
        if (lane == 0u) {
            B.unit_cand[(size_t)gu * 16 + wave] = o.n;
            B.unit_prot[(size_t)gu * 16 + wave] = o.np;
            if (o.overflow) atomicOr(&st->fuse_bad, 2u);
        }
        // (a unit's cells are clean before the next one's first barrier)
    }
}

// ------------------------------------------------------------------------------------------
// the boundaries
// ------------------------------------------------------------------------------------------
constexpr u32 FS_PER = 8;    // keys per thread and step
constexpr u32 FS_PARTS = 2;  // workgroups that share a unit

// last of the n open bins whose first key is at or below the key (the key lies in one of them)
__device__ __forceinline__ u32 open_bin(const u32 *first, u32 n, u32 key)
{
    u32 u = 0u;
#pragma unroll
    for (u32 step = 128u; step > 0u; step >>= 1)
        if (u + step < n && first[u + step] <= key) u += step;
    return u;
}

__global__ __launch_bounds__(BLOCK) void k_fsplit(const QDesc *__restrict__ qd, Bufs B)
{
    __shared__ u32 first[256], count[256], base[256], off[256], s_tot[4];
    __shared__ u32 stage[64 * FS_PER * (BLOCK / 64)];
    __shared__ unsigned char stage_u[64 * FS_PER * (BLOCK / 64)];
    const u32 gu = blockIdx.x;
    const Unit un = B.gunits[gu];
    const int t = (int)un.tensor;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TState *st = B.ts + t;
    if (st->fuse_bad) return;
    const QDesc q = qd[t];
    const u32 c = B.unit_cand[(size_t)gu * 16 + wave];
    u32 cmax = 0u;
    for (u32 w = 0; w < BLOCK / 64; w++) cmax = max(cmax, B.unit_cand[(size_t)gu * 16 + w]);
    if (cmax <= blockIdx.y * 64u * FS_PER) return;
    const u32 U = st->n_groups;
    const u32 *goff = B.grp_off + (size_t)t * MAX_GROUPS;
    u32 *gcur = B.grp_cur + (size_t)t * MAX_GROUPS;
    const GLOBAL_AS u32 *src = gptr(open_keys(B, un, wave));
    GLOBAL_AS u32 *dst = gptr(B.pool) + q.span + q.span_len / 2u;
    u32 my_off = 0u, my_room = 0u;
    if (tid < 256u) {
        first[tid] = tid < U ? B.tgt_klo[(size_t)t * TGT_STRIDE + tid] : 0u;
        count[tid] = 0u;
        if (tid < U) {
            my_off = goff[tid];
            my_room = goff[tid + 1u] - my_off;
        }
    }
    __syncthreads();
    for (u32 b = blockIdx.y * 64u * FS_PER; b < cmax; b += FS_PARTS * 64u * FS_PER) {
        u32 key[FS_PER], ur[FS_PER]; // bin << 16 | rank inside (step, bin)
#pragma unroll
        for (u32 j = 0; j < FS_PER; j++) {
            const u32 i = b + lane + j * 64u;
            key[j] = i < c ? src[i] : 0u;
        }
#pragma unroll
        for (u32 j = 0; j < FS_PER; j++) {
            ur[j] = 0xFFFFFFFFu;
            if (b + lane + j * 64u < c) {
                const u32 u = open_bin(first, U, key[j]);
                ur[j] = (u << 16) | atomicAdd(&count[u], 1u);
            }
        }
        __syncthreads();
        u32 mine = 0u, in = 0u;
        if (tid < 256u) { // room for the step's keys in every bin, and their place in the stage
            mine = count[tid];
            count[tid] = 0u;
            in = wave_incl_scan(mine);
            if (lane == 63u) s_tot[wave] = in;
            if (mine) {
                const u32 at = atomicAdd(&gcur[tid], mine);
                base[tid] = my_off + at;
                if (at + mine > my_room) { // (more keys than the histogram counted: nothing is stored)
                    base[tid] = 0xFFFFFFFFu;
                    atomicOr(&st->internal_err, 128u);
                }
            }
        }
        __syncthreads();
        if (tid < 256u) {
            u32 o = in - mine;
            for (u32 w = 0; w < wave; w++) o += s_tot[w];
            off[tid] = o;
        }
        const u32 all = s_tot[0] + s_tot[1] + s_tot[2] + s_tot[3];
        __syncthreads();
#pragma unroll
        for (u32 j = 0; j < FS_PER; j++) {
            if (ur[j] == 0xFFFFFFFFu) continue;
            const u32 u = ur[j] >> 16, at = off[u] + (ur[j] & 0xFFFFu);
            stage[at] = key[j];
            stage_u[at] = (unsigned char)u;
        }
        __syncthreads();
        for (u32 at = tid; at < all; at += BLOCK) { // a wave's stores go to a few runs of addresses
            const u32 u = stage_u[at];
            if (base[u] != 0xFFFFFFFFu) dst[base[u] + (at - off[u])] = stage[at];
        }
        __syncthreads();
    }
}

// One wave per boundary: the key of rank res among the n keys of its bin, which agree but for their low
// bits.  Up to 1024 keys are held in registers and the bits chosen one by one from ballots; more are
// counted in LDS by digits of 8 bits.
constexpr u32 SEL_WAVES = 4;
constexpr u32 SEL_ROWS = 16;
__global__ __launch_bounds__(64 * SEL_WAVES) void k_fsel(const GridDesc *__restrict__ gd, const QDesc *__restrict__ qd, Bufs B)
{
    __shared__ u32 hist[SEL_WAVES][256];
    const int t = blockIdx.x; // (a grid's second dimension ends at 65535)
    const QDesc q = qd[t];
    if (!q.fused) return;
    TState *st = B.ts + t;
    if (st->fuse_bad) return;
    const u32 lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32 j = blockIdx.y * SEL_WAVES + wave, K = gd->cfg_K[q.cfg];
    if (j >= K - 1u) return; // (no barrier below)
    const u32 u = B.tgt_bin[(size_t)t * TGT_STRIDE + j];
    if (u == RESOLVED) return;
    const u32 off = B.grp_off[(size_t)t * MAX_GROUPS + u], n = B.grp_off[(size_t)t * MAX_GROUPS + u + 1u] - off;
    u32 k = B.tgt_res[(size_t)t * TGT_STRIDE + j];
    const u32 klo = B.tgt_klo[(size_t)t * TGT_STRIDE + u];
    int R = (int)B.tgt_khi[(size_t)t * TGT_STRIDE + u]; // bits that vary inside the bin
    const GLOBAL_AS u32 *src = gptr(B.pool) + q.span + q.span_len / 2u + off;
    if (k >= n || B.grp_cur[(size_t)t * MAX_GROUPS + u] != n) {
        if (lane == 0u) atomicOr(&st->internal_err, 128u);
        return;
    }
    u32 P = 0u; // chosen high part of key - klo
    if (n <= 64u * SEL_ROWS) {
        u32 x[SEL_ROWS];
#pragma unroll
        for (u32 r = 0; r < SEL_ROWS; r++) x[r] = r * 64u + lane < n ? src[r * 64u + lane] - klo : 0xFFFFFFFFu;
        while (R > 0) {
            R--;
            u32 below = 0u; // keys that agree so far and have a 0 here
#pragma unroll
            for (u32 r = 0; r < SEL_ROWS; r++) below += (u32)__popcll(__ballot((x[r] >> R) == 2u * P));
            const bool up = k >= below;
            k -= up ? below : 0u;
            P = 2u * P + (up ? 1u : 0u);
        }
    } else {
        u32 *h = hist[wave];
        while (R > 0) {
            const int wd = R < 8 ? R : 8;
            for (u32 i = lane; i < 256u; i += 64u) h[i] = 0u;
            asm volatile("" ::: "memory"); // (a wave's LDS operations complete in order)
            for (u32 i0 = 0; i0 < n; i0 += 256u) {
                u32 x[4];
#pragma unroll
                for (u32 r = 0; r < 4u; r++) x[r] = i0 + r * 64u + lane < n ? src[i0 + r * 64u + lane] - klo : 0xFFFFFFFFu;
#pragma unroll
                for (u32 r = 0; r < 4u; r++) {
                    const bool in = i0 + r * 64u + lane < n && (u32)((u64)x[r] >> R) == P;
                    if (in) atomicAdd(&h[(x[r] >> (R - wd)) & ((1u << wd) - 1u)], 1u);
                }
            }
            asm volatile("" ::: "memory");
            u32 c[4], s = 0u;
#pragma unroll
            for (u32 r = 0; r < 4u; r++) {
                c[r] = h[lane * 4u + r];
                s += c[r];
            }
            const u32 inc = wave_incl_scan(s);
            u32 run = inc - s, digit = 0u, rest = 0u;
            const bool here = k >= run && k < inc;
            if (here) {
#pragma unroll
                for (u32 r = 0; r < 4u; r++) {
                    if (k >= run && k < run + c[r]) {
                        digit = lane * 4u + r;
                        rest = k - run;
                    }
                    run += c[r];
                }
            }
            const u64 m = __ballot(here);
            if (!m) { // (cannot be: k is below the number of keys)
                if (lane == 0u) atomicOr(&st->internal_err, 128u);
                return;
            }
            const int at = (int)__builtin_ctzll(m);
            digit = (u32)__shfl((int)digit, at);
            k = (u32)__shfl((int)rest, at);
            R -= wd;
            P = (P << wd) | digit;
            asm volatile("" ::: "memory");
        }
    }
    if (lane == 0u) B.tgt_key[(size_t)t * TGT_STRIDE + gd->cfg_pair[q.cfg] * NBT + bnd_index(K, j + 1u)] = klo + P;
}

// ------------------------------------------------------------------------------------------
// symbols that the guess got wrong
// ------------------------------------------------------------------------------------------
constexpr u32 FP_PARTS = 4;
__global__ __launch_bounds__(BLOCK) void k_fpatch(const GridDesc *__restrict__ gd, const QDesc *__restrict__ qd, Bufs B)
{
    __shared__ QuantTables qt;
    __shared__ u32 gbp[QBP + 8]; // the breakpoints that the sweep took, and their slots' symbols
    __shared__ u16 gsym[QBP + 8];
    __shared__ unsigned long long cm[F_CELLS];
    __shared__ u32 cc[F_CELLS];
    const u32 gu = blockIdx.x;
    const Unit un = B.gunits[gu];
    const int t = (int)un.tensor;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TState *st = B.ts + t;
    if (st->fuse_bad || st->internal_err) return; // (the same for the whole workgroup: no other kernel runs)
    const QDesc q = qd[t];
    const u32 c = B.unit_cand[(size_t)gu * 16 + wave];
    u32 cmax = 0u;
    for (u32 w = 0; w < BLOCK / 64; w++) cmax = max(cmax, B.unit_cand[(size_t)gu * 16 + w]);
    if (cmax <= blockIdx.y * 256u) return;
    const u32 pair = gd->cfg_pair[q.cfg], K = gd->cfg_K[q.cfg], w = symbol_bits(K), n_bp = K + 3u;
    for (u32 i = tid; i < F_CELLS; i += BLOCK) {
        cm[i] = 0ull;
        cc[i] = 0u;
    }
    if (tid < (u32)QBP + 8u) {
        gbp[tid] = B.edges[(size_t)t * MAX_EDGES + tid];
        gsym[tid] = B.edge_item[(size_t)t * MAX_EDGES + tid];
    }
    const u32 tau_o = st->thr_mag[gd->n_p + gd->pair_o[pair]];
    make_breakpoints(qt, B.tgt_key + (size_t)t * TGT_STRIDE + pair * NBT, K, st->thr_mag[gd->pair_p[pair]], tau_o);
    const GLOBAL_AS u32 *kp = gptr(open_keys(B, un, wave)), *ip = kp + open_cap(un);
    GLOBAL_AS unsigned long long *packed = gptr(q.packed);
    for (u32 b = blockIdx.y * 256u; b < c; b += FP_PARTS * 256u) {
        u32 key[4], idx[4];
#pragma unroll
        for (u32 j = 0; j < 4u; j++) {
            const u32 i = b + lane + j * 64u;
            key[j] = i < c ? kp[i] : 0u;
            idx[j] = q.packed && i < c ? ip[i] : 0u;
        }
#pragma unroll
        for (u32 j = 0; j < 4u; j++) {
            if (b + lane + j * 64u >= c) continue;
            const u32 old = listed_symbol(gsym[slot_of_key(gbp, n_bp, key[j])], key[j], tau_o);
            const u32 sym = qt.symtab[slot_of_key(qt.bp, n_bp, key[j])];
            if (old == sym) continue;
            if (q.packed) {
                const u64 bit = (u64)idx[j] * w;
                const u32 sh = (u32)(bit & 63u);
                GLOBAL_AS unsigned long long *p = packed + (bit >> 6);
                __hip_atomic_fetch_xor(p, (unsigned long long)(old ^ sym) << sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (sh + w > 64u)
                    __hip_atomic_fetch_xor(p + 1, (unsigned long long)(old ^ sym) >> (64u - sh), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const u32 x = key[j] >> 23, m = bits_of_key(key[j]) & 0x7fffffu;
            if (old >= 2u) { // (sums modulo 2^64 and 2^32: what leaves one cell enters another)
                atomicAdd(&cc[old + x], 0xFFFFFFFFu);
                atomicAdd(&cm[old + x], 0ull - (unsigned long long)m);
            }
            if (sym >= 2u) {
                atomicAdd(&cc[sym + x], 1u);
                atomicAdd(&cm[sym + x], (unsigned long long)m);
            }
        }
    }
    __syncthreads();
    unsigned long long *gm = (unsigned long long *)B.mom_sx + (size_t)t * MAX_SUB;
    for (u32 i = tid; i < F_CELLS; i += BLOCK) {
        if (cm[i]) atomicAdd(&gm[i], cm[i]);
        if (cc[i]) atomicAdd(&gm[F_CELLS + i], (unsigned long long)(long long)(int)cc[i]);
    }
}

// ------------------------------------------------------------------------------------------
// protected values
// ------------------------------------------------------------------------------------------
// A unit's lists, one per wave, hold for every tile and quarter those of the wave's 256 consecutive values, in
// index order.  The tensor's order is tile, quarter, wave.  The tiles' counts stay behind for k_quant, which takes a
// further call for the same configuration (6.7 G values: 8.5 ms, this sweep again 12.4).  Without output buffers the
// unit's sum of their squares is all that is wanted, in a fixed order; it goes where the unit's numbers of listed values
// were (unit_cand, read no more).
__global__ __launch_bounds__(BLOCK) void k_fprot(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                 const u32 *__restrict__ t_gu_off,
                                                 const QDesc *__restrict__ qd, Bufs B)
{
    constexpr u32 NW = BLOCK / 64;
    __shared__ u32 seg[NW][16]; // entries per list in every wave's share of the tiles
    __shared__ u32 s_before[NW];
    __shared__ double s_sq[NW];
    const u32 gu = blockIdx.x;
    const Unit un = B.gunits[gu];
    const int t = (int)un.tensor;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TState *st = B.ts + t;
    if (st->fuse_bad) return;
    u32 own = lane < 16u ? B.unit_prot[(size_t)gu * 16 + lane] : 0u;
    const QDesc q = qd[t];
    const TDesc d = td[t];
    const u32 tiles = un.tile1 - un.tile0, per = (tiles + NW - 1u) / NW;
    GLOBAL_AS u32 *tile_out = gptr(B.tile_out) + (size_t)un.tile0 * MAX_FRAC + gd->pair_o[gd->cfg_pair[q.cfg]];
    GLOBAL_AS double *squares = (GLOBAL_AS double *)gptr(B.unit_cand + (size_t)gu * 16);
    if (__ballot(own != 0u) == 0ull) {
        for (u32 k = tid; k < tiles; k += BLOCK) tile_out[(size_t)k * MAX_FRAC] = 0u;
        if (!q.packed && tid == 0u) *squares = 0.0;
        return;
    }
    double sq = 0.0;
    // protected values of the tensor's units before this one
    u32 before = 0u;
    for (u32 k = t_gu_off[t] * 16u + tid; k < gu * 16u; k += BLOCK) before += B.unit_prot[k];
    before = wave_sum(before);
    if (lane == 0u) s_before[wave] = before;
    const ProtLists pl = prot_lists(un, q.span);
    const GLOBAL_AS u32 *counts = gptr(B.pool) + pl.counts, *list = gptr(B.pool) + pl.list;
    const u32 lo = wave * per < tiles ? wave * per : tiles, hi = lo + per < tiles ? lo + per : tiles;
    // lane = quarter * 16 + list: its count of a tile is u16 number `quarter` of the list's four
    const u32 l = lane & 15u, j = lane >> 4;
    auto count_of = [&](u32 tile) { return (counts[tile * F_TILEW + 2u * l + (j >> 1)] >> (16u * (j & 1u))) & 0xFFFFu; };
    u32 mine = 0u;
#pragma unroll 4
    for (u32 k = lo; k < hi; k++) mine += count_of(k);
    mine += (u32)__shfl_xor((int)mine, 16);
    mine += (u32)__shfl_xor((int)mine, 32);
    if (lane < 16u) seg[wave][lane] = mine;
    __syncthreads();
    u32 src = 0u; // entries of list l before this wave's tiles
    for (u32 w = 0; w < wave; w++) src += seg[w][l];
    u64 dst = 0ull; // ... of all lists
    for (u32 w = 0; w < NW; w++) dst += s_before[w];
    dst += wave_sum(j == 0u ? src : 0u);
    for (u32 k = lo; k < hi; k++) {
        const u32 c = count_of(k);
        const u32 inc = wave_incl_scan(c); // in the order of the lanes: quarter, list
        if (lane == 63u) tile_out[(size_t)k * MAX_FRAC] = inc;
        if (__ballot(c != 0u) == 0ull) continue;
        const u32 c0 = (u32)__shfl((int)c, (int)l), c1 = (u32)__shfl((int)c, (int)(l + 16u)), c2 = (u32)__shfl((int)c, (int)(l + 32u));
        const u32 c3 = (u32)__shfl((int)c, (int)(l + 48u));
        const u32 from = src + (j > 0u ? c0 : 0u) + (j > 1u ? c1 : 0u) + (j > 2u ? c2 : 0u);
        const GLOBAL_AS u32 *p = list + (u64)l * pl.cap + from;
        for (u32 i = 0; i < c; i++) { // (rarely more than one or two)
            const u32 x = p[i];
            const float value = gptr(d.data)[x];
            if (q.packed)
                store_protected(q, dst + (inc - c) + i, x, value);
            else
                sq = fma((double)value, (double)value, sq);
        }
        src += c0 + c1 + c2 + c3;
        dst += (u32)__builtin_amdgcn_readlane((int)inc, 63);
    }
    if (q.packed) return;
    sq = wave_sum_f64(sq);
    if (lane == 0u) s_sq[wave] = sq;
    __syncthreads();
    if (tid == 0u) {
        double all = 0.0;
        for (u32 w = 0; w < NW; w++) all += s_sq[w];
        *squares = all;
    }
}

// ------------------------------------------------------------------------------------------
// centres
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_fhead(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                 const u32 *__restrict__ t_fu_off, const u32 *__restrict__ t_gu_off,
                                                 const QDesc *__restrict__ qd, QInfo *__restrict__ qi, Bufs B)
{
    __shared__ double part[256], s_sq[2]; // of the bins: 2 c S - n c^2; sums of squares: all, protected
    __shared__ unsigned long long cm[F_CELLS], cc[F_CELLS];
    __shared__ float cb[256];
    __shared__ unsigned long long s_n;
    __shared__ u32 s_prot;
    const int t = blockIdx.x;
    const QDesc q = qd[t];
    if (!q.fused) return;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TState *st = B.ts + t;
    const u32 pair = gd->cfg_pair[q.cfg], K = gd->cfg_K[q.cfg];
    if (st->fuse_bad || st->internal_err) {
        if (tid == 0u) store_result(st, B.res + t);
        return;
    }
    if (tid == 0u) {
        s_n = 0ull;
        s_prot = 0u;
    }
    __syncthreads();
    const u64 *gm = B.mom_sx + (size_t)t * MAX_SUB;
    u64 have = 0ull;
    for (u32 i = tid; i < F_CELLS; i += BLOCK) {
        cm[i] = gm[i];
        cc[i] = gm[F_CELLS + i];
        have += cc[i];
    }
    if (have) atomicAdd(&s_n, (unsigned long long)have);
    u32 prot = 0u;
    for (u32 k = t_gu_off[t] * 16u + tid; k < t_gu_off[t + 1] * 16u; k += BLOCK) prot += B.unit_prot[k];
    prot = wave_sum(prot);
    if (lane == 0u && prot) atomicAdd(&s_prot, prot);
    __syncthreads();
    const u32 *tk = B.tgt_key + (size_t)t * TGT_STRIDE + pair * NBT;
    const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + gd->pair_o[pair]];
    float *codebook = B.codebook + ((size_t)t * gd->n_cfg + q.cfg) * CB_STRIDE; // (for a further call)
    // As many lanes per bin as there are threads, at most a wave: its cells by sign and exponent, lowest key to highest,
    // then the lanes in a fixed order.  (A wave per bin, sixteen bins of 256 one after the other: 28 us, 13 so.)
    const u32 per = K > 128u ? 4u : K > 64u ? 8u : K > 32u ? 16u : K > 16u ? 32u : 64u;
    for (u32 k = tid / per; k < K; k += BLOCK / per) { // (once)
        const u32 lo = k ? tk[bnd_index(K, k)] : class_edge_key(0u, tau_p, tau_o);
        const u32 hi = k + 1u < K ? tk[bnd_index(K, k + 1u)] : class_edge_key(3u, tau_p, tau_o);
        double s = 0.0;
        u64 n = 0ull;
        if (hi > lo)
            for (u32 x = (lo >> 23) + tid % per; x <= ((hi - 1u) >> 23); x += per) {
                const u64 c = cc[2u + k + x], m = cm[2u + k + x];
                if (!c) continue;
                n += c;
                const bool neg = (x & 256u) == 0u; // key >> 23: the top bit is set for values >= 0, else all bits are flipped
                const int E = (int)((neg ? ~x : x) & 255u);
                const double v = E ? ldexp((double)((c << 23) + m), E - 150) : ldexp((double)m, -149);
                s += neg ? -v : v;
            }
        for (u32 o = per / 2u; o > 0u; o >>= 1) {
            s += __shfl_xor(s, (int)o);
            n += __shfl_xor(n, (int)o);
        }
        if (tid % per == 0u) {
            const float c = n ? (float)(s / (double)n) : __uint_as_float(bits_of_key(tk[bnd_index(K, k == 0u ? 1u : k)]));
            codebook[k] = cb[k] = c;
            part[k] = 2.0 * (double)c * s - (double)n * (double)c * (double)c;
        }
    }
    if (tid == 0u && s_n != st->pair_M[pair]) atomicOr(&st->internal_err, 2048u); // every quantized value is in a cell
    __syncthreads();
    if (q.packed) {
        store_head(q, st, gd, tk, cb, s_prot, qi + t);
        if (tid == 0u) store_result(st, B.res + t);
        return;
    }
    // the configuration's score, as k_final works it out; sums of squares of the units in a fixed order
    if (wave < 2u) {
        const u32 *off = wave ? t_gu_off : t_fu_off;
        double x = 0.0;
        for (u32 u = off[t] + lane; u < off[t + 1]; u += 64u)
            x += wave ? *(const double *)(B.unit_cand + (size_t)u * 16) : B.sq_part[(size_t)u * SQ_STRIDE];
        x = wave_sum_f64(x);
        if (lane == 0u) s_sq[wave] = x;
    }
    __syncthreads();
    if (wave == 0u) {
        double acc = 0.0;
        for (u32 k = lane; k < K; k += 64u) acc += part[k];
        acc = wave_sum_f64(acc);
        if (lane == 0u) {
            const double sse = s_sq[0] - s_sq[1] - acc;
            Score r;
            r.sse = sse < 0.0 ? 0.0 : sse;
            r.sumsq = s_sq[0];
            r.n_pruned = st->pair_Pn[pair] + st->pair_Pp[pair];
            r.n_outlier = st->pair_An[pair] + st->pair_Ap[pair];
            r.n_kept = st->pair_M[pair];
            r.cost_bits = payload_bits(r.n_kept, r.n_outlier, K, gd->cfg_l16[q.cfg]);
            B.scores[(size_t)t * gd->n_cfg + q.cfg] = r;
            st->sumsq = r.sumsq;
            if (r.n_pruned + r.n_outlier + r.n_kept != td[t].n || (u64)s_prot != r.n_outlier) atomicOr(&st->internal_err, 256u);
            settle_choice(st, q.cfg, r.sse, r.sumsq, gd->eps);
            store_result(st, B.res + t);
        }
    }
}

hipError_t launch_fused(const Batch &bt, const QDesc *qd, QInfo *qi, hipStream_t s)
{
    const Bufs &B = bt.bufs;
    PROF("k_fplan", s, k_fplan<<<bt.nB, BLOCK, 0, s>>>(bt.td, bt.gd, qd, B));
    if (qi)
        PROF("k_fuse", s, k_fuse<false><<<bt.n_gwg, BLOCK, 0, s>>>(bt.td, bt.wg_gu0, bt.gd, qd, B));
    else
        PROF("k_fuse_dry", s, k_fuse<true><<<bt.n_gwg, BLOCK, 0, s>>>(bt.td, bt.wg_gu0, bt.gd, qd, B));
    PROF("k_fsplit", s, k_fsplit<<<dim3(bt.n_gunits, FS_PARTS), BLOCK, 0, s>>>(qd, B));
    PROF("k_fsel", s, k_fsel<<<dim3(bt.nB, 256 / SEL_WAVES), 64 * SEL_WAVES, 0, s>>>(bt.gd, qd, B));
    PROF("k_fpatch", s, k_fpatch<<<dim3(bt.n_gunits, FP_PARTS), BLOCK, 0, s>>>(bt.gd, qd, B));
    PROF("k_fprot", s, k_fprot<<<bt.n_gunits, BLOCK, 0, s>>>(bt.td, bt.gd, bt.t_gu_off, qd, B));
    PROF("k_fhead", s, k_fhead<<<bt.nB, BLOCK, 0, s>>>(bt.td, bt.gd, bt.t_fu_off, bt.t_gu_off, qd, qi, B));
    return hipGetLastError();
}

} // namespace inshr
