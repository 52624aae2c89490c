// What the quantizing kernels share: breakpoints and their symbols, the outputs that are not symbols.
#pragma once
#include "inshr_launch.h"

namespace inshr {

// The symbol is a step function of the key: the 255 bin boundaries and the four class edges
// (first quantized negative key, first pruned key, first quantized positive key, first protected
// positive key) cut the key axis into at most 260 slots, each with one symbol.  The search's
// equal-population bins (32768 of them) are far finer than the slots, so a table gives the symbol
// of every bin that holds no breakpoint; in the few bins that do, the key is compared with the
// breakpoints from the bin's first one on.
constexpr int QBP = 264;          // breakpoints, padded
constexpr int PKW = 256 * 9;      // most packed words of a tile

struct QuantTables {
    u32 bp[QBP + 8];   // sorted breakpoints, then 0xFFFFFFFF
    u32 raw[QBP];      // boundaries of the configuration, then the class edges
    u16 symtab[QBP];   // symbol of slot s = #{breakpoints <= key}
    u32 wcnt[2][64];   // protected values per (quarter j, wave) of the tile, per buffer
};

// cj (0 .. 4) summed over the lower lanes of the wave in `below`; returns the wave's total.
__device__ __forceinline__ u32 rank_counts(u32 cj, u32 &below)
{
    const u64 m0 = __ballot(cj & 1u), m1 = __ballot(cj & 2u), m2 = __ballot(cj & 4u);
    below = __builtin_amdgcn_mbcnt_hi((u32)(m0 >> 32), __builtin_amdgcn_mbcnt_lo((u32)m0, 0u)) +
            2u * __builtin_amdgcn_mbcnt_hi((u32)(m1 >> 32), __builtin_amdgcn_mbcnt_lo((u32)m1, 0u)) +
            4u * __builtin_amdgcn_mbcnt_hi((u32)(m2 >> 32), __builtin_amdgcn_mbcnt_lo((u32)m2, 0u));
    return (u32)__popcll(m0) + 2u * (u32)__popcll(m1) + 4u * (u32)__popcll(m2);
}

// The 256 symbols of a wave's lanes, four of w bits each, are 4 w whole words of the stream, which the wave packs by itself:
// the symbols of 4, 2 or 1 lanes (as many as fit a word) are joined in registers, these pieces exchanged through the
// wave's own 64 words of LDS, and lane k < 4 w takes word k from the two or three pieces that it lies in.
// (A wave's LDS operations complete in order: no other wave is asked.  Pieces of one lane each, up to nine of them a word:
// k_quant on 1.6 G values of 3 to 9 bits 2.37 ms, 2.29 so; k_fuse on 6.7 G of 9 bits, with the same means otherwise, 10.54 and 10.29.)
struct WavePack {
    u32 w, join, bits, p0, skip; // lanes per piece; bits of a piece; the word's first piece, bits of it before the word
    __device__ __forceinline__ WavePack(u32 w_, u32 lane) : w(w_)
    {
        join = w <= 4u ? 4u : w <= 8u ? 2u : 1u;
        bits = 4u * w * join;
        p0 = 64u * lane / bits;
        skip = 64u * lane - bits * p0;
    }
    static __device__ __forceinline__ unsigned long long swapped(unsigned long long x, bool pairs)
    {
        const int lo = (int)(u32)x, hi = (int)(u32)(x >> 32);
        u32 a, b;
        if (pairs) { // lanes 1 0 3 2 of every four
            a = (u32)__builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true);
            b = (u32)__builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true);
        } else { // lanes 2 3 0 1
            a = (u32)__builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, true);
            b = (u32)__builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, true);
        }
        return (unsigned long long)b << 32 | a;
    }
    // the pieces of a wave's lanes
    __device__ __forceinline__ void put(unsigned long long piece, unsigned long long *mine, u32 lane) const
    {
        if (join > 1u) piece |= swapped(piece, true) << (4u * w); // (right in the first lane of two)
        if (join > 2u) piece |= swapped(piece, false) << (8u * w); // (... of four)
        asm volatile("" ::: "memory");
        if ((lane & (join - 1u)) == 0u) mine[place(lane)] = piece;
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ u32 place(u32 lane) const { return join == 4u ? lane >> 2 : join == 2u ? lane >> 1 : lane; }
    // a symbol that put() found zero: value c of a lane
    __device__ __forceinline__ void add(unsigned long long *mine, u32 lane, u32 c, u32 sym) const
    {
        atomicOr(&mine[place(lane)], (unsigned long long)sym << ((4u * (lane & (join - 1u)) + c) * w));
    }
    // word `lane` of the 4 w, in lanes below 4 w
    __device__ __forceinline__ unsigned long long word(const unsigned long long *mine, u32 lane) const
    {
        unsigned long long x = 0ull;
        if (lane < 4u * w) {
            x = mine[p0] >> skip;
            const u32 s1 = bits - skip, s2 = s1 + bits; // (at most 64: 1 <= s1)
            if (s1 < 64u) x |= mine[p0 + 1u] << s1;
            if (s2 < 64u) x |= mine[p0 + 2u] << s2;
        }
        return x;
    }
};

// Breakpoints in key order and the symbol of every slot, by a workgroup of at least QBP + 8 threads.
// tk: the pair's boundary keys (they ascend); at equal keys a boundary goes before a class edge.
__device__ __forceinline__ void make_breakpoints(QuantTables &qt, const u32 *tk, u32 K, u32 tau_p, u32 tau_o)
{
    const u32 tid = threadIdx.x, n_bnd = K - 1u, n_bp = n_bnd + 4u;
    if (tid < n_bnd) qt.raw[tid] = tk[bnd_index(K, tid + 1u)];
    if (tid < 4u) qt.raw[n_bnd + tid] = class_edge_key(tid, tau_p, tau_o);
    __syncthreads();
    auto boundaries_upto = [&](u32 key) -> u32 {
        u32 lo = 0u, hi = n_bnd;
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if (qt.raw[mid] <= key)
                lo = mid + 1u;
            else
                hi = mid;
        }
        return lo;
    };
    if (tid < n_bp) {
        const u32 x = qt.raw[tid];
        u32 r = tid < n_bnd ? tid : boundaries_upto(x);
#pragma unroll
        for (u32 e = 0; e < 4u; e++) {
            const u32 y = qt.raw[n_bnd + e];
            r += (y < x || (y == x && tid >= n_bnd && n_bnd + e < tid)) ? 1u : 0u;
        }
        qt.bp[r] = x;
    } else if (tid < (u32)QBP + 8u) {
        qt.bp[tid] = 0xFFFFFFFFu;
    }
    __syncthreads();
    if (tid <= n_bp) { // symbol of each slot, from its smallest key
        const u32 rep = tid ? qt.bp[tid - 1u] : 0u;
        const u32 m = mag_of_key(rep);
        qt.symtab[tid] = (u16)(m < tau_p ? 0u : m > tau_o ? 1u : 2u + boundaries_upto(rep));
    }
    __syncthreads();
}

// Breakpoints at or below the key, by bisection.
__device__ __forceinline__ u32 slot_of_key(const u32 *bp, u32 n_bp, u32 key)
{
    u32 s = 0u;
#pragma unroll
    for (u32 step = 256u; step > 0u; step >>= 1)
        if (s + step <= n_bp && bp[s + step - 1u] <= key) s += step;
    return s;
}

__device__ __forceinline__ void store_protected(const QDesc &q, u64 pos, u32 index, float x)
{
    if (pos >= q.out_cap) return;
    gptr(q.out_idx)[pos] = index;
    if (q.val_bf16) { // upper 16 bits, rounded to nearest even
        const u32 b = __float_as_uint(x);
        ((GLOBAL_AS u16 *)gptr(q.out_val))[pos] = (u16)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
    } else {
        gptr(q.out_val)[pos] = x;
    }
}

// What a quantized tensor's descriptor, boundaries and codebook are, by the whole workgroup.
__device__ __forceinline__ void store_head(const QDesc &q, const TState *st, const GridDesc *gd, const u32 *tk,
                                           const float *cb, u32 found, QInfo *qi)
{
    const u32 g = q.cfg, pair = gd->cfg_pair[g], K = gd->cfg_K[g], o = gd->pair_o[pair];
    const u32 tid = threadIdx.x;
    if (q.boundaries)
        for (u32 j = 1 + tid; j < K; j += blockDim.x)
            gptr(q.boundaries)[j - 1] = __uint_as_float(bits_of_key(tk[bnd_index(K, j)]));
    for (u32 k = tid; k < K; k += blockDim.x) gptr(q.codebook)[k] = cb[k];
    if (tid == 0) {
        QInfo r;
        r.n_pruned = st->pair_Pn[pair] + st->pair_Pp[pair];
        r.n_outlier = st->pair_An[pair] + st->pair_Ap[pair];
        r.n_kept = st->pair_M[pair];
        r.tau_p = st->thr_mag[gd->pair_p[pair]];
        r.tau_o = st->thr_mag[gd->n_p + o];
        r.flags = 0u;
        if ((u64)found != r.n_outlier) r.flags |= 1u;  // self-check
        if (r.n_outlier > q.out_cap) r.flags |= 2u;    // caller buffer too small
        *qi = r;
    }
}

} // namespace inshr
