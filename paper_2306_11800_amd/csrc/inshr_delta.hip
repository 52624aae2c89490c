// Delta Encoder (Sec. 6): d = (s_prev - s_cur) mod B with B = max(K_prev, K_cur) + 2, regrouped in
// the stable order of the previous checkpoint's symbol (Algorithm 5) and bit-packed.
//
// The regrouping is a stable partition into at most 258 groups:
//   k_dhist     per chunk (1 .. 64 tiles of 12288 elements): population of every previous symbol
//   k_dgroups   per tensor: group offsets and the start of every chunk inside every group; clears
//               the stream words that k_dscatter ORs into; checks the offsets that came with a stream
//   k_dscatter  one workgroup of 12 waves per chunk walks its tiles in order.  Per tile each wave
//               owns 1024 consecutive elements, 64 consecutive elements per step; a returning LDS
//               add per element (or lane bits OR-ed into the symbol's LDS slot) gives the stable
//               rank.  The tile's deltas are written to an LDS array in regrouped order, one thread
//               per output word packs the fields of its bits and stores it (first / last word of a
//               chunk's run are OR-ed into words that k_dgroups cleared).
// A tensor of one tile needs neither of the first two: its workgroup of k_dscatter (k_drestore) has all counts.
#include "inshr_launch.h"

namespace inshr {

constexpr int DTILE = DELTA_TILE;   // elements per tile = 1024 per wave of the scatter workgroup
constexpr int SS = DELTA_SS;        // symbol stride (258 symbols at most)
constexpr int NWAVE = DTILE / 1024; // waves of a scatter workgroup (two workgroups share a CU)
constexpr int DBLOCK = NWAVE * 64;
constexpr int TWORDS = DTILE * 9 / 64;            // most packed u64 words of one tile
constexpr int HTILE = 16384;                      // step of the gathering kernel
constexpr int HBLOCK = 256;                       // threads of a counting workgroup
static_assert(DTILE % 64 == 0, "a chunk starts at a whole word of any symbol width");

__device__ __forceinline__ u32 lds_extract(const u32 *W, u32 idx, u32 w)
{
    const u32 off = idx * w;
    const u32 wd = off >> 5, sh = off & 31u;
    const u64 two = ((u64)W[wd + 1] << 32) | (u64)W[wd];
    return (u32)(two >> sh) & ((1u << w) - 1u);
}

// Symbols of one chunk counted by width W: every lane takes runs of 64 consecutive symbols (W whole
// words), extracts them from registers with compile-time shifts and counts the non-zero ones in its
// wave's LDS histogram.  Symbol 0 (pruned: the most frequent one when pruning is on) is not counted:
// its population is what the others leave of the chunk.
// Narrow symbols (few clusters, unequal populations: the bins of the sketch quantizer) make many
// lanes of a wave hit the same counter at once; their lanes are spread over DH_COPIES rows.
constexpr int DH_COPIES = 4;
template <int W, bool WHOLE>
__device__ __forceinline__ void count_run(const u32 (&x)[2 * W + 1], u32 nvalid, u32 S, u32 *hrow)
{
    if (W <= 7) hrow += (threadIdx.x & (u32)(DH_COPIES - 1)) * (u32)SS;
#pragma unroll
    for (int i = 0; i < 64; i++) {
        constexpr u32 mask = (1u << W) - 1u;
        const int p = i * W, dw = p >> 5, sh = p & 31;
        u32 sym = (sh + W <= 32) ? (x[dw] >> sh) & mask
                                 : __builtin_amdgcn_alignbit(x[dw + 1], x[dw], sh) & mask;
        sym = sym < S ? sym : S; // a malformed stream counts into the unused entry S
        if (sym != 0u && (WHOLE || (u32)i < nvalid)) atomicAdd(&hrow[sym], 1u);
    }
}

template <int W>
__device__ __forceinline__ void count_symbols(const DDesc &d, u64 c0, u64 c1, u32 S, u32 *hrow)
{
    const u32 tid = threadIdx.x;
    const GLOBAL_AS unsigned long long *src = gptr(d.prev);
    const u64 total_words = (d.n * W + 63u) >> 6;
    const u32 n_runs = (u32)((c1 - c0 + 63u) >> 6);
    for (u32 u = tid; u < n_runs; u += HBLOCK) {
        const u64 e = c0 + 64ull * u;
        const u32 nvalid = tile_len(c1 - e, 64u);
        const u64 w0 = (e >> 6) * W; // e is a multiple of 64
        u32 x[2 * W + 1];
#pragma unroll
        for (int k = 0; k < W; k++) {
            const unsigned long long v = (w0 + k < total_words) ? src[w0 + k] : 0ull;
            x[2 * k] = (u32)v;
            x[2 * k + 1] = (u32)(v >> 32);
        }
        x[2 * W] = 0u;
        if (__ballot(nvalid < 64u) == 0ull) // the same for every active lane
            count_run<W, true>(x, nvalid, S, hrow);
        else
            count_run<W, false>(x, nvalid, S, hrow);
    }
}

// Population of every previous symbol in one chunk.  Workgroups of 256 threads: the rows of a
// workgroup take 17 KB of LDS, eight of them fill a CU, and a chunk of one tile (192 runs of 64
// symbols) still occupies most of its threads.
__global__ __launch_bounds__(HBLOCK) void k_dhist(const DDesc *__restrict__ dd,
                                                  const u32 *__restrict__ chunk_tensor,
                                                  u32 *__restrict__ chunk_tot, u32 *__restrict__ totals)
{
    __shared__ u32 hw[HBLOCK / 64][DH_COPIES * SS];
    __shared__ u32 s_nonzero;
    const u64 chunk = blockIdx.x;
    const u32 t = __builtin_amdgcn_readfirstlane(chunk_tensor[chunk]);
    const DDesc d = dd[t];
    if (delta_single(d)) return;
    const u32 tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 S = d.Kp + 2u;
    const u64 c_elems = (u64)d.ctiles * DTILE;
    const u64 c0 = (chunk - d.chunk0) * c_elems;
    const u64 c1 = (c0 + c_elems < d.n) ? c0 + c_elems : d.n;
    for (u32 k = tid; k < (HBLOCK / 64) * DH_COPIES * SS; k += HBLOCK) (&hw[0][0])[k] = 0u;
    if (tid == 0u) s_nonzero = 0u;
    __syncthreads();
    switch (d.wp) {
    case 2: count_symbols<2>(d, c0, c1, S, hw[wave]); break;
    case 3: count_symbols<3>(d, c0, c1, S, hw[wave]); break;
    case 4: count_symbols<4>(d, c0, c1, S, hw[wave]); break;
    case 5: count_symbols<5>(d, c0, c1, S, hw[wave]); break;
    case 6: count_symbols<6>(d, c0, c1, S, hw[wave]); break;
    case 7: count_symbols<7>(d, c0, c1, S, hw[wave]); break;
    case 8: count_symbols<8>(d, c0, c1, S, hw[wave]); break;
    default: count_symbols<9>(d, c0, c1, S, hw[wave]); break;
    }
    __syncthreads();
    const u32 copies = d.wp <= 7u ? (u32)DH_COPIES : 1u;
    u32 mine[2] = {0u, 0u}, sum = 0u; // populations of symbols tid, tid + 256 (those above S - 1 are in entry S)
    for (u32 h = 0; h < 2u; h++) {
        const u32 sy = tid + h * HBLOCK;
        if (sy < 1u || sy > S) continue;
        for (u32 wv = 0; wv < HBLOCK / 64u; wv++)
            for (u32 cp = 0; cp < copies; cp++) mine[h] += hw[wv][cp * SS + sy];
        sum += mine[h];
    }
    sum = wave_sum(sum);
    if ((tid & 63u) == 0u && sum) atomicAdd(&s_nonzero, sum);
    __syncthreads();
    if (tid == 0u) mine[0] = (u32)(c1 - c0) - s_nonzero;
    for (u32 h = 0; h < 2u; h++) {
        const u32 sy = tid + h * HBLOCK;
        if (sy < (u32)SS) chunk_tot[chunk * SS + sy] = sy < S ? mine[h] : 0u;
        if (d.n_chunks > DELTA_FEW && sy < S && mine[h]) // (cleared beforehand)
            atomicAdd(&totals[(d.part0 + (u32)(chunk - d.chunk0) / DELTA_PART) * SS + sy], mine[h]);
    }
}

// Per tensor: group offsets; chunk_tot becomes the start of each chunk inside its group.  With CLEAR
// also the stream words that k_dscatter ORs into are cleared: the first word of every (chunk, group)
// run, which is also where the run before it ends, and the word where the stream ends.  Without, the offsets that
// came with the stream are compared.
// A workgroup takes 64 symbols, a lane each, of a part of up to 128 chunks, sixteen of them a wave: one round of loads,
// asked for together with the sums of all parts (at most some forty), which give the offsets and what lies before the
// part.  Bound by the latency of four dependent reads.  (One workgroup per 64 symbols walked all chunks of a
// tensor: 3072 chunks 107 us, 887 of them 43 us; so 23 and 10.  k_dhist, whose additions to one row per tensor met
// each other, 66 and 27; now 30 and 13.)
// With at most DELTA_FEW chunks one workgroup does it all, a wave per 64 symbols, and adds the populations up itself.
constexpr u32 DG_WAVES = 8, DG_AHEAD = 16, DG_BLOCKS = (SS + 63) / 64;
static_assert(DELTA_PART == DG_WAVES * DG_AHEAD, "a part is one round of loads");
static_assert(DELTA_FEW <= DG_AHEAD && DG_BLOCKS <= DG_WAVES, "one round of loads, a wave per 64 symbols");
template <bool CLEAR>
__global__ __launch_bounds__(64 * DG_WAVES) void k_dgroups(const DDesc *__restrict__ dd, const XDesc *__restrict__ xd,
                                                           const u32 *__restrict__ part_tensor, u32 *__restrict__ chunk_tot,
                                                           const u32 *__restrict__ totals, u32 *__restrict__ flags)
{
    __shared__ u32 share[DG_WAVES][64];                   // sums of the waves' chunks
    __shared__ u32 all[DG_WAVES][DG_BLOCKS * 64], pre[DG_WAVES][64]; // the waves' parts added up: all; those before this one
    const u32 p = blockIdx.x / DG_BLOCKS, block = blockIdx.x % DG_BLOCKS;
    const u32 t = part_tensor ? __builtin_amdgcn_readfirstlane(part_tensor[p]) : p;
    const u32 lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const DDesc d = dd[t];
    if (delta_single(d)) return;
    const u32 S = d.Kp + 2u, nc = (u32)d.n_chunks, part = p - d.part0;
    const bool few = nc <= DELTA_FEW, clear = CLEAR && !d.prev_perm;
    if (few ? block != 0u : block * 64u > S) return;
    const u32 sb = few ? wave : block, g = sb * 64u + lane; // this lane's symbol
    const bool is = sb < DG_BLOCKS && g < S;
    GLOBAL_AS u32 *ct = gptr(chunk_tot) + d.chunk0 * SS + (is ? g : 0u);
    GLOBAL_AS unsigned long long *out = gptr(d.out);
    const u32 c0 = few ? 0u : part * DELTA_PART + wave * DG_AHEAD, c1 = c0 + DG_AHEAD < nc ? c0 + DG_AHEAD : nc;
    u32 v[DG_AHEAD], sum = 0u; // of the wave's chunks
#pragma unroll
    for (u32 j = 0; j < DG_AHEAD; j++) v[j] = is && c0 + j < c1 ? ct[(u64)(c0 + j) * SS] : 0u;
    if (!few) {
        const u32 n_parts = (nc + DELTA_PART - 1u) / DELTA_PART;
        u32 a[DG_BLOCKS] = {}, before = 0u;
        for (u32 r = wave; r < n_parts; r += DG_WAVES) {
            const GLOBAL_AS u32 *row = gptr(totals) + (u64)(d.part0 + r) * SS;
#pragma unroll
            for (u32 b = 0; b < DG_BLOCKS; b++) {
                const u32 x = b <= block && b * 64u + lane < S ? row[b * 64u + lane] : 0u;
                a[b] += x;
                before += b == block && r < part ? x : 0u;
            }
        }
#pragma unroll
        for (u32 b = 0; b < DG_BLOCKS; b++) all[wave][b * 64u + lane] = a[b];
        pre[wave][lane] = before;
    }
#pragma unroll
    for (u32 j = 0; j < DG_AHEAD; j++) sum += v[j];
    share[wave][lane] = sum;
    __syncthreads();
    u32 off = 0u, run = 0u; // symbols of lower groups (below 2^32, as n is); of this one before the wave's chunks
    if (few) {
        for (u32 w = 0; w < wave; w++) off += wave_sum(share[w][lane]);
        off += wave_incl_scan(sum) - sum;
    } else {
        for (u32 b = 0; b <= block; b++) {
            u32 x = 0u;
#pragma unroll
            for (u32 w = 0; w < DG_WAVES; w++) x += all[w][b * 64u + lane];
            off += b < block ? wave_sum(x) : wave_incl_scan(x) - x;
        }
#pragma unroll
        for (u32 w = 0; w < DG_WAVES; w++) run += pre[w][lane] + (w < wave ? share[w][lane] : 0u);
    }
    if ((few || (wave == 0u && part == 0u)) && g <= S) { // (entry S: everything)
        gptr(d.group_off)[g] = off;
        if (!CLEAR) {
            const u64 *given = xd[t].group_off_in;
            if (given && gptr(given)[g] != (u64)off) raise_flag(flags, RF_GROUPS);
        }
        if (clear && g == S) {
            const u64 word = (d.n * d.wB) >> 6; // where the stream ends
            if (word < d.out_words) out[word] = 0ull;
        }
    }
    if (!is) return;
#pragma unroll
    for (u32 j = 0; j < DG_AHEAD; j++) {
        if (c0 + j >= c1) break;
        ct[(u64)(c0 + j) * SS] = run; // (n < 2^32)
        const u64 word = ((u64)(off + run) * d.wB) >> 6;
        if (clear && word < d.out_words) out[word] = 0ull;
        run += v[j];
    }
}

// The packed words of one tile's symbols go from device memory straight into LDS (no registers in
// between, nothing waits here): every lane moves 16 bytes per instruction when the source is
// 16-byte aligned, 4 bytes otherwise; a wave's lanes write consecutive LDS addresses.  NW waves
// share the work, the calling wave being number widx of them.  The words are complete after
// `s_waitcnt vmcnt(0)` and a barrier.
template <int NW>
__device__ __forceinline__ void lds_fetch(const GLOBAL_AS unsigned long long *src, u64 e0, u32 cnt,
                                          u32 w, u32 *dst, u32 widx)
{
    u32 lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane)); // the addresses below are cheap: recomputing them in every tile
                                   // beats keeping them in (spilled) registers across the loop
    const GLOBAL_AS u32 *g = (const GLOBAL_AS u32 *)(src + e0 * w / 64u); // exact: e0 % 64 == 0
    LDS_AS u32 *l = (LDS_AS u32 *)dst;
    const u32 nd = 2u * ((cnt * w + 63u) >> 6); // dwords of the tile, all inside the packed array
    constexpr u32 MAXD = DTILE * 9 / 32;        // at most 3456 dwords
    constexpr u32 R16 = (MAXD / 4 + NW * 64 - 1) / (NW * 64), R4 = (MAXD + NW * 64 - 1) / (NW * 64);
    u32 done = 0u;
    if ((((u64)g) & 15u) == 0u) {
        const u32 n16 = nd >> 2;
#pragma unroll
        for (u32 it = 0; it < R16; it++) {
            const u32 c0 = (it * NW + widx) * 64u;
            if (c0 + lane < n16)
                __builtin_amdgcn_global_load_lds(g + (c0 + lane) * 4u, l + c0 * 4u, 16, 0, 0);
        }
        done = n16 << 2;
    }
    if (done < nd) { // (the same for the whole workgroup: nothing is left after the 16-byte pieces
                     // of a whole tile)
#pragma unroll
        for (u32 it = 0; it < R4; it++) {
            const u32 c0 = done + (it * NW + widx) * 64u;
            if (c0 + lane < nd) __builtin_amdgcn_global_load_lds(g + (c0 + lane), l + c0, 4, 0, 0);
        }
    }
}

// Output words of one tile: item k of group g's run is stream word gWf[g] + k - wstart[g].  A run of b
// bits touches at most b / 64 + 2 words.
constexpr int BWORDS = TWORDS + 2 * SS + 2;
constexpr int GS = 258 + 2;           // groups, and room behind them (SS is the stride in device memory)
constexpr int WST = NWAVE * 259;      // per-(wave, symbol) counters; the row stride is S + 1
constexpr int ISETS = BWORDS / 64 + 1; // sets of 64 items
constexpr int FRONT = 32;             // fields before the regrouped tile that pack_fields may look at

constexpr int LINE = 4; // stream words (32 bytes) per output line

// f(w) with the width as a compile-time constant
template <u32 W> struct Width {
    static constexpr u32 value = W;
};
template <class F> __device__ __forceinline__ void with_width(u32 w, F &&f)
{
    switch (w) {
    case 2: f(Width<2>()); break;
    case 3: f(Width<3>()); break;
    case 4: f(Width<4>()); break;
    case 5: f(Width<5>()); break;
    case 6: f(Width<6>()); break;
    case 7: f(Width<7>()); break;
    case 8: f(Width<8>()); break;
    default: f(Width<9>()); break;
    }
}

// Which group an item belongs to: the groups with a run in the tile, in order, and the items that
// are the first of a run; an item's group is found by counting these up to the item.
struct ItemSets {
    unsigned long long first[ISETS]; // (zero before the tile's runs are entered)
    u16 before[ISETS];               // first ones in the sets before
    u16 list[GS];
    __device__ __forceinline__ void clear(u32 tid)
    {
        if (tid < 2u * ISETS) ((u32 *)first)[tid] = 0u;
    }
    // group g: `rank` groups have a run before its own, which takes n items from `at` on
    __device__ __forceinline__ void enter(u32 g, u32 rank, u32 at, u32 n)
    {
        if (!n) return;
        atomicOr(&first[at >> 6], 1ull << (at & 63u));
        list[rank] = (u16)g;
        if ((at & 63u) == 0u) before[at >> 6] = (u16)rank;
        for (u32 k = (at >> 6) + 1u; k * 64u < at + n; k++) before[k] = (u16)(rank + 1u);
    }
    __device__ __forceinline__ u32 group(u32 item) const
    {
        const u64 upto = first[item >> 6] << (63u - (item & 63u));
        return list[before[item >> 6] + (u32)__popcll(upto) - 1u];
    }
};

struct ScatterShared {
    u32 wst[WST];                   // counts, then where the elements of (wave, symbol) start in the
                                    // regrouped tile, in bytes
    u32 wstart[GS];             // first word item of each group's run; [S] = items in use
    unsigned long long lw[GS][LINE]; // per group: the words of its current, incomplete output line
    unsigned long long carry[GS];   // bits of earlier tiles in the first word of the tile's run
    u32 fo[GS];                     // first stream word that this chunk's run of the group owns
                                    // alone; bit 31: the word before it is shared with the run before
    u32 gb[GS];                     // stream position after each group's runs so far (n < 2^32)
    u32 gWf[GS];                    // the group's run of the current tile: stream word of its first bit,
    u32 gse[GS];                    // ... s0 | end << 8: its first bit and its end, from that word on
    u16 les[GS];                // ... its first element in the regrouped tile; [S] = elements
    u32 wtot[5], etot[5], rtot[5];
    unsigned long long hotkey;      // population << 9 | symbol, maximum over the tensor's groups
    ItemSets items;
};

// Where a group's runs so far, `pos` symbols in all, end in the stream.
struct RunEnd {
    u32 word, bits; // first word that is still incomplete; its bits that are filled
};
__device__ __forceinline__ RunEnd run_end(u32 pos, u32 wB)
{
    RunEnd r;
    const u64 e = (u64)pos * wB;
    r.word = (u32)(e >> 6);
    r.bits = (u32)(e & 63u);
    return r;
}

// 64 bits of a stream of W-bit fields that lie one per u16 in LDS (f: aligned to a dword): field i
// starts at bit `at` of the word (-W < at <= 0), the fields after it follow; what lies past the last
// field may be anything (the caller masks).  Fields are read as aligned dwords (unaligned LDS reads
// take several times as long); a dot product joins the two of a dword.
template <u32 W>
__device__ __forceinline__ unsigned long long pack_fields(const u16 *f, int i, int at)
{
    typedef u16 us2 __attribute__((ext_vector_type(2)));
    constexpr u32 NP = (64u + 2u * W - 1u + 2u * W - 1u) / (2u * W); // pairs that reach bit 2 W - 1 + 64
    const u32 sh = (u32)(-at) + ((i & 1) ? W : 0u);                  // bits before the word: below 2 W
    const u32 *p = (const u32 *)f + (i >> 1);
    u32 d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (u32 q = 0; q < NP; q++) {
        const us2 one = {1, (u16)(1u << W)};
        const u32 v = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, p[q]), one, 0u, false);
        const u32 k = (q * 2u * W) >> 5, s = (q * 2u * W) & 31u;
        d[k] |= v << s;
        if (s + 2u * W > 32u) d[k + 1u] |= v >> (32u - s);
    }
    return ((u64)__builtin_amdgcn_alignbit(d[2], d[1], sh) << 32) | __builtin_amdgcn_alignbit(d[1], d[0], sh);
}

// Cross-check of the ordered ranking, once per chunk and wave, before the tile loop: the 64 previous
// symbols of the wave's first row of the chunk's first tile are ranked once with returning adds into
// the wave's (zero) counter row and once from ballots; the counters are zero again afterwards.  Returns 1 when the two disagree (the
// device did not serve same-address LDS atomics in lane order).
__device__ __forceinline__ u32 ordered_rank_check(const u32 *P, u32 *wrow, u32 ebase, u32 cnt, u32 S, u32 wp)
{
    const u32 lane = threadIdx.x & 63u;
    const u32 off = ebase * wp;
    u32 sp = S; // lanes past the end share the unused symbol S
    if (ebase < cnt) {
        sp = __builtin_amdgcn_alignbit(P[(off >> 5) + 1u], P[off >> 5], off & 31u) & ((1u << wp) - 1u);
        sp = sp < S - 1u ? sp : S - 1u;
    }
    const u32 got = atomicAdd(&wrow[sp], 1u);
    u64 peers = ~0ull;
#pragma unroll
    for (int b = 0; b < 9; b++) {
        const bool bit = (sp >> b) & 1u;
        const u64 m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    const u32 bad = got != (u32)__popcll(peers & ((1ull << lane) - 1ull)) ? 1u : 0u;
    wrow[sp] = 0u; // (after the add: the wave's LDS operations complete in order)
    return bad;
}

// Sweep 1 of a tile: stable rank of every element among the equal symbols of its wave's 1024
// elements.  Row r of a lane is element ebase + 64 r: its bit offset in the packed words moves by 64 w
// per row, so the shift is a lane constant and the word address advances by 2 w.
// reg[r] = byte offset of the (wave, symbol) counter | rank << 16; with CUR dv[r / 2] takes the delta
// of row r in its half r & 1.
template <bool FULL, bool ORDERED, bool CUR>
__device__ __forceinline__ void rank_rows(const u32 *P, const u32 *C, u32 *wst, u32 row_bytes,
                                          unsigned long long *myslot, u32 ebase, u32 cnt, u32 S,
                                          u32 Bm, u32 wp, u32 wc, u32 hot, u32 (&reg)[16], u32 (&dv)[8])
{
    u32 hot_seen = 0u; // elements of the wave so far that hold the most frequent symbol
    const u32 lane = threadIdx.x & 63u;
    const u64 ltmask = (1ull << lane) - 1ull;
    const unsigned long long lanebit = 1ull << lane;
    const u32 offP = ebase * wp, offC = ebase * wc;
    const u32 shP = offP & 31u, shC = offC & 31u;
    const u32 mP = (1u << wp) - 1u, mC = (1u << wc) - 1u;
    const u32 *pp = P + (offP >> 5), *pc = C + (offC >> 5);
#pragma unroll
    for (u32 rb = 0; rb < 16u; rb += 4u) {
        u32 xp[4][2], xc[4][2];
        asm volatile("" ::: "memory"); // (the reads of more rows would be spilled)
#pragma unroll
        for (u32 q = 0; q < 4u; q++) { // the reads of four rows are in flight together
            const u32 r = rb + q;
            xp[q][0] = pp[r * 2u * wp];
            xp[q][1] = pp[r * 2u * wp + 1u];
            if (CUR) {
                xc[q][0] = pc[r * 2u * wc];
                xc[q][1] = pc[r * 2u * wc + 1u];
            }
        }
#pragma unroll
        for (u32 q = 0; q < 4u; q++) {
            const u32 r = rb + q;
            const bool valid = FULL || (ebase + r * 64u < cnt);
            u32 sp = __builtin_amdgcn_alignbit(xp[q][1], xp[q][0], shP) & mP;
            u32 sc = CUR ? __builtin_amdgcn_alignbit(xc[q][1], xc[q][0], shC) & mC : 0u;
            sp = sp < S - 1u ? sp : S - 1u; // clamps a malformed stream
            if (!FULL && !valid) { // lanes past the end share the unused symbol S
                sp = S;
                sc = 0u;
            }
            const u32 at = sp * 4u + row_bytes;
            u32 *cell = (u32 *)((char *)wst + at);
            u32 within; // elements of this wave with the same symbol and a lower index
            if (ORDERED) {
                // the most frequent symbol (the pruned one, typically a fifth of all elements) would
                // serialise the atomic: its lanes rank themselves from the ballot instead
                const u64 hm = __ballot(sp == hot);
                within = __builtin_amdgcn_mbcnt_hi((u32)(hm >> 32), __builtin_amdgcn_mbcnt_lo((u32)hm, hot_seen));
                hot_seen += (u32)__popcll(hm);
                if (__builtin_amdgcn_inverse_ballot_w64(~hm)) within = atomicAdd(cell, 1u);
            } else {
                atomicOr(&myslot[sp], lanebit);
                const unsigned long long peers = myslot[sp];
                const u32 rank = __popcll(peers & ltmask);
                const u32 old = *cell;
                if (rank == 0u) {
                    myslot[sp] = 0ull;
                    *cell = old + (u32)__popcll(peers);
                }
                within = old + rank;
            }
            reg[r] = at | (within << 16);
            if (CUR) {
                u32 m = delta_of(sp, sc, Bm);
                asm volatile("" : "+v"(m)); // (computed here: its operands take twice the registers)
                dv[r >> 1] = (r & 1u) ? dv[r >> 1] | (m << 16) : m;
            }
        }
    }
    if (ORDERED && lane == 0u) *(u32 *)((char *)wst + row_bytes + hot * 4u) = hot_seen;
}

// One thread per (group, word j of a line), before the tile's words are made: word j of the line that
// the tile completes, if earlier tiles had buffered it, is stored; the bits of earlier tiles in the
// run's first word go where the thread that makes the word finds them.
__device__ __forceinline__ void flush_lines(ScatterShared &sh, GLOBAL_AS unsigned long long *out, u32 item)
{
    asm volatile("" : "+v"(item)); // the item's addresses are recomputed here, not kept across the
                                   // tile loop in spilled registers (a reload would wait for stores)
    const u32 g = item / LINE, j = item % LINE;
    const u32 se = sh.gse[g], s0 = se & 255u, end = se >> 8;
    if (end <= s0) return; // the group has no element in the tile
    const u32 Wf = sh.gWf[g], We = Wf + (end >> 6), wl = Wf & (LINE - 1u);
    if (j > wl) return;
    const unsigned long long v = sh.lw[g][j];
    const u32 L = Wf & ~(u32)(LINE - 1);
    if (j == wl) sh.carry[g] = s0 ? v : 0ull;
    else if (L >= (sh.fo[g] & 0x7fffffffu) && L < (We & ~(u32)(LINE - 1))) out[L + j] = v;
}

// Sweep 2: the tile's elements in regrouped order.
template <bool FULL, class F>
__device__ __forceinline__ void regroup_rows(const u32 *wst, u16 *to, const u32 (&reg)[16], u32 ebase, u32 cnt, F &&value)
{
#pragma unroll
    for (u32 rb = 0; rb < 16u; rb += 8u) {
        u32 start[8];
#pragma unroll
        for (u32 q = 0; q < 8u; q++) start[q] = *(const u32 *)((const char *)wst + (reg[rb + q] & 0xFFFFu));
#pragma unroll
        for (u32 q = 0; q < 8u; q++) {
            const u32 r = rb + q;
            if (FULL || ebase + r * 64u < cnt) *(u16 *)((char *)to + start[q] + (reg[r] >> 16) * 2u) = value(r);
        }
    }
}

// Words of W-bit fields that lie in LDS in the order of the stream, `cnt` of them: a thread per word.
template <u32 W>
__device__ __forceinline__ void store_packed(const u16 *fields, u32 cnt, GLOBAL_AS unsigned long long *dst)
{
    const u32 bits = cnt * W, n_words = (bits + 63u) >> 6;
    u32 k0 = threadIdx.x;
    asm volatile("" : "+v"(k0)); // (what depends on it is computed here, for the width at hand)
    for (u32 k = k0; k < n_words; k += DBLOCK) {
        const u32 bit0 = k * 64u, i = bit0 / W;
        unsigned long long v = pack_fields<W>(fields, (int)i, (int)(i * W) - (int)bit0);
        if (bits - bit0 < 64u) v &= (1ull << (bits - bit0)) - 1ull;
        dst[k] = v;
    }
}

// A tensor of one tile, after its ranking: the counts of every (wave, symbol) become the start of its elements,
// start(elements of the tile before them); returns the group offset of this thread's symbol (thread S: everything).
// wtot: LDS for five words.
template <class F> __device__ __forceinline__ u32 single_starts(u32 *wst, u32 srow, u32 S, u32 *wtot, F &&start)
{
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u32 c[NWAVE], tot = 0u, off = 0u;
    if (tid < 320u) { // waves 0..4 hold the 258 symbols
#pragma unroll
        for (int w = 0; w < NWAVE; w++) {
            c[w] = tid < S ? wst[w * srow + tid] : 0u;
            tot += c[w];
        }
        off = wave_incl_scan(tot);
        if (lane == 63u) wtot[wave] = off;
        off -= tot;
    }
    __syncthreads();
    if (tid < 320u) {
#pragma unroll
        for (u32 w = 0; w < 4u; w++) off += w < wave ? wtot[w] : 0u;
        if (tid < S) {
            u32 at = off;
#pragma unroll
            for (int w = 0; w < NWAVE; w++) {
                wst[w * srow + tid] = start(at);
                at += c[w];
            }
        }
    }
    __syncthreads();
    return off;
}

// ORDERED: same-address LDS atomics with return are served in ascending lane order on this device
// (checked by k_lds_order_check before the library relies on it); one returning add then ranks an
// element.  Otherwise equal symbols of a step find each other through the slot array.
//
// Output: a group's run of one tile is a few dozen bytes, and 258 groups interleave, so storing it
// as it comes would reach memory as partial lines.  Each group therefore keeps the words of its
// current 32-byte line in LDS until the line is complete; complete lines are stored whole.  Only the
// ends of a (chunk, group) run are different: its first partial line is stored word by word, its
// first word, when shared with the run before, and its last partial word are OR-ed into words that
// k_dgroups cleared.
//
// Bound by instruction issue and the LDS pipe together (6.7 G elements of 9-bit symbols, 11.5 ms: per 64
// elements 43 vector and 9.5 LDS instructions, vector issue 0.68 and LDS 0.65 of the time; 1.06 G elements
// of narrower ones, 1.72 ms: 35 and 7.5, 0.61 and 0.63).  Packing words from regrouped fields costs fewer
// vector instructions than OR-ing every delta into an image of the words (49, and 10.2 of LDS; 11.6 ms) and
// leaves room for the permutation in the same array: 100 M elements of 4 bits with it 0.37 -> 0.26 ms.
template <bool PERM, bool ORDERED>
__global__ __launch_bounds__(DBLOCK, 6) void k_dscatter(const DDesc *__restrict__ dd,
                                                     const u32 *__restrict__ chunk_tensor,
                                                     const u32 *__restrict__ chunk_tot,
                                                     u32 *__restrict__ flags)
{
    __shared__ ScatterShared sh;
    // packed symbols of the current tile (variables of their own: the loads that fill them are
    // asynchronous, and only reads of these two arrays have to wait for them)
    __shared__ __attribute__((aligned(16))) u32 Pw[DTILE * 9 / 32 + 1];
    __shared__ __attribute__((aligned(16))) u32 Cw[DTILE * 9 / 32 + 1];
    // the tile's deltas in regrouped order (with room for what pack_fields reads around them, zero in
    // front); before that, with the ballot ranking, slot[wave][symbol]: lanes of the wave's current step
    // that hold the symbol
    constexpr int FWORDS = (FRONT + DTILE + 40) / 4;
    __shared__ unsigned long long slot[ORDERED ? FWORDS : NWAVE * SS];
    u16 *fields = (u16 *)slot + FRONT;
    static_assert(NWAVE * SS >= FWORDS, "the regrouped tile fits the slot array");

    const u64 chunk = blockIdx.x;
    const DDesc d = dd[__builtin_amdgcn_readfirstlane(chunk_tensor[chunk])];
    if (d.prev_perm) return; // this tensor's regrouping is given: k_dgather writes its stream
    if (PERM != (d.perm != nullptr)) return;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 S = d.Kp + 2u, Bm = d.B, wB = d.wB, wp = d.wp, wc = d.wc;
    const u32 srow = S + 1u; // row stride of the (wave, symbol) tables
    const u64 n_tiles = (d.n + DTILE - 1) / DTILE;
    const u64 lt0 = (chunk - d.chunk0) * d.ctiles;
    const u64 lt1 = (lt0 + d.ctiles < n_tiles) ? lt0 + d.ctiles : n_tiles;
    GLOBAL_AS unsigned long long *out = gptr(d.out);
    if (delta_single(d)) {
        // One tile: its own counts give the group offsets, and the regrouped tile is the stream.  (4096 values by
        // k_dhist, k_dgroups and the general walk: 28 us in three launches, 12 us so.)
        const u32 cnt = (u32)d.n;
        lds_fetch<NWAVE>(gptr(d.prev), 0u, cnt, wp, Pw, wave);
        lds_fetch<NWAVE>(gptr(d.cur), 0u, cnt, wc, Cw, wave);
        for (u32 k = tid; k < NWAVE * srow; k += DBLOCK) sh.wst[k] = 0u;
        if (!ORDERED)
            for (u32 k = tid; k < (u32)(NWAVE * SS); k += DBLOCK) slot[k] = 0ull;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's share of the words
        __syncthreads();
        u32 order_bad = 0u, reg[16], dv[8];
        const u32 ebase = wave * 1024u + lane, row_bytes = wave * srow * 4u;
        if (ORDERED) order_bad = ordered_rank_check(Pw, sh.wst + wave * srow, ebase, cnt, S, wp);
        // (symbol 0, the pruned one, is taken for the most frequent)
        rank_rows<false, ORDERED, true>(Pw, Cw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wc, 0u, reg, dv);
        __syncthreads();
        const u32 off = single_starts(sh.wst, srow, S, sh.wtot, [](u32 at) { return at * 2u; });
        if (tid <= S) gptr(d.group_off)[tid] = off;
        regroup_rows<false>(sh.wst, fields, reg, ebase, cnt, [&](u32 r) { return (u16)((r & 1u) ? dv[r >> 1] >> 16 : dv[r >> 1]); });
        __syncthreads();
        with_width(wB, [&](auto width) { store_packed<decltype(width)::value>(fields, cnt, out); });
        if (PERM) {
            __syncthreads();
            regroup_rows<false>(sh.wst, fields, reg, ebase, cnt, [&](u32 r) { return (u16)(ebase + r * 64u); });
            __syncthreads();
            for (u32 i = tid; i < cnt; i += DBLOCK) gptr(d.perm)[i] = fields[i];
        }
        if (ORDERED && order_bad) raise_flag(flags, DF_ORDER);
        return;
    }
    if (tid < S) {
        const u32 g0 = (u32)gptr(d.group_off)[tid] + chunk_tot[chunk * SS + tid];
        sh.gb[tid] = g0;
        const u64 sb = (u64)g0 * wB;
        sh.fo[tid] = (u32)((sb + 63u) >> 6) | ((sb & 63u) ? 0x80000000u : 0u);
    }
    for (u32 k = tid; k < S * LINE; k += DBLOCK) (&sh.lw[0][0])[k] = 0ull;
    if (tid == 0u) sh.hotkey = 0ull;
    if (tid < (u32)FRONT / 4u) slot[tid] = 0ull;
    for (u32 k = tid; k < (u32)WST; k += DBLOCK) sh.wst[k] = 0u;
    __syncthreads();
    if (tid < S)
        atomicMax(&sh.hotkey, ((gptr(d.group_off)[tid + 1u] - gptr(d.group_off)[tid]) << 9) | tid);
    __syncthreads();
    const u32 hot = __builtin_amdgcn_readfirstlane((u32)sh.hotkey & 511u);
    const u32 row_bytes = wave * srow * 4u;
    u32 order_bad = 0u;

    auto tile_cnt = [&](u64 lt) -> u32 {
        const u64 rem = d.n - lt * (u64)DTILE;
        return tile_len(rem, (u32)DTILE);
    };
    lds_fetch<NWAVE>(gptr(d.prev), lt0 * (u64)DTILE, tile_cnt(lt0), wp, Pw, wave);
    lds_fetch<NWAVE>(gptr(d.cur), lt0 * (u64)DTILE, tile_cnt(lt0), wc, Cw, wave);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's share of the first tile's words
    if (ORDERED) {
        __syncthreads(); // all shares of the first tile's words are in LDS
        order_bad = ordered_rank_check(Pw, sh.wst + wave * srow, wave * 1024u + lane, tile_cnt(lt0), S, wp);
    }
    for (u64 lt = lt0; lt < lt1; lt++) {
        const u64 e0 = lt * (u64)DTILE;
        const u32 cnt = tile_cnt(lt);
        __syncthreads(); // all shares of the tile's words are in LDS (every wave waited for its own
                         // before its output phase); the previous tile's output phase is over
        if (!ORDERED) { // sweep 1 uses the slots
            for (u32 k = tid; k < (u32)(NWAVE * SS); k += DBLOCK) slot[k] = 0ull;
            __syncthreads();
        }
        const bool full = cnt == (u32)DTILE;
        u32 reg[16], dv[8];
        u32 ebase = wave * 1024u + lane;
        asm volatile("" : "+v"(ebase)); // keeps the per-row LDS addresses from being hoisted out of
                                        // the tile loop and spilled
        if (full)
            rank_rows<true, ORDERED, true>(Pw, Cw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wc, hot, reg, dv);
        else
            rank_rows<false, ORDERED, true>(Pw, Cw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wc, hot, reg, dv);
        __syncthreads();
        // counts -> positions: population of each symbol, the stream words its run touches,
        // exclusive scans over symbols, start of every (wave, symbol)
        u32 tot = 0, nW = 0, s0 = 0, preW = 0, preE = 0, preR = 0;
        u64 fb = 0;
        u32 sy = tid;  // this thread's symbol
        asm volatile("" : "+v"(sy)); // its table addresses are recomputed per tile, not kept (and
                                     // spilled: a reload would wait for the words in flight)
        sh.items.clear(sy);
        if (tid < 320u) { // waves 0..4 hold the 258 symbols
            if (tid < S) {
#pragma unroll
                for (int wv = 0; wv < NWAVE; wv++) tot += sh.wst[wv * srow + sy];
                const u32 pos = sh.gb[sy]; // after the previous tile's run
                fb = (u64)pos * wB;
                s0 = (u32)(fb & 63u);
                nW = tot ? (s0 + tot * wB + 63u) >> 6 : 0u;
            }
            const u32 incW = wave_incl_scan(nW), incE = wave_incl_scan(tot);
            const u64 runs = __ballot(tot != 0u);
            preW = incW - nW;
            preE = incE - tot;
            preR = __builtin_amdgcn_mbcnt_hi((u32)(runs >> 32), __builtin_amdgcn_mbcnt_lo((u32)runs, 0u));
            if (lane == 63u) {
                sh.wtot[wave] = incW;
                sh.etot[wave] = incE;
                sh.rtot[wave] = (u32)__popcll(runs);
            }
        }
        __syncthreads();
        // the symbols are in registers: the next tile's words start travelling, asked for by the
        // waves that have no scan to do
        if (lt + 1 < lt1 && wave >= 5u) {
            lds_fetch<NWAVE - 5>(gptr(d.prev), e0 + DTILE, tile_cnt(lt + 1), wp, Pw, wave - 5u);
            lds_fetch<NWAVE - 5>(gptr(d.cur), e0 + DTILE, tile_cnt(lt + 1), wc, Cw, wave - 5u);
        }
        if (tid < S) {
            u32 ws = preW, es = preE, rank = preR;
#pragma unroll
            for (u32 w2 = 0; w2 < 4u; w2++) { // (all read together, the needed ones added)
                const u32 a = sh.wtot[w2], b = sh.etot[w2], c = sh.rtot[w2];
                ws += w2 < wave ? a : 0u;
                es += w2 < wave ? b : 0u;
                rank += w2 < wave ? c : 0u;
            }
            sh.gb[sy] += tot;
            sh.gWf[sy] = (u32)(fb >> 6);
            sh.gse[sy] = s0 | (s0 + tot * wB) << 8;
            sh.wstart[sy] = ws;
            sh.les[sy] = (u16)es;
            if (tid == S - 1u) {
                sh.wstart[S] = ws + nW;
                sh.les[S] = (u16)(es + tot);
            }
            sh.items.enter(sy, rank, ws, nW);
            u32 start = es * 2u;
            static_assert(NWAVE % 4 == 0, "the waves are taken four at a time");
#pragma unroll
            for (int w0 = 0; w0 < NWAVE; w0 += 4) { // four counts are read together, then replaced
                u32 c4[4];
#pragma unroll
                for (int j = 0; j < 4; j++) c4[j] = sh.wst[(w0 + j) * srow + sy];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    sh.wst[(w0 + j) * srow + sy] = start;
                    start += c4[j] * 2u;
                }
            }
        }
        __syncthreads();
        // sweep 2: the deltas in regrouped order
        auto delta = [&](u32 r) { return (u16)((r & 1u) ? dv[r >> 1] >> 16 : dv[r >> 1]); };
        if (full)
            regroup_rows<true>(sh.wst, fields, reg, ebase, cnt, delta);
        else
            regroup_rows<false>(sh.wst, fields, reg, ebase, cnt, delta);
        // The next tile's words were asked for a while ago: waiting for them here is free, while at
        // the top of the loop it would also wait for the stores of the output phase below.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (tid < S * LINE) flush_lines(sh, out, tid);
        if (tid + (u32)DBLOCK < S * LINE) flush_lines(sh, out, tid + (u32)DBLOCK);
        __syncthreads();
        // one thread per word of the runs: complete words leave now, unless their line is still open
        auto words = [&](auto width) {
            constexpr u32 W = decltype(width)::value;
            const u32 n_items = sh.wstart[S];
            u32 k0 = tid;
            asm volatile("" : "+v"(k0)); // (what depends on it is computed here, for the width at hand)
            for (u32 k = k0; k < n_items; k += DBLOCK) {
                const u32 g = sh.items.group(k);
                const u32 j = k - sh.wstart[g], se = sh.gse[g], s0 = se & 255u, end = se >> 8;
                const int i = (int)((j * 64u - s0 + 64u * W) / W) - 64; // (fields before the run: masked)
                unsigned long long val = pack_fields<W>(fields, (int)sh.les[g] + i, i * (int)W - (int)(j * 64u - s0));
                if (j == 0u) val = (val & (~0ull << s0)) | sh.carry[g]; // bits of earlier tiles in this word
                const u32 left = end - j * 64u; // bits of the run from this word on
                const u32 Wg = sh.gWf[g] + j, We = sh.gWf[g] + (end >> 6);
                const u32 fo = sh.fo[g], own = fo & 0x7fffffffu, L = Wg & ~(u32)(LINE - 1);
                if (left < 64u) { // the run's last, partial word waits in LDS
                    sh.lw[g][Wg & (LINE - 1u)] = val & ((1ull << left) - 1ull);
                } else if ((fo >> 31) && Wg + 1u == own) { // shared with the run before this chunk's
                    if (val) __hip_atomic_fetch_or(out + Wg, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else if (L >= own && L == (We & ~(u32)(LINE - 1))) {
                    sh.lw[g][Wg & (LINE - 1u)] = val; // a line of this chunk's own that is not complete yet
                } else {
                    out[Wg] = val;
                }
            }
        };
        with_width(wB, words);
        if (PERM) {
            __syncthreads();
            auto index = [&](u32 r) { return (u16)(ebase + r * 64u); };
            if (full)
                regroup_rows<true>(sh.wst, fields, reg, ebase, cnt, index);
            else
                regroup_rows<false>(sh.wst, fields, reg, ebase, cnt, index);
            __syncthreads();
            for (u32 g = wave; g < S; g += NWAVE) {
                const u32 l0 = sh.les[g], c = sh.les[g + 1u] - l0;
                const u32 p0 = sh.gb[g] - c;
                for (u32 i = lane; i < c; i += 64u) gptr(d.perm)[p0 + i] = (u32)(e0 + fields[l0 + i]);
            }
        }
        u32 k0 = tid;
        asm volatile("" : "+v"(k0));
        for (u32 k = k0; k < NWAVE * srow; k += DBLOCK) sh.wst[k] = 0u; // for the next tile's counts
    }
    __syncthreads();
    if (tid < S) { // what the chunk leaves behind: the words of an open line, the last partial word
        const RunEnd r = run_end(sh.gb[tid], wB);
        const u32 L = r.word & ~(u32)(LINE - 1), wl = r.word & (LINE - 1u);
        if (L >= (sh.fo[tid] & 0x7fffffffu))
            for (u32 j = 0; j < wl; j++) out[L + j] = sh.lw[tid][j];
        const unsigned long long part = sh.lw[tid][wl];
        if (r.bits && part)
            __hip_atomic_fetch_or(out + r.word, part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (ORDERED && order_bad) raise_flag(flags, DF_ORDER);
}

// regrouping given: e[r] = d[perm[r]] by gathering
// A given permutation is checked as it is used: an index outside the tensor is skipped and raises
// DF_PERM; symbols are clamped, so that a delta always fits its field.
__global__ __launch_bounds__(BLOCK) void k_dgather(const DDesc *__restrict__ dd,
                                                   const u32 *__restrict__ chunk_tensor,
                                                   u32 *__restrict__ flags)
{
    __shared__ unsigned long long pk[256 * 9];
    const u64 chunk = blockIdx.x;
    const DDesc d = dd[__builtin_amdgcn_readfirstlane(chunk_tensor[chunk])];
    if (!d.prev_perm) return;
    const u32 tid = threadIdx.x;
    const u32 wB = d.wB, Bm = d.B;
    const u32 smax[2] = {d.Kp + 1u, Bm - 1u}; // largest symbol of either stream that is taken as it is
    bool bad_index = false;
    const u64 c_elems = (u64)d.ctiles * DTILE;
    const u64 c0 = (chunk - d.chunk0) * c_elems;
    const u64 c1 = (c0 + c_elems < d.n) ? c0 + c_elems : d.n;
    for (u64 r0 = c0; r0 < c1; r0 += HTILE) {
        const u32 cnt = tile_len(c1 - r0, (u32)HTILE);
        __syncthreads();
        for (u32 k = tid; k < 256u * wB; k += BLOCK) pk[k] = 0ull;
        __syncthreads();
        for (u32 j = 0; j < 16u; j++) {
            const u32 l = tid + j * BLOCK;
            if (l >= cnt) break;
            const u64 i = gptr(d.prev_perm)[r0 + l];
            if (i >= d.n) { // not a permutation of this tensor
                bad_index = true;
                continue;
            }
            u32 sym[2];
            for (int which = 0; which < 2; which++) {
                const GLOBAL_AS unsigned long long *src = which ? gptr(d.cur) : gptr(d.prev);
                const u32 w = which ? d.wc : d.wp;
                const u64 off = i * w;
                const u64 wd = off >> 6;
                const u32 sh = (u32)(off & 63u);
                unsigned long long x = src[wd] >> sh;
                if (sh + w > 64u) x |= src[wd + 1] << (64u - sh);
                sym[which] = (u32)x & ((1u << w) - 1u);
                sym[which] = sym[which] < smax[which] ? sym[which] : smax[which];
            }
            u32 dv = sym[0] + Bm - sym[1];
            if (dv >= Bm) dv -= Bm;
            const u32 bitoff = l * wB;
            const u32 word = bitoff >> 6, shf = bitoff & 63u;
            if (dv) {
                atomicOr(&pk[word], (unsigned long long)dv << shf);
                if (shf + wB > 64u) atomicOr(&pk[word + 1u], (unsigned long long)dv >> (64u - shf));
            }
        }
        __syncthreads();
        const u32 n_words = (cnt * wB + 63u) >> 6;
        GLOBAL_AS unsigned long long *dst = gptr(d.out) + r0 * wB / 64u;
        for (u32 k = tid; k < n_words; k += BLOCK) dst[k] = pk[k];
    }
    if (bad_index) raise_flag(flags, DF_PERM);
}

// Restore side (Algorithm 6): s_cur[i] = (s_prev[i] - e[r]) mod B, where r is the position of element
// i in the stable order of s_prev.  Same chunk and tile walk as k_dscatter, with the data flowing the
// other way: sweep 1 ranks the elements of a tile; the stream words of every group's run of the tile
// are copied into an LDS image (one thread per word, consecutive words of a run by consecutive
// threads); sweep 2 takes every element's delta from the image and writes the current symbol to LDS, and
// one thread per output word packs the fields of its bits and stores it (1.06 G elements, 9 bits:
// 2.49 ms with the symbols OR-ed into an image of the words, 2.00 ms so).
struct RestoreShared {
    u32 wst[WST];       // counts, then bit position in the stream image of (wave, symbol)
    u32 wstart[GS]; // first image word of each group's run; [S] = words in use
    u32 gWf[SS];        // stream word of the first bit of each group's run of this tile
    u32 gb[SS];         // stream position after each group's runs so far
    u32 wtot[5], rtot[5];
    unsigned long long hotkey;
    ItemSets items;
};

// The current symbols of a tile's elements from the image of its stream words: reg as rank_rows leaves it, wst the
// bit position of every (wave, symbol) in the image.
__device__ __forceinline__ void restore_rows(const u32 *img, const u32 *wst, u16 *fields, const u32 (&reg)[16], u32 ebase,
                                             u32 cnt, u32 row_bytes, u32 wB, u32 Bm, u32 &e_max, u32 &s_max)
{
    const u32 mB = (1u << wB) - 1u;
    // sweep 2 (lanes past the tile's end read some word of the image and write fields that are masked)
#pragma unroll
    for (u32 rb = 0; rb < 16u; rb += 4u) {
        u32 bo[4], x2[4][2];
#pragma unroll
        for (u32 q = 0; q < 4u; q++) bo[q] = *(const u32 *)((const char *)wst + (reg[rb + q] & 0xFFFFu));
#pragma unroll
        for (u32 q = 0; q < 4u; q++) {
            const u32 r = rb + q;
            const bool valid = ebase + r * 64u < cnt;
            bo[q] = valid ? bo[q] + (reg[r] >> 16) * wB : 0u;
            x2[q][0] = img[bo[q] >> 5];
            x2[q][1] = img[(bo[q] >> 5) + 1u];
        }
#pragma unroll
        for (u32 q = 0; q < 4u; q++) {
            const u32 r = rb + q;
            const u32 sp = ((reg[r] & 0xFFFFu) - row_bytes) >> 2;
            const u32 e = __builtin_amdgcn_alignbit(x2[q][1], x2[q][0], bo[q]) & mB;
            const u32 a = sp - e, b = a + Bm; // the one that did not wrap below zero is the smaller
            const u32 sc = a < b ? a : b;
            if (ebase + r * 64u < cnt) {
                e_max = e > e_max ? e : e_max;
                s_max = sc > s_max ? sc : s_max;
            }
            fields[ebase + r * 64u] = (u16)sc;
        }
    }
}

template <bool ORDERED>
__global__ __launch_bounds__(DBLOCK, 6) void k_drestore(const DDesc *__restrict__ dd,
                                                        const XDesc *__restrict__ xd,
                                                        const u32 *__restrict__ chunk_tensor,
                                                        const u32 *__restrict__ chunk_tot,
                                                        u32 *__restrict__ flags)
{
    __shared__ RestoreShared sh;
    __shared__ __attribute__((aligned(16))) u32 Pw[DTILE * 9 / 32 + 1];
    __shared__ __attribute__((aligned(8))) u16 fields[DTILE + 40]; // the tile's current symbols
    // slots of sweep 1 (ballot ranking only); then the image of the tile's stream words
    __shared__ unsigned long long slot[ORDERED ? BWORDS : NWAVE * SS];
    static_assert(NWAVE * SS >= BWORDS, "stream image fits the slot array");
    const u64 chunk = blockIdx.x;
    const u32 t = __builtin_amdgcn_readfirstlane(chunk_tensor[chunk]);
    const DDesc d = dd[t];
    const XDesc x = xd[t];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 S = d.Kp + 2u, Bm = d.B, wB = d.wB, wp = d.wp, wc = d.wc;
    const u32 srow = S + 1u;
    const u64 n_tiles = (d.n + DTILE - 1) / DTILE;
    const u64 lt0 = (chunk - d.chunk0) * d.ctiles;
    const u64 lt1 = (lt0 + d.ctiles < n_tiles) ? lt0 + d.ctiles : n_tiles;
    if (delta_single(d)) { // one tile, as in k_dscatter: the image is the stream
        const u32 cnt = (u32)d.n, n_words = (cnt * wB + 63u) >> 6, row_bytes = wave * srow * 4u;
        const u32 ebase = wave * 1024u + lane;
        lds_fetch<NWAVE>(gptr(d.prev), 0u, cnt, wp, Pw, wave);
        for (u32 k = tid; k < NWAVE * srow; k += DBLOCK) sh.wst[k] = 0u;
        if (!ORDERED)
            for (u32 k = tid; k < (u32)(NWAVE * SS); k += DBLOCK) slot[k] = 0ull;
        constexpr u32 PER = (TWORDS + DBLOCK - 1) / DBLOCK;
        unsigned long long w[PER];
#pragma unroll
        for (u32 j = 0; j < PER; j++) w[j] = tid + j * DBLOCK < n_words ? gptr(d.out)[tid + j * DBLOCK] : 0ull;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's share of the words
        __syncthreads();
        u32 e_max = 0u, s_max = 0u, order_bad = 0u, reg[16], unused[8];
        if (ORDERED) order_bad = ordered_rank_check(Pw, sh.wst + wave * srow, ebase, cnt, S, wp);
        rank_rows<false, ORDERED, false>(Pw, Pw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wp, 0u, reg, unused);
        __syncthreads();
#pragma unroll
        for (u32 j = 0; j < PER; j++)
            if (tid + j * DBLOCK < n_words + 1u) slot[tid + j * DBLOCK] = w[j]; // (a word behind the last: zero)
        const u32 off = single_starts(sh.wst, srow, S, sh.wtot, [&](u32 at) { return at * wB; });
        if (tid <= S && x.group_off_in && gptr(x.group_off_in)[tid] != (u64)off) raise_flag(flags, RF_GROUPS);
        restore_rows((const u32 *)slot, sh.wst, fields, reg, ebase, cnt, row_bytes, wB, Bm, e_max, s_max);
        __syncthreads();
        with_width(wc, [&](auto width) { store_packed<decltype(width)::value>(fields, cnt, gptr(x.cur_out)); });
        if (__ballot(e_max >= Bm || s_max >= x.Sc) && lane == 0u) raise_flag(flags, RF_DELTA);
        if (ORDERED && order_bad) raise_flag(flags, RF_ORDER);
        return;
    }
    if (tid < S) sh.gb[tid] = (u32)gptr(d.group_off)[tid] + chunk_tot[chunk * SS + tid];
    if (tid == 0u) sh.hotkey = 0ull;
    for (u32 k = tid; k < (u32)WST; k += DBLOCK) sh.wst[k] = 0u;
    __syncthreads();
    if (tid < S)
        atomicMax(&sh.hotkey, ((gptr(d.group_off)[tid + 1u] - gptr(d.group_off)[tid]) << 9) | tid);
    __syncthreads();
    const u32 hot = __builtin_amdgcn_readfirstlane((u32)sh.hotkey & 511u);
    const u32 row_bytes = wave * srow * 4u;
    const GLOBAL_AS unsigned long long *stream = gptr(d.out);
    u32 e_max = 0u, s_max = 0u, order_bad = 0u; // largest delta, largest symbol
    auto tile_cnt = [&](u64 lt) -> u32 {
        const u64 rem = d.n - lt * (u64)DTILE;
        return tile_len(rem, (u32)DTILE);
    };
    lds_fetch<NWAVE>(gptr(d.prev), lt0 * (u64)DTILE, tile_cnt(lt0), wp, Pw, wave);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (ORDERED) {
        __syncthreads(); // all shares of the first tile's words are in LDS
        order_bad = ordered_rank_check(Pw, sh.wst + wave * srow, wave * 1024u + lane, tile_cnt(lt0), S, wp);
    }
    for (u64 lt = lt0; lt < lt1; lt++) {
        const u64 e0 = lt * (u64)DTILE;
        const u32 cnt = tile_cnt(lt);
        __syncthreads(); // the tile's previous symbols are in LDS; the previous tile has been stored
        if (!ORDERED) {
            for (u32 k = tid; k < (u32)(NWAVE * SS); k += DBLOCK) slot[k] = 0ull;
            __syncthreads();
        }
        u32 reg[16], unused[8];
        u32 ebase = wave * 1024u + lane;
        asm volatile("" : "+v"(ebase)); // (the per-row LDS addresses are not kept across tiles)
        if (cnt == (u32)DTILE)
            rank_rows<true, ORDERED, false>(Pw, Pw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wp, hot, reg, unused);
        else
            rank_rows<false, ORDERED, false>(Pw, Pw, sh.wst, row_bytes, slot + wave * SS, ebase, cnt, S, Bm, wp, wp, hot, reg, unused);
        __syncthreads();
        // counts -> positions, as in the scatter: the stream words each group's run touches,
        // exclusive scan over symbols, bit position of every (wave, symbol) in the image
        sh.items.clear(tid);
        u32 tot = 0, nW = 0, s0 = 0, preW = 0, preR = 0;
        u64 fb = 0;
        u32 sy = tid;
        asm volatile("" : "+v"(sy));
        if (tid < 320u) { // waves 0..4 hold the 258 symbols
            if (tid < S) {
#pragma unroll
                for (int wv = 0; wv < NWAVE; wv++) tot += sh.wst[wv * srow + sy];
                fb = (u64)sh.gb[sy] * wB;
                s0 = (u32)(fb & 63u);
                nW = tot ? (s0 + tot * wB + 63u) >> 6 : 0u;
            }
            const u32 incW = wave_incl_scan(nW);
            const u64 runs = __ballot(tot != 0u);
            preW = incW - nW;
            preR = __builtin_amdgcn_mbcnt_hi((u32)(runs >> 32), __builtin_amdgcn_mbcnt_lo((u32)runs, 0u));
            if (lane == 63u) {
                sh.wtot[wave] = incW;
                sh.rtot[wave] = (u32)__popcll(runs);
            }
        }
        __syncthreads();
        // the next tile's previous symbols start travelling, asked for by the waves without a scan
        if (lt + 1 < lt1 && wave >= 5u)
            lds_fetch<NWAVE - 5>(gptr(d.prev), e0 + DTILE, tile_cnt(lt + 1), wp, Pw, wave - 5u);
        if (tid < S) {
            u32 ws = preW, rank = preR;
#pragma unroll
            for (u32 w2 = 0; w2 < 4u; w2++) {
                ws += w2 < wave ? sh.wtot[w2] : 0u;
                rank += w2 < wave ? sh.rtot[w2] : 0u;
            }
            sh.gb[sy] += tot;
            sh.gWf[sy] = (u32)(fb >> 6);
            sh.wstart[sy] = ws;
            if (tid == S - 1u) sh.wstart[S] = ws + nW;
            sh.items.enter(sy, rank, ws, nW);
            u32 bitpos = ws * 64u + s0;
#pragma unroll
            for (int w0 = 0; w0 < NWAVE; w0 += 4) { // four counts are read together, then replaced
                u32 c4[4];
#pragma unroll
                for (int j = 0; j < 4; j++) c4[j] = sh.wst[(w0 + j) * srow + sy];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    sh.wst[(w0 + j) * srow + sy] = bitpos;
                    bitpos += c4[j] * wB;
                }
            }
        }
        __syncthreads();
        { // the stream words of the tile: image word k is stream word gWf[g] + k - wstart[g]
            const u32 n_img = sh.wstart[S];
            for (u32 k = tid; k < n_img; k += DBLOCK) {
                const u32 g = sh.items.group(k);
                const u64 W = (u64)sh.gWf[g] + (k - sh.wstart[g]);
                slot[k] = W < d.out_words ? stream[W] : 0ull;
            }
        }
        __syncthreads();
        restore_rows((const u32 *)slot, sh.wst, fields, reg, ebase, cnt, row_bytes, wB, Bm, e_max, s_max);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's share of the next tile's words
        __syncthreads();
        {
            GLOBAL_AS unsigned long long *dst = gptr(x.cur_out) + e0 * wc / 64u;
            with_width(wc, [&](auto width) { store_packed<decltype(width)::value>(fields, cnt, dst); });
            for (u32 k = tid; k < NWAVE * srow; k += DBLOCK) sh.wst[k] = 0u; // for the next tile's counts
        }
    }
    if (__ballot(e_max >= Bm || s_max >= x.Sc) && lane == 0u) raise_flag(flags, RF_DELTA);
    if (ORDERED && order_bad) raise_flag(flags, RF_ORDER);
}

// populations and group starts of the tensors that have more than one tile
template <bool CLEAR> static void launch_counts_and_groups(const DeltaCall &c, const XDesc *xd, hipStream_t s)
{
    if (!c.any_long) return;
    PROF("k_dhist", s, k_dhist<<<(unsigned)c.n_chunks, HBLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.chunk_tot, c.totals));
    PROF("k_dgroups", s, k_dgroups<CLEAR><<<(unsigned)(c.n_parts * DG_BLOCKS), 64 * DG_WAVES, 0, s>>>(
                             c.dd, xd, c.part_tensor, c.chunk_tot, c.totals, c.flags));
}

hipError_t launch_reconstruct(const DeltaCall &c, const XDesc *xd, hipStream_t s)
{
    launch_counts_and_groups<false>(c, xd, s);
    if (c.lds_ordered)
        PROF("k_drestore", s, k_drestore<true><<<(unsigned)c.n_chunks, DBLOCK, 0, s>>>(c.dd, xd, c.chunk_tensor, c.chunk_tot, c.flags));
    else
        PROF("k_drestore_slots", s, k_drestore<false><<<(unsigned)c.n_chunks, DBLOCK, 0, s>>>(c.dd, xd, c.chunk_tensor, c.chunk_tot, c.flags));
    return hipGetLastError();
}

// 1 if same-address LDS atomics with return are served in ascending lane order, for every pattern
// tried: all lanes on one address, few addresses, many addresses, with inactive lanes
__global__ __launch_bounds__(256) void k_lds_order_check(u32 *__restrict__ violations)
{
    __shared__ u32 cnt[4][SS];
    const u32 lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    for (u32 i = threadIdx.x; i < 4 * SS; i += 256) (&cnt[0][0])[i] = 0u;
    __syncthreads();
    u32 bad = 0;
    const u32 mods[6] = {1u, 2u, 5u, 18u, 66u, 258u};
    for (u32 t = 0; t < 600u; t++) {
        u32 x = lane * 7919u + t * 104729u + blockIdx.x * 31u + wave * 977u;
        x ^= x >> 16;
        x *= 0x7feb352du;
        x ^= x >> 15;
        x *= 0x846ca68bu;
        x ^= x >> 16;
        const u32 sym = x % mods[t % 6u];
        const bool active = ((x >> 20) & 7u) != 0u;
        const u32 before = cnt[wave][sym];
        u32 got = 0;
        if (active) got = atomicAdd(&cnt[wave][sym], 1u);
        u64 peers = __ballot(active);
        for (int b = 0; b < 9; b++) {
            const bool bit = (sym >> b) & 1u;
            const u64 m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const u32 rank = __popcll(peers & ((1ull << lane) - 1ull));
        if (active && got != before + rank) bad++;
    }
    if (bad) atomicAdd(violations, bad);
}

hipError_t launch_lds_order_check(u32 *violations, hipStream_t s)
{
    k_lds_order_check<<<64, 256, 0, s>>>(violations);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// The delta without any allocation: descriptors, the chunk -> tensor table, the per-chunk symbol
// populations and the flag words live in one file-scope device array.  Every GPU holds its own copy
// at its own address; delta_static_init asks for it once per device, and host code uses that
// pointer only (the array's name is not a device address on the host side).
// ------------------------------------------------------------------------------------------
constexpr size_t DST_DD = 0;                                                   // DDesc[MAX_TENSORS]
constexpr size_t DST_FLAGS = DST_DD + sizeof(DDesc) * DELTA_STATIC_MAX_TENSORS; // u32 flag words
constexpr size_t DST_CT = (DST_FLAGS + 256) & ~(size_t)255;                    // u32[MAX_CHUNKS]
constexpr size_t DST_CK = DST_CT + sizeof(u32) * DELTA_STATIC_MAX_CHUNKS;      // u32[MAX_CHUNKS][SS]
constexpr size_t DST_MAX_PARTS = DELTA_STATIC_MAX_TENSORS + DELTA_STATIC_MAX_CHUNKS / DELTA_PART;
constexpr size_t DST_TOT = DST_CK + sizeof(u32) * (size_t)DELTA_STATIC_MAX_CHUNKS * DELTA_SS; // u32[MAX_PARTS][SS]
constexpr size_t DST_PT = DST_TOT + sizeof(u32) * DST_MAX_PARTS * DELTA_SS;    // u32[MAX_PARTS]
constexpr size_t DST_BYTES = DST_PT + sizeof(u32) * DST_MAX_PARTS;
static_assert(DST_CT - DST_FLAGS >= FLAG_WORDS * sizeof(u32), "room for the flag words");
static __device__ __align__(256) unsigned char scratch[DST_BYTES];

constexpr int MAX_DEVICES = 64;
static unsigned char *g_scratch_ptr[MAX_DEVICES]; // per device: where its copy of `scratch` lies

hipError_t delta_static_init(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    if (g_scratch_ptr[device]) return hipSuccess;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)); // (the current device's copy)
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = (unsigned char *)p;
    return hipSuccess;
}

u32 *delta_static_flags(int device)
{
    if (device < 0 || device >= MAX_DEVICES || !g_scratch_ptr[device]) return nullptr;
    return (u32 *)(g_scratch_ptr[device] + DST_FLAGS);
}

// descriptors from the kernel arguments into the scratch array; tensor of every chunk and part; totals and flags cleared
__global__ __launch_bounds__(256) void k_dstatic_setup(DeltaStaticArgs a, DDesc *__restrict__ dd,
                                                       u32 *__restrict__ chunk_tensor, u32 *__restrict__ part_tensor,
                                                       u32 *__restrict__ totals, u32 n_parts, u32 *__restrict__ flags)
{
    const u32 tid = threadIdx.x;
    if (tid < a.n_tensors) dd[tid] = a.dd[tid];
    if (tid < (u32)FLAG_WORDS) flags[tid] = 0u;
    for (u32 i = tid; i < n_parts * (u32)SS; i += 256u) totals[i] = 0u;
    u32 part_of = 0u; // the tensor of part tid
    for (u32 t = 0; t < a.n_tensors; t++) {
        const u64 c0 = a.dd[t].chunk0, c1 = c0 + a.dd[t].n_chunks;
        for (u64 c = c0 + tid; c < c1; c += 256u) chunk_tensor[c] = t;
        part_of = tid >= a.dd[t].part0 ? t : part_of;
    }
    static_assert(DST_MAX_PARTS <= 256, "a thread per part");
    if (tid < n_parts) part_tensor[tid] = part_of;
}

hipError_t launch_delta_static(int device, const DeltaStaticArgs &a, u64 n_chunks, u64 n_parts, bool any_long,
                               bool any_scatter, bool any_perm, bool lds_ordered, hipStream_t s)
{
    if (device < 0 || device >= MAX_DEVICES || !g_scratch_ptr[device]) return hipErrorNotInitialized;
    if (a.n_tensors > (u32)DELTA_STATIC_MAX_TENSORS || n_chunks > (u64)DELTA_STATIC_MAX_CHUNKS || n_parts > DST_MAX_PARTS)
        return hipErrorInvalidValue;
    unsigned char *base = g_scratch_ptr[device];
    DDesc *dd = (DDesc *)(base + DST_DD);
    u32 *chunk_tensor = (u32 *)(base + DST_CT), *part_tensor = (u32 *)(base + DST_PT);
    DeltaCall c;
    c.dd = dd;
    c.chunk_tensor = chunk_tensor;
    c.part_tensor = part_tensor;
    c.chunk_tot = (u32 *)(base + DST_CK); // every entry of the chunks in use is written by k_dhist
    c.totals = (u32 *)(base + DST_TOT);
    c.flags = (u32 *)(base + DST_FLAGS);
    c.n_chunks = n_chunks;
    c.n_parts = n_parts;
    c.any_long = any_long;
    c.lds_ordered = lds_ordered;
    PROF("k_dstatic_setup", s, k_dstatic_setup<<<1, 256, 0, s>>>(a, dd, chunk_tensor, part_tensor, c.totals, (u32)n_parts, c.flags));
    return launch_delta(c, any_scatter, any_perm, false, s);
}

hipError_t launch_delta(const DeltaCall &c, bool any_scatter, bool any_perm, bool any_gather, hipStream_t s)
{
    launch_counts_and_groups<true>(c, nullptr, s);
    const unsigned n = (unsigned)c.n_chunks;
    if (any_scatter) {
        if (c.lds_ordered)
            PROF("k_dscatter", s, k_dscatter<false, true><<<n, DBLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.chunk_tot, c.flags));
        else
            PROF("k_dscatter_slots", s, k_dscatter<false, false><<<n, DBLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.chunk_tot, c.flags));
    }
    if (any_perm) {
        if (c.lds_ordered)
            PROF("k_dscatter_perm", s, k_dscatter<true, true><<<n, DBLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.chunk_tot, c.flags));
        else
            PROF("k_dscatter_perm_slots", s, k_dscatter<true, false><<<n, DBLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.chunk_tot, c.flags));
    }
    if (any_gather) PROF("k_dgather", s, k_dgather<<<n, BLOCK, 0, s>>>(c.dd, c.chunk_tensor, c.flags));
    return hipGetLastError();
}

} // namespace inshr
