// Quantizer output (Sec. 4): symbols (0 pruned, 1 protected, 2 + bin) bit-packed at bits + 1 bits,
// the codebook of bin centres and the list of protected values in ascending index.
//
// The thresholds, boundaries and centres come from the per-tensor search state; this sweep only
// classifies, searches the boundary list, packs and gathers the protected values.  The position
// of a tile's protected values in the output list is the prefix sum of the per-tile counts that
// the gathering sweep of the search recorded.
//
// (This sweep is for tensors whose boundaries and centres the state holds; where it holds thresholds only, the
// sweep of launch_fused works them out and quantizes in one.)
#include "inshr_quant.h"

namespace inshr {

// How the symbol of a key is found.  BINS: the search's equal-population bins; building the table
// of 32768 bins takes a walk over 32 bins per thread (with a search per bin a workgroup needed about 40 us; 355 M values in
// 292 tensors 0.73 -> 0.65 ms), so it is for long runs of tiles.  CELLS: cells of the
// key's upper 14 bits, each with its first breakpoint and their number (a dozen of them in the
// densest cells: a few bisection steps); a thread per breakpoint finds the cells that hold some.
constexpr int Q_BINS = 0, Q_CELLS = 1;
template <int M> struct Mode {
    static constexpr int value = M;
};
constexpr int QUANT_CELL_TILES = 16; // most tiles of a run classified by cells (4 .. 40 are alike; 100 costs 20 %)
constexpr int CELL_SHIFT = 18, CELLS = 1 << (32 - CELL_SHIFT);
constexpr u32 CELL_MANY = 63u; // number field of a cell: this many or more

struct QuantShared {
    u32 T[COARSE];                   // key prefix -> bins
    u16 symt[L2_BINS];               // symbol, or 0x8000 | first breakpoint of the bin
    unsigned long long piece[BLOCK]; // four symbols of every lane: a wave's 64 are 4 w words of the stream
    u32 held[CELLS / 32];            // cells that hold breakpoints
    u32 sum[BLOCK / 64];
    QuantTables qt;
};

template <bool FULL, int MODE>
__device__ __forceinline__ void classify_tile(QuantShared &qs, u32 tid, const float (&v)[16], u32 mask, u32 n_bp, u32 zero_slot, u32 w,
                                              GLOBAL_AS unsigned long long *dst, u32 n_words, bool any_prot, u32 *wcnt,
                                              u32 &omask, u32 (&pre)[4])
{
    const u32 lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (Of a whole tile every lane stores a word, those past the wave's 4 w its first one again: the number of stores since a
    // load is the same on every way, and waiting for the next tile's values does not wait for these stores, too.)
    const u32 word = FULL && lane >= 4u * w ? 0u : lane;
    const WavePack wp(w, word);
    const u16 *symt = qs.symt;
    const QuantTables &qt = qs.qt;
    omask = 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        u32 e[4], key[4];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            key[c] = key_of_float(v[4 * j + c]);
            e[c] = MODE == Q_BINS ? qs.T[key[c] >> COARSE_SHIFT] : (u32)symt[key[c] >> CELL_SHIFT];
        }
        if (MODE == Q_BINS) {
#pragma unroll
            for (int c = 0; c < 4; c++) e[c] = lookup_u16(symt, key[c], e[c]);
        }
        u32 lo32 = 0u, s3 = 0u;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            u32 sym = e[c];
            if (sym & 0x8000u) { // the bin holds breakpoints: count those at or below the key
                u32 s;
                if (key[c] == ZERO_KEY) { // (checkpoints of sparse updates are mostly zeros, with many a boundary there)
                    s = zero_slot;
                } else if (MODE == Q_BINS) {
                    s = sym & 0x7fffu;
                    if (qt.bp[s] <= key[c]) { // (the bin's first breakpoint exists: s < n_bp)
                        s++;
                        if (qt.bp[s] <= key[c]) { // many equal values put many breakpoints into one bin
                            s++;
                            for (u32 step = 256u; step > 0u; step >>= 1)
                                if (s + step <= n_bp && qt.bp[s + step - 1u] <= key[c]) s += step;
                        }
                    }
                } else {
                    s = sym & 511u;
                    const u32 m = (sym >> 9) & CELL_MANY; // breakpoints of the cell
                    const u32 end = m == CELL_MANY ? n_bp : s + m;
                    for (u32 step = m == CELL_MANY ? 256u : 1u << (31u - (u32)__clz((int)m)); step > 0u; step >>= 1)
                        if (s + step <= end && qt.bp[s + step - 1u] <= key[c]) s += step;
                }
                sym = qt.symtab[s];
            }
            if (!FULL && !((mask >> (4 * j + c)) & 1u)) sym = 0u;
            if (c < 3)
                lo32 |= sym << (c * w);
            else
                s3 = sym;
            omask |= (sym == 1u ? 1u : 0u) << (4 * j + c);
        }
        unsigned long long *mine = qs.piece + wave * 64u;
        wp.put((unsigned long long)lo32 | ((unsigned long long)s3 << (3u * w)), mine, lane);
        const unsigned long long x = wp.word(mine, word);
        const u32 at = ((u32)j * (BLOCK / 64) + wave) * 4u * w + word;
        if (FULL || (lane < 4u * w && at < n_words)) dst[at] = x;
        if (any_prot) { // protected values of this wave's 256 elements: total, and those of lower lanes
            const u32 cj = __popc((omask >> (4 * j)) & 0xFu);
            u32 tot = 0u;
            pre[j] = 0u;
            if (__ballot(cj != 0u)) tot = rank_counts(cj, pre[j]);
            if (lane == 0u) wcnt[j * 16 + wave] = tot;
        }
    }
}

// Small tensors (one tile at most): a workgroup each, no table, every symbol by bisection.
constexpr int QS_NT = 512;                       // threads
constexpr int QS_J = SMALL_MAX / (4 * QS_NT);    // groups of four values per thread
__global__ __launch_bounds__(QS_NT) void k_qsmall(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                  const QDesc *__restrict__ qd, QInfo *__restrict__ qi, Bufs B, int t0)
{
    __shared__ unsigned long long pk[PKW];
    __shared__ QuantTables qt;
    __shared__ u32 wc[64];
    static_assert(QS_J * (QS_NT / 64) == 64, "one lane per (group, wave)");
    static_assert(QS_NT >= QBP + 8, "one thread per breakpoint");
    const int t = t0 + (int)blockIdx.x;
    const QDesc q = qd[t];
    if (q.packed == nullptr) return;
    const TDesc d = td[t];
    const TState *st = B.ts + t;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 n = (u32)d.n;
    const u32 g = q.cfg, pair = gd->cfg_pair[g], K = gd->cfg_K[g], w = symbol_bits(K);
    const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + gd->pair_o[pair]];
    const u32 *tk = q.alt_key ? q.alt_key : B.tgt_key + (size_t)t * TGT_STRIDE + pair * NBT;
    const u32 n_words = (n * w + 63u) >> 6;
    const u32 n_j = (n + 4u * QS_NT - 1u) / (4u * QS_NT);
    float v[4 * QS_J];
    const GLOBAL_AS float *src = gptr(d.data);
#pragma unroll
    for (int j = 0; j < QS_J; j++)
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const u32 i = 4u * (tid + (u32)QS_NT * j) + c;
            v[4 * j + c] = i < n ? src[i] : 0.0f;
        }
    for (u32 k = tid; k < n_words + 1u && k < (u32)PKW; k += QS_NT) pk[k] = 0ull;
    if (tid < 64u) wc[tid] = 0u;
    make_breakpoints(qt, tk, K, tau_p, tau_o);
    u32 omask = 0u, pre[QS_J];
#pragma unroll
    for (int j = 0; j < QS_J; j++) {
        pre[j] = 0u;
        if ((u32)j >= n_j) continue;
        const u32 i0 = 4u * (tid + (u32)QS_NT * j);
        u32 sym[4], key[4];
#pragma unroll
        for (int c = 0; c < 4; c++) key[c] = key_of_float(v[4 * j + c]);
#pragma unroll
        for (int c = 0; c < 4; c++) {
            sym[c] = qt.symtab[slot_of_key(qt.bp, K + 3u, key[c])];
            if (i0 + c >= n) sym[c] = 0u;
        }
        const unsigned long long piece = (unsigned long long)(sym[0] | (sym[1] << w) | (sym[2] << (2u * w))) |
                                         ((unsigned long long)sym[3] << (3u * w));
        const u32 bitoff = i0 * w, word = bitoff >> 6, shf = bitoff & 63u;
        if (piece) {
            atomicOr(&pk[word], piece << shf);
            if (shf + 4u * w > 64u) atomicOr(&pk[word + 1u], piece >> (64u - shf));
        }
        u32 cj = 0u;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            omask |= (sym[c] == 1u ? 1u : 0u) << (4 * j + c);
            cj += sym[c] == 1u ? 1u : 0u;
        }
        if (__ballot(cj != 0u)) {
            const u32 tot = rank_counts(cj, pre[j]);
            if (lane == 0u) wc[j * (QS_NT / 64) + wave] = tot;
        }
    }
    __syncthreads();
    for (u32 k = tid; k < n_words; k += QS_NT) gptr(q.packed)[k] = pk[k];
    const u32 x = wc[lane], inc = wave_incl_scan(x), excl = inc - x; // ascending index: group, wave, lane
    const u32 found = __builtin_amdgcn_readlane(inc, 63);
    if (found) {
#pragma unroll
        for (int j = 0; j < QS_J; j++) {
            u32 r = __builtin_amdgcn_readlane(excl, j * (QS_NT / 64) + wave) + pre[j];
#pragma unroll
            for (int c = 0; c < 4; c++)
                if ((omask >> (4 * j + c)) & 1u)
                    store_protected(q, r++, 4u * (tid + (u32)QS_NT * j) + c, v[4 * j + c]);
        }
    }
    const float *cb = q.alt_cb ? q.alt_cb : B.codebook + ((size_t)t * gd->n_cfg + g) * CB_STRIDE;
    store_head(q, st, gd, tk, cb, found, qi + t);
}

// Long runs: bound by vector issue and the table's dependent LDS reads (355 M values in 292 tensors, 9 bits, 0.53 ms: 2.7 TB/s of
// values; 6.7 G in 291 7.9).  Runs of one tile: by the latency of what comes before the tile (64 of them 21 us).
// Whole tiles have a loop of their own in which nothing waits for the stores of the tile before (with the last tile's code in it
// the compiler waited for all of them: 8.5 ms), and their waves meet once a tile, also where nothing is protected: waves
// that drift apart read from too many places (8 bits, nothing protected: 7.9 ms, 7.05 so; protected values kept in
// a list per wave and the waves meeting every few tiles: 9.0).
// A wave packs its own words without waiting for the others (0.60 ms, 64 runs 30 us with lane pieces OR-ed into a
// buffer of the tile behind a barrier, every held cell of the table bisected and the tile read after it; that needed a
// kernel before, of 8 us, for the places of the protected values.  A unit now adds the counts of the tiles before it up itself,
// one per thread and 1024 tiles: a few loads for ordinary tensors, 256 for the last units of 2^32 values, where the kernel
// before took 217 us; eight in flight, 4.2 G values 4.66 ms, 4.70 one after the other.)
__global__ __launch_bounds__(BLOCK) void k_quant(const TDesc *__restrict__ td, const Unit *__restrict__ units,
                                                 const u32 *__restrict__ wg_u0,
                                                 const GridDesc *__restrict__ gd,
                                                 const QDesc *__restrict__ qd_by_tensor, QInfo *__restrict__ qi,
                                                 Bufs B)
{
    // one static LDS object (it starts at LDS address 0): table offsets then fold into the LDS
    // instructions, which the base of a dynamic array does not allow
    __shared__ QuantShared qs;
    u32 *T = qs.T;
    u16 *symt = qs.symt;
    QuantTables &qt = qs.qt;

    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u32 buf = 0u;
    for (u32 u = wg_u0[blockIdx.x]; u < wg_u0[blockIdx.x + 1]; u++) {
        u32 tid = threadIdx.x;
        asm volatile("" : "+v"(tid)); // (what is derived from it is cheap: worked out per unit it is not kept in scratch)
        const u32 lane = tid & 63u;
        const Unit un = units[u];
        const int t = (int)un.tensor;
        u64 tile = un.tile0;
        const u64 stop = un.tile1;
        const TDesc d = td[t];
        const QDesc q = qd_by_tensor[t];
        const TState *st = B.ts + t;
        const u32 g = q.cfg, pair = gd->cfg_pair[g], K = gd->cfg_K[g];
        const u32 w = symbol_bits(K);
        const u32 o = gd->pair_o[pair];
        const u32 tau_p = st->thr_mag[gd->pair_p[pair]], tau_o = st->thr_mag[gd->n_p + o];
        const u32 nb2 = st->nb2;
        const u32 *tk = q.alt_key ? q.alt_key : B.tgt_key + (size_t)t * TGT_STRIDE + pair * NBT;
        const u32 n_bp = K + 3u;
        auto tile_cnt = [&](u64 tl) -> u32 {
            const u64 rem = d.n - (tl - d.tile0) * (u64)TILE;
            return tile_len(rem, (u32)TILE);
        };
        // the first tile is asked for, and the protected values of the tiles before are added up, beside the tables
        float vn[16];
        bool ahead = tile_cnt(tile) == (u32)TILE; // vn holds the tile about to be worked on (uniform)
        if (ahead) load_tile_ahead(d, (tile - d.tile0) * (u64)TILE, vn);
        const GLOBAL_AS u32 *n_prot = gptr(B.tile_out) + o; // (u64 index below: tiles of a call x MAX_FRAC)
        u32 obase = 0u;
        {
            constexpr u32 AHEAD = 8; // (loads in flight: the tiles before may be 2^18, 256 for each thread)
            u64 k = d.tile0 + tid;
            for (; k + (AHEAD - 1u) * BLOCK < tile; k += AHEAD * BLOCK) {
                u32 x[AHEAD];
#pragma unroll
                for (u32 j = 0; j < AHEAD; j++) x[j] = n_prot[(k + j * BLOCK) * MAX_FRAC];
#pragma unroll
                for (u32 j = 0; j < AHEAD; j++) obase += x[j];
            }
            for (; k < tile; k += BLOCK) obase += n_prot[k * MAX_FRAC];
        }
        obase = wave_sum(obase);
        __syncthreads(); // (nothing of the unit before is read any more)
        if (lane == 0u) qs.sum[wave] = obase;
        if (tid < (u32)(CELLS / 32)) qs.held[tid] = 0u;
        const bool cells = stop - tile <= (u64)QUANT_CELL_TILES; // (the same for the whole workgroup)
        if (!cells)
            for (u32 i = tid; i < (u32)COARSE; i += BLOCK) T[i] = entry_for_u16(B.table2[(size_t)t * COARSE + i]);
        make_breakpoints(qt, tk, K, tau_p, tau_o);
        if (cells) {
            // The cells that hold breakpoints, by the first one of each; then sixteen cells a thread: the breakpoints
            // below them by one bisection, and from there on what the held ones say.  (Held cells lie side by side, up to
            // sixteen for one thread, which took a bisection for each.)
            if (tid < n_bp) {
                const u32 c = qt.bp[tid] >> CELL_SHIFT;
                if (tid == 0u || qt.bp[tid - 1u] >> CELL_SHIFT != c) {
                    const u32 m = slot_of_key(qt.bp, n_bp, (c << CELL_SHIFT) | ((1u << CELL_SHIFT) - 1u)) - tid;
                    symt[c] = (u16)(0x8000u | ((m < CELL_MANY ? m : CELL_MANY) << 9) | tid);
                    atomicOr(&qs.held[c >> 5], 1u << (c & 31u));
                }
            }
            __syncthreads();
            constexpr u32 PER = CELLS / BLOCK;
            static_assert(PER == 16, "half a word of held cells per thread");
            const u32 held = qs.held[tid >> 1] >> ((tid & 1u) * PER);
            u32 s = slot_of_key(qt.bp, n_bp, tid * PER ? (tid * PER << CELL_SHIFT) - 1u : 0u); // (no breakpoint is key 0)
            for (u32 i = 0; i < PER; i++) {
                const u32 c = tid * PER + i;
                if ((held >> i) & 1u) {
                    const u32 m = (symt[c] >> 9) & CELL_MANY;
                    s = m == CELL_MANY ? slot_of_key(qt.bp, n_bp, (c << CELL_SHIFT) | ((1u << CELL_SHIFT) - 1u)) : s + m;
                } else {
                    symt[c] = qt.symtab[s];
                }
            }
        }
        constexpr u32 PER_BINS = L2_BINS / BLOCK;
        if (!cells && tid * PER_BINS < nb2) { // symbol of every bin, or its first breakpoint: 32 bins in a row
            u32 lo = 0u, hi = COARSE - 1u; // key prefix of the first one: last one that starts at or below it
            while (lo < hi) {
                const u32 mid = (lo + hi + 1u) >> 1;
                if ((T[mid] >> 6) <= tid * PER_BINS)
                    lo = mid;
                else
                    hi = mid - 1u;
            }
            u32 e = T[lo], sub = tid * PER_BINS - (e >> 6);
            const u32 start = (lo << COARSE_SHIFT) | (sub << (COARSE_SHIFT - (e & 31u)));
            u32 s = start ? slot_of_key(qt.bp, n_bp, start - 1u) : 0u; // breakpoints in lower bins
            u32 next = qt.bp[s], sym = qt.symtab[s], row[PER_BINS / 2];
#pragma unroll
            for (u32 i = 0; i < PER_BINS; i++) { // (entries past the last bin are not looked at)
                const u32 dd = e & 31u;
                const u32 last = (lo << COARSE_SHIFT) | (sub << (COARSE_SHIFT - dd)) | ((1u << (COARSE_SHIFT - dd)) - 1u);
                u32 x = sym;
                if (s < n_bp && next <= last) {
                    x = 0x8000u | s;
                    if (qt.bp[++s] <= last) s = slot_of_key(qt.bp, n_bp, last); // (many equal values in one bin)
                    next = qt.bp[s];
                    sym = qt.symtab[s];
                }
                row[i >> 1] = (i & 1u) ? row[i >> 1] | (x << 16) : x;
                if (++sub >> dd) {
                    sub = 0u;
                    lo = lo + 1u < (u32)COARSE ? lo + 1u : lo;
                    e = T[lo];
                }
            }
            typedef u32 u4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (u32 i = 0; i < PER_BINS / 8; i++) ((u4 *)symt)[tid * (PER_BINS / 8) + i] = {row[4 * i], row[4 * i + 1], row[4 * i + 2], row[4 * i + 3]};
        }
        const u32 zero_slot = __builtin_amdgcn_readfirstlane(slot_of_key(qt.bp, n_bp, ZERO_KEY));
        __syncthreads();
        GLOBAL_AS unsigned long long *packed = gptr(q.packed);
        obase = 0u;
#pragma unroll
        for (u32 i = 0; i < BLOCK / 64; i++) obase += qs.sum[i]; // (wave-uniform)
        obase = __builtin_amdgcn_readfirstlane(obase);
        // A wave's symbols are whole words of their own, which it packs and stores; the places of a tile's protected values
        // depend on the other waves' counts.  The next tile is asked for before a tile is worked on.
        auto walk = [&](auto mode) {
            constexpr int MODE = decltype(mode)::value;
            u32 found = __builtin_amdgcn_readfirstlane(n_prot[tile * MAX_FRAC]);
            u32 omask, pre[4];
            float v[16];
            auto place_protected = [&](u64 e0, const u32 *wcnt) {
                __syncthreads();
                buf ^= 1u; // (a wave that writes these counts again has passed the next such barrier)
                // protected values in ascending index: quarter j, wave, lane, c
                const u32 wc = wcnt[lane], excl = wave_incl_scan(wc) - wc;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    u32 r = __builtin_amdgcn_readlane(excl, j * 16 + wave) + pre[j];
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        const int i = 4 * j + c;
                        if ((omask >> i) & 1u) {
                            store_protected(q, (u64)obase + r, (u32)(e0 + 4u * (tid + 1024u * j) + c), v[i]);
                            r++;
                        }
                    }
                }
                obase += found;
            };
            for (; ahead; tile++) { // whole tiles
                const u64 e0 = (tile - d.tile0) * (u64)TILE;
#pragma unroll
                for (int i = 0; i < 16; i++) v[i] = vn[i];
#pragma unroll
                for (int i = 0; i < 16; i++)
                    asm volatile("" : "+v"(v[i])); // the values are taken here, before any store below
                const u32 next = n_prot[(tile + 1 < stop ? tile + 1 : tile) * MAX_FRAC]; // (asked for before the values)
                ahead = tile + 1 < stop && tile_cnt(tile + 1) == (u32)TILE;
                if (ahead) load_tile_ahead(d, e0 + TILE, vn);
                GLOBAL_AS unsigned long long *dst = packed + (tile - d.tile0) * (u64)(256u * w);
                u32 *wcnt = qt.wcnt[buf];
                classify_tile<true, MODE>(qs, tid, v, 0xFFFFu, n_bp, zero_slot, w, dst, 0u, found != 0u, wcnt, omask, pre);
                if (found)
                    place_protected(e0, wcnt);
                else
                    __syncthreads(); // (only to keep the waves together)
                found = __builtin_amdgcn_readfirstlane(next);
            }
            if (tile < stop) { // the tensor's last, not a whole one
                const u64 e0 = (tile - d.tile0) * (u64)TILE;
                const u32 cnt = tile_cnt(tile), mask = load_tile(d, e0, cnt, v);
                GLOBAL_AS unsigned long long *dst = packed + (tile - d.tile0) * (u64)(256u * w);
                u32 *wcnt = qt.wcnt[buf];
                classify_tile<false, MODE>(qs, tid, v, mask, n_bp, zero_slot, w, dst, (cnt * w + 63u) >> 6, found != 0u, wcnt, omask, pre);
                if (found) place_protected(e0, wcnt);
            }
        };
        if (cells)
            walk(Mode<Q_CELLS>());
        else
            walk(Mode<Q_BINS>());
        if (stop == d.tile0 + (d.n + TILE - 1) / TILE) { // the tensor's last unit
            const float *cb = q.alt_cb ? q.alt_cb : B.codebook + ((size_t)t * gd->n_cfg + g) * CB_STRIDE;
            store_head(q, st, gd, tk, cb, obase, qi + t);
        }
    }
}

hipError_t launch_quantize(const Batch &bt, const QDesc *qd, const Unit *units, const u32 *wg_u0, int n_wg, QInfo *qi,
                           hipStream_t s)
{
    if (n_wg) PROF("k_quant", s, k_quant<<<n_wg, BLOCK, 0, s>>>(bt.td, units, wg_u0, bt.gd, qd, qi, bt.bufs));
    if (bt.nT > bt.nB)
        PROF("k_qsmall", s, k_qsmall<<<bt.nT - bt.nB, QS_NT, 0, s>>>(bt.td, bt.gd, qd, qi, bt.bufs, bt.nB));
    return hipGetLastError();
}

} // namespace inshr
