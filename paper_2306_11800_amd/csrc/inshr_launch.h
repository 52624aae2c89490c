// Batch description shared by the kernels' translation units and the host API.
#pragma once
#include "inshr_dev.h"

namespace inshr {

constexpr int TGT_STRIDE = 4096;            // per-tensor stride of boundary targets (15 * NBT fits)
constexpr int SQ_STRIDE = MAX_FRAC + 1;     // partial sums of squares per (workgroup, tensor) unit
constexpr int SEL_WORDS = MAX_THR * 1024;    // a tensor's selection histograms ([slot][sign][512])
constexpr int CB_STRIDE = 256;              // codebook entries per configuration

struct Unit {       // the tiles of one tensor that one workgroup of a sweep walks
    u32 off16;        // the unit's share of the sweep's gather pool (u32 units, off() = 16 * off16): wave w owns
    u32 capw;         // [off + w * capw, off + (w + 1) * capw)
    u32 tile0, tile1; // batch-wide tile numbers
    u32 tensor;
    __host__ __device__ u64 off() const { return 16ull * off16; } // (a share is BLOCK / 64 = 16 times capw long)
};

// Which configurations of the grid the boundaries, centres and errors of a tensor are worked out for
// (`View` below): none, all, or one of them (its index).
constexpr u32 VIEW_NONE = 0xFFFFFFFFu, VIEW_ALL = 0xFFFFFFFEu;
// TState::best where the choice hangs on one configuration: its index with this bit set
constexpr u32 CHOICE_IF = 0x80000000u;
static_assert(MAX_CFG < (1 << 16), "no index looks like VIEW_ALL");

struct Bufs { // device pointers, indexed by the tensor's position on the device unless noted; nB rows
              // (tensors searched by the sweeps) except ts, table2, tgt_key, codebook, scores (all)
    TState *ts;
    SearchResult *res; // [nT], in host memory
    u32 *hist1;     // [nT][32768]
    u32 *pool_h1;   // [nT][32768] row of a group's leader: the first-level histograms of the group, added up
    u32 *pool_sel;  // [nT][2][SEL_WORDS] row of a group's leader: the group's selection histograms, per pass
    u32 *table2;    // [nT][4096]
    const Unit *units;   // [units] of sweeps 1 and 2 (and of the pool they gather into)
    const Unit *gunits;  // [gather units] of sweep 3
    const u32 *view;     // [nB] VIEW_NONE, VIEW_ALL or a configuration
    u32 *unit_thr;   // [units][16] threshold-bucket keys each wave of the unit gathered
    u32 *hist2;     // [nT][32768]
    u32 *binfo;     // [nT][32768] offset of an active bin's elements in the gather pool, or INACTIVE
    u32 *tgt_bin;   // [nT][TGT_STRIDE] boundary i of pair q at q*NBT + i
    u32 *tgt_res;
    u32 *tgt_key;   // results: boundary keys
    u32 *pool;      // first gather pool: the keys of the threshold windows (sweep 2), wave-private shares;
                    // afterwards every tensor's keys of active bins in bin-group order (TDesc::pool_grp)
    u32 *pool2;     // second gather pool, same layout: the keys of active bins as sweep 3 gathers them
    u32 *unit_cand; // [gather units][16] active-bin keys each wave of the unit gathered (in hist1, read no more)
    u32 *unit_prot; // [gather units][16] protected values each wave listed (fused; in hist1, read no more)
    u16 *bin_group; // [nT][32768] group of each active bin
    u32 *grp_off;   // [nT][MAX_GROUPS] first / one-past-last position of each group in bin order
    u32 *grp_end;
    u32 *grp_cur;   // [nT][MAX_GROUPS] keys placed so far
    u32 *tgt_rank;  // [nT][TGT_STRIDE] rank of each boundary among all keys of the tensor
    u32 *tgt_klo;   // [nT][TGT_STRIDE] first and last key of each boundary's bin
    u32 *tgt_khi;
    u32 *tile_out;  // [tiles][MAX_FRAC] protected values per tile and protect fraction
    double *sq_part; // [units][SQ_STRIDE]
    double *sq_prot; // [gather units][MAX_FRAC] squares of the protected values (in hist1, read no more)
    // scoring: all boundaries and class edges of all pairs in one list ordered by key ("edges");
    // slot s holds the keys with exactly s edges at or below them
    u32 *edges;     // [nT][MAX_EDGES] edge keys in that order
    u32 *edge_bin;  // [nT][MAX_EDGES] second-level bin of each edge
    u16 *edge_item; // [nT][MAX_EDGES] pair * 259 + (boundary j - 1, or 255 + class edge)
    u16 *sl;        // [nT][32768 + 64] sub-slot of every bin without an edge; 0xFFFF for the others
    u32 *sub_code;  // [nT][MAX_SUB] slot << 9 | sign and exponent (key >> 23) of each sub-slot
    u32 *sub_cnt;   // [nT][MAX_SUB] keys per sub-slot (in bins without an edge)
    u16 *pair_eidx; // [nT][MAX_PAIRS][EIDX_STRIDE] position of each pair's edges in the list
    u32 *grp_elo;   // [nT][MAX_GROUPS] first / one-past-last edge of each group of active bins
    u32 *grp_ehi;
    u32 *seg_cnt;   // [nT][MAX_EDGES] keys per slot that lie in bins without an edge
    u32 *grp_cnt;   // [nT][2][MAX_EDGES] keys per slot from the group of the slot's lower / upper edge
    double *grp_sx; // [nT][2][MAX_EDGES] ... and their sums
    u64 *mom_sx;    // [nT][MAX_SUB] per sub-slot: sum of the 23 mantissa bits over the keys in bins
                    // without an edge
    float *codebook; // [nT][n_cfg][CB_STRIDE]
    Score *scores;  // [nT][n_cfg]
};

struct Batch {
    const TDesc *td;     // device
    const GridDesc *gd;  // device
    const u64 *wg_tile0; // device [n_wg + 1]
    const u32 *wg_fu0;   // device [n_wg + 1] (workgroup, tensor) units of each workgroup
    const u32 *t_fu_off; // device [nT + 1] first unit of each tensor (in ascending workgroup order)
    const u32 *wg_gu0;   // device [n_gwg + 1] gather units of each workgroup of sweep 3
    const u32 *t_gu_off; // device [nB + 1] gather units of each tensor
    u32 *grp_list;       // device [nT * MAX_GROUPS] (tensor << 13 | group) of every group
    u32 *n_grp_total;    // device
    const u64 *wg_tile0_all; // device [n_wg_all + 1] partition of the tiles of all tensors (quantizing)
    int nT;              // tensors; on the device in the order: searched by sweeps, small ones
    int nB;              // tensors searched by the sweeps (the partition wg_tile0 covers their tiles)
    int nS1, nS0;        // small tensors behind them: up to SMALL_MAX, up to SMALL_TINY values
    int n_wg, n_wg_all;
    int n_units;
    int n_gwg, n_gunits; // workgroups and units of sweep 3
    int n_bucket_blocks;
    int n_cu;
    bool lds_ordered;    // same-address LDS atomics return in lane order on this device
    bool spread;         // k_decide or the sketch kernels work with the second histogram's bins
    bool light;          // thresholds and class counts only: no boundaries, no scores (the sketch
                         // quantizer brings its own bins)
    bool any_sampled;    // some tensor's sweep 1 is sampled
    bool any_pooled;     // some tensors share their thresholds (TDesc::pooled)
    bool force_miss;     // (tests) every sampled tensor is sent through the exact sweeps again
    u32 n_pairs, n_cfg;
    u64 n_tiles;
    Bufs bufs;
};

struct QDesc { // one tensor of a quantize call (indexed like the batch)
    unsigned long long *packed; // NULL: tensor not part of the call (or, where fused is set, no outputs)
    float *codebook;
    float *boundaries;
    u32 *out_idx;
    float *out_val;
    u64 out_cap;
    u32 cfg;   // index into the grid of the search state
    u32 val_bf16; // protected values are stored as bfloat16 (u16), rounded to nearest even
    const u32 *alt_key; // NULL, or 256 boundary keys that replace the search's (boundary j of K at
                        // (j << (8 - bits)) - 1) ...
    const float *alt_cb; // ... and the K centres that go with them
    u64 span, span_len;  // fused: the tensor's span of either gather pool (u32 units)
    u32 fused, pad;      // boundaries and centres are worked out while quantizing (launch_fused)
};
struct QInfo {
    u64 n_pruned, n_outlier, n_kept;
    u32 tau_p, tau_o, flags, pad;
};

constexpr int SENS_RUN = 16384;
struct SDesc { // one tensor of a call that partitions by magnitude and sensitivity
    const float *w, *g;
    float *S;           // scratch: the sensitivity scores |g * w|; then the classes (sens_masks)
    float *Wm;          // scratch: the quantized values in index order
    u64 n;
    u32 run0, pad;      // first run of SENS_RUN elements of this tensor in the call-wide numbering
    u32 tau_p;          // prune threshold: image of the pruning metric (magnitude or score bits)
    u32 tau_om, tau_os; // protect thresholds: magnitude image, score bits
    u32 by_sens;        // the pruning metric is the score
    unsigned long long *packed;
    u32 *out_idx;
    float *out_val;
    u64 out_cap;
    float *codebook, *boundaries;
    const u32 *bkeys;   // the compact tensor's boundary keys (one pair: NBT candidates)
    const float *cb;    // ... and the centres of the chosen number of bins
    u32 K, sym_bits;
};
struct SInfo {
    u64 n_pruned, n_outlier, n_kept;
    double sq_pruned, sq_prot; // sums of squares of the pruned / protected values
};

struct DDesc { // one tensor of a delta call
    const unsigned long long *prev, *cur;
    unsigned long long *out;
    u64 *group_off;
    u32 *perm;
    const u32 *prev_perm;
    u64 n, out_words;
    u64 chunk0, n_chunks;
    u32 wp, wc, Kp, B, wB;
    u32 ctiles;          // tiles of a chunk (delta_chunk_tiles)
    u32 part0, pad;      // first of its parts (DELTA_PART) in the call-wide numbering
};
struct RDesc { // one tensor of a dequantize call
    const unsigned long long *packed;
    const float *codebook;
    const u32 *out_idx;
    const float *out_val;
    float *dst;
    u64 n, n_outlier, tile0;
    u32 w, K;
    u32 val_bf16, pad; // out_val holds bfloat16 values (u16)
};
constexpr int DEQUANT_TILE = 16384; // elements per workgroup of the decoding kernel (RDesc::tile0 counts these)
struct XDesc { // one tensor of a reconstruct call: the delta descriptor plus what is checked
    unsigned long long *cur_out; // receives the current symbols
    const u64 *group_off_in;     // group offsets that came with the stream, or NULL
    u32 Sc, pad;                 // symbols of the current checkpoint
};
// flags the restore kernels raise
constexpr u32 RF_SYMBOL = 1u;  // a symbol outside 0 .. K + 1
constexpr u32 RF_LIST = 2u;    // protected list and symbol stream disagree
constexpr u32 RF_GROUPS = 4u;  // group offsets do not match the previous symbols
constexpr u32 RF_DELTA = 8u;   // a delta outside 0 .. B - 1, or a result outside 0 .. K_cur + 1
constexpr u32 RF_ORDER = 16u;  // ranks from returning LDS adds disagree with ranks from ballots
// flags of a delta call
constexpr u32 DF_PERM = 1u;    // a given permutation holds an index outside its tensor
constexpr u32 DF_ORDER = 2u;   // ranks from returning LDS adds disagree with ranks from ballots
constexpr int DELTA_TILE = 12288;
constexpr int DELTA_CHUNK = 64; // most tiles of a chunk
constexpr u32 DELTA_FEW = 16;   // chunks of a tensor up to which nobody adds its symbols' populations up in `totals`
constexpr u32 DELTA_PART = 128; // chunks of a part: the unit in which they are added up, and that a workgroup of
                                // k_dgroups takes
inline u64 delta_parts(u64 n_chunks) { return (n_chunks + DELTA_PART - 1) / DELTA_PART; }
// A tensor of one tile is regrouped by one workgroup from the tile's own counts (unless its regrouping is given).
__host__ __device__ inline bool delta_single(const DDesc &d) { return d.n <= (u64)DELTA_TILE && !d.prev_perm; }
// Tiles per chunk of a delta / reconstruct call over n_tiles tiles in all.  A chunk is walked by one
// workgroup and costs about a tile's time on top of its tiles (its groups' runs are found, opened and
// closed), so chunks are as long as possible; but two workgroups fit a CU, and with fewer than
// about six rounds of them the last round leaves much of the chip idle (a 1 Mi tensor in chunks of
// 64 tiles kept two workgroups busy for 0.44 ms; one-tile chunks: 0.02 ms).
inline u32 delta_chunk_tiles(u64 n_tiles, int n_cu)
{
    const u64 rounds = 6ull * 2ull * (u64)n_cu;
    const u64 c = (n_tiles + rounds - 1) / rounds;
    return (u32)(c < 1ull ? 1ull : c > (u64)DELTA_CHUNK ? (u64)DELTA_CHUNK : c);
}
constexpr int DELTA_SS = 264;
// the delta entry point that allocates nothing: its limits, and its descriptors as kernel arguments
constexpr int DELTA_STATIC_MAX_TENSORS = 16;
constexpr int DELTA_STATIC_MAX_CHUNKS = 2048; // chunks of DELTA_TILE * DELTA_CHUNK elements, all tensors
struct DeltaStaticArgs {
    DDesc dd[DELTA_STATIC_MAX_TENSORS];
    u32 n_tensors, pad;
};

// What a call uploads and clears before its kernels (inshr_stage.hip).  Sizes are rounded up to 16 bytes: sources
// and destinations have that room (they come from allocations and offsets in multiples of 256).
struct Stage {
    static constexpr int PARTS = 4;
    struct Copy {
        const void *from; // pinned host memory
        void *to;
        u64 pieces;       // of 16 bytes
    } copy[PARTS];
    struct Clear {
        void *at;
        u64 pieces;
    } clear[PARTS];
    int n_copy = 0, n_clear = 0;
    void add(void *to, const void *from, size_t bytes) { copy[n_copy++] = {from, to, (bytes + 15) / 16}; }
    void zero(void *at, size_t bytes)
    {
        if (bytes) clear[n_clear++] = {at, (bytes + 15) / 16};
    }
};
hipError_t launch_stage(const Stage &st, int n_cu, hipStream_t s);

// Flags that kernels raise for the host: a word per bit, so that a plain store does (the words may lie in
// host memory).
constexpr int FLAG_WORDS = 8;
__device__ __forceinline__ void raise_flag(u32 *flags, u32 bit) { gptr(flags)[__builtin_ctz(bit)] = 1u; }
inline u32 raised_flags(const u32 *words)
{
    u32 f = 0;
    for (int i = 0; i < FLAG_WORDS; i++) f |= words[i] ? 1u << i : 0u;
    return f;
}

// Optional per-kernel timing with HIP events on the launch stream (off by default).
void prof_begin(const char *name, hipStream_t s);
void prof_end(hipStream_t s);
#define PROF(name, s, ...)                                                                        \
    do {                                                                                          \
        prof_begin(name, s);                                                                      \
        __VA_ARGS__;                                                                              \
        prof_end(s);                                                                              \
    } while (0)

hipError_t launch_select(const Batch &bt, hipStream_t s); // thresholds: sweeps 1 and 2 and what follows from them
hipError_t launch_counts(const Batch &bt, hipStream_t s); // class counts of every pair: ends a search without a choice
// the choice of a search without scores: small tensors searched, the others where bounds of the errors settle it
hipError_t launch_decide(const Batch &bt, hipStream_t s);
// boundaries, centres and errors of the configurations in view (sweep 3 and what follows from it)
hipError_t launch_resolve(const Batch &bt, hipStream_t s);
hipError_t launch_edges(const Batch &bt, hipStream_t s); // edge order, bins without edges (inside launch_resolve)
hipError_t launch_score(const Batch &bt, hipStream_t s); // centres, errors, choice (inside launch_resolve)
hipError_t launch_small(const Batch &bt, hipStream_t s); // the whole search of the small tensors
hipError_t launch_small_many(const Batch &bt, hipStream_t s); // of those of up to SMALL_TINY values (small_crowd)
// the tensors of the units (and the small ones), whose boundaries and centres the state holds
hipError_t launch_quantize(const Batch &bt, const QDesc *qd, const Unit *units, const u32 *wg_u0, int n_wg, QInfo *qi,
                           hipStream_t s);
// The tensors marked in their descriptors, which the batch's gather units cover.  Without qi no descriptor has output
// buffers: boundaries, centres and the error of the configuration stay in the state, and a choice that hangs on it is
// settled.
hipError_t launch_fused(const Batch &bt, const QDesc *qd, QInfo *qi, hipStream_t s);
struct DeltaCall { // what the kernels of a delta or reconstruct call share
    const DDesc *dd;           // device
    const u32 *chunk_tensor;   // device [n_chunks]
    const u32 *part_tensor;    // device [n_parts], NULL: every tensor has one part
    u32 *chunk_tot;            // device [n_chunks][DELTA_SS] populations of the previous symbols
    u32 *totals;               // device [n_parts][DELTA_SS], cleared; NULL: no tensor has more than DELTA_FEW chunks
    u32 *flags;
    u64 n_chunks, n_parts;
    bool any_long;             // some tensor is not delta_single
    bool lds_ordered;
};
hipError_t launch_delta(const DeltaCall &c, bool any_scatter, bool any_perm, bool any_gather, hipStream_t s);
hipError_t delta_static_init(int device); // once per device, with that device current
u32 *delta_static_flags(int device);      // the flag words of launch_delta_static on that device
hipError_t launch_delta_static(int device, const DeltaStaticArgs &a, u64 n_chunks, u64 n_parts, bool any_long,
                               bool any_scatter, bool any_perm, bool lds_ordered, hipStream_t s);
hipError_t launch_sens_score(const SDesc *sd, int nT, u32 n_runs, hipStream_t s);
hipError_t launch_sens_partition(const SDesc *sd, int nT, u32 n_runs, u32 *ticket, u64 *state,
                                 u32 *run_prot, double *run_sq, SInfo *info, hipStream_t s);
hipError_t launch_sens_quant(const SDesc *sd, int nT, u32 n_runs, const u32 *run_prot, u32 *flags,
                             hipStream_t s);
hipError_t launch_lds_order_check(u32 *violations, hipStream_t s);
hipError_t launch_dequantize(const RDesc *rd, int nT, u64 n_tiles, u64 max_outlier, u32 *flags,
                             u32 *ones, int n_cu, hipStream_t s);
hipError_t launch_reconstruct(const DeltaCall &c, const XDesc *xd, hipStream_t s);

// ------------------------------------------------------------------------------------------
// the pairs and boundaries in view
// ------------------------------------------------------------------------------------------
struct View {
    u32 q0, n_pairs; // pairs q0 .. q0 + n_pairs - 1
    u32 n_bnd;       // boundaries per pair
    u32 K;           // bins of the one configuration, or 0: all of the grid's
    u32 cfg;         // the one configuration
};
__device__ __forceinline__ View view_of(const GridDesc *gd, u32 view)
{
    View v;
    if (view == VIEW_ALL) {
        v.q0 = 0u;
        v.n_pairs = gd->n_pairs;
        v.n_bnd = gd->n_bnd;
        v.K = 0u;
        v.cfg = 0u;
    } else {
        v.q0 = gd->cfg_pair[view];
        v.n_pairs = 1u;
        v.K = gd->cfg_K[view];
        v.n_bnd = v.K - 1u;
        v.cfg = view;
    }
    return v;
}
// the i-th boundary of a pair in view
__device__ __forceinline__ u32 view_bnd(const GridDesc *gd, const View &v, u32 i)
{
    return v.K ? bnd_index(v.K, i + 1u) : (u32)gd->bnd[i];
}

// A choice that hangs on configuration g (CHOICE_IF), whose error is known now; compared as choose_config does.
__device__ __forceinline__ void settle_choice(TState *st, u32 g, double sse, double sumsq, double eps)
{
    if (st->best != (CHOICE_IF | g)) return;
    const bool in = (sumsq > 0.0 ? sse / sumsq : 0.0) <= eps;
    st->best = in ? g : st->best_else;
    st->feasible = in ? 1u : st->feasible_else;
}

// Class counts of every (prune, protect) pair from the exact thresholds, by the first n_pairs threads.
__device__ __forceinline__ void store_pairs(TState *st, const GridDesc *gd, u64 n)
{
    const u32 tid = threadIdx.x;
    if (tid >= gd->n_pairs) return;
    const u32 tp = gd->pair_p[tid], to = gd->n_p + gd->pair_o[tid];
    const u64 n_neg = st->n_neg, n_pos = n - n_neg;
    const u64 Pn = st->thr_lt_neg[tp], Pp = st->thr_lt_pos[tp];
    const u64 An = st->thr_gt_neg[to], Ap = st->thr_gt_pos[to];
    const u64 Mn = n_neg - An - Pn, Mp = n_pos - Ap - Pp;
    st->pair_An[tid] = An;
    st->pair_Ap[tid] = Ap;
    st->pair_Pn[tid] = Pn;
    st->pair_Pp[tid] = Pp;
    st->pair_Mn[tid] = Mn;
    st->pair_M[tid] = Mn + Mp;
    if (Mn + Mp == 0ull || Mn > n || Mp > n) {
        // (shared thresholds can leave a tensor without quantized values: reported, and the
        // tensor's gathered keys are not processed)
        atomicOr(&st->internal_err, 32u);
        atomicOr(&st->pool_overflow, 8u);
    }
}

// ------------------------------------------------------------------------------------------
// tile iteration shared by the streaming kernels
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int find_tensor(const TDesc *td, int nT, u64 tile)
{
    int lo = 0, hi = nT - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (td[mid].tile0 <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Elements of a tile of `full` when rem (below 2^32, as every tensor is) are left from its first on.  In 32
// bits: where the compiler knew a tile to be whole from the 64-bit comparison that also chose its length, it
// has taken the length from a condition code that address arithmetic had overwritten since.
__device__ __forceinline__ u32 tile_len(u64 rem, u32 full)
{
    const u32 r = (u32)rem;
    return r < full ? r : full;
}

// four values at a 4-byte aligned address, which is what a 16-byte global load asks for
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));

// A whole tile, asked for without any branch: the values may stay in flight until their first use (a tile
// fetched ahead).
__device__ __forceinline__ void load_tile_ahead(const TDesc &d, u64 e0, float (&v)[16])
{
    const GLOBAL_AS f4_any *p4 = (const GLOBAL_AS f4_any *)(gptr(d.data) + e0);
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const f4_any q = p4[threadIdx.x + 1024u * j];
        v[4 * j + 0] = q.x;
        v[4 * j + 1] = q.y;
        v[4 * j + 2] = q.z;
        v[4 * j + 3] = q.w;
    }
}

// v[4*j + c] = element 4*(tid + 1024*j) + c of the tile; returns the mask of valid entries
__device__ __forceinline__ u32 load_tile(const TDesc &d, u64 e0, u32 cnt, float (&v)[16])
{
    if (cnt == (u32)TILE) {
        load_tile_ahead(d, e0, v);
        return 0xFFFFu;
    }
    const GLOBAL_AS float *p = gptr(d.data) + e0;
    const u32 tid = threadIdx.x;
    u32 mask = 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) {
#pragma unroll
        for (int c = 0; c < 4; c++) {
            u32 idx = 4u * (tid + 1024u * j) + c;
            float x = 0.0f;
            if (idx < cnt) {
                x = p[idx];
                mask |= 1u << (4 * j + c);
            }
            v[4 * j + c] = x;
        }
    }
    return mask;
}

} // namespace inshr
