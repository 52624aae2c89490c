// Partition by magnitude and sensitivity (Sec. 4.1-4.2) for one configuration per tensor.
//
// The sensitivity score of a weight is s = |gradient * weight|.  A weight is protected when its
// magnitude or its score lies above the respective threshold, pruned when it is not protected and
// its pruning metric (magnitude or score) lies below the prune threshold; the rest is quantized.
// The classes are then no rank ranges of one key any more, so the bins are not found by the grid
// search's shared order statistics: the quantized values are copied out in index order and searched
// as a tensor of their own (no pruning, no protection), and a last pass writes the symbols of all
// elements from the thresholds and the boundaries found.
//
//   k_sens_score      s = |g * w| for every element (the thresholds of s come from the ordinary
//                     threshold search over s)
//   k_sens_partition  per run of 16384 consecutive elements: classes as bit masks, quantized values ->
//                     the compact tensor in index order, protected count, squares of the pruned and of
//                     the protected values
//   k_sens_scan       per tensor: exclusive prefixes of the runs' protected counts, totals
//   k_sens_quant      symbols (packed), protected list in index order, boundaries and centres
//
// All but the scan stream; the masks (2 bits per element) save the last pass the scores.  202 M values
// in 9 tensors, 4 bits: score 460 us (5.3 TB/s), partition 580 us (4.0 TB/s; a counting, a serial
// scan and a compacting pass took 430 + 980 + 630), quant 380 us (from masks; from the scores 711; bound
// by vector issue: 75 instructions per 64 elements).
#include "inshr_launch.h"

namespace inshr {

constexpr int SBLK = 1024;           // elements of a block: one wave
constexpr int SWG = 1024;            // threads per workgroup: 16 blocks, one run
constexpr int SRUN = SENS_RUN;       // elements of a run; a tensor's runs are its own
constexpr int SROWS = SBLK / 64;
static_assert(SRUN == SBLK * (SWG / 64), "a workgroup is a run");

__device__ __forceinline__ int sens_tensor_of(const SDesc *sd, int nT, u32 run)
{
    int lo = 0, hi = nT - 1; // last tensor whose first run is <= run
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sd[mid].run0 <= run)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// class of an element: 0 pruned, 1 protected, 2 quantized
__device__ __forceinline__ u32 sens_class(const SDesc &d, float w, float s)
{
    const u32 mag = __float_as_uint(w) & 0x7fffffffu;
    const u32 sc = __float_as_uint(s); // non-negative: its bits order like the value
    if (mag > d.tau_om || sc > d.tau_os) return 1u;
    const u32 m = d.by_sens ? sc : mag;
    return m < d.tau_p ? 0u : 2u;
}

__global__ __launch_bounds__(SWG) void k_sens_score(const SDesc *__restrict__ sd, int nT)
{
    const u32 lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const SDesc d = sd[sens_tensor_of(sd, nT, blockIdx.x)];
    const u64 e0 = (u64)(blockIdx.x - d.run0) * SRUN + wave * SBLK + lane;
    const GLOBAL_AS float *gw = gptr(d.w) + e0, *gg = gptr(d.g) + e0;
    GLOBAL_AS float *gs = gptr(d.S) + e0;
    const u64 left = d.n > e0 ? d.n - e0 : 0ull;
    float w[SROWS], g[SROWS];
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        const u32 i = r * 64u;
        w[r] = i < left ? gw[i] : 0.0f;
        g[r] = i < left ? gg[i] : 0.0f;
    }
#pragma unroll
    for (u32 r = 0; r < SROWS; r++)
        if (r * 64u < left) gs[r * 64u] = fabsf(g[r] * w[r]);
}

// The quantized values of the runs before this one in its tensor.  Every run publishes its own count
// and, once it knows them, the sum up to its end; wave 0 walks back over the runs before it, 64 at a
// time, until it meets such a sum.  Runs are handed out in order, so the ones waited for have
// started, and they publish their counts without waiting for anybody.
constexpr u64 RUN_COUNT = 1ull << 62, RUN_SUM = 2ull << 62, RUN_VALUE = RUN_COUNT - 1ull;
__device__ __forceinline__ u64 sens_before(u64 *state, u32 run, u32 first, u32 count)
{
    const u32 lane = threadIdx.x & 63u;
    u64 sum = 0ull;
    if (lane == 0u)
        __hip_atomic_store(&state[run], (run == first ? RUN_SUM : RUN_COUNT) | count, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    if (run == first) return 0ull;
    for (u32 end = run; end > first;) { // runs [first, end) are not in the sum yet
        const bool is = lane < end - first;
        u64 v = RUN_SUM;
        u64 sums, none;
        do {
            if (is) v = __hip_atomic_load(&state[end - 1u - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sums = __ballot((v & RUN_SUM) != 0ull);
            none = __ballot((v >> 62) == 0ull);
            // (what lies before the nearest sum is not needed)
            if (sums) none &= (sums & (0ull - sums)) - 1ull;
            if (none) __builtin_amdgcn_s_sleep(1);
        } while (none);
        const u64 need = sums ? ((sums & (0ull - sums)) << 1) - 1ull : ~0ull;
        u64 x = (need >> lane) & 1ull ? v & RUN_VALUE : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
        sum += x;
        if (sums) break;
        end -= 64u; // (64 counts and no sum: all of them were runs)
    }
    if (lane == 0u)
        __hip_atomic_store(&state[run], RUN_SUM | (sum + count), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return sum;
}

// Classes of a block of SBLK elements: two masks (quantized, protected) per row of 64.  They take the
// place of the block's scores once its wave has read these (16 bytes per row; a row has at least one score, and
// a tensor's scores end at a multiple of 64 bytes).  Lane r holds the first mask of row r, lane
// SROWS + r the second.
__device__ __forceinline__ GLOBAL_AS u64 *sens_masks(const SDesc &d, u64 block)
{
    return (GLOBAL_AS u64 *)(gptr(d.S) + block);
}
__device__ __forceinline__ bool has_mask(u32 lane, u64 left) // left: elements from the block's first on
{
    return lane < 2u * SROWS && (lane % SROWS) * 64u < left;
}
__device__ __forceinline__ u32 mask_at(u32 lane) { return 2u * (lane % SROWS) + lane / SROWS; }

__global__ __launch_bounds__(SWG) void k_sens_partition(const SDesc *__restrict__ sd, int nT, u32 *__restrict__ ticket,
                                                        u64 *__restrict__ state,
                                                        u32 *__restrict__ run_prot, double *__restrict__ run_sq)
{
    __shared__ u32 s_run, s_kept[SWG / 64], s_prot[SWG / 64];
    __shared__ u64 s_before;
    __shared__ double s_sq[2][SWG / 64];
    const u32 lane = threadIdx.x & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0u) s_run = atomicAdd(ticket, 1u);
    __syncthreads();
    const u32 run = (u32)__builtin_amdgcn_readfirstlane(s_run);
    const SDesc d = sd[sens_tensor_of(sd, nT, run)];
    const u64 e0 = (u64)(run - d.run0) * SRUN + wave * SBLK + lane;
    const GLOBAL_AS float *gw = gptr(d.w) + e0, *gs = gptr(d.S) + e0;
    const u64 left = d.n > e0 ? d.n - e0 : 0ull;
    float w[SROWS], s[SROWS];
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        const u32 i = r * 64u;
        w[r] = i < left ? gw[i] : 0.0f;
        s[r] = i < left ? gs[i] : 0.0f;
    }
    u32 kept = 0u, prot = 0u;
    double q_pruned = 0.0, q_prot = 0.0;
    u64 mine = 0ull; // lane r: quantized of row r, lane 16 + r: protected
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        const u32 c = r * 64u < left ? sens_class(d, w[r], s[r]) : 3u;
        const u64 mk = __ballot(c == 2u), mp = __ballot(c == 1u);
        kept += (u32)__popcll(mk);
        prot += (u32)__popcll(mp);
        if (lane == r) mine = mk;
        if (lane == SROWS + r) mine = mp;
        const double xd = (double)w[r];
        if (c == 0u) q_pruned = fma(xd, xd, q_pruned);
        if (c == 1u) q_prot = fma(xd, xd, q_prot);
    }
    const u64 block = e0 - lane;
    if (has_mask(lane, d.n > block ? d.n - block : 0ull)) sens_masks(d, block)[mask_at(lane)] = mine; // (all scores are in registers)
    q_pruned = wave_sum_f64(q_pruned);
    q_prot = wave_sum_f64(q_prot);
    if (lane == 0u) {
        s_kept[wave] = kept;
        s_prot[wave] = prot;
        s_sq[0][wave] = q_pruned;
        s_sq[1][wave] = q_prot;
    }
    __syncthreads();
    const u32 k_in = wave_incl_scan(lane < SWG / 64 ? s_kept[lane] : 0u);
    if (wave == 0u) {
        const u64 before = sens_before(state, run, d.run0, (u32)__builtin_amdgcn_readlane(k_in, SWG / 64 - 1));
        if (lane == 0u) s_before = before;
    } else if (wave == 1u && lane == 0u) {
        u32 p = 0u;
        double a = 0.0, b = 0.0;
        for (u32 k = 0; k < SWG / 64; k++) {
            p += s_prot[k];
            a += s_sq[0][k];
            b += s_sq[1][k];
        }
        run_prot[run] = p;
        run_sq[2u * run] = a;
        run_sq[2u * run + 1u] = b;
    }
    __syncthreads();
    u64 pos = s_before + (wave ? (u32)__builtin_amdgcn_readlane(k_in, wave - 1u) : 0u);
    GLOBAL_AS float *to = gptr(d.Wm);
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        const u64 m = ((u64)(u32)__builtin_amdgcn_readlane((u32)(mine >> 32), r) << 32) |
                      (u32)__builtin_amdgcn_readlane((u32)mine, r);
        if ((m >> lane) & 1ull)
            to[pos + __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u))] = w[r];
        pos += (u64)__popcll(m);
    }
}

// one workgroup per tensor: protected counts of its runs -> exclusive prefixes (in place), totals
__global__ __launch_bounds__(SWG) void k_sens_scan(const SDesc *__restrict__ sd, const u64 *__restrict__ state,
                                                   u32 *__restrict__ run_prot, const double *__restrict__ run_sq,
                                                   SInfo *__restrict__ info)
{
    __shared__ u32 tot[SWG / 64];
    __shared__ double sq[2][SWG / 64];
    const int t = blockIdx.x;
    const SDesc d = sd[t];
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 runs = (u32)((d.n + SRUN - 1) / SRUN);
    u32 carry = 0u;
    double a = 0.0, b = 0.0;
    for (u32 k = 0; k < runs; k += SWG) {
        const u32 i = k + tid;
        const bool is = i < runs;
        const u32 p = is ? run_prot[d.run0 + i] : 0u;
        if (is) {
            a += run_sq[2u * (d.run0 + i)];
            b += run_sq[2u * (d.run0 + i) + 1u];
        }
        const u32 in = wave_incl_scan(p);
        if (lane == 63u) tot[wave] = in;
        __syncthreads();
        const u32 wt = wave_incl_scan(lane < SWG / 64 ? tot[lane] : 0u);
        const u32 base = carry + (wave ? (u32)__builtin_amdgcn_readlane(wt, wave - 1u) : 0u);
        if (is) run_prot[d.run0 + i] = base + in - p;
        carry += (u32)__builtin_amdgcn_readlane(wt, SWG / 64 - 1);
        __syncthreads();
    }
    a = wave_sum_f64(a);
    b = wave_sum_f64(b);
    if (lane == 0u) {
        sq[0][wave] = a;
        sq[1][wave] = b;
    }
    __syncthreads();
    if (tid == 0u) {
        a = b = 0.0;
        for (int k = 0; k < SWG / 64; k++) {
            a += sq[0][k];
            b += sq[1][k];
        }
        const u64 kept = state[d.run0 + runs - 1u] & RUN_VALUE; // (written by the kernel before: a sum)
        SInfo r;
        r.n_kept = kept;
        r.n_outlier = carry;
        r.n_pruned = d.n - kept - carry;
        r.sq_pruned = a;
        r.sq_prot = b;
        info[t] = r;
    }
}

__global__ __launch_bounds__(SWG) void k_sens_quant(const SDesc *__restrict__ sd, int nT,
                                                    const u32 *__restrict__ run_prot, u32 *__restrict__ flags)
{
    __shared__ u32 bk[256];               // boundary keys, ascending, and no key above them
    __shared__ u16 ssym[SWG / 64][SBLK];  // symbols of the wave's block
    __shared__ u32 s_prot[SWG / 64];
    const u32 tid = threadIdx.x, lane = tid & 63u, run = blockIdx.x;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane(tid >> 6);
    const SDesc d = sd[sens_tensor_of(sd, nT, run)];
    const u32 K = d.K, wb = d.sym_bits;
    const u64 e0 = (u64)(run - d.run0) * SRUN + wave * SBLK; // of the wave's block
    const u64 left = d.n > e0 ? d.n - e0 : 0ull;
    const GLOBAL_AS float *gw = gptr(d.w) + e0 + lane;
    float w[SROWS];
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) w[r] = r * 64u + lane < left ? gw[r * 64u] : 0.0f;
    u64 mine = 0ull;
    if (has_mask(lane, left)) mine = sens_masks(d, e0)[mask_at(lane)];
    const u32 n_mine = (u32)__popcll(mine);
    if (tid < 256u) {
        const u32 key = tid + 1u < K ? d.bkeys[bnd_index(K, tid + 1u)] : 0xFFFFFFFFu;
        bk[tid] = key;
        if (run == d.run0) { // the tensor's first run also hands out boundaries and centres
            if (tid + 1u < K && d.boundaries) d.boundaries[tid] = __uint_as_float(bits_of_key(key));
            if (tid < K) d.codebook[tid] = d.cb[tid];
        }
    }
    const u32 n_prot = wave_sum(lane >= SROWS ? n_mine : 0u);
    if (lane == 0u) s_prot[wave] = n_prot;
    __syncthreads();
    u16 *sy = ssym[wave];
    // symbols: 2 + the number of boundaries at or below the key, by halving (one step of all rows
    // after another: the reads of a step do not wait for each other)
    u32 key[SROWS], lo[SROWS];
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        key[r] = key_of_float(w[r]);
        lo[r] = 0u;
    }
    u32 half = 1u;
    while (2u * half < K) half *= 2u; // 2 * half >= K: K - 1 boundaries in 2 * half - 1 places
    for (u32 step = half; step; step >>= 1) {
#pragma unroll
        for (u32 r = 0; r < SROWS; r++) lo[r] += bk[lo[r] + step - 1u] <= key[r] ? step : 0u;
    }
    const u32 p_in = wave_incl_scan(lane < SWG / 64 ? s_prot[lane] : 0u);
    u64 ppos = (u64)run_prot[run] + (wave ? (u32)__builtin_amdgcn_readlane(p_in, wave - 1u) : 0u);
    bool overflow = false;
#pragma unroll
    for (u32 r = 0; r < SROWS; r++) {
        auto row = [&](u32 k) {
            return ((u64)(u32)__builtin_amdgcn_readlane((u32)(mine >> 32), k) << 32) |
                   (u32)__builtin_amdgcn_readlane((u32)mine, k);
        };
        const u64 mk = row(r), mp = row(SROWS + r);
        sy[r * 64u + lane] = (u16)((mk >> lane) & 1ull ? 2u + lo[r] : (u32)((mp >> lane) & 1ull));
        if (mp) {
            if ((mp >> lane) & 1ull) {
                const u64 at = ppos + __builtin_amdgcn_mbcnt_hi((u32)(mp >> 32), __builtin_amdgcn_mbcnt_lo((u32)mp, 0u));
                if (at < d.out_cap) {
                    d.out_idx[at] = (u32)(e0 + r * 64u + lane);
                    d.out_val[at] = w[r];
                } else {
                    overflow = true;
                }
            }
            ppos += (u64)__popcll(mp);
        }
    }
    if (__ballot(overflow) && lane == 0u) raise_flag(flags, 2u);
    __syncthreads();
    if (!left) return;
    // 1024 symbols of wb bits are 16 * wb whole words; the tensor's last block may end earlier
    const u32 n_here = tile_len(left, (u32)SBLK);
    const u32 n_words = (n_here * wb + 63u) >> 6;
    const u32 inv = (1u << 20) / wb + 1u; // bit0 / wb for bit0 < 1024 wb
    GLOBAL_AS unsigned long long *dst = gptr(d.packed) + (e0 * wb >> 6); // e0 * wb is a multiple of 64
    for (u32 k = lane; k < n_words; k += 64u) {
        const u32 bit0 = k * 64u;
        u32 e = (bit0 * inv) >> 20;        // first element with bits in this word
        unsigned long long word = 0ull;
        for (; e < n_here && e * wb < bit0 + 64u; e++) {
            const unsigned long long v = sy[e];
            const int sh = (int)(e * wb) - (int)bit0;
            word |= sh >= 0 ? v << sh : v >> (-sh);
        }
        dst[k] = word;
    }
}

hipError_t launch_sens_score(const SDesc *sd, int nT, u32 n_runs, hipStream_t s)
{
    PROF("k_sens_score", s, k_sens_score<<<n_runs, SWG, 0, s>>>(sd, nT));
    return hipGetLastError();
}

// ticket and state are clear before
hipError_t launch_sens_partition(const SDesc *sd, int nT, u32 n_runs, u32 *ticket, u64 *state,
                                 u32 *run_prot, double *run_sq, SInfo *info, hipStream_t s)
{
    PROF("k_sens_partition", s, k_sens_partition<<<n_runs, SWG, 0, s>>>(sd, nT, ticket, state, run_prot, run_sq));
    PROF("k_sens_scan", s, k_sens_scan<<<nT, SWG, 0, s>>>(sd, state, run_prot, run_sq, info));
    return hipGetLastError();
}

hipError_t launch_sens_quant(const SDesc *sd, int nT, u32 n_runs, const u32 *run_prot, u32 *flags,
                             hipStream_t s)
{
    PROF("k_sens_quant", s, k_sens_quant<<<n_runs, SWG, 0, s>>>(sd, nT, run_prot, flags));
    return hipGetLastError();
}

} // namespace inshr
