// Decoding a quantized tensor (Sec. 4, the inverse of the Quantizer): symbol 0 gives +0.0, symbol
// 2 + b gives the centre of bin b, and the elements with symbol 1 take their original values from
// the protected list.
//
//   k_dequant            workgroups of 256 threads (seven per CU) walk runs of tiles of 16384 elements:
//                        the tile's packed words (asked for one tile ahead) and the codebook are
//                        staged in LDS, every thread decodes 4 consecutive elements at a time and
//                        stores them as one 16-byte piece, 16 pieces per tile.  Waiting for the next
//                        tile's words also waits for this tile's stores, so a tile has to be long
//                        enough to hide that.  Elements with symbol 1 are counted (ballots) and left
//                        at +0.0.
//   k_dequant_protected  one thread per entry of the protected list: checks that the element's symbol
//                        is 1 and stores the value.
#include "inshr_launch.h"

namespace inshr {

__device__ __forceinline__ int find_rdesc(const RDesc *rd, int nT, u64 tile)
{
    int lo = 0, hi = nT - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (rd[mid].tile0 <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

constexpr int DQ_BLOCK = 256;
constexpr int DQ_TILE = DEQUANT_TILE; // 64 elements per thread
constexpr int DQ_ROUNDS = DQ_TILE / (4 * DQ_BLOCK);
constexpr int DQ_PRE = (DQ_TILE * 9 / 128 + DQ_BLOCK - 1) / DQ_BLOCK; // 16-byte pieces of packed words per thread and tile
typedef u32 dq_u4 __attribute__((ext_vector_type(4)));
// device memory: 16 bytes at any 4-byte (words: 8-byte) address
typedef u32 dq_u4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float dq_f4_any __attribute__((ext_vector_type(4), aligned(4)));

// 4 symbols of w bits from bit off of the words on, as values; their largest enters s_max, the number of those
// that are 1 comes back (the same for the whole wave).  Symbols at index `left` and above are no elements.
template <bool FULL>
__device__ __forceinline__ u32 decode4(const u32 *W, const float *value, u32 off, u32 w, u32 left, u32 &s_max, float (&x)[4])
{
    const u32 wd = off >> 5, mask = (1u << w) - 1u;
    const u32 a = W[wd], b = W[wd + 1u], c = W[wd + 2u];
    const u32 lo = __builtin_amdgcn_alignbit(b, a, off & 31u), hi = __builtin_amdgcn_alignbit(c, b, off & 31u);
    // (three symbols are at most 27 bits)
    const u32 sym[4] = {lo & mask, (lo >> w) & mask, (lo >> (2u * w)) & mask, __builtin_amdgcn_alignbit(hi, lo, 3u * w) & mask};
    u32 ones = 0u;
#pragma unroll
    for (u32 k = 0; k < 4u; k++) {
        const bool valid = FULL || k < left;
        ones += (u32)__popcll(__ballot(valid && sym[k] == 1u));
        s_max = valid && sym[k] > s_max ? sym[k] : s_max;
        x[k] = value[sym[k]];
    }
    return ones;
}

// Bound by memory, as far as the seven workgroups of a CU keep requests in flight: the rounds of a tile are unrolled four at a time, so that
// a thread gets by with 54 registers (all sixteen at once took 197, two workgroups per CU: 1.06 G elements
// 1.52 ms, 1.05 ms so, 5.2 GB: 4.9 TB/s).  The value table holds zeros for the symbols that have no centre,
// so a symbol is one read of it and no comparison.
__global__ __launch_bounds__(DQ_BLOCK, 7) void k_dequant(const RDesc *__restrict__ rd, int nT, u64 n_tiles,
                                                         u32 *__restrict__ flags, u32 *__restrict__ ones)
{
    __shared__ __attribute__((aligned(16))) u32 W[DQ_PRE * DQ_BLOCK * 4];
    static_assert(DQ_TILE * 9 / 32 + 2 < DQ_PRE * DQ_BLOCK * 4, "two words past the last symbol's first");
    __shared__ float value[512]; // of every symbol that 9 bits can hold
    const u32 tid = threadIdx.x;
    // every workgroup takes a run of consecutive tiles: the tensor of the first is searched for, the
    // others follow from it
    const u64 per = (n_tiles + gridDim.x - 1) / gridDim.x;
    const u64 tile_lo = (u64)blockIdx.x * per;
    const u64 tile_hi = tile_lo + per < n_tiles ? tile_lo + per : n_tiles;
    if (tile_lo >= tile_hi) return;
    int t = __builtin_amdgcn_readfirstlane(find_rdesc(rd, nT, tile_lo));
    int t_value = -1; // tensor whose values are in LDS
    bool bad = false;
    dq_u4 pre[DQ_PRE]; // the next tile's packed words, asked for one tile ahead
    auto fetch = [&](int tt, u64 tile) {
        const RDesc &d = rd[tt];
        const u64 e0 = (tile - d.tile0) * DQ_TILE;
        const u32 cnt = tile_len(d.n - e0, (u32)DQ_TILE);
        const u32 nd = 2u * ((cnt * d.w + 63u) >> 6); // dwords of the tile, all inside the packed array
        const GLOBAL_AS u32 *src = (const GLOBAL_AS u32 *)(gptr(d.packed) + e0 * d.w / 64u);
#pragma unroll
        for (int j = 0; j < DQ_PRE; j++) {
            const u32 k = 4u * (tid + (u32)DQ_BLOCK * j);
            pre[j] = {0u, 0u, 0u, 0u};
            if (k + 4u <= nd) {
                pre[j] = *(const GLOBAL_AS dq_u4_any *)(src + k);
            } else if (k < nd) { // (an even number of dwords)
                pre[j].x = src[k];
                pre[j].y = src[k + 1u];
            }
        }
    };
    fetch(t, tile_lo);
    for (u64 tile = tile_lo; tile < tile_hi; tile++) {
        const int t_now = t;
        const u64 e0 = (tile - rd[t].tile0) * DQ_TILE;
        const u32 cnt = tile_len(rd[t].n - e0, (u32)DQ_TILE);
        const u32 w = rd[t].w, K = rd[t].K;
        GLOBAL_AS float *dst = gptr(rd[t].dst) + e0;
        __syncthreads(); // the previous tile has been decoded
#pragma unroll
        for (int j = 0; j < DQ_PRE; j++) ((dq_u4 *)W)[tid + (u32)DQ_BLOCK * j] = pre[j]; // zero past the tile's words
        if (t != t_value) {
            for (u32 s = tid; s < 512u; s += DQ_BLOCK) value[s] = s >= 2u && s < K + 2u ? gptr(rd[t].codebook)[s - 2u] : 0.0f;
            t_value = t;
        }
        __syncthreads();
        if (tile + 1 < tile_hi) {
            while (t + 1 < nT && rd[t + 1].tile0 <= tile + 1) t++;
            fetch(t, tile + 1);
        }
        u32 n_one = 0u, s_max = 0u;
        if (cnt == (u32)DQ_TILE) {
#pragma unroll 4
            for (u32 j = 0; j < (u32)DQ_ROUNDS; j++) {
                const u32 i0 = 4u * (tid + (u32)DQ_BLOCK * j);
                float x[4];
                n_one += decode4<true>(W, value, i0 * w, w, 4u, s_max, x);
                *(GLOBAL_AS dq_f4_any *)(dst + i0) = {x[0], x[1], x[2], x[3]};
            }
        } else {
            for (u32 r0 = 0; r0 < cnt; r0 += 4u * DQ_BLOCK) {
                const u32 i0 = r0 + 4u * tid;
                float x[4];
                n_one += decode4<false>(W, value, i0 * w, w, i0 < cnt ? cnt - i0 : 0u, s_max, x);
#pragma unroll
                for (u32 c = 0; c < 4u; c++)
                    if (i0 + c < cnt) dst[i0 + c] = x[c];
            }
        }
        bad |= s_max >= K + 2u;
        if ((tid & 63u) == 0u && n_one) atomicAdd(&ones[t_now], n_one);
    }
    if (__ballot(bad) && (tid & 63u) == 0u) raise_flag(flags, RF_SYMBOL);
}

__global__ __launch_bounds__(256) void k_dequant_protected(const RDesc *__restrict__ rd,
                                                           u32 *__restrict__ flags,
                                                           const u32 *__restrict__ ones)
{
    const RDesc d = rd[blockIdx.y];
    if (blockIdx.x == 0 && threadIdx.x == 0 && (u64)ones[blockIdx.y] != d.n_outlier)
        raise_flag(flags, RF_LIST);
    const u32 mask = (1u << d.w) - 1u;
    for (u64 j = (u64)blockIdx.x * 256u + threadIdx.x; j < d.n_outlier; j += (u64)gridDim.x * 256u) {
        const u64 i = gptr(d.out_idx)[j];
        bool ok = i < d.n && (j == 0 || gptr(d.out_idx)[j - 1] < i); // ascending, hence distinct
        if (ok) {
            const u64 off = i * d.w, wd = off >> 6;
            const u32 sh = (u32)(off & 63u);
            unsigned long long x = gptr(d.packed)[wd] >> sh;
            if (sh + d.w > 64u) x |= gptr(d.packed)[wd + 1] << (64u - sh);
            ok = ((u32)x & mask) == 1u;
        }
        if (ok)
            gptr(d.dst)[i] = d.val_bf16
                                 ? __uint_as_float((u32)((const GLOBAL_AS u16 *)gptr(d.out_val))[j] << 16)
                                 : gptr(d.out_val)[j];
        else
            raise_flag(flags, RF_LIST);
    }
}

hipError_t launch_dequantize(const RDesc *rd, int nT, u64 n_tiles, u64 max_outlier, u32 *flags,
                             u32 *ones, int n_cu, hipStream_t s)
{
    // the workgroups that are resident together, each with one run of tiles (more and shorter runs end with a
    // round that is partly empty, and each starts without words asked for ahead: 8 rounds 1.26, 2 rounds 1.21 ms)
    u64 grid = (u64)n_cu * 7u;
    if (grid > n_tiles) grid = n_tiles;
    PROF("k_dequant", s, k_dequant<<<(unsigned)grid, DQ_BLOCK, 0, s>>>(rd, nT, n_tiles, flags, ones));
    u64 blocks = (max_outlier + 255u) / 256u;
    if (blocks < 1) blocks = 1;
    if (blocks > 1024) blocks = 1024;
    PROF("k_dequant_protected", s,
         k_dequant_protected<<<dim3((unsigned)blocks, (unsigned)nT), 256, 0, s>>>(rd, flags, ones));
    return hipGetLastError();
}

} // namespace inshr
