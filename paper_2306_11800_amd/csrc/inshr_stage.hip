// What a call sends to the device and clears there before its kernels run, by one launch.
//
// A copy, a memset and the kernels of a small call cost about the same each (4 to 5 us from one to the next), so the
// parts are gathered first.  The staging buffer is pinned host memory, read over the bus in 16-byte pieces, a few
// KB to some hundred; what is cleared is written in the same launch by workgroups of its own.  Results of a few
// bytes per tensor and flags go the other way without a copy: the kernels store them to pinned host memory.
// One search, quantize and delta of a 4096-value tensor: eight launches where there were thirteen launches, copies
// and memsets, 134 -> 117 us; of a 1 Mi one 366 -> 329, of 483 tensors of 77 M values 1549 -> 1470.
#include "inshr_launch.h"

namespace inshr {

constexpr int ST_BLOCK = 256;
constexpr u32 ST_COPY_PER = 4;  // pieces of 16 bytes per thread of a copying workgroup
constexpr u32 ST_CLEAR_PER = 16; // ... of a clearing one, at a time

__global__ __launch_bounds__(ST_BLOCK) void k_stage(Stage s, u32 copy_blocks)
{
    typedef u32 u4 __attribute__((ext_vector_type(4)));
    const u32 tid = threadIdx.x;
    if (blockIdx.x < copy_blocks) {
        u64 at = (u64)blockIdx.x * (ST_BLOCK * ST_COPY_PER); // pieces of all parts, one after the other
        u64 n = s.copy[0].pieces;
        int p = 0;
#pragma unroll
        for (int k = 1; k < Stage::PARTS; k++) { // (a workgroup copies from one part: they are rounded up to whole ones)
            const u64 whole = (n + ST_BLOCK * ST_COPY_PER - 1) / (ST_BLOCK * ST_COPY_PER) * (ST_BLOCK * ST_COPY_PER);
            if (p + 1 == k && k < s.n_copy && at >= whole) {
                at -= whole;
                p = k;
                n = s.copy[k].pieces;
            }
        }
        const GLOBAL_AS u4 *from = (const GLOBAL_AS u4 *)gptr((const u4 *)s.copy[p].from);
        GLOBAL_AS u4 *to = (GLOBAL_AS u4 *)gptr((u4 *)s.copy[p].to);
        u4 v[ST_COPY_PER];
#pragma unroll
        for (u32 j = 0; j < ST_COPY_PER; j++) {
            const u64 i = at + tid + j * ST_BLOCK;
            if (i < n) v[j] = from[i];
        }
#pragma unroll
        for (u32 j = 0; j < ST_COPY_PER; j++) {
            const u64 i = at + tid + j * ST_BLOCK;
            if (i < n) to[i] = v[j];
        }
        return;
    }
    const u4 z = {0u, 0u, 0u, 0u};
    const u64 step = (u64)(gridDim.x - copy_blocks) * ST_BLOCK;
    for (int k = 0; k < s.n_clear; k++) {
        GLOBAL_AS u4 *at = (GLOBAL_AS u4 *)gptr((u4 *)s.clear[k].at);
        for (u64 i = (u64)(blockIdx.x - copy_blocks) * ST_BLOCK + tid; i < s.clear[k].pieces; i += step) at[i] = z;
    }
}

hipError_t launch_stage(const Stage &s, int n_cu, hipStream_t st)
{
    u64 copies = 0, most = 0, clears;
    for (int k = 0; k < s.n_copy; k++) copies += (s.copy[k].pieces + ST_BLOCK * ST_COPY_PER - 1) / (ST_BLOCK * ST_COPY_PER);
    for (int k = 0; k < s.n_clear; k++) most = most > s.clear[k].pieces ? most : s.clear[k].pieces;
    clears = (most + ST_BLOCK * ST_CLEAR_PER - 1) / (ST_BLOCK * ST_CLEAR_PER);
    if (clears > 8ull * (u64)n_cu) clears = 8ull * (u64)n_cu;
    if (copies + clears == 0) return hipSuccess;
    PROF("k_stage", st, k_stage<<<(unsigned)(copies + clears), ST_BLOCK, 0, st>>>(s, (u32)copies));
    return hipGetLastError();
}

} // namespace inshr
