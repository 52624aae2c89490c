// The search of small tensors by itself (inshr_small.h; with a choice beside k_decide, see there).
#include "inshr_small.h"

namespace inshr {

// n16 tensors of up to SMALL_MAX values from position t0 on, and after them tensors of up to SMALL_TINY
template <bool ORDERED>
__global__ __launch_bounds__(BLOCK) void k_small(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                 Bufs B, int t0, int n16)
{
    extern __shared__ double sm_small[];
    small_beside<ORDERED>(sm_small, td, gd, B, t0 + (int)blockIdx.x, (int)blockIdx.x < n16);
}

// by 512 threads, two workgroups to a CU
template <bool ORDERED>
__global__ __launch_bounds__(512) void k_small_many(const TDesc *__restrict__ td, const GridDesc *__restrict__ gd,
                                                    Bufs B, int t0)
{
    extern __shared__ double sm_small[];
    search_small<512, SMALL_TINY / 512, ORDERED>(*reinterpret_cast<SmallShared<512, SMALL_TINY / 512> *>(sm_small),
                                                 t0 + (int)blockIdx.x, td, gd, B);
}

static hipError_t set_attrs()
{
    static bool done = false;
    if (done) return hipSuccess;
    constexpr int many = (int)sizeof(SmallShared<512, SMALL_TINY / 512>);
    static_assert(512 >= 256 + 64 && MAX_CFG <= 512, "one thread per digit and per configuration");
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void *)k_small<true>, hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_LDS))) return e;
    if ((e = hipFuncSetAttribute((const void *)k_small<false>, hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_LDS))) return e;
    if ((e = hipFuncSetAttribute((const void *)k_small_many<true>, hipFuncAttributeMaxDynamicSharedMemorySize, many))) return e;
    if ((e = hipFuncSetAttribute((const void *)k_small_many<false>, hipFuncAttributeMaxDynamicSharedMemorySize, many))) return e;
    done = true;
    return hipSuccess;
}

hipError_t launch_small_many(const Batch &bt, hipStream_t s)
{
    const hipError_t e = set_attrs();
    if (e) return e;
    constexpr int lds = (int)sizeof(SmallShared<512, SMALL_TINY / 512>);
    const int t0 = bt.nB + bt.nS1;
    if (bt.lds_ordered)
        PROF("k_small_many", s, (k_small_many<true><<<bt.nS0, 512, lds, s>>>(bt.td, bt.gd, bt.bufs, t0)));
    else
        PROF("k_small_many", s, (k_small_many<false><<<bt.nS0, 512, lds, s>>>(bt.td, bt.gd, bt.bufs, t0)));
    return hipGetLastError();
}

hipError_t launch_small(const Batch &bt, hipStream_t s)
{
    hipError_t e = set_attrs();
    if (e) return e;
    const bool crowd = small_crowd(bt, 0);
    if (crowd && bt.nS0 && (e = launch_small_many(bt, s))) return e;
    const int n = bt.nS1 + (crowd ? 0 : bt.nS0);
    if (n) {
        if (bt.lds_ordered)
            PROF("k_small", s, (k_small<true><<<n, BLOCK, SMALL_LDS, s>>>(bt.td, bt.gd, bt.bufs, bt.nB, bt.nS1)));
        else
            PROF("k_small", s, (k_small<false><<<n, BLOCK, SMALL_LDS, s>>>(bt.td, bt.gd, bt.bufs, bt.nB, bt.nS1)));
    }
    return hipGetLastError();
}

} // namespace inshr
