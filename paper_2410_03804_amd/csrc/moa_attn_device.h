// What the attention kernels of moa_attn.hip and moa_attn_long.hip share.
#ifndef MOA_ATTN_DEVICE_H
#define MOA_ATTN_DEVICE_H
#include "moa_attn_plan.h"
#include "moa_common.h"
#include "../../include/moa.h"

namespace moa {

__device__ __forceinline__ int clamp_len(int len, int cap, int32_t *dev_status)
{
    if (len < 0 || len > cap) {
        if (dev_status) atomicOr(dev_status, MOA_DEV_BAD_LENGTH);
        len = len < 0 ? 0 : cap;
    }
    return len;
}

typedef _Float16 f16_t;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;

// independent calls of the same shape in one launch (blockIdx.z / nbg picks the call).  What picks it comes first and a call begins a
// line of its own: every 64 bytes of arguments that a kernel has to wait for are a trip to memory.
// (CALLS: ATTN_FEW or ATTN_CALLS, see LinDev.)
template <int CALLS>
struct AttnGroup {
    int nbg;      // B * Hkv of one call
    int ncalls;
    int nrb;      // whole key range: row blocks of a (sequence, KV head)
    alignas(64) AttnArgs a[CALLS];
};

typedef short i16x4 __attribute__((ext_vector_type(4)));

// 2^x by the hardware instruction alone: arguments here are <= 0 and results below the normal range may
// become 0, which a softmax weight may
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// the launch of the split pass in 256-row tiles (moa_attn_long.hip)
template <int CALLS>
hipError_t launch_attn_long(const AttnGroup<CALLS> &grp, const SplitGeom &g, hipStream_t stream);

}  // namespace moa
#endif
