// Buffer accesses that are to reach no memory: the offsets they take, and what makes them safe.  Plain code for host and
// device: the rule is checked without a GPU.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define SIDA_HD __host__ __device__ __forceinline__
#else
#define SIDA_HD inline
#endif

namespace sida {

// Lane offset of a load or store that is to be dropped: 2^31 as the range check takes it.
constexpr int32_t kPastEnd = INT32_MIN;

// The range check of a raw buffer access compares the lane's offset with the descriptor's records less the scalar offset.
// A scalar offset beyond the records (an empty descriptor, say) would have to be clamped there for the access to be dropped;
// nothing here relies on that.
SIDA_HD constexpr bool dropped(uint32_t records, int32_t lane, int32_t scalar)
{
    return scalar >= 0 && (uint32_t)scalar <= records && (uint32_t)lane >= records - (uint32_t)scalar;
}

// Behind a workgroup's last tile the grouped GEMM's loads run on for as many K-steps as they are ahead (at most K / 64).  They
// keep the last tile's descriptors, take kPastEnd as lane offset and count their scalar offsets from 0; the largest are:
SIDA_HD constexpr int32_t last_token_scalar(int ahead) { return (ahead - 1) * 128; }           // a K-step of a row
SIDA_HD constexpr int32_t last_weight_scalar(int ahead) { return (ahead - 1) * 4096 + 3072; }  // ... of a stripe, and its last fragment

}  // namespace sida
