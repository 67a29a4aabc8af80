// Device helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sv {
namespace dev {

typedef float vf4 __attribute__((ext_vector_type(4)));
typedef double vd2 __attribute__((ext_vector_type(2)));

// A read-only value through the scalar cache (uniform index).
template <typename V>
__device__ __forceinline__ V scalar_load(const V *p, uint32_t i)
{
    typedef const __attribute__((address_space(4))) V *cptr;
    return reinterpret_cast<cptr>(reinterpret_cast<uintptr_t>(p))[i];
}

// The amplitudes of a 16-byte slot (two of complex64, one of complex128), widened.
__device__ __forceinline__ void slot_amps(vf4 v, double (&re)[2], double (&im)[2])
{
    re[0] = v.x; im[0] = v.y; re[1] = v.z; im[1] = v.w;
}
__device__ __forceinline__ void slot_amps(vd2 v, double (&re)[1], double (&im)[1])
{
    re[0] = v.x; im[0] = v.y;
}

}  // namespace dev
}  // namespace sv
