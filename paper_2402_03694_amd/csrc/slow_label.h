// The label of a row whose logits two lanes of a wave hold, for every kernel of the slow model that ends in a 32 x 32 accumulator.
#pragma once

#include <hip/hip_runtime.h>

// The label of a row whose classes two lanes hold, lane l and lane l ^ 32: class 0 first, then every class that is strictly larger
// than all before it.  A NaN is larger than nothing, and nothing than a NaN in class 0, which counts as infinity here; so what a
// lane holds is never NaN, and the two lanes come to the same label.
// A lane starts before its first class (the lower lane's is class 0, whose logit is y0) and takes c where y > bv.
static __device__ __forceinline__ float label_start(uint32_t half, float y0) { return half ? -__builtin_inff() : y0 == y0 ? y0 : __builtin_inff(); }
static __device__ __forceinline__ uint32_t label_of(uint32_t best, float bv)
{
    const float ov = __shfl_xor(bv, 32, 64);
    const uint32_t ob = (uint32_t)__shfl_xor((int)best, 32, 64);
    return ov > bv || (ov == bv && ob < best) ? ob : best; // (a lane without classes holds -infinity and a number past the last)
}
