/* pq_root.h -- square roots of the angle counting (pq_fit.hip); pq_rootcheck.hip compares the two forms. */
#ifndef PQ_ROOT_H
#define PQ_ROOT_H

/* x^(1/2), correctly rounded.  MID: x lies in [2^-100, 2^101], and one correction of the hardware's
   reciprocal root gives the rounded root (five instructions instead of sqrtf's fourteen): the same as sqrtf for every
   number of that range. */
template <bool MID = false>
__device__ __forceinline__ float fit_root(float x)
{
    if (!MID) return sqrtf(x);
    const float y = __builtin_amdgcn_rsqf(x), s = x * y;
    return __builtin_fmaf(__builtin_fmaf(-s, s, x), 0.5f * y, s);
}

#endif
