// What the backward kernels of both tensor types share: how a kept query is found.  P has the fields sel, u, u_stride.
#pragma once

#include "psa_device.h"
#include "psa_internal.h"

namespace psa {

template <typename P>
__device__ __forceinline__ int kept_count(const P& p, int b, int n)
{
    int ub = p.u[b];
    ub = ub < 0 ? 0 : (ub > p.u_stride ? p.u_stride : ub);
    return ub > n ? n : ub;
}
// kept query `t` of the head (an index into its list): its row, or -1 when the entry lies beyond u_b or outside [0, n)
template <typename P>
__device__ __forceinline__ int kept_row(const P& p, int head, int t, int n, int ub)
{
    if (t >= ub) return -1;
    const int i = p.sel[(size_t)head * p.u_stride + t];
    return (i < 0 || i >= n) ? -1 : i;
}

}  // namespace psa
