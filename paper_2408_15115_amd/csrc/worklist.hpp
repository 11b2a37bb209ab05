// worklist.hpp -- the work list of a pass over a case's region (kernels.hip).
//
// Only some of a region's cells take part in a step (a sixth at the
// 256 x 256 x 768 ellipsoid), so a workgroup looks through its cells, one per
// thread, and the ones that are wanted go to its first threads: most wavefronts
// end at once, which counts where the rest wait for slots that the lattice kernel
// frees.  More cells per workgroup pack them closer but leave a small region too
// few workgroups (1024 cells: 119 us a step instead of 101 in a 53 x 117 x 123
// box, and nothing gained at the ellipsoid).  (At the ellipsoid 9 us a step on
// moment storage, 3 us on FP32, against a thread per cell; nothing either way in
// small boxes.)
#pragma once

namespace turret {

struct ScanList {
    unsigned char at[256];
    int n[4];
};

// The cell of thread k of a workgroup of 256: the k-th of the cells first ..
// first + 255 below count that marked() wants, -1 past them.  err: the case's
// error bits as the calling wavefront read them; with any set nothing is wanted.
// The kernels of the other stream may set them at any time, so wavefronts of one
// workgroup can disagree, and none may leave before the barriers for it: the
// others count on every entry of n.
template <class Marked>
__device__ inline int scan_cells(ScanList &l, int first, int count, int err, Marked &&marked)
{
    const int i = first + (int)threadIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool want = (marked(i < count ? i : count - 1) != 0) & (i < count) & (err == 0);
    const unsigned long long m = __ballot(want);
    if (lane == 0) l.n[w] = __popcll(m);
    __syncthreads();
    int at = 0;
    for (int j = 0; j < w; j++) at += l.n[j];
    if (want) l.at[at + __popcll(m & ((1ull << lane) - 1))] = (unsigned char)threadIdx.x;
    __syncthreads();
    const int n = l.n[0] + l.n[1] + l.n[2] + l.n[3];
    return (int)threadIdx.x < n ? first + l.at[threadIdx.x] : -1;
}

}  // namespace turret
