// Which plane of posted centroids holds the centroid of a cluster, for one workgroup of lc_kmeans_rounds_kernel.
// An iteration posts the centroids that it changes into a plane of its own, piece by piece and by whoever comes first, so
// that plane holds unposted words until the workgroup has seen all of it.  A cluster without members keeps its centroid: what
// keeps it must come from before that plane.  So there are two numbers to a cluster, by the parity of the iteration: the one of this
// iteration is written while its plane is still being posted and read after the barrier behind that; the one before is read meanwhile.
// Plain C++ (no HIP types), so that a test on the host can play through the orders in which waves come to it.
#pragma once

#ifdef __HIPCC__
#define LC_PLANES_FN __host__ __device__ inline
#else
#define LC_PLANES_FN inline
#endif

template <int CLUSTERS>
struct LcPlanes {
    signed char at[2][CLUSTERS];
    // before the first iteration
    LC_PLANES_FN void start(int c) { at[0][c] = at[1][c] = 0; }
    // once per cluster and iteration, before the barrier behind the posts; fresh: this iteration posts a new centroid of it
    LC_PLANES_FN void enter(int it, int c, bool fresh) { at[it & 1][c] = fresh ? (signed char)it : at[(it & 1) ^ 1][c]; }
    // behind that barrier: the centroid to compare with
    LC_PLANES_FN int now(int it, int c) const { return at[it & 1][c]; }
    // while iteration it's plane is being posted: the centroid before it, all of which this workgroup has seen
    LC_PLANES_FN int before(int it, int c) const { return at[(it & 1) ^ 1][c]; }
};
