// qg_graph.h -- launch interface of the index-construction kernels (Algorithm 2).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qgg {

// Candidate lists of vertices u0 .. u0+nu-1 from their search results
// sids[nu][EF] and the current graph G[N][R], NSG pruning and, with refine,
// the refinement to R edges and random fill (fill[N][R]): rows u0 .. u0+nu-1 of
// Gout[N][R], which must not overlap G.
hipError_t launch_prune(const float* X, int D, const int32_t* sids, int EF, const int32_t* G, int R, int64_t N,
                        int64_t u0, int64_t nu, int refine, const int32_t* fill, int32_t* Gout, hipStream_t st);
// Rows ids[0..n) of X gathered into out[n][D].
hipError_t launch_gather(const float* X, int D, const int32_t* ids, int64_t n, float* out, hipStream_t st);
// Level `level` of a run of breadth-first levels (count[0 .. level] final, count[level + 1] zero before).
hipError_t launch_bfs_level(const int32_t* G, int R, int64_t n, int level, int64_t base, int32_t* queue,
                            uint32_t* seen, int32_t* count, hipStream_t st);
// The vertices below n not in seen, in any order; *count (zero before) receives their number.
hipError_t launch_unseen(const uint32_t* seen, int64_t n, int32_t* out, int32_t* count, hipStream_t st);
// Repair: the nearest result with a slot not taken, per search (ids[nq][EF]); -1 if none.
hipError_t launch_pick(const int32_t* ids, int64_t nq, int EF, int R, const unsigned long long* taken, int32_t* pick,
                       hipStream_t st);
// Repair: links v[off[g] .. off[g + 1]) from w[g] for every group g (distinct w); *made counts the links.
hipError_t launch_link(const float* X, int D, int R, int64_t groups, const int32_t* w, const int32_t* off,
                       const int32_t* v, int32_t* G, unsigned long long* taken, int32_t* made, hipStream_t st);

}  // namespace qgg
