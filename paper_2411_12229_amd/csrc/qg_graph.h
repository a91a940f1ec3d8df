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
// For each w in ws[0..nw): squared distances from x_w to its R neighbours in G (+inf for -1), out[nw][R].
hipError_t launch_rows_dist(const float* X, int D, int R, const int32_t* ws, int64_t nw, const int32_t* G, double* out,
                            hipStream_t st);

}  // namespace qgg
