// qg_internal.h -- pieces of the index shared by the host-side parts of libqg
// (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "qg.h"

namespace qgi {

// A second handle on an index: it shares the rotation and the vertex blocks
// (which stay owned by `base`) but has its own scratch, counters and stream, so
// searches through different views may run concurrently.  Freed with
// qg_free_index; `base` must outlive it.  nullptr on failure (qg_last_error).
qg_index* make_view(const qg_index* base);

// qg_build_index in two parts, for callers that encode one set of vectors with
// several graphs: an index without blocks and the rotated vectors (device
// memory, the caller's to hipFree), then the blocks for a graph (synchronous;
// checks the graph's ids).  Both set the error message.
int begin_index(const float* vectors, int64_t n, int32_t d, int32_t r, const float* rotation, int32_t entry,
                int device, qg_index** out, float** rotated);
int encode_index(qg_index* idx, const float* vectors, const float* rotated, const int32_t* graph);

// What decides, with a batch, which kernels a search launches.
struct Setting {
  int D, R;
  int64_t n;
  bool beam_regs, lut32;
};
Setting setting_of(const qg_index* idx);

// The kernels of one search: side of the rotation's blocks (qgk::rotate_tiles),
// beam registers (qgk::beam_regs), bytes of a LUT entry, and whether it is one
// launch without an overflow pass.  ls_mode as in qgk::launch_search.
struct Route {
  int tiles, nb, lb;
  bool inl;
  bool same_search(const Route& o) const { return nb == o.nb && lb == o.lb && inl == o.inl; }
};
Route search_route(const Setting& s, int64_t nq, int32_t ef, int ls_mode, int32_t flags, bool aligned);

// Batches (queries and bound on ef) that between them launch every kernel that
// mixed batches of up to max_batch queries and beams of up to ef_max can launch.
struct WarmBatch {
  int64_t nq;
  int32_t ef;
};
std::vector<WarmBatch> warm_batches(const Setting& s, int64_t max_batch, int32_t ef_max, bool stop);

// Sets the thread's qg_last_error message and returns `code`.
int set_error(int code, const std::string& msg);

int device_of(const qg_index* idx);
int dim_of(const qg_index* idx);

}  // namespace qgi
