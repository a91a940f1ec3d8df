// qg_graph.cpp -- Algorithm 2 (Indexing, Sec. 3.2) on the device: qg_build_graph.
//
// Each iteration encodes the current graph into a temporary index (the FastScan
// data of every vertex), searches every vector with Algorithm 1 (beam EF, EF
// results) through the same search kernels as queries, turns the results and
// the current neighbours into sorted candidate lists, and applies the NSG
// pruning rule; every list is replaced at once.  In the last iteration the
// refinement supplements edges up to R and random ids fill vertices with too
// few candidates.  Then unreachable vertices are linked from their nearest
// reachable vertex; the graph is on the device throughout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "qg.h"
#include "qg_graph.h"
#include "qg_internal.h"

namespace {

struct DevBuf {
  void* p = nullptr;
  ~DevBuf() { (void)hipFree(p); }
  hipError_t alloc(size_t n) { return hipMalloc(&p, n); }
  template <class T>
  T* as() const {
    return static_cast<T*>(p);
  }
};

int hip_err(hipError_t e, const char* what) {
  return qgi::set_error(QG_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_OR_FAIL(call, what)           \
  do {                                    \
    hipError_t e_ = (call);               \
    if (e_ != hipSuccess) return hip_err(e_, what); \
  } while (0)

// Frees an index and the rotated vectors it is encoded from.
struct Builder {
  qg_index* idx = nullptr;
  float* rotated = nullptr;
  ~Builder() {
    if (idx) qg_free_index(idx);
    (void)hipFree(rotated);
  }
};

constexpr int kLevels = 16;  // breadth-first levels launched between two looks of the host

// The rest of a breadth-first search on the host: `frontier` vertices from
// queue[base] on are in `seen` but not walked yet; `reached` receives base and
// everything found from there on.
int walk_on_host(const int32_t* G, int64_t n, int r, uint32_t* seen, const int32_t* queue, int64_t base,
                 int64_t frontier, int64_t* reached) {
  std::vector<int32_t> rows, found;
  std::vector<uint32_t> bits;
  try {
    rows.resize((size_t)(n * r));
    bits.resize((size_t)(n + 31) / 32);
    found.reserve((size_t)(n - base));
    found.resize((size_t)frontier);
  } catch (const std::bad_alloc&) {
    return qgi::set_error(QG_ENOMEM, "host buffer");
  }
  HIP_OR_FAIL(hipMemcpy(rows.data(), G, sizeof(int32_t) * rows.size(), hipMemcpyDeviceToHost), "download graph");
  HIP_OR_FAIL(hipMemcpy(bits.data(), seen, sizeof(uint32_t) * bits.size(), hipMemcpyDeviceToHost), "reachability");
  HIP_OR_FAIL(hipMemcpy(found.data(), queue + base, sizeof(int32_t) * found.size(), hipMemcpyDeviceToHost),
              "reachability");
  for (size_t h = 0; h < found.size(); ++h) {
    const int32_t* row = rows.data() + (size_t)found[h] * (size_t)r;
    for (int j = 0; j < r; ++j) {
      const int32_t v = row[j];
      if (v < 0 || v >= n || ((bits[(size_t)v >> 5] >> (v & 31)) & 1u)) continue;
      bits[(size_t)v >> 5] |= 1u << (v & 31);
      found.push_back(v);  // each vertex once: within what was reserved
    }
  }
  HIP_OR_FAIL(hipMemcpy(seen, bits.data(), sizeof(uint32_t) * bits.size(), hipMemcpyHostToDevice), "reachability");
  *reached = base + (int64_t)found.size();
  return QG_OK;
}

// Breadth-first reachability from the entry over rows of r ids (-1 = empty):
// `reached` receives the count, seen one bit per vertex.  Levels run on the
// device, 85 us for the kLevels of a look however few vertices they find, while
// the host walks a vertex in 65 ns (both measured on paths, the copy of the
// graph included).  So a graph that is not done after one look per 8,192
// vertices, about an eighth of what the host needs for all of it, is finished
// there: a path of 200,000 vertices takes 1,060 ms by levels alone, 13 ms on the
// host alone and 10 ms this way.
int reach_from(const int32_t* G, int64_t n, int r, int32_t entry, uint32_t* seen, int32_t* queue, int32_t* count,
               int64_t* reached) {
  const size_t words = (size_t)(n + 31) / 32;
  const uint32_t bit = 1u << (entry & 31);
  int32_t host[kLevels + 1] = {1};
  HIP_OR_FAIL(hipMemset(seen, 0, sizeof(uint32_t) * words), "reachability");
  HIP_OR_FAIL(hipMemcpy(seen + (entry >> 5), &bit, sizeof bit, hipMemcpyHostToDevice), "reachability");
  HIP_OR_FAIL(hipMemcpy(queue, &entry, sizeof entry, hipMemcpyHostToDevice), "reachability");
  int64_t base = 0;
  for (int64_t looks = 1 + n / 8192; looks > 0; --looks) {
    for (int l = 1; l <= kLevels; ++l) host[l] = 0;
    HIP_OR_FAIL(hipMemcpy(count, host, sizeof host, hipMemcpyHostToDevice), "reachability");
    for (int l = 0; l < kLevels; ++l)
      HIP_OR_FAIL(qgg::launch_bfs_level(G, r, n, l, base, queue, seen, count, nullptr), "reachability");
    HIP_OR_FAIL(hipMemcpy(host, count, sizeof host, hipMemcpyDeviceToHost), "reachability");
    for (int l = 0; l < kLevels; ++l) base += host[l];
    if (!host[kLevels]) {
      *reached = base;
      return QG_OK;
    }
    host[0] = host[kLevels];
  }
  return walk_on_host(G, n, r, seen, queue, base, host[0], reached);
}

class DeviceScope {
 public:
  explicit DeviceScope(int dev) {
    (void)hipGetDevice(&old_);
    if (old_ != dev) (void)hipSetDevice(dev);
  }
  ~DeviceScope() { (void)hipSetDevice(old_); }

 private:
  int old_ = 0;
};

}  // namespace

extern "C" int qg_build_graph(const float* vectors, int64_t n, int32_t d, int32_t r, int32_t ef_build, int32_t iters,
                              const float* rotation, int32_t entry, const int32_t* init_graph, const int32_t* fill,
                              int32_t flags, int device, int32_t* out_graph, int64_t* out_stats) {
  if (!vectors || !rotation || !init_graph || !out_graph) return qgi::set_error(QG_EINVAL, "NULL array");
  if (n < 2 || n > 0x3fffffffLL) return qgi::set_error(QG_EINVAL, "n must be in [2, 2^30)");
  if (d <= 0 || d % 8 || r <= 0 || r > 64) return qgi::set_error(QG_EINVAL, "bad d or r");
  if (ef_build < 1 || ef_build > QG_MAX_K || iters < 0) return qgi::set_error(QG_EINVAL, "bad ef_build or iters");
  if (entry < 0 || entry >= n) return qgi::set_error(QG_EINVAL, "entry out of range");
  if (flags & ~(QG_GRAPH_REFINE | QG_GRAPH_REPAIR | QG_GRAPH_PROGRESS))
    return qgi::set_error(QG_EINVAL, "unknown flags");
  const bool refine = (flags & QG_GRAPH_REFINE) && iters > 0;
  if (refine && !fill) return qgi::set_error(QG_EINVAL, "refinement needs the fill ids");
  int ndev = 0;
  HIP_OR_FAIL(hipGetDeviceCount(&ndev), "hipGetDeviceCount");
  if (device < 0 || device >= ndev) return qgi::set_error(QG_EINVAL, "bad device");
  DeviceScope scope(device);
  const auto t0 = std::chrono::steady_clock::now();
  auto note = [&](const char* what, int i, int64_t count) {
    if (!(flags & QG_GRAPH_PROGRESS)) return;
    const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    std::fprintf(stderr, "[qg_build_graph] %.1fs %s %d: %lld\n", s, what, i, (long long)count);
    std::fflush(stderr);
  };
  const int64_t chunk = std::min<int64_t>(n, 65536);
  DevBuf G, Gnew, sids, sdist;
  HIP_OR_FAIL(G.alloc(sizeof(int32_t) * (size_t)(n * r)), "hipMalloc graph");
  HIP_OR_FAIL(Gnew.alloc(sizeof(int32_t) * (size_t)(n * r)), "hipMalloc next graph");
  HIP_OR_FAIL(sids.alloc(sizeof(int32_t) * (size_t)(chunk * ef_build)), "hipMalloc search ids");
  HIP_OR_FAIL(sdist.alloc(sizeof(float) * (size_t)(chunk * ef_build)), "hipMalloc search distances");
  HIP_OR_FAIL(hipMemcpy(G.p, init_graph, sizeof(int32_t) * (size_t)(n * r), hipMemcpyDeviceToDevice), "copy graph");

  // one index for the whole build: each graph is encoded into its blocks from
  // the vectors rotated once
  Builder B;
  auto encode = [&]() {
    int rc = B.idx ? QG_OK : qgi::begin_index(vectors, n, d, r, rotation, entry, device, &B.idx, &B.rotated);
    return rc ? rc : qgi::encode_index(B.idx, vectors, B.rotated, G.as<int32_t>());
  };
  for (int it = 0; it < iters; ++it) {
    int rc = encode();
    if (rc) return rc;  // the message is set
    qg_index* const idx = B.idx;
    for (int64_t q0 = 0; q0 < n && rc == QG_OK; q0 += chunk) {
      const int64_t nq = std::min(chunk, n - q0);
      rc = qg_search_ex(idx, vectors + q0 * d, nq, ef_build, ef_build, 0, sids.as<int32_t>(), sdist.as<float>(),
                        nullptr);
      if (rc == QG_OK) {
        const hipError_t e = qgg::launch_prune(vectors, d, sids.as<int32_t>(), ef_build, G.as<int32_t>(), r, n, q0,
                                               nq, refine && it + 1 == iters, fill, Gnew.as<int32_t>(), nullptr);
        if (e != hipSuccess) rc = hip_err(e, "pruning");
      }
    }
    const hipError_t es = hipDeviceSynchronize();
    if (rc) return rc;
    HIP_OR_FAIL(es, "search and pruning");
    std::swap(G.p, Gnew.p);  // all lists are replaced at once
    note("iteration, vertices searched and lists pruned", it, n);
  }
  if (refine) note("refinement done", iters - 1, n);

  int64_t stats[4] = {0, 0, 0, 0};
  if (flags & QG_GRAPH_REPAIR) {
    // An addition to the paper, in rounds.  A round finds the vertices
    // unreachable from the entry; each such v runs Algorithm 1 on the current
    // graph (beam ef_build, ef_build results) and picks the nearest result
    // that still has a slot not taken by an earlier repair (every result was
    // visited from the entry, so it is reachable).  Per picked vertex w in
    // increasing id, its v's in increasing id take w's empty slots in slot
    // order, then w's edges not taken by a repair, farthest first (fp64, ties
    // to the larger id).  Rounds repeat until every vertex is reachable or a
    // round links none.
    // The graph stays on the device; the host only orders the picks.
    const size_t words = (size_t)(n + 31) / 32;
    DevBuf seen, queue, count, taken, unr_d, pick_d, qv_d, w_d, off_d, v_d;
    HIP_OR_FAIL(seen.alloc(sizeof(uint32_t) * words), "hipMalloc reachability");
    HIP_OR_FAIL(queue.alloc(sizeof(int32_t) * (size_t)n), "hipMalloc reachability");
    HIP_OR_FAIL(count.alloc(sizeof(int32_t) * (kLevels + 1)), "hipMalloc reachability");
    HIP_OR_FAIL(taken.alloc(sizeof(uint64_t) * (size_t)n), "hipMalloc repaired slots");
    HIP_OR_FAIL(hipMemset(taken.p, 0, sizeof(uint64_t) * (size_t)n), "clear repaired slots");
    std::vector<int32_t> unr, pick, ws, off, vs;
    std::vector<int64_t> order;
    int64_t cap = 0;
    int rc = reach_from(G.as<int32_t>(), n, r, entry, seen.as<uint32_t>(), queue.as<int32_t>(), count.as<int32_t>(),
                        &stats[0]);
    if (rc) return rc;
    note("repair, reachable before", 0, stats[0]);
    int64_t reached = stats[0];
    for (int round = 0; round < 64 && reached < n; ++round) {
      if (round) note("repair round, reachable", round, reached);
      const int64_t nu = n - reached;
      if (nu > cap) {  // (the first round has the most, but for links that cost a vertex its only way in)
        cap = nu;
        for (DevBuf* b : {&unr_d, &pick_d, &qv_d, &w_d, &off_d, &v_d}) {
          (void)hipFree(b->p);
          b->p = nullptr;
        }
        HIP_OR_FAIL(unr_d.alloc(sizeof(int32_t) * (size_t)cap), "hipMalloc");
        HIP_OR_FAIL(pick_d.alloc(sizeof(int32_t) * (size_t)cap), "hipMalloc");
        HIP_OR_FAIL(qv_d.alloc(sizeof(float) * (size_t)(cap * d)), "hipMalloc");
        HIP_OR_FAIL(w_d.alloc(sizeof(int32_t) * (size_t)cap), "hipMalloc");
        HIP_OR_FAIL(off_d.alloc(sizeof(int32_t) * (size_t)(cap + 1)), "hipMalloc");
        HIP_OR_FAIL(v_d.alloc(sizeof(int32_t) * (size_t)cap), "hipMalloc");
      }
      HIP_OR_FAIL(hipMemset(count.p, 0, sizeof(int32_t)), "unreachable vertices");
      HIP_OR_FAIL(qgg::launch_unseen(seen.as<uint32_t>(), n, unr_d.as<int32_t>(), count.as<int32_t>(), nullptr),
                  "unreachable vertices");
      HIP_OR_FAIL(qgg::launch_gather(vectors, d, unr_d.as<int32_t>(), nu, qv_d.as<float>(), nullptr), "gather");
      if ((rc = encode())) return rc;
      for (int64_t q0 = 0; q0 < nu; q0 += chunk) {
        const int64_t nq = std::min(chunk, nu - q0);
        rc = qg_search_ex(B.idx, qv_d.as<float>() + q0 * d, nq, ef_build, ef_build, 0, sids.as<int32_t>(),
                          sdist.as<float>(), nullptr);
        if (rc) return rc;
        HIP_OR_FAIL(qgg::launch_pick(sids.as<int32_t>(), nq, ef_build, r, taken.as<unsigned long long>(),
                                     pick_d.as<int32_t>() + q0, nullptr),
                    "repair picks");
      }
      try {
        unr.resize((size_t)nu);
        pick.resize((size_t)nu);
        order.clear();
        order.reserve((size_t)nu);
        ws.clear();
        off.clear();
        vs.clear();
        HIP_OR_FAIL(hipMemcpy(unr.data(), unr_d.p, sizeof(int32_t) * (size_t)nu, hipMemcpyDeviceToHost), "download");
        HIP_OR_FAIL(hipMemcpy(pick.data(), pick_d.p, sizeof(int32_t) * (size_t)nu, hipMemcpyDeviceToHost), "download");
        for (int64_t a = 0; a < nu; ++a)
          if (pick[(size_t)a] >= 0)
            order.push_back((int64_t)((uint64_t)(uint32_t)pick[(size_t)a] << 32 | (uint32_t)unr[(size_t)a]));
        std::sort(order.begin(), order.end());
        for (int64_t x : order) {
          const int32_t w = (int32_t)(x >> 32);
          if (ws.empty() || ws.back() != w) {
            ws.push_back(w);
            off.push_back((int32_t)vs.size());
          }
          vs.push_back((int32_t)(x & 0xffffffff));
        }
        off.push_back((int32_t)vs.size());
      } catch (const std::bad_alloc&) {
        return qgi::set_error(QG_ENOMEM, "host buffer");
      }
      int32_t made = 0;
      HIP_OR_FAIL(hipMemcpy(w_d.p, ws.data(), sizeof(int32_t) * ws.size(), hipMemcpyHostToDevice), "upload");
      HIP_OR_FAIL(hipMemcpy(off_d.p, off.data(), sizeof(int32_t) * off.size(), hipMemcpyHostToDevice), "upload");
      HIP_OR_FAIL(hipMemcpy(v_d.p, vs.data(), sizeof(int32_t) * vs.size(), hipMemcpyHostToDevice), "upload");
      HIP_OR_FAIL(hipMemset(count.p, 0, sizeof(int32_t)), "links");
      HIP_OR_FAIL(qgg::launch_link(vectors, d, r, (int64_t)ws.size(), w_d.as<int32_t>(), off_d.as<int32_t>(),
                                   v_d.as<int32_t>(), G.as<int32_t>(), taken.as<unsigned long long>(),
                                   count.as<int32_t>(), nullptr),
                  "links");
      HIP_OR_FAIL(hipMemcpy(&made, count.p, sizeof made, hipMemcpyDeviceToHost), "links");
      stats[1] += made;
      rc = reach_from(G.as<int32_t>(), n, r, entry, seen.as<uint32_t>(), queue.as<int32_t>(), count.as<int32_t>(),
                      &reached);
      if (rc) return rc;
      if (!made) break;
    }
    stats[2] = reached;
    if (stats[2] != n) return qgi::set_error(QG_EUNSUPPORTED, "connectivity repair could not reach every vertex");
  }
  HIP_OR_FAIL(hipMemcpy(out_graph, G.p, sizeof(int32_t) * (size_t)(n * r), hipMemcpyDeviceToDevice), "copy graph");
  HIP_OR_FAIL(hipDeviceSynchronize(), "copy graph");
  stats[3] = std::chrono::duration_cast<std::chrono::microseconds>(std::chrono::steady_clock::now() - t0).count();
  if (out_stats) std::memcpy(out_stats, stats, sizeof stats);
  return QG_OK;
}
