// qg_graph.hip -- gfx950 kernels of the index construction (Algorithm 2,
// Sec. 3.2): candidate lists with exact distances, the NSG pruning rule, the
// angle-based refinement to exactly R edges with random fill, and the helpers
// of the connectivity repair.
//
// Arithmetic: every distance, norm and inner product the decisions rest on is
// an fp64 sum over dimensions 0 .. D-1 in ascending order, with a separate
// multiply and add per term (compiled with -ffp-contract=off), of differences
// of fp32 coordinates widened to fp64; cosines divide by the product of two
// square roots.  One lane computes one such sum, so its order is the
// sequential one.  Where an approximation with a known error already decides
// a comparison, the sum is not computed (prune_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qg_graph.h"

namespace qgg {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ int first_lane(uint64_t m) { return __ffsll((unsigned long long)m) - 1; }

// sum_t ((double)a[t] - (double)b[t])^2, t ascending
template <int U>  // four-dimension steps unrolled (their loads in flight together)
__device__ __forceinline__ double dist2_seq(const float* __restrict__ a, const float* __restrict__ b, int D) {
  double s = 0.0;
#pragma unroll U
  for (int t = 0; t < D; t += 4) {
    const float4 x = *reinterpret_cast<const float4*>(a + t);
    const float4 y = *reinterpret_cast<const float4*>(b + t);
    double d = (double)x.x - (double)y.x;
    s = s + d * d;
    d = (double)x.y - (double)y.y;
    s = s + d * d;
    d = (double)x.z - (double)y.z;
    s = s + d * d;
    d = (double)x.w - (double)y.w;
    s = s + d * d;
  }
  return s;
}

// ------------------------------------------------------------------ pruning

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kPruneWaves = 8;
constexpr int kPruneThreads = 64 * kPruneWaves;
// Bound on the error of a cosine the matrix cores compute from unit vectors
// rounded to f16 (see prune_kernel): each element is off by at most 2^-11 of
// itself, so the product sum by at most (2^-10 + 2^-22) sum |a||b| <= 2^-10 +
// 2^-22 (Cauchy-Schwarz); f16 subnormals flushed to zero add below 2^-19
// (elements are scaled by 2^12) and fp32 accumulation below D 2^-23 <= 2^-13
// for D <= 1024.  Sum 1.11e-3.
constexpr float kCosErr = 1.25e-3f;
constexpr float kUnitScale = 4096.0f;                        // f16 elements hold 2^12 times the unit vector's
// Smallest norm, relative to the largest, of a vector that is approximated: the
// factors 2^12 / norm and 2^23 / norm (which scales the limits, and times norms
// of at most 1 also the limits) then stay below 2^124 in fp32.  A shorter one,
// zero and NaN among them, gets NaN for a factor, and with it NaN products and
// limits: no comparison with them holds, so its pairs are left open.
constexpr double kMinNorm = 0x1p-100;

// Dynamic LDS of prune_kernel (bytes).  stage: the f16 rows of one chunk of KC
// dimensions, and before that the sort; occ: row w's bits over the 32-blocks
// from its own on; per candidate: exact distance, t value, id, the two scaled
// norms and the largest approximate cosine.
// stash: every thread's open pairs of `passes` passes (T tiles each).
struct PruneLds {
  int stage, occ, cd, tv, id, rw, hv, cmax, queue, kept, stash, total;
};
__host__ __device__ inline PruneLds prune_lds(int C, int R, int KC, int T, int passes) {
  const int nt = (C + 31) / 32, Cp = 32 * nt;
  int P = 1;
  while (P < C) P <<= 1;
  PruneLds s{};
  int o = 0;
  const int st = 2 * KC * Cp, so = 12 * P;
  s.stage = o;  o += ((st > so ? st : so) + 15) & ~15;
  s.occ = o;    o += 4 * 32 * (nt * (nt + 1) / 2);
  s.cd = o;     o += 8 * Cp;
  s.tv = o;     o += 8 * Cp;
  s.id = o;     o += 4 * Cp;
  s.rw = o;     o += 4 * Cp;
  s.hv = o;     o += 4 * Cp;
  s.cmax = o;   o += 4 * Cp;
  s.queue = o;  o += 4 * 128 * kPruneWaves;
  s.kept = o;   o += 4 * R + 4 * 64 + 16;  // kept ids, kept bits, scalars
  s.stash = (o + 15) & ~15;
  o = s.stash + 4 * kPruneThreads * ((T + 1) / 2) * passes;
  s.total = (o + 15) & ~15;
  return s;
}

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }
__device__ __forceinline__ bool lanes(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Doubles as integers of the same order (cosines; no NaN is ever stored).
__device__ __forceinline__ unsigned long long sortable64(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ int sortable32(float x) {
  const int u = __float_as_int(x);
  return u < 0 ? (u ^ 0x7fffffff) : u;
}
__device__ __forceinline__ float unsortable32(int s) { return __int_as_float(s < 0 ? (s ^ 0x7fffffff) : s); }

// sum_t (w_t - u_t)(v_t - u_t), t ascending, every term in fp64.
__device__ __forceinline__ double dot_seq(const float* __restrict__ xw, const float* __restrict__ xv,
                                          const float* __restrict__ xu, int D) {
  double s = 0.0;
#pragma unroll 8
  for (int t = 0; t < D; t += 4) {
    const float4 w4 = *reinterpret_cast<const float4*>(xw + t);
    const float4 v4 = *reinterpret_cast<const float4*>(xv + t);
    const float4 u4 = *reinterpret_cast<const float4*>(xu + t);
    s = s + ((double)w4.x - (double)u4.x) * ((double)v4.x - (double)u4.x);
    s = s + ((double)w4.y - (double)u4.y) * ((double)v4.y - (double)u4.y);
    s = s + ((double)w4.z - (double)u4.z) * ((double)v4.z - (double)u4.z);
    s = s + ((double)w4.w - (double)u4.w) * ((double)v4.w - (double)u4.w);
  }
  return s;
}

// One vertex u per workgroup of 8 wavefronts: candidate list, NSG rule and, on
// the last iteration, refinement and random fill.
//
// Candidates (Alg. 2, the search step of each iteration): the search results
// for x_u that are not u, then u's current neighbours not among them and not
// u; each with its exact squared distance to u; sorted by (distance, id).
//
// NSG rule (Sec. 3.2.1): scan the sorted candidates and keep v unless an
// already kept w is closer to v than u is, until R are kept.
//
// Refinement (Sec. 3.2.2).  For a vertex with fewer than R kept neighbours,
// each pruned candidate v gets t_v = the largest cosine, at u, between v and a
// candidate w closer to u (by (distance, id)); v survives an angle threshold
// theta iff t_v <= cos(theta).  The largest threshold leaving R - nk survivors
// has cos(theta*) = the (R - nk)-th smallest t_v (the limit of the paper's
// binary search); survivors are added in distance order.  Then fill[u]
// supplies neighbours while fewer than R are held (the paper's footnote:
// random neighbours when candidates are too few).
//
// Both rules ask about every pair of candidates w < v: is |w - v| < |v - u|,
// and is cos(w, v) the largest for v.  The pairs' cosines at u are products of
// a matrix of unit vectors with its transpose, so the matrix cores compute
// them all, from f16, with an error of at most kCosErr.  |w - v|^2 < |v - u|^2
// iff cos > |w - u| / (2 |v - u|), so every pair further than the error from
// that line is decided, and only a cosine within twice the error of its
// column's largest can be that column's largest.  The pairs that are left
// (about one in a hundred) are computed as the rules state them, in fp64, by
// lanes in parallel, for the refinement only in the columns whose largest
// cosine is near the threshold; every decision is therefore exactly that of
// the fp64 rule.  What remains of the NSG scan is one AND of a bit row per
// kept vertex.
//
// Computing every tested pair in fp64 by one lane each is what bound the
// pruning before: 50,000 x 128 at 232 candidates took 123 ms for the
// refinement, 4.4 ms per NSG pass and 2.9 ms for the candidate lists, and
// takes 5.0 ms per iteration now, refinement included; 6,001 x 960 at 214
// candidates 287, 8.6 and 1.5 ms, now 3.3 ms (4.45 while every column's largest
// cosine was computed exactly).  What bounds it now: at 960 dimensions the
// rows' bytes (about 3 MB a vertex, 6 TB/s through L2 and the last-level
// cache); at 128 latency, two workgroups a compute unit, of about 120,000
// cycles each 30,000 for the products with their loads, 18,000 for the
// comparisons, 15,000 for the distances, 15,000 for the exact sums, 12,000 for
// the order.
// T: 32 x 32 tiles of cosines a wavefront holds in one pass over the
// dimensions (16 registers each).
struct PruneArgs {
  const float* X;
  int64_t N;
  const int32_t* sids;  // [nu][EF] search results of vertices u0 ..
  const int32_t* G;     // [N][R] the current graph
  const int32_t* fill;
  int32_t* Gout;  // [N][R] (not G)
  int64_t u0;
  int D, EF, R, C, KC, refine;
  int stash;  // passes whose open pairs for the refinement are kept for later (all of them, or none)
};

template <int T>
__global__ __launch_bounds__(kPruneThreads, T <= 5 ? 4 : 2) void prune_kernel(PruneArgs a) {
  extern __shared__ __align__(16) uint8_t sm[];
  const int tid = threadIdx.x, lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, R = a.R, C = a.C, KC = a.KC;
  const float* __restrict__ X = a.X;
  const PruneLds L = prune_lds(C, R, KC, T, a.stash);
  _Float16* stage = reinterpret_cast<_Float16*>(sm + L.stage);
  uint32_t* occ = reinterpret_cast<uint32_t*>(sm + L.occ);
  double* cd = reinterpret_cast<double*>(sm + L.cd);
  unsigned long long* tv = reinterpret_cast<unsigned long long*>(sm + L.tv);
  int32_t* id = reinterpret_cast<int32_t*>(sm + L.id);
  float* rw = reinterpret_cast<float*>(sm + L.rw);
  float* hv = reinterpret_cast<float*>(sm + L.hv);
  int32_t* cmax = reinterpret_cast<int32_t*>(sm + L.cmax);
  uint32_t* queue = reinterpret_cast<uint32_t*>(sm + L.queue) + 128 * wave;
  int32_t* kept = reinterpret_cast<int32_t*>(sm + L.kept);  // R ids
  uint32_t* kbits = reinterpret_cast<uint32_t*>(kept + R);  // kept candidates, 32 a word (at most 34 words)
  int32_t* scal = reinterpret_cast<int32_t*>(kbits + 64);   // [0] candidate count, [1] kept count, [2] the approximate
                                                            // threshold, [3] some cosine is not approximated
  uint32_t* stash = reinterpret_cast<uint32_t*>(sm + L.stash) + tid;
  unsigned long long* cstar = reinterpret_cast<unsigned long long*>(sm + L.queue);  // once the queues are empty
  const int64_t u = a.u0 + blockIdx.x;
  const float* xu = X + u * D;

  // ---- the candidates' ids
  int P = 1;
  while (P < C) P <<= 1;
  unsigned long long* sk = reinterpret_cast<unsigned long long*>(sm + L.stage);  // P sort keys: distance bits
  int32_t* si = reinterpret_cast<int32_t*>(sk + P);                               // P ids
  int nres;  // search results among the candidates (the first ones)
  if (wave == 0) {
    const int32_t* srow = a.sids + (int64_t)blockIdx.x * a.EF;
    int n = 0;
    for (int e0 = 0; e0 < a.EF; e0 += 64) {
      const int e = e0 + lane;
      const int32_t v = e < a.EF ? srow[e] : -1;
      const bool ok = v >= 0 && v != (int32_t)u;
      const uint64_t m = ballot(ok);
      if (ok) si[n + lanes_below(m)] = v;
      n += __popcll(m);
    }
    if (lane == 0) {
      scal[0] = n;
      scal[3] = 0;
    }
  }
  __syncthreads();
  {
    // a neighbour list holds no id twice, so each is compared with the results
    // alone; the order of appending does not matter (the list is sorted next)
    nres = __builtin_amdgcn_readfirstlane(scal[0]);
    __syncthreads();
    const int32_t row = lane < R ? a.G[u * R + lane] : -1;  // R <= 64
    for (int j = wave; j < R; j += kPruneWaves) {
      const int32_t v = __builtin_amdgcn_readlane(row, j);
      if (v < 0 || v == (int32_t)u) continue;
      bool dup = false;
      for (int i = lane; i < nres; i += 64) dup |= si[i] == v;
      if (!ballot(dup) && lane == 0) si[atomicAdd(&scal[0], 1)] = v;
    }
  }
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(scal[0]);
  for (int i = tid; i < P; i += kPruneThreads) {
    unsigned long long k = ~0ull;  // padding sorts last
    if (i < n)
      k = (unsigned long long)__double_as_longlong(dist2_seq<8>(xu, X + (int64_t)si[i] * D, D));
    else
      si[i] = 0x7fffffff;
    sk[i] = k;  // a sum of squares: its bits order as the value does
  }
  __syncthreads();
  // The search results come ordered by their fp32 distances, which is nearly
  // always the fp64 order too.  If it is, only the neighbours after them have
  // to be merged in: everyone's place is its own number plus the others before
  // it.  Otherwise the whole list is sorted.
  auto before = [&](int i, int j) { return sk[i] < sk[j] || (sk[i] == sk[j] && si[i] < si[j]); };
  bool ordered = true;
  for (int i = tid; i + 1 < nres; i += kPruneThreads) ordered &= before(i, i + 1);
  if (__syncthreads_and(ordered)) {
    unsigned long long key[3];
    int32_t who[3];
    int place[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {  // n <= 1088
      const int i = tid + c * kPruneThreads;
      place[c] = -1;
      if (i < n) {
        key[c] = sk[i];
        who[c] = si[i];
        int pl = 0;
        for (int j = nres; j < n; ++j) pl += before(j, i);
        if (i < nres) {
          pl += i;
        } else {
          int lo = 0, hi = nres;  // results [0, lo) precede it
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (before(mid, i))
              lo = mid + 1;
            else
              hi = mid;
          }
          pl += lo;
        }
        place[c] = pl;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (place[c] >= 0) {
        sk[place[c]] = key[c];
        si[place[c]] = who[c];
      }
  } else {
    // bitonic sort; with a distance of at most 64 between partners a
    // wavefront's 128 elements are its own, so only the wider steps need the
    // barrier
    for (int k = 2; k <= P; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int t = tid; t < P / 2; t += kPruneThreads) {
          const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i | j;
          const bool up = (i & k) == 0;
          const unsigned long long di = sk[i], dl = sk[l];
          const int32_t ii = si[i], il = si[l];
          if ((di > dl || (di == dl && ii > il)) == up) {
            sk[i] = dl;
            sk[l] = di;
            si[i] = il;
            si[l] = ii;
          }
        }
        if (j > 64 || (j == 1 && k >= 128))
          __syncthreads();
        else
          wave_sync();
      }
  }
  __syncthreads();
  const int nt = (n + 31) / 32, nc = 32 * nt;
  const double smax = n > 0 ? __builtin_sqrt(__longlong_as_double((long long)sk[n - 1])) : 0.0;
  const double ismax = smax > 0.0 ? 1.0 / smax : 0.0;
  for (int i = tid; i < nc; i += kPruneThreads) {
    const bool live = i < n;
    const double d = live ? __longlong_as_double((long long)sk[i]) : 0.0;
    const double r = __builtin_sqrt(d) * ismax;
    cd[i] = d;
    id[i] = live ? si[i] : 0;
    rw[i] = (float)r;
    hv[i] = live ? (r >= kMinNorm ? 0.5f / (float)r : __builtin_nanf("")) : 0.0f;
    cmax[i] = sortable32(-2.0f * kUnitScale * kUnitScale);
    tv[i] = sortable64(-2.0);
  }

  // ---- every pair's cosine, and the pairs it does not decide
  // tile p of the triangle: columns (v) block J, rows (w) block I <= J
  auto occ_row = [&](int w) {  // word of block w / 32 in row w
    const int I = w >> 5;
    return 32 * (I * nt - I * (I - 1) / 2) + (w & 31) * (nt - I);
  };
  auto eval = [&](int which, uint32_t e) {
    const int w = (int)(e >> 16), v = (int)(e & 0xffffu);
    const float* xw = X + (int64_t)id[w] * D;
    const float* xv = X + (int64_t)id[v] * D;
    if (which == 0) {
      if (dist2_seq<8>(xw, xv, D) < cd[v]) atomicOr(&occ[occ_row(w) + (v >> 5) - (w >> 5)], 1u << (v & 31));
    } else {
      const double nw = cd[w], nv = cd[v];
      const double cs = (nv > 0.0 && nw > 0.0) ? dot_seq(xw, xv, xu, D) / (__builtin_sqrt(nv) * __builtin_sqrt(nw))
                                               : 1.0;
      if (cs > -2.0) atomicMax(&tv[v], sortable64(cs));
    }
  };
  const int half = lane >> 5;
  // Computes the pairs marked in mask (bit i of tile t: register i of its
  // cosines) exactly, 64 at a time: marked pairs are compacted into the
  // wavefront's queue, one bit per lane and step.
  auto drain = [&](int which, uint32_t (&mask)[(T + 1) / 2], const int (&tile)[T]) {
    int qn = 0;
    bool more = true;
    while (more) {
      more = false;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int I = tile[t] & 255, J = tile[t] >> 8;
        for (;;) {
          const uint32_t mine = (mask[t >> 1] >> (16 * (t & 1))) & 0xffffu;
          const uint64_t m = ballot(mine != 0);
          if (!m) break;
          if (qn >= 64) {
            more = true;
            break;
          }
          if (mine) {
            const int i = __builtin_ctz(mine);
            const int w = 32 * I + 8 * (i >> 2) + 4 * half + (i & 3);
            queue[qn + lanes_below(m)] = (uint32_t)w << 16 | (uint32_t)(32 * J + (lane & 31));
            mask[t >> 1] &= ~(1u << (i + 16 * (t & 1)));
          }
          qn += __popcll(m);
        }
      }
      wave_sync();
      if (lane < qn) eval(which, queue[lane]);
      qn = qn > 64 ? qn - 64 : 0;
      const uint32_t rest = lane < qn ? queue[64 + lane] : 0u;
      wave_sync();
      if (lane < qn) queue[lane] = rest;
      wave_sync();
      more = more || qn > 0;
    }
  };
  const int npairs = nt * (nt + 1) / 2;
  const int passes = (npairs + T * kPruneWaves - 1) / (T * kPruneWaves);
  const int per = passes ? (npairs + passes * kPruneWaves - 1) / (passes * kPruneWaves) : 0;  // tiles a wavefront holds
  auto tiles_from = [&](int p0, int (&tile)[T]) {  // the T tiles from p0 on
    int J = 0;
    while ((J + 1) * (J + 2) / 2 <= p0) ++J;
    int I = p0 - J * (J + 1) / 2;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      tile[t] = __builtin_amdgcn_readfirstlane(I | (J << 8));
      if (++I > J) {
        ++J;
        I = 0;
      }
    }
  };
  const int rowsh = KC == 64 ? 4 : KC == 32 ? 3 : 2;  // log2 of the lanes staging one row (four dimensions each)
  // place of a row's 16-byte slot s
  auto slot_of = [&](int s, int r) {
    return KC == 64 ? s ^ (r & 7) : KC == 32 ? s ^ ((r >> 1) & 3) : s ^ ((r >> 2) & 1);
  };
  for (int pass = 0; pass < passes; ++pass) {
    const int p0 = (pass * kPruneWaves + wave) * per;
    const int mine = p0 >= npairs ? 0 : (npairs - p0 < per ? npairs - p0 : per);
    int tile[T];  // I | J << 8
    tiles_from(p0, tile);
    float16v acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
    for (int k0 = 0; k0 < D; k0 += KC) {
      __syncthreads();
      {
        // row r's KC dimensions, 16-byte slots swizzled by the row so that the
        // operand reads of eight consecutive rows fall in different banks
        const int c = (tid & ((1 << rowsh) - 1)) * 4;
        const float4 u4 = *reinterpret_cast<const float4*>(xu + k0 + c);
        for (int r = tid >> rowsh; r < nc; r += kPruneThreads >> rowsh) {
          const float4 x4 = *reinterpret_cast<const float4*>(X + (int64_t)id[r] * D + k0 + c);
          const float f = hv[r] * (2.0f * kUnitScale);  // 2^12 |max| / |r|; 0 for padding
          half4 h;
          h.x = (_Float16)((float)(((double)x4.x - (double)u4.x) * ismax) * f);
          h.y = (_Float16)((float)(((double)x4.y - (double)u4.y) * ismax) * f);
          h.z = (_Float16)((float)(((double)x4.z - (double)u4.z) * ismax) * f);
          h.w = (_Float16)((float)(((double)x4.w - (double)u4.w) * ismax) * f);
          const int slot = slot_of(c >> 3, r);
          *reinterpret_cast<half4*>(stage + r * KC + slot * 8 + (c & 4)) = h;
        }
      }
      __syncthreads();
      for (int ks = 0; ks < KC; ks += 16) {
        const int s = (ks >> 3) + (lane >> 5), r = lane & 31;
        const int slot = slot_of(s, r);
        const _Float16* base = stage + r * KC + slot * 8;
#pragma unroll
        for (int t = 0; t < T; ++t)
          if (t < mine) {
            const half8 A = *reinterpret_cast<const half8*>(base + (tile[t] & 255) * 32 * KC);
            const half8 B = *reinterpret_cast<const half8*>(base + (tile[t] >> 8) * 32 * KC);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B, acc[t], 0, 0, 0);
          }
      }
    }
    // lane l holds column v = 32 J + l % 32, rows w = 32 I + 8 (i / 4) + 4 (l / 32) + i % 4
    // The comparisons are made on the products as they are, against limits
    // scaled alike.  A pair with a norm below kMinNorm has a NaN product, and is
    // left open by every comparison.  So is one whose |w - u| is lost beside
    // |v - u|; that is looked for once a tile, in its first row, which has the
    // smallest |w - u|.
    uint32_t mask[(T + 1) / 2], maskb[(T + 1) / 2];
#pragma unroll
    for (int t = 0; t < (T + 1) / 2; ++t) mask[t] = maskb[t] = 0;
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (t < mine) {
        const int I = tile[t] & 255, J = tile[t] >> 8, v = 32 * J + (lane & 31);
        const float h = hv[v] * (kUnitScale * kUnitScale);
        const int w0 = 32 * I + 4 * half;
        const int below = (I == J ? v - w0 : 32) & (v < n ? -1 : 0);  // rows w0 + o with o < below are pairs
        const bool plain = (ballot(rw[32 * I] * h < 1e-6f * kUnitScale * kUnitScale) & ballot(v < n)) == 0;
        float cm = -2.0f * kUnitScale * kUnitScale;
        uint32_t open = 0;  // pairs the approximation leaves open
        uint32_t word = 0;  // lane i, 32 + i: the bits of this tile's register i
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int o = 8 * (i >> 2) + (i & 3);
          const float c = acc[t][i], r = rw[w0 + o];
          const uint64_t pair = ballot(o < below);
          uint64_t yes = ballot(c > __builtin_fmaf(r, h, kCosErr * kUnitScale * kUnitScale)) & pair;
          uint64_t no = ballot(c < __builtin_fmaf(r, h, -kCosErr * kUnitScale * kUnitScale));
          uint64_t can = ~0ull;
          if (!plain) {
            can = ballot(r * h >= 1e-6f * kUnitScale * kUnitScale);
            yes &= can;
            no &= can;
            if ((pair & ~can) && lane == 0) scal[3] = 1;
          }
          word = lanes(1ull << i) ? (uint32_t)yes : word;
          word = lanes(1ull << (32 + i)) ? (uint32_t)(yes >> 32) : word;
          open |= lanes(pair & ~yes & ~no) ? 1u << i : 0u;
          if (a.refine) cm = lanes(pair & can) ? fmaxf(cm, c) : cm;
          asm volatile("" : "+v"(open), "+v"(cm), "+v"(word));  // row by row
        }
        const int wr = 32 * I + 8 * ((lane & 15) >> 2) + 4 * half + (lane & 3);
        if ((lane & 31) < 16) occ[occ_row(wr) + J - I] = word;
        mask[t >> 1] |= open << (16 * (t & 1));
        if (ballot(v < n && !(h < 3e38f)) && lane == 0) scal[3] = 1;
        if (a.refine && below > 0) atomicMax(&cmax[v], sortable32(cm));
      }
    if (a.refine) {
      __syncthreads();  // every wavefront's column maxima of this pass
#pragma unroll
      for (int t = 0; t < T; ++t)
        if (t < mine) {
          const int I = tile[t] & 255, J = tile[t] >> 8, v = 32 * J + (lane & 31);
          const float h = hv[v] * (kUnitScale * kUnitScale);
          const float lim = unsortable32(cmax[v]) - 2.0f * kCosErr * kUnitScale * kUnitScale;
          const int w0 = 32 * I + 4 * half;
          const int below = (I == J ? v - w0 : 32) & (v < n ? -1 : 0);
          const bool plain = (ballot(rw[32 * I] * h < 1e-6f * kUnitScale * kUnitScale) & ballot(v < n)) == 0;
          uint32_t open = 0;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int o = 8 * (i >> 2) + (i & 3);
            uint64_t out = ballot(acc[t][i] < lim);
            if (!plain) out &= ballot(rw[w0 + o] * h >= 1e-6f * kUnitScale * kUnitScale);
            open |= lanes(ballot(o < below) & ~out) ? 1u << i : 0u;
            asm volatile("" : "+v"(open));
          }
          maskb[t >> 1] |= open << (16 * (t & 1));
        }
    }
    // the products are used up: their registers hold the rows of the exact sums
    drain(0, mask, tile);
    if (a.refine) {
      if (a.stash) {
#pragma unroll
        for (int t = 0; t < (T + 1) / 2; ++t) stash[kPruneThreads * (pass * ((T + 1) / 2) + t)] = maskb[t];
      } else {
        drain(1, maskb, tile);
      }
    }
  }
  __syncthreads();

  // ---- the NSG scan: wavefront 0, lane l holds the undecided candidates 32 l ..
  if (wave == 0) {
    uint32_t alive = 0, kb = 0;
    if (lane < nt) alive = n - 32 * lane >= 32 ? ~0u : (1u << (n - 32 * lane)) - 1u;
    int nk = 0;
    while (nk < R) {
      const uint64_t m = ballot(alive != 0);
      if (!m) break;
      const int J = first_lane(m);
      const int b = __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)alive, J));
      const int f = 32 * J + b;
      if (lane == 0) kept[nk] = id[f];
      ++nk;
      if (lane >= J && lane < nt) alive &= ~occ[occ_row(f) + lane - J];
      if (lane == J) {
        alive &= ~(1u << b);
        kb |= 1u << b;
      }
    }
    if (lane < nt) kbits[lane] = kb;
    if (lane == 0) scal[1] = nk;
  }
  __syncthreads();
  int nk = __builtin_amdgcn_readfirstlane(scal[1]);
  if (a.refine && nk < R) {
    // ---- refinement: the threshold is the need-th smallest t of the pruned
    const int np = n - nk, need = R - nk < np ? R - nk : np;
    auto is_kept = [&](int i) { return (kbits[i >> 5] >> (i & 31)) & 1; };
    if (a.stash) {
      // The need-th smallest of the columns' approximate maxima is within
      // kCosErr of the threshold, so a column further than twice that from it
      // survives or does not whatever its exact value; the few others are
      // computed.  (All are, where some cosine has no approximation.)
      int32_t* exact = reinterpret_cast<int32_t*>(hv);  // the norms are used up
      const bool all = scal[3] != 0;
      for (int i = tid; i < nc; i += kPruneThreads)
        if (i >= n || is_kept(i)) cmax[i] = 0x7fffffff;  // after every pruned one
      __syncthreads();
      for (int i = tid; i < n; i += kPruneThreads) {
        const int x = cmax[i];
        if (x == 0x7fffffff) continue;
        int lt = 0, le = 0;
        for (int j = 0; j < nc; j += 4) {
          const int4 y = *reinterpret_cast<const int4*>(cmax + j);
          lt += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
          le += (y.x <= x) + (y.y <= x) + (y.z <= x) + (y.w <= x);
        }
        if (lt < need && need <= le) scal[2] = x;  // the same value from every lane that finds it
      }
      __syncthreads();
      const float c = unsortable32(scal[2]), w = 2.0f * kCosErr * kUnitScale * kUnitScale;
      for (int i = tid; i < nc; i += kPruneThreads) {
        const bool pruned = i < n && !is_kept(i);
        const float x = unsortable32(cmax[i]);
        const bool lower = !all && x < c - w, upper = !all && x > c + w;
        exact[i] = pruned && !lower && !upper;
        if (pruned && lower) tv[i] = 0;
        if (pruned && upper) tv[i] = ~1ull;
      }
      __syncthreads();
      for (int pass = 0; pass < passes; ++pass) {
        const int p0 = (pass * kPruneWaves + wave) * per;
        const int mine = p0 >= npairs ? 0 : (npairs - p0 < per ? npairs - p0 : per);
        int tile[T];
        tiles_from(p0, tile);
        uint32_t mask[(T + 1) / 2];
#pragma unroll
        for (int t = 0; t < (T + 1) / 2; ++t) mask[t] = stash[kPruneThreads * (pass * ((T + 1) / 2) + t)];
#pragma unroll
        for (int t = 0; t < T; ++t)
          if (t >= mine || !exact[t < mine ? 32 * (tile[t] >> 8) + (lane & 31) : 0])
            mask[t >> 1] &= ~(0xffffu << (16 * (t & 1)));
        drain(1, mask, tile);
      }
      __syncthreads();
    }
    for (int i = tid; i < n; i += kPruneThreads)
      if (is_kept(i)) tv[i] = ~0ull;  // kept: counts above every pruned one
    __syncthreads();
    for (int i = tid; i < n; i += kPruneThreads) {
      const unsigned long long x = tv[i];
      if (x == ~0ull) continue;
      int lt = 0, le = 0;
#pragma unroll 4
      for (int j = 0; j < n; ++j) {
        const unsigned long long y = tv[j];
        lt += y < x;
        le += y <= x;
      }
      if (lt < need && need <= le) *cstar = x;  // the same value from every lane that finds it
    }
    __syncthreads();
    if (wave == 0) {
      const unsigned long long cut = np > 0 ? *cstar : 0ull;
      for (int b = 0; b < n && nk < R; b += 64) {
        const int i = b + lane;
        const bool ok = i < n && tv[i] <= cut;
        const uint64_t m = ballot(ok);
        const int pos = nk + lanes_below(m);
        if (ok && pos < R) kept[pos] = id[i];
        nk = nk + __popcll(m) < R ? nk + __popcll(m) : R;
      }
      wave_sync();
      // too few candidates: random neighbours
      for (int f = 0; nk < R && f < R; ++f) {
        const int32_t v = a.fill[u * R + f];
        if (v < 0 || v == (int32_t)u) continue;
        bool dup = false;
        for (int k = lane; k < nk; k += 64) dup |= kept[k] == v;
        if (ballot(dup)) continue;
        if (lane == 0) kept[nk] = v;
        ++nk;
        wave_sync();
      }
    }
  }
  if (wave == 0) {
    wave_sync();
    for (int j = lane; j < R; j += 64) a.Gout[u * R + j] = j < nk ? kept[j] : -1;
  }
}

// Repair helper: rows of X listed in ids, gathered into out[n][D].
__global__ __launch_bounds__(256) void gather_kernel(const float* __restrict__ X, int D, const int32_t* __restrict__ ids,
                                                     int64_t n, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n * D) return;
  const int64_t r = i / D, c = i % D;
  out[i] = X[(int64_t)ids[r] * D + c];
}

// One level of a breadth-first search: the neighbours of the `size` vertices
// queue[base, base + size) that are not in `seen` yet enter it and the queue
// behind them.  Level l of a run of levels (l = level): its size is count[l] and
// its start `base` plus the sizes of the levels before it, all written by the
// launches before; the vertices it finds are counted in count[l + 1].  So
// several levels run without the host (on the host the search of a 50,000 x 32
// graph took 2 ms, mostly cache misses; here a level takes about 5 us).
__global__ __launch_bounds__(256) void bfs_level_kernel(const int32_t* __restrict__ G, int R, int64_t n, int level,
                                                        int64_t base, int32_t* __restrict__ queue,
                                                        uint32_t* __restrict__ seen, int32_t* count) {
  for (int l = 0; l < level; ++l) base += count[l];
  const int64_t size = count[level], next = base + size;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < size * R; e += (int64_t)gridDim.x * 256) {
    const int32_t v = G[(int64_t)queue[base + e / R] * R + e % R];
    if (v < 0 || v >= n) continue;
    const uint32_t bit = 1u << (v & 31);
    if (seen[v >> 5] & bit) continue;  // a stale word only costs the atomic
    if (!(atomicOr(seen + (v >> 5), bit) & bit)) queue[next + atomicAdd(count + level + 1, 1)] = v;
  }
}

// The vertices not in `seen`, in any order, counted in *count.
__global__ __launch_bounds__(256) void unseen_kernel(const uint32_t* __restrict__ seen, int64_t n,
                                                     int32_t* __restrict__ out, int32_t* count) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v < n && !((seen[v >> 5] >> (v & 31)) & 1u)) out[atomicAdd(count, 1)] = (int32_t)v;
}

// Repair: for each of nq searches (ids[nq][EF], padded with -1) the nearest
// result that has a slot not taken by a repair, or -1.  One wavefront each;
// taken[v]: bit j = slot j of v.
__global__ __launch_bounds__(64) void pick_kernel(const int32_t* __restrict__ ids, int EF, int R,
                                                  const unsigned long long* __restrict__ taken,
                                                  int32_t* __restrict__ pick) {
  const int lane = lane_id();
  const int32_t* row = ids + (int64_t)blockIdx.x * EF;
  const unsigned long long full = R >= 64 ? ~0ull : (1ull << R) - 1ull;
  int32_t w = -1;
  for (int b = 0; b < EF; b += 64) {
    const int32_t x = b + lane < EF ? row[b + lane] : -1;
    const uint64_t m = ballot(x >= 0 && taken[x >= 0 ? x : 0] != full);
    if (m) {
      w = __builtin_amdgcn_readlane(x, first_lane(m));
      break;
    }
  }
  if (lane == 0) pick[blockIdx.x] = w;
}

// Repair: group g links the vertices v[off[g] .. off[g + 1]) (in that order)
// from w[g]: they take w's empty slots in slot order, then its edges not taken
// by a repair, farthest first (fp64, ties to the larger id), while slots are
// left.  One wavefront per group, lane j slot j (R <= 64); *made counts the
// links.
__global__ __launch_bounds__(64) void link_kernel(const float* __restrict__ X, int D, int R,
                                                  const int32_t* __restrict__ w, const int32_t* __restrict__ off,
                                                  const int32_t* __restrict__ v, int32_t* __restrict__ G,
                                                  unsigned long long* __restrict__ taken, int32_t* made) {
  const int lane = lane_id();
  const int64_t u = w[blockIdx.x];
  const int o = off[blockIdx.x], cnt = off[blockIdx.x + 1] - o;
  const unsigned long long tk = taken[u];
  const int32_t id = lane < R ? G[u * R + lane] : 0;
  const bool empty = lane < R && id < 0, edge = lane < R && id >= 0 && !((tk >> lane) & 1ull);
  const uint64_t em = ballot(empty), ed = ballot(edge);
  const double d = edge ? dist2_seq<8>(X + u * D, X + (int64_t)id * D, D) : 0.0;
  int rank = empty ? lanes_below(em) : __popcll(em);
  for (uint64_t m = ed; m; m &= m - 1) {
    const int i = first_lane(m);
    const uint64_t b = (uint64_t)__double_as_longlong(d);
    const double di = __longlong_as_double(
        (long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), i) << 32 |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, i)));
    const int32_t ii = __builtin_amdgcn_readlane(id, i);
    if (edge) rank += di > d || (di == d && ii > id);
  }
  const bool use = (empty || edge) && rank < cnt;
  if (use) G[u * R + lane] = v[o + rank];
  const uint64_t um = ballot(use);
  if (lane == 0) {
    taken[u] = tk | um;
    atomicAdd(made, __popcll(um));
  }
}

hipError_t launch_prune(const float* X, int D, const int32_t* sids, int EF, const int32_t* G, int R, int64_t N,
                        int64_t u0, int64_t nu, int refine, const int32_t* fill, int32_t* Gout, hipStream_t st) {
  if (nu <= 0) return hipSuccess;
  const int C = EF + R;  // EF results and R old neighbours
  if (D % 32 || D > 1024 || R > 64 || C > 32 * 34) return hipErrorInvalidValue;
  // lists of up to 256 candidates are 36 tiles, 5 a wavefront: few enough
  // registers for two workgroups on a compute unit; longer lists hold 10 a
  // wavefront and go over the dimensions again for the tiles beyond 80
  const int T = C <= 256 ? 5 : 10, nt = (C + 31) / 32;
  const int passes = (nt * (nt + 1) / 2 + T * kPruneWaves - 1) / (T * kPruneWaves);
  // Chunks of 64 dimensions where they divide (half as many waits for the rows'
  // loads as with 32; two workgroups of the five-tile kernel still fit a
  // compute unit), fewer where the lists are so long that the LDS asks for it;
  // beyond that the refinement's pairs are computed pass by pass, not kept
  int KC = D % 64 ? 32 : 64, stash = refine ? passes : 0;
  while (prune_lds(C, R, KC, T, stash).total > 160 * 1024) {
    if (KC > 32)
      KC = 32;
    else if (stash)
      stash = 0;
    else
      KC = 16;
  }
  const size_t lds = (size_t)prune_lds(C, R, KC, T, stash).total;
  const PruneArgs a{X, N, sids, G, fill, Gout, u0, D, EF, R, C, KC, refine, stash};
  auto go = [&](auto kern) {
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)nu), dim3(kPruneThreads), lds, st, a);
    return hipGetLastError();
  };
  return T == 5 ? go(prune_kernel<5>) : go(prune_kernel<10>);
}

hipError_t launch_gather(const float* X, int D, const int32_t* ids, int64_t n, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((n * D + 255) / 256)), dim3(256), 0, st, X, D, ids, n, out);
  return hipGetLastError();
}

hipError_t launch_bfs_level(const int32_t* G, int R, int64_t n, int level, int64_t base, int32_t* queue,
                            uint32_t* seen, int32_t* count, hipStream_t st) {
  const int64_t blocks = (n * R + 255) / 256;
  hipLaunchKernelGGL(bfs_level_kernel, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), 0, st, G, R, n, level,
                     base, queue, seen, count);
  return hipGetLastError();
}

hipError_t launch_unseen(const uint32_t* seen, int64_t n, int32_t* out, int32_t* count, hipStream_t st) {
  hipLaunchKernelGGL(unseen_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, seen, n, out, count);
  return hipGetLastError();
}

hipError_t launch_pick(const int32_t* ids, int64_t nq, int EF, int R, const unsigned long long* taken, int32_t* pick,
                       hipStream_t st) {
  if (nq <= 0) return hipSuccess;
  hipLaunchKernelGGL(pick_kernel, dim3((unsigned)nq), dim3(64), 0, st, ids, EF, R, taken, pick);
  return hipGetLastError();
}

hipError_t launch_link(const float* X, int D, int R, int64_t groups, const int32_t* w, const int32_t* off,
                       const int32_t* v, int32_t* G, unsigned long long* taken, int32_t* made, hipStream_t st) {
  if (groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(link_kernel, dim3((unsigned)groups), dim3(64), 0, st, X, D, R, w, off, v, G, taken, made);
  return hipGetLastError();
}

}  // namespace qgg
