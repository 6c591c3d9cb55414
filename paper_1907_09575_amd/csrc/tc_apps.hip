// tc_apps.hip - the uses of exact triangle counts that the paper's
// introduction (Section 1) names, built on the per-edge support of Eq. 1's
// intersections: per-vertex triangle counts, local clustering coefficients
// and transitivity, and the k-truss decomposition.
//
// Per-vertex counts: the count kernels credit every triangle a < b < k to its
// three vertices: a by task, b by hashed row, k by the hashed row's keys, each
// summed on chip before its atomic. (Summing half the full support over every
// vertex's edges needs an atomic per triangle for the edges (a, k) and the
// column lists below: clustering at RMAT scale 20
// 6.29 ms, 1.90 ms this way.)
//
// k-truss needs every vertex's full neighbourhood, not only U: the lower part
// L_v = {a : v in U_a} (U's column lists) is built by a stable radix sort of
// U's entries by column, each keeping the U position of its edge. In rank
// space every entry of L_v is below v and every entry of U_v above it, so
// N(v) in ascending order is L_v followed by U_v, with no merge.
//
// k-truss: the k-truss is the largest subgraph whose every edge lies in at
// least k - 2 of its triangles; an edge's trussness is the largest k whose
// k-truss holds it. Peeling, level by level: starting from the full support,
// every round removes the alive edges whose current support is below k - 2
// (trussness k - 1) and takes the triangles they close out of the support of
// their other two edges; when a round removes nothing, k rises to the next
// level that removes something. A triangle that loses several edges in one
// round is taken out once, by its removed edge of smallest id; a triangle
// with an edge removed in an earlier round is already gone.
#include <algorithm>
#include <cstdlib>

#include "tc_prims.h"

namespace tc {

namespace {

constexpr int kAT = 256;
inline unsigned grid_threads(int64_t n) { return (unsigned)std::max<int64_t>(1, div_up(n, kAT)); }
inline unsigned grid_waves(int64_t n) { return wave_grid(n); }  // (one wave per item, grid-stride)

// ---- lower adjacency ---------------------------------------------------------

struct Lower {
  DevBuf ptr;   // int64 [n + 1]: L_v = [ptr[v], ptr[v + 1])
  DevBuf nbr;   // int32 [m]: a of every entry, ascending within a column
  DevBuf eid;   // int32 [m]: U position of the edge (a, v)
  DevBuf erow;  // uint32 [m]: row of every U entry
};

__global__ void k_lower_keys(const int32_t* __restrict__ col, const uint32_t* __restrict__ erow, int64_t m,
                             uint32_t* __restrict__ key, uint64_t* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  key[i] = (uint32_t)col[i];
  val[i] = (uint64_t)erow[i] | ((uint64_t)i << 32);
}

__global__ void k_lower_split(const uint64_t* __restrict__ val, int64_t m, int32_t* __restrict__ nbr,
                              int32_t* __restrict__ eid) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const uint64_t v = val[i];
  nbr[i] = (int32_t)(uint32_t)v;
  eid[i] = (int32_t)(v >> 32);
}

__global__ void k_fill_i64v(int64_t* p, int64_t n, int64_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

void build_lower(Lower& L, const Graph& g, hipStream_t st) {
  const int64_t n = g.n, m = g.m;
  L.ptr.alloc(sizeof(int64_t) * (size_t)(n + 1));
  L.nbr.alloc(sizeof(int32_t) * (size_t)std::max<int64_t>(m, 1));
  L.eid.alloc(sizeof(int32_t) * (size_t)std::max<int64_t>(m, 1));
  L.erow.alloc(sizeof(uint32_t) * (size_t)std::max<int64_t>(m, 1));
  if (m == 0) {
    TC_LAUNCH("fill_i64", k_fill_i64v, dim3(grid_threads(n + 1)), dim3(kAT), 0, st, L.ptr.as<int64_t>(), n + 1,
              (int64_t)0);
    return;
  }
  TC_LAUNCH("entry_rows", k_entry_rows, dim3(entry_rows_grid(n)), dim3(kAT), 0, st, g.row_ptr, n,
            L.erow.as<uint32_t>());
  DevBuf ka(sizeof(uint32_t) * (size_t)m), kb(sizeof(uint32_t) * (size_t)m);
  DevBuf va(sizeof(uint64_t) * (size_t)m), vb(sizeof(uint64_t) * (size_t)m);
  TC_LAUNCH("lower_keys", k_lower_keys, dim3(grid_threads(m)), dim3(kAT), 0, st, g.col, L.erow.as<uint32_t>(), m,
            ka.as<uint32_t>(), va.as<uint64_t>());
  // stable by column: within a column the rows keep U's ascending order
  const bool alt = radix_sort<uint32_t, uint64_t>(ka.as<uint32_t>(), kb.as<uint32_t>(), va.as<uint64_t>(),
                                                  vb.as<uint64_t>(), m, 0, g.sbits, st, "lower");
  const uint32_t* keys = alt ? kb.as<uint32_t>() : ka.as<uint32_t>();
  const uint64_t* vals = alt ? vb.as<uint64_t>() : va.as<uint64_t>();
  TC_LAUNCH("bounds", (k_bounds<uint32_t>), dim3(grid_threads(n + 1)), dim3(kAT), 0, st, keys, m, 0, n,
            L.ptr.as<int64_t>());
  TC_LAUNCH("lower_split", k_lower_split, dim3(grid_threads(m)), dim3(kAT), 0, st, vals, m, L.nbr.as<int32_t>(),
            L.eid.as<int32_t>());
  TC_HIP(hipGetLastError());
}

// ---- per-vertex counts and clustering ------------------------------------------

// Per original vertex u (rank r = perm[u]): t, the local clustering
// coefficient t / C(d, 2) (0 if d < 2; one correctly rounded division of two
// exact integers) and the sums of t (= 3T) and of C(d, 2) over all vertices.
// (every work-group ends on two atomics to the sums, of 12 ns each: few
// work-groups)
constexpr unsigned kVertexOutGrid = 1024;
__global__ __launch_bounds__(256) void k_vertex_out(const int32_t* __restrict__ perm, int64_t n,
                                                    const unsigned long long* __restrict__ t_rank,
                                                    const uint32_t* __restrict__ deg, int64_t* __restrict__ t_orig,
                                                    double* __restrict__ cc, unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long s_t[4], s_w[4];
  uint64_t t_all = 0, pairs_all = 0;
  const uint32_t hot = vertex_hot(n);
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = perm[u], top = n - 1 - r;
    uint64_t t = 0;
    if (top >= hot) {
      t = t_rank[r];
    } else {
#pragma unroll
      for (uint32_t c = 0; c < kVertexCopies; ++c) t += t_rank[n + (int64_t)c * hot + top];
    }
    const uint64_t d = deg[r];
    const uint64_t pairs = d * (d - (d > 0)) / 2;
    if (t_orig) t_orig[u] = (int64_t)t;
    if (cc) cc[u] = pairs ? (double)t / (double)pairs : 0.0;
    t_all += t;
    pairs_all += pairs;
  }
  if (!sums) return;
  const unsigned long long wt = wave_sum((unsigned long long)t_all), ww = wave_sum((unsigned long long)pairs_all);
  if (lane_id() == 0) {
    s_t[threadIdx.x >> 6] = wt;
    s_w[threadIdx.x >> 6] = ww;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long a = s_t[0] + s_t[1] + s_t[2] + s_t[3], b = s_w[0] + s_w[1] + s_w[2] + s_w[3];
    if (a) atomicAdd(&sums[0], a);
    if (b) atomicAdd(&sums[1], b);
  }
}

__global__ void k_zero_u64x2(unsigned long long* p) {
  if (threadIdx.x < 2) p[threadIdx.x] = 0;
}

// Per-vertex counts are not for a stream that is being captured: their
// temporaries go back to the cache when the call returns, so a replay would
// write into memory of others. Checked before anything is recorded (the fill of
// a first temporary would be).
void require_no_capture(hipStream_t st) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  TC_HIP(hipStreamIsCapturing(st, &cs));
  TC_REQUIRE(cs == hipStreamCaptureStatusNone, TC_EDEVICE, "per-vertex triangle counts: the stream is being captured");
}

void vertex_counts(const Graph& g, int64_t* d_tri, double* d_cc, int64_t* d_sums, hipStream_t st) {
  require_plain(g, "per-vertex triangle counts");
  require_no_capture(st);
  TempStream temps(st);
  const int64_t n = g.n;
  auto* sums = reinterpret_cast<unsigned long long*>(d_sums);
  if (sums) TC_LAUNCH("zero_sums", k_zero_u64x2, dim3(1), dim3(64), 0, st, sums);
  const int64_t nc = vertex_counters(n);
  DevBuf t_rank(sizeof(unsigned long long) * (size_t)nc), erow(sizeof(uint32_t) * (size_t)std::max<int64_t>(g.m, 1));
  TC_LAUNCH("fill_i64", k_fill_i64v, dim3(grid_threads(nc)), dim3(kAT), 0, st, t_rank.as<int64_t>(), nc, (int64_t)0);
  if (g.m > 0)
    TC_LAUNCH("entry_rows", k_entry_rows, dim3(entry_rows_grid(n)), dim3(kAT), 0, st, g.row_ptr, n,
              erow.as<uint32_t>());
  const VertexCounts vc{erow.as<uint32_t>(), t_rank.as<unsigned long long>()};
  launch_count(graph_view(g), MODE_VERTEX, nullptr, nullptr, nullptr, st, &vc);
  TC_LAUNCH("vertex_out", k_vertex_out, dim3(std::min(grid_threads(n), kVertexOutGrid)), dim3(kAT), 0, st, g.perm, n,
            t_rank.as<unsigned long long>(), g.deg, d_tri, d_cc, sums);
  TC_HIP(hipGetLastError());
  note_use(g, st);
}

// ---- k-truss ---------------------------------------------------------------------

constexpr int kPeelWaves = 8, kPeelThreads = 64 * kPeelWaves;
constexpr unsigned kPeelGrid = 1024;    // work-groups of a round: those resident at 8 waves per SIMD
constexpr int32_t kAlive = 0x7FFFFFFF;  // state of an edge not yet removed (else: its round)

// A removed edge's triangles are found by walking the neighbourhood of its
// endpoint of smaller degree d, cut into work entries of walk_chunk(d)
// neighbours (one wave each): the longest walk of a round would otherwise be
// one wave's, and a round is as long as its chain of dependent loads. At most
// `parts` entries per edge, 1 .. kWalkParts, of no fewer than 1024 / parts
// neighbours (RMAT scale 18, 1251 rounds: 46.5 ms with 8 of 256, 40.6 ms with
// 16 of 128, 38.2 ms with 16 of 64).
constexpr uint32_t kWalkParts = 16;
constexpr int kWalkChoices = 5;  // parts 16, 8, 4, 2, 1
__host__ __device__ inline uint32_t walk_chunk(uint32_t d, uint32_t parts) {
  const uint32_t c = ((d + parts - 1) / parts + 63) & ~63u, least = 1024 / parts;
  return c < least ? least : c;
}
__device__ __forceinline__ uint32_t walk_entries(uint32_t d, uint32_t parts) {
  const uint32_t c = walk_chunk(d, parts);
  return d ? (d + c - 1) / c : 1;
}

// Entries per edge at most: kWalkParts, or less by the environment variable
// TC_TRUSS_WALKS (so that tests reach the coarser walks at small sizes).
uint32_t truss_walks() {
  const char* v = std::getenv("TC_TRUSS_WALKS");
  return v != nullptr && v[0] != '\0' ? (uint32_t)std::strtoul(v, nullptr, 10) : kWalkParts;
}

// The peel's arrays. A work entry is an edge id and, above it, its chunk. Every
// edge is appended once in the whole peel, so one list of all entries holds
// them, round after round: rounds are numbered by the launches of
// k_truss_peel, round i takes the cnt[i] entries from start[i] on and appends
// the edges that its triangles bring below lim after them. No list is ever
// compacted from all edges but at a new level.
struct TrussArrays {
  const uint32_t* erow;
  const int32_t* col;
  const uint32_t* deg;
  int32_t* state;  // kAlive, or the round that removes the edge
  int32_t* sup;
  int32_t* tau;
  uint64_t* list;
  uint32_t parts;    // entries of an edge at most (walk_chunk)
  uint32_t entries;  // of all edges: a list that holds them has every edge removed
};

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__device__ __forceinline__ uint32_t min_degree(const TrussArrays& A, int32_t e) {
  return min(A.deg[A.erow[e]], A.deg[A.col[e]]);
}

// What the peel starts from: the work entries of all edges together, for 16, 8,
// 4, 2 and 1 entries per edge at most (what the list must hold), and the
// largest value of kAlive less the support and of the support. (Every
// work-group ends on seven atomics to one line, 12 ns each: few work-groups.)
struct TrussStart {
  unsigned long long entries[kWalkChoices];
  int room, top;
};
__global__ __launch_bounds__(256) void k_truss_start(TrussArrays A, int64_t m, TrussStart* __restrict__ out) {
  __shared__ unsigned long long s_w[4][kWalkChoices];
  __shared__ int s_room[4], s_top[4];
  unsigned long long c[kWalkChoices] = {};
  int room = 0, top = 0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t d = min_degree(A, (int32_t)e);
    const int s = A.sup[e];
    room = max(room, kAlive - s);
    top = max(top, s);
#pragma unroll
    for (int i = 0; i < kWalkChoices; ++i) c[i] += walk_entries(d, kWalkParts >> i);
  }
  room = wave_max(room);
  top = wave_max(top);
#pragma unroll
  for (int i = 0; i < kWalkChoices; ++i) {
    c[i] = wave_sum(c[i]);
    if (lane_id() == 0) s_w[threadIdx.x >> 6][i] = c[i];
  }
  if (lane_id() == 0) {
    s_room[threadIdx.x >> 6] = room;
    s_top[threadIdx.x >> 6] = top;
  }
  __syncthreads();
  if (threadIdx.x < kWalkChoices) {
    unsigned long long t = 0;
    for (int w = 0; w < 4; ++w) t += s_w[w][threadIdx.x];
    atomicAdd(&out->entries[threadIdx.x], t);
  } else if (threadIdx.x == kWalkChoices) {
    atomicMax(&out->room, max(max(s_room[0], s_room[1]), max(s_room[2], s_room[3])));
    atomicMax(&out->top, max(max(s_top[0], s_top[1]), max(s_top[2], s_top[3])));
  }
}

// A wave's edges for the next frontier, kept in LDS until there are enough for
// one atomic on the list's counter (an atomic per 64 edges serialises on it:
// 12 ns each, 0.76 ms for the first level of 4M edges).
constexpr uint32_t kPushQueue = 256;
struct PushQueue {
  int32_t* q;   // kPushQueue entries of this wave
  uint32_t n;   // (uniform)
  int32_t round, tau;
  uint64_t* list;  // the round's first entry
  uint32_t* cnt;
};

// Removes the queued edges in round Q.round (trussness Q.tau) and appends
// their work entries to Q.list, at the place that reserve(entries of the
// wave, held by lane 63) returns (to every lane).
template <class F>
__device__ __forceinline__ void truss_take(const TrussArrays& A, PushQueue& Q, F&& reserve) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int lane = lane_id();
  constexpr int kQ = kPushQueue / 64;
  uint32_t n[kQ], mine = 0;
#pragma unroll
  for (int j = 0; j < kQ; ++j) {
    const uint32_t i = 64u * j + (uint32_t)lane;
    n[j] = i < Q.n ? walk_entries(min_degree(A, Q.q[i]), A.parts) : 0;
    mine += n[j];
  }
  const uint32_t inc = wave_incl_scan(mine);
  uint32_t base = reserve(inc) + inc - mine;
#pragma unroll
  for (int j = 0; j < kQ; ++j) {
    if (n[j] == 0) continue;
    const int32_t e = Q.q[64 * j + lane];
    A.state[e] = Q.round;
    A.tau[e] = Q.tau;
    for (uint32_t c = 0; c < n[j]; ++c) Q.list[base++] = (uint64_t)(uint32_t)e | ((uint64_t)c << 32);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  Q.n = 0;
}

// One wave's queue, when it is full.
__device__ __forceinline__ void truss_flush(const TrussArrays& A, PushQueue& Q) {
  truss_take(A, Q, [&](uint32_t inc) {
    uint32_t base = 0;
    if (lane_id() == 63) base = atomicAdd(Q.cnt, inc);
    return (uint32_t)__shfl((int)base, 63, 64);
  });
}

// What is left in the queues of all waves of a work-group at its end, with
// one atomic (RMAT scale 18, k_truss_level on average: 22.5 us with one per
// wave, 11.5 us so). Call from all threads.
__device__ __forceinline__ void truss_flush_all(const TrussArrays& A, PushQueue& Q) {
  __shared__ uint32_t s_n[kPeelWaves], s_base;
  const int wave = threadIdx.x >> 6;
  truss_take(A, Q, [&](uint32_t inc) {
    if (lane_id() == 63) s_n[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < kPeelWaves; ++w) {
      if (w < wave) before += s_n[w];
      all += s_n[w];
    }
    if (threadIdx.x == 0 && all) s_base = atomicAdd(Q.cnt, all);
    __syncthreads();
    return (all ? s_base : 0u) + before;
  });
}

// Queues the edge e of the lanes with `take` set.
__device__ __forceinline__ void truss_push(const TrussArrays& A, PushQueue& Q, bool take, int32_t e) {
  const uint64_t mask = __ballot(take);
  if (mask == 0) return;
  if (take)
    Q.q[Q.n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0))] = e;
  Q.n += (uint32_t)__popcll(mask);
  if (Q.n > kPushQueue - 64) truss_flush(A, Q);
}

// A batch of rounds, b: when the frontier cnt[i] of its first round i is
// empty, k_truss_min finds the smallest support left, and k_truss_level makes
// the edges that have it the frontier of the next level (lim = it + 1, the
// trussness of what the level removes). Otherwise both do nothing and the
// level goes on. room: kAlive less the smallest support (cleared: none found).
__global__ __launch_bounds__(256) void k_truss_min(TrussArrays A, int64_t m, const uint32_t* __restrict__ start,
                                                   const uint32_t* __restrict__ cnt, int* __restrict__ room,
                                                   int* __restrict__ fresh) {
  if (*cnt != 0 || *start == A.entries) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) *fresh = 1;
  __shared__ int s_v[4];
  int v = kAlive;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const int s = A.sup[i];
    v = A.state[i] == kAlive ? min(v, s) : v;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = min(v, __shfl_xor(v, d, 64));
  if (lane_id() == 0) s_v[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    v = min(min(s_v[0], s_v[1]), min(s_v[2], s_v[3]));
    // (most work-groups find what another has written: 16.9 -> 11.7 us)
    if (kAlive - v > __hip_atomic_load(room, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(room, kAlive - v);
  }
}

// (lim, lim_out: the level's bound before and after; start: the first entry of
// the round)
__global__ __launch_bounds__(kPeelThreads) void k_truss_level(TrussArrays A, int64_t m, const int* __restrict__ fresh,
                                                     const int* __restrict__ room, const int* __restrict__ lim,
                                                     int* __restrict__ lim_out, int32_t round, const uint32_t* __restrict__ start,
                                                     uint32_t* __restrict__ cnt) {
  const bool go = *fresh != 0;  // (then an edge is left)
  const int bound = go ? kAlive - *room + 1 : *lim;
  if (blockIdx.x == 0 && threadIdx.x == 0) *lim_out = bound;
  if (!go) return;
  __shared__ int32_t s_q[kPeelWaves][kPushQueue];
  PushQueue Q{s_q[threadIdx.x >> 6], 0, round, bound + 1, A.list + *start, cnt};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < m; i0 += stride) {  // (uniform)
    const int64_t i = i0 + threadIdx.x;
    const bool take = i < m && A.state[i] == kAlive && A.sup[i] < bound;
    truss_push(A, Q, take, (int32_t)i);
  }
  truss_flush_all(A, Q);
}

// N(v) = L_v followed by U_v (ascending), with the U position of each edge.
struct FullAdj {
  const int64_t* row_ptr;
  const int32_t* col;
  const int64_t* lptr;
  const int32_t* lnbr;
  const int32_t* leid;
};

// Position in the sorted list a[0, len) holding w, or -1 (distinct entries,
// len < 2^31).
__device__ __forceinline__ int32_t find_sorted(const int32_t* __restrict__ a, uint32_t len, int32_t w) {
  // three pivots a step, read together: a walk is a chain of these loads
  uint32_t lo = 0, hi = len;  // the first entry >= w lies in [lo, hi]
  while (hi - lo > 3) {
    const uint32_t q = (hi - lo) >> 2, p1 = lo + q, p2 = p1 + q, p3 = p2 + q;
    const int32_t v1 = a[p1], v2 = a[p2], v3 = a[p3];
    hi = v1 >= w ? p1 : v2 >= w ? p2 : v3 >= w ? p3 : hi;
    lo = v3 < w ? p3 + 1 : v2 < w ? p2 + 1 : v1 < w ? p1 + 1 : lo;
  }
  int32_t at = -1;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j)
    if (lo + j < len && lo + j <= hi && a[lo + j] == w) at = (int32_t)(lo + j);
  return at;
}

// One wave per work entry of this round: edge e = (a, b), a chunk of the
// neighbourhood of the endpoint of smaller degree, whose every w is looked up
// in the other's (binary search in its L or U part); each triangle (e, e1, e2)
// still whole before this round, and whose removed edge of smallest id is e,
// takes one from the support of each of e1, e2 that stays, and an edge that
// this brings below lim goes to the next round's list (the one subtraction
// that crosses lim sees it). Edges marked for the next round count as staying.
__global__ __launch_bounds__(kPeelThreads) __attribute__((amdgpu_waves_per_eu(8)))
void k_truss_peel(TrussArrays T, FullAdj A, int32_t round, const int* __restrict__ limp,
                  const uint32_t* __restrict__ start, uint32_t* __restrict__ start_next,
                  const uint32_t* __restrict__ cnt, uint32_t* __restrict__ cnt_next) {
  const uint32_t nF = *cnt, end = *start + nF;
  if (blockIdx.x == 0 && threadIdx.x == 0) *start_next = end;
  // (with the last edges listed, none stays whose support would matter)
  if (blockIdx.x * kPeelWaves >= nF || end == T.entries) return;
  const uint64_t* const F = T.list + (end - nF);
  const int lim = *limp;
  __shared__ int32_t s_q[kPeelWaves][kPushQueue];
  PushQueue Q{s_q[threadIdx.x >> 6], 0, round + 1, lim + 1, T.list + end, cnt_next};
  const int lane = lane_id();
  const uint32_t stride = gridDim.x * (blockDim.x / 64);
  for (uint32_t f = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6); f < nF; f += stride) {
    const uint64_t w0 = F[f];
    const int32_t e = (int32_t)(uint32_t)w0;
    const int32_t a = (int32_t)T.erow[e], b = A.col[e];
    const int64_t lpa = A.lptr[a], lpb = A.lptr[b], rpa = A.row_ptr[a], rpb = A.row_ptr[b];
    const uint32_t la = (uint32_t)(A.lptr[a + 1] - lpa), lb = (uint32_t)(A.lptr[b + 1] - lpb);
    const uint32_t da = T.deg[a], db = T.deg[b];
    const bool a_small = da <= db;
    const int32_t y = a_small ? b : a;
    const uint32_t lx = a_small ? la : lb, dx = a_small ? da : db;
    const uint32_t ly = a_small ? lb : la, uy = (a_small ? db : da) - ly;
    const int64_t lpx = a_small ? lpa : lpb, rpx = (a_small ? rpa : rpb) - (int64_t)lx;
    const int64_t lpy = a_small ? lpb : lpa, rpy = a_small ? rpb : rpa;
    const uint32_t c = walk_chunk(dx, T.parts), first = (uint32_t)(w0 >> 32) * c;
    const uint32_t i_end = min(dx, first + c);
    for (uint32_t i0 = first; i0 < i_end; i0 += 64) {  // (uniform across the wave)
      const uint32_t i = i0 + (uint32_t)lane;
      int32_t e1 = -1, e2 = -1;
      if (i < i_end) {
        const bool in_l = i < lx;  // (entry i of N(x): L_x, then U_x)
        const int32_t w = in_l ? A.lnbr[lpx + i] : A.col[rpx + i];
        if (w < y) {
          const int32_t j = find_sorted(A.lnbr + lpy, ly, w);
          if (j >= 0) e2 = A.leid[lpy + j];
        } else if (w > y) {
          const int32_t j = find_sorted(A.col + rpy, uy, w);
          if (j >= 0) e2 = (int32_t)(rpy + j);
        }
        if (e2 >= 0) e1 = in_l ? A.leid[lpx + i] : (int32_t)(rpx + i);
      }
      bool t1 = false, t2 = false;
      if (e1 >= 0) {
        const int32_t s1 = T.state[e1], s2 = T.state[e2];
        const bool whole = s1 >= round && s2 >= round;  // no edge went in an earlier round
        int32_t owner = e;
        if (s1 == round && e1 < owner) owner = e1;
        if (s2 == round && e2 < owner) owner = e2;
        if (whole && owner == e) {
          if (s1 > round) t1 = atomicSub(&T.sup[e1], 1) == lim;
          if (s2 > round) t2 = atomicSub(&T.sup[e2], 1) == lim;
        }
      }
      truss_push(T, Q, t1, e1);
      truss_push(T, Q, t2, e2);
    }
  }
  truss_flush_all(T, Q);
}

int32_t truss(const Graph& g, int32_t* d_tau, hipStream_t st) {
  require_plain(g, "tc_truss");
  TempStream temps(st);
  const int64_t m = g.m;
  if (m == 0) return 0;
  TC_REQUIRE(m < ((int64_t)1 << 31), TC_EOVERFLOW, "tc_truss: 2^31 or more edges");
  DevBuf sup(sizeof(int32_t) * (size_t)m), state(sizeof(int32_t) * (size_t)m);
  launch_count(graph_view(g), MODE_SUPPORT_FULL, nullptr, sup.as<int32_t>(), nullptr, st);
  Lower L;
  build_lower(L, g, st);
  TC_LAUNCH("truss_fill", k_fill_i32, dim3(grid_threads(m)), dim3(kAT), 0, st, state.as<int32_t>(), m, kAlive);
  TrussArrays T{L.erow.as<uint32_t>(), g.col, g.deg, state.as<int32_t>(), sup.as<int32_t>(), d_tau, nullptr, kWalkParts, 0};
  const unsigned sweep = (unsigned)std::min<int64_t>(2048, grid_threads(m));  // (whole-array kernels)
  DevBuf total(sizeof(TrussStart));
  zero_i32(total.as<int32_t>(), sizeof(TrussStart) / 4, st, true);
  TC_LAUNCH("truss_start", k_truss_start, dim3(std::min(sweep, 512u)), dim3(kAT), 0, st, T, m, total.as<TrussStart>());
  TrussStart first;
  TC_HIP(hipMemcpyAsync(&first, total.p, sizeof(first), hipMemcpyDeviceToHost, st));
  check_sorts(st);  // (synchronises st)
  if (kAlive - first.room == first.top) {
    // all supports are the same (no triangles, or a clique): one level removes
    // every edge at once
    TC_LAUNCH("truss_fill", k_fill_i32, dim3(grid_threads(m)), dim3(kAT), 0, st, d_tau, m, first.top + 2);
    TC_HIP(hipGetLastError());
    TC_HIP(hipStreamSynchronize(st));
    note_use(g, st);
    return first.top + 2;
  }
  // the most entries per edge whose list is indexed by 31 bits and fits the
  // memory left (one per edge: m < 2^31 of them)
  DevBuf list;
  for (int i = 0; T.list == nullptr; ++i) {
    const bool last = i + 1 == kWalkChoices;
    if (!last && (first.entries[i] >> 31 || (kWalkParts >> i) > truss_walks())) continue;
    try {
      list.alloc(sizeof(uint64_t) * (size_t)first.entries[i]);
    } catch (const Error& e) {
      if (last || e.status != TC_ENOMEM) throw;
      continue;
    }
    T.list = list.as<uint64_t>();
    T.parts = kWalkParts >> i;
    T.entries = (uint32_t)first.entries[i];
  }
  const FullAdj A{g.row_ptr, g.col, L.ptr.as<int64_t>(), L.nbr.as<int32_t>(), L.eid.as<int32_t>()};

  // Batches of kRounds rounds, kBatches to a host read-back. Everything a
  // round decides (its frontier, the level) stays on the device; a round
  // with nothing to do costs its launch.
  constexpr int kRounds = 8, kBatches = 4;
  struct Ctl {  // of one read-back (cleared before it)
    int room[kBatches], fresh[kBatches];
    int lim[kBatches];
    uint32_t cnt[kBatches * kRounds], start[kBatches * kRounds];
  };
  // (the last bound, frontier and its place are read where the read-back before
  // left them)
  DevBuf ctl(3 * sizeof(Ctl));
  Ctl* const ring = ctl.as<Ctl>();
  zero_i32(ctl.as<int32_t>(), 3 * sizeof(Ctl) / 4, st, true);
  int* lim = &ring[2].lim[0];
  uint32_t *cnt = &ring[2].cnt[0], *start = &ring[2].start[0];
  int32_t round = 0;
  Ctl h;
  for (int trip = 0;; ++trip) {
    TC_REQUIRE(round < kAlive - 2 * kBatches * kRounds, TC_EOVERFLOW, "tc_truss: too many rounds");
    Ctl* d = &ring[trip % 2];
    if (trip >= 2) zero_i32(reinterpret_cast<int32_t*>(d), sizeof(Ctl) / 4, st, true);
    int i = 0;  // round of this read-back
    for (int b = 0; b < kBatches; ++b) {
      TC_LAUNCH("truss_min", k_truss_min, dim3(sweep), dim3(kAT), 0, st, T, m, start, cnt, &d->room[b], &d->fresh[b]);
      TC_LAUNCH("truss_level", k_truss_level, dim3((sweep + 1) / 2), dim3(kPeelThreads), 0, st, T, m, &d->fresh[b],
                &d->room[b], lim, &d->lim[b], round, start, cnt);
      lim = &d->lim[b];
      for (int r = 0; r < kRounds; ++r, ++round, ++i) {
        TC_LAUNCH("truss_peel", k_truss_peel, dim3(kPeelGrid), dim3(kPeelThreads), 0, st, T, A, round, lim, start,
                  &d->start[i], cnt, &d->cnt[i]);
        start = &d->start[i];
        cnt = &d->cnt[i];
      }
    }
    TC_HIP(hipGetLastError());
    TC_HIP(hipMemcpyAsync(&h, d, sizeof(Ctl), hipMemcpyDeviceToHost, st));
    TC_HIP(hipStreamSynchronize(st));
    if (h.start[i - 1] + h.cnt[i - 1] == T.entries) {  // every edge is removed
      note_use(g, st);
      return h.lim[kBatches - 1] + 1;  // the last level's trussness
    }
  }
}

template <class F>
tc_status guarded(const char* where, F&& f) {
  try {
    f();
    set_last_error("");
    return TC_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.status;
  } catch (const std::bad_alloc&) {
    set_last_error(std::string(where) + ": host allocation failed");
    return TC_ENOMEM;
  } catch (const std::exception& e) {
    set_last_error(e.what());
    return TC_EDEVICE;
  }
}

}  // namespace

}  // namespace tc

extern "C" {

tc_status tc_vertex_triangles(const tc_graph* gh, int64_t* d_tri, void* stream) {
  return tc::guarded("tc_vertex_triangles", [&] {
    TC_REQUIRE(gh != nullptr && d_tri != nullptr, TC_EINVAL, "tc_vertex_triangles: null argument");
    tc::vertex_counts(*tc::G(gh), d_tri, nullptr, nullptr, static_cast<hipStream_t>(stream));
  });
}

tc_status tc_clustering(const tc_graph* gh, double* d_cc, int64_t* d_tri, int64_t* d_sums, void* stream) {
  return tc::guarded("tc_clustering", [&] {
    TC_REQUIRE(gh != nullptr, TC_EINVAL, "tc_clustering: null graph");
    TC_REQUIRE(d_cc || d_tri || d_sums, TC_EINVAL, "tc_clustering: no output array");
    tc::vertex_counts(*tc::G(gh), d_tri, d_cc, d_sums, static_cast<hipStream_t>(stream));
  });
}

tc_status tc_transitivity(const tc_graph* gh, double* out, void* stream) {
  return tc::guarded("tc_transitivity", [&] {
    TC_REQUIRE(gh != nullptr && out != nullptr, TC_EINVAL, "tc_transitivity: null argument");
    hipStream_t st = static_cast<hipStream_t>(stream);
    tc::require_no_capture(st);
    tc::TempStream temps(st);
    tc::DevBuf sums(2 * sizeof(int64_t));
    tc::vertex_counts(*tc::G(gh), nullptr, nullptr, sums.as<int64_t>(), st);
    int64_t h[2] = {0, 0};
    TC_HIP(hipMemcpyAsync(h, sums.p, sizeof(h), hipMemcpyDeviceToHost, st));
    TC_HIP(hipStreamSynchronize(st));
    *out = h[1] ? (double)h[0] / (double)h[1] : 0.0;
  });
}

tc_status tc_truss(const tc_graph* gh, int32_t* d_tau, int32_t* kmax, void* stream) {
  return tc::guarded("tc_truss", [&] {
    TC_REQUIRE(gh != nullptr, TC_EINVAL, "tc_truss: null graph");
    const tc::Graph& g = *tc::G(gh);
    TC_REQUIRE(d_tau != nullptr || g.m == 0, TC_EINVAL, "tc_truss: null trussness array");
    const int32_t k = tc::truss(g, d_tau, static_cast<hipStream_t>(stream));
    if (kmax) *kmax = k;
  });
}

}  // extern "C"
