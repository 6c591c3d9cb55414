// tc_preprocess.hip - device preprocessing (Section 5.3 of the paper, on one GPU).
//
// Pipeline, all on the caller's stream:
//   1. keys: each pair {u, v}, u != v, becomes a 2s-bit key of min(u,v) and
//      max(u,v) (s = ceil(log2 n)); self loops are marked (small graphs: a
//      sentinel).
//   2. stable LSD radix sort of the keys by as many of their top bits as leave
//      groups that fit a hash set in LDS, which finds the duplicates (small
//      graphs: by all bits, and by comparing neighbours): the distinct keys
//      are the simple undirected graph of Section 2 / Section 6.1; they are
//      selected from the sorted keys by each later reader, never copied out.
//   3. degrees counted in LDS per vertex range: lower endpoints from the
//      sorted keys, upper endpoints from a radix partition of them by their
//      top bits; rank = position in the order (degree, id)
//      (a stable radix sort of degree * 2^s + id on the degree bits): the
//      non-decreasing degree relabelling of Section 5.3.
//   4. orientation by rank (Section 5.3: the global position stands in for the
//      degree), radix sort of rank keys -> U in CSR with sorted rows
//      (Section 5.2 requires sorted rows).
//   5. tasks (Section 3.1, <j,i,k>): every nonzero (a, b) of U whose row a has
//      entries after b and whose row b is non-empty probes U_a's entries after b
//      against a hash of U_b. Tasks are grouped by b (the transpose L = U^T of
//      Section 3.1), stably, so within one b the rows a ascend.
//   6. work classes and items for the count kernels (see tc_count.hip): rows b
//      are split by table size and work; the tasks are reordered class-major
//      (and their probe counts prefix-summed) so that each class, and each pack
//      of consecutive light rows, owns one contiguous task range; light rows
//      are packed, heavy rows are cut into per-wave probe ranges.
#include <algorithm>
#include <map>
#include <memory>
#include <mutex>

#include "tc_prims.h"

namespace tc {

namespace {

constexpr int kT = 256;
inline unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, div_up(n, kT)); }

// Elementwise gathers take 2 * kEw elements per thread, issued together
// (more bytes in flight per wave).
constexpr int kEw = 4;
// Grid of a key producer that also counts digits (grid-stride loop; one LDS
// histogram flush per work-group).
constexpr unsigned kProducerBlocks = 2048;

// The dedup sort's source: raw pair i as its canonical key (lo << s | hi),
// or the sentinel for a self loop or an id outside [0, n) (the digit
// counting kernel reports the latter).
struct CanonSrc {
  const int32_t* src;
  const int32_t* dst;
  int64_t n;
  int s;
  uint64_t sent;
  __device__ uint64_t key(int64_t i, bool& bad) const {
    const int64_t u = src[i], v = dst[i];
    bad = (u < 0) | (u >= n) | (v < 0) | (v >= n);
    const uint64_t lo = (uint64_t)(u < v ? u : v), hi = (uint64_t)(u < v ? v : u);
    return (bad | (u == v)) ? sent : ((lo << s) | hi);
  }
  __device__ bool operator()(int64_t i, uint64_t& k, char&) const {
    bool bad;
    k = key(i, bad);
    return true;
  }
};

// Keys take at most 62 bits (s <= 31); bit 63 marks one that is no distinct
// edge (a duplicate, a self loop).
constexpr uint64_t kDupMark = 1ull << 63;

// The edge {lo, hi} as a 2s-bit key for a sort that only has to bring equal
// edges close together: the upper s - low bits of lo, then s bits that mix hi
// with the low bits of lo (x = hi c1 + lo_low c2 mod 2^s, c1 odd: hi is
// recovered from x and lo_low), then the low bits of lo. Sorted by its top
// bits alone, such a key is grouped by an interval of lo (the degree count
// finds its lower endpoints by it) and, within it, by a hash that spreads
// any vertex's edges evenly.
struct MixCode {
  static constexpr uint32_t c1 = 0x9E3779B1u, c2 = 0x6A09E667u;  // 2^32 / golden ratio (odd); fraction of sqrt 2
  static constexpr uint32_t inverse(uint32_t c) {  // mod 2^32 (Newton: bits double)
    uint32_t x = c;
    for (int i = 0; i < 5; ++i) x *= 2u - c * x;
    return x;
  }
  int s, low;
  __device__ uint64_t key(uint32_t lo, uint32_t hi) const {
    const uint32_t l = lo & ((1u << low) - 1u), mask = (1u << s) - 1u;
    return ((uint64_t)(lo >> low) << (s + low)) | ((uint64_t)((hi * c1 + l * c2) & mask) << low) | l;
  }
  __device__ uint32_t lo(uint64_t k) const {  // (of a marked key too)
    return ((uint32_t)((k & ~kDupMark) >> (s + low)) << low) | ((uint32_t)k & ((1u << low) - 1u));
  }
  __device__ uint32_t hi(uint64_t k) const {
    constexpr uint32_t c1inv = inverse(c1);
    static_assert(c1 * c1inv == 1u, "inverse of c1");
    const uint32_t l = (uint32_t)k & ((1u << low) - 1u);
    return (((uint32_t)(k >> low) - l * c2) * c1inv) & ((1u << s) - 1u);
  }
};

// The dedup sort's source beyond small graphs: raw pair i as its mixed key,
// marked if it is a self loop (which spread over the groups like any edge)
// or holds an id outside [0, n) (reported by the digit counts).
struct MixSrc {
  const int32_t* src;
  const int32_t* dst;
  int64_t n;
  MixCode mc;
  __device__ uint64_t key(int64_t i, bool& bad) const {
    const int64_t u = src[i], v = dst[i];
    bad = (u < 0) | (u >= n) | (v < 0) | (v >= n);
    const uint64_t k = mc.key((uint32_t)(u < v ? u : v), (uint32_t)(u < v ? v : u));
    return bad ? kDupMark : u == v ? k | kDupMark : k;
  }
  __device__ bool operator()(int64_t i, uint64_t& k, char&) const {
    bool bad;
    k = key(i, bad);
    return true;
  }
};

// Digit counts of the keys for every pass of the dedup sort (bits [bit_lo,
// bit_hi)), and the id check, in one read of the raw pairs (grid-stride,
// kDigitBatch pairs in flight per thread; one LDS histogram flush per
// work-group).
template <class Src>
__global__ __launch_bounds__(256) void k_canon_digits(Src cs, int64_t m, int bit_lo, int bit_hi,
                                                      uint32_t* __restrict__ ghist, int* __restrict__ err) {
  extern __shared__ uint32_t h_dyn[];
  DigitCounter dc;
  dc.init(h_dyn, bit_lo, bit_hi);
  bool bad_any = false;
  const int64_t stride = (int64_t)gridDim.x * 256 * kDigitBatch;
  for (int64_t base = (int64_t)blockIdx.x * 256 * kDigitBatch + threadIdx.x; base < m; base += stride) {
    uint64_t k[kDigitBatch];
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      const int64_t i = base + (int64_t)j * 256;
      bool bad;
      k[j] = cs.key(i < m ? i : m - 1, bad);  // (no branch around the loads)
      bad_any |= bad;
    }
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      if (base + (int64_t)j * 256 >= m) break;
      dc.add(k[j]);
    }
  }
  if (bad_any) atomicOr(err, 1);
  dc.flush(ghist);
}

// Distinct edges of S, the mixed keys sorted by their top bits or by all of
// them: the unmarked ones. They are never copied out: k_distinct_groups (or
// k_distinct_mark) marks duplicates with kDupMark, and later readers (the
// degree count, its partition and the orientation) select a key by its own
// word alone and mask the mark off where they use an unselected key's bits.
struct DistinctSel {
  const uint64_t* S;
  __device__ bool operator()(int64_t i, uint64_t& k) const {
    k = S[i];
    return (k & kDupMark) == 0;
  }
};

// The degree partition's source: the upper endpoint of each distinct key.
struct DistinctHiSrc {
  DistinctSel d;
  MixCode mc;
  __device__ bool operator()(int64_t i, uint32_t& hi, char&) const {
    uint64_t k;
    const bool ok = d(i, k);
    hi = mc.hi(k);
    return ok;
  }
};

// Duplicates of a fully sorted S marked (a key that equals its predecessor),
// distinct keys counted, with the digit counts of their upper endpoints for
// the degree partition's passes (bits [bit_lo, s)), in one read of S. A
// neighbour may have marked S[i - 1] already: keys are compared with the
// mark masked off.
__global__ __launch_bounds__(256) void k_distinct_mark(uint64_t* __restrict__ S, MixCode mc, int64_t m_raw,
                                                       int bit_lo, uint32_t* __restrict__ ghist,
                                                       unsigned long long* __restrict__ total) {
  extern __shared__ uint32_t h_dyn[];
  __shared__ uint32_t s_c;
  if (threadIdx.x == 0) s_c = 0;
  DigitCounter dc;
  dc.init(h_dyn, bit_lo, mc.s);  // (ends with a barrier)
  uint32_t c = 0;
  const int64_t stride = (int64_t)gridDim.x * 256 * kDigitBatch;
  for (int64_t base = (int64_t)blockIdx.x * 256 * kDigitBatch + threadIdx.x; base < m_raw; base += stride) {
    uint64_t k[kDigitBatch], prev[kDigitBatch];
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      const int64_t i = base + (int64_t)j * 256;
      const int64_t ic = i < m_raw ? i : m_raw - 1;
      k[j] = S[ic];
      prev[j] = S[ic > 0 ? ic - 1 : 0];
    }
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      const int64_t i = base + (int64_t)j * 256;
      if (i < m_raw && !(k[j] & kDupMark)) {
        if (i == 0 || (prev[j] & ~kDupMark) != k[j]) {
          dc.add(mc.hi(k[j]));
          ++c;
        } else {
          S[i] = k[j] | kDupMark;
        }
      }
    }
  }
  if (c) atomicAdd(&s_c, c);
  dc.flush(ghist);  // (starts with a barrier: s_c is complete)
  if (threadIdx.x == 0 && s_c) atomicAdd(total, (unsigned long long)s_c);
}

// The same for an S that is sorted by the bits from gshift up only: keys that
// agree there (a group) are adjacent, in any order. A tile's work-group takes
// the groups that begin in its kGrpTile keys (the first may have begun
// before: skipped; the last may run on past the tile: read on) and enters
// their keys into a hash set in LDS, whose words are 11 bits of the key's
// hash and its position in the tile + 1: the first to claim a word is the
// distinct key, and one whose word already holds an equal key is marked.
// What a group may hold: the sort's bits are chosen so that even edges that
// all share one interval of lo average at most kGrpMean keys a group, so a
// tile and a group fit the set; a group of more than `most` keys (one edge
// that often; seen before any of it is read), or a set that is so full that a
// key finds no word in kGrpProbes, sets *fail: what is left of the launch is
// skipped, and the host sorts by all bits instead.
// A group that runs far past its tile is one edge many times over, and one
// work-group reads it: kGrpFar keys a thread at a time, and a key equal to one
// that its wave has entered is marked without a look at the set (2^20 copies of
// an edge: 1.87 ms with a key a thread and every one looked up, 0.6 ms so).
// Two or three passes of the sort, of 1.28 ms each at scale 24 (256 M pairs),
// become LDS work of the read that the mark needs anyway.
constexpr int kGrpThreads = 1024;
constexpr int kGrpKeys = 4;  // per thread
constexpr int kGrpTile = kGrpThreads * kGrpKeys;
constexpr int kGrpSlots = 16384;  // 64 KiB: two work-groups a CU
constexpr int kGrpMeanLog2 = 13;
// Keys of a group at most: its work-group reads 2^20 of them in 0.6 ms, and a
// sort by all bits costs as much at 16M pairs, 0.15 ms at 2M (positions take
// 21 bits).
inline int64_t group_max(int64_t m_raw) {
  return std::min<int64_t>((int64_t)1 << 20, std::max<int64_t>((int64_t)1 << 17, m_raw / 16));
}
constexpr int kGrpAhead = 64;  // keys past the tile read with it
constexpr int kGrpFar = 4;     // keys per thread and step beyond those
constexpr int kGrpProbes = 1024;

__global__ __launch_bounds__(kGrpThreads, 8) void k_distinct_groups(uint64_t* S, MixCode mc, int64_t m_raw, int gshift,
                                                                    int64_t most, int bit_lo, uint32_t* __restrict__ ghist,
                                                                    unsigned long long* __restrict__ total,
                                                                    int* __restrict__ fail) {
  extern __shared__ uint32_t h_dyn[];
  __shared__ int4 s_tab4[kGrpSlots / 4];
  __shared__ uint32_t s_c;
  __shared__ int s_stop;
  uint32_t* const tab = reinterpret_cast<uint32_t*>(s_tab4);
  const int tid = threadIdx.x;
  if (tid == 0) s_c = 0;
  DigitCounter dc;
  dc.init(h_dyn, bit_lo, mc.s);
  uint32_t c = 0;
  auto group = [&](uint64_t k) -> uint64_t { return (k & ~kDupMark) >> gshift; };
  auto at = [&](int64_t i) -> uint64_t { return S[i < m_raw ? i : m_raw - 1]; };
  const int64_t ntiles = (m_raw + kGrpTile - 1) / kGrpTile;
  int64_t t = blockIdx.x;
  uint64_t nk[kGrpKeys], n_ahead, n_before, n_last, n_far;  // the next tile's loads
  auto load = [&](int64_t tt) {
    const int64_t i0 = tt * kGrpTile;
#pragma unroll
    for (int j = 0; j < kGrpKeys; ++j) nk[j] = at(i0 + j * kGrpThreads + tid);
    n_ahead = at(i0 + kGrpTile + (tid & (kGrpAhead - 1)));
    n_before = S[i0 > 0 ? i0 - 1 : 0];
    n_last = at(i0 + kGrpTile - 1);
    n_far = at(i0 + kGrpTile + kGrpAhead - 1);
  };
  if (t < ntiles) load(t);
  for (; t < ntiles; t += gridDim.x) {
    const int64_t i0 = t * kGrpTile;
    uint64_t k[kGrpKeys];
#pragma unroll
    for (int j = 0; j < kGrpKeys; ++j) k[j] = nk[j];
    const uint64_t ahead = n_ahead, last = group(n_last), far = group(n_far);
    // (no group is all ones: it would need lo = 2^s - 1)
    const uint64_t before = t == 0 ? ~0ull : group(n_before);
    if (t + gridDim.x < ntiles) load(t + gridDim.x);
#pragma unroll
    for (int j = 0; j < kGrpSlots / 4 / kGrpThreads; ++j) s_tab4[j * kGrpThreads + tid] = make_int4(0, 0, 0, 0);
    if (tid == 0) s_stop = __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_stop) break;  // (uniform: it is written again after the barrier below)
    auto enter = [&](uint64_t key, int64_t i) {
      uint32_t h = (uint32_t)key * 0x9E3779B1u ^ (uint32_t)(key >> 32) * 0x6A09E667u;
      h = (h ^ (h >> 15)) * 0x510E527Fu;
      h ^= h >> 16;
      uint32_t slot = h >> 18;
      const uint32_t word = (h << 21) | (uint32_t)(i - i0 + 1);
      for (int probes = 0; probes < kGrpProbes; ++probes, slot = (slot + 1) & (kGrpSlots - 1)) {
        const uint32_t old = atomicCAS(&tab[slot], 0u, word);
        if (old == 0) {
          dc.add(mc.hi(key));
          ++c;
          return;
        }
        // (the owner of a word is never marked)
        if (((old ^ word) >> 21) == 0 && S[i0 + (old & 0x1FFFFFu) - 1] == key) {
          S[i] = key | kDupMark;
          return;
        }
      }
      atomicOr(fail, 1);
    };
#pragma unroll
    for (int j = 0; j < kGrpKeys; ++j) {
      const int64_t i = i0 + j * kGrpThreads + tid;
      if (i < m_raw && !(k[j] & kDupMark) && group(k[j]) != before) enter(k[j], i);
    }
    if (last != before) {  // the tile's last group, past the tile
      int64_t i = i0 + kGrpTile + tid;
      if (tid < kGrpAhead && i < m_raw && !(ahead & kDupMark) && group(ahead) == last) enter(ahead, i);
      const int64_t far0 = i0 + kGrpTile + kGrpAhead;
      if (far == last && far0 < m_raw) {  // (uniform)
        if (i0 + most < m_raw && group(at(i0 + most)) == last) {
          if (tid == 0) atomicOr(fail, 1);
        } else {
          bool on = true;
          uint64_t known = 0;  // an edge that this wave has entered (0: none; it is no unmarked key)
          for (int64_t base = far0; on && base < m_raw; base += (int64_t)kGrpThreads * kGrpFar) {
            // (no barrier in this loop: a wave may leave it when it sees the flag)
            if (__hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
            uint64_t key[kGrpFar];
#pragma unroll
            for (int j = 0; j < kGrpFar; ++j) key[j] = at(base + j * kGrpThreads + tid);
            on = group(at(base + (int64_t)kGrpThreads * kGrpFar - 1)) == last;
            uint32_t rest = 0;  // items to enter
#pragma unroll
            for (int j = 0; j < kGrpFar; ++j) {
              i = base + j * kGrpThreads + tid;
              const bool mine = i < m_raw && !(key[j] & kDupMark) && group(key[j]) == last;
              if (mine && key[j] == known) S[i] = key[j] | kDupMark;
              else rest |= mine ? 1u << j : 0u;
            }
            if (__ballot(rest != 0)) {
              for (; rest; rest &= rest - 1) {
                i = base + (__ffs((int)rest) - 1) * kGrpThreads + tid;
                known = S[i];  // (not marked: its own thread marks it)
                enter(known, i);
              }
              known = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(known >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)known);
            }
          }
          // (again: nothing of the next tile is held in registers through the loop)
          if (t + gridDim.x < ntiles) load(t + gridDim.x);
        }
      }
    }
    __syncthreads();
  }
  if (c) atomicAdd(&s_c, c);
  dc.flush(ghist);  // (starts with a barrier: s_c is complete)
  if (tid == 0 && s_c) atomicAdd(total, (unsigned long long)s_c);
}

// Entry i of U (row a, column b) starts a task iff U_a has entries after i
// and U_b is not empty (one bit per row); the task's key is b and its value
// the probe range [i + 1, row end of a).
struct TaskPred {
  const uint64_t* okey;
  int s;
  const int64_t* row_ptr;
  const uint64_t* nonempty;
  uint32_t* tkey;
  uint64_t* tval;
  struct Item {
    uint32_t b, end;
  };
  __device__ bool operator()(int64_t i, Item& it) const {
    const uint64_t k = okey[i];
    const int64_t a = (int64_t)(k >> s);
    it.b = (uint32_t)(k & ((1ull << s) - 1));
    it.end = (uint32_t)row_ptr[a + 1];
    // (no short circuit: the loads of several entries can then be in flight)
    return ((int64_t)it.end - i - 1 > 0) & (bool)((nonempty[it.b >> 6] >> (it.b & 63)) & 1ull);
  }
  __device__ void emit(int64_t i, const Item& it, uint32_t pos) const {
    tkey[pos] = it.b;
    tval[pos] = (uint64_t)(i + 1) | ((uint64_t)it.end << 32);
  }
};

// The task sort's source: entry i of U gives the task (key b, value first
// probe | end << 32) when TaskPred selects it.
struct TaskSrc {
  TaskPred p;
  __device__ bool operator()(int64_t i, uint32_t& b, uint64_t& v) const {
    TaskPred::Item it;
    const bool ok = p(i, it);
    b = it.b;
    v = (uint64_t)(i + 1) | ((uint64_t)it.end << 32);
    return ok;
  }
};

// Tasks of U counted, with the digit counts of their keys for every pass of
// the task sort, in one read of U (grid-stride, kDigitBatch entries in
// flight per thread; one LDS histogram flush and one count per work-group).
__global__ __launch_bounds__(256) void k_task_digits(TaskSrc src, int64_t m, int key_bits,
                                                     uint32_t* __restrict__ ghist, uint32_t* __restrict__ total) {
  extern __shared__ uint32_t h_dyn[];
  __shared__ uint32_t s_c;
  if (threadIdx.x == 0) s_c = 0;
  DigitCounter dc;
  dc.init(h_dyn, 0, key_bits);  // (ends with a barrier)
  uint32_t c = 0;
  const int64_t stride = (int64_t)gridDim.x * 256 * kDigitBatch;
  for (int64_t base = (int64_t)blockIdx.x * 256 * kDigitBatch + threadIdx.x; base < m; base += stride) {
    uint32_t b[kDigitBatch];
    bool ok[kDigitBatch];
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      const int64_t i = base + (int64_t)j * 256;
      uint64_t v;
      ok[j] = src(i < m ? i : m - 1, b[j], v) & (i < m);  // (no branch around the loads)
    }
#pragma unroll
    for (int j = 0; j < kDigitBatch; ++j) {
      if (ok[j]) {
        dc.add(b[j]);
        ++c;
      }
    }
  }
  if (c) atomicAdd(&s_c, c);
  dc.flush(ghist);  // (starts with a barrier: s_c is complete)
  if (threadIdx.x == 0 && s_c) atomicAdd(total, s_c);
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_i64(int64_t* p, int64_t n, int64_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// deg(v) = (edges whose lower endpoint is v) + (edges whose upper endpoint is
// v). The upper endpoints arrive partitioned by their top bits (bucket = v >>
// hshift; bucket j at [start(j), start(j + 1)), start(j) = bs32[j] or bs64[j]
// for j < nbs, m beyond). Each work-group counts one range [v0, v1) of at
// most kDegBins vertices of one bucket in LDS: the upper endpoints from that
// bucket's entries, the lower endpoints from the distinct keys of S whose lo
// lies in [v0, v1) (S is sorted by lo >> mc.low, and v0 is a multiple of
// 2^mc.low; the range is found by binary search), with kDegBatch loads in
// flight per thread before they are counted. It writes the rank keys
// deg(v) << s | v of its vertices.
constexpr int kDegBinsLog2 = 15;
constexpr int kDegBins = 1 << kDegBinsLog2;   // LDS counters of one work-group (128 KiB)
constexpr int kDegThreads = 1024;
constexpr int kDegBatch = 8;

// First position of the sorted S[0, n) whose key (duplicate mark masked
// off) is >= x.
__device__ int64_t lower_bound_u64(const uint64_t* __restrict__ S, int64_t n, uint64_t x) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((S[mid] & ~kDupMark) < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(kDegThreads) void k_degree_hist(const uint32_t* __restrict__ hi,
                                                             const uint32_t* __restrict__ bs32,
                                                             const int64_t* __restrict__ bs64, int64_t nbs, int64_t m,
                                                             int hshift, int sub, DistinctSel d, int64_t m_raw,
                                                             int64_t n, MixCode mc, uint64_t* __restrict__ rk) {
  extern __shared__ uint32_t h_deg[];
  __shared__ int64_t s_r[2];
  const uint32_t bucket = blockIdx.x / (uint32_t)sub, part = blockIdx.x % (uint32_t)sub;
  const int64_t v0 = ((int64_t)bucket << hshift) + (int64_t)part * kDegBins;
  const int64_t span_end = (int64_t)(bucket + 1) << hshift;
  const int64_t v1 = std::min(std::min(v0 + kDegBins, span_end), n);
  if (v0 >= v1) return;  // (uniform per work-group)
  const int nv = (int)(v1 - v0);
  for (int j = threadIdx.x; j < nv; j += blockDim.x) h_deg[j] = 0;
  if (threadIdx.x < 2) {
    // (v1 = n: up to the end of its interval, where no lo lies past it)
    const uint64_t v = (uint64_t)(threadIdx.x ? v1 : v0) + ((1ull << mc.low) - 1);
    s_r[threadIdx.x] = lower_bound_u64(d.S, m_raw, (v >> mc.low) << (mc.s + mc.low));
  }
  __syncthreads();
  // upper endpoints
  auto start = [&](int64_t j) -> int64_t { return j >= nbs ? m : bs64 ? bs64[j] : (int64_t)bs32[j]; };
  const int64_t e0 = start(bucket), e1 = start((int64_t)bucket + 1);
  for (int64_t base = e0 + threadIdx.x; base < e1; base += (int64_t)blockDim.x * kDegBatch) {
    uint32_t v[kDegBatch];
#pragma unroll
    for (int b = 0; b < kDegBatch; ++b) {
      const int64_t i = base + (int64_t)b * blockDim.x;
      v[b] = i < e1 ? hi[i] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int b = 0; b < kDegBatch; ++b) {
      const int64_t x = (int64_t)v[b];  // (the fill value is past every range)
      if (x >= v0 && x < v1) atomicAdd(&h_deg[x - v0], 1u);
    }
  }
  // lower endpoints: the distinct keys among S[r0, r1) all have lo in [v0, v1).
  // The keys of a wave that share the first one's lo are added with one
  // atomic (a vertex that most of a range's edges start at would otherwise
  // take one lane at a time).
  const int64_t r0 = s_r[0], r1 = s_r[1];
  const int lane = threadIdx.x & 63;
  // (wb, a wave's first position, is uniform across the wave: every lane
  // takes part in the ballots; lanes past r1 read S[r1 - 1] and select nothing)
  for (int64_t wb = r0 + (int64_t)(threadIdx.x - lane) * kDegBatch; wb < r1;
       wb += (int64_t)blockDim.x * kDegBatch) {
    uint64_t k[kDegBatch];
    bool ok[kDegBatch];
#pragma unroll
    for (int b = 0; b < kDegBatch; ++b) {
      const int64_t i = wb + (int64_t)b * 64 + lane;
      ok[b] = d(i < r1 ? i : r1 - 1, k[b]) & (i < r1);
    }
#pragma unroll
    for (int b = 0; b < kDegBatch; ++b) {
      const uint32_t lo = mc.lo(k[b]);
      const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
      const uint64_t same = __ballot(ok[b] && lo == lead);
      if (lane == 0) {
        if (same) atomicAdd(&h_deg[(int64_t)lo - v0], (uint32_t)__popcll(same));
      } else if (ok[b] && lo != lead) {
        atomicAdd(&h_deg[(int64_t)lo - v0], 1u);
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nv; j += blockDim.x) {
    const int64_t v = v0 + j;
    rk[v] = ((uint64_t)h_deg[j] << mc.s) | (uint64_t)v;
  }
}

__global__ void k_rank_keys(const uint32_t* __restrict__ deg, int64_t n, int s,
                            uint64_t* __restrict__ rk) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) rk[v] = ((uint64_t)deg[v] << s) | (uint64_t)v;
}

__global__ void k_perm(const uint64_t* __restrict__ rk, int64_t n, int s, int32_t* __restrict__ perm,
                       uint32_t* __restrict__ deg) {
  int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const uint64_t k = rk[r];
  perm[k & ((1ull << s) - 1)] = (int32_t)r;
  deg[r] = (uint32_t)(k >> s);
}

// Orientation in two steps, so that no rank is read at random from the
// whole rank map. (1) One radix pass partitions the distinct edges by the
// top 8 bits of their upper endpoint (the last digit pass of the degree
// count's partition, whose scanned digit starts it reuses); its source reads
// S in order, so the lower endpoints' ranks are read interval by interval of
// at most 32768 vertices (128 KiB of the map): element = rank(lo) << 32 | hi.
// (2) k_orient_hi reads the ranks of the upper endpoints bucket by bucket (a bucket spans 2^(s-8) vertices: a
// 256 KiB slice of the rank map at s = 24, 1 MiB at s = 26, which stays in
// L2) and writes the oriented key in place.
struct LoRankSrc {
  DistinctSel d;
  const int32_t* perm;
  MixCode mc;
  __device__ bool operator()(int64_t i, uint64_t& k, char&) const {
    uint64_t e;
    const bool ok = d(i, e);
    // (an unselected key's lower endpoint is a vertex too)
    k = ((uint64_t)(uint32_t)perm[mc.lo(e)] << 32) | mc.hi(e);
    return ok;
  }
};

// XCD-aware grid-stride sweep: work-groups are dealt to the 8 XCDs in turn,
// so work-group b sweeps the chunks of the b % 8-th eighth of [0, chunks)
// and each XCD's L2 holds the rank slices of its own eighth only. The grid
// is a multiple of 8.
__global__ __launch_bounds__(256) void k_orient_hi(uint64_t* __restrict__ pk, int64_t m, int s,
                                                   const int32_t* __restrict__ perm, uint32_t* __restrict__ hist) {
  extern __shared__ uint32_t h_dyn[];
  constexpr int kI = 2 * kEw;  // gathers: more in flight
  constexpr int64_t kChunk = (int64_t)kT * kI;
  DigitCounter dc;
  dc.init(h_dyn, 0, 2 * s);
  const uint64_t mask = (1ull << s) - 1;
  const int64_t chunks = (m + kChunk - 1) / kChunk;
  const int64_t per_xcd = (chunks + 7) / 8;
  const int64_t c0 = (int64_t)(blockIdx.x & 7) * per_xcd;
  const int64_t c1 = c0 + per_xcd < chunks ? c0 + per_xcd : chunks;
  for (int64_t c = c0 + (blockIdx.x >> 3); c < c1; c += gridDim.x >> 3) {
    const int64_t i0 = c * kChunk + threadIdx.x;
    uint64_t e[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int64_t i = i0 + (int64_t)j * kT;
      e[j] = pk[i < m ? i : m - 1];
    }
    uint32_t rv[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) rv[j] = (uint32_t)perm[e[j] & mask];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int64_t i = i0 + (int64_t)j * kT;
      if (i < m) {
        const uint64_t a = e[j] >> 32, b = rv[j];
        const uint64_t k = a < b ? ((a << s) | b) : ((b << s) | a);
        pk[i] = k;
        dc.add(k);
      }
    }
  }
  dc.flush(hist);
}

// Column of a sorted orient key and its short form, written by the orient
// sort's last pass (k_rows clears the first entry of every row).
struct ColEpi {
  int32_t* col;
  uint16_t* col16;
  int64_t n;
  int s;
  __device__ void operator()(uint64_t pos, uint64_t key) const {
    const int32_t k = (int32_t)(key & ((1ull << s) - 1));
    col[pos] = k;
    const int64_t v = n - k;
    col16[pos] = (uint16_t)(v <= kShortSpan ? v : 0);
  }
};

__global__ void k_col(const uint64_t* __restrict__ okey, int64_t m, int s, int32_t* __restrict__ col) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) col[i] = (int32_t)(okey[i] & ((1ull << s) - 1));
}

// Grids of the reducing kernels below: a few blocks per CU, each looping
// over its rows, so that the per-block global atomics stay few.
constexpr unsigned kReduceBlocks = 1024;
inline unsigned grid_reduce(int64_t n) { return (unsigned)std::min<int64_t>(kReduceBlocks, grid_for(n)); }

// From the sorted orient keys: U's row pointers (binary search), the bitmap of
// non-empty rows, W+ = sum_a C(d+(a), 2), max d+(a), and the zeros of the
// short columns: the first entry of every row and the padding. A work-group
// searches the starts of its 512 rows and, in a ninth wave, that of the row
// after them, and takes the degrees from LDS (three launches, of which
// two read the row pointers again: 84 us at scale 20, 70 us for 10^6 rows of
// 8; this one: 62 us and 55 us).
constexpr int kRowsPer = 512, kRowsThreads = kRowsPer + 64;
constexpr unsigned kRowsBlocks = 1024;  // (each ends on two atomics, 12 ns one after the other)
__global__ __launch_bounds__(kRowsThreads) void k_rows(const uint64_t* __restrict__ keys, int64_t m, int s, int64_t n,
                                                       int64_t* __restrict__ row_ptr, uint16_t* __restrict__ col16,
                                                       uint64_t* __restrict__ bits,
                                                       unsigned long long* __restrict__ wplus,
                                                       unsigned int* __restrict__ maxd) {
  __shared__ int64_t s_lo[kRowsPer + 1];
  __shared__ uint64_t s_w[kRowsPer / 64];
  __shared__ uint32_t s_m[kRowsPer / 64];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  uint64_t w = 0;
  uint32_t md = 0;
  for (int64_t r0 = (int64_t)blockIdx.x * kRowsPer; r0 <= n; r0 += (int64_t)gridDim.x * kRowsPer) {
    const int64_t r = r0 + tid;
    if (tid <= kRowsPer) {
      int64_t lo = 0, hi = m;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)(keys[mid] >> s) < r) lo = mid + 1;
        else hi = mid;
      }
      s_lo[tid] = lo;
      if (tid < kRowsPer && r <= n) {
        row_ptr[r] = lo;
        col16[lo] = 0;  // (an empty row: the first entry of a later one, or the padding)
        if (r == n) col16[m + 1] = 0;
      }
    }
    __syncthreads();
    if (tid < kRowsPer) {
      const uint64_t d = r < n ? (uint64_t)(s_lo[tid + 1] - s_lo[tid]) : 0;
      const uint64_t ne = __ballot(d > 0);
      if (lane == 0 && r < n) bits[r >> 6] = ne;
      w += d * (d - (d > 0)) / 2;
      md = max(md, (uint32_t)d);
    }
    __syncthreads();
  }
  if (tid < kRowsPer) {
    w = wave_sum(w);
    md = wave_max(md);
    if (lane == 0) {
      s_w[wave] = w;
      s_m[wave] = md;
    }
  }
  __syncthreads();
  if (tid == 0) {
    uint64_t tw = 0;
    uint32_t tm = 0;
    for (int i = 0; i < kRowsPer / 64; ++i) {
      tw += s_w[i];
      tm = max(tm, s_m[i]);
    }
    if (tw) atomicAdd(wplus, (unsigned long long)tw);
    if (tm) atomicMax(maxd, tm);
  }
}

// Class of every hashed row b (-1 = no work), each class's largest table and
// weight, and the weight of its short rows (reduced per wave before one atomic
// per wave and class).
// Work of a hashed row is weighed in probes, a short row's units as two each.
__device__ __forceinline__ uint64_t row_weight(uint64_t w, int64_t b, int64_t b16) { return b >= b16 ? 2 * w : w; }

__global__ __launch_bounds__(256) void k_classify(const int64_t* __restrict__ tptr,
                                                  const uint64_t* __restrict__ tprefix,
                                                  const int64_t* __restrict__ row_ptr, int64_t n, bool all_rows,
                                                  uint64_t heavy_min, uint64_t heavy_min16, int64_t b16,
                                                  int8_t* __restrict__ cls,
                                                  int* __restrict__ cls_log2S,
                                                  unsigned long long* __restrict__ cls_probes) {
  __shared__ int s_max[NUM_CLASSES];
  __shared__ unsigned long long s_w[2 * NUM_CLASSES];  // all rows, short rows
  if (threadIdx.x < NUM_CLASSES) s_max[threadIdx.x] = 0;
  if (threadIdx.x < 2 * NUM_CLASSES) s_w[threadIdx.x] = 0;
  __syncthreads();
  int lmax[NUM_CLASSES];
  unsigned long long lw[NUM_CLASSES], lw16[NUM_CLASSES];
#pragma unroll
  for (int k = 0; k < NUM_CLASSES; ++k) {
    lmax[k] = 0;
    lw[k] = 0;
    lw16[k] = 0;
  }
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n; b += (int64_t)gridDim.x * blockDim.x) {
    int c = -1, l = 0;
    const uint64_t W = row_weight(tprefix[tptr[b + 1]] - tprefix[tptr[b]], b, b16);
    if (W > 0) {
      l = table_log2(row_ptr[b + 1] - row_ptr[b]);
      if (l > kMaxLog2S) c = CLS_GLOBAL;
      else if (l > 13) c = CLS_WG_GIANT;
      else if (l > 12) c = CLS_WG_HUGE;
      else if (W < (b >= b16 ? heavy_min16 : heavy_min) && l <= 10) c = l <= 8 ? CLS_PACK_SMALL : CLS_PACK_LARGE;
      else c = l <= 10 ? CLS_WG_SMALL : CLS_WG_LARGE;
    } else if (all_rows) {
      // no doubly sparse traversal: a row without work is still visited (a
      // pack member whose table stays empty: it has no task to look up)
      c = CLS_PACK_SMALL;
      l = table_log2(0);
    }
    cls[b] = (int8_t)c;
#pragma unroll
    for (int k = 0; k < NUM_CLASSES; ++k) {
      lmax[k] = c == k && l > lmax[k] ? l : lmax[k];
      lw[k] += c == k ? W : 0;
      lw16[k] += c == k && b >= b16 ? W : 0;
    }
  }
#pragma unroll
  for (int k = 0; k < NUM_CLASSES; ++k) {
    const int mk = wave_max(lmax[k]);
    const unsigned long long wk = wave_sum(lw[k]);
    if (lane_id() == 0 && mk > 0) atomicMax(&s_max[k], mk);
    if (lane_id() == 0 && wk > 0) atomicAdd(&s_w[k], wk);
    const unsigned long long wk16 = wave_sum(lw16[k]);
    if (lane_id() == 0 && wk16 > 0) atomicAdd(&s_w[NUM_CLASSES + k], wk16);
  }
  __syncthreads();
  if (threadIdx.x < NUM_CLASSES && s_max[threadIdx.x] > 0) atomicMax(&cls_log2S[threadIdx.x], s_max[threadIdx.x]);
  if (threadIdx.x < 2 * NUM_CLASSES && s_w[threadIdx.x] > 0) atomicAdd(&cls_probes[threadIdx.x], s_w[threadIdx.x]);
}

// Per-class sums (rows, table keys, tasks; the probes come from
// k_task_permute): LDS accumulation per block, one partial row per block, then
// a column reduction.
constexpr int kStatCols = NUM_CLASSES * 4;

__global__ __launch_bounds__(256) void k_class_stats(const int8_t* __restrict__ cls, int64_t n,
                                                     const uint32_t* __restrict__ tbeg,
                                                     const uint32_t* __restrict__ tend,
                                                     const int64_t* __restrict__ row_ptr,
                                                     unsigned long long* __restrict__ partial) {
  __shared__ unsigned long long acc[kStatCols];
  if (threadIdx.x < kStatCols) acc[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n; b += (int64_t)gridDim.x * blockDim.x) {
    const int c = cls[b];
    if (c >= 0) {
      atomicAdd(&acc[c * 4 + 0], 1ull);
      atomicAdd(&acc[c * 4 + 1], (unsigned long long)(row_ptr[b + 1] - row_ptr[b]));
      atomicAdd(&acc[c * 4 + 2], (unsigned long long)(tend[b] - tbeg[b]));
    }
  }
  __syncthreads();
  if (threadIdx.x < kStatCols) partial[(int64_t)blockIdx.x * kStatCols + threadIdx.x] = acc[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_reduce_cols(const unsigned long long* __restrict__ partial,
                                                     int64_t rows, int cols,
                                                     unsigned long long* __restrict__ out) {
  __shared__ unsigned long long s_w[4];
  const int c = blockIdx.x;
  unsigned long long v = 0;
  for (int64_t r = threadIdx.x; r < rows; r += blockDim.x) v += partial[r * cols + c];
  v = wave_sum(v);
  if (lane_id() == 0) s_w[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) out[c] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// Wave items of a heavy row with W probes: a multiple of the class's waves
// per work-group (each group of `waves` consecutive items shares one table).
__device__ __forceinline__ uint32_t wg_parts(uint64_t W, int waves, uint32_t chunk) {
  // (chunk >= kWaveChunkMin: per > 0)
  const uint64_t per = (uint64_t)waves * chunk;
  return (uint32_t)(waves * ((W + per - 1) / per));
}

// Rows with work (class >= 0): key = class, value = row (compacted in row
// order, then stably sorted by class: the class-major row order).
struct WorkRowPred {
  const int8_t* cls;
  uint32_t* key;
  uint32_t* row;
  struct Item {
    int8_t c;
  };
  __device__ bool operator()(int64_t b, Item& it) const {
    it.c = cls[b];
    return it.c >= 0;
  }
  __device__ void emit(int64_t b, const Item& it, uint32_t pos) const {
    key[pos] = (uint32_t)it.c;
    row[pos] = (uint32_t)b;
  }
};

// Per class-major row i (row b = crow[i]): its number of tasks, its probes
// W_b, and its wave items (item classes only).
struct CmTasks {
  const uint32_t* crow;
  const int64_t* tptr;
  __device__ uint32_t operator()(int64_t i) const {
    const uint32_t b = crow[i];
    return (uint32_t)(tptr[b + 1] - tptr[b]);
  }
};
struct CmProbes {
  const uint32_t* crow;
  const int64_t* tptr;
  const uint64_t* tprefix;
  __device__ uint64_t operator()(int64_t i) const {
    const uint32_t b = crow[i];
    return tprefix[tptr[b + 1]] - tprefix[tptr[b]];
  }
};
struct CmItems {
  const uint32_t* crow;
  const int8_t* cls;
  const int64_t* tptr;
  const uint64_t* tprefix;
  int64_t b16;
  uint32_t chunk16;  // short rows
  uint32_t chunk[NUM_CLASSES];
  __device__ uint32_t operator()(int64_t i) const {
    const uint32_t b = crow[i];
    const int c = cls[b];
    if (c == CLS_PACK_SMALL || c == CLS_PACK_LARGE) return 0;
    const uint64_t W = tprefix[tptr[b + 1]] - tprefix[tptr[b]];
    return (int64_t)b >= b16 ? wg_parts(2 * W, kWaves, chunk16) : wg_parts(W, class_waves(c), chunk[c]);
  }
};

// Task range of every row with work in the class-major task order, and the
// row's class-major position.
__global__ void k_cm_place(const uint32_t* __restrict__ crow, int64_t R, const uint32_t* __restrict__ tsc,
                           uint32_t* __restrict__ tbeg, uint32_t* __restrict__ tend,
                           uint32_t* __restrict__ cm_pos) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= R) return;
  const uint32_t b = crow[i];
  tbeg[b] = tsc[i];
  tend[b] = tsc[i + 1];
  cm_pos[b] = (uint32_t)i;
}

// Task t (hashed-row order) to its class-major slot: first probe and the
// class-major exclusive prefix (the row's base plus the prefix within the
// row, which keeps its order); and the probes of every class, kPermuteTasks
// tasks per thread so that the global atomics stay few.
constexpr int kPermuteTasks = 16;
__global__ __launch_bounds__(256) void k_task_permute(int64_t T, const uint32_t* __restrict__ tb_row,
                                                      const int64_t* __restrict__ tb_ptr,
                                                      const uint64_t* __restrict__ tb_val,
                                                      const uint64_t* __restrict__ tb_prefix,
                                                      const int8_t* __restrict__ cls,
                                                      const uint32_t* __restrict__ tbeg,
                                                      const uint32_t* __restrict__ cm_pos,
                                                      const uint64_t* __restrict__ wsc,
                                                      uint32_t* __restrict__ tstart, uint64_t* __restrict__ tprefix,
                                                      unsigned long long* __restrict__ cls_probes) {
  __shared__ unsigned long long s_p[NUM_CLASSES];
  if (threadIdx.x < NUM_CLASSES) s_p[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (256 * kPermuteTasks) + threadIdx.x;
  int c_run = -1;  // probes of a run of this thread's tasks in one class
  unsigned long long p_run = 0;
  constexpr int kB = 4;  // tasks whose loads are in flight together (positions clamped, no branch)
  for (int j0 = 0; j0 < kPermuteTasks; j0 += kB) {
    uint32_t b[kB];
    uint64_t v[kB], pre[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      const int64_t t = base + (int64_t)(j0 + j) * 256, tc = t < T ? t : T - 1;
      b[j] = tb_row[tc];
      v[j] = tb_val[tc];
      pre[j] = tb_prefix[tc];
    }
    int64_t p0[kB];
    uint32_t tb[kB], cm[kB];
    int c[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      p0[j] = tb_ptr[b[j]];
      tb[j] = tbeg[b[j]];
      cm[j] = cm_pos[b[j]];
      c[j] = cls[b[j]];
    }
    uint64_t off[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) off[j] = wsc[cm[j]] - tb_prefix[p0[j]];
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      const int64_t t = base + (int64_t)(j0 + j) * 256;
      if (t >= T) continue;
      const int64_t nt = (int64_t)tb[j] + (t - p0[j]);
      const uint32_t first = (uint32_t)v[j];
      tstart[nt] = first;
      tprefix[nt] = off[j] + pre[j];
      if (c[j] != c_run) {
        if (p_run) atomicAdd(&s_p[c_run], p_run);
        c_run = c[j];
        p_run = 0;
      }
      p_run += (uint32_t)(v[j] >> 32) - first;
    }
  }
  if (p_run) atomicAdd(&s_p[c_run], p_run);
  __syncthreads();
  if (threadIdx.x < NUM_CLASSES && s_p[threadIdx.x]) atomicAdd(&cls_probes[threadIdx.x], s_p[threadIdx.x]);
}

// Where each class begins among the class-major rows (cptr), where its short
// rows begin (a class's rows ascend), and the item offsets at both.
struct ClassBounds {
  int64_t row[NUM_CLASSES + 1], row16[NUM_CLASSES];
  uint32_t item[NUM_CLASSES + 1], item16[NUM_CLASSES];
  uint32_t tasks;  // of all rows (a check)
  uint32_t packs[2], packs32[2];
};
__global__ void k_class_bounds(const uint32_t* __restrict__ crow, int64_t R, const int64_t* __restrict__ cptr,
                               const uint32_t* __restrict__ usc, const uint32_t* __restrict__ tsc, int64_t b16,
                               ClassBounds* __restrict__ out) {
  const int c = threadIdx.x;
  if (c > NUM_CLASSES) return;
  out->row[c] = cptr[c];
  out->item[c] = usc[cptr[c]];
  if (c == NUM_CLASSES) {
    out->tasks = tsc[R];
    return;
  }
  int64_t lo = cptr[c], hi = cptr[c + 1];
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)crow[mid] < b16) lo = mid + 1;
    else hi = mid;
  }
  out->row16[c] = lo;
  out->item16[c] = usc[lo];
}

// Packs of a class of nr rows, and those of its rows below i16.
__global__ void k_pack_totals(const uint32_t* __restrict__ flags, const uint32_t* __restrict__ pos, int64_t nr,
                              int64_t i16, int c, ClassBounds* __restrict__ out) {
  const uint32_t total = pos[nr - 1] + flags[nr - 1];
  out->packs[c] = total;
  out->packs32[c] = i16 < nr ? pos[i16] : total;
}

__global__ void k_rows_work(const int32_t* __restrict__ rows, int64_t nr,
                            const uint32_t* __restrict__ tbeg, const uint32_t* __restrict__ tend,
                            const uint64_t* __restrict__ tprefix, const int64_t* __restrict__ row_ptr,
                            int64_t b16, uint64_t* __restrict__ w, uint32_t* __restrict__ slots) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nr) return;
  int64_t b = rows[i];
  w[i] = row_weight(tprefix[tend[b]] - tprefix[tbeg[b]], b, b16);
  // a row without tasks (visited only without the doubly sparse traversal)
  // needs no table
  slots[i] = 1u << pack_table_log2(tend[b] > tbeg[b] ? row_ptr[b + 1] - row_ptr[b] : 0);
}

// A pack starts at row i when the running probe total, the running table
// slots or the row index enters a new multiple of its budget; so a pack holds
// at most kPackRows rows, at most `slots` slots plus one row's table, and at
// most `target` probes plus one row's. The short rows (from row i16 on) start
// a pack of their own and hold `slots16`.
__global__ void k_pack_flags(const uint64_t* __restrict__ pw, const uint32_t* __restrict__ ps,
                             int64_t nr, int64_t i16, uint64_t target, uint32_t slots32,
                             uint32_t slots16, uint32_t* __restrict__ flags) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nr) return;
  const uint32_t slots = i >= i16 ? slots16 : slots32;
  flags[i] = (i == 0 || i == i16 || pw[i] / target != pw[i - 1] / target || ps[i] / slots != ps[i - 1] / slots ||
              i / kPackRows != (i - 1) / kPackRows)
                 ? 1u
                 : 0u;
}

// Records of the pack rows (one thread per row) and of the packs (one thread
// per share of a pack: the share's first task, by binary search in the pack's
// task prefixes; the first share's also the rows and the probe range).
__global__ void k_pack_recs(const int32_t* __restrict__ rows, int64_t nr, const int64_t* __restrict__ row_ptr,
                            const uint32_t* __restrict__ tbeg, const uint32_t* __restrict__ tend,
                            PackRow* __restrict__ recs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nr) return;
  const int32_t b = rows[i];
  PackRow r;
  r.rs = (uint32_t)row_ptr[b];
  r.tb = tbeg[b];
  r.te = tend[b];
  r.d = r.te > r.tb ? (uint32_t)(row_ptr[b + 1] - row_ptr[b]) : 0u;
  recs[i] = r;
}

__global__ void k_pack_info(const uint32_t* __restrict__ pack_ptr, int64_t np, const PackRow* __restrict__ recs,
                            const uint64_t* __restrict__ tprefix, PackInfo* __restrict__ info) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t p = i / kPackWavesMax;
  const int w = (int)(i % kPackWavesMax);
  if (p >= np) return;
  const uint32_t r0 = pack_ptr[p], r1 = pack_ptr[p + 1];
  const uint32_t t_lo = recs[r0].tb, t_hi = recs[r1 - 1].te;
  const uint64_t q0 = tprefix[t_lo], q1 = tprefix[t_hi];
  const uint64_t wq0 = q0 + pack_share(q1 - q0, w);
  // last task t in [t_lo, t_hi) with tprefix[t] <= wq0 (t_lo when the pack
  // has no task: the share is then empty and never probed)
  uint32_t lo = t_lo, hi = t_hi > t_lo ? t_hi : t_lo + 1;
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (tprefix[mid] <= wq0) lo = mid;
    else hi = mid;
  }
  info[p].wt[w] = lo;
  if (w == 0) {
    info[p].q0 = q0;
    info[p].q1 = q1;
    info[p].r0 = r0;
    info[p].r1 = r1;
  }
}

// Launch order of a class's packs: heaviest first (longest-processing-time
// order), so that the launch does not end on a few long packs. Classes of
// fewer than kPackLptMin packs keep pack order (their launch is short; the
// sort would cost more than it saves, and batch plans order units themselves).
// Key = the complement of the pack's weight (its probes plus 64 per row), so
// that an ascending sort puts the heaviest first; the packs of short rows
// (from pack p16 on) carry the top bit, so that they stay last.
constexpr int64_t kPackLptMin = 2048;

// Short rows. Their bitmaps are cheap to set up, so a row gets work-groups of
// its own from kShortHeavyMin probes on (if heavy_min is not lower).
constexpr uint64_t kShortHeavyMin = 2048;
// Probes of a bundle, one work-group's share of the short rows' items, W
// probes in all: 1 / 16384 of them, but no less than 24K, under which a
// work-group's set-up shows (RMAT scale 18, 205M probes: 225 us in 8192
// bundles, 289 us in 16384), unless that would leave the 2048 work-groups
// that the GPU holds at once without one each, and no more than 256K, above
// which the last ones show (scale 22, 7.2G probes: 2662 us in 16384 bundles,
// 2586 us in 32768).
__host__ __device__ inline uint64_t bundle_weight(uint64_t W) {
  const uint64_t fill = W / 2048 < (24 << 10) ? W / 2048 : 24 << 10, least = fill < 4096 ? 4096 : fill;
  const uint64_t w = W / 16384 < least ? least : W / 16384;
  return w < (256 << 10) ? w : 256 << 10;
}

// Bundle boundaries of one class's short groups (items: the first of them;
// q0 grows along the groups): bundle i starts at the first group whose first
// probe lies i * per units after the first group's.
__global__ void k_bundles(const CountItem* __restrict__ items, int64_t groups, uint64_t per, int64_t n_bundles,
                          uint32_t* __restrict__ bundle) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= groups) return;
  const uint64_t q0 = items[0].q0;
  const int64_t at = (int64_t)((items[j * kWaves].q0 - q0) / per);
  const int64_t before = j ? (int64_t)((items[(j - 1) * kWaves].q0 - q0) / per) : -1;
  for (int64_t i = before + 1; i <= at; ++i) bundle[i] = (uint32_t)j;
  if (j == groups - 1)
    for (int64_t i = at + 1; i <= n_bundles; ++i) bundle[i] = (uint32_t)groups;
}
// Sort key of a pack: heavier first, to an eighth of its power of two (2^8 ..
// 2^24), short rows after the others. One digit: the order only has to start
// the long packs early. (All 31 bits took four passes: 100 us of the
// preprocessing at scale 20 against 26 us, and the counts take the same time.)
constexpr int kPackKeyBits = 8;
__global__ void k_pack_keys(const PackInfo* __restrict__ info, int64_t np, int64_t p16, uint32_t* __restrict__ key,
                            uint32_t* __restrict__ idx) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= np) return;
  const uint64_t w = info[p].q1 - info[p].q0 + 64ull * (info[p].r1 - info[p].r0);
  // exponent and three mantissa bits
  const int e = (int)(__float_as_uint((float)w) >> 20) - ((127 + 8) << 3);
  key[p] = (uint32_t)(127 - (e < 0 ? 0 : e > 127 ? 127 : e)) | (p >= p16 ? 128u : 0u);
  idx[p] = (uint32_t)p;
}

__global__ void k_pack_gather(const PackInfo* __restrict__ in, const uint32_t* __restrict__ idx, int64_t np,
                              PackInfo* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < np) out[p] = in[idx[p]];
}

__global__ void k_pack_emit(const uint32_t* __restrict__ flags, const uint32_t* __restrict__ pos,
                            int64_t nr, uint32_t* __restrict__ pack_ptr, int64_t np) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nr && flags[i]) pack_ptr[pos[i]] = (uint32_t)i;
  if (i == 0) pack_ptr[np] = (uint32_t)nr;
}

// One thread per wave item of a work-group class: find its row b (upper bound
// in the per-row item offsets), cut the row's probe range evenly and find the
// task holding the first probe.
// Wave items of the nr class-major rows crow[0..nr) of one class: offs
// (nr + 1 entries, absolute) is the exclusive prefix of their item counts;
// item j (0 <= j < total) is part idx of the row whose range holds offs[0] + j.
__global__ void k_emit_items(const uint32_t* __restrict__ offs, const uint32_t* __restrict__ crow, int64_t nr,
                             int64_t total, const uint32_t* __restrict__ tbeg,
                             const uint32_t* __restrict__ tend, const uint64_t* __restrict__ tprefix,
                             const int64_t* __restrict__ row_ptr, CountItem* __restrict__ items) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= total) return;
  const int64_t target = (int64_t)offs[0] + j;
  // largest r with offs[r] <= target (every row has at least one item)
  int64_t lo = 0, hi = nr;  // invariant offs[lo] <= target < offs[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)offs[mid] <= target) lo = mid;
    else hi = mid;
  }
  const int64_t b = crow[lo];
  const uint64_t parts = offs[lo + 1] - offs[lo];
  const uint64_t idx = (uint64_t)(target - (int64_t)offs[lo]);
  const int64_t t_lo = tbeg[b], t_hi = tend[b];
  const uint64_t P0 = tprefix[t_lo];
  const uint64_t W = tprefix[t_hi] - P0;
  const uint64_t per = W / parts, extra = W % parts;
  const uint64_t q0 = P0 + per * idx + (idx < extra ? idx : extra);
  const uint64_t q1 = q0 + per + (idx < extra ? 1 : 0);
  // task t in [t_lo, t_hi) with tprefix[t] <= q0 < tprefix[t+1]
  int64_t a = t_lo, z = t_hi;  // tprefix[a] <= q0 < tprefix[z] (if q0 < end)
  while (z - a > 1) {
    int64_t mid = (a + z) >> 1;
    if (tprefix[mid] <= q0) a = mid;
    else z = mid;
  }
  CountItem it;
  it.b = (int32_t)b;
  it.t0 = (uint32_t)a;
  it.q0 = q0;
  it.len = (uint32_t)(q1 - q0);
  it.rs = (uint32_t)row_ptr[b];
  it.d = (uint32_t)(row_ptr[b + 1] - row_ptr[b]);
  it.log2S = (uint32_t)table_log2(it.d);
  items[j] = it;
}

// ---- small graphs -----------------------------------------------------------
// A graph of at most kSmallN vertices and kSmallRaw raw pairs is bound by its
// launches and host round trips, not by its bytes: its degrees are counted in
// LDS from the sorted keys (no partition), its ranks are sorted by one
// work-group, its edges are oriented by the orient sort's own first pass (the
// rank map stays in L2: no partition either), and one work-group orders its
// rows by class and cuts its packs. Up to kBlockSortMax raw pairs every sort
// is one work-group's too (k_small_dedup, k_small_orient, k_small_tasks): a
// sort of three passes is 10 launches of 2-16 us otherwise.
constexpr int64_t kSmallN = 32768, kSmallRaw = 1 << 20;
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int64_t kBlockSortMax = 16 * kSmallThreads;
// Look-back words of a small graph's sorts (two bytes a pair hold those of its
// three sorts of up to four passes) and scans.
inline size_t sort_pool_bytes(int64_t m_raw) { return ((size_t)64 << 10) + ((2 * (size_t)m_raw + 255) & ~(size_t)255); }
constexpr size_t kSmallScanPool = (size_t)32 << 10;
// Up to as many pairs a small graph's temporaries are carved from one block:
// taking each from the cache and returning it records an event, and some 25 of
// them were a seventh of a small call (4096 vertices, 32768 pairs,
// preprocessing and count: 533 us, 460 us so). Past
// this, what a block without reuse holds beyond the peak would show in a
// server's memory budget (build_graph_bytes).
constexpr int64_t kArenaRaw = (int64_t)1 << 16;
inline size_t arena_bytes_of(int64_t m_raw, int64_t n) { return (size_t)(48 * m_raw + 48 * n) + ((size_t)256 << 10); }

// LDS of a block sort: the keys, per wave and digit a count, scratch. (At most
// 16 keys per thread: with 32 they spill, 105 us for 32768 pairs against 75 us
// in passes.)
template <int IPT>
struct BlockSort {
  uint32_t key[kSmallThreads * IPT];
  uint32_t cnt[kSmallWaves][256];
  uint32_t start[256];
  uint32_t tmp[4];
};

// Item i of lane l of wave w is element w * 64 IPT + 64 i + l.
template <int IPT>
__device__ __forceinline__ int block_item(int i) {
  return (int)(threadIdx.x >> 6) * 64 * IPT + 64 * i + (int)(threadIdx.x & 63);
}

// Stable sort of the work-group's keys by bits [bit_lo, bit_hi), ascending
// (the ranking of k_rs_onesweep, the whole array one tile). On return k[i] is
// element block_item(i) of the sorted array, and L.key holds it whole.
template <int IPT>
__device__ void block_sort(uint32_t (&k)[IPT], int bit_lo, int bit_hi, BlockSort<IPT>& L) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  for (int shift = bit_lo; shift < bit_hi; shift += 8) {
    const uint32_t dmask = (1u << (bit_hi - shift < 8 ? bit_hi - shift : 8)) - 1u;
    for (int x = tid; x < kSmallWaves * 256; x += kSmallThreads) (&L.cnt[0][0])[x] = 0;
    __syncthreads();
    uint32_t rank[IPT];
    uint32_t* cnt_w = L.cnt[wave];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const uint32_t d = (k[i] >> shift) & dmask;
      const uint64_t peers = rs_peers(d, true);
      const uint32_t before = cnt_w[d];
      rank[i] = before + (uint32_t)__popcll(peers & lt_mask);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if ((peers & lt_mask) == 0) cnt_w[d] = before + (uint32_t)__popcll(peers);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
    uint32_t total = 0, inc = 0;
    if (tid < 256) {
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        const uint32_t c = L.cnt[w][tid];
        L.cnt[w][tid] = total;
        total += c;
      }
      inc = wave_incl_scan(total);
      if (lane == 63) L.tmp[wave] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t before = 0;
      for (int w = 0; w < wave; ++w) before += L.tmp[w];
      L.start[tid] = before + inc - total;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const uint32_t d = (k[i] >> shift) & dmask;
      L.key[L.start[d] + L.cnt[wave][d] + rank[i]] = k[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) k[i] = L.key[block_item<IPT>(i)];
  }
}

// The sorted canonical keys S of at most 1024 IPT raw pairs (2 s <= 30 bits).
// Places past m_raw take all ones, whose sorted bits are the sentinel's: they
// stay behind the self loops.
template <int IPT>
__global__ __launch_bounds__(kSmallThreads) void k_small_dedup(CanonSrc cs, int m_raw, uint64_t* __restrict__ S,
                                                               int* __restrict__ err) {
  extern __shared__ int4 smem4[];
  BlockSort<IPT>& L = *reinterpret_cast<BlockSort<IPT>*>(smem4);
  uint32_t k[IPT];
  bool bad_any = false;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    bool bad;
    const uint32_t v = (uint32_t)cs.key(x < m_raw ? x : m_raw - 1, bad);
    bad_any |= bad;
    k[i] = x < m_raw ? v : 0xFFFFFFFFu;
  }
  if (bad_any) atomicOr(err, 1);
  block_sort<IPT>(k, 0, 2 * cs.s, L);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    if (x < m_raw) S[x] = k[i];
  }
}

// Distinct keys of S counted, and the degree of every vertex (deg zeroed
// before): each work-group counts its share of S in LDS (n counters), lower
// endpoints a run at a time (see k_degree_hist).
__global__ __launch_bounds__(kSmallThreads) void k_small_degree(const uint64_t* __restrict__ S, uint64_t sent,
                                                                int64_t m_raw, int64_t per, int s, int n,
                                                                uint32_t* __restrict__ deg,
                                                                unsigned long long* __restrict__ total) {
  extern __shared__ uint32_t h_deg[];
  __shared__ uint32_t s_c;
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x; j < n; j += kSmallThreads) h_deg[j] = 0;
  if (threadIdx.x == 0) s_c = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < m_raw ? i0 + per : m_raw;
  const uint64_t mask = (1ull << s) - 1, below = (1ull << lane) - 1ull;
  uint32_t c = 0;
  constexpr int kB = 4;
  for (int64_t wb = i0 + (int64_t)(threadIdx.x - lane) * kB; wb < i1; wb += (int64_t)kSmallThreads * kB) {
    uint64_t k[kB], prev[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int64_t i = wb + (int64_t)b * 64 + lane, ic = i < m_raw ? i : m_raw - 1;
      k[b] = S[ic];
      prev[b] = S[ic > 0 ? ic - 1 : 0];
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int64_t i = wb + (int64_t)b * 64 + lane;
      const bool ok = (i < i1) & (k[b] != sent) & ((i == 0) | (prev[b] != k[b]));
      const uint32_t lo = (uint32_t)(k[b] >> s);
      const uint32_t plo = (uint32_t)__shfl_up((int)lo, 1);
      const uint64_t heads = __ballot(lane == 0 || plo != lo), oks = __ballot(ok);
      if ((heads >> lane) & 1ull) {
        const uint64_t after = heads & ~below & ~(1ull << lane);
        const uint64_t run = (after ? (after & (~after + 1ull)) - 1ull : ~0ull) & ~below;
        const uint32_t r = (uint32_t)__popcll(oks & run);
        if (r) atomicAdd(&h_deg[lo], r);
      }
      if (ok) atomicAdd(&h_deg[k[b] & mask], 1u);
      if (lane == 0) c += (uint32_t)__popcll(oks);
    }
  }
  if (c) atomicAdd(&s_c, c);
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += kSmallThreads)
    if (h_deg[j]) atomicAdd(&deg[j], h_deg[j]);
  if (threadIdx.x == 0 && s_c) atomicAdd(total, (unsigned long long)s_c);
}

// Ranks of at most 1024 IPT vertices: stable by degree (below 2^15).
template <int IPT>
__global__ __launch_bounds__(kSmallThreads) void k_small_rank(const uint32_t* __restrict__ deg, int n, int deg_bits,
                                                              int32_t* __restrict__ perm,
                                                              uint32_t* __restrict__ deg_rank) {
  extern __shared__ int4 smem4[];
  BlockSort<IPT>& L = *reinterpret_cast<BlockSort<IPT>*>(smem4);
  uint32_t k[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int v = block_item<IPT>(i);
    k[i] = v < n ? (deg[v] << 16) | (uint32_t)v : 0xFFFFFFFFu;
  }
  block_sort<IPT>(k, 16, 16 + deg_bits, L);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int r = block_item<IPT>(i);
    if (r < n) {
      perm[k[i] & 0xFFFFu] = r;
      deg_rank[r] = k[i] >> 16;
    }
  }
}

// The orient sort's source: position i of S as the oriented key of its
// distinct edge.
struct OrientSrc {
  const uint64_t* S;
  uint64_t sent;
  const int32_t* perm;
  int s;
  __device__ bool operator()(int64_t i, uint64_t& k, char&) const {
    const uint64_t e = S[i], prev = S[i > 0 ? i - 1 : 0];
    const bool ok = (e != sent) & ((i == 0) | (prev != e));
    const uint64_t lo = ok ? e >> s : 0, hi = ok ? e & ((1ull << s) - 1) : 0;
    const uint64_t a = (uint32_t)perm[lo], b = (uint32_t)perm[hi];
    k = a < b ? ((a << s) | b) : ((b << s) | a);
    return ok;
  }
};

__global__ __launch_bounds__(256) void k_orient_digits(OrientSrc src, int64_t m_raw, int key_bits,
                                                       uint32_t* __restrict__ ghist) {
  extern __shared__ uint32_t h_dyn[];
  DigitCounter dc;
  dc.init(h_dyn, 0, key_bits);
  constexpr int kB = 4;
  const int64_t stride = (int64_t)gridDim.x * 256 * kB;
  for (int64_t base = (int64_t)blockIdx.x * 256 * kB + threadIdx.x; base < m_raw; base += stride) {
    uint64_t k[kB];
    bool ok[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      const int64_t i = base + (int64_t)j * 256;
      char none;
      ok[j] = src(i < m_raw ? i : m_raw - 1, k[j], none) & (i < m_raw);
    }
#pragma unroll
    for (int j = 0; j < kB; ++j)
      if (ok[j]) dc.add(k[j]);
  }
  dc.flush(ghist);
}

// The oriented keys and columns of U from at most 1024 IPT positions of S.
template <int IPT>
__global__ __launch_bounds__(kSmallThreads) void k_small_orient(OrientSrc src, int m_raw, int m,
                                                                uint64_t* __restrict__ okey, ColEpi epi) {
  extern __shared__ int4 smem4[];
  BlockSort<IPT>& L = *reinterpret_cast<BlockSort<IPT>*>(smem4);
  uint32_t k[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    uint64_t key;
    char none;
    const bool ok = src(x < m_raw ? x : m_raw - 1, key, none) & (x < m_raw);
    k[i] = ok ? (uint32_t)key : 0xFFFFFFFFu;  // (no oriented key has all 2 s bits set)
  }
  block_sort<IPT>(k, 0, 2 * src.s, L);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    if (x < m) {
      okey[x] = k[i];
      epi((uint64_t)x, (uint64_t)k[i]);
    }
  }
}

// The tasks of at most 1024 IPT entries of U, sorted by row (key: row and the
// entry, which keeps U's order within a row), and their number.
template <int IPT>
__global__ __launch_bounds__(kSmallThreads) void k_small_tasks(TaskSrc src, int m, int s, uint32_t* __restrict__ row,
                                                               uint64_t* __restrict__ val, uint32_t* __restrict__ total) {
  extern __shared__ int4 smem4[];
  BlockSort<IPT>& L = *reinterpret_cast<BlockSort<IPT>*>(smem4);
  uint32_t k[IPT], c = 0;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    uint32_t b;
    uint64_t v;
    const bool ok = src(x < m ? x : m - 1, b, v) & (x < m);
    k[i] = ok ? (b << 15) | (uint32_t)x : 0xFFFFFFFFu;  // (row 2^s - 1 has no task: no key of it follows)
    c += ok ? 1u : 0u;
  }
  block_sort<IPT>(k, 15, 15 + s, L);
  c = wave_sum(c);
  if (lane_id() == 0 && c) atomicAdd(total, c);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int x = block_item<IPT>(i);
    if (k[i] == 0xFFFFFFFFu) continue;
    uint32_t b;
    uint64_t v;
    (void)src((int64_t)(k[i] & 0x7FFFu), b, v);
    row[x] = b;
    val[x] = v;
  }
}

// Launches a block-sort kernel template at the smallest size that holds
// `count` elements.
#define TC_LAUNCH_BLOCK(name, kern, count, st, ...)                                                             \
  do {                                                                                                          \
    if ((count) <= 4 * kSmallThreads) launch_block<4>(name, kern<4>, st, __VA_ARGS__);                          \
    else if ((count) <= 8 * kSmallThreads) launch_block<8>(name, kern<8>, st, __VA_ARGS__);                     \
    else launch_block<16>(name, kern<16>, st, __VA_ARGS__);                                                     \
  } while (0)

// hipFuncSetAttribute for a kernel of more than 64 KiB of dynamic LDS: once per
// device and kernel, and again when a launch takes more than the launches
// before it.
void allow_lds(const void* f, size_t lds) {
  if (lds <= 65536) return;
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, size_t> allowed;
  int dev = 0;
  TC_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(mu);
  size_t& most = allowed[{dev, f}];
  if (lds <= most) return;
  TC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  most = lds;
}

template <int IPT, class... P, class... A>
void launch_block(const char* name, void (*kern)(P...), hipStream_t st, A... args) {
  allow_lds((const void*)kern, sizeof(BlockSort<IPT>));
  TC_LAUNCH(name, kern, dim3(1), dim3(kSmallThreads), sizeof(BlockSort<IPT>), st, args...);
  TC_HIP(hipGetLastError());
}

// ---- class-major order of a small graph's rows --------------------------------
// What the compaction, the class sort, the scans and the pack kernels below do
// for a large row set, by one work-group for at most kSmallN rows: the
// class-major row order, the prefixes of tasks, units and items along it, and
// the packs of the two pack classes. (A thread's rows per class, and those
// before it, are 16-bit fields.)
struct SmallOrder {
  ClassBounds cb;
  unsigned long long stats[NUM_CLASSES][3];  // rows, keys, tasks
  unsigned long long cw[NUM_CLASSES], cw16[NUM_CLASSES];
  uint64_t bundle_w;
  uint32_t chunk16, chunk[NUM_CLASSES];
  int cl[NUM_CLASSES];
};

// A class-major row: its units, tasks and keys.
struct alignas(16) RowRec {
  uint64_t W;
  uint32_t tasks, d;
};

// Exclusive scan over the work-group and the total (two barriers).
template <class T>
__device__ __forceinline__ T small_scan(T v, T* s_w, T& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T inc = wave_incl_scan(v);
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  T before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSmallWaves; ++w) {
    const T x = s_w[w];
    before += w < wave ? x : T(0);
    tot += x;
  }
  __syncthreads();
  total = tot;
  return before + inc - v;
}

// Probes per wave item of each item class, and of the short rows' bundles.
__host__ __device__ inline uint32_t class_chunk(uint64_t cw, int c, const WorkParams& wp) {
  const uint64_t per_group = wp.min_groups ? cw / ((uint64_t)wp.min_groups * class_waves(c)) : ~0ull;
  return per_group < kWaveChunkMin ? wp.wave_chunk
                                   : (uint32_t)(per_group < wp.wave_chunk ? per_group : wp.wave_chunk);
}

__global__ __launch_bounds__(kSmallThreads) void k_small_order(
    int n, const int8_t* __restrict__ cls, const int64_t* __restrict__ tptr, const uint64_t* __restrict__ tprefix,
    const int64_t* __restrict__ row_ptr, int64_t b16, WorkParams wp, const unsigned long long* __restrict__ cw,
    const unsigned long long* __restrict__ cw16, const int* __restrict__ cl, uint32_t* __restrict__ crow,
    uint32_t* __restrict__ tbeg, uint32_t* __restrict__ tend, uint32_t* __restrict__ cm_pos,
    uint64_t* __restrict__ wsc, uint32_t* __restrict__ usc, uint32_t* __restrict__ pack_ptr0,
    uint32_t* __restrict__ pack_ptr1, RowRec* __restrict__ rec, SmallOrder* __restrict__ out) {
  __shared__ uint64_t s_w64[kSmallWaves];
  __shared__ unsigned long long s_wu[kSmallWaves];
  __shared__ uint32_t s_w32[kSmallWaves];
  __shared__ uint64_t s_flag[kSmallWaves][kSmallN / kSmallWaves / 64];
  __shared__ unsigned long long s_stat[NUM_CLASSES][3];
  __shared__ uint32_t s_row[NUM_CLASSES + 1], s_row16[NUM_CLASSES], s_chunk[NUM_CLASSES];
  __shared__ uint32_t s_item[NUM_CLASSES + 1], s_item16[NUM_CLASSES];
  __shared__ uint16_t s_crow[kSmallN];
  const int tid = threadIdx.x;
  uint64_t cw_short = 0;
  for (int c = CLS_WG_SMALL; c < NUM_CLASSES; ++c) cw_short += cw16[c];
  const uint64_t bundle_w = bundle_weight(cw_short);
  const uint32_t chunk16 = (uint32_t)(bundle_w / kWaves < wp.wave_chunk ? bundle_w / kWaves : wp.wave_chunk);
  if (tid < NUM_CLASSES) {
    s_chunk[tid] = class_chunk(cw[tid], tid, wp);
    for (int j = 0; j < 3; ++j) s_stat[tid][j] = 0;
  }
  __syncthreads();
  // rows per class: of this thread, then before it
  const int R = (n + kSmallThreads - 1) / kSmallThreads;  // at most 32
  const int r0 = tid * R < n ? tid * R : n, r1 = r0 + R < n ? r0 + R : n;
  uint64_t lo = 0, hi = 0;  // 16-bit counts of classes 0-3, 4-6
  uint32_t cpack[4] = {0, 0, 0, 0};  // the rows' classes + 1, four bits each
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (8 * g >= R) break;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = r0 + 8 * g + j;
      const int c = r < r1 ? cls[r] : -1;
      cpack[g] |= (uint32_t)(c + 1) << (4 * j);
      lo += c >= 0 && c < 4 ? 1ull << (16 * c) : 0;
      hi += c >= 4 ? 1ull << (16 * (c - 4)) : 0;
    }
  }
  uint64_t lo_all, hi_all;
  lo = small_scan(lo, s_w64, lo_all);
  hi = small_scan(hi, s_w64, hi_all);
  if (tid == 0) {
    uint32_t at = 0;
    for (int c = 0; c <= NUM_CLASSES; ++c) {
      s_row[c] = at;
      if (c < NUM_CLASSES) at += (uint32_t)((c < 4 ? lo_all >> (16 * c) : hi_all >> (16 * (c - 4))) & 0xFFFFu);
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    if (j >= R) break;
    const int r = r0 + j;
    const int c = (int)((cpack[j / 8] >> (4 * (j % 8))) & 15u) - 1;
    if (c < 0) {
      if (r < r1) {  // a row without work: an empty task range
        tbeg[r] = 0;
        tend[r] = 0;
      }
      continue;
    }
    uint32_t p;
    if (c < 4) {
      p = (uint32_t)(lo >> (16 * c)) & 0xFFFFu;
      lo += 1ull << (16 * c);
    } else {
      p = (uint32_t)(hi >> (16 * (c - 4))) & 0xFFFFu;
      hi += 1ull << (16 * (c - 4));
    }
    s_crow[s_row[c] + p] = (uint16_t)r;
  }
  __syncthreads();
  const int Rt = (int)s_row[NUM_CLASSES];
  auto class_of = [&](int i) {
    int c = 0;
    while (i >= (int)s_row[c + 1]) ++c;
    return c;
  };
  if (tid < NUM_CLASSES) {  // first short row of each class
    uint32_t a = s_row[tid], z = s_row[tid + 1];
    while (a < z) {
      const uint32_t mid = (a + z) >> 1;
      if ((int64_t)s_crow[mid] < b16) a = mid + 1;
      else z = mid;
    }
    s_row16[tid] = a;
  }
  // prefixes along the class-major rows: each wave takes a contiguous share,
  // 64 rows at a time (consecutive lanes read and write consecutive rows: one
  // CU moves a cache line per cycle, and with consecutive rows per thread the
  // lines alone took 130 us of 16384 rows)
  auto items_of = [&](uint32_t b, int c, uint64_t W) -> uint32_t {
    if (c <= CLS_PACK_LARGE) return 0;
    return (int64_t)b >= b16 ? wg_parts(2 * W, kWaves, chunk16) : wg_parts(W, class_waves(c), s_chunk[c]);
  };
  const int lane = tid & 63, wave = tid >> 6;
  const int C = ((Rt + kSmallWaves - 1) / kSmallWaves + 63) & ~63;
  const int i0 = wave * C < Rt ? wave * C : Rt, i1 = i0 + C < Rt ? i0 + C : Rt;
  uint32_t tasks = 0, items = 0;
  uint64_t units = 0;
  {
    int c_run = -1;
    unsigned long long st[3] = {0, 0, 0};
    auto flush = [&]() {
      if (c_run >= 0)
        for (int j = 0; j < 3; ++j) atomicAdd(&s_stat[c_run][j], st[j]);
    };
    constexpr int kB = 4;
    for (int ib = i0 + lane; ib < i1; ib += 64 * kB) {
      RowRec q[kB];
      int64_t p0[kB], p1[kB];
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        const uint32_t b = s_crow[ib + 64 * j < i1 ? ib + 64 * j : i1 - 1];
        p0[j] = tptr[b];
        p1[j] = tptr[b + 1];
        q[j].d = (uint32_t)(row_ptr[b + 1] - row_ptr[b]);
      }
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        q[j].W = tprefix[p1[j]] - tprefix[p0[j]];
        q[j].tasks = (uint32_t)(p1[j] - p0[j]);
      }
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        const int i = ib + 64 * j;
        if (i >= i1) break;
        rec[i] = q[j];
        const int c = class_of(i);
        if (c != c_run) {
          flush();
          c_run = c;
          st[0] = st[1] = st[2] = 0;
        }
        st[0] += 1;
        st[1] += q[j].d;
        st[2] += q[j].tasks;
        tasks += q[j].tasks;
        units += q[j].W;
        items += items_of(s_crow[i], c, q[j].W);
      }
    }
    flush();
  }
  // (small_scan of the waves' totals: lane 63 brings them, the others 0)
  auto wave_base = [&](auto v, auto* s_w, auto& all) {
    const auto sum = wave_sum(v);
    const auto ex = small_scan(lane == 63 ? sum : decltype(v)(0), s_w, all);
    return __shfl(ex, 0, 64);
  };
  uint32_t tasks_all, items_all;
  unsigned long long units_all;
  tasks = wave_base(tasks, s_w32, tasks_all);
  items = wave_base(items, s_w32, items_all);
  unsigned long long ubase = wave_base((unsigned long long)units, s_wu, units_all);
  for (int ib = i0; ib < i1; ib += 64) {
    const int i = ib + lane;
    const bool in = i < i1;
    const RowRec q = rec[in ? i : i1 - 1];
    const uint32_t b = s_crow[in ? i : i1 - 1];
    const int c = class_of(in ? i : i1 - 1);
    const uint32_t it = in ? items_of(b, c, q.W) : 0;
    const uint32_t ts = wave_incl_scan(in ? q.tasks : 0u), is = wave_incl_scan(it);
    const unsigned long long us = wave_incl_scan((unsigned long long)(in ? q.W : 0));
    if (in) {
      crow[i] = b;
      cm_pos[b] = (uint32_t)i;
      tbeg[b] = tasks + ts - q.tasks;
      tend[b] = tasks + ts;
      wsc[i] = ubase + us - q.W;
      usc[i] = items + is - it;
      if (i == (int)s_row[c]) s_item[c] = items + is - it;
      if (i == (int)s_row16[c]) s_item16[c] = items + is - it;
    }
    tasks += (uint32_t)__shfl((int)ts, 63, 64);
    items += (uint32_t)__shfl((int)is, 63, 64);
    ubase += __shfl(us, 63, 64);
  }
  if (tid == 0) {
    wsc[Rt] = units_all;
    usc[Rt] = items_all;
    s_item[NUM_CLASSES] = items_all;
  }
  __syncthreads();
  // packs: a boundary where the running weight, the running slots or the row
  // enters a new multiple of its budget, and at the first short row
  const double inv_target = 1.0 / (double)wp.pack_target;
  auto target_of = [&](unsigned long long x) {  // x / pack_target (x < 2^53)
    unsigned long long q = (unsigned long long)((double)x * inv_target);
    if (q * wp.pack_target > x) --q;
    if ((q + 1) * wp.pack_target <= x) ++q;
    return q;
  };
#pragma unroll 1
  for (int c = CLS_PACK_SMALL; c <= CLS_PACK_LARGE; ++c) {
    const int c0 = (int)s_row[c], nr = (int)s_row[c + 1] - c0, i16 = (int)s_row16[c] - c0;
    const int P = ((nr + kSmallWaves - 1) / kSmallWaves + 63) & ~63;
    const int a = wave * P < nr ? wave * P : nr, z = a + P < nr ? a + P : nr;
    auto weigh = [&](int i, unsigned long long& w, uint32_t& sl) {
      const RowRec q = rec[c0 + i];
      w = row_weight(q.W, s_crow[c0 + i], b16);
      sl = 1u << pack_table_log2(q.tasks ? q.d : 0);
    };
    unsigned long long w = 0, all64;
    uint32_t sl = 0, all32, np;
    for (int i = a + lane; i < z; i += 64) {
      unsigned long long wi;
      uint32_t si;
      weigh(i, wi, si);
      w += wi;
      sl += si;
    }
    unsigned long long pw = wave_base(w, s_wu, all64);
    uint32_t ps = wave_base(sl, s_w32, all32);
    uint32_t count = 0;  // (uniform)
    for (int ib = a; ib < z; ib += 64) {
      const int i = ib + lane;
      unsigned long long wi = 0, lw = 0;
      uint32_t si = 0, ls = 0;  // l: the row before
      if (i < z) weigh(i, wi, si);
      if (i > 0 && i < z) weigh(i - 1, lw, ls);
      const unsigned long long wx = pw + wave_incl_scan(wi) - wi;
      const uint32_t sx = ps + wave_incl_scan(si) - si;
      const uint32_t budget = i >= i16 ? short_pack_slots(wp.pack_slots) : wp.pack_slots;
      const bool start = i < z && (i == 0 || i == i16 || target_of(wx) != target_of(wx - lw) ||
                                   sx / budget != (sx - ls) / budget || i % kPackRows == 0);
      const uint64_t f = __ballot(start);
      if (lane == 0) s_flag[wave][(ib - a) >> 6] = f;
      count += (uint32_t)__popcll(f);
      pw = __shfl(wx + wi, 63, 64);
      ps = (uint32_t)__shfl((int)(sx + si), 63, 64);
    }
    uint32_t at = wave_base(lane == 63 ? count : 0u, s_w32, np);
    uint32_t* ptr = c == 0 ? pack_ptr0 : pack_ptr1;
    for (int ib = a; ib < z; ib += 64) {
      const int i = ib + lane;
      const uint64_t f = s_flag[wave][(ib - a) >> 6];
      const uint32_t p = at + (uint32_t)__popcll(f & ((1ull << lane) - 1ull));
      if (i < z && i == i16) out->cb.packs32[c] = p;
      if ((f >> lane) & 1ull) ptr[p] = (uint32_t)i;
      at += (uint32_t)__popcll(f);
    }
    if (tid == 0) {
      ptr[np] = (uint32_t)nr;
      if (i16 >= nr) out->cb.packs32[c] = np;
      out->cb.packs[c] = np;
    }
    __syncthreads();  // (s_flag is written again)
  }
  if (tid == 0) {
    // (an empty class, and one without short rows, end where the next begins)
    for (int c = NUM_CLASSES - 1; c >= 0; --c) {
      if (s_row[c] == s_row[c + 1]) s_item[c] = s_item[c + 1];
      if (s_row16[c] == s_row[c + 1]) s_item16[c] = s_item[c + 1];
    }
    for (int c = 0; c <= NUM_CLASSES; ++c) {
      out->cb.row[c] = s_row[c];
      out->cb.item[c] = s_item[c];
      if (c == NUM_CLASSES) break;
      out->cb.row16[c] = s_row16[c];
      out->cb.item16[c] = s_item16[c];
      for (int j = 0; j < 3; ++j) out->stats[c][j] = s_stat[c][j];
      out->cw[c] = cw[c];
      out->cw16[c] = cw16[c];
      out->cl[c] = cl[c];
      out->chunk[c] = s_chunk[c];
    }
    out->cb.tasks = tasks_all;
    out->bundle_w = bundle_w;
    out->chunk16 = chunk16;
  }
}

}  // namespace

struct GraphImpl : Graph {
  Owned owned;
};

void destroy_graph_idle(Graph* g) {
  GraphImpl* gi = static_cast<GraphImpl*>(g);
  gi->owned.release(true);
  delete gi;
}

void destroy_graph(Graph* g) {
  // work on the graph may still be queued on the streams that used it: the
  // memory goes back to the cache, reusable once that work is done
  GraphImpl* gi = static_cast<GraphImpl*>(g);
  gi->uses.release_after_uses(gi->owned);
  delete gi;
}

Graph* build_graph(const int32_t* d_src, const int32_t* d_dst, int64_t m_raw, int64_t n,
                   hipStream_t st, bool lean) {
  std::unique_ptr<GraphImpl> g(new GraphImpl());
  g->owned.st = st;
  TC_HIP(hipGetDevice(&g->device));
  TempStream temps(st);  // temporaries are stream-ordered on st
  g->n = n;
  g->m_raw = m_raw;
  const int s = std::max(1, ceil_log2_u64((uint64_t)n));
  g->sbits = s;
  const uint64_t sent = (2 * s >= 64) ? ~0ull : ((1ull << (2 * s)) - 1);

  // Everything below that starts at zero, in one buffer cleared by one
  // memset: 64 bytes of scalars (id error (int) at 0, dedup refused (int) at 4, distinct count m
  // (u64) at 8, W+ (u64) at 16, largest d+ (u32) at 24, task count (u32) at
  // 28: two host reads of 16 bytes), then the digit counts of the degree
  // partition (2 x 256), of the canonical keys, of the oriented keys and of
  // the tasks (kSortPassesMax x 256 each).
  // A small graph's vertex degrees follow, and the look-back words of its
  // sorts.
  const bool small = n <= kSmallN && m_raw <= kSmallRaw;
  const bool block_sorts = small && m_raw <= kBlockSortMax;
  constexpr size_t kHistWords = 256 * kSortPassesMax;
  const size_t deg_at = 64 + sizeof(uint32_t) * (256 * 2 + 3 * kHistWords);
  const size_t pool_at = deg_at + (small ? (sizeof(uint32_t) * (size_t)n + 255) & ~(size_t)255 : 0);
  // (and of the scans)
  const size_t pool_bytes = small && !block_sorts ? sort_pool_bytes(m_raw) : 0;
  // (every part begins at a multiple of 64 bytes: the scan words are 64-bit)
  const size_t scan_at = pool_at + pool_bytes, scan_bytes = small ? kSmallScanPool : kScanPool;
  DevBuf arena;
  if (small && m_raw <= kArenaRaw && !lean) {
    arena.alloc(arena_bytes_of(m_raw, n));
    temps.carve_from(arena.as<char>(), arena.bytes);
  }
  DevBuf zs(scan_at + scan_bytes);
  TC_HIP(hipMemsetAsync(zs.p, 0, zs.bytes, st));
  if (pool_bytes) temps.zero_pool(zs.as<char>() + pool_at, pool_bytes);
  temps.scan_pool(zs.as<char>() + scan_at, scan_bytes);
  char* const zb = zs.as<char>();
  int* d_err = reinterpret_cast<int*>(zb);
  int* d_refused = reinterpret_cast<int*>(zb + 4);
  unsigned long long* d_m = reinterpret_cast<unsigned long long*>(zb + 8);
  unsigned long long* d_wplus = reinterpret_cast<unsigned long long*>(zb + 16);
  unsigned int* d_maxd = reinterpret_cast<unsigned int*>(zb + 24);
  uint32_t* d_T = reinterpret_cast<uint32_t*>(zb + 28);
  uint32_t* const dh = reinterpret_cast<uint32_t*>(zb + 64);
  uint32_t* const ch = dh + 256 * 2;
  uint32_t* const ohist = ch + kHistWords;
  uint32_t* const th = ohist + kHistWords;

  // ---- 1-2: simple graph -------------------------------------------------
  // The keys are sorted (duplicates close together) into S; the distinct keys
  // are never written out: the degree count, its partition and the
  // orientation select them from S (DistinctSel). The other sort buffer later
  // holds the oriented keys, and S's buffer is the orient sort's ping-pong
  // partner.
  int64_t m = 0;
  DevBuf ka(sizeof(uint64_t) * (size_t)std::max<int64_t>(m_raw, 1));
  DevBuf kb(sizeof(uint64_t) * (size_t)std::max<int64_t>(m_raw, 1));
  bool salt = false;  // S is in kb
  // degree partition: one radix pass (8 bits) up to s = 24 (a bucket then
  // spans at most 2 LDS ranges, each reading the bucket's entries), two
  // beyond; dh: its digit counts, which the sort scans into digit starts
  // (the bucket starts of the degree count; the last pass's are reused by
  // the orientation's partition)
  const int hshift = s <= 8 ? 0 : s <= 24 ? s - 8 : s - 16;
  const int hpasses = digit_passes(hshift, s);
  // mixed keys: intervals of lo as the degree count's ranges begin at
  const MixCode mc{s, std::min(hshift, kDegBinsLog2)};
  // Passes over the top 8 bits each that leave at most 2^kGrpMeanLog2 keys a
  // group on average if all edges shared one interval of lo (the mixed bits
  // are even). Preprocessing and count: 53.6 -> 50.6 ms at scale 24 (3 passes
  // instead of 6), 4031 -> 3819 us at scale 20 and 2564 -> 2449 us for a
  // million vertices of equal degree (3 instead of 5).
  int gpasses = digit_passes(0, s - mc.low);
  while (8 * gpasses < 2 * s && m_raw > (int64_t)1 << std::min(62, 8 * gpasses + kGrpMeanLog2 - (s - mc.low)))
    ++gpasses;
  for (bool grouped = !small && 8 * gpasses < 2 * s;; grouped = false) {
    // the keys are built by the first pass of the dedup sort from the raw
    // pairs (7168-pair tiles: the largest whose registers allow four waves per
    // SIMD); one read of the pairs before it counts their digits and checks
    // the ids
    const CanonSrc csrc{d_src, d_dst, n, s, sent};
    const MixSrc msrc{d_src, d_dst, n, mc};
    const int bit_lo = grouped ? 2 * s - 8 * gpasses : 0;
    const unsigned pblocks = (unsigned)std::min<int64_t>(kProducerBlocks, div_up(m_raw, kT * kDigitBatch));
    if (m_raw > 0 && block_sorts) {
      TC_LAUNCH_BLOCK("small_dedup", k_small_dedup, m_raw, st, csrc, (int)m_raw, ka.as<uint64_t>(), d_err);
    } else if (m_raw > 0 && small) {
      TC_LAUNCH("canon_digits", (k_canon_digits<CanonSrc>), dim3(pblocks), dim3(kT), digit_lds_bytes(0, 2 * s), st,
                csrc, m_raw, 0, 2 * s, ch, d_err);
      TC_HIP(hipGetLastError());
      salt = radix_sort_from<uint64_t, NoVal, CanonSrc, 14>(csrc, m_raw, ka.as<uint64_t>(), kb.as<uint64_t>(),
                                                            nullptr, nullptr, m_raw, 0, 2 * s, ch,
                                                            st, "dedup");
    } else if (m_raw > 0) {
      TC_LAUNCH("canon_digits", (k_canon_digits<MixSrc>), dim3(pblocks), dim3(kT), digit_lds_bytes(bit_lo, 2 * s), st,
                msrc, m_raw, bit_lo, 2 * s, ch, d_err);
      TC_HIP(hipGetLastError());
      salt = radix_sort_from<uint64_t, NoVal, MixSrc, 14>(msrc, m_raw, ka.as<uint64_t>(), kb.as<uint64_t>(),
                                                          nullptr, nullptr, m_raw, bit_lo, 2 * s, ch,
                                                          st, "dedup");
    }
    uint64_t* const S = salt ? kb.as<uint64_t>() : ka.as<uint64_t>();
    if (m_raw > 0 && small) {
      const int64_t per = std::max<int64_t>(8192, div_up(m_raw, 64));
      allow_lds((const void*)k_small_degree, sizeof(uint32_t) * (size_t)n);
      TC_LAUNCH("small_degree", k_small_degree, dim3((unsigned)div_up(m_raw, per)), dim3(kSmallThreads),
                sizeof(uint32_t) * (size_t)n, st, S, sent, m_raw, per, s, (int)n,
                reinterpret_cast<uint32_t*>(zb + deg_at), d_m);
      TC_HIP(hipGetLastError());
    } else if (m_raw > 0) {
      // duplicates marked, distinct keys counted, with their upper
      // endpoints' partition digits
      const size_t lds = digit_lds_bytes(hshift, s);
      if (grouped) {
        allow_lds((const void*)k_distinct_groups, lds);
        TC_LAUNCH("distinct_groups", k_distinct_groups,
                  dim3((unsigned)std::min<int64_t>(512, div_up(m_raw, kGrpTile))), dim3(kGrpThreads), lds, st, S, mc,
                  m_raw, bit_lo, group_max(m_raw), hshift, dh, d_m, d_refused);
      } else {
        TC_LAUNCH("distinct_mark", k_distinct_mark, dim3(pblocks), dim3(kT), lds, st, S, mc, m_raw, hshift, dh, d_m);
      }
      TC_HIP(hipGetLastError());
    }
    // the id check and the distinct count: one host sync for both
    struct {
      int err;
      int refused;
      unsigned long long m;
    } h;
    static_assert(sizeof(h) == 16, "scalar layout");
    TC_HIP(hipMemcpyAsync(&h, zb, sizeof(h), hipMemcpyDeviceToHost, st));
    TC_HIP(hipStreamSynchronize(st));
    const unsigned long long h_m = h.m;
    TC_REQUIRE(h.err == 0, TC_EINVAL, "tc_preprocess: vertex id outside [0, n)");
    if (h.refused) {  // (a group too large for its hash set: all counts again, from a full sort)
      TC_HIP(hipMemsetAsync(zs.p, 0, zs.bytes, st));
      continue;
    }
    TC_REQUIRE(h_m < (unsigned long long)kMaxEdges, TC_EOVERFLOW, "tc_preprocess: 2^32 - 256 or more edges");
    m = (int64_t)h_m;
    break;
  }
  g->m = m;
  DevBuf& sbuf = salt ? kb : ka;     // S
  DevBuf& obuf = salt ? ka : kb;     // free: the oriented keys go here
  const DistinctSel dsel{sbuf.as<uint64_t>()};

  // ---- 3: degree order ---------------------------------------------------
  g->perm = g->owned.alloc<int32_t>(n);
  g->deg = g->owned.alloc<uint32_t>(n);
  const uint32_t* hi_starts = dh + 256 * (hpasses - 1);  // valid once m > 0
  if (small && n <= kBlockSortMax) {
    TC_LAUNCH_BLOCK("small_rank", k_small_rank, n, st, reinterpret_cast<const uint32_t*>(zb + deg_at), (int)n, s,
                    g->perm, g->deg);
  } else {
    DevBuf ra(sizeof(uint64_t) * (size_t)n), rb(sizeof(uint64_t) * (size_t)n);
    if (small) {
      TC_LAUNCH("rank_keys", k_rank_keys, dim3(grid_for(n)), dim3(kT), 0, st,
                reinterpret_cast<const uint32_t*>(zb + deg_at), n, s, ra.as<uint64_t>());
      TC_HIP(hipGetLastError());
    } else if (m > 0) {
      // upper endpoints partitioned by their top bits (read from S through
      // the distinct keys) and counted per bucket in LDS with the lower
      // endpoints (k_degree_hist, which writes the rank keys)
      DevBuf hb(sizeof(uint32_t) * (size_t)m), hb2(hpasses > 1 ? sizeof(uint32_t) * (size_t)m : 0);
      const bool halt = radix_sort_from<uint32_t, NoVal>(DistinctHiSrc{dsel, mc}, m_raw, hb.as<uint32_t>(),
                                                         hb2.as<uint32_t>(), nullptr, nullptr, m, hshift, s,
                                                         dh, st, "degree", NoEpi{}, false, true);
      const uint32_t* hsorted = halt ? hb2.as<uint32_t>() : hb.as<uint32_t>();
      const int64_t span = (int64_t)1 << hshift;  // vertices per bucket
      const int sub = (int)div_up(span, kDegBins);
      const int64_t nbuckets = div_up(n, span);
      const int64_t groups = nbuckets * sub;
      const size_t lds = sizeof(uint32_t) * kDegBins;
      allow_lds((const void*)k_degree_hist, lds);
      // bucket starts: with one digit pass, its digit starts as the sort
      // scanned them (256 exclusive starts); else found by binary search
      DevBuf bp;
      const uint32_t* bs32 = dh;
      int64_t nbs = 256;
      if (hpasses != 1) {
        bp.alloc(sizeof(int64_t) * (size_t)(nbuckets + 1));
        TC_LAUNCH("bounds", (k_bounds<uint32_t>), dim3(grid_for(nbuckets + 1)), dim3(kT), 0, st, hsorted, m,
                  hshift, nbuckets, bp.as<int64_t>());
        bs32 = nullptr;
        nbs = nbuckets + 1;
      }
      TC_LAUNCH("degree_hist", k_degree_hist, dim3((unsigned)groups), dim3(kDegThreads), lds, st, hsorted, bs32,
                bs32 ? nullptr : bp.as<int64_t>(), nbs, m, hshift, sub, dsel, m_raw, n, mc, ra.as<uint64_t>());
      TC_HIP(hipGetLastError());
    } else {
      DevBuf deg(sizeof(uint32_t) * (size_t)n);
      TC_LAUNCH("fill_u32", k_fill_u32, dim3(grid_for(n)), dim3(kT), 0, st, deg.as<uint32_t>(), n, 0u);
      TC_LAUNCH("rank_keys", k_rank_keys, dim3(grid_for(n)), dim3(kT), 0, st, deg.as<uint32_t>(), n, s,
                ra.as<uint64_t>());
      TC_HIP(hipGetLastError());
    }
    bool alt = radix_sort<uint64_t, NoVal>(ra.as<uint64_t>(), rb.as<uint64_t>(), nullptr, nullptr, n,
                                           s, 2 * s, st, "rank");
    TC_LAUNCH("perm", k_perm, dim3(grid_for(n)), dim3(kT), 0, st,
                       alt ? rb.as<uint64_t>() : ra.as<uint64_t>(), n, s, g->perm, g->deg);
    TC_HIP(hipGetLastError());
  }

  // ---- 4: orient, U in CSR -------------------------------------------------
  g->row_ptr = g->owned.alloc<int64_t>(n + 1);
  g->col = g->owned.alloc<int32_t>(m);
  g->col16 = g->owned.alloc<uint16_t>(m + 2);
  const uint64_t* okey = obuf.as<uint64_t>();
  DevBuf ne;  // bitmap of U's non-empty rows
  const ColEpi col_epi{g->col, g->col16, n, s};
  if (small && m > 0) {
    const OrientSrc osrc{sbuf.as<uint64_t>(), sent, g->perm, s};
    if (block_sorts) {
      TC_LAUNCH_BLOCK("small_orient", k_small_orient, m_raw, st, osrc, (int)m_raw, (int)m, obuf.as<uint64_t>(),
                      col_epi);
    } else {
      TC_LAUNCH("orient_digits", k_orient_digits, dim3((unsigned)std::min<int64_t>(256, div_up(m_raw, kT * 4))),
                dim3(kT), digit_lds_bytes(0, 2 * s), st, osrc, m_raw, 2 * s, ohist);
      TC_HIP(hipGetLastError());
      // (S is read by the first pass alone: its buffer is the partner of the others)
      if (radix_sort_from<uint64_t, NoVal, OrientSrc, 14, ColEpi>(osrc, m_raw, obuf.as<uint64_t>(),
                                                                  sbuf.as<uint64_t>(), nullptr, nullptr, m, 0, 2 * s,
                                                                  ohist, st, "orient", col_epi))
        okey = sbuf.as<uint64_t>();
    }
  } else {
    if (m > 0) {
      // partition by the top 8 bits of hi (one pass from S into the free
      // buffer), then the oriented keys in place
      // (14 edges per thread, as the canonicalising pass: a source that
      // loads twice per element needs the registers)
      const bool palt = radix_sort_from<uint64_t, NoVal, LoRankSrc, 14>(
          LoRankSrc{dsel, g->perm, mc}, m_raw, obuf.as<uint64_t>(), nullptr, nullptr, nullptr, m,
          s > 8 ? s - 8 : 0, s, const_cast<uint32_t*>(hi_starts), st, "orient_part", NoEpi{}, true);
      TC_REQUIRE(!palt, TC_EDEVICE, "tc_preprocess: the orientation partition is one pass");
      const int64_t og = std::min<int64_t>(kProducerBlocks, div_up(m, kT * 2 * kEw));
      TC_LAUNCH("orient", k_orient_hi, dim3((unsigned)(div_up(og, 8) * 8)), dim3(kT), digit_lds_bytes(0, 2 * s),
                st, obuf.as<uint64_t>(), m, s, g->perm, ohist);
      TC_HIP(hipGetLastError());
      // S's buffer is the ping-pong partner (S is not read after the
      // partition); the last pass also writes each key's column: U's col
      bool alt = radix_sort<uint64_t, NoVal, ColEpi>(obuf.as<uint64_t>(), sbuf.as<uint64_t>(), nullptr, nullptr,
                                                     m, 0, 2 * s, st, "orient", col_epi,
                                                     ohist);
      if (alt) okey = sbuf.as<uint64_t>();
      if (m == 1)  // no sort pass ran
        TC_LAUNCH("col", k_col, dim3(grid_for(m)), dim3(kT), 0, st, okey, m, s, g->col);
    } else {
      TC_LAUNCH("fill_i64", k_fill_i64, dim3(grid_for(n + 1)), dim3(kT), 0, st, g->row_ptr, n + 1,
                         (int64_t)0);
    }
  }
  if (m > 0) {
    ne.alloc(sizeof(uint64_t) * (size_t)div_up(n, 64));
    TC_LAUNCH("rows", k_rows, dim3((unsigned)std::min<int64_t>(kRowsBlocks, div_up(n + 1, kRowsPer))), dim3(kRowsThreads), 0, st, okey, m, s, n,
              g->row_ptr, g->col16, ne.as<uint64_t>(), d_wplus, d_maxd);
  }
  TC_HIP(hipGetLastError());
  // the buffer that does not hold the oriented keys is free now
  (okey == sbuf.as<uint64_t>() ? obuf : sbuf).release();
  // (W+ and the largest d+ are read back with the task count below: one
  // host sync)

  // ---- 5: tasks grouped by hashed row b -----------------------------------
  // one read of U counts the tasks and their key digits; the first pass of
  // the task sort reads U again and builds the tasks it ranks (no task list
  // is written in U order)
  TaskLists tl;
  {
    TaskSrc src{};
    if (m > 0) src.p = TaskPred{okey, s, g->row_ptr, ne.as<uint64_t>(), nullptr, nullptr};
    const bool block_tasks = block_sorts && m > 0;  // (m <= m_raw)
    if (block_tasks) {
      tl.row.alloc(sizeof(uint32_t) * (size_t)m);
      tl.val.alloc(sizeof(uint64_t) * (size_t)m);
      TC_LAUNCH_BLOCK("small_tasks", k_small_tasks, m, st, src, (int)m, s, tl.row.as<uint32_t>(),
                      tl.val.as<uint64_t>(), d_T);
    } else if (m > 0) {
      TC_LAUNCH("task_digits", k_task_digits,
                dim3((unsigned)std::min<int64_t>(kProducerBlocks, div_up(m, kT * kDigitBatch))), dim3(kT),
                digit_lds_bytes(0, s), st, src, m, s, th, d_T);
      TC_HIP(hipGetLastError());
    }
    struct {
      unsigned long long wplus;
      unsigned int maxd;
      uint32_t T;
    } h;
    static_assert(sizeof(h) == 16, "scalar layout");
    TC_HIP(hipMemcpyAsync(&h, zb + 16, sizeof(h), hipMemcpyDeviceToHost, st));
    TC_HIP(hipStreamSynchronize(st));  // the task count, W+ and the largest d+
    const int64_t T = h.T;
    tl.T = T;
    tl.ptr.alloc(sizeof(int64_t) * (size_t)(n + 1));
    if (T > 0 && !block_tasks) {
      tl.row.alloc(sizeof(uint32_t) * (size_t)T);
      tl.val.alloc(sizeof(uint64_t) * (size_t)T);
      DevBuf tk(sizeof(uint32_t) * (size_t)T), tv(sizeof(uint64_t) * (size_t)T);
      const bool alt = radix_sort_from<uint32_t, uint64_t, TaskSrc, 11>(src, m, tl.row.as<uint32_t>(), tk.as<uint32_t>(),
                                                           tl.val.as<uint64_t>(), tv.as<uint64_t>(), T, 0, s,
                                                           th, st, "tasks");
      if (alt) {
        tl.row.swap(tk);
        tl.val.swap(tv);
      }
    }
    g->wedges_plus = (int64_t)h.wplus;
    g->max_dplus = (int64_t)h.maxd;
    finish_tasks(tl, n, short_rows_begin(n, m, g->max_dplus), st);
  }
  ka.release();
  kb.release();

  // ---- 6: work classes ------------------------------------------------------
  build_work(g->w, g->owned, n, g->row_ptr, tl.T, tl.row.as<uint32_t>(), tl.ptr.as<int64_t>(),
             tl.val.as<uint64_t>(), tl.prefix.as<uint64_t>(), short_rows_begin(n, m, g->max_dplus),
             default_work_params(m), st);
  check_sorts(st);
  finish_work(g->w);
  g->arena_bytes = g->owned.bytes;
  note_use(*g, st);
  return g.release();
}

// The blocks of build_graph that live together, phase by phase, as the cache
// rounds them; m <= m_raw, at most as many tasks, rows with work at most that
// many and at most n.
size_t build_graph_bytes(int64_t m_raw, int64_t n) {
  const int64_t m = std::max<int64_t>(m_raw, 1), r = std::min(n, m);
  auto B = [](int64_t bytes) { return cache_block_bytes((size_t)bytes); };
  const size_t upload = B(8 * m);
  const size_t ranks = 2 * B(4 * n), u = B(8 * (n + 1)) + B(4 * m) + B(2 * m + 4);
  // task arrays, row order, pack pointers and records; work units: 8 bytes an
  // edge up to 2^20 of them, 1 beyond
  const size_t work = 2 * B(4 * n) + B(4 * m) + B(8 * (m + 1)) + B(4 * n) + 2 * B(4 * (n + 1)) + 2 * B(8 * r) +
                      B(8 * std::min(m, (int64_t)1 << 20) + m);
  const size_t fixed = (size_t)1 << 20;  // zeroed words, scalars, rounding of the classes' arrays
  if (m_raw <= kArenaRaw && n <= kSmallN) return upload + B((int64_t)arena_bytes_of(m_raw, n)) + ranks + u + work + fixed;
  const size_t words = B(m / 4);  // look-back words of a sort
  const size_t dedup = 2 * B(8 * m) + words;
  const size_t degree = dedup + ranks + 2 * B(8 * n) + B(4 * m) + (n > (1 << 24) ? B(4 * m) : 0);
  const size_t tasks = B(8 * m) + ranks + u + B(8 * (n + 1)) + 2 * (B(4 * m) + B(8 * m)) + words;
  const size_t rows = B(n) + B(4 * n) + 5 * B(4 * r) + 4 * B(8 * r) + 4 * B(4 * r);
  const size_t order = ranks + u + B(8 * (n + 1)) + B(4 * m) + 2 * B(8 * m) + work + rows;
  return upload + std::max(std::max(degree, tasks), order) + fixed;
}

void check_task_sorts(hipStream_t st) { check_sorts(st); }

namespace {

// Tasks of a variant work set, one test per nonzero p = (a, b) of U (a from
// erow). <j,i,k> (the default): hashed row b, probes = U_a's entries after b,
// skipped when there are none, and also when U_b is empty unless keep_empty.
// <i,j,k>: hashed row a, probes = all of U_b (skipped when U_b is empty: such
// a task has nothing to look up).
struct VariantTaskPred {
  const int64_t* row_ptr;
  const int32_t* col;
  const uint32_t* erow;
  bool ijk, keep_empty;
  uint32_t* tkey;
  uint64_t* tval;
  struct Item {
    uint32_t key;
    uint64_t val;
  };
  __device__ bool operator()(int64_t p, Item& it) const {
    const uint32_t a = erow[p];
    const int32_t b = col[p];
    const int64_t bs = row_ptr[b], be = row_ptr[b + 1];
    if (ijk) {
      it.key = a;
      it.val = (uint64_t)bs | ((uint64_t)be << 32);
      return be > bs;
    }
    const int64_t end = row_ptr[a + 1];
    it.key = (uint32_t)b;
    it.val = (uint64_t)(p + 1) | ((uint64_t)end << 32);
    return end - p - 1 > 0 && (keep_empty || be > bs);
  }
  __device__ void emit(int64_t, const Item& it, uint32_t pos) const {
    tkey[pos] = it.key;
    tval[pos] = it.val;
  }
};

}  // namespace

Graph* build_variant(const Graph& base, int flags, const WorkParams& wp, hipStream_t st) {
  std::unique_ptr<GraphImpl> g(new GraphImpl());
  g->owned.st = st;
  TC_HIP(hipGetDevice(&g->device));
  TC_REQUIRE(g->device == base.device, TC_EINVAL, "tc_graph_variant: graph built on another device");
  TempStream temps(st);
  g->n = base.n;
  g->m_raw = base.m_raw;
  g->m = base.m;
  g->wedges_plus = base.wedges_plus;
  g->max_dplus = base.max_dplus;
  g->sbits = base.sbits;
  g->row_ptr = base.row_ptr;  // U is shared, not owned
  g->col = base.col;
  g->perm = base.perm;
  g->col16 = base.col16;
  g->deg = base.deg;
  g->variant = flags;
  g->hash = (flags & TC_VARIANT_MUL_HASH) ? 1 : 0;
  g->base = &base;
  const bool ijk = (flags & TC_VARIANT_IJK) != 0, no_dcsr = (flags & TC_VARIANT_NO_DCSR) != 0;
  const int64_t n = g->n, m = g->m;
  // (<i,j,k> looks up whole rows, first entries included, and the hashing
  // ablation compares 32-bit tables: no short rows there)
  const int64_t b16 = ijk || g->hash ? n : short_rows_begin(n, m, base.max_dplus);
  TaskLists tl;
  if (m > 0) {
    DevBuf erow(sizeof(uint32_t) * (size_t)m);
    TC_LAUNCH("entry_rows", k_entry_rows, dim3(entry_rows_grid(n)), dim3(kT), 0, st, g->row_ptr, n,
              erow.as<uint32_t>());
    DevBuf tk, tv;
    VariantTaskPred vp{g->row_ptr, g->col, erow.as<uint32_t>(), ijk, no_dcsr, nullptr, nullptr};
    const int64_t T = compact("variant_tasks", m, vp, [&](int64_t total, VariantTaskPred& pr) {
      tk.alloc(sizeof(uint32_t) * (size_t)total);
      tv.alloc(sizeof(uint64_t) * (size_t)total);
      pr.tkey = tk.as<uint32_t>();
      pr.tval = tv.as<uint64_t>();
    }, st);
    if (T > 0) sort_tasks(tl, tk, tv, T, n, g->sbits, b16, st, "variant_tasks");
  }
  build_work(g->w, g->owned, n, g->row_ptr, tl.T, tl.row.as<uint32_t>(), tl.ptr.as<int64_t>(),
             tl.val.as<uint64_t>(), tl.prefix.as<uint64_t>(), b16, wp, st, no_dcsr);
  check_sorts(st);
  finish_work(g->w);
  g->arena_bytes = g->owned.bytes;
  note_use(*g, st);  // (and the base, whose U the build read)
  return g.release();
}

// Length of a task from its (first probe | end << 32) value: its probes, or
// its units if its row is a short one.
struct TaskLenLoad {
  const uint64_t* val;
  const uint32_t* row;
  int64_t b16;
  __device__ uint64_t operator()(int64_t t) const {
    const uint64_t v = val[t];
    const uint32_t first = (uint32_t)v, end = (uint32_t)(v >> 32);
    return (int64_t)row[t] >= b16 ? short_units(first, end) : end - first;
  }
};

// Probe prefixes and row pointers of the tasks in tl.row / tl.val (tl.T of
// them, sorted by row; tl.ptr allocated with nrows + 1 entries).
void finish_tasks(TaskLists& tl, int64_t nrows, int64_t b16, hipStream_t st) {
  const int64_t T = tl.T;
  if (T == 0) {
    TC_LAUNCH("fill_i64", k_fill_i64, dim3(grid_for(nrows + 1)), dim3(kT), 0, st, tl.ptr.as<int64_t>(),
              nrows + 1, (int64_t)0);
    return;
  }
  tl.prefix.alloc(sizeof(uint64_t) * (size_t)(T + 1));
  device_excl_scan_f<uint64_t>(TaskLenLoad{tl.val.as<uint64_t>(), tl.row.as<uint32_t>(), b16},
                               tl.prefix.as<uint64_t>(), T, tl.prefix.as<uint64_t>() + T, st);
  TC_LAUNCH("bounds", (k_bounds<uint32_t>), dim3(grid_for(nrows + 1)), dim3(kT), 0, st,
            tl.row.as<uint32_t>(), T, 0, nrows, tl.ptr.as<int64_t>());
  TC_HIP(hipGetLastError());
}

void sort_tasks(TaskLists& tl, DevBuf& tk, DevBuf& tv, int64_t T, int64_t nrows, int key_bits, int64_t b16,
                hipStream_t st, const char* name) {
  tl.T = T;
  tl.ptr.alloc(sizeof(int64_t) * (size_t)(nrows + 1));
  if (T > 0) {
    tl.row.alloc(sizeof(uint32_t) * (size_t)T);
    tl.val.alloc(sizeof(uint64_t) * (size_t)T);
    const bool alt = radix_sort<uint32_t, uint64_t>(tk.as<uint32_t>(), tl.row.as<uint32_t>(),
                                                    tv.as<uint64_t>(), tl.val.as<uint64_t>(), T, 0, key_bits, st,
                                                    name);
    if (!alt) {  // sorted data ended in the input buffers: take them over
      tl.row.swap(tk);
      tl.val.swap(tv);
    }
  }
  finish_tasks(tl, nrows, b16, st);
}

namespace {

// Bundles of class c's short rows (cw16: their weight), whose items are there.
void make_bundles(WorkSet& w, Owned& own, int c, uint64_t cw16, hipStream_t st) {
  const int64_t groups = (w.n_items[c] - w.n_items32[c]) / kWaves;
  if (groups == 0) return;
  const uint64_t per = w.bundle_w / 2;  // units
  w.n_bundles[c] = div_up((int64_t)(cw16 / 2), (int64_t)per);
  w.bundle[c] = own.alloc<uint32_t>(w.n_bundles[c] + 1);
  TC_LAUNCH("bundles", k_bundles, dim3(grid_for(groups)), dim3(kT), 0, st, w.items[c] + w.n_items32[c], groups, per,
            w.n_bundles[c], w.bundle[c]);
  TC_HIP(hipGetLastError());
}

// The rest of build_work for at most kSmallN rows (k_small_order).
void build_work_small(WorkSet& w, Owned& own, int64_t n, const int64_t* hrow_ptr, int64_t T, const uint32_t* tb_row,
                      const int64_t* tb_ptr, const uint64_t* tb_val, const uint64_t* tb_prefix, hipStream_t st,
                      const int8_t* cls, unsigned long long* d_cp, const unsigned long long* d_cw, const int* d_cl) {
  uint32_t* crow = reinterpret_cast<uint32_t*>(own.alloc<int32_t>(n));
  uint32_t* pack_ptr[2] = {own.alloc<uint32_t>(n + 1), own.alloc<uint32_t>(n + 1)};
  DevBuf cm_pos(sizeof(uint32_t) * (size_t)n), wsc(sizeof(uint64_t) * (size_t)(n + 1));
  DevBuf usc(sizeof(uint32_t) * (size_t)(n + 1)), so(sizeof(SmallOrder)), rec(sizeof(RowRec) * (size_t)n);
  TC_LAUNCH("small_order", k_small_order, dim3(1), dim3(kSmallThreads), 0, st, (int)n, cls, tb_ptr, tb_prefix,
            hrow_ptr, w.b16, w.wp, d_cw, d_cw + NUM_CLASSES, d_cl, crow, w.tbeg, w.tend, cm_pos.as<uint32_t>(),
            wsc.as<uint64_t>(), usc.as<uint32_t>(), pack_ptr[0], pack_ptr[1], rec.as<RowRec>(), so.as<SmallOrder>());
  TC_LAUNCH("task_permute", k_task_permute, dim3((unsigned)div_up(T, kT * kPermuteTasks)), dim3(kT), 0, st, T,
            tb_row, tb_ptr, tb_val, tb_prefix, cls, w.tbeg, cm_pos.as<uint32_t>(), wsc.as<uint64_t>(), w.tstart,
            w.tprefix, d_cp);
  TC_HIP(hipGetLastError());
  TC_HIP(hipMemcpyAsync(w.tprefix + T, tb_prefix + T, sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
  SmallOrder h;
  TC_HIP(hipMemcpyAsync(&h, so.p, sizeof(h), hipMemcpyDeviceToHost, st));
  TC_HIP(hipMemcpyAsync(w.cls_probes, d_cp, sizeof(w.cls_probes), hipMemcpyDeviceToHost, st));
  TC_HIP(hipStreamSynchronize(st));
  TC_REQUIRE((int64_t)h.cb.tasks == T && h.cb.row[NUM_CLASSES] > 0, TC_EDEVICE,
             "build_work: class-major task order lost tasks");
  w.bundle_w = h.bundle_w;
  for (int c = 0; c < NUM_CLASSES; ++c) {
    for (int j = 0; j < 3; ++j) w.cls_stats[c][j] = (int64_t)h.stats[c][j];
    w.cls_log2S[c] = h.cl[c];
    w.cls_chunk[c] = h.chunk[c];
    const int64_t r0 = h.cb.row[c], nr = h.cb.row[c + 1] - r0;
    if (nr == 0) continue;
    if (c <= CLS_PACK_LARGE) {
      const int64_t np = h.cb.packs[c];
      w.pack_rows[c] = reinterpret_cast<int32_t*>(crow + r0);
      w.pack_ptr[c] = pack_ptr[c];
      w.pack_recs[c] = own.alloc<PackRow>(nr);
      w.pack_info[c] = own.alloc<PackInfo>(np);
      TC_LAUNCH("pack_recs", k_pack_recs, dim3(grid_for(nr)), dim3(kT), 0, st, w.pack_rows[c], nr, hrow_ptr, w.tbeg,
                w.tend, w.pack_recs[c]);
      TC_LAUNCH("pack_info", k_pack_info, dim3(grid_for(np * kPackWavesMax)), dim3(kT), 0, st, pack_ptr[c], np,
                w.pack_recs[c], w.tprefix, w.pack_info[c]);
      w.n_pack_rows[c] = nr;
      w.n_packs[c] = np;
      w.n_packs32[c] = h.cb.packs32[c];
      w.pack_log2S[c] = h.cl[c];
    } else {
      const int64_t total = (int64_t)h.cb.item[c + 1] - (int64_t)h.cb.item[c];
      if (total == 0) continue;
      w.items[c] = own.alloc<CountItem>(total);
      w.n_items[c] = total;
      w.n_items32[c] = (int64_t)h.cb.item16[c] - (int64_t)h.cb.item[c];
      TC_LAUNCH("emit_items", k_emit_items, dim3(grid_for(total)), dim3(kT), 0, st, usc.as<uint32_t>() + r0,
                crow + r0, nr, total, w.tbeg, w.tend, w.tprefix, hrow_ptr, w.items[c]);
      make_bundles(w, own, c, h.cw16[c], st);
    }
    TC_HIP(hipGetLastError());
  }
}

}  // namespace

void build_work(WorkSet& w, Owned& own, int64_t n, const int64_t* hrow_ptr, int64_t T,
                const uint32_t* tb_row, const int64_t* tb_ptr, const uint64_t* tb_val,
                const uint64_t* tb_prefix, int64_t b16, const WorkParams& wp, hipStream_t st, bool all_rows) {
  w.nrows = n;
  w.wp = wp;
  w.b16 = b16;
  w.n_tasks = T;
  w.tbeg = own.alloc<uint32_t>(n);
  w.tend = own.alloc<uint32_t>(n);
  w.tstart = own.alloc<uint32_t>(T);
  w.tprefix = own.alloc<uint64_t>(T + 1);
  DevBuf dscal(64);
  uint32_t* d_tot32 = dscal.as<uint32_t>();
  uint64_t* d_tot64 = reinterpret_cast<uint64_t*>(dscal.as<char>() + 32);
  const bool small = T > 0 && n <= kSmallN;
  if (!small) {
    // rows without tasks keep the empty range [0, 0)
    TC_LAUNCH("fill_u32", k_fill_u32, dim3(grid_for(n)), dim3(kT), 0, st, w.tbeg, n, 0u);
    TC_LAUNCH("fill_u32", k_fill_u32, dim3(grid_for(n)), dim3(kT), 0, st, w.tend, n, 0u);
  }
  if (T == 0) {
    TC_HIP(hipMemsetAsync(w.tprefix, 0, sizeof(uint64_t), st));
    w.probes = 0;
    return;
  }
  DevBuf cls(sizeof(int8_t) * (size_t)n);
  // per class: weight and probes (64-bit counters first: 8-byte aligned for
  // their atomics), then the largest table (log2 slots)
  DevBuf clsl(sizeof(unsigned long long) * 3 * NUM_CLASSES + sizeof(int) * NUM_CLASSES);
  TC_HIP(hipMemsetAsync(clsl.p, 0, clsl.bytes, st));
  unsigned long long* d_cp = clsl.as<unsigned long long>();  // probes (k_task_permute)
  unsigned long long* d_cw = d_cp + NUM_CLASSES;
  int* d_cl = reinterpret_cast<int*>(d_cw + 2 * NUM_CLASSES);
  TC_LAUNCH("classify", k_classify, dim3(grid_reduce(n)), dim3(kT), 0, st, tb_ptr, tb_prefix, hrow_ptr, n,
            all_rows, wp.heavy_min, std::min(wp.heavy_min, kShortHeavyMin), b16, cls.as<int8_t>(), d_cl, d_cw);
  TC_HIP(hipGetLastError());
  if (small) {
    build_work_small(w, own, n, hrow_ptr, T, tb_row, tb_ptr, tb_val, tb_prefix, st, cls.as<int8_t>(), d_cp, d_cw,
                     d_cl);
    return;
  }
  struct {
    unsigned long long cw[NUM_CLASSES], cw16[NUM_CLASSES];
    int cl[NUM_CLASSES];
  } hc;
  TC_HIP(hipMemcpyAsync(&hc, d_cw, sizeof(unsigned long long) * 2 * NUM_CLASSES + sizeof(int) * NUM_CLASSES,
                        hipMemcpyDeviceToHost, st));
  const unsigned long long* h_cw = hc.cw;
  const int* h_cl = hc.cl;

  // class-major row order: the rows of class 0 (ascending b), then class 1,
  // ...; each row keeps its tasks in b order, so every class - and every pack
  // of consecutive rows of a class - owns one contiguous task range
  DevBuf ckey, crow_in;
  WorkRowPred rowp{cls.as<int8_t>(), nullptr, nullptr};
  const int64_t R = compact("work_rows", n, rowp, [&](int64_t total, WorkRowPred& p) {
    ckey.alloc(sizeof(uint32_t) * (size_t)total);
    crow_in.alloc(sizeof(uint32_t) * (size_t)total);
    p.key = ckey.as<uint32_t>();
    p.row = crow_in.as<uint32_t>();
  }, st);
  TC_REQUIRE(R > 0, TC_EDEVICE, "build_work: tasks but no row with work");
  uint32_t* crow = reinterpret_cast<uint32_t*>(own.alloc<int32_t>(R));  // pack classes keep their rows
  {
    DevBuf ckey2(sizeof(uint32_t) * (size_t)R);
    const bool alt = radix_sort<uint32_t, uint32_t>(ckey.as<uint32_t>(), ckey2.as<uint32_t>(),
                                                    crow_in.as<uint32_t>(), crow, R, 0, 3, st, "classes");
    if (!alt) TC_HIP(hipMemcpyAsync(crow, crow_in.p, sizeof(uint32_t) * (size_t)R, hipMemcpyDeviceToDevice, st));
    const uint32_t* skey = alt ? ckey2.as<uint32_t>() : ckey.as<uint32_t>();
    DevBuf cptr(sizeof(int64_t) * (NUM_CLASSES + 1));
    TC_LAUNCH("bounds", (k_bounds<uint32_t>), dim3(1), dim3(kT), 0, st, skey, R, 0, (int64_t)NUM_CLASSES,
              cptr.as<int64_t>());
    // per class-major row: exclusive prefixes of tasks, probes and items
    DevBuf tsc(sizeof(uint32_t) * (size_t)(R + 1)), wsc(sizeof(uint64_t) * (size_t)(R + 1));
    DevBuf usc(sizeof(uint32_t) * (size_t)(R + 1));
    device_excl_scan_f<uint32_t>(CmTasks{crow, tb_ptr}, tsc.as<uint32_t>(), R, tsc.as<uint32_t>() + R, st);
    device_excl_scan_f<uint64_t>(CmProbes{crow, tb_ptr, tb_prefix}, wsc.as<uint64_t>(), R,
                                 wsc.as<uint64_t>() + R, st);
    // probes per wave item of each item class: wp.wave_chunk, smaller for a
    // class that would otherwise get fewer than wp.min_groups work-groups,
    // provided it has the probes to fill them with items of kWaveChunkMin (a
    // class too small for that stays at wp.wave_chunk: few, large units suit
    // a batch of many small graphs). h_cw is valid: compact synchronised st.
    CmItems cmi{crow, cls.as<int8_t>(), tb_ptr, tb_prefix, b16, 0, {}};
    // Short rows: bundles of groups of about equal weight (k_bundles), enough
    // of them to fill the GPU several times, and items that cut a heavy row
    // at that weight.
    uint64_t cw16 = 0;
    for (int c = CLS_WG_SMALL; c < NUM_CLASSES; ++c) cw16 += hc.cw16[c];
    const uint64_t bundle_w = w.bundle_w = bundle_weight(cw16);
    cmi.chunk16 = (uint32_t)std::min<uint64_t>(wp.wave_chunk, bundle_w / kWaves);
    for (int c = 0; c < NUM_CLASSES; ++c) w.cls_chunk[c] = cmi.chunk[c] = class_chunk(h_cw[c], c, wp);
    device_excl_scan_f<uint32_t>(cmi, usc.as<uint32_t>(), R,
                                 usc.as<uint32_t>() + R, st);
    DevBuf cm_pos(sizeof(uint32_t) * (size_t)n);
    TC_LAUNCH("cm_place", k_cm_place, dim3(grid_for(R)), dim3(kT), 0, st, crow, R, tsc.as<uint32_t>(), w.tbeg,
              w.tend, cm_pos.as<uint32_t>());
    TC_LAUNCH("task_permute", k_task_permute, dim3((unsigned)div_up(T, kT * kPermuteTasks)), dim3(kT), 0, st, T,
              tb_row, tb_ptr, tb_val, tb_prefix, cls.as<int8_t>(), w.tbeg, cm_pos.as<uint32_t>(),
              wsc.as<uint64_t>(), w.tstart, w.tprefix, d_cp);
    TC_HIP(hipMemcpyAsync(w.tprefix + T, tb_prefix + T, sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    // class boundaries, where each class's short rows begin, and the item
    // offsets there
    DevBuf cb(sizeof(ClassBounds));
    TC_LAUNCH("class_bounds", k_class_bounds, dim3(1), dim3(64), 0, st, crow, R, cptr.as<int64_t>(),
              usc.as<uint32_t>(), tsc.as<uint32_t>(), b16, cb.as<ClassBounds>());
    ClassBounds h;
    TC_HIP(hipMemcpyAsync(&h, cb.p, offsetof(ClassBounds, packs), hipMemcpyDeviceToHost, st));
    TC_HIP(hipStreamSynchronize(st));
    const int64_t* h_cp = h.row;
    TC_REQUIRE((int64_t)h.tasks == T && h_cp[NUM_CLASSES] == R, TC_EDEVICE,
               "build_work: class-major task order lost tasks");
    TC_HIP(hipGetLastError());

    // packs of the two pack classes: flags for both, one host sync for both
    // pack counts, then the pack pointers
    DevBuf pf[2], pp[2];
    for (int c = CLS_PACK_SMALL; c <= CLS_PACK_LARGE; ++c) {
      const int64_t r0 = h_cp[c], total = h_cp[c + 1] - h_cp[c];
      if (total == 0) continue;
      int32_t* rows = reinterpret_cast<int32_t*>(crow + r0);
      DevBuf wk(sizeof(uint64_t) * (size_t)total), pw(sizeof(uint64_t) * (size_t)total);
      DevBuf sl(sizeof(uint32_t) * (size_t)total), psl(sizeof(uint32_t) * (size_t)total);
      TC_LAUNCH("rows_work", k_rows_work, dim3(grid_for(total)), dim3(kT), 0, st, rows, total, w.tbeg,
                w.tend, w.tprefix, hrow_ptr, b16, wk.as<uint64_t>(), sl.as<uint32_t>());
      device_excl_scan<uint64_t, uint64_t>(wk.as<uint64_t>(), pw.as<uint64_t>(), total, d_tot64, st);
      device_excl_scan<uint32_t, uint32_t>(sl.as<uint32_t>(), psl.as<uint32_t>(), total, d_tot32, st);
      pf[c].alloc(sizeof(uint32_t) * (size_t)total);
      pp[c].alloc(sizeof(uint32_t) * (size_t)total);
      TC_LAUNCH("pack_flags", k_pack_flags, dim3(grid_for(total)), dim3(kT), 0, st, pw.as<uint64_t>(),
                psl.as<uint32_t>(), total, h.row16[c] - r0, wp.pack_target, wp.pack_slots,
                short_pack_slots(wp.pack_slots), pf[c].as<uint32_t>());
      device_excl_scan<uint32_t, uint32_t>(pf[c].as<uint32_t>(), pp[c].as<uint32_t>(), total, nullptr, st);
      TC_LAUNCH("pack_totals", k_pack_totals, dim3(1), dim3(1), 0, st, pf[c].as<uint32_t>(), pp[c].as<uint32_t>(),
                total, h.row16[c] - r0, c, cb.as<ClassBounds>());
    }
    if (h_cp[CLS_PACK_LARGE + 1] > h_cp[CLS_PACK_SMALL]) {
      TC_HIP(hipMemcpyAsync(h.packs, cb.as<ClassBounds>()->packs, sizeof(h.packs) + sizeof(h.packs32),
                            hipMemcpyDeviceToHost, st));
      TC_HIP(hipStreamSynchronize(st));
    }
    for (int c = 0; c < NUM_CLASSES; ++c) {
      w.cls_log2S[c] = h_cl[c];
      const int64_t r0 = h_cp[c], nr = h_cp[c + 1] - h_cp[c];
      if (nr == 0) continue;
      if (c == CLS_PACK_SMALL || c == CLS_PACK_LARGE) {
        const int64_t np = h.packs[c], np32 = h.packs32[c];
        uint32_t* pack_ptr = own.alloc<uint32_t>(np + 1);
        TC_LAUNCH("pack_emit", k_pack_emit, dim3(grid_for(nr)), dim3(kT), 0, st, pf[c].as<uint32_t>(),
                  pp[c].as<uint32_t>(), nr, pack_ptr, np);
        TC_HIP(hipGetLastError());
        w.pack_rows[c] = reinterpret_cast<int32_t*>(crow + r0);
        w.pack_ptr[c] = pack_ptr;
        w.pack_recs[c] = own.alloc<PackRow>(nr);
        w.pack_info[c] = own.alloc<PackInfo>(np);
        TC_LAUNCH("pack_recs", k_pack_recs, dim3(grid_for(nr)), dim3(kT), 0, st, w.pack_rows[c], nr, hrow_ptr,
                  w.tbeg, w.tend, w.pack_recs[c]);
        if (np < kPackLptMin) {
          // few packs (a launch of one or two rounds): pack order
          TC_LAUNCH("pack_info", k_pack_info, dim3(grid_for(np * kPackWavesMax)), dim3(kT), 0, st, pack_ptr, np, w.pack_recs[c],
                    w.tprefix, w.pack_info[c]);
        } else {
          // the class's packs in launch order: heaviest first
          DevBuf raw(sizeof(PackInfo) * (size_t)np);
          DevBuf key(sizeof(uint32_t) * (size_t)np), key2(sizeof(uint32_t) * (size_t)np);
          DevBuf idx(sizeof(uint32_t) * (size_t)np), idx2(sizeof(uint32_t) * (size_t)np);
          TC_LAUNCH("pack_info", k_pack_info, dim3(grid_for(np * kPackWavesMax)), dim3(kT), 0, st, pack_ptr, np, w.pack_recs[c],
                    w.tprefix, raw.as<PackInfo>());
          TC_LAUNCH("pack_keys", k_pack_keys, dim3(grid_for(np)), dim3(kT), 0, st, raw.as<PackInfo>(), np, np32,
                    key.as<uint32_t>(), idx.as<uint32_t>());
          const bool alt = radix_sort<uint32_t, uint32_t>(key.as<uint32_t>(), key2.as<uint32_t>(), idx.as<uint32_t>(),
                                                          idx2.as<uint32_t>(), np, 0, kPackKeyBits, st, "pack_lpt");
          TC_LAUNCH("pack_gather", k_pack_gather, dim3(grid_for(np)), dim3(kT), 0, st, raw.as<PackInfo>(),
                    alt ? idx2.as<uint32_t>() : idx.as<uint32_t>(), np, w.pack_info[c]);
        }
        TC_HIP(hipGetLastError());
        w.n_pack_rows[c] = nr;
        w.n_packs[c] = np;
        w.n_packs32[c] = np32;
        w.pack_log2S[c] = h_cl[c];
      } else {
        const int64_t total = (int64_t)h.item[c + 1] - (int64_t)h.item[c];
        if (total == 0) continue;
        CountItem* items = own.alloc<CountItem>(total);
        TC_LAUNCH("emit_items", k_emit_items, dim3(grid_for(total)), dim3(kT), 0, st, usc.as<uint32_t>() + r0,
                  crow + r0, nr, total, w.tbeg, w.tend, w.tprefix, hrow_ptr, items);
        TC_HIP(hipGetLastError());
        w.items[c] = items;
        w.n_items[c] = total;
        w.n_items32[c] = (int64_t)h.item16[c] - (int64_t)h.item[c];
        make_bundles(w, own, c, hc.cw16[c], st);
      }
    }
  }
  {
    const int64_t nb = (int64_t)grid_reduce(n);
    DevBuf part(sizeof(unsigned long long) * (size_t)nb * kStatCols);
    DevBuf sums(sizeof(unsigned long long) * kStatCols);
    TC_LAUNCH("class_stats", k_class_stats, dim3((unsigned)nb), dim3(kT), 0, st, cls.as<int8_t>(), n,
              w.tbeg, w.tend, hrow_ptr, part.as<unsigned long long>());
    TC_LAUNCH("reduce_cols", k_reduce_cols, dim3(kStatCols), dim3(kT), 0, st,
              part.as<unsigned long long>(), nb, kStatCols, sums.as<unsigned long long>());
    TC_HIP(hipGetLastError());
    // (valid once st is synchronised: every caller checks its sorts next)
    TC_HIP(hipMemcpyAsync(&w.cls_stats[0][0], sums.p, sizeof(w.cls_stats), hipMemcpyDeviceToHost, st));
    TC_HIP(hipMemcpyAsync(w.cls_probes, d_cp, sizeof(w.cls_probes), hipMemcpyDeviceToHost, st));
  }
}

void finish_work(WorkSet& w) {
  w.probes = 0;
  for (int c = 0; c < NUM_CLASSES; ++c) {
    w.cls_stats[c][3] = (int64_t)w.cls_probes[c];
    w.probes += w.cls_stats[c][3];
  }
}

}  // namespace tc

extern "C" tc_status tc_graph_variant(const tc_graph* gh, int32_t flags, void* stream, tc_graph** out) {
  try {
    TC_REQUIRE(out != nullptr, TC_EINVAL, "tc_graph_variant: out is NULL");
    *out = nullptr;
    TC_REQUIRE(gh != nullptr, TC_EINVAL, "tc_graph_variant: null graph");
    TC_REQUIRE((flags & ~(TC_VARIANT_IJK | TC_VARIANT_NO_DCSR | TC_VARIANT_MUL_HASH)) == 0, TC_EINVAL,
               "tc_graph_variant: unknown flags");
    const tc::Graph& base = *tc::G(gh);
    tc::require_plain(base, "tc_graph_variant");
    tc::Graph* g = tc::build_variant(base, flags, base.w.wp, static_cast<hipStream_t>(stream));
    *out = reinterpret_cast<tc_graph*>(g);
    tc::set_last_error("");
    return TC_OK;
  } catch (const tc::Error& e) {
    tc::set_last_error(e.what());
    return e.status;
  } catch (const std::bad_alloc&) {
    tc::set_last_error("tc_graph_variant: host allocation failed");
    return TC_ENOMEM;
  } catch (const std::exception& e) {
    tc::set_last_error(e.what());
    return TC_EDEVICE;
  }
}

extern "C" tc_status tc_preprocess(const int32_t* d_src, const int32_t* d_dst, int64_t m_raw,
                                   int32_t n, void* stream, tc_graph** out) {
  try {
    TC_REQUIRE(out != nullptr, TC_EINVAL, "tc_preprocess: out is NULL");
    *out = nullptr;
    TC_REQUIRE(n >= 1, TC_EINVAL, "tc_preprocess: n must be >= 1");
    TC_REQUIRE(m_raw >= 0, TC_EINVAL, "tc_preprocess: m_raw must be >= 0");
    TC_REQUIRE(m_raw == 0 || (d_src != nullptr && d_dst != nullptr), TC_EINVAL,
               "tc_preprocess: null edge arrays");
    TC_REQUIRE(m_raw < (int64_t)0xFFFFFFFFLL, TC_EOVERFLOW, "tc_preprocess: m_raw >= 2^32 - 1");
    tc::Graph* g = tc::build_graph(d_src, d_dst, m_raw, n, static_cast<hipStream_t>(stream));
    *out = reinterpret_cast<tc_graph*>(g);
    tc::set_last_error("");
    return TC_OK;
  } catch (const tc::Error& e) {
    tc::set_last_error(e.what());
    return e.status;
  } catch (const std::bad_alloc&) {
    tc::set_last_error("tc_preprocess: host allocation failed");
    return TC_ENOMEM;
  } catch (const std::exception& e) {
    tc::set_last_error(e.what());
    return TC_EDEVICE;
  }
}
