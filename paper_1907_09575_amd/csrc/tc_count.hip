// tc_count.hip - the map-based intersection of Section 3.1 (<j,i,k> order) and
// its reductions: exact triangle count (Eq. 2) and per-edge support (Eq. 1).
//
// Work unit. For a hashed row b, a task is a nonzero (a, b) of U (a in L_b,
// the column of b); it probes the entries of U_a after b - all of them exceed
// b, which is Eq. 1's k > j bound - against a hash of U_b. A hit is a
// triangle a < b < k. The probes of all tasks of one b form one contiguous
// range of the global probe index space (tasks grouped by b, prefix-summed by
// preprocessing).
//
// Hash table (Section 5.2's change to the hashing routine): U_b in LDS in
// buckets of four 32-bit slots, bucket = k & (buckets - 1) (the direct bitwise
// AND of the paper), at least 4 |U_b| slots (2 |U_b| for rows of more than
// 2048 keys). A key goes to the first free slot of its bucket or, if the
// bucket is full, of the next ones; slots fill left to right, so a lookup
// reads one bucket with a single 16-byte LDS read and stops there unless the
// bucket is full. The build records the longest bucket displacement D, which
// bounds every lookup; exactness never depends on the absence of collisions.
//
// Probe loop (one wave, flattened over tasks). A wave walks a range of
// probes in batches of 64, lane l taking probe base + l, so every col[] read
// is a coalesced run; kU batches form a super-batch whose loads and lookups
// are all in flight together. A window of 64 consecutive tasks sits one per
// lane (end of the task relative to the wave's position, and the col index its
// probes start from); the next window is prefetched while the current one is
// probed. The task of a probe r is c0 (tasks ended at or before the
// super-batch start, one ballot) plus the number of task ends inside the
// super-batch that lie at or before r: ends set bits of a per-wave LDS bitmap,
// whose words are read back as wave-uniform masks and counted per lane with
// mbcnt. The task's col base then comes from its lane by one bpermute.
// Probe reads are raw buffer loads with a 32-bit byte offset; a lane past the
// range gets an offset beyond the buffer and reads 0, which is never a key of
// U_b (every key exceeds b >= 0), so it needs no branch.
//
// Launch classes (decided in preprocessing from |U_b| and the row's probes):
//   packs  - light rows b are packed (up to 256 rows per work-group); the
//            work-group builds all their tables in LDS, then its waves probe
//            the pack's task range, each task looking up its own row's table.
//   heavy  - a row's probes are cut into per-wave ranges (16K probes); the 4
//            waves of a work-group share one table of that row. One launch per
//            table size class (wg_small / wg_large / wg_huge / wg_giant), each
//            compiled for the occupancy its LDS allows.
//   global - a row whose table would not fit LDS (|U_b| > 8192): lookups are
//            binary searches in the sorted U_b in HBM.
// Short rows (b >= b16, see kShortSpan) of the same classes are launched apart:
// their probes are read from the 16-bit columns, two per load, and looked up
//   - in a bitmap over the column distances n - k (item classes, global
//     included): one 4-byte LDS read and a bit extract per probe, no
//     collisions, at most 8 KiB for a row of any length;
//   - in buckets of four 16-bit slots (packs): one 8-byte LDS read.
// The 32-bit kernels are bound by HBM at 4 bytes per probe; these move half
// of that and are bound by vector issue (about 8 instructions per probe and
// lane of which half is the lookup). tc_count, RMAT: scale 20 1215 -> 645 us,
// scale 22 5427 -> 3300 us, scale 24 29.9 -> 19.1 ms, scale 14
// (n = 16384, all rows short) 170 -> 57 us.
// Reductions: per-lane 32-bit hit counters, wave reduction by xor shuffles,
// one 64-bit atomic per work-group into the caller's counter (order-free and
// exact).
#include "tc_prims.h"

namespace tc {

namespace {

using Args = CountArgs;

constexpr int kU = 8;                   // 64-probe batches per super-batch
constexpr int kBmWords = 2 * kU;        // per-wave task-end bitmap (64 * kU bits)

// Modes that count the hits of every task, and those that count the hits of
// every key of U_b.
__host__ __device__ constexpr bool mode_tasks(int mode) {
  return mode == MODE_SUPPORT_FULL || mode == MODE_SUPPORT_ORIENTED || mode == MODE_VERTEX;
}
__host__ __device__ constexpr bool mode_keys(int mode) { return mode == MODE_SUPPORT_FULL || mode == MODE_VERTEX; }

// LDS words of one wave: its task-end bitmap and, in the support modes, the
// running hit count at the end of each of its window's tasks.
__host__ __device__ constexpr int wave_words(int mode) {
  return kBmWords + (mode_tasks(mode) ? 64 : 0);
}

constexpr int32_t kEmpty = -1;
// FULL support, single-row LDS tables: a slot's value word is the key's index
// in its row (< 2^13: such rows have at most 8192 keys) plus its hits in this
// work-group times 2^13 (at most one per task, and a work-group holds at most
// 8 wave items of at most 32767 probes: < 2^18, so the word stays below 2^31).
constexpr int kValBits = 13;
static_assert((1 << kValBits) >= (1 << kMaxLog2S) / 2, "row index of an LDS table below the hit count");
static_assert((uint64_t)kWavesBig * kWaveChunkMax < (1ull << (31 - kValBits)),
              "hits of one slot in one work-group keep the value word below 2^31");
constexpr uint32_t kOffNone = 0xFFFFFFF0u;  // byte offset past any col buffer

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t col_rsrc(const int32_t* col, uint32_t m) {
  // raw buffer over col[0, m): stride 0, num_records = bytes; reads at or past
  // the end return 0
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(col), (short)0, (int)(m * 4u),
                                           0x00020000);
}

__device__ __forceinline__ int32_t col_load(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0);
}

// Code variants of the count kernels (template argument VAR):
//   VAR_BASE  - the direct AND of Section 5.2; probes read by raw buffer loads
//               with 32-bit byte offsets (probe sides of fewer than 2^30
//               entries);
//   VAR_MUL   - the ablation of the direct AND (tc_graph_variant): a
//               multiplicative hash for every table;
//   VAR_WIDE  - probe sides of 2^30 entries or more: probes read with 64-bit
//               addresses (positions stay 32-bit), masked for lanes past the
//               range.
enum CountVariant : int { VAR_BASE = 0, VAR_MUL = 1, VAR_WIDE = 2 };

// Bucket of key k in a table of bmask + 1 buckets: the direct bitwise AND of
// Section 5.2 (the key's low bits), or, MH (the ablation of that choice,
// tc_graph_variant), a multiplicative hash: the top log2(buckets) bits of
// k times 2^32 / golden ratio.
template <bool MH>
__device__ __forceinline__ uint32_t bucket_of(int32_t k, uint32_t bmask) {
  if constexpr (!MH) {
    return (uint32_t)k & bmask;
  } else {
    const uint32_t B = (uint32_t)__popc(bmask);
    return (uint32_t)(((uint64_t)((uint32_t)k * 0x9E3779B1u) << B) >> 32);
  }
}

// Lookup by binary search in the sorted row col[rs, rs + d); returns the
// position of k or -1.
__device__ __forceinline__ int64_t hbm_find(const int32_t* __restrict__ col, int64_t rs, int64_t d,
                                            int32_t k) {
  int64_t lo = rs, hi = rs + d;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    int32_t v = col[mid];
    if (v < k) lo = mid + 1;
    else hi = mid;
  }
  return (lo < rs + d && col[lo] == k) ? lo : -1;
}

// Insert U_b = col[rs, rs + d) into a cleared bucketed table of (bmask + 1)
// buckets; threads tid, tid + nt, ... share the work. Returns this thread's
// longest bucket displacement. VALS: also store every key's index in the row
// (its U position is rs + index), with a zero hit count above it.
template <bool VALS, bool MH>
__device__ int build_table(int32_t* tab, int32_t* val, uint32_t bmask, const int32_t* __restrict__ col,
                           int64_t rs, int64_t d, int tid, int nt) {
  constexpr int kB = 8;  // keys fetched at once so that their loads overlap
  int md = 0;
  for (int64_t i0 = tid; i0 < d; i0 += (int64_t)kB * nt) {
    int32_t key[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      const int64_t i = i0 + (int64_t)j * nt;
      key[j] = i < d ? col[rs + i] : kEmpty;
    }
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      if (key[j] == kEmpty) continue;
      uint32_t bk = bucket_of<MH>(key[j], bmask);
      int disp = 0;
      int slot = -1;
      while (true) {
#pragma unroll
        for (int s = 0; s < kBucket; ++s) {
          if (slot < 0 && atomicCAS(&tab[bk * kBucket + s], kEmpty, key[j]) == kEmpty)
            slot = (int)(bk * kBucket + s);
        }
        if (slot >= 0) break;
        bk = (bk + 1) & bmask;
        ++disp;
      }
      if (VALS) val[slot] = (int32_t)(i0 + (int64_t)j * nt);
      md = disp > md ? disp : md;
    }
  }
  return md;
}

// FULL support in packs: a pack of fewer than 2^17 probes keeps its (b, k)
// credits in LDS, the slot's value word holding the key's index in the pack's
// key list (kPackValBits, below 2^15 since a pack has at most kPackSlotsMax
// plus 1024 slots) plus its hits shifted by kPackValBits (at most the pack's
// probes, so the word stays below 2^32); larger packs hold U positions and
// credit (b, k) per hit.
constexpr int kPackValBits = 15;
static_assert(kPackSlotsMax + 1024 <= (1u << kPackValBits), "a pack's key index fits its field");
constexpr uint64_t kPackLdsHitsMax = (uint64_t)1 << (32 - kPackValBits);

struct TableRef {
  const int32_t* tab;  // (bmask + 1) * kBucket slots (a pack: all its rows' tables)
  int32_t* val;        // FULL support: single-row tables hold row index | hits <<
                       // kValBits, packs key index | hits << kPackValBits (both
                       // summed in LDS) or, in packs of 2^17 probes or more, U
                       // positions
  uint32_t bmask;
  int D;
  int64_t rs, d;  // the row itself (HBM fallback)
  // packs: row i of the pack owns tasks [row_t0[i], row_t0[i + 1]) and the
  // table at bucket (desc & 0xFFFF) with (desc >> 16) + 1 buckets
  const uint32_t* row_t0;
  const uint32_t* row_desc;
  int nrows;
  int lds_hits;  // packs, FULL: the (b, k) credits are counted in LDS
  uint32_t* row_hits;  // packs, VERTEX: hits of every row
  // bitmaps, FULL: keys of smaller distance than each word's (pfx), hits per
  // key in order of distance (cnt; null: credited to U directly)
  const uint16_t* pfx;
  uint32_t* cnt;
};

// Short rows: TK_MULTI16 (packs), TK_BITS (bitmap), TK_GLOBAL16 (HBM).
enum TableKind : int { TK_SINGLE = 0, TK_MULTI = 1, TK_GLOBAL = 2, TK_MULTI16 = 3, TK_BITS = 4, TK_GLOBAL16 = 5 };
// Batches per super-batch of a kind: a window (64 tasks) holds about half as
// many units as probes, so the short rows' kinds take half; a batch beyond
// the window's end costs as much as a full one (ER, n = 30000, 400000 pairs:
// 58 us with 8, 43 us with 4).
constexpr int kPacks16U = 4, kBitsU = 4;
constexpr int kind_batches(int kind) { return kind == TK_MULTI16 ? kPacks16U : kind == TK_BITS ? kBitsU : kU; }
constexpr uint32_t kEmpty16 = 0xFFFFu;  // empty 16-bit slot: above every distance (kShortSpan)

// A hit: k = col[pos] was found in U_b at `where` (an LDS slot, or for the HBM
// fallback its position in col); ts is the first probe position of the task,
// so ts - 1 is the U entry of the task's own edge (a, b).
// Per-shift triangle counters of one work-group (MODE_BLOCK).
__device__ unsigned int* shift_counters() {
  __shared__ unsigned int s_shift[64];
  return s_shift;
}

// VERTEX: c triangles at vertex v (a rank). The vertices of highest degree
// are keys of almost every row, and atomics to one address follow each other
// at 12 ns each: their counters exist kVertexCopies times, the work-group's
// number chooses one (clustering, RMAT scale 20: 2.54 -> 1.90 ms).
__device__ __forceinline__ void credit_vertex(const Args& A, uint32_t v, uint32_t c) {
  const uint32_t n = (uint32_t)A.n;
  if (v >= n) return;
  const uint32_t top = n - 1 - v, hot = vertex_hot(A.n);
  uint64_t at = v;
  if (top < hot) at = (uint64_t)n + (uint64_t)(blockIdx.x % kVertexCopies) * hot + top;
  atomicAdd(&A.vcount[at], (unsigned long long)c);
}

// The per-hit credits other than the task's own edge (a, b), which goes
// through the wave's per-task counters (wave_probe). VERTEX: like FULL for the
// keys k of U_b, whose hits go to the vertex k. BLOCK: the shift
// counter of k; FULL: the probed entry (a, k) of U_a and k's entry (b, k) of
// U_b.
template <int MODE, int KIND>
__device__ __forceinline__ void credit(const Args& A, const TableRef& t, int where, uint32_t pos, int32_t k) {
  // indices are checked against m so that no credit can leave the array
  if (MODE == MODE_BLOCK) {
    // shift z of Eq. 5 closes the triangle with k = x + y + z (mod q)
    int z = (int)((uint32_t)k % (uint32_t)A.q) - A.xy;
    if (z < 0) z += A.q;
    atomicAdd(&shift_counters()[z], 1u);
  } else if (mode_keys(MODE)) {
    if (MODE == MODE_SUPPORT_FULL && pos < A.m) atomicAdd(&A.support[pos], 1);  // edge (a, k): probed entry of U_a
    // edge (b, k): k's entry in U_b. A single-row table counts it in the
    // slot's LDS word (added to the array once per work-group, after the
    // probe loop of items_body).
    if (KIND == TK_SINGLE) {
      atomicAdd(&t.val[where], 1 << kValBits);
    } else if (KIND == TK_MULTI && t.lds_hits) {
      atomicAdd(reinterpret_cast<unsigned int*>(&t.val[where]), 1u << kPackValBits);
    } else if (MODE == MODE_VERTEX) {
      credit_vertex(A, (uint32_t)k, 1u);
    } else {
      const uint32_t other = (uint32_t)(KIND == TK_GLOBAL ? where : t.val[where]);
      if (other < A.m) atomicAdd(&A.support[other], 1);
    }
  }
}

// The (a, k) credits of a batch of units (FULL): lanes of hm hit with the
// first entry of their unit, lanes of hm1 with the second. A wave's units are
// runs of consecutive entries, so the credits are dealt to the lanes in entry
// order, 64 entries at a time: an atomic instruction then covers half the
// cache lines it would with every other entry per lane (RMAT scale 20, FULL:
// 6.19 ms with an atomic per half word, 4.48 ms so; one 8-byte atomic per unit
// touches the same lines: no faster).
__device__ __forceinline__ void credit_probed(const Args& A, uint32_t pos, uint64_t hm, uint64_t hm1) {
  const int lane = lane_id();
  const uint64_t mine = (lane & 1) ? hm1 : hm;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = 32 * h + (lane >> 1);
    const uint32_t p = 2 * (uint32_t)__builtin_amdgcn_ds_bpermute(j << 2, (int)pos) + (uint32_t)(lane & 1);
    if (((mine >> j) & 1ull) && p < A.m) atomicAdd(&A.support[p], 1);
  }
}

// A short row's hit (FULL) with a key of distance v of U_b: its (b, k) credit.
// `where` is the key's slot (packs), its bitmap word's contents (bitmaps) or
// its position in U (HBM).
template <int MODE, int KIND>
__device__ __forceinline__ void credit16(const Args& A, const TableRef& t, uint32_t where, uint32_t v) {
  if (KIND == TK_BITS) {
    // keys of smaller distance come after k in U_b
    const uint32_t r = (uint32_t)t.pfx[v >> 5] + (uint32_t)__builtin_popcount(where & ((1u << (v & 31)) - 1u));
    if (t.cnt) {
      atomicAdd(&t.cnt[r], 1u);
    } else if (MODE == MODE_VERTEX) {
      credit_vertex(A, (uint32_t)A.n - v, 1u);
    } else {
      const uint64_t p = (uint64_t)(t.rs + t.d - 1) - r;
      if (p < A.m) atomicAdd(&A.support[p], 1);
    }
  } else if (KIND == TK_MULTI16 && t.lds_hits) {
    atomicAdd(reinterpret_cast<unsigned int*>(&t.val[where]), 1u << kPackValBits);
  } else if (MODE == MODE_VERTEX) {
    credit_vertex(A, (uint32_t)A.n - v, 1u);
  } else {
    const uint32_t other = KIND == TK_GLOBAL16 ? where : (uint32_t)t.val[where];
    if (other < A.m) atomicAdd(&A.support[other], 1);
  }
}

// Support modes credit every hit to its task's own edge (a, b) through the
// task window. Along a window the wave keeps the number of its hits so far;
// the lane that holds a task's last probe (the end marks name it) notes the
// count there, inclusive, in the task's LDS word, and when the window is done
// lane j adds the difference of its task's word and the one before to the
// task's edge with one global atomic. A batch without a task end costs only
// its ballot and a scalar add. A task cut between waves gets one atomic from
// each. (kEndCounts; packs of 32-bit rows, whose windows are one super-batch of
// short tasks, mask every batch's ballot to the lanes of each task instead:
// oriented support of an ER graph, n = 10^6: 582 us against 625 us.)
__device__ __forceinline__ uint64_t lane_range_mask(int lo, int hi) {
  lo = lo < 0 ? 0 : (lo > 64 ? 64 : lo);
  hi = hi < 0 ? 0 : (hi > 64 ? 64 : hi);
  if (hi <= lo) return 0;
  const uint64_t below_hi = hi >= 64 ? ~0ull : ((1ull << hi) - 1ull);
  return below_hi & ~((1ull << lo) - 1ull);
}

// Count mode needs only whether the bucket holds k: an OR of four compares
// (no slot index, no branch).
__device__ __forceinline__ bool bucket_has(const int4& v, int32_t k) {
  return (v.x == k) | (v.y == k) | (v.z == k) | (v.w == k);
}

__device__ __forceinline__ int match_slot(const int4& v, int32_t k) {
  return v.x == k ? 0 : v.y == k ? 1 : v.z == k ? 2 : v.w == k ? 3 : -1;
}

// The same for a bucket of four 16-bit slots. Each half of x ^ vv is 0 where
// the slot holds v; the packed minimum with 1 leaves 0 there and 1 elsewhere.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_ne(uint32_t x, uint32_t vv) {
  const u16x2 one = {1, 1};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, x ^ vv), one));
}
__device__ __forceinline__ bool bucket16_has(const uint2& b, uint32_t vv) {
  const uint32_t e = pk_ne(b.x, vv) & pk_ne(b.y, vv);
  return (e & (e >> 16) & 1u) == 0;
}
__device__ __forceinline__ int match_slot16(const uint2& b, uint32_t v) {
  return (b.x & 0xFFFFu) == v ? 0 : (b.x >> 16) == v ? 1 : (b.y & 0xFFFFu) == v ? 2 : (b.y >> 16) == v ? 3 : -1;
}

// Lookups of a super-batch of units (short rows): w[u] holds this lane's two
// column distances of batch u; 0 is no key. Hits of
// the first and the second probe of batch u set bit u of f0 and f1 (support
// modes).
template <int MODE, int KIND, int U>
__device__ __forceinline__ void probe_units(const Args& A, const TableRef& tr, const int32_t (&w)[U],
                                            const uint32_t (&bbase)[U], const uint32_t (&bmask)[U],
                                            uint32_t& hits, uint32_t& f0, uint32_t& f1) {
  constexpr bool kMask = mode_tasks(MODE);
  constexpr bool FULL = mode_keys(MODE);
  if constexpr (KIND == TK_BITS) {
    const uint32_t* bits = reinterpret_cast<const uint32_t*>(tr.tab);
    uint32_t x0[U], x1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x0[u] = bits[((uint32_t)w[u] >> 5) & 0x7FFu];
      x1[u] = bits[(uint32_t)w[u] >> 21];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t b0 = __builtin_amdgcn_ubfe(x0[u], (uint32_t)w[u] & 31u, 1);
      const uint32_t b1 = __builtin_amdgcn_ubfe(x1[u], ((uint32_t)w[u] >> 16) & 31u, 1);
      hits += b0 + b1;
      if (kMask) {
        f0 |= b0 << u;
        f1 |= b1 << u;
      }
      if (FULL) {
        if (b0) credit16<MODE, KIND>(A, tr, x0[u], (uint32_t)w[u] & 0xFFFFu);
        if (b1) credit16<MODE, KIND>(A, tr, x1[u], (uint32_t)w[u] >> 16);
      }
    }
  } else if constexpr (KIND == TK_MULTI16) {
    const uint2* tab2 = reinterpret_cast<const uint2*>(tr.tab);
    constexpr int kG = 4;  // batches whose buckets are read together
#pragma unroll
    for (int g0 = 0; g0 < U; g0 += kG) {
      uint2 x[2 * kG];
#pragma unroll
      for (int u = g0; u < g0 + kG; ++u) {
        x[2 * (u - g0)] = tab2[bbase[u] + ((uint32_t)w[u] & bmask[u])];  // (a pack's tables: bmask < 2^16)
        x[2 * (u - g0) + 1] = tab2[bbase[u] + (((uint32_t)w[u] >> 16) & bmask[u])];
      }
#pragma unroll
      for (int u = g0; u < g0 + kG; ++u) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t v = h ? (uint32_t)w[u] >> 16 : (uint32_t)w[u] & 0xFFFFu;
          const uint32_t vv = v | (v << 16);
          uint2 b = x[2 * (u - g0) + h];
          bool found = bucket16_has(b, vv);
          uint32_t bk = v & bmask[u];
          // full first bucket: continue into the next ones (bounded by D)
          for (int i = 0; !found && (b.y >> 16) != kEmpty16 && i < tr.D; ++i) {
            bk = (bk + 1) & bmask[u];
            b = tab2[bbase[u] + bk];
            found = bucket16_has(b, vv);
          }
          hits += found ? 1u : 0u;
          if (kMask) (h ? f1 : f0) |= (found ? 1u : 0u) << u;
          if (FULL && found)
            credit16<MODE, KIND>(A, tr, (bbase[u] + bk) * kBucket + (uint32_t)match_slot16(b, v), v);
        }
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t v = h ? (uint32_t)w[u] >> 16 : (uint32_t)w[u] & 0xFFFFu;
        const int64_t where = v ? hbm_find(A.hcol, tr.rs, tr.d, A.n - (int32_t)v) : -1;
        if (where < 0) continue;
        ++hits;
        if (kMask) (h ? f1 : f0) |= 1u << u;
        if (FULL) credit16<MODE, KIND>(A, tr, (uint32_t)where, v);
      }
    }
  }
}

// The first window of a wave's probe range [q, q + len) (task t holds probe
// q): each lane's task end, relative to q and clamped to len, and first-probe
// position, and the window's own start. Loaded before the table is built, so
// that these loads overlap the build.
struct Window {
  uint32_t Pe, tsj, P0;
};

__device__ __forceinline__ Window window_first(const Args& A, uint32_t t, uint64_t q, uint32_t len) {
  const int lane = lane_id();
  const int64_t T = A.T;
  const int64_t tj = (int64_t)t + lane;
  const uint64_t p = A.tprefix[tj + 1 < T ? tj + 1 : T] - q;
  Window w;
  w.Pe = p > (uint64_t)len ? len : (uint32_t)p;
  w.tsj = A.tstart[tj < T ? tj : T - 1];
  w.P0 = (uint32_t)(A.tprefix[t] - q);  // may wrap (a task starting before q)
  return w;
}

// c hits of the task whose first probe is ts: to its own edge, or (VERTEX) to
// its row a and, in a pack, to its hashed row's counter.
template <int MODE, bool MULTI>
__device__ __forceinline__ void credit_task(const Args& A, const TableRef& tr, uint32_t ts, int row, uint32_t c) {
  if (ts - 1u >= A.m) return;
  if constexpr (MODE == MODE_VERTEX) {
    credit_vertex(A, A.erow[ts - 1u], c);
    if (MULTI) atomicAdd(&tr.row_hits[row], c);
  } else {
    atomicAdd(&A.support[ts - 1u], (int)c);
  }
}

// One wave processes the probes [q, q + len) of the tasks of one hashed row;
// task t contains probe q; w0 = window_first(A, t, q, len).
template <int MODE, int KIND, int VAR>
__device__ void wave_probe(const Args& A, const TableRef& tr, uint32_t t, uint64_t q, uint32_t len,
                           uint32_t* bm, uint32_t& hits, const Window& w0) {
  uint32_t* const tend = bm + kBmWords;  // support modes: hits up to each window task's end
  // the range is the wave's own (uniform across its lanes): scalar registers
  // (readfirstlane returns int: widen through uint32_t, never sign-extend)
  t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
  len = (uint32_t)__builtin_amdgcn_readfirstlane((int)len);
  q = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(q >> 32)) << 32) |
      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)q);
  constexpr bool GLOBAL = KIND == TK_GLOBAL;
  constexpr bool SHORT = KIND == TK_MULTI16 || KIND == TK_BITS || KIND == TK_GLOBAL16;  // probes are units
  constexpr bool MULTI = KIND == TK_MULTI || KIND == TK_MULTI16;
  constexpr bool MH = VAR == VAR_MUL, WIDE = VAR == VAR_WIDE && !SHORT;
  constexpr bool kTaskHits = mode_tasks(MODE);
  constexpr bool kEndCounts = kTaskHits && KIND != TK_MULTI;
  constexpr int U = kind_batches(KIND);
  constexpr uint32_t SB = 64u * U;
  const int lane = lane_id();
  const int64_t T = A.T;
  const __amdgpu_buffer_rsrc_t rsrc =
      SHORT ? col_rsrc(reinterpret_cast<const int32_t*>(A.col16), (A.m + 1) / 2) : col_rsrc(A.col, A.m);
  const int4* tab4 = reinterpret_cast<const int4*>(tr.tab);

  // window of tasks t .. t + 63, one per lane: end prefix and col start (the
  // start prefix of a task is the end prefix of the previous one). Prefixes
  // are kept relative to the range start q0 in 32 bits: ends are clamped to
  // len (a task ending past the range is cut there; the start of a task that
  // begins past the range is never used), and a start before q0 wraps.
  const uint64_t q0 = q;
  auto fetch = [&](int64_t tj, uint32_t& Pe, uint32_t& ts) {
    const uint64_t p = A.tprefix[tj + 1 < T ? tj + 1 : T] - q0;
    Pe = p > (uint64_t)len ? len : (uint32_t)p;
    ts = A.tstart[tj < T ? tj : T - 1];
  };
  uint32_t Pe = w0.Pe;
  uint32_t tsj = w0.tsj;
  uint32_t P0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)w0.P0);  // start of the window's first task

  uint32_t done = 0;
  while (done < len) {
    const uint32_t rem = len - done;
    // end of the lane's task relative to the current position, within the range
    const uint32_t e = Pe - done;
    // start of the lane's task relative to the current position (wraps below
    // it for lane 0 when the range begins inside its task), so cbase = col
    // index (short rows: unit) of relative probe 0
    const uint32_t e_prev = (uint32_t)__shfl_up((int)e, 1, 64);
    const uint32_t s_rel = lane == 0 ? P0 - done : e_prev;
    const uint32_t cbase = (SHORT ? tsj >> 1 : tsj) - s_rel;
    // probes of this window (wave-uniform: kept in a scalar register)
    const uint32_t lim = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)e, 63, 64));
    if (lim == 0) break;  // unreachable when every task has a probe; guards progress
    // packs: the table of the lane's task (last row whose first task <= it)
    uint32_t tdesc = 0;
    int trow = 0;
    if constexpr (MULTI) {
      const uint32_t tj = t + (uint32_t)lane;
      int lo = 0, hi = tr.nrows;  // row_t0[lo] <= tj (lanes past the pack clamp to the last row)
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tr.row_t0[mid] <= tj) lo = mid;
        else hi = mid;
      }
      tdesc = tr.row_desc[lo];
      trow = lo;
    }
    const bool more = lim < rem;
    uint32_t nPe = 0;
    uint32_t ntsj = 0;
    if (more) fetch((int64_t)t + 64 + lane, nPe, ntsj);  // next window, in flight meanwhile

    uint32_t run = 0;   // kEndCounts: the window's hits so far (uniform)
    uint32_t tcnt = 0;  // otherwise: hits of this lane's window task
    for (uint32_t sb = 0; sb < lim; sb += SB) {
      const uint32_t c0 = (uint32_t)__popcll(__ballot(e <= sb));
      const bool inner = e > sb && e <= sb + SB;
      uint32_t jl[U];
      uint64_t ends[U];  // kEndCounts: lanes of batch u that hold a task's last probe
      if (__ballot(inner) == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          jl[u] = c0;
          if (kEndCounts) ends[u] = 0;
        }
      } else {
        // bit p set <=> some task ends right after probe sb + p
        if (inner) atomicOr(&bm[(e - sb - 1) >> 5], 1u << ((e - sb - 1) & 31));
        wave_sync_lds();
        uint32_t pre = c0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t lo = __builtin_amdgcn_readfirstlane(bm[2 * u]);
          const uint32_t hi = __builtin_amdgcn_readfirstlane(bm[2 * u + 1]);
          jl[u] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, pre));
          pre += (uint32_t)__builtin_popcount(lo) + (uint32_t)__builtin_popcount(hi);
          if (kEndCounts) ends[u] = ((uint64_t)hi << 32) | lo;
        }
        wave_sync_lds();
        if (lane < (int)(SB / 32)) bm[lane] = 0;
        wave_sync_lds();
      }
      uint32_t pos[U], bbase[U], bmask[U];
      int32_t k[U];
      bool ok[U];
      uint32_t fmask = 0;  // support modes: bit u = this lane's probe of batch u hit
      uint32_t fmask1 = 0;  // short rows: its second probe (bits of fmask: the first)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // ds_bpermute uses lane index bits only, so lanes past the window
        // (jl >= 64, never used) wrap harmlessly
        const uint32_t r = sb + 64u * u + (uint32_t)lane;
        pos[u] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(jl[u] << 2), (int)cbase) + r;
        ok[u] = r < lim;
        if constexpr (MULTI) {
          const uint32_t dsc = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(jl[u] << 2), (int)tdesc);
          bbase[u] = dsc & 0xFFFFu;
          bmask[u] = dsc >> 16;
        } else {
          bbase[u] = 0;
          bmask[u] = tr.bmask;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if constexpr (WIDE) k[u] = ok[u] ? A.col[(uint64_t)pos[u]] : 0;
        else k[u] = col_load(rsrc, ok[u] ? pos[u] * 4u : kOffNone);
      }

      if constexpr (SHORT) {
        probe_units<MODE, KIND, U>(A, tr, k, bbase, bmask, hits, fmask, fmask1);
      } else if constexpr (!GLOBAL) {
        // buckets are read in groups of kG so that the 16-byte results of one
        // group fit the register budget of 8 waves per SIMD
        constexpr int kG = 2;
        uint32_t bk[U];
        bool unres[U];
        bool any_unres = false;
#pragma unroll
        for (int g0 = 0; g0 < U; g0 += kG) {
          int4 v[kG];
#pragma unroll
          for (int u = g0; u < g0 + kG; ++u) {
            bk[u] = bbase[u] + bucket_of<MH>(k[u], bmask[u]);
            v[u - g0] = tab4[bk[u]];
          }
#pragma unroll
          for (int u = g0; u < g0 + kG; ++u) {
            bool found;
            if constexpr (MODE != MODE_BLOCK && !mode_keys(MODE)) {
              found = bucket_has(v[u - g0], k[u]);
            } else {
              const int j = match_slot(v[u - g0], k[u]);
              found = j >= 0;
              if (found) credit<MODE, KIND>(A, tr, (int)(bk[u] * kBucket + j), pos[u], k[u]);
            }
            hits += found ? 1u : 0u;
            if (kTaskHits) fmask |= (found ? 1u : 0u) << u;
            unres[u] = ok[u] & !found & (v[u - g0].w != kEmpty);
            any_unres |= unres[u];
          }
        }
        // full first bucket: continue into the next ones (bounded by D)
        if (tr.D > 0 && __ballot(any_unres)) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            uint32_t b2 = bk[u] - bbase[u];
            for (int i = 1; i <= tr.D && unres[u]; ++i) {
              b2 = (b2 + 1) & bmask[u];
              const int4 w = tab4[bbase[u] + b2];
              bool found;
              if constexpr (MODE != MODE_BLOCK && !mode_keys(MODE)) {
                found = bucket_has(w, k[u]);
              } else {
                const int j = match_slot(w, k[u]);
                found = j >= 0;
                if (found) credit<MODE, KIND>(A, tr, (int)((bbase[u] + b2) * kBucket + j), pos[u], k[u]);
              }
              hits += found ? 1u : 0u;
              if (kTaskHits) fmask |= (found ? 1u : 0u) << u;
              unres[u] = !found & (w.w != kEmpty);
            }
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t where = ok[u] ? hbm_find(A.hcol, tr.rs, tr.d, k[u]) : -1;
          if (where >= 0) {
            ++hits;
            if (MODE != MODE_COUNT) credit<MODE, TK_GLOBAL>(A, tr, (int)where, pos[u], k[u]);
            if (kTaskHits) fmask |= 1u << u;
          }
        }
      }
      if constexpr (kTaskHits && !kEndCounts) {
        // this lane's task covers the relative probes [s_rel, e) (s_rel may
        // be below 0 for lane 0); add the hits of batch u that fall there
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint64_t hm = __ballot((fmask >> u) & 1u);
          if (hm) {
            const int base = (int)(sb + 64u * (uint32_t)u);
            tcnt += (uint32_t)__popcll(hm & lane_range_mask((int)s_rel - base, (int)e - base));
          }
        }
      }
      if constexpr (kEndCounts) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint64_t hm = __ballot((fmask >> u) & 1u);
          const uint64_t hm1 = SHORT ? __ballot((fmask1 >> u) & 1u) : 0;
          if (MODE == MODE_SUPPORT_FULL && SHORT && (hm | hm1)) credit_probed(A, pos[u], hm, hm1);
          if (ends[u]) {
            // hits of this lane's probes and the ones before it
            uint32_t c = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, run));
            c += (fmask >> u) & 1u;
            if (SHORT) {
              c = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm1, c));
              c += (fmask1 >> u) & 1u;
            }
            if ((ends[u] >> lane) & 1ull) tend[jl[u]] = c;
          }
          run += (uint32_t)__popcll(hm) + (SHORT ? (uint32_t)__popcll(hm1) : 0u);
        }
      }
    }
    if (kTaskHits && !kEndCounts && tcnt) credit_task<MODE, MULTI>(A, tr, tsj, trow, tcnt);
    if constexpr (kEndCounts) {
      wave_sync_lds();
      if (run) {
        // (a task without probes here ends where the one before it does, and
        // its word was not written)
        const uint32_t ce = tend[lane];
        const uint32_t cp = (uint32_t)__shfl_up((int)ce, 1, 64);
        const uint32_t c = ce - (lane == 0 ? 0u : cp);
        const bool any = lane == 0 ? e > 0 : e != e_prev;
        if (any && c) credit_task<MODE, MULTI>(A, tr, tsj, trow, c);
        wave_sync_lds();
      }
    }
    if (more) {
      t += 64;  // a window that is not the last covers exactly its 64 tasks
      P0 = done + lim;
      Pe = nPe;
      tsj = ntsj;
    }
    done += lim;
  }
}

// Work-group total of the hits (returned to thread 0, which also adds it to
// A.count when that is set).
template <int MODE>
__device__ __forceinline__ unsigned long long block_flush(unsigned long long hits, const Args& A) {
  __shared__ unsigned long long s_sum[kPackWavesMax];
  unsigned long long h = wave_sum(hits);
  if (lane_id() == 0) s_sum[threadIdx.x >> 6] = h;
  __syncthreads();
  unsigned long long tot = 0;
  if (threadIdx.x == 0) {
    const int nw = (int)(blockDim.x >> 6);
    for (int w = 0; w < nw; ++w) tot += s_sum[w];
    if (A.count && tot) atomicAdd(A.count, tot);
  }
  if (MODE == MODE_BLOCK && A.per_shift && (int)threadIdx.x < A.q) {
    const unsigned int c = shift_counters()[threadIdx.x];
    if (c) atomicAdd(&A.per_shift[threadIdx.x], (unsigned long long)c);
  }
  return tot;
}

// Clear the work-group's shift counters (MODE_BLOCK); a barrier follows in
// every kernel before any credit.
template <int MODE>
__device__ __forceinline__ void block_init() {
  if (MODE == MODE_BLOCK && threadIdx.x < 64) shift_counters()[threadIdx.x] = 0;
}

// Puts distance v into the first free 16-bit slot of bucket bk (two words of
// two slots); the slot's index, or -1 if the bucket is full.
__device__ __forceinline__ int insert16(uint32_t* tab, uint32_t bk, uint32_t v) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t* w = &tab[bk * 2 + i];
    uint32_t old = *w;
    while ((old >> 16) == kEmpty16) {  // a slot of this word is free
      const bool low = (old & 0xFFFFu) == kEmpty16;
      const uint32_t want = low ? (old & 0xFFFF0000u) | v : (old & 0xFFFFu) | (v << 16);
      const uint32_t was = atomicCAS(w, old, want);
      if (was == old) return (int)(bk * kBucket + 2 * i + (low ? 0 : 1));
      old = was;
    }
  }
  return -1;
}

// VERTEX: a wave's hits of hashed row b.
__device__ __forceinline__ void credit_row(const Args& A, int32_t b, uint32_t hits) {
  const uint32_t h = wave_sum(hits);  // (a work-group holds fewer than 2^18 probes)
  if (lane_id() == 0 && h) credit_vertex(A, (uint32_t)b, h);
}

// Packs of light rows (one work-group each): up to kPackRows rows, one per
// thread for its metadata; all their tables are built together in LDS (keys
// flattened over the work-group), then the pack's probe range - the tasks of
// its rows are contiguous - is split over the 4 waves and probed flattened,
// each task looking up its own row's table.
constexpr int kPackMetaWords = 3 * kPackRows + 1;  // row_t0, row_desc, key prefix (+ end)

// LDS words before a pack's tables (a multiple of four: buckets are read as
// 16 bytes).
__host__ __device__ constexpr int pack_head_words(int mode, int waves) {
  return (waves * wave_words(mode) + kPackMetaWords + (mode == MODE_VERTEX ? kPackRows : 0) + 3) & ~3;
}

// Exclusive scan over the first kPackRows threads of a work-group (the others
// bring 0) and the total; two barriers.
__device__ __forceinline__ uint32_t pack_scan(uint32_t v, uint32_t* s_w, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v);
  if (lane == 63 && wave < kPackRows / 64) s_w[wave] = inc;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kPackRows / 64; ++w) {
    if (w < wave) before += s_w[w];
    tot += s_w[w];
  }
  __syncthreads();
  total = tot;
  return before + inc - v;
}

// WAVES: waves of the work-group, which share the pack's probes (4, or more
// where a class has too few packs to fill the GPU: see launch_packs16). In a
// batch the pack may be cut into 2^cut units, of which this is number `part`.
template <int MODE, int VAR, bool SHORT, int WAVES>
__device__ __forceinline__ unsigned long long pack_body(const Args& A, const PackRow* __restrict__ recs,
                                          const PackInfo* __restrict__ info, uint32_t pack,
                                          uint32_t pack_slots, int32_t* smem, uint32_t part = 0,
                                          uint32_t cut = 0) {
  __shared__ int s_D;
  __shared__ uint32_t s_w[4], s_w2[4];
  constexpr bool VALS = mode_keys(MODE);
  constexpr int NT = 64 * WAVES;
  static_assert(kPackWavesMax % WAVES == 0 && NT >= kPackRows, "pack work-group shape");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t* bm = reinterpret_cast<uint32_t*>(smem) + wave * wave_words(MODE);
  uint32_t* row_t0 = reinterpret_cast<uint32_t*>(smem) + WAVES * wave_words(MODE);
  uint32_t* row_desc = row_t0 + kPackRows;
  uint32_t* row_k0 = row_desc + kPackRows;  // kPackRows + 1 entries
  uint32_t* row_hits = row_k0 + kPackRows + 1;  // VERTEX
  int32_t* tab = smem + pack_head_words(MODE, WAVES);
  int32_t* val = tab + (SHORT ? pack_slots / 2 : pack_slots);  // (short rows: 16-bit slots)
  if (lane < kBmWords) bm[lane] = 0;
  block_init<MODE>();

  const PackInfo& pi = info[pack];
  const uint32_t r0 = pi.r0, r1 = pi.r1;
  const int nr = (int)(r1 - r0);  // 1 .. kPackRows
  // this wave's share of the pack's probes, its first task, and its first
  // window (in flight while the tables are built)
  const uint64_t q0 = pi.q0, W = pi.q1 - pi.q0;
  const int shares = (kPackWavesMax / WAVES) >> cut, share0 = ((int)part * WAVES + wave) * shares;
  const uint64_t wq0 = q0 + pack_share(W, share0);
  const uint64_t wq1 = q0 + pack_share(W, share0 + shares);
  const uint32_t wt = (uint32_t)__builtin_amdgcn_readfirstlane((int)pi.wt[share0]);
  const uint32_t wlen = (uint32_t)(wq1 - wq0);
  const Window w0 = window_first(A, wt, wq0, wlen);
  const bool lds_hits = VALS && (SHORT ? 2 * W : W) < kPackLdsHitsMax;  // (uniform: the pack's probes)
  uint32_t d = 0, S = 0, rs = 0;
  if (tid < nr) {
    const PackRow pr = recs[r0 + tid];
    rs = pr.rs;
    // a row without tasks (a pack member only without the doubly sparse
    // traversal, tc_graph_variant) has d = 0: no table
    d = pr.d;
    S = 1u << pack_table_log2(d);
    row_t0[tid] = pr.tb;
  }
  uint32_t S_tot, K_tot;
  const uint32_t off = pack_scan(S, s_w, S_tot);
  const uint32_t k0 = pack_scan(d, s_w2, K_tot);
  if (tid < nr) {
    row_desc[tid] = (off / kBucket) | ((S / kBucket - 1) << 16);
    row_k0[tid] = k0;
  }
  if (tid == 0) {
    row_k0[nr] = K_tot;
    s_D = 0;
  }
  for (uint32_t i = tid; i < (SHORT ? S_tot / 2 : S_tot); i += NT) tab[i] = kEmpty;
  __syncthreads();

  // build: key x of the pack belongs to the last row i with row_k0[i] <= x;
  // this thread also remembers its own row's start (rows are few per thread)
  __shared__ uint32_t s_rs[kPackRows];
  if (tid < nr) s_rs[tid] = rs;
  if (MODE == MODE_VERTEX && tid < kPackRows) row_hits[tid] = 0;
  __syncthreads();
  int md = 0;
  for (uint32_t x = tid; x < K_tot; x += NT) {
    int lo = 0, hi = nr;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (row_k0[mid] <= x) lo = mid;
      else hi = mid;
    }
    const uint32_t p = s_rs[lo] + (x - row_k0[lo]);
    const int32_t key = A.hcol[p];
    const uint32_t dsc = row_desc[lo];
    const uint32_t base = dsc & 0xFFFFu, bmask = dsc >> 16;
    const uint32_t v = (uint32_t)(A.n - key);  // (short rows)
    uint32_t bk = SHORT ? v & bmask : bucket_of<VAR == VAR_MUL>(key, bmask);
    int disp = 0, slot = -1;
    while (true) {
      if constexpr (SHORT) {
        slot = insert16(reinterpret_cast<uint32_t*>(tab), base + bk, v);
      } else
#pragma unroll
      for (int s2 = 0; s2 < kBucket; ++s2) {
        if (slot < 0 && atomicCAS(&tab[(base + bk) * kBucket + s2], kEmpty, key) == kEmpty)
          slot = (int)((base + bk) * kBucket + s2);
      }
      if (slot >= 0) break;
      bk = (bk + 1) & bmask;
      ++disp;
    }
    if (VALS) val[slot] = lds_hits ? (int32_t)x : (int32_t)p;  // key index, or U position
    md = disp > md ? disp : md;
  }
  // (a plain LDS max per lane: a wave reduction here would share its lane
  // addresses with the final one and keep them live across the probe loop)
  if (md) atomicMax(&s_D, md);
  __syncthreads();

  TableRef tr{tab, val, 0, s_D, 0, 0, row_t0, row_desc, nr, lds_hits ? 1 : 0, row_hits, nullptr, nullptr};
  uint32_t hits = 0;
  if (wlen > 0) wave_probe<MODE, SHORT ? TK_MULTI16 : TK_MULTI, VAR>(A, tr, wt, wq0, wlen, bm, hits, w0);
  if constexpr (VALS) {
    if (lds_hits) {
      // the (b, k) credits of the pack: one atomic per slot that was hit, at
      // the U position of its key (row found from the key index)
      __syncthreads();
      for (uint32_t i = tid; i < S_tot; i += NT) {
        if (SHORT ? reinterpret_cast<const uint16_t*>(tab)[i] == kEmpty16 : tab[i] == kEmpty) continue;
        const uint32_t w = (uint32_t)val[i];
        const uint32_t c = w >> kPackValBits;
        if (c == 0) continue;
        const uint32_t x = w & ((1u << kPackValBits) - 1u);
        int lo = 0, hi = nr;
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (row_k0[mid] <= x) lo = mid;
          else hi = mid;
        }
        const uint32_t p = s_rs[lo] + (x - row_k0[lo]);
        if (MODE == MODE_VERTEX) credit_vertex(A, (uint32_t)A.hcol[p], c);
        else if (p < A.m) atomicAdd(&A.support[p], (int)c);
      }
    }
  }
  if constexpr (MODE == MODE_VERTEX) {
    __syncthreads();
    // (the hashed row is the column of the entry before its first task's first probe)
    if (tid < nr && row_hits[tid]) credit_vertex(A, (uint32_t)A.hcol[A.tstart[row_t0[tid]] - 1u], row_hits[tid]);
  }
  return block_flush<MODE>(hits, A);
}

// Register budgets (waves per SIMD) of the pack kernel and of the persistent
// batch kernel in count mode (their LDS use would allow about 6 work-groups per
// CU; 5 with spill-free registers runs faster).
constexpr int kOccPacks = 5, kOccBatch = 5, kOccBatch16 = 6;

template <int MODE, int VAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    MODE == MODE_COUNT || MODE == MODE_SUPPORT_ORIENTED ? kOccPacks : 4)))
void k_count_packs(Args A, const PackRow* __restrict__ recs, const PackInfo* __restrict__ info,
                   uint32_t pack_slots) {
  extern __shared__ int4 smem4[];  // 16-byte aligned: tables are read as int4 buckets
  pack_body<MODE, VAR, false, kWaves>(A, recs, info, blockIdx.x, pack_slots, reinterpret_cast<int32_t*>(smem4));
}

// The short rows' packs of both pack classes in one launch: the first n0
// work-groups take those of the first list.
template <int MODE, int OCC, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_count_packs16(Args A, const PackRow* __restrict__ recs0, const PackInfo* __restrict__ info0, uint32_t n0,
                     const PackRow* __restrict__ recs1, const PackInfo* __restrict__ info1, uint32_t pack_slots) {
  extern __shared__ int4 smem4[];
  const bool first = blockIdx.x < n0;
  pack_body<MODE, VAR_BASE, true, WAVES>(A, first ? recs0 : recs1, first ? info0 : info1,
                                         first ? blockIdx.x : blockIdx.x - n0, pack_slots,
                                         reinterpret_cast<int32_t*>(smem4));
}

// Heavy rows: work-group = kWaves consecutive items of the same row b.
template <int MODE, bool GLOBAL, int VAR>
__device__ __forceinline__ unsigned long long items_body(const Args& A, const CountItem* __restrict__ grp,
                                                         int32_t* smem) {
  __shared__ int s_D;
  constexpr bool VALS = mode_keys(MODE);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t* bm = reinterpret_cast<uint32_t*>(smem) + wave * wave_words(MODE);
  const int64_t rs = grp[0].rs, d = grp[0].d;
  // this wave's item and its first window (in flight while the table is built)
  const CountItem it = grp[wave];
  const Window w0 = window_first(A, it.t0, it.q0, it.len);
  if (lane < kBmWords) bm[lane] = 0;
  block_init<MODE>();
  uint32_t hits = 0;
  TableRef tr{nullptr, nullptr, 0, 0, rs, d, nullptr, nullptr, 0, 0, nullptr, nullptr, nullptr};
  if (GLOBAL) {
    __syncthreads();  // shift counters cleared before any credit
  } else {
    const uint32_t S = 1u << grp[0].log2S;
    int32_t* tab = smem + kWavesBig * wave_words(MODE);
    int32_t* val = tab + S;
    for (uint32_t i = tid; i < S; i += blockDim.x) tab[i] = kEmpty;
    if (tid == 0) s_D = 0;
    __syncthreads();
    const uint32_t bmask = S / kBucket - 1;
    int md = build_table<VALS, VAR == VAR_MUL>(tab, val, bmask, A.hcol, rs, d, tid, (int)blockDim.x);
    if (md) atomicMax(&s_D, md);  // per lane: see pack_body
    __syncthreads();
    tr.tab = tab;
    tr.val = val;
    tr.bmask = bmask;
    tr.D = s_D;
  }
  wave_sync_lds();
  if (it.len) wave_probe<MODE, GLOBAL ? TK_GLOBAL : TK_SINGLE, VAR>(A, tr, it.t0, it.q0, it.len, bm, hits, w0);
  if constexpr (VALS && !GLOBAL) {
    // the (b, k) credits of the work-group: one atomic per slot that was hit
    __syncthreads();
    const uint32_t S = 1u << grp[0].log2S;
    for (uint32_t i = threadIdx.x; i < S; i += blockDim.x) {
      if (tr.tab[i] == kEmpty) continue;
      const uint32_t w = (uint32_t)tr.val[i];
      const uint32_t c = w >> kValBits;
      const int64_t p = rs + (int64_t)(w & ((1u << kValBits) - 1u));
      if (MODE == MODE_VERTEX && c) credit_vertex(A, (uint32_t)A.hcol[p], c);
      else if (c && p < (int64_t)A.m) atomicAdd(&A.support[p], (int)c);
    }
  }
  if constexpr (MODE == MODE_VERTEX) credit_row(A, grp[0].b, hits);
  return block_flush<MODE>(hits, A);
}

// A group of kWaves items of one short row: its keys in a bitmap over the
// distances [0, n - b]. FULL support also holds, for every bitmap word with
// keys, the number of keys of smaller distance, and a hit counter per key, if
// the row's keys fit the max_keys counters of the launch.
struct BitsLds {
  uint32_t* bm;    // this wave's words
  uint32_t* bits;
  uint32_t* cnt;
  uint16_t* pfx;
};
template <int MODE>
__device__ __forceinline__ BitsLds bits_lds(const Args& A, uint32_t max_keys, int32_t* smem) {
  BitsLds L;
  L.bm = reinterpret_cast<uint32_t*>(smem) + (threadIdx.x >> 6) * wave_words(MODE);
  L.bits = reinterpret_cast<uint32_t*>(smem) + kWaves * wave_words(MODE);
  L.cnt = L.bits + bitmap_words(A.n);
  L.pfx = reinterpret_cast<uint16_t*>(L.cnt + max_keys);
  return L;
}

// Keys of the row a thread holds in registers (loaded ahead).
constexpr int kKeyRegs = 4;
__device__ __forceinline__ void bits_keys(const Args& A, const CountItem& it, int32_t (&key)[kKeyRegs]) {
#pragma unroll
  for (int j = 0; j < kKeyRegs; ++j) {
    const uint32_t i = threadIdx.x + (uint32_t)j * (64 * kWaves);
    key[j] = i < it.d ? A.hcol[(uint64_t)it.rs + i] : 0;
  }
}

// Clears and fills the bitmap of `it`'s row; ends with a barrier. The caller
// has passed a barrier since the bitmap was last read.
template <int MODE>
__device__ __forceinline__ void bits_build(const Args& A, const BitsLds& L, const CountItem& it, uint32_t max_keys,
                                           const int32_t (&key)[kKeyRegs]) {
  constexpr bool FULL = mode_keys(MODE);
  constexpr uint32_t NT = 64 * kWaves;
  const uint32_t words = ((uint32_t)(A.n - it.b) >> 5) + 1;
  for (uint32_t i = threadIdx.x; i < words; i += NT) L.bits[i] = 0;
  if (FULL && it.d <= max_keys)
    for (uint32_t i = threadIdx.x; i < it.d; i += NT) L.cnt[i] = 0;
  __syncthreads();
  auto put = [&](uint32_t i, int32_t k) {
    const uint32_t v = (uint32_t)(A.n - k);
    atomicOr(&L.bits[v >> 5], 1u << (v & 31));
    // (ascending columns: distances fall along the row, and the last key of
    // a word is the word's smallest distance)
    if (FULL && (i + 1 == it.d || (uint32_t)(A.n - A.hcol[(uint64_t)it.rs + i + 1]) >> 5 != v >> 5))
      L.pfx[v >> 5] = (uint16_t)(it.d - 1 - i);
  };
#pragma unroll
  for (int j = 0; j < kKeyRegs; ++j) {
    const uint32_t i = threadIdx.x + (uint32_t)j * NT;
    if (i < it.d) put(i, key[j]);
  }
  for (uint32_t i = threadIdx.x + kKeyRegs * NT; i < it.d; i += NT) put(i, A.hcol[(uint64_t)it.rs + i]);
  __syncthreads();
}

template <int MODE>
__device__ __forceinline__ void bits_probe(const Args& A, const BitsLds& L, const CountItem& it, uint32_t max_keys,
                                           const Window& w0, uint32_t& hits) {
  constexpr bool FULL = mode_keys(MODE);
  TableRef tr{reinterpret_cast<const int32_t*>(L.bits), nullptr, 0, 0, (int64_t)it.rs, (int64_t)it.d, nullptr,
              nullptr, 0, 0, nullptr, L.pfx, it.d <= max_keys ? L.cnt : nullptr};
  if (it.len) wave_probe<MODE, TK_BITS, VAR_BASE>(A, tr, it.t0, it.q0, it.len, L.bm, hits, w0);
  if constexpr (FULL) {
    // the (b, k) credits of the work-group: one atomic per key that was hit
    if (it.d <= max_keys) {
      __syncthreads();
      for (uint32_t i = threadIdx.x; i < it.d; i += 64 * kWaves) {
        const uint32_t c = L.cnt[i];
        const uint64_t p = (uint64_t)it.rs + it.d - 1 - i;
        if (MODE == MODE_VERTEX && c) credit_vertex(A, (uint32_t)A.hcol[p], c);
        else if (c && p < (uint64_t)A.m) atomicAdd(&A.support[p], (int)c);
      }
    }
  }
  if constexpr (MODE == MODE_VERTEX) credit_row(A, it.b, hits);
}

// The groups [g, end) of one class's short rows (items: the first of them),
// end > g. A group's chain of dependent loads (item, then the row's keys and
// the wave's first window) costs more than the probes of most groups, so the
// next group's keys and window and the item of the one after are loaded while
// the present one is probed. Returns this thread's hits.
template <int MODE>
__device__ __forceinline__ unsigned long long bits_groups(const Args& A, const CountItem* __restrict__ items,
                                                          uint32_t g, uint32_t end, uint32_t max_keys,
                                                          int32_t* smem) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const BitsLds L = bits_lds<MODE>(A, max_keys, smem);
  if (lane < kBmWords) L.bm[lane] = 0;
  auto item = [&](uint32_t i) { return items[(uint64_t)(i < end ? i : end - 1) * kWaves + wave]; };
  CountItem it = item(g), next = item(g + 1);
  int32_t key[kKeyRegs];
  bits_keys(A, it, key);
  Window w = window_first(A, it.t0, it.q0, it.len);
  unsigned long long sum = 0;
  for (;;) {
    bits_build<MODE>(A, L, it, max_keys, key);
    const CountItem cur = it;
    const Window w0 = w;
    it = next;
    bits_keys(A, it, key);
    w = window_first(A, it.t0, it.q0, it.len);
    next = item(g + 2);
    uint32_t hits = 0;
    bits_probe<MODE>(A, L, cur, max_keys, w0, hits);
    sum += hits;
    if (++g >= end) break;
    __syncthreads();  // every wave is done with the bitmap
  }
  return sum;
}

// The same with the rows looked up in U_b in HBM (batch units under an LDS cap).
template <int MODE>
__device__ __forceinline__ unsigned long long bits_groups_hbm(const Args& A, const CountItem* __restrict__ items,
                                                              uint32_t g, uint32_t end, int32_t* smem) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* bm = reinterpret_cast<uint32_t*>(smem) + wave * wave_words(MODE);
  if (lane < kBmWords) bm[lane] = 0;
  wave_sync_lds();
  unsigned long long sum = 0;
  for (; g < end; ++g) {
    const CountItem it = items[(uint64_t)g * kWaves + wave];
    TableRef tr{nullptr, nullptr, 0, 0, (int64_t)it.rs, (int64_t)it.d, nullptr, nullptr, 0, 0, nullptr, nullptr, nullptr};
    uint32_t hits = 0;
    if (it.len)
      wave_probe<MODE, TK_GLOBAL16, VAR_BASE>(A, tr, it.t0, it.q0, it.len, bm, hits,
                                              window_first(A, it.t0, it.q0, it.len));
    sum += hits;
  }
  return sum;
}

// The short rows' items of all item classes in one launch: a work-group takes
// one bundle of groups (kWaves items of one row each); the work-groups from
// end[c - 1] to end[c] take those of list c.
constexpr int kItemLists = NUM_CLASSES - CLS_WG_SMALL;
struct ItemLists {
  const CountItem* items[kItemLists];
  const uint32_t* bundle[kItemLists];
  uint32_t end[kItemLists];
};

template <int MODE, int OCC>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_count_bits(Args A, ItemLists lists, uint32_t max_keys) {
  extern __shared__ int4 smem4[];
  const CountItem* items = lists.items[0];
  const uint32_t* bundle = lists.bundle[0];
  uint32_t base = 0;
#pragma unroll
  for (int c = 1; c < kItemLists; ++c) {
    if (blockIdx.x >= lists.end[c - 1]) {
      items = lists.items[c];
      bundle = lists.bundle[c];
      base = lists.end[c - 1];
    }
  }
  const uint32_t g = bundle[blockIdx.x - base];
  const uint32_t end = bundle[blockIdx.x - base + 1];
  if (g >= end) return;  // (a group longer than a bundle leaves the next one empty)
  block_flush<MODE>(bits_groups<MODE>(A, items, g, end, max_keys, reinterpret_cast<int32_t*>(smem4)), A);
}

// OCC: waves per SIMD the kernel's registers are budgeted for. A class whose
// tables limit a CU to fewer work-groups gets the registers that would
// otherwise go unused (fewer spills in the probe loop).
template <int MODE, bool GLOBAL, int OCC, int WAVES, int VAR>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_count_items(Args A, const CountItem* __restrict__ items) {
  extern __shared__ int4 smem4[];  // 16-byte aligned: tables are read as int4 buckets
  items_body<MODE, GLOBAL, VAR>(A, items + (int64_t)blockIdx.x * WAVES, reinterpret_cast<int32_t*>(smem4));
}

// Count mode per class (chosen by timing at RMAT scale 24): wg_small and
// wg_large tables (<= 4 / 16 KiB) would allow 8 or more work-groups per CU,
// but 7 waves per SIMD with spill-free registers run faster; wg_huge tables
// (32 KiB) allow 4-5 work-groups per CU and wg_giant tables (64 KiB) 2.
// Support modes hold more state per probe and run at 4.
constexpr int kOccBits = 8, kOccBitsOriented = 6, kOccBitsFull = 5;  // (bitmaps take at most 8 KiB: registers limit the waves)
constexpr int kOccPacks16 = 7;
constexpr uint32_t kPacks16Waves = 1024;  // packs up to which 16 waves share one
constexpr int kOccSmall = 7, kOccLarge = 7, kOccHuge = 5, kOccGiant = 4, kOccSupport = 5;

template <int MODE, bool GLOBAL, int VAR>
const void* items_kernel(int cls) {
  static_assert(class_waves(CLS_WG_HUGE) == kWavesBig && class_waves(CLS_WG_GIANT) == kWavesBig &&
                    class_waves(CLS_WG_LARGE) == kWaves && class_waves(CLS_GLOBAL) == kWaves,
                "work-group shapes of the item classes");
  // oriented support adds only the per-task counters to the count: same budgets;
  // wide probe addresses take more registers: the support budget
  constexpr bool kCountLike = (MODE == MODE_COUNT || MODE == MODE_SUPPORT_ORIENTED) && VAR != VAR_WIDE;
  if constexpr (GLOBAL) {  // no table: LDS does not limit
    return (const void*)k_count_items<MODE, GLOBAL, kCountLike ? kOccSmall : kOccSupport, kWaves, VAR>;
  } else if constexpr (!kCountLike) {
    if (class_waves(cls) == kWavesBig) return (const void*)k_count_items<MODE, GLOBAL, kOccSupport, kWavesBig, VAR>;
    return (const void*)k_count_items<MODE, GLOBAL, kOccSupport, kWaves, VAR>;
  } else {
    switch (cls) {
      case CLS_WG_LARGE: return (const void*)k_count_items<MODE, GLOBAL, kOccLarge, kWaves, VAR>;
      case CLS_WG_HUGE: return (const void*)k_count_items<MODE, GLOBAL, kOccHuge, kWavesBig, VAR>;
      case CLS_WG_GIANT: return (const void*)k_count_items<MODE, GLOBAL, kOccGiant, kWavesBig, VAR>;
      default: return (const void*)k_count_items<MODE, GLOBAL, kOccSmall, kWaves, VAR>;
    }
  }
}

__global__ void k_zero_i64(int64_t* p) { *p = 0; }

__global__ void k_zero_i32(int32_t* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// launch names seen by the phase timer: "<mode>:<class>"
const char* const kLaunchNames[5][NUM_CLASSES] = {
    {"count:pack_small", "count:pack_large", "count:wg_small", "count:wg_large", "count:wg_huge",
     "count:wg_giant", "count:global"},
    {"support_full:pack_small", "support_full:pack_large", "support_full:wg_small",
     "support_full:wg_large", "support_full:wg_huge", "support_full:wg_giant", "support_full:global"},
    {"support_oriented:pack_small", "support_oriented:pack_large", "support_oriented:wg_small",
     "support_oriented:wg_large", "support_oriented:wg_huge", "support_oriented:wg_giant",
     "support_oriented:global"},
    {"block:pack_small", "block:pack_large", "block:wg_small", "block:wg_large", "block:wg_huge",
     "block:wg_giant", "block:global"},
    {"vertex:pack_small", "vertex:pack_large", "vertex:wg_small", "vertex:wg_large", "vertex:wg_huge",
     "vertex:wg_giant", "vertex:global"}};

const char* const kBitsNames[5] = {"count:short_items", "support_full:short_items", "support_oriented:short_items", "",
                                   "vertex:short_items"};
const char* const kPacks16Names[5] = {"count:short_packs", "support_full:short_packs", "support_oriented:short_packs", "",
                                      "vertex:short_packs"};

// Work-groups per launch of one class: a dispatch holds fewer than 2^32
// work-items (a class of more groups, e.g. small wave items on a very large
// graph, is launched in pieces; each group finds its data by its index).
constexpr int64_t kClassLaunchMax = (int64_t)1 << 22;

// The short rows' items.
template <int MODE>
void launch_bits(const WorkSet& w, const Args& A, hipStream_t st) {
  ItemLists lists;
  uint32_t bundles = 0;
  int log2S = 6;
  for (int i = 0; i < kItemLists; ++i) {
    const int c = CLS_WG_SMALL + i;
    lists.items[i] = w.items[c] + w.n_items32[c];
    lists.bundle[i] = w.bundle[c];
    if (w.n_items[c] > w.n_items32[c]) log2S = std::max(log2S, std::min(w.cls_log2S[c], kMaxLog2S));
    bundles += (uint32_t)w.n_bundles[c];
    lists.end[i] = bundles;
  }
  if (bundles == 0) return;
  const size_t lds = bits_lds_bytes(A.n, log2S, MODE);
  const uint32_t max_keys = bits_max_keys(log2S, MODE);
  constexpr int OCC = mode_keys(MODE) ? kOccBitsFull : MODE == MODE_COUNT ? kOccBits : kOccBitsOriented;
  TC_LAUNCH(kBitsNames[MODE], (k_count_bits<MODE, OCC>), dim3(bundles), dim3(64 * kWaves), lds, st, A, lists,
            max_keys);
}

// The short rows' packs. With few of them (a small graph) more waves share
// each pack: four would leave most of the GPU idle behind a few long chains
// of windows. Count of ER graphs with 4 / 8 / 16 waves: 418 packs 81 / 54 / 52 us,
// 1029 packs 103 / 81 / 83, 1728 packs 150 / 116 / 137, 3167 packs 245 / 154 / 228;
// where most probes are in items, which the packs run beside, more waves gain
// little and then cost (RMAT n = 700001, 2806 packs: count 431 / 416 / 468 us,
// oriented support 594 / 607 / 653 us).
template <int MODE>
void launch_packs16(const WorkSet& w, const Args& A, hipStream_t st) {
  uint32_t n[2], slots = 0;
  const PackInfo* info[2];
  for (int c = 0; c < 2; ++c) {
    n[c] = (uint32_t)(w.n_packs[c] - w.n_packs32[c]);
    info[c] = w.pack_info[c] + w.n_packs32[c];
    if (n[c]) slots = std::max(slots, pack16_slots(w.wp.pack_slots, w.pack_log2S[c]));
  }
  const uint32_t packs = n[0] + n[1];
  if (packs == 0) return;
  constexpr int OCC = mode_keys(MODE) ? 4 : kOccPacks16;
  const bool most = 2 * (w.cls_probes[CLS_PACK_SMALL] + w.cls_probes[CLS_PACK_LARGE]) >= (uint64_t)w.probes;
  const int waves = packs <= kPacks16Waves ? 16 : packs <= (most ? 4 : 2) * kPacks16Waves ? 8 : kWaves;
  const size_t lds = pack16_lds_bytes(slots, MODE, waves);
  auto* f = waves == 16 ? k_count_packs16<MODE, 4, 16> : waves == 8 ? k_count_packs16<MODE, 4, 8>
                                                                    : k_count_packs16<MODE, OCC, kWaves>;
  if (lds > 65536)
    TC_HIP(hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  // (at most one pack per short row: fewer than 2^16)
  TC_LAUNCH(kPacks16Names[MODE], f, dim3(packs), dim3(64 * waves), lds, st, A, w.pack_recs[0], info[0], n[0],
            w.pack_recs[1], info[1], slots);
}

template <int MODE, int VAR>
void launch_items_class(const WorkSet& w, const Args& A, int c, size_t mark_bytes, hipStream_t st) {
  if (w.n_items32[c] == 0) return;
  const int64_t groups = w.n_items32[c] / class_waves(c);
  const bool global = c == CLS_GLOBAL;
  const void* f = global ? items_kernel<MODE, true, VAR>(c) : items_kernel<MODE, false, VAR>(c);
  const size_t lds = global ? mark_bytes : items_lds_bytes(w.cls_log2S[c], MODE);
  if (lds > 65536) TC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  LaunchScope ls(kLaunchNames[MODE][c], st);
  for (int64_t g0 = 0; g0 < groups; g0 += kClassLaunchMax) {
    const unsigned grid = (unsigned)std::min<int64_t>(kClassLaunchMax, groups - g0);
    const CountItem* items = w.items[c] + g0 * class_waves(c);
    void* kargs[] = {const_cast<Args*>(&A), &items};
    TC_HIP(hipLaunchKernel(f, dim3(grid), dim3(64 * class_waves(c)), kargs, lds, st));
  }
}

// The light classes (packs, wg_small: small tables, few probes per row) run
// on a side stream beside the heavy ones, so that their launches - short,
// and ending on a few long work-groups that nothing else overlaps - fill the
// GPU while the heavy classes stream. One side stream per (device, caller
// stream), with a fork and a join event; never destroyed; default priority.
// At most kSideStreams of them exist: calls on further caller streams run
// every class on the caller's stream.
struct SideStream {
  hipStream_t aux = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};

constexpr size_t kSideStreams = 64;

SideStream* side_stream(hipStream_t st) {
  static std::mutex mu;
  static std::map<std::pair<int, hipStream_t>, SideStream> streams;
  int dev = 0;
  TC_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(mu);
  auto it = streams.find({dev, st});
  if (it == streams.end()) {
    if (streams.size() >= kSideStreams) return nullptr;
    SideStream s;
    TC_HIP(hipStreamCreateWithFlags(&s.aux, hipStreamNonBlocking));
    TC_HIP(hipEventCreateWithFlags(&s.fork, hipEventDisableTiming));
    TC_HIP(hipEventCreateWithFlags(&s.join, hipEventDisableTiming));
    it = streams.emplace(std::make_pair(dev, st), s).first;
  }
  return &it->second;
}

// Probes below which a graph's classes all run on the caller's stream (the
// fork and join would cost more than they save).
constexpr int64_t kSideMinProbes = (int64_t)1 << 24;

template <int MODE, int VAR>
void launch_mode(const WorkSet& w, const Args& A, hipStream_t st) {
  constexpr bool VALS = mode_keys(MODE);
  const size_t mark_bytes = items_lds_bytes(-1, MODE);
  // the light classes go to the side stream when both sides have work
  bool light = false, heavy = false;
  for (int c = 0; c < NUM_CLASSES; ++c) {
    const bool any = c <= CLS_PACK_LARGE ? w.n_packs[c] > 0 : w.n_items[c] > 0;
    (c <= CLS_WG_SMALL ? light : heavy) |= any;
  }
  // (one rank's block keeps its classes on the caller's stream: its launches
  // are small, and its per-class times stay separable)
  SideStream* side =
      MODE != MODE_BLOCK && light && heavy && w.probes >= kSideMinProbes ? side_stream(st) : nullptr;
  if (side) {
    TC_HIP(hipEventRecord(side->fork, st));
    TC_HIP(hipStreamWaitEvent(side->aux, side->fork, 0));
  }
  // heavy classes first (on st), then the light ones (on the side stream)
  if constexpr (MODE == MODE_BLOCK)
    TC_REQUIRE(w.b16 >= w.nrows, TC_EDEVICE, "launch_count: short rows in a rank's block");
  else
    launch_bits<MODE>(w, A, st);
  for (int c = CLS_WG_LARGE; c <= CLS_GLOBAL; ++c) launch_items_class<MODE, VAR>(w, A, c, mark_bytes, st);
  const hipStream_t ls = side ? side->aux : st;
  // A launch of small packs is short and its work-groups wait for memory most of
  // the time: beside wg_large they cost nothing, alone they take as long (RMAT
  // n = 700001, 32-bit rows by multiplicative hashing: 827 us with them first,
  // 992 us with them last; scale 20: 1205 and 1505 us). Where short rows leave
  // wg_large little to do, the longer launch goes first (n = 700001: 436 us with
  // the large packs first, 441 us with the small ones; scale 24: 19.20 and
  // 19.29 ms).
  const bool small_first = w.b16 >= w.nrows;
  for (int i = 0; i < 2; ++i) {
    const int c = small_first ? CLS_PACK_SMALL + i : CLS_PACK_LARGE - i;
    if (w.n_packs32[c] == 0) continue;
    // a pack's tables take at most wp.pack_slots plus one row's table
    const uint32_t slots = w.wp.pack_slots + (1u << w.pack_log2S[c]);
    const size_t lds = pack_lds_bytes(slots, MODE);
    if (lds > 65536)
      TC_HIP(hipFuncSetAttribute((const void*)k_count_packs<MODE, VAR>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    for (int64_t p0 = 0; p0 < w.n_packs32[c]; p0 += kClassLaunchMax)  // (pieces: see kClassLaunchMax)
      TC_LAUNCH(kLaunchNames[MODE][c], (k_count_packs<MODE, VAR>),
                dim3((unsigned)std::min<int64_t>(kClassLaunchMax, w.n_packs32[c] - p0)), dim3(256), lds, ls, A,
                w.pack_recs[c], w.pack_info[c] + p0, slots);
  }
  if constexpr (MODE != MODE_BLOCK) launch_packs16<MODE>(w, A, ls);
  launch_items_class<MODE, VAR>(w, A, CLS_WG_SMALL, mark_bytes, ls);
  if (side) {
    TC_HIP(hipEventRecord(side->join, side->aux));
    TC_HIP(hipStreamWaitEvent(st, side->join, 0));
  }
  TC_HIP(hipGetLastError());
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Batched count: clears the per-graph counters and the unit queue (a kernel,
// not a memset, so that the pair can be captured in a HIP graph).
__global__ void k_batch_clear(unsigned long long* counts, int64_t n, unsigned int* queue) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counts[i] = 0;
  if (i == 0) *queue = 0;
}

// Persistent work-groups pull units from one queue until it is empty (every
// work-group reaches the exit once the counter passes the last chunk); the
// units were ordered when the plan was made (largest first by default). One
// atomic takes `chunk` consecutive units (a tuning choice: fewer atomics on
// the one counter against coarser balance). Each unit runs the same body as
// its class's own kernel with its graph's arguments.
// Bodies that a plan needs none of are left out, since all bodies' registers
// limit the waves: BATCH_SHORT holds those of short rows with their tables in LDS
// (all graphs of up to kShortSpan vertices), BATCH_LONG those of 32-bit rows,
// BATCH_ALL everything, at four waves a SIMD, without spills (128 even graphs of
// 80000 vertices and more, input order: 2956 us with all bodies at five waves,
// 2677 us with those of 32-bit rows alone).
template <int MODE, int BODIES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    MODE == MODE_SUPPORT_FULL || BODIES == BATCH_ALL ? 4
    : BODIES == BATCH_SHORT                           ? kOccBatch16
    : MODE == MODE_COUNT                              ? kOccBatch
                                                      : 4)))
void k_count_batch(const Args* __restrict__ gargs, const BatchUnit* __restrict__ units, uint32_t n_units,
                   uint32_t chunk, unsigned int* __restrict__ queue, unsigned long long* __restrict__ counts) {
  extern __shared__ int4 smem4[];
  int32_t* smem = reinterpret_cast<int32_t*>(smem4);
  __shared__ uint32_t s_chunk;
  const uint32_t n_chunks = (n_units + chunk - 1) / chunk;
  for (;;) {
    __syncthreads();  // the previous chunk is done with s_chunk
    if (threadIdx.x == 0) s_chunk = atomicAdd(queue, 1u);
    __syncthreads();
    const uint32_t ci = __builtin_amdgcn_readfirstlane(s_chunk);  // uniform: unit loads go scalar
    if (ci >= n_chunks) break;
    const uint32_t u_end = ci * chunk + chunk < n_units ? ci * chunk + chunk : n_units;
    for (uint32_t u = ci * chunk; u < u_end; ++u) {
      __syncthreads();  // the previous unit is done with LDS
      const BatchUnit bu = units[u];
      Args A = gargs[bu.graph];
      A.count = counts + bu.graph;
      const auto* recs = static_cast<const PackRow*>(bu.p0);
      const auto* info = static_cast<const PackInfo*>(bu.p1);
      const auto* items = static_cast<const CountItem*>(bu.p0);
      auto short_rows = [&] {
        if ((bu.kind & 0xFF) == BK_PACK16)
          pack_body<MODE, VAR_BASE, true, kWaves>(A, recs, info, bu.index, bu.slots, smem, (bu.kind >> 8) & 0xFF,
                                                  bu.kind >> 16);
        else if (bu.index < bu.end)
          block_flush<MODE>(bits_groups<MODE>(A, items, bu.index, (uint32_t)bu.end, bu.slots, smem), A);
      };
      auto long_rows = [&] {
        if (bu.kind == BK_PACK)
          pack_body<MODE, VAR_BASE, false, kWaves>(A, recs, info, bu.index, bu.slots, smem);
        else if (bu.kind == BK_ITEMS)
          items_body<MODE, false, VAR_BASE>(A, items, smem);
        else
          items_body<MODE, true, VAR_BASE>(A, items, smem);
      };
      if constexpr (BODIES == BATCH_SHORT) {
        short_rows();
      } else if constexpr (BODIES == BATCH_LONG) {
        long_rows();
      } else if ((bu.kind & 0xFF) == BK_PACK16 || bu.kind == BK_BITS) {
        short_rows();
      } else if (bu.kind == BK_BITS_HBM) {
        block_flush<MODE>(bits_groups_hbm<MODE>(A, items, bu.index, (uint32_t)bu.end, smem), A);
      } else {
        long_rows();
      }
    }
  }
}

template <int MODE>
void launch_batch_mode(const Args* d_args, const BatchUnit* d_units, int64_t n_units, uint32_t chunk,
                       unsigned int* d_queue, unsigned long long* counts, unsigned grid, size_t lds,
                       BatchBodies bodies, hipStream_t st, bool timed) {
  static const char* const kNames[3] = {"count:batch", "support_full:batch", "support_oriented:batch"};
  if (n_units == 0) return;
  auto* f = bodies == BATCH_SHORT  ? k_count_batch<MODE, BATCH_SHORT>
            : bodies == BATCH_LONG ? k_count_batch<MODE, BATCH_LONG>
                                   : k_count_batch<MODE, BATCH_ALL>;
  if (timed)
    TC_LAUNCH(kNames[MODE], f, dim3(grid), dim3(256), lds, st, d_args, d_units, (uint32_t)n_units, chunk, d_queue,
              counts);
  else
    hipLaunchKernelGGL(f, dim3(grid), dim3(256), lds, st, d_args, d_units,
                       (uint32_t)n_units, chunk, d_queue, counts);
}

}  // namespace

size_t pack_lds_bytes(uint32_t slots, int mode) {
  const size_t vals = mode_keys(mode) ? 2 : 1;
  return sizeof(int32_t) * ((size_t)pack_head_words(mode, kWaves) + (size_t)slots * vals);
}

size_t items_lds_bytes(int log2S, int mode) {
  const size_t vals = mode_keys(mode) ? 2 : 1;
  return sizeof(int32_t) * ((size_t)kWavesBig * wave_words(mode) + (log2S < 0 ? 0 : ((size_t)1 << log2S) * vals));
}

size_t pack16_lds_bytes(uint32_t slots, int mode, int waves) {
  return sizeof(int32_t) * ((size_t)pack_head_words(mode, waves) + slots / 2 +
                            (mode_keys(mode) ? (size_t)slots : 0));
}

// Hit counters of a bitmap work-group (FULL): one per key of the class's
// longest row, as far as its 32-bit table would fit LDS.
uint32_t bits_max_keys(int log2S, int mode) {
  return mode_keys(mode) && log2S <= kMaxLog2S ? 1u << (log2S <= 12 ? log2S - 2 : log2S - 1) : 0u;
}

size_t bits_lds_bytes(int64_t n, int log2S, int mode) {
  const size_t words = bitmap_words((int32_t)n);
  return sizeof(int32_t) * ((size_t)kWaves * wave_words(mode) + words + bits_max_keys(log2S, mode)) +
         (mode_keys(mode) ? sizeof(uint16_t) * ((words + 1) & ~(size_t)1) : 0);
}

void launch_batch(CountMode mode, const CountArgs* d_args, const BatchUnit* d_units, int64_t n_units,
                  uint32_t chunk, int64_t n_out, unsigned int* d_queue, int64_t* d_counts, unsigned grid,
                  size_t lds, BatchBodies bodies, hipStream_t st, bool timed) {
  TC_REQUIRE(chunk >= 1, TC_EINVAL, "launch_batch: chunk must be >= 1");
  TC_REQUIRE(mode == MODE_COUNT || mode == MODE_SUPPORT_FULL || mode == MODE_SUPPORT_ORIENTED, TC_EINVAL,
             "launch_batch: unsupported mode");
  auto* counts = reinterpret_cast<unsigned long long*>(d_counts);
  const unsigned cg = (unsigned)std::max<int64_t>(1, div_up(n_out, 256));
  if (timed) TC_LAUNCH("batch_clear", k_batch_clear, dim3(cg), dim3(256), 0, st, counts, n_out, d_queue);
  else hipLaunchKernelGGL(k_batch_clear, dim3(cg), dim3(256), 0, st, counts, n_out, d_queue);
  switch (mode) {
    case MODE_COUNT:
      launch_batch_mode<MODE_COUNT>(d_args, d_units, n_units, chunk, d_queue, counts, grid, lds, bodies, st, timed);
      break;
    case MODE_SUPPORT_FULL:
      launch_batch_mode<MODE_SUPPORT_FULL>(d_args, d_units, n_units, chunk, d_queue, counts, grid, lds, bodies, st, timed);
      break;
    default:
      launch_batch_mode<MODE_SUPPORT_ORIENTED>(d_args, d_units, n_units, chunk, d_queue, counts, grid, lds, bodies,
                                               st, timed);
      break;
  }
  TC_HIP(hipGetLastError());
}

void launch_count(const CountView& v, CountMode mode, int64_t* d_count, int32_t* d_support,
                  int64_t* d_per_shift, hipStream_t st, const VertexCounts* vc) {
  const WorkSet& w = *v.w;
  if (d_count) TC_LAUNCH("zero_i64", k_zero_i64, dim3(1), dim3(1), 0, st, d_count);
  if ((mode == MODE_SUPPORT_FULL || mode == MODE_SUPPORT_ORIENTED) && v.pm > 0)
    TC_LAUNCH("zero_i32", k_zero_i32, dim3((unsigned)div_up(v.pm, 256)), dim3(256), 0, st, d_support,
              v.pm);
  if (mode == MODE_BLOCK && d_per_shift)
    TC_LAUNCH("zero_u64", k_zero_u64, dim3(1), dim3(64), 0, st,
              reinterpret_cast<unsigned long long*>(d_per_shift), (int64_t)v.q);
  TC_HIP(hipGetLastError());
  if (w.n_tasks == 0) return;
  TC_REQUIRE(v.pm < kMaxEdges, TC_EOVERFLOW, "launch_count: probe side of 2^32 - 256 entries or more");
  const bool wide = v.pm > kMaxBufferEdges;
  TC_REQUIRE(!wide || mode != MODE_BLOCK, TC_EOVERFLOW, "launch_count: a rank's probe side of 2^30 entries or more");
  TC_REQUIRE(w.b16 >= w.nrows || v.pcol16 != nullptr, TC_EDEVICE, "launch_count: no short columns");
  Args A{v.hrow_ptr, v.hcol, v.pcol, w.tstart, w.tprefix, w.tbeg, w.tend, w.n_tasks, (uint32_t)v.pm,
         v.pcol16, (int32_t)w.nrows, reinterpret_cast<unsigned long long*>(d_count), d_support,
         reinterpret_cast<unsigned long long*>(d_per_shift), v.q, v.xy, vc ? vc->erow : nullptr,
         vc ? vc->count : nullptr};
  TC_REQUIRE(mode != MODE_VERTEX || (vc && vc->erow && vc->count), TC_EINVAL, "launch_count: no vertex counters");
  TC_REQUIRE(v.hash == 0 || mode == MODE_COUNT, TC_EINVAL, "launch_count: multiplicative hashing counts only");
  TC_REQUIRE(!(wide && v.hash), TC_EOVERFLOW, "launch_count: multiplicative hashing below 2^30 edges only");
  switch (mode) {
    case MODE_COUNT:
      if (v.hash) launch_mode<MODE_COUNT, VAR_MUL>(w, A, st);
      else if (wide) launch_mode<MODE_COUNT, VAR_WIDE>(w, A, st);
      else launch_mode<MODE_COUNT, VAR_BASE>(w, A, st);
      break;
    case MODE_SUPPORT_FULL:
      if (wide) launch_mode<MODE_SUPPORT_FULL, VAR_WIDE>(w, A, st);
      else launch_mode<MODE_SUPPORT_FULL, VAR_BASE>(w, A, st);
      break;
    case MODE_SUPPORT_ORIENTED:
      if (wide) launch_mode<MODE_SUPPORT_ORIENTED, VAR_WIDE>(w, A, st);
      else launch_mode<MODE_SUPPORT_ORIENTED, VAR_BASE>(w, A, st);
      break;
    case MODE_BLOCK: launch_mode<MODE_BLOCK, VAR_BASE>(w, A, st); break;
    case MODE_VERTEX:
      if (wide) launch_mode<MODE_VERTEX, VAR_WIDE>(w, A, st);
      else launch_mode<MODE_VERTEX, VAR_BASE>(w, A, st);
      break;
  }
}

template <int BODIES>
static const void* batch_kernel(CountMode mode) {
  return mode == MODE_COUNT          ? (const void*)k_count_batch<MODE_COUNT, BODIES>
         : mode == MODE_SUPPORT_FULL ? (const void*)k_count_batch<MODE_SUPPORT_FULL, BODIES>
                                     : (const void*)k_count_batch<MODE_SUPPORT_ORIENTED, BODIES>;
}

void batch_kernel_lds(CountMode mode, size_t lds, BatchBodies bodies) {
  if (lds <= 65536) return;
  const void* f = bodies == BATCH_SHORT  ? batch_kernel<BATCH_SHORT>(mode)
                  : bodies == BATCH_LONG ? batch_kernel<BATCH_LONG>(mode)
                                         : batch_kernel<BATCH_ALL>(mode);
  TC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
}

void zero_i32(int32_t* p, int64_t n, hipStream_t st, bool timed) {
  if (n <= 0) return;
  if (timed) TC_LAUNCH("zero_i32", k_zero_i32, dim3((unsigned)div_up(n, 256)), dim3(256), 0, st, p, n);
  else hipLaunchKernelGGL(k_zero_i32, dim3((unsigned)div_up(n, 256)), dim3(256), 0, st, p, n);
}

}  // namespace tc
