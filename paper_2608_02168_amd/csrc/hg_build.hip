// hg_build_csr: risk-aware overlapping-subgraph construction on the GPU.
//
// Steps (Methodology, "Risk-Aware Subgraph Construction"; Algorithm 1,
// construction loop):
//   1. one pass over the edges: range checks, out-degrees, and for every node
//      outside V_k the smallest index of an edge joining it to V_k (either
//      direction) -- a node is a candidate of C_k iff that index exists;
//   2. node keys: out-degree, or the h-index of the out-neighbour multiset
//      (edges sorted by source);
//   3. C'_k = candidates with key <= theta, listed in no order;
//   4. TopM: an exact search by digits for the last of the min(M, |C'_k|)
//      smallest composites (key, splitmix64(seed ^ gid)) -- the hash is a
//      bijection of gid, so composites are unique and so is the selected set;
//   5. local ids in (node type, gid) order from tile counts and ballots (more
//      than two node types: by a stable bucket partition);
//   6. induced-subgraph edge compaction in original edge order (local ids
//      from a 32-byte-per-64-nodes rank table, per-tile counts, ballots);
//   7. stable LSD radix sorts by (dst, r) and (src, r) give the CSR and CSC;
//      row pointers read off the sorted keys; csc_scale = 1/deg_r(dst);
//   8. the execution plan: per-relation active-source lists and the chunked
//      work list of the atomic-free transposed SpMM.
#include <algorithm>
#include <vector>

#include "hg_internal.h"

namespace hg {

namespace {

constexpr int kBT = 256;  // threads per block for the elementwise passes
inline unsigned grid_for(int64_t n, int64_t cap = 16384) {
  int64_t b = cdiv(n > 0 ? n : 1, kBT);
  return (unsigned)(b < cap ? b : cap);
}

__device__ __forceinline__ int64_t cdiv_dev(int64_t a, int64_t b) { return (a + b - 1) / b; }

#define GRID_STRIDE(i, n)                                                        \
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n);     \
       i += (int64_t)gridDim.x * blockDim.x)

// Device counters written by the build.
enum : int { C_ERR = 0, C_NSUB, C_ESUB, C_MSEL, C_ITEMS, C_HEAVY, C_PARTS, C_CPRIME, C_BASE, C_FHEAVY, C_FPARTS,
             C_ASLOTS, C_GAP_CSR, C_GAP_CSC, C_GAP_HI, C_HI_BLOCK,
             C_HI_LONG, C_HI_PARTS, C_COUNT };

// The row-indexed layout of the relation transforms is kept when nq rows cost
// at most kRowLayoutMaxSpread times the a active ones.
__host__ __device__ inline bool row_layout(int64_t nq, int64_t a) { return nq <= kRowLayoutMaxSpread * a; }

// A subgraph that holds three quarters of the graph's nodes or more (|V_k|
// plus the budget) is built the "dense" way: the base edge of every candidate
// is found in the first edge pass, whose LDS tables absorb the hub nodes'
// many edges.  Otherwise the first pass only marks candidates and the base
// edges of the few selected nodes are found with the induced edges.  Both
// give the same outputs.
__host__ __device__ inline bool dense_build(int64_t n_base, int64_t budget, int64_t n_nodes) {
  const int64_t b = budget < n_nodes ? budget : n_nodes;
  return 4 * (n_base + b) >= 3 * n_nodes;
}

// TopM takes the smallest composites (key, splitmix64(seed ^ gid)); the hash is
// a bijection of the gid, so composites are unique.  The search narrows the
// range [lo, hi] that holds the last one taken, a digit of up to 11 bits at a
// time; the selected set is then every candidate up to (khi, hhi).
constexpr int kSelBins = 2048;   // values of a digit
constexpr int kSelSmall = 256;   // a range this small is ranked by one block
enum : uint32_t { S_SEARCH = 0, S_DONE, S_NONE, S_COLLECT, S_RANK };
struct SelectState {
  uint64_t hlo, hhi;  // hash range, when klo == khi
  uint32_t klo, khi;  // key range
  uint32_t k_rem;     // how many to take from the range
  uint32_t mode;      // S_DONE: all of the range; S_NONE: no candidate; S_COLLECT, S_RANK: the range is small
  uint32_t level;     // digit of the next histogram
  uint32_t done;      // blocks of the current launch that have finished
  uint32_t n_small;
  uint32_t pad;
  uint64_t small[kSelSmall][2];  // (key, hash) of a small range
  int32_t hist[kSelBins];
};

__device__ __forceinline__ uint64_t splitmix64_first(uint64_t state) {
  // SplitMix64 (Steele, Lea, Flood 2014): advance by the golden gamma, then
  // the variant-13 finaliser.
  uint64_t z = state + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Digit of a level: small keys whole (0; larger ones share its last value),
// larger keys in three digits (1-3), then the hash from the top (4-9).
__device__ __forceinline__ uint32_t select_digit(uint32_t level, uint32_t key, uint64_t h) {
  switch (level) {
    case 0: return key < kSelBins - 1 ? key : kSelBins - 1;
    case 1: return key >> 21;
    case 2: return (key >> 10) & 2047u;
    case 3: return key & 1023u;
    case 9: return (uint32_t)(h & 511u);
    default: return (uint32_t)(h >> (53 - 11 * (level - 4))) & 2047u;
  }
}

// The range left by digit d of a level, and the next level.
__device__ __forceinline__ void select_narrow(SelectState* st, uint32_t level, uint32_t d) {
  if (level == 0) {
    st->klo = d;
    st->khi = d < kSelBins - 1 ? d : ~0u;
    st->level = d < kSelBins - 1 ? 4 : 1;
  } else if (level <= 3) {
    const int sh = level == 1 ? 21 : (level == 2 ? 10 : 0);
    const uint32_t top = level == 1 ? 0u : st->khi & ~((1u << (level == 2 ? 21 : 10)) - 1u);
    const uint32_t lo = top | (d << sh);
    st->klo = lo > st->klo ? lo : st->klo;
    st->khi = lo | ((1u << sh) - 1u);
    st->level = level + 1;
    if (level == 3) st->klo = st->khi;
  } else {
    const int sh = level == 9 ? 0 : 53 - 11 * ((int)level - 4);
    st->hlo |= (uint64_t)d << sh;
    st->hhi = st->hlo | ((1ull << sh) - 1ull);
    st->level = level + 1;
  }
}

__device__ __forceinline__ bool select_in_range(const SelectState* st, uint32_t key, uint64_t h) {
  if (key < st->klo || key > st->khi) return false;
  return st->klo != st->khi || (h >= st->hlo && h <= st->hhi);
}

// Every node's start: base_bits[v / 32] bit v % 32 = (part[v] == k) (one wave
// covers 64 nodes, two words), first[v] = n_edges, outdeg[v] = 0, the range
// check of its type; |V_k| and the check as one word per block (count, and bit
// 31 for a type out of range), summed by k_init_counts.
__global__ void __launch_bounds__(kBT) k_init_nodes(const int32_t* __restrict__ part, int32_t k,
                                                    const uint8_t* __restrict__ ntype, int32_t n_ntype, int64_t n,
                                                    int32_t n_edges, uint32_t* __restrict__ bits,
                                                    int32_t* __restrict__ first, int32_t* __restrict__ outdeg,
                                                    uint32_t* __restrict__ block_cnt) {
  __shared__ uint32_t wc[kBT / 64];
  uint32_t c = 0;  // the same in every lane of a wave
  GRID_STRIDE(v0, cdiv_dev(n, 64) * 64) {
    const bool live = v0 < n;
    const uint64_t m = __ballot(live && part[v0] == k);
    if (__ballot(live && ntype[v0] >= n_ntype)) c |= 0x80000000u;
    c += (uint32_t)__popcll(m);
    if (live) {
      first[v0] = n_edges;
      outdeg[v0] = 0;
    }
    if ((threadIdx.x & 63) == 0) {
      const int64_t wd = v0 >> 5;
      bits[wd] = (uint32_t)m;
      if ((v0 + 32) < n) bits[wd + 1] = (uint32_t)(m >> 32);
    }
  }
  if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0, bad = 0;
    for (int q = 0; q < kBT / 64; ++q) {
      t += wc[q] & 0x7FFFFFFFu;
      bad |= wc[q] & 0x80000000u;
    }
    block_cnt[blockIdx.x] = t | bad;
  }
}

// One block: the counters' and the selection's start, and the sums of
// k_init_nodes.
__global__ void __launch_bounds__(256) k_init_counts(const uint32_t* __restrict__ block_cnt, int nb,
                                                     int32_t* __restrict__ cnt, SelectState* __restrict__ st) {
  __shared__ uint32_t red[256];
  __shared__ uint32_t bad[256];
  uint32_t t = 0, b = 0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    t += block_cnt[i] & 0x7FFFFFFFu;
    b |= block_cnt[i] >> 31;
  }
  red[threadIdx.x] = t;
  bad[threadIdx.x] = b;
  for (int i = threadIdx.x; i < kSelBins; i += 256) st->hist[i] = 0;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      red[threadIdx.x] += red[threadIdx.x + o];
      bad[threadIdx.x] |= bad[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x < C_COUNT)
    cnt[threadIdx.x] = threadIdx.x == C_BASE ? (int32_t)red[0] : (threadIdx.x == C_ERR && bad[0] ? 2 : 0);
  if (threadIdx.x == 0) {
    st->hlo = 0;
    st->hhi = ~0ull;
    st->klo = 0;
    st->khi = ~0u;
    st->k_rem = 0;
    st->mode = S_SEARCH;
    st->level = 0;
    st->done = 0;
    st->n_small = 0;
  }
}

// Membership of the subgraph's node set: base nodes and selected overlap nodes.
__global__ void k_member_bits(const int32_t* __restrict__ part, int32_t k, const uint8_t* __restrict__ sel,
                              int64_t n, uint32_t* __restrict__ bits) {
  GRID_STRIDE(v0, cdiv_dev(n, 64) * 64) {
    const bool in = v0 < n && (part[v0] == k || sel[v0]);
    const uint64_t m = __ballot(in);
    if ((threadIdx.x & 63) == 0) {
      const int64_t wd = v0 >> 5;
      bits[wd] = (uint32_t)m;
      if ((v0 + 32) < n) bits[wd + 1] = (uint32_t)(m >> 32);
    }
  }
}

// Summary of the base bitmap by groups of 2^sum_shift nodes, at most kSumGroups
// of them: sum[g / 32] bit g % 32 of x: some node of the group is in V_k, of y:
// some node is not.  Both lookups of an edge go to the bitmap only for groups
// that hold nodes of both kinds, else they end in the summary, which the edge
// pass keeps in LDS (8 KB).  The pass was bound by the lookups' L2 requests, one
// per endpoint (1.9 of its 2.7 ms at 200M edges, 211 G requests/s): with a base
// set of contiguous ids, as the prefix sets of the workloads or a partition by
// id ranges, nearly all of them go; with a random partition none do, and the
// LDS reads cost nothing beside the requests.
constexpr int kSumGroups = 1 << 15;
inline int sum_shift(int64_t n) {
  int s = 6;
  while ((n - 1) >> s >= kSumGroups) ++s;
  return s;
}

__global__ void __launch_bounds__(kBT) k_base_summary(const uint32_t* __restrict__ bits, int64_t n, int shift,
                                                      uint2* __restrict__ sum) {
  const int64_t g = (int64_t)blockIdx.x * kBT + threadIdx.x, v0 = g << shift;
  bool in = false, out = false;
  for (int64_t v = v0; v < n && v < v0 + ((int64_t)1 << shift); v += 32) {
    const uint32_t m = bits[v >> 5], all = n - v < 32 ? (1u << (n - v)) - 1u : ~0u;
    in |= (m & all) != 0;
    out |= (m & all) != all;
  }
  const uint64_t mi = __ballot(in), mo = __ballot(out);
  const int h = threadIdx.x & 63;
  if (h < 2 && (g & ~63ll) + 32 * h < kSumGroups) sum[((g & ~63ll) >> 5) + h] = make_uint2((uint32_t)(mi >> (32 * h)), (uint32_t)(mo >> (32 * h)));
}

__device__ __forceinline__ bool bit_of(const uint32_t* __restrict__ bits, int32_t v) {
  return (bits[v >> 5] >> (v & 31)) & 1u;
}

// ---- block-aggregated atomics -----------------------------------------------
// A heavy-tailed graph sends a large share of all edges to a few hub nodes and
// many edges to each of the next thousand or so: one global atomic per edge
// on such a counter serialises (a 1M-node graph whose top source holds 19% of
// 20M edges spent ~18 ms in one such pass).  Each block therefore combines its
// updates in an LDS hash table first (open addressing, 4 probes; integer add or
// min, whose result does not depend on the order) and sends one global
// atomic per table entry when it is done; a key that finds no free slot goes
// straight to the global atomic.  Hot keys arrive early and keep their slots.
constexpr int kAggBits = 11, kAggSlots = 1 << kAggBits;
constexpr uint32_t kAggEmpty = 0xFFFFFFFFu;

template <bool kMin, int kBits = kAggBits>
struct LdsAgg {
  static constexpr int kSlots = 1 << kBits;
  uint32_t* key;  // [kSlots] in LDS
  int32_t* val;
  __device__ __forceinline__ void init() {
    for (int q = threadIdx.x; q < kSlots; q += blockDim.x) {
      key[q] = kAggEmpty;
      val[q] = kMin ? INT32_MAX : 0;
    }
  }
  __device__ __forceinline__ void put(uint32_t k, int32_t v, int32_t* __restrict__ tgt) {
    uint32_t h = (k * 0x9E3779B1u) >> (32 - kBits);
#pragma unroll
    for (int probe = 0; probe < 4; ++probe) {
      // a plain read first: a full table costs loads, not compare-and-swaps
      uint32_t cur = __atomic_load_n(&key[h], __ATOMIC_RELAXED);
      if (cur == kAggEmpty) cur = atomicCAS(&key[h], kAggEmpty, k);
      if (cur == kAggEmpty || cur == k) {
        if (kMin) {
          atomicMin(&val[h], v);
        } else {
          atomicAdd(&val[h], v);
        }
        return;
      }
      h = (h + 1) & (kSlots - 1);
    }
    if (kMin) {
      atomicMin(&tgt[k], v);
    } else {
      atomicAdd(&tgt[k], v);
    }
  }
  // after a __syncthreads: one global atomic per filled slot
  __device__ __forceinline__ void flush(int32_t* __restrict__ tgt) {
    for (int q = threadIdx.x; q < kSlots; q += blockDim.x) {
      const uint32_t k = key[q];
      if (k != kAggEmpty) {
        if (kMin) {
          atomicMin(&tgt[k], val[q]);
        } else {
          atomicAdd(&tgt[k], val[q]);
        }
      }
    }
  }
};

// Launch shape of the aggregation passes: blocks of 512 threads, two per
// compute unit (the edge pass's three tables and the base summary take 56 KB of
// LDS, the out-degree table 64), each working through a long stretch of edges
// before it flushes its tables.
constexpr int kAggBT = 512, kAggPerCu = 2;
inline unsigned agg_grid(int64_t n) {
  const int64_t b = cdiv(n > 0 ? n : 1, kAggBT), cap = (int64_t)num_cus() * kAggPerCu;
  return (unsigned)(b < cap ? b : cap);
}

// The out-degree counts: every edge adds 1 to its source, and with Zipf
// sources a few thousand hubs take most of the edges.  A table of 2^13 slots
// keeps far more of them than the 2^11-slot tables of the pass that holds
// several tables at once.
constexpr int kDegBits = 13, kDegSlots = 1 << kDegBits;
constexpr int kEpItems = 4;

// Range checks and the candidates C_k: every node outside V_k joined to V_k
// by an edge gets first[v] < n_edges -- in a dense build the smallest index of
// such an edge (block-aggregated atomic minimum), otherwise 0 (a plain store:
// every writer stores the same value, and a node already marked is only
// read).  Out-degrees: of the nodes outside V_k when count_out (the out-degree
// key of the candidates, all of which lie outside V_k), else none (the h-index,
// or keys given by the caller).
__global__ void __launch_bounds__(kAggBT) k_edges_pass(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                   const uint8_t* __restrict__ rel,
                                                   const uint32_t* __restrict__ base_bits, int64_t n_nodes,
                                                   int64_t n_edges, int32_t n_rel, int count_out,
                                                   int64_t budget, const uint2* __restrict__ sum, int shift,
                                                   int32_t* __restrict__ outdeg,
                                                   int32_t* __restrict__ first, int32_t* __restrict__ cnt) {
  __shared__ uint2 ls[kSumGroups / 32];
  __shared__ uint32_t lk[3][kAggSlots];
  __shared__ int32_t lv[3][kAggSlots];
  LdsAgg<false> deg{lk[0], lv[0]};
  LdsAgg<true> fs{lk[1], lv[1]}, fd{lk[2], lv[2]};
  const bool exact = dense_build(cnt[C_BASE], budget, n_nodes);
  for (int i = threadIdx.x; i < (int)(((n_nodes - 1) >> shift) >> 5) + 1; i += kAggBT) ls[i] = sum[i];
  if (count_out) deg.init();
  if (exact) {
    fs.init();
    fd.init();
  }
  __syncthreads();
  // kEpItems edges per thread and round (strided by the grid), every load of
  // a round issued before the lookups that depend on it
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e0 < n_edges; e0 += kEpItems * stride) {
    int32_t sv[kEpItems], dv[kEpItems];
    uint32_t rv[kEpItems], ws[kEpItems], wd[kEpItems];
    bool ok[kEpItems], ps[kEpItems], pd[kEpItems];
    // loads without branches (an index past the end reads the last edge and
    // counts for nothing; an endpoint out of range reads word 0), so the
    // loads of all items are in flight together
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      const int64_t e = e0 + j * stride;
      const int64_t ec = e < n_edges ? e : n_edges - 1;
      sv[j] = src[ec];
      dv[j] = dst[ec];
      rv[j] = rel[ec];
    }
    // word 0 of the bitmap stands in where the summary answers (one line for
    // the whole wave)
    uint32_t is[kEpItems], id[kEpItems];
    bool gs[kEpItems], gd[kEpItems], mixs[kEpItems], mixd[kEpItems];
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      ok[j] = sv[j] >= 0 && sv[j] < n_nodes && dv[j] >= 0 && dv[j] < n_nodes;
      const uint32_t a = ok[j] ? (uint32_t)sv[j] >> shift : 0u, b = ok[j] ? (uint32_t)dv[j] >> shift : 0u;
      const uint2 wa = ls[a >> 5], wb = ls[b >> 5];
      gs[j] = (wa.x >> (a & 31)) & 1u;
      gd[j] = (wb.x >> (b & 31)) & 1u;
      mixs[j] = gs[j] && ((wa.y >> (a & 31)) & 1u);
      mixd[j] = gd[j] && ((wb.y >> (b & 31)) & 1u);
      is[j] = ok[j] && mixs[j] ? (uint32_t)sv[j] >> 5 : 0u;
      id[j] = ok[j] && mixd[j] ? (uint32_t)dv[j] >> 5 : 0u;
    }
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      ws[j] = base_bits[is[j]];
      wd[j] = base_bits[id[j]];
    }
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      const int64_t e = e0 + j * stride;
      ok[j] = e < n_edges && ok[j] && rv[j] < (uint32_t)n_rel;
      if (e < n_edges && !ok[j]) atomicOr(&cnt[C_ERR], 1);
      ps[j] = ok[j] && (mixs[j] ? (ws[j] >> (sv[j] & 31)) & 1u : gs[j]);
      pd[j] = ok[j] && (mixd[j] ? (wd[j] >> (dv[j] & 31)) & 1u : gd[j]);
    }
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      if (!ok[j]) continue;
      const int64_t e = e0 + j * stride;
      const int32_t s = sv[j], d = dv[j];
      if (count_out && !ps[j]) deg.put((uint32_t)s, 1, outdeg);
      if (exact) {
        if (pd[j] && !ps[j]) fs.put((uint32_t)s, (int32_t)e, first);
        if (ps[j] && !pd[j]) fd.put((uint32_t)d, (int32_t)e, first);
      } else {
        if (pd[j] && !ps[j] && first[s] != 0) first[s] = 0;
        if (ps[j] && !pd[j] && first[d] != 0) first[d] = 0;
      }
    }
  }
  __syncthreads();
  if (count_out) deg.flush(outdeg);
  if (exact) {
    fs.flush(first);
    fd.flush(first);
  }
}

// The range checks of the edge arrays alone.
__global__ void __launch_bounds__(kBT) k_check_edges(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                     const uint8_t* __restrict__ rel, int64_t n_nodes,
                                                     int64_t n_edges, int32_t n_rel, int32_t* __restrict__ cnt) {
  bool bad = false;
  GRID_STRIDE(e, n_edges) {
    const int32_t s = src[e], d = dst[e];
    bad |= s < 0 || s >= n_nodes || d < 0 || d >= n_nodes || rel[e] >= (uint32_t)n_rel;
  }
  if (bad) atomicOr(&cnt[C_ERR], 1);
}

// Out-degrees of every node, with the range checks of the edge arrays.
__global__ void __launch_bounds__(kAggBT) k_all_outdeg(const int32_t* __restrict__ src,
                                                   const int32_t* __restrict__ dst,
                                                   const uint8_t* __restrict__ rel, int64_t n_nodes,
                                                   int64_t n_edges, int32_t n_rel, int32_t* __restrict__ outdeg,
                                                   int32_t* __restrict__ cnt) {
  __shared__ uint32_t lk[kDegSlots];
  __shared__ int32_t lv[kDegSlots];
  LdsAgg<false, kDegBits> deg{lk, lv};
  deg.init();
  __syncthreads();
  // kEpItems edges per thread and round, all their loads issued first
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e0 < n_edges; e0 += kEpItems * stride) {
    int32_t sv[kEpItems], dv[kEpItems];
    uint32_t rv[kEpItems];
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      const int64_t e = e0 + j * stride;
      const int64_t ec = e < n_edges ? e : n_edges - 1;
      sv[j] = src[ec];
      dv[j] = dst[ec];
      rv[j] = rel[ec];
    }
#pragma unroll
    for (int j = 0; j < kEpItems; ++j) {
      if (e0 + j * stride >= n_edges) continue;
      if (sv[j] < 0 || sv[j] >= n_nodes || dv[j] < 0 || dv[j] >= n_nodes || rv[j] >= (uint32_t)n_rel) {
        atomicOr(&cnt[C_ERR], 1);
        continue;
      }
      deg.put((uint32_t)sv[j], 1, outdeg);
    }
  }
  __syncthreads();
  deg.flush(outdeg);
}

// Row pointers of sorted keys: ptr[q] = the number of keys below q, for q in
// [0, nq].  Every position p whose key differs from its predecessor's owns the
// rows (key[p - 1], key[p]] and the last position also those up to nq; one
// thread takes kRpItems keys a block's width apart, so a wave's keys and most
// of its pointers are consecutive.  A gap of more than kRpInline empty rows
// goes to a list in pieces of kRpPiece rows, filled by k_row_gaps over the
// whole grid (one thread would write a graph's whole tail of nodes without
// out-edges by itself).  Bound by its bytes: at 200M keys and 50M rows 1.0 GB
// in 0.27 ms a sort; counting the rows with LDS and atomics, then scanning the
// 50M counts, took 0.75 ms (fill 0.06, counts 0.33, scan 0.36).
constexpr int kRpItems = 8;
constexpr int kRpInline = 64;

__device__ __forceinline__ void row_gap(int32_t* __restrict__ ptr, int32_t lo, int32_t hi, int32_t p,
                                        int4* __restrict__ gaps, int32_t* __restrict__ n_gaps) {
  if (hi - lo <= kRpInline) {
    for (int32_t q = lo; q < hi; ++q) ptr[q] = p;
    return;
  }
  const int32_t np = gap_pieces(lo, hi);
  const int32_t at = atomicAdd(n_gaps, np);
  for (int32_t i = 0; i < np; ++i) {
    const RowRange r = gap_piece(lo, hi, i);
    gaps[at + i] = make_int4(r.beg, r.end, p, 0);
  }
}

__global__ void __launch_bounds__(kBT) k_row_ptr(const uint32_t* __restrict__ keys, int64_t n, int32_t nq,
                                                 int32_t* __restrict__ ptr, int4* __restrict__ gaps,
                                                 int32_t* __restrict__ n_gaps, const int32_t* __restrict__ err) {
  if (err && *err) return;  // keys may lie past nq
  const int64_t base = (int64_t)blockIdx.x * (kBT * kRpItems) + threadIdx.x;
  const int lane = threadIdx.x & 63;
  int32_t k[kRpItems], head[kRpItems];
#pragma unroll
  for (int j = 0; j < kRpItems; ++j) {
    const int64_t p = base + (int64_t)j * kBT;
    k[j] = (int32_t)keys[p < n ? p : n - 1];
    // the key before the wave's first one (-1 before the first key)
    head[j] = -1;
    if (lane == 0 && p > 0 && p < n) head[j] = (int32_t)keys[p - 1];
  }
#pragma unroll
  for (int j = 0; j < kRpItems; ++j) {
    const int64_t p = base + (int64_t)j * kBT;
    const int32_t up = __shfl_up(k[j], 1, 64);
    const int32_t prev = lane == 0 ? head[j] : up;
    if (p < n) {
      if (k[j] != prev) row_gap(ptr, prev + 1, k[j] + 1, (int32_t)p, gaps, n_gaps);
      if (p == n - 1) row_gap(ptr, k[j] + 1, nq + 1, (int32_t)n, gaps, n_gaps);
    }
  }
}

__global__ void __launch_bounds__(kBT) k_row_gaps(const int4* __restrict__ gaps, const int32_t* __restrict__ n_gaps,
                                                  int32_t* __restrict__ ptr) {
  const int32_t n = *n_gaps;
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int4 g = gaps[i];
    HG_ROW_WALK(q, g.x + threadIdx.x, g.y, kBT) ptr[q] = g.z;
  }
}

// Entries the gap list can hold: gaps longer than kRpInline rows, each a
// piece more than its full pieces.
inline int64_t gap_cap(int64_t nq) { return nq / kRpInline + nq / kRpPiece + 2; }

int row_pointers(const uint32_t* keys, int64_t n, int64_t nq, int32_t* ptr, int4* gaps, int32_t* n_gaps,
                 const int32_t* err, hipStream_t s) {
  if (n <= 0) return fill_i32(ptr, 0, nq + 1, s);
  HG_LAUNCH("build_row_ptr", k_row_ptr, dim3((unsigned)cdiv(n, kBT * kRpItems)), dim3(kBT), 0, s, keys, n, (int32_t)nq,
            ptr, gaps, n_gaps, err);
  const int64_t cap = gap_cap(nq), most = 4 * (int64_t)num_cus();
  HG_LAUNCH("build_row_gaps", k_row_gaps, dim3((unsigned)(cap < most ? cap : most)), dim3(kBT), 0, s,
            (const int4*)gaps, (const int32_t*)n_gaps, ptr);
  return HG_OK;
}

int bits_for(int64_t nvals) {
  int b = 0;
  while (b < 32 && ((int64_t)1 << b) < nvals) ++b;
  return b;
}

// ---- h-index keys ---------------------------------------------------------------
// key[v] = the largest h with at least h out-neighbours (one per edge) of
// out-degree at least h.  The edges are sorted by source, so a node's
// out-neighbours lie together and out-degrees are differences of row pointers;
// one histogram bin per edge and node, filled by a global atomic per edge, took
// 2.3 ms at 50M edges besides the 1.0 ms that counted the degrees, the sort and
// the rows below take 1.5 ms.  h = max_i min(x_i, #{j : x_j >= x_i}), found
//   - for up to kHiSmall neighbours by 16 lanes, all pairs;
//   - up to kHiWave by one wave, a binary search over h on ballots;
//   - up to kHiBlock by one block, longer rows by blocks of kHiPart neighbours
//     each (parts): a histogram of the degrees below kHiBins (values below 8, most of
//     them, counted by ballots), whose suffix sums meet h.
// A row with kHiBins neighbours of degree kHiBins and more has its h above the
// histogram (parallel edges to hubs count each, so h may be as large as the row).
// Ranges of 2^s degrees up to the row's length are counted beside it; the range
// that holds h is found the same way, and further walks, by the parts again,
// count its values, kHiSplit bits at a time: one walk more for rows of up to
// 2.7M neighbours, two for all others.  A walk per kHiBins values of h, in one
// block, took 70 ms for a row of 50M neighbours with h = 9000.
constexpr int kHiSmall = 16, kHiWave = 1024, kHiBlock = 16384, kHiPart = 8192;
constexpr int kHiBins = 4096;
constexpr int kHiRanges = 1344, kHiSplit = 11;
// a row's histogram: degrees below kHiBins, the count of the others, their ranges
constexpr int kHiWords = kHiBins + 1 + kHiRanges;
constexpr int kHiBT = 1024;

__device__ __forceinline__ int32_t deg_of(const int32_t* __restrict__ ptr, int32_t v) { return ptr[v + 1] - ptr[v]; }

// Rows of up to kHiWave neighbours; the longer ones go to lists.  A caller that
// filters by key <= theta needs no key above it: a row with theta + 1 = over
// neighbours of at least that degree among its first 64 gets the key over (most
// rows of more than 16 neighbours end here; at theta = 2 the h-index of 50M
// edges takes 0.3 ms after the sort instead of 0.7).
__global__ void __launch_bounds__(kBT) k_hindex_rows(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                     const int32_t* __restrict__ first, int64_t n, int32_t n_edges,
                                                     int32_t* __restrict__ key, int32_t* __restrict__ list_b,
                                                     int32_t* __restrict__ list_l, int2* __restrict__ parts,
                                                     int32_t* __restrict__ n_list, int32_t over,
                                                     const int32_t* __restrict__ err) {
  if (*err) return;
  const int l = threadIdx.x & 63, sub = l & (kHiSmall - 1), grp = l >> 4;
  const int64_t waves = (int64_t)gridDim.x * (kBT / 64);
  for (int64_t b = (int64_t)blockIdx.x * (kBT / 64) + (threadIdx.x >> 6); b * 64 < n; b += waves) {
    const int64_t v = b * 64 + l;
    const bool want = v < n && (!first || first[v] < n_edges);
    const int32_t beg = want ? ptr[v] : 0;
    const int32_t D = want ? ptr[v + 1] - beg : 0;
    if (want && D == 0) key[v] = 0;
    // four nodes at a time
    for (uint64_t left = __ballot(D > 0 && D <= kHiSmall); left;) {
      int mine = -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (left) {
          const int u = __ffsll((unsigned long long)left) - 1;
          left &= left - 1;
          if (grp == q) mine = u;
        }
      }
      const int from = mine < 0 ? 0 : mine;
      const int32_t mb = __shfl(beg, from, 64), fd = __shfl(D, from, 64), md = mine < 0 ? 0 : fd;
      int32_t x = -1;
      if (sub < md) x = deg_of(ptr, col[mb + sub]);
      int ge = 0;
#pragma unroll
      for (int q = 0; q < kHiSmall; ++q) ge += __shfl(x, (l & ~(kHiSmall - 1)) + q, 64) >= x;
      int h = sub < md ? (x < ge ? x : ge) : 0;
#pragma unroll
      for (int o = kHiSmall / 2; o > 0; o >>= 1) {
        const int y = __shfl_xor(h, o, 64);
        h = h > y ? h : y;
      }
      if (mine >= 0 && sub == 0) key[b * 64 + mine] = h;
    }
    for (uint64_t left = __ballot(D > kHiSmall); left; left &= left - 1) {
      const int u = __ffsll((unsigned long long)left) - 1;
      const int32_t mb = __shfl(beg, u, 64), md = __shfl(D, u, 64);
      if (over <= 64) {
        const int32_t x = l < md ? deg_of(ptr, col[mb + l]) : -1;
        if ((int)__popcll(__ballot(x >= over)) >= over) {
          if (l == 0) key[b * 64 + u] = over;
          continue;
        }
      }
      if (md > kHiWave) {
        if (l != u) continue;
        if (md <= kHiBlock) {
          list_b[atomicAdd(&n_list[0], 1)] = (int32_t)v;
          continue;
        }
        const int32_t at = atomicAdd(&n_list[1], 1), np = (md - 1) / kHiPart + 1;
        const int32_t p0 = atomicAdd(&n_list[2], np);
        list_l[at] = (int32_t)v;
        for (int32_t c = 0; c < np; ++c) parts[p0 + c] = make_int2(at, c);
        continue;
      }
      int32_t x[kHiWave / 64];
#pragma unroll
      for (int q = 0; q < kHiWave / 64; ++q) x[q] = 64 * q + l < md ? col[mb + 64 * q + l] : -1;
#pragma unroll
      for (int q = 0; q < kHiWave / 64; ++q) x[q] = x[q] >= 0 ? deg_of(ptr, x[q]) : -1;
      int lo = 0, hi = md;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        int c = 0;
#pragma unroll
        for (int q = 0; q < kHiWave / 64; ++q)
          if (64 * q < md) c += (int)__popcll(__ballot(x[q] >= mid));
        if (c >= mid) lo = mid; else hi = mid - 1;
      }
      if (l == 0) key[b * 64 + u] = lo;
    }
  }
}

// Calls f with the degrees of neighbours [beg, end), kU of each thread at a time
// (-1 past the end), in all threads of the block.
template <class F>
__device__ __forceinline__ void hindex_walk(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                            int32_t beg, int32_t end, F f) {
  constexpr int kU = 4;
  HG_ROW_WALK(p0, beg, end, kHiBT * kU) {
    int32_t x[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const row_pos p = p0 + j * kHiBT + threadIdx.x;
      x[j] = p < (row_pos)end ? col[p] : -1;
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) x[j] = x[j] >= 0 ? deg_of(ptr, x[j]) : -1;
#pragma unroll
    for (int j = 0; j < kU; ++j) f(x[j]);
  }
}

// Bits of the ranges' width in a row of n neighbours, -1 for one too short to
// need ranges.  The last range takes the degrees past the row's length, so h is
// never in it.
__device__ __forceinline__ int hindex_shift(int32_t n) {
  if (n < kHiBins) return -1;
  int s = 0;
  while ((n - kHiBins) >> s >= kHiRanges - 1) ++s;
  return s;
}

// Adds the degrees of neighbours [beg, end) into the block's histogram.
__device__ __forceinline__ void hindex_add(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                           int32_t beg, int32_t end, int shift, int32_t* lh) {
  constexpr int kLow = 8;
  int32_t low[kLow], many = 0;
#pragma unroll
  for (int t = 0; t < kLow; ++t) low[t] = 0;
  hindex_walk(ptr, col, beg, end, [&](int32_t x) {
#pragma unroll
    for (int t = 0; t < kLow; ++t) low[t] += (int32_t)__popcll(__ballot(x == t));
    many += (int32_t)__popcll(__ballot(x >= kHiBins));
    if (x >= kHiBins) {
      if (shift < 0) return;
      const int r = (x - kHiBins) >> shift;
      atomicAdd(&lh[kHiBins + 1 + (r < kHiRanges ? r : kHiRanges - 1)], 1);
    } else if (x >= kLow) {
      atomicAdd(&lh[x], 1);
    }
  });
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int t = 0; t < kLow; ++t)
      if (low[t]) atomicAdd(&lh[t], low[t]);
    if (many) atomicAdd(&lh[kHiBins], many);
  }
}

// Degrees [lo, lo + 2^shift) hold h, and `above` neighbours have degrees past
// them; h is lo once shift is 0.
struct HiRange {
  uint32_t lo, above;
  int shift;
};

// Bits of the bins in which a range is walked again, and their number.
__device__ __forceinline__ int hindex_bin_shift(const HiRange& r) { return r.shift > kHiSplit ? r.shift - kHiSplit : 0; }
__device__ __forceinline__ int hindex_bins(const HiRange& r) { return 1 << (r.shift - hindex_bin_shift(r)); }

// The last of n <= kHiBins bins, of 2^shift degrees from lo on, whose first
// degree t has #{x >= t} >= t (the first bin has), to all threads of the block.
__device__ __forceinline__ HiRange hindex_meet(const int32_t* bins, int n, uint32_t lo, int shift, uint32_t above,
                                               uint32_t* red, int* best) {
  constexpr int kPer = kHiBins / kHiBT;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int i = kPer - 1; i >= 0; --i) {  // neighbours of bin kPer tid + i and the thread's later ones
    const int b = (int)threadIdx.x * kPer + i;
    sum += b < n ? (uint32_t)bins[b] : 0u;
    c[i] = sum;
  }
  red[threadIdx.x] = sum;
  if (threadIdx.x == 0) *best = 0;
  __syncthreads();
  for (int o = 1; o < kHiBT; o <<= 1) {  // inclusive suffix sums
    const uint32_t u = threadIdx.x + o < kHiBT ? red[threadIdx.x + o] : 0u;
    __syncthreads();
    red[threadIdx.x] += u;
    __syncthreads();
  }
  const uint32_t later = above + (red[threadIdx.x] - sum);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int b = (int)threadIdx.x * kPer + i;
    if (b < n && c[i] + later >= lo + ((uint32_t)b << shift)) atomicMax(best, b);
  }
  __syncthreads();
  const int b = *best;
  // the thread of bin b leaves the neighbours past it in red[0]
  if (b / kPer == (int)threadIdx.x) {
    uint32_t past = later;
#pragma unroll
    for (int i = 1; i < kPer; ++i)
      if (i == b % kPer + 1) past = c[i] + later;
    red[0] = past;
  }
  __syncthreads();
  return {lo + ((uint32_t)b << shift), red[0], shift};
}

// h, or the range that holds it, from a row's histogram.
__device__ __forceinline__ HiRange hindex_first(const int32_t* lh, int shift, uint32_t* red, int* best) {
  const int32_t many = lh[kHiBins];
  if (many < kHiBins) return hindex_meet(lh, kHiBins, 0, 0, (uint32_t)many, red, best);
  return hindex_meet(lh + kHiBins + 1, kHiRanges, kHiBins, shift, 0, red, best);
}

// Counts the neighbours [beg, end) of a range by its bins.
__device__ __forceinline__ void hindex_add_range(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                 int32_t beg, int32_t end, const HiRange& r, int32_t* bins) {
  const int shift = hindex_bin_shift(r);
  hindex_walk(ptr, col, beg, end, [&](int32_t x) {
    const uint32_t at = (uint32_t)x - r.lo;  // past the range for a degree below it
    if (at >> r.shift == 0) atomicAdd(&bins[at >> shift], 1);
  });
}

__global__ void __launch_bounds__(kHiBT) k_hindex_block(const int32_t* __restrict__ ptr,
                                                        const int32_t* __restrict__ col,
                                                        const int32_t* __restrict__ list,
                                                        const int32_t* __restrict__ n_list,
                                                        int32_t* __restrict__ key) {
  __shared__ int32_t lh[kHiWords];
  __shared__ uint32_t red[kHiBT];
  __shared__ int best;
  const int32_t n = n_list[0];
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t v = list[i], beg = ptr[v], end = ptr[v + 1];
    const int shift = hindex_shift(end - beg);
    for (int b = threadIdx.x; b < (shift < 0 ? kHiBins + 1 : kHiWords); b += kHiBT) lh[b] = 0;
    __syncthreads();
    hindex_add(ptr, col, beg, end, shift, lh);
    __syncthreads();
    HiRange r = hindex_first(lh, shift, red, &best);
    while (r.shift > 0) {
      for (int b = threadIdx.x; b < hindex_bins(r); b += kHiBT) lh[b] = 0;
      __syncthreads();
      hindex_add_range(ptr, col, beg, end, r, lh);
      __syncthreads();
      r = hindex_meet(lh, hindex_bins(r), r.lo, hindex_bin_shift(r), r.above, red, &best);
    }
    if (threadIdx.x == 0) key[v] = (int32_t)r.lo;
    __syncthreads();
  }
}

// Long rows: their parts' histograms added into one of kHiWords words per row
// (zeroed here first), then met by a block per row, which writes the key or
// leaves the range that holds it, with zeroed bins, in the row's words (a first
// word of 0: done).  The parts are then walked by those bins, and met again.
enum : int { HI_LO = 0, HI_ABOVE, HI_SHIFT, HI_BIN };
static_assert(HI_BIN + (1 << kHiSplit) <= kHiWords, "a range's bins in the row's words");

__global__ void __launch_bounds__(kHiBT) k_hindex_zero(const int32_t* __restrict__ n_list, int32_t* __restrict__ hist) {
  const int64_t n = (int64_t)n_list[1] * kHiWords;
  GRID_STRIDE(i, n) hist[i] = 0;
}

__device__ __forceinline__ RowRange hindex_part(const int32_t* __restrict__ ptr, int32_t v, int part) {
  const int32_t end = ptr[v + 1], p = ptr[v] + part * kHiPart;
  return {p, end - p < kHiPart ? end : p + kHiPart};
}

__device__ __forceinline__ HiRange hindex_left(const int32_t* row) {
  return {(uint32_t)row[HI_LO], (uint32_t)row[HI_ABOVE], row[HI_SHIFT]};
}

// Ends a row or leaves its range (all threads of a block; the row's words have
// been read).
__device__ __forceinline__ void hindex_leave(const HiRange& r, int32_t* __restrict__ row, int32_t* __restrict__ key) {
  const bool more = r.shift > 0;
  if (threadIdx.x == 0) {
    row[HI_LO] = more ? (int32_t)r.lo : 0;
    row[HI_ABOVE] = (int32_t)r.above;
    row[HI_SHIFT] = r.shift;
    if (!more) *key = (int32_t)r.lo;
  }
  if (more)
    for (int b = threadIdx.x; b < hindex_bins(r); b += kHiBT) row[HI_BIN + b] = 0;
}

__global__ void __launch_bounds__(kHiBT) k_hindex_parts(const int32_t* __restrict__ ptr,
                                                        const int32_t* __restrict__ col,
                                                        const int32_t* __restrict__ list,
                                                        const int2* __restrict__ parts,
                                                        const int32_t* __restrict__ n_list,
                                                        int32_t* __restrict__ hist) {
  __shared__ int32_t lh[kHiWords];
  const int32_t n = n_list[2];
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int2 pt = parts[i];
    const int32_t v = list[pt.x];
    const RowRange p = hindex_part(ptr, v, pt.y);
    for (int b = threadIdx.x; b < kHiWords; b += kHiBT) lh[b] = 0;
    __syncthreads();
    hindex_add(ptr, col, p.beg, p.end, hindex_shift(deg_of(ptr, v)), lh);
    __syncthreads();
    for (int b = threadIdx.x; b < kHiWords; b += kHiBT)
      if (lh[b]) atomicAdd(&hist[(int64_t)pt.x * kHiWords + b], lh[b]);
    __syncthreads();
  }
}

// exact: a key of kHiBins or more may not come out as any other such key.
__global__ void __launch_bounds__(kHiBT) k_hindex_long(const int32_t* __restrict__ ptr,
                                                       const int32_t* __restrict__ list,
                                                       const int32_t* __restrict__ n_list, bool exact,
                                                       int32_t* __restrict__ hist, int32_t* __restrict__ key) {
  __shared__ int32_t lh[kHiWords];
  __shared__ uint32_t red[kHiBT];
  __shared__ int best;
  const int32_t n = n_list[1];
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    int32_t* row = hist + (int64_t)i * kHiWords;
    const int32_t v = list[i];
    for (int b = threadIdx.x; b < kHiWords; b += kHiBT) lh[b] = row[b];
    __syncthreads();
    HiRange r = hindex_first(lh, hindex_shift(deg_of(ptr, v)), red, &best);
    if (!exact) r.shift = 0;
    hindex_leave(r, row, key + v);
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kHiBT) k_hindex_range_parts(const int32_t* __restrict__ ptr,
                                                              const int32_t* __restrict__ col,
                                                              const int32_t* __restrict__ list,
                                                              const int2* __restrict__ parts,
                                                              const int32_t* __restrict__ n_list,
                                                              int32_t* __restrict__ hist) {
  __shared__ int32_t lh[1 << kHiSplit];
  const int32_t n = n_list[2];
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int2 pt = parts[i];
    int32_t* row = hist + (int64_t)pt.x * kHiWords;
    const HiRange r = hindex_left(row);
    if (r.lo == 0) continue;  // the whole block
    const RowRange p = hindex_part(ptr, list[pt.x], pt.y);
    for (int b = threadIdx.x; b < hindex_bins(r); b += kHiBT) lh[b] = 0;
    __syncthreads();
    hindex_add_range(ptr, col, p.beg, p.end, r, lh);
    __syncthreads();
    for (int b = threadIdx.x; b < hindex_bins(r); b += kHiBT)
      if (lh[b]) atomicAdd(&row[HI_BIN + b], lh[b]);
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kHiBT) k_hindex_range(const int32_t* __restrict__ list,
                                                        const int32_t* __restrict__ n_list,
                                                        int32_t* __restrict__ hist, int32_t* __restrict__ key) {
  __shared__ int32_t lh[1 << kHiSplit];
  __shared__ uint32_t red[kHiBT];
  __shared__ int best;
  const int32_t n = n_list[1];
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    int32_t* row = hist + (int64_t)i * kHiWords;
    const HiRange r = hindex_left(row);
    if (r.lo == 0) continue;  // the whole block
    for (int b = threadIdx.x; b < hindex_bins(r); b += kHiBT) lh[b] = row[HI_BIN + b];
    __syncthreads();
    hindex_leave(hindex_meet(lh, hindex_bins(r), r.lo, hindex_bin_shift(r), r.above, red, &best), row, key + list[i]);
    __syncthreads();
  }
}

// Buffers of the h-index: the sort's ping-pong pairs (n_edges each), row
// pointers (n_nodes + 1), the lists of long rows and the longest ones'
// histograms.
struct HindexBufs {
  uint32_t *k0, *k1;
  int32_t *v0, *v1, *ptr, *list_b, *list_l, *hist, *scratch;
  int2* parts;
  int4* gaps;
  int32_t *n_gaps, *n_list;  // zero on entry (one and three words)
};
inline int64_t hindex_list_b(int64_t E) { return E / kHiWave + 1; }
inline int64_t hindex_list_l(int64_t E) { return E / kHiBlock + 1; }
inline int64_t hindex_parts(int64_t E) { return E / kHiPart + hindex_list_l(E); }
inline int64_t hindex_hist_elems(int64_t E) { return hindex_list_l(E) * kHiWords; }

// key[v] for every node with first[v] < n_edges (every node if first is
// null); keys above theta may come out as any value above it.  err: device flag,
// non-zero when an endpoint is out of range (the keys are then unspecified, and
// nothing is read or written out of bounds).
int hindex_keys(const int32_t* src, const int32_t* dst, int64_t N, int64_t E, const int32_t* first, int32_t theta,
                int32_t* key, const HindexBufs& b, const int32_t* err, hipStream_t s) {
  uint32_t* ko;
  int32_t *col, *none;
  HG_TRY(radix_sort_pairs(b.k0, b.k1, b.v0, b.v1, nullptr, nullptr, E, bits_for(N), b.scratch, s, &ko, &col, &none,
                          nullptr, nullptr, nullptr, reinterpret_cast<const uint32_t*>(src), dst));
  HG_TRY(row_pointers(ko, E, N, b.ptr, b.gaps, b.n_gaps, err, s));
  const unsigned cus = (unsigned)num_cus();
  HG_LAUNCH("hindex_rows", k_hindex_rows, dim3(grid_for(N)), dim3(kBT), 0, s, (const int32_t*)b.ptr,
            (const int32_t*)col, first, N, (int32_t)E, key, b.list_b, b.list_l, b.parts, b.n_list,
            theta < HG_THETA_NONE ? theta + 1 : theta, err);
  if (E > kHiWave)
    HG_LAUNCH("hindex_block", k_hindex_block, dim3(2 * cus), dim3(kHiBT), 0, s, (const int32_t*)b.ptr,
              (const int32_t*)col, (const int32_t*)b.list_b, (const int32_t*)b.n_list, key);
  if (E > kHiBlock) {
    // a block per part and per row, as far as there can be any
    const dim3 gp((unsigned)std::min<int64_t>(2 * cus, hindex_parts(E)));
    const dim3 gl((unsigned)std::min<int64_t>(cus, hindex_list_l(E)));
    HG_LAUNCH("hindex_zero", k_hindex_zero, gl, dim3(kHiBT), 0, s, (const int32_t*)b.n_list, b.hist);
    HG_LAUNCH("hindex_parts", k_hindex_parts, gp, dim3(kHiBT), 0, s, (const int32_t*)b.ptr, (const int32_t*)col,
              (const int32_t*)b.list_l, (const int2*)b.parts, (const int32_t*)b.n_list, b.hist);
    const bool exact = theta >= kHiBins;
    HG_LAUNCH("hindex_long", k_hindex_long, gl, dim3(kHiBT), 0, s, (const int32_t*)b.ptr, (const int32_t*)b.list_l,
              (const int32_t*)b.n_list, exact, b.hist, key);
    // the walks that narrow a row's ranges to one degree: bits of its widest range by kHiSplit
    const int walks = !exact ? 0 : (E - kHiBins < ((int64_t)(kHiRanges - 1) << kHiSplit) ? 1 : 2);
    for (int k = 0; k < walks; ++k) {
      HG_LAUNCH("hindex_range_parts", k_hindex_range_parts, gp, dim3(kHiBT), 0, s, (const int32_t*)b.ptr,
                (const int32_t*)col, (const int32_t*)b.list_l, (const int2*)b.parts, (const int32_t*)b.n_list, b.hist);
      HG_LAUNCH("hindex_range", k_hindex_range, gl, dim3(kHiBT), 0, s, (const int32_t*)b.list_l,
                (const int32_t*)b.n_list, b.hist, key);
    }
  }
  return HG_OK;
}

// ---- TopM ---------------------------------------------------------------------
// One launch per digit: each block adds its candidates' digits into an LDS
// histogram and that into the state's; the block that finishes last picks the
// digit holding the k_rem-th smallest and narrows the range.  The first launch
// also finds the candidates (their list is in no order: the search needs only
// the set).  Two hash digits leave about a candidate in four million, one a
// range small enough to rank where there are up to 2^18, and one more launch
// lists that range for the ranking.  Candidates that share a key of 2047 or more
// need three key digits before those, so five launches end the search among up to
// 2^18 candidates and six among 10^9.  With five for all, k_select_finish's one
// block went on with the list: 26 ms at 10M equal keys, where the build takes 3.2
// with small ones.  8 launches of about 4 us where 16 digits of 8 bits took 33;
// one with nothing left to do takes 2.
inline int select_steps(int64_t n) { return n <= ((int64_t)1 << 18) ? 5 : 6; }
constexpr int kSelBT = 256;
constexpr int kSelItems = 8;

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Adds a block's histogram into the state's and tells, to all threads,
// whether the block is the launch's last one.
__device__ __forceinline__ bool select_add(SelectState* st, const int32_t* lh, int* flag) {
  // Everything one block hands to the last (histogram, list count, a small
  // range's composites) goes through device-scope atomics, which are complete
  // once each wave has waited for them; a full fence would write the block's
  // L2 back (the step 42 us instead of 10 at 2M candidates).
  __syncthreads();
  for (int b = threadIdx.x; b < kSelBins; b += kSelBT)
    if (lh[b]) atomicAdd(&st->hist[b], lh[b]);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) *flag = atomicAdd(&st->done, 1u) == gridDim.x - 1;
  __syncthreads();
  return *flag != 0;
}

// The last block: the digit with the k-th smallest of the range.
__device__ __forceinline__ void select_pick(SelectState* st, uint32_t k, int32_t* lh) {
  constexpr int kPer = kSelBins / kSelBT;
  const uint32_t level = st->level;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    uint32_t* h = reinterpret_cast<uint32_t*>(&st->hist[threadIdx.x * kPer + i]);
    c[i] = load_agent(h);
    *h = 0;
    sum += c[i];
  }
  uint32_t* acc = reinterpret_cast<uint32_t*>(lh);
  acc[threadIdx.x] = sum;
  __syncthreads();
  for (int o = 1; o < kSelBT; o <<= 1) {  // inclusive sums
    const uint32_t u = (int)threadIdx.x >= o ? acc[threadIdx.x - o] : 0u;
    __syncthreads();
    acc[threadIdx.x] += u;
    __syncthreads();
  }
  uint32_t lo = acc[threadIdx.x] - sum;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (c[i] > 0 && lo < k && k <= lo + c[i]) {  // one thread
      select_narrow(st, level, (uint32_t)(threadIdx.x * kPer + i));
      st->k_rem = k - lo;
      st->mode = k - lo == c[i] ? S_DONE : (c[i] <= (uint32_t)kSelSmall ? S_COLLECT : S_SEARCH);
    }
    lo += c[i];
  }
  if (threadIdx.x == 0) st->done = 0;
}

// Candidates with key <= theta: their list, their count and the histogram of
// the first digit.
__global__ void __launch_bounds__(kSelBT) k_candidates(const int32_t* __restrict__ first,
                                                       const int32_t* __restrict__ key, int64_t n, int32_t n_edges,
                                                       int32_t theta, int64_t budget, int32_t* __restrict__ list,
                                                       int32_t* __restrict__ cnt, SelectState* __restrict__ st) {
  __shared__ int32_t lh[kSelBins];
  __shared__ int32_t wsum[kSelBT / 64];
  __shared__ int32_t base_s;
  __shared__ int flag;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
  for (int b = threadIdx.x; b < kSelBins; b += kSelBT) lh[b] = 0;
  __syncthreads();
  for (int64_t v0 = (int64_t)blockIdx.x * (kSelBT * kSelItems); v0 < n;
       v0 += (int64_t)gridDim.x * (kSelBT * kSelItems)) {
    bool in[kSelItems];
    int32_t rank[kSelItems];
    int32_t c = 0;
#pragma unroll
    for (int j = 0; j < kSelItems; ++j) {
      const int64_t v = v0 + j * kSelBT + threadIdx.x;
      in[j] = false;
      if (v < n && first[v] < n_edges) {
        const int32_t kv = key[v];
        in[j] = kv <= theta;
        if (in[j]) atomicAdd(&lh[select_digit(0, (uint32_t)kv, 0)], 1);
      }
      const uint64_t m = __ballot(in[j]);
      rank[j] = c + (int32_t)__popcll(m & lt);
      c += (int32_t)__popcll(m);
    }
    if (l == 0) wsum[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t t = 0;
#pragma unroll
      for (int q = 0; q < kSelBT / 64; ++q) {
        const int32_t x = wsum[q];
        wsum[q] = t;
        t += x;
      }
      base_s = t > 0 ? atomicAdd(&cnt[C_CPRIME], t) : 0;
    }
    __syncthreads();
    const int32_t base = base_s + wsum[w];
#pragma unroll
    for (int j = 0; j < kSelItems; ++j)
      if (in[j]) list[base + rank[j]] = (int32_t)(v0 + j * kSelBT + threadIdx.x);
    __syncthreads();
  }
  if (!select_add(st, lh, &flag)) return;
  const int64_t c = (int64_t)load_agent(reinterpret_cast<const uint32_t*>(&cnt[C_CPRIME]));
  const int64_t take = budget < c ? budget : c;
  if (take == 0 || take == c) {  // nothing, or every candidate (the range is all composites)
    for (int b = threadIdx.x; b < kSelBins; b += kSelBT) st->hist[b] = 0;
    if (threadIdx.x == 0) st->mode = take == 0 ? S_NONE : S_DONE;
  } else {
    select_pick(st, (uint32_t)take, lh);
  }
}

// One round of the search by the launch's blocks.
__device__ __forceinline__ void select_round(SelectState* st, const int32_t* __restrict__ list, int64_t c,
                                             const int32_t* __restrict__ key, uint64_t seed, int32_t* lh, int* flag) {
  const uint32_t mode = load_agent(&st->mode);
  const uint32_t level = st->level;
  for (int b = threadIdx.x; b < kSelBins; b += kSelBT) lh[b] = 0;
  __syncthreads();
  GRID_STRIDE(i, c) {
    const uint32_t gid = (uint32_t)list[i];
    const uint32_t kv = (uint32_t)key[gid];
    if (kv < st->klo || kv > st->khi) continue;
    const uint64_t h = splitmix64_first(seed ^ (uint64_t)gid);
    if (!select_in_range(st, kv, h)) continue;
    if (mode == S_COLLECT) {
      const uint32_t at = atomicAdd(&st->n_small, 1u);
      __hip_atomic_store(&st->small[at][0], (uint64_t)kv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&st->small[at][1], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      atomicAdd(&lh[select_digit(level, kv, h)], 1);
    }
  }
  if (!select_add(st, lh, flag)) return;
  if (mode == S_COLLECT) {
    if (threadIdx.x == 0) {
      st->mode = S_RANK;
      st->done = 0;
    }
  } else {
    select_pick(st, st->k_rem, lh);
  }
}

__global__ void __launch_bounds__(kSelBT) k_select_step(SelectState* __restrict__ st, const int32_t* __restrict__ list,
                                                        const int32_t* __restrict__ cnt,
                                                        const int32_t* __restrict__ key, uint64_t seed) {
  __shared__ int32_t lh[kSelBins];
  __shared__ int flag;
  if (st->mode != S_SEARCH && st->mode != S_COLLECT) return;
  select_round(st, list, cnt[C_CPRIME], key, seed, lh, &flag);
}

// One block: what is left of the search (each round narrows the range by a
// digit, and there are ten), then the k_rem-th smallest of a small range.
__global__ void __launch_bounds__(kSelBT) k_select_finish(SelectState* st, const int32_t* __restrict__ list,
                                                          const int32_t* __restrict__ cnt,
                                                          const int32_t* __restrict__ key, uint64_t seed) {
  __shared__ int32_t lh[kSelBins];
  __shared__ uint64_t comp[kSelSmall][2];
  __shared__ int flag;
  for (int round = 0; round < 12; ++round) {
    const uint32_t mode = load_agent(&st->mode);
    if (mode != S_SEARCH && mode != S_COLLECT) break;
    select_round(st, list, cnt[C_CPRIME], key, seed, lh, &flag);
    __threadfence();
    __syncthreads();
  }
  if (load_agent(&st->mode) != S_RANK) return;
  const int n = (int)st->n_small, k = (int)st->k_rem;
  for (int i = threadIdx.x; i < n; i += kSelBT) {
    comp[i][0] = st->small[i][0];
    comp[i][1] = st->small[i][1];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kSelBT) {
    const uint64_t a = comp[i][0], b = comp[i][1];
    int less = 0;
    for (int q = 0; q < n; ++q) less += comp[q][0] < a || (comp[q][0] == a && comp[q][1] < b);
    if (less == k - 1) {  // composites are unique: one thread
      st->khi = (uint32_t)a;
      st->hhi = b;
      st->mode = S_DONE;
    }
  }
}

// Whether a node outside V_k is selected.
__device__ __forceinline__ bool selected(const SelectState* __restrict__ st, uint64_t seed, int32_t first, int32_t key,
                                         int64_t v, int32_t n_edges, int32_t theta) {
  if (first >= n_edges || key > theta || st->mode != S_DONE) return false;
  const uint32_t kv = (uint32_t)key;
  if (kv != st->khi) return kv < st->khi;
  return st->hhi == ~0ull || splitmix64_first(seed ^ (uint64_t)v) <= st->hhi;
}

// Node-set digits for the relabel (more than two node types).
__global__ void k_member_digit(const int32_t* __restrict__ part, int32_t k, const uint8_t* __restrict__ sel,
                               const uint8_t* __restrict__ ntype, int64_t n, uint8_t* __restrict__ digit,
                               int32_t* __restrict__ iota) {
  GRID_STRIDE(v, n) {
    digit[v] = (part[v] == k || sel[v]) ? ntype[v] : (uint8_t)255;
    iota[v] = (int32_t)v;
  }
}

__global__ void k_global2local(const int32_t* __restrict__ l2g, const int32_t* __restrict__ type_off,
                               int32_t n_ntype, int32_t* __restrict__ g2l, int32_t* __restrict__ cnt) {
  const int64_t ns = type_off[n_ntype];
  if (blockIdx.x == 0 && threadIdx.x == 0) cnt[C_NSUB] = (int32_t)ns;
  GRID_STRIDE(i, ns) { g2l[l2g[i]] = (int32_t)i; }
}

__global__ void k_overlap_flags(const int32_t* __restrict__ l2g, const uint8_t* __restrict__ sel,
                                const int32_t* __restrict__ cnt, int64_t n, int32_t* __restrict__ flag) {
  const int64_t ns = cnt[C_NSUB];
  GRID_STRIDE(i, n) { flag[i] = (i < ns && sel[l2g[i]]) ? 1 : 0; }
}

__global__ void k_overlap_fill(const int32_t* __restrict__ l2g, const int32_t* __restrict__ flag,
                               const int32_t* __restrict__ pos, const int32_t* __restrict__ cnt,
                               const int32_t* __restrict__ part, int32_t* __restrict__ overlap,
                               int32_t* __restrict__ home) {
  const int64_t ns = cnt[C_NSUB];
  GRID_STRIDE(i, ns) {
    if (flag[i]) {
      const int32_t p = pos[i];
      overlap[p] = (int32_t)i;
      home[p] = part[l2g[i]];
    }
  }
}

// The relation of every overlap node's base edge (after the induced edges,
// which find it in a sparse build).
__global__ void k_overlap_rel(const int32_t* __restrict__ l2g, const int32_t* __restrict__ overlap,
                              const int32_t* __restrict__ cnt, const int32_t* __restrict__ first,
                              const uint8_t* __restrict__ rel, uint8_t* __restrict__ orel) {
  if (cnt[C_ERR]) return;
  const int64_t m = cnt[C_MSEL];
  GRID_STRIDE(p, m) orel[p] = rel[first[l2g[overlap[p]]]];
}

// ---- induced edges from a rank table (node types 0 and 1) ------------------
// Local ids order the node set by (type, gid).  For 32 consecutive gids an
// entry holds the masks of their type-0 and type-1 members and the number of
// type-0 and type-1 members before them (16 bytes per 32 nodes, 5 MB for 10M
// nodes, where global2local takes 40 MB), so
//   local(v) = pre0 + popc(mem0 below v)                          (type 0)
//   local(v) = type_off[1] + pre1 + popc(mem1 below v)            (type 1)
// and -1 outside the node set: one 16-byte load per endpoint.
struct __align__(16) RankEnt {
  uint32_t mem0, mem1, pre0, pre1;
};
constexpr int kRankGroup = 32;

// Tiles of kNTile nodes, kNTile / 4 consecutive ones per wave.  k_nodes_count
// finds the selected nodes (and gives first[] of them back to n_edges in a
// sparse build, for the base-edge minimum of the induced-edge pass), writes the
// rank table's masks and the selected nodes' bits, and the tile's counts of
// type-0 and type-1 members and of type-0 and type-1 selected nodes as four
// streams of one count per tile; a scan of the four later, k_nodes_assign
// writes local ids both ways, the overlap with its home blocks, the rank
// table's counts and the type ranges.  Two passes over the nodes (25 bytes
// each); a partition by type, a fill, flags and three scans over all nodes took
// 0.25 ms more at 10M nodes, and 20 launches more at any size.
constexpr int kNRounds = 8;
constexpr int kNTile = kBT * kNRounds;

__global__ void __launch_bounds__(kBT) k_nodes_count(const uint32_t* __restrict__ base_bits,
                                                     const uint8_t* __restrict__ ntype, int32_t* __restrict__ first,
                                                     const int32_t* __restrict__ key,
                                                     const SelectState* __restrict__ st, uint64_t seed, int64_t n,
                                                     int32_t n_edges, int32_t theta, int64_t budget,
                                                     const int32_t* __restrict__ cnt, RankEnt* __restrict__ rt,
                                                     uint64_t* __restrict__ sel_bits, uint8_t* __restrict__ sel,
                                                     int64_t tiles, int32_t* __restrict__ tcnt) {
  __shared__ int32_t wtot[kBT / 64][4];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t v00 = (int64_t)blockIdx.x * kNTile + w * (64 * kNRounds);
  const bool sparse = !dense_build(cnt[C_BASE], budget, n);
  int32_t c[4] = {0, 0, 0, 0};
#pragma unroll 2
  for (int j = 0; j < kNRounds; ++j) {
    const int64_t v = v00 + 64 * j + l;
    const bool live = v < n;
    const bool base = live && bit_of(base_bits, (int32_t)v);
    const bool s = live && !base && selected(st, seed, first[v], key[v], v, n_edges, theta);
    const uint64_t m = __ballot(base || s), ms = __ballot(s);
    const uint64_t m1 = __ballot(live && ntype[v] == 1) & m, m0 = m & ~m1;
    if (sparse && s) first[v] = n_edges;
    if (sel && live) sel[v] = s ? 1 : 0;
    if (l < 2 && 64 * j + v00 < n) {  // lane h writes group 2 (v / 64) + h, the half h of the wave's 64 nodes
      const int64_t b = (v >> 6) * 2 + l;
      rt[b].mem0 = (uint32_t)(m0 >> (32 * l));
      rt[b].mem1 = (uint32_t)(m1 >> (32 * l));
      if (l == 0) sel_bits[v >> 6] = ms;
    }
    c[0] += (int32_t)__popcll(m0);
    c[1] += (int32_t)__popcll(m1);
    c[2] += (int32_t)__popcll(m0 & ms);
    c[3] += (int32_t)__popcll(m1 & ms);
  }
  if (l < 4) wtot[w][l] = l == 0 ? c[0] : (l == 1 ? c[1] : (l == 2 ? c[2] : c[3]));
  __syncthreads();
  if (threadIdx.x < 4) {
    int32_t t = 0;
#pragma unroll
    for (int q = 0; q < kBT / 64; ++q) t += wtot[q][threadIdx.x];
    tcnt[threadIdx.x * tiles + blockIdx.x] = t;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) tcnt[4 * tiles] = 0;  // the scan's end
}

__global__ void __launch_bounds__(kBT) k_nodes_assign(RankEnt* __restrict__ rt, const uint64_t* __restrict__ sel_bits,
                                                      const int32_t* __restrict__ part, int64_t n, int32_t n_ntype,
                                                      int64_t tiles, const int32_t* __restrict__ S,
                                                      int32_t* __restrict__ l2g, int32_t* __restrict__ g2l,
                                                      int32_t* __restrict__ type_off, int32_t* __restrict__ type_copy,
                                                      int32_t* __restrict__ overlap, int32_t* __restrict__ home,
                                                      int32_t* __restrict__ cnt) {
  __shared__ int32_t wtot[kBT / 64][4];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
  const int64_t tile = blockIdx.x, v00 = tile * kNTile + w * (64 * kNRounds);
  const int32_t n0 = S[tiles] - S[0], o0 = S[3 * tiles] - S[2 * tiles];
  const int32_t ns = S[2 * tiles] - S[0], ms_all = S[4 * tiles] - S[2 * tiles];
  // the wave's groups: lane j < kNRounds holds the masks of its nodes 64 j .. 64 j + 63
  uint64_t g0 = 0, g1 = 0, gs = 0;
  if (l < kNRounds && v00 + 64 * l < n) {
    const uint4 a = reinterpret_cast<const uint4*>(rt)[((v00 >> 6) + l) * 2];
    const uint4 b = reinterpret_cast<const uint4*>(rt)[((v00 >> 6) + l) * 2 + 1];
    g0 = ((uint64_t)b.x << 32) | a.x;
    g1 = ((uint64_t)b.y << 32) | a.y;
    gs = sel_bits[(v00 >> 6) + l];
  }
  const int32_t pc[4] = {(int32_t)__popcll(g0), (int32_t)__popcll(g1), (int32_t)__popcll(g0 & gs),
                         (int32_t)__popcll(g1 & gs)};
  int32_t pre[4];  // in lane j: before group j, inside the wave
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int32_t inc = pc[i];
#pragma unroll
    for (int o = 1; o < kNRounds; o <<= 1) {
      const int32_t u = __shfl_up(inc, o, 64);
      if (l >= o) inc += u;
    }
    pre[i] = inc - pc[i];
    if (l == kNRounds - 1) wtot[w][i] = inc;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    pre[i] += S[i * tiles + tile] - S[i * tiles];
    for (int q = 0; q < w; ++q) pre[i] += wtot[q][i];
  }
  if (l < kNRounds && v00 + 64 * l < n) {
    RankEnt* e = rt + ((v00 >> 6) + l) * 2;
    e[0].pre0 = (uint32_t)pre[0];
    e[0].pre1 = (uint32_t)pre[1];
    e[1].pre0 = (uint32_t)(pre[0] + __popc((uint32_t)g0));
    e[1].pre1 = (uint32_t)(pre[1] + __popc((uint32_t)g1));
  }
#pragma unroll
  for (int j = 0; j < kNRounds; ++j) {
    const int64_t v = v00 + 64 * j + l;
    const uint64_t m0 = __shfl(g0, j, 64), m1 = __shfl(g1, j, 64), ms = __shfl(gs, j, 64);
    const int32_t p0 = __shfl(pre[0], j, 64), p1 = __shfl(pre[1], j, 64);
    const int32_t q0 = __shfl(pre[2], j, 64), q1 = __shfl(pre[3], j, 64);
    const bool t0 = (m0 >> l) & 1ull, t1 = (m1 >> l) & 1ull;
    if (v < n) {
      const int32_t id = t0 ? p0 + (int32_t)__popcll(m0 & lt) : (t1 ? n0 + p1 + (int32_t)__popcll(m1 & lt) : -1);
      g2l[v] = id;
      if (id >= 0) l2g[id] = (int32_t)v;
      if ((ms >> l) & 1ull) {
        const int32_t at = t0 ? q0 + (int32_t)__popcll(m0 & ms & lt) : o0 + q1 + (int32_t)__popcll(m1 & ms & lt);
        overlap[at] = id;
        home[at] = part[v];
      }
    }
  }
  if (tile == 0 && threadIdx.x == 0) {
    cnt[C_NSUB] = ns;
    cnt[C_MSEL] = ms_all;
    for (int t = 0; t <= n_ntype; ++t) type_off[t] = type_copy[t] = t == 0 ? 0 : (t < n_ntype ? n0 : ns);
  }
}

// The local id of v from its group's entry (already loaded), -1 outside.
__device__ __forceinline__ int32_t rank_of(uint4 a, int32_t off1, int32_t v) {
  const uint32_t bit = 1u << (v & 31), below = bit - 1u;
  const int32_t r0 = (int32_t)a.z + __popc(a.x & below);
  const int32_t r1 = off1 + (int32_t)a.w + __popc(a.y & below);
  return (a.x & bit) ? r0 : ((a.y & bit) ? r1 : -1);
}

// Edges in tiles of kETile = 16 rounds of kBT consecutive edges (round j of a
// tile: edges base + kBT j .. + kBT - 1, one per thread, coalesced).
constexpr int kERounds = 16;
constexpr int kETile = kBT * kERounds;

// The CSR entry of every kept edge at its edge index: key dst_local * R + r
// and the source's local id (and the edge id or weight when the sort
// carries one); a bit per edge, set when the edge is kept (both endpoints in
// the node set, not after the snapshot cut: keep[e / 64] bit e % 64, one
// ballot per wave and round); and the number of kept edges per tile.  When
// every edge is kept the entries are the sort's input as they stand;
// otherwise k_edge_emit compacts them.  In a sparse build also the base edge
// of every selected node: the smallest index of an edge of the node set
// joining it to V_k (atomic minimum; the selected nodes are few and of small
// key).  Bound by the lookups' L2 requests (147 G/s at 200M edges); the edges and
// entries pass by with non-temporal loads and stores, which leaves the cache to
// the table (2.79 to 2.73 ms at 200M edges, 0.18 to 0.15 ms at 20M); half the
// table would give 2.36 ms.
template <bool kTs, bool kW>
__global__ void __launch_bounds__(kBT) k_edge_ids(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                  const uint8_t* __restrict__ rel, int32_t n_rel,
                                                  const RankEnt* __restrict__ rt, const int32_t* __restrict__ type_off,
                                                  const uint32_t* __restrict__ base_bits, const int32_t* __restrict__ ts,
                                                  int32_t t_cut, int64_t n_edges, int64_t n_nodes, int64_t budget,
                                                  const int32_t* __restrict__ cnt,
                                                  uint32_t* __restrict__ kcsr, int32_t* __restrict__ vsrc,
                                                  int32_t* __restrict__ veid, const float* __restrict__ edge_w,
                                                  int32_t* __restrict__ vw, uint64_t* __restrict__ keep_bits,
                                                  int32_t* __restrict__ tile_cnt, int32_t* __restrict__ first) {
  __shared__ int32_t wsum[kBT / 64];
  if (cnt[C_ERR]) return;  // an endpoint out of range: no lookups
  const int64_t base = (int64_t)blockIdx.x * kETile;
  const int32_t off1 = type_off[1];
  const bool sparse = !dense_build(cnt[C_BASE], budget, n_nodes);
  int32_t c = 0;
  // kEiItems rounds at a time, each phase's loads issued for all of them
  // before any is used: the endpoints (with relation, weight and timestamp),
  // then the sources' rank entries, then the destinations' (looked up only
  // for an edge whose source is in the node set -- in a sparse build most
  // are not -- and neither for an edge after the snapshot cut in a dense
  // build; a sparse build still needs such an edge for the base edges)
  constexpr int kEiItems = 4;
  for (int j0 = 0; j0 < kERounds; j0 += kEiItems) {
    int32_t sv[kEiItems], dv[kEiItems], wv[kEiItems];
    uint32_t rv[kEiItems];
    bool in[kEiItems], late[kEiItems];
#pragma unroll
    for (int u = 0; u < kEiItems; ++u) {
      // past the end: the last edge's loads, and nothing kept
      const int64_t e = base + (int64_t)(j0 + u) * kBT + threadIdx.x;
      in[u] = e < n_edges;
      const int64_t ec = in[u] ? e : n_edges - 1;
      sv[u] = __builtin_nontemporal_load(src + ec);
      dv[u] = __builtin_nontemporal_load(dst + ec);
      rv[u] = __builtin_nontemporal_load(rel + ec);
      wv[u] = kW ? __float_as_int(edge_w[ec]) : 0;
      late[u] = kTs ? ts[ec] > t_cut : false;
    }
    uint4 ra[kEiItems];
#pragma unroll
    for (int u = 0; u < kEiItems; ++u) {
      ra[u] = uint4{0u, 0u, 0u, 0u};
      if (in[u] && !(late[u] && !sparse)) ra[u] = *reinterpret_cast<const uint4*>(rt + (sv[u] >> 5));
    }
    int32_t a[kEiItems];
#pragma unroll
    for (int u = 0; u < kEiItems; ++u) a[u] = rank_of(ra[u], off1, sv[u]);
    uint4 rb[kEiItems];
#pragma unroll
    for (int u = 0; u < kEiItems; ++u) {
      rb[u] = uint4{0u, 0u, 0u, 0u};
      if (a[u] >= 0) rb[u] = *reinterpret_cast<const uint4*>(rt + (dv[u] >> 5));
    }
#pragma unroll
    for (int u = 0; u < kEiItems; ++u) {
      const int64_t e = base + (int64_t)(j0 + u) * kBT + threadIdx.x;
      const int32_t b = a[u] >= 0 ? rank_of(rb[u], off1, dv[u]) : -1;
      if (sparse && a[u] >= 0 && b >= 0) {
        const bool ps = bit_of(base_bits, sv[u]), pd = bit_of(base_bits, dv[u]);
        if (pd && !ps) atomicMin(&first[sv[u]], (int32_t)e);
        if (ps && !pd) atomicMin(&first[dv[u]], (int32_t)e);
      }
      const bool keep = !late[u] && a[u] >= 0 && b >= 0;
      if (keep) {
        __builtin_nontemporal_store((uint32_t)b * (uint32_t)n_rel + rv[u], kcsr + e);
        __builtin_nontemporal_store(a[u], vsrc + e);
        if (veid) veid[e] = (int32_t)e;
        if (kW) vw[e] = wv[u];
      }
      const uint64_t kb = __ballot(keep);
      // the wave's 64 edges start at a multiple of 64 (tiles of kETile)
      if ((threadIdx.x & 63) == 0 && base + (int64_t)(j0 + u) * kBT + (threadIdx.x & ~63) < n_edges)
        keep_bits[(base + (int64_t)(j0 + u) * kBT + threadIdx.x) >> 6] = kb;
      c += __popcll(kb);
    }
  }
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
#pragma unroll
    for (int q = 0; q < kBT / 64; ++q) t += wsum[q];
    tile_cnt[blockIdx.x] = t;
  }
}

// Stable compaction of the kept CSR entries of a tile at tile_off[tile]
// (exclusive scan of the tile counts): the rank of a kept entry is the
// number of kept entries before it in (round, wave, lane) order, i.e. in
// edge order.  v2 / o2: the second sort value (edge id or weight), or null.
__global__ void __launch_bounds__(kBT) k_edge_emit(const uint32_t* __restrict__ kin, const int32_t* __restrict__ v1,
                                                   const int32_t* __restrict__ v2,
                                                   const uint64_t* __restrict__ keep_bits, int64_t n_edges,
                                                   const int32_t* __restrict__ tile_off, uint32_t* __restrict__ kout,
                                                   int32_t* __restrict__ o1, int32_t* __restrict__ o2) {
  constexpr int NW = kBT / 64;
  __shared__ int32_t cnt[kERounds * NW];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
  const int64_t base = (int64_t)blockIdx.x * kETile;
  uint64_t bal[kERounds];
#pragma unroll
  for (int j = 0; j < kERounds; ++j) {
    const int64_t e0 = base + (int64_t)j * kBT + 64 * w;
    bal[j] = e0 < n_edges ? keep_bits[e0 >> 6] : 0ull;
    if (l == 0) cnt[j * NW + w] = (int32_t)__popcll(bal[j]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // exclusive prefix in (round, wave) order
    int32_t run = 0;
    for (int q = 0; q < kERounds * NW; ++q) {
      const int32_t c = cnt[q];
      cnt[q] = run;
      run += c;
    }
  }
  __syncthreads();
  const int32_t t0 = tile_off[blockIdx.x];
#pragma unroll
  for (int j = 0; j < kERounds; ++j) {
    if ((bal[j] >> l) & 1ull) {
      const int64_t e = base + (int64_t)j * kBT + threadIdx.x;
      const int32_t p = t0 + cnt[j * NW + w] + (int32_t)__popcll(bal[j] & lt);
      kout[p] = kin[e];
      o1[p] = v1[e];
      if (v2) o2[p] = v2[e];
    }
  }
}

// Keep flag of every edge: both endpoints in the node set (two lookups in the
// membership bitmap, N/8 bytes, which stays in the L2 cache).  With
// timestamps, an edge after the cut is dropped like an edge that leaves the
// node set.
// An edge of the node set (timestamps aside) between a selected node and a
// base node is a candidate edge of the selected node: the smallest such index
// is its base edge (atomic minimum; selected nodes are few and of small key).
__global__ void k_edge_keep(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                            const uint32_t* __restrict__ member, const uint32_t* __restrict__ base_bits,
                            const int32_t* __restrict__ ts, int32_t t_cut, int64_t n_edges,
                            int32_t* __restrict__ keep, int32_t* __restrict__ first,
                            const int32_t* __restrict__ cnt) {
  if (cnt[C_ERR]) return;
  GRID_STRIDE(e, n_edges) {
    const int32_t s = src[e], d = dst[e];
    const bool in = bit_of(member, s) && bit_of(member, d);
    if (in) {
      const bool ps = bit_of(base_bits, s), pd = bit_of(base_bits, d);
      if (pd && !ps) atomicMin(&first[s], (int32_t)e);
      if (ps && !pd) atomicMin(&first[d], (int32_t)e);
    }
    keep[e] = (in && !(ts && ts[e] > t_cut)) ? 1 : 0;
  }
}

// Stable compaction of the kept edges (pos = exclusive scan of keep,
// pos[n_edges] = their count); the local ids of a kept edge's endpoints are
// gathered here, so an edge that leaves the node set costs no lookup.
__global__ void k_edge_compact(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                               const int32_t* __restrict__ g2l, const uint8_t* __restrict__ rel,
                               const int32_t* __restrict__ pos, int64_t n_edges, int32_t n_rel,
                               uint32_t* __restrict__ kcsr, int32_t* __restrict__ vsrc, int32_t* __restrict__ veid,
                               const float* __restrict__ edge_w, int32_t* __restrict__ vw,
                               const int32_t* __restrict__ cnt) {
  if (cnt[C_ERR]) return;
  GRID_STRIDE(e, n_edges) {
    const int32_t p = pos[e];
    if (pos[e + 1] != p) {
      kcsr[p] = (uint32_t)g2l[dst[e]] * (uint32_t)n_rel + (uint32_t)rel[e];
      vsrc[p] = g2l[src[e]];
      if (veid) veid[p] = (int32_t)e;
      if (vw) vw[p] = __float_as_int(edge_w[e]);
    }
  }
}

// The CSC sort's input, taken from the CSR in its order: the key (source, r)
// = csr_col[p] * R + r and, as the value, the destination with the in-degree
// of its row, read from csr_ptr while the row is at hand (rows arrive in
// order).  packed: value = destination | min(deg, 255) << 24 (destinations
// below 2^24), which the sort's last pass unpacks into csc_row and the scale;
// else the destination and, as a second value, the scale w / deg itself (a
// correctly rounded float32 quotient; w = the entry's weight, or 1).  A
// stable sort of this input by its key lists a CSC row by (destination,
// original edge index).  Each thread takes kCiItems entries, one per round of
// the block, all loads of a round issued before any store.
constexpr int kCiItems = 4;
__global__ void __launch_bounds__(kBT) k_csc_input(const uint32_t* __restrict__ kcsr,
                                                   const int32_t* __restrict__ csr_col,
                                                   const int32_t* __restrict__ csr_ptr,
                                                   const float* __restrict__ csr_w, int64_t n, int32_t n_rel,
                                                   int packed, uint32_t* __restrict__ kcsc, int32_t* __restrict__ v1,
                                                   int32_t* __restrict__ v2) {
  const int64_t base = (int64_t)blockIdx.x * (kBT * kCiItems) + threadIdx.x;
  uint32_t key[kCiItems];
  int32_t col[kCiItems], lo[kCiItems], hi[kCiItems];
#pragma unroll
  for (int j = 0; j < kCiItems; ++j) {
    const int64_t p = base + (int64_t)j * kBT;
    key[j] = p < n ? kcsr[p] : 0u;
    col[j] = p < n ? csr_col[p] : 0;
  }
#pragma unroll
  for (int j = 0; j < kCiItems; ++j) {
    const int64_t p = base + (int64_t)j * kBT;
    lo[j] = p < n ? csr_ptr[key[j]] : 0;
    hi[j] = p < n ? csr_ptr[key[j] + 1] : 1;
  }
#pragma unroll
  for (int j = 0; j < kCiItems; ++j) {
    const int64_t p = base + (int64_t)j * kBT;
    if (p < n) {
      const uint32_t dst = key[j] / (uint32_t)n_rel, r = key[j] - dst * (uint32_t)n_rel;
      const int32_t deg = hi[j] - lo[j];
      kcsc[p] = (uint32_t)col[j] * (uint32_t)n_rel + r;
      if (packed) {
        v1[p] = (int32_t)(dst | ((uint32_t)(deg < 255 ? deg : 255) << 24));
      } else {
        v1[p] = (int32_t)dst;
        v2[p] = __float_as_int((csr_w ? csr_w[p] : 1.0f) / (float)deg);
      }
    }
  }
}

__global__ void k_gather_w(const int32_t* __restrict__ eid, const float* __restrict__ edge_w, int64_t n,
                           float* __restrict__ out) {
  GRID_STRIDE(p, n) out[p] = edge_w[eid[p]];
}

// ---- execution plan -----------------------------------------------------------
// Tiles of kPN consecutive nodes (kPN * R rows of the CSC: whole 64-row groups
// of the slot table).  k_plan_count writes, per tile, the number of active rows,
// the long destination rows and their chunks, the split rows and their pieces per
// block of both cuts, the entries split by blocks, and the active sources of every
// relation, as P_REL + R streams of one count per tile laid end to end; one scan
// of the whole turns a stream's entry minus its first into the tile's offset
// (sums may wrap, differences do not).  k_plan_fill takes the cut that pays, forms
// the in-tile ranks again from ballots and writes the plan.  Two reads of csc_ptr
// and the plan's own bytes bound it; digits, counts and source ids per row (17
// bytes a row) with four scans over all rows and a partition by relation took 1.6
// ms at 50M rows where this takes 0.6 ms.
constexpr int kPN = kBT;
constexpr int kPW = kPN / 64;
enum : int { P_ACT = 0, P_FHEAVY, P_FPARTS, P_HEAVY, P_PARTS, P_LHEAVY, P_LPARTS, P_SPLIT, P_REL };

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Exclusive sum over the lanes of a wave.
__device__ __forceinline__ int wave_before(int v) {
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(inc, o, 64);
    if ((int)(threadIdx.x & 63) >= o) inc += u;
  }
  return inc - v;
}

// Bit of tile row w (w = node * R + r inside the tile) in the tile's masks.
__device__ __forceinline__ bool tile_bit(const uint64_t* mask, int w) { return (mask[w >> 6] >> (w & 63)) & 1ull; }

__global__ void __launch_bounds__(kBT) k_plan_count(const int32_t* __restrict__ csc_ptr,
                                                    const int32_t* __restrict__ csr_ptr, int64_t ns, int32_t R,
                                                    PlanCut cut, int64_t tiles, int32_t* __restrict__ cnt) {
  __shared__ uint64_t mask[kPW * HG_MAX_REL];
  __shared__ int32_t wcnt[kPW][HG_MAX_REL];
  __shared__ int32_t wtot[kPW][P_REL];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t tile = blockIdx.x, nq = ns * R;
  const PlanCut len_cut = by_length(cut);
  int act = 0, heavy = 0, parts = 0, lheavy = 0, lparts = 0, split = 0;
  for (int g = 0; g < R; ++g) {  // the wave's 64 nodes: R groups of 64 rows
    const int64_t q = (tile * kPN + 64 * w) * R + 64 * g + l;
    const int32_t len = q < nq ? csc_ptr[q + 1] - csc_ptr[q] : 0;
    const uint64_t m = __ballot(len > 0);
    if (l == 0) mask[w * R + g] = m;
    const int m_row = cuts_of(len, cut), l_row = cuts_of(len, len_cut);
    act += len > 0;
    heavy += m_row > 0;
    parts += m_row;
    split += m_row > 0 ? len : 0;
    lheavy += l_row > 0;
    lparts += l_row;
  }
  const int64_t j = tile * kPN + threadIdx.x;
  const int fch = j < ns ? fwd_chunks_of(csr_ptr[(j + 1) * R] - csr_ptr[j * R]) : 0;
  const int v[P_REL] = {act, fch > 0, fch, heavy, parts, lheavy, lparts, split};
#pragma unroll
  for (int i = 0; i < P_REL; ++i) {
    const int t = wave_sum(v[i]);
    if (l == 0) wtot[w][i] = t;
  }
  // per relation, from the masks the wave's first lane wrote
  __builtin_amdgcn_wave_barrier();
  for (int r = 0; r < R; ++r) {
    const uint64_t m = __ballot(tile_bit(mask, (64 * w + l) * R + r));
    if (l == 0) wcnt[w][r] = (int32_t)__popcll(m);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < P_REL + R; i += kBT) {
    int32_t t = 0;
#pragma unroll
    for (int q = 0; q < kPW; ++q) t += i < P_REL ? wtot[q][i] : wcnt[q][i - P_REL];
    cnt[(int64_t)i * tiles + tile] = t;
  }
  if (tile == 0 && threadIdx.x == 0) cnt[(int64_t)(P_REL + R) * tiles] = 0;  // the scan's end: the grand total
}

struct PlanOut {
  int4 *items, *heavy, *fitems, *fheavy;
  int32_t *act, *act_off, *act_off_copy, *act_slot, *slot_q;
  SlotEnt* tab;
};

// Chunks of a long destination row by all lanes: item (x, begin, end, partial slot) c of
// the row at out[c].
__device__ __forceinline__ void wave_chunks(int4* __restrict__ out, int32_t x, int32_t beg, int32_t end, int32_t so,
                                            int nch, int chunk) {
  for (int c = threadIdx.x & 63; c < nch; c += 64) {
    const int32_t b = beg + c * chunk;
    out[c] = make_int4(x, b, end - b < chunk ? end : b + chunk, so + c);
  }
}

// Pieces of a split CSC row by all lanes: piece c = b * m + i of its m * blocks
// goes to place b * per_block + first + i of the items, its partial row is
// first * blocks + c.
__device__ __forceinline__ void wave_pieces(int4* __restrict__ items, int32_t per_block, int32_t sl, int32_t beg,
                                            int32_t end, int32_t first, int m, int blocks) {
  const int n = m * blocks;
  for (int c = threadIdx.x & 63; c < n; c += 64) {
    const int b = c / m;
    const RowRange r = row_piece(beg, end, c, n);
    items[(int64_t)b * per_block + first + (c - b * m)] = make_int4(sl, r.beg, r.end, first * blocks + c);
  }
}

__global__ void __launch_bounds__(kBT) k_plan_fill(const int32_t* __restrict__ csc_ptr,
                                                   const int32_t* __restrict__ csr_ptr, int64_t ns, int32_t R,
                                                   PlanCut want, int64_t tiles, const int32_t* __restrict__ S, PlanOut o,
                                                   int32_t* __restrict__ cnt) {
  __shared__ uint64_t mask[kPW * HG_MAX_REL];
  __shared__ int32_t before[kPW * HG_MAX_REL];  // active rows before each 64-row group
  __shared__ int32_t wcnt[kPW][HG_MAX_REL];
  __shared__ int32_t wtot[kPW][P_PARTS + 1];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
  const int64_t tile = blockIdx.x, nq = ns * R;
  const auto total = [&](int stream) { return S[(stream + 1) * tiles] - S[stream * tiles]; };
  const bool by_row = row_layout(nq, total(P_ACT));
  const bool in_blocks =
      want.blocks > 1 && blocks_pay(want, csr_ptr[nq], (int64_t)total(P_PARTS) * want.blocks, total(P_SPLIT));
  const PlanCut cut = in_blocks ? want : by_length(want);
  const int cut_at = in_blocks ? 0 : P_LHEAVY - P_HEAVY;  // streams of the cut taken
  int act = 0, heavy = 0, parts = 0;
  for (int g = 0; g < R; ++g) {
    const int64_t q = (tile * kPN + 64 * w) * R + 64 * g + l;
    const int32_t len = q < nq ? csc_ptr[q + 1] - csc_ptr[q] : 0;
    const uint64_t m = __ballot(len > 0);
    if (l == 0) mask[w * R + g] = m;
    const int m_row = cuts_of(len, cut);
    act += len > 0;
    heavy += m_row > 0;
    parts += m_row;
  }
  const int64_t j = tile * kPN + threadIdx.x;
  const int32_t fbeg = j < ns ? csr_ptr[j * R] : 0, fend = j < ns ? csr_ptr[(j + 1) * R] : 0;
  const int fch = fwd_chunks_of(fend - fbeg);
  const int v[P_PARTS + 1] = {act, fch > 0, fch, heavy, parts};
#pragma unroll
  for (int i = 0; i <= P_PARTS; ++i) {
    const int t = wave_sum(v[i]);
    if (l == 0) wtot[w][i] = t;
  }
  __builtin_amdgcn_wave_barrier();
  for (int r = 0; r < R; ++r) {
    const uint64_t m = __ballot(tile_bit(mask, (64 * w + l) * R + r));
    if (l == 0) wcnt[w][r] = (int32_t)__popcll(m);
  }
  __syncthreads();
  const int32_t per_block = total(P_PARTS + cut_at);  // pieces of each block
  int32_t at[P_PARTS + 1];  // the wave's offset in each stream
#pragma unroll
  for (int i = 0; i <= P_PARTS; ++i) {
    const int64_t p = i < P_HEAVY ? i : i + cut_at;
    at[i] = S[p * tiles + tile] - S[p * tiles];
    for (int q = 0; q < w; ++q) at[i] += wtot[q][i];
  }
  for (int g = 0; g < R; ++g) {
    const int64_t q = (tile * kPN + 64 * w) * R + 64 * g + l;
    const bool live = q < nq;
    const int32_t beg = live ? csc_ptr[q] : 0, end = live ? csc_ptr[q + 1] : 0;
    const int mr = cuts_of(end - beg, cut);
    const uint64_t m = __ballot(end > beg), hm = __ballot(mr > 0), om = m & ~hm;
    const int32_t rank = at[P_ACT] + (int32_t)__popcll(m & lt);
    const int32_t sl = by_row ? (int32_t)q : rank;
    if (l == 0) before[w * R + g] = at[P_ACT];
    if (!by_row) {
      if (end > beg) o.slot_q[rank] = (int32_t)q;
      if (l == 0 && live) o.tab[q >> 6] = SlotEnt{m, at[P_ACT], 0};
    }
    // the pieces of the split rows come first, block by block
    if (end > beg && mr == 0)  // after the whole rows, i.e. active ones not split, before it
      o.items[per_block * cut.blocks + at[P_ACT] - at[P_HEAVY] + (int32_t)__popcll(om & lt)] =
          make_int4(sl, beg, end, -1);
    if (hm) {
      const int32_t so = at[P_PARTS] + wave_before(mr);
      if (mr > 0) o.heavy[at[P_HEAVY] + (int32_t)__popcll(hm & lt)] = make_int4(sl, so * cut.blocks, mr * cut.blocks, 0);
      for (uint64_t left = hm; left; left &= left - 1) {
        const int u = __ffsll((unsigned long long)left) - 1;
        wave_pieces(o.items, per_block, __shfl(sl, u, 64), __shfl(beg, u, 64), __shfl(end, u, 64), __shfl(so, u, 64),
                    __shfl(mr, u, 64), cut.blocks);
      }
      at[P_PARTS] += wave_sum(mr);
      at[P_HEAVY] += (int32_t)__popcll(hm);
    }
    at[P_ACT] += (int32_t)__popcll(m);
  }
  // active sources of every relation, ascending, with their slots
  __builtin_amdgcn_wave_barrier();
  for (int r = 0; r < R; ++r) {
    const int row = (64 * w + l) * R + r;
    const bool on = tile_bit(mask, row);
    const uint64_t m = __ballot(on);
    if (on) {
      int32_t p = S[(int64_t)(P_REL + r) * tiles + tile] - S[(int64_t)P_REL * tiles];
      for (int q = 0; q < w; ++q) p += wcnt[q][r];
      p += (int32_t)__popcll(m & lt);
      o.act[p] = (int32_t)j;
      o.act_slot[p] = by_row ? (int32_t)(j * R + r)
                             : before[row >> 6] + (int32_t)__popcll(mask[row >> 6] & ((1ull << (row & 63)) - 1ull));
    }
  }
  // long destination rows
  const uint64_t fm = __ballot(fch > 0);
  if (fm) {
    const int32_t so = at[P_FPARTS] + wave_before(fch);
    if (fch > 0) o.fheavy[at[P_FHEAVY] + (int32_t)__popcll(fm & lt)] = make_int4((int32_t)j, so, fch, 0);
    for (uint64_t left = fm; left; left &= left - 1) {
      const int u = __ffsll((unsigned long long)left) - 1;
      const int32_t so_u = __shfl(so, u, 64);
      wave_chunks(o.fitems + so_u, (int32_t)(tile * kPN + 64 * w + u), __shfl(fbeg, u, 64), __shfl(fend, u, 64), so_u,
                  __shfl(fch, u, 64), kFwdChunk);
    }
  }
  if (tile == 0) {
    for (int r = threadIdx.x; r <= R; r += kBT)
      o.act_off[r] = o.act_off_copy[r] = S[(int64_t)(P_REL + r) * tiles] - S[(int64_t)P_REL * tiles];
    if (threadIdx.x == 0) {
      cnt[C_ASLOTS] = total(P_ACT);
      cnt[C_HEAVY] = total(P_HEAVY + cut_at);
      cnt[C_PARTS] = per_block * cut.blocks;
      cnt[C_ITEMS] = cnt[C_ASLOTS] - cnt[C_HEAVY] + cnt[C_PARTS];
      cnt[C_FHEAVY] = total(P_FHEAVY);
      cnt[C_FPARTS] = total(P_FPARTS);
    }
  }
}

// Slot of the (source, relation) row of each CSR entry; the relation is the
// low part of the entry's sorted CSR key dst * R + r.
__global__ void k_csr_slot(const int32_t* __restrict__ csr_col, const uint32_t* __restrict__ kcsr, int64_t n,
                           int32_t n_rel, int64_t nq, const int32_t* __restrict__ a_total,
                           const SlotEnt* __restrict__ tab, int32_t* __restrict__ csr_slot) {
  if (row_layout(nq, *a_total)) return;  // the kernels index by q
  GRID_STRIDE(p, n) {
    const int64_t q = (int64_t)csr_col[p] * n_rel + (int64_t)(kcsr[p] % (uint32_t)n_rel);
    csr_slot[p] = slot_of(tab, q);
  }
}

// The CSC sort packs destination and row degree into one value while the
// destinations fit in 24 bits.
constexpr int64_t kPackedMaxNodes = (int64_t)1 << 24;

// Counts of the plan's tiles: P_REL + R streams and the end of the scan.
inline int64_t plan_counts(int64_t n, int64_t R) { return (P_REL + R) * cdiv(n > 0 ? n : 1, kPN) + 1; }

// Workspace layout, shared by the sizing and the run.
template <class A>
struct BuildWs {
  int32_t *cnt, *outdeg, *first, *key, *flag, *pos, *list, *iota, *hptr, *list_b, *list_l, *hist;
  uint8_t *sel, *digit;
  SelectState* st;
  int32_t *keep, *vsrc, *vdst, *veid, *alt1, *alt2, *alt3, *pcnt, *tcnt, *scratch;
  uint32_t* bcnt;
  uint64_t* sel_bits;
  int2* parts;
  uint2* bsum;
  int4* gaps;
  int32_t* vw;                // weighted graphs: edge weights (float bits) of the kept edges in edge order
  int32_t *vsc, *vsc_alt;     // unpacked CSC sort: the scales (float bits) and their ping-pong buffer
  uint32_t *kcsr, *kcsc, *kalt, *bbits, *mbits;
  RankEnt* rt;
  int32_t* tile_cnt;
  void layout(A& a, int64_t N, int64_t E, int64_t R, int64_t T, bool hindex, bool weighted) {
    const int64_t NQ = N * R + 1;
    const bool ranks = T <= 2;              // local ids from the rank table, keep as a bit per edge
    const int64_t NT = ranks ? 0 : N;       // the buffers of more node types
    cnt = a.template take<int32_t>(C_COUNT + HG_MAX_NTYPE + 1 + HG_MAX_REL + 1);
    bcnt = a.template take<uint32_t>(16384);  // block counts of k_init_nodes (grid_for caps it there)
    outdeg = a.template take<int32_t>(N);
    first = a.template take<int32_t>(N);
    key = a.template take<int32_t>(N);
    flag = a.template take<int32_t>(NT);
    pos = a.template take<int32_t>(NT);
    list = a.template take<int32_t>(N);
    iota = a.template take<int32_t>(NT);
    hptr = a.template take<int32_t>(hindex ? N + 1 : 0);
    list_b = a.template take<int32_t>(hindex ? hindex_list_b(E) : 0);
    list_l = a.template take<int32_t>(hindex ? hindex_list_l(E) : 0);
    parts = a.template take<int2>(hindex ? hindex_parts(E) : 0);
    hist = a.template take<int32_t>(hindex ? hindex_hist_elems(E) : 0);
    sel = a.template take<uint8_t>(NT);
    bbits = a.template take<uint32_t>(N / 32 + 2);
    bsum = a.template take<uint2>(kSumGroups / 32);
    mbits = a.template take<uint32_t>(ranks ? 0 : 2 * (N / 64 + 1));
    // rank groups: cdiv(N, 64) * 2 <= N / 32 + 2
    rt = a.template take<RankEnt>(N / kRankGroup + 2);
    sel_bits = a.template take<uint64_t>(N / 64 + 1);
    tcnt = a.template take<int32_t>(4 * cdiv(N, kNTile) + 1);
    tile_cnt = a.template take<int32_t>(E / kETile + 2);
    digit = a.template take<uint8_t>(NT);
    st = a.template take<SelectState>(1);
    keep = a.template take<int32_t>(ranks ? 2 * cdiv(E, 64) : E + 1);
    kcsr = a.template take<uint32_t>(E);
    kcsc = a.template take<uint32_t>(E);
    kalt = a.template take<uint32_t>(E);
    vsrc = a.template take<int32_t>(E);
    vdst = a.template take<int32_t>(E);
    veid = a.template take<int32_t>(E);
    alt1 = a.template take<int32_t>(E);
    alt2 = a.template take<int32_t>(E);
    alt3 = a.template take<int32_t>(E);
    gaps = a.template take<int4>(gap_cap(NQ));
    pcnt = a.template take<int32_t>(plan_counts(N, R));
    vw = a.template take<int32_t>(weighted ? E : 0);
    const bool unpacked = weighted || N >= kPackedMaxNodes;
    vsc = a.template take<int32_t>(unpacked ? E : 0);
    vsc_alt = a.template take<int32_t>(unpacked ? E : 0);
    const int64_t longest = E + N + 1 > plan_counts(N, R) ? E + N + 1 : plan_counts(N, R);
    int64_t sc = scan_scratch_elems(longest);
    int64_t rs = radix_scratch_elems(E > N ? E : N);
    scratch = a.template take<int32_t>(sc > rs ? sc : rs);
  }
};

struct PlanLayout {
  size_t s_off, soff_off, aslot_off, slotq_off, cslot_off, tab_off, items_off, heavy_off, fitems_off, fheavy_off,
      total;
  int64_t cap_s, cap_items, cap_heavy, cap_tab, cap_fitems, cap_fheavy;
  PlanLayout(int64_t N, int64_t E, int64_t R) {
    const int64_t nq = N * R;
    cap_s = nq < E ? nq : E;
    // in blocks: a split row of L entries has 2 kMinPiece <= L, and at most L / kMinPiece + L / chunk pieces;
    // in one: chunk < L, and less than 2 L / chunk
    cap_heavy = E / std::min(plan_chunk(E), 2 * kMinPiece) + 1;
    cap_items = cap_s + E / kMinPiece + 2 * (E / plan_chunk(E)) + 2;
    cap_tab = nq / 64 + 1;
    // a row of L > kFwdChunk entries has ceil(L / kFwdChunk) < 2 L / kFwdChunk chunks
    cap_fheavy = E / kFwdChunk + 1;
    cap_fitems = 2 * (E / kFwdChunk) + 2;
    const size_t ns = (size_t)(cap_s > 0 ? cap_s : 1);
    size_t o = 0;
    s_off = o; o = align_up(o + sizeof(int32_t) * ns);
    soff_off = o; o = align_up(o + sizeof(int32_t) * (size_t)(R + 1));
    aslot_off = o; o = align_up(o + sizeof(int32_t) * ns);
    slotq_off = o; o = align_up(o + sizeof(int32_t) * ns);
    cslot_off = o; o = align_up(o + sizeof(int32_t) * (size_t)(E > 0 ? E : 1));
    tab_off = o; o = align_up(o + sizeof(SlotEnt) * (size_t)cap_tab);
    items_off = o; o = align_up(o + sizeof(int4) * (size_t)cap_items);
    heavy_off = o; o = align_up(o + sizeof(int4) * (size_t)cap_heavy);
    fitems_off = o; o = align_up(o + sizeof(int4) * (size_t)cap_fitems);
    fheavy_off = o; o = align_up(o + sizeof(int4) * (size_t)cap_fheavy);
    total = o;
  }
};

}  // namespace

PlanView plan_view(const hg_subgraph* s) {
  PlanLayout pl(s->n_nodes, s->n_edges, s->n_rel);
  const char* b = static_cast<const char*>(s->plan);
  PlanView v;
  v.active = reinterpret_cast<const int32_t*>(b + pl.s_off);
  v.act_slot = reinterpret_cast<const int32_t*>(b + pl.aslot_off);
  const bool by_row = s->plan_slot_rows == s->n_sub * (int64_t)s->n_rel;
  v.slot_q = by_row ? nullptr : reinterpret_cast<const int32_t*>(b + pl.slotq_off);
  v.csr_slot = by_row ? nullptr : reinterpret_cast<const int32_t*>(b + pl.cslot_off);
  v.slot_tab = by_row ? nullptr : reinterpret_cast<const SlotEnt*>(b + pl.tab_off);
  v.items = reinterpret_cast<const int4*>(b + pl.items_off);
  v.heavy = reinterpret_cast<const int4*>(b + pl.heavy_off);
  v.fwd_items = reinterpret_cast<const int4*>(b + pl.fitems_off);
  v.fwd_heavy = reinterpret_cast<const int4*>(b + pl.fheavy_off);
  return v;
}

}  // namespace hg

using namespace hg;

extern "C" size_t hg_plan_size(int64_t n_nodes, int64_t n_edges, int32_t n_rel) {
  if (n_nodes < 0 || n_edges < 0 || n_rel < 1) return 0;
  return PlanLayout(n_nodes, n_edges, n_rel).total;
}

static int validate_build(const hg_graph_desc* g, const hg_overlap_desc* o) {
  if (!g || !o) return fail(HG_ERR_ARG, "null descriptor");
  if (g->n_nodes < 1 || g->n_nodes >= ((int64_t)1 << 31))
    return fail(HG_ERR_ARG, "n_nodes %lld outside [1, 2^31)", (long long)g->n_nodes);
  if (g->n_edges < 0) return fail(HG_ERR_ARG, "n_edges %lld < 0", (long long)g->n_edges);
  if (g->n_edges >= ((int64_t)1 << 31))
    return fail(HG_ERR_UNSUPPORTED, "n_edges %lld >= 2^31", (long long)g->n_edges);
  if (g->n_rel < 1 || g->n_rel > HG_MAX_REL) return fail(HG_ERR_UNSUPPORTED, "n_rel %d", g->n_rel);
  if (g->n_ntype < 1 || g->n_ntype > HG_MAX_NTYPE)
    return fail(HG_ERR_UNSUPPORTED, "n_ntype %d", g->n_ntype);
  if (g->n_nodes * (int64_t)g->n_rel >= ((int64_t)1 << 31) - 1)
    return fail(HG_ERR_UNSUPPORTED, "n_nodes * n_rel >= 2^31");
  if (g->n_edges > 0 && (!g->src || !g->dst || !g->rel))
    return fail(HG_ERR_ARG, "null edge array");
  if (!g->ntype || !g->part) return fail(HG_ERR_ARG, "null node array");
  if (o->budget_M < 0) return fail(HG_ERR_ARG, "budget_M < 0");
  if (o->key != HG_KEY_OUTDEG && o->key != HG_KEY_HINDEX) return fail(HG_ERR_ARG, "key %d", o->key);
  if (o->key_dir != HG_KEYDIR_OUT) return fail(HG_ERR_UNSUPPORTED, "key_dir %d", o->key_dir);
  if (o->theta < 0) return fail(HG_ERR_ARG, "theta < 0");
  return HG_OK;
}

// ---- node keys of the whole graph (the same for every partition block) ----

namespace {

struct KeyWs {
  int32_t *cnt, *hptr, *list_b, *list_l, *hist, *v0, *v1, *scratch;
  uint32_t *k0, *k1;
  int2* parts;
  int4* gaps;
  template <class A>
  void layout(A& a, int64_t N, int64_t E, bool hindex) {
    cnt = a.template take<int32_t>(C_COUNT + 8);
    if (!hindex) return;
    hptr = a.template take<int32_t>(N + 1);
    list_b = a.template take<int32_t>(hindex_list_b(E));
    list_l = a.template take<int32_t>(hindex_list_l(E));
    parts = a.template take<int2>(hindex_parts(E));
    hist = a.template take<int32_t>(hindex_hist_elems(E));
    k0 = a.template take<uint32_t>(E);
    k1 = a.template take<uint32_t>(E);
    v0 = a.template take<int32_t>(E);
    v1 = a.template take<int32_t>(E);
    gaps = a.template take<int4>(gap_cap(N));
    scratch = a.template take<int32_t>(radix_scratch_elems(E));
  }
};

int validate_keys(const hg_graph_desc* g, int32_t key) {
  if (!g) return fail(HG_ERR_ARG, "null descriptor");
  if (g->n_nodes < 1 || g->n_nodes >= ((int64_t)1 << 31))
    return fail(HG_ERR_ARG, "n_nodes %lld outside [1, 2^31)", (long long)g->n_nodes);
  if (g->n_edges < 0) return fail(HG_ERR_ARG, "n_edges %lld < 0", (long long)g->n_edges);
  if (g->n_edges + g->n_nodes >= ((int64_t)1 << 31))
    return fail(HG_ERR_UNSUPPORTED, "n_edges + n_nodes >= 2^31");
  if (g->n_rel < 1 || g->n_rel > HG_MAX_REL) return fail(HG_ERR_UNSUPPORTED, "n_rel %d", g->n_rel);
  if (g->n_edges > 0 && (!g->src || !g->dst || !g->rel)) return fail(HG_ERR_ARG, "null edge array");
  if (key != HG_KEY_OUTDEG && key != HG_KEY_HINDEX) return fail(HG_ERR_ARG, "key %d", key);
  return HG_OK;
}

}  // namespace

extern "C" size_t hg_node_keys_workspace_size(const hg_graph_desc* g, int32_t key) {
  if (validate_keys(g, key) != HG_OK) return 0;
  Sizer sz;
  KeyWs w;
  w.layout(sz, g->n_nodes, g->n_edges, key == HG_KEY_HINDEX);
  return sz.used + 256;
}

extern "C" int hg_node_keys(const hg_graph_desc* g, int32_t key, int32_t* keys, void* ws, size_t ws_bytes,
                            void* stream) {
  HG_TRY(validate_keys(g, key));
  if (!keys) return fail(HG_ERR_ARG, "null keys");
  const size_t need = hg_node_keys_workspace_size(g, key);
  if (!ws || ws_bytes < need) return fail(HG_ERR_CAPACITY, "workspace needs %zu bytes, got %zu", need, ws_bytes);
  const int64_t N = g->n_nodes, E = g->n_edges;
  const bool hindex = key == HG_KEY_HINDEX;
  hipStream_t s = static_cast<hipStream_t>(stream);
  Arena arena(ws, ws_bytes);
  KeyWs w;
  w.layout(arena, N, E, hindex);
  if (!arena.ok()) return fail(HG_ERR_CAPACITY, "workspace layout overflow");
  HG_TRY(fill_i32(w.cnt, 0, C_COUNT + 8, s));
  HG_TRY(fill_i32(keys, 0, N, s));
  if (E > 0 && hindex) {
    HG_LAUNCH("keys_check", k_check_edges, dim3(grid_for(E)), dim3(kBT), 0, s, g->src, g->dst, g->rel, N, E, g->n_rel,
              w.cnt);
    const HindexBufs hb{w.k0, w.k1, w.v0, w.v1, w.hptr, w.list_b, w.list_l, w.hist, w.scratch,
                        w.parts, w.gaps, w.cnt + C_GAP_HI, w.cnt + C_HI_BLOCK};
    HG_TRY(hindex_keys(g->src, g->dst, N, E, nullptr, HG_THETA_NONE, keys, hb, w.cnt + C_ERR, s));
  } else if (E > 0) {
    HG_LAUNCH("keys_outdeg", k_all_outdeg, dim3(agg_grid(E)), dim3(kAggBT), 0, s, g->src, g->dst, g->rel, N, E,
              g->n_rel, keys, w.cnt);
  }
  int32_t herr = 0;
  HG_HIP_TRY(hipMemcpyAsync(&herr, w.cnt + C_ERR, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HG_HIP_TRY(hipStreamSynchronize(s));
  if (herr) return fail(HG_ERR_RANGE, "input ids out of range (flags 0x%x)", herr);
  return HG_OK;
}

extern "C" size_t hg_build_csr_workspace_size(const hg_graph_desc* g, const hg_overlap_desc* o) {
  if (validate_build(g, o) != HG_OK) return 0;
  Sizer sz;
  BuildWs<Sizer> w;
  w.layout(sz, g->n_nodes, g->n_edges, g->n_rel, g->n_ntype, o->key == HG_KEY_HINDEX, g->edge_w != nullptr);
  return sz.used + 256;
}

extern "C" int hg_build_csr(const hg_graph_desc* g, const hg_overlap_desc* o, hg_subgraph* out,
                            void* ws, size_t ws_bytes, void* stream) {
  HG_TRY(validate_build(g, o));
  if (!out) return fail(HG_ERR_ARG, "null output");
  if (!out->local2global || !out->global2local || !out->type_off || !out->csr_ptr ||
      !out->csc_ptr || !out->plan || (!out->overlap && o->budget_M > 0) ||
      (!out->overlap_home && o->budget_M > 0) || (!out->overlap_rel && o->budget_M > 0) ||
      (g->n_edges > 0 && (!out->csr_col || !out->csc_row || !out->csc_scale)))
    return fail(HG_ERR_ARG, "null output array");
  const bool weighted = g->edge_w != nullptr;
  const bool want_eid = out->csr_eid != nullptr;
  if (weighted && g->n_edges > 0 && !out->csr_w) return fail(HG_ERR_ARG, "a weighted graph needs the csr_w output");
  const int64_t N = g->n_nodes, E = g->n_edges, R = g->n_rel, T = g->n_ntype;
  const size_t need_plan = hg_plan_size(N, E, (int32_t)R);
  if (out->plan_bytes < need_plan)
    return fail(HG_ERR_CAPACITY, "plan needs %zu bytes, got %zu", need_plan, out->plan_bytes);
  const size_t need = hg_build_csr_workspace_size(g, o);
  if (!ws || ws_bytes < need) return fail(HG_ERR_CAPACITY, "workspace needs %zu bytes, got %zu", need, ws_bytes);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool hindex = o->key == HG_KEY_HINDEX;

  Arena arena(ws, ws_bytes);
  BuildWs<Arena> w;
  w.layout(arena, N, E, R, T, hindex, g->edge_w != nullptr);
  if (!arena.ok()) return fail(HG_ERR_CAPACITY, "workspace layout overflow");

  const unsigned gN = grid_for(N), gE = grid_for(E);
  // the type ranges and the offsets of the active lists beside the counters, for one copy to the host
  int32_t* type_copy = w.cnt + C_COUNT;
  int32_t* act_copy = type_copy + T + 1;
  const int n_head = C_COUNT + (int)(T + 1 + R + 1);
  // 1. degrees, base-edge index, range checks (kernels that index by an edge's
  // ids end at once when one is out of range; the counts' copy below reports it)
  const unsigned gB = grid_for(cdiv(N, 64) * 64);
  HG_LAUNCH("build_init_nodes", k_init_nodes, dim3(gB), dim3(kBT), 0, s, g->part, g->k, g->ntype, (int32_t)T, N,
            (int32_t)E, w.bbits, w.first, w.outdeg, w.bcnt);
  HG_LAUNCH("build_init_counts", k_init_counts, dim3(1), dim3(256), 0, s, (const uint32_t*)w.bcnt, (int)gB, w.cnt,
            w.st);
  const int sshift = sum_shift(N);
  HG_LAUNCH("build_base_summary", k_base_summary, dim3((unsigned)cdiv(((N - 1) >> sshift) + 1, kBT)), dim3(kBT), 0, s,
            (const uint32_t*)w.bbits, N, sshift, w.bsum);
  if (E > 0)
    HG_LAUNCH("build_edges_pass", k_edges_pass, dim3(agg_grid(E)), dim3(kAggBT), 0, s, g->src, g->dst,
              g->rel, (const uint32_t*)w.bbits, N, E, (int32_t)R, (!hindex && !o->node_key) ? 1 : 0,
              o->budget_M, (const uint2*)w.bsum, sshift, w.outdeg, w.first, w.cnt);
  // 2. keys: the caller's, when given (they do not depend on k); the h-index;
  // or the out-degrees of the nodes outside V_k (every candidate among them)
  const int32_t* key = o->node_key ? o->node_key : (hindex ? w.key : w.outdeg);
  if (hindex && !o->node_key) {
    if (E > 0) {
      const HindexBufs hb{w.kcsr, w.kalt, w.vsrc, w.alt1, w.hptr, w.list_b, w.list_l, w.hist, w.scratch,
                          w.parts, w.gaps, w.cnt + C_GAP_HI, w.cnt + C_HI_BLOCK};
      HG_TRY(hindex_keys(g->src, g->dst, N, E, w.first, o->theta, w.key, hb, w.cnt + C_ERR, s));
    }
  }
  // 3, 4. filtered candidates and TopM
  const unsigned gS = (unsigned)std::min<int64_t>(cdiv(N, kSelBT * kSelItems), 2 * (int64_t)num_cus());
  HG_LAUNCH("build_candidates", k_candidates, dim3(gS), dim3(kSelBT), 0, s, (const int32_t*)w.first, key, N,
            (int32_t)E, o->theta, o->budget_M, w.list, w.cnt, w.st);
  for (int p = 0, steps = select_steps(N); p < steps; ++p)
    HG_LAUNCH("build_select_step", k_select_step, dim3(gS), dim3(kSelBT), 0, s, w.st, (const int32_t*)w.list,
              (const int32_t*)w.cnt, key, o->seed);
  HG_LAUNCH("build_select_finish", k_select_finish, dim3(1), dim3(kSelBT), 0, s, w.st, (const int32_t*)w.list,
            (const int32_t*)w.cnt, key, o->seed);
  // 5. the node set and its local ids in (ntype, gid) order
  const bool rank_path = T <= 2;
  const int64_t ntiles_n = cdiv(N, kNTile);
  HG_LAUNCH("build_nodes_count", k_nodes_count, dim3((unsigned)ntiles_n), dim3(kBT), 0, s, (const uint32_t*)w.bbits,
            g->ntype, w.first, key, (const SelectState*)w.st, o->seed, N, (int32_t)E, o->theta, o->budget_M,
            (const int32_t*)w.cnt, w.rt, w.sel_bits, rank_path ? nullptr : w.sel, ntiles_n, w.tcnt);
  if (rank_path) {
    HG_TRY(scan_exclusive_i32(w.tcnt, w.tcnt, 4 * ntiles_n + 1, nullptr, w.scratch, s));
    HG_LAUNCH("build_nodes_assign", k_nodes_assign, dim3((unsigned)ntiles_n), dim3(kBT), 0, s, w.rt,
              (const uint64_t*)w.sel_bits, g->part, N, (int32_t)T, ntiles_n, (const int32_t*)w.tcnt,
              out->local2global, out->global2local, out->type_off, type_copy, out->overlap, out->overlap_home, w.cnt);
  } else {
    HG_LAUNCH("build_member_digit", k_member_digit, dim3(gN), dim3(kBT), 0, s, g->part, g->k,
              (const uint8_t*)w.sel, g->ntype, N, w.digit, w.iota);
    HG_TRY(bucket_partition(w.digit, w.iota, N, (int)T, out->local2global, out->type_off, w.scratch, s));
    HG_TRY(fill_i32(out->global2local, -1, N, s));
    HG_LAUNCH("build_global2local", k_global2local, dim3(gN), dim3(kBT), 0, s,
              (const int32_t*)out->local2global, (const int32_t*)out->type_off, (int32_t)T,
              out->global2local, w.cnt);
    HG_LAUNCH("build_overlap_flags", k_overlap_flags, dim3(gN), dim3(kBT), 0, s,
              (const int32_t*)out->local2global, (const uint8_t*)w.sel, (const int32_t*)w.cnt, N, w.flag);
    HG_TRY(scan_exclusive_i32(w.flag, w.pos, N, w.cnt + C_MSEL, w.scratch, s));
    if (o->budget_M > 0)
      HG_LAUNCH("build_overlap_fill", k_overlap_fill, dim3(gN), dim3(kBT), 0, s,
                (const int32_t*)out->local2global, (const int32_t*)w.flag, (const int32_t*)w.pos,
                (const int32_t*)w.cnt, g->part, out->overlap, out->overlap_home);
  }
  // 6. induced-subgraph edges in original order, and the base edges of the
  // selected nodes
  // the CSR sort carries the edge id if asked for, else a weighted graph's weight
  const bool emit_w = weighted && !want_eid;
  // with at most two node types the CSR entries are formed in edge order and
  // compacted only if some edge was dropped (below, once the count is known)
  const int64_t ntiles = cdiv(E, kETile);
  if (E > 0) {
    if (rank_path) {
#define HG_EDGE_IDS(TS_, W_)                                                                                   \
  HG_LAUNCH("build_edge_ids", (k_edge_ids<TS_, W_>), dim3((unsigned)ntiles), dim3(kBT), 0, s, g->src, g->dst,     \
            g->rel, (int32_t)R, (const RankEnt*)w.rt, (const int32_t*)out->type_off, (const uint32_t*)w.bbits,    \
            g->edge_ts, g->t_cut, E, N, o->budget_M, (const int32_t*)w.cnt, w.kcsr, w.vsrc,                       \
            want_eid ? w.veid : nullptr, g->edge_w, emit_w ? w.vw : nullptr,                                      \
            reinterpret_cast<uint64_t*>(w.keep), w.tile_cnt, w.first)
      if (g->edge_ts) {
        if (emit_w) HG_EDGE_IDS(true, true); else HG_EDGE_IDS(true, false);
      } else {
        if (emit_w) HG_EDGE_IDS(false, true); else HG_EDGE_IDS(false, false);
      }
#undef HG_EDGE_IDS
      HG_TRY(scan_exclusive_i32(w.tile_cnt, w.tile_cnt, ntiles, w.cnt + C_ESUB, w.scratch, s));
    } else {
      // more than two node types: local ids from global2local, membership from a bitmap
      HG_LAUNCH("build_member_bits", k_member_bits, dim3(gB), dim3(kBT), 0, s, g->part, g->k,
                (const uint8_t*)w.sel, N, w.mbits);
      HG_LAUNCH("build_edge_keep", k_edge_keep, dim3(gE), dim3(kBT), 0, s, g->src, g->dst,
                (const uint32_t*)w.mbits, (const uint32_t*)w.bbits, g->edge_ts, g->t_cut, E, w.keep, w.first,
                (const int32_t*)w.cnt);
      // keep[E] = 0, so the scan's entry E is the number of kept edges
      HG_TRY(fill_i32(w.keep + E, 0, 1, s));
      HG_TRY(scan_exclusive_i32(w.keep, w.keep, E + 1, w.cnt + C_ESUB, w.scratch, s));
      HG_LAUNCH("build_edge_compact", k_edge_compact, dim3(gE), dim3(kBT), 0, s, g->src, g->dst,
                (const int32_t*)out->global2local, g->rel, (const int32_t*)w.keep, E, (int32_t)R, w.kcsr, w.vsrc,
                want_eid ? w.veid : nullptr, g->edge_w, emit_w ? w.vw : nullptr, (const int32_t*)w.cnt);
    }
    if (o->budget_M > 0)
      HG_LAUNCH("build_overlap_rel", k_overlap_rel, dim3(grid_for(o->budget_M < N ? o->budget_M : N)), dim3(kBT), 0, s,
                (const int32_t*)out->local2global, (const int32_t*)out->overlap, (const int32_t*)w.cnt,
                (const int32_t*)w.first, g->rel, out->overlap_rel);
  }
  // counts needed to size the sorts
  int32_t hc[C_COUNT];
  HG_HIP_TRY(hipMemcpyAsync(hc, w.cnt, sizeof(hc), hipMemcpyDeviceToHost, s));
  HG_HIP_TRY(hipStreamSynchronize(s));
  if (hc[C_ERR]) return fail(HG_ERR_RANGE, "input ids out of range (flags 0x%x)", hc[C_ERR]);
  const int64_t NS = hc[C_NSUB], ES = hc[C_ESUB];
  const int64_t NQ = NS * R;
  // 7. CSR: stable sort by dst*R + r; CSC: stable sort of the CSR-ordered entries by src*R + r
  const int bits = bits_for(NQ);
  uint32_t* csr_keys = w.kcsr;  // the CSR's sorted keys, kept for the slots of its entries
  {
    uint32_t* ko;
    int32_t *v1o, *v2o;
    // second value: the edge id if asked for, else the weight of a weighted graph
    int32_t* v2 = want_eid ? w.veid : (weighted ? w.vw : nullptr);
    int32_t* v2_final = want_eid ? out->csr_eid : (weighted ? reinterpret_cast<int32_t*>(out->csr_w) : nullptr);
    uint32_t *sk = w.kcsr, *sk_alt = w.kalt;
    int32_t *s1 = w.vsrc, *s1_alt = w.alt1, *s2 = v2, *s2_alt = v2 ? w.alt2 : nullptr;
    if (rank_path && ES < E) {
      // some edges were dropped: compact the entries into the ping-pong buffers
      HG_LAUNCH("build_edge_compact", k_edge_emit, dim3((unsigned)ntiles), dim3(kBT), 0, s, (const uint32_t*)w.kcsr,
                (const int32_t*)w.vsrc, (const int32_t*)v2, (const uint64_t*)w.keep, E, (const int32_t*)w.tile_cnt,
                w.kalt, w.alt1, v2 ? w.alt2 : nullptr);
      std::swap(sk, sk_alt);
      std::swap(s1, s1_alt);
      std::swap(s2, s2_alt);
    }
    HG_TRY(radix_sort_pairs(sk, sk_alt, s1, s1_alt, s2, s2_alt, ES, bits, w.scratch, s, &ko, &v1o, &v2o,
                            out->csr_col, v2_final));
    csr_keys = ko;
    if (ES > 0 && v1o != out->csr_col) {  // no pass ran (a single key value)
      HG_HIP_TRY(hipMemcpyAsync(out->csr_col, v1o, sizeof(int32_t) * ES, hipMemcpyDeviceToDevice, s));
      if (v2)
        HG_HIP_TRY(hipMemcpyAsync(v2_final, v2o, sizeof(int32_t) * ES, hipMemcpyDeviceToDevice, s));
    }
    // both edge ids and weights asked for: the weights through the edge ids
    if (want_eid && weighted && ES > 0)
      HG_LAUNCH("build_csr_w", k_gather_w, dim3(grid_for(ES)), dim3(kBT), 0, s, (const int32_t*)out->csr_eid,
                g->edge_w, ES, out->csr_w);
    HG_TRY(row_pointers(ko, ES, NQ, out->csr_ptr, w.gaps, w.cnt + C_GAP_CSR, nullptr, s));
  }
  {
    // the CSC sort's input from the CSR in its order (the CSR keys stay
    // where the CSR sort left them, for the slots of its entries)
    uint32_t* ko;
    int32_t *v1o, *v2o;
    const bool packed = !weighted && NS < kPackedMaxNodes;
    if (ES > 0)
      HG_LAUNCH("build_csc_input", k_csc_input, dim3((unsigned)cdiv(ES, kBT * kCiItems)), dim3(kBT), 0, s,
                (const uint32_t*)csr_keys, (const int32_t*)out->csr_col, (const int32_t*)out->csr_ptr,
                weighted ? (const float*)out->csr_w : nullptr, ES, (int32_t)R, packed ? 1 : 0, w.kcsc, w.vdst,
                packed ? nullptr : w.vsc);
    int32_t* scale_bits = reinterpret_cast<int32_t*>(out->csc_scale);
    const SortUnpack up{out->csr_ptr, (int32_t)R, out->csc_scale};
    HG_TRY(radix_sort_pairs(w.kcsc, csr_keys == w.kalt ? w.kcsr : w.kalt, w.vdst, w.alt3, packed ? nullptr : w.vsc,
                            packed ? nullptr : w.vsc_alt, ES, bits, w.scratch, s, &ko, &v1o, &v2o, out->csc_row,
                            packed ? nullptr : scale_bits, packed ? &up : nullptr));
    if (ES > 0 && v1o != out->csc_row) {  // no pass ran (unpacked, a single key value)
      HG_HIP_TRY(hipMemcpyAsync(out->csc_row, v1o, sizeof(int32_t) * ES, hipMemcpyDeviceToDevice, s));
      HG_HIP_TRY(hipMemcpyAsync(scale_bits, v2o, sizeof(int32_t) * ES, hipMemcpyDeviceToDevice, s));
    }
    HG_TRY(row_pointers(ko, ES, NQ, out->csc_ptr, w.gaps, w.cnt + C_GAP_CSC, nullptr, s));
  }
  // 8. plan: active-source lists and backward work items
  PlanLayout pl(N, E, R);
  char* pb = static_cast<char*>(out->plan);
  int32_t* act = reinterpret_cast<int32_t*>(pb + pl.s_off);
  int32_t* act_off = reinterpret_cast<int32_t*>(pb + pl.soff_off);
  int4* items = reinterpret_cast<int4*>(pb + pl.items_off);
  int4* heavy = reinterpret_cast<int4*>(pb + pl.heavy_off);
  int32_t* act_slot = reinterpret_cast<int32_t*>(pb + pl.aslot_off);
  int32_t* slot_q = reinterpret_cast<int32_t*>(pb + pl.slotq_off);
  int32_t* csr_slot = reinterpret_cast<int32_t*>(pb + pl.cslot_off);
  SlotEnt* tab = reinterpret_cast<SlotEnt*>(pb + pl.tab_off);
  if (NQ > 0) {
    const int64_t tiles = cdiv(NS, kPN);
    const PlanCut cut = plan_cut(E, NS);
    const PlanOut po{items,
                     heavy,
                     reinterpret_cast<int4*>(pb + pl.fitems_off),
                     reinterpret_cast<int4*>(pb + pl.fheavy_off),
                     act,
                     act_off,
                     act_copy,
                     act_slot,
                     slot_q,
                     tab};
    HG_LAUNCH("build_plan_count", k_plan_count, dim3((unsigned)tiles), dim3(kBT), 0, s, (const int32_t*)out->csc_ptr,
              (const int32_t*)out->csr_ptr, NS, (int32_t)R, cut, tiles, w.pcnt);
    HG_TRY(scan_exclusive_i32(w.pcnt, w.pcnt, (P_REL + R) * tiles + 1, nullptr, w.scratch, s));
    HG_LAUNCH("build_plan_fill", k_plan_fill, dim3((unsigned)tiles), dim3(kBT), 0, s, (const int32_t*)out->csc_ptr,
              (const int32_t*)out->csr_ptr, NS, (int32_t)R, cut, tiles, (const int32_t*)w.pcnt, po, w.cnt);
    if (ES > 0)
      HG_LAUNCH("build_csr_slot", k_csr_slot, dim3(grid_for(ES)), dim3(kBT), 0, s, (const int32_t*)out->csr_col,
                (const uint32_t*)csr_keys, ES, (int32_t)R, NQ, (const int32_t*)(w.cnt + C_ASLOTS),
                (const SlotEnt*)tab, csr_slot);
  } else {
    HG_TRY(fill_i32(act_off, 0, R + 1, s));
    HG_TRY(fill_i32(act_copy, 0, R + 1, s));
  }
  // final sync: host counts
  std::vector<int32_t> head(n_head);
  HG_HIP_TRY(hipMemcpyAsync(head.data(), w.cnt, sizeof(int32_t) * n_head, hipMemcpyDeviceToHost, s));
  if (!rank_path)
    HG_HIP_TRY(hipMemcpyAsync(head.data() + C_COUNT, out->type_off, sizeof(int32_t) * (T + 1), hipMemcpyDeviceToHost, s));
  HG_HIP_TRY(hipStreamSynchronize(s));
  std::copy(head.begin(), head.begin() + C_COUNT, hc);
  const int32_t *tof = head.data() + C_COUNT, *aof = tof + T + 1;
  out->n_nodes = N;
  out->n_edges = E;
  out->n_sub = NS;
  out->e_sub = ES;
  out->m_sel = hc[C_MSEL];
  out->n_rel = (int32_t)R;
  out->n_ntype = (int32_t)T;
  for (int t = 0; t <= HG_MAX_NTYPE; ++t) out->type_off_host[t] = t <= T ? tof[t] : 0;
  for (int r = 0; r < HG_MAX_REL; ++r) out->n_active[r] = r < R ? (int64_t)aof[r + 1] - aof[r] : 0;
  out->plan_items = hc[C_ITEMS];
  out->plan_heavy = hc[C_HEAVY];
  out->plan_partials = hc[C_PARTS];
  out->plan_fwd_heavy = hc[C_FHEAVY];
  out->plan_fwd_parts = hc[C_FPARTS];
  out->plan_slot_rows = row_layout(NQ, hc[C_ASLOTS]) ? NQ : hc[C_ASLOTS];
  out->weighted = weighted ? 1 : 0;
  return HG_OK;
}
