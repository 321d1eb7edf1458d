// Exact single linkage on the GPU: the maximum spanning forest of the
// similarity graph, updated tile by tile from device-resident LCS tiles.
//
// The paper builds its guide tree by single linkage, incrementally and with
// O(k) memory (Methods, "Determination of the guide tree").  Single linkage
// merges clusters in the order of the maximum spanning tree of the
// similarities, so keeping that tree is enough: after every tile, the forest
// F becomes the maximum spanning forest of F plus the tile's pairs (a forest
// that is optimal for a set of edges stays a valid summary of it, by the
// cycle property).  In steps:
//   1. a pair (i, j) of the tile can enter the forest only if it is better
//      than the worst edge on F's path between i and j; one pass over the
//      tile (mst_filter) keeps the pairs that are, the survivors (rows that F
//      does not reach yet are tied to it first, mst_attach);
//   2. an update, Boruvka on F plus the survivors of one or several tiles,
//      gives the new forest: every component takes the best edge that leaves
//      it, components hook along these edges and are renumbered, edges inside
//      a component are dropped;
//   3. the rounds' components are the hierarchy that answers the next pass's
//      path queries (mst_view).
// The path query (King's lemma on Boruvka trees): the worst edge on the path
// between i and j in the forest is the worst of the edges that i's and j's
// components chose in the rounds before they became one.  So per vertex and
// round the component's label and the worst edge chosen so far suffice: a
// pair looks up the lowest round in which its labels agree.
// The tile is read once (four bytes a pair) instead of once and then in parts
// in each of five or six rounds, and the rounds work on the forest and a few
// edges a vertex.  Per 1,024-row tile of 30,000 columns the pass takes 12-50 us
// (later tiles are narrower) and an update, once in several tiles, 150-250 us,
// most of it launches, against 560 us a tile for dense rounds; k = 12,000
// sequences of 60 residues to their guide tree 9.3 -> 3.8 ms, k = 30,000 of
// 250 91.0 -> 67.7 ms (the LCS kernels are 60 of them).
//
// Similarity (Methods, "Pairwise similarities calculation") is
// LCS / indel^2 with indel = |A| + |B| - 2 LCS, +infinity when indel = 0.
// It is compared as the correctly rounded double of that ratio: for lengths up
// to 65535 two different ratios differ by at least four units in the last
// place, so the order is exact.  Ties between equal similarities are broken
// by the edge (u, v), u < v, lexicographically, which makes every choice
// unique (no cycles).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "runtime.h"

namespace famsa {

// Key of an edge's similarity: the double's bits plus one (similarities are
// >= 0 or +inf, so the bits order like the values); 0 means "no edge".
__device__ __forceinline__ uint64_t sim_key(int32_t L, uint32_t la, uint32_t lb) {
  const int64_t d = (int64_t)la + (int64_t)lb - 2 * (int64_t)L;
  const double s = d == 0 ? __builtin_inf() : (double)L / (double)(d * d);
  return (uint64_t)__double_as_longlong(s) + 1ull;
}

// (key, id) pairs: larger key wins, then smaller id.
__device__ __forceinline__ bool better(uint64_t ka, uint64_t ia, uint64_t kb, uint64_t ib) {
  return ka > kb || (ka == kb && ia < ib);
}

// A vertex's place in the last hierarchy, the coarsest rounds first: slot s
// is round D - s of D.  label: the vertex's component after that round (the
// vertex itself where the hierarchy has no such round: labels of different
// vertices then never agree).  bound: the worst similarity its components
// chose up to that round, rounded down.
constexpr uint32_t kMstSlots = 8;
struct MstView {
  uint32_t label[kMstSlots];
  float bound[kMstSlots];
};
struct MstExact {  // the same choice exactly
  uint64_t key[kMstSlots], id[kMstSlots];
};

constexpr uint32_t kMstMaxRounds = 40;
constexpr uint32_t kAll = 0xFFFFFFFFu;
struct MstCtl {
  uint32_t nf;      // edges in the forest
  uint32_t pad;
  uint64_t rounds;  // Boruvka rounds with hooks, over all updates
};
struct MstPass {  // one update; the next one's is cleared by this one's last launch
  uint64_t surv;    // low half: survivors so far; high half: blocks of the passes that are through
  uint32_t nnew;    // edges in the new forest
  uint32_t ntot;    // component labels given out: vertices first, then each round's components
  uint32_t levels;  // rounds with hooks
  uint32_t act[kMstMaxRounds];  // round r runs on the whole GPU
  uint32_t cnt[kMstMaxRounds];  // edges between components in round r
  uint32_t hi[kMstMaxRounds];   // labels of round r's components end here
};

struct MstComp {  // per component label, 2 k of them
  uint64_t* key;  // best outgoing edge
  uint64_t* id;
  uint32_t* par;  // hook target, then the root of the hooked tree
  uint32_t* nid;  // of a root: its label in the next round
};

struct MstDev {
  const uint32_t* len;
  uint32_t k;
  uint32_t room;      // survivors the e* arrays hold after the forest's k - 1 edges
  uint32_t n;         // survivors that this update takes in, kAll: as many as there are by then
  uint32_t* eu;       // forest edges (ctl->nf), then the survivors
  uint32_t* ev;
  uint64_t* ekey;
  int32_t* eL;
  uint32_t* nu;       // the new forest (ps->nnew)
  uint32_t* nv;
  uint64_t* nkey;
  int32_t* nL;
  uint32_t* lu[2];    // edges between components: labels of the ends, index in e*, key
  uint32_t* lv[2];
  uint32_t* le[2];
  uint64_t* lk[2];
  MstComp c;          // this update's components
  MstComp next;       // the next update's
  MstPass* ps;
  MstPass* ps_next;
  MstView* view;
  MstExact* exact;
  MstCtl* ctl;
  uint32_t* host;     // pinned: [0] survivors so far
};

// The last rounds run in one workgroup, components in LDS.
constexpr uint32_t kFinThreads = 1024;
constexpr uint32_t kFinComps = 4096;
constexpr uint32_t kFinEdges = 8192;
constexpr size_t kFinLds = (size_t)kFinComps * 24;

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A slot of *counter for every lane that is `on`: one atomic a wave.  Every
// lane of the wave calls it.
__device__ __forceinline__ uint32_t wave_slot(bool on, uint32_t* counter) {
  const uint64_t mask = __ballot(on);
  if (mask == 0) return 0;
  const int lead = __builtin_ctzll(mask);
  uint32_t base = 0;
  if ((int)__lane_id() == lead) base = atomicAdd(counter, (uint32_t)__popcll(mask));
  base = (uint32_t)__shfl((int)base, lead, 64);
  return base + lanes_below(mask);
}

__device__ __forceinline__ void offer(uint64_t* slot, uint64_t key) {
  if (key > *slot) atomicMax((unsigned long long*)slot, (unsigned long long)key);  // a stale read only costs an atomic
}

// The same for a block, with one global atomic: appends from all eight XCDs to
// one counter are served one after another, about 60 ns each.  Every thread of
// the block calls it; `red` is LDS of its own.
struct BlockSlots {
  uint32_t wave[16];
  uint32_t base;
};
__device__ __forceinline__ uint32_t block_slot(bool on, uint32_t* counter, BlockSlots* red) {
  const uint32_t w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint64_t mask = __ballot(on);
  if ((threadIdx.x & 63u) == 0) red->wave[w] = (uint32_t)__popcll(mask);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t sum = 0;
    for (uint32_t i = 0; i < nw; ++i) {
      const uint32_t n = red->wave[i];
      red->wave[i] = sum;
      sum += n;
    }
    red->base = sum ? atomicAdd(counter, sum) : 0u;
  }
  __syncthreads();
  const uint32_t at = red->base + red->wave[w] + lanes_below(mask);
  __syncthreads();  // the LDS is used again by the next call
  return at;
}

// A block's offers, gathered in LDS by component before they go out: where few
// components are left, thousands of edges offer to the same slot, and those
// atomics would be served one after another too.  A component whose place in
// the table is taken by another goes out at once.
constexpr uint32_t kOffers = 2048;
struct OfferTable {
  uint32_t comp[kOffers];
  uint64_t key[kOffers];
};
__device__ __forceinline__ void offers_begin(OfferTable* t) {
  for (uint32_t x = threadIdx.x; x < kOffers; x += blockDim.x) {
    t->comp[x] = 0xFFFFFFFFu;
    t->key[x] = 0;
  }
  __syncthreads();
}
__device__ __forceinline__ void offers_add(OfferTable* t, uint64_t* slots, uint32_t c, uint64_t key) {
  const uint32_t x = (c * 2654435761u) >> 21;  // 11 bits
  uint32_t have = t->comp[x];
  if (have == 0xFFFFFFFFu) {
    have = atomicCAS(&t->comp[x], 0xFFFFFFFFu, c);
    if (have == 0xFFFFFFFFu) have = c;
  }
  if (have == c) offer(&t->key[x], key);
  else offer(&slots[c], key);
}
__device__ __forceinline__ void offers_end(OfferTable* t, uint64_t* slots) {
  __syncthreads();
  for (uint32_t x = threadIdx.x; x < kOffers; x += blockDim.x)
    if (t->comp[x] != 0xFFFFFFFFu) offer(&slots[t->comp[x]], t->key[x]);
}

__device__ __forceinline__ uint32_t mst_taken(const MstDev& m) { return m.n == kAll ? (uint32_t)m.ps->surv : m.n; }

// An update that was queued behind its pass is left undone when the survivors
// do not fit (the host repeats it with fewer rows), and has nothing to do when
// there are none.
__device__ __forceinline__ bool mst_idle(const MstDev& m) {
  const uint32_t n = mst_taken(m);
  return n == 0 || n > m.room;
}

// Clear the components and counters of an update.
__device__ __forceinline__ void mst_clear(const MstComp& c, MstPass* ps, uint32_t k) {
  const uint64_t n = 2ull * k, step = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += step) {
    c.key[x] = 0;
    c.id[x] = ~0ull;
    c.par[x] = (uint32_t)x;
  }
  if (blockIdx.x == 0 && threadIdx.x < kMstMaxRounds) {
    ps->act[threadIdx.x] = 0;
    ps->cnt[threadIdx.x] = 0;
    ps->hi[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
      ps->surv = 0;
      ps->nnew = 0;
      ps->ntot = k;
      ps->levels = 0;
    }
  }
}

// A block of the pass is through, with n survivors to append: their place.
// The last one tells the host how many there are now.
__device__ __forceinline__ uint32_t mst_leave(const MstDev& m, uint32_t n, uint32_t last) {
  const uint64_t old = atomicAdd((unsigned long long*)&m.ps->surv, (1ull << 32) | n);
  if ((uint32_t)(old >> 32) == last)
    __hip_atomic_store(m.host, (uint32_t)old + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return (uint32_t)old;
}

// Values before tile row i (rows r0.. of the upper triangle, k - 1 - t per row t).
__device__ __forceinline__ uint64_t row_off(uint64_t k, uint32_t r0, uint32_t i) {
  const uint64_t n = i - r0;
  return n * (k - 1) - ((uint64_t)r0 + i - 1) * n / 2;
}

// The pass over the tile: rows r0 + t stride for t in [t0, t1), without every
// eighth (t a multiple of 8) when `skip` is set (taken by an earlier pass).
// A block takes 128 columns and a slice of rows; each of its waves holds the
// columns' labels and bounds in registers (two columns a lane: four would take
// twice the registers and hide no more latency) and walks rows four at a time,
// their labels and bounds wave-uniform and their loads in flight together.  A
// pair costs four instructions a slot and a float comparison, so the pass is
// bound by reading the tile.  Pairs the rounded bound does not drop (few) are
// compared exactly with the edge the bound stands for.  Survivors gather in
// LDS and leave with one global atomic a block.
constexpr uint32_t kFiltCols = 2;
constexpr uint32_t kFiltWaves = 16;
constexpr uint32_t kFiltChunk = 4;
constexpr uint32_t kFiltBuf = 3072;

__global__ __launch_bounds__(64 * kFiltWaves) void mst_filter(MstDev m, const MstView* __restrict__ view,
                                                              const uint32_t* __restrict__ len,
                                                              const int32_t* __restrict__ tile, uint32_t r0,
                                                              uint32_t r1, uint32_t t0, uint32_t t1, uint32_t slice,
                                                              uint32_t stride, uint32_t skip, uint32_t j0,
                                                              uint32_t last_block) {
  __shared__ uint32_t bi[kFiltBuf], bj[kFiltBuf];
  __shared__ int32_t bL[kFiltBuf];
  __shared__ uint32_t s_n, s_base;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t k = m.k, nf = m.ctl->nf;
  const uint32_t jb = j0 + blockIdx.x * (64u * kFiltCols);  // < k
  const uint32_t tb = t0 + blockIdx.y * slice, te = min(t1, tb + slice);
  const uint32_t last = min(r1, k - 1u) - 1u;  // the tile's last row with a pair
  if (r0 + tb * stride >= jb + 64u * kFiltCols - 1u) {  // no column of the block is after its first row
    if (threadIdx.x == 0) (void)mst_leave(m, 0, last_block);
    return;
  }
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  uint32_t lj[kFiltCols];
  MstView vj[kFiltCols];
#pragma unroll
  for (int c = 0; c < (int)kFiltCols; ++c) {
    const uint32_t j = min(jb + 64u * c + lane, k - 1u);
    vj[c] = view[j];
    lj[c] = len[j];
  }
  for (uint32_t t = tb + wave * kFiltChunk; t < te; t += kFiltChunk * kFiltWaves) {
    if (r0 + t * stride >= jb + 64u * kFiltCols - 1u) break;  // nor after this row or later ones
    int32_t L[kFiltChunk][kFiltCols];
#pragma unroll
    for (int u = 0; u < (int)kFiltChunk; ++u) {  // unconditional loads from clamped pairs of the tile
      const uint32_t i = min(r0 + min(t + (uint32_t)u, te - 1u) * stride, last);
      const uint64_t off = row_off(k, r0, i);
#pragma unroll
      for (int c = 0; c < (int)kFiltCols; ++c) {
        const uint32_t j = min(max(jb + 64u * c + lane, i + 1u), k - 1u);
        L[u][c] = tile[off + (j - i - 1u)];
      }
    }
    uint64_t keep[kFiltChunk][kFiltCols];
    uint32_t total = 0;
#pragma unroll
    for (int u = 0; u < (int)kFiltChunk; ++u) {
      const uint32_t tu = t + (uint32_t)u, i = r0 + tu * stride;
      const bool live = tu < te && i <= last && !(skip && (tu & 7u) == 0);
      const uint32_t ic = min(i, last);
      const MstView& vi = view[ic];
      const uint32_t li = len[ic];
#pragma unroll
      for (int c = 0; c < (int)kFiltCols; ++c) {
        const uint32_t j = jb + 64u * c + lane;
        float T = -1.0f;  // no round in which the pair is one component: nothing to beat
        uint32_t slot = kMstSlots;
#pragma unroll
        for (int s = 0; s < (int)kMstSlots; ++s) {
          const bool eq = vi.label[s] == vj[c].label[s];
          T = eq ? fminf(vi.bound[s], vj[c].bound[s]) : T;
          slot = eq ? (uint32_t)s : slot;
        }
        const float d = (float)((int32_t)(li + lj[c]) - 2 * L[u][c]);
        // not (L < T d^2): an infinite bound and d = 0 compare as unordered and are looked at exactly
        bool on = live && j > i && j < k && !((float)L[u][c] < T * d * d);
        if (__any(on)) {
          if (on && slot < kMstSlots) {
            const uint64_t key = sim_key(L[u][c], li, lj[c]), id = (uint64_t)i * k + j;
            const MstExact *xi = m.exact + i, *xj = m.exact + j;
            const uint64_t ki = xi->key[slot], ii = xi->id[slot], kj = xj->key[slot], ij = xj->id[slot];
            const bool w = better(ki, ii, kj, ij);  // the worse of the two is j's
            on = better(key, id, w ? kj : ki, w ? ij : ii);
          }
        }
        keep[u][c] = __ballot(on);
        total += (uint32_t)__popcll(keep[u][c]);
      }
    }
    if (total == 0) continue;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&s_n, total);
    base = __builtin_amdgcn_readfirstlane(base);
    uint32_t over = 0;  // past the block's buffer: straight to the list
    if (base + total > kFiltBuf) {
      const uint32_t out = base + total - max(base, kFiltBuf);
      if (lane == 0) over = (uint32_t)atomicAdd((unsigned long long*)&m.ps->surv, (unsigned long long)out);
      over = __builtin_amdgcn_readfirstlane(over) - max(base, kFiltBuf);
    }
#pragma unroll
    for (int u = 0; u < (int)kFiltChunk; ++u) {
      const uint32_t i = r0 + (t + (uint32_t)u) * stride;
#pragma unroll
      for (int c = 0; c < (int)kFiltCols; ++c) {
        const uint32_t at = base + lanes_below(keep[u][c]);
        if ((keep[u][c] >> lane) & 1ull) {
          if (at < kFiltBuf) {
            bi[at] = i;
            bj[at] = jb + 64u * c + lane;
            bL[at] = L[u][c];
          } else if (over + at < m.room) {
            const uint32_t e = nf + over + at;
            m.eu[e] = i;
            m.ev[e] = jb + 64u * c + lane;
            m.ekey[e] = sim_key(L[u][c], len[i], lj[c]);
            m.eL[e] = L[u][c];
          }
        }
        base += (uint32_t)__popcll(keep[u][c]);
      }
    }
  }
  __syncthreads();
  const uint32_t n = min(s_n, kFiltBuf);
  if (threadIdx.x == 0) s_base = mst_leave(m, n, last_block);
  __syncthreads();
  const uint32_t base = s_base;
  for (uint32_t x = threadIdx.x; x < n && base + x < m.room; x += 64 * kFiltWaves) {
    const uint32_t e = nf + base + x, i = bi[x], j = bj[x];
    m.eu[e] = i;
    m.ev[e] = j;
    m.ekey[e] = sim_key(bL[x], len[i], len[j]);
    m.eL[e] = bL[x];
  }
}

// Rows a..b-1 of the tile, whose vertices the forest does not reach yet, are
// tied to the vertices from `cover` on, which it joins (cover >= b): every row's
// best pair with one of those (by the similarity in single precision: any pair
// would do, a good one lets fewer pairs through the pass) goes into the list of
// survivors at `at`, and the row's vertex takes its partner's place in the
// hierarchy, as a leaf on it: the partner's labels, and the worse of the
// partner's bound and the new edge.  (Too low a bound in the partner's lowest
// rounds, where the path is the new edge alone; that only lets more through.)
// With cover 0 the best pair may be with any later vertex, so rows that are like each
// other but not like the forest's find each other (every edge leads to a later
// vertex, so these edges close no cycle); the hierarchy is then the next update's.
// A wave a row, eight loads in flight: 1,024 rows of 9,000 columns 20 us.
constexpr uint32_t kAttachRows = 4;  // of a block

__global__ __launch_bounds__(64 * kAttachRows) void mst_attach(MstDev m, const int32_t* __restrict__ tile, uint32_t r0,
                                                               uint32_t a, uint32_t b, uint32_t cover, uint32_t at) {
  const uint32_t lane = threadIdx.x & 63u, i = a + blockIdx.x * kAttachRows + (threadIdx.x >> 6), k = m.k;
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd((unsigned long long*)&m.ps->surv, (unsigned long long)(b - a));
  if (i >= b) return;
  const uint32_t li = m.len[i];
  const int32_t* row = tile + row_off(k, r0, i) - (uint64_t)(i + 1);  // row[j]: the pair (i, j)
  const uint32_t from = max(cover, i + 1u);
  float best = -1.0f;
  uint32_t bj = from;
  int32_t bL = 0;
  for (uint32_t j0 = from; j0 < k; j0 += 8 * 64) {
    int32_t L[8];
    uint32_t lj[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t j = min(j0 + 64u * u + lane, k - 1u);
      L[u] = row[j];
      lj[u] = m.len[j];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {  // a repeated last column changes nothing
      const float d = (float)((int32_t)(li + lj[u]) - 2 * L[u]);
      const float f = d == 0.0f ? __builtin_inff() : (float)L[u] / (d * d);
      if (f > best) {
        best = f;
        bj = min(j0 + 64u * u + lane, k - 1u);
        bL = L[u];
      }
    }
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) {
    const float f = __shfl_xor(best, x, 64);
    const uint32_t j = (uint32_t)__shfl_xor((int)bj, x, 64);
    const int32_t L = __shfl_xor(bL, x, 64);
    if (f > best || (f == best && j < bj)) {
      best = f;
      bj = j;
      bL = L;
    }
  }
  const uint64_t key = sim_key(bL, li, m.len[bj]), id = (uint64_t)i * k + bj;
  if (lane == 0) {
    const uint32_t e = m.ctl->nf + at + (i - a);
    m.eu[e] = i;
    m.ev[e] = bj;
    m.ekey[e] = key;
    m.eL[e] = bL;
  }
  if (cover != 0 && lane < kMstSlots) {
    const uint32_t lab = m.view[bj].label[lane];
    const bool in = lab >= k;  // a round of the hierarchy (the forest joins bj: every round has relabelled it)
    uint64_t wk = key, wi = id;
    if (in && better(wk, wi, m.exact[bj].key[lane], m.exact[bj].id[lane])) {
      wk = m.exact[bj].key[lane];
      wi = m.exact[bj].id[lane];
    }
    m.view[i].label[lane] = in ? lab : i;
    m.view[i].bound[lane] = in ? (float)(__longlong_as_double((long long)(wk - 1ull)) * (1.0 - 0x1p-20)) : -1.0f;
    m.exact[i].key[lane] = wk;
    m.exact[i].id[lane] = wi;
  }
}

// Boruvka round r, in four launches over the whole GPU while there are more
// components or edges than one workgroup takes.  mst_edges: edges get their
// ends' labels in this round, those inside a component are dropped, the
// others offer their key to both ends' components.
constexpr uint32_t kEdgeThreads = 1024;

struct MstList {  // a round's edges; round 0's are the e* arrays themselves
  const uint32_t *u, *v, *x;
  const uint64_t* key;
};
__device__ __forceinline__ MstList mst_list(const MstDev& m, uint32_t r) {
  return r == 0 ? MstList{m.eu, m.ev, nullptr, m.ekey}
                : MstList{m.lu[r & 1], m.lv[r & 1], m.le[r & 1], m.lk[r & 1]};
}

__global__ __launch_bounds__(kEdgeThreads) void mst_edges(MstDev m, uint32_t r) {
  __shared__ BlockSlots red;
  __shared__ OfferTable table;
  MstPass* ps = m.ps;
  const uint32_t n = r == 0 ? m.ctl->nf + mst_taken(m) : ps->cnt[r - 1];
  const uint32_t nc = r == 0 ? m.k : ps->ntot - ps->hi[r - 1];
  const bool go = !mst_idle(m) && (r == 0 || ps->act[r - 1]) && n > 0 && !(nc <= kFinComps && n <= kFinEdges);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ps->act[r] = go ? 1u : 0u;
    if (r == 0) ps->cnt[0] = go ? n : 0u;
  }
  if (!go) return;
  const uint32_t step = gridDim.x * kEdgeThreads;
  if (blockIdx.x * kEdgeThreads >= n) return;
  offers_begin(&table);
  if (r == 0) {
    for (uint64_t e = blockIdx.x * kEdgeThreads + threadIdx.x; e < n; e += step) {
      const uint64_t key = m.ekey[e];
      offers_add(&table, m.c.key, m.eu[e], key);
      offers_add(&table, m.c.key, m.ev[e], key);
    }
    offers_end(&table, m.c.key);
    return;
  }
  const MstList l = mst_list(m, r - 1);
  uint32_t *du = m.lu[r & 1], *dv = m.lv[r & 1], *de = m.le[r & 1];
  uint64_t* dk = m.lk[r & 1];
  for (uint64_t e0 = blockIdx.x * kEdgeThreads; e0 < n; e0 += step) {  // uniform: every thread takes part in block_slot
    const uint64_t e = e0 + threadIdx.x;
    uint32_t a = 0, b = 0, x = 0;
    uint64_t key = 0;
    if (e < n) {
      a = m.c.nid[m.c.par[l.u[e]]];
      b = m.c.nid[m.c.par[l.v[e]]];
      x = l.x ? l.x[e] : (uint32_t)e;
      key = l.key[e];
    }
    const bool on = a != b;
    const uint32_t at = block_slot(on, &ps->cnt[r], &red);
    if (on) {
      du[at] = a;
      dv[at] = b;
      de[at] = x;
      dk[at] = key;
      offers_add(&table, m.c.key, a, key);
      offers_add(&table, m.c.key, b, key);
    }
  }
  offers_end(&table, m.c.key);
}

// Edges with their component's best key offer their id.
__global__ __launch_bounds__(kEdgeThreads) void mst_ids(MstDev m, uint32_t r) {
  if (!m.ps->act[r]) return;
  const uint32_t step = gridDim.x * kEdgeThreads, tid = blockIdx.x * kEdgeThreads + threadIdx.x, n = m.ps->cnt[r];
  if (tid == 0) m.ps->hi[r] = m.ps->ntot;
  const MstList l = mst_list(m, r);
  for (uint64_t e = tid; e < n; e += step) {
    const uint32_t a = l.u[e], b = l.v[e];
    const uint64_t key = l.key[e];
    const bool wa = m.c.key[a] == key, wb = m.c.key[b] == key;
    if (wa || wb) {
      const uint32_t x = l.x ? l.x[e] : (uint32_t)e;
      const uint64_t id = (uint64_t)m.eu[x] * m.k + m.ev[x];
      if (wa) atomicMin((unsigned long long*)&m.c.id[a], (unsigned long long)id);
      if (wb) atomicMin((unsigned long long*)&m.c.id[b], (unsigned long long)id);
    }
  }
}

// Chosen edges hook their components (two that chose the same edge hook once,
// the larger label onto the smaller) and join the new forest: the one that
// moved the component, where a caller gave the same pair twice.
__global__ __launch_bounds__(kEdgeThreads) void mst_hook(MstDev m, uint32_t r) {
  __shared__ BlockSlots red;
  if (!m.ps->act[r]) return;
  const uint32_t step = gridDim.x * kEdgeThreads, n = m.ps->cnt[r];
  const MstList l = mst_list(m, r);
  for (uint64_t e0 = blockIdx.x * kEdgeThreads; e0 < n; e0 += step) {
    const uint64_t e = e0 + threadIdx.x;
    bool wa = false, wb = false;
    uint32_t a = 0, b = 0, x = 0, u = 0, v = 0;
    uint64_t key = 0;
    if (e < n) {
      a = l.u[e];
      b = l.v[e];
      key = l.key[e];
      wa = m.c.key[a] == key;
      wb = m.c.key[b] == key;
      if (wa || wb) {
        x = l.x ? l.x[e] : (uint32_t)e;
        u = m.eu[x];
        v = m.ev[x];
        const uint64_t id = (uint64_t)u * m.k + v;
        wa = wa && m.c.id[a] == id;
        wb = wb && m.c.id[b] == id;
      }
    }
    bool in = false;
    if (wa && !(wb && a < b)) in = atomicCAS(&m.c.par[a], a, b) == a;
    if (wb && !(wa && b < a)) in = atomicCAS(&m.c.par[b], b, a) == b || in;
    const uint32_t at = block_slot(in, &m.ps->nnew, &red);
    if (in) {
      m.nu[at] = u;
      m.nv[at] = v;
      m.nkey[at] = key;
      m.nL[at] = m.eL[x];
    }
  }
}

// Every component follows its hook chain to the root (chains are acyclic:
// with a strict order on edges the only cycles of chosen edges are the mutual
// pairs, which hook once; concurrent shortcuts by other threads only move
// entries further up the same chain), and roots get the next round's labels.
// A component without an outgoing edge keeps its label for good.
__global__ __launch_bounds__(kEdgeThreads) void mst_roots(MstDev m, uint32_t r) {
  __shared__ BlockSlots red;
  MstPass* ps = m.ps;
  if (!ps->act[r] || ps->cnt[r] == 0) return;
  const uint32_t lo = r == 0 ? 0u : ps->hi[r - 1], hi = ps->hi[r];
  const uint32_t step = gridDim.x * kEdgeThreads;
  for (uint64_t c0 = lo + (uint64_t)blockIdx.x * kEdgeThreads; c0 < hi; c0 += step) {
    const uint64_t c = c0 + threadIdx.x;
    bool isroot = false;
    if (c < hi) {
      if (m.c.key[c] == 0) {
        m.c.nid[c] = (uint32_t)c;
      } else {
        uint32_t x = m.c.par[c];
        while (m.c.par[x] != x) x = m.c.par[x];
        m.c.par[c] = x;
        isroot = x == (uint32_t)c;
      }
    }
    const uint32_t at = block_slot(isroot, &ps->ntot, &red);
    if (isroot) m.c.nid[c] = at;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ps->levels = r + 1;
    m.ctl->rounds += 1;
  }
}

// The rounds that are left, in one workgroup: the same steps with the
// components' slots in LDS (24 bytes each) and barriers between them, so a
// round costs a few microseconds instead of four launches.  Fewer than half
// of the components are left after a round, so after ceil(log2(k / kFinComps))
// rounds on the whole GPU they always fit.
__global__ __launch_bounds__(kFinThreads) void mst_finish(MstDev m, uint32_t queued) {
  extern __shared__ uint64_t mst_lds[];
  uint64_t* skey = mst_lds;
  uint64_t* sid = skey + kFinComps;
  uint32_t* spar = reinterpret_cast<uint32_t*>(sid + kFinComps);
  uint32_t* sup = spar + kFinComps;
  __shared__ uint32_t s_cnt, s_new, s_forest;
  MstPass* ps = m.ps;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  if (mst_idle(m)) return;
  uint32_t r = 0;
  while (r < queued && ps->act[r]) ++r;
  uint32_t n = r == 0 ? m.ctl->nf + mst_taken(m) : ps->cnt[r - 1];
  uint32_t lo = r == 0 ? 0u : ps->hi[r - 1], tot = ps->ntot, nc = tot - lo, levels = ps->levels;
  if (n == 0 || nc > kFinComps) return;  // (never more: see above)
  MstList l = mst_list(m, r == 0 ? 0 : r - 1);
  if (tid == 0) s_forest = ps->nnew;
  uint32_t to = r & 1;
  const uint32_t levels0 = levels;
  for (bool begin = true;; begin = false) {
    for (uint32_t c = tid; c < nc; c += kFinThreads) {
      skey[c] = 0;
      sid[c] = ~0ull;
      spar[c] = c;
    }
    if (tid == 0) s_cnt = 0;
    __syncthreads();
    uint32_t *du = m.lu[to], *dv = m.lv[to], *de = m.le[to];
    uint64_t* dk = m.lk[to];
    // four edges a thread at a time, their loads in flight together
    for (uint32_t e0 = tid; e0 - lane < n; e0 += 4 * kFinThreads) {
      uint32_t a[4], b[4], x[4];
      uint64_t key[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t e = min(e0 + q * kFinThreads, n - 1u);
        a[q] = l.u[e];
        b[q] = l.v[e];
        x[q] = l.x ? l.x[e] : e;
        key[q] = l.key[e];
      }
      if (!begin) {  // labels within the last round's components
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[q] = sup[a[q]];
          b[q] = sup[b[q]];
        }
      } else if (r > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[q] = m.c.par[a[q]];
          b[q] = m.c.par[b[q]];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[q] = m.c.nid[a[q]] - lo;
          b[q] = m.c.nid[b[q]] - lo;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool on = e0 + q * kFinThreads < n && a[q] != b[q];
        const uint32_t at = wave_slot(on, &s_cnt);
        if (on) {
          du[at] = a[q];
          dv[at] = b[q];
          de[at] = x[q];
          dk[at] = key[q];
          offer(&skey[a[q]], key[q]);
          offer(&skey[b[q]], key[q]);
        }
      }
    }
    __threadfence_block();
    __syncthreads();
    n = s_cnt;
    if (n == 0) break;
    l = MstList{du, dv, de, dk};
    to ^= 1u;
    for (uint32_t e0 = tid; e0 < n; e0 += 4 * kFinThreads) {
      uint32_t a[4], b[4];
      uint64_t key[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t e = min(e0 + q * kFinThreads, n - 1u);  // a repeated edge offers the same id again
        a[q] = l.u[e];
        b[q] = l.v[e];
        key[q] = l.key[e];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool wa = skey[a[q]] == key[q], wb = skey[b[q]] == key[q];
        if (wa || wb) {
          const uint32_t x = l.x[min(e0 + q * kFinThreads, n - 1u)];
          const uint64_t id = (uint64_t)m.eu[x] * m.k + m.ev[x];
          if (wa) atomicMin((unsigned long long*)&sid[a[q]], (unsigned long long)id);
          if (wb) atomicMin((unsigned long long*)&sid[b[q]], (unsigned long long)id);
        }
      }
    }
    if (tid == 0) s_new = 0;
    __syncthreads();
    for (uint32_t e0 = tid; e0 - lane < n; e0 += 4 * kFinThreads) {
      uint32_t a[4], b[4];
      uint64_t key[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t e = min(e0 + q * kFinThreads, n - 1u);
        a[q] = l.u[e];
        b[q] = l.v[e];
        key[q] = l.key[e];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t e = e0 + q * kFinThreads;
        bool wa = e < n && skey[a[q]] == key[q], wb = e < n && skey[b[q]] == key[q];
        uint32_t x = 0, u = 0, v = 0;
        if (wa || wb) {
          x = l.x[e];
          u = m.eu[x];
          v = m.ev[x];
          const uint64_t id = (uint64_t)u * m.k + v;
          wa = wa && sid[a[q]] == id;
          wb = wb && sid[b[q]] == id;
        }
        bool in = false;
        if (wa && !(wb && a[q] < b[q])) in = atomicCAS(&spar[a[q]], a[q], b[q]) == a[q];
        if (wb && !(wa && b[q] < a[q])) in = atomicCAS(&spar[b[q]], b[q], a[q]) == b[q] || in;
        const uint32_t at = wave_slot(in, &s_forest);
        if (in) {
          m.nu[at] = u;
          m.nv[at] = v;
          m.nkey[at] = key[q];
          m.nL[at] = m.eL[x];
        }
      }
    }
    __syncthreads();
    for (uint32_t c = tid; c < nc; c += kFinThreads) {
      uint32_t x = spar[c];
      while (spar[x] != x) x = spar[x];
      sup[c] = x;
      m.c.key[lo + c] = skey[c];
      m.c.id[lo + c] = sid[c];
      m.c.par[lo + c] = lo + x;
    }
    __syncthreads();
    for (uint32_t c0 = tid & ~63u; c0 < nc; c0 += kFinThreads) {
      const uint32_t c = c0 + lane;
      const bool live = c < nc && skey[c] != 0;
      const bool isroot = live && sup[c] == c;
      const uint32_t at = wave_slot(isroot, &s_new);
      if (c < nc && !live) m.c.nid[lo + c] = lo + c;
      if (isroot) {
        m.c.nid[lo + c] = tot + at;
        spar[c] = at;
      }
    }
    __syncthreads();
    for (uint32_t c = tid; c < nc; c += kFinThreads)
      if (skey[c] != 0) sup[c] = spar[sup[c]];  // (a component without an edge has no edges to relabel)
    lo = tot;
    nc = s_new;
    tot += nc;
    ++levels;
    __syncthreads();  // s_new and the slots are reused by the next round
  }
  if (tid == 0) {
    ps->levels = levels;
    ps->ntot = tot;
    ps->nnew = s_forest;
    m.ctl->rounds += levels - levels0;
  }
}

// A pass whose survivors do not fit, on an empty list: the list is empty again.
__global__ void mst_forget(MstPass* ps) { ps->surv = 0; }

// The hierarchy of this update, per vertex, for the next pass; the new forest
// becomes the current one, and the next update's components and counters are
// cleared.  `init`: no forest yet, every vertex by itself.
__global__ __launch_bounds__(256) void mst_view(MstDev m, uint32_t init) {
  mst_clear(m.next, m.ps_next, m.k);
  const uint32_t step = gridDim.x * blockDim.x, tid = blockIdx.x * blockDim.x + threadIdx.x;
  if (init && tid == 0) {
    m.ctl->nf = 0;
    m.ctl->rounds = 0;
  }
  if (!init && mst_idle(m)) return;
  const uint32_t D = init ? 0u : m.ps->levels, nnew = init ? 0u : m.ps->nnew;
  for (uint64_t v = tid; v < m.k; v += step) {
    MstView& w = m.view[v];
    MstExact& x = m.exact[v];
    uint32_t c = (uint32_t)v;
    uint64_t key = ~0ull, id = 0;  // nothing chosen yet
    for (uint32_t s = D; s < kMstSlots; ++s) {  // round 0 and the slots past it
      w.label[s] = (uint32_t)v;
      w.bound[s] = -1.0f;
    }
    for (uint32_t l = 1; l <= D; ++l) {
      const uint64_t ck = m.c.key[c];
      if (ck != 0) {
        const uint64_t ci = m.c.id[c];
        if (better(key, id, ck, ci)) {
          key = ck;
          id = ci;
        }
        c = m.c.nid[m.c.par[c]];
      }
      const uint32_t s = D - l;
      if (s < kMstSlots) {
        w.label[s] = c;
        w.bound[s] = (float)(__longlong_as_double((long long)(key - 1ull)) * (1.0 - 0x1p-20));
        x.key[s] = key;
        x.id[s] = id;
      }
    }
  }
  for (uint64_t e = tid; e < nnew; e += step) {
    m.eu[e] = m.nu[e];
    m.ev[e] = m.nv[e];
    m.ekey[e] = m.nkey[e];
    m.eL[e] = m.nL[e];
  }
  if (!init && tid == 0) m.ctl->nf = nnew;
}

}  // namespace famsa

using namespace famsa;

struct famsa_mst_s {
  uint32_t k = 0;
  int device = 0;
  uint32_t surv_cap = 0;       // survivors an update holds: at least one row's pairs
  uint32_t cover = 0xFFFFFFFFu;  // the forest joins all vertices from this one on
  DevMem mem;                  // every array below, in one allocation
  MstDev dev{};
  size_t read_bytes = 0;  // ctl, the last update's forest and the lengths, from mem's start
  PinMem hflag;
  uint64_t tiles = 0;
  // Tiles arrive on whatever stream their producer used (a plan alternates
  // two); this event marks the end of the last tile's work, and the next
  // tile's work waits for it, so merges never overlap whatever the streams.
  hipEvent_t last = nullptr;
  hipEvent_t read = nullptr;  // the last pass over a tile is done
  bool has_last = false;
  bool kinds = false;    // a block of rows tied to the forest by its own vertices alone let too many pairs through
  uint32_t pending = 0;  // survivors that the forest has not taken in yet
  uint32_t blocks = 0;   // of the passes they are from
  std::mutex mu;         // reading the forest takes them in
  ~famsa_mst_s() {
    if (last) {
      if (has_last) (void)hipEventSynchronize(last);
      (void)hipEventDestroy(last);
    }
    if (read) (void)hipEventDestroy(read);
  }
  int layout();
  struct Rows {  // rows t0..t1-1 of stride `stride` in a tile; skip: every eighth left out
    uint32_t t0, t1, stride, skip;
  };
  int filter(const famsa_lcs_tile* t, const Rows& rows, bool take, hipStream_t s, bool* fits);
  int update(uint32_t n, uint64_t most, hipStream_t s);
  int settle();
  int attach(const famsa_lcs_tile* t, uint32_t a, uint32_t b, uint32_t from, hipStream_t s);
  int merge_block(const famsa_lcs_tile* t, uint32_t a, uint32_t b, bool more, hipStream_t s);
  int merge_rows(const famsa_lcs_tile* t, const Rows& rows, bool covered, hipStream_t s);
  int merge_upwards(const famsa_lcs_tile* t, hipStream_t s);
  int merge_tile(const famsa_lcs_tile* t, hipStream_t s);
};

// One allocation, most of it room for survivors: 1.2 KB a vertex and 0.96 KB
// more for the first 8,192 (2.2 KB a vertex for small families, 129 MB for
// 100,000); past a million vertices 0.43 KB a vertex and 0.5 GB.
int famsa_mst_s::layout() {
  const uint64_t n = std::max<uint32_t>(k, 1);
  const uint64_t pairs = n * (n - 1) / 2;
  const uint64_t room = k <= (1u << 20) ? 14 * n + std::min<uint64_t>(16 * n, 1u << 17) : n + (8u << 20);
  surv_cap = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({pairs, room, 0xFFFFFFF0ull - n}));
  const uint64_t E = n + surv_cap;
  uint64_t off = 0;
  auto part = [&](uint64_t bytes) {
    const uint64_t at = off;
    off += (bytes + 255) & ~255ull;
    return at;
  };
  // first what a reader copies, in one piece
  const uint64_t o_ctl = part(sizeof(MstCtl)), o_nu = part(4 * n), o_nv = part(4 * n), o_nL = part(4 * n),
                 o_len = part(4 * n);
  read_bytes = off;
  const uint64_t o_eu = part(4 * E), o_ev = part(4 * E), o_ek = part(8 * E), o_eL = part(4 * E), o_nk = part(8 * n),
                 o_lk = part(16 * E), o_l = part(24 * E), o_ck = part(32 * n),
                 o_ci = part(32 * n), o_pa = part(16 * n), o_ni = part(16 * n), o_ps = part(2 * sizeof(MstPass)),
                 o_vw = part(sizeof(MstView) * n), o_ex = part(sizeof(MstExact) * n);
  int rc = mem.alloc(off);
  if (rc) return rc;
  if ((rc = hflag.alloc(64))) return rc;
  uint8_t* b = mem.as<uint8_t>();
  MstDev& d = dev;
  d.k = k;
  d.room = surv_cap;
  d.len = reinterpret_cast<uint32_t*>(b + o_len);
  d.ctl = reinterpret_cast<MstCtl*>(b + o_ctl);
  d.eu = reinterpret_cast<uint32_t*>(b + o_eu);
  d.ev = reinterpret_cast<uint32_t*>(b + o_ev);
  d.ekey = reinterpret_cast<uint64_t*>(b + o_ek);
  d.eL = reinterpret_cast<int32_t*>(b + o_eL);
  d.nu = reinterpret_cast<uint32_t*>(b + o_nu);
  d.nv = reinterpret_cast<uint32_t*>(b + o_nv);
  d.nkey = reinterpret_cast<uint64_t*>(b + o_nk);
  d.nL = reinterpret_cast<int32_t*>(b + o_nL);
  for (int i = 0; i < 2; ++i) {
    uint32_t* l = reinterpret_cast<uint32_t*>(b + o_l) + 3 * E * i;
    d.lu[i] = l;
    d.lv[i] = l + E;
    d.le[i] = l + 2 * E;
    d.lk[i] = reinterpret_cast<uint64_t*>(b + o_lk) + E * i;
    (i ? d.next : d.c) = MstComp{reinterpret_cast<uint64_t*>(b + o_ck) + 2 * n * i,
                                 reinterpret_cast<uint64_t*>(b + o_ci) + 2 * n * i,
                                 reinterpret_cast<uint32_t*>(b + o_pa) + 2 * n * i,
                                 reinterpret_cast<uint32_t*>(b + o_ni) + 2 * n * i};
    (i ? d.ps_next : d.ps) = reinterpret_cast<MstPass*>(b + o_ps) + i;
  }
  d.view = reinterpret_cast<MstView*>(b + o_vw);
  d.exact = reinterpret_cast<MstExact*>(b + o_ex);
  d.host = hflag.as<uint32_t>();
  return 0;
}

static inline uint32_t grid_for(uint64_t n, uint32_t threads) {
  return (uint32_t)std::min<uint64_t>(512, std::max<uint64_t>(1, (n + threads - 1) / threads));
}

// The pass over some of the tile's rows; the host waits for it and so knows
// the survivors so far.  *fits: all of them are in the list; else
// the list is what it was before.  take (on an empty list): the update that
// takes them in, if they fit, is queued behind the pass without waiting.
int famsa_mst_s::filter(const famsa_lcs_tile* t, const Rows& rows, bool take, hipStream_t s, bool* fits) {
  const uint32_t r0 = t->row_begin, r1 = t->row_end;
  const MstDev& m = dev;
  const uint32_t nrows = rows.t1 - rows.t0;
  // blocks of 128 columns; a slice of rows so that about 256 blocks share the
  // tile (the survivors' appends are one atomic a block), 64 rows at least:
  // four for each wave
  const uint32_t j0 = (uint32_t)((r0 + (uint64_t)rows.t0 * rows.stride + 1ull) & ~63ull);
  const uint32_t strips = (k - j0 + 64u * kFiltCols - 1u) / (64u * kFiltCols);
  const uint32_t per = kFiltWaves * kFiltChunk;
  const uint32_t want = std::max(1u, 256u / strips);
  const uint32_t slice = (std::max(1u, (nrows + want - 1) / want) + per - 1) / per * per;
  const dim3 g(strips, (nrows + slice - 1) / slice);
  blocks += g.x * g.y;
  hipLaunchKernelGGL(mst_filter, g, dim3(64 * kFiltWaves), 0, s, m, m.view, m.len, t->lcs, r0, r1, rows.t0, rows.t1,
                     slice, rows.stride, rows.skip, j0, blocks - 1u);
  FAMSA_HIP(hipGetLastError());
  if (take) {
    FAMSA_HIP(hipEventRecord(read, s));
    const int rc = update(kAll, (uint64_t)nrows * (k - 1 - (r0 + rows.t0 * rows.stride)), s);
    if (rc) return rc;
    FAMSA_HIP(hipEventSynchronize(read));
    *fits = *static_cast<volatile uint32_t*>(hflag.p) <= surv_cap;
    return 0;
  }
  FAMSA_HIP(hipEventRecord(last, s));
  has_last = true;
  FAMSA_HIP(hipEventSynchronize(last));
  const uint32_t n = *static_cast<volatile uint32_t*>(hflag.p);
  *fits = n <= surv_cap;
  if (*fits) {
    pending = n;
  } else if (pending == 0) {
    hipLaunchKernelGGL(mst_forget, dim3(1), dim3(1), 0, s, m.ps);
    FAMSA_HIP(hipGetLastError());
    FAMSA_HIP(hipEventRecord(last, s));
    blocks = 0;
  }
  return 0;
}

// The forest takes in the survivors so far, n of them (or kAll, at most
// `most`).  Launches are queued without waiting; kernels of rounds that are
// not needed return at once.
int famsa_mst_s::update(uint32_t n, uint64_t most, hipStream_t s) {
  if (n == 0) return 0;
  dev.n = n;
  const MstDev& m = dev;
  most = std::min<uint64_t>(most, surv_cap);
  uint32_t rounds = 0;  // on the whole GPU
  while ((k >> rounds) >= kFinComps && rounds < 32) ++rounds;  // then fewer than kFinComps are left
  if (k <= kFinComps) rounds = 0;
  // many survivors: one workgroup takes 82 us and more over what two rounds
  // leave of 70,000 edges, a round on the whole GPU 30 (k = 12,000 sequences
  // of 60 residues in all: 3.2 ms with no more rounds, 2.9 with two, 2.6 with
  // four, 2.6 with five).  With no more components than it takes from the
  // start, most edges stay between two of them round after round: k = 4,000 in
  // one tile, LCS and all, 998 us with two rounds whatever the edges, 936 with
  // two or four, 905 with three or five
  if (most > 2 * kFinEdges) rounds += k > kFinComps ? 4 : (most > 4 * kFinEdges ? 5 : 3);
  most += k;  // edges
  const dim3 ge(grid_for(most, kEdgeThreads)), gc(grid_for(k, kEdgeThreads)), b(kEdgeThreads);
  for (uint32_t r = 0; r < rounds; ++r) {
    hipLaunchKernelGGL(mst_edges, ge, b, 0, s, m, r);
    hipLaunchKernelGGL(mst_ids, ge, b, 0, s, m, r);
    hipLaunchKernelGGL(mst_hook, ge, b, 0, s, m, r);
    hipLaunchKernelGGL(mst_roots, gc, b, 0, s, m, r);
  }
  hipLaunchKernelGGL(mst_finish, dim3(1), dim3(kFinThreads), kFinLds, s, m, rounds);
  hipLaunchKernelGGL(mst_view, dim3(grid_for(2ull * k, 256)), dim3(256), 0, s, m, 0u);
  FAMSA_HIP(hipGetLastError());
  FAMSA_HIP(hipEventRecord(last, s));
  has_last = true;
  // the next update's components and counters are cleared by this one
  std::swap(dev.c, dev.next);
  std::swap(dev.ps, dev.ps_next);
  pending = 0;
  blocks = 0;
  return 0;
}

// The forest of every tile so far, for a reader.
int famsa_mst_s::settle() {
  if (!has_last) return 0;
  if (pending) {
    hipStream_t s = nullptr;
    int rc = lib_stream(device, 0, &s);
    if (rc) return rc;
    FAMSA_HIP(hipStreamWaitEvent(s, last, 0));
    if ((rc = update(pending, pending, s))) return rc;
  }
  FAMSA_HIP(hipEventSynchronize(last));
  return 0;
}

// Most tiles are one pass.  An update costs 150 us and more, whatever it takes
// in, so survivors wait in the list until they are six a vertex, or the list
// has no room for the next pass, or the forest is read.  A pass against an
// older hierarchy lets more pairs through, but not many: where the rows seen
// double, about one a vertex.  Twelve tiles of k = 12,000 sequences of 60
// residues take 4.0 ms with an update each, 3.2 with one every two survivors a
// vertex, 2.6 every five, 2.5 every eight; k = 30,000 of 250 66.0, 64.9, 64.4
// and 64.1.
// Where the forest does not join the rows' vertices yet, or the survivors of all
// rows do not fit, the rows are taken in passes of growing size spread over
// them, every 8^n-th row first, with an update after each: the first pass fits
// (one row's pairs always do), and each pass's forest then drops most pairs of
// the next (a row seldom beats eight times as many like it).  A pass whose
// survivors do not fit is halved.
int famsa_mst_s::merge_rows(const famsa_lcs_tile* t, const Rows& all, bool covered, hipStream_t s) {
  const uint32_t R = all.t1 - all.t0;
  const uint32_t first = std::max(1u, surv_cap / k);  // rows whose pairs fit, all of them
  const uint32_t wait = (uint32_t)std::min(6ull * k, surv_cap / 3ull);
  std::vector<Rows> todo;  // last first
  auto passes = [&]() {
    uint32_t st = 1;
    while ((R + st - 1) / st > first) st *= 8;
    std::vector<Rows> p;
    for (uint32_t skip = 0;; skip = 1, st /= 8) {
      p.push_back(Rows{0, (R + st - 1) / st, st, skip});
      if (st == 1) break;
    }
    todo.insert(todo.end(), p.rbegin(), p.rend());
  };
  uint64_t pairs = 0;
  for (uint32_t x = all.t0; x < all.t1 && pairs <= surv_cap; ++x) pairs += k - 1 - (t->row_begin + x);
  const bool spread = all.t0 == 0;  // passes count a tile's rows from its first
  if (covered || pairs <= surv_cap || !spread) todo.push_back(all);
  else passes();
  while (!todo.empty()) {
    const Rows rows = todo.back();
    todo.pop_back();
    const uint32_t mid = rows.t0 + (rows.t1 - rows.t0) / 2;
    // survivors are counted in 32 bits
    if ((uint64_t)(rows.t1 - rows.t0) * k + pending > 0xFFFFFFFFull && mid > rows.t0) {
      todo.push_back(Rows{mid, rows.t1, rows.stride, rows.skip});
      todo.push_back(Rows{rows.t0, mid, rows.stride, rows.skip});
      continue;
    }
    bool fits = false;
    int rc = 0;
    if (!covered && pending && (rc = update(pending, pending, s))) return rc;
    if ((rc = filter(t, rows, !covered, s, &fits))) return rc;
    if (fits) {
      if (pending > wait && (rc = update(pending, pending, s))) return rc;
      continue;
    }
    if (pending) {  // room first
      if ((rc = update(pending, pending, s))) return rc;
      todo.push_back(rows);
      continue;
    }
    if (rows.t1 - rows.t0 <= 1) return set_error(FAMSA_LCS_EDEVICE, "one row's pairs do not fit");
    if (spread && rows.stride == 1 && rows.skip == 0 && rows.t0 == 0 && rows.t1 == R && R > 8) {
      passes();
    } else {
      todo.push_back(Rows{mid, rows.t1, rows.stride, rows.skip});
      todo.push_back(Rows{rows.t0, mid, rows.stride, rows.skip});
    }
  }
  return 0;
}

// Ties rows a..b-1 (family-local) of the tile to the forest (from = cover), or
// to any later vertex (from = 0).
int famsa_mst_s::attach(const famsa_lcs_tile* t, uint32_t a, uint32_t b, uint32_t from, hipStream_t s) {
  int rc = 0;
  if (pending + (b - a) > surv_cap && (rc = update(pending, pending, s))) return rc;
  hipLaunchKernelGGL(mst_attach, dim3((b - a + kAttachRows - 1) / kAttachRows), dim3(64 * kAttachRows), 0, s, dev, t->lcs,
                     t->row_begin, a, b, from, pending);
  FAMSA_HIP(hipGetLastError());
  pending += b - a;
  return 0;
}

// Rows a..b-1, above the forest's vertices: tied to them, then one pass.  more:
// rows above these follow at once, so the update does too, behind the pass.
// Rows of kinds that the forest has none of (families listed clade by clade) let
// all pairs of their kind through; where these do not fit, such rows are tied to
// each other as well, and the forest takes that in before the pass.
int famsa_mst_s::merge_block(const famsa_lcs_tile* t, uint32_t a, uint32_t b, bool more, hipStream_t s) {
  const Rows rows{a - t->row_begin, b - t->row_begin, 1, 0};
  // so does it where nothing is left to come and the survivors are few whatever
  // their number (else the exact number saves the rounds that it does not need)
  const bool take = more || (a == 0 && !pending && std::min<uint64_t>((uint64_t)(b - a) * (k - 1), surv_cap) <= 2 * kFinEdges);
  int rc = 0;
  if (more && pending && (rc = update(pending, pending, s))) return rc;
  if (!kinds) {
    if ((rc = attach(t, a, b, cover, s))) return rc;
    if (take) pending = 0;  // the update behind the pass counts the list itself
    bool fits = false;
    if ((rc = filter(t, rows, take, s, &fits))) return rc;
    if (fits) return 0;
    kinds = true;
  }
  if (pending && (rc = update(pending, pending, s))) return rc;
  if ((rc = attach(t, a, b, 0, s)) || (rc = update(pending, pending, s))) return rc;
  return merge_rows(t, rows, true, s);
}

// A tile above the vertices that the forest joins (tiles in descending order),
// or at the end of the triangle (a family in one tile): its rows are taken
// from the last one up, each block of them tied to the forest first and then
// in one pass against it, as many rows as kUpRatio times the forest's vertices.
// The first kUpFirst rows of all are taken with all their pairs.  With passes
// spread over the tile instead, every tile in descending order cost three
// updates (k = 9,000 of 60 residues in tiles of 1,024 rows, LCS and all:
// 5.9 ms, now 1.7; dense rounds over every tile 4.6), and a family in one tile
// four, of many survivors each (k = 4,000: 1.54 ms, now 0.87; dense rounds
// 0.97).  First rows and ratio, k = 700, 2,000 and 4,000 in one tile: 128 and 7
// 429, 627, 873 us; 128 and 5 429, 662, 887; 160 and 4 474, 718, 934; 256 and
// 3 514, 670, 904.
constexpr uint32_t kUpFirst = 128, kUpRatio = 7;

int famsa_mst_s::merge_upwards(const famsa_lcs_tile* t, hipStream_t s) {
  const uint32_t r0 = t->row_begin, r1 = std::min(t->row_end, k - 1);
  int rc = 0;
  uint32_t b = r1;
  if (cover < b) {
    if ((rc = merge_rows(t, Rows{cover - r0, b - r0, 1, 0}, true, s))) return rc;
    b = cover;
  }
  while (b > r0) {
    uint32_t n;
    if (cover >= k - 1) {  // no forest: b is k - 1
      n = std::min(b - r0, kUpFirst);
      while ((uint64_t)n * (n + 1) / 2 > surv_cap) n /= 2;  // (one pair always fits)
      if ((rc = merge_rows(t, Rows{b - n - r0, b - r0, 1, 0}, false, s))) return rc;
    } else {
      const uint64_t most = std::min<uint64_t>((uint64_t)std::max(k - cover, 64u) * kUpRatio, surv_cap / 2);
      n = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({b - r0, most, 0xF0000000u / k}));  // survivors in 32 bits
      if ((rc = merge_block(t, b - n, b, n < b - r0, s))) return rc;
    }
    b -= n;
    cover = b;
  }
  return 0;
}

int famsa_mst_s::merge_tile(const famsa_lcs_tile* t, hipStream_t s) {
  const uint32_t r0 = t->row_begin, r1 = t->row_end;
  if (r1 - r0 > 65535u) return set_error(FAMSA_LCS_EINVAL, "tiles of more than 65535 rows are not supported");
  if (!t->count) {
    ++tiles;
    return 0;
  }
  if (has_last) FAMSA_HIP(hipStreamWaitEvent(s, last, 0));  // the previous tile's merge, on any stream
  const uint32_t R = std::min(r1, k - 1) - r0;  // rows with a pair
  int rc;
  const bool joined = r0 >= cover, none = cover >= k - 1;  // the forest joins every vertex of the tile, or nothing yet
  const bool above = !joined && std::min(r1, k - 1) >= std::min(cover, k - 1);  // or all from the tile's end on
  if (above && !(none && t->count <= surv_cap)) rc = merge_upwards(t, s);
  else rc = merge_rows(t, Rows{0, R, 1, 0}, joined, s);
  if (rc) return rc;
  cover = std::min(cover, r0);
  ++tiles;
  return 0;
}

extern "C" {

int famsa_mst_create(const uint32_t* lengths, uint32_t k, int device, famsa_mst_t** out) {
  clear_error();
  if (!out) return set_error(FAMSA_LCS_EINVAL, "out is NULL");
  *out = nullptr;
  if (k && !lengths) return set_error(FAMSA_LCS_EINVAL, "lengths is NULL");
  if (k > (1u << 31)) return set_error(FAMSA_LCS_EINVAL, "k %u too large", k);
  for (uint32_t i = 0; i < k; ++i)
    if (lengths[i] > FAMSA_LCS_MAX_LEN)
      return set_error(FAMSA_LCS_EINVAL, "length %u of sequence %u exceeds %u", lengths[i], i, FAMSA_LCS_MAX_LEN);
  if (device < 0) return set_error(FAMSA_LCS_EINVAL, "device %d < 0", device);
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) {
    (void)hipGetLastError();
    return set_error(FAMSA_LCS_EDEVICE, "no HIP device available");
  }
  if (device >= ndev) return set_error(FAMSA_LCS_EINVAL, "device %d >= device count %d", device, ndev);
  FAMSA_HIP(hipSetDevice(device));
  famsa_mst_s* m = new (std::nothrow) famsa_mst_s();
  if (!m) return set_error(FAMSA_LCS_ENOMEM, "out of host memory");
  m->k = k;
  m->device = device;
  int rc = m->layout();
  if (rc) {
    delete m;
    return rc;
  }
  hipStream_t st = nullptr;
  if ((rc = lib_stream(device, 0, &st))) {
    delete m;
    return rc;
  }
  if (hipEventCreateWithFlags(&m->last, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&m->read, hipEventDisableTiming) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&mst_finish), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)kFinLds) != hipSuccess) {
    delete m;
    return set_error(FAMSA_LCS_EDEVICE, "setting up the forest failed");
  }
  if ((k && hipMemcpyAsync(const_cast<uint32_t*>(m->dev.len), lengths, (size_t)k * 4, hipMemcpyHostToDevice, st) !=
                hipSuccess)) {
    delete m;
    return set_error(FAMSA_LCS_EDEVICE, "initialising the forest failed");
  }
  hipLaunchKernelGGL(mst_view, dim3(grid_for(2ull * k, 256)), dim3(256), 0, st, m->dev, 1u);
  // the lengths are the caller's: wait for their copy
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
    delete m;
    return set_error(FAMSA_LCS_EDEVICE, "initialising the forest failed");
  }
  std::swap(m->dev.c, m->dev.next);
  std::swap(m->dev.ps, m->dev.ps_next);
  *out = m;
  return 0;
}

int famsa_mst_consume(void* user, const famsa_lcs_tile* t) {
  famsa_mst_s* m = static_cast<famsa_mst_s*>(user);
  if (!m || !t || t->k != m->k || t->row_begin > t->row_end || t->row_end > m->k) return 1;
  if (t->count && !t->lcs) return 1;
  if (t->values != FAMSA_LCS_VALUES_LCS) return 1;  // the forest is built from LCS values
  if (t->count != tri_rows(m->k, t->row_begin, t->row_end)) return 1;
  if (hipSetDevice(m->device) != hipSuccess) return 1;
  std::lock_guard<std::mutex> lock(m->mu);
  return m->merge_tile(t, (hipStream_t)t->stream) == 0 ? 0 : 1;
}

int famsa_mst_result(const famsa_mst_t* m, uint32_t* u, uint32_t* v, int64_t* lcs, int64_t* indel2,
                     uint32_t* nedges) {
  clear_error();
  if (!m || !nedges) return set_error(FAMSA_LCS_EINVAL, "NULL argument");
  FAMSA_HIP(hipSetDevice(m->device));
  famsa_mst_s* const f = const_cast<famsa_mst_s*>(m);
  std::lock_guard<std::mutex> lock(f->mu);
  int rc = f->settle();
  if (rc) return rc;
  std::vector<uint8_t> h(m->read_bytes);
  if ((rc = copy_now(m->device, h.data(), m->mem.p, h.size(), hipMemcpyDeviceToHost))) return rc;
  auto at = [&](const void* d) { return h.data() + (static_cast<const uint8_t*>(d) - m->mem.as<uint8_t>()); };
  const uint32_t n = reinterpret_cast<const MstCtl*>(at(m->dev.ctl))->nf;
  const uint32_t *hu = reinterpret_cast<const uint32_t*>(at(m->dev.nu)), *hv = reinterpret_cast<const uint32_t*>(at(m->dev.nv));
  const uint32_t* hl = reinterpret_cast<const uint32_t*>(at(m->dev.len));
  const int32_t* hL = reinterpret_cast<const int32_t*>(at(m->dev.nL));
  for (uint32_t e = 0; e < n; ++e) {
    if (u) u[e] = hu[e];
    if (v) v[e] = hv[e];
    if (lcs) lcs[e] = hL[e];
    const int64_t d = (int64_t)hl[hu[e]] + hl[hv[e]] - 2 * (int64_t)hL[e];
    if (indel2) indel2[e] = d * d;
  }
  *nedges = n;
  return 0;
}

int famsa_mst_guide_tree(const famsa_mst_t* m, uint32_t* left, uint32_t* right, int64_t* lcs, int64_t* indel2,
                         uint32_t* nmerges) {
  clear_error();
  if (!m || !nmerges) return set_error(FAMSA_LCS_EINVAL, "NULL argument");
  const size_t n = std::max<uint32_t>(m->k, 1);
  std::vector<uint32_t> u(n), v(n);
  std::vector<int64_t> L(n), D(n);
  uint32_t ne = 0;
  int rc = famsa_mst_result(m, u.data(), v.data(), L.data(), D.data(), &ne);
  if (rc) return rc;
  return guide_tree(m->k, u.data(), v.data(), L.data(), D.data(), ne, left, right, lcs, indel2, nmerges);
}

int famsa_mst_get_stats(const famsa_mst_t* m, uint64_t* tiles, uint64_t* rounds) {
  clear_error();
  if (!m) return set_error(FAMSA_LCS_EINVAL, "mst is NULL");
  FAMSA_HIP(hipSetDevice(m->device));
  famsa_mst_s* const f = const_cast<famsa_mst_s*>(m);
  std::lock_guard<std::mutex> lock(f->mu);
  int rc = f->settle();
  if (rc) return rc;
  MstCtl c;
  if ((rc = copy_now(m->device, &c, m->dev.ctl, sizeof c, hipMemcpyDeviceToHost))) return rc;
  if (tiles) *tiles = m->tiles;
  if (rounds) *rounds = c.rounds;
  return 0;
}

void famsa_mst_destroy(famsa_mst_t* m) {
  if (!m) return;
  (void)hipSetDevice(m->device);
  delete m;  // waits for the last tile's work
}

}  // extern "C"
