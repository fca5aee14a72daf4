// Path-tree kernels: level-synchronous extension of simple paths, the
// backward-extendability filter, canonical-order ranking and prime-path
// materialization.
//
// What is computed (paper Sec. 5, Update-Vertex and ExtendPath; Def. 1):
//  * level 1 holds one path <v> per vertex (the host initialisation of the
//    paper's algorithm puts each vertex on its own list);
//  * a path p = (v1..vL) that has not closed a cycle is extended by every
//    successor w of vL that is not on p, and by w = v1, which closes a cycle;
//  * a path that gets no extension at all is terminal; a terminal path is a
//    prime path iff it cannot be extended backward, i.e. every predecessor of
//    v1 lies on p (the pruning of paths covered by a longer path ending at the
//    same vertex); every closed cycle is a prime path.
//
// How (the paper's asynchronous thread-per-vertex schedule and its per-vertex
// path tables are not used):
//  * The graph's straight lines (chains) are taken as single vertices, so a
//    node of the tree is a path of chains, and level L holds the paths of L
//    chains.  That is exact: an acyclic prime path is made of whole chains, a
//    cycle through a chain starts at each of its vertices once (k_rotations),
//    and the simple paths that begin or end inside a chain follow from the
//    chains' lengths (k_path_lengths).  A CFG's statements sit mostly on such
//    lines: the 400-vertex stress CFG has 189 chains, and its tree 1.85e8
//    nodes on 36 levels instead of 4.66e8 on 213; a ~200-vertex CFG about a
//    quarter of the nodes and half the levels.  A whole call
//    on it takes 17.8 ms, one on a 212-vertex CFG 1.74, on a 1000-vertex one
//    (174 chains) 2.1, and a batch of 4096 5.6 (each kernel below has its own
//    share of that).  "Vertex" below means a vertex of the graph of chains.
//  * All paths of one level form a frontier of (parent index, vertex) nodes;
//    the children of one parent are contiguous and in ascending successor
//    order, and each node records where its children start and how many
//    there are.
//  * The visited set of a frontier path lives as a bitmask of W 64-bit words
//    (registers while testing).  In HBM only the odd levels' sets are kept,
//    two stored levels alive: a path on an even level is a path of the odd
//    level before plus its last vertex, so its set is rebuilt from its
//    parent's (siblings read the same stored set).  Sets are stored
//    word-major: word q of slot j sits at q * stride + j, so the threads of
//    a wave, which own consecutive slots, read and write consecutive words.
//  * One workgroup handles a tile of its threads * ITEMS parents: choice masks
//    over successor slots, a block scan of child counts, then ONE device-scope
//    atomic claim of the tile's slice of the next level, then the children's
//    records and sets on neighbouring slots.  No workgroup ever
//    waits for another one; the order of tile slices inside a level is the
//    order in which the claims landed, which ranking does not depend on.
//  * Levels follow each other on the device: per-level counts and offsets
//    live in device memory; a launch extends the level that the one before
//    it has left (narrow levels many at a time, see LevelCursor) and derives
//    its offset from the level before, or raises the overflow flag when that
//    level's nodes did not fit; the host then grows the buffers to the exact
//    size and replays the level.
//  * The plain two-pass form (count, scan, host-visible size, fill) keeps
//    children in parent order and serves as the exact reference form.

#include <hip/hip_ext.h>

#include <type_traits>

#include "kernels.h"
#include "sizing.h"

namespace tpg {

// ---------------------------------------------------------------------------
// level 1
// ---------------------------------------------------------------------------
__global__ void k_seed(ExtArgs a, int limit, int64_t tot_words) {
  const int n = a.seed_n;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  LevelState* ls = a.ls;
  // every level's claim counter starts at zero
  for (int64_t k = i; k < kMaxLevels; k += (int64_t)gridDim.x * blockDim.x) {
    ls->count[k] = k == 1 ? n : 0;
    ls->off[k] = 0;
  }
  if (i == 0) {
    ls->batch_start = 1;
    ls->limit = limit;
    ls->overflow = 0;
    ls->overflow_level = 0;
  }
  if (i < n) {
    const int v = a.seed_lo + (int)i;
    a.t.par[i] = -1;
    a.t.info[i] = make_info(v, a.g.loc[v], 0);
    a.t.tl[i] = (uint16_t)a.g.len[v];
  }
  for (int64_t k = i; k < tot_words; k += (int64_t)gridDim.x * blockDim.x) a.tot[k] = 0;
  // visited sets of level 1 (stored, buffer 0): one bit each, at the
  // chain's local id
  const int W = a.t.mask_words;
  for (int64_t k = i; k < (int64_t)n * W; k += (int64_t)gridDim.x * blockDim.x) {
    const int q = (int)(k / n), j = (int)(k % n);
    const int l = a.g.loc[a.seed_lo + j];
    a.t.mask[0][(int64_t)q * a.t.mask_cap + j] = (q == (l >> 6)) ? (1ull << (l & 63)) : 0ull;
  }
}

hipError_t launch_seed(const ExtArgs& a, int limit, hipStream_t st) {
  if (limit < 1 || limit > kMaxLevels - 2) return hipErrorInvalidValue;
  if (a.seed_lo < 0 || a.seed_n < 1 || a.seed_lo + a.seed_n > a.g.n) return hipErrorInvalidValue;
  const int64_t work = std::max<int64_t>(kMaxLevels, (int64_t)a.seed_n * a.t.mask_words);
  // one thread at least per seed
  const int64_t grid = std::max<int64_t>((a.seed_n + kBlock - 1) / kBlock,
                                         std::min<int64_t>(1024, (work + kBlock - 1) / kBlock + 1));
  k_seed<<<(unsigned)grid, kBlock, 0, st>>>(a, limit, PathTotals::words(a.g));
  return hipGetLastError();
}

// Resume after an overflow: the level is extended again from a zero claim.
__global__ void k_resume_fix(ExtArgs a, int level) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.ls->count[level + 1] = 0;
    a.ls->overflow = 0;
    a.ls->overflow_level = 0;
  }
}

hipError_t launch_resume_fix(const ExtArgs& a, int level, hipStream_t st) {
  if (level < 1 || level + 1 >= kMaxLevels) return hipErrorInvalidValue;
  k_resume_fix<<<1, 64, 0, st>>>(a, level);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// shared per-parent step: choice mask over successor slots + terminal filter
// ---------------------------------------------------------------------------
// Choice mask over the successor slots [k0, k1) of the path's last vertex:
// slot k is set when successor w is not on the path, or is its first vertex
// (closes a cycle).  cb = graph-wide id of local id 0 of the component.
template <int W>
__device__ __forceinline__ uint64_t choices(const DGraph& g, uint32_t inf, const uint64_t (&m)[W],
                                            int k0, int k1, int cb) {
  const int v1l = node_v1l(inf);
  uint64_t vm = 0;
  for (int k = k0; k < k1; ++k) {
    const int wl = g.s[k] - cb;
    const bool ok = (wl == v1l) || !mask_has<W>(m, wl);
    vm |= ok ? (1ull << (k - k0)) : 0ull;
  }
  return vm;
}

// Backward-extendability test of a terminal path: prime iff every
// predecessor of its first vertex is on it.
template <int W>
__device__ __forceinline__ bool all_preds_on(const DGraph& g, int base, int v1l,
                                             const uint64_t (&m)[W]) {
  const int v1 = base + v1l;
  for (int k = g.pp[v1]; k < g.pp[v1 + 1]; ++k)
    if (!mask_has<W>(m, g.p[k] - base)) return false;
  return true;
}

// Visited set of slot j of a level (word-major, stride S slots).  Only the
// first Wu words are stored (ceil(largest component / 64)); the register
// copy is padded with zero words up to W.
template <int W>
__device__ __forceinline__ void load_mask(const uint64_t* src, int64_t S, int Wu, int64_t j,
                                          uint64_t (&m)[W]) {
#pragma unroll
  for (int q = 0; q < W; ++q) m[q] = q < Wu ? src[q * S + j] : 0ull;
}

// Visited set of child slot c: the parent's set plus local vertex w.
template <int W>
__device__ __forceinline__ void store_child_mask(uint64_t* dst, int64_t S, int Wu, int64_t c,
                                                 const uint64_t (&m)[W], int w) {
  const int q = w >> 6;
  const uint64_t bit = 1ull << (w & 63);
#pragma unroll
  for (int k = 0; k < W; ++k)
    if (k < Wu) dst[k * S + c] = m[k] | (k == q ? bit : 0ull);
}

// Stored levels (odd) alternate between the two buffers.
__device__ __forceinline__ int mask_buf(int L) { return ((L - 1) >> 1) & 1; }

// Visited set of the path in slot j of level L: an odd level's set is
// stored; an even level's is its parent's (slot par - prev of level L - 1,
// which starts at node prev) plus its own last vertex, local id vl.
template <int W>
__device__ __forceinline__ void path_mask_load(const ExtArgs& a, int L, int64_t prev, int64_t node,
                                               int64_t j, uint64_t (&m)[W]) {
  if (L & 1) {
    load_mask<W>(a.t.mask[mask_buf(L)], a.t.mask_cap, a.t.mask_words, j, m);
  } else {
    const int64_t jp = (int64_t)a.t.par[node] - prev;
    load_mask<W>(a.t.mask[mask_buf(L - 1)], a.t.mask_cap, a.t.mask_words, jp, m);
  }
}
template <int W>
__device__ __forceinline__ void path_mask_own(int L, int vl, uint64_t (&m)[W]) {
  if (L & 1) return;  // stored sets already hold the last vertex
  const int q = vl >> 6;
  const uint64_t bit = 1ull << (vl & 63);
#pragma unroll
  for (int k = 0; k < W; ++k) m[k] |= (k == q) ? bit : 0ull;
}

// ---------------------------------------------------------------------------
// one-pass extension of level L -> L+1 (device-sized, claim per tile)
// ---------------------------------------------------------------------------
// Launch `li` of a batch extends the level that the launch before it has left
// (batch_start for the first).  Its offset is derived from the previous level's
// final offset and size, so no kernel has to advance a level counter; a level
// whose nodes did not fit (claimed beyond the capacities by the launch before)
// raises the overflow flag and ends the batch.
//
// A narrow level (kNarrowExtend, kNarrowWords) is workgroup 0's alone, which then
// goes on to the levels after it until one is wide, empty or past the limit: a
// launch costs 5 to 8 us and the host's look at the sizes some 40, while the
// workgroup needs 2 to 3 us a level.  48 small functions, none seen
// just before, took 20.6 ms without it, 17.0 with the line at 1024 nodes and 16.7 from
// 2048 to 8192; a 212-vertex CFG 1.83, 1.79, 1.79 and from 8192 on 1.82 ms.  One
// CU is soon busy with wide sets: 4000 early exits (63 words) took 140 ms
// without a line on the words, 103 with 65536, 94.6 with 32768, 93.2 with 16384 and
// less; 1000 (16 words) 14.7, 14.7, 14.7, 13.2, and 14.8 without any narrow level.
struct LevelCursor {
  int L, limit;
  bool narrow;
  int64_t F, base, prev;
  int children;  // of a narrow level, so far (< 2^17)

  // Sets the cursor to the launch's first level; false: nothing to extend.
  __device__ __forceinline__ bool begin(const ExtArgs& a, int li) {
    LevelState* ls = a.ls;
    if (ls->overflow) return false;
    L = li == 0 ? ls->batch_start : ls->next[li];
    limit = ls->limit;
    F = L < limit ? ls->count[L] : 0;
    if (F == 0) {
      leave(ls, li);
      return false;
    }
    prev = ls->off[L - 1];
    base = prev + ls->count[L - 1];
    narrow = narrow_level(F, a.t.mask_words);
    return !narrow || blockIdx.x == 0;
  }
  __device__ __forceinline__ int64_t step() const { return narrow ? 1 : (int64_t)gridDim.x; }
  // Parents per thread of a tile.
  __device__ __forceinline__ int items(int nt, int most, int64_t target) const {
    const int64_t want = narrow ? 1 : target;
    int ir = 1;
    while (ir < most && (F + (int64_t)nt * ir - 1) / ((int64_t)nt * ir) > want) ir <<= 1;
    return ir;
  }
  __device__ __forceinline__ bool has_tile(int nt, int most, int64_t target) const {
    return (int64_t)blockIdx.x * nt * items(nt, most, target) < F;
  }
  // The level's nodes must be there: false (and the overflow raised) if the
  // children of the level before it did not fit.
  __device__ __forceinline__ bool open(const ExtArgs& a) {
    const bool fits = level_fits(L, base, F, a.t.rec_cap, a.t.mask_cap);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (fits) {
        a.ls->off[L] = base;
      } else {
        a.ls->overflow_level = L - 1;
        a.ls->overflow = 1;
      }
    }
    children = 0;
    return fits;
  }
  // The place of a tile's `total` children in the next level (one thread).
  __device__ __forceinline__ int64_t claim(LevelState* ls, int total) const {
    if (narrow) return children;
    if (!total) return 0;
    return (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(&ls->count[L + 1]),
                              (unsigned long long)total);
  }
  // total comes from LDS: said to be uniform, or it and all that follows from
  // it would take vector registers
  __device__ __forceinline__ void claimed(int total) {
    children += __builtin_amdgcn_readfirstlane(total);
  }
  // After a level: on to the next one, or leaves it to the next launch.
  __device__ __forceinline__ bool advance(const ExtArgs& a, int li) {
    LevelState* ls = a.ls;
    if (narrow && threadIdx.x == 0) ls->count[L + 1] = children;
    ++L;
    if (narrow) {
      prev = base;
      base += F;
      F = children;
    }
    if (!narrow || F == 0 || !narrow_level(F, a.t.mask_words) || L >= limit) {
      leave(ls, li);
      return false;
    }
    return true;
  }
  __device__ __forceinline__ void leave(LevelState* ls, int li) const {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ls->next[li + 1] = L;
      ls->reached = L;
    }
  }
};

// A tile is NT * ir consecutive parents (ir <= ITEMS, chosen per level so
// that large levels need few claims and small ones still spread over the
// grid); tile t goes to workgroup t mod grid.  Thread tid owns parents
// i * NT + tid (i < ir): their records and visited sets are loaded together
// (coalesced), the visited sets stay in registers, and the thread writes its
// own parents' children.  Children are laid out item-major and, inside an
// item, in thread order, so a wave's stores land on neighbouring slots.  A
// level that fits one tile stores its size instead of claiming.
//
// GL: the CSR (row pointers, successors, predecessors, local ids) is copied
// into LDS by every workgroup that has a tile, so the per-parent chain of
// graph lookups (row range -> successor ids -> predecessor ids) reads LDS
// instead of L2.
//
// Up to four words two workgroups of 1024 fit a CU (64 registers, no scratch);
// eight words spill at that, and 300 early exits took 1.92 ms with it, 1.55 with
// one workgroup, 2.6 million nodes over 347 chains 2.96 and 2.61.
template <int W, int ITEMS, int NT, bool GL>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 1024 && ITEMS == 1 && W <= 4 ? 8 : 1))) void k_extend_tp(ExtArgs a, int li) {
  constexpr int NW = NT / 64;
  __shared__ int32_t s_tot[ITEMS][NW];
  __shared__ int64_t s_prefix;
  extern __shared__ int32_t s_graph[];

  const int tid = (int)threadIdx.x;
  const int lane = lane_id(), wave = tid >> 6;
  LevelCursor cur;
  if (!cur.begin(a, li)) return;
  DGraph g = a.g;
  if constexpr (GL) {
    if (!cur.has_tile(NT, ITEMS, a.tiles_target)) return;
    for (int i = tid; i < a.g.n_stage; i += NT) s_graph[i] = a.g.sp[i];
    __syncthreads();
    g.sp = s_graph;
    g.s = s_graph + (a.g.s - a.g.sp);
    g.pp = s_graph + (a.g.pp - a.g.sp);
    g.p = s_graph + (a.g.p - a.g.sp);
    g.loc = s_graph + (a.g.loc - a.g.sp);
    g.len = s_graph + (a.g.len - a.g.sp);
  }
  do {
    if (!cur.open(a)) return;
    const int L = cur.L;
    const int64_t F = cur.F, base = cur.base, prev = cur.prev;
    const int64_t nbase = base + F;
    // children's sets are stored when they land on an odd level
    uint64_t* mnxt = (L & 1) ? nullptr : a.t.mask[mask_buf(L + 1)];
    const int ir = cur.items(NT, ITEMS, a.tiles_target);
    const int64_t TR = (int64_t)NT * ir;
    const int64_t ntiles = (F + TR - 1) / TR;
    for (int64_t t = blockIdx.x; t < ntiles; t += cur.step()) {
      const int64_t tb = t * TR;
      // records and visited sets of the thread's parents (independent loads;
      // rows outside the level read parent 0's set and are ignored)
      uint32_t inf[ITEMS];
      int tl[ITEMS];
      uint64_t m[ITEMS][W];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = tb + i * NT + tid;
        const bool ok = i < ir && j < F;
        inf[i] = ok ? a.t.info[base + j] : F_CYC;
        tl[i] = ok ? a.t.tl[base + j] : 0;
        path_mask_load<W>(a, L, prev, base + (ok ? j : 0), ok ? j : 0, m[i]);
      }
      // choice masks and the terminal filter
      uint64_t vm[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        vm[i] = 0;
        if (!(inf[i] & F_CYC)) {
          const int v = node_v(inf[i]);
          const int cb = v - g.loc[v];
          path_mask_own<W>(L, v - cb, m[i]);
          vm[i] = choices<W>(g, inf[i], m[i], g.sp[v], g.sp[v + 1], cb);
          if (vm[i] == 0) {
            const bool pp = all_preds_on<W>(g, cb, node_v1l(inf[i]), m[i]);
            inf[i] |= F_TERM | (pp ? F_PP : 0u);  // recorded through nch_code below
          }
        }
      }
      // child offsets: item-major, thread order inside an item
      int excl[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int c = __builtin_popcountll(vm[i]);
        const int inc = wave_incl_scan(c);
        excl[i] = inc - c;
        if (lane == 63) s_tot[i][wave] = inc;
      }
      __syncthreads();
      int total = 0;
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const int x = i < ir ? s_tot[i][w] : 0;
          before += w < wave ? x : 0;
          all += x;
        }
        excl[i] += total + before;
        total += all;
      }
      if (tid == 0) {
        s_prefix = cur.claim(a.ls, total);
      }
      __syncthreads();
      const int64_t prefix = s_prefix;
      cur.claimed(total);
      // expansion: each thread writes its parents' children in slot order
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = tb + i * NT + tid;
        if (i < ir && j < F) {
          int64_t cl = prefix + excl[i];
          a.t.cstart[base + j] = (int32_t)(nbase + cl);
          a.t.nch[base + j] = nch_code(inf[i], __builtin_popcountll(vm[i]));
          const int v1l = node_v1l(inf[i]);
          uint64_t rest = vm[i];
          const int pv = node_v(inf[i]);
          const int k0 = rest ? g.sp[pv] : 0;
          const int cb = rest ? pv - g.loc[pv] : 0;
          while (rest) {
            const int slot = __builtin_ctzll(rest);
            rest &= rest - 1;
            const int w = g.s[k0 + slot];
            const int wl = w - cb;
            const int64_t cg = nbase + cl;
            if (cg < a.t.rec_cap) {
              a.t.par[cg] = (int32_t)(base + j);
              a.t.info[cg] = make_info(w, v1l, wl == v1l ? F_CYC : 0u);
              a.t.tl[cg] = (uint16_t)(tl[i] + (wl == v1l ? 0 : g.len[w]));
            }
            if (mnxt && wl != v1l && cl < a.t.mask_cap)
              store_child_mask<W>(mnxt, a.t.mask_cap, a.t.mask_words, cl, m[i], wl);
            ++cl;
          }
        }
      }
      __syncthreads();
    }
  } while (cur.advance(a, li));
}

// Load-balanced form of the same step: the tile's parents are staged in LDS
// (choice masks, records, successor-row starts, visited sets when they fit)
// and thread k writes the k-th child of the tile, found by binary search
// over the parents' child offsets.
template <int W, int ITEMS>
__global__ __launch_bounds__(kBlock) void k_extend_lb(ExtArgs a, int li) {
  constexpr int TILE = kBlock * ITEMS;
  constexpr bool kLdsMask = W * ITEMS <= 16;  // visited sets of the tile in LDS (<= 32 KiB)
  __shared__ int64_t s_prefix;
  __shared__ int32_t s_off[TILE];
  __shared__ uint64_t s_vm[TILE];
  __shared__ uint32_t s_inf[TILE];
  __shared__ int32_t s_kk[TILE];
  __shared__ uint64_t s_mask[kLdsMask ? TILE * W : 1];
  __shared__ int32_t s_w[kBlock / 64];

  const int tid = (int)threadIdx.x;
  LevelCursor cur;
  if (!cur.begin(a, li)) return;
  do {
    if (!cur.open(a)) return;
    const int L = cur.L;
    const int64_t F = cur.F, base = cur.base, prev = cur.prev;
    const int64_t nbase = base + F;
    uint64_t* mnxt = (L & 1) ? nullptr : a.t.mask[mask_buf(L + 1)];
    const int ir = cur.items(kBlock, ITEMS, a.tiles_target);
    const int TR = kBlock * ir;
    const int64_t ntiles = (F + TR - 1) / TR;
    for (int64_t t = blockIdx.x; t < ntiles; t += cur.step()) {
      const int64_t tb = t * TR;
      uint32_t inf[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = tb + i * kBlock + tid;
        inf[i] = (i < ir && j < F) ? a.t.info[base + j] : F_CYC;
      }
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        if (i < ir) {
          const int p = i * kBlock + tid;
          const int64_t j = tb + p;
          uint32_t in = inf[i];
          uint64_t m[W];
#pragma unroll
          for (int q = 0; q < W; ++q) m[q] = 0;
          uint64_t vm = 0;
          int k0 = 0;
          if (!(in & F_CYC)) {
            const int v = node_v(in);
            const int cb = v - a.g.loc[v];
            k0 = a.g.sp[v];
            path_mask_load<W>(a, L, prev, base + j, j, m);
            path_mask_own<W>(L, v - cb, m);
            vm = choices<W>(a.g, in, m, k0, a.g.sp[v + 1], cb);
            if (vm == 0) {
              const bool pp = all_preds_on<W>(a.g, cb, node_v1l(in), m);
              in |= F_TERM | (pp ? F_PP : 0u);  // recorded through nch_code
            }
          }
          s_off[p] = __builtin_popcountll(vm);
          s_vm[p] = vm;
          s_inf[p] = in;
          s_kk[p] = k0;
          if constexpr (kLdsMask) {
#pragma unroll
            for (int q = 0; q < W; ++q) s_mask[p * W + q] = m[q];
          }
        }
      }
      __syncthreads();
      int c[ITEMS];
      int sum = 0;
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        c[i] = i < ir ? s_off[tid * ir + i] : 0;
        sum += c[i];
      }
      int32_t total32;
      int32_t run = block_excl_scan<kBlock, int32_t>(sum, total32, s_w);
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        if (i < ir) s_off[tid * ir + i] = run;
        run += c[i];
      }
      if (tid == 0) {
        s_prefix = cur.claim(a.ls, total32);
      }
      __syncthreads();
      const int64_t prefix = s_prefix;
      cur.claimed(total32);
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int p = i * kBlock + tid;
        if (i < ir && tb + p < F) {
          a.t.cstart[base + tb + p] = (int32_t)(nbase + prefix + s_off[p]);
          a.t.nch[base + tb + p] = nch_code(s_inf[p], __builtin_popcountll(s_vm[p]));
        }
      }
      for (int k = tid; k < total32; k += kBlock) {
        int lo = 0, hi = TR - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (s_off[mid] <= k) lo = mid; else hi = mid - 1;
        }
        const int o = lo;
        const int slot = select_bit(s_vm[o], k - s_off[o]);
        const uint32_t pinf = s_inf[o];
        const int v1l = node_v1l(pinf);
        const int pv = node_v(pinf);
        const int w = a.g.s[s_kk[o] + slot];
        const int wl = w - (pv - a.g.loc[pv]);
        const int64_t cl = prefix + k;
        const int64_t cg = nbase + cl;
        if (cg < a.t.rec_cap) {
          a.t.par[cg] = (int32_t)(base + tb + o);
          a.t.info[cg] = make_info(w, v1l, wl == v1l ? F_CYC : 0u);
          a.t.tl[cg] = (uint16_t)(a.t.tl[base + tb + o] + (wl == v1l ? 0 : a.g.len[w]));
        }
        if (mnxt && wl != v1l && cl < a.t.mask_cap) {
          uint64_t pm[W];
          if constexpr (kLdsMask) {
#pragma unroll
            for (int q = 0; q < W; ++q) pm[q] = s_mask[o * W + q];
          } else {
            path_mask_load<W>(a, L, prev, base + tb + o, tb + o, pm);
            path_mask_own<W>(L, a.g.loc[pv], pm);
          }
          store_child_mask<W>(mnxt, a.t.mask_cap, a.t.mask_words, cl, pm, wl);
        }
      }
      __syncthreads();
    }
  } while (cur.advance(a, li));
}

// Launch with optional start / stop events recorded by the dispatch itself
// (the kernel's own execution interval, without queueing around it).
template <class K>
static hipError_t launch_timed(K kernel, int grid, int threads, hipEvent_t e0, hipEvent_t e1,
                               const ExtArgs& a, int li, hipStream_t st, size_t lds = 0) {
  if (e0 && e1)
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, st, e0, e1, 0, a, li);
  else
    kernel<<<grid, threads, lds, st>>>(a, li);
  return hipGetLastError();
}

// variant 0: load-balanced (256 threads); 1: thread-per-parent, 256
// threads; 2: thread-per-parent, 1024 threads.  Register-resident visited
// sets are capped at 32 words per thread; wider sets always take variant 0.
template <int W, int ITEMS>
static hipError_t launch_extend_wi(int variant, const ExtArgs& a, int grid, int li, hipStream_t st,
                                   hipEvent_t e0, hipEvent_t e1) {
  if constexpr (ITEMS * W <= 32) {
    const size_t gb = sizeof(int32_t) * (size_t)a.g.n_stage;
    if (gb <= (size_t)kGraphLdsBytes) {
      if (variant == 1)
        return launch_timed(k_extend_tp<W, ITEMS, 256, true>, grid, 256, e0, e1, a, li, st, gb);
      if (variant == 2)
        return launch_timed(k_extend_tp<W, ITEMS, 1024, true>, grid, 1024, e0, e1, a, li, st, gb);
    }
    if (variant == 1) return launch_timed(k_extend_tp<W, ITEMS, 256, false>, grid, 256, e0, e1, a, li, st);
    if (variant == 2) return launch_timed(k_extend_tp<W, ITEMS, 1024, false>, grid, 1024, e0, e1, a, li, st);
  }
  return launch_timed(k_extend_lb<W, ITEMS>, grid, kBlock, e0, e1, a, li, st);
}

template <int W>
static hipError_t launch_extend_w(int items, int variant, const ExtArgs& a, int grid, int li,
                                  hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  int it = items;
  if (variant != 0)
    while (it > 1 && it * W > 32) it >>= 1;
  switch (it) {
    case 1: return launch_extend_wi<W, 1>(variant, a, grid, li, st, e0, e1);
    case 2: return launch_extend_wi<W, 2>(variant, a, grid, li, st, e0, e1);
    case 4: return launch_extend_wi<W, 4>(variant, a, grid, li, st, e0, e1);
    case 8: return launch_extend_wi<W, 8>(variant, a, grid, li, st, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_extend(int W, int items, int variant, const ExtArgs& a, int grid, int li,
                         hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (variant < 0 || variant > 2) return hipErrorInvalidValue;
  switch (W) {
    case 1: return launch_extend_w<1>(items, variant, a, grid, li, st, e0, e1);
    case 2: return launch_extend_w<2>(items, variant, a, grid, li, st, e0, e1);
    case 4: return launch_extend_w<4>(items, variant, a, grid, li, st, e0, e1);
    case 8: return launch_extend_w<8>(items, variant, a, grid, li, st, e0, e1);
    case 16: return launch_extend_w<16>(items, variant, a, grid, li, st, e0, e1);
    case 32: return launch_extend_w<32>(items, variant, a, grid, li, st, e0, e1);
    case 64: return launch_extend_w<64>(items, variant, a, grid, li, st, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------
// two-pass (plain) form: count, host-visible scan, fill
// ---------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(kBlock) void k_count(ExtArgs a, int L, int64_t prev, int64_t base,
                                                  int64_t F) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= F) return;
  uint32_t inf = a.t.info[base + j];
  int cnt = 0;
  if (!(inf & F_CYC)) {
    uint64_t m[W];
    path_mask_load<W>(a, L, prev, base + j, j, m);
    const int v = node_v(inf);
    const int cb = v - a.g.loc[v];
    path_mask_own<W>(L, v - cb, m);
    const uint64_t vm = choices<W>(a.g, inf, m, a.g.sp[v], a.g.sp[v + 1], cb);
    cnt = __builtin_popcountll(vm);
    if (cnt == 0) {
      const bool pp = all_preds_on<W>(a.g, cb, node_v1l(inf), m);
      inf |= F_TERM | (pp ? F_PP : 0u);  // recorded through nch_code
    }
  }
  a.t.cstart[base + j] = cnt;
  a.t.nch[base + j] = nch_code(inf, cnt);
}

template <int W>
__global__ __launch_bounds__(kBlock) void k_fill(ExtArgs a, int L, int64_t prev, int64_t base,
                                                 int64_t F) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= F) return;
  const uint32_t inf = a.t.info[base + j];
  if (inf & F_CYC) return;
  uint64_t m[W];
  path_mask_load<W>(a, L, prev, base + j, j, m);
  const int v = node_v(inf);
  const int k0 = a.g.sp[v];
  const int cb = v - a.g.loc[v];
  path_mask_own<W>(L, v - cb, m);
  uint64_t vm = choices<W>(a.g, inf, m, k0, a.g.sp[v + 1], cb);
  const int v1l = node_v1l(inf);
  const int64_t nbase = base + F;
  int64_t c = a.t.cstart[base + j];
  uint64_t* mnxt = (L & 1) ? nullptr : a.t.mask[mask_buf(L + 1)];
  while (vm) {
    const int slot = __builtin_ctzll(vm);
    vm &= vm - 1;
    const int w = a.g.s[k0 + slot];
    const int wl = w - cb;
    a.t.par[c] = (int32_t)(base + j);
    a.t.info[c] = make_info(w, v1l, wl == v1l ? F_CYC : 0u);
    a.t.tl[c] = (uint16_t)(a.t.tl[base + j] + (wl == v1l ? 0 : a.g.len[w]));
    if (mnxt && wl != v1l) store_child_mask<W>(mnxt, a.t.mask_cap, a.t.mask_words, c - nbase, m, wl);
    ++c;
  }
}

#define TPG_W_SWITCH(W, KERNEL, GRID, ...)                                        \
  switch (W) {                                                                      \
    case 1: KERNEL<1><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;                 \
    case 2: KERNEL<2><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;                 \
    case 4: KERNEL<4><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;                 \
    case 8: KERNEL<8><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;                 \
    case 16: KERNEL<16><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;               \
    case 32: KERNEL<32><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;               \
    case 64: KERNEL<64><<<GRID, kBlock, 0, st>>>(__VA_ARGS__); break;               \
    default: return hipErrorInvalidValue;                                           \
  }

hipError_t launch_count(int W, const ExtArgs& a, int L, int64_t prev, int64_t base, int64_t F,
                        hipStream_t st) {
  if (F == 0) return hipSuccess;
  const int64_t grid = (F + kBlock - 1) / kBlock;
  TPG_W_SWITCH(W, k_count, (unsigned)grid, a, L, prev, base, F);
  return hipGetLastError();
}

hipError_t launch_fill(int W, const ExtArgs& a, int L, int64_t prev, int64_t base, int64_t F,
                       hipStream_t st) {
  if (F == 0) return hipSuccess;
  const int64_t grid = (F + kBlock - 1) / kBlock;
  TPG_W_SWITCH(W, k_fill, (unsigned)grid, a, L, prev, base, F);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// canonical order: subtree counts bottom-up, ranks top-down
// ---------------------------------------------------------------------------
// sub_cnt[g] = prime-path leaves in g's subtree (k_up), then rewritten top-down
// into the output position of the subtree's first prime path, or kNoRank when
// the subtree holds none (k_down then skips it after one 4-byte read).
constexpr uint32_t kNoRank = 0xFFFFFFFFu;
__device__ __forceinline__ bool nch_internal(uint8_t k) { return k >= 1 && k < kNchPP; }

// Simple paths by length, from the nodes.  A node <x1 .. xk> of chains (k >=
// 2, not a cycle) of T vertices stands for the paths that start at any of
// x1's m1 vertices and end at any of xk's mk: lengths T - d, as many as there
// are (a, b) with a < m1, b < mk, a + b = d.  A cycle of S vertices stands
// for the paths that come back into x1, up to the vertex they started at:
// m1 - d of length S + 1 - d for d < m1 (the m1 with d = 0 are the closed
// cycles).  Both are sums over the bins from the top: with m1 = 1 two entries
// of the first histogram, summed once, else three or four of the second,
// summed twice.  Bins are counted in LDS (kept `copies` times, by lane, as a
// wave's nodes share few lengths) and added to a.tot once per workgroup.
// Reads 6 bytes a node; the lookups behind a node are a chain of small loads,
// so a thread takes kLenItems nodes at a time (1.85e8 nodes: 1.02 ms one at a
// time, 0.58 four).
constexpr int kLenItems = 4;
__global__ __launch_bounds__(kBlock) void k_path_lengths(ExtArgs a, int64_t first, int64_t n_nodes,
                                                         int bins, int copies, int lds_roots) {
  extern __shared__ unsigned long long s_hist[];
  unsigned long long* h2 = s_hist;                                   // [bins * copies]
  int32_t* h1 = reinterpret_cast<int32_t*>(h2 + bins * copies);      // [bins * copies]
  uint32_t* s_cyc = reinterpret_cast<uint32_t*>(h1 + bins * copies); // [lds_roots]
  uint32_t* g_cyc = PathTotals::root_cycles(a.g, a.tot);
  const int tid = (int)threadIdx.x;
  for (int i = tid; i < bins * copies; i += kBlock) {
    h2[i] = 0;
    h1[i] = 0;
  }
  for (int i = tid; i < lds_roots; i += kBlock) s_cyc[i] = 0;
  __syncthreads();
  const int cp = tid & (copies - 1);
  auto add1 = [&](int bin, int x) { atomicAdd(&h1[bin * copies + cp], x); };
  auto add2 = [&](int bin, int x) {
    atomicAdd(&h2[bin * copies + cp], (unsigned long long)(long long)x);
  };
  // kLenItems nodes of a thread in flight together: the lookups behind a node
  // are a chain of small loads
  const int64_t step = (int64_t)gridDim.x * kBlock * kLenItems;
  for (int64_t x0 = first + (int64_t)blockIdx.x * kBlock * kLenItems + tid; x0 < n_nodes;
       x0 += step) {
    uint32_t inf[kLenItems];
    int T[kLenItems], v1[kLenItems], m1[kLenItems], mk[kLenItems];
#pragma unroll
    for (int j = 0; j < kLenItems; ++j) {
      const int64_t x = x0 + j * kBlock;
      const bool in = x < n_nodes;
      inf[j] = in ? a.t.info[x] : 0u;
      T[j] = in ? (int)a.t.tl[x] : -1;
    }
#pragma unroll
    for (int j = 0; j < kLenItems; ++j) {
      const int v = node_v(inf[j]);
      v1[j] = v - a.g.loc[v] + node_v1l(inf[j]);
      mk[j] = a.g.len[v];
    }
#pragma unroll
    for (int j = 0; j < kLenItems; ++j) m1[j] = T[j] < 0 ? 1 : a.g.len[v1[j]];
#pragma unroll
    for (int j = 0; j < kLenItems; ++j) {
      if (T[j] < 0) continue;
      if (inf[j] & F_CYC) {
        atomicAdd(lds_roots ? &s_cyc[v1[j]] : &g_cyc[v1[j]], 1u);
        if (m1[j] == 1) {
          add1(T[j] + 1, 1);
          add1(T[j], -1);
        } else {
          add2(T[j] + 1, m1[j]);
          add2(T[j], -(m1[j] + 1));
          add2(T[j] - m1[j], 1);
        }
      } else if (m1[j] == 1) {
        add1(T[j], 1);
        add1(T[j] - mk[j], -1);
      } else {
        add2(T[j], 1);
        add2(T[j] - m1[j], -1);
        add2(T[j] - mk[j], -1);
        add2(T[j] - m1[j] - mk[j], 1);
      }
    }
  }
  __syncthreads();
  unsigned long long* out = reinterpret_cast<unsigned long long*>(a.tot) + PathTotals::kHist;
  for (int i = tid; i < bins; i += kBlock) {
    long long c1 = 0;
    unsigned long long c2 = 0;
    for (int c = 0; c < copies; ++c) {
      c1 += h1[i * copies + c];
      c2 += h2[i * copies + c];
    }
    if (c1) atomicAdd(out + i, (unsigned long long)c1);
    if (c2) atomicAdd(out + bins + i, c2);
  }
  for (int i = tid; i < lds_roots; i += kBlock)
    if (s_cyc[i]) atomicAdd(&g_cyc[i], s_cyc[i]);
}

hipError_t launch_path_lengths(const ExtArgs& a, int64_t first, int64_t n_nodes, hipStream_t st) {
  if (n_nodes <= first) return hipSuccess;
  const int bins = (int)PathTotals::bins(a.g);
  const int copies = bins <= 512 ? 4 : 1;
  // every root's cycles counted in LDS when they fit 4 KiB (a large union's
  // roots share few addresses anyway)
  const int lds_roots = a.g.n <= 1024 ? a.g.n : 0;
  const size_t lds = (size_t)bins * copies * 12 + sizeof(uint32_t) * (size_t)lds_roots;
  if (lds > 65536) return hipErrorInvalidValue;
  const int64_t grid = std::min<int64_t>(1024, (n_nodes - first + 8 * kBlock - 1) / (8 * kBlock));
  k_path_lengths<<<(unsigned)grid, kBlock, lds, st>>>(a, first, n_nodes, bins, copies, lds_roots);
  return hipGetLastError();
}

// What a node counts for itself: TP the test-path marks, else the PP leaves.
template <bool TP>
__device__ __forceinline__ uint32_t own_count(uint8_t k, const int32_t* rep, int64_t x) {
  if constexpr (TP) return rep[x] != 0 ? 1u : 0u;
  return k >= kNchPP ? 1u : 0u;
}

// The count of node x's subtree from its children's.
template <bool TP>
__device__ __forceinline__ uint32_t up_node(const ExtArgs& a, const int32_t* rep, int64_t x,
                                            const uint32_t* sub_cnt) {
  const uint8_t k = a.t.nch[x];
  uint32_t c = own_count<TP>(k, rep, x);
  if (nch_internal(k)) {
    const int64_t c0 = a.t.cstart[x], c1 = c0 + k;
    for (int64_t y = c0; y < c1; ++y) c += sub_cnt[y];
  }
  return c;
}

template <bool TP>
__global__ __launch_bounds__(kBlock) void k_up(ExtArgs a, int64_t base, int64_t F,
                                               const int32_t* rep, uint32_t* sub_cnt) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= F) return;
  sub_cnt[base + j] = up_node<TP>(a, rep, base + j, sub_cnt);
}

// Narrow levels, bottom to top, in one launch of one workgroup: a level waits
// for the one below at the barrier, two or three load latencies, instead of
// for a launch (5 to 8 us however little it does).  A 20-vertex function's
// call went from 403 to 367 us, the host's round trips being most of the rest.
template <bool TP>
__global__ __launch_bounds__(1024) void k_up_span(ExtArgs a, LevelSpan s, const int32_t* rep,
                                                  uint32_t* sub_cnt) {
  for (int l = s.n - 1; l >= 0; --l) {
    const uint32_t end = s.off[l + 1];
    for (uint32_t x = s.off[l] + threadIdx.x; x < end; x += 1024)
      sub_cnt[x] = up_node<TP>(a, rep, x, sub_cnt);
    __syncthreads();
  }
}

hipError_t launch_up_span(const ExtArgs& a, const LevelSpan& s, const int32_t* rep,
                          uint32_t* sub_cnt, hipStream_t st) {
  if (s.n < 1 || s.n > kSpanLevels) return hipErrorInvalidValue;
  if (rep)
    k_up_span<true><<<1, 1024, 0, st>>>(a, s, rep, sub_cnt);
  else
    k_up_span<false><<<1, 1024, 0, st>>>(a, s, nullptr, sub_cnt);
  return hipGetLastError();
}

hipError_t launch_up(const ExtArgs& a, int64_t base, int64_t F, uint32_t* sub_cnt,
                     hipStream_t st) {
  if (F == 0) return hipSuccess;
  k_up<false><<<(unsigned)((F + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, base, F, nullptr,
                                                                        sub_cnt);
  return hipGetLastError();
}

hipError_t launch_tp_up(const ExtArgs& a, int64_t base, int64_t F, const int32_t* rep,
                        uint32_t* cnt, hipStream_t st) {
  if (F == 0) return hipSuccess;
  k_up<true><<<(unsigned)((F + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, base, F, rep, cnt);
  return hipGetLastError();
}

// Output positions by first vertex: a scan over the range's vertices in id
// order of the prime paths that start there, which are all of its root's for
// the head of a chain and its root's cycles for another vertex of one.  The
// head's position is where its root's leaves go.  One workgroup, kRootItems
// vertices per thread and step.
constexpr int kRootItems = 8;
__global__ __launch_bounds__(1024) void k_roots(ExtArgs a, DChains ch, int32_t range_lo,
                                                int32_t range_n, uint32_t* sub_cnt, int64_t* rb) {
  __shared__ int64_t s_w[16];
  const uint32_t* cyc = PathTotals::root_cycles(a.g, a.tot);
  int64_t carry = 0, cycles = 0;
  for (int32_t b = 0; b < range_n; b += 1024 * kRootItems) {
    const int32_t i0 = b + (int32_t)threadIdx.x * kRootItems;
    int32_t root[kRootItems];  // the root whose head this vertex is (-1: not a head)
    int64_t c[kRootItems];
    int64_t sum = 0;
#pragma unroll
    for (int j = 0; j < kRootItems; ++j) {
      root[j] = -1;
      c[j] = 0;
      if (i0 + j < range_n) {
        const int v = range_lo + i0 + j;
        const int x = ch.of[v];
        const uint32_t cx = cyc[x];
        cycles += cx;
        c[j] = cx;
        if (ch.pos[v] == 0) {
          root[j] = x - a.seed_lo;
          c[j] = sub_cnt[root[j]];
        }
        sum += c[j];
      }
    }
    int64_t total;
    int64_t at = carry + block_excl_scan<1024, int64_t>(sum, total, s_w);
#pragma unroll
    for (int j = 0; j < kRootItems; ++j) {
      if (i0 + j < range_n) rb[i0 + j] = at;
      if (root[j] >= 0) sub_cnt[root[j]] = c[j] ? (uint32_t)at : kNoRank;
      at += c[j];
    }
    carry += total;
  }
  int64_t all;
  (void)block_excl_scan<1024, int64_t>(cycles, all, s_w);
  if (threadIdx.x == 0) {
    rb[range_n] = carry;
    a.tot[PathTotals::kPP] = (uint64_t)carry;
    a.tot[PathTotals::kCycles] = (uint64_t)all;
  }
}

// The same for a large union, around a scan over the chip: its numbers, then
// the roots' positions.  100 k vertices of 4096 CFGs took one workgroup 170 to
// 210 us, about 35 this way; up to kOneRoots its two steps are as fast.
constexpr int32_t kOneRoots = 2 * 1024 * kRootItems;
__global__ __launch_bounds__(kBlock) void k_root_counts(ExtArgs a, DChains ch, int32_t range_lo,
                                                        int32_t range_n, const uint32_t* sub_cnt,
                                                        int32_t* cnt) {
  const int32_t i = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
  uint32_t cx = 0;
  if (i < range_n) {
    const int v = range_lo + i, x = ch.of[v];
    cx = PathTotals::root_cycles(a.g, a.tot)[x];
    cnt[i] = (int32_t)(ch.pos[v] == 0 ? sub_cnt[x - a.seed_lo] : cx);
  }
  __shared__ int64_t s_w[kBlock / 64];
  int64_t cycles;
  (void)block_excl_scan<kBlock, int64_t>(cx, cycles, s_w);
  if (threadIdx.x == 0 && cycles)
    atomicAdd(reinterpret_cast<unsigned long long*>(a.tot) + PathTotals::kCycles,
              (unsigned long long)cycles);
}

__global__ __launch_bounds__(kBlock) void k_root_places(ExtArgs a, DChains ch, int32_t range_lo,
                                                        int32_t range_n, const int32_t* cnt,
                                                        const int64_t* rb, uint32_t* sub_cnt) {
  const int32_t i = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
  if (i >= range_n) return;
  const int v = range_lo + i;
  if (ch.pos[v] == 0) sub_cnt[ch.of[v] - a.seed_lo] = cnt[i] ? (uint32_t)rb[i] : kNoRank;
}

hipError_t launch_roots(const ExtArgs& a, const DChains& ch, int32_t range_lo, int32_t range_n,
                        uint32_t* sub_cnt, int64_t* rb, int32_t* cnt, uint64_t* scan_status,
                        hipStream_t st) {
  if (range_n > kOneRoots) {
    const unsigned grid = (unsigned)((range_n + kBlock - 1) / kBlock);
    k_root_counts<<<grid, kBlock, 0, st>>>(a, ch, range_lo, range_n, sub_cnt, cnt);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
      e = scan_i32_to_i64(cnt, rb, range_n, 0,
                          reinterpret_cast<int64_t*>(a.tot) + PathTotals::kPP, scan_status,
                          nullptr, st);
    if (e != hipSuccess) return e;
    k_root_places<<<grid, kBlock, 0, st>>>(a, ch, range_lo, range_n, cnt, rb, sub_cnt);
    return hipGetLastError();
  }
  k_roots<<<1, 1024, 0, st>>>(a, ch, range_lo, range_n, sub_cnt, rb);
  return hipGetLastError();
}

// A prime-path leaf's record under its output position: a cycle's path holds
// its first vertex twice.
__device__ __forceinline__ void put_leaf(const ExtArgs& a, int64_t x, uint8_t k, uint32_t r,
                                         uint64_t* leaf, int32_t* pp_len) {
  const bool cyc = k == kNchCycle;
  leaf[r] = (uint64_t)x | (cyc ? kLeafCycle : 0ull);
  pp_len[r] = (int32_t)a.t.tl[x] + (cyc ? 1 : 0);
}

// The node of the child's path without its BFS-tree part (see TpTree), from
// that of its parent x (k children), cx, where child y is x's slot-th.  The
// dropped chains only took choices away, so the parent's node has at least
// x's children, in the same order.
__device__ __forceinline__ int32_t canon_child(const ExtArgs& a, const TpTree& t, int64_t x,
                                               uint8_t k, int32_t cx, int64_t y, int slot) {
  if (cx == (int32_t)x) return (int32_t)y;
  if (cx < 0) {
    const int vx = node_v(a.t.info[x]), vy = node_v(a.t.info[y]);
    if (t.tpar[vy] == vx) return -1;
    // the first arc off the BFS tree: the child of vx's root (root k is chain
    // k), whose children are all of vx's successors
    int s = slot;
    const int s0 = a.g.sp[vx], s1 = a.g.sp[vx + 1];
    while (s0 + s + 1 < s1 && a.g.s[s0 + s] != vy) ++s;
    return a.t.cstart[vx] + s;
  }
  const int32_t c0 = a.t.cstart[cx];
  const int kc = a.t.nch[cx];
  if (kc == k) return c0 + slot;
  const int vy = node_v(a.t.info[y]);
  int s = slot;
  while (s + 1 < kc && node_v(a.t.info[c0 + s]) != vy) ++s;
  return c0 + s;
}

// x (position r, nch code k, canon cx) hands positions to its children in slot
// order; with D > 0 each internal child with prime paths below then does the
// same for its own children.
template <int D, bool TP>
__device__ __forceinline__ void down_node(const ExtArgs& a, const TpTree& t, int64_t x, uint8_t k,
                                          int32_t cx, uint32_t r, uint32_t* sub_cnt,
                                          uint64_t* leaf, int32_t* pp_len) {
  if (k == 0 || k >= kNchPP) return;
  const int64_t c0 = a.t.cstart[x], c1 = c0 + k;
  for (int64_t y = c0; y < c1; ++y) {
    const uint32_t cc = sub_cnt[y];
    const uint8_t ky = a.t.nch[y];
    if (D == 0) sub_cnt[y] = cc ? r : kNoRank;
    if (cc) {
      int32_t cy = -1;
      if constexpr (TP) cy = canon_child(a, t, x, k, cx, y, (int)(y - c0));
      if (ky >= kNchPP) {
        put_leaf(a, y, ky, r, leaf, pp_len);
        if constexpr (TP) t.leaf_canon[r] = cy;
      } else if constexpr (D > 0) {
        down_node<D - 1, TP>(a, t, y, ky, cy, r, sub_cnt, leaf, pp_len);
      } else {
        if constexpr (TP) t.canon[y] = cy;
      }
    }
    r += cc;
  }
}

// Node x of level L, as a parent.  A level-1 node can be a leaf itself.
template <int D, bool TP>
__device__ __forceinline__ void down_parent(const ExtArgs& a, const TpTree& t, int L, int64_t x,
                                            uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len) {
  const uint32_t r = sub_cnt[x];
  if (r == kNoRank) return;
  const uint8_t k = a.t.nch[x];
  int32_t cx = -1;
  if (TP && L > 1 && nch_internal(k)) cx = t.canon[x];
  if (L == 1 && k >= kNchPP) {
    put_leaf(a, x, k, r, leaf, pp_len);
    if constexpr (TP) t.leaf_canon[r] = -1;
  }
  down_node<D, TP>(a, t, x, k, cx, r, sub_cnt, leaf, pp_len);
}

// Parents of levels L .. L + D in one launch (thread per node of L).  The
// nodes' canons pass from launch to launch in t.canon, one level in D + 1.
template <int D, bool TP>
__global__ __launch_bounds__(kBlock) void k_down_run(ExtArgs a, TpTree t, int L, int64_t base,
                                                     int64_t F, uint32_t* sub_cnt, uint64_t* leaf,
                                                     int32_t* pp_len) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= F) return;
  down_parent<D, TP>(a, t, L, base + j, sub_cnt, leaf, pp_len);
}

// Narrow levels, top to bottom (see k_up_span).
template <bool TP>
__global__ __launch_bounds__(1024) void k_down_span(ExtArgs a, TpTree t, int L, LevelSpan s,
                                                    uint32_t* sub_cnt, uint64_t* leaf,
                                                    int32_t* pp_len) {
  for (int l = 0; l < s.n; ++l) {
    const uint32_t end = s.off[l + 1];
    for (uint32_t x = s.off[l] + threadIdx.x; x < end; x += 1024)
      down_parent<0, TP>(a, t, L + l, x, sub_cnt, leaf, pp_len);
    __syncthreads();
  }
}

hipError_t launch_down_span(const ExtArgs& a, const TpTree& t, int L, const LevelSpan& s,
                            uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st) {
  if (s.n < 1 || s.n > kSpanLevels) return hipErrorInvalidValue;
  if (t.canon)
    k_down_span<true><<<1, 1024, 0, st>>>(a, t, L, s, sub_cnt, leaf, pp_len);
  else
    k_down_span<false><<<1, 1024, 0, st>>>(a, t, L, s, sub_cnt, leaf, pp_len);
  return hipGetLastError();
}

hipError_t launch_down(const ExtArgs& a, const TpTree& t, int L, int64_t base, int64_t F,
                       uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st) {
  if (F == 0) return hipSuccess;
  const unsigned grid = (unsigned)((F + kBlock - 1) / kBlock);
  if (t.canon)
    k_down_run<0, true><<<grid, kBlock, 0, st>>>(a, t, L, base, F, sub_cnt, leaf, pp_len);
  else
    k_down_run<0, false><<<grid, kBlock, 0, st>>>(a, t, L, base, F, sub_cnt, leaf, pp_len);
  return hipGetLastError();
}

hipError_t launch_down_run(const ExtArgs& a, const TpTree& t, int L, int64_t base, int64_t F,
                           uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st) {
  if (F == 0) return hipSuccess;
  const unsigned grid = (unsigned)((F + kBlock - 1) / kBlock);
  if (t.canon)
    k_down_run<1, true><<<grid, kBlock, 0, st>>>(a, t, L, base, F, sub_cnt, leaf, pp_len);
  else
    k_down_run<1, false><<<grid, kBlock, 0, st>>>(a, t, L, base, F, sub_cnt, leaf, pp_len);
  return hipGetLastError();
}

// Two levels per launch: a launch costs ~7 us however little it
// does, and a sweep has one per level.  One thread per node x of the run's
// upper level does the work for x and for its children (they are x's alone,
// and each count is read right after this thread wrote it).  The loads are
// batched: x's children's codes and child ranges kSweepBatch at a time, then
// their own children's counts all together, so that a thread waits for about
// three load latencies instead of a few per child.  (The down sweep keeps its
// per-child loop: batched the same way it measured slower, its stores and
// position chain per child.)
constexpr int kSweepBatch = 4;

template <bool TP>
__global__ __launch_bounds__(kBlock) void k_up_run(ExtArgs a, int64_t base, int64_t F,
                                                   const int32_t* rep, uint32_t* sub_cnt) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= F) return;
  const int64_t x = base + t;
  const uint8_t k = a.t.nch[x];
  uint32_t c = own_count<TP>(k, rep, x);
  if (nch_internal(k)) {
    const int64_t c0 = a.t.cstart[x];
    for (int j0 = 0; j0 < k; j0 += kSweepBatch) {
      uint8_t ky[kSweepBatch];
      int64_t cs[kSweepBatch];
#pragma unroll
      for (int j = 0; j < kSweepBatch; ++j) {
        const bool in = j0 + j < k;
        ky[j] = in ? a.t.nch[c0 + j0 + j] : (uint8_t)0;
        cs[j] = in ? (int64_t)a.t.cstart[c0 + j0 + j] : 0;
      }
      uint32_t cy[kSweepBatch];
#pragma unroll
      for (int j = 0; j < kSweepBatch; ++j)
        cy[j] = j0 + j < k ? own_count<TP>(ky[j], rep, c0 + j0 + j) : 0u;
      for (int g0 = 0;; g0 += kSweepBatch) {
        uint32_t v[kSweepBatch][kSweepBatch];
#pragma unroll
        for (int j = 0; j < kSweepBatch; ++j)
#pragma unroll
          for (int g = 0; g < kSweepBatch; ++g)
            v[j][g] = nch_internal(ky[j]) && g0 + g < ky[j] ? sub_cnt[cs[j] + g0 + g] : 0u;
        bool more = false;
#pragma unroll
        for (int j = 0; j < kSweepBatch; ++j) {
#pragma unroll
          for (int g = 0; g < kSweepBatch; ++g) cy[j] += v[j][g];
          more |= nch_internal(ky[j]) && g0 + kSweepBatch < ky[j];
        }
        if (!more) break;
      }
#pragma unroll
      for (int j = 0; j < kSweepBatch; ++j) {
        if (j0 + j < k) {
          sub_cnt[c0 + j0 + j] = cy[j];
          c += cy[j];
        }
      }
    }
  }
  sub_cnt[x] = c;
}

hipError_t launch_up_run(const ExtArgs& a, int64_t base, int64_t F, uint32_t* sub_cnt,
                         hipStream_t st) {
  if (F == 0) return hipSuccess;
  k_up_run<false><<<(unsigned)((F + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, base, F, nullptr,
                                                                            sub_cnt);
  return hipGetLastError();
}

hipError_t launch_tp_up_run(const ExtArgs& a, int64_t base, int64_t F, const int32_t* rep,
                            uint32_t* cnt, hipStream_t st) {
  if (F == 0) return hipSuccess;
  k_up_run<true><<<(unsigned)((F + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, base, F, rep, cnt);
  return hipGetLastError();
}

// A cycle of chains found from the head of its first chain x is a prime path
// from each of x's other vertices too: the j-th vertex's prime paths are the
// root's cycles, in the same order (they pass the rest of x, then differ
// where the root's do).  One workgroup per chain of two or more vertices
// takes its root's leaves 16 a thread at a time and gives the cycles among them
// their places after every other vertex's position.
// Unions of many graphs have many such chains with few leaves each: 256 threads
// and a quarter of the leaves a step then (4096 CFGs: 163 us a union with 1024,
// 32 with 256).
constexpr int kRotItems = 16;
constexpr int32_t kManyRot = 1024;
template <int NT>
__global__ __launch_bounds__(NT) void k_rotations(ExtArgs a, DChains ch, TpTree t,
                                                    const int32_t* rot, int32_t range_lo,
                                                    const int64_t* rb,
                                                    uint64_t* leaf, int32_t* pp_len) {
  __shared__ int32_t s_w[NT / 64];
  const int x = rot[blockIdx.x];
  if (PathTotals::root_cycles(a.g, a.tot)[x] == 0) return;
  const int o = ch.off[x], m = ch.off[x + 1] - o;
  const int head = ch.v[o] - range_lo;
  const int64_t p0 = rb[head], p1 = rb[head + 1];
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  int64_t carry = 0;
  for (int64_t b = p0; b < p1; b += NT * kRotItems) {
    // a wave's leaves are consecutive: 64 at a time
    const int64_t w0 = b + (int64_t)wave * 64 * kRotItems + lane;
    uint64_t lf[kRotItems];
#pragma unroll
    for (int i = 0; i < kRotItems; ++i) lf[i] = w0 + 64 * i < p1 ? leaf[w0 + 64 * i] : 0ull;
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kRotItems; ++i) mine += __builtin_popcountll(__ballot(lf[i] >> 63));
    if (lane == 0) s_w[wave] = mine;
    __syncthreads();
    int64_t at = carry;
    int all = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      at += w < wave ? s_w[w] : 0;
      all += s_w[w];
    }
    carry += all;
#pragma unroll
    for (int i = 0; i < kRotItems; ++i) {
      const uint64_t cyc = __ballot(lf[i] >> 63);
      if (lf[i] >> 63) {
        const int64_t k = at + __builtin_popcountll(cyc & ((1ull << lane) - 1));
        const int32_t len = pp_len[w0 + 64 * i];
        const int32_t canon = t.canon ? t.leaf_canon[w0 + 64 * i] : 0;
        for (int j = 1; j < m; ++j) {
          const int64_t r = rb[ch.v[o + j] - range_lo] + k;
          leaf[r] = lf[i] | (uint64_t)j << kLeafStartShift;
          pp_len[r] = len;
          if (t.canon) t.leaf_canon[r] = canon;
        }
      }
      at += __builtin_popcountll(cyc);
    }
    __syncthreads();  // s_w is read before the next step writes it
  }
}

hipError_t launch_rotations(const ExtArgs& a, const DChains& ch, const TpTree& t,
                            const int32_t* rot, int32_t n_rot, int32_t range_lo, const int64_t* rb,
                            uint64_t* leaf, int32_t* pp_len, hipStream_t st) {
  if (n_rot <= 0) return hipSuccess;
  if (n_rot >= kManyRot)
    k_rotations<256><<<(unsigned)n_rot, 256, 0, st>>>(a, ch, t, rot, range_lo, rb, leaf, pp_len);
  else
    k_rotations<1024><<<(unsigned)n_rot, 1024, 0, st>>>(a, ch, t, rot, range_lo, rb, leaf, pp_len);
  return hipGetLastError();
}

// Each wave writes the prime paths of 64 consecutive ranks, one per lane, by
// walking parent links from their leaves.  The walks are aligned by depth: a
// lane starts when the wave reaches the depth of its leaf, so at every step
// the active lanes stand on one tree level, mostly at nodes close together
// in that level's array (consecutive ranks are neighbours in depth-first
// order, and a tile's children are stored in its parents' order), and a load
// touches few cache lines.  The entries of kPPSeg consecutive depths
// go to LDS, one row per lane; then the wave stores the rows, kPPSeg lanes
// per row, so that a store covers a few whole row segments instead of one
// word in each of 64 lines.

// LDS: the chains' rows (off, v) are staged as 16-bit words (the union has at
// most kStageVertices vertices), so that a step inside a chain costs an LDS
// read; only a step to the parent's chain loads from the tree.  The rows are
// 16-bit words there too, which makes room for segments of 32 depths: the
// stress CFG's 3.5 GB took 2.58 ms in segments of 16 (5.4 GB written, since a
// segment's ends share their lines with its neighbours', written at another
// time), 2.05 in segments of 32, 2.4 in 64; windows shifted so that a segment
// is a whole line take the lanes off their common depth and cost more, 2.9.
constexpr int kStageVertices = 2048;

template <bool LDS>
__global__ __launch_bounds__(kBlock) void k_pp_write(ExtArgs a, DChains ch, int32_t n,
                                                     const uint64_t* leaf, const int64_t* pp_off,
                                                     int64_t n_pp, int32_t* pp_vtx) {
  using Entry = std::conditional_t<LDS, uint16_t, int32_t>;
  constexpr int kPPSeg = LDS ? 32 : 16;
  constexpr int kPPRow = kPPSeg + 4 / (int)sizeof(Entry);  // odd in words: rows in different banks
  __shared__ Entry s_row[kBlock * kPPRow];
  __shared__ int64_t s_lo[kBlock];
  __shared__ int32_t s_len[kBlock];
  __shared__ int32_t s_done[kBlock];
  extern __shared__ uint16_t s_ch[];  // v [n], then off [g.n + 1]
  const int tid = (int)threadIdx.x, lane = lane_id(), wb = tid - lane;
  const int64_t i = (int64_t)blockIdx.x * kBlock + tid;
  if constexpr (LDS) {
    for (int k = tid; k < n; k += kBlock) s_ch[k] = (uint16_t)ch.v[k];
    for (int k = tid; k <= a.g.n; k += kBlock) s_ch[n + k] = (uint16_t)ch.off[k];
    __syncthreads();
  }
  auto row_of = [&](int x) { return LDS ? (int)s_ch[n + x] : ch.off[x]; };
  auto vertex = [&](int k) { return LDS ? (int)s_ch[k] : ch.v[k]; };
  int64_t lo = 0;
  int32_t len = 0;
  int32_t up = -1;          // parent of the node whose chain is being walked
  int32_t c0 = 0, at = -1;  // the chain's row begins at c0; the next vertex is v[at]
  if (i < n_pp) {
    lo = pp_off[i];
    len = (int32_t)(pp_off[i + 1] - lo);
    const uint64_t lf = leaf[i];
    const int32_t x = (int32_t)(lf & 0xFFFFFFFFu);
    const int c = node_v(a.t.info[x]);
    up = a.t.par[x];
    c0 = row_of(c);
    // a cycle ends at the vertex it starts at
    at = (lf & kLeafCycle) ? c0 + (int)((lf >> kLeafStartShift) & 0x1FFF) : row_of(c + 1) - 1;
  }
  s_lo[tid] = lo;
  s_len[tid] = len;
  int32_t lmax = len;  // the wave's longest path
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const int32_t y = __shfl_xor(lmax, d, 64);
    lmax = y > lmax ? y : lmax;
  }
  int32_t done = len;  // entries done .. len - 1 are walked
  Entry* row = s_row + tid * kPPRow;
  for (int kb = lmax > 0 ? (lmax - 1) / kPPSeg * kPPSeg : -1; kb >= 0; kb -= kPPSeg) {
    // depths kb + kPPSeg - 1 down to kb: one dependent load per chain
    Entry v[kPPSeg];
#pragma unroll
    for (int m = kPPSeg - 1; m >= 0; --m) {
      const int k = kb + m;
      v[m] = 0;
      if (k < len) {
        v[m] = (Entry)vertex(at);
        done = k;
        if (--at < c0 && up >= 0) {  // on to the parent's chain
          const int c = node_v(a.t.info[up]);
          up = a.t.par[up];
          c0 = row_of(c);
          at = row_of(c + 1) - 1;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < kPPSeg; ++m) row[m] = v[m];
    s_done[tid] = done;
    wave_sync();
    // the wave's rows, kPPSeg lanes per row: depths kb .. kb + kPPSeg - 1 of
    // each path, those walked in this round
#pragma unroll
    for (int r0 = 0; r0 < 64; r0 += 64 / kPPSeg) {
      const int r = wb + r0 + lane / kPPSeg, k = kb + lane % kPPSeg;
      if (k >= s_done[r] && k < s_len[r]) pp_vtx[s_lo[r] + k] = s_row[r * kPPRow + (k - kb)];
    }
    wave_sync();  // the rows are read before the next round writes them
  }
}

hipError_t launch_pp_write(const ExtArgs& a, const DChains& ch, int32_t n, const uint64_t* leaf,
                           const int64_t* pp_off, int64_t n_pp, int32_t* pp_vtx, hipStream_t st) {
  if (n_pp == 0) return hipSuccess;
  const unsigned grid = (unsigned)((n_pp + kBlock - 1) / kBlock);
  if (n <= kStageVertices) {
    const size_t lds = sizeof(uint16_t) * ((size_t)n + a.g.n + 1);
    k_pp_write<true><<<grid, kBlock, lds, st>>>(a, ch, n, leaf, pp_off, n_pp, pp_vtx);
  } else {
    k_pp_write<false><<<grid, kBlock, 0, st>>>(a, ch, n, leaf, pp_off, n_pp, pp_vtx);
  }
  return hipGetLastError();
}

}  // namespace tpg

namespace tpg {

// After the positions and the offsets exist: first prime path of each
// component and the offset of that path's first entry.
__global__ void k_comp_pp_starts(DGraph g, const int64_t* rb, const int64_t* pp_off,
                                 int64_t* pp_start, int64_t* ppv_start) {
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (c > g.n_comp) return;
  const int64_t r = rb[g.cbase[c]];
  pp_start[c] = r;
  ppv_start[c] = pp_off[r];
}

hipError_t launch_comp_pp_starts(const DGraph& g, const int64_t* rb, const int64_t* pp_off,
                                 int64_t* pp_start, int64_t* ppv_start, hipStream_t st) {
  k_comp_pp_starts<<<(unsigned)((g.n_comp + 1 + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      g, rb, pp_off, pp_start, ppv_start);
  return hipGetLastError();
}

// Every node's paths by length, one by one (see k_path_lengths; level 1: the
// paths inside one chain).
__global__ void k_level_comp_counts(ExtArgs a, int64_t n_nodes, int64_t* lvl) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n_nodes) return;
  const uint32_t inf = a.t.info[x];
  const int T = a.t.tl[x], v = node_v(inf);
  const int m1 = a.g.len[v - a.g.loc[v] + node_v1l(inf)], mk = a.g.len[v];
  const bool cyc = inf & F_CYC, one = x < a.seed_n;
  unsigned long long* row = reinterpret_cast<unsigned long long*>(lvl) + (int64_t)a.g.comp[v] * 64;
  const int top = cyc ? T + 1 : T, nd = one || cyc ? m1 : m1 + mk - 1;
  unsigned long long deep = 0;
  for (int d = 0; d < nd; ++d) {
    const int c = cyc ? m1 - d : one ? d + 1 : min(min(d + 1, nd - d), min(m1, mk));
    if (top - d >= 64) deep += (unsigned long long)c;
    else atomicAdd(row + (top - d) - 1, (unsigned long long)c);
  }
  if (deep) atomicAdd(row + 63, deep);
}

hipError_t launch_level_comp_counts(const ExtArgs& a, int64_t n_nodes, int64_t* lvl_comp,
                                    hipStream_t st) {
  if (n_nodes == 0) return hipSuccess;
  k_level_comp_counts<<<(unsigned)((n_nodes + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, n_nodes,
                                                                                      lvl_comp);
  return hipGetLastError();
}

}  // namespace tpg
