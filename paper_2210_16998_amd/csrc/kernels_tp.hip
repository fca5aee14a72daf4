// Test-path kernels: BFS tables, splice, canonical sort and deduplication.
//
// A test path extends a prime path to the initial and final nodes (paper
// Sec. 7.3, the Ammann-Offutt construction; Problem 1 asks for test paths
// covering every prime path).  The shortest connection is taken, and among
// shortest ones the lexicographically smallest, so the result is unique:
//  * prefix(v): smallest shortest entry -> v path.  A FIFO breadth-first
//    search that scans successors in ascending order discovers it (each
//    layer's queue order is the lexicographic order of those paths); the
//    level-synchronous search here reproduces FIFO discovery order by giving
//    every vertex the discoverer with the smallest (queue position, successor
//    slot) key.
//  * suffix(v): smallest shortest v -> exit path: distances to the exit by a
//    reverse search, then the smallest successor one step closer.
//  * TP(p) = prefix(v1) without v1 ++ p ++ suffix(vk) without vk.
//
// Order and duplicates are read off the path tree; no test path is compared
// with another (see k_tp_mark).  Every distinct test path owns one node of
// the tree, two subtree sweeps like the prime paths' give the nodes' places
// in lexicographic order, and the rows are written where they belong.

#include <climits>

#include "kernels.h"

namespace tpg {

constexpr int kBfsThreads = 256;
constexpr int kMaxComp = 4096;  // vertices per component

// Exclusive scan of data[0..m) in place (m <= kMaxComp), in chunks of
// 4 * kBfsThreads; returns the total.
__device__ int lds_excl_scan(int16_t* data, int m, int32_t* s_w) {
  int carry = 0;
  for (int c0 = 0; c0 < m; c0 += 4 * kBfsThreads) {
    const int b = c0 + (int)threadIdx.x * 4;
    int v[4];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = (b + k < m) ? (int)data[b + k] : 0;
      sum += v[k];
    }
    int tot;
    int pre = block_excl_scan<kBfsThreads, int>(sum, tot, s_w) + carry;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (b + k < m) data[b + k] = (int16_t)pre;
      pre += v[k];
    }
    carry += tot;
    __syncthreads();
  }
  return carry;
}

// One workgroup per component: distances from the entry with the FIFO
// (smallest discoverer) parent, the BFS tree's preorder (children in
// ascending order) as rank ranges, distances to the exit, and next[].
//
// The forward search keeps one queue in LDS whose layers are contiguous;
// the children of a vertex form a contiguous ascending block of the next
// layer, which gives subtree sizes bottom-up and preorder ranks top-down.
__global__ __launch_bounds__(kBfsThreads) void k_bfs_dist(DGraph g, BfsOut b) {
  __shared__ int16_t s_df[kMaxComp];
  __shared__ int16_t s_db[kMaxComp];
  __shared__ int32_t s_key[kMaxComp];   // smallest discoverer key, then the parent (local id)
  __shared__ int16_t s_q[kMaxComp];     // forward queue (layers contiguous), then reverse queue
  __shared__ int16_t s_lb[kMaxComp + 2];  // layer d of the forward queue: [s_lb[d], s_lb[d + 1])
  __shared__ int16_t s_cnt[kMaxComp];   // per-layer child counts, then preorder ranks
  __shared__ int32_t s_sz[kMaxComp];    // subtree sizes, then reverse-search marks
  __shared__ int32_t s_w[kBfsThreads / 64];
  __shared__ int32_t s_m;
  const int c = (int)blockIdx.x;
  const int base = g.cbase[c];
  const int nc = g.cbase[c + 1] - base;
  const int tid = (int)threadIdx.x;
  for (int v = tid; v < nc; v += kBfsThreads) {
    s_df[v] = -1;
    s_db[v] = -1;
    s_key[v] = INT_MAX;
    s_sz[v] = 1;
    b.parent[base + v] = -1;
    b.next[base + v] = -1;
  }
  const int el = g.centry[c] - base;
  if (tid == 0) {
    s_df[el] = 0;
    s_key[el] = -1;
    s_q[0] = (int16_t)el;
    s_lb[0] = 0;
    s_lb[1] = 1;
  }
  __syncthreads();
  int qb = 0, qe = 1, d = 0;
  while (qe > qb) {
    const int m = qe - qb;
    for (int q = tid; q < m; q += kBfsThreads) {
      const int u = base + s_q[qb + q];
      for (int k = g.sp[u]; k < g.sp[u + 1]; ++k) {
        const int wl = g.s[k] - base;
        if (s_df[wl] == -1) atomicMin(&s_key[wl], q * 64 + (k - g.sp[u]));
      }
    }
    __syncthreads();
    for (int q = tid; q < m; q += kBfsThreads) {
      const int u = base + s_q[qb + q];
      int cnt = 0;
      for (int k = g.sp[u]; k < g.sp[u + 1]; ++k) {
        const int wl = g.s[k] - base;
        if (s_df[wl] == -1 && s_key[wl] == q * 64 + (k - g.sp[u])) ++cnt;
      }
      s_cnt[q] = (int16_t)cnt;
    }
    __syncthreads();
    const int m2 = lds_excl_scan(s_cnt, m, s_w);
    for (int q = tid; q < m; q += kBfsThreads) {
      const int u = base + s_q[qb + q];
      int pos = qe + s_cnt[q];
      for (int k = g.sp[u]; k < g.sp[u + 1]; ++k) {
        const int wl = g.s[k] - base;
        if (s_df[wl] == -1 && s_key[wl] == q * 64 + (k - g.sp[u])) {
          s_q[pos++] = (int16_t)wl;
          b.parent[base + wl] = u;
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < m2; i += kBfsThreads) {
      const int wl = s_q[qe + i];
      s_df[wl] = (int16_t)(d + 1);
      s_key[wl] = s_q[qb + s_key[wl] / 64];
    }
    qb = qe;
    qe += m2;
    ++d;
    if (tid == 0) s_lb[d + 1] = (int16_t)qe;
    __syncthreads();
  }
  const int nlayers = d;  // layers 0 .. nlayers - 1
  // subtree sizes, deepest layer first
  for (int l = nlayers - 1; l >= 1; --l) {
    for (int i = s_lb[l] + tid; i < s_lb[l + 1]; i += kBfsThreads) {
      const int v = s_q[i];
      atomicAdd(&s_sz[s_key[v]], s_sz[v]);
    }
    __syncthreads();
  }
  // preorder ranks, top layer first: a vertex follows its parent and the
  // subtrees of its smaller siblings
  if (tid == 0) s_cnt[el] = 0;
  __syncthreads();
  for (int l = 1; l < nlayers; ++l) {
    const int lo = s_lb[l];
    for (int i = lo + tid; i < s_lb[l + 1]; i += kBfsThreads) {
      const int v = s_q[i];
      const int p = s_key[v];
      int acc = 0;
      for (int j = i - 1; j >= lo && s_key[s_q[j]] == p; --j) acc += s_sz[s_q[j]];
      s_cnt[v] = (int16_t)(s_cnt[p] + 1 + acc);
    }
    __syncthreads();
  }
  for (int v = tid; v < nc; v += kBfsThreads) {
    const bool r = s_df[v] >= 0;
    b.pre[base + v] = r ? base + s_cnt[v] : -1;
    b.pend[base + v] = r ? base + s_cnt[v] + s_sz[v] : -1;
  }
  __syncthreads();
  // distances to the exit (reverse search; order does not matter)
  for (int v = tid; v < nc; v += kBfsThreads) s_sz[v] = 0;
  __syncthreads();
  const int xl = g.cexit[c] - base;
  if (tid == 0) {
    s_db[xl] = 0;
    s_q[0] = (int16_t)xl;
    s_sz[xl] = 1;
  }
  __syncthreads();
  qb = 0;
  qe = 1;
  d = 0;
  while (qe > qb) {
    if (tid == 0) s_m = 0;
    __syncthreads();
    for (int q = qb + tid; q < qe; q += kBfsThreads) {
      const int u = base + s_q[q];
      for (int k = g.pp[u]; k < g.pp[u + 1]; ++k) {
        const int wl = g.p[k] - base;
        if (atomicExch(&s_sz[wl], 1) == 0) s_q[qe + atomicAdd(&s_m, 1)] = (int16_t)wl;
      }
    }
    __syncthreads();
    const int m2 = s_m;
    for (int i = tid; i < m2; i += kBfsThreads) s_db[s_q[qe + i]] = (int16_t)(d + 1);
    qb = qe;
    qe += m2;
    ++d;
    __syncthreads();
  }
  for (int v = tid; v < nc; v += kBfsThreads) {
    b.dist_f[base + v] = s_df[v];
    b.dist_b[base + v] = s_db[v];
    if (v != xl && s_db[v] > 0) {
      const int u = base + v;
      for (int k = g.sp[u]; k < g.sp[u + 1]; ++k)
        if (s_db[g.s[k] - base] == s_db[v] - 1) {
          b.next[u] = g.s[k];
          break;
        }
    }
  }
}

hipError_t launch_bfs_dist(const DGraph& g, const BfsOut& b, hipStream_t st) {
  k_bfs_dist<<<(unsigned)g.n_comp, kBfsThreads, 0, st>>>(g, b);
  return hipGetLastError();
}

// Prefix / suffix tables (graph-wide ids): entries before v on its
// smallest shortest path from the entry, entries after v to the exit.
__global__ void k_bfs_tables(DGraph g, BfsOut b) {
  const int v = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (v >= g.n) return;
  const int df = b.dist_f[v], db = b.dist_b[v];
  if (df > 0) {
    const int64_t lo = b.pfx_off[v];
    int64_t pos = lo + df - 1;
    int x = b.parent[v];
    while (x >= 0 && pos >= lo) {
      b.pfx[pos--] = x;
      x = b.parent[x];
    }
  }
  if (db > 0) {
    int64_t pos = b.sfx_off[v];
    const int64_t hi = pos + db;
    int x = b.next[v];
    while (x >= 0 && pos < hi) {
      b.sfx[pos++] = x;
      x = b.next[x];
    }
  }
}

hipError_t launch_bfs_tables(const DGraph& g, const BfsOut& b, hipStream_t st) {
  k_bfs_tables<<<(unsigned)((g.n + kBlock - 1) / kBlock), kBlock, 0, st>>>(g, b);
  return hipGetLastError();
}

// Graph-wide ids -> ids local to each component (batched output).
__global__ void k_localize(const int32_t* loc, int32_t* v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    v[i] = loc[v[i]];
}

hipError_t launch_localize(const int32_t* loc, int32_t* v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_localize<<<(unsigned)std::min<int64_t>(4096, (n + kBlock - 1) / kBlock), kBlock, 0, st>>>(loc, v, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// test-path order from the path tree
// ---------------------------------------------------------------------------
// In chains, a test path is the BFS-tree path to its prime path's first chain,
// the prime path, and the shortest way on from its last chain (a cycle that
// closes inside its first chain goes on to that chain's end, so the cycle's
// prime paths from the chain's other vertices give the same test path as the
// one from its head).  Let (W, Y) be the first arc on it that is not a
// BFS-tree arc: what follows depends on the test path only from W on, and
// <W, Y> is a node of W's tree.  Following the test path's chains from there
// as far as there are nodes ends at its node E:
//  * the prime path's part is always there: a simple path with its first
//    chains dropped is a simple path from the later chain;
//  * equal test paths end at the same node, and different ones do not: below
//    E the path goes on along the shortest way from E's last chain, which E
//    alone decides;
//  * in lexicographic order, test paths with the same (W, Y) follow the depth-
//    first order of their nodes, the one of an inner node E coming where its
//    next chain would (no child of E is that chain);
//  * test paths with different (W, Y) follow the depth-first order of the BFS
//    tree with the other arcs as leaves (k_tp_arc_order); the one test path
//    that is a BFS-tree path all along belongs to the exit.
// So the test paths' nodes are marked (k_tp_mark, with a prime path for each),
// counted bottom-up, and given their places top-down.  k_down_run finds, for
// every node with prime paths below it, the node of the path with its
// BFS-tree part dropped, from its parent's.  Before, every test path was
// spliced packed, sorted by merge rounds that compared them and unpacked
// again: the test-path stage of the 400-vertex stress CFG took 21 ms of a
// 30.8 ms call, now 11 ms of 19.9 (its rows alone are 21.8 GB); a batch of
// 4096 CFGs went from 11.1 to 7.6 ms, a 1000-vertex CFG from 6.7 to 4.3.

// First chain of the BFS tree (tpar) and next chain on the shortest way to
// the exit (nx), -1 for none.  One thread per chain.
__global__ void k_tp_chain_links(DGraph x, DChains ch, BfsOut b, TpTree t) {
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= x.n) return;
  const int p = b.parent[ch.v[ch.off[c]]];
  const int q = b.next[ch.v[ch.off[c + 1] - 1]];
  t.tpar[c] = p >= 0 ? ch.of[p] : -1;
  t.nx[c] = q >= 0 ? ch.of[q] : -1;
  t.cdist[c] = b.dist_f[ch.v[ch.off[c]]];
  t.cback[c] = b.dist_b[ch.v[ch.off[c + 1] - 1]];
}

// The places of every component's arcs off the BFS tree, and of the exit's
// tree path, in test-path order: order[gbase[c] ..) lists the arcs as W <<
// kArcSlotBits | slot of Y among W's successors, and the exit's chain X as ~X.
// With the vertices' BFS-tree preorder, an arc (w, e) comes right before the
// first tree child of w above e (rank s), or at the end of w's subtree; among
// arcs at the same rank s, those that end a subtree come first, deepest first,
// then those before child s, w's own in the order of e; the exit's path comes
// last at the exit's rank.  The arcs that end the subtrees nested in w's end
// are counted by walking down the last tree children.  One workgroup per
// component.
__global__ __launch_bounds__(kBlock) void k_tp_arc_order(DGraph g, DGraph x, DChains ch, BfsOut b,
                                                         const int32_t* gbase, int32_t* order) {
  __shared__ int32_t s_at[kMaxComp + 1];   // arcs per rank, then their first place
  __shared__ int32_t s_end[kMaxComp + 1];  // of them, arcs that end a subtree
  __shared__ int32_t s_w[kBlock / 64];
  const int c = (int)blockIdx.x, tid = (int)threadIdx.x;
  const int base = g.cbase[c], nc = g.cbase[c + 1] - base;
  const int x0 = x.cbase[c], x1 = x.cbase[c + 1];
  for (int k = tid; k <= nc; k += kBlock) {
    s_at[k] = 0;
    s_end[k] = 0;
  }
  __syncthreads();
  // rank (local) at which arc k out of w comes; the successors ascend
  auto rank_of = [&](int w, int k, int k1, bool& ends) {
    int r = b.pend[w] - base;
    ends = true;
    for (int j = k + 1; j < k1; ++j) {
      const int u = ch.v[ch.off[x.s[j]]];
      if (b.parent[u] == w) {
        r = b.pre[u] - base;
        ends = false;
        break;
      }
    }
    return r;
  };
  auto tree_arc = [&](int w, int k) { return b.parent[ch.v[ch.off[x.s[k]]]] == w; };
  const int xl = g.cexit[c];
  for (int i = x0 + tid; i < x1; i += kBlock) {
    const int w = ch.v[ch.off[i + 1] - 1];
    const int k0 = x.sp[i], k1 = x.sp[i + 1];
    for (int k = k0; k < k1; ++k) {
      if (tree_arc(w, k)) continue;
      bool ends;
      const int r = rank_of(w, k, k1, ends);
      atomicAdd(&s_at[r], 1);
      if (ends) atomicAdd(&s_end[r], 1);
    }
    if (w == xl) atomicAdd(&s_at[b.pre[w] - base], 1);
  }
  __syncthreads();
  // first place of every rank
  int carry = gbase[c];
  for (int k0 = 0; k0 <= nc; k0 += kBlock) {
    const int k = k0 + tid;
    const int v = k <= nc ? s_at[k] : 0;
    int tot;
    const int pre = block_excl_scan<kBlock, int>(v, tot, s_w);
    if (k <= nc) s_at[k] = carry + pre;
    carry += tot;
  }
  __syncthreads();
  for (int i = x0 + tid; i < x1; i += kBlock) {
    const int w = ch.v[ch.off[i + 1] - 1];
    const int k0 = x.sp[i], k1 = x.sp[i + 1];
    int deeper = -1;  // arcs that end the subtrees nested in the end of w's
    int same = 0, last_r = -1;
    for (int k = k0; k < k1; ++k) {
      if (tree_arc(w, k)) continue;
      bool ends;
      const int r = rank_of(w, k, k1, ends);
      same = r == last_r ? same + 1 : 0;  // earlier arcs of w at this rank
      last_r = r;
      int before = s_end[r];
      if (ends) {
        if (deeper < 0) {
          deeper = 0;
          for (int y = i;;) {  // down the last tree children
            const int wy = ch.v[ch.off[y + 1] - 1];
            int child = -1, tail = 0;
            for (int j = x.sp[y + 1] - 1; j >= x.sp[y]; --j) {
              if (tree_arc(wy, j)) {
                child = x.s[j];
                break;
              }
              ++tail;  // an arc after the last tree child: it ends wy's subtree
            }
            if (y != i) deeper += tail;
            if (child < 0) break;
            y = child;
          }
        }
        before = deeper;
      }
      order[s_at[r] + before + same] = i << kArcSlotBits | (k - k0);
    }
    if (w == xl) {
      const int r = b.pre[w] - base;
      order[(r < nc ? s_at[r + 1] : carry) - 1] = ~i;
    }
  }
}

hipError_t launch_tp_arcs(const DGraph& g, const DGraph& x, const DChains& ch, const BfsOut& b,
                          const TpTree& t, const int32_t* gbase, int32_t* order, hipStream_t st) {
  k_tp_chain_links<<<(unsigned)((x.n + kBlock - 1) / kBlock), kBlock, 0, st>>>(x, ch, b, t);
  k_tp_arc_order<<<(unsigned)g.n_comp, kBlock, 0, st>>>(g, x, ch, b, gbase, order);
  return hipGetLastError();
}

// The child of node c labelled chain y (-1: none).
__device__ __forceinline__ int64_t child_of(const TreeBufs& t, int64_t c, int y) {
  const uint8_t k = t.nch[c];
  if (k == 0 || k >= kNchPP) return -1;
  const int64_t c0 = t.cstart[c];
  for (int64_t z = c0; z < c0 + k; ++z)
    if (node_v(t.info[z]) == y) return z;
  return -1;
}

// Marks the node of every prime path's test path (rep: a prime path of the
// node + 1; all of a node's prime paths give the same test path, so any of
// them may win).  canon: the prime paths' nodes with their BFS-tree parts
// dropped.  state (longest-first covering; may be null): only the chosen
// prime paths; else the paths from the head of a chain, which cover the rest.
__global__ __launch_bounds__(kBlock) void k_tp_mark(ExtArgs a, TpTree t, const uint64_t* leaf,
                                                    int64_t n_pp, const uint8_t* state,
                                                    int32_t* rep) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n_pp) return;
  const uint64_t lf = leaf[i];
  if (state ? state[i] != 1 : ((lf >> kLeafStartShift) & 0x1FFF) != 0) return;
  int z = node_v(a.t.info[lf & 0xFFFFFFFFu]);
  int64_t c = t.leaf_canon[i];
  while (c < 0) {  // still a BFS-tree path: on towards the exit
    const int y = t.nx[z];
    if (y < 0) {
      c = z;  // all along: the exit's root (root k is chain k)
      break;
    }
    if (t.tpar[y] != z) c = child_of(a.t, z, y);
    z = y;
  }
  for (int y = t.nx[z]; y >= 0; y = t.nx[y]) {
    const int64_t d = child_of(a.t, c, y);
    if (d < 0) break;
    c = d;
  }
  rep[c] = (int32_t)(i + 1);
}

hipError_t launch_tp_mark(const ExtArgs& a, const TpTree& t, const uint64_t* leaf, int64_t n_pp,
                          const uint8_t* state, int32_t* rep, hipStream_t st) {
  if (n_pp == 0) return hipSuccess;
  k_tp_mark<<<(unsigned)((n_pp + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, t, leaf, n_pp, state,
                                                                         rep);
  return hipGetLastError();
}

// Places of the arcs' test paths: a scan of the marked nodes below each arc's
// node in the arcs' order.  cnt: place + 1 of the subtree's first test path
// (0: it has none), as k_tp_down reads it; first[j] = the place of arc j's
// first test path, first[n] = their number.  One workgroup, kArcItems arcs
// per thread and step.
constexpr int kArcItems = 8;
__global__ __launch_bounds__(1024) void k_tp_arc_starts(TreeBufs t, const int32_t* order, int32_t n,
                                                        const int32_t* rep, uint32_t* cnt,
                                                        int64_t* first, int32_t* src,
                                                        int32_t* len, const int32_t* cdist) {
  __shared__ int64_t s_w[16];
  int64_t carry = 0;
  for (int32_t b = 0; b < n; b += 1024 * kArcItems) {
    const int32_t j0 = b + (int32_t)threadIdx.x * kArcItems;
    int64_t node[kArcItems];
    uint32_t c[kArcItems];
    int64_t sum = 0;
#pragma unroll
    for (int j = 0; j < kArcItems; ++j) {
      node[j] = -1;
      c[j] = 0;
      if (j0 + j < n) {
        const int32_t g = order[j0 + j];
        node[j] = g < 0 ? (int64_t)~g
                        : (int64_t)t.cstart[g >> kArcSlotBits] + (g & ((1 << kArcSlotBits) - 1));
        c[j] = g < 0 ? (rep[node[j]] != 0 ? 1u : 0u) : cnt[node[j]];
        sum += c[j];
      }
    }
    int64_t tot;
    int64_t at = carry + block_excl_scan<1024, int64_t>(sum, tot, s_w);
#pragma unroll
    for (int j = 0; j < kArcItems; ++j) {
      if (j0 + j < n) {
        first[j0 + j] = at;
        const bool exit_path = order[j0 + j] < 0;
        if (exit_path && c[j]) {
          src[at] = rep[node[j]] - 1;
          len[at] = cdist[node[j]] + t.tl[node[j]];
        }
        if (!exit_path) cnt[node[j]] = c[j] ? (uint32_t)(at + 1) : 0u;
        at += c[j];
      }
    }
    carry += tot;
  }
  if (threadIdx.x == 0) first[n] = carry;
}

hipError_t launch_tp_arc_starts(const ExtArgs& a, const TpTree& tt, const int32_t* order, int32_t n,
                                const int32_t* rep, uint32_t* cnt, int64_t* first, int32_t* src,
                                int32_t* len, hipStream_t st) {
  k_tp_arc_starts<<<1, 1024, 0, st>>>(a.t, order, n, rep, cnt, first, src, len, tt.cdist);
  return hipGetLastError();
}

// Node x with its first test path at place r: its own goes before its first
// child above the chain that follows on the shortest way to the exit; with
// D > 0 the children do the same for theirs.
template <int D>
__device__ __forceinline__ void tp_down_node(const ExtArgs& a, const TpTree& tt, int64_t x,
                                             uint32_t r, const int32_t* rep, uint32_t* cnt,
                                             int32_t* src, int32_t* len) {
  const TreeBufs& t = a.t;
  int32_t own = rep[x];
  int next = 0, row = 0;
  const uint8_t k = t.nch[x];
  if (own) {
    // entries: the way to the node's first chain, its chains (a cycle's first
    // one twice), the way on from its last
    const uint32_t inf = t.info[x];
    const int v = node_v(inf), v1 = v - a.g.loc[v] + node_v1l(inf);
    next = tt.nx[v];
    row = tt.cdist[v1] + t.tl[x] + (k == kNchCycle ? a.g.len[v1] : 0) + tt.cback[v];
  }
  if (k > 0 && k < kNchPP) {
    const int64_t c0 = t.cstart[x];
    for (int64_t y = c0; y < c0 + k; ++y) {
      if (own && node_v(t.info[y]) > next) {
        src[r] = own - 1;
        len[r++] = row;
        own = 0;
      }
      const uint32_t c = cnt[y];
      if constexpr (D > 0) {
        if (c) tp_down_node<D - 1>(a, tt, y, r, rep, cnt, src, len);
      } else {
        cnt[y] = c ? r + 1 : 0u;
      }
      r += c;
    }
  }
  if (own) {
    src[r] = own - 1;
    len[r] = row;
  }
}

// Two levels from the level [base, base + F) on, a thread per node of it.
__global__ __launch_bounds__(kBlock) void k_tp_down_run(ExtArgs a, TpTree tt, int64_t base,
                                                        int64_t F, const int32_t* rep,
                                                        uint32_t* cnt, int32_t* src, int32_t* len) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= F) return;
  const uint32_t r = cnt[base + j];
  if (r) tp_down_node<1>(a, tt, base + j, r - 1, rep, cnt, src, len);
}

hipError_t launch_tp_down_run(const ExtArgs& a, const TpTree& tt, int64_t base, int64_t F,
                              const int32_t* rep, uint32_t* cnt, int32_t* src, int32_t* len,
                              hipStream_t st) {
  if (F == 0) return hipSuccess;
  k_tp_down_run<<<(unsigned)((F + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, tt, base, F, rep, cnt,
                                                                          src, len);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// rows from prime paths
// ---------------------------------------------------------------------------
// Row r is prime path src[r] (r itself without src), with b given between its
// first vertex's prefix row and its last vertex's suffix row.
template <bool ENDS>
__global__ __launch_bounds__(kBlock) void k_row_len(const int32_t* src, int64_t n,
                                                    const int64_t* pp_off, const int32_t* pp_vtx,
                                                    BfsOut b, int32_t* len) {
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (r >= n) return;
  const int64_t i = src ? (int64_t)src[r] : r;
  const int64_t o0 = pp_off[i], o1 = pp_off[i + 1];
  int32_t l = (int32_t)(o1 - o0);
  if constexpr (ENDS) l += b.dist_f[pp_vtx[o0]] + b.dist_b[pp_vtx[o1 - 1]];
  len[r] = l;
}

// A wave writes `rows` (a multiple of R, at most 64) consecutive rows: the
// lanes first load the rows' places and parts, one row each, then the wave
// copies R rows at a time, lane k entries k, 64 + k, .. of each, the first U
// steps of all of them loaded before any is stored.  Bound by memory: on the
// 400-vertex stress CFG (1.94e7 rows, 21.8 GB) it reads 6 GB (the prime paths
// in the test paths' order) and writes 21.5 in 7.2 ms, 3.8 TB/s against 4.9
// for a plain copy.  Measured there as whole calls: one row in flight and 64
// rows a wave 19.5 ms, two 18.8, four 19.0, eight 19.6; stores that bypass the
// cache 21 to 22 (the lines at row ends then go out in parts); 16 bytes a
// lane, seldom aligned, 19.6; a row's prefix and suffix kept in registers for
// the next row 18.9.
template <int U, int R, bool ENDS>
__global__ __launch_bounds__(kBlock) void k_emit_rows(const int32_t* src, int64_t n, int rows,
                                                      const int64_t* pp_off, const int32_t* pp_vtx,
                                                      BfsOut b, const int64_t* out_off,
                                                      int32_t* out_vtx) {
  const int lane = lane_id();
  const int64_t r0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * rows;
  if (r0 >= n) return;
  const int nr = (int)(n - r0 < rows ? n - r0 : rows);
  int64_t out = 0, o0 = 0, p0 = 0, s0 = 0;
  int lq = 0, lp = 0, ls = 0;  // lanes past the last row: empty rows
  if (lane < nr) {
    const int64_t i = src ? (int64_t)src[r0 + lane] : r0 + lane;
    out = out_off[r0 + lane];
    o0 = pp_off[i];
    lq = (int)(pp_off[i + 1] - o0);
    if constexpr (ENDS) {
      const int v1 = pp_vtx[o0], vk = pp_vtx[o0 + lq - 1];
      lp = b.dist_f[v1];
      ls = b.dist_b[vk];
      p0 = b.pfx_off[v1];
      s0 = b.sfx_off[vk];
    }
  }
  auto get = [&](int x, int q) { return __builtin_amdgcn_readlane(x, q); };
  auto get64 = [&](int64_t x, int q) {
    return (int64_t)((uint64_t)(uint32_t)get((int)(uint32_t)x, q) |
                     (uint64_t)(uint32_t)get((int)(x >> 32), q) << 32);
  };
  // row q's parts, each pointer moved so that entry k is at [k]
  struct Row {
    const int32_t *a, *b, *c;
    int np, nq, len;
    __device__ __forceinline__ int32_t at(int k) const {
      if constexpr (!ENDS) return b[k];
      const int32_t* p = k < np ? a : k < np + nq ? b : c;
      return p[k];
    }
  };
  auto row = [&](int q) {
    Row w{};
    w.nq = get(lq, q);
    w.len = w.nq;
    if constexpr (ENDS) {
      w.np = get(lp, q);
      w.len += w.np + get(ls, q);
      w.a = b.pfx + get64(p0, q);
      w.c = b.sfx + get64(s0, q) - (w.np + w.nq);
    }
    w.b = pp_vtx + get64(o0, q) - w.np;
    return w;
  };
  for (int q0 = 0; q0 < nr; q0 += R) {
    int32_t v[R][U];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const Row w = row(q0 + r);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (lane + 64 * u < w.len) v[r][u] = w.at(lane + 64 * u);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const Row w = row(q0 + r);
      int32_t* to = out_vtx + get64(out, q0 + r);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (lane + 64 * u < w.len) to[lane + 64 * u] = v[r][u];
      for (int k = lane + 64 * U; k < w.len; k += 64) to[k] = w.at(k);
    }
  }
}

hipError_t launch_row_len(const int32_t* src, int64_t n, const int64_t* pp_off,
                          const int32_t* pp_vtx, const BfsOut* b, int32_t* len, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  if (b)
    k_row_len<true><<<grid, kBlock, 0, st>>>(src, n, pp_off, pp_vtx, *b, len);
  else
    k_row_len<false><<<grid, kBlock, 0, st>>>(src, n, pp_off, pp_vtx, BfsOut{}, len);
  return hipGetLastError();
}

hipError_t launch_emit_rows(const int32_t* src, int64_t n, int64_t n_entries, const int64_t* pp_off,
                            const int32_t* pp_vtx, const BfsOut* b, const int64_t* out_off,
                            int32_t* out_vtx, hipStream_t st) {
  if (n == 0) return hipSuccess;
  // more rows a wave spread the first loads' cost, fewer keep the chip full:
  // 573 k rows 1.90 ms a call with 16 and 1.95 with 64, 1.9e7 rows 19.2 and 18.8
  const int rows = n >= (int64_t)1 << 20 ? 64 : 16;
  const int64_t waves = (n + rows - 1) / rows;
  const unsigned grid = (unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64));
  // the steps that hold a row of average length, to 5
  const int64_t steps = n_entries / (64 * n) + 1;
#define TPG_EMIT(U, R, E, B)                                                                    \
  k_emit_rows<U, R, E><<<grid, kBlock, 0, st>>>(src, n, rows, pp_off, pp_vtx, B, out_off, out_vtx)
  if (b) {
    if (steps <= 1) TPG_EMIT(1, 4, true, *b);
    else if (steps <= 2) TPG_EMIT(2, 4, true, *b);
    else TPG_EMIT(5, 2, true, *b);
  } else {
    if (steps <= 1) TPG_EMIT(1, 4, false, BfsOut{});
    else TPG_EMIT(2, 4, false, BfsOut{});
  }
#undef TPG_EMIT
  return hipGetLastError();
}

// Starts of the components' test paths: start[c] = first[gbase[c]] (first:
// see k_tp_arc_starts), vstart[c] = the offset there (c = 0 .. n_comp).
__global__ void k_comp_tp_starts(int n_comp, const int32_t* gbase, const int64_t* first,
                                 const int64_t* off, int64_t* start, int64_t* vstart) {
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (c > n_comp) return;
  const int64_t r = first[gbase[c]];
  start[c] = r;
  vstart[c] = off[r];
}

hipError_t launch_comp_tp_starts(int n_comp, const int32_t* gbase, const int64_t* first,
                                 const int64_t* off, int64_t* start, int64_t* vstart,
                                 hipStream_t st) {
  k_comp_tp_starts<<<(unsigned)((n_comp + 1 + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      n_comp, gbase, first, off, start, vstart);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// prime paths grouped by last vertex (the paper's per-end-vertex output)
// ---------------------------------------------------------------------------
// A stable counting sort of the canonical list by last vertex: per tile of
// kGroupTile paths a histogram over the keys, an exclusive scan of the
// histograms taken key-major (so each key's slots run tile after tile),
// then each path's slot = its key's base in its tile + the number of
// earlier paths of the tile with the same key.
__global__ __launch_bounds__(kBlock) void k_last_hist(const int64_t* off, const int32_t* vtx,
                                                      int64_t n, int64_t ntiles, int32_t* key,
                                                      unsigned long long* hist) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int32_t k = vtx[off[i + 1] - 1];
  key[i] = k;
  atomicAdd(&hist[(int64_t)k * ntiles + i / kGroupTile], 1ull);
}

__global__ __launch_bounds__(kGroupTile) void k_last_place(const int32_t* key, int64_t n,
                                                           int64_t ntiles, const int64_t* base,
                                                           int32_t* perm) {
  __shared__ int32_t s_key[kGroupTile];
  const int tid = (int)threadIdx.x;
  const int64_t t = blockIdx.x;
  const int64_t i = t * kGroupTile + tid;
  const int32_t k = i < n ? key[i] : -1;
  s_key[tid] = k;
  __syncthreads();
  if (i >= n) return;
  int r = 0;
  for (int j = 0; j < tid; ++j) r += s_key[j] == k ? 1 : 0;
  perm[base[(int64_t)k * ntiles + t] + r] = (int32_t)i;
}

hipError_t launch_last_hist(const int64_t* off, const int32_t* vtx, int64_t n, int64_t ntiles,
                            int32_t* key, uint64_t* hist, hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_last_hist<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      off, vtx, n, ntiles, key, reinterpret_cast<unsigned long long*>(hist));
  return hipGetLastError();
}

hipError_t launch_last_place(const int32_t* key, int64_t n, int64_t ntiles, const int64_t* base,
                             int32_t* perm, hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_last_place<<<(unsigned)ntiles, kGroupTile, 0, st>>>(key, n, ntiles, base, perm);
  return hipGetLastError();
}

int64_t group_tiles(int64_t n) { return (n + kGroupTile - 1) / kGroupTile; }

// ---------------------------------------------------------------------------
// batched form: packing in caller order
// ---------------------------------------------------------------------------
// One workgroup per chunk of a union's segments: the chunk's segment is the
// last descriptor whose first chunk is at or before it (a segment with no
// chunks shares its first chunk with the next one, which wins the search).
// Fixed-size chunks keep the largest graphs of a batch from leaving one
// workgroup copying long after the others are done.
__global__ __launch_bounds__(kBlock) void k_pack(const int64_t* src_off, const int32_t* src_vtx,
                                                 const PackDesc* d, int32_t n_desc,
                                                 int64_t* dst_off, int32_t* dst_vtx) {
  const int64_t b = blockIdx.x;
  int lo = 0, hi = n_desc - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].chunk0 <= b) lo = mid;
    else hi = mid - 1;
  }
  const PackDesc e = d[lo];
  const int64_t c = b - e.chunk0;
  const int64_t n_oc = (e.n_paths + kPackPaths - 1) / kPackPaths;
  if (c < n_oc) {
    const int64_t j0 = c * kPackPaths, j1 = min(e.n_paths, j0 + kPackPaths);
    const int64_t shift = e.dst_v - e.src_v0;
    for (int64_t j = j0 + threadIdx.x; j < j1; j += kBlock)
      dst_off[e.dst_path + j] = src_off[e.src_path + j] + shift;
  } else {
    const int64_t q0 = (c - n_oc) * kPackVtx, q1 = min(e.n_v, q0 + kPackVtx);
    for (int64_t q = q0 + threadIdx.x; q < q1; q += kBlock)
      dst_vtx[e.dst_v + q] = src_vtx[e.src_v0 + q];
  }
}

hipError_t launch_pack(const int64_t* src_off, const int32_t* src_vtx, const PackDesc* d,
                       int32_t n_desc, int64_t n_chunks, int64_t* dst_off, int32_t* dst_vtx,
                       hipStream_t st) {
  if (n_desc <= 0 || n_chunks <= 0) return hipSuccess;
  if (n_chunks > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  k_pack<<<(unsigned)n_chunks, kBlock, 0, st>>>(src_off, src_vtx, d, n_desc, dst_off, dst_vtx);
  return hipGetLastError();
}

}  // namespace tpg
