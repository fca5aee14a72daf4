// Test-path kernels: shortest paths from the entry and to the exit, the test
// paths' order and duplicates read off the path tree, and their rows.
//
// A test path extends a prime path to the initial and final nodes (paper
// Sec. 7.3, the Ammann-Offutt construction; Problem 1 asks for test paths
// covering every prime path).  The shortest connection is taken, and among
// shortest ones the lexicographically smallest, so the result is unique:
//  * prefix(v): smallest shortest entry -> v path; suffix(v): smallest shortest
//    v -> exit path.  Both are made of whole chains, so they are found on the
//    graph of chains (k_chain_bfs).
//  * TP(p) = prefix(v1) without v1 ++ p ++ suffix(vk) without vk.
//
// Order and duplicates are read off the path tree; no test path is compared
// with another (see k_tp_mark).  Every distinct test path owns one node of
// the tree, two subtree sweeps like the prime paths' give the nodes' places
// in lexicographic order, and the rows are written where they belong.

#include "kernels.h"

namespace tpg {

constexpr int kMaxComp = 4096;  // vertices per component

// Shortest paths from the entry and to the exit over one component's chains,
// the BFS tree (every chain's predecessor on its lexicographically smallest
// shortest path, the one a first-in first-out search with ascending
// successors finds) and the test-path order of the arcs off it.  One workgroup
// per component, everything in LDS.  No step walks a chain's ancestors or all
// arcs once per level, so a deep graph (early exits: 1000 vertices, 1000
// levels) costs a barrier per level and not a pass over the graph:
//  * distances by relaxing the arcs of the chains whose distance fell in the
//    round before (a bit per chain), both ways in the same rounds; a chain of
//    more than kBusy predecessors is a wave's;
//  * where several predecessors are on shortest paths, the two paths are
//    compared by walking them up, the longer one first, to the chain they
//    share: the smaller chain after it decides.  The walk uses the tree as
//    found so far, so it is repeated until no choice changes.  Two walks
//    mostly meet after a few chains; where they do not, or the choices do not
//    settle, one thread searches depth-first along the shortest
//    paths' arcs, successors ascending, which meets every chain first on its
//    smallest shortest path;
//  * subtree sizes, preorder ranks (children ascending) and the arcs that end
//    the subtrees along last children, by doubling the distance over which
//    they are summed;
//  * the arcs' order.  An arc (W, Y) off the tree comes right before W's first
//    tree child above Y (rank s), or at the end of W's subtree; among arcs at
//    one rank those that end a subtree come first, deepest first, then W's own
//    before child s in the order of Y; the exit's path comes last at the exit's
//    rank.  order[gbase[c] ..) lists the arcs as W << kArcSlotBits | slot of Y
//    among W's successors, and the exit's chain X as ~X.
// Bound by the LDS latencies of the rounds, a few hundred ns each: 51 us for
// 212 vertices (98 chains), 82 for 1000 (174 chains), 1.06 ms for 1000 early
// exits.  A search by vertices, one queue layer after the other, took 0.26 and
// 2.5 ms for the first two; relaxing all arcs in every round, and walking up and
// down the tree for the sums, 68 us, 129 us and 98 ms, and 0.85 ms for a switch of
// 30 switches of 30 (0.06 now).
constexpr int kBusy = 64;
template <int MAXC, int NT, bool STAGE>
__global__ __launch_bounds__(NT) void k_chain_bfs(DGraph g, DGraph x, DChains ch, TpTree t,
                                                  const int32_t* gbase, int32_t* order,
                                                  const int32_t* pbase, const int32_t* sbase) {
  constexpr int Q = (MAXC + NT - 1) / NT;  // chains per thread: tid, tid + NT, ..
  constexpr int kWords = MAXC / 32;
  __shared__ int32_t s_d[MAXC + 1];  // distance before the chain; later arcs along last children, arcs per rank
  __shared__ int32_t s_b[MAXC + 1];  // distance after it; later subtree sizes, arcs that end one
  __shared__ int16_t s_par[MAXC];
  __shared__ int16_t s_pre[MAXC];    // busy chains; later a step of the doublings, preorder ranks
  __shared__ int16_t s_pend[MAXC];   // sibling sums; later ranks past the subtrees
  __shared__ uint32_t s_f[3][2][kWords];  // chains to relax, from the entry and to the exit
  __shared__ int64_t s_w[NT / 64];
  __shared__ int32_t s_nb[3], s_nbusy;
  extern __shared__ int32_t s_g[];  // STAGE: the component's sp, s, pp, p, len
  constexpr int kFar = 1 << 29;
  const int c = (int)blockIdx.x, tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int x0 = x.cbase[c], n = x.cbase[c + 1] - x0;
  const int e0 = x.sp[x0], m = x.sp[x0 + n] - e0, f0 = x.pp[x0];
  int32_t* const l_sp = s_g;
  int32_t* const l_s = l_sp + n + 1;
  int32_t* const l_pp = l_s + m;
  int32_t* const l_p = l_pp + n + 1;
  int32_t* const l_len = l_p + m;
  if constexpr (STAGE) {
    for (int i = tid; i <= n; i += NT) {
      l_sp[i] = x.sp[x0 + i] - e0;
      l_pp[i] = x.pp[x0 + i] - f0;
    }
    for (int i = tid; i < m; i += NT) {
      l_s[i] = x.s[e0 + i] - x0;
      l_p[i] = x.p[f0 + i] - x0;
    }
    for (int i = tid; i < n; i += NT) l_len[i] = x.len[x0 + i];
  }
  // local ids and arc indices throughout
  auto sp = [&](int i) { return STAGE ? l_sp[i] : x.sp[x0 + i] - e0; };
  auto succ = [&](int k) { return STAGE ? l_s[k] : x.s[e0 + k] - x0; };
  auto pp = [&](int i) { return STAGE ? l_pp[i] : x.pp[x0 + i] - f0; };
  auto pred = [&](int k) { return STAGE ? l_p[k] : x.p[f0 + k] - x0; };
  auto len = [&](int i) { return STAGE ? l_len[i] : x.len[x0 + i]; };
  const int en = ch.of[g.centry[c]] - x0, ex = ch.of[g.cexit[c]] - x0;
  for (int i = tid; i < n; i += NT) {
    s_d[i] = i == en ? 0 : kFar;
    s_b[i] = i == ex ? 0 : kFar;
  }
  for (int i = tid; i < 6 * kWords; i += NT) (&s_f[0][0][0])[i] = 0;
  if (tid == 0) s_nb[0] = s_nb[1] = s_nb[2] = s_nbusy = 0;
  __syncthreads();
  if (tid == 0) {
    s_f[0][0][en >> 5] = 1u << (en & 31);
    s_f[0][1][ex >> 5] = 1u << (ex & 31);
  }
  __syncthreads();
  int more, any;
  for (int cur = 0;;) {
    const int nxt = cur == 2 ? 0 : cur + 1, old = cur == 0 ? 2 : cur - 1;
    for (int i = tid; i < 2 * kWords; i += NT) (&s_f[old][0][0])[i] = 0;
    if (tid == 0) s_nb[nxt] = 0;  // read two rounds ago
    more = 0;
    // chain y is d away over an arc
    auto relax = [&](int dir, int y, int d) {
      if (atomicMin(dir ? &s_b[y] : &s_d[y], d) > d) {
        atomicOr(&s_f[nxt][dir][y >> 5], 1u << (y & 31));
        more = 1;
      }
    };
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      if (i >= n) break;
      if (s_f[cur][0][i >> 5] >> (i & 31) & 1) {
        const int d = s_d[i] + len(i), k1 = sp(i + 1);
        for (int k = sp(i); k < k1; ++k) relax(0, succ(k), d);
      }
      if (s_f[cur][1][i >> 5] >> (i & 31) & 1) {
        const int b = s_b[i] + len(i), k0 = pp(i), k1 = pp(i + 1);
        if (k1 - k0 > kBusy) {
          s_pre[atomicAdd(&s_nb[cur], 1)] = (int16_t)i;
          more = 1;
        } else {
          for (int k = k0; k < k1; ++k) relax(1, pred(k), b);
        }
      }
    }
    any = __syncthreads_or(more);
    const int nb = s_nb[cur];
    if (nb) {
      for (int j = wave; j < nb; j += NT / 64) {
        const int i = s_pre[j], b = s_b[i] + len(i), k1 = pp(i + 1);
        for (int k = pp(i) + lane; k < k1; k += 64) relax(1, pred(k), b);
      }
      __syncthreads();
    }
    if (!any) break;
    cur = nxt;
  }
  // a predecessor on a shortest path (the first), the next chain to the exit
  auto tight = [&](int p, int i) { return s_d[p] + len(p) == s_d[i]; };
  for (int i = tid; i < n; i += NT) {
    int par = -1, nx = -1;
    const int k0 = pp(i), k1 = pp(i + 1);
    if (k1 - k0 > kBusy) {
      s_pre[atomicAdd(&s_nbusy, 1)] = (int16_t)i;
    } else {
      for (int k = k0; k < k1 && par < 0; ++k)
        if (tight(pred(k), i)) par = pred(k);
    }
    for (int k = sp(i); k < sp(i + 1) && nx < 0; ++k)
      if (s_b[succ(k)] + len(succ(k)) == s_b[i]) nx = succ(k);
    if (i == en) par = -1;
    if (i == ex) nx = -1;
    s_par[i] = (int16_t)par;
    t.nx[x0 + i] = nx < 0 ? -1 : x0 + nx;
    t.cdist[x0 + i] = s_d[i];
    t.cback[x0 + i] = s_b[i];
  }
  __syncthreads();
  // the chains' rows one after another, prefixes in the low half of the sums
  int64_t at = (int64_t)sbase[c] << 32 | pbase[c];
  for (int k0 = 0; k0 < n; k0 += NT) {
    const int i = k0 + tid;
    const int64_t v = i < n ? (int64_t)(s_b[i] + len(i)) << 32 | (s_d[i] + len(i)) : 0;
    int64_t tot;
    const int64_t to = at + block_excl_scan<NT, int64_t>(v, tot, s_w);
    if (i < n) {
      t.prow[x0 + i] = (int32_t)to;
      t.srow[x0 + i] = (int32_t)(to >> 32);
    }
    at += tot;
  }
  const int nbusy = s_nbusy;
  for (int j = wave; j < nbusy; j += NT / 64) {
    const int i = s_pre[j], k1 = pp(i + 1);
    for (int k0 = pp(i); k0 < k1; k0 += 64) {
      const int p = k0 + lane < k1 ? pred(k0 + lane) : -1;
      const uint64_t on = __ballot(p >= 0 && tight(p, i));
      if (!on) continue;
      if (lane == 0) s_par[i] = (int16_t)pred(k0 + __builtin_ctzll(on));
      break;
    }
  }
  __syncthreads();
  // whether the tree path to a's end precedes the equally long one to b's;
  // every step up shortens a path, whatever the tree holds so far
  int steps = 0;
  auto before = [&](int a, int b) {
    int ca = a, cb = b;
    while (a != b && a >= 0 && b >= 0) {
      const int da = s_d[a], db = s_d[b];
      if (da >= db) {
        ca = a;
        a = s_par[a];
      }
      if (db >= da) {
        cb = b;
        b = s_par[b];
      }
      ++steps;
    }
    return ca < cb;
  };
  // steps of a thread's walks before the search takes over, which needs about
  // as many for n chains
  const int walks = 4 * n + 256;
  bool over = false;
  auto chosen = [&](int i, int best) {
    if (best != s_par[i]) {
      s_par[i] = (int16_t)best;
      more = 1;
    }
  };
  for (int round = 0;; ++round) {
    more = 0;
    for (int i = tid; i < n && steps <= walks; i += NT) {
      const int k0 = pp(i), k1 = pp(i + 1);
      if (i == en || k1 - k0 > kBusy) continue;
      int best = -1;
      for (int k = k0; k < k1 && steps <= walks; ++k) {
        const int p = pred(k);
        if (tight(p, i) && (best < 0 || before(p, best))) best = p;
      }
      chosen(i, best);
    }
    for (int j = wave; j < nbusy; j += NT / 64) {
      const int i = s_pre[j], k1 = pp(i + 1);
      int best = -1;
      for (int k = pp(i) + lane; k < k1 && steps <= walks; k += 64) {
        const int p = pred(k);
        if (tight(p, i) && (best < 0 || before(p, best))) best = p;
      }
      for (int d = 32; d >= 1; d >>= 1) {
        const int o = __shfl_xor(best, d, 64);
        if (o >= 0 && (best < 0 || before(o, best))) best = o;
      }
      if (lane == 0) chosen(i, best);
    }
    any = __syncthreads_or(more);
    over = __syncthreads_or(steps > walks || (more && round == 16));
    if (!any || over) break;
  }
  if (over) {
    for (int i = tid; i < n; i += NT) {
      s_pre[i] = i == en;  // seen
      s_pend[i] = 0;       // arcs looked at
    }
    __syncthreads();
    if (tid == 0) {
      for (int u = en; u >= 0;) {
        const int k = sp(u) + s_pend[u];
        if (k == sp(u + 1)) {
          u = s_par[u];
          continue;
        }
        ++s_pend[u];
        const int y = succ(k);
        if (s_pre[y] || !tight(u, y)) continue;
        s_pre[y] = 1;
        s_par[y] = (int16_t)u;
        u = y;
      }
    }
    __syncthreads();
  }
  for (int i = tid; i < n; i += NT) t.tpar[x0 + i] = s_par[i] < 0 ? -1 : x0 + s_par[i];
  // One step of a doubling: link (2^k steps up or down) goes on to its link's
  // link, and `add` gets the sum held where it led.
  auto tree_arc = [&](int w, int k) { return s_par[succ(k)] == w; };
  for (int i = tid; i < n; i += NT) {
    s_b[i] = 1;
    s_pre[i] = s_par[i];
  }
  __syncthreads();
  // subtree sizes: s_b[i] of the descendants less than 2^k below
  do {
    int16_t up[Q], on[Q];
    int32_t v[Q];
    more = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      up[q] = i < n ? s_pre[i] : (int16_t)-1;
      v[q] = i < n ? s_b[i] : 0;
      on[q] = up[q] >= 0 ? s_pre[up[q]] : (int16_t)-1;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (up[q] < 0) continue;
      atomicAdd(&s_b[up[q]], v[q]);
      s_pre[tid + q * NT] = on[q];
      more |= on[q] >= 0;
    }
  } while (__syncthreads_or(more));
  // per chain: its tree children's sibling sums, its last tree child (s_pre),
  // the arcs after it (s_d)
  int32_t tail[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int w = tid + q * NT;
    tail[q] = 0;
    if (w >= n) continue;
    int last = -1, sum = 1;
    for (int k = sp(w); k < sp(w + 1); ++k) {
      ++tail[q];
      if (!tree_arc(w, k)) continue;
      tail[q] = 0;
      last = succ(k);
      s_pend[last] = (int16_t)sum;
      sum += s_b[last];
    }
    if (w == en) s_pend[w] = 0;
    s_pre[w] = (int16_t)last;
    s_d[w] = tail[q];
  }
  __syncthreads();
  // arcs that end the subtrees along the last tree children below w
  do {
    int16_t on[Q];
    int32_t v[Q];
    more = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      const int l = i < n ? s_pre[i] : -1;
      v[q] = l >= 0 ? s_d[l] : 0;
      on[q] = l >= 0 ? s_pre[l] : (int16_t)-1;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      if (i >= n) continue;
      s_d[i] += v[q];
      s_pre[i] = on[q];
      more |= on[q] >= 0;
    }
  } while (__syncthreads_or(more));
  int32_t deeper[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = tid + q * NT;
    deeper[q] = i < n ? s_d[i] - tail[q] : 0;
    if (i < n) s_pre[i] = s_par[i];
  }
  __syncthreads();
  // preorder ranks: sibling sums along the way up
  do {
    int16_t on[Q], v[Q];
    more = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      const int u = i < n ? s_pre[i] : -1;
      v[q] = u >= 0 ? s_pend[u] : (int16_t)0;
      on[q] = u >= 0 ? s_pre[u] : (int16_t)-1;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = tid + q * NT;
      if (i >= n) continue;
      s_pend[i] += v[q];
      s_pre[i] = on[q];
      more |= on[q] >= 0;
    }
  } while (__syncthreads_or(more));
  for (int i = tid; i < n; i += NT) {
    s_pre[i] = s_pend[i];
    s_pend[i] = (int16_t)(s_pend[i] + s_b[i]);
  }
  __syncthreads();
  int32_t* s_at = s_d;   // arcs per rank, then their first place
  int32_t* s_end = s_b;  // of them, arcs that end a subtree
  for (int i = tid; i <= n; i += NT) {
    s_at[i] = 0;
    s_end[i] = 0;
  }
  __syncthreads();
  // w's arcs off the tree in runs [k, j) of one rank
  auto runs = [&](int w, auto&& f) {
    const int k1 = sp(w + 1);
    for (int k = sp(w); k < k1;) {
      int j = k;
      while (j < k1 && !tree_arc(w, j)) ++j;
      if (j > k) f(k, j, j == k1, j == k1 ? (int)s_pend[w] : (int)s_pre[succ(j)]);
      k = j + 1;
    }
  };
  for (int w = tid; w < n; w += NT) {
    runs(w, [&](int k, int j, bool ends, int r) {
      atomicAdd(&s_at[r], j - k);
      if (ends) atomicAdd(&s_end[r], j - k);
    });
    if (w == ex) atomicAdd(&s_at[s_pre[w]], 1);
  }
  __syncthreads();
  int carry = gbase[c];
  for (int k0 = 0; k0 <= n; k0 += NT) {
    const int k = k0 + tid;
    const int v = k <= n ? s_at[k] : 0;
    int64_t tot;
    const int pre = (int)block_excl_scan<NT, int64_t>(v, tot, s_w);
    if (k <= n) s_at[k] = carry + pre;
    carry += (int)tot;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int w = tid + q * NT;
    if (w >= n) continue;
    runs(w, [&](int k, int j, bool ends, int r) {
      int at = s_at[r] + (ends ? deeper[q] : s_end[r]);
      for (int i = k; i < j; ++i) order[at++] = (x0 + w) << kArcSlotBits | (i - sp(w));
    });
    if (w == ex) {
      const int r = s_pre[w];
      order[(r < n ? s_at[r + 1] : carry) - 1] = ~(x0 + w);
    }
  }
}

// The rows that the prefixes and suffixes are cut from, one wave per chain x:
// the way to x and x itself, x and the way on from it.  Then per vertex of x
// where its prefix and suffix are and how long.
__global__ __launch_bounds__(64) void k_chain_rows(DChains ch, TpTree t, EndRows b) {
  const int c0 = (int)blockIdx.x, lane = lane_id();
  const int pat = t.prow[c0], sat = t.srow[c0];
  const int o = ch.off[c0], m = ch.off[c0 + 1] - o;
  const int df = t.cdist[c0], db = t.cback[c0];
  // both ways in step
  for (int p = c0, q = c0; p >= 0 || q >= 0;) {
    if (p >= 0) {
      const int po = ch.off[p], pm = ch.off[p + 1] - po, pd = t.cdist[p];
      const int up = t.tpar[p];
      for (int j = lane; j < pm; j += 64) b.pfx[pat + pd + j] = ch.v[po + j];
      p = up;
    }
    if (q >= 0) {
      const int qo = ch.off[q], qm = ch.off[q + 1] - qo, qd = db + m - t.cback[q] - qm;
      const int on = t.nx[q];
      for (int j = lane; j < qm; j += 64) b.sfx[sat + qd + j] = ch.v[qo + j];
      q = on;
    }
  }
  for (int j = lane; j < m; j += 64) {
    const int v = ch.v[o + j];
    b.n_pfx[v] = df + j;
    b.n_sfx[v] = db + m - 1 - j;
    b.pfx_at[v] = pat;
    b.sfx_at[v] = sat + j + 1;
  }
}

hipError_t launch_chain_bfs(const DGraph& g, const DGraph& x, const DChains& ch, const TpTree& t,
                            const int32_t* gbase, int32_t* order, const int32_t* pbase,
                            const int32_t* sbase, const EndRows& b, int max_chains, int max_words,
                            hipStream_t st) {
  const unsigned grid = (unsigned)x.n_comp;
  // staged graphs of up to 16 KiB (40 KiB from 257 chains on, which are seldom
  // many at a time); a wave per component when there are many (18 chains alone
  // take four waves 22 us and one 21)
  const size_t lds = sizeof(int32_t) * (size_t)max_words;
  auto run = [&](auto staged, auto plain, int threads, size_t most) {
    if (lds <= most) staged<<<grid, threads, lds, st>>>(g, x, ch, t, gbase, order, pbase, sbase);
    else plain<<<grid, threads, 0, st>>>(g, x, ch, t, gbase, order, pbase, sbase);
  };
  if (max_chains <= 256 && x.n_comp >= 64)
    run(k_chain_bfs<256, 64, true>, k_chain_bfs<256, 64, false>, 64, 16384);
  else if (max_chains <= 256)
    run(k_chain_bfs<256, 256, true>, k_chain_bfs<256, 256, false>, 256, 16384);
  else if (max_chains <= 1024)
    run(k_chain_bfs<1024, 256, true>, k_chain_bfs<1024, 256, false>, 256, 40960);
  else
    k_chain_bfs<kMaxComp, 1024, false><<<grid, 1024, 0, st>>>(g, x, ch, t, gbase, order, pbase,
                                                              sbase);
  k_chain_rows<<<(unsigned)x.n, 64, 0, st>>>(ch, t, b);
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
//    tree with the other arcs as leaves (k_chain_bfs); the one test path
//    that is a BFS-tree path all along belongs to the exit.
// So the test paths' nodes are marked (k_tp_mark, with a prime path for each),
// counted bottom-up, and given their places top-down.  k_down_run finds, for
// every node with prime paths below it, the node of the path with its
// BFS-tree part dropped, from its parent's.  The test-path stage of the
// 400-vertex stress CFG takes 9.3 ms of a 17.8 ms call (its rows alone are
// 21.8 GB, 7.2 ms); splicing every test path, sorting them by merge rounds that
// compared them and unpacking them took 21 of 30.8.  The same change took a
// batch of 4096 CFGs from 11.1 to 7.6 ms and a 1000-vertex CFG from 6.7 to 4.3
// (5.6 and 2.1 with what has changed elsewhere since).

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

// The node of an arc of the order (the exit's own path: its root).
__device__ __forceinline__ int64_t arc_node(const TreeBufs& t, int32_t g) {
  return g < 0 ? (int64_t)~g
               : (int64_t)t.cstart[g >> kArcSlotBits] + (g & ((1 << kArcSlotBits) - 1));
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
                                                        int32_t* len, const int32_t* cdist,
                                                        int64_t room, int64_t* n_out) {
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
        node[j] = arc_node(t, g);
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
  for (int64_t r = carry + threadIdx.x; r < room; r += 1024) len[r] = 0;
  if (threadIdx.x == 0) {
    first[n] = carry;
    *n_out = carry;
  }
}

// The same for a large union, around a scan over the chip (see k_root_counts):
// 4096 CFGs took one workgroup 97 us a union, about 35 this way.
constexpr int32_t kOneArcs = 2 * 1024 * kArcItems;
__global__ __launch_bounds__(kBlock) void k_arc_counts(TreeBufs t, const int32_t* order, int32_t n,
                                                       const int32_t* rep, const uint32_t* cnt,
                                                       int32_t* out) {
  const int32_t j = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
  if (j >= n) return;
  const int32_t g = order[j];
  const int64_t x = arc_node(t, g);
  out[j] = g < 0 ? (rep[x] != 0 ? 1 : 0) : (int32_t)cnt[x];
}

__global__ __launch_bounds__(kBlock) void k_arc_places(TreeBufs t, const int32_t* order, int32_t n,
                                                       const int32_t* rep, uint32_t* cnt,
                                                       const int32_t* num, const int64_t* first,
                                                       int32_t* src, int32_t* len,
                                                       const int32_t* cdist) {
  const int32_t j = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
  if (j >= n) return;
  const int32_t g = order[j], c = num[j];
  const int64_t x = arc_node(t, g), at = first[j];
  if (g >= 0) {
    cnt[x] = c ? (uint32_t)(at + 1) : 0u;
  } else if (c) {
    src[at] = rep[x] - 1;
    len[at] = cdist[x] + t.tl[x];
  }
}

hipError_t launch_tp_arc_starts(const ExtArgs& a, const TpTree& tt, const int32_t* order, int32_t n,
                                const int32_t* rep, uint32_t* cnt, int64_t* first, int32_t* src,
                                int32_t* len, int64_t room, int64_t* n_out, int32_t* num,
                                uint64_t* scan_status, hipStream_t st) {
  if (n > kOneArcs) {
    const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
    hipError_t e = launch_zero_u32(reinterpret_cast<uint32_t*>(len), room, st);
    if (e != hipSuccess) return e;
    k_arc_counts<<<grid, kBlock, 0, st>>>(a.t, order, n, rep, cnt, num);
    e = hipGetLastError();
    if (e == hipSuccess) e = scan_i32_to_i64(num, first, n, 0, n_out, scan_status, nullptr, st);
    if (e != hipSuccess) return e;
    k_arc_places<<<grid, kBlock, 0, st>>>(a.t, order, n, rep, cnt, num, first, src, len, tt.cdist);
    return hipGetLastError();
  }
  k_tp_arc_starts<<<1, 1024, 0, st>>>(a.t, order, n, rep, cnt, first, src, len, tt.cdist, room,
                                      n_out);
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

// Narrow levels, top to bottom (see k_up_span).
__global__ __launch_bounds__(1024) void k_tp_down_span(ExtArgs a, TpTree tt, LevelSpan s,
                                                       const int32_t* rep, uint32_t* cnt,
                                                       int32_t* src, int32_t* len) {
  for (int l = 0; l < s.n; ++l) {
    const uint32_t end = s.off[l + 1];
    for (uint32_t x = s.off[l] + threadIdx.x; x < end; x += 1024) {
      const uint32_t r = cnt[x];
      if (r) tp_down_node<0>(a, tt, x, r - 1, rep, cnt, src, len);
    }
    __syncthreads();
  }
}

hipError_t launch_tp_down_span(const ExtArgs& a, const TpTree& tt, const LevelSpan& s,
                               const int32_t* rep, uint32_t* cnt, int32_t* src, int32_t* len,
                               hipStream_t st) {
  if (s.n < 1 || s.n > kSpanLevels) return hipErrorInvalidValue;
  k_tp_down_span<<<1, 1024, 0, st>>>(a, tt, s, rep, cnt, src, len);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// rows from prime paths
// ---------------------------------------------------------------------------
// Row r is prime path src[r], with b given between its first vertex's prefix
// row and its last vertex's suffix row.
//
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
__global__ __launch_bounds__(kBlock) void k_emit_rows(const int32_t* src, int64_t n,
                                                      const int64_t* n_dev, int rows,
                                                      const int64_t* pp_off, const int32_t* pp_vtx,
                                                      EndRows b, const int64_t* out_off,
                                                      int32_t* out_vtx) {
  const int lane = lane_id();
  if (n_dev) n = *n_dev < n ? *n_dev : n;
  const int64_t r0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * rows;
  if (r0 >= n) return;
  const int nr = (int)(n - r0 < rows ? n - r0 : rows);
  int64_t out = 0, o0 = 0;
  int lq = 0, lp = 0, ls = 0, p0 = 0, s0 = 0;  // lanes past the last row: empty rows
  if (lane < nr) {
    const int64_t i = src[r0 + lane];
    out = out_off[r0 + lane];
    o0 = pp_off[i];
    lq = (int)(pp_off[i + 1] - o0);
    if constexpr (ENDS) {
      const int v1 = pp_vtx[o0], vk = pp_vtx[o0 + lq - 1];
      lp = b.n_pfx[v1];
      ls = b.n_sfx[vk];
      p0 = b.pfx_at[v1];
      s0 = b.sfx_at[vk];
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
      w.a = b.pfx + get(p0, q);
      w.c = b.sfx + get(s0, q) - (w.np + w.nq);
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

hipError_t launch_emit_rows(const int32_t* src, int64_t n, int64_t n_entries, const int64_t* pp_off,
                            const int32_t* pp_vtx, const EndRows* b, const int64_t* out_off,
                            int32_t* out_vtx, hipStream_t st, const int64_t* n_dev) {
  if (n == 0) return hipSuccess;
  // more rows a wave spread the first loads' cost, fewer keep the chip full:
  // 573 k rows 1.90 ms a call with 16 and 1.95 with 64, 1.9e7 rows 19.2 and 18.8
  const int rows = n >= (int64_t)1 << 20 ? 64 : 16;
  const int64_t waves = (n + rows - 1) / rows;
  const unsigned grid = (unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64));
  // the steps that hold a row of average length, to 5
  const int64_t steps = n_entries / (64 * n) + 1;
#define TPG_EMIT(U, R, E, B)                                                                    \
  k_emit_rows<U, R, E><<<grid, kBlock, 0, st>>>(src, n, n_dev, rows, pp_off, pp_vtx, B, out_off,  \
                                               out_vtx)
  if (b) {
    if (steps <= 1) TPG_EMIT(1, 4, true, *b);
    else if (steps <= 2) TPG_EMIT(2, 4, true, *b);
    else TPG_EMIT(5, 2, true, *b);
  } else {
    if (steps <= 1) TPG_EMIT(1, 4, false, EndRows{});
    else TPG_EMIT(2, 4, false, EndRows{});
  }
#undef TPG_EMIT
  return hipGetLastError();
}

// A set as it is, 16 bytes a lane and step.
__global__ __launch_bounds__(kBlock) void k_copy_rows(const int64_t* off, const int32_t* vtx,
                                                      int64_t n, int64_t* out_off,
                                                      int32_t* out_vtx) {
  const int64_t at = (int64_t)blockIdx.x * kBlock + threadIdx.x, step = (int64_t)gridDim.x * kBlock;
  const int64_t nv = off[n];
  for (int64_t i = at; i <= n; i += step) out_off[i] = off[i];
  const int4* from = reinterpret_cast<const int4*>(vtx);
  int4* to = reinterpret_cast<int4*>(out_vtx);
  for (int64_t i = at; i < nv / 4; i += step) to[i] = from[i];
  if (at < nv % 4) out_vtx[nv / 4 * 4 + at] = vtx[nv / 4 * 4 + at];
}

hipError_t launch_copy_rows(const int64_t* off, const int32_t* vtx, int64_t n, int64_t n_entries,
                            int64_t* out_off, int32_t* out_vtx, hipStream_t st) {
  const int64_t work = std::max(n + 1, n_entries / 4 + 1);
  const int64_t grid = std::min<int64_t>(8192, (work + kBlock - 1) / kBlock);
  k_copy_rows<<<(unsigned)grid, kBlock, 0, st>>>(off, vtx, n, out_off, out_vtx);
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
//
// Histogram and rank come from one pass over the tile: the lanes of a wave that
// share a key find each other by ballots over its bits, and the waves add their
// counts to the tile's histogram in LDS in turn.  With a global atomic per path
// (few keys: a loop's paths mostly end at its exit) and a look back over the
// tile for the rank it was 84 + 18 us for 163841 paths, 6 + 2 this way.
__global__ __launch_bounds__(kGroupTile) void k_last_rank(const int64_t* off, const int32_t* vtx,
                                                          int64_t n, int64_t ntiles, int n_keys,
                                                          int key_bits, uint32_t* key_rank,
                                                          uint64_t* hist) {
  extern __shared__ int32_t s_hist[];
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int64_t t = blockIdx.x, i = t * kGroupTile + tid;
  for (int k = tid; k < n_keys; k += kGroupTile) s_hist[k] = 0;
  const bool in = i < n;
  const int k = in ? vtx[off[i + 1] - 1] : 0;
  uint64_t peers = __ballot(in);
  for (int b = 0; b < key_bits; ++b) {
    const uint64_t m = __ballot(k >> b & 1);
    peers &= k >> b & 1 ? m : ~m;
  }
  const int before = __builtin_popcountll(peers & ((1ull << lane) - 1));
  int first = 0;
  for (int w = 0; w < kGroupTile / 64; ++w) {
    __syncthreads();
    if (w == wave && in && before == 0) {
      first = s_hist[k];
      s_hist[k] = first + __builtin_popcountll(peers);
    }
  }
  __syncthreads();
  first = __shfl(first, in ? __builtin_ctzll(peers) : lane, 64);
  if (in) key_rank[i] = (uint32_t)k | (uint32_t)(first + before) << kGroupKeyBits;
  for (int q = tid; q < n_keys; q += kGroupTile) hist[(int64_t)q * ntiles + t] = (uint64_t)s_hist[q];
}

__global__ __launch_bounds__(kBlock) void k_last_place(const uint32_t* key_rank, int64_t n,
                                                       int64_t ntiles, const int64_t* base,
                                                       const int64_t* off, int32_t* perm,
                                                       int32_t* len) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t kr = key_rank[i];
  const int64_t k = kr & ((1u << kGroupKeyBits) - 1);
  const int64_t at = base[k * ntiles + i / kGroupTile] + (kr >> kGroupKeyBits);
  perm[at] = (int32_t)i;
  len[at] = (int32_t)(off[i + 1] - off[i]);
}

hipError_t launch_last_rank(const int64_t* off, const int32_t* vtx, int64_t n, int64_t ntiles,
                            int n_keys, uint32_t* key_rank, uint64_t* hist, hipStream_t st) {
  if (n_keys < 1 || n_keys > 1 << kGroupKeyBits) return hipErrorInvalidValue;
  if (n == 0) return launch_zero_u64(hist, n_keys, st);
  int bits = 0;
  while (1 << bits < n_keys) ++bits;
  k_last_rank<<<(unsigned)ntiles, kGroupTile, sizeof(int32_t) * (size_t)n_keys, st>>>(
      off, vtx, n, ntiles, n_keys, bits, key_rank, hist);
  return hipGetLastError();
}

hipError_t launch_last_place(const uint32_t* key_rank, int64_t n, int64_t ntiles,
                             const int64_t* base, const int64_t* off, int32_t* perm, int32_t* len,
                             hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_last_place<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, st>>>(key_rank, n, ntiles, base,
                                                                         off, perm, len);
  return hipGetLastError();
}

int64_t group_tiles(int64_t n) { return (n + kGroupTile - 1) / kGroupTile; }

// ---------------------------------------------------------------------------
// batched form: packing in caller order
// ---------------------------------------------------------------------------
// One workgroup per chunk of a union's segments: the chunk's segment is the
// last descriptor whose first chunk is at or before it (a segment with no
// chunks shares its first chunk with the next one, which wins the search).
// Vertices become ids of their graph on the way (in passes of their own before
// it took 380 us of 1030 for 651 MB).  Fixed-size chunks keep the largest graphs of a batch from leaving one
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
      dst_vtx[e.dst_v + q] = src_vtx[e.src_v0 + q] - e.base;
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
