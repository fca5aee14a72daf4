// Host-visible declarations of the device structures and kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace tpg {

constexpr int kMaxLevels = 4096 + 4;  // path entries <= n + 1

// Level bookkeeping kept in device memory so that levels can follow each
// other without the host learning their sizes.  The 32-byte header is what
// the host polls.
struct LevelState {
  int32_t batch_start;     // first level that launch 0 of the running batch extends
  int32_t limit;           // the batch leaves levels from this one on alone
  int32_t overflow;        // non-zero: the children of overflow_level did not fit
  int32_t overflow_level;
  int32_t reached;         // first level that the last launch has left to the next
  int32_t pad[3];
  // nodes (paths) per level, cycle closures included; while level L is
  // extended, count[L + 1] is the running claim counter of its tiles
  int64_t count[kMaxLevels];
  int64_t off[kMaxLevels];    // global index of the first node of each level
  int32_t next[kMaxLevels];   // first level that each launch of the batch extends
};
constexpr int kLevelHeader = 32;  // bytes before count
// Levels of at most this many nodes, with at most this many words of visited
// sets, are extended many to a launch.
constexpr int kNarrowExtend = 2048, kNarrowWords = 16384;
__host__ __device__ inline bool narrow_level(int64_t nodes, int set_words) {
  return nodes <= kNarrowExtend && (int)nodes * set_words <= kNarrowWords;
}

// Buffers of the path tree and of the frontier.
struct TreeBufs {
  int32_t* par;       // [rec_cap]
  uint32_t* info;     // [rec_cap]
  int32_t* cstart;    // [rec_cap + 1] global index of the first child
  uint8_t* nch;       // [rec_cap] number of children (<= 64) or leaf kind (nch_code)
  uint16_t* tl;       // [rec_cap] vertices of the node's chains, each chain once
  uint64_t* mask[2];  // visited sets of the odd levels, alternating [mask_cap * mask_words]
  int64_t rec_cap;
  int64_t mask_cap;
  int32_t mask_words;  // words stored per visited set (<= the kernel width W)
  int32_t pad;
};

struct ExtArgs {
  DGraph g;
  TreeBufs t;
  LevelState* ls;
  int64_t tiles_target;  // one-pass tiles per level aimed at (tile size grows above it)
  // level 1: paths <x> for the chains x = seed_lo .. seed_lo + seed_n - 1
  // (node k holds chain seed_lo + k; all chains unless a call streams by
  // first-vertex range)
  int32_t seed_lo, seed_n;
  uint64_t* tot;  // PathTotals of this tree, cleared by the seeding
};

// What the ranking reports of a tree, int64 words: the prime paths, the
// closed cycles, then two histograms of kLenPad + max_comp bins by path
// length (see k_path_lengths), then one uint32 per chain: the cycles closed
// in its tree.
struct PathTotals {
  static constexpr int kPP = 0, kCycles = 1, kHist = 2, kLenPad = 2;
  __host__ __device__ static int64_t bins(const DGraph& g) { return kLenPad + (int64_t)g.max_comp; }
  __host__ __device__ static int64_t host_words(const DGraph& g) { return kHist + 2 * bins(g); }
  __host__ __device__ static int64_t words(const DGraph& g) { return host_words(g) + ((int64_t)g.n + 1) / 2; }
  __host__ __device__ static uint32_t* root_cycles(const DGraph& g, uint64_t* tot) {
    return reinterpret_cast<uint32_t*>(tot + host_words(g));
  }
};

// --- path tree -------------------------------------------------------------
hipError_t launch_seed(const ExtArgs& a, int limit, hipStream_t st);
// items: most parents per thread (tile <= threads * items); variant: 0
// load-balanced tiles of 256 threads, 1 / 2 thread-per-parent with 256 /
// 1024 threads; grid: persistent workgroups; li: index of the launch in its
// batch (it goes on from the level that the launch before it has left)
// e0 / e1 (optional): events recorded at the kernel's own start and end
hipError_t launch_extend(int W, int items, int variant, const ExtArgs& a, int grid, int li,
                         hipStream_t st, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_resume_fix(const ExtArgs& a, int level, hipStream_t st);
// two-pass (plain) form
// prev: first node of level L - 1 (an even level's visited sets are rebuilt
// from its parents' stored sets)
hipError_t launch_count(int W, const ExtArgs& a, int L, int64_t prev, int64_t base, int64_t F,
                        hipStream_t st);
hipError_t launch_fill(int W, const ExtArgs& a, int L, int64_t prev, int64_t base, int64_t F,
                       hipStream_t st);

// --- ranking / materialization ---------------------------------------------
// Lengths of all simple paths behind the nodes [first, n_nodes) (first: the
// level-1 nodes are left to the host) into a.tot's histograms, and the cycles
// closed in every root's tree.
hipError_t launch_path_lengths(const ExtArgs& a, int64_t first, int64_t n_nodes, hipStream_t st);
// sub_cnt: PP leaves per subtree (k_up), then rewritten top-down into the
// output position of the subtree's first PP (0xFFFFFFFF when it has none).
hipError_t launch_up(const ExtArgs& a, int64_t base, int64_t F, uint32_t* sub_cnt, hipStream_t st);
// Consecutive narrow levels that one workgroup sweeps in one launch: nodes
// [off[i], off[i + 1]) are the i-th of them from the top.
constexpr int kSpanLevels = 64;
struct LevelSpan {
  int32_t n;
  uint32_t off[kSpanLevels + 1];
};
// rep null: the PP leaves, else the test-path marks
hipError_t launch_up_span(const ExtArgs& a, const LevelSpan& s, const int32_t* rep,
                          uint32_t* sub_cnt, hipStream_t st);
// rb[v - range_lo] = output position of the first prime path whose first
// vertex is >= v, for the range_n vertices from range_lo (those of the seeded
// chains) and one past them; the roots' positions into sub_cnt; the prime
// paths and the closed cycles into a.tot.  cnt: scratch, range_n entries.
hipError_t launch_roots(const ExtArgs& a, const DChains& ch, int32_t range_lo, int32_t range_n,
                        uint32_t* sub_cnt, int64_t* rb, int32_t* cnt, uint64_t* scan_status,
                        hipStream_t st);
// A prime path's leaf: its node (bits 0-31), the place in its first chain
// where it starts (bits 32-44), and bit 63 when it is a cycle.
constexpr int kLeafStartShift = 32;
constexpr uint64_t kLeafCycle = 1ull << 63;
// What the test paths' order needs of the tree (see k_tp_mark in
// kernels_tp.hip); canon null: not wanted.
struct TpTree {
  int32_t* tpar;        // per chain: the chain before it in the BFS tree (-1: none)
  int32_t* nx;          // per chain: the chain after it on the shortest way to the exit
  int32_t* cdist;       // per chain: vertices before its first on the way from the entry
  int32_t* cback;       // per chain: vertices after its last on the way to the exit
  int32_t *prow, *srow; // per chain: its row among the prefix (suffix) rows
  int32_t* canon;       // per node: the node of its path without the chains before the
                        // last one of its first BFS-tree part (-1: all of it is one)
  int32_t* leaf_canon;  // the same per prime path
};
// parents of a span's levels, L the first of them
hipError_t launch_down_span(const ExtArgs& a, const TpTree& t, int L, const LevelSpan& s,
                            uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st);
// parents of level L: positions to the children; PP leaves record node and length
hipError_t launch_down(const ExtArgs& a, const TpTree& t, int L, int64_t base, int64_t F,
                       uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st);
// the same for two levels in one launch (base, F: the upper one, level L)
hipError_t launch_up_run(const ExtArgs& a, int64_t base, int64_t F, uint32_t* sub_cnt,
                         hipStream_t st);
// both for the test paths' marked nodes instead of the PP leaves
hipError_t launch_tp_up(const ExtArgs& a, int64_t base, int64_t F, const int32_t* rep,
                        uint32_t* cnt, hipStream_t st);
hipError_t launch_tp_up_run(const ExtArgs& a, int64_t base, int64_t F, const int32_t* rep,
                            uint32_t* cnt, hipStream_t st);
hipError_t launch_down_run(const ExtArgs& a, const TpTree& t, int L, int64_t base, int64_t F,
                           uint32_t* sub_cnt, uint64_t* leaf, int32_t* pp_len, hipStream_t st);
// the prime paths that start inside the n_rot chains rot[] (see k_rotations)
hipError_t launch_rotations(const ExtArgs& a, const DChains& ch, const TpTree& t,
                            const int32_t* rot, int32_t n_rot, int32_t range_lo, const int64_t* rb,
                            uint64_t* leaf, int32_t* pp_len, hipStream_t st);
// n: vertices of the union
hipError_t launch_pp_write(const ExtArgs& a, const DChains& ch, int32_t n, const uint64_t* leaf,
                           const int64_t* pp_off, int64_t n_pp, int32_t* pp_vtx, hipStream_t st);

// --- scans -------------------------------------------------------------------
// out[i] = add + sum(in[0..i)), *total = add + sum(in); n may be 0.
hipError_t scan_i32_to_i32(const int32_t* in, int32_t* out, int64_t n, int64_t add,
                           int64_t* total, uint64_t* status, uint32_t* ctr, hipStream_t st);
hipError_t scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, int64_t add,
                           int64_t* total, uint64_t* status, uint32_t* ctr, hipStream_t st);
hipError_t scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t add, int64_t* total,
                    uint64_t* status, uint32_t* ctr, hipStream_t st);
int64_t scan_tiles(int64_t n);  // status slots needed by the scans for n items

hipError_t launch_zero_u64(uint64_t* p, int64_t n, hipStream_t st);
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st);

// --- strongly connected components and prime-path types (Sec. 2) ----------
// per-vertex flags (Defs. 4-5) and path types (Defs. 2, 9, 10, 11); the values
// are the ones the C API exports
constexpr uint8_t kSccCyclic = 1, kSccEntryVertex = 2, kSccExitVertex = 4;
constexpr uint8_t kPpComplete = 1, kPpSccInternal = 2, kPpSccExit = 3, kPpSccEntry = 4,
                  kPpOther = 5;
constexpr int kPpTypes = 6;  // counts are indexed by type (index 0 unused)
// comp[v] = smallest vertex of v's component, flags[v], n_comp[0] = number of
// components; x, ch: the graph of its chains (empty: not at hand); m: arcs of the
// union; work: 6 n int32 of scratch
hipError_t launch_scc(const DGraph& g, const DGraph& x, const DChains& ch, int32_t m,
                      int32_t* work, int32_t* comp, uint8_t* flags, int32_t* n_comp,
                      hipStream_t st);
// --- the paper's per-vertex schedule (comparison variant) ------------------
hipError_t launch_pv_init(int n, int64_t* voff, int32_t* rows, hipStream_t st);
hipError_t launch_pv_count(const DGraph& g, int L, const int64_t* voff, const int32_t* rows,
                           int32_t* cnt, hipStream_t st);
hipError_t launch_pv_fill(const DGraph& g, int L, const int64_t* voff, const int32_t* rows,
                          uint8_t* extended, const int64_t* nvoff, int32_t* nrows,
                          hipStream_t st);
hipError_t launch_pv_prime(const DGraph& g, int L, const int32_t* rows, const uint8_t* extended,
                           int64_t n_rows, int32_t* flag, hipStream_t st);
hipError_t launch_pv_emit(int L, const int32_t* rows, const int32_t* flag, const int64_t* pos,
                          int64_t n_rows, int64_t base, int64_t voff0, int64_t* out_off,
                          int32_t* out_vtx, hipStream_t st);
// types[i] (may be null) and counts[0 .. kPpTypes) of a prime-path set
// --- compositional method (Sec. 2.1): component graph, extraction, merge ---
hipError_t launch_ccfg_count(const DGraph& g, const int32_t* comp, int32_t* cnt, hipStream_t st);
hipError_t launch_ccfg_write(const DGraph& g, const int32_t* comp, const int64_t* off, int32_t* src,
                             int32_t* dst, hipStream_t st);
// mode 0: forward tree of the components (set 0 entry-exit paths, set 1 entry
// paths); mode 1: tree of the reversed components (set 0 exit paths)
hipError_t launch_ex_up(const ExtArgs& a, int64_t base, int64_t F, const uint8_t* vfl, int mode,
                        uint8_t* qb, uint32_t* cnt0, uint32_t* cnt1, hipStream_t st);
// the same for the levels of a span (L: its first)
hipError_t launch_ex_up_span(const ExtArgs& a, const LevelSpan& s, const uint8_t* vfl, int mode,
                             uint8_t* qb, uint32_t* cnt0, uint32_t* cnt1, hipStream_t st);
hipError_t launch_ex_down_span(const ExtArgs& a, int L, const LevelSpan& s, const uint8_t* qb,
                               uint32_t* cnt, int mode, int set, int64_t* out_node,
                               int32_t* out_len, hipStream_t st);
hipError_t launch_ex_roots(uint32_t* cnt, int64_t n_roots, int64_t* total, hipStream_t st);
hipError_t launch_ex_down(const ExtArgs& a, int L, int64_t base, int64_t F, const uint8_t* qb,
                          uint32_t* cnt, int mode, int set, int64_t* out_node, int32_t* out_len,
                          hipStream_t st);
hipError_t launch_ex_write(const ExtArgs& a, const int64_t* out_node, const int64_t* off,
                           int64_t n, int reversed, const int32_t* orig, int32_t* vtx,
                           hipStream_t st);
hipError_t launch_merge_class(const int64_t* off, const int32_t* vtx, int64_t n,
                              const uint8_t* hkind, const int32_t* horig, const DGraph& g,
                              int h_entry, int h_exit, uint8_t* cls, int32_t* len, hipStream_t st);
hipError_t launch_internal_class(const int64_t* off, const int32_t* vtx, int64_t n,
                                 const uint8_t* vfl, uint8_t* cls, int32_t* len, hipStream_t st);
hipError_t launch_merge_sel(const uint8_t* cls, const int32_t* len, int64_t n, int c, int32_t* flag,
                            int32_t* lens, hipStream_t st);
hipError_t launch_merge_emit(const int64_t* off, const int32_t* vtx, int64_t n, const uint8_t* cls,
                             int c, const int64_t* pos, const int64_t* voff, const int32_t* len,
                             const int32_t* horig, int64_t* out_off, int32_t* out_vtx,
                             hipStream_t st);
hipError_t launch_pp_types(const DGraph& g, const int32_t* comp, const uint8_t* flags,
                           const int64_t* off, const int32_t* vtx, int64_t n_pp, uint8_t* types,
                           unsigned long long* counts, hipStream_t st);
// --- prime paths grouped by last vertex (stable counting sort) ---------------
constexpr int kGroupTile = 1024;
constexpr int kGroupKeyBits = 13;  // keys below 2^13, ranks in a tile above them
int64_t group_tiles(int64_t n);
// key_rank[i] = last vertex of path i and the number of its tile's earlier paths
// with the same one; hist[key * ntiles + tile] their counts (n_keys * ntiles)
hipError_t launch_last_rank(const int64_t* off, const int32_t* vtx, int64_t n, int64_t ntiles,
                            int n_keys, uint32_t* key_rank, uint64_t* hist, hipStream_t st);
// perm[slot] = path index and len[slot] its entries, slot = base[key * ntiles +
// tile] + rank (base: exclusive scan of hist)
hipError_t launch_last_place(const uint32_t* key_rank, int64_t n, int64_t ntiles,
                             const int64_t* base, const int64_t* off, int32_t* perm, int32_t* len,
                             hipStream_t st);
struct EndRows;
// --- test paths by longest-first covering (kernels_cover.hip) ----------------
// Hash table of the prime paths (keys / vals of mask + 1 slots, keys zeroed);
// dups counts hashes shared by two prime paths (then retry with another mul).
uint64_t cover_hash_mul(int attempt);
hipError_t launch_pp_hash_insert(const int64_t* off, const int32_t* vtx, int64_t n, uint64_t mul,
                                 uint64_t* keys, int32_t* vals, int64_t mask, uint64_t* dups,
                                 hipStream_t st);
// Pairs (p, q) of prime paths (at most cap of them written, all counted): q is
// contained in the test path that b's rows make of p and comes after p in the
// order of decreasing length, then of index; missing counts accepted windows
// absent from the table (never, unless the input is bad).  One graph of n
// vertices, np prime paths.
hipError_t launch_cover(const DGraph& g, int n, const int64_t* pp_off, const int32_t* pp_vtx,
                        int64_t np, const EndRows& b, uint64_t mul, const uint64_t* keys,
                        const int32_t* vals, int64_t mask, int32_t* pair_p, int32_t* pair_q,
                        int64_t cap, uint64_t* count, uint64_t* missing, int num_cus,
                        hipStream_t st);
// A round of the covering decision: pass over the pairs (drop / block
// flags, state read only), then decide every undecided path (state 0 ->
// 1 chosen, 2 dropped) and add the ones left to *undecided (may be null).
hipError_t launch_round_pairs(const int32_t* pair_p, const int32_t* pair_q, int64_t np,
                              const uint8_t* state, uint8_t* drop, uint8_t* block,
                              hipStream_t st);
hipError_t launch_round_decide(int64_t n, uint8_t* state, uint8_t* drop, uint8_t* block,
                               uint64_t* undecided, hipStream_t st);
// Set digest of paths [0, n) (offsets off, entries vtx): out[0] = sum and
// out[1] = xor of the per-path FNV-1a 64 hashes of (k, v_1 .. v_k) as int32
// little-endian bytes; out is cleared first.
hipError_t launch_digest(const int64_t* off, const int32_t* vtx, int64_t n, uint64_t* out,
                         hipStream_t st);
hipError_t launch_zero_u32(uint32_t* p, int64_t n, hipStream_t st);

// --- test paths --------------------------------------------------------------
// Prefix and suffix of every vertex: n_pfx[v] entries from pfx[pfx_at[v]],
// n_sfx[v] entries from sfx[sfx_at[v]] (see k_chain_rows).
struct EndRows {
  int32_t *n_pfx, *n_sfx, *pfx_at, *sfx_at;  // [n]
  int32_t *pfx, *sfx;
};
// The BFS tree over the chains into t, the arcs' test-path order (gbase[c]:
// the components' first places, c = 0 .. n_comp), and b's rows (pbase[c],
// sbase[c]: the components' first entries).  max_chains, max_words: chains, and words of
// sp, s, pp, p and len, of the largest component.
constexpr int kArcSlotBits = 6;  // a successor slot; chain ids take 17 bits
hipError_t launch_chain_bfs(const DGraph& g, const DGraph& x, const DChains& ch, const TpTree& t,
                            const int32_t* gbase, int32_t* order, const int32_t* pbase,
                            const int32_t* sbase, const EndRows& b, int max_chains, int max_words,
                            hipStream_t st);
// per-component output starts: pp_start[c] = rank of the first PP of c and
// ppv_start[c] = offset of its first entry (after the PP offsets exist; rb:
// see launch_roots, over all vertices; c = n_comp: the totals)
hipError_t launch_comp_pp_starts(const DGraph& g, const int64_t* rb, const int64_t* pp_off,
                                 int64_t* pp_start, int64_t* ppv_start, hipStream_t st);

// rep[node] = prime path + 1 for the node of every test path (state: see
// k_tp_mark); rep must be zero
hipError_t launch_tp_mark(const ExtArgs& a, const TpTree& t, const uint64_t* leaf, int64_t n_pp,
                          const uint8_t* state, int32_t* rep, hipStream_t st);
// cnt: marked nodes per subtree (launch_tp_up*), rewritten into places (see
// k_tp_arc_starts) for the n arcs of order; src[place] = prime path, len[place]
// = entries of the test path (0 for the places from their number up to `room`);
// their number also into *n_out.  num: scratch, n entries
hipError_t launch_tp_arc_starts(const ExtArgs& a, const TpTree& tt, const int32_t* order, int32_t n,
                                const int32_t* rep, uint32_t* cnt, int64_t* first, int32_t* src,
                                int32_t* len, int64_t room, int64_t* n_out, int32_t* num,
                                uint64_t* scan_status, hipStream_t st);
// places from the nodes of a span's levels down
hipError_t launch_tp_down_span(const ExtArgs& a, const TpTree& tt, const LevelSpan& s,
                               const int32_t* rep, uint32_t* cnt, int32_t* src, int32_t* len,
                               hipStream_t st);
// places from the nodes of a level down through the next one
hipError_t launch_tp_down_run(const ExtArgs& a, const TpTree& tt, int64_t base, int64_t F,
                              const int32_t* rep, uint32_t* cnt, int32_t* src, int32_t* len,
                              hipStream_t st);
// rows r < n, each prime path src[r], with b between its prefix and suffix rows,
// at out_off (n_entries in all; n_dev: where the number of rows is, at most n, if
// the host does not know it yet)
hipError_t launch_emit_rows(const int32_t* src, int64_t n, int64_t n_entries, const int64_t* pp_off,
                            const int32_t* pp_vtx, const EndRows* b, const int64_t* out_off,
                            int32_t* out_vtx, hipStream_t st, const int64_t* n_dev = nullptr);
// the n rows at off (off[n]: their entries, at most n_entries) and their offsets,
// both arrays 16-byte aligned
hipError_t launch_copy_rows(const int64_t* off, const int32_t* vtx, int64_t n, int64_t n_entries,
                            int64_t* out_off, int32_t* out_vtx, hipStream_t st);
// start[c] / vstart[c] (c = 0 .. n_comp) of the test paths
hipError_t launch_comp_tp_starts(int n_comp, const int32_t* gbase, const int64_t* first,
                                 const int64_t* off, int64_t* start, int64_t* vstart,
                                 hipStream_t st);
hipError_t launch_set_i64(int64_t* p, const int64_t* src, hipStream_t st);
hipError_t launch_set_value_i64(int64_t* p, int64_t value, hipStream_t st);

// --- batched form --------------------------------------------------------------
// One graph's segment of a union's output, where it goes in the packed
// output (caller order), and the first of its copy chunks in the launch
// (its offsets in chunks of kPackPaths, then its entries in chunks of
// kPackVtx).
constexpr int kPackPaths = 1024;
constexpr int kPackVtx = 4096;
struct PackDesc {
  int64_t src_path, n_paths, src_v0, n_v;
  int64_t dst_path, dst_v;
  int64_t chunk0;
  int64_t base;  // the graph's first vertex id in the union
};
inline int64_t pack_chunks(const PackDesc& e) {
  return (e.n_paths + kPackPaths - 1) / kPackPaths + (e.n_v + kPackVtx - 1) / kPackVtx;
}
// copies the segments d[0 .. n_desc) of one union (chunk0 ascending from 0;
// n_chunks in all): one workgroup per chunk
hipError_t launch_pack(const int64_t* src_off, const int32_t* src_vtx, const PackDesc* d,
                       int32_t n_desc, int64_t n_chunks, int64_t* dst_off, int32_t* dst_vtx,
                       hipStream_t st);
// lvl_comp[c * 64 + min(L, 64) - 1] += simple paths of L entries in component
// c, over the tree's n_nodes nodes
hipError_t launch_level_comp_counts(const ExtArgs& a, int64_t n_nodes, int64_t* lvl_comp,
                                    hipStream_t st);

}  // namespace tpg
