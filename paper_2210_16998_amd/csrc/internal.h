// Internal declarations shared by the host-side sources of libtpg.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/tpg.h"

namespace tpg {

// A graph with its straight lines contracted: a chain v_1 -> .. -> v_m, where
// each v_i (i < m) has v_(i+1) as its only successor and is its only
// predecessor, becomes one vertex.  Chains are numbered by their first vertex
// (the head), ascending; a chain's successors are its last vertex's, its
// predecessors its head's.  What the path kernels make of it:
//  * a simple path that enters a chain goes through it to its end or stops
//    inside it, so every acyclic prime path is made of whole chains;
//  * a closed cycle through a chain of m vertices is one cycle of chains and
//    gives m prime paths, one from each of the chain's vertices.
struct Chains {
  int32_t n = 0;                 // chains
  std::vector<int32_t> off, v;   // vertices of chain x, in order: v[off[x] .. off[x + 1])
  std::vector<int32_t> of, pos;  // per vertex: its chain and its place there
  std::vector<int32_t> sp, s, pp, p;  // contracted CSR and its reverse (rows ascending)
  // Entries of the rows that the test paths' prefixes (suffixes) are cut from:
  // every chain behind the shortest way to it (before the one on to the exit);
  // 0 without an entry and an exit.
  int32_t pfx_entries = 0, sfx_entries = 0;
};

}  // namespace tpg

struct tpg_graph {
  int32_t n = 0;
  int32_t entry = 0, exit = 0;
  uint32_t load_flags = 0;
  int32_t max_out_degree = 0;
  // canonical forward CSR (rows ascending, unique) and reverse CSR
  std::vector<int32_t> succ_ptr, succ;
  std::vector<int32_t> pred_ptr, pred;
  tpg::Chains chains;  // the graph with its straight lines contracted
  uint64_t uid = 0;  // identifies the graph in device caches
  // structural features, computed once on first use
  mutable std::once_flag feat_once;
  mutable float feat[32];
};

namespace tpg {

// Chains of g.  block > 0: a chain holds vertices of one block of `block`
// consecutive ids only (block 1: every vertex is a chain of its own).
Chains contract_chains(const tpg_graph& g, int32_t block);

void set_error(const char* fmt, ...);
tpg_status fail(tpg_status s, const char* fmt, ...);

#define TPG_HIP(call)                                                              \
  do {                                                                             \
    hipError_t e_ = (call);                                                        \
    if (e_ != hipSuccess)                                                          \
      return ::tpg::fail(e_ == hipErrorOutOfMemory ? TPG_ERR_OOM_DEVICE : TPG_ERR_DEVICE, \
                         "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),  \
                         __FILE__, __LINE__);                                      \
  } while (0)

#define TPG_TRY(call)                       \
  do {                                      \
    tpg_status s_ = (call);                 \
    if (s_ != TPG_OK) return s_;            \
  } while (0)

// A device buffer that grows on demand (contents are not preserved unless
// grow_keep is used).
struct DevBuf {
  void* p = nullptr;
  size_t cap = 0;
  template <class T>
  T* as() const { return reinterpret_cast<T*>(p); }
};

}  // namespace tpg
