// Device-side building blocks shared by the kernels of libtpg (gfx950,
// wave64): node encoding, wave/block scans, visited-set bit tests.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tpg {

constexpr int kBlock = 256;  // threads per workgroup for path kernels (4 waves)

// The path tree is built over chains (straight lines of the graph, each
// taken as one vertex; see Chains).  A node is one path of chains, stored as
//   par  : global index of the parent node (-1 for a single chain)
//   info : last chain, graph-wide id (bits 0-16) | first chain, id local to
//          its component (bits 17-28) | flags (bits 29-31)
//   tl   : vertices of its chains, each chain once
// Several CFGs can be processed as one disjoint union ("components"); a
// visited set indexes the local ids of the path's own component.
constexpr uint32_t kVMask = 0x1FFFFu;
constexpr int kV1Shift = 17;
constexpr uint32_t kV1Mask = 0xFFFu;
constexpr uint32_t F_CYC = 1u << 29;   // closes a cycle (last vertex = first)
// F_PP and F_TERM live only in registers while a level is extended; the
// stored leaf kind is the node's nch code
constexpr uint32_t F_PP = 1u << 30;    // prime path leaf (terminal and not backward-extendable)
constexpr uint32_t F_TERM = 1u << 31;  // acyclic, cannot be extended forward
constexpr int kMaxUnionVertices = 1 << 17;

__device__ __forceinline__ int node_v(uint32_t info) { return (int)(info & kVMask); }
__device__ __forceinline__ int node_v1l(uint32_t info) { return (int)((info >> kV1Shift) & kV1Mask); }
__device__ __forceinline__ uint32_t make_info(int v, int v1l, uint32_t flags) {
  return (uint32_t)v | ((uint32_t)v1l << kV1Shift) | flags;
}

// A node's child count with its leaf kind folded in, so that the ranking
// sweeps read one byte per node: a node with children stores their number
// (1..64); a leaf stores kNchCycle for a closed cycle, kNchPP for an acyclic
// prime path and 0 for a terminal path that is not prime.
constexpr uint8_t kNchPP = 254;
constexpr uint8_t kNchCycle = 255;
__device__ __forceinline__ uint8_t nch_code(uint32_t info, int nchildren) {
  return nchildren ? (uint8_t)nchildren
                   : (info & F_CYC) ? kNchCycle : (info & F_PP) ? kNchPP : (uint8_t)0;
}

struct DGraph {
  const int32_t* sp;    // successor row pointers [n+1] (graph-wide ids)
  const int32_t* s;     // successors, ascending per row
  const int32_t* pp;    // predecessor row pointers [n+1]
  const int32_t* p;     // predecessors
  const int32_t* loc;   // [n] id of each vertex inside its component
  const int32_t* comp;  // [n] component of each vertex
  const int32_t* cbase; // [n_comp+1] first graph-wide id of each component
  const int32_t* centry;// [n_comp] entry (graph-wide id)
  const int32_t* cexit; // [n_comp] exit (graph-wide id)
  int32_t n, n_comp;
  // The graph of chains only: vertices per chain; sp, s, pp, p, loc and len
  // lie back to back in one buffer starting at sp, n_stage int32 words in
  // all (what a kernel stages in LDS).
  const int32_t* len;   // [n]
  int32_t n_stage;
  int32_t max_comp;     // vertices of the largest component, every chain's counted
};

// The vertices behind a graph of chains (graph-wide ids).
struct DChains {
  const int32_t* off;  // [n + 1] rows of v
  const int32_t* v;    // vertices of every chain, in order
  const int32_t* of;   // per vertex: its chain
  const int32_t* pos;  // per vertex: its place there
};

// Largest CSR (sp .. len, bytes) that the extension kernel stages in LDS.
constexpr int kGraphLdsBytes = 16384;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

template <class T>
__device__ __forceinline__ T wave_incl_scan(T x) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T y = __shfl_up(x, d, 64);
    if (lane_id() >= d) x += y;
  }
  return x;
}

// Orders the LDS accesses of one wave's lanes: what a lane wrote before it is
// seen by the other lanes of its wave after it (a wave runs in lockstep; this
// keeps the compiler from moving LDS accesses across it and waits for them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive scan across a workgroup of NT threads; s_w needs NT/64 slots.
template <int NT, class T>
__device__ __forceinline__ T block_excl_scan(T x, T& total, T* s_w) {
  T inc = wave_incl_scan(x);
  const int w = (int)(threadIdx.x >> 6);
  if (lane_id() == 63) s_w[w] = inc;
  __syncthreads();
  T pre = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    T v = s_w[i];
    pre += (i < w) ? v : (T)0;
    tot += v;
  }
  __syncthreads();
  total = tot;
  return pre + inc - x;
}

// Visited-set bit test on a register-resident mask of W 64-bit words.
template <int W>
__device__ __forceinline__ bool mask_has(const uint64_t (&m)[W], int w) {
  const int q = w >> 6;
  uint64_t word = 0;
#pragma unroll
  for (int k = 0; k < W; ++k) word = (k == q) ? m[k] : word;
  return (word >> (w & 63)) & 1ull;
}

// r-th set bit (0-based) of x; x has more than r set bits.
__device__ __forceinline__ int select_bit(uint64_t x, int r) {
  for (int i = 0; i < r; ++i) x &= x - 1;
  return __builtin_ctzll(x);
}

}  // namespace tpg
