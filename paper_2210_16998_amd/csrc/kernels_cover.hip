// Test paths by longest-first covering (the Ammann-Offutt generation the
// paper cites among the methods for TPs): prime paths are taken in order of
// decreasing length (ties: canonical order); a prime path already contained,
// as a contiguous subpath, in the test path of a prime path taken before it
// gets no test path of its own.
//
// How it runs on the device:
//  * every spliced test path t finds the prime paths it contains.  A prime
//    path is a simple path that cannot be extended either way, or a simple
//    cycle, so among the windows of t starting at position i only the
//    longest simple one, t[i..j(i)), can be a prime path (a shorter simple
//    window is extended by t's next entry), or the cycle t[i..j(i)] when
//    t[j(i)] = t[i].  If the longest window of i - 1 ends where that of i
//    does, it extends it backward; so an acyclic candidate starts at 0 or
//    right after the start of a cycle.  The local prime rule (no successor of
//    the last vertex outside the window or equal to the first; every
//    predecessor of the first vertex inside) accepts the candidates, and a
//    hash table of the prime paths gives the accepted window's index.  The
//    table is exact for these lookups: an accepted window is a prime path,
//    and the table is built only when no two prime paths share a hash.
//  * t is a prefix, the prime path and a suffix, each of them simple (or the
//    path a cycle), so a vertex has at most one place in each, and the next
//    place of t[k] after k is a table entry; j(i) is the least of them from i
//    on, a scan.  One wave takes a path, its lanes the positions.
//  * The sequential rule "chosen iff no earlier chooser covers it" is
//    resolved in rounds: a path with a chosen earlier coverer is dropped, a
//    path whose earlier coverers are all dropped is chosen.  The first
//    undecided path in the order is decided in every round, so the rounds
//    end; in practice a handful suffice.  A round is one pass over the
//    covering pairs that only stores constant flags (a few short prime
//    paths are contained in most test paths, so per-path atomics or lists
//    would serialize), then one pass that decides.

#include "kernels.h"

namespace tpg {

namespace {

constexpr uint64_t kHashMul = 0x9E3779B97F4A7C15ull;  // odd multiplier of the polynomial hash

// Polynomial hash of a vertex sequence v_0 .. v_(k-1): the sum of
// (v_i + 1) mul^(k - 1 - i), never 0.
__device__ __forceinline__ uint64_t seq_hash_fix(uint64_t h) { return h ? h : 1ull; }

// mul^(2^b) and mul^-(2^b): exponents below 2^14 (rows of 3 * 4096 + 1)
constexpr int kPowers = 14;
struct HashPowers {
  uint64_t pow[kPowers], inv[kPowers];
};

HashPowers hash_powers(uint64_t mul) {
  HashPowers w;
  uint64_t inv = mul;  // Newton's iteration for the inverse of an odd number mod 2^64
  for (int r = 0; r < 6; ++r) inv *= 2 - mul * inv;
  for (int b = 0; b < kPowers; ++b, mul *= mul, inv *= inv) {
    w.pow[b] = mul;
    w.inv[b] = inv;
  }
  return w;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t x, int from) {
  return (uint64_t)(uint32_t)__shfl((int)(uint32_t)x, from, 64) |
         (uint64_t)(uint32_t)__shfl((int)(x >> 32), from, 64) << 32;
}

// Sixteen lanes take a path: as the polynomial's value is mul^(k - 1) times the
// sum of (v_i + 1) mul^-i (mul is odd), they add up strided parts of the sum.
// A thread per path waited for its entries one after another: 368 us for
// 376808 paths, 66 this way.
constexpr int kHashLanes = 16;
__global__ __launch_bounds__(kBlock) void k_pp_hash_insert(const int64_t* off, const int32_t* vtx,
                                                           int64_t n, HashPowers w,
                                                           unsigned long long* keys, int32_t* vals,
                                                           int64_t mask, unsigned long long* dups) {
  const int l = (int)threadIdx.x & (kHashLanes - 1);
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kHashLanes;
  if (i >= n) return;
  const int64_t o = off[i];
  const int len = (int)(off[i + 1] - o);
  uint64_t sum = 0, f = 1;
  for (int b = 0; b < 4; ++b)
    if (l >> b & 1) f *= w.inv[b];
  for (int k = l; k < len; k += kHashLanes) {
    sum += (uint64_t)(vtx[o + k] + 1) * f;
    f *= w.inv[4];
  }
#pragma unroll
  for (int d = kHashLanes / 2; d >= 1; d >>= 1) sum += shfl64(sum, lane_id() ^ d);
  if (l) return;
  uint64_t h = sum;
  for (int e = len - 1, k = 0; e; e >>= 1, ++k)
    if (e & 1) h *= w.pow[k];
  h = seq_hash_fix(h);
  int64_t s = (int64_t)(h & (uint64_t)mask);
  for (int64_t probe = 0; probe <= mask; ++probe) {
    const unsigned long long prev = atomicCAS(&keys[s], 0ull, (unsigned long long)h);
    if (prev == 0ull) {
      vals[s] = (int32_t)i;
      return;
    }
    if (prev == h) {  // two prime paths share this hash: the table cannot be used
      atomicAdd(dups, 1ull);
      return;
    }
    s = (s + 1) & mask;
  }
  atomicAdd(dups, 1ull);  // table full (cannot happen at load factor 1/2)
}

__device__ __forceinline__ int32_t table_find(const unsigned long long* keys, const int32_t* vals,
                                              int64_t mask, uint64_t h) {
  int64_t s = (int64_t)(h & (uint64_t)mask);
  for (int64_t probe = 0; probe <= mask; ++probe) {
    const unsigned long long k = keys[s];
    if (k == h) return vals[s];
    if (k == 0ull) return -1;
    s = (s + 1) & mask;
  }
  return -1;
}

struct CoverArgs {
  DGraph g;
  int n;  // vertices
  const int64_t* pp_off;
  const int32_t* pp_vtx;
  int64_t np;
  EndRows b;
  HashPowers w;
  const unsigned long long* keys;
  const int32_t* vals;
  int64_t mask;
  int32_t *pair_p, *pair_q;
  int64_t cap;
  unsigned long long* count;
  unsigned long long* missing;
};

// Orders a wave's own LDS accesses (no other wave shares its rows).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Pairs (p, q): the test path spliced for p contains prime path q, which comes
// after p in the order of decreasing length.  One wave per p; LDS per wave:
// the row t (3 n + 2 entries) and each vertex's place in its prefix, its prime
// path and its suffix.  The spliced rows are not written anywhere.
//
// A window's hash is sum of (t[k] + 1) mul^(end - 1 - k), which the wave takes
// as mul^(end - 1) times the sum of (t[k] + 1) mul^-k (mul is odd).
//
// Bound by instructions, the LDS lookups and the scan of j for the most part.
// 376808 prime paths of a 182-vertex CFG: 548 us; a thread per path that walked
// rows written before took two passes of 1250 us, and a sort by length besides,
// which the lengths of p and of the window make needless.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_cover(CoverArgs a) {
  extern __shared__ uint16_t s_cover[];
  const int lane = lane_id(), wave = (int)threadIdx.x >> 6;
  const int n = a.n, row = (3 * n + 3) & ~1;
  uint16_t* t = s_cover + (size_t)wave * (row + 3 * (n + (n & 1)));
  uint16_t* at_a = t + row;
  uint16_t* at_b = at_a + n + (n & 1);
  uint16_t* at_c = at_b + n + (n & 1);
  uint32_t* at_all = reinterpret_cast<uint32_t*>(at_a);
  const int at_words = 3 * (n + (n & 1)) / 2;
  constexpr int kNone = 0xFFFF;
  const uint64_t inv64 = a.w.inv[6];
  uint64_t inv_lane = 1;
  for (int b = 0; b < 6; ++b)
    if (lane >> b & 1) inv_lane *= a.w.inv[b];
  __shared__ int32_t s_p[NW][64], s_q[NW][64];  // found pairs, not written yet
  int held = 0;
  auto flush = [&]() {
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(a.count, (unsigned long long)held);
    at = shfl64(at, 0);
    if (lane < held && (int64_t)at + lane < a.cap) {
      a.pair_p[at + lane] = s_p[wave][lane];
      a.pair_q[at + lane] = s_q[wave][lane];
    }
    held = 0;
  };
  for (int64_t p = (int64_t)blockIdx.x * NW + wave; p < a.np; p += (int64_t)gridDim.x * NW) {
    const int64_t o0 = a.pp_off[p];
    const int lq = (int)(a.pp_off[p + 1] - o0);
    const int32_t* pp = a.pp_vtx + o0;
    const int v1 = pp[0], vk = pp[lq - 1];
    const bool cyc = lq > 1 && v1 == vk;
    const int lp = a.b.n_pfx[v1], lpq = lp + lq, L = lpq + a.b.n_sfx[vk];
    const int32_t* pfx = a.b.pfx + a.b.pfx_at[v1];
    const int32_t* sfx = a.b.sfx + a.b.sfx_at[vk];
    const int last = lpq - 1;  // the path's last entry
    for (int k = lane; k < at_words; k += 64) at_all[k] = 0xFFFFFFFFu;
    wave_lds_fence();
    for (int k = lane; k < L; k += 64) {
      const int x = k < lp ? pfx[k] : k < lpq ? pp[k - lp] : sfx[k - lpq];
      t[k] = (uint16_t)x;
      if (k < lp) at_a[x] = (uint16_t)k;
      else if (k >= lpq) at_c[x] = (uint16_t)k;
      else if (!cyc || k != last) at_b[x] = (uint16_t)k;  // a cycle's vertex: its first place
    }
    wave_lds_fence();
    // is vertex w on t[i..j)?
    auto on = [&](int w, int i, int j) {
      const int x = at_a[w], y = at_b[w], z = at_c[w];
      return (x >= i && x < j) || (y >= i && y < j) || (z >= i && z < j) ||
             (cyc && w == v1 && last >= i && last < j);
    };
    // windows that come before p in the order, or are p, make no pair
    auto wanted = [&](int i, int end) {
      return end - i <= lq && !(i == lp && end == lpq);
    };
    // the local prime rule for the window t[i..j)
    auto prime = [&](int i, int j) {
      const int x = t[i], y = t[j - 1];
      bool ok = true;
      for (int k = a.g.sp[y]; k < a.g.sp[y + 1] && ok; ++k) {
        const int w = a.g.s[k];
        ok = w != x && on(w, i, j);
      }
      for (int k = a.g.pp[x]; k < a.g.pp[x + 1] && ok; ++k) ok = on(a.g.p[k], i, j);
      return ok;
    };
    // t[i..end) (the same in all lanes) is a prime path
    auto found = [&](int i, int end) {
      const int len = end - i;
      uint64_t sum = 0, f = inv_lane;
      for (int k = lane; k < end; k += 64) {
        if (k >= i) sum += (uint64_t)(t[k] + 1) * f;
        f *= inv64;
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) sum += shfl64(sum, lane ^ d);
      uint64_t h = sum;
      for (int e = end - 1, k = 0; e; e >>= 1, ++k)
        if (e & 1) h *= a.w.pow[k];
      const int32_t q = table_find(a.keys, a.vals, a.mask, seq_hash_fix(h));
      if (q < 0) {
        if (lane == 0) atomicAdd(a.missing, 1ull);  // not a prime path: a bug, reported to the host
      } else if (lq > len || p < q) {
        if (held == 64) flush();
        if (lane == 0) {
          s_p[wave][held] = (int32_t)p;
          s_q[wave][held] = q;
        }
        wave_lds_fence();
        ++held;
      }
    };
    // from the last positions to the first: j(k), and with a cycle at k that
    // cycle and the window that starts after it
    int next_j = L;          // j of the position after the block
    bool next_cyc = true;    // nothing starts after the row
    for (int k0 = (L - 1) & ~63; k0 >= 0; k0 -= 64) {
      const int k = k0 + lane;
      int nx = L;
      if (k < lpq) {
        const int x = t[k], c = at_c[x], b = at_b[x];
        nx = c != kNone ? c : L;
        if (k < lp && b != kNone) nx = b;
        if (cyc && k == lp) nx = last;
      }
      int j = nx;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_down(j, d, 64);
        if (lane + d < 64) j = min(j, o);
      }
      j = min(j, next_j);
      const bool is_cyc = k < L && nx == j && j < L;
      // the position after this one
      int j1 = __shfl_down(j, 1, 64);
      int c1 = __shfl_down((int)is_cyc, 1, 64);
      if (lane == 63) {
        j1 = next_j;
        c1 = next_cyc;
      }
      const bool after = is_cyc && !c1 && wanted(k + 1, j1) && prime(k + 1, j1);
      const bool head = k == 0 && !is_cyc && wanted(0, j) && prime(0, j);
      next_j = __builtin_amdgcn_readfirstlane(j);
      next_cyc = (bool)__builtin_amdgcn_readfirstlane((int)is_cyc);
      for (uint64_t m = __ballot(is_cyc && wanted(k, j + 1)); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        found(k0 + l, __builtin_amdgcn_readlane(j, l) + 1);
      }
      for (uint64_t m = __ballot(after); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        found(k0 + l + 1, __builtin_amdgcn_readlane(j1, l));
      }
      if (__ballot(head)) found(0, __builtin_amdgcn_readfirstlane(j));
    }
    wave_lds_fence();
  }
  if (held) flush();
}

// One round over the pairs (p covers q, p before q in the order): q is
// dropped if p is chosen, and blocked (cannot be chosen yet) if p is still
// undecided.  Only constant values are stored.
__global__ __launch_bounds__(kBlock) void k_round_pairs(const int32_t* pair_p, const int32_t* pair_q,
                                                        int64_t np, const uint8_t* state,
                                                        uint8_t* drop, uint8_t* block) {
  const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (k >= np) return;
  const int32_t p = pair_p[k], q = pair_q[k];
  if (state[q] != 0) return;
  const uint8_t sp = state[p];
  if (sp == 1) drop[q] = 1;
  else if (sp == 0) block[q] = 1;
}

// Decide: 1 chosen, 2 dropped, 0 undecided; clears the flags for the next
// round and counts the undecided paths (one atomic per wave) if asked to.
__global__ __launch_bounds__(kBlock) void k_round_decide(int64_t n, uint8_t* state, uint8_t* drop,
                                                         uint8_t* block,
                                                         unsigned long long* undecided) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  int und = 0;
  if (q < n && state[q] == 0) {
    if (drop[q]) state[q] = 2;
    else if (!block[q]) state[q] = 1;
    else und = 1;
    drop[q] = 0;
    block[q] = 0;
  }
  if (!undecided) return;
  const uint64_t b = __ballot(und);
  if (lane_id() == 0 && b) atomicAdd(undecided, (unsigned long long)__builtin_popcountll(b));
}

}  // namespace

hipError_t launch_pp_hash_insert(const int64_t* off, const int32_t* vtx, int64_t n, uint64_t mul,
                                 uint64_t* keys, int32_t* vals, int64_t mask, uint64_t* dups,
                                 hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t rows = kBlock / kHashLanes;
  k_pp_hash_insert<<<(unsigned)((n + rows - 1) / rows), kBlock, 0, st>>>(
      off, vtx, n, hash_powers(mul), reinterpret_cast<unsigned long long*>(keys), vals, mask,
      reinterpret_cast<unsigned long long*>(dups));
  return hipGetLastError();
}

uint64_t cover_hash_mul(int attempt) { return kHashMul + 2ull * (uint64_t)attempt * 0x2545F4914F6CDD1Dull; }

hipError_t launch_cover(const DGraph& g, int n, const int64_t* pp_off, const int32_t* pp_vtx,
                        int64_t np, const EndRows& b, uint64_t mul, const uint64_t* keys,
                        const int32_t* vals, int64_t mask, int32_t* pair_p, int32_t* pair_q,
                        int64_t cap, uint64_t* count, uint64_t* missing, int num_cus,
                        hipStream_t st) {
  if (np == 0) return hipSuccess;
  if (n < 1 || 3 * n + 1 >= 1 << kPowers) return hipErrorInvalidValue;
  CoverArgs a{};
  a.g = g;
  a.n = n;
  a.pp_off = pp_off;
  a.pp_vtx = pp_vtx;
  a.np = np;
  a.b = b;
  a.w = hash_powers(mul);
  a.keys = reinterpret_cast<const unsigned long long*>(keys);
  a.vals = vals;
  a.mask = mask;
  a.pair_p = pair_p;
  a.pair_q = pair_q;
  a.cap = cap;
  a.count = reinterpret_cast<unsigned long long*>(count);
  a.missing = reinterpret_cast<unsigned long long*>(missing);
  const size_t lds = sizeof(uint16_t) * (size_t)(((3 * n + 3) & ~1) + 3 * (n + (n & 1)));
  // four waves a workgroup while that leaves the CU its 32 waves (20 KB each);
  // one for the large graphs, up to 49 KB
  if (4 * lds <= 20 << 10) {
    const int64_t grid = std::min<int64_t>((np + 3) / 4, (int64_t)num_cus * 8);
    k_cover<4><<<(unsigned)grid, 256, 4 * lds, st>>>(a);
  } else {
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(32, (160 << 10) / (int64_t)(lds + 512)));
    const int64_t grid = std::min<int64_t>(np, (int64_t)num_cus * per_cu);
    k_cover<1><<<(unsigned)grid, 64, lds, st>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_round_pairs(const int32_t* pair_p, const int32_t* pair_q, int64_t np,
                              const uint8_t* state, uint8_t* drop, uint8_t* block,
                              hipStream_t st) {
  if (np == 0) return hipSuccess;
  k_round_pairs<<<(unsigned)((np + kBlock - 1) / kBlock), kBlock, 0, st>>>(pair_p, pair_q, np, state,
                                                                          drop, block);
  return hipGetLastError();
}

hipError_t launch_round_decide(int64_t n, uint8_t* state, uint8_t* drop, uint8_t* block,
                               uint64_t* undecided, hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_round_decide<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      n, state, drop, block, reinterpret_cast<unsigned long long*>(undecided));
  return hipGetLastError();
}

}  // namespace tpg
