// Path-count predictor: a 32 -> 128 -> 128 -> 65 multilayer perceptron with
// BF16 operands on the matrix cores and FP32 accumulation, trained with Adam
// on FP32 master weights.  Inputs are the 32 structural features of a CFG;
// outputs are log1p of the number of simple paths with L entries (L = 1..64,
// deeper levels pooled into 64) and log1p of the prime-path count.  The
// predictions size the path pool of the batched form; results never depend on
// them.
//
// Rows are independent up to the weight gradients, so one kernel takes 16 rows
// through everything that belongs to them (k_mlp_rows), a second one forms the
// weight gradients' products over the rows, split along them (k_mlp_wgrad),
// and a third one adds the parts up (k_mlp_reduce).  Gradients of 1024 rows,
// host arrays in and out: 95 us, 950 as a chain of separate products, column
// sums and copies.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "internal.h"

namespace tpg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = 32, kHid = 128, kOut = 65, kOutPad = 128;

// fp32 -> bf16, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
static inline uint16_t f2bf_host(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Operands of one pass over n rows (ld: the transposed arrays' row length).
struct RowArgs {
  const float* x;          // [n][32]
  const float* t;          // [n][65]; null: forward only
  int n, ld;
  const float *mean, *stdv;
  const uint16_t *w1t, *w2t, *w3t;  // W^T, [out][in], rows of 64 / 128 / 128
  const uint16_t *w2, *w3;          // W, [in][out], rows of 128
  const float *b1, *b2, *b3;
  float* y;                // [n][65]
  // for the weight gradients, bf16, [column][row]
  uint16_t *xt, *h1t, *h2t, *dyt, *dh2t, *dh1t;
  // sums over a block's 16 rows: 3 x 128 bias gradients, then the squared error
  float* part;             // [blocks][kPart]
};
constexpr int kRowTile = 16;
constexpr int kPart = 3 * kHid + 1;
constexpr int kOutK = 96;  // 65 outputs padded to whole steps of 32

// A 16 x 16 product tile: A rows in LDS (row-major, `lda`), B^T rows in memory
// (`ldb`), both K contiguous; lane l holds D[4 (l / 16) + j][l % 16].
template <int K>
__device__ __forceinline__ f32x4 tile_product(const uint16_t* a, int lda, const uint16_t* bt,
                                              int ldb) {
  const int lane = (int)(threadIdx.x & 63), r = lane & 15, kq = (lane >> 4) * 8;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 32) {
    const bf16x8 av = *reinterpret_cast<const bf16x8*>(a + r * lda + kq + k0);
    const bf16x8 bv = *reinterpret_cast<const bf16x8*>(bt + (size_t)r * ldb + kq + k0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
  }
  return acc;
}

// The lane's four values of a tile (rows row0 .., column col), in bf16 to the
// next product's A rows and, transposed, to `t` (null: not kept).
__device__ __forceinline__ void tile_put(const f32x4& v, int col, int row0, int block_row,
                                         uint16_t* a, int lda, uint16_t* t, int ld) {
  uint16_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = f2bf(v[j]);
    if (a) a[(row0 + j) * lda + col] = h[j];
  }
  if (t)
    *reinterpret_cast<uint2*>(t + (size_t)col * ld + block_row + row0) =
        make_uint2((uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16);
}

// Sum of a column over the tile's 16 rows, to the lanes of its first four.
__device__ __forceinline__ float tile_colsum(const f32x4& v) {
  float c = (v[0] + v[1]) + (v[2] + v[3]);
  c += __shfl_xor(c, 16, 64);
  c += __shfl_xor(c, 32, 64);
  return c;
}

// 16 rows per workgroup, from features to outputs and, with targets, back to
// the first hidden layer's gradient; four waves share the columns.  Bound by
// the latency of its seven dependent products (the weights come from L2, the
// activations stay in LDS): 15 us for 1024 rows.  Separate products and column
// sums took 0.85 ms, most of it three serial column sums of 222 us.
__global__ __launch_bounds__(256) void k_mlp_rows(RowArgs g) {
  constexpr int LX = kIn + 8, LH = kHid + 8, LO = kOutK + 8;  // LDS row strides
  __shared__ __align__(16) uint16_t s_x[kRowTile * LX];
  __shared__ __align__(16) uint16_t s_h1[kRowTile * LH];
  __shared__ __align__(16) uint16_t s_h2[kRowTile * LH];
  __shared__ __align__(16) uint16_t s_dy[kRowTile * LO];
  __shared__ float s_sq[4];
  const int tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b0 = (int)blockIdx.x * kRowTile;      // first row
  const int r0 = 4 * (lane >> 4), cl = lane & 15;  // the lane's rows and column in a tile
  const bool grad = g.t != nullptr;
  float* part = g.part + (size_t)blockIdx.x * kPart;
  auto valid = [&](int j) { return b0 + r0 + j < g.n; };
  for (int i = tid; i < kRowTile * kIn; i += 256) {
    const int r = i / kIn, f = i % kIn, row = b0 + r;
    const float v = row < g.n ? (g.x[(size_t)row * kIn + f] - g.mean[f]) / g.stdv[f] : 0.f;
    const uint16_t h = f2bf(v);
    s_x[r * LX + f] = h;
    if (grad) g.xt[(size_t)f * g.ld + row] = h;
  }
  for (int i = tid; i < kRowTile * LO; i += 256) s_dy[i] = 0;
  __syncthreads();
  // hidden layers: two tiles of 16 columns a wave; on[..]: the unit is active
  bool on1[2][4], on2[2][4];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c0 = 16 * (wave + 4 * q), col = c0 + cl;
    f32x4 v = tile_product<kIn>(s_x, LX, g.w1t + (size_t)c0 * 64, 64);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] += g.b1[col];
      on1[q][j] = v[j] > 0.f && valid(j);
      v[j] = on1[q][j] ? v[j] : 0.f;
    }
    tile_put(v, col, r0, b0, s_h1, LH, grad ? g.h1t : nullptr, g.ld);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c0 = 16 * (wave + 4 * q), col = c0 + cl;
    f32x4 v = tile_product<kHid>(s_h1, LH, g.w2t + (size_t)c0 * kHid, kHid);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] += g.b2[col];
      on2[q][j] = v[j] > 0.f && valid(j);
      v[j] = on2[q][j] ? v[j] : 0.f;
    }
    tile_put(v, col, r0, b0, s_h2, LH, grad ? g.h2t : nullptr, g.ld);
  }
  __syncthreads();
  // outputs: five tiles; with targets their gradient and the squared error
  float sq = 0.f;
  for (int c0 = 16 * wave; c0 < kOut; c0 += 64) {
    const int col = c0 + cl;
    f32x4 v = tile_product<kHid>(s_h2, LH, g.w3t + (size_t)c0 * kHid, kHid);
    f32x4 d{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (col >= kOut || !valid(j)) continue;
      const size_t at = (size_t)(b0 + r0 + j) * kOut + col;
      const float y = v[j] + g.b3[col];
      if (!grad) {
        g.y[at] = y;
        continue;
      }
      const float e = y - g.t[at];
      d[j] = 2.f * e / (float)(g.n * kOut);
      sq += e * e;
    }
    if (grad) {
      tile_put(d, col, r0, b0, s_dy, LO, g.dyt, g.ld);
      const float c = tile_colsum(d);
      if (lane < 16) part[2 * kHid + col] = c;
    }
  }
  if (!grad) return;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) sq += __shfl_xor(sq, d, 64);
  if (lane == 0) s_sq[wave] = sq;
  __syncthreads();
  if (tid == 0) part[3 * kHid] = (s_sq[0] + s_sq[1]) + (s_sq[2] + s_sq[3]);
  // dH2 = dY W3^T and dH1 = dH2 W2^T where the units are active; dH2's rows
  // take the place of H1's, which no product reads any more
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c0 = 16 * (wave + 4 * q), col = c0 + cl;
    f32x4 v = tile_product<kOutK>(s_dy, LO, g.w3 + (size_t)c0 * kOutPad, kOutPad);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = on2[q][j] ? v[j] : 0.f;
    tile_put(v, col, r0, b0, s_h1, LH, g.dh2t, g.ld);
    const float c = tile_colsum(v);
    if (lane < 16) part[kHid + col] = c;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c0 = 16 * (wave + 4 * q), col = c0 + cl;
    f32x4 v = tile_product<kHid>(s_h1, LH, g.w2 + (size_t)c0 * kHid, kHid);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = on1[q][j] ? v[j] : 0.f;
    tile_put(v, col, r0, b0, nullptr, 0, g.dh1t, g.ld);
    const float c = tile_colsum(v);
    if (lane < 16) part[col] = c;
  }
}

// Weight gradients dW = A^T dB as C[m][n] = sum over rows of at[m][row]
// bt[n][row], in 64 x 64 tiles: two for W1 (32 of its 64 rows), four for W2,
// four for W3 (65 of its 128 columns).  Split z of gridDim.y takes the rows
// [z * k_split, (z + 1) * k_split) and writes its tile on its own: 4.5 us for
// 1024 rows in eight splits; in one piece ten workgroups took 17 us a product.
constexpr int kTiles = 10;
__global__ __launch_bounds__(256) void k_mlp_wgrad(RowArgs g, int rows, int k_split, float* out) {
  const int tile = (int)blockIdx.x;
  const uint16_t *at, *bt;
  int m0, n0;
  if (tile < 2) {
    at = g.xt, bt = g.dh1t, m0 = 0, n0 = 64 * tile;
  } else {
    at = tile < 6 ? g.h1t : g.h2t;
    bt = tile < 6 ? g.dh2t : g.dyt;
    m0 = 64 * ((tile - 2) / 2 % 2), n0 = 64 * ((tile - 2) % 2);
  }
  const int wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const int r = lane & 15, kq = (lane >> 4) * 8;
  const int k0 = (int)blockIdx.y * k_split, k1 = min(rows, k0 + k_split);
  f32x4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* arow = at + (size_t)(m0 + wave * 16 + r) * g.ld + kq;
  for (int k = k0; k < k1; k += 32) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(arow + k);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(bt + (size_t)(n0 + 16 * t + r) * g.ld + kq + k);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
    }
  }
  float* o = out + ((size_t)blockIdx.y * kTiles + tile) * 4096;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[(wave * 16 + 4 * (lane >> 4) + j) * 64 + 16 * t + (lane & 15)] = acc[t][j];
}

// fp32 block layout (floats): w1 64 x 128 (rows 32..63 stay 0), b1 128, w2
// 128 x 128, b2 128, w3 128 x 128, b3 128 (columns 65.. stay 0)
constexpr size_t oW1 = 0, oB1 = oW1 + 64 * kHid, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid,
                 oW3 = oB2 + kHid, oB3 = oW3 + kHid * kOutPad, oEnd = oB3 + kOutPad;

// Gradients in the block layout and the loss from the parts.  The first
// kWeightBlocks workgroups take a weight per thread, the others 32 columns of
// the row pass's parts each, a part in eight per thread: latency of a few
// dependent loads, 3.8 us for 64 parts (26 with one workgroup for all columns).
constexpr int kWeightBlocks = (64 * kHid + 2 * kHid * kHid) / 256;
constexpr int kPartBlocks = (kPart + 31) / 32;
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* tiles, int splits,
                                                    const float* part, int blocks, float inv_n,
                                                    float* grad, float* loss) {
  const int i = (int)(blockIdx.x * 256 + threadIdx.x);
  if (blockIdx.x < kWeightBlocks) {
    int tile, row, col;
    size_t at;
    if (i < 64 * kHid) {  // W1
      row = i / kHid, col = i % kHid, tile = col / 64, at = oW1 + i;
    } else {
      const int w = (i - 64 * kHid) / (kHid * kHid);  // 0: W2, 1: W3
      const int e = (i - 64 * kHid) % (kHid * kHid);
      row = e / kHid, col = e % kHid;
      tile = 2 + 4 * w + 2 * (row / 64) + col / 64, at = (w ? oW3 : oW2) + e;
    }
    const float* p = tiles + (size_t)tile * 4096 + (row % 64) * 64 + col % 64;
    float s = 0.f;
    for (int z = 0; z < splits; ++z) s += p[(size_t)z * kTiles * 4096];
    if ((i < 64 * kHid && row >= kIn) || (at >= oW3 && col >= kOut)) s = 0.f;
    grad[at] = s;
    return;
  }
  __shared__ float s_sum[256];
  const int tid = (int)threadIdx.x, c = ((int)blockIdx.x - kWeightBlocks) * 32 + (tid & 31);
  // columns past the 65th of the output bias are not written by the row pass
  const int l = c / kHid;
  const bool live = c < kPart && (l != 2 || c % kHid < kOut);
  float s = 0.f;
  if (live)
#pragma unroll 4
    for (int b = tid >> 5; b < blocks; b += 8) s += part[(size_t)b * kPart + c];
  s_sum[tid] = s;
  __syncthreads();
  if (tid >= 32 || c >= kPart) return;
  s = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) s += s_sum[q * 32 + tid];
  if (l < 3) grad[(l == 0 ? oB1 : l == 1 ? oB2 : oB3) + c % kHid] = s;
  else *loss = s * inv_n;
}

struct AdamArgs {
  float* w;
  float* m;
  float* v;
  const float* g;
  int n;
  float lr, b1, b2, eps, c1, c2;  // c1 = 1 - b1^t, c2 = 1 - b2^t
};

__global__ void k_adam(AdamArgs a) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= a.n) return;
  const float g = a.g[i];
  const float m = a.b1 * a.m[i] + (1.f - a.b1) * g;
  const float v = a.b2 * a.v[i] + (1.f - a.b2) * g * g;
  a.m[i] = m;
  a.v[i] = v;
  a.w[i] -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// fp32 master W (rows x cols, first valid_cols used) -> bf16 W and W^T
__global__ void k_refresh(const float* w, int rows, int cols, uint16_t* wb, uint16_t* wbt,
                          int ld_t) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= rows * cols) return;
  const int r = i / cols, c = i % cols;
  const uint16_t h = f2bf(w[i]);
  wb[i] = h;
  wbt[(size_t)c * ld_t + r] = h;
}

}  // namespace tpg

using namespace tpg;

// parameters, packed: W1 [32][128], b1 [128], W2 [128][128], b2 [128],
// W3 [128][65], b3 [65]
#define TPG_MLP_NPARAMS_ (kIn * kHid + kHid + kHid * kHid + kHid + kHid * kOut + kOut)

struct tpg_mlp {
  int device = 0;
  hipStream_t st = nullptr;
  // fp32 masters (W3 / b3 padded to 128 columns), Adam moments, gradients
  float* w1 = nullptr; float* w2 = nullptr; float* w3 = nullptr;
  float* b1 = nullptr; float* b2 = nullptr; float* b3 = nullptr;
  float* mom = nullptr;   // m then v for all of the above, same layout
  float* grad = nullptr;  // gradients, same layout
  float* master = nullptr;  // base of the fp32 block
  size_t n_master = 0;
  // bf16 copies: W (in x out) and W^T (out x in); W1^T is 128 x 32, W1 is 64 x 128
  uint16_t* w1b = nullptr; uint16_t* w1bt = nullptr;
  uint16_t* w2b = nullptr; uint16_t* w2bt = nullptr;
  uint16_t* w3b = nullptr; uint16_t* w3bt = nullptr;
  float* mean = nullptr; float* stdv = nullptr;
  float h_mean[kIn], h_std[kIn];
  int64_t step = 0;
  // arrays for up to `rows` rows (a multiple of 64)
  int rows = 0;
  void* act = nullptr;
  float *x = nullptr, *t = nullptr, *y = nullptr, *part = nullptr, *tiles = nullptr;
  float* loss = nullptr;
  uint16_t *xt = nullptr, *h1t = nullptr, *h2t = nullptr, *dyt = nullptr, *dh2t = nullptr,
           *dh1t = nullptr;
  // pinned room that arrays pass through on their way up (features, targets) and
  // back (outputs, or the gradient block and the loss)
  float* host = nullptr;
  size_t host_floats = 0, host_used = 0;
  bool seen = false;  // a call has been made
  bool busy = false;  // work that uses `host` may not have ended
};

namespace {

tpg_status mlp_alloc(tpg_mlp* m) {
  TPG_HIP(hipSetDevice(m->device));
  TPG_HIP(hipStreamCreateWithFlags(&m->st, hipStreamNonBlocking));
  m->n_master = oEnd;
  TPG_HIP(hipMalloc(&m->master, sizeof(float) * oEnd * 4));  // w, m, v, grad
  TPG_HIP(hipMemsetAsync(m->master, 0, sizeof(float) * oEnd * 4, m->st));
  m->w1 = m->master + oW1;
  m->b1 = m->master + oB1;
  m->w2 = m->master + oW2;
  m->b2 = m->master + oB2;
  m->w3 = m->master + oW3;
  m->b3 = m->master + oB3;
  m->mom = m->master + oEnd;
  m->grad = m->master + 3 * oEnd;
  uint16_t* bb = nullptr;
  const size_t nb = 2 * (64 * kHid + kHid * kHid + kHid * kOutPad);
  TPG_HIP(hipMalloc(&bb, sizeof(uint16_t) * nb));
  TPG_HIP(hipMemsetAsync(bb, 0, sizeof(uint16_t) * nb, m->st));
  m->w1b = bb;
  m->w1bt = m->w1b + 64 * kHid;
  m->w2b = m->w1bt + 64 * kHid;
  m->w2bt = m->w2b + kHid * kHid;
  m->w3b = m->w2bt + kHid * kHid;
  m->w3bt = m->w3b + kHid * kOutPad;
  TPG_HIP(hipMalloc(&m->mean, sizeof(float) * 2 * kIn));
  m->stdv = m->mean + kIn;
  for (int i = 0; i < kIn; ++i) m->h_mean[i] = 0.f, m->h_std[i] = 1.f;
  TPG_HIP(hipMemcpy(m->mean, m->h_mean, sizeof(float) * kIn, hipMemcpyHostToDevice));
  TPG_HIP(hipMemcpy(m->stdv, m->h_std, sizeof(float) * kIn, hipMemcpyHostToDevice));
  return TPG_OK;
}

// Rows a split of the weight gradients takes at least (four matrix steps: less
// is all reduction), and splits at most (160 workgroups, 2.6 MB of parts).
constexpr int kSplitRows = 128, kSplits = 16;

tpg_status mlp_rows(tpg_mlp* m, int n) {
  const int rows = ((n + 63) / 64) * 64;
  if (rows > m->rows) {
    if (m->act) TPG_HIP(hipFree(m->act));
    m->act = nullptr;
    m->rows = 0;
    const size_t R = (size_t)rows;
    const size_t tiles = (size_t)std::min(kSplits, (rows + kSplitRows - 1) / kSplitRows) * kTiles * 4096;
    const size_t floats = R * kIn + 2 * R * kOut + R / kRowTile * kPart + tiles + 64;
    const size_t halves = R * (64 + 2 * kHid + kOutPad + 2 * kHid);
    const size_t bytes = floats * 4 + halves * 2 + 1024;
    TPG_HIP(hipMalloc(&m->act, bytes));
    // the padding rows of the transposed arrays stay zero
    TPG_HIP(hipMemsetAsync(m->act, 0, bytes, m->st));
    uint16_t* h = (uint16_t*)m->act;
    m->xt = h; h += 64 * R;
    m->h1t = h; h += R * kHid;
    m->h2t = h; h += R * kHid;
    m->dyt = h; h += R * kOutPad;
    m->dh2t = h; h += R * kHid;
    m->dh1t = h; h += R * kHid;
    float* f = (float*)h;
    m->tiles = f; f += tiles;
    m->x = f; f += R * kIn;
    m->t = f; f += R * kOut;
    m->y = f; f += R * kOut;
    m->part = f; f += R / kRowTile * kPart;
    m->loss = f;
    m->rows = rows;
  }
  return TPG_OK;
}

// Room for a call of n rows, up to kRoomFloats.  Pinning costs some 0.3 ms a MB,
// so a handle's first call, which may be its only one, goes without (a first
// forward of 1024 rows: 0.68 ms with it, 0.40 without), and larger arrays pass
// through in pieces.  Without room the copies take the caller's arrays as they
// are.
constexpr size_t kRoomFloats = (size_t)4 << 20;
void mlp_room(tpg_mlp* m, int n) {
  const size_t need = std::min(kRoomFloats, (size_t)n * (kIn + kOut) +
                                                std::max((size_t)n * kOut, oEnd + 1));
  m->host_used = 0;
  if (m->seen && need > m->host_floats) {
    if (m->host) (void)hipHostFree(m->host);
    m->host_floats = need;
    if (hipHostMalloc((void**)&m->host, sizeof(float) * need, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      m->host = nullptr;
      m->host_floats = 0;
    }
  }
  m->seen = true;
}

// Room for `floats` of it (null: there is none so large), all of it if need be.
tpg_status mlp_take(tpg_mlp* m, size_t floats, float** at) {
  *at = nullptr;
  if (floats > m->host_floats) return TPG_OK;
  if (floats > m->host_floats - m->host_used) {
    TPG_HIP(hipStreamSynchronize(m->st));
    m->host_used = 0;
  }
  *at = m->host + m->host_used;
  m->host_used += floats;
  return TPG_OK;
}

tpg_status mlp_up(tpg_mlp* m, float* dev, const float* src, size_t floats) {
  while (floats > 0) {
    const size_t left = m->host_floats - m->host_used;
    const size_t k = m->host ? std::min(floats, left ? left : m->host_floats) : floats;
    float* at = nullptr;
    TPG_TRY(mlp_take(m, k, &at));
    if (at) memcpy(at, src, sizeof(float) * k);
    TPG_HIP(hipMemcpyAsync(dev, at ? at : src, sizeof(float) * k, hipMemcpyHostToDevice, m->st));
    if (!at) TPG_HIP(hipStreamSynchronize(m->st));  // the caller's array is its own again
    dev += k;
    src += k;
    floats -= k;
  }
  return TPG_OK;
}

// (dst holds the array when it returns)
tpg_status mlp_down(tpg_mlp* m, float* dst, const float* dev, size_t floats) {
  while (floats > 0) {
    const size_t k = m->host ? std::min(floats, m->host_floats) : floats;
    float* at = nullptr;
    TPG_TRY(mlp_take(m, k, &at));
    TPG_HIP(hipMemcpyAsync(at ? at : dst, dev, sizeof(float) * k, hipMemcpyDeviceToHost, m->st));
    TPG_HIP(hipStreamSynchronize(m->st));
    if (at) memcpy(dst, at, sizeof(float) * k);
    dst += k;
    dev += k;
    floats -= k;
  }
  return TPG_OK;
}

tpg_status refresh_bf16(tpg_mlp* m) {
  hipStream_t st = m->st;
  // W1 master is 64 x 128 (rows >= 32 zero): W1^T is 128 x 32 for the forward
  k_refresh<<<(64 * kHid + 255) / 256, 256, 0, st>>>(m->w1, 64, kHid, m->w1b, m->w1bt, 64);
  k_refresh<<<(kHid * kHid + 255) / 256, 256, 0, st>>>(m->w2, kHid, kHid, m->w2b, m->w2bt, kHid);
  k_refresh<<<(kHid * kOutPad + 255) / 256, 256, 0, st>>>(m->w3, kHid, kOutPad, m->w3b, m->w3bt, kHid);
  TPG_HIP(hipGetLastError());
  return TPG_OK;
}

// Features and targets (null: forward only) to the device, and the row pass.
tpg_status run_rows(tpg_mlp* m, const float* x, const float* t, int n, RowArgs& g) {
  hipStream_t st = m->st;
  // a training step that returns no loss does not wait for its uploads
  if (m->busy) TPG_HIP(hipStreamSynchronize(st));
  m->busy = false;
  TPG_TRY(mlp_rows(m, n));
  mlp_room(m, n);
  m->busy = true;
  TPG_TRY(mlp_up(m, m->x, x, (size_t)n * kIn));
  if (t) TPG_TRY(mlp_up(m, m->t, t, (size_t)n * kOut));
  g = RowArgs{};
  g.x = m->x;
  g.t = t ? m->t : nullptr;
  g.n = n;
  g.ld = m->rows;
  g.mean = m->mean;
  g.stdv = m->stdv;
  g.w1t = m->w1bt;
  g.w2t = m->w2bt;
  g.w3t = m->w3bt;
  g.w2 = m->w2b;
  g.w3 = m->w3b;
  g.b1 = m->b1;
  g.b2 = m->b2;
  g.b3 = m->b3;
  g.y = m->y;
  g.xt = m->xt;
  g.h1t = m->h1t;
  g.h2t = m->h2t;
  g.dyt = m->dyt;
  g.dh2t = m->dh2t;
  g.dh1t = m->dh1t;
  g.part = m->part;
  // whole steps of 32 rows for the weight gradients: rows past n are zero
  const int blocks = (n + 31) / 32 * 2;
  k_mlp_rows<<<(unsigned)blocks, 256, 0, st>>>(g);
  TPG_HIP(hipGetLastError());
  return TPG_OK;
}

// gradients of the mean squared error into m->grad (fp32 block layout), the
// loss into m->loss
tpg_status run_backward(tpg_mlp* m, const RowArgs& g) {
  hipStream_t st = m->st;
  const int rows = (g.n + 31) / 32 * 32;
  int split = std::max(kSplitRows, (rows + kSplits - 1) / kSplits);
  split = (split + 31) / 32 * 32;
  const int splits = (rows + split - 1) / split;
  k_mlp_wgrad<<<dim3(kTiles, (unsigned)splits), 256, 0, st>>>(g, rows, split, m->tiles);
  k_mlp_reduce<<<kWeightBlocks + kPartBlocks, 256, 0, st>>>(
      m->tiles, splits, m->part, rows / kRowTile, 1.f / (float)(g.n * kOut), m->grad, m->loss);
  TPG_HIP(hipGetLastError());
  return TPG_OK;
}

// packed <-> padded fp32 block
void pack_params(const float* blk, float* p) {
  size_t q = 0;
  for (int i = 0; i < kIn; ++i)
    for (int j = 0; j < kHid; ++j) p[q++] = blk[oW1 + i * kHid + j];
  for (int j = 0; j < kHid; ++j) p[q++] = blk[oB1 + j];
  for (int i = 0; i < kHid; ++i)
    for (int j = 0; j < kHid; ++j) p[q++] = blk[oW2 + i * kHid + j];
  for (int j = 0; j < kHid; ++j) p[q++] = blk[oB2 + j];
  for (int i = 0; i < kHid; ++i)
    for (int j = 0; j < kOut; ++j) p[q++] = blk[oW3 + i * kOutPad + j];
  for (int j = 0; j < kOut; ++j) p[q++] = blk[oB3 + j];
}

void unpack_params(const float* p, std::vector<float>& blk) {
  blk.assign(oEnd, 0.f);
  size_t q = 0;
  for (int i = 0; i < kIn; ++i)
    for (int j = 0; j < kHid; ++j) blk[oW1 + i * kHid + j] = p[q++];
  for (int j = 0; j < kHid; ++j) blk[oB1 + j] = p[q++];
  for (int i = 0; i < kHid; ++i)
    for (int j = 0; j < kHid; ++j) blk[oW2 + i * kHid + j] = p[q++];
  for (int j = 0; j < kHid; ++j) blk[oB2 + j] = p[q++];
  for (int i = 0; i < kHid; ++i)
    for (int j = 0; j < kOut; ++j) blk[oW3 + i * kOutPad + j] = p[q++];
  for (int j = 0; j < kOut; ++j) blk[oB3 + j] = p[q++];
}

uint64_t splitmix(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

extern "C" {

int32_t tpg_mlp_num_params(void) { return TPG_MLP_NPARAMS_; }

tpg_status tpg_mlp_create(int32_t device, uint64_t seed, tpg_mlp** out) {
  if (!out) return fail(TPG_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) {
    (void)hipGetLastError();
    return fail(TPG_ERR_DEVICE, "no HIP device available");
  }
  if (device < 0) TPG_HIP(hipGetDevice(&device));
  tpg_mlp* m = new (std::nothrow) tpg_mlp;
  if (!m) return fail(TPG_ERR_OOM_HOST, "mlp");
  m->device = device;
  tpg_status s = mlp_alloc(m);
  if (s != TPG_OK) {
    tpg_mlp_free(m);
    return s;
  }
  // He-uniform initialization from a counter-based generator; biases zero
  std::vector<float> p(TPG_MLP_NPARAMS_, 0.f);
  uint64_t st = seed;
  auto uni = [&]() { return (double)(splitmix(st) >> 11) * (1.0 / 9007199254740992.0); };
  size_t q = 0;
  const int fan[3] = {kIn, kHid, kHid}, outs[3] = {kHid, kHid, kOut};
  for (int l = 0; l < 3; ++l) {
    const double lim = std::sqrt(6.0 / fan[l]);
    for (int i = 0; i < fan[l] * outs[l]; ++i) p[q++] = (float)((2.0 * uni() - 1.0) * lim);
    q += outs[l];
  }
  s = tpg_mlp_set_params(m, p.data());
  if (s != TPG_OK) {
    tpg_mlp_free(m);
    return s;
  }
  *out = m;
  return TPG_OK;
}

void tpg_mlp_free(tpg_mlp* m) {
  if (!m) return;
  (void)hipSetDevice(m->device);
  if (m->st) (void)hipStreamSynchronize(m->st);
  if (m->master) (void)hipFree(m->master);
  if (m->w1b) (void)hipFree(m->w1b);
  if (m->mean) (void)hipFree(m->mean);
  if (m->act) (void)hipFree(m->act);
  if (m->host) (void)hipHostFree(m->host);
  if (m->st) (void)hipStreamDestroy(m->st);
  delete m;
}

tpg_status tpg_mlp_set_params(tpg_mlp* m, const float* params) {
  if (!m || !params) return fail(TPG_ERR_INVALID_ARG, "NULL argument");
  std::vector<float> blk;
  unpack_params(params, blk);
  TPG_HIP(hipSetDevice(m->device));
  // a step that returned no loss may still be at work on the parameters
  TPG_HIP(hipStreamSynchronize(m->st));
  TPG_HIP(hipMemcpy(m->master, blk.data(), sizeof(float) * oEnd, hipMemcpyHostToDevice));
  TPG_HIP(hipMemsetAsync(m->mom, 0, sizeof(float) * 2 * oEnd, m->st));
  m->step = 0;
  TPG_TRY(refresh_bf16(m));
  TPG_HIP(hipStreamSynchronize(m->st));
  return TPG_OK;
}

tpg_status tpg_mlp_get_params(const tpg_mlp* m, float* params) {
  if (!m || !params) return fail(TPG_ERR_INVALID_ARG, "NULL argument");
  std::vector<float> blk(oEnd);
  TPG_HIP(hipStreamSynchronize(m->st));
  TPG_HIP(hipMemcpy(blk.data(), m->master, sizeof(float) * oEnd, hipMemcpyDeviceToHost));
  pack_params(blk.data(), params);
  return TPG_OK;
}

tpg_status tpg_mlp_set_normalizer(tpg_mlp* m, const float* mean, const float* stdv) {
  if (!m || !mean || !stdv) return fail(TPG_ERR_INVALID_ARG, "NULL argument");
  for (int i = 0; i < kIn; ++i) {
    m->h_mean[i] = mean[i];
    m->h_std[i] = stdv[i] > 1e-12f ? stdv[i] : 1.f;
  }
  TPG_HIP(hipStreamSynchronize(m->st));  // as for the parameters
  TPG_HIP(hipMemcpy(m->mean, m->h_mean, sizeof(float) * kIn, hipMemcpyHostToDevice));
  TPG_HIP(hipMemcpy(m->stdv, m->h_std, sizeof(float) * kIn, hipMemcpyHostToDevice));
  return TPG_OK;
}

tpg_status tpg_mlp_forward(tpg_mlp* m, const float* x, int32_t n, float* y) {
  if (!m || !x || !y || n < 1) return fail(TPG_ERR_INVALID_ARG, "bad argument");
  TPG_HIP(hipSetDevice(m->device));
  RowArgs g;
  TPG_TRY(run_rows(m, x, nullptr, n, g));
  TPG_TRY(mlp_down(m, y, m->y, (size_t)n * kOut));
  m->busy = false;
  return TPG_OK;
}

tpg_status tpg_mlp_gradients(tpg_mlp* m, const float* x, const float* t, int32_t n, float* grad,
                             float* loss) {
  if (!m || !x || !t || n < 1) return fail(TPG_ERR_INVALID_ARG, "bad argument");
  TPG_HIP(hipSetDevice(m->device));
  RowArgs g;
  TPG_TRY(run_rows(m, x, t, n, g));
  TPG_TRY(run_backward(m, g));
  float* back = nullptr;
  TPG_TRY(mlp_take(m, oEnd + 1, &back));
  std::vector<float> own;
  if (!back) {
    own.resize(oEnd + 1);
    back = own.data();
  }
  if (grad) TPG_HIP(hipMemcpyAsync(back, m->grad, sizeof(float) * oEnd, hipMemcpyDeviceToHost, m->st));
  if (loss)
    TPG_HIP(hipMemcpyAsync(back + oEnd, m->loss, sizeof(float), hipMemcpyDeviceToHost, m->st));
  TPG_HIP(hipStreamSynchronize(m->st));
  m->busy = false;
  if (grad) pack_params(back, grad);
  if (loss) *loss = back[oEnd];
  return TPG_OK;
}

tpg_status tpg_mlp_train_step(tpg_mlp* m, const float* x, const float* t, int32_t n, float lr,
                              float* loss) {
  if (!m || !x || !t || n < 1) return fail(TPG_ERR_INVALID_ARG, "bad argument");
  TPG_HIP(hipSetDevice(m->device));
  RowArgs g;
  TPG_TRY(run_rows(m, x, t, n, g));
  TPG_TRY(run_backward(m, g));
  m->step += 1;
  AdamArgs a{};
  a.w = m->master;
  a.m = m->mom;
  a.v = m->mom + oEnd;
  a.g = m->grad;
  a.n = (int)oEnd;
  a.lr = lr;
  a.b1 = 0.9f;
  a.b2 = 0.999f;
  a.eps = 1e-8f;
  a.c1 = (float)(1.0 - std::pow(0.9, (double)m->step));
  a.c2 = (float)(1.0 - std::pow(0.999, (double)m->step));
  k_adam<<<(unsigned)((oEnd + 255) / 256), 256, 0, m->st>>>(a);
  TPG_HIP(hipGetLastError());
  TPG_TRY(refresh_bf16(m));
  if (loss) {
    TPG_TRY(mlp_down(m, loss, m->loss, 1));
    m->busy = false;
  }
  return TPG_OK;
}

// File: "TPGMLP1\n", int32 n_params, 32 means, 32 stds, n_params fp32 values.
tpg_status tpg_mlp_save(const tpg_mlp* m, const char* path) {
  if (!m || !path) return fail(TPG_ERR_INVALID_ARG, "NULL argument");
  std::vector<float> p(TPG_MLP_NPARAMS_);
  TPG_TRY(tpg_mlp_get_params(m, p.data()));
  FILE* f = fopen(path, "wb");
  if (!f) return fail(TPG_ERR_INVALID_ARG, "cannot open %s", path);
  const int32_t np = TPG_MLP_NPARAMS_;
  bool ok = fwrite("TPGMLP1\n", 1, 8, f) == 8 && fwrite(&np, 4, 1, f) == 1 &&
            fwrite(m->h_mean, 4, kIn, f) == (size_t)kIn && fwrite(m->h_std, 4, kIn, f) == (size_t)kIn &&
            fwrite(p.data(), 4, p.size(), f) == p.size();
  ok = (fclose(f) == 0) && ok;
  return ok ? TPG_OK : fail(TPG_ERR_INVALID_ARG, "write failed: %s", path);
}

tpg_status tpg_mlp_load(int32_t device, const char* path, tpg_mlp** out) {
  if (!path || !out) return fail(TPG_ERR_INVALID_ARG, "NULL argument");
  *out = nullptr;
  FILE* f = fopen(path, "rb");
  if (!f) return fail(TPG_ERR_INVALID_ARG, "cannot open %s", path);
  char magic[8];
  int32_t np = 0;
  float mean[kIn], stdv[kIn];
  std::vector<float> p(TPG_MLP_NPARAMS_);
  bool ok = fread(magic, 1, 8, f) == 8 && memcmp(magic, "TPGMLP1\n", 8) == 0 &&
            fread(&np, 4, 1, f) == 1 && np == TPG_MLP_NPARAMS_ &&
            fread(mean, 4, kIn, f) == (size_t)kIn && fread(stdv, 4, kIn, f) == (size_t)kIn &&
            fread(p.data(), 4, p.size(), f) == p.size();
  fclose(f);
  if (!ok) return fail(TPG_ERR_INVALID_ARG, "%s is not a predictor file", path);
  tpg_mlp* m = nullptr;
  TPG_TRY(tpg_mlp_create(device, 0, &m));
  tpg_status s = tpg_mlp_set_params(m, p.data());
  if (s == TPG_OK) s = tpg_mlp_set_normalizer(m, mean, stdv);
  if (s != TPG_OK) {
    tpg_mlp_free(m);
    return s;
  }
  *out = m;
  return TPG_OK;
}

}  // extern "C"
