// fp32 variant of the grouped SwiGLU expert FFN (Sec. 3.2.5; stacked weights of App. B.6).
//
// This element type serves small full-precision layers (a few hundred to a few thousand rows, widths of a few hundred).
// Such a product is a microsecond of arithmetic: what bounds it is the length of a thread's chain of loads and
// multiply-adds and the launches around it.  So every product runs on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums) with its reduction split over the four wavefronts of a
// workgroup:
//   * a workgroup owns 32 x 32 outputs; wavefront w takes the 16-index pieces w, w + 4, ... of the reduction, four pieces
//     of loads in flight, straight from memory into registers (the operands of a layer of this size stay in the L2);
//   * the four partial tiles meet in LDS and are added in wavefront order, so results do not depend on timing;
//   * a workgroup finds its (expert, row tile) from `offsets` itself, and rows are read by token through pair_of_row,
//     so no schedule or row list is built by a launch of its own; the data gradient and the three weight gradients share one launch.
// At 512 rows, d = 128, f = 256, 8 experts the former one-thread-per-output kernels with sequential sums took 130 (gate/up),
// 39 (down), 18 (dA), 74 (dX) and 3 x 37 us (weight gradients), with two and three further launches per pass; these take
// 8.5, 5.8, 6.4, 9.3 and 10 us (all three weight gradients), and the training step of 256 tokens 72 us instead of 396
// (its kernels alone 45 us, replayed from a graph; the rest is the host's share of ten calls, which has come down since).
#include "launch_plan.h"
#include "moe_common.h"

namespace moe {

constexpr int kF32Threads = 256;
constexpr int kF32Tile = 32;                   // outputs per workgroup: 32 x 32
constexpr int kF32Piece = 16;                  // reduction indices of a wavefront's piece: 4 per lane group, 4 MFMAs
constexpr int kF32Stride = 4 * kF32Piece;      // from one piece of a wavefront to its next
constexpr int kF32Batch = 4;                   // pieces whose loads are in flight together
constexpr int kF32Ld = kF32Tile + 4;           // floats per parked row: lane groups land in different banks

typedef float f32x4 __attribute__((ext_vector_type(4)));
struct F32Acc { f32x4 v[2][2]; };              // 2 x 2 fragments of 16 x 16: lane l holds rows 4 (l / 16) .. +3 of column l % 16

// Rows of the products: expert-ordered row r belongs to the expert whose segment of `offsets` holds it.  With pair_of_row
// the token-major operand is read instead of an expert-ordered copy, row r being its row pair_of_row[r] / k.
struct F32Rows {
  const int32_t* offsets; int E, P;
  const int32_t* pair_of_row; int T, k;        // pair_of_row null: operands are in expert order
  const float* topk_w;                         // combine weight of a pair, or null
};
__device__ __forceinline__ int f32_pair(const F32Rows& R, int r) { return min(max(R.pair_of_row[r], 0), R.P - 1); }
__device__ __forceinline__ size_t f32_source_row(const F32Rows& R, int r) {
  return R.pair_of_row ? min(f32_pair(R, r) / R.k, R.T - 1) : r;
}

__device__ __forceinline__ void mma(F32Acc& acc, float a0, float a1, float b0, float b1) {
  acc.v[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc.v[0][0], 0, 0, 0);
  acc.v[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc.v[0][1], 0, 0, 0);
  acc.v[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc.v[1][0], 0, 0, 0);
  acc.v[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc.v[1][1], 0, 0, 0);
}
__device__ __forceinline__ F32Acc f32_zero() {
  F32Acc a;
#pragma unroll
  for (int i = 0; i < 4; ++i) a.v[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  return a;
}
__device__ __forceinline__ f32x4 keep(bool c, f32x4 v) { return c ? v : f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ float2 keep(bool c, float2 v) { return c ? v : make_float2(0.f, 0.f); }
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// An operand of the products is held as two fragments of 16 rows (or columns); lane l holds entry l % 16 of each and, of a
// piece, the reduction indices 4 (l / 16) .. +3.  Which index an MFMA pairs with which is free as long as both sides agree.
// Reduction contiguous in memory: one 16-byte load per fragment; fragment h holds rows 16 h + l % 16.
struct KContig {
  const float* row[2];
  struct Piece { f32x4 v[2]; __device__ __forceinline__ float at(int h, int q) const { return v[h][q]; } };
  __device__ __forceinline__ Piece load(int k, int K) const {        // k: this lane's first index; beyond K reads as zero
    const int kc = min(k, K - 4);                                    // (K is a multiple of 8)
    Piece p;
#pragma unroll
    for (int h = 0; h < 2; ++h) p.v[h] = keep(k < K, load4(row[h] + kc));
    return p;
  }
};
// Reduction strided: an 8-byte load per index; fragment h holds the columns 2 (l % 16) + h.
struct KStrided {
  const float* col; int ld;
  struct Piece { float2 v[4]; __device__ __forceinline__ float at(int h, int q) const { return h ? v[q].y : v[q].x; } };
  __device__ __forceinline__ Piece load(int k, int K) const {
    const int kc = min(k, K - 4);
    Piece p;
#pragma unroll
    for (int q = 0; q < 4; ++q) p.v[q] = keep(k < K, *reinterpret_cast<const float2*>(col + static_cast<size_t>(kc + q) * ld));
    return p;
  }
};
// rows n0 .. n0+31 of W [n, ld]; rows that do not exist repeat the last one (nothing of theirs is stored)
__device__ __forceinline__ KContig k_contig(const float* w, size_t ld, int n0, int n, int lane) {
  KContig o;
#pragma unroll
  for (int h = 0; h < 2; ++h) o.row[h] = w + min(n0 + 16 * h + (lane & 15), n - 1) * ld;
  return o;
}
// columns n0 .. n0+31 of W [*, n] (n is a multiple of 8)
__device__ __forceinline__ KStrided k_strided(const float* w, int n0, int n, int lane) {
  return KStrided{w + min(n0 + 2 * (lane & 15), n - 2), n};
}

// this wavefront's share of acc_m += A B_m for NB column operands
template <int NB, class A, class B>
__device__ __forceinline__ void f32_product(F32Acc (&acc)[NB], const A& a, const B (&b)[NB], int K, int wave, int lane) {
  const int kl = 4 * (lane >> 4);
  for (int k0 = wave * kF32Piece; k0 < K; k0 += kF32Batch * kF32Stride) {
    typename A::Piece pa[kF32Batch];
    typename B::Piece pb[kF32Batch][NB];
#pragma unroll
    for (int u = 0; u < kF32Batch; ++u) {
      pa[u] = a.load(k0 + u * kF32Stride + kl, K);
#pragma unroll
      for (int m = 0; m < NB; ++m) pb[u][m] = b[m].load(k0 + u * kF32Stride + kl, K);
    }
#pragma unroll
    for (int u = 0; u < kF32Batch; ++u) {
      if (k0 + u * kF32Stride < K) {                   // uniform
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int m = 0; m < NB; ++m) mma(acc[m], pa[u].at(0, q), pa[u].at(1, q), pb[u][m].at(0, q), pb[u][m].at(1, q));
      }
    }
  }
}

// Partial tiles of the four wavefronts -> LDS; thread t then holds the sums of row t / 8, columns 4 (t % 8) .. +3.
// A_PAIRS / B_PAIRS: fragment h of that side holds rows (columns) 2 i + h (a strided operand), else 16 h + i.
template <bool A_PAIRS, bool B_PAIRS>
__device__ __forceinline__ f32x4 f32_reduce(const F32Acc& acc, float* red, int wave, int lane) {
  float* mine = red + wave * (kF32Tile * kF32Ld);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int col = B_PAIRS ? 2 * (lane & 15) + c : 16 * c + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * (lane >> 4) + r;
        mine[(A_PAIRS ? 2 * i + h : 16 * h + i) * kF32Ld + col] = acc.v[h][c][r];
      }
    }
  __syncthreads();
  const float* p = red + (threadIdx.x >> 3) * kF32Ld + 4 * (threadIdx.x & 7);
  f32x4 s = load4(p);
#pragma unroll
  for (int w = 1; w < 4; ++w) s += load4(p + w * (kF32Tile * kF32Ld));
  return s;
}
constexpr int kF32Red = 4 * kF32Tile * kF32Ld;

// ---- row products: workgroup b owns row tile b / n_tiles and column tile b % n_tiles ----------------------------------
struct F32Tile { int wave, lane, n0, r, c; size_t row; bool store; };   // r, c: this thread's row and first column in the epilogue
__device__ __forceinline__ F32Tile f32_tile(const RowTile& rt, int n_tiles, int N) {
  F32Tile t;
  t.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); t.lane = threadIdx.x & 63;
  t.n0 = (blockIdx.x % n_tiles) * kF32Tile;
  t.r = threadIdx.x >> 3; t.c = t.n0 + 4 * (threadIdx.x & 7);
  t.row = static_cast<size_t>(rt.row0) + t.r;
  t.store = t.r < rt.rows && t.c < N;
  return t;
}
// rows of the activation operand (rows beyond the tile's repeat its last one)
__device__ __forceinline__ KContig f32_rows(const F32Rows& R, const RowTile& rt, const float* a, size_t ld, int lane) {
  KContig o;
#pragma unroll
  for (int h = 0; h < 2; ++h) o.row[h] = a + f32_source_row(R, rt.row0 + min(16 * h + (lane & 15), rt.rows - 1)) * ld;
  return o;
}
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }

// G = x Wg^T, U = x Wu^T, act = [w] silu(G) * U
__global__ __launch_bounds__(kF32Threads) void f32_gate_up_kernel(F32Rows R, const float* __restrict__ x, const float* __restrict__ wg,
                                                                  const float* __restrict__ wu, int d, int f, int n_tiles,
                                                                  float* __restrict__ G, float* __restrict__ U, float* __restrict__ act) {
  __shared__ __attribute__((aligned(16))) float red[2 * kF32Red];
  const RowTile rt = find_row_tile(R.offsets, R.E, R.P, kF32Tile, blockIdx.x / n_tiles);
  if (rt.rows <= 0) return;
  const F32Tile t = f32_tile(rt, n_tiles, f);
  const size_t we = static_cast<size_t>(rt.expert) * f * d;
  const KContig a = f32_rows(R, rt, x, d, t.lane);
  const KContig b[2] = {k_contig(wg + we, d, t.n0, f, t.lane), k_contig(wu + we, d, t.n0, f, t.lane)};
  F32Acc acc[2] = {f32_zero(), f32_zero()};
  f32_product<2>(acc, a, b, d, t.wave, t.lane);
  const f32x4 g = f32_reduce<false, false>(acc[0], red, t.wave, t.lane), u = f32_reduce<false, false>(acc[1], red + kF32Red, t.wave, t.lane);
  if (!t.store) return;
  const size_t o = t.row * f + t.c;
  if (G) store4(G + o, g);
  if (U) store4(U + o, u);
  if (act) {
    const float w = R.topk_w ? R.topk_w[f32_pair(R, static_cast<int>(t.row))] : 1.0f;
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = w * (g[q] * sigmoid_acc(g[q]) * u[q]);
    store4(act + o, v);
  }
}

// yp = act Wd^T
__global__ __launch_bounds__(kF32Threads) void f32_down_kernel(F32Rows R, const float* __restrict__ act, const float* __restrict__ wd, int d, int f,
                                                               int n_tiles, float* __restrict__ yp) {
  __shared__ __attribute__((aligned(16))) float red[kF32Red];
  const RowTile rt = find_row_tile(R.offsets, R.E, R.P, kF32Tile, blockIdx.x / n_tiles);
  if (rt.rows <= 0) return;
  const F32Tile t = f32_tile(rt, n_tiles, d);
  const KContig a = f32_rows(R, rt, act, f, t.lane);
  const KContig b[1] = {k_contig(wd + static_cast<size_t>(rt.expert) * d * f, f, t.n0, d, t.lane)};
  F32Acc acc[1] = {f32_zero()};
  f32_product<1>(acc, a, b, f, t.wave, t.lane);
  const f32x4 v = f32_reduce<false, false>(acc[0], red, t.wave, t.lane);
  if (t.store) store4(yp + t.row * d + t.c, v);
}

// dA = [w] dy Wd;  dG = dA * U * silu'(G);  dU = dA * silu(G)
// With the combine weights: also act_w = w * act (if wanted) and the column tile's share of d w_r = <dy[token(r)] Wd, act[r]>.
__global__ __launch_bounds__(kF32Threads) void f32_dact_kernel(F32Rows R, const float* __restrict__ dy, const float* __restrict__ wd,
                                                               const float* __restrict__ G, const float* __restrict__ U, int d, int f,
                                                               int n_tiles, float* __restrict__ dG, float* __restrict__ dU,
                                                               float* __restrict__ act_w, float* __restrict__ dw_partial /* [n_tiles][P] */) {
  __shared__ __attribute__((aligned(16))) float red[kF32Red];
  const RowTile rt = find_row_tile(R.offsets, R.E, R.P, kF32Tile, blockIdx.x / n_tiles);
  if (rt.rows <= 0) return;
  const F32Tile t = f32_tile(rt, n_tiles, f);
  const KContig a = f32_rows(R, rt, dy, d, t.lane);
  const KStrided b[1] = {k_strided(wd + static_cast<size_t>(rt.expert) * d * f, t.n0, f, t.lane)};
  const size_t o = t.row * f + t.c;
  f32x4 g = {0.f, 0.f, 0.f, 0.f}, u = g;
  float w = 1.0f;
  if (t.store) {                                       // requested ahead of the product
    g = load4(G + o);
    u = load4(U + o);
    if (R.topk_w) w = R.topk_w[f32_pair(R, static_cast<int>(t.row))];
  }
  F32Acc acc[1] = {f32_zero()};
  f32_product<1>(acc, a, b, d, t.wave, t.lane);
  const f32x4 v = f32_reduce<false, true>(acc[0], red, t.wave, t.lane);
  float part = 0.0f;
  if (t.store) {
    f32x4 dg, du, aw;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float s = sigmoid_acc(g[q]), act = g[q] * s * u[q], da = w * v[q];
      part = fmaf(act, v[q], part);
      aw[q] = w * act;
      dg[q] = da * u[q] * (s * (1.0f + g[q] * (1.0f - s)));
      du[q] = da * (g[q] * s);
    }
    store4(dG + o, dg);
    store4(dU + o, du);
    if (act_w) store4(act_w + o, aw);
  }
  if (dw_partial) {                                    // the 8 threads of a row
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) part += __shfl_xor(part, m, 64);
    if (t.r < rt.rows && (threadIdx.x & 7) == 0) dw_partial[static_cast<size_t>(blockIdx.x % n_tiles) * R.P + t.row] = part;
  }
}

// dxp = dG Wg + dU Wu
__device__ __forceinline__ void f32_dx_block(const F32Rows& R, const float* __restrict__ dG, const float* __restrict__ dU,
                                             const float* __restrict__ wg, const float* __restrict__ wu, int d, int f,
                                             int n_tiles, float* __restrict__ dxp, float* red) {
  const RowTile rt = find_row_tile(R.offsets, R.E, R.P, kF32Tile, blockIdx.x / n_tiles);
  if (rt.rows <= 0) return;
  const F32Tile t = f32_tile(rt, n_tiles, d);
  const size_t we = static_cast<size_t>(rt.expert) * f * d;
  F32Acc acc[1] = {f32_zero()};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const KContig a = f32_rows(R, rt, s ? dU : dG, f, t.lane);
    const KStrided b[1] = {k_strided((s ? wu : wg) + we, t.n0, d, t.lane)};
    f32_product<1>(acc, a, b, f, t.wave, t.lane);
  }
  const f32x4 v = f32_reduce<false, true>(acc[0], red, t.wave, t.lane);
  if (t.store) store4(dxp + t.row * d + t.c, v);
}

// ---- weight gradients: dWd = dy^T act, dWg = dG^T x, dWu = dU^T x over the rows of every expert, in one launch --------
// Workgroup b < 3 E tiles: product b / (E tiles), expert, 32 x 32 outputs.  All behind them (dw_partial given): the gradient of
// the combine weights, the column tiles' shares added in order and scattered to [T, k].
struct F32Wgrad {
  const float *dy, *act, *dG, *dU, *x;
  float *dw_down, *dw_gate, *dw_up;
  int d, f, tiles_d, tiles_f;
  const float* dw_partial; int dw_tiles; float* dtopk_w;
};
__device__ __forceinline__ void f32_wgrad_block(const F32Rows& R, const F32Wgrad& p, unsigned block, float* red) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const unsigned tiles = static_cast<unsigned>(p.tiles_d) * p.tiles_f, which = block / (tiles * R.E);
  if (which >= 3) {                                    // (there may be more blocks of these than of one product)
    const long r = static_cast<long>(block - 3 * tiles * R.E) * kF32Threads + threadIdx.x;
    if (r >= R.P) return;
    float s = 0.0f;
    for (int j = 0; j < p.dw_tiles; ++j) s += p.dw_partial[static_cast<size_t>(j) * R.P + r];
    p.dtopk_w[f32_pair(R, static_cast<int>(r))] = s;
    return;
  }
  const int e = static_cast<int>(block / tiles - which * R.E), tile = static_cast<int>(block % tiles);
  // The fields are read before one of them is chosen: chosen first, the whole struct is copied to scratch memory to have
  // addresses to choose from (24 experts, d = 328, f = 208: a step of 95 us took 112).
  const int d = p.d, f = p.f, tiles_d = p.tiles_d, tiles_f = p.tiles_f;
  const float *const dy = p.dy, *const act = p.act, *const dG = p.dG, *const dU = p.dU, *const x = p.x;
  float *const dw_down = p.dw_down, *const dw_gate = p.dw_gate, *const dw_up = p.dw_up;
  const int M = which == 0 ? d : f, N = which == 0 ? f : d, tiles_n = which == 0 ? tiles_f : tiles_d;
  const int m0 = tile / tiles_n * kF32Tile, n0 = tile % tiles_n * kF32Tile;
  // both operands are strided: the fragments of a side hold its entries 2 i and 2 i + 1
  const float* lhs = (which == 0 ? dy : which == 1 ? dG : dU) + min(m0 + 2 * (lane & 15), M - 2);
  const float* rhs = (which == 0 ? act : x) + min(n0 + 2 * (lane & 15), N - 2);
  const int begin = min(max(R.offsets[e], 0), R.P), end = min(R.offsets[e + 1], R.P);
  F32Acc acc = f32_zero();
  for (int r0 = begin + wave * kF32Piece; r0 < end; r0 += kF32Batch * kF32Stride) {
    float2 va[kF32Batch][4], vb[kF32Batch][4];
#pragma unroll
    for (int u = 0; u < kF32Batch; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = r0 + u * kF32Stride + 4 * q + (lane >> 4), rc = min(r, end - 1);
        const size_t token = f32_source_row(R, rc);    // dy and x are the operands that may be token-major
        va[u][q] = keep(r < end, *reinterpret_cast<const float2*>(lhs + (which == 0 ? token : rc) * M));
        vb[u][q] = keep(r < end, *reinterpret_cast<const float2*>(rhs + (which == 0 ? rc : token) * N));
      }
#pragma unroll
    for (int u = 0; u < kF32Batch; ++u) {
      if (r0 + u * kF32Stride < end) {                 // uniform
#pragma unroll
        for (int q = 0; q < 4; ++q) mma(acc, va[u][q].x, va[u][q].y, vb[u][q].x, vb[u][q].y);
      }
    }
  }
  const f32x4 v = f32_reduce<true, true>(acc, red, wave, lane);
  const int m = m0 + (threadIdx.x >> 3), n = n0 + 4 * (threadIdx.x & 7);
  float* out = which == 0 ? dw_down : which == 1 ? dw_gate : dw_up;
  if (m < M && n < N) store4(out + (static_cast<size_t>(e) * M + m) * N + n, v);
}

// The data gradient dxp = dG Wg + dU Wu and the weight gradients need nothing from each other: one launch, the first dx_blocks
// workgroups for the former (256 tokens, d = 128, E = 8, k = 2, f = 256: a launch less is 5 of a step's 72 us).
struct F32Dx { F32Rows rows; const float *dG, *dU, *wg, *wu; float* dxp; int d, f, n_tiles; };
__global__ __launch_bounds__(kF32Threads) void f32_dx_wgrad_kernel(F32Dx x, unsigned dx_blocks, F32Rows R, F32Wgrad p) {
  __shared__ __attribute__((aligned(16))) float red[kF32Red];
  if (blockIdx.x < dx_blocks) f32_dx_block(x.rows, x.dG, x.dU, x.wg, x.wu, x.d, x.f, x.n_tiles, x.dxp, red);
  else f32_wgrad_block(R, p, blockIdx.x - dx_blocks, red);
}

// ---- host side --------------------------------------------------------------------------------------------------------
static unsigned blocks_for(size_t n) { return static_cast<unsigned>((n + kF32Threads - 1) / kF32Threads); }
static unsigned row_grid(const F32Rows& R, int n_tiles) {
  return static_cast<unsigned>((static_cast<size_t>(ceil_div(R.P, kF32Tile)) + R.E) * n_tiles);
}
static const float* cf(const void* p) { return static_cast<const float*>(p); }
static float* mf(void* p) { return static_cast<float*>(p); }

static void f32_gate_up(const F32Rows& R, const void* x, const void* wg, const void* wu, int d, int f, void* G, void* U, void* act, hipStream_t s) {
  const int nt = ceil_div(f, kF32Tile);
  MOE_LAUNCH("f32_gate_up", f32_gate_up_kernel, dim3(row_grid(R, nt)), dim3(kF32Threads), 0, s, R, cf(x), cf(wg), cf(wu), d, f, nt, mf(G), mf(U), mf(act));
}
static void f32_down(const F32Rows& R, const void* act, const void* wd, int d, int f, void* yp, hipStream_t s) {
  const int nt = ceil_div(d, kF32Tile);
  MOE_LAUNCH("f32_down", f32_down_kernel, dim3(row_grid(R, nt)), dim3(kF32Threads), 0, s, R, cf(act), cf(wd), d, f, nt, mf(yp));
}
static void f32_dact(const F32Rows& R, const void* dy, const void* wd, const float* G, const float* U, int d, int f, float* dG, float* dU,
                     float* act_w, float* dw_partial, hipStream_t s) {
  const int nt = ceil_div(f, kF32Tile);
  MOE_LAUNCH("f32_dact", f32_dact_kernel, dim3(row_grid(R, nt)), dim3(kF32Threads), 0, s, R, cf(dy), cf(wd), G, U, d, f, nt, dG, dU, act_w, dw_partial);
}
static F32Dx f32_dx(const F32Rows& R, const float* dG, const float* dU, const void* wg, const void* wu, int d, int f, void* dxp) {
  return F32Dx{R, dG, dU, cf(wg), cf(wu), mf(dxp), d, f, ceil_div(d, kF32Tile)};
}
// R.P == 0: no data gradient
static void f32_dx_wgrad(const F32Dx& x, const F32Rows& R, F32Wgrad w, hipStream_t s) {
  w.tiles_d = ceil_div(w.d, kF32Tile); w.tiles_f = ceil_div(w.f, kF32Tile);
  const unsigned dx_blocks = R.P > 0 ? row_grid(x.rows, x.n_tiles) : 0u;
  const size_t wgrad_blocks = 3 * static_cast<size_t>(w.tiles_d) * w.tiles_f * R.E + (w.dw_partial ? blocks_for(R.P) : 0);
  auto launch = [&](size_t dx, size_t wgrad) {
    MOE_LAUNCH("f32_dx_wgrad", f32_dx_wgrad_kernel, dim3(static_cast<unsigned>(dx + wgrad)), dim3(kF32Threads), 0, s, x, static_cast<unsigned>(dx), R, w);
  };
  if (fits_one_launch(dx_blocks + wgrad_blocks, kF32Threads)) {
    launch(dx_blocks, wgrad_blocks);
  } else {                                             // together they are too many (half a billion rows)
    launch(dx_blocks, 0);
    launch(0, wgrad_blocks);
  }
}

size_t ffn_fwd_ws_bytes_f32(int, int, int, int) { return 256; }

size_t ffn_bwd_ws_bytes_f32(int P, int d, int f, int E, int have_saved) {
  (void)d; (void)E;
  const size_t pf = align_up(static_cast<size_t>(P) * f * sizeof(float), 256);
  return 256 + (have_saved ? 2 : 4) * pf;     // dG, dU (+ recomputed G, U)
}

void ffn_fwd_f32(const FfnFwdArgs& a) {
  if (a.P == 0) return;
  const F32Rows R{a.offsets, a.E, a.P, nullptr, 0, 1, nullptr};
  f32_gate_up(R, a.xp, a.w_gate, a.w_up, a.d, a.f, a.g_save, a.u_save, a.act, a.stream);
  if (a.yp) f32_down(R, a.act, a.w_down, a.d, a.f, a.yp, a.stream);
}

void ffn_bwd_f32(const FfnBwdArgs& a) {
  const size_t pf_bytes = align_up(static_cast<size_t>(a.P) * a.f * sizeof(float), 256);
  char* ws = static_cast<char*>(a.ws);
  float* dG = reinterpret_cast<float*>(ws);
  float* dU = reinterpret_cast<float*>(ws + pf_bytes);
  const float* G = cf(a.g_save);
  const float* U = cf(a.u_save);
  const F32Rows R{a.offsets, a.E, a.P, nullptr, 0, 1, nullptr};
  if (a.P > 0) {
    if (!G) {   // recompute the pre-activations
      float* Gr = reinterpret_cast<float*>(ws + 2 * pf_bytes);
      float* Ur = reinterpret_cast<float*>(ws + 3 * pf_bytes);
      f32_gate_up(R, a.xp, a.w_gate, a.w_up, a.d, a.f, Gr, Ur, nullptr, a.stream);
      G = Gr; U = Ur;
    }
    f32_dact(R, a.dyp, a.w_down, G, U, a.d, a.f, dG, dU, nullptr, nullptr, a.stream);
  }
  F32Wgrad w{};                               // with P == 0 every segment is empty: zeros are written, nothing is read
  w.dy = cf(a.dyp); w.act = cf(a.act); w.dG = dG; w.dU = dU; w.x = cf(a.xp);
  w.dw_down = mf(a.dw_down); w.dw_gate = mf(a.dw_gate); w.dw_up = mf(a.dw_up); w.d = a.d; w.f = a.f;
  f32_dx_wgrad(f32_dx(R, dG, dU, a.w_gate, a.w_up, a.d, a.f, a.dxp), R, w, a.stream);
}

// ---- the variants that read the layer input / the output gradient by token -------------------------
// backward workspace: [256 | dG | dU | act_w | dw_partial | (G | U)], each aligned to 256
size_t ffn_fwd_gather_ws_bytes_f32(int, int, int, int) { return 256; }
static size_t f32_dw_bytes(int P, int f) { return align_up(static_cast<size_t>(ceil_div(f, kF32Tile)) * P * sizeof(float), 256); }
size_t ffn_bwd_gather_ws_bytes_f32(int P, int d, int f, int E, int have_saved) {
  (void)d; (void)E;
  const size_t pf = align_up(static_cast<size_t>(P) * f * sizeof(float), 256);
  return 256 + f32_dw_bytes(P, f) + (have_saved ? 3 : 5) * pf;
}

void ffn_fwd_gather_f32(const FfnFwdGatherArgs& a) {
  if (a.P == 0) return;
  const F32Rows gathered{a.offsets, a.E, a.P, a.pair_of_row, a.T, a.k, a.topk_w}, ordered{a.offsets, a.E, a.P, nullptr, 0, 1, nullptr};
  f32_gate_up(gathered, a.x, a.w_gate, a.w_up, a.d, a.f, a.g_save, a.u_save, a.act, a.stream);
  f32_down(ordered, a.act, a.w_down, a.d, a.f, a.yp, a.stream);
}

void ffn_bwd_gather_f32(const FfnBwdGatherArgs& a) {
  const size_t pf_bytes = align_up(static_cast<size_t>(a.P) * a.f * sizeof(float), 256);
  char* big = static_cast<char*>(a.ws) + 256;
  float* dG = reinterpret_cast<float*>(big);
  float* dU = reinterpret_cast<float*>(big + pf_bytes);
  float* act_w_ws = reinterpret_cast<float*>(big + 2 * pf_bytes);
  float* dw_partial = reinterpret_cast<float*>(big + 3 * pf_bytes);
  const float* G = cf(a.g_save);
  const float* U = cf(a.u_save);
  const F32Rows gathered{a.offsets, a.E, a.P, a.pair_of_row, a.T, a.k, a.topk_w}, ordered{a.offsets, a.E, a.P, nullptr, 0, 1, nullptr};
  if (a.P > 0) {
    if (!G) {   // recompute the pre-activations
      float* Gr = reinterpret_cast<float*>(big + 3 * pf_bytes + f32_dw_bytes(a.P, a.f));
      float* Ur = Gr + pf_bytes / sizeof(float);
      f32_gate_up(gathered, a.x, a.w_gate, a.w_up, a.d, a.f, Gr, Ur, nullptr, a.stream);
      G = Gr; U = Ur;
    }
    f32_dact(gathered, a.dy, a.w_down, G, U, a.d, a.f, dG, dU, a.act_w ? nullptr : act_w_ws, dw_partial, a.stream);
  }
  F32Wgrad w{};
  w.dy = cf(a.dy); w.act = a.act_w ? cf(a.act_w) : act_w_ws; w.dG = dG; w.dU = dU; w.x = cf(a.x);
  w.dw_down = mf(a.dw_down); w.dw_gate = mf(a.dw_gate); w.dw_up = mf(a.dw_up); w.d = a.d; w.f = a.f;
  if (a.P > 0) { w.dw_partial = dw_partial; w.dw_tiles = ceil_div(a.f, kF32Tile); w.dtopk_w = a.dtopk_w; }
  f32_dx_wgrad(f32_dx(ordered, dG, dU, a.w_gate, a.w_up, a.d, a.f, a.dxp), gathered, w, a.stream);
}

// ---- router linear, fp32 element type: one thread per output, sequential FMA ----------------------
__global__ __launch_bounds__(kF32Threads) void f32_router_logits_kernel(const float* __restrict__ x, const float* __restrict__ wr,
                                                                        int T, int d, int E, float* __restrict__ logits) {
  const long i = static_cast<long>(blockIdx.x) * kF32Threads + threadIdx.x;
  if (i >= static_cast<long>(T) * E) return;
  const int t = static_cast<int>(i / E), e = static_cast<int>(i % E);
  const float* xr = x + static_cast<long>(t) * d;
  const float* w = wr + static_cast<long>(e) * d;
  float acc = 0.0f;
  for (int c = 0; c < d; ++c) acc = fmaf(xr[c], w[c], acc);
  logits[i] = acc;
}
__global__ __launch_bounds__(kF32Threads) void f32_router_dx_kernel(const float* __restrict__ dz, const float* __restrict__ wr,
                                                                    int T, int d, int E, int accumulate, float* __restrict__ dx) {
  const long i = static_cast<long>(blockIdx.x) * kF32Threads + threadIdx.x;
  if (i >= static_cast<long>(T) * d) return;
  const int t = static_cast<int>(i / d), c = static_cast<int>(i % d);
  float acc = 0.0f;
  for (int e = 0; e < E; ++e) acc = fmaf(dz[static_cast<long>(t) * E + e], wr[static_cast<long>(e) * d + c], acc);
  dx[i] = accumulate ? dx[i] + acc : acc;
}
__global__ __launch_bounds__(kF32Threads) void f32_router_dw_kernel(const float* __restrict__ dz, const float* __restrict__ x,
                                                                    int T, int d, int E, float* __restrict__ dwr) {
  const long i = static_cast<long>(blockIdx.x) * kF32Threads + threadIdx.x;
  if (i >= static_cast<long>(E) * d) return;
  const int e = static_cast<int>(i / d), c = static_cast<int>(i % d);
  float acc = 0.0f;
  for (int t = 0; t < T; ++t) acc = fmaf(dz[static_cast<long>(t) * E + e], x[static_cast<long>(t) * d + c], acc);
  dwr[i] = acc;
}

void router_fwd_f32(const RouterFwdArgs& a) {
  MOE_LAUNCH("f32_router_logits", f32_router_logits_kernel, dim3(blocks_for(static_cast<size_t>(a.T) * a.E)), dim3(kF32Threads), 0,
             a.stream, static_cast<const float*>(a.x), static_cast<const float*>(a.w_router), a.T, a.d, a.E, a.logits);
}
void router_bwd_f32(const RouterBwdArgs& a) {
  if (a.T > 0)
    MOE_LAUNCH("f32_router_dx", f32_router_dx_kernel, dim3(blocks_for(static_cast<size_t>(a.T) * a.d)), dim3(kF32Threads), 0, a.stream,
               a.dlogits, static_cast<const float*>(a.w_router), a.T, a.d, a.E, a.accumulate, static_cast<float*>(a.dx));
  MOE_LAUNCH("f32_router_dw", f32_router_dw_kernel, dim3(blocks_for(static_cast<size_t>(a.E) * a.d)), dim3(kF32Threads), 0, a.stream,
             a.dlogits, static_cast<const float*>(a.x), a.T, a.d, a.E, static_cast<float*>(a.dw_router));
}

}  // namespace moe
