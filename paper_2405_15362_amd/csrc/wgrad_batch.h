// A W pass in one launch: which workgroup does what, the column sums of its bias gradients, and the time that tiles of a shape take.
//
// The products of a W pass are independent, and most of them leave compute units idle at their end or, at a few hundred
// tokens, all along; each launch also costs a ramp of 3 to 5 us.  In one launch the last round is the pass's, not the product's, small
// tiles become affordable because their number adds up, and the workgroups that share a compute unit drift out of phase, so
// that one's read-modify-write of C runs under another's K loop.
#pragma once
#include <cmath>

#include "dev_common.h"
#include "kernels.h"

namespace pmc {
namespace k {

// Output tiles of one layer's four products.
inline long batch_tiles(const WgradBatchArgs& a, int bm, int bn) {
  long n = 0;
  for (int j = 0; j < 4; ++j) n += (long)((a.M[j] + bm - 1) / bm) * ((a.N[j] + bn - 1) / bn);
  return n;
}
// us of a batch: n tiles per compute unit at K tokens take a fixed time, the chain of one tile (per 1024 of K), a share of the
// compute unit per tile (per 1024 of K, and once), and the chain again for every round of tiles (per_cu workgroups run side by side).
// Beyond 3072 tokens a share of K costs more the longer K is: the passes are long enough for the chip's power limit, and the smaller the tile the
// more of its operands come from memory again (long_k, relative to the shape that costs least).
struct BatchTime {
  double fixed, chain_k, tile_k, tile, round_k, round;
  int per_cu;
  double long_k = 0.;
};
inline double batch_us(const BatchTime& t, double tiles, double K) {
  const double n = tiles / 256., k = K / 1024., rounds = (double)(long)((n + t.per_cu * 0.999999) / t.per_cu);
  const double tile_k = t.tile_k + (k > 3. ? t.long_k * std::log2(k / 3.) : 0.);
  return t.fixed + t.chain_k * k + n * (tile_k * k + t.tile) + rounds * (t.round_k * k + t.round);
}

// Column sums of 64 columns from col0 of `pieces` matrices [rows][n] (pitch lda) by 256 threads (tid): out[c] += the sum of each
// piece in turn.  The threads form 256/LPR row slots of LPR lanes (16 bytes of a row each); slot s adds rows s, s + slots, ...
// in that order (sixteen loads in flight), and 64 threads then add the slots in slot order: the result depends on the
// rows alone, whoever calls it.  red: 256 / LPR x 65 floats of LDS.  All threads of the workgroup call it together.
template <typename T, class PieceOf>
__device__ __forceinline__ void column_sum_block(PieceOf piece_of, int pieces, int rows, int n, int lda, int col0, float* out, float* red, int tid) {
  constexpr int V = Vec<T>::N, LPR = 64 / V, SLOTS = 256 / LPR, UNROLL = 16;
  const int slot = tid / LPR, sub = (tid % LPR) * V, col = col0 + sub, c = col0 + tid;
  float total = tid < 64 && c < n ? out[c] : 0.f;
  for (int s = 0; s < pieces; ++s) {
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    if (col < n) {
      const T* p = piece_of(s) + col;
      int r = slot;
      for (; r + (UNROLL - 1) * SLOTS < rows; r += UNROLL * SLOTS) {
        float v[UNROLL][V];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) Vec<T>::load(p + (size_t)(r + u * SLOTS) * lda, v[u]);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
          for (int i = 0; i < V; ++i) acc[i] += v[u][i];
      }
      for (; r < rows; r += SLOTS) {
        float v[V];
        Vec<T>::load(p + (size_t)r * lda, v);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] += v[i];
      }
    }
    if (s) __syncthreads();  // the sums of the piece before have been read
#pragma unroll
    for (int i = 0; i < V; ++i) red[slot * 65 + sub + i] = acc[i];
    __syncthreads();
    if (tid < 64) {
      float sum = 0.f;
#pragma unroll
      for (int sl = 0; sl < SLOTS; ++sl) sum += red[sl * 65 + tid];
      total += sum;
    }
  }
  if (tid < 64 && c < n) out[c] = total;
}

// Tile of a workgroup of the batch (block: its number behind the column-sum ones).  Ids are dealt round-robin over the 8
// XCDs: each XCD gets a contiguous run of tiles, walked in column groups group_m tall inside a product.
struct BatchTile {
  int layer, product, tile_m, tile_n;
};
__device__ __forceinline__ BatchTile batch_tile(const WgradBatchParams& q, int block) {
  const int per_layer = q.first_tile[4], ntiles = per_layer * q.w.layers;
  const int xcd = block & 7, lo = ntiles >> 3, rem = ntiles & 7;
  int t = xcd * lo + min(xcd, rem) + (block >> 3);
  BatchTile b;
  b.layer = t / per_layer;
  t -= b.layer * per_layer;
  b.product = (t >= q.first_tile[1]) + (t >= q.first_tile[2]) + (t >= q.first_tile[3]);
  t -= q.first_tile[b.product];
  const int tiles_n = q.tiles_n[b.product], tiles = q.first_tile[b.product + 1] - q.first_tile[b.product], tiles_m = tiles / tiles_n;
  const int per_group = q.group_m * tiles_n, group = t / per_group, in = t - group * per_group;
  const int height = min(tiles_m - group * q.group_m, q.group_m);
  b.tile_m = group * q.group_m + in % height;
  b.tile_n = in / height;
  return b;
}

// The bias-gradient share of a workgroup of the batch: 64 columns to every 256 threads.
template <typename T, int NT>
__device__ __forceinline__ void batch_column_sums(const WgradBatchParams& q, int block, float* smem) {
  static_assert(NT % 256 == 0, "256 threads to 64 columns");
  const int per_layer = q.first_sum[4];
  if (block >= per_layer * q.w.layers) return;  // the count is rounded up to whole rounds over the XCDs
  const int layer = block / per_layer, t = block - layer * per_layer;
  const int j = (t >= q.first_sum[1]) + (t >= q.first_sum[2]) + (t >= q.first_sum[3]);
  const WgradBatchArgs::Layer& l = q.w.layer[layer];
  const size_t off = l.b[j];
  const int part = threadIdx.x >> 8, n = q.w.N[j];
  column_sum_block<T>([&](int s) { return reinterpret_cast<const T*>(q.w.piece[s] + off); }, q.w.pieces, q.w.K, n, n,
                      64 * ((NT / 256) * (t - q.first_sum[j]) + part), l.bias[j], smem + part * (256 / (64 / Vec<T>::N)) * 65, threadIdx.x & 255);
}

}  // namespace k
}  // namespace pmc
