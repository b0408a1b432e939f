// fp32-mode GEMM on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32): fp32 products and fp32
// accumulation throughout, as PMC_F32 mode needs (results agree with the fp64 oracle to 1e-5).
//
// The instruction runs at 256 FLOP per clock and compute unit, 1/16 of the bf16 rate, so LDS and the
// load path are never near their limits; what bounds a product is how many compute units have a tile
// and how long the serial K chain of one tile is.  Three kernels:
//
//  * gemm_f32_tile_kernel: operand tiles go straight from global memory into an LDS ring
//    (buffer_load ... lds), waves are a WAVES_M x WAVES_N grid times WK groups that share K (each
//    group has its own ring and takes every WK-th 32-deep tile; the partial sums are added in group
//    order through LDS).  WK > 1 puts eight waves on an output tile too small for as many.
//  * gemm_f32_direct_kernel: a 16 x 16 output tile per workgroup, K dealt over its eight waves in
//    16-deep groups, operands loaded in the fragment layout without LDS (one memory latency per few
//    groups, no barrier before the final fold).  For products whose 32 x 32 tiles would leave most
//    compute units idle and, with element-wise loads, for small products of sizes, pitches or pointers
//    that are not multiples of four elements.
//  * gemm_f32_fma_kernel: 64 x 64 tiles of plain FMAs staged element by element through LDS, for the
//    larger products of such sizes and of operands of 2 GB and more: it reads an operand element once per
//    64 outputs, the direct kernel once per 16, one 4-byte load at a time.
//
// Measured against a 64 x 64 tile of plain FMAs with scalar loads (before), mean over the products of a
// pass, F / B / W: hidden 256, 128 tokens 65 / 74 / 23 -> 5.2 / 5.2 / 5.1 us; hidden 1024, 512 tokens
// 308 / 322 / 107 -> 41 / 37 / 40 us (about 90 TFLOP/s; the library's fp32 product reaches 154 at 8192^3).
//
// Both contract k in the same assignment: in a 16-deep group, lane quarter q = lane / 16 holds
// k = 4 q .. 4 q + 3 and instruction j takes element j of every quarter, so an operand whose
// contraction index is contiguous is read 16 bytes at a time.
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"
#include "wgrad_batch.h"

namespace pmc {
namespace k {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;

struct F32Params {
  const float* A;
  const float* B;
  float* C;
  const float* bias;
  const float* resid;
  float* aux;
  int M, N, K, lda, ldb, ldc, epi;
  int tiles_m, tiles_n;
};

__device__ __forceinline__ float apply_epilogue(const F32Params& p, float v, size_t idx, int n) {
  switch (p.epi) {
    case PMC_EPI_NONE: return v;
    case PMC_EPI_BIAS: return v + p.bias[n];
    case PMC_EPI_BIAS_RESID: return v + p.bias[n] + p.resid[idx];
    case PMC_EPI_BIAS_GELU: v += p.bias[n]; p.aux[idx] = gelu_f(v); return v;
    case PMC_EPI_DGELU: return v * gelu_grad_f(p.aux[idx]);
    case PMC_EPI_ACCUM_F32: return p.C[idx] + v;
    case PMC_EPI_BIAS_GELU_GRAD: v += p.bias[n]; p.aux[idx] = gelu_f(v); return gelu_grad_f(v);
    case PMC_EPI_MUL: return v * p.aux[idx];
  }
  return v;
}

// Four consecutive columns of one row; every pointer and pitch is a multiple of 16 bytes.
__device__ __forceinline__ void store_quad_f32(const F32Params& p, f32x4 v, int m, int n) {
  const size_t idx = (size_t)m * p.ldc + n;
  f32x4 out;
  if (p.epi == PMC_EPI_NONE) {
    out = v;
  } else if (p.epi == PMC_EPI_ACCUM_F32) {
    out = *reinterpret_cast<const f32x4*>(p.C + idx) + v;
  } else if (p.epi == PMC_EPI_MUL) {
    out = v * *reinterpret_cast<const f32x4*>(p.aux + idx);
  } else if (p.epi == PMC_EPI_DGELU) {
    const f32x4 u = *reinterpret_cast<const f32x4*>(p.aux + idx);
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = v[e] * gelu_grad_f(u[e]);
  } else {
    out = v + *reinterpret_cast<const f32x4*>(p.bias + n);
    if (p.epi == PMC_EPI_BIAS_RESID) {
      out += *reinterpret_cast<const f32x4*>(p.resid + idx);
    } else if (p.epi == PMC_EPI_BIAS_GELU || p.epi == PMC_EPI_BIAS_GELU_GRAD) {
      f32x4 g;
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = gelu_f(out[e]);
      *reinterpret_cast<f32x4*>(p.aux + idx) = g;
      if (p.epi == PMC_EPI_BIAS_GELU_GRAD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = gelu_grad_f(out[e]);
      }
    }
  }
  *reinterpret_cast<f32x4*>(p.C + idx) = out;
}

// One operand's 32-deep K tile in LDS, 128 bytes per row.  KMAJ (contraction contiguous): [rows][32],
// 16-byte chunk c of row r at position c ^ ((r >> 1) & 7), so 16 rows at one chunk hit 16 bank groups.
// Otherwise [32][ROWS] with the 64-byte spans of k-row k exchanged by (k >> 2) & 3, so that the four
// lane quarters of a fragment read (k-rows 4 apart) fall into different bank quarters.
// Rows past the edge are clamped (the epilogue does not store them); what lies past K is read as zero:
// [k][rows] tiles by the size of the buffer descriptor, [rows][k] tiles by an offset outside it.
template <int ROWS, bool KMAJ, int NW>
struct F32Loader {
  static constexpr int NL = ROWS / 8 / NW;  // 1 KB loads per wave and tile
  static_assert(ROWS % (8 * NW) == 0, "tile must split evenly over the waves");
  uint32_t voff[NL];
  int kc[KMAJ ? NL : 1];  // first k of this lane's chunk

  __device__ __forceinline__ static int swz(int k) { return ROWS >= 64 ? ((k >> 2) & 3) << 2 : ROWS == 32 ? ((k >> 2) & 1) << 2 : 0; }
  __device__ __forceinline__ void init(int ld, int mn0, int mn_total, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int q = wave * NL + i;
      if constexpr (KMAJ) {
        const int row = q * 8 + (lane >> 3);
        kc[i] = 4 * ((lane & 7) ^ ((row >> 1) & 7));
        voff[i] = ((uint32_t)min(mn0 + row, mn_total - 1) * (uint32_t)ld + kc[i]) * 4;
      } else {
        constexpr int CPR = ROWS / 4;
        const int idx = q * 64 + lane, kr = idx / CPR, chunk = (idx % CPR) ^ swz(kr);
        voff[i] = ((uint32_t)kr * (uint32_t)ld + min(mn0 + 4 * chunk, mn_total - 4)) * 4;
      }
    }
  }
  __device__ __forceinline__ void issue(i32x4 rsrc, float* tile, int k0, int K, uint32_t ld, int wave) const {
    const bool past = k0 >= K;  // a whole tile past the end
    const uint32_t soff = past ? 0u : KMAJ ? (uint32_t)k0 * 4 : (uint32_t)k0 * ld * 4;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)((lds_void_ptr)(tile + (wave * NL + i) * 256)));
      const uint32_t v = past || (KMAJ && k0 + kc[KMAJ ? i : 0] >= K) ? 0x80000000u : voff[i];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds_addr), "v"(v), "s"(rsrc), "s"(soff) : "memory");
    }
  }
  // Fragment of 16 rows from r0 for the 16-deep group c of the tile: element j is the operand of instruction j.
  __device__ __forceinline__ static f32x4 frag(const float* tile, int r0, int c, int lane) {
    const int row = r0 + (lane & 15), quarter = lane >> 4;
    if constexpr (KMAJ) {
      return *reinterpret_cast<const f32x4*>(tile + row * 32 + (((4 * c + quarter) ^ ((row >> 1) & 7)) << 2));
    } else {
      const float* t = tile + (16 * c + 4 * quarter) * ROWS + (row ^ (swz(4 * quarter) << 2));
      f32x4 v = {t[0], t[ROWS], t[2 * ROWS], t[3 * ROWS]};
      return v;
    }
  }
};

// Workgroup id -> tile, giving each of the 8 XCDs a contiguous run of tiles (ids are dealt round-robin)
// walked in column groups 8 tiles tall, so that neighbours share operand panels in one L2.
__device__ __forceinline__ void tile_of(const F32Params& p, int& tm, int& tn) {
  const int ntiles = p.tiles_m * p.tiles_n, pid0 = blockIdx.x;
  const int xcd = pid0 & 7, lo = ntiles >> 3, rem = ntiles & 7;
  const int pid = xcd * lo + min(xcd, rem) + (pid0 >> 3);
  const int per_group = 8 * p.tiles_n, group = pid / per_group, in = pid % per_group;
  const int height = min(p.tiles_m - 8 * group, 8);
  tm = 8 * group + in % height;
  tn = in / height;
}

// Output tile (tile_m, tile_n), by the whole workgroup.
template <int BM, int BN, int WAVES_M, int WAVES_N, int WK, int NSTAGE, bool A_KMAJ, bool B_KMAJ>
__device__ __forceinline__ void f32_tile(const F32Params& p, float* smem_f32, int tile_m, int tile_n) {
  constexpr int NW = WAVES_M * WAVES_N, TM = BM / WAVES_M / 16, TN = BN / WAVES_N / 16;
  constexpr int TA = 32 * BM, TB = 32 * BN, STAGE = TA + TB, RING = NSTAGE * STAGE;
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave_all / NW, wave = wave_all % NW;
  const int wm0 = (wave / WAVES_N) * (BM / WAVES_M), wn0 = (wave % WAVES_N) * (BN / WAVES_N);
  float* ring = smem_f32 + kg * RING;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  auto make_rsrc = [](const void* ptr, size_t bytes) {
    const uint64_t a = (uint64_t)ptr;
    i32x4 r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    return r;
  };
  const i32x4 ra = make_rsrc(p.A, (size_t)(A_KMAJ ? p.M : p.K) * p.lda * 4), rb = make_rsrc(p.B, (size_t)(B_KMAJ ? p.N : p.K) * p.ldb * 4);
  using LA = F32Loader<BM, A_KMAJ, NW>;
  using LB = F32Loader<BN, B_KMAJ, NW>;
  LA la;
  LB lb;
  la.init(p.lda, m0, p.M, wave, lane);
  lb.init(p.ldb, n0, p.N, wave, lane);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Tile t of this group is K tile t WK + kg.  Every group runs the same number of steps (tiles past
  // the end lie past K and read as zeros), so all waves meet at the same barriers and the number of
  // loads in flight is the same at every wait.
  const int nk = (p.K + 32 * WK - 1) / (32 * WK);
  auto request = [&](int t, int stage) {
    const int k0 = (min(t, nk - 1) * WK + kg) * 32;
    la.issue(ra, ring + stage * STAGE, k0, p.K, p.lda, wave);
    lb.issue(rb, ring + stage * STAGE + TA, k0, p.K, p.ldb, wave);
  };
  constexpr int INFL = (NSTAGE - 2) * (LA::NL + LB::NL);
  static_assert(INFL < 64, "vmcnt is a 6-bit field");
  constexpr int WAIT_TILE = (INFL & 15) | ((INFL >> 4) << 14) | (7 << 4) | (15 << 8);
#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t) request(t, t);
  f32x4 fa[2][TM], fb[2][TN];
  auto read = [&](int set, const float* ta, int c) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[set][i] = LA::frag(ta, wm0 + 16 * i, c, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[set][j] = LB::frag(ta + TA, wn0 + 16 * j, c, lane);
    __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the products they run under
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[set][j][e], fa[set][i][e], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  __builtin_amdgcn_s_waitcnt(WAIT_TILE);
  __syncthreads();
  read(0, ring, 0);
  int cur = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // the stage refilled here was read for the last time before the last barrier
    request(kt + NSTAGE - 1, cur == 0 ? NSTAGE - 1 : cur - 1);
    read(1, ring + cur * STAGE, 1);
    multiply(0);
    __builtin_amdgcn_s_waitcnt(WAIT_TILE);  // tile kt + 1 has landed
    __syncthreads();
    cur = cur + 1 == NSTAGE ? 0 : cur + 1;
    read(0, ring + cur * STAGE, 0);  // after the last tile: a clamped tile, unused
    multiply(1);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the clamped tail loads
  if constexpr (WK > 1) {
    // group g > 0 leaves its sums in LDS ([tile register][64 lanes] per wave), group 0 adds them in order
    constexpr int SLOT = TM * TN * 256;
    static_assert((WK - 1) * NW * SLOT <= WK * RING, "partial sums must fit in the rings");
    __syncthreads();
    if (kg > 0) {
      float* my = smem_f32 + ((kg - 1) * NW + wave) * SLOT + 4 * lane;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(my + (i * TN + j) * 256) = acc[i][j];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < WK; ++g) {
      const float* other = smem_f32 + ((g - 1) * NW + wave) * SLOT + 4 * lane;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] += *reinterpret_cast<const f32x4*>(other + (i * TN + j) * 256);
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm0 + 16 * i + (lane & 15);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + 16 * j + 4 * (lane >> 4);
      if (m < p.M && n < p.N) store_quad_f32(p, acc[i][j], m, n);
    }
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int WK, int NSTAGE, bool A_KMAJ, bool B_KMAJ>
// (at least two waves per SIMD: within the 256 registers that leaves, the compiler keeps the sums in
// vector registers; given 512 it rotates them through accumulation registers and waits for every
// product of a K step to copy them)
__global__ __launch_bounds__(WAVES_M * WAVES_N * WK * 64, 2) void gemm_f32_tile_kernel(F32Params p) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) float smem_f32[];
  int tile_m, tile_n;
  tile_of(p, tile_m, tile_n);
  f32_tile<BM, BN, WAVES_M, WAVES_N, WK, NSTAGE, A_KMAJ, B_KMAJ>(p, smem_f32, tile_m, tile_n);
#endif
}

// Every weight gradient and bias gradient of a W pass (see WgradBatchParams).
template <int BM, int BN, int WAVES_M, int WAVES_N, int WK, int NSTAGE>
__global__ __launch_bounds__(WAVES_M * WAVES_N * WK * 64, 2) void gemm_f32_wgrad_batch_kernel(WgradBatchParams q) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) float smem_f32[];
  if ((int)blockIdx.x < q.sum_blocks) {
    batch_column_sums<float, WAVES_M * WAVES_N * WK * 64>(q, blockIdx.x, smem_f32);
    return;
  }
  const BatchTile t = batch_tile(q, (int)blockIdx.x - q.sum_blocks);
  const WgradBatchArgs::Layer& l = q.w.layer[t.layer];
  F32Params p;
  p.A = reinterpret_cast<const float*>(q.w.piece[0] + l.a[t.product]);
  p.B = reinterpret_cast<const float*>(q.w.piece[0] + l.b[t.product]);
  p.C = l.c[t.product];
  p.bias = p.resid = nullptr;
  p.aux = nullptr;
  p.M = p.lda = q.w.M[t.product];
  p.N = p.ldb = p.ldc = q.w.N[t.product];
  p.K = q.w.K;
  p.epi = PMC_EPI_ACCUM_F32;
  f32_tile<BM, BN, WAVES_M, WAVES_N, WK, NSTAGE, false, false>(p, smem_f32, t.tile_m, t.tile_n);
#endif
}

// Four k-consecutive elements (k .. k+3) of row `row` of an operand; zeros past K.
template <bool KMAJ, bool VEC>
__device__ __forceinline__ f32x4 load_k4(const float* __restrict__ X, int ld, int row, int k, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (KMAJ && VEC) {
    if (k < K) v = *reinterpret_cast<const f32x4*>(X + (size_t)row * ld + k);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k + j < K) v[j] = KMAJ ? X[(size_t)row * ld + k + j] : X[(size_t)(k + j) * ld + row];
  }
  return v;
}

template <bool A_KMAJ, bool B_KMAJ, bool VEC>
__global__ __launch_bounds__(512, 2) void gemm_f32_direct_kernel(F32Params p) {
  constexpr int NWAVE = 8, UNROLL = 4;
  __shared__ float part[NWAVE][16][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tm, tn;
  tile_of(p, tm, tn);
  const int m = min(16 * tm + (lane & 15), p.M - 1), n = min(16 * tn + (lane & 15), p.N - 1), kq = 4 * (lane >> 4);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int step = 16 * NWAVE;
  for (int k = 16 * wave; k < p.K; k += UNROLL * step) {
    f32x4 a[UNROLL], b[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      a[u] = load_k4<A_KMAJ, VEC>(p.A, p.lda, m, k + u * step + kq, p.K);
      b[u] = load_k4<B_KMAJ, VEC>(p.B, p.ldb, n, k + u * step + kq, p.K);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][e], a[u][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[wave][lane & 15][kq + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < 256) {
    const int r = threadIdx.x >> 4, c = threadIdx.x & 15, gm = 16 * tm + r, gn = 16 * tn + c;
    if (gm < p.M && gn < p.N) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NWAVE; ++w) v += part[w][r][c];
      const size_t idx = (size_t)gm * p.ldc + gn;
      p.C[idx] = apply_epilogue(p, v, idx, gn);
    }
  }
}

// Sum over k in ascending order, any sizes, pitches and alignments.
template <bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(256) void gemm_f32_fma_kernel(F32Params p) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < p.K; k0 += BK) {
    for (int i = tid; i < BM * BK; i += 256) {
      const int k = A_KMAJ ? i % BK : i / BM, m = A_KMAJ ? i / BK : i % BM, gm = m0 + m, gk = k0 + k;
      As[k][m] = gm < p.M && gk < p.K ? (A_KMAJ ? p.A[(size_t)gm * p.lda + gk] : p.A[(size_t)gk * p.lda + gm]) : 0.f;
    }
    for (int i = tid; i < BN * BK; i += 256) {
      const int k = B_KMAJ ? i % BK : i / BN, n = B_KMAJ ? i / BK : i % BN, gn = n0 + n, gk = k0 + k;
      Bs[k][n] = gn < p.N && gk < p.K ? (B_KMAJ ? p.B[(size_t)gn * p.ldb + gk] : p.B[(size_t)gk * p.ldb + gn]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= p.N) continue;
      const size_t idx = (size_t)m * p.ldc + n;
      p.C[idx] = apply_epilogue(p, acc[i][j], idx, n);
    }
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int WK, int NSTAGE, bool TA, bool TB>
int launch_tile_f32(hipStream_t st, F32Params p) {
  constexpr size_t lds = (size_t)WK * NSTAGE * 32 * (BM + BN) * sizeof(float);
  static_assert(lds <= 160 * 1024, "rings do not fit the 160 KB LDS");
  auto kern = gemm_f32_tile_kernel<BM, BN, WAVES_M, WAVES_N, WK, NSTAGE, !TA, TB>;
  static std::atomic<bool> configured{false};
  if (int rc = reserve_lds(kern, lds, configured, "gemm_f32")) return rc;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  kern<<<dim3(p.tiles_m * p.tiles_n), dim3(WAVES_M * WAVES_N * WK * 64), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_f32 launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

template <bool TA, bool TB>
int launch_direct_f32(hipStream_t st, F32Params p, bool vec) {
  p.tiles_m = (p.M + 15) / 16;
  p.tiles_n = (p.N + 15) / 16;
  const dim3 grid(p.tiles_m * p.tiles_n), block(512);
  if (vec) gemm_f32_direct_kernel<!TA, TB, true><<<grid, block, 0, st>>>(p);
  else gemm_f32_direct_kernel<!TA, TB, false><<<grid, block, 0, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_f32 launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

template <bool TA, bool TB>
int launch_fma_f32(hipStream_t st, const F32Params& p) {
  gemm_f32_fma_kernel<!TA, TB><<<dim3((p.N + 63) / 64, (p.M + 63) / 64), dim3(256), 0, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_f32 launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

// Kernel and output tile of a product: 128 x 128, 64 x 128, 64 x 64, 32 x 64 and 32 x 32 tiles staged in LDS, 16 x 16
// ones in the direct kernel with 16-byte loads, and, with element-wise loads, 16 x 16 ones in the direct
// kernel or 64 x 64 ones in the FMA kernel.
enum F32Shape { kTile128, kTile64, kTile32x64, kTile32, kDirect, kDirectElements, kFmaElements, kTile64x128, kTile32Four, kNoTile };
// One dimension of a launch holds fewer than 2^32 threads (one past that is not refused, it leaves workgroups out).
bool one_launch(F32Shape shape, long tiles) { return tiles < (1LL << 32) / (shape == kTile32Four ? 256 : 512); }

// With 16-byte loads: the tile with the least fitted time, us = fixed + n (tile_k k + tile) + ceil(n / per_cu) (group_k k + group)
// + ceil(n) (round_k k + round) at n tiles per compute unit, per_cu of them side by side, and k = K / 1024.  Fitted to
// 2323 products of more than 12 us (operands of 200 MB in turn) and 4697 smaller ones (in a graph, so that the host does
// not count), M = 16 .. 6144, N = 64 .. 5120, K = 64 .. 5120: the tile picked is 0.8 % slower than the best one on average, 1.24
// times at worst.  The fit overrates 16 x 16 tiles just past a round of 256, which is no round for four of them to a unit: with 0.94 of their
// time none of the 7020 products loses more than 7.6 % to the choice among the same five shapes with four waves, with all of it 31 lose more than 10 % (up to
// 18 %), with 0.88 of it 14 (up to 25 %).  In 250 steps of hidden 64 .. 768 and 16 .. 640 tokens the three are within 0.03 % on average.  All but the 32 x 32 tile of four waves have two waves to a SIMD or more, eight waves to a workgroup, with K
// in two groups where the tile is too small for eight: with four waves to a unit nothing covered the reads from LDS.  The
// larger products run in 0.89 and the smaller in 0.95 of the time that the same tiles with four waves take; four waves / eight:
// 512 x 1024 x 4096 (F, 32 x 64) 49.2 / 45.3 us, 768 x 5120 x 1280 (F, 64 x 64 / 64 x 128) 97 / 88, 512 x 3072 x 1024 (F) 45 / 38,
// 128 x 128 tiles of 512 x 4096 x 1024 79.7 / 74.5; what few tiles gain by sixteen rows and no LDS: 128 x 256 x 1024 5.8 us
// against 9.2 in 32 x 32 tiles.  64 x 128 tiles are measured up to four rounds of 128 x 128 ones, which read less, and not taken beyond.
// The gemm_tile switch forces one of the first five (tests).
F32Shape pick_tile_f32(bool tb, int M, int N, int K) {
  struct T {
    F32Shape shape;
    int bm, bn, per_cu;
    double fixed[2], tile_k[2], tile[2], group_k[2], group[2], round_k[2], round[2];  // B stored [K,N] / [N,K]
  };
  static constexpr T kTimes[7] = {
      {kTile128, 128, 128, 1, {2.91, 2.48}, {0.851, 0.}, {5.08, 3.95}, {0., 0.}, {4.21, 0.}, {65.6, 61.9}, {0., 2.45}},
      {kTile64x128, 64, 128, 2, {3.96, 3.31}, {1.09, 0.427}, {2.23, 2.01}, {5.4, 4.67}, {0., 0.}, {28.4, 29.2}, {0.833, 0.744}},
      {kTile64, 64, 64, 2, {3.03, 2.65}, {0.165, 0.197}, {1.62, 1.58}, {4.07, 3.15}, {0., 0.}, {15.5, 15.3}, {0.294, 0.159}},
      {kTile32x64, 32, 64, 2, {2.64, 2.57}, {0., 0.0612}, {1.06, 0.991}, {2.17, 2.07}, {0.486, 0.0135}, {8.2, 8.33}, {0.249, 0.364}},
      {kTile32, 32, 32, 4, {2.2, 2.33}, {0., 0.0676}, {0.718, 0.68}, {1.54, 1.44}, {0.319, 0.}, {4.72, 4.55}, {0.394, 0.35}},
      {kTile32Four, 32, 32, 5, {2.47, 2.24}, {0.189, 0.176}, {0.545, 0.53}, {3.27, 2.7}, {0., 0.}, {4.55, 4.5}, {0., 0.}},
      {kDirect, 16, 16, 4, {2.54, 2.21}, {0., 0.0346}, {0.373, 0.247}, {0.713, 0.508}, {0., 0.}, {2.5, 2.91}, {0.234, 0.}}};
  auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  F32Shape best = kNoTile;
  double best_us = 1e300;
  for (const T& t : kTimes) {
    if (t.shape == kTile64x128 && tiles(128, 128) >= 4 * 256) continue;
    const long count = tiles(t.bm, t.bn), rounds = (count + 255) / 256, groups = (count + 256L * t.per_cu - 1) / (256L * t.per_cu);
    if (!one_launch(t.shape, count)) continue;
    const double k = K / 1024.0, n = (double)count / 256.0;
    double us = t.fixed[tb] + n * (t.tile_k[tb] * k + t.tile[tb]) + (double)groups * (t.group_k[tb] * k + t.group[tb]) +
                (double)rounds * (t.round_k[tb] * k + t.round[tb]);
    if (t.shape == kDirect) us *= 0.94;  // see above
    if (us < best_us) {
      best_us = us;
      best = t.shape;
    }
  }
  if (const int f = tuning(kTuneGemmTile); f >= 0) {  // where the launch would not hold them, the next larger tiles from 64 x 64 on that it does
    best = kNoTile;
    for (F32Shape shape : {(F32Shape)f, kTile64, kTile64x128, kTile128})
      for (const T& t : kTimes)
        if (best == kNoTile && t.shape == shape && one_launch(shape, tiles(t.bm, t.bn))) best = shape;
  }
  return best;
}

// With element-wise loads: the kernel with the smaller fitted time in us, u = 16 x 16 tiles per compute unit.
// The direct kernel's grows with the tiles, by what a quarter-wave's loads of the layout cost; the FMA kernel's
// is the chain of one workgroup until about five of its tiles share a unit.  Fitted to 260 products of odd
// sizes, M, N = 129 .. 3073, K = 37 .. 2051, where the kernel picked is at most 14 % slower than the other, 0.2 %
// on average; direct / FMA kernel: A [M,K] B [K,N] 255 x 513 x 517 11.3 / 60.8 us, 2049 x 3073 x 517 292 / 130;
// A [M,K] B [N,K] 17.3 / 61.5 and 493 / 131; A [K,M] B [K,N] 8.5 / 60.3 and 223 / 136; 1025 x 2049 x 37 32 / 11.8.
F32Shape pick_elements_f32(bool ta, bool tb, int M, int N, int K) {
  const double u = (double)((M + 15) / 16) * ((N + 15) / 16) / 256.0;
  const double per_tile = ta == tb ? 0.85 : tb ? 0.5 : 1.03, per_k = ta == tb ? 0.0046 : tb ? 0.0084 : 0.0029;
  double chain = 0.12 + 0.0027 * u;
  if (chain > 0.195) chain = 0.195;
  if (chain < 0.0025 * u) chain = 0.0025 * u;
  return u * (per_tile + per_k * K) < 0.15 * u + chain * K ? kDirectElements : kFmaElements;
}

F32Shape shape_of(const GemmArgs& a) {
  auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  // whole 16-byte chunks everywhere, operands inside the 2 GB that an offset of the tile loads can reach
  const size_t a_bytes = (size_t)(a.trans_a ? a.K : a.M) * a.lda * 4, b_bytes = (size_t)(a.trans_b ? a.N : a.K) * a.ldb * 4;
  const bool vec = a.M % 4 == 0 && a.N % 4 == 0 && a.K % 4 == 0 && a.lda % 4 == 0 && a.ldb % 4 == 0 && a.ldc % 4 == 0 && al(a.A) &&
                   al(a.B) && al(a.C) && al(a.bias) && al(a.resid) && al(a.aux) && a_bytes < 0x7fffffffull && b_bytes < 0x7fffffffull;
  return vec ? pick_tile_f32(a.trans_b, a.M, a.N, a.K) : pick_elements_f32(a.trans_a, a.trans_b, a.M, a.N, a.K);
}

template <bool TA, bool TB>
int launch_f32(hipStream_t st, const F32Params& p, F32Shape shape) {
  switch (shape) {
    case kTile128: return launch_tile_f32<128, 128, 4, 2, 1, 3, TA, TB>(st, p);
    case kTile64x128: return launch_tile_f32<64, 128, 2, 4, 1, 3, TA, TB>(st, p);
    case kTile64: return launch_tile_f32<64, 64, 4, 2, 1, 4, TA, TB>(st, p);
    case kTile32x64: return launch_tile_f32<32, 64, 2, 2, 2, 3, TA, TB>(st, p);
    case kTile32: return launch_tile_f32<32, 32, 2, 2, 2, 4, TA, TB>(st, p);
    case kTile32Four: return launch_tile_f32<32, 32, 2, 2, 1, 4, TA, TB>(st, p);
    case kDirect: return launch_direct_f32<TA, TB>(st, p, true);
    case kDirectElements: return launch_direct_f32<TA, TB>(st, p, false);
    case kFmaElements: return launch_fma_f32<TA, TB>(st, p);
    case kNoTile: break;
  }
  return fail(PMC_ERR_INVALID, "gemm_f32: %d x %d outputs are more than one launch holds", p.M, p.N);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int WK, int NSTAGE>
int launch_wgrad_batch_f32(hipStream_t st, WgradBatchParams& p) {
  constexpr size_t lds = (size_t)WK * NSTAGE * 32 * (BM + BN) * sizeof(float);
  auto kern = gemm_f32_wgrad_batch_kernel<BM, BN, WAVES_M, WAVES_N, WK, NSTAGE>;
  static std::atomic<bool> configured{false};
  if (int rc = reserve_lds(kern, lds, configured, "gemm_f32")) return rc;
  wgrad_batch_layout(p, BM, BN, WAVES_M * WAVES_N * WK * 64);
  kern<<<dim3(p.sum_blocks + p.first_tile[4] * p.w.layers), dim3(WAVES_M * WAVES_N * WK * 64), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_f32 weight-gradient launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

}  // namespace

int gemm_f32(hipStream_t st, const GemmArgs& a) {
  F32Params p;
  p.A = (const float*)a.A; p.B = (const float*)a.B; p.C = (float*)a.C;
  p.bias = (const float*)a.bias; p.resid = (const float*)a.resid; p.aux = (float*)a.aux;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.ldc = a.ldc; p.epi = a.epilogue;
  p.tiles_m = p.tiles_n = 0;
  const F32Shape shape = shape_of(a);
  if (!a.trans_a && !a.trans_b) return launch_f32<false, false>(st, p, shape);
  if (!a.trans_a && a.trans_b) return launch_f32<false, true>(st, p, shape);
  if (a.trans_a && !a.trans_b) return launch_f32<true, false>(st, p, shape);
  return launch_f32<true, true>(st, p, shape);
}

// Tiles of the one launch, by times fitted (batch_us) to 1555 W passes, hidden 64 .. 1280, 16 .. 6144 tokens, 1 .. 4 layers: the
// shape picked is 0.4 % slower than the best one on average, 1.25 times at worst, and 3.2 times as fast as the products launched
// one by one (geometric mean; 1.2 times at least).  1 layer of hidden 256, 128 tokens 26 -> 9 us; 2 of 1024, 512 tokens 323 -> 236.
// With all tiles of a pass in one launch small workgroups, several to a compute unit, beat the larger tiles that read less.
//   0: 64x64, 3 stages (three workgroups per compute unit)   1: 32x32 in four waves   2: 32x32 whose waves split K
int gemm_f32_wgrad_batch_shape(const WgradBatchArgs& a) {
  constexpr int kB[3] = {64, 32, 32};
  static constexpr BatchTime kTimes[3] = {{6.48, 15.32, 14.92, 1.56, 0., 0., 3}, {5.70, 5.40, 4.69, 0.61, 0., 0., 5}, {5.80, 2.97, 6.06, 3.04, 0., 0., 1}};
  int best = 0;
  double best_us = 1e300;
  for (int s = 0; s < 3; ++s) {
    const double us = batch_us(kTimes[s], (double)batch_tiles(a, kB[s], kB[s]) * a.layers, a.K);
    if (us < best_us) {
      best_us = us;
      best = s;
    }
  }
  return best;
}

int gemm_f32_wgrad_batch(hipStream_t st, const WgradBatchArgs& a, int shape) {
  if (a.pieces != 1) return fail(PMC_ERR_INVALID, "gemm_f32: weight gradients of %d microbatches in one launch", a.pieces);
  WgradBatchParams p;
  p.w = a;
  switch (shape) {
    case 0: return launch_wgrad_batch_f32<64, 64, 2, 2, 1, 3>(st, p);
    case 1: return launch_wgrad_batch_f32<32, 32, 2, 2, 1, 4>(st, p);
    case 2: return launch_wgrad_batch_f32<32, 32, 1, 1, 4, 3>(st, p);
  }
  return fail(PMC_ERR_INVALID, "gemm_f32: no weight-gradient tiles %d", shape);
}

// Tiles of the W pass in one launch, -1: its products are launched one by one.  That is also what happens where an operand needs
// more than the 2 GB of a buffer descriptor or a pointer is not aligned for 16-byte accesses (the products by themselves
// then take other kernels, or refuse), where a launch would not hold the tiles, and where a switch forces the kernel of a product.
int wgrad_batch_shape(int dtype, const WgradBatchArgs& a) {
  for (Tuning t : {kTuneGemmTile, kTuneGemmGroup, kTuneGemmWgrad, kTuneWStreams})
    if (tuning(t) >= 0) return -1;
  const size_t e = dtype == PMC_F32 ? 4 : 2;
  uintptr_t bits = 0;
  for (int i = 0; i < a.pieces; ++i) bits |= (uintptr_t)a.piece[i];
  for (int j = 0; j < 4; ++j) {
    if ((size_t)a.K * std::max(a.M[j], a.N[j]) * e >= 0x7fffffffull) return -1;
    for (int l = 0; l < a.layers; ++l) bits |= a.layer[l].a[j] | a.layer[l].b[j] | (uintptr_t)a.layer[l].c[j];
  }
  if (bits & 15) return -1;
  if (batch_tiles(a, 32, 32) * a.layers >= 1L << 23) return -1;
  return dtype == PMC_F32 ? gemm_f32_wgrad_batch_shape(a) : gemm_bf16_wgrad_batch_shape(a);
}

int wgrad_batch(hipStream_t st, int dtype, const WgradBatchArgs& a, int shape) {
  return dtype == PMC_F32 ? gemm_f32_wgrad_batch(st, a, shape) : gemm_bf16_wgrad_batch(st, a, shape);
}

GemmPlan gemm_f32_plan(const GemmArgs& a) {
  const F32Shape shape = shape_of(a);
  return {shape == kNoTile ? -1 : kPlanF32 + (int)shape, 1, 0};
}

// Shape and pointer checks common to both precisions, then dispatch.
int gemm(hipStream_t st, const GemmArgs& a) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return fail(PMC_ERR_INVALID, "gemm: M=%d N=%d K=%d", a.M, a.N, a.K);
  if (!a.A || !a.B || !a.C) return fail(PMC_ERR_INVALID, "gemm: NULL operand");
  const int a_cols = a.trans_a ? a.M : a.K, b_cols = a.trans_b ? a.K : a.N;
  if (a.lda < a_cols || a.ldb < b_cols || a.ldc < a.N)
    return fail(PMC_ERR_INVALID, "gemm: pitch too small (lda=%d ldb=%d ldc=%d)", a.lda, a.ldb, a.ldc);
  switch (a.epilogue) {
    case PMC_EPI_NONE:
    case PMC_EPI_ACCUM_F32:
      break;
    case PMC_EPI_BIAS:
      if (!a.bias) return fail(PMC_ERR_INVALID, "gemm: bias epilogue without bias");
      break;
    case PMC_EPI_BIAS_RESID:
      if (!a.bias || !a.resid) return fail(PMC_ERR_INVALID, "gemm: bias+residual epilogue needs both");
      break;
    case PMC_EPI_BIAS_GELU:
    case PMC_EPI_BIAS_GELU_GRAD:
      if (!a.bias || !a.aux) return fail(PMC_ERR_INVALID, "gemm: bias+gelu epilogue needs bias and aux");
      break;
    case PMC_EPI_DGELU:
    case PMC_EPI_MUL:
      if (!a.aux) return fail(PMC_ERR_INVALID, "gemm: this epilogue needs aux");
      break;
    default:
      return fail(PMC_ERR_INVALID, "gemm: unknown epilogue %d", a.epilogue);
  }
  if (a.dtype == PMC_F32) return gemm_f32(st, a);
  if (a.dtype == PMC_BF16) return gemm_bf16(st, a);
  return fail(PMC_ERR_INVALID, "gemm: bad dtype %d", a.dtype);
}

}  // namespace k
}  // namespace pmc
