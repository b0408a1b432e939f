// Flash-style attention on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32): fp32 products, fp32
// accumulation and the library's accurate exp / log.  This is the PMC_F32-mode path, where results must
// agree with the fp64 oracle to 1e-5, and the path of bf16 head sizes that are not a multiple of 8
// (widened on load).  Packed qkv is [batch*seq, 3h], h = heads*dh; no s x s matrix is ever stored.
//
// What bounds it is latency: the shapes are short, so there are few (row block, head) pairs and the chain
// load -> S -> softmax -> product of one pair is what takes the time.  A workgroup therefore owns only 16
// rows of one head (queries in the forward and dQ kernels, keys in the dK/dV kernel) and its eight waves
// deal the other side's 16-row groups among them, each with its own online softmax or partial sums; the
// partial results are folded in wave order through LDS, so every output element has one writer and a
// fixed summation order.  Operands are loaded in the fragment layout straight from global memory (L2
// holds a head's K and V), without LDS tiles and without a barrier before the fold.
//
// Measured against plain FMAs on LDS tiles (before), forward / dQ / dK,dV: 4 heads of 64, 128 tokens
// 38.9 / 32.4 / 45.4 -> 6.5 / 8.4 / 8.9 us; 16 heads of 64, 512 tokens 154 / 170 / 180 -> 16 / 25 / 27 us.
//
// Fragment layouts, quarter q = lane / 16:
//   rows:    lane holds row lane % 16, columns 16 c + 4 q .. + 3 of column group c; instruction e of a
//            group contracts columns 16 c + 4 q + e.
//   cols(j): lane holds columns 4 (lane % 16) .. + 3 of row 4 q + j; element e is the operand of a
//            product whose output rows are the columns 4 i + e, so after all four a lane owns the 16
//            consecutive columns 16 q .. 16 q + 15 of its row, and both kinds of load are 16 bytes wide.
// A score tile (rows 4 q + r in register r, column lane % 16) is already the second operand of the
// product that contracts its rows.
#include "dev_common.h"
#include "kernels.h"

namespace pmc {
namespace k {
namespace {

constexpr int kMaxDh = 128;
constexpr int kWavesF = 8;
constexpr int kRows = 16;  // rows a workgroup owns
constexpr int kMaxGrid = 65535;  // workgroups in the second and third dimension of a launch

// Four consecutive columns of a row, zeros past dh.  VEC: dh is a multiple of 4 and the four are one aligned load.
template <typename T, bool VEC>
__device__ __forceinline__ f32x4 load4(const T* __restrict__ row, int col, int dh) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (col < dh) {
      if constexpr (sizeof(T) == 4) {
        v = *reinterpret_cast<const f32x4*>(row + col);
      } else {
        const u32x2 p = *reinterpret_cast<const u32x2*>(row + col);
        v = f32x4{bf16lo_to_f32(p[0]), bf16hi_to_f32(p[0]), bf16lo_to_f32(p[1]), bf16hi_to_f32(p[1])};
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < dh) v[e] = to_f32(row[col + e]);
  }
  return v;
}

template <typename T, bool VEC>
__device__ __forceinline__ void store4(T* row, int col, int dh, f32x4 v) {
  if constexpr (VEC) {
    if (col < dh) {
      if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<f32x4*>(row + col) = v;
      } else {
        const u32x2 p = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        *reinterpret_cast<u32x2*>(row + col) = p;
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < dh) row[col + e] = from_f32<T>(v[e]);
  }
}

// [16 rows][DH] fragment set in the `rows` layout; base: column 0 of row 0, rows clamped to `last`.
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void load_rows(f32x4 (&f)[DH / 16], const T* __restrict__ base, size_t pitch, int row0, int last, int dh, int lane) {
  const T* p = base + (size_t)min(row0 + (lane & 15), last) * pitch;
#pragma unroll
  for (int c = 0; c < DH / 16; ++c) f[c] = load4<T, VEC>(p, 16 * c + 4 * (lane >> 4), dh);
}
// The same 16 rows in the `cols` layout.
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void load_cols(f32x4 (&f)[4][DH / 64], const T* __restrict__ base, size_t pitch, int row0, int last, int dh, int lane) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const T* p = base + (size_t)min(row0 + 4 * (lane >> 4) + j, last) * pitch;
#pragma unroll
    for (int b = 0; b < DH / 64; ++b) f[j][b] = load4<T, VEC>(p, 64 * b + 4 * (lane & 15), dh);
  }
}

// out[row 4 q + r of a][column lane % 16 of b] = sum over columns, both in the `rows` layout.
template <int NC>
__device__ __forceinline__ f32x4 dot_rows(const f32x4 (&a)[NC], const f32x4 (&b)[NC]) {
  // two chains, so that consecutive products do not wait for each other
  f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][e], b[c][e], s[c & 1], 0, 0, 0);
  return s[0] + s[1];
}

// acc[b][e]: output column 64 b + 4 (4 q + r) + e (register r) of row lane % 16; adds X^T . w for 16 rows
// of X in the `cols` layout and w in the layout of a score tile.
template <int NB>
__device__ __forceinline__ void add_outer(f32x4 (&acc)[NB][4], const f32x4 (&x)[4][NB], f32x4 w) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[b][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][b][e], w[j], acc[b][e], 0, 0, 0);
}

// A wave's accumulators to its [16 rows][DH + 4] slab of the fold buffer.
template <int DH>
__device__ __forceinline__ void park(float* slab, const f32x4 (&acc)[DH / 64][4], int lane) {
  float* p = slab + (lane & 15) * (DH + 4) + 16 * (lane >> 4);
#pragma unroll
  for (int b = 0; b < DH / 64; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 v = {acc[b][0][r], acc[b][1][r], acc[b][2][r], acc[b][3][r]};
      *reinterpret_cast<f32x4*>(p + 64 * b + 4 * r) = v;
    }
}
// Sum over the waves, in wave order, of four columns of one row of the fold buffer.
template <int DH>
__device__ __forceinline__ f32x4 fold(const float* slabs, int row, int col) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kWavesF; ++w) v += *reinterpret_cast<const f32x4*>(slabs + (w * kRows + row) * (DH + 4) + col);
  return v;
}

__device__ __forceinline__ float quarters_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float quarters_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// Workgroup -> (row block, head, sequence); the grid is (heads, sequences, row blocks from `block0` on), see
// for_row_blocks.  Under a causal mask late query blocks and early key blocks see the most of the other side:
// they are dealt out first and the short ones fill the tail.
struct Place {
  int row0, head, b;
};
__device__ __forceinline__ Place place(int seq, int block, bool late_first) {
  const int blocks = (seq + kRows - 1) / kRows;
  return {(late_first ? blocks - 1 - block : block) * kRows, (int)blockIdx.x, (int)blockIdx.y};
}

template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(kWavesF * 64, 2) void attn_fwd_f32(int block0, int seq, int heads, int dh, int causal, const T* __restrict__ qkv,
                                                             T* __restrict__ o, float* __restrict__ lse) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) float fold_f32[];  // [8 waves][16][DH + 4]
  __shared__ float stat_m[kWavesF][kRows], stat_l[kWavesF][kRows];
  const Place at = place(seq, block0 + (int)blockIdx.z, causal != 0);
  const int h = heads * dh, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = lane >> 4;
  const size_t pitch = (size_t)3 * h;
  const T* base = qkv + (size_t)at.b * seq * pitch + (size_t)at.head * dh;
  const int qi = at.row0 + (lane & 15);
  const float sigma = 1.0f / sqrtf((float)dh);
  f32x4 qf[DH / 16], acc[DH / 64][4];
  load_rows<T, DH, VEC>(qf, base, pitch, at.row0, seq - 1, dh, lane);
#pragma unroll
  for (int b = 0; b < DH / 64; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;  // of this wave's keys; l is this lane quarter's part
  const int kend = causal ? min(seq, at.row0 + kRows) : seq;
  for (int k0 = kRows * wave; k0 < kend; k0 += kRows * kWavesF) {
    f32x4 kf[DH / 16], vf[4][DH / 64];
    load_rows<T, DH, VEC>(kf, base + h, pitch, k0, seq - 1, dh, lane);
    load_cols<T, DH, VEC>(vf, base + 2 * h, pitch, k0, seq - 1, dh, lane);
    f32x4 s = dot_rows(kf, qf);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kj = k0 + 4 * quarter + r;
      s[r] = (kj < seq && (!causal || kj <= qi)) ? s[r] * sigma : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    const float m_new = fmaxf(m, quarters_max(mx));
    // m_new stays -inf for a query that has seen none of this wave's keys yet
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - m_use);
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = expf(s[r] - m_use);
      l += s[r];
    }
#pragma unroll
    for (int b = 0; b < DH / 64; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[b][e] *= alpha;
    m = m_new;
    add_outer(acc, vf, s);
  }
  l = quarters_sum(l);
  park<DH>(fold_f32 + wave * kRows * (DH + 4), acc, lane);
  if (quarter == 0) {
    stat_m[wave][lane] = m;
    stat_l[wave][lane] = l;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * (DH / 4); i += kWavesF * 64) {
    const int row = i / (DH / 4), col = 4 * (i % (DH / 4)), q = at.row0 + row;
    float mt = stat_m[0][row];
#pragma unroll
    for (int w = 1; w < kWavesF; ++w) mt = fmaxf(mt, stat_m[w][row]);
    float lt = 0.f;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWavesF; ++w) {
      const float f = expf(stat_m[w][row] - mt);  // a wave without keys has m = -inf: weight 0
      lt += stat_l[w][row] * f;
      v += *reinterpret_cast<const f32x4*>(fold_f32 + (w * kRows + row) * (DH + 4) + col) * f;
    }
    if (q < seq) {
      store4<T, VEC>(o + ((size_t)at.b * seq + q) * h + (size_t)at.head * dh, col, dh, v * (1.0f / lt));
      if (col == 0) lse[((size_t)at.b * heads + at.head) * seq + q] = mt + logf(lt);
    }
  }
#endif
}

// dq[i] = sigma * sum_j dS[i][j] k[j],  dS = P * (dP - delta),  P = exp(S - lse),  dP = dO . V^T, for 16 queries; also
// emits delta = rowsum(dO * O) unless it is NULL.
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void dq_block_f32(float* fold_f32, const Place at, int seq, int heads, int dh, int causal, const T* __restrict__ qkv,
                                             const T* __restrict__ o, const float* __restrict__ lse, const T* __restrict__ d_o, T* __restrict__ dq,
                                             size_t ld_dq, float* __restrict__ delta) {
  const int h = heads * dh, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = lane >> 4;
  const size_t pitch = (size_t)3 * h, own = (size_t)at.b * seq * h + (size_t)at.head * dh;
  const T* base = qkv + (size_t)at.b * seq * pitch + (size_t)at.head * dh;
  const int qi = at.row0 + (lane & 15);
  const size_t stat = ((size_t)at.b * heads + at.head) * seq + min(qi, seq - 1);
  const float sigma = 1.0f / sqrtf((float)dh);
  f32x4 qf[DH / 16], df[DH / 16], acc[DH / 64][4];
  load_rows<T, DH, VEC>(qf, base, pitch, at.row0, seq - 1, dh, lane);
  load_rows<T, DH, VEC>(df, d_o + own, (size_t)h, at.row0, seq - 1, dh, lane);
  float dl = 0.f;
  {
    f32x4 of[DH / 16];
    load_rows<T, DH, VEC>(of, o + own, (size_t)h, at.row0, seq - 1, dh, lane);
#pragma unroll
    for (int c = 0; c < DH / 16; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) dl = fmaf(df[c][e], of[c][e], dl);
  }
  dl = quarters_sum(dl);
  if (delta && wave == 0 && quarter == 0 && qi < seq) delta[stat] = dl;
  const float my_lse = lse[stat];
#pragma unroll
  for (int b = 0; b < DH / 64; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int kend = causal ? min(seq, at.row0 + kRows) : seq;
  for (int k0 = kRows * wave; k0 < kend; k0 += kRows * kWavesF) {
    f32x4 kf[DH / 16], vf[DH / 16], kc[4][DH / 64];
    load_rows<T, DH, VEC>(kf, base + h, pitch, k0, seq - 1, dh, lane);
    load_rows<T, DH, VEC>(vf, base + 2 * h, pitch, k0, seq - 1, dh, lane);
    load_cols<T, DH, VEC>(kc, base + h, pitch, k0, seq - 1, dh, lane);
    const f32x4 s = dot_rows(kf, qf), dp = dot_rows(vf, df);
    f32x4 ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kj = k0 + 4 * quarter + r;
      ds[r] = (kj < seq && (!causal || kj <= qi)) ? expf(s[r] * sigma - my_lse) * (dp[r] - dl) : 0.f;
    }
    add_outer(acc, kc, ds);
  }
  park<DH>(fold_f32 + wave * kRows * (DH + 4), acc, lane);
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * (DH / 4); i += kWavesF * 64) {
    const int row = i / (DH / 4), col = 4 * (i % (DH / 4));
    if (at.row0 + row < seq)
      store4<T, VEC>(dq + ((size_t)at.b * seq + at.row0 + row) * ld_dq + (size_t)at.head * dh, col, dh, fold<DH>(fold_f32, row, col) * sigma);
  }
}

// For 16 keys: dv[j] = sum_i P[i][j] dO[i],  dk[j] = sigma * sum_i dS[i][j] q[i].  dqkv may be qkv itself (a key block is read only by
// the workgroup that owns it, before its fold).  DELTA: delta is formed
// here from dO and O (o), otherwise read from `delta`.
template <typename T, int DH, bool VEC, bool DELTA>
__device__ __forceinline__ void dkv_block_f32(float* fold_f32, const Place at, int seq, int heads, int dh, int causal, const T* qkv,
                                              const T* __restrict__ o, const float* __restrict__ lse,
                                              const float* __restrict__ delta, const T* __restrict__ d_o, T* dqkv) {
  const int h = heads * dh, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = lane >> 4;
  const size_t pitch = (size_t)3 * h;
  const T* base = qkv + (size_t)at.b * seq * pitch + (size_t)at.head * dh;
  const T* dob = d_o + (size_t)at.b * seq * h + (size_t)at.head * dh;
  const float* lse_b = lse + ((size_t)at.b * heads + at.head) * seq;
  const float* delta_b = DELTA ? nullptr : delta + ((size_t)at.b * heads + at.head) * seq;
  const int kj = at.row0 + (lane & 15);
  const float sigma = 1.0f / sqrtf((float)dh);
  f32x4 kf[DH / 16], vf[DH / 16], acck[DH / 64][4], accv[DH / 64][4];
  load_rows<T, DH, VEC>(kf, base + h, pitch, at.row0, seq - 1, dh, lane);
  load_rows<T, DH, VEC>(vf, base + 2 * h, pitch, at.row0, seq - 1, dh, lane);
#pragma unroll
  for (int b = 0; b < DH / 64; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) acck[b][e] = accv[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int q0 = (causal ? at.row0 : 0) + kRows * wave; q0 < seq; q0 += kRows * kWavesF) {
    f32x4 p, ds;
    {
      f32x4 qf[DH / 16], df[DH / 16];
      load_rows<T, DH, VEC>(qf, base, pitch, q0, seq - 1, dh, lane);
      load_rows<T, DH, VEC>(df, dob, (size_t)h, q0, seq - 1, dh, lane);
      float dl = 0.f;  // of query q0 + lane % 16
      if constexpr (DELTA) {
        f32x4 of[DH / 16];
        load_rows<T, DH, VEC>(of, o + (dob - d_o), (size_t)h, q0, seq - 1, dh, lane);
#pragma unroll
        for (int c = 0; c < DH / 16; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) dl = fmaf(df[c][e], of[c][e], dl);
        dl = quarters_sum(dl);
      }
      const f32x4 s = dot_rows(qf, kf), dp = dot_rows(df, vf);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qi = q0 + 4 * quarter + r, qc = min(qi, seq - 1);
        p[r] = (qi < seq && (!causal || kj <= qi)) ? expf(s[r] * sigma - lse_b[qc]) : 0.f;
        ds[r] = p[r] * (dp[r] - (DELTA ? __shfl(dl, 4 * quarter + r, 64) : delta_b[qc]));
      }
    }
    f32x4 qc[4][DH / 64], dc[4][DH / 64];
    load_cols<T, DH, VEC>(dc, dob, (size_t)h, q0, seq - 1, dh, lane);
    load_cols<T, DH, VEC>(qc, base, pitch, q0, seq - 1, dh, lane);
    add_outer(accv, dc, p);
    add_outer(acck, qc, ds);
  }
#pragma unroll
  for (int which = 0; which < 2; ++which) {  // dV, then dK through the same fold buffer
    if (which) __syncthreads();
    park<DH>(fold_f32 + wave * kRows * (DH + 4), which ? acck : accv, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < kRows * (DH / 4); i += kWavesF * 64) {
      const int row = i / (DH / 4), col = 4 * (i % (DH / 4));
      if (at.row0 + row < seq)
        store4<T, VEC>(dqkv + ((size_t)at.b * seq + at.row0 + row) * pitch + (size_t)at.head * dh + (which ? h : 2 * h), col, dh,
                       fold<DH>(fold_f32, row, col) * (which ? sigma : 1.0f));
    }
  }
}

template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(kWavesF * 64, 2) void attn_bwd_dq_f32(int block0, int seq, int heads, int dh, int causal, const T* __restrict__ qkv,
                                                                const T* __restrict__ o, const float* __restrict__ lse,
                                                                const T* __restrict__ d_o, T* __restrict__ dq, size_t ld_dq,
                                                                float* __restrict__ delta) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) float fold_f32[];
  dq_block_f32<T, DH, VEC>(fold_f32, place(seq, block0 + (int)blockIdx.z, causal != 0), seq, heads, dh, causal, qkv, o, lse, d_o, dq, ld_dq,
                           delta);
#endif
}

template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(kWavesF * 64, 2) void attn_bwd_dkv_f32(int block0, int seq, int heads, int dh, int causal, const T* qkv,
                                                                 const float* __restrict__ lse,
                                                                 const float* __restrict__ delta, const T* __restrict__ d_o, T* dqkv) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) float fold_f32[];
  dkv_block_f32<T, DH, VEC, false>(fold_f32, place(seq, block0 + (int)blockIdx.z, false), seq, heads, dh, causal, qkv, nullptr, lse,
                                   delta, d_o, dqkv);
#endif
}

// Both halves in one launch: a workgroup is a block of 16 queries (odd blocks) or of 16 keys, dealt out alternately with the
// longest of each first.  Nothing passes between them, and qkv must not be dqkv: every query block reads all keys.
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(kWavesF * 64, 2) void attn_bwd_f32(int block0, int seq, int heads, int dh, int causal, const T* __restrict__ qkv,
                                                             const T* __restrict__ o, const float* __restrict__ lse,
                                                             const T* __restrict__ d_o, T* __restrict__ dqkv) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) float fold_f32[];
  const int block = block0 + (int)blockIdx.z;
  const size_t pitch = (size_t)3 * heads * dh;
  if (block & 1)
    dq_block_f32<T, DH, VEC>(fold_f32, place(seq, block >> 1, causal != 0), seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, pitch, nullptr);
  else
    dkv_block_f32<T, DH, VEC, true>(fold_f32, place(seq, block >> 1, false), seq, heads, dh, causal, qkv, o, lse, nullptr, d_o, dqkv);
#endif
}

int check(const char* what, int batch, int seq, int heads, int dh) {
  if (batch <= 0 || seq <= 0 || heads <= 0) return fail(PMC_ERR_INVALID, "%s: batch=%d seq=%d heads=%d", what, batch, seq, heads);
  if (dh <= 0 || dh > kMaxDh) return fail(PMC_ERR_INVALID, "%s: head size %d not in 1..%d", what, dh, kMaxDh);
  if (heads > kMaxGrid || batch > kMaxGrid) return fail(PMC_ERR_INVALID, "%s: heads/batch exceed the grid limit", what);
  return PMC_OK;
}

// Calls launch(first row block, grid) for the row blocks of every (head, sequence) pair, in as many launches as the
// grid's third dimension needs.  (One dimension for all three holds fewer than 2^32 threads, 2^23 of these workgroups;
// a launch past that is not refused but leaves workgroups out.)
// halves = 2: query and key blocks are both counted.
template <typename Launch>
int for_row_blocks(const char* what, int batch, int seq, int heads, int halves, Launch launch) {
  const int64_t blocks = ((int64_t)seq + kRows - 1) / kRows * halves;
  for (int64_t b0 = 0; b0 < blocks; b0 += kMaxGrid) {
    launch((int)b0, dim3(heads, batch, (unsigned)(blocks - b0 < kMaxGrid ? blocks - b0 : kMaxGrid)));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PMC_ERR_HIP, "%s launch failed: %s", what, hipGetErrorString(e));
  }
  return PMC_OK;
}

template <int DH>
constexpr size_t fold_bytes() {
  return (size_t)kWavesF * kRows * (DH + 4) * sizeof(float);
}

// vec: 16-byte (fp32) or 8-byte (bf16) loads of four columns are aligned
template <typename T>
bool four_columns_aligned(int dh, const void* a, const void* b, const void* c) {
  const uintptr_t all = reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c);
  return dh % 4 == 0 && (all & (4 * sizeof(T) - 1)) == 0;
}

template <typename T, int DH, bool VEC>
int fwd_launch(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o, float* lse) {
  static std::atomic<bool> done{false};
  if (int rc = reserve_lds(attn_fwd_f32<T, DH, VEC>, fold_bytes<DH>(), done, "attention_forward")) return rc;
  return for_row_blocks("attention_forward", batch, seq, heads, 1, [&](int block0, dim3 grid) {
    attn_fwd_f32<T, DH, VEC><<<grid, dim3(kWavesF * 64), fold_bytes<DH>(), st>>>(block0, seq, heads, dh, causal, (const T*)qkv, (T*)o, lse);
  });
}

// dq (pitch ld_dq): a buffer of its own if dqkv is qkv, otherwise dqkv.
template <typename T, int DH, bool VEC>
int bwd_launch(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o, const float* lse,
               const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  static std::atomic<bool> done_dq{false}, done_dkv{false}, done_both{false};
  constexpr size_t lds = fold_bytes<DH>();
  if (dq == dqkv && attention_merged_f32(batch, seq, heads, causal)) {
    if (int rc = reserve_lds(attn_bwd_f32<T, DH, VEC>, lds, done_both, "attention_backward")) return rc;
    return for_row_blocks("attention_backward", batch, seq, heads, 2, [&](int block0, dim3 grid) {
      attn_bwd_f32<T, DH, VEC><<<grid, dim3(kWavesF * 64), lds, st>>>(block0, seq, heads, dh, causal, (const T*)qkv, (const T*)o, lse,
                                                                       (const T*)d_o, (T*)dqkv);
    });
  }
  if (int rc = reserve_lds(attn_bwd_dq_f32<T, DH, VEC>, lds, done_dq, "attention_backward")) return rc;
  if (int rc = reserve_lds(attn_bwd_dkv_f32<T, DH, VEC>, lds, done_dkv, "attention_backward")) return rc;
  int rc = for_row_blocks("attention_backward", batch, seq, heads, 1, [&](int block0, dim3 grid) {
    attn_bwd_dq_f32<T, DH, VEC><<<grid, dim3(kWavesF * 64), lds, st>>>(block0, seq, heads, dh, causal, (const T*)qkv, (const T*)o, lse,
                                                                        (const T*)d_o, (T*)dq, (size_t)ld_dq, delta);
  });
  if (rc) return rc;
  return for_row_blocks("attention_backward", batch, seq, heads, 1, [&](int block0, dim3 grid) {
    attn_bwd_dkv_f32<T, DH, VEC><<<grid, dim3(kWavesF * 64), lds, st>>>(block0, seq, heads, dh, causal, (const T*)qkv, lse, delta,
                                                                         (const T*)d_o, (T*)dqkv);
  });
}

template <typename T>
int fwd_t(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o, float* lse) {
  const bool vec = four_columns_aligned<T>(dh, qkv, o, o);
  if (dh <= 64)
    return vec ? fwd_launch<T, 64, true>(st, batch, seq, heads, dh, causal, qkv, o, lse)
               : fwd_launch<T, 64, false>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  return vec ? fwd_launch<T, 128, true>(st, batch, seq, heads, dh, causal, qkv, o, lse)
             : fwd_launch<T, 128, false>(st, batch, seq, heads, dh, causal, qkv, o, lse);
}

template <typename T>
int bwd_t(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o, const float* lse,
          const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  const bool vec = four_columns_aligned<T>(dh, qkv, o, d_o) && four_columns_aligned<T>(dh, dqkv, dq, dq);
  if (dh <= 64)
    return vec ? bwd_launch<T, 64, true>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta)
               : bwd_launch<T, 64, false>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  return vec ? bwd_launch<T, 128, true>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta)
             : bwd_launch<T, 128, false>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
}

}  // namespace

int attention_forward_f32(hipStream_t st, int dtype, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o,
                          float* lse) {
  if (int rc = check("attention_forward", batch, seq, heads, dh)) return rc;
  if (dtype == PMC_F32) return fwd_t<float>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  return fwd_t<bf16_t>(st, batch, seq, heads, dh, causal, qkv, o, lse);
}

// dq: see bwd_launch.  delta: fp32 [batch, heads, seq].
int attention_backward_f32(hipStream_t st, int dtype, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o,
                           const float* lse, const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  if (int rc = check("attention_backward", batch, seq, heads, dh)) return rc;
  if (dtype == PMC_F32) return bwd_t<float>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  return bwd_t<bf16_t>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
}

}  // namespace k
}  // namespace pmc
