// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate) for the
// projections of the three passes:
//   F: Y  = X . W  (+ bias, + residual, GeLU)      A stored [M,K], B stored [K,N]
//   B: dX = dY . W^T  (* GeLU')                    A stored [M,K], B stored [N,K]
//   W: dW += X^T . dY  (fp32 accumulate)           A stored [K,M], B stored [K,N]
// Two kernels share the fragment layouts and the epilogue:
//
//  * gemm_bf16_dma_kernel, the fast path.  Operand tiles go straight from
//    global memory into LDS (buffer_load ... lds, no registers in between) into a ring of 2 to 8
//    stages; rows past the edge are clamped, never branched on; what lies past K in the last K tile
//    arrives as zeros, because its addresses are outside the buffer descriptor.  LDS tiles are unpadded and
//    XOR-swizzled in 16-byte chunks so that both the DMA writes and the fragment reads are free of
//    bank conflicts.  The K loop is software pipelined by hand: while the MFMAs of one 16-wide K
//    step run, the fragments of the next step are read from LDS into a second register set, in a
//    fixed interleave; the barrier that releases a stage sits before the last K step of a tile, so
//    the first fragments of the next tile are read under that step's MFMAs and no LDS latency is
//    exposed at tile boundaries.  The DMA loads are issued as inline assembly and waited for with
//    explicit vmcnt values, because the compiler would otherwise drain every outstanding load
//    before each LDS read.
//  * gemm_bf16_kernel, the general path (operands of 2 GB and more, all layout/epilogue combinations):
//    global -> registers -> padded LDS tiles, double buffered.
//
// An operand whose contraction index is contiguous in memory is read from LDS with 16-byte loads;
// one whose contraction index is the slow dimension (W in F; X and dY in W) keeps its natural
// layout in LDS and is read with the transposing load ds_read_b64_tr_b16, so no operand is ever
// transposed in HBM.  The MFMA is issued with the operand roles exchanged (B-fragment as first
// operand), which leaves every lane with four consecutive output columns of one row and lets the
// epilogue use 8/16-byte accesses.  Workgroup ids are remapped so that the ids resident on one XCD
// (they are dealt round-robin over the 8 XCDs) cover a compact group of tiles and share operand
// panels in that XCD's L2.
#include <algorithm>
#include <cstdlib>

#include "dev_common.h"
#include "kernels.h"
#include "wgrad_batch.h"

namespace pmc {
namespace k {
namespace {

constexpr int kMaxSegments = PMC_MAX_QUEUED_W;

struct GemmParams {
  const bf16_t* A;
  const bf16_t* B;
  void* C;
  const bf16_t* bias;
  const bf16_t* resid;
  bf16_t* aux;
  int M, N, K, lda, ldb, ldc;
  int tiles_m, tiles_n;
  int group_m;            // height, in tiles, of the column groups the tiles are walked in (see tile_of_pid)
  int splits, k_tiles_per_split;  // fast path: 64-wide K tiles of each range (all of K when not split)
  bool own_xcds;                  // partial products: a range of K has XCDs of its own (see split_of_block)
  // Segmented contraction (weight gradients of several queued microbatches in one product): the K
  // axis is the concatenation of nseg pieces of seg_k rows each (every piece fills whole K tiles of its
  // own, the last one with zeros), piece i living at (Aseg[i], Bseg[i]) with the pitches lda, ldb.
  // nseg = 0: one piece at (A, B).
  const bf16_t* Aseg[kMaxSegments];
  const bf16_t* Bseg[kMaxSegments];
  int nseg, seg_k;
  __device__ __forceinline__ const bf16_t* piece_a(int i) const { return Aseg[i]; }
  __device__ __forceinline__ const bf16_t* piece_b(int i) const { return Bseg[i]; }
};

// K tiles of depth BK of the whole (possibly segmented) contraction.
template <bool SEG, int BK>
__host__ __device__ inline int k_tiles(const GemmParams& p) {
  return SEG ? p.nseg * ((p.seg_k + BK - 1) / BK) : (p.K + BK - 1) / BK;
}

constexpr int kEpiPartial = 100;  // fast path, split K: store an fp32 partial product

constexpr int kPadK = 8;    // K-major tile: row pitch BK + 8 elements (144 B for BK = 64)
constexpr int kPadMN = 32;  // MN-major tile: row pitch ROWS + 32 elements (pitch = 64 mod 256 bytes)

template <int ROWS, int BK, bool KMAJ>
struct Tile {
  static constexpr int pitch = KMAJ ? BK + kPadK : ROWS + kPadMN;
  static constexpr int elems = KMAJ ? ROWS * pitch : BK * pitch;
};

// Global -> register staging of one operand tile: CH 16-byte chunks per thread.
template <int ROWS, int BK, bool KMAJ, int NT>
struct Stager {
  static constexpr int CH = ROWS * BK / 8 / NT;
  static_assert(ROWS * BK / 8 % NT == 0, "tile must split evenly over the threads");
  u32x4 r[CH];

  __device__ __forceinline__ void load(const bf16_t* __restrict__ base, int ld, int mn0, int k0, int mn_total, int K,
                                       int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT;
      int mn, kk;
      if (KMAJ) {
        mn = c / (BK / 8);
        kk = (c % (BK / 8)) * 8;
      } else {
        kk = c / (ROWS / 8);
        mn = (c % (ROWS / 8)) * 8;
      }
      const bool ok = (mn0 + mn < mn_total) && (k0 + kk < K);
      const size_t off = KMAJ ? (size_t)(mn0 + mn) * ld + (k0 + kk) : (size_t)(k0 + kk) * ld + (mn0 + mn);
      u32x4 z = {0u, 0u, 0u, 0u};
      r[i] = ok ? *reinterpret_cast<const u32x4*>(base + off) : z;
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds, int tid) const {
    constexpr int pitch = Tile<ROWS, BK, KMAJ>::pitch;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT;
      int off;
      if (KMAJ) off = (c / (BK / 8)) * pitch + (c % (BK / 8)) * 8;
      else off = (c / (ROWS / 8)) * pitch + (c % (ROWS / 8)) * 8;
      *reinterpret_cast<u32x4*>(lds + off) = r[i];
    }
  }
};

// MFMA operand fragment for 32 rows starting at r0 and 16 contraction indices starting at ks:
// lane l holds row r0 + l%32, contraction indices ks + 8*(l/32) .. +7.
template <int ROWS, int BK, bool KMAJ>
__device__ __forceinline__ bf16x8 read_frag(const bf16_t* lds, int r0, int ks, int lane) {
  constexpr int pitch = Tile<ROWS, BK, KMAJ>::pitch;
  if (KMAJ) {
    return *reinterpret_cast<const bf16x8*>(lds + (r0 + (lane & 31)) * pitch + ks + 8 * (lane >> 5));
  } else {
    // ds_read_b64_tr_b16 works on groups of 16 lanes: lane j of a group supplies the address of 4
    // consecutive elements of row j/4 (piece j%4 of a 16-element span) and receives the 4 rows of
    // column j.  Groups 0..3 of the wave cover (columns 0-15 | 16-31) x (k 0-7 | 8-15).
    const int g = lane >> 4, j = lane & 15;
    const bf16_t* p = lds + (ks + 8 * (g >> 1) + (j >> 2)) * pitch + r0 + 16 * (g & 1) + 4 * (j & 3);
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * pitch));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

__device__ __forceinline__ void unpack4(u32x2 v, float* f) {
  f[0] = bf16lo_to_f32(v[0]); f[1] = bf16hi_to_f32(v[0]); f[2] = bf16lo_to_f32(v[1]); f[3] = bf16hi_to_f32(v[1]);
}
__device__ __forceinline__ u32x2 pack4(const float* f) {
  u32x2 v = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])};
  return v;
}

// Applies epilogue EPI to four consecutive output columns n .. n+3 of row m and stores them.
template <int EPI>
__device__ __forceinline__ void store_quad(const GemmParams& p, float (&v)[4], int m, int n) {
  const size_t idx = (size_t)m * p.ldc + n;
  if (EPI == kEpiPartial) {
    float* c = reinterpret_cast<float*>(p.C) + (size_t)m * p.N + n;
    f32x4 out = {v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4*>(c) = out;
    return;
  }
  if (EPI == PMC_EPI_ACCUM_F32) {
    float* c = reinterpret_cast<float*>(p.C) + idx;
    f32x4 old = *reinterpret_cast<f32x4*>(c);
    f32x4 out = {old[0] + v[0], old[1] + v[1], old[2] + v[2], old[3] + v[3]};
    *reinterpret_cast<f32x4*>(c) = out;
    return;
  }
  bf16_t* c = reinterpret_cast<bf16_t*>(p.C) + idx;
  if (EPI == PMC_EPI_BIAS || EPI == PMC_EPI_BIAS_RESID || EPI == PMC_EPI_BIAS_GELU || EPI == PMC_EPI_BIAS_GELU_GRAD) {
    float b[4];
    unpack4(*reinterpret_cast<const u32x2*>(p.bias + n), b);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += b[e];
  }
  if (EPI == PMC_EPI_BIAS_RESID) {
    float r[4];
    unpack4(*reinterpret_cast<const u32x2*>(p.resid + idx), r);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += r[e];
  }
  if (EPI == PMC_EPI_DGELU) {
    float u[4];
    unpack4(*reinterpret_cast<const u32x2*>(p.aux + idx), u);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_fast(u[e]);
  }
  if (EPI == PMC_EPI_MUL) {
    float u[4];
    unpack4(*reinterpret_cast<const u32x2*>(p.aux + idx), u);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= u[e];
  }
  if (EPI == PMC_EPI_BIAS_GELU_GRAD) {
    float g[4], dg[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) gelu_both_fast(v[e], g[e], dg[e]);
    *reinterpret_cast<u32x2*>(c) = pack4(dg);
    *reinterpret_cast<u32x2*>(p.aux + idx) = pack4(g);
    return;
  }
  *reinterpret_cast<u32x2*>(c) = pack4(v);
  if (EPI == PMC_EPI_BIAS_GELU) {
    float g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = gelu_fast(v[e]);
    *reinterpret_cast<u32x2*>(p.aux + idx) = pack4(g);
  }
}

// Epilogue shared by both kernels.  acc[i][j][r] of a wave whose tile starts at (mw0, nw0): row
// m = mw0 + 32 i + lane%32, columns n = nw0 + 32 j + 8 (r/4) + 4 (lane/32) + r%4.
template <int TM, int TN, int EPI>
__device__ __forceinline__ void epilogue(const GemmParams& p, f32x16 (&acc)[TM][TN], int mw0, int nw0, int lane) {
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = mw0 + 32 * i + (lane & 31);
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = nw0 + 32 * j + 8 * q + 4 * (lane >> 5);
        if (n >= p.N) continue;
        float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        store_quad<EPI>(p, v, m, n);
      }
    }
  }
}

__device__ __forceinline__ void unpack8(u32x4 v, float* f) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = bf16lo_to_f32(v[e]);
    f[2 * e + 1] = bf16hi_to_f32(v[e]);
  }
}
__device__ __forceinline__ u32x4 pack8(const float* f) {
  u32x4 v = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])};
  return v;
}

// What an epilogue reads besides the bias for eight consecutive output columns: the old fp32 sums
// (ACCUM), the residual (BIAS_RESID) or the GeLU input (DGELU).  Fetched ahead of use, a whole
// 32-row slab at a time, so that many loads are in flight per wave.
template <int EPI>
struct OctOperand {
  f32x4 lo, hi;  // ACCUM
  u32x4 packed;  // BIAS_RESID, DGELU
  static constexpr bool used =
      EPI == PMC_EPI_ACCUM_F32 || EPI == PMC_EPI_BIAS_RESID || EPI == PMC_EPI_DGELU || EPI == PMC_EPI_MUL;
  __device__ __forceinline__ void load(const GemmParams& p, int m, int n) {
    const size_t idx = (size_t)m * p.ldc + n;
    if (EPI == PMC_EPI_ACCUM_F32) {
      // streamed once: keep the fp32 sums out of the way of the operand panels in L2
      const float* c = reinterpret_cast<const float*>(p.C) + idx;
      lo = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(c));
      hi = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(c + 4));
    } else if (EPI == PMC_EPI_BIAS_RESID) {
      packed = *reinterpret_cast<const u32x4*>(p.resid + idx);
    } else if (EPI == PMC_EPI_DGELU || EPI == PMC_EPI_MUL) {
      packed = *reinterpret_cast<const u32x4*>(p.aux + idx);
    }
  }
};

// Applies epilogue EPI to eight consecutive output columns n .. n+7 of row m and stores them
// (16 bytes per lane for bf16 results, 32 for fp32 ones).  Same arithmetic as store_quad.
template <int EPI>
__device__ __forceinline__ void store_oct(const GemmParams& p, float (&v)[8], int m, int n, const OctOperand<EPI>& x) {
  const size_t idx = (size_t)m * p.ldc + n;
  if (EPI == kEpiPartial || EPI == PMC_EPI_ACCUM_F32) {
    float* c = EPI == kEpiPartial
                   ? reinterpret_cast<float*>(p.C) + (size_t)m * p.N + n
                   : reinterpret_cast<float*>(p.C) + idx;
    f32x4 lo = {v[0], v[1], v[2], v[3]}, hi = {v[4], v[5], v[6], v[7]};
    if (EPI == PMC_EPI_ACCUM_F32) {
      lo = x.lo + lo;
      hi = x.hi + hi;
      __builtin_nontemporal_store(lo, reinterpret_cast<f32x4*>(c));
      __builtin_nontemporal_store(hi, reinterpret_cast<f32x4*>(c + 4));
      return;
    }
    *reinterpret_cast<f32x4*>(c) = lo;
    *reinterpret_cast<f32x4*>(c + 4) = hi;
    return;
  }
  if (EPI == PMC_EPI_BIAS || EPI == PMC_EPI_BIAS_RESID || EPI == PMC_EPI_BIAS_GELU || EPI == PMC_EPI_BIAS_GELU_GRAD) {
    float b[8];
    unpack8(*reinterpret_cast<const u32x4*>(p.bias + n), b);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += b[e];
  }
  if (EPI == PMC_EPI_BIAS_RESID) {
    float r[8];
    unpack8(x.packed, r);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += r[e];
  }
  if (EPI == PMC_EPI_DGELU) {
    float u[8];
    unpack8(x.packed, u);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_fast(u[e]);
  }
  if (EPI == PMC_EPI_MUL) {
    float u[8];
    unpack8(x.packed, u);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= u[e];
  }
  if (EPI == PMC_EPI_BIAS_GELU_GRAD) {
    float g[8], dg[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) gelu_both_fast(v[e], g[e], dg[e]);
    *reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(p.C) + idx) = pack8(dg);
    *reinterpret_cast<u32x4*>(p.aux + idx) = pack8(g);
    return;
  }
  *reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(p.C) + idx) = pack8(v);
  if (EPI == PMC_EPI_BIAS_GELU) {
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = gelu_fast(v[e]);
    *reinterpret_cast<u32x4*>(p.aux + idx) = pack8(g);
  }
}

// Epilogue of the fast path.  In the accumulator layout a store instruction would touch 32 rows
// with 16 bytes each; instead each wave passes its tile, 32 rows at a time, through a private
// LDS slab [32][32 TN + 4] of fp32 and reads it back with 8 consecutive columns per lane, so a
// store instruction covers whole 128-byte (bf16) or 256-byte (fp32) row segments.  The pitch of
// 32 TN + 4 words spreads both the column-quad writes and the row-major reads over all banks.
// Only the wave itself touches its slab: LDS operations of one wave complete in order, so no
// barrier is needed between the passes.
// J0, JN: the column tiles J0 .. J0 + JN - 1 of the wave's TN are staged (JN a power of two, so that
// whole rows divide a wave's 64 lanes); a tile that is 5 wide goes out as 4 + 1.
template <int TM, int TN, int EPI, int J0 = 0, int JN = TN>
__device__ __forceinline__ void epilogue_staged(const GemmParams& p, f32x16 (&acc)[TM][TN], float* slab, int mw0,
                                                int nw0_wave, int lane) {
  static_assert((JN & (JN - 1)) == 0 && JN <= 8 && J0 + JN <= TN, "column group");
  constexpr int WN = 32 * JN, PITCH = WN + 4;
  const int nw0 = nw0_wave + 32 * J0;
  constexpr int LPR = WN / 8;     // lanes per row on the way out
  constexpr int RPP = 64 / LPR;   // rows per pass
  constexpr int NPASS = 32 / RPP;
  const int orow = lane / LPR, ocol = 8 * (lane % LPR);
  const int n = nw0 + ocol;
  // operands of slab i + 1 are requested before slab i is staged and stored
  OctOperand<EPI> ahead[2][NPASS];
  auto fetch = [&](int i, OctOperand<EPI> (&dst)[NPASS]) {
    if (!OctOperand<EPI>::used) return;
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int m = mw0 + 32 * i + pass * RPP + orow;
      if (m < p.M && n < p.N) dst[pass].load(p, m, n);
    }
  };
  fetch(0, ahead[0]);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (i + 1 < TM) fetch(i + 1, ahead[(i + 1) & 1]);
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 t = {acc[i][J0 + j][4 * q], acc[i][J0 + j][4 * q + 1], acc[i][J0 + j][4 * q + 2], acc[i][J0 + j][4 * q + 3]};
        *reinterpret_cast<f32x4*>(slab + (lane & 31) * PITCH + 32 * j + 8 * q + 4 * (lane >> 5)) = t;
      }
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int row = pass * RPP + orow;
      const f32x4 lo = *reinterpret_cast<const f32x4*>(slab + row * PITCH + ocol);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(slab + row * PITCH + ocol + 4);
      const int m = mw0 + 32 * i + row;
      if (m < p.M && n < p.N) {
        float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        store_oct<EPI>(p, v, m, n, ahead[i & 1][pass]);
      }
    }
  }
}

// Epilogue of the K-split kernels: every wave holds a partial sum of the whole BM x BN tile.  Each leaves its
// sums in an LDS slab of its own; after the barrier the workgroup's threads add the slabs in wave order, eight
// columns per thread, and store whole row segments.
template <int BM, int BN, int NW, int EPI>
__device__ __forceinline__ void epilogue_ksplit(const GemmParams& p, f32x16 (&acc)[BM / 32][BN / 32], float* slabs, int m0, int n0,
                                                int wave, int lane) {
  constexpr int PITCH = BN + 4, SLAB = BM * PITCH, LPR = BN / 8, RPP = 64 * NW / LPR, NPASS = (BM + RPP - 1) / RPP;
  const int tid = wave * 64 + lane, orow = tid / LPR, ocol = 8 * (tid % LPR), n = n0 + ocol;
  OctOperand<EPI> ahead[NPASS];
#pragma unroll
  for (int pass = 0; pass < NPASS; ++pass) {
    const int row = pass * RPP + orow;
    if (OctOperand<EPI>::used && row < BM && m0 + row < p.M && n < p.N) ahead[pass].load(p, m0 + row, n);
  }
  float* my = slabs + wave * SLAB + (lane & 31) * PITCH + 4 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < BM / 32; ++i)
#pragma unroll
    for (int j = 0; j < BN / 32; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 t = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        *reinterpret_cast<f32x4*>(my + 32 * i * PITCH + 32 * j + 8 * q) = t;
      }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < NPASS; ++pass) {
    const int row = pass * RPP + orow;
    if (row >= BM || m0 + row >= p.M || n >= p.N) continue;
    const float* from = slabs + row * PITCH + ocol;
    f32x4 lo = *reinterpret_cast<const f32x4*>(from), hi = *reinterpret_cast<const f32x4*>(from + 4);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      lo += *reinterpret_cast<const f32x4*>(from + w * SLAB);
      hi += *reinterpret_cast<const f32x4*>(from + w * SLAB + 4);
    }
    float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    store_oct<EPI>(p, v, m0 + row, n, ahead[pass]);
  }
}

// Second half of a split-K product: adds the fp32 partials of the splits in ascending order (a
// fixed order, so the result does not depend on scheduling) and applies the epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmParams p, const float* __restrict__ partial, int splits) {
#if defined(__HIP_DEVICE_COMPILE__)
  const size_t quad = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t e0 = quad * 4, total = (size_t)p.M * p.N;
  if (e0 >= total) return;
  const int m = (int)(e0 / p.N), n = (int)(e0 % p.N);
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; ++s) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(partial + (size_t)s * total + e0);
    v[0] += t[0]; v[1] += t[1]; v[2] += t[2]; v[3] += t[3];
  }
  store_quad<EPI>(p, v, m, n);
#endif
}

// Workgroup id -> (tile_m, tile_n).  Ids are dealt round-robin over 8 XCDs; give each XCD a
// contiguous run of tile indices, then walk tiles in column groups group_m tiles of M tall.  The 32
// tiles an XCD works on at a time are then a block of group_m x 32/group_m tiles, whose operand
// panels (group_m BM rows of A, 32/group_m BN rows of B per K step) are what that XCD's L2 has to
// fetch.  Measured on whole steps: 4 for the 256-row tiles (+1 % at hidden 4096 over 8, nothing at
// 5120), 8 for the smaller ones (4 costs the 64 x 128 products 2 %).  The gemm_group tuning switch forces a height.
__device__ __forceinline__ void walk_tiles(const GemmParams& p, int pid, int& tile_m, int& tile_n) {
  const int GROUP = p.group_m;
  const int per_group = GROUP * p.tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GROUP;
  const int group_m = min(p.tiles_m - first_m, GROUP);
  tile_m = first_m + (pid % per_group) % group_m;
  tile_n = (pid % per_group) / group_m;
}
__device__ __forceinline__ void tile_of_pid(const GemmParams& p, int pid, int& tile_m, int& tile_n) {
  const int ntiles = p.tiles_m * p.tiles_n;
  const int xcd = pid & 7, local = pid >> 3, lo = ntiles >> 3, rem = ntiles & 7;
  walk_tiles(p, xcd * lo + (xcd < rem ? xcd : rem) + local, tile_m, tile_n);
}
// Partial product: workgroup -> (range of K, tile).  2, 4 or 8 ranges go to XCDs of their own, 4, 2 or 1 to a range, each a
// contiguous run of tiles: an XCD then fetches a share of K only, over a block of tiles that much larger, and an operand crosses the
// fabric 2 to 4 times less often (1024 x 2048 x 8192 in 4 ranges of 128x128 tiles: 67 MB instead of 168).  The grid is
// 8 x tiles per XCD; false: nothing to do.  Other counts (7 ranges of a K that is not divisible) deal the ranges out one after the other, and so
// does a single row of tiles, which shares no panel of B, with much to fetch: with B stored [K][N] from 64 MB of operands on (time with XCDs of their own over
// that in turn, 309 products, 0.99 in the memory-side cache and 1.01 from HBM, up to 1.14: 40 x 19968 x 6656 in 4 ranges, in turn / of their own, 52 / 57 and 63 / 70 us; below
// 0.97 and 0.99), with B stored [N][K] beyond the 256 MB of that cache (142: 1.00 and 1.01, up to 1.09: 112 x 8192 x 24576 in 8 ranges 98 / 106 us; below 0.99 and 1.01).
__host__ __device__ inline int tiles_per_xcd(int tiles, int splits) { return (tiles * splits + 7) / 8; }
}  // namespace
bool gemm_bf16_split_own_xcds(bool tb, int tiles_m, int M, int N, int K, int splits) {
  return 8 % splits == 0 && (tiles_m > 1 || ((size_t)M + N) * K * sizeof(bf16_t) < (tb ? 256u : 64u) << 20);
}
namespace {
__device__ __forceinline__ bool split_of_block(const GemmParams& p, int& split, int& tile_m, int& tile_n) {
  const int ntiles = p.tiles_m * p.tiles_n, id = blockIdx.x;
  if (p.own_xcds) {
    const int xcd = id & 7, local = id >> 3, per = tiles_per_xcd(ntiles, p.splits), tile = (xcd / p.splits) * per + local;
    split = xcd % p.splits;
    if (tile >= ntiles || local >= per) return false;
    walk_tiles(p, tile, tile_m, tile_n);
    return true;
  }
  split = id / ntiles;
  if (split >= p.splits) return false;
  tile_of_pid(p, id - split * ntiles, tile_m, tile_n);
  return true;
}
__device__ __forceinline__ void tile_of_block(const GemmParams& p, int& tile_m, int& tile_n) {
  tile_of_pid(p, blockIdx.x, tile_m, tile_n);
}

// ---------------------------------------------------------------------------------------------
// Fast path: direct-to-LDS operand tiles, swizzled, hand-pipelined.
//
// LDS tile layouts (BK = 64, no padding; a "chunk" is 16 bytes = 8 elements):
//   contraction-contiguous operand: [rows][64]; chunk position p of row r holds k-chunk
//       p ^ ((r >> 1) & 7)   -> 16 lanes reading 16 consecutive rows at one k hit 16 distinct
//       16-byte bank groups;
//   other operand: [64 k][ROWS]; chunk position p of k-row kr holds chunk p ^ kswz(kr) = p ^ ((kr & 3) << 2)
//       -> the four k-rows one half-wave touches in a transposing read fall into four different
//       64-byte bank quarters.
// One buffer_load...lds instruction of a wave fills 1 KB of LDS (lane l writes bytes 16 l .. 16 l + 15
// of it), so the swizzle is applied to the GLOBAL address each lane fetches from.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Chunk swizzle of k-row kr in a [64 k][ROWS] tile.  A k-row of 128 n rows (a multiple of 256 bytes)
// starts in the same bank as its neighbours, so the four k-rows of a transposing read are moved to
// four different 64-byte quarters by their two low bits.  In a 320-row tile (640 bytes per k-row)
// consecutive k-rows already sit 128 bytes apart; bit 1 of kr supplies the other 64 bytes, and
// flipping only bit 2 of the chunk index keeps every chunk inside its own group of 8 (320 / 8 = 40
// chunks per k-row is not a multiple of 16).  The 128-byte k-rows of a 64-row tile are the same case; the 64-byte ones
// of a 32-row tile fall into four quarters as they are.
template <int ROWS>
__device__ __forceinline__ constexpr int kswz(int kr) {
  return ROWS % 128 == 0 ? ((kr & 3) << 2) : ROWS == 32 ? 0 : (((kr >> 1) & 1) << 2);
}

// BK: K rows of the tile; 64 everywhere except the [32 k][ROWS] tiles of the two-workgroup weight-gradient kernel
// (the [rows][64] layout's swizzle is defined for 64 only).
template <int ROWS, bool KMAJ, int NW, int BK = 64>
struct DmaLoader {
  static constexpr int NL = ROWS * BK * 2 / 1024 / NW;  // 1 KB loads per wave per tile
  static_assert(ROWS * BK * 2 / 1024 % NW == 0, "tile must split evenly over the waves");
  static_assert(BK == 64 || (!KMAJ && BK == 32), "K depth of a tile");
  static_assert(KMAJ || ROWS % 128 == 0 || ROWS == 320 || ROWS == 64 || ROWS == 32, "the [64 k][rows] swizzle is not defined for this width");
  uint32_t voff[NL];  // byte offset of this lane's chunk at K offset 0

  // Wave w issues loads w*NL .. w*NL+NL-1; load q fills tile bytes [1024 q, 1024 q + 1024).
  // Rows (or columns) past the edge of the matrix are clamped to the last valid ones: what they
  // produce lands in output rows/columns that the epilogue does not store.
  __device__ __forceinline__ void init(int ld, int mn0, int mn_total, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int q = wave * NL + i;
      if (KMAJ) {
        const int row = q * 8 + (lane >> 3), pos = lane & 7;
        const int kc = pos ^ ((row >> 1) & 7);
        int grow = mn0 + row;
        grow = grow < mn_total ? grow : mn_total - 1;
        voff[i] = ((uint32_t)grow * (uint32_t)ld + kc * 8) * 2;
      } else {
        constexpr int CPR = ROWS / 8;  // chunks per k-row
        const int idx = q * 64 + lane, kr = idx / CPR, pos = idx % CPR;
        const int mc = pos ^ kswz<ROWS>(kr);
        int gmn = mn0 + mc * 8;
        gmn = gmn < mn_total ? gmn : mn_total - 8;
        voff[i] = ((uint32_t)kr * (uint32_t)ld + gmn) * 2;
      }
    }
  }
  // Last K tile of a contraction-contiguous operand, of which only `valid` (a multiple of 8) columns
  // exist: the chunks past them get an offset outside the descriptor, which reads as zero.
  __device__ __forceinline__ void cut(int valid, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = (wave * NL + i) * 8 + (lane >> 3);
      if ((((lane & 7) ^ ((row >> 1) & 7)) << 3) >= valid) voff[i] = 0x80000000u;
    }
  }
  __device__ __forceinline__ void issue(i32x4 rsrc, bf16_t* tile, uint32_t soff, int wave) const {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int q = wave * NL + i;
      const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)((lds_void_ptr)(tile + q * 512)));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds_addr), "v"(voff[i]), "s"(rsrc), "s"(soff) : "memory");
    }
  }
};

template <int ROWS, bool KMAJ>
__device__ __forceinline__ bf16x8 read_frag_swz(const bf16_t* tile, int r0, int ks, int lane) {
  if (KMAJ) {
    const int row = r0 + (lane & 31), kc = (ks >> 3) + (lane >> 5);
    return *reinterpret_cast<const bf16x8*>(tile + row * 64 + ((kc ^ ((row >> 1) & 7)) << 3));
  } else {
    const int g = lane >> 4, j = lane & 15;
    const int kr = ks + 8 * (g >> 1) + (j >> 2);  // the swizzle is the same for kr and kr + 4
    const int col = r0 + 16 * (g & 1) + 4 * (j & 3);
    const bf16_t* p = tile + kr * ROWS + (col ^ (kswz<ROWS>(kr) << 3));
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * ROWS));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

// One output tile (tile_m, tile_n) over the K tiles kt0 .. kt0 + nk - 1: ring prologue, K loop,
// staged epilogue.  All waves of the workgroup call it together; on return the LDS ring holds
// epilogue slabs that other waves may still be reading (barrier before the ring is filled again).
// BK = 32 (both operands [k][rows] only): kt0 and nk count 32-wide K tiles, two 16-wide steps per tile.
// KSPLIT: for tiles of 64 x 64 and less, which are bound by the serial chain of a K tile (LDS latency, then
// matrix instructions, four times per tile) rather than by any rate.  Every wave owns the whole output tile and
// one of the four 16-wide steps of each K tile, so a K tile is one such link instead of four and each LDS byte
// is read once; the four partial tiles are added at the end.  Kernel times, 128x128 / 64x128 tiles (before)
// against these: 192 x 256 x 1024 (F) 13.7 / 8.3 -> 5.7 us, 496 x 832 x 3328 (F) 39 / 18.6 -> 10.3,
// 1024 x 1024 x 4096 (W) 46.7 -> 17.1, 256 x 256 x 2048 (W) 25.6 -> 7.0.
// KG = 2: two groups of waves cover the output tile, each with one half of every K tile, and add their sums at the end.  For a
// workgroup that is alone on its compute unit with a wave to a SIMD: nothing covers that wave's reads from LDS and its waits, while
// more waves on smaller pieces of the tile would read more from LDS.  128x128 tiles, 4 waves / 8 in two groups, operands in the
// memory-side cache and from HBM: 2000 x 1600 x 6400 (F) 58.2 / 49.9 and 59.5 / 54.6 us, 2000 x 1600 x 1600 (F) 19.5 / 17.2 and 20.7 /
// 19.6, 4096 x 1024 x 4096 (F) 42.0 / 38.1 and 44.2 / 42.4, (B) 40.0 / 36.5 and 42.3 / 41.9, 4096 x 1024 x 1024 (B) 13.1 / 12.6 and 15.7 /
// 16.1.  Not for weight gradients (2048 x 2048 x 1024 from HBM 19.1 / 20.4) and not for 256x128 tiles, whose eight waves are two to
// a SIMD already (1024 x 8192 x 2048 36.9 / 37.6).
// CUT: the last K tile of a contraction-contiguous operand is partial.  (A kernel of its own: the test for
// that tile in the K loop cost the steps whose K is whole 0.3 to 1 %.)
template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KMAJ, bool B_KMAJ, int NSTAGE, int EPI, bool SEG = false, int BK = 64, bool CUT = false,
          bool KSPLIT = false, int KG = 1, class Params>
__device__ __forceinline__ void dma_tile(const Params& p, bf16_t* smem, int tile_m, int tile_n, int kt0, int nk) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NWG = WAVES_M * WAVES_N, NW = NWG * KG, WM = KSPLIT ? BM : BM / WAVES_M, WN = KSPLIT ? BN : BN / WAVES_N, TM = WM / 32, TN = WN / 32;
  constexpr int TA = BM * BK, TB = BN * BK, STAGE = TA + TB;
  static_assert(!KSPLIT || BK == 16 * NW, "K split over the waves: one 16-wide step of a K tile each");
  static_assert(KG == 1 || (KG == 2 && BK == 64 && !KSPLIT && TM % 2 == 0), "K groups");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = wave % NWG, kg = KG > 1 ? wave / NWG : 0;
  const int wm0 = KSPLIT ? 0 : (wg / WAVES_N) * WM, wn0 = KSPLIT ? 0 : (wg % WAVES_N) * WN;
  const int ks0 = KSPLIT ? 16 * wave : (BK / KG) * kg;  // first contraction index of this wave in a K tile
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // Raw buffer descriptor: base, no stride, size.  A [k][rows] operand's size ends with its last k-row,
  // so the k-rows of the last K tile that do not exist read as zeros; a [rows][k] operand has a 2 GB
  // window and its last K tile is cut (see request).
  auto make_rsrc = [](const void* ptr, uint32_t bytes) {
    const uint64_t a = (uint64_t)ptr;
    i32x4 r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    return r;
  };
  const uint32_t k_rows = SEG ? p.seg_k : p.K;
  const uint32_t size_a = A_KMAJ ? 0x7fffffffu : k_rows * (uint32_t)p.lda * 2, size_b = B_KMAJ ? 0x7fffffffu : k_rows * (uint32_t)p.ldb * 2;
  i32x4 ra = make_rsrc(p.A, size_a), rb = make_rsrc(p.B, size_b);
  DmaLoader<BM, A_KMAJ, NW, BK> la;
  DmaLoader<BN, B_KMAJ, NW, BK> lb;
  la.init(p.lda, m0, p.M, wave, lane);
  lb.init(p.ldb, n0, p.N, wave, lane);
  const uint32_t stepa = A_KMAJ ? BK * 2 : (uint32_t)BK * p.lda * 2;
  const uint32_t stepb = B_KMAJ ? BK * 2 : (uint32_t)BK * p.ldb * 2;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  bf16x8 fa[2][TM], fb[2][TN];
  // One 16-wide K step: the MFMAs on fragment set c, interleaved in a fixed order with the LDS
  // reads that fill set c^1 from (src_a, src_b) at K offset ks.
  auto step = [&](int c, const bf16_t* src_a, const bf16_t* src_b, int ks) {
#pragma unroll
    for (int q = 0; q < TM + TN; ++q) {
      if (q < TM) fa[c ^ 1][q] = read_frag_swz<BM, A_KMAJ>(src_a, wm0 + 32 * q, ks, lane);
      else fb[c ^ 1][q - TM] = read_frag_swz<BN, B_KMAJ>(src_b, wn0 + 32 * (q - TM), ks, lane);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int NP = TM + TN, TOT = TM * TN;
#pragma unroll
      for (int idx = (q * TOT) / NP; idx < ((q + 1) * TOT) / NP; ++idx) {
        const int i = idx / TN, j = idx % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][j], fa[c][i], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Ring of NSTAGE stages.  Tiles past the end are clamped (fetched again, never used) so that the
  // number of loads in flight is the same at every wait.
  constexpr int LPT = DmaLoader<BM, A_KMAJ, NW, BK>::NL + DmaLoader<BN, B_KMAJ, NW, BK>::NL;  // loads per tile per wave
  constexpr int INFL = (NSTAGE - 2) * LPT;  // loads that may stay in flight at a wait
  static_assert(INFL < 64, "vmcnt is a 6-bit field");
  constexpr int WAIT_TILE = (INFL & 15) | ((INFL >> 4) << 14) | (7 << 4) | (15 << 8);  // s_waitcnt vmcnt(INFL)
  auto tile_k = [&](int t) { return kt0 + (t < nk ? t : nk - 1); };
  // Requests K tile t of this call into a stage.  Segmented: tile kt0 + t of the concatenated axis
  // is tile `local` of piece `seg`; the two are stepped along with the requests (which come in
  // ascending t), so no division sits in the loop.
  int seg = 0, local = 0;
  const int seg_tiles = SEG ? (p.seg_k + BK - 1) / BK : 0;  // K tiles of this depth per piece
  if constexpr (SEG) {
    seg = kt0 / seg_tiles;
    local = kt0 - seg * seg_tiles;
    ra = make_rsrc(p.piece_a(seg), size_a);
    rb = make_rsrc(p.piece_b(seg), size_b);
  }
  auto request = [&](int t, int stage) {
    const int kt = SEG ? local : tile_k(t);
    if constexpr (CUT) {
      if (kt == p.K >> 6) {  // requests come in ascending order, and past the end this tile is requested again
        if constexpr (A_KMAJ) la.cut(p.K & 63, wave, lane);
        if constexpr (B_KMAJ) lb.cut(p.K & 63, wave, lane);
      }
    }
    la.issue(ra, smem + stage * STAGE, kt * stepa, wave);
    lb.issue(rb, smem + stage * STAGE + TA, kt * stepb, wave);
    if (SEG && t + 1 < nk) {  // past the end the last tile is requested again
      if (++local == seg_tiles) {
        local = 0;
        ++seg;
        ra = make_rsrc(p.piece_a(seg), size_a);
        rb = make_rsrc(p.piece_b(seg), size_b);
      }
    }
  };
#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t) request(t, t);
  __builtin_amdgcn_s_waitcnt(WAIT_TILE);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[0][i] = read_frag_swz<BM, A_KMAJ>(smem, wm0 + 32 * i, ks0, lane);
#pragma unroll
  for (int j = 0; j < TN; ++j) fb[0][j] = read_frag_swz<BN, B_KMAJ>(smem + TA, wn0 + 32 * j, ks0, lane);
  int cur = 0;
  if constexpr (KSPLIT) {
    auto k_tile = [&](int c, int kt) {
      request(kt + NSTAGE - 1, cur == 0 ? NSTAGE - 1 : cur - 1);  // all its readers passed the last barrier
      __builtin_amdgcn_s_waitcnt(WAIT_TILE);
      __syncthreads();
      cur = cur + 1 == NSTAGE ? 0 : cur + 1;
      step(c, smem + cur * STAGE, smem + cur * STAGE + TA, 16 * wave);  // after the last tile: reads a clamped tile, unused
    };
    for (int kt = 0; kt < nk; kt += 2) {
      k_tile(0, kt);
      if (kt + 1 < nk) k_tile(1, kt + 1);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    epilogue_ksplit<BM, BN, NW, EPI>(p, acc, reinterpret_cast<float*>(smem), m0, n0, wave, lane);
    static_assert(!KSPLIT || NW * BM * (BN + 4) * 4 <= NSTAGE * STAGE * 2, "partial tiles must fit in the stage ring");
    return;
  }
  for (int kt = 0; kt < nk; ++kt) {
    const bf16_t* cur_a = smem + cur * STAGE;
    const bf16_t* cur_b = cur_a + TA;
    const int nxt = cur + 1 == NSTAGE ? 0 : cur + 1;
    const int fill = cur == 0 ? NSTAGE - 1 : cur - 1;  // all its readers passed the last barrier
    request(kt + NSTAGE - 1, fill);
    step(0, cur_a, cur_b, ks0 + 16);
    if constexpr (BK / KG == 64) {
      step(1, cur_a, cur_b, 32);
      step(0, cur_a, cur_b, 48);
    }
    // Tile kt+1 must have landed (younger tiles may still be in flight).  Every fragment of tile
    // kt is in registers, so after this barrier its stage may be refilled.
    __builtin_amdgcn_s_waitcnt(WAIT_TILE);
    __syncthreads();
    step(1, smem + nxt * STAGE, smem + nxt * STAGE + TA, ks0);  // after the last tile: a clamped tile, unused
    cur = nxt;
  }
  // vmcnt(0): drain the clamped tail loads; after the barrier no wave reads or fills a stage any
  // more and the ring is reused for the epilogue slabs.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  constexpr int JN = TN == 5 ? 4 : TN;  // widest column group of the staged epilogue
  static_assert(NW * 32 * (32 * JN + 4) * 4 <= NSTAGE * STAGE * 2, "epilogue slabs must fit in the stage ring");
  float* slab = reinterpret_cast<float*>(smem) + wave * (32 * (32 * JN + 4));
  if constexpr (KG == 2) {
    // The two waves of a tile exchange halves of their sums: group g finishes the rows 32 (TM / 2) g on.  What a wave
    // receives lies where its own slab will be.
    constexpr int H = TM / 2;
    static_assert(H * TN * 1024 <= 32 * (32 * JN + 4) || H == 1, "the sums of half a tile must fit in a slab");
    float* to = reinterpret_cast<float*>(smem) + ((1 - kg) * NWG + wg) * (32 * (32 * JN + 4)) + lane;
    f32x16 half[H][TN];
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x16 give = kg ? acc[i][j] : acc[H + i][j];
        half[i][j] = kg ? acc[H + i][j] : acc[i][j];
#pragma unroll
        for (int r = 0; r < 16; ++r) to[((i * TN + j) * 16 + r) * 64] = give[r];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) half[i][j][r] += slab[((i * TN + j) * 16 + r) * 64 + lane];
    epilogue_staged<H, TN, EPI, 0, JN>(p, half, slab, m0 + wm0 + 32 * H * kg, n0 + wn0, lane);
    return;
  }
  epilogue_staged<TM, TN, EPI, 0, JN>(p, acc, slab, m0 + wm0, n0 + wn0, lane);
  if constexpr (TN == 5) epilogue_staged<TM, TN, EPI, 4, 1>(p, acc, slab, m0 + wm0, n0 + wn0, lane);
#endif
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KMAJ, bool B_KMAJ, int NSTAGE, int EPI, bool SEG = false, int BK = 64,
          bool CUT = false, bool KSPLIT = false, int KG = 1>
__global__ __launch_bounds__(WAVES_M * WAVES_N * KG * 64) void gemm_bf16_dma_kernel(GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  int tile_m, tile_n;
  const int per = p.k_tiles_per_split * (64 / BK);
  if constexpr (EPI == kEpiPartial) {
    int split;
    if (!split_of_block(p, split, tile_m, tile_n)) return;
    GemmParams part = p;
    part.C = reinterpret_cast<float*>(p.C) + (size_t)split * p.M * p.N;
    dma_tile<BM, BN, WAVES_M, WAVES_N, A_KMAJ, B_KMAJ, NSTAGE, EPI, SEG, BK, CUT, KSPLIT, KG>(part, smem, tile_m, tile_n, split * per,
                                                                                         min(per, k_tiles<SEG, BK>(p) - split * per));
  } else {
    tile_of_block(p, tile_m, tile_n);
    dma_tile<BM, BN, WAVES_M, WAVES_N, A_KMAJ, B_KMAJ, NSTAGE, EPI, SEG, BK, CUT, KSPLIT, KG>(p, smem, tile_m, tile_n, 0, k_tiles<SEG, BK>(p));
  }
#endif
}

// Weight-gradient products (fp32 C += A^T B) with several rounds of tiles per compute unit: one
// persistent workgroup per unit walks its tiles.  The read-modify-write of C runs at HBM speed and
// the K loop at matrix-core speed, and a workgroup cannot do both at once; if all workgroups start
// together they stay in step, every K loop finds the memory idle and every epilogue finds it
// saturated.  So the workgroups are put out of phase, without idling anyone: group g of G (by
// workgroup id) starts its first tile at K tile g/G of the way through, and comes back for that
// tile's first K tiles after its last tile.  Both parts are added into C by the same workgroup, in
// that order, so the result depends on the launch shape alone.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, int GROUPS, bool SEG = false, int BK = 64>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64) void gemm_bf16_wgrad_persistent_kernel(GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  const int ntiles = p.tiles_m * p.tiles_n, G = gridDim.x, b = blockIdx.x;
  const int nk = k_tiles<SEG, BK>(p);
  const int group = (b >> 3) % GROUPS;  // neighbours on one XCD fall into different groups
  const int head = (nk * group) / GROUPS;  // K tiles of the first tile left for the end
  bool first = true;
  int tm0 = 0, tn0 = 0;
  for (int pid = b; pid < ntiles; pid += G) {
    int tile_m, tile_n;
    tile_of_pid(p, pid, tile_m, tile_n);
    if (first) {
      tm0 = tile_m;
      tn0 = tile_n;
      dma_tile<BM, BN, WAVES_M, WAVES_N, false, false, NSTAGE, PMC_EPI_ACCUM_F32, SEG, BK>(p, smem, tile_m, tile_n, head, nk - head);
      first = false;
    } else {
      dma_tile<BM, BN, WAVES_M, WAVES_N, false, false, NSTAGE, PMC_EPI_ACCUM_F32, SEG, BK>(p, smem, tile_m, tile_n, 0, nk);
    }
    __syncthreads();
  }
  if (!first && head > 0)
    dma_tile<BM, BN, WAVES_M, WAVES_N, false, false, NSTAGE, PMC_EPI_ACCUM_F32, SEG, BK>(p, smem, tm0, tn0, 0, head);
#endif
}

// Weight-gradient products, two workgroups per compute unit: 256x128 tiles, four waves of 128x64
// (the same wave tile as the kernels above, so the same LDS traffic per matrix instruction), a ring of
// three 32-deep stages (72 KB).  Two such workgroups fit a compute unit (144 KB of LDS, two waves per
// SIMD), each with its own barriers: while one adds its finished tile into C at memory speed, the other
// runs its K loop, without any arrangement between them, and the two waves of a SIMD no longer wait at
// the same barrier.  Both operands of a weight gradient are stored [k][rows], so a 32-deep tile still
// reads whole 256- and 512-byte rows.
template <bool SEG>
__global__ __launch_bounds__(256, 2) void gemm_bf16_wgrad_pair_kernel(GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  int tile_m, tile_n;
  tile_of_block(p, tile_m, tile_n);
  dma_tile<256, 128, 2, 2, false, false, 3, PMC_EPI_ACCUM_F32, SEG, 32>(p, smem, tile_m, tile_n, 0, k_tiles<SEG, 32>(p));
#endif
}

// One product of a W pass in one launch: what dma_tile and the epilogue read, with the operands taken from the slabs.
struct BatchProduct : GemmParams {
  const WgradBatchParams* q;
  size_t off_a, off_b;
  __device__ __forceinline__ const bf16_t* piece_a(int i) const { return reinterpret_cast<const bf16_t*>(q->w.piece[i] + off_a); }
  __device__ __forceinline__ const bf16_t* piece_b(int i) const { return reinterpret_cast<const bf16_t*>(q->w.piece[i] + off_b); }
};

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, int BK, bool KSPLIT, int WAVES_PER_SIMD>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, WAVES_PER_SIMD) void gemm_bf16_wgrad_batch_kernel(WgradBatchParams q) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  if ((int)blockIdx.x < q.sum_blocks) {
    batch_column_sums<bf16_t, WAVES_M * WAVES_N * 64>(q, blockIdx.x, reinterpret_cast<float*>(smem));
    return;
  }
  const BatchTile t = batch_tile(q, (int)blockIdx.x - q.sum_blocks);
  const WgradBatchArgs::Layer& l = q.w.layer[t.layer];
  BatchProduct p;
  p.q = &q;
  p.off_a = l.a[t.product];
  p.off_b = l.b[t.product];
  p.C = l.c[t.product];
  p.A = p.B = nullptr;
  p.bias = p.resid = nullptr;
  p.aux = nullptr;
  p.M = p.lda = q.w.M[t.product];
  p.N = p.ldb = p.ldc = q.w.N[t.product];
  p.nseg = q.w.pieces;
  p.seg_k = q.w.K;
  p.K = q.w.K;
  dma_tile<BM, BN, WAVES_M, WAVES_N, false, false, NSTAGE, PMC_EPI_ACCUM_F32, true, BK, false, KSPLIT>(p, smem, t.tile_m, t.tile_n, 0,
                                                                                                  k_tiles<true, BK>(p));
#endif
}

// ---------------------------------------------------------------------------------------------
// General path.
template <int BM, int BN, int BK, int WM, int WN, bool A_KMAJ, bool B_KMAJ, int EPI>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void gemm_bf16_kernel(GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int WAVES_N = BN / WN;
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  constexpr int TM = WM / 32, TN = WN / 32;
  using TileA = Tile<BM, BK, A_KMAJ>;
  using TileB = Tile<BN, BK, B_KMAJ>;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int kStage = TileA::elems + TileB::elems;  // one buffer: A tile then B tile

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;

  int tile_m, tile_n;
  tile_of_block(p, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  Stager<BM, BK, A_KMAJ, NT> sa;
  Stager<BN, BK, B_KMAJ, NT> sb;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (p.K + BK - 1) / BK;
  sa.load(p.A, p.lda, m0, 0, p.M, p.K, tid);
  sb.load(p.B, p.ldb, n0, 0, p.N, p.K, tid);
  sa.store(smem, tid);
  sb.store(smem + TileA::elems, tid);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const bf16_t* cur_a = smem + (kt & 1) * kStage;
    const bf16_t* cur_b = cur_a + TileA::elems;
    if (kt + 1 < nk) {
      sa.load(p.A, p.lda, m0, (kt + 1) * BK, p.M, p.K, tid);
      sb.load(p.B, p.ldb, n0, (kt + 1) * BK, p.N, p.K, tid);
    }
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      bf16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = read_frag<BM, BK, A_KMAJ>(cur_a, wm0 + 32 * i, ks, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = read_frag<BN, BK, B_KMAJ>(cur_b, wn0 + 32 * j, ks, lane);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      bf16_t* nxt = smem + ((kt + 1) & 1) * kStage;
      sa.store(nxt, tid);
      sb.store(nxt + TileA::elems, tid);
    }
    __syncthreads();
  }

  epilogue<TM, TN, EPI>(p, acc, m0 + wm0, n0 + wn0, lane);
#endif
}

template <int BM, int BN, int BK, int WM, int WN, bool A_KMAJ, bool B_KMAJ, int EPI>
int launch(hipStream_t st, GemmParams p) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  constexpr size_t lds = 2 * sizeof(bf16_t) * (Tile<BM, BK, A_KMAJ>::elems + Tile<BN, BK, B_KMAJ>::elems);
  static_assert(lds <= 160 * 1024, "tile does not fit the 160 KB LDS");
  auto kern = gemm_bf16_kernel<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, EPI>;
  static std::atomic<bool> configured{false};  // per instantiation
  if (int rc = reserve_lds(kern, lds, configured, "gemm_bf16")) return rc;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  p.group_m = 8;
  kern<<<dim3(p.tiles_m * p.tiles_n), dim3(NT), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

template <int BM, int BN, int BK, int WM, int WN, bool A_KMAJ, bool B_KMAJ>
int launch_epi(hipStream_t st, const GemmParams& p, int epi) {
  switch (epi) {
    case PMC_EPI_NONE: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_NONE>(st, p);
    case PMC_EPI_BIAS: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_BIAS>(st, p);
    case PMC_EPI_BIAS_RESID: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_BIAS_RESID>(st, p);
    case PMC_EPI_BIAS_GELU: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_BIAS_GELU>(st, p);
    case PMC_EPI_DGELU: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_DGELU>(st, p);
    case PMC_EPI_ACCUM_F32: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_ACCUM_F32>(st, p);
    case PMC_EPI_BIAS_GELU_GRAD: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_BIAS_GELU_GRAD>(st, p);
    case PMC_EPI_MUL: return launch<BM, BN, BK, WM, WN, A_KMAJ, B_KMAJ, PMC_EPI_MUL>(st, p);
  }
  return fail(PMC_ERR_INVALID, "gemm_bf16: unknown epilogue %d", epi);
}

template <bool A_KMAJ, bool B_KMAJ>
int launch_tile(hipStream_t st, const GemmParams& p, int epi) {
  return launch_epi<128, 128, 64, 64, 64, A_KMAJ, B_KMAJ>(st, p, epi);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KMAJ, bool B_KMAJ, int NSTAGE, int EPI, bool SEG = false, int BK = 64,
          bool CUT = false, bool KSPLIT = false, int KG = 1>
int launch_dma(hipStream_t st, GemmParams p) {
  if constexpr ((A_KMAJ || B_KMAJ) && !CUT && KG == 1)
    if (p.K & 63) return launch_dma<BM, BN, WAVES_M, WAVES_N, A_KMAJ, B_KMAJ, NSTAGE, EPI, SEG, BK, true, KSPLIT, KG>(st, p);
  constexpr int NT = WAVES_M * WAVES_N * KG * 64;
  constexpr size_t lds = (size_t)NSTAGE * (BM + BN) * BK * sizeof(bf16_t);
  static_assert(lds <= 160 * 1024, "stages do not fit the 160 KB LDS");
  auto kern = gemm_bf16_dma_kernel<BM, BN, WAVES_M, WAVES_N, A_KMAJ, B_KMAJ, NSTAGE, EPI, SEG, BK, CUT, KSPLIT, KG>;
  static std::atomic<bool> configured{false};  // per instantiation
  if (int rc = reserve_lds(kern, lds, configured, "gemm_bf16")) return rc;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  {
    const int forced = tuning(kTuneGemmGroup);
    p.group_m = forced > 0 ? forced : (BM >= 256 ? 4 : 8);
  }
  const int tiles = p.tiles_m * p.tiles_n;
  p.own_xcds = EPI == kEpiPartial && gemm_bf16_split_own_xcds(B_KMAJ, p.tiles_m, p.M, p.N, p.K, p.splits);
  kern<<<dim3(p.own_xcds ? 8 * tiles_per_xcd(tiles, p.splits) : EPI == kEpiPartial ? tiles * p.splits : tiles), dim3(NT), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

// Layout of a product, by what its operands' contraction index is in memory; index into the times below.
enum Layout { kLayoutF = 0, kLayoutB = 1, kLayoutW = 2 };
constexpr Layout layout_of(bool a_kmaj, bool b_kmaj) { return !a_kmaj ? kLayoutW : b_kmaj ? kLayoutB : kLayoutF; }

// Tile shapes of the fast path.
//   0: 256x256, 8 waves, 2 stages    1: 256x128, 8 waves, 3 stages
//   2: 128x128, 4 waves: 4 stages as long as a compute unit gets one tile at most, otherwise 2 stages, so that
//      two workgroups fit a unit.  With one workgroup per unit nothing else covers the latency of a tile's
//      loads: 4096 x 1024 x 4096, F / B / W layout, 2 stages 52.1 / 47.2 / 52.8 us, 4 stages 39.8 / 36.4 / 43.0.  In the F and
//      B layouts such a workgroup has eight waves in two groups that share the K of every tile where gemm_bf16_k_groups says so
//   3: 64x128, 4 waves, 3 stages (skinny outputs; only where A is contraction-contiguous)
//   4: 256x320, 8 waves, 2 stages (not with the fp32 read-modify-write epilogue: registers)
//   5: 64x64, 5 stages   6: 32x64, 6 stages   7: 32x32, 8 stages; 4 waves that split K (see dma_tile)
//   8: 64x128, 6 stages, K split likewise, in the B layout: at long K the reads from LDS, 6 KB per 16 of K instead of
//      shape 3's 12, are what counts (1024 x 2048 x 8192 41.1 us against 44.0, x 2048 14.1 against 13.6; in the F
//      layout 43.2 against 43.8 alone and 68 against 69 inside a step, not worth a kernel)
// The gemm_tile tuning switch (0..4) forces a shape (for tests and tuning).
constexpr int kShapes = 9;
constexpr int kBm[kShapes] = {256, 256, 128, 64, 256, 64, 32, 32, 64}, kBn[kShapes] = {256, 128, 128, 128, 320, 64, 64, 32, 128};

long tiles_of(int shape, int M, int N) {
  return (long)((M + kBm[shape] - 1) / kBm[shape]) * ((N + kBn[shape] - 1) / kBn[shape]);
}

// Time of a product in us: fixed + rounds of tiles over the 256 compute units x (per_k for every 1024 of K +
// per_round); 1e9 where a layout has no such shape.  Fitted to every shape's time at the products of layers of hidden
// 64 .. 7168 with 16 .. 4096 tokens (308 products) with operands and C mostly in the memory-side cache; from HBM a time
// is 1.0 to 1.4 times the fitted one on average, 3 times at most (a 256x256 tile of a short W product, whose C is
// read and written once per few K tiles).  What the table is for is the order of the shapes, and that holds there too:
// with operands and C from HBM the shape picked is 1.2 / 0.6 / 2.7 % slower than the best one (F / B / W, 130 products).
double shape_us(Layout layout, int shape, long tiles, double K) {
  struct T { double fixed, per_k, per_round; };
  static constexpr T kTimes[3][kShapes] = {
      {{0., 19.5, 6.1}, {0., 11.4, 4.9}, {0., 8.1, 4.8}, {2.5, 4.9, 1.1}, {0., 23.1, 8.2}, {2.75, 3.1, 0.93}, {2.5, 2.2, 0.78}, {2.5, 1.8, 0.64}, {1e9, 0., 0.}},
      {{0., 18.3, 4.7}, {0., 10.6, 3.7}, {0., 7.5, 3.7}, {2.5, 5.0, 0.5}, {0., 21.5, 5.9}, {2.2, 2.8, 1.05}, {2.3, 2.0, 0.74}, {2.3, 1.3, 0.68}, {0.3, 4.7, 4.0}},
      {{0., 21.0, 8.6}, {0., 13.0, 6.6}, {0., 8.3, 5.9}, {1e9, 0., 0.}, {0., 23.1, 8.2}, {1.8, 2.7, 2.2}, {2.1, 2.3, 1.2}, {2.2, 2.1, 0.96}, {1e9, 0., 0.}}};
  static constexpr T kShallow[3] = {{4.5, 9.4, 0.}, {3.3, 9.2, 0.}, {0., 9.6, 5.3}};  // shape 2, two workgroups per unit
  const T& t = shape == 2 && tiles > 256 ? kShallow[layout] : kTimes[layout][shape];
  return t.fixed + (double)((tiles + 255) / 256) * (t.per_k * K / 1024. + t.per_round);
}

int pick_tile(Layout layout, int M, int N, long K, bool wide_ok, double* us = nullptr) {
  if (const int f = tuning(kTuneGemmTile); f >= 0) return (f == 4 && !wide_ok) ? 0 : f;
  int best = 0;
  double best_us = 1e300;
  for (int c = 0; c < kShapes; ++c) {
    if (c == 4 && !wide_ok) continue;
    const double t = shape_us(layout, c, tiles_of(c, M, N), (double)K);
    if (t < best_us) {
      best_us = t;
      best = c;
    }
  }
  if (us) *us = best_us;
  return best;
}

// the 320-wide tile holds 10 accumulator tiles per wave; with the fp32 read-modify-write epilogue on
// top it would spill registers, so weight-gradient products do not use it
constexpr bool wide_ok(int epi) { return epi != PMC_EPI_ACCUM_F32; }

}  // namespace

// 128x128 tiles of the F and B layouts, one at most to a compute unit: eight waves in two K groups (see dma_tile) or four.  Time of eight
// over that of four, over 6982 such products of layers of hidden 64 .. 8192 with 16 .. 8192 tokens, operands in the memory-side cache / from HBM
// (geometric means of F, B): here 0.89, 0.88 / 1.00, 1.00, nowhere more than 1.02 in the mean of the two.  Where the last K tile is partial 1.01, 1.03 / 1.04, 1.09
// (four / eight waves: 400 x 4952 x 14856 in B 157 / 179 us); whole K below 1024 1.03, 1.01 / 1.07, 1.06, as adding the groups up takes longer than what they cover; one row
// of tiles, or operands beyond the 256 MB of that cache, 0.98, 0.98 / 1.02, 1.00 and up to 1.10, as they come at the rate of HBM either way (128 x 31744 x 7936 in F 97 / 106 us).
bool gemm_bf16_k_groups(int M, int N, int K) {
  return tiles_of(2, M, N) <= 256 && K % 64 == 0 && K >= 1024 && M > 128 && ((size_t)M + N) * K * sizeof(bf16_t) <= 256u << 20;
}

namespace {
template <bool A_KMAJ, bool B_KMAJ, int EPI, bool SEG = false>
int launch_dma_tile(hipStream_t st, const GemmParams& p, int shape) {
  switch (shape) {
    case 0:
      // both operands stored [k][rows] (weight gradients): four 32-deep stages instead of two 64-deep ones, see
      // launch_wgrad_persistent
      if constexpr (!A_KMAJ && !B_KMAJ) return launch_dma<256, 256, 2, 4, A_KMAJ, B_KMAJ, 4, EPI, SEG, 32>(st, p);
      else return launch_dma<256, 256, 2, 4, A_KMAJ, B_KMAJ, 2, EPI, SEG>(st, p);
    case 1: return launch_dma<256, 128, 4, 2, A_KMAJ, B_KMAJ, 3, EPI, SEG>(st, p);
    case 4:
      if constexpr (wide_ok(EPI)) return launch_dma<256, 320, 4, 2, A_KMAJ, B_KMAJ, 2, EPI, SEG>(st, p);
      else break;
    case 3:
      if constexpr (A_KMAJ) return launch_dma<64, 128, 1, 4, A_KMAJ, B_KMAJ, 3, EPI, SEG>(st, p);
      else break;
    case 5: return launch_dma<64, 64, 2, 2, A_KMAJ, B_KMAJ, 5, EPI, SEG, 64, false, true>(st, p);
    case 6: return launch_dma<32, 64, 2, 2, A_KMAJ, B_KMAJ, 6, EPI, SEG, 64, false, true>(st, p);
    case 7: return launch_dma<32, 32, 2, 2, A_KMAJ, B_KMAJ, 8, EPI, SEG, 64, false, true>(st, p);
    case 8:
      if constexpr (A_KMAJ && B_KMAJ) return launch_dma<64, 128, 2, 2, A_KMAJ, B_KMAJ, 6, EPI, SEG, 64, false, true>(st, p);
      else break;
    default: break;
  }
  if constexpr (A_KMAJ)
    if (gemm_bf16_k_groups(p.M, p.N, p.K)) return launch_dma<128, 128, 2, 2, A_KMAJ, B_KMAJ, 4, EPI, SEG, 64, false, false, 2>(st, p);
  if (tiles_of(2, p.M, p.N) <= 256) return launch_dma<128, 128, 2, 2, A_KMAJ, B_KMAJ, 4, EPI, SEG>(st, p);
  return launch_dma<128, 128, 2, 2, A_KMAJ, B_KMAJ, 2, EPI, SEG>(st, p);
}

// Compute units of the current device, asked once (0 if the query fails).
int compute_units() {
  static std::atomic<int> units{0};
  int u = units.load(std::memory_order_relaxed);
  if (u > 0) return u;
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  units.store(prop.multiProcessorCount, std::memory_order_relaxed);
  return prop.multiProcessorCount;
}

// Persistent, phase-shifted weight-gradient kernel: when every compute unit gets at least two
// 256x256 tiles.  The gemm_wgrad tuning switch (0|1) forces the choice (tests, tuning).
bool use_wgrad_persistent(int M, int N, long K) {
  if (K < 4 * 64) return false;
  if (const int f = tuning(kTuneGemmWgrad); f >= 0) return f == 1;
  if (tuning(kTuneGemmTile) >= 0) return false;
  return (long)((M + 255) / 256) * ((N + 255) / 256) >= 2 * 256;
}

template <bool SEG>
int launch_wgrad_persistent(hipStream_t st, GemmParams p) {
  // measured: 2 phases give the most (1: -6 % W-pass time, 2: -8 %, 4 and 8: -7 %).  The ring is four 32-deep
  // stages rather than two 64-deep ones: the same LDS, but a tile is requested three steps (1.5 times as
  // far) ahead of its use, which the weight gradient's operand panels, the least shared in L2 of all products,
  // need most; both operands are stored [k][rows], so a 32-deep tile still reads whole rows.  Measured on
  // whole steps: W pass -3 % at 4096 tokens, -5 % at 2048.
  constexpr int NSTAGE = 4, GROUPS = 2, BK = 32;
  constexpr size_t lds = (size_t)NSTAGE * (256 + 256) * BK * sizeof(bf16_t);
  auto kern = gemm_bf16_wgrad_persistent_kernel<256, 256, 2, 4, NSTAGE, GROUPS, SEG, BK>;
  static std::atomic<bool> configured{false};
  if (int rc = reserve_lds(kern, lds, configured, "gemm_bf16")) return rc;
  const int units = compute_units();
  if (units <= 0) return fail(PMC_ERR_HIP, "gemm_bf16: cannot query the device");
  p.tiles_m = (p.M + 255) / 256;
  p.tiles_n = (p.N + 255) / 256;
  p.group_m = 8;
  const int ntiles = p.tiles_m * p.tiles_n;
  int grid = ntiles < units ? ntiles : units;
  if (grid >= 8) grid &= ~7;  // whole rounds over the 8 XCDs keep a workgroup's tiles on one XCD
  kern<<<dim3(grid), dim3(512), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 weight-gradient launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

// The two-workgroup kernel, for W products launched one by one (layers that share gradients, one stream or two forced), pays 1.5x the operand traffic of 256x256 tiles and a barrier every 16 matrix
// instructions; it wins where the K loop is short, so that a tile's ring fill and read-modify-write
// epilogue weigh as much as its K loop (measured on whole steps: -5 % of the W pass at 1024 tokens,
// +6 % at 2048, +26 % at 4096).  It does not win alone (2048 x 2048 at K = 1024 takes 27.4 us, 18.3 in 128x128
// tiles; 8192 x 2048 48.4 against 51.2) but beside its own kind on the second stream, so all four products of a layer
// take it or none.  What they share is the smaller side, hidden: steps of two layers at 512 / 1000 / 1024 tokens with it
// everywhere against nowhere, hidden 1024 +5 / +4 / +5 %, 1152 +1 / +3 / +3 %, 1280 0 / +2 / +2 %, 1408 -1 / -1 / -1 %,
// 1664 -2 / -2 / -2 %, 2560 -2 / -1 / -2 %; a bar on the tile count, which some of the products of hidden 1024 .. 1920
// passed, cost 1 to 3 %.  (An FFN narrower than hidden and up to 1280 keeps its two products out beside the others; steps
// of hidden / FFN 4096 / 1024, 2048 / 1024, 3072 / 1280 are within 0.4 % of the tile-count bar.)  gemm_wgrad = 2 forces it.
bool use_wgrad_pair(int M, int N, long K) {
  if (const int f = tuning(kTuneGemmWgrad); f >= 0) return f == 2;
  if (tuning(kTuneGemmTile) >= 0) return false;
  return K <= 1024 && std::min(M, N) > 1280;
}

template <bool SEG>
int launch_wgrad_pair(hipStream_t st, GemmParams p) {
  constexpr size_t lds = (size_t)3 * (256 + 128) * 32 * sizeof(bf16_t);
  auto kern = gemm_bf16_wgrad_pair_kernel<SEG>;
  static std::atomic<bool> configured{false};
  if (int rc = reserve_lds(kern, lds, configured, "gemm_bf16")) return rc;
  p.tiles_m = (p.M + 255) / 256;
  p.tiles_n = (p.N + 127) / 128;
  {
    const int forced = tuning(kTuneGemmGroup);
    p.group_m = forced > 0 ? forced : 4;
  }
  kern<<<dim3(p.tiles_m * p.tiles_n), dim3(256), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 weight-gradient launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

// Split K: when the output has too few tiles for the compute units and K is long, K is cut into ranges, each
// range writes an fp32 partial product to the workspace and a second kernel adds them and applies the epilogue.
// The partial products run in 64x64 tiles or in large ones: 128x128 (2 stages, two workgroups per unit) or, in the F and B layouts,
// 256x128, whichever split_us says is faster.  From HBM, 128x128 as they were before a range had XCDs of its own / since / 256x128:
// 1024 x 2048 x 8192 (F) in 4 ranges 62 / 53 / 48 us, 512 x 4096 x 16384 (F) 94 / 92 / 78; 200 x 5120 x 20480 (F) in 8 ranges
// 104 / 102 / 95, in 4 of 256x128 tiles 81.
struct SplitPlan {
  int splits, tiles_per_split, shape;  // splits = 1: no split
};

// The split with the least time, if it beats the product in one piece.  Partial sums and the second launch cost
// 4.5 us and 1.6 us per million partial sums (9.1 us with the larger tiles).
//  * Where the product in one piece fills the units (256-row tiles, or more than one round of 128x128 ones) a split
//    does not pay, whatever the fitted times say: W 3912 x 4104 x 16168 584 us in one piece, 655 in two ranges, F
//    2176 x 2560 x 10240 140 / 175, W 1408 x 5632 x 13440 224 / 248.
//  * The fitted times are those of operands in the caches.  From HBM, few workgroups with a long K loop take 1.3 to 1.5
//    times as long (shapes 3 and 5 .. 8), 128x128 tiles 1.1 to 1.25 times, partial products, whose ranges load side by
//    side, about what the fit says.  Inside a step an operand comes from HBM where it is large against the 256 MB
//    memory-side cache (its layer has ten times these bytes with the other weights and the gradients): from 32 MB on the
//    small shapes give way to a split of up to 1.25 times their fitted time.  Below that the operands may be cached, where
//    a split has to be clearly better.  Time in the split picked / in one piece over 422 products of layers, K from 1024:
//    32 MB and more, from HBM: F 0.90, B 0.93, W 0.59, worst 1.10 (40 x 16680 x 5560: 54 -> 60 us); smaller ones,
//    cached: 0.98, 1.00, 0.90, worst 1.07.  From HBM, one piece / split: F 56 x 4000 x 16000 49.1 / 31.6 us,
//    W 96 x 288 x 12376 50.3 / 16.9; inside a step F 1024 x 2048 x 8192 69 / 64, F 512 x 4096 x 16384 121 / 94.
double split_us(int shape, int M, int N, int ranges, int k_tiles) {
  const long tiles = tiles_of(shape, M, N) * ranges;
  const double sums = 1.6e-6 * (double)M * N * ranges, rounds = (double)((tiles + 255) / 256);
  if (shape == 1) return 9.1 + rounds * (15. * k_tiles / 16. - 4.5) + sums;
  return 9.1 + (tiles <= 256 ? 14. : 7.6 * rounds) * k_tiles / 16. + sums;
}
SplitPlan pick_splits(Layout layout, int M, int N, int K, int epi, size_t ws_bytes) {
  SplitPlan best = {1, 0, 0};
  if (tuning(kTuneGemmTile) >= 0 || K < 2048) return best;
  if (ws_bytes != (size_t)-1) {  // the plan of unlimited scratch, if it fits
    best = pick_splits(layout, M, N, K, epi, (size_t)-1);
    if (best.splits == 1 || (size_t)best.splits * M * N * sizeof(float) <= ws_bytes) return best;
    best = {1, 0, 0};
  }
  double limit;
  const int whole = pick_tile(layout, M, N, K, wide_ok(epi), &limit);
  const bool small = whole == 3 || whole >= 5;
  if (!small && (whole != 2 || tiles_of(2, M, N) > 256)) return best;
  limit *= small && (double)std::max(M, N) * K * sizeof(bf16_t) >= 32e6 ? 1.25 : 0.85;
  const int nkt = (K + 63) / 64;
  for (int shape : {2, 5})
    for (int s : {2, 4, 8}) {
      const int per = (nkt + s - 1) / s, n = (nkt + per - 1) / per;
      if (per < 4 || (size_t)n * M * N * sizeof(float) > ws_bytes) continue;
      const double us = shape == 2 ? split_us(2, M, N, n, per)
                                   : 4.5 + shape_us(layout, 5, tiles_of(5, M, N) * n, per * 64.) + 1.6e-6 * (double)M * N * n;
      if (us < limit) {
        limit = us;
        best = {n, per, shape};
      }
    }
  // the number of ranges that suits 256x128 tiles
  if (best.splits > 1 && best.shape == 2 && layout != kLayoutW)
    for (int s : {2, 4, 8}) {
      const int per = (nkt + s - 1) / s, n = (nkt + per - 1) / per;
      if (per < 4 || (size_t)n * M * N * sizeof(float) > ws_bytes) continue;
      if (const double us = split_us(1, M, N, n, per); us < limit) {
        limit = us;
        best = {n, per, 2};
      }
    }
  return best;
}

template <bool A_KMAJ, bool B_KMAJ>
int launch_partial(hipStream_t st, GemmParams p, void* ws, const GemmPlan& plan) {
  p.C = ws;
  p.splits = plan.splits;
  p.k_tiles_per_split = plan.k_tiles_per_split;
  if (plan.kernel == kPlanSplit + 5) return launch_dma<64, 64, 2, 2, A_KMAJ, B_KMAJ, 5, kEpiPartial, false, 64, false, true>(st, p);
  if constexpr (A_KMAJ)
    if (split_us(1, p.M, p.N, plan.splits, plan.k_tiles_per_split) < split_us(2, p.M, p.N, plan.splits, plan.k_tiles_per_split))
      return launch_dma<256, 128, 4, 2, A_KMAJ, B_KMAJ, 3, kEpiPartial>(st, p);
  return launch_dma<128, 128, 2, 2, A_KMAJ, B_KMAJ, 2, kEpiPartial>(st, p);
}

template <int EPI>
int launch_reduce_epi(hipStream_t st, const GemmParams& p, const float* ws, int splits) {
  const size_t quads = (size_t)p.M * p.N / 4;
  splitk_reduce_kernel<EPI><<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st>>>(p, ws, splits);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 split-K reduce launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

int launch_reduce(hipStream_t st, const GemmParams& p, const float* ws, int splits, int epi) {
  switch (epi) {
    case PMC_EPI_NONE: return launch_reduce_epi<PMC_EPI_NONE>(st, p, ws, splits);
    case PMC_EPI_BIAS: return launch_reduce_epi<PMC_EPI_BIAS>(st, p, ws, splits);
    case PMC_EPI_BIAS_RESID: return launch_reduce_epi<PMC_EPI_BIAS_RESID>(st, p, ws, splits);
    case PMC_EPI_BIAS_GELU: return launch_reduce_epi<PMC_EPI_BIAS_GELU>(st, p, ws, splits);
    case PMC_EPI_DGELU: return launch_reduce_epi<PMC_EPI_DGELU>(st, p, ws, splits);
    case PMC_EPI_ACCUM_F32: return launch_reduce_epi<PMC_EPI_ACCUM_F32>(st, p, ws, splits);
    case PMC_EPI_BIAS_GELU_GRAD: return launch_reduce_epi<PMC_EPI_BIAS_GELU_GRAD>(st, p, ws, splits);
    case PMC_EPI_MUL: return launch_reduce_epi<PMC_EPI_MUL>(st, p, ws, splits);
  }
  return fail(PMC_ERR_INVALID, "gemm_bf16: unknown epilogue %d", epi);
}

// The layout/epilogue combinations the passes use (and the plain product of each layout) have a
// fast-path instantiation.
bool has_fast_path(bool a_kmaj, bool b_kmaj, int epi) {
  if (a_kmaj && !b_kmaj)
    return epi == PMC_EPI_NONE || epi == PMC_EPI_BIAS || epi == PMC_EPI_BIAS_RESID || epi == PMC_EPI_BIAS_GELU || epi == PMC_EPI_BIAS_GELU_GRAD;
  if (a_kmaj && b_kmaj) return epi == PMC_EPI_NONE || epi == PMC_EPI_DGELU || epi == PMC_EPI_MUL;
  return !a_kmaj && !b_kmaj && (epi == PMC_EPI_NONE || epi == PMC_EPI_ACCUM_F32);
}

int launch_fast(hipStream_t st, const GemmParams& p, bool a_kmaj, bool b_kmaj, int epi, int shape) {
  if (a_kmaj && !b_kmaj) {  // F: Y = X . W
    switch (epi) {
      case PMC_EPI_NONE: return launch_dma_tile<true, false, PMC_EPI_NONE>(st, p, shape);
      case PMC_EPI_BIAS: return launch_dma_tile<true, false, PMC_EPI_BIAS>(st, p, shape);
      case PMC_EPI_BIAS_RESID: return launch_dma_tile<true, false, PMC_EPI_BIAS_RESID>(st, p, shape);
      case PMC_EPI_BIAS_GELU: return launch_dma_tile<true, false, PMC_EPI_BIAS_GELU>(st, p, shape);
      case PMC_EPI_BIAS_GELU_GRAD: return launch_dma_tile<true, false, PMC_EPI_BIAS_GELU_GRAD>(st, p, shape);
    }
  } else if (a_kmaj && b_kmaj) {  // B: dX = dY . W^T
    switch (epi) {
      case PMC_EPI_NONE: return launch_dma_tile<true, true, PMC_EPI_NONE>(st, p, shape);
      case PMC_EPI_DGELU: return launch_dma_tile<true, true, PMC_EPI_DGELU>(st, p, shape);
      case PMC_EPI_MUL: return launch_dma_tile<true, true, PMC_EPI_MUL>(st, p, shape);
    }
  } else if (!a_kmaj && !b_kmaj) {  // W: dW += X^T . dY
    switch (epi) {
      case PMC_EPI_NONE: return launch_dma_tile<false, false, PMC_EPI_NONE>(st, p, shape);
      case PMC_EPI_ACCUM_F32: return launch_dma_tile<false, false, PMC_EPI_ACCUM_F32>(st, p, shape);
    }
  }
  return fail(PMC_ERR_INVALID, "gemm_bf16: no direct-to-LDS kernel for epilogue %d in this layout", epi);
}

// Kernel of an fp32 read-modify-write product of stored-[k][rows] operands (K: all pieces).
int wgrad_kernel(int M, int N, long K) {
  if (use_wgrad_pair(M, N, K)) return kPlanPair;
  if (use_wgrad_persistent(M, N, K)) return kPlanPersistent;
  return kPlanTile + pick_tile(kLayoutW, M, N, K, false);
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

}  // namespace

// Fast path: operands inside the 2 GB window of a buffer descriptor.  A K that is no multiple of 64 only
// costs it a partly empty last tile.  (Two layers of hidden 2048: 1208 us a step at 1024 tokens; at 1000
// tokens 1379 us with the weight gradients on the general kernel, 1237 us here.)
GemmPlan gemm_bf16_plan(const GemmArgs& a) {
  const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
  const size_t a_bytes = (size_t)(a.trans_a ? a.K : a.M) * a.lda * 2, b_bytes = (size_t)(a.trans_b ? a.N : a.K) * a.ldb * 2;
  const GemmPlan general = {kPlanGeneral, 1, 0};
  if ((!a_kmaj && b_kmaj) || a_bytes >= 0x7fffffffull || b_bytes >= 0x7fffffffull) return general;
  const Layout layout = layout_of(a_kmaj, b_kmaj);
  if (a.ws) {
    const SplitPlan split = pick_splits(layout, a.M, a.N, a.K, a.epilogue, a.ws_bytes);
    if (split.splits > 1) return {kPlanSplit + split.shape, split.splits, split.tiles_per_split};
  }
  if (!has_fast_path(a_kmaj, b_kmaj, a.epilogue)) return general;
  if (a.epilogue == PMC_EPI_ACCUM_F32) return {wgrad_kernel(a.M, a.N, a.K), 1, 0};
  return {kPlanTile + pick_tile(layout, a.M, a.N, a.K, true), 1, 0};
}

int gemm_bf16(hipStream_t st, const GemmArgs& a) {
  if (a.M % 8 || a.N % 8 || a.K % 8) return fail(PMC_ERR_INVALID, "gemm_bf16: M=%d N=%d K=%d must be multiples of 8", a.M, a.N, a.K);
  if (a.lda % 8 || a.ldb % 8 || a.ldc % 4) return fail(PMC_ERR_INVALID, "gemm_bf16: pitches must be multiples of 8 (lda=%d ldb=%d ldc=%d)", a.lda, a.ldb, a.ldc);
  if (!aligned(a.A, 16) || !aligned(a.B, 16) || !aligned(a.C, 16) || (a.bias && !aligned(a.bias, 8)) ||
      (a.resid && !aligned(a.resid, 8)) || (a.aux && !aligned(a.aux, 8)))
    return fail(PMC_ERR_INVALID, "gemm_bf16: operands must be 16-byte aligned");
  GemmParams p;
  p.A = (const bf16_t*)a.A; p.B = (const bf16_t*)a.B; p.C = a.C;
  p.bias = (const bf16_t*)a.bias; p.resid = (const bf16_t*)a.resid; p.aux = (bf16_t*)a.aux;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.ldc = a.ldc;
  p.tiles_m = p.tiles_n = 0;
  p.group_m = 8;
  p.splits = 1;
  p.k_tiles_per_split = k_tiles<false, 64>(p);
  p.nseg = p.seg_k = 0;
  for (int i = 0; i < kMaxSegments; ++i) p.Aseg[i] = p.Bseg[i] = nullptr;
  const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
  const GemmPlan plan = gemm_bf16_plan(a);
  if (plan.splits > 1) {
    int rc = a_kmaj ? (b_kmaj ? launch_partial<true, true>(st, p, a.ws, plan) : launch_partial<true, false>(st, p, a.ws, plan))
                    : launch_partial<false, false>(st, p, a.ws, plan);
    if (rc != PMC_OK) return rc;
    return launch_reduce(st, p, (const float*)a.ws, plan.splits, a.epilogue);
  }
  if (plan.kernel == kPlanPair) return launch_wgrad_pair<false>(st, p);
  if (plan.kernel == kPlanPersistent) return launch_wgrad_persistent<false>(st, p);
  if (plan.kernel != kPlanGeneral) return launch_fast(st, p, a_kmaj, b_kmaj, a.epilogue, plan.kernel - kPlanTile);
  if (a_kmaj && b_kmaj) return launch_tile<true, true>(st, p, a.epilogue);
  if (a_kmaj && !b_kmaj) return launch_tile<true, false>(st, p, a.epilogue);
  if (!a_kmaj && b_kmaj) return launch_tile<false, true>(st, p, a.epilogue);
  return launch_tile<false, false>(st, p, a.epilogue);
}

// C[M,N] (fp32) += sum over pieces i of A_i^T . B_i, A_i stored [K,M], B_i stored [K,N]: one product
// whose contraction runs through the pieces one after the other, one read-modify-write of C.
int gemm_bf16_grouped_wgrad(hipStream_t st, const GroupedWgradArgs& a) {
  if (a.count < 1 || a.count > kMaxSegments) return fail(PMC_ERR_INVALID, "grouped weight gradient: %d pieces (1..%d)", a.count, kMaxSegments);
  if (a.M % 8 || a.N % 8 || a.K % 8) return fail(PMC_ERR_INVALID, "grouped weight gradient: M=%d N=%d K=%d must be multiples of 8", a.M, a.N, a.K);
  if (a.lda % 8 || a.ldb % 8 || a.ldc % 4 || a.lda < a.M || a.ldb < a.N || a.ldc < a.N)
    return fail(PMC_ERR_INVALID, "grouped weight gradient: bad pitches (lda=%d ldb=%d ldc=%d)", a.lda, a.ldb, a.ldc);
  if ((size_t)a.K * a.lda * 2 >= 0x7fffffffull || (size_t)a.K * a.ldb * 2 >= 0x7fffffffull)
    return fail(PMC_ERR_INVALID, "grouped weight gradient: a piece exceeds the 2 GB window of a buffer descriptor");
  if (!aligned(a.C, 16)) return fail(PMC_ERR_INVALID, "grouped weight gradient: C must be 16-byte aligned");
  GemmParams p;
  p.A = (const bf16_t*)a.A[0]; p.B = (const bf16_t*)a.B[0]; p.C = a.C;
  p.bias = p.resid = nullptr; p.aux = nullptr;
  p.M = a.M; p.N = a.N; p.K = a.K * a.count; p.lda = a.lda; p.ldb = a.ldb; p.ldc = a.ldc;
  p.tiles_m = p.tiles_n = 0;
  p.group_m = 8;
  p.nseg = a.count;
  p.seg_k = a.K;
  p.splits = 1;
  p.k_tiles_per_split = k_tiles<true, 64>(p);
  for (int i = 0; i < kMaxSegments; ++i) {
    const int j = i < a.count ? i : a.count - 1;
    if (!a.A[j] || !a.B[j] || !aligned(a.A[j], 16) || !aligned(a.B[j], 16))
      return fail(PMC_ERR_INVALID, "grouped weight gradient: piece %d is NULL or not 16-byte aligned", j);
    p.Aseg[i] = (const bf16_t*)a.A[j];
    p.Bseg[i] = (const bf16_t*)a.B[j];
  }
  const int kernel = wgrad_kernel(p.M, p.N, p.K);
  if (kernel == kPlanPair) return launch_wgrad_pair<true>(st, p);
  if (kernel == kPlanPersistent) return launch_wgrad_persistent<true>(st, p);
  return launch_dma_tile<false, false, PMC_EPI_ACCUM_F32, true>(st, p, kernel - kPlanTile);
}

namespace {
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, int BK, bool KSPLIT, int WPS>
int launch_wgrad_batch(hipStream_t st, WgradBatchParams& p) {
  constexpr size_t lds = (size_t)NSTAGE * (BM + BN) * BK * sizeof(bf16_t);
  auto kern = gemm_bf16_wgrad_batch_kernel<BM, BN, WAVES_M, WAVES_N, NSTAGE, BK, KSPLIT, WPS>;
  static std::atomic<bool> configured{false};
  if (int rc = reserve_lds(kern, lds, configured, "gemm_bf16")) return rc;
  wgrad_batch_layout(p, BM, BN, WAVES_M * WAVES_N * 64);
  kern<<<dim3(p.sum_blocks + p.first_tile[4] * p.w.layers), dim3(WAVES_M * WAVES_N * 64), lds, st>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "gemm_bf16 weight-gradient launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}
}  // namespace

// Tiles of the one launch; picked by fitted times (see batch_us in wgrad_batch.h) of 4030 W passes, hidden 64 .. 8192, 16 .. 65536 tokens
// in 1 .. 8 pieces, 1 .. 4 layers, FFN 1 .. 4.5 x hidden: the shape picked is 1.1 % slower than the best one on average (1.31 times at
// worst, at a few microseconds; 0.8 % beyond 2048 tokens and 0.2 % beyond 8192), and 1.86 times as fast as the products launched one by one on two streams (geometric mean).
// Some of them, us one by one / in one launch: 2 layers of hidden 256, 192 tokens 52 / 9; 2 of 1024, 4096 tokens 333 / 226; 2 of 2048, 1024 tokens
// 321 / 290; 2 of 4096, 1024 tokens 1140 / 1015; 2 of 5120, 4096 tokens 4584 / 4577; 1 of 2304 x 2776, 8 x 5488 tokens 3104 / 3087 (4178 in tiles of shape 1).
//   0: 256x256, four 32-deep stages   1: 256x128, two workgroups per compute unit   2: 128x128, likewise
//   3: 64x128   4: 64x64   5: 32x32 whose waves split K (few outputs over many tokens)
enum BatchShape { kBatch256, kBatchPair, kBatch128, kBatch64x128, kBatch64, kBatch32, kBatchShapes };

// The shape, or -1 where the products go out one by one: where each of them fills whole rounds of 256x256 tiles over the compute units, to 98 %, a launch
// of its own leaves nothing idle, and from 2048 tokens on the persistent kernel beside a second stream is as fast.  Time of one launch over that of
// two streams: 11 such passes of 2104 .. 6360 tokens 0.97 .. 1.04, 1.00 on average (2 layers of 4096, 2048 tokens 1683 and 1663 us); fewer tokens 0.94; rounds filled to 0.90 .. 0.98
// 0.98 (0.86 .. 1.03), to 0.80 .. 0.90 0.96 (0.86 .. 1.03), less 0.88 (0.64 .. 1.09: 2 layers of 2048 x 6416, 6464 tokens 1102 and 1014 us, whose last round is a quarter full).
int gemm_bf16_wgrad_batch_shape(const WgradBatchArgs& a) {
  constexpr int kBm[kBatchShapes] = {256, 256, 128, 64, 64, 32}, kBn[kBatchShapes] = {256, 128, 128, 128, 64, 32};
  static constexpr BatchTime kTimes[kBatchShapes] = {
      {11.06, 0.86, 8.73, 26.8, 13.6, 0., 1, 0.},     {6.78, 1.87, 6.93, 11.4, 9.66, 3.07, 2, 1.14},  {6.48, 1.41, 4.35, 5.60, 5.97, 1.18, 2, 1.58},
      {4.52, 2.57, 3.42, 2.40, 3.47, 2.20, 3, 0.69}, {4.51, 2.71, 2.70, 1.15, 1.19, 1.82, 4, 0.48}, {5.33, 1.57, 1.75, 0.65, 0.74, 1.01, 2, 0.}};
  const double K = (double)a.K * a.pieces;
  double filled = 0., rounds = 0.;
  for (int j = 0; j < 4; ++j) {
    const long tiles = (long)((a.M[j] + 255) / 256) * ((a.N[j] + 255) / 256);
    filled += (double)tiles;
    rounds += (double)((tiles + 255) / 256);
  }
  if (K >= 2048 && filled >= 0.98 * 256. * rounds) return -1;
  int best = -1;
  double best_us = 1e300;
  for (int s = 0; s < kBatchShapes; ++s) {
    const double us = batch_us(kTimes[s], (double)batch_tiles(a, kBm[s], kBn[s]) * a.layers, K);
    if (us < best_us) {
      best_us = us;
      best = s;
    }
  }
  return best;
}

int gemm_bf16_wgrad_batch(hipStream_t st, const WgradBatchArgs& a, int shape) {
  WgradBatchParams p;
  p.w = a;
  switch (shape) {
    case kBatch256: return launch_wgrad_batch<256, 256, 2, 4, 4, 32, false, 1>(st, p);
    case kBatchPair: return launch_wgrad_batch<256, 128, 2, 2, 3, 32, false, 2>(st, p);
    case kBatch128: return launch_wgrad_batch<128, 128, 2, 2, 4, 32, false, 2>(st, p);
    case kBatch64x128: return launch_wgrad_batch<64, 128, 2, 2, 4, 32, false, 3>(st, p);
    case kBatch64: return launch_wgrad_batch<64, 64, 2, 2, 4, 32, false, 3>(st, p);
    case kBatch32: return launch_wgrad_batch<32, 32, 2, 2, 8, 64, true, 1>(st, p);
  }
  return fail(PMC_ERR_INVALID, "gemm_bf16: no weight-gradient tiles %d", shape);
}

size_t gemm_scratch_bytes(GemmArgs a) {
  if (a.dtype != PMC_BF16) return 0;
  a.ws = &a;  // any non-NULL pointer: nothing is launched
  a.ws_bytes = (size_t)-1;
  const GemmPlan plan = gemm_bf16_plan(a);
  return plan.splits > 1 ? (size_t)plan.splits * a.M * a.N * sizeof(float) : 0;
}

}  // namespace k
}  // namespace pmc
