// Fused flash-style attention for bf16 storage on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16), packed qkv [batch*seq, 3h].  The tiles are 64 or 128 columns wide; a head
// size that is another multiple of 8 runs in the next wider tile with the remaining columns at zero.
//
// Forward: a workgroup owns a block of queries of one head and streams blocks of K and V through
// LDS (double buffered); its waves form a grid over (32-query group, key group).  Scores are
// produced transposed, S^T[key][query], so every lane owns ONE query column: the online-softmax
// max/sum over keys are in-lane reductions plus one exchange between the two half-waves, and the
// probabilities already sit in the register layout of the B operand of the second product
// O^T = V^T . P^T.  V^T is never formed in memory: the V tile stays [key][dh] in LDS and is read
// with the transposing LDS load.  Saves O and the log-sum-exp.
//
// Backward is two halves, one kernel each or both in one launch, each output element having one writer and a fixed
// summation order (results are reproducible run to run):
//   dQ   per query block, streaming K/V blocks: recomputes P from the saved log-sum-exp,
//        dS = P * (dO.V^T - delta), dQ^T += K^T . dS^T; also emits delta = rowsum(dO * O).
//   dKdV per key block, streaming Q/dO blocks: dV^T += dO^T . P, dK^T += Q^T . dS.
// The launch shapes are chosen by the number of (row block, head) pairs: few pairs get small
// row blocks and more waves per block so that all compute units have work.
#include <cstdlib>
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"

namespace pmc {
namespace k {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSlack = 8.0f;  // forward: how far (in log2 units) a score may exceed the softmax reference

typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
typedef short s16x8 __attribute__((ext_vector_type(8)));

// LDS tiles are [rows][DH] bf16 without padding, filled by direct-to-LDS loads (one wave instruction
// writes 1 KB, lane l the bytes 16 l .. 16 l + 15 of it) and XOR-swizzled in 16-byte chunks: chunk c
// of row r sits at position c ^ swz(r).  swz is chosen so that both read patterns are free of bank
// conflicts: 16 consecutive rows at one chunk fall into 16 different 16-byte bank groups (operand
// fragments along the rows), and the four rows a transposing read touches fall into the four 64-byte
// quarters of the banks.
template <int DH>
__device__ __forceinline__ int swz(int row) {
  return DH == 128 ? (((row & 3) << 2) | ((row >> 2) & 3))           // 16 chunks per 256-byte row
                   : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));   // 8 chunks per 128-byte row, two rows per bank pass
}

// Fragment with the contraction index contiguous in the LDS row: lane l gets row row0 + l%32,
// contraction indices k0 + 8*(l/32) .. +7.
template <int DH>
__device__ __forceinline__ bf16x8 frag_rows(const bf16_t* tile, int row0, int k0, int lane) {
  const int row = row0 + (lane & 31), c = (k0 >> 3) + (lane >> 5);
  return *reinterpret_cast<const bf16x8*>(tile + row * DH + ((c ^ swz<DH>(row)) << 3));
}

// Fragment of the TRANSPOSE of an LDS tile: lane l gets tile column col0 + l%32 and, as its 8
// contraction entries, tile rows  krow0 + 4*(l/32) + {0,1,2,3}  and  krow0 + 8 + 4*(l/32) + {0,1,2,3}.
// That row order is exactly the one in which a lane holds a 32x32 accumulator tile's registers
// 8t .. 8t+7 (rows 8*(r/4) + 4*(l/32) + r%4), so accumulators can be fed back as the other operand.
template <int DH>
__device__ __forceinline__ bf16x8 frag_cols(const bf16_t* tile, int col0, int krow0, int lane) {
  const int g = lane >> 4, j = lane & 15;
  const int row = krow0 + 4 * (g >> 1) + (j >> 2), col = col0 + 16 * (g & 1) + 4 * (j & 3);
  const int c = col >> 3, within = col & 7;
  const bf16_t* p = tile + row * DH + ((c ^ swz<DH>(row)) << 3) + within;
  const bf16_t* q = tile + (row + 8) * DH + ((c ^ swz<DH>(row + 8)) << 3) + within;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q));
  const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// Registers 8t .. 8t+7 of an accumulator tile as a bf16 operand fragment.
__device__ __forceinline__ bf16x8 acc_to_frag(const f32x16& a, int t) {
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)a[8 * t + e];
  return v;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Raw buffer descriptor with a 2 GB window at ptr (every offset used stays below that: checked on the host).
__device__ __forceinline__ i32x4 make_rsrc(const void* ptr) {
  const uint64_t a = (uint64_t)ptr;
  i32x4 r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), 0x7fffffff, 0x00020000};
  return r;
}

// Cooperative direct-to-LDS copy of a [ROWS][DH] block of rows (row pitch ld elements in global
// memory) by the NT threads of the workgroup: the data never passes through registers.  Rows past
// the last one are clamped to it, so every access stays inside the tensor; what those rows
// contribute is masked by the caller.  The loads are inline assembly: the caller waits for them
// with s_waitcnt vmcnt(0) before the barrier that publishes the tile.
template <int ROWS, int DH, int NT>
struct BlockDma {
  static constexpr int CPR = DH / 8;                 // chunks per row
  static constexpr int RPI = 64 / CPR;               // rows per wave instruction
  static constexpr int NI = ROWS / RPI;              // wave instructions per block
  static constexpr int NW = NT / 64;
  static constexpr int PER = (NI + NW - 1) / NW;     // per wave (the last waves idle if NI % NW)
  static_assert(ROWS % RPI == 0, "block must be whole wave instructions");
  static constexpr uint32_t kSkip = 0xffffffffu;
  int row_in_block[PER];
  uint32_t col_bytes[PER];
  // dh: columns a row really has (a multiple of 8, at most DH).  Lanes whose chunk lies past them
  // load nothing; their LDS positions keep the zeros the kernel wrote there once.
  __device__ __forceinline__ void init(int wave, int lane, int dh = DH) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int q = wave + i * NW, row = q * RPI + lane / CPR, pos = lane % CPR;
      const int chunk = pos ^ swz<DH>(row);
      row_in_block[i] = row;
      col_bytes[i] = 8 * chunk < dh ? (uint32_t)(chunk << 4) : kSkip;
    }
  }
  // row0: first row of the block; last_row: the last valid row; ld_bytes: row pitch in bytes
  template <bool PAD = false>
  __device__ __forceinline__ void issue(i32x4 rsrc, bf16_t* tile, uint32_t ld_bytes, int row0, int last_row, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int q = wave + i * NW;
      if (NI % NW != 0 && q >= NI) break;
      const uint32_t voff = (uint32_t)min(row0 + row_in_block[i], last_row) * ld_bytes + col_bytes[i];
      const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)((lds_void_ptr)(tile + q * 512)));
      if (!PAD || col_bytes[i] != kSkip)  // a lane writes its own 16 bytes of the instruction's 1 KB whoever else is active
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds_addr), "v"(voff), "s"(rsrc) : "memory");
    }
  }
};

constexpr int kWaitAllLoads = 0x0F70;  // s_waitcnt vmcnt(0)

__device__ __forceinline__ void zero(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}

// Writes an accumulator tile holding OUT^T[dh][row] (lane = row, registers = dh) times `mul` to
// out[row][col0 + 32*dt + ...] as bf16, four consecutive columns per store; only the first `cols`
// of the tile's 32 columns exist (a multiple of 4).
__device__ __forceinline__ void store_tile_t(bf16_t* row_ptr, const f32x16& a, float mul, int lane, int cols = 32) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    u32x2 v = {pack_bf16x2(a[4 * q] * mul, a[4 * q + 1] * mul), pack_bf16x2(a[4 * q + 2] * mul, a[4 * q + 3] * mul)};
    if (8 * q + 4 * (lane >> 5) < cols) *reinterpret_cast<u32x2*>(row_ptr + 8 * q + 4 * (lane >> 5)) = v;
  }
}

// Eight consecutive elements of a row from global memory, zeros if they lie past the row's dh columns.
__device__ __forceinline__ bf16x8 load_frag(const bf16_t* p, int col, int dh) {
  bf16x8 z;
#pragma unroll
  for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.f;
  return col < dh ? *reinterpret_cast<const bf16x8*>(p + col) : z;
}

// Head sizes below the tile width: the tiles' columns past dh are zeroed once (the loads skip them).
template <int NT>
__device__ __forceinline__ void zero_tiles(bf16_t* smem, int elems, int tid) {
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (int i = tid * 8; i < elems; i += NT * 8) *reinterpret_cast<u32x4*>(smem + i) = z;
  __syncthreads();
}

// Forward.  The workgroup is a QW x KW grid of waves: wave (qg, kg) owns queries 32 qg .. 32 qg + 31
// of the workgroup's 32 QW queries and, of every streamed block of 32 NKT KW keys, the 32 NKT keys
// starting at 32 NKT kg.
// Each wave runs its own online softmax over the keys it sees; at the end the KW partial results of
// a query group are merged in key-group order through LDS.  Splitting the keys over waves puts two
// waves on every SIMD even when there are few (query block, head) pairs, and shortens the serial
// chain of a long row of key blocks.
// PAD: the head size dh is smaller than the tile width DH (the columns past dh are kept at zero).
// OWN: each of the wave's first OWN 32-key tiles is summed against a reference of its own, the tile's maximum (what is summed so far is
// rescaled to it).  Probabilities are rounded to bf16, all but the reference's, which is 1, and of up to a few hundred keys the
// largest few are a good part of the sum of squares that the rounding error of o is made of.  Four key groups have four exact ones to
// a query from the start; with OWN = 4 / KW the shapes of fewer groups have the same four, and they move the reference sooner
// (SLACK), which keeps pace with four groups where scores are spread widely.  Error of o against 64 bits over that of four groups, one reference
// to a group / OWN: 8 x 128 tokens, 16 heads of 64, no mask, two groups 1.08 / 1.00 and one 1.10 / 1.00; over 80 sizes of
// up to 2048 tokens with q and k ~ N(0, 0.25), N(0, 1), N(0, 4) at worst 1.15 / 1.004, on average 1.03 / 1.00, 1.00, 0.97.  It costs two groups
// 0.5 % and one 2 % of the time: the first tiles run in a loop of their own, which leaves the other loop as it is.
template <int DH, int QW, int KW, int NKT, bool PAD, int OWN>
__global__ __launch_bounds__(QW * KW * 64, QW * KW == 4 ? 2 : 1) void attn_fwd_mfma(int seq, int heads, int dh, int causal, const bf16_t* __restrict__ qkv,
                                                               bf16_t* __restrict__ o, float* __restrict__ lse,
                                                               float scale_log2) {
  constexpr int NT = QW * KW * 64, BQW = 32 * QW, WK = 32 * NKT, BSW = WK * KW;
  constexpr int KT = BSW * DH, VT = BSW * DH;
  constexpr float SLACK = OWN > 0 ? 3.0f : kSlack;
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];  // [2][K tile | V tile]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hl = lane >> 5;
  const int qg = wave % QW, kg = wave / QW;
  // grid = (heads * batch, query blocks); under a causal mask late query blocks see the most keys,
  // so they are dealt out first and the short ones fill the tail
  const int h = heads * dh, head = blockIdx.x % heads, b = blockIdx.x / heads;
  const int q0 = (causal ? (int)(gridDim.y - 1 - blockIdx.y) : (int)blockIdx.y) * BQW, qw0 = q0 + 32 * qg, qrow = qw0 + (lane & 31);
  const size_t ld = (size_t)3 * h;
  const bf16_t* base = qkv + (size_t)b * seq * ld + (size_t)head * dh;

  bf16x8 qf[DH / 16];
  {
    const bf16_t* qp = base + (size_t)min(qrow, seq - 1) * ld;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) qf[ks] = load_frag(qp, 16 * ks + 8 * hl, PAD ? dh : DH);
  }
  f32x16 oacc[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) zero(oacc[dt]);
  float m2 = -INFINITY, lsum = 0.f;  // softmax reference (log2 units, scale applied; see below) and sum
  float top = -INFINITY;             // OWN: maximum of the tiles with a reference of their own

  const int kend = causal ? min(seq, q0 + BQW) : seq;
  const int nblk = (kend + BSW - 1) / BSW;
  const i32x4 rk = make_rsrc(base + h), rv = make_rsrc(base + 2 * h);
  const uint32_t ldb = (uint32_t)ld * 2;
  if (PAD) zero_tiles<NT>(smem, 2 * (KT + VT), tid);
  BlockDma<BSW, DH, NT> dma;
  dma.init(wave, lane, PAD ? dh : DH);
  dma.template issue<PAD>(rk, smem, ldb, 0, seq - 1, wave);
  dma.template issue<PAD>(rv, smem + KT, ldb, 0, seq - 1, wave);
  __builtin_amdgcn_s_waitcnt(kWaitAllLoads);
  __syncthreads();
  // The query fragments must have arrived before the loop: left pending, the compiler's wait for
  // them inside the loop would also cover the loads that prefetch the next block.
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) asm volatile("" ::"v"(qf[ks]));
  auto block = [&](int blk, auto own_references) {
    constexpr bool own = decltype(own_references)::value;
    const int k0 = blk * BSW + WK * kg;  // this wave's 32 NKT keys
    const bf16_t* kt_ = smem + (blk & 1) * (KT + VT);
    const bf16_t* vt_ = kt_ + KT;
    if (blk + 1 < nblk) {  // the other stage: every wave left it at the last barrier
      bf16_t* nxt = smem + ((blk + 1) & 1) * (KT + VT);
      dma.template issue<PAD>(rk, nxt, ldb, (blk + 1) * BSW, seq - 1, wave);
      dma.template issue<PAD>(rv, nxt + KT, ldb, (blk + 1) * BSW, seq - 1, wave);
    }
    if (k0 < seq && (!causal || k0 <= qw0 + 31)) {
      // The K fragments of a 32-key tile are requested together, and those of the next tile each
      // as soon as its register is free, so that the LDS latency is paid once, not per product; the
      // first V fragments are requested before the softmax arithmetic for the same reason.
      f32x16 s[NKT];
      bf16x8 kf[DH / 16];
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) kf[ks] = frag_rows<DH>(kt_, WK * kg, 16 * ks, lane);
      __builtin_amdgcn_sched_barrier(0);  // the compiler would sink the reads to their uses again
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        zero(s[kt]);
#pragma unroll
        for (int ks = 0; ks < DH / 16; ++ks) {
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s[kt], 0, 0, 0);
          if (kt + 1 < NKT) kf[ks] = frag_rows<DH>(kt_, WK * kg + 32 * (kt + 1), 16 * ks, lane);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      bf16x8 vf[2][DH / 32];
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) vf[0][dt] = frag_cols<DH>(vt_, 32 * dt, WK * kg, lane);
      __builtin_amdgcn_sched_barrier(0);
      // only blocks that cross the diagonal of this wave's rows or the end of the sequence need masks
      if ((causal && k0 + WK - 1 > qw0) || (k0 + WK > seq)) {
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + 32 * kt + 8 * (r >> 2) + 4 * hl + (r & 3);
            if (key >= seq || (causal && key > qrow)) s[kt][r] = -INFINITY;
          }
      }
      auto finite = [](float m) { return m == -INFINITY ? 0.f : m; };  // no key so far: exp2(-inf - 0) = 0
      auto rescale = [&](float m) {                                    // what is summed so far, from reference m2 to m
        const float alpha = __builtin_amdgcn_exp2f(m2 - finite(m));
        lsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
        m2 = m;
      };
      float ref[NKT];
      if constexpr (own) {
        // one for each tile; it may also fall, to kSlack below the largest score so far, so that probabilities stay below 2^kSlack
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
          float mx = s[kt][0];
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
          mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;
          top = fmaxf(top, mx);
          ref[kt] = mx == -INFINITY ? (kt ? ref[0] : m2) : fmaxf(mx, top - kSlack);
        }
        rescale(ref[0]);
      } else {
        float mx = s[0][0];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        // m2 is the reference the exponentials are taken against, not necessarily the exact running
        // maximum: it moves (and what is summed so far is rescaled) only when some query's maximum
        // has risen by more than SLACK above it, so probabilities stay below 2^kSlack and the
        // quotient o / lsum and lse = m2 + log2(lsum) are the same as with the exact maximum.
        const float m_new = fmaxf(m2, mx * scale_log2);
        if (__any(m_new > m2 + SLACK)) rescale(m_new);
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) ref[kt] = m2;
      }
      float rowsum = 0.f;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        const float m_use = finite(ref[kt]);
        if (own && kt > 0) {
          lsum += rowsum + __shfl_xor(rowsum, 32, 64);
          rowsum = 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r], scale_log2, -m_use));
          s[kt][r] = p;
          rowsum += p;
        }
      }
      rowsum += __shfl_xor(rowsum, 32, 64);
      if (!own || NKT == 1) lsum += rowsum;
#pragma unroll
      for (int g = 0; g < 2 * NKT; ++g) {  // 16 keys at a time: tile g / 2, half g % 2
        if (g + 1 < 2 * NKT) {
#pragma unroll
          for (int dt = 0; dt < DH / 32; ++dt) vf[(g + 1) & 1][dt] = frag_cols<DH>(vt_, 32 * dt, WK * kg + 16 * (g + 1), lane);
        }
        if (own && g == 2) {
          rescale(ref[NKT - 1]);
          lsum += rowsum;
        }
        const bf16x8 pb = acc_to_frag(s[g >> 1], g & 1);
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[g & 1][dt], pb, oacc[dt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitAllLoads);  // this wave's part of the next block has landed
    __syncthreads();
  };
  int blk = 0;
  if constexpr (OWN > 0)
    for (; blk < min(nblk, OWN / NKT); ++blk) block(blk, std::true_type{});
  for (; blk < nblk; ++blk) block(blk, std::false_type{});
  if (KW > 1) {
    // Merge the key groups of each query group: groups 1.. park (O, m, l) in LDS (the tiles are no
    // longer read), group 0 folds them in ascending order.  Slot layout: [DH/2 + 2][64 lanes] fp32.
    constexpr int SLOT = (DH / 2 + 2) * 64;
    static_assert((size_t)QW * (KW - 1) * SLOT * 4 <= (size_t)2 * (KT + VT) * 2, "merge slots must fit in the tiles");
    float* slots = reinterpret_cast<float*>(smem);
    if (kg > 0) {
      float* my = slots + ((kg - 1) * QW + qg) * SLOT;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) my[(dt * 16 + r) * 64 + lane] = oacc[dt][r];
      my[(DH / 2) * 64 + lane] = m2;
      my[(DH / 2 + 1) * 64 + lane] = lsum;
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll 1
    for (int g = 1; g < KW; ++g) {
      const float* other = slots + ((g - 1) * QW + qg) * SLOT;
      const float mo = other[(DH / 2) * 64 + lane], lo = other[(DH / 2 + 1) * 64 + lane];
      const float m_new = fmaxf(m2, mo);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      const float a = __builtin_amdgcn_exp2f(m2 - m_use), bo = __builtin_amdgcn_exp2f(mo - m_use);
      lsum = lsum * a + lo * bo;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = oacc[dt][r] * a + other[(dt * 16 + r) * 64 + lane] * bo;
      m2 = m_new;
    }
  }
  if (qrow < seq) {
    const float inv = 1.0f / lsum;
    bf16_t* orow = o + ((size_t)b * seq + qrow) * h + (size_t)head * dh;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) store_tile_t(orow + 32 * dt, oacc[dt], inv, lane, PAD ? dh - 32 * dt : 32);
    if (hl == 0) lse[((size_t)b * heads + head) * seq + qrow] = (m2 + log2f(lsum)) * kLn2;
  }
}

// Backward, dQ of one block of queries.  Same wave grid as the forward kernel: wave (qg, kg) owns 32 queries and the 32 NKT
// keys starting at 32 NKT kg of every streamed block; 32-key tiles are taken one at a time
// (S and dP, then dS, then dQ^T += K^T dS^T) to keep the register footprint at two waves per SIMD.
// The KW partial dQ of a query group are added in key-group order through LDS at the end.  delta may be NULL.
template <int DH, int QW, int KW, int NKT, bool PAD>
__device__ __forceinline__ void dq_block(bf16_t* smem, int head_batch, int block, int seq, int heads, int dh, int causal,
                                         const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const float* __restrict__ lse,
                                         const bf16_t* __restrict__ d_o, bf16_t* __restrict__ dq, int ld_dq, float* __restrict__ delta, float scale, float scale_log2) {
  constexpr int NT = QW * KW * 64, BQW = 32 * QW, WK = 32 * NKT, BSW = WK * KW;
  constexpr int KT = BSW * DH, VT = BSW * DH;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hl = lane >> 5;
  const int qg = wave % QW, kg = wave / QW;
  const int h = heads * dh, head = head_batch % heads, b = head_batch / heads;
  const int q0 = block * BQW, qw0 = q0 + 32 * qg, qrow = qw0 + (lane & 31);
  const int qclamp = min(qrow, seq - 1);
  const size_t ld = (size_t)3 * h;
  const bf16_t* base = qkv + (size_t)b * seq * ld + (size_t)head * dh;

  bf16x8 qf[DH / 16], dof[DH / 16];
  float dl4[4] = {0.f, 0.f, 0.f, 0.f};
  {
    const bf16_t* qp = base + (size_t)qclamp * ld;
    const size_t orow = ((size_t)b * seq + qclamp) * h + (size_t)head * dh;
    const int cols = PAD ? dh : DH;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      qf[ks] = load_frag(qp, 16 * ks + 8 * hl, cols);
      dof[ks] = load_frag(d_o + orow, 16 * ks + 8 * hl, cols);
      const bf16x8 of = load_frag(o + orow, 16 * ks + 8 * hl, cols);
#pragma unroll
      for (int e = 0; e < 8; ++e) dl4[ks & 3] = __builtin_fmaf((float)dof[ks][e], (float)of[e], dl4[ks & 3]);
    }
  }
  // in the order of the key blocks' own delta, eight lanes to a query: both forms of the backward pass give the same bits
  float dl = (dl4[0] + dl4[2]) + (dl4[1] + dl4[3]);
  dl += __shfl_xor(dl, 32, 64);
  const size_t stat = ((size_t)b * heads + head) * seq + qclamp;
  if (delta && kg == 0 && hl == 0 && qrow < seq) delta[stat] = dl;
  const float lse2 = lse[stat] * kLog2e;
  f32x16 acc[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) zero(acc[dt]);

  const int kend = causal ? min(seq, q0 + BQW) : seq;
  const int nblk = (kend + BSW - 1) / BSW;
  const i32x4 rk = make_rsrc(base + h), rv = make_rsrc(base + 2 * h);
  const uint32_t ldb = (uint32_t)ld * 2;
  if (PAD) zero_tiles<NT>(smem, 2 * (KT + VT), tid);
  BlockDma<BSW, DH, NT> dma;
  dma.init(wave, lane, PAD ? dh : DH);
  dma.template issue<PAD>(rk, smem, ldb, 0, seq - 1, wave);
  dma.template issue<PAD>(rv, smem + KT, ldb, 0, seq - 1, wave);
  __builtin_amdgcn_s_waitcnt(kWaitAllLoads);
  __syncthreads();
  for (int blk = 0; blk < nblk; ++blk) {
    const bf16_t* kt_ = smem + (blk & 1) * (KT + VT);
    const bf16_t* vt_ = kt_ + KT;
    if (blk + 1 < nblk) {
      bf16_t* nxt = smem + ((blk + 1) & 1) * (KT + VT);
      dma.template issue<PAD>(rk, nxt, ldb, (blk + 1) * BSW, seq - 1, wave);
      dma.template issue<PAD>(rv, nxt + KT, ldb, (blk + 1) * BSW, seq - 1, wave);
    }
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      const int trow = WK * kg + 32 * kt;   // tile row of this 32-key tile
      const int k0 = blk * BSW + trow;      // its first key
      if (k0 >= seq || (causal && k0 > qw0 + 31)) continue;
      f32x16 s, dp;
      zero(s);
      zero(dp);
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DH>(kt_, trow, 16 * ks, lane), qf[ks], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DH>(vt_, trow, 16 * ks, lane), dof[ks], dp, 0, 0, 0);
      }
      if ((causal && k0 + 31 > qw0) || (k0 + 32 > seq)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + 8 * (r >> 2) + 4 * hl + (r & 3);
          const bool dead = key >= seq || (causal && key > qrow);
          const float p = dead ? 0.f : __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -lse2));
          s[r] = p * (dp[r] - dl);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -lse2)) * (dp[r] - dl);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8 dsb = acc_to_frag(s, t);
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
          acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols<DH>(kt_, 32 * dt, trow + 16 * t, lane), dsb, acc[dt],
                                                            0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitAllLoads);
    __syncthreads();
  }
  if (KW > 1) {
    constexpr int SLOT = (DH / 2) * 64;  // [DH/2 registers][64 lanes] fp32
    static_assert((size_t)QW * (KW - 1) * SLOT * 4 <= (size_t)2 * (KT + VT) * 2, "merge slots must fit in the tiles");
    float* slots = reinterpret_cast<float*>(smem);
    if (kg > 0) {
      float* my = slots + ((kg - 1) * QW + qg) * SLOT;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) my[(dt * 16 + r) * 64 + lane] = acc[dt][r];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll 1
    for (int g = 1; g < KW; ++g) {
      const float* other = slots + ((g - 1) * QW + qg) * SLOT;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] += other[(dt * 16 + r) * 64 + lane];
    }
  }
  if (qrow < seq) {
    bf16_t* row = dq + ((size_t)b * seq + qrow) * ld_dq + (size_t)head * dh;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) store_tile_t(row + 32 * dt, acc[dt], scale, lane, PAD ? dh - 32 * dt : 32);
  }
}

template <int DH, int QW, int KW, int NKT, bool PAD>
__global__ __launch_bounds__(QW * KW * 64, QW * KW == 4 ? 2 : 1) void attn_bwd_dq_mfma(
    int seq, int heads, int dh, int causal, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const float* __restrict__ lse,
    const bf16_t* __restrict__ d_o, bf16_t* __restrict__ dq, int ld_dq, float* __restrict__ delta, float scale, float scale_log2) {
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  // grid = (heads * batch, query blocks); under a causal mask late query blocks see the most keys,
  // so they are dealt out first and the short ones fill the tail
  const int block = causal ? (int)(gridDim.y - 1 - blockIdx.y) : (int)blockIdx.y;
  dq_block<DH, QW, KW, NKT, PAD>(smem, blockIdx.x, block, seq, heads, dh, causal, qkv, o, lse, d_o, dq, ld_dq, delta, scale, scale_log2);
}

// delta = rowsum(dO * O) of a block of BSQ queries by NT = 8 BSQ threads, eight to a query: rows requested with load(), sums left
// in LDS by put().
template <int DH, int BSQ, int NT, bool PAD>
struct OwnDelta {
  static_assert(NT == 0 || NT == 8 * BSQ, "eight threads to a query");
  u32x4 rd[DH / 64], ro[DH / 64];
  __device__ __forceinline__ void load(const bf16_t* dob, const bf16_t* d_o, const bf16_t* o, int q0, int seq, int h, int dh, int tid) {
    const size_t row = (size_t)(dob - d_o) + (size_t)min(q0 + (tid >> 3), seq - 1) * h;
#pragma unroll
    for (int v = 0; v < DH / 64; ++v) {
      const int col = 8 * ((tid & 7) + 8 * v);
      const u32x4 z = {0u, 0u, 0u, 0u};
      const bool in = !PAD || col < dh;
      rd[v] = in ? *reinterpret_cast<const u32x4*>(d_o + row + col) : z;
      ro[v] = in ? *reinterpret_cast<const u32x4*>(o + row + col) : z;
    }
  }
  __device__ __forceinline__ void put(float* to, int tid) const {
    float d = 0.f;
#pragma unroll
    for (int v = 0; v < DH / 64; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d = __builtin_fmaf(bf16lo_to_f32(rd[v][e]), bf16lo_to_f32(ro[v][e]), d);
        d = __builtin_fmaf(bf16hi_to_f32(rd[v][e]), bf16hi_to_f32(ro[v][e]), d);
      }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
    if ((tid & 7) == 0) to[tid >> 3] = d;
  }
};

// Backward, dK and dV.  A workgroup owns 32 KG keys of one head and streams blocks of 32 QG queries
// (Q and dO tiles plus their log-sum-exp and delta).  Each (key group, query group) pair is served
// by TWO waves with different roles, which halves the accumulators a wave has to hold:
//   role 0 keeps K:  S = Q K^T,  P = exp2(S scale - lse),  dV^T += dO^T P;   hands P over through LDS;
//   role 1 keeps V:  dP = dO V^T,  dS = P (dP - delta),     dK^T += Q^T dS.
// Both roles run the same two matrix products per tile (one against Q, one against dO); only the
// elementwise step between them differs.  The QG partial sums of a key group are added in
// query-group order through LDS at the end.  dqkv may be qkv itself: a key block is read only by the workgroup that owns it.
//
// KW > 0: both halves of the backward pass in one launch, for shapes that leave compute units idle: a workgroup is either a block
// of queries (odd blockIdx.y, a wave grid of KG x KW) or one of keys, dealt out alternately with the longest of each first, so one kind
// fills what the other leaves.  Nothing passes between them: delta = rowsum(dO * O) is formed here too, eight threads to a
// query, from rows of dO and O requested a block ahead.  qkv must not be dqkv then: every query block reads all keys.
// bf16, causal, two launches / one: 2 heads of 128, 192 tokens 24 / 12 us; 16 heads of 128, 1024 tokens 50 / 44 us.
template <int DH, int KG, int QG, bool PAD, int KW>
__global__ __launch_bounds__(KG * QG * 128, KG * QG == 2 ? (KW > 0 ? 2 : 3) : 1) void attn_bwd_dkv_mfma(
    int seq, int heads, int dh, int causal, const bf16_t* qkv, const bf16_t* __restrict__ o, const float* __restrict__ lse,
    const float* __restrict__ delta, const bf16_t* __restrict__ d_o, bf16_t* dqkv, float scale, float scale_log2) {
  constexpr bool DELTA = KW > 0;
  constexpr int NP = KG * QG, NT = NP * 128, BK = 32 * KG, BSQ = 32 * QG;
  constexpr int QT = BSQ * DH;
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];  // [2][Q tile | dO tile], stats, P exchange
  if constexpr (KW > 0) {
    static_assert(KG * KW * 64 == NT, "one block size for both halves");
    if (blockIdx.y & 1) {
      const int block = causal ? (int)((gridDim.y - 1 - blockIdx.y) >> 1) : (int)(blockIdx.y >> 1);
      dq_block<DH, KG, KW, 1, PAD>(smem, blockIdx.x, block, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, 3 * heads * dh, nullptr, scale,
                                   scale_log2);
      return;
    }
  }
  float* stats = reinterpret_cast<float*>(smem + 4 * QT);       // [2][lse2[BSQ] | delta[BSQ]]
  float* xch = stats + 4 * BSQ;                                  // [NP][16 registers][64 lanes]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hl = lane >> 5;
  const int role = wave / NP, pair = wave % NP, kg = pair % KG, qg = pair / KG;
  // grid = (heads * batch, key blocks): early key blocks see the most queries and go first
  const int h = heads * dh, head = blockIdx.x % heads, b = blockIdx.x / heads;
  const int k0 = (KW > 0 ? blockIdx.y >> 1 : blockIdx.y) * BK, kw0 = k0 + 32 * kg, krow = kw0 + (lane & 31);
  const size_t ld = (size_t)3 * h;
  const bf16_t* base = qkv + (size_t)b * seq * ld + (size_t)head * dh;
  const bf16_t* dob = d_o + (size_t)b * seq * h + (size_t)head * dh;
  const float* lse_b = lse + ((size_t)b * heads + head) * seq;
  const float* delta_b = delta + ((size_t)b * heads + head) * seq;

  bf16x8 kvf[DH / 16];  // role 0: K rows of this key group; role 1: V rows
  {
    const bf16_t* kp = base + (size_t)min(krow, seq - 1) * ld + (role ? 2 * h : h);
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) kvf[ks] = load_frag(kp, 16 * ks + 8 * hl, PAD ? dh : DH);
  }
  f32x16 acc[DH / 32];  // role 0: dV^T, role 1: dK^T (unscaled)
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) zero(acc[dt]);
  const int qstart = causal ? (k0 / BSQ) * BSQ : 0;
  const int nblk = (seq - qstart + BSQ - 1) / BSQ;
  const i32x4 rq = make_rsrc(base), rdo = make_rsrc(dob);
  const uint32_t ldb = (uint32_t)ld * 2, hb = (uint32_t)h * 2;
  if (PAD) zero_tiles<NT>(smem, 4 * QT, tid);
  BlockDma<BSQ, DH, NT> dma;
  dma.init(wave, lane, PAD ? dh : DH);
  float st_reg = 0.f;  // threads 0..BSQ-1: lse2 of query tid; BSQ..2 BSQ-1: delta of query tid-BSQ
  auto load_stats = [&](int q0) {
    if (tid < 2 * BSQ) {
      const int qi = q0 + (tid % BSQ);
      st_reg = qi < seq ? (tid < BSQ ? lse_b[qi] * kLog2e : DELTA ? 0.f : delta_b[qi]) : 0.f;
    }
  };
  OwnDelta<DH, BSQ, DELTA ? NT : 0, PAD> own;
  dma.template issue<PAD>(rq, smem, ldb, qstart, seq - 1, wave);
  dma.template issue<PAD>(rdo, smem + QT, hb, qstart, seq - 1, wave);
  load_stats(qstart);
  if constexpr (DELTA) own.load(dob, d_o, o, qstart, seq, h, dh, tid);
  if (tid < (DELTA ? 1 : 2) * BSQ) stats[tid] = st_reg;
  if constexpr (DELTA) own.put(stats + BSQ, tid);
  __builtin_amdgcn_s_waitcnt(kWaitAllLoads);
  __syncthreads();
  float* my_xch = xch + pair * (16 * 64) + lane;
  for (int blk = 0; blk < nblk; ++blk) {
    const int q0 = qstart + blk * BSQ + 32 * qg;  // the pair's 32 queries
    const int trow = 32 * qg;
    const bf16_t* qt_ = smem + (blk & 1) * 2 * QT;
    const bf16_t* dot_ = qt_ + QT;
    const bf16_t* first = role ? dot_ : qt_;    // role 0: S = Q K^T        role 1: dP = dO V^T
    const bf16_t* second = role ? qt_ : dot_;   // role 0: dV^T += dO^T P   role 1: dK^T += Q^T dS
    const float* st_ = stats + (blk & 1) * 2 * BSQ + (role ? BSQ : 0) + trow;  // lse2 (role 0) or delta (role 1)
    if (blk + 1 < nblk) {  // the other stage: every wave left it at the last barrier
      bf16_t* nxt = smem + ((blk + 1) & 1) * 2 * QT;
      dma.template issue<PAD>(rq, nxt, ldb, qstart + (blk + 1) * BSQ, seq - 1, wave);
      dma.template issue<PAD>(rdo, nxt + QT, hb, qstart + (blk + 1) * BSQ, seq - 1, wave);
      load_stats(qstart + (blk + 1) * BSQ);
      if constexpr (DELTA) own.load(dob, d_o, o, qstart + (blk + 1) * BSQ, seq, h, dh, tid);
    }
    const bool active = q0 < seq && (!causal || q0 + 31 >= kw0);  // the same for both waves of a pair
    f32x16 t;
    if (active) {
      zero(t);
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks)
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DH>(first, trow, 16 * ks, lane), kvf[ks], t, 0, 0, 0);
      if (role == 0) {
        if ((causal && q0 < kw0 + 31) || (q0 + 32 > seq) || (kw0 + 32 > seq)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int qi = 8 * (r >> 2) + 4 * hl + (r & 3);
            const int query = q0 + qi;
            const bool dead = query >= seq || krow >= seq || (causal && krow > query);
            t[r] = dead ? 0.f : __builtin_amdgcn_exp2f(__builtin_fmaf(t[r], scale_log2, -st_[qi]));
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int qi = 8 * (r >> 2) + 4 * hl + (r & 3);
            t[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(t[r], scale_log2, -st_[qi]));
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) my_xch[r * 64] = t[r];
      }
    }
    __syncthreads();  // P of every active pair is in LDS
    if (active) {
      if (role == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int qi = 8 * (r >> 2) + 4 * hl + (r & 3);
          t[r] = my_xch[r * 64] * (t[r] - st_[qi]);
        }
      }
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const bf16x8 fb = acc_to_frag(t, tt);
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
          acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols<DH>(second, 32 * dt, trow + 16 * tt, lane), fb,
                                                            acc[dt], 0, 0, 0);
      }
    }
    if (blk + 1 < nblk && tid < (DELTA ? 1 : 2) * BSQ) stats[((blk + 1) & 1) * 2 * BSQ + tid] = st_reg;
    if constexpr (DELTA) {
      if (blk + 1 < nblk) own.put(stats + ((blk + 1) & 1) * 2 * BSQ + BSQ, tid);
    }
    __builtin_amdgcn_s_waitcnt(kWaitAllLoads);
    __syncthreads();  // next tiles staged; the exchange slots may be rewritten
  }
  // Merge the query groups, one after the other so that one set of slots is enough:
  // slot of (role, key group) = [DH/2 registers][64 lanes] fp32.
  if (QG > 1) {
    constexpr int SLOT = (DH / 2) * 64;
    float* slot = reinterpret_cast<float*>(smem) + (role * KG + kg) * SLOT + lane;
#pragma unroll 1
    for (int g = 1; g < QG; ++g) {
      if (qg == g) {
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) slot[(dt * 16 + r) * 64] = acc[dt][r];
      }
      __syncthreads();
      if (qg == 0) {
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[dt][r] += slot[(dt * 16 + r) * 64];
      }
      __syncthreads();
    }
  }
  if (qg == 0 && krow < seq) {
    bf16_t* row = dqkv + ((size_t)b * seq + krow) * ld + (size_t)head * dh + (role ? h : 2 * h);
    const float mul = role ? scale : 1.0f;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) store_tile_t(row + 32 * dt, acc[dt], mul, lane, PAD ? dh - 32 * dt : 32);
  }
}

template <int DH, int QW, int KW, int NKT, bool PAD, int OWN = 0>
int fwd_launch(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o, float* lse) {
  constexpr size_t lds = 2 * sizeof(bf16_t) * 32 * NKT * KW * 2 * DH;
  static std::atomic<bool> done{false};
  if (int rc = reserve_lds(attn_fwd_mfma<DH, QW, KW, NKT, PAD, OWN>, lds, done, "attention_forward")) return rc;
  const float scale_log2 = kLog2e / sqrtf((float)dh);
  attn_fwd_mfma<DH, QW, KW, NKT, PAD, OWN><<<dim3(heads * batch, (seq + 32 * QW - 1) / (32 * QW)), dim3(QW * KW * 64), lds, st>>>(
      seq, heads, dh, causal, (const bf16_t*)qkv, (bf16_t*)o, lse, scale_log2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "attention_forward launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

// Forward.  Few tokens and heads leave the chain of one workgroup as the time, so rows get small workgroups whose waves split the other
// side; the more workgroups there are (w of 64 rows), the less that is worth and the more it costs to fetch and to fold.
//   128 queries, every wave all keys: from 512 such workgroups on; with references of its own (see attn_fwd_mfma) also below that, from
//       w = 768 on, for heads of more than 64 without a mask from 512 on
//   32 queries, four waves that take every fourth 32-key tile: more than 192 tokens, up to 256 of these workgroups
//   64 queries, eight waves in four key groups: long sequences, whose chain counts most.  Longer than 512 tokens (256 with heads of up to
//       64) up to w = 256; than 2 w (1.5 w; without a mask 512 tokens, and never with heads of more than 64) up to 512; beyond that only heads
//       of up to 64 under a mask, longer than 5 (w - 512) + 500
//   64 queries, four waves in two key groups: everything else
// Over 5220 calls (1 .. 64 heads of 40 .. 128, 1 .. 8 sequences of 8 .. 4096 tokens) the shape picked is 0.6 % slower than the best one on
// average, 1.24 times at worst; against 64-row workgroups of eight waves below 512 128-row ones (the rule it replaced at first) 0.83 of the time, 1.06 at
// worst.  us of 32 / 64 four waves / 64 eight waves / 128 queries, heads of 128, causal: 16 x 256 tokens (w 64) 7.9 / 8.6 / 9.7 / 11.4, 64 x 192 (w 192) 12.1 / 8.0 / 9.7 /
// 9.1, 16 x 1000 (w 256) 21.4 / 19.4 / 18.0 / 26.8, 64 x 512 (w 512) 32 / 15.9 / 21 / 18.4, 16 x 2048 (w 512) 57 / 38.6 / 36.5 / 47.6, 8 x 4096 (w 512) 91 / 69 / 57 / 87,
// 26 x 1500 (w 624) 63 / 32 / 45 / 40, 60 x 1000 (w 960) 81 / 36 / 51 / 32; not causal 32 x 1000 (w 512) 55 / 30.3 / 35.6 / 28.6, 5 x 3000 (w 235) 69 / 50 / 41 / 66;
// heads of 64, causal 16 x 2048 (w 512) 26 / 24.7 / 21.7 / 34.8, 48 x 768 (w 576) 19.4 / 13.0 / 15.9 / 17.0; not causal 16 x 2048 41 / 31.8 / 30.4 / 34.7.
// The attn_shape tuning switch (0|1|2) forces the eight-wave one (0) or the last (1, 2), and a family of the backward pass in two launches
// (tests and tuning).
enum FwdShape { kFwd32, kFwd64, kFwd64Eight, kFwd128, kFwd128Own };
FwdShape fwd_shape(int batch, int seq, int heads, int dh, int causal) {
  if (const int f = tuning(kTuneAttnShape); f >= 0) return f == 0 ? kFwd64Eight : kFwd128;
  const int64_t pairs = (int64_t)heads * batch, w = (seq + 63) / 64 * pairs;
  const bool wide = dh > 64;
  if ((seq + 127) / 128 * pairs >= 512) return kFwd128;
  if (seq <= 64) return kFwd64;
  if ((seq + 31) / 32 * pairs <= 256) return seq <= 192 ? kFwd64 : kFwd32;
  if (w <= 256) return seq <= (wide ? 512 : 256) ? kFwd64 : kFwd64Eight;
  if (w <= 512) {
    if (causal) return 2 * (int64_t)seq <= (wide ? 4 : 3) * w ? kFwd64 : kFwd64Eight;
    return wide || seq <= 512 ? kFwd64 : kFwd64Eight;
  }
  if (causal && !wide) return seq <= 5 * (w - 512) + 500 ? kFwd64 : kFwd64Eight;
  return w > 768 || (wide && !causal) ? kFwd128Own : kFwd64;
}

// Backward in two launches.  Family 0: 64-row workgroups of 8 waves, the dQ ones with four key groups; one workgroup fills a unit.  Family 1:
// 128-query workgroups (64-key ones in the dK/dV kernel) of 4 waves, two or three to a unit.  Family 3: the 64-row workgroups of 4 waves that
// attention_merged's kind 2 has in one launch.  By w = 64-row workgroups: 0 as long as its workgroups fit the 256 units at once; 1 from 512 (128-row
// block, head) pairs on.  Between, the chain counts for long sequences and the units for many workgroups: 0 up to w = 512 (1 where many
// workgroups of up to 1024 tokens and wide heads fill the units without a mask), beyond that the longer the sequence the more workgroups 0
// stays the faster for, and 3 between the two.  Where kind 2 does the one launch beyond one round of it, and for one block of rows, 3 is as fast in place and
// gives the same bits.  us of 0 / 1 / 3 in place, heads of 128: causal 16 heads x 1000 tokens (w 256) 54 / 81 / 67, 28 x 600 (w 280) 53 / 61 / 56, 16 x 2048 (w 512) 108 / 148 / 126,
// 20 x 2048 (w 640) 147 / 163 / 138, 26 x 1500 (w 624) 131 / 132 / 114, 12 x 4096 (w 768) 265 / 303 / 254, 60 x 1000 (w 960) 146 / 108 / 107; not causal 32 x 768 (w 384) 86 / 73 / 71, 32 x 1000 (w 512) 117 /
// 114 / 109; heads of 64, causal 16 x 2048 70 / 106 / 94, 12 x 4096 143 / 203 / 178, 48 x 768 (w 576) 48 / 54 / 49, 4 x 24 x 512 (w 768) 51 / 44 / 41.  Over the calls that attention_merged
// names, 0.93 of the time of 0 below 512 pairs and 1 from there on, 1.06 at worst.
int bwd_family(int batch, int seq, int heads, int dh, int causal) {
  if (const int f = tuning(kTuneAttnShape); f >= 0) return f;
  const int64_t pairs = (int64_t)heads * batch, w = (seq + 63) / 64 * pairs;
  if (attention_merged(batch, seq, heads, dh, causal) == 2 && (seq <= 64 || w > 256)) return 3;
  if (w <= 256) return 0;
  if ((seq + 127) / 128 * pairs >= 512) return 1;
  const bool wide = dh > 64;
  if (w <= 512) return !causal && wide && w > 384 && seq <= 1024 ? 1 : 0;
  if (!wide) return seq < w - (causal ? 128 : 0) ? 1 : 0;
  if (!causal) return 1;
  return seq < 4 * (w - 512) + 500 ? 1 : seq < 10 * (w - 512) + 900 ? 3 : 0;
}

// The one-launch form of the backward pass apart from qkv (0: two launches, as in place).
int bwd_merged(int batch, int seq, int heads, int dh, int causal) {
  return tuning(kTuneAttnShape) >= 0 ? 0 : attention_merged(batch, seq, heads, dh, causal);
}

template <int DH, bool PAD>
int fwd_t(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o, float* lse) {
  switch (fwd_shape(batch, seq, heads, dh, causal)) {
    case kFwd32: return fwd_launch<DH, 1, 4, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse);
    case kFwd64: return fwd_launch<DH, 2, 2, 1, PAD, 2>(st, batch, seq, heads, dh, causal, qkv, o, lse);
    case kFwd64Eight: return fwd_launch<DH, 2, 4, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse);
    case kFwd128Own: return fwd_launch<DH, 4, 1, 2, PAD, 4>(st, batch, seq, heads, dh, causal, qkv, o, lse);
    default: return fwd_launch<DH, 4, 1, 2, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  }
}

template <int DH, int QW, int KW, int NKT>
constexpr size_t lds_dq() { return 2 * sizeof(bf16_t) * 32 * NKT * KW * 2 * DH; }
template <int DH, int KG, int QG>
constexpr size_t lds_dkv() {
  constexpr size_t tiles = 4 * sizeof(bf16_t) * 32 * QG * DH + (4 * 32 * QG + (size_t)KG * QG * 16 * 64) * sizeof(float);
  constexpr size_t merge = QG > 1 ? (size_t)2 * KG * (DH / 2) * 64 * sizeof(float) : 0;
  return tiles > merge ? tiles : merge;
}

template <int DH, int QW, int KW, int NKT, int KG, int QG, bool PAD>
int bwd_launch(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o, const float* lse,
               const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  constexpr size_t dq_bytes = lds_dq<DH, QW, KW, NKT>(), dkv_bytes = lds_dkv<DH, KG, QG>();
  static_assert(dq_bytes <= 160 * 1024 && dkv_bytes <= 160 * 1024, "tiles exceed the LDS of a compute unit");
  static std::atomic<bool> done_dq{false}, done_dkv{false};
  if (int rc = reserve_lds(attn_bwd_dq_mfma<DH, QW, KW, NKT, PAD>, dq_bytes, done_dq, "attention_backward")) return rc;
  if (int rc = reserve_lds(attn_bwd_dkv_mfma<DH, KG, QG, PAD, 0>, dkv_bytes, done_dkv, "attention_backward")) return rc;
  const float scale = 1.0f / sqrtf((float)dh), scale_log2 = kLog2e * scale;
  attn_bwd_dq_mfma<DH, QW, KW, NKT, PAD><<<dim3(heads * batch, (seq + 32 * QW - 1) / (32 * QW)), dim3(QW * KW * 64), dq_bytes, st>>>(
      seq, heads, dh, causal, (const bf16_t*)qkv, (const bf16_t*)o, lse, (const bf16_t*)d_o, (bf16_t*)dq, ld_dq, delta, scale, scale_log2);
  attn_bwd_dkv_mfma<DH, KG, QG, PAD, 0><<<dim3(heads * batch, (seq + 32 * KG - 1) / (32 * KG)), dim3(KG * QG * 128), dkv_bytes, st>>>(
      seq, heads, dh, causal, (const bf16_t*)qkv, nullptr, lse, delta, (const bf16_t*)d_o, (bf16_t*)dqkv, scale, scale_log2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "attention_backward launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

template <int DH, int QW, int KW, int NKT, int KG, int QG, bool PAD>
int bwd_merged_launch(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o, const float* lse,
                      const void* d_o, void* dqkv) {
  constexpr size_t lds = lds_dq<DH, QW, KW, NKT>() > lds_dkv<DH, KG, QG>() ? lds_dq<DH, QW, KW, NKT>() : lds_dkv<DH, KG, QG>();
  static std::atomic<bool> done{false};
  static_assert(QW == KG && NKT == 1, "one row block for both halves");
  auto kern = attn_bwd_dkv_mfma<DH, KG, QG, PAD, KW>;
  if (int rc = reserve_lds(kern, lds, done, "attention_backward")) return rc;
  const float scale = 1.0f / sqrtf((float)dh);
  kern<<<dim3(heads * batch, 2 * ((seq + 32 * QW - 1) / (32 * QW))), dim3(QW * KW * 64), lds, st>>>(
      seq, heads, dh, causal, (const bf16_t*)qkv, (const bf16_t*)o, lse, nullptr, (const bf16_t*)d_o, (bf16_t*)dqkv, scale, kLog2e * scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "attention_backward launch failed: %s", hipGetErrorString(e));
  return PMC_OK;
}

template <int DH, bool PAD>
int bwd_t(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o, const float* lse,
          const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  const int fam = bwd_family(batch, seq, heads, dh, causal), merged = bwd_merged(batch, seq, heads, dh, causal);
  if (dq == dqkv && merged == 1)
    return bwd_merged_launch<DH, 2, 4, 1, 2, 2, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv);
  if (dq == dqkv && merged == 2)
    return bwd_merged_launch<DH, 2, 2, 1, 2, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv);
  if (fam == 3)
    return bwd_launch<DH, 2, 2, 1, 2, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  if (fam == 0)
    return bwd_launch<DH, 2, 4, 1, 2, 2, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  if (fam == 2)
    return bwd_launch<DH, 4, 1, 2, 4, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  return bwd_launch<DH, 4, 1, 2, 2, 1, PAD>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
}

int check(const char* what, int batch, int seq, int heads, int dh, const void* qkv) {
  if (batch <= 0 || seq <= 0 || heads <= 0) return fail(PMC_ERR_INVALID, "%s: batch=%d seq=%d heads=%d", what, batch, seq, heads);
  if (dh < 8 || dh > 128 || dh % 8)
    return fail(PMC_ERR_INVALID, "%s: matrix-core path needs a head size that is a multiple of 8 up to 128, got %d", what, dh);
  if (seq > 65535 * 32 || (long)heads * batch > 0x7fffffffL) return fail(PMC_ERR_INVALID, "%s: seq or heads*batch exceed the grid limit", what);
  if (reinterpret_cast<uintptr_t>(qkv) & 15) return fail(PMC_ERR_INVALID, "%s: qkv must be 16-byte aligned", what);
  // the tile loads address one sequence's rows with 32-bit byte offsets inside a 2 GB window
  if ((size_t)seq * 3 * heads * dh * 2 > 0x7fffffffull)
    return fail(PMC_ERR_INVALID, "%s: one sequence's q|k|v rows (%d x %d) exceed 2 GB", what, seq, 3 * heads * dh);
  return PMC_OK;
}

}  // namespace

// Head sizes 64 and 128 fill the kernels' tiles; the other multiples of 8 run in the next larger
// tile with its remaining columns held at zero.
void attention_mfma_plan(int batch, int seq, int heads, int dh, int causal, int* out) {
  out[0] = fwd_shape(batch, seq, heads, dh, causal);
  out[1] = bwd_merged(batch, seq, heads, dh, causal);
  out[2] = bwd_family(batch, seq, heads, dh, causal);
}

int attention_forward_mfma(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o,
                           float* lse) {
  if (int rc = check("attention_forward", batch, seq, heads, dh, qkv)) return rc;
  if (reinterpret_cast<uintptr_t>(o) & 15) return fail(PMC_ERR_INVALID, "attention_forward: o must be 16-byte aligned");
  if (dh == 64) return fwd_t<64, false>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  if (dh == 128) return fwd_t<128, false>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  if (dh < 64) return fwd_t<64, true>(st, batch, seq, heads, dh, causal, qkv, o, lse);
  return fwd_t<128, true>(st, batch, seq, heads, dh, causal, qkv, o, lse);
}

// dq (pitch ld_dq): a buffer of its own if dqkv is qkv, otherwise dqkv.
int attention_backward_mfma(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o,
                            const float* lse, const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  if (int rc = check("attention_backward", batch, seq, heads, dh, qkv)) return rc;
  if ((reinterpret_cast<uintptr_t>(o) | reinterpret_cast<uintptr_t>(d_o) | reinterpret_cast<uintptr_t>(dqkv) |
       reinterpret_cast<uintptr_t>(dq)) & 15)
    return fail(PMC_ERR_INVALID, "attention_backward: tensors must be 16-byte aligned");
  if (dh == 64) return bwd_t<64, false>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  if (dh == 128) return bwd_t<128, false>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  if (dh < 64) return bwd_t<64, true>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  return bwd_t<128, true>(st, batch, seq, heads, dh, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
}

}  // namespace k
}  // namespace pmc
