// Row-wise kernels bounded by HBM bandwidth: LayerNorm forward, LayerNorm input-gradient (with the
// gain/bias gradient partial sums), column sums for the bias gradients, and a pitched row copy.
// Forward: one 64-lane wave owns a row and the row reductions are wave shuffles.  Backward: one to
// eight waves share a row.  Reductions across rows go through fixed-order partial sums, so results
// do not depend on scheduling.
#include <mutex>

#include "dev_common.h"
#include "kernels.h"
#include "wgrad_batch.h"

namespace pmc {
namespace k {
namespace {

// Scratch of layernorm_backward_static: the partial sums of the gain/bias gradients, in a device
// array that exists from the moment the code object is loaded (one copy per GPU, held until the
// process ends), so that callers who cannot allocate device memory need no workspace.  In host code
// the name `scratch` is only a handle for hipGetSymbolAddress; kernels get the address it returns.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kWaves = 4;
constexpr int kBwdWaves = 8;  // LayerNorm backward: waves (= rows in flight) per workgroup
// LayerNorm backward: copies of the column sums a workgroup keeps in LDS (at most 48 KB with WR = 1 .. 4 waves to a row,
// so that two or three workgroups still fit a compute unit).
constexpr int ln_bwd_copies(int wr) { return kBwdWaves / wr > 1 ? kBwdWaves / wr / 2 : 1; }

template <typename T, int NC>
__global__ __launch_bounds__(256) void ln_fwd_kernel(int rows, int h, const T* __restrict__ x,
                                                      const T* __restrict__ gain, const T* __restrict__ bias,
                                                      float eps, T* __restrict__ y, float* __restrict__ mean,
                                                      float* __restrict__ rstd, T* __restrict__ x_copy) {
  constexpr int V = Vec<T>::N;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = blockIdx.x * kWaves + wave;
  if (row >= rows) return;
  const T* xr = x + (size_t)row * h;
  // The row stays in registers as it is in memory (4 registers per 16-byte chunk; unpacked again for each of
  // the three passes): at 5120 bf16 columns that is 7 waves per SIMD instead of 2, and a wave lives for
  // little more than the latency of its loads, so the waves in flight are what the bandwidth comes from.
  u32x4 raw[NC];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * V;
    if (col < h) {
      raw[c] = Vec<T>::load_raw(xr + col);
      if (x_copy) Vec<T>::store_raw(x_copy + (size_t)row * h + col, raw[c]);
    }
  }

#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * V;
    if (col < h) {
      float v[V];
      Vec<T>::unpack(raw[c], v);
#pragma unroll
      for (int i = 0; i < V; ++i) sum += v[i];
    }
  }
  const float mu = wave_sum(sum) / (float)h;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * V;
    if (col < h) {
      float v[V];
      Vec<T>::unpack(raw[c], v);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float d = v[i] - mu;
        sq += d * d;
      }
    }
  }
  const float rs = 1.0f / sqrtf(wave_sum(sq) / (float)h + eps);
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * V;
    if (col < h) {
      float v[V], g[V], b[V], out[V];
      Vec<T>::unpack(raw[c], v);
      Vec<T>::load(gain + col, g);
      Vec<T>::load(bias + col, b);
#pragma unroll
      for (int i = 0; i < V; ++i) out[i] = g[i] * ((v[i] - mu) * rs) + b[i];
      Vec<T>::store(y + (size_t)row * h + col, out);
    }
  }
}

// Workgroup `block` of `blocks` copies its share of the rows.  It rides along in a launch that is there anyway: a kernel of its own
// took 2 to 5 us at up to 1024 tokens, nearly all of it launch and ramp.
template <typename T, int NT>
__device__ __forceinline__ void copy_rows_part(const RowCopy& copy, int rows, int block, int blocks) {
  constexpr int V = Vec<T>::N;
  const int chunks = copy.cols / V, across = min(chunks, NT), down = NT / across, r0 = threadIdx.x / across, c0 = threadIdx.x % across;
  if (r0 >= down) return;
  for (int r = block * down + r0; r < rows; r += blocks * down)
    for (int c = c0; c < chunks; c += across)
      Vec<T>::store_raw(static_cast<T*>(copy.dst) + (size_t)r * copy.ld_dst + V * c,
                        Vec<T>::load_raw(static_cast<const T*>(copy.src) + (size_t)r * copy.ld_src + V * c));
}
template <typename T>
int copy_blocks(const RowCopy& copy, int rows, int threads) {
  if (!copy.cols) return 0;
  const int down = std::max(1, threads / (copy.cols / Vec<T>::N));
  return std::min((rows + down - 1) / down, 1024);
}

// dx = resid + rstd * (g - mean(g) - xhat * mean(g * xhat)),  g = dy * gain,  xhat = (x - mean) * rstd.
// A workgroup is 8 waves; WR of them share a row (wave w takes the column slice w % WR, NC chunks
// of 64 lanes x V elements), so a lane holds at most 3*V elements per tensor and 8/WR rows are in
// flight per workgroup.  The two row means are summed from the WR slices' wave sums in slice
// order through LDS.  Each lane keeps running column sums of dy * xhat and dy for its own
// columns; at the end the 8/WR waves that share a slice are folded in wave order and the
// workgroup writes one row of partials: partial[block][0..h) = d gain, [h..2h) = d bias.
template <typename T, int NC, int WR>
__global__ __launch_bounds__(kBwdWaves * 64) void ln_bwd_kernel(int rows, int h, const T* __restrict__ dy,
                                                      const T* x, const T* __restrict__ gain,
                                                      const float* __restrict__ mean, const float* __restrict__ rstd,
                                                      const T* resid, T* dx, float* __restrict__ partial, int blocks, RowCopy copy) {
  if ((int)blockIdx.x >= blocks) {
    copy_rows_part<T, kBwdWaves * 64>(copy, rows, blockIdx.x - blocks, gridDim.x - blocks);
    return;
  }
  constexpr int V = Vec<T>::N;
  constexpr int RG = kBwdWaves / WR;  // rows in flight
  constexpr int COPIES = ln_bwd_copies(WR);
  extern __shared__ float red[];      // [COPIES][2][WR * NC * V * 64], then the row sums [2][RG][WR][2]
  float (*stat)[RG][WR][2] = reinterpret_cast<float (*)[RG][WR][2]>(red + COPIES * 2 * WR * NC * V * 64);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rg = wave / WR, slice = wave % WR;
  const int col0 = (slice * NC * 64 + lane) * V;  // chunk c starts at col0 + c * 64 * V
  float pg[NC][V], pb[NC][V], gn[NC][V];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = col0 + c * 64 * V;
#pragma unroll
    for (int i = 0; i < V; ++i) pg[c][i] = pb[c][i] = gn[c][i] = 0.f;
    if (col < h) Vec<T>::load(gain + col, gn[c]);
  }
  int it = 0;
  for (int base = blockIdx.x * RG; base < rows; base += blocks * RG, ++it) {
    const int row = base + rg;
    const bool live = row < rows;
    float xh[NC][V], g[NC][V], r[NC][V];
    float mu = 0.f, rs = 0.f, s1 = 0.f, s2 = 0.f;
    if (live) {
      mu = mean[row];
      rs = rstd[row];
      float xv[NC][V], d[NC][V];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = col0 + c * 64 * V;
#pragma unroll
        for (int i = 0; i < V; ++i) xv[c][i] = d[c][i] = r[c][i] = 0.f;
        if (col < h) {
          Vec<T>::load(x + (size_t)row * h + col, xv[c]);
          Vec<T>::load(dy + (size_t)row * h + col, d[c]);
          if (resid) Vec<T>::load(resid + (size_t)row * h + col, r[c]);
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const bool in = col0 + c * 64 * V < h;  // lanes past the row end hold zeros, but mu != 0
#pragma unroll
        for (int i = 0; i < V; ++i) {
          xh[c][i] = in ? (xv[c][i] - mu) * rs : 0.f;
          g[c][i] = d[c][i] * gn[c][i];
          s1 += g[c][i];
          s2 += g[c][i] * xh[c][i];
          pg[c][i] += d[c][i] * xh[c][i];
          pb[c][i] += d[c][i];
        }
      }
      s1 = wave_sum(s1);
      s2 = wave_sum(s2);
    }
    if constexpr (WR > 1) {
      // Slots alternate with the iteration: a wave can only overwrite a slot two barriers after
      // every wave has read it.
      if (lane == 0) {
        stat[it & 1][rg][slice][0] = s1;
        stat[it & 1][rg][slice][1] = s2;
      }
      __syncthreads();
      s1 = s2 = 0.f;
#pragma unroll
      for (int w = 0; w < WR; ++w) {
        s1 += stat[it & 1][rg][w][0];
        s2 += stat[it & 1][rg][w][1];
      }
    }
    s1 /= (float)h;
    s2 /= (float)h;
    if (live) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = col0 + c * 64 * V;
        if (col < h) {
          float out[V];
#pragma unroll
          for (int i = 0; i < V; ++i) out[i] = r[c][i] + rs * (g[c][i] - s1 - xh[c][i] * s2);
          Vec<T>::store(dx + (size_t)row * h + col, out);
        }
      }
    }
  }
  // Fold: element (c, i) of lane l of slice s lives at red[((s*NC + c)*V + i) * 64 + (l + i*64/V) % 64]
  // (the d-bias half kHalf further on): a wave's 64 lanes hit 64 different words of one 64-word
  // line, and so does the write-out below, which walks i fastest.  Row group w adds into copy w % COPIES, and
  // the write-out adds the copies in order: two barriers, where one copy for all took one per group (4096 rows of
  // 1024 columns 17.6 us, now 13.1; 496 of 832: 8.5, now 5.3; 192 of 256: 6.0, now 4.1).
  constexpr int kHalf = WR * NC * V * 64;
  float* mine = red + (rg % COPIES) * 2 * kHalf;
#pragma unroll
  for (int phase = 0; phase < RG / COPIES; ++phase) {
    if (rg / COPIES == phase) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const int a = ((slice * NC + c) * V + i) * 64 + ((lane + i * (64 / V)) & 63);
          mine[a] = phase ? mine[a] + pg[c][i] : pg[c][i];
          mine[kHalf + a] = phase ? mine[kHalf + a] + pb[c][i] : pb[c][i];
        }
      }
    }
    __syncthreads();
  }
  float* out = partial + (size_t)blockIdx.x * 2 * h;
  for (int j = threadIdx.x; j < h; j += kBwdWaves * 64) {
    const int i = j % V, l = (j / V) & 63, c = j / (V * 64);  // c counts chunks across slices
    const int a = (c * V + i) * 64 + ((l + i * (64 / V)) & 63);
    float dg = red[a], db = red[kHalf + a];
#pragma unroll
    for (int w = 1; w < COPIES; ++w) {
      dg += red[w * 2 * kHalf + a];
      db += red[w * 2 * kHalf + kHalf + a];
    }
    out[j] = dg;
    out[h + j] = db;
  }
}

// For every job j: out_a[i] += sum_p partial_j[p*stride + i] (i < split),
// out_b[i - split] += ... (i >= split).  A block handles 64 columns; its sixteen waves each sum a
// contiguous sixteenth of the parts (loads are independent, so many are in flight), and these sums
// are added in ascending order: the summation order is fixed by (parts) alone.  The chain of loads of one wave is
// the whole time: with four waves four jobs
// of 512 parts of 2048 columns took 15.1 us, now 8.2; 128 parts of 4096 columns 10.5, now 7.1.
constexpr int kSumWaves = 16;
__global__ __launch_bounds__(kSumWaves * 64) void sum_partials_kernel(LnPartialJobs jobs, int width, int split, size_t stride, int copy_rows, bool copy_f32, RowCopy copy) {
  const int sum_blocks = (width + 63) / 64;
  if ((int)blockIdx.x >= sum_blocks * jobs.count) {
    const int block = blockIdx.x - sum_blocks * jobs.count, blocks = gridDim.x - sum_blocks * jobs.count;
    if (copy_f32) copy_rows_part<float, kSumWaves * 64>(copy, copy_rows, block, blocks);
    else copy_rows_part<bf16_t, kSumWaves * 64>(copy, copy_rows, block, blocks);
    return;
  }
  __shared__ float share[kSumWaves][64];
  const int job = blockIdx.x / sum_blocks;
  const float* __restrict__ partial = jobs.partial[job];
  const int parts = jobs.parts[job];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int i = ((int)blockIdx.x - job * sum_blocks) * 64 + lane;
  const int per = (parts + kSumWaves - 1) / kSumWaves, p0 = g * per, p1 = min(parts, p0 + per);
  float acc = 0.f;
  if (i < width) {
    int p = p0;
    for (; p + 8 <= p1; p += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(p + u) * stride + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; p < p1; ++p) acc += partial[(size_t)p * stride + i];
  }
  share[g][lane] = acc;
  __syncthreads();
  if (g == 0 && i < width) {
    float total = share[0][lane];
#pragma unroll
    for (int w = 1; w < kSumWaves; ++w) total += share[w][lane];
    if (i < split) jobs.dgain[job][i] += total;
    else jobs.dbias[job][i - split] += total;
  }
}

// Column sums of up to four matrices with the same row count in one launch: out_j[c] += sum over
// rows of a_j[row][c].  A workgroup owns 64 columns of one matrix.
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(int rows, ColumnSumJobs jobs) {
  __shared__ float red[256 / (64 / Vec<T>::N) * 65];
  int j = 0;
  while (j + 1 < jobs.count && (int)blockIdx.x >= jobs.first_block[j + 1]) ++j;
  column_sum_block<T>([&](int) { return static_cast<const T*>(jobs.a[j]); }, 1, rows, jobs.n[j], jobs.lda[j],
                           ((int)blockIdx.x - jobs.first_block[j]) * 64, jobs.out[j], red, threadIdx.x);
}

template <typename T>
__global__ __launch_bounds__(256) void copy_rows_kernel(int rows, int vec_cols, const T* __restrict__ src, int ld_src,
                                                         T* __restrict__ dst, int ld_dst) {
  constexpr int V = Vec<T>::N;
  const size_t total = (size_t)rows * vec_cols;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i / vec_cols), c = (int)(i % vec_cols) * V;
    *reinterpret_cast<u32x4*>(dst + (size_t)r * ld_dst + c) = *reinterpret_cast<const u32x4*>(src + (size_t)r * ld_src + c);
  }
}

int pick_nc(int h, int vec) {
  const int need = (h + 64 * vec - 1) / (64 * vec);
  for (int nc : {1, 2, 3, 4, 6, 8, 12, 16, 20, 24})
    if (nc >= need) return nc;
  return 0;
}

// LayerNorm backward launch shape: WR waves per row so that a lane holds at most 3 chunks.
struct LnBwdShape {
  int nc, wr;
};
LnBwdShape ln_bwd_shape(int h, int vec) {
  const int need = (h + 64 * vec - 1) / (64 * vec);
  for (int wr : {1, 2, 4, 8}) {
    const int nc = (need + wr - 1) / wr;
    if (nc <= 3) return {nc, wr};
  }
  return {0, 0};
}

constexpr int kLnBwdMaxBlocks = 512;

int ln_bwd_blocks(int rows, int rows_in_flight) {
  const int b = (rows + rows_in_flight - 1) / rows_in_flight;
  return b < 1 ? 1 : (b > kLnBwdMaxBlocks ? kLnBwdMaxBlocks : b);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

#define PMC_LAUNCH_CHECK(what)                                                                \
  do {                                                                                        \
    hipError_t e_ = hipGetLastError();                                                        \
    if (e_ != hipSuccess) return fail(PMC_ERR_HIP, "%s launch failed: %s", what, hipGetErrorString(e_)); \
  } while (0)

template <typename T>
int ln_fwd_t(hipStream_t st, int rows, int h, const void* x, const void* gain, const void* bias, float eps, void* y,
             float* mean, float* rstd, void* x_copy) {
  const int nc = pick_nc(h, Vec<T>::N);
  dim3 grid((rows + kWaves - 1) / kWaves), block(256);
#define LN_FWD_CASE(NC)                                                                                          \
  case NC:                                                                                                       \
    ln_fwd_kernel<T, NC><<<grid, block, 0, st>>>(rows, h, (const T*)x, (const T*)gain, (const T*)bias, eps, (T*)y, \
                                                  mean, rstd, (T*)x_copy);                                       \
    break;
  switch (nc) {
    LN_FWD_CASE(1) LN_FWD_CASE(2) LN_FWD_CASE(3) LN_FWD_CASE(4) LN_FWD_CASE(6) LN_FWD_CASE(8) LN_FWD_CASE(12)
    LN_FWD_CASE(16) LN_FWD_CASE(20) LN_FWD_CASE(24)
    default:
      return fail(PMC_ERR_INVALID, "LayerNorm width %d too large", h);
  }
#undef LN_FWD_CASE
  PMC_LAUNCH_CHECK("layernorm_forward");
  return PMC_OK;
}

template <typename T>
int ln_bwd_t(hipStream_t st, int rows, int h, const void* dy, const void* x, const void* gain, const float* mean,
             const float* rstd, const void* resid, void* dx, float* dgain, float* dbias, float* partial,
             LnPartialJobs* defer, const RowCopy& copy) {
  const LnBwdShape sh = ln_bwd_shape(h, Vec<T>::N);
  if (!sh.nc) return fail(PMC_ERR_INVALID, "LayerNorm width %d too large", h);
  const int blocks = ln_bwd_blocks(rows, kBwdWaves / sh.wr), copying = copy_blocks<T>(copy, rows, kBwdWaves * 64);
  const size_t lds = ((size_t)ln_bwd_copies(sh.wr) * 2 * sh.wr * sh.nc * Vec<T>::N * 64 + 4 * kBwdWaves) * sizeof(float);
#define LN_BWD_CASE(NC, WR)                                                                                  \
  case NC * 16 + WR:                                                                                         \
    if (lds > 64 * 1024 &&                                                                                   \
        hipFuncSetAttribute(reinterpret_cast<const void*>(ln_bwd_kernel<T, NC, WR>),                         \
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)             \
      return fail(PMC_ERR_HIP, "layernorm_backward: cannot reserve %zu bytes of LDS", lds);                  \
    ln_bwd_kernel<T, NC, WR><<<dim3(blocks + copying), dim3(kBwdWaves * 64), lds, st>>>(                               \
        rows, h, (const T*)dy, (const T*)x, (const T*)gain, mean, rstd, (const T*)resid, (T*)dx, partial, blocks, copy); \
    break;
  switch (sh.nc * 16 + sh.wr) {
    LN_BWD_CASE(1, 1) LN_BWD_CASE(2, 1) LN_BWD_CASE(3, 1) LN_BWD_CASE(2, 2) LN_BWD_CASE(3, 2) LN_BWD_CASE(2, 4)
    LN_BWD_CASE(3, 4) LN_BWD_CASE(2, 8) LN_BWD_CASE(3, 8)
    default:
      return fail(PMC_ERR_INVALID, "LayerNorm width %d: no kernel for %d chunks x %d waves", h, sh.nc, sh.wr);
  }
#undef LN_BWD_CASE
  PMC_LAUNCH_CHECK("layernorm_backward");
  LnPartialJobs now;
  LnPartialJobs& jobs = defer ? *defer : now;
  if (jobs.count >= LnPartialJobs::kMax) return fail(PMC_ERR_INVALID, "layernorm_backward: too many deferred reductions");
  jobs.partial[jobs.count] = partial;
  jobs.dgain[jobs.count] = dgain;
  jobs.dbias[jobs.count] = dbias;
  jobs.parts[jobs.count] = blocks;
  ++jobs.count;
  return defer ? PMC_OK : layernorm_backward_reduce(st, h, jobs);
}

}  // namespace

int layernorm_forward(hipStream_t st, int dtype, int rows, int h, const void* x, const void* gain, const void* bias,
                      float eps, void* y, float* mean, float* rstd, void* x_copy) {
  if (rows <= 0 || h <= 0) return fail(PMC_ERR_INVALID, "layernorm: rows=%d h=%d", rows, h);
  const int vec = dtype == PMC_F32 ? 4 : 8;
  if (h % vec) return fail(PMC_ERR_INVALID, "layernorm: h=%d must be a multiple of %d", h, vec);
  if (!x || !gain || !bias || !y || !mean || !rstd) return fail(PMC_ERR_INVALID, "layernorm: NULL pointer");
  if (!aligned16(x) || !aligned16(gain) || !aligned16(bias) || !aligned16(y) || (x_copy && !aligned16(x_copy)))
    return fail(PMC_ERR_INVALID, "layernorm: pointers must be 16-byte aligned");
  if (dtype == PMC_F32) return ln_fwd_t<float>(st, rows, h, x, gain, bias, eps, y, mean, rstd, x_copy);
  if (dtype == PMC_BF16) return ln_fwd_t<bf16_t>(st, rows, h, x, gain, bias, eps, y, mean, rstd, x_copy);
  return fail(PMC_ERR_INVALID, "layernorm: bad dtype %d", dtype);
}

size_t layernorm_backward_scratch_floats(int rows, int h) {
  // Bound over both element types: at most one workgroup per row and kLnBwdMaxBlocks in all.
  return (size_t)ln_bwd_blocks(rows, 1) * 2 * h;
}

// Larger copies are launches of their own: their workgroups would wait for those that they share the launch with, and move their
// bytes no faster.  12.6 MB (q|k|v of 1024 tokens of hidden 2048) by themselves 6.1 us, riding along 1.8 (a step of two layers 1140 -> 1132).
bool copy_rides_along(int dtype, int rows, int cols) { return (size_t)rows * cols * (dtype == PMC_F32 ? 4 : 2) <= 16u << 20; }

int check_copy(int dtype, const RowCopy& copy) {
  const int vec = dtype == PMC_F32 ? 4 : 8;
  if (copy.cols && (copy.cols < 0 || !copy.src || !copy.dst || !aligned16(copy.src) || !aligned16(copy.dst) || copy.cols % vec || copy.ld_src % vec ||
                    copy.ld_dst % vec || copy.ld_src < copy.cols || copy.ld_dst < copy.cols))
    return fail(PMC_ERR_INVALID, "rows to copy: %d columns, pitches %d and %d, must be multiples of %d and 16-byte aligned", copy.cols, copy.ld_src,
                copy.ld_dst, vec);
  return PMC_OK;
}

int layernorm_backward_reduce(hipStream_t st, int h, const LnPartialJobs& jobs, int dtype, int rows, RowCopy copy) {
  if (jobs.count < 1 || jobs.count > LnPartialJobs::kMax) return fail(PMC_ERR_INVALID, "layernorm_backward_reduce: %d jobs", jobs.count);
  const bool f32 = dtype == PMC_F32;
  if (int rc = check_copy(dtype, copy)) return rc;
  const int copying = f32 ? copy_blocks<float>(copy, rows, kSumWaves * 64) : copy_blocks<bf16_t>(copy, rows, kSumWaves * 64);
  sum_partials_kernel<<<dim3((2 * h + 63) / 64 * jobs.count + copying), dim3(kSumWaves * 64), 0, st>>>(jobs, 2 * h, h, (size_t)2 * h, rows, f32, copy);
  PMC_LAUNCH_CHECK("layernorm_backward reduce");
  return PMC_OK;
}

int layernorm_backward(hipStream_t st, int dtype, int rows, int h, const void* dy, const void* x, const void* gain,
                       const float* mean, const float* rstd, const void* resid, void* dx, float* dgain, float* dbias,
                       float* partial, LnPartialJobs* defer, RowCopy copy) {
  if (rows <= 0 || h <= 0) return fail(PMC_ERR_INVALID, "layernorm_backward: rows=%d h=%d", rows, h);
  const int vec = dtype == PMC_F32 ? 4 : 8;
  if (h % vec) return fail(PMC_ERR_INVALID, "layernorm_backward: h=%d must be a multiple of %d", h, vec);
  if (!dy || !x || !gain || !mean || !rstd || !dx || !dgain || !dbias || !partial)
    return fail(PMC_ERR_INVALID, "layernorm_backward: NULL pointer");
  if (!aligned16(dy) || !aligned16(x) || !aligned16(gain) || !aligned16(dx) || (resid && !aligned16(resid)))
    return fail(PMC_ERR_INVALID, "layernorm_backward: pointers must be 16-byte aligned");
  if (int rc = check_copy(dtype, copy)) return rc;
  if (dtype == PMC_F32) return ln_bwd_t<float>(st, rows, h, dy, x, gain, mean, rstd, resid, dx, dgain, dbias, partial, defer, copy);
  if (dtype == PMC_BF16) return ln_bwd_t<bf16_t>(st, rows, h, dy, x, gain, mean, rstd, resid, dx, dgain, dbias, partial, defer, copy);
  return fail(PMC_ERR_INVALID, "layernorm_backward: bad dtype %d", dtype);
}

size_t layernorm_backward_static_scratch_bytes() { return kStaticScratchBytes; }

int layernorm_backward_static(hipStream_t st, int dtype, int rows, int h, const void* dy, const void* x, const void* gain,
                              const float* mean, const float* rstd, const void* resid, void* dx, float* dgain,
                              float* dbias) {
  if (rows <= 0 || h <= 0) return fail(PMC_ERR_INVALID, "layernorm_backward_static: rows=%d h=%d", rows, h);
  const size_t need = layernorm_backward_scratch_floats(rows, h) * sizeof(float);
  if (need > kStaticScratchBytes)
    return fail(PMC_ERR_NOMEM, "layernorm_backward_static: rows=%d x h=%d needs %zu bytes of scratch, the built-in array holds %zu",
                rows, h, need, kStaticScratchBytes);
  // The array has its own address on every GPU: looked up once per device, with that device current.
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* base[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(PMC_ERR_HIP, "layernorm_backward_static: cannot tell the current device");
  float* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!base[dev]) {
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p)
        return fail(PMC_ERR_HIP, "layernorm_backward_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
      base[dev] = static_cast<float*>(p);
    }
    ptr = base[dev];
  }
  // every workgroup overwrites its whole row of partials before the reduction reads it: nothing
  // of the previous call's contents is read, nothing has to be cleared
  return layernorm_backward(st, dtype, rows, h, dy, x, gain, mean, rstd, resid, dx, dgain, dbias, ptr, nullptr);
}

int column_sums(hipStream_t st, int dtype, int rows, ColumnSumJobs jobs) {
  if (rows <= 0 || jobs.count < 1 || jobs.count > 4) return fail(PMC_ERR_INVALID, "column_sum: rows=%d jobs=%d", rows, jobs.count);
  if (dtype != PMC_F32 && dtype != PMC_BF16) return fail(PMC_ERR_INVALID, "column_sum: bad dtype %d", dtype);
  const int vec = dtype == PMC_F32 ? 4 : 8;
  int blocks = 0;
  for (int j = 0; j < jobs.count; ++j) {
    const int n = jobs.n[j], lda = jobs.lda[j];
    if (n <= 0 || n % vec || lda % vec || lda < n)
      return fail(PMC_ERR_INVALID, "column_sum: n=%d lda=%d must be multiples of %d", n, lda, vec);
    if (!jobs.a[j] || !jobs.out[j] || !aligned16(jobs.a[j])) return fail(PMC_ERR_INVALID, "column_sum: bad pointer");
    jobs.first_block[j] = blocks;
    blocks += (n + 63) / 64;
  }
  for (int j = jobs.count; j < 5; ++j) jobs.first_block[j] = blocks;
  if (dtype == PMC_F32) colsum_kernel<float><<<dim3(blocks), dim3(256), 0, st>>>(rows, jobs);
  else colsum_kernel<bf16_t><<<dim3(blocks), dim3(256), 0, st>>>(rows, jobs);
  PMC_LAUNCH_CHECK("column_sum");
  return PMC_OK;
}

// Tiles of bm x bn and the column-sum workgroups of a W pass in one launch.
void wgrad_batch_layout(WgradBatchParams& p, int bm, int bn, int threads) {
  const int sum_cols = 64 * (threads / 256);
  int tiles = 0, sums = 0;
  for (int j = 0; j < 4; ++j) {
    p.first_tile[j] = tiles;
    p.first_sum[j] = sums;
    p.tiles_n[j] = (p.w.N[j] + bn - 1) / bn;
    tiles += p.tiles_n[j] * ((p.w.M[j] + bm - 1) / bm);
    sums += (p.w.N[j] + sum_cols - 1) / sum_cols;
  }
  p.first_tile[4] = tiles;
  p.first_sum[4] = sums;
  p.sum_blocks = (sums * p.w.layers + 7) & ~7;  // whole rounds over the 8 XCDs, so that a tile's XCD is its id modulo 8
  p.group_m = bm >= 256 ? 4 : 8;
}

int column_sum(hipStream_t st, int dtype, int rows, int n, const void* a, int lda, float* out) {
  ColumnSumJobs jobs = {};
  jobs.count = 1;
  jobs.a[0] = a;
  jobs.out[0] = out;
  jobs.n[0] = n;
  jobs.lda[0] = lda;
  return column_sums(st, dtype, rows, jobs);
}

int copy_rows(hipStream_t st, int dtype, int rows, int cols, const void* src, int ld_src, void* dst, int ld_dst) {
  const int vec = dtype == PMC_F32 ? 4 : 8;
  if (rows <= 0 || cols <= 0 || cols % vec || ld_src % vec || ld_dst % vec)
    return fail(PMC_ERR_INVALID, "copy_rows: bad shape rows=%d cols=%d", rows, cols);
  if (!aligned16(src) || !aligned16(dst)) return fail(PMC_ERR_INVALID, "copy_rows: pointers must be 16-byte aligned");
  const size_t total = (size_t)rows * (cols / vec);
  int blocks = (int)((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (dtype == PMC_F32) copy_rows_kernel<float><<<dim3(blocks), dim3(256), 0, st>>>(rows, cols / vec, (const float*)src, ld_src, (float*)dst, ld_dst);
  else copy_rows_kernel<bf16_t><<<dim3(blocks), dim3(256), 0, st>>>(rows, cols / vec, (const bf16_t*)src, ld_src, (bf16_t*)dst, ld_dst);
  PMC_LAUNCH_CHECK("copy_rows");
  return PMC_OK;
}

}  // namespace k
}  // namespace pmc
