// Host-callable launchers of the HIP kernels.  Every launcher validates what its kernel assumes
// about shapes and alignment, enqueues on `stream` and returns a pmc_status.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "pmc_internal.h"

namespace pmc {
namespace k {

// One-time reservation of a kernel's dynamic LDS, reachable from several host threads at once: the
// flag is atomic and the attribute call is idempotent, so a race at first use only repeats the call.
template <typename Kern>
int reserve_lds(Kern kern, size_t bytes, std::atomic<bool>& done, const char* what) {
  if (done.load(std::memory_order_acquire)) return PMC_OK;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return fail(PMC_ERR_HIP, "%s: cannot reserve %zu bytes of LDS: %s", what, bytes, hipGetErrorString(e));
  done.store(true, std::memory_order_release);
  return PMC_OK;
}

struct GemmArgs {
  int dtype = PMC_BF16;
  bool trans_a = false, trans_b = false;
  int M = 0, N = 0, K = 0;
  const void* A = nullptr;
  int lda = 0;
  const void* B = nullptr;
  int ldb = 0;
  void* C = nullptr;
  int ldc = 0;
  int epilogue = PMC_EPI_NONE;
  const void* bias = nullptr;   // [N], storage type
  const void* resid = nullptr;  // [M, N], pitch ldc
  void* aux = nullptr;          // [M, N], pitch ldc
  void* ws = nullptr;           // optional scratch for split-K partial products (256-byte aligned)
  size_t ws_bytes = 0;
};

// Weight gradients of several queued microbatches as ONE product: C[M,N] (fp32) += sum_i A_i^T . B_i
// with A_i stored [K,M] (pitch lda) and B_i stored [K,N] (pitch ldb), bf16.  M, N, K multiples of 8.
struct GroupedWgradArgs {
  int M = 0, N = 0, K = 0;  // K of ONE piece
  int count = 0;            // 1 .. PMC_MAX_QUEUED_W pieces
  const void* A[PMC_MAX_QUEUED_W] = {};
  const void* B[PMC_MAX_QUEUED_W] = {};
  int lda = 0, ldb = 0;
  float* C = nullptr;
  int ldc = 0;
};
int gemm_bf16_grouped_wgrad(hipStream_t stream, const GroupedWgradArgs& a);

// The W pass of one microbatch (fp32, bf16) or of several queued ones (bf16) as ONE launch: for every layer the four
// products C_j[M_j,N_j] (fp32) += sum over the pieces of A_j^T . B_j and the four bias gradients bias_j[n] += column sums
// of B_j.  Every operand of piece i lies at piece[i] + its offset, A_j stored [K,M_j] and B_j stored [K,N_j] without
// padding, C_j without padding.
struct WgradBatchArgs {
  static constexpr int kMaxLayers = 8;
  struct Layer {
    size_t a[4], b[4];  // byte offsets
    float* c[4];
    float* bias[4];
  };
  Layer layer[kMaxLayers];
  const char* piece[PMC_MAX_QUEUED_W];
  int M[4], N[4];
  int K = 0, layers = 0, pieces = 0;
};
// Kernel argument of the batch: the products of a layer are cut into tiles numbered one product after the other (first_tile),
// layer after layer; the first sum_blocks workgroups (64 columns of a bias gradient to 256 threads, first_sum per layer) do the column sums.
struct WgradBatchParams {
  WgradBatchArgs w;
  int tiles_n[4], first_tile[5], first_sum[5];
  int group_m, sum_blocks;
};
void wgrad_batch_layout(WgradBatchParams& p, int bm, int bn, int threads);
int wgrad_batch_shape(int dtype, const WgradBatchArgs& a);  // -1: not in one launch
int wgrad_batch(hipStream_t stream, int dtype, const WgradBatchArgs& a, int shape);
int gemm_bf16_wgrad_batch_shape(const WgradBatchArgs& a);
int gemm_bf16_wgrad_batch(hipStream_t stream, const WgradBatchArgs& a, int shape);

// Scratch for the plan that this product gets where there is room for any (0: it is not split).
size_t gemm_scratch_bytes(GemmArgs a);

// What gemm() launches for a product: host arithmetic only, so that the rules can be tested without a GPU.
// kernel: in bf16 tiles of a shape (see gemm_bf16.hip), the two weight-gradient kernels, the general kernel, or partial
// products over `splits` ranges of K (+ 2: in large tiles, + 5: in 64x64 ones); kPlanF32 + F32Shape in fp32 (-1: refused, more tiles than a launch holds).
enum { kPlanTile = 0, kPlanPersistent = 20, kPlanPair = 21, kPlanGeneral = 22, kPlanSplit = 30, kPlanF32 = 100 };
struct GemmPlan {
  int kernel, splits, k_tiles_per_split;
};
GemmPlan gemm_f32_plan(const GemmArgs& a);
GemmPlan gemm_bf16_plan(const GemmArgs& a);
bool gemm_bf16_split_own_xcds(bool tb, int tiles_m, int M, int N, int K, int splits);  // partial products: a range of K has XCDs of its own
bool gemm_bf16_k_groups(int M, int N, int K);  // 128x128 tiles of the F and B layouts: eight waves in two K groups (else four)

int gemm(hipStream_t stream, const GemmArgs& a);
int gemm_f32(hipStream_t stream, const GemmArgs& a);
int gemm_bf16(hipStream_t stream, const GemmArgs& a);

int layernorm_forward(hipStream_t stream, int dtype, int rows, int h, const void* x, const void* gain,
                      const void* bias, float eps, void* y, float* mean, float* rstd, void* x_copy);
// partial: fp32 scratch of layernorm_backward_scratch_floats(rows, h) floats.  The kernel leaves one
// row of gain/bias-gradient partial sums per workgroup there; a second, tiny kernel adds them into
// dgain/dbias.  With `defer` given that second step is only noted down (the scratch must then stay
// untouched, one region per call) and layernorm_backward_reduce runs all noted reductions in ONE
// launch: a backward pass has two LayerNorms per layer and pays for one such launch, not for 2 L.
struct LnPartialJobs {
  static constexpr int kMax = 16;
  const float* partial[kMax];
  float* dgain[kMax];
  float* dbias[kMax];
  int parts[kMax];
  int count = 0;
};
size_t layernorm_backward_scratch_floats(int rows, int h);
// Rows that a launch copies beside its own work, whose tensors must not overlap them: dst[row][0..cols) = src[row][0..cols), columns
// and pitches in whole 16-byte chunks.
struct RowCopy {
  const void* src = nullptr;
  int ld_src = 0;
  void* dst = nullptr;
  int ld_dst = 0, cols = 0;
};
bool copy_rides_along(int dtype, int rows, int cols);  // else it is better off as a launch of its own (copy_rows)
int layernorm_backward(hipStream_t stream, int dtype, int rows, int h, const void* dy, const void* x,
                       const void* gain, const float* mean, const float* rstd, const void* resid, void* dx,
                       float* dgain, float* dbias, float* partial, LnPartialJobs* defer = nullptr, RowCopy copy = {});
int layernorm_backward_reduce(hipStream_t stream, int h, const LnPartialJobs& jobs, int dtype = PMC_F32, int rows = 0, RowCopy copy = {});
// As layernorm_backward with the partial sums in a device array built into the library (no workspace,
// no allocation); PMC_ERR_NOMEM when layernorm_backward_scratch_floats(rows, h) floats do not fit in
// layernorm_backward_static_scratch_bytes().
size_t layernorm_backward_static_scratch_bytes();
int layernorm_backward_static(hipStream_t stream, int dtype, int rows, int h, const void* dy, const void* x,
                              const void* gain, const float* mean, const float* rstd, const void* resid, void* dx,
                              float* dgain, float* dbias);

int attention_forward(hipStream_t stream, int dtype, int batch, int seq, int heads, int head_dim, int causal,
                      const void* qkv, void* o, float* lse);
// scratch: delta fp32 [batch, heads, seq], then, where dqkv overlaps qkv (in_place), dq staging [batch*seq, heads*head_dim] in
// the storage type.
size_t attention_backward_scratch_bytes(int dtype, int batch, int seq, int heads, int head_dim, bool in_place = true);
int attention_backward(hipStream_t stream, int dtype, int batch, int seq, int heads, int head_dim, int causal,
                       const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                       void* scratch);
// Columns of qkv (3 heads head_dim or 0) that a caller who wants dqkv in qkv's place is better off copying elsewhere first, to call
// attention_backward from the copy: with qkv and dqkv apart few blocks run as one launch.
int attention_backward_kept_columns(int dtype, int batch, int seq, int heads, int head_dim, int causal);
int attention_merged(int batch, int seq, int heads, int head_dim, int causal);  // 0: two launches
bool attention_merged_f32(int batch, int seq, int heads, int causal);
// What a bf16 call on the matrix cores launches (host arithmetic only): the forward shape, the one-launch form of the backward pass apart from
// qkv (0: two launches) and the family of its two launches (see attn_mfma.hip).
void attention_mfma_plan(int batch, int seq, int heads, int head_dim, int causal, int* out);

// out[c] += sum over rows of a[row][c] (fp32 out), for up to four matrices of `rows` rows in one
// launch; first_block is filled in by column_sums.
struct ColumnSumJobs {
  const void* a[4];
  float* out[4];
  int n[4];
  int lda[4];
  int first_block[5];
  int count;
};
int column_sums(hipStream_t stream, int dtype, int rows, ColumnSumJobs jobs);
int column_sum(hipStream_t stream, int dtype, int rows, int n, const void* a, int lda, float* out);

int copy_rows(hipStream_t stream, int dtype, int rows, int cols, const void* src, int ld_src, void* dst, int ld_dst);

}  // namespace k
}  // namespace pmc
