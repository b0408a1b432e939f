// Chooses the attention kernels for a storage type and checks the shapes they assume.
#include "kernels.h"

namespace pmc {
namespace k {

int attention_forward_f32(hipStream_t st, int dtype, int batch, int seq, int heads, int dh, int causal,
                             const void* qkv, void* o, float* lse);
int attention_backward_f32(hipStream_t st, int dtype, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o,
                           const float* lse, const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta);

int attention_forward_mfma(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, void* o,
                           float* lse);
int attention_backward_mfma(hipStream_t st, int batch, int seq, int heads, int dh, int causal, const void* qkv, const void* o,
                            const float* lse, const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta);

namespace {
// bf16 storage with a head size that is a multiple of 8 (up to 128) runs on the matrix cores;
// everything else (fp32 mode, other head sizes) on the kernels of the fp32 matrix instruction.
bool use_mfma(int dtype, int head_dim) { return dtype == PMC_BF16 && head_dim >= 8 && head_dim <= 128 && head_dim % 8 == 0; }
size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
size_t elem(int dtype) { return dtype == PMC_F32 ? 4 : 2; }
}  // namespace

int attention_forward(hipStream_t st, int dtype, int batch, int seq, int heads, int head_dim, int causal,
                      const void* qkv, void* o, float* lse) {
  if (!qkv || !o || !lse) return fail(PMC_ERR_INVALID, "attention_forward: NULL pointer");
  if (dtype != PMC_F32 && dtype != PMC_BF16) return fail(PMC_ERR_INVALID, "attention_forward: bad dtype %d", dtype);
  if (use_mfma(dtype, head_dim)) return attention_forward_mfma(st, batch, seq, heads, head_dim, causal, qkv, o, lse);
  return attention_forward_f32(st, dtype, batch, seq, heads, head_dim, causal, qkv, o, lse);
}

size_t attention_backward_scratch_bytes(int dtype, int batch, int seq, int heads, int head_dim) {
  const size_t tokens = (size_t)batch * seq;
  return align256(tokens * heads * head_dim * elem(dtype)) + align256(tokens * heads * sizeof(float));
}

// Where both halves of the backward pass go out as one launch, by w = 64-row workgroups of one half.
//   1: 8 waves to a workgroup, one workgroup to a compute unit; as long as each half has at most one per unit (w <= 256).
//   2: 4 waves, two to a unit; for one block of rows, where there is nothing to split over more waves, and for short sequences
//      beyond w = 128, where two rounds of the larger ones meet.
// Otherwise two launches are faster, whose workgroups need less LDS and fewer registers each.  us of 1 / 2 / two launches, without
// the copy that in-place results need, heads of 128, causal unless said: 16 heads x 512 tokens 21.8 / 29.1 / 30; 16 x 1000 (w 256) 45 / 53 / 50;
// 16 x 64 11.4 / 9.6 / 16; 128 x 128 (w 256) 22.9 / 15.8 / 25; 64 x 192 (w 192) 22.7 / 18.2; 128 x 192 (w 384) - / 25.9 / 29.5, not causal
// 30.2 / 30.5; 64 x 512 (w 512) - / 43 / 51, not causal 65 / 54; 16 x 2048 (w 512) - / 122 / 106.  fp32 (16-row blocks): 8 heads of 64, 512
// tokens 31 in one, 36 in two; 16 heads 57 and 50.
int attention_merged(int batch, int seq, int heads, int head_dim, int causal) {
  const int64_t w = (int64_t)((seq + 63) / 64) * heads * batch;
  if (seq <= 64) return w <= 512 ? 2 : 0;
  if (w > 128 && w <= (causal ? 512 : 384) && seq <= (causal && w > 256 ? 512 : 256)) return 2;
  return w <= 256 ? 1 : 0;
}
bool attention_merged_f32(int batch, int seq, int heads) { return (int64_t)((seq + 15) / 16) * heads * batch <= 256; }

int attention_backward_kept_columns(int dtype, int batch, int seq, int heads, int head_dim, int causal) {
  const bool merged =
      use_mfma(dtype, head_dim) ? attention_merged(batch, seq, heads, head_dim, causal) > 0 : attention_merged_f32(batch, seq, heads);
  return merged ? 3 * heads * head_dim : 0;
}

namespace {
int backward(hipStream_t st, int dtype, int batch, int seq, int heads, int head_dim, int causal, const void* qkv, const void* o,
             const float* lse, const void* d_o, void* dqkv, void* dq, int ld_dq, float* delta) {
  if (use_mfma(dtype, head_dim))
    return attention_backward_mfma(st, batch, seq, heads, head_dim, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
  return attention_backward_f32(st, dtype, batch, seq, heads, head_dim, causal, qkv, o, lse, d_o, dqkv, dq, ld_dq, delta);
}
}  // namespace

int attention_backward(hipStream_t st, int dtype, int batch, int seq, int heads, int head_dim, int causal,
                       const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, void* scratch) {
  if (!qkv || !o || !lse || !d_o || !dqkv || !scratch) return fail(PMC_ERR_INVALID, "attention_backward: NULL pointer");
  if (dtype != PMC_F32 && dtype != PMC_BF16) return fail(PMC_ERR_INVALID, "attention_backward: bad dtype %d", dtype);
  const size_t tokens = (size_t)batch * seq;
  const int h = heads * head_dim;
  const int vec = dtype == PMC_F32 ? 4 : 8;
  if (h % vec) return fail(PMC_ERR_INVALID, "attention_backward: hidden %d must be a multiple of %d", h, vec);
  char* dq_stage = (char*)scratch;
  float* delta = (float*)(dq_stage + align256(tokens * h * elem(dtype)));
  const size_t bytes = tokens * 3 * h * elem(dtype);
  if ((const char*)qkv + bytes <= (const char*)dqkv || (const char*)dqkv + bytes <= (const char*)qkv)
    return backward(st, dtype, batch, seq, heads, head_dim, causal, qkv, o, lse, d_o, dqkv, dqkv, 3 * h, delta);
  // In place.  dq goes to the staging buffer because q is still needed by the dk/dv kernel, which reads k, v
  // from qkv and writes dk, dv to the same columns of dqkv (a key tile is read only by the workgroup that later overwrites it).
  if (int rc = backward(st, dtype, batch, seq, heads, head_dim, causal, qkv, o, lse, d_o, dqkv, dq_stage, h, delta)) return rc;
  return copy_rows(st, dtype, (int)tokens, h, dq_stage, h, dqkv, 3 * h);
}

}  // namespace k
}  // namespace pmc
