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

// Where both halves of the backward pass go out as one launch: as long as each half has at most one workgroup per compute unit.
// Beyond, two launches are faster, whose workgroups need less LDS and fewer registers each.  us of the one launch / of two, without
// the copy that in-place results need (bf16, causal): 16 heads of 64, 512 tokens 15.6 / 22; 16 of 128, 1024 tokens 44 / 50;
// 32 of 128, 4 x 256 tokens 49 / 48; 16 of 64, 2048 tokens 95 / 65; 8 of 128, 4096 tokens 242 / 165.  fp32 (16-row blocks): 8 heads of
// 64, 512 tokens 31 / 36; 16 heads 57 / 50.
bool attention_merged(int batch, int seq, int heads) { return (int64_t)((seq + 63) / 64) * heads * batch <= 256; }
bool attention_merged_f32(int batch, int seq, int heads) { return (int64_t)((seq + 15) / 16) * heads * batch <= 256; }

int attention_backward_kept_columns(int dtype, int batch, int seq, int heads, int head_dim) {
  const bool merged = use_mfma(dtype, head_dim) ? attention_merged(batch, seq, heads) : attention_merged_f32(batch, seq, heads);
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
