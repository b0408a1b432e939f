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

size_t attention_backward_scratch_bytes(int dtype, int batch, int seq, int heads, int head_dim, bool in_place) {
  const size_t tokens = (size_t)batch * seq;
  return align256(tokens * heads * sizeof(float)) + (in_place ? align256(tokens * heads * head_dim * elem(dtype)) : 0);
}

// Where both halves of the backward pass go out as one launch, by w = 64-row workgroups of one half.
//   1: 8 waves to a workgroup, one workgroup to a compute unit.  Up to w = 128 the workgroups of both halves fit the units at once; up to
//      256 they do not, and all but the causal ones, whose lengths differ, meet in two rounds that take longer than two launches.
//   2: 4 waves, two to a unit; for one block of rows, where there is nothing to split over more waves, and for short sequences
//      beyond w = 128.
// Otherwise two launches are faster, whose workgroups need less LDS and fewer registers each.  us of 1 / 2 / two launches in place with their copy,
// heads of 128: causal 16 heads x 512 tokens (w 128) 22.0 / 29.6 / 36.1, 16 x 1000 (w 256) 46 / 55 / 54, 5 x 3000 (w 235) 97 / 152 / 124, 16 x 64 11.2 / 9.5 / 18.1,
// 128 x 128 (w 256) 22.7 / 15.5 / 25.8, 64 x 192 (w 192) 22.5 / 17.7 / 27.1, 128 x 192 (w 384) 34.8 / 25.5 / 34.2, 64 x 512 (w 512) 57 / 43 / 52, 32 x 768 (w 384) 52 / 44 / 59,
// 16 x 2048 (w 512) 141 / 123 / 108; not causal 128 x 192 35.8 / 29.9 / 35.2, 16 x 1000 78 / 83 / 66, 5 x 3000 204 / 217 / 149.  Over 5220 calls (1 .. 64 heads of
// 40 .. 128, 1 .. 8 sequences of 8 .. 4096 tokens), with the copy of q|k|v that one launch needs in a pass: 0.59 of the time of two launches of one
// family per size in place, the rule that came before, and nowhere more than 2 % slower.
int attention_merged(int batch, int seq, int heads, int head_dim, int causal) {
  const int64_t w = (int64_t)((seq + 63) / 64) * heads * batch;
  if (seq <= 64) return w <= 512 ? 2 : 0;
  if (w <= 128) return 1;
  if (w <= 256) return seq <= (head_dim > 64 ? 256 : 128) ? 2 : causal || seq <= 256 ? 1 : 0;
  return (causal ? w <= 512 && seq <= 512 : w <= 384 && seq <= 256) ? 2 : 0;
}
// fp32, by 16-row workgroups: as kind 1.  us of one / two launches: causal 8 heads of 64 x 512 tokens (256 workgroups) 30 / 39, 16 x 512 57 / 53, 8 of 128 x 500 53 / 72;
// not causal 4 of 64 x 1000 (252) 82 / 66, 8 of 128 x 500 86 / 74, 32 of 64 x 100 (224) 15.6 / 18.2.
bool attention_merged_f32(int batch, int seq, int heads, int causal) {
  const int64_t w = (int64_t)((seq + 15) / 16) * heads * batch;
  return w <= (causal || seq <= 128 ? 256 : 128);
}

int attention_backward_kept_columns(int dtype, int batch, int seq, int heads, int head_dim, int causal) {
  const bool merged =
      use_mfma(dtype, head_dim) ? attention_merged(batch, seq, heads, head_dim, causal) > 0 : attention_merged_f32(batch, seq, heads, causal);
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
  float* delta = (float*)scratch;
  char* dq_stage = (char*)scratch + align256(tokens * heads * sizeof(float));
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
