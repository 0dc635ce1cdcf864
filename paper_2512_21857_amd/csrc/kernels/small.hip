// Tiny device-side setters: scalars and index arrays are written by kernels that take the
// values as arguments, so a cycle needs no host-to-device copies.
#include "../launch.h"

namespace adt {

__global__ void set_i32_kernel(int32_t* dst, SmallI32 vals, int count) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = vals.v[i];
}

__global__ void fill_pairs_kernel(int32_t* dst, int rows, int lo, int hi) {
  for (int i = threadIdx.x; i < rows; i += blockDim.x) {
    dst[i * 2] = lo;
    dst[i * 2 + 1] = hi;
  }
}

// The tree of a root alone, whose successor may be any id of [lo, hi): every array of the tree in
// one launch (six small ones had taken 16 us of a prefill's trace).
__global__ void root_tree_kernel(int token_id, int L, int lo, int hi, int n_max, int32_t* n, int32_t* parent,
                                 int32_t* token, int32_t* depth, int32_t* pos, float* score, int32_t* allowed_rows,
                                 uint64_t* mask) {
  for (int i = threadIdx.x; i < n_max; i += blockDim.x) {
    mask[i * 2] = i == 0 ? 1 : 0;
    mask[i * 2 + 1] = 0;
    depth[i] = 0;
  }
  if (threadIdx.x == 0) {
    *n = 1;
    parent[0] = -1;
    token[0] = token_id;
    pos[0] = L;
    score[0] = 0.f;
    allowed_rows[0] = lo;
    allowed_rows[1] = hi;
  }
}

// Rows of a prompt of P tokens: positions 0.., the masks of a chain, and for the draft the feature of
// the row before (none for row 0).
__global__ void prompt_rows_kernel(int P, int32_t* pos, int32_t* fsrc, uint64_t* mask) {
  for (int i = threadIdx.x; i < P; i += blockDim.x) {
    pos[i] = i;
    fsrc[i] = i - 1;
    const int b = i + 1;
    mask[i * 2] = b >= 64 ? ~0ull : ((1ull << b) - 1);
    mask[i * 2 + 1] = b <= 64 ? 0ull : (b >= 128 ? ~0ull : ((1ull << (b - 64)) - 1));
  }
}

// Positions, successor allowed ranges and zero scores of a caller-supplied tree.
__global__ void tree_rows_kernel(const int32_t* depth, const int32_t* n_nodes, int n_max, int L, int P, int n_image,
                                 const int32_t* allowed_img, int32_t* pos, int32_t* allowed_rows, float* score) {
  const int n = min(*n_nodes, n_max);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    pos[i] = L + depth[i];
    int cell = L + depth[i] + 1 - P;
    cell = cell < 0 ? 0 : (cell >= n_image ? n_image - 1 : cell);
    allowed_rows[i * 2] = allowed_img[cell * 2];
    allowed_rows[i * 2 + 1] = allowed_img[cell * 2 + 1];
    score[i] = 0.f;
  }
}

// Row indices of a caller-supplied draft-logit table: (depth * 131 + token) mod rows.
__global__ void table_rows_kernel(const int32_t* tok, int count, int depth, int rows, int32_t* idx) {
  for (int i = threadIdx.x; i < count; i += blockDim.x) idx[i] = (int)(((int64_t)depth * 131 + tok[i]) % rows);
}

adt_status launch_table_rows(const int32_t* tok, int count, int depth, int rows, int32_t* idx, hipStream_t st) {
  table_rows_kernel<<<1, 128, 0, st>>>(tok, count, depth, rows, idx);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}

adt_status launch_set_i32(int32_t* dst, const SmallI32& vals, int count, hipStream_t st) {
  ADT_CHECK_ARG(count >= 0 && count <= 32, ADT_E_ARG, "set_i32: count %d", count);
  if (count == 0) return ADT_OK;
  set_i32_kernel<<<1, 32, 0, st>>>(dst, vals, count);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}
adt_status launch_fill_pairs(int32_t* dst, int rows, int lo, int hi, hipStream_t st) {
  fill_pairs_kernel<<<1, 128, 0, st>>>(dst, rows, lo, hi);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}
adt_status launch_root_tree(int token_id, int L, int lo, int hi, int n_max, int32_t* n, int32_t* parent, int32_t* token,
                            int32_t* depth, int32_t* pos, float* score, int32_t* allowed_rows, uint64_t* mask,
                            hipStream_t st) {
  root_tree_kernel<<<1, 128, 0, st>>>(token_id, L, lo, hi, n_max, n, parent, token, depth, pos, score, allowed_rows, mask);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}
adt_status launch_prompt_rows(int P, int32_t* pos, int32_t* fsrc, uint64_t* mask, hipStream_t st) {
  prompt_rows_kernel<<<1, 128, 0, st>>>(P, pos, fsrc, mask);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}
adt_status launch_tree_rows(const int32_t* depth, const int32_t* n_nodes, int n_max, int L, int P, int n_image,
                            const int32_t* allowed_img, int32_t* pos, int32_t* allowed_rows, float* score,
                            hipStream_t st) {
  tree_rows_kernel<<<1, 128, 0, st>>>(depth, n_nodes, n_max, L, P, n_image, allowed_img, pos, allowed_rows, score);
  ADT_LAUNCH_CHECK();
  return ADT_OK;
}

}  // namespace adt
