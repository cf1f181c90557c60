// Arguments of the launch that takes blocks of views through the whole Sparse Part (rows.hip).
#pragma once

#include "gear_internal.hpp"

namespace gear {

constexpr int kRowsThreads = 512, kRowsWaves = kRowsThreads / kWave;

struct RowsBuf {       // an activation tile in LDS
  int at, stride;      // bytes; of a row
};
struct RowsLayer {     // a hidden layer
  const void *w, *wt;  // operands in operand order (prep.hip): W [out x in] and its transpose
  const float *bias;
  void *h, *delta;     // [B x out]
  float *colsum;       // [blocks x out] column sums of delta
  int in, out;
  RowsBuf buf;
};
struct RowsArgs {
  int B, nnz, d, D, F, L, H;   // H: width of the last hidden layer
  int emb_bf16, dfv_bf16, scratch, logit_w;
  int64_t n_users, n_urls, n_images;
  const int32_t *user_id, *url_id, *img_off, *img_id;
  const float *label;
  int32_t *occ_view;              // [nnz] left for the bookkeeping: the view of every occurrence,
  float *occ_scale;               // and one over its number of images
  const void *user_emb, *url_emb, *dfv;
  const float *w_last, *b_last;   // the logit layer, fp32
  void *x;                        // [B x F]
  float *logits, *dz, *dx_emb;
  void *dx_dfv;
  float *part_w, *part_b, *part_loss;   // sums of a block: [blocks x H], [blocks], [blocks]
  RowsBuf x_buf;
  RowsLayer layer[GEAR_MAX_LAYERS - 1];
};

// parts of a block's rows that a column is added in by as many threads (a power of two), for a quarter of the columns each
__host__ __device__ inline int rows_split(int rows, int owners) {
  int split = 1;
  while (2 * split <= rows && 2 * split * owners <= kRowsThreads) split *= 2;
  return split;
}

// How a step goes about it: decided by sizes alone.
struct RowsPlan {
  bool direct;                         // the blocks read the weights as they are, and the step has no prologue
  int rows, blocks;                    // views of a block; blocks of the batch
  int lds, room;                       // bytes of LDS; items of the sorts in them
  int digit_bits;                      // of the sorts that run beside
  int parts_log2[kMaxProblems];        // of the lists of ids (local_group.hpp)
  int value_bits[kMaxProblems];
  size_t colsum;                       // workspace offset of the column sums of the deltas below the last
  size_t colsum_at[GEAR_MAX_LAYERS];   // floats before those that layer l's product leaves
};
// `local`: with the grouping (else the ids are sorted elsewhere).  false: layer by layer.
bool plan_rows(const gear_config &cfg, const Layout &lay, int B, int nnz, bool local, RowsPlan *plan);
LogitSums rows_sums(const RowsPlan &plan, const float *partials, int H);
BlockSums block_sums_of(const RowsPlan &plan, const Layout &lay, const gear_batch &b, char *ws);   // the same sums, from the launches of the layers
LocalResult local_result(const RowsPlan &plan, const GroupBatch &gb, int nnz, int ready_cap);
LocalTask local_task(const RowsPlan &plan, const GroupBatch &gb, const PlanArgs &args, const ViewCheck &views, int32_t *failed, float *loss);
void local_zero_list(const GroupBatch &gb, ZeroList *z);
hipError_t launch_rows(const gear_config &cfg, const Layout &lay, const RowsPlan &plan, const gear_batch &b, const gear_tables &t,
                       const void *dfv_cache, char *ws, const LocalTask &local, hipStream_t s);

}  // namespace gear
