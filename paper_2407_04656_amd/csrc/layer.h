// What the whole-layer calls of layer.hip share with the translation units of the single steps.  Not part of the C ABI.
#pragma once
#include "tiles.h"

namespace lz {

struct Dispatch {
  const lz_shape* shape;
  int32_t* topk_ids;  // written where the dispatcher routes, else read
  const int32_t *rank_tok_off, *slot_expert;
  int32_t *slot_counts, *slot_offsets, *pair_to_row, *row_to_pair, *Tej_opt, *D_opt, *status_opt;
  void* ws;
  size_t ws_bytes;
};

// lz_plan_dispatch, which also builds the listed tables, and, given logits (where plan_routes says that it can), routes first.
bool plan_routes(const lz_shape* shape);
int32_t plan_dispatch(const Dispatch& d, const float* logits, float* topk_gates, const TileSpecs& tables, hipStream_t st);

// The tables that lz_ffn_tiles, or lz_ffn_forward_train, builds in a workspace; none if the call would be refused.
TileSpecs ffn_tables(const lz_shape* shape, void* ws, size_t ws_bytes);
TileSpecs train_tables(const lz_shape* shape, const void* const* tensors, int n_tensors, void* ws, size_t ws_bytes);

// lz_ffn_forward_train, its tables built already or not.
int32_t ffn_forward_train(const void* xp, const int32_t* slot_offsets, const void* w1, const void* w2, const lz_shape* shape,
                          void* z, void* h, void* yp, void* ws, size_t ws_bytes, bool tables_built, void* stream);

// The tables of lz_ffn_backward (_accumulate), where they can be built beside the combine backward; none if not, or if refused.
TileSpecs backward_tables(const lz_shape* shape, const void* const* tensors, int n_tensors, void* ws, size_t ws_bytes, bool accumulate);
// lz_combine_backward, in the same launch lz_route_backward (gate) and the tables.
int32_t combine_backward_with(const void* dy, const lz_shape* shape, const lz_layer_buffers& b, bool gate, const TileSpecs& tables,
                              void* stream);
// lz_ffn_backward, lz_ffn_backward_accumulate, their tables built already or not; in_pass: as part of a whole backward pass.
int32_t ffn_backward(const void* dyp, const void* xp, const void* z, const void* h, const int32_t* slot_offsets, const void* w1,
                     const void* w2, const lz_shape* shape, void* dxp, void* dw1, void* dw2, bool accumulate, void* ws,
                     size_t ws_bytes, bool tables_built, bool in_pass, void* stream);
// lz_reduce_replica_grads_dtype of both matrices, of elems1 and elems2 a slot, in one launch where both are whole 16-byte pieces.
int32_t reduce_pair(const lz_shape* shape, const lz_layer_buffers& b, int64_t elems1, int64_t elems2, void* stream);

}  // namespace lz
