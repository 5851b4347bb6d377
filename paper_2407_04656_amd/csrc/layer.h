// What the whole-layer calls of layer.hip share with the translation units of the single steps.  Not part of the C ABI.
#pragma once
#include <initializer_list>

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

// The tables that lz_ffn_tiles builds in a workspace; none if the call would be refused.
TileSpecs ffn_tables(const lz_shape* shape, void* ws, size_t ws_bytes);

// The tensors of lz_ffn_forward_train and of lz_ffn_backward (_accumulate).  Which kernels serve a call, and so which tables it reads,
// hangs on their alignment: tables built ahead of the call and the call itself ask the same struct.
struct FfnTrain {
  const void *xp, *w1, *w2;
  void *z, *h, *yp;
  bool aligned() const { return all16({xp, w1, w2, z, h, yp}); }
  static bool all16(std::initializer_list<const void*> tensors) {
    for (const void* t : tensors)
      if (((uintptr_t)t & 15) != 0) return false;
    return true;
  }
};
struct FfnBackward {
  const void *dyp, *xp, *z, *h, *w1, *w2;
  void *dxp, *dw1, *dw2;
  bool aligned() const { return FfnTrain::all16({dyp, xp, z, h, w1, w2, dxp, dw1, dw2}); }
};

// The tables that ffn_forward_train reads; none if the call would be refused.
TileSpecs train_tables(const lz_shape* shape, const FfnTrain& t, void* ws, size_t ws_bytes);
// lz_ffn_forward_train, its tables built already or not.
int32_t ffn_forward_train(const lz_shape* shape, const FfnTrain& t, const int32_t* slot_offsets, void* ws, size_t ws_bytes,
                          bool tables_built, void* stream);

// The tables of a whole pass's ffn_backward, where they can be built beside the combine backward; none if not, or if refused.
TileSpecs backward_tables(const lz_shape* shape, const FfnBackward& t, void* ws, size_t ws_bytes, bool accumulate);
// lz_combine_backward, in the same launch lz_route_backward (gate) and the tables.
int32_t combine_backward_with(const void* dy, const lz_shape* shape, const lz_layer_buffers& b, bool gate, const TileSpecs& tables,
                              void* stream);
// lz_ffn_backward, lz_ffn_backward_accumulate, their tables built already or not; in_pass: as part of a whole backward pass.
int32_t ffn_backward(const lz_shape* shape, const FfnBackward& t, const int32_t* slot_offsets, bool accumulate, void* ws, size_t ws_bytes,
                     bool tables_built, bool in_pass, void* stream);
// lz_reduce_replica_grads_dtype of both matrices, of elems1 and elems2 a slot, in one launch where both are whole 16-byte pieces.
int32_t reduce_pair(const lz_shape* shape, const lz_layer_buffers& b, int64_t elems1, int64_t elems2, void* stream);

}  // namespace lz
