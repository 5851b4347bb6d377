// The whole layer in one call: the steps of the single calls in their order, on the caller's buffers.  What a caller of small batches
// pays for is launches and calls (from Python a forward of 256 fp32 tokens, 20 in a row, takes 30 us of the host as five calls of seven
// launches, 23 to 24 as one of five): the dispatcher's launches also build the tables of the grouped GEMMs, and route where the batch is
// small enough for one workgroup.
#include "layer.h"

namespace {

thread_local const char* g_refused = "";

// rc, which `call` returned, or a launch that stands for it
int32_t of(const char* call, int32_t rc) {
  if (rc != LZ_OK) g_refused = call;
  return rc;
}

lz::Dispatch dispatch_of(const lz_shape* shape, const lz_layer_buffers& b) {
  return lz::Dispatch{shape, b.topk_ids, b.rank_tok_off, b.slot_expert, b.slot_counts, b.slot_offsets, b.pair_to_row, b.row_to_pair,
                      b.Tej_opt, b.D_opt, b.status_opt, b.plan_ws, b.plan_ws_bytes};
}

// lz_route, lz_plan_dispatch and `tables`
int32_t route_and_plan(const lz_shape* shape, const lz_layer_buffers& b, const float* logits, const TileSpecs& tables, void* stream) {
  if (!shape) return of("lz_route", LZ_ESHAPE);
  const bool in_plan = lz::plan_routes(shape) && logits && b.topk_ids && b.topk_gates;
  if (!in_plan) {
    const int32_t rc = of("lz_route", lz_route(logits, shape->T, shape->E, shape->k, b.topk_ids, b.topk_gates, stream));
    if (rc != LZ_OK) return rc;
  }
  return of("lz_plan_dispatch",
            lz::plan_dispatch(dispatch_of(shape, b), in_plan ? logits : nullptr, b.topk_gates, tables, (hipStream_t)stream));
}

// the FFN on tables that the dispatcher has built
int32_t ffn_on_tables(const lz_shape* shape, const lz_layer_buffers& b, const void* x, bool fused, void* stream) {
  if (!(fused ? x : b.xp) || !b.w1 || !b.w2 || !b.yp) return LZ_EINVAL;
  const int32_t rc = fused ? lz_ffn_up_gather(x, b.row_to_pair, b.w1, shape, b.ffn_ws, b.ffn_ws_bytes, stream)
                           : lz_ffn_up(b.xp, b.w1, shape, b.ffn_ws, b.ffn_ws_bytes, stream);
  return rc != LZ_OK ? rc : lz_ffn_down(b.w2, shape, b.yp, b.ffn_ws, b.ffn_ws_bytes, stream);
}

}  // namespace

extern "C" const char* lz_layer_refused(void) { return g_refused; }

extern "C" int32_t lz_layer_forward(const lz_shape* shape, const lz_layer_buffers* buffers, const float* logits, const void* x,
                                    int32_t fused, void* stream) {
  if (!buffers) return of("lz_layer_forward", LZ_EINVAL);
  const lz_layer_buffers& b = *buffers;
  const TileSpecs tables = lz::ffn_tables(shape, b.ffn_ws, b.ffn_ws_bytes);
  int32_t rc = route_and_plan(shape, b, logits, tables, stream);
  if (rc != LZ_OK) return rc;
  if (!fused && (rc = of("lz_permute_scatter", lz_permute_scatter(x, b.pair_to_row, shape, b.xp, stream))) != LZ_OK) return rc;
  if (tables.n > 0) rc = ffn_on_tables(shape, b, x, fused, stream);
  else  // no rows, or a workspace that is refused
    rc = fused ? lz_expert_ffn_gather(x, b.row_to_pair, b.slot_offsets, b.w1, b.w2, shape, b.yp, b.ffn_ws, b.ffn_ws_bytes, stream)
               : lz_expert_ffn(b.xp, b.slot_offsets, b.w1, b.w2, shape, b.yp, b.ffn_ws, b.ffn_ws_bytes, stream);
  if (of(fused ? "lz_expert_ffn_gather" : "lz_expert_ffn", rc) != LZ_OK) return rc;
  return of("lz_unpermute_combine", lz_unpermute_combine(b.yp, b.pair_to_row, b.topk_gates, shape, b.y, stream));
}

extern "C" int32_t lz_layer_forward_train(const lz_shape* shape, const lz_layer_buffers* buffers, const float* logits, const void* x,
                                          void* stream) {
  if (!buffers) return of("lz_layer_forward_train", LZ_EINVAL);
  const lz_layer_buffers& b = *buffers;
  const lz::FfnTrain ffn{b.xp, b.w1, b.w2, b.z, b.h, b.yp};
  const TileSpecs tables = lz::train_tables(shape, ffn, b.train_ws, b.train_ws_bytes);
  int32_t rc = route_and_plan(shape, b, logits, tables, stream);
  if (rc != LZ_OK) return rc;
  if ((rc = of("lz_permute_scatter", lz_permute_scatter(x, b.pair_to_row, shape, b.xp, stream))) != LZ_OK) return rc;
  rc = lz::ffn_forward_train(shape, ffn, b.slot_offsets, b.train_ws, b.train_ws_bytes, tables.n > 0, stream);
  if (of("lz_ffn_forward_train", rc) != LZ_OK) return rc;
  return of("lz_unpermute_combine", lz_unpermute_combine(b.yp, b.pair_to_row, b.topk_gates, shape, b.y, stream));
}

extern "C" int32_t lz_layer_backward(const lz_shape* shape, const lz_layer_buffers* buffers, const void* dy, int32_t accumulate,
                                     void* stream) {
  if (!buffers) return of("lz_layer_backward", LZ_EINVAL);
  const lz_layer_buffers& b = *buffers;
  const bool gate = shape && shape->T > 0 && b.topk_ids && b.dlogits;
  const lz::FfnBackward ffn{b.dyp, b.xp, b.z, b.h, b.w1, b.w2, b.dxp, b.dw1_slot, b.dw2_slot};
  const TileSpecs tables = b.slot_offsets ? lz::backward_tables(shape, ffn, b.train_ws, b.train_ws_bytes, accumulate) : TileSpecs{};
  int32_t rc = of("lz_combine_backward", lz::combine_backward_with(dy, shape, b, gate, tables, stream));
  if (rc != LZ_OK) return rc;
  rc = lz::ffn_backward(shape, ffn, b.slot_offsets, accumulate, b.train_ws, b.train_ws_bytes, tables.n > 0, true, stream);
  if (of(accumulate ? "lz_ffn_backward_accumulate" : "lz_ffn_backward", rc) != LZ_OK) return rc;
  if ((rc = of("lz_permute_backward", lz_permute_backward(b.dxp, b.pair_to_row, shape, b.dx, stream))) != LZ_OK) return rc;
  if (!gate) {
    rc = of("lz_route_backward", lz_route_backward(b.dgates, b.topk_gates, b.topk_ids, shape, b.dlogits, stream));
    if (rc != LZ_OK) return rc;
  }
  if (accumulate) return LZ_OK;
  const int64_t elems = (int64_t)shape->d * shape->ffn;
  return of("lz_reduce_replica_grads_dtype", lz::reduce_pair(shape, b, elems * (shape->act == LZ_SWIGLU ? 2 : 1), elems, stream));
}
