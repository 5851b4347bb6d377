// The gate's routing call; the selection itself is in route.h.
#include "route.h"

namespace {

template <int G, int V, bool VEC, bool SORTED>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                    int32_t* __restrict__ ids, float* __restrict__ gates) {
  route_token<G, V, VEC, SORTED>(logits, (long long)blockIdx.x * (256 / G) + threadIdx.x / G, T, E, k,
                                 [&](long long t, int kk, int id, float gate) {
                                   ids[t * k + kk] = id;
                                   gates[t * k + kk] = gate;
                                 });
}

template <int G, int V>
void launch(const float* logits, int T, int E, int k, int32_t* ids, float* gates, hipStream_t st) {
  const int per_block = 256 / G;
  const unsigned blocks = unsigned((T + per_block - 1) / per_block);
  const bool vec = E % 4 == 0 && (uintptr_t)logits % 16 == 0;
  // Rounds up to four choices (figures in route.h).  Above them sorted keys, but for 65 to 128 experts whose rows are no 16-byte pieces:
  // that kernel falls behind as tokens grow, the later the more choices.  us sorted and by rounds, 81 experts, 4096 tokens, top-5 3.4, 3.7,
  // 6144 4.2, 4.0, 65536 14.3, 12.2; top-6 8192 4.4, 4.3, 65536 15.2, 13.5; top-7 12288 5.3, 5.3, 65536 15.6, 15.0; of 80 experts, top-5,
  // 65536 11.3, 11.4.
  const bool rounds = k <= 4 || (G * V == 128 && !vec && T > 4096 * (k - 4));
  void (*kern)(const float*, int, int, int, int32_t*, float*) =
      rounds ? (vec ? route_kernel<G, V, true, false> : route_kernel<G, V, false, false>)
             : (vec ? route_kernel<G, V, true, true> : route_kernel<G, V, false, true>);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, st, logits, T, E, k, ids, gates);
}

}  // namespace

extern "C" int32_t lz_route(const float* logits, int32_t T, int32_t E, int32_t k, int32_t* topk_ids,
                            float* topk_gates, void* stream) {
  if (T < 0 || E < 1 || E > lz::kMaxE || k < 1 || k > lz::kMaxK || k > E) return LZ_ESHAPE;
  if (T == 0) return LZ_OK;
  if (!logits || !topk_ids || !topk_gates) return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (E <= 4) launch<1, 4>(logits, T, E, k, topk_ids, topk_gates, st);
  else if (E <= 8) launch<2, 4>(logits, T, E, k, topk_ids, topk_gates, st);
  else if (E <= 16) launch<4, 4>(logits, T, E, k, topk_ids, topk_gates, st);
  else if (E <= 32) launch<8, 4>(logits, T, E, k, topk_ids, topk_gates, st);
  else if (E <= 64) launch<16, 4>(logits, T, E, k, topk_ids, topk_gates, st);
  else if (E <= 128) launch<16, 8>(logits, T, E, k, topk_ids, topk_gates, st);
  else launch<16, 16>(logits, T, E, k, topk_ids, topk_gates, st);
  return lz::launch_status();
}
