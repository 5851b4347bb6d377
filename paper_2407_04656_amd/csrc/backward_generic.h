// Training entry points for what the MFMA kernels do not serve (fp32 tensors, bf16 rows that are no whole
// 16-byte pieces, unaligned tensors): the same chain-rule steps as backward.hip on the fp32 matrix-core
// kernel of gemm_f32.h and element-wise kernels.  fp32 accumulation, every stored tensor rounded once
// to the tensor type; the fp32 path uses erff / expf so that it meets the fp32 error bar.
// Device code, not part of the C ABI; included by backward.hip.
#pragma once
#include <type_traits>

#include "gemm_split.h"

namespace {

// What a whole backward pass does in the launch of the combine backward: the gates', whose input that is (dlogits given), and
// the tables of the grouped GEMMs, by the first tables.n workgroups.  Each was a launch of 3 to 6 us.
struct WithCombine {
  const int32_t* ids;
  int E;
  float* dlogits;
  const int32_t* slot_offsets;
  int S, workgroups;
  int tokens;  // of a workgroup, a wave each; its other waves are there for the tables
  TileSpecs tables;
};
struct CombineAlone {};  // lz_combine_backward: none of it, in arguments and LDS neither
template <bool WITH>
using CombineExtra = typename std::conditional<WITH, WithCombine, CombineAlone>::type;
// More slots get a launch of their own: 6 KB of LDS that every workgroup carries; with 48 KB for all 4096 training steps of 528
// slots gain what the launch costs (763 -> 748 us, 2000 tokens 301 -> 295), those of many short rows lose as much (30000 tokens, 64 fp32
// columns 213 -> 216, 60000 of 33 513 -> 518).  Beside the combine up to here: 64 slots 95.6, by themselves 101.2.
constexpr int kTableSlots = 512;
constexpr int kTokensAlone = 4;
template <bool WITH>
constexpr int kCombineThreads = WITH ? kTileThreads : kTokensAlone * lz::kWave;
struct CombineLds {
  SlotRows<kTableSlots> slots;
  TableScratch<kTableSlots> scratch;
};
// true: this workgroup has built a table
__device__ __forceinline__ bool table_workgroup(const WithCombine& with, CombineLds& m) {
  if ((int)blockIdx.x >= with.tables.n) return false;
  const TileSpec& spec = with.tables.spec[blockIdx.x];
  for (int s = threadIdx.x; s < with.S; s += kTileThreads) {
    long long a, b;
    clip_slot(with.slot_offsets, s, spec.P, &a, &b);
    m.slots.first[s] = int(a);
    m.slots.end[s] = int(b);
  }
  __syncthreads();
  build_table(spec, false, m.slots, with.S, m.scratch, threadIdx.x, with.workgroups);
  return true;
}
// The token of this wave, -1: none.
template <bool WITH>
__device__ __forceinline__ long long combine_token(int T, const CombineExtra<WITH>& with) {
  const int w = threadIdx.x / lz::kWave;
  if constexpr (WITH) {
    __shared__ CombineLds lds;
    if (table_workgroup(with, lds) || w >= with.tokens) return -1;
    const long long t = ((long long)blockIdx.x - with.tables.n) * with.tokens + w;
    return t < T ? t : -1;
  } else {
    const long long t = (long long)blockIdx.x * kTokensAlone + w;
    return t < T ? t : -1;
  }
}

// A token's gates' gradients by its whole wave, lane by lane an expert: dlogits[e] = g_e (dg_e - sum_i g_i dg_i).
template <int MAXK>
__device__ __forceinline__ void gate_backward(const WithCombine& with, long long t, int k, const int* id, const float* g, const float* dg) {
  const int lane = threadIdx.x % lz::kWave;
  float inner = 0.f;
#pragma unroll
  for (int kk = 0; kk < MAXK; ++kk)
    if (kk < k) inner = fmaf(g[kk], dg[kk], inner);
  for (int e = lane; e < with.E; e += lz::kWave) {
    float mine_g = 0.f, mine_dg = 0.f;
#pragma unroll
    for (int kk = 0; kk < MAXK; ++kk)
      if (kk < k && id[kk] == e) {
        mine_g = g[kk];
        mine_dg = dg[kk];
      }
    with.dlogits[t * with.E + e] = mine_g * (mine_dg - inner);  // an expert the token did not select has mine_g = 0
  }
}

// combine backward, one wave per token, by elements (rows that are no whole 16-byte pieces, unaligned tensors):
// dgates[t,kk] = <dy[t], yp[row]>, dyp[row] = gates[t,kk] dy[t]
template <typename Elem, bool WITH>
__global__ __launch_bounds__(kCombineThreads<WITH>) void combine_backward_generic_kernel(
    const Elem* __restrict__ dy, const Elem* __restrict__ yp, const int32_t* __restrict__ pair_to_row, const float* __restrict__ gates,
    int T, int k, long long P, int d, Elem* __restrict__ dyp, float* __restrict__ dgates, CombineExtra<WITH> with) {
  const int lane = threadIdx.x % lz::kWave;
  const long long t = combine_token<WITH>(T, with);
  if (t < 0) return;
  int own_id = 0;  // lane kk: the kk-th choice, its gate and that one's gradient
  float own_gate = 0.f, own = 0.f;
  if constexpr (WITH)
    if (with.dlogits != nullptr && lane < k) {
      own_id = with.ids[t * k + lane];
      own_gate = gates[t * k + lane];
    }
  for (int kk = 0; kk < k; ++kk) {
    const int r = pair_to_row[t * k + kk];
    float dot = 0.f;
    if (r >= 0 && r < P) {
      const float g = gates[t * k + kk];
      for (int v = lane; v < d; v += lz::kWave) {
        const float gy = load_elem<Elem>(dy + (size_t)t * d + v);
        dot = fmaf(gy, load_elem<Elem>(yp + (size_t)r * d + v), dot);
        store_elem<Elem>(dyp + (size_t)r * d + v, g * gy);
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off, 64);
    if (lane == 0) dgates[t * k + kk] = dot;
    if constexpr (WITH) own = lane == kk ? dot : own;
  }
  if constexpr (WITH) {
    if (with.dlogits == nullptr) return;
    auto of = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    int id[lz::kMaxK];
    float g[lz::kMaxK], dg[lz::kMaxK];
#pragma unroll
    for (int kk = 0; kk < lz::kMaxK; ++kk) {
      id[kk] = __builtin_amdgcn_readlane(own_id, kk);
      g[kk] = of(own_gate, kk);
      dg[kk] = of(own, kk);
    }
    gate_backward<lz::kMaxK>(with, t, k, id, g, dg);
  }
}

// dW[e] = sum over the slots holding e, ascending slot, fp32 sum, one rounding
template <typename Elem>
__global__ __launch_bounds__(256) void reduce_replicas_generic_kernel(const Elem* __restrict__ dw_slot,
                                                                      const int32_t* __restrict__ slot_expert, int S,
                                                                      long long elems, Elem* __restrict__ dw) {
  const long long v = (long long)blockIdx.x * 256 + threadIdx.x;
  if (v >= elems) return;
  const int e = blockIdx.y;
  float acc = 0.f;
  for (int s = 0; s < S; ++s)
    if (slot_expert[s] == e) acc += load_elem<Elem>(dw_slot + (size_t)s * elems + v);
  store_elem<Elem>(dw + (size_t)e * elems + v, acc);
}

// ---- workspace and drivers of the generic path
struct GenericTrainWorkspace {
  void* dz;     // [P, n1]
  void* tiles;  // kF32Rows-row tiles of the batch
  void* tiles_split;  // fp32: kSplitRows-row tiles
  size_t total_bytes;
  int n1;
};

inline GenericTrainWorkspace carve_train_generic(void* ws, const lz_shape* s) {
  GenericTrainWorkspace w{};
  const long long P = (long long)s->T * s->k;
  w.n1 = s->ffn * (s->act == LZ_SWIGLU ? 2 : 1);
  char* p = (char*)ws;
  auto take = [&](size_t bytes) {
    char* r = p;
    p += lz::align256(bytes);
    return r;
  };
  w.dz = take((size_t)P * w.n1 * lz::elem_bytes(s->dtype));
  w.tiles = take(tile_table_bytes(P, s->N * s->c, kF32Rows));
  if (s->dtype == LZ_F32) w.tiles_split = take(tile_table_bytes(P, s->N * s->c, kSplitRows));
  w.total_bytes = size_t(p - (char*)ws);
  return w;
}

// The tables of a GEMM's arguments, to be built; `split`: that of the 64-row tiles too.
inline TileSpecs generic_tables(F32Args& a, int S, long long P, const GenericTrainWorkspace& w, bool split) {
  TileSpecs specs{};
  a.t = carve_tiles(w.tiles, P, S, kF32Rows);
  add_rows(specs, kF32Rows, P, a.t);
  if (split) {
    a.t_split = carve_tiles(w.tiles_split, P, S, kSplitRows);
    add_rows(specs, kSplitRows, P, a.t_split);
  }
  return specs;
}

template <typename Elem>
int32_t generic_forward_train(const void* xp, const int32_t* slot_offsets, const void* w1, const void* w2,
                              const lz_shape* s, void* z, void* h, void* yp, const GenericTrainWorkspace& w,
                              bool tables_built, hipStream_t st) {
  const long long P = (long long)s->T * s->k;
  const int S = s->N * s->c, d = s->d, ffn = s->ffn, n1 = w.n1;
  // z = xp W1 and h = act(z) from one epilogue   (W1[s] = [d, n1])
  F32Args a{};
  const TileSpecs tables = generic_tables(a, S, P, w, split_forward(s));
  int32_t r = tables_built ? LZ_OK : launch_build_tiles(slot_offsets, S, tables, st);
  if (r != LZ_OK) return r;
  a.A = xp;
  a.W = w1;
  a.C = h;
  a.Z = z;
  a.K = a.lda = d;
  a.ldw = a.ldz = n1;
  a.w_slot = (long long)d * n1;
  a.ldc = a.n_out = a.ffn = ffn;
  a.gather_T = s->T;
  r = s->act == LZ_SWIGLU ? launch_f32_rows<Elem, EPI_SWIGLU_KEEP, true>(a, S, P, st)
                          : launch_f32_rows<Elem, EPI_GELU_KEEP, true>(a, S, P, st);
  if (r != LZ_OK) return r;
  // yp = h W2   (W2[s] = [ffn, d])
  F32Args b{};
  b.t = a.t;
  b.t_split = a.t_split;
  b.A = h;
  b.W = w2;
  b.C = yp;
  b.K = b.lda = ffn;
  b.w_slot = (long long)ffn * d;
  b.ldw = b.ldc = b.n_out = d;
  return launch_f32_rows<Elem, EPI_NONE, true>(b, S, P, st);
}

template <typename Elem>
int32_t generic_ffn_backward(const void* dyp, const void* xp, const void* z, const void* h,
                             const int32_t* slot_offsets, const void* w1, const void* w2, const lz_shape* s,
                             void* dxp, void* dw1, void* dw2, bool accumulate, const GenericTrainWorkspace& w,
                             bool tables_built, bool in_pass, hipStream_t st) {
  const long long P = (long long)s->T * s->k;
  const int S = s->N * s->c, d = s->d, ffn = s->ffn, n1 = w.n1;
  int32_t r;
  if (P > 0) {
    // dZ = (dyp W2^T) * act'(Z): W2[s] [ffn, d] along its rows
    F32Args a{};
    const TileSpecs tables = generic_tables(a, S, P, w, false);  // the data gradients stay on the 32-row tiles
    if (!tables_built && (r = launch_build_tiles(slot_offsets, S, tables, st)) != LZ_OK) return r;
    a.A = dyp;
    a.W = w2;
    a.C = w.dz;
    a.Z = const_cast<void*>(z);
    a.K = a.lda = a.ldw = d;
    a.w_slot = (long long)ffn * d;
    a.ldc = a.ldz = n1;
    a.n_out = a.ffn = ffn;
    r = s->act == LZ_SWIGLU ? launch_f32_rows<Elem, EPI_DSWIGLU, false>(a, S, P, st)
                            : launch_f32_rows<Elem, EPI_DGELU, false>(a, S, P, st);
    if (r != LZ_OK) return r;
    // dxp = dZ W1^T: W1[s] [d, n1] along its rows
    F32Args b{};
    b.t = a.t;
    b.A = w.dz;
    b.W = w1;
    b.C = dxp;
    b.K = b.lda = b.ldw = n1;
    b.w_slot = (long long)d * n1;
    b.ldc = b.n_out = d;
    if ((r = launch_f32_rows<Elem, EPI_NONE, false>(b, S, P, st)) != LZ_OK) return r;
  }
  // dW2[s] = H_s^T dyp_s  [ffn, d],   dW1[s] = xp_s^T dZ_s  [d, n1]
  const F32Wgrad g2 = f32_wgrad<Elem>(h, ffn, dyp, d, slot_offsets, S, P, accumulate ? nullptr : dw2, accumulate ? (float*)dw2 : nullptr);
  const F32Wgrad g1 = f32_wgrad<Elem>(xp, d, w.dz, n1, slot_offsets, S, P, accumulate ? nullptr : dw1, accumulate ? (float*)dw1 : nullptr);
  return accumulate ? launch_f32_wgrads<Elem, EPI_ACCUM>(g2, g1, in_pass, st) : launch_f32_wgrads<Elem, EPI_NONE>(g2, g1, in_pass, st);
}

}  // namespace
