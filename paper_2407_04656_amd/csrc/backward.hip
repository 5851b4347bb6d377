// Backward pass of the MoE layer: the chain rule applied to the forward of Sec. 2.1, step by
// step in reverse (the paper trains the layer and all-reduces each expert's gradient over its
// replicas, Sec. 5, but prints no backward formulas).
//
//   combine      dgates[t,kk] = <dy[t], yp[row]>,  dyp[row] = gates[t,kk] dy[t]      HBM streaming
//   GEMM-2       dH = dyp W2^T          (dgrad)    dW2[s] = H_s^T dyp_s   (wgrad)     MFMA   W2[s] = [ffn, d]
//   activation   dZ = dH * act'(Z)                                                  HBM streaming
//   GEMM-1       dxp = dZ W1^T          (dgrad)    dW1[s] = xp_s^T dZ_s   (wgrad)     MFMA   W1[s] = [d, n1]
//   permute      dx[t] = sum_kk dxp[row(t,kk)]                                      HBM streaming
//   gate         dlogits = softmax backward on the k selected logits
//   replicas     dW[e] = sum over the slots that hold e                             HBM streaming
//
// Every contraction runs on the forward's grouped MFMA kernel in one of its three operand
// modes.  The weights are stored input-major ([d, n1] and [ffn, d]: the forward contracts over
// their rows), so the data gradients contract along their rows' direction (both operands
// k-contiguous) and the weight gradients over a slot's rows of two activation matrices (both
// operands k-major, a different length for every slot).  k-major tiles stream into LDS as they
// lie in memory and are transposed on the way to the registers (gfx950's transposing LDS
// reads): no transposed copy of weights or activations is ever written.  The weight gradients
// run over S x (rows of the weight matrix) virtual rows; each tile takes its contraction range
// from slot_offsets.
#include "backward_generic.h"
#include "gemm_narrow.h"
#include "layer.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ void unpack8(const u32x4& v, float* f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f[2 * q] = __uint_as_float(w[q] << 16);
    f[2 * q + 1] = __uint_as_float(w[q] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ u32x4 pack8(const float* f) {
  u32x4 o;
  o.x = pack_bf16x2(f[0], f[1]);
  o.y = pack_bf16x2(f[2], f[3]);
  o.z = pack_bf16x2(f[4], f[5]);
  o.w = pack_bf16x2(f[6], f[7]);
  return o;
}

// the elements of a 16-byte piece
__device__ __forceinline__ void unpack(const u32x4& v, float* f, uint16_t) { unpack8(v, f); }
__device__ __forceinline__ void unpack(const u32x4& v, float* f, float) {
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = __uint_as_float(v[q]);
}
__device__ __forceinline__ u32x4 pack(const float* f, uint16_t) { return pack8(f); }
__device__ __forceinline__ u32x4 pack(const float* f, float) {
  return u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
}

template <bool STREAM>
__device__ __forceinline__ u32x4 load_piece(const u32x4* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool STREAM>
__device__ __forceinline__ void store_piece(const u32x4& v, u32x4* p) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ---- combine backward: one wave per token.  dy[t] is read once, every yp row once, every
// dyp row written once; the k dot products are reduced over the wave at the end.
// MAXK: the most choices a token can have.  Room for eight of them is 100 registers and four waves a SIMD, which costs an fp32 row,
// whose elements' kernel runs eight: us for 40000 tokens of 128 columns, top-2, elements 20.5, this kernel with room for eight 32.4, for
// two 22.0; 10897 of 368, top-4, 32.0, 30.0, and 27.1 for four; 5448 of 320, top-1, 4.4, 6.0, and 4.4 for one.
// STREAM: past the caches.  fp32, 40000 tokens of 384 columns, top-4 (553 MB) 117 us, 125 through them; 8000 of 1024, top-2 (164 MB, left in
// the caches by the call before) 38 and 27.
template <typename Elem, bool WITH, int MAXK, bool STREAM>
__global__ __launch_bounds__(kCombineThreads<WITH>) void combine_backward_kernel(
    const u32x4* __restrict__ dy, const u32x4* __restrict__ yp, const int32_t* __restrict__ pair_to_row, const float* __restrict__ gates,
    int T, int k, long long P, int vec_per_row, u32x4* __restrict__ dyp, float* __restrict__ dgates, CombineExtra<WITH> with) {
  const int lane = threadIdx.x % lz::kWave;
  const long long t = combine_token<WITH>(T, with);
  if (t < 0) return;
  long long rows[MAXK];
  float g[MAXK], dot[MAXK];
#pragma unroll
  for (int kk = 0; kk < MAXK; ++kk) {
    rows[kk] = -1;
    g[kk] = 0.f;
    dot[kk] = 0.f;
    if (kk < k) {
      const int r = pair_to_row[t * k + kk];
      rows[kk] = (r >= 0 && r < P) ? r : -1;
      g[kk] = gates[t * k + kk];
    }
  }
  for (int v = lane; v < vec_per_row; v += lz::kWave) {
    constexpr int kElems = 16 / sizeof(Elem);
    float gy[kElems];
    unpack(load_piece<STREAM>(dy + (size_t)t * vec_per_row + v), gy, Elem{});
    u32x4 in[MAXK];
#pragma unroll
    for (int kk = 0; kk < MAXK; ++kk)
      if (kk < k && rows[kk] >= 0) in[kk] = load_piece<STREAM>(yp + (size_t)rows[kk] * vec_per_row + v);
#pragma unroll
    for (int kk = 0; kk < MAXK; ++kk)
      if (kk < k && rows[kk] >= 0) {
        float y[kElems], o[kElems];
        unpack(in[kk], y, Elem{});
#pragma unroll
        for (int q = 0; q < kElems; ++q) {
          dot[kk] = fmaf(gy[q], y[q], dot[kk]);
          o[q] = g[kk] * gy[q];
        }
        store_piece<STREAM>(pack(o, Elem{}), dyp + (size_t)rows[kk] * vec_per_row + v);
      }
  }
#pragma unroll
  for (int kk = 0; kk < MAXK; ++kk)
    if (kk < k) {
      dot[kk] = wave_sum(dot[kk]);
      if (lane == 0) dgates[t * k + kk] = dot[kk];
    }
  if constexpr (WITH)
    if (with.dlogits != nullptr) {
      int id[MAXK];
#pragma unroll
      for (int kk = 0; kk < MAXK; ++kk) id[kk] = kk < k ? with.ids[t * k + kk] : 0;
      gate_backward<MAXK>(with, t, k, id, g, dot);
    }
}

// ---- gate backward: thread per (token, expert)
__global__ __launch_bounds__(256) void route_backward_kernel(const float* __restrict__ dgates,
                                                             const float* __restrict__ gates,
                                                             const int32_t* __restrict__ ids, int T, int E, int k,
                                                             float* __restrict__ dlogits) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)T * E) return;
  const long long t = i / E;
  const int e = int(i % E);
  float inner = 0.f, mine_g = 0.f, mine_dg = 0.f;
  for (int kk = 0; kk < k; ++kk) {
    const float g = gates[t * k + kk], dg = dgates[t * k + kk];
    inner = fmaf(g, dg, inner);
    if (ids[t * k + kk] == e) {
      mine_g = g;
      mine_dg = dg;
    }
  }
  dlogits[i] = mine_g * (mine_dg - inner);  // an expert the token did not select has mine_g = 0
}

// ---- activations on stored pre-activations (bf16, 8 elements per lane)
__device__ __forceinline__ float sigmoid_fast(float v) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * v));
}
// gelu'(v) = Phi(v) + v phi(v), Phi through the rational erf of Abramowitz-Stegun 7.1.26, absolute error below 2e-7
__device__ __forceinline__ float gelu_grad_fast(float v) {
  const float x = fabsf(v) * 0.70710678118654752440f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(-1.44269504088896341f * x * x);  // exp(-v^2/2)
  const float erf_abs = 1.0f - p * t * e;
  const float cdf = 0.5f + 0.5f * (v < 0.f ? -erf_abs : erf_abs);
  return fmaf(v * 0.3989422804014327f, e, cdf);
}

// dZ = dH * act'(Z)
template <bool SWIGLU>
__global__ __launch_bounds__(256) void act_backward_kernel(const u32x4* __restrict__ dH, const u32x4* __restrict__ Z,
                                                           long long P, int ffn_vec, u32x4* __restrict__ dZ) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= P * ffn_vec) return;
  const long long row = i / ffn_vec;
  const int v = int(i % ffn_vec);
  const int z_vec = SWIGLU ? 2 * ffn_vec : ffn_vec;
  float g[8], a[8];
  unpack8(__builtin_nontemporal_load(dH + i), g);
  unpack8(__builtin_nontemporal_load(Z + row * z_vec + v), a);
  if (SWIGLU) {
    float u[8], dg[8], du[8];
    unpack8(__builtin_nontemporal_load(Z + row * z_vec + ffn_vec + v), u);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float s = sigmoid_fast(a[q]);
      dg[q] = g[q] * u[q] * (s * fmaf(a[q], 1.0f - s, 1.0f));
      du[q] = g[q] * (a[q] * s);
    }
    __builtin_nontemporal_store(pack8(dg), dZ + row * z_vec + v);
    __builtin_nontemporal_store(pack8(du), dZ + row * z_vec + ffn_vec + v);
  } else {
    float o[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = g[q] * gelu_grad_fast(a[q]);
    __builtin_nontemporal_store(pack8(o), dZ + row * z_vec + v);
  }
}

// dW[e] = sum over slots s with slot_expert[s] == e of dW_slot[s], ascending s, fp32 sum, one rounding.
// HBM bound: (S + E) x elems read and written once.  A thread owns one 16-byte vector of an expert's
// gradient and has it loaded from kReduceAhead of the expert's slots before the first is added; the
// slots are found 64 at a time with one coalesced load of slot_expert and a ballot (a loop of scalar
// loads over all S slots costs more than the sums where S is in the hundreds).  fp32, 128 slots of 64
// experts, 4.4 GB in and 2.2 GB out: 11.4 ms with one 4-byte element per thread and the slot loop,
// 1.24 ms now (5.3 TB/s).  Four vectors of one slot in flight per thread instead are level there, but
// leave a long tail where one expert holds half the slots (60 slots of 8 experts, 0.6 GB: +40 %).
// fp32 sums of a few experts whose gradients are short are too few threads for that: they load kReduceAheadFew slots
// ahead, where 64 slots hold that many of one expert.  512 slots of 1 expert of 65536, 2048 of 2 experts of 4096:
// 140, 192 us by elements with caching loads, 234, 237 us with four ahead, 59, 90 us so.  With more experts the longer
// chain of tests costs up to 70 %; bf16 is within 5 % either way.
constexpr int kReduceAhead = 4, kReduceAheadFew = 16, kReduceFewExperts = 4, kReduceFewBlocks = 1024;

__device__ __forceinline__ void add_vec(float* acc, const u32x4& v, float) {
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] += __uint_as_float(v[q]);
}
__device__ __forceinline__ void add_vec(float* acc, const u32x4& v, uint16_t) {
  float f[8];
  unpack8(v, f);
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] += f[q];
}
__device__ __forceinline__ u32x4 sum_vec(const float* acc, float) {
  return u32x4{__float_as_uint(acc[0]), __float_as_uint(acc[1]), __float_as_uint(acc[2]), __float_as_uint(acc[3])};
}
__device__ __forceinline__ u32x4 sum_vec(const float* acc, uint16_t) { return pack8(acc); }

// One matrix of every slot; a launch sums one or two.
struct ReducePart {
  const u32x4* dw_slot;
  u32x4* dw;
  long long vec_per_slot;
};
template <typename Elem, int AHEAD>
__global__ __launch_bounds__(256) void reduce_replicas_kernel(ReducePart part0, ReducePart part1, unsigned blocks0,
                                                              const int32_t* __restrict__ slot_expert, int S) {
  const int e = blockIdx.y, lane = threadIdx.x % lz::kWave;
  const bool second = blockIdx.x >= blocks0;
  const u32x4* __restrict__ const dw_slot = second ? part1.dw_slot : part0.dw_slot;
  u32x4* __restrict__ const dw = second ? part1.dw : part0.dw;
  const long long vec_per_slot = second ? part1.vec_per_slot : part0.vec_per_slot;
  const long long v = (long long)(blockIdx.x - (second ? blocks0 : 0)) * 256 + threadIdx.x;
  const bool live = v < vec_per_slot;
  float acc[16 / sizeof(Elem)] = {};
  for (int s0 = 0; s0 < S; s0 += lz::kWave) {
    unsigned long long mine = __ballot(s0 + lane < S && slot_expert[s0 + lane < S ? s0 + lane : 0] == e);
    while (mine) {
      u32x4 in[AHEAD];
      int n = 0;
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (mine) {
          const int s = s0 + __ffsll((long long)mine) - 1;
          mine &= mine - 1;
          if (live) in[u] = __builtin_nontemporal_load(dw_slot + (size_t)s * vec_per_slot + v);
          n = u + 1;
        }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (u < n && live) add_vec(acc, in[u], Elem{});
    }
  }
  if (live) __builtin_nontemporal_store(sum_vec(acc, Elem{}), dw + (size_t)e * vec_per_slot + v);
}

// ---- workspace of the training entry points
struct TrainWorkspace {
  uint16_t* dh;        // [P, ffn]
  uint16_t* dz;        // [P, n1]
  void* units_up;      // rows of the batch, ffn / 128 (gated) or 256 column tiles
  void* units_ffn;     // rows of the batch, ffn / 256 column tiles
  void* units_d;       // rows of the batch, d / 256 column tiles
  void* units_w2;      // S * ffn virtual rows, d / 256 column tiles
  void* units_w1;      // S * d virtual rows, n1 / 256 column tiles
  void* tiles_narrow;  // rows of the batch, tiles of the GEMMs on narrow tiles
  bool narrow_up, narrow_ffn, narrow_d;  // z, h; dH; yp and dxp on narrow tiles
  size_t total_bytes;
  int n1;
};

TrainWorkspace carve_train(void* ws, const lz_shape* s) {
  TrainWorkspace w;
  const long long P = (long long)s->T * s->k;
  const int S = s->N * s->c;
  w.n1 = s->ffn * (s->act == LZ_SWIGLU ? 2 : 1);
  char* p = (char*)ws;
  auto take = [&](size_t bytes) {
    char* r = p;
    p += lz::align256(bytes);
    return r;
  };
  w.dh = (uint16_t*)take((size_t)P * s->ffn * 2);
  w.dz = (uint16_t*)take((size_t)P * w.n1 * 2);
  w.units_up = take(unit_table_bytes(P, S, ceil_div(s->ffn, s->act == LZ_SWIGLU ? BN / 2 : BN)));
  w.units_ffn = take(unit_table_bytes(P, S, ceil_div(s->ffn, BN)));
  w.units_d = take(unit_table_bytes(P, S, ceil_div(s->d, BN)));
  w.units_w2 = take(unit_table_bytes((long long)S * s->ffn, S, ceil_div(s->d, BN)));
  w.units_w1 = take(unit_table_bytes((long long)S * s->d, S, ceil_div(w.n1, BN)));
  w.narrow_ffn = use_narrow(P, S, s->ffn);
  w.narrow_up = w.narrow_ffn && s->act == LZ_GELU;
  w.narrow_d = use_narrow(P, S, s->d);
  w.tiles_narrow = take(tile_table_bytes(P, S, kNarrow));  // also where this P does not use it, as in the forward
  w.total_bytes = size_t(p - (char*)ws);
  return w;
}

// the fp32 kernels' envelope: every valid shape of at most 65535 64-row tiles
inline bool generic_train_shape(const lz_shape* s) {
  if (!lz::shape_ok(s)) return false;
  return tile_capacity((long long)s->T * s->k, s->N * s->c, 64) <= 65535;
}

// The shapes the MFMA kernels serve: bf16 rows of whole 16-byte pieces, virtual row indices within int32.  Sizes
// that the tiles do not divide stay inside the envelope above: they also take unaligned tensors, on the fp32
// kernels (each call by itself: no state passes between the calls through the workspace).
inline bool train_whole_tiles(const lz_shape* s) { return s->d % BN == 0 && s->ffn % 64 == 0; }
inline bool train_shape(const lz_shape* s) {
  if (!lz::shape_ok(s) || !mfma_sizes(s)) return false;
  const long long S = (long long)s->N * s->c;
  return S * s->d * 2 < (1ll << 31) && S * s->ffn * 2 < (1ll << 31) && (train_whole_tiles(s) || generic_train_shape(s));
}

int32_t check_train(const lz_shape* shape, void* ws, size_t ws_bytes, TrainWorkspace* w) {
  if (!train_shape(shape)) return LZ_ESHAPE;
  *w = carve_train(ws, shape);
  if (!ws || (uintptr_t)ws % 256 != 0 || ws_bytes < w->total_bytes) return LZ_EWORKSPACE;
  return LZ_OK;
}

TileTable narrow_tiles(const TrainWorkspace& w, int S, long long P) { return carve_tiles(w.tiles_narrow, P, S, kNarrow); }

// C[rows, n_out] = A[rows, K] W[slot][n_out, K]^T over the batch's ragged row ranges
int32_t gemm_nt(const uint16_t* A, const uint16_t* W, uint16_t* C, long long P, int K, int n_out,
                const UnitTable& u, bool narrow, const TrainWorkspace& w, int S, hipStream_t st) {
  MfmaArgs g{};
  g.A = A;
  g.W = W;
  g.C = C;
  g.P = P;
  g.K = K;
  g.w_rows = n_out;
  g.n_out = n_out;
  g.n_tiles = ceil_div(n_out, BN);
  g.u = u;
  if (narrow) return launch_narrow<EPI_NONE, MODE_NT>(g, narrow_tiles(w, S, P), st);
  return launch_mfma<EPI_NONE>(g, st);
}

// C[rows, n_out] = A[rows, K] W[slot][K, n_out] over the batch's ragged row ranges
int32_t gemm_nn(const uint16_t* A, const uint16_t* W, uint16_t* C, long long P, int K, int n_out,
                const UnitTable& u, bool narrow, const TrainWorkspace& w, int S, hipStream_t st) {
  MfmaArgs g{};
  g.A = A;
  g.W = W;
  g.C = C;
  g.P = P;
  g.K = K;
  g.w_rows = n_out;
  g.n_out = n_out;
  g.n_tiles = ceil_div(n_out, BN);
  g.u = u;
  g.ldw = n_out;
  if (narrow) return launch_narrow<EPI_NONE, MODE_NN>(g, narrow_tiles(w, S, P), st);
  return launch_mfma<EPI_NONE, MODE_NN>(g, st);
}

// dW[s] [rows_per_slot, n_out] = A[rows of s, :rows_per_slot]^T W[rows of s, :n_out], stored as bf16 in C,
// or, if Cacc is given, added to that fp32 matrix instead
MfmaArgs wgrad_args(const uint16_t* A, const uint16_t* W, uint16_t* C, float* Cacc, int S, int rows_per_slot, int n_out,
                    const UnitTable& u) {
  MfmaArgs g{};
  g.A = A;
  g.W = W;
  g.C = C;
  g.Cacc = Cacc;
  g.P = (long long)S * rows_per_slot;
  g.w_rows = n_out;
  g.n_out = n_out;
  g.n_tiles = ceil_div(n_out, BN);
  g.u = u;
  g.lda = rows_per_slot;
  g.ldw = n_out;
  g.rows_per_slot = rows_per_slot;
  return g;
}

// 32-bit byte offsets do if no operand reaches 4 GiB, the K steps past a slot's end included
inline bool wgrad_is_wide(long long P, int lda, int ldw) {
  return ((unsigned long long)P + 4 * BK) * (unsigned)(lda > ldw ? lda : ldw) * 2ull > 0xFFFFFFFFull;
}

// Whether a whole pass has both weight gradients in one launch.  The second's tiles fill what the first's last round leaves idle, and where
// tiles are few they run side by side: a training step of 73 tokens over 33 slots, 768 x 2240, 318 -> 302 us, of 40960 tokens, top-1,
// 768 x 3072, over 60 slots 1691 -> 1673.  Backward passes of 2573 drawn layers, geometric mean by the rounds of 256 x 256 tiles of both:
// below 1 round 0.87 of two launches' time, to 4 0.93, 16 0.96, 32 0.99, and from there on, with 128 rows a slot and more, 0.994; with
// fewer 0.999, at the worst 1.024 (276 tokens, 42 slots, 1920 x 3136; 429 tokens over 50 slots, 3072 x 3840, 1.007): two launches.
inline bool pair_wgrads(const lz_shape* s) {
  const long long P = (long long)s->T * s->k, slots = (long long)s->N * s->c;
  const int n1 = s->act == LZ_SWIGLU ? 2 * s->ffn : s->ffn;
  const long long tiles = slots * ceil_div(s->d, BN) * (ceil_div(s->ffn, BM) + ceil_div(n1, BN));
  return (tiles < 32ll * device_cus() || P >= 128 * slots) && !wgrad_is_wide(P, s->ffn, s->d) && !wgrad_is_wide(P, s->d, n1);
}
int32_t gemm_wgrads(const MfmaArgs& g0, const MfmaArgs& g1, long long P, bool accumulate, bool pair, hipStream_t st) {
  if (pair) return accumulate ? launch_mfma_pair<EPI_ACCUM>(g0, g1, st) : launch_mfma_pair<EPI_NONE>(g0, g1, st);
  auto one = [&](const MfmaArgs& g) {
    if (wgrad_is_wide(P, g.lda, g.ldw)) return accumulate ? launch_mfma<EPI_ACCUM, MODE_TN_WIDE>(g, st) : launch_mfma<EPI_NONE, MODE_TN_WIDE>(g, st);
    return accumulate ? launch_mfma<EPI_ACCUM, MODE_TN>(g, st) : launch_mfma<EPI_NONE, MODE_TN>(g, st);
  };
  const int32_t r = one(g0);
  return r != LZ_OK ? r : one(g1);
}

int32_t check_train_generic(const lz_shape* shape, void* ws, size_t ws_bytes, GenericTrainWorkspace* w) {
  if (!generic_train_shape(shape)) return LZ_ESHAPE;
  *w = carve_train_generic(ws, shape);
  if (!ws || (uintptr_t)ws % 256 != 0 || ws_bytes < w->total_bytes) return LZ_EWORKSPACE;
  return LZ_OK;
}

}  // namespace

extern "C" size_t lz_train_workspace_bytes(const lz_shape* shape) {
  const size_t generic = generic_train_shape(shape) ? carve_train_generic(nullptr, shape).total_bytes : 0;
  if (!train_shape(shape)) return generic;
  const size_t bytes = carve_train(nullptr, shape).total_bytes;
  return bytes > generic || train_whole_tiles(shape) ? bytes : generic;
}

namespace {

// Whether the bf16 kernels serve the call.
bool on_mfma(const lz_shape* shape, bool aligned) { return train_shape(shape) && (aligned || train_whole_tiles(shape)); }

TileSpecs forward_tables(const TrainWorkspace& w, const lz_shape* shape) {
  const long long P = (long long)shape->T * shape->k;
  const int S = shape->N * shape->c, n_up = ceil_div(shape->ffn, shape->act == LZ_SWIGLU ? BN / 2 : BN), n_d = ceil_div(shape->d, BN);
  TileSpecs specs{};
  if (!w.narrow_up) add_units(specs, n_up, 0, P, carve_units(w.units_up, P, S, n_up));
  if (!w.narrow_d) add_units(specs, n_d, 0, P, carve_units(w.units_d, P, S, n_d));
  if (w.narrow_up || w.narrow_d) add_rows(specs, kNarrow, P, narrow_tiles(w, S, P));
  return specs;
}

}  // namespace

TileSpecs lz::train_tables(const lz_shape* shape, const FfnTrain& t, void* ws, size_t ws_bytes) {
  if (!lz::shape_ok(shape) || (long long)shape->T * shape->k == 0) return TileSpecs{};
  if (on_mfma(shape, t.aligned())) {
    TrainWorkspace w;
    return check_train(shape, ws, ws_bytes, &w) == LZ_OK ? forward_tables(w, shape) : TileSpecs{};
  }
  GenericTrainWorkspace w;
  F32Args a{};
  if (check_train_generic(shape, ws, ws_bytes, &w) != LZ_OK) return TileSpecs{};
  return generic_tables(a, shape->N * shape->c, (long long)shape->T * shape->k, w, split_forward(shape));
}

int32_t lz::ffn_forward_train(const lz_shape* shape, const FfnTrain& t, const int32_t* slot_offsets, void* ws, size_t ws_bytes,
                              bool tables_built, void* stream) {
  const auto [xp, w1, w2, z, h, yp] = t;
  const bool aligned = t.aligned();
  if (!on_mfma(shape, aligned)) {
    GenericTrainWorkspace gw;
    const int32_t grc = check_train_generic(shape, ws, ws_bytes, &gw);
    if (grc != LZ_OK) return grc;
    if ((long long)shape->T * shape->k == 0) return LZ_OK;
    if (!xp || !slot_offsets || !w1 || !w2 || !z || !h || !yp) return LZ_EINVAL;
    return shape->dtype == LZ_F32
               ? generic_forward_train<float>(xp, slot_offsets, w1, w2, shape, z, h, yp, gw, tables_built, (hipStream_t)stream)
               : generic_forward_train<uint16_t>(xp, slot_offsets, w1, w2, shape, z, h, yp, gw, tables_built, (hipStream_t)stream);
  }
  TrainWorkspace w;
  const int32_t rc = check_train(shape, ws, ws_bytes, &w);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  if (P == 0) return LZ_OK;
  if (!xp || !slot_offsets || !w1 || !w2 || !z || !h || !yp) return LZ_EINVAL;
  if (!aligned) return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int S = shape->N * shape->c;
  const bool swiglu = shape->act == LZ_SWIGLU;
  const int n_up = ceil_div(shape->ffn, swiglu ? BN / 2 : BN);
  const UnitTable u_up = carve_units(w.units_up, P, S, n_up);
  const UnitTable u_d = carve_units(w.units_d, P, S, ceil_div(shape->d, BN));
  int32_t r = tables_built ? LZ_OK : launch_build_tiles(slot_offsets, S, forward_tables(w, shape), st);
  if (r != LZ_OK) return r;
  // z = xp W1 and h = act(z) from one epilogue
  MfmaArgs g{};
  g.A = (const uint16_t*)xp;
  g.W = (const uint16_t*)w1;
  g.C = (uint16_t*)h;
  g.Z = (uint16_t*)z;
  g.z_cols = w.n1;
  g.P = P;
  g.K = shape->d;
  g.w_rows = w.n1;
  g.n_out = shape->ffn;
  g.up_row0 = swiglu ? shape->ffn : 0;
  g.n_tiles = n_up;
  g.u = u_up;
  g.ldw = w.n1;
  if (w.narrow_up) r = launch_narrow<EPI_GELU_KEEP, MODE_NN>(g, narrow_tiles(w, S, P), st);
  else r = swiglu ? launch_mfma<EPI_SWIGLU_KEEP, MODE_NN>(g, st) : launch_mfma<EPI_GELU_KEEP, MODE_NN>(g, st);
  if (r != LZ_OK) return r;
  return gemm_nn((const uint16_t*)h, (const uint16_t*)w2, (uint16_t*)yp, P, shape->ffn, shape->d, u_d,
                 w.narrow_d, w, S, st);
}

extern "C" int32_t lz_ffn_forward_train(const void* xp, const int32_t* slot_offsets, const void* w1, const void* w2,
                                        const lz_shape* shape, void* z, void* h, void* yp, void* ws,
                                        size_t ws_bytes, void* stream) {
  return lz::ffn_forward_train(shape, lz::FfnTrain{xp, w1, w2, z, h, yp}, slot_offsets, ws, ws_bytes, false, stream);
}

namespace {

// Bytes of the combine backward's rows that the memory-side cache holds.
constexpr long long kCachedBytes = 256ll << 20;

// Which of fp32 rows of whole 16-byte pieces the vector kernel takes; bits of dgates depend on it.  Rows of fewer than 24 pieces leave lanes
// without work, and more than four choices their room for eight (see the kernel), which few tokens and rows from memory do not feel.
// us by elements, by vectors: 16000 tokens of 32 columns, top-4 8.6, 11.1; 8000 of 96, top-4 8.0, 8.3; 8000 of 256, top-6 18.6, 23.1;
// 4096 of them 14.5, 11.8; 1000 of 96, top-8 7.0, 6.5; 40000 of 128, top-8 (348 MB) 107, 87.
inline bool vectors_f32(const lz_shape* s, long long bytes) {
  return s->d >= 96 && (s->k <= 4 || s->T <= 4096 || bytes > kCachedBytes);
}

template <typename Elem, bool WITH>
auto combine_kernel_of(int k, bool stream) {
  if constexpr (sizeof(Elem) == 2) return combine_backward_kernel<Elem, WITH, lz::kMaxK, true>;
  else
    return stream ? (k > 4   ? combine_backward_kernel<Elem, WITH, lz::kMaxK, true>
                     : k > 2 ? combine_backward_kernel<Elem, WITH, 4, true>
                     : k > 1 ? combine_backward_kernel<Elem, WITH, 2, true>
                             : combine_backward_kernel<Elem, WITH, 1, true>)
                  : (k > 4   ? combine_backward_kernel<Elem, WITH, lz::kMaxK, false>
                     : k > 2 ? combine_backward_kernel<Elem, WITH, 4, false>
                     : k > 1 ? combine_backward_kernel<Elem, WITH, 2, false>
                             : combine_backward_kernel<Elem, WITH, 1, false>);
}

int32_t check_combine(const void* dy, const void* yp, const int32_t* pair_to_row, const float* topk_gates, const lz_shape* shape,
                      const void* dyp, const float* dgates) {
  if (!lz::shape_ok(shape)) return LZ_ESHAPE;
  return shape->T == 0 || (dy && yp && pair_to_row && topk_gates && dyp && dgates) ? LZ_OK : LZ_EINVAL;
}

template <bool WITH>
int32_t combine_backward(const void* dy, const void* yp, const int32_t* pair_to_row, const float* topk_gates, const lz_shape* shape,
                         void* dyp, float* dgates, const CombineExtra<WITH>& with, hipStream_t st) {
  const int32_t rc = check_combine(dy, yp, pair_to_row, topk_gates, shape, dyp, dgates);
  if (rc != LZ_OK || shape->T == 0) return rc;
  const long long P = (long long)shape->T * shape->k;
  int tokens = kTokensAlone, first = 0;
  if constexpr (WITH) tokens = with.tokens, first = with.tables.n;
  const dim3 grid((unsigned)((shape->T + tokens - 1) / tokens + first)), threads(kCombineThreads<WITH>);
  const size_t row_bytes = (size_t)shape->d * lz::elem_bytes(shape->dtype);
  const long long bytes = (2 * P + shape->T) * (long long)row_bytes;
  const bool whole = row_bytes % 16 == 0 && aligned16(dy) && aligned16(yp) && aligned16(dyp) &&
                     (shape->dtype == LZ_BF16 || vectors_f32(shape, bytes));
  auto launch = [&](auto elem) {
    using Elem = decltype(elem);
    if (whole)
      hipLaunchKernelGGL((combine_kernel_of<Elem, WITH>(shape->k, bytes > kCachedBytes)), grid, threads, 0, st, (const u32x4*)dy,
                         (const u32x4*)yp, pair_to_row, topk_gates, shape->T, shape->k, P, int(row_bytes / 16), (u32x4*)dyp, dgates, with);
    else
      hipLaunchKernelGGL((combine_backward_generic_kernel<Elem, WITH>), grid, threads, 0, st, (const Elem*)dy, (const Elem*)yp,
                         pair_to_row, topk_gates, shape->T, shape->k, P, shape->d, (Elem*)dyp, dgates, with);
  };
  if (shape->dtype == LZ_F32) launch(float{});
  else launch(uint16_t{});
  return lz::launch_status();
}

}  // namespace

extern "C" int32_t lz_combine_backward(const void* dy, const void* yp, const int32_t* pair_to_row,
                                       const float* topk_gates, const lz_shape* shape, void* dyp, float* dgates,
                                       void* stream) {
  return combine_backward<false>(dy, yp, pair_to_row, topk_gates, shape, dyp, dgates, CombineAlone{}, (hipStream_t)stream);
}

int32_t lz::combine_backward_with(const void* dy, const lz_shape* shape, const lz_layer_buffers& b, bool gate, const TileSpecs& tables,
                                  void* stream) {
  if (!gate && tables.n == 0) return lz_combine_backward(dy, b.yp, b.pair_to_row, b.topk_gates, shape, b.dyp, b.dgates, stream);
  const int32_t rc = check_combine(dy, b.yp, b.pair_to_row, b.topk_gates, shape, b.dyp, b.dgates);
  if (rc != LZ_OK) return rc;
  const int workgroups = device_cus();
  if (workgroups == 0) return LZ_EHIP;
  // Four tokens a workgroup while that gives no CU a second one: us for 225 tokens, top-8, 3944 bf16 columns 29 with eight, 21 with
  // four; 2450, top-6, 672 17 and 18; 40960, top-1, 768 52 and 66.
  const WithCombine with{b.topk_ids, shape->E, gate ? b.dlogits : nullptr, b.slot_offsets, shape->N * shape->c, workgroups,
                         shape->T <= 4 * workgroups ? 4 : kTileThreads / lz::kWave, tables};
  return combine_backward<true>(dy, b.yp, b.pair_to_row, b.topk_gates, shape, b.dyp, b.dgates, with, (hipStream_t)stream);
}

extern "C" int32_t lz_route_backward(const float* dgates, const float* topk_gates, const int32_t* topk_ids,
                                     const lz_shape* shape, float* dlogits, void* stream) {
  if (!lz::shape_ok(shape)) return LZ_ESHAPE;
  if (shape->T == 0) return LZ_OK;
  if (!dgates || !topk_gates || !topk_ids || !dlogits) return LZ_EINVAL;
  const long long n = (long long)shape->T * shape->E;
  hipLaunchKernelGGL(route_backward_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     dgates, topk_gates, topk_ids, shape->T, shape->E, shape->k, dlogits);
  return lz::launch_status();
}

namespace {

TileSpecs backward_tables(const TrainWorkspace& w, const lz_shape* shape, bool accumulate, bool pair) {
  const long long P = (long long)shape->T * shape->k;
  const int S = shape->N * shape->c, d = shape->d, ffn = shape->ffn;
  const int n_ffn = ceil_div(ffn, BN), n_d = ceil_div(d, BN), n_n1 = ceil_div(w.n1, BN);
  TileSpecs specs{};
  if (!w.narrow_ffn) add_units(specs, n_ffn, 0, P, carve_units(w.units_ffn, P, S, n_ffn));
  if (!w.narrow_d) add_units(specs, n_d, 0, P, carve_units(w.units_d, P, S, n_d));
  add_units(specs, n_d, ffn, P, carve_units(w.units_w2, (long long)S * ffn, S, n_d), accumulate);
  add_units(specs, n_n1, d, P, carve_units(w.units_w1, (long long)S * d, S, n_n1), accumulate);
  // Longer slots keep the rows that suit each list: there the tiles of the fullest slot, which few rows make short, end last (30617 tokens,
  // top-2, over 66 slots of unlike loads, 256 x 256: a training step 484 us with rows for both, 435).
  if (pair && P < 128ll * S) share_launch(specs);
  if (w.narrow_ffn || w.narrow_d) add_rows(specs, kNarrow, P, narrow_tiles(w, S, P));
  return specs;
}

}  // namespace

TileSpecs lz::backward_tables(const lz_shape* shape, const FfnBackward& t, void* ws, size_t ws_bytes, bool accumulate) {
  if (!lz::shape_ok(shape) || shape->N * shape->c > kTableSlots || shape->T == 0) return TileSpecs{};
  if (on_mfma(shape, t.aligned())) {
    TrainWorkspace w;
    return check_train(shape, ws, ws_bytes, &w) == LZ_OK ? ::backward_tables(w, shape, accumulate, pair_wgrads(shape)) : TileSpecs{};
  }
  GenericTrainWorkspace w;
  F32Args a{};
  if (check_train_generic(shape, ws, ws_bytes, &w) != LZ_OK) return TileSpecs{};
  return generic_tables(a, shape->N * shape->c, (long long)shape->T * shape->k, w, false);
}

// dw1 / dw2 are bf16 gradients (accumulate == false: overwritten) or fp32 sums (accumulate == true: added to)
int32_t lz::ffn_backward(const lz_shape* shape, const FfnBackward& t, const int32_t* slot_offsets, bool accumulate, void* ws,
                         size_t ws_bytes, bool tables_built, bool in_pass, void* stream) {
  const auto [dyp, xp, z, h, w1, w2, dxp, dw1, dw2] = t;
  const bool aligned = t.aligned();
  if (!on_mfma(shape, aligned)) {
    GenericTrainWorkspace gw;
    const int32_t grc = check_train_generic(shape, ws, ws_bytes, &gw);
    if (grc != LZ_OK) return grc;
    if (!dw1 || !dw2 || !slot_offsets) return LZ_EINVAL;
    if ((long long)shape->T * shape->k > 0 && (!dyp || !xp || !z || !h || !w1 || !w2 || !dxp)) return LZ_EINVAL;
    return shape->dtype == LZ_F32
               ? generic_ffn_backward<float>(dyp, xp, z, h, slot_offsets, w1, w2, shape, dxp, dw1, dw2, accumulate,
                                             gw, tables_built, in_pass, (hipStream_t)stream)
               : generic_ffn_backward<uint16_t>(dyp, xp, z, h, slot_offsets, w1, w2, shape, dxp, dw1, dw2,
                                                accumulate, gw, tables_built, in_pass, (hipStream_t)stream);
  }
  TrainWorkspace w;
  const int32_t rc = check_train(shape, ws, ws_bytes, &w);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  const int S = shape->N * shape->c;
  if (!dw1 || !dw2 || !slot_offsets) return LZ_EINVAL;
  if (!aligned16(dw1) || !aligned16(dw2)) return LZ_EINVAL;
  if (P > 0 && (!dyp || !xp || !z || !h || !w1 || !w2 || !dxp)) return LZ_EINVAL;
  if (P > 0 && (!aligned16(dyp) || !aligned16(xp) || !aligned16(z) || !aligned16(h) || !aligned16(dxp) ||
                !aligned16(w1) || !aligned16(w2)))
    return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int d = shape->d, ffn = shape->ffn, n1 = w.n1;
  const bool swiglu = shape->act == LZ_SWIGLU;

  const int n_ffn = ceil_div(ffn, BN), n_d = ceil_div(d, BN), n_n1 = ceil_div(n1, BN);
  const long long rows_w2 = (long long)S * ffn, rows_w1 = (long long)S * d;
  const UnitTable u_ffn = carve_units(w.units_ffn, P, S, n_ffn), u_d = carve_units(w.units_d, P, S, n_d);
  const UnitTable u_w2 = carve_units(w.units_w2, rows_w2, S, n_d), u_w1 = carve_units(w.units_w1, rows_w1, S, n_n1);
  const bool pair = in_pass && pair_wgrads(shape);
  int32_t r = tables_built ? LZ_OK : launch_build_tiles(slot_offsets, S, ::backward_tables(w, shape, accumulate, pair), st);
  if (r != LZ_OK) return r;

  if (P > 0) {
    // dH = dyp W2^T    (W2 [ffn, d]: contraction along its rows)
    if ((r = gemm_nt((const uint16_t*)dyp, (const uint16_t*)w2, w.dh, P, d, ffn, u_ffn, w.narrow_ffn, w, S, st)) != LZ_OK) return r;
    // dZ = dH * act'(Z)
    const int ffn_vec = ffn / 8;
    const unsigned blocks = (unsigned)((P * ffn_vec + 255) / 256);
    if (swiglu)
      hipLaunchKernelGGL(act_backward_kernel<true>, dim3(blocks), dim3(256), 0, st, (const u32x4*)w.dh,
                         (const u32x4*)z, P, ffn_vec, (u32x4*)w.dz);
    else
      hipLaunchKernelGGL(act_backward_kernel<false>, dim3(blocks), dim3(256), 0, st, (const u32x4*)w.dh,
                         (const u32x4*)z, P, ffn_vec, (u32x4*)w.dz);
    if ((r = lz::launch_status()) != LZ_OK) return r;
    // dxp = dZ W1^T    (W1 [d, n1])
    if ((r = gemm_nt(w.dz, (const uint16_t*)w1, (uint16_t*)dxp, P, n1, d, u_d, w.narrow_d, w, S, st)) != LZ_OK) return r;
  }
  // dW2[s] = H_s^T dyp_s  [ffn, d],   dW1[s] = xp_s^T dZ_s  [d, n1]
  uint16_t* const none = nullptr;
  return gemm_wgrads(wgrad_args((const uint16_t*)h, (const uint16_t*)dyp, accumulate ? none : (uint16_t*)dw2,
                                accumulate ? (float*)dw2 : nullptr, S, ffn, d, u_w2),
                     wgrad_args((const uint16_t*)xp, w.dz, accumulate ? none : (uint16_t*)dw1, accumulate ? (float*)dw1 : nullptr, S, d,
                                n1, u_w1),
                     P, accumulate, pair, st);
}

extern "C" int32_t lz_ffn_backward(const void* dyp, const void* xp, const void* z, const void* h,
                                   const int32_t* slot_offsets, const void* w1, const void* w2,
                                   const lz_shape* shape, void* dxp, void* dw1, void* dw2, void* ws,
                                   size_t ws_bytes, void* stream) {
  return lz::ffn_backward(shape, lz::FfnBackward{dyp, xp, z, h, w1, w2, dxp, dw1, dw2}, slot_offsets, false, ws, ws_bytes, false, false,
                          stream);
}

extern "C" int32_t lz_ffn_backward_accumulate(const void* dyp, const void* xp, const void* z, const void* h,
                                              const int32_t* slot_offsets, const void* w1, const void* w2,
                                              const lz_shape* shape, void* dxp, float* dw1_acc, float* dw2_acc,
                                              void* ws, size_t ws_bytes, void* stream) {
  return lz::ffn_backward(shape, lz::FfnBackward{dyp, xp, z, h, w1, w2, dxp, dw1_acc, dw2_acc}, slot_offsets, true, ws, ws_bytes, false,
                          false, stream);
}

namespace {

// 16-byte aligned tensors whose slots are whole 16-byte vectors; elems1 = 0: one matrix
template <typename Elem>
int32_t reduce_vectors(const void* dw_slot0, int64_t elems0, void* dw0, const void* dw_slot1, int64_t elems1, void* dw1,
                       const int32_t* slot_expert, int32_t S, int32_t E, void* stream) {
  auto part = [](const void* in, int64_t elems, void* out) { return ReducePart{(const u32x4*)in, (u32x4*)out, elems / (16 / (int)sizeof(Elem))}; };
  const ReducePart p0 = part(dw_slot0, elems0, dw0), p1 = part(dw_slot1, elems1, dw1);
  const long long blocks0 = (p0.vec_per_slot + 255) / 256, blocks = blocks0 + (p1.vec_per_slot + 255) / 256;
  if (blocks > 0x7FFFFFFFll) return LZ_ESHAPE;
  auto* kern = reduce_replicas_kernel<Elem, kReduceAhead>;
  if constexpr (sizeof(Elem) == 4)
    if (E <= kReduceFewExperts && blocks * E < kReduceFewBlocks) kern = reduce_replicas_kernel<Elem, kReduceAheadFew>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)E), dim3(256), 0, (hipStream_t)stream, p0, p1, (unsigned)blocks0, slot_expert, S);
  return lz::launch_status();
}

}  // namespace

int32_t lz::reduce_pair(const lz_shape* s, const lz_layer_buffers& b, int64_t elems1, int64_t elems2, void* stream) {
  const int S = s->N * s->c, per = s->dtype == LZ_F32 ? 4 : 8;
  const bool whole = elems1 % per == 0 && elems2 % per == 0 && aligned16(b.dw1_slot) && aligned16(b.dw2_slot) && aligned16(b.dw1) &&
                     aligned16(b.dw2) && (elems1 + elems2) / per + 512 < 1ll << 32;  // a grid's threads in x
  if (whole && b.dw1_slot && b.dw2_slot && b.dw1 && b.dw2 && b.slot_expert)
    return s->dtype == LZ_F32
               ? reduce_vectors<float>(b.dw1_slot, elems1, b.dw1, b.dw2_slot, elems2, b.dw2, b.slot_expert, S, s->E, stream)
               : reduce_vectors<uint16_t>(b.dw1_slot, elems1, b.dw1, b.dw2_slot, elems2, b.dw2, b.slot_expert, S, s->E, stream);
  const int32_t rc = lz_reduce_replica_grads_dtype(b.dw1_slot, b.slot_expert, S, s->E, elems1, s->dtype, b.dw1, stream);
  if (rc != LZ_OK) return rc;
  return lz_reduce_replica_grads_dtype(b.dw2_slot, b.slot_expert, S, s->E, elems2, s->dtype, b.dw2, stream);
}

extern "C" int32_t lz_reduce_replica_grads(const void* dw_slot, const int32_t* slot_expert, int32_t S, int32_t E,
                                           int64_t elems_per_slot, void* dw, void* stream) {
  if (S < 1 || E < 1 || E > 65535 || elems_per_slot < 0 || elems_per_slot % 8 != 0) return LZ_ESHAPE;
  if (elems_per_slot == 0) return LZ_OK;
  if (!dw_slot || !slot_expert || !dw || !aligned16(dw_slot) || !aligned16(dw)) return LZ_EINVAL;
  return reduce_vectors<uint16_t>(dw_slot, elems_per_slot, dw, nullptr, 0, nullptr, slot_expert, S, E, stream);
}

extern "C" int32_t lz_reduce_replica_grads_dtype(const void* dw_slot, const int32_t* slot_expert, int32_t S,
                                                 int32_t E, int64_t elems_per_slot, int32_t dtype, void* dw,
                                                 void* stream) {
  if (dtype != LZ_F32 && dtype != LZ_BF16) return LZ_ESHAPE;
  if (dtype == LZ_BF16 && elems_per_slot % 8 == 0 && aligned16(dw_slot) && aligned16(dw))
    return lz_reduce_replica_grads(dw_slot, slot_expert, S, E, elems_per_slot, dw, stream);
  if (S < 1 || E < 1 || E > 65535 || elems_per_slot < 0) return LZ_ESHAPE;
  if (elems_per_slot == 0) return LZ_OK;
  if (!dw_slot || !slot_expert || !dw) return LZ_EINVAL;
  if (dtype == LZ_F32 && elems_per_slot % 4 == 0 && aligned16(dw_slot) && aligned16(dw))
    return reduce_vectors<float>(dw_slot, elems_per_slot, dw, nullptr, 0, nullptr, slot_expert, S, E, stream);
  if ((elems_per_slot + 255) / 256 > 0x7FFFFFFFll) return LZ_ESHAPE;
  const dim3 grid((unsigned)((elems_per_slot + 255) / 256), (unsigned)E);
  if (dtype == LZ_F32)
    hipLaunchKernelGGL(reduce_replicas_generic_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream,
                       (const float*)dw_slot, slot_expert, S, (long long)elems_per_slot, (float*)dw);
  else
    hipLaunchKernelGGL(reduce_replicas_generic_kernel<uint16_t>, grid, dim3(256), 0, (hipStream_t)stream,
                       (const uint16_t*)dw_slot, slot_expert, S, (long long)elems_per_slot, (uint16_t*)dw);
  return lz::launch_status();
}
