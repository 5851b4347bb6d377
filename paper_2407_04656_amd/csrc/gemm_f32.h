// Grouped GEMM with fp32 products on the gfx950 matrix cores (v_mfma_f32_16x16x4_f32): fp32 tensors, and the
// bf16 tensors the kernel of gemm_mfma.h cannot load (rows or pointers that are no whole 16-byte pieces).  Large fp32
// forwards and weight gradients run on the kernel of gemm_split.h.
// Device code shared by the forward and the backward, not part of the C ABI.
//
//   C[rows of a slot, n] = epi( sum_k A(row, k) * W[slot](n, k) )      rows and W, or a slot's k range, ragged
//
// fp32 MFMAs need little operand bandwidth (a 16x16x4 step holds the pipe for 32 cycles against 8 bytes read
// per lane), so tiles are small and several workgroups share a CU; what bounds the kernel is the matrix pipe
// where there are enough tiles and the latency of the few K steps where there are not.  A workgroup's tile is
// 32 rows (ragged slots waste little) x 32 NW columns, NW = 4 or 1 waves side by side; the 4 / NW waves that
// share a column range split each stage's k and add up through LDS at the end.  f32_waves() below picks NW.
// Operands go global -> registers -> LDS, fetched two stages ahead (two LDS stages, one barrier a stage), in
// 4-element pieces: 16-byte accesses (VEC) or single elements for odd sizes and alignments.  A lane's four
// MFMAs of a 16-k block take k = 4 (lane / 16) + i: any order of k serves as long as both operands agree,
// and a k-contiguous tile is then read with one ds_read_b128.
// Against 64 x 64 x 16 tiles on fp32 FMAs: a training step of T = 1024, d = 512, ffn = 2048, 16 slots 1603 -> 433 us
// (4.3 GFLOP a GEMM: 54-63 us), the forward of T = 256, d = 128, ffn = 256 99 -> 56 us; relative errors against
// fp64 0.2-0.6e-6, 0.36-0.94e-6 before (shorter chains of roundings).
#pragma once
#include "gemm_mfma.h"

namespace {

// dZ = dH * act'(Z) in the epilogue of dH = dyp W2^T: C is dZ, Z is read
enum { EPI_DGELU = 6, EPI_DSWIGLU = 7 };

constexpr int kF32Rows = 32;  // rows of a tile

struct F32Args {
  const void* A;        // [rows, K] or, k-major, [k rows, lda]
  const void* W;        // per slot [n, K] or, k-major, [K, ldw];  weight gradients: [k rows, ldw]
  void* C;              // [rows, ldc]
  void* Z;              // pre-activations [rows, ldz] (written by *_KEEP, read by EPI_D*)
  float* Cacc;          // EPI_ACCUM
  int K;                // contraction length (weight gradients: from slot_offsets)
  int lda, ldw, ldc, ldz;
  long long w_slot;     // elements between the weights of two slots
  int n_out;            // result columns
  int n_tiles;          // column tiles
  int slots, m_tiles;   // weight gradients: row tiles of a slot's result
  int ffn;              // gated epilogues: columns between the gate and the up half
  TileTable t, t_split;  // of the kernel here; of gemm_split.h
  const int32_t* gather;  // row r of A is row gather[r] / gather_k (forward's first GEMM), or nullptr
  int gather_k;
  long long gather_T;     // rows of x (first GEMM, gathered or not), 0 for the others
  const int32_t* slot_offsets;  // weight gradients
  long long P;
  int m_rows;           // weight gradients: rows of one slot's result
};

template <typename Elem>
__device__ __forceinline__ float load_elem(const Elem* p);
template <>
__device__ __forceinline__ float load_elem<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float load_elem<uint16_t>(const uint16_t* p) { return lz::bf16_to_f32(*p); }
template <typename Elem>
__device__ __forceinline__ void store_elem(Elem* p, float v);
template <>
__device__ __forceinline__ void store_elem<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_elem<uint16_t>(uint16_t* p, float v) { *p = lz::f32_to_bf16(v); }
template <typename Elem>
__device__ __forceinline__ float stored(float v);  // the value that is stored
template <>
__device__ __forceinline__ float stored<float>(float v) { return v; }
template <>
__device__ __forceinline__ float stored<uint16_t>(float v) { return lz::bf16_to_f32(lz::f32_to_bf16(v)); }

__device__ __forceinline__ float gelu_exact(float v) { return 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad_exact(float v) {
  const float cdf = 0.5f * (1.0f + erff(v * 0.70710678118654752440f));
  return fmaf(v * 0.3989422804014327f, expf(-0.5f * v * v), cdf);
}
__device__ __forceinline__ float sigmoid_exact(float v) { return 1.0f / (1.0f + expf(-v)); }

// Elements [0, n) of a 4-element piece at p (n <= 0: none, zeros), `safe` any readable piece.
template <typename Elem, bool VEC>
__device__ __forceinline__ f32x4 load_piece(const Elem* p, const Elem* safe, int n) {
  f32x4 v;
  if constexpr (VEC) {  // float, whole pieces only
    v = *(const f32x4*)(n > 0 ? p : safe);
    if (n <= 0) v = f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float e = load_elem<Elem>(j < n ? p + j : safe);
      v[j] = j < n ? e : 0.f;
    }
  }
  return v;
}
template <typename Elem>
struct Raw4 {
  Elem e[4];
};

template <typename Elem, bool VEC>
__device__ __forceinline__ void store_piece(Elem* p, const f32x4& v, int n) {
  if constexpr (VEC) {
    if (n > 0) *(f32x4*)p = v;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < n) store_elem<Elem>(p + j, v[j]);
  }
}

// Epilogue on 4 consecutive columns of one row.  col is the result column; gated: v and u belong to it.
template <typename Elem, int EPI, bool WGRAD, bool VEC>
__device__ __forceinline__ void f32_emit(const F32Args& a, int slot, int row, int row_end, int col, const f32x4& v,
                                         const f32x4& u) {
  constexpr bool kGated = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP;
  const int n = row < row_end ? a.n_out - col : 0;
  const size_t grow = WGRAD ? (size_t)slot * a.m_rows + row : (size_t)row;
  if (n <= 0) return;
  Elem* const c = (Elem*)a.C + grow * a.ldc + col;
  if constexpr (EPI == EPI_ACCUM) {
    float* const s = a.Cacc + grow * a.ldc + col;
    store_piece<float, VEC>(s, load_piece<float, VEC>(s, a.Cacc, n) + v, n);
    return;
  }
  if constexpr (EPI == EPI_GELU_KEEP || EPI == EPI_SWIGLU_KEEP) {
    Elem* const z = (Elem*)a.Z + grow * a.ldz + col;
    store_piece<Elem, VEC>(z, v, n);
    if constexpr (kGated) store_piece<Elem, VEC>(z + a.ffn, u, n);
  }
  f32x4 o = v, o2;
  if constexpr (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) {
    const Elem* const z = (const Elem*)a.Z + grow * a.ldz + col;
    const f32x4 zg = load_piece<Elem, VEC>(z, (const Elem*)a.Z, n);
    if constexpr (EPI == EPI_DGELU) {
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = v[j] * gelu_grad_exact(zg[j]);
    } else {
      const f32x4 zu = load_piece<Elem, VEC>(z + a.ffn, (const Elem*)a.Z, n);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float sg = sigmoid_exact(zg[j]);
        o[j] = v[j] * zu[j] * (sg * fmaf(zg[j], 1.0f - sg, 1.0f));
        o2[j] = v[j] * (zg[j] * sg);
      }
      store_piece<Elem, VEC>(c + a.ffn, o2, n);
    }
  } else if constexpr (EPI == EPI_GELU || EPI == EPI_GELU_KEEP) {
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = gelu_exact(EPI == EPI_GELU ? v[j] : stored<Elem>(v[j]));
  } else if constexpr (kGated) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float g = EPI == EPI_SWIGLU ? v[j] : stored<Elem>(v[j]), w = EPI == EPI_SWIGLU ? u[j] : stored<Elem>(u[j]);
      o[j] = g * sigmoid_exact(g) * w;
    }
  }
  store_piece<Elem, VEC>(c, o, n);
}

// WGRAD: both operands k-major, C = [S, m_rows, n_out]; otherwise the rows of the tile table, W k-major or not
// by WKM.  Persistent: the grid is what fits the chip at once and a workgroup strides over the tiles, columns
// fastest (an XCD meets the same columns of a slot's weights again).  Against
// one workgroup per tile: 4-8 % on the 32 x 32 tiles, level on the wide ones.
// PAIR: two of them in one launch, the tiles of one behind those of the other.
template <bool PAIR>
struct F32Launch {
  F32Args gemm[PAIR ? 2 : 1];
  // a weight gradient's tiles
  static __device__ __forceinline__ long long tiles(const F32Args& a) { return (long long)a.slots * a.m_tiles * a.n_tiles; }
};
template <typename Elem, int EPI, bool WGRAD, bool WKM, int NW, bool VEC, bool PAIR>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Launch<PAIR> launch) {
  constexpr int KSPLIT = 4 / NW, TM = kF32Rows, TN = 32 * NW, TK = NW == 4 ? 32 : 64;
  constexpr int kBlocks = TK / KSPLIT / 16;  // 16-k blocks of a stage per wave
  constexpr bool kGated = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP;
  constexpr bool AKM = WGRAD;
  // LDS pitches in floats: k-contiguous [row][k] reads 16 rows x 16 bytes at a time, k-major [k][col] 4 k x 16
  // columns; both cover the 64 banks once with 4 floats of padding
  constexpr int kPitchA = AKM ? TM + 4 : TK + 4, kPitchW = WKM ? TN + 4 : TK + 4;
  constexpr int kSizeA = AKM ? TK * kPitchA : TM * kPitchA, kSizeW = WKM ? TK * kPitchW : TN * kPitchW;
  constexpr int kPiecesA = TM * TK / 4 / 256, kPiecesW = TN * TK / 4 / 256;  // per thread
  __shared__ __attribute__((aligned(16))) float lds[2 * (kSizeA + kSizeW)];
  static_assert(2 * (kSizeA + kSizeW) >= KSPLIT * 32 * (TN + 4), "the K split's partial sums reuse the stages");

  constexpr int kOutCols = kGated ? TN / 2 : TN;
  static_assert(WGRAD || !PAIR, "pairs are of weight gradients");
  const F32Args* const args = launch.gemm;
  const long long n_first = WGRAD ? F32Launch<PAIR>::tiles(args[0]) : (long long)args[0].t.header[0] * args[0].n_tiles;
  const long long n_all = n_first + (PAIR ? F32Launch<PAIR>::tiles(args[PAIR ? 1 : 0]) : 0);
  for (long long t = blockIdx.x; t < n_all; t += gridDim.x) {
    const int part = PAIR && t >= n_first ? 1 : 0;
    // By value: a field read through an address that is chosen here would be loaded anew in every loop (odd sizes, whose pieces are
    // fetched by elements: both gradients of 14091 tokens, 64 slots, 137 x 128 SwiGLU cost a training step of 431 us 64 more).
    const F32Args a = PAIR && part ? args[PAIR ? 1 : 0] : args[0];
    const long long tile = t - (part ? n_first : 0);
    const int row_tile = int(tile / a.n_tiles), n0 = int(tile % a.n_tiles) * kOutCols;
    int slot, row0, row_end, K = a.K;
    const Elem* A = (const Elem*)a.A;
    const Elem* W = (const Elem*)a.W;
    if constexpr (WGRAD) {
      slot = row_tile / a.m_tiles;
      row0 = row_tile % a.m_tiles * TM;
      row_end = a.m_rows;
      long long lo, hi;
      clip_slot(a.slot_offsets, slot, a.P, &lo, &hi);
      lo = __builtin_amdgcn_readfirstlane((int)lo);
      K = __builtin_amdgcn_readfirstlane((int)(hi)) - (int)lo;
      A += (size_t)lo * a.lda;
      W += (size_t)lo * a.ldw;
      if (EPI == EPI_ACCUM && K == 0) continue;
    } else {
      slot = __builtin_amdgcn_readfirstlane(a.t.slot[row_tile]);  // the same in every lane: buffer bases are scalar
      row0 = __builtin_amdgcn_readfirstlane(a.t.row0[row_tile]);
      row_end = __builtin_amdgcn_readfirstlane(a.t.row_end[row_tile]);
      W += (size_t)slot * a.w_slot;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wn = wave % NW, wk = wave / NW;

    // ---- this thread's pieces of a stage: element offset from the tile's (uniform) base at k = 0, k of the first
    // element, valid elements (0: none; k-contiguous pieces also end with K), LDS place
    const Elem* const baseA = AKM ? A + row0 : a.gather != nullptr ? A : A + (size_t)row0 * a.lda;
    const Elem* const baseW = WKM ? W + n0 : W + (size_t)n0 * a.ldw;
    long long pa[kPiecesA], pw[kPiecesW];
    int ka[kPiecesA], kw[kPiecesW], na[kPiecesA], nw[kPiecesW], la[kPiecesA], lw[kPiecesW];
#pragma unroll
    for (int i = 0; i < kPiecesA; ++i) {
      const int c = tid + 256 * i;
      if constexpr (AKM) {
        const int col = c % (TM / 4) * 4;
        ka[i] = c / (TM / 4);
        na[i] = row_end - (row0 + col);
        pa[i] = (long long)ka[i] * a.lda + col;
        la[i] = ka[i] * kPitchA + col;
      } else {
        const int r = c / (TK / 4), row = row0 + r;
        ka[i] = c % (TK / 4) * 4;
        long long src = r;
        bool ok = row < row_end;
        if (a.gather != nullptr) {
          const long long pair = ok ? a.gather[row] : -1;
          ok = pair >= 0 && pair < a.gather_T * a.gather_k;
          src = pair / a.gather_k;
        }
        na[i] = ok ? 4 : 0;
        pa[i] = (ok ? src : 0) * a.lda + ka[i];
        la[i] = r * kPitchA + ka[i];
      }
    }
#pragma unroll
    for (int i = 0; i < kPiecesW; ++i) {
      const int c = tid + 256 * i;
      if constexpr (WKM) {
        // gated: every 32 tile columns are 16 gate columns and the 16 up columns of the same outputs
        const int cc = c % (TN / 4) * 4;
        const int col = kGated ? (cc >> 5) * 16 + (cc & 15) : cc;
        kw[i] = c / (TN / 4);
        nw[i] = a.n_out - (n0 + col);
        pw[i] = (long long)kw[i] * a.ldw + col + (kGated && (cc & 16) ? a.ffn : 0);
        lw[i] = kw[i] * kPitchW + cc;
      } else {
        const int r = c / (TK / 4);
        kw[i] = c % (TK / 4) * 4;
        nw[i] = n0 + r < a.n_out ? 4 : 0;
        pw[i] = (long long)r * a.ldw + kw[i];
        lw[i] = r * kPitchW + kw[i];
      }
    }
    // A fetched piece stays raw in registers until it goes to LDS, so that nothing waits for it earlier.  VEC:
    // buffer loads; a piece that is not there gets an offset outside the descriptor and arrives as zeros (the
    // host checked that a stage spans less than 2 GiB).  Otherwise single elements from clamped addresses, masked
    // on the way to LDS.
    using Piece = typename std::conditional<VEC, u32x4_t, Raw4<Elem>>::type;
    Piece ra[2][kPiecesA], rw[2][kPiecesW];
    auto valid_a = [&](int i, int k0) {
      const int left = K - k0 - ka[i];
      return AKM ? (left > 0 ? na[i] : 0) : (na[i] > 0 ? left : 0);
    };
    auto valid_w = [&](int i, int k0) {
      const int left = K - k0 - kw[i];
      return WKM ? (left > 0 ? nw[i] : 0) : (nw[i] > 0 ? left : 0);
    };
    auto fetch = [&](auto set_c, int k0) {
      constexpr int set = decltype(set_c)::value;
      const Elem* const stA = baseA + (AKM ? (size_t)k0 * a.lda : (size_t)k0);
      const Elem* const stW = baseW + (WKM ? (size_t)k0 * a.ldw : (size_t)k0);
      if constexpr (VEC) {
        const auto bufA = __builtin_amdgcn_make_buffer_rsrc((void*)stA, 0, 0x7FFFFFFF, 0x00020000);
        const auto bufW = __builtin_amdgcn_make_buffer_rsrc((void*)stW, 0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
        for (int i = 0; i < kPiecesA; ++i)
          ra[set][i] = __builtin_amdgcn_raw_buffer_load_b128(bufA, valid_a(i, k0) > 0 ? (int)pa[i] * 4 : (int)0x80000000, 0, 0);
#pragma unroll
        for (int i = 0; i < kPiecesW; ++i)
          rw[set][i] = __builtin_amdgcn_raw_buffer_load_b128(bufW, valid_w(i, k0) > 0 ? (int)pw[i] * 4 : (int)0x80000000, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < kPiecesA; ++i) {
          const int n = valid_a(i, k0);
#pragma unroll
          for (int j = 0; j < 4; ++j) ra[set][i].e[j] = *(j < n ? stA + pa[i] + j : (const Elem*)a.A);
        }
#pragma unroll
        for (int i = 0; i < kPiecesW; ++i) {
          const int n = valid_w(i, k0);
#pragma unroll
          for (int j = 0; j < 4; ++j) rw[set][i].e[j] = *(j < n ? stW + pw[i] + j : (const Elem*)a.W);
        }
      }
    };
    auto put = [&](auto set_c, int k0) {
      constexpr int set = decltype(set_c)::value;
      float* const sa = lds + set * (kSizeA + kSizeW);
      auto value = [&](const Piece& p, [[maybe_unused]] int n) {
        if constexpr (VEC) return __builtin_bit_cast(f32x4, p);
        else {
          f32x4 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = j < n ? load_elem<Elem>(&p.e[j]) : 0.f;
          return v;
        }
      };
#pragma unroll
      for (int i = 0; i < kPiecesA; ++i) *(f32x4*)(sa + la[i]) = value(ra[set][i], valid_a(i, k0));
#pragma unroll
      for (int i = 0; i < kPiecesW; ++i) *(f32x4*)(sa + kSizeA + lw[i]) = value(rw[set][i], valid_w(i, k0));
    };
    f32x4 acc[2][2] = {};  // [weight fragment][activation fragment]
    const int frag = lane & 15, quad = lane >> 4;
    auto compute = [&](int stage) {
      const float* const sa = lds + stage * (kSizeA + kSizeW);
      const float* const sw = sa + kSizeA;
#pragma unroll
      for (int kb = 0; kb < kBlocks; ++kb) {
        const int k = (wk * kBlocks + kb) * 16 + 4 * quad;
        f32x4 x[2], w[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          const int ax = f * 16 + frag, wx = wn * 32 + f * 16 + frag;
          if constexpr (AKM) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[f][i] = sa[(k + i) * kPitchA + ax];
          } else {
            x[f] = *(const f32x4*)(sa + ax * kPitchA + k);
          }
          if constexpr (WKM) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[f][i] = sw[(k + i) * kPitchW + wx];
          } else {
            w[f] = *(const f32x4*)(sw + wx * kPitchW + k);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int m = 0; m < 2; ++m)
              acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[n][i], x[m][i], acc[n][m], 0, 0, 0);
      }
    };

    const int stages = (K + TK - 1) / TK;
    {
      using S0 = std::integral_constant<int, 0>;
      using S1 = std::integral_constant<int, 1>;
      // stage s is in LDS, stage s + 1 in registers or on its way; a fetch past the end has no valid piece
      auto step = [&](int s, auto cur, auto next) {
        fetch(cur, (s + 2) * TK);
        compute(decltype(cur)::value);
        put(next, (s + 1) * TK);  // this LDS stage was last read before the previous barrier
        __syncthreads();
      };
      // Rows of one stage: no fetches past the end (8 columns to 8, 200000 rows, 128 slots: 104 -> 71 us a forward).
      // Leaving them out of the loop below by a test costs the longer rows up to 8 %, weight gradients half.
      if (!WGRAD && stages == 1) {
        fetch(S0{}, 0);
        put(S0{}, 0);
        __syncthreads();
        compute(0);
        __syncthreads();
      } else if (stages > 0) {
        fetch(S0{}, 0);
        fetch(S1{}, TK);
        put(S0{}, 0);
        __syncthreads();
        for (int s = 0; s < stages; s += 2) {
          step(s, S0{}, S1{});
          if (s + 1 < stages) step(s + 1, S1{}, S0{});
        }
      }
    }

    auto emit = [&](int r, int col, const f32x4& v, const f32x4& u) {
      f32_emit<Elem, EPI, WGRAD, VEC>(a, slot, row0 + r, row_end, col, v, u);
    };
    // lane l of block (n, m) holds row 16 m + l % 16 and the columns 16 n + 4 (l / 16) + 0..3
    const int out_n = n0 + wn * (kGated ? 16 : 32);
    if constexpr (KSPLIT == 1) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int r = m * 16 + frag;
        if constexpr (kGated) emit(r, out_n + 4 * quad, acc[0][m], acc[1][m]);
        else {
          emit(r, out_n + 4 * quad, acc[0][m], acc[0][m]);
          emit(r, out_n + 16 + 4 * quad, acc[1][m], acc[1][m]);
        }
      }
    } else {
      // partial sums [k part][row][column] (the stages are dead: the loop ends with a barrier), then 4 columns each
      constexpr int kPitch = TN + 4;
      float* const mine = lds + wk * 32 * kPitch + wn * 32;
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int m = 0; m < 2; ++m) *(f32x4*)(mine + (m * 16 + frag) * kPitch + n * 16 + 4 * quad) = acc[n][m];
      __syncthreads();
      auto sum = [&](int r, int c) {
        f32x4 v = *(const f32x4*)(lds + r * kPitch + c);
#pragma unroll
        for (int p = 1; p < KSPLIT; ++p) v += *(const f32x4*)(lds + (p * 32 + r) * kPitch + c);
        return v;
      };
      if constexpr (kGated) {
        if (tid < 32 * TN / 8) {
          const int r = tid / (TN / 8), c = tid % (TN / 8) * 4;  // c: result column of the tile
          const int g = (c >> 4) * 32 + (c & 15);
          emit(r, n0 + c, sum(r, g), sum(r, g + 16));
        }
      } else {
#pragma unroll
        for (int q = 0; q < NW; ++q) {
          const int i = tid + 256 * q, r = i / (TN / 4), c = i % (TN / 4) * 4;
          const f32x4 v = sum(r, c);
          emit(r, n0 + c, v, v);
        }
      }
      __syncthreads();  // the partial sums are read: the next tile may fill the stages
    }
  }
}

// Waves side by side: four where their tiles fill the chip (three workgroups on each of 256 CUs; tiles32 = tiles
// of 32 x 32), else one.  Measured at 72 row tiles, K x columns 512 x 2048 (4608 tiles32): 4 waves 60 us,
// 1 wave 63; 2048 x 512 (1152): 88 and 58; weight gradients of 16384: 58 and 81.  Two were never the best.
inline int f32_waves(long long tiles32) { return tiles32 >= 4 * 768 ? 4 : 1; }

// 16-byte accesses on fp32 tensors, and a stage's pieces within 31-bit offsets.
inline bool whole_pieces(const F32Args& a) {
  const long long stage_bytes = 128ll * 4 * (a.lda > a.ldw ? a.lda : a.ldw);  // at most 128 rows of either operand
  return stage_bytes < (1ll << 31) && (!a.gather || a.gather_T * a.lda * 4 < (1ll << 31)) &&
         a.K % 4 == 0 && a.lda % 4 == 0 && a.ldw % 4 == 0 && a.ldc % 4 == 0 && a.ldz % 4 == 0 &&
         a.n_out % 4 == 0 && a.ffn % 4 == 0 && a.m_rows % 4 == 0 && a.w_slot % 4 == 0 && aligned16(a.A) &&
         aligned16(a.W) && aligned16(a.C) && aligned16(a.Z) && aligned16(a.Cacc);
}

template <typename Elem, int EPI, bool WGRAD, bool WKM, int NW, bool PAIR = false>
void launch_f32_waves(const F32Launch<PAIR>& a, dim3 grid, bool vec, hipStream_t st) {
  if constexpr (sizeof(Elem) == 4) {
    if (vec) {
      hipLaunchKernelGGL((gemm_f32_kernel<Elem, EPI, WGRAD, WKM, NW, true, PAIR>), grid, dim3(256), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_f32_kernel<Elem, EPI, WGRAD, WKM, NW, false, PAIR>), grid, dim3(256), 0, st, a);
}

// workgroups that the LDS of the chip holds; 0 on an error
inline long long f32_resident(int nw) { return (long long)device_cus() * (nw == 1 ? 4 : 3); }

// rows32: 32-row tiles expected to hold rows; max_rows32: those the grid may have to cover
template <typename Elem, int EPI, bool WGRAD, bool WKM>
int32_t launch_f32(F32Args a, long long rows32, long long max_rows32, hipStream_t st) {
  const int cols = a.n_out * (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP ? 2 : 1);
  const int nw = f32_waves(rows32 * ceil_div(cols, 32));
  a.n_tiles = ceil_div(cols, 32 * nw);
  const long long resident = f32_resident(nw);
  if (resident == 0) return LZ_EHIP;
  const dim3 grid((unsigned)(max_rows32 * a.n_tiles < resident ? max_rows32 * a.n_tiles : resident));
  const bool vec = whole_pieces(a);
  if (nw == 4) launch_f32_waves<Elem, EPI, WGRAD, WKM, 4>(F32Launch<false>{{a}}, grid, vec, st);
  else launch_f32_waves<Elem, EPI, WGRAD, WKM, 1>(F32Launch<false>{{a}}, grid, vec, st);
  return lz::launch_status();
}

}  // namespace
