// Grouped fp32 GEMM on the bf16 matrix cores of gfx950: every fp32 operand is split into three bf16 numbers whose sum
// it is exactly, and all but the smallest of the nine products are summed in fp32.  The forward's GEMMs and the weight
// gradients of fp32 tensors in whole 16-byte pieces, where use_split() below says so; the others run on the kernel of
// gemm_f32.h.  Device code shared by the forward and the backward, not part of the C ABI.
//
//   C[rows of a slot, n] = epi( sum_k A(row, k) * W[slot](k, n) )      rows, or a slot's k range, ragged
//
// Why: v_mfma_f32_16x16x4_f32 does 64 flops a cycle and SIMD, v_mfma_f32_16x16x32_bf16 1024: eight of them twice the
// fp32 instruction.  The split a = a0 + a1 + a2: a0 the upper 16 bits, a1 the rest rounded to bf16, a2 what is then left
// (at most 8 bits, exact; G. Henry, P. Tang and A. Heinecke, 2019, arXiv 1904.06376).  Left out is a2 w2, below 2^-30 of
// a product (with a1 w2 and a2 w1 left out too, six instructions, a product was off by up to 4.4 2^-24, which shows in
// sums of one).  The seven small products of 32 k are summed from zero and added to the accumulator of a0 w0 once, which
// is thus rounded twice in 32 k where the fp32 instruction rounds it 8 times or more.  Errors against fp64 in 2^-24 of
// the products' magnitudes, rms of sums of 1, 4, 32 and 1183 of them: 0.42, 0.29, 0.18 and 0.12, by the fp32
// instruction 0.42, 0.45, 0.47 and 0.47.
//
// Tile: 64 rows x 128 columns, stages of 64 k, four waves: two column ranges of 64 times two halves of each stage's k,
// added through LDS at the end.  A goes global -> registers (one stage ahead) -> split -> LDS, [row][plane][k] with a
// pitch of 25 x 16 bytes, so that a fragment's 16 rows (one ds_read_b128 a lane) cover the banks once.  W no other wave
// needs: it goes from global straight to the fragments, a lane loading 4 adjacent columns at its 8 k and splitting the
// pairs of k in place; its four fragments are the columns 4 i + j, j = 0..3, and a lane's accumulators of them are
// adjacent columns again.  Two workgroups share a CU.  What bounds it: the split and the additions (some 400 vector
// instructions to 128 MFMAs a stage) and the latency of a stage.  Tried, with six products: both operands through LDS
// (up projection of 512 x 2048, 16 slots, 2048 rows 53 us against 49), column ranges of one wave (tiles of 64 x 256,
// all k: 54, and 114 against 70 where tiles are few) or of four (64 x 64: 63), one run of tiles per XCD (level,
// gradients 20 % slower), and the data gradients, whose W lies along k (65 us against 58 of the fp32 instruction).
#pragma once
#include "gemm_f32.h"

namespace {

constexpr int kSplitRows = 64, kSplitCols = 128;  // of a tile

// Operands are split at 2^24 times their size: the last bit of an fp32 number is 2^-149 or larger, so none of its parts is then
// below the smallest normal number 2^-126.  Costs 48 multiplications of some 400 vector instructions a stage.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// Two fp32 (scaled) -> the three planes' dwords.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&d)[3]) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  d[0] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
  const float ra = a - __uint_as_float(ua & 0xFFFF0000u), rb = b - __uint_as_float(ub & 0xFFFF0000u);
  d[1] = pack_bf16x2(ra, rb);
  d[2] = pack_bf16x2(ra - __uint_as_float(d[1] << 16), rb - __uint_as_float(d[1] & 0xFFFF0000u));
}

template <int EPI, bool WGRAD, bool PAIR = false>
__global__ __launch_bounds__(256, 2) void gemm_split_kernel(F32Launch<PAIR> launch) {
  constexpr int TM = kSplitRows, TN = kSplitCols, TK = 64;
  constexpr bool kGated = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP;
  constexpr bool AKM = WGRAD;
  constexpr int kPlane = TK * 2, kPitch = 3 * kPlane + 16;  // bytes
  constexpr int kPieces = TM * TK / 4 / 256;  // of A, per thread
  constexpr int kExchange = 4 * 2 * 4 * 64 * 16;  // [wave][row fragment][weight fragment][lane] partial sums
  __shared__ __attribute__((aligned(16))) char lds[TM * kPitch > kExchange ? TM * kPitch : kExchange];

  constexpr int kOutCols = kGated ? TN / 2 : TN;

  const F32Args* const args = launch.gemm;
  const long long n_first = WGRAD ? F32Launch<PAIR>::tiles(args[0]) : (long long)args[0].t.header[0] * args[0].n_tiles;
  const long long n_all = n_first + (PAIR ? F32Launch<PAIR>::tiles(args[PAIR ? 1 : 0]) : 0);
  for (long long t = blockIdx.x; t < n_all; t += gridDim.x) {
    const int part = PAIR && t >= n_first ? 1 : 0;
    const F32Args a = PAIR && part ? args[PAIR ? 1 : 0] : args[0];  // by value, as in gemm_f32_kernel
    const long long tile = t - (part ? n_first : 0);
    // The empty asm keeps the per-lane address arithmetic inside the tile: hoisted out of the loop it would be carried in
    // registers through the stages and spill.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wk = wave >> 1;
    const int frag = lane & 15, quad = lane >> 4;
    const int row_tile = int(tile / a.n_tiles), n0 = int(tile % a.n_tiles) * kOutCols;
    int slot, row0, row_end, K = a.K;
    const float* A = (const float*)a.A;
    const float* W = (const float*)a.W;
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
    // row of A (its index r within the tile) in memory, or -1
    auto source_row = [&](int r) -> long long {
      const int row = row0 + r;
      if (row >= row_end) return -1;
      if (a.gather == nullptr) return r;
      const long long pair = a.gather[row];
      return pair >= 0 && pair < a.gather_T * a.gather_k ? pair / a.gather_k : -1;
    };

    // ---- byte offsets of this thread's pieces of a stage from the tile's (uniform) base at k = 0, or one that is
    // outside every buffer; k of the first element
    constexpr int kNowhere = (int)0x80000000;
    const float* const baseA = AKM ? A + row0 : a.gather != nullptr ? A : A + (size_t)row0 * a.lda;
    const float* const baseW = W + n0;
    // k-major: 4 columns of kPieces consecutive k; otherwise pieces 256 apart in [row][k / 4]
    const int a_group = tid % (TM / 4), a_k = AKM ? tid / (TM / 4) * kPieces : tid % (TK / 4) * 4;
    int pa[AKM ? 1 : kPieces];
    if constexpr (AKM) {
      pa[0] = row0 + 4 * a_group < row_end ? (a_k * a.lda + 4 * a_group) * 4 : kNowhere;
    } else {
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const long long src = source_row((tid + 256 * i) / (TK / 4));
        pa[i] = src >= 0 ? int(src * a.lda + a_k) * 4 : kNowhere;
      }
    }
    // W goes straight to the fragments: this lane's 8 k of 4 adjacent columns.  Gated: the first 32 weight columns of a
    // wave are gates, the others the up projection of the same results.
    const int w_col = kGated ? (wn * 8 + (frag & 1) * 4 + (frag >> 2)) * 4 : (wn * 16 + (frag & 3) * 4 + (frag >> 2)) * 4;
    const int w_k = wk * 32 + quad * 8;
    const int w_at = w_col + (kGated && (frag & 2) ? a.ffn : 0);
    int pw = n0 + w_col < a.n_out ? (w_k * a.ldw + w_at) * 4 : kNowhere;
    u32x4_t ra[kPieces], rw[8];
    // A piece that is not there arrives as zeros: its offset is outside the descriptor, which for a k-major operand
    // ends with row K (the host checked that a stage spans less than 2 GiB).
    auto buffer = [&](const float* base, bool k_major, int ld, int k0) {
      const long long left = (long long)(K - k0) * ld * 4;
      const int bytes = !k_major || left > 0x7FFFFFFF ? 0x7FFFFFFF : left < 0 ? 0 : (int)left;
      return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (k_major ? (size_t)k0 * ld : (size_t)k0)), 0, bytes, 0x00020000);
    };
    auto fetch_a = [&](int k0) {
      const auto buf = buffer(baseA, AKM, a.lda, k0);
      if constexpr (AKM) asm("" : "+v"(pa[0]));  // the sums below are made again in each stage, not kept in registers
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        ra[i] = __builtin_amdgcn_raw_buffer_load_b128(buf, AKM ? pa[0] + i * a.lda * 4 : k0 + a_k < K ? pa[AKM ? 0 : i] : kNowhere, 0, 0);
    };
    auto fetch_w = [&](int k0) {
      const auto buf = buffer(baseW, true, a.ldw, k0);
      asm("" : "+v"(pw));
#pragma unroll
      for (int i = 0; i < 8; ++i) rw[i] = __builtin_amdgcn_raw_buffer_load_b128(buf, pw + i * a.ldw * 4, 0, 0);
    };
    auto put_a = [&]() {
      f32x4 v[kPieces];
#pragma unroll
      for (int i = 0; i < kPieces; ++i) v[i] = __builtin_bit_cast(f32x4, ra[i]) * kSplitScale;
      auto store = [&](char* at, float v0, float v1, float v2, float v3) {
        uint32_t lo[3], hi[3];
        split_pair(v0, v1, lo);
        split_pair(v2, v3, hi);
#pragma unroll
        for (int p = 0; p < 3; ++p) *(uint2*)(at + p * kPlane) = uint2{lo[p], hi[p]};
      };
      if constexpr (AKM) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < kPieces; i += 4)
            store(lds + (j * (TM / 4) + a_group) * kPitch + (a_k + i) * 2, v[i][j], v[i + 1][j], v[i + 2][j], v[i + 3][j]);
      } else {
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
          store(lds + (tid + 256 * i) / (TK / 4) * kPitch + a_k * 2, v[i][0], v[i][1], v[i][2], v[i][3]);
      }
    };

    f32x4 acc[4][4] = {};  // [weight fragment][row fragment]
    const char* const read_a = lds + frag * kPitch + w_k * 2;
    const bool second_half = WGRAD || row0 + 32 < row_end;  // rows 32 to 63 are not all padding
    const int stages = (K + TK - 1) / TK;
    if (stages > 0) {
      fetch_a(0);
      fetch_w(0);
    }
    for (int s = 0; s < stages; ++s) {
      put_a();
      __syncthreads();
      fetch_a((s + 1) * TK);  // past the end: no valid piece
      u32x4_t w[4][3];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          uint32_t d[3];
          split_pair(__uint_as_float(rw[2 * h][j]) * kSplitScale, __uint_as_float(rw[2 * h + 1][j]) * kSplitScale, d);
#pragma unroll
          for (int p = 0; p < 3; ++p) w[j][p][h] = d[p];
        }
      fetch_w((s + 1) * TK);
      auto multiply = [&](int f) {
        bf16x8 x[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) x[p] = *(const bf16x8*)(read_a + f * 16 * kPitch + p * kPlane);
        f32x4 low[4] = {};
#pragma unroll
        for (int term = 0; term < 8; ++term) {
          constexpr int kTermW[8] = {2, 1, 0, 2, 1, 0, 1, 0}, kTermX[8] = {1, 2, 2, 0, 1, 1, 0, 0};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            f32x4& to = term == 7 ? acc[j][f] : low[j];
            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j][kTermW[term]]), x[kTermX[term]], to, 0, 0, 0);
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j][f] += low[j];
      };
      multiply(0);
      multiply(1);
      if (second_half) {
        multiply(2);
        multiply(3);
      }
      __syncthreads();
    }

    // row within the tile and first of the 4 result columns of this lane's accumulators [0..3][f][t]
    auto tile_row = [&](int f) { return AKM ? 4 * frag + f : f * 16 + frag; };
    auto out_col = [&](int t) { return kGated ? (wn * 8 + (t & 1) * 4 + quad) * 4 : (wn * 16 + t * 4 + quad) * 4; };
    // The two waves of a column range exchange two row fragments each and finish the other two: 0 and 1 the wave of the
    // first half of k.  The barrier lies behind the branch, one for all waves.
    f32x4* const mine = (f32x4*)lds + wave * 8 * 64 + lane;
    const f32x4* const theirs = (const f32x4*)lds + (wave ^ 2) * 8 * 64 + lane;
    f32x4 own[2][4];
    auto give = [&](auto f0_c) {
      constexpr int f0 = decltype(f0_c)::value;
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          own[o][j] = acc[j][f0 + o];
          mine[(o * 4 + j) * 64] = acc[j][2 - f0 + o];
        }
    };
    if (wk == 0) give(std::integral_constant<int, 0>{});
    else give(std::integral_constant<int, 2>{});
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int r = tile_row(2 * wk + o);
      float bad = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        own[o][j] = (own[o][j] + theirs[(o * 4 + j) * 64]) * kSplitUnscale;
#pragma unroll
        for (int t = 0; t < 4; ++t) bad += own[o][j][t] * 0.f;
      }
      // Infinities, and sums past the largest scaled number (2^80 unscaled), make infinities and NaNs of the parts' products:
      // those results, and no others, are taken from a sum by the fp32 instruction, so that a result is that of its own row
      // and column whatever its neighbours hold.  16 rows at a time and without stages in LDS: a training step of 8192 rows,
      // 8 slots, 1024 x 4096, takes 3150 us, 9100 if all of x is infinite.
      if (__any(bad != bad)) {
        const long long src = AKM ? (row0 + r < row_end ? r : -1) : source_row(r);
        const float* const at_a = baseA + (AKM ? src : src * a.lda);  // of k = 0
        f32x4 full[4] = {};
        for (int k0 = 0; k0 < K; k0 += 16) {
          float x[4];
          f32x4 y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k = k0 + 4 * i + quad;
            x[i] = k < K && src >= 0 ? at_a[AKM ? (size_t)k * a.lda : (size_t)k] : 0.f;
            y[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (k < K && n0 + w_col < a.n_out) y[i] = *(const f32x4*)(baseW + (size_t)k * a.ldw + w_at);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) full[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[i][j], x[i], full[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (own[o][j][t] * 0.f != 0.f) own[o][j][t] = full[j][t];
      }
      auto vec = [&](int t) { return f32x4{own[o][0][t], own[o][1][t], own[o][2][t], own[o][3][t]}; };
#pragma unroll
      for (int t = 0; t < (kGated ? 2 : 4); ++t)
        f32_emit<float, EPI, WGRAD, true>(a, slot, row0 + r, row_end, n0 + out_col(t), vec(t), vec(kGated ? t + 2 : t));
    }
    __syncthreads();  // the partial sums are read: the next tile may fill the stage
  }
}

// Which fp32 GEMMs run here: those with two tiles a CU and more (gradients, whose tiles are often of one stage, four), columns
// and k (gradients: both widths) that fill three quarters of their tiles, and 48 rows a slot on average.  us on the fp32
// instruction and here: 4096 tokens, 1024 x 4096, 8 slots, top-2: 644 -> 490, 659 -> 524, gradients 596 -> 484 and 591 -> 478;
// 3000 tokens, 512 x 512 gated, top-6, 80 slots: 217 -> 176, 108 -> 94, 116 -> 104, 225 -> 186; 1024 tokens, 512 x 2048,
// 16 slots: 63 -> 60, 62 -> 55.  Of 300 layers drawn from S = 4 to 96, 16 to 600 rows a slot, d to 1300, ffn to 2600, within
// the lines 388 GEMMs by 10 % (geometric mean; 18 slower by 3 to 14 %, just past a line); outside: 16 to 24 rows a
// slot 3 % slower (forwards) and 6 % (gradients), 24 to 48 level, gradients of 512 to 1024 tiles 2 % slower, one tile a CU and
// less 59 -> 70 (the down projection of 2048 x 512 at 160 tiles).
// rows64: row tiles expected to hold rows;  fill: k, or a gradient's rows
inline bool use_split(long long P, int S, long long rows64, int cols, int fill, int tiles_a_cu) {
  const long long padded = (long long)ceil_div(cols, kSplitCols) * kSplitCols * ceil_div(fill, 64) * 64;
  return P >= 48ll * S && rows64 * ceil_div(cols, kSplitCols) >= (long long)tiles_a_cu * device_cus() && 4ll * cols * fill >= 3 * padded;
}
inline bool use_split_rows(long long P, int S, int cols, int K) {
  const long long used = P < S ? P : S;  // slots that can have rows, half a tile more each
  return use_split(P, S, P / kSplitRows + (used + 1) / 2, cols, K, 2);
}
// Whether a forward of this shape reads the table of 64-row tiles.
inline bool split_forward(const lz_shape* s) {
  const long long P = (long long)s->T * s->k;
  const int S = s->N * s->c;
  return s->dtype == LZ_F32 && (use_split_rows(P, S, s->ffn * (s->act == LZ_SWIGLU ? 2 : 1), s->d) || use_split_rows(P, S, s->d, s->ffn));
}

template <int EPI, bool WGRAD>
int32_t launch_split(F32Args a, int cols, long long max_rows64, hipStream_t st) {
  const int cus = device_cus();
  if (cus == 0) return LZ_EHIP;
  a.n_tiles = ceil_div(cols, kSplitCols);
  const long long resident = 2ll * cus, tiles = max_rows64 * a.n_tiles;
  hipLaunchKernelGGL((gemm_split_kernel<EPI, WGRAD, false>), dim3((unsigned)(tiles < resident ? tiles : resident)), dim3(256), 0, st,
                     F32Launch<false>{{a}});
  return lz::launch_status();
}

// One GEMM over the batch's row tiles (a.t: kF32Rows rows an entry, a.t_split: kSplitRows); S and P size the launch only.
template <typename Elem, int EPI, bool WKM>
int32_t launch_f32_rows(F32Args a, int S, long long P, hipStream_t st) {
  const long long used = P < S ? P : S;  // slots that can have rows, half a tile more each
  if constexpr (sizeof(Elem) == 4 && WKM) {
    const int cols = a.n_out * (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP ? 2 : 1);
    // x past 31-bit offsets cannot be gathered: the calls that need not gather it take the same kernel and give the same bits
    const bool x_fits = a.gather_T * a.lda * 4 < (1ll << 31);
    if (use_split_rows(P, S, cols, a.K) && x_fits && whole_pieces(a)) {
      a.t = a.t_split;
      return launch_split<EPI, false>(a, cols, a.t.capacity, st);
    }
  }
  return launch_f32<Elem, EPI, false, WKM>(a, P / kF32Rows + (used + 1) / 2, a.t.capacity, st);
}

// A weight gradient of all slots, C[s] [m_rows, n_out] = A[rows of s]^T W[rows of s], or added to Cacc, and how it is launched.
struct F32Wgrad {
  F32Args a;
  bool split, vec;
  int nw;           // of the fp32 kernel
  long long tiles;  // of the kernel that serves it
};
template <typename Elem>
F32Wgrad f32_wgrad(const void* A, int m_rows, const void* W, int n_out, const int32_t* slot_offsets, int S, long long P, void* C,
                   float* Cacc) {
  F32Wgrad g{};
  F32Args& a = g.a;
  a.A = A;
  a.W = W;
  a.C = C;
  a.Cacc = Cacc;
  a.lda = a.m_rows = m_rows;
  a.ldw = a.ldc = a.n_out = n_out;
  a.slot_offsets = slot_offsets;
  a.P = P;
  a.slots = S;
  g.vec = whole_pieces(a);
  g.split = sizeof(Elem) == 4 && g.vec && use_split(P, S, (long long)S * ceil_div(m_rows, kSplitRows), n_out, m_rows, 4);
  a.m_tiles = ceil_div(m_rows, g.split ? kSplitRows : kF32Rows);
  g.nw = f32_waves((long long)S * a.m_tiles * ceil_div(n_out, 32));
  a.n_tiles = ceil_div(n_out, g.split ? kSplitCols : 32 * g.nw);
  g.tiles = (long long)S * a.m_tiles * a.n_tiles;
  return g;
}

template <typename Elem, int EPI>
int32_t launch_f32_wgrad(const F32Wgrad& g, hipStream_t st) {
  const long long rows = (long long)g.a.slots * g.a.m_tiles;
  if constexpr (sizeof(Elem) == 4)
    if (g.split) return launch_split<EPI, true>(g.a, g.a.n_out, rows, st);
  return launch_f32<Elem, EPI, true, true>(g.a, rows, rows, st);
}

// Both of a backward pass; in_pass: as part of a whole one, in one launch where one kernel serves both.  Backward passes of 2700 drawn
// fp32 layers, whole pieces and odd sizes, half of them with skewed loads, geometric mean and worst of two launches' time: 32-column tiles of
// slots of under 512 rows 0.94 and 1.01, of 128 columns and split 0.96 and 1.01 (past 16 rounds of the chip's workgroups 0.99).  Slots of
// more rows on 32-column tiles: below 1.5 rounds 0.89, 1.02, above 0.95, from 0.73 (12715 tokens, top-3, 36 slots, 120 x 256,
// 388 -> 282 us) to 1.08 (11952, top-6, 36 slots, 216 x 192, 629 -> 681): a workgroup's tiles are fixed, and which of them get two
// of the fullest slot's is luck with one launch and with two.
template <typename Elem, int EPI>
int32_t launch_f32_wgrads(const F32Wgrad& g0, const F32Wgrad& g1, bool in_pass, hipStream_t st) {
  if (in_pass && g0.split == g1.split && g0.vec == g1.vec && (g0.split || g0.nw == g1.nw)) {
    const F32Launch<true> both{{g0.a, g1.a}};
    const long long tiles = g0.tiles + g1.tiles, resident = g0.split ? 2ll * device_cus() : f32_resident(g0.nw);
    if (resident == 0) return LZ_EHIP;
    const dim3 grid((unsigned)(tiles < resident ? tiles : resident));
    if (g0.split) {
      if constexpr (sizeof(Elem) == 4) hipLaunchKernelGGL((gemm_split_kernel<EPI, true, true>), grid, dim3(256), 0, st, both);
    } else if (g0.nw == 4) {
      launch_f32_waves<Elem, EPI, true, true, 4>(both, grid, g0.vec, st);
    } else {
      launch_f32_waves<Elem, EPI, true, true, 1>(both, grid, g0.vec, st);
    }
    return lz::launch_status();
  }
  const int32_t r = launch_f32_wgrad<Elem, EPI>(g0, st);
  return r != LZ_OK ? r : launch_f32_wgrad<Elem, EPI>(g1, st);
}

}  // namespace
