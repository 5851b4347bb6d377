// Grouped bf16 GEMM on the gfx950 matrix cores, drawing its work from the tables of tiles.h;
// shared by the forward and the backward translation units (device code, not part of the C ABI).
//
//   C[rows of a slot, n] = epi( sum_k A(row, k) * W[slot](n, k) )
//
// Persistent kernel, one workgroup per CU, drawing tiles of up to 256 rows (256, 192, 128 or 64 by the launch, a slot's last
// one fewer) x 256 columns from its XCD's queue.  4 waves
// in 2x2, each wave a 128x128 patch (of 256 rows) = 8x8 v_mfma_f32_16x16x32_bf16 accumulators (fp32, 256
// AGPRs).  With every CU busy the chip is power-limited, and an MFMA-only loop of this shape
// sustains 15 % more flops than one of v_mfma_f32_32x32x16_bf16 (2.03 against 1.76 PFLOP/s on
// random operands; at a quarter of the CUs both reach the nominal rate).  Operand tiles are
// streamed HBM -> LDS with 16-byte buffer loads that write LDS
// directly, through LDS stages of 64 k (two for the activation tile, three for the weight tile:
// all 160 KiB); fragment reads are software pipelined over two register sets.  An operand may be k-contiguous ([row, k]: 256 tile rows of 128 B, read with
// ds_read_b128) or k-major ([k, column]: 64 k-rows of 512 B, read with the transposing
// ds_read_b64_tr_b16); see the MODE_* list below.  The XOR swizzles that keep the fragment
// reads free of bank conflicts are applied on the global-address side, because a direct-to-LDS
// load fixes the LDS side to lane order.  Buffer descriptors bound every load, so ragged tiles
// cannot fault.  The MFMA takes the weight fragment as its row operand, which leaves each lane
// with 4 consecutive output columns per accumulator group; the epilogue regroups them through
// a per-wave LDS patch into whole 128-byte lines.  For SwiGLU the weight tile interleaves
// 32-wide fragments of the gate and the up projection, so the gate and up values of one output
// element sit in the same lane and register index of two accumulators.
#pragma once
#include "tiles.h"
#include <atomic>
#include <type_traits>

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// *_KEEP: the training forward; besides act(z) the pre-activation z goes to MfmaArgs::Z.
// EPI_ACCUM: the result is added to the fp32 matrix MfmaArgs::Cacc (weight gradients summed over
// micro-batches) instead of being stored as bf16.
enum { EPI_NONE = 0, EPI_GELU = 1, EPI_SWIGLU = 2, EPI_GELU_KEEP = 3, EPI_SWIGLU_KEEP = 4, EPI_ACCUM = 5 };

// ------------------------------------------------------------------------------------------
// gfx950 MFMA kernel, bf16 in / fp32 accumulate / bf16 out
// ------------------------------------------------------------------------------------------
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int kRowBytes = BK * 2;                  // one tile row of a stage in LDS: 128 B = 8 chunks of 16 B
constexpr int kATile = BM * kRowBytes, kWTile = BN * kRowBytes;  // 32 KiB each
// LDS map: two activation stages, then a ring of three weight stages (its loads get two K steps
// to land); together all of the CU's 160 KiB
constexpr int kWStages = 3;
constexpr int kLdsBytes = 2 * kATile + kWStages * kWTile;
__device__ __forceinline__ constexpr int a_stage_off(int s) { return s * kATile; }
__device__ __forceinline__ constexpr int w_stage_off(int w) { return 2 * kATile + w * kWTile; }

struct MfmaArgs {
  const uint16_t* A;    // MODE_NT, MODE_NN: [P, K];  MODE_TN: [rows of the batch, lda]
  const uint16_t* W;    // MODE_NT: [S, w_rows, K];  MODE_NN: [S, K, ldw];  MODE_TN: [rows of the batch, ldw]
  uint16_t* C;          // [P, n_out]
  float* Cacc;          // EPI_ACCUM: [P, n_out] fp32, read, added to and written back
  long long P;          // rows of C (MODE_TN: S * rows_per_slot virtual rows)
  int K;                // contraction length (MODE_TN: per slot, in its units' records)
  int w_rows;           // MODE_NT: weight rows per slot
  int n_out;            // output columns
  int up_row0;          // SwiGLU: offset of the up projection inside a slot's W (rows, or columns if k-major)
  int n_tiles;          // column tiles per row tile
  TileTable t;          // narrow kernel
  UnitTable u;          // wide kernel
  uint16_t* Z;          // *_KEEP epilogues: pre-activations [P, z_cols] (SwiGLU: gate columns, then up columns)
  int z_cols;
  int lda, ldw;         // row strides (elements) of the k-major operands
  // MODE_TN (weight gradients): slot s contracts over its rows of the batch of both operands and owns rows_per_slot rows
  // of C (row index = s * rows_per_slot + m, m = column of A)
  int rows_per_slot;
  // GATHER (forward only): A is x [gather_T, K] and row r of the permuted buffer is row
  // gather[r] / gather_k of it (gather = row_to_pair of the dispatcher)
  const int32_t* gather;
  int gather_k;
  long long gather_T;
};

// stores of an epilogue's last pass (EPI_ACCUM: not the same in every wave)
template <int EPI>
constexpr int kLastStores = EPI == EPI_ACCUM ? 0 : EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP ? 4 : 8;

// Operand layouts of the contraction C[m, n] = sum_k A(m, k) W(n, k):
//   MODE_NT  A [m, k], W [n, k]: both contiguous along k (the data gradients)
//   MODE_NN  A [m, k], W [k, n] (the forward: weights are stored input-major)
//   MODE_TN  A [k, m], W [k, n], a different k range for every slot (the weight gradients)
//   MODE_TN_WIDE  the same when an operand may span more than 4 GiB inside one slot (64-bit
//            arithmetic where MODE_TN rebuilds its buffer descriptors for a K step)
// A k-major operand tile lies in LDS as 64 k-rows of 256 columns (512 B each) and is read with
// ds_read_b64_tr_b16, which hands every lane four k-values of one column: the 16 lanes of a
// group supply the addresses of 4 k-rows x 4 column quads, and lane i receives column i of the
// group's 16 at those four k.  Two such reads give the lane the same 8 consecutive k of its
// column that a ds_read_b128 gives it from a k-contiguous tile, so the MFMAs and the epilogue
// do not change.
enum { MODE_NT = 0, MODE_NN = 1, MODE_TN = 2, MODE_TN_WIDE = 3 };
typedef short i16x4 __attribute__((ext_vector_type(4)));

// The four words of a raw buffer descriptor (base, stride 0, bytes, data format word).
__device__ __forceinline__ i32x4 rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  return i32x4{(int)(uint32_t)b, (int)(uint32_t)((b >> 32) & 0xFFFFu), (int)bytes, 0x00020000};
}

// 16 bytes per lane from a buffer straight into LDS at lds_base + 16 * lane, written as assembly:
// in the k-major modes the compiler must not know that loads into LDS are in flight, or it
// makes every transposing LDS read wait for all of them (it cannot tell that the two never
// touch the same bytes).  The kernel orders loads and reads itself (s_waitcnt vmcnt + barrier).
__device__ __forceinline__ void load16_to_lds(i32x4 rsrc, uint32_t lds_base, int voffset, int soffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_base), "v"(voffset), "s"(rsrc), "s"(soffset)
               : "memory");  // m0 is scratch to the compiler as well: it loads it right before each use
}

// The same load with an MFMA between the write of M0 and the load: the MFMA stands in for the wait
// state the hardware wants there, and the three instructions fit the gap between two MFMAs.
__device__ __forceinline__ void mfma_then_load16_to_lds(f32x4& acc, const bf16x8& w, const bf16x8& x, i32x4 rsrc,
                                                        uint32_t lds_base, int voffset, int soffset) {
  asm volatile("s_mov_b32 m0, %3\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tbuffer_load_dwordx4 %4, %5, %6 offen lds"
               : "+a"(acc)
               : "v"(w), "v"(x), "s"(lds_base), "v"(voffset), "s"(rsrc), "s"(soffset)
               : "memory");
}

// Activations on the fp32 accumulators of the bf16 path.  The result is rounded to bf16
// (relative step 2^-9), so hardware exp2 / rcp (1 ulp) are used.
//
// GELU: v Phi(v) = v / 2 + |v| (1/2 - Phi(-|v|)), Phi(-u) = 2^P(u) with P of degree 8 fitted to log2 Phi(-u) on [0, 5.4] by
// weighted least squares, reweighted until the errors of u 2^P(u) are level; P falls without end past it, so that large
// u give exactly v / 2 + |v| / 2, and infinities and NaNs what those two terms make of them.  What bounds it is the vector unit,
// one wave a SIMD with the matrix cores idle: a quarter-rate instruction counts as four, 15 slots where Abramowitz-Stegun
// 7.1.26 (four steps, exp2 and rcp) takes 21.  Largest and rms error against fp64 at 2^20 + 1 even points of [-8, 8], in fp32 with
// exp2 and rcp rounded correctly: 3.1e-7 and 0.56e-7, by that 3.8e-7 and 0.96e-7 (the exact value rounded 2.4e-7 and 0.51e-7); largest
// of negative v 0.8e-7 and 2.6e-7; relative, v > 0: 1.8e-7 and 5.3e-7.
__device__ __forceinline__ float silu_fast(float v) {
  return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * v));
}
__device__ __forceinline__ float gelu_fast(float v) {
  const float u = fabsf(v);
  float p = fmaf(-1.8467128484189743e-06f, u, 2.7774511181632988e-05f);
  p = fmaf(p, u, -0.00013225268048699945f);
  p = fmaf(p, u, -0.00026397229521535337f);
  p = fmaf(p, u, 0.0072246030904352665f);
  p = fmaf(p, u, -0.052603982388973236f);
  p = fmaf(p, u, -0.45917391777038574f);
  p = fmaf(p, u, -1.151109218597412f);
  p = fmaf(p, u, -0.9999999403953552f);
  return fmaf(u, 0.5f - __builtin_amdgcn_exp2f(p), 0.5f * v);
}

// Two fp32 -> one dword of two bf16, round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// 16-byte chunk c of tile row r lives at chunk position c ^ swz(r) of its 128-byte LDS row.
// LDS has 64 banks of 4 B, so a ds_read_b128 is served 16 lanes at a time: 16 consecutive
// rows at one logical chunk must cover 16 distinct 16-byte bank groups (256 B = 2 rows), hence
// the key row/2.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// 16-byte piece p (8 columns) of k-row kr of a k-major tile lives at piece position p ^ swz_kmajor(kr)
// of its 512-byte LDS row.  A transposing read is served 32 lanes at a time: two lane groups, each
// touching 4 consecutive k-rows (kr % 4 = 0..3) at the same 32 bytes (one 16-column fragment), the
// two groups 8 k-rows apart.  Bits 2-3 of the key move the four k-rows of a group into four
// different quarters of the banks, bit 1 moves the second group's fragments 32 bytes on, so the
// eight 32-byte runs fall into eight different bank groups.
__device__ __forceinline__ int swz_kmajor(int kr) { return ((kr & 3) << 2) | (((kr >> 3) & 1) << 1); }

// A tile: rows [row0, row_end) of a slot, at most 256, output columns from n0; weight gradients: the rows [k0, k1) of the batch that the slot contracts over.  slot < 0: none.
struct Tile {
  int slot, row0, row_end, n0, k0, k1;
  int part;  // of a pair of GEMMs in one launch: which
};

// Where a tile's operands lie, and their direct-to-LDS loads.
//
// KTAIL: K is not a multiple of 64 and an operand is k-contiguous, so the last K step's 128-byte rows run
// past the end of K into the next row.  The lanes whose 16-byte chunk lies there fetch from beyond the
// descriptor instead and get zeros (both operands: a zero against what the other row holds would let an
// infinity or NaN of a neighbouring row through).  k-major operands end with their descriptor.
template <int EPI, int MODE, bool GATHER, bool KTAIL>
struct Operands {
  static constexpr bool TA = MODE == MODE_TN || MODE == MODE_TN_WIDE, TB = MODE != MODE_NT;  // k-major left / right operand
  static constexpr bool kGated = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP;
  i32x4 wordsA, wordsW, wordsNull;  // descriptors; Null has no bytes
  const uint16_t *tileA, *tileW;
  uint32_t a_extent, w_extent;      // bytes the two descriptors cover
  int stepA, stepW;                 // bytes one K step advances in each operand
  // MODE_TN, MODE_TN_WIDE: the contraction ends with the slot's last row, wherever in a K step that
  // is, so the descriptors are rebuilt for every K step (base advanced by whole steps, extent =
  // what is left of the slot); in 64-bit arithmetic where a slot's rows may cover more than 4 GiB
  unsigned long long a_bytes, w_bytes, stepA64, stepW64;
  int k_steps;
  uint32_t lds;                     // LDS address of the stages, this wave's place in a 4-KiB row of loads added
  int voffX[8], voffW[8];           // byte offsets of the loads of one stage
  int tail_or;                      // KTAIL: what the last K step ORs into them
  int no_row;                       // GATHER: bit i: load i's row lies past the tile's end

  // ---- buffer descriptors: out-of-range loads return zero instead of faulting.  The activation
  // descriptor covers just this tile's rows, so 32-bit offsets do however large P is.
  //
  // ---- per-lane global offsets of the direct-to-LDS loads of one stage.
  // Load i of a wave fills the LDS bytes [u*1024, u*1024+1024), u = 4 i + wave: 8 whole rows, lane l
  // landing at row 8u + l/8, 16-byte chunk l%8.  That LDS chunk must hold logical chunk
  // (l%8) ^ swz(row), so the lane fetches that one (the swizzle is applied on the global side
  // because a direct-to-LDS load fixes the LDS side to lane order).  The first 2 XF loads of the four
  // waves hold the first 64 XF rows.
  //
  // k-major operand: load i fills two k-rows of 512 B, lane l landing at k-row 2u + l/32, 16-byte
  // piece l%32, which must hold logical piece (l%32) ^ swz_kmajor(k-row).
  __device__ __forceinline__ void set(const MfmaArgs& a, char* smem, const Tile& t) {
    if (t.slot < 0) {  // no tile: its loads have no bytes
      k_steps = 0;
      a_bytes = w_bytes = 0;
      return;
    }
    // The empty asm keeps the per-lane address arithmetic below inside the tile: hoisted out of
    // the caller's tile loop it would be carried in registers through the whole kernel and spill.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    const int n_rows = t.row_end - t.row0;
    int K = a.K;
    stepA = stepW = BK * 2;
    if constexpr (TA) {
      // The descriptors start at the slot's first row and this tile's first column and end with
      // the slot's last row: the rows of the last, partial K step that belong to the next slot
      // read as zero.
      K = t.k1 - t.k0;
      const int m0 = t.row0 - t.slot * a.rows_per_slot;
      tileA = a.A + (size_t)t.k0 * a.lda + m0;
      tileW = a.W + (size_t)t.k0 * a.ldw + t.n0;
      a_bytes = K > 0 ? ((unsigned long long)K * (unsigned)a.lda - (unsigned)m0) * 2ull : 0ull;
      w_bytes = K > 0 ? ((unsigned long long)K * (unsigned)a.ldw - (unsigned)t.n0) * 2ull : 0ull;
      stepA64 = 64ull * (unsigned)a.lda * 2ull;
      stepW64 = 64ull * (unsigned)a.ldw * 2ull;
      a_extent = (uint32_t)a_bytes;  // MODE_TN: the host checked that they fit; MODE_TN_WIDE: unused, see words_*()
      w_extent = (uint32_t)w_bytes;
      stepA = stepW = 0;
    } else if constexpr (MODE == MODE_NN) {
      if constexpr (GATHER) {
        tileA = a.A;  // the whole of x: a tile's rows lie anywhere in it (the host checked that it fits 32-bit offsets)
        a_extent = (uint32_t)((unsigned long long)a.gather_T * (unsigned)K * 2ull);
      } else {
        tileA = a.A + (size_t)t.row0 * K;
        a_extent = (uint32_t)n_rows * (uint32_t)K * 2u;
      }
      tileW = a.W + (size_t)t.slot * K * a.ldw;
      w_extent = (uint32_t)K * (uint32_t)a.ldw * 2u;
      stepW = 64 * a.ldw * 2;
    } else {
      tileA = a.A + (size_t)t.row0 * K;
      a_extent = (uint32_t)n_rows * (uint32_t)K * 2u;
      tileW = a.W + (size_t)t.slot * a.w_rows * K;
      w_extent = (uint32_t)((unsigned long long)a.w_rows * K * 2);
    }
    k_steps = (K + BK - 1) / BK;
    wordsA = rsrc_words(tileA, a_extent);
    wordsW = rsrc_words(tileW, w_extent);
    wordsNull = rsrc_words(a.A, 0);
    no_row = 0;
    auto voff_kmajor = [&](int i, int ld, int col0) {
      const int kr = (i * 4 + wave) * 2 + (lane >> 5);
      const int piece = (lane & 31) ^ swz_kmajor(kr);
      return (int)(((uint32_t)kr * (uint32_t)ld + (uint32_t)col0 + (uint32_t)piece * 8u) * 2u);
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (TA) {
        voffX[i] = voff_kmajor(i, a.lda, 0);  // columns past the operand's edge fetch its neighbours: never stored
      } else {
        const int r = (i * 4 + wave) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ swz(r);
        // rows past the tile's end (never stored), and rows without a pair, lie beyond the descriptor: zeros
        if constexpr (GATHER) {
          voffX[i] = a.gather[t.row0 + (r < n_rows ? r : n_rows - 1)];  // the pair; the offset once it has arrived
          if (r >= n_rows) no_row |= 1 << i;
        } else {
          voffX[i] = (int)(((uint32_t)r * (uint32_t)K + (uint32_t)chunk * 8u) * 2u);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (TB && kGated) {
        // k-major SwiGLU weights [K, 2 ffn]: 32-column fragments alternate gate and up columns
        const int kr = (i * 4 + wave) * 2 + (lane >> 5);
        const int piece = (lane & 31) ^ swz_kmajor(kr);
        const int f = piece >> 2;
        const int col = t.n0 + (f >> 1) * 32 + (piece & 3) * 8 + ((f & 1) ? a.up_row0 : 0);
        voffW[i] = (int)(((uint32_t)kr * (uint32_t)a.ldw + (uint32_t)col) * 2u);
      } else if constexpr (TB) {
        voffW[i] = voff_kmajor(i, a.ldw, MODE == MODE_NN ? t.n0 : 0);
      } else {
        static_assert(!kGated || TB, "gated weights are k-major");
        const int r = (i * 4 + wave) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ swz(r);
        voffW[i] = (int)(((uint32_t)(t.n0 + r) * (uint32_t)K + (uint32_t)chunk * 8u) * 2u);
      }
    }
    if constexpr (KTAIL) {  // the swizzle of a load's rows is the same for all of a wave's loads
      const int k_left = K - (K - 1) / BK * BK;  // 1..64; multiples of 8, so chunks are whole
      tail_or = ((lane & 7) ^ swz(wave * 8 + (lane >> 3))) * 8 >= k_left ? (int)0x80000000 : 0;
    }
  }

  // The descriptors for K step `step`.  A step past the end of K is "loaded" through a zero-length one: no memory traffic.
  __device__ __forceinline__ i32x4 words_x(int step) const {
    const bool real = step < k_steps;
    if constexpr (MODE == MODE_TN) {
      // bytes left of the slot: a step that begins inside the slot begins inside both extents (the
      // tile's first column lies inside the operand's row)
      const uint32_t off = (uint32_t)step * (uint32_t)stepA64;
      return rsrc_words((const char*)tileA + off, real ? a_extent - off : 0u);
    } else if constexpr (MODE == MODE_TN_WIDE) {
      const unsigned long long off = (unsigned long long)(unsigned)step * stepA64, left = a_bytes > off ? a_bytes - off : 0ull;
      return rsrc_words((const char*)tileA + off, left > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)left);
    } else {
      return real ? wordsA : wordsNull;
    }
  }
  __device__ __forceinline__ i32x4 words_w(int step) const {
    const bool real = step < k_steps;
    if constexpr (MODE == MODE_TN) {
      const uint32_t off = (uint32_t)step * (uint32_t)stepW64;
      return rsrc_words((const char*)tileW + off, real ? w_extent - off : 0u);
    } else if constexpr (MODE == MODE_TN_WIDE) {
      const unsigned long long off = (unsigned long long)(unsigned)step * stepW64, left = w_bytes > off ? w_bytes - off : 0ull;
      return rsrc_words((const char*)tileW + off, left > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)left);
    } else {
      return real ? wordsW : wordsNull;
    }
  }
  // Load i of a wave for K step `step` into an activation / weight stage; with_mfma: an MFMA (accumulator, weight and
  // activation fragment) to issue together with it
  __device__ __forceinline__ void load_x(int stage, int step, int i, const i32x4& words, f32x4* with_mfma = nullptr,
                                         const bf16x8* mw = nullptr, const bf16x8* mx = nullptr) const {
    int voff = voffX[i];
    if constexpr (KTAIL && !TA) voff |= tail_or & (step == k_steps - 1 ? -1 : 0);
    const uint32_t to = lds + a_stage_off(stage) + i * 4096;
    if (with_mfma != nullptr) mfma_then_load16_to_lds(*with_mfma, *mw, *mx, words, to, voff, step * stepA);
    else load16_to_lds(words, to, voff, step * stepA);
  }
  __device__ __forceinline__ void load_w(int stage, int step, int i, const i32x4& words, f32x4* with_mfma = nullptr,
                                         const bf16x8* mw = nullptr, const bf16x8* mx = nullptr) const {
    int voff = voffW[i];
    if constexpr (KTAIL && !TB) voff |= tail_or & (step == k_steps - 1 ? -1 : 0);
    const uint32_t to = lds + w_stage_off(stage) + i * 4096;
    if (with_mfma != nullptr) mfma_then_load16_to_lds(*with_mfma, *mw, *mx, words, to, voff, step * stepW);
    else load16_to_lds(words, to, voff, step * stepW);
  }
  // GATHER: pairs to offsets
  __device__ __forceinline__ void gather_rows(const MfmaArgs& a) {
    if constexpr (GATHER) {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      const uint32_t n_pairs = (uint32_t)(a.gather_T * a.gather_k);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int chunk = (lane & 7) ^ swz((i * 4 + wave) * 8 + (lane >> 3));
        const uint32_t pair = (uint32_t)voffX[i];
        const bool ok = pair < n_pairs && (no_row >> i & 1) == 0;
        voffX[i] = ok ? (int)((pair / (uint32_t)a.gather_k * (uint32_t)a.K + (uint32_t)chunk * 8u) * 2u) : (int)a_extent;
      }
    }
  }
  // Load l of the 32 of the first two K steps.
  __device__ __forceinline__ void load_first(int l) const {
    const int step = l / 16, i = l % 8;
    if (l % 16 < 8) load_w(step, step, i, words_w(step));
    else load_x(step, step, i, words_x(step));
  }
};
constexpr int kFirstLoads = 32;  // of which the first half belong to step 0

// Draws a workgroup's tiles.  Every XCD has a queue of tickets, its unit list's; a workgroup
// starts with the ticket of its index in its own XCD's queue, draws the next ones with an atomic,
// and once that queue is empty helps with the other XCDs' queues, of which it looks at the counters
// first.  Atomics from all CUs on one line take their turns: with all counters in one line and a ticket
// drawn past the end of every queue by every workgroup, the draws alone held the second GEMM at 80 us
// and more however small it was.
//
// Wave 0 draws; the ticket goes to the other waves through LDS, and each looks its tile up by itself.
//
// A launch of one or two rounds, a small batch's, feels every trip to memory on the way: the records of the first unit are fetched with the
// list's header, before it is known that they exist, the first ticket needs no exchange, and a workgroup that has found all queues empty
// says so ahead of its last epilogue.  A launch of one round draws nothing and counts nobody.  (Counters read with every draw, to know of that earlier, keep the draws waiting: 1 to 5 % slower.)
//
// PAIR: two GEMMs in one launch, the lists of one behind those of the other; the counters of the first serve both.
template <bool PAIR>
struct Draws {
  const UnitTable u, u1;
  const int per_xcd, xcd;
  int tile_rows, tile_rows1;
  int q, tickets, units, units1;  // the queue it draws from, tickets and units in it
  int first1;                     // PAIR: tickets from here on belong to the second list
  int part, local;                // of the ticket: its list, its index there
  int ticket, drawn;      // drawn: what the atomic returned (lane 0 of wave 0)
  int total, taken;       // lane h < 8: tickets in queue h, and, wave 0, drawn from it when last looked at
  bool one_round;         // no queue has more tickets than workgroups: none is ever drawn
  int others_left;        // lane 0 of wave 0: workgroups of this XCD that had left before, once this one has
  i32x4 rec[2];           // lane l: record `at` + l of queue q
  int at;

  // takes the first ticket, the workgroup's index in its XCD's queue (workgroups are dealt round-robin to the 8 XCDs)
  __device__ __forceinline__ Draws(const UnitTable& table, const UnitTable& table1, char* smem)
      : u(table), u1(table1), per_xcd(gridDim.x / 8), xcd(blockIdx.x % 8), taken(0), others_left(0) {
    const int lane = (int)(threadIdx.x & 63);
    const int rows = u.header[kTileRows], n_tickets = u.header[xcd], n_units = u.header[8 + xcd];
    total = u.header[lane & 7];
    int rows1 = 0, n_tickets1 = 0, n_units1 = 0;
    if constexpr (PAIR) {
      rows1 = u1.header[kTileRows], n_tickets1 = u1.header[xcd], n_units1 = u1.header[8 + xcd];
      total += u1.header[lane & 7];
    }
    const int i = lane < u.cap ? lane : u.cap - 1;
    const i32x4* const from = (const i32x4*)(u.records + ((size_t)xcd * u.cap + i) * kRecord);
    rec[0] = from[0];
    rec[1] = from[1];
    q = xcd;
    tile_rows = __builtin_amdgcn_readfirstlane(rows);
    first1 = __builtin_amdgcn_readfirstlane(n_tickets);
    units = __builtin_amdgcn_readfirstlane(n_units);
    tickets = first1;
    if constexpr (PAIR) {
      tile_rows1 = __builtin_amdgcn_readfirstlane(rows1);
      tickets += __builtin_amdgcn_readfirstlane(n_tickets1);
      units1 = __builtin_amdgcn_readfirstlane(n_units1);
    }
    ticket = blockIdx.x / 8;
    part = at = 0;
    local = ticket;
    one_round = (__ballot(total > per_xcd) & 255) == 0;
    if (lane >= units) rec[0].x = 0x7FFFFFFF;
    if (ticket >= tickets && one_round) {
      ticket = -1;
    } else if (ticket >= tickets) {  // the same in all waves
      if (mine()) publish_ticket(ticket, smem);
      receive(smem);
    } else if (ticket >= kGroupM * kGroupN || (PAIR && ticket >= first1)) {
      locate();
    }
  }
  static __device__ __forceinline__ bool mine() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x) == 0; }
  __device__ __forceinline__ int* counter(int x) const { return u.header + kTicket + x * kLine; }
  __device__ __forceinline__ void set_queue(int x) {
    q = x;
    first1 = __builtin_amdgcn_readfirstlane(u.header[x]);
    units = __builtin_amdgcn_readfirstlane(u.header[8 + x]);
    tickets = first1;
    if constexpr (PAIR) {
      tickets += __builtin_amdgcn_readfirstlane(u1.header[x]);
      units1 = __builtin_amdgcn_readfirstlane(u1.header[8 + x]);
    }
  }
  __device__ __forceinline__ void look() { taken = __hip_atomic_load(counter(threadIdx.x & 7), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  // asks for the next ticket of the queue
  __device__ __forceinline__ void request() {
    if (mine() && !one_round) {
      drawn = 0;
      if (threadIdx.x == 0) drawn = atomicAdd(counter(q), 1);
    }
  }
  // the ticket asked for, or one of another queue, -1 when no queue has one left, to `to` in LDS
  __device__ __forceinline__ void publish(char* to) {
    if (mine() && !one_round) publish_ticket(per_xcd + __builtin_amdgcn_readfirstlane(drawn), to);
  }
  __device__ __forceinline__ void publish_ticket(int t, char* to) {
    while (t >= tickets) {
      // the first queue from this XCD's on with a ticket left (counters only grow: one that reads as empty is)
      look();
      const unsigned some = (unsigned)__ballot(per_xcd + taken < total) & 255u;
      if (some == 0) {
        t = -1;
        break;
      }
      const unsigned from_own = (some >> xcd | some << (8 - xcd)) & 255u;
      set_queue((xcd + __ffs((int)from_own) - 1) & 7);
      request();
      t = per_xcd + __builtin_amdgcn_readfirstlane(drawn);
    }
    if (threadIdx.x == 0) *(int2*)to = int2{t, q};
  }
  // what was published goes to every wave, which loads the records the ticket may belong to
  __device__ __forceinline__ void receive(const char* from) {
    __syncthreads();
    if (one_round) {
      ticket = -1;
      return;
    }
    const int2 v = *(const int2*)from;
    ticket = __builtin_amdgcn_readfirstlane(v.x);
    const int from_q = __builtin_amdgcn_readfirstlane(v.y);
    __syncthreads();  // the place may be written again
    if (ticket < 0) {
      leave();
      return;
    }
    if (from_q != q) set_queue(from_q);
    locate();
  }
  __device__ __forceinline__ void locate() {
    part = PAIR && ticket >= first1 ? 1 : 0;
    local = ticket - (part ? first1 : 0);
    at = local / (kGroupM * kGroupN);  // a unit has at most that many tiles
    load_records();
  }
  // This workgroup draws no more.  The last one to leave resets the counters (finish(), once it has nothing else to do).
  __device__ __forceinline__ void leave() {
    if (threadIdx.x == 0) others_left = atomicAdd(counter(8 + xcd), 1);
  }
  __device__ __forceinline__ void finish() {
    if (threadIdx.x == 0 && !one_round && others_left == per_xcd - 1 && atomicAdd(counter(16), 1) == 7)
      for (int i = 0; i < 17; ++i) *counter(i) = 0;
  }
  __device__ __forceinline__ void load_records() {
    const bool second = PAIR && part != 0;
    const int n = second ? units1 : units, i = at + (int)(threadIdx.x & 63), last = n > 0 ? n - 1 : 0;
    const int32_t* const list = second ? u1.records + (size_t)q * u1.cap * kRecord : u.records + (size_t)q * u.cap * kRecord;
    const i32x4* const from = (const i32x4*)(list + (size_t)(i < last ? i : last) * kRecord);
    rec[0] = from[0];
    rec[1] = from[1];
    if (i > last) rec[0].x = 0x7FFFFFFF;
  }
  __device__ __forceinline__ Tile tile(int n_out_cols) {
    if (ticket < 0) return Tile{-1, 0, 0, 0, 0, 0, 0};
    unsigned long long le;
    while ((le = __ballot(rec[0].x <= local)) == ~0ull) {
      at += 63;
      load_records();
    }
    const int l = __popcll(le) - 1;  // the unit: the last that starts at or before the ticket
    auto of = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
    const int within = local - of(rec[0].x), nr = of(rec[1].x) & 255, rows = PAIR && part ? tile_rows1 : tile_rows;
    const int col = within / nr;
    const int row0 = of(rec[0].z) + (within - col * nr) * rows, end = of(rec[0].w);
    return Tile{of(rec[0].y), row0, end - row0 < rows ? end : row0 + rows, (of(rec[1].y) + col) * n_out_cols, of(rec[1].z), of(rec[1].w),
                part};
  }
};

template <int EPI>
constexpr int kOutCols = (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP) ? BN / 2 : BN;

// One output tile of 64*XF rows x 256 columns n of the weight operand W(n, k) ("weight rows"
// below, whichever way W lies in memory).  XF = 32-row activation fragments per wave: the 2x2 waves each own (32*XF) x 128 of the tile, so a slot's ragged last tile costs
// MFMAs and activation loads only for its rows rounded up to 64.
//
// ops: the tile's operands, whose first loads are under way.  The next tile is drawn while the last K steps run; its operands
// go to ops and its first loads out within the epilogue.
template <int EPI, int XF, int MODE, bool GATHER, bool KTAIL, bool PAIR>
__device__ __forceinline__ Tile gemm_tile(const MfmaArgs* args, char* smem, const Tile tile, Operands<EPI, MODE, GATHER, KTAIL>& ops,
                                          Draws<PAIR>& draws) {
  const MfmaArgs& a = args[PAIR ? __builtin_amdgcn_readfirstlane(tile.part) : 0];
  constexpr bool TA = MODE == MODE_TN || MODE == MODE_TN_WIDE, TB = MODE != MODE_NT;  // k-major left / right operand
  constexpr bool kGated = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_KEEP;
  constexpr int KS = BK / 32;             // 32-wide MFMA slices per stage
  constexpr int kLoadsX = TA ? 8 : 2 * XF;  // 1-KiB wave loads per wave for the left tile (8 rows, or 2 k-rows, each)
  constexpr int kLoadsW = 8;              // ... for the 256-row weight tile
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // see Operands::set
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int row0 = tile.row0, row_end = tile.row_end, n0 = tile.n0;

  // ---- fragment read addresses.  A fragment is 16 rows (of the activation tile, or weight rows) x
  // the 32 k of a slice; lane l holds row l%16, the 8 consecutive k of chunk l/16 (the operand
  // layout of v_mfma_f32_16x16x32_bf16).  k-contiguous tile: one ds_read_b128 at row l%16, logical
  // chunk 4*slice + l/16 of the stage's 8.
  constexpr int NA = 2 * XF;  // activation fragments per wave (16 rows each)
  constexpr int NW = 8;       // weight fragments per wave (16 weight rows each)
  int fragoff[KS];
  {
    const int r = lane & 15;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fragoff[ks] = r * kRowBytes + (((ks * 4 + (lane >> 4)) ^ swz(r)) << 4);
  }
  const int xbase = wm * 32 * XF * kRowBytes;               // this wave's activation rows
  const int wbase = wn * 128 * kRowBytes;                   // this wave's 128 weight rows
  // k-major tiles: lane 16g + q supplies the address of k-row 8g + q/4 of the 32-wide slice, column
  // quad q%4 of the fragment's 16 columns; the transposing read hands lane 16g + i column i at those
  // four k-rows, a second read 4 k-rows on completes the lane's 8 consecutive k.
  int tfo[2];  // byte offset inside a stage's k-major tile for fragment 0 (and its second piece position), slice 0
  {
    const int g = lane >> 4, q = lane & 15;
    const int kr = 8 * g + (q >> 2);
    // fragment f = pieces 2f, 2f+1 of the k-row; the swizzle key (even) is added by XOR per fragment below
    tfo[0] = kr * 512 + ((q & 1) << 3) + (((q >> 1) & 1) << 4);
    tfo[1] = swz_kmajor(kr);
  }
  auto kmajor_addr = [&](int frag16) {  // fragment frag16 (0..15) of the 256-column tile, slice 0
    return tfo[0] + ((((frag16 << 1) ^ tfo[1]) & 31) << 4);
  };
  auto read_kmajor = [&](const char* p) {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p + 4 * 512));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto frag_x = [&](int stage, int ks, int j) {
    const char* base = smem + a_stage_off(stage);
    if constexpr (TA) return read_kmajor(base + ks * 32 * 512 + kmajor_addr(NA * wm + j));
    else return *(const bf16x8*)(base + xbase + j * 16 * kRowBytes + fragoff[ks]);
  };
  auto frag_w = [&](int stage, int ks, int i) {
    const char* base = smem + w_stage_off(stage);
    if constexpr (TB) return read_kmajor(base + ks * 32 * 512 + kmajor_addr(NW * wn + i));
    else return *(const bf16x8*)(base + wbase + i * 16 * kRowBytes + fragoff[ks]);
  };

  f32x4 acc[NW][NA];
#pragma unroll
  for (int i = 0; i < NW; ++i)
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  // ---- main loop: K steps of 64 columns; step kt reads activation stage kt%2 and weight stage kt%3.
  // One barrier per step, placed after the last reads of the step's stages have been issued: past it
  // nobody reads them any more, so the activation loads of step kt+2 and the weight loads of step
  // kt+3 can start into them, and the next step's stages (whose loads every wave has waited for
  // before the barrier) can be read.
  //
  // A step's loads are not issued in one burst: a wave that issues a burst stands still until the
  // texture unit has accepted it, and the MFMA pipe with it.  The activation loads go out during
  // the unit after barrier kt (they must have landed by the next barrier); the weight loads, which
  // have a whole step longer, are spread over the three units that follow.
  const int k_steps = ops.k_steps;
  constexpr int kLoads = kLoadsW + kLoadsX;
  // Loads [q0, q1) of a wave's per step: the activation loads (q < kLoadsX) of K step a_step into
  // activation stage a_stage, the weight loads of K step w_step into weight stage w_stage.
  // with_mfma: an MFMA (accumulator, weight and activation fragment) to issue together with load q0
  auto issue = [&](int a_stage, int a_step, int w_stage, int w_step, int q0, int q1, f32x4* with_mfma = nullptr,
                   const bf16x8* mw = nullptr, const bf16x8* mx = nullptr) {
#pragma unroll
    for (int q = q0; q < q1; ++q) {
      f32x4* const mfma = q == q0 ? with_mfma : nullptr;
      if (q < kLoadsX) ops.load_x(a_stage, a_step, q, ops.words_x(a_step), mfma, mw, mx);
      else ops.load_w(w_stage, w_step, q - kLoadsX, ops.words_w(w_step), mfma, mw, mx);
    }
  };
  // A stage is consumed as four units: 32-wide slice s (0, 1) x half hw (0, 1) of the wave's weight
  // fragments.  Unit (s, hw) needs the NA activation fragments of slice s and the weight fragments
  // 4 hw .. 4 hw + 3 of slice s: 4 NA MFMAs.  Two register sets of each kind alternate (activation
  // fragments by slice, weight fragments by unit), so that the ds_reads of the next unit are in
  // flight while the MFMAs of the current one run.
  //
  // The MFMAs are written as assembly with the accumulator tied to the destination (left to the
  // register allocator, this MFMA shape gets a destination different from its accumulator input,
  // and with all 256 accumulator registers live the copies that needs go through VGPRs: 3.5 moves
  // per MFMA).  A volatile asm also pins the order: memory operations do not cross it, so the
  // fragment reads and direct-to-LDS loads below issue exactly where they are written, one read per
  // MFMA from the start of a unit (the next unit waits on them), the loads spread over the unit.
  constexpr int kMfmas = 4 * NA;                             // MFMAs per unit
  // Loads [0, kAfterBarrier) go out in the unit after the barrier, [kAfterBarrier, kL1), [kL1, kL2) and
  // [kL2, kLoads) in the three units of the next step: the 8 weight loads as 2 + 3 + 3.
  // (Measured on configs 2-4: with the weight loads bunched behind the activation loads, 4 in the unit after
  // the barrier and 4 in the next, the second GEMM is 3-5 % slower and the first level; all 16 after the barrier
  // costs both 5-7 %; other even spreads, also with half of the activation loads a unit later, are within 1 %.
  // Spreading a unit's loads over the whole unit beats its first half or quarter by 1-3 %; a barrier moved up
  // to just behind the stage's last reads, with all loads after it, is level.)
  constexpr int kAfterBarrier = kLoadsX, kL1 = kLoadsX + 2, kL2 = kLoadsX + 5;
  bf16x8 xf[2][NA], wf[2][4];
  // r-th fragment read of a unit's look-ahead: the weight fragments of unit (s, hw) go into set ws,
  // the activation fragments [j0, j1) of slice xs into set xset; with x_first in the order of first
  // use by the MFMAs (weight fragment 0, the activation fragments, weight fragments 1..3).
  auto read_r = [&](int r, int w_stage, int s, int hw, int ws, int x_stage, int xs, int xset, int j0,
                    int j1, bool x_first) {
    const int NX = j1 - j0;
    int wi = -1, xj = -1;
    if (x_first) {
      if (r == 0) wi = 0;
      else if (r <= NX) xj = j0 + r - 1;
      else wi = r - NX;
    } else {
      if (r < 4) wi = r;
      else xj = j0 + r - 4;
    }
    if (wi >= 0) wf[ws][wi] = frag_w(w_stage, s, 4 * hw + wi);
    else xf[xset][xj] = frag_x(x_stage, xs, xj);
  };
  // One unit: the MFMAs of weight half hw on the sets (xset, ws), interleaved with the reads for the
  // next unit and the loads [q0, q1) of the activation and weight steps named by the ld_ arguments.
  auto unit = [&](int hw, int xset, int ws, int w_stage, int ns, int nhw, int nws, int x_stage, int xs, int nxset, int j0,
                  int j1, bool x_first, int ld_a_stage, int ld_a_step, int ld_w_stage, int ld_w_step, int q0, int q1) {
    const int NR = 4 + (j1 - j0), NL = q1 - q0;
#pragma unroll
    for (int m = 0; m < kMfmas; ++m) {
      if (m < NR) read_r(m, w_stage, ns, nhw, nws, x_stage, xs, nxset, j0, j1, x_first);
      const int l0 = q0 + (NL * m) / kMfmas, l1 = q0 + (NL * (m + 1)) / kMfmas;
      if (l1 > l0) {
        issue(ld_a_stage, ld_a_step, ld_w_stage, ld_w_step, l0, l1, &acc[4 * hw + m / NA][m % NA], &wf[ws][m / NA],
              &xf[xset][m % NA]);
      } else {
        issue(ld_a_stage, ld_a_step, ld_w_stage, ld_w_step, l0, l1);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc[4 * hw + m / NA][m % NA])
                     : "v"(wf[ws][m / NA]), "v"(xf[xset][m % NA]));
      }
    }
  };
  constexpr int kHalf = NA / 2;

  constexpr int D = kWStages;
  // In flight when the tile starts: the first two steps' loads and behind them at least the stores of the previous
  // epilogue's last pass (the first tile's caller has waited for all).  The units of step 0 issue the weight loads of
  // step 2.  s_waitcnt with only vmcnt set (bits [3:0] and [15:14]).
  constexpr int kAhead = kFirstLoads / 2 + kLastStores<EPI>;
  __builtin_amdgcn_s_waitcnt(0x0F70 | (kAhead & 15) | ((kAhead >> 4) << 14));
  __syncthreads();  // ... everyone's are; and everyone has read its last patch
#pragma unroll
  for (int r = 0; r < 4 + NA; ++r) read_r(r, 0, 0, 0, 0, 0, 0, 0, 0, NA, true);  // unit (0, 0) of stage 0

  // One K step on activation stage `as` and weight stage `wst`.  The loop below is unrolled so that
  // both are compile-time constants and every LDS address of the step folds into an instruction's
  // offset field or a literal (otherwise a dozen address additions per step queue up at the head of
  // the loop and in front of the loads, and the MFMA pipe waits for them).
  // Loads: after barrier kt the activations of step kt+2 go into the stage just read; the weights
  // of step kt+3 follow in the units of step kt+1, into the weight stage freed by barrier kt.  A
  // step's weight loads are thus still in flight at the next barrier, and its wait leaves the
  // newest kLoadsW loads out.
  auto k_step = [&](int kt, auto as_c, auto wst_c) {
    constexpr int as = decltype(as_c)::value, wst = decltype(wst_c)::value;
    constexpr int as_next = as ^ 1, wst_next = (wst + 1) % D, wst_prev = (wst + D - 1) % D;
    // unit (0, 0) runs; weight fragments of (0, 1), first half of slice 1's activation fragments
    unit(0, 0, 0, wst, 0, 1, 1, as, 1, 1, 0, kHalf, false, as_next, kt + 1, wst_prev, kt - 1 + D, kAfterBarrier, kL1);
    // unit (0, 1) runs; weight fragments of (1, 0), the rest of slice 1's activation fragments
    unit(1, 0, 1, wst, 1, 0, 0, as, 1, 1, kHalf, NA, false, as_next, kt + 1, wst_prev, kt - 1 + D, kL1, kL2);
    // unit (1, 0) runs; weight fragments of (1, 1): the last reads of this stage
    unit(0, 1, 0, wst, 1, 1, 1, as, 1, 1, 0, 0, false, as_next, kt + 1, wst_prev, kt - 1 + D, kL2, kLoads);
    // this wave's loads of the next step are in LDS (step 0: behind them lie the previous epilogue's last stores) ...
    if (as == 0 && wst == 0 && kt == 0) {
      constexpr int kNewer = kLoadsW + kLastStores<EPI>;
      __builtin_amdgcn_s_waitcnt(0x0F70 | (kNewer & 15) | ((kNewer >> 4) << 14));
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70 | kLoadsW);
    }
    __syncthreads();  // ... everyone's are; nobody reads these stages any more
    // unit (1, 1) runs; all of unit (0, 0) of the next step
    unit(1, 1, 1, wst_next, 0, 0, 0, as_next, 0, 0, 0, NA, true, as, kt + 2, wst, kt + D, 0, kAfterBarrier);
  };
  {
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    int kt = 0;
    for (; kt + 6 < k_steps; kt += 6) {  // one to six steps are left behind it
      k_step(kt, I0{}, I0{});
      k_step(kt + 1, I1{}, I1{});
      k_step(kt + 2, I0{}, I2{});
      k_step(kt + 3, I1{}, I0{});
      k_step(kt + 4, I0{}, I1{});
      k_step(kt + 5, I1{}, I2{});
    }
    draws.request();  // of the next tile: the answer is there when the last steps are done
    if (kt < k_steps) k_step(kt, I0{}, I0{});
    if (kt + 1 < k_steps) k_step(kt + 1, I1{}, I1{});
    if (kt + 2 < k_steps) k_step(kt + 2, I0{}, I2{});
    if (kt + 3 < k_steps) k_step(kt + 3, I1{}, I0{});
    if (kt + 4 < k_steps) k_step(kt + 4, I0{}, I1{});
    if (kt + 5 < k_steps) k_step(kt + 5, I1{}, I2{});
  }
  // the compiler does not know that the assembly above is MFMAs: keep their results away from the
  // VALU reads of the epilogue for the wait states such reads need (at most 18)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  // The trailing loads (steps past the end of K, zero-length descriptor) still write zeros into
  // their stages, and each wave only waits for its own: the epilogue patches and the next tile's first stages
  // lie there.  Drain this wave's, then wait
  // until every wave has drained its own, before anybody writes a patch.
  char* const patch0 = smem + w_stage_off(2);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  draws.publish(patch0);  // into what only this wave's loads write
  draws.receive(patch0);

  // ---- epilogue.  acc[i][j] is the 16x16 block (weight fragment i) x (activation fragment j);
  // lane l holds activation row j*16 + l%16 and the 4 consecutive weight rows i*16 + 4*(l/16) + 0..3
  // -> 4 consecutive output columns.  Stored straight from there, a wave store would touch 16
  // rows with 8 bytes each; such partial-line writes cost the second GEMM 10 % (timed with the
  // stores removed).  So 32 rows at a time go through a per-wave LDS patch and leave as 16 bytes per lane, whole 128-byte
  // lines at a time.
  //
  // The four patches fill weight stage 2, 8 KiB each; the other stages take the next tile's first loads meanwhile.  A
  // patch row is 2 kWaveCols bytes, its 16-byte pieces XORed with the row: 16 rows at one column, or a row at 16
  // columns, fall into different banks.
  constexpr int kWaveCols = kGated ? 64 : 128;             // output columns of this wave
  constexpr int kPitch = kWaveCols * 2;
  constexpr int kLanesPerRow = kWaveCols / 8;              // 16-byte pieces of a patch row
  constexpr int kRowsPerStore = 64 / kLanesPerRow;
  char* const patch = patch0 + wave * 8192;
  const int quad = lane >> 4;
  // Before pass kTurn of kPasses the next tile is looked up, and its first loads go out one by one within the writes to the
  // patch of the last two passes (a burst of 32 holds the wave for 2600 to 4700 cycles, until the texture unit has taken it).
  constexpr int kPerRows = EPI == EPI_SWIGLU_KEEP ? 3 : EPI == EPI_GELU_KEEP ? 2 : 1;  // passes over the same 32 rows
  constexpr int kPasses = EPI == EPI_ACCUM ? 2 * XF : XF * kPerRows;
  constexpr int kFeedPasses = kPasses < 2 ? 1 : 2, kFeed0 = kPasses - kFeedPasses;
  constexpr int kTurn = kFeed0 - (GATHER && kFeed0 > 0 ? 1 : 0);
  Tile next;
  auto begin_pass = [&](int p) {
    if (p == kTurn) {
      next = draws.tile(kOutCols<EPI>);
      ops.set(args[PAIR ? __builtin_amdgcn_readfirstlane(next.part) : 0], smem, next);
    }
    if (p == kFeed0) ops.gather_rows(args[0]);
    __builtin_amdgcn_sched_barrier(0);
  };
  // after cell c of n of pass p's writes
  auto feed = [&](int p, int c, int n) {
    if (p < kFeed0) return;
    constexpr int kEach = kFirstLoads / kFeedPasses;
    const int l0 = (p - kFeed0) * kEach;
#pragma unroll
    for (int l = l0 + kEach * c / n; l < l0 + kEach * (c + 1) / n; ++l) ops.load_first(l);
  };
  // the accumulators of activation fragment j stay in their registers up to here (left alone, the compiler moves all 256
  // into VGPRs when the K loop ends, and spills)
  auto hold = [&](int j) {
#pragma unroll
    for (int i = 0; i < NW; ++i) asm volatile("" : "+a"(acc[i][j]));
  };
  const uint32_t n_rows = row_end - row0;
  // One pass of the 32 activation rows [32 jj, 32 jj + 32) through the patch: value(c, h, v) is the
  // number for patch row 16 h + l%16, patch column 16 c + 4 quad + v; the patch then leaves for
  // dst[row, col0 + ...], columns from col_end on are not stored (nor rows past the tile's end: their offsets lie
  // beyond the descriptor, so that a pass has the same number of stores everywhere).
  auto pass = [&](int p, auto value, uint16_t* dst, int ld, int col0, int col_end) {
    const int jj = p / kPerRows;
    begin_pass(p);
    hold(2 * jj);
    hold(2 * jj + 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 16 * h + (lane & 15);
#pragma unroll
      for (int c = 0; c < kWaveCols / 16; ++c) {
        uint2 pk;
        pk.x = pack_bf16x2(value(c, h, 0), value(c, h, 1));
        pk.y = pack_bf16x2(value(c, h, 2), value(c, h, 3));
        *(uint2*)(patch + r * kPitch + ((((2 * c) | (quad >> 1)) ^ (r & (kLanesPerRow - 1))) << 4) + (quad & 1) * 8) = pk;
        feed(p, h * (kWaveCols / 16) + c, kWaveCols / 8);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // keep the patch writes before the reads below
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const auto buf = __builtin_amdgcn_make_buffer_rsrc((void*)(dst + (size_t)row0 * ld), 0, (int)(n_rows * (uint32_t)ld * 2u), 0x00020000);
    const int lane_row = lane / kLanesPerRow, piece = lane % kLanesPerRow;
    const int col = col0 + piece * 8;  // row lengths are multiples of 8
    const uint32_t off = ((uint32_t)(wm * 32 * XF + lane_row) * (uint32_t)ld + (uint32_t)col) * 2u;
#pragma unroll
    for (int t = 0; t < 32 / kRowsPerStore; ++t) {
      const int r = t * kRowsPerStore + lane_row;
      const u32x4_t v = *(const u32x4_t*)(patch + r * kPitch + ((piece ^ (r & (kLanesPerRow - 1))) << 4));
      const uint32_t at = off + (uint32_t)(jj * 32 + t * kRowsPerStore) * (uint32_t)ld * 2u;
      __builtin_amdgcn_raw_buffer_store_b128(v, buf, (int)(col < col_end ? at : 0xFFFFFFF0u), 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // ... and the reads before the next pass's writes
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto rounded = [](float v) { return __uint_as_float(pack_bf16x2(v, 0.f) << 16); };  // the bf16 value that is stored
  const int out0 = n0 + wn * kWaveCols;
  if constexpr (EPI == EPI_ACCUM) {
    // fp32 read-modify-write of 16 rows x 128 columns at a time: through the patch into whole 512-byte runs of
    // the fp32 matrix, whose old values are fetched two passes ahead.  HBM bound where slots are short: an optimizer
    // step of two micro-batches on 128 slots of 192 rows (d = 2048, ffn = 1408, SwiGLU; 17.7 GB of old and new
    // sums in the weight gradients) takes 8.4 ms, 12.0 ms with 32 x 32 blocks read only when they are added.
    constexpr int kRuns = 8;  // 16-byte pieces per lane and pass, two rows per wave access
    const int piece = lane & 31, col = n0 + wn * 128 + piece * 4;  // row lengths are multiples of 8
    const bool col_ok = col < a.n_out;
    f32x4* const base = (f32x4*)(a.Cacc + (col_ok ? col : 0));
    auto row_of = [&](int j, int t) { return row0 + wm * 32 * XF + j * 16 + 2 * t + (lane >> 5); };
    f32x4 old[3][kRuns];
    auto fetch = [&](int j) {  // pieces outside the tile fetch its last row or the row's first column: not stored
#pragma unroll
      for (int t = 0; t < kRuns; ++t) {
        const int row = row_of(j, t);
        old[j % 3][t] = __builtin_nontemporal_load(base + (size_t)(row < row_end ? row : row_end - 1) * (a.n_out / 4));
      }
    };
    fetch(0);
    fetch(1);
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      begin_pass(j);
      if (j + 2 < NA) fetch(j + 2);
      hold(j);
      const int r = lane & 15;
#pragma unroll
      for (int c = 0; c < NW; ++c) {
        *(f32x4*)(patch + r * 512 + (((4 * c + quad) ^ r) << 4)) = acc[c][j];
        feed(j, c, NW);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int t = 0; t < kRuns; ++t) {
        const int pr = 2 * t + (lane >> 5), row = row_of(j, t);
        const f32x4 v = *(const f32x4*)(patch + pr * 512 + ((piece ^ pr) << 4));
        if (row < row_end && col_ok) __builtin_nontemporal_store(old[j % 3][t] + v, base + (size_t)row * (a.n_out / 4));
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    return next;
  }
  // Gated weights: the tile's 32-column groups alternate gate and up columns, so of a wave's eight
  // 16-wide weight fragments 0, 1, 4, 5 are gate columns and i + 2 holds the up columns of the same
  // outputs; output column block c (16 wide) of the wave comes from fragment 4 (c/2) + c%2.
  auto gate_frag = [](int c) { return 4 * (c >> 1) + (c & 1); };
#pragma unroll
  for (int jj = 0; jj < XF; ++jj) {
    if constexpr (EPI == EPI_SWIGLU) {
      pass(jj, [&](int c, int h, int v) { return silu_fast(acc[gate_frag(c)][2 * jj + h][v]) * acc[gate_frag(c) + 2][2 * jj + h][v]; },
           a.C, a.n_out, out0, a.n_out);
    } else if constexpr (EPI == EPI_SWIGLU_KEEP) {
      pass(3 * jj, [&](int c, int h, int v) { return acc[gate_frag(c)][2 * jj + h][v]; }, a.Z, a.z_cols, out0, a.n_out);
      pass(3 * jj + 1, [&](int c, int h, int v) { return acc[gate_frag(c) + 2][2 * jj + h][v]; }, a.Z, a.z_cols, a.up_row0 + out0,
           a.up_row0 + a.n_out);
      pass(3 * jj + 2, [&](int c, int h, int v) {
             return silu_fast(rounded(acc[gate_frag(c)][2 * jj + h][v])) * rounded(acc[gate_frag(c) + 2][2 * jj + h][v]);
           },
           a.C, a.n_out, out0, a.n_out);
    } else if constexpr (EPI == EPI_GELU_KEEP) {
      pass(2 * jj, [&](int c, int h, int v) { return acc[c][2 * jj + h][v]; }, a.Z, a.z_cols, out0, a.n_out);
      pass(2 * jj + 1, [&](int c, int h, int v) { return gelu_fast(rounded(acc[c][2 * jj + h][v])); }, a.C, a.n_out, out0, a.n_out);
    } else if constexpr (EPI == EPI_GELU) {
      pass(jj, [&](int c, int h, int v) { return gelu_fast(acc[c][2 * jj + h][v]); }, a.C, a.n_out, out0, a.n_out);
    } else {
      pass(jj, [&](int c, int h, int v) { return acc[c][2 * jj + h][v]; }, a.C, a.n_out, out0, a.n_out);
    }
  }
  return next;
}

// Persistent kernel: one workgroup per CU, whose matrix cores rest between two K loops.  What lies there is the draw of the
// next tile, its first loads and the epilogue: 4000, 5500 and 7000 cycles one after the other (weight gradients of 60
// slots of 680 rows, 768 x 3072, against 30500 of K loop), 13500 in all with the draw under the last K steps and
// the loads within the epilogue.  That training step (40960 tokens, top-1) 1795 -> 1737 us, the headline layer's (8192
// tokens, 4096 x 14336) 16350 -> 16090; both the texture unit's and the stores' paths are busy for half of the rest.
// The 32 tiles an XCD works on at a time share
// their activation and weight panels through that XCD's L2, and each XCD drains its queue at
// its own pace.  (The hardware hands the workgroups of an ordinary launch to the XCDs strictly
// in order of their index: there an XCD whose tiles take longer holds back the workgroups
// queued behind it for every other XCD, which costs 10-40 % on ragged plans.)
template <bool PAIR>
struct MfmaLaunch {
  MfmaArgs gemm[PAIR ? 2 : 1];
};
template <int EPI, int MODE, bool GATHER, bool KTAIL, bool PAIR>
__global__ __launch_bounds__(256, 1) void gemm_mfma_kernel(MfmaLaunch<PAIR> launch) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub, not the gfx950 builtins
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const MfmaArgs* const args = launch.gemm;
  Draws<PAIR> draws(args[0].u, args[PAIR ? 1 : 0].u, smem);
  Tile tile = draws.tile(kOutCols<EPI>);
  Operands<EPI, MODE, GATHER, KTAIL> ops;
  ops.set(args[PAIR ? __builtin_amdgcn_readfirstlane(tile.part) : 0], smem, tile);
  ops.gather_rows(args[0]);
  if (tile.slot >= 0) {
#pragma unroll
    for (int l = 0; l < kFirstLoads; ++l) ops.load_first(l);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // no stores are behind them
  }
  while (tile.slot >= 0) {
    const int rows = tile.row_end - tile.row0;  // 1..256
    if (rows > 192) tile = gemm_tile<EPI, 4, MODE, GATHER, KTAIL, PAIR>(args, smem, tile, ops, draws);
    else if (rows > 128) tile = gemm_tile<EPI, 3, MODE, GATHER, KTAIL, PAIR>(args, smem, tile, ops, draws);
    else if (rows > 64) tile = gemm_tile<EPI, 2, MODE, GATHER, KTAIL, PAIR>(args, smem, tile, ops, draws);
    else tile = gemm_tile<EPI, 1, MODE, GATHER, KTAIL, PAIR>(args, smem, tile, ops, draws);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the loads of no tile are done with LDS
  draws.finish();  // (a workgroup ends when it has received no tile, and has left then)
#endif
}

template <int EPI, int MODE, bool GATHER, bool KTAIL, bool PAIR = false>
int32_t launch_mfma_kernel(const MfmaLaunch<PAIR>& a, hipStream_t st) {
  static_assert(!GATHER || MODE == MODE_NN, "the gather is part of the forward's first GEMM only");
  void (*kern)(MfmaLaunch<PAIR>) = gemm_mfma_kernel<EPI, MODE, GATHER, KTAIL, PAIR>;
  // per device: the LDS attribute is set on the first launch there (idempotent, so two threads racing through
  // the set-up do the same thing twice)
  static std::atomic<int> workgroups_of_device[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LZ_EHIP;
  int n_workgroups = workgroups_of_device[dev].load(std::memory_order_acquire);
  if (n_workgroups == 0) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) !=
        hipSuccess)
      return LZ_EHIP;
    n_workgroups = device_cus();  // one per CU (the LDS a workgroup takes allows no more)
    if (n_workgroups == 0) return LZ_EHIP;
    workgroups_of_device[dev].store(n_workgroups, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3(n_workgroups), dim3(256), kLdsBytes, st, a);
  return lz::launch_status();
}

template <int EPI, int MODE = MODE_NT, bool GATHER = false>
int32_t launch_mfma(const MfmaArgs& a, hipStream_t st) {
  if constexpr (MODE == MODE_NT || MODE == MODE_NN) {
    if (a.K % BK != 0) return launch_mfma_kernel<EPI, MODE, GATHER, true>(MfmaLaunch<false>{{a}}, st);
  }
  return launch_mfma_kernel<EPI, MODE, GATHER, false>(MfmaLaunch<false>{{a}}, st);
}

// Both weight gradients of a backward pass in one launch.
template <int EPI>
int32_t launch_mfma_pair(const MfmaArgs& a0, const MfmaArgs& a1, hipStream_t st) {
  return launch_mfma_kernel<EPI, MODE_TN, false, false, true>(MfmaLaunch<true>{{a0, a1}}, st);
}

// bf16 shapes the MFMA kernel takes: rows of whole 16-byte pieces, one slot's weights and one 256-row
// activation tile (rows of d, ffn or, dZ, n1 elements) within 32-bit byte offsets.
inline bool mfma_sizes(const lz_shape* s) {
  if (s->dtype != LZ_BF16 || s->d % 8 != 0 || s->ffn % 8 != 0 || (long long)s->d * s->ffn * 4 >= (1ll << 31)) return false;
  const long long n1 = (long long)s->ffn * (s->act == LZ_SWIGLU ? 2 : 1);
  if ((long long)BM * 2 * (s->d > n1 ? s->d : n1) >= (1ll << 32)) return false;
  // KTAIL sets bit 31 of such an offset
  return (s->d % BK == 0 && s->ffn % BK == 0) || (long long)BM * (s->d > s->ffn ? s->d : s->ffn) * 4 < (1ll << 31);
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace
