// The grouped bf16 GEMM of gemm_mfma.h on 64 x 64 tiles, for launches whose 256 x 256 tiles are too few for the
// chip: a batch of some tens or hundreds of tokens, whose GEMMs are a stream of weights that a quarter of the
// CUs or fewer would read.  4 waves in 2 x 2, each 32 x 32; two workgroups share a CU.  Same operand layouts,
// swizzled direct-to-LDS loads and K order as the wide kernel (a row's result has the same bits on either), but
// one ring of whole K steps for both operands: a workgroup keeps three steps of 16 KiB in flight (96 KiB a CU)
// and leaves the order of LDS reads and MFMAs to the compiler.  Measured (rows per slot x slots, K x columns;
// wide, narrow): 8 x 16, 4096 x 1024 35, 24 us; 60 x 8, 768 x 3072 GELU 21, 13; 300 x 12, 3072 x 768 58, 45;
// 200 x 40, 512 x 512 GELU 30, 19.  128 x 64 tiles were within 15 % of these either way; the gated first GEMM was
// slower on either (32 gate + 32 up columns are 64-byte runs of W: 50, 79 us), so it has no narrow form.
// Device code, not part of the C ABI.
#pragma once
#include "gemm_mfma.h"

namespace {

constexpr int kNarrow = 64;                             // rows and columns of a tile
constexpr int kNarrowStages = 4;
constexpr int kNarrowOperand = kNarrow * kRowBytes;      // 8 KiB of either operand per K step
constexpr int kNarrowStage = 2 * kNarrowOperand;
constexpr int kNarrowLds = kNarrowStages * kNarrowStage;  // 64 KiB

// k-major W tile: 64 k-rows of 128 B (8 pieces of 16 B).  A transposing read is served 32 lanes at a time: 4
// consecutive k-rows and the 4 eight rows on, 32 bytes each.  Two k-rows fill the 64 banks, so the key moves
// row pairs 64 bytes and the second group 32 bytes apart: eight different bank groups.
__device__ __forceinline__ int swz_narrow(int kr) { return (((kr >> 1) & 1) << 2) | (((kr >> 3) & 1) << 1); }

// blockIdx.x = row tile of the table (64 rows) x column tile, columns fastest and padded
// to a multiple of 8 from 8 on: the row tiles that share a column panel of W run on one XCD.
template <int EPI, int MODE, bool GATHER, bool KTAIL>
__global__ __launch_bounds__(256, 2) void gemm_narrow_kernel(MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr bool TB = MODE == MODE_NN;  // W k-major
  static_assert(EPI == EPI_NONE || EPI == EPI_GELU || EPI == EPI_GELU_KEEP, "no gated narrow tiles");
  constexpr int NS = kNarrowStages, kLoadsX = 2, kLoadsW = 2, kLoads = kLoadsX + kLoadsW;  // 1-KiB loads per wave and step
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int n_pad = a.n_tiles < 8 ? a.n_tiles : (a.n_tiles + 7) / 8 * 8;
  const int row_tile = blockIdx.x / n_pad, col_tile = blockIdx.x % n_pad;
  if (col_tile >= a.n_tiles || row_tile >= a.t.header[0]) return;
  const int slot = __builtin_amdgcn_readfirstlane(a.t.slot[row_tile]);
  const int row0 = __builtin_amdgcn_readfirstlane(a.t.row0[row_tile]);
  const int row_end = __builtin_amdgcn_readfirstlane(a.t.row_end[row_tile]);
  const int n0 = col_tile * kNarrow;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int n_rows = row_end - row0 < kNarrow ? row_end - row0 : kNarrow;
  const int K = a.K;

  // ---- descriptors and per-lane offsets, as in the wide kernel
  const uint16_t* const tileA = GATHER ? a.A : a.A + (size_t)row0 * K;
  const uint32_t a_extent = GATHER ? (uint32_t)((unsigned long long)a.gather_T * (unsigned)K * 2ull) : (uint32_t)n_rows * (uint32_t)K * 2u;
  const uint16_t* const tileW = TB ? a.W + (size_t)slot * K * a.ldw : a.W + (size_t)slot * a.w_rows * K;
  const uint32_t w_extent = TB ? (uint32_t)K * (uint32_t)a.ldw * 2u : (uint32_t)((unsigned long long)a.w_rows * K * 2);
  const int stepW = TB ? BK * a.ldw * 2 : BK * 2;
  const i32x4 wordsA = rsrc_words(tileA, a_extent), wordsW = rsrc_words(tileW, w_extent), wordsNull = rsrc_words(a.A, 0);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  int voffX[kLoadsX], voffW[kLoadsW];
#pragma unroll
  for (int i = 0; i < kLoadsX; ++i) {
    const int r = (wave * kLoadsX + i) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ swz(r);
    const int ga = r < n_rows ? r : n_rows - 1;  // rows past the tile's end repeat its last row (never stored)
    if constexpr (GATHER) {
      const uint32_t pair = (uint32_t)a.gather[row0 + ga], n_pairs = (uint32_t)(a.gather_T * a.gather_k);
      voffX[i] = pair < n_pairs ? (int)((pair / (uint32_t)a.gather_k * (uint32_t)K + (uint32_t)chunk * 8u) * 2u) : (int)a_extent;
    } else {
      voffX[i] = (int)(((uint32_t)ga * (uint32_t)K + (uint32_t)chunk * 8u) * 2u);
    }
  }
#pragma unroll
  for (int i = 0; i < kLoadsW; ++i) {
    const int r = (wave * kLoadsW + i) * 8 + (lane >> 3);  // k-row (k-major) or weight row
    if constexpr (TB) {
      const int piece = (lane & 7) ^ swz_narrow(r);
      voffW[i] = (int)(((uint32_t)r * (uint32_t)a.ldw + (uint32_t)(n0 + piece * 8)) * 2u);
    } else {
      const int chunk = (lane & 7) ^ swz(r);
      voffW[i] = (int)(((uint32_t)(n0 + r) * (uint32_t)K + (uint32_t)chunk * 8u) * 2u);
    }
  }
  [[maybe_unused]] int tail_or[2] = {0, 0};  // last K step, see the wide kernel
  if constexpr (KTAIL) {
    const int k_left = K - (K - 1) / BK * BK;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      tail_or[i] = ((lane & 7) ^ swz(i * 8 + (lane >> 3))) * 8 >= k_left ? (int)0x80000000 : 0;
  }
  const int k_steps = (K + BK - 1) / BK;
  auto issue = [&](int step, int stage) {  // a step past the end writes zeros, without memory traffic
    const bool real = step < k_steps;
    const i32x4 wa = real ? wordsA : wordsNull, ww = real ? wordsW : wordsNull;
    const uint32_t lds = lds0 + stage * kNarrowStage;
    const int tail = step == k_steps - 1 ? -1 : 0;
#pragma unroll
    for (int i = 0; i < kLoadsW; ++i) {
      int voff = voffW[i];
      if constexpr (KTAIL && !TB) voff |= tail_or[i & 1] & tail;
      load16_to_lds(ww, lds + kNarrowOperand + (wave * kLoadsW + i) * 1024, voff, real ? step * stepW : 0);
    }
#pragma unroll
    for (int i = 0; i < kLoadsX; ++i) {
      int voff = voffX[i];
      if constexpr (KTAIL) voff |= tail_or[i & 1] & tail;
      load16_to_lds(wa, lds + (wave * kLoadsX + i) * 1024, voff, real ? step * BK * 2 : 0);
    }
  };

  // ---- fragment addresses inside a stage: 16 rows x 32 k of the activations, 32 k x 16 columns of W
  int fragoff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int r = lane & 15;
    fragoff[ks] = r * kRowBytes + (((ks * 4 + (lane >> 4)) ^ swz(r)) << 4);
  }
  int woff[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if constexpr (TB) {
      const int q = lane & 15, kr = 8 * (lane >> 4) + (q >> 2);
      woff[c] = kr * kRowBytes + ((q & 1) << 3) + (((((2 * wn + c) << 1) | ((q >> 1) & 1)) ^ swz_narrow(kr)) << 4);
    } else {
      woff[c] = (2 * wn + c) * 16 * kRowBytes;
    }
  }
  auto read_x = [&](const char* st, int ks, int j) { return *(const bf16x8*)(st + (2 * wm + j) * 16 * kRowBytes + fragoff[ks]); };
  auto read_w = [&](const char* st, int ks, int c) {
    if constexpr (TB) {
      const char* p = st + kNarrowOperand + woff[c] + ks * 32 * kRowBytes;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p);
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p + 4 * kRowBytes));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      return *(const bf16x8*)(st + kNarrowOperand + woff[c] + fragoff[ks]);
    }
  };

  f32x4 acc[2][2] = {};
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) issue(s, s);
  int stage = 0;
  for (int kt = 0; kt < k_steps; ++kt) {
    constexpr int kAhead = (NS - 2) * kLoads;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (kAhead & 15) | ((kAhead >> 4) << 14));  // this wave's loads of step kt are in LDS
    __syncthreads();  // ... everyone's are; and nobody reads the stage of step kt - 1 any more
    const int prev = stage == 0 ? NS - 1 : stage - 1;
    issue(kt + NS - 1, prev);
    const char* const st = smem + stage * kNarrowStage;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 x[2], w[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) w[c] = read_w(st, ks, c);
#pragma unroll
      for (int j = 0; j < 2; ++j) x[j] = read_x(st, ks, j);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[c], x[j], acc[c][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }
  // the trailing loads still write zeros into stages: drained by every wave before the patches overwrite them
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  // ---- epilogue: lane l of acc[c][j] holds row 16 j + l % 16 and the columns 16 c + 4 (l / 16) + 0..3; the wave's
  // 32 x 32 block leaves through a patch of its own in 16-byte pieces
  constexpr int kPitch = 32 * 2 + 16;
  char* const patch = smem + wave * (32 * kPitch);
  const int quad = lane >> 4;
  auto pass = [&](auto value, uint16_t* dst, int ld) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        uint2 pk;
        pk.x = pack_bf16x2(value(acc[c][h][0]), value(acc[c][h][1]));
        pk.y = pack_bf16x2(value(acc[c][h][2]), value(acc[c][h][3]));
        *(uint2*)(patch + (16 * h + (lane & 15)) * kPitch + (c * 16 + 4 * quad) * 2) = pk;
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = t * 16 + (lane >> 2), piece = lane & 3;
      const uint4 v = *(const uint4*)(patch + r * kPitch + piece * 16);
      const int row = row0 + wm * 32 + r, col = n0 + wn * 32 + piece * 8;
      if (row < row_end && col < a.n_out) *(uint4*)(dst + (size_t)row * ld + col) = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto same = [](float v) { return v; };
  auto rounded = [](float v) { return __uint_as_float(pack_bf16x2(v, 0.f) << 16); };
  if constexpr (EPI == EPI_GELU_KEEP) {
    pass(same, a.Z, a.z_cols);
    pass([&](float v) { return gelu_fast(rounded(v)); }, a.C, a.n_out);
  } else if constexpr (EPI == EPI_GELU) {
    pass([](float v) { return gelu_fast(v); }, a.C, a.n_out);
  } else {
    pass(same, a.C, a.n_out);
  }
#endif
}

template <int EPI, int MODE, bool GATHER, bool KTAIL>
int32_t launch_narrow_kernel(const MfmaArgs& a, hipStream_t st) {
  void (*kern)(MfmaArgs) = gemm_narrow_kernel<EPI, MODE, GATHER, KTAIL>;
  static std::atomic<bool> ready_on_device[kMaxDevices];  // the LDS attribute is set (idempotent)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LZ_EHIP;
  if (!ready_on_device[dev].load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kNarrowLds) != hipSuccess)
      return LZ_EHIP;
    ready_on_device[dev].store(true, std::memory_order_release);
  }
  const int n_pad = a.n_tiles < 8 ? a.n_tiles : (a.n_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.t.capacity * n_pad)), dim3(256), kNarrowLds, st, a);
  return lz::launch_status();
}

// `a` as for the wide kernel (its n_tiles is replaced), t: the table of 64-row tiles
template <int EPI, int MODE, bool GATHER = false>
int32_t launch_narrow(MfmaArgs a, const TileTable& t, hipStream_t st) {
  a.t = t;
  a.n_tiles = ceil_div(a.n_out, kNarrow);
  if (a.K % BK != 0) return launch_narrow_kernel<EPI, MODE, GATHER, true>(a, st);
  return launch_narrow_kernel<EPI, MODE, GATHER, false>(a, st);
}

// Whether a GEMM over the batch's rows runs on narrow tiles: where it has fewer than 96 wide ones (half a tile
// more per slot that can have rows).  In the sweep the figures above are from, all 15 launches under 93 gained, by
// 4 % (64 tiles, 940 MB of weights) to half; of the eight from 100 to 150 six lost, 11 to 51 %, and the two of
// 40 slots with rows of 512 gained (30 -> 19, 22 -> 18 us), as did two of 196 and 294 tiles with 3 rows a slot (58 ->
// 53, 66 -> 55): the tile count alone does not tell these apart.  And where one narrow tile holds all columns,
// three quarters and more of a wide one are padding: 40000 rows of 8 columns to 8 over 32 slots 40 -> 19 us a
// forward, 64 to 64 40 -> 19 (a grid has fewer than 2^32 threads: a workgroup per 64 rows of P up to 2^28).
inline bool use_narrow(long long P, int S, int n_out) {
  const long long used = P < S ? P : S;
  return (n_out <= kNarrow && P <= (1ll << 28)) || (P / BM + (used + 1) / 2) * ceil_div(n_out, BN) < 96;
}

}  // namespace
