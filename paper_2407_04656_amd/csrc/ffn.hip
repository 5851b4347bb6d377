// Expert FFN as a grouped GEMM over the per-slot row ranges (Sec. 2.1: experts are
// parallel FFNs; every replica processes the rows dispatched to its slot).
//
//   GEMM-1   hidden[P, ffn] = act(xp[P, d] * W1[slot])        act = GELU | SwiGLU, fused;  W1[slot] = [d, n1]
//   GEMM-2   yp[P, d]       = hidden[P, ffn] * W2[slot]                                        W2[slot] = [ffn, d]
//
// Group sizes are data dependent and only known on the device, so a small kernel
// first turns slot_offsets into a table of row tiles (slot, first row, end row) or, for the
// wide MFMA kernel, into one list of work units per XCD.
//
// bf16 path: the MFMA kernel of gemm_mfma.h.
//
// fp32 tensors, and bf16 rows that are no whole 16-byte pieces: the fp32 matrix-core kernel of gemm_f32.h.
#include "gemm_split.h"
#include "gemm_narrow.h"
#include "layer.h"

namespace {

// Shapes on the MFMA kernels: every bf16 shape whose rows are whole 16-byte pieces.  Where a size is no
// multiple of the tile the kernel computes the tile's padding too and stores the real part; a forward
// of T = 3001, d = 1000, ffn = 2664, top-2 over 12 slots, SwiGLU: 2413 us on an fp32-FMA kernel, 200 us here.
// Their activations are this kernel's (hardware exp2 and rcp, see gelu_fast), not the fp32 kernel's erff and expf: after the
// rounding to bf16 both have the same error.
// Sizes that are not whole_tiles additionally accept unaligned tensors (on the fp32 kernel) and fused gathers of any
// x; the MFMA gather's 32-bit offsets hold x up to 2 GiB there, and a shape decides for all its calls.
inline bool whole_tiles(const lz_shape* s) {
  return s->d % BN == 0 && s->ffn % 64 == 0 && s->ffn % (s->act == LZ_SWIGLU ? BN / 2 : BN) == 0;
}
inline bool mfma_shape(const lz_shape* s) {
  return mfma_sizes(s) && (whole_tiles(s) || (long long)s->T * s->d * 2 < (1ll << 31));
}

struct FfnWorkspace {
  void* hidden;
  void* units_up;      // of the wide bf16 GEMMs
  void* units_down;
  void* tiles_narrow;  // of the GEMMs on narrow tiles
  void* tiles_f32;     // of the fp32 kernel
  void* tiles_split;   // of the split fp32 kernel
  size_t total_bytes;
  int n_up, n_down;    // column tiles of the two wide GEMMs
  bool narrow_up, narrow_down;  // GEMMs on narrow tiles
};

UnitTable units_up_of(const FfnWorkspace& w, const lz_shape* s) {
  return carve_units(w.units_up, (long long)s->T * s->k, s->N * s->c, w.n_up);
}

UnitTable units_down_of(const FfnWorkspace& w, const lz_shape* s) {
  return carve_units(w.units_down, (long long)s->T * s->k, s->N * s->c, w.n_down);
}

TileTable narrow_tiles_of(const FfnWorkspace& w, const lz_shape* s) {
  return carve_tiles(w.tiles_narrow, (long long)s->T * s->k, s->N * s->c, kNarrow);
}

TileTable f32_tiles_of(const FfnWorkspace& w, const lz_shape* s) {
  return carve_tiles(w.tiles_f32, (long long)s->T * s->k, s->N * s->c, kF32Rows);
}

TileTable split_tiles_of(const FfnWorkspace& w, const lz_shape* s) {
  return carve_tiles(w.tiles_split, (long long)s->T * s->k, s->N * s->c, kSplitRows);
}

// Every table that some number of tokens of the same layer uses has its room, so that a workspace made for the
// largest batch serves the smaller ones.
FfnWorkspace carve_ffn(void* ws, const lz_shape* s) {
  FfnWorkspace w{};
  const long long P = (long long)s->T * s->k;
  const int S = s->N * s->c;
  w.n_up = ceil_div(s->ffn, s->act == LZ_SWIGLU ? BN / 2 : BN);
  w.n_down = ceil_div(s->d, BN);
  char* p = (char*)ws;
  auto take = [&](size_t bytes) {
    char* r = p;
    p += lz::align256(bytes);
    return r;
  };
  w.hidden = take((size_t)P * s->ffn * lz::elem_bytes(s->dtype));
  if (mfma_sizes(s)) {
    w.units_up = take(unit_table_bytes(P, S, w.n_up));
    w.units_down = take(unit_table_bytes(P, S, w.n_down));
    w.tiles_narrow = take(tile_table_bytes(P, S, kNarrow));
  }
  if (!mfma_sizes(s) || !whole_tiles(s)) w.tiles_f32 = take(tile_table_bytes(P, S, kF32Rows));
  if (s->dtype == LZ_F32) w.tiles_split = take(tile_table_bytes(P, S, kSplitRows));
  w.narrow_up = mfma_shape(s) && s->act == LZ_GELU && use_narrow(P, S, s->ffn);
  w.narrow_down = mfma_shape(s) && use_narrow(P, S, s->d);
  w.total_bytes = size_t(p - (char*)ws);
  return w;
}

}  // namespace

extern "C" size_t lz_ffn_workspace_bytes(const lz_shape* shape) {
  if (!lz::shape_ok(shape)) return 0;
  return carve_ffn(nullptr, shape).total_bytes;
}

namespace {

int32_t check_ffn(const lz_shape* shape, void* ws, size_t ws_bytes, FfnWorkspace* w) {
  if (!lz::shape_ok(shape)) return LZ_ESHAPE;
  *w = carve_ffn(ws, shape);
  if (!ws || (uintptr_t)ws % 256 != 0 || ws_bytes < w->total_bytes) return LZ_EWORKSPACE;
  return LZ_OK;
}

}  // namespace

namespace {

TileSpecs tables_of(const FfnWorkspace& w, const lz_shape* shape) {
  const long long P = (long long)shape->T * shape->k;
  TileSpecs specs{};
  if (mfma_shape(shape)) {
    if (!w.narrow_up) add_units(specs, w.n_up, 0, P, units_up_of(w, shape));
    if (!w.narrow_down) add_units(specs, w.n_down, 0, P, units_down_of(w, shape));
  }
  if (w.narrow_up || w.narrow_down) add_rows(specs, kNarrow, P, narrow_tiles_of(w, shape));
  // the calls that follow may bring unaligned tensors where that is allowed
  if (!mfma_shape(shape) || !whole_tiles(shape)) add_rows(specs, kF32Rows, P, f32_tiles_of(w, shape));
  if (split_forward(shape)) add_rows(specs, kSplitRows, P, split_tiles_of(w, shape));
  return specs;
}

}  // namespace

TileSpecs lz::ffn_tables(const lz_shape* shape, void* ws, size_t ws_bytes) {
  FfnWorkspace w;
  if (check_ffn(shape, ws, ws_bytes, &w) != LZ_OK || (long long)shape->T * shape->k == 0) return TileSpecs{};
  return tables_of(w, shape);
}

extern "C" int32_t lz_ffn_tiles(const int32_t* slot_offsets, const lz_shape* shape, void* ws,
                                size_t ws_bytes, void* stream) {
  FfnWorkspace w;
  const int32_t rc = check_ffn(shape, ws, ws_bytes, &w);
  if (rc != LZ_OK) return rc;
  if ((long long)shape->T * shape->k == 0) return LZ_OK;
  if (!slot_offsets) return LZ_EINVAL;
  return launch_build_tiles(slot_offsets, shape->N * shape->c, tables_of(w, shape), (hipStream_t)stream);
}

namespace {

// hidden = act(A W1) per slot; A = xp, or x read through the row map when `gather` is given
int32_t ffn_up(const void* xp, const int32_t* gather, const void* w1, const lz_shape* shape, void* ws,
               size_t ws_bytes, void* stream) {
  FfnWorkspace w;
  const int32_t rc = check_ffn(shape, ws, ws_bytes, &w);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  if (P == 0) return LZ_OK;
  if (!xp || !w1) return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const bool swiglu = shape->act == LZ_SWIGLU;
  const int n1 = shape->ffn * (swiglu ? 2 : 1);
  const int gk = shape->k;
  const long long gT = shape->T;
  const bool aligned = aligned16(xp) && aligned16(w1);  // 16-byte loads per lane
  if (!mfma_shape(shape) || (!aligned && !whole_tiles(shape))) {
    F32Args a{};
    a.A = xp;
    a.W = w1;
    a.C = w.hidden;
    a.K = a.lda = shape->d;
    a.ldw = n1;
    a.w_slot = (long long)shape->d * n1;
    a.ldc = a.n_out = a.ffn = shape->ffn;
    a.t = f32_tiles_of(w, shape);
    a.t_split = split_tiles_of(w, shape);
    a.gather = gather;
    a.gather_k = gk;
    a.gather_T = gT;
    const int S = shape->N * shape->c;
    if (shape->dtype == LZ_F32)
      return swiglu ? launch_f32_rows<float, EPI_SWIGLU, true>(a, S, P, st)
                    : launch_f32_rows<float, EPI_GELU, true>(a, S, P, st);
    return swiglu ? launch_f32_rows<uint16_t, EPI_SWIGLU, true>(a, S, P, st)
                  : launch_f32_rows<uint16_t, EPI_GELU, true>(a, S, P, st);
  }
  if (!aligned) return LZ_EINVAL;
  // the MFMA gather addresses all of x with 32-bit byte offsets
  if (gather && (unsigned long long)shape->T * shape->d * 2ull >= (1ull << 32)) return LZ_ESHAPE;
  MfmaArgs g1{};
  g1.A = (const uint16_t*)xp;
  g1.W = (const uint16_t*)w1;
  g1.C = (uint16_t*)w.hidden;
  g1.P = P;
  g1.K = shape->d;
  g1.w_rows = n1;
  g1.n_out = shape->ffn;
  g1.up_row0 = swiglu ? shape->ffn : 0;
  g1.n_tiles = w.n_up;
  g1.u = units_up_of(w, shape);
  g1.ldw = n1;
  g1.gather = gather;
  g1.gather_k = gk;
  g1.gather_T = gT;
  if (w.narrow_up)
    return gather ? launch_narrow<EPI_GELU, MODE_NN, true>(g1, narrow_tiles_of(w, shape), st)
                  : launch_narrow<EPI_GELU, MODE_NN>(g1, narrow_tiles_of(w, shape), st);
  if (gather)
    return swiglu ? launch_mfma<EPI_SWIGLU, MODE_NN, true>(g1, st) : launch_mfma<EPI_GELU, MODE_NN, true>(g1, st);
  return swiglu ? launch_mfma<EPI_SWIGLU, MODE_NN>(g1, st) : launch_mfma<EPI_GELU, MODE_NN>(g1, st);
}

}  // namespace

extern "C" int32_t lz_ffn_up(const void* xp, const void* w1, const lz_shape* shape, void* ws,
                             size_t ws_bytes, void* stream) {
  return ffn_up(xp, nullptr, w1, shape, ws, ws_bytes, stream);
}

extern "C" int32_t lz_ffn_up_gather(const void* x, const int32_t* row_to_pair, const void* w1,
                                    const lz_shape* shape, void* ws, size_t ws_bytes, void* stream) {
  if (!row_to_pair && shape && (long long)shape->T * shape->k > 0) return LZ_EINVAL;
  return ffn_up(x, row_to_pair, w1, shape, ws, ws_bytes, stream);
}

extern "C" int32_t lz_ffn_down(const void* w2, const lz_shape* shape, void* yp, void* ws,
                               size_t ws_bytes, void* stream) {
  FfnWorkspace w;
  const int32_t rc = check_ffn(shape, ws, ws_bytes, &w);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  if (P == 0) return LZ_OK;
  if (!w2 || !yp) return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const bool aligned = aligned16(yp) && aligned16(w2);  // 16-byte accesses per lane
  if (!mfma_shape(shape) || (!aligned && !whole_tiles(shape))) {
    F32Args a{};
    a.A = w.hidden;
    a.W = w2;
    a.C = yp;
    a.K = a.lda = shape->ffn;
    a.w_slot = (long long)shape->ffn * shape->d;
    a.ldw = a.ldc = a.n_out = shape->d;
    a.t = f32_tiles_of(w, shape);
    a.t_split = split_tiles_of(w, shape);
    const int S = shape->N * shape->c;
    return shape->dtype == LZ_F32 ? launch_f32_rows<float, EPI_NONE, true>(a, S, P, st)
                                  : launch_f32_rows<uint16_t, EPI_NONE, true>(a, S, P, st);
  }
  if (!aligned) return LZ_EINVAL;
  MfmaArgs g2{};
  g2.A = (const uint16_t*)w.hidden;
  g2.W = (const uint16_t*)w2;
  g2.C = (uint16_t*)yp;
  g2.P = P;
  g2.K = shape->ffn;
  g2.w_rows = shape->d;
  g2.n_out = shape->d;
  g2.up_row0 = 0;
  g2.n_tiles = w.n_down;
  g2.u = units_down_of(w, shape);
  g2.ldw = shape->d;
  if (w.narrow_down) return launch_narrow<EPI_NONE, MODE_NN>(g2, narrow_tiles_of(w, shape), st);
  return launch_mfma<EPI_NONE, MODE_NN>(g2, st);
}

extern "C" int32_t lz_expert_ffn(const void* xp, const int32_t* slot_offsets, const void* w1,
                                 const void* w2, const lz_shape* shape, void* yp, void* ws,
                                 size_t ws_bytes, void* stream) {
  int32_t rc = lz_ffn_tiles(slot_offsets, shape, ws, ws_bytes, stream);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  if (P == 0) return LZ_OK;
  if (!xp || !w1 || !w2 || !yp) return LZ_EINVAL;
  rc = lz_ffn_up(xp, w1, shape, ws, ws_bytes, stream);
  if (rc != LZ_OK) return rc;
  return lz_ffn_down(w2, shape, yp, ws, ws_bytes, stream);
}

extern "C" int32_t lz_expert_ffn_gather(const void* x, const int32_t* row_to_pair, const int32_t* slot_offsets,
                                        const void* w1, const void* w2, const lz_shape* shape, void* yp,
                                        void* ws, size_t ws_bytes, void* stream) {
  int32_t rc = lz_ffn_tiles(slot_offsets, shape, ws, ws_bytes, stream);
  if (rc != LZ_OK) return rc;
  const long long P = (long long)shape->T * shape->k;
  if (P == 0) return LZ_OK;
  if (!x || !row_to_pair || !w1 || !w2 || !yp) return LZ_EINVAL;
  rc = lz_ffn_up_gather(x, row_to_pair, w1, shape, ws, ws_bytes, stream);
  if (rc != LZ_OK) return rc;
  return lz_ffn_down(w2, shape, yp, ws, ws_bytes, stream);
}

// ------------------------------------------------------------------------------------------
// Diagnostic: which XCD does the hardware give the workgroups of a launch shaped like the
// persistent GEMM's (256 threads, the same dynamic LDS, hence one workgroup per CU)?
// ------------------------------------------------------------------------------------------
namespace {
__global__ __launch_bounds__(256, 1) void xcc_ids_kernel(int32_t* __restrict__ out) {
  extern __shared__ __attribute__((aligned(1024))) char smem_probe[];
  uint32_t id;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
  if (threadIdx.x == 0) out[blockIdx.x] = (int32_t)(id & 0xFu);
}
}  // namespace

extern "C" int32_t lz_debug_xcc_ids(int32_t* xcc_of_workgroup, int32_t n_workgroups, void* stream) {
  if (n_workgroups < 0 || n_workgroups > 65535) return LZ_EINVAL;
  if (n_workgroups == 0) return LZ_OK;
  if (!xcc_of_workgroup) return LZ_EINVAL;
  if (hipFuncSetAttribute((const void*)xcc_ids_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) !=
      hipSuccess)
    return LZ_EHIP;
  hipLaunchKernelGGL(xcc_ids_kernel, dim3(n_workgroups), dim3(256), kLdsBytes, (hipStream_t)stream,
                     xcc_of_workgroup);
  return lz::launch_status();
}
