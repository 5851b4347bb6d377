// Error strings, version, the one-time conversion of expert weights into the library's
// input-major layout, and the device-side weight copies of a re-plan (Sec. 4.3 / 5: the state
// transfers that move expert replicas to their new slots).
#include <algorithm>
#include <new>
#include <vector>

#include "lz_common.h"

namespace {

// The transfers of one launch, by value: destinations ordered by source slot, so that a source is read once for
// all the slots it goes to.
constexpr int kCopySources = 128, kCopySlots = 256;
struct CopyList {
  int32_t src[kCopySources];
  int32_t first[kCopySources + 1];  // destinations of source g: dst[first[g]] .. dst[first[g + 1] - 1]
  int32_t dst[kCopySlots];
  int32_t sources;
};
struct CopyMatrix {
  const void* from;
  void* to;
  long long vecs;  // 16-byte pieces of a slot
};
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kCopyAhead = 4;  // pieces of a thread, 256 apart, loaded before the first is stored

// blockIdx.y = source, blockIdx.z = matrix.  HBM bound: every source read once, every destination written once,
// at the rate of a plain large copy.  48 slots filled from 32 experts of 67 MB: 1318 us as 96 device copies
// (each destination re-reads its source, 4.9 TB/s of that), 901 us.
__global__ __launch_bounds__(256) void copy_slots_kernel(CopyList list, CopyMatrix a, CopyMatrix b) {
  const CopyMatrix m = blockIdx.z == 0 ? a : b;
  const long long v0 = (long long)blockIdx.x * (256 * kCopyAhead) + threadIdx.x;
  const u32x4* const from = (const u32x4*)m.from + (size_t)list.src[blockIdx.y] * m.vecs;
  u32x4 in[kCopyAhead];
#pragma unroll
  for (int u = 0; u < kCopyAhead; ++u)
    if (v0 + u * 256 < m.vecs) in[u] = __builtin_nontemporal_load(from + v0 + u * 256);
  for (int i = list.first[blockIdx.y]; i < list.first[blockIdx.y + 1]; ++i) {
    u32x4* const to = (u32x4*)m.to + (size_t)list.dst[i] * m.vecs;
#pragma unroll
    for (int u = 0; u < kCopyAhead; ++u)
      if (v0 + u * 256 < m.vecs) __builtin_nontemporal_store(in[u], to + v0 + u * 256);
  }
}

inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// Whether all of `ptrs` is memory of the stream's own GPU: only that can a kernel read and write without peer access
// or a mapping; a device-to-device copy finds its way between any two places.
bool on_device_of(hipStream_t st, const void* const* ptrs, int n) {
  hipDevice_t dev = 0;
  if (hipStreamGetDevice(st, &dev) != hipSuccess) return (void)hipGetLastError(), false;
  for (int i = 0; i < n; ++i) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, ptrs[i]) != hipSuccess) return (void)hipGetLastError(), false;
    if (at.type != hipMemoryTypeDevice || at.device != dev) return false;
  }
  return true;
}

int32_t copy_slots(std::vector<lz_transfer>& order, CopyMatrix a, CopyMatrix b, hipStream_t st) {
  const int n = (int)order.size();
  std::stable_sort(order.begin(), order.end(), [](const lz_transfer& x, const lz_transfer& y) { return x.src_slot < y.src_slot; });
  const long long vecs = a.vecs > b.vecs ? a.vecs : b.vecs;
  const unsigned blocks = (unsigned)((vecs + 256 * kCopyAhead - 1) / (256 * kCopyAhead));
  for (int i = 0; i < n;) {
    CopyList list;
    list.sources = 0;
    int filled = 0;
    for (; i < n && filled < kCopySlots; ++i) {
      if (list.sources == 0 || order[i].src_slot != list.src[list.sources - 1]) {
        if (list.sources == kCopySources) break;
        list.src[list.sources] = order[i].src_slot;
        list.first[list.sources++] = filled;
      }
      list.dst[filled++] = order[i].dst_slot;
    }
    list.first[list.sources] = filled;
    hipLaunchKernelGGL(copy_slots_kernel, dim3(blocks, (unsigned)list.sources, 2), dim3(256), 0, st, list, a, b);
  }
  return lz::launch_status();
}

// dst[s][c][r] = src[s][r][c]: 32 x 32 tiles through LDS, both sides coalesced, any sizes
template <typename Elem>
__global__ __launch_bounds__(256) void transpose_kernel(const Elem* __restrict__ src, int rows, int cols,
                                                        Elem* __restrict__ dst) {
  __shared__ Elem tile[32][33];
  const size_t base = (size_t)blockIdx.z * rows * cols;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;  // 32 x 8 threads
  for (int i = ty; i < 32; i += 8)
    if (r0 + i < rows && c0 + tx < cols) tile[i][tx] = src[base + (size_t)(r0 + i) * cols + c0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (c0 + i < cols && r0 + tx < rows) dst[base + (size_t)(c0 + i) * rows + r0 + tx] = tile[tx][i];
}

}  // namespace

extern "C" int32_t lz_pack_weights(const void* w, int32_t S, int32_t rows, int32_t cols, int32_t dtype,
                                   void* packed, void* stream) {
  if (S < 0 || rows < 1 || cols < 1 || (dtype != LZ_F32 && dtype != LZ_BF16)) return LZ_ESHAPE;
  if (S > 65535 || (rows + 31) / 32 > 65535) return LZ_ESHAPE;
  if (S == 0) return LZ_OK;
  if (!w || !packed || w == packed) return LZ_EINVAL;
  const dim3 grid((cols + 31) / 32, (rows + 31) / 32, S);
  if (dtype == LZ_F32)
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream, (const float*)w, rows, cols,
                       (float*)packed);
  else
    hipLaunchKernelGGL(transpose_kernel<uint16_t>, grid, dim3(256), 0, (hipStream_t)stream, (const uint16_t*)w,
                       rows, cols, (uint16_t*)packed);
  return lz::launch_status();
}

extern "C" const char* lz_strerror(int32_t code) {
  switch (code) {
    case LZ_OK: return "ok";
    case LZ_EINVAL: return "invalid argument";
    case LZ_ESHAPE: return "shape outside the supported limits";
    case LZ_EWORKSPACE: return "workspace missing, misaligned or too small";
    case LZ_EUNRECOVERABLE: return "an expert has no replica on any surviving rank";
    case LZ_EINFEASIBLE: return "fewer replica slots than experts";
    case LZ_EHIP: return "HIP runtime error";
    default: return "unknown error";
  }
}

extern "C" int32_t lz_version(void) { return 100; }

extern "C" int32_t lz_apply_transfers(const lz_transfer* xfers, int32_t n, const void* w1_old,
                                      const void* w2_old, int32_t S_old, void* w1_new, void* w2_new,
                                      int32_t S_new, const lz_shape* shape, void* stream) {
  if (!lz::shape_ok(shape)) return LZ_ESHAPE;
  if (n < 0 || S_old < 1 || S_new < 1) return LZ_EINVAL;
  if (n == 0) return LZ_OK;
  if (!xfers || !w1_old || !w2_old || !w1_new || !w2_new) return LZ_EINVAL;
  const size_t eb = lz::elem_bytes(shape->dtype);
  const size_t w1_bytes = (size_t)shape->ffn * (shape->act == LZ_SWIGLU ? 2 : 1) * shape->d * eb;
  const size_t w2_bytes = (size_t)shape->d * shape->ffn * eb;
  for (int i = 0; i < n; ++i)
    if (xfers[i].dst_slot < 0 || xfers[i].dst_slot >= S_new || xfers[i].src_slot < 0 ||
        xfers[i].src_slot >= S_old)
      return LZ_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  // One kernel for slots of whole, aligned 16-byte pieces that nothing else in the list reads or writes, on one GPU;
  // else copies in the order of the list.
  const void* const ptrs[4] = {w1_old, w2_old, w1_new, w2_new};
  const size_t sizes[4] = {w1_bytes * S_old, w2_bytes * S_old, w1_bytes * S_new, w2_bytes * S_new};
  // (a grid holds fewer than 2^32 threads in x, one for kCopyAhead pieces each)
  constexpr size_t kMostVecs = ((1ull << 32) - 256) * kCopyAhead;
  bool plain = w1_bytes % 16 == 0 && w2_bytes % 16 == 0 && w1_bytes / 16 <= kMostVecs && w2_bytes / 16 <= kMostVecs;
  for (int p = 0; p < 4; ++p) {
    plain = plain && (uintptr_t)ptrs[p] % 16 == 0;
    for (int q = 2; q < 4; ++q) plain = plain && (p >= q || !overlap(ptrs[p], sizes[p], ptrs[q], sizes[q]));
  }
  plain = plain && on_device_of(st, ptrs, 4);
  std::vector<lz_transfer> order;
  if (plain) try {
      std::vector<bool> written((size_t)S_new, false);
      for (int i = 0; i < n && plain; ++i) {
        plain = !written[xfers[i].dst_slot];
        written[xfers[i].dst_slot] = true;
      }
      order.assign(xfers, xfers + n);
    } catch (const std::bad_alloc&) {
      plain = false;
    }
  if (plain)
    return copy_slots(order, {w1_old, w1_new, (long long)(w1_bytes / 16)}, {w2_old, w2_new, (long long)(w2_bytes / 16)}, st);
  for (int i = 0; i < n; ++i) {
    const size_t d = (size_t)xfers[i].dst_slot, s = (size_t)xfers[i].src_slot;
    if (hipMemcpyAsync((char*)w1_new + d * w1_bytes, (const char*)w1_old + s * w1_bytes, w1_bytes,
                       hipMemcpyDeviceToDevice, st) != hipSuccess)
      return LZ_EHIP;
    if (hipMemcpyAsync((char*)w2_new + d * w2_bytes, (const char*)w2_old + s * w2_bytes, w2_bytes,
                       hipMemcpyDeviceToDevice, st) != hipSuccess)
      return LZ_EHIP;
  }
  return LZ_OK;
}
