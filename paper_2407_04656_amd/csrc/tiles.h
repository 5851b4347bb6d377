// Tables that the grouped GEMMs draw their work from, made on the device from slot_offsets: row tiles for the kernels that index
// by workgroup, lists of units for the persistent one.  Device code and host helpers shared by the translation units, not part of the C ABI.
#pragma once
#include "lz_common.h"
#include <atomic>

namespace lz {

constexpr int kLine = 32;        // ints of a 128-byte line
constexpr int kGroupM = 4;       // row tiles of a work unit (same slot)
constexpr int kGroupN = 8;       // column tiles of a work unit

// Row tiles of a grouped GEMM, slot after slot: what the narrow and the fp32 kernels index by workgroup.
struct TileTable {
  int32_t* header;  // [0] = number of row tiles
  int32_t* slot;
  int32_t* row0;
  int32_t* row_end;
  int capacity;
};
constexpr int kTileHeader = 64;

inline int tile_capacity(long long P, int S, int BM) { return int((P + BM - 1) / BM + S); }

inline size_t tile_table_bytes(long long P, int S, int BM) {
  return lz::align256(sizeof(int32_t) * (kTileHeader + 3 * (size_t)tile_capacity(P, S, BM)));
}

inline TileTable carve_tiles(void* base, long long P, int S, int BM) {
  TileTable t;
  t.capacity = tile_capacity(P, S, BM);
  t.header = (int32_t*)base;
  t.slot = t.header + kTileHeader;
  t.row0 = t.slot + t.capacity;
  t.row_end = t.row0 + t.capacity;
  return t;
}

// Work of one launch of the persistent GEMM: a list of units per XCD.  A unit is up to kGroupM row tiles of one slot x up
// to kGroupN column tiles; its tiles have consecutive tickets, so that a ticket leads to its tile by one look at the
// list, and none is padding.
struct UnitTable {
  int32_t* header;   // [x] = tickets of XCD x's list, [8 + x] = its units, [kTileRows], then, a line each, the counters below
  int32_t* records;  // 8 lists of `cap` records
  int cap, groups;   // room: records of a list, groups of row tiles in all
};
// A record: first ticket, slot, first row, end of the slot's rows, row tiles | column tiles << 8, first column tile, and
// for the weight gradients the rows [k0, k1) that the slot contracts over.
constexpr int kRecord = 8;
// Counters: header[kTicket + x * kLine] = tickets drawn from XCD x's list, x < 8;  x = 8..15: workgroups of XCD
// x - 8 that have finished;  x = 16: XCDs that have finished
constexpr int kTileRows = 16;  // rows of a tile
constexpr int kTicket = 64;
constexpr int kUnitHeader = kTicket + 17 * kLine;

// Room for tiles of the fewest rows that build_tiles_kernel chooses.
constexpr int kLeastTileRows = 64;
inline int unit_groups(long long P, int S) { return int(P / (kLeastTileRows * kGroupM) + S); }
inline int unit_capacity(long long P, int S, int n_tiles) {
  return int(((long long)unit_groups(P, S) * ((n_tiles + kGroupN - 1) / kGroupN) + 7) / 8);
}
inline size_t unit_table_bytes(long long P, int S, int n_tiles) {
  return lz::align256(sizeof(int32_t) * (kUnitHeader + 8 * kRecord * (size_t)unit_capacity(P, S, n_tiles)));
}
inline UnitTable carve_units(void* base, long long P, int S, int n_tiles) {
  return UnitTable{(int32_t*)base, (int32_t*)base + kUnitHeader, unit_capacity(P, S, n_tiles), unit_groups(P, S)};
}

// slot_offsets -> row tiles or units.  Offsets are clipped to [0, P] and made non-decreasing.
//
// Units are dealt to the 8 XCDs' lists in (row group, column group) order, eight at a time, alternate eights in
// opposite directions.  The XCDs thus work on neighbouring
// column groups of the same row group at the same time and share its activation panel in the
// memory-side cache, and a regular pattern of large and small units (a narrow last column
// group, say) does not pile the large ones on the same XCDs; what imbalance is left the GEMM
// kernel evens out by itself.  (Dealing by estimated cost, least-loaded queue first, was
// within 2 % of this and costs a serial pass over the units; dealing the full row groups
// first and the ragged ones last measured 1-5 % slower.)
struct TileSpec {
  int rows_per_tile; // of row tiles; units choose theirs
  int n_tiles;       // column tiles; 0: row tiles for `rows`, else units for `units`
  int virtual_rows;  // > 0: every slot has this many rows (weight gradients)
  bool skip_empty;   // those of slots without rows of the batch have no units: nothing is added to their sums
  int with_tiles, with_rows;  // > 0: n_tiles and virtual_rows of a list that shares this one's launch
  long long P;       // rows of the batch
  TileTable rows;
  UnitTable units;
};
struct TileSpecs {
  TileSpec spec[5];
  int n;
};
inline void add_rows(TileSpecs& specs, int rows, long long P, const TileTable& t) {
  specs.spec[specs.n++] = TileSpec{rows, 0, 0, false, 0, 0, P, t, UnitTable{}};
}
inline void add_units(TileSpecs& specs, int n_tiles, int virtual_rows, long long P, const UnitTable& u, bool skip_empty = false) {
  specs.spec[specs.n++] = TileSpec{0, n_tiles, virtual_rows, skip_empty, 0, 0, P, TileTable{}, u};
}
// The two lists added last share a launch.
inline void share_launch(TileSpecs& specs) {
  TileSpec &a = specs.spec[specs.n - 2], &b = specs.spec[specs.n - 1];
  a.with_tiles = b.n_tiles, a.with_rows = b.virtual_rows;
  b.with_tiles = a.n_tiles, b.with_rows = a.virtual_rows;
}

}  // namespace lz

namespace {

using namespace lz;

typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void clip_slot(const int32_t* slot_offsets, int s, long long P, long long* a,
                                          long long* b) {
  long long lo = slot_offsets[s], hi = slot_offsets[s + 1];
  lo = lo < 0 ? 0 : (lo > P ? P : lo);
  hi = hi < lo ? lo : (hi > P ? P : hi);
  *a = lo;
  *b = hi;
}

// The batch's rows of every slot, clipped, in LDS.
constexpr int kMostSlots = lz::kMaxN * lz::kMaxC;
template <int SLOTS>
struct SlotRows {
  int first[SLOTS], end[SLOTS];
};

constexpr int kTileThreads = 512, kTileWaves = kTileThreads / lz::kWave;  // of a table: a wave per unit list

// The unit lists: a wave each, a record a lane, 64 at a time; s_first: first group of every slot.  A record's slot is found
// by bisection, a read of LDS per factor of two of the slots.  What bounds the tables is one chain of latencies: runs of records a
// lane that step from slot to slot, a division per slot, scans by shuffles, tables of constants in memory and specs that every lane
// reads from the kernel's arguments took 7.4, 8.7 and 20.4 us for a forward's tables of 16, 128 and 1024 slots, where this takes
// 5.6, 6.3 and 11.3 (a launch of nothing: 4).
template <int SLOTS>
__device__ __forceinline__ void deal_units(const SlotRows<SLOTS>& slots, int S, const TileSpec& spec, int rows_per_tile,
                                           const int* s_first, int tid) {
  const int ncg = (spec.n_tiles + kGroupN - 1) / kGroupN;
  const int n_units = s_first[S] * ncg;
  const int x = __builtin_amdgcn_readfirstlane(tid / lz::kWave), lane = tid % lz::kWave;
  static_assert(kTileWaves == 8, "one list per XCD");
  const int full = n_units / 8, count = full + (((full & 1) ? 7 - x : x) < n_units % 8 ? 1 : 0);
  const int cols = spec.n_tiles / ncg, more = spec.n_tiles % ncg;  // column groups of `cols`, the first `more` of one more
  i32x4* const list = (i32x4*)(spec.units.records + (size_t)x * spec.units.cap * kRecord);
  int tickets = 0;  // of the records before r0
  for (int r0 = 0; r0 < count; r0 += lz::kWave) {
    const bool in = r0 + lane < count;
    const int r = in ? r0 + lane : count - 1;
    const int u = r * 8 + ((r & 1) ? 7 - x : x), g = u / ncg, c = u - g * ncg;
    int s = 0;  // the last slot that starts at or before the group
    for (int hi = S - 1; s < hi;) {
      const int mid = (s + hi + 1) >> 1;
      if (s_first[mid] <= g) s = mid;
      else hi = mid - 1;
    }
    const int k0 = slots.first[s], k1 = slots.end[s];
    const int a = spec.virtual_rows > 0 ? s * spec.virtual_rows : k0;
    const int b = spec.virtual_rows > 0 ? a + spec.virtual_rows : k1;
    const int row0 = a + (g - s_first[s]) * (kGroupM * rows_per_tile);
    int nr = 1;  // of at most kGroupM row tiles
#pragma unroll
    for (int i = 1; i < kGroupM; ++i) nr += b - row0 > i * rows_per_tile ? 1 : 0;
    const int nc = cols + (c < more ? 1 : 0);
    const int mine = in ? nr * nc : 0;
    const int incl = lz::wave_scan(mine, [](int x, int y) { return x + y; });
    if (in) {
      list[2 * r] = i32x4{tickets + incl - mine, s, row0, b};
      list[2 * r + 1] = i32x4{nr | nc << 8, c * cols + (c < more ? c : more), k0, k1};
    }
    tickets += __builtin_amdgcn_readlane(incl, lz::kWave - 1);
  }
  if (lane == 0) {
    spec.units.header[x] = tickets;
    spec.units.header[8 + x] = count;
  }
  if (tid == 0) spec.units.header[kTileRows] = rows_per_tile;
  if (tid < 17) spec.units.header[kTicket + tid * kLine] = 0;
}

// Rows of the wide kernel's tiles, 256, 192, 128 or 64: those with which the launch ends first.  A launch of N tiles takes
// ceil(N / workgroups) rounds, and a tile of fewer rows costs more than its share (it streams the same columns of W):
// 100, 82, 65, 50 measured on K loops of 22 to 224 steps.  Where rounds are many 256 rows are the cheapest; with
// 2.2 rounds of them (the down projection of 40960 tokens over 60 slots, 3072 x 768) 192 rows make 2.9 shorter ones:
// that training step 1743 -> 1706 us, a forward of 3001 tokens (12 slots, 1000 x 2664, SwiGLU) 197 -> 186.
// A row's result does not depend on the tile it is in.
// Two lists that share a launch (with_tiles) get the rows that suit their sum: what one's last round leaves idle the other fills.  Backward
// passes of some 550 drawn layers of up to 128 rows a slot, below 1, 4 and 16 rounds of both weight gradients, with rows that suit each
// list alone 0.93, 0.95 and 0.97 of two launches' time, with these 0.89, 0.93 and 0.96, none above 1.005.  Accumulating passes of one K step and
// a round or two: 9 of 300 are above 1.01 (28 before): the costs are those of longer loops.  Worst: 97 tokens, top-2, 11 slots,
// 768 x 768, 53 -> 62 us.
__device__ __forceinline__ int tile_cost(int n64) { return int(0x6452413200ull >> (8 * n64)) & 255; }  // by rows in 64s
// Of a table's 512 threads each wave leaves one sum in s_sum: tiles (wave w < 4) or cost of tiles of 64 (w % 4 + 1) rows.
// rows_of(slot, virtual rows of the list)
template <typename RowsOf>
__device__ __forceinline__ void sum_tile_costs(const TileSpec& spec, int S, int tid, unsigned* s_sum, RowsOf rows_of) {
  const int lane = tid % lz::kWave, wave = __builtin_amdgcn_readfirstlane(tid / lz::kWave), n64 = wave % 4 + 1;
  static_assert(kTileWaves == 8, "a wave per sum");
  auto sum_of = [&](int virtual_rows) {
    unsigned sum = 0;
    for (int s = lane; s < S; s += lz::kWave) {
      const int all64 = (int)(((unsigned)rows_of(s, virtual_rows) + 63) / 64), full = n64 == 3 ? all64 / 3 : all64 >> (n64 / 2),
                tail = all64 - full * n64;
      sum += wave < 4 ? full + (tail > 0 ? 1 : 0) : full * tile_cost(n64) + tile_cost(tail);
    }
    return sum;
  };
  unsigned sum = spec.n_tiles * sum_of(spec.virtual_rows);
  if (spec.with_tiles > 0) sum += spec.with_tiles * sum_of(spec.with_rows);
  sum = lz::wave_scan(sum, [](int x, int y) { return (int)((unsigned)x + (unsigned)y); });
  if (lane == lz::kWave - 1) s_sum[wave] = sum;
}
__device__ __forceinline__ bool many_rounds(int S, const TileSpec& spec, int workgroups) {
  const float rows = spec.virtual_rows > 0 ? (float)S * (float)spec.virtual_rows : (float)spec.P;
  const float tiles = rows / 256.f * (float)spec.n_tiles + (float)S * (float)spec.with_rows / 256.f * (float)spec.with_tiles;
  return tiles > 16.f * (float)workgroups;
}
__device__ __forceinline__ int choose_tile_rows(int workgroups, const unsigned* s_sum) {
  const float one_round = (float)workgroups;
  int best = 256;
  float best_time = 0.f;
#pragma unroll
  for (int c = 3; c >= 0; --c) {
    const float n = (float)s_sum[c], rounds = ceilf(n / one_round);
    const float time = n > 0.f ? rounds * (float)s_sum[4 + c] / n : 0.f;
    if (c == 3 || time < 0.95f * best_time) {
      best = 64 * (c + 1);
      best_time = time;
    }
  }
  return best;
}

template <int SLOTS>
struct TableScratch {
  int first[SLOTS + 1];  // row tiles, or groups of them, of the slots before
  int wave[kTileWaves];
  unsigned sum[kTileWaves];
};

// One table, by 512 threads of a workgroup that has filled `slots`; other threads of it may build another at the same time: the
// barriers are the workgroup's.  idle: follows the others' steps up to the last barrier and writes no table.
template <int SLOTS>
__device__ __forceinline__ void build_table(const TileSpec& spec, bool idle, const SlotRows<SLOTS>& slots, int S,
                                            TableScratch<SLOTS>& scratch, int tid, int workgroups) {
  const TileTable t = spec.rows;
  const bool units = spec.n_tiles > 0;
  const int capacity = units ? spec.units.groups : t.capacity;
  const int lane = tid % lz::kWave, wave = __builtin_amdgcn_readfirstlane(tid / lz::kWave);
  // Without skip_empty the sums of empty slots are read and written back: two micro-batches of 50 rows on 90 slots,
  // 768 x 1792, 1423 us a step, 927 with it.
  auto rows_of = [&](int s, int virtual_rows) {
    const int own = slots.end[s] - slots.first[s];
    return virtual_rows > 0 && (own > 0 || !spec.skip_empty) ? virtual_rows : own;
  };
  const bool choose = units && !many_rounds(S, spec, workgroups);
  if (choose) sum_tile_costs(spec, S, tid, scratch.sum, rows_of);
  __syncthreads();
  const int rows = !units ? spec.rows_per_tile : choose ? choose_tile_rows(workgroups, scratch.sum) : 256;
  const unsigned group_rows = units ? rows * kGroupM : rows;
  // tile or group count of every slot and its exclusive sum: each thread owns a run of consecutive slots.  The sums
  // end at the table's capacity, which the slots of ascending offsets stay within: offsets that fall again make
  // slots overlap, any number of tiles in all.
  auto add = [&](int x, int y) { return x + y < capacity ? x + y : capacity; };  // both at most capacity < 2^26
  const int per = (S + kTileThreads - 1) / kTileThreads, first = tid * per;
  int mine = 0;
  for (int s = first; s < first + per && s < S; ++s) {
    const int tiles = int(((unsigned)rows_of(s, spec.virtual_rows) + group_rows - 1) / group_rows);
    scratch.first[s] = mine;
    mine = add(mine, tiles < capacity ? tiles : capacity);
  }
  const int incl = lz::wave_scan(mine, add);
  if (lane == lz::kWave - 1) scratch.wave[wave] = incl;
  const int before = __shfl_up(incl, 1);
  __syncthreads();
  int base = lane == 0 ? 0 : before;
  for (int w = 0; w < wave; ++w) base = add(base, scratch.wave[w]);
  for (int s = first; s < first + per && s < S; ++s) scratch.first[s] = add(scratch.first[s], base);
  if (tid == kTileThreads - 1) scratch.first[S] = add(base, mine);
  __syncthreads();
  if (idle) return;
  if (units) {
    deal_units(slots, S, spec, rows, scratch.first, tid);
    return;
  }
  if (tid == 0) t.header[0] = scratch.first[S];
  // Few entries: a thread each, its slot found by bisection.  More: a thread writes the entries of its slot, 45 ns
  // each, and where a wave holds a few long slots (few slots share a large batch) it writes what is past kOwn of
  // those together, slot after slot: 130 ns a slot and 64 entries a step.
  // 32-row tiles of 10^6 rows in 1, 4, 32, 128 slots: 1390, 867, 136, 64 us by the threads alone, 28, 29, 31, 31 us so.
  constexpr int kOwn = 64;
  auto entry = [&](int i, int s, int first_i) {
    t.slot[i] = s;
    t.row0[i] = slots.first[s] + (i - first_i) * rows;
    t.row_end[i] = slots.end[s];
  };
  const bool few = scratch.first[S] <= 1024;
  for (int i = tid; few && i < scratch.first[S]; i += kTileThreads) {
    int s = 0;
    for (int hi = S - 1; s < hi;) {  // the last slot that starts at or before i
      const int mid = (s + hi + 1) >> 1;
      if (scratch.first[mid] <= i) s = mid;
      else hi = mid - 1;
    }
    entry(i, s, scratch.first[s]);
  }
  for (int s0 = wave * lz::kWave; !few && s0 < S; s0 += kTileThreads) {  // the same trips in every lane
    const int s = s0 + lane, from = s < S ? scratch.first[s] : 0, to = s < S ? scratch.first[s + 1] : 0;
    unsigned long long many = __ballot(to - from > kOwn);
    if (!__any(to - from > kOwn + 4 * __popcll(many))) many = 0;
    const int own_end = many && to - from > kOwn ? from + kOwn : to;
    for (int i = from; i < own_end; ++i) entry(i, s, from);
    for (; many; many &= many - 1) {
      const int l = __ffsll((long long)many) - 1;
      const int f = __shfl(from, l), end = __shfl(to, l);
      for (int i = f + kOwn + lane; i < end; i += lz::kWave) entry(i, s0 + l, f);
    }
  }
}

// Tables of units first, two a workgroup (side by side, 512 threads each), then those of row tiles, one a workgroup.
__global__ __launch_bounds__(2 * kTileThreads) void build_tiles_kernel(const int32_t* __restrict__ slot_offsets, int S,
                                                          TileSpecs specs, int n_units, int workgroups) {
  __shared__ SlotRows<kMostSlots> slots;
  __shared__ TableScratch<kMostSlots> scratch[2];
  // scalar: so that a table's spec is read by scalar loads, not by every lane from the kernel's arguments
  const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / kTileThreads), tid = threadIdx.x % kTileThreads;
  const int unit_groups = (n_units + 1) / 2, b = blockIdx.x;
  const int table = b < unit_groups ? 2 * b + half : b - unit_groups + n_units;
  const bool idle = b < unit_groups ? table >= n_units : half > 0;
  const TileSpec& spec = specs.spec[idle ? (b < unit_groups ? 2 * b : table) : table];
  for (int s = threadIdx.x; s < S; s += blockDim.x) {
    long long a, b;
    clip_slot(slot_offsets, s, spec.P, &a, &b);  // the tables of a launch have one P
    slots.first[s] = int(a);
    slots.end[s] = int(b);
  }
  __syncthreads();
  build_table(spec, idle, slots, S, scratch[half], tid, workgroups);
}

constexpr int kMaxDevices = 64;

// CUs of the current device in whole multiples of the 8 XCDs, read once per device; 0 on an error
inline int device_cus() {
  static std::atomic<int> cus_of_device[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  int cus = cus_of_device[dev].load(std::memory_order_acquire);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cus = cus >= 8 ? cus / 8 * 8 : 8;
    cus_of_device[dev].store(cus, std::memory_order_release);
  }
  return cus;
}

inline int32_t launch_build_tiles(const int32_t* slot_offsets, int S, const TileSpecs& specs, hipStream_t st) {
  const int workgroups = device_cus();  // of the wide kernel, below
  if (workgroups == 0) return LZ_EHIP;
  int n_units = 0;
  while (n_units < specs.n && specs.spec[n_units].n_tiles > 0) ++n_units;
  hipLaunchKernelGGL(build_tiles_kernel, dim3((n_units + 1) / 2 + specs.n - n_units), dim3(n_units > 1 ? 2 * kTileThreads : kTileThreads),
                     0, st, slot_offsets, S, specs, n_units, workgroups);
  return lz::launch_status();
}

}  // namespace
