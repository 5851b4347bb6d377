// The flexible token dispatcher (Algorithm 1, Sec. 4.2) for all source ranks at once.
//
// Three kernels on one stream, no host synchronisation, no order-dependent atomics:
//   count    each wave owns a chunk of <= 128 consecutive pairs of ONE source rank and
//            histograms their expert ids with LDS atomics (counts commute); a workgroup's chunks are neighbours of
//            one rank, so that tables of (expert, chunk) are written and read in runs
//   schedule one workgroup per expert scans the chunk counts into per-(expert, rank) list
//            positions, evaluates the algorithm's counts in exact integers, in LDS, and cuts the expert's
//            receive lists over its slots
//   place    every workgroup scans the slot sizes; each wave revisits its chunk: a pair's position in its (expert, source rank)
//            list is chunk base + ordered rank inside the chunk (wave ballots, one per
//            bit of an expert index), which fixes destination rank, slot and row
// Up to 8192 pairs the expert's workgroup counts its pairs itself (direct_counts), and small batches take all of it in one
// workgroup (plan_small_kernel).
// Each is a chain of dependent lookups over little data, and a launch of nothing takes 2.7 us: latency bound.  us of a plan, with a
// launch of one workgroup for the slots, scans by shuffles, tables of (chunk, expert) and every lookup in memory, and now (chunks
// a workgroup: 4, 8, 16): 16384 pairs, 8 experts, 8 ranks of 2 slots 18.7, now 13.3, 13.5, 14.4; 98304 pairs, 64 experts, 16 ranks of
// 8 21.8, now 15.7, 15.4, 16.4; 262144 pairs, 256 experts, 32 ranks of 10 41.7, now 31.7, 28.3, 28.1.
#include <mutex>

#include "layer.h"
#include "route.h"

namespace {

constexpr int kChunk = 128;          // pairs per wave-chunk
constexpr int kGroup = 8;            // chunks of a workgroup, a wave each, all of one source rank
constexpr int kSchedThreads = 1024;

struct PlanTables {
  // per chunk
  int nch;             // room for chunks
  int32_t* chunkcnt;   // [E, nch]
  int32_t* chunkbase;  // [E, nch]  position of the chunk's first pair of e in its (e, rank) list
  int32_t* chunkflag;  // [nch]
  // per (expert, rank)
  int4* lists;         // [E, N]  pairs that rank j receives for e, its replicas of e, the first of those in its sorted slots
  int32_t* estatus;    // [E]     status bits raised while scheduling expert e
  // per (expert, src, dst)
  int32_t* cumDst;     // [N src, E, N+1] prefix of D over dst
  int32_t* preSrc;     // [E, N, N]   prefix of D over src
  // per slot
  int32_t* slot_sorted;  // [S] rank j's slots ordered by (expert, slot id)
  size_t total_bytes;
};

inline int max_chunks(long long P, int N) { return int((P + kChunk - 1) / kChunk) + N; }
inline int max_groups(long long P, int N) { return int((P + kChunk * kGroup - 1) / (kChunk * kGroup)) + N; }

PlanTables carve(void* ws, const lz_shape* s) {
  PlanTables t{};
  const size_t E = s->E, N = s->N, S = size_t(s->N) * s->c;
  const size_t nch = max_chunks((long long)s->T * s->k, s->N);
  char* base = (char*)ws;
  size_t off = 0;
  auto take = [&](size_t n_ints) {
    int32_t* p = (int32_t*)(base + off);
    off += lz::align256(n_ints * sizeof(int32_t));
    return p;
  };
  t.nch = (int)nch;
  t.chunkcnt = take(nch * E);
  t.chunkbase = take(nch * E);
  t.chunkflag = take(nch);
  t.lists = (int4*)take(E * N);
  for (int i = 1; i < 4; ++i) take(E * N);  // ... of four ints each: what is taken follows on, with room to spare by its rounding up
  t.estatus = take(E);
  take(E * N * N);  // room that no kernel uses: which shapes fit LZ_PLAN_NOALLOC_SCRATCH_BYTES is part of the interface
  t.cumDst = take(E * N * (N + 1));
  t.preSrc = take(E * N * N);
  t.slot_sorted = take(S);
  t.total_bytes = off;
  return t;
}

__device__ __forceinline__ int scan_sum(int v) {
  return lz::wave_scan(v, [](int x, int y) { return x + y; });
}
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, lz::kWave - 1); }
// of the lane below, 0 in the first
__device__ __forceinline__ int from_lane_below(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, false);  // wave_shr 1
#else
  return v;
#endif
}

// Sanitised batch split and the chunk table derived from it, rebuilt by every workgroup: called by its first
// wave, lane i for the end of rank i (N <= 64).  An entry counts for at least its predecessors and at most T,
// the last for T.  Returns true (in every lane) if rank_tok_off had to be repaired.
// s_off: first tokens, s_cf: first chunks, s_gf (if any): first workgroups of the ranks.
__device__ bool build_split(const int32_t* __restrict__ rank_tok_off, int T, int N, int k,
                            int* s_off, int* s_cf, int* s_gf = nullptr) {
  const int lane = threadIdx.x;  // < 64
  const int raw = lane < N ? rank_tok_off[lane + 1] : T;
  const int own = lane < N - 1 ? (raw < 0 ? 0 : raw > T ? T : raw) : T;
  const int v = lz::wave_scan(own, [](int x, int y) { return x > y ? x : y; });
  const int prev = from_lane_below(v);
  const bool bad = lane < N - 1 ? raw < 0 || raw > T || own < prev : lane == N - 1 && raw != T;
  const int own_chunks = lane < N ? int(((long long)(v - prev) * k + kChunk - 1) / kChunk) : 0;
  const int chunks = scan_sum(own_chunks);
  if (lane == 0) s_off[0] = s_cf[0] = 0;
  if (lane < N) {
    s_off[lane + 1] = v;
    s_cf[lane + 1] = chunks;
  }
  if (s_gf != nullptr) {
    const int groups = scan_sum((own_chunks + kGroup - 1) / kGroup);
    if (lane == 0) s_gf[0] = 0;
    if (lane < N) s_gf[lane + 1] = groups;
  }
  return __any(bad) || rank_tok_off[0] != 0;
}

// chunk b -> its source rank (or -1) and pair range
__device__ __forceinline__ int chunk_range(int b, int N, int k, const int* s_off, const int* s_cf,
                                           long long* p0, long long* p1) {
  if (b >= s_cf[N]) return -1;
  int i = 0;  // the first rank whose chunks end past b
  for (int hi = N - 1; i < hi;) {
    const int mid = (i + hi) >> 1;
    if (s_cf[mid + 1] <= b) i = mid + 1;
    else hi = mid;
  }
  const long long begin = (long long)s_off[i] * k + (long long)(b - s_cf[i]) * kChunk;
  const long long end = (long long)s_off[i + 1] * k;
  *p0 = begin;
  *p1 = begin + kChunk < end ? begin + kChunk : end;
  return i;
}

// This workgroup's source rank, N if it has no chunks.
__device__ __forceinline__ int group_rank(const int* s_gf, int N) {
  const int lane = threadIdx.x % lz::kWave;
  return __popcll(__ballot(lane < N && s_gf[lane + 1] <= (int)blockIdx.x));
}

// The chunk of wave w of this workgroup, whose rank is i: index (or -1) and pair range.
__device__ __forceinline__ int group_chunk(int i, int w, int k, const int* s_off, const int* s_cf, const int* s_gf, long long* p0,
                                           long long* p1) {
  const int in_rank = ((int)blockIdx.x - s_gf[i]) * kGroup + w, b = s_cf[i] + in_rank;
  if (b >= s_cf[i + 1]) return -1;
  const long long begin = (long long)s_off[i] * k + (long long)in_rank * kChunk, end = (long long)s_off[i + 1] * k;
  *p0 = begin;
  *p1 = begin + kChunk < end ? begin + kChunk : end;
  return b;
}

constexpr int kRowE = lz::kMaxE + 1;  // of LDS rows of experts, one a wave: a column's entries lie in different banks

__global__ __launch_bounds__(kGroup * lz::kWave) void count_kernel(const int32_t* __restrict__ ids,
                                                    const int32_t* __restrict__ rank_tok_off, int T,
                                                    int E, int N, int k, PlanTables t,
                                                    int32_t* __restrict__ row_to_pair) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1], s_gf[lz::kMaxN + 1];
  __shared__ int s_cnt[kGroup * kRowE];
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave;
  int* const own = s_cnt + w * kRowE;
  if (tid < lz::kWave) build_split(rank_tok_off, T, N, k, s_off, s_cf, s_gf);
  for (int e = lane; e < E; e += lz::kWave) own[e] = 0;
  __syncthreads();
  const int i = group_rank(s_gf, N);
  if (i == N) return;
  long long p0 = 0, p1 = 0;
  const int b = group_chunk(i, w, k, s_off, s_cf, s_gf, &p0, &p1);
  int flag = 0;
  for (long long p = p0 + lane; p < p1; p += lz::kWave) {
    const int e = ids[p];
    if (e >= 0 && e < E) atomicAdd(&own[e], 1);
    else flag = LZ_PLAN_BAD_EXPERT_ID;
    row_to_pair[p] = -1;  // rows and pairs share the index range [0, P)
  }
  flag = __any(flag) ? LZ_PLAN_BAD_EXPERT_ID : 0;
  if (b >= 0 && lane == 0) t.chunkflag[b] = flag;
  __syncthreads();
  const int b0 = s_cf[i] + ((int)blockIdx.x - s_gf[i]) * kGroup, chunks = s_cf[i + 1] - b0 < kGroup ? s_cf[i + 1] - b0 : kGroup;
  for (int x = tid; x < E * kGroup; x += kGroup * lz::kWave) {
    const int e = x / kGroup, u = x % kGroup;
    if (u < chunks) t.chunkcnt[(size_t)e * t.nch + b0 + u] = s_cnt[u * kRowE + e];
  }
}

// a / b for a >= 0, b > 0; the 64-bit quotient costs several times the 32-bit one
__device__ __forceinline__ long long div_floor(long long a, long long b) {
  if (((unsigned long long)(a | b) >> 32) == 0) return (uint32_t)a / (uint32_t)b;
  return a / b;
}

// Algorithm 1's first lines for one expert, by a whole wave with lane = rank (R, T of the rank, 0 past the last):
// r_e, t_e, then this rank's capacity split into what it keeps, its residual and its overflow.
struct Shares {
  int keep, overflow, residual_upto;  // residual_upto: residual capacity of the ranks up to this one
  bool uncovered;                     // pairs but no replica (the same in every lane)
};
__device__ __forceinline__ Shares shares_of(int R, int T) {
  const long long hi = scan_sum(R), re = last_lane((int)hi);  // at most N c slots and P pairs
  const long long te = last_lane(scan_sum(T));
  const long long lo = hi - R;
  const int cap = re > 0 ? int(div_floor(hi * te, re) - div_floor(lo * te, re)) : 0;
  Shares s;
  s.keep = cap < T ? cap : T;
  s.overflow = T - s.keep;
  s.residual_upto = scan_sum(cap - s.keep);
  s.uncovered = te > 0 && re == 0;
  return s;
}

// D[e, i, j]: local share on the diagonal, overflow spread by the residual capacity of the others.  With
// q(j) = floor(o cumP(j) / tot), cumP(j) that capacity before j without i's own, the shares are q(j + 1) - q(j)
// and their prefix is q(j), plus the local share once j has passed i.  L, O: of the ranks; Pre: residual prefix.
__device__ __forceinline__ int assignment(int i, int j, int N, const int* L, const int* Pre, const int* O, int* cum) {
  const long long o = O[i], tot = Pre[N];
  const bool spread = o > 0 && tot > 0;
  const int own = Pre[i + 1] - Pre[i], before = Pre[j] - (j > i ? own : 0);
  const int q = spread ? int(div_floor(o * before, tot)) : 0;
  const int next = spread && j != i ? int(div_floor(o * (before + Pre[j + 1] - Pre[j]), tot)) : 0;
  *cum = q + (j > i ? L[i] : 0);
  return j == i ? L[i] : next - q;
}

// Algorithm 1 for one expert per workgroup.  Everything an expert needs (N counts, N x N
// assignments) lives in LDS between the phases, so the chain of dependent steps costs barriers,
// not global-memory round trips; the tables that place_kernel reads are written out once.
// What bounds it is the latency of those steps: a wave per source rank for the chunk scans (up to 16 waves),
// a thread per (source, destination) for the assignments, whose prefix over destinations has a closed form,
// a wave per destination for the prefix over sources and the slots.
// DIRECT: the expert's pairs of every chunk are counted here, by ballots, where count_kernel would be a launch before.
constexpr int kDirectPairs = 8192, kDirectChunks = kDirectPairs / kChunk + lz::kMaxN;

template <bool DIRECT>
__global__ __launch_bounds__(1024) void schedule_expert_kernel(
    const int32_t* __restrict__ ids, const int32_t* __restrict__ rank_tok_off, const int32_t* __restrict__ slot_expert, int T,
    int E, int N, int c, int k, PlanTables t, int32_t* __restrict__ slot_counts, int32_t* __restrict__ row_to_pair,
    int32_t* __restrict__ Tej_opt, int32_t* __restrict__ D_opt) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_T[lz::kMaxN], s_L[lz::kMaxN], s_P[lz::kMaxN + 1], s_O[lz::kMaxN];
  __shared__ int s_before[lz::kMaxN];                 // slots of rank j with a lower expert
  __shared__ unsigned long long s_mine[lz::kMaxN];    // slots of rank j with this one, a bit each (c <= 64)
  __shared__ int s_D[lz::kMaxN * (lz::kMaxN + 1)];
  __shared__ int s_count[DIRECT ? kDirectChunks : 1];
  __shared__ int s_status;
  const int e = blockIdx.x;
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = __builtin_amdgcn_readfirstlane(tid / lz::kWave), n_waves = blockDim.x / lz::kWave;
  const int pitch = N | 1;  // of s_D: a column's entries lie in different banks
  if (tid == 0) s_status = 0;
  if (w == 0) build_split(rank_tok_off, T, N, k, s_off, s_cf);
  int flag = 0;
  for (int j = w; j < N; j += n_waves) {
    const int se = lane < c ? slot_expert[j * c + lane] : -1;
    const unsigned long long own = __ballot(lane < c && se == e), lower = __ballot(lane < c && se >= 0 && se < e);
    if (lane == 0) {
      s_mine[j] = own;
      s_before[j] = __popcll(lower);
    }
    if (e == 0 && lane < c && (se < 0 || se >= E)) {  // a slot of no expert
      slot_counts[j * c + lane] = 0;
      flag = LZ_PLAN_BAD_EXPERT_ID;
    }
  }
  __syncthreads();

  if constexpr (DIRECT) {
    const int P = T * k;
    // lane m looks up the wave's m-th chunk, n_waves apart
    const int chunks = s_cf[N], own = chunks > w ? (chunks - w + n_waves - 1) / n_waves : 0;  // at most 64
    long long p0 = 0, p1 = 0;
    chunk_range(w + n_waves * lane, N, k, s_off, s_cf, &p0, &p1);
    constexpr int kAhead = 4;  // chunks whose ids are loaded before the first is counted
    for (int m0 = 0; m0 < own; m0 += kAhead) {
      int id[kAhead][2];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int m = m0 + u < own ? m0 + u : own - 1;
        const int from = __builtin_amdgcn_readlane((int)p0, m), to = m0 + u < own ? __builtin_amdgcn_readlane((int)p1, m) : 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int p = from + h * lz::kWave + lane;
          id[u][h] = p < to ? ids[p] : E;
          // (E: none; an id that is E is caught here)
          if (p < to && (id[u][h] < 0 || id[u][h] >= E)) flag = LZ_PLAN_BAD_EXPERT_ID;
        }
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int n = __popcll(__ballot(id[u][0] == e)) + __popcll(__ballot(id[u][1] == e));
        if (lane == 0 && m0 + u < own) s_count[w + n_waves * (m0 + u)] = n;
      }
    }
    for (int p = e * blockDim.x + tid; p < P; p += gridDim.x * blockDim.x) row_to_pair[p] = -1;  // rows and pairs share [0, P)
    __syncthreads();
  }
  if (flag) atomicOr(&s_status, flag);

  // ---- per source rank j (one wave each): positions of the chunks in the (e, j) list, T[e,j]
  for (int j = w; j < N; j += n_waves) {
    const int b_end = s_cf[j + 1];
    auto count_of = [&](int b) {
      if constexpr (DIRECT) return b < b_end ? s_count[b] : 0;
      else return b < b_end ? t.chunkcnt[(size_t)e * t.nch + b] : 0;
    };
    int running = 0, b = s_cf[j] + lane;
    int v = count_of(b);
    for (int b0 = s_cf[j]; b0 < b_end; b0 += lz::kWave) {
      const int v_next = count_of(b + lz::kWave);
      const int incl = scan_sum(v);
      if (b < b_end) t.chunkbase[(size_t)e * t.nch + b] = running + incl - v;
      running += last_lane(incl);
      b += lz::kWave;
      v = v_next;
    }
    if (lane == 0) {
      s_T[j] = running;
      if (Tej_opt) Tej_opt[e * N + j] = running;
    }
  }
  __syncthreads();

  // ---- one wave, lane = rank: capacity, local share, residual and its prefix over ranks, overflow
  if (w == 0) {
    const Shares sh = shares_of(lane < N ? __popcll(s_mine[lane]) : 0, lane < N ? s_T[lane] : 0);
    if (lane < N) {
      s_L[lane] = sh.keep;
      s_P[lane + 1] = sh.residual_upto;
      s_O[lane] = sh.overflow;
    }
    if (lane == 0) {
      s_P[0] = 0;
      t.estatus[e] = s_status | (sh.uncovered ? LZ_PLAN_UNCOVERED_EXPERT : 0);
    }
  }
  __syncthreads();

  // ---- D[e, i, j] and its prefix over destinations
  for (int ij = tid; ij < N * N; ij += blockDim.x) {
    const int i = ij / N, j = ij % N;
    int cum;
    const int dval = assignment(i, j, N, s_L, s_P, s_O, &cum);
    s_D[i * pitch + j] = dval;
    if (D_opt) D_opt[(size_t)(e * N + i) * N + j] = dval;
    int32_t* const row = t.cumDst + (size_t)(i * E + e) * (N + 1);
    row[j] = cum;
    if (j == N - 1) row[N] = cum + dval;
  }
  __syncthreads();

  // ---- per destination rank j (one wave each): prefix over source ranks, the received pairs, and their balanced
  // cut over the rank's slots of e
  for (int j = w; j < N; j += n_waves) {
    const int v = lane < N ? s_D[lane * pitch + j] : 0;
    const int incl = scan_sum(v), n = last_lane(incl);
    if (lane < N) t.preSrc[(size_t)(e * N + lane) * N + j] = incl - v;
    const unsigned long long own = s_mine[j];
    const int reps = __popcll(own), before = s_before[j];
    if (own >> lane & 1) {
      const long long m = __popcll(own & ((1ull << lane) - 1ull));
      slot_counts[j * c + lane] = int(div_floor((m + 1) * n, reps) - div_floor(m * n, reps));
      t.slot_sorted[j * c + before + (int)m] = j * c + lane;
    }
    if (lane == 0) t.lists[e * N + j] = int4{n, reps, before, 0};
  }
}

// The tables of place_chunk for one source rank: prefix of D over destinations (an expert's row every cum_stride), over
// sources, {received, replicas, first slot} of an (expert, rank) list, a rank's slots in order, first rows of slots.
template <typename Cum, typename Pre, typename List, typename Sorted, typename First>
struct PlaceTables {
  Cum cum;
  Pre pre;
  List list;
  Sorted sorted;
  First first;
};
template <typename Cum, typename Pre, typename List, typename Sorted, typename First>
__device__ PlaceTables(Cum, Pre, List, Sorted, First) -> PlaceTables<Cum, Pre, List, Sorted, First>;

// One wave places the pairs [p0, p1) of a chunk; run[e]: position of its first pair of e in the
// (e, source rank) list, advanced here.
template <typename Tables>
__device__ __forceinline__ void place_chunk(const int32_t* __restrict__ ids, long long p0, long long p1, int* run, int E,
                                            int N, int c, long long P, const Tables& t, int32_t* __restrict__ pair_to_row,
                                            int32_t* __restrict__ row_to_pair) {
  const int lane = threadIdx.x % lz::kWave;
  const unsigned long long lower = (1ull << lane) - 1ull;
  const int e_bits = 32 - __clz(E - 1 | 1);
  constexpr int kPairs = kChunk / lz::kWave;  // of this lane: their lookups below run side by side

  // ordered rank of each pair among the chunk's pairs of the same expert.  The lanes that hold the same expert
  // are found bit by bit, one ballot per bit of an expert index.
  int ex[kPairs], q[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const long long p = p0 + u * lz::kWave + lane;
    const int id = p < p1 ? ids[p] : -1;
    ex[u] = id >= 0 && id < E ? id : -1;
  }
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    unsigned long long same = __ballot(ex[u] >= 0);
    for (int bit = 0; bit < e_bits; ++bit) {
      const unsigned long long set = __ballot((ex[u] >> bit) & 1);
      same &= (ex[u] >> bit) & 1 ? set : ~set;
    }
    q[u] = -1;
    if (ex[u] >= 0) q[u] = run[ex[u]] + __popcll(same & lower);
    __builtin_amdgcn_wave_barrier();
    if (ex[u] >= 0 && (same & lower) == 0) run[ex[u]] += __popcll(same);  // one lane per expert
    __builtin_amdgcn_wave_barrier();
  }
  int row[kPairs], dst[kPairs];
  bool ok[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    row[u] = -1;
    dst[u] = 0;
    ok[u] = ex[u] >= 0 && q[u] < t.cum(ex[u] < 0 ? 0 : ex[u], N);
  }
  // destination rank: the last j with cum[j] <= q (cum[0] = 0)
  int step = 1;
  while (step * 2 < N) step *= 2;
  for (; step > 0; step >>= 1) {
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const int j = dst[u] + step;
      if (j < N && t.cum(ex[u] < 0 ? 0 : ex[u], j) <= q[u]) dst[u] = j;
    }
  }
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    if (ok[u]) {
      const int j = dst[u];
      const int3 list = t.list(ex[u], j);
      const long long pos = t.pre(ex[u], j) + (q[u] - t.cum(ex[u], j));
      const long long n = list.x, reps = list.y;
      if (n > 0 && reps > 0) {
        // slot m of the (e, j) list holds positions [floor(m*n/reps), floor((m+1)*n/reps))
        long long m = div_floor((pos + 1) * reps - 1, n);
        m = m < reps ? m : reps - 1;
        const int s = t.sorted(j * c + list.z + (int)m);
        const long long r = t.first(s) + pos - div_floor(m * n, reps);
        if (r >= 0 && r < P) row[u] = (int)r;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const long long p = p0 + u * lz::kWave + lane;
    if (p < p1) pair_to_row[p] = row[u];
    if (row[u] >= 0) row_to_pair[row[u]] = (int)p;
  }
}

// First rows of the slots from their sizes, by a whole workgroup (each thread a run of consecutive slots); returns their sum
// in the last thread.  s_first may be written when the workgroup has passed its first barrier.
// end_of(slot, end of its rows): to be kept by the caller.
template <typename EndOf>
__device__ __forceinline__ int scan_slots(const int32_t* __restrict__ slot_counts, int S, int* s_first, int* s_wave, EndOf end_of) {
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave;
  const int per = (S + (int)blockDim.x - 1) / (int)blockDim.x, first = tid * per;
  int own = 0;
  for (int s = first; s < first + per && s < S; ++s) own += slot_counts[s];
  const int incl = scan_sum(own);
  if (lane == lz::kWave - 1) s_wave[w] = incl;
  __syncthreads();
  int running = incl - own;
  for (int v = 0; v < w; ++v) running += s_wave[v];
  const int end = running + own;
  for (int s = first; s < first + per && s < S; ++s) {
    s_first[s] = running;
    running += slot_counts[s];
    end_of(s, running);
  }
  return end;
}

// The first rows of all slots are scanned by every workgroup, which is cheaper than a launch of one workgroup for them (5 us
// of a plan).  What bounds it is latency, and with many experts the lookups of single entries: what a workgroup's chunks need of the
// tables is fetched at the start, all at once, but for the entries of the pairs' lists; the prefix over destinations of the
// workgroup's rank is searched in LDS where it fits.
// What fits beside the other tables with two workgroups a CU.  us of a plan of 262144 pairs, top-8: 256 experts, 32 ranks 28.6, searched in
// memory 29.1; with room for 16640 entries and one workgroup a CU, 33 ranks (in memory so) 37.0 -> 39.5, 200 experts, 42 ranks
// 35.8 -> 39.6, 64 experts, 16 ranks 16.7 -> 18.0.
constexpr int kCumSlice = 8448;

struct PlaceLds {
  int run[kGroup * kRowE];
  int cum[kCumSlice];
  int first[kMostSlots];
  unsigned short sorted[kMostSlots];
};
struct TableLds {
  SlotRows<kMostSlots> slots;
  TableScratch<kMostSlots> scratch;
};

// Workgroups from place_groups on build a table of the grouped GEMMs each, from the slot sizes too: a launch of their own
// behind this one took 5 us of every forward.
__global__ __launch_bounds__(kGroup * lz::kWave) void place_kernel(const int32_t* __restrict__ ids,
                                                    const int32_t* __restrict__ rank_tok_off, int T,
                                                    int E, int N, int c, int k, PlanTables t, bool counted,
                                                    const int32_t* __restrict__ slot_counts,
                                                    int32_t* __restrict__ slot_offsets,
                                                    int32_t* __restrict__ pair_to_row,
                                                    int32_t* __restrict__ row_to_pair, int32_t* __restrict__ status_opt,
                                                    int place_groups, TileSpecs tables, int workgroups) {
  constexpr int kThreads = kGroup * lz::kWave;
  static_assert(kThreads == kTileThreads, "a table a workgroup");
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1], s_gf[lz::kMaxN + 1];
  __shared__ __attribute__((aligned(16))) char lds[sizeof(PlaceLds) > sizeof(TableLds) ? sizeof(PlaceLds) : sizeof(TableLds)];
  __shared__ int s_wave[kGroup];
  __shared__ int s_status;
  const int tid = threadIdx.x, w = tid / lz::kWave;
  const int S = N * c;
  if ((int)blockIdx.x >= place_groups) {
    TableLds& m = *(TableLds*)lds;
    scan_slots(slot_counts, S, m.slots.first, s_wave, [&](int s, int end) { m.slots.end[s] = end; });
    __syncthreads();
    build_table(tables.spec[blockIdx.x - place_groups], false, m.slots, S, m.scratch, tid, workgroups);
    return;
  }
  int* const s_run = ((PlaceLds*)lds)->run;
  int* const s_cum = ((PlaceLds*)lds)->cum;
  int* const s_first = ((PlaceLds*)lds)->first;
  unsigned short* const s_sorted = ((PlaceLds*)lds)->sorted;
  if (tid < lz::kWave) {
    const bool bad = build_split(rank_tok_off, T, N, k, s_off, s_cf, s_gf);
    if (tid == 0) s_status = bad ? LZ_PLAN_BAD_RANK_SPLIT : 0;
  }
  for (int s = tid; s < S; s += kThreads) s_sorted[s] = (unsigned short)t.slot_sorted[s];
  const int end = scan_slots(slot_counts, S, s_first, s_wave, [](int, int) {});
  if (blockIdx.x == 0) {
    int flag = 0;
    for (int e = tid; e < E; e += kThreads) flag |= t.estatus[e];
    if (counted)
      for (int b = tid; b < s_cf[N]; b += kThreads) flag |= t.chunkflag[b];
    if (flag) atomicOr(&s_status, flag);
  }
  const int i = group_rank(s_gf, N), slice = E * (N + 1);
  if (i < N) {
    const int b0 = s_cf[i] + ((int)blockIdx.x - s_gf[i]) * kGroup, chunks = s_cf[i + 1] - b0 < kGroup ? s_cf[i + 1] - b0 : kGroup;
#pragma unroll 4
    for (int x = tid; x < E * kGroup; x += kThreads) {
      const int e = x / kGroup, u = x % kGroup;
      if (u < chunks) s_run[u * kRowE + e] = t.chunkbase[(size_t)e * t.nch + b0 + u];
    }
    if (slice <= kCumSlice) {
#pragma unroll 4  // (9: 256 experts, 32 ranks, 16384, 65536 and 262144 pairs 20.0, 22.4, 27.7 -> 21.0, 23.2, 28.6 us)
      for (int x = tid; x < slice; x += kThreads) s_cum[x] = t.cumDst[(size_t)i * slice + x];
    }
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int s = tid; s < S; s += kThreads) slot_offsets[s] = s_first[s];
    if (tid == kThreads - 1) slot_offsets[S] = end;
    if (tid == 0 && status_opt) *status_opt = s_status;
  }
  if (i == N) return;
  long long p0 = 0, p1 = 0;
  if (group_chunk(i, w, k, s_off, s_cf, s_gf, &p0, &p1) < 0) return;
  int* const run = s_run + w * kRowE;
  auto pre = [&](int e, int j) { return t.preSrc[(size_t)(e * N + i) * N + j]; };
  auto list = [&](int e, int j) {
    const int4 v = t.lists[e * N + j];
    return int3{v.x, v.y, v.z};
  };
  auto sorted = [&](int at) { return (int)s_sorted[at]; };
  auto first = [&](int s) { return s_first[s]; };
  if (slice <= kCumSlice) {
    const PlaceTables lookups{[&](int e, int j) { return s_cum[e * (N + 1) + j]; }, pre, list, sorted, first};
    place_chunk(ids, p0, p1, run, E, N, c, (long long)T * k, lookups, pair_to_row, row_to_pair);
  } else {
    const int32_t* const cum = t.cumDst + (size_t)i * slice;
    const PlaceTables lookups{[=](int e, int j) { return cum[e * (N + 1) + j]; }, pre, list, sorted, first};
    place_chunk(ids, p0, p1, run, E, N, c, (long long)T * k, lookups, pair_to_row, row_to_pair);
  }
}

// ------------------------------------------------------------------------------------------
// The whole dispatcher in one workgroup, tables in LDS: small batches, where two launches and the trips of
// their tables through memory are the time.  Same steps, same results.
// ------------------------------------------------------------------------------------------
constexpr int kSmallPairs = 2048, kSmallExperts = 24;
constexpr int kSmallCounts = 2048, kSmallTriples = 2048, kSmallLists = 512, kSmallSlots = 512;

// Where one workgroup is the faster dispatcher.  Measured (us, this kernel against two launches, 8 ranks): 64 pairs, 8 experts
// 8.0, 11.0; 2048 pairs, 8, 16, 24, 32 experts 9.5, 10.5, 11.3, 12.8 against 11.6, 11.9, 12.1, 12.5; 3072 pairs 11.8, 13.0, 13.9,
// 15.4 against 11.7 to 12.2.  The other bounds are the LDS tables'.
inline bool small_plan(const lz_shape* s) {
  const long long P = (long long)s->T * s->k;
  return P > 0 && P <= kSmallPairs && s->E <= kSmallExperts && (long long)max_chunks(P, s->N) * s->E <= kSmallCounts &&
         s->E * s->N * s->N <= kSmallTriples && s->E * s->N <= kSmallLists && s->N * s->c <= kSmallSlots;
}

// G > 0: it routes the tokens first, G lanes each (logits to ids and gates); tables: it then builds those of the grouped GEMMs.
template <int G>
__global__ __launch_bounds__(kSchedThreads) void plan_small_kernel(
    const float* __restrict__ logits, float* __restrict__ gates, int32_t* __restrict__ ids, const int32_t* __restrict__ rank_tok_off,
    const int32_t* __restrict__ slot_expert,
    int T, int E, int N, int c, int k, int32_t* __restrict__ slot_counts, int32_t* __restrict__ slot_offsets,
    int32_t* __restrict__ pair_to_row, int32_t* __restrict__ row_to_pair, int32_t* __restrict__ Tej_opt,
    int32_t* __restrict__ D_opt, int32_t* __restrict__ status_opt, TileSpecs tables, int workgroups) {
  constexpr int kWaves = kSchedThreads / lz::kWave;
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_cnt[kSmallCounts];                       // [chunk][e] counts, then positions of the first pair
  __shared__ int s_T[kSmallLists], s_R[kSmallLists], s_start[kSmallLists], s_L[kSmallLists], s_O[kSmallLists];
  __shared__ int s_Pre[kSmallLists + lz::kMaxE], s_recv[kSmallLists];
  __shared__ int s_cum[kSmallTriples + kSmallLists];        // [e][i][N + 1]
  __shared__ int s_D[kSmallTriples];                        // [e][i][j], then its prefix over i
  __shared__ int s_expert[kSmallSlots], s_sorted[kSmallSlots], s_first[kSmallSlots];
  __shared__ int s_wave[kWaves];
  __shared__ int s_status;
  __shared__ int s_ids[kSmallPairs];
  __shared__ SlotRows<kSmallSlots> s_rows;
  __shared__ TableScratch<kSmallSlots> s_scratch[2];
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave;
  const int S = N * c;
  const long long P = (long long)T * k;
  if constexpr (G > 0) {
    // (one go: plan_routes)
    route_token<G, 4, false, false>(logits, tid / G, T, E, k, [&](long long t, int kk, int id, float gate) {
      ids[t * k + kk] = id;
      gates[t * k + kk] = gate;
      s_ids[t * k + kk] = id;
    });
  } else {
    for (int p = tid; p < (int)P; p += kSchedThreads) s_ids[p] = ids[p];
  }
  if (tid < lz::kWave) {
    const bool bad = build_split(rank_tok_off, T, N, k, s_off, s_cf);
    if (tid == 0) s_status = bad ? LZ_PLAN_BAD_RANK_SPLIT : 0;
  }
  int flag = 0;
  for (int s = tid; s < S; s += kSchedThreads) {
    const int se = slot_expert[s];
    s_expert[s] = se >= 0 && se < E ? se : E;
    if (s_expert[s] == E) flag |= LZ_PLAN_BAD_EXPERT_ID;
  }
  for (int i = tid; i < kSmallCounts; i += kSchedThreads) s_cnt[i] = 0;
  __syncthreads();
  const int chunks = s_cf[N];

  // ---- counts of the chunks
  for (int b = w; b < chunks; b += kWaves) {
    long long p0 = 0, p1 = 0;
    chunk_range(b, N, k, s_off, s_cf, &p0, &p1);
    for (long long p = p0 + lane; p < p1; p += lz::kWave) {
      const int e = s_ids[p];
      if (e >= 0 && e < E) atomicAdd(&s_cnt[b * E + e], 1);
      else flag |= LZ_PLAN_BAD_EXPERT_ID;
      row_to_pair[p] = -1;  // rows and pairs share the index range [0, P)
    }
  }
  __syncthreads();

  // ---- per (e, j): positions of the chunks, T, R and the index of the first slot in rank j's order
  for (int ej = tid; ej < E * N; ej += kSchedThreads) {
    const int e = ej / N, j = ej % N;
    int running = 0;
    for (int b = s_cf[j]; b < s_cf[j + 1]; ++b) {
      const int n = s_cnt[b * E + e];
      s_cnt[b * E + e] = running;
      running += n;
    }
    int reps = 0, before = 0;
    for (int s = j * c; s < j * c + c; ++s) {
      reps += s_expert[s] == e;
      before += s_expert[s] < e;
    }
    s_T[ej] = running;
    s_R[ej] = reps;
    s_start[ej] = before;
    if (Tej_opt) Tej_opt[ej] = running;
  }
  __syncthreads();
  for (int e = w; e < E; e += kWaves) {
    const Shares sh = shares_of(lane < N ? s_R[e * N + lane] : 0, lane < N ? s_T[e * N + lane] : 0);
    int* const pre = s_Pre + e * (N + 1);
    if (lane < N) {
      s_L[e * N + lane] = sh.keep;
      s_O[e * N + lane] = sh.overflow;
      pre[lane + 1] = sh.residual_upto;
    }
    if (lane == 0) pre[0] = 0;
    if (sh.uncovered) flag |= LZ_PLAN_UNCOVERED_EXPERT;
  }
  __syncthreads();
  for (int x = tid; x < E * N * N; x += kSchedThreads) {
    const int e = x / (N * N), i = x / N % N, j = x % N;
    int cum;
    const int dval = assignment(i, j, N, s_L + e * N, s_Pre + e * (N + 1), s_O + e * N, &cum);
    s_D[x] = dval;
    if (D_opt) D_opt[x] = dval;
    int* const row = s_cum + (e * N + i) * (N + 1);
    row[j] = cum;
    if (j == N - 1) row[N] = cum + dval;
  }
  __syncthreads();
  for (int ej = tid; ej < E * N; ej += kSchedThreads) {
    const int e = ej / N, j = ej % N;
    int running = 0;
    for (int i = 0; i < N; ++i) {
      int& d = s_D[(e * N + i) * N + j];
      const int n = d;
      d = running;
      running += n;
    }
    s_recv[ej] = running;
  }
  if (flag) atomicOr(&s_status, flag);
  __syncthreads();

  // ---- slots: order inside the rank, sizes, offsets (one slot per thread: S <= kSmallSlots < kSchedThreads)
  int count = 0;
  if (tid < S) {
    const int j = tid / c, se = s_expert[tid];
    int pos = 0;
    for (int s2 = j * c; s2 < j * c + c; ++s2) pos += s_expert[s2] < se || (s_expert[s2] == se && s2 < tid);
    s_sorted[j * c + pos] = tid;
    if (se < E) {
      const int ej = se * N + j;
      const long long m = pos - s_start[ej], n = s_recv[ej], reps = s_R[ej];
      count = int(div_floor((m + 1) * n, reps) - div_floor(m * n, reps));
    }
    slot_counts[tid] = count;
  }
  int incl = scan_sum(count);
  if (lane == lz::kWave - 1) s_wave[w] = incl;
  __syncthreads();
  for (int w2 = 0; w2 < w; ++w2) incl += s_wave[w2];
  if (tid < S) {
    s_first[tid] = incl - count;
    slot_offsets[tid] = incl - count;
    s_rows.first[tid] = incl - count;
    s_rows.end[tid] = incl;
  }
  if (tid == kSchedThreads - 1) slot_offsets[S] = incl;
  if (tid == 0 && status_opt) *status_opt = s_status;
  __syncthreads();

  // ---- rows
  for (int b = w; b < chunks; b += kWaves) {
    long long p0 = 0, p1 = 0;
    const int i = chunk_range(b, N, k, s_off, s_cf, &p0, &p1);
    const PlaceTables lookups{[=](int e, int j) { return s_cum[(e * N + i) * (N + 1) + j]; },
                             [=](int e, int j) { return s_D[(e * N + i) * N + j]; },
                             [=](int e, int j) { return int3{s_recv[e * N + j], s_R[e * N + j], s_start[e * N + j]}; },
                             [=](int at) { return s_sorted[at]; }, [=](int s) { return s_first[s]; }};
    place_chunk(s_ids, p0, p1, s_cnt + b * E, E, N, c, P, lookups, pair_to_row, row_to_pair);
  }

  // ---- tables, two at a time
  for (int i = 0; i < tables.n; i += 2) {
    const int half = __builtin_amdgcn_readfirstlane(tid / kTileThreads);
    if (i > 0) __syncthreads();  // the scratch has been read
    build_table(tables.spec[i + half < tables.n ? i + half : i], i + half >= tables.n, s_rows, S, s_scratch[half], tid % kTileThreads,
                workgroups);
  }
}

}  // namespace

extern "C" size_t lz_plan_workspace_bytes(const lz_shape* shape) {
  if (!lz::shape_ok(shape)) return 0;
  return carve(nullptr, shape).total_bytes;
}

namespace {

// Lanes of a token where the one workgroup routes, four logits each.
inline int route_lanes(int E) { return E <= 4 ? 1 : E <= 8 ? 2 : E <= 16 ? 4 : 8; }

// Whether the expert's workgroups count their pairs themselves, each reading all ids.  us, so and with a launch that counts: 2000 pairs,
// 8 and 53 experts 11.4, 12.9 and 12.6, 14.2; 8000 pairs, 16 experts 12.9, 13.7; 8192 pairs, 128 and 256 experts on 4 ranks 14.1, 14.8
// and 15.2, 15.9, on 32 ranks 18.1, 19.1 and 19.2, 20.3; 16384 pairs, 8 experts 14.4, 13.5; 32768 pairs, 32 experts 18.0, 13.9.
inline bool direct_counts(const lz_shape* s) {
  const long long P = (long long)s->T * s->k;
  return P <= kDirectPairs;
}

// The launches of the dispatcher on tables carved from its workspace (already checked by the caller); with logits (where
// plan_routes says so) the routing too, and the tables of the grouped GEMMs that `tables` lists.
int32_t enqueue_plan(const lz::Dispatch& d, const float* logits, float* topk_gates, const TileSpecs& tables, const PlanTables& t,
                     hipStream_t st) {
  const lz_shape* const s = d.shape;
  const long long P = (long long)s->T * s->k;
  const int workgroups = tables.n > 0 ? device_cus() : 0;
  if (tables.n > 0 && workgroups == 0) return LZ_EHIP;
  if (small_plan(s)) {
    const int g = logits == nullptr ? 0 : route_lanes(s->E);
    auto* const kern = g == 0 ? plan_small_kernel<0> : g == 1 ? plan_small_kernel<1> : g == 2 ? plan_small_kernel<2>
                       : g == 4 ? plan_small_kernel<4> : plan_small_kernel<8>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(kSchedThreads), 0, st, logits, topk_gates, d.topk_ids, d.rank_tok_off, d.slot_expert,
                       s->T, s->E, s->N, s->c, s->k, d.slot_counts, d.slot_offsets, d.pair_to_row, d.row_to_pair, d.Tej_opt,
                       d.D_opt, d.status_opt, tables, workgroups);
    return lz::launch_status();
  }
  const unsigned blocks = P > 0 ? (unsigned)max_groups(P, s->N) : 1;
  constexpr int threads = kGroup * lz::kWave;
  const bool direct = direct_counts(s);
  if (direct) {
    hipLaunchKernelGGL(schedule_expert_kernel<true>, dim3(s->E), dim3(1024), 0, st, d.topk_ids, d.rank_tok_off, d.slot_expert,
                       s->T, s->E, s->N, s->c, s->k, t, d.slot_counts, d.row_to_pair, d.Tej_opt, d.D_opt);
  } else {
    if (P > 0)
      hipLaunchKernelGGL(count_kernel, dim3(blocks), dim3(threads), 0, st, d.topk_ids, d.rank_tok_off, s->T, s->E, s->N, s->k, t,
                         d.row_to_pair);
    const int expert_waves = s->N < 4 ? 4 : s->N < 16 ? s->N : 16;  // one per source rank
    hipLaunchKernelGGL(schedule_expert_kernel<false>, dim3(s->E), dim3(lz::kWave * expert_waves), 0, st, d.topk_ids, d.rank_tok_off,
                       d.slot_expert, s->T, s->E, s->N, s->c, s->k, t, d.slot_counts, d.row_to_pair, d.Tej_opt, d.D_opt);
  }
  hipLaunchKernelGGL(place_kernel, dim3(blocks + tables.n), dim3(threads), 0, st, d.topk_ids, d.rank_tok_off, s->T, s->E, s->N, s->c,
                     s->k, t, !direct, d.slot_counts, d.slot_offsets, d.pair_to_row, d.row_to_pair, d.status_opt, (int)blocks, tables,
                     workgroups);
  return lz::launch_status();
}

int32_t check_plan_args(const lz::Dispatch& d) {
  if (!lz::shape_ok(d.shape)) return LZ_ESHAPE;
  if (!d.rank_tok_off || !d.slot_expert || !d.slot_counts || !d.slot_offsets) return LZ_EINVAL;
  const long long P = (long long)d.shape->T * d.shape->k;
  if (P > 0 && (!d.topk_ids || !d.pair_to_row || !d.row_to_pair)) return LZ_EINVAL;
  return LZ_OK;
}

}  // namespace

namespace lz {

// Where the one workgroup routes its tokens in one go.  us of a forward (64 x 64, top-2), routing launched before and inside: 64 and 512
// tokens of 8 experts 22.5, 21.2 and 23.8, 22.8; 256 of 16 experts 24.3, 23.0; two goes, 512 of them, 25.0, 25.2; four 26.2, 29.1.
bool plan_routes(const lz_shape* s) { return shape_ok(s) && small_plan(s) && s->T * route_lanes(s->E) <= kSchedThreads; }

int32_t plan_dispatch(const Dispatch& d, const float* logits, float* topk_gates, const TileSpecs& tables, hipStream_t st) {
  const int32_t rc = check_plan_args(d);
  if (rc != LZ_OK) return rc;
  const PlanTables t = carve(d.ws, d.shape);
  if (!d.ws || (uintptr_t)d.ws % 256 != 0 || d.ws_bytes < t.total_bytes) return LZ_EWORKSPACE;
  return enqueue_plan(d, logits, topk_gates, tables, t, st);
}

}  // namespace lz

extern "C" int32_t lz_plan_dispatch(const int32_t* topk_ids, const lz_shape* shape,
                                    const int32_t* rank_tok_off, const int32_t* slot_expert,
                                    int32_t* slot_counts, int32_t* slot_offsets, int32_t* pair_to_row,
                                    int32_t* row_to_pair, int32_t* Tej_opt, int32_t* D_opt,
                                    int32_t* status_opt, void* ws, size_t ws_bytes, void* stream) {
  const lz::Dispatch d{shape, const_cast<int32_t*>(topk_ids), rank_tok_off, slot_expert, slot_counts, slot_offsets, pair_to_row,
                       row_to_pair, Tej_opt, D_opt, status_opt, ws, ws_bytes};
  return lz::plan_dispatch(d, nullptr, nullptr, TileSpecs{}, (hipStream_t)stream);
}

// ------------------------------------------------------------------------------------------
// The same dispatcher for callers that cannot allocate: its tables live in a fixed array in
// device memory that belongs to the library (one copy per GPU, held until the process ends).
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[LZ_PLAN_NOALLOC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU, looked up once

// Address of this GPU's copy of `scratch`.  In host code the array's name is only a handle for
// the runtime's symbol lookup, never a device address; every GPU has its own copy at its own address.
int32_t scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LZ_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return LZ_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LZ_OK;
}

}  // namespace

extern "C" int32_t lz_plan_dispatch_noalloc(const int32_t* topk_ids, const lz_shape* shape,
                                            const int32_t* rank_tok_off, const int32_t* slot_expert,
                                            int32_t* slot_counts, int32_t* slot_offsets,
                                            int32_t* pair_to_row, int32_t* row_to_pair, int32_t* Tej_opt,
                                            int32_t* D_opt, int32_t* status_opt, void* stream) {
  const lz::Dispatch d{shape, const_cast<int32_t*>(topk_ids), rank_tok_off, slot_expert, slot_counts, slot_offsets, pair_to_row,
                       row_to_pair, Tej_opt, D_opt, status_opt, nullptr, 0};
  const int32_t rc = check_plan_args(d);
  if (rc != LZ_OK) return rc;
  if (carve(nullptr, shape).total_bytes > (size_t)LZ_PLAN_NOALLOC_SCRATCH_BYTES) return LZ_EWORKSPACE;
  void* base = nullptr;
  const int32_t rs = scratch_of_current_device(&base);
  if (rs != LZ_OK) return rs;
  // Every table entry a kernel reads was written earlier in the same call, so what the previous
  // call left in the array does not matter and nothing has to be cleared.
  const PlanTables t = carve(base, shape);
  return enqueue_plan(d, nullptr, nullptr, TileSpecs{}, t, (hipStream_t)stream);
}
