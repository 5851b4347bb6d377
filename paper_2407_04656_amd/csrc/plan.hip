// The flexible token dispatcher (Algorithm 1, Sec. 4.2) for all source ranks at once.
//
// Four kernels on one stream, no host synchronisation, no order-dependent atomics:
//   count    each wave owns a chunk of <= 128 consecutive pairs of ONE source rank and
//            histograms their expert ids with LDS atomics (counts commute)
//   schedule one workgroup per expert scans the chunk histograms into per-(expert, rank) list
//            positions and evaluates the algorithm's counts in exact integers, in LDS; one
//            more workgroup then cuts every (expert, rank) receive list over that rank's
//            replicas and scans the slot sizes
//   place    each wave revisits its chunk; a pair's position in its (expert, source rank)
//            list is chunk base + ordered rank inside the chunk (wave ballots, one per
//            bit of an expert index), which fixes destination rank, slot and row
// Small batches take all of it in one workgroup (plan_small_kernel).
// Each is a chain of dependent lookups over little data: latency bound.  32768 tokens, 256 experts, top-8, 32
// ranks of 10 slots, the four kernels and the routing: 109 us -> 50 us with the lookups of a chunk's two halves
// side by side, more waves on the chunk scans and the closed form of the assignments.
#include <mutex>

#include "lz_common.h"

namespace {

constexpr int kChunk = 128;          // pairs per wave-chunk
constexpr int kWavesPerBlock = 4;
constexpr int kSchedThreads = 1024;

struct PlanTables {
  // per chunk
  int32_t* chunkcnt;   // [nch, E]
  int32_t* chunkbase;  // [nch, E]  position of the chunk's first pair of e in its (e, rank) list
  int32_t* chunkflag;  // [nch]
  // per (expert, rank)
  int32_t* Tej;        // [E, N]
  int32_t* R;          // [E, N]
  int32_t* recv;       // [E, N]
  int32_t* ejstart;    // [E, N]  index of the first slot of e in rank j's sorted slot list
  int32_t* estatus;    // [E]     status bits raised while scheduling expert e
  // per (expert, src, dst)
  int32_t* D;          // [E, N, N]
  int32_t* cumDst;     // [E, N, N+1] prefix of D over dst
  int32_t* preSrc;     // [E, N, N]   prefix of D over src
  // per slot
  int32_t* slot_sorted;  // [S] rank j's slots ordered by (expert, slot id)
  size_t total_bytes;
};

__host__ __device__ inline int max_chunks(long long P, int N) { return int((P + kChunk - 1) / kChunk) + N; }

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
  t.chunkcnt = take(nch * E);
  t.chunkbase = take(nch * E);
  t.chunkflag = take(nch);
  t.Tej = take(E * N);
  t.R = take(E * N);
  t.recv = take(E * N);
  t.ejstart = take(E * N);
  t.estatus = take(E);
  t.D = take(E * N * N);
  t.cumDst = take(E * N * (N + 1));
  t.preSrc = take(E * N * N);
  t.slot_sorted = take(S);
  t.total_bytes = off;
  return t;
}

// Sanitised batch split and the chunk table derived from it, rebuilt by every workgroup: called by its first
// wave, lane i for the end of rank i (N <= 64).  An entry counts for at least its predecessors and at most T,
// the last for T.  Returns true (in every lane) if rank_tok_off had to be repaired.
__device__ bool build_split(const int32_t* __restrict__ rank_tok_off, int T, int N, int k,
                            int* s_off, int* s_cf) {
  const int lane = threadIdx.x;  // < 64
  const int raw = lane < N ? rank_tok_off[lane + 1] : T;
  int v = lane < N - 1 ? (raw < 0 ? 0 : raw > T ? T : raw) : T;
  const int own = v;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const int n = __shfl_up(v, off);
    if (lane >= off && n > v) v = n;
  }
  const int up = __shfl_up(v, 1);
  const int prev = lane == 0 ? 0 : up;
  const bool bad = lane < N - 1 ? raw < 0 || raw > T || own < prev : lane == N - 1 && raw != T;
  int chunks = lane < N ? int(((long long)(v - prev) * k + kChunk - 1) / kChunk) : 0;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const int n = __shfl_up(chunks, off);
    if (lane >= off) chunks += n;
  }
  if (lane == 0) s_off[0] = s_cf[0] = 0;
  if (lane < N) {
    s_off[lane + 1] = v;
    s_cf[lane + 1] = chunks;
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

__global__ __launch_bounds__(256) void count_kernel(const int32_t* __restrict__ ids,
                                                    const int32_t* __restrict__ rank_tok_off, int T,
                                                    int E, int N, int k, PlanTables t,
                                                    int32_t* __restrict__ row_to_pair) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_cnt[kWavesPerBlock][lz::kMaxE];
  const int lane = threadIdx.x % lz::kWave, w = threadIdx.x / lz::kWave;
  if (threadIdx.x < lz::kWave) build_split(rank_tok_off, T, N, k, s_off, s_cf);
  for (int e = lane; e < E; e += lz::kWave) s_cnt[w][e] = 0;
  __syncthreads();
  const int b = blockIdx.x * kWavesPerBlock + w;
  long long p0 = 0, p1 = 0;
  const int rank = chunk_range(b, N, k, s_off, s_cf, &p0, &p1);
  if (rank < 0) return;
  int flag = 0;
  for (long long p = p0 + lane; p < p1; p += lz::kWave) {
    const int e = ids[p];
    if (e >= 0 && e < E) atomicAdd(&s_cnt[w][e], 1);
    else flag = LZ_PLAN_BAD_EXPERT_ID;
    row_to_pair[p] = -1;  // rows and pairs share the index range [0, P)
  }
  flag = __any(flag) ? LZ_PLAN_BAD_EXPERT_ID : 0;
  // LDS atomics of this wave have completed before its own later LDS reads
  __builtin_amdgcn_wave_barrier();
  for (int e = lane; e < E; e += lz::kWave) t.chunkcnt[(size_t)b * E + e] = s_cnt[w][e];
  if (lane == 0) t.chunkflag[b] = flag;
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
  const int lane = threadIdx.x % lz::kWave;
  long long hi = R, te = T;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const long long nr = __shfl_up(hi, off), nt = __shfl_up(te, off);
    if (lane >= off) {
      hi += nr;
      te += nt;
    }
  }
  const long long re = __shfl(hi, lz::kWave - 1);
  te = __shfl(te, lz::kWave - 1);
  const long long lo = hi - R;
  const int cap = re > 0 ? int(div_floor(hi * te, re) - div_floor(lo * te, re)) : 0;
  Shares s;
  s.keep = cap < T ? cap : T;
  s.overflow = T - s.keep;
  s.residual_upto = cap - s.keep;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const int n = __shfl_up(s.residual_upto, off);
    if (lane >= off) s.residual_upto += n;
  }
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
// not global-memory round trips; the tables the other kernels read are written out once.
// What bounds it is the latency of those steps: a wave per source rank for the chunk scans (up to 16 waves),
// a thread per (source, destination) for the assignments, whose prefix over destinations has a closed form.
__global__ __launch_bounds__(1024) void schedule_expert_kernel(
    const int32_t* __restrict__ rank_tok_off, const int32_t* __restrict__ slot_expert, int T, int E,
    int N, int c, int k, PlanTables t, int32_t* __restrict__ Tej_opt, int32_t* __restrict__ D_opt) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_R[lz::kMaxN], s_T[lz::kMaxN], s_L[lz::kMaxN], s_P[lz::kMaxN + 1], s_O[lz::kMaxN];
  __shared__ int s_D[lz::kMaxN * lz::kMaxN];
  const int e = blockIdx.x;
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave, n_waves = blockDim.x / lz::kWave;
  if (tid < lz::kWave) build_split(rank_tok_off, T, N, k, s_off, s_cf);
  __syncthreads();

  // ---- per source rank j (one wave each): positions of the chunks in the (e, j) list, T[e,j],
  // the replicas of e on rank j and the index of their first slot in j's sorted slot list
  for (int j = w; j < N; j += n_waves) {
    const int b_end = s_cf[j + 1];
    int running = 0, b = s_cf[j] + lane;
    int v = b < b_end ? t.chunkcnt[(size_t)b * E + e] : 0;
    int reps = 0, before = 0;
    for (int l0 = 0; l0 < c; l0 += lz::kWave) {
      const int l = l0 + lane;
      const int se = l < c ? slot_expert[j * c + l] : -1;
      reps += __popcll(__ballot(l < c && se == e));
      before += __popcll(__ballot(l < c && se >= 0 && se < e));
    }
    for (int b0 = s_cf[j]; b0 < b_end; b0 += lz::kWave) {
      const int b_next = b + lz::kWave;
      const int v_next = b_next < b_end ? t.chunkcnt[(size_t)b_next * E + e] : 0;
      int incl = v;
#pragma unroll
      for (int off = 1; off < lz::kWave; off <<= 1) {
        const int n = __shfl_up(incl, off);
        if (lane >= off) incl += n;
      }
      if (b < b_end) t.chunkbase[(size_t)b * E + e] = running + incl - v;
      running += __shfl(incl, lz::kWave - 1);
      b = b_next;
      v = v_next;
    }
    if (lane == 0) {
      const int idx = e * N + j;
      s_T[j] = running;
      s_R[j] = reps;
      t.Tej[idx] = running;
      if (Tej_opt) Tej_opt[idx] = running;
      t.R[idx] = reps;
      t.ejstart[idx] = before;
    }
  }
  __syncthreads();

  // ---- one wave, lane = rank: capacity, local share, residual and its prefix over ranks, overflow
  if (w == 0) {
    const Shares sh = shares_of(lane < N ? s_R[lane] : 0, lane < N ? s_T[lane] : 0);
    if (lane < N) {
      s_L[lane] = sh.keep;
      s_P[lane + 1] = sh.residual_upto;
      s_O[lane] = sh.overflow;
    }
    if (lane == 0) {
      s_P[0] = 0;
      t.estatus[e] = sh.uncovered ? LZ_PLAN_UNCOVERED_EXPERT : 0;
    }
  }
  __syncthreads();

  // ---- D[e, i, j] and its prefix over destinations
  for (int ij = tid; ij < N * N; ij += blockDim.x) {
    const int i = ij / N, j = ij % N, idx = e * N + i;
    int cum;
    const int dval = assignment(i, j, N, s_L, s_P, s_O, &cum);
    s_D[ij] = dval;
    t.D[(size_t)idx * N + j] = dval;
    if (D_opt) D_opt[(size_t)idx * N + j] = dval;
    t.cumDst[(size_t)idx * (N + 1) + j] = cum;
    if (j == N - 1) t.cumDst[(size_t)idx * (N + 1) + N] = cum + dval;
  }
  __syncthreads();

  // ---- receive side: prefix over source ranks, recv[e, j]
  if (tid < N) {
    const int j = tid;
    int running = 0;
    for (int i = 0; i < N; ++i) {
      t.preSrc[((size_t)(e * N + i)) * N + j] = running;
      running += s_D[i * N + j];
    }
    t.recv[e * N + j] = running;
  }
}

// Slot order inside every rank, slot sizes (balanced cut of the (e, j) receive list over its
// R[e, j] slots), their exclusive scan, and the status word.  One workgroup.
__global__ __launch_bounds__(kSchedThreads) void schedule_slots_kernel(
    const int32_t* __restrict__ rank_tok_off, const int32_t* __restrict__ slot_expert, int T, int E,
    int N, int c, int k, PlanTables t, int32_t* __restrict__ slot_counts,
    int32_t* __restrict__ slot_offsets, int32_t* __restrict__ status_opt) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_status;
  __shared__ int s_wave[kSchedThreads / lz::kWave];
  __shared__ int s_expert[lz::kMaxN * lz::kMaxC], s_count[lz::kMaxN * lz::kMaxC];
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave;
  const int S = N * c;
  for (int s = tid; s < S; s += kSchedThreads) {
    const int se = slot_expert[s];
    s_expert[s] = se >= 0 && se < E ? se : E;
  }
  if (tid < lz::kWave) {
    const bool bad = build_split(rank_tok_off, T, N, k, s_off, s_cf);
    if (tid == 0) s_status = bad ? LZ_PLAN_BAD_RANK_SPLIT : 0;
  }
  __syncthreads();
  int flag = 0;
  for (int b = tid; b < s_cf[N]; b += kSchedThreads) flag |= t.chunkflag[b];
  for (int e = tid; e < E; e += kSchedThreads) flag |= t.estatus[e];
  for (int s = tid; s < S; s += kSchedThreads) {
    const int j = s / c, se = s_expert[s];
    if (se == E) flag |= LZ_PLAN_BAD_EXPERT_ID;
    int pos = 0;
    for (int s2 = j * c; s2 < j * c + c; ++s2) pos += s_expert[s2] < se || (s_expert[s2] == se && s2 < s);
    t.slot_sorted[j * c + pos] = s;
    int cnt = 0;
    if (se < E) {
      const int ej = se * N + j;
      const long long m = pos - t.ejstart[ej];
      const long long n = t.recv[ej], reps = t.R[ej];
      cnt = int(div_floor((m + 1) * n, reps) - div_floor(m * n, reps));
    }
    slot_counts[s] = cnt;
    s_count[s] = cnt;
  }
  if (flag) atomicOr(&s_status, flag);
  __syncthreads();

  // ---- exclusive scan over slot id (each thread owns a run of consecutive slots)
  const int per = (S + kSchedThreads - 1) / kSchedThreads;
  const int first = tid * per;
  int local = 0;
  for (int s = first; s < first + per && s < S; ++s) local += s_count[s];
  int incl = local;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const int n = __shfl_up(incl, off);
    if (lane >= off) incl += n;
  }
  if (lane == lz::kWave - 1) s_wave[w] = incl;
  __syncthreads();
  for (int w2 = 0; w2 < w; ++w2) incl += s_wave[w2];
  int running = incl - local;
  for (int s = first; s < first + per && s < S; ++s) {
    slot_offsets[s] = running;
    running += s_count[s];
  }
  if (tid == kSchedThreads - 1) slot_offsets[S] = incl;
  if (tid == 0 && status_opt) *status_opt = s_status;
}

// One wave places the pairs [p0, p1) of a chunk of source rank i; run[e]: position of its first pair of e in the
// (e, i) list, advanced here.
__device__ __forceinline__ void place_chunk(const int32_t* __restrict__ ids, long long p0, long long p1, int i, int* run, int E,
                                            int N, int c, long long P, const int32_t* cumDst, const int32_t* preSrc,
                                            const int32_t* recv, const int32_t* R, const int32_t* ejstart,
                                            const int32_t* slot_sorted, const int32_t* slot_offsets,
                                            int32_t* __restrict__ pair_to_row, int32_t* __restrict__ row_to_pair) {
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
  const int32_t* cum[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    cum[u] = cumDst + (size_t)((ex[u] < 0 ? 0 : ex[u]) * N + i) * (N + 1);
    row[u] = -1;
    dst[u] = 0;
    ok[u] = ex[u] >= 0 && q[u] < cum[u][N];
  }
  // destination rank: the last j with cum[j] <= q (cum[0] = 0)
  int step = 1;
  while (step * 2 < N) step *= 2;
  for (; step > 0; step >>= 1) {
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const int j = dst[u] + step;
      if (j < N && cum[u][j] <= q[u]) dst[u] = j;
    }
  }
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    if (ok[u]) {
      const int ei = ex[u] * N + i, j = dst[u], ej = ex[u] * N + j;
      const long long pos = preSrc[(size_t)ei * N + j] + (q[u] - cum[u][j]);
      const long long n = recv[ej], reps = R[ej];
      if (n > 0 && reps > 0) {
        // slot m of the (e, j) list holds positions [floor(m*n/reps), floor((m+1)*n/reps))
        long long m = div_floor((pos + 1) * reps - 1, n);
        m = m < reps ? m : reps - 1;
        const int s = slot_sorted[j * c + ejstart[ej] + (int)m];
        const long long r = slot_offsets[s] + pos - div_floor(m * n, reps);
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

__global__ __launch_bounds__(256) void place_kernel(const int32_t* __restrict__ ids,
                                                    const int32_t* __restrict__ rank_tok_off, int T,
                                                    int E, int N, int c, int k, PlanTables t,
                                                    const int32_t* __restrict__ slot_offsets,
                                                    int32_t* __restrict__ pair_to_row,
                                                    int32_t* __restrict__ row_to_pair) {
  __shared__ int s_off[lz::kMaxN + 1], s_cf[lz::kMaxN + 1];
  __shared__ int s_run[kWavesPerBlock][lz::kMaxE];
  const int lane = threadIdx.x % lz::kWave, w = threadIdx.x / lz::kWave;
  if (threadIdx.x < lz::kWave) build_split(rank_tok_off, T, N, k, s_off, s_cf);
  __syncthreads();
  const int b = blockIdx.x * kWavesPerBlock + w;
  long long p0 = 0, p1 = 0;
  const int i = chunk_range(b, N, k, s_off, s_cf, &p0, &p1);
  if (i < 0) return;
  for (int e = lane; e < E; e += lz::kWave) s_run[w][e] = t.chunkbase[(size_t)b * E + e];
  __builtin_amdgcn_wave_barrier();
  place_chunk(ids, p0, p1, i, s_run[w], E, N, c, (long long)T * k, t.cumDst, t.preSrc, t.recv, t.R, t.ejstart, t.slot_sorted,
              slot_offsets, pair_to_row, row_to_pair);
}

// ------------------------------------------------------------------------------------------
// The whole dispatcher in one workgroup, tables in LDS: small batches, where the four launches and the trips of
// their tables through memory are the time.  Same steps, same results.
// ------------------------------------------------------------------------------------------
constexpr int kSmallPairs = 4096, kSmallCounts = 4096, kSmallTriples = 2048, kSmallLists = 512, kSmallSlots = 512;

// Where one workgroup is the faster dispatcher.  Measured (us, this kernel against the four): 128 pairs, 8 experts, 8
// ranks 9.6, 17.8; 2048 pairs 11.1, 18.8; 4096 pairs 15.0, 19.2; 16 experts 16.7, 19.3; 32 experts, 2048 pairs 15.9,
// 19.5; 60 experts, 3600 pairs 23.4, 20.6; 128 experts, 120 pairs 28.1, 18.9.  The other bounds are the LDS tables'.
inline bool small_plan(const lz_shape* s) {
  const long long P = (long long)s->T * s->k;
  return P > 0 && P <= kSmallPairs && s->E <= 32 && (long long)max_chunks(P, s->N) * s->E <= kSmallCounts &&
         s->E * s->N * s->N <= kSmallTriples && s->E * s->N <= kSmallLists && s->N * s->c <= kSmallSlots;
}

__global__ __launch_bounds__(kSchedThreads) void plan_small_kernel(
    const int32_t* __restrict__ ids, const int32_t* __restrict__ rank_tok_off, const int32_t* __restrict__ slot_expert,
    int T, int E, int N, int c, int k, int32_t* __restrict__ slot_counts, int32_t* __restrict__ slot_offsets,
    int32_t* __restrict__ pair_to_row, int32_t* __restrict__ row_to_pair, int32_t* __restrict__ Tej_opt,
    int32_t* __restrict__ D_opt, int32_t* __restrict__ status_opt) {
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
  const int tid = threadIdx.x, lane = tid % lz::kWave, w = tid / lz::kWave;
  const int S = N * c;
  const long long P = (long long)T * k;
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
      const int e = ids[p];
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
  int incl = count;
#pragma unroll
  for (int off = 1; off < lz::kWave; off <<= 1) {
    const int n = __shfl_up(incl, off);
    if (lane >= off) incl += n;
  }
  if (lane == lz::kWave - 1) s_wave[w] = incl;
  __syncthreads();
  for (int w2 = 0; w2 < w; ++w2) incl += s_wave[w2];
  if (tid < S) {
    s_first[tid] = incl - count;
    slot_offsets[tid] = incl - count;
  }
  if (tid == kSchedThreads - 1) slot_offsets[S] = incl;
  if (tid == 0 && status_opt) *status_opt = s_status;
  __syncthreads();

  // ---- rows
  for (int b = w; b < chunks; b += kWaves) {
    long long p0 = 0, p1 = 0;
    const int i = chunk_range(b, N, k, s_off, s_cf, &p0, &p1);
    place_chunk(ids, p0, p1, i, s_cnt + b * E, E, N, c, P, s_cum, s_D, s_recv, s_R, s_start, s_sorted, s_first, pair_to_row,
                row_to_pair);
  }
}

}  // namespace

extern "C" size_t lz_plan_workspace_bytes(const lz_shape* shape) {
  if (!lz::shape_ok(shape)) return 0;
  return carve(nullptr, shape).total_bytes;
}

namespace {

// The four launches of the dispatcher on tables carved from `ws` (already checked by the caller).
int32_t enqueue_plan(const int32_t* topk_ids, const lz_shape* shape, const int32_t* rank_tok_off,
                     const int32_t* slot_expert, int32_t* slot_counts, int32_t* slot_offsets,
                     int32_t* pair_to_row, int32_t* row_to_pair, int32_t* Tej_opt, int32_t* D_opt,
                     int32_t* status_opt, const PlanTables& t, hipStream_t st) {
  const long long P = (long long)shape->T * shape->k;
  if (small_plan(shape)) {
    hipLaunchKernelGGL(plan_small_kernel, dim3(1), dim3(kSchedThreads), 0, st, topk_ids, rank_tok_off, slot_expert, shape->T,
                       shape->E, shape->N, shape->c, shape->k, slot_counts, slot_offsets, pair_to_row, row_to_pair, Tej_opt,
                       D_opt, status_opt);
    return lz::launch_status();
  }
  const int nch = max_chunks(P, shape->N);
  const unsigned blocks = unsigned((nch + kWavesPerBlock - 1) / kWavesPerBlock);
  if (P > 0)
    hipLaunchKernelGGL(count_kernel, dim3(blocks), dim3(256), 0, st, topk_ids, rank_tok_off, shape->T,
                       shape->E, shape->N, shape->k, t, row_to_pair);
  const int expert_waves = shape->N < 4 ? 4 : shape->N < 16 ? shape->N : 16;  // one per source rank
  hipLaunchKernelGGL(schedule_expert_kernel, dim3(shape->E), dim3(lz::kWave * expert_waves), 0, st, rank_tok_off,
                     slot_expert, shape->T, shape->E, shape->N, shape->c, shape->k, t, Tej_opt, D_opt);
  hipLaunchKernelGGL(schedule_slots_kernel, dim3(1), dim3(kSchedThreads), 0, st, rank_tok_off, slot_expert,
                     shape->T, shape->E, shape->N, shape->c, shape->k, t, slot_counts, slot_offsets,
                     status_opt);
  if (P > 0)
    hipLaunchKernelGGL(place_kernel, dim3(blocks), dim3(256), 0, st, topk_ids, rank_tok_off, shape->T,
                       shape->E, shape->N, shape->c, shape->k, t, slot_offsets, pair_to_row,
                       row_to_pair);
  return lz::launch_status();
}

int32_t check_plan_args(const int32_t* topk_ids, const lz_shape* shape, const int32_t* rank_tok_off,
                        const int32_t* slot_expert, const int32_t* slot_counts, const int32_t* slot_offsets,
                        const int32_t* pair_to_row, const int32_t* row_to_pair) {
  if (!lz::shape_ok(shape)) return LZ_ESHAPE;
  if (!rank_tok_off || !slot_expert || !slot_counts || !slot_offsets) return LZ_EINVAL;
  const long long P = (long long)shape->T * shape->k;
  if (P > 0 && (!topk_ids || !pair_to_row || !row_to_pair)) return LZ_EINVAL;
  return LZ_OK;
}

}  // namespace

extern "C" int32_t lz_plan_dispatch(const int32_t* topk_ids, const lz_shape* shape,
                                    const int32_t* rank_tok_off, const int32_t* slot_expert,
                                    int32_t* slot_counts, int32_t* slot_offsets, int32_t* pair_to_row,
                                    int32_t* row_to_pair, int32_t* Tej_opt, int32_t* D_opt,
                                    int32_t* status_opt, void* ws, size_t ws_bytes, void* stream) {
  const int32_t rc = check_plan_args(topk_ids, shape, rank_tok_off, slot_expert, slot_counts, slot_offsets,
                                     pair_to_row, row_to_pair);
  if (rc != LZ_OK) return rc;
  PlanTables t = carve(ws, shape);
  if (!ws || (uintptr_t)ws % 256 != 0 || ws_bytes < t.total_bytes) return LZ_EWORKSPACE;
  return enqueue_plan(topk_ids, shape, rank_tok_off, slot_expert, slot_counts, slot_offsets, pair_to_row,
                      row_to_pair, Tej_opt, D_opt, status_opt, t, (hipStream_t)stream);
}

// ------------------------------------------------------------------------------------------
// The same dispatcher for callers that cannot allocate: its tables live in a fixed array in
// device memory that belongs to the library (one copy per GPU, held until the process ends).
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[LZ_PLAN_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
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
  const int32_t rc = check_plan_args(topk_ids, shape, rank_tok_off, slot_expert, slot_counts, slot_offsets,
                                     pair_to_row, row_to_pair);
  if (rc != LZ_OK) return rc;
  if (carve(nullptr, shape).total_bytes > (size_t)LZ_PLAN_NOALLOC_SCRATCH_BYTES) return LZ_EWORKSPACE;
  void* base = nullptr;
  const int32_t rs = scratch_of_current_device(&base);
  if (rs != LZ_OK) return rs;
  // Every table entry a kernel reads was written earlier in the same call, so what the previous
  // call left in the array does not matter and nothing has to be cleared.
  const PlanTables t = carve(base, shape);
  return enqueue_plan(topk_ids, shape, rank_tok_off, slot_expert, slot_counts, slot_offsets, pair_to_row,
                      row_to_pair, Tej_opt, D_opt, status_opt, t, (hipStream_t)stream);
}
