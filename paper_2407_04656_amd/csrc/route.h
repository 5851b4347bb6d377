// Top-k gate routing (Sec. 2.1): for each token the k largest of E logits, descending,
// ties towards the lower expert index, and the softmax over those k logits.
//
// A group of G <= 16 lanes owns one token; a lane keeps V logits in registers, as order-preserving 32-bit
// images.  What bounds the kernel at wide mixtures is ALU work, else the launch.  Two ways of selecting:
//
// Few choices: one selection round is a maximum over the group, then a minimum over the expert indices that hold
// it (the tie rule), both with DPP moves inside a row of 16 lanes.  Few lanes per token: four tokens or more
// share each of those moves.
//
// SORTED, from 5 choices on (the line is drawn in route.hip): a logit and its expert are one key of 40 bits, the image above 255
// minus the expert, so that one maximum decides by both.  The keys are mantissas of doubles between 1 and 2, whose order is theirs: v_max_f64 is one instruction
// where a maximum of 64-bit integers is three.  A lane sorts its keys by a network and keeps the first; a round is a maximum over
// the group's heads, and the lane it came from steps to its next key.  us for 32768 tokens of 256 experts, top-1, 2, 4 and 8: 5.6, 6.7,
// 9.0 and 13.3 the first way, 5.9, 7.9, 9.0 and 10.5 this way; of 64 experts 3.2, 3.6, 4.6, 6.3 and 3.3, 3.8, 4.6, 5.8; 256 tokens of
// 8 experts, top-8 3.6 and 3.4.
// Device code, not part of the C ABI.
#pragma once
#include <type_traits>

#include "lz_common.h"

namespace {

__device__ __forceinline__ uint32_t ordered_bits(float v) {
  v = v + 0.0f;  // -0.0 -> +0.0 so the two zeros compare equal
  uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t o) {
  uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
  return __uint_as_float(u);
}

// Maximum / minimum over the G lanes of a group, in all of them.  quad_perm swaps neighbours, then pairs; the
// mirrors of 8 and 16 lanes combine quads and halves, whose lanes already agree.
template <int G, bool MAX>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v) {
  auto with = [&](uint32_t other) { v = MAX ? (other > v ? other : v) : (other < v ? other : v); };
  if constexpr (G >= 2) with(__builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  if constexpr (G >= 4) with(__builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  if constexpr (G >= 8) with(__builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));   // row_half_mirror
  if constexpr (G >= 16) with(__builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true));  // row_mirror
  return v;
}

// A key as a double, and back: 1 + key 2^-52.
__device__ __forceinline__ double make_key(uint32_t order, uint32_t low) {  // low: 255 minus the expert
  const uint32_t hi = __builtin_amdgcn_alignbit(0x3FF000u, order, 24);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | (uint64_t)((order << 8) + low));
}
__device__ __forceinline__ uint32_t order_of(double key) { return (uint32_t)(__builtin_bit_cast(uint64_t, key) >> 8); }
__device__ __forceinline__ uint32_t expert_of_key(double key) { return 255u - (uint32_t)(__builtin_bit_cast(uint64_t, key) & 255u); }

// (as assembly: the library's forms first make sure that an operand is no signalling NaN)
__device__ __forceinline__ double larger(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
#else
  return a;
#endif
}
__device__ __forceinline__ double smaller(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
#else
  return a;
#endif
}
__device__ __forceinline__ void order2(double& a, double& b) {  // the larger first
  const double hi = larger(a, b);
  b = smaller(a, b);
  a = hi;
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// Maximum over the G lanes of a group, in all of them.  quad_perm swaps neighbours, then pairs; the
// mirrors of 8 and 16 lanes combine quads and halves, whose lanes already agree.
template <int G>
__device__ __forceinline__ double group_max(double v) {
  if constexpr (G >= 2) v = larger(v, dpp<0xB1>(v));    // quad_perm [1,0,3,2]
  if constexpr (G >= 4) v = larger(v, dpp<0x4E>(v));    // quad_perm [2,3,0,1]
  if constexpr (G >= 8) v = larger(v, dpp<0x141>(v));   // row_half_mirror
  if constexpr (G >= 16) v = larger(v, dpp<0x140>(v));  // row_mirror
  return v;
}

__device__ __forceinline__ void sort4(double* v) {
  order2(v[0], v[1]), order2(v[2], v[3]);
  order2(v[0], v[2]), order2(v[1], v[3]);
  order2(v[1], v[2]);
}
// v[0..3] and v[4..7] descending -> v[0..7] descending (odd-even merge)
__device__ __forceinline__ void merge8(double* v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) order2(v[i], v[i + 4]);
#pragma unroll
  for (int i = 2; i < 4; ++i) order2(v[i], v[i + 2]);
#pragma unroll
  for (int i = 1; i < 6; i += 2) order2(v[i], v[i + 1]);
}
// The largest min(V, 8) of V keys, descending, in v[0..].
template <int V>
__device__ __forceinline__ void sort_head(double* v) {
#pragma unroll
  for (int i = 0; i < V; i += 4) sort4(v + i);
#pragma unroll
  for (int i = 0; i + 4 < V; i += 8) merge8(v + i);
  if constexpr (V == 16) {
    // of two descending lists: the larger of one's first against the other's last, and so on, are their eight largest, which
    // rise and fall once at most
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = larger(v[i], v[15 - i]);
#pragma unroll
    for (int d = 4; d > 0; d /= 2)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & d) == 0) order2(v[i], v[i + d]);
  }
}

// Lane l of a group holds the experts 4 (G q + l) + 0..3, q = 0 .. V/4 - 1; VEC: as one 16-byte load each.
// A token's choices go to emit(token, kk, expert, gate).
template <int G, int V, bool VEC, bool SORTED, typename Emit>
__device__ __forceinline__ void route_token(const float* __restrict__ logits, long long token, int T, int E, int k, Emit emit) {
  const int lane_in_group = threadIdx.x % G;
  const bool live = token < T;
  const long long tok = live ? token : 0;  // idle groups shadow token 0 and write nothing
  const float* const row = logits + tok * E;
  const int e0 = 4 * lane_in_group;  // expert of v: e0 + expert_of(v)
  auto expert_of = [](int v) { return (v >> 2) * 4 * G + (v & 3); };

  // 0 = absent / already taken; any real image is larger
  typename std::conditional<SORTED, double, uint32_t>::type key[V];
#pragma unroll
  for (int q = 0; q < V / 4; ++q) {
    // Absent logits read the row's first: loads under a test would each be waited for before the next (256 experts, top-8, with the
    // plan 35.7 -> 38.4 us).  A lane's only load is under one: 512 tokens of 4 experts, top-3, 2.77 us without, 2.65 with.
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    const int e = e0 + expert_of(4 * q);
    if constexpr (VEC) {
      constexpr bool kOnly = V == 4 && !SORTED;
      if (!kOnly || e < E) {
        const float4 f = *(const float4*)(row + (kOnly || e < E ? e : 0));
        x[0] = f.x, x[1] = f.y, x[2] = f.z, x[3] = f.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = row[e + i < E ? e + i : 0];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool real = (VEC ? e : e + i) < E;
      const uint32_t bits = ordered_bits(x[i]), o = real ? (bits > 0 ? bits : 1) : 0;
      if constexpr (SORTED) key[4 * q + i] = make_key(o, real ? (uint32_t)(255 - e - i) : 0u);
      else key[4 * q + i] = o;
    }
  }

  // lane kk of the group (every lane where G < 8) keeps the kk-th selection
  uint32_t sel[lz::kMaxK], sel_id[lz::kMaxK], top = 0, my_key = 0, my_id = 0;
  if constexpr (SORTED) sort_head<V>(key);
#pragma unroll
  for (int kk = 0; kk < lz::kMaxK; ++kk) {
    sel[kk] = 0;
    sel_id[kk] = 0;
    if (kk < k) {
      uint32_t best, at;
      if constexpr (SORTED) {
        constexpr int kHead = V < lz::kMaxK ? V : lz::kMaxK;
        const double of_group = group_max<G>(key[0]);
        const bool own = key[0] == of_group;  // in one lane: the keys of a token differ
#pragma unroll
        for (int v = 0; v < kHead; ++v)
          if (v < lz::kMaxK - 1 - kk) {
            const double next = v + 1 < kHead ? key[v + 1] : make_key(0, 0);  // (by value: a choice of two elements would be an index)
            if (own) key[v] = next;
          }
        best = order_of(of_group);
        at = expert_of_key(of_group);
      } else {
        best = key[0];
#pragma unroll
        for (int v = 1; v < V; ++v) best = key[v] > best ? key[v] : best;
        best = group_reduce<G, true>(best);
        at = 0xFFFFFFFFu;
#pragma unroll
        for (int v = V - 1; v >= 0; --v) at = key[v] == best ? (uint32_t)(e0 + expert_of(v)) : at;
        at = group_reduce<G, false>(at);
        const int mine = (int)at - e0;
#pragma unroll
        for (int v = 0; v < V; ++v) key[v] = mine == expert_of(v) ? 0 : key[v];
      }
      if (kk == 0) top = best;
      if constexpr (G < 8) {
        sel[kk] = best;
        sel_id[kk] = at;
      } else if (lane_in_group == kk) {
        my_key = best;
        my_id = at;
      }
    }
  }

  const float first = from_ordered_bits(top);
  if constexpr (G < 8) {
    if (live && lane_in_group == 0) {
      float ex[lz::kMaxK];
      float denom = 0.f;
#pragma unroll
      for (int kk = 0; kk < lz::kMaxK; ++kk) {
        ex[kk] = 0.f;
        if (kk < k) {
          ex[kk] = expf(from_ordered_bits(sel[kk]) - first);
          denom += ex[kk];
        }
      }
#pragma unroll
      for (int kk = 0; kk < lz::kMaxK; ++kk)
        if (kk < k) {
          emit(tok, kk, (int)sel_id[kk], ex[kk] / denom);
        }
    }
  } else {
    const float ex = expf(from_ordered_bits(my_key) - first);
    float denom = 0.f;
    for (int kk = 0; kk < k; ++kk) denom += __shfl(ex, kk, G);  // ascending, like the other branch
    if (live && lane_in_group < k) emit(tok, lane_in_group, (int)my_id, ex / denom);
  }
}

}  // namespace
