// Candidates of the beam step, ordered in registers: higher value first, then lower index.
#pragma once
#include "common.h"

namespace san {

struct Cand {
  float v;
  int i;
};
// a is better than b
__device__ __forceinline__ bool better(float av, int ai, float bv, int bi) {
  return av > bv || (av == bv && ai < bi);
}

constexpr int kNone = 0x7fffffff;   // index of an empty candidate slot (value -inf)

// One compare-exchange stage of a bitonic network over the 64 lanes: partner is
// lane ^ J; inside blocks of K lanes that sort "best first" the lower lane of a
// pair keeps the better element, in the other blocks the worse one.
template <int K, int J> __device__ __forceinline__ void sort_stage(Cand& c, int lane) {
  const float ov = __uint_as_float(lane_xor<J>(__float_as_uint(c.v)));
  const int oi = (int)lane_xor<J>((unsigned)c.i);
  const bool lower = (lane & J) == 0;
  const bool best_first = K == kWave || (lane & K) == 0;
  const bool other_better = better(ov, oi, c.v, c.i);
  if ((lower == best_first) ? other_better : !other_better) { c.v = ov; c.i = oi; }
}
// Sorts the (value, index) pairs of each aligned group of N lanes (N = 16, 32 or 64),
// best first: lane r of the group ends up with rank r.  Register-only stages (10
// for N = 16, 15 for N = 32, 21 for N = 64); equal pairs can only be empty slots.
template <int N> __device__ __forceinline__ void wave_sort(Cand& c, int lane) {
  static_assert(N == 16 || N == 32 || N == kWave, "group size");
  sort_stage<2, 1>(c, lane);
  sort_stage<4, 2>(c, lane); sort_stage<4, 1>(c, lane);
  sort_stage<8, 4>(c, lane); sort_stage<8, 2>(c, lane); sort_stage<8, 1>(c, lane);
  if (N == 16) {
    // last merge of a 16-lane group: every group sorts best first
    sort_stage<kWave, 8>(c, lane); sort_stage<kWave, 4>(c, lane); sort_stage<kWave, 2>(c, lane);
    sort_stage<kWave, 1>(c, lane);
    return;
  }
  sort_stage<16, 8>(c, lane); sort_stage<16, 4>(c, lane); sort_stage<16, 2>(c, lane); sort_stage<16, 1>(c, lane);
  if (N == 32) {
    sort_stage<kWave, 16>(c, lane); sort_stage<kWave, 8>(c, lane); sort_stage<kWave, 4>(c, lane);
    sort_stage<kWave, 2>(c, lane); sort_stage<kWave, 1>(c, lane);
    return;
  }
  sort_stage<32, 16>(c, lane); sort_stage<32, 8>(c, lane); sort_stage<32, 4>(c, lane); sort_stage<32, 2>(c, lane);
  sort_stage<32, 1>(c, lane);
  sort_stage<64, 32>(c, lane); sort_stage<64, 16>(c, lane); sort_stage<64, 8>(c, lane); sort_stage<64, 4>(c, lane);
  sort_stage<64, 2>(c, lane); sort_stage<64, 1>(c, lane);
}
// The k best of the candidates load(0..nc-1), best first in lanes 0..k-1 (k <= 32).
// Up to 16 candidates: one short sort.  Otherwise 64 candidates per pass; the running
// k best ride along in lanes k..2k-1 of the next pass.
template <typename F> __device__ __forceinline__ Cand wave_topk(F load, int nc, int k, int lane) {
  Cand cur = {-INFINITY, kNone};
  if (nc <= 16) {
    if (lane < nc) cur = load(lane);
    wave_sort<16>(cur, lane);
    return cur;
  }
  for (int base = 0; base < nc; base += kWave) {
    Cand c = {-INFINITY, kNone};
    if (base + lane < nc) c = load(base + lane);
    wave_sort<kWave>(c, lane);
    if (base > 0) {
      const float mv = __shfl(cur.v, lane - k, kWave);
      const int mi = __shfl(cur.i, lane - k, kWave);
      if (lane >= k) {
        c.v = lane < 2 * k ? mv : -INFINITY;
        c.i = lane < 2 * k ? mi : kNone;
      }
      wave_sort<kWave>(c, lane);
    }
    cur = c;
  }
  return cur;
}

// c: per half-wave 32 candidates, best first; o: the candidates of another such list at the mirrored place.  Keeps the 32
// best of both, best first (the better one of each mirrored pair, then the last merge of a bitonic sort).
__device__ __forceinline__ void merge_mirrored(Cand& c, float ov, int oi, int lane) {
  if (better(ov, oi, c.v, c.i)) { c.v = ov; c.i = oi; }
  sort_stage<kWave, 16>(c, lane); sort_stage<kWave, 8>(c, lane); sort_stage<kWave, 4>(c, lane);
  sort_stage<kWave, 2>(c, lane); sort_stage<kWave, 1>(c, lane);
}
// The k best (k <= 32) of `lists` <= 32 lists of k candidates load(list, position), by a block of four waves; lanes
// 0..k-1 of wave 0 end up with them, best first (s_v, s_i: LDS, 128 entries).  All candidates are requested at once,
// each half-wave sorts its up to four lists (15 stages) and merges them (6 each), then the halves and the waves meet:
// 15 + 6 stages per list after the first, 18 more for the meeting: 75 for 20 lists, 96 for 32, where one wave sorting 64
// candidates per pass needs 42 for every 64 (400 candidates: 294).  Beam tail of 24 sentences, beam 20: 44 -> 15 us, half of it the sentence's state and embedding.
template <typename F> __device__ __forceinline__ Cand block_topk(F load, int lists, int k, int tid, float* s_v, int* s_i) {
  const int lane = tid & 63, wid = tid >> 6, half = lane >> 5, pos = lane & 31;
  Cand l[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int list = u * 8 + wid * 2 + half;
    l[u] = {-INFINITY, kNone};
    if (list < lists && pos < k) l[u] = load(list, pos);
  }
  Cand c = l[0];
  wave_sort<32>(c, lane);
#pragma unroll
  for (int u = 1; u < 4; ++u)
    if (u * 8 < lists) {   // uniform
      wave_sort<32>(l[u], lane);
      merge_mirrored(c, __shfl_xor(l[u].v, 31, kWave), __shfl_xor(l[u].i, 31, kWave), lane);
    }
  merge_mirrored(c, __shfl_xor(c.v, 63, kWave), __shfl_xor(c.i, 63, kWave), lane);   // both halves: the same 32 best
  if (half == 0) { s_v[wid * 32 + pos] = c.v; s_i[wid * 32 + pos] = c.i; }
  __syncthreads();
  if (wid != 0) return Cand{-INFINITY, kNone};
  c = {s_v[half * 32 + pos], s_i[half * 32 + pos]};
  merge_mirrored(c, s_v[(half + 2) * 32 + 31 - pos], s_i[(half + 2) * 32 + 31 - pos], lane);
  merge_mirrored(c, __shfl_xor(c.v, 63, kWave), __shfl_xor(c.i, 63, kWave), lane);
  return c;
}

// (max, sum of exp(x - max)) pairs combine associatively
__device__ __forceinline__ void lse_merge(float& m, float& s, float om, float os) {
  const float M = fmaxf(m, om);
  if (M == -INFINITY) { s = 0.f; return; }
  s = s * expf(m - M) + os * expf(om - M);
  m = M;
}

}  // namespace san
