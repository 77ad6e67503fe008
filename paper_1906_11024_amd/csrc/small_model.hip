// Small fp32 models: a decoder step, or a whole stretch of beam search, with one workgroup per sentence.
//
// A step of a small model is a chain of launches that each cost 2 to 5 us whatever they compute.  Hypotheses of different
// sentences never meet, so a workgroup can take its sentence through every layer, the output layer and the beam step with
// barriers of its own between them, and through the next step too: nothing has to be synchronised across the chip.  It
// reads all of the model's weights itself, 0.7 MB of them out of L2 at 64 bytes a cycle (4.6 us), which is why the model
// has to be small (small_model_faster in rules.h has the line and both sides' times).  What bounds it is latency: some 25
// phases a step of a round trip to L2, a few dependent reductions and a barrier each.  So a product's first weights are
// requested in front of the barrier that ends the phase before it, a lane keeps them for all of the sentence's rows, sums
// over lanes are dealt out as they are formed (one epilogue a lane, not one a value), and heads of several rows go through
// sixteen lanes each, four side by side.
// Two sentences, 2 layers of 64 columns, 1000 words, a step of the loop (us, launches / here): beam 1 70 / 21, beam 4
// 73 / 32, beam 8 78 / 44; 64 sentences of beam 4 79 / 34.  Tried: the next product's weights kept in registers across a
// phase (spills: 28 us at beam 1); beams of more than 8 (92 / 210 at beam 20: rows of a sentence are sequential here).
#include <atomic>
#include <type_traits>

#include "beam_sort.h"
#include "common.h"
#include "kernels.h"

namespace san {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSmThreads = 512, kSmWaves = kSmThreads / kWave;

// LDS traffic inside one wave: its own writes are read back by other lanes
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Sums of NV values over groups of LPC lanes, dealt out: v[i] of lane q becomes the sum of value i + first, where `first`
// is returned (NV / LPC values a lane, or one where there are fewer values than lanes; then only lanes with
// q < NV keep one each).
template <int LPC, int NV, int M = 1> __device__ __forceinline__ int deal_sums(float (&v)[NV], int q) {
  if constexpr (M < LPC) {
    constexpr int live = NV / M;   // values a lane still holds
    if constexpr (live > 1) {
      constexpr int half = live / 2;
      const bool up = (q & M) != 0;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        const float keep = up ? v[i + half] : v[i], send = up ? v[i] : v[i + half];
        v[i] = keep + __uint_as_float(lane_xor<M>(__float_as_uint(send)));
      }
      return (up ? half : 0) + deal_sums<LPC, NV, M * 2>(v, q);
    } else {
      v[0] += __uint_as_float(lane_xor<M>(__float_as_uint(v[0])));
      return deal_sums<LPC, NV, M * 2>(v, q);
    }
  }
  return 0;
}

// The weights a lane holds of one pass of a product (k = 4 LPC U): C columns, U times four k-values of each.  LPC lanes
// share a column (consecutive lanes read consecutive 16 bytes of a weight row).
template <int LPC, int U, int C> struct SmWeights { f32x4 w[C][U]; float b[C]; };
template <int LPC, int U, int C>
__device__ __forceinline__ SmWeights<LPC, U, C> request(const float* W, const float* bias, int N, int n0) {
  SmWeights<LPC, U, C> o;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // the offsets of one product are not kept in registers through all the others
  const int q = tid % LPC, g = tid / LPC;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int n = min(n0 + g + (kSmThreads / LPC) * c, N - 1);
    const unsigned at = (unsigned)(n * (4 * LPC * U) + 4 * q) * 4u;   // a uniform base and 32 bits of offset
#pragma unroll
    for (int u = 0; u < U; ++u) o.w[c][u] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(W) + (at + u * 16 * LPC));
    o.b[c] = bias ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(bias) + (unsigned)n * 4u) : 0.f;
  }
  return o;
}
// epi(r, n, sum_k xs[r][k] W[n][k] + bias[n]) for r < R, n < N.  The first weights are requested in front of the barrier
// that waits for the rows, every pass's in front of the one before it.
template <int RB, int LPC, int U, int C, typename Epi>
__device__ __forceinline__ void product(const float* xs, const float* W, const float* bias, int N, int R, Epi epi) {
  constexpr int G = kSmThreads / LPC, K = 4 * LPC * U, NV = RB * C;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int q = tid % LPC, g = tid / LPC;
  SmWeights<LPC, U, C> cur = request<LPC, U, C>(W, bias, N, 0);
  __syncthreads();   // the rows are there
  for (int n0 = 0; n0 < N; n0 += G * C) {
    SmWeights<LPC, U, C> nx;
    if (n0 + G * C < N) nx = request<LPC, U, C>(W, bias, N, n0 + G * C);
    if (n0 + (tid & ~(kWave - 1)) / LPC < N) {   // uniform in a wave: it has a column
      for (int r0 = 0; r0 < R; r0 += RB) {
        float acc[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(xs + min(r0 + r, R - 1) * K + 4 * (q + LPC * u));
#pragma unroll
            for (int c = 0; c < C; ++c) {
              float& o = acc[r * C + c];
              o = fmaf(x.x, cur.w[c][u].x, o);
              o = fmaf(x.y, cur.w[c][u].y, o);
              o = fmaf(x.z, cur.w[c][u].z, o);
              o = fmaf(x.w, cur.w[c][u].w, o);
            }
          }
        const int first = deal_sums<LPC, NV>(acc, q);
        if (NV >= LPC || q < NV) {
#pragma unroll
          for (int i = 0; i < (NV > LPC ? NV / LPC : 1); ++i) {
            const int r = r0 + (first + i) / C, c = (first + i) % C, n = n0 + g + G * c;
            float bv = cur.b[0];
#pragma unroll
            for (int k = 1; k < C; ++k) bv = c == k ? cur.b[k] : bv;
            if (r < R && n < N) epi(r, n, acc[i] + bv);
          }
        }
      }
    }
    cur = nx;
  }
}
// the same where k is the feed-forward width
template <int RB, typename Epi>
__device__ __forceinline__ void product_f(const float* xs, int F, const float* W, const float* bias, int N, int R, Epi epi) {
  constexpr int C = RB == 1 ? 2 : 4;
  if (F == 64) product<RB, 16, 1, C>(xs, W, bias, N, R, epi);
  else if (F == 128) product<RB, 16, 2, C>(xs, W, bias, N, R, epi);
  else if (F == 256) product<RB, 16, 4, C>(xs, W, bias, N, R, epi);
  else product<RB, 32, 4, C>(xs, W, bias, N, R, epi);
}

template <int LANES> __device__ __forceinline__ float lanes_max(float v) {
  v = group_max<16>(v);
  return LANES == 64 ? max_xor32(max_xor16(v)) : v;
}
// One head's attention of one query by LANES lanes: out[0 .. dh) = softmax(q K^T scale) V over n positions (Eq. 1, 2), key
// j at K + at(j), or with the weights S read instead (Eq. 4).  S (optional): the weights go there too.  p: n floats of LDS.
template <int LANES, typename At>
__device__ __forceinline__ void attend(const float* q, const float* K, const float* V, At at, int n, int dh, float scale,
                                       bool apply, float* S, float* p, float* out) {
  int lane = threadIdx.x & (LANES - 1);
  asm volatile("" : "+v"(lane));
  float inv = 1.f;
  if (!apply) {
    float m = -INFINITY;
    for (int j = lane; j < n; j += LANES) {
      const float* k = K + at(j);
      float s = 0.f;
      for (int c = 0; c < dh; c += 16) {
        f32x4 kv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kv[i] = *reinterpret_cast<const f32x4*>(k + c + 4 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 qv = *reinterpret_cast<const f32x4*>(q + c + 4 * i);
          s = fmaf(qv.x, kv[i].x, s); s = fmaf(qv.y, kv[i].y, s); s = fmaf(qv.z, kv[i].z, s); s = fmaf(qv.w, kv[i].w, s);
        }
      }
      s *= scale;
      p[j] = s;
      m = fmaxf(m, s);
    }
    m = lanes_max<LANES>(m);
    float l = 0.f;
    for (int j = lane; j < n; j += LANES) {   // a lane's own entries
      const float e = p[j] == -INFINITY ? 0.f : expf(p[j] - m);
      p[j] = e;
      l += e;
    }
    l = group_sum<16>(l);
    if (LANES == 64) l = sum_xor32(sum_xor16(l));
    inv = l > 0.f ? 1.f / l : 0.f;   // no position, or none with a score above -inf: zero
    if (S)
      for (int j = lane; j < n; j += LANES) S[j] = p[j] * inv;
  } else {
    for (int j = lane; j < n; j += LANES) p[j] = S[j];
  }
  wave_sync();
  const int per = dh / 4, c4 = (lane % per) * 4;   // `per` lanes cover one position's channels
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int j = lane / per; j < n; j += LANES / per) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(V + at(j) + c4);
    const float w = p[j];
    acc.x = fmaf(w, v.x, acc.x); acc.y = fmaf(w, v.y, acc.y); acc.z = fmaf(w, v.z, acc.z); acc.w = fmaf(w, v.w, acc.w);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v = acc[i];
    if (per <= 4) v += dpp_mov<0x124>(v);    // rotations of the 16-lane row reach the other positions' lanes
    if (per <= 8) v += dpp_mov<0x128>(v);
    if (LANES == 64) {
      if (per <= 16) v = sum_xor16(v);
      v = sum_xor32(v);
    }
    acc[i] = v;
  }
  if (lane < per) *reinterpret_cast<f32x4*>(out + c4) = f32x4{acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
  wave_sync();   // p is free again
}
// Few (row, head) pairs: a wave for each.  Many, and short enough histories: sixteen lanes, four pairs of a wave side by
// side, so that their round trips to memory overlap.
__host__ __device__ inline bool small_pairs16(int R, int H, int dh, int Tm) { return R * H > kSmWaves && dh <= 64 && Tm <= 256; }

// x[r] = LayerNorm(y[r]): a wave per row, d = 64 or 128
struct SmNorm { float g0, b0, g1, b1; };
__device__ __forceinline__ SmNorm request_norm(const float* g, const float* b, int d) {
  const int lane = threadIdx.x & 63, hi = d > kWave ? kWave : 0;
  return SmNorm{g[lane], b[lane], g[lane + hi], b[lane + hi]};
}
__device__ __forceinline__ void norm_rows(const float* y, float* x, const SmNorm& w, int d, int R, float eps) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const bool two = d > kWave;
  const float rd = 1.f / (float)d;
  __syncthreads();   // y is there
  for (int r = wid; r < R; r += kSmWaves) {
    const float v0 = y[r * d + lane], v1 = two ? y[r * d + kWave + lane] : 0.f;
    const float mean = wave_sum(v0 + v1) * rd;
    const float d0 = v0 - mean, d1 = two ? v1 - mean : 0.f;
    const float rs = rsqrtf(wave_sum(d0 * d0 + d1 * d1) * rd + eps);
    x[r * d + lane] = d0 * rs * w.g0 + w.b0;
    if (two) x[r * d + kWave + lane] = d1 * rs * w.g1 + w.b1;
  }
}

// Part `part` of `parts` of one row's scores (words part * 64 + lane, every 64 * parts), by one wave: the maximum and the sum
// of exp(x - maximum) to stat[0], stat[1], its k best words to cv / ci (empty slots: -inf, kNone).
// Threshold: the k-th largest distinct one of the lanes' maxima, so that at least k words reach it; those that do are listed (list_v,
// list_i: 64 entries of LDS) and sorted.  More than 64 of them (equal scores in masses, or fewer than k lanes with words):
// k rounds, each taking the best word after the previous pick.
__device__ __forceinline__ void best_words(const float* row, int V, int part, int parts, int k, float* stat, float* cv, int* ci,
                                           float* list_v, int* list_i) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int first = part * 64 + lane, step = 64 * parts;
  float lm = -INFINITY;
  for (int i = first; i < V; i += step) lm = fmaxf(lm, row[i]);
  const float m = wave_max(lm);
  float s = 0.f;
  for (int i = first; i < V; i += step) s += row[i] == -INFINITY ? 0.f : __expf(row[i] - m);
  s = wave_sum(s);
  if (lane == 0) { stat[0] = m; stat[1] = s; }
  float thr = m;
  for (int round = 1; round < k; ++round) thr = wave_max(lm < thr ? lm : -INFINITY);
  int n = 0;
  for (int i0 = part * 64; i0 < V; i0 += step) {
    const float v = i0 + lane < V ? row[i0 + lane] : -INFINITY;
    const bool take = i0 + lane < V && v >= thr;
    const unsigned long long who = __ballot(take);
    const int at = n + __builtin_amdgcn_mbcnt_hi((unsigned)(who >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)who, 0));
    if (take && at < 64) { list_v[at] = v; list_i[at] = i0 + lane; }
    n += __popcll(who);
  }
  wave_sync();
  if (n >= 1 && n <= 64) {
    Cand c = {-INFINITY, kNone};
    if (lane < n) c = Cand{list_v[lane], list_i[lane]};
    if (n <= 16) wave_sort<16>(c, lane);
    else wave_sort<kWave>(c, lane);
    if (lane < k) { cv[lane] = c.v; ci[lane] = c.i; }
    wave_sync();
    return;
  }
  float pv = INFINITY;
  int pi = -1;
  for (int round = 0; round < k; ++round) {
    Cand best = {-INFINITY, kNone};
    for (int i = first; i < V; i += step) {
      const float v = row[i];
      const bool after = v < pv || (v == pv && i > pi);
      if (after && better(v, i, best.v, best.i)) best = Cand{v, i};
    }
    wave_sort<kWave>(best, lane);
    if (lane == 0) { cv[round] = best.v; ci[round] = best.i; }
    pv = __shfl(best.v, 0, kWave);
    pi = __shfl(best.i, 0, kWave);
  }
}
// parts a row's words are dealt to: all waves have work where the rows are few
__host__ __device__ inline int small_parts(int R) { return R == 1 ? 8 : R == 2 ? 4 : R <= 4 ? 2 : 1; }

// The workgroup's LDS, in floats (k = beam)
struct SmLds {
  int x, y, a, actx, q, h, p, anc, cand_v, cand_i, stat, list_v, list_i, tok, par, cum, lse, lg, total;
};
__host__ __device__ inline SmLds small_lds(int d, int F, int H, int R, int T, int max_src, int lg_words) {
  SmLds l;
  int o = 0;
  auto take = [&](int n) { const int at = o; o += (n + 3) / 4 * 4; return at; };
  l.x = take(R * d); l.y = take(R * d); l.a = take(R * d); l.actx = take(R * d); l.q = take(R * d);
  l.h = take(R * F);
  const int Tm = T > max_src ? T : max_src;
  l.p = take((small_pairs16(R, H, d / H, Tm) ? 4 : 1) * kSmWaves * Tm);
  l.anc = take(2 * R * T);
  const int lists = lg_words ? R * small_parts(R) : 0;
  l.cand_v = take(lists * R); l.cand_i = take(lists * R); l.stat = take(lists * 2);
  l.list_v = take(kSmWaves * 64); l.list_i = take(kSmWaves * 64);
  l.tok = take(R); l.par = take(R); l.cum = take(R); l.lse = take(R);
  l.lg = take(lg_words);
  l.total = o;
  return l;
}

template <int LD, int RB>
__global__ __launch_bounds__(kSmThreads) void small_decode_kernel(SmallDecode P) {
  extern __shared__ __align__(16) float lds[];
  constexpr int d = LD * 16;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int b = blockIdx.x, R = P.beam, F = P.F, V = P.V, H = P.H, dh = d / H, T = P.T, row0 = b * R;
  const bool search = P.logits == nullptr;
  const SmLds l = small_lds(d, F, H, R, T, P.max_src_cap, search ? R * V : 0);
  float* const x = lds + l.x;
  float* const y = lds + l.y;
  float* const a = lds + l.a;
  float* const actx = lds + l.actx;
  float* const q = lds + l.q;
  float* const h = lds + l.h;
  const int Tm = max(T, P.max_src_cap);
  const bool pairs16 = small_pairs16(R, H, dh, Tm);
  float* const p = lds + l.p + (pairs16 ? tid >> 4 : wid) * Tm;
  int* anc = reinterpret_cast<int*>(lds + l.anc);
  int* anc_next = anc + R * T;
  float* const cand_v = lds + l.cand_v;
  int* const cand_i = reinterpret_cast<int*>(lds + l.cand_i);
  int* const tok = reinterpret_cast<int*>(lds + l.tok);
  int* const par = reinterpret_cast<int*>(lds + l.par);
  float* const cum = lds + l.cum;
  float* const stat = lds + l.stat;
  float* const list_v = lds + l.list_v;
  int* const list_i = reinterpret_cast<int*>(lds + l.list_i);
  float* const lse = lds + l.lse;
  float* const lg = lds + l.lg;

  const int t0 = *P.t_dev;
  const int n_src = max(0, min(P.src_len[b], P.max_src));
  const size_t mem0 = (size_t)(P.group_map ? P.group_map[b] : b) * P.max_src;
  for (int i = tid; i < R * t0; i += kSmThreads) anc[i / t0 * T + i % t0] = P.anc[(size_t)(row0 + i / t0) * T + i % t0];
  if (tid < R) {
    tok[tid] = P.tok_in[row0 + tid];
    cum[tid] = search ? P.cum_in[row0 + tid] : 0.f;
  }
  bool done = search && P.eos >= 0 && P.done[b] != 0;
  // products of d inputs: many outputs, or d
  const auto wide = [&](const float* xs, const float* W, const float* bias, int N, auto epi) {
    if constexpr (RB == 1) product<1, LD, 4, 2>(xs, W, bias, N, R, epi);
    else product<RB, 2 * LD, 2, 4>(xs, W, bias, N, R, epi);
  };
  const auto narrow = [&](const float* xs, const float* W, const float* bias, auto epi) {
    if constexpr (RB == 1) product<1, LD, 4, LD / 4>(xs, W, bias, d, R, epi);
    else product<RB, 16, LD / 4, 4>(xs, W, bias, d, R, epi);
  };
  int last_in = 0;                    // the word this thread's row was fed last
  __syncthreads();

  for (int s = 0; s < P.steps; ++s) {
    const int t = t0 + s;
    const float* pe = P.pe + (size_t)t * d;
    for (int i = tid; i < R * (d / 4); i += kSmThreads) {
      const int r = i / (d / 4), c = (i % (d / 4)) * 4;
      const f32x4 e = *reinterpret_cast<const f32x4*>(P.emb + (size_t)min(max(tok[r], 0), V - 1) * d + c);
      const f32x4 o = *reinterpret_cast<const f32x4*>(pe + c);
      *reinterpret_cast<f32x4*>(x + r * d + c) = f32x4{fmaf(e.x, P.emb_scale, o.x), fmaf(e.y, P.emb_scale, o.y),
                                                       fmaf(e.z, P.emb_scale, o.z), fmaf(e.w, P.emb_scale, o.w)};
    }
    if (tid < R) {
      anc[tid * T + t] = row0 + tid;
      last_in = tok[tid];
    }
    const size_t slot = ((size_t)t * P.cache_rows + row0) * d;   // this position's cache entries
    for (int n = 0; n < P.n_layers; ++n) {
      const SmallLayer& L = P.layers[n];
      const auto to_y = [&](int r, int c, float v) { y[r * d + c] = v + x[r * d + c]; };
      // runs attention(pair's row, head, lanes) over the workgroup
      const auto pairs = [&](auto one) {
        __syncthreads();
        if (pairs16) for (int i = tid >> 4; i < R * H; i += kSmThreads / 16) one(i / H, i % H, std::integral_constant<int, 16>{});
        else for (int i = wid; i < R * H; i += kSmWaves) one(i / H, i % H, std::integral_constant<int, 64>{});
      };
      // ---- self-attention
      if (L.self_head) {
        float *const Kc = L.Kc + slot, *const Vc = L.Vc + slot;
        wide(x, L.w_self, L.b_self, 3 * d, [&](int r, int c, float v) {
          float* const o = c < d ? q : c < 2 * d ? Kc - d : Vc - 2 * d;
          o[r * d + c] = v;
        });
      } else {
        float* const Vc = L.Vc + slot;
        narrow(x, L.w_self, L.b_self, [&](int r, int c, float v) { Vc[r * d + c] = v; });
      }
      const SmNorm n1 = request_norm(L.ln1g, L.ln1b, d);
      pairs([&](int r, int hd, auto lanes) {
        const int* const ar = anc + r * T;
        float* const S = L.S_self ? L.S_self + ((size_t)(row0 + r) * H + hd) * T : nullptr;
        attend<lanes.value>(q + r * d + hd * dh, L.Kc + hd * dh, L.Vc + hd * dh,
               [&](int j) { return ((size_t)j * P.cache_rows + ar[j]) * d; }, t + 1, dh, P.scale, !L.self_head, S, p, a + r * d + hd * dh);
      });
      narrow(a, L.wo, L.bo, to_y);
      const SmNorm n2 = request_norm(L.ln2g, L.ln2b, d);
      norm_rows(y, x, n1, d, R, P.eps);
      // ---- encoder-decoder attention: a block's followers reuse the head's A (actx), or its weights (S_ctx)
      if (L.ctx_head)
        narrow(x, L.wq_c, L.bq_c, [&](int r, int c, float v) { q[r * d + c] = v; });
      if (L.ctx_head || L.ctx_ld == d)
        pairs([&](int r, int hd, auto lanes) {
          float* const S = L.S_ctx ? L.S_ctx + ((size_t)(row0 + r) * H + hd) * P.max_src_cap : nullptr;
          attend<lanes.value>(q + r * d + hd * dh, L.mem_k + hd * dh, L.mem_v + hd * dh,
                 [&](int j) { return (mem0 + j) * L.ctx_ld; }, n_src, dh, P.scale, !L.ctx_head, S, p, actx + r * d + hd * dh);
          if (L.dbg_hidden && L.ctx_head)   // copies for inspection: zeros past the sentence
            for (int j = n_src + (tid & (lanes.value - 1)); j < P.max_src; j += lanes.value) S[j] = 0.f;
        });
      narrow(actx, L.wo_c, L.bo_c, to_y);
      const SmNorm n3 = request_norm(L.ln3g, L.ln3b, d);
      norm_rows(y, x, n2, d, R, P.eps);
      // ---- feed-forward
      wide(x, L.w1, L.b1, F, [&](int r, int c, float v) { h[r * F + c] = fmaxf(v, 0.f); });
      product_f<RB>(h, F, L.w2, L.b2, d, R, to_y);
      norm_rows(y, x, n3, d, R, P.eps);
      if (L.dbg_hidden) {   // copies for inspection
        __syncthreads();
        for (int i = tid; i < R * d; i += kSmThreads) {
          L.dbg_A_self[(size_t)row0 * d + i] = a[i];
          L.dbg_A_ctx[(size_t)row0 * d + i] = actx[i];
          L.dbg_hidden[(size_t)row0 * d + i] = x[i];
        }
      }
    }
    if (!search) {
      float* const out = P.logits + (size_t)row0 * V;
      wide(x, P.w_out, nullptr, V, [&](int r, int c, float v) { out[(size_t)r * V + c] = v; });
      if (tid < R) {
        P.last_tok[row0 + tid] = last_in;
        P.anc[(size_t)(row0 + tid) * T + t] = row0 + tid;
      }
      break;
    }
    wide(x, P.w_out, nullptr, V, [&](int r, int c, float v) { lg[r * V + c] = v; });
    __syncthreads();
    // ---- the k = beam best words of every row (in parts), then of the sentence
    const int parts = small_parts(R), lists = R * parts;
    for (int i = wid; i < lists; i += kSmWaves)
      best_words(lg + i / parts * V, V, i % parts, parts, R, stat + 2 * i, cand_v + i * R, cand_i + i * R, list_v + wid * 64, list_i + wid * 64);
    __syncthreads();
    if (tid < R) {
      float m = stat[2 * tid * parts], s_ = stat[2 * tid * parts + 1];
      for (int i = 1; i < parts; ++i) lse_merge(m, s_, stat[2 * (tid * parts + i)], stat[2 * (tid * parts + i) + 1]);
      lse[tid] = m + logf(s_);
    }
    // The parts hold more than the row's R best words.  The others must not win a tie by their lower index where the score before
    // swallows what sets words apart: all of it in a dead row's -inf, or -1e9.  Beside the sums above: 0.1 us a step for one or
    // two rows (eight or four parts) and 0.4 for three or four (two parts), 0.6 to 0.9 in the merge below or with eight
    // comparisons here for the latter too.
    if constexpr (RB < 4) {
      if (wid == 1 && lane < 8 * R) {
        const int first = lane & ~7;   // a row's words
        const float v = cand_v[lane];
        const int id = cand_i[lane];
        Cand c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = Cand{cand_v[first + i], cand_i[first + i]};
        int ahead = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) ahead += better(c[i].v, c[i].i, v, id);
        wave_sync();   // all of them have been read
        if (ahead >= R) cand_i[lane] = kNone;
      }
    } else if (parts == 2 && wid == 1 && lane < 2 * R * R) {
      // j words of its own part and, if this one of the other is, R - j of that are better
      const int list = R == 3 ? lane / 3 : lane / 4, o = ((list ^ 1) + list + 1) * R - 1 - lane;
      const bool out = better(cand_v[o], cand_i[o], cand_v[lane], cand_i[lane]);
      wave_sync();   // all of them have been read
      if (out) cand_i[lane] = kNone;
    }
    __syncthreads();
    {
      // a finished hypothesis can only be extended by the end symbol, at cost 0; an empty slot, or a score that is no
      // number, never wins
      const auto load = [&](int list, int j) {
        const int r = list / parts;
        float lp = cand_v[list * R + j] - lse[r];
        int id = cand_i[list * R + j];
        if (P.eos >= 0 && tok[r] == P.eos) {
          lp = j == 0 ? 0.f : -INFINITY;
          id = list % parts != 0 ? kNone : j == 0 ? P.eos : (j - 1 < P.eos ? j - 1 : j);
        }
        const float sc = cum[r] + lp;
        return id == kNone || !(sc == sc) ? Cand{-INFINITY, kNone} : Cand{sc, r * V + id};
      };
      Cand best = {-INFINITY, kNone};
      if (wid == 0) best = wave_topk([&](int q) { return load(q / R, q % R); }, lists * R, R, lane);
      __syncthreads();
      if (tid < R) {
        const bool ok = best.i != kNone;
        tok[tid] = ok ? best.i % V : 0;
        par[tid] = ok ? best.i / V : -1;   // -1: an empty slot
        cum[tid] = ok ? best.v : -INFINITY;
        const int to = P.row_map ? P.row_map[row0 + tid] : row0 + tid, from = row0 + max(par[tid], 0);
        const size_t o = (size_t)(P.step0 + s) * P.out_ld + to;
        P.out_tok[o] = tok[tid];
        P.out_par[o] = P.row_map ? P.row_map[from] : from;
      }
      __syncthreads();
    }
    if (P.eos >= 0 && wid == 0) {   // finished once every hypothesis kept ends in the end symbol; counted once
      const bool open = lane < R && (par[min(lane, R - 1)] < 0 || tok[min(lane, R - 1)] != P.eos);
      if (__ballot(open) == 0 && !done) {
        done = true;
        if (lane == 0) {
          P.done[b] = 1;
          atomicAdd(P.done_count, 1);
        }
      }
    }
    // row r of the ancestry table continues row par[r]
    if (R > 1) {
      for (int j = tid; j <= t; j += kSmThreads)
        for (int r = 0; r < R; ++r) anc_next[r * T + j] = anc[max(par[r], 0) * T + j];
      int* const swap = anc;
      anc = anc_next;
      anc_next = swap;
    }
    __syncthreads();
  }
  if (search) {
    const int t1 = t0 + P.steps;
    for (int i = tid; i < R * t1; i += kSmThreads) P.anc[(size_t)(row0 + i / t1) * T + i % t1] = anc[i / t1 * T + i % t1];
    if (tid < R) {
      P.tok_out[row0 + tid] = tok[tid];
      P.cum_out[row0 + tid] = cum[tid];
      P.last_tok[row0 + tid] = P.feed_last && t1 < T ? tok[tid] : last_in;
      if (P.feed_last && t1 < T) P.anc[(size_t)(row0 + tid) * T + t1] = row0 + tid;
    }
  }
  // the step counter moves once every workgroup has read it
  if (tid == 0 && __hip_atomic_fetch_add(P.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1) {
    *P.ticket = 0;
    *P.t_dev = t0 + P.steps;
  }
}

size_t small_decode_lds(const SmallDecode& P) {
  return (size_t)small_lds(P.d, P.F, P.H, P.beam, P.T, P.max_src_cap, P.logits ? 0 : P.beam * P.V).total * 4;
}

template <int LD, int RB> static hipError_t launch_small(const SmallDecode& P, int batch, size_t smem, hipStream_t stream) {
  if (smem > 64 * 1024) {
    static std::atomic<unsigned long long> raised{0};   // bit = device ordinal
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&small_decode_kernel<LD, RB>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
      raised.fetch_or(bit, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL((small_decode_kernel<LD, RB>), dim3(batch), dim3(kSmThreads), smem, stream, P);
  return hipGetLastError();
}
hipError_t launch_small_decode(const SmallDecode& P, int batch, hipStream_t stream) {
  const size_t smem = small_decode_lds(P);
  if ((P.d != 64 && P.d != 128) || (P.F != 64 && P.F != 128 && P.F != 256 && P.F != 512) || P.beam < 1 || P.beam > kSmallBeam || P.H < 1 ||
      P.d % P.H || smem > 160 * 1024 || P.steps < 1 || (P.logits && P.steps != 1) || batch < 1)
    return hipErrorInvalidValue;
  const int dh = P.d / P.H;
  if (dh != 16 && dh != 32 && dh != 64 && dh != 128) return hipErrorInvalidValue;
#define SAN_SMALL(LD_) \
  (P.beam == 1 ? launch_small<LD_, 1>(P, batch, smem, stream) : P.beam == 2 ? launch_small<LD_, 2>(P, batch, smem, stream) : launch_small<LD_, 4>(P, batch, smem, stream))
  return P.d == 64 ? SAN_SMALL(4) : SAN_SMALL(8);
#undef SAN_SMALL
}

}  // namespace san
