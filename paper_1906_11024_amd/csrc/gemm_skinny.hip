// Projections of few rows (M <= 16: one sentence with its beam, a handful of greedy sentences).
//
// Bound: such a product is one pass over the weights (1-8 MB at the paper's sizes, in the Infinity Cache from step to
// step) behind a launch; a 64-wide tile kernel spends its time on the staging of rows that are not there and leaves
// most CUs without a block.  Here a block of eight waves owns 16 * NB output columns and deals the k range to its
// waves; a wave requests all its weights (up to 16 loads of 16 bytes a lane) before anything else, straight into the
// registers that feed the 16-row MFMA, with no LDS stage, and the eight partial tiles meet in LDS once, in wave order.
// NV > 0: the rows are the LayerNorm of a preceding product (split-K partials + bias + residual, one or two stages as
// in ln_reduce_kernel).  Every block normalises them itself while its weights travel, so the LayerNorm costs no launch of
// its own; block 0 also stores them, as the residual of the next sub-layer.  Every block reads all their partials (4 rows
// of 512 columns in four splits: 40 KB; 12 rows 120 KB), each wave its share of the rows one after the other, so this
// pays for few and narrow rows only: few_rows_faster.
// Measured (one sentence, beam 4, 4 rows; us per decoder step): fp32, 6 layers of 512: 276 -> 223; bf16, 6 layers of
// 1024: 245 -> 231.  Per launch (kernel trace): the product alone 5.4 where the tile kernel took 7.2-8.1, with its
// LayerNorm 6.1-7.5 against 3.8 + 7.5; what is left is launch, argument fetch, one trip to the Infinity Cache for the
// weights, the reduction through LDS.  (Prologue in the output layer too: 20.5 against 17.4 + 3.2, its blocks want the
// registers for weights; at 1024 columns it then spilled and took 44.)
#include <algorithm>
#include <atomic>

#include "candidates.h"
#include "common.h"
#include "kernels.h"

namespace san {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSkWaves = 8;
constexpr int kUnit = 64;   // bytes of k per row and load instruction: 16 columns x 64 bytes

// acc[m][n] += x-rows W-rows^T over one unit.  A lane holds 16 bytes of row lane % 16 at byte 16 * (lane / 16) of
// the unit, on both sides; which k-values meet in one instruction does not matter as both operands agree on it.
template <typename T> __device__ __forceinline__ void mma_unit(f32x4& acc, const u32x4& x, const u32x4& w);
template <> __device__ __forceinline__ void mma_unit<float>(f32x4& acc, const u32x4& x, const u32x4& w) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.x), __uint_as_float(w.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.y), __uint_as_float(w.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.z), __uint_as_float(w.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.w), __uint_as_float(w.w), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ void mma_unit<bf16_t>(f32x4& acc, const u32x4& x, const u32x4& w) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, w), acc, 0, 0, 0);
}

// LayerNorm of a row held by one wave, NV float4 per lane (lanes past the row are inactive)
template <int NV>
__device__ __forceinline__ void wave_layer_norm(float4 (&v)[NV], const bool (&act)[NV], int d, const float4 (&g)[NV],
                                                const float4 (&b)[NV], float eps) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) s += act[i] ? (v[i].x + v[i].y) + (v[i].z + v[i].w) : 0.f;
  const float mean = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (act[i]) {
      const float d0 = v[i].x - mean, d1 = v[i].y - mean, d2 = v[i].z - mean, d3 = v[i].w - mean;
      q += fmaf(d0, d0, fmaf(d1, d1, fmaf(d2, d2, d3 * d3)));
    }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < NV; ++i)
    v[i] = make_float4((v[i].x - mean) * rstd * g[i].x + b[i].x, (v[i].y - mean) * rstd * g[i].y + b[i].y,
                       (v[i].z - mean) * rstd * g[i].z + b[i].z, (v[i].w - mean) * rstd * g[i].w + b[i].w);
}

// v += the partials of one row, in split order; all NS are requested (absent ones re-read the first and are dropped),
// so that nothing is loaded behind a branch
template <int NV, int NS> struct Partials {
  float4 t[NS][NV];
  __device__ __forceinline__ void request(const float* part, int nsplit, size_t stride, const int (&col)[NV]) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int i = 0; i < NV; ++i) t[s][i] = *reinterpret_cast<const float4*>(part + (s < nsplit ? s * stride : 0) + col[i]);
  }
  __device__ __forceinline__ void add(float4 (&v)[NV], int nsplit) const {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float4 a = t[0][i];
#pragma unroll
      for (int s = 1; s < NS; ++s)
        if (s < nsplit) { a.x += t[s][i].x; a.y += t[s][i].y; a.z += t[s][i].z; a.w += t[s][i].w; }
      v[i] = make_float4(v[i].x + a.x, v[i].y + a.y, v[i].z + a.z, v[i].w + a.w);
    }
  }
};

template <typename T, int NB, int NV, bool S2, bool CAND>
__global__ __launch_bounds__(kSkWaves * 64) void skinny_kernel(GemmParams p, LnInput ln) {
  constexpr int U = NB == 1 ? 8 : 4;                 // units in flight per wave
  constexpr int BN = 16 * NB;
  constexpr int NT = kSkWaves * 64;
  constexpr int RED = kSkWaves * NB * 256;           // fp32 words of the eight partial tiles
  constexpr int NE = (NB * 256 + NT - 1) / NT;       // result elements per thread
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int n0 = blockIdx.x * BN;
  const int t_step = p.t_dev ? *p.t_dev : 0;

  // this wave's units of the block's k range; requests past it re-read the row's last unit and are not used
  const int nu_row = p.K * (int)sizeof(T) / kUnit;
  const int nu_blk = nu_row / p.ksplit;              // the launcher's ksplit divides
  const int u_blk = blockIdx.y * nu_blk;
  const int u_begin = u_blk + nu_blk * wid / kSkWaves, u_end = u_blk + nu_blk * (wid + 1) / kSkWaves;
  const unsigned char* wp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
    wp[j] = reinterpret_cast<const unsigned char*>(p.W) +
            ((size_t)min(n0 + 16 * j + l16, p.N - 1) * p.K) * sizeof(T) + 16 * kq;
  u32x4 wq[U][NB], xq[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < NB; ++j)
      wq[u][j] = *reinterpret_cast<const u32x4*>(wp[j] + (size_t)min(u_begin + u, nu_row - 1) * kUnit);

  // result elements of this thread (see the reduction below) and their bias
  float bias_v[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = tid + NT * i, n = n0 + (e >> 8) * 16 + (e & 15);
    bias_v[i] = (p.bias && e < NB * 256 && n < p.N) ? to_f32(reinterpret_cast<const T*>(p.bias)[n]) : 0.f;
  }

  const unsigned char* xp;
  if constexpr (NV > 0) {
    const int d = p.K, xs_row = d * (int)sizeof(T) + 16;   // 16 bytes of padding: 16-byte reads of 16 rows cover all banks
    const T* const gamma = reinterpret_cast<const T*>(ln.gamma);
    const T* const beta = reinterpret_cast<const T*>(ln.beta);
    int col[NV];
    bool act[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (lane + 64 * i) * 4;
      act[i] = c < d;
      col[i] = act[i] ? c : 0;
    }
    for (int m = wid; m < p.M; m += kSkWaves) {
      Partials<NV, S2 ? 2 : 4> p1, p2;   // two stages: at most two splits each (registers)
      float4 v[NV], g1[NV], b1[NV], u2[NV], g2[NV], b2[NV];
      p1.request(ln.part + (size_t)m * ln.ldp, ln.nsplit, (size_t)p.M * ln.ldp, col);
      if constexpr (S2) p2.request(ln.s2.part + (size_t)m * ln.s2.ldp, ln.s2.nsplit, (size_t)p.M * ln.s2.ldp, col);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const float4 r = load4(reinterpret_cast<const T*>(ln.res) + (size_t)m * d + col[i]);
        const float4 bi = load4(reinterpret_cast<const T*>(ln.bias) + col[i]);
        v[i] = make_float4(bi.x + r.x, bi.y + r.y, bi.z + r.z, bi.w + r.w);
        g1[i] = load4(gamma + col[i]);
        b1[i] = load4(beta + col[i]);
        if constexpr (S2) {
          u2[i] = load4(reinterpret_cast<const T*>(ln.s2.bias) + col[i]);
          g2[i] = load4(reinterpret_cast<const T*>(ln.s2.gamma) + col[i]);
          b2[i] = load4(reinterpret_cast<const T*>(ln.s2.beta) + col[i]);
        }
      }
      p1.add(v, ln.nsplit);
      wave_layer_norm<NV>(v, act, d, g1, b1, ln.eps);
      if constexpr (S2) {
        p2.add(u2, ln.s2.nsplit);
        // the first LayerNorm's output keeps the rounding to the storage type that it has as a launch of its own
#pragma unroll
        for (int i = 0; i < NV; ++i)
          v[i] = make_float4(to_f32(from_f32<T>(v[i].x)) + u2[i].x, to_f32(from_f32<T>(v[i].y)) + u2[i].y,
                             to_f32(from_f32<T>(v[i].z)) + u2[i].z, to_f32(from_f32<T>(v[i].w)) + u2[i].w);
        wave_layer_norm<NV>(v, act, d, g2, b2, ln.eps);
      }
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (act[i]) {
          store4(reinterpret_cast<T*>(smem + (size_t)m * xs_row) + col[i], v[i]);
          if (ln.x_out && blockIdx.x == 0) store4(reinterpret_cast<T*>(ln.x_out) + (size_t)m * d + col[i], v[i]);
        }
    }
    __syncthreads();
    xp = smem + (size_t)min(l16, p.M - 1) * xs_row + 16 * kq;
  } else {
    xp = reinterpret_cast<const unsigned char*>(p.A) + ((size_t)min(l16, p.M - 1) * p.lda) * sizeof(T) + 16 * kq;
  }

  f32x4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int ub = u_begin; ub < u_end; ub += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) xq[u] = *reinterpret_cast<const u32x4*>(xp + (size_t)min(ub + u, nu_row - 1) * kUnit);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ub + u < u_end) {   // wave-uniform
#pragma unroll
        for (int j = 0; j < NB; ++j) mma_unit<T>(acc[j], xq[u], wq[u][j]);
      }
    if (ub + U < u_end) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          wq[u][j] = *reinterpret_cast<const u32x4*>(wp[j] + (size_t)min(ub + U + u, nu_row - 1) * kUnit);
    }
  }

  // ---- the eight partial tiles, added in wave order.  acc[j][v]: row 4 * (lane / 16) + v, column 16 j + lane % 16.
  float* red = reinterpret_cast<float*>(smem);
  if constexpr (NV > 0) __syncthreads();   // the normalised rows are dead
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wid * NB + j) * 4 + v) * 64 + lane] = acc[j][v];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = tid + NT * i;   // [j][v][lane]
    if (e >= NB * 256) break;
    float val = bias_v[i];
#pragma unroll
    for (int w = 0; w < kSkWaves; ++w) val += red[w * NB * 256 + e];
    const int cl = (e >> 8) * 16 + (e & 15), n = n0 + cl;
    const int m = ((e & 63) >> 4) * 4 + ((e >> 6) & 3);
    if constexpr (CAND) {
      red[RED + m * (BN + 4) + cl] = n < p.N ? val : -INFINITY;
    } else {
      if (m >= p.M || n >= p.N) continue;
      if (p.out_kind == 2) {
        reinterpret_cast<float*>(p.out[0])[((size_t)blockIdx.y * p.M + m) * p.N + n] = val;
        continue;
      }
      if (p.flags & kGemmRelu) val = fmaxf(val, 0.f);
      const int s = ((unsigned)n >= (unsigned)p.seg_w) + ((unsigned)n >= 2u * (unsigned)p.seg_w);
      void* obase = s == 0 ? p.out[0] : (s == 1 ? p.out[1] : p.out[2]);
      const size_t ld = (size_t)(s == 0 ? p.ldo[0] : (s == 1 ? p.ldo[1] : p.ldo[2]));
      const long long ts = s == 0 ? p.tstride[0] : (s == 1 ? p.tstride[1] : p.tstride[2]);
      const size_t off = (size_t)t_step * ts + (size_t)m * ld + (n - s * p.seg_w);
      if (p.out_kind == 1) reinterpret_cast<float*>(obase)[off] = val;
      else reinterpret_cast<T*>(obase)[off] = from_f32<T>(val);
    }
  }
  if constexpr (CAND) {
    __syncthreads();
    const int m = tid >> 4;   // 16 lanes per row; waves 4-7 have none
    if (m < 16) emit_row_candidates<BN>(p, red + RED + m * (BN + 4), m, m < p.M, blockIdx.x, n0, tid & 15);
  }
  if (p.bump && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *p.bump = *p.bump + 1;
}

template <typename T, int NB, int NV, bool S2, bool CAND>
static hipError_t launch_one(const GemmParams& p, const LnInput& ln, hipStream_t stream) {
  size_t smem = ((size_t)kSkWaves * NB * 256 + (CAND ? 16 * (16 * NB + 4) : 0)) * 4;
  if (NV > 0) smem = std::max(smem, (size_t)p.M * (p.K * sizeof(T) + 16));
  if (smem > 64 * 1024) {
    static std::atomic<unsigned long long> raised{0};   // bit = device ordinal
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&skinny_kernel<T, NB, NV, S2, CAND>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
      raised.fetch_or(bit, std::memory_order_release);
    }
  }
  const dim3 grid((p.N + 16 * NB - 1) / (16 * NB), p.ksplit);
  hipLaunchKernelGGL((skinny_kernel<T, NB, NV, S2, CAND>), grid, dim3(kSkWaves * 64), smem, stream, p, ln);
  return hipGetLastError();
}

template <typename T> static hipError_t launch_t(const GemmParams& p, const LnInput& ln, hipStream_t stream) {
  if (ln.part) {
    if (p.K <= 512)
      return ln.s2.part ? launch_one<T, 1, 2, true, false>(p, ln, stream) : launch_one<T, 1, 2, false, false>(p, ln, stream);
    return ln.s2.part ? launch_one<T, 1, 4, true, false>(p, ln, stream) : launch_one<T, 1, 4, false, false>(p, ln, stream);
  }
  if (p.out_kind == 3)
    return gemm_skinny_cand_n(p.N) == 128 ? launch_one<T, 8, 0, false, true>(p, ln, stream)
                                          : launch_one<T, 4, 0, false, true>(p, ln, stream);
  return p.N >= 16384 ? launch_one<T, 8, 0, false, false>(p, ln, stream) : launch_one<T, 1, 0, false, false>(p, ln, stream);
}

hipError_t launch_gemm_skinny(int dtype, const GemmParams& p, const LnInput& ln, hipStream_t stream) {
  const int esz = dtype == 1 ? 2 : 4;
  const int units = p.K * esz / kUnit;
  if (p.M < 1 || p.M > kSkinnyRows || p.N < 1 || p.K < 1 || p.K * esz % kUnit || p.ksplit < 1 || units % p.ksplit ||
      (p.ksplit > 1 && p.out_kind != 2) || (p.out_kind == 2 && (p.bias || (p.flags & kGemmRelu))))
    return hipErrorInvalidValue;
  if (p.out_kind == 3 && (p.cand_k < 1 || p.cand_k > kGemmCandMaxK || !p.cand_ms || !p.cand_v || !p.cand_i ||
                          p.cand_tiles != (p.N + gemm_skinny_cand_n(p.N) - 1) / gemm_skinny_cand_n(p.N)))
    return hipErrorInvalidValue;
  if (ln.part) {   // the rows are LayerNorm outputs of width K
    const int most = ln.s2.part ? 2 : 4;
    auto split_ok = [&](int s) { return s >= 1 && s <= most; };
    if (p.K % 4 || p.K > kSkinnyLnWidth || p.out_kind == 3 || !ln.bias || !ln.res || !ln.gamma || !ln.beta || !split_ok(ln.nsplit) ||
        (ln.s2.part && (!split_ok(ln.s2.nsplit) || !ln.s2.bias)))
      return hipErrorInvalidValue;
  }
  return dtype == 1 ? launch_t<bf16_t>(p, ln, stream) : launch_t<float>(p, ln, stream);
}

}  // namespace san
