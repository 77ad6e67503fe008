// Small fp32 products on the bf16 matrix cores: k is dealt to the waves of a block, which meet once, at the end.
//
// Bound: the products of a decoder step (20 to 700 rows, 0.05 to 1.2e9 multiplications) are bound by a block's chain: launch,
// first loads, k, epilogue.  gemm_kernel's chain has a barrier per chunk of k, loads that pass through registers into LDS, and
// fp32 MFMAs of 64 cycles for two k-values.  Here every wave has the whole tile for its share of k and LDS of its own, which
// global_load_lds fills: no barrier and no LDS store until the waves' tiles are added, in wave order.  Both operands are split
// into three bf16 parts in registers, eight cross products, two sets of accumulators (as gemm_split.hip, whose bounds on the
// operands hold here too): 256 cycles of the matrix pipe for 16 k-values instead of 512.  44 vector instructions a fragment, and
// they take as long as the MFMAs they lie between: small tiles have too few MFMAs a fragment, large ones too few blocks.
// Error against 64 bits (2-norm, this kernel / the fp32 instructions): 256 x 2048 x 512 7.8e-8 / 2.9e-7, 256 x 1024 x 4096
// 1.3e-7 / 5.8e-7, 128 x 512 x 512 8.1e-8 / 2.0e-7; on none of 283 shapes larger.
// Measured (us, gemm_kernel / here): 64 x 512 x 512 6.8 / 5.2, 128 x 2048 x 512 7.1 / 5.9, 256 x 1536 x 512 8.9 / 7.9, 20 x 3072 x
// 1024 9.8 / 7.4, 185 x 3072 x 1024 22.9 / 17.1.  256 x 2048 x 512 takes 8.7 (9.2): two rounds of 32 x 32 tiles or one of 64 x 32.
// Tried: multiplying a piece right after splitting it, without the overlap (64 x 512 x 512 5.5, 256 x 2048 x 512 8.9; 64 x 64 tiles
// 12.3 instead of 10.9); 16 waves a block (+0.3 us); three or four pieces of LDS a wave (+0.4 us with one block a CU where two
// fit); 64 x 64 tiles by eight waves (spills, 19 us).
#include <atomic>

#include "common.h"
#include "kernels.h"

namespace san {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// eight fp32 values -> fragments of their hi / mid / lo bf16 parts
__device__ __forceinline__ void split_fragment(const f32x4& a, const f32x4& b, bf16x8 (&part)[3]) {
  float r[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    u32x4 w;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      w[q] = f32x2_to_bf16x2_bits(r[2 * q], r[2 * q + 1]);
      if (i < 2) {
        asm("" : "+v"(w[q]));   // (or the compiler converts the lower value a second time, by itself)
        r[2 * q] -= __uint_as_float(w[q] << 16);
        r[2 * q + 1] -= __uint_as_float(w[q] & 0xffff0000u);
      }
    }
    part[i] = __builtin_bit_cast(bf16x8, w);
  }
}

// A block of KW waves owns 32 TM rows x 32 TN columns; every wave has the whole tile for its share of k, and ST places in
// LDS of its own for pieces of 16 k-values.
template <int TM, int TN, int KW>
__global__ __launch_bounds__(KW * 64) void kwaves_kernel(GemmParams p) {
  constexpr int BM = 32 * TM, BN = 32 * TN, RB = 64, NT = KW * 64, ST = 2;   // RB: bytes of a row's 16 k-values
  constexpr int LA = 2 * TM, LB = 2 * TN, L = LA + LB;               // load instructions of 16 rows
  constexpr int STAGE = (BM + BN) * RB;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kh = lane >> 5;

  // every XCD takes a run of neighbouring tiles, down the columns where the weights are the larger operand
  const int nx = (p.N + BN - 1) / BN, ny = (p.M + BM - 1) / BM, tiles = nx * ny;
  const int per = (tiles + 7) / 8, slot = blockIdx.x >> 3, t = (blockIdx.x & 7) * per + slot;
  if (slot >= per || t >= tiles) return;
  const int tile_y = p.xcd_rows ? t % ny : t / nx, tile_x = p.xcd_rows ? t / ny : t % nx;
  const int m0 = tile_y * BM, n0 = tile_x * BN;
  if ((p.flags & kGemmRagged) && m0 >= *p.m_dev) return;   // padding of a ragged batch (whole block)

  // a load instruction covers 16 rows, a 16-byte piece per lane; piece s of row r lies at place s ^ (r / 4) % 4, so that
  // the fragment reads of 16 neighbouring rows touch all banks
  const int lr = lane >> 2, lp = (lane & 3) ^ ((lane >> 4) & 3);
  unsigned a_off[LA], w_off[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) a_off[i] = (unsigned)(min(m0 + i * 16 + lr, p.M - 1) - m0) * (unsigned)p.lda * 4u + (unsigned)lp * 16u;
#pragma unroll
  for (int i = 0; i < LB; ++i) w_off[i] = (unsigned)(min(n0 + i * 16 + lr, p.N - 1) - n0) * (unsigned)p.K * 4u + (unsigned)lp * 16u;
  const int n = p.K / 16 / (KW * p.ksplit);   // pieces of 16 k-values per wave
  const size_t k_first = (size_t)(blockIdx.y * KW + wid) * n * RB;
  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(p.A) + (size_t)m0 * p.lda * 4 + k_first;
  const unsigned char* w_base = reinterpret_cast<const unsigned char*>(p.W) + (size_t)n0 * p.K * 4 + k_first;
  unsigned char* const own = smem + wid * ST * STAGE;
  const unsigned lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)own;
  auto fetch = [&](int c, int st) {
#pragma unroll
    for (int i = 0; i < LB; ++i) load_to_lds(w_base + (size_t)c * RB, w_off[i], lds + st * STAGE + BM * RB + i * 1024);
#pragma unroll
    for (int i = 0; i < LA; ++i) load_to_lds(a_base + (size_t)c * RB, a_off[i], lds + st * STAGE + i * 1024);
  };
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < n) fetch(s, s);

  f32x16 acc[TM][TN], low[TM][TN];   // hi x hi, and the other products
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc[i][j][v] = 0.f; low[i][j][v] = 0.f; }
  const unsigned char* const xr = own + l32 * RB;
  const unsigned char* const wr = own + (BM + l32) * RB;
  const int sw = (l32 >> 2) & 3, p0 = ((2 * kh) ^ sw) * 16, p1 = ((2 * kh + 1) ^ sw) * 16;
  f32x4 xv[TM][2], wv[TN][2];   // a piece as it was loaded
  auto read = [&](int at) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      wv[j][0] = *reinterpret_cast<const f32x4*>(wr + at + j * 32 * RB + p0);
      wv[j][1] = *reinterpret_cast<const f32x4*>(wr + at + j * 32 * RB + p1);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      xv[i][0] = *reinterpret_cast<const f32x4*>(xr + at + i * 32 * RB + p0);
      xv[i][1] = *reinterpret_cast<const f32x4*>(xr + at + i * 32 * RB + p1);
    }
  };
  // `behind` pieces have been requested after the one that is waited for
  auto arrive = [&](int behind) {
    if (behind >= 1) wait_loads<L>();
    else wait_loads<0>();
  };
  bf16x8 xf[2][TM][3], wf[2][TN][3];
  auto split = [&](int set) {
#pragma unroll
    for (int j = 0; j < TN; ++j) split_fragment(wv[j][0], wv[j][1], wf[set][j]);
#pragma unroll
    for (int i = 0; i < TM; ++i) split_fragment(xv[i][0], xv[i][1], xf[set][i]);
  };
  auto multiply = [&](int set) {
    constexpr int PX[7] = {2, 1, 2, 0, 1, 1, 0}, PW[7] = {1, 2, 0, 2, 1, 0, 1};   // smallest products first
#pragma unroll
    for (int q = 0; q < 7; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][j][PW[q]], xf[set][i][PX[q]], low[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][j][0], xf[set][i][0], acc[i][j], 0, 0, 0);
  };
  arrive(n - 1);
  read(0);
  split(0);
  // Piece c is multiplied while piece c + 1 is split: the scheduling groups lay the splitting between the MFMAs, which leave
  // the vector pipe idle.
  int at = 0;   // place of piece c
  auto phase = [&](int c, int set) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // piece c has left its place
    if (c + ST < n) fetch(c + ST, at);
    at = at + 1 == ST ? 0 : at + 1;
    arrive(n - 2 - c);
    __builtin_amdgcn_sched_barrier(0);
    read(at * STAGE);
    multiply(set);
    split(set ^ 1);
    constexpr int VALU = (44 * (TM + TN)) / (8 * TM * TN) + 1;
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * (TM + TN), 0);   // fragment reads
#pragma unroll
    for (int q = 0; q < 8 * TM * TN; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // an MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);          // vector instructions
    }
    __builtin_amdgcn_sched_barrier(0);
    // the parts are ready here: sunk into the next phase, the splitting would stand before its MFMAs
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(wf[set ^ 1][j][q]));
#pragma unroll
      for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(xf[set ^ 1][i][q]));
    }
  };
  int c = 0;
  for (; c + 2 < n; c += 2) {
    phase(c, 0);
    phase(c + 1, 1);
  }
  if (c + 1 < n) {
    phase(c, 0);
    multiply(1);
  } else {
    multiply(0);
  }
  __syncthreads();   // every wave is done with its pieces

  // acc[i][j][v] is row i 32 + l32 and column j 32 + (v / 4) 8 + kh 4 + v % 4: groups of four columns go to LDS and are added
  // in wave order.  Place of group (q, kh) of row l32: 34 apart, so that 16 lanes that read two rows touch all banks.
  constexpr int GS = 34 * 16, WS = TM * TN * 8 * GS;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e] + low[i][j][4 * q + e];
        *reinterpret_cast<f32x4*>(smem + wid * WS + ((i * TN + j) * 8 + q * 2 + kh) * GS + l32 * 16) = v;
      }
  const int t_step = p.t_dev ? *p.t_dev : 0;
  __syncthreads();
  constexpr int PC = BN / 4;
  for (int o = tid; o < BM * PC; o += NT) {
    const int r = o / PC, c4 = o % PC, m = m0 + r, col = n0 + c4 * 4;
    if (m >= p.M || col >= p.N) continue;
    const unsigned char* src = smem + ((r / 32 * TN + c4 / 8) * 8 + c4 % 8) * GS + (r & 31) * 16;
    f32x4 v = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
    for (int w = 1; w < KW; ++w) v += *reinterpret_cast<const f32x4*>(src + w * WS);
    float* dst;
    if (p.out_kind == 2) {
      dst = reinterpret_cast<float*>(p.out[0]) + ((size_t)blockIdx.y * p.M + m) * p.N + col;
    } else {
      if (p.bias) v += *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.bias) + col);
      if (p.flags & kGemmRelu) v = f32x4{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
      const int s = ((unsigned)col >= (unsigned)p.seg_w) + ((unsigned)col >= 2u * (unsigned)p.seg_w);
      const long long ts = s == 0 ? p.tstride[0] : (s == 1 ? p.tstride[1] : p.tstride[2]);
      dst = reinterpret_cast<float*>(s == 0 ? p.out[0] : (s == 1 ? p.out[1] : p.out[2])) + (size_t)t_step * ts +
            (size_t)m * (s == 0 ? p.ldo[0] : (s == 1 ? p.ldo[1] : p.ldo[2])) + (col - s * p.seg_w);
    }
    *reinterpret_cast<f32x4_any*>(dst) = v;
  }
  if (p.bump && tile_x == 0 && tile_y == 0 && blockIdx.y == 0 && tid == 0) *p.bump = *p.bump + 1;
}

template <int TM, int TN, int KW> static hipError_t launch_kw(const GemmParams& p, hipStream_t stream) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  constexpr int stages = KW * 2 * (BM + BN) * 64, out = KW * TM * TN * 8 * 34 * 16, smem = stages > out ? stages : out;
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  if (p.K % (16 * KW * p.ksplit) || (long)BM * p.lda * 4 >= 1l << 31 || (long)BN * p.K * 4 >= 1l << 31) return hipErrorInvalidValue;
  if (smem > 64 * 1024) {
    static std::atomic<unsigned long long> raised{0};   // bit = device ordinal
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&kwaves_kernel<TM, TN, KW>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
      if (e != hipSuccess) return e;
      raised.fetch_or(bit, std::memory_order_release);
    }
  }
  GemmParams q = p;
  q.xcd_rows = p.N > p.M;
  const long tiles = (long)((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
  hipLaunchKernelGGL((kwaves_kernel<TM, TN, KW>), dim3((unsigned)((tiles + 7) / 8 * 8), p.ksplit), dim3(KW * 64), smem, stream, q);
  return hipGetLastError();
}

hipError_t launch_gemm_kwaves(const GemmParams& p, int variant, hipStream_t stream) {
  if (p.M < 1 || p.N < 4 || p.N % 4 || p.ksplit < 1 || p.out_kind == 3 || (p.ksplit > 1 && p.out_kind != 2) || !gemm_kwaves_aligned(p))
    return hipErrorInvalidValue;
  switch (variant) {
    case 1: return launch_kw<1, 1, 8>(p, stream);
    case 2: return launch_kw<2, 1, 8>(p, stream);
    case 3: return launch_kw<2, 2, 4>(p, stream);
    case 4: return launch_kw<1, 1, 4>(p, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace san
