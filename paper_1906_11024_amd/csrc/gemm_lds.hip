// bf16 products whose operands go from global memory straight to LDS (global_load_lds), in tiles from 64 x 64 to 320 x 256.
//
// Bound: the products of an encoder are bound by what feeds the matrix cores, the small ones of a decoder step by the
// chain inside a block (where their weights lie, L2, Infinity Cache or HBM, moves a launch by 0.2 us).  gemm_kernel
// brings a chunk of k through registers: load, wait, LDS store, barrier, fragment reads.  Here a chunk needs neither
// registers nor LDS stores, so that tiles can be large (fewer fragment reads per MFMA: 256 x 256 by eight waves of 128 x 64
// reads as long as it multiplies) or two blocks of small ones share a CU and cover each other's waits.  ST chunks of BK
// k-values lie in LDS; fragments are read a step of 16 ahead, and the last step of a chunk is multiplied behind the barrier
// that the next chunk waits at, so that its first reads have something to hide behind.  Rows have no padding (the
// hardware writes 64 x 16 bytes in a row): a row's 16-byte pieces are permuted by the row's number instead.
// The weights are the A operand, so that a lane holds four neighbouring columns of one row: the tile goes through LDS in
// 8- and 16-byte writes and leaves in whole lines (2-byte stores of 64-byte pieces took 3 us of a 64 x 128 tile).
// Every XCD takes a run of neighbouring tiles, of rows or columns as the larger operand asks.
// Sums have the bits of gemm_kernel's, which deals small products to groups of waves: the 64 x 64 tiles keep as many sums per
// output (a decode of 300 to 1020 rows is within 1 % of one sum's time; with those products left to gemm_kernel up to 8 % slower).
// Measured (us, gemm_kernel / here; K in the middle of the encoder's and the decoder's): 8900 x 2048 x 512 48.8 / 24.8,
// x 1536 x 512 46.8 / 22.2, x 512 x 2048 (fp32 out) 54 / 30, x 512 x 512 20.3 / 12.7; 12300 x 3072 x 1024 144 / 86, x 1024 x 4096
// 156 / 112 (0.93 PFLOP/s; rates of 1.3 where the tiles fill the chip); 1024 x 2048 x 512 7.5 / 6.7, 512 x 4096 x 1024
// 11.5 / 10.1, 301 x 4096 x 1024 10.4 / 9.0; output layers 1024 x 32000 x 512 59 / 52, 512 x 32000 x 1024 47.5 / 41.6.
// Tried: chunks of 32 in four stages for the large tiles (+5 %), waves of 128 x 64 in 256 x 128 tiles (+15 %: one wave per
// SIMD), reads without the interleaving (the same time for large tiles).
#include <atomic>

#include "candidates.h"
#include "common.h"
#include "kernels.h"

namespace san {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// WM x WN waves, each TM x TN tiles of 32 x 32; k in chunks of BK, ST chunks of LDS.  G sums per output, CU chunks to each in
// turn, added up in order at the end: what gemm_kernel does with its groups of waves, bit for bit (gemm_k_groups).
template <int WM, int WN, int TM, int TN, int BK, int ST, bool CAND, int G, int CU>
__global__ __launch_bounds__(WM* WN * 64) void lds_kernel(GemmParams p) {
  constexpr int NW = WM * WN, NT = NW * 64;
  constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN;
  constexpr int RB = BK * 2;                       // bytes of a row chunk
  constexpr int RPI = 1024 / RB;                   // rows per load instruction of a wave
  constexpr int LA = BM / RPI / NW, LB = BN / RPI / NW;   // load instructions per wave and chunk
  constexpr int STAGE = (BM + BN) * RB;
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "rows deal out evenly");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid % WM, wn = wid / WM, l32 = lane & 31, kh = lane >> 5;

  const int M = (p.flags & kGemmRagged) ? *p.m_dev : p.M;
  const int nx = (p.N + BN - 1) / BN, ny = (M + BM - 1) / BM, tiles = nx * ny;
  // Every XCD takes a run of neighbouring tiles: rows of tiles where the activations are the larger operand (they leave
  // HBM once, the weights once per XCD), columns of tiles where the weights are.
  const int per = (tiles + 7) / 8, slot = blockIdx.x >> 3, t = (blockIdx.x & 7) * per + slot;
  if (slot >= per || t >= tiles) return;
  const int tile_y = p.xcd_rows ? t % ny : t / nx, tile_x = p.xcd_rows ? t / ny : t % nx;
  const int m0 = tile_y * BM, n0 = tile_x * BN;

  const int t_step = p.t_dev ? *p.t_dev : 0;
  // this wave's loads: instruction i covers rows (wid * LA + i) * RPI + lane / (RB / 16), one 16-byte piece per lane;
  // piece s of row r lies in LDS at place s ^ swz(r), so that the fragment reads of 16 neighbouring rows touch all banks
  constexpr int PPR = RB / 16;                     // pieces per row
  const int lr = lane / PPR, lp = lane % PPR;
  auto swz = [](int r) { return PPR == 16 ? r & 15 : PPR == 8 ? (r >> 1) & 7 : (r >> 2) & 3; };
  unsigned a_off[LA], w_off[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (wid * LA + i) * RPI + lr;
    a_off[i] = (unsigned)(min(m0 + r, p.M - 1) - m0) * (unsigned)p.lda * 2u + (unsigned)(lp ^ swz(r)) * 16u;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int r = (wid * LB + i) * RPI + lr;
    w_off[i] = (unsigned)(min(n0 + r, p.N - 1) - n0) * (unsigned)p.K * 2u + (unsigned)(lp ^ swz(r)) * 16u;
  }
  const int nch = p.K / BK / p.ksplit;             // chunks of this block's k range
  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(p.A) + (size_t)m0 * p.lda * 2 + (size_t)blockIdx.y * nch * RB;
  const unsigned char* w_base = reinterpret_cast<const unsigned char*>(p.W) + (size_t)n0 * p.K * 2 + (size_t)blockIdx.y * nch * RB;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const unsigned a_lds = lds0 + wid * LA * 1024, w_lds = lds0 + BM * RB + wid * LB * 1024;
  auto fetch = [&](int c, int st) {
#pragma unroll
    for (int i = 0; i < LA; ++i) load_to_lds(a_base + (size_t)c * RB, a_off[i], a_lds + st * STAGE + i * 1024);
#pragma unroll
    for (int i = 0; i < LB; ++i) load_to_lds(w_base + (size_t)c * RB, w_off[i], w_lds + st * STAGE + i * 1024);
  };
#pragma unroll
  for (int s = 0; s < ST - 1; ++s)
    if (s < nch) fetch(s, s);

  // The weights are the MFMA's A operand: acc[i][j][v] is row (wm TM + i) 32 + l32 and column (wn TN + j) 32 + (v / 4) 8 +
  // kh 4 + v % 4, so that a lane holds four neighbouring columns and the tile goes to LDS in wide writes
  f32x16 accs[G][TM][TN];
  auto& acc = accs[0];
#pragma unroll
  for (int g = 1; g < G; ++g)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) accs[g][i][j][v] = 0.f;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    float bv[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) bv[v] = 0.f;
    if (p.bias && p.out_kind != 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = min(n0 + (wn * TN + j) * 32 + q * 8 + kh * 4, p.N - 4);   // N is a multiple of 4
        const float4 b4 = load4(reinterpret_cast<const bf16_t*>(p.bias) + n);
        bv[4 * q] = b4.x; bv[4 * q + 1] = b4.y; bv[4 * q + 2] = b4.z; bv[4 * q + 3] = b4.w;
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = bv[v];
  }

  const unsigned char* const xr = smem + (wm * TM * 32 + l32) * RB;
  const unsigned char* const wr = smem + (BM + wn * TN * 32 + l32) * RB;
  const int sw = swz(l32);
  constexpr int STEPS = BK / 16;
  static_assert(STEPS % 2 == 0, "two sets of fragments");
  bf16x8 xf[2][TM], wf[2][TN];
  auto read = [&](int set, int at) {
#pragma unroll
    for (int i = 0; i < TM; ++i) xf[set][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xr + at + i * 32 * RB));
#pragma unroll
    for (int j = 0; j < TN; ++j) wf[set][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wr + at + j * 32 * RB));
  };
  auto multiply = [&](int set, int g) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) accs[g][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][j], xf[set][i], accs[g][i][j], 0, 0, 0);
  };
  // the reads of the next step go between the MFMAs of this one
  auto interleave = [&] {
#pragma unroll
    for (int q = 0; q < TM + TN; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // a fragment read
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an MFMA
    }
    if constexpr (TM * TN > TM + TN) __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - TM - TN, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto piece = [&](int c, int s) { return (c % ST) * STAGE + ((s * 2 + kh) ^ sw) * 16; };
  // chunk c is there once the ST - 2 chunks behind it are all that is outstanding (in the last rounds: nothing is)
  auto arrive = [&](int c) {
    if (c + ST - 2 < nch) wait_loads<(ST - 2) * (LA + LB)>();
    else wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  arrive(0);
  if (ST - 1 < nch) fetch(ST - 1, ST - 1);
  read(0, piece(0, 0));
  auto chunk = [&](int c, int g) {
#pragma unroll
    for (int s = 0; s < STEPS - 1; ++s) {
      read((s + 1) & 1, piece(c, s + 1));
      multiply(s & 1, g);
      interleave();
    }
    // all of the chunk is in registers: its LDS is free, and the last step covers the first reads of the next chunk
    if (c + 1 < nch) {
      arrive(c + 1);
      if (c + ST < nch) fetch(c + ST, c % ST);
      read(0, piece(c + 1, 0));
    }
    multiply((STEPS - 1) & 1, g);
    interleave();
  };
  for (int c = 0; c < nch; c += G * CU) {
#pragma unroll
    for (int u = 0; u < G * CU; ++u)
      if (u == 0 || c + u < nch) chunk(c + u, u / CU);
  }
#pragma unroll
  for (int g = 1; g < G; ++g)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] += accs[g][i][j][v];
  __syncthreads();   // the stages are dead

  if (!CAND && p.out_kind == 0) {
    // bf16: the whole tile through LDS (a row leaves in 16-byte pieces of whole lines), half of it where it is too tall
    constexpr int LDB = BN * 2 + 16, PASSES = BM * LDB <= 160 * 1024 ? 1 : 2;   // bytes of a row
    unsigned char* const tile = smem;
    const bool relu = (p.flags & kGemmRelu) != 0;
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      if (pass) __syncthreads();
      if (PASSES == 1 || wm == pass) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float4 v = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
              if (relu) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
              const int r = ((PASSES == 1 ? wm * TM : 0) + i) * 32 + l32, c = (wn * TN + j) * 32 + q * 8 + kh * 4;
              store4(reinterpret_cast<bf16_t*>(tile + r * LDB + c * 2), v);
            }
      }
      __syncthreads();
      constexpr int PC = BN / 8, ROWS = BM / PASSES;   // pieces per row
      for (int q = tid; q < ROWS * PC; q += NT) {
        const int r = q / PC, n = n0 + (q % PC) * 8, m = m0 + pass * ROWS + r;
        if (m >= p.M || n >= p.N) continue;
        const int s = ((unsigned)n >= (unsigned)p.seg_w) + ((unsigned)n >= 2u * (unsigned)p.seg_w);
        const long long ts = s == 0 ? p.tstride[0] : (s == 1 ? p.tstride[1] : p.tstride[2]);
        bf16_t* const o = reinterpret_cast<bf16_t*>(s == 0 ? p.out[0] : (s == 1 ? p.out[1] : p.out[2])) + (size_t)t_step * ts +
                          (size_t)m * (s == 0 ? p.ldo[0] : (s == 1 ? p.ldo[1] : p.ldo[2])) + (n - s * p.seg_w);
        *reinterpret_cast<u32x4*>(o) = *reinterpret_cast<const u32x4*>(tile + r * LDB + (q % PC) * 16);
      }
    }
  } else {
    // fp32 (or its candidates): in passes of at most 128 rows, a wave row's tiles at a time
    constexpr int LDW = BN + 4, TP = TM < 3 ? TM : 2, PR = TP * 32 * WM;   // tile rows of a wave per pass
    float* const tile = reinterpret_cast<float*>(smem);
    const bool relu = (p.flags & kGemmRelu) != 0;
    float* const base = CAND ? nullptr : reinterpret_cast<float*>(p.out[0]) + (size_t)t_step * p.tstride[0] + (size_t)blockIdx.y * p.M * p.N;
    const size_t ld = p.out_kind == 2 ? (size_t)p.N : (size_t)p.ldo[0];
#pragma unroll
    for (int i0 = 0; i0 < TM; i0 += TP) {
      if (i0) __syncthreads();
#pragma unroll
      for (int i = i0; i < (i0 + TP < TM ? i0 + TP : TM); ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float4 v = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
            if (relu) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
            const int c = (wn * TN + j) * 32 + q * 8 + kh * 4;
            if (CAND && n0 + c >= p.N) v = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);   // N is a multiple of 4
            *reinterpret_cast<float4*>(tile + ((wm * TP + i - i0) * 32 + l32) * LDW + c) = v;
          }
      __syncthreads();
      // row r of the pass: tile row i0 + r / 32 % TP of wave row r / 32 / TP
      if constexpr (CAND) {
        for (int r = tid >> 4; r < PR; r += NT / 16) {
          const int i = i0 + r / 32 % TP, m = m0 + (r / 32 / TP * TM + i) * 32 + r % 32;
          if (i < TM) emit_row_candidates<BN>(p, tile + r * LDW, m, m < p.M, tile_x, n0, lane & 15);
        }
      } else {
        constexpr int PC = BN / 4;
        for (int q = tid; q < PR * PC; q += NT) {
          const int r = q / PC, n = n0 + (q % PC) * 4, i = i0 + r / 32 % TP, m = m0 + (r / 32 / TP * TM + i) * 32 + r % 32;
          if (i < TM && m < p.M && n < p.N) *reinterpret_cast<f32x4_any*>(base + (size_t)m * ld + n) = *reinterpret_cast<const f32x4*>(tile + r * LDW + (q % PC) * 4);
        }
      }
    }
  }
  if (p.bump && tile_x == 0 && tile_y == 0 && tid == 0) *p.bump = *p.bump + 1;
}

template <int WM, int WN, int TM, int TN, int BK, int ST, bool CAND, int G = 1, int CU = 1>
static hipError_t launch_lds_t(const GemmParams& p, hipStream_t stream) {
  constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN;
  constexpr int TP = TM < 3 ? TM : 2, full = BM * (BN * 2 + 16), half = full <= 160 * 1024 ? full : full / 2;
  constexpr int stages = ST * (BM + BN) * BK * 2, wide = TP * 32 * WM * (BN + 4) * 4, out = CAND || wide > half ? wide : half;
  constexpr int smem = stages > out ? stages : out;
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  if (p.K % (BK * p.ksplit) || (long)BM * p.lda * 2 >= 1l << 31 || (long)BN * p.K * 2 >= 1l << 31) return hipErrorInvalidValue;
  static std::atomic<unsigned long long> raised{0};   // bit = device ordinal
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (!(raised.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lds_kernel<WM, WN, TM, TN, BK, ST, CAND, G, CU>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    raised.fetch_or(bit, std::memory_order_release);
  }
  GemmParams q = p;
  q.xcd_rows = p.N > p.M;   // tiles run down the columns of the larger operand
  const long tiles = (long)((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
  hipLaunchKernelGGL((lds_kernel<WM, WN, TM, TN, BK, ST, CAND, G, CU>), dim3((unsigned)((tiles + 7) / 8 * 8), p.ksplit), dim3(WM * WN * 64), smem, stream, q);
  return hipGetLastError();
}

// three chunks of LDS where a block has its CU to itself, two where two blocks share one (of 128 rows, k = 1024 and weights
// from HBM: 128 x 32000 with candidates 19.4 us with three, 22.9 with two; 512 rows 60 and 50)
template <int TM, bool CAND> static hipError_t launch_lds_128(const GemmParams& p, hipStream_t stream) {
  const long tiles = (long)((p.M + 64 * TM - 1) / (64 * TM)) * ((p.N + 127) / 128) * p.ksplit;
  return tiles <= 256 ? launch_lds_t<2, 4, TM, 1, 64, 3, CAND>(p, stream) : launch_lds_t<2, 4, TM, 1, 64, 2, CAND>(p, stream);
}

// 64 x 64 tiles; a group's turn is 128 values of k where K is a multiple of it, else 64
template <int BK, int ST> static hipError_t launch_lds_64(const GemmParams& p, int groups, hipStream_t stream) {
  if (groups == 1) return launch_lds_t<2, 2, 1, 1, BK, ST, false>(p, stream);
  if (BK == 64 && p.K % 128 == 0)
    return groups == 2 ? launch_lds_t<2, 2, 1, 1, BK, ST, false, 2, 128 / BK>(p, stream) : launch_lds_t<2, 2, 1, 1, BK, ST, false, 4, 128 / BK>(p, stream);
  return groups == 2 ? launch_lds_t<2, 2, 1, 1, BK, ST, false, 2>(p, stream) : launch_lds_t<2, 2, 1, 1, BK, ST, false, 4>(p, stream);
}

hipError_t launch_gemm_lds(const GemmParams& p, int variant, int groups, hipStream_t stream) {
  if (p.M < 1 || p.N < 4 || p.N % 4 || p.ksplit < 1 || (p.ksplit > 1 && p.out_kind != 2) || !gemm_lds_aligned(p)) return hipErrorInvalidValue;
  const bool cand = p.out_kind == 3;
  if (cand && (variant < 3 || variant > 5)) return hipErrorInvalidValue;
  if (groups != 1 && ((groups != 2 && groups != 4) || (variant != 1 && variant != 2))) return hipErrorInvalidValue;
  switch (variant) {
    case 1: return launch_lds_64<128, 2>(p, groups, stream);
    case 2: return launch_lds_64<64, 4>(p, groups, stream);
    case 3: return cand ? launch_lds_128<2, true>(p, stream) : launch_lds_128<2, false>(p, stream);
    case 4: return cand ? launch_lds_128<3, true>(p, stream) : launch_lds_128<3, false>(p, stream);
    case 5: return cand ? launch_lds_t<2, 4, 4, 2, 64, 2, true>(p, stream) : launch_lds_t<2, 4, 4, 2, 64, 2, false>(p, stream);
    case 6: return launch_lds_t<2, 4, 5, 2, 64, 2, false>(p, stream);
    case 7: return launch_lds_t<4, 2, 1, 1, 64, 4, false>(p, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace san
