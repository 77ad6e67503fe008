// Which route a call takes, as functions of its sizes alone (host code without HIP, so that tests can compile it and
// check that the sizes they run still take the route they are meant for).
#pragma once

namespace san {

// fp32 through the bf16 matrix cores (gemm_split.hip): tile height (64 wm rows; 0: the fp32 instructions are faster)
// and k split in [ks_min, ks_max].  A model of both routes, in us:
//   split   3 + 21 (128 rows) or 30 (192) for k = 512 and every round of one block per CU, in proportion to k, and
//           what the consumer pays for further partials (written and read at 4 TB/s)
//   plain   4 + 2 M N K flops at 95 TFLOP/s, M in whole tiles of 64
// Where the column tiles are no multiple of eight the row tiles of one column tile stay on one XCD, so a round is 32
// blocks of the XCD that has most of them (plain: the 128 x 128 tiles, which products of 200 such tiles take).
// Measured (us, split / plain): outputs of 65, 185, 256 and 512 rows x 32000 at k = 512 24.7 / 37.0, 34.7 / 66.7,
// 46.6 / 67.4, 87.9 / 130, 128 x 32000 x 256 16.6 / 21.5, x 1024 44.0 / 65.1; 3840 x 2048 x 512 47.3 / 67.3,
// 2257 x 1536 x 512 33.1 / 66.1, 1000 x 4096 x 1024 44.8 / 65.6, 3840 x 512 x 2048 (k in two) 44.3 / 69.9,
// 2048 x 1024 x 4096 (two) 81.7 / 133; left to the plain kernel 256 x 8000 x 512 23.3 / 22.2, 3840 x 512 x 512
// 25.2 / 22.9, 512 x 1024 x 1024 14.8 / 13.1.  Over 361 shapes of 64 to 7680 rows, k 256 to 4096, the choice lost
// 4 % or more on one.
struct SplitShape { int wm, ks; };
inline SplitShape gemm_split_shape(int M, int N, int K, int ks_min, int ks_max) {
  SplitShape best{0, 1};
  if (K % 64 || M < 1 || N < 1) return best;
  const long cols = ((long)N + 127) / 128, rows128 = ((long)M + 127) / 128;
  const bool by_xcd = cols % 8 != 0;
  const float uneven = by_xcd && M > 128 && rows128 * cols >= 200 ? (float)((cols + 7) / 8 * 8) / (float)cols : 1.f;
  float best_us = 0.85f * (4.f + uneven * 2.f * ((M + 63) / 64 * 64) * (float)N * (float)K / 95e6f);
  for (int wm = 2; wm <= 3; ++wm)
    for (int ks = ks_min; ks <= ks_max; ks *= 2) {
      if (K % (64 * ks) || (ks > 1 && K / ks < 512)) continue;
      const long rows = ((long)M + 64 * wm - 1) / (64 * wm);
      const long rounds = by_xcd && rows > 1 && ks == 1 ? ((cols + 7) / 8 * rows + 31) / 32 : (cols * rows * ks + 255) / 256;
      const float us = 3.f + (float)rounds * (wm == 2 ? 21.f : 30.f) * (float)K / (512.f * ks) + 2e-6f * (ks - 1) * (float)M * (float)N;
      if (us < best_us) { best_us = us; best = SplitShape{wm, ks}; }
    }
  return best;
}

constexpr int kSkinnyRows = 16, kSkinnyLnWidth = 1024;   // products of few rows (gemm_skinny.hip)
// k split of its products that write partials
inline int gemm_skinny_ksplit(int N, int K, int dtype) {
  // a wave keeps two units or more, and splitting stops at half a block per CU: what a split saves in load time it
  // costs in partials, which every block of the consumer reads
  const int units = K * (dtype == 1 ? 2 : 4) / 64;   // of 64 bytes: a load instruction's share of a row
  const int tiles = (N + 15) / 16;
  int ks = 1;
  while (ks < 4 && tiles * ks < 128 && units % (ks * 2) == 0 && units / (ks * 2) >= 2 * 8) ks *= 2;
  return ks;
}
// Columns per block of its candidate form: 128 halve the slots that the beam step reads, 64 give twice the blocks.
// Steps of 4 rows, beam 4, fp32 512 / 256 columns (us, 64 / 128): 16384 words 216 / 219, 202 / 205, 20000 words 222 / 221,
// 206 / 204, 32000 words 224 / 223, 213 / 211.
constexpr int kSkinnyCandWide = 18432;
inline int gemm_skinny_cand_n(int N) { return N >= kSkinnyCandWide ? 128 : 64; }

// Whether it is the faster kernel for a product of its own (us, the tile kernels / this one; weights from the Infinity
// Cache; kind: GemmParams::out_kind).
//   candidates: fp32 always (8000 x 512 18 / 9.5, 32000 x 512 28 / 18, 32000 x 256 19 / 14), bf16 below the line above
//     (16000 x 512 11.6 / 8.5; 32000 x 512 12.1 / 13.4)
//   k split over blocks: never, the tile kernels split further (512 x 512 4.1 / 5.0, bf16 3.5 / 4.4, 1024 x 4096 8.1 / 9.1)
//   others, fp32: from k = 512 on (2048 x 512 6.9 / 5.5 at 4 rows, 7.0 / 6.3 at 16; 3072 x 1024 9.9 / 6.2; 1024 x 256
//     4.9 / 5.1), where a block's 16 columns are enough of them (16000 x 512 12.6 / 14.1; with 128 columns, from 16384
//     words on, 32000 x 512 21.6 / 16.5)
//   others, bf16: from k = 1024 on and up to 6 rows (3072 x 1024 5.4 / 5.2 at 4 rows, 5.5 / 5.6 at 8; 2048 x 512 4.8 / 5.0),
//     up to 16 where k = 2048 meets few columns (512 x 2048 7.2 / 4.9 at 4 rows, 7.4 / 5.9 at 16)
inline bool gemm_skinny_faster(int dtype, int M, int N, int K, int kind, int ksplit) {
  if (M > kSkinnyRows) return false;
  if (kind == 3) return dtype == 0 || N < kSkinnyCandWide;
  if (ksplit > 1) return false;
  if (dtype == 0) return K >= 512 && (N <= 8 * K || (kind == 1 && N >= 16384));
  return K >= 1024 && N <= 8 * K && (M <= 6 || (K >= 2048 && N <= 2048));
}

// Whether a cached step of `rows` rows runs with the LayerNorms inside its projections (decode_few_rows): what the
// launches cost against what every block pays for normalising all rows itself.  A step in us, the general route / this
// one, on both sides of each line: fp32, 64 columns 1 row 67 / 68; 128: 4 rows 135 / 133, 6 136.5 / 137; 256: 8 225 / 223,
// 12 227 / 236; 384: 12 257 / 244, 16 258 / 258; 512: 12 253 / 252, 16 257 / 264; 768: 1 288 / 275, 6 297 / 311;
// 1024: 1 332 / 337.  bf16, 256: 4 188 / 184, 6 187 / 193; 512: 4 211 / 201, 8 213 / 215; 768: 4 229 / 222, 6 229 / 231;
// 1024: 4 237 / 231, 6 238 / 241, 16 251 / 294.
inline bool few_rows_faster(int dtype, int rows, int d) {
  if (d < 128 || d > kSkinnyLnWidth) return false;
  if (dtype == 0) return rows <= (d < 256 ? 4 : d < 384 ? 8 : d <= 512 ? 12 : d <= 768 ? 4 : 0);
  return rows <= (d == 512 ? 6 : 4);
}

// Models whose decoder steps run with one workgroup per sentence (small_model.hip), and whether they do for `batch`
// sentences.  A model of both routes, in us a step of R = beam rows a sentence and L layers, with MB the weights a step
// reads, all of them by one workgroup, and keys the positions that its attentions read (2 a position for a head, which reads
// keys and values, 1 for a follower):
//   one workgroup a sentence   6 + 6.2 L + (5 + 4 R) MB + p keys for every 256 sentences
//   launches                   21 + 27 L + 0.006 keys
// p = d / H times the larger of 3e-4 + 4e-5 R H and 7e-5 R H (8 waves deal with the R H pairs of rows and heads), 1.4 times that
// where 32 sentences or more want their caches at once; the launches' attention has the whole chip.
// Measured (us, launches / one workgroup): 64 columns, F 256, 2 layers, 1000 words (0.7 MB) beam 1 70 / 21, 4 73 / 32,
// 8 78 / 44, 300 sentences of beam 1 79 / 42; 6 layers (1.6 MB) beam 4 182 / 76; 4000 words (1.5 MB) beam 4 74 / 48;
// 128 columns, F 512, 2 layers, 1000 words (2.3 MB) beam 1 72 / 35, 4 77 / 59; 6 layers, 2004 words (6.5 MB) beam 1
// 190 / 111, 4 192 / 175, 8 196 / 240.  The line leaves 15 % to the launches.  With positions (2 and 64 sentences, 2 layers of
// 64 columns, 4 heads, means of a decode): 512 target positions beam 1 77 / 28 and 84 / 30, beam 8 84 / 89 and 99 / 106; 1024
// source positions beam 1 85 / 36 and 98 / 50, beam 4 78 / 79 and 100 / 93, beam 8 82 / 140 and 130 / 155; 1024 of both beam 1
// 96 / 50 and 112 / 74.  Of 586 such settings (1 to 8 heads, 16 to 1024 positions) none is more than 3 % slower than with the
// launches, 45 stay with them that would gain 10 % or more: here 8 % are left.
constexpr int kSmallLds = 160 * 1024, kSmallBeam = 8;   // LDS of a workgroup; its search sorts the candidates of this beam at once
inline bool small_model_faster(int d, int F, int V, int layers, int beam, int batch, int H = 1, float keys = 0.f) {
  if ((d != 64 && d != 128) || (F != 64 && F != 128 && F != 256 && F != 512) || beam < 1 || beam > kSmallBeam || batch < 1) return false;
  const float mb = 4e-6f * ((float)layers * (6.f * d * d + 2.f * d * F) + (float)V * d);
  const float rounds = (float)((batch + 255) / 256), launches = 21.f + 27.f * layers;
  const float here = rounds * (6.f + 6.2f * layers + (5.f + 4.f * beam) * mb);
  if (here > 0.85f * launches) return false;
  const float rh = (float)(beam * H), few = 3e-4f + 4e-5f * rh, many = 7e-5f * rh;
  const float p = (float)(d / H) * (few > many ? few : many) * (batch >= 32 ? 1.4f : 1.f);
  return here + rounds * p * keys <= 0.92f * (launches + 0.006f * keys);
}

// bf16 products with their operands straight to LDS (gemm_lds.hip): which tile, or 0 for gemm_kernel.  kind: GemmParams::
// out_kind; ragged: M is the padded row count of a batch whose words lie back to back.
//   1 64 x 64, chunks of 128   2 64 x 64, four chunks of 64   3 128 x 128   4 192 x 128   5 256 x 256   6 320 x 256
//   7 128 x 64, four chunks of 64
// A model of each, in us: 2 + the larger of one block alone on its CU, e1 + g1 k / 512, and of n blocks on a CU one
// after the other or two at a time, n (e2 + g2 k / 512), n between the tiles per CU and that rounded up (q: how near the
// former).  Fitted to 142 shapes of 64 to 15300 rows; over them the choice costs 0.4 % against the best of them, 10 % at
// worst.  Products with candidates (the last three lines) pay their selection too.  1, and 2 with more tiles than CUs, hold
// a chunk or two in flight per block: enough for k of 512, but the weights of wider models come from HBM (512 x 4096 x 1024 with
// weights of 320 MB: 1 11.5, 2 11.8, 7 10.1, gemm_kernel 11.5).
// gemm_kernel keeps: products split over blocks whose parts of k are short (1024 x 512 x 2048 in four 6.9 / 7.25,
// 512 x 1024 x 1024 in four 5.5 / 5.6; but 512 x 1024 x 4096 in four 11.8 / 11.5, 301 rows 10.3 / 9.5); few tiles with a long
// k, which it splits over the waves of a block (1024 x 512 x 2048 9.8 / 10.9, 512 x 1024 x 1024 6.5 / 6.7, 68 x 4096 x 1024
// 6.7 / 7.3); output layers of candidates with few tiles (40 x 32000 x 512 10.0 / 11.8, 256 x 8000 9.2 / 11.3; 68 x 32000
// 15.2 / 11.7, 300 28.7 / 21.2, 700 48.7 / 38.3).  Padding is a quarter to a half of a ragged batch: 0.7 of it stand for M.
struct LdsModel { int bm, bn; float e1, g1, e2, g2, q; };
constexpr int kLdsVariants = 7;
constexpr LdsModel kLdsModels[kLdsVariants] = {
    {64, 64, 0.65f, 2.28f, 0.88f, 1.73f, 0.55f},   {64, 64, 1.09f, 2.01f, 0.91f, 1.72f, 0.46f},
    {128, 128, 0.41f, 4.71f, 1.22f, 4.43f, 0.35f}, {192, 128, 3.81f, 0.54f, 2.12f, 5.49f, 0.22f},
    {256, 256, 0.67f, 11.19f, 4.70f, 10.95f, 0.f}, {320, 256, 2.81f, 8.57f, 6.85f, 12.66f, 0.f},
    {128, 64, 1.90f, 2.30f, 2.00f, 2.30f, 0.1f}};
constexpr LdsModel kLdsCandModels[3] = {   // of 3, 4 and 5
    {128, 128, 0.8f, 9.6f, 1.0f, 5.0f, 0.3f}, {192, 128, 2.5f, 10.f, 2.7f, 5.8f, 0.2f}, {256, 256, 12.7f, 13.4f, 12.7f, 13.4f, 0.f}};
inline int gemm_k_groups(int M, int N, int K, int ksplit, bool partials);
inline int gemm_lds_variant(int M, int N, int K, int kind, int ksplit, bool ragged) {
  if (M <= 16 || N < 64 || ksplit < 1 || K % (64 * ksplit)) return 0;
  if (K % 128 == 0 && K / 128 % ksplit) return 0;   // gemm_kernel splits between other values of k, which would be other sums
  const int k = K / ksplit;
  const bool cand = kind == 3;
  if (cand && (M <= 64 || (long)((M + 127) / 128) * ((N + 127) / 128) < 200)) return 0;
  if (ksplit > 1 && k < 1024) return 0;
  // 5 to 15 us of a 460 us pass over 16 sentences of up to 9 words.  Not output layers: gemm_kernel has no large tile in bf16
  // (128 x 32000 x 512 with its logits 17.9 / 13.6, 256 rows 27.7 / 16.7; a 128 x 128 tile of it took 15.1 and 20.1).
  if (!cand && M <= 256 && k <= 512 && (M < 128 || (long)((M + 127) / 128) * ((N + 127) / 128) < 200)) return 0;
  long tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64) * ksplit;
  if (!cand && k >= 1024 && tiles64 <= 128) return 0;
  // The sums have the bits of gemm_kernel's, so those of a ragged batch are the padded one's: the padded rows say how many
  // groups of k there are (64 x 64 tiles only).
  const int groups = cand ? 1 : gemm_k_groups(M, N, K, ksplit, kind == 2);
  if (ragged) M = M - M * 3 / 10;
  tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64) * ksplit;
  int best = 0;
  float best_us = 0.f;
  for (int v = 1; v <= kLdsVariants; ++v) {
    if (groups > 1 && v > 2) break;
    if (cand ? v < 3 || v > 5 : (v == 1 && (k % 128 || k > 512)) || (v == 2 && k > 512 && tiles64 > 256)) continue;
    const LdsModel& m = cand ? kLdsCandModels[v - 3] : kLdsModels[v - 1];
    const float tiles = (float)((M + m.bm - 1) / m.bm) * (float)((N + m.bn - 1) / m.bn) * (float)ksplit / 256.f;
    const float n = (1.f - m.q) * (float)(long)(tiles + 0.9999f) + m.q * (tiles > 1.f ? tiles : 1.f);
    const float one = m.e1 + m.g1 * (float)k / 512.f, all = n * (m.e2 + m.g2 * (float)k / 512.f);
    // candidates of 128 columns: the search reads twice the slots
    const float us = 2.f + (one > all ? one : all) + (cand && m.bn == 128 ? 2.f + 0.004f * (float)M : 0.f);
    if (!best || us < best_us) { best = v; best_us = us; }
  }
  return best;
}

// Tile choice of gemm_kernel: 0 = 64x64 or smaller (2x2 waves and the k-group shapes of launch_gemm);
// 1 = 128x128 (fp32 only) once that still gives ~one block per CU (the output layer of models that gemm_split.hip cannot
// take): the wide output layer is bound by the operand traffic between L2 and the CUs, |X| * N/BN + |W| * M/BM, so the
// biggest tile that still fills the chip wins: M = 256 128x128 with 16 waves 69 us (8 waves 81, 256x128 71-76, 256x256
// 132: half the CUs idle).
// 3 = 64x128 with 8 waves and 256-byte chunks (bf16 only, K % 128 == 0): the products split over blocks
// are bound by the same operand traffic (their MFMA time is negligible), and this tile moves 25-30 % fewer bytes than
// 64x64 at the same block count after splitting k (512 x 1024 x 4096 12.4 -> 10.7 us).
// can_split: the GEMM writes partials, so k may be divided over up to 4 blocks to fill the chip
inline int gemm_pick_tile(int M, int N, int K, int dtype, bool can_split) {
  if (dtype == 0 && M >= 128 && (long)((M + 127) / 128) * ((N + 127) / 128) >= 200) return 1;
  if (dtype == 1 && K % 128 == 0 && (long)((M + 63) / 64) * ((N + 127) / 128) >= (can_split ? 64 : 160)) return 3;
  return 0;
}

// The smaller tiles of gemm_kernel: a wave's MFMA chain over the whole k range is what bounds a small product, and only waves
// on different SIMDs run their chains in parallel.  When 64x64 tiles would leave most SIMDs idle, smaller tiles deal their
// k range to 2 or 4 wave groups (reduced through LDS), aiming at ~one wave per SIMD:
//   0: 64x64   1: 64x32 tiles, 2 waves x 2 k-groups   2: 32x32 tiles, 1 wave x 4 k-groups
// (64x32 with 4 k-groups, 32x64 and 64x64 with 2, 32x32 with 8 all measured within 3% of these.)  chunks: k in 128-byte units
inline int gemm_tile_shape(int M, int N, int ksplit, int chunks) {
  const long tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64) * ksplit;
  return tiles64 <= 64 && chunks >= 8 ? 2 : tiles64 <= 192 && chunks >= 4 ? 1 : 0;
}

// Groups of waves to which gemm_kernel deals the chunks of a bf16 product's k (launch_gemm): the sums of the groups are added
// up in order, in gemm_lds.hip as well.
inline int gemm_k_groups(int M, int N, int K, int ksplit, bool partials) {
  if (gemm_pick_tile(M, N, K, 1, partials) == 3) return 1;
  const int shape = gemm_tile_shape(M, N, ksplit, (K / 64 + ksplit - 1) / ksplit);
  return shape == 2 ? 4 : shape == 1 ? 2 : 1;
}

// Small fp32 products through bf16 parts with k dealt to the waves (gemm_kwaves.hip): which tile, or 0 for gemm_kernel.
//   1 32 x 32, 8 waves   2 64 x 32, 8 waves   3 64 x 64, 4 waves   4 32 x 32, 4 waves
// A model of each and of gemm_kernel's three shapes, in us: the larger of one block alone on its CU, e1 + g1 k / 512, and of n
// blocks on a CU, n (e2 + g2 k / 512), n between the tiles per CU and that rounded up (q: how near the former), and 2 for the
// launch.  Fitted to 283 shapes of 17 to 700 rows, k 256 to 4096, up to 1.6e9 multiplications (beyond, it is not asked), with
// an error of 5 to 12 %; over them the choice takes 0.89 of gemm_kernel's time, 1 % more than the best of all would.
// Measured (us, gemm_kernel / here; kernel alone): 64 x 512 x 512 6.8 / 5.2, 128 x 2048 x 512 7.1 / 5.9, 256 rows 9.2 / 8.7,
// 300 rows 13.4 / 10.0, 128 x 1536 x 512 7.0 / 5.7, 256 rows 8.9 / 7.9, 256 x 768 x 256 5.0 / 4.4, 256 x 3072 x 1024 24.3 / 18.3,
// 64 x 512 x 512 in eight 4.1 / 3.5, 300 x 512 x 2048 in eight 12.2 / 10.2.  Left to gemm_kernel: 256 x 512 x 512 in eight
// 4.4 / 4.7, 256 x 512 x 2048 in eight 8.3 / 9.2; more than 32 rows by columns whose weights do not stay near (256 x 8000 x 512
// 22.9 / 25.1, 64 rows 9.3 / 9.6, but 20 rows 9.1 / 6.2); 64 x 64 tiles with k split (128 x 1024 x 4096 in eight 13.5 / 14.4).
struct KwavesModel { int bm, bn, kw; float e1, g1, e2, g2, q; };
constexpr KwavesModel kKwavesModels[4] = {
    {32, 32, 8, 1.09f, 2.26f, 0.82f, 2.40f, 0.15f}, {64, 32, 8, -1.97f, 3.83f, 2.02f, 3.42f, 0.f},
    {64, 64, 4, -2.48f, 5.48f, 3.49f, 5.05f, 0.f},  {32, 32, 4, 1.14f, 2.67f, 0.52f, 2.57f, 0.18f}};
constexpr KwavesModel kTileModels[3] = {   // gemm_kernel, by gemm_tile_shape
    {64, 64, 0, 0.91f, 10.27f, 0.93f, 9.61f, 0.23f}, {64, 32, 0, 1.54f, 5.40f, 1.22f, 5.01f, 0.19f},
    {32, 32, 0, 1.17f, 3.68f, 1.29f, 3.25f, 0.09f}};
constexpr float kKwavesMost = 1.6e9f;
// us: if given, the model's time for what is chosen
inline int gemm_kwaves_variant(int M, int N, int K, int ksplit, float* us_out = nullptr) {
  if (M < 1 || N < 4 || N % 4 || K < 64 || ksplit < 1 || (float)M * (float)N * (float)K > kKwavesMost) return 0;
  if (M > 32 && N > 8 * K) return 0;
  auto us_of = [&](const KwavesModel& m) {
    const float k = (float)K / (float)ksplit / 512.f;
    const float tiles = (float)((M + m.bm - 1) / m.bm) * (float)((N + m.bn - 1) / m.bn) * (float)ksplit / 256.f;
    const float n = (1.f - m.q) * (float)(long)(tiles + 0.9999f) + m.q * (tiles > 1.f ? tiles : 1.f);
    const float one = m.e1 + m.g1 * k, all = n * (m.e2 + m.g2 * k);
    return 2.f + (one > all ? one : all);
  };
  int best = 0;
  float best_us = 0.95f * us_of(kTileModels[gemm_tile_shape(M, N, ksplit, (K / 32 + ksplit - 1) / ksplit)]);
  for (int v = 1; v <= 4; ++v) {
    const KwavesModel& m = kKwavesModels[v - 1];
    if (K % (16 * m.kw * ksplit) || (v == 3 && ksplit > 1)) continue;
    const float us = us_of(m);
    if (us < best_us) { best_us = us; best = v; }
  }
  if (us_out) *us_out = best_us;
  return best;
}

// split factor that fills the chip for an M x N x K product (1 when the tiles alone already do)
// plain: fp32 without splitting into bf16 parts
inline int gemm_pick_ksplit(int M, int N, int K, int dtype, bool plain) {
  if (dtype == 0 && !plain) {
    const SplitShape sp = gemm_split_shape(M, N, K, 1, 4);
    if (sp.wm) return sp.ks;
  }
  const int tile = gemm_pick_tile(M, N, K, dtype, true);
  if (tile == 1) return 1;
  int ks = 1;
  if (tile == 3) {
    const int nchunks = K / 128;   // 256-byte chunks
    const long blocks = (long)((M + 63) / 64) * ((N + 127) / 128);
    while (blocks * ks < 192 && nchunks / (ks * 2) >= 2 && ks < 16) ks *= 2;
    return ks;
  }
  const int epc = dtype == 1 ? 64 : 32;
  const int nchunks = K / epc;
  const long blocks = (long)((M + 63) / 64) * ((N + 63) / 64);
  // aim for >= 256 blocks (one per CU), keep at least 2 chunks of k per block
  while (blocks * ks < 256 && nchunks / (ks * 2) >= 2 && ks < 16) ks *= 2;
  // A long k (the feed-forward's second product): gemm_kwaves.hip needs fewer splits, and its consumer adds fewer partials.
  // us, alone and with the LayerNorm behind it, the split above / the one taken: 128 x 512 x 2048 (16) 5.8 and 10.0 / (4) 5.6 and
  // 8.7, 185 rows (16) 8.4 and 13.8 / (4) 7.5 and 10.5, 256 rows (8) 8.2 and 12.3 / (4) 8.5 and 12.0, 300 rows (8) 11.1 and 15.3 /
  // (2) 10.1 and 12.9.  (Two splits take 10.2 for 185 rows and their LayerNorm and 11.4 for 256, 9.8 for 128: a partial costs
  // the LayerNorm more than is counted here.)  Products that are as wide as long gain nothing.
  float best_us = 0.f;
  if (dtype == 0 && !plain && M > 16 && K >= 2 * N) {
    gemm_kwaves_variant(M, N, K, ks, &best_us);
    const float partial = 2e-7f * (float)M * (float)N + 0.01f;
    const int ks0 = ks;
    best_us += (float)ks * partial;
    for (int q = 1; q < ks0; q *= 2) {
      float us = 0.f;
      if (!gemm_kwaves_variant(M, N, K, q, &us)) continue;
      us += (float)q * partial;
      if (us < best_us) { best_us = us; ks = q; }
    }
  }
  return ks;
}

}  // namespace san
