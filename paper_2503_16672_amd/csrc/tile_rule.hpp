// Rules on sizes: which block tile a GEMM takes, and which tile a feature-wise re-compression (host code, no HIP: it compiles by itself).
#pragma once

namespace ffn24 {

// The 256 x 256 tile does the least operand traffic per matrix op, but a shape with fewer than 256 of them leaves CUs idle and one
// with, say, 300 makes half of them do two while the others wait; the smaller tiles cost more per output element and spread better.
// The rule estimates, for every tile, (tiles a CU gets, rounded up) x (K x time per k + time of fill and epilogue) and takes the least,
// preferring the larger tile within 3 %.  A stage of an fp8 kernel holds twice the k in the same bytes and time.
// The constants are effective ones: fitted to whole steps in a sustained loop on one MI355X (a round of 256 x 256 tiles runs at the power
// limit there, and a last round that leaves CUs idle at a higher clock, which single launches do not show), with one GEMM at a time taken
// off the 256 x 256 tile, over 136 shapes: T 256-16384, D 256-5632, F 1024-16384, 0.08 to 6.8 rounds of 256 x 256 tiles in the up-projection,
// bf16 and both fp8 recipes, 2:4 and dense.  The fit is of before the small tiles read a whole stage ahead and the epilogues went through LDS.
// What it is worth with the present kernels, at 40 other shapes (T 256-14080, D 256-5120, F 1024-16384, 0.03 to 5.5 rounds): of 280 steps
// and forwards (seven kinds) none takes more than 0.5 % longer than with 256 x 256 tiles throughout, and the mean (geometric) is 1.45 x
// faster.  GEMM by GEMM, each of the five tiles in whole steps: 78 % of 480 choices cost at most 0.4 % of a step over the best one, 90 % at most
// 2 %; the worst are 7.2 and 6.0 % (T 1792 D 2304 F 6400, dense and bf16 step: 128 x 128 where 256 x 256 is the better), the others
// above 3 % mostly small shapes that take a tile one size too large and weight gradients of half a round that are faster on 128 x 128.
// The 256 x 256 tile has since been given the 16 x 16 matrix ops (gemm_core.hpp) and gained 2-6 % on the others.  Looked at again, 88 training steps (four kinds,
// T 256-16384, D 512-4864, F 1024-16384), with every GEMM one tile smaller, one larger, or 256 x 256: 76 are within 0.5 % of the best of the four, the worst 3.5 % from it
// (row-wise fp8, 768 768 3072: 65.7 us, 63.5 with the smaller tiles), the worst that would gain from 256 x 256 2.0 % (dense 12288 2048 6144: 1549, 1518); the
// mean against 256 x 256 throughout is 1.31 x, the least 0.98.
// What the rule avoids: a bf16 step at T 2304 D 4864 F 15616 (2.1 rounds) is 1.8 % longer with 256 x 128 up-projection and dH than with 256 x 256.
struct TileCost { int mi, ni, per_k, fixed; };   // 0.1 ns per (bf16) k; ns per tile
constexpr TileCost TILES_SPARSE[] = {{4, 4, 140, 6000}, {4, 2, 92, 5000}, {2, 2, 57, 3000}, {2, 1, 39, 2000}, {1, 1, 26, 1500}};
constexpr TileCost TILES_DENSE[] = {{4, 4, 205, 19000}, {4, 2, 132, 5000}, {2, 2, 84, 1750}, {2, 1, 52, 2000}, {1, 1, 34, 1000}};
constexpr int NUM_TILES = 5;   // the tables list the same tiles
constexpr long long CHIP_CUS = 256;

// What an epilogue adds to the fill and store of the two largest dense tiles (ns).  The fp8 epilogues scale or quantise every value beside
// 256 accumulators, and half the reduction time covers it less.  The dense row-wise one spills 42 registers on the 256 x 128 tile and 6 on the
// 256 x 256 (44 and 22 when these were fitted): the two were equal at 1.8-2.6 rounds (544 us either way at T 5888 D 2304 F 5120, 690 and 691 at T 7168 D 2048 F 6144), where
// the accumulators alone would make 256 x 128 the better.
struct EpiCost { int t256x256, t256x128; };
constexpr EpiCost EPI_PLAIN = {0, 0}, EPI_FP8 = {3000, 0}, EPI_FP8_SPILLS = {3000, 8000};

// The same for a caller's row-major 2:4 operand (spmm24) with K >= ROWS_MIN_K, single launches: 256 x 256 with the main loop of the panel forms,
// the others with gemm_rows_kernel, whose slots take whole lines of the rows and do not fit the LDS with 256 x 256.  Fitted to 70 shapes (M 256-8192, N
// 256-4096, K 256-16384).  At 21 other M x N and K 2048-16384, even and odd multiples of 64, the choice is the fastest of the five but for one,
// 3 % from it, and no slower anywhere than the kernels of the panel forms with their rule: 1.0-1.45 x (K 4096: M N 512 14.8 -> 12.3 us, M 2048 N
// 1024 26.5 -> 19.2, M N 2048 32.8 -> 27.7, M 4096 N 2048 50.1 -> 44.2; from 130 tiles of 256 x 256 on the same kernel).
// The line is on the safe side.  Short reductions have little to gain in slots and lose where the larger slots leave one workgroup on a CU
// that took two (M N 1536 K 256 4.6 -> 5.1 us, M 8192 N 4096 K 512 on 128 x 128 33 -> 42); between K 1024 and 1984 single launches would gain
// 3-20 % (M 2048 N 1024 K 1536 10.8 -> 9.0), or 0.3-1.5 us, of which a caller that is bound by its launches sees nothing.
constexpr int ROWS_MIN_K = 2048;
constexpr TileCost TILES_ROWS[] = {{4, 4, 155, 5000}, {4, 2, 105, 3700}, {2, 2, 62, 2000}, {2, 1, 39, 2100}, {1, 1, 28, 400}};

inline long long tile_time(const TileCost& t, int K, bool f8) { return (long long)(f8 ? K / 2 : K) * t.per_k / 10 + t.fixed; }
inline long long tile_count(const TileCost& t, int M, int N) { return (long long)(M / (64 * t.mi)) * (N / (64 * t.ni)); }

inline int pick_tile(bool sparse, bool f8, EpiCost epi, int M, int N, int K, int gemms = 1, bool rows = false) {   // gemms: that many of this size share the launch
  int best = 0;
  long long best_time = 0;
  for (int i = 0; i < NUM_TILES; i++) {
    const TileCost& t = rows ? TILES_ROWS[i] : sparse ? TILES_SPARSE[i] : TILES_DENSE[i];
    const long long one = tile_time(t, K, f8) + (i == 0 ? epi.t256x256 : i == 1 ? epi.t256x128 : 0);
    const long long time = (gemms * tile_count(t, M, N) + CHIP_CUS - 1) / CHIP_CUS * one;
    if (i == 0 || time * 100 < best_time * 97) { best = i; best_time = time; }
  }
  return best;
}

// Two launches of n 256 x 256 tiles each (a weight gradient; with the split the dense and the sparse tiles of one) that could be one go out
// one after the other where sharing saves no round of the chip and the reduction is long: the other's operands then no longer share the
// L2 with the first's for as long as the launches overlap, and the gap between them is short beside them.  Measured, together -> apart:
// K = T = 6912, 3.8 rounds each: bf16 step 3539 -> 3512 us, split 3655 -> 3616; K 3584, 2.6 rounds: 1384 -> 1367; K 7680, 1.6 rounds, fp8
// row-wise: 1046 -> 1032.  Short reductions like one launch (K 256-2048, 1.9-3.8 rounds: 0.5-2.5 % of a step), fp8 up to K 5888.  With
// the split whole rounds of tiles are together too: its dense tiles outlast their round (K 4096, 2 rounds: 1117 us, 1138 apart).
inline bool apart_is_better(bool f8, long long n, int K, int min_rounds) {
  const long long one = (n + CHIP_CUS - 1) / CHIP_CUS, both = (2 * n + CHIP_CUS - 1) / CHIP_CUS;
  return n >= min_rounds * CHIP_CUS && n % CHIP_CUS != 0 && both == 2 * one && (f8 ? K : 2 * K) >= 6144;
}

// The feature-wise re-compression in one launch with the dX GEMM (M x N, reduction K; the re-compression goes over M x K): where the tiles, of a kind that
// shares a CU, leave places free from the start, and the GEMM is short.  Apart, together, whole steps (us, T D F).  64 x 64 tiles: 256 512 2048 35.7, 33.5; 1536
// 512 2048 46.7, 45.4; 768 768 3072 59.3, 58.5; 1280 768 3072 65.9, 65.4; 512 1024 4096 62.5, 62.2.  128 x 64: 4096 512 1024 50.3, 48.9; 8192 256 512 52.2, 50.7.
// 128 x 128: 8192 512 512 61.4, 59.8; 2304 1024 1280 65.3, 64.9; 4096 1024 1024 69.3, 67.9; 3072 1024 1280 71.8, 70.9.  Beyond the lines 1024 1024 4096 78.0, 78.8; 2048 1024
// 2048 69.0, 70.1; 1536 1024 2560 74.4, 75.5; 2048 768 3072 83.8, 86.1; 2048 512 4096 79.7, 80.6; 1024 1536 2048 64.9, 65.9; 1280 1280 5120 121.5, 126.3.
inline bool side_rides(bool sparse, int tile, int M, int N, int K) {
  return tile >= 2 && tile_count(sparse ? TILES_SPARSE[tile] : TILES_DENSE[tile], M, N) <= CHIP_CUS && (long long)M * K <= 1 << 22 && N <= 1024 &&
         (K <= 1280 || (long long)M * N * K <= 3LL << 30);
}

// A matrix read k-major as the B operand saves the pass that would re-arrange it, but the lanes of a 256 x 256 tile exchange their accumulators before they
// are stored, 2.2-3.5 us for every round of the chip and GEMM, which a pass over a matrix that is small beside the result does not cost.
// GEMMs: of that many results of `values` each; pass_ns: what the pass takes.
inline bool in_place_is_better(long long values, int gemms, long long pass_ns) { return values < 2LL << 24 || gemms * 2900 * values >> 24 <= pass_ns; }

// Weight gradients (D x F from T tokens; the pass goes over dY and X).  In place / copies, bf16 backwards (us, T D F): 256 4096 16384 238, 220; 1024
// 4096 16384 435, 419; 2048 4096 16384 687, 670; 4096 4096 16384 1184, 1184; 256 8192 28672 703, 628; 2048 8192 28672 2204, 2131; 256 4096 8192 124, 118;
// 512 8192 4096 164, 170; 3072 4096 8192 516, 513; 8192 4096 8192 1172, 1186; 16384 4096 8192 2275, 2353.  Below two rounds copies gain nothing that can be
// told from noise and lose up to 20 % where launches count (512 512 2048 19.3, 23.4; 512 2048 12288 121, 122; dense 119, 133).
// Few columns and a 2:4 operand: tiles of 64 columns read 128 bytes of a token's row at a time, which is slower than panels once the step's
// tensors (6 T D + 4 1/4 T F bytes) no longer fit the last-level cache: 65536 512 512 349, 305; 65536 512 1024 451, 416; 65536 256 1024 352, 308; 131072 256 512
// 627, 524; 262144 512 512 1460, 1364; still within it 32768 512 512 136, 154; 65536 256 256 188, 209; more columns 131072 768 768 971, 1047; 131072 512 2048
// 1290, 1305; dense 65536 512 512 425, 420, 65536 512 1024 525, 538.
inline bool acts_in_place(long long T, long long D, long long F, bool dense) {
  if (!dense && D <= 512 && D * F <= 1 << 19 && T * (6 * D + 17 * F / 4) > 1 << 28) return false;
  return in_place_is_better(D * F, 2, 5000 + T * D / 625);
}
// The weights in a forward, for W2 as the down-projection's B (keep: the context copies them in any case, for the backward).  In place / copies (us, T D F):
// 65536 2048 512 262, 236; 131072 1024 512 281, 265; 16384 8192 1024 423, 375; 65536 4096 1024 767, 732; level 131072 1024 4096 1512, 1498.
inline bool weights_in_place(long long T, long long D, long long F, bool keep) { return in_place_is_better(T * D, 1, keep ? D * F / 1150 : 5000 + D * F / 625); }

// The tile of a dense and a sparse GEMM in one launch (same N and K, the dense tiles first), `sets` times: all tiles over the CUs, but no
// less than the dense ones take by themselves (their epilogue is a plain store, and their tiles share CUs with sparse ones instead of
// running in full rounds: the time per k of single launches).  The two parts make the estimate rougher, so a
// smaller tile has to promise 10 % (fp8, T 8192 D 2048 F 8192, 512 dense features: 98.4 us with 256 x 256 and 99.0 with 256 x 128, which
// the estimate puts 7 % ahead).
constexpr int PAIR_DENSE_PER_K[] = {205, 125, 74, 52, 34};
inline int pick_pair_tile(bool f8, int Md, int Ms, int N, int K, int sets) {
  int best = 0;
  long long best_time = 0;
  for (int i = 0; i < NUM_TILES; i++) {
    const long long nd = sets * tile_count(TILES_DENSE[i], Md, N), ns = sets * tile_count(TILES_SPARSE[i], Ms, N);
    const long long ts = tile_time(TILES_SPARSE[i], K, f8), td = tile_time({0, 0, PAIR_DENSE_PER_K[i], TILES_SPARSE[i].fixed}, K, f8);
    long long time = (nd + ns + CHIP_CUS - 1) / CHIP_CUS * ts;
    const long long dense = (nd + CHIP_CUS - 1) / CHIP_CUS * td, even = (nd * td + ns * ts) / CHIP_CUS;
    time = time > dense ? time : dense;
    time = time > even ? time : even;
    if (i == 0 || time * 100 < best_time * 90) { best = i; best_time = time; }
  }
  return best;
}

// quantise_e4m3 per column (k_stream.hip): in one launch that holds strips of 32 columns in registers, or in three that read the matrix twice.
// Three launches cost 5 us more to begin with; a strip keeps a workgroup of 1024 for 5 us and more whatever it holds, and its rows are half
// lines.  So the strips win while they are few: one round of two workgroups a CU (16384 columns) up to 640 rows, whose registers that allows, one
// workgroup a CU (8192 columns) up to 1536.  From 1024 rows on they win again where the matrix is larger than the caches and the second
// reading costs, until the strips' partial lines do.  Three launches / one (R x C): 1 x 16384 1.34, 1 x 32768 0.78, 8 x 2^20 0.05, 512 x 8192 1.70, 512 x
// 16384 1.22, 512 x 20480 0.88, 512 x 131072 0.85; 640 x 16384 1.05, 640 x 32768 0.96; 1024 x 8192 1.49, 1024 x 9216 0.93, 1024 x 24576 1.08, 1024 x 65536
// 1.16, 1024 x 98304 0.94; 1536 x 8192 1.20, 1536 x 10240 0.78, 1536 x 14336 1.07, 1536 x 32768 1.35, 1536 x 65536 0.98.  Beyond 1536 rows the registers run out
// (8192 x 12896 93 -> 130 us) or the CUs idle (2048 x 4096 13.4 -> 14.4, 4096 x 1024 12.1 -> 15.8).
inline bool held_columns(long long R, long long C) {
  if (R <= 640 && C <= 16384) return true;
  return R <= 1536 && (C <= 8192 || (R >= 768 && R * C >= 5 << 22 && R * C <= 1 << 26));
}

// Row-major feature-wise re-compression (k_stream.hip): 64 x 64 tiles, 3-4 us whatever there is to do, up to 2^22 elements; above, tiles of
// 128 tokens x 256 features, which move whole lines but keep a workgroup busy for 7.5 us.  Measured, 64 x 64 against 128 x 256, with
// dZ: 128 x 64 2.8 / 7.4 us, 128 x 16384 4.6 / 9.3, 1280 x 3200 9.1 / 10.0, 2048 x 2048 7.8 / 9.8; 5248 x 896 10.7 / 9.8, 1792 x 3712 13.1 / 10.3.
inline bool featurewise_small(long long T, long long F) { return T * F <= 1 << 22; }

}  // namespace ffn24
