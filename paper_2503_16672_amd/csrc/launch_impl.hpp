// Included by the k_*.hip translation units that instantiate the GEMM kernel.
#pragma once
#include "epilogues.hpp"
#include "launch.hpp"

namespace ffn24 {

// Which block tile a GEMM takes.  The 256 x 256 tile does the least operand traffic per matrix op, but a shape with fewer than 256 of
// them leaves CUs idle and one with, say, 300 makes half of them do two while the others wait; the smaller tiles cost more per
// output element and spread better.  The rule estimates, for every tile, (tiles a CU gets, rounded up) x (K x time per k + time
// of fill and epilogue) and takes the least, preferring the larger tile within 3 %.  The constants are measured (median launch
// times on one MI355X at (T, D, F) from (256, 512, 2048) to (16384, 4096, 16384), both precisions): over all 132 GEMMs of six such
// shapes the rule's choices sum to 1.001 x the best choice of each, and the 256 x 256 tile alone to 1.24 x.  Examples (us, 256 x 256 ->
// the choice): sparse down-projection T 1024 D 1024 F 4096 55 -> 17.5 (64 x 64); dense T 4096 D 2048 F 8192 166 -> 109 (256 x 128);
// up-projection T 1280 D 768 F 3072 29 -> 15 (128 x 128).  A stage of an fp8 kernel holds twice the k in the same bytes and time.
struct TileCost { int mi, ni, per_k, fixed; };   // 0.1 ns per (bf16) k; ns per tile
constexpr TileCost TILES_SPARSE[] = {{4, 4, 140, 6000}, {4, 2, 92, 5000}, {2, 2, 57, 3000}, {2, 1, 39, 2000}, {1, 1, 26, 1500}};
constexpr TileCost TILES_DENSE[] = {{4, 4, 205, 19000}, {4, 2, 125, 5000}, {2, 2, 74, 2500}, {2, 1, 52, 2000}, {1, 1, 34, 1000}};
constexpr int NUM_TILES = 5;   // the two tables list the same tiles
constexpr long long CHIP_CUS = 256;

inline long long tile_time(const TileCost& t, int K, bool f8) { return (long long)(f8 ? K / 2 : K) * t.per_k / 10 + t.fixed; }
inline long long tile_count(const TileCost& t, int M, int N) { return (long long)(M / (64 * t.mi)) * (N / (64 * t.ni)); }

inline int pick_tile(bool sparse, bool f8, int M, int N, int K, int gemms = 1) {   // gemms: that many of this size share the launch
  int best = 0;
  long long best_time = 0;
  for (int i = 0; i < NUM_TILES; i++) {
    const TileCost& t = sparse ? TILES_SPARSE[i] : TILES_DENSE[i];
    const long long time = (gemms * tile_count(t, M, N) + CHIP_CUS - 1) / CHIP_CUS * tile_time(t, K, f8);
    if (i == 0 || time * 100 < best_time * 97) { best = i; best_time = time; }
  }
  return best;
}

// The same for a dense and a sparse GEMM in one launch (same N and K, the dense tiles first): all tiles over the CUs, but no less than
// the dense ones take by themselves (their epilogue is a plain store here, not one of the fused ones the dense table is priced for).
// The two parts make the estimate rougher, so a smaller tile has to promise 10 % (fp8, T 8192 D 2048 F 8192, 512 dense features:
// 98.4 us with 256 x 256 and 99.0 with 256 x 128, which the estimate puts 7 % ahead).
inline int pick_pair_tile(bool f8, int Md, int Ms, int N, int K, int sets) {
  int best = 0;
  long long best_time = 0;
  for (int i = 0; i < NUM_TILES; i++) {
    const long long nd = sets * tile_count(TILES_DENSE[i], Md, N), ns = sets * tile_count(TILES_SPARSE[i], Ms, N);
    const long long ts = tile_time(TILES_SPARSE[i], K, f8), td = tile_time(TILES_DENSE[i], K, f8) - TILES_DENSE[i].fixed + TILES_SPARSE[i].fixed;
    long long time = (nd + ns + CHIP_CUS - 1) / CHIP_CUS * ts;
    const long long dense = (nd + CHIP_CUS - 1) / CHIP_CUS * td, even = (nd * td + ns * ts) / CHIP_CUS;
    time = time > dense ? time : dense;
    time = time > even ? time : even;
    if (i == 0 || time * 100 < best_time * 90) { best = i; best_time = time; }
  }
  return best;
}

template <bool SPARSE, class Epi, bool F8, int PROBE, int MI, int NI>
static int launch_tile(const GemmArgs& g, const typename Epi::Args& ea, hipStream_t s) {
  using G = Geo<SPARSE, F8, MI, NI>;
  auto kern = gemm_kernel<SPARSE, Epi, F8, PROBE, MI, NI>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  int nblocks = (g.M / G::BM) * (g.N / G::BN);
  if constexpr ((PROBE & PROBE_PERSIST) != 0) nblocks = nblocks < PERSIST_WORKGROUPS ? nblocks : PERSIST_WORKGROUPS;
  hipLaunchKernelGGL(kern, dim3(nblocks), dim3(GEMM_THREADS), G::LDS_TOTAL, s, g, ea);
  return (int)hipGetLastError();
}

template <bool SPARSE, class Epi, bool F8 = false>
static int launch_gemm(const GemmArgs& g_in, const typename Epi::Args& ea, hipStream_t s) {
  GemmArgs g = g_in;
  g.clk = tl_gemm_clk;
  switch (pick_tile(SPARSE, F8, g.M, g.N, g.K)) {
    case 0: return launch_tile<SPARSE, Epi, F8, 0, 4, 4>(g, ea, s);
    case 1: return launch_tile<SPARSE, Epi, F8, 0, 4, 2>(g, ea, s);
    case 2: return launch_tile<SPARSE, Epi, F8, 0, 2, 2>(g, ea, s);
    case 3: return launch_tile<SPARSE, Epi, F8, 0, 2, 1>(g, ea, s);
    default: return launch_tile<SPARSE, Epi, F8, 0, 1, 1>(g, ea, s);
  }
}

template <bool SPARSE, class EpiA, class EpiB, bool F8, int MI, int NI>
static int launch_duo_tile(const GemmArgs& ga, const typename EpiA::Args& ea, const GemmArgs& gb, const typename EpiB::Args& eb, hipStream_t s) {
  using G = Geo<SPARSE, F8, MI, NI>;
  auto kern = gemm_duo_kernel<SPARSE, EpiA, EpiB, F8, MI, NI>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  const int n = (ga.M / G::BM) * (ga.N / G::BN);
  hipLaunchKernelGGL(kern, dim3(2 * n), dim3(GEMM_THREADS), G::LDS_TOTAL, s, ga, ea, n, gb, eb);
  return (int)hipGetLastError();
}

// Two GEMMs of the same M, N, K and operand forms (gemm_duo_kernel), with the tile that suits both together.  Where that is the 256 x 256
// tile and each of them fills the chip by itself, there is nothing to gain and they go out one after the other.
template <bool SPARSE, class EpiA, class EpiB, bool F8 = false>
static int launch_gemm_duo(const GemmArgs& ga, const typename EpiA::Args& ea, const GemmArgs& gb, const typename EpiB::Args& eb, hipStream_t s) {
  const int tile = pick_tile(SPARSE, F8, ga.M, ga.N, ga.K, 2);
  if (tile == 0 && tile_count(TILES_SPARSE[0], ga.M, ga.N) % CHIP_CUS == 0) {
    const int rc = launch_gemm<SPARSE, EpiA, F8>(ga, ea, s);
    return rc ? rc : launch_gemm<SPARSE, EpiB, F8>(gb, eb, s);
  }
  switch (tile) {
    case 0: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 4, 4>(ga, ea, gb, eb, s);
    case 1: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 4, 2>(ga, ea, gb, eb, s);
    case 2: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 2, 2>(ga, ea, gb, eb, s);
    case 3: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 2, 1>(ga, ea, gb, eb, s);
    default: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 1, 1>(ga, ea, gb, eb, s);
  }
}

template <class Epi, bool F8, int MI, int NI>
static int launch_pair_tile(const PairSet<Epi>& a, const PairSet<Epi>& b, int sets, hipStream_t s) {
  using GS = Geo<true, F8, MI, NI>;
  using GD = Geo<false, F8, MI, NI>;
  auto kern = gemm_pair_kernel<Epi, F8, MI, NI>;
  constexpr int lds = GS::LDS_TOTAL > GD::LDS_TOTAL ? GS::LDS_TOTAL : GD::LDS_TOTAL;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, configured)) return rc;
  const int nd = (a.gd.M / GD::BM) * (a.gd.N / GD::BN), ns = (a.gs.M / GS::BM) * (a.gs.N / GS::BN);
  hipLaunchKernelGGL(kern, dim3(sets * (nd + ns)), dim3(GEMM_THREADS), lds, s, a, b, sets, nd, ns);
  return (int)hipGetLastError();
}

// a dense and a sparse GEMM in one launch (gemm_pair_kernel), or two such sets of the same sizes; b is read with sets == 2 only
template <class Epi, bool F8 = false>
static int launch_gemm_pair(const PairSet<Epi>& a_in, const PairSet<Epi>& b, int sets, hipStream_t s) {
  PairSet<Epi> a = a_in;
  a.gs.clk = tl_gemm_clk;
  switch (pick_pair_tile(F8, a.gd.M, a.gs.M, a.gs.N, a.gs.K, sets)) {
    case 0: return launch_pair_tile<Epi, F8, 4, 4>(a, b, sets, s);
    case 1: return launch_pair_tile<Epi, F8, 4, 2>(a, b, sets, s);
    case 2: return launch_pair_tile<Epi, F8, 2, 2>(a, b, sets, s);
    case 3: return launch_pair_tile<Epi, F8, 2, 1>(a, b, sets, s);
    default: return launch_pair_tile<Epi, F8, 1, 1>(a, b, sets, s);
  }
}

}  // namespace ffn24
