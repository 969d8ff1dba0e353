// Included by the k_*.hip translation units that instantiate the GEMM kernel.
#pragma once
#include "epilogues.hpp"
#include "launch.hpp"
#include "stream_core.hpp"
#include "tile_rule.hpp"

namespace ffn24 {

// An epilogue that costs more than a store declares `static constexpr EpiCost COST` (tile_rule.hpp).
template <class E, class = void> struct epi_cost { static constexpr EpiCost value = EPI_PLAIN; };
template <class E> struct epi_cost<E, std::void_t<decltype(E::COST)>> { static constexpr EpiCost value = E::COST; };

template <bool SPARSE, class Epi, bool F8, int PROBE, int MI, int NI, int TR = 0>
static int launch_tile(const GemmArgs& g, const typename Epi::Args& ea, hipStream_t s) {
  using G = Geo<SPARSE, F8, MI, NI>;
  void (*kern)(GemmArgs, typename Epi::Args);
  if constexpr (TR != 0) kern = gemm_k_major_kernel<SPARSE, Epi, TR, MI, NI>;
  else kern = gemm_kernel<SPARSE, Epi, F8, PROBE, MI, NI>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  int nblocks = (g.M / G::BM) * (g.N / G::BN);
  if constexpr ((PROBE & PROBE_PERSIST) != 0) nblocks = nblocks < PERSIST_WORKGROUPS ? nblocks : PERSIST_WORKGROUPS;
  hipLaunchKernelGGL(kern, dim3(nblocks), dim3(GEMM_THREADS), G::LDS_TOTAL, s, g, ea);
  return (int)hipGetLastError();
}

template <bool SPARSE, class Epi, bool F8 = false, int TR = 0>
static int launch_gemm(const GemmArgs& g_in, const typename Epi::Args& ea, hipStream_t s) {
  GemmArgs g = g_in;
  g.clk = tl_gemm_clk;
  switch (pick_tile(SPARSE, F8, epi_cost<Epi>::value, g.M, g.N, g.K)) {
    case 0: return launch_tile<SPARSE, Epi, F8, 0, 4, 4, TR>(g, ea, s);
    case 1: return launch_tile<SPARSE, Epi, F8, 0, 4, 2, TR>(g, ea, s);
    case 2: return launch_tile<SPARSE, Epi, F8, 0, 2, 2, TR>(g, ea, s);
    case 3: return launch_tile<SPARSE, Epi, F8, 0, 2, 1, TR>(g, ea, s);
    default: return launch_tile<SPARSE, Epi, F8, 0, 1, 1, TR>(g, ea, s);
  }
}

template <bool SPARSE, class Epi, int TR, int MI, int NI, class Side>
static int launch_side_tile(const GemmArgs& g, const typename Epi::Args& ea, const typename Side::Args& sa, unsigned side_blocks, hipStream_t s) {
  using G = Geo<SPARSE, false, MI, NI>;
  static_assert(G::LDS_TOTAL >= FW_LDS, "what a side job needs");
  auto kern = gemm_side_kernel<SPARSE, Epi, TR, MI, NI, Side>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  const int n = (g.M / G::BM) * (g.N / G::BN);
  hipLaunchKernelGGL(kern, dim3((unsigned)n + side_blocks), dim3(GEMM_THREADS), G::LDS_TOTAL, s, g, ea, n, sa);
  return (int)hipGetLastError();
}

// A bf16 GEMM with other work in the same launch (gemm_side_kernel) where side_rides says so; *rode tells.
template <bool SPARSE, class Epi, int TR, class Side>
static int launch_gemm_side(const GemmArgs& g, const typename Epi::Args& ea, const typename Side::Args& sa, unsigned side_blocks, bool* rode, hipStream_t s) {
  const int tile = pick_tile(SPARSE, false, epi_cost<Epi>::value, g.M, g.N, g.K);
  *rode = side_rides(SPARSE, tile, g.M, g.N, g.K);
  if (!*rode) return 0;
  switch (tile) {
    case 2: return launch_side_tile<SPARSE, Epi, TR, 2, 2, Side>(g, ea, sa, side_blocks, s);
    case 3: return launch_side_tile<SPARSE, Epi, TR, 2, 1, Side>(g, ea, sa, side_blocks, s);
    default: return launch_side_tile<SPARSE, Epi, TR, 1, 1, Side>(g, ea, sa, side_blocks, s);
  }
}
template <class Epi, int MI, int NI, bool SHIFT>
static int launch_rows_tile(const GemmArgs& g, const typename Epi::Args& ea, hipStream_t s) {
  using G = GeoRows<MI, NI>;
  static_assert(ROWS_MIN_K / G::BK >= G::NB, "the kernel fills its ring before it starts");
  auto kern = gemm_rows_kernel<Epi, MI, NI, SHIFT>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  hipLaunchKernelGGL(kern, dim3((g.M / G::BM) * (g.N / G::BN)), dim3(GEMM_THREADS), G::LDS_TOTAL, s, g, ea);
  return (int)hipGetLastError();
}

// A 2:4 operand and a dense one as a caller has them, row-major (gemm_rows_kernel), bf16, K >= ROWS_MIN_K.
template <class Epi>
static int launch_gemm_rows(const GemmArgs& g, const typename Epi::Args& ea, hipStream_t s) {
  switch (pick_tile(true, false, EPI_PLAIN, g.M, g.N, g.K, 1, true)) {
    case 0: return launch_tile<true, Epi, false, 0, 4, 4>(g, ea, s);
    case 1: return launch_rows_tile<Epi, 4, 2, false>(g, ea, s);
    case 2: return launch_rows_tile<Epi, 2, 2, false>(g, ea, s);
    case 3: return g.K % 128 ? launch_rows_tile<Epi, 2, 1, true>(g, ea, s) : launch_rows_tile<Epi, 2, 1, false>(g, ea, s);
    default: return launch_rows_tile<Epi, 1, 1, false>(g, ea, s);
  }
}

template <bool SPARSE, class EpiA, class EpiB, bool F8, int MI, int NI, int TR>
static int launch_duo_tile(const GemmArgs& ga, const typename EpiA::Args& ea, const GemmArgs& gb, const typename EpiB::Args& eb, hipStream_t s) {
  using G = Geo<SPARSE, F8, MI, NI>;
  auto kern = gemm_duo_kernel<SPARSE, EpiA, EpiB, F8, MI, NI, TR>;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), G::LDS_TOTAL, configured)) return rc;
  const int n = (ga.M / G::BM) * (ga.N / G::BN);
  hipLaunchKernelGGL(kern, dim3(2 * n), dim3(GEMM_THREADS), G::LDS_TOTAL, s, ga, ea, n, gb, eb);
  return (int)hipGetLastError();
}

// Two GEMMs of the same M, N, K and operand forms (gemm_duo_kernel), with the tile that suits both together.
template <bool SPARSE, class EpiA, class EpiB, bool F8 = false, int TR = 0>
static int launch_gemm_duo(const GemmArgs& ga, const typename EpiA::Args& ea, const GemmArgs& gb, const typename EpiB::Args& eb, hipStream_t s) {
  const int tile = pick_tile(SPARSE, F8, EPI_PLAIN, ga.M, ga.N, ga.K, 2);
  const long long n = tile_count(TILES_SPARSE[0], ga.M, ga.N);
  if (tile == 0 && (n % CHIP_CUS == 0 || apart_is_better(F8, n, ga.K, 1))) {   // (whole rounds each: nothing to share)
    const int rc = launch_tile<SPARSE, EpiA, F8, 0, 4, 4, TR>(ga, ea, s);   // (the tile one of them takes alone, too)
    return rc ? rc : launch_tile<SPARSE, EpiB, F8, 0, 4, 4, TR>(gb, eb, s);
  }
  switch (tile) {
    case 0: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 4, 4, TR>(ga, ea, gb, eb, s);
    case 1: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 4, 2, TR>(ga, ea, gb, eb, s);
    case 2: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 2, 2, TR>(ga, ea, gb, eb, s);
    case 3: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 2, 1, TR>(ga, ea, gb, eb, s);
    default: return launch_duo_tile<SPARSE, EpiA, EpiB, F8, 1, 1, TR>(ga, ea, gb, eb, s);
  }
}

template <class Epi, bool F8, int MI, int NI, int TR>
static int launch_pair_tile(const PairSet<Epi>& a, const PairSet<Epi>& b, int sets, hipStream_t s) {
  using GS = Geo<true, F8, MI, NI>;
  using GD = Geo<false, F8, MI, NI>;
  auto kern = gemm_pair_kernel<Epi, F8, MI, NI, TR>;
  constexpr int lds = GS::LDS_TOTAL > GD::LDS_TOTAL ? GS::LDS_TOTAL : GD::LDS_TOTAL;
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, configured)) return rc;
  const int nd = (a.gd.M / GD::BM) * (a.gd.N / GD::BN), ns = (a.gs.M / GS::BM) * (a.gs.N / GS::BN);
  hipLaunchKernelGGL(kern, dim3(sets * (nd + ns)), dim3(GEMM_THREADS), lds, s, a, b, sets, nd, ns);
  return (int)hipGetLastError();
}

// a dense and a sparse GEMM in one launch (gemm_pair_kernel), or two such sets of the same sizes; b is read with sets == 2 only
template <class Epi, bool F8 = false, int TR = 0>
static int launch_gemm_pair(const PairSet<Epi>& a_in, const PairSet<Epi>& b, int sets, hipStream_t s) {
  if (sets == 2 && apart_is_better(F8, tile_count(TILES_DENSE[0], a_in.gd.M + a_in.gs.M, a_in.gs.N), a_in.gs.K, 2)) {
    const int rc = launch_gemm_pair<Epi, F8, TR>(a_in, a_in, 1, s);
    return rc ? rc : launch_gemm_pair<Epi, F8, TR>(b, b, 1, s);
  }
  PairSet<Epi> a = a_in;
  a.gs.clk = tl_gemm_clk;
  switch (pick_pair_tile(F8, a.gd.M, a.gs.M, a.gs.N, a.gs.K, sets)) {
    case 0: return launch_pair_tile<Epi, F8, 4, 4, TR>(a, b, sets, s);
    case 1: return launch_pair_tile<Epi, F8, 4, 2, TR>(a, b, sets, s);
    case 2: return launch_pair_tile<Epi, F8, 2, 2, TR>(a, b, sets, s);
    case 3: return launch_pair_tile<Epi, F8, 2, 1, TR>(a, b, sets, s);
    default: return launch_pair_tile<Epi, F8, 1, 1, TR>(a, b, sets, s);
  }
}

}  // namespace ffn24
