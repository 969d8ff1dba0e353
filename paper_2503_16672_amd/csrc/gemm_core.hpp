// MFMA / sparse-MFMA GEMM core for gfx950 (CDNA4), bf16 operands, fp32 accumulation.
//
// One kernel template computes C[m][n] = sum_k A[m][k] * B[n][k]; both operands are K-contiguous in memory, or (bf16: a dense A, B) k-major,
// k the slow dimension, as W1, W2, X and dY come (fp8 operands that are not K-contiguous are transposed once by a streaming kernel, k_stream.hip).  Four wavefronts (2x2), each owning a
// wave tile of 32 MI x 32 NI, so a block tile is 64 MI x 64 NI.  Block tile 256x256 (MI = NI = 4: 256 accumulator
// registers per lane, pinned to the AGPR file) is the one that streams the fewest operand bytes per matrix op and carries the
// large problems; 256x128, 128x128, 128x64 and 64x64 take the shapes whose 256x256 tiles would leave CUs idle (pick_tile in
// tile_rule.hpp).  The 256x256 tile, at the power limit, uses the 16x16 matrix ops (gemm_tile_big), the smaller ones the 32x32 ops.
// An output element sums the same k in the same order in every tile, so the results are the same bit for bit.
//
//   A dense  : [M][K]                         -> v_mfma_f32_16x16x32_bf16, v_mfma_f32_32x32x16_bf16
//   A sparse : 2:4-compressed [M][K/2] + metadata [M][K/8] -> v_smfmac_f32_16x16x64_bf16, v_smfmac_f32_32x32x32_bf16
//   B        : [N][K]
//
// 2:4 operand (Sec. 1 of the paper, "Hardware-accelerated (2:4) sparsity"; Fig. 2): of every 4 consecutive K entries
// of a row only two are stored, with a 2-bit position each.  The metadata byte layout used throughout (nibble
// i0 | i1<<2 per group, even group in the low nibble) is exactly the index word the sparse MFMA consumes: a lane's
// 8 stored values of one instruction take 16 consecutive metadata bits, selected from a 32-bit register by ABID.
//
// Panel form of a 2:4 operand.  The compressed operands that the library produces for itself (never the ones a
// caller hands in) are stored by pieces: piece (r, kp) = the 32 stored values (64 bytes) and the 8 metadata bytes of
// row r for the dense k range [64 kp, 64 kp + 64), at piece index ((r / 256) * (K / 64) + kp) * 256 + r % 256.
// The 256 rows x 64 k that a block tile consumes per stage are then one contiguous 16 KiB (+ 2 KiB) run, fetched as
// full 128-byte lines, instead of 256 pieces of 64 (8) bytes that are a whole matrix row apart.  Measured: the
// sparse GEMM is bound by its global->LDS stream, and the 8-byte metadata pieces alone cost it 17 %.
//
// A dense A operand can be in panel form too: piece (r, kp) = the 32 k (64 bytes) [32 kp, 32 kp + 32) of row r,
// same piece index with K / 32 panels per row (the weight copies the library makes for itself).
//
// Data movement.  Global memory goes straight to LDS (buffer loads with LDS as their destination: no VGPR staging, no LDS store
// instructions) into a ring of stage buffers, 2-3 stages ahead of the math, so that L2/HBM latency is covered:
//   dense : stage = 32 k  (A 16 KiB + B 16 KiB), ring of 4  -> 128 KiB of the CU's 160 KiB LDS (fp8: 64 k, ring of 5, all of it)
//   sparse: stage = 64 k  (A 16 KiB stored values + 2 KiB metadata + B 32 KiB), ring of 3 -> 151 KiB
// A wave-level DMA instruction fills 1 KiB of LDS in lane order, so the swizzled, row-permuted LDS layout is
// produced by choosing which global 16 bytes each lane fetches.
//
// Lane layouts of the matrix instructions (measured on gfx950 with one-hot operands; the 16x16 ops at gemm_tile_big):
//   dense 32x32x16:  A lane l holds row l%32, k = 8*(l/32)..+7;  B lane l holds column l%32, same k;
//                    C register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.
//   sparse 32x32x32: A lane l holds row l%32 and the 8 stored values of dense k 16*(l/32)..+15;
//                    B lane l holds column l%32, registers 0..7 = k 8*(l/32)..+7, registers 8..15 = k 16+8*(l/32)..+7.
//
// Row remapping.  Which global row sits in which MFMA-tile row is free, so it is chosen to make every lane's
// accumulators contiguous in memory.  32x32 ops:  wave-tile row 16*MI*hc + 16*mi + v belongs to lane half hc, M-tile mi,
// accumulator register v (16 MI consecutive rows per lane, in groups of 4 that never straddle lanes -- the 2:4 groups of
// the fused prune epilogue);  wave-tile column NI*c + ni belongs to lane column c, N-tile ni (NI consecutive columns
// per lane).  16x16 ops: rows 32*q + 4*t + v and columns 8*c + t, 32 x 8 a lane.  The permutation is applied when a tile is brought into LDS
// or when its fragments are read.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>
#include "launch.hpp"

namespace ffn24 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(1))) const char glb_char;

constexpr int TILE_M = 256, TILE_N = 256, GEMM_THREADS = 256;
constexpr int GEMM_K_MULTIPLE = 64;   // K must be a multiple of this for both kernels

struct GemmArgs {
  const void* A;         // dense [M][K] or stored values [M][K/2]
  const uint8_t* Ameta;  // sparse only: [M][K/8]
  const void* B;         // [N][K]
  int M, N, K;           // K is the dense reduction length
  int a_panel;           // A (and its metadata) is in panel form (see above) instead of row-major
  const int* b_rowmap;   // optional: row n of B is taken from memory row b_rowmap[n] (token permutation, gathered by the DMA)
  int b_panel;           // B is in the B panel form (below) instead of row-major; not together with b_rowmap
  unsigned long long* clk;   // optional (profiling): workgroup i < CLK_SLOTS stores its own {shader-clock ticks, 100 MHz ticks} at 2 i
};

// Measurement variants of the GEMM core (bit mask; 0 = the product).  They exist so that what bounds the main loop can be
// measured with this very code -- the same DMA plan, LDS image, fragment reads and schedule -- with one ingredient taken
// out; they compute nothing useful.  Only the probe entry points of the library instantiate them.
constexpr int PROBE_NO_DMA = 1;      // no global->LDS DMA is issued (the matrix ops run on whatever the LDS holds)
constexpr int PROBE_NO_MFMA = 2;     // no matrix ops
constexpr int PROBE_NO_FRAG = 4;     // no LDS fragment reads
constexpr int PROBE_K_WRAP = 8;      // the K stages walk round the first 8 stages of the operands: every line is an L2 hit
// other tile walks (the product's is a 4 x 2 grid of 8 x 4 patches), to measure what the walk does to time and to L2 fills:
constexpr int PROBE_WALK_BANDS = 16;   // bands of 8 tile-rows, each XCD a contiguous run of tiles (the fallback walk, always)
constexpr int PROBE_WALK_8x1 = 32;     // the 8 patches of a round side by side along M
constexpr int PROBE_PATCH_4x8 = 64;    // per-XCD patches of 4 x 8 tiles
constexpr int PROBE_PATCH_16x2 = 128;  // per-XCD patches of 16 x 2 tiles
constexpr int PROBE_UNPACED = 256;     // DMA instructions on consecutive matrix-op slots (of each half of a step)
constexpr int PROBE_PERSIST = 1024;    // one workgroup per CU walks the tiles id, id + grid, ...; the next tile's first stages are asked for
                                       // before the epilogue of the present one
constexpr int PROBE_FILL_LESS = 512;   // sparse: the last 3 of a wave's 14 DMA instructions of every stage are left out -- 38 KiB a stage
                                       // instead of 50, about the bytes per matrix op of a 384 x 256 tile (what a taller tile could gain)

// B panel form: the dense panel form (64-byte pieces, a24_piece) whose rows are, inside every block of 256, stored at b_panel_pos(n): the four
// rows n .. n + 3 of a multiple of 4 at places 32 apart, rows 4 apart next to each other.
// A stage of a block tile's B operand is then one (sparse: two) contiguous 16 KiB run(s), and every DMA instruction
// reads whole 128-byte lines.  Used for every B operand the library makes itself (re-arranged weights, transposed
// activations); a caller's row-major B (spmm24; X and dY) is read as it is.
__host__ __device__ __forceinline__ int b_panel_pos(int n) { return (n & ~255) | ((n & 3) << 5) | ((n >> 2) & 31) | (n & 128); }

// piece index of row r, 64-k panel kp, for an operand with `npanels` = K / 64 panels per row
__host__ __device__ __forceinline__ size_t a24_piece(int r, int kp, int npanels) {
  return ((size_t)(r >> 8) * npanels + kp) * 256 + (r & 255);
}

// Ring depth (stages) of each tile.  256 x 256 fills the LDS by itself.  The smaller tiles keep their ring under half of the LDS where three
// stages fit, so that a second workgroup shares the CU and fills this one's barrier and epilogue gaps: a deeper ring with one workgroup
// is 10-25 % slower once a CU has two tiles to do (sparse 128 x 128, T = 4096, D = 2048, F = 8192: 103 us against 113) and no faster
// when it has one.  Sparse 256 x 128 has room for two stages a workgroup only, and those expose the memory latency (112 us; 81 us with
// four stages and the CU to itself).
constexpr int ring_depth(bool sparse, bool f8, int mi, int ni) {
  return mi * ni == 16 ? (sparse ? 3 : f8 ? 5 : 4) : mi * ni == 8 ? (sparse ? 4 : 3) : mi * ni == 4 ? (sparse ? 3 : 4) : mi * ni == 2 || !sparse ? 4 : 6;
}
// A dense 64 x 64 stage holds twice the k, in rows of 128 bytes: half the waits and barriers, and a row-major operand is read in whole
// lines (1024 x 1024, one tile a CU: K 1024 7.1 -> 6.0 us, K 4096 19.8 -> 15.0, with a row-major B too; two tiles a CU 8.1 -> 7.4, 25 -> 25, row-major
// 30 -> 26).  With larger tiles it leaves no room for a second workgroup on the CU: 128 x 64 10.7 -> 12.6 with two tiles.
constexpr bool wide_stage(int mi, int ni) { return mi * ni == 1; }
// The main loop that reads the fragments of a whole stage ahead (gemm_tile): not for the 256 x 256 tiles, whose registers are full, nor
// dense 256 x 128, which would spill 18 registers beside a second workgroup, nor sparse 128 x 128, where one tile a CU is bound
// by the operand stream already (K 4096 22.8 -> 23.9 us, 8192 41.9 -> 42.7; K 1024 9.7 -> 9.0).
constexpr bool whole_stage_ahead(bool sparse, int mi, int ni) { return sparse ? mi * ni <= 2 || mi * ni == 8 : mi * ni <= 4; }

// Stage geometry.  Everything is laid out in bytes, and an fp8 kernel has exactly the byte geometry of its bf16
// counterpart with twice the k per byte: the LDS tiles, swizzles, DMA plan and fragment addresses are shared.
template <bool SPARSE, bool F8 = false, int MI = 4, int NI = 4>
struct Geo {
  static constexpr int BM = 64 * MI, BN = 64 * NI;        // block tile: 2 x 2 waves of 32 MI x 32 NI
  static constexpr int ESIZE = F8 ? 1 : 2;
  static constexpr bool WIDE = !SPARSE && wide_stage(MI, NI);
  static constexpr bool BIG = MI * NI == 16;             // 16 x 16 matrix ops, in an order of LDS rows of its own
  static constexpr int A_ROW = WIDE ? 128 : 64;          // dense k, or the stored values of twice as many k
  static constexpr int B_ROW = SPARSE || WIDE ? 128 : 64;
  static constexpr int BK = B_ROW / ESIZE;               // dense k per stage
  static constexpr int A_BYTES = BM * A_ROW;
  static constexpr int META_ROW = SPARSE ? (F8 ? 16 : 8) : 0;   // metadata bytes per row and stage (4 bits per group of 4 k)
  // metadata: BM rows; the 256 x 256 tile shifts every KiB (bf16: 256 bytes) a DMA instruction brings by a few banks (big_meta)
  static constexpr int META_BYTES = BIG ? 4 * (F8 ? 1024 + 128 : 2 * (256 + 32)) * (SPARSE ? 1 : 0) : BM * META_ROW;
  static constexpr int B_BYTES = BN * B_ROW;
  static constexpr int META_OFF = A_BYTES;
  static constexpr int B_OFF = A_BYTES + META_BYTES;
  static constexpr int STAGE = A_BYTES + META_BYTES + B_BYTES;
  static constexpr int NB = ring_depth(SPARSE, F8, MI, NI);
  static constexpr int LDS_TOTAL = NB * STAGE;
  static constexpr int PER_CU = LDS_TOTAL <= 80 * 1024 ? 2 : 1;   // workgroups a CU is meant to hold (bounds the registers)
  // metadata DMA instructions per wave and stage (where a tile has less metadata than the four waves fetch, waves fetch the
  // same bytes to the same place: every wave then has the same count of instructions in flight)
  static constexpr int NM = SPARSE ? (F8 || MI < 4 ? 1 : 2) : 0;
  static constexpr int NA = MI * (A_ROW / 64), NVB = NI * (B_ROW / 64);   // ... of the A values and of B
  static constexpr int NDMA = NA + NM + NVB;             // DMA instructions per wave and stage
};

// LDS row -> row of the block tile (inverse of the permutation described above; in general wave-tile row 16 MI hc + 16 mi + v
// belongs to lane half hc, M-tile mi, register v, and wave-tile column NI c + ni to lane column c, N-tile ni)
template <int MI>
__device__ __forceinline__ int unperm_m(int p) {
  return (p & (32 * MI)) | (((p >> 2) & 1) * (16 * MI)) | (((p >> 5) & (MI - 1)) << 4) | (((p >> 3) & 3) << 2) | (p & 3);
}
template <int NI>
__device__ __forceinline__ int unperm_n(int p) { return (p & (32 * NI)) | ((p & 31) * NI) | ((p >> 5) & (NI - 1)); }
// The 256 x 256 tile: row 32 q + 4 t + v of the wave tile belongs to lane quarter q, M-tile t, register v, and column 8 c + t to lane column c, N-tile t.
// A rows lie in LDS as they are.  B: LDS row -> lane column and N-tile; what one DMA instruction fetches (16 rows of 64 bytes, 8 of 128) are
// neighbouring pieces of the B panel form (n at b_panel_pos(n)) in an order that puts the rows a fragment read takes together
// into one run: 8 of 64 bytes, 4 of 128.
template <bool SPARSE> __device__ __forceinline__ int big_n_col(int p) { return SPARSE ? ((p >> 3) & 3) << 2 | (p & 3) : ((p >> 4) & 1) << 3 | (p & 7); }
template <bool SPARSE> __device__ __forceinline__ int big_n_tile(int p) { return ((p >> 5) & 3) | (SPARSE ? (p >> 2) & 1 : (p >> 3) & 1) << 2; }
template <bool SPARSE> __device__ __forceinline__ int big_unperm_n(int p) { return (p & 128) | big_n_col<SPARSE>(p) << 3 | big_n_tile<SPARSE>(p); }
// 16-byte chunk swizzles.  A 16-byte-per-lane LDS read of a wavefront is served 16 lanes per clock, and the lanes
// that share a clock are not consecutive: {0-3, 20-23} and {4-7, 16-19} each pair up with {8-11, 28-31} or
// {12-15, 24-27} (likewise +32); they must hit 16 different 16-byte slots of the 256-byte bank row (measured on
// gfx950 with a read-throughput probe: both swizzles run at the rate of a linear read).
__device__ __forceinline__ int swz8(int p) { return (p ^ (p >> 3)) & 7; }          // 128-byte rows
__device__ __forceinline__ int swz4(int p) { return ((p >> 2) & 1) | ((((p >> 1) ^ (p >> 3)) & 1) << 1); }   // 64-byte rows
// The same for the 256 x 256 tiles, whose fragments are 16 rows (of lanes i = 0 .. 15) by four chunks: the lanes that share a clock are four
// neighbouring i of each i / 4, neighbouring i / 4 on different quarters.  64-byte rows, four of them in a bank row: the quarters take chunks
// 0 1 2 3 (dense; neighbours differ in bit 0, so bit 3 of i goes to bit 1) or 0 2 1 3 (2:4; the other way round).  128-byte rows: chunks
// 0 1 4 5 and two on, so bits 1 and 3 of i go to bits 1 and 2.
template <bool SPARSE> __device__ __forceinline__ int swz4_big(int i) { return SPARSE ? (i >> 3) & 1 : ((i >> 3) & 1) << 1; }
__device__ __forceinline__ int swz8_big(int i) { return (i & 2) | (((i >> 3) & 1) << 2); }

// k-major operands (TR): a caller's matrix with k as its slow dimension -- A [K][M] dense, B [K][N] -- read as it stands, bf16 only, under 4 GiB.  A
// stage's k rows lie in LDS as they come, 512 (256 x 256 tile) to 128 bytes of 16-byte pieces, and a fragment is read with the transposing LDS
// reads: the 16 lanes of a group hand in 8 bytes each, four consecutive rows (columns) of the tile at four k, and lane i gets the four k of
// row (column) i (measured: result lane i, element j = element i % 4 of the bytes lane 4 j + i / 4 points at).  So lanes 4 c .. 4 c + 3 always
// hold neighbours in memory.  For A that is the row order of the tiles anyway (four accumulators of a lane are four rows); of B every lane
// wants neighbouring columns, which the lanes of a quad exchange after the main loop (unquad).
// Against a pass that transposed them first: forward at T 1024 D 1024 F 4096 39.4 -> 25.6 us, bf16 step at T 1280 D 768 F 3072 78.7 -> 67.5, dense
// step at T 4096 D 2048 F 8192 732 -> 709; GEMM by GEMM (panel form -> k-major) T 8192 D 2048 F 8192 up-projection 222 -> 215, down-projection 121 -> 114,
// dW2 122 -> 116, T = F = 16384 D 4096 within 1 %, sparse 128 x 64 at T 2048 D 1024 F 4096 17.2 -> 19.0.
// Swizzles: what 32 lanes (16 where only one half of each piece is used) read at a time lies in different banks.  The rate of such reads is near that of
// 16-byte reads then (221 against 256 B/clk in a loop of nothing else; 32 without the swizzle).  Inside the 256 x 256 loops, beside the DMA's writes, the counters
// see conflicts in 0-1 % of the LDS-active cycles with B k-major, but in a third of them with A k-major (panels: none), T = F = 16384, D 4096.
constexpr int TR_A = 1, TR_B = 2;
template <int MI, int NI> __device__ __forceinline__ int tr_swz_a(int k) {
  if constexpr (MI * NI == 16) return (k & 3) | ((k >> 3) & 1) << 2;
  else if constexpr (MI == 4) return (k & 3) << 1;
  else if constexpr (MI == 2) return (k & 1) << 1 | (k & 2) << 2;
  else return (k & 2) << 1;
}
template <int MI, int NI> __device__ __forceinline__ int tr_swz_b(int k) {
  if constexpr (MI * NI == 16) return (k & 3) | ((k >> 3) & 1) << 2;
  else if constexpr (NI == 2) return (k & 3) << 2;
  else return (k & 2) << 1;
}
// a fragment of 8 k: the lane's 8 bytes of k .. k + 3 at p, of k + 4 .. k + 7 four rows on.  (__restrict__: without the alias scope it brings the compiler
// takes the read for one of what any DMA in flight writes and waits for all of them; the loops wait for the stage they read themselves.)
template <int KROW>
__device__ __forceinline__ bf16x8 tr_read(const char* __restrict__ p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * KROW));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// lane i of a quad gets a value of lane P(i) of it, P packed two bits a lane
template <int P>
__device__ __forceinline__ float quad(float x) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), P, 0xF, 0xF, true)); }
constexpr int quad_perm(int a, int b, int c, int d) { return a | b << 2 | c << 4 | d << 6; }

// compile-time loop: f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N-1>)
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) { (f(std::integral_constant<int, Is>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// Nothing may be moved across this point by the instruction scheduler.  The main loop is written as a sequence of
// slots {one matrix op + the memory ops that ride on it}, fenced from each other, so the issue order is the source order.
#define FFN24_FENCE() __builtin_amdgcn_sched_barrier(0)

// The lane's number, counted anew: kept in a register from the start of the kernel through the main loop it is one more than the 256 x 256 tiles have.
__device__ __forceinline__ int fresh_lane() {
  uint32_t all;
  asm volatile("s_mov_b32 %0, -1" : "=s"(all));
  return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt = bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xC07F); }   // vmcnt(63) expcnt(7) lgkmcnt(0)

// ------------------------------------------------------------------------------------------------
// global -> LDS DMA plan of one wave
// ------------------------------------------------------------------------------------------------
template <bool SPARSE, bool F8 = false, int PROBE = 0, int MI = 4, int NI = 4, int TR = 0>
struct Dma {
  using G = Geo<SPARSE, F8, MI, NI>;
  static constexpr int NA = G::NA, NVB = G::NVB;
  static constexpr bool TRA = (TR & TR_A) != 0, TRB = (TR & TR_B) != 0;
  __amdgpu_buffer_rsrc_t a;      // from the block's first A row on (uniform)
  __amdgpu_buffer_rsrc_t am;     // metadata
  __amdgpu_buffer_rsrc_t b;
  uint32_t va[NA], vm[2], vb[NVB];   // per-lane byte offsets from the uniform bases
  uint32_t a_stage, m_stage, b_stage;          // bytes from one stage to the next in the A values / metadata / B stream
  int wave;

  __device__ __forceinline__ void init(const GemmArgs& g, int m0, int n0, int tid) {
    int lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t b_row = (uint32_t)g.K * G::ESIZE;                 // bytes per B row in memory
    const uint32_t a_row = SPARSE ? b_row / 2 : b_row;               // bytes per A row (stored values only if sparse)
    // 256 rows occupy the same byte range in both forms; only the order of the pieces inside differs.  A tile of fewer rows
    // starts m0 % 256 (n0 % 256) rows into such a block.
    const bool panel = g.a_panel != 0, bp = g.b_panel != 0;
    const uint32_t a_pitch = panel ? 64u : a_row, m_pitch = panel ? (uint32_t)G::META_ROW : (uint32_t)(g.K / 8);
    const int ma = MI == 4 ? 0 : m0 & 255, mb = m0 - ma, na = NI == 4 || !bp ? 0 : n0 & 255, nb = n0 - na;
    if constexpr (TRA) a = from(static_cast<const char*>(g.A) + (size_t)m0 * G::ESIZE);
    else a = from(static_cast<const char*>(g.A) + (size_t)mb * a_row + (size_t)ma * a_pitch);
    if constexpr (SPARSE) am = from(reinterpret_cast<const char*>(g.Ameta) + (size_t)mb * (g.K / 8) + (size_t)ma * m_pitch);
    if constexpr (TRB) b = from(static_cast<const char*>(g.B) + (size_t)n0 * G::ESIZE);
    else b = from(static_cast<const char*>(g.B) + (g.b_rowmap ? (size_t)0 : (size_t)nb * b_row));
    const uint32_t a_krow = (uint32_t)g.M * G::ESIZE, b_krow = (uint32_t)g.N * G::ESIZE;   // bytes per k of a k-major operand
    a_stage = TRA ? (uint32_t)G::BK * a_krow : panel ? 256u * (uint32_t)G::A_ROW : (uint32_t)G::A_ROW;
    m_stage = panel ? 256u * G::META_ROW : (uint32_t)G::META_ROW;
    b_stage = TRB ? (uint32_t)G::BK * b_krow : bp ? 256u * (uint32_t)G::B_ROW : (uint32_t)G::B_ROW;
#pragma unroll
    for (int j = 0; j < NA; j++) {
      if constexpr (TRA) { va[j] = k_major<MI>(NA * wave + j, lane, a_krow, [](int k) { return tr_swz_a<MI, NI>(k); }); continue; }
      // 64-byte rows, 16 an instruction; 128-byte rows, 8 an instruction, of which the panel form has two 64-byte pieces in
      // consecutive 16 KiB runs
      const int p = G::WIDE ? 8 * (NA * wave + j) + (lane >> 3) : 16 * (NA * wave + j) + (lane >> 2);
      const int c = G::BIG ? (lane & 3) ^ swz4_big<SPARSE>((p >> 3) & 12) : G::WIDE ? (lane & 7) ^ swz8(p) : (lane & 3) ^ swz4(p);
      va[j] = (uint32_t)(G::BIG ? p : unperm_m<MI>(p)) * a_pitch + (G::WIDE && panel ? (uint32_t)(c >> 2) * (256u * 64u) + (c & 3) * 16 : (uint32_t)c * 16);
    }
#pragma unroll
    for (int j = 0; j < NVB; j++) {
      if constexpr (TRB) { vb[j] = k_major<NI>(NVB * wave + j, lane, b_krow, [](int k) { return tr_swz_b<MI, NI>(k); }); continue; }
      int p = G::B_ROW == 128 ? 8 * (NVB * wave + j) + (lane >> 3) : 16 * (NVB * wave + j) + (lane >> 2);
      int c = G::B_ROW == 128 ? (lane & 7) ^ (G::BIG ? swz8_big(big_n_col<SPARSE>(p)) : swz8(p)) : (lane & 3) ^ (G::BIG ? swz4_big<false>(big_n_col<SPARSE>(p)) : swz4(p));
      const int n = G::BIG ? big_unperm_n<SPARSE>(p) : unperm_n<NI>(p);
      if (bp) vb[j] = (uint32_t)(c >> 2) * (256u * 64u) + (uint32_t)b_panel_pos(na + n) * 64u + (c & 3) * 16;
      else vb[j] = (g.b_rowmap ? (uint32_t)g.b_rowmap[n0 + n] : (uint32_t)n) * b_row + c * 16;
    }
    if constexpr (SPARSE) {
      vm[1] = 0;
      if constexpr (F8) {
        // one row's 16 metadata bytes per lane (256 x 256: place 8 t + 4 q + v of the KiB is row 32 q + 4 t + v)
        const int r = G::BIG ? 64 * wave + 32 * ((lane >> 2) & 1) + 4 * (lane >> 3) + (lane & 3) : unperm_m<MI>(64 * (wave % MI) + lane);
        vm[0] = (uint32_t)r * m_pitch;
      } else {
#pragma unroll
        for (int j = 0; j < G::NM; j++) {
          int d = 64 * ((G::NM * wave + j) % (2 * MI)) + lane;
          vm[j] = (uint32_t)(G::BIG ? d >> 1 : unperm_m<MI>(d >> 1)) * m_pitch + 4 * (d & 1);
        }
      }
    }
  }

  // What a lane of instruction j fetches of a k-major operand: 8 / W rows of 128 W bytes of LDS an instruction, the 16-byte pieces of row k at
  // places XORed with the swizzle of k.
  template <int W, class Swz>
  static __device__ __forceinline__ uint32_t k_major(int j, int lane, uint32_t krow, Swz swz) {
    const int k = (8 / W) * j + lane / (8 * W);
    return (uint32_t)k * krow + (uint32_t)(((lane & (8 * W - 1)) ^ swz(k)) * 16);
  }

  // DMA instruction J of stage kt into the stage buffer at `buf` (uniform LDS pointer)
  template <int J>
  __device__ __forceinline__ void issue(int kt, char* buf) const {
    if constexpr ((PROBE & PROBE_NO_DMA) != 0) return;
    if constexpr ((PROBE & PROBE_K_WRAP) != 0) kt &= 7;
    // Buffer loads: descriptor + lane's 32-bit offset + the stage's scalar offset.  A fetch is the setting of M0 and the load, where the form with a
    // 64-bit address took three instructions more (a scalar base, a copy of the offset that the selector would accept); beside a
    // 16 x 16 op (16 cycles) there is room for three in all.
    if constexpr (J < NA) {
      load<16>(a, buf + (NA * wave + J) * 1024, va[J], (uint32_t)kt * a_stage);
    } else if constexpr (J < NA + G::NM) {
      constexpr int j = J - NA;
      if constexpr (F8) load<16>(am, buf + G::META_OFF + (G::BIG ? wave * (1024 + 128) : (wave % MI) * 1024), vm[0], (uint32_t)kt * m_stage);
      else load<4>(am, buf + G::META_OFF + (G::BIG ? (G::NM * wave + j) * (256 + 32) : ((G::NM * wave + j) % (2 * MI)) * 256), vm[j], (uint32_t)kt * m_stage);
    } else {
      constexpr int j = J - NA - G::NM;
      load<16>(b, buf + G::B_OFF + (NVB * wave + j) * 1024, vb[j], (uint32_t)kt * b_stage);
    }
  }
  // (no bound: every offset lies inside the operand, less than 4 GiB from the block's first row)
  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t from(const char* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, -1, 0x00020000); }
  template <int BYTES>
  static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, char* lds, uint32_t off, uint32_t stage) {
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_char*)lds, 16, (int)off, (int)stage, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_char*)lds, 4, (int)off, (int)stage, 0, 0);
  }
};

// ------------------------------------------------------------------------------------------------
// fragments and matrix ops
// ------------------------------------------------------------------------------------------------
struct LaneCtx {
  int rho, h;       // lane & 31, lane >> 5
  int wy, wx;       // wave row / column inside the block tile
  int a_row64;      // byte offset of the lane's LDS row among the wave's first 32 rows of A (64-byte rows)
  int b_row64;      // ... of B, 64-byte rows
  int a_row128;     // ... of A, 128-byte rows
  int b_row128;     // ... of B, 128-byte rows
  int sw4;          // swz4 of the lane's row (the same for every 32-row tile)
  int sw8;          // swz8 of the lane's B row for even ni (odd ni: ^4)
  int sw8a;         // swz8 of the lane's A row for even mi (odd mi: ^4)
  int a_tr, b_tr;   // k-major operands: the lane's first 8 bytes of the stage's A, of its B
  template <int MI, int NI>
  __device__ __forceinline__ void set_tr(int lane) {
    const int i = lane & 15, odd = (lane >> 4) & 1, k = 8 * h + (i >> 2);
    // quad 4 odd + i % 4 of the 32 rows is lane half hc's vh-th group of four
    const int quad = 4 * odd + (i & 3), hc = quad & 1, vh = quad >> 1;
    a_tr = k * (128 * MI) + (((4 * MI * wy + 2 * MI * hc + (vh >> 1)) ^ tr_swz_a<MI, NI>(k)) << 4) + 8 * (vh & 1);
    // NI = 2: N-tile ni has the ni-th half of every 16-byte piece
    b_tr = NI == 2 ? k * 256 + (((8 * wx + quad) ^ tr_swz_b<MI, NI>(k)) << 4) : k * 128 + (((4 * wx + (quad >> 1)) ^ tr_swz_b<MI, NI>(k)) << 4) + 8 * (quad & 1);
  }
};

// Dense: K step S (0,1) of the 64-byte stage rows; fragment I < MI -> a[I], else b[I-MI]
template <int MI, int NI>
struct FragD {
  bf16x8 a[MI], b[NI];
};
template <class G, int S, int I, int TR = 0, int MI, int NI>
__device__ __forceinline__ void load_frag_dense1(const char* buf, const LaneCtx& L, FragD<MI, NI>& f) {
  if constexpr (I < MI && (TR & TR_A)) { f.a[I] = tr_read<128 * MI>(buf + (L.a_tr ^ (I << 5)) + S * (16 * 128 * MI)); return; }
  if constexpr (I >= MI && (TR & TR_B)) { f.b[I - MI] = tr_read<128 * NI>(buf + G::B_OFF + L.b_tr + 8 * (I - MI) + S * (16 * 128 * NI)); return; }
  if constexpr (G::WIDE) {
    constexpr int i = I < MI ? I : I - MI;
    const int c = ((2 * S + L.h) ^ (I < MI ? L.sw8a : L.sw8) ^ ((i & 1) << 2)) << 4;
    if constexpr (I < MI) f.a[I] = *reinterpret_cast<const bf16x8*>(buf + L.a_row128 + i * (32 * 128) + c);
    else f.b[I - MI] = *reinterpret_cast<const bf16x8*>(buf + G::B_OFF + L.b_row128 + i * (32 * 128) + c);
    return;
  }
  int c = ((2 * S + L.h) ^ L.sw4) << 4;
  if constexpr (I < MI) f.a[I] = *reinterpret_cast<const bf16x8*>(buf + L.a_row64 + I * (32 * 64) + c);
  else f.b[I - MI] = *reinterpret_cast<const bf16x8*>(buf + G::B_OFF + L.b_row64 + (I - MI) * (32 * 64) + c);
}
template <int M, int MI, int NI>
__device__ __forceinline__ void mfma_dense1(const FragD<MI, NI>& f, f32x16 (&acc)[MI][NI]) {
  constexpr int mi = M / NI, ni = M % NI;
  acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[mi], f.b[ni], acc[mi][ni], 0, 0, 0);
}
// fp8 e4m3, v_mfma_f32_32x32x64_f8f6f4: 32 operand bytes per lane, paired byte by byte between A and B (measured:
// any assignment of the 64 k to (lane half, byte) works if both operands use the same one).  The two 16-byte
// fragments of a stage (S = 0 and S = 1 above) are exactly one such operand, so a 64-byte-row stage is one K step.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ i32x8 cat16(const bf16x8& lo, const bf16x8& hi) {
  i32x4 l = __builtin_bit_cast(i32x4, lo), h = __builtin_bit_cast(i32x4, hi);
  return __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
}
// The smaller tiles have registers to spare, and their accumulators come round again within a few ops: the builtin, whose
// hazards the compiler handles (formats 0 = e4m3; scale operands 0 = the unscaled instruction).
__device__ __forceinline__ void mfma_f8(const i32x8& a, const i32x8& b, f32x16& c) {
  c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}
template <int M, int MI, int NI>
__device__ __forceinline__ void mfma_dense_f8(const FragD<MI, NI>& f0, const FragD<MI, NI>& f1, f32x16 (&acc)[MI][NI]) {
  constexpr int mi = M / NI, ni = M % NI;
  mfma_f8(cat16(f0.a[mi], f1.a[mi]), cat16(f0.b[ni], f1.b[ni]), acc[mi][ni]);
}

// Sparse: the stage's K window of 64 = four 16-wide windows w.  Instruction S (0,1) gives lane half q the window
// 2q+S, so a lane's two instructions use 32 consecutive stored-value bytes and one 32-bit metadata word (ABID = S
// picks the half).  B lane half h then needs, for instruction S, the 8-k chunks 2S+h (registers 0..7) and 4+2S+h
// (registers 8..15).
template <int MI, int NI>
struct FragS {
  bf16x8 a[MI];
  bf16x8 blo[NI], bhi[NI];
};
// Metadata of a lane for the stage's two instructions: bf16 one 32-bit word (16 bits per instruction, picked by
// ABID); fp8 (twice the groups per stored byte) two words, one per instruction.
template <bool F8> struct IdxWords { uint32_t w[F8 ? 2 : 1]; };
template <class G, bool F8, int I, int MI>
__device__ __forceinline__ void load_idx_sparse1(const char* buf, const LaneCtx& L, IdxWords<F8> (&idx)[MI]) {
  const char* p = buf + G::META_OFF + (L.wy * (32 * MI) + L.rho + 32 * I) * G::META_ROW;
  if constexpr (F8) {
    u32x2 v = *reinterpret_cast<const u32x2*>(p + 8 * L.h);
    idx[I].w[0] = v[0]; idx[I].w[1] = v[1];
  } else {
    idx[I].w[0] = *reinterpret_cast<const uint32_t*>(p + 4 * L.h);
  }
}
// fragment I of instruction S: I < MI -> a[I]; the next NI -> low halves of b; the last NI -> high halves of b
template <class G, int S, int I, int TR = 0, int MI, int NI>
__device__ __forceinline__ void load_frag_sparse1(const char* buf, const LaneCtx& L, FragS<MI, NI>& f) {
  if constexpr (I >= MI && (TR & TR_B)) {
    constexpr int i = (I - MI) % NI;
    const char* p = buf + G::B_OFF + L.b_tr + 8 * i + S * (16 * 128 * NI);
    if constexpr (I < MI + NI) f.blo[i] = tr_read<128 * NI>(p);
    else f.bhi[i] = tr_read<128 * NI>(p + 32 * 128 * NI);
  } else if constexpr (I < MI) {
    f.a[I] = *reinterpret_cast<const bf16x8*>(buf + L.a_row64 + I * (32 * 64) + (((2 * L.h + S) ^ L.sw4) << 4));
  } else {
    constexpr int i = (I - MI) % NI;
    int sw = L.sw8 ^ ((i & 1) << 2);
    const char* row = buf + G::B_OFF + L.b_row128 + i * (32 * 128);
    if constexpr (I < MI + NI) f.blo[i] = *reinterpret_cast<const bf16x8*>(row + (((2 * S + L.h) ^ sw) << 4));
    else f.bhi[i] = *reinterpret_cast<const bf16x8*>(row + (((4 + 2 * S + L.h) ^ sw) << 4));
  }
}
// fp8: v_smfmac_f32_32x32x64_fp8_fp8 has, byte for byte, the operand layout of the bf16 instruction (measured): A 16
// stored bytes of the lane half's window, B the two 16-byte chunks, and a full 32-bit index word per instruction.
template <bool F8, int S, int M, int MI, int NI>
__device__ __forceinline__ void mfma_sparse1(const FragS<MI, NI>& f, const IdxWords<F8> (&idx)[MI], f32x16 (&acc)[MI][NI]) {
  constexpr int mi = M / NI, ni = M % NI;
  if constexpr (F8) {
    acc[mi][ni] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(__builtin_bit_cast(i32x4, f.a[mi]), cat16(f.blo[ni], f.bhi[ni]), acc[mi][ni],
                                                               (int)idx[mi].w[S], 0, 0);
  } else {
    bf16x16 b = __builtin_shufflevector(f.blo[ni], f.bhi[ni], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    acc[mi][ni] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(f.a[mi], b, acc[mi][ni], (int)idx[mi].w[0], 0, S);
  }
}

// What a wave of the smaller tiles holds of one whole stage: the fragments (and metadata) as READS LDS reads, consumed by OPS matrix ops
// that come in the order of k.
template <bool SPARSE, bool F8, int MI, int NI, int TR = 0>
struct StageRegs {                           // dense: chunk pairs q of 32 bytes of k, one K step each (fp8: two a step)
  static constexpr int PAIRS = wide_stage(MI, NI) ? 4 : 2, NF = MI + NI;
  static constexpr int READS = PAIRS * NF, OPS = MI * NI * PAIRS / (F8 ? 2 : 1);
  static constexpr int READ_SLOTS = OPS > 1 ? OPS / 2 : 1;
  FragD<MI, NI> f[PAIRS];
  template <class G, int I> __device__ __forceinline__ void read(const char* buf, const LaneCtx& L) { load_frag_dense1<G, I / NF, I % NF, TR>(buf, L, f[I / NF]); }
  template <int M> __device__ __forceinline__ void op(f32x16 (&acc)[MI][NI]) const {
    constexpr int s = M / (MI * NI), m = M % (MI * NI);
    if constexpr (F8) mfma_dense_f8<m>(f[2 * s], f[2 * s + 1], acc);
    else mfma_dense1<m>(f[s], acc);
  }
};
template <bool F8, int MI, int NI, int TR>
struct StageRegs<true, F8, MI, NI, TR> {
  static constexpr int NF = MI + 2 * NI;
  static constexpr int READS = MI + 2 * NF, OPS = 2 * MI * NI;
  static constexpr int READ_SLOTS = OPS / 2;
  FragS<MI, NI> f[2];
  IdxWords<F8> idx[MI];
  template <class G, int I> __device__ __forceinline__ void read(const char* buf, const LaneCtx& L) {
    if constexpr (I < MI) load_idx_sparse1<G, F8, I>(buf, L, idx);
    else load_frag_sparse1<G, (I - MI) / NF, (I - MI) % NF, TR>(buf, L, f[(I - MI) / NF]);
  }
  template <int M> __device__ __forceinline__ void op(f32x16 (&acc)[MI][NI]) const {
    mfma_sparse1<F8, M / (MI * NI), M % (MI * NI)>(f[M / (MI * NI)], idx, acc);
  }
};

// ------------------------------------------------------------------------------------------------
// the kernel
// ------------------------------------------------------------------------------------------------

// tile id -> (tile_m, tile_n).  Consecutive workgroup ids go round-robin over the 8 XCDs (each with its own L2) and an
// XCD hands its ids to its 32 CUs in order, so 256 consecutive ids are one "round" of the chip: XCD x runs ids
// x, x + 8, ... of it.  A round is laid out as a 4 x 2 grid of per-XCD patches of 8 x 4 tiles (32 tile-rows x 8
// tile-columns in all): inside a patch the 8 + 4 operand panels are shared through the XCD's L2, and XCDs that sit in
// the same grid row (column) read the same A (B) panels at the same time, so that what one of them brings in from HBM
// the others find in the memory-side cache.  Measured against one 8 x 4 patch per XCD with all XCDs side by side
// along M (every round then streams the whole A operand): 3.5 % on the sparse GEMMs, nothing on the dense ones.
// Tile-rows beyond the last whole round (ntm not a multiple of 32: the sparse part of a split weight gradient) and shapes whose
// tile-columns the grid does not divide fall back to bands of 8 tile-rows, each XCD a contiguous run of tiles: of 4 tile-rows if a tile
// is twice as tall as wide (256 x 128, 128 x 64), so that an XCD's 32 tiles still cover a square of the result (a bf16 step at T 4864 D 3328
// F 7680, dense GEMMs on 256 x 128: 1115 -> 1092 us, 1099 with 256 x 256; T 11008 D 1536 F 5120 dense 989 -> 971).  The rounds keep
// their patch of 8 x 4 tiles for it: 4 x 8 costs 1.5 % at T 4096 D 2048 F 8192.
template <int PROBE = 0, bool TALL = false>
__device__ __forceinline__ void tile_coords(int ntm, int ntn, int pid, int& tm, int& tn) {
  // XCD grid, patch shape; GX * GY = 8 XCDs, PM * PN = 32 CUs
  constexpr int GX = (PROBE & PROBE_WALK_8x1) ? 8 : 4, GY = 8 / GX;
  constexpr int PM = (PROBE & PROBE_PATCH_4x8) ? 4 : ((PROBE & PROBE_PATCH_16x2) ? 16 : 8), PN = 32 / PM;
  int tm0 = 0;   // tile-rows [0, tm0) are walked in rounds, the rest in bands
  if (!(PROBE & PROBE_WALK_BANDS) && ntn % (PN * GY) == 0) tm0 = ntm - ntm % (PM * GX);
  if (pid < tm0 * ntn) {
    const int xcd = pid & 7, idx = pid >> 3;
    const int round = idx >> 5, j = idx & 31;
    const int rounds_n = ntn / (PN * GY);
    tm = ((round / rounds_n) * GX + (xcd % GX)) * PM + (j % PM);
    tn = ((round % rounds_n) * GY + (xcd / GX)) * PN + (j / PM);
    return;
  }
  pid -= tm0 * ntn;   // a multiple of 256: the low three bits are still the XCD
  ntm -= tm0;
  int nb = ntm * ntn;
  if ((nb & 7) == 0) pid = (pid & 7) * (nb >> 3) + (pid >> 3);
  const int GROUP = TALL ? 4 : 8;
  int per_group = GROUP * ntn;
  int gid = pid / per_group;
  int first = gid * GROUP;
  int gsz = min(ntm - first, GROUP);
  int in = pid - gid * per_group;
  tm = tm0 + first + in % gsz;
  tn = in / gsz;
}

// an epilogue that declares `static constexpr bool STAGED` takes a fifth argument: LDS private to the wave for its part of the result in bf16
template <class E, class = void> struct epi_is_staged : std::false_type {};
template <class E> struct epi_is_staged<E, std::void_t<decltype(E::STAGED)>> : std::true_type {};

// Epilogue concept:  struct E { struct Args {...}; template <int MI, int NI, class Acc> static __device__ void run(const Args&, Acc& acc, m_lane, n_lane); }
//   m_lane = global row of acc[0][*][0] for this lane (its 16 MI rows are m_lane + 16*mi + v),
//   n_lane = global column of acc[*][0][*] (its NI columns are n_lane + ni).
// Acc: f32x16 [MI][NI], or (256 x 256) float [MI][NI][16]; either is indexed acc[mi][ni][v].
// run<2, 8> is the 256 x 256 tile (see LaneTile), the others are the smaller tiles' wave tiles.
template <class G, class Epi, int MI, int NI, class Acc>
__device__ __forceinline__ void run_epilogue(const typename Epi::Args& ea, Acc& acc, int m_lane, int n_lane, char* smem, int wave) {
  if constexpr (epi_is_staged<Epi>::value) {
    // the epilogue stages its stores through the operand ring: every wave must have read its last fragments first
    constexpr int WAVE_BYTES = (G::BN / 2) * G::BM;   // the wave's part of the result in bf16
    static_assert(G::LDS_TOTAL >= GEMM_THREADS / 64 * WAVE_BYTES, "a staging area per wave");
    __builtin_amdgcn_s_barrier();
    Epi::template run<MI, NI>(ea, acc, m_lane, n_lane, smem + wave * WAVE_BYTES);
  } else {
    Epi::template run<MI, NI>(ea, acc, m_lane, n_lane);
  }
}

// The smaller tiles (several workgroups a CU, whose issue gaps fill each other) spread N memory instructions over the slots of a K
// step by whole runs: slot M carries instructions [M * per, M * per + per).
template <int N, int SLOTS, int M, class F>
__device__ __forceinline__ void ride(F&& f) {
  constexpr int per = (N + SLOTS - 1) / SLOTS, lo = M * per < N ? M * per : N, hi = (M + 1) * per < N ? (M + 1) * per : N;
  static_for<hi - lo>([&](auto i) { f(std::integral_constant<int, lo + decltype(i)::value>{}); });
}

// NI = 2, B k-major: lane i of a quad has columns 8 g + i and 8 g + 4 + i and wants 8 g + 2 i and 8 g + 2 i + 1
template <int MI>
__device__ __forceinline__ void unquad(f32x16 (&acc)[MI][2]) {
  const bool upper = (fresh_lane() & 2) != 0;
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const float x = acc[i][0][v], y = acc[i][1][v];
      constexpr int EVEN = quad_perm(0, 2, 0, 2), ODD = quad_perm(1, 3, 1, 3);
      const float x0 = quad<EVEN>(x), y0 = quad<EVEN>(y), x1 = quad<ODD>(x), y1 = quad<ODD>(y);
      acc[i][0][v] = upper ? y0 : x0;
      acc[i][1][v] = upper ? y1 : x1;
    }
}

template <bool SPARSE, class Epi, bool F8, int MI, int NI, int TR>
__device__ __forceinline__ void gemm_tile_small(const GemmArgs& g, const typename Epi::Args& ea, char* smem, int pid) {
  using G = Geo<SPARSE, F8, MI, NI>;
  constexpr int NMF = MI * NI;              // matrix ops (slots) per K step
  constexpr int FRAG_SLOTS = (NMF + 1) / 2; // slots of a K step that carry fragment reads
  constexpr int NB = G::NB, NDMA = G::NDMA;

  int tid = threadIdx.x;
  int lane = tid & 63, wave = tid >> 6;
  int tm, tn;
  tile_coords<0, MI == 2 * NI>(g.M / G::BM, g.N / G::BN, pid, tm, tn);
  int m0 = tm * G::BM, n0 = tn * G::BN;

  LaneCtx L;
  L.rho = lane & 31; L.h = lane >> 5; L.wy = wave >> 1; L.wx = wave & 1;
  L.a_row64 = (L.wy * (32 * MI) + L.rho) * 64;
  L.b_row64 = (L.wx * (32 * NI) + L.rho) * 64;
  L.a_row128 = (L.wy * (32 * MI) + L.rho) * 128;
  L.b_row128 = (L.wx * (32 * NI) + L.rho) * 128;
  L.sw4 = swz4(L.rho);
  // (from NI = 2, MI = 2 on the wave column, wave row moves the row by a multiple of 64, which the swizzle does not see)
  L.sw8 = NI == 1 ? swz8(L.wx * 32 + L.rho) : swz8(L.rho);
  L.sw8a = MI == 1 ? swz8(L.wy * 32 + L.rho) : swz8(L.rho);

  if constexpr (TR != 0) L.set_tr<MI, NI>(lane);

  Dma<SPARSE, F8, 0, MI, NI, TR> dma;
  dma.init(g, m0, n0, tid);

  const int nk = g.K / G::BK;
  // prologue: stages 0 .. min(NB, nk)-1 into their ring slots; wait for stage 0 only
  const int npro = nk < NB ? nk : NB;
  for (int s = 0; s < npro; s++) static_for<NDMA>([&](auto J) { dma.template issue<J>(s, smem + s * G::STAGE); });
  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  if (npro == NB) wait_vmcnt<(NB - 1) * NDMA>(); else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  FFN24_FENCE();

  // MODE 0: steady state -- after the barrier the stage kt+NB is issued into the buffer this stage frees
  // MODE 1: tail -- nothing left to issue, wait for everything outstanding before the barrier
  // MODE 2: last stage -- no barrier, no next fragments
  if constexpr (whole_stage_ahead(SPARSE, MI, NI)) {
    // A smaller tile has few matrix ops a stage, so what a wave waits for itself counts: reading the second K step's fragments, the
    // barrier and reading the next stage's first ones were one chain of 360 cycles a stage of the sparse 64 x 64 tile, beside the 350
    // its operands take to arrive, and the two added up to 500.  Here the fragments of the WHOLE next stage are read while this
    // stage's ops run (two register sets), with one wait and one barrier a stage, and the DMA of the stage that reuses this
    // stage's buffer, whose fragments are in registers, rides along.  One tile a CU, K 4096: sparse 64 x 64 15.0 -> 13.0 us, 128 x 64 16.6
    // -> 15.2, 256 x 128 37.0 -> 35.8; dense 64 x 64 see wide_stage, 128 x 128 29.8 -> 29.6.  What bounds them now is the operand stream.
    StageRegs<SPARSE, F8, MI, NI, TR> r0, r1;
    using SR = StageRegs<SPARSE, F8, MI, NI, TR>;
    auto stage = [&](int kt, char* cur, char* nxt, const SR& now, SR& next, auto mode, auto left) {
      constexpr int MODE = decltype(mode)::value, LEFT = decltype(left)::value;
      FFN24_FENCE();
      static_for<SR::OPS>([&](auto M) {
        now.template op<M>(acc);
        if constexpr (MODE != 2) ride<SR::READS, SR::READ_SLOTS, M>([&](auto I) { next.template read<G, I>(nxt, L); });
        // (from 4 matrix ops a K step on, behind the fragment reads: 256 x 128 36.5 -> 35.8 us, dense 128 x 128 11.2 -> 10.6; 128 x 64 15.2 -> 15.7)
        constexpr int FIRST = NMF >= 4 ? SR::OPS / 2 : 0;
        if constexpr (MODE == 0 && M >= FIRST) ride<NDMA, SR::OPS - FIRST, M - FIRST>([&](auto J) { dma.template issue<J>(kt + NB, cur); });
        FFN24_FENCE();
      });
      if constexpr (MODE != 2 && LEFT >= 0) {
        wait_vmcnt<(LEFT > 0 ? LEFT : 0) * NDMA>();   // LEFT: the stages behind stage kt + 2, which the next stage reads, that may be in flight
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
      }
      FFN24_FENCE();
    };
    using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>; using I2 = std::integral_constant<int, 2>;
    int slot = 0;
    auto advance = [&](int kt, const SR& now, SR& next, auto mode, auto left) {
      int ns = slot + 1 == NB ? 0 : slot + 1;
      stage(kt, smem + slot * G::STAGE, smem + ns * G::STAGE, now, next, mode, left);
      slot = ns;
    };
    static_for<SR::READS>([&](auto I) { r0.template read<G, I>(smem, L); });
    if (npro == NB) wait_vmcnt<(NB - 2) * NDMA>(); else wait_vmcnt<0>();   // stage 1, which stage 0 reads
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    FFN24_FENCE();
    int kt = 0;
    if (nk >= NB) {
      const int n0 = nk - NB;            // stages that have a stage to ask for
      using INB = std::integral_constant<int, NB - 2>;
      for (; kt + 1 < n0; kt += 2) { advance(kt, r0, r1, I0{}, INB{}); advance(kt + 1, r1, r0, I0{}, INB{}); }
      if (kt < n0) { advance(kt, r0, r1, I0{}, INB{}); kt++; r0 = r1; }
      static_for<NB>([&](auto i) {
        constexpr int I = decltype(i)::value;
        using Mode = std::integral_constant<int, (I == NB - 1 ? 2 : 1)>;
        using Left = std::integral_constant<int, (I == NB - 2 ? -1 : (NB - 3 - I))>;   // (the last stage reads nothing: no barrier before it)
        if constexpr (I % 2 == 0) advance(kt + I, r0, r1, Mode{}, Left{}); else advance(kt + I, r1, r0, Mode{}, Left{});
      });
    } else {                             // shorter than the ring: everything has landed
      for (; kt < nk - 1; kt++) { advance(kt, r0, r1, I1{}, I0{}); r0 = r1; }
      advance(kt, r0, r1, I2{}, I0{});
    }
  } else if constexpr (SPARSE) {
    FragS<MI, NI> f0, f1;
    constexpr int NF = MI + 2 * NI;
    IdxWords<F8> idx[MI];
    static_for<MI>([&](auto I) { load_idx_sparse1<G, F8, I>(smem, L, idx); });
    static_for<NF>([&](auto I) { load_frag_sparse1<G, 0, I, TR>(smem, L, f0); });
    auto stage = [&](int kt, char* cur, char* nxt, auto mode) {
      constexpr int MODE = decltype(mode)::value;
      IdxWords<F8> idx_n[MI] = {};
      FFN24_FENCE();
      static_for<NMF>([&](auto M) {
        mfma_sparse1<F8, 0, M>(f0, idx, acc);
        ride<NF, FRAG_SLOTS, M>([&](auto I) { load_frag_sparse1<G, 1, I, TR>(cur, L, f1); });
        FFN24_FENCE();
      });
      if constexpr (MODE != 2) {
        // stage kt+1 must have landed; behind it in issue order are the NB - 2 stages kt+2 .. kt+NB-1
        if constexpr (MODE == 0) wait_vmcnt<(NB - 2) * NDMA>(); else wait_vmcnt<0>();
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
      }
      FFN24_FENCE();
      static_for<NMF>([&](auto M) {
        mfma_sparse1<F8, 1, M>(f1, idx, acc);
        if constexpr (MODE == 0) ride<NDMA, NMF, M>([&](auto J) { dma.template issue<J>(kt + NB, cur); });
        if constexpr (MODE != 2) {
          if constexpr (M < MI) load_idx_sparse1<G, F8, M>(nxt, L, idx_n);
          ride<NF, FRAG_SLOTS, M>([&](auto I) { load_frag_sparse1<G, 0, I, TR>(nxt, L, f0); });
        }
        FFN24_FENCE();
      });
#pragma unroll
      for (int i = 0; i < MI; i++) idx[i] = idx_n[i];
    };
    int slot = 0;
    auto advance = [&](int kt, auto mode) {
      int ns = slot + 1 == NB ? 0 : slot + 1;
      stage(kt, smem + slot * G::STAGE, smem + ns * G::STAGE, mode);
      slot = ns;
    };
    int kt = 0;
    for (; kt < nk - NB; kt++) advance(kt, std::integral_constant<int, 0>{});
    for (; kt < nk - 1; kt++) advance(kt, std::integral_constant<int, 1>{});
    advance(kt, std::integral_constant<int, 2>{});
  } else if constexpr (F8) {
    // Dense fp8, 256 x 128: a stage is ONE K step of 8 matrix ops (64 cycles each).  The fragments of the whole next stage and
    // the DMA of the stage that reuses this stage's buffer (its fragments are already in registers) ride on them;
    // one barrier at the end of the stage.  Two fragment sets alternate.
    FragD<MI, NI> fr[2][2];
    constexpr int NF = MI + NI;
    static_for<NF>([&](auto I) { load_frag_dense1<G, 0, I, TR>(smem, L, fr[0][0]); });
    static_for<NF>([&](auto I) { load_frag_dense1<G, 1, I, TR>(smem, L, fr[0][1]); });
    auto stage = [&](int kt, char* cur, char* nxt, auto par, auto mode) {
      constexpr int P = decltype(par)::value, MODE = decltype(mode)::value;
      FFN24_FENCE();
      static_for<NMF>([&](auto M) {
        mfma_dense_f8<M>(fr[P][0], fr[P][1], acc);
        if constexpr (MODE == 0) ride<NDMA, NMF, M>([&](auto J) { dma.template issue<J>(kt + NB, cur); });
        if constexpr (MODE != 2) ride<2 * NF, NMF, M>([&](auto I) {
          if constexpr (I < NF) load_frag_dense1<G, 0, I, TR>(nxt, L, fr[P ^ 1][0]);
          else load_frag_dense1<G, 1, I - NF, TR>(nxt, L, fr[P ^ 1][1]);
        });
        FFN24_FENCE();
      });
      if constexpr (MODE != 2) {
        // the next stage reads fragments of stage kt+2 from the first op on: it must have landed, everywhere
        if constexpr (MODE == 0) wait_vmcnt<(NB - 2) * NDMA>(); else wait_vmcnt<0>();
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
      }
      FFN24_FENCE();
    };
    // the loop above reads stage 1 during stage 0: the prologue's wait covered stage 0 only
    if (npro == NB) wait_vmcnt<(NB - 2) * NDMA>(); else wait_vmcnt<0>();
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    FFN24_FENCE();
    // The two fragment sets alternate by stage parity.  The stage count is even (K is a multiple of 128 here), so
    // the stages are walked in pairs, straight-line: a parity branch inside the loop makes the compiler shuffle the
    // accumulation registers between its two arms.
    int slot = 0;
    auto advance = [&](int kt, auto par, auto mode) {
      int ns = slot + 1 == NB ? 0 : slot + 1;
      stage(kt, smem + slot * G::STAGE, smem + ns * G::STAGE, par, mode);
      slot = ns;
    };
    using P0 = std::integral_constant<int, 0>; using P1 = std::integral_constant<int, 1>;
    using M0 = std::integral_constant<int, 0>; using M1 = std::integral_constant<int, 1>; using M2 = std::integral_constant<int, 2>;
    int kt = 0;
    for (; kt + 1 < nk - NB; kt += 2) { advance(kt, P0{}, M0{}); advance(kt + 1, P1{}, M0{}); }
    if (NB % 2 != 0 && kt < nk - NB) { advance(kt, P0{}, M0{}); advance(kt + 1, P1{}, M1{}); kt += 2; }
    for (; kt < nk - 2; kt += 2) { advance(kt, P0{}, M1{}); advance(kt + 1, P1{}, M1{}); }
    advance(kt, P0{}, M1{});
    advance(kt + 1, P1{}, M2{});
  } else {
    FragD<MI, NI> f0, f1;
    constexpr int NF = MI + NI;
    static_for<NF>([&](auto I) { load_frag_dense1<G, 0, I, TR>(smem, L, f0); });
    auto stage = [&](int kt, char* cur, char* nxt, auto mode) {
      constexpr int MODE = decltype(mode)::value;
      FFN24_FENCE();
      static_for<NMF>([&](auto M) {
        mfma_dense1<M>(f0, acc);
        ride<NF, FRAG_SLOTS, M>([&](auto I) { load_frag_dense1<G, 1, I, TR>(cur, L, f1); });
        FFN24_FENCE();
      });
      if constexpr (MODE != 2) {
        if constexpr (MODE == 0) wait_vmcnt<(NB - 2) * NDMA>(); else wait_vmcnt<0>();
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
      }
      FFN24_FENCE();
      static_for<NMF>([&](auto M) {
        mfma_dense1<M>(f1, acc);
        if constexpr (MODE == 0) ride<NDMA, NMF, M>([&](auto J) { dma.template issue<J>(kt + NB, cur); });
        if constexpr (MODE != 2) ride<NF, FRAG_SLOTS, M>([&](auto I) { load_frag_dense1<G, 0, I, TR>(nxt, L, f0); });
        FFN24_FENCE();
      });
    };
    int slot = 0;
    auto advance = [&](int kt, auto mode) {
      int ns = slot + 1 == NB ? 0 : slot + 1;
      stage(kt, smem + slot * G::STAGE, smem + ns * G::STAGE, mode);
      slot = ns;
    };
    int kt = 0;
    for (; kt < nk - NB; kt++) advance(kt, std::integral_constant<int, 0>{});
    for (; kt < nk - 1; kt++) advance(kt, std::integral_constant<int, 1>{});
    advance(kt, std::integral_constant<int, 2>{});
  }

  if constexpr ((TR & TR_B) && NI == 2) unquad(acc);
  int m_lane = m0 + L.wy * (32 * MI) + (16 * MI) * L.h;
  int n_lane = n0 + L.wx * (32 * NI) + NI * L.rho;
  run_epilogue<G, Epi, MI, NI>(ea, acc, m_lane, n_lane, smem, wave);
}

// The 256 x 256 block tile: four waves of 128 x 128, one a SIMD, 256 accumulators a lane pinned to the AGPR file.  Its matrix ops are the
// 16 x 16 ones: under matrix load the chip is bound by its power limit, and a 16 x 16 op moves fewer accumulator bytes a flop through the
// register file than a 32 x 32 one.  Register-resident loops at the power limit, N(0, 1) operands, 32 x 32 -> 16 x 16 (PFLOP/s dense equivalent):
// dense bf16 1.83 -> 2.09, 2:4 bf16 3.37 -> 3.55, dense fp8 4.11 -> 4.47, 2:4 fp8 6.49 -> 6.89 (the rates depend on the operands: with the
// uniform ones of probe_mfma_rate the 16 x 16 loops give 2.01, 3.41, 4.66 and 7.07).  The whole loop, pseudo-random operands, M 16384
// N 4096: dense bf16 K 16384 1.59 -> 1.53 ms, K 4096 0.495 -> 0.467, 2:4 1.02 -> 0.98, 0.262 -> 0.256; the steps of the block at T = F = 16384, D 4096
// 7.45 -> 7.09 ms, fp8 forward at T = D = 8192, F 32768 2.48 -> 2.33 ms.  What bounds it is energy: the clock settles 15 % higher than with the
// 32 x 32 ops (1.75 against 1.52 GHz) and a stage takes 10 % more cycles (1290 against 1180 of 1024), and whatever saves cycles alone (B fragments read two
// at a time or spread, DMA on every 64 or 128 cycles, five stages, a serpentine over the ops) lowers the clock again: all within 1 %.
// With the k of a stage given to the lane quarters as below an op adds up what two 32 x 32 ops add up, in the same order: the results are the
// same bit for bit (all four types), so the smaller tiles, which are not at the power limit, keep theirs.
//   lane l, quarter q = l / 16, c = l % 16: A row / B column c of a 16-row tile; accumulators = rows 4 q .. 4 q + 3, column c.
//   dense bf16 16x16x32: k 8 q .. + 7 of the stage's 32 (16-byte chunk q of the row).
//   dense fp8 16x16x128: chunk q of two consecutive stages (a K step is two stages).
//   2:4 16x16x64 (fp8 16x16x128): the stored values of window 0, 2, 1, 3 of the stage's four for q = 0 .. 3, with their metadata;
//     B: chunks c0 = (q & 1) + 4 (q / 2) and c0 + 2 of the stage row's eight.
// A K step is 64 ops in two halves of 32, one for each half of the columns, the ops of a row of four next to each other:
//   half 0: the other half's B fragments of this step are read;
//   wait for the next stage's DMA, one workgroup barrier: this stage's buffer is free;
//   half 1: the next step's first B fragments take the place of the ones half 0 used up, its A fragments follow row by row behind the
//           last op that uses theirs, and the DMA of the stage that reuses the buffer rides along.
// So no fragment is held twice, and every read has at least 28 ops to arrive.
template <bool SPARSE, bool F8>
struct BigFrags {
  static constexpr bool PAIR = F8 && !SPARSE;                 // 32 bytes of A a lane
  bf16x8 a[8][PAIR ? 2 : 1], b[2][4][SPARSE || PAIR ? 2 : 1];
  uint32_t idx[SPARSE ? 8 : 1];
};
struct BigLane { int a, b, m; };   // byte offsets of the lane's first fragment of A, of B and of its metadata inside a stage

// The ops are inline assembly with the accumulator tied in place in the AGPR file.  Through the builtins the compiler, with all 256 of those
// registers in use, copies accumulators to the other file and back round the ops of the loops' tails, or spills some of them.  What
// its hazard handling then does not see: the same accumulator comes round again 64 ops later, the operands come from LDS reads (which it
// does wait for; no vector instruction writes one within two instructions of its op, tests/test_kernel_hazards.py), and the end of the
// main loop waits for the last ops.  Default modifiers of the f8f6f4 op: both operands e4m3, unscaled.
__device__ __forceinline__ void op16_bf16(const bf16x8& a, const bf16x8& b, f32x4& c) { asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b)); }
__device__ __forceinline__ void op16_f8(const i32x8& a, const i32x8& b, f32x4& c) { asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b)); }
__device__ __forceinline__ void op16_sp_bf16(const bf16x8& a, const i32x8& b, uint32_t idx, f32x4& c) { asm volatile("v_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3" : "+a"(c) : "v"(a), "v"(b), "v"(idx)); }
__device__ __forceinline__ void op16_sp_f8(const bf16x8& a, const i32x8& b, uint32_t idx, f32x4& c) { asm volatile("v_smfmac_f32_16x16x128_fp8_fp8 %0, %1, %2, %3" : "+a"(c) : "v"(a), "v"(b), "v"(idx)); }
template <bool SPARSE, bool F8, int H, int M>
__device__ __forceinline__ void big_op(const BigFrags<SPARSE, F8>& f, f32x4 (&acc)[8][8]) {
  constexpr int mi = M / 4, n = M % 4, ni = 4 * H + n;
  if constexpr (!SPARSE && !F8) op16_bf16(f.a[mi][0], f.b[H][n][0], acc[mi][ni]);
  else if constexpr (!SPARSE) op16_f8(cat16(f.a[mi][0], f.a[mi][1]), cat16(f.b[H][n][0], f.b[H][n][1]), acc[mi][ni]);
  else if constexpr (!F8) op16_sp_bf16(f.a[mi][0], cat16(f.b[H][n][0], f.b[H][n][1]), f.idx[mi], acc[mi][ni]);
  else op16_sp_f8(f.a[mi][0], cat16(f.b[H][n][0], f.b[H][n][1]), f.idx[mi], acc[mi][ni]);
}
// fragment reads of A tile T (with its metadata) and of read I of B half H; buf: the stage's buffer, buf2: the second stage's (dense fp8)
template <class G, bool SPARSE, bool F8, int T, int TR = 0>
__device__ __forceinline__ void big_read_a(const char* buf, const char* buf2, const BigLane& L, BigFrags<SPARSE, F8>& f) {
  if constexpr ((TR & TR_A) != 0) { f.a[T][0] = tr_read<512>(buf + (L.a ^ ((T / 2) << 4)) + 8 * (T % 2)); return; }
  f.a[T][0] = *reinterpret_cast<const bf16x8*>(buf + L.a + T * (4 * 64));
  if constexpr (F8 && !SPARSE) f.a[T][1] = *reinterpret_cast<const bf16x8*>(buf2 + L.a + T * (4 * 64));
  if constexpr (SPARSE && F8) f.idx[T] = *reinterpret_cast<const uint32_t*>(buf + L.m + T * (8 * 16));
  if constexpr (SPARSE && !F8) f.idx[T] = *reinterpret_cast<const uint16_t*>(buf + L.m + T * (4 * 8));
}
template <class G, bool SPARSE, bool F8, int H, int I, int TR = 0>
__device__ __forceinline__ void big_read_b(const char* buf, const char* buf2, const BigLane& L, BigFrags<SPARSE, F8>& f) {
  // N-tile 4 H + n
  if constexpr ((TR & TR_B) != 0) {
    constexpr int n = SPARSE ? I / 2 : I, hi = SPARSE ? I % 2 : 0;
    f.b[H][n][hi] = tr_read<512>(buf + (L.b ^ (n << 4 | H << 3)) + hi * (16 * 512));
    return;
  }
  if constexpr (SPARSE) f.b[H][I / 2][I % 2] = *reinterpret_cast<const bf16x8*>(buf + (L.b ^ ((I % 2) << 5)) + (32 * (I / 2) + 4 * H) * 128);
  else if constexpr (F8) f.b[H][I / 2][I % 2] = *reinterpret_cast<const bf16x8*>((I % 2 ? buf2 : buf) + L.b + (32 * (I / 2) + 8 * H) * 64);
  else f.b[H][I][0] = *reinterpret_cast<const bf16x8*>(buf + L.b + (32 * I + 8 * H) * 64);
}

// Pacing of the DMA issue.  The four waves run in step, one per SIMD, and share one address unit that takes about
// 14 cycles per 16-byte-a-lane DMA instruction; an op takes 16 (dense fp8: 32) cycles.  When every wave hands over a DMA
// instruction on every 32 cycles, the unit is oversubscribed (4 x 14 > 32), the waves stall in the issue and their matrix
// pipes idle: measured per 512 cycles of matrix ops, the ones that carried 14 DMA instructions took 1200 cycles.  So they are spread over
// the whole step from its barrier to the next one: half of them in half 1, the rest in half 0 of the NEXT step, still into the buffer that the stage
// before freed -- one stage buffer is therefore half filled across a stage boundary, which costs nothing because the ring keeps NB - 2 whole
// stages in flight anyway.  One instruction on every 64 cycles (2:4, 13 or 14 a stage) or 128 (dense, 8 a stage).  Fragment reads take the slots between.
// which fragment read of B rides on op M of a half: two on every four ops
constexpr int big_read_slot(int M) { return M % 4 == 1 ? M / 4 * 2 : M % 4 == 2 ? M / 4 * 2 + 1 : -1; }
template <int SLOTS, int N> constexpr int paced(int M) { return M % SLOTS == 0 && M / SLOTS < N ? M / SLOTS : -1; }

// B k-major: N-tile 4 H + n of lane 4 g + i has column 32 g + 8 n + 4 (H ^ g % 2) + i (both halves of the 16-byte pieces are then read at a time,
// by neighbouring quads).  Of the eight columns in x, lane 4 g + i gets 32 g + 8 i + 0 .. 7.
__device__ __forceinline__ void unquad(float (&x)[8], int lane) {
  const bool swap = (lane & 4) != 0, odd = (lane & 1) != 0, upper = (lane & 2) != 0;
  constexpr int XOR1 = quad_perm(1, 0, 3, 2), XOR2 = quad_perm(2, 3, 0, 1);
#pragma unroll
  for (int n = 0; n < 4; n++) {
    const float a = x[n], b = x[4 + n];
    x[n] = swap ? b : a;
    x[4 + n] = swap ? a : b;
  }
#pragma unroll
  for (int h = 0; h < 8; h += 4) {
#pragma unroll
    for (int n = 0; n < 4; n += 2) {
      const float a = x[h + n], b = x[h + n + 1], qa = quad<XOR1>(a), qb = quad<XOR1>(b);
      x[h + n] = odd ? qb : a;
      x[h + n + 1] = odd ? b : qa;
    }
#pragma unroll
    for (int n = 0; n < 2; n++) {
      const float a = x[h + n], b = x[h + n + 2], qa = quad<XOR2>(a), qb = quad<XOR2>(b);
      x[h + n] = upper ? qb : a;
      x[h + n + 2] = upper ? b : qa;
    }
  }
}

template <bool SPARSE, class Epi, bool F8, int PROBE, int TR>
__device__ __forceinline__ void gemm_tile_big(const GemmArgs& g, const typename Epi::Args& ea, char* smem, int pid, int pid_end, int pid_step) {
  using G = Geo<SPARSE, F8, 4, 4>;
  constexpr int NB = G::NB, NDMA = G::NDMA - ((SPARSE && (PROBE & PROBE_FILL_LESS)) ? 3 : 0);
  constexpr bool PERSIST = (PROBE & PROBE_PERSIST) != 0, FRAG = (PROBE & PROBE_NO_FRAG) == 0, MATH = (PROBE & PROBE_NO_MFMA) == 0;
  constexpr int PACE = (PROBE & PROBE_UNPACED) ? 1 : F8 || SPARSE ? 4 : 8;
  using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>;

  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wy = wave >> 1, wx = wave & 1;
  int tm, tn;
  tile_coords<PROBE>(g.M / G::BM, g.N / G::BN, pid, tm, tn);
  int m0 = tm * G::BM, n0 = tn * G::BN;
  const int win = SPARSE ? ((q & 1) << 1) | (q >> 1) : q;      // chunk of A
  BigLane L;
  // lane c of a quarter holds row 32 (c / 4) + c % 4 of A's first tile
  L.a = (wy * 128 + 32 * (c >> 2) + (c & 3)) * 64 + ((win ^ swz4_big<SPARSE>(c)) << 4);
  L.b = SPARSE ? G::B_OFF + (wx * 128 + 8 * (c >> 2) + (c & 3)) * 128 + ((((q & 1) | ((q >> 1) << 2)) ^ swz8_big(c)) << 4)
               : G::B_OFF + (wx * 128 + 16 * (c >> 3) + (c & 7)) * 64 + ((q ^ swz4_big<false>(c)) << 4);
  if constexpr ((TR & TR_A) != 0) {
    const int k = 8 * q + (c >> 2);
    L.a = k * 512 + (((16 * wy + 4 * (c & 3)) ^ tr_swz_a<4, 4>(k)) << 4);
  }
  if constexpr ((TR & TR_B) != 0) {
    const int k = 8 * (SPARSE ? (q & 1) | (q >> 1) << 2 : q) + (c >> 2);
    L.b = G::B_OFF + k * 512 + (((16 * wx + 4 * (c & 3)) ^ tr_swz_b<4, 4>(k)) << 4) + 8 * (c & 1);
  }
  L.m = G::META_OFF + (F8 ? (2 * wy + (c >> 3)) * (1024 + 128) + ((c >> 2) & 1) * 64 + (c & 3) * 16 + 4 * win : (4 * wy + (c >> 2)) * (256 + 32) + (c & 3) * 8 + 2 * win);

  Dma<SPARSE, F8, PROBE, 4, 4, TR> dma;
  dma.init(g, m0, n0, tid);
  const int nk = g.K / G::BK;
  constexpr int STEP = F8 && !SPARSE ? 2 : 1;                  // stages a K step
  constexpr int H1 = NDMA * STEP / 2;                          // DMA instructions of a full step in half 1
  constexpr int AHEAD = NB - 1;                                // stages that are asked for before the first step ...
  constexpr int PART = STEP == 1 ? H1 : 0;                     // ... and instructions of the next one; the first step brings the rest of it
  const bool ring_full = nk > AHEAD;
  auto prologue = [&]() {
    const int n = ring_full ? AHEAD : nk;
    for (int s = 0; s < n; s++) static_for<NDMA>([&](auto J) { dma.template issue<J>(s, smem + s * G::STAGE); });
    if (PART > 0 && ring_full) static_for<PART>([&](auto J) { dma.template issue<J>(AHEAD, smem + AHEAD * G::STAGE); });
  };
  prologue();
  bool first = true;

  for (;;) {   // one pass per tile (PERSIST: several tiles per workgroup)
  f32x4 acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 8; j++) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      // Pin the accumulators to the accumulation register file: an empty asm with an AGPR constraint gives their
      // live ranges the AGPR class, so the 256 arch VGPRs stay free for fragments and addresses.
      asm volatile("" : "+a"(acc[i][j]));
    }
  BigFrags<SPARSE, F8> f;
  constexpr int NRB = SPARSE || F8 ? 8 : 4;                    // reads of half of B

  // the first step's stages have landed.  (A later tile's prologue went out before the previous epilogue, whose stores count in the same counter and
  // complete in no fixed order with the loads: wait for all of it.)
  if (first && ring_full) wait_vmcnt<(AHEAD - STEP) * NDMA + PART>(); else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  FFN24_FENCE();
  if constexpr (FRAG) {
    static_for<8>([&](auto T) { big_read_a<G, SPARSE, F8, T, TR>(smem, smem + G::STAGE, L, f); });
    static_for<NRB>([&](auto I) { big_read_b<G, SPARSE, F8, 0, I, TR>(smem, smem + G::STAGE, L, f); });
  }

  int slot = 0;
  auto ring = [&](int s) { return smem + (s >= NB ? s - NB : s) * G::STAGE; };
  // The step that starts with stage kt.  REST: its first half asks for what is left of stage kt - 1 + NB (dense fp8: for stage kt + 4); ISSUE: its second half
  // begins stage kt + NB; LEFT: DMA instructions behind the next step's that may be in flight at the barrier (-1: the last step,
  // no barrier and nothing to read)
  auto step = [&](int kt, auto rest, auto issue, auto left) {
    constexpr bool REST = decltype(rest)::value != 0, ISSUE = decltype(issue)::value != 0;
    constexpr int LEFT = decltype(left)::value;
    char *cur = ring(slot), *cur2 = ring(slot + 1), *nxt = ring(slot + STEP), *nxt2 = ring(slot + STEP + 1), *prv = ring(slot + NB - 1);
    FFN24_FENCE();
    static_for<32>([&](auto M) {
      if constexpr (MATH) big_op<SPARSE, F8, 0, M>(f, acc);
      constexpr int J = paced<PACE, NDMA - PART>(M);
      if constexpr (REST && J >= 0) dma.template issue<PART + (J >= 0 ? J : 0)>(kt - 1 + NB, prv);
      constexpr int I = big_read_slot(M);
      if constexpr (FRAG && I >= 0 && I < NRB) big_read_b<G, SPARSE, F8, 1, (I >= 0 ? I : 0), TR>(cur, cur2, L, f);
      FFN24_FENCE();
    });
    if constexpr (LEFT >= 0) {
      wait_vmcnt<(LEFT > 0 ? LEFT : 0)>();
      wait_lgkmcnt0();
      __builtin_amdgcn_s_barrier();
    }
    FFN24_FENCE();
    static_for<32>([&](auto M) {
      if constexpr (MATH) big_op<SPARSE, F8, 1, M>(f, acc);
      constexpr int J = paced<PACE, H1>(M);
      if constexpr (ISSUE && J >= 0) dma.template issue<(J >= 0 ? J : 0)>(kt + NB, cur);
      if constexpr (FRAG && LEFT >= 0) {
        constexpr int I = big_read_slot(M);
        if constexpr (I >= 0 && I < NRB) big_read_b<G, SPARSE, F8, 0, (I >= 0 ? I : 0), TR>(nxt, nxt2, L, f);
        if constexpr (M % 4 == 3) big_read_a<G, SPARSE, F8, M / 4, TR>(nxt, nxt2, L, f);
      }
      FFN24_FENCE();
    });
    slot += STEP;
    if (slot >= NB) slot -= NB;
  };
  using None = std::integral_constant<int, -1>;
  using Steady = std::integral_constant<int, STEP == 1 ? (NB - 2) * NDMA : NDMA>;
  int kt = 0;
  if (ring_full) {
    // (dense fp8: the number of stages is even, K is a multiple of 128, and stages kt + 4 and kt + 5 are there or not together)
    for (; kt < nk - NB; kt += STEP) step(kt, I1{}, I1{}, Steady{});
    if constexpr (STEP == 1) { step(kt, I1{}, I0{}, I0{}); kt++; }
  }
  for (; kt < nk - STEP; kt += STEP) step(kt, I0{}, I0{}, I0{});
  step(kt, I0{}, I0{}, None{});

  // let the last ops (8 passes each at most) drain before the epilogue reads the accumulators
  asm volatile("s_nop 15\n s_nop 15\n s_nop 15" ::: "memory");
  // and tie the accumulators to a point after the wait (volatile statements keep their order), so that no read of
  // them can be scheduled above it
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 8; j++) asm volatile("" : "+a"(acc[i][j]));
  // 16 rows of a lane are four M-tiles' registers.  (Single floats: as vectors of 16 they would each take 16 registers of the other file from the first
  // element read to the last one used, all 256, and spill what else an epilogue holds.)
  float out[2][8][16];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 8; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) out[i][j][v] = acc[4 * i + v / 4][j][v % 4];
  const int at = fresh_lane();
  if constexpr ((TR & TR_B) != 0) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; j++) x[j] = out[i][j][v];
        unquad(x, at);
#pragma unroll
        for (int j = 0; j < 8; j++) out[i][j][v] = x[j];
      }
  }
  const int m_lane = m0 + wy * 128 + 32 * (at >> 4), n_lane = n0 + wx * 128 + 8 * (at & 15);
  if constexpr (PERSIST) {
    pid += pid_step;
    const bool more = pid < pid_end;
    if (more) {
      // every wave has read its last fragments: the ring is free for the next tile's first stages, which then land while
      // the epilogue runs
      __builtin_amdgcn_s_barrier();
      tile_coords<PROBE>(g.M / G::BM, g.N / G::BN, pid, tm, tn);
      m0 = tm * G::BM; n0 = tn * G::BN;
      dma.init(g, m0, n0, tid);
      prologue();
    }
    Epi::template run<2, 8>(ea, out, m_lane, n_lane);
    if (!more) break;
    first = false;
  } else {
    run_epilogue<G, Epi, 2, 8>(ea, out, m_lane, n_lane, smem, wave);
    break;
  }
  }   // tiles
}

template <bool SPARSE, class Epi, bool F8 = false, int PROBE = 0, int MI = 4, int NI = 4, int TR = 0>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const typename Epi::Args& ea, char* smem, int pid, int pid_end = 0, int pid_step = 0) {
  static_assert(TR == 0 || (!F8 && !(SPARSE && (TR & TR_A))), "k-major operands: bf16, and a 2:4 operand has its own form");
  if constexpr (MI * NI == 16) gemm_tile_big<SPARSE, Epi, F8, PROBE, TR>(g, ea, smem, pid, pid_end, pid_step);
  else gemm_tile_small<SPARSE, Epi, F8, MI, NI, TR>(g, ea, smem, pid);
}

// Clock sample of a workgroup (profiling only): ticks of the shader clock and of the constant 100 MHz clock between its
// first and last instruction; their ratio is the clock the kernel really ran at (it drops well below the nominal 2.4 GHz
// under matrix load).
struct ClkSample {
  unsigned long long t0, r0;
  int wave;
  __device__ __forceinline__ void begin(const GemmArgs& g) {
    wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (g.clk) { t0 = __builtin_amdgcn_s_memtime(); r0 = __builtin_amdgcn_s_memrealtime(); }
  }
  __device__ __forceinline__ void end(const GemmArgs& g) {
    if (g.clk && blockIdx.x < CLK_SLOTS) {
      unsigned long long t1 = __builtin_amdgcn_s_memtime(), r1 = __builtin_amdgcn_s_memrealtime();
      if (wave == 0 && fresh_lane() == 0) { g.clk[2 * blockIdx.x] = t1 - t0; g.clk[2 * blockIdx.x + 1] = r1 - r0; }
    }
  }
};

template <bool SPARSE, class Epi, bool F8 = false, int PROBE = 0, int MI = 4, int NI = 4>
__global__ void __launch_bounds__(GEMM_THREADS, (Geo<SPARSE, F8, MI, NI>::PER_CU)) gemm_kernel(GemmArgs g, typename Epi::Args ea) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  ClkSample cs;
  cs.begin(g);
  gemm_tile<SPARSE, Epi, F8, PROBE, MI, NI>(g, ea, smem, blockIdx.x, (g.M / TILE_M) * (g.N / TILE_N), gridDim.x);
  cs.end(g);
}

// The same with a k-major operand.
template <bool SPARSE, class Epi, int TR, int MI, int NI>
__global__ void __launch_bounds__(GEMM_THREADS, (Geo<SPARSE, false, MI, NI>::PER_CU)) gemm_k_major_kernel(GemmArgs g, typename Epi::Args ea) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  ClkSample cs;
  cs.begin(g);
  gemm_tile<SPARSE, Epi, false, 0, MI, NI, TR>(g, ea, smem, blockIdx.x);
  cs.end(g);
}

// A GEMM and other work that neither waits for it nor it for: the workgroups from n_tiles on run Side (stream_core.hpp), on what the tiles leave of the chip.
template <bool SPARSE, class Epi, int TR, int MI, int NI, class Side>
__global__ void __launch_bounds__(GEMM_THREADS, (Geo<SPARSE, false, MI, NI>::PER_CU)) gemm_side_kernel(GemmArgs g, typename Epi::Args ea, int n_tiles,
                                                                                                        typename Side::Args sa) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if ((int)blockIdx.x < n_tiles) gemm_tile<SPARSE, Epi, false, 0, MI, NI, TR>(g, ea, smem, blockIdx.x);
  else Side::run(sa, blockIdx.x - n_tiles, smem);
}

// A dense and a sparse GEMM (same epilogue type, separate arguments, same N and K) in one launch, for one weight gradient or for both
// (`sets` = 2).  The split weight-gradient GEMMs use it (Sec. 2, "Optimization 1": a 2:4 GEMM over most hidden features plus a dense one
// over the few that are not sparse enough): alone, the small dense GEMM would occupy a fraction of the CUs for as long as a full round
// of tiles.  The dense tiles, which take longer, come first, those of both sets before any sparse one: with one set a launch, a
// shape whose sparse tiles take just one round waited twice for its dense tiles (fp8, T = F = 8192, D = 2048, 512 dense features: 2 x
// 93-97 us; both sets in one launch: 178 us).
template <class Epi>
struct PairSet { GemmArgs gd; typename Epi::Args ed; GemmArgs gs; typename Epi::Args es; };

template <class Epi, bool F8 = false, int MI = 4, int NI = 4, int TR = 0>
__global__ void __launch_bounds__(GEMM_THREADS, (Geo<true, F8, MI, NI>::PER_CU)) gemm_pair_kernel(PairSet<Epi> a, PairSet<Epi> b, int sets, int nd_tiles,
                                                                                                 int ns_tiles) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int pid = blockIdx.x;
  ClkSample cs;
  cs.begin(a.gs);
  if (pid < sets * nd_tiles) {
    GemmArgs g = a.gd;                   // (the sets differ in their operands only)
    typename Epi::Args e = a.ed;
    if (pid >= nd_tiles) { pid -= nd_tiles; g.A = b.gd.A; g.B = b.gd.B; e = b.ed; }
    gemm_tile<false, Epi, F8, 0, MI, NI, TR>(g, e, smem, pid);
  } else {
    pid -= sets * nd_tiles;
    GemmArgs g = a.gs;
    typename Epi::Args e = a.es;
    if (pid >= ns_tiles) { pid -= ns_tiles; g.A = b.gs.A; g.Ameta = b.gs.Ameta; g.B = b.gs.B; e = b.es; }
    gemm_tile<true, Epi, F8, 0, MI, NI, TR>(g, e, smem, pid);
  }
  cs.end(a.gs);
}

// Two GEMMs of one kind and size in one launch, each with its own epilogue: workgroups [0, n_first) take the tiles of the first.  The two
// weight gradients of a step run like this where one of them alone would leave CUs idle.  One main loop serves both; EpiB is a staged
// epilogue (transposing store), EpiA a plain one.
template <class EpiA, class EpiB>
struct EpiDuo {
  static constexpr bool STAGED = true;
  struct Args { typename EpiA::Args a; typename EpiB::Args b; bool second; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    if (e.second) EpiB::template run<MI, NI>(e.b, acc, m_lane, n_lane, wbuf);
    else EpiA::template run<MI, NI>(e.a, acc, m_lane, n_lane);
  }
};
template <bool SPARSE, class EpiA, class EpiB, bool F8, int MI, int NI, int TR>
__global__ void __launch_bounds__(GEMM_THREADS, (Geo<SPARSE, F8, MI, NI>::PER_CU)) gemm_duo_kernel(GemmArgs ga, typename EpiA::Args ea, int n_first,
                                                                                                  GemmArgs gb, typename EpiB::Args eb) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int bid = blockIdx.x;
  const bool second = bid >= n_first;
  GemmArgs g = ga;                       // (same M, N, K and operand forms)
  if (second) { g.A = gb.A; g.Ameta = gb.Ameta; g.B = gb.B; }
  const typename EpiDuo<EpiA, EpiB>::Args e{ea, eb, second};
  gemm_tile<SPARSE, EpiDuo<EpiA, EpiB>, F8, 0, MI, NI, TR>(g, e, smem, second ? bid - n_first : bid);
}

// ------------------------------------------------------------------------------------------------
// the sparse GEMM on a caller's row-major operands (spmm24)
// ------------------------------------------------------------------------------------------------
// Row-major, the 64 k of a stage are 64 bytes of an A row, half a line, and 8 bytes of metadata: 256 of the 128 x 64 tile's 320 requests a stage
// are for pieces of a line, and a CU's global->LDS stream takes about three cycles a request whatever its size (the main loop above
// spent 53.2 of its 54.5 us at M 2048 N 1024 K 8256 waiting for it, now 37.6 in all; in panel form the same stream takes 25.7).  So a ring slot here holds
// 128 k: whole lines of A, 16 bytes of metadata a row, and B as two halves of 64 k in the layout of the loop above.  The halves are
// walked with two register sets, each read while the other's matrix ops run; one wait and one barrier for both.  K need not be a
// multiple of 128: lanes that would pass the end of a row fetch its last bytes again, and the last half is not walked.  Every
// second row of A then starts in the middle of a line.  SHIFT (taken then by the 128 x 64 tile, which has four slots): a slot holds those rows' 128 bytes
// from 64 before, so that they are whole lines too, their two halves stand the other way round, and the second half
// of what the others have in slot kt is the first of slot kt + 1 (K 8256, 128 x 64: 39.7 us, 43.9 without, 34.4 with K 8192).  Three slots leave
// no time for it: 128 x 128 at K 8256 65 us against 53 without, 64 x 64 at M N 512 K 2112 8.3 against 7.7 and at K 8256 42.7 against 25.6.
template <int MI, int NI>
struct GeoRows {
  static constexpr int BM = 64 * MI, BN = 64 * NI, BK = 128;
  static constexpr int A_BYTES = BM * 128, META_BYTES = BM * 16, B_HALF = BN * 128;
  static constexpr int META_OFF = A_BYTES, B_OFF = A_BYTES + META_BYTES, STAGE = B_OFF + 2 * B_HALF;
  static constexpr int NB = MI * NI == 8 ? 2 : MI * NI == 2 ? 4 : 3;    // slots: what the LDS holds, of the smallest tile what half of it holds
  static constexpr int LDS_TOTAL = NB * STAGE, PER_CU = LDS_TOTAL <= 80 * 1024 ? 2 : 1;
  static constexpr int NA = 2 * MI, NM = MI, NVB = 4 * NI, NDMA = NA + NM + NVB;   // DMA instructions per wave and slot
};

template <int MI, int NI, bool SHIFT>
struct DmaRows {
  using G = GeoRows<MI, NI>;
  const char *a, *am, *b;
  uint32_t ra[G::NA], rm[G::NM], rb[G::NVB];        // the lane's row, as a byte offset from the uniform bases
  uint32_t la, lm, lb;                              // the last place inside a row that a fetch may start at
  int wave;
  __device__ __forceinline__ void init(const GemmArgs& g, int m0, int n0, int tid) {
    const int lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t a_row = (uint32_t)g.K, m_row = (uint32_t)g.K / 8, b_row = 2 * (uint32_t)g.K;
    a = static_cast<const char*>(g.A) + (size_t)m0 * a_row;
    am = reinterpret_cast<const char*>(g.Ameta) + (size_t)m0 * m_row;
    b = static_cast<const char*>(g.B) + (size_t)n0 * b_row;
    la = a_row - 16; lm = m_row - 4; lb = b_row - 16;
    // 8 rows of 128 bytes an instruction
#pragma unroll
    for (int j = 0; j < G::NA; j++) ra[j] = (uint32_t)unperm_m<MI>(8 * (G::NA * wave + j) + (lane >> 3)) * a_row;
    // 16 rows of 16 bytes, a dword a lane
#pragma unroll
    for (int j = 0; j < G::NM; j++) rm[j] = (uint32_t)unperm_m<MI>(16 * (G::NM * wave + j) + (lane >> 2)) * m_row;
    // the two halves of B lie one after the other; 8 rows of 128 bytes an instruction
#pragma unroll
    for (int j = 0; j < G::NVB; j++) rb[j] = (uint32_t)unperm_n<NI>((8 * (G::NVB * wave + j) + (lane >> 3)) & (G::BN - 1)) * b_row;
  }
  template <int J>
  __device__ __forceinline__ void issue(int kt, char* buf) const {
    const int lane = threadIdx.x & 63;
    if constexpr (J < G::NA) {
      const int p = 8 * (G::NA * wave + J) + (lane >> 3);
      const int at = kt * 128 + (((lane & 7) ^ swz8(p)) << 4) - (SHIFT ? (p & 1) << 6 : 0);   // (unperm_m keeps the low bits: odd rows)
      const uint32_t in = (uint32_t)min(max(at, 0), (int)la);
      __builtin_amdgcn_global_load_lds((glb_char*)(a + (ra[J] + in)), (lds_char*)(buf + (G::NA * wave + J) * 1024), 16, 0, 0);
    } else if constexpr (J < G::NA + G::NM) {
      constexpr int j = J - G::NA;
      const uint32_t in = min((uint32_t)kt * 16u + 4u * (lane & 3), lm);
      __builtin_amdgcn_global_load_lds((glb_char*)(am + (rm[j] + in)), (lds_char*)(buf + G::META_OFF + (G::NM * wave + j) * 256), 4, 0, 0);
    } else {
      constexpr int j = J - G::NA - G::NM;
      const int q = 8 * (G::NVB * wave + j), p = (q + (lane >> 3)) & (G::BN - 1);   // (an instruction's 8 rows lie in one half)
      const uint32_t in = min((uint32_t)kt * 256u + (q >= G::BN ? 128u : 0u) + (uint32_t)(((lane & 7) ^ swz8(p)) << 4), lb);
      __builtin_amdgcn_global_load_lds((glb_char*)(b + (rb[j] + in)), (lds_char*)(buf + G::B_OFF + (G::NVB * wave + j) * 1024), 16, 0, 0);
    }
  }
};

// read I of half HALF of the slot at buf (the order of StageRegs<true>: metadata, then the fragments of either K step); abuf: the slot that
// holds this lane's A rows
template <int MI, int NI, int HALF, int I>
__device__ __forceinline__ void read_rows(const char* buf, const char* abuf, const LaneCtx& L, StageRegs<true, false, MI, NI>& r) {
  using G = GeoRows<MI, NI>;
  constexpr int NF = MI + 2 * NI;
  if constexpr (I < MI) {
    r.idx[I].w[0] = *reinterpret_cast<const uint32_t*>(buf + G::META_OFF + (L.wy * (32 * MI) + L.rho + 32 * I) * 16 + 8 * HALF + 4 * L.h);
  } else {
    constexpr int S = (I - MI) / NF, i = (I - MI) % NF;
    FragS<MI, NI>& f = r.f[S];
    if constexpr (i < MI) {
      f.a[i] = *reinterpret_cast<const bf16x8*>(abuf + L.a_row128 + i * (32 * 128) + (((4 * HALF + 2 * L.h + S) ^ L.sw8a ^ ((i & 1) << 2)) << 4));
    } else {
      constexpr int n = (i - MI) % NI;
      const int sw = L.sw8 ^ ((n & 1) << 2);
      const char* row = buf + G::B_OFF + HALF * G::B_HALF + L.b_row128 + n * (32 * 128);
      if constexpr (i < MI + NI) f.blo[n] = *reinterpret_cast<const bf16x8*>(row + (((2 * S + L.h) ^ sw) << 4));
      else f.bhi[n] = *reinterpret_cast<const bf16x8*>(row + (((4 + 2 * S + L.h) ^ sw) << 4));
    }
  }
}

template <class Epi, int MI, int NI, bool SHIFT>
__global__ void __launch_bounds__(GEMM_THREADS, (GeoRows<MI, NI>::PER_CU)) gemm_rows_kernel(GemmArgs g, typename Epi::Args ea) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  using G = GeoRows<MI, NI>;
  using SR = StageRegs<true, false, MI, NI>;
  constexpr int NB = G::NB, NDMA = G::NDMA;
  constexpr int AHEAD = SHIFT ? 2 : 1;               // slots beyond the present one that must have landed when its second half begins
  static_assert(NB > AHEAD, "a slot is asked for after that");
  const int tid = threadIdx.x;
  int tm, tn;
  tile_coords<0, MI == 2 * NI>(g.M / G::BM, g.N / G::BN, blockIdx.x, tm, tn);
  const int m0 = tm * G::BM, n0 = tn * G::BN;
  const int lane = tid & 63, wave = tid >> 6;
  LaneCtx L = {};
  L.rho = lane & 31; L.h = lane >> 5; L.wy = wave >> 1; L.wx = wave & 1;
  L.a_row128 = (L.wy * (32 * MI) + L.rho) * 128;
  L.b_row128 = (L.wx * (32 * NI) + L.rho) * 128;
  L.sw8 = NI == 1 ? swz8(L.wx * 32 + L.rho) : swz8(L.rho);
  L.sw8a = MI == 1 ? swz8(L.wy * 32 + L.rho) : swz8(L.rho);
  const bool shifted = SHIFT && (L.rho & 1);
  if (shifted) L.sw8a ^= 4;                          // the halves the other way round
  DmaRows<MI, NI, SHIFT> dma;
  dma.init(g, m0, n0, tid);
  const int nk = (g.K + G::BK - 1) / G::BK;         // at least NB (launch_rows_tile)
  const bool odd = (g.K & 64) != 0;                  // the last slot's second half does not exist
  for (int s = 0; s < NB; s++) static_for<NDMA>([&](auto J) { dma.template issue<J>(s, smem + s * G::STAGE); });
  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
  wait_vmcnt<(NB - AHEAD) * NDMA>();
  __builtin_amdgcn_s_barrier();
  FFN24_FENCE();
  SR r0, r1;
  static_for<SR::READS>([&](auto I) { read_rows<MI, NI, 0, I>(smem, smem, L, r0); });
  // first half of a slot; the second half's fragments are read meanwhile
  auto first = [&](const char* cur, const char* nxt) {
    const char* abuf = shifted ? nxt : cur;
    static_for<SR::OPS>([&](auto M) {
      r0.template op<M>(acc);
      ride<SR::READS, SR::READ_SLOTS, M>([&](auto I) { read_rows<MI, NI, 1, I>(cur, abuf, L, r1); });
      FFN24_FENCE();
    });
  };
  // second half; the next slot's first fragments are read and, ISSUE, the slot kt + NB asked for into this slot, which every wave has read
  auto second = [&](int kt, char* cur, const char* nxt, auto issue, auto more) {
    constexpr bool ISSUE = decltype(issue)::value, MORE = decltype(more)::value;
    static_for<SR::OPS>([&](auto M) {
      r1.template op<M>(acc);
      if constexpr (MORE) ride<SR::READS, SR::READ_SLOTS, M>([&](auto I) { read_rows<MI, NI, 0, I>(nxt, nxt, L, r0); });
      if constexpr (ISSUE) ride<NDMA, SR::OPS, M>([&](auto J) { dma.template issue<J>(kt + NB, cur); });
      FFN24_FENCE();
    });
  };
  using Yes = std::true_type; using No = std::false_type;
  int slot = 0;
  auto advance = [&](int kt, auto issue, auto left) {
    constexpr int LEFT = decltype(left)::value;
    const int ns = slot + 1 == NB ? 0 : slot + 1;
    char *cur = smem + slot * G::STAGE, *nxt = smem + ns * G::STAGE;
    FFN24_FENCE();
    first(cur, nxt);
    wait_vmcnt<(LEFT > 0 ? LEFT : 0) * NDMA>();      // slot kt + AHEAD has landed; LEFT later ones may be in flight
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    FFN24_FENCE();
    second(kt, cur, nxt, issue, Yes{});
    slot = ns;
  };
  int kt = 0;
  for (; kt < nk - NB; kt++) advance(kt, Yes{}, std::integral_constant<int, NB - 1 - AHEAD>{});
  static_for<NB - 1>([&](auto i) { advance(kt + decltype(i)::value, No{}, std::integral_constant<int, NB - 1 - AHEAD - decltype(i)::value>{}); });
  first(smem + slot * G::STAGE, smem + slot * G::STAGE);   // (reads a second half even where there is none: nothing is made of it)
  if (!odd) second(0, smem, smem, No{}, No{});
  Epi::template run<MI, NI>(ea, acc, m0 + L.wy * (32 * MI) + (16 * MI) * L.h, n0 + L.wx * (32 * NI) + NI * L.rho);
}

// ------------------------------------------------------------------------------------------------
// small device helpers shared by the epilogues
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = (__bf16)lo;   // round-to-nearest-even
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf16_lo_to_f32(uint32_t pk) { return __builtin_bit_cast(float, pk << 16); }
__device__ __forceinline__ float bf16_hi_to_f32(uint32_t pk) { return __builtin_bit_cast(float, pk & 0xFFFF0000u); }

// Keep-2-of-4 on four storage words (Sec. 2 of the paper: keep the two largest magnitudes of each block of 4;
// ties go to the lower index).  k_i = (magnitude << 2) | (3 - i) makes all four keys distinct and orders them
// by (magnitude, then lower index first), so the two largest keys are the picks.
// Returns the nibble i0 | i1<<2 and the two kept keys ordered by position (key_first has the lower index).
__device__ __forceinline__ uint32_t pick24_keys(uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3,
                                                uint32_t& key_first, uint32_t& key_second) {
  uint32_t a = max(k0, k1), b = min(k0, k1), c = max(k2, k3), d = min(k2, k3);
  uint32_t top = max(a, c);
  uint32_t e = max(b, d);
  uint32_t second = max(min(a, c), min(max(a, c), e));         // median of (a, c, e) = second largest of the four
  uint32_t ct = top & 3u, cs = second & 3u;                    // 3 - index
  bool top_first = ct > cs;                                    // larger complement = lower index
  key_first = top_first ? top : second;
  key_second = top_first ? second : top;
  uint32_t cmax = max(ct, cs), cmin = min(ct, cs);
  return (cmax | (cmin << 2)) ^ 15u;
}

// The pick for two groups at a time (the activation epilogues): p_i holds entry i of one group in its low half and entry i of another in
// its high half, non-negative bf16 words (15 bits, so that 16-bit differences keep their sign and integer order is value order).  No key
// with the position in it is needed: with a = max, b = min of entries 0, 1 and c, d those of 2, 3, both of the first pair stay
// iff b >= c, both of the second iff d > a, and otherwise the larger of each pair, the earlier one if they are equal (ties go to the
// lower index throughout).  All of it is packed 16-bit and bitwise arithmetic: 28 instructions for two groups and their
// metadata against 44 with one group at a time and 32-bit keys, in an epilogue that overlaps with nothing.  T = F = 8192, D = 2048: bf16
// up-projection 223 -> 221 us, row-wise fp8 with the per-feature counts, 256 x 128 tiles, 146 -> 128 (133 -> 123 without).
// first, second: the kept entries in position order; bits: the nibble i0 | i1 << 2 of each half as four masks.
struct Pick24x2 { uint32_t first, second, bit[4]; };
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ i16x2 as_i16x2(uint32_t w) { return __builtin_bit_cast(i16x2, w); }
__device__ __forceinline__ uint32_t pk_max16(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(as_i16x2(a), as_i16x2(b))); }
__device__ __forceinline__ uint32_t pk_min16(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(as_i16x2(a), as_i16x2(b))); }
__device__ __forceinline__ uint32_t pk_less16(uint32_t a, uint32_t b) {   // all ones in the halves where a < b
  uint32_t m = __builtin_bit_cast(uint32_t, (i16x2)((as_i16x2(a) - as_i16x2(b)) >> (i16x2)(15)));
  asm("" : "+v"(m));   // opaque: the compiler would turn the masks back into a compare and a select for each half
  return m;
}
__device__ __forceinline__ Pick24x2 pick24_two(uint32_t p0, uint32_t p1, uint32_t p2, uint32_t p3) {
  const uint32_t a = pk_max16(p0, p1), b = pk_min16(p0, p1), c = pk_max16(p2, p3), d = pk_min16(p2, p3);
  const uint32_t some = pk_less16(b, c);         // not both of the first pair
  const uint32_t late = pk_less16(a, d);         // both of the second pair (then `some` is set too)
  const uint32_t e = pk_less16(p0, p1), f = pk_less16(p2, p3);
  Pick24x2 r;
  r.first = (late & p2) | (~late & ((some & a) | (~some & p0)));
  r.second = (some & ((late & p3) | (~late & c))) | (~some & p1);
  r.bit[0] = e & some & ~late;
  r.bit[1] = late;
  r.bit[2] = ~some | late | f;
  r.bit[3] = some;
  return r;
}
// the nibbles of a pick at bits 4 k of both halves of w
__device__ __forceinline__ uint32_t put_nibbles(uint32_t w, const Pick24x2& p, int k) {
#pragma unroll
  for (int i = 0; i < 4; i++) w |= p.bit[i] & (0x00010001u << (4 * k + i));
  return w;
}

}  // namespace ffn24
