// Epilogues of the GEMM core: what happens to a lane's accumulators.
// A lane owns rows m_lane + 16*mi + v (16 MI consecutive) and columns n_lane + ni (NI consecutive), MI x NI = 2 x 8 for the 256 x 256
// block tile and 4 x 2 to 1 x 1 for the smaller ones.  Where a lane holds less than a whole piece of a panel form (64 features), it starts
// m_lane % 64 features into it.
#pragma once
#include "gemm_core.hpp"
#include "launch.hpp"
#include "tile_rule.hpp"

namespace ffn24 {

// (counted: an epilogue that needs it does not keep the work item's number in a register through the main loop)
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// How a wave's lanes share its part of the tile: LANES consecutive ones hold the same 16 MI rows and side by side NI columns each.
template <int MI, int NI>
struct LaneTile {
  static constexpr int LANES = NI == 8 ? 16 : 32, GROUPS = 64 / LANES;
  static constexpr int ROWS = GROUPS * 16 * MI, COLS = LANES * NI;      // of the wave
  // the wave holds whole runs of the panel forms, which go through LDS
  static constexpr bool STAGED = ROWS == 128;
  static __device__ __forceinline__ int rho() { return lane_id() & (LANES - 1); }             // which columns
  static __device__ __forceinline__ int h() { return lane_id() / LANES; }              // which rows
};

// Sums two 16-bit fields over the wave (each field's total must stay below 65536) and has lane 0 add them to slot
// `slot` of quantities ka and kb.
__device__ __forceinline__ void tele_add2(unsigned long long* tele, uint32_t packed, int ka, int kb, int slot) {
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) packed += (uint32_t)__shfl_xor((int)packed, sft, 64);
  if (lane_id() == 0) {
    atomicAdd(tele + tele_index(ka, slot), (unsigned long long)(packed & 0xFFFFu));
    if (kb >= 0) atomicAdd(tele + tele_index(kb, slot), (unsigned long long)(packed >> 16));
  }
}

// A per-feature fp32 vector (bias, weight scale) over the lane's 16 MI features from m_lane on, loaded once with
// 16-byte loads and shared by the lane's tokens; `fill` everywhere if the vector is absent.
template <int MI>
struct LaneVec {
  f32x4 v[4 * MI];
  __device__ __forceinline__ void load(const float* p, int m_lane, float fill) {
#pragma unroll
    for (int i = 0; i < 4 * MI; i++) v[i] = f32x4{fill, fill, fill, fill};
    if (p) {
#pragma unroll
      for (int i = 0; i < 4 * MI; i++) v[i] = *reinterpret_cast<const f32x4*>(p + m_lane + 4 * i);
    }
  }
  __device__ __forceinline__ float at(int i) const { return v[i >> 2][i & 3]; }   // feature m_lane + i
};

// The lane's 16 MI entries of a row map from m_lane on, loaded with 16-byte loads (the map and m_lane are 16-byte aligned).
template <int MI>
struct LaneIdx {
  i32x4 v[4 * MI];
  __device__ __forceinline__ void load(const int* p, int m_lane) {
#pragma unroll
    for (int i = 0; i < 4 * MI; i++) v[i] = *reinterpret_cast<const i32x4*>(p + m_lane + 4 * i);
  }
  __device__ __forceinline__ int at(int i) const { return v[i >> 2][i & 3]; }
};

// The 4 MI nibbles of a lane's groups (MI 16-bit words, low group first) to and from the metadata bytes.
template <int MI> __device__ __forceinline__ void st_nibbles(uint8_t* p, const uint32_t (&nib)[2]) {
  if constexpr (MI == 4) *reinterpret_cast<u32x2*>(p) = u32x2{nib[0], nib[1]};
  else if constexpr (MI == 2) *reinterpret_cast<uint32_t*>(p) = nib[0];
  else *reinterpret_cast<uint16_t*>(p) = (uint16_t)nib[0];
}
template <int MI> __device__ __forceinline__ u32x2 ld_nibbles(const uint8_t* p) {
  if constexpr (MI == 4) return *reinterpret_cast<const u32x2*>(p);
  else if constexpr (MI == 2) return u32x2{*reinterpret_cast<const uint32_t*>(p), 0u};
  else return u32x2{*reinterpret_cast<const uint16_t*>(p), 0u};
}

// NI consecutive bf16 results of one row, rounded and stored in one go
template <int NI> __device__ __forceinline__ void st_cols(__bf16* p, const float (&x)[NI]) {
  if constexpr (NI == 8) *reinterpret_cast<u32x4*>(p) = u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
  else if constexpr (NI == 2) *reinterpret_cast<uint32_t*>(p) = pack_bf16x2(x[0], x[1]);
  else *p = (__bf16)x[0];
}
// byte b of NI words, stored as NI consecutive bytes
template <int NI> __device__ __forceinline__ void st_bytes(uint8_t* p, const uint32_t (&w)[NI], int b) {
  uint32_t o[2] = {};
#pragma unroll
  for (int i = 0; i < NI; i++) o[i / 4] |= ((w[i] >> (8 * b)) & 0xFFu) << (8 * (i % 4));
  if constexpr (NI == 8) *reinterpret_cast<u32x2*>(p) = u32x2{o[0], o[1]};
  else if constexpr (NI == 2) *reinterpret_cast<uint16_t*>(p) = (uint16_t)o[0];
  else *p = (uint8_t)o[0];
}
// 2 MI words (8 MI bytes) of e4m3 codes
template <int MI> __device__ __forceinline__ void st_codes(uint8_t* p, const uint32_t (&q)[2 * MI]) {
  if constexpr (MI == 1) *reinterpret_cast<u32x2*>(p) = u32x2{q[0], q[1]};
  else {
#pragma unroll
    for (int i = 0; i < MI / 2; i++) *reinterpret_cast<u32x4*>(p + 16 * i) = u32x4{q[4 * i], q[4 * i + 1], q[4 * i + 2], q[4 * i + 3]};
  }
}

// HERE: x is computed here.  What an epilogue collects tile by tile and uses at its end (row maxima, counts, metadata) the compiler otherwise
// moves there, with all the words it is made of kept until then.  In the row-wise 2:4 epilogue on 256 x 256 tiles that is 200 of them beside
// the accumulators, and spilled 7-9 registers; where nothing spills it is the better order (row-wise with counts, 256 x 128, T 2048 D
// 1024 F 4096: 17.4 us, 18.4 with HERE; bf16 with counts 256 x 256 T = F = 8192 242.5, 245).
template <bool HERE> __device__ __forceinline__ void keep_here(uint32_t& x) { if constexpr (HERE) asm volatile("" : "+v"(x)); }

// A wave's part of an operand in a bf16 panel form (MI = 4: a lane's 64 features of a token are one 64-byte piece, or two of a dense operand, the
// two lane halves two panels, or four), through LDS.  A store instruction of a lane's own pieces would put 64 16-byte parts into 64 different lines, 16 times
// over with 4 columns; the wave's tokens are neighbours, so what it owns of a panel is one contiguous run of 2 NI KiB.  The pieces go to
// a wave-private image in the operand ring (free by then) and leave, or come in, as whole kilobytes: LDS rows are 256 bytes = 4 tokens, and
// 16-byte place s of row r holds the run's s ^ (r & 15), so that the lanes of an LDS instruction meet in no bank either way.
// 256 x 128 tiles, D 2048: row-wise fp8 dH at T = F = 8192 129 -> 120 us, its up-projection 124 -> 119; bf16 at T 4096 F 8192 dH 120 -> 115.5, up-projection
// 119.5 -> 117.  256 x 256, T = F = 8192: bf16 dH 227.5 -> 225.7, row-wise fp8 140 -> 133, the up-projections within 1 %.
// Dense form: a bf16 dense step at T 4096 D 2048 F 8192 762 -> 751 us (up-projection and dH 157 -> 142 each in a kernel trace).
// P: panels of 64 features (1: the 2:4 form, 64 features of 32 kept values each; 2: the dense form, 32 features each).
template <int MI, int NI, int P = 1>
struct PanelStage {
  using LT = LaneTile<MI, NI>;
  static constexpr int RUN = LT::COLS * 64;          // a panel's run: bytes of the wave's tokens
  static constexpr size_t PANEL = 256 * 64;          // from one panel's pieces to the next one's in memory
  static constexpr int PARTS = P * MI;               // 16-byte parts of a token that a lane holds
  static constexpr int RUNS = 2 * P, KB = RUN / 1024;
  // place of part s of LDS row r: rows that lanes next to each other write to differ in the four bits that are taken
  static __device__ __forceinline__ int swz(int r, int s) { return r * 256 + ((s ^ ((NI == 8 ? r >> 1 : r) & 15)) << 4); }
  static __device__ __forceinline__ char* at(char* wbuf, int ni, int part) {   // part `part` of the lane's of its token ni
    const int tok = NI * LT::rho() + ni, p = LT::h() * PARTS + part;
    return wbuf + (p >> 2) * RUN + swz(tok >> 2, (tok & 3) * 4 + (p & 3));
  }
  // the wave's first piece of its lowest panel
  static __device__ __forceinline__ size_t first(int m_lane, int n_lane, int F) {
    return a24_piece(n_lane - NI * LT::rho(), ((m_lane - 16 * MI * LT::h()) >> 6) * P, F / (64 / P)) * 64;
  }
  static __device__ __forceinline__ void flush(const char* wbuf, char* out) {
    const int lane = lane_id();
#pragma unroll
    for (int j = 0; j < RUNS * KB; j++) {
      const int q = j % KB, r = 4 * q + (lane >> 4);
      *reinterpret_cast<u32x4*>(out + (j / KB) * PANEL + q * 1024 + 16 * lane) = *reinterpret_cast<const u32x4*>(wbuf + (j / KB) * RUN + swz(r, lane & 15));
    }
  }
  // by DMA: the caller waits for vmcnt(0) before the first `at`
  static __device__ __forceinline__ void fetch(char* wbuf, const char* in) {
    const int lane = lane_id();
#pragma unroll
    for (int j = 0; j < RUNS * KB; j++) {
      const int q = j % KB, r = 4 * q + (lane >> 4);
      __builtin_amdgcn_global_load_lds((glb_char*)(in + (j / KB) * PANEL + swz(r, lane & 15)), (lds_char*)(wbuf + j * 1024), 16, 0, 0);
    }
  }
};

// What the backward epilogues read back of the forward's saved activation, for the lane's tokens x features, requested in one
// go before any arithmetic or store: a load placed inside the loops is followed by stores through pointers the compiler must assume
// may alias, so each one waited out a full memory round trip by itself (16 of them in the 2:4 epilogue, 32 in the dense one -- the
// latter had made the dense dH kernel 0.4 ms slower than the GEMM alone).
// 2:4: one 64-byte piece (or part) of kept values + its metadata bytes per token (bf16 panel form).
// LaneTile::STAGED: the kept values come through LDS (PanelStage) and are read from there token by token, `wbuf` staying the place a result of the same
// form may be put to piece by piece.
template <int MI, int NI>
struct LaneSaved24 {
  static constexpr bool STAGED = LaneTile<MI, NI>::STAGED;
  u32x4 h[STAGED ? 1 : NI][MI];    // [ni][mi]: the kept values of groups 4 mi .. 4 mi + 3
  u32x2 mt[NI];
  char* wbuf;
  __device__ __forceinline__ u32x4 kept(int ni, int mi) const {
    if constexpr (STAGED) return *reinterpret_cast<const u32x4*>(PanelStage<MI, NI>::at(wbuf, ni, mi));
    else return h[ni][mi];
  }
  __device__ __forceinline__ void load(const __bf16* Hc, const uint8_t* meta, int F, int m_lane, int n_lane, char* buf) {
    wbuf = buf;
    if constexpr (STAGED) {
      PanelStage<MI, NI>::fetch(wbuf, reinterpret_cast<const char*>(Hc) + PanelStage<MI, NI>::first(m_lane, n_lane, F));
#pragma unroll
      for (int ni = 0; ni < NI; ni++) mt[ni] = ld_nibbles<MI>(meta + a24_piece(n_lane + ni, m_lane >> 6, F >> 6) * 8 + ((m_lane & 63) >> 3));
      wait_vmcnt<0>();
      asm volatile("" ::: "memory");                 // (the compiler does not see the DMA write what `kept` reads)
      return;
    }
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      size_t piece = a24_piece(n_lane + ni, m_lane >> 6, F >> 6);
      mt[ni] = ld_nibbles<MI>(meta + piece * 8 + ((m_lane & 63) >> 3));
#pragma unroll
      for (int mi = 0; mi < MI; mi++) h[STAGED ? 0 : ni][mi] = *reinterpret_cast<const u32x4*>(Hc + piece * 32 + ((m_lane & 63) >> 1) + 8 * mi);
    }
  }
};
// dense: the bf16 activation in dense panel form (64-byte pieces of 32 features), 16 features per (mi, ni).
template <int MI, int NI>
struct LaneSavedDense {
  u32x4 h[MI][NI][2];   // [mi][ni][q]: features 16 mi + 8 q .. + 7 of token ni
  __device__ __forceinline__ void load(const __bf16* H, int F, int m_lane, int n_lane) {
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        int f = m_lane + 16 * mi;
        const __bf16* p = H + a24_piece(n_lane + ni, f >> 5, F >> 5) * 32 + (f & 31);
        h[mi][ni][0] = *reinterpret_cast<const u32x4*>(p);
        h[mi][ni][1] = *reinterpret_cast<const u32x4*>(p + 8);
      }
  }
};

// C[m][n], n contiguous: a lane's neighbouring columns of a row leave in one store, 16 bytes (8 columns) with the 256 x 256 tile, 2 NI bytes with the others.
struct EpiRowMajor {
  struct Args { __bf16* C; int ldc; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
        st_cols<NI>(e.C + (size_t)(m_lane + 16 * mi + v) * e.ldc + n_lane, o);
      }
  }
};

// Transposing store of a wave's part of the tile, out[n][m] with m contiguous, through LDS.  With the 256 x 256
// tile a lane owns 32 consecutive m of 8 columns n, half lines of 8 output rows, and one store instruction of the wave
// would put 64 16-byte pieces into 64 different lines (32 instructions, 2048 line transactions a wave; on the short-K
// weight-gradient GEMMs that alone made the transposing kernels 15 % slower than the row-major ones).  So the packed pieces first
// go to a wave-private image [n][m] in the operand ring, which is free by then (row n, 16-byte piece c at
// piece position c ^ key(n), so that the 16 lanes an LDS instruction serves together hit different positions both ways: lanes of different
// rho, and with LANES = 16 of two neighbouring h, whose pieces differ in the bit that key leaves out),
// and leave as instructions that write whole rows of the image: 256 contiguous bytes each with 128 rows a wave.
template <int MI, int NI>
struct ColMajorStage {
  using LT = LaneTile<MI, NI>;
  static constexpr int PIECES = LT::ROWS / 8;
  static __device__ __forceinline__ int at(int r, int c) { return (r * PIECES + (c ^ ((r / NI) & (LT::LANES == 16 ? 11 : PIECES - 1)))) << 4; }
  // piece `c` (of 8 m, among the lane's own) of its column ni
  static __device__ __forceinline__ void put(char* wbuf, int ni, int c, u32x4 v) { *reinterpret_cast<u32x4*>(wbuf + at(NI * LT::rho() + ni, 2 * MI * LT::h() + c)) = v; }
  // C, ldc: the whole result; m_lane, n_lane: the lane's
  static __device__ __forceinline__ void flush(const char* wbuf, __bf16* C, int ldc, int m_lane, int n_lane) {
    // (256 x 256: uniform up to here; copied to vector registers ahead of the main loop's tail, with k-major operands, it was spilled)
    if constexpr (LT::LANES == 16) asm volatile("" : "+s"(C));
    __bf16* out = C + (size_t)(n_lane - NI * LT::rho()) * ldc + (m_lane - 16 * MI * LT::h());
    const int lane = lane_id(), c = lane & (PIECES - 1), sub = lane / PIECES;
    constexpr int PER = 64 / PIECES;   // rows per store instruction
#pragma unroll
    for (int j = 0; j < LT::COLS / PER; j++) {
      const int r = PER * j + sub;
      *reinterpret_cast<u32x4*>(out + (size_t)r * ldc + 8 * c) = *reinterpret_cast<const u32x4*>(wbuf + at(r, c));
    }
  }
};

// C stored transposed, out[n][m] with m contiguous (staged through LDS, see ColMajorStage).
struct EpiColMajor {
  static constexpr bool STAGED = true;
  struct Args { __bf16* C; int ldc; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
#pragma unroll
    for (int ni = 0; ni < NI; ni++)
#pragma unroll
      for (int mi = 0; mi < MI; mi++)
#pragma unroll
        for (int q = 0; q < 2; q++) {
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; d++) o[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d], acc[mi][ni][8 * q + 2 * d + 1]);
          ColMajorStage<MI, NI>::put(wbuf, ni, 2 * mi + q, o);
        }
    ColMajorStage<MI, NI>::flush(wbuf, e.C, e.ldc, m_lane, n_lane);
  }
};

// Dense FFN up-projection epilogue (Sec. 1, Squared ReLU): rows m are features, columns n are tokens;
// H[t][f] = bf16( max(0, acc + b1[f])^2 ), stored as the [T][F] operand of the down-projection; if Ht is given the
// same values are also stored as the [F][T] operand of the weight-gradient GEMM that reduces over tokens.  Both in
// the dense panel form of gemm_core.hpp (64-byte pieces of 32 k), like every A operand the library makes for itself.
// STATS: also counts the non-zero stored activations of the launch into tele (may be NULL), the sparsity level the
// dense path reports while 2:4 is still switched off (Sec. 2, last paragraph: the dense warm-up).
template <bool STATS>
struct EpiRelu2T {
  static constexpr bool STAGED = true;
  struct Args { __bf16* H; __bf16* Ht; const float* b1; int F; int T; unsigned long long* tele; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    uint32_t nonzero = 0u;   // of this lane's 256 activations
    LaneVec<MI> lb;
    lb.load(e.b1, m_lane, 0.f);
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float r = fmaxf(acc[mi][ni][v] + lb.at(16 * mi + v), 0.f);
          acc[mi][ni][v] = r * r;
        }
        int f = m_lane + 16 * mi;
        __bf16* row = e.H + a24_piece(n_lane + ni, f >> 5, e.F >> 5) * 32 + (f & 31);
#pragma unroll
        for (int q = 0; q < 2; q++) {
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; d++) {
            o[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d], acc[mi][ni][8 * q + 2 * d + 1]);
            if constexpr (STATS) nonzero += min(o[d] & 0xFFFFu, 1u) + min(o[d] >> 16, 1u);
          }
          if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(PanelStage<MI, NI, 2>::at(wbuf, ni, 2 * mi + q)) = o;
          else *reinterpret_cast<u32x4*>(row + 8 * q) = o;
        }
      }
      if (e.Ht) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float o[NI];
#pragma unroll
          for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
          st_cols<NI>(e.Ht + a24_piece(m_lane + 16 * mi + v, n_lane >> 5, e.T >> 5) * 32 + (n_lane & 31), o);
        }
      }
    }
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI, 2>::flush(wbuf, reinterpret_cast<char*>(e.H) + PanelStage<MI, NI, 2>::first(m_lane, n_lane, e.F));
    if constexpr (STATS) {
      if (e.tele) tele_add2(e.tele, nonzero, TELE_NONZERO, -1, blockIdx.x + (m_lane >> 6) + (n_lane >> 6));
    }
  }
};
using EpiRelu2 = EpiRelu2T<false>;

// Two 2:4 groups at a time, one in each half of a word (pick24_two).  With two or more columns a lane pairs the same group of two
// neighbouring tokens; with one (NI = 1) it pairs groups a and a + 2 of the token.  Entry v of a word's low half is feature 16 mi + v of
// token ni, of its high half the same feature of token ni + 1, or (NI = 1) feature 16 mi + v + 8 of the one token.
// TwoTokens: what 16 features (an M-tile's) make of two tokens (NI = 1: of one, and index 1 is not used).
template <int NI>
struct TwoTokens {
  static constexpr int TOK = NI > 1 ? 2 : 1, ROWS = NI > 1 ? 16 : 8;   // tokens a word holds; words of an M-tile
  using Words = uint32_t[ROWS];
  u32x4 vals[TOK];                   // kept pairs in position order
  uint32_t nib[TOK];                 // their metadata, 16 bits
  __device__ __forceinline__ void pick(const Words& h) {
    uint32_t w = 0u;
#pragma unroll
    for (int a = 0; a < ROWS / 4; a++) {
      const Pick24x2 p = pick24_two(h[4 * a], h[4 * a + 1], h[4 * a + 2], h[4 * a + 3]);
      w = put_nibbles(w, p, a);
      const uint32_t lo = __builtin_amdgcn_perm(p.second, p.first, 0x05040100u), hi = __builtin_amdgcn_perm(p.second, p.first, 0x07060302u);
      vals[0][a] = lo;
      if constexpr (NI > 1) vals[1][a] = hi; else vals[0][a + 2] = hi;
    }
    if constexpr (NI > 1) { nib[0] = w & 0xFFFFu; nib[1] = w >> 16; }
    else nib[0] = (w & 0xFFu) | ((w >> 8) & 0xFF00u);
  }
};
// A lane's rounded activations of two tokens (or one) for M-tile mi, in the order TwoTokens takes them; z(mi, ni, v) = the pre-activation
template <int NI, class Z>
__device__ __forceinline__ void relu2_words(typename TwoTokens<NI>::Words& h, int mi, int ni, Z&& z) {
#pragma unroll
  for (int v = 0; v < TwoTokens<NI>::ROWS; v++) {
    const float r0 = fmaxf(z(mi, ni, v), 0.f), r1 = fmaxf(NI > 1 ? z(mi, ni + 1, v) : z(mi, ni, v + 8), 0.f);
    h[v] = pack_bf16x2(r0 * r0, r1 * r1);
  }
}
// The same words as rows of 16 features, row-major (parity checks)
template <int NI>
__device__ __forceinline__ void st_debug(__bf16* row, int F, const typename TwoTokens<NI>::Words& h) {
#pragma unroll
  for (int half = 0; half < 2; half++) {
    const uint32_t sel = half ? 0x07060302u : 0x05040100u;
#pragma unroll
    for (int q = 0; q < TwoTokens<NI>::ROWS / 8; q++) {
      u32x4 o;
#pragma unroll
      for (int d = 0; d < 4; d++) o[d] = __builtin_amdgcn_perm(h[8 * q + 2 * d + 1], h[8 * q + 2 * d], sel);
      *reinterpret_cast<u32x4*>(row + (NI > 1 ? (size_t)half * F + 8 * q : 8 * half)) = o;
    }
  }
}

// Per-feature non-zero counts of the activation epilogues (Sec. 2, "Optimization 1": the column-level sparsity the first GEMM's
// epilogue can compute for free).  A lane first counts in 8-bit fields as the words come, one word for 2 v and 2 v + 1 of an
// M-tile: bytes 0, 1 from the low halves, bytes 2, 3 from the high halves; fold brings that into 4 features a register, feature f of
// the lane in field f % 4 of register f / 4.
template <int MI, int NI, bool HERE = false> struct NnzCount {
  static constexpr int ROWS = TwoTokens<NI>::ROWS;
  uint32_t c[MI * ROWS / 2];
  __device__ __forceinline__ NnzCount() {
#pragma unroll
    for (int i = 0; i < MI * ROWS / 2; i++) c[i] = 0u;
  }
  __device__ __forceinline__ void add(int mi, const uint32_t (&h)[ROWS]) {
#pragma unroll
    for (int v = 0; v < ROWS; v += 2) {
      c[(mi * ROWS + v) / 2] += pk_min16(h[v], 0x00010001u) + (pk_min16(h[v + 1], 0x00010001u) << 8);
      keep_here<HERE>(c[(mi * ROWS + v) / 2]);
    }
  }
  __device__ __forceinline__ void fold(uint32_t (&cnt)[4 * MI]) const {
#pragma unroll
    for (int i = 0; i < 4 * MI; i++) {
      if constexpr (NI > 1) {                            // both halves are tokens of the same two features
        const uint32_t a = c[2 * i] + (c[2 * i] >> 16), b = c[2 * i + 1] + (c[2 * i + 1] >> 16);
        cnt[i] = __builtin_amdgcn_perm(b, a, 0x05040100u);
      } else {                                           // the high halves are features 8 further on
        const int mi = i / 4, j = i % 4, w = mi * 4 + 2 * (j & 1);
        cnt[i] = __builtin_amdgcn_perm(c[w + 1], c[w], j < 2 ? 0x05040100u : 0x07060302u);
      }
    }
  }
};
// The lanes that hold the same 16 MI features add their fields up with a butterfly (<= 128 per field); each then adds the
// totals of every LANES-th feature to nnz [F] with atomics (the caller zeroes it).
template <int MI, int NI>
__device__ __forceinline__ void nnz_flush(uint32_t (&cnt)[4 * MI], uint32_t* nnz, int m_lane) {
  constexpr int LANES = LaneTile<MI, NI>::LANES, REGS = LANES / 4;
#pragma unroll
  for (int i = 0; i < 4 * MI; i++)
#pragma unroll
    for (int sft = 1; sft < LANES; sft <<= 1) cnt[i] += (uint32_t)__shfl_xor((int)cnt[i], sft, 64);
  int r = LaneTile<MI, NI>::rho();
#pragma unroll
  for (int b = 0; b < 4 * MI; b += REGS) {   // registers b .. b + REGS - 1: features 4 b .. 4 b + LANES - 1
    uint32_t w = 0u;
#pragma unroll
    for (int i = 0; i < REGS; i++)
      if (b + i < 4 * MI) w = (r >> 2) == i ? cnt[b + i] : w;
    uint32_t c = (w >> (8 * (r & 3))) & 0xFFu;
    if (c) atomicAdd(nnz + m_lane + 4 * b + r, c);
  }
}

// Fused up-projection epilogue of the 2:4 FFN (Sec. 2: activation, then sparsification, in one pass):
// h = bf16(max(0, acc + b1)^2); of every 4 consecutive features of a token keep the 2 largest
// (ties -> lower index); write the kept pair and its metadata nibble.  The 4 members of a group are the
// accumulator registers 4a..4a+3 of one MFMA tile, so the pick needs no cross-lane traffic.
//   Hc, meta: the compressed activation [T][F/2] + [T][F/8] in panel form (gemm_core.hpp): a lane's 64 features of
//   one token are exactly one piece, 64 bytes of kept values (position order) + 8 metadata bytes (nibble
//   i0 | i1<<2, even group low).
//   Hdbg [T][F]    optional, row-major: the rounded activation before pruning (parity checks)
//   nnz  [F] optional: per-feature count of non-zero activations before pruning (Sec. 2, "Optimization 1": the
//   column-level sparsity the first GEMM's epilogue can compute for free), accumulated with atomics; the caller
//   zeroes it.  A lane counts its 4 tokens in 8-bit fields (4 features per register), the 32 lanes that hold the
//   same 64 features add their fields up with a butterfly, and each lane then adds two features' totals.
//   tele optional (STATS only): the launch's totals of non-zero activations before pruning and of non-zero kept values
//   (Sec. 2, first paragraph: the share of non-zeros that 2:4 drops), one pair of atomics per wave.
template <bool STATS>
struct EpiPrune24T {
  static constexpr bool STAGED = true;
  struct Args { __bf16* Hc; uint8_t* meta; __bf16* Hdbg; const float* b1; int F; uint32_t* nnz; unsigned long long* tele; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    constexpr int TOK = TwoTokens<NI>::TOK;
    NnzCount<MI, NI> nz;
    uint32_t kept = 0u;   // non-zero values among the lane's stored ones, first and second of a pair apart (16-bit fields)
    LaneVec<MI> lb;
    lb.load(e.b1, m_lane, 0.f);
#pragma unroll
    for (int ni = 0; ni < NI; ni += TOK) {
      uint32_t nib[TOK][2] = {};
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        TwoTokens<NI> tt;
        typename TwoTokens<NI>::Words h;
        relu2_words<NI>(h, mi, ni, [&](int i, int n, int v) { return acc[i][n][v] + lb.at(16 * i + v); });
        if constexpr (STATS) nz.add(mi, h);
        if (e.Hdbg) st_debug<NI>(e.Hdbg + (size_t)(n_lane + ni) * e.F + m_lane + 16 * mi, e.F, h);
        tt.pick(h);
#pragma unroll
        for (int t = 0; t < TOK; t++) {
          if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(PanelStage<MI, NI>::at(wbuf, ni + t, mi)) = tt.vals[t];
          else *reinterpret_cast<u32x4*>(e.Hc + a24_piece(n_lane + ni + t, m_lane >> 6, e.F >> 6) * 32 + ((m_lane & 63) >> 1) + 8 * mi) = tt.vals[t];
          nib[t][mi >> 1] |= tt.nib[t] << (16 * (mi & 1));
          if constexpr (STATS) {
#pragma unroll
            for (int i = 0; i < 4; i++) kept += pk_min16(tt.vals[t][i], 0x00010001u);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < TOK; t++) st_nibbles<MI>(e.meta + a24_piece(n_lane + ni + t, m_lane >> 6, e.F >> 6) * 8 + ((m_lane & 63) >> 3), nib[t]);
    }
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI>::flush(wbuf, reinterpret_cast<char*>(e.Hc) + PanelStage<MI, NI>::first(m_lane, n_lane, e.F));
    if constexpr (STATS) {
      uint32_t cnt[4 * MI];
      nz.fold(cnt);
      if (e.tele) {
        // the lane's own non-zero count is the sum of its fields (at most 4 each); with the kept count, over the wave
        uint32_t tot = 0u;
#pragma unroll
        for (int i = 0; i < 4 * MI; i++) tot += (cnt[i] & 0xFFu) + ((cnt[i] >> 8) & 0xFFu) + ((cnt[i] >> 16) & 0xFFu) + (cnt[i] >> 24);
        tele_add2(e.tele, tot | (((kept & 0xFFFFu) + (kept >> 16)) << 16), TELE_NONZERO, TELE_KEPT_TOK, blockIdx.x + (m_lane >> 6) + (n_lane >> 6));
      }
      if (e.nnz) nnz_flush<MI, NI>(cnt, e.nnz, m_lane);
    }
  }
};
using EpiPrune24 = EpiPrune24T<false>;   // without the statistic (a compile-time switch: the plain kernel carries no trace of it)

// C[map[m]][n], n contiguous: the rows of the result are scattered through a row map (the split weight-gradient
// GEMMs work on a permutation of the hidden features and write each row back to its feature).
struct EpiRowMajorMapped {
  struct Args { __bf16* C; int ldc; const int* rowmap; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    LaneIdx<MI> rows;
    rows.load(e.rowmap, m_lane);
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
        st_cols<NI>(e.C + (size_t)rows.at(16 * mi + v) * e.ldc + n_lane, o);
      }
  }
};

// Dense backward, pointwise part: rows m are features, columns n are tokens; acc = dH[t][f];
// dZ[t][f] = bf16( acc * 2 sqrt(H[t][f]) )  (derivative of max(0,z)^2 is 2 max(0,z) = 2 sqrt(h)).
// Stored as a [T][F] operand and, for the weight-gradient GEMM that reduces over tokens, also as an [F][T] operand;
// H, dZ and dZt are all in dense panel form.
struct EpiDRelu {
  static constexpr bool STAGED = true;
  struct Args { const __bf16* H; __bf16* dZ; __bf16* dZt; int F; int T; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    constexpr bool STAGED = LaneTile<MI, NI>::STAGED;   // through LDS, like the result
    LaneSavedDense<STAGED ? 1 : MI, STAGED ? 1 : NI> sv;
    const size_t run = STAGED ? PanelStage<MI, NI, 2>::first(m_lane, n_lane, e.F) : 0;
    if constexpr (LaneTile<MI, NI>::STAGED) {
      PanelStage<MI, NI, 2>::fetch(wbuf, reinterpret_cast<const char*>(e.H) + run);
      wait_vmcnt<0>();
      asm volatile("" ::: "memory");                 // (the compiler does not see the DMA write what is read below)
    } else sv.load(e.H, e.F, m_lane, n_lane);
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        int f = m_lane + 16 * mi;
        size_t o = a24_piece(n_lane + ni, f >> 5, e.F >> 5) * 32 + (f & 31);
#pragma unroll
        for (int q = 0; q < 2; q++) {
          char* place = nullptr;
          u32x4 h;
          if constexpr (LaneTile<MI, NI>::STAGED) {
            place = PanelStage<MI, NI, 2>::at(wbuf, ni, 2 * mi + q);
            h = *reinterpret_cast<const u32x4*>(place);
          } else h = sv.h[mi][ni][q];
          u32x4 r;
#pragma unroll
          for (int d = 0; d < 4; d++) {
            float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[d]));
            float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[d]));
            acc[mi][ni][8 * q + 2 * d] *= g0;
            acc[mi][ni][8 * q + 2 * d + 1] *= g1;
            r[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d], acc[mi][ni][8 * q + 2 * d + 1]);
          }
          if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(place) = r;
          else *reinterpret_cast<u32x4*>(e.dZ + o + 8 * q) = r;
        }
      }
      if (e.dZt) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float o[NI];
#pragma unroll
          for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
          st_cols<NI>(e.dZt + a24_piece(m_lane + 16 * mi + v, n_lane >> 5, e.T >> 5) * 32 + (n_lane & 31), o);
        }
      }
    }
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI, 2>::flush(wbuf, reinterpret_cast<char*>(e.dZ) + run);
  }
};

// 2:4 backward, pointwise part (Fig. 4 caption; Sec. 2, last paragraph): acc = dH[t][f]; on the positions
// the forward kept, dZ = dH * 2 sqrt(h); elsewhere dZ = 0 and nothing is stored.  Output is compressed with
// the forward's metadata: dZc [T][F/2].  Hc, meta and dZc are in panel form: one piece per lane and token.
struct EpiDGather {
  static constexpr bool STAGED = true;
  struct Args { const __bf16* Hc; const uint8_t* meta; __bf16* dZc; int F; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    LaneSaved24<MI, NI> sv;
    sv.load(e.Hc, e.meta, e.F, m_lane, n_lane, wbuf);
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      size_t t = (size_t)(n_lane + ni);
      size_t piece = a24_piece((int)t, m_lane >> 6, e.F >> 6);
      const u32x2 mt = sv.mt[ni];
      __bf16* zrow = e.dZc + piece * 32 + ((m_lane & 63) >> 1);
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        const u32x4 h = sv.kept(ni, mi);
        u32x4 z;
#pragma unroll
        for (int a = 0; a < 4; a++) {
          int gi = 4 * mi + a;
          uint32_t n4 = (mt[gi >> 3] >> (4 * (gi & 7))) & 15u;
          uint32_t i0 = n4 & 3u, i1 = n4 >> 2;
          float x0 = acc[mi][ni][4 * a], x1 = acc[mi][ni][4 * a + 1], x2 = acc[mi][ni][4 * a + 2], x3 = acc[mi][ni][4 * a + 3];
          float s0 = i0 == 0 ? x0 : (i0 == 1 ? x1 : x2);
          float s1 = i1 == 3 ? x3 : (i1 == 2 ? x2 : x1);
          float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[a]));
          float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[a]));
          z[a] = pack_bf16x2(s0 * g0, s1 * g1);
        }
        if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(PanelStage<MI, NI>::at(wbuf, ni, mi)) = z;
        else *reinterpret_cast<u32x4*>(zrow + 8 * mi) = z;
      }
    }
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI>::flush(wbuf, reinterpret_cast<char*>(e.dZc) + PanelStage<MI, NI>::first(m_lane, n_lane, e.F));
  }
};

// ------------------------------------------------------------------------------------------------
// fp8 (e4m3) forward: per-tensor scales; order of Sec. 2: activation, sparsification, then FP8 quantisation
// ------------------------------------------------------------------------------------------------

// Saturating round-to-nearest-even conversion of two floats to e4m3 (the conversion instruction alone turns values
// beyond the format's largest finite number, 448, into NaN codes).
__device__ __forceinline__ uint32_t cvt_e4m3x2(float lo, float hi, uint32_t old, bool high_half) {
  lo = __builtin_fminf(__builtin_fmaxf(lo, -448.f), 448.f);
  hi = __builtin_fminf(__builtin_fmaxf(hi, -448.f), 448.f);
  return high_half ? (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(lo, hi, (int)old, true)
                   : (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(lo, hi, (int)old, false);
}

// Correctly rounded division by a scale that divides many values: with r the correctly rounded reciprocal of s and q = RN(a r), the
// remainder a - q s is exact in one fused multiply-add and RN(q + remainder * r) is RN(a / s) (Markstein's theorem).  Six operations a
// value instead of the ten of the division sequence, and the same e4m3 codes as with an IEEE division for every pair of operands:
//   - q is clamped to +-2^20 first, beyond the largest code by far, so that a quotient that overflows (or an infinity) keeps its sign
//     instead of turning into a NaN; copysign keeps the sign of a zero;
//   - the theorem wants no underflow on the way: both operands are multiplied by a power of two p that keeps s within 2^+-60, so a
//     remainder can underflow only where |a / s| is below 2^-20, which every rounding to e4m3 takes to zero;
//   - an infinite scale becomes p = 0, s = 1: finite values give their zero, infinite ones NaN.
struct ExactDiv {
  float p, s, r;
  __device__ __forceinline__ ExactDiv() {}
  __device__ __forceinline__ explicit ExactDiv(float scale) {
    const bool inf = scale > 0x1.fffffep127f;
    p = inf ? 0.f : scale > 0x1p60f ? 0x1p-100f : scale < 0x1p-60f ? 0x1p100f : 1.f;
    s = inf ? 1.f : scale * p;
    r = 1.f / s;
  }
  __device__ __forceinline__ float operator()(float a) const {
    const float ap = a * p, q = __builtin_amdgcn_fmed3f(ap * r, -0x1p20f, 0x1p20f);
    return __builtin_copysignf(__builtin_fmaf(__builtin_fmaf(-q, s, ap), r, q), a);
  }
};

// fp8 up-projection: z = zscale * acc + b1 (zscale = sx * sw1); h = bf16(max(0, z)^2); the keep-2-of-4 pick is made on
// the bf16 words exactly as in EpiPrune24; the kept values are then quantised, e4m3(h / sh).
//   Hc8, meta: panel form of the fp8 operand: piece = 64 stored bytes + 16 metadata bytes for 128 features of a token;
//   a lane's 64 features are one half of a piece.
//   Hc16, meta16 (optional, a training context): the kept values before quantisation, bf16, with their metadata, in the
//   bf16 panel form -- what the backward takes the activation's derivative from (the e4m3 code of h keeps 4
//   significant bits, too few for 2 sqrt(h)).
struct EpiPrune24F8 {
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { uint8_t* Hc8; uint8_t* meta; __bf16* Hdbg; const float* b1; int F; float zscale; float sh; __bf16* Hc16; uint8_t* meta16; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    constexpr int TOK = TwoTokens<NI>::TOK;
    LaneVec<MI> lb;
    lb.load(e.b1, m_lane, 0.f);
    const ExactDiv by_sh(e.sh);
#pragma unroll
    for (int ni = 0; ni < NI; ni += TOK) {
      uint32_t nib[TOK][2] = {}, q8[TOK][2 * MI];
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        TwoTokens<NI> tt;
        typename TwoTokens<NI>::Words h;
        relu2_words<NI>(h, mi, ni, [&](int i, int n, int v) { return acc[i][n][v] * e.zscale + lb.at(16 * i + v); });
        if (e.Hdbg) st_debug<NI>(e.Hdbg + (size_t)(n_lane + ni) * e.F + m_lane + 16 * mi, e.F, h);
        tt.pick(h);
#pragma unroll
        for (int t = 0; t < TOK; t++) {
          nib[t][mi >> 1] |= tt.nib[t] << (16 * (mi & 1));
#pragma unroll
          for (int a = 0; a < 4; a++) {
            // group 4 mi + a's two stored bytes are bytes 8 mi + 2 a and + 1 of the lane's 8 MI
            const float v0 = by_sh(bf16_lo_to_f32(tt.vals[t][a])), v1 = by_sh(bf16_hi_to_f32(tt.vals[t][a]));
            uint32_t& q = q8[t][2 * mi + (a >> 1)];
            q = cvt_e4m3x2(v0, v1, (a & 1) ? q : 0u, (a & 1) != 0);
          }
          if (e.Hc16) *reinterpret_cast<u32x4*>(e.Hc16 + a24_piece(n_lane + ni + t, m_lane >> 6, e.F >> 6) * 32 + ((m_lane & 63) >> 1) + 8 * mi) = tt.vals[t];
        }
      }
#pragma unroll
      for (int t = 0; t < TOK; t++) {
        const size_t piece = a24_piece(n_lane + ni + t, m_lane >> 7, e.F >> 7);
        st_codes<MI>(e.Hc8 + piece * 64 + ((m_lane & 127) >> 1), q8[t]);
        st_nibbles<MI>(e.meta + piece * 16 + ((m_lane & 127) >> 3), nib[t]);
        if (e.Hc16) st_nibbles<MI>(e.meta16 + a24_piece(n_lane + ni + t, m_lane >> 6, e.F >> 6) * 8 + ((m_lane & 63) >> 3), nib[t]);
      }
    }
  }
};

// fp8 backward, pointwise part (the abstract's FP8 backward pass; Sec. 2's fused backward pointwise step with its FP8
// scaling): acc = (W2_8 . dY8) for a lane's 64 features x 4 tokens; dH = scale * acc (scale = sdy * sw2); on the
// positions the forward kept dZ = dH * 2 sqrt(h) with h the bf16 kept value the forward saved (Hc16, meta16: bf16 panel
// form); the result is quantised, e4m3(dZ / sdz) (saturating), and stored compressed with the forward's metadata in
// the fp8 panel form (the operand of the sparse dX GEMM).
struct EpiDGatherF8 {
  static constexpr bool STAGED = true;
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { const __bf16* Hc16; const uint8_t* meta16; uint8_t* dZc8; int F; float scale; float sdz; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    LaneSaved24<MI, NI> sv;
    sv.load(e.Hc16, e.meta16, e.F, m_lane, n_lane, wbuf);
    const ExactDiv by_sdz(e.sdz);
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      size_t t = (size_t)(n_lane + ni);
      const u32x2 mt = sv.mt[ni];
      uint32_t q8[2 * MI];
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        const u32x4 h = sv.kept(ni, mi);
#pragma unroll
        for (int a = 0; a < 4; a++) {
          int gi = 4 * mi + a;
          uint32_t n4 = (mt[gi >> 3] >> (4 * (gi & 7))) & 15u;
          uint32_t i0 = n4 & 3u, i1 = n4 >> 2;
          float x0 = acc[mi][ni][4 * a], x1 = acc[mi][ni][4 * a + 1], x2 = acc[mi][ni][4 * a + 2], x3 = acc[mi][ni][4 * a + 3];
          float s0 = i0 == 0 ? x0 : (i0 == 1 ? x1 : x2);
          float s1 = i1 == 3 ? x3 : (i1 == 2 ? x2 : x1);
          float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[a]));
          float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[a]));
          float v0 = by_sdz(s0 * e.scale * g0), v1 = by_sdz(s1 * e.scale * g1);
          q8[gi >> 1] = cvt_e4m3x2(v0, v1, (gi & 1) ? q8[gi >> 1] : 0u, (gi & 1) != 0);
        }
      }
      size_t piece = a24_piece((int)t, m_lane >> 7, e.F >> 7);
      st_codes<MI>(e.dZc8 + piece * 64 + ((m_lane & 127) >> 1), q8);
    }
  }
};

// out[n][m] = bf16(scale * acc), m contiguous: the transposing store of EpiColMajor with a scale (fp8 dW1).
struct EpiColMajorScaled {
  static constexpr bool STAGED = true;
  struct Args { __bf16* C; int ldc; float scale; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
#pragma unroll
    for (int ni = 0; ni < NI; ni++)
#pragma unroll
      for (int mi = 0; mi < MI; mi++)
#pragma unroll
        for (int q = 0; q < 2; q++) {
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; d++) o[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d] * e.scale, acc[mi][ni][8 * q + 2 * d + 1] * e.scale);
          ColMajorStage<MI, NI>::put(wbuf, ni, 2 * mi + q, o);
        }
    ColMajorStage<MI, NI>::flush(wbuf, e.C, e.ldc, m_lane, n_lane);
  }
};

// Row maxima of a launch: rowmax[t] is raised to the largest bf16 magnitude word of row t.  A token row spans F / (16 MI) lanes of the
// launch, and one atomic for each of them was the larger part of the row-wise epilogues (T = F = 8192: a million atomics, 15 us of the
// dH GEMM's 157 with 256 x 256 tiles and 40 of 167 with 256 x 128).  So the lane groups, which hold the same tokens, are
// combined first, and what is already there is looked at before: the values are requested before they are needed,
// and an atomic goes out only where it would raise one.  That spares the later rounds of a launch and most of a tile that starts late;
// tiles of one round that finish together all see the cleared value and all send theirs.  A value that is out of date is lower and
// only costs an atomic.
// What bounds those that do go out is how many lines each touches and how many tiles raise the same ones.  The 256 x 256 tile's four lane
// groups therefore exchange halves of what they hold instead of each adding up all of it, and every lane raises two neighbouring tokens:
// a wave's 128 tokens are two instructions of 64 lanes over four lines each.  Eight instructions of the 16 lanes of one group, four lines
// each again, took longer the fewer the tokens and the more the tiles (row-wise fp8, up-projection and dH, us: T 512 D 4096 F 32768 106 -> 76
// and 93 -> 73; T 512 D 8192 F 32768 157 -> 129 and 128 -> 114; T 4096 D 4096 F 16384 218 -> 208 and 215 -> 211; T = F = 8192, D 2048
// 117 -> 116 and 121 -> 119).
template <int MI, int NI>
struct RowMax {
  using LT = LaneTile<MI, NI>;
  static constexpr bool SCATTER = LT::GROUPS == 4;
  static constexpr int OWN = SCATTER ? NI / 4 : NI;   // tokens a lane raises
  uint32_t seen[OWN];
  static __device__ __forceinline__ int first(int n_lane) { return SCATTER ? n_lane + OWN * LT::h() : n_lane; }
  __device__ __forceinline__ void load(const uint32_t* rowmax, int n_lane) {
#pragma unroll
    for (int i = 0; i < OWN; i++) seen[i] = __hip_atomic_load(rowmax + first(n_lane) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // mx: the lane's maxima of its tokens, two to a word (NI = 1: both halves are of its one token)
  __device__ __forceinline__ void raise(uint32_t* rowmax, int n_lane, const uint32_t (&mx)[(NI + 1) / 2]) const {
    if constexpr (SCATTER) {
      const bool up = (LT::h() & 2) != 0, odd = (LT::h() & 1) != 0;
      uint32_t k[2];
#pragma unroll
      for (int i = 0; i < 2; i++) k[i] = pk_max16(up ? mx[2 + i] : mx[i], (uint32_t)__shfl_xor((int)(up ? mx[i] : mx[2 + i]), 32, 64));
      const uint32_t m = pk_max16(odd ? k[1] : k[0], (uint32_t)__shfl_xor((int)(odd ? k[0] : k[1]), 16, 64));
      int at = first(n_lane);
      asm volatile("" : "+v"(at));                   // (counted anew: the address kept since the load is two registers more)
      if ((m & 0xFFFFu) > seen[0]) atomicMax(rowmax + at, m & 0xFFFFu);
      if ((m >> 16) > seen[1]) atomicMax(rowmax + at + 1, m >> 16);
    } else {
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        uint32_t m = NI == 1 ? max(mx[0] & 0xFFFFu, mx[0] >> 16) : ni & 1 ? mx[0] >> 16 : mx[0] & 0xFFFFu;
        m = max(m, (uint32_t)__shfl_xor((int)m, 32, 64));
        if (LT::h() == 0 && m > seen[ni]) atomicMax(rowmax + n_lane + ni, m);
      }
    }
  }
};

// fp8 up-projection with ROW-WISE scaling (the paper's precision recipe, Sec. 2: "FP8 rowwise scaling"): the
// activation operand carries one scale per token, the weight one per output channel:
//   z = sx[t] sw1[f] acc + b1[f];  h = bf16(max(0, z)^2);  keep-2-of-4 as in EpiPrune24.
// The kept values cannot be quantised here -- their scale is the maximum of the whole token row, which spans many
// block tiles -- so they are written as bf16 in the bf16 panel form (Hc, meta), and rowmax[t] (bf16
// word of the largest activation, non-negative, so integer order = value order) is raised with atomics (RowMax).
// A streaming kernel then quantises with sh[t] = rowmax[t] / 448 (k_stream.hip).
// STATS: also the per-feature non-zero counts of the activation before pruning, into nnz [F] (as in EpiPrune24T).
template <bool STATS>
struct EpiPrune24RwT {
  static constexpr EpiCost COST = EPI_FP8;
  static constexpr bool STAGED = true;
  struct Args { __bf16* Hc; uint8_t* meta; __bf16* Hdbg; const float* b1; int F; const float* sx; const float* sw1; uint32_t* rowmax; uint32_t* nnz; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    constexpr int TOK = TwoTokens<NI>::TOK;
    constexpr bool HERE = NI == 8;
    NnzCount<MI, NI, HERE> nz;
    RowMax<MI, NI> rm;
    rm.load(e.rowmax, n_lane);
    float sxt[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) sxt[ni] = e.sx[n_lane + ni];
    // M-tile by M-tile, each with its 16 features' biases and scales (asked for one M-tile ahead): all 64 of both beside the accumulators
    // spilled 17-26 registers with 256 x 128 tiles
    LaneVec<1> lb[2], lw[2];
    lb[0].load(e.b1, m_lane, 0.f);
    lw[0].load(e.sw1, m_lane, 1.f);
    uint32_t mx[(NI + 1) / 2] = {}, nib[NI][2] = {};     // mx: of each half
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
      if (mi + 1 < MI) {
        lb[(mi + 1) & 1].load(e.b1, m_lane + 16 * (mi + 1), 0.f);
        lw[(mi + 1) & 1].load(e.sw1, m_lane + 16 * (mi + 1), 1.f);
      }
#pragma unroll
      for (int ni = 0; ni < NI; ni += TOK) {
        TwoTokens<NI> tt;
        typename TwoTokens<NI>::Words h;
        relu2_words<NI>(h, mi, ni, [&](int i, int n, int v) { return acc[i][n][v] * (sxt[n] * lw[i & 1].at(v)) + lb[i & 1].at(v); });
#pragma unroll
        for (int v = 0; v < TwoTokens<NI>::ROWS; v++) mx[ni / 2] = pk_max16(mx[ni / 2], h[v]);
        if constexpr (STATS) nz.add(mi, h);
        if (e.Hdbg) st_debug<NI>(e.Hdbg + (size_t)(n_lane + ni) * e.F + m_lane + 16 * mi, e.F, h);
        tt.pick(h);
#pragma unroll
        for (int t = 0; t < TOK; t++) {
          if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(PanelStage<MI, NI>::at(wbuf, ni + t, mi)) = tt.vals[t];
          else *reinterpret_cast<u32x4*>(e.Hc + a24_piece(n_lane + ni + t, m_lane >> 6, e.F >> 6) * 32 + ((m_lane & 63) >> 1) + 8 * mi) = tt.vals[t];
          nib[ni + t][mi >> 1] |= tt.nib[t] << (16 * (mi & 1));
          keep_here<HERE>(nib[ni + t][mi >> 1]);
        }
        keep_here<HERE>(mx[ni / 2]);
      }
      FFN24_FENCE();
    }
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI>::flush(wbuf, reinterpret_cast<char*>(e.Hc) + PanelStage<MI, NI>::first(m_lane, n_lane, e.F));
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      st_nibbles<MI>(e.meta + a24_piece(n_lane + ni, m_lane >> 6, e.F >> 6) * 8 + ((m_lane & 63) >> 3), nib[ni]);
    }
    rm.raise(e.rowmax, n_lane, mx);
    if constexpr (STATS) {
      uint32_t cnt[4 * MI];
      nz.fold(cnt);
      nnz_flush<MI, NI>(cnt, e.nnz, m_lane);
    }
  }
};
using EpiPrune24Rw = EpiPrune24RwT<false>;

// Dense fp8 up-projection with ROW-WISE scaling (the baseline the paper's forward benchmark compares with: all FP8 GEMMs of
// both sides use row-wise scales): z = sx[t] sw1[f] acc + b1[f];  h = bf16(max(0, z)^2), every one of them stored, as the
// bf16 [T][F] operand in dense panel form (64-byte pieces of 32 k); rowmax[t] is raised to the row's largest word.  A
// streaming kernel then quantises each row with sh[t] = rowmax[t] / 448.
// Ht16 (optional, a training context): the same values once more as the bf16 [F][T] operand (dense panel form, K = T) that the
// backward quantises per hidden feature for its dW2 GEMM.
struct EpiRelu2Rw {
  static constexpr EpiCost COST = EPI_FP8_SPILLS;
  struct Args { __bf16* H16; const float* b1; int F; const float* sx; const float* sw1; uint32_t* rowmax; __bf16* Ht16; int T; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    RowMax<MI, NI> rm;
    rm.load(e.rowmax, n_lane);
    LaneVec<MI> lb, lw;
    lb.load(e.b1, m_lane, 0.f);
    lw.load(e.sw1, m_lane, 1.f);
    uint32_t mx[NI] = {};
    float sxt[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) sxt[ni] = e.sx[n_lane + ni];
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        const int t = n_lane + ni;
        int f = m_lane + 16 * mi;
        __bf16* row = e.H16 + a24_piece(t, f >> 5, e.F >> 5) * 32 + (f & 31);
#pragma unroll
        for (int q = 0; q < 2; q++) {
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; d++) {
            int i = 16 * mi + 8 * q + 2 * d;
            float r0 = fmaxf(acc[mi][ni][8 * q + 2 * d] * (sxt[ni] * lw.at(i)) + lb.at(i), 0.f);
            float r1 = fmaxf(acc[mi][ni][8 * q + 2 * d + 1] * (sxt[ni] * lw.at(i + 1)) + lb.at(i + 1), 0.f);
            acc[mi][ni][8 * q + 2 * d] = r0 * r0;
            acc[mi][ni][8 * q + 2 * d + 1] = r1 * r1;
            o[d] = pack_bf16x2(r0 * r0, r1 * r1);
            mx[ni] = max(mx[ni], max(o[d] & 0xFFFFu, o[d] >> 16));
          }
          *reinterpret_cast<u32x4*>(row + 8 * q) = o;
        }
      }
      if (e.Ht16) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float o[NI];
#pragma unroll
          for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
          st_cols<NI>(e.Ht16 + a24_piece(m_lane + 16 * mi + v, n_lane >> 5, e.T >> 5) * 32 + (n_lane & 31), o);
        }
      }
    }
    uint32_t two[(NI + 1) / 2] = {};
#pragma unroll
    for (int ni = 0; ni < NI; ni++) two[ni / 2] |= mx[ni] << (16 * (ni & 1));
    rm.raise(e.rowmax, n_lane, two);
  }
};

// Dense fp8 backward with ROW-WISE scaling, pointwise part: dH = rs[f] cs[t] acc (rs = the scale of each hidden feature's row of W2,
// cs = the scale of each token's row of dY);  dZ = bf16(dH * 2 sqrt(h)), h the bf16 activation the dense forward kept (H16, dense
// bf16 panel form), at every position.  Stored in bf16 twice, as the [T][F] and the [F][T] operand (dense panel forms) that
// streaming kernels then quantise per token and per hidden feature; rowmax[t] is raised to the largest magnitude word of the row.
struct EpiDReluRw {
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { const __bf16* H16; __bf16* dZ16; __bf16* dZt16; int F; int T; const float* rs; const float* cs; uint32_t* rowmax; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    RowMax<MI, NI> rm;
    rm.load(e.rowmax, n_lane);
    LaneVec<MI> lr;
    lr.load(e.rs, m_lane, 1.f);
    uint32_t mx[NI] = {};
    float cs[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) cs[ni] = e.cs[n_lane + ni];
    LaneSavedDense<MI, NI> sv;
    sv.load(e.H16, e.F, m_lane, n_lane);
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        int f = m_lane + 16 * mi;
        size_t o = a24_piece(n_lane + ni, f >> 5, e.F >> 5) * 32 + (f & 31);
#pragma unroll
        for (int q = 0; q < 2; q++) {
          const u32x4 h = sv.h[mi][ni][q];
          u32x4 r;
#pragma unroll
          for (int d = 0; d < 4; d++) {
            int i = 16 * mi + 8 * q + 2 * d;
            float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[d]));
            float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[d]));
            acc[mi][ni][8 * q + 2 * d] *= (cs[ni] * lr.at(i)) * g0;
            acc[mi][ni][8 * q + 2 * d + 1] *= (cs[ni] * lr.at(i + 1)) * g1;
            r[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d], acc[mi][ni][8 * q + 2 * d + 1]);
            mx[ni] = max(mx[ni], max(r[d] & 0x7FFFu, (r[d] >> 16) & 0x7FFFu));
          }
          *reinterpret_cast<u32x4*>(e.dZ16 + o + 8 * q) = r;
        }
      }
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v];
        st_cols<NI>(e.dZt16 + a24_piece(m_lane + 16 * mi + v, n_lane >> 5, e.T >> 5) * 32 + (n_lane & 31), o);
      }
    }
    uint32_t two[(NI + 1) / 2] = {};
#pragma unroll
    for (int ni = 0; ni < NI; ni++) two[ni / 2] |= mx[ni] << (16 * (ni & 1));
    rm.raise(e.rowmax, n_lane, two);
  }
};

// C[m][n] = bf16(acc * rs[m] * cs[n]), n contiguous (row-wise-scaled fp8 down-projection: rs = sh per token, cs = sw2).
struct EpiRowMajorRowCol {
  struct Args { __bf16* C; int ldc; const float* rs; const float* cs; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    float cs[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) cs[ni] = e.cs[n_lane + ni];
    LaneVec<MI> lr;                                  // the lane's 64 row scales: 16 loads of 16 bytes, not 64 of 4
    lr.load(e.rs, m_lane, 1.f);
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float r = lr.at(16 * mi + v);
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v] * r * cs[ni];
        st_cols<NI>(e.C + (size_t)(m_lane + 16 * mi + v) * e.ldc + n_lane, o);
      }
  }
};

// C[rowmap[m]][n] = bf16(acc * rs[m] * cs[n]): the split weight-gradient GEMMs of the row-wise fp8 backward (rows are positions
// of the permuted feature space, rs their scales in that order; each row goes back to its feature).
struct EpiRowMajorRowColMapped {
  struct Args { __bf16* C; int ldc; const float* rs; const float* cs; const int* rowmap; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    float cs[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) cs[ni] = e.cs[n_lane + ni];
    LaneVec<MI> lr;
    lr.load(e.rs, m_lane, 1.f);
    LaneIdx<MI> rows;
    rows.load(e.rowmap, m_lane);
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float r = lr.at(16 * mi + v);
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v] * r * cs[ni];
        st_cols<NI>(e.C + (size_t)rows.at(16 * mi + v) * e.ldc + n_lane, o);
      }
  }
};

// C stored transposed, out[n][m] = bf16(acc * rs[m] * cs[n]) with m contiguous (row-wise-scaled fp8 dW1 GEMM: rs = the scale of
// each hidden feature's row of the transposed dZ operand, cs = the scale of each model dimension's row of the transposed X).
struct EpiColMajorRowCol {
  static constexpr bool STAGED = true;
  struct Args { __bf16* C; int ldc; const float* rs; const float* cs; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    LaneVec<MI> lr;
    lr.load(e.rs, m_lane, 1.f);
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      const float cs = e.cs[n_lane + ni];
#pragma unroll
      for (int mi = 0; mi < MI; mi++)
#pragma unroll
        for (int q = 0; q < 2; q++) {
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; d++) {
            int i = 16 * mi + 8 * q + 2 * d;
            o[d] = pack_bf16x2(acc[mi][ni][8 * q + 2 * d] * lr.at(i) * cs, acc[mi][ni][8 * q + 2 * d + 1] * lr.at(i + 1) * cs);
          }
          ColMajorStage<MI, NI>::put(wbuf, ni, 2 * mi + q, o);
        }
    }
    ColMajorStage<MI, NI>::flush(wbuf, e.C, e.ldc, m_lane, n_lane);
  }
};

// fp8 backward with ROW-WISE scaling, pointwise part (Sec. 2: the fused backward pointwise step with its FP8 scaling; the
// precision recipe of the paper's benchmarks scales every FP8 GEMM row-wise): acc = (W2_8r . dY8r) for a lane's 64 features x
// 4 tokens; dH = rs[f] cs[t] acc (rs = the scale of each hidden feature's row of W2, cs = the scale of each token's row of dY);
// on the positions the forward kept dZ = dH * 2 sqrt(h), h the bf16 kept value the forward saved (Hc16, meta16: bf16 panel form).
// Like the activation in the row-wise forward, dZ cannot be quantised here -- the scale of a token row spans many block tiles
// -- so it is written as bf16, compressed with the forward's metadata (dZc16, bf16 panel form), and rowmax[t] is
// raised to the largest magnitude word of the row (RowMax); a streaming kernel then quantises with rowmax[t] / 448.
struct EpiDGatherRw {
  static constexpr bool STAGED = true;
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { const __bf16* Hc16; const uint8_t* meta16; __bf16* dZc16; int F; const float* rs; const float* cs; uint32_t* rowmax; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane, char* wbuf) {
    RowMax<MI, NI> rm;
    if constexpr (NI < 8) rm.load(e.rowmax, n_lane);
    LaneVec<MI> lr;
    lr.load(e.rs, m_lane, 1.f);
    LaneSaved24<MI, NI> sv;
    sv.load(e.Hc16, e.meta16, e.F, m_lane, n_lane, wbuf);
    float csv[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++) csv[ni] = e.cs[n_lane + ni];
    uint32_t mx[(NI + 1) / 2] = {};
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      if (NI == 8 && ni == NI / 2) rm.load(e.rowmax, n_lane);   // (from the start on it is two registers too many)
      size_t t = (size_t)(n_lane + ni);
      const float cs = csv[ni];
      size_t piece = a24_piece((int)t, m_lane >> 6, e.F >> 6);
      const u32x2 mt = sv.mt[ni];
      __bf16* zrow = e.dZc16 + piece * 32 + ((m_lane & 63) >> 1);
      uint32_t m = 0u;
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        const u32x4 h = sv.kept(ni, mi);
        u32x4 z;
#pragma unroll
        for (int a = 0; a < 4; a++) {
          int gi = 4 * mi + a;
          uint32_t n4 = (mt[gi >> 3] >> (4 * (gi & 7))) & 15u;
          uint32_t i0 = n4 & 3u, i1 = n4 >> 2;
          float x0 = acc[mi][ni][4 * a] * (cs * lr.at(16 * mi + 4 * a)), x1 = acc[mi][ni][4 * a + 1] * (cs * lr.at(16 * mi + 4 * a + 1));
          float x2 = acc[mi][ni][4 * a + 2] * (cs * lr.at(16 * mi + 4 * a + 2)), x3 = acc[mi][ni][4 * a + 3] * (cs * lr.at(16 * mi + 4 * a + 3));
          float s0 = i0 == 0 ? x0 : (i0 == 1 ? x1 : x2);
          float s1 = i1 == 3 ? x3 : (i1 == 2 ? x2 : x1);
          float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[a]));
          float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[a]));
          z[a] = pack_bf16x2(s0 * g0, s1 * g1);
          m = max(m, max(z[a] & 0x7FFFu, (z[a] >> 16) & 0x7FFFu));
        }
        if constexpr (LaneTile<MI, NI>::STAGED) *reinterpret_cast<u32x4*>(PanelStage<MI, NI>::at(wbuf, ni, mi)) = z;
        else *reinterpret_cast<u32x4*>(zrow + 8 * mi) = z;
      }
      mx[ni / 2] |= m << (16 * (ni & 1));
      keep_here<NI == 8>(mx[ni / 2]);
    }
    rm.raise(e.rowmax, n_lane, mx);
    if constexpr (LaneTile<MI, NI>::STAGED) PanelStage<MI, NI>::flush(wbuf, reinterpret_cast<char*>(e.dZc16) + PanelStage<MI, NI>::first(m_lane, n_lane, e.F));
  }
};

// fp8 dense up-projection (baseline): H8[t][f] = e4m3( bf16(max(0, zscale acc + b1)^2) / sh ), the [T][F] byte operand
// of the dense down-projection, in dense panel form (64-byte pieces of 64 k).
// H16, H8t (optional, a training context): the activation before quantisation as bf16 [T][F] (dense bf16 panel form; the
// backward takes the derivative from it) and the codes once more as the [F][T] operand of the weight-gradient GEMM that
// reduces over tokens (dense fp8 panel form).
struct EpiRelu2F8 {
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { uint8_t* H8; const float* b1; int F; float zscale; float sh; __bf16* H16; uint8_t* H8t; int T; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    LaneVec<MI> lb;
    lb.load(e.b1, m_lane, 0.f);
    uint32_t qs[NI][4 * MI];   // the lane's codes: [token][4 features per word]
    const ExactDiv by_sh(e.sh);
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      uint8_t* row = e.H8 + a24_piece(n_lane + ni, m_lane >> 6, e.F >> 6) * 64 + (m_lane & 63);
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        uint32_t q[4], hp[8];
#pragma unroll
        for (int d = 0; d < 8; d++) {
          float b0 = lb.at(16 * mi + 2 * d), b1v = lb.at(16 * mi + 2 * d + 1);
          float r0 = fmaxf(acc[mi][ni][2 * d] * e.zscale + b0, 0.f);
          float r1 = fmaxf(acc[mi][ni][2 * d + 1] * e.zscale + b1v, 0.f);
          hp[d] = pack_bf16x2(r0 * r0, r1 * r1);
          q[d >> 1] = cvt_e4m3x2(by_sh(bf16_lo_to_f32(hp[d])), by_sh(bf16_hi_to_f32(hp[d])), (d & 1) ? q[d >> 1] : 0u, (d & 1) != 0);
        }
        *reinterpret_cast<u32x4*>(row + 16 * mi) = u32x4{q[0], q[1], q[2], q[3]};
        if (e.H16) {
          int f = m_lane + 16 * mi;
          __bf16* r16 = e.H16 + a24_piece(n_lane + ni, f >> 5, e.F >> 5) * 32 + (f & 31);
          *reinterpret_cast<u32x4*>(r16) = u32x4{hp[0], hp[1], hp[2], hp[3]};
          *reinterpret_cast<u32x4*>(r16 + 8) = u32x4{hp[4], hp[5], hp[6], hp[7]};
        }
#pragma unroll
        for (int d = 0; d < 4; d++) qs[ni][4 * mi + d] = q[d];
      }
    }
    if (e.H8t) {
      // feature m_lane + 4 w + b: its codes of the lane's NI consecutive tokens -> one store
#pragma unroll
      for (int w = 0; w < 4 * MI; w++)
#pragma unroll
        for (int b = 0; b < 4; b++) {
          uint32_t t[NI];
#pragma unroll
          for (int ni = 0; ni < NI; ni++) t[ni] = qs[ni][w];
          st_bytes<NI>(e.H8t + a24_piece(m_lane + 4 * w + b, n_lane >> 6, e.T >> 6) * 64 + (n_lane & 63), t, b);
        }
    }
  }
};

// Dense fp8 backward, pointwise part: acc = (W2_8 . dY8) for a lane's 64 features x 4 tokens; dZ = scale * acc * 2 sqrt(h) with h
// the bf16 activation the dense forward saved (H16, dense bf16 panel form); stored as e4m3(dZ / sdz) twice: the [T][F]
// operand of the dX GEMM and the [F][T] operand of the dW1 GEMM (dense fp8 panel forms).
struct EpiDReluF8 {
  static constexpr EpiCost COST = EPI_FP8;
  struct Args { const __bf16* H16; uint8_t* dZ8; uint8_t* dZ8t; int F; int T; float scale; float sdz; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
    uint32_t qs[NI][4 * MI];
    const ExactDiv by_sdz(e.sdz);
    LaneSavedDense<MI, NI> sv;
    sv.load(e.H16, e.F, m_lane, n_lane);
#pragma unroll
    for (int ni = 0; ni < NI; ni++) {
      uint8_t* row = e.dZ8 + a24_piece(n_lane + ni, m_lane >> 6, e.F >> 6) * 64 + (m_lane & 63);
#pragma unroll
      for (int mi = 0; mi < MI; mi++) {
        uint32_t q[4];
#pragma unroll
        for (int hq = 0; hq < 2; hq++) {
          const u32x4 h = sv.h[mi][ni][hq];
#pragma unroll
          for (int d = 0; d < 4; d++) {
            float g0 = 2.f * __builtin_amdgcn_sqrtf(bf16_lo_to_f32(h[d]));
            float g1 = 2.f * __builtin_amdgcn_sqrtf(bf16_hi_to_f32(h[d]));
            float v0 = by_sdz(acc[mi][ni][8 * hq + 2 * d] * e.scale * g0), v1 = by_sdz(acc[mi][ni][8 * hq + 2 * d + 1] * e.scale * g1);
            int dd = 4 * hq + d;
            q[dd >> 1] = cvt_e4m3x2(v0, v1, (dd & 1) ? q[dd >> 1] : 0u, (dd & 1) != 0);
          }
        }
        *reinterpret_cast<u32x4*>(row + 16 * mi) = u32x4{q[0], q[1], q[2], q[3]};
#pragma unroll
        for (int d = 0; d < 4; d++) qs[ni][4 * mi + d] = q[d];
      }
    }
#pragma unroll
    for (int w = 0; w < 4 * MI; w++)
#pragma unroll
      for (int b = 0; b < 4; b++) {
        uint32_t t[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) t[ni] = qs[ni][w];
        st_bytes<NI>(e.dZ8t + a24_piece(m_lane + 4 * w + b, n_lane >> 6, e.T >> 6) * 64 + (n_lane & 63), t, b);
      }
  }
};

// C[m][n] = bf16(scale * acc), n contiguous (fp8 down-projection: scale = sh * sw2).
struct EpiRowMajorScaled {
  struct Args { __bf16* C; int ldc; float scale; };
  template <int MI, int NI, class Acc>
  static __device__ __forceinline__ void run(const Args& e, Acc& acc, int m_lane, int n_lane) {
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float o[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ni++) o[ni] = acc[mi][ni][v] * e.scale;
        st_cols<NI>(e.C + (size_t)(m_lane + 16 * mi + v) * e.ldc + n_lane, o);
      }
  }
};

}  // namespace ffn24
