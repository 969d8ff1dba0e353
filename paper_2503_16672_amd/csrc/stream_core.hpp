// Streaming work that kernels of its own (k_stream.hip) and launches that carry it beside a GEMM share.
#pragma once
#include "gemm_core.hpp"
#include "launch.hpp"

namespace ffn24 {

// Streaming accesses: every byte these kernels touch is read or written once, so loads and stores carry the non-temporal
// hint (measured on a plain copy: 6.0-6.5 TB/s with it, 5.6-6.1 without).
template <class T> __device__ __forceinline__ T ld_stream(const T* p) { return __builtin_nontemporal_load(p); }
template <class T> __device__ __forceinline__ void st_stream(T* p, T v) { __builtin_nontemporal_store(v, p); }
// What the next kernels read again is stored without it (operands brought into another form, small transposed ones): the caches then still hold some of it.
template <class T> __device__ __forceinline__ void st_keep(T* p, T v) { *p = v; }

// Feature-wise 2:4 on top of the token-wise mask (Sec. 2, last paragraph; Fig. 2c).
// Input: token-wise compressed Hc [T][F/2] + meta [T][F/8], and optionally dZc [T][F/2] with the same metadata.
// Output: for every feature, groups of 4 consecutive tokens of the pruned activation keep their top-2:
//   Hc_t [F][T/2], meta_t [F][T/8], and dZc_t [F][T/2] = dZ at the positions picked for H.
// Inputs and outputs in the panel form of gemm_core.hpp (a caller's row-major tensors: PANEL = false, and featurewise24_rows_kernel in k_stream.hip).
// One workgroup handles 64 tokens x 64 features at a time: decompress into LDS, then each work item takes two features and 8 consecutive
// tokens (two groups each).  A tile's input is one contiguous 4 KiB run per tensor and it writes one contiguous 4 KiB run; 128-token
// tiles, with twice the LDS per workgroup and half the workgroups per CU, ran at 5.0 instead of 5.9 TB/s.  Words are pairs of features
// throughout, f in the low half and f + 8 in the high half, so that the decompression and the pick are packed and bitwise arithmetic on
// two groups, LDS is accessed by whole dwords (a pitch of 33: a wave's reads, 8 words of 8 token octets, fall into 64 different banks),
// and a wave's stores cover 8 consecutive features at a time.
// A workgroup walks `tiles` tiles of 64 tokens (fw_tiles), the next one's input on its way while this one is worked on, and raises the row maxima
// once: with one tile a workgroup two million atomics went out at T = F = 8192.  What bounds it is HBM; feature by feature and tile by tile
// it took 82.9 us there with the maxima and a split, now 52-57 = 5.0 TB/s and more; without them, T = F = 16384, 206 -> 180 = 6.3 TB/s; T 1280
// F 3072 5.7 -> 4.5.
constexpr int FW_TOK = 64, FW_FEAT = 64, FW_LDW = FW_FEAT / 2 + 1, FW_TILES = 4;
constexpr int FW_LDS = 4 * (2 * FW_TOK * FW_LDW + 4);

// all ones in the halves of the mask where bit b of the half is set
__device__ __forceinline__ uint32_t half_mask(uint32_t w, int b) {
  uint32_t m = __builtin_bit_cast(uint32_t, (i16x2)((i16x2)(as_i16x2(w) << (i16x2)(15 - b)) >> (i16x2)(15)));
  asm("" : "+v"(m));   // (opaque, as in pk_less16)
  return m;
}
__device__ __forceinline__ uint32_t sel(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }
__device__ __forceinline__ uint32_t halves_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }   // a's low half, b's above it
__device__ __forceinline__ uint32_t halves_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// PANEL: in the panel form; otherwise row-major, for matrices too small for featurewise24_rows_kernel's tiles to fill the chip.
// SPLIT (Sec. 2, "Optimization 1"; panel form only): feature f becomes row row_of_feat[f] of the outputs; rows below
// n_sparse are 2:4-compressed along tokens as above, the others -- the least sparse features -- are written out
// uncompressed, as rows [row - n_sparse] of the dense operands Hdn_t, dZdn_t [n_dense][T] (dense panel form).
// KEEP (compressed outputs in the panel form; fw_keep): stored without the streaming hint.  A template argument: where only a value tells two such
// stores apart the compiler makes one store of them, without the hint.
// (bx, by): which workgroup of a grid of F / FW_FEAT by T / (FW_TOK tiles); sH: FW_LDS bytes
template <bool PANEL, bool SPLIT = false, bool KEEP = false>
__device__ __forceinline__ void featurewise24_tiles(const uint16_t* __restrict__ Hc, const uint8_t* __restrict__ meta, const uint16_t* __restrict__ dZc, int T,
                                                    int F, int tiles, uint16_t* __restrict__ Hc_t, uint8_t* __restrict__ meta_t,
                                                    uint16_t* __restrict__ dZc_t, const int* __restrict__ row_of_feat, int n_sparse,
                                                    uint16_t* __restrict__ Hdn_t, uint16_t* __restrict__ dZdn_t,
                                                    unsigned long long* __restrict__ tele, uint32_t* __restrict__ hmax, uint32_t* __restrict__ zmax,
                                                    int bx, int by, uint32_t* sH) {
  uint32_t* sZ = sH + FW_TOK * FW_LDW;
  const int f0 = bx * FW_FEAT, t_first = by * FW_TOK * tiles;
  const int tid = threadIdx.x;
  const bool has_z = dZc != nullptr;
  const int tok = tid >> 2, ch = tid & 3;            // in: 16 features of a token
  const int oct = tid & 7, word = tid >> 3;          // out: 8 tokens of features fa and fa + 8
  const int fa = ((word >> 3) << 4) | (word & 7);
  u32x4 hv, zv = {0u, 0u, 0u, 0u};
  uint32_t mv;
  auto request = [&](int t0) {
    // offsets of this item's 8 stored values (in elements) and of its 2 metadata bytes
    const int t = t0 + tok;
    const size_t piece = PANEL ? a24_piece(t, f0 >> 6, F >> 6) : (size_t)t * (F >> 6) + (f0 >> 6), vo = piece * 32 + 8 * ch, mo = piece * 8 + 2 * ch;
    hv = ld_stream(reinterpret_cast<const u32x4*>(Hc + vo));
    if (has_z) zv = ld_stream(reinterpret_cast<const u32x4*>(dZc + vo));
    mv = ld_stream(reinterpret_cast<const uint16_t*>(meta + mo));
  };
  request(t_first);
  int orow[2];
  uint32_t dense = 0u;                               // SPLIT: the halves whose feature is written out uncompressed
#pragma unroll
  for (int b = 0; b < 2; b++) {
    orow[b] = SPLIT ? row_of_feat[f0 + fa + 8 * b] : f0 + fa + 8 * b;
    if (SPLIT && orow[b] >= n_sparse) dense |= 0xFFFFu << (16 * b);
  }
  uint32_t kept = 0u, mh = 0u, mz = 0u;              // non-zero activations this work item writes out; its largest magnitudes (of either half)
  for (int it = 0; it < tiles; it++) {
    const int t0 = t_first + FW_TOK * it;
    const uint32_t mm = (mv & 0xFFu) | ((mv & 0xFF00u) << 8);   // nibbles of groups 0, 1 below, of groups 2, 3 in the high half
#pragma unroll
    for (int g = 0; g < 2; g++) {                    // groups g and g + 2
      const uint32_t b0 = half_mask(mm, 4 * g), b1 = half_mask(mm, 4 * g + 1), b2 = half_mask(mm, 4 * g + 2), b3 = half_mask(mm, 4 * g + 3);
      const uint32_t at0[4] = {~b0 & ~b1, b0 & ~b1, ~b0 & b1, b0 & b1}, at1[4] = {~b2 & ~b3, b2 & ~b3, ~b2 & b3, b2 & b3};
      const uint32_t h0 = halves_lo(hv[g], hv[g + 2]), h1 = halves_hi(hv[g], hv[g + 2]), z0 = halves_lo(zv[g], zv[g + 2]), z1 = halves_hi(zv[g], zv[g + 2]);
      const int o = tok * FW_LDW + 8 * ch + 4 * g;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        sH[o + j] = sel(at0[j], h0, h1 & at1[j]);
        if (has_z) sZ[o + j] = sel(at0[j], z0, z1 & at1[j]);
      }
    }
    __syncthreads();
    if (it + 1 < tiles) request(t0 + FW_TOK);
    uint32_t h[8], z[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
      h[j] = sH[(8 * oct + j) * FW_LDW + word];
      z[j] = has_z ? sZ[(8 * oct + j) * FW_LDW + word] : 0u;
    }
    if (it + 1 < tiles) __syncthreads();             // the next tile may overwrite the image
    uint32_t hp[2][2], zp[2][2], nib = 0u;           // [feature][group]
    uint32_t zall = 0u;
#pragma unroll
    for (int g = 0; g < 2; g++) {
      uint32_t m[4];
#pragma unroll
      for (int j = 0; j < 4; j++) m[j] = h[4 * g + j] & 0x7FFF7FFFu;   // the pick is by magnitude
      const Pick24x2 p = pick24_two(m[0], m[1], m[2], m[3]);
      const uint32_t second0 = p.bit[0] /* i0 == 1 */, third0 = p.bit[1], last1 = p.bit[2] & p.bit[3], not_first1 = p.bit[3];
      const uint32_t *a = h + 4 * g, *c = z + 4 * g;
      const uint32_t hf = sel(third0, a[2], sel(second0, a[1], a[0])), hs = sel(not_first1, sel(last1, a[3], a[2]), a[1]);
      const uint32_t zf = sel(third0, c[2], sel(second0, c[1], c[0])), zs = sel(not_first1, sel(last1, c[3], c[2]), c[1]);
      hp[0][g] = halves_lo(hf, hs); hp[1][g] = halves_hi(hf, hs);
      zp[0][g] = halves_lo(zf, zs); zp[1][g] = halves_hi(zf, zs);
      nib = put_nibbles(nib, p, g);
      if (hmax) {
        mh = pk_max16(mh, pk_max16(pk_max16(m[0], m[1]), pk_max16(m[2], m[3])));   // (the largest of a group is always kept)
        mz = pk_max16(mz, SPLIT ? ~dense & pk_max16(zf & 0x7FFF7FFFu, zs & 0x7FFF7FFFu) : pk_max16(zf & 0x7FFF7FFFu, zs & 0x7FFF7FFFu));
        if constexpr (SPLIT) {
#pragma unroll
          for (int j = 0; j < 4; j++) zall = pk_max16(zall, c[j] & 0x7FFF7FFFu);
        }
      }
      if (tele) {
        uint32_t n = pk_min16(hf & 0x7FFF7FFFu, 0x00010001u) + pk_min16(hs & 0x7FFF7FFFu, 0x00010001u);
        if constexpr (SPLIT) {
          uint32_t all = 0u;
#pragma unroll
          for (int j = 0; j < 4; j++) all += pk_min16(m[j], 0x00010001u);
          n = sel(dense, all, n);
        }
        kept += (n & 0xFFFFu) + (n >> 16);
      }
    }
    if (SPLIT) mz = pk_max16(mz, dense & zall);
    const int t = t0 + 8 * oct;
#pragma unroll
    for (int b = 0; b < 2; b++) {
      if (SPLIT && orow[b] >= n_sparse) {            // dense feature: its 8 tokens as they are (already token-wise pruned)
        const size_t o = a24_piece(orow[b] - n_sparse, t >> 5, T >> 5) * 32 + (t & 31);
        u32x4 x, y;
#pragma unroll
        for (int d = 0; d < 4; d++) {
          x[d] = b ? halves_hi(h[2 * d], h[2 * d + 1]) : halves_lo(h[2 * d], h[2 * d + 1]);
          y[d] = b ? halves_hi(z[2 * d], z[2 * d + 1]) : halves_lo(z[2 * d], z[2 * d + 1]);
        }
        *reinterpret_cast<u32x4*>(Hdn_t + o) = x;
        if (has_z) *reinterpret_cast<u32x4*>(dZdn_t + o) = y;
        continue;
      }
      const size_t piece = PANEL ? a24_piece(orow[b], t >> 6, T >> 6) : (size_t)orow[b] * (T >> 6) + (t >> 6);
      const size_t vo = piece * 32 + 4 * oct, mo = piece * 8 + oct;
      const u32x2 hv2 = {hp[b][0], hp[b][1]}, zv2 = {zp[b][0], zp[b][1]};
      const uint8_t mv2 = (uint8_t)(b ? nib >> 16 : nib);
      if constexpr (KEEP) {
        st_keep(reinterpret_cast<u32x2*>(Hc_t + vo), hv2);
        if (has_z) st_keep(reinterpret_cast<u32x2*>(dZc_t + vo), zv2);
        st_keep(meta_t + mo, mv2);
      } else {
        st_stream(reinterpret_cast<u32x2*>(Hc_t + vo), hv2);
        if (has_z) st_stream(reinterpret_cast<u32x2*>(dZc_t + vo), zv2);
        st_stream(meta_t + mo, mv2);
      }
    }
  }
  if (hmax) {
    // largest stored magnitude word of a feature's row, for a row-wise quantisation that follows (the eight work items of two features
    // are neighbouring lanes: one atomic per feature, tensor and workgroup)
#pragma unroll
    for (int sft = 1; sft < 8; sft <<= 1) {
      mh = pk_max16(mh, (uint32_t)__shfl_xor((int)mh, sft, 64));
      mz = pk_max16(mz, (uint32_t)__shfl_xor((int)mz, sft, 64));
    }
    if (oct < 2) {                                   // lane 0 of the eight raises the one feature's, lane 1 the other's
      const uint32_t a = oct ? mh >> 16 : mh & 0xFFFFu, c = oct ? mz >> 16 : mz & 0xFFFFu;
      const int r = oct ? orow[1] : orow[0];
      if (a) atomicMax(hmax + r, a);
      if (c && has_z) atomicMax(zmax + r, c);
    }
  }
  // what the weight-gradient GEMMs still see of the activation (Sec. 2: the second, feature-wise drop): one atomic
  // per workgroup (tele is a kernel argument, so the barrier is reached by all or none)
  if (tele) {
    uint32_t* s_kept = sH + 2 * FW_TOK * FW_LDW;
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) kept += (uint32_t)__shfl_xor((int)kept, sft, 64);
    if ((tid & 63) == 0) s_kept[tid >> 6] = kept;
    __syncthreads();
    if (tid == 0)
      atomicAdd(tele + tele_index(TELE_KEPT_FEAT, bx + 5 * by),
                (unsigned long long)(s_kept[0] + s_kept[1] + s_kept[2] + s_kept[3]));
  }
}

// Operands that the last-level cache (256 MB) can hold beside what else the weight gradients read stay there for them; larger ones would push that out.
// With the hint / without, whole steps (us, T D F): bf16 8192 512 4096 204, 192; 8192 1024 4096 323, 313; 4096 1024 5120 228, 222; 8192 1024 6144 level;
// 16384 512 4096 375, 394; 8192 2048 8192 982, 991; 10240 2048 8192 1283, 1314; 131072 512 1024 1063, 1164; 16384 4096 16384 7067, 7088; the other way round at
// 16384 1024 4096 599, 581 and 12288 1024 8192 864, 853; with a split or row maxima within 1 %.
inline bool fw_keep(int T, int F) { return (size_t)T * F < 1 << 26; }

// Work that rides beside a GEMM's tiles in one launch (gemm_side_kernel): run(args, workgroup, LDS).
// The feature-wise re-compression (panel form, one tile of tokens a workgroup), beside the dX GEMM, which needs nothing of it.
struct SideFeaturewise {
  struct Args { const uint16_t* Hc; const uint8_t* meta; const uint16_t* dZc; int T, F; uint16_t* Hc_t; uint8_t* meta_t; uint16_t* dZc_t; };
  static __device__ __forceinline__ void run(const Args& a, unsigned bid, char* smem) {
    const unsigned nx = (unsigned)a.F / FW_FEAT;
    featurewise24_tiles<true, false, true>(a.Hc, a.meta, a.dZc, a.T, a.F, 1, a.Hc_t, a.meta_t, a.dZc_t, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr, (int)(bid % nx),
                              (int)(bid / nx), reinterpret_cast<uint32_t*>(smem));
  }
};

}  // namespace ffn24
