// Streaming (HBM-bound) kernels: the standalone 2:4 compression of an activation matrix, the feature-wise
// (along-token) re-compression the weight-gradient GEMMs need, and the bf16 matrix transpose that brings a GEMM
// operand into K-contiguous form.
#include "epilogues.hpp"
#include "launch.hpp"
#include "stream_core.hpp"
#include "tile_rule.hpp"

namespace ffn24 {

// key of a bf16 storage word at position i of its group: ((magnitude << 2) | (3 - i)) << 1 | sign.
// The sign rides in the lowest bit, below the position, so it never takes part in the ordering.
__device__ __forceinline__ uint32_t key_of(uint32_t w, uint32_t i) { return ((((w & 0x7FFFu) << 2) | (3u - i)) << 1) | (w >> 15); }
__device__ __forceinline__ uint32_t word_of(uint32_t key) { return (key >> 3) | ((key & 1u) << 15); }

// pick on keys that carry the sign bit: strip it for the position arithmetic of pick24_keys
__device__ __forceinline__ uint32_t pick24_words(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t& pair) {
  uint32_t k0 = key_of(w0, 0), k1 = key_of(w1, 1), k2 = key_of(w2, 2), k3 = key_of(w3, 3);
  uint32_t a = max(k0, k1), b = min(k0, k1), c = max(k2, k3), d = min(k2, k3);
  uint32_t top = max(a, c);
  uint32_t e = max(b, d);
  uint32_t second = max(min(a, c), min(max(a, c), e));
  uint32_t ct = (top >> 1) & 3u, cs = (second >> 1) & 3u;
  bool top_first = ct > cs;
  uint32_t kf = top_first ? top : second, ks = top_first ? second : top;
  pair = word_of(kf) | (word_of(ks) << 16);
  uint32_t cmax = max(ct, cs), cmin = min(ct, cs);
  return (cmax | (cmin << 2)) ^ 15u;
}

// Standalone sparsify24 (Sec. 2 of the paper, first paragraph): each thread takes 8 consecutive elements
// (two groups): one 16-byte load, one 8-byte store of kept values, one metadata byte.  The matrix is
// processed as a flat array, which is valid because cols % 8 == 0.
__global__ void __launch_bounds__(256) sparsify24_kernel(const u32x4* __restrict__ in, int64_t n_oct,
                                                         u32x2* __restrict__ vals, uint8_t* __restrict__ meta) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n_oct; o += stride) {
    u32x4 v = ld_stream(in + o);
    uint32_t p0, p1;
    uint32_t n0 = pick24_words(v[0] & 0xFFFFu, v[0] >> 16, v[1] & 0xFFFFu, v[1] >> 16, p0);
    uint32_t n1 = pick24_words(v[2] & 0xFFFFu, v[2] >> 16, v[3] & 0xFFFFu, v[3] >> 16, p1);
    st_stream(vals + o, u32x2{p0, p1});
    st_stream(meta + o, (uint8_t)(n0 | (n1 << 4)));
  }
}

// largest magnitudes of a bf16 vector, lane by lane of its 16-bit halves (sign cleared, as unsigned integers)
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ u16x8 max_mag(u16x8 m, u32x4 v) {
  return __builtin_elementwise_max(m, __builtin_bit_cast(u16x8, v & u32x4{0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu}));
}
__device__ __forceinline__ float scale_of_max(uint32_t word) {
  const float mx = __builtin_bit_cast(float, word << 16);
  return mx > 0.f ? mx / 448.f : 1.f;
}

// 8 bf16 values -> 8 codes, value j divided by d[j] (or all by the one divider)
template <int N>
__device__ __forceinline__ u32x2 quantise8(u32x4 v, const ExactDiv (&d)[N]) {
  uint32_t q[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int j = 4 * i;
    q[i] = cvt_e4m3x2(d[j % N](bf16_lo_to_f32(v[2 * i])), d[(j + 1) % N](bf16_hi_to_f32(v[2 * i])), 0u, false);
    q[i] = cvt_e4m3x2(d[(j + 2) % N](bf16_lo_to_f32(v[2 * i + 1])), d[(j + 3) % N](bf16_hi_to_f32(v[2 * i + 1])), q[i], true);
  }
  return u32x2{q[0], q[1]};
}
// Standalone activation-side kernel of Sec. 2 (sparsification and FP8 quantisation in one pass): the pick is made on the
// bf16 words exactly as above, the two kept values of each group are then quantised, e4m3(kept / scale), saturating.
// Per work item 8 elements: one 16-byte load, 4 code bytes, one metadata byte (2.625 bytes per element in all).
__global__ void __launch_bounds__(256) sparsify24_quant_kernel(const u32x4* __restrict__ in, int64_t n_oct, float scale,
                                                               uint32_t* __restrict__ vals8, uint8_t* __restrict__ meta) {
  const ExactDiv by_scale(scale);
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n_oct; o += stride) {
    u32x4 v = ld_stream(in + o);
    uint32_t p0, p1;
    uint32_t n0 = pick24_words(v[0] & 0xFFFFu, v[0] >> 16, v[1] & 0xFFFFu, v[1] >> 16, p0);
    uint32_t n1 = pick24_words(v[2] & 0xFFFFu, v[2] >> 16, v[3] & 0xFFFFu, v[3] >> 16, p1);
    uint32_t q = cvt_e4m3x2(by_scale(bf16_lo_to_f32(p0)), by_scale(bf16_hi_to_f32(p0)), 0u, false);
    q = cvt_e4m3x2(by_scale(bf16_lo_to_f32(p1)), by_scale(bf16_hi_to_f32(p1)), q, true);
    st_stream(vals8 + o, q);
    st_stream(meta + o, (uint8_t)(n0 | (n1 << 4)));
  }
}

// 2:4 compression of a tensor that already is e4m3: the pick on the code bytes (sign cleared, as integers; ties -> lower
// index).  A work item takes 16 bytes (four groups) and writes 8 code bytes and 2 metadata bytes.
__global__ void __launch_bounds__(256) sparsify24_bytes_kernel(const u32x4* __restrict__ in, int64_t n16,
                                                               u32x2* __restrict__ vals8, uint16_t* __restrict__ meta) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n16; o += stride) {
    u32x4 v = ld_stream(in + o);
    uint32_t out[2] = {0u, 0u}, m = 0u;
#pragma unroll
    for (int g = 0; g < 4; g++) {
      uint32_t w = v[g];
      uint32_t b0 = w & 0xFFu, b1 = (w >> 8) & 0xFFu, b2 = (w >> 16) & 0xFFu, b3 = w >> 24;
      uint32_t k0 = ((b0 & 0x7Fu) << 2) | 3u, k1 = ((b1 & 0x7Fu) << 2) | 2u, k2 = ((b2 & 0x7Fu) << 2) | 1u, k3 = (b3 & 0x7Fu) << 2;
      uint32_t kf, ks;
      uint32_t nib = pick24_keys(k0, k1, k2, k3, kf, ks);
      uint32_t i0 = nib & 3u, i1 = nib >> 2;
      uint32_t a = (w >> (8 * i0)) & 0xFFu, b = (w >> (8 * i1)) & 0xFFu;
      out[g >> 1] |= (a | (b << 8)) << (16 * (g & 1));
      m |= nib << (4 * g);
    }
    st_stream(vals8 + o, u32x2{out[0], out[1]});
    st_stream(meta + o, (uint16_t)m);
  }
}

int launch_sparsify24_quant(const void* H, int64_t rows, int64_t cols, float scale, void* vals8, uint8_t* meta, hipStream_t s) {
  int64_t n_oct = rows * cols / 8;
  if (n_oct == 0) return 0;
  int64_t blocks = (n_oct + 255) / 256;
  if (blocks > 0x7FFFFFFF) blocks = 0x7FFFFFFF;   // one work item per thread: the fastest shape for a streaming kernel here
  hipLaunchKernelGGL(sparsify24_quant_kernel, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const u32x4*>(H), n_oct, scale,
                     static_cast<uint32_t*>(vals8), meta);
  return (int)hipGetLastError();
}

int launch_sparsify24_bytes(const void* H8, int64_t rows, int64_t cols, void* vals8, uint8_t* meta, hipStream_t s) {
  int64_t n16 = rows * cols / 16;
  if (n16 == 0) return 0;
  int64_t blocks = (n16 + 255) / 256;
  if (blocks > 0x7FFFFFFF) blocks = 0x7FFFFFFF;   // one work item per thread: the fastest shape for a streaming kernel here
  hipLaunchKernelGGL(sparsify24_bytes_kernel, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const u32x4*>(H8), n16,
                     static_cast<u32x2*>(vals8), reinterpret_cast<uint16_t*>(meta));
  return (int)hipGetLastError();
}

int launch_sparsify24(const void* H, int64_t rows, int64_t cols, void* vals, uint8_t* meta, hipStream_t s) {
  int64_t n_oct = rows * cols / 8;
  if (n_oct == 0) return 0;
  int64_t blocks = (n_oct + 255) / 256;
  if (blocks > 0x7FFFFFFF) blocks = 0x7FFFFFFF;   // one work item per thread: the fastest shape for a streaming kernel here
  hipLaunchKernelGGL(sparsify24_kernel, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const u32x4*>(H), n_oct,
                     static_cast<u32x2*>(vals), meta);
  return (int)hipGetLastError();
}

template <bool PANEL, bool SPLIT = false, bool KEEP = false>
__global__ void __launch_bounds__(256) featurewise24_kernel(const uint16_t* __restrict__ Hc, const uint8_t* __restrict__ meta,
                                                            const uint16_t* __restrict__ dZc, int T, int F, int tiles,
                                                            uint16_t* __restrict__ Hc_t, uint8_t* __restrict__ meta_t,
                                                            uint16_t* __restrict__ dZc_t, const int* __restrict__ row_of_feat,
                                                            int n_sparse, uint16_t* __restrict__ Hdn_t, uint16_t* __restrict__ dZdn_t,
                                                            unsigned long long* __restrict__ tele, uint32_t* __restrict__ hmax,
                                                            uint32_t* __restrict__ zmax) {
  __shared__ uint32_t lds[FW_LDS / 4];
  featurewise24_tiles<PANEL, SPLIT, KEEP>(Hc, meta, dZc, T, F, tiles, Hc_t, meta_t, dZc_t, row_of_feat, n_sparse, Hdn_t, dZdn_t, tele, hmax, zmax, blockIdx.x,
                                    blockIdx.y, lds);
}

// Tiles of 64 tokens a workgroup of the panel form walks (T a multiple of 256): four with a split and row maxima, whose atomics go to rows all
// over the matrix, from a workgroup a CU on; one otherwise.  One, four, in a kernel trace of whole steps (us, T F), with split and maxima: 1280
// 3072 8.8, 9.2; 2048 2048 11.2, 9.7; 2048 4096 13.1, 11.5; 4096 4096 21.0, 18.8; 8192 2048 28.6, 17.8; 8192 8192 80, 61; 16384 8192 158, 111.
// Maxima without a split: 2048 4096 8.5, 10.6; 8192 2048 19.4, 18.2; 4096 8192 28.4, 29.8; 8192 8192 50.2, 48.7; 16384 8192 112, 115; 16384 16384
// 198, 214.  Neither: 2048 4096 6.9, 8.1; 4096 8192 23.9, 24.9; 8192 8192 44.5, 47.8; 16384 16384 180, 197 (telemetry 186, 200); a split alone lies
// within 4 % either way from 2048 4096 on.  The level differs from program to program, for one and four alike: in a loop
// with a dense step in between, neither at 8192 8192 takes 59 and 60.
static int fw_tiles(int T, int F, bool split_maxima) { return split_maxima && (F / FW_FEAT) * (T / (FW_TOK * FW_TILES)) >= 256 ? FW_TILES : 1; }

// out[0] = elements, out[1 + k] = the sum of the slots of quantity k, out[4] = path: what a telemetry snapshot holds
__global__ void __launch_bounds__(64) tele_sum_kernel(const unsigned long long* __restrict__ tele, long long elements, long long path,
                                                      long long* __restrict__ out) {
  int k = threadIdx.x;
  if (k < TELE_KINDS) {
    unsigned long long sum = 0;
    for (int i = 0; i < TELE_SLOTS; i++) sum += tele[tele_index(k, i)];
    out[1 + k] = (long long)sum;
  }
  if (k == TELE_KINDS) { out[0] = elements; out[1 + TELE_KINDS] = path; }
}

int launch_tele_sum(const unsigned long long* tele, long long elements, long long path, long long* out, hipStream_t s) {
  hipLaunchKernelGGL(tele_sum_kernel, dim3(1), dim3(64), 0, s, tele, elements, path, out);
  return (int)hipGetLastError();
}

// The same for a caller's row-major tensors (T a multiple of 128, F of 64).  What bounds it is HBM, so both sides move whole lines.  A
// workgroup takes 128 tokens x 256 features; a lane owns one group of 4 features and reads its 4-byte pair of each of its wave's
// 32 tokens, so a wave's load is 256 contiguous bytes of a token row, all 64 of them are in flight before the first is used, and
// nothing has to be spread out in LDS first.  A lane then holds 8 consecutive tokens (two groups) of 4 features at a time; the picked
// values go to an LDS image of the transposed rows (H first, dZ after it through the same space) and leave as whole lines, 128 bytes
// of a feature row.  In the image the rows of features 4 l + j stand at j * 64 + l: a wave's 8-byte writes then step through
// consecutive rows, whose pitch keeps them on different banks.  Each XCD takes a contiguous run of the tiles, features fastest: a token
// row's metadata line serves four neighbouring tiles and should be fetched by one L2.
// Measured at 8064 x 8256 / 16384 x 16384 (with dZ): 67 us = 4.2 TB/s / 230 us = 5.0 TB/s; tiles dealt round-robin over the XCDs 69 / 259-307
// us; 64-token tiles 81 / 373 us, 32-token tiles 207 / 1005 us (half and quarter lines out); three workgroups a CU 135 / 538 us (spills).
// 64 x 64 tiles spread out in LDS (featurewise24_kernel<false>), which read and write half lines and 8-byte metadata pieces, take 71 us at 8064 x
// 4160, where these take 38, but fill the chip from eight times fewer elements on: small matrices take them (featurewise_small).
constexpr int FWR_CH = 4, FWR_TOK = 32 * FWR_CH;   // chunks of 8 tokens per wave, tokens per workgroup
__global__ void __launch_bounds__(256, 2) featurewise24_rows_kernel(const uint32_t* __restrict__ Hc, const uint8_t* __restrict__ meta,
                                                                    const uint32_t* __restrict__ dZc, int T, int F, uint8_t* __restrict__ Hc_t,
                                                                    uint8_t* __restrict__ meta_t, uint8_t* __restrict__ dZc_t) {
  constexpr int CH = FWR_CH, TOK = FWR_TOK, ROWB = TOK, PITCH = ROWB + 16;   // bytes of stored values per transposed row; LDS pitch
  __shared__ __attribute__((aligned(16))) uint8_t sV[256 * PITCH];
  __shared__ __attribute__((aligned(16))) uint32_t sM[256 * CH];             // 4 CH metadata bytes per feature, CH of each wave
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // workgroup id -> tile: ids go round-robin over the 8 XCDs; XCD x takes the tiles from x (n / 8) + min(x, n % 8) on
  const unsigned nf = gridDim.x, n = nf * gridDim.y, bid = blockIdx.x + nf * blockIdx.y, xcd = bid & 7;
  const unsigned tile = xcd * (n >> 3) + min(xcd, n & 7) + (bid >> 3);
  const int f0 = (int)(tile % nf) * 256, t0 = (int)(tile / nf) * TOK;
  const int G = F >> 2;                                           // groups (4-byte pairs) per token row
  const int g = min((f0 >> 2) + lane, G - 1);                     // lanes beyond the last group repeat it; nothing of theirs is stored
  const bool has_z = dZc != nullptr;
  const size_t tw = (size_t)(t0 + 8 * CH * wave);
  uint32_t h[8 * CH], z[8 * CH], m[8 * CH];
#pragma unroll
  for (int i = 0; i < 8 * CH; i++) {
    h[i] = ld_stream(Hc + (tw + i) * G + g);
    m[i] = meta[(tw + i) * (G >> 1) + (g >> 1)];
    z[i] = has_z ? ld_stream(dZc + (tw + i) * G + g) : 0u;
  }
  uint32_t zo[CH][4][2];
  uint32_t mo[4] = {0u, 0u, 0u, 0u};                              // the wave's CH metadata bytes of the lane's 4 features
#pragma unroll
  for (int c = 0; c < CH; c++) {
    uint32_t ho[4][2];
#pragma unroll
    for (int q = 0; q < 2; q++) {                                 // group of 4 tokens
      uint64_t hw[4], zw[4];                                      // a token's 4 features, 16 bits each
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const int i = 8 * c + 4 * q + t;
        const uint32_t nib = m[i] >> (4 * (g & 1)), s0 = (nib & 3u) << 4, s1 = (nib & 12u) << 2;
        hw[t] = ((uint64_t)(h[i] & 0xFFFFu) << s0) | ((uint64_t)(h[i] >> 16) << s1);
        zw[t] = ((uint64_t)(z[i] & 0xFFFFu) << s0) | ((uint64_t)(z[i] >> 16) << s1);
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        uint32_t w[4], x[4];
#pragma unroll
        for (int t = 0; t < 4; t++) { w[t] = (uint32_t)(hw[t] >> (16 * j)) & 0xFFFFu; x[t] = (uint32_t)(zw[t] >> (16 * j)) & 0xFFFFu; }
        const uint32_t nb = pick24_words(w[0], w[1], w[2], w[3], ho[j][q]);
        const uint32_t i0 = nb & 3u, i1 = nb >> 2;
        const uint32_t za = i0 == 0 ? x[0] : (i0 == 1 ? x[1] : x[2]), zb = i1 == 3 ? x[3] : (i1 == 2 ? x[2] : x[1]);
        zo[c][j][q] = za | (zb << 16);
        mo[j] |= nb << (8 * c + 4 * q);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; j++) *reinterpret_cast<u32x2*>(sV + (64 * j + lane) * PITCH + 8 * (CH * wave + c)) = u32x2{ho[j][0], ho[j][1]};
  }
#pragma unroll
  for (int j = 0; j < 4; j++) {
    static_assert(CH == 4, "a wave's metadata bytes of a feature are one word");
    sM[(64 * j + lane) * CH + wave] = mo[j];
  }
  __syncthreads();
  constexpr int PIECES = ROWB / 16;                               // 16-byte pieces of a row
  auto flush = [&](uint8_t* out) {
#pragma unroll
    for (int i = 0; i < PIECES; i++) {
      const int item = tid + 256 * i, r = item / PIECES, pc = item % PIECES, f = f0 + 4 * (r & 63) + (r >> 6);
      if (f < F) st_stream(reinterpret_cast<u32x4*>(out + (size_t)f * T + t0 + 16 * pc), *reinterpret_cast<const u32x4*>(sV + r * PITCH + 16 * pc));
    }
  };
  flush(Hc_t);
  {
    const int f = f0 + 4 * (tid & 63) + (tid >> 6);
    uint8_t* out = meta_t + (size_t)f * (T >> 3) + (t0 >> 3);
    if (f < F) *reinterpret_cast<u32x4*>(out) = *reinterpret_cast<const u32x4*>(sM + tid * CH);
  }
  if (!has_z) return;                                             // (a kernel argument: all work items or none)
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CH; c++)
#pragma unroll
    for (int j = 0; j < 4; j++) *reinterpret_cast<u32x2*>(sV + (64 * j + lane) * PITCH + 8 * (CH * wave + c)) = u32x2{zo[c][j][0], zo[c][j][1]};
  __syncthreads();
  flush(dZc_t);
}

int launch_featurewise24_rows(const void* Hc, const uint8_t* meta, const void* dZc, int T, int F, void* Hc_t, uint8_t* meta_t, void* dZc_t, hipStream_t s) {
  if (featurewise_small(T, F)) {
    hipLaunchKernelGGL(featurewise24_kernel<false>, dim3(F / FW_FEAT, T / FW_TOK), dim3(256), 0, s, static_cast<const uint16_t*>(Hc), meta,
                       static_cast<const uint16_t*>(dZc), T, F, 1, static_cast<uint16_t*>(Hc_t), meta_t, static_cast<uint16_t*>(dZc_t),
                       nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr);
    return (int)hipGetLastError();
  }
  hipLaunchKernelGGL(featurewise24_rows_kernel, dim3((F + 255) / 256, T / FWR_TOK), dim3(256), 0, s, static_cast<const uint32_t*>(Hc), meta, static_cast<const uint32_t*>(dZc),
                     T, F, static_cast<uint8_t*>(Hc_t), meta_t, static_cast<uint8_t*>(dZc_t));
  return (int)hipGetLastError();
}

int launch_featurewise24(const void* Hc, const uint8_t* meta, const void* dZc, int T, int F,
                         void* Hc_t, uint8_t* meta_t, void* dZc_t, unsigned long long* tele, hipStream_t s) {
  dim3 grid(F / FW_FEAT, T / FW_TOK);
  auto kern = fw_keep(T, F) ? featurewise24_kernel<true, false, true> : featurewise24_kernel<true>;
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, static_cast<const uint16_t*>(Hc), meta,
                     static_cast<const uint16_t*>(dZc), T, F, 1, static_cast<uint16_t*>(Hc_t), meta_t, static_cast<uint16_t*>(dZc_t),
                     nullptr, 0, nullptr, nullptr, tele, nullptr, nullptr);
  return (int)hipGetLastError();
}

// the same (panel form) with the largest stored magnitude word of every output row: hmax, zmax [F], zeroed by the caller
int launch_featurewise24_rowmax(const void* Hc, const uint8_t* meta, const void* dZc, int T, int F, void* Hc_t, uint8_t* meta_t, void* dZc_t,
                                uint32_t* hmax, uint32_t* zmax, hipStream_t s) {
  dim3 grid(F / FW_FEAT, T / FW_TOK);
  auto kern = fw_keep(T, F) ? featurewise24_kernel<true, false, true> : featurewise24_kernel<true>;
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, static_cast<const uint16_t*>(Hc), meta,
                     static_cast<const uint16_t*>(dZc), T, F, 1, static_cast<uint16_t*>(Hc_t), meta_t, static_cast<uint16_t*>(dZc_t),
                     nullptr, 0, nullptr, nullptr, nullptr, hmax, zmax);
  return (int)hipGetLastError();
}

int launch_featurewise24_split(const void* Hc, const uint8_t* meta, const void* dZc, int T, int F, const int* row_of_feat, int n_sparse,
                               void* Hc_t, uint8_t* meta_t, void* dZc_t, void* Hdn_t, void* dZdn_t, unsigned long long* tele,
                               uint32_t* hmax, uint32_t* zmax, hipStream_t s) {
  const int tiles = fw_tiles(T, F, hmax != nullptr);
  dim3 grid(F / FW_FEAT, T / (FW_TOK * tiles));
  auto kern = fw_keep(T, F) ? featurewise24_kernel<true, true, true> : featurewise24_kernel<true, true>;
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, static_cast<const uint16_t*>(Hc), meta,
                     static_cast<const uint16_t*>(dZc), T, F, tiles, static_cast<uint16_t*>(Hc_t), meta_t, static_cast<uint16_t*>(dZc_t),
                     row_of_feat, n_sparse, static_cast<uint16_t*>(Hdn_t), static_cast<uint16_t*>(dZdn_t), tele, hmax, zmax);
  return (int)hipGetLastError();
}

// Feature partition of the split weight-gradient GEMMs (Sec. 2, "Optimization 1", where the paper sorts the features by their statistic).
// Only the set matters, so no sort: the threshold count c* = the smallest c with #{nnz > c} <= n_dense is found with a histogram of
// the counts' top 11 bits, summed from the top, and one of the remaining bits inside the bin that c* falls into; every feature above
// c* is dense, and of those equal to it the first (n_dense - #above) by index.  Sparse features become rows 0 .. F - n_dense - 1,
// dense ones the rows after, both in ascending feature order.  One workgroup of 1024; F <= 2^20 (beyond 32768 features the counts
// stay in global memory).  What bounds it is the chain of block-wide steps, each a few hundred cycles whatever it adds up: three or
// four here against one for each bit of the token count and three more when c* was found by bisection (F = 8192, T = 8192: 23.7 us
// with bisection, 14.6 now).
// In LDS count f sits at word f + f / 32: the ranking passes give every thread a run of consecutive features, and without the
// padding the lanes' runs would start a multiple of 32 words apart, all in two banks.  The rows are first written over the counts
// in LDS and leave in feature order, so that the stores to row_of_feat are whole lines and those to feat_of_row nearly so.
constexpr int PART_LDS_FEATS = 32768, PART_BINS = 2048;   // one workgroup of 1024: two bins a thread
// In a launch with the quantisation of dZ, whose workgroups get the LDS of the counts too: two of them a CU up to here, one beyond it (not tried).  Apart, together,
// whole row-wise steps (us, T D F): 256 512 2048 60.1, 57.8; 1280 768 3072 90.0, 86.6; 8192 2048 8192 720, 711; 512 3072 12288 277, 274; 4096 3072 12288 813, 803;
// 512 4096 16384 421, 417; 4096 4096 16384 1221, 1211; 16384 4096 16384 4215, 4210.
constexpr int PART_SHARED_FEATS = 16384;
__device__ __forceinline__ int part_slot(int f) { return f + (f >> 5); }

// (a workgroup of 1024; s_nnz: F counts if they fit)
template <bool IN_LDS>
__device__ __forceinline__ void split_partition(uint32_t* s_nnz, const uint32_t* __restrict__ nnz_g, int F, int n_dense, uint32_t max_count,
                                                int* __restrict__ row_of_feat, int* __restrict__ feat_of_row) {
  __shared__ uint32_t s_part[16];
  __shared__ int s_bin, s_above;
  __shared__ uint32_t s_hist[PART_BINS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr bool in_lds = IN_LDS;
  if (in_lds) for (int f = tid; f < F; f += 1024) s_nnz[part_slot(f)] = min(nnz_g[f], max_count);
  auto nnz = [&](int f) { return in_lds ? s_nnz[part_slot(f)] : min(nnz_g[f], max_count); };   // every count indexes the histogram
  // block-wide exclusive prefix over threads of one word per thread (wave shuffles + 16 partials in LDS)
  auto block_scan = [&](uint32_t v) {
    uint32_t incl = v;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)incl, st, 64);
      if (lane >= st) incl += o;
    }
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    uint32_t before = 0u;
#pragma unroll
    for (int w = 0; w < 16; w++) before += w < wave ? s_part[w] : 0u;
    __syncthreads();
    return before + incl - v;
  };
  // the bin in which the number of features above it passes n_dense, with `base` of them above all bins, and how many are above the bin:
  // thread t adds up bins 2047 - 2 t and 2046 - 2 t, and exactly one thread finds it (more than n_dense features in all)
  auto find_bin = [&](int base, int& bin, int& above) {
    __syncthreads();
    const int top = PART_BINS - 1 - 2 * tid, h0 = (int)s_hist[top], h1 = (int)s_hist[top - 1];
    const int a0 = base + (int)block_scan((uint32_t)(h0 + h1)), a1 = a0 + h0;
    if (a0 <= n_dense && a1 > n_dense) { s_bin = top; s_above = a0; }
    if (a1 <= n_dense && a1 + h1 > n_dense) { s_bin = top - 1; s_above = a1; }
    __syncthreads();
    bin = s_bin; above = s_above;
  };
  // no count exceeds max_count (the number of tokens, at most 2^20), so at most 10 bits are left below the first histogram
  const int bits = 32 - __clz((int)max_count), shift = bits > 11 ? bits - 11 : 0;
  s_hist[tid] = s_hist[tid + 1024] = 0u;
  __syncthreads();
  for (int f = tid; f < F; f += 1024) atomicAdd(&s_hist[nnz(f) >> shift], 1u);
  int bin, n_above;
  find_bin(0, bin, n_above);
  uint32_t cstar = (uint32_t)bin;
  if (shift) {
    s_hist[tid] = s_hist[tid + 1024] = 0u;
    __syncthreads();
    for (int f = tid; f < F; f += 1024) if ((int)(nnz(f) >> shift) == bin) atomicAdd(&s_hist[nnz(f) & ((1u << shift) - 1u)], 1u);
    int low;
    find_bin(n_above, low, n_above);
    cstar = ((uint32_t)bin << shift) | (uint32_t)low;
  }
  // consecutive features per thread from here on, so that ranks follow the feature index
  const int per = (F + 1023) / 1024;
  const int f_lo = min(tid * per, F), f_hi = min(f_lo + per, F);
  int above = 0, equal = 0;
  for (int f = f_lo; f < f_hi; f++) { above += nnz(f) > cstar; equal += nnz(f) == cstar; }
  const int take_eq = n_dense - n_above;             // how many of the features equal to c* become dense (by index)
  int eq_before, above_before;
  if constexpr (in_lds) {                            // at most 32768 features: both prefixes fit one word
    static_assert(PART_LDS_FEATS < 65536, "two 16-bit prefixes");
    const uint32_t both = block_scan((uint32_t)above | ((uint32_t)equal << 16));
    above_before = (int)(both & 0xFFFFu); eq_before = (int)(both >> 16);
  } else {
    above_before = (int)block_scan((uint32_t)above);
    eq_before = (int)block_scan((uint32_t)equal);
  }
  const int d_before = above_before + min(eq_before, take_eq);
  const int n_sparse = F - n_dense;
  int e = eq_before, dpos = d_before;
  for (int f = f_lo; f < f_hi; f++) {
    bool d = nnz(f) > cstar || (nnz(f) == cstar && e < take_eq);
    e += nnz(f) == cstar;
    int row = d ? n_sparse + dpos : f - dpos;
    dpos += d;
    if (in_lds) s_nnz[part_slot(f)] = (uint32_t)row;   // the thread's own slot: its count is not needed again
    else { row_of_feat[f] = row; feat_of_row[row] = f; }
  }
  if (in_lds) {
    __syncthreads();
    for (int f = tid; f < F; f += 1024) {
      int row = (int)s_nnz[part_slot(f)];
      row_of_feat[f] = row;
      feat_of_row[row] = f;
    }
  }
}

template <bool IN_LDS>
__global__ void __launch_bounds__(1024) split_partition_kernel(const uint32_t* __restrict__ nnz, int F, int n_dense, uint32_t max_count,
                                                               int* __restrict__ row_of_feat, int* __restrict__ feat_of_row) {
  extern __shared__ uint32_t s_nnz[];
  split_partition<IN_LDS>(s_nnz, nnz, F, n_dense, max_count, row_of_feat, feat_of_row);
}

int launch_split_partition(const uint32_t* nnz, int F, int n_dense, int max_count, int* row_of_feat, int* feat_of_row, hipStream_t s) {
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (F > PART_LDS_FEATS) {
    hipLaunchKernelGGL(split_partition_kernel<false>, dim3(1), dim3(1024), 0, s, nnz, F, n_dense, (uint32_t)max_count, row_of_feat, feat_of_row);
    return (int)hipGetLastError();
  }
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(split_partition_kernel<true>), 4 * (PART_LDS_FEATS + PART_LDS_FEATS / 32), configured)) return rc;
  hipLaunchKernelGGL(split_partition_kernel<true>, dim3(1), dim3(1024), 4 * ((size_t)F + (size_t)F / 32), s, nnz, F, n_dense, (uint32_t)max_count,
                     row_of_feat, feat_of_row);
  return (int)hipGetLastError();
}

// Panel form -> row-major.  The operand has `rows` rows and `npanels` pieces of PIECE bytes per row (64: stored
// values, 8 / 16: bf16 / fp8 metadata); each work item moves 8 bytes.
template <int PIECE>
__global__ void __launch_bounds__(256) unpanel_kernel(const u32x2* __restrict__ src, int rows, int npanels, u32x2* __restrict__ dst) {
  constexpr int W = PIECE / 8;                       // 8-byte words per piece
  size_t n = (size_t)rows * npanels * W;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    size_t pc = i / W;                               // row-major piece number: r * npanels + kp
    int w = (int)(i % W);
    int r = (int)(pc / npanels), kp = (int)(pc % npanels);
    dst[i] = src[a24_piece(r, kp, npanels) * W + w];
  }
}

// Clears n 32-bit words.  A kernel rather than a memset node, so that a caller may record the sequence into a HIP graph.
__global__ void __launch_bounds__(256) zero32_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

int launch_zero32(uint32_t* p, size_t n, hipStream_t s) {
  if (n == 0) return 0;
  size_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(zero32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  return (int)hipGetLastError();
}

int launch_unpanel(const void* src, int rows, int npanels, int piece_bytes, void* dst, hipStream_t s) {
  size_t n = (size_t)rows * npanels * (piece_bytes / 8);
  size_t blocks = (n + 255) / 256;
  if (blocks > 0x7FFFFFFF) blocks = 0x7FFFFFFF;   // one work item per thread: the fastest shape for a streaming kernel here
  auto kern = piece_bytes == 64 ? unpanel_kernel<64> : (piece_bytes == 16 ? unpanel_kernel<16> : unpanel_kernel<8>);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const u32x2*>(src), rows, npanels, static_cast<u32x2*>(dst));
  return (int)hipGetLastError();
}

// out[c][r] = in[r][c] for a bf16 matrix [R][C], R a multiple of 64 and C of 128.  One workgroup per tile of 64 rows x 128
// columns: a work item reads 16 bytes of each of 2 consecutive rows (a row's 256 bytes are read by 16 neighbouring work items),
// pairs the rows' elements column by column with byte permutes, and writes 8 dwords -- 2 elements along r of 8 transposed rows --
// into an LDS image [c][r] (pitch 33 dwords; a row's dwords are rotated by 4 for the second 64 columns, which spreads a wave's
// writes over all banks); then 16 bytes of a transposed row per work item go out: 128 rows x 128 bytes.  (One 64 x 64 tile per
// workgroup with element-wise LDS scatter, the first version, moved 4.3-4.9 TB/s.)
// OUT_FORM: 0 row-major; 1 the dense panel form of gemm_core.hpp (64-byte pieces of 32 k, K = R), as A operands take it;
// 2 the B panel form (the same with row n of every block of 256 at b_panel_pos(n)).
// in_panel (optional): a copy of the input itself in panel form (K = C), made in the same pass; in_panel_b: in the B form.
// in_rowmap (optional): input row r is read from memory row in_rowmap[r] (token permutation).
// Two transposes may share a launch (a step needs them in pairs, both weights or both activations: at small sizes a launch costs as much
// as its work, T = 1280 D = 768 F = 3072: 5.2 + 5.0 -> 6.4 us): workgroups [0, n_first) take the first job.
constexpr int TR_COLS = 128, TR_LDW = 33;
struct TransposeJob {
  const void* in; int R, C; void* out; void* in_panel; int in_panel_b; const int* in_rowmap;
};

template <int OUT_FORM>
__device__ __forceinline__ void transpose_tile(const TransposeJob& job, int tile, uint32_t* sT) {
  const uint16_t* __restrict__ in = static_cast<const uint16_t*>(job.in);
  uint16_t* __restrict__ out = static_cast<uint16_t*>(job.out);
  uint16_t* __restrict__ in_panel = static_cast<uint16_t*>(job.in_panel);
  const int* __restrict__ in_rowmap = job.in_rowmap;
  const int R = job.R, C = job.C, in_panel_b = job.in_panel_b;
  const int nc = C / TR_COLS, r0 = (tile / nc) * 64, c0 = (tile % nc) * TR_COLS;
  const int tid = threadIdx.x;
  const int ch = tid & 15;                   // 16-byte chunk of a row segment: columns 8 ch .. 8 ch + 7 of the tile
  const int rot = ch >> 3;                   // (c >> 6) of every column this work item holds
  u32x4 v[2][2];
#pragma unroll
  for (int pass = 0; pass < 2; pass++)
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int r = r0 + 2 * ((tid >> 4) + 16 * pass) + i;
      const size_t src_row = in_rowmap ? (size_t)in_rowmap[r] : (size_t)r;
      v[pass][i] = ld_stream(reinterpret_cast<const u32x4*>(in + src_row * C + c0 + 8 * ch));
    }
#pragma unroll
  for (int pass = 0; pass < 2; pass++) {
    const int rp = (tid >> 4) + 16 * pass;   // pair of rows 2 rp, 2 rp + 1 of the tile
    if (in_panel) {
      const int c = c0 + 8 * ch;
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const int r = r0 + 2 * rp + i;
        const int prow = in_panel_b ? b_panel_pos(r) : r;
        st_keep(reinterpret_cast<u32x4*>(in_panel + a24_piece(prow, c >> 5, C >> 5) * 32 + (c & 31)), v[pass][i]);
      }
    }
    uint32_t* dst = sT + ((rp + 4 * rot) & 31);
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int c = 8 * ch + 2 * g;
      dst[c * TR_LDW] = __builtin_amdgcn_perm(v[pass][1][g], v[pass][0][g], 0x05040100u);         // column c: rows 2 rp, 2 rp + 1
      dst[(c + 1) * TR_LDW] = __builtin_amdgcn_perm(v[pass][1][g], v[pass][0][g], 0x07060302u);   // column c + 1
    }
  }
  __syncthreads();
  const int q = tid & 7;                     // 16-byte chunk of a transposed row: 8 of the tile's 64 rows r
#pragma unroll
  for (int p = 0; p < TR_COLS / 32; p++) {
    const int c = (tid >> 3) + 32 * p;       // transposed row
    const uint32_t* src = sT + c * TR_LDW + 4 * ((q + (c >> 6)) & 7);
    u32x4 o = {src[0], src[1], src[2], src[3]};
    const int r = r0 + 8 * q;
    if constexpr (OUT_FORM == 1) st_keep(reinterpret_cast<u32x4*>(out + a24_piece(c0 + c, r >> 5, R >> 5) * 32 + (r & 31)), o);
    else if constexpr (OUT_FORM == 2) st_keep(reinterpret_cast<u32x4*>(out + a24_piece(b_panel_pos(c0 + c), r >> 5, R >> 5) * 32 + (r & 31)), o);
    else st_stream(reinterpret_cast<u32x4*>(out + (size_t)(c0 + c) * R + r), o);
  }
}

template <int FORM_A, int FORM_B>
__global__ void __launch_bounds__(256) transpose_kernel(TransposeJob a, int n_first, TransposeJob b) {
  __shared__ uint32_t sT[TR_COLS * TR_LDW];
  const int bid = blockIdx.x;
  if (bid < n_first) transpose_tile<FORM_A>(a, bid, sT);
  else transpose_tile<FORM_B>(b, bid - n_first, sT);
}

static int transpose_tiles(const TransposeJob& j) { return (j.C / TR_COLS) * (j.R / 64); }

int launch_transpose(const void* in, int R, int C, void* out, hipStream_t s) {
  const TransposeJob j{in, R, C, out, nullptr, 0, nullptr};
  hipLaunchKernelGGL((transpose_kernel<0, 0>), dim3((unsigned)transpose_tiles(j)), dim3(256), 0, s, j, transpose_tiles(j), j);
  return (int)hipGetLastError();
}

int launch_transpose_weights(const void* W1, const void* W2, int D, int F, void* W1t, void* W1p, void* W2t, void* W2p, hipStream_t s) {
  const TransposeJob a{W1, D, F, W1t, W1p, 1, nullptr}, b{W2, F, D, W2t, W2p, 0, nullptr};
  hipLaunchKernelGGL((transpose_kernel<1, 2>), dim3((unsigned)(transpose_tiles(a) + transpose_tiles(b))), dim3(256), 0, s, a, transpose_tiles(a), b);
  return (int)hipGetLastError();
}

int launch_transpose_acts(const void* dY, const void* X, int T, int D, void* dYt, void* Xt, const int* rowmap, hipStream_t s) {
  const TransposeJob a{dY, T, D, dYt, nullptr, 0, rowmap}, b{X, T, D, Xt, nullptr, 0, rowmap};
  hipLaunchKernelGGL((transpose_kernel<2, 2>), dim3((unsigned)(transpose_tiles(a) + transpose_tiles(b))), dim3(256), 0, s, a, transpose_tiles(a), b);
  return (int)hipGetLastError();
}

// Byte-matrix transpose (fp8 operands): out[c][r] = in[r][c], in [R][C], R a multiple of 64 and C of 256.  One workgroup per
// tile of 64 rows x 256 columns: a work item reads 16 bytes of each of 4 consecutive rows (a row's 256 bytes are read by 16
// neighbouring work items), transposes its four 4 x 4 byte blocks in registers with byte permutes, and writes 16 dwords -- 4
// bytes along r of 16 transposed rows -- into an LDS image [c][r] (pitch 68 bytes; a row's 16 dwords are rotated by 4 for every 64
// columns, which spreads a wave's writes over all banks); then 16 bytes of a transposed row per work item go out: 256 rows x
// 64 bytes, one contiguous 16 KiB run in the panel forms.  (One 64 x 64 tile per workgroup with byte-wise LDS scatter, the
// first version, moved 3.8 TB/s.)  OUT_FORM: 0 row-major, 1 dense panel form (64-byte pieces of 64 k, K = R), 2 the B panel form.
// in_panel (optional): a copy of the input itself in panel form (K = C, 64-byte pieces), made in the same pass; in the
// B form if in_panel_b.  in_rowmap (optional): input row r is read from memory row in_rowmap[r] (token permutation).
constexpr int T8_COLS = 256, T8_LD = 68;

template <int OUT_FORM>
__device__ __forceinline__ void transpose8_tile(const TransposeJob& job, int tile, uint8_t* sT) {
  const uint8_t* __restrict__ in = static_cast<const uint8_t*>(job.in);
  uint8_t* __restrict__ out = static_cast<uint8_t*>(job.out);
  uint8_t* __restrict__ in_panel = static_cast<uint8_t*>(job.in_panel);
  const int* __restrict__ in_rowmap = job.in_rowmap;
  const int R = job.R, C = job.C, in_panel_b = job.in_panel_b;
  const int nc = C / T8_COLS, r0 = (tile / nc) * 64, c0 = (tile % nc) * T8_COLS;
  const int tid = threadIdx.x;
  const int ch = tid & 15, rq = tid >> 4;    // 16-byte column chunk of the tile; group of 4 rows
  u32x4 v[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = r0 + 4 * rq + i;
    const size_t src_row = in_rowmap ? (size_t)in_rowmap[r] : (size_t)r;
    v[i] = ld_stream(reinterpret_cast<const u32x4*>(in + src_row * C + c0 + 16 * ch));
  }
  if (in_panel) {
    const int c = c0 + 16 * ch;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int r = r0 + 4 * rq + i;
      const int prow = in_panel_b ? b_panel_pos(r) : r;
      st_keep(reinterpret_cast<u32x4*>(in_panel + a24_piece(prow, c >> 6, C >> 6) * 64 + (c & 63)), v[i]);
    }
  }
  const int rot = ch >> 2;                   // (c >> 6) & 3 of every column this work item holds
  uint32_t* dst = reinterpret_cast<uint32_t*>(sT) + ((rq + 4 * rot) & 15);
#pragma unroll
  for (int g = 0; g < 4; g++) {
    // rows i = 0..3, bytes j = 0..3 of column group g  ->  for every j the bytes of rows 0..3
    const uint32_t lo01 = __builtin_amdgcn_perm(v[1][g], v[0][g], 0x05010400u), hi01 = __builtin_amdgcn_perm(v[1][g], v[0][g], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(v[3][g], v[2][g], 0x05010400u), hi23 = __builtin_amdgcn_perm(v[3][g], v[2][g], 0x07030602u);
    const int c = 16 * ch + 4 * g;
    dst[(c + 0) * (T8_LD / 4)] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    dst[(c + 1) * (T8_LD / 4)] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    dst[(c + 2) * (T8_LD / 4)] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    dst[(c + 3) * (T8_LD / 4)] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
  __syncthreads();
  const int q = tid & 3;                     // 16-byte chunk of a transposed row (16 of the tile's 64 rows r)
#pragma unroll
  for (int p = 0; p < T8_COLS / 64; p++) {
    const int c = (tid >> 2) + 64 * p;       // transposed row; (c >> 6) & 3 == p
    const uint32_t* src = reinterpret_cast<const uint32_t*>(sT) + c * (T8_LD / 4) + 4 * ((q + p) & 3);
    u32x4 o = {src[0], src[1], src[2], src[3]};
    const int r = r0 + 16 * q;
    if constexpr (OUT_FORM == 1) st_keep(reinterpret_cast<u32x4*>(out + a24_piece(c0 + c, r >> 6, R >> 6) * 64 + (r & 63)), o);
    else if constexpr (OUT_FORM == 2) st_keep(reinterpret_cast<u32x4*>(out + a24_piece(b_panel_pos(c0 + c), r >> 6, R >> 6) * 64 + (r & 63)), o);
    else st_stream(reinterpret_cast<u32x4*>(out + (size_t)(c0 + c) * R + r), o);
  }
}

// What a forward or backward needs done before its first GEMM, in one launch (each of these passes by itself is about as long as its
// launch: T = 8192 D = 2048 F = 8192, token permutation and split, 4 + 6 launches of 4.7-9 us became 2):
//   copies: byte matrices [R][C] (row-major, C a multiple of 64) into the dense fp8 panel form (64-byte pieces of 64 k, K = C) as A
//     operands take it, or, b_form, into the B panel form (row n of every block of 256 at b_panel_pos(n)); row r is taken from memory row
//     rowmap[r] if one is given (token permutation); 16 bytes per work item;
//   zero: 32-bit words cleared (row maxima, counts);
//   gather: dst[i] = src[map[i]], a per-token scale vector brought into the order of a token permutation.
// No streaming hints: what is copied here is read again, the copy right away and the input by a later pass of the step (weights with the hints on loads and
// stores: the down-projection behind them at T 1024 D 1024 F 4096 20.8 us against 15.2, the copies at T = F = 16384 D 4096 100 against 83; X with the
// hint on its loads alone: fp8 step at T 4096 D 2048 F 8192 325 against 322.6).
__device__ __forceinline__ void panelise8_block(const PaneliseJobs& jobs, unsigned bid) {
#pragma unroll
  for (int j = 0; j < PaneliseJobs::COPIES; j++) {
    const PaneliseJobs::Copy& cp = jobs.copy[j];
    if (bid < cp.blocks) {
      const unsigned per_row = (unsigned)cp.C >> 4;
      const size_t i = (size_t)bid * 256 + threadIdx.x, n = (size_t)cp.R * per_row;
      if (i >= n) return;
      const unsigned rq = n >> 32 ? (unsigned)(i / per_row) : (unsigned)i / per_row;   // (the long division only where it has to be)
      const int r = (int)rq, cq = (int)((unsigned)i - rq * per_row), c = cq << 4;
      const int prow = cp.b_form ? b_panel_pos(r) : r;
      const size_t src = cp.rowmap ? (size_t)cp.rowmap[r] * per_row + cq : i;
      u32x4* out = reinterpret_cast<u32x4*>(static_cast<uint8_t*>(cp.out) + a24_piece(prow, c >> 6, cp.C >> 6) * 64 + (c & 63));
      const u32x4* in = static_cast<const u32x4*>(cp.in) + src;
      *out = *in;
      return;
    }
    bid -= cp.blocks;
  }
  int i = (int)(bid * 256 + threadIdx.x);
#pragma unroll
  for (int j = 0; j < PaneliseJobs::ZEROS; j++) {
    if (i < jobs.zero_n[j]) { jobs.zero[j][i] = 0u; return; }
    i -= jobs.zero_n[j];
  }
  if (i < jobs.gather_n) jobs.gather_dst[i] = jobs.gather_src[jobs.gather_map[i]];
}
__global__ void __launch_bounds__(256) panelise8_kernel(PaneliseJobs jobs) { panelise8_block(jobs, blockIdx.x); }

struct NoJobs {};
template <int FORM_A, int FORM_B, class Jobs>
__global__ void __launch_bounds__(256) transpose8_kernel(TransposeJob a, int n_first, TransposeJob b, int n_tiles, Jobs jobs) {
  __shared__ __attribute__((aligned(16))) uint8_t sT[T8_COLS * T8_LD];
  const int bid = blockIdx.x;
  if constexpr (std::is_same_v<Jobs, PaneliseJobs>) {
    if (bid >= n_tiles) { panelise8_block(jobs, (unsigned)(bid - n_tiles)); return; }
  }
  if (bid < n_first) transpose8_tile<FORM_A>(a, bid, sT);
  else transpose8_tile<FORM_B>(b, bid - n_first, sT);
}

static int transpose8_tiles(const TransposeJob& j) { return (j.C / T8_COLS) * (j.R / 64); }

static unsigned panelise8_blocks(const PaneliseJobs& jobs) {
  unsigned blocks = 0;
  int side = jobs.gather_n;
  for (const auto& c : jobs.copy) blocks += c.blocks;
  for (int n : jobs.zero_n) side += n;
  return blocks + (unsigned)((side + 255) / 256);
}
template <int FORM_A, int FORM_B>
static int launch_transpose8(const TransposeJob& a, const TransposeJob& b, const PaneliseJobs* jobs, hipStream_t s) {
  const int na = transpose8_tiles(a), n = na + transpose8_tiles(b);
  if (jobs) hipLaunchKernelGGL((transpose8_kernel<FORM_A, FORM_B, PaneliseJobs>), dim3((unsigned)n + panelise8_blocks(*jobs)), dim3(256), 0, s, a, na, b, n, *jobs);
  else hipLaunchKernelGGL((transpose8_kernel<FORM_A, FORM_B, NoJobs>), dim3((unsigned)n), dim3(256), 0, s, a, na, b, n, NoJobs());
  return (int)hipGetLastError();
}

int launch_transpose8_weights(const void* W1, const void* W2, int D, int F, void* W1t, void* W1p, void* W2t, void* W2p, const PaneliseJobs* jobs, hipStream_t s) {
  return launch_transpose8<1, 2>({W1, D, F, W1t, W1p, 1, nullptr}, {W2, F, D, W2t, W2p, 0, nullptr}, jobs, s);
}

int launch_transpose8_acts(const void* dY, const void* X, int T, int D, void* dYt, void* dYp, void* Xt, const int* rowmap, const PaneliseJobs* jobs, hipStream_t s) {
  return launch_transpose8<2, 2>({dY, T, D, dYt, dYp, 1, rowmap}, {X, T, D, Xt, nullptr, 0, rowmap}, jobs, s);
}

int launch_panelise8(const PaneliseJobs& jobs, hipStream_t s) {
  hipLaunchKernelGGL(panelise8_kernel, dim3(panelise8_blocks(jobs)), dim3(256), 0, s, jobs);
  return (int)hipGetLastError();
}

// Feature-wise 2:4 on top of the token-wise mask for the fp8 operands (Sec. 2, last paragraph; the FP8 side of the fused
// backward pointwise step).  Everything is in the fp8 panel form: input pieces = 128 hidden features of one token (64
// stored e4m3 bytes + 16 metadata bytes), output pieces = 128 tokens of one feature.  The picks are made on the stored
// codes of the activation (sign bit cleared, as integers; ties -> lower token); dZ is gathered at the same positions.
// One workgroup handles 128 tokens x 128 features: it reads 128 consecutive input pieces of each tensor (8 KiB + 2 KiB
// runs), spreads them out in LDS, and every work item then takes one feature and 16 consecutive tokens (four groups):
// 8 stored bytes and 2 metadata bytes of an output piece.
constexpr int FW8_TOK = 128, FW8_FEAT = 128, FW8_LD = FW8_FEAT + 4;

__device__ __forceinline__ uint32_t pick24_codes(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t& i0, uint32_t& i1) {
  // keys ((magnitude << 2) | (3 - i)): distinct, ordered by (magnitude, then lower index first)
  uint32_t k0 = ((w0 & 0x7Fu) << 2) | 3u, k1 = ((w1 & 0x7Fu) << 2) | 2u, k2 = ((w2 & 0x7Fu) << 2) | 1u, k3 = (w3 & 0x7Fu) << 2;
  uint32_t kf, ks;
  uint32_t nib = pick24_keys(k0, k1, k2, k3, kf, ks);
  i0 = nib & 3u; i1 = nib >> 2;
  return nib;
}

__global__ void __launch_bounds__(256) featurewise24_f8_kernel(const uint8_t* __restrict__ Hc8, const uint8_t* __restrict__ meta,
                                                               const uint8_t* __restrict__ dZc8, int T, int F,
                                                               uint8_t* __restrict__ Hc8_t, uint8_t* __restrict__ meta_t,
                                                               uint8_t* __restrict__ dZc8_t) {
  __shared__ __attribute__((aligned(16))) uint8_t sH[FW8_TOK * FW8_LD];
  __shared__ __attribute__((aligned(16))) uint8_t sZ[FW8_TOK * FW8_LD];
  const int f0 = blockIdx.x * FW8_FEAT, t0 = blockIdx.y * FW8_TOK;
  const int tid = threadIdx.x;
  const bool has_z = dZc8 != nullptr;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    int item = tid + 256 * i;
    int tok = item >> 2, ch = item & 3;              // 16 stored bytes = 8 groups = 32 features
    size_t piece = a24_piece(t0 + tok, f0 >> 7, F >> 7);
    u32x4 hv = ld_stream(reinterpret_cast<const u32x4*>(Hc8 + piece * 64 + 16 * ch));
    u32x4 zv = {0u, 0u, 0u, 0u};
    if (has_z) zv = ld_stream(reinterpret_cast<const u32x4*>(dZc8 + piece * 64 + 16 * ch));
    uint32_t m32 = ld_stream(reinterpret_cast<const uint32_t*>(meta + piece * 16 + 4 * ch));
#pragma unroll
    for (int g = 0; g < 8; g++) {
      uint32_t nib = (m32 >> (4 * g)) & 15u;
      uint32_t i0 = nib & 3u, i1 = nib >> 2;
      uint32_t hb = (hv[g >> 1] >> (16 * (g & 1))) & 0xFFFFu, zb = (zv[g >> 1] >> (16 * (g & 1))) & 0xFFFFu;
      // the group's four bytes as one word: kept byte 0 at position i0, kept byte 1 at position i1
      uint32_t hw = ((hb & 0xFFu) << (8 * i0)) | ((hb >> 8) << (8 * i1));
      uint32_t zw = ((zb & 0xFFu) << (8 * i0)) | ((zb >> 8) << (8 * i1));
      int o = tok * FW8_LD + 32 * ch + 4 * g;         // a multiple of 4
      *reinterpret_cast<uint32_t*>(&sH[o]) = hw;
      *reinterpret_cast<uint32_t*>(&sZ[o]) = zw;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int item = tid + 256 * i;
    int c = item & 7, f = item >> 3;                   // 16 tokens 16 c .. 16 c + 15 of feature f0 + f
    uint32_t hq[2] = {0u, 0u}, zq[2] = {0u, 0u}, mq = 0u;
#pragma unroll
    for (int g = 0; g < 4; g++) {
      uint32_t h[4], z[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        h[j] = sH[(16 * c + 4 * g + j) * FW8_LD + f];
        z[j] = sZ[(16 * c + 4 * g + j) * FW8_LD + f];
      }
      uint32_t i0, i1;
      uint32_t nib = pick24_codes(h[0], h[1], h[2], h[3], i0, i1);
      uint32_t ha = i0 == 0 ? h[0] : (i0 == 1 ? h[1] : h[2]), hb = i1 == 3 ? h[3] : (i1 == 2 ? h[2] : h[1]);
      uint32_t za = i0 == 0 ? z[0] : (i0 == 1 ? z[1] : z[2]), zb = i1 == 3 ? z[3] : (i1 == 2 ? z[2] : z[1]);
      hq[g >> 1] |= (ha | (hb << 8)) << (16 * (g & 1));
      zq[g >> 1] |= (za | (zb << 8)) << (16 * (g & 1));
      mq |= nib << (4 * g);
    }
    size_t piece = a24_piece(f0 + f, t0 >> 7, T >> 7);
    st_stream(reinterpret_cast<u32x2*>(Hc8_t + piece * 64 + 8 * c), u32x2{hq[0], hq[1]});
    if (has_z) st_stream(reinterpret_cast<u32x2*>(dZc8_t + piece * 64 + 8 * c), u32x2{zq[0], zq[1]});
    st_stream(reinterpret_cast<uint16_t*>(meta_t + piece * 16 + 2 * c), (uint16_t)mq);
  }
}

int launch_featurewise24_f8(const void* Hc8, const uint8_t* meta, const void* dZc8, int T, int F, void* Hc8_t, uint8_t* meta_t, void* dZc8_t, hipStream_t s) {
  dim3 grid(F / FW8_FEAT, T / FW8_TOK);
  hipLaunchKernelGGL(featurewise24_f8_kernel, grid, dim3(256), 0, s, static_cast<const uint8_t*>(Hc8), meta, static_cast<const uint8_t*>(dZc8),
                     T, F, static_cast<uint8_t*>(Hc8_t), meta_t, static_cast<uint8_t*>(dZc8_t));
  return (int)hipGetLastError();
}

// Row-wise fp8 quantisation of an operand in panel form (Sec. 2 describes one kernel for activation, sparsification
// and FP8 quantisation; here only the last step is left to a kernel of its own, because the scale of a token row,
// sh[t] = (largest activation of the row) / 448, is known only once the whole row exists).
// Compressed (META): bf16 kept values + metadata, 64-byte / 8-byte pieces per 64 features, become e4m3 codes + metadata, 64-byte /
// 16-byte pieces per 128 features.  Dense: bf16 pieces of 32 features become e4m3 pieces of 64.  Either way two input pieces of a
// row, one panel (256 pieces) apart, make one output piece, and sh [T] is written.
// HBM-bound (3.375 bytes per stored value compressed, 3 dense).  Four neighbouring lanes take a row's piece, 16 bytes each, so that
// a wave reads whole contiguous kilobytes; a lane's 8 codes of either input piece are exchanged with its neighbour's, so that each
// stores 16 bytes and the wave a contiguous kilobyte again.  One output piece per lane and workgroups in memory order (a
// quarter of a block of 256 rows each, then the next panel).  The stores are plain: the next kernel reads the codes.
// A launch takes one matrix or two of one kind and size (QuantJobs): the operands of one stage of a step, whose launches by themselves end one after the
// other.  The kind and the place come from the grid: found by division and a walk over the jobs they cost a workgroup that lives this short 4 us of a
// launch's 21 (T = F = 8192).
template <bool META>
__device__ __forceinline__ void quantise_rows_piece(const QuantJobs::Job& job, int np8, int j, int t, int c) {
  const u32x4* __restrict__ H16 = static_cast<const u32x4*>(job.H16);
  u32x4* __restrict__ H8 = static_cast<u32x4*>(job.H8);
  const size_t pin = a24_piece(t, 2 * j, 2 * np8), pout = a24_piece(t, j, np8);
  const u32x4 v0 = ld_stream(H16 + pin * 4 + c), v1 = ld_stream(H16 + (pin + 256) * 4 + c);
  if (META && c < 2) reinterpret_cast<u32x2*>(job.meta8)[pout * 2 + c] = ld_stream(reinterpret_cast<const u32x2*>(job.meta16) + pin + 256 * c);
  const float s = scale_of_max(job.rowmax[t]);
  if (j == 0 && c == 0) job.sh[t] = s;
  const ExactDiv d[1] = {ExactDiv(s)};
  const u32x2 q0 = quantise8(v0, d), q1 = quantise8(v1, d);
  const bool odd = c & 1;                              // even lanes store of the first input piece, odd ones of the second
  const u32x2 keep = odd ? q1 : q0, send = odd ? q0 : q1;
  const uint32_t r0 = (uint32_t)__shfl_xor((int)send[0], 1, 64), r1 = (uint32_t)__shfl_xor((int)send[1], 1, 64);
  H8[pout * 4 + 2 * odd + (c >> 1)] = odd ? u32x4{r0, r1, keep[0], keep[1]} : u32x4{keep[0], keep[1], r0, r1};
}
template <bool META>
__global__ void __launch_bounds__(256) quantise_rows_kernel(QuantJobs jobs) {
  quantise_rows_piece<META>(blockIdx.z ? jobs.job[1] : jobs.job[0], jobs.np8, (int)(blockIdx.x >> 2), (int)(blockIdx.y * 256 + 64 * (blockIdx.x & 3) + (threadIdx.x >> 2)),
                            threadIdx.x & 3);
}

int launch_quantise_rows(const QuantJobs& jobs, hipStream_t s) {
  const dim3 grid(4u * (unsigned)jobs.np8, (unsigned)(jobs.rows / 256), (unsigned)jobs.jobs);
  if (jobs.job[0].meta16) hipLaunchKernelGGL(quantise_rows_kernel<true>, grid, dim3(256), 0, s, jobs);
  else hipLaunchKernelGGL(quantise_rows_kernel<false>, grid, dim3(256), 0, s, jobs);
  return (int)hipGetLastError();
}

// One compressed matrix, with the feature partition of the split, which everything after it waits for and which keeps one workgroup busy: it runs beside the
// quantisation of dZ instead of after it (T = F = 8192, D = 2048: 10.6 us of a step).  Workgroups of 1024, as the partition's is: a whole block of 256 rows
// each; the first row of the grid is the partition's.
__global__ void __launch_bounds__(1024) quantise_rows_partition_kernel(QuantJobs jobs, const uint32_t* __restrict__ nnz, int F, int n_dense, uint32_t max_count,
                                                                       int* __restrict__ row_of_feat, int* __restrict__ feat_of_row) {
  extern __shared__ uint32_t s_nnz[];
  if (blockIdx.y == 0) {
    if (blockIdx.x == 0) split_partition<true>(s_nnz, nnz, F, n_dense, max_count, row_of_feat, feat_of_row);
    return;
  }
  quantise_rows_piece<true>(jobs.job[0], jobs.np8, (int)blockIdx.x, (int)((blockIdx.y - 1) * 256 + (threadIdx.x >> 2)), threadIdx.x & 3);
}

int launch_quantise_rows_partition(const QuantJobs& jobs, const uint32_t* nnz, int F, int n_dense, int max_count, int* row_of_feat, int* feat_of_row, hipStream_t s) {
  if (F > PART_SHARED_FEATS) {
    const int rc = launch_quantise_rows(jobs, s);
    return rc ? rc : launch_split_partition(nnz, F, n_dense, max_count, row_of_feat, feat_of_row, s);
  }
  static std::atomic<bool> configured[MAX_DEVICES] = {};
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(quantise_rows_partition_kernel), 4 * (PART_SHARED_FEATS + PART_SHARED_FEATS / 32), configured)) return rc;
  hipLaunchKernelGGL(quantise_rows_partition_kernel, dim3((unsigned)jobs.np8, 1u + (unsigned)(jobs.rows / 256)), dim3(1024), 4 * ((size_t)F + (size_t)F / 32), s, jobs, nnz,
                     F, n_dense, (uint32_t)max_count, row_of_feat, feat_of_row);
  return (int)hipGetLastError();
}

// Largest magnitude word of every row of a bf16 matrix [R][C] in dense panel form (64-byte pieces of 32 k): rmax[r] is raised
// with an atomic (the caller zeroes it).  A workgroup takes one block of 256 rows (one row per work item, so its loads of a
// panel are one contiguous 16 KiB run) and a slice of the panels.
constexpr int ROWMAX_SLICES = 32;
__global__ void __launch_bounds__(256) rowmax_dense_kernel(const u32x4* __restrict__ X16, int R, int C, uint32_t* __restrict__ rmax) {
  const int np = C >> 5;
  const int per = (np + ROWMAX_SLICES - 1) / ROWMAX_SLICES;
  const int k0 = blockIdx.y * per, k1 = min(np, k0 + per);
  const size_t base = (size_t)blockIdx.x * np * 256 + threadIdx.x;
  uint32_t m = 0u;
  for (int kp = k0; kp < k1; kp++) {
    const u32x4* p = X16 + (base + (size_t)kp * 256) * 4;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      u32x4 v = ld_stream(p + c);
#pragma unroll
      for (int d = 0; d < 4; d++) m = max(m, max(v[d] & 0x7FFFu, (v[d] >> 16) & 0x7FFFu));
    }
  }
  if (m) atomicMax(rmax + blockIdx.x * 256 + threadIdx.x, m);
}

int launch_rowmax_dense(const void* X16, int R, int C, uint32_t* rmax, hipStream_t s) {
  hipLaunchKernelGGL(rowmax_dense_kernel, dim3(R / 256, ROWMAX_SLICES), dim3(256), 0, s, static_cast<const u32x4*>(X16), R, C, rmax);
  return (int)hipGetLastError();
}

// Row-wise / column-wise e4m3 quantisation of a bf16 matrix X [R][C] (the operands a caller hands to the row-wise-scaled
// GEMMs; Sec. 2 of the paper: FP8 row-wise scaling).  scale = (largest magnitude of the row or column) / 448, 1 if that is
// zero; codes = e4m3(x / scale), row-major [R][C].

// Per row, the whole row held in registers between the maximum and the quantisation: LANES work items per row (a wave, or the workgroup
// for rows beyond 4096 values), up to NV 16-byte pieces each, all requested before the first is used.  KEEP: without the streaming hint, for a matrix
// that the last-level cache (256 MB) holds and that is quantised per column as well (rows and columns in either order, with the hint / without: 8192 x
// 2048 34.5, 33.2 us; 8192 x 4096 55.4, 52.7; 8192 x 6144 73.9, 70.1; 12288 x 4096 78.3, 76.3; 16384 x 4096 99.2, 98.5; 8192 x 16384 182, 186; 16384 x 16384 356, 368; the
// rows alone 3 % either way up to 2^27 values, 16384 x 16384 129, 143).
constexpr int64_t KEEP_VALUES = 1 << 26;
template <int LANES, int NV, bool KEEP>
__global__ void __launch_bounds__(256) quantise_bf16_rows_kernel(const u32x4* __restrict__ X, int64_t R, int C8, u32x2* __restrict__ codes,
                                                                 float* __restrict__ scales) {
  const int t = threadIdx.x & (LANES - 1);
  const int64_t r = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (256 / LANES) + threadIdx.x / LANES;
  if (r >= R) return;                                  // (whole waves; with LANES = 256 there is one row per workgroup)
  const u32x4* row = X + r * C8;
  u32x4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) {
    const int c = t + LANES * i;
    v[i] = c < C8 ? (KEEP ? row[c] : ld_stream(row + c)) : u32x4{0u, 0u, 0u, 0u};
  }
  u16x8 mv = {};
#pragma unroll
  for (int i = 0; i < NV; i++) mv = max_mag(mv, v[i]);
  uint32_t m = 0u;
#pragma unroll
  for (int j = 0; j < 8; j++) m = max(m, (uint32_t)mv[j]);
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, sft, 64));
  if constexpr (LANES == 256) {
    __shared__ uint32_t sm[4];
    if ((t & 63) == 0) sm[t >> 6] = m;
    __syncthreads();
    m = max(max(sm[0], sm[1]), max(sm[2], sm[3]));
  }
  const float s = scale_of_max(m);
  if (t == 0) scales[r] = s;
  const ExactDiv d[1] = {ExactDiv(s)};
  u32x2* out = codes + r * C8;
#pragma unroll
  for (int i = 0; i < NV; i++) {
    const int c = t + LANES * i;
    if (c < C8) st_stream(out + c, quantise8(v[i], d));
  }
}

// Rows too long for the registers: one wave per row, two passes over it (the second one finds it in the caches).
__global__ void __launch_bounds__(256) quantise_bf16_long_rows_kernel(const u32x4* __restrict__ X, int64_t R, int C8, u32x2* __restrict__ codes,
                                                                      float* __restrict__ scales) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= R) return;
  const u32x4* row = X + r * C8;
  u16x8 mv = {};
  for (int c = lane; c < C8; c += 64) mv = max_mag(mv, row[c]);
  uint32_t m = 0u;
#pragma unroll
  for (int j = 0; j < 8; j++) m = max(m, (uint32_t)mv[j]);
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, sft, 64));
  const float s = scale_of_max(m);
  if (lane == 0) scales[r] = s;
  const ExactDiv d[1] = {ExactDiv(s)};
  u32x2* out = codes + r * C8;
  for (int c = lane; c < C8; c += 64) st_stream(out + c, quantise8(row[c], d));
}

// Per column (matrices that held_columns leaves), three kernels: (1) the largest magnitude words of every column over slabs of rows, (2) their
// maximum over the slabs and the scale, (3) the codes.  A workgroup of (1) and (3) covers 64 pieces of 8 columns x 4 interleaved row groups, so that a wave's load is
// 1024 contiguous bytes of a row and QC_UNROLL rows are in flight per work item.  The slab maxima [slab][C] (16-bit words) stand in the
// codes buffer, which (3) overwrites afterwards: 2 C ceil(R / QC_ROWS) bytes of its R C.  With a single slab (1) writes the scales.
constexpr int QC_UNROLL = 16, QC_ROWS = 4 * QC_UNROLL, QC_SLABS = 256;

__global__ void __launch_bounds__(256) colmax_bf16_kernel(const u32x4* __restrict__ X, int64_t R, int C8, int64_t slab_rows, u16x8* __restrict__ part,
                                                          float* __restrict__ scales) {
  __shared__ u16x8 sm[4][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane;
  const int64_t r0 = (int64_t)blockIdx.y * slab_rows, r1 = r0 + slab_rows < R ? r0 + slab_rows : R;
  u16x8 m = {};
  if (c < C8) {
    for (int64_t rb = r0 + grp; rb < r1; rb += QC_ROWS) {
      u32x4 v[QC_UNROLL];
#pragma unroll
      for (int i = 0; i < QC_UNROLL; i++) {
        const int64_t r = rb + 4 * i;
        v[i] = X[(r < r1 ? r : rb) * C8 + c];          // past the slab's end: its first row again
      }
#pragma unroll
      for (int i = 0; i < QC_UNROLL; i++) m = max_mag(m, v[i]);
    }
  }
  sm[grp][lane] = m;
  __syncthreads();
  if (grp != 0 || c >= C8) return;
  m = __builtin_elementwise_max(__builtin_elementwise_max(m, sm[1][lane]), __builtin_elementwise_max(sm[2][lane], sm[3][lane]));
  if (part) part[(size_t)blockIdx.y * C8 + c] = m;
  else {
#pragma unroll
    for (int j = 0; j < 8; j++) scales[8 * c + j] = scale_of_max(m[j]);
  }
}

// (2): 16 pieces of 8 columns x 16 groups of slabs per workgroup
__global__ void __launch_bounds__(256) col_scales_kernel(const u16x8* __restrict__ part, int C8, int slabs, float* __restrict__ scales) {
  __shared__ u16x8 sm[16][16];
  const int ci = threadIdx.x & 15, grp = threadIdx.x >> 4, c = blockIdx.x * 16 + ci;
  u16x8 m = {};
  if (c < C8)
    for (int k = grp; k < slabs; k += 16) m = __builtin_elementwise_max(m, part[(size_t)k * C8 + c]);
  sm[grp][ci] = m;
  __syncthreads();
  if (threadIdx.x >= 128) return;
  const int col = threadIdx.x;                          // 16 pieces x 8 columns
  if (blockIdx.x * 128 + col >= 8 * C8) return;
  uint32_t w = 0u;
#pragma unroll
  for (int k = 0; k < 16; k++) w = max(w, (uint32_t)reinterpret_cast<const uint16_t*>(&sm[k][col >> 3])[col & 7]);
  scales[blockIdx.x * 128 + col] = scale_of_max(w);
}

__global__ void __launch_bounds__(256) quantise_bf16_cols_kernel(const u32x4* __restrict__ X, int64_t R, int C8, const float* __restrict__ scales,
                                                                 u32x2* __restrict__ codes) {
  const unsigned nc = (unsigned)((C8 + 63) / 64);      // (one grid dimension: rows / QC_ROWS may pass the limit of the second)
  const int c = (int)(blockIdx.x % nc) * 64 + (threadIdx.x & 63);
  const int64_t rb = (int64_t)(blockIdx.x / nc) * QC_ROWS + (threadIdx.x >> 6);
  if (c >= C8 || rb >= R) return;
  u32x4 v[QC_UNROLL];
#pragma unroll
  for (int i = 0; i < QC_UNROLL; i++) {
    const int64_t r = rb + 4 * i;
    v[i] = ld_stream(X + (r < R ? r : rb) * C8 + c);
  }
  ExactDiv d[8];
#pragma unroll
  for (int j = 0; j < 8; j++) d[j] = ExactDiv(scales[8 * c + j]);
#pragma unroll
  for (int i = 0; i < QC_UNROLL; i++) {
    const int64_t r = rb + 4 * i;
    if (r < R) st_stream(codes + r * C8 + c, quantise8(v[i], d));
  }
}

// Per column, the whole strip of W pieces of 8 columns held in registers between the maximum and the quantisation (one launch, X read once): a
// workgroup of 1024, W neighbouring work items a row, NV rows each.  A strip's rows are parts of lines; strips next to each other go to the same
// XCD, whose L2 puts the lines together.  For which matrices, and what it measured beside the three launches: held_columns (tile_rule.hpp).
template <int W, int NV>
__global__ void __launch_bounds__(1024) quantise_bf16_held_cols_kernel(const u32x4* __restrict__ X, int R, int C8, u32x2* __restrict__ codes,
                                                                       float* __restrict__ scales) {
  constexpr int GROUPS = 1024 / W;
  __shared__ u16x8 sm[16][W];
  const int per_xcd = (int)gridDim.x >> 3, strip = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  const int ci = threadIdx.x & (W - 1), c = strip * W + ci, r0 = threadIdx.x / W;
  const bool in = c < C8;
  const u32x4* col = X + c;
  u32x4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) {
    const int r = r0 + GROUPS * i;
    v[i] = in && r < R ? col[(size_t)r * C8] : u32x4{0u, 0u, 0u, 0u};
  }
  u16x8 m = {};
#pragma unroll
  for (int i = 0; i < NV; i++) m = max_mag(m, v[i]);
#pragma unroll
  for (int sft = W; sft < 64; sft <<= 1) {
    u32x4 o, w = __builtin_bit_cast(u32x4, m);
#pragma unroll
    for (int d = 0; d < 4; d++) o[d] = (uint32_t)__shfl_xor((int)w[d], sft, 64);
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x8, o));
  }
  if ((threadIdx.x & 63) < W) sm[threadIdx.x >> 6][ci] = m;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; k++) m = __builtin_elementwise_max(m, sm[k][ci]);
  if (!in) return;
  ExactDiv d[8];
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const float s = scale_of_max(m[j]);
    if (r0 == 0) scales[8 * c + j] = s;
    d[j] = ExactDiv(s);
  }
  u32x2* out = codes + c;
#pragma unroll
  for (int i = 0; i < NV; i++) {
    const int r = r0 + GROUPS * i;
    if (r < R) st_keep(out + (size_t)r * C8, quantise8(v[i], d));
  }
}

template <int W, int NV>
static int launch_held_cols(const u32x4* X, int64_t R, int C8, u32x2* codes, float* scales, hipStream_t s) {
  const unsigned per_xcd = (unsigned)(((C8 + W - 1) / W + 7) / 8);
  hipLaunchKernelGGL((quantise_bf16_held_cols_kernel<W, NV>), dim3(8 * per_xcd), dim3(1024), 0, s, X, (int)R, C8, codes, scales);
  return (int)hipGetLastError();
}

int launch_quantise_bf16(const void* X, int64_t R, int64_t C, int axis, void* codes, float* scales, hipStream_t s) {
  const int C8 = (int)(C / 8);
  const u32x4* x = static_cast<const u32x4*>(X);
  u32x2* out = static_cast<u32x2*>(codes);
  if (axis == 1) {
    const bool keep = R * C <= KEEP_VALUES;
    auto kern = C8 <= 64 * 2 ? (keep ? quantise_bf16_rows_kernel<64, 2, true> : quantise_bf16_rows_kernel<64, 2, false>)
              : C8 <= 64 * 8 ? (keep ? quantise_bf16_rows_kernel<64, 8, true> : quantise_bf16_rows_kernel<64, 8, false>)
              : C8 <= 256 * 8 ? (keep ? quantise_bf16_rows_kernel<256, 8, true> : quantise_bf16_rows_kernel<256, 8, false>) : quantise_bf16_long_rows_kernel;
    const int per = C8 > 64 * 8 && C8 <= 256 * 8 ? 1 : 4;   // rows per workgroup
    // 2^24 rows, the most there can be, of a workgroup each are 2^32 work items, one more than a grid dimension may have: two halves then
    const int64_t groups = (R + per - 1) / per, most = 1 << 23;
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups < most ? groups : most), (unsigned)((groups + most - 1) / most)), dim3(256), 0, s, x, R, C8, out, scales);
    return (int)hipGetLastError();
  }
  if (held_columns(R, C)) return R <= 512 ? launch_held_cols<4, 2>(x, R, C8, out, scales, s) : launch_held_cols<4, 6>(x, R, C8, out, scales, s);
  // at most QC_SLABS slabs, each a whole number of QC_ROWS rows
  const int64_t slab_rows = ((R + QC_SLABS - 1) / QC_SLABS + QC_ROWS - 1) / QC_ROWS * QC_ROWS;
  const int slabs = (int)((R + slab_rows - 1) / slab_rows);
  u16x8* part = slabs > 1 ? static_cast<u16x8*>(codes) : nullptr;
  const unsigned nc = (unsigned)((C8 + 63) / 64);
  hipLaunchKernelGGL(colmax_bf16_kernel, dim3(nc, (unsigned)slabs), dim3(256), 0, s, x, R, C8, slab_rows, part, scales);
  if (part) hipLaunchKernelGGL(col_scales_kernel, dim3((unsigned)((C8 + 15) / 16)), dim3(256), 0, s, part, C8, slabs, scales);
  hipLaunchKernelGGL(quantise_bf16_cols_kernel, dim3(nc * (unsigned)((R + QC_ROWS - 1) / QC_ROWS)), dim3(256), 0, s, x, R, C8, scales, out);
  return (int)hipGetLastError();
}

}  // namespace ffn24
