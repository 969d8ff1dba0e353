// fp8 (e4m3) kernels with a scale per row of each operand: up-projections, dH GEMMs, and the products with a scale per row and per column
// of the result (forward and backward, 2:4 and dense baseline).
#include "launch_impl.hpp"

namespace ffn24 {

// row-wise-scaled variants (scales per token for the activation operand, per output channel for the weight)
int launch_up_prune24_f8_rowwise(const void* W1t8, const void* X8, const float* b1, int T, int D, int F, const float* sx, const float* sw1,
                                 void* Hc16, uint8_t* meta16, void* Hdbg, uint32_t* rowmax, uint32_t* nnz, hipStream_t s) {
  GemmArgs g{W1t8, nullptr, X8, F, T, D, 1, nullptr, 1};
  EpiPrune24Rw::Args ea{static_cast<__bf16*>(Hc16), meta16, static_cast<__bf16*>(Hdbg), b1, F, sx, sw1, rowmax, nnz};
  if (nnz) {
    EpiPrune24RwT<true>::Args eas{static_cast<__bf16*>(Hc16), meta16, static_cast<__bf16*>(Hdbg), b1, F, sx, sw1, rowmax, nnz};
    return launch_gemm<false, EpiPrune24RwT<true>, true>(g, eas, s);
  }
  return launch_gemm<false, EpiPrune24Rw, true>(g, ea, s);
}

int launch_sp_rowmajor_f8_rowwise_mapped(const void* vals8, const uint8_t* meta, const void* B8, int b_panel, int M, int N, int K, const float* rs, const float* cs,
                                         void* C, const int* rowmap, hipStream_t s) {
  GemmArgs g{vals8, meta, B8, M, N, K, 1, nullptr, b_panel};
  EpiRowMajorRowColMapped::Args ea{static_cast<__bf16*>(C), N, rs, cs, rowmap};
  return launch_gemm<true, EpiRowMajorRowColMapped, true>(g, ea, s);
}

static PairSet<EpiRowMajorRowColMapped> split_set(const void* vals8, const uint8_t* meta, int ns, const void* Ad8, int nd, const void* B8, int N, int K,
                                                  const float* rs, const float* cs, void* C, int ldc, const int* rowmap) {
  return {GemmArgs{Ad8, nullptr, B8, nd, N, K, 1, nullptr, 1}, {static_cast<__bf16*>(C), ldc, rs + ns, cs, rowmap + ns},
          GemmArgs{vals8, meta, B8, ns, N, K, 1, nullptr, 1}, {static_cast<__bf16*>(C), ldc, rs, cs, rowmap}};
}

int launch_split_wgrad_f8_rowwise(const void* vals8, const uint8_t* meta, int ns, const void* Ad8, int nd, const void* B8, int N, int K,
                                  const float* rs, const float* cs, void* C, int ldc, const int* rowmap, hipStream_t s) {
  const PairSet<EpiRowMajorRowColMapped> a = split_set(vals8, meta, ns, Ad8, nd, B8, N, K, rs, cs, C, ldc, rowmap);
  return launch_gemm_pair<EpiRowMajorRowColMapped, true>(a, a, 1, s);
}

int launch_split_wgrads_f8_rowwise(const void* H, const void* Z, const uint8_t* meta, int ns, const void* Hd, const void* Zd, int nd, const void* dYt,
                                   const void* Xt, int N, int K, const float* rs2, const float* cs2, const float* rs1, const float* cs1, void* dW2, void* dW1t,
                                   int ldc, const int* rowmap, hipStream_t s) {
  return launch_gemm_pair<EpiRowMajorRowColMapped, true>(split_set(H, meta, ns, Hd, nd, dYt, N, K, rs2, cs2, dW2, ldc, rowmap),
                                                         split_set(Z, meta, ns, Zd, nd, Xt, N, K, rs1, cs1, dW1t, ldc, rowmap), 2, s);
}

int launch_up_relu2_f8_rowwise(const void* W1t8, const void* X8, const float* b1, int T, int D, int F, const float* sx, const float* sw1,
                               void* H16, uint32_t* rowmax, void* Ht16, hipStream_t s) {
  GemmArgs g{W1t8, nullptr, X8, F, T, D, 1, nullptr, 1};
  EpiRelu2Rw::Args ea{static_cast<__bf16*>(H16), b1, F, sx, sw1, rowmax, static_cast<__bf16*>(Ht16), T};
  return launch_gemm<false, EpiRelu2Rw, true>(g, ea, s);
}

int launch_dense_rowmajor_f8_rowwise(const void* A8, const void* B8, int b_panel, int M, int N, int K, const float* rs, const float* cs, void* C, hipStream_t s) {
  GemmArgs g{A8, nullptr, B8, M, N, K, 1, nullptr, b_panel};
  EpiRowMajorRowCol::Args ea{static_cast<__bf16*>(C), N, rs, cs};
  return launch_gemm<false, EpiRowMajorRowCol, true>(g, ea, s);
}

int launch_sp_rowmajor_f8_rowwise(const void* vals8, const uint8_t* meta, const void* B8, int b_panel, int M, int N, int K, const float* rs, const float* cs,
                                  void* C, hipStream_t s) {
  GemmArgs g{vals8, meta, B8, M, N, K, 1, nullptr, b_panel};
  EpiRowMajorRowCol::Args ea{static_cast<__bf16*>(C), N, rs, cs};
  return launch_gemm<true, EpiRowMajorRowCol, true>(g, ea, s);
}

// row-wise-scaled backward: the dH GEMM with the pointwise part fused (bf16 compressed dZ + row maxima out), and the sparse GEMM
// with the transposing store and a scale per row and per column (dW1)
int launch_dh_gather_f8_rowwise(const void* W2rp8, const void* dY8r, const void* Hc16, const uint8_t* meta16, int T, int D, int F,
                                const float* sw2_f, const float* sdy_t, void* dZc16, uint32_t* rowmax, hipStream_t s) {
  GemmArgs g{W2rp8, nullptr, dY8r, F, T, D, 1, nullptr, 1};
  EpiDGatherRw::Args ea{static_cast<const __bf16*>(Hc16), meta16, static_cast<__bf16*>(dZc16), F, sw2_f, sdy_t, rowmax};
  return launch_gemm<false, EpiDGatherRw, true>(g, ea, s);
}

int launch_sp_colmajor_f8_rowwise(const void* vals8, const uint8_t* meta, const void* B8, int M, int N, int K, const float* rs, const float* cs,
                                  void* Ct, hipStream_t s) {
  GemmArgs g{vals8, meta, B8, M, N, K, 1, nullptr, 1};
  EpiColMajorRowCol::Args ea{static_cast<__bf16*>(Ct), M, rs, cs};
  return launch_gemm<true, EpiColMajorRowCol, true>(g, ea, s);
}

// dense row-wise-scaled backward: the dH GEMM with the pointwise part fused (bf16 dZ as [T][F] and [F][T], row maxima), and the
// dense GEMM with the transposing store scaled per row and per column
int launch_dh_drelu_f8_rowwise(const void* W2rp8, const void* dY8r, const void* H16, int T, int D, int F, const float* sw2_f, const float* sdy_t,
                               void* dZ16, void* dZt16, uint32_t* rowmax, hipStream_t s) {
  GemmArgs g{W2rp8, nullptr, dY8r, F, T, D, 1, nullptr, 1};
  EpiDReluRw::Args ea{static_cast<const __bf16*>(H16), static_cast<__bf16*>(dZ16), static_cast<__bf16*>(dZt16), F, T, sw2_f, sdy_t, rowmax};
  return launch_gemm<false, EpiDReluRw, true>(g, ea, s);
}

int launch_dense_colmajor_f8_rowwise(const void* A8, const void* B8, int M, int N, int K, const float* rs, const float* cs, void* Ct, hipStream_t s) {
  GemmArgs g{A8, nullptr, B8, M, N, K, 1, nullptr, 1};
  EpiColMajorRowCol::Args ea{static_cast<__bf16*>(Ct), M, rs, cs};
  return launch_gemm<false, EpiColMajorRowCol, true>(g, ea, s);
}

}  // namespace ffn24
