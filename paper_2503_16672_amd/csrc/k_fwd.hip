// Forward kernels of the 2:4 FFN: fused up-projection (dense MFMA + ReLU^2 + keep-2-of-4) and the
// sparse-MFMA GEMM with a row-major result (down-projection, dX, dW2).
#include "launch_impl.hpp"

namespace ffn24 {

int launch_up_prune24(const void* W1, int w1_form, const void* X, const float* b1, int T, int D, int F,
                      void* Hc, uint8_t* meta, void* Hdbg, uint32_t* nnz, unsigned long long* tele, const int* token_map, hipStream_t s) {
  GemmArgs g{W1, nullptr, X, F, T, D, w1_form == FORM_PANEL, token_map};
  EpiPrune24::Args ea{static_cast<__bf16*>(Hc), meta, static_cast<__bf16*>(Hdbg), b1, F, nullptr, nullptr};
  if (nnz || tele) {
    EpiPrune24T<true>::Args eas{static_cast<__bf16*>(Hc), meta, static_cast<__bf16*>(Hdbg), b1, F, nnz, tele};
    return w1_form == FORM_K_MAJOR ? launch_gemm<false, EpiPrune24T<true>, false, TR_A>(g, eas, s) : launch_gemm<false, EpiPrune24T<true>>(g, eas, s);
  }
  return w1_form == FORM_K_MAJOR ? launch_gemm<false, EpiPrune24, false, TR_A>(g, ea, s) : launch_gemm<false, EpiPrune24>(g, ea, s);
}

int launch_sp_rowmajor(const void* vals, const uint8_t* meta, int a_panel, const void* B, int b_form, int M, int N, int K, void* C, hipStream_t s) {
  GemmArgs g{vals, meta, B, M, N, K, a_panel, nullptr, b_form == FORM_PANEL};
  EpiRowMajor::Args ea{static_cast<__bf16*>(C), N};
  if (b_form == FORM_K_MAJOR) return launch_gemm<true, EpiRowMajor, false, TR_B>(g, ea, s);
  if (!a_panel && b_form == FORM_ROWS && K >= ROWS_MIN_K) return launch_gemm_rows<EpiRowMajor>(g, ea, s);
  return launch_gemm<true, EpiRowMajor>(g, ea, s);
}

int launch_dx_featurewise(const void* Hc, const uint8_t* meta, const void* dZc, const void* W1p, int T, int D, int F, void* dX, void* Hc_t, uint8_t* meta_t, void* dZc_t,
                          hipStream_t s) {
  const GemmArgs g{dZc, meta, W1p, T, D, F, 1, nullptr, 1};
  const EpiRowMajor::Args ea{static_cast<__bf16*>(dX), D};
  const SideFeaturewise::Args sa{static_cast<const uint16_t*>(Hc), meta, static_cast<const uint16_t*>(dZc), T, F, static_cast<uint16_t*>(Hc_t), meta_t,
                                 static_cast<uint16_t*>(dZc_t)};
  bool rode = false;
  int rc = launch_gemm_side<true, EpiRowMajor, 0, SideFeaturewise>(g, ea, sa, (unsigned)(F / FW_FEAT) * (unsigned)(T / FW_TOK), &rode, s);
  if (rode) return rc;
  rc = launch_gemm<true, EpiRowMajor>(g, ea, s);
  return rc ? rc : launch_featurewise24(Hc, meta, dZc, T, F, Hc_t, meta_t, dZc_t, nullptr, s);
}

int launch_sp_rowmajor_mapped(const void* vals, const uint8_t* meta, int a_panel, const void* B, int b_form, int M, int N, int K, void* C,
                              const int* rowmap, hipStream_t s) {
  GemmArgs g{vals, meta, B, M, N, K, a_panel, nullptr, b_form == FORM_PANEL};
  EpiRowMajorMapped::Args ea{static_cast<__bf16*>(C), N, rowmap};
  return b_form == FORM_K_MAJOR ? launch_gemm<true, EpiRowMajorMapped, false, TR_B>(g, ea, s) : launch_gemm<true, EpiRowMajorMapped>(g, ea, s);
}

}  // namespace ffn24
