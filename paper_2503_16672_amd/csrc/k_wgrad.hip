// The two weight gradients of a step in one launch: dW2 = A2 . dYt^T, row-major [F][D], and dW1 = (A1 . Xt^T)^T, stored transposed [D][F].
// A2 / A1 are the transposed activation / dZ (2:4 along tokens with their metadata, or dense), all operands in panel form.
#include "launch_impl.hpp"

namespace ffn24 {

static GemmArgs wgrad_args(const void* A, const uint8_t* meta, const void* B, int F, int D, int T, int b_form = FORM_PANEL) {
  return GemmArgs{A, meta, B, F, D, T, 1, nullptr, b_form == FORM_PANEL};
}

int launch_wgrad(const void* H, const void* Z, const uint8_t* meta, const void* dYt, const void* Xt, int b_form, int F, int D, int T, void* dW2, void* dW1,
                 hipStream_t s) {
  const GemmArgs g2 = wgrad_args(H, meta, dYt, F, D, T, b_form), g1 = wgrad_args(Z, meta, Xt, F, D, T, b_form);
  const EpiRowMajor::Args e2{static_cast<__bf16*>(dW2), D};
  const EpiColMajor::Args e1{static_cast<__bf16*>(dW1), F};
  if (b_form == FORM_K_MAJOR)
    return meta ? launch_gemm_duo<true, EpiRowMajor, EpiColMajor, false, TR_B>(g2, e2, g1, e1, s)
                : launch_gemm_duo<false, EpiRowMajor, EpiColMajor, false, TR_B>(g2, e2, g1, e1, s);
  return meta ? launch_gemm_duo<true, EpiRowMajor, EpiColMajor>(g2, e2, g1, e1, s) : launch_gemm_duo<false, EpiRowMajor, EpiColMajor>(g2, e2, g1, e1, s);
}

int launch_wgrad_f8(const void* H, const void* Z, const uint8_t* meta, const void* dYt, const void* Xt, int F, int D, int T, float scale2, float scale1,
                    void* dW2, void* dW1, hipStream_t s) {
  const GemmArgs g2 = wgrad_args(H, meta, dYt, F, D, T), g1 = wgrad_args(Z, meta, Xt, F, D, T);
  const EpiRowMajorScaled::Args e2{static_cast<__bf16*>(dW2), D, scale2};
  const EpiColMajorScaled::Args e1{static_cast<__bf16*>(dW1), F, scale1};
  return meta ? launch_gemm_duo<true, EpiRowMajorScaled, EpiColMajorScaled, true>(g2, e2, g1, e1, s)
              : launch_gemm_duo<false, EpiRowMajorScaled, EpiColMajorScaled, true>(g2, e2, g1, e1, s);
}

int launch_wgrad_f8_rowwise(const void* H, const void* Z, const uint8_t* meta, const void* dYt, const void* Xt, int F, int D, int T, const float* rs2,
                            const float* cs2, const float* rs1, const float* cs1, void* dW2, void* dW1, hipStream_t s) {
  const GemmArgs g2 = wgrad_args(H, meta, dYt, F, D, T), g1 = wgrad_args(Z, meta, Xt, F, D, T);
  const EpiRowMajorRowCol::Args e2{static_cast<__bf16*>(dW2), D, rs2, cs2};
  const EpiColMajorRowCol::Args e1{static_cast<__bf16*>(dW1), F, rs1, cs1};
  return meta ? launch_gemm_duo<true, EpiRowMajorRowCol, EpiColMajorRowCol, true>(g2, e2, g1, e1, s)
              : launch_gemm_duo<false, EpiRowMajorRowCol, EpiColMajorRowCol, true>(g2, e2, g1, e1, s);
}

}  // namespace ffn24
