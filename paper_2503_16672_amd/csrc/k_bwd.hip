// Backward kernels of the 2:4 FFN that are not shared with the forward.
#include "launch_impl.hpp"

namespace ffn24 {

int launch_dh_gather(const void* W2, const void* dY, const void* Hc, const uint8_t* meta, int T, int D, int F, void* dZc,
                     const int* token_map, hipStream_t s) {
  GemmArgs g{W2, nullptr, dY, F, T, D, 1, token_map};
  EpiDGather::Args ea{static_cast<const __bf16*>(Hc), meta, static_cast<__bf16*>(dZc), F};
  return launch_gemm<false, EpiDGather>(g, ea, s);
}

int launch_sp_colmajor(const void* vals, const uint8_t* meta, int a_panel, const void* B, int b_form, int M, int N, int K, void* Ct, hipStream_t s) {
  GemmArgs g{vals, meta, B, M, N, K, a_panel, nullptr, b_form == FORM_PANEL};
  EpiColMajor::Args ea{static_cast<__bf16*>(Ct), M};
  return b_form == FORM_K_MAJOR ? launch_gemm<true, EpiColMajor, false, TR_B>(g, ea, s) : launch_gemm<true, EpiColMajor>(g, ea, s);
}

static PairSet<EpiRowMajorMapped> split_set(const void* vals, const uint8_t* meta, int ns, const void* Ad, int nd, const void* B, int b_form, int N, int K, void* C, int ldc,
                                            const int* rowmap) {
  return {GemmArgs{Ad, nullptr, B, nd, N, K, 1, nullptr, b_form == FORM_PANEL}, {static_cast<__bf16*>(C), ldc, rowmap + ns},
          GemmArgs{vals, meta, B, ns, N, K, 1, nullptr, b_form == FORM_PANEL}, {static_cast<__bf16*>(C), ldc, rowmap}};
}

// split weight gradient: rows [0, ns) of the permuted feature space from the sparse GEMM over (vals, meta), rows
// [ns, ns + nd) from the dense GEMM over Ad, both against the same B, in one launch; row m goes to C[rowmap[m]][*]
int launch_split_wgrad(const void* vals, const uint8_t* meta, int ns, const void* Ad, int nd, const void* B, int b_form, int N, int K,
                       void* C, int ldc, const int* rowmap, hipStream_t s) {
  const PairSet<EpiRowMajorMapped> a = split_set(vals, meta, ns, Ad, nd, B, b_form, N, K, C, ldc, rowmap);
  return b_form == FORM_K_MAJOR ? launch_gemm_pair<EpiRowMajorMapped, false, TR_B>(a, a, 1, s) : launch_gemm_pair<EpiRowMajorMapped>(a, a, 1, s);
}

int launch_split_wgrads(const void* H, const void* Z, const uint8_t* meta, int ns, const void* Hd, const void* Zd, int nd, const void* dYt, const void* Xt, int b_form,
                        int N, int K, void* dW2, void* dW1t, int ldc, const int* rowmap, hipStream_t s) {
  const PairSet<EpiRowMajorMapped> a = split_set(H, meta, ns, Hd, nd, dYt, b_form, N, K, dW2, ldc, rowmap), b = split_set(Z, meta, ns, Zd, nd, Xt, b_form, N, K, dW1t, ldc, rowmap);
  return b_form == FORM_K_MAJOR ? launch_gemm_pair<EpiRowMajorMapped, false, TR_B>(a, b, 2, s) : launch_gemm_pair<EpiRowMajorMapped>(a, b, 2, s);
}

}  // namespace ffn24
