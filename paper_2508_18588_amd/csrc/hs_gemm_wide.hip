// Instances of the bf16 MFMA GEMM (hs_gemm_stream.h) with four wavefronts per workgroup, for many rows.
#include "hs_gemm_stream.h"

// (External linkage: the host takes the kernel's address to raise its dynamic LDS limit.)
template <int EPI, bool PARTIAL, int NU>
__global__ __launch_bounds__(256, 1) void hs_gemm_wide(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                       const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                                       float* __restrict__ part, const int32_t* __restrict__ m_dev, int m_max,
                                                       int N, int K, int tpc, int n_groups, int n_pass) {
    stream_kernel<EPI, PARTIAL, false, NU, 2, 2, 3, 4>(A, W, W2, Cout, part, m_dev, m_max, N, K, tpc, n_groups, n_pass);
}

namespace {

template <int EPI, bool PARTIAL, int NU>
void launch_wide(const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part, const int32_t* m_dev, int m_max,
                 int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st) {
    static bool configured = false;
    // (a quarter more passes than expected: without rows they cost nothing, while rows beyond the grid's passes are a second
    // round; 2200 rows at a hint of 2000: 7B QKV 139 -> 100 us, down 409 -> 347)
    launch_shape<EPI, NU, 2, 2, 3, 256>(&hs_gemm_wide<EPI, PARTIAL, NU>, configured, a, w, w2, c, part, m_dev, m_max, n, k, chunks,
                                        tpc, rows_hint + rows_hint / 4, st);
}

}  // namespace

void hs_launch_gemm_wide(int epi, bool partial, const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                         const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st) {
#define HS_ARGS a, w, w2, c, part, m_dev, m_max, n, k, chunks, tpc, rows_hint, st
    if (epi == HS_EPI_SWIGLU_BF16) launch_wide<HS_EPI_SWIGLU_BF16, false, 8>(HS_ARGS);
    else if (partial) launch_wide<HS_EPI_STORE_F32, true, 8>(HS_ARGS);
    else if (epi == HS_EPI_ADD_F32) launch_wide<HS_EPI_ADD_F32, false, 8>(HS_ARGS);
    else launch_wide<HS_EPI_STORE_F32, false, 8>(HS_ARGS);
#undef HS_ARGS
}
