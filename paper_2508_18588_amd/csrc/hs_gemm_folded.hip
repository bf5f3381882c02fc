// Instances of the bf16 MFMA GEMM (hs_gemm_stream.h) in which a workgroup takes all K chunks of a split-K projection, and when they
// are taken.
#include "hs_gemm_stream.h"

// Split K fills the chip where there are few rows and writes a partial sum per chunk for the next kernel to read.  With many rows
// the tiles of the output fill it, too, and the partial sums (the 7B shape's down projection at 4096 rows: 528 MB written and 528 MB
// read) are what is left to save: a workgroup of 256 rows x NU units multiplies chunk after chunk, its loads running on across
// them, and adds each chunk's sum to a second set of accumulators.  Same bits: the same products in each chunk, from zero, and
// the chunks' sums added left to right.
// Eight wavefronts of up to 2 x 2 tiles, twice 64 registers; twice 96 (six units, or 384 rows of four) and the twice 128 of four
// wavefronts do not fit beside the fragments.  A k-tile and round takes 0.70, 0.77, 0.88 us with 2, 3, 4 units.
// Five prompts of 129 to 1500 tokens, 1.5B shape, two layers: 749 -> 679 us (QKV at 2048 rows 32 and 18 of the rotary kernel -> 23 and 8,
// O 28 and 13 of the norm -> 24 and 6); 8 x 4096 tokens of the 7B shape 18990 -> 17610; 256 sequences with 1078 rows, 7B, 1337 -> 1320.
// (External linkage: the host takes the kernel's address to raise its dynamic LDS limit.)
template <int EPI, int NU, int SW>
__global__ __launch_bounds__(512) void hs_gemm_folded(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                      const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                                      float* __restrict__ part, const int32_t* __restrict__ m_dev, int m_max,
                                                      int N, int K, int tpc, int n_groups, int n_pass) {
    stream_kernel<EPI, false, true, NU, 2, 2, SW, 8>(A, W, W2, Cout, part, m_dev, m_max, N, K, tpc, n_groups, n_pass);
}

namespace {

template <int EPI, int NU, int SW>
void launch_folded(const bf16_t* a, const bf16_t* w, void* c, const int32_t* m_dev, int m_max, int n, int k, int tpc,
                   int rows_hint, hipStream_t st) {
    static bool configured = false;
    launch_shape<EPI, NU, 2, 2, SW, 512>(&hs_gemm_folded<EPI, NU, SW>, configured, a, w, w, c, nullptr, m_dev, m_max, n, k, 1, tpc,
                                         rows_hint, st);
}

template <int EPI>
void launch_folded_units(int nu, const bf16_t* a, const bf16_t* w, void* c, const int32_t* m_dev, int m_max, int n, int k,
                         int tpc, int rows_hint, hipStream_t st) {
    if (nu == 2) launch_folded<EPI, 2, 8>(a, w, c, m_dev, m_max, n, k, tpc, rows_hint, st);
    else if (nu == 3) launch_folded<EPI, 3, 6>(a, w, c, m_dev, m_max, n, k, tpc, rows_hint, st);
    else launch_folded<EPI, 4, 5>(a, w, c, m_dev, m_max, n, k, tpc, rows_hint, st);
}

}  // namespace

// Rounds count for more here than anywhere else (a round walks all of K): those of an XCD's 32 compute units, which take whole
// weight groups, each k-tiles x the time above + 5 us.  Against the split execution's estimate with 8 % to spare: of 57 (shape,
// projection, rows) measured in whole passes, 1.5B, 7B and 14B shapes at 600 to 4096 rows, what it takes is faster (7B O at 4096 rows 120
// against 170 us, down 590 against 621; 14B O at 1500, 79 against 101) and what it leaves loses, gains less
// than 8 us, or is the long K of the 14B shape in three rounds (4096 rows, 28 us of 2687 a pass).
bool hs_launch_gemm_folded(int epi, const bf16_t* a, const bf16_t* w, void* c, const int32_t* m_dev, int m_max, int n, int k,
                           int chunks, int tpc, int rows_hint, hipStream_t st) {
    const int rows = std::min(rows_hint, m_max), passes = (rows + 255) / 256, units = (n + 31) / 32;
    if (rows < 512) return false;   // one or two passes: too few workgroups
    const bool add = epi == HS_EPI_ADD_F32;
    constexpr double TILE_US[5] = {0, 0, 0.70, 0.77, 0.88};
    double best = hs_gemm_split_us(add, n, chunks, tpc, rows) / 1.08;
    int nu = 0;
    for (int u : {2, 3, 4}) {
        const int groups = (units + u - 1) / u, rounds = ((groups + 7) / 8 * passes + 31) / 32;
        const double us = rounds * (k / BK * TILE_US[u] + 5.) + (add ? 4e-6 * rows * n / 5.5 : 0.);
        if (us < best) { best = us; nu = u; }
    }
    if (nu == 0) return false;
    if (add) launch_folded_units<HS_EPI_ADD_F32>(nu, a, w, c, m_dev, m_max, n, k, tpc, rows_hint, st);
    else launch_folded_units<HS_EPI_STORE_F32>(nu, a, w, c, m_dev, m_max, n, k, tpc, rows_hint, st);
    return true;
}
