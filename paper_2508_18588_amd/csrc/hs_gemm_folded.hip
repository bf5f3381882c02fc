// Instances of the bf16 MFMA GEMM (hs_gemm_stream.h) in which a workgroup takes all K chunks of a split-K projection, and when they
// are taken.
#include "hs_gemm_stream.h"

// Split K fills the chip where there are few rows and writes a partial sum per chunk for the next kernel to read.  With many rows
// the tiles of the output fill it, too, and the partial sums (the 7B shape's down projection at 4096 rows: 528 MB written and 528 MB
// read) are what is left to save: a workgroup of 256 rows x NU units multiplies chunk after chunk, its loads running on across
// them, and adds each chunk's sum to a second set of accumulators.  Same bits: the same products in each chunk, from zero, and
// the chunks' sums added left to right.
// Eight wavefronts of up to 2 x 2 tiles, twice 64 registers; twice 96 (six units, or 384 rows of four) and the twice 128 of four
// wavefronts do not fit beside the fragments.
// Five prompts of 129 to 1500 tokens, 1.5B shape, two layers: 749 -> 679 us (QKV at 2048 rows 32 and 18 of the rotary kernel -> 23 and 8,
// O 28 and 13 of the norm -> 24 and 6); 8 x 4096 tokens of the 7B shape 18990 -> 17610; 1078 rows of a 7B step, QKV and the rotary
// kernel 52 and 17 -> 47 and 11.
// (External linkage: the host takes the kernel's address to raise its dynamic LDS limit.)
template <int EPI, int NU, int SW>
__global__ __launch_bounds__(512) void hs_gemm_folded(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                      const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                                      float* __restrict__ part, const int32_t* __restrict__ m_dev, int m_max,
                                                      int N, int K, int tpc, int n_groups, int n_pass, int split_rows) {
    stream_kernel<EPI, false, true, NU, 2, 2, SW, 8>(A, W, W2, Cout, part, m_dev, m_max, N, K, tpc, n_groups, n_pass, split_rows);
}

namespace {

template <int EPI, int NU, int SW>
void launch_folded(const bf16_t* a, const bf16_t* w, void* c, float* part, const int32_t* m_dev, int m_max, int n, int k, int tpc,
                   int rows_hint, int split_rows, hipStream_t st) {
    static bool configured = false;
    launch_shape<EPI, NU, 2, 2, SW, 512>(&hs_gemm_folded<EPI, NU, SW>, configured, a, w, w, c, part, m_dev, m_max, n, k, 1, tpc,
                                         rows_hint, st, split_rows);
}

template <int EPI>
void launch_folded_units(int nu, const bf16_t* a, const bf16_t* w, void* c, float* part, const int32_t* m_dev, int m_max, int n,
                         int k, int tpc, int rows_hint, int split_rows, hipStream_t st) {
#define HS_ARGS a, w, c, part, m_dev, m_max, n, k, tpc, rows_hint, split_rows, st
    if (nu == 2) launch_folded<EPI, 2, 8>(HS_ARGS);
    else if (nu == 3) launch_folded<EPI, 3, 6>(HS_ARGS);
    else launch_folded<EPI, 4, 5>(HS_ARGS);
#undef HS_ARGS
}

// Microseconds of a k-tile and round with this many units.
constexpr double TILE_US[5] = {0, 0, 0.70, 0.77, 0.88};

// What `passes` row passes take: rounds of an XCD's 32 compute units, which take whole weight groups, and what adding reads and
// writes of the output; and with the chunks one to a workgroup: rounds of all compute units, and the partial sums.
double folded_us(bool add, int n, int k, int nu, int passes, int rows) {
    const int groups = ((n + 31) / 32 + nu - 1) / nu, rounds = ((groups + 7) / 8 * passes + 31) / 32;
    return rounds * (k / BK * TILE_US[nu] + 5.) + (add ? 4e-6 * rows * n / 5.5 : 0.);
}
double chunks_apart_us(bool add, int n, int nu, int chunks, int tpc, int passes) {
    const int groups = ((n + 31) / 32 + nu - 1) / nu, rounds = (groups * passes * chunks + 255) / 256;
    return rounds * (tpc * TILE_US[nu] + 8.) + (add ? chunks + 1 : chunks - 1) * 4e-6 * 256 * passes * n / 5.5;
}

}  // namespace

// Rounds count for more here than anywhere else: a round walks all of K.  The split execution's estimate has to be `gain` times this
// one's.  HS_FOLD_KNOWN: of 57 (shape, projection, rows) measured in whole passes, 1.5B, 7B and 14B shapes at 600 to 4096 rows,
// what it takes is faster or within 1 % (7B O at 4096 rows 120 against 170 us, down 590 against 621; 14B O at 1500, 79 against
// 101, at 2176 161 against 161) and what it leaves loses, gains less than 8 us, or is the long K of the 14B shape in three rounds
// (4096 rows, 28 us of 2687 a pass).
// Drafting makes the row count swing around what is expected, and a walk along all of K takes its time however few rows there are.
// With up to split_rows rows, by the same estimates, the kernel leaves partial sums after all (a tenth in their favour: a partly filled
// round is faster than a whole one; 7B QKV at 300, 400, 540 and 700 rows, the rotary kernel included, folded 47, 46, 49, 50 us, apart
// 41, 43, 46, 51), and HS_FOLD_GUESSED asks for more.
// us with 1078 expected and 64, 220, 300, 540, 1078, 1300 there, the next kernel included, split / always folded / now: 7B QKV 20, 29,
// 33, 51, 69, 90 / 34, 51, 47, 50, 57, 85 / 20, 29, 41, 46, 57, 86; O, which is split (1.09 expected), 18, 24, 28, 42, 60, 85 / 33, 51, 47,
// 49, 57, 83; O of 4096 columns 19, 26, 32, 52, 73, 92 / 36, 55, 50, 53, 65, 92 / 19, 27, 37, 52, 64, 90.
bool hs_launch_gemm_folded(int epi, const bf16_t* a, const bf16_t* w, void* c, float* part, const int32_t* m_dev, int m_max, int n,
                           int k, int chunks, int tpc, int rows_hint, double gain, hipStream_t st, int* split_rows) {
    const int rows = std::min(rows_hint, m_max), passes = (rows + 255) / 256;
    if (rows < 512) return false;   // one or two passes: too few workgroups
    const bool add = epi == HS_EPI_ADD_F32;
    double best = hs_gemm_split_us(add, n, chunks, tpc, rows) / gain;
    int nu = 0;
    for (int u : {2, 3, 4}) {
        const double us = folded_us(add, n, k, u, passes, rows);
        if (us < best) { best = us; nu = u; }
    }
    if (nu == 0) return false;
    int live = 0;       // passes up to which the chunks are taken apart
    while (split_rows && live + 1 < passes && chunks_apart_us(add, n, nu, chunks, tpc, live + 1) < 1.1 * folded_us(add, n, k, nu, live + 1, 256 * (live + 1))) live++;
    if (split_rows) *split_rows = 256 * live;
#define HS_ARGS nu, a, w, c, part, m_dev, m_max, n, k, tpc, rows_hint, 256 * live, st
    if (add) launch_folded_units<HS_EPI_ADD_F32>(HS_ARGS);
    else launch_folded_units<HS_EPI_STORE_F32>(HS_ARGS);
#undef HS_ARGS
    return true;
}
