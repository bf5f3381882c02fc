// Instances of the bf16 MFMA GEMM (hs_gemm_stream.h) with eight wavefronts per workgroup, and the choice of an instance.
#include "hs_gemm_stream.h"

// NU weight units per workgroup, MT row tiles per wavefront pair (128*MT rows per pass; 64 for MT = 0), SA / SW ring stages
// (three and more activation stages: the two operands are fetched by a wavefront group each; MT = 0: of passes of 64 rows,
// with more rows few_rows_fallback says).
// (External linkage: the host takes the kernel's address to raise its dynamic LDS limit.)
template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW>
__global__ __launch_bounds__(512) void hs_gemm_stream(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                      const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                                      float* __restrict__ part, const int32_t* __restrict__ m_dev,
                                                      int m_max, int N, int K, int tpc, int n_groups, int n_pass) {
    stream_kernel<EPI, PARTIAL, false, NU, MT, SA, SW, 8>(A, W, W2, Cout, part, m_dev, m_max, N, K, tpc, n_groups, n_pass);
}

namespace {

template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW>
void launch_stream(const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part, const int32_t* m_dev,
                   int m_max, int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st) {
    static bool configured = false;
    launch_shape<EPI, NU, MT, SA, SW, 512>(&hs_gemm_stream<EPI, PARTIAL, NU, MT, SA, SW>, configured, a, w, w2, c, part, m_dev,
                                           m_max, n, k, chunks, tpc, rows_hint, st);
}

// Passes of 64 rows up to this hint: a step with twice the rows expected still takes one.  (With more the same launch takes
// passes of 256: drafting can bring any number of rows after a step that had few.)
#ifndef HS_FEW_ROWS
#define HS_FEW_ROWS 32
#endif
constexpr int HS_TALL_ROWS = 160, HS_WIDE_KERNEL_ROWS = 512;
// A round of 256 workgroups takes this long per k-tile (four wavefronts; eight, for each unit).
constexpr int HS_WIDE_TILE_NS = 1600, HS_UNIT_TILE_NS = 305;
#ifndef HS_WIDE_GROUP_ROWS
#define HS_WIDE_GROUP_ROWS 352   // measured cross-over at the 7B shape: 33 vs 40 us at 300 rows, 49 vs 37 us at 385
#endif

// Units per workgroup: the candidate with the least (rounds of 256 workgroups) x (time of one); a round grows by less than
// its units, because the activation tile's share does not grow with them.  (One round of a SwiGLU projection with K = 3584
// in 3, 4 and 5 units: 38, 43, 53 us at 64 rows, 56, 67, 80 at 220, which is units + 2; for the benchmark configurations'
// shapes at 16 to 4096 rows any constant from 2 to 6 picks the same.)
// The reduction order does not depend on it, so the expected number of row passes counts, too.
int choose_units(int units, int chunks, int passes) {
    int best = 4, best_cost = 1 << 30;
    for (int nu : {5, 4, 3}) {
        const int wgs = ((units + nu - 1) / nu) * chunks * passes;
        const int cost = ((wgs + 255) / 256) * (nu + 6);
        if (cost < best_cost) { best = nu; best_cost = cost; }
    }
    return best;
}

// The row-maximum epilogue's column groups are part of its output's layout: a function of the width alone.
int rowmax_units(int n) {
    const int units = (n + 31) / 32;
    return (units + 1279) / 1280 * 5 <= (units + 1023) / 1024 * 4 ? 5 : 4;
}

// How a projection of so many weight units (and K chunks) runs when rows_hint rows are expected.
struct launch_plan {
    int nu;                             // weight units per workgroup of eight wavefronts
    long long rounds, wide_rounds;      // of 256 workgroups; and of four wavefronts
    bool wide;
};
launch_plan plan_launch(int units, int chunks, int rows_hint, int m_max) {
    const int rows = std::min(rows_hint, m_max), pass_rows = rows_hint > HS_TALL_ROWS ? 384 : 256;
    const int passes = std::max(1, (rows + pass_rows - 1) / pass_rows);
    launch_plan p;
    p.nu = choose_units(units, chunks, passes);
    p.rounds = ((long long)((units + p.nu - 1) / p.nu) * chunks * passes + 255) / 256;
    p.wide_rounds = ((long long)((units + 7) / 8) * chunks * ((rows + 255) / 256) + 255) / 256;
    // Workgroups of 256 rows x 8 units in four wavefronts, where their rounds take less time.  A round is 1.6 us per k-tile
    // there and 0.305 us per unit here (gate/up, down and QKV of the 7B and 14B shapes at 1000 to 4096 rows; of these 36
    // the rule picks the faster one or one that is within 2 %.  us, here against there: 7B gate/up at 1280 rows, 4 rounds
    // against 3: 318, 278; at 1500, 4 against 4: 344, 346; QKV at 1500, 2 of 4 units against 2: 73, 83; 14B gate/up at
    // 2048, 5 against 4: 544, 480; 7B down at 4096, 9 against 8: 674, 615).
    p.wide = rows_hint >= HS_WIDE_KERNEL_ROWS && p.wide_rounds * HS_WIDE_TILE_NS < p.rounds * HS_UNIT_TILE_NS * p.nu;
    return p;
}

template <int EPI, bool PARTIAL>
void launch_stream_shape(const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                         const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint,
                         hipStream_t st) {
    // Rows per pass: 256 leaves LDS for a deeper weight ring; 384 once the hint is within a factor 1.6 of 256 (the
    // row count of a speculative step swings by a third around its mean), so that a step above its average does
    // not pay a second pass over the weights.  Row tiles that do not exist cost nothing in either shape.
    const bool tall = rows_hint > HS_TALL_ROWS, few = rows_hint <= HS_FEW_ROWS && !PARTIAL && k >= 16 * BK;
    const int unit_cols = (EPI == HS_EPI_SWIGLU_BF16) ? 16 : 32;
    const launch_plan plan = plan_launch((n + unit_cols - 1) / unit_cols, chunks, rows_hint, m_max);
    const int nu = EPI == HS_EPI_ROWMAX ? rowmax_units(n) : plan.nu;
#define HS_ARGS a, w, w2, c, part, m_dev, m_max, n, k, chunks, tpc, rows_hint, st
    if (EPI != HS_EPI_ROWMAX && plan.wide) {
        hs_launch_gemm_wide(EPI, PARTIAL, HS_ARGS);
        return;
    }
    // The 64-row groups of the smaller split-K shapes (QKV, O, the 1.5B down projection) pay at a few hundred rows, where they halve the
    // partial sums; with many row passes every group re-reads the whole activation slab of its pass, and wider groups
    // (half as many re-reads) win.  The K chunking -- the reduction order -- is the shape's either way.
    if (PARTIAL && chunks > 1 && hs_gemm_narrow_groups(n, k) && rows_hint < HS_WIDE_GROUP_ROWS) {
        if constexpr (PARTIAL) {
            if (tall) launch_stream<EPI, PARTIAL, 2, 3, 2, 6>(HS_ARGS);
            else launch_stream<EPI, PARTIAL, 2, 2, 2, 8>(HS_ARGS);
        }
    } else if (nu == 5) {
        if (tall) launch_stream<EPI, PARTIAL, 5, 3, 2, 3>(HS_ARGS);
        else launch_stream<EPI, PARTIAL, 5, 2, 2, 4>(HS_ARGS);
    } else if (nu == 3) {
        if constexpr (EPI != HS_EPI_ROWMAX) {
            if (tall) launch_stream<EPI, PARTIAL, 3, 3, 2, 5>(HS_ARGS);
            else if (few) { if constexpr (!PARTIAL) launch_stream<EPI, PARTIAL, 3, 0, 4, 5>(HS_ARGS); }
            else launch_stream<EPI, PARTIAL, 3, 2, 3, 5>(HS_ARGS);
        }
    } else {
        if (tall) launch_stream<EPI, PARTIAL, 4, 3, 2, 4>(HS_ARGS);
        else if (few) { if constexpr (!PARTIAL) launch_stream<EPI, PARTIAL, 4, 0, 3, 4>(HS_ARGS); }
        else launch_stream<EPI, PARTIAL, 4, 2, 3, 4>(HS_ARGS);
    }
#undef HS_ARGS
}

}  // namespace

int hs_gemm_rowmax_groups(int n) {
    const int nu = rowmax_units(n);
    return (n + 32 * nu - 1) / (32 * nu);
}

// By the rounds of the kernel that is taken at this many rows (512 and more): what its k-tiles take and about 8 us for
// a round's first tiles and its stores, and the partial sums read back at 5.5 TB/s (7B shape, 4096 rows, us: QKV 148 and 27 for
// 152 and 34, O 117 and 53 for 120 and 53, down 486 and 107 for 491 and 107; 14B at 1088: 89, 65, 156 for 92, 68, 158).
double hs_gemm_split_us(bool add, int n, int chunks, int tpc, int rows) {
    const launch_plan p = plan_launch((n + 31) / 32, chunks, rows, rows);
    const double gemm = p.wide ? p.wide_rounds * (tpc * 1e-3 * HS_WIDE_TILE_NS + 8.) : p.rounds * (tpc * 1e-3 * HS_UNIT_TILE_NS * p.nu + 8.);
    return gemm + (add ? chunks + 1 : chunks - 1) * 4e-6 * rows * n / 5.5;
}

void hs_launch_gemm_stream(int epi, const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                           const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint,
                           hipStream_t st) {
#define HS_ARGS a, w, w2, c, part, m_dev, m_max, n, k, chunks, tpc, rows_hint, st
    if (epi == HS_EPI_SWIGLU_BF16) {
        launch_stream_shape<HS_EPI_SWIGLU_BF16, false>(HS_ARGS);
    } else if (chunks > 1) {
        // partial sums: the ordered reduce applies the epilogue
        launch_stream_shape<HS_EPI_STORE_F32, true>(HS_ARGS);
    } else if (epi == HS_EPI_ROWMAX) {
        launch_stream_shape<HS_EPI_ROWMAX, false>(HS_ARGS);
    } else if (epi == HS_EPI_ADD_F32) {
        launch_stream_shape<HS_EPI_ADD_F32, false>(HS_ARGS);
    } else {
        launch_stream_shape<HS_EPI_STORE_F32, false>(HS_ARGS);
    }
#undef HS_ARGS
}
