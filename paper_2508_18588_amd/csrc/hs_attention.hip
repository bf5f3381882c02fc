// Ragged multi-query paged attention for the verify step.
//
// For sequence b with L cached positions and nn draft-tree nodes, every node's query (all G query heads that
// share one KV head) attends to cache positions [0, L) and to the slots L + i of the nodes i that are its
// ancestors or itself.  The KV cache is read once per (sequence, KV head) and step, shared by all G * nn query
// rows -- which is why verifying a whole draft costs about one KV traversal (Sec. 2.2 of the paper).
//
// Work decomposition.  Keys are cut into partitions of `part_keys` absolute positions; every (partition, KV head,
// sequence) yields one partial result (unnormalised O, running max, running sum) per query row, and a second
// kernel merges a row's partitions in index order.  Inside a partition, keys are visited in 32-key sub-tiles (two
// 16-token pages), each through the same routine: scores transposed, S^T = K . Q^T (v_mfma_f32_32x32x16_bf16,
// A = K tile from LDS, B = Q^T held in registers), so that each lane owns one query row -- the online-softmax
// statistics are per-lane scalars and the exponentiated scores are already in the register layout the second
// product O^T = V^T . P^T needs as its B operand.  V is stored in the cache with the token index fastest so V^T
// operands are two plain 8-byte LDS reads (see load_values).
//
// Two ways to run a unit (= one partition of one (sequence, KV head)), chosen per sequence by its number of query
// rows R = G * nn:
//   R <= 32 (one-token decoding and short drafts): one WAVEFRONT per unit.  A wavefront streams its units one after
//     the other through a private LDS slice and never synchronises with the others.  With a single 32-row tile the
//     softmax arithmetic of a partition is one instruction stream; giving every wavefront its own stream keeps all
//     four SIMDs of a compute unit busy and the KV stream bandwidth-bound.
//   R > 32: one WORKGROUP per unit; the (up to four) 32-row tiles are dealt to the 4 wavefronts, and the 32-key sub-tiles
//     travel from global memory straight into a ring in LDS that all four fill and all four read (attn_wg_stream).
//     A sequence with more than 128 query rows per KV head is cut into units of four row tiles, each of which walks the
//     partition's keys on its own: holding two row tiles per wavefront instead would cost every workgroup unit of the
//     launch half the resident workgroups (registers), which was measured to be far dearer than reading the K/V of the
//     few very long drafts twice.
// Both run the identical per-row arithmetic on the identical partitions: masked keys contribute exact zeros and
// partitions merge in index order, so a row's result is bit-identical whether it is verified next to other draft
// rows or decoded alone.
//
// Launch.  The units of a step are listed on the device once per verify call (hs_worklist.h) and a
// persistent grid -- exactly the workgroups that are resident at once -- works the lists off: wavefront units by a
// static deal, workgroup units through a counter (see attn_verify_mfma).  K and V are read with non-temporal loads.
// A second entry, attn_prefill_mfma, does the same causally over a chunk of consecutive tokens.
#include "hs_gemm_common.h"   // fragment types, loads into LDS
#include "hs_internal.h"

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int ATT_RING = 4;   // sub-tiles of 32 keys in LDS: one per wavefront, or a ring of them per workgroup

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A 32-key sub-tile (two pages) in LDS: K as 32 rows of HD elements, then V^T as two pages of HD rows of 16 tokens, both
// without padding, so that a page's K or V^T block is one contiguous run that a load into LDS can fill.  16-byte chunks are
// permuted instead: within a row of K, so that 16 consecutive rows read at the same chunk cover the 64 banks once; of 16 rows of
// V^T first the first halves, then the second ones, so that an operand is two 8-byte pieces a constant distance apart.  (32 lanes
// read the same half of their chunks, so two of them meet on each bank: the counters show LDS busy 50 % of the cycles, 20 of
// them conflicts, where single 16-byte pieces had 23 % and none; a 14B step with trees 1388 -> 1391 us.)
template <int HD>
struct sub_tile {
    static constexpr int PAGE = 32 * HD, V = 2 * PAGE, BYTES = 4 * PAGE;   // a page's K (or V^T) block, V^T's place, all
    static __device__ __forceinline__ int k_at(int key, int chunk) {
        return key * 2 * HD + ((chunk ^ (HD == 128 ? key & 15 : (key >> 1) & 7)) << 4);
    }
    // what 1 KB further on changes in the permutation
    static constexpr int k_step(int i) { return (HD == 128 ? 4 * i & 15 : 4 * i & 7) << 4; }
    static constexpr int V_HALF = 256;   // from a row's first to its second half
    static __device__ __forceinline__ int v_at(int dim, int chunk) { return (dim >> 4) * 512 + chunk * V_HALF + (dim & 15) * 16; }
    // where in a page's V^T block the 16 bytes that belong at 16 c of it in LDS come from
    static __device__ __forceinline__ int v_from(int c) { return ((c >> 5) * 16 + (c & 15)) * 32 + ((c >> 4) & 1) * 16; }
};

// One 32-key sub-tile for one 32-row query tile: S^T = K.Q^T, online softmax per lane, O^T += V^T.P^T.
// Every query row's arithmetic is independent of which other rows are in flight.
// Element e of a lane's scores is key 8 (e / 4) + 4 half + e % 4: the eight probabilities of a page that a lane feeds to the
// second product belong to two runs of four tokens, and so do the V^T operand's two pieces.  (With the A operand's rows
// permuted so that they are one run and the operand one 16-byte piece, the launch was 0 to 0.4 % shorter and every output
// differed, by 0.002 to 0.003 of its size: the sums' order is kept.)
template <int HD>
__device__ __forceinline__ void load_keys(const unsigned char* tile, bf16x8 (&ka)[HD / 16], int half, int l32) {
    int k0 = sub_tile<HD>::k_at(l32, half);  // chunk 2 ks + half: the permutation is an exclusive or, and so is 2 ks
    asm volatile("" : "+v"(k0));              // (eight addresses kept across the caller's loop would spill)
#pragma unroll
    for (int ks = 0; ks < HD / 16; ks++) ka[ks] = *reinterpret_cast<const bf16x8*>(tile + (k0 ^ (ks << 5)));
}
template <int HD>
__device__ __forceinline__ f32x16 scores(const bf16x8 (&ka)[HD / 16], const bf16x8 (&qf)[HD / 16]) {
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; e++) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < HD / 16; ks++) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], s, 0, 0, 0);
    return s;
}

// Masks the scores (in tiles that reach past the cached prefix) and moves the running maximum.  (A maximum that only moves
// where a score exceeds it by 2^8 spares most of the rescales, 1 % of a step with trees, but its probabilities are no longer
// exactly 1 at the maximum: the error of a layer against 64 bits grew by 3 %.)
// Returns what the sum so far is to be scaled by.
template <int HD>
__device__ __forceinline__ float take_maximum(f32x16& s, f32x16 (&o)[HD / 32], float& m_run, uint64_t anc, int kbase, int L,
                                               int total, float scale_log2, int half) {
    // query row = this lane's.  Only tiles that reach past the cached prefix need the tree mask.
    if (kbase + 32 > L) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int kp = kbase + 8 * (e >> 2) + 4 * half + (e & 3);
            const bool vis = (kp < L) | ((kp < total) & (bool)((anc >> ((kp - L) & 63)) & 1ull));
            s[e] = vis ? s[e] : -INFINITY;
        }
    }
    float tmax = s[0];
#pragma unroll
    for (int e = 1; e < 16; e++) tmax = fmaxf(tmax, s[e]);
    // lanes l and l+32 hold the two halves of a query row: v_permlane32_swap puts the upper half of its first
    // operand and the lower half of its second in each other's place, so the two results are, in some order, a
    // lane's own value and its partner's -- enough for a maximum and for a sum, with no trip through the LDS
    {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
        tmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2;   // scale > 0: commutes with max
    }
    const float m_new = fmaxf(m_run, tmax);
    // where it does not move for any of the 32 rows, multiplying by exactly 1 is skipped
    float alpha = 1.f;
    if (__any(m_new != m_run)) {
        alpha = fast_exp2(m_run - (m_new == -INFINITY ? 0.f : m_new));
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < HD / 32; dt++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[dt][e] *= alpha;
    }
    return alpha;
}

// Probabilities of a sub-tile, as the second product's operand, and their sum.
__device__ __forceinline__ void probabilities(const f32x16& s, float m_run, float alpha, float& l_run, float scale_log2,
                                              bf16x8 (&pb)[2]) {
    const float m_safe = (m_run == -INFINITY) ? 0.f : m_run;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e++) {
        const float p = fast_exp2(__builtin_fmaf(s[e], scale_log2, -m_safe));
        psum += p;
        pb[e >> 3][e & 7] = (__bf16)p;
    }
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(psum), __float_as_uint(psum), false, false);
    l_run = __builtin_fmaf(l_run, alpha, __uint_as_float(sw[0]) + __uint_as_float(sw[1]));
}

template <int HD>
__device__ __forceinline__ bf16x8 load_values(const unsigned char* tile, int i, int half, int l32) {
    using T = sub_tile<HD>;
    constexpr int NDT = HD / 32;
    const unsigned char* at = tile + T::V + T::v_at(l32, 0) + 8 * half + (i / NDT) * T::PAGE + (i % NDT) * 1024;
    union { u32x2 u[2]; bf16x8 v; } va;
    va.u[0] = *reinterpret_cast<const u32x2*>(at);
    va.u[1] = *reinterpret_cast<const u32x2*>(at + T::V_HALF);
    return va.v;
}

template <int HD>
__device__ inline void attn_subtile(const unsigned char* tile, const bf16x8 (&qf)[HD / 16], f32x16 (&o)[HD / 32], float& m_run,
                                    float& l_run, uint64_t anc, int kbase, int L, int total, float scale_log2, int half,
                                    int l32) {
    constexpr int NDT = HD / 32;
    bf16x8 ka[HD / 16], pb[2];
    load_keys<HD>(tile, ka, half, l32);
    f32x16 s = scores<HD>(ka, qf);
    const float alpha = take_maximum<HD>(s, o, m_run, anc, kbase, L, total, scale_log2, half);
    probabilities(s, m_run, alpha, l_run, scale_log2, pb);
#pragma unroll
    for (int i = 0; i < 2 * NDT; i++)
        o[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_values<HD>(tile, i, half, l32), pb[i / NDT], o[i % NDT], 0, 0, 0);
}

// A 64-key tile (four pages) of the prefill: the same steps with one maximum and one rescale per 64 keys and the two
// halves' products independent of each other.  The rows are consecutive tokens: every row of the tile sees every key below
// `all`, and the lane's own row the keys below `mine`.
// A page's keys are in order: of a tile of scores a lane of half h holds keys 4h .. 4h+3 and 8+4h .. 8+4h+3 of each page.  The values
// that belong to them lie together in LDS, where in a row's 16 prefill_value_at says: one 16-byte read.  The half that
// lies first is the other one in every second set of eight rows, so that no two lanes meet in a bank.
__device__ __forceinline__ int prefill_value_at(int row, int half) { return row * 16 + ((half ^ (row >> 3)) & 1) * 8; }
template <int HD>
__device__ inline void attn_tile64(const bf16_t* sK, const bf16_t* sV, const bf16x8 (&qf)[HD / 16], f32x16 (&o)[HD / 32],
                                   float& m_run, float& l_run, int kbase, int all, int mine, float scale_log2, int half,
                                   int l32) {
    constexpr int KS = HD + 8, NKS = HD / 16, NDT = HD / 32;
    f32x16 s[2];
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int e = 0; e < 16; e++) s[u][e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const bf16x8 ka = *reinterpret_cast<const bf16x8*>(&sK[(32 * u + l32) * KS + ks * 16 + half * 8]);
            s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[ks], s[u], 0, 0, 0);
        }
    if (kbase + 64 > all) {
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const int kp = kbase + 32 * u + 8 * (e >> 2) + 4 * half + (e & 3);
                s[u][e] = kp < all || kp < mine ? s[u][e] : -INFINITY;
            }
    }
    float tmax = s[0][0];
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int e = 0; e < 16; e++) tmax = fmaxf(tmax, s[u][e]);
    {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
        tmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2;
    }
    const float m_new = fmaxf(m_run, tmax);
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = fast_exp2(m_run - m_safe);
    float psum[2] = {0.f, 0.f};
    bf16x8 pb[4];
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const float p = fast_exp2(__builtin_fmaf(s[u][e], scale_log2, -m_safe));
            psum[u] += p;
            pb[2 * u + (e >> 3)][e & 7] = (__bf16)p;
        }
    float sum = psum[0] + psum[1];
    {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
        sum = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    l_run = l_run * alpha + sum;
    m_run = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[dt][e] *= alpha;
    }
#pragma unroll
    for (int kk = 0; kk < 4; kk++)
#pragma unroll
        for (int dt = 0; dt < NDT; dt++) {
            const bf16x8 va = *reinterpret_cast<const bf16x8*>(&sV[prefill_value_at(kk * HD + dt * 32 + l32, half)]);
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[kk], o[dt], 0, 0, 0);
        }
}

// Page holding position p0 (which differs from lane to lane).  Positions at or beyond `total` (nothing written yet) and
// malformed table entries resolve to the sequence's first page: its keys are masked and its finite values are
// multiplied by exact zeros, so every load can be unconditional.
__device__ inline int safe_page_lane(const int32_t* bt, int p0, int total, int max_blocks, int n_blocks) {
    int pidx = p0 >> 4;
    int page = (p0 < total && pidx < max_blocks) ? bt[pidx] : bt[0];
    return (page >= 0 && page < n_blocks) ? page : 0;
}

// Query fragments (B operand of S^T) and ancestor mask of the lane's row; rows beyond R read as zero.
template <int HD>
__device__ inline void load_query_tile(const bf16_t* q, const uint64_t* anc_mask, int r0, int rt, int R, int G,
                                       int hq, int j, int half, int l32, bf16x8 (&qf)[HD / 16], uint64_t& anc) {
    int rho = rt * 32 + l32;
    bool ok = rho < R;
    int node = ok ? rho / G : 0;
    int g = ok ? rho - node * G : 0;
    anc = (ok && anc_mask) ? anc_mask[r0 + node] : 0ull;
    const bf16_t* qp = q + ((size_t)(r0 + node) * hq + j * G + g) * HD;
#pragma unroll
    for (int ks = 0; ks < HD / 16; ks++) {
        if (ok) {
            qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16 + half * 8);
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++) qf[ks][e] = (__bf16)0.f;
        }
    }
}

// Partial result of one partition for the lane's row: running max (log2 domain) and sum in fp32, and the partition's
// own normalised output O / l in fp16 -- a convex combination of V rows, so within fp16's range whenever V is, and
// rounded 8 times finer than the bf16 result of the merge.  Half the bytes of an fp32 partial: the partial results
// are the one write stream of the launch, and writes in the middle of the K/V read stream are dear.
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

template <int HD>
__device__ inline void store_partial(const f32x16 (&o)[HD / 32], float m_run, float l_run, _Float16* part_o,
                                     float* part_ml, int r0, int rt, int R, int G, int hq, int j, int max_parts,
                                     int part, int half, int l32) {
    int rho = rt * 32 + l32;
    if (rho >= R) return;
    int node = rho / G, g = rho - node * G;
    size_t prow = ((size_t)(r0 + node) * hq + j * G + g) * max_parts + part;
    _Float16* po = part_o + prow * HD;
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;   // a partition in which the row sees no key: all zero
#pragma unroll
    for (int dt = 0; dt < HD / 32; dt++)
#pragma unroll
        for (int g4 = 0; g4 < 4; g4++) {
            f16x4 v = {(_Float16)(o[dt][4 * g4] * inv), (_Float16)(o[dt][4 * g4 + 1] * inv),
                       (_Float16)(o[dt][4 * g4 + 2] * inv), (_Float16)(o[dt][4 * g4 + 3] * inv)};
            *reinterpret_cast<f16x4*>(po + dt * 32 + 8 * g4 + 4 * half) = v;
        }
    if (half == 0) {
        part_ml[prow * 2] = m_run;
        part_ml[prow * 2 + 1] = l_run;
    }
}

// Everything a unit of work needs besides its own (sequence, KV head, partition).
struct AttnArgs {
    const bf16_t* q;
    const bf16_t* kc;     // already offset to the layer
    const bf16_t* vc;
    const int32_t* seq_len;
    const int32_t* block_table;
    const int32_t* row_off;
    const uint64_t* anc_mask;
    _Float16* part_o;
    float* part_ml;
    int max_blocks, n_blocks, max_parts, part_keys, hq, hkv;
    float scale_log2;
};

// A unit of work: one partition of one (sequence, KV head), with the sequence's row range and cached length, as the
// list kernel wrote it (two int4 per unit).
struct AttnUnit { int b, j, part, r0, nn, L, rt0; };   // rt0: first 32-row tile this unit covers (workgroup units)

__device__ inline AttnUnit attn_unit_from(const int4& p, const int4& q) {
    AttnUnit u;
    u.b = __builtin_amdgcn_readfirstlane(p.x);
    u.j = __builtin_amdgcn_readfirstlane(p.y);
    u.part = __builtin_amdgcn_readfirstlane(p.z);
    u.r0 = __builtin_amdgcn_readfirstlane(p.w);
    u.nn = __builtin_amdgcn_readfirstlane(q.x);
    u.L = __builtin_amdgcn_readfirstlane(q.y);
    u.rt0 = __builtin_amdgcn_readfirstlane(q.z);
    return u;
}

// Units with at most 32 query rows, taken by ONE WAVEFRONT each: the wavefront walks its units (first, first + stride,
// ...) as one uninterrupted stream of 32-key sub-tiles through a private LDS slice, always with the next sub-tile's
// K/V in flight in registers -- also across a unit boundary: the next unit's list entry is read during the current
// unit's first sub-tile, its page numbers during the second, its first sub-tile during the current unit's last.
// There is no workgroup synchronisation (a wavefront's LDS operations execute in order) and no atomic: a load or an
// atomic that returns late holds back every later load of its wavefront.
template <int HD>
__device__ inline void attn_wave_stream(const AttnArgs& a, const int4* __restrict__ list, int n_units, int first,
                                        int stride, unsigned char* tile, int lane) {
    using T = sub_tile<HD>;
    constexpr int NKS = HD / 16, NDT = HD / 32;
    if (first >= n_units) return;
    const int half = lane >> 5, l32 = lane & 31;
    const int G = a.hq / a.hkv;
    const size_t page_stride = (size_t)a.hkv * 16 * HD;

    AttnUnit cu = attn_unit_from(list[2 * first], list[2 * first + 1]);
    int total = cu.L + cu.nn;
    int k_begin = cu.part * a.part_keys;
    int k_end = min(total, k_begin + a.part_keys);
    const bf16_t* kbase_ptr = a.kc + (size_t)cu.j * 16 * HD;   // + page * page_stride
    const bf16_t* vbase_ptr = a.vc + (size_t)cu.j * HD * 16;
    // the unit's page numbers: lane l holds the page of positions k_begin + 16 l .. + 15 (at most 64 pages), handed out by
    // readlane -- no table look-up sits between two sub-tiles
    int my_page = safe_page_lane(a.block_table + (size_t)cu.b * a.max_blocks, k_begin + 16 * lane, total, a.max_blocks,
                                 a.n_blocks);

    int it_n = first + stride;
    bool have_n = it_n < n_units;
    int4 en0 = list[2 * (have_n ? it_n : first)], en1 = list[2 * (have_n ? it_n : first) + 1];
    bool n_ready = false;
    AttnUnit nu = cu;
    int total_n = total, k_begin_n = k_begin, k_end_n = k_end, my_page_n = my_page;
    const bf16_t *kbase_n = kbase_ptr, *vbase_n = vbase_ptr;

    bf16x8 qf[NKS];
    uint64_t anc;
    f32x16 o[NDT];
    float m_run = -INFINITY, l_run = 0.f;
    load_query_tile<HD>(a.q, a.anc_mask, cu.r0, 0, cu.nn * G, G, a.hq, cu.j, half, l32, qf, anc);
#pragma unroll
    for (int dt = 0; dt < NDT; dt++)
#pragma unroll
        for (int e = 0; e < 16; e++) o[dt][e] = 0.f;

    // one 32-key sub-tile = two pages; a page's K block and V^T block are each 16*HD contiguous elements, copied as
    // NCP 16-byte chunks per lane (chunk c = lane + 64*ii covers elements [8c, 8c+8)).  The loads are non-temporal:
    // K/V is read once per launch, and kept out of the caches it leaves the queries and the partial results (which
    // the merge kernel reads right after) there -- 10 % of the launch
    constexpr int NCP = HD / 32;
    u32x4 rk[2 * NCP], rv[2 * NCP];
#define HS_W_FETCH(PAGES, KPTR, VPTR, PAGE0)                                                                      \
    {                                                                                                             \
        _Pragma("unroll") for (int pp = 0; pp < 2; pp++) {                                                        \
            const size_t pofs = (size_t)__builtin_amdgcn_readlane(PAGES, (PAGE0) + pp) * page_stride;             \
            const bf16_t* kp_ = (KPTR) + pofs + lane * 8;                                                         \
            const bf16_t* vp_ = (VPTR) + pofs + lane * 8;                                                         \
            _Pragma("unroll") for (int ii = 0; ii < NCP; ii++) {                                                  \
                rk[pp * NCP + ii] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp_ + ii * 512));                           \
                rv[pp * NCP + ii] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vp_ + ii * 512));                           \
            }                                                                                                     \
        }                                                                                                         \
    }
    HS_W_FETCH(my_page, kbase_ptr, vbase_ptr, 0)
    const int k_put = T::k_at(lane / (HD / 8), lane % (HD / 8)), v_put = T::V + T::v_at(lane >> 1, lane & 1);
    int kb = k_begin;
    for (;;) {
        int k_to = k_put;
        asm volatile("" : "+v"(k_to));   // (see load_keys)
#pragma unroll
        for (int pp = 0; pp < 2; pp++)
#pragma unroll
            for (int ii = 0; ii < NCP; ii++) {
                // (64 chunks further on: 512 / HD rows, whose permutation differs by an exclusive or, or 32 rows of V^T)
                *reinterpret_cast<u32x4*>(tile + (k_to ^ T::k_step(ii)) + pp * T::PAGE + ii * 1024) = rk[pp * NCP + ii];
                *reinterpret_cast<u32x4*>(tile + v_put + pp * T::PAGE + ii * 1024) = rv[pp * NCP + ii];
            }
        const bool last = kb + 32 >= k_end;
        if (!n_ready && have_n && (last || kb > k_begin)) {
            nu = attn_unit_from(en0, en1);
            total_n = nu.L + nu.nn;
            k_begin_n = nu.part * a.part_keys;
            k_end_n = min(total_n, k_begin_n + a.part_keys);
            kbase_n = a.kc + (size_t)nu.j * 16 * HD;
            vbase_n = a.vc + (size_t)nu.j * HD * 16;
            my_page_n = safe_page_lane(a.block_table + (size_t)nu.b * a.max_blocks, k_begin_n + 16 * lane, total_n,
                                       a.max_blocks, a.n_blocks);
            n_ready = true;
        }
        if (!last) HS_W_FETCH(my_page, kbase_ptr, vbase_ptr, (kb + 32 - k_begin) >> 4)
        else if (have_n) HS_W_FETCH(my_page_n, kbase_n, vbase_n, 0)
        attn_subtile<HD>(tile, qf, o, m_run, l_run, anc, kb, cu.L, total, a.scale_log2, half, l32);
        kb += 32;
        if (last) {
            store_partial<HD>(o, m_run, l_run, a.part_o, a.part_ml, cu.r0, 0, cu.nn * G, G, a.hq, cu.j, a.max_parts, cu.part,
                              half, l32);
            if (!have_n) break;
            cu = nu;
            total = total_n; k_begin = k_begin_n; k_end = k_end_n; my_page = my_page_n;
            kbase_ptr = kbase_n; vbase_ptr = vbase_n;
            kb = k_begin;
            it_n += stride;
            have_n = it_n < n_units;
            n_ready = false;
            en0 = list[2 * (have_n ? it_n : first)];
            en1 = list[2 * (have_n ? it_n : first) + 1];
            load_query_tile<HD>(a.q, a.anc_mask, cu.r0, 0, cu.nn * G, G, a.hq, cu.j, half, l32, qf, anc);
#pragma unroll
            for (int dt = 0; dt < NDT; dt++)
#pragma unroll
                for (int e = 0; e < 16; e++) o[dt][e] = 0.f;
            m_run = -INFINITY;
            l_run = 0.f;
        }
    }
#undef HS_W_FETCH
}

// A word that is the same for the whole wavefront and that no kernel in flight writes, read through the scalar cache: its
// wait does not touch the vector memory counter, on which the loads into LDS are counted.
__device__ __forceinline__ int scalar_word(const int32_t* p) {
    return *reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<unsigned long long>(p));
}
__device__ inline AttnUnit attn_unit_scalar(const int4* list, int it) {
    const int32_t* p = reinterpret_cast<const int32_t*>(list + 2 * (size_t)it);
    return {scalar_word(p), scalar_word(p + 1), scalar_word(p + 2), scalar_word(p + 3), scalar_word(p + 4), scalar_word(p + 5),
            scalar_word(p + 6)};
}

// Units with more than 32 query rows, taken by the WORKGROUP one after the other: a stream of 32-key sub-tiles through a ring
// of RING of them in LDS, across unit boundaries.  Sub-tile s is a page's K or V^T block per wavefront, fetched straight into
// LDS while s - 3 .. s - 1 are multiplied: no staging registers, no LDS writes and no wavefronts that only stage, and up
// to 48 KB on their way per workgroup at any time (a 128-key tile at a time through registers, two barriers per tile, left
// the memory system idle while it was written and multiplied).  One barrier per sub-tile: it says that the sub-tile has
// landed (every wavefront has waited for its own part) and that its predecessor has been read, whose place in the ring is
// then refilled.  The unit's 32-row tiles (rt0 .. rt0 + 3) are dealt round-robin, from a unit-dependent wavefront on so that
// two-tile sequences do not all use the same SIMDs.
// The next unit is claimed (`take`, zeroed by the list writers) shortly before the fetches reach it, not earlier: with
// about as many units as workgroups an early claim gives some of them two and others none.
// The keys run one sub-tile ahead of the values, so that the next sub-tile's first product is issued between this one's
// exponentials: an instruction takes a wavefront about eight clocks, and there are two of them on a SIMD.
// Steps with a 128-key tile at a time and now (us; launches of the first 45 -> 42): 64 sequences of 2560 tokens, a third of
// them with 9 rows, four 1.5B layers 573 -> 553; 64 trees of 17 rows over 8192 keys, one 14B layer 1404 -> 1378;
// 256 sequences with a long tail of lengths, a 7B layer 1335 -> 1323.  What is
// left there: without its arithmetic the 14B launch takes 400 us of 470, without its loads 250, and the partial results
// (see hs_create) are 70 of the 400.
template <int HD>
__device__ inline void attn_wg_stream(const AttnArgs& a, const int4* __restrict__ list, int n_units, int first_idle,
                                      int32_t* __restrict__ take, unsigned char* ring, int* s_item, int tid) {
    using T = sub_tile<HD>;
    constexpr int NKS = HD / 16, NDT = HD / 32, CPW = T::PAGE / 1024;   // 1 KB loads per wavefront and sub-tile
    static_assert(ATT_RING == 4, "the wait counts below");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int G = a.hq / a.hkv;
    const size_t page_bytes = (size_t)a.hkv * T::PAGE;

    // the wavefront's share of a sub-tile: K (is_v = 0) or V^T of its page `pg`
    const int is_v = wave & 1, pg = wave >> 1;
    const unsigned ring_off = (unsigned)(size_t)(hs_gemm_detail::lds_ptr_t)ring + is_v * T::V + pg * T::PAGE;
    unsigned from[CPW];   // where in the page's block a lane's 16 bytes of load i come from
#pragma unroll
    for (int i = 0; i < CPW; i++) {
        const int c = lane + 64 * i;
        from[i] = is_v ? T::v_from(c) : T::k_at(c / (HD / 8), c % (HD / 8));   // (K's permutation is its own inverse)
    }

    // Workgroups without wavefront units take the first ones by their number, all others what the counter hands out.
    const int n_given = max(0, (int)gridDim.x - first_idle);
    const bool more = n_units > n_given;
    int it = (int)blockIdx.x - first_idle, par = 0;
    if (it < 0) {
        if (!more) return;
        if (tid == 0) s_item[1] = n_given + atomicAdd(take, 1);
        __syncthreads();   // (also: every private slice of the ring has been read)
        it = __builtin_amdgcn_readfirstlane(s_item[1]);
    }
    if (it >= n_units) return;
    AttnUnit cu = attn_unit_scalar(list, it), nu = cu;
    bool have_n = false;

    // fetches: the sub-tile after the last one asked for
    const unsigned char* f_base = nullptr;
    const int32_t* f_bt = nullptr;
    int f_pos = 0, f_end = 0, f_total = 0, f_page = 0, f_slot = 0;
    auto page_of = [&](int pos) __attribute__((always_inline)) {   // (see safe_page_lane)
        const int p = pos >> 4;
        const int page = scalar_word(f_bt + (pos < f_total && p < a.max_blocks ? p : 0));
        return page >= 0 && page < a.n_blocks ? page : 0;
    };
    auto fetch_unit = [&](const AttnUnit& u) __attribute__((always_inline)) {
        f_total = u.L + u.nn;
        f_pos = u.part * a.part_keys;
        f_end = min(f_total, f_pos + a.part_keys);
        f_bt = a.block_table + (size_t)u.b * a.max_blocks;
        f_base = reinterpret_cast<const unsigned char*>(is_v ? a.vc : a.kc) + (size_t)u.j * T::PAGE;
        f_page = page_of(f_pos + 16 * pg);
    };
    // asks for one sub-tile and looks up the page of the one after it; false at the unit's end
    auto fetch = [&]() __attribute__((always_inline)) {
        if (f_pos >= f_end) return false;
        const unsigned char* src = f_base + (size_t)f_page * page_bytes;
        const unsigned dst = ring_off + f_slot * T::BYTES;
#pragma unroll
        for (int i = 0; i < CPW; i++) hs_gemm_detail::load_to_lds_16_stream(src, from[i], dst + i * 1024);
        f_slot = (f_slot + 1) & (ATT_RING - 1);
        f_pos += 32;
        if (f_pos < f_end) f_page = page_of(f_pos + 16 * pg);
        return true;
    };
    fetch_unit(cu);
    int ahead = 0;   // sub-tiles asked for and not yet waited for
    while (ahead < ATT_RING - 1 && fetch()) ahead++;
    bool f_in_next = false;
    int slot = 0;
    for (;;) {
        const int total = cu.L + cu.nn, R = cu.nn * G, nrt = (R + 31) >> 5;
        const int k_begin = cu.part * a.part_keys, k_end = min(total, k_begin + a.part_keys);
        const int my_rt = cu.rt0 + ((wave - (cu.part + cu.j + cu.b)) & 3);
        const bool computes = my_rt < nrt;
        const int k_put = max(k_begin, k_begin + ((k_end - k_begin - 1) & ~31) - 96);   // the claim is handed round here
        const int k_claim = k_put - 64;                                                // ... and made here (or before the first)
        int claim = 0;
        if (more && k_claim < k_begin && tid == 0) claim = n_given + atomicAdd(take, 1);
        bf16x8 qf[NKS];
        uint64_t anc;
        f32x16 o[NDT];
        float m_run = -INFINITY, l_run = 0.f;
        load_query_tile<HD>(a.q, a.anc_mask, cu.r0, computes ? my_rt : 0, computes ? R : 0, G, a.hq, cu.j, half, l32, qf, anc);
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[dt][e] = 0.f;
        // (waited for here: inside the loop the wait would be for every load in flight, each time round)
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) asm volatile("" : "+v"(qf[ks]));
        asm volatile("" : "+v"(anc));
        // waits for the wavefront's own part of the sub-tile at the head of what it asked for (what was asked for later may
        // still be on its way), then for everybody's
        auto landed = [&](bool take_one) __attribute__((always_inline)) {
            if (take_one) {
                ahead--;
                if (ahead >= 2) HS_WAIT_VMCNT(2 * CPW);
                else if (ahead == 1) HS_WAIT_VMCNT(CPW);
                else HS_WAIT_VMCNT(0);
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        };
        landed(!is_v);        // the first keys
        while (ahead < ATT_RING - 1 && fetch()) ahead++;
        f32x16 sc = {};
        if (computes) {
            bf16x8 ka[NKS];
            load_keys<HD>(ring + slot * T::BYTES, ka, half, l32);
            sc = scores<HD>(ka, qf);
        }
        for (int kb = k_begin; kb < k_end; kb += 32) {
            if (more && kb == k_put && tid == 0) s_item[par] = claim;
            landed(is_v || kb + 32 < k_end);     // this sub-tile's values, the next one's keys
            if (more && kb == k_claim && tid == 0) claim = n_given + atomicAdd(take, 1);
            if (more && kb == k_put) {
                const int n = __builtin_amdgcn_readfirstlane(s_item[par]);
                have_n = n < n_units;
                if (have_n) nu = attn_unit_scalar(list, n);
                par ^= 1;
            }
            if (f_pos >= f_end && have_n && !f_in_next && kb >= k_put) {
                fetch_unit(nu);
                f_in_next = true;
            }
            while (ahead < ATT_RING - 1 && fetch()) ahead++;
            if (computes) {
                bf16x8 ka[NKS], pb[2], va[2 * NDT];
                load_keys<HD>(ring + ((slot + 1) & (ATT_RING - 1)) * T::BYTES, ka, half, l32);
#pragma unroll
                for (int i = 0; i < 2 * NDT; i++) va[i] = load_values<HD>(ring + slot * T::BYTES, i, half, l32);
                const float alpha = take_maximum<HD>(sc, o, m_run, anc, kb, cu.L, total, a.scale_log2, half);
                const f32x16 next = scores<HD>(ka, qf);     // (of the last sub-tile: of whatever lies there, not used)
                probabilities(sc, m_run, alpha, l_run, a.scale_log2, pb);
#pragma unroll
                for (int i = 0; i < 2 * NDT; i++)
                    o[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pb[i / NDT], o[i % NDT], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NKS; i++) {             // a product, its share of the exponentials
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x402, 64 / NKS, 0);
                }
                sc = next;
            }
            slot = (slot + 1) & (ATT_RING - 1);
        }
        if (computes)
            store_partial<HD>(o, m_run, l_run, a.part_o, a.part_ml, cu.r0, my_rt, R, G, a.hq, cu.j, a.max_parts, cu.part, half,
                              l32);
        if (!have_n) break;
        cu = nu;
        have_n = f_in_next = false;   // (the fetches got into it at the latest with its predecessor's last sub-tile)
    }
}

// Persistent launch: exactly as many workgroups as are resident at once.  First every wavefront streams its share
// of the wavefront units (wavefront w of workgroup g: units 4 g + w, 4 g + w + 4 gridDim.x, ... -- dealt out
// statically, so that nothing but K/V tiles is ever waited for); then the workgroups take the workgroup units one by
// one through a counter.  These are short -- four wavefronts share one partition -- and fill the ragged end of the first
// phase: a workgroup that had less to stream takes more of them.  No workgroup is launched for work that does not
// exist, and which workgroup computes a unit has no influence on the unit's result.
template <int HD>
__global__ __launch_bounds__(256, 2) void attn_verify_mfma(AttnArgs a, const int32_t* __restrict__ work,
                                                           int32_t* __restrict__ take, const int4* __restrict__ list_a,
                                                           const int4* __restrict__ list_b) {
    // four private sub-tiles (wavefront units) or the ring of them shared by the workgroup (workgroup units)
    __shared__ __attribute__((aligned(1024))) unsigned char ring[ATT_RING * sub_tile<HD>::BYTES];
    __shared__ int s_item[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_a = work[0], n_b = work[1];
    attn_wave_stream<HD>(a, list_b, n_b, blockIdx.x * 4 + wave, gridDim.x * 4, ring + wave * sub_tile<HD>::BYTES, lane);
    if (n_a == 0) return;
    attn_wg_stream<HD>(a, list_a, n_a, (n_b + 3) / 4, take, ring, s_item, tid);
}

// Prefill of a chunk of consecutive tokens per sequence (KV recomputation of a resumed rollout): token i of the chunk
// attends to positions [0, L + i].  One workgroup per (block of 128 query rows, KV head, sequence) walks the keys
// from position 0 in 64-key tiles -- a row's arithmetic depends on absolute key positions only, not on how the text
// was cut into chunks -- and writes the normalised output itself: with hundreds of rows per sequence there is
// enough parallelism without cutting the key axis.  A wavefront has one row tile of 32 rows (rows of one token's G query
// heads are adjacent); a row tile skips the key tiles that lie wholly behind it.
// Bound by LDS and by what a wavefront waits for between the phases of a tile (counters: LDS busy 68 % of the cycles -- every
// wavefront reads all of K and V for its 32 rows -- vector ALUs 37 %, matrix cores 30 %); a wavefront alternates between
// matrix and vector work, so it takes two wavefronts per SIMD to keep either busy: two workgroups per compute unit, each
// with its own barriers.
// One workgroup per compute unit with two row tiles per wavefront, which ran them one after the other: 467 us for 4096
// rows of 28 heads against 512 to 4096 keys, 115 us for 2048 rows of 12 heads.  Two workgroups: 225 and 49 us.  With two
// tiles of keys in LDS (one barrier per tile instead of two, the next tile written while this one is multiplied), page
// numbers held in a register and one softmax step per 64 keys: 190 and 38 us (630 TFLOP/s).  (One maximum per 64 instead of
// 32 keys leaves fewer probabilities at exactly 1: the error against 64 bits grows by 0.1 to 0.2 %, 0.004629 to 0.004635.)
// Those counters are of values in rows of 40 bytes, read in two pieces of 8.  Now they lie in rows of 32 in the order in which a lane
// needs them (prefill_value_at), written in pieces of 8 and read in one of 16: 182 -> 176 and 41 -> 38, same bits.  (With a
// page's keys in another order in LDS the writes are one piece, too: 174 and 35, but every sum of probabilities is another one.)  Multiplying
// the next tile's keys between the exponentials needs 32 registers more than there are (182 and 42 us, with 10 spilled).
template <int HD>
__global__ __launch_bounds__(256, 2) void attn_prefill_mfma(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ kc, const bf16_t* __restrict__ vc, size_t layer_off,
    const int32_t* __restrict__ len_plus1, const int32_t* __restrict__ block_table, int max_blocks, int n_blocks,
    const int32_t* __restrict__ row_off, bf16_t* __restrict__ out, int hq, int hkv, float scale_log2, int batch, int nx) {
    constexpr int KS = HD + 8, NKS = HD / 16, NDT = HD / 32, TILE = 64, NCK = HD / 32;
    constexpr int K_BUF = TILE * KS, V_BUF = 4 * HD * 16;
    __shared__ __attribute__((aligned(16))) bf16_t sK[2 * K_BUF];
    __shared__ __attribute__((aligned(16))) bf16_t sV[2 * V_BUF];

    // Workgroup id -> (sequence, KV head) pair and block of rows, the blocks that see the most keys first.  Ids are dealt
    // round-robin to the eight XCDs: with a multiple of eight pairs, all blocks of a pair go to one XCD and find its K
    // and V in that L2 (other numbers of pairs would leave some XCDs with more pairs than others).
    const int pairs = hkv * batch;
    int pair = blockIdx.x / nx, bx = blockIdx.x % nx;
    if ((pairs & 7) == 0) {
        const int local = blockIdx.x >> 3;
        pair = (local / nx) * 8 + (blockIdx.x & 7);
        bx = local % nx;
    }
    bx = nx - 1 - bx;
    const int j = pair % hkv, b = pair / hkv;
    const int r0 = row_off[b];
    const int nn = row_off[b + 1] - r0;
    if (nn <= 0) return;
    const int L = len_plus1[b] - 1;
    const int total = L + nn;
    const int G = hq / hkv;
    const int R = nn * G;
    const int row_base = bx * 128;
    if (row_base >= R) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int32_t* bt = block_table + (size_t)b * max_blocks;
    const bf16_t* kbase_ptr = kc + layer_off + (size_t)j * 16 * HD;
    const bf16_t* vbase_ptr = vc + layer_off + (size_t)j * HD * 16;
    const size_t page_stride = (size_t)hkv * 16 * HD;
    // keys this block needs: up to the position of its last row's token
    const int last_node = min(nn - 1, (min(R, row_base + 128) - 1) / G);
    const int k_end = L + last_node + 1;

    const int rt = bx * 4 + wave;              // the wavefront's row tile
    const bool rt_on = rt * 32 < R;
    bf16x8 qf[NKS];
    f32x16 o[NDT];
    float m_run = -INFINITY, l_run = 0.f;
    {
        uint64_t unused;
        load_query_tile<HD>(q, nullptr, r0, rt_on ? rt : 0, rt_on ? R : 0, G, hq, j, half, l32, qf, unused);
    }
    const int rho = rt * 32 + l32;
    const int lim_lane = rho < R ? L + rho / G + 1 : 0;
    const int lim_min = L + (rt * 32) / G + 1;
    const int lim_max = L + min(nn - 1, (rt * 32 + 31) / G) + 1;
#pragma unroll
    for (int dt = 0; dt < NDT; dt++)
#pragma unroll
        for (int e = 0; e < 16; e++) o[dt][e] = 0.f;

    // Two tiles in LDS, a third on its way in registers: tile t + 1 is written while tile t is multiplied, one barrier per
    // tile.  Lane p holds the page of keys 1024 n + 16 p .. + 15, handed out by readlane (a table look-up per tile and
    // page would put a trip to memory between two tiles).  Every wavefront fetches one page of a tile.
    static_assert(TILE == 64, "a wavefront per page");
    u32x4 rk[NCK], rv[NCK];
    int my_page = safe_page_lane(bt, 16 * lane, total, max_blocks, n_blocks);
    auto fetch = [&](int kb) {
        if ((kb & 1023) == 0 && kb > 0) my_page = safe_page_lane(bt, kb + 16 * lane, total, max_blocks, n_blocks);
        const size_t pofs = (size_t)__builtin_amdgcn_readlane(my_page, ((kb >> 4) & 63) + wave) * page_stride;
#pragma unroll
        for (int i = 0; i < NCK; i++) {
            rk[i] = *reinterpret_cast<const u32x4*>(kbase_ptr + pofs + (lane + 64 * i) * 8);
            rv[i] = *reinterpret_cast<const u32x4*>(vbase_ptr + pofs + (lane + 64 * i) * 8);
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NCK; i++) {
            const int c = lane + 64 * i;
            *reinterpret_cast<u32x4*>(&sK[buf * K_BUF + (wave * 16 + c / (HD / 8)) * KS + (c % (HD / 8)) * 8]) = rk[i];
            bf16_t* dst = &sV[buf * V_BUF + (c & 1) * 4];
            *reinterpret_cast<u32x2*>(dst + prefill_value_at(wave * HD + (c >> 1), 0)) = u32x2{rv[i].x, rv[i].y};
            *reinterpret_cast<u32x2*>(dst + prefill_value_at(wave * HD + (c >> 1), 1)) = u32x2{rv[i].z, rv[i].w};
        }
    };
    fetch(0);
    stage(0);
    if (TILE < k_end) fetch(TILE);
    __syncthreads();
    int buf = 0;
    for (int kbase = 0; kbase < k_end; kbase += TILE, buf ^= 1) {
        if (kbase + TILE < k_end) stage(buf ^ 1);
        if (kbase + 2 * TILE < k_end) fetch(kbase + 2 * TILE);
        if (rt_on && kbase < lim_max)          // wavefront-uniform: something of this tile is visible
            attn_tile64<HD>(sK + buf * K_BUF, sV + buf * V_BUF, qf, o, m_run, l_run, kbase, lim_min, lim_lane, scale_log2,
                            half, l32);
        __syncthreads();
    }
    if (!rt_on || rho >= R) return;
    const int node = rho / G, g = rho - node * G;
    const float inv = 1.f / l_run;     // a row always sees its own key: the sum is positive
    bf16_t* po = out + ((size_t)(r0 + node) * hq + j * G + g) * HD;
#pragma unroll
    for (int dt = 0; dt < NDT; dt++)
#pragma unroll
        for (int g4 = 0; g4 < 4; g4++) {
            u32x2 w;
            w.x = (uint32_t)f32_to_bf16(o[dt][4 * g4] * inv) | ((uint32_t)f32_to_bf16(o[dt][4 * g4 + 1] * inv) << 16);
            w.y = (uint32_t)f32_to_bf16(o[dt][4 * g4 + 2] * inv) | ((uint32_t)f32_to_bf16(o[dt][4 * g4 + 3] * inv) << 16);
            *reinterpret_cast<u32x2*>(po + dt * 32 + 8 * g4 + 4 * half) = w;
        }
}

// Combine the partitions of one (row, query head) in partition order: one wavefront per (row, head), four per
// workgroup; rows are strided over the grid's x dimension (the row count is only known on the device).  Lane p
// holds partition p's (max, sum); weights are broadcast from there.
// A chain of memory round trips per row: the number of partitions (one load, written once per pass; the next row's is asked
// for a row ahead), then the weights and the first eight partitions' outputs together, in 4-byte pieces of two elements.
// With few rows expected the first row's loads do not wait for the number of partitions either (up to max_parts, in bounds).
constexpr int HS_MERGE_EARLY_ROWS = 32;
template <int HD>
__global__ __launch_bounds__(256) void attn_merge(const _Float16* part_o, const float* part_ml,
                                                  const hs_row_info* infos, const int32_t* m_dev,
                                                  int max_parts, int max_rows, int hq, bf16_t* __restrict__ out, int expected) {
    constexpr int E = HD / 64, AHEAD = 8;      // elements of a lane: E * lane, ...
    typedef _Float16 piece __attribute__((ext_vector_type(E)));
    const int head = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (head >= hq) return;
    int row = blockIdx.x, lim = max_parts;
    if (row >= expected || expected > HS_MERGE_EARLY_ROWS) {
        if (row >= *m_dev) return;
        lim = max(infos[row].parts, 1);     // (a sequence without tokens has no partition: its first is read, and not used)
    }
    for (;;) {
        const unsigned zero = hs_opaque_zero();     // (all of a row's loads inside the loop: one in front of it would be waited for there)
        const int m_lane = m_dev[zero], parts_lane = infos[row + zero].parts;
        const int next = min(row + (int)gridDim.x, max_rows - 1);
        const size_t prow = ((size_t)row * hq + head) * max_parts;
        const float2* ml = reinterpret_cast<const float2*>(part_ml) + prow;
        const _Float16* po = part_o + prow * HD + E * lane;
        const float2 ml0 = ml[min(lane, lim - 1)];
        piece v[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; q++) v[q] = *reinterpret_cast<const piece*>(po + (size_t)min(q, lim - 1) * HD);
        const int next_lane = infos[next + zero].parts;
        hs_loads_issued();
        const int m = hs_uniform(m_lane), nparts = hs_uniform(parts_lane);
        if (row >= m) return;
        float mg = -INFINITY;
        for (int p0 = 0; p0 < nparts; p0 += 64) {
            float mp = p0 + lane < nparts ? (p0 == 0 ? ml0.x : ml[p0 + lane].x) : -INFINITY;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) mp = fmaxf(mp, __shfl_xor(mp, o));
            mg = fmaxf(mg, mp);
        }
        float den = 0.f, acc[E];
#pragma unroll
        for (int i = 0; i < E; i++) acc[i] = 0.f;
        for (int p0 = 0; p0 < nparts; p0 += 64) {
            float wl = 0.f, ll = 0.f;
            if (p0 + lane < nparts) {
                const float2 t = p0 == 0 ? ml0 : ml[p0 + lane];
                wl = fast_exp2(t.x - mg);
                ll = t.y;
            }
            const int n = min(64, nparts - p0);
            // partition order; the values of eight partitions are fetched before the first is added, so that the loop
            // waits for memory once per eight partitions instead of once per partition
            for (int pb = 0; pb < n; pb += AHEAD) {
                if (p0 + pb > 0) {
#pragma unroll
                    for (int q = 0; q < AHEAD; q++) v[q] = *reinterpret_cast<const piece*>(po + (size_t)(p0 + min(pb + q, n - 1)) * HD);
                }
#pragma unroll
                for (int q = 0; q < AHEAD; q++) {
                    if (pb + q < n) {
                        // the partition's weight in the whole: exp2(m_p - m) l_p; its output is stored normalised
                        const float w = __shfl(wl, pb + q) * __shfl(ll, pb + q);
                        den += w;
#pragma unroll
                        for (int i = 0; i < E; i++) acc[i] += w * (float)v[q][i];
                    }
                }
            }
        }
        bf16_t* dst = out + ((size_t)row * hq + head) * HD + E * lane;
        if constexpr (E == 2)
            *reinterpret_cast<uint32_t*>(dst) = (uint32_t)f32_to_bf16(acc[0] / den) | ((uint32_t)f32_to_bf16(acc[E - 1] / den) << 16);
        else
            *dst = f32_to_bf16(acc[0] / den);
        row += gridDim.x;
        if (row >= m) return;
        lim = max(hs_uniform(next_lane), 1);
    }
}

// Plain kernel for debugging and for the fp32-activation mode: one wavefront per (row, query head), keys visited one
// by one.  T = bf16_t (queries, cache and output are bf16; fp32 arithmetic) or float (nothing rounded below fp32, the
// running sum and output carried in fp64, library exponential).
__device__ __forceinline__ float plain_ld(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ float plain_ld(const float* p) { return *p; }
__device__ __forceinline__ void plain_st(bf16_t* p, double v) { *p = f32_to_bf16((float)v); }
__device__ __forceinline__ void plain_st(float* p, double v) { *p = (float)v; }

template <typename T, typename ACC>
__global__ __launch_bounds__(64) void attn_verify_plain(
    const T* __restrict__ q, const T* __restrict__ kc, const T* __restrict__ vc, size_t layer_off,
    const int32_t* __restrict__ seq_len, const int32_t* __restrict__ block_table, int max_blocks, int n_blocks,
    const int32_t* __restrict__ row_off, const int32_t* __restrict__ row2seq, const uint64_t* __restrict__ anc_mask,
    int batch, int hq, int hkv, int hd, float scale, T* __restrict__ out) {
    constexpr bool PRECISE = sizeof(ACC) == 8;
    int row = blockIdx.x, head = blockIdx.y, lane = threadIdx.x;
    if (row >= row_off[batch]) return;
    int b = row2seq[row];
    int L = seq_len[b] - 1, nn = row_off[b + 1] - row_off[b];
    int total = L + nn, j = head / (hq / hkv);
    uint64_t anc = anc_mask[row];
    const T* qp = q + ((size_t)row * hq + head) * hd;
    float q0 = lane < hd ? plain_ld(qp + lane) : 0.f;
    float q1 = lane + 64 < hd ? plain_ld(qp + lane + 64) : 0.f;
    ACC m = -INFINITY, l = 0, o0 = 0, o1 = 0;
    for (int kp = 0; kp < total; kp++) {
        bool vis = kp < L || ((anc >> (kp - L)) & 1ull);
        if (!vis) continue;
        if ((kp >> 4) >= max_blocks) break;
        int page = block_table[(size_t)b * max_blocks + (kp >> 4)];
        if (page < 0 || page >= n_blocks) break;
        int ip = kp & 15;
        const T* kr = kc + layer_off + (((size_t)page * hkv + j) * 16 + ip) * hd;
        ACC dot = 0;
        if (lane < hd) dot += (ACC)q0 * (ACC)plain_ld(kr + lane);
        if (lane + 64 < hd) dot += (ACC)q1 * (ACC)plain_ld(kr + lane + 64);
        if (PRECISE) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double dd = (double)dot;
                const int lo = __shfl_xor(__double2loint(dd), o), hi = __shfl_xor(__double2hiint(dd), o);
                dot += (ACC)__hiloint2double(hi, lo);
            }
        } else {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) dot += (ACC)__shfl_xor((float)dot, o);
        }
        ACC s = dot * (ACC)scale;
        ACC mn = s > m ? s : m;
        ACC a, p;
        if (PRECISE) { a = (ACC)exp((double)(m - mn)); p = (ACC)exp((double)(s - mn)); }
        else { a = (ACC)__expf((float)(m - mn)); p = (ACC)__expf((float)(s - mn)); }
        l = l * a + p;
        const T* vr = vc + layer_off + ((size_t)page * hkv + j) * hd * 16 + ip;
        float v0 = lane < hd ? plain_ld(vr + (size_t)lane * 16) : 0.f;
        float v1 = lane + 64 < hd ? plain_ld(vr + (size_t)(lane + 64) * 16) : 0.f;
        o0 = o0 * a + p * (ACC)v0;
        o1 = o1 * a + p * (ACC)v1;
        m = mn;
    }
    T* op = out + ((size_t)row * hq + head) * hd;
    if (lane < hd) plain_st(op + lane, (double)(o0 / l));
    if (lane + 64 < hd) plain_st(op + lane + 64, (double)(o1 / l));
}

template <int HD>
void launch_mfma(const hs_ctx* ctx, int layer, size_t layer_off, const hs_kv_cache* cache, const hs_seq_state* seq,
                 const hs_step* step, const bf16_t* q, hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    AttnArgs a;
    a.q = q;
    a.kc = (const bf16_t*)cache->k + layer_off;
    a.vc = (const bf16_t*)cache->v + layer_off;
    a.seq_len = seq->seq_len;
    a.block_table = seq->block_table;
    a.row_off = step->row_off;
    a.anc_mask = step->anc_mask;
    a.part_o = reinterpret_cast<_Float16*>(ctx->ws + ctx->lay.part_o);
    a.part_ml = reinterpret_cast<float*>(ctx->ws + ctx->lay.part_ml);
    a.max_blocks = ctx->lim.max_blocks_per_seq;
    a.n_blocks = cache->n_blocks;
    a.max_parts = ctx->max_parts;
    a.part_keys = ctx->att_part;
    a.hq = d.n_q_heads;
    a.hkv = d.n_kv_heads;
    a.scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
    int32_t* work = reinterpret_cast<int32_t*>(ctx->ws + ctx->lay.att_work);
    const int4* list_a = reinterpret_cast<const int4*>(ctx->ws + ctx->lay.att_list);
    const int4* list_b = list_a + 2 * hs_attention_max_units(ctx);
    // the wavefront units are dealt out statically: the grid is what is resident at once, no more
    static int per_cu = 0;
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)attn_verify_mfma<HD>, 256, 0) != hipSuccess ||
            n < 1)
            n = 1;
        per_cu = n < 2 ? n : 2;   // (a third would fit at head size 64: two toy layers are launches of idle workgroups then)
    }
    dim3 grid(ctx->n_cu * per_cu);
    hipLaunchKernelGGL((attn_verify_mfma<HD>), grid, dim3(256), 0, st, a, work, work + 2 + layer, list_a, list_b);
}

}  // namespace

void hs_launch_attention(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                         const hs_step* step, const void* q_any, void* out, hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    size_t layer_off = (size_t)layer * cache->n_blocks * d.n_kv_heads * 16 * d.head_dim;
    if (hs_plain_kernels(ctx)) {
        const dim3 grid(ctx->lim.max_rows, d.n_q_heads);
        const float scale = 1.f / sqrtf((float)d.head_dim);
        if (hs_fp32_activations(ctx))
            hipLaunchKernelGGL((attn_verify_plain<float, double>), grid, dim3(64), 0, st, (const float*)q_any,
                               (const float*)cache->k, (const float*)cache->v, layer_off, seq->seq_len,
                               seq->block_table, ctx->lim.max_blocks_per_seq, cache->n_blocks, step->row_off,
                               step->row2seq, step->anc_mask, seq->batch, d.n_q_heads, d.n_kv_heads, d.head_dim,
                               scale, (float*)out);
        else
            hipLaunchKernelGGL((attn_verify_plain<bf16_t, float>), grid, dim3(64), 0, st, (const bf16_t*)q_any,
                               (const bf16_t*)cache->k, (const bf16_t*)cache->v, layer_off, seq->seq_len,
                               seq->block_table, ctx->lim.max_blocks_per_seq, cache->n_blocks, step->row_off,
                               step->row2seq, step->anc_mask, seq->batch, d.n_q_heads, d.n_kv_heads, d.head_dim,
                               scale, (bf16_t*)out);
        return;
    }
    const bf16_t* q = (const bf16_t*)q_any;
    // one row tile per wavefront, two workgroups per compute unit, whatever the longest draft: a sequence with more
    // than 128 query rows per KV head comes as several units (see hs_worklist.h)
    if (d.head_dim == 128) launch_mfma<128>(ctx, layer, layer_off, cache, seq, step, q, st);
    else launch_mfma<64>(ctx, layer, layer_off, cache, seq, step, q, st);
}

size_t hs_attention_max_units(const hs_ctx* ctx) {
    // a sequence's (partition, KV head) pairs, times the groups of four row tiles its query rows can fill
    const int r_max = (ctx->desc.n_q_heads / ctx->desc.n_kv_heads) * (1 + ctx->lim.c_max * ctx->lim.k_max);
    return (size_t)ctx->lim.max_batch * ctx->max_parts * ctx->desc.n_kv_heads * ((r_max + 127) / 128);
}

hs_attn_lists hs_attention_lists(const hs_ctx* ctx) {
    const hs_model_desc& d = ctx->desc;
    hs_attn_lists l;
    l.work = reinterpret_cast<int32_t*>(ctx->ws + ctx->lay.att_work);
    l.list_a = reinterpret_cast<int4*>(ctx->ws + ctx->lay.att_list);
    l.list_b = l.list_a + 2 * hs_attention_max_units(ctx);
    l.part_keys = ctx->att_part;
    l.G = d.n_q_heads / d.n_kv_heads;
    l.hkv = d.n_kv_heads;
    l.max_parts = ctx->max_parts;
    l.n_layers = d.n_layers;
    return l;
}

void hs_launch_attention_prefill(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                                 const int32_t* len_plus1, const hs_step* step, const bf16_t* q, bf16_t* out, int chunk,
                                 hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    const size_t layer_off = (size_t)layer * cache->n_blocks * d.n_kv_heads * 16 * d.head_dim;
    const int G = d.n_q_heads / d.n_kv_heads;
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)d.head_dim);
    const int nx = (chunk * G + 127) / 128;
    const dim3 grid(nx * d.n_kv_heads * seq->batch);
    if (d.head_dim == 128)
        hipLaunchKernelGGL((attn_prefill_mfma<128>), grid, dim3(256), 0, st, q, (const bf16_t*)cache->k,
                           (const bf16_t*)cache->v, layer_off, len_plus1, seq->block_table,
                           ctx->lim.max_blocks_per_seq, cache->n_blocks, step->row_off, out, d.n_q_heads, d.n_kv_heads,
                           scale_log2, seq->batch, nx);
    else
        hipLaunchKernelGGL((attn_prefill_mfma<64>), grid, dim3(256), 0, st, q, (const bf16_t*)cache->k,
                           (const bf16_t*)cache->v, layer_off, len_plus1, seq->block_table,
                           ctx->lim.max_blocks_per_seq, cache->n_blocks, step->row_off, out, d.n_q_heads, d.n_kv_heads,
                           scale_log2, seq->batch, nx);
}

void hs_launch_attention_merge(const hs_ctx* ctx, const hs_seq_state* seq, const hs_step* step, void* out_any,
                               int expected, hipStream_t st) {
    if (hs_plain_kernels(ctx)) return;  // the plain kernel writes the final output itself
    bf16_t* out = (bf16_t*)out_any;
    const hs_model_desc& d = ctx->desc;
    const _Float16* part_o = reinterpret_cast<const _Float16*>(ctx->ws + ctx->lay.part_o);
    float* part_ml = reinterpret_cast<float*>(ctx->ws + ctx->lay.part_ml);
    const hs_row_info* infos = reinterpret_cast<const hs_row_info*>(ctx->ws + ctx->lay.row_info);
    dim3 grid(hs_row_grid(ctx, 256, (d.n_q_heads + 3) / 4), (d.n_q_heads + 3) / 4);
    if (d.head_dim == 128)
        hipLaunchKernelGGL((attn_merge<128>), grid, dim3(256), 0, st, part_o, part_ml, infos, step->row_off + seq->batch,
                           ctx->max_parts, ctx->lim.max_rows, d.n_q_heads, out, expected);
    else
        hipLaunchKernelGGL((attn_merge<64>), grid, dim3(256), 0, st, part_o, part_ml, infos, step->row_off + seq->batch,
                           ctx->max_parts, ctx->lim.max_rows, d.n_q_heads, out, expected);
}
