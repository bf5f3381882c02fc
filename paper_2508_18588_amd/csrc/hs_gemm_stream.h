// The bf16 MFMA GEMM of the projections:  C[M,N] (+)= A[M,K] . W[N,K]^T,  built for the row counts of a verify
// step (a few hundred draft-tree rows) and run in row passes for more (prefill, wide drafts).
//
// At a verify step's row count a projection is bound by streaming its weights from HBM exactly once, with the
// matrix cores needed at roughly half their rate just to keep up (220 rows: 220 flop per weight byte).  The kernel
// is laid out around the weight stream:
//   * One workgroup per (group of NU 32-row weight units, K chunk, row pass); unit and chunk counts are chosen by
//     the host so that one round of workgroups covers the 256 compute units.  A workgroup holds all rows of its
//     pass (up to 128*MT) against its weight slab, so with one pass every weight byte is fetched once.
//   * Eight wavefronts, two per SIMD: row tile t (32 rows) belongs to wavefronts t % 4 and 4 + t % 4, the first of which
//     multiplies it against the first half of the NU weight units, the second against the others.  A wavefront
//     multiplies only the row tiles that exist (M is read on the device); its accumulators stay in registers for the
//     whole chunk.
//   * Tiles (64 deep in K) travel from global memory straight into LDS (global_load_lds_dwordx4) through an
//     SA-stage activation ring and an SW-stage weight ring.
//   * A wavefront issues one instruction at a time, about one per eight clocks when it is alone on its SIMD, and an MFMA
//     takes 32: with four wavefronts (all units each, 28 instead of 36 KB of fragment reads per k-step at 220 rows) the
//     200 instructions of a tile's 40 MFMAs were what a tile took.  With a second wavefront on the SIMD to issue from,
//     every shape gains, those with few rows most (four 1.5B layers: 7 rows 320 -> 300 us, 264 rows 640 -> 605 us; a 7B
//     layer with its attention at 220 rows 679 -> 662 us, prefill of 8 x 4096 tokens 21.6 -> 20.3 ms; with the choice of
//     units below), same bits.
//   * The loop is software-pipelined over k-steps of 16: the fragments of step s+1 are read while step s is multiplied,
//     across tile boundaries, one by one behind single MFMAs, and the steady state carries no modulo arithmetic and as
//     few guards as possible.  The tile hand-over (wait for the loads of the next tile, workgroup barrier, issue of new
//     loads) sits before a tile's last k-step, after the last fragment read of the tile has been issued.
//   * A load's constant distances (weight unit, row tile, stage slot) lie in the instruction itself: one scalar add (into m0), a
//     nop and the load.  So do a fragment's, which then is one ds_read.  (With an address computation and a guard at each,
//     a tile of the four-wavefront kernel was 302 instructions for its 64 MFMAs and took 1.15 times as long as the
//     eight-wavefront one; at 188 it takes less.)  Only eight wavefronts with passes of 384 rows, which LDS binds, and fewer than five
//     units compute a fragment's address: it spaces their reads.  16448 columns of K = 3584, us at 256, 320, 352 and 384
//     rows: 47.6, 52.7, 58.2 and 60.7, as single instructions 49.0, 56.0, 60.6 and 62.8.  Five units are the same from 288 rows
//     on and gain with single instructions below: 152064 columns at 220 rows 285 -> 281; the 5 us of a split-K launch with few rows 0.1.
//   * Four wavefronts (hs_gemm_wide.hip) of 4 x 4 tiles, 256 rows x 8 units per workgroup, for many rows: a fragment is
//     used four times, not three or two and a half, so that an MFMA costs 0.75 instead of 1.07 KB through LDS, less of
//     the chip's power and fewer rounds of workgroups.  7B gate/up at 4096 rows 942 -> 890 us (1250 TFLOP/s), at 2048 rows
//     490 -> 446; down at 4096 674 -> 615.  Without its loads 816, without its MFMAs 628; counters: matrix cores busy 65 % of the
//     cycles at the 1.76 GHz that this load leaves the chip, LDS 32 %.
//   * Split K with many rows: a workgroup takes all chunks of its tile in turn (FOLD, hs_gemm_folded.hip), no partial sums.
//   * Up to 160 rows expected (three and four units): three activation stages, and one wavefront group fetches the activations,
//     the other the weights.  Loads count as landed in the order of their issue: while every wavefront fetched both, waiting for
//     the next tile's activations, asked for last, meant waiting for weights asked for a tile before, and the weight ring
//     was never more than that deep however many stages it had.  us, before and now: 1.5B gate/up at 7, 32, 64 and 100 rows
//     13.9, 15.2, 16.5, 17.9 -> 12.0, 13.0, 15.0, 17.5; 16448 columns of K = 3584 at 7, 32, 64 and 128 rows 23.4, 25.3, 31.0,
//     36.8 -> 22.1, 23.5, 27.0, 35.5; 14B gate/up at 7 and 32 rows 47.8, 52.2 -> 46.1, 50.1; 7B down at 64 rows 31.3 -> 30.2.
//     Two units (the shapes with short chunks of split K: 1.5B QKV, chunks of 4 tiles, would take 5.4 us instead of 5.1, its down
//     projection, of 14, the same either way), five units (42 us either way) and passes of 384 rows (two activation
//     stages are what LDS holds; 16448 columns at 217 rows 45.8, fetched apart 50.5) stay as they were.  From 96 rows on the gain
//     is what a shape makes of it: 16448 columns at 128 rows, K = 1536, 3584, 4096, 5120: 18.6, 38.7, 42.8, 54.2 -> 19.3, 38.2,
//     40.8, 55.7.  With more rows than expected, 217 to 990, nothing is lost (14B gate/up at 990: 339 -> 325).
//   * Passes of 64 rows (MT = 0) for up to 32 rows expected: another 1 to 5 %.
//   * What bounds it now: at up to 128 rows the weight stream (271 MB of gate/up weights in 50 us); from 160 rows on the two
//     operands' ways into a compute unit, one after the other (1.5B gate/up at 165 rows, clocks a tile: weights alone 880, activations
//     alone 820, both 1600, everything 1550, without either 1000); at 220 rows of a 7B shape LDS and the power they all draw (184 KB a
//     tile are 1440 clocks, its MFMAs 1280; without its loads the head takes 210 of 285 us, without its MFMAs 258; a
//     deeper weight ring changes nothing), with a prologue and an epilogue that nothing overlaps.  A third activation stage in
//     passes of 256 rows made every such shape slower (71 -> 77 us), the row pitch of the operands (55 to 65 lines of 128 bytes) is worth 5 % either way.
// SwiGLU pairs the gate and up rows of 16 output columns in one 32-row weight unit, so that both pre-activations of
// a column meet in one MFMA tile.
#pragma once
#include <algorithm>
#include <type_traits>

#include "hs_gemm_common.h"
#include "hs_lanes.h"

using namespace hs_gemm_detail;

namespace {

constexpr int TILE_BYTES = 32 * ROW_BYTES;  // a 32-row tile of either operand, 64 deep: 4 KB

// A fragment at an LDS byte address.
__device__ __forceinline__ bf16x8 lds_fragment(unsigned at) {
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(at);
}

// A pointer known to be the same in every lane, moved to scalar registers.
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (const unsigned char*)(((unsigned long long)hi << 32) | lo);
}

struct stream_args {
    const unsigned char* A;
    const unsigned char* wb[2];  // weight matrices (gate, up) or (W, W)
    void* Cout;
    float* part;
    int M, m_max, N, K, n0, m0, kt0, kt1, chunk, group, n_groups;
    int w_once;  // the launch reads every weight byte once (one row pass): non-temporal weight loads
    int fold;    // FOLD: k-tiles of a chunk
    int w_pre;   // the weight-only part of the prologue has been issued already (by the kernel, before M was known)
};

// Rows of a pass: 128 MT, or 64 (MT = 0).
template <int MT>
struct pass_shape {
    static constexpr int ROWS = MT ? 128 * MT : 64, TILES = ROWS / 32;
};

// The weight units of a wavefront group: group 0 multiplies units 0 .. NU0-1, group 1 the others.
template <int NU, int GRP>
struct wave_units {
    static constexpr int NU0 = (NU + 1) / 2, U0 = GRP ? NU0 : 0, N = GRP ? NU - NU0 : NU0;
};

// How the work of a workgroup lies on its WV wavefronts (8 or 4).  Two groups share the weight units; RG row groups share
// the row tiles (tile t: row group t % RG), at most MI of them each.  Each wavefront fetches quarter `quad` (8 of 32 rows, a
// 1 KB block) of weight units and row tiles: with eight wavefronts of its own group's units and of every second row
// tile, with four of all.  With three and more activation stages (eight wavefronts) the first group fetches the row tiles
// and the second the weight units: a wavefront's loads count as landed in the order they were issued, so where one
// wavefront fetches both, waiting for the activations of the next tile (an L2 away, asked for last) means waiting for the
// weights asked for just before them (a memory latency away) and the weight ring is never more than a tile deep.
template <int NU, int MT, int SA, int GRP, int WV>
struct wave_shape {
    static constexpr bool SPLIT = SA > 2;
    static_assert(!SPLIT || WV == 8, "four wavefronts fetch a quarter of everything each");
    static constexpr int RG = WV / 2, MI = (pass_shape<MT>::TILES + RG - 1) / RG;
    static constexpr bool OWN = WV == 8 && !SPLIT;                                                // own group's share of both
    static constexpr int FETCH_U0 = OWN ? wave_units<NU, GRP>::U0 : 0;
    static constexpr int FETCH_U = OWN ? wave_units<NU, GRP>::N : SPLIT && GRP == 0 ? 0 : NU;     // weight units fetched
    static constexpr int FETCH_A = SPLIT && GRP == 1 ? 0 : pass_shape<MT>::TILES / (OWN ? 2 : 1); // row tiles fetched ...
    static constexpr int FETCH_A0 = OWN ? GRP : 0, FETCH_AS = OWN ? 2 : 1;                         // ... first, stride
    static constexpr int U_SIZE = FETCH_U ? FETCH_U : 1, A_SIZE = FETCH_A ? FETCH_A : 1;          // (of arrays)
};

// The 1 KB blocks of weight tile kt that a wavefront fetches, into stage kt % SW of the weight ring.  (A SwiGLU unit holds 16
// gate rows then the 16 up rows of the same columns, so a wavefront's blocks are all gate rows -- quarters 0, 1 -- or all
// up rows -- 2, 3.)
template <int NU, int MT, int SA, int SW, int GRP, int WV>
__device__ __forceinline__ void issue_weight_tile(const stream_args& p, const unsigned char* w_mine, unsigned smem_off,
                                                  const unsigned (&w_off)[wave_shape<NU, MT, SA, GRP, WV>::U_SIZE], int quad, int kt) {
    constexpr int W_RING = SA * pass_shape<MT>::TILES * TILE_BYTES, W_STAGE = NU * TILE_BYTES;
    const unsigned dst = smem_off + W_RING + (kt % SW) * W_STAGE + wave_shape<NU, MT, SA, GRP, WV>::FETCH_U0 * TILE_BYTES + quad * 1024;
    const unsigned char* base = w_mine + (size_t)kt * ROW_BYTES;
#pragma unroll
    for (int j = 0; j < wave_shape<NU, MT, SA, GRP, WV>::FETCH_U; j++) {
        if (WV == 8 && p.w_once) load_to_lds_16_stream(base, w_off[j], dst, j * 4096);
        else load_to_lds_16(base, w_off[j], dst, j * 4096);
    }
}

// One K chunk (FOLD: all of them, p.fold k-tiles each) of one row pass for a wavefront of group GRP and row group rg that owns NMI live row tiles (0 = loads and
// barriers only).
template <int EPI, bool PARTIAL, bool FOLD, int NU, int MT, int SA, int SW, int GRP, int NMI, int WV>
__device__ __forceinline__ void stream_chunk(const stream_args& p, unsigned char* smem, unsigned smem_off,
                                             const unsigned (&w_off)[wave_shape<NU, MT, SA, GRP, WV>::U_SIZE], int quad, int rg, int lane) {
    using WS = wave_shape<NU, MT, SA, GRP, WV>;
    static_assert(SA >= 2 && SW > SA, "the wait counts below");
    constexpr int A_STAGE = pass_shape<MT>::TILES * TILE_BYTES, W_STAGE = NU * TILE_BYTES, W_RING = SA * A_STAGE;
    constexpr int NUW = wave_units<NU, GRP>::N, U0 = wave_units<NU, GRP>::U0;
    constexpr int NLW = WS::FETCH_U;   // 1 KB load instructions per weight tile and wavefront
    constexpr int NSA = WS::FETCH_A;   // and at most this many per activation tile
    constexpr int NM = NMI > 0 ? NMI : 1;
    const int lrow = lane >> 3, lpos = lane & 7;
    const int l32 = lane & 31, g = lane >> 5, fl = swz(l32);
    const int frag_row = l32 * ROW_BYTES;
    const unsigned a_chunk = (unsigned)((lpos ^ swz(8 * quad + lrow)) << 4);
    const int a_row = p.m0 + 32 * WS::FETCH_A0 + 8 * quad + lrow;
    const unsigned row_pitch = (unsigned)p.K * 2u;
    // 8-row blocks of the activation tile this wavefront fetches, one per row tile FETCH_A0, FETCH_A0 + FETCH_AS, ...; blocks
    // past the last row are not fetched.
    constexpr int A_ROWS = 32 * WS::FETCH_AS, A_BYTES = WS::FETCH_AS * TILE_BYTES;
    int n_a = 0;
#pragma unroll
    for (int l = 0; l < NSA; l++)
        if (p.m0 + 32 * WS::FETCH_A0 + 8 * quad + A_ROWS * l < p.M) n_a = l + 1;
    n_a = __builtin_amdgcn_readfirstlane(n_a);
    unsigned a_off[WS::A_SIZE];
#pragma unroll
    for (int l = 0; l < NSA; l++) a_off[l] = (unsigned)min(a_row + A_ROWS * l, p.M - 1) * row_pitch + a_chunk;
    const unsigned a_dst0 = smem_off + WS::FETCH_A0 * TILE_BYTES + quad * 1024;              // + stage + l * A_BYTES
    const unsigned w_dst0 = smem_off + W_RING + WS::FETCH_U0 * TILE_BYTES + quad * 1024;     // + stage + j * 4096

    auto issue_a = [&](int kt) {
        const unsigned char* base = p.A + (size_t)kt * ROW_BYTES;
#pragma unroll
        for (int l = 0; l < NSA; l++)
            if (l < n_a) load_to_lds_16(base, a_off[l], a_dst0 + (kt % SA) * A_STAGE, l * A_BYTES);
    };
    const unsigned char* w_mine = uniform_ptr((EPI == HS_EPI_SWIGLU_BF16 && quad >= 2) ? p.wb[1] : p.wb[0]);
    auto issue_w = [&](int kt) { if constexpr (NLW > 0) issue_weight_tile<NU, MT, SA, SW, GRP, WV>(p, w_mine, smem_off, w_off, quad, kt); };
    // Hand-over number h (h < kt0 before the loop, then in the last quarter of tile h): first the activation tile h+SA,
    // then the weight tile h+SW.  The issue order fixes the wait counts below.
    auto issue_for = [&](int h) {
        if (h + SA >= p.kt0 && h + SA < p.kt1) issue_a(h + SA);
        if (h + SW >= p.kt0 && h + SW < p.kt1) issue_w(h + SW);
    };
    // Loads complete in issue order.  Tile t is awaited in tile t-1, when the hand-overs up to t-2 have been made.  Its
    // activation part was issued at hand-over t-SA, its weight part at t-SW (earlier).  What may still be outstanding is
    // what the wavefront issued after the last of its own parts of tile t: where it fetches activations, the weight tiles of
    // hand-overs t-SA to t-2 and the activation tiles of t-SA+1 to t-2; where it fetches weights alone, the weight tiles of
    // hand-overs t-SW+1 to t-2; as far as there are such tiles.
    auto wait_tile = [&](int t) {
        int n = 0;
#pragma unroll
        for (int h = NSA ? -SA : -SW + 1; h <= -2; h++) {
            if (t + h + SW < p.kt1) n += NLW;
            if (h > -SA && t + h + SA < p.kt1) n += n_a;
        }
        static_assert((NSA ? (SA - 1) * NLW + (SA - 2) * NSA : (SW - 2) * NLW) <= 9, "the cases below");
        switch (n) {
#define HS_CASE(i) case i: HS_WAIT_VMCNT(i); break;
            HS_CASE(1) HS_CASE(2) HS_CASE(3) HS_CASE(4) HS_CASE(5) HS_CASE(6) HS_CASE(7) HS_CASE(8) HS_CASE(9)
#undef HS_CASE
            default: HS_WAIT_VMCNT(0);
        }
    };

    // A SwiGLU tile is computed transposed (weights as the first operand): a lane then holds a row's gate and up values of
    // the same columns, four columns in a row, and stores 8 bytes.  (As lanes c and c + 16 of a row, exchanged and stored by 2
    // bytes: 7B gate/up at 4096 rows 885 us, now 857, at 300 to 1000 rows 1 %, with fewer the same.)  Same products, same order, same bits.
    constexpr bool TRANSPOSED = EPI == HS_EPI_SWIGLU_BF16;
    f32x16 acc[NM][NUW];
#pragma unroll
    for (int i = 0; i < NM; i++)
#pragma unroll
        for (int j = 0; j < NUW; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
    // FOLD: the chunks of split K one after the other, their sums added left to right as the ordered reduce adds them.
    f32x16 sum[FOLD ? NM : 1][FOLD ? NUW : 1];
    int left = p.fold;      // k-tiles of the chunk still to come
    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < NM; i++)
#pragma unroll
            for (int j = 0; j < NUW; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) sum[i][j][e] = -0.f;    // (the first chunk's sum stays as it is)
    }
    auto fold = [&]() __attribute__((always_inline)) {
        if constexpr (FOLD) {
            if (--left == 0) {
                left = p.fold;
                if (NMI > 0) {
#pragma unroll
                    for (int i = 0; i < NM; i++)
#pragma unroll
                        for (int j = 0; j < NUW; j++)
#pragma unroll
                            for (int e = 0; e < 16; e++) { sum[i][j][e] += acc[i][j][e]; acc[i][j][e] = 0.f; }
                }
            }
        }
    };

    // prologue: the hand-overs a longer-running loop would have made before tile kt0; of the last one only the
    // activation part (its weight part goes out during the first half of tile kt0, see below)
    // (its first SW - SA hand-overs carry weight tiles only: the kernel issues those itself before it knows M)
#pragma unroll
    for (int h = -SW; h < -1; h++)
        if (h >= -SA || !p.w_pre) issue_for(p.kt0 + h);
    wait_tile(p.kt0);
    __builtin_amdgcn_s_barrier();
    if (p.kt0 - 1 + SA < p.kt1) issue_a(p.kt0 - 1 + SA);

    // Ring positions, kept incrementally: scalar instructions between MFMAs (a modulo, a guard, an address) are issued by
    // the same wavefront that should issue the next MFMA.
    int a_cur = (int)((unsigned)p.kt0 % SA) * A_STAGE;                   // stage of tile kt ...
    int w_cur = (int)((unsigned)p.kt0 % SW) * W_STAGE;
    int w_nxt = w_cur + W_STAGE == SW * W_STAGE ? 0 : w_cur + W_STAGE;   // ... and of tile kt+1
    int w_prv = w_cur == 0 ? (SW - 1) * W_STAGE : w_cur - W_STAGE;       // stage of tile kt-1 = of tile kt-1+SW
    const unsigned char* a_src = p.A + (size_t)(p.kt0 + SA) * ROW_BYTES;          // activation tile of hand-over kt
    const unsigned char* w_src = w_mine + (size_t)(p.kt0 - 1 + SW) * ROW_BYTES;   // weight tile of hand-over kt-1

    bf16x8 fa[2][NM], fb[2][NUW];
    // Fragment r (weight units, then row tiles) of the k-step whose addresses are at_a / at_w: lane l reads tile row l%32,
    // k-chunk 2 ks + l/32, at its swizzled position; units and row tiles are constant distances, within a read's offset.
    unsigned at_ks[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) at_ks[ks] = smem_off + frag_row + (((2 * ks + g) ^ fl) << 4);
    const int a_mine = rg * TILE_BYTES, w_mine_off = W_RING + U0 * TILE_BYTES;
    auto frag = [&](int set, int r, unsigned at_a, unsigned at_w) __attribute__((always_inline)) {
        if constexpr (WV == 4 || MT < 3 || NU == 5) {
            if (r < NUW) fb[set][r < NUW ? r : 0] = lds_fragment(at_w + r * TILE_BYTES);
            else fa[set][r >= NUW ? r - NUW : 0] = lds_fragment(at_a + WS::RG * (r - NUW) * TILE_BYTES);
        } else {
            if (r < NUW) fb[set][r < NUW ? r : 0] = *reinterpret_cast<const bf16x8*>(smem + (at_w - smem_off) + r * TILE_BYTES);
            else fa[set][r >= NUW ? r - NUW : 0] = *reinterpret_cast<const bf16x8*>(smem + (at_a - smem_off) + WS::RG * (r - NUW) * TILE_BYTES);
        }
    };
    // One k-step in a pinned order: behind each MFMA of the step that is in set KS % 2 come its share of the next step's
    // fragment reads and of the NLD loads that `load(l)` issues.
    // (a, w: the stages that the next step's fragments lie in; READ: there is a next step)
    auto step = [&](auto ks_c, auto read_c, int a, int w, auto nld_c, auto load) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value, NLD = decltype(nld_c)::value, NMF = NM * NUW, NR = NM + NUW;
        constexpr int set = KS & 1, kr = (KS + 1) & 3;
        constexpr bool READ = decltype(read_c)::value;
        const unsigned at_a = at_ks[kr] + (unsigned)(a + a_mine), at_w = at_ks[kr] + (unsigned)(w + w_mine_off);
#pragma unroll
        for (int q = 0; q < NMF; q++) {
            const int mi = q / NUW, ni = q % NUW;
            if (TRANSPOSED) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][ni], fa[set][mi], acc[mi][ni], 0, 0, 0);
            else acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mi], fb[set][ni], acc[mi][ni], 0, 0, 0);
            if (READ) {
#pragma unroll
                for (int r = q * NR / NMF; r < (q + 1) * NR / NMF; r++) frag(set ^ 1, r, at_a, at_w);
            }
#pragma unroll
            for (int l = q * NLD / NMF; l < (q + 1) * NLD / NMF; l++) load(l);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto no_load = [](int) __attribute__((always_inline)) {};
    if (NMI > 0) {
#pragma unroll
        for (int r = 0; r < NM + NUW; r++) frag(0, r, at_ks[0] + (unsigned)(a_cur + a_mine), at_ks[0] + (unsigned)(w_cur + w_mine_off));
    }
    __builtin_amdgcn_sched_barrier(0);
    int kt = p.kt0;
    // One tile of the k-loop.  k-steps 0 to 2, each reading the next step's fragments; meanwhile the weight blocks of
    // hand-over kt-1 (tile kt-1+SW, into the stage that tile kt-1 left).
    // Hand-over: every fragment read of tile kt has been issued; once they have returned (lgkmcnt) and all wavefronts have
    // met, the activation stage of tile kt is free to be refilled.  Tile kt+1 must have landed: each wavefront waits for
    // its own part before the barrier (a bare barrier: a fenced one would wait for the tiles in flight as well).
    // k-step 3 then reads the first fragments of tile kt+1 and issues the activation blocks of this hand-over (tile
    // kt+SA, into the stage of tile kt).
    // The steady state (kt + SW < kt1: every load of both parts exists, the wait count is a constant) comes in two forms:
    // G = 0 for a wavefront whose activation slots are all live (no guard at all), G = 2 with one guard per slot.  G = 1:
    // the last tiles, with every load guarded.
    auto tile = [&](auto g_c) __attribute__((always_inline)) {
        constexpr int G = decltype(g_c)::value;
        const bool w_on = G == 1 ? kt - 1 + SW < p.kt1 : true;
        const unsigned w_dst = w_dst0 + w_prv, a_dst = a_dst0 + a_cur;
        const int a_nxt = a_cur + A_STAGE == SA * A_STAGE ? 0 : a_cur + A_STAGE;   // stage of tile kt+1
        auto load_w = [&](int l) __attribute__((always_inline)) {
            if (w_on) {
                if (WV == 8 && p.w_once) load_to_lds_16_stream(w_src, w_off[l], w_dst, l * 4096);
                else load_to_lds_16(w_src, w_off[l], w_dst, l * 4096);
            }
        };
        int na_eff = G == 0 ? NSA : G == 2 ? n_a : (kt + SA < p.kt1 ? n_a : 0);
        if (G) asm volatile("" : "+s"(na_eff)); /* one scalar compare per slot, not a mask expression */
        auto load_a = [&](int l) __attribute__((always_inline)) {
            if (l < na_eff) load_to_lds_16(a_src, a_off[l], a_dst, l * A_BYTES);
        };
        if (NMI > 0) {
            step(std::integral_constant<int, 0>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, NLW>{}, load_w);
            step(std::integral_constant<int, 1>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
            step(std::integral_constant<int, 2>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        } else {
#pragma unroll
            for (int l = 0; l < NLW; l++) load_w(l);
        }
        if (G == 1) wait_tile(kt + 1);
        else if (!NSA) HS_WAIT_VMCNT((SW - 2) * NLW);
        else if (SA == 2) HS_WAIT_VMCNT(NLW);
        else if (G == 0) HS_WAIT_VMCNT((SA - 2) * NSA);
        else wait_tile(kt + 1);
        __builtin_amdgcn_s_waitcnt((63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8)); /* lgkmcnt(0) */
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (NMI > 0) {
            step(std::integral_constant<int, 3>{}, std::true_type{}, a_nxt, w_nxt, std::integral_constant<int, NSA>{}, load_a);
        } else {
#pragma unroll
            for (int l = 0; l < NSA; l++) load_a(l);
        }
        a_cur = a_nxt;
        w_prv = w_cur;
        w_cur = w_nxt;
        w_nxt = w_nxt + W_STAGE == SW * W_STAGE ? 0 : w_nxt + W_STAGE;
        a_src += ROW_BYTES;
        w_src += ROW_BYTES;
        fold();
    };
    if (n_a == NSA) {
        for (; kt + SW < p.kt1; kt++) tile(std::integral_constant<int, 0>{});
    } else {
        for (; kt + SW < p.kt1; kt++) tile(std::integral_constant<int, 2>{});
    }
    for (; kt + 1 < p.kt1; kt++) tile(std::integral_constant<int, 1>{});
    // last tile of the chunk: nothing follows it
    if (NMI > 0) {
        step(std::integral_constant<int, 0>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 1>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 2>{}, std::true_type{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 3>{}, std::false_type{}, 0, 0, std::integral_constant<int, 0>{}, no_load);
    }

    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < NM; i++)
#pragma unroll
            for (int j = 0; j < NUW; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[i][j][e] = sum[i][j][e] + acc[i][j][e];
    }

    // (the lane number anew: values derived from it would otherwise stay in registers, or spill, through the whole loop)
    int lane_e;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane_e));
    // Epilogue.  Accumulator element e of a 32x32 tile: row 8*(e/4) + 4*(lane/32) + e%4, column lane%32.
    if (EPI == HS_EPI_ROWMAX) {
        // Each row's largest value among this workgroup's columns, as a key that orders by value and then by lower column:
        // first over the lane's columns, then over the 32 lanes that hold the row, then over the two wavefronts that share
        // it: every wavefront leaves its keys in LDS (every fragment has been read), a thread per row takes the larger.
        // (152064 columns of K = 3584 at 220 and 2176 rows: one group after the other, with exchanges through the LDS unit,
        // 310 and 2276 us; as it is 276 and 1987; four wavefronts with all units each, 295 and 2105.)
        constexpr int ROWS = pass_shape<MT>::ROWS;
        unsigned long long* keys = reinterpret_cast<unsigned long long*>(p.Cout);
        unsigned long long* wave_keys = reinterpret_cast<unsigned long long*>(smem);   // [2][ROWS]
        const int lr = 4 * (lane_e >> 5), lc = lane_e & 31;
        __syncthreads();
        if (NMI > 0) {
#pragma unroll
            for (int mi = 0; mi < NMI; mi++) {
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    unsigned long long key = 0ull;
#pragma unroll
                    for (int ni = 0; ni < NUW; ni++) {
                        const int col = p.n0 + 32 * (U0 + ni) + lc;
                        unsigned u = __float_as_uint(acc[mi][ni][e]);
                        u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
                        const unsigned long long k2 = ((unsigned long long)u << 32) | (0xFFFFFFFFu - (unsigned)col);
                        if (col < p.N && k2 > key) key = k2;
                    }
                    auto take = [&](unsigned lo, unsigned hi) __attribute__((always_inline)) {
                        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
                        if (other > key) key = other;
                    };
                    take(lane_xor<16>((unsigned)key), lane_xor<16>((unsigned)(key >> 32)));
                    take(lane_xor<8>((unsigned)key), lane_xor<8>((unsigned)(key >> 32)));
                    take(lane_xor<4>((unsigned)key), lane_xor<4>((unsigned)(key >> 32)));
                    take(lane_xor<2>((unsigned)key), lane_xor<2>((unsigned)(key >> 32)));
                    take(lane_xor<1>((unsigned)key), lane_xor<1>((unsigned)(key >> 32)));
                    __builtin_amdgcn_sched_barrier(0);   // (one row at a time: the accumulators leave few registers)
                    if (lc == 0) wave_keys[GRP * ROWS + 32 * (rg + WS::RG * mi) + lr + 8 * (e >> 2) + (e & 3)] = key;
                }
            }
        }
        __syncthreads();
        const int row = (GRP * WS::RG + rg) * 64 + lane_e;  // within the pass
        if (row < ROWS && p.m0 + row < p.M) {
            const unsigned long long k0 = wave_keys[row], k1 = wave_keys[ROWS + row];
            keys[(size_t)(p.m0 + row) * p.n_groups + p.group] = k0 > k1 ? k0 : k1;
        }
        return;
    }
    if (NMI > 0) {
        const int lr = 4 * (lane_e >> 5), lc = lane_e & 31;
#pragma unroll
        for (int mi = 0; mi < NMI; mi++) {
            const int row0 = p.m0 + 32 * (rg + WS::RG * mi) + lr;
            if (EPI == HS_EPI_SWIGLU_BF16) {
                // Element e of the transposed tile: row of the weight unit 8*(e/4) + 4*(lane/32) + e%4, of which 0 to 15 are gate
                // rows and 16 to 31 the up rows of the same columns, activation row lane%32.  (32-bit element offsets: the
                // host checks that the output stays below 4 GiB.)
                bf16_t* C = reinterpret_cast<bf16_t*>(p.Cout);
                const int row = p.m0 + 32 * (rg + WS::RG * mi) + lc;
                const bool whole = (p.N & 3) == 0 && ((unsigned long long)C & 7ull) == 0;    // four columns end within N, 8-byte stores
                if (row < p.M) {
#pragma unroll
                    for (int ni = 0; ni < NUW; ni++) {
#pragma unroll
                        for (int q = 0; q < 2; q++) {
                            const int col = p.n0 + 16 * (U0 + ni) + 8 * q + lr;
                            bf16_t v[4];
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                const float gate = acc[mi][ni][4 * q + e], up = acc[mi][ni][8 + 4 * q + e];
                                const float s = gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate));
                                v[e] = f32_to_bf16(s * up);
                            }
                            bf16_t* dst = C + ((unsigned)row * (unsigned)p.N + (unsigned)col);
                            if (whole) {
                                if (col < p.N) *reinterpret_cast<uint2*>(dst) = make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; e++)
                                    if (col + e < p.N) dst[e] = v[e];
                            }
                        }
                    }
                }
            } else {
                float* C = PARTIAL ? p.part + (size_t)p.chunk * p.m_max * p.N : reinterpret_cast<float*>(p.Cout);
                // A row tile that lies wholly below M (all but the last one of a pass) is stored without row checks,
                // through a wavefront-uniform row pointer plus a 32-bit lane offset.
                const int tile_row = p.m0 + 32 * (rg + WS::RG * mi);
                unsigned char* tile = reinterpret_cast<unsigned char*>(C + (size_t)tile_row * p.N);
                __builtin_amdgcn_sched_barrier(0);
                const unsigned lane_bytes = ((unsigned)lr * (unsigned)p.N + (unsigned)(p.n0 + 32 * U0 + lc)) * 4u;
                if (tile_row + 32 <= p.M) {
#pragma unroll
                    for (int ni = 0; ni < NUW; ni++) {
                        if (p.n0 + 32 * (U0 + ni) + lc >= p.N) continue;
                        // (adding: all of a tile's loads before its first store -- element by element each load waited for
                        // the one before it, 17 us of a launch with 16 rows)
                        float old[16];
                        if (!PARTIAL && EPI == HS_EPI_ADD_F32) {
#pragma unroll
                            for (int e = 0; e < 16; e++)
                                old[e] = *reinterpret_cast<float*>(tile + (size_t)(8 * (e >> 2) + (e & 3)) * p.N * 4 +
                                                                   (lane_bytes + 128u * ni));
                        }
#pragma unroll
                        for (int e = 0; e < 16; e++) {
                            unsigned char* rowp = tile + (size_t)(8 * (e >> 2) + (e & 3)) * p.N * 4;
                            float* dst = reinterpret_cast<float*>(rowp + (lane_bytes + 128u * ni));
                            if (!PARTIAL && EPI == HS_EPI_ADD_F32) *dst = old[e] + acc[mi][ni][e];
                            else *dst = acc[mi][ni][e];
                        }
                    }
                } else {
#pragma unroll
                    for (int ni = 0; ni < NUW; ni++) {
                        const int col = p.n0 + 32 * (U0 + ni) + lc;
                        if (col >= p.N) continue;
                        float old[16];
                        if (!PARTIAL && EPI == HS_EPI_ADD_F32) {
#pragma unroll
                            for (int e = 0; e < 16; e++)   // (rows beyond M: the last row's element, not stored)
                                old[e] = C[(size_t)min(row0 + 8 * (e >> 2) + (e & 3), p.M - 1) * p.N + col];
                        }
#pragma unroll
                        for (int e = 0; e < 16; e++) {
                            const int row = row0 + 8 * (e >> 2) + (e & 3);
                            if (row < p.M) {
                                float* dst = &C[(size_t)row * p.N + col];
                                if (!PARTIAL && EPI == HS_EPI_ADD_F32) *dst = old[e] + acc[mi][ni][e];
                                else *dst = acc[mi][ni][e];
                            }
                        }
                    }
                }
            }
        }
    }
}

}  // namespace

namespace {

// What a 64-row instance falls back to: passes of 256 rows with the rings of the 256-row instance.  They need more LDS than its own
// rings, which are no deeper than this: with more on its way a launch takes longer (7 rows of 3584, head of 16448 columns, three
// units: 4 and 5 stages 22.1 us, 3 and 4 22.7, 5 and 6 22.9, 6 and 9 25.3).
template <int NU>
struct few_rows_fallback {
    static constexpr int SA = 3, SW = NU == 3 ? 5 : 4;
    static_assert(NU == 3 || NU == 4, "the 64-row instances");
};

// Weight stages of the four-wavefront kernel's smaller shares of a group's units: as many as LDS holds, at most 8.
template <int NU>
struct wide_share {
    static constexpr int SW = NU == 4 ? 6 : 8;
    static_assert((2 * pass_shape<2>::TILES + SW * NU) * TILE_BYTES <= 160 * 1024, "LDS of one compute unit");
};

// What a wavefront of group GRP does: the row passes of its workgroup.
template <int EPI, bool PARTIAL, bool FOLD, int NU, int MT, int SA, int SW, int GRP, int WV>
__device__ __forceinline__ void stream_group(stream_args& p, unsigned char* smem, unsigned smem_off, int quad, int rg, int lane,
                                             int pass, int n_pass) {
    using WS = wave_shape<NU, MT, SA, GRP, WV>;
    // Weight loader geometry: instruction j of quarter w fills the 1 KB block of rows 8w..8w+7 of unit FETCH_U0 + j; lane i
    // lands on row i/8, chunk position i%8 and therefore fetches chunk (i%8) ^ swz(row).  Rows beyond N are clamped to
    // the last valid row: their products are computed and never stored.
    // (32-bit byte offsets: the host checks that every operand stays below 4 GiB.)
    const int lrow = lane >> 3, lpos = lane & 7;
    unsigned w_off[WS::U_SIZE];
#pragma unroll
    for (int j = 0; j < WS::FETCH_U; j++) {
        const int row = 8 * quad + lrow, unit = WS::FETCH_U0 + j;  // (row within the unit)
        const int gn = (EPI == HS_EPI_SWIGLU_BF16) ? p.n0 + 16 * unit + 8 * (quad & 1) + lrow : p.n0 + 32 * unit + row;
        w_off[j] = (unsigned)min(gn, p.N - 1) * (unsigned)(p.K * 2) + ((lpos ^ swz(row)) << 4);
    }
    // The weight-only hand-overs of the first chunk's prologue go out now: they do not depend on the row count,
    // whose load from device memory (the kernel's first statement) is still on its way -- nothing has used it yet.
    if constexpr (WS::FETCH_U > 0) {
        const unsigned char* w_mine = uniform_ptr((EPI == HS_EPI_SWIGLU_BF16 && quad >= 2) ? p.wb[1] : p.wb[0]);
#pragma unroll
        for (int h = -SW; h < -SA; h++)
            if (p.kt0 + h + SW < p.kt1) issue_weight_tile<NU, MT, SA, SW, GRP, WV>(p, w_mine, smem_off, w_off, quad, p.kt0 + h + SW);
    }
    p.w_pre = 1;
    if constexpr (MT == 0) {
        // More rows than the hint let expect: passes of 256 after all (of 64 they would read the weights four times as often:
        // 16448 columns of K = 3584 with 990 rows 460 us, 185 in passes of 256).  The early loads land first, they lie elsewhere.
        if (p.M > pass_shape<0>::ROWS) {
            HS_WAIT_VMCNT(0);
            __syncthreads();
            p.w_pre = 0;
            stream_group<EPI, PARTIAL, FOLD, NU, 2, few_rows_fallback<NU>::SA, few_rows_fallback<NU>::SW, GRP, WV>(p, smem, smem_off, quad, rg, lane, pass, n_pass);
            return;
        }
    }
    for (p.m0 = pass * pass_shape<MT>::ROWS; p.m0 < p.M; p.m0 += n_pass * pass_shape<MT>::ROWS) {
        int nmi = 0;
#pragma unroll
        for (int s = 0; s < WS::MI; s++)
            if (rg + WS::RG * s < pass_shape<MT>::TILES && p.m0 + 32 * (rg + WS::RG * s) < p.M) nmi = s + 1;
        nmi = __builtin_amdgcn_readfirstlane(nmi);
#define HS_CHUNK(N) stream_chunk<EPI, PARTIAL, FOLD, NU, MT, SA, SW, GRP, (N <= WS::MI ? N : 1), WV>(p, smem, smem_off, w_off, quad, rg, lane)
        if (nmi == 0) HS_CHUNK(0);
        else if (nmi == 1) HS_CHUNK(1);
        else if (WS::MI >= 2 && nmi == 2) HS_CHUNK(2);
        else if (WS::MI >= 3 && nmi == 3) HS_CHUNK(3);
        else if (WS::MI >= 4) HS_CHUNK(4);
#undef HS_CHUNK
        __syncthreads();  // the rings are reused by the next row pass
        p.w_pre = 0;
    }
    HS_WAIT_VMCNT(0);     // (a workgroup without rows leaves with its early weight loads landed)
}

}  // namespace

namespace {

// The kernel, for WV wavefronts.  (FOLD: a single grid row, tpc k-tiles per chunk; with up to split_rows rows the workgroups take the
// chunks one each and leave partial sums.)
template <int EPI, bool PARTIAL, bool FOLD, int NU, int MT, int SA, int SW, int WV>
__device__ __forceinline__ void stream_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                              const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                              float* __restrict__ part, const int32_t* __restrict__ m_dev,
                                              int m_max, int N, int K, int tpc, int n_groups, int n_pass, int split_rows = 0) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const unsigned smem_off = (unsigned)(size_t)(lds_ptr_t)smem;
    constexpr int NCOLS = (EPI == HS_EPI_SWIGLU_BF16) ? 16 * NU : 32 * NU;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    stream_args p;
    p.M = *m_dev;
    p.A = reinterpret_cast<const unsigned char*>(A);
    p.wb[0] = reinterpret_cast<const unsigned char*>(W);
    p.wb[1] = reinterpret_cast<const unsigned char*>(EPI == HS_EPI_SWIGLU_BF16 ? W2 : W);
    p.Cout = Cout;
    p.part = part;
    p.m_max = m_max;
    p.N = N;
    p.K = K;
    const int nk = K / BK;
    if constexpr (FOLD) {
        p.M = __builtin_amdgcn_readfirstlane(p.M);
        if (p.M <= split_rows) {
            // (chunk, group, pass) triples, pass fastest, an XCD's workgroups taking consecutive ones (as split K below)
            const int live = (p.M + pass_shape<MT>::ROWS - 1) / pass_shape<MT>::ROWS, per_chunk = n_groups * live;
            const int total = per_chunk * ((nk + tpc - 1) / tpc), full = total >> 3, extra = total & 7;
            const int xcd = blockIdx.x & 7, share = full + (xcd < extra ? 1 : 0);
            p.n_groups = n_groups;
            p.w_once = live == 1;
            for (int nth = blockIdx.x >> 3; nth < share; nth += gridDim.x >> 3) {
                const int w = xcd * full + min(xcd, extra) + nth, rem = w % per_chunk;
                p.chunk = w / per_chunk;
                p.group = rem / live;
                p.n0 = p.group * NCOLS;
                p.kt0 = p.chunk * tpc;
                p.kt1 = min(nk, p.kt0 + tpc);
                if (wave < 4) stream_group<HS_EPI_STORE_F32, true, false, NU, MT, SA, SW, 0, 8>(p, smem, smem_off, wave, wave, lane, rem % live, live);
                else stream_group<HS_EPI_STORE_F32, true, false, NU, MT, SA, SW, 1, 8>(p, smem, smem_off, wave - 4, wave - 4, lane, rem % live, live);
            }
            return;
        }
    }
    // Workgroup id -> (weight group, row pass): ids are dealt round-robin to the 8 XCDs (each with its own L2).
    // Unsplit K: an XCD takes a weight group and runs its row passes back to back, so that the passes which stream
    // the same weight slab meet in one L2.
    // (With a single pass the id is the group: no padding of the grid, a workgroup that only exits still has to
    // wait for a compute unit with this kernel's LDS free.)
    // Four wavefronts: there may be fewer rows than the hint let expect (or there was none).  Then the first ids take the
    // passes that have rows -- ids n_pass apart would lie on a few of the chip's shader engines -- and the others share their
    // units, in halves or quarters of a group, where that takes less time: by rounds of 256 workgroups, each units + 3 (with
    // 2 to 6 the choice is within 1 % of the best of the three, 64 to 1536 rows of the 1.5B and 7B shapes with hints of 3000).
    // us at hints of 990 and of 2048 or more, before there was this kernel / with every pass in its place and whole / now: 14B
    // gate/up at 64 rows 56, 105 / 150, 84 / 55, 55, at 220 rows 83, 146 / 203, 111 / 79, 79; 7B down at 220 rows 60, 65 /
    // 95, 96 / 45, 46; QKV 23, 28 / 37, 38 / 24, 25.  (For this the count is waited for first, half a microsecond.)
    int passes = n_pass, units = NU;
    if constexpr (WV == 4) {
        p.M = __builtin_amdgcn_readfirstlane(p.M);
        const int live = (p.M + pass_shape<MT>::ROWS - 1) / pass_shape<MT>::ROWS, wgs = n_groups * (int)gridDim.y * live;
        if (live <= 0) return;
        if (live < n_pass) {
            auto cost = [&](int u) { return (wgs * (NU / u) + 255) / 256 * (u + 3); };
            if (live * 2 <= n_pass && cost(NU / 2) < cost(units)) units = NU / 2;
            if (live * 4 <= n_pass && cost(NU / 4) < cost(units)) units = NU / 4;
            passes = live;
        }
    }
    const int slots = passes * (NU / units);    // workgroups of a group: its passes, then its other shares' ...
    int group = blockIdx.x, slot = 0, chunk = blockIdx.y;
    if (gridDim.y > 1) {
        // Split-K: the workgroups that land on one XCD (ids congruent mod 8) take consecutive (chunk, group, pass)
        // triples, pass fastest, i.e. one or two K chunks -- the slices of the activations they re-read then fit that
        // XCD's L2 (all chunks together, e.g. 8 MB for the down projection at 220 rows and 27 MB at 720, do not), and
        // the row passes that stream the same weight slice run side by side.  (grid.x = groups x passes, no padding.)
        const int per_chunk = n_groups * slots, total = per_chunk * gridDim.y, id = blockIdx.x + gridDim.x * blockIdx.y;
        const int xcd = id & 7, nth = id >> 3;
        const int full = total >> 3, extra = total & 7;          // XCDs 0 .. extra-1 hold one workgroup more
        if (WV == 4 && nth >= full + (xcd < extra ? 1 : 0)) return;
        const int w = xcd * full + min(xcd, extra) + nth;
        chunk = w / per_chunk;
        const int rem = w - chunk * per_chunk;
        group = rem / slots;
        slot = rem - group * slots;
    } else if (n_pass > 1) {
        // (With many passes four groups side by side, the passes one after the other: the 32 workgroups of an XCD then share
        // the operand tiles of 8 passes and 4 groups, 12 of them, where 16 passes and 2 groups are 18: 152064 columns of K = 3584 at 2176 rows, stored, 1966 -> 1897 us.)
        const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, per_xcd = (n_groups + 7) >> 3;
        if (WV == 4 && local >= per_xcd * slots) return;
        const int side = slots >= 8 || 2 * passes <= n_pass ? 4 : 1, first = local / (side * slots) * side, n_side = min(side, per_xcd - first);
        const int rem = local - first * slots;
        slot = side > 1 ? rem / n_side : rem;
        group = (first + (side > 1 ? rem - slot * n_side : 0)) * 8 + xcd;
    }
    if (group >= n_groups) return;
    const int share = WV == 4 && units < NU ? slot / passes : 0, pass = slot - share * passes;
    p.n0 = group * NCOLS + share * units * (NCOLS / NU);
    if (WV == 4 && p.n0 >= N) return;
    p.group = group;
    p.n_groups = n_groups;
    p.chunk = chunk;
    p.w_once = n_pass == 1;
    p.kt0 = FOLD ? 0 : chunk * tpc;
    p.kt1 = FOLD ? nk : min(nk, p.kt0 + tpc);
    p.fold = tpc;

    if constexpr (WV == 8) {
        if (wave < 4) stream_group<EPI, PARTIAL, FOLD, NU, MT, SA, SW, 0, 8>(p, smem, smem_off, wave, wave, lane, pass, passes);
        else stream_group<EPI, PARTIAL, FOLD, NU, MT, SA, SW, 1, 8>(p, smem, smem_off, wave - 4, wave - 4, lane, pass, passes);
    } else {
        auto run = [&](auto nu_c, auto sw_c) __attribute__((always_inline)) {
            constexpr int U = decltype(nu_c)::value, S = decltype(sw_c)::value;
            if (wave < 2) stream_group<EPI, PARTIAL, FOLD, U, MT, SA, S, 0, 4>(p, smem, smem_off, wave, wave, lane, pass, passes);
            else stream_group<EPI, PARTIAL, FOLD, U, MT, SA, S, 1, 4>(p, smem, smem_off, wave, wave - 2, lane, pass, passes);
        };
        if (units == NU) run(std::integral_constant<int, NU>{}, std::integral_constant<int, SW>{});
        else if (units == NU / 2) run(std::integral_constant<int, NU / 2>{}, std::integral_constant<int, wide_share<NU / 2>::SW>{});
        else run(std::integral_constant<int, NU / 4>{}, std::integral_constant<int, wide_share<NU / 4>::SW>{});
    }
}

}  // namespace

namespace {

// Launches a kernel of the shape <EPI, NU, MT, SA, SW>.
template <int EPI, int NU, int MT, int SA, int SW, int THREADS, typename Kernel, typename... More>
void launch_shape(Kernel kernel, bool& configured, const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                  const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st, More... more) {
    constexpr int NCOLS = (EPI == HS_EPI_SWIGLU_BF16) ? 16 * NU : 32 * NU, ROWS = pass_shape<MT>::ROWS;
    constexpr size_t rings = (size_t)(SA * pass_shape<MT>::TILES + SW * NU) * TILE_BYTES;
    size_t lds = rings;
    if constexpr (MT == 0) {
        constexpr size_t fallback = (size_t)(few_rows_fallback<NU>::SA * pass_shape<2>::TILES + few_rows_fallback<NU>::SW * NU) * TILE_BYTES;
        static_assert(rings <= fallback && fallback <= 160 * 1024, "LDS of one compute unit");
        lds = fallback;
    }
    static_assert(rings <= 160 * 1024, "LDS of one compute unit");
    if (!configured) {      // more than 64 KB of dynamic LDS has to be asked for once per kernel
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        configured = true;
    }
    // row passes in the grid: what the hint calls for (rows beyond are reached by the pass loop of the kernel)
    const int n_groups = (n + NCOLS - 1) / NCOLS;
    int n_pass = (rows_hint + ROWS - 1) / ROWS;
    if (n_pass < 1) n_pass = 1;
    if (n_pass > (m_max + ROWS - 1) / ROWS) n_pass = (m_max + ROWS - 1) / ROWS;
    dim3 grid(chunks > 1 ? n_groups * n_pass : (n_pass > 1 ? ((n_groups + 7) / 8) * 8 * n_pass : n_groups), chunks);
    hipLaunchKernelGGL(kernel, grid, dim3(THREADS), lds, st, a, w, w2, c, part, m_dev, m_max, n, k, tpc, n_groups, n_pass, more...);
}

}  // namespace

// The same work in workgroups of 256 rows x 8 weight units (hs_gemm_wide.hip).
void hs_launch_gemm_wide(int epi, bool partial, const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                         const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st);
