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
//   * What bounds it now: at up to 128 rows the weight stream (271 MB of gate/up weights in 50 us); at 220 rows LDS and
//     matrix cores in balance (counters: matrix cores busy 39 % of gate/up's cycles; 184 KB through LDS a tile are 1440
//     clocks, its MFMAs 1280), with a prologue and an epilogue that nothing overlaps; at 2176 rows LDS (65 to 70 %) and
//     matrix cores (62 to 67 %) at the 1.6 to 1.8 GHz that this load leaves the chip.  A third activation stage made
//     every shape slower (71 -> 77 us), the row pitch of the operands (55 to 65 lines of 128 bytes) is worth 5 % either way.
// SwiGLU pairs the gate and up rows of 16 output columns in one 32-row weight unit, so that both pre-activations of
// a column meet in one MFMA tile (lanes c and c+16).
#include <algorithm>
#include <type_traits>

#include "hs_gemm_common.h"
#include "hs_lanes.h"

using namespace hs_gemm_detail;

namespace {

constexpr int TILE_BYTES = 32 * ROW_BYTES;  // a 32-row tile of either operand, 64 deep: 4 KB

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
    int w_pre;   // the weight-only part of the prologue has been issued already (by the kernel, before M was known)
};

// The weight units of a wavefront group: group 0 multiplies units 0 .. NU0-1, group 1 the others.
template <int NU, int GRP>
struct wave_units {
    static constexpr int NU0 = (NU + 1) / 2, U0 = GRP ? NU0 : 0, N = GRP ? NU - NU0 : NU0;
};

// The 1 KB blocks of weight tile kt that a wavefront fetches: quarter `quad` of each of its group's units, into stage
// kt % SW of the weight ring.  (A SwiGLU unit holds 16 gate rows then the 16 up rows of the same columns, so a
// wavefront's blocks are all gate rows -- quarters 0, 1 -- or all up rows -- 2, 3.)
template <int NU, int MT, int SA, int SW, int GRP>
__device__ __forceinline__ void issue_weight_tile(const stream_args& p, const unsigned char* w_mine, unsigned smem_off,
                                                  const unsigned (&w_off)[wave_units<NU, GRP>::N], int quad, int kt) {
    constexpr int W_RING = SA * 4 * MT * TILE_BYTES, W_STAGE = NU * TILE_BYTES;
    const unsigned dst = smem_off + W_RING + (kt % SW) * W_STAGE + wave_units<NU, GRP>::U0 * TILE_BYTES + quad * 1024;
    const unsigned char* base = w_mine + (size_t)kt * ROW_BYTES;
#pragma unroll
    for (int j = 0; j < wave_units<NU, GRP>::N; j++) {
        if (p.w_once) load_to_lds_16_stream(base, w_off[j], dst + j * 4096);
        else load_to_lds_16(base, w_off[j], dst + j * 4096);
    }
}

// One K chunk of one row pass for a wavefront of group GRP that owns NMI live row tiles (0 = loads and barriers only).
template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW, int GRP, int NMI>
__device__ __forceinline__ void stream_chunk(const stream_args& p, unsigned char* smem, unsigned smem_off,
                                             const unsigned (&w_off)[wave_units<NU, GRP>::N], int quad, int lane) {
    static_assert(SA == 2 && SW > SA, "the wait counts are written for a two-stage activation ring and a longer weight ring");
    constexpr int A_STAGE = 4 * MT * TILE_BYTES, W_STAGE = NU * TILE_BYTES, W_RING = SA * A_STAGE;
    constexpr int NUW = wave_units<NU, GRP>::N, U0 = wave_units<NU, GRP>::U0;
    constexpr int NLW = NUW;      // 1 KB load instructions per weight tile and wavefront
    constexpr int NSA = 2 * MT;   // and at most this many per activation tile: row tiles GRP, GRP + 2, ...
    constexpr int NM = NMI > 0 ? NMI : 1;
    const int lrow = lane >> 3, lpos = lane & 7;
    const int l32 = lane & 31, g = lane >> 5, fl = swz(l32);
    const int frag_row = l32 * ROW_BYTES;
    const unsigned a_chunk = (unsigned)((lpos ^ swz(8 * quad + lrow)) << 4);
    const int a_row = p.m0 + 32 * GRP + 8 * quad + lrow;
    const unsigned row_pitch = (unsigned)p.K * 2u;
    // 8-row blocks of the activation tile this wavefront fetches: slot l covers rows 64 l + 32 GRP + 8 quad .. +7 of the
    // pass; blocks past the last row are not fetched.
    int n_a = 0;
#pragma unroll
    for (int l = 0; l < NSA; l++)
        if (p.m0 + 32 * GRP + 8 * quad + 64 * l < p.M) n_a = l + 1;
    n_a = __builtin_amdgcn_readfirstlane(n_a);
    unsigned a_off[NSA];
#pragma unroll
    for (int l = 0; l < NSA; l++) a_off[l] = (unsigned)min(a_row + 64 * l, p.M - 1) * row_pitch + a_chunk;
    const unsigned a_dst0 = smem_off + GRP * TILE_BYTES + quad * 1024;                       // + stage + l * 8192
    const unsigned w_dst0 = smem_off + W_RING + U0 * TILE_BYTES + quad * 1024;               // + stage + j * 4096

    auto issue_a = [&](int kt) {
        const unsigned char* base = p.A + (size_t)kt * ROW_BYTES;
#pragma unroll
        for (int l = 0; l < NSA; l++)
            if (l < n_a) load_to_lds_16(base, a_off[l], a_dst0 + (kt % SA) * A_STAGE + l * 8192);
    };
    const unsigned char* w_mine = uniform_ptr((EPI == HS_EPI_SWIGLU_BF16 && quad >= 2) ? p.wb[1] : p.wb[0]);
    auto issue_w = [&](int kt) { issue_weight_tile<NU, MT, SA, SW, GRP>(p, w_mine, smem_off, w_off, quad, kt); };
    // Hand-over number h (h < kt0 before the loop, then in the last quarter of tile h): first the activation tile h+SA,
    // then the weight tile h+SW.  The issue order fixes the wait counts below.
    auto issue_for = [&](int h) {
        if (h + SA >= p.kt0 && h + SA < p.kt1) issue_a(h + SA);
        if (h + SW >= p.kt0 && h + SW < p.kt1) issue_w(h + SW);
    };
    // Loads complete in issue order.  Tile t is awaited in tile t-1, when the hand-overs up to t-2 have been made.  Its
    // activation part was issued at hand-over t-2, its weight part at t-SW (earlier).  What may still be outstanding is
    // what was issued after the activation part: the weight tile of hand-over t-2, if there is one.
    auto wait_tile = [&](int t) {
        if (t - SA + SW < p.kt1) HS_WAIT_VMCNT(NLW);
        else HS_WAIT_VMCNT(0);
    };

    f32x16 acc[NM][NUW];
#pragma unroll
    for (int i = 0; i < NM; i++)
#pragma unroll
        for (int j = 0; j < NUW; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

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
    // fragment r (weight units, then row tiles) of k-step ks of the tile whose stages start at a / w: lane l reads tile
    // row l%32, k-chunk 2 ks + l/32, at its swizzled position
    auto frag = [&](int set, int r, int ks, int a, int w) __attribute__((always_inline)) {
        const int pos = ((2 * ks + g) ^ fl) << 4;
        if (r < NUW)
            fb[set][r < NUW ? r : 0] = *reinterpret_cast<const bf16x8*>(smem + W_RING + w + (U0 + r) * TILE_BYTES + frag_row + pos);
        else
            fa[set][r >= NUW ? r - NUW : 0] = *reinterpret_cast<const bf16x8*>(smem + a + (quad + 4 * (r - NUW)) * TILE_BYTES + frag_row + pos);
    };
    // One k-step in a pinned order: behind each MFMA of the step that is in set KS % 2 come its share of the next step's
    // fragment reads and of the NLD loads that `load(l)` issues.
    auto step = [&](auto ks_c, int a, int w, auto nld_c, auto load) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value, NLD = decltype(nld_c)::value, NMF = NM * NUW, NR = NM + NUW;
        constexpr int set = KS & 1, kr = (KS + 1) & 3;
#pragma unroll
        for (int q = 0; q < NMF; q++) {
            const int mi = q / NUW, ni = q % NUW;
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mi], fb[set][ni], acc[mi][ni], 0, 0, 0);
            if (a >= 0) {
#pragma unroll
                for (int r = q * NR / NMF; r < (q + 1) * NR / NMF; r++) frag(set ^ 1, r, kr, a, w);
            }
#pragma unroll
            for (int l = q * NLD / NMF; l < (q + 1) * NLD / NMF; l++) load(l);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto no_load = [](int) __attribute__((always_inline)) {};
    if (NMI > 0) {
#pragma unroll
        for (int r = 0; r < NM + NUW; r++) frag(0, r, 0, a_cur, w_cur);
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
        const unsigned w_dst = w_dst0 + w_prv;
        const int a_nxt = a_cur == 0 ? A_STAGE : 0;   // stage of tile kt+1
        auto load_w = [&](int l) __attribute__((always_inline)) {
            if (w_on) {
                if (p.w_once) load_to_lds_16_stream(w_src, w_off[l], w_dst + l * 4096);
                else load_to_lds_16(w_src, w_off[l], w_dst + l * 4096);
            }
        };
        int na_eff = G == 0 ? NSA : G == 2 ? n_a : (kt + SA < p.kt1 ? n_a : 0);
        if (G) asm volatile("" : "+s"(na_eff)); /* one scalar compare per slot, not a mask expression */
        auto load_a = [&](int l) __attribute__((always_inline)) {
            if (l < na_eff) load_to_lds_16(a_src, a_off[l], a_dst0 + a_cur + l * 8192);
        };
        if (NMI > 0) {
            step(std::integral_constant<int, 0>{}, a_cur, w_cur, std::integral_constant<int, NLW>{}, load_w);
            step(std::integral_constant<int, 1>{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
            step(std::integral_constant<int, 2>{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        } else {
#pragma unroll
            for (int l = 0; l < NLW; l++) load_w(l);
        }
        if (G == 1) wait_tile(kt + 1);
        else HS_WAIT_VMCNT(NLW);
        __builtin_amdgcn_s_waitcnt((63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8)); /* lgkmcnt(0) */
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (NMI > 0) {
            step(std::integral_constant<int, 3>{}, a_nxt, w_nxt, std::integral_constant<int, NSA>{}, load_a);
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
    };
    if (n_a == NSA) {
        for (; kt + SW < p.kt1; kt++) tile(std::integral_constant<int, 0>{});
    } else {
        for (; kt + SW < p.kt1; kt++) tile(std::integral_constant<int, 2>{});
    }
    for (; kt + 1 < p.kt1; kt++) tile(std::integral_constant<int, 1>{});
    // last tile of the chunk: nothing follows it
    if (NMI > 0) {
        step(std::integral_constant<int, 0>{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 1>{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 2>{}, a_cur, w_cur, std::integral_constant<int, 0>{}, no_load);
        step(std::integral_constant<int, 3>{}, -1, -1, std::integral_constant<int, 0>{}, no_load);
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
        constexpr int ROWS = 128 * MT;
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
                    if (lc == 0) wave_keys[GRP * ROWS + 32 * (quad + 4 * mi) + lr + 8 * (e >> 2) + (e & 3)] = key;
                }
            }
        }
        __syncthreads();
        const int row = GRP * 256 + quad * 64 + lane_e;     // within the pass
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
            const int row0 = p.m0 + 32 * (quad + 4 * mi) + lr;
            if (EPI == HS_EPI_SWIGLU_BF16) {
                // Lanes c (gate) and c+16 (up) hold the two pre-activations of output column c.  Elements are taken
                // in pairs: the gate lanes finish the row of element e and the up lanes the row of element e+1, so
                // every lane computes an output.  One v_permlane16_swap does the exchange: it swaps the odd
                // 16-lane rows of its first operand (element e: the up values) with the even rows of its second
                // (element e+1: the gate values), after which the first holds every lane's gate and the second
                // every lane's up.  (32-bit element offsets: the host checks that the output stays below 4 GiB.)
                bf16_t* C = reinterpret_cast<bf16_t*>(p.Cout);
                const bool up_lane = (lc & 16) != 0;
                const int rbase = row0 + (up_lane ? 1 : 0);
#pragma unroll
                for (int ni = 0; ni < NUW; ni++) {
                    const int col = p.n0 + 16 * (U0 + ni) + (lc & 15);
#pragma unroll
                    for (int e = 0; e < 16; e += 2) {
                        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[mi][ni][e]),
                                                                         __float_as_uint(acc[mi][ni][e + 1]), false, false);
                        const float gate = __uint_as_float(sw[0]), up = __uint_as_float(sw[1]);
                        const int row = rbase + 8 * (e >> 2) + (e & 3);
                        if (col < p.N && row < p.M) {
                            const float s = gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate));
                            C[(unsigned)row * (unsigned)p.N + (unsigned)col] = f32_to_bf16(s * up);
                        }
                    }
                }
            } else {
                float* C = PARTIAL ? p.part + (size_t)p.chunk * p.m_max * p.N : reinterpret_cast<float*>(p.Cout);
                // A row tile that lies wholly below M (all but the last one of a pass) is stored without row checks,
                // through a wavefront-uniform row pointer plus a 32-bit lane offset.
                const int tile_row = p.m0 + 32 * (quad + 4 * mi);
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

// What a wavefront of group GRP does: the row passes of its workgroup.
template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW, int GRP>
__device__ __forceinline__ void stream_group(stream_args& p, unsigned char* smem, unsigned smem_off, int quad, int lane,
                                             int pass, int n_pass) {
    constexpr int NUW = wave_units<NU, GRP>::N, U0 = wave_units<NU, GRP>::U0;
    // Weight loader geometry: instruction j of quarter w fills the 1 KB block of rows 8w..8w+7 of unit U0 + j; lane i
    // lands on row i/8, chunk position i%8 and therefore fetches chunk (i%8) ^ swz(row).  Rows beyond N are clamped to
    // the last valid row: their products are computed and never stored.
    // (32-bit byte offsets: the host checks that every operand stays below 4 GiB.)
    const int lrow = lane >> 3, lpos = lane & 7;
    unsigned w_off[NUW];
#pragma unroll
    for (int j = 0; j < NUW; j++) {
        const int row = 8 * quad + lrow;  // within the unit
        const int gn = (EPI == HS_EPI_SWIGLU_BF16) ? p.n0 + 16 * (U0 + j) + 8 * (quad & 1) + lrow : p.n0 + 32 * (U0 + j) + row;
        w_off[j] = (unsigned)min(gn, p.N - 1) * (unsigned)(p.K * 2) + ((lpos ^ swz(row)) << 4);
    }
    // The weight-only hand-overs of the first chunk's prologue go out now: they do not depend on the row count,
    // whose load from device memory (the kernel's first statement) is still on its way -- nothing has used it yet.
    {
        const unsigned char* w_mine = uniform_ptr((EPI == HS_EPI_SWIGLU_BF16 && quad >= 2) ? p.wb[1] : p.wb[0]);
#pragma unroll
        for (int h = -SW; h < -SA; h++)
            if (p.kt0 + h + SW < p.kt1) issue_weight_tile<NU, MT, SA, SW, GRP>(p, w_mine, smem_off, w_off, quad, p.kt0 + h + SW);
    }
    p.w_pre = 1;
    for (p.m0 = pass * 128 * MT; p.m0 < p.M; p.m0 += n_pass * 128 * MT) {
        int nmi = 0;
#pragma unroll
        for (int s = 0; s < MT; s++)
            if (p.m0 + 32 * (quad + 4 * s) < p.M) nmi = s + 1;
        nmi = __builtin_amdgcn_readfirstlane(nmi);
        if (nmi == 0) stream_chunk<EPI, PARTIAL, NU, MT, SA, SW, GRP, 0>(p, smem, smem_off, w_off, quad, lane);
        else if (nmi == 1) stream_chunk<EPI, PARTIAL, NU, MT, SA, SW, GRP, 1>(p, smem, smem_off, w_off, quad, lane);
        else if (MT >= 2 && nmi == 2)
            stream_chunk<EPI, PARTIAL, NU, MT, SA, SW, GRP, (MT >= 2 ? 2 : 1)>(p, smem, smem_off, w_off, quad, lane);
        else if (MT >= 3)
            stream_chunk<EPI, PARTIAL, NU, MT, SA, SW, GRP, (MT >= 3 ? 3 : 1)>(p, smem, smem_off, w_off, quad, lane);
        __syncthreads();  // the rings are reused by the next row pass
        p.w_pre = 0;
    }
    HS_WAIT_VMCNT(0);     // (a workgroup without rows leaves with its early weight loads landed)
}

}  // namespace

// NU weight units per workgroup, MT row tiles per wavefront pair (128*MT rows per pass), SA / SW ring stages.
// (External linkage: the host takes the kernel's address to raise its dynamic LDS limit.)
template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW>
__global__ __launch_bounds__(512) void hs_gemm_stream(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                      const bf16_t* __restrict__ W2, void* __restrict__ Cout,
                                                      float* __restrict__ part, const int32_t* __restrict__ m_dev,
                                                      int m_max, int N, int K, int tpc, int n_groups, int n_pass) {
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
    // Workgroup id -> (weight group, row pass): ids are dealt round-robin to the 8 XCDs (each with its own L2).
    // Unsplit K: an XCD takes a weight group and runs its row passes back to back, so that the passes which stream
    // the same weight slab meet in one L2.
    // (With a single pass the id is the group: no padding of the grid, a workgroup that only exits still has to
    // wait for a compute unit with this kernel's LDS free.)
    int group = blockIdx.x, pass = 0, chunk = blockIdx.y;
    if (gridDim.y > 1) {
        // Split-K: the workgroups that land on one XCD (ids congruent mod 8) take consecutive (chunk, group, pass)
        // triples, pass fastest, i.e. one or two K chunks -- the slices of the activations they re-read then fit that
        // XCD's L2 (all chunks together, e.g. 8 MB for the down projection at 220 rows and 27 MB at 720, do not), and
        // the row passes that stream the same weight slice run side by side.  (grid.x = groups x passes, no padding.)
        const int total = gridDim.x * gridDim.y, id = blockIdx.x + gridDim.x * blockIdx.y;
        const int xcd = id & 7, slot = id >> 3;
        const int full = total >> 3, extra = total & 7;          // XCDs 0 .. extra-1 hold one workgroup more
        const int w = xcd * full + min(xcd, extra) + slot;
        chunk = w / (int)gridDim.x;
        const int rem = w - chunk * (int)gridDim.x;
        group = rem / n_pass;
        pass = rem - group * n_pass;
    } else if (n_pass > 1) {
        const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
        group = (local / n_pass) * 8 + xcd;
        pass = local % n_pass;
    }
    if (group >= n_groups) return;
    p.n0 = group * NCOLS;
    p.group = group;
    p.n_groups = n_groups;
    p.chunk = chunk;
    p.w_once = n_pass == 1;
    const int nk = K / BK;
    p.kt0 = chunk * tpc;
    p.kt1 = min(nk, p.kt0 + tpc);

    if (wave < 4) stream_group<EPI, PARTIAL, NU, MT, SA, SW, 0>(p, smem, smem_off, wave, lane, pass, n_pass);
    else stream_group<EPI, PARTIAL, NU, MT, SA, SW, 1>(p, smem, smem_off, wave - 4, lane, pass, n_pass);
}

namespace {

template <int EPI, bool PARTIAL, int NU, int MT, int SA, int SW>
void launch_stream(const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part, const int32_t* m_dev,
                   int m_max, int n, int k, int chunks, int tpc, int rows_hint, hipStream_t st) {
    constexpr int NCOLS = (EPI == HS_EPI_SWIGLU_BF16) ? 16 * NU : 32 * NU;
    constexpr size_t lds = (size_t)(SA * 4 * MT + SW * NU) * TILE_BYTES;
    static_assert(lds <= 160 * 1024, "LDS of one compute unit");
    static bool configured = false;  // more than 64 KB of dynamic LDS has to be asked for once per kernel
    if (!configured) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&hs_gemm_stream<EPI, PARTIAL, NU, MT, SA, SW>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        configured = true;
    }
    // row passes in the grid: what the hint calls for (rows beyond are reached by the pass loop of the kernel)
    const int n_groups = (n + NCOLS - 1) / NCOLS;
    int n_pass = (rows_hint + 128 * MT - 1) / (128 * MT);
    if (n_pass < 1) n_pass = 1;
    if (n_pass > (m_max + 128 * MT - 1) / (128 * MT)) n_pass = (m_max + 128 * MT - 1) / (128 * MT);
    dim3 grid(chunks > 1 ? n_groups * n_pass : (n_pass > 1 ? ((n_groups + 7) / 8) * 8 * n_pass : n_groups), chunks);
    hipLaunchKernelGGL((hs_gemm_stream<EPI, PARTIAL, NU, MT, SA, SW>), grid, dim3(512), lds, st, a, w, w2, c, part,
                       m_dev, m_max, n, k, tpc, n_groups, n_pass);
}

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

template <int EPI, bool PARTIAL>
void launch_stream_shape(const bf16_t* a, const bf16_t* w, const bf16_t* w2, void* c, float* part,
                         const int32_t* m_dev, int m_max, int n, int k, int chunks, int tpc, int rows_hint,
                         hipStream_t st) {
    // Rows per pass: 256 leaves LDS for a deeper weight ring; 384 once the hint is within a factor 1.6 of 256 (the
    // row count of a speculative step swings by a third around its mean), so that a step above its average does
    // not pay a second pass over the weights.  Row tiles that do not exist cost nothing in either shape.
    const bool tall = rows_hint > 160;
    const int unit_cols = (EPI == HS_EPI_SWIGLU_BF16) ? 16 : 32, pass_rows = tall ? 384 : 256;
    const int passes = std::max(1, (std::min(rows_hint, m_max) + pass_rows - 1) / pass_rows);
    const int nu = EPI == HS_EPI_ROWMAX ? rowmax_units(n) : choose_units((n + unit_cols - 1) / unit_cols, chunks, passes);
#define HS_ARGS a, w, w2, c, part, m_dev, m_max, n, k, chunks, tpc, rows_hint, st
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
            else launch_stream<EPI, PARTIAL, 3, 2, 2, 7>(HS_ARGS);
        }
    } else {
        if (tall) launch_stream<EPI, PARTIAL, 4, 3, 2, 4>(HS_ARGS);
        else launch_stream<EPI, PARTIAL, 4, 2, 2, 5>(HS_ARGS);
    }
#undef HS_ARGS
}

}  // namespace

int hs_gemm_rowmax_groups(int n) {
    const int nu = rowmax_units(n);
    return (n + 32 * nu - 1) / (32 * nu);
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
