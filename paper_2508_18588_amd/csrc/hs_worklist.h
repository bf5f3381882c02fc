// The unit lists of the verify attention and the rows' places, written on the device once per hs_verify call.
#pragma once
#include "hs_internal.h"

constexpr int HS_LIST_THREADS = 1024;   // most threads of a workgroup that writes
// workgroups of `threads` that write the lists: 256 wavefronts in all
static inline int hs_list_groups(int threads) { return 256 * 64 / threads; }

// A unit = one partition of one (sequence, KV head), in (sequence, partition, head) order.  List A: units of sequences
// with more than 32 query rows per KV head (taken by whole workgroups), list B: the others (taken by single wavefronts).
// An entry is two int4: (sequence, head, partition, first row) (rows, cached length, first row tile, 0).  work[0] = |A|,
// work[1] = |B|, work[2 + l] = the counter through which layer l's launch hands out list A (zeroed here).
// Called by `groups` workgroups: each computes every sequence's place in the lists (a
// prefix sum over the batch), a wavefront then writes the units of one sequence.  These workgroups are part of the launch
// that gathers the embeddings, which needs nothing of the lists: one workgroup of four wavefronts in a launch of its own
// took 8 us at 64 sequences, 14 at 128 and 26 at 256, with the rest of the chip idle.
__device__ inline void hs_write_worklist(const hs_attn_lists& l, const hs_row_places& pl, const int32_t* __restrict__ seq_len,
                                         const int32_t* __restrict__ row_off, int batch, int group, int groups) {
    constexpr int NW_MAX = HS_LIST_THREADS / 64;
    const int nt = blockDim.x, nw = nt >> 6;
    __shared__ int s_nu[HS_LIST_THREADS], s_off[HS_LIST_THREADS], s_r0[HS_LIST_THREADS], s_nn[HS_LIST_THREADS],
        s_len[HS_LIST_THREADS];
    __shared__ int sw_a[NW_MAX], sw_b[NW_MAX];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (group == 0)
        for (int i = tid; i < l.n_layers; i += nt) l.work[2 + i] = 0;
    int carry_a = 0, carry_b = 0;
    for (int b0 = 0; b0 < batch; b0 += nt) {
        const int b = b0 + tid;
        int nu = 0, r0 = 0, nn = 0, L = 0;
        bool is_a = false;
        if (b < batch) {
            r0 = row_off[b];
            nn = row_off[b + 1] - r0;
            L = seq_len[b] - 1;
            if (nn > 0 && L >= 0) {
                const int nparts = min(l.max_parts, (L + nn + l.part_keys - 1) / l.part_keys);
                is_a = nn * l.G > 32;
                // a workgroup covers four 32-row tiles: a sequence with more query rows per KV head than that gets one
                // unit per group of four tiles (each walks the partition's keys on its own)
                nu = nparts * l.hkv * (is_a ? (nn * l.G + 127) / 128 : 1);
            }
        }
        const int va = is_a ? nu : 0, vb = is_a ? 0 : nu;
        int ia = va, ib = vb;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int ta = __shfl_up(ia, o), tb = __shfl_up(ib, o);
            if (lane >= o) { ia += ta; ib += tb; }
        }
        __syncthreads();   // the previous round's arrays have been read
        if (lane == 63) { sw_a[wave] = ia; sw_b[wave] = ib; }
        __syncthreads();
        int ba = carry_a, bb = carry_b;
        for (int w = 0; w < nw; w++) {
            if (w < wave) { ba += sw_a[w]; bb += sw_b[w]; }
            carry_a += sw_a[w];
            carry_b += sw_b[w];
        }
        // the sign of s_nu tells the list: positive = B, negative = A
        s_nu[tid] = is_a ? -nu : nu;
        s_off[tid] = is_a ? ba + ia - va : bb + ib - vb;
        s_r0[tid] = r0;
        s_nn[tid] = nn;
        s_len[tid] = L;
        __syncthreads();
        const int nb = min(nt, batch - b0);
        for (int i = group * nw + wave; i < nb; i += groups * nw) {
            const int n = s_nu[i], rows = s_nn[i];
            const int parts = min(l.max_parts, (s_len[i] + rows + l.part_keys - 1) / l.part_keys);
            for (int r = lane; r < rows; r += 64)
                pl.info[s_r0[i] + r] = hs_place_row(pl.block_table + (size_t)(b0 + i) * pl.max_blocks, pl.max_blocks, pl.n_blocks,
                                                    pl.max_pos, s_len[i] + r, pl.pos[s_r0[i] + r], parts);
            int4* dst = (n < 0 ? l.list_a : l.list_b) + 2 * (size_t)s_off[i];
            const int cnt = n < 0 ? -n : n, grp = n < 0 ? (rows * l.G + 127) / 128 : 1;
            for (int u = lane; u < cnt; u += 64) {
                // v = (partition, head); the tile groups of one (partition, head) are neighbours (grp is 1 or 2: at most
                // 256 query rows per KV head)
                const int v = grp == 1 ? u : (grp == 2 ? (u >> 1) : u / grp);
                dst[2 * u] = make_int4(b0 + i, v % l.hkv, v / l.hkv, s_r0[i]);
                dst[2 * u + 1] = make_int4(rows, s_len[i], 4 * (u - v * grp), 0);
            }
        }
    }
    if (group == 0 && tid == 0) { l.work[0] = carry_a; l.work[1] = carry_b; }
}
