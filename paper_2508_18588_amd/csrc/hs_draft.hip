// History-drafted speculation, draft side (Sec. 5.2 and 5.4 of the paper): every in-flight response looks for
// the longest suffix of its committed tokens (at most `window`, at least `m_min` tokens) inside its previous-epoch
// response and takes the tokens that follow as its draft.
//
// Kernel 1 (scan): one workgroup per (history segment, candidate), or for several segments in turn.  The segment plus a
// `window`-token halo is staged in LDS with coalesced loads; every thread then tests end positions p against the pattern,
// and the best (match length, leftmost p) is reduced with wavefront shuffles as one packed 64-bit key.  Kernel 2 (build):
// one thread per sequence reduces the segment winners, applies the draft-length policy
// and finds the candidates' shared prefix, a workgroup-wide prefix sum over node counts yields the ragged row offsets,
// and the rows of the token trees are written a node per lane.
#include <mutex>

#include "hs_internal.h"
#include "hs_lanes.h"

namespace {

__device__ inline unsigned long long shfl_xor_u64(unsigned long long v, int o) {
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    lo = __shfl_xor(lo, o);
    hi = __shfl_xor(hi, o);
    return ((unsigned long long)hi << 32) | lo;
}

// key = (match length << 32) | ~p : larger is better, ties -> smaller p.  COUNT: bits 40 and up hold how many places of
// the segment reach that match length (draft_key_len / draft_key_count take it apart).
__device__ inline int draft_key_len(unsigned long long k) { return (int)((k >> 32) & 0xFFu); }
__device__ inline int draft_key_count(unsigned long long k) { return (int)(k >> 40); }

// Bound by reading the histories, and by what a workgroup waits for before it can: offsets and lengths (asked for
// together), then the tokens (all in flight at once, in registers), then LDS.  A workgroup takes the segments blockIdx.x,
// blockIdx.x + gridDim.x, ... of its history, the next one's tokens on their way while it compares the current one.
// 2048 histories of 2k to 16k tokens (75 MB, 12 us at the rate of a plain read): 25 -> 20 us; 128 sequences with up to
// 16k tokens, a workgroup per segment: 5.8 -> 5.3 us.  A cap at 64 registers for eight workgroups per compute unit
// instead of five: 22 us.
template <bool COUNT>
__global__ __launch_bounds__(256) void draft_scan_kernel(const int32_t* __restrict__ hist,
                                                          const int32_t* __restrict__ hist_off, int n_cand,
                                                          const int32_t* __restrict__ tail,
                                                          const int32_t* __restrict__ tail_len,
                                                          const int32_t* __restrict__ budget_left, int w_max,
                                                          int window, int m_min, int max_segs,
                                                          unsigned long long* __restrict__ best) {
    __shared__ __attribute__((aligned(16))) int32_t sh[HS_DRAFT_SEG + 32 + 8];
    __shared__ int32_t pat[32];
    __shared__ unsigned long long red[4];
    __shared__ int red_cnt[4];
    const int bc = blockIdx.y, b = bc / n_cand;
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned long long* dst = best + (size_t)bc * max_segs;
    const int32_t* newest = tail + (size_t)b * w_max + (w_max - 1);
    // all asked for before any is used
    const int off = hist_off[bc], g_end = hist_off[bc + 1], n_tail = tail_len[b], left = budget_left[b];
    const int pat0 = newest[0];
    const int lh = g_end - off;
    const int n_pat = min(min(n_tail, window), w_max);
    // segments with a place to test (end positions p run from 1 to lh - 1); none if nothing is looked for
    const bool looks = left > 0 && n_pat >= m_min && n_pat > 0;
    const int n_seg = looks ? min(max_segs, (lh - 1 + HS_DRAFT_SEG - 1) / HS_DRAFT_SEG) : 0;
    for (int seg = max(n_seg, 0) + tid; seg < max_segs; seg += 256)
        if (seg % (int)gridDim.x == (int)blockIdx.x) dst[seg] = 0ull;
    if ((int)blockIdx.x >= n_seg) return;
    // tokens hist[base .. p_hi) of a segment are needed: base = p_lo - window (clamped).  They are fetched with 16-byte
    // loads from the 16-byte boundary at or below the first token: LDS entry `shift` + i holds hist[off + base + i].
    // (Tokens in front of that boundary belong to this or the previous history: in bounds, never compared.  Up to three
    // tokens of a vector that would reach past this history's end are loaded one by one.)
    constexpr int NV = (HS_DRAFT_SEG + 32 + 3 + 4 * 256 - 1) / (4 * 256);
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    i32x4 r[NV] = {};
    int32_t r_end = 0;
    auto fetch = [&](int seg) {
        const int p_lo = seg * HS_DRAFT_SEG + 1, p_hi = min((seg + 1) * HS_DRAFT_SEG, lh - 1);
        const int base = max(0, p_lo - window), a0 = (off + base) & ~3, n = off + p_hi - a0;
        const int n_vec = min((n + 3) & ~3, (g_end - a0) & ~3);
#pragma unroll
        for (int j = 0; j < NV; j++)
            if (4 * (tid + 256 * j) < n_vec) r[j] = *reinterpret_cast<const i32x4*>(hist + a0 + 4 * (tid + 256 * j));
        if (n_vec + tid < n && tid < 4) r_end = hist[a0 + n_vec + tid];
    };
    fetch(blockIdx.x);
    // pattern, newest token first: pat[i] = i-th token from the end
    if (tid < n_pat) pat[tid] = newest[-tid];
    for (int seg = blockIdx.x; seg < n_seg; seg += gridDim.x) {
        const int p_lo = seg * HS_DRAFT_SEG + 1;                   // end positions handled here: [p_lo, p_hi]
        const int p_hi = min((seg + 1) * HS_DRAFT_SEG, lh - 1);
        const int base = max(0, p_lo - window), a0 = (off + base) & ~3, n = off + p_hi - a0;
        const int n_vec = min((n + 3) & ~3, (g_end - a0) & ~3);
        if (seg != (int)blockIdx.x) __syncthreads();               // the previous segment has been compared
#pragma unroll
        for (int j = 0; j < NV; j++)
            if (4 * (tid + 256 * j) < n_vec) *reinterpret_cast<i32x4*>(&sh[4 * (tid + 256 * j)]) = r[j];
        if (n_vec + tid < n && tid < 4) sh[n_vec + tid] = r_end;
        __syncthreads();
        if (seg + (int)gridDim.x < n_seg) fetch(seg + gridDim.x);
        const int32_t* shb = sh + off - a0;              // shb[i] = hist[off + i]
        // a match ends with the pattern's newest token: sixteen places per thread are tested for it at once
        // (places past p_hi read LDS entries that nothing was staged to; they are masked)
        int32_t t[HS_DRAFT_SEG / 256];
#pragma unroll
        for (int i = 0; i < HS_DRAFT_SEG / 256; i++) t[i] = shb[p_lo - 1 + tid + 256 * i];
        unsigned hits = 0u;
#pragma unroll
        for (int i = 0; i < HS_DRAFT_SEG / 256; i++)
            hits |= ((p_lo + tid + 256 * i <= p_hi) & (t[i] == pat0)) ? 1u << i : 0u;
        unsigned long long k = 0ull;
        int cnt = 0;   // places that reach the length in k
        for (; hits; hits &= hits - 1) {
            const int p = p_lo + tid + 256 * (__ffs(hits) - 1);
            const int lim = min(n_pat, p);
            int m = 1;
            while (m < lim && shb[p - 1 - m] == pat[m]) m++;
            if (m >= m_min) {
                unsigned long long cand = ((unsigned long long)m << 32) | (0xFFFFFFFFu - (unsigned)p);
                if (COUNT) cnt = (cand >> 32) > (k >> 32) ? 1 : cnt + ((cand >> 32) == (k >> 32));
                if (cand > k) k = cand;
            }
        }
        if (__any(k != 0ull)) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                unsigned long long other = shfl_xor_u64(k, o);
                if (COUNT) {
                    const int oc = __shfl_xor(cnt, o);
                    cnt = (other >> 32) > (k >> 32) ? oc : (other >> 32) == (k >> 32) ? cnt + oc : cnt;
                }
                if (other > k) k = other;
            }
        }
        if (lane == 0) { red[tid >> 6] = k; red_cnt[tid >> 6] = cnt; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 4; w++) {
                if (COUNT)
                    cnt = (red[w] >> 32) > (k >> 32) ? red_cnt[w] : (red[w] >> 32) == (k >> 32) ? cnt + red_cnt[w] : cnt;
                if (red[w] > k) k = red[w];
            }
            dst[seg] = COUNT && k ? k | ((unsigned long long)cnt << 40) : k;
        }
    }
}

// Workgroups per history: all of its segments side by side, unless there are more histories than that fills the chip with
// (eight workgroups per compute unit; 2048 histories of up to 5 segments take 19.6 us with one each, 21.5 with five); no
// more than eight segments in turn, so that one long history does not keep the others waiting.
int hs_scan_groups(const hs_ctx* ctx, int histories) {
    const int fill = (8 * ctx->n_cu + histories - 1) / histories, most = (ctx->max_segs + 7) / 8;
    return min(ctx->max_segs, max(fill, most));
}

// Exclusive prefix sum over a workgroup of NT threads: wavefront scans by shuffles, then the wavefront totals.
template <int NT>
__device__ inline int block_excl_scan(int v, int* total, int* sw) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    __syncthreads();
    if (lane == 63) sw[wave] = inc;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; w++) {
        if (w < wave) before += sw[w];
        sum += sw[w];
    }
    *total = sum;
    return before + inc - v;
}

constexpr int BUILD_THREADS = 1024;   // one workgroup for the batch: sixty-four sequences' rows are written at a time

__global__ __launch_bounds__(BUILD_THREADS) void draft_build_kernel(
    const int32_t* __restrict__ hist, const int32_t* __restrict__ hist_off, int n_cand, int batch,
    const unsigned long long* __restrict__ best, int max_segs, const int32_t* __restrict__ seq_len,
    const int32_t* __restrict__ tail, int w_max, const int32_t* __restrict__ k_state,
    const int32_t* __restrict__ budget_left, hs_policy pol, int max_blocks, int max_pos, int max_rows,
    int32_t* __restrict__ draft_start, int32_t* __restrict__ match_len, int32_t* __restrict__ draft_len,
    int32_t* __restrict__ row_off, int32_t* __restrict__ tok, int32_t* __restrict__ pos,
    int32_t* __restrict__ parent, uint64_t* __restrict__ anc_mask, int32_t* __restrict__ row2seq,
    uint32_t* __restrict__ err, int group_n, const int32_t* __restrict__ draft_src, int32_t* __restrict__ gate,
    const unsigned long long* __restrict__ counters) {
    // group_n > 0: the draft of sequence b was chosen by the group walk (response draft_src[b] of its group_n
    // responses, start draft_start[b], length draft_len[b]); this kernel then only lays out the rows (n_cand == 1)
    __shared__ int sw[BUILD_THREADS / 64];
    __shared__ int carry_s;
    __shared__ int live_s, spec_on_s;
    // what the row writers need of each sequence: first row, nodes, tokens of either chain, their start, shared prefix
    __shared__ int s_r0[BUILD_THREADS], s_nn[BUILD_THREADS], s_len[BUILD_THREADS], s_tok[BUILD_THREADS], s_k0[BUILD_THREADS],
        s_h0[BUILD_THREADS], s_h1[BUILD_THREADS], s_sh[BUILD_THREADS];
    if (threadIdx.x == 0) { carry_s = 0; live_s = 0; spec_on_s = 1; }
    __syncthreads();
    if (gate) {
        // Throughput-aware speculation control (Sec. 5.4, last paragraph): one decision per step for the whole batch.
        // The monitor takes the previous step's drafted / accepted tokens from the counters hs_kv_commit keeps.
        int live = 0;
        for (int b = threadIdx.x; b < batch; b += BUILD_THREADS) live += budget_left[b] > 0;
        if (live) atomicAdd(&live_s, live);
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t dt = (uint32_t)counters[1], at = (uint32_t)counters[2];
            const uint32_t d = dt - (uint32_t)gate[5], a = at - (uint32_t)gate[6];
            gate[5] = (int32_t)dt;
            gate[6] = (int32_t)at;
            gate[0] = gate[0] - (gate[0] >> 3) + (int32_t)d;
            gate[1] = gate[1] - (gate[1] >> 3) + (int32_t)a;
            const int steps_off = (gate[7] > 0 && gate[3] == 0) ? gate[2] + 1 : 0;
            int bucket = 16;
            if (gate[0] > 0) {
                const long long q = (long long)gate[1] * 16 / gate[0];
                bucket = q > 16 ? 16 : (int)q;
            }
            const int on = live_s <= gate[HS_GATE_TABLE + bucket] || (gate[4] > 0 && steps_off >= gate[4]);
            gate[2] = steps_off;
            gate[3] = on;
            gate[7] += 1;
            spec_on_s = on;
        }
        __syncthreads();
    }
    const bool spec_on = spec_on_s != 0;
    for (int b0 = 0; b0 < batch; b0 += BUILD_THREADS) {
        const int b = b0 + threadIdx.x;
        int nn = 0, L = 0;
        int pstart[2] = {-1, -1}, klen[2] = {0, 0}, hoff[2] = {0, 0};
        int shared = 0;
        if (b < batch && budget_left[b] > 0) {
            L = seq_len[b] - 1;
            if (group_n > 0) {
                const int g = draft_src[b];
                pstart[0] = draft_start[b];
                klen[0] = (g >= 0 && spec_on) ? draft_len[b] : 0;
                hoff[0] = g >= 0 ? hist_off[b * group_n + g] + pstart[0] : 0;
            }
            for (int c = 0; c < n_cand && group_n == 0; c++) {
                const int bc = b * n_cand + c;
                const int off = hist_off[bc], lh = hist_off[bc + 1] - off;
                unsigned long long k = 0ull;
                const int nseg = (lh - 1 + HS_DRAFT_SEG - 1) / HS_DRAFT_SEG;
                for (int s = 0; s < nseg && s < max_segs; s++) {
                    unsigned long long v = best[(size_t)bc * max_segs + s];
                    if (v > k) k = v;
                }
                int m = (int)(k >> 32);
                int p = m > 0 ? (int)(0xFFFFFFFFu - (unsigned)(k & 0xFFFFFFFFull)) : -1;
                int kk = 0;
                if (m > 0) {
                    if (pol.k_mode == HS_K_FIXED) kk = pol.k_fixed;
                    else if (pol.k_mode == HS_K_MATCHLEN) kk = m < 1 ? 1 : m;
                    else kk = k_state[b];
                    kk = min(kk, pol.k_max);
                    kk = min(kk, lh - p);
                    kk = min(kk, budget_left[b] - 1);
                    kk = max(kk, 0);
                    if (!spec_on) kk = 0;
                }
                pstart[c] = p; klen[c] = kk; hoff[c] = off + (p < 0 ? 0 : p);
                draft_start[bc] = p;
                match_len[bc] = m;
            }
            if (n_cand == 2) {
                int lim = min(klen[0], klen[1]);
                while (shared < lim && hist[hoff[0] + shared] == hist[hoff[1] + shared]) shared++;
            }
            nn = 1 + klen[0] + (n_cand == 2 ? klen[1] - shared : 0);
            // capacity: every node needs a cache slot L + i and a rotary position below max_pos
            int cap_tokens = max_blocks * 16;
            if (L < 0 || L + 1 > cap_tokens || L + 1 > max_pos) {
                atomicOr(err, L + 1 > max_pos ? HS_DEV_POSITION_OVERFLOW : HS_DEV_BLOCK_TABLE_OVERFLOW);
                nn = 0; klen[0] = klen[1] = 0; shared = 0;
            } else if (L + nn > cap_tokens || L + 1 + max(klen[0], klen[1]) > max_pos) {
                atomicOr(err, L + nn > cap_tokens ? HS_DEV_BLOCK_TABLE_OVERFLOW : HS_DEV_POSITION_OVERFLOW);
                nn = 1; klen[0] = klen[1] = 0; shared = 0;
            }
            for (int c = 0; c < n_cand; c++) draft_len[b * n_cand + c] = klen[c];
        } else if (b < batch) {
            for (int c = 0; c < n_cand; c++) {
                draft_start[b * n_cand + c] = -1;
                match_len[b * n_cand + c] = 0;
                draft_len[b * n_cand + c] = 0;
            }
        }
        int total;
        int excl = block_excl_scan<BUILD_THREADS>(nn, &total, sw);
        int carry = carry_s;
        int r0 = carry + excl;
        if (b < batch) {
            if (r0 + nn > max_rows) { atomicOr(err, HS_DEV_ROW_OVERFLOW); nn = 0; }
            row_off[b] = r0;
            s_r0[threadIdx.x] = r0;
            s_nn[threadIdx.x] = nn;
            s_len[threadIdx.x] = L;
            s_tok[threadIdx.x] = tail[(size_t)b * w_max + (w_max - 1)];
            s_k0[threadIdx.x] = klen[0];
            s_h0[threadIdx.x] = hoff[0];
            s_h1[threadIdx.x] = hoff[1];
            s_sh[threadIdx.x] = shared;
        }
        __syncthreads();
        // The rows, a node per lane and sixteen lanes per sequence: candidate 0's chain (nodes 1 .. k0), then candidate 1's
        // nodes after the shared prefix, hanging off node `shared`.  (A thread per sequence that wrote its nodes one by one
        // waited for the history once per node: 8.0 -> 5.5 us for 128 chains of up to 16.)
        for (int i = threadIdx.x >> 4; i < min(BUILD_THREADS, batch - b0); i += BUILD_THREADS / 16) {
            const int k0 = s_k0[i], sh = s_sh[i], row0 = s_r0[i];
            for (int node = threadIdx.x & 15; node < s_nn[i]; node += 16) {
                const bool main = node <= k0;
                const int depth = main ? node : node - k0 + sh;
                const int row = row0 + node;
                tok[row] = node == 0 ? s_tok[i] : hist[(main ? s_h0[i] : s_h1[i]) + depth - 1];
                pos[row] = s_len[i] + depth;
                parent[row] = main ? node - 1 : (node == k0 + 1 ? sh : node - 1);
                // ancestors: the chain so far, or the shared prefix and the second chain's own nodes
                anc_mask[row] = main ? (2ull << node) - 1ull
                                     : ((2ull << sh) - 1ull) | (((2ull << node) - 1ull) & ~((2ull << k0) - 1ull));
                row2seq[row] = b0 + i;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int total = carry_s;
        if (total > max_rows) {
            // Only with limits that hs_create does not admit (max_rows < max_batch * nodes): the first sequence that
            // does not fit and every one after it get no rows, consistently for the kernels that read row_off.
            int cut = -1;
            for (int b = 0; b < batch; b++) {
                const int end = b + 1 < batch ? row_off[b + 1] : total;
                if (cut < 0 && end > max_rows) cut = row_off[b];
                if (cut >= 0 && b + 1 < batch) row_off[b + 1] = cut;
            }
            total = cut;
        }
        row_off[batch] = total;
    }
}


// ---- reward-aware draft over all responses of the prompt's last rollout (Sec. 5.3) ----
//
// The paper keeps one suffix tree per prompt over the responses of its last rollout, with a priority on every node
// (the summed rewards of the responses whose text runs through it), and follows the highest-priority child where
// the continuations of the matched pattern branch.  On the GPU the tree is never built: the scan kernel above finds
// the longest match in every response segment; this kernel, one workgroup per sequence, collects the occurrences of
// that longest pattern in (response, position) order and lets them vote, draft token by draft token, for their
// next token with their response's reward (ties: more votes, then the smaller token id).  Occurrences that voted
// for another token, or ran out of text, drop out.  The draft is the text after the first surviving occurrence.
constexpr int HS_OCC_MAX = 1024;  // occurrences kept per sequence (in order); part of the rule, see the header

__device__ inline unsigned long long block_max_u64(unsigned long long v, unsigned long long* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long other = shfl_xor_u64(v, o);
        if (other > v) v = other;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned long long r = red[0];
    for (int w = 1; w < 4; w++) if (red[w] > r) r = red[w];
    return r;
}

// Over a wavefront, by moves that stay out of the LDS unit: the walk is a chain of these.
template <int O>
__device__ __forceinline__ void take_larger(unsigned long long& v) {
    const unsigned long long other = ((unsigned long long)lane_xor<O>((unsigned)(v >> 32)) << 32) | lane_xor<O>((unsigned)v);
    if (other > v) v = other;
}
__device__ __forceinline__ unsigned long long lanes_max_u64(unsigned long long v) {
    take_larger<32>(v); take_larger<16>(v); take_larger<8>(v); take_larger<4>(v); take_larger<2>(v); take_larger<1>(v);
    return v;
}
__device__ __forceinline__ int lanes_min(int v) {
    v = min(v, (int)lane_xor<32>((unsigned)v));
    v = min(v, (int)lane_xor<16>((unsigned)v));
    v = min(v, (int)lane_xor<8>((unsigned)v));
    v = min(v, (int)lane_xor<4>((unsigned)v));
    v = min(v, (int)lane_xor<2>((unsigned)v));
    return min(v, (int)lane_xor<1>((unsigned)v));
}

__global__ __launch_bounds__(256) void draft_group_walk_kernel(
    const int32_t* __restrict__ hist, const int32_t* __restrict__ hist_off, const int32_t* __restrict__ reward,
    int n_resp, const unsigned long long* __restrict__ best, int max_segs, const int32_t* __restrict__ tail,
    const int32_t* __restrict__ tail_len, int w_max, const int32_t* __restrict__ k_state,
    const int32_t* __restrict__ budget_left, hs_policy pol, int32_t* __restrict__ draft_start,
    int32_t* __restrict__ match_len, int32_t* __restrict__ draft_len, int32_t* __restrict__ draft_src) {
    __shared__ int32_t pat[32];
    __shared__ int32_t occ_off[HS_OCC_MAX];   // offset in `hist` of the token that follows the occurrence
    __shared__ int32_t occ_end[HS_OCC_MAX];   // end offset of its response
    __shared__ int32_t occ_rew[HS_OCC_MAX];
    __shared__ int32_t occ_resp[HS_OCC_MAX];  // which response
    __shared__ int32_t occ_tok[HS_OCC_MAX];   // this step's vote; -2 = live but out of text, -1 = dropped out
    __shared__ unsigned long long red[4];
    __shared__ int sw[4];
    __shared__ int n_occ_s, n_multi_s, first_s, len_s;
    __shared__ int32_t multi_item[256], multi_at[256];   // segments with several occurrences, and their first's index
    __shared__ int32_t ahead[32][64];                    // token j after occurrence i (few occurrences)
    const int b = blockIdx.x, tid = threadIdx.x;
    auto none = [&]() {
        if (tid == 0) { draft_start[b] = -1; match_len[b] = 0; draft_len[b] = 0; draft_src[b] = -1; }
    };
    // Everything that a thread needs of its first segment is asked for at once, with the sequence's state: one trip to memory
    // instead of a chain of them.  (That, and exchanges between lanes that stay out of the LDS unit: 13.6 -> 10.5 us.)
    const int n_items = n_resp * max_segs;
    const int g0 = tid / max_segs, seg0 = tid - g0 * max_segs;
    const bool mine = tid < n_items;
    const int r_at = b * n_resp + (mine ? g0 : 0);
    const int off0 = hist_off[r_at], end0 = hist_off[r_at + 1], rew0 = reward[r_at];
    const unsigned long long raw0 = best[(size_t)b * n_items + (mine ? tid : 0)];
    const int left = budget_left[b], state = k_state[b];
    const int n_pat = min(min(tail_len[b], pol.window), w_max);
    if (left <= 0 || n_pat < pol.m_min || n_pat <= 0) { none(); return; }
    if (tid < n_pat) pat[tid] = tail[(size_t)b * w_max + (w_max - 1 - tid)];
    if (tid == 0) n_occ_s = 0;
    // longest match over all segments of all responses
    const unsigned long long key0 = mine && seg0 * HS_DRAFT_SEG + 1 <= end0 - off0 - 1 ? raw0 : 0ull;
    auto item_key = [&](int i) -> unsigned long long {
        if (i < 256) return key0;      // (the thread's first)
        if (i >= n_items) return 0ull;
        const int g = i / max_segs, sgm = i - g * max_segs;
        const int lh = hist_off[b * n_resp + g + 1] - hist_off[b * n_resp + g];
        return sgm * HS_DRAFT_SEG + 1 <= lh - 1 ? best[(size_t)b * n_items + i] : 0ull;
    };
    unsigned long long k = 0ull;
    for (int i = tid; i < n_items; i += 256) {
        const unsigned long long v = (unsigned long long)draft_key_len(item_key(i));
        if (v > k) k = v;
    }
    const int m_star = (int)block_max_u64(k, red);   // (contains the barriers that publish pat and n_occ_s)
    if (m_star < pol.m_min || m_star <= 0) { none(); return; }
    // Occurrences, in (response, position) order: only segments whose best match reaches m_star hold any.  The scan has
    // counted them and named the first, so a segment with one occurrence (the usual case) is not read again.
    for (int i0 = 0; i0 < n_items; i0 += 256) {
        const unsigned long long key = item_key(i0 + tid);
        const int n = key && draft_key_len(key) == m_star ? draft_key_count(key) : 0;
        if (tid == 0) n_multi_s = 0;
        int total;
        const int at = n_occ_s + block_excl_scan<256>(n, &total, sw);
        if (n > 0 && at < HS_OCC_MAX) {
            const int g = (i0 + tid) / max_segs;
            if (n == 1) {
                const bool first = i0 == 0;
                occ_off[at] = (first ? off0 : hist_off[b * n_resp + g]) + (int)(0xFFFFFFFFu - (unsigned)key);
                occ_end[at] = first ? end0 : hist_off[b * n_resp + g + 1];
                occ_rew[at] = first ? rew0 : reward[b * n_resp + g];
                occ_resp[at] = g;
            } else {
                const int q = atomicAdd(&n_multi_s, 1);
                multi_item[q] = i0 + tid;
                multi_at[q] = at;
            }
        }
        __syncthreads();
        for (int q = 0; q < n_multi_s; q++) {
            const int g = multi_item[q] / max_segs, sgm = multi_item[q] - g * max_segs;
            const int off = hist_off[b * n_resp + g], lh = hist_off[b * n_resp + g + 1] - off;
            const int p_hi = min((sgm + 1) * HS_DRAFT_SEG, lh - 1);
            const int p0 = sgm * HS_DRAFT_SEG + 1 + tid * (HS_DRAFT_SEG / 256);   // 16 places in a row per thread
            unsigned hits = 0u;
            for (int e = 0; e < HS_DRAFT_SEG / 256; e++) {
                const int p = p0 + e;
                if (p > p_hi || p < m_star) continue;
                int m = 0;
                while (m < m_star && hist[off + p - 1 - m] == pat[m]) m++;
                if (m == m_star) hits |= 1u << e;
            }
            int sum;
            int dst = multi_at[q] + block_excl_scan<256>(__popc(hits), &sum, sw);
            for (; hits && dst < HS_OCC_MAX; hits &= hits - 1, dst++) {
                occ_off[dst] = off + p0 + __ffs(hits) - 1;
                occ_end[dst] = off + lh;
                occ_rew[dst] = reward[b * n_resp + g];
                occ_resp[dst] = g;
            }
        }
        __syncthreads();
        if (tid == 0) n_occ_s = min(HS_OCC_MAX, n_occ_s + total);
        __syncthreads();
        if (n_occ_s >= HS_OCC_MAX) break;
    }
    const int n_occ = n_occ_s;
    // draft length the policy asks for
    int kk = pol.k_mode == HS_K_FIXED ? pol.k_fixed : (pol.k_mode == HS_K_MATCHLEN ? m_star : state);
    kk = max(0, min(min(kk, pol.k_max), left - 1));
    // Few occurrences (the usual case): their next tokens are fetched at once and one wavefront walks alone, an occurrence
    // per lane -- no memory and no barrier between two draft tokens.  128 prompts with 16 responses: the whole kernel
    // 88 -> 13 us.
    if (n_occ <= 64) {
        for (int i = tid; i < n_occ * kk; i += 256) {
            const int q = i / kk, j = i - q * kk;
            ahead[j][q] = occ_off[q] + j < occ_end[q] ? hist[occ_off[q] + j] : -2;
        }
        __syncthreads();
        if (tid < 64) {
            bool live = tid < n_occ;
            const unsigned long long rew = live ? (unsigned long long)occ_rew[tid] : 0ull;
            int n = 0;
            for (; n < kk; n++) {
                const int t = live ? ahead[n][tid] : -1;
                live = t != -1;   // (as below, an id of -1 drops its occurrence; other negative ids have no vote)
                // every live occurrence prices its own token: (reward sum, votes) packed, larger is better
                unsigned long long sum = 0ull;
                unsigned votes = 0u;
                for (unsigned long long todo = __ballot(t >= 0); todo; todo &= todo - 1) {
                    const int q = __ffsll(todo) - 1;
                    if (__builtin_amdgcn_readlane(t, q) == t) {
                        sum += ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(rew >> 32), q) << 32) |
                               (unsigned)__builtin_amdgcn_readlane((int)rew, q);
                        votes++;
                    }
                }
                const unsigned long long price = t >= 0 ? ((sum << 11) | votes) + 1ull : 0ull;
                const unsigned long long top = lanes_max_u64(price);
                if (top == 0ull) break;   // nobody has a token left: the live occurrences stay live
                // among the tokens with the top price, the smallest id
                const int chosen = lanes_min(price == top ? t : 0x7FFFFFFF);
                live = live && t == chosen;
            }
            const unsigned long long alive = __ballot(live);
            if (tid == 0) { first_s = n == 0 ? 0 : __ffsll(alive) - 1; len_s = n; }   // (nothing drafted: all are live)
        }
        __syncthreads();
    } else {
        // the walk, all occurrences by the whole workgroup
        for (int i = tid; i < n_occ; i += 256) occ_tok[i] = 0;   // live
        __syncthreads();
        int len = 0;
        for (int j = 0; j < kk; j++) {
            for (int i = tid; i < n_occ; i += 256)
                if (occ_tok[i] != -1) occ_tok[i] = (occ_off[i] + j < occ_end[i]) ? hist[occ_off[i] + j] : -2;
            __syncthreads();
            // every live occurrence prices its own token: (reward sum, votes) packed, larger is better
            unsigned long long key = 0ull;
            for (int i = tid; i < n_occ; i += 256) {
                const int t = occ_tok[i];
                if (t < 0) continue;
                unsigned long long sum = 0ull;
                unsigned votes = 0u;
                for (int q = 0; q < n_occ; q++)
                    if (occ_tok[q] == t) { sum += (unsigned long long)occ_rew[q]; votes++; }
                const unsigned long long v = ((sum << 11) | votes) + 1ull;   // + 1: a live vote always beats "none"
                if (v > key) key = v;
            }
            const unsigned long long top = block_max_u64(key, red);
            if (top == 0ull) break;   // nobody has a token left: the live occurrences stay live (marked -2)
            // among the tokens with the top price, the smallest id
            unsigned long long cand = 0ull;
            for (int i = tid; i < n_occ; i += 256) {
                const int t = occ_tok[i];
                if (t < 0) continue;
                unsigned long long sum = 0ull;
                unsigned votes = 0u;
                for (int q = 0; q < n_occ; q++)
                    if (occ_tok[q] == t) { sum += (unsigned long long)occ_rew[q]; votes++; }
                if (((sum << 11) | votes) + 1ull == top) {
                    const unsigned long long v = 0xFFFFFFFFull - (unsigned)t;
                    if (v > cand) cand = v;
                }
            }
            const int chosen = (int)(0xFFFFFFFFull - block_max_u64(cand, red));
            for (int i = tid; i < n_occ; i += 256)
                if (occ_tok[i] != chosen) occ_tok[i] = -1;
            len++;
            __syncthreads();
        }
    // first surviving occurrence (every occurrence is live if nothing was drafted; one that only ran out of text
        // at the step that ended the walk is still live)
        unsigned long long firstk = 0ull;
        for (int i = tid; i < n_occ; i += 256)
            if (len == 0 || occ_tok[i] != -1) { firstk = 0xFFFFFFFFull - (unsigned)i; break; }
        const unsigned long long fk = block_max_u64(firstk, red);
        if (tid == 0) { first_s = fk ? (int)(0xFFFFFFFFull - fk) : -1; len_s = len; }
        __syncthreads();
    }
    const int first = first_s;
    if (first < 0 || n_occ <= 0) { none(); return; }   // (every occurrence ran into an id of -1)
    if (tid == 0) {
        const int g = occ_resp[first];
        draft_src[b] = g;
        draft_start[b] = occ_off[first] - hist_off[b * n_resp + g];
        match_len[b] = m_star;
        draft_len[b] = len_s;
    }
}

}  // namespace

namespace {

void launch_draft(const hs_ctx* ctx, const hs_draft_args* args, const hs_seq_state* seq, hs_step* step,
                  unsigned long long* best, uint32_t* err, hipStream_t st) {
    const hs_policy& p = args->policy;
    dim3 grid(hs_scan_groups(ctx, seq->batch * args->n_cand), seq->batch * args->n_cand);
    hipLaunchKernelGGL(draft_scan_kernel<false>, grid, dim3(256), 0, st, args->hist, args->hist_off, args->n_cand,
                       seq->tail, seq->tail_len, seq->budget_left, ctx->lim.w_max, p.window, p.m_min,
                       ctx->max_segs, best);
    hipLaunchKernelGGL(draft_build_kernel, dim3(1), dim3(BUILD_THREADS), 0, st, args->hist, args->hist_off, args->n_cand,
                       seq->batch, best, ctx->max_segs, seq->seq_len, seq->tail, ctx->lim.w_max, seq->k_state,
                       seq->budget_left, p, ctx->lim.max_blocks_per_seq, ctx->lim.max_pos, ctx->lim.max_rows,
                       step->draft_start, step->match_len, step->draft_len, step->row_off, step->tok, step->pos,
                       step->parent, step->anc_mask, step->row2seq, err, 0, nullptr, seq->gate,
                       (const unsigned long long*)seq->counters);
}

}  // namespace

void hs_launch_draft(const hs_ctx* ctx, const hs_draft_args* args, const hs_seq_state* seq, hs_step* step,
                     hipStream_t st) {
    launch_draft(ctx, args, seq, step, reinterpret_cast<unsigned long long*>(ctx->ws + ctx->lay.draft_best),
                 reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.err), st);
}

// ---- hs_draft for callers that cannot allocate: the segment winners (and, with no workspace bound, the error word)
// live in a static device array instead of the caller's workspace.
namespace {

// [0, HS_DRAFT_STATIC_ENTRIES): segment winners, 8 bytes each; then one 8-byte slot whose first word is the error word.
static __device__ __align__(256) unsigned long long scratch[HS_DRAFT_STATIC_ENTRIES + 1];

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
unsigned long long* scratch_ptr[MAX_DEVICES];   // device address of `scratch` on each device (each has its own copy)

// The address of this device's copy of the array, looked up once per device with that device current.
unsigned long long* scratch_on_current_device(hipError_t* why) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= MAX_DEVICES) { *why = e != hipSuccess ? e : hipErrorInvalidDevice; return nullptr; }
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) { *why = e != hipSuccess ? e : hipErrorInvalidSymbol; return nullptr; }
        scratch_ptr[dev] = static_cast<unsigned long long*>(p);
    }
    return scratch_ptr[dev];
}

}  // namespace

uint32_t* hs_draft_static_error_word(hipError_t* why) {
    unsigned long long* base = scratch_on_current_device(why);
    return base ? reinterpret_cast<uint32_t*>(base + HS_DRAFT_STATIC_ENTRIES) : nullptr;
}

bool hs_launch_draft_static(const hs_ctx* ctx, const hs_draft_args* args, const hs_seq_state* seq, hs_step* step,
                            hipStream_t st, hipError_t* why) {
    unsigned long long* base = scratch_on_current_device(why);
    if (!base) return false;
    uint32_t* err = ctx->ws ? reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.err)
                            : reinterpret_cast<uint32_t*>(base + HS_DRAFT_STATIC_ENTRIES);
    // every winner slot the build kernel reads is written by the scan kernel of the same call: nothing to clear
    launch_draft(ctx, args, seq, step, base, err, st);
    return true;
}

void hs_launch_draft_group(const hs_ctx* ctx, const hs_group_draft_args* args, const hs_seq_state* seq,
                           hs_step* step, hipStream_t st) {
    unsigned long long* best = reinterpret_cast<unsigned long long*>(ctx->ws + ctx->lay.draft_best);
    uint32_t* err = reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.err);
    const hs_policy& p = args->policy;
    dim3 grid(hs_scan_groups(ctx, seq->batch * args->n_resp), seq->batch * args->n_resp);
    hipLaunchKernelGGL(draft_scan_kernel<true>, grid, dim3(256), 0, st, args->hist, args->hist_off, args->n_resp,
                       seq->tail, seq->tail_len, seq->budget_left, ctx->lim.w_max, p.window, p.m_min,
                       ctx->max_segs, best);
    hipLaunchKernelGGL(draft_group_walk_kernel, dim3(seq->batch), dim3(256), 0, st, args->hist, args->hist_off,
                       args->reward, args->n_resp, best, ctx->max_segs, seq->tail, seq->tail_len, ctx->lim.w_max,
                       seq->k_state, seq->budget_left, p, step->draft_start, step->match_len, step->draft_len,
                       step->draft_src);
    hipLaunchKernelGGL(draft_build_kernel, dim3(1), dim3(BUILD_THREADS), 0, st, args->hist, args->hist_off, 1, seq->batch,
                       best, ctx->max_segs, seq->seq_len, seq->tail, ctx->lim.w_max, seq->k_state, seq->budget_left,
                       p, ctx->lim.max_blocks_per_seq, ctx->lim.max_pos, ctx->lim.max_rows, step->draft_start,
                       step->match_len, step->draft_len, step->row_off, step->tok, step->pos, step->parent,
                       step->anc_mask, step->row2seq, err, args->n_resp, step->draft_src, seq->gate,
                       (const unsigned long long*)seq->counters);
}
