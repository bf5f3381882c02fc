// Acceptance and KV commit (Sec. 2.2 of the paper: the verified draft tokens that are valid are kept, and the
// output distribution is preserved; Sec. 5.4: the per-response speculation window update).
//
// Greedy acceptance walks the draft tree from the root, following the child whose token equals the parent row's
// argmax.  Rejection acceptance is speculative sampling with a point-mass draft distribution: child j of a node
// is accepted with probability p(tok_j) under softmax(logits / T) with the tokens of earlier rejected siblings
// removed; the walk ends with one inverse-CDF sample in token-id order.  Uniforms come from Philox-4x32-10
// (Salmon et al., SC'11) keyed by the seed, with counter (position, draw kind, sequence id): the stream does not
// depend on the batch slot or on how many steps it took to reach the position.
#include <algorithm>

#include "hs_internal.h"
#include "hs_lanes.h"

namespace {

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                     uint32_t out[4]) {
#pragma unroll
    for (int r = 0; r < 10; r++) {
        uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

__device__ __forceinline__ double uniform01(uint64_t seed, uint64_t seq_id, uint32_t position, uint32_t kind) {
    uint32_t o[4];
    philox4x32_10(position, kind, (uint32_t)seq_id, (uint32_t)(seq_id >> 32), (uint32_t)seed, (uint32_t)(seed >> 32), o);
    return (double)(o[0] >> 8) * (1.0 / 16777216.0);
}

// Greedy walk of one sequence's tree (one thread): follow the child whose token is the current node's argmax.
__device__ __forceinline__ void accept_greedy_walk(int b, int r0, int nn, const int32_t* __restrict__ tok,
                                          const int32_t* __restrict__ parent, const int32_t* __restrict__ argmax,
                                          int k_stride, int32_t* __restrict__ accept_len, int32_t* __restrict__ n_out,
                                          int32_t* __restrict__ out_tok, int32_t* __restrict__ path_row) {
    int cur = 0, a = 0;
    path_row[(size_t)b * k_stride] = 0;
    for (;;) {
        int g = argmax[r0 + cur];
        out_tok[(size_t)b * k_stride + a] = g;
        int next = -1;
        for (int i = 1; i < nn; i++)
            if (parent[r0 + i] == cur && tok[r0 + i] == g) { next = i; break; }
        if (next < 0 || a + 1 >= k_stride) break;
        cur = next;
        a++;
        path_row[(size_t)b * k_stride + a] = cur;
    }
    accept_len[b] = a;
    n_out[b] = a + 1;
}

template <int O>
__device__ __forceinline__ double lane_xor_f64(double v) {
    return __hiloint2double((int)lane_xor<O>((unsigned)__double2hiint(v)), (int)lane_xor<O>((unsigned)__double2loint(v)));
}
// Butterflies over 64 lanes (WIDTH = 32: over either half): every lane gets the result, added up in the same tree.
template <int WIDTH = 64>
__device__ __forceinline__ double wave_sum_f64(double v) {
    if constexpr (WIDTH == 64) v += lane_xor_f64<32>(v);
    v += lane_xor_f64<16>(v);
    v += lane_xor_f64<8>(v);
    v += lane_xor_f64<4>(v);
    v += lane_xor_f64<2>(v);
    return v + lane_xor_f64<1>(v);
}
template <int WIDTH = 64>
__device__ __forceinline__ float wave_max_f32(float v) {
    auto step = [&](unsigned other) { v = fmaxf(v, __uint_as_float(other)); };
    if constexpr (WIDTH == 64) step(lane_xor<32>(__float_as_uint(v)));
    step(lane_xor<16>(__float_as_uint(v)));
    step(lane_xor<8>(__float_as_uint(v)));
    step(lane_xor<4>(__float_as_uint(v)));
    step(lane_xor<2>(__float_as_uint(v)));
    step(lane_xor<1>(__float_as_uint(v)));
    return v;
}

// Workgroup barrier for values in LDS alone: unlike __syncthreads it leaves loads from memory on their way.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
    v = wave_sum_f64(v);
    lds_barrier();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    lds_barrier();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ float block_max_f32(float v, float* red) {
    v = wave_max_f32(v);
    lds_barrier();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    lds_barrier();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// ---- rejection sampling.  Probabilities are evaluated in fp64 from the fp32 logits.
//
// A decision at a node needs the node's largest logit and the sum of exp((logit - largest) / T) over the vocabulary:
// some 20 operations, most of them fp64, for each of up to 152064 tokens, which is what bounds this path.  The walk from
// node to node is a chain, but the sums of different nodes are independent: they are computed by launches of their own, cut
// into slices of SLICE tokens (a workgroup keeps a slice in registers, so every logit is read once), and the walk that
// follows only combines the slices of the rows it visits.  64 trees of 17 rows over 152064 tokens: 0.15 ms for the sums
// of all rows (4.3 TB/s of logits) and 0.025 ms for the walk; with everything in one workgroup per sequence, two passes over
// the vocabulary per visited node and one lane that walked 594 tokens at the end, it was 2.6 to 3.4 ms.  Slices of 8192
// tokens took 5 % longer (twice the registers, half the wavefronts).
// Most rows of a large batch are never visited: a walk leaves its tree where a draft is rejected.  So the sums of many rows
// come in stages: the roots; then, time and again, a small kernel takes every walk as far as the sums go and says what the
// next launch sums for it: the node reached and the ones below it, 2, 4, 8 ... levels at a time, as fewer and fewer walks
// are still under way.
// Another rejection-sampling call of the context may run at the same time on another stream, with rows of its own and the
// same place in the workspace.  So every sum and plan carries a word made of itself and the number of the call that wrote
// it.  Where a workgroup of a stage finds anything but its own call's plan, it sums all nodes of its sequence, whatever the
// others of its slice have found (a call replayed from a graph has the number of its earlier replays: nothing that is visited
// may be left over from those); where the last walk finds another call's sum, it computes the node's sums itself, into LDS.
constexpr int SLICE = HS_REJECT_SLICE, PER = SLICE / 256;   // tokens of a slice; of a slice, per thread

// exp((l - ref) / T) in fp64 for l <= ref, with c = 32 / (T ln 2): (l - ref) c = n + f, |f| <= 1/2, and the result is
// 2^(n >> 5) tab[n & 31] exp(f ln2/32), tab[j] = 2^(j/32) -- the table method of P. T. P. Tang (ACM TOMS 15, 1989) -- the
// last factor by its Taylor series to the sixth power (remainder 3.4e-18).  14 fp64 operations against about 30 of the
// library's exp, and the sums are bound by them.  Error: c is a rounded product of a rounded constant, 2^-52 |x| of the
// result x = (l - ref) / T, plus 2 ulp for the factors.  The table's entries cover the 64 LDS banks once: no lookup
// conflicts with another.  Differences below `low` are taken as that; a NaN comes out as such a value, too, so callers look
// for NaNs themselves.  (The clamp is on the fp64 difference: at a low temperature it is less than an fp32 logit resolves.)
struct exp_scale { double low, c; };
__device__ __forceinline__ exp_scale make_scale(double inv_temp, double least) { return {-least / inv_temp, inv_temp * 46.16624130844683}; }
struct exp_parts { int n; double p; };     // 2^(n/32) p
__device__ __forceinline__ exp_parts exp_split(float l, float ref, const exp_scale& k) {
    const double d = fmax((double)l - (double)ref, k.low);
    const double t = __builtin_fma(d, k.c, 6755399441055744.0);      // + 1.5 2^52: n in the low bits
    const double f = __builtin_fma(d, k.c, -(t - 6755399441055744.0));
    double p = 1.4345655584131934e-13;
    p = __builtin_fma(p, f, 3.973709984549416e-11);
    p = __builtin_fma(p, f, 9.172562701824643e-09);
    p = __builtin_fma(p, f, 1.693850972437182e-06);
    p = __builtin_fma(p, f, 0.0002345961982022468);
    p = __builtin_fma(p, f, 0.02166084939249829);
    return {__double2loint(t), __builtin_fma(p, f, 1.0)};
}
// With a clamp at -746 T, -inf among what it takes, the result there is 0.
__device__ __forceinline__ exp_scale exact_scale(double inv_temp) { return make_scale(inv_temp, 746.0); }
__device__ __forceinline__ double exp_diff(float l, float ref, const exp_scale& k, const double* tab) {
    const exp_parts e = exp_split(l, ref, k);
    return __builtin_amdgcn_ldexp(e.p * tab[e.n & 31], e.n >> 5);
}
__device__ __forceinline__ void fill_exp_table(double* tab) {
    if (threadIdx.x < 32) tab[threadIdx.x] = exp2((double)threadIdx.x * 0.03125);
    __syncthreads();
}

// A thread's share of a slice, -inf beyond the vocabulary: 16-byte pieces 4 KB apart where rows are 16-byte aligned.
__device__ __forceinline__ int slice_token(int slice, int j, bool vec) {
    return slice * SLICE + (vec ? 4 * ((int)threadIdx.x + 256 * (j >> 2)) + (j & 3) : (int)threadIdx.x + 256 * j);
}
__device__ __forceinline__ void load_slice(const float* __restrict__ lg, int vocab, int slice, bool vec, float (&v)[PER]) {
    if (vec) {
#pragma unroll
        for (int j = 0; j < PER / 4; j++) {
            const int i = slice_token(slice, 4 * j, true);
            float4 f = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (i < vocab) f = *reinterpret_cast<const float4*>(lg + i);
            v[4 * j] = f.x; v[4 * j + 1] = f.y; v[4 * j + 2] = f.z; v[4 * j + 3] = f.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < PER; j++) {
            const int i = slice_token(slice, j, false);
            v[j] = i < vocab ? lg[i] : -INFINITY;
        }
    }
}

// Sum of exp((logit - ref) / T) over a thread's logits; a NaN makes it NaN.
__device__ __forceinline__ double check_sum(const float (&v)[PER], float ref, double s) {
    bool nan = ref == INFINITY;
#pragma unroll
    for (int j = 0; j < PER; j++) nan |= __builtin_isnan(v[j]);
    return nan ? NAN : ref != -INFINITY ? s : 0.0;
}
// Excluded ones (-inf) add nothing.
__device__ __forceinline__ double sum_weights(const float (&v)[PER], float ref, double inv_temp, const double* tab) {
    const exp_scale k = exact_scale(inv_temp);
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < PER; j++) s += exp_diff(v[j], ref, k, tab);
    return check_sum(v, ref, s);
}
// The same where ref is the largest logit of a slice, so that the slice's sum is at least 1 and weights of e^-700 don't
// show in it: excluded ones add that much, and a weight's power of two is an addition to its exponent.
__device__ __forceinline__ double sum_slice(const float (&v)[PER], float largest, double inv_temp, const double* tab) {
    const exp_scale k = make_scale(inv_temp, 700.0);
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < PER; j++) {
        const exp_parts e = exp_split(v[j], largest, k);
        const double t = tab[e.n & 31];
        s = __builtin_fma(__hiloint2double(__double2hiint(t) + ((e.n & ~31) << 15), __double2loint(t)), e.p, s);
    }
    return check_sum(v, largest, s);
}

// The sums come in stages from so many megabytes of logits on, by the hint (trees of 17 rows over 152064 tokens, all rows at
// once against stages: 16 sequences, 165 MB, 64.5 against 67.7 us; 24, 79 against 67; 32, 105 against 71; 64, 177 against 104;
// where more drafts are accepted 176 against 134).  Without a hint there is only the most that the limits allow, and there may
// be far fewer rows: 64 sequences of one row take 27 us at once and 40 in stages, four launches of which find nothing to do.
// So the limits only speak from the second figure on, where stages cost little against all the rows that there might be (64
// chains of 9 rows: 104 against 108).
#ifndef HS_REJECT_STAGED_MB
#define HS_REJECT_STAGED_MB 200
#define HS_REJECT_STAGED_UNKNOWN_MB 1200
#endif

// Largest logit and sum of one slice, relative to that largest logit, by a workgroup of 256 threads.
// A slice in which every token is excluded (-inf) has the sum 0; a NaN anywhere makes the sum NaN.
struct slice_stat { float m; double s; };
__device__ __forceinline__ slice_stat slice_stats(const float (&v)[PER], double inv_temp, const double* tab) {
    __shared__ float redf[4];
    __shared__ double redd[4];
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER; j++) mx = fmaxf(mx, v[j]);
    mx = block_max_f32(mx, redf);
    const double s = block_sum_f64(sum_slice(v, mx, inv_temp, tab), redd);
    // (the same in every lane: in scalar registers from here on)
    return {__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(mx))),
            __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(s)), __builtin_amdgcn_readfirstlane(__double2loint(s)))};
}

// A slice's entry in the workspace, one 16-byte access.  The check word ties the value to the call: an entry of another
// call, or put together from two, passes for one of this call's in one of 2^32 cases.
__device__ __forceinline__ uint32_t stat_check(const slice_stat& v, uint32_t call) {
    uint32_t h = __float_as_uint(v.m) * 0x9E3779B1u;
    h = (h ^ (h >> 15)) + (uint32_t)__double2loint(v.s);
    h *= 0x85EBCA6Bu;
    h = (h ^ (h >> 13)) + (uint32_t)__double2hiint(v.s);
    h *= 0xC2B2AE35u;
    return h ^ (h >> 16) ^ call;
}
__device__ __forceinline__ void put_stat(hs_reject_stat* dst, const slice_stat& v, uint32_t call) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(__float_as_uint(v.m), stat_check(v, call), (uint32_t)__double2loint(v.s),
                                                (uint32_t)__double2hiint(v.s));
}
__device__ __forceinline__ bool take_stat(const uint4& u, uint32_t call, slice_stat& v) {
    v = {__uint_as_float(u.x), __hiloint2double((int)u.w, (int)u.z)};
    return u.y == stat_check(v, call);
}
__device__ __forceinline__ bool get_stat(const hs_reject_stat* src, uint32_t call, slice_stat& v) {
    return take_stat(*reinterpret_cast<const uint4*>(src), call, v);
}

// A row's largest logit and sum, put together by half a wavefront from its slices: slice(s, v) gets one, false if it
// cannot be used.
template <typename Slice>
__device__ __forceinline__ bool row_total(Slice slice, int n_slices, double inv_temp, int lane, float& mx, double& z) {
    bool ok = true;
    slice_stat v;
    mx = -INFINITY;
    for (int s = lane & 31; s < n_slices; s += 32) { ok &= slice(s, v); mx = fmaxf(mx, v.m); }
    mx = wave_max_f32<32>(mx);
    z = 0.0;
    for (int s = lane & 31; s < n_slices; s += 32) { ok &= slice(s, v); z += v.s * exp(((double)v.m - (double)mx) * inv_temp); }
    z = wave_sum_f64<32>(z);
    return (__ballot(ok) >> (lane & 32) & 0xFFFFFFFFull) == 0xFFFFFFFFull;
}

// What a walk may ask of a sequence's nodes, a node per lane: parent, token, position and the token's logit at the parent.
struct node_lanes { int par, tok, pos; float lg; };
__device__ __forceinline__ node_lanes load_nodes(int r0, int nn, int vocab, const int32_t* __restrict__ tok,
                                                 const int32_t* __restrict__ parent, const int32_t* __restrict__ pos,
                                                 const float* __restrict__ logits, int lane) {
    node_lanes n = {-2, 0, pos[r0], -INFINITY};
    if (lane < nn) {
        n.par = parent[r0 + lane];
        n.tok = tok[r0 + lane];
        n.pos = pos[r0 + lane];
        // (a drafted id outside the vocabulary has no logit: it is a token of weight 0, rejected like any other)
        if (lane > 0 && n.par >= 0 && n.par < nn && n.tok >= 0 && n.tok < vocab)
            n.lg = logits[(size_t)(r0 + n.par) * vocab + n.tok];
    }
    return n;
}

// The decision at node cur, whose largest logit is mx and whose sum z, by a wavefront: its children are tried in node order.
// Returns the accepted one or -1; lane q < nrej holds the q-th rejected token.
__device__ __forceinline__ int try_children(const node_lanes& n, int cur, int nn, float mx, double z, double inv_temp,
                                            uint64_t seed, uint64_t sid, int lane, int& nrej, int& rej) {
    const bool child = lane > 0 && lane < nn && n.par == cur;
    const double my_w = child ? exp(((double)n.lg - (double)mx) * inv_temp) : 0.0;
    const uint32_t position = (uint32_t)(__shfl(n.pos, cur) + 1);
    int next = -1, tried = 0;
    double zr = z;
    for (unsigned long long todo = __ballot(child); todo && next < 0; todo &= todo - 1) {
        const int q = __ffsll(todo) - 1;
        const int t = __shfl(n.tok, q);
        double w = __hiloint2double(__shfl(__double2hiint(my_w), q), __shfl(__double2loint(my_w), q));
        if (__any(lane < nrej && rej == t)) w = 0.0;
        const double u = uniform01(seed, sid, position, (uint32_t)tried);
        if (u < w / zr) {
            next = q;
        } else if (nrej < 8) {
            if (lane == nrej) rej = t;
            nrej++;
            zr -= w;
        }
        tried++;
    }
    return next;
}

// Where a sequence's walk stands between two stages (node cur, a drafts accepted), and the nodes that the next one sums: none
// once the walk has ended.
struct walk_plan { unsigned long long todo; int cur, a; };
__device__ __forceinline__ uint4 pack_plan(const walk_plan& w, uint32_t call) {
    uint4 u = make_uint4((uint32_t)w.todo, (uint32_t)(w.todo >> 32), (uint32_t)(w.cur | w.a << 8), 0u);
    uint32_t h = u.x * 0x9E3779B1u;
    h = (h ^ (h >> 15)) + u.y;
    h *= 0x85EBCA6Bu;
    h = (h ^ (h >> 13)) + u.z;
    h *= 0xC2B2AE35u;
    u.w = h ^ (h >> 16) ^ call;
    return u;
}
// (read by one thread for the workgroup: another call may be writing here, and barriers depend on what it says)
__device__ __forceinline__ bool get_plan(const uint4* src, uint32_t call, walk_plan& w) {
    __shared__ uint4 s_plan;
    if (threadIdx.x == 0) s_plan = *src;
    __syncthreads();
    const uint4 u = s_plan;
    w = {(unsigned long long)u.y << 32 | u.x, (int)(u.z & 255u), (int)(u.z >> 8 & 255u)};
    return u.w == pack_plan(w, call).w && u.z <= 0xFFFFu;
}

// Node cur and what lies at most levels - 1 below it, a bit per node.
__device__ __forceinline__ unsigned long long nodes_below(const node_lanes& n, int cur, int nn, int levels, int lane) {
    unsigned long long in = 1ull << cur;
    for (int l = 1; l < levels; l++) {
        const unsigned long long more = in | __ballot(lane > 0 && lane < nn && n.par >= 0 && n.par < nn && (in >> (n.par & 63) & 1ull));
        if (more == in) break;
        in = more;
    }
    return in;
}

struct reject_stage_args {
    const int32_t *row_off, *tok, *parent, *pos;
    const float* logits;
    int batch, vocab, n_slices, k_stride;
    const uint64_t* seq_id;
    double inv_temp;
    uint64_t seed;
    uint32_t call;
    hs_reject_stat* stats;
    uint4* plan;          // per sequence
    int all_rows;         // up to so many rows the first stage sums all of them
};

__device__ __forceinline__ unsigned long long node_bits(int nn) { return nn < 64 ? (1ull << nn) - 1 : ~0ull; }

// grid (sequences, slices, node split): a workgroup sums a slice of the nodes number blockIdx.z, blockIdx.z + gridDim.z,
// ... of those that its stage computes, the next one's logits on their way while it sums the current one's.
__global__ __launch_bounds__(256, 5) void reject_stats_kernel(reject_stage_args p, int first) {
    __shared__ double tab[32];
    // (workgroups are dealt round-robin to the eight XCDs: a sequence's slices go to all of them, or those of the walks that
    // are still under way would share a few: 64 trees 122 -> 105 us)
    const int n_slices = p.n_slices, slice = blockIdx.y, b = (int)((blockIdx.x + blockIdx.y) % gridDim.x);
    const int r0 = p.row_off[b], nn = min(p.row_off[b + 1] - r0, HS_MAX_NODES);
    if (nn <= 0) return;
    unsigned long long todo = node_bits(nn);
    int skip = (int)blockIdx.z, stride = (int)gridDim.z;
    if (first) {
        if (p.row_off[p.batch] > p.all_rows) todo = 1ull;
    } else {
        walk_plan w;
        if (get_plan(p.plan + b, p.call, w)) todo &= w.todo;
        // (not the call's own plan: the other workgroups of this slice may have read it before it was overwritten and count
        // other nodes, so this one leaves none to them)
        else { skip = 0; stride = 1; }
    }
    for (int q = 0; q < skip; q++) todo &= todo - 1;
    todo = (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(todo >> 32)) << 32 | __builtin_amdgcn_readfirstlane((unsigned)todo);
    if (!todo) return;
    fill_exp_table(tab);
    const bool vec = (p.vocab & 3) == 0 && ((unsigned long long)p.logits & 15ull) == 0;
    int i = __ffsll(todo) - 1;
    float v[PER], w[PER];
    load_slice(p.logits + (size_t)(r0 + i) * p.vocab, p.vocab, slice, vec, v);
    while (todo) {
        for (int q = 0; q < stride; q++) todo &= todo - 1;
        const int next = __ffsll(todo) - 1;
        if (todo) load_slice(p.logits + (size_t)(r0 + next) * p.vocab, p.vocab, slice, vec, w);
        const slice_stat sum = slice_stats(v, p.inv_temp, tab);
        if (threadIdx.x == 0) put_stat(p.stats + (size_t)(r0 + i) * n_slices + slice, sum, p.call);
#pragma unroll
        for (int j = 0; j < PER; j++) v[j] = w[j];
        i = next;
    }
}

// Between two stages: a workgroup per sequence takes its walk through the nodes that have been summed and plans the `levels`
// from where it arrives.
__global__ __launch_bounds__(256) void reject_plan_kernel(reject_stage_args p, int first, int levels) {
    __shared__ float node_max[HS_MAX_NODES];
    __shared__ double node_sum[HS_MAX_NODES];
    __shared__ int node_ok[HS_MAX_NODES];
    const int b = blockIdx.x, n_slices = p.n_slices, lane = threadIdx.x & 63;
    const int r0 = p.row_off[b], nn = min(p.row_off[b + 1] - r0, HS_MAX_NODES);
    if (nn <= 0) return;
    walk_plan w = {1ull, 0, 0};
    bool known = true;
    if (first) { if (p.row_off[p.batch] <= p.all_rows) w.todo = 0ull; }
    else known = get_plan(p.plan + b, p.call, w);
    if (!known) w = {node_bits(nn), 0, 0};
    else if (w.todo == node_bits(nn) && nn > 1) w.todo = 0ull;   // (everything has been summed)
    else if (w.todo) {
        const node_lanes n = load_nodes(r0, nn, p.vocab, p.tok, p.parent, p.pos, p.logits, lane);
        for (int i = threadIdx.x >> 5; i < nn; i += 8) {
            if (!(w.todo >> i & 1ull)) continue;
            const hs_reject_stat* st = p.stats + (size_t)(r0 + i) * n_slices;
            float mx;
            double z;
            const bool ok = row_total([&](int s, slice_stat& v) __attribute__((always_inline)) { return get_stat(st + s, p.call, v); },
                                      n_slices, p.inv_temp, lane, mx, z);
            if ((lane & 31) == 0) { node_max[i] = mx; node_sum[i] = z; node_ok[i] = ok; }
        }
        __syncthreads();
        const uint64_t sid = p.seq_id[b];
        bool ended = false;
        while (!ended && known && (w.todo >> w.cur & 1ull)) {      // (a child's number need not be above its parent's,
            known = node_ok[w.cur];                                //  but a walk of k_stride steps is over)
            int nrej = 0, rej = -1;
            const int next = try_children(n, w.cur, nn, node_max[w.cur], node_sum[w.cur], p.inv_temp, p.seed, sid, lane, nrej, rej);
            if (next >= 0 && w.a + 1 < p.k_stride) { w.cur = next; w.a++; }
            else ended = true;
        }
        w.todo = !known ? node_bits(nn) : ended ? 0ull : nodes_below(n, w.cur, nn, levels, lane);
    }
    if (threadIdx.x == 0) p.plan[b] = pack_plan(w, p.call);
}

// Sum over the lanes up to and including this one, in lane order by a fixed tree.
__device__ __forceinline__ double wave_prefix_f64(double v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double t = __hiloint2double(__shfl_up(__double2hiint(v), o), __shfl_up(__double2loint(v), o));
        if (lane >= o) v += t;
    }
    return v;
}

// Rejection sampling of one sequence by its workgroup (nn > 0).  The four wavefronts take every decision redundantly:
// same values, same order, no exchange.
__device__ __forceinline__ void accept_rejection_seq(
    int b, int r0, int nn, int vocab, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ parent, const int32_t* __restrict__ pos, const float* __restrict__ logits,
    const hs_reject_stat* __restrict__ stats, int n_slices, uint32_t call,
    const uint64_t* __restrict__ seq_id, double inv_temp, uint64_t seed, int k_stride,
    int32_t* __restrict__ accept_len, int32_t* __restrict__ n_out, int32_t* __restrict__ out_tok,
    int32_t* __restrict__ path_row) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
    slice_stat* own = reinterpret_cast<slice_stat*>(dyn_lds);   // [n_slices]: the sums of the node at hand
    __shared__ double wave_tot[4];
    __shared__ int s_first, s_last, s_pick;
    __shared__ double tab[32];
    __shared__ float node_max[HS_MAX_NODES];
    __shared__ double node_sum[HS_MAX_NODES];
    __shared__ int node_ok[HS_MAX_NODES];
    fill_exp_table(tab);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t sid = seq_id[b];
    const bool vec = (vocab & 3) == 0 && ((unsigned long long)logits & 15ull) == 0;
    nn = min(nn, HS_MAX_NODES);   // (a draft tree has no more: hs_create)
    auto in_vocab = [&](int t) { return t >= 0 && t < vocab; };
    // Everything that the walk may ask of the nodes, fetched side by side instead of node after node.
    for (int i = tid >> 5; i < nn; i += 8) {
        const hs_reject_stat* st = stats + (size_t)(r0 + i) * n_slices;
        float mx;
        double z;
        const bool ok = row_total([&](int s, slice_stat& v) __attribute__((always_inline)) { return get_stat(st + s, call, v); },
                                  n_slices, inv_temp, lane, mx, z);
        if ((lane & 31) == 0) { node_max[i] = mx; node_sum[i] = z; node_ok[i] = ok; }
    }
    const node_lanes n = load_nodes(r0, nn, vocab, tok, parent, pos, logits, lane);
    __syncthreads();
    int cur = 0, a = 0;
    if (tid == 0) path_row[(size_t)b * k_stride] = 0;
    // Two turns at a node: decide about its children, then -- at the last node -- sample among what is left.
    bool last = false;
    int nrej = 0, rej = -1;     // lane q < nrej: the q-th rejected token
    float mx = 0.f;
    uint4 my_stat = make_uint4(0u, 0u, 0u, 0u);
    for (;;) {
        const float* lg = logits + (size_t)(r0 + cur) * vocab;
        const uint4* st = reinterpret_cast<const uint4*>(stats + (size_t)(r0 + cur) * n_slices);
        bool all = !node_ok[cur] && !last;          // every slice has to be summed here ...
        if (!last && tid < n_slices) my_stat = st[tid];   // (for the sample, if this is the last node: not waited for here)
        if (last && node_ok[cur]) {
            bool ok = true;
            for (int s = tid; s < n_slices; s += 256) {
                slice_stat v;
                ok &= take_stat(s < 256 ? my_stat : st[s], call, v);
                own[s] = v;
            }
            all = __syncthreads_or(!ok);
        }
        // ... or, before the sample, those that hold rejected tokens, without these (subtracting would leave rounding where a
        // rejected token had nearly all the weight)
        if (all || last) {
            const int rej_slice = lane < nrej && in_vocab(rej) ? rej / SLICE : -1;
            auto next_slice = [&](int s) __attribute__((always_inline)) {   // the first one from s on
                if (all) return s;
                int next = n_slices;
                for (int q = 0; q < nrej; q++) {
                    const int t = __shfl(rej_slice, q);
                    if (t >= s && t < next) next = t;
                }
                return next;
            };
            int s = next_slice(0);
            const bool any = s < n_slices;
            float v[PER], w[PER];
            if (any) load_slice(lg, vocab, s, vec, v);
            while (s < n_slices) {
                const int sn = next_slice(s + 1);
                if (sn < n_slices) load_slice(lg, vocab, sn, vec, w);   // (on its way while this one is summed)
                for (int q = 0; q < nrej; q++) {
                    const int t = __shfl(rej, q);
#pragma unroll
                    for (int j = 0; j < PER; j++)
                        if (slice_token(s, j, vec) == t) v[j] = -INFINITY;
                }
                const slice_stat sum = slice_stats(v, inv_temp, tab);
                if (tid == 0) own[s] = sum;
#pragma unroll
                for (int j = 0; j < PER; j++) v[j] = w[j];
                s = sn;
            }
            if (any) __syncthreads();
        }
        if (!last) {
            double z;
            if (all) row_total([&](int s, slice_stat& v) __attribute__((always_inline)) { v = own[s]; return true; }, n_slices, inv_temp, lane, mx, z);
            else { mx = node_max[cur]; z = node_sum[cur]; }
            const int next = try_children(n, cur, nn, mx, z, inv_temp, seed, sid, lane, nrej, rej);
            if (next >= 0 && a + 1 < k_stride) {
                const int next_tok = __shfl(n.tok, next);
                if (tid == 0) {
                    out_tok[(size_t)b * k_stride + a] = next_tok;
                    path_row[(size_t)b * k_stride + a + 1] = next;
                }
                cur = next;
                a++;
                nrej = 0;
                rej = -1;
            } else {
                last = true;
            }
            if (all) __syncthreads();   // (own[] has been read)
            continue;
        }
        // Final sample from the remaining distribution, in token-id order.
        const uint32_t position = (uint32_t)(__shfl(n.pos, cur) + 1);
        auto slice_weight = [&](int s) __attribute__((always_inline)) { return s < n_slices ? own[s].s * exp(((double)own[s].m - (double)mx) * inv_temp) : 0.0; };
        double zt = 0.0;
        for (int s0 = 0; s0 < n_slices; s0 += 64) {
            zt += wave_sum_f64(slice_weight(s0 + lane));
        }
        const double target = uniform01(seed, sid, position, 7u) * zt;
        int slice = -1;
        double before = 0.0;   // weight in front of the chosen slice
        for (int s0 = 0; s0 < n_slices && slice < 0; s0 += 64) {
            const double w = slice_weight(s0 + lane), incl = wave_prefix_f64(w, lane);
            const unsigned long long hit = __ballot(w > 0.0 && before + incl >= target);
            const int q = hit ? __ffsll(hit) - 1 : 63;
            const double upto = hit ? incl - w : incl;
            before += __hiloint2double(__shfl(__double2hiint(upto), q), __shfl(__double2loint(upto), q));
            if (hit) slice = s0 + q;
        }
        if (tid == 0) { s_first = 256; s_last = -1; s_pick = -1; }
        __syncthreads();
        if (slice >= 0) {
            // PER consecutive tokens per thread: the first thread whose running sum reaches the target holds the token
            const int lo = slice * SLICE + tid * PER;
            float v[PER];
            if (vec) {
#pragma unroll
                for (int j = 0; j < PER; j += 4) {
                    float4 f = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                    if (lo + j < vocab) f = *reinterpret_cast<const float4*>(lg + lo + j);
                    v[j] = f.x; v[j + 1] = f.y; v[j + 2] = f.z; v[j + 3] = f.w;
                }
            } else {
#pragma unroll
                for (int j = 0; j < PER; j++) v[j] = lo + j < vocab ? lg[lo + j] : -INFINITY;
            }
            for (int q = 0; q < nrej; q++) {
                const int t = __shfl(rej, q);
#pragma unroll
                for (int j = 0; j < PER; j++)
                    if (lo + j == t) v[j] = -INFINITY;
            }
            const double sum = sum_weights(v, mx, inv_temp, tab);
            const double incl = wave_prefix_f64(sum, lane);
            if (lane == 63) wave_tot[wave] = incl;
            __syncthreads();
            double base = before + (incl - sum);
            for (int q = 0; q < wave; q++) base += wave_tot[q];
            if (sum > 0.0) {
                atomicMax(&s_last, tid);
                if (base + sum >= target) atomicMin(&s_first, tid);
            }
            __syncthreads();
            // (rounding can leave the target just beyond the slice: its last token with weight then)
            const int owner = s_first < 256 ? s_first : s_last;
            if (owner >= 0 && wave == owner >> 6) {
                const int at = slice * SLICE + owner * PER, i = at + lane;
                bool in = lane < PER && i < vocab;
                for (int q = 0; q < nrej; q++) in = in && __shfl(rej, q) != i;
                const float l = in ? lg[i] : -INFINITY;
                const double w = exp_diff(l, mx, exact_scale(inv_temp), tab);
                const double cum = __hiloint2double(__shfl(__double2hiint(base), owner & 63), __shfl(__double2loint(base), owner & 63)) +
                                   wave_prefix_f64(w, lane);
                const unsigned long long nz = __ballot(w > 0.0), hit = __ballot(w > 0.0 && cum >= target);
                if (lane == 0) s_pick = hit ? at + __ffsll(hit) - 1 : nz ? at + 63 - __clzll(nz) : -1;
            }
            __syncthreads();
        }
        int pick = s_pick;
        if (pick < 0) {  // no slice reaches the target (NaN among the logits): the last token that was not rejected
            for (pick = vocab - 1; pick >= 0; pick--) {
                if (!__any(lane < nrej && rej == pick)) break;
            }
        }
        if (tid == 0) {
            out_tok[(size_t)b * k_stride + a] = pick;
            accept_len[b] = a;
            n_out[b] = a + 1;
        }
        break;
    }
}

// Commit of one sequence by its workgroup: relocate accepted tree nodes' K/V to consecutive slots, then advance the
// state.  CT = cache element type (bf16 bits, or float in the fp32-activation mode).
template <typename CT>
__device__ __forceinline__ void commit_seq(
    int b, int n_layers, int hkv, int hd, int n_blocks, CT* __restrict__ kc, CT* __restrict__ vc,
    const int32_t* __restrict__ block_table, int max_blocks, int32_t* __restrict__ seq_len,
    int32_t* __restrict__ tail, int32_t* __restrict__ tail_len, int w_max, int32_t* __restrict__ k_state,
    int32_t* __restrict__ budget_left, int32_t* __restrict__ tokens, int tokens_stride,
    unsigned long long* __restrict__ counters, const int32_t* __restrict__ row_off,
    const int32_t* __restrict__ parent, const int32_t* __restrict__ accept_len, const int32_t* __restrict__ n_out,
    const int32_t* __restrict__ out_tok, const int32_t* __restrict__ path_row, int k_stride, const hs_policy& pol) {
    const int tid = threadIdx.x;
    const int r0 = row_off[b], nn = row_off[b + 1] - r0;
    const int no = n_out[b];
    if (nn <= 0 || no <= 0) return;
    const int a = accept_len[b];
    const int n_old = seq_len[b];
    const int L = n_old - 1;
    const int32_t* bt = block_table + (size_t)b * max_blocks;
    // accepted node path_row[j] (j = 1..a) must end up in slot L + j
    const size_t per_layer = (size_t)n_blocks * hkv * 16 * hd;
    for (int jn = 1; jn <= a; jn++) {
        int node = path_row[(size_t)b * k_stride + jn];
        if (node == jn) continue;
        int s_slot = L + node, d_slot = L + jn;
        int sp = bt[s_slot >> 4], dp = bt[d_slot >> 4];
        if (sp < 0 || sp >= n_blocks || dp < 0 || dp >= n_blocks) continue;
        int si = s_slot & 15, di = d_slot & 15;
        int per = hkv * hd;
        for (int e = tid; e < n_layers * per; e += 256) {
            int layer = e / per, r = e % per, head = r / hd, d = r % hd;
            size_t lo = (size_t)layer * per_layer;
            kc[lo + (((size_t)dp * hkv + head) * 16 + di) * hd + d] = kc[lo + (((size_t)sp * hkv + head) * 16 + si) * hd + d];
            vc[lo + (((size_t)dp * hkv + head) * hd + d) * 16 + di] = vc[lo + (((size_t)sp * hkv + head) * hd + d) * 16 + si];
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    // pattern tail: the last w_max (at most 32) tokens of (old valid tail ++ emitted tokens), an entry per lane: all lanes
    // have loaded before the first one stores
    const int tl = tail_len[b], new_len = min(w_max, tl + no);
    if (tid < new_len) {
        int32_t* tb = tail + (size_t)b * w_max;
        const int ci = tl + no - new_len + tid;  // index in the concatenation
        tb[w_max - new_len + tid] = ci < tl ? tb[w_max - tl + ci] : out_tok[(size_t)b * k_stride + ci - tl];
    }
    if (tid != 0) return;
    tail_len[b] = new_len;
    // window rule: every drafted token on the path accepted <=> the last accepted node is a leaf
    if (pol.k_mode == HS_K_AIMD && nn > 1) {
        int last = path_row[(size_t)b * k_stride + a];
        bool leaf = true;
        for (int i = 1; i < nn; i++) if (parent[r0 + i] == last) { leaf = false; break; }
        int k = k_state[b];
        if (leaf && a > 0) k = min(k + pol.aimd_inc, pol.aimd_cap);
        else k = pol.aimd_reset;
        k_state[b] = k;
    }
    if (tokens) {
        for (int i = 0; i < no; i++)
            if (n_old + i < tokens_stride) tokens[(size_t)b * tokens_stride + n_old + i] = out_tok[(size_t)b * k_stride + i];
    }
    seq_len[b] = n_old + no;
    budget_left[b] -= no;
    if (counters) {
        atomicAdd(&counters[1], (unsigned long long)(nn - 1));
        atomicAdd(&counters[2], (unsigned long long)a);
        atomicAdd(&counters[3], (unsigned long long)no);
        atomicAdd(&counters[0], 1ull);
    }
}

// Acceptance and commit of one step in one launch (behind reject_stats_kernel's where it samples), one workgroup per sequence (either half can be switched off: the
// two entry points that run them separately use the same kernel).
//   1. With `keys` (the LM head ran with its row-maximum epilogue and no logits exist): every row's argmax = the
//      largest of its n_keys per-column-group keys, one wavefront per row; written to argmax[].
//   2. Acceptance: greedy walk (thread 0) or rejection sampling (the workgroup).
//   3. Commit.
struct accept_commit_args {
    int batch, vocab, k_stride, do_accept, do_commit;
    const int32_t *row_off, *tok, *parent, *pos;
    const float* logits;
    const unsigned long long* keys;
    int n_keys;
    const hs_reject_stat* stats;
    int n_slices;
    uint32_t call;
    int32_t* argmax;
    const uint64_t* seq_id;
    double inv_temp;
    uint64_t seed;
    int32_t *accept_len, *n_out, *out_tok, *path_row;
    // commit
    int n_layers, hkv, hd, n_blocks, max_blocks, w_max, tokens_stride;
    void *kc, *vc;
    const int32_t* block_table;
    int32_t *seq_len, *tail, *tail_len, *k_state, *budget_left, *tokens;
    unsigned long long* counters;
    hs_policy pol;
};

// REJECT: acceptance is rejection sampling; else greedy, or commit alone.  Two kernels, because the sampler takes
// nearly two hundred registers and the rest 23: in one kernel the greedy walk of more than 256 sequences ran in rounds of a
// workgroup per compute unit (greedy acceptance of 1024 trees of 17 nodes 40 us, on its own 16).
template <typename CT, bool REJECT>
__global__ __launch_bounds__(256, REJECT ? 1 : 7) void accept_commit_kernel(accept_commit_args p) {
    const int b = blockIdx.x, tid = threadIdx.x;
    const int r0 = p.row_off[b], nn = p.row_off[b + 1] - r0;
    if (p.do_accept) {
        if (nn <= 0) {
            if (tid == 0) { p.accept_len[b] = 0; p.n_out[b] = 0; }
        } else {
            if (!REJECT && p.keys) {
                const int lane = tid & 63, wave = tid >> 6;
                for (int r = wave; r < nn; r += 4) {
                    const unsigned long long* kr = p.keys + (size_t)(r0 + r) * p.n_keys;
                    unsigned long long best = 0ull;
                    for (int g = lane; g < p.n_keys; g += 64) {
                        const unsigned long long k = kr[g];
                        if (k > best) best = k;
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) {
                        const unsigned lo = __shfl_xor((unsigned)best, o), hi = __shfl_xor((unsigned)(best >> 32), o);
                        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
                        if (other > best) best = other;
                    }
                    if (lane == 0) p.argmax[r0 + r] = (int32_t)(0xFFFFFFFFu - (unsigned)best);
                }
                __syncthreads();   // the walk reads argmax[] written by the other wavefronts
            }
            if (REJECT) {
                accept_rejection_seq(b, r0, nn, p.vocab, p.tok, p.parent, p.pos, p.logits,
                                     p.stats, p.n_slices, p.call, p.seq_id, p.inv_temp, p.seed, p.k_stride, p.accept_len,
                                     p.n_out, p.out_tok, p.path_row);
            } else if (tid == 0) {
                accept_greedy_walk(b, r0, nn, p.tok, p.parent, p.argmax, p.k_stride, p.accept_len, p.n_out, p.out_tok,
                                   p.path_row);
            }
        }
        __syncthreads();           // the commit reads what thread 0 wrote
    }
    if (p.do_commit)
        commit_seq<CT>(b, p.n_layers, p.hkv, p.hd, p.n_blocks, (CT*)p.kc, (CT*)p.vc, p.block_table, p.max_blocks,
                       p.seq_len, p.tail, p.tail_len, p.w_max, p.k_state, p.budget_left, p.tokens, p.tokens_stride,
                       p.counters, p.row_off, p.parent, p.accept_len, p.n_out, p.out_tok, p.path_row, p.k_stride,
                       p.pol);
}

// The generator on its own: counter i -> its four output words (for bit-exact comparison with another
// implementation on many counters).
__global__ __launch_bounds__(256) void philox_debug_kernel(const uint32_t* __restrict__ ctr, uint32_t k0, uint32_t k1,
                                                            uint32_t* __restrict__ out, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    uint32_t o[4];
    philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1, o);
    out[4 * i] = o[0]; out[4 * i + 1] = o[1]; out[4 * i + 2] = o[2]; out[4 * i + 3] = o[3];
}

// The sums of a rejection-sampling call.  rows_hint: an estimate of the number of rows, or 0 (no result depends on it).
void launch_reject_stats(const hs_ctx* ctx, const accept_commit_args& a, int batch, int rows_hint, hs_reject_stat* stats, hipStream_t st) {
    reject_stage_args p = {a.row_off, a.tok, a.parent, a.pos, a.logits, batch, a.vocab, a.n_slices, a.k_stride, a.seq_id,
                           a.inv_temp, a.seed, a.call, stats, reinterpret_cast<uint4*>(ctx->ws + ctx->lay.reject_walk), 0};
    const int depth = ctx->lim.k_max + 1, nodes = 1 + ctx->lim.c_max * ctx->lim.k_max;
    const double row_mb = a.vocab * 4e-6;
    double mb = (double)batch * nodes * row_mb;
    if (rows_hint > 0) mb = std::min(mb, rows_hint * row_mb);
    // enough workgroups to fill the chip: small batches split a sequence's rows, too
    auto split = [&](int per_seq) { return dim3(batch, a.n_slices, std::max(1, std::min(2048 / (a.n_slices * batch), per_seq))); };
    if (depth < 3 || mb < (rows_hint > 0 ? HS_REJECT_STAGED_MB : HS_REJECT_STAGED_UNKNOWN_MB)) {
        p.all_rows = INT32_MAX;
        hipLaunchKernelGGL(reject_stats_kernel, split(nodes), dim3(256), 0, st, p, 1);
        return;
    }
    p.all_rows = (int)(HS_REJECT_STAGED_MB / 2 / row_mb);
    hipLaunchKernelGGL(reject_stats_kernel, split(1), dim3(256), 0, st, p, 1);
    for (int done = 1, levels = 2; done < depth; done += levels, levels *= 2) {
        if (depth - done - levels <= levels / 2) levels = depth - done;
        hipLaunchKernelGGL(reject_plan_kernel, dim3(batch), dim3(256), 0, st, p, done == 1, levels);
        dim3 grid = split(levels);
        grid.z = std::max(grid.z, 2u);     // (half of the walks are over: 32 trees 77 -> 71 us; four instead of two, 121 -> 123 of 64)
        hipLaunchKernelGGL(reject_stats_kernel, grid, dim3(256), 0, st, p, 0);
    }
}

}  // namespace

extern "C" hs_status hs_debug_philox(const uint32_t* ctr, uint64_t seed, uint32_t* out, int32_t n, hs_stream stream) {
    if (!ctr || !out || n < 0) return HS_ERR_INVALID_ARG;
    if (n == 0) return HS_OK;
    (void)hipGetLastError();
    hipLaunchKernelGGL(philox_debug_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, ctr,
                       (uint32_t)seed, (uint32_t)(seed >> 32), out, n);
    return hipGetLastError() == hipSuccess ? HS_OK : HS_ERR_HIP;
}

void hs_launch_accept_commit(const hs_ctx* ctx, const hs_accept_args* args, const hs_kv_cache* cache,
                             const hs_seq_state* seq, const hs_step* step, const float* logits,
                             const unsigned long long* keys, int n_keys, const hs_policy* policy, hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    accept_commit_args p = {};
    p.batch = seq->batch;
    p.vocab = d.vocab;
    p.k_stride = ctx->lim.k_max + 1;
    p.do_accept = args != nullptr;
    p.do_commit = policy != nullptr;
    p.row_off = step->row_off; p.tok = step->tok; p.parent = step->parent; p.pos = step->pos;
    p.logits = logits;
    p.keys = keys;
    p.n_keys = n_keys;
    p.argmax = step->argmax;
    p.seq_id = seq->seq_id;
    if (args) {
        // (at an infinite temperature every finite difference still scales to nothing against 1, while an excluded logit,
        // -inf, keeps the weight 0: -inf times a true 0 would be a NaN)
        p.inv_temp = args->mode == HS_ACCEPT_REJECTION ? std::max(1.0 / (double)args->temperature, 1e-300) : 1.0;
        p.seed = args->seed;
    }
    if (args && args->mode == HS_ACCEPT_REJECTION) {
        hs_reject_stat* stats = reinterpret_cast<hs_reject_stat*>(ctx->ws + ctx->lay.reject_stats);
        p.stats = stats;
        p.n_slices = hs_reject_slices(d.vocab);
        p.call = ctx->reject_calls.fetch_add(1, std::memory_order_relaxed);
        launch_reject_stats(ctx, p, seq->batch, step->rows_hint, stats, st);
    }
    p.accept_len = step->accept_len; p.n_out = step->n_out; p.out_tok = step->out_tok; p.path_row = step->path_row;
    if (policy) {
        p.n_layers = d.n_layers; p.hkv = d.n_kv_heads; p.hd = d.head_dim;
        p.n_blocks = cache->n_blocks; p.max_blocks = ctx->lim.max_blocks_per_seq;
        p.w_max = ctx->lim.w_max; p.tokens_stride = seq->tokens_stride;
        p.kc = cache->k; p.vc = cache->v;
        p.block_table = seq->block_table;
        p.seq_len = seq->seq_len; p.tail = seq->tail; p.tail_len = seq->tail_len; p.k_state = seq->k_state;
        p.budget_left = seq->budget_left; p.tokens = seq->tokens;
        p.counters = (unsigned long long*)seq->counters;
        p.pol = *policy;
    }
    const dim3 grid(seq->batch), block(256);
    const bool fp32 = hs_fp32_activations(ctx);
    if (args && args->mode == HS_ACCEPT_REJECTION) {
        const size_t lds = (size_t)p.n_slices * sizeof(slice_stat);
        const auto kernel = fp32 ? &accept_commit_kernel<float, true> : &accept_commit_kernel<bf16_t, true>;
        if (lds > 48 * 1024)   // (vocabularies beyond 12 million)
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kernel, grid, block, lds, st, p);
    } else {
        if (fp32) hipLaunchKernelGGL((accept_commit_kernel<float, false>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((accept_commit_kernel<bf16_t, false>), grid, block, 0, st, p);
    }
}
