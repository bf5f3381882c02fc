// Row-wise kernels of the verify forward pass: embedding gather, RMSNorm, rotary embedding + KV-cache write,
// and the per-row argmax over the vocabulary.  All are bandwidth-trivial next to attention and the GEMMs; each
// row is processed independently with a reduction order that depends only on the row's own length.
// The row count lives on the device, so a launch cannot size its grid to it: the grid is what the chip holds at
// once (hs_row_grid) and a workgroup takes rows blockIdx.x, blockIdx.x + gridDim.x, ...  A grid of max_rows
// workgroups, most of which only find that their row does not exist, costs several rounds of workgroup launches
// (a few microseconds) in each of the ~150 row-kernel launches of a step.
#include "hs_internal.h"
#include "hs_worklist.h"

namespace {

// A row's norm is a workgroup of norm_threads(d) threads, each with 4 elements in each of up to NORM_ITEMS rounds: thread t
// holds elements 4 t .. 4 t + 3, the same 4096 further on, ... (d_model <= 16384, checked by hs_create).
constexpr int NORM_ITEMS = 4, NORM_THREADS_MAX = 1024;

__device__ __forceinline__ void put(bf16_t* p, float v) { *p = f32_to_bf16(v); }
__device__ __forceinline__ void put(float* p, float v) { *p = v; }

// once, before the first block_sum (whose first barrier publishes it)
__device__ inline void clear_sums(float* red) {
    if (threadIdx.x < NORM_THREADS_MAX / 64) red[threadIdx.x] = 0.f;
}

__device__ inline float block_sum(float v, float* red) {
    // fixed tree: xor-shuffle inside each wavefront, then the wavefront sums left to right
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = red[0];
#pragma unroll
    for (int w = 1; w < NORM_THREADS_MAX / 64; w++) s += red[w];     // (0 beyond the last wavefront: clear_sums)
    return s;
}

__device__ __forceinline__ void put4(bf16_t* p, float4 v) {
    uint2 o;
    o.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
    o.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
    *reinterpret_cast<uint2*>(p) = o;
}
__device__ __forceinline__ void put4(float* p, float4 v) { p[0] = v.x; p[1] = v.y; p[2] = v.z; p[3] = v.w; }   // (any alignment)

typedef float f32x4 __attribute__((ext_vector_type(4)));

// four floats `bytes` from a pointer that all threads share (a 32-bit offset leaves the address in scalar registers)
template <typename T>
__device__ __forceinline__ T load4(const float* base, unsigned bytes) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}

template <typename OutT, int ITEMS>
__device__ inline void norm_row(const float4 (&v)[ITEMS], const float4 (&g)[ITEMS], bool store_x, float* xr,
                                OutT* out, int d, float eps, float* red) {
    // the sum of squares: same element-to-thread assignment and order wherever the row came from -- the norm must not
    // depend on which execution the preceding projection used
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < ITEMS; it++) {
        const int i = (threadIdx.x + it * blockDim.x) * 4;
        if (i >= d) continue;
        if (store_x) *reinterpret_cast<float4*>(xr + i) = v[it];
        // (fused multiply-adds written out, the very first one onto y y: a sum left to the compiler is rounded the one way
        // in one instance of the kernel and the other way in the next)
        ss = __builtin_fmaf(v[it].x, v[it].x, it == 0 ? v[it].y * v[it].y : ss);
        if (it > 0) ss = __builtin_fmaf(v[it].y, v[it].y, ss);
        ss = __builtin_fmaf(v[it].z, v[it].z, ss);
        ss = __builtin_fmaf(v[it].w, v[it].w, ss);
    }
    ss = block_sum(ss, red);
    const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int it = 0; it < ITEMS; it++) {
        const int i = (threadIdx.x + it * blockDim.x) * 4;
        if (i >= d) continue;
        float4 o;
        o.x = v[it].x * r * g[it].x; o.y = v[it].y * r * g[it].y;
        o.z = v[it].z * r * g[it].z; o.w = v[it].w * r * g[it].w;
        put4(out + i, o);
    }
}

// The first norm of a forward pass: the residual stream starts as the token's embedding.  The first list_groups
// workgroups write the attention's unit lists instead (nothing here depends on them), the others take rows.
// (As three launches -- 2-byte gathers, the lists by one workgroup, the norm reading the gathers back -- 28 us at 220 rows
// of 3584 and 128 sequences, now 6.5; 1067 rows of 5120: 45, now 19.)
template <typename OutT, int ITEMS>
__global__ __launch_bounds__(NORM_THREADS_MAX, ITEMS <= 2 ? 8 : 4) void embed_norm_kernel(
    const bf16_t* __restrict__ embed, const int32_t* __restrict__ tok, int vocab, float* __restrict__ x,
    const float* __restrict__ w, OutT* __restrict__ out, const int32_t* __restrict__ row_off, int batch, int d, float eps,
    int list_groups, hs_attn_lists lists, const int32_t* __restrict__ seq_len, hs_row_places places) {
    __shared__ float red[NORM_THREADS_MAX / 64];
    if ((int)blockIdx.x < list_groups) {
        hs_write_worklist(lists, places, seq_len, row_off, batch, blockIdx.x, list_groups);
        return;
    }
    clear_sums(red);
    const int m = row_off[batch];
    // (the embedding rows may start at any bf16: 8-byte loads where their base allows)
    const bool vec = ((unsigned long long)embed & 7ull) == 0;
    for (int row = (int)blockIdx.x - list_groups; row < m; row += (int)gridDim.x - list_groups) {
        int t = tok[row];
        if (t < 0 || t >= vocab) t = 0;
        const bf16_t* e = embed + (size_t)t * d;
        float4 v[ITEMS], g[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; it++) {
            const int i = (threadIdx.x + it * blockDim.x) * 4;
            if (i >= d) continue;
            g[it] = *reinterpret_cast<const float4*>(w + i);
            ushort4 b;
            if (vec) b = *reinterpret_cast<const ushort4*>(e + i);
            else b = make_ushort4(e[i], e[i + 1], e[i + 2], e[i + 3]);
            v[it] = make_float4(bf16_to_f32(b.x), bf16_to_f32(b.y), bf16_to_f32(b.z), bf16_to_f32(b.w));
        }
        norm_row<OutT, ITEMS>(v, g, true, x + (size_t)row * d, out + (size_t)row * d, d, eps, red);
    }
}

// One workgroup per row.  With chunks > 0 the row of the residual stream first receives the pending partial sums of
// the preceding projection: t = p0 + p1 + ... in chunk order, x += t -- the arithmetic of the stand-alone ordered
// reduce, so that the split execution gives the same bits whichever kernel finishes it.
// OutT = bf16_t (rounded activations) or float (fp32-activation mode).
// The kernel is a chain of memory round trips, not a stream: a thread keeps its (up to NORM_ITEMS x 4) elements in
// registers from the first load to the normalised store, and the norm weights are fetched with them.  With many rows the
// other rows of a compute unit hide the chain: 64 registers and eight wavefronts per SIMD, so that two workgroups of 1024 threads
// share one and the grid (hs_row_grid) is resident.  EARLY, for a few rows (hs_early_rows), hides it by what is on its way at
// once: the row count, the row and ten partials of it, in 70 registers.  us, 64 registers and 70: 1078 rows of 3584 with nine
// partials 29.0 and 33.3, of 4096 with seven 30.1 and 33.6, of 3584 with none 7.6 and 10.2; 540 rows 17.2 and 19.0; 7 rows
// of 1536 with ten 4.3 and 3.7.
template <typename OutT, int ITEMS, bool EARLY>
__global__ __launch_bounds__(NORM_THREADS_MAX, ITEMS > 2 ? 4 : EARLY && ITEMS == 1 ? 7 : 8) void rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ w,
                                                       OutT* __restrict__ out, const int32_t* m_dev,
                                                       int d, float eps,
                                                       const float* __restrict__ part, int chunks, int pending_rows,
                                                       size_t chunk_stride, int early) {
    __shared__ float red[NORM_THREADS_MAX / 64];
    clear_sums(red);
    int row = blockIdx.x, m = EARLY && row < early ? INT32_MAX : *m_dev;
    if (row >= m) return;
    if (!EARLY && m > pending_rows) chunks = 0;     // (where few rows are expected, partials pend whatever their number)
    for (;;) {
        // (EARLY: all of a row's loads inside the loop; one that is moved in front of it is waited for there)
        const unsigned zero = EARLY ? hs_opaque_zero() : 0u;
        int m_lane = m;
        if constexpr (EARLY) m_lane = m_dev[zero];
        float* xr = x + (size_t)row * d;
        const float* pr = part + (size_t)row * d;
        float4 v[ITEMS], g[ITEMS];
        unsigned at[ITEMS]; // byte offsets (beyond the row's end its last elements': no branch between the loads)
#pragma unroll
        for (int it = 0; it < ITEMS; it++) {
            at[it] = min((int)(threadIdx.x + it * blockDim.x) * 4, d - 4) * 4u + zero;
            v[it] = load4<float4>(xr, at[it]);
            g[it] = load4<float4>(w, at[it]);
        }
        if (chunks > 0) {
            // PER partials of each element in flight at once (written out: left to itself the compiler waits for each)
            constexpr int PER = ITEMS == 1 ? (EARLY ? 10 : 5) : ITEMS == 2 ? 3 : 2;
            float4 t[ITEMS];
            const float* pc = pr;
            for (int c0 = 0; c0 < chunks; c0 += PER) {
                f32x4 q[PER][ITEMS];
#pragma unroll
                for (int j = 0; j < PER; j++)
                    if (c0 + j < chunks) {
#pragma unroll
                        for (int it = 0; it < ITEMS; it++)
                            q[j][it] = load4<f32x4>(pc, at[it]);
                        pc += chunk_stride;
                    }
                hs_loads_issued();
#pragma unroll
                for (int j = 0; j < PER; j++)
                    if (c0 + j < chunks) {
#pragma unroll
                        for (int it = 0; it < ITEMS; it++) {
                            const f32x4 u = q[j][it];
                            if (c0 + j == 0) t[it] = make_float4(u.x, u.y, u.z, u.w);
                            else { t[it].x += u.x; t[it].y += u.y; t[it].z += u.z; t[it].w += u.w; }
                        }
                    }
            }
#pragma unroll
            for (int it = 0; it < ITEMS; it++) {
                v[it].x += t[it].x; v[it].y += t[it].y; v[it].z += t[it].z; v[it].w += t[it].w;
            }
        }
        if constexpr (EARLY) {
            m = hs_uniform(m_lane);
            if (row >= m) return;
        }
        norm_row<OutT, ITEMS>(v, g, chunks > 0, xr, out + (size_t)row * d, d, eps, red);
        row += gridDim.x;
        if (row >= m) return;
    }
}

template <typename OutT, int ITEMS>
constexpr auto early_rmsnorm = &rmsnorm_kernel<OutT, ITEMS, true>;
template <typename OutT, int ITEMS>
constexpr auto counted_rmsnorm = &rmsnorm_kernel<OutT, ITEMS, false>;

// Rotates q and k heads at the row's position (pairs i, i + h/2), writes q as bf16, K into its page row-major and V into
// its page with the token index fastest.  T = bf16_t, or float in the fp32-activation mode (queries and cache entries
// then keep every bit).
// One workgroup per row, an item per thread: four neighbouring pairs of a q or k head, or four elements of a v head.  A
// thread adds up its own elements' pending partials (chunk order) and rotates them; nothing passes through LDS, no
// barrier, and the loads depend on nothing but the row, as does that of the row's place (hs_row_info).  Bound by the partial
// sums it reads.  With the row gathered in LDS by 1024 threads first:
// 74 us for 4096 rows of 4608 in three chunks, 28 us for 1067 rows of 7168 in two, 28 us
// for 2048 rows of 2048 in six; now 70, 25 and 21 (2.7 to 5 TB/s of partial sums).
// EARLY as in the norm: with few rows six chunks in flight and 70 registers (74 where T is float), else three and 64, for eight
// wavefronts per SIMD: two workgroups of 1024 threads (40 and 8 heads of 128) share a compute unit.  us, 64 registers and 70:
// 540 rows of that shape 12.5 and 12.9, 1078 rows 20.0 and 20.2, of 28 and 4 heads 10.6 and 11.1; 7 rows of 12 and 2 heads
// in six chunks 4.4 and 3.7.
template <typename T, bool EARLY>
__global__ __launch_bounds__(1024, EARLY ? 4 : 8) void rope_kv_kernel(const float* __restrict__ qkv, const float* __restrict__ rope_cs,
                                                       const hs_row_info* infos, const int32_t* m_dev, T* __restrict__ q_out,
                                                       T* __restrict__ kc, T* __restrict__ vc, size_t layer_off, int hq,
                                                       int hkv, int h, const float* __restrict__ part, int chunks,
                                                       int pending_rows, size_t chunk_stride, int early, int by_page) {
    const int half = h >> 1, per_head = half >> 2;         // items of a q or k head
    const int n_rot = (hq + hkv) * per_head, n_items = n_rot + hkv * (h >> 2);
    const int nqkv = (hq + 2 * hkv) * h;
    const bool cs_vec = ((unsigned long long)rope_cs & 15ull) == 0;
    // by_page: of 128 neighbouring rows 16 at a time go to one XCD (workgroups are dealt to the eight of them in turn; the grid
    // is a multiple of 128).
    int row = blockIdx.x;
    if (by_page) row = (row & ~127) | (row & 7) << 4 | (row >> 3 & 15);
    int m = EARLY && row < early ? INT32_MAX : *m_dev;
    if (row >= m) return;
    if (!EARLY && m > pending_rows) chunks = 0;     // (where few rows are expected, partials pend whatever their number)
    for (;;) {
        const float* src = (chunks > 0 ? part : qkv) + (size_t)row * nqkv;
        const int n_src = chunks > 0 ? chunks : 1;
        if constexpr (EARLY) m = 0;      // (stays 0 for a wavefront without items; lane 0 has one if any lane has)
        for (int i = threadIdx.x; i < n_items; i += blockDim.x) {
            const unsigned zero = EARLY ? hs_opaque_zero() : 0u;     // (all of an item's loads inside the loop, as in the norm)
            int m_lane = m;
            if constexpr (EARLY) m_lane = m_dev[zero];
            const hs_row_info info = infos[row + zero];
            const bool rot = i < n_rot;
            const int head = rot ? i / per_head : hq + hkv + (i - n_rot) / (h >> 2);      // head of the QKV vector
            const int j = rot ? 4 * (i % per_head) : 4 * ((i - n_rot) % (h >> 2));        // first element in it
            // PER chunks in flight at once (v items load their elements twice: no branch between the loads)
            constexpr int PER = EARLY ? 6 : 3;
            const unsigned at = (unsigned)(head * h + j) * 4u, at_y = at + (rot ? (unsigned)half * 4u : 0u);
            const float* pc = src;
            float4 x, y;
            for (int c0 = 0; c0 < n_src; c0 += PER) {
                f32x4 qx[PER], qy[PER];
#pragma unroll
                for (int c = 0; c < PER; c++)
                    if (c0 + c < n_src) {
                        qx[c] = load4<f32x4>(pc, at);
                        qy[c] = load4<f32x4>(pc, at_y);
                        pc += chunk_stride;
                    }
                hs_loads_issued();
#pragma unroll
                for (int c = 0; c < PER; c++)
                    if (c0 + c < n_src) {
                        const f32x4 t = qx[c], u = qy[c];
                        if (c0 + c == 0) {
                            x = make_float4(t.x, t.y, t.z, t.w);
                            y = make_float4(u.x, u.y, u.z, u.w);
                        } else {
                            x.x += t.x; x.y += t.y; x.z += t.z; x.w += t.w;
                            y.x += u.x; y.y += u.y; y.z += u.z; y.w += u.w;
                        }
                    }
            }
            // (no such row, or one that writes nothing: the same for all threads of the workgroup)
            const int place = hs_uniform(info.slot);
            if constexpr (EARLY) m = hs_uniform(m_lane);
            if (row >= m || place < 0) break;
            const int page = place >> 4, in_page = place & 15;
            if (!rot) {   // v head -> cache [page][kv head][h][16]
                T* dst = vc + layer_off + (((size_t)page * hkv + (head - hq - hkv)) * h + j) * 16 + in_page;
                put(dst, x.x); put(dst + 16, x.y); put(dst + 32, x.z); put(dst + 48, x.w);
                continue;
            }
            const float* cs = rope_cs + ((size_t)hs_uniform(info.pos) * half + j) * 2;
            float4 c0, c1;   // (cos, sin) of pairs j, j + 1 and j + 2, j + 3
            if (cs_vec) {
                c0 = *reinterpret_cast<const float4*>(cs);
                c1 = *reinterpret_cast<const float4*>(cs + 4);
            } else {
                c0 = make_float4(cs[0], cs[1], cs[2], cs[3]);
                c1 = make_float4(cs[4], cs[5], cs[6], cs[7]);
            }
            float4 lo, hi;
            // (fused multiply-adds written out: left to contract x s + y c by itself the compiler rounds one product of the
            // four pairs' second halves the other way round, and results change with the shape of the code)
            lo.x = __builtin_fmaf(x.x, c0.x, -(y.x * c0.y)); hi.x = __builtin_fmaf(x.x, c0.y, y.x * c0.x);
            lo.y = __builtin_fmaf(x.y, c0.z, -(y.y * c0.w)); hi.y = __builtin_fmaf(x.y, c0.w, y.y * c0.z);
            lo.z = __builtin_fmaf(x.z, c1.x, -(y.z * c1.y)); hi.z = __builtin_fmaf(x.z, c1.y, y.z * c1.x);
            lo.w = __builtin_fmaf(x.w, c1.z, -(y.w * c1.w)); hi.w = __builtin_fmaf(x.w, c1.w, y.w * c1.z);
            // k heads -> cache [page][kv head][16][h]
            T* dst = head < hq ? q_out + ((size_t)row * hq + head) * h + j
                               : kc + layer_off + (((size_t)page * hkv + (head - hq)) * 16 + in_page) * h + j;
            put4(dst, lo);
            put4(dst + half, hi);
        }
        row += gridDim.x;
        if (row >= hs_uniform(m)) return;
    }
}

// One workgroup of 16 wavefronts per row; 16-byte loads where the row is aligned, four of a thread on their way at once.  Ties
// resolve to the lowest id at every level, so the result is the first maximum whatever the reduction shape.
// (The last, incomplete four by a loop of their own.  Clamped to the row's end and loaded all the same: 220 rows of 16448
// columns 7.1 us, now 6.4, 1078 of 4096 12.9, now 10.2; one load after the other: 220 rows of 152064 24.9, now 22.4.)
__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ logits, int32_t* __restrict__ out,
                                                       const int32_t* m_dev, int vocab, int early) {
    __shared__ float sv[16];
    __shared__ int si[16];
    int row = blockIdx.x;
    if (row >= early && row >= *m_dev) return;
    for (;;) {
        const int m_lane = m_dev[hs_opaque_zero()];
        if (row != (int)blockIdx.x) __syncthreads();  // the previous row's candidates have been read
        const float* l = logits + (size_t)row * vocab;
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        auto take = [&](float v, int i) { if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; } };
        if ((vocab & 3) == 0) {
            const float4* l4 = reinterpret_cast<const float4*>(l);
            const int n4 = vocab / 4;
            int i = threadIdx.x;
            for (int end = 4 * 1024; end <= n4; end += 4 * 1024) {
                float4 v[4];
#pragma unroll
                for (int j = 0; j < 4; j++) v[j] = l4[i + 1024 * j];
                hs_loads_issued();
                // (behind the first loads the count has arrived: of a row that does not exist 64 KB are read, not its whole vocabulary)
                if (row >= hs_uniform(m_lane)) return;
#pragma unroll
                for (int j = 0; j < 4; j++, i += 1024) {
                    take(v[j].x, 4 * i); take(v[j].y, 4 * i + 1); take(v[j].z, 4 * i + 2); take(v[j].w, 4 * i + 3);
                }
            }
            for (; i < n4; i += 1024) {
                float4 v = l4[i];
                take(v.x, 4 * i); take(v.y, 4 * i + 1); take(v.z, 4 * i + 2); take(v.w, 4 * i + 3);
            }
        } else if (row < hs_uniform(m_lane)) {
            for (int i = threadIdx.x; i < vocab; i += 1024) take(l[i], i);
        }
        const int m = hs_uniform(m_lane);
        if (row >= m) return;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            float ov = __shfl_xor(bv, o);
            int oi = __shfl_xor(bi, o);
            take(ov, oi);
        }
        if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 16; w++) take(sv[w], si[w]);
            out[row] = bi;
        }
        row += gridDim.x;
        if (row >= m) return;
    }
}

// Rows of one prefill call: sequence b contributes its next n_b = min(chunk, seq_len - 1 - kv_done) tokens (taken
// from its token log), sequences served in index order until max_rows rows are laid out.  One workgroup.
// len_plus1[b] = kv_done[b] + 1 before the call (the later kernels' "sequence length": cached positions + 1);
// kv_done advances by n_b.
__global__ __launch_bounds__(1024) void prefill_rows_kernel(
    const int32_t* __restrict__ seq_len, int32_t* __restrict__ kv_done, const int32_t* __restrict__ tokens,
    int tokens_stride, int batch, int chunk, int max_rows, int max_pos, const int32_t* __restrict__ block_table,
    int max_blocks, int32_t* __restrict__ row_off,
    int32_t* __restrict__ tok, int32_t* __restrict__ pos, int32_t* __restrict__ parent, int32_t* __restrict__ row2seq,
    int32_t* __restrict__ len_plus1, uint32_t* __restrict__ err, int n_blocks, hs_row_info* __restrict__ infos) {
    __shared__ int sw[16];
    __shared__ int s_first[1024], s_n[1024], s_done[1024];
    __shared__ int carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int b0 = 0; b0 < batch; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        int want = 0, done = 0;
        if (b < batch) {
            done = max(kv_done[b], 0);
            want = max(0, min(chunk, seq_len[b] - 1 - done));
            if (done + want > max_pos) {        // rotary table too short: nothing of this sequence is laid out
                atomicOr(err, (uint32_t)HS_DEV_POSITION_OVERFLOW);
                want = 0;
            } else if (want > 0 && (done + want > max_blocks * 16 ||
                                    block_table[(size_t)b * max_blocks + ((done + want - 1) >> 4)] < 0)) {
                // the sequence outgrows its block table (or the pages the caller gave it): likewise
                atomicOr(err, (uint32_t)HS_DEV_BLOCK_TABLE_OVERFLOW);
                want = 0;
            }
        }
        int incl = want;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) sw[wave] = incl;
        __syncthreads();
        int before = carry_s;
        for (int w2 = 0; w2 < wave; w2++) before += sw[w2];
        const int start = before + incl - want;
        if (b < batch) {
            const int s0 = min(start, max_rows);
            const int n = max(0, min(want, max_rows - s0));
            row_off[b] = s0;
            len_plus1[b] = done + 1;
            kv_done[b] = done + n;
            s_first[threadIdx.x] = s0;
            s_n[threadIdx.x] = n;
            s_done[threadIdx.x] = done;
        }
        __syncthreads();
        // A thread per row, four at a time, so that the rows' tokens and pages come in one trip to memory however few sequences
        // there are; a row's sequence is the last one that starts at or before it (those without rows start where the next one does).
        // (A wavefront per sequence: five sequences of 2048 rows 13.6 us, now 7.8; eight of 4096 10.1, now 9.3.)
        const int nb = min(1024, batch - b0), end = s_first[nb - 1] + s_n[nb - 1];
        for (int r0 = s_first[0] + threadIdx.x; r0 < end; r0 += 4 * 1024) {
            int q[4], t[4];
            hs_row_info info[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int r = min(r0 + 1024 * j, end - 1);
                int lo = 0;
                for (int step = 512; step > 0; step >>= 1)
                    if (lo + step < nb && s_first[lo + step] <= r) lo += step;
                const int at = s_done[lo] + r - s_first[lo];
                q[j] = lo;
                t[j] = tokens[(size_t)(b0 + lo) * tokens_stride + at];
                info[j] = hs_place_row(block_table + (size_t)(b0 + lo) * max_blocks, max_blocks, n_blocks, max_pos, at, at, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int r = r0 + 1024 * j;
                if (r < end) {
                    tok[r] = t[j];
                    pos[r] = info[j].pos;
                    parent[r] = r - s_first[q[j]] - 1;
                    row2seq[r] = b0 + q[j];
                    infos[r] = info[j];
                }
            }
        }
        if (threadIdx.x == 1023) carry_s = before + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) row_off[batch] = min(carry_s, max_rows);
}

}  // namespace

void hs_launch_prefill_rows(const hs_ctx* ctx, const hs_kv_cache* cache, const hs_seq_state* seq, int32_t* kv_done, int chunk, hs_step* step,
                            int32_t* len_plus1, hipStream_t st) {
    hipLaunchKernelGGL(prefill_rows_kernel, dim3(1), dim3(1024), 0, st, seq->seq_len, kv_done, seq->tokens,
                       seq->tokens_stride, seq->batch, chunk, ctx->lim.max_rows, ctx->lim.max_pos, seq->block_table,
                       ctx->lim.max_blocks_per_seq, step->row_off,
                       step->tok, step->pos, step->parent, step->row2seq, len_plus1,
                       reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.err), cache->n_blocks,
                       reinterpret_cast<hs_row_info*>(ctx->ws + ctx->lay.row_info));
}

// Rounds of a row's elements over its workgroup, and its threads: one round where 1024 threads hold the row, no more threads
// than it has elements for, and at least 256 (the list writers).
static int norm_rounds(int d) { return std::min(NORM_ITEMS, (d / 4 + NORM_THREADS_MAX - 1) / NORM_THREADS_MAX); }
static int norm_threads(int d) { return std::max(256, std::min(NORM_THREADS_MAX, (d / 4 + 63) / 64 * 64)); }

#define HS_NORM_LAUNCH(KERNEL, OUT, GRID, ...)                                                                        \
    switch (norm_rounds(d.d_model)) {                                                                                 \
        case 1: hipLaunchKernelGGL((KERNEL<OUT, 1>), GRID, block, 0, st, __VA_ARGS__); break;                         \
        case 2: hipLaunchKernelGGL((KERNEL<OUT, 2>), GRID, block, 0, st, __VA_ARGS__); break;                         \
        case 3: hipLaunchKernelGGL((KERNEL<OUT, 3>), GRID, block, 0, st, __VA_ARGS__); break;                         \
        default: hipLaunchKernelGGL((KERNEL<OUT, 4>), GRID, block, 0, st, __VA_ARGS__);                               \
    }

void hs_launch_embed_norm(const hs_ctx* ctx, const hs_kv_cache* cache, const hs_seq_state* seq, const hs_step* step,
                          bool lists, float* x, const float* w, void* out, hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    static_assert(HS_LIST_THREADS == NORM_THREADS_MAX, "the list writers are workgroups of this launch");
    const dim3 block(norm_threads(d.d_model));
    const int groups = lists ? hs_list_groups(block.x) : 0;
    const hs_attn_lists l = lists ? hs_attention_lists(ctx) : hs_attn_lists{};
    const dim3 grid(hs_row_grid(ctx, block.x) + groups);
    const hs_row_places pl = hs_row_places_of(ctx, cache, seq, step);
    if (hs_fp32_activations(ctx)) {
        HS_NORM_LAUNCH(embed_norm_kernel, float, grid, ctx->embed, step->tok, d.vocab, x, w, (float*)out, step->row_off,
                       seq->batch, d.d_model, d.rms_eps, groups, l, seq->seq_len, pl)
    } else {
        HS_NORM_LAUNCH(embed_norm_kernel, bf16_t, grid, ctx->embed, step->tok, d.vocab, x, w, (bf16_t*)out, step->row_off,
                       seq->batch, d.d_model, d.rms_eps, groups, l, seq->seq_len, pl)
    }
}

void hs_launch_rmsnorm(const hs_ctx* ctx, float* x, const float* w, void* out, const int32_t* m_dev,
                       hs_pending pending, int expected, hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    const float* part = reinterpret_cast<const float*>(ctx->ws + ctx->lay.gemm_part);
    const size_t stride = (size_t)ctx->lim.max_rows * d.d_model;
    const dim3 block(norm_threads(d.d_model)), grid(hs_row_grid(ctx, block.x));
    const int early = hs_early_rows(expected);
#define HS_ARGS(T) x, w, (T*)out, m_dev, d.d_model, d.rms_eps, part, pending.chunks, pending.rows, stride, early
    if (hs_fp32_activations(ctx)) {
        if (early) { HS_NORM_LAUNCH(early_rmsnorm, float, grid, HS_ARGS(float)) }
        else { HS_NORM_LAUNCH(counted_rmsnorm, float, grid, HS_ARGS(float)) }
    } else {
        if (early) { HS_NORM_LAUNCH(early_rmsnorm, bf16_t, grid, HS_ARGS(bf16_t)) }
        else { HS_NORM_LAUNCH(counted_rmsnorm, bf16_t, grid, HS_ARGS(bf16_t)) }
    }
#undef HS_ARGS
}
#undef HS_NORM_LAUNCH

// From this many expected rows on, neighbouring rows go to one XCD in sets of 16.  A page of V holds 16 positions side by side, 2
// bytes each: rows of a sequence that are dealt to eight XCDs write parts of the same 32 bytes into eight L2s, and each goes to
// memory on its own.  us, dealt in turn and in sets: 4096 rows of 4608 columns 32.4, 27.0; 1078 rows 14.2, 11.6; 1088 of 7168
// 21.4, 18.8; 2048 of 2048 9.8, 8.3.  (With few rows sets of 16 would leave XCDs without any.)
constexpr int HS_PAGE_ROWS = 512;

void hs_launch_rope_kv(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                       const hs_step* step, const float* qkv, void* q, hs_pending pending, int expected,
                       hipStream_t st) {
    const hs_model_desc& d = ctx->desc;
    size_t layer_off = (size_t)layer * cache->n_blocks * d.n_kv_heads * 16 * d.head_dim;
    const float* part = reinterpret_cast<const float*>(ctx->ws + ctx->lay.gemm_part);
    const hs_row_info* infos = reinterpret_cast<const hs_row_info*>(ctx->ws + ctx->lay.row_info);
    const size_t nqkv = (size_t)(d.n_q_heads + 2 * d.n_kv_heads) * d.head_dim;
    // an item per thread if a workgroup has that many, else as many rounds of equal size as it takes
    const int items = (d.n_q_heads + d.n_kv_heads) * (d.head_dim / 8) + d.n_kv_heads * (d.head_dim / 4);
    const int rounds = (items + 1023) / 1024, threads = ((items + rounds - 1) / rounds + 63) / 64 * 64;
    const int by_page = expected >= HS_PAGE_ROWS, early = hs_early_rows(expected), resident = hs_row_grid(ctx, threads);
    static_assert(HS_PAGE_ROWS > HS_EARLY_ROWS, "a grid beyond max_rows: the count comes before anything is read");
    const dim3 grid(by_page ? (resident + 127) / 128 * 128 : resident), block(threads);      // (whole sets of 128)
#define HS_ROPE_ARGS(T)                                                                                          \
    qkv, ctx->rope_cs, infos, step->row_off + seq->batch, (T*)q, (T*)cache->k, (T*)cache->v, layer_off,          \
        d.n_q_heads, d.n_kv_heads, d.head_dim, part, pending.chunks, pending.rows, (size_t)ctx->lim.max_rows * nqkv, early, by_page
    if (hs_fp32_activations(ctx)) {
        if (early) hipLaunchKernelGGL((rope_kv_kernel<float, true>), grid, block, 0, st, HS_ROPE_ARGS(float));
        else hipLaunchKernelGGL((rope_kv_kernel<float, false>), grid, block, 0, st, HS_ROPE_ARGS(float));
    } else {
        if (early) hipLaunchKernelGGL((rope_kv_kernel<bf16_t, true>), grid, block, 0, st, HS_ROPE_ARGS(bf16_t));
        else hipLaunchKernelGGL((rope_kv_kernel<bf16_t, false>), grid, block, 0, st, HS_ROPE_ARGS(bf16_t));
    }
#undef HS_ROPE_ARGS
}

void hs_launch_argmax(const hs_ctx* ctx, const float* logits, int32_t* argmax, const int32_t* m_dev,
                      int expected, hipStream_t st) {
    hipLaunchKernelGGL(argmax_kernel, dim3(hs_row_grid(ctx, 1024)), dim3(1024), 0, st, logits, argmax, m_dev,
                       ctx->desc.vocab, hs_early_rows(expected));
}
