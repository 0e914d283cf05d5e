// Device code shared by the gate kernels (gate.hip) and by the launches of a decode-sized block that can carry the next
// block's pre-gate in a few extra workgroups (expert FFN: ffn.hip, combine: combine.hip): reductions over a
// group of 16 lanes, softmax / top-k, token grouping inside a workgroup, the body of the
// smallest gate (at most GS_TOK tokens, 8 or 16 experts) and the matrix-core gate in two halves.
#ifndef PGMOE_GATE_SMALL_H
#define PGMOE_GATE_SMALL_H
#include <climits>

#include "pgmoe_internal.h"
#include "wave.h"

namespace pgmoe {

// Reductions over a group of 16 lanes (one DPP row) by rotating the row by 8, 4, 2 and 1 lanes:
// every lane ends with the reduction over all 16, each step is one VALU operation (no LDS
// crossbar traffic as with a shuffle).  All 64 lanes of the wavefront must be active.
template <int N>
__device__ inline int row_ror(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);  // row_ror:N
}
template <int N>
__device__ inline float row_ror(float v) {
    return __int_as_float(row_ror<N>(__float_as_int(v)));
}
__device__ inline float group_sum(float s) {  // fixed order: bit-reproducible
    s += row_ror<8>(s);
    s += row_ror<4>(s);
    s += row_ror<2>(s);
    return s + row_ror<1>(s);
}
__device__ inline int group_max(int m) {
    m = max(m, row_ror<8>(m));
    m = max(m, row_ror<4>(m));
    m = max(m, row_ror<2>(m));
    return max(m, row_ror<1>(m));
}
__device__ inline int group_min(int m) {
    m = min(m, row_ror<8>(m));
    m = min(m, row_ror<4>(m));
    m = min(m, row_ror<2>(m));
    return min(m, row_ror<1>(m));
}
// Integers in the order of the floats (no NaN; +0 and -0 are one), and back.
__device__ inline int sort_key(float v) {
    const int b = __float_as_int(v + 0.f);
    return b ^ (b >> 31 & 0x7fffffff);
}
__device__ inline float sort_value(int key) { return __int_as_float(key ^ (key >> 31 & 0x7fffffff)); }

// Softmax over the E logits of each token and k rounds of arg-max (ties to the lowest index,
// NaN ranks as -infinity and raises the NaN flag).  zs: LDS [tokens][zstride] logits.
// Sixteen lanes per token, so a wavefront works on four tokens at once; lane s of a group holds
// experts s, s+16, s+32, ...: NQ of them (compile time, E <= 16*NQ), fully unrolled without a
// branch per slice (a skipped slice of a 16-slice version still costs its branch, some 60 clocks,
// which is what a batch-1 gate with 8 experts then spends its time on).
// A round of arg-max is a maximum over sort keys, then the lowest index among the keys that equal it, each over the lane's slices and by
// rotation: one operation a step, where (value, index) pairs took seven. With 128 experts and two choices that was 5000
// of the 18500 clocks of a gate.
template <int NQ>
__device__ inline void softmax_topk_n(const float *zs, int zstride, int t0, int nt, int E, int k,
                                      int32_t *__restrict__ idx_out, float *__restrict__ prob_out,
                                      float *__restrict__ probs_out, uint32_t *flags, int32_t *idx_lds, float *prob_lds = nullptr) {
    const int tid = threadIdx.x;
    const int sub = tid & 15, grp = tid >> 4;  // 16 lanes per group
    constexpr int NONE = INT_MIN;              // key of an expert that does not exist or has been chosen
    int nans = 0;
    for (int tb = 0; tb < nt; tb += (int)blockDim.x / 16) {
        if (tb + (grp & ~3) >= nt) continue;  // none of this wavefront's four tokens exists (uniform over the wavefront)
        const int t = tb + grp;
        const bool live = t < nt;  // idle groups of a live wavefront work on its first token and skip the writes
        const float *row = zs + (live ? t : tb + (grp & ~3)) * zstride + sub;  // zstride >= 16 * NQ
        float v[NQ];
        int key[NQ], top = NONE;
        bool any_nan = false;
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = row[16 * q];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const bool real = sub + 16 * q < E, nan = v[q] != v[q];
            any_nan |= real && nan;
            v[q] = real && !nan ? v[q] : -INFINITY;
            key[q] = real ? sort_key(v[q]) : NONE;
            top = max(top, key[q]);
        }
        nans |= any_nan ? 1 : 0;
        asm volatile("" : "+v"(nans));  // as a lane mask over the loop it cost the matrix-core gates their last scalar registers and a stack frame: 9.6 -> 9.4 us a
                                          // gate of 4096 tokens, 1024 x 128, one behind the other, 23.2 -> 22.1 waited for
        top = group_max(top);
        const float m = sort_value(top);
        float p[NQ], s = 0.f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            p[q] = (sub + 16 * q < E) ? expf(v[q] - m) : 0.f;
            s += p[q];
        }
        s = group_sum(s);
        const float inv = 1.f / s;
        const size_t tok = (size_t)(t0 + t);
        if (probs_out && live) {
            float *out = probs_out + tok * E + sub;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (sub + 16 * q < E) out[16 * q] = p[q] * inv;
        }
        for (int j = 0;;) {
            int bi = INT_MAX;
#pragma unroll
            for (int q = NQ - 1; q >= 0; --q) bi = key[q] == top ? sub + 16 * q : bi;
            bi = group_min(bi);
            if (sub == 0 && live) {
                const float prob = expf(sort_value(top) - m) * inv;
                idx_out[tok * k + j] = bi;
                prob_out[tok * k + j] = prob;
                if (idx_lds) idx_lds[t * k + j] = bi;
                if (prob_lds) prob_lds[t * k + j] = prob;
            }
            if (++j >= k) break;  // uniform
            top = NONE;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                key[q] = sub + 16 * q == bi ? NONE : key[q];  // the lane that holds the winner retires it
                top = max(top, key[q]);
            }
            top = group_max(top);
        }
    }
    if (__any(nans) && (tid & 63) == 0) atomicOr(flags, kFlagNaN);
}

// MAXQ: the most slices the calling kernel can need (E <= 16*MAXQ there).
template <int MAXQ = 16>
__device__ inline void softmax_topk(const float *zs, int zstride, int t0, int nt, int E, int k,
                                    int32_t *__restrict__ idx_out, float *__restrict__ prob_out,
                                    float *__restrict__ probs_out, uint32_t *flags,
                                    int32_t *idx_lds = nullptr) {  // nullable: LDS copy [nt*k] of the chosen indices
#define PG_SOFTMAX(NQ_) softmax_topk_n<NQ_>(zs, zstride, t0, nt, E, k, idx_out, prob_out, probs_out, flags, idx_lds)
    if (E <= 16) PG_SOFTMAX(1);  // uniform over the kernel
    else if (E <= 32) PG_SOFTMAX(2);
    else if (E <= 64) PG_SOFTMAX(4);
    else if (MAXQ <= 8 || E <= 128) PG_SOFTMAX(8);
    else PG_SOFTMAX(16);
#undef PG_SOFTMAX
}

// Token grouping inside a gate kernel whose single workgroup holds the whole (decode-sized)
// batch: the same integers as route_kernel (counts, exclusive prefix sum, stable rank, inverse
// map), from the LDS copy r_idx[n_sel] of the chosen experts.  r_cnt, r_off: LDS [E] each.  Up to 64 selections one wavefront does it with
// ballots over the bits of the expert numbers, instead of three loops over LDS: the gate of 16 tokens and 64 experts with this and the arg-max above
// 9.8 -> 6.3 us, the combine that carries its second half 5.8 -> 4.7.
__device__ inline void group_in_workgroup(const int32_t *r_idx, int32_t *r_cnt, int32_t *r_off, int n_sel, int E, int k,
                                          int n_threads, int32_t *__restrict__ row_of, int32_t *__restrict__ offsets,
                                          int32_t *__restrict__ src_row) {
    const int tid = threadIdx.x;
    __syncthreads();
    // Uniform, and known at compile time to the batch-1 stack, which has no registers for the general case (171 -> 176 and a stack frame; without: six blocks of 768 x 3072
    // 44.9 -> 44.0 us one step behind the other, 56.4 -> 55.7 waited for).
    if (n_sel == 1) {
        for (int e = tid; e <= E; e += n_threads) offsets[e] = e > r_idx[0] ? 1 : 0;
        if (tid == 0) row_of[0] = src_row[0] = 0;
        return;
    }
    if (n_sel <= 64) {  // uniform: one wavefront, an entry a lane, in registers
        if (tid >= 64) return;
        const int mine = tid < n_sel ? r_idx[tid] : 0;
        unsigned long long bits[8], peers = n_sel == 64 ? ~0ull : (1ull << n_sel) - 1ull;
        const unsigned long long valid = peers;
#pragma unroll
        for (int b = 0; b < 8; ++b) {  // E <= 256
            bits[b] = __ballot(mine >> b & 1);
            peers &= mine >> b & 1 ? bits[b] : ~bits[b];
        }
        const int rank = __popcll(peers & ((1ull << tid) - 1ull));
        int before = 0, row = 0;  // entries of the experts 64 * q .. before this lane's
        for (int q = 0; 64 * q < E; ++q) {
            const int e = 64 * q + tid;
            unsigned long long same = valid;
#pragma unroll
            for (int b = 0; b < 8; ++b) same &= e >> b & 1 ? bits[b] : ~bits[b];
            const int c = __popcll(same);
            const int incl = wave_incl_scan(c);
            const int first = before + incl - c;
            if (e < E) offsets[e] = first;
            const int at = __shfl(first, mine & 63);
            if (mine >> 6 == q) row = at + rank;
            before += __builtin_amdgcn_readlane(incl, 63);
        }
        if (tid == 0) offsets[E] = n_sel;
        if (tid < n_sel) {
            row_of[tid] = row;
            src_row[row] = tid / k;
        }
        return;
    }
    for (int e = tid; e < E; e += n_threads) {
        int c = 0;
        for (int i = 0; i < n_sel; ++i) c += r_idx[i] == e ? 1 : 0;
        r_cnt[e] = c;
    }
    __syncthreads();
    for (int e = tid; e < E; e += n_threads) {
        int o = 0;
        for (int q = 0; q < e; ++q) o += r_cnt[q];
        r_off[e] = o;
        offsets[e] = o;
    }
    if (tid == 0) offsets[E] = n_sel;
    __syncthreads();
    for (int i = tid; i < n_sel; i += n_threads) {
        const int e = r_idx[i];
        int rank = 0;
        for (int q = 0; q < i; ++q) rank += r_idx[q] == e ? 1 : 0;
        const int r = r_off[e] + rank;
        row_of[i] = r;
        src_row[r] = i / k;
    }
}

// Smallest gates (bf16, at most GS_TOK tokens, 8 or 16 experts: batch-1 decode of the 8-expert
// models): latency is everything, the arithmetic is a few thousand multiply-adds.  One workgroup;
// thread i owns rows 8i .. 8i+7 of W (whole rows: E contiguous values) and the matching eight
// features of every token, all requested at once; partial logits are summed over the 16 lanes
// of a row by rotation, then over the rows of all wavefronts in LDS in ascending order.
constexpr int GS_TOK = 4;
constexpr int GS_THREADS = 256;
typedef __bf16 gs_bf16x8 __attribute__((ext_vector_type(8)));

// x8(t, first): features first .. first + 7 of token t, asked for once W has been requested.  chosen(idx, prob): called by every thread with the choices
// (LDS [T*k], only thread 0's own are sure to be there yet) before the tokens are grouped.
template <int EV, int NTOK, typename Features, typename Chosen>  // EV = E / 8 (1 or 2); NTOK = tokens the arithmetic is unrolled for (T <= NTOK <= GS_TOK)
__device__ inline void gate_small_rows(
    Features x8, const __bf16 *__restrict__ w, const float *__restrict__ bias, int T, int d, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags,
    int32_t *__restrict__ row_of, int32_t *__restrict__ offsets, int32_t *__restrict__ src_row, Chosen chosen) {
    constexpr int E = 8 * EV;
    constexpr int ROWS = GS_THREADS / 16;                // 16-lane rows in the workgroup
    __shared__ float part[ROWS][NTOK * E];
    __shared__ float zs[GS_TOK * 16];
    __shared__ int32_t r_idx[GS_TOK * E], r_cnt[E], r_off[E];
    __shared__ float r_prob[GS_TOK * E];
    const int tid = threadIdx.x;
    const bool mine = 8 * tid < d;                       // d <= 8 * GS_THREADS (checked by the host)
    const int r0 = mine ? 8 * tid : 0;                   // idle threads read rows 0..7 and add nothing
    const float b = (bias && tid < NTOK * E) ? bias[tid % E] : 0.f;  // needed last, requested first
    gs_bf16x8 xv[NTOK], wv[8][EV];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int v = 0; v < EV; ++v) wv[j][v] = *reinterpret_cast<const gs_bf16x8 *>(w + (size_t)(r0 + j) * E + 8 * v);
#pragma unroll
    for (int t = 0; t < NTOK; ++t) xv[t] = x8(t < T ? t : 0, r0);
    float acc[NTOK][E];
#pragma unroll
    for (int t = 0; t < NTOK; ++t)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float a = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) a = fmaf((float)xv[t][j], (float)wv[j][e >> 3][e & 7], a);
            a = mine ? a : 0.f;
            acc[t][e] = group_sum(a);
        }
    if ((tid & 15) == 0) {
#pragma unroll
        for (int t = 0; t < NTOK; ++t)
#pragma unroll
            for (int e = 0; e < E; ++e) part[tid >> 4][t * E + e] = acc[t][e];
    }
    __syncthreads();
    if (tid < NTOK * E) {
        const int e = tid % E;
        float sum = part[0][tid];
#pragma unroll
        for (int r = 1; r < ROWS; ++r) sum += part[r][tid];
        zs[(tid / E) * 16 + e] = sum + b;
    }
    __syncthreads();
    const bool route = row_of != nullptr;
    softmax_topk_n<1>(zs, 16, 0, T, E, k, idx_out, prob_out, probs_out, flags, route ? r_idx : nullptr, r_prob);
    chosen(r_idx, r_prob);
    if (!route) return;
    group_in_workgroup(r_idx, r_cnt, r_off, T * k, E, k, GS_THREADS, row_of, offsets, src_row);
}

template <int EV, int NTOK>
__device__ inline void gate_small_body(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias, int T, int d, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags,
    int32_t *__restrict__ row_of, int32_t *__restrict__ offsets, int32_t *__restrict__ src_row) {
    gate_small_rows<EV, NTOK>([&](int t, int first) { return *reinterpret_cast<const gs_bf16x8 *>(x + (size_t)t * d + first); }, w, bias, T, d, k,
                              idx_out, prob_out, probs_out, flags, row_of, offsets, src_row, [](const int32_t *, const float *) {});
}

// Runs the smallest gate for 8*EV experts and T tokens in the calling workgroup of GS_THREADS threads (uniform call).
template <int EV>
__device__ inline void gate_small_dispatch(const __bf16 *x, const __bf16 *w, const float *bias, int T, int d, int k,
                                           int32_t *idx_out, float *prob_out, float *probs_out, uint32_t *flags,
                                           int32_t *row_of, int32_t *offsets, int32_t *src_row) {
#define PG_GS(NTOK_) gate_small_body<EV, NTOK_>(x, w, bias, T, d, k, idx_out, prob_out, probs_out, flags, row_of, offsets, src_row)
    if (T == 1) PG_GS(1);
    else if (T == 2) PG_GS(2);
    else PG_GS(4);
#undef PG_GS
}

typedef __bf16 gbf16x8 __attribute__((ext_vector_type(8)));
typedef float gfloatx4 __attribute__((ext_vector_type(4)));
constexpr int GM_TOK = 16;  // tokens per workgroup
constexpr int GATE_ROUTE_MAX = 256;  // most (token, choice) pairs the gate kernel groups by itself

// ------------------------------------------------------------------------------------------
// The matrix-core gate (gate_topk_mfma_kernel, E <= 128) in two halves for a decode-sized block: its logits are sums of GATE_PLANES partial
// planes, plane v over the k-tiles v, v + GATE_PLANES, ..; the first half, carried by the launch that streams the experts'
// weights, leaves the planes in memory, the second, carried by the combine behind it, adds them in order and selects.
// Nothing crosses workgroups inside a launch, and every sum is the one kernel's, so results are its bits.
// Why: alone the gate is a chain of latencies (8 us for 16 tokens and 64 experts, 12 for 64 and 128) in front of every block;
// here the first half ends long before the weights have been streamed and the second is as long as the combine.  As one
// workgroup inside the expert launch the whole gate took longer than the experts and cost that kernel its registers.
constexpr int GATE_PLANES = 8;
constexpr int GATE_PLANE = 8 * 64 * 4;        // floats of one plane of 16 tokens: [product q][lane][r]
constexpr int GATE_CARRY_TOKENS = 128;        // most tokens of a carried gate
struct CarriedGate {
    const __bf16 *x, *w;  // x == nullptr: none
    const float *bias;
    int T, d, k, E;
    int32_t *idx;
    float *prob;
    uint32_t *flags;
    int32_t *row_of, *offsets, *src_row;  // null: the tokens are grouped elsewhere
    float *planes;                        // [token tile][GATE_PLANES][GATE_PLANE]
};
__device__ inline const CarriedGate &the_gate(const CarriedGate &gate) { return gate; }  // of a kernel whose last argument may be missing

// First half, 256 threads: workgroup u < 2 * token tiles computes four planes of tile u / 2, one per wavefront.
__device__ inline void gate_planes_body(const CarriedGate &c, int u) {
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int tile = u >> 1, plane = (u & 1) * 4 + (threadIdx.x >> 6);
    const int t0 = tile * GM_TOK, nt = min(GM_TOK, c.T - t0), KT = c.d >> 5, ncv = c.E >> 3;
    const __bf16 *xrow = c.x + (size_t)(t0 + (n < nt ? n : 0)) * c.d + 8 * g;  // rows past the batch: its first token, never used
    const gbf16x8 *wcol = reinterpret_cast<const gbf16x8 *>(c.w) + min(n, ncv - 1);  // column vectors past E: the last one, never used
    gfloatx4 acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = gfloatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int kt = plane; kt < KT; kt += GATE_PLANES) {
        const gbf16x8 a = *reinterpret_cast<const gbf16x8 *>(xrow + kt * 32);
        gbf16x8 rows[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) rows[j] = wcol[(size_t)(kt * 32 + 8 * g + j) * ncv];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            gbf16x8 cell;
#pragma unroll
            for (int j = 0; j < 8; ++j) cell[j] = rows[j][q];
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, cell, acc[q], 0, 0, 0);
        }
    }
    gfloatx4 *dst = reinterpret_cast<gfloatx4 *>(c.planes + ((size_t)tile * GATE_PLANES + plane) * GATE_PLANE) + lane;
#pragma unroll
    for (int q = 0; q < 8; ++q) dst[q * 64] = acc[q];
}

// Second half, 256 threads: the 16 tokens of a tile.
__device__ inline void gate_finish_body(const CarriedGate &c, int tile) {
    __shared__ float zs[GM_TOK * 128];
    __shared__ int32_t r_idx[GATE_ROUTE_MAX], r_cnt[PGMOE_MAX_EXPERTS], r_off[PGMOE_MAX_EXPERTS];
    const int t0 = tile * GM_TOK, nt = min(GM_TOK, c.T - t0);
    const gfloatx4 *src = reinterpret_cast<const gfloatx4 *>(c.planes + (size_t)tile * GATE_PLANES * GATE_PLANE);
    for (int o = threadIdx.x; o < GATE_PLANE / 4; o += 256) {
        const int l = o & 63, e = 8 * (l & 15) + (o >> 6);
        gfloatx4 v[GATE_PLANES];
#pragma unroll
        for (int p = 0; p < GATE_PLANES; ++p) v[p] = src[p * (GATE_PLANE / 4) + o];
        const float b = c.bias && e < c.E ? c.bias[e] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float sum = v[0][r];
#pragma unroll
            for (int p = 1; p < GATE_PLANES; ++p) sum += v[p][r];
            zs[(4 * (l >> 4) + r) * 128 + e] = sum + b;
        }
    }
    __syncthreads();
    const bool route = c.row_of != nullptr;
    softmax_topk<8>(zs, 128, t0, nt, c.E, c.k, c.idx, c.prob, nullptr, c.flags, route ? r_idx : nullptr);
    if (route) group_in_workgroup(r_idx, r_cnt, r_off, nt * c.k, c.E, c.k, 256, c.row_of, c.offsets, c.src_row);
}

// Host side: is (T tokens, this configuration) a gate the smallest-gate code serves?
inline bool gate_small_applies(const pgmoe_config &c, int T) {
    return c.dtype == PGMOE_BF16 && T >= 1 && T <= GS_TOK && (c.n_experts == 8 || c.n_experts == 16) && c.d_model <= 8 * GS_THREADS;
}

// Host side: is this a gate the matrix-core code serves?
inline bool gate_mfma_applies(const pgmoe_config &c) { return c.dtype == PGMOE_BF16 && c.n_experts % 8 == 0 && c.d_model % 32 == 0; }
// Does one workgroup hold the whole batch, so that the gate can group the tokens itself?
inline bool gate_mfma_routes(const pgmoe_config &c, int T) { return T <= GM_TOK && T * c.top_k <= GATE_ROUTE_MAX; }
// Is it one that a decode-sized block can carry in two halves?
inline bool gate_planes_apply(const pgmoe_config &c, int T) {
    return gate_mfma_applies(c) && c.n_experts <= 128 && T <= GATE_CARRY_TOKENS && !gate_small_applies(c, T);
}
// Floats of scratch the planes take for T tokens.
inline size_t gate_planes_floats(int T) { return (size_t)((T + GM_TOK - 1) / GM_TOK) * GATE_PLANES * GATE_PLANE; }

}  // namespace pgmoe
#endif  // PGMOE_GATE_SMALL_H
