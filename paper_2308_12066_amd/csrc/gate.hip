// Gate / pre-gate: logits z = x.W (+ bias), softmax over the experts, top-k on the logits
// (Sec. II-B: the gate gives every expert a probability per token and the best ones are
// activated; Sec. IV-B: the same function, placed in block N, routes block N+1).
//
// The kernels share one softmax / top-k routine (16 lanes per token, k rounds of arg-max with
// shuffles, ties to the lowest index, NaN ranks as -infinity and raises a flag):
//   gate_small_kernel      bf16, up to four tokens, 8 or 16 experts: one workgroup, all loads at once;
//   gate_topk_mfma_kernel  bf16, E a multiple of 8: logits on the matrix cores, 16 tokens per
//                          workgroup, W transposed in registers (no LDS staging on the way in);
//   gate_topk_tiles_kernel the same for more than 224 tiles of 16 tokens: pairs of tiles, W stays in registers;
//   gate_topk_vec_kernel   f32 (and bf16 when the matrix-core kernel does not apply) for
//                          power-of-two E: token rows staged in LDS as float32, threads split W
//                          by expert columns and feature rows and fold their partial sums in a
//                          fixed order (bit-reproducible);
//   gate_topk_route_kernel the same for one or two gates of a small float32 batch, whose last workgroup also groups the tokens;
//   gate_topk_kernel       the scalar version of that for any other E.
#include <cstdlib>

#include "gate_small.h"
#include "pgmoe_internal.h"

namespace pgmoe {

constexpr int GATE_ZS = 128 + 16;  // floats from one token's logits to the next: the four tokens of a wavefront on banks of their own
constexpr int GATE_TB = 8;
constexpr int GATE_DC = 1024;
constexpr int GATE_THREADS = 256;

__device__ inline float to_float(float v) { return v; }
__device__ inline float to_float(__bf16 v) { return (float)v; }

template <typename XT>
__global__ __launch_bounds__(GATE_THREADS) void gate_topk_kernel(
    const XT *__restrict__ x, const XT *__restrict__ w, const float *__restrict__ bias, int T, int d, int E, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags) {
    __shared__ float xs[GATE_TB * GATE_DC];
    __shared__ float part[GATE_THREADS * GATE_TB];  // [G][TB][E], G*E <= 256
    __shared__ float zs[GATE_TB * PGMOE_MAX_EXPERTS];

    const int tid = threadIdx.x;
    const int t0 = blockIdx.x * GATE_TB;
    const int nt = min(GATE_TB, T - t0);
    const int G = GATE_THREADS / E;
    const int g = tid / E, e = tid - g * E;
    const bool active = g < G;

    float acc[GATE_TB];
#pragma unroll
    for (int t = 0; t < GATE_TB; ++t) acc[t] = 0.f;

    for (int c0 = 0; c0 < d; c0 += GATE_DC) {
        const int dc = min(GATE_DC, d - c0);
        __syncthreads();
        for (int i = tid; i < GATE_TB * dc; i += GATE_THREADS) {
            const int t = i / dc, c = i - t * dc;
            xs[t * GATE_DC + c] = t < nt ? to_float(x[(size_t)(t0 + t) * d + c0 + c]) : 0.f;
        }
        __syncthreads();
        if (active) {
            for (int i = g; i < dc; i += G) {
                const float wv = to_float(w[(size_t)(c0 + i) * E + e]);
#pragma unroll
                for (int t = 0; t < GATE_TB; ++t) acc[t] = fmaf(xs[t * GATE_DC + i], wv, acc[t]);
            }
        }
    }
    if (active) {
#pragma unroll
        for (int t = 0; t < GATE_TB; ++t) part[(g * GATE_TB + t) * E + e] = acc[t];
    }
    __syncthreads();
    for (int o = tid; o < GATE_TB * E; o += GATE_THREADS) {
        const int t = o / E, ee = o - t * E;
        float s = 0.f;
        for (int gg = 0; gg < G; ++gg) s += part[(gg * GATE_TB + t) * E + ee];
        zs[t * PGMOE_MAX_EXPERTS + ee] = s + (bias ? bias[ee] : 0.f);
    }
    __syncthreads();

    softmax_topk(zs, PGMOE_MAX_EXPERTS, t0, nt, E, k, idx_out, prob_out, probs_out, flags);
}

// Fast path for E in {8, 16, 32, 64, 128, 256}: thread (rg, cv) owns the 8 experts 8*cv..8*cv+7
// (one 16-byte load of a W row for bf16, two for f32) and every RG-th feature row, so the 256
// threads sweep W in fully contiguous 4 KiB strides.  The RG partial sums per expert are folded
// with a fixed butterfly inside the wavefront and then across the 4 wavefronts in order.
template <typename XT, int TB>
__device__ inline void gate_vec_body(
    const XT *__restrict__ x, const XT *__restrict__ w, const float *__restrict__ bias, int T, int d, int E, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags, int32_t *idx_lds = nullptr) {
    __shared__ float xs[TB * GATE_DC];
    __shared__ float part[4 * TB * PGMOE_MAX_EXPERTS];
    __shared__ float zs[TB * PGMOE_MAX_EXPERTS];
    typedef XT vec8 __attribute__((ext_vector_type(8)));

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * TB;
    const int nt = min(TB, T - t0);
    const int CV = E >> 3;            // 8-expert column vectors per row (power of two, <= 32)
    const int RG = GATE_THREADS / CV; // row groups
    const int cv = tid & (CV - 1), rg = tid / CV;

    float acc[TB][8];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[t][j] = 0.f;

    for (int c0 = 0; c0 < d; c0 += GATE_DC) {
        const int dc = min(GATE_DC, d - c0);
        __syncthreads();
        for (int i = tid; i < TB * dc; i += GATE_THREADS) {
            const int t = i / dc, c = i - t * dc;
            xs[t * GATE_DC + c] = t < nt ? to_float(x[(size_t)(t0 + t) * d + c0 + c]) : 0.f;
        }
        __syncthreads();
        const vec8 *wv = reinterpret_cast<const vec8 *>(w + (size_t)c0 * E) + cv;
#pragma unroll 4
        for (int i = rg; i < dc; i += RG) {
            const vec8 v = wv[(size_t)i * CV];
            float xr[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) xr[t] = xs[t * GATE_DC + i];
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[t][j] = fmaf(xr[t], to_float(v[j]), acc[t][j]);
        }
    }
    // fold the row groups that live in this wavefront (lanes with equal cv are CV apart)
    for (int off = 32; off >= CV; off >>= 1) {
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[t][j] += __shfl_xor(acc[t][j], off);
    }
    if (lane < CV) {
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) part[(wave * TB + t) * PGMOE_MAX_EXPERTS + 8 * lane + j] = acc[t][j];
    }
    __syncthreads();
    for (int o = tid; o < TB * E; o += GATE_THREADS) {
        const int t = o / E, e = o - t * E;
        float sum = part[t * PGMOE_MAX_EXPERTS + e];
#pragma unroll
        for (int wv2 = 1; wv2 < 4; ++wv2) sum += part[(wv2 * TB + t) * PGMOE_MAX_EXPERTS + e];
        zs[t * PGMOE_MAX_EXPERTS + e] = sum + (bias ? bias[e] : 0.f);
    }
    __syncthreads();
    softmax_topk(zs, PGMOE_MAX_EXPERTS, t0, nt, E, k, idx_out, prob_out, probs_out, flags, idx_lds);
}

template <typename XT, int TB>
__global__ __launch_bounds__(GATE_THREADS) void gate_topk_vec_kernel(
    const XT *__restrict__ x, const XT *__restrict__ w, const float *__restrict__ bias, int T, int d, int E, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags) {
    gate_vec_body<XT, TB>(x, w, bias, T, d, E, k, idx_out, prob_out, probs_out, flags);
}

// Gates of small batches that also group the tokens (what route_kernel does for larger ones), one or two of them on the same tokens (a
// step's first two: block 0's own and the pre-gate of block 1).  A workgroup per token as above; whichever workgroup of a gate
// ends last groups: the choices are written through to memory and counted, so there is no fence and nobody waits.  Bound by latency and
// launches: a step of two float32 blocks of 64 x 256 (8 experts, 32 tokens) was ten launches and 38.8 us with steps of several stacks in flight, and is five
// and 21.5 us with this kernel and the combine in the second expert kernel; one block of 768 x 3072, 100 tokens, 39.6 -> 37.5 us.
struct RoutedGate {
    const void *w;
    const float *bias;
    int32_t *idx;
    float *prob;
    int32_t *row_of, *offsets, *src_row;
    uint32_t *counter;  // of batches of this size; zero, left zero
};
constexpr int GATE_ROUTE_ENTRIES = 512;  // most (token, choice) pairs

// The grouping of n <= GATE_ROUTE_ENTRIES entries by 256 threads: entry tid + 256 * r is thread tid's r-th; entries of a wavefront are in order
// inside a round and rounds follow each other, so a stable rank is: earlier entries of the round's earlier wavefronts, of
// earlier rounds, and of lower lanes.
__device__ inline void group_entries(const int32_t *__restrict__ idx, int n, int E, int k, int32_t *__restrict__ row_of,
                                     int32_t *__restrict__ offsets, int32_t *__restrict__ src_row) {
    constexpr int ROUNDS = GATE_ROUTE_ENTRIES / GATE_THREADS, RUNS = ROUNDS * 4;  // a run: 64 neighbouring entries
    __shared__ int count[RUNS][PGMOE_MAX_EXPERTS];
    __shared__ int first[PGMOE_MAX_EXPERTS + 1];
    __shared__ int wave_total[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int e[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int i = tid + r * GATE_THREADS;
        e[r] = i < n ? __hip_atomic_load(idx + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
#pragma unroll
    for (int q = 0; q < RUNS; ++q) count[q][tid] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
        if (tid + r * GATE_THREADS < n) atomicAdd(&count[r * 4 + wave][e[r]], 1);
    __syncthreads();
    int total = 0;  // thread tid: expert tid
#pragma unroll
    for (int q = 0; q < RUNS; ++q) {
        const int c = count[q][tid];
        count[q][tid] = total;
        total += c;
    }
    int incl = total;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wave_total[wave] = incl;
    __syncthreads();
    int before = incl - total;
    for (int q = 0; q < wave; ++q) before += wave_total[q];
    first[tid] = before;
    if (tid < E) offsets[tid] = before;
    if (tid == 0) offsets[E] = n;
    __syncthreads();
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int i = tid + r * GATE_THREADS;
        const bool valid = i < n;
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (e[r] >> b) & 1;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        if (!valid) continue;
        const int row = first[e[r]] + count[r * 4 + wave][e[r]] + __popcll(peers & ((1ull << lane) - 1ull));
        row_of[i] = row;
        src_row[row] = i / k;
    }
}

template <typename XT>
__global__ __launch_bounds__(GATE_THREADS) void gate_topk_route_kernel(const XT *__restrict__ x, int T, int d, int E, int k, uint32_t *flags,
                                                                       RoutedGate g0, RoutedGate g1) {
    __shared__ int32_t chosen[PGMOE_MAX_EXPERTS];
    __shared__ int last;
    const RoutedGate g = blockIdx.y ? g1 : g0;  // uniform
    gate_vec_body<XT, 1>(x, (const XT *)g.w, g.bias, T, d, E, k, g.idx, g.prob, nullptr, flags, chosen);
    __syncthreads();
    const int tid = threadIdx.x;
    for (int j = tid; j < k; j += GATE_THREADS)  // again, past this XCD's L2: the workgroup that groups may run on another
        __hip_atomic_store(g.idx + (size_t)blockIdx.x * k + j, chosen[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // goes round after T workgroups: zero again behind any number of gates, in whatever order their workgroups came, and a
    // gate of one workgroup is not told from another by it
    if (tid == 0) last = atomicInc(g.counter, T - 1) == (uint32_t)T - 1;
    __syncthreads();
    if (!last) return;  // uniform over the workgroup
    group_entries(g.idx, T * k, E, k, g.row_of, g.offsets, g.src_row);
}

// The smallest gate as a kernel of its own (its body lives in gate_small.h).
__global__ __launch_bounds__(GS_THREADS) void gate_small_kernel(
    int E, const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias, int T, int d, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags,
    int32_t *__restrict__ row_of, int32_t *__restrict__ offsets, int32_t *__restrict__ src_row) {
    if (E == 8) gate_small_dispatch<1>(x, w, bias, T, d, k, idx_out, prob_out, probs_out, flags, row_of, offsets, src_row);
    else gate_small_dispatch<2>(x, w, bias, T, d, k, idx_out, prob_out, probs_out, flags, row_of, offsets, src_row);
}

// Matrix-core path (bf16, E a multiple of 8, d_model a multiple of 32): the gate is a skinny
// GEMM [T,d] x [d,E].  A workgroup takes 16 tokens (one matrix-core tile); its NW wavefronts
// (eight for E <= 128, four above) split the d_model reduction (k-tile kt goes to wavefront
// kt % NW) and their partial logits are added in LDS in wavefront order.  Nothing is staged through LDS on the way in:
//   * the token operand (16 tokens x 32 k) is one 16-byte load per lane straight from x;
//   * W is row-major [d,E], an expert's weights are strided, but lane (n, g) can load rows
//     32*kt + 8*g .. +7 of the eight experts 8*n .. 8*n+7 with eight contiguous 16-byte loads and
//     transpose the 8x8 block in registers.  Product q (q = 0..7) then takes from every lane the
//     eight k-values of expert 8*n + q: that is a valid operand for the 16 experts
//     {q, 8+q, 16+q, ...}, i.e. output column n of product q is expert 8*n + q.  Eight products
//     cover 128 experts per k-tile; E = 256 takes a second pass.
// The expert of place o = [p][q][lane] of a plane of partial logits.
__device__ inline int gate_expert_of(int o) { return 8 * ((o & 15) + 16 * (o >> 9)) + (o >> 6 & 7); }

// NP: passes of 128 experts (1: E <= 128, 2: E <= 256); NW: wavefronts that split d_model; KW: k-tiles of a wavefront (d_model = 32 * NW * KW),
// 0: any number of them
template <int NP, int NW, int KW>
__global__ __launch_bounds__(NW * 64) void gate_topk_mfma_kernel(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias, int T, int d, int E, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags,
    int32_t *__restrict__ row_of, int32_t *__restrict__ offsets, int32_t *__restrict__ src_row) {  // routing outputs: see below
    extern __shared__ __attribute__((aligned(16))) char gsm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int t0 = blockIdx.x * GM_TOK;
    const int nt = min(GM_TOK, T - t0);
    const int KT = d >> 5;
    const int ncv = E >> 3;           // 8-expert column vectors per W row
    const int ecols = NP * 128;       // logit columns kept per token in LDS
    constexpr int NT = NW * 64;                              // threads
    float *part = reinterpret_cast<float *>(gsm);            // [NW][GM_TOK][ecols]
    float *zs = part + NW * GM_TOK * ecols;                  // [GM_TOK][ecols]

    gfloatx4 acc[NP][8];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[p][q] = gfloatx4{0.f, 0.f, 0.f, 0.f};

    // the experts whose planes this thread adds: their bias is needed last and requested first
    float b_of[NP * 8 / NW];
#pragma unroll
    for (int i = 0; i < NP * 8 / NW; ++i) {
        const int e = gate_expert_of(tid + NT * i);
        b_of[i] = bias && e < E ? bias[e] : 0.f;
    }
    const __bf16 *xrow = x + (size_t)(t0 + (n < nt ? n : 0)) * d + 8 * g;  // rows past the batch read its first token; their logits are never used
    // Register prefetch ring, PF k-tiles deep: the operands of a wavefront's k-tile i + PF are requested when
    // k-tile i is consumed, so it pays the memory latency once, not once per k-tile.
    // Every request is an unconditional load from a clamped (always valid) address, so nothing
    // makes the compiler wait for one load before it issues the next: column vectors past E read the last real one (their logits are
    // never used).  With a number of k-tiles known here none is requested that does not exist; else a stage past the last
    // k-tile reads the last one again and has its token operand zeroed when it is used (it adds nothing), up to twice the loads:
    // 4096 tokens of 1024 x 128 read 594 KB per workgroup that way, 264 KB now, 9.5 -> 7.5 us.
    constexpr int PF = KW > 0 && NP == 1 ? (KW < 4 ? KW : 4) : (NP == 1 ? 3 : 2);
    const gbf16x8 zero8 = gbf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    gbf16x8 a_buf[PF], rows_buf[PF][NP][8];
    auto request = [&](int kt, gbf16x8 &a, gbf16x8 (&rows)[NP][8]) {
        a = *reinterpret_cast<const gbf16x8 *>(xrow + kt * 32);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int cv = min(n + 16 * p, ncv - 1);
            const gbf16x8 *src = reinterpret_cast<const gbf16x8 *>(w + (size_t)(kt * 32 + 8 * g) * E) + cv;
#pragma unroll
            for (int j = 0; j < 8; ++j) rows[p][j] = src[(size_t)j * ncv];
        }
    };
    auto transpose = [&](const gbf16x8 (&rows)[NP][8], gbf16x8 (&cells)[NP][8]) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int j = 0; j < 8; ++j) cells[p][q][j] = rows[p][j][q];
    };
    auto multiply = [&](const gbf16x8 a, const gbf16x8 (&cells)[NP][8]) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc[p][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, cells[p][q], acc[p][q], 0, 0, 0);
    };
    // the instruction scheduler must not move the loads down to their uses to save registers
    // (that would pay the memory latency once per stage): nothing crosses a scheduling barrier
    if constexpr (KW > 0) {
#pragma unroll
        for (int i = 0; i < PF; ++i) request(wave + NW * i, a_buf[i], rows_buf[i]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            const gbf16x8 a = a_buf[i % PF];
            gbf16x8 cells[NP][8];
            transpose(rows_buf[i % PF], cells);
            if (i + PF < KW) {
                request(wave + NW * (i + PF), a_buf[i % PF], rows_buf[i % PF]);
                __builtin_amdgcn_sched_barrier(0);
            }
            multiply(a, cells);
        }
    } else {
#pragma unroll
        for (int st = 0; st < PF; ++st) request(min(wave + NW * st, KT - 1), a_buf[st], rows_buf[st]);
        __builtin_amdgcn_sched_barrier(0);
        for (int kt0 = wave; kt0 < KT; kt0 += NW * PF) {
#pragma unroll
            for (int st = 0; st < PF; ++st) {
                const gbf16x8 a = kt0 + NW * st < KT ? a_buf[st] : zero8;
                gbf16x8 cells[NP][8];
                transpose(rows_buf[st], cells);
                request(min(kt0 + NW * (st + PF), KT - 1), a_buf[st], rows_buf[st]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a, cells);
            }
        }
    }
    // lane holds tokens 4*g + r (r = 0..3), column n of product q = expert 8*(n + 16*p) + q.  The
    // partial logits are parked as [wave][p][q][lane][r] (one 16-byte LDS write per accumulator
    // tile) and added over the wavefronts in wave order.
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q)
            reinterpret_cast<gfloatx4 *>(part)[(((size_t)wave * NP + p) * 8 + q) * 64 + lane] = acc[p][q];
    __syncthreads();
    constexpr int PLACES = NP * 8 * 64;  // of four floats, per wavefront
#pragma unroll
    for (int i = 0; i < PLACES / NT; ++i) {
        const int o = tid + NT * i;
        const gfloatx4 *src = reinterpret_cast<const gfloatx4 *>(part) + o;
        gfloatx4 sum = src[0];
#pragma unroll
        for (int wv = 1; wv < NW; ++wv) sum += src[wv * PLACES];
#pragma unroll
        for (int r = 0; r < 4; ++r) zs[(4 * (lane >> 4) + r) * ecols + gate_expert_of(o)] = sum[r] + b_of[i];
    }
    __syncthreads();
    // Decode-sized batch (the whole batch in this one workgroup, at most GATE_ROUTE_MAX
    // selections): group the tokens by expert right here instead of in a kernel of its own.
    // Same integers as route_kernel: counts, exclusive prefix sum, stable rank, inverse map.
    const bool route = row_of != nullptr;   // uniform; the host passes it only for a single-workgroup launch
    int32_t *r_idx = reinterpret_cast<int32_t *>(part);      // [n]   (the partial planes are dead by now)
    int32_t *r_cnt = r_idx + GATE_ROUTE_MAX;                 // [E]
    int32_t *r_off = r_cnt + PGMOE_MAX_EXPERTS;              // [E]
    softmax_topk<8 * NP>(zs, ecols, t0, nt, E, k, idx_out, prob_out, probs_out, flags, route ? r_idx : nullptr);
    if (!route) return;
    group_in_workgroup(r_idx, r_cnt, r_off, nt * k, E, k, NT, row_of, offsets, src_row);
}

// The same for batches of many tiles (E <= 128, d_model = 256*KW, KW <= 4: the share of W is 32*KW registers a lane,
// as many as the accumulators and the next tokens leave): a workgroup keeps its share of W in registers,
// transposed once, and walks pairs of token tiles.  One tile alone is bound by its 264 KB of W (4600 clocks at the 64 bytes a clock of a CU's
// path to L2) and by a softmax of half the wavefronts, each alone on its SIMD; a pair shares the first and fills the
// second, and leaves half the CUs to others, but takes longer by itself.  4096 tokens of 1024 x 128, launches of three streams: 6.3 us with a tile per workgroup, 4.7
// so (9.6 before either); by itself 7.2 and 9.3.  16384 in a step 22.  Sums and their order are the kernel's above: same bits.
template <int KW>
__global__ __launch_bounds__(512) void gate_topk_tiles_kernel(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias, int T, int E, int k,
    int32_t *__restrict__ idx_out, float *__restrict__ prob_out, float *__restrict__ probs_out, uint32_t *flags) {
    constexpr int NW = 8, d = 256 * KW, PLACES = 8 * 64, PAIR = 2 * GM_TOK;
    extern __shared__ __attribute__((aligned(16))) char gsm[];
    gfloatx4 *part = reinterpret_cast<gfloatx4 *>(gsm);             // [NW][PLACES]
    float *zs = reinterpret_cast<float *>(part + NW * PLACES);      // [PAIR][GATE_ZS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int ncv = E >> 3;
    gbf16x8 cells[KW][8], rows[KW][8];
    const gbf16x8 *wcol = reinterpret_cast<const gbf16x8 *>(w) + min(n, ncv - 1);  // column vectors past E: the last one, never used
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) rows[i][j] = wcol[(size_t)((wave + NW * i) * 32 + 8 * g + j) * ncv];
    gbf16x8 a[2][KW];
    auto request = [&](int t0) {  // this wavefront's k-tiles of the pair's tokens; past the batch: its last token, never used
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const __bf16 *xrow = x + (size_t)min(t0 + u * GM_TOK + n, T - 1) * d + 8 * g;
#pragma unroll
            for (int i = 0; i < KW; ++i) a[u][i] = *reinterpret_cast<const gbf16x8 *>(xrow + (wave + NW * i) * 32);
        }
    };
    request(blockIdx.x * PAIR);
    const int e_of = gate_expert_of(tid);  // the expert this thread adds the planes of
    const float b = bias && e_of < E ? bias[e_of] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int j = 0; j < 8; ++j) cells[i][q][j] = rows[i][j][q];
    for (int t0 = blockIdx.x * PAIR; t0 < T; t0 += gridDim.x * PAIR) {
        gfloatx4 acc[2][8];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[u][q] = gfloatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < KW; ++i)
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    acc[u][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][i], cells[i][q], acc[u][q], 0, 0, 0);
        if (t0 + (int)gridDim.x * PAIR < T) request(t0 + gridDim.x * PAIR);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int q = 0; q < 8; ++q) part[wave * PLACES + q * 64 + lane] = acc[u][q];
            __syncthreads();
            // thread (q = wave, lane) adds the planes' four floats of that place, in plane order
            gfloatx4 sum = part[tid];
#pragma unroll
            for (int v = 1; v < NW; ++v) sum += part[v * PLACES + tid];
#pragma unroll
            for (int r = 0; r < 4; ++r) zs[(u * GM_TOK + 4 * g + r) * GATE_ZS + e_of] = sum[r] + b;
            __syncthreads();
        }
        // zs is written again only behind the first barrier of the next pair
        softmax_topk<8>(zs, GATE_ZS, t0, min(PAIR, T - t0), E, k, idx_out, prob_out, probs_out, flags);
    }
}

template <typename XT>
static void launch_gate_t(const pgmoe_config &c, const XT *x, const XT *w, const float *bias, int T, int32_t *idx,
                          float *prob, float *probs, uint32_t *flags, hipStream_t s) {
    const int E = c.n_experts;
    const bool vec = E >= 8 && E <= PGMOE_MAX_EXPERTS && (E & (E - 1)) == 0;
    if (!vec) {
        hipLaunchKernelGGL(gate_topk_kernel<XT>, dim3((T + GATE_TB - 1) / GATE_TB), dim3(GATE_THREADS), 0, s, x, w, bias, T,
                           c.d_model, E, c.top_k, idx, prob, probs, flags);
        return;
    }
    // tokens per workgroup: one while every workgroup has a CU to itself (each reads W whatever it serves), then more; the two-token
    // kernel falls behind with many experts.  float32, one / two / four: 100 tokens of 1024 x 128 9.9 / 16.4 / -, 400 tokens of 768 x 8
    // - / 7.7 / 14.6, of 2048 x 256 - / 80 / 55 us
#define PG_GATE(TB_)                                                                                                  \
    hipLaunchKernelGGL((gate_topk_vec_kernel<XT, TB_>), dim3((T + TB_ - 1) / TB_), dim3(GATE_THREADS), 0, s, x, w, bias, T, \
                       c.d_model, E, c.top_k, idx, prob, probs, flags)
    if (T <= 256) PG_GATE(1);
    else if (T <= 512 && E <= 64) PG_GATE(2);
    else if (T <= 1024) PG_GATE(4);
    else PG_GATE(8);
#undef PG_GATE
}

static int launch_gate_mfma(pgmoe_ctx *ctx, const __bf16 *x, const __bf16 *w, const float *bias, int T, int32_t *idx,
                            float *prob, float *probs, hipStream_t s, int32_t *row_of, int32_t *offsets, int32_t *src_row,
                            bool *routed) {
    const pgmoe_config &c = ctx->cfg;
    const int np = c.n_experts <= 128 ? 1 : 2;
    const dim3 grid((T + GM_TOK - 1) / GM_TOK);
    // grouping inside the gate kernel: one workgroup holds the whole batch and the selections fit
    const bool route = row_of && offsets && src_row && gate_mfma_routes(c, T);
    if (!route) row_of = offsets = src_row = nullptr;
    if (routed) *routed = route;
    if (gate_small_applies(c, T)) {
        hipLaunchKernelGGL(gate_small_kernel, dim3(1), dim3(GS_THREADS), 0, s, c.n_experts, x, w, bias, T, c.d_model, c.top_k, idx,
                           prob, probs, ctx->dev_flags, row_of, offsets, src_row);
        PG_HIP(ctx, hipGetLastError());
        return PGMOE_OK;
    }
    // More tiles than seven CUs of eight: workgroups of pairs of tiles, as few as keep the rounds over the CUs equal. Below, a tile for each CU ends sooner and
    // launches of several streams share the chip either way; from there on they queue for it (tiles / pairs, 1024 x 128, by itself | waited for | three
    // streams: 2049 tokens 6.5 / 9.0 | 19.5 / 21.6 | 4.7 / 4.3 us, 3584 6.8 / 9.2 | 19.8 / 22.2 | 5.3 / 4.5, 3840 6.9 / 9.3 | 19.9 / 22.3 | 5.9 / 4.4; 768 x 64: 2049
    // 5.1 / 6.7 | 17.9 / 19.6 | 4.5 / 4.4, 4096 5.1 / 6.7 | 18.1 / 19.6 | 4.6 / 4.3). Up to 4096 tokens that favours several streams over a call by itself.
    if (np == 1 && grid.x > 224 && !route && c.d_model % 256 == 0 && c.d_model <= 1024) {
        const int pairs = ((int)grid.x + 1) / 2, per = (pairs + 255) / 256;
        const dim3 wgs((pairs + per - 1) / per);
#define PG_GATE_TILES(KW_)                                                                                              \
    do {                                                                                                                \
        auto kern = gate_topk_tiles_kernel<KW_>;                                                                        \
        constexpr size_t lds = (8 * 2048 + 2 * GM_TOK * GATE_ZS) * sizeof(float);                                       \
        if (int rc_ = allow_dynamic_lds(ctx, reinterpret_cast<const void *>(kern), lds)) return rc_;                    \
        hipLaunchKernelGGL(kern, wgs, dim3(512), lds, s, x, w, bias, T, c.n_experts, c.top_k, idx, prob, probs, ctx->dev_flags); \
    } while (0)
        if (c.d_model == 256) PG_GATE_TILES(1);
        else if (c.d_model == 512) PG_GATE_TILES(2);
        else if (c.d_model == 768) PG_GATE_TILES(3);
        else PG_GATE_TILES(4);
#undef PG_GATE_TILES
        PG_HIP(ctx, hipGetLastError());
        return PGMOE_OK;
    }
    // With up to 128 experts eight wavefronts split d_model, and up to d_model 1024 each has all of its four k-tiles at most in flight at once, i.e. the kernel
    // pays the memory latency once; with more experts four wavefronts have two k-tiles each in flight.
#define PG_GATE_MFMA(NP_, NW_, KW_)                                                                                     \
    do {                                                                                                                \
        auto kern = gate_topk_mfma_kernel<NP_, NW_, KW_>;                                                               \
        const size_t lds = (size_t)(NW_ + 1) * GM_TOK * NP_ * 128 * sizeof(float); /* NW partial planes + the logits */ \
        if (int rc_ = allow_dynamic_lds(ctx, reinterpret_cast<const void *>(kern), lds)) return rc_;                    \
        hipLaunchKernelGGL(kern, grid, dim3(NW_ * 64), lds, s, x, w, bias, T, c.d_model, c.n_experts, c.top_k, idx, prob, probs, \
                           ctx->dev_flags, row_of, offsets, src_row);                                                   \
    } while (0)
    if (np == 1) {
        if (c.d_model == 256) PG_GATE_MFMA(1, 8, 1);
        else if (c.d_model == 512) PG_GATE_MFMA(1, 8, 2);
        else if (c.d_model == 768) PG_GATE_MFMA(1, 8, 3);
        else if (c.d_model == 1024) PG_GATE_MFMA(1, 8, 4);
        else if (c.d_model == 2048) PG_GATE_MFMA(1, 8, 8);
        else PG_GATE_MFMA(1, 8, 0);
    } else {
        if (c.d_model == 512) PG_GATE_MFMA(2, 4, 4);
        else if (c.d_model == 768) PG_GATE_MFMA(2, 4, 6);
        else if (c.d_model == 1024) PG_GATE_MFMA(2, 4, 8);
        else if (c.d_model == 2048) PG_GATE_MFMA(2, 4, 16);
        else PG_GATE_MFMA(2, 4, 0);
    }
#undef PG_GATE_MFMA
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

// Gates the vector kernel serves with a workgroup per token and whose choices its last workgroup can group.
bool gate_groups_tokens(const pgmoe_config &c, int T) {
    const int E = c.n_experts;
    return ffn_f32_reads_rows_in_place(c) && E >= 8 && E <= PGMOE_MAX_EXPERTS && (E & (E - 1)) == 0 && T <= GATE_GROUP_TOKENS && T * c.top_k <= GATE_ROUTE_ENTRIES;
}

int launch_gates_grouped(pgmoe_ctx *ctx, const void *x, int T, const FusedGate *gates, int n, const int *blocks, hipStream_t s) {
    const pgmoe_config &c = ctx->cfg;
    RoutedGate g[2] = {};
    for (int i = 0; i < n; ++i)
        g[i] = RoutedGate{gates[i].w, gates[i].bias, gates[i].idx, gates[i].prob, gates[i].row_of, gates[i].offsets, gates[i].src_row,
                          ctx->gate_counter + (size_t)blocks[i] * gate_counters(c) + T - 1};
    hipLaunchKernelGGL(gate_topk_route_kernel<float>, dim3(T, n), dim3(GATE_THREADS), 0, s, (const float *)x, T, c.d_model, c.n_experts,
                       c.top_k, ctx->dev_flags, g[0], g[1]);
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

int launch_gate(pgmoe_ctx *ctx, const void *x, const void *w, const float *bias, int T, int32_t *idx,
                float *prob, float *probs, hipStream_t s, int32_t *row_of, int32_t *offsets, int32_t *src_row, bool *routed) {
    const pgmoe_config &c = ctx->cfg;
    if (routed) *routed = false;
    if (gate_mfma_applies(c))
        return launch_gate_mfma(ctx, (const __bf16 *)x, (const __bf16 *)w, bias, T, idx, prob, probs, s,
                                row_of, offsets, src_row, routed);
    if (c.dtype == PGMOE_F32)
        launch_gate_t<float>(c, (const float *)x, (const float *)w, bias, T, idx, prob, probs, ctx->dev_flags, s);
    else
        launch_gate_t<__bf16>(c, (const __bf16 *)x, (const __bf16 *)w, bias, T, idx, prob, probs, ctx->dev_flags, s);
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

}  // namespace pgmoe
