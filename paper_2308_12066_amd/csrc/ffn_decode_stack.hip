// A whole pre-gated stack step (Sec. IV-B wiring) of one token with one expert per block in two launches: smallest gates, decode-sized experts, every
// expert resident (batch-1 decode of the 8- and 16-expert models).
//
// Block by block the step is a chain of two launches each, a dozen launches of a few microseconds that a host needs 45 to 57 us to
// enqueue.  Here the first launch is block 0's own gate, beside workgroups that clear the words the second one hands over with, and in the second
// the workgroups of all blocks are one grid and hand over inside it:
//   gate of block i+1 (one workgroup)   needs x_i;                                     leaves the expert of block i+1 and its probability
//   experts of block i (one workgroup per 32-column sub-slab of d_ff)   need the expert to request its weights, then x_i;   leave partial sums
//   combine of block i (one per 64 columns)                       needs the partial sums, probability and x_i;   leaves x_{i+1}
// The arithmetic and its order are those of the separate launches: same bits.
//
// Hand-over: what crosses workgroups is stored past the XCD's L2 and loaded past it, so there are no fences.  Routing and x travel as 64-bit words of
// 32 bits of payload and a tag (number of the step and of the block) that whoever needs them polls until the tag is right: one store and one load.
// The partial sums, 295 KB a block, are counted instead (polling them as tagged words held up what it waited for: 52 us a step).
//
// Everything a step shares lies in the workspace its caller brought, and the first launch clears it whatever the workspace held: steps with
// buffers of their own have nothing in common, also those of one context on several streams or in several graphs.
//
// No workgroup waits for one that may not have started: work is drawn as tickets in the order above, and whoever holds a ticket waits for
// lower ones only, so the lowest one still at work never waits, whatever else occupies the GPU.  Waits are bounded all the same, by the looks
// taken and not by the clock, which goes on while the queue is not on the GPU; after that the context's flags say that results
// are wrong, and whoever combines then leaves NaN.
//
// 8 experts of 768 x 3072, six blocks: 32 us a step with steps of several stacks in flight, 45 one after the other on a stream, 56 waited for;
// 55, 58 and 73 as launches.  Clearing costs nothing beside block 0's gate: with state that was left ready by the step
// before, all in one launch, it was 32 as well.  Bound by hand-overs: a block is two of them, about a microsecond each for the store and the load, around two
// memory latencies of its own (weights are there when x is).  With more than one (token, expert) pair it does not pay: a
// first version that took up to fifteen pairs took 52, 93 and 92 us for two tokens, four tokens and two tokens of two experts, the
// launches 56, 66 and 70; two tokens alone were little faster.
#include "ffn_common.h"
#include "ffn_decode.h"
#include "gate_small.h"

namespace pgmoe {

constexpr int STACK_BLOCKS = 16;  // most blocks of a launch (their gates are arguments)
constexpr int STACK_AHEAD = 2;    // blocks whose workgroups are there at once: those of the next one have their weights on the way while a
                                  // block runs; more would only wait, in places that steps of other stacks could use
constexpr int PAST_L2 = 16;       // cache policy of loads and stores: sc1
constexpr int SPREAD = 8;         // counters of a block's finished expert workgroups, each of the form workgroup number % SPREAD
constexpr int STACK_PATIENCE = 1 << 20;  // most looks of a wait: half a second and more, each is a load past L2

typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));

// In the workspace: ticket, tagged words of the routing (two a block) and of x (even and odd blocks), counters [L][SPREAD] (a memory channel
// apart), all of them zero when the step begins; then the partial sums of a block.
struct StackScratch {
    static constexpr int APART = 256, ROUTING = APART, X = ROUTING + STACK_BLOCKS * 2 * 8;
    __host__ __device__ static constexpr int counters(int d) { return X + 2 * (d / 2 * 8); }
    __host__ __device__ static constexpr int cleared(int d, int L) { return counters(d) + L * SPREAD * APART; }  // the partial sums begin there
    static size_t bytes(int d, int f, int L) { return cleared(d, L) + (size_t)(f / 32) * d * 4; }
};

struct DecodeStack {
    const __bf16 *x;  // x_states [L+1][d]
    __bf16 *y;        // y_blocks [L][d] | nullptr
    int32_t *idx;     // [L]
    float *prob;
    int32_t *row_of, *offsets, *src_row;  // [L], [L][E+1], [L][src_stride]
    const char *w_base;
    size_t w_stride, block_stride;
    char *scratch;  // the step's workspace
    uint32_t *flags;
    int f, L, src_stride;
    const __bf16 *gate_w[STACK_BLOCKS];
    const float *gate_b[STACK_BLOCKS];
};

__device__ inline uint32x4 load_past_l2(__amdgpu_buffer_rsrc_t buf, int offset) { return __builtin_amdgcn_raw_buffer_load_b128(buf, offset, 0, PAST_L2); }
__device__ inline __amdgpu_buffer_rsrc_t buffer_at(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00027000);
}
// Sixteen bytes: two tagged words.
__device__ inline void put_pair(__amdgpu_buffer_rsrc_t buf, int offset, uint32_t a, uint32_t b, uint32_t tag) {
    __builtin_amdgcn_raw_buffer_store_b128(uint32x4{a, tag, b, tag}, buf, offset, 0, PAST_L2);
}
// A wait of this wavefront has run out: known to whoever sees what this workgroup hands over next.
__device__ inline void wait_failed(uint32_t *flags) {
    if ((threadIdx.x & 63) == 0) atomicOr(flags, kFlagStalled);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// N pairs of tagged words per lane, at offset(n), polled until all of a wavefront's have the tag (lanes that are not `live` take what they get).
template <int N, typename Offset>
__device__ inline void take_pairs(__amdgpu_buffer_rsrc_t buf, Offset offset, uint32_t tag, bool live, uint32_t (&a)[N], uint32_t (&b)[N], uint32_t *flags) {
    for (int looks = 1;; ++looks) {
        uint32x4 v[N];
        bool there = true;
#pragma unroll
        for (int n = 0; n < N; ++n) v[n] = load_past_l2(buf, offset(n));
#pragma unroll
        for (int n = 0; n < N; ++n) {
            there = there && v[n].y == tag && v[n].w == tag;
            a[n] = v[n].x;
            b[n] = v[n].z;
        }
        if (__all(there || !live)) return;
        if (looks == STACK_PATIENCE) return wait_failed(flags);
        __builtin_amdgcn_s_sleep(1);
    }
}

// Block 0's gate and, in the other workgroups, the step's shared words set to zero.
template <int EV>
__global__ __launch_bounds__(GS_THREADS) void ffn_decode_stack_begin_kernel(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ w, const float *__restrict__ bias, int d, int32_t *__restrict__ idx, float *__restrict__ prob,
    uint32_t *flags, int32_t *__restrict__ row_of, int32_t *__restrict__ offsets, int32_t *__restrict__ src_row, uint4 *__restrict__ words, int n_words) {
    if (blockIdx.x == 0) {
        gate_small_body<EV, 1>(x, w, bias, 1, d, 1, idx, prob, nullptr, flags, row_of, offsets, src_row);
        return;
    }
    const int i = (blockIdx.x - 1) * GS_THREADS + threadIdx.x;
    if (i < n_words) words[i] = make_uint4(0, 0, 0, 0);
}

template <int KT, int EV>
__global__ __launch_bounds__(256, 2) void ffn_decode_stack_kernel(DecodeStack s) {
    constexpr int d = KT * 32, E = 8 * EV, PL = 16, COLS = 256 / PL;  // p-lanes and float4 columns of a combine workgroup, as combine_partials_kernel<16>
    constexpr int n_combine = d / 4 / COLS;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ uint32_t drawn;
    __shared__ floatx4 sub[PL][COLS + 1];
    const int tid = threadIdx.x;
    const int P = s.f / 32, per_block = 1 + P + n_combine, tickets = s.L * per_block - 1;  // the last block has no gate
    uint32_t *ticket = reinterpret_cast<uint32_t *>(s.scratch);
    const __amdgpu_buffer_rsrc_t routing = buffer_at(s.scratch + StackScratch::ROUTING);
    const __amdgpu_buffer_rsrc_t partial = buffer_at(s.scratch + StackScratch::cleared(d, s.L));
    auto x_words = [&](int i) { return buffer_at(s.scratch + StackScratch::X + (i & 1) * (d / 2 * 8)); };
    auto done = [&](int i, int c) { return reinterpret_cast<uint32_t *>(s.scratch + StackScratch::counters(d)) + (i * SPREAD + c) * (StackScratch::APART / 4); };
#pragma unroll 1
    while (true) {
        __syncthreads();
        if (tid == 0) drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        int at = __builtin_amdgcn_readfirstlane(drawn);
        if (at >= tickets) break;
        const int i = at / per_block;  // block
        at -= i * per_block;
        if (i == s.L - 1) at += 1;
        int what = 0;  // 0: gate of block i + 1, 1: experts, 2: combine
        if (at > 0) {
            at -= 1;
            what = at < P ? 1 : 2;
            if (what == 2) at -= P;
        }
        // eight features of x_i, the first of them `first`; x_i and the routing of block i, i > 0, have the tag i
        auto features = [&](int first, bool live) {
            if (i == 0) return *reinterpret_cast<const uint4 *>(s.x + first);
            uint32_t a[2], b[2];
            take_pairs<2>(x_words(i), [&](int n) { return first / 2 * 8 + n * 16; }, i, live, a, b, s.flags);
            return make_uint4(a[0], b[0], a[1], b[1]);
        };
        if (what == 0) {
            const int b = i + 1;
            gate_small_rows<EV, 1>([&](int, int first) { return __builtin_bit_cast(gs_bf16x8, features(first, 8 * tid < d)); }, s.gate_w[b], s.gate_b[b], 1,
                                   d, 1, s.idx + b, s.prob + b, nullptr, s.flags, s.row_of + b, s.offsets + b * (E + 1),
                                   s.src_row + (size_t)b * s.src_stride, [&](const int32_t *idx, const float *prob) {
                                       if (tid == 0) put_pair(routing, b * 16, (uint32_t)idx[0], __float_as_uint(prob[0]), b);
                                   });
            continue;
        }
        uint32_t expert[1], prob[1];
        if (i == 0) {
            expert[0] = s.idx[0];
            prob[0] = __float_as_uint(s.prob[0]);
        } else {
            take_pairs<1>(routing, [&](int) { return i * 16; }, i, true, expert, prob, s.flags);
        }
        const int e = min((uint32_t)(E - 1), (uint32_t)__builtin_amdgcn_readfirstlane(expert[0]));
        if (what == 1) {
            decode_sub_slab<KT>(
                smem, s.w_base + (size_t)i * s.block_stride + (size_t)e * s.w_stride, s.f, at,
                [&](bf16x8 *xs) {
                    uint4 *dst = reinterpret_cast<uint4 *>(xs);
                    const bool row0 = tid < d / 8;
                    uint4 v = make_uint4(0, 0, 0, 0);
                    if (tid < (d / 8 + 63) / 64 * 64) v = features(row0 ? tid * 8 : 0, row0);  // uniform over the wavefront
#pragma unroll
                    for (int j = 0; j < KT / 4; ++j) {
                        const int c = tid + 256 * j, m = c / (d / 8), k8 = c - m * (d / 8);
                        dst[((k8 >> 2) << 6) + m + 16 * (k8 & 3)] = j == 0 && row0 ? v : make_uint4(0, 0, 0, 0);
                    }
                },
                [&](int column, int row, const floatx4 &y) {
                    if (row == 0) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint32x4, y), partial, (at * d + column) * 4, 0, PAST_L2);
                });
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sums are in memory
            __syncthreads();
            if (tid == 0) __hip_atomic_fetch_add(done(i, at % SPREAD), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        // combine: as combine_partials_kernel<16>, of one row
        const int col = tid % COLS, pl = tid / COLS, c4 = at * COLS + col;
        bf16x4 res = bf16x4{0, 0, 0, 0};
        if (i == 0) {
            res = reinterpret_cast<const bf16x4 *>(s.x)[c4];
        } else if (tid < 64) {  // all of it has been there since the experts began
            uint32_t a[1], b[1];
            take_pairs<1>(x_words(i), [&](int) { return c4 * 16; }, i, true, a, b, s.flags);
            res = __builtin_bit_cast(bf16x4, make_uint2(a[0], b[0]));
        }
        {   // all partial sums of the block: every wavefront waits by itself
            const int c = tid & 63;
            const uint32_t want = c < SPREAD ? (P - c + SPREAD - 1) / SPREAD : 0;
            for (int looks = 1; __any(c < SPREAD && __hip_atomic_load(done(i, c & (SPREAD - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want);
                 ++looks) {
                if (looks == STACK_PATIENCE) {
                    wait_failed(s.flags);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            asm volatile("" ::: "memory");
        }
        const uint32_t flags = __hip_atomic_load(s.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
        constexpr int U = 8;
        for (int p0 = pl; p0 < P; p0 += PL * U) {
            floatx4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[u] = __builtin_bit_cast(floatx4, load_past_l2(partial, (min(p0 + u * PL, P - 1) * d + 4 * c4) * 4));
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (p0 + u * PL < P) sum += v[u];
        }
        sub[pl][col] = sum;
        __syncthreads();
        if (pl == 0) {  // sixteen lanes of the first wavefront
            sum = sub[0][col];
#pragma unroll
            for (int l = 1; l < PL; ++l) sum += sub[l][col];
            const float p = flags & kFlagStalled ? NAN : __uint_as_float(prob[0]);
            bf16x4 y, x;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float acc = fmaf(p, (float)(__bf16)sum[c], 0.f);
                y[c] = (__bf16)acc;
                x[c] = (__bf16)((float)res[c] + acc);
            }
            const uint2 words = __builtin_bit_cast(uint2, x);
            if (i + 1 < s.L) put_pair(x_words(i + 1), c4 * 16, words.x, words.y, i + 1);
            reinterpret_cast<bf16x4 *>(const_cast<__bf16 *>(s.x) + (size_t)(i + 1) * d)[c4] = x;
            if (s.y) reinterpret_cast<bf16x4 *>(s.y + (size_t)i * d)[c4] = y;
        }
    }
}

size_t decode_stack_workspace_bytes(const pgmoe_config &c) {
    const bool may = c.dtype == PGMOE_BF16 && c.top_k == 1 && c.n_blocks >= DECODE_STACK_LEAST && c.n_blocks <= STACK_BLOCKS && gate_small_applies(c, 1) &&
                     ffn_launch_is_decode_sized(c, 1) && reduce_lanes(c.d_ff / 32) == 16;
    return may ? StackScratch::bytes(c.d_model, c.d_ff, c.n_blocks) : 0;
}

bool decode_stack_applies(const pgmoe_ctx *ctx, int T) {
    return T == 1 && ctx->decode_stack && ctx->store_mode == STORE_RESIDENT && ctx->schedule == PGMOE_SCHED_PREGATED && ctx->distance == 1 &&
           !ctx->trace && !ctx->tim_on && ctx->standin_us <= 0.f;
}

int launch_decode_stack(pgmoe_ctx *ctx, const pgmoe_step_buffers *io, hipStream_t stream) {
    const pgmoe_config &c = ctx->cfg;
    DecodeStack s = {};
    s.x = (const __bf16 *)io->x_states;
    s.y = (__bf16 *)io->y_blocks;
    s.idx = io->topk_idx;
    s.prob = io->topk_prob;
    s.row_of = io->row_of;
    s.offsets = io->expert_offsets;
    s.src_row = ctx->dev_src_row;
    s.w_base = ctx->store_base;
    s.w_stride = ctx->expert_stride;
    s.block_stride = ctx->block_stride;
    s.scratch = (char *)io->workspace;
    s.flags = ctx->dev_flags;
    s.f = c.d_ff;
    s.L = c.n_blocks;
    s.src_stride = c.max_tokens;
    for (int b = 0; b < c.n_blocks; ++b) {
        s.gate_w[b] = (const __bf16 *)io->gate_w[b];
        s.gate_b[b] = io->gate_b ? io->gate_b[b] : nullptr;
        if (!aligned(s.gate_w[b], 16) || !aligned(s.gate_b[b], 4))
            return fail(ctx, PGMOE_EINVAL, "pgmoe_stack_step: misaligned hidden state, gate weight or bias of block %d", b);
    }
    const dim3 grid((unsigned)std::min(c.n_blocks, STACK_AHEAD) * (1 + c.d_ff / 32 + c.d_model / 64));
    const size_t lds = decode_lds_bytes(c.d_model / 32);
    const int n_words = StackScratch::cleared(c.d_model, c.n_blocks) / 16;
    hipLaunchKernelGGL(c.n_experts == 8 ? ffn_decode_stack_begin_kernel<1> : ffn_decode_stack_begin_kernel<2>, dim3(1 + (n_words + GS_THREADS - 1) / GS_THREADS),
                       dim3(GS_THREADS), 0, stream, s.x, s.gate_w[0], s.gate_b[0], c.d_model, s.idx, s.prob, s.flags, s.row_of, s.offsets, s.src_row,
                       (uint4 *)s.scratch, n_words);
    PG_HIP(ctx, hipGetLastError());
#define PG_STACK(KT_, EV_) hipLaunchKernelGGL((ffn_decode_stack_kernel<KT_, EV_>), grid, dim3(256), lds, stream, s)
    if (c.d_model == 768) {
        if (c.n_experts == 8) PG_STACK(24, 1);
        else PG_STACK(24, 2);
    } else {
        if (c.n_experts == 8) PG_STACK(32, 1);
        else PG_STACK(32, 2);
    }
#undef PG_STACK
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

}  // namespace pgmoe
