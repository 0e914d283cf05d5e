// Weighted combine (Sec. II-B: the gate's probabilities weigh the outputs of the activated
// experts): y[t] = sum_j prob[t,j] * y_perm[row_of[t*k+j]], gathered per token so that no
// atomics are needed and the sum order (j ascending) is fixed.  Optionally also writes the
// residual stand-in x_next = x_res + y that feeds the next MoE block.
#include "gate_small.h"
#include "pgmoe_internal.h"

namespace pgmoe {

template <typename XT, int N>
struct Vec {
    typedef XT type __attribute__((ext_vector_type(N)));
};

// One wavefront per token (small batches: per token and round of columns), VEC neighbouring columns per lane and round, so that the rows of all k experts and the residual
// are requested together and whole lines leave at once (a workgroup per token, four columns per thread: 15 us for 8191 tokens
// of d_model 768 with two experts each, now 10.4; 45 us for 16384 of 1024, now 28.7).
template <typename XT, int VEC>
__global__ __launch_bounds__(256) void combine_rows_kernel(const XT *__restrict__ y_perm, const int32_t *__restrict__ row_of,
                                                           const float *__restrict__ prob, int T, int d, int k, XT *__restrict__ y,
                                                           const XT *__restrict__ x_res, XT *__restrict__ x_next) {
    typedef typename Vec<XT, VEC>::type vec;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)t * d;
#pragma unroll 2
    for (int c = (blockIdx.y * 64 + lane) * VEC; c < d; c += gridDim.y * 64 * VEC) {
        vec res = {};
        if (x_next) res = *reinterpret_cast<const vec *>(x_res + row + c);
        float acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
        auto add = [&](int j) {
            const float p = prob[(size_t)t * k + j];
            const vec s = *reinterpret_cast<const vec *>(y_perm + (size_t)row_of[(size_t)t * k + j] * d + c);
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = fmaf(p, (float)s[v], acc[v]);
        };
        if (k == 2) {  // uniform: both rows in flight
            add(0);
            add(1);
        } else {
            for (int j = 0; j < k; ++j) add(j);
        }
        vec o, n;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            o[v] = (XT)acc[v];
            n[v] = (XT)((float)res[v] + acc[v]);
        }
        if (y) *reinterpret_cast<vec *>(y + row + c) = o;
        if (x_next) *reinterpret_cast<vec *>(x_next + row + c) = n;
    }
}

// d_model that is no multiple of four: a column at a time.
template <typename XT>
__global__ __launch_bounds__(256) void combine_scalar_kernel(const XT *__restrict__ y_perm, const int32_t *__restrict__ row_of,
                                                             const float *__restrict__ prob, int d, int k, XT *__restrict__ y,
                                                             const XT *__restrict__ x_res, XT *__restrict__ x_next) {
    const int t = blockIdx.x, c = blockIdx.y * 256 + threadIdx.x;
    if (c >= d) return;
    float acc = 0.f;
    for (int j = 0; j < k; ++j) acc = fmaf(prob[(size_t)t * k + j], (float)y_perm[(size_t)row_of[(size_t)t * k + j] * d + c], acc);
    const size_t o = (size_t)t * d + c;
    if (y) y[o] = (XT)acc;
    if (x_next) x_next[o] = (XT)((float)x_res[o] + acc);
}

// Combine straight from the FFN's unreduced float32 partials: for every selected row the P
// partials are added exactly as ffn_reduce_kernel<PL> adds them (PL interleaved sub-sums, then
// the sub-sums in ascending order), rounded to bf16 as y_perm would have been, and only then
// weighted and accumulated, so the result is bit-identical to reduce + combine.
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Gate: nothing, or CarriedGate: the first workgroups then finish the pre-gate whose partial planes the expert launch left.  The
// variant without one has no such argument (64 bytes of arguments a launch, 160 with it: 8 experts of 768 x 3072, one token, six
// blocks, each step waited for: 87.6 us a step on a slow host core, 90.3 with it).
template <int PL, typename... Gate>
__global__ __launch_bounds__(256) void combine_partials_kernel(const float *__restrict__ partial, int P, int n_rows,
                                                                const int32_t *__restrict__ row_of,
                                                                const float *__restrict__ prob, int d, int k,
                                                                __bf16 *__restrict__ y, const __bf16 *__restrict__ x_res,
                                                                __bf16 *__restrict__ x_next, Gate... carried) {
    int tiles = 0;
    if constexpr (sizeof...(Gate) > 0) {
        const CarriedGate &gate = the_gate(carried...);
        tiles = (gate.T + GM_TOK - 1) / GM_TOK;
        if ((int)blockIdx.x < tiles) {  // uniform over the workgroup
            if (blockIdx.y == 0) gate_finish_body(gate, blockIdx.x);
            return;
        }
    }
    // 256 threads = PL p-lanes x COLS float4 columns of one token (same split as ffn_reduce_kernel<PL>)
    constexpr int COLS = 256 / PL;
    __shared__ floatx4 sub[PL][COLS + 1];
    const int t = blockIdx.x - tiles;
    const int col = threadIdx.x % COLS, pl = threadIdx.x / COLS;
    const int c4 = blockIdx.y * COLS + col;
    const bool live = c4 < d / 4;
    const size_t plane4 = (size_t)n_rows * d / 4;
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    // the residual is needed last: request it first, so that its latency is not paid at the end
    bf16x4 res = bf16x4{0, 0, 0, 0};
    if (x_next && pl == 0 && live) res = *reinterpret_cast<const bf16x4 *>(x_res + (size_t)t * d + 4 * (size_t)c4);
    for (int j = 0; j < k; ++j) {
        floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
        const float p_j = prob[(size_t)t * k + j];  // used after the reduction: requested with the row index
        if (live) {
            const floatx4 *src = reinterpret_cast<const floatx4 *>(partial) + (size_t)row_of[(size_t)t * k + j] * (d / 4) + c4;
            // eight partials are requested at a time and then added in ascending order (the order
            // of ffn_reduce_kernel); a plain loop waits for every load before it issues the next
            constexpr int U = 8;
            for (int p0 = pl; p0 < P; p0 += PL * U) {
                floatx4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = p0 + u * PL;
                    v[u] = src[(size_t)(p < P ? p : pl) * plane4];  // past the end: a valid address, value unused
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p0 + u * PL < P) s += v[u];
            }
        }
        if (PL > 1) {
            __syncthreads();  // previous round's readers are done with sub
            sub[pl][col] = s;
            __syncthreads();
            if (pl == 0) {
                s = sub[0][col];
#pragma unroll
                for (int l = 1; l < PL; ++l) s += sub[l][col];
            }
        }
        if (pl == 0) {
            const float p = p_j;
            acc.x = fmaf(p, (float)(__bf16)s.x, acc.x);
            acc.y = fmaf(p, (float)(__bf16)s.y, acc.y);
            acc.z = fmaf(p, (float)(__bf16)s.z, acc.z);
            acc.w = fmaf(p, (float)(__bf16)s.w, acc.w);
        }
    }
    if (pl != 0 || !live) return;
    const size_t o = (size_t)t * d + 4 * (size_t)c4;
    if (y) {
        bf16x4 v;
        v.x = (__bf16)acc.x; v.y = (__bf16)acc.y; v.z = (__bf16)acc.z; v.w = (__bf16)acc.w;
        *reinterpret_cast<bf16x4 *>(y + o) = v;
    }
    if (x_next) {
        const bf16x4 r = res;
        bf16x4 v;
        v.x = (__bf16)((float)r.x + acc.x); v.y = (__bf16)((float)r.y + acc.y);
        v.z = (__bf16)((float)r.z + acc.z); v.w = (__bf16)((float)r.w + acc.w);
        *reinterpret_cast<bf16x4 *>(x_next + o) = v;
    }
}

int launch_combine_partials(pgmoe_ctx *ctx, const float *partial, int P, int n_rows, const int32_t *row_of,
                            const float *prob, int T, void *y, const void *x_res, void *x_next, hipStream_t s, const FusedGate *gate) {
    const pgmoe_config &c = ctx->cfg;
    const int pl = reduce_lanes(P);
    const int cols = 256 / pl;
    const dim3 grid(T + (gate ? (gate->T + GM_TOK - 1) / GM_TOK : 0), (c.d_model / 4 + cols - 1) / cols);
#define PG_CP(PL_)                                                                                                                  \
    hipLaunchKernelGGL(combine_partials_kernel<PL_>, grid, dim3(256), 0, s, partial, P, n_rows, row_of, prob, c.d_model, c.top_k,      \
                       (__bf16 *)y, (const __bf16 *)x_res, (__bf16 *)x_next)
#define PG_CP_GATE(PL_)                                                                                                             \
    hipLaunchKernelGGL((combine_partials_kernel<PL_, CarriedGate>), grid, dim3(256), 0, s, partial, P, n_rows, row_of, prob, c.d_model, \
                       c.top_k, (__bf16 *)y, (const __bf16 *)x_res, (__bf16 *)x_next, cg)
    if (gate) {
        const bool route = gate_mfma_routes(c, gate->T);
        const CarriedGate cg = {(const __bf16 *)gate->x, (const __bf16 *)gate->w, gate->bias, gate->T, c.d_model, c.top_k, c.n_experts,
                                gate->idx, gate->prob, ctx->dev_flags, route ? gate->row_of : nullptr, route ? gate->offsets : nullptr,
                                route ? gate->src_row : nullptr, ctx->gate_planes};
        if (pl == 1) PG_CP_GATE(1);
        else if (pl == 4) PG_CP_GATE(4);
        else PG_CP_GATE(16);
    } else {
        if (pl == 1) PG_CP(1);
        else if (pl == 4) PG_CP(4);
        else PG_CP(16);
    }
#undef PG_CP_GATE
#undef PG_CP
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

template <typename XT>
static void launch_t(const pgmoe_config &c, const void *y_perm, const int32_t *row_of, const float *prob, int T, void *y,
                     const void *x_res, void *x_next, hipStream_t s) {
    const int d = c.d_model;
    constexpr int WIDE = 16 / (int)sizeof(XT);  // columns of a 16-byte access
    auto grid = [&](int vec) { return dim3((T + 3) / 4, T <= 1024 ? (d + 64 * vec - 1) / (64 * vec) : 1); };  // few tokens: as many wavefronts as there are
    // 16 bytes per lane where whole rounds of 64 lanes come out, else the narrower access (whose rows are aligned to it, too)
    if (d % (64 * WIDE) == 0)
        hipLaunchKernelGGL((combine_rows_kernel<XT, WIDE>), grid(WIDE), dim3(256), 0, s, (const XT *)y_perm, row_of, prob, T, d, c.top_k, (XT *)y,
                           (const XT *)x_res, (XT *)x_next);
    else if (d % 4 == 0)
        hipLaunchKernelGGL((combine_rows_kernel<XT, 4>), grid(4), dim3(256), 0, s, (const XT *)y_perm, row_of, prob, T, d, c.top_k, (XT *)y,
                           (const XT *)x_res, (XT *)x_next);
    else
        hipLaunchKernelGGL(combine_scalar_kernel<XT>, dim3(T, (d + 255) / 256), dim3(256), 0, s, (const XT *)y_perm, row_of, prob, d,
                           c.top_k, (XT *)y, (const XT *)x_res, (XT *)x_next);
}

int launch_combine(pgmoe_ctx *ctx, const void *y_perm, const int32_t *row_of, const float *prob, int T, void *y,
                   const void *x_res, void *x_next, hipStream_t s) {
    if (ctx->cfg.dtype == PGMOE_F32)
        launch_t<float>(ctx->cfg, y_perm, row_of, prob, T, y, x_res, x_next, s);
    else
        launch_t<__bf16>(ctx->cfg, y_perm, row_of, prob, T, y, x_res, x_next, s);
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

}  // namespace pgmoe
