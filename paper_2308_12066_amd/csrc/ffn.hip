// Expert execution (Sec. II-B: every activated expert, a dense FFN, processes the tokens
// routed to it):  y_perm[rows of e] = ReLU(x_perm[rows of e] . W1_e) . W2_e.
//
// bf16 path - three kernels, picked from the shape of the launch alone (plan_ffn and friends):
//   ffn_fused_kernel   the general, HBM-bound case (described next);
//   ffn_decode_kernel  a handful of active experts with <= 16 rows each (batch-1 decode);
//   ffn_gemm_pack_rows_kernel + ffn_gemm_tile_kernel (twice)  many rows per expert: two tiled GEMMs (ffn_gemm.hip).
// The fused kernel streams the weights from HBM exactly once per 16*MT-row chunk:
//   workgroup = (chunk of <= 16*MT rows of one expert) x (a range of d_ff columns)
//   = (blockIdx.x, blockIdx.y).
//   It keeps the chunk's activations in LDS, already in matrix-core operand order, and walks
//   its d_ff range in sub-slabs of SUB = 16*NW columns (NW wavefronts per workgroup):
//     phase A  wave w computes the 16 hidden features of n-tile w over the full d_model
//              reduction (W1 tiles are contiguous in memory along k), applies ReLU, rounds to
//              bf16 and drops the result into LDS in operand order for phase B;
//     phase B  every wave multiplies that sub-slab of hidden features into its own d_model/NW
//              output columns (W2 tiles of one k-tile are contiguous along n) and keeps the
//              running output in registers across all sub-slabs.
//   The hidden activation never leaves the CU.  With P > 1 d_ff ranges per chunk the partial
//   outputs go to a float32 scratch [P][rows][d] and ffn_reduce_kernel adds them in fixed
//   order (no atomics: results are bit-reproducible); with P == 1 the kernel writes y_perm.
//   The weights are the A operand (v_mfma_f32_16x16x32_bf16, 16 features x 32 k) and the
//   tokens the B operand, so each lane ends up with 4 consecutive features of one token.
//
// f32 path - float32 matrix instructions (d_model and d_ff multiples of 4), else plain scalar kernels.
#include <mutex>

#include "ffn_common.h"
#include "ffn_decode.h"
#include "gate_small.h"

namespace pgmoe {

// An address that is the same for the whole wavefront, in scalar registers.
__device__ inline const char *uniform_address(const void *p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (const char *)(((unsigned long long)hi << 32) | lo);
}

// MT: 16-row tiles per chunk; KT = d_model/32; NW: wavefronts per workgroup (sub-slab = 16*NW
// d_ff columns); D: weight tiles (1 KiB each) a wavefront keeps in flight.
//
// Per sub-slab a wavefront consumes NT = KT + KTB*NTB weight tiles in a fixed order: first the
// KT tiles of its own W1 n-tile (phase A), then, for each of the KTB k-tiles of the sub-slab,
// its NTB W2 tiles (phase B).  The tiles form one linear stream over all sub-slabs; tile g+D is
// requested when tile g is consumed, so loads run ahead of the matrix cores across both phases
// and across the LDS barrier between them.
//
// Gate: nothing, or CarriedGate: grid row 0 then runs that gate's first half and the d_ff ranges follow.  A variant of its own, because
// the gate's code costs small kernels registers (d_model 64: 106 with it, 48 without) that a launch without a gate has no use for.
constexpr int FUSED_PINNED = 0x6;  // what the scheduler may move past a request: scalar and vector arithmetic, not products, loads or LDS reads
template <int MT, int KT, int NW, int D, typename... Gate>
__global__ __launch_bounds__(NW * 64) void ffn_fused_kernel(
    const __bf16 *__restrict__ x_perm, const int32_t *__restrict__ offsets, int E, int f, int f_range,
    const char *__restrict__ w_base, size_t w_stride, int slot_by_rank, int n_slots,
    const unsigned long long *__restrict__ table, float *__restrict__ partial, __bf16 *__restrict__ y_perm, int n_rows,
    const int32_t *__restrict__ src_row,  // nullable: grouped row r is row src_row[r] of x_perm (rows not gathered yet)
    Gate... carried) {
    constexpr int SUB = 16 * NW;      // d_ff columns per sub-slab
    constexpr int KTB = SUB / 32;     // k-tiles of phase B per sub-slab
    constexpr int NTD = KT * 2;       // n-tiles of the output (d_model / 16)
    constexpr int NTB = NTD / NW;     // output n-tiles per wavefront
    constexpr int NT_A = KT, NT_B = KTB * NTB, NT = NT_A + NT_B;
    constexpr int d = KT * 32;
    static_assert(NTD % NW == 0 && SUB % 32 == 0, "tile split");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int range = blockIdx.y;
    if constexpr (sizeof...(Gate) > 0) {
        static_assert(NW == 4, "the first half is 256 threads'");
        const CarriedGate &gate = the_gate(carried...);
        if (range-- == 0) {  // uniform over the workgroup
            for (int u = blockIdx.x; u < 2 * ((gate.T + GM_TOK - 1) / GM_TOK); u += gridDim.x) gate_planes_body(gate, u);
            return;
        }
    }

    const ChunkInfo ci = find_chunk(offsets, E, 16 * MT, blockIdx.x);
    if (ci.nrows == 0) return;  // uniform over the workgroup
    // where the expert's blob is: through the cache's pointer table, by slot rank, or by expert id
    const char *wexp = table ? reinterpret_cast<const char *>(table[ci.expert])
                             : w_base + (size_t)(slot_by_rank ? ci.slot : ci.expert) * w_stride;
    const bool no_weights = table ? wexp == nullptr : (slot_by_rank && ci.slot >= n_slots);  // no slot: rows are zeroed

    const int n_sub = no_weights ? 0 : f_range / SUB;
    const int fs0 = range * f_range;

    // tile i (0 <= i < NT, compile-time after unrolling) of sub-slab s
    // A wavefront's tiles of sub-slab s: scalar addresses, to which a lane adds its 16 bytes, through descriptors of up to four tiles.  Past the last
    // sub-slab these are empty: requests for tiles there read no memory, so every request is made and the compiler knows how many loads are in
    // flight at any point.  With requests that depended on s it waited for all of them towards the end of every sub-slab, and it moved them down to
    // where it waited: 64 experts of 1024 x 4096, 2000 skewed rows 278 -> 237 us a block, 128 experts 1500 rows 413 -> 397, 128 rows 130 -> 122.
    const char *const w1 = uniform_address(wexp), *const w2 = w1 + (size_t)d * f * 2;
    struct Slab {
        const char *a, *b;
        int window;  // bytes of a descriptor
    };
    auto slab = [&](int s) {
        const int fs = fs0 + s * SUB;
        return Slab{w1 + ((size_t)((fs >> 4) + wave) * KT << 10), w2 + ((size_t)((fs >> 5) * NTD + wave * NTB) << 10), s < n_sub ? 4096 : 0};
    };
    // The 16-row chunks of d_model 256 keep plain conditional loads: their launches are of about four workgroups per CU, for which the steady stream has no
    // registers (128 experts of 256 x 1024, one row each: 29.8 us so, 31.3 steady, 30.1 steady with eight tiles in flight; of 256 x 4096, 128 skewed rows 38.1,
    // 44.3 and 37.2, three rows each 86.5, 92.6 and 92.1).
    constexpr bool PLAIN = MT == 1 && KT == 8;
    auto load_tile = [&](const Slab &sl, int i) -> bf16x8 {
        const int j = i - NT_A, kb = j / NTB, a = j - kb * NTB, in_run = i < NT_A ? i : a;
        const char *run = i < NT_A ? sl.a : sl.b + ((size_t)(kb * NTD) << 10);
        if constexpr (PLAIN) return *(const global_bf16x8 *)(run + ((size_t)in_run << 10) + lane * 16);
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(run + ((size_t)(in_run & ~3) << 10)), 0, sl.window, 0x00020000);
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16 + ((in_run & 3) << 10), 0, 0));
    };

    // Tiles in flight: sixteen for a wavefront of 16-row chunks, eight where the accumulators of 32 and 64 rows would leave fewer wavefronts per SIMD (d_model 256:
    // 18 rows for each of 64 experts of 256 x 1024 25.2 us with sixteen, 16.3 with eight; 45 for each of 128 47.2 and 33.7), four for the eight wavefronts of the
    // 64-row chunks of 1024 and two of 768, which HBM paces: rows that lie evenly pass with few tiles in flight, skewed ones want more (three streams, conditional requests with
    // eight / steady ones with two / four / eight: 128 experts of 768 x 3072, 4096 rows 231.3 / 227.8 / 231.3 / 231.2 us, 32 uneven rows each 215.8 / 216.3 /
    // 219.4 / 221.8, 28 skewed ones 253.8 / 243.9 / 240.8 / 244.3, 4096 skewed ones 260.5 / 246.6 / 240.7 / 242.7).
    static_assert(D <= NT && NT % D == 0, "the ring reaches into the next sub-slab at most, where a tile finds the place that was filled for it");
    // The 16- and 32-row chunks of d_model 512 leave it to the compiler: launches of theirs that fill the chip are paced by HBM, which the pauses do not
    // slow (256 experts of 512 x 2048, 3000 rows: 214 us a block, 218 with the steady stream), and the steady stream's registers cost a wavefront per SIMD.
    constexpr bool STEADY = !PLAIN && (KT != 16 || MT == 4);
    bf16x8 ring[D];
    Slab now = slab(0);
#pragma unroll
    for (int g = 0; g < D; ++g)
        if (!PLAIN || n_sub > 0) ring[g] = load_tile(now, g);

    bf16x8 *xs = reinterpret_cast<bf16x8 *>(smem);   // [MT][KT][64] operand cells
    bf16x8 *hs = xs + (size_t)MT * KT * 64;          // [2][MT][KTB][64]

    // stage the chunk's rows (zero-filling rows beyond nrows) while the first weight tiles fly
    {
        constexpr int cells_per_row = d >> 3;
        const uint4 *src = reinterpret_cast<const uint4 *>(x_perm);
        uint4 *dst = reinterpret_cast<uint4 *>(xs);
        for (int i = tid; i < 16 * MT * cells_per_row; i += NW * 64) {
            const int m = i / cells_per_row, k8 = i - m * cells_per_row;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (m < ci.nrows) {
                const int row = ci.row0 + m;
                v = src[(size_t)(src_row ? src_row[row] : row) * cells_per_row + k8];
            }
            dst[(((m >> 4) * KT + (k8 >> 2)) << 6) + (m & 15) + 16 * (k8 & 3)] = v;
        }
    }
    lds_barrier();

    floatx4 yacc[NTB][MT];
#pragma unroll
    for (int a = 0; a < NTB; ++a)
#pragma unroll
        for (int m = 0; m < MT; ++m) yacc[a][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    // The rows' operand cells are read from LDS AHEAD tiles before their products, or with 0 where the compiler puts it: in the largest chunks of d_model 512
    // and 768 and at d_model 2048 the registers are worth more as they are (128 experts of 512 x 2048, some 50 rows each: 182 us with reads ahead and
    // conditional requests, 113 steady and without; 128 of 768 x 3072, 28 skewed rows 253 and 244, 256 of 768 x 1536, 27 skewed rows 302 and 281; 4 of
    // 2048 x 8192, 10 rows each, three launches at a time 55.3 and 53.7).
    constexpr bool AS_IT_COMES = (MT == 4 && (KT == 16 || (KT == 24 && NW == 8))) || KT == 64;
    constexpr int AHEAD = AS_IT_COMES ? 0 : (KT < 4 ? 1 : (KT == 8 ? 2 : (MT == 1 ? 4 : (MT == 2 || NW == 8 ? 2 : 1))));
    static_assert(AHEAD <= NT_A && AHEAD <= NT_B, "the cells of the next sub-slab replace none that is still to be used");
    bf16x8 xa[AHEAD + 1][MT];
    constexpr int HB = MT * NTB >= 32 || KT == 8 || AS_IT_COMES ? 1 : 2;  // hidden cells of the next k-tile, too, where the accumulators leave registers for them
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) xa[i][m] = xs[((m * KT + i) << 6) + lane];

    const int q = lane >> 4;
    for (int s = 0; s < n_sub; ++s) {
        const Slab next = slab(s + 1);
        floatx4 hacc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) hacc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        bf16x8 hfrag[HB][MT];
        const bf16x8 *hb = hs + (size_t)(s & 1) * MT * KTB * 64;
        static_for<NT>([&](auto tile) {
            constexpr int i = decltype(tile)::value;
            const bf16x8 v = ring[i % D];
            // request tile g + D of the stream; where STEADY it stays where it is written
            if (STEADY || i + D < NT || s + 1 < n_sub) ring[i % D] = load_tile(i + D < NT ? now : next, (i + D) % NT);
            if constexpr (AHEAD > 0 && (i + AHEAD) % NT < NT_A) {
#pragma unroll
                for (int m = 0; m < MT; ++m) xa[(i + AHEAD) % NT % (AHEAD + 1)][m] = xs[((m * KT + (i + AHEAD) % NT) << 6) + lane];
            }
            if constexpr (STEADY) __builtin_amdgcn_sched_barrier(FUSED_PINNED);
            if constexpr (i < NT_A) {
                // ---- phase A: hidden features [fs + 16*wave, +16) over the full d_model reduction
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    hacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, AHEAD > 0 ? xa[i % (AHEAD + 1)][m] : xs[((m * KT + i) << 6) + lane], hacc[m], 0, 0, 0);
                if (i == NT_A - 1) {
                    // ReLU, round to bf16, store as phase-B operand: feature 16*wave + 4*q + r is
                    // k-tile wave/2, k-group 2*(wave%2) + q/2, position 4*(q%2) + r of token lane%16
                    char *hbase = reinterpret_cast<char *>(hs + (size_t)(s & 1) * MT * KTB * 64);
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        bf16x4 h;
                        h.x = (__bf16)fmaxf(hacc[m].x, 0.f);
                        h.y = (__bf16)fmaxf(hacc[m].y, 0.f);
                        h.z = (__bf16)fmaxf(hacc[m].z, 0.f);
                        h.w = (__bf16)fmaxf(hacc[m].w, 0.f);
                        const int cell = ((m * KTB + (wave >> 1)) << 6) + (lane & 15) + 16 * (2 * (wave & 1) + (q >> 1));
                        *reinterpret_cast<bf16x4 *>(hbase + (size_t)cell * 16 + 8 * (q & 1)) = h;
                    }
                    // one barrier per sub-slab is enough: the next sub-slab writes the other half of hs
                    lds_barrier();
                }
            } else {
                // ---- phase B: y[:, wave's columns] += H_sub . W2[fs .. fs+SUB, wave's columns]
                constexpr int j = i - NT_A, kb = j / NTB, a = j - kb * NTB;
                if (a == 0 && (HB == 1 || kb == 0)) {
#pragma unroll
                    for (int m = 0; m < MT; ++m) hfrag[0][m] = hb[((m * KTB + kb) << 6) + lane];
                }
                if (HB > 1 && a == 0 && kb + 1 < KTB) {
#pragma unroll
                    for (int m = 0; m < MT; ++m) hfrag[(kb + 1) % HB][m] = hb[((m * KTB + kb + 1) << 6) + lane];
                }
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    yacc[a][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, hfrag[kb % HB][m], yacc[a][m], 0, 0, 0);
            }
        });
        now = next;
    }

    // ---- epilogue: lane holds token (lane%16) of tile m, output columns 16*(wave*NTB+a) + 4*q + {0..3}
    const int tok = lane & 15;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int r = m * 16 + tok;
        if (r >= ci.nrows) continue;
        const size_t row = (size_t)ci.row0 + r;
        if (partial) {
            float *dst = partial + ((size_t)range * n_rows + row) * d + (wave * NTB) * 16 + 4 * q;
#pragma unroll
            for (int a = 0; a < NTB; ++a) *reinterpret_cast<floatx4 *>(dst + a * 16) = yacc[a][m];
        } else {
            __bf16 *dst = y_perm + row * d + (wave * NTB) * 16 + 4 * q;
#pragma unroll
            for (int a = 0; a < NTB; ++a) {
                bf16x4 o;
                o.x = (__bf16)yacc[a][m].x;
                o.y = (__bf16)yacc[a][m].y;
                o.z = (__bf16)yacc[a][m].z;
                o.w = (__bf16)yacc[a][m].w;
                *reinterpret_cast<bf16x4 *>(dst + a * 16) = o;
            }
        }
    }
}

// Decode-sized variant (at most a few experts active, <= 16 rows each): one workgroup of four
// wavefronts per (chunk, 32-column sub-slab of d_ff), every weight tile it needs requested before
// anything else happens, so the kernel is one round of memory latency deep instead of a ring of
// dependent rounds.  Phase A splits the d_model reduction over wavefront pairs (wave = n-tile
// + 2 * k-half; the two halves are added in LDS, k-half 0 first), phase B gives each wavefront a
// quarter of the output columns.  Always writes float32 partials (one per sub-slab).
// The chunk's rows of x are fetched after the weights have been requested, through the row ->
// token map: asking for the map at kernel start and for x ahead of the weights, or right behind
// them, was measured 0.5 and 0.3 us slower per launch (same box, alternating builds): whatever
// delays the first weight request costs more than the late x saves.
// One instantiation per kind of gate: with all of them in one kernel it took 288 registers and 352 bytes of scratch per lane (the 16-expert
// gate still does), and fewer workgroups of neighbouring steps shared a CU (T = 4, 8 experts of 768 x 3072, six blocks: 56 us a
// step with steps of several stacks in flight, now 48).
enum DecodeGateKind { DECODE_NO_GATE, DECODE_SMALL_GATE_8, DECODE_SMALL_GATE_16, DECODE_GATE_PLANES };  // small: for 8 / 16 experts
template <int KT, DecodeGateKind GATE>
__global__ __launch_bounds__(256) void ffn_decode_kernel(
    const __bf16 *__restrict__ x_perm, const int32_t *__restrict__ offsets, int E, int f,
    const char *__restrict__ w_base, size_t w_stride, int slot_by_rank, int n_slots,
    const unsigned long long *__restrict__ table, float *__restrict__ partial, int n_rows,
    const int32_t *__restrict__ src_row,  // nullable: grouped row r is row src_row[r] of x_perm
    CarriedGate gate) {           // the last grid row runs that gate (planes: its first half) instead of a sub-slab
    constexpr int d = KT * 32;
    if (GATE != DECODE_NO_GATE && blockIdx.y == gridDim.y - 1) {  // uniform over the workgroup
        if constexpr (GATE == DECODE_GATE_PLANES)
            for (int u = blockIdx.x; u < 2 * ((gate.T + GM_TOK - 1) / GM_TOK); u += gridDim.x) gate_planes_body(gate, u);
        else if (blockIdx.x == 0)
            gate_small_dispatch<GATE == DECODE_SMALL_GATE_8 ? 1 : 2>(gate.x, gate.w, gate.bias, gate.T, d, gate.k, gate.idx, gate.prob, nullptr,
                                                                     gate.flags, gate.row_of, gate.offsets, gate.src_row);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const ChunkInfo ci = find_chunk(offsets, E, 16, blockIdx.x);
    if (ci.nrows == 0) return;  // uniform over the workgroup
    const char *wexp = table ? reinterpret_cast<const char *>(table[ci.expert])
                             : w_base + (size_t)(slot_by_rank ? ci.slot : ci.expert) * w_stride;
    const bool no_weights = table ? wexp == nullptr : (slot_by_rank && ci.slot >= n_slots);  // no slot: rows are zeroed
    decode_sub_slab<KT>(
        smem, no_weights ? nullptr : wexp, f, blockIdx.y,
        [&](bf16x8 *xs) {
            constexpr int cells_per_row = d >> 3;
            const uint4 *src = reinterpret_cast<const uint4 *>(x_perm);
            uint4 *dst = reinterpret_cast<uint4 *>(xs);
            for (int i = threadIdx.x; i < 16 * cells_per_row; i += 256) {
                const int m = i / cells_per_row, k8 = i - m * cells_per_row;
                uint4 v = make_uint4(0, 0, 0, 0);
                if (m < ci.nrows) {
                    const int row = ci.row0 + m;
                    v = src[(size_t)(src_row ? src_row[row] : row) * cells_per_row + k8];
                }
                dst[((k8 >> 2) << 6) + m + 16 * (k8 & 3)] = v;
            }
        },
        [&](int column, int tok, const floatx4 &y) {
            if (tok < ci.nrows) *reinterpret_cast<floatx4 *>(partial + ((size_t)blockIdx.y * n_rows + (size_t)ci.row0 + tok) * d + column) = y;
        });
}

// y_perm[row][c] = bf16( sum_p partial[p][row][c] ).  A workgroup of 256 threads covers 256/PL
// float4 columns; its PL "p-lanes" each add every PL-th partial (p = pl, pl+PL, ...) and the PL
// sub-sums are added in ascending order, so the result does not depend on scheduling.  PL is
// picked from P alone (1 for P <= 2, 4 for P <= 8, else 16).
template <int PL>
__global__ __launch_bounds__(256) void ffn_reduce_kernel(const float *__restrict__ partial, int P, int n_rows, int d,
                                                          __bf16 *__restrict__ y_perm) {
    constexpr int COLS = 256 / PL;
    __shared__ floatx4 sub[PL][COLS + 1];
    const size_t total4 = (size_t)n_rows * d / 4;
    const int col = threadIdx.x % COLS, pl = threadIdx.x / COLS;
    const size_t i = (size_t)blockIdx.x * COLS + col;
    floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
    if (i < total4) {
        const floatx4 *src = reinterpret_cast<const floatx4 *>(partial) + i;
        for (int p = pl; p < P; p += PL) s += src[(size_t)p * total4];
    }
    static_assert(PL == 1 || PL == 4 || PL == 16, "keep in step with reduce_lanes()");
    if (PL > 1) {
        sub[pl][col] = s;
        __syncthreads();
        if (pl != 0) return;
        s = sub[0][col];
#pragma unroll
        for (int k = 1; k < PL; ++k) s += sub[k][col];
    }
    if (i < total4) {
        bf16x4 o;
        o.x = (__bf16)s.x;
        o.y = (__bf16)s.y;
        o.z = (__bf16)s.z;
        o.w = (__bf16)s.w;
        reinterpret_cast<bf16x4 *>(y_perm)[i] = o;
    }
}

// ------------------------------------------------------------------------------------------
// float32 path on the float32 matrix instruction (v_mfma_f32_16x16x4_f32: float32 products and sums).
//
// A workgroup takes up to 16*MT rows of one expert and 16*V columns; its NW wavefronts deal the reduction among
// themselves in blocks of 16 k and add their sums in LDS in wavefront order (bit-reproducible).  The weights are
// row-major, so nothing is transposed: lane l loads V neighbouring columns V*(l%16) .. of weight row 16*b + 4*(l/16) + s
// and the four k of its token 4*(l/16) .. +3; instruction (s, j) then multiplies component j of the weights with component s
// of the row, i.e. its output row i is column V*i + j, and every lane ends up with 4*V neighbouring columns of one token.
// Bound by the weight stream (HBM); F32_DEPTH blocks of loads are in flight per wavefront.  One thread
// per output column walking k by itself, which this replaces, re-read the weights once per row and paid a
// memory latency every few k: 8 experts of 768 x 3072, 100 rows, 284 us + 836 us, now 17 + 20 from the last-level cache (75 MB of weights each).
// 18.4 + 23.7 while the requests were conditional: the compiler, which then cannot count them, waited for every load in flight once per round of blocks,
// so the blocks came in batches with a memory latency between them.
constexpr int F32_DEPTH = 4;
constexpr size_t F32_ALONE = 52 * 1024;  // of LDS beside the 32 KiB of a workgroup of 64 rows, 16 columns and eight wavefronts: more than half a CU's

template <int V>
struct F32Vec {
    typedef float type __attribute__((ext_vector_type(V)));
};
template <>
struct F32Vec<1> {
    typedef float type;
};
template <int V>
__device__ inline float f32_comp(const typename F32Vec<V>::type &v, int j) {
    if constexpr (V == 1) return v;
    else return v[j];
}

template <int V>
__device__ inline typename F32Vec<V>::type f32_load(__amdgpu_buffer_rsrc_t rsrc, int lane_off) {
    if constexpr (V == 1) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_off, 0, 0));
    else if constexpr (V == 2) return __builtin_bit_cast(typename F32Vec<V>::type, __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane_off, 0, 0));
    else return __builtin_bit_cast(typename F32Vec<V>::type, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off, 0, 0));
}

__device__ inline const RowCombine &the_combine(const RowCombine &combine) { return combine; }

// out[rows, n0 .. n0 + 16*V) = (RELU) a[rows, K] . w[K, N] for the rows of one chunk; a_row0: row of a that is the chunk's
// first (through src_row if given).  K % 4 == 0, N % V == 0.
// Combine: nothing, or RowCombine: grouped row r is the one row of token tokens[r], whose weighted result and residual sum are written instead of out
// (the arithmetic of combine_rows_kernel with one expert per token).
template <int V, int MT, int NW, bool RELU, typename... Combine>
__device__ inline void f32_tile(const float *__restrict__ a, const int32_t *__restrict__ src_row, const float *__restrict__ w,
                                float *__restrict__ out, const ChunkInfo &ci, int K, int N, bool no_weights,
                                const int32_t *__restrict__ tokens = nullptr, Combine... combine) {
    typedef typename F32Vec<V>::type vec;
    __shared__ floatx4 sums[NW][V * MT][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.y * 16 * V;
    const int col = n0 + V * i16;
    const char *weights = uniform_address(w);
    const int row_bytes = N * 4;
    int w_off[4];  // in a lane's offset, not the scalar one: that would move the descriptor's end, too
#pragma unroll
    for (int s = 0; s < 4; ++s) w_off[s] = (4 * g + s) * row_bytes + (col < N ? col : 0) * 4;  // columns past the end: valid ones, never stored
    const floatx4 *ap[MT];
    floatx4 acc[V][MT];
#pragma unroll
    for (int j = 0; j < V; ++j)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[j][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int n_blk = no_weights ? 0 : (K + 15) >> 4, quads = K >> 2;
    vec wv[F32_DEPTH][4];
    floatx4 av[F32_DEPTH][MT];
    // Every request is made, also past the end of K, so that the compiler knows how many are in flight: behind conditional ones it waited for all.
    // Weights past the end come from no memory, as zeros (the descriptor ends there); activations are the row's last ones, zeroed when used.
    auto request_weights = [&](int b, vec (&wb)[4]) {
        const int rows = __builtin_amdgcn_readfirstlane(max(0, min(16, K - 16 * b)));  // (the clamp alone would be a vector instruction)
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(weights + (size_t)min(16 * b, K) * row_bytes), 0, rows * row_bytes, 0x00020000);
#pragma unroll
        for (int s = 0; s < 4; ++s) wb[s] = f32_load<V>(rsrc, w_off[s]);
    };
    auto request_rows = [&](int b, floatx4 (&ab)[MT]) {
#pragma unroll
        for (int m = 0; m < MT; ++m) ab[m] = ap[m][min(4 * b + g, quads - 1)];
    };
    auto multiply = [&](int b, const vec (&wb)[4], const floatx4 (&ab)[MT]) {
        const bool live = 4 * b + g < quads;  // false only past the end of K
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < V; ++j)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(f32_comp<V>(wb[s], j), live ? ab[m][s] : 0.f, acc[j][m], 0, 0, 0);
    };
    int row[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int r = m * 16 + i16;
        row[m] = ci.row0 + (r < ci.nrows ? r : 0);  // rows past the end: a valid row, never stored
        if (src_row) row[m] = src_row[row[m]];
    }
    __builtin_amdgcn_sched_barrier(0);
    // With no second round for any wavefront each asks for what there is: surplus requests cost rows that nobody needs, and short sums have nothing to hide them behind (100 rows
    // for each of 4 experts of 256 x 512 18.8 us with them, 14.5 so; 40 for each of 16 of 64 x 256 11.2 and 9.7).
    if (n_blk < NW * F32_DEPTH) {
        typedef __attribute__((address_space(1))) vec gvec;
        const gvec *wp = (const gvec *)(w + (col < N ? col : 0));
        auto each = [&](auto f) {
#pragma unroll
            for (int p = 0; p < F32_DEPTH; ++p)
                if (wave + NW * p < n_blk) f(wave + NW * p, min(4 * (wave + NW * p) + g, quads - 1), wv[p], av[p]);  // uniform over the wavefront, as below
        };
        each([&](int, int q, vec (&wb)[4], floatx4 (&)[MT]) {
#pragma unroll
            for (int s = 0; s < 4; ++s) wb[s] = wp[(size_t)(4 * q + s) * (N / V)];
        });
#pragma unroll
        for (int m = 0; m < MT; ++m) ap[m] = reinterpret_cast<const floatx4 *>(a + (size_t)row[m] * K);
        each([&](int, int q, vec (&)[4], floatx4 (&ab)[MT]) {
#pragma unroll
            for (int m = 0; m < MT; ++m) ab[m] = ap[m][q];
        });
        each([&](int b, int, vec (&wb)[4], floatx4 (&ab)[MT]) {
#pragma unroll
            for (int s = 0; s < 4; ++s) wb[s] = 4 * b + g < quads ? wb[s] : vec{};
            multiply(b, wb, ab);
        });
    } else {
#pragma unroll
        for (int p = 0; p < F32_DEPTH; ++p) request_weights(wave + NW * p, wv[p]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MT; ++m) ap[m] = reinterpret_cast<const floatx4 *>(a + (size_t)row[m] * K);  // the weights did not wait for it
#pragma unroll
        for (int p = 0; p < F32_DEPTH; ++p) request_rows(wave + NW * p, av[p]);
        int b0 = wave;
        auto round = [&]() {
#pragma unroll
            for (int p = 0; p < F32_DEPTH; ++p) {
                multiply(b0 + NW * p, wv[p], av[p]);
                __builtin_amdgcn_sched_barrier(0);
                request_weights(b0 + NW * (p + F32_DEPTH), wv[p]);
                request_rows(b0 + NW * (p + F32_DEPTH), av[p]);
                __builtin_amdgcn_sched_barrier(0);
            }
            b0 += NW * F32_DEPTH;
        };
        if (b0 + NW * F32_DEPTH < n_blk) {
            round();  // on its own: what it waits for lies in another order than in the rounds after it
            while (b0 + NW * F32_DEPTH < n_blk) round();
        }
#pragma unroll
        for (int p = 0; p < F32_DEPTH; ++p) {
            if (b0 + NW * p >= n_blk) break;
            multiply(b0 + NW * p, wv[p], av[p]);
        }
    }
#pragma unroll
    for (int j = 0; j < V; ++j)
#pragma unroll
        for (int m = 0; m < MT; ++m) sums[wave][j * MT + m][lane] = acc[j][m];
    // thread -> (row tile, lane, r): V neighbouring columns of one row
    constexpr int OUT = (MT * 256 + NW * 64 - 1) / (NW * 64);
    vec res[OUT];
    float prob[OUT];
    int token[OUT];
    if constexpr (sizeof...(Combine) > 0) {  // on their way while the sums meet (ahead of the products they delayed the first weights)
        const RowCombine &rc = the_combine(combine...);
#pragma unroll
        for (int o = threadIdx.x, i = 0; o < MT * 256; o += NW * 64, ++i) {
            const int l = (o >> 2) & 63, m = o >> 8, row = m * 16 + (l & 15), c = n0 + V * (4 * (l >> 4) + (o & 3));
            token[i] = tokens[ci.row0 + (row < ci.nrows ? row : 0)];
            prob[i] = rc.prob[token[i]];
            res[i] = *reinterpret_cast<const vec *>(rc.x_res + (size_t)token[i] * N + (c < N ? c : 0));
        }
    }
    __syncthreads();
#pragma unroll
    for (int o = threadIdx.x, i = 0; o < MT * 256; o += NW * 64, ++i) {
        const int r = o & 3, l = (o >> 2) & 63, m = o >> 8;
        const int row = m * 16 + (l & 15), c = n0 + V * (4 * (l >> 4) + r);
        if (row >= ci.nrows || c >= N) continue;
        vec y;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float t = sums[0][j * MT + m][l][r];
#pragma unroll
            for (int v = 1; v < NW; ++v) t += sums[v][j * MT + m][l][r];
            if (RELU) t = fmaxf(t, 0.f);
            if constexpr (V == 1) y = t;
            else y[j] = t;
        }
        if constexpr (sizeof...(Combine) > 0) {
            const RowCombine &rc = the_combine(combine...);
            const size_t at = (size_t)token[i] * N + c;
            vec n;
            if constexpr (V == 1) {
                y = fmaf(prob[i], y, 0.f);
                n = res[i] + y;
            } else {
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    y[j] = fmaf(prob[i], y[j], 0.f);
                    n[j] = res[i][j] + y[j];
                }
            }
            if (rc.y) *reinterpret_cast<vec *>(rc.y + at) = y;
            *reinterpret_cast<vec *>(rc.x_next + at) = n;
        } else {
            *reinterpret_cast<vec *>(out + (size_t)(ci.row0 + row) * N + c) = y;
        }
    }
}

template <int V, int MT, int NW>
__global__ __launch_bounds__(NW * 64) void ffn_f32_hidden_kernel(const float *__restrict__ x_perm, const int32_t *__restrict__ src_row,
                                                                 const int32_t *__restrict__ offsets, int E, int d, int f,
                                                                 const char *__restrict__ w_base, size_t w_stride, int slot_by_rank,
                                                                 int n_slots, const unsigned long long *__restrict__ table,
                                                                 float *__restrict__ h) {
    const ChunkInfo ci = find_chunk(offsets, E, 16 * MT, blockIdx.x);
    if (ci.nrows == 0) return;  // uniform over the workgroup
    const char *wexp = table ? reinterpret_cast<const char *>(table[ci.expert])
                             : w_base + (size_t)(slot_by_rank ? ci.slot : ci.expert) * w_stride;
    const bool no_weights = table ? wexp == nullptr : (slot_by_rank && ci.slot >= n_slots);  // no slot: rows are zeroed
    f32_tile<V, MT, NW, true>(x_perm, src_row, reinterpret_cast<const float *>(wexp), h, ci, d, f, no_weights);
}

template <int V, int MT, int NW, typename... Combine>
__global__ __launch_bounds__(NW * 64) void ffn_f32_out_kernel(const float *__restrict__ h, const int32_t *__restrict__ offsets, int E,
                                                              int d, int f, const char *__restrict__ w_base, size_t w_stride,
                                                              int slot_by_rank, int n_slots,
                                                              const unsigned long long *__restrict__ table, float *__restrict__ y_perm,
                                                              const int32_t *__restrict__ tokens, Combine... combine) {
    const ChunkInfo ci = find_chunk(offsets, E, 16 * MT, blockIdx.x);
    if (ci.nrows == 0) return;  // uniform over the workgroup
    const char *wexp = table ? reinterpret_cast<const char *>(table[ci.expert])
                             : w_base + (size_t)(slot_by_rank ? ci.slot : ci.expert) * w_stride;
    const bool no_weights = table ? wexp == nullptr : (slot_by_rank && ci.slot >= n_slots);
    f32_tile<V, MT, NW, false>(h, nullptr, reinterpret_cast<const float *>(wexp) + (size_t)d * f, y_perm, ci, f, d, no_weights, tokens, combine...);
}

// Any other float32 shape (d_model or d_ff not a multiple of 4: rows cannot be read 16 bytes at a time).  One workgroup per
// (row = blockIdx.x, 256 output columns = blockIdx.y); the row's expert and slot are found once per workgroup.
__device__ inline void find_row_expert(const int32_t *offsets, int E, int row, int *expert, int *slot) {
    int e = 0, s = -1;
    for (int i = 0; i < E; ++i) {
        const int lo = offsets[i], hi = offsets[i + 1];
        if (hi > lo) ++s;
        if (row >= lo && row < hi) {
            e = i;
            break;
        }
    }
    *expert = e;
    *slot = s < 0 ? 0 : s;
}

__global__ __launch_bounds__(256) void ffn_f32_hidden_scalar_kernel(const float *__restrict__ x_perm,
                                                              const int32_t *__restrict__ offsets, int E, int d, int f,
                                                              const char *__restrict__ w_base, size_t w_stride,
                                                              int slot_by_rank, int n_slots,
                                                              const unsigned long long *__restrict__ table,
                                                              float *__restrict__ h) {
    __shared__ int s_e, s_s;
    const int row = blockIdx.x;
    if (threadIdx.x == 0) find_row_expert(offsets, E, row, &s_e, &s_s);
    __syncthreads();
    const float *w1 = table ? reinterpret_cast<const float *>(table[s_e])
                            : reinterpret_cast<const float *>(w_base + (size_t)(slot_by_rank ? s_s : s_e) * w_stride);
    const int j = blockIdx.y * 256 + threadIdx.x;
    if (j >= f) return;
    if (table ? w1 == nullptr : (slot_by_rank && s_s >= n_slots)) {  // expert did not get a slot
        h[(size_t)row * f + j] = 0.f;
        return;
    }
    const float *xr = x_perm + (size_t)row * d;
    float acc = 0.f;
    for (int i = 0; i < d; ++i) acc = fmaf(xr[i], w1[(size_t)i * f + j], acc);
    h[(size_t)row * f + j] = fmaxf(acc, 0.f);
}

__global__ __launch_bounds__(256) void ffn_f32_out_scalar_kernel(const float *__restrict__ h, const int32_t *__restrict__ offsets,
                                                           int E, int d, int f, const char *__restrict__ w_base,
                                                           size_t w_stride, int slot_by_rank, int n_slots,
                                                           const unsigned long long *__restrict__ table,
                                                           float *__restrict__ y_perm) {
    __shared__ int s_e, s_s;
    const int row = blockIdx.x;
    if (threadIdx.x == 0) find_row_expert(offsets, E, row, &s_e, &s_s);
    __syncthreads();
    const float *wb = table ? reinterpret_cast<const float *>(table[s_e])
                            : reinterpret_cast<const float *>(w_base + (size_t)(slot_by_rank ? s_s : s_e) * w_stride);
    const float *w2 = wb + (size_t)d * f;
    const int c = blockIdx.y * 256 + threadIdx.x;
    if (c >= d) return;
    if (table ? wb == nullptr : (slot_by_rank && s_s >= n_slots)) {
        y_perm[(size_t)row * d + c] = 0.f;
        return;
    }
    const float *hr = h + (size_t)row * f;
    float acc = 0.f;
    for (int j = 0; j < f; ++j) acc = fmaf(hr[j], w2[(size_t)j * d + c], acc);
    y_perm[(size_t)row * d + c] = acc;
}

// ------------------------------------------------------------------------------------------
static int smallest_divisor_at_least(int n, int want) {
    for (int p = std::max(1, want); p <= n; ++p)
        if (n % p == 0) return p;
    return n;
}

// Geometry of the fused kernel for n_rows rows, from the shape of the launch alone.  slices: d_ff ranges the caller needs (0: the plan's choice).
FfnPlan plan_ffn(const pgmoe_config &c, int n_rows, int slices) {
    FfnPlan p;
    const int E = c.n_experts;
    const int kt = c.d_model / 32;
    const int active = std::max(1, std::min(E, n_rows));  // upper bound of the distinct experts
    const int mean_rows = (n_rows + E - 1) / E;
    // rows per chunk: 16 for decode-sized batches, up to 64 when experts see tens of rows
    int mt = mean_rows <= 4 ? 1 : (mean_rows <= 20 ? 2 : 4);
    // wavefronts per workgroup: 2 (32-column sub-slabs) when there are too few experts to fill
    // the chip otherwise, 8 for the 64-row chunks (halves the accumulators per wavefront)
    int nw = 4;
    if (mt == 1 && active * (c.d_ff / 64) < 256 && (kt == 24 || kt == 32)) nw = 2;
    if (mt == 4 && (kt == 24 || kt == 32) && c.d_ff % (128 * std::max(1, slices)) == 0) nw = 8;
    if (mt == 4 && nw == 4 && kt > 24) mt = 2;
    if (mt == 2 && kt > 32) mt = 1;
    p.mt = mt;
    p.nw = nw;
    p.max_chunks = active + n_rows / (16 * mt);
    const int sub = 16 * nw;
    const int nsub = c.d_ff / sub;
    // partial sums: aim at >= 768 workgroups, but keep the float32 partial traffic
    // (write + read = 8 bytes per element per partial) below ~6 % of the weight bytes
    int want = (768 + active - 1) / active;
    const double traffic_cap = 0.06 * (double)active * c.d_ff / (2.0 * n_rows);
    want = std::max(1, std::min(want, (int)traffic_cap));
    p.n_partial = smallest_divisor_at_least(nsub, std::min(want, nsub));
    if (n_rows > 4096 && p.n_partial > 16) {  // what ffn_workspace_bytes sets aside for launches this large
        p.n_partial = 16;
        while (nsub % p.n_partial) --p.n_partial;
    }
    if (slices) p.n_partial = slices;
    p.f_range = c.d_ff / p.n_partial;
    return p;
}

// Instantiations of ffn_fused_kernel that are built: X(MT, KT, NW, D) = 16*MT rows per chunk,
// d_model = 32*KT, NW wavefronts, prefetch ring of D tiles.  plan_ffn only ever picks from this
// list for a d_model that appears in it (pgmoe_create refuses any other d_model for bf16).
#define PG_FUSED_CASES(X)                                                                                   \
    X(1, 2, 4, 4) X(1, 4, 4, 8) X(1, 8, 4, 16) X(1, 16, 4, 16) X(1, 24, 4, 16) X(1, 32, 4, 16) X(1, 64, 4, 16) \
    X(1, 24, 2, 16) X(1, 32, 2, 16)                                                                         \
    X(2, 2, 4, 4) X(2, 4, 4, 8) X(2, 8, 4, 8) X(2, 16, 4, 16) X(2, 24, 4, 16) X(2, 32, 4, 8)              \
    X(4, 2, 4, 4) X(4, 4, 4, 8) X(4, 8, 4, 8) X(4, 16, 4, 8) X(4, 24, 4, 8) X(4, 24, 8, 2) X(4, 32, 8, 4)

static bool fused_case_built(int mt, int kt, int nw) {
#define X(MT_, KT_, NW_, D_) \
    if (mt == MT_ && kt == KT_ && nw == NW_) return true;
    PG_FUSED_CASES(X)
#undef X
    return false;
}

// Every d_model of the list has the 16-row, four-wavefront instantiation; what else plan_ffn may
// pick for it is in the list too (checked shape by shape by the host-side tests).
bool ffn_supports_d_model(int d_model) { return d_model % 32 == 0 && fused_case_built(1, d_model / 32, 4); }

// The decode-sized kernel serves launches of 16-row chunks split into one partial per
// 32-column sub-slab (what plan_ffn picks when only a few experts are active).
static bool uses_decode_kernel(const pgmoe_config &c, const FfnPlan &p) {
    const int kt = c.d_model / 32;
    return p.mt == 1 && p.nw == 2 && p.n_partial == c.d_ff / 32 && (kt == 24 || kt == 32);
}

bool ffn_launch_is_decode_sized(const pgmoe_config &c, int n_rows) {
    return c.dtype == PGMOE_BF16 && n_rows > 0 && !uses_gemm_kernels(c, n_rows) && uses_decode_kernel(c, plan_ffn(c, n_rows));
}

const char *ffn_kernel_name(const pgmoe_config &c, int n_rows) {
    if (c.dtype == PGMOE_F32)
        return ffn_f32_reads_rows_in_place(c) ? "ffn_f32_hidden_kernel+ffn_f32_out_kernel" : "ffn_f32_hidden_scalar_kernel+ffn_f32_out_scalar_kernel";
    if (uses_gemm_kernels(c, n_rows)) return "ffn_gemm_pack_rows_kernel+ffn_gemm_tile_kernel";
    const FfnPlan p = plan_ffn(c, n_rows);
    if (uses_decode_kernel(c, p)) return "ffn_decode_kernel";
    return fused_case_built(p.mt, c.d_model / 32, p.nw) && c.d_ff % (16 * p.nw) == 0 ? "ffn_fused_kernel" : nullptr;
}

size_t ffn_workspace_bytes(const pgmoe_config &c) {
    const int64_t max_rows = (int64_t)c.max_tokens * c.top_k;
    if (c.dtype == PGMOE_F32) return (size_t)max_rows * c.d_ff * 4;
    // worst case over every geometry plan_ffn can pick: one partial per 32-column sub-slab
    const size_t worst = (size_t)(c.d_ff / 32) * std::min<int64_t>(max_rows, 4096) * c.d_model * 4;
    const size_t big = (size_t)16 * max_rows * c.d_model * 4;
    const size_t gemm = ffn_gemm_workspace_bytes(c);  // two-GEMM path
    return ((std::max(std::max(worst, big), gemm) + 255) & ~(size_t)255);
}

size_t ffn_partial_bytes(const pgmoe_config &c, int n_rows) {
    const FfnPlan p = plan_ffn(c, n_rows);
    return uses_decode_kernel(c, p) || p.n_partial > 1 ? (size_t)p.n_partial * n_rows * c.d_model * 4 : 0;
}

// Scratch by which pgmoe_expert_ffn_static admits a launch of n_rows rows.
size_t ffn_launch_workspace_bytes(const pgmoe_config &c, int n_rows) {
    if (n_rows <= 0) return 0;
    if (c.dtype == PGMOE_F32) return (size_t)n_rows * c.d_ff * 4;
    return uses_gemm_kernels(c, n_rows) ? ffn_gemm_launch_bytes(c, n_rows) : ffn_partial_bytes(c, n_rows);
}

// Scratch of pgmoe_expert_ffn_static(): part of the library's device image, so no call ever
// allocates it; every GPU the library runs on holds its own copy at its own address.  In host
// code the array's name is only a handle for hipGetSymbolAddress: the address kernels and
// copies take is resolved once per device, here, and kept.
static __device__ __align__(256) unsigned char scratch[PGMOE_STATIC_SCRATCH_BYTES];
static void *g_scratch_ptr[64] = {};
static std::mutex g_scratch_mutex;  // contexts may be created from several host threads

int resolve_static_scratch(pgmoe_ctx *ctx) {  // the context's device is current (pgmoe_create)
    const int dev = ctx->device;
    if (dev < 0 || dev >= (int)(sizeof g_scratch_ptr / sizeof g_scratch_ptr[0]))
        return fail(ctx, PGMOE_EINVAL, "pgmoe_create: device ordinal %d outside 0..63", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        PG_HIP(ctx, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || !aligned(ptr, 256)) return fail(ctx, PGMOE_EHIP, "pgmoe_create: the static scratch buffer resolved to %p", ptr);
        g_scratch_ptr[dev] = ptr;
    }
    ctx->static_scratch = g_scratch_ptr[dev];
    return PGMOE_OK;
}

int ffn_timing_slot(pgmoe_ctx *ctx) {
    if (!ctx->tim_on || ctx->tim_n >= ctx->tim_cap) return -1;
    return ctx->tim_n++;
}

int launch_ffn_reduce(pgmoe_ctx *ctx, const float *partial, int P, int n_rows, void *y_perm, hipStream_t s) {
    const int d = ctx->cfg.d_model;
    const size_t total4 = (size_t)n_rows * d / 4;
    const int pl = reduce_lanes(P);  // p-lanes per column: 256 / pl float4 columns per workgroup
    const dim3 grid((unsigned)((total4 + 256 / pl - 1) / (256 / pl)));
    if (pl == 1) hipLaunchKernelGGL(ffn_reduce_kernel<1>, grid, dim3(256), 0, s, partial, P, n_rows, d, (__bf16 *)y_perm);
    else if (pl == 4) hipLaunchKernelGGL(ffn_reduce_kernel<4>, grid, dim3(256), 0, s, partial, P, n_rows, d, (__bf16 *)y_perm);
    else hipLaunchKernelGGL(ffn_reduce_kernel<16>, grid, dim3(256), 0, s, partial, P, n_rows, d, (__bf16 *)y_perm);
    PG_HIP(ctx, hipGetLastError());
    return PGMOE_OK;
}

// The gate a launch is asked to carry, as the kernels take it (x == nullptr: it cannot), and what becomes of it.
static CarriedGate carry_gate(pgmoe_ctx *ctx, const FusedGate *gate, bool decode_kernel, bool partials_kept, GateCarried *done) {
    const pgmoe_config &c = ctx->cfg;
    CarriedGate g = {};
    if (!gate) return g;
    const bool small = decode_kernel && gate_small_applies(c, gate->T);
    // the second half goes with the combine that adds the partial sums
    if (!small && !(partials_kept && ctx->gate_planes && gate_planes_apply(c, gate->T))) return g;
    const bool route = small || gate_mfma_routes(c, gate->T);
    g = CarriedGate{(const __bf16 *)gate->x, (const __bf16 *)gate->w, gate->bias, gate->T, c.d_model, c.top_k, c.n_experts, gate->idx,
                    gate->prob, ctx->dev_flags, route ? gate->row_of : nullptr, route ? gate->offsets : nullptr,
                    route ? gate->src_row : nullptr, small ? nullptr : ctx->gate_planes};
    *done = small ? GATE_ROUTED : GATE_STARTED;
    return g;
}

template <int MT, int KT, int NW, int D>
static int launch_fused(pgmoe_ctx *ctx, const FfnPlan &p, const char *w_base, size_t w_stride, bool slot_by_rank, int n_slots,
                        const void *x_perm, const int32_t *offsets, int n_rows, void *y_perm, void *workspace,
                        hipStream_t s, int *keep_partials, const unsigned long long *table, const int32_t *src_row, const FusedGate *gate,
                        GateCarried *gate_done) {
    const pgmoe_config &c = ctx->cfg;
    constexpr bool CARRIES = NW == 4 && MT <= 2;  // decode-sized chunks
    CarriedGate cg = {};
    if (CARRIES) cg = carry_gate(ctx, gate, false, keep_partials && p.n_partial > 1, gate_done);
    // The dispatcher fills a CU before the next one, so a kernel of which two find room on a CU leaves CUs idle in a launch that has a workgroup for each. Two
    // kernels take more LDS than they use in launches of 256 workgroups at most, the even case that the shape says; each alone was what their registers once made it:
    // 128 experts of 512 x 2048, 30 rows each 123 us with two, 101 alone, 24 uneven rows 123 and 100 (30 skewed rows, which are more workgroups: 126 and 138);
    // 32 of 768 x 3072, 12 and 16 uneven rows 75 and 64, 88 and 66.  Not the others: 16 of 1024 x 4096, 9 rows each 67 and 73, 16 of 256 x 1024, 3 rows 8.9 and 10.3.
    constexpr size_t needed = (size_t)MT * KT * 1024 + 2u * MT * (16 * NW / 32) * 1024, half = 82 * 1024;
    constexpr bool crowded = (MT == 2 && KT == 24) || (MT == 4 && KT == 16);
    const int gate_wgs = cg.x ? 2 * ((gate->T + GM_TOK - 1) / GM_TOK) : 0, active = std::max(1, std::min(c.n_experts, n_rows));
    const bool alone = crowded && std::max((double)active, 0.5 * active + n_rows / (16.0 * MT)) * p.n_partial + gate_wgs <= 256;
    // With a carried gate the 16-row chunks of d_model 512 leave room for three, but two are right for more of the launches (six blocks of 512 x 2048, two / three: 64 experts,
    // 16 tokens 125 / 130 us; 128 experts, 64 tokens 303 / 315, 128 tokens of two experts 548 / 567; 64 skewed experts, 64 tokens 190 / 203). Where
    // between 512 and 768 workgroups come out three are: 64 experts, 64 tokens 273 / 261, 48 experts 253 / 236; the shape alone does not tell.
    const size_t lds = std::max<size_t>(alone ? half : (KT == 16 && cg.x ? 54 * 1024 : 0), needed);
    float *partial = p.n_partial > 1 ? (float *)workspace : nullptr;
    if (partial && (size_t)p.n_partial * n_rows * c.d_model * 4 > ffn_workspace_bytes(c))
        return fail(ctx, PGMOE_EINVAL, "pgmoe_expert_ffn: %d partial sums of %d rows do not fit the workspace", p.n_partial, n_rows);
    const int tslot = ffn_timing_slot(ctx);
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_begin[tslot], s));
    auto launch = [&](auto kern, int rows, auto... carried) {
        // the limit is raised once, so for the most that any launch of the kernel takes
        if (int rc = allow_dynamic_lds(ctx, reinterpret_cast<const void *>(kern), crowded ? std::max(lds, half) : lds)) return rc;
        hipLaunchKernelGGL(kern, dim3(p.max_chunks, rows), dim3(NW * 64), lds, s, (const __bf16 *)x_perm, offsets, c.n_experts, c.d_ff,
                           p.f_range, w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, partial, (__bf16 *)y_perm, n_rows, src_row,
                           carried...);
        return (int)PGMOE_OK;
    };
    int rc;
    if constexpr (CARRIES) {
        rc = cg.x ? launch(ffn_fused_kernel<MT, KT, NW, D, CarriedGate>, p.n_partial + 1, cg) : launch(ffn_fused_kernel<MT, KT, NW, D>, p.n_partial);
    } else {
        rc = launch(ffn_fused_kernel<MT, KT, NW, D>, p.n_partial);
    }
    if (rc) return rc;
    PG_HIP(ctx, hipGetLastError());
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_end[tslot], s));
    if (keep_partials) {
        *keep_partials = partial ? p.n_partial : 0;
        return PGMOE_OK;
    }
    if (partial) return launch_ffn_reduce(ctx, partial, p.n_partial, n_rows, y_perm, s);
    return PGMOE_OK;
}

bool ffn_f32_reads_rows_in_place(const pgmoe_config &c) { return c.dtype == PGMOE_F32 && c.d_model % 4 == 0 && c.d_ff % 4 == 0; }

static int launch_ffn_f32(pgmoe_ctx *ctx, const char *w_base, size_t w_stride, bool slot_by_rank, int n_slots, const float *x,
                          const int32_t *offsets, int n_rows, float *y_perm, float *h, hipStream_t s,
                          const unsigned long long *table, const int32_t *src_row, const RowCombine *combine) {
    const pgmoe_config &c = ctx->cfg;
    const int tslot = ffn_timing_slot(ctx);
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_begin[tslot], s));
    if (ffn_f32_reads_rows_in_place(c)) {
        // rows per workgroup by the rows an expert has (8 experts of 768 x 3072 with 12.5 rows each: both products 46 us with 16-row
        // chunks, 63 with 32); columns per lane: four (wide pieces of a weight row, the least share of the activations in what
        // a CU has in flight) where 96 workgroups come out all the same and the experts see eight rows or more.  Measured over 315 launches
        // (d_model 64 .. 2048, 1 .. 64 experts, 1 .. 60 rows each), both products with four / with two columns: at 96 workgroups 45 / 51 us (8 experts of
        // 768, 12 rows), 33 / 37 (12 of 512), 56 / 61 (6 of 1024) and 104 / 134, 73 / 95, 141 / 165 with 60 rows; at 72 (6 of 768) 41 / 35 and 99 / 82;
        // with 4 rows 44 / 36 at 96.  The rule is within 2 % of the best choice on the geometric mean, at worst 1.37 times it (4 of 768, 12 rows).
        const int active = std::max(1, std::min(c.n_experts, n_rows)), mean = (n_rows + active - 1) / active;
        const int mt = mean <= 16 ? 1 : (mean <= 32 ? 2 : 4);
        const int chunks = active + n_rows / (16 * mt);
        auto cols = [&](int N) { return active * ((N + 63) / 64) >= (mean >= 8 ? 96 : 256) ? 4 : (active * ((N + 31) / 32) >= 128 ? 2 : 1); };
        // twice the wavefronts per workgroup where half the CUs have one at most and a wavefront still keeps its four blocks in flight: 8 experts of
        // 768 x 3072 with 12 rows each, steps from HBM 46.8 -> 43.8 us. With one for every CU they gain or lose little in a launch by itself and lose where
        // those of several streams meet (eight / sixteen, three streams: 4 experts of 1024 x 4096, 8 rows each 31.9 / 34.0 us, one row 27.5 / 31.1; 8 of
        // 2048 x 1024, one row 23.5 / 29.3; by themselves 45.8 / 48.4, 38.0 / 37.8 and 31.0 / 33.0).
        auto wide = [&](int N, int K) { return active * ((N + 63) / 64) <= 128 && K >= 16 * 16 * F32_DEPTH; };
        // A workgroup of 64 rows and 16 columns leaves room for a second one on its CU, and the dispatcher fills a CU before the next: launches with a workgroup
        // for each CU take more LDS than half of one (4 experts of 768 x 3072, 40 rows each: 72.6 us with two on a CU, 57.2 alone; one of them, three
        // streams 20.4 and 15.1; but 2 of 256 x 512, 1000 rows each, which are 1000 workgroups, 30.2 and 37.4).
        const double full_chunks = active == 1 ? (n_rows + 16 * mt - 1) / (16 * mt) : std::max((double)active, 0.5 * active + n_rows / (16.0 * mt));
        auto spare_lds = [&](int v, int rows16, int N) -> size_t { return v == 1 && rows16 == 4 && full_chunks * ((N + 15) / 16) <= 256 ? F32_ALONE : 0; };
#define PG_F32_LAUNCH(N_, V_, MT_, NW_, KERN_, ...)                                                                             \
    do {                                                                                                                        \
        auto kern_ = KERN_;                                                                                                     \
        const size_t lds_ = spare_lds(V_, MT_, N_);                                                                             \
        if (int rc_ = allow_dynamic_lds(ctx, reinterpret_cast<const void *>(kern_), lds_)) return rc_;                          \
        hipLaunchKernelGGL(kern_, dim3(chunks, (N_ + 16 * V_ - 1) / (16 * V_)), dim3(NW_ * 64), lds_, s, __VA_ARGS__);          \
    } while (0)
#define PG_F32_HIDDEN(V_, MT_, NW_)                                                                                             \
    PG_F32_LAUNCH(c.d_ff, V_, MT_, NW_, (ffn_f32_hidden_kernel<V_, MT_, NW_>), x, src_row, offsets, c.n_experts, c.d_model, c.d_ff, w_base, \
                  w_stride, slot_by_rank ? 1 : 0, n_slots, table, h)
#define PG_F32_OUT_ARGS h, offsets, c.n_experts, c.d_model, c.d_ff, w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, y_perm, src_row
#define PG_F32_OUT(V_, MT_, NW_)                                                                                                \
    do {                                                                                                                        \
        if (combine) PG_F32_LAUNCH(c.d_model, V_, MT_, NW_, (ffn_f32_out_kernel<V_, MT_, NW_, RowCombine>), PG_F32_OUT_ARGS, *combine); \
        else PG_F32_LAUNCH(c.d_model, V_, MT_, NW_, (ffn_f32_out_kernel<V_, MT_, NW_>), PG_F32_OUT_ARGS);                       \
    } while (0)
#define PG_F32(KERN_, N_, K_)                                                                                                    \
    do {                                                                                                                       \
        const int v_ = cols(N_);                                                                                               \
        if (mt == 1) {                                                                                                         \
            if (v_ == 4 && wide(N_, K_)) KERN_(4, 1, 16);                                                                      \
            else if (v_ == 4) KERN_(4, 1, 8);                                                                                  \
            else if (v_ == 2) KERN_(2, 1, 8);                                                                                  \
            else KERN_(1, 1, 8);                                                                                               \
        } else if (mt == 2) {                                                                                                  \
            if (v_ == 4) KERN_(4, 2, 8);                                                                                       \
            else if (v_ == 2) KERN_(2, 2, 8);                                                                                  \
            else KERN_(1, 2, 8);                                                                                               \
        } else {                                                                                                               \
            if (v_ == 4) KERN_(4, 4, 4);                                                                                       \
            else if (v_ == 2) KERN_(2, 4, 8);                                                                                  \
            else KERN_(1, 4, 8);                                                                                               \
        }                                                                                                                      \
        PG_HIP(ctx, hipGetLastError());                                                                                        \
    } while (0)
        PG_F32(PG_F32_HIDDEN, c.d_ff, c.d_model);
        PG_F32(PG_F32_OUT, c.d_model, c.d_ff);
#undef PG_F32
#undef PG_F32_OUT
#undef PG_F32_OUT_ARGS
#undef PG_F32_LAUNCH
#undef PG_F32_HIDDEN
    } else {
        hipLaunchKernelGGL(ffn_f32_hidden_scalar_kernel, dim3(n_rows, (c.d_ff + 255) / 256), dim3(256), 0, s, x, offsets, c.n_experts,
                           c.d_model, c.d_ff, w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, h);
        PG_HIP(ctx, hipGetLastError());
        hipLaunchKernelGGL(ffn_f32_out_scalar_kernel, dim3(n_rows, (c.d_model + 255) / 256), dim3(256), 0, s, h, offsets, c.n_experts,
                           c.d_model, c.d_ff, w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, y_perm);
        PG_HIP(ctx, hipGetLastError());
    }
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_end[tslot], s));
    return PGMOE_OK;
}

int launch_ffn(pgmoe_ctx *ctx, const char *w_base, size_t w_stride, bool slot_by_rank, int n_slots, const void *x_perm,
               const int32_t *offsets, int n_rows, void *y_perm, void *workspace, hipStream_t s, int *keep_partials,
               const unsigned long long *table, const int32_t *src_row, const FusedGate *gate, GateCarried *gate_done,
               const RowCombine *combine) {
    const pgmoe_config &c = ctx->cfg;
    if (keep_partials) *keep_partials = 0;
    if (gate_done) *gate_done = GATE_LEFT;
    if (n_rows == 0) return PGMOE_OK;
    if (c.dtype == PGMOE_F32)
        return launch_ffn_f32(ctx, w_base, w_stride, slot_by_rank, n_slots, (const float *)x_perm, offsets, n_rows, (float *)y_perm,
                              (float *)workspace, s, table, src_row, combine);
    int slices = 0;
    if (uses_gemm_kernels(c, n_rows)) {
        const size_t bytes = workspace == ctx->static_scratch ? PGMOE_STATIC_SCRATCH_BYTES : ffn_workspace_bytes(c);
        slices = gemm_slices_for_fused(c, n_rows, bytes);
        if (!slices)
            return launch_ffn_gemm(ctx, w_base, w_stride, slot_by_rank, n_slots, x_perm, offsets, n_rows, y_perm, workspace, bytes, s,
                                   keep_partials, table, src_row);
    }
    const FfnPlan p = plan_ffn(c, n_rows, slices);
    const int kt = c.d_model / 32;
    if (uses_decode_kernel(c, p)) {
        // a few experts with at most 16 rows each, one partial per 32-column sub-slab
        float *partial = (float *)workspace;
        if ((size_t)p.n_partial * n_rows * c.d_model * 4 > ffn_workspace_bytes(c))
            return fail(ctx, PGMOE_EINVAL, "pgmoe_expert_ffn: %d partial sums of %d rows do not fit the workspace", p.n_partial, n_rows);
        const int tslot = ffn_timing_slot(ctx);
        if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_begin[tslot], s));
        // one more row of workgroups for the pre-gate this launch carries
        const CarriedGate dg = carry_gate(ctx, gate, true, keep_partials != nullptr, gate_done);
        const dim3 grid(p.max_chunks, p.n_partial + (dg.x ? 1 : 0));
        const size_t lds = decode_lds_bytes(kt);
#define PG_DECODE(KT_, GATE_)                                                                                                    \
    hipLaunchKernelGGL((ffn_decode_kernel<KT_, GATE_>), grid, dim3(256), lds, s, (const __bf16 *)x_perm, offsets, c.n_experts, c.d_ff, \
                       w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, partial, n_rows, src_row, dg)
        const DecodeGateKind kind = !dg.x ? DECODE_NO_GATE : (dg.planes ? DECODE_GATE_PLANES : (c.n_experts == 8 ? DECODE_SMALL_GATE_8 : DECODE_SMALL_GATE_16));
        if (kt == 24) {
            if (kind == DECODE_NO_GATE) PG_DECODE(24, DECODE_NO_GATE);
            else if (kind == DECODE_SMALL_GATE_8) PG_DECODE(24, DECODE_SMALL_GATE_8);
            else if (kind == DECODE_SMALL_GATE_16) PG_DECODE(24, DECODE_SMALL_GATE_16);
            else PG_DECODE(24, DECODE_GATE_PLANES);
        } else {
            if (kind == DECODE_NO_GATE) PG_DECODE(32, DECODE_NO_GATE);
            else if (kind == DECODE_SMALL_GATE_8) PG_DECODE(32, DECODE_SMALL_GATE_8);
            else if (kind == DECODE_SMALL_GATE_16) PG_DECODE(32, DECODE_SMALL_GATE_16);
            else PG_DECODE(32, DECODE_GATE_PLANES);
        }
#undef PG_DECODE
        PG_HIP(ctx, hipGetLastError());
        if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_end[tslot], s));
        if (keep_partials) {
            *keep_partials = p.n_partial;
            return PGMOE_OK;
        }
        return launch_ffn_reduce(ctx, partial, p.n_partial, n_rows, y_perm, s);
    }
    if (c.d_ff % (16 * p.nw)) return fail(ctx, PGMOE_EINVAL, "pgmoe_expert_ffn: d_ff=%d is not a multiple of the %d-column sub-slab", c.d_ff, 16 * p.nw);
#define X(MT_, KT_, NW_, D_)                                                                                                  \
    if (p.mt == MT_ && kt == KT_ && p.nw == NW_)                                                                              \
        return launch_fused<MT_, KT_, NW_, D_>(ctx, p, w_base, w_stride, slot_by_rank, n_slots, x_perm, offsets, n_rows, y_perm, \
                                               workspace, s, keep_partials, table, src_row, gate, gate_done);
    PG_FUSED_CASES(X)
#undef X
    return fail(ctx, PGMOE_EINVAL, "pgmoe_expert_ffn: no bf16 kernel built for d_model=%d with %d-row chunks and %d wavefronts", c.d_model, 16 * p.mt, p.nw);
}

}  // namespace pgmoe
