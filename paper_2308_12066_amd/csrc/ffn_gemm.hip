// Expert execution for launches with many rows per expert (Sec. II-B: every activated expert, a
// dense FFN, processes the tokens routed to it): the two products as two tiled GEMMs.
#include <climits>
#include <cmath>
#include <type_traits>

#include "ffn_common.h"

namespace pgmoe {

// ------------------------------------------------------------------------------------------
// With many rows per expert the weights must be reused across many rows, so the two
// products run as two tiled GEMMs with the hidden activation (bf16) parked in the workspace
// between them, after a small kernel that gathers the rows and packs them as operand tiles:
//   ffn_gemm_pack_rows_kernel   Xp = rows of x, chunk by chunk, as 1 KiB operand tiles
//   ffn_gemm_tile_kernel<UP>    H[rows, f] = ReLU(Xp . W1)                           K = d
//   ffn_gemm_tile_kernel<DOWN>  y_perm[rows, d] = H . W2, or with K slices
//                               partial[s][rows, d] = H[rows, K-slice s] . W2        K = f / n_split
// A workgroup of eight wavefronts takes up to 320 rows of one expert and 256 (or 128) output columns and loads
// BOTH operands straight from memory into LDS in operand order (every operand tile is 1 KiB contiguous: the
// packed rows, the packed hidden activation the up-projection writes, and the pre-tiled weights).
//
// What bounds it and why the tile looks like this (measured on one MI355X):
//  * large launches (128 experts of 1024 x 4096, 32768 rows): the stream of weights, 1.07 GB a product, beside the products it feeds.
//    289 us up and 314 down, 0.95 and 0.88 PFLOP/s, at 5.0 and 4.6 TB/s read and written; what is read past L2 is 1.02 and 1.03 times the operands,
//    so no column block fetches its chunk's rows again; the matrix cores are busy 46 and 40 % of the time, at 2.0 to 2.1 GHz (counters of passes
//    that are waited for; the loop below took 329 and 360 us where the one before it took 358 and 397).  Hence as many rows per weight tile as the
//    registers hold (320: 160 accumulator registers), no second chunk for an expert that has a few rows more than a power of two, and neither
//    a request nor a product for a row tile the chunk lacks;
//  * 8 experts of 768 x 3072, 4096 rows: 26.5 us up, 29.7 down with the weights in the last-level cache (30.5 and 34.6 before; the vendor GEMM
//    library: 27 + 41).  A 32-k stage of 16 row tiles takes 0.62 us (0.76), 1170 clocks for 1024 of products: with a batch of LDS reads and
//    loads behind every barrier it took 1540.  512 rows per expert are two chunks each, 192 workgroups; chunks of at most
//    256 rows and 192-column blocks were no better;
//  * few rows per expert: the stream of weights.  A chunk of one or two row tiles gets eight stages instead of four: a stage 0.46 -> 0.38 us;
//  * matrix-core accumulators must be ordinary vector registers (build flag): with the accumulator-register form the
//    register allocator copies accumulators about inside the k loop and every copy waits for the product before it;
//  * one result straight in bf16 where no K slices are needed: the float32 partials of one slice cost the combine 14 us
//    of 59 on the large launch.
constexpr int GEMM_ROWS = 320;           // most rows of a chunk
constexpr int GEMM_RT = GEMM_ROWS / 16;  // 16-row tiles of the largest chunk
constexpr int GEMM_RING = 144 * 1024;    // bytes of LDS both operands pass through
// A chunk's ring has the row tiles of the first of these that holds it: small chunks get more stages, not empty places.
constexpr int GEMM_RING_TILES[] = {2, 8, GEMM_RT};

// The chunks of an expert are of equal size (its rows dealt to as few chunks as hold them, in whole
// 16-row tiles): 330 rows are two chunks of 176 and 154 rows, not 320 and 10, so no workgroup streams a whole
// slab of weights for a handful of rows.  tile0 counts the 16-row tiles of all chunks before this one: the
// packed rows and the packed hidden activation are laid out by it.
struct GemmChunk {
    int expert, slot, row0, nrows, tile0;  // tile0 counts from the launch's first tile; nrows == 0: there is no such chunk
};
struct GemmScan {  // per lane: four experts, lane + 64 * q; everything a lookup needs, from one round of loads
    int lo[4], n[4], k0[4], c[4], c_incl[4], t_incl[4], nz_incl[4];
    int total, active;  // chunks of all experts, experts with chunks (uniform)
};
__device__ inline int gemm_chunks_of(int n) { return (n + GEMM_ROWS - 1) / GEMM_ROWS; }
__device__ inline int gemm_rows_of(int n, int chunks) { return (((n + chunks - 1) / chunks) + 15) & ~15; }
// Chunks whose first tile lies in [tiles_lo, tiles_hi): a launch whose scratch does not hold every row at once works
// through them in several passes.
__device__ inline void gemm_scan(const int32_t *__restrict__ offsets, int E, int tiles_lo, int tiles_hi, GemmScan &s) {
    const int lane = threadIdx.x & 63;
    int hi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s.lo[q] = hi[q] = 0;
        if (q * 64 < E) {  // uniform
            s.lo[q] = offsets[min(q * 64 + lane, E)];
            hi[q] = offsets[min(q * 64 + lane + 1, E)];
        }
    }
    int c = 0, t = 0, z = 0, a = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = s.n[q] = hi[q] - s.lo[q];
        s.k0[q] = s.c[q] = s.c_incl[q] = s.t_incl[q] = s.nz_incl[q] = 0;
        if (q * 64 < E) {
            s.t_incl[q] = t + wave_incl_scan((n + 15) >> 4);
            s.nz_incl[q] = z + wave_incl_scan(n > 0 ? 1 : 0);
            s.c[q] = gemm_chunks_of(n);
            if (tiles_hi < INT_MAX) {  // uniform: only these chunks of the expert, from the k0-th on
                const int rt = max(1, gemm_rows_of(n, max(1, s.c[q])) >> 4), first = s.t_incl[q] - ((n + 15) >> 4);
                const int from = min(s.c[q], max(0, (tiles_lo - first + rt - 1) / rt));
                const int to = min(s.c[q], max(0, (tiles_hi - first + rt - 1) / rt));
                s.k0[q] = from;
                s.c[q] = to - from;
            }
            s.c_incl[q] = c + wave_incl_scan(s.c[q]);
            a += __popcll(__ballot(s.c[q] > 0));
            c = __builtin_amdgcn_readlane(s.c_incl[q], 63);
            t = __builtin_amdgcn_readlane(s.t_incl[q], 63);
            z = __builtin_amdgcn_readlane(s.nz_incl[q], 63);
        }
    }
    s.total = c;
    s.active = a;
}
__device__ inline GemmChunk gemm_find(const GemmScan &s, int E, int tiles_lo, int chunk) {
    GemmChunk ci = {0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q * 64 >= E) break;
        const int c_excl = s.c_incl[q] - s.c[q];
        const unsigned long long hit = __ballot(chunk >= c_excl && chunk < s.c_incl[q]);
        if (hit) {
            const int src = __ffsll((long long)hit) - 1;  // uniform: read that lane's values directly
            const int n = __builtin_amdgcn_readlane(s.n[q], src);
            const int k = chunk - __builtin_amdgcn_readlane(c_excl, src) + __builtin_amdgcn_readlane(s.k0[q], src);
            const int rows = gemm_rows_of(n, gemm_chunks_of(n));
            ci.expert = q * 64 + src;
            ci.slot = __builtin_amdgcn_readlane(s.nz_incl[q], src) - 1;
            ci.row0 = __builtin_amdgcn_readlane(s.lo[q], src) + k * rows;
            ci.nrows = min(rows, n - k * rows);
            ci.tile0 = __builtin_amdgcn_readlane(s.t_incl[q], src) - ((n + 15) >> 4) + k * (rows >> 4) - tiles_lo;
            return ci;
        }
    }
    return ci;
}

// XCD-aware dealing of the (chunk, column block) items of a GEMM launch.  Workgroups go to the 8
// XCDs round-robin in launch order and every XCD has its own L2.  All column blocks of a chunk go to one XCD (they
// share its rows), and so do G consecutive chunks, G being how many an expert has on average (they share its
// weights); such groups are dealt round-robin, so that the large chunks of a popular expert do not all end up on
// one XCD.  Where the experts have G chunks each on the mean, with nothing over, all of a group take a column block before the next is begun: its weights are then
// read by G workgroups side by side and not G times (16 experts of 2048 x 8192, 512 rows each: 522 -> 493 us a block; 8 of 1024 x 4096, 2048 rows each: 267 -> 263).
// Experts of one and three chunks pass for two each by that, and their groups straddle; it costs as much as it gives (by column block / chunk after chunk: 200 and 900
// rows for 32 experts of 1024 x 4096 310 / 300 us with three streams, 314 / 312 by itself, for 8 of 2048 x 8192 260 / 262 and 322 / 337, 300 rows for fifteen of
// 768 x 3072 and 5420 for one 122 / 124). With a remainder the order was up to 9 % slower.  What is left over is cut into eight equal runs of items.
// The items are the first total * gy workgroups of a launch in this order.
// What a workgroup of the tile kernel needs to know is looked up once, by the kernel that packs the rows, and left as a record per item: with the
// lookup in every workgroup (the prefix sums over the experts, five divisions) every item began a microsecond later: 512 rows for each of 8
// experts of 768 x 3072 71.8 -> 70.2 us a block, 94 for 64 169 -> 166, 128 for 64 of 512 x 2048 115 -> 112.
struct alignas(32) GemmItem {
    const char *w;          // the expert's blob; null: it got no slot, its rows are written as zeros
    int row0, nrows, tile0; // nrows == 0: no item
    int col;                // column block and K slice
};
static_assert(sizeof(GemmItem) == 32, "two of a 64-byte line");
__device__ inline int gemm_launch_order(const GemmScan &s, int chunk, int col, int gy) {
    const int G = s.active > 0 ? (s.total + s.active - 1) / s.active : 1;
    const int full = s.total / (8 * G) * G;  // chunks per XCD dealt in groups
    if (chunk < 8 * full) {
        const int deal = chunk / G, k = chunk - deal * G, xcd = deal & 7, round = deal >> 3;
        const int turn = s.total == G * s.active ? round * G * gy + col * G + k : (round * G + k) * gy + col;
        return turn * 8 + xcd;
    }
    const int rest = (s.total - 8 * full) * gy, run = rest >> 3, longer = rest & 7;  // the first `longer` XCDs get one item more
    int item = (chunk - 8 * full) * gy + col, xcd, turn;
    if (item < longer * (run + 1)) {
        xcd = item / (run + 1);
        turn = item - xcd * (run + 1);
    } else {
        item -= longer * (run + 1);
        xcd = longer + item / run;
        turn = item - (xcd - longer) * run;
    }
    return (full * gy + turn) * 8 + xcd;
}

// The rows of every chunk, gathered through the row -> token map and stored as the 1 KiB
// operand tiles the tile kernel below loads straight into LDS: per chunk [d/32 k-tiles][its row
// tiles][1 KiB], a tile holding 16 rows x 32 features in matrix-core operand order (cell row%16 +
// 16*((feature%32)/8), 8 features per cell): the layout of the packed hidden activation.  Rows
// past the chunk's end are zero.  One workgroup packs PACK_KT k-tiles of one chunk: wavefront w
// packs row tiles w, w + 8, .., a lane reads 16 bytes of a row per row tile and k-tile (64 contiguous bytes
// per row and wavefront) and consecutive lanes write consecutive cells, so whole tiles go out as
// contiguous kilobytes; every load is requested before the first store.
constexpr int PACK_KT = 2;
__global__ __launch_bounds__(512) void ffn_gemm_pack_rows_kernel(
    const __bf16 *__restrict__ x_rows, const int32_t *__restrict__ offsets, int E, int d,
    const int32_t *__restrict__ src_row,  // nullable: grouped row r is row src_row[r] of x_rows
    __bf16 *__restrict__ x_packed, int tiles_lo, int tiles_hi, const char *__restrict__ w_base, size_t w_stride, int slot_by_rank, int n_slots,
    const unsigned long long *__restrict__ table, GemmItem *__restrict__ items, int gy_up, int gy_down) {
    GemmScan scan;
    gemm_scan(offsets, E, tiles_lo, tiles_hi, scan);
    const GemmChunk ci = gemm_find(scan, E, tiles_lo, blockIdx.x);
    if (blockIdx.y == 0) {  // the records of this chunk's items, or of the items that a chunk of the launch at most would have
        const char *w = table ? reinterpret_cast<const char *>(table[ci.expert]) : w_base + (size_t)(slot_by_rank ? ci.slot : ci.expert) * w_stride;
        if (!table && slot_by_rank && ci.slot >= n_slots) w = nullptr;
        for (int i = threadIdx.x; i < gy_up + gy_down; i += 512) {
            const bool up = i < gy_up;
            const int col = up ? i : i - gy_up, gy = up ? gy_up : gy_down;
            const int at = ci.nrows ? gemm_launch_order(scan, blockIdx.x, col, gy) : blockIdx.x * gy + col;
            items[(up ? 0 : (size_t)gridDim.x * gy_up) + at] = GemmItem{w, ci.row0, ci.nrows, ci.tile0, col};
        }
    }
    if (ci.nrows == 0) return;  // uniform over the workgroup
    const int rt = (ci.nrows + 15) >> 4;
    const int kt0 = blockIdx.y * PACK_KT;
    const int cell = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint4 *src = reinterpret_cast<const uint4 *>(x_rows);
    uint4 *dst = reinterpret_cast<uint4 *>(x_packed) + (size_t)ci.tile0 * 16 * (d >> 3);
    const int cells_per_row = d >> 3;
    constexpr int J = (GEMM_RT + 7) / 8;
    size_t from[J];
    bool live[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int row = (wave + 8 * j) * 16 + (cell & 15);
        live[j] = row < ci.nrows;
        const int r = ci.row0 + (live[j] ? row : 0);
        from[j] = (size_t)(src_row ? src_row[r] : r) * cells_per_row + (cell >> 4);
    }
    uint4 v[J][PACK_KT];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int k = 0; k < PACK_KT; ++k) v[j][k] = src[from[j] + (size_t)(kt0 + k) * 4];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int k = 0; k < PACK_KT; ++k)
            if (wave + 8 * j < rt)
                dst[((size_t)(kt0 + k) * rt + wave + 8 * j) * 64 + cell] = live[j] ? v[j][k] : make_uint4(0, 0, 0, 0);
}

// Both operands are loaded straight into LDS (global_load_lds_dwordx4: each
// lane's 16 bytes land at LDS base + 16 * lane, so a 1 KiB operand tile that is contiguous in
// memory arrives in operand order with no register round trip and no staging writes).  A stage
// is one 32-k tile of both operands; NS stages of LDS form a ring.
//
// The loads are issued from inline assembly rather than through the compiler's builtin: the
// compiler cannot tell which stage a later LDS read belongs to and would wait for every load in
// flight before it, which is exactly the prefetch.  Here the kernel counts its own loads (they
// complete in order) and waits with explicit s_waitcnt vmcnt.  M0 (the LDS base of such a load)
// is written inside the statement; nothing else in this kernel keeps a value in M0.  The hardware needs one wait
// state between a scalar write of M0 and a direct-to-LDS load (without it the tile may land at the address of the load
// before); the compiler inserts it behind its own writes only, so the statement carries it.
__device__ inline unsigned lds_address(const void *p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)p;
}
__device__ inline void load_tile_to_lds(const char *src, unsigned lane_off, unsigned lds_tile) {  // src: uniform; lane_off: 16 bytes a lane
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(src), "s"(lds_tile) : "memory", "m0");
}

// What a workgroup of the tile kernel works on (all uniform).
struct GemmTile {
    const char *a;   // the chunk's packed operand tiles of the first k-tile: [n_kt][rt][1 KiB]
    const char *w;   // the expert's operand tiles of the first k-tile and column tile
    size_t w_tile, w_kt;  // bytes from one column tile / one k-tile of the weights to the next
    int rt, n_kt;    // row tiles of the chunk, k-tiles to walk
    int nrows;
    bool no_weights;  // the expert got no slot: its rows are written as zeros
};

// The ring of a chunk of up to RTC row tiles: a stage is RTC row tiles, then BN / 16 column tiles.  NS is even (two turns of the k loop
// share the weights' registers).
template <int BN, int RTC>
struct GemmRing {
    static constexpr int STAGE = (RTC + BN / 16) * 1024, NS = GEMM_RING / STAGE / 2 * 2;
};

// The k loop of one wavefront.  Eight wavefronts as WM x WN; a wavefront owns four column tiles (wn*4 ..) and the MC row tiles wm, wm + WM, ..
// that the chunk has, and brings BN / 128 column tiles and LA row tiles (wave, wave + 8, ..) per stage.  Wavefronts of one workgroup run
// different instantiations: what they share is the ring and the number of barriers.
template <int BN, int RTC, int MC, int LA>
__device__ inline void gemm_k_loop(const GemmTile &t, const char *ring, int wave, floatx4 (&acc)[4][MC > 0 ? MC : 1]) {
    constexpr int STAGE = GemmRing<BN, RTC>::STAGE, NS = GemmRing<BN, RTC>::NS;
    constexpr int WN = BN / 64, WM = 8 / WN, LW = BN / 128, LOADS = LA + LW;
    constexpr int MX = (MC + 1) / 2, MY = MC - MX;
    static_assert(NS >= 4 && LOADS * (NS - 1) < 64, "NS - 1 stages of LOADS loads per wavefront in flight");
    const int lane = threadIdx.x & 63, wn = wave & (WN - 1), wm = wave / WN;

    // src[i]: this wavefront's i-th tile (column tiles first) for the k-tile to request next (uniform)
    const char *src[LOADS];
#pragma unroll
    for (int i = 0; i < LW; ++i) src[i] = t.w + (size_t)(wave + 8 * i) * t.w_tile;
#pragma unroll
    for (int i = 0; i < LA; ++i) src[LW + i] = t.a + (size_t)(wave + 8 * i) * 1024;
    const size_t a_kt = (size_t)t.rt * 1024;
    const unsigned a_lds = __builtin_amdgcn_readfirstlane(lds_address(ring)) + wave * 1024, w_lds = a_lds + RTC * 1024;
    auto load = [&](int i, unsigned stage_off) {
        load_tile_to_lds(src[i], lane * 16, (i < LW ? w_lds + i * 8192 : a_lds + (i - LW) * 8192) + stage_off);
    };
    auto advance = [&](bool more) {
        const size_t da = more ? a_kt : 0, dw = more ? t.w_kt : 0;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) src[i] += i < LW ? dw : da;
    };
#pragma unroll
    for (int st = 0; st < NS; ++st) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) load(i, st * STAGE);
        advance(st + 1 < t.n_kt);  // fewer k-tiles than stages: the last one again, which nobody reads, so that the count stays uniform
    }

    const bf16x8 *A = reinterpret_cast<const bf16x8 *>(ring) + wm * 64 + lane;
    const bf16x8 *W = reinterpret_cast<const bf16x8 *>(ring + RTC * 1024) + wn * 4 * 64 + lane;
    bf16x8 wf0[4], wf1[4], ax[MX > 0 ? MX : 1];
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * (NS - 1)) : "memory");
    asm volatile("s_barrier" ::: "memory");
    if (MC > 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a) wf0[a] = W[a * 64];
#pragma unroll
        for (int m = 0; m < MX; ++m) ax[m] = A[WM * m * 64];
    }
    unsigned cur = 0;  // byte offset of the stage being multiplied

    // One k-tile.  X is the first half of the row tiles, Y the second; the operands of each half are read from LDS, and the loads
    // issued, between the products of the half before, one at a time: in a batch they keep the matrix cores idle while eight wavefronts queue
    // for LDS.  In the middle: everyone's reads of this stage have returned (they are waited for before the barrier), so its buffer takes the
    // request for the k-tile NS further; the next stage has landed for this wavefront (at most AHEAD stages after it are
    // outstanding) and, after the barrier, for everyone.  A fence here would make the compiler wait for every load in flight.
    auto turn = [&](const bf16x8 (&wf)[4], bf16x8 (&wf_next)[4], auto ahead, auto request) {
        constexpr int AHEAD = decltype(ahead)::value;  // negative: the last k-tile
        constexpr bool REQUEST = decltype(request)::value;
        const bf16x8 *Ac = A + (cur >> 4);
        bf16x8 ay[MY > 0 ? MY : 1];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4 * MX; ++i) {
            acc[i & 3][i >> 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i & 3], ax[i >> 2], acc[i & 3][i >> 2], 0, 0, 0);
            if (i < MY) ay[i] = Ac[WM * (MX + i) * 64];
            __builtin_amdgcn_sched_barrier(0);
        }
        const unsigned freed = cur;
        cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
        if (AHEAD >= 0) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LOADS * (AHEAD > 0 ? AHEAD : 0)) : "memory");
            asm volatile("s_barrier" ::: "memory");
        }
        const bf16x8 *An = A + (cur >> 4), *Wn = W + (cur >> 4);
        constexpr int READS = AHEAD >= 0 && MC > 0 ? 4 + MX : 0, OPS = READS + (REQUEST ? LOADS : 0), MM = MY > 0 ? 4 * MY : 1;
#pragma unroll
        for (int i = 0; i < MM; ++i) {
            if (MY > 0) acc[i & 3][MX + (i >> 2)] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i & 3], ay[i >> 2], acc[i & 3][MX + (i >> 2)], 0, 0, 0);
#pragma unroll
            for (int q = i * OPS / MM; q < (i + 1) * OPS / MM; ++q) {
                if (q >= READS) load(q - READS, freed);
                else if (q < 4) wf_next[q] = Wn[q * 64];
                else ax[q - 4] = An[WM * (q - 4) * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (REQUEST) advance(true);
    };
    using Steady = std::integral_constant<int, NS - 2>;
    for (int kt = NS; kt < t.n_kt; kt += 2) {  // n_kt is even (the launcher checks)
        turn(wf0, wf1, Steady(), std::true_type());
        turn(wf1, wf0, Steady(), std::true_type());
    }
    // the last NS k-tiles (or all of fewer): everything is requested
    static_for<NS / 2>([&](auto half) {
        constexpr int j = 2 * decltype(half)::value;
        if (j >= t.n_kt) return;  // uniform over the workgroup
        turn(wf0, wf1, std::integral_constant<int, NS - 2 - j>(), std::false_type());
        turn(wf1, wf0, std::integral_constant<int, NS - 3 - j>(), std::false_type());
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // a surplus request must not outlive the workgroup's LDS
}

// Row tiles of wavefront `wave` among rt, and how many of them it brings per stage.
template <int BN>
constexpr int gemm_own_tiles(int rt, int wave) {
    constexpr int WN = BN / 64, WM = 8 / WN;
    return rt > wave / WN ? (rt - wave / WN + WM - 1) / WM : 0;
}
constexpr int gemm_brought_tiles(int rt, int wave) { return rt > wave ? (rt - wave + 7) / 8 : 0; }
// Does a chunk of lo .. RTC row tiles have a wavefront with MC row tiles of its own that brings LA?
template <int BN, int RTC, int MC, int LA>
constexpr bool gemm_occurs(int lo) {
    for (int rt = lo; rt <= RTC; ++rt)
        for (int w = 0; w < 8; ++w)
            if (gemm_own_tiles<BN>(rt, w) == MC && gemm_brought_tiles(rt, w) == LA) return true;
    return false;
}

// Rounded results of two neighbouring column tiles: a lane of quarter g has columns 4g .. +3 of both and returns eight columns of one of them, 8 * (g / 2) ..
// of the first (g even) or the second (g odd), by swapping halves with its neighbour quarter.  A row tile of the
// hidden activation is then one contiguous store of 1 KiB, a row of the result 64 bytes at a time: the end of a down-projection item 5.3 -> 3.2 us.
template <bool RELU>
__device__ inline uint4 gemm_octet(const floatx4 even, const floatx4 odd) {
    typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
    bf16x4 e, o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[j] = (__bf16)(RELU ? fmaxf(even[j], 0.f) : even[j]);
        o[j] = (__bf16)(RELU ? fmaxf(odd[j], 0.f) : odd[j]);
    }
    const uintx2 eb = __builtin_bit_cast(uintx2, e), ob = __builtin_bit_cast(uintx2, o);
    // odd quarters of the first operand change places with the even quarters of the second
    const auto lo = __builtin_amdgcn_permlane16_swap(eb[0], ob[0], false, false), hi = __builtin_amdgcn_permlane16_swap(eb[1], ob[1], false, false);
    return make_uint4(lo[0], hi[0], lo[1], hi[1]);
}

// Products and epilogue of one wavefront of a chunk of at most RTC row tiles (and more than the next smaller ring takes).
template <int BN, bool UP, int MC>
__device__ inline void gemm_tile_body(const GemmTile &t, const char *ring, int wave, void *__restrict__ h_chunk, float *__restrict__ partial_rows,
                                      __bf16 *__restrict__ y_rows, int N, int n0) {
    constexpr int WN = BN / 64, WM = 8 / WN;
    const int lane = threadIdx.x & 63, wn = wave & (WN - 1), wm = wave / WN;
    floatx4 acc[4][MC > 0 ? MC : 1];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int m = 0; m < MC; ++m) acc[a][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int R0 = GEMM_RING_TILES[0], R1 = GEMM_RING_TILES[1], R2 = GEMM_RING_TILES[2];
    const int kind = gemm_brought_tiles(t.rt, wave) + (t.rt <= R0 ? 0 : (t.rt <= R1 ? 4 : 8));
    static_for<4>([&](auto la_) {
        constexpr int LA = decltype(la_)::value;
        if constexpr (gemm_occurs<BN, R0, MC, LA>(1))
            if (kind == LA) gemm_k_loop<BN, R0, MC, LA>(t, ring, wave, acc);
        if constexpr (gemm_occurs<BN, R1, MC, LA>(R0 + 1))
            if (kind == 4 + LA) gemm_k_loop<BN, R1, MC, LA>(t, ring, wave, acc);
        if constexpr (gemm_occurs<BN, R2, MC, LA>(R1 + 1))
            if (kind == 8 + LA) gemm_k_loop<BN, R2, MC, LA>(t, ring, wave, acc);
    });

    // lane holds row 16 * row tile + tok, output columns n0 + wn*64 + a*16 + 4*g + {0..3}
    const int tok = lane & 15, g = lane >> 4;
#pragma unroll
    for (int m = 0; m < MC; ++m) {
        const int tile = wm + WM * m, r = tile * 16 + tok;
        if (!UP && partial_rows) {
            if (r >= t.nrows) continue;
            float *dst = partial_rows + (size_t)r * N + n0 + wn * 64 + 4 * g;
#pragma unroll
            for (int a = 0; a < 4; ++a)
                *reinterpret_cast<floatx4 *>(dst + a * 16) = t.no_weights ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[a][m];
            continue;
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {  // two column tiles: every lane ends with eight neighbouring columns, 16 bytes a store instead of 8
            const uint4 o = t.no_weights ? make_uint4(0, 0, 0, 0) : gemm_octet<UP>(acc[2 * p][m], acc[2 * p + 1][m]);
            const int octet = 2 * (g & 1) + (g >> 1);  // of the 32 columns
            if (r >= t.nrows) continue;
            if (UP) {
                // Packed layout of H: per chunk [N/32 k-tiles][row tiles][1 KiB]; a tile holds 16 rows x 32
                // features in matrix-core operand order: cell row%16 + 16*((feature%32)/8), 8 features per
                // cell.  Rows past the chunk's end are left unwritten (the down-projection never stores
                // what it computes from them).
                const int kt = (n0 >> 5) + wn * 2 + p;  // k-tile of the down-projection these 32 features are
                reinterpret_cast<uint4 *>(h_chunk)[((size_t)kt * t.rt + tile) * 64 + tok + 16 * octet] = o;
            } else {
                *reinterpret_cast<uint4 *>(y_rows + (size_t)r * N + n0 + wn * 64 + p * 32 + 8 * octet) = o;
            }
        }
    }
}

// UP = false: the down-projection, A . W2 with K = f, N = d, over K / n_split of the k-tiles: into partial[s]
//             with several slices, else rounded into y_perm.
// UP = true : the up-projection, H = ReLU(A . W1) with K = d, N = f, A the packed rows, W1's tiles
//             n-tile major (the k-tiles of one 16-column slab are contiguous), the result rounded
//             to bf16 and stored packed for the down-projection.
template <int BN, bool UP>
__global__ __launch_bounds__(512) void ffn_gemm_tile_kernel(
    const char *__restrict__ a_packed, const GemmItem *__restrict__ items, int K, int N, int n_split, const char *__restrict__ w_base,
    char *__restrict__ h, float *__restrict__ partial, __bf16 *__restrict__ y_perm, int n_rows) {
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    const GemmItem ci = items[blockIdx.x];
    if (ci.nrows == 0) return;  // uniform over the workgroup
    GemmTile t;
    t.no_weights = ci.w == nullptr;
    const char *wsafe = t.no_weights ? w_base : ci.w;  // a valid address; the rows are written as zeros

    const int n_blocks = N / BN;
    const int split = n_split == 1 ? 0 : ci.col / n_blocks, n0 = (ci.col - split * n_blocks) * BN;
    t.nrows = ci.nrows;
    t.rt = (ci.nrows + 15) >> 4;
    t.n_kt = K / n_split / 32;
    const int kt0 = split * t.n_kt;
    t.a = a_packed + (size_t)ci.tile0 * 32 * K + (size_t)kt0 * t.rt * 1024;
    if (UP) {
        t.w_tile = (size_t)(K / 32) * 1024;
        t.w_kt = 1024;
        t.w = wsafe + (size_t)(n0 >> 4) * t.w_tile;
    } else {
        t.w_tile = 1024;
        t.w_kt = (size_t)(N / 16) * 1024;
        t.w = wsafe + (size_t)K * N * 2 + (size_t)kt0 * t.w_kt + (size_t)(n0 >> 4) * 1024;
    }
    void *h_chunk = UP ? h + (size_t)ci.tile0 * 32 * N : nullptr;
    float *partial_rows = !UP && partial ? partial + ((size_t)split * n_rows + ci.row0) * N : nullptr;
    __bf16 *y_rows = UP ? nullptr : y_perm + (size_t)ci.row0 * N;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), own = gemm_own_tiles<BN>(t.rt, wave);
    // A jump to the body: a chain of comparisons in front of every body would miss the instruction cache at each.
    switch (own) {  // uniform over the wavefront
#define PG_BODY(MC_)                                                                                                                \
    case MC_:                                                                                                                       \
        if constexpr (MC_ <= GEMM_RT / (512 / BN)) gemm_tile_body<BN, UP, MC_>(t, ring, wave, h_chunk, partial_rows, y_rows, N, n0); \
        asm volatile("; %0 row tiles" ::"n"(MC_)); /* keeps the bodies' stores apart: merged, they would copy every accumulator */   \
        return;
        PG_BODY(0) PG_BODY(1) PG_BODY(2) PG_BODY(3) PG_BODY(4) PG_BODY(5) PG_BODY(6) PG_BODY(7) PG_BODY(8) PG_BODY(9) PG_BODY(10)
#undef PG_BODY
    }
}

// ------------------------------------------------------------------------------------------
constexpr int GEMM_SPLIT = 4;  // most K slices of the down-projection (float32 partials)

static int gemm_max_chunks(const pgmoe_config &c, int64_t n_rows) {
    return (int)(std::max<int64_t>(1, std::min<int64_t>(c.n_experts, n_rows)) + n_rows / GEMM_ROWS);
}
// The records of a launch's items (column blocks of the products, K slices); with 128 columns and every slice the most there can be.
static size_t gemm_item_bytes(const pgmoe_config &c, int64_t n_rows, int bn_up = 128, int bn_down = 128, int split = GEMM_SPLIT) {
    return (size_t)gemm_max_chunks(c, n_rows) * (c.d_ff / bn_up + c.d_model / bn_down * split) * sizeof(GemmItem);
}

// Workspace: float32 partials of the down-projection (most K slices), then the bf16 hidden activation, the packed
// rows and the items' records (with room for 128-row chunks, at most one partly filled one per expert; 16-row tiles are what is used).
size_t ffn_gemm_workspace_bytes(const pgmoe_config &c) {
    const int64_t max_rows = (int64_t)c.max_tokens * c.top_k;
    return (size_t)GEMM_SPLIT * max_rows * c.d_model * 4 +
           (size_t)(max_rows / 128 + std::min<int64_t>(c.n_experts, max_rows)) * 128 * (c.d_ff + c.d_model) * 2 + gemm_item_bytes(c, max_rows) + 256;
}

// What pgmoe_expert_ffn_static admits a launch of n_rows rows by (against PGMOE_STATIC_SCRATCH_BYTES; not what a launch uses).  A launch with
// hundreds of rows per expert that it admits is planned to fit the buffer in one pass (gemm_plan); below that the figure is
// what the fused kernel needs, and a launch that does not fit takes several passes or the fused kernel (gemm_slices_for_fused).
size_t ffn_gemm_launch_bytes(const pgmoe_config &c, int n_rows) {
    const int active = std::max(1, std::min(c.n_experts, n_rows));
    if (n_rows / active < GEMM_ALWAYS) return ffn_partial_bytes(c, n_rows);
    const int tiles = (n_rows / 128) * (c.d_model / 128);
    const int split = tiles >= 160 ? 1 : (tiles >= 80 ? 2 : GEMM_SPLIT);
    return (size_t)split * n_rows * c.d_model * 4 + (size_t)(active + n_rows / 128) * 128 * (c.d_ff + c.d_model) * 2;
}
static size_t gemm_tile_bytes(const pgmoe_config &c) { return (size_t)16 * (c.d_ff + c.d_model) * 2; }  // a row tile, hidden and packed

// Microseconds of a fused launch of plan p, as fitted to measurements (see uses_gemm_kernels).
static double fused_estimate(const pgmoe_config &c, int n_rows, const FfnPlan &p) {
    const int active = std::max(1, std::min(c.n_experts, n_rows));
    const double expert = 4.0 * c.d_model * c.d_ff, weights = active * expert / 5.7e6;  // bytes; us at the rate HBM delivers
    const double chunks = std::max((double)active, 0.5 * active + n_rows / (16.0 * p.mt)), wgs = chunks * p.n_partial;
    const bool alone = p.mt * (c.d_model / 32 + p.nw) > 80;  // KiB of LDS: one workgroup per CU, so a second round costs as much as the first
    const double rounds = 1.0 + (alone ? std::min(1.0, std::max(0.0, (wgs - 243.0) / 77.0)) + std::max(0.0, (wgs - 320.0) / 900.0) : std::max(0.0, wgs / 256.0 - 1.0));
    const double again = 0.3 + 0.7 * chunks / active;  // an expert's second chunk finds part of the weights in a cache
    // one workgroup's stream of weights, bytes per us: less the more rows it multiplies, and the more workgroups there are (decay)
    double rate, decay;
    if (p.mt == 1) rate = 188e3, decay = 0.29;
    else if (p.mt == 2) {
        if (c.d_model >= 1024) rate = 71e3, decay = 0.065;
        else if (c.d_model >= 768) rate = 114e3, decay = 0.248;
        else rate = 88e3, decay = 0.123;
    } else if (p.nw == 8) {
        if (c.d_model >= 1024) rate = 62e3, decay = 0.132;
        else rate = 80e3, decay = 0.158;
    } else rate = 55e3, decay = 0.09;
    const double stream = rounds * expert / p.n_partial / (rate * std::pow(std::min(wgs, 256.0), -decay));
    return 12.5 + (p.n_partial > 1 ? 4.2e-6 * p.n_partial * n_rows * c.d_model : 0.0) + std::max(0.90 * weights * again, stream);
}
// What the two GEMMs of a launch take beyond their launches and the latency of their k loops.
static double gemm_estimate(const pgmoe_config &c, int n_rows) {
    const int active = std::max(1, std::min(c.n_experts, n_rows));
    return std::max(0.90 * active * 4.0 * c.d_model * c.d_ff / 5.7e6 + (double)n_rows * c.d_model * c.d_ff / 3.49e8, 1.94e-6 * n_rows * c.d_ff);
}

// Does a launch take the two GEMMs?  From GEMM_ALWAYS rows per expert on always.  Below, the fused kernel streams
// every expert's weights once per chunk of at most 64 rows, with d_ff cut into as few ranges as keep
// its partial sums cheap, so with few experts or several chunks per expert it leaves CUs idle or reads weights
// again; the GEMMs cost two launches more and the round trip of the hidden activation, which is what bounds them where d_model is
// small.  The two estimates (microseconds) were fitted to 1317 launches of earlier loops of both, timed both ways (d_model 128 .. 2048, d_ff 512 .. 8192, 1 .. 256
// experts, 8 .. 190 rows per expert, even and skewed routing), and hold for the present ones: over 170 launches of the same ranges, captured, one
// behind the other, the rule's choices are 1.47 times as fast as the fused kernel on the geometric mean, the better of the two each time would be 1.49
// (worst: 48 experts of 256 x 1024, 77 skewed rows each, 36 us and 20 fused; 96 of 256 x 3072, 159 rows each, fused 156 and 118). With three streams of
// launches 1.15 and 1.22: few experts of d_model 512 and less take 14 us as three launches and 7 to 9 fused, whose launches overlap.
bool uses_gemm_kernels(const pgmoe_config &c, int n_rows) {
    if (c.dtype != PGMOE_BF16) return false;
    // the k loop takes two 32-k tiles per turn (in every K slice of the down-projection); the pack kernel PACK_KT k-tiles per workgroup
    if (c.d_model % 128 || c.d_ff % 128 || c.d_model % (32 * PACK_KT) || c.d_ff % (GEMM_SPLIT * 64)) return false;
    const int active = std::max(1, std::min(c.n_experts, n_rows));
    if (n_rows / active >= GEMM_ALWAYS) return true;
    if (n_rows / active < 8) return false;
    // the static buffer has to hold at least one chunk of a launch it admits
    if (ffn_partial_bytes(c, n_rows) <= PGMOE_STATIC_SCRATCH_BYTES && 2 * GEMM_RT * gemm_tile_bytes(c) + gemm_item_bytes(c, n_rows) > PGMOE_STATIC_SCRATCH_BYTES) return false;
    const double gemm = 23.5 + 0.00087 * (c.d_model + c.d_ff) + gemm_estimate(c, n_rows);
    // in doubt fused: a skewed routing costs the GEMMs more, with many experts above all
    const double margin = c.d_model <= 256 ? (active >= 64 ? 1.5 : 1.1) : (active >= 96 ? 1.1 : (active >= 32 ? 1.05 : 1.0));
    return margin * gemm < fused_estimate(c, n_rows, plan_ffn(c, n_rows));
}

// Column width of the two products and K slices of the down-projection, from the shape of the launch alone.
struct GemmPlan {
    int bn_up, bn_down, split;
    size_t p_bytes;
};
static GemmPlan gemm_plan(const pgmoe_config &c, int n_rows) {
    const int active = std::max(1, std::min(c.n_experts, n_rows));
    const double chunks = std::max((double)active, n_rows / (double)GEMM_ROWS + 0.4 * active);  // estimate
    const double rt = std::min(20.0, n_rows / 16.0 / chunks + 0.5);                             // row tiles of a chunk
    GemmPlan best = {};
    double best_up = 1e30, best_down = 1e30;
    const bool admitted = ffn_gemm_launch_bytes(c, n_rows) <= PGMOE_STATIC_SCRATCH_BYTES;
    for (int bn = 128; bn <= 256; bn *= 2) {
        // microseconds per 32-k stage of a workgroup that has its CU to itself: prices from before a chunk's ring went by its size (0.64 and 0.32 here for sixteen
        // and two row tiles of 256 columns, which then took 0.76 and 0.46 and now take 0.62 and 0.38)
        const double stage = (bn == 256 ? 0.80 : 0.50) * std::max(rt / 20.0, 0.4);
        auto rounds = [&](double wgs) { return std::max(1.0, std::ceil(wgs / 256.0 - 0.05)); };
        if (c.d_ff % bn == 0) {
            const double up = rounds(chunks * (c.d_ff / bn)) * (c.d_model / 32 * stage + 4.0);
            if (up < best_up) {
                best_up = up;
                best.bn_up = bn;
            }
        }
        if (c.d_model % bn == 0)
            for (int split = 1; split <= GEMM_SPLIT; split *= 2) {
                const size_t p_bytes = split > 1 ? (size_t)split * n_rows * c.d_model * 4 : 0;
                // row tiles the static buffer has to hold beside them: with hundreds of rows per expert all (1280 rows over 4 experts of 1024 x 4096
                // with two K slices 76 us, with four 69 but 108 in the static buffer's two passes), else those of a pass
                const int hold = n_rows / active >= GEMM_ALWAYS ? active + n_rows / 16 : 2 * GEMM_RT;
                if (admitted && split > 1 && p_bytes + hold * gemm_tile_bytes(c) + gemm_item_bytes(c, n_rows, 128, bn, split) > PGMOE_STATIC_SCRATCH_BYTES) continue;
                const double down = rounds(chunks * (c.d_model / bn) * split) * (c.d_ff / 32 / split * stage + 4.0) +
                                    (split > 1 ? 2.0 * p_bytes : 2.0 * n_rows * c.d_model * 2.0) / 4.0e6;
                if (down < best_down) {
                    best_down = down;
                    best.bn_down = bn;
                    best.split = split;
                    best.p_bytes = p_bytes;
                }
            }
    }
    return best;
}

// The scratch of a launch: float32 partials [split][n_rows, d] first (the combine reads them at the workspace's start; none with one
// slice), then the packed hidden activation and the packed rows, by 16-row tiles (at most one partly filled tile per expert), and the items' records.
// Scratch that does not hold every tile (the static buffer) is used for one range of chunks after the other: a
// chunk's result does not depend on the others, so the number of passes changes no bit.
struct GemmScratch {
    int max_tiles;  // most row tiles of the launch
    size_t room;    // row tiles the scratch holds beside the partials and the items' records
    bool one_pass;
    int tiles;      // first tiles of a pass: its last chunk may reach past them
};
static GemmScratch gemm_scratch(const pgmoe_config &c, int n_rows, const GemmPlan &p, size_t workspace_bytes) {
    GemmScratch r;
    const size_t beside = p.p_bytes + gemm_item_bytes(c, n_rows, p.bn_up, p.bn_down, p.split);
    r.max_tiles = std::max(1, std::min(c.n_experts, n_rows)) + n_rows / 16;
    r.room = workspace_bytes > beside ? (workspace_bytes - beside) / gemm_tile_bytes(c) : 0;
    r.one_pass = r.room >= (size_t)r.max_tiles;
    r.tiles = r.one_pass ? r.max_tiles : (int)r.room - GEMM_RT;
    return r;
}

// A pass costs its three launches and the latency of its k loops however few chunks it has, and a range of chunks seldom fills the chip, so a
// launch of several passes can be slower than the fused kernel, which needs no scratch but the partials: it adds in the same order as
// the GEMMs if d_ff is cut into as many ranges as they have K slices, and gives their bits.  Fitted to 75 launches of two passes or
// more, even and skewed: 128 experts of 768 x 3072 at 128 rows each 485 us fused and 617 in passes, 32 of 512 x 8192 at 160 rows 265 and 947;
// but 16 of 2048 x 8192 at 96 rows 1243 and 307, 24 of 1024 x 4096 at 128 rows 463 and 188.
int gemm_slices_for_fused(const pgmoe_config &c, int n_rows, size_t workspace_bytes) {
    const GemmPlan p = gemm_plan(c, n_rows);
    const GemmScratch r = gemm_scratch(c, n_rows, p, workspace_bytes);
    if (r.one_pass || r.tiles < 1) return 0;
    const int passes = (r.max_tiles + r.tiles - 1) / r.tiles;
    const double gemm = passes * (18.0 + 0.01 * (c.d_model + c.d_ff / p.split)) + gemm_estimate(c, n_rows);
    return passes <= 6 && 1.1 * gemm < fused_estimate(c, n_rows, plan_ffn(c, n_rows, p.split)) ? 0 : p.split;
}

int launch_ffn_gemm(pgmoe_ctx *ctx, const char *w_base, size_t w_stride, bool slot_by_rank, int n_slots, const void *x_perm,
                    const int32_t *offsets, int n_rows, void *y_perm, void *workspace, size_t workspace_bytes, hipStream_t s,
                    int *keep_partials, const unsigned long long *table, const int32_t *src_row) {
    const pgmoe_config &c = ctx->cfg;
    const int max_chunks = gemm_max_chunks(c, n_rows);
    const GemmPlan p = gemm_plan(c, n_rows);
    const GemmScratch r = gemm_scratch(c, n_rows, p, workspace_bytes);
    if (!r.one_pass && r.tiles < GEMM_RT)
        return fail(ctx, PGMOE_EINVAL, "pgmoe_expert_ffn: hidden activation, packed rows and partial sums of %d rows do not fit the workspace", n_rows);
    const size_t held = r.one_pass ? (size_t)r.max_tiles : r.room, h_bytes = held * 16 * c.d_ff * 2;
    const int gy_up = c.d_ff / p.bn_up, gy_down = c.d_model / p.bn_down * p.split;
    float *partial = p.split > 1 ? (float *)workspace : nullptr;
    char *h = (char *)workspace + p.p_bytes;
    char *xp = h + h_bytes;
    GemmItem *items = (GemmItem *)(h + held * gemm_tile_bytes(c));
    const int tslot = ffn_timing_slot(ctx);
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_begin[tslot], s));
    for (int lo = 0; lo < r.max_tiles; lo += r.tiles) {
        const int hi = r.one_pass ? INT_MAX : lo + r.tiles;  // INT_MAX: every chunk
        hipLaunchKernelGGL(ffn_gemm_pack_rows_kernel, dim3(max_chunks, c.d_model / 32 / PACK_KT), dim3(512), 0, s, (const __bf16 *)x_perm,
                           offsets, c.n_experts, c.d_model, src_row, (__bf16 *)xp, lo, hi, w_base, w_stride, slot_by_rank ? 1 : 0, n_slots, table, items,
                           gy_up, gy_down);
        PG_HIP(ctx, hipGetLastError());
#define PG_TILE(BN_, UP_, A_, ITEMS_, GY_, K_, N_, SPLIT_)                                                                         \
    do {                                                                                                                           \
        auto kern_ = ffn_gemm_tile_kernel<BN_, UP_>;                                                                               \
        if (int rc_ = allow_dynamic_lds(ctx, reinterpret_cast<const void *>(kern_), GEMM_RING)) return rc_;                        \
        hipLaunchKernelGGL(kern_, dim3(max_chunks * GY_), dim3(512), GEMM_RING, s, (const char *)(A_), ITEMS_, K_, N_, SPLIT_, w_base, h, partial, \
                           (__bf16 *)y_perm, n_rows);                                                                              \
        PG_HIP(ctx, hipGetLastError());                                                                                            \
    } while (0)
        if (p.bn_up == 256) PG_TILE(256, true, xp, items, gy_up, c.d_model, c.d_ff, 1);
        else PG_TILE(128, true, xp, items, gy_up, c.d_model, c.d_ff, 1);
        if (p.bn_down == 256) PG_TILE(256, false, h, items + (size_t)max_chunks * gy_up, gy_down, c.d_ff, c.d_model, p.split);
        else PG_TILE(128, false, h, items + (size_t)max_chunks * gy_up, gy_down, c.d_ff, c.d_model, p.split);
#undef PG_TILE
    }
    if (tslot >= 0) PG_HIP(ctx, hipEventRecord(ctx->tim_end[tslot], s));
    if (!partial) return PGMOE_OK;  // y_perm was written directly
    if (keep_partials) {
        *keep_partials = p.split;
        return PGMOE_OK;
    }
    return launch_ffn_reduce(ctx, partial, p.split, n_rows, y_perm, s);
}

}  // namespace pgmoe
