// One sub-slab of the decode-sized expert kernel, shared by the launch of a single block (ffn.hip) and the one of a whole stack
// (ffn_decode_stack.hip).
#ifndef PGMOE_FFN_DECODE_H
#define PGMOE_FFN_DECODE_H
#include "ffn_common.h"

namespace pgmoe {

constexpr size_t decode_lds_bytes(int kt) { return (size_t)kt * 1024 + 4096; }

// At most 16 rows of one expert times hidden features 32*sub .. +31, 256 threads; see ffn_decode_kernel.  wexp: the expert's blob (uniform; null: the
// rows are zeroed).  fill(xs) puts the rows into LDS as operand cells [KT][64], zeros past the last one, once the weights have been requested;
// store(column, tok, y) takes four neighbouring columns of row tok's partial sum.
template <int KT, typename Fill, typename Store>
__device__ inline void decode_sub_slab(char *smem, const char *__restrict__ wexp, int f, int sub, Fill fill, Store store) {
    constexpr int d = KT * 32;
    constexpr int NTD = KT * 2;   // output n-tiles
    constexpr int NA = KT / 2;    // phase-A tiles per wavefront
    constexpr int NB = NTD / 4;   // phase-B tiles per wavefront
    static_assert(KT % 2 == 0, "k split");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cw = wave & 1, ks = wave >> 1;

    const int fs = sub * 32;

    bf16x8 ta[NA], tb[NB];
    if (wexp) {
        const global_bf16x8 *w1 = (const global_bf16x8 *)wexp + (((size_t)((fs >> 4) + cw) * KT) << 6) + lane;
        const global_bf16x8 *w2 = (const global_bf16x8 *)(wexp + (size_t)d * f * 2) +
                           (((size_t)(fs >> 5) * NTD + wave * NB) << 6) + lane;
#pragma unroll
        for (int i = 0; i < NA; ++i) ta[i] = w1[(size_t)(ks + 2 * i) << 6];
#pragma unroll
        for (int a = 0; a < NB; ++a) tb[a] = w2[(size_t)a << 6];
    } else {
#pragma unroll
        for (int i = 0; i < NA; ++i) ta[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int a = 0; a < NB; ++a) tb[a] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    }

    bf16x8 *xs = reinterpret_cast<bf16x8 *>(smem);                       // [KT][64] operand cells
    floatx4 *hsum = reinterpret_cast<floatx4 *>(xs + (size_t)KT * 64);   // [2 k-halves][2 n-tiles][64]
    fill(xs);
    lds_barrier();

    // ---- phase A: 16 hidden features (n-tile cw of the sub-slab) over this wavefront's k-tiles
    floatx4 hacc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NA; ++i)
        hacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ta[i], xs[((ks + 2 * i) << 6) + lane], hacc, 0, 0, 0);
    hsum[(ks * 2 + cw) * 64 + lane] = hacc;
    lds_barrier();

    // ---- hidden activation as phase-B operand: lane (token lane%16, k-group g = lane/16) needs
    // features 8g .. 8g+7 of the 32, i.e. n-tile g/2, accumulator rows 4*q' + r for q' = 2*(g%2), +1
    const int tok = lane & 15, g = lane >> 4;
    bf16x8 hfrag;
    {
        const int src = (g >> 1) * 64 + (2 * (g & 1)) * 16 + tok;
        const floatx4 lo = hsum[src] + hsum[128 + src];
        const floatx4 hi = hsum[src + 16] + hsum[128 + src + 16];
        hfrag[0] = (__bf16)fmaxf(lo.x, 0.f);
        hfrag[1] = (__bf16)fmaxf(lo.y, 0.f);
        hfrag[2] = (__bf16)fmaxf(lo.z, 0.f);
        hfrag[3] = (__bf16)fmaxf(lo.w, 0.f);
        hfrag[4] = (__bf16)fmaxf(hi.x, 0.f);
        hfrag[5] = (__bf16)fmaxf(hi.y, 0.f);
        hfrag[6] = (__bf16)fmaxf(hi.z, 0.f);
        hfrag[7] = (__bf16)fmaxf(hi.w, 0.f);
    }

    // ---- phase B: this wavefront's NB output n-tiles; lane holds token tok, columns 16*tile + 4*g + {0..3}
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        const floatx4 y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tb[a], hfrag, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        store((wave * NB + a) * 16 + 4 * g, tok, y);
    }
}

}  // namespace pgmoe
#endif  // PGMOE_FFN_DECODE_H
