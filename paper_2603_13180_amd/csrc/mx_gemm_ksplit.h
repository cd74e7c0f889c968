// mx_gemm_ksplit.h -- the MX product for outputs of few small tiles: one
// BM x BN tile per workgroup, its K steps dealt to the NW waves.
//
// What bounds it: the serial chain of a tile's K steps.  With the waves on
// different parts of one tile every step costs a barrier and an LDS round
// trip (0.4 us at 64 x 64); here wave w multiplies the whole tile for steps w,
// w + NW, ... from a ring of S steps of LDS that only this wave loads and
// reads.  Nothing synchronises the waves until their NW partial sums meet in
// LDS, where they are added in wave order.  Per compute unit the operand
// stream then runs at its limit of about 55 GB/s.  Measured (E4M3, K = 4096):
// 16 x 6144 47.7 us on 256 x 256 tiles, 12.5 us as a ring of 64 x 64 tiles,
// 6.8 us here with 16 x 32 tiles; 1024 x 768 x 2304 31.2 -> 8.7 us with
// 64 x 64.
#pragma once

#include "mx_gemm.h"

namespace mxg {

template <int BM_, int BN_, int NW_, int S_> struct KSplit {
    static constexpr int BM = BM_, BN = BN_, NW = NW_, S = S_, NT = 64 * NW;
    static constexpr int FM = BM / 16, FN = BN / 16;
    static constexpr int LC = (BM + BN) / 8; // code loads per step
};

template <class C, int ELEM> struct KSplitOp {
    static constexpr int SB = kSB<ELEM>;
    static constexpr int LS = ((C::BM + C::BN) * SB + 255) / 256; // scale loads per step
    static constexpr int L = C::LC + LS;
    static constexpr int SLOT = (C::BM + C::BN) * KB + LS * 256;
    static_assert((C::S - 1) * L <= 63, "vmcnt range");
    // a wave's part of LDS: its ring, then its partial sums
    static constexpr int PART = C::S * SLOT > C::FM * C::FN * 1024 ? C::S * SLOT : C::FM * C::FN * 1024;
    static_assert(C::NW * PART <= 160 * 1024, "LDS");
};

template <int ELEM, int OUT, class C>
__global__ void __launch_bounds__(C::NT) mx_gemm_ksplit_kernel(Args A)
{
    using O = KSplitOp<C, ELEM>;
    constexpr int SB = O::SB, DW = SB / 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[C::NW * O::PART];

    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    const int g = l >> 4, qd = l & 15;
    int64_t m0, n0;
    tile_of(A, C::BM, C::BN, blockIdx.x, m0, n0);
    if (m0 >= A.M || n0 >= A.N) // a part of a cell that lies outside H
        return;

    // Lane offsets of the rows this lane loads (A's BM rows, then B's; 8 rows
    // x 128 bytes per instruction, swizzled as in the fragment reads; scale
    // dword 64 t + l of the step).  Rows past M or N read the last row: their
    // results are never stored.
    const uint8_t *ta = A.a + m0 * A.rb, *tb = A.b + n0 * A.rb;
    const int rr = l >> 3, ch = (l & 7) ^ rr;
    uint32_t code[C::LC];
#pragma unroll
    for (int t = 0; t < C::LC; ++t) {
        const int r = 8 * t;
        const int64_t off = r < C::BM ? min(m0 + r + rr, A.M - 1) - m0
                                      : min(n0 + (r - C::BM) + rr, A.N - 1) - n0;
        code[t] = (uint32_t)(off * A.rb) + 16 * ch;
    }
    const uint8_t *sc[O::LS];
#pragma unroll
    for (int t = 0; t < O::LS; ++t) {
        const int dw = 64 * t + l, r = min(dw / DW, C::BM + C::BN - 1);
        sc[t] = (r < C::BM ? A.as + min(m0 + r, A.M - 1) * A.rs
                           : A.bs + min(n0 + (r - C::BM), A.N - 1) * A.rs) + 4 * (dw % DW);
    }

    LDS_AS uint8_t *ring = (LDS_AS uint8_t *)lds + w * O::PART;
    const uint32_t ring_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)ring);
    auto issue = [&](int k, int slot) {
        const uint32_t st = ring_addr + slot * O::SLOT;
#pragma unroll
        for (int t = 0; t < C::LC; ++t)
            lds_load16(8 * t < C::BM ? ta : tb, code[t] + (uint32_t)k * KB, st + 8 * t * KB);
#pragma unroll
        for (int t = 0; t < O::LS; ++t)
            lds_load4(sc[t] + (uint32_t)k * SB, st + (C::BM + C::BN) * KB + 256 * t);
    };
    const FragBase ba = frag_base<ELEM>(0, (C::BM + C::BN) * KB, 0, qd, g);
    const FragBase bb = frag_base<ELEM>(C::BM * KB, (C::BM + C::BN) * KB + C::BM * SB, 0, qd, g);

    v4f acc[C::FM][C::FN];
#pragma unroll
    for (int j = 0; j < C::FM; ++j)
#pragma unroll
        for (int i = 0; i < C::FN; ++i)
            acc[j][i] = v4f{0.f, 0.f, 0.f, 0.f};
    const int mine = w < A.steps ? (A.steps - w - 1) / C::NW + 1 : 0; // this wave's steps
#pragma unroll 1
    for (int p = 0; p < C::S && p < mine; ++p)
        issue(w + p * C::NW, p);
    int slot = 0;
#pragma unroll 1
    for (int p = 0; p < mine; ++p) {
        wait_steps<O::L, C::S - 1>(mine - 1 - p);
        const LDS_AS uint8_t *st = ring + slot * O::SLOT;
        Frag fa[C::FM], fb[C::FN];
        read_frags<ELEM, C::FN>(fb, st, bb, std::make_integer_sequence<int, C::FN>{});
        read_frags<ELEM, C::FM>(fa, st, ba, std::make_integer_sequence<int, C::FM>{});
        // the slot is in registers: its next step may land in it
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (p + C::S < mine)
            issue(w + (p + C::S) * C::NW, slot);
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
            mma_column<ELEM, C::FN>(acc[j], fb, fa[j]);
        slot = slot + 1 == C::S ? 0 : slot + 1;
    }

    // partial sums, each wave's in its own ring
    LDS_AS v4f *sum = reinterpret_cast<LDS_AS v4f *>(ring);
#pragma unroll
    for (int j = 0; j < C::FM; ++j)
#pragma unroll
        for (int i = 0; i < C::FN; ++i)
            sum[(j * C::FN + i) * 64 + l] = acc[j][i];
    barrier();
    for (int f = w; f < C::FM * C::FN; f += C::NW) {
        v4f v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < C::NW; ++u)
            v += reinterpret_cast<const LDS_AS v4f *>((LDS_AS uint8_t *)lds +
                                                      u * O::PART)[f * 64 + l];
        // lane (g, qd) of tile (j, i) holds H[m0 + 16 j + qd][n0 + 16 i + 4 g .. +3]
        const int64_t m = m0 + 16 * (f / C::FN) + qd, n = n0 + 16 * (f % C::FN) + 4 * g;
        if (m < A.M && n < A.N) { // N is a multiple of 16
            if (A.bgain) {
                const uint2 gw = *reinterpret_cast<const uint2 *>(A.bgain + n);
                v[0] = v[0] * __uint_as_float(gw.x << 16);
                v[1] = v[1] * __uint_as_float(gw.x & 0xFFFF0000u);
                v[2] = v[2] * __uint_as_float(gw.y << 16);
                v[3] = v[3] * __uint_as_float(gw.y & 0xFFFF0000u);
            }
            if constexpr (OUT == MX_OUT_F32)
                *reinterpret_cast<v4f *>(static_cast<float *>(A.out) + m * A.N + n) = v;
            else
                *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(A.out) + m * A.N + n) =
                    make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        }
    }
}

template <int ELEM, int OUT, class C> hipError_t launch_ksplit(const Args &A, hipStream_t stream)
{
    hipLaunchKernelGGL((mx_gemm_ksplit_kernel<ELEM, OUT, C>), dim3((unsigned)(A.cells * A.sub_m * A.sub_n)),
                       dim3(C::NT), 0, stream, A);
    return hipGetLastError();
}

} // namespace mxg
