// mx_gemm_ring.h -- the MX product on tiles smaller than 256 x 256, for
// outputs that do not fill the chip with those: BM x BN tiles, WM x WN waves,
// a ring of S K steps in LDS.
//
// What bounds it: with few K steps' worth of products per workgroup the DMA's
// latency (1-3 us from issue to landing when every compute unit loads), not
// its bandwidth, sets the pace, so the ring keeps S - 1 steps in flight: one
// barrier per step, at which this step's DMA has landed for every wave and
// the slot of the step before is free for the step S - 1 ahead.  The steps of
// all tiles of a workgroup form one sequence, so the loads of the next tiles
// run under the last steps and the stores of this one.  Four waves and at most
// 80 KB of LDS: two workgroups share a compute unit, one's products under the
// other's waits.  Measured (E4M3) against 256 x 256 tiles: 61 x 28672 x 4096
// 58 -> 34 us (64 x 128 tiles), 1000 x 8192 x 2048 29.4 -> 22.9 us and 2048 x
// 4096 x 4096 51.9 -> 43.3 us (128 x 128).  At those sizes the operand stream
// (about 13 TB/s over the chip) sets the pace.
#pragma once

#include "mx_gemm.h"

namespace mxg {

template <int BM_, int BN_, int WM_, int WN_, int S_> struct Ring {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, S = S_;
    static constexpr int NW = WM * WN, NT = 64 * NW;
    static constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
    static constexpr int CODE_INSTR = (BM + BN) / 8; // 8 rows each
    static constexpr int LPW = CODE_INSTR / NW;      // code loads per wave and step
    static_assert(CODE_INSTR % NW == 0 && BM % 8 == 0 && FN % 2 == 0, "tile shape");
};

template <class C, int ELEM> struct RingOp {
    static constexpr int SB = kSB<ELEM>;
    static constexpr int SROWS = 256 / SB;                    // rows per scale instruction
    static constexpr int SINSTR = (C::BM + C::BN) / SROWS;    // scale instructions per step
    static constexpr int SPW = (SINSTR + C::NW - 1) / C::NW;  // per wave
    static constexpr int L = C::LPW + SPW;                    // loads per wave and step
    static constexpr int STAGE = (C::BM + C::BN) * (KB + SB);
    static_assert(C::BM % SROWS == 0 && C::BN % SROWS == 0, "a scale instruction covers one operand");
    static_assert((C::S - 2) * L <= 63, "vmcnt range");
    static_assert(C::S * STAGE <= 160 * 1024, "LDS");
};

// The tile whose steps are being loaded.
template <class C, int ELEM> struct RingTile {
    const uint8_t *a, *b, *as, *bs;              // rows m0 / n0
    uint32_t code[C::LPW];                       // lane offsets of the code rows
    uint32_t sc[RingOp<C, ELEM>::SPW];           // and of the scale dwords
};

// Wave w moves code rows 8 LPW w .. of the stage (A's BM rows, then B's):
// per instruction 8 rows x 128 bytes, lane l filling slot l % 8 of row l / 8
// with source chunk (l % 8) ^ (l / 8).  Scale instruction u moves the scale
// bytes of 256 / SB stage rows; with fewer instructions than waves, several
// waves move the same bytes, so that every wave counts L loads per step.
// Rows past M or N read the last row: their results are never stored.
template <class C, int ELEM>
__device__ __forceinline__ RingTile<C, ELEM> ring_tile(const Args &A, int64_t m0, int64_t n0, int w,
                                                       int l)
{
    using O = RingOp<C, ELEM>;
    constexpr int DW = O::SB / 4;
    RingTile<C, ELEM> T;
    const int64_t mb = min(m0, A.M - 1), nb = min(n0, A.N - 1);
    T.a = A.a + mb * A.rb;
    T.b = A.b + nb * A.rb;
    T.as = A.as + mb * A.rs;
    T.bs = A.bs + nb * A.rs;
    const int rr = l >> 3, ch = (l & 7) ^ rr;
#pragma unroll
    for (int t = 0; t < C::LPW; ++t) {
        const int r = 8 * (w * C::LPW + t); // wave-uniform first stage row
        const int64_t off = r < C::BM ? min(m0 + r + rr, A.M - 1) - mb
                                      : min(n0 + (r - C::BM) + rr, A.N - 1) - nb;
        T.code[t] = (uint32_t)(off * A.rb) + 16 * ch;
    }
#pragma unroll
    for (int t = 0; t < O::SPW; ++t) {
        const int r = ((w * O::SPW + t) % O::SINSTR) * O::SROWS;
        const int64_t off = r < C::BM ? min(m0 + r + l / DW, A.M - 1) - mb
                                      : min(n0 + (r - C::BM) + l / DW, A.N - 1) - nb;
        T.sc[t] = (uint32_t)(off * A.rs) + 4 * (l % DW);
    }
    return T;
}

template <class C, int ELEM>
__device__ __forceinline__ void ring_issue(const RingTile<C, ELEM> &T, int s, uint32_t stage, int w)
{
    using O = RingOp<C, ELEM>;
    const uint32_t kc = (uint32_t)s * KB, ks = (uint32_t)s * O::SB;
#pragma unroll
    for (int t = 0; t < C::LPW; ++t) {
        const int r = 8 * (w * C::LPW + t);
        lds_load16(r < C::BM ? T.a : T.b, T.code[t] + kc, stage + r * KB);
    }
#pragma unroll
    for (int t = 0; t < O::SPW; ++t) {
        const int r = ((w * O::SPW + t) % O::SINSTR) * O::SROWS;
        lds_load4(r < C::BM ? T.as : T.bs, T.sc[t] + ks, stage + (C::BM + C::BN) * KB + r * O::SB);
    }
}

// Tiles first, first + stride, ... of the launch on this workgroup.
template <int ELEM, int OUT, class C>
__device__ __forceinline__ void ring_tiles(const Args &A, LDS_AS uint8_t *st0, int first, int stride)
{
    using O = RingOp<C, ELEM>;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63;
    const int g = l >> 4, qd = l & 15;
    const int wm = (w % C::WM) * (C::BM / C::WM), wn = (w / C::WM) * (C::BN / C::WN);

    const uint32_t st0_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)st0);
    const FragBase ba = frag_base<ELEM>(0, (C::BM + C::BN) * KB, wm, qd, g);
    const FragBase bb =
        frag_base<ELEM>(C::BM * KB, (C::BM + C::BN) * KB + C::BM * O::SB, wn, qd, g);

    // (iv, is) is the next step to load, `ahead` the steps loaded past the one
    // being multiplied
    const int G = A.cells * A.sub_m * A.sub_n;
    int iv = first, is = 0, islot = 0, ahead = -1;
    RingTile<C, ELEM> T;
    int64_t im, in;
    tile_of(A, C::BM, C::BN, iv, im, in);
    T = ring_tile<C, ELEM>(A, im, in, w, l);
    auto issue = [&] {
        if (iv >= G)
            return;
        ring_issue<C, ELEM>(T, is, st0_addr + islot * O::STAGE, w);
        islot = islot + 1 == C::S ? 0 : islot + 1;
        ++ahead;
        if (++is == A.steps) {
            is = 0;
            iv += stride;
            if (iv < G) {
                tile_of(A, C::BM, C::BN, iv, im, in);
                T = ring_tile<C, ELEM>(A, im, in, w, l);
            }
        }
    };
#pragma unroll 1
    for (int p = 0; p < C::S - 1; ++p)
        issue();

    int slot = 0;
    for (int v = first; v < G; v += stride) {
        int64_t m0, n0;
        tile_of(A, C::BM, C::BN, v, m0, n0);
        v4f acc[C::FM][C::FN];
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
#pragma unroll
            for (int i = 0; i < C::FN; ++i)
                acc[j][i] = v4f{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < A.steps; ++s) {
            wait_steps<O::L, C::S - 2>(ahead);
            barrier();
            issue();
            const LDS_AS uint8_t *st = st0 + slot * O::STAGE;
            Frag fa[C::FM], fb[C::FN];
            read_frags<ELEM, C::FN>(fb, st, bb, std::make_integer_sequence<int, C::FN>{});
            read_frags<ELEM, C::FM>(fa, st, ba, std::make_integer_sequence<int, C::FM>{});
#pragma unroll
            for (int j = 0; j < C::FM; ++j)
                mma_column<ELEM, C::FN>(acc[j], fb, fa[j]);
            slot = slot + 1 == C::S ? 0 : slot + 1;
            --ahead;
        }
        v4f at[C::FN][C::FM];
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
#pragma unroll
            for (int i = 0; i < C::FN; ++i)
                at[i][j] = acc[j][i];
        store_tile<OUT, C::FM, C::FN>(A, at, m0, n0, wm, wn, g, qd);
    }
}

template <int ELEM, int OUT, class C>
__global__ void __launch_bounds__(C::NT) mx_gemm_ring_kernel(Args A)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[C::S * RingOp<C, ELEM>::STAGE];
    ring_tiles<ELEM, OUT, C>(A, (LDS_AS uint8_t *)lds, blockIdx.x, gridDim.x);
}

// Two products whose tiles are all resident at once, one tile per workgroup:
// product 0 (float output) in workgroups 0 .. n0 - 1 or, if product 1 (bf16)
// has the longer K, in those after product 1's.  Each alone leaves compute
// units idle (1024 x 768 x 2304 has 96 tiles): both in one launch, 1024 x 768 x
// 2304 and 2304 x 768 x 1024 (E4M3), 14.2 us against 16.2 apart.
struct RingPair {
    Args p[2];
    int n0, n1;
    int second_first;
};

template <int ELEM, class C>
__global__ void __launch_bounds__(C::NT) mx_gemm_ring_pair_kernel(RingPair W)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[C::S * RingOp<C, ELEM>::STAGE];
    const int b = blockIdx.x;
    const bool second = W.second_first ? b < W.n1 : b >= W.n0;
    if (second) {
        const int v = W.second_first ? b : b - W.n0;
        ring_tiles<ELEM, MX_OUT_BF16, C>(W.p[1], (LDS_AS uint8_t *)lds, v, W.n1);
    } else {
        const int v = W.second_first ? b - W.n1 : b;
        ring_tiles<ELEM, MX_OUT_F32, C>(W.p[0], (LDS_AS uint8_t *)lds, v, W.n0);
    }
}

template <int ELEM, int OUT, class C> hipError_t launch_ring(const Args &A, hipStream_t stream)
{
    using O = RingOp<C, ELEM>;
    const int per_cu = std::min((160 * 1024) / (C::S * O::STAGE), 2048 / C::NT);
    const int64_t G = (int64_t)A.cells * A.sub_m * A.sub_n;
    const int64_t grid = std::min<int64_t>(G, (int64_t)A.grid_max * per_cu);
    hipLaunchKernelGGL((mx_gemm_ring_kernel<ELEM, OUT, C>), dim3((unsigned)grid), dim3(C::NT), 0,
                       stream, A);
    return hipGetLastError();
}

} // namespace mxg
