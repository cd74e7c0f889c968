// MX matrix product H = dec(A) dec(B)^T on the gfx950 block-scaled matrix
// cores (Sec. 3.7 eq. (mx-matmul): the product MXNormLinear takes of MXNorm's
// output and the gain-folded weight cast; the implementation appendix's
// mx_norm_linear_forward ends in this product).
//
// A [M, K] (activations, MXNorm codes) and B [N, K] (weights) are both blocked
// along K with one E8M0 scale per 32 elements; elements are E4M3 (one byte)
// or E2M1 (two per byte, element 2j in the low nibble).  The hardware
// instruction v_mfma_scale_f32_16x16x128_f8f6f4 multiplies a 16x128 tile of
// each operand with one scale byte per row and 32-element block applied
// exactly, accumulating in fp32.
//
// Tiling: a workgroup of 8 waves (two per SIMD) computes a 256 (M) x 256 (N)
// output tile; wave w owns the 128 x 64 quarter-column (w & 1, w >> 1) as
// 8 x 4 matrix-core tiles of 16 x 16, 128 accumulator registers.  Two waves
// per SIMD are what lets the matrix core run while the other wave waits on
// LDS or a barrier: with one wave per SIMD the E2M1 instruction issues at
// about half its rate.  The K loop moves 128 bytes of every row per step
// (128 E4M3 or 256 E2M1 elements) from global memory straight into LDS
// (16-byte global_load_lds, no staging registers) into two stages of 66 KB;
// each step reads its four B fragments into registers and streams the eight
// A fragments two ahead of the matrix core.  In LDS, 16-byte chunk c of row r
// lives at chunk c ^ (r & 7) of the row, so the fragment reads of 8
// consecutive rows hit distinct banks.
//
// What bounds it: at 256 x 256 the operand stream is 64 KB per K step per
// workgroup, about 10 TB/s of L2 requests at half the fp8 peak.  Two stages
// fill LDS, so the DMA runs one step ahead of the products and each step
// waits for it; the tile's stores slow the operand stream (the non-temporal
// policy below halves that); and after each step's barrier every wave reads
// fragments before its first product.  The eight waves' accumulators fill
// half the register file, which leaves no room for a third stage in
// registers.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "mx_gemm.h"
#include "mx_gemm_ksplit.h"
#include "mx_gemm_ring.h"
#include "mxnorm.h"
#include "products.h"
#include "status.h"
#include "testing.h"

namespace mxg {

constexpr int BM = 256;    // tile rows of A (M)
constexpr int BN = 256;    // tile rows of B (N)
constexpr int NT = 512;    // threads: 8 waves, two per SIMD
constexpr int WTM = 128;   // wave tile along M
constexpr int WTN = 64;    // wave tile along N
constexpr int FM = WTM / 16, FN = WTN / 16;

// Tile v of a launch whose cells are 256 x 256 (fewer divisions than tile_of:
// they stand between two tiles' loads).
__device__ __forceinline__ void whole_tile(const Args &A, int v, int64_t &m0, int64_t &n0)
{
    int cm, cn;
    cell_of(A, xcd_range(v, A.cells), cm, cn);
    m0 = (int64_t)cm * BM;
    n0 = (int64_t)cn * BN;
}

template <int ELEM> struct Op {
    static constexpr int SB = kSB<ELEM>;
    static constexpr int STAGE = (BM + BN) * KB + (BM + BN) * SB;
};

// Per-lane part of the DMA addresses, fixed for the whole K loop: byte
// offsets, relative to the tile's first row, of the rows this lane moves.
// Wave w moves code rows 32w .. 32w+31 of both tiles (4 instructions of
// 8 rows x 128 bytes each: lane l fills LDS slot l % 8 of row l / 8 of its
// group, which holds source chunk (l % 8) ^ (l / 8)); waves 0-3 move the
// scale bytes of A's rows 64w .. 64w+63, waves 4-7 those of B's rows
// 64(w-4) .. 64(w-4)+63 (lane i of scale instruction u moves dword
// i % (SB/4) of row u (64 / (SB/4)) + i / (SB/4)).  Rows past M or N read
// row M-1 or N-1: their results are never stored.
template <int ELEM> struct Rows {
    uint32_t a[4], b[4];
    uint32_t s[Op<ELEM>::SB / 4];
};

template <int ELEM>
__device__ __forceinline__ Rows<ELEM> lane_rows(const Args &A, int64_t m0, int64_t n0, int w,
                                                int l)
{
    constexpr int DW = Op<ELEM>::SB / 4;
    Rows<ELEM> R;
    const int rr = l >> 3;       // row within the 8-row group
    const int ch = (l & 7) ^ rr; // source chunk for this LDS slot (the swizzle)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int r = 32 * w + 8 * t + rr;
        R.a[t] = (uint32_t)((min(m0 + r, A.M - 1) - m0) * A.rb) + 16 * ch;
        R.b[t] = (uint32_t)((min(n0 + r, A.N - 1) - n0) * A.rb) + 16 * ch;
    }
    const bool on_a = w < 4;
    const int64_t base = on_a ? m0 : n0, lim = on_a ? A.M : A.N;
#pragma unroll
    for (int u = 0; u < DW; ++u) {
        const int r = 64 * (w & 3) + u * (64 / DW) + l / DW;
        R.s[u] = (uint32_t)((min(base + r, lim - 1) - base) * A.rs) + 4 * (l % DW);
    }
    return R;
}

// Issue this wave's loads of K step s into one LDS stage, laid out as
// [A codes 256 x 128][B codes 256 x 128][A scales 256 x SB][B scales 256 x SB].
template <int ELEM>
__device__ __forceinline__ void issue_step(const uint8_t *ta, const uint8_t *tb,
                                           const uint8_t *tsa, const uint8_t *tsb,
                                           const Rows<ELEM> &R, int s, uint32_t stage, int w)
{
    constexpr int SB = Op<ELEM>::SB;
    constexpr int DW = SB / 4;
    const uint32_t xa = stage;
    const uint32_t xb = stage + BM * KB;
    const uint32_t kc = (uint32_t)s * KB, ks = (uint32_t)s * SB;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        lds_load16(ta, R.a[t] + kc, xa + (32 * w + 8 * t) * KB);
        lds_load16(tb, R.b[t] + kc, xb + (32 * w + 8 * t) * KB);
    }
    const uint8_t *ts = w < 4 ? tsa : tsb;
    const uint32_t xs = stage + (BM + BN) * KB + (w < 4 ? 0 : BM * SB) + 64 * (w & 3) * SB;
#pragma unroll
    for (int u = 0; u < DW; ++u)
        lds_load4(ts, R.s[u] + ks, xs + u * (64 / DW) * SB);
}

// The products of one K step from the stage at st: the step's four B
// fragments held in registers, the eight A fragments streamed, each requested
// two ahead of the products that use it.
template <int ELEM>
__device__ __forceinline__ void step_products(v4f (&acc)[FN][FM], const LDS_AS uint8_t *st,
                                              const FragBase &ba, const FragBase &bb)
{
    if constexpr (ELEM == MX_ELEM_E2M1) {
        // Whole fragments, read in the E4M3 order below (the lane's low and
        // high 16-byte chunks each feed one instruction: E2M1 blocks g and
        // 4 + g of the step).  Per column, the four tiles' products of the
        // low halves, then those of the high halves: an accumulator's two
        // instructions sit four apart, not back to back (where the second
        // waits for the first's result), in the same order of additions.
        // (Two passes over the 32 tiles, every low half and then every high
        // half from half-fragment reads, were 1.5-3% slower at the QKV and
        // gate+up shapes.)
        Frag fb[FN], fa[FM];
        fb[0] = read_frag<ELEM, 0>(st, bb);
        fb[1] = read_frag<ELEM, 1>(st, bb);
        fa[0] = read_frag<ELEM, 0>(st, ba);
        __builtin_amdgcn_sched_barrier(0);
        fb[2] = read_frag<ELEM, 2>(st, bb);
        fb[3] = read_frag<ELEM, 3>(st, bb);
        fa[1] = read_frag<ELEM, 1>(st, ba);
        __builtin_amdgcn_sched_barrier(0);
        auto column = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j + 2 < FM)
                fa[j + 2] = read_frag<ELEM, j + 2>(st, ba);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < FN; ++i)
                mma_e2m1_lo(acc[i][j], fb[i], fa[j]);
#pragma unroll
            for (int i = 0; i < FN; ++i)
                mma_e2m1_hi(acc[i][j], fb[i], fa[j]);
            __builtin_amdgcn_sched_barrier(0);
        };
        column(std::integral_constant<int, 0>{});
        column(std::integral_constant<int, 1>{});
        column(std::integral_constant<int, 2>{});
        column(std::integral_constant<int, 3>{});
        column(std::integral_constant<int, 4>{});
        column(std::integral_constant<int, 5>{});
        column(std::integral_constant<int, 6>{});
        column(std::integral_constant<int, 7>{});
        return;
    }
    // The step starts with every wave reading fragments after the barrier:
    // B0, B1 and A0 first, so that the first two products wait for three
    // fragments, not six (QKV shape: 1-3% faster).
    Frag fb[FN], fa[FM];
    fb[0] = read_frag<ELEM, 0>(st, bb);
    fb[1] = read_frag<ELEM, 1>(st, bb);
    fa[0] = read_frag<ELEM, 0>(st, ba);
    __builtin_amdgcn_sched_barrier(0);
    fb[2] = read_frag<ELEM, 2>(st, bb);
    fb[3] = read_frag<ELEM, 3>(st, bb);
    fa[1] = read_frag<ELEM, 1>(st, ba);
    __builtin_amdgcn_sched_barrier(0);
    fa[2] = read_frag<ELEM, 2>(st, ba);
    __builtin_amdgcn_sched_barrier(0);
    mma_e4m3(acc[0][0], fb[0], fa[0]);
    mma_e4m3(acc[1][0], fb[1], fa[0]);
    __builtin_amdgcn_sched_barrier(0);
    mma_e4m3(acc[2][0], fb[2], fa[0]);
    mma_e4m3(acc[3][0], fb[3], fa[0]);
    __builtin_amdgcn_sched_barrier(0);
    auto column = [&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j + 2 < FM)
            fa[j + 2] = read_frag<ELEM, j + 2>(st, ba);
        // keep the read ahead of this fragment's products
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < FN; ++i)
            mma_e4m3(acc[i][j], fb[i], fa[j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    column(std::integral_constant<int, 1>{});
    column(std::integral_constant<int, 2>{});
    column(std::integral_constant<int, 3>{});
    column(std::integral_constant<int, 4>{});
    column(std::integral_constant<int, 5>{});
    column(std::integral_constant<int, 6>{});
    column(std::integral_constant<int, 7>{});
}

template <int ELEM, int OUT>
__global__ void __launch_bounds__(NT) mx_gemm_kernel(Args A)
{
    constexpr int SB = Op<ELEM>::SB;
    constexpr int STAGE = Op<ELEM>::STAGE;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * STAGE];

    // The grid is at most one workgroup per compute unit, and workgroup b
    // takes tiles v = b, b + grid, b + 2 grid, ...
    const int G = A.cells;

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform
    const int l = tid & 63;
    const int g = l >> 4, qd = l & 15; // lane group (K block / output row quad), row in fragment
    const int wm = (w & 1) * WTM, wn = (w >> 1) * WTN;

    LDS_AS uint8_t *st0 = (LDS_AS uint8_t *)lds;
    const uint32_t st0_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)st0);
    const FragBase ba = frag_base<ELEM>(0, (BM + BN) * KB, wm, qd, g);
    const FragBase bb = frag_base<ELEM>(BM * KB, (BM + BN) * KB + BM * SB, wn, qd, g);

    int v = blockIdx.x;
    int64_t m0, n0;
    whole_tile(A, v, m0, n0);
    Rows<ELEM> R = lane_rows<ELEM>(A, m0, n0, w, l);

    // Pipeline, one barrier per K step.  At the top of a step every wave has
    // its own DMA of the step landed (vmcnt) and, past the barrier, so has
    // every other wave, and no wave still reads the other stage (the previous
    // step): the DMA of the next step goes there, and after a tile's last
    // step the DMA of the next tile's first step, which then runs under that
    // last step's products and the tile's stores.
    issue_step<ELEM>(A.a + m0 * A.rb, A.b + n0 * A.rb, A.as + m0 * A.rs, A.bs + n0 * A.rs, R, 0,
                     st0_addr, w);
    bool prev_full = false; // the previous tile lies inside H (all its stores ran)
    for (int gs = 0;;) {
        v4f acc[FN][FM];
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
                acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        const int nv = v + (int)gridDim.x;
        int64_t m1 = 0, n1 = 0;
        for (int s = 0; s < A.steps; ++s, ++gs) {
            const int cur = gs & 1;
            // this step's DMA has landed.  In a tile's first step the
            // previous tile's stores, issued after this DMA, need not have
            // completed: operations complete in order, so at most that many
            // may remain (a partial tile ran fewer stores: wait for all).
            if (s == 0 && prev_full)
                wait_vmcnt<kTileStores<OUT, FM, FN>>();
            else
                wait_vmcnt<0>();
            barrier();
            const uint32_t nxt = st0_addr + (cur ^ 1) * STAGE;
            if (s + 1 < A.steps) {
                issue_step<ELEM>(A.a + m0 * A.rb, A.b + n0 * A.rb, A.as + m0 * A.rs,
                                 A.bs + n0 * A.rs, R, s + 1, nxt, w);
            } else if (nv < G) {
                whole_tile(A, nv, m1, n1);
                R = lane_rows<ELEM>(A, m1, n1, w, l);
                issue_step<ELEM>(A.a + m1 * A.rb, A.b + n1 * A.rb, A.as + m1 * A.rs,
                                 A.bs + n1 * A.rs, R, 0, nxt, w);
            }
            step_products<ELEM>(acc, st0 + cur * STAGE, ba, bb);
        }
        store_tile<OUT, FM, FN>(A, acc, m0, n0, wm, wn, g, qd);
        prev_full = m0 + BM <= A.M && n0 + BN <= A.N;
        if (nv >= G)
            break;
        v = nv;
        m0 = m1;
        n0 = n1;
    }
}

template <int ELEM, int OUT>
hipError_t launch(const Args &A, hipStream_t stream)
{
    const int G = A.cells;
    const int grid = G < A.grid_max ? G : A.grid_max;
    hipLaunchKernelGGL((mx_gemm_kernel<ELEM, OUT>), dim3((unsigned)grid), dim3(NT), 0, stream, A);
    return hipGetLastError();
}

// ------------------------------------------------- two products, one launch --

// Two products in one persistent launch, so that the last, partly empty round
// of one is filled with tiles of the other (the weight gradient's 384 tiles
// on 256 compute units leave half of them idle for a round of 256 K steps).
// A step takes about 2 us whether all compute units or half of them run, so
// the fullest workgroup's load is the time.  Measured against the two
// launches: 6144 x 4096 x 32768 with 32768 x 4096 x 6144 (E4M3) 1795 -> 1690
// us, 6144 x 4096 x 4096 with 4096 x 4096 x 6144 142 -> 130 us (E2M1) and 216
// -> 199 us (E4M3).
// Workgroup b is of class b >= split; a workgroup of class c takes n[c][0]
// tiles of product 0 (float output), then n[c][1] of product 1 (bf16 output).
struct PairArgs {
    Args p[2];
    int split; // workgroups of class 0
    int n[2][2];
};

// Product i's tile that is number j of workgroup b's share: the shares both
// classes have in whole rounds over the grid, the rest in rounds over the
// class that has more.  Past the product's last tile: -1.
__device__ __forceinline__ int pair_tile(const PairArgs &W, int i, int j, int b, int grid)
{
    const int c = b >= W.split;
    const int both = min(W.n[0][i], W.n[1][i]);
    const int first = c ? W.split : 0, size = c ? grid - W.split : W.split;
    const int v = j < both ? j * grid + b : both * grid + (j - both) * size + (b - first);
    return j < W.n[c][i] && v < W.p[i].cells ? v : -1;
}

template <int ELEM> __global__ void __launch_bounds__(NT) mx_gemm_pair_kernel(PairArgs W)
{
    constexpr int SB = Op<ELEM>::SB;
    constexpr int STAGE = Op<ELEM>::STAGE;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * STAGE];

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform
    const int l = tid & 63;
    const int g = l >> 4, qd = l & 15;
    const int wm = (w & 1) * WTM, wn = (w >> 1) * WTN;
    const int b = blockIdx.x, grid = gridDim.x;

    LDS_AS uint8_t *st0 = (LDS_AS uint8_t *)lds;
    const uint32_t st0_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)st0);
    const FragBase ba = frag_base<ELEM>(0, (BM + BN) * KB, wm, qd, g);
    const FragBase bb = frag_base<ELEM>(BM * KB, (BM + BN) * KB + BM * SB, wn, qd, g);

    // tile number j of product i, and the one after it
    int i = 0, j = 0, v = pair_tile(W, 0, 0, b, grid);
    if (v < 0) {
        i = 1;
        v = pair_tile(W, 1, 0, b, grid);
        if (v < 0)
            return;
    }
    int64_t m0, n0;
    whole_tile(W.p[i], v, m0, n0);
    Rows<ELEM> R = lane_rows<ELEM>(W.p[i], m0, n0, w, l);
    const uint8_t *ta = W.p[i].a + m0 * W.p[i].rb, *tb = W.p[i].b + n0 * W.p[i].rb;
    const uint8_t *tsa = W.p[i].as + m0 * W.p[i].rs, *tsb = W.p[i].bs + n0 * W.p[i].rs;

    // the pipeline of mx_gemm_kernel
    issue_step<ELEM>(ta, tb, tsa, tsb, R, 0, st0_addr, w);
    int stores = 0; // stores of the previous tile, if it lies inside its H
    for (int gs = 0;;) {
        v4f acc[FN][FM];
#pragma unroll
        for (int n = 0; n < FN; ++n)
#pragma unroll
            for (int m = 0; m < FM; ++m)
                acc[n][m] = v4f{0.f, 0.f, 0.f, 0.f};
        int ni = i, nj = j + 1, nv = pair_tile(W, i, nj, b, grid);
        if (nv < 0 && i == 0) {
            ni = 1;
            nj = 0;
            nv = pair_tile(W, 1, 0, b, grid);
        }
        int64_t m1 = 0, n1 = 0;
        const int steps = W.p[i].steps;
        for (int s = 0; s < steps; ++s, ++gs) {
            const int cur = gs & 1;
            if (s == 0 && stores == kTileStores<MX_OUT_F32, FM, FN>)
                wait_vmcnt<kTileStores<MX_OUT_F32, FM, FN>>();
            else if (s == 0 && stores == kTileStores<MX_OUT_BF16, FM, FN>)
                wait_vmcnt<kTileStores<MX_OUT_BF16, FM, FN>>();
            else
                wait_vmcnt<0>();
            barrier();
            const uint32_t nxt = st0_addr + (cur ^ 1) * STAGE;
            if (s + 1 < steps) {
                issue_step<ELEM>(ta, tb, tsa, tsb, R, s + 1, nxt, w);
            } else if (nv >= 0) {
                const Args &A = W.p[ni];
                whole_tile(A, nv, m1, n1);
                R = lane_rows<ELEM>(A, m1, n1, w, l);
                ta = A.a + m1 * A.rb;
                tb = A.b + n1 * A.rb;
                tsa = A.as + m1 * A.rs;
                tsb = A.bs + n1 * A.rs;
                issue_step<ELEM>(ta, tb, tsa, tsb, R, 0, nxt, w);
            }
            step_products<ELEM>(acc, st0 + cur * STAGE, ba, bb);
        }
        const bool full = m0 + BM <= W.p[i].M && n0 + BN <= W.p[i].N;
        if (i == 0) {
            store_tile<MX_OUT_F32, FM, FN>(W.p[0], acc, m0, n0, wm, wn, g, qd);
            stores = full ? kTileStores<MX_OUT_F32, FM, FN> : 0;
        } else {
            store_tile<MX_OUT_BF16, FM, FN>(W.p[1], acc, m0, n0, wm, wn, g, qd);
            stores = full ? kTileStores<MX_OUT_BF16, FM, FN> : 0;
        }
        if (nv < 0)
            break;
        i = ni;
        j = nj;
        v = nv;
        m0 = m1;
        n0 = n1;
    }
}

// ------------------------------------------------------- choice of kernel --

// Ring tiles: 4 waves, two workgroups per compute unit.
using R64x128 = Ring<64, 128, 2, 2, 3>;
using R128x128 = Ring<128, 128, 2, 2, 2>;
// K-split tiles: 8 waves, one workgroup per compute unit.
using K16x32 = KSplit<16, 32, 8, 3>;
using K32x32 = KSplit<32, 32, 8, 2>;
using K32x64 = KSplit<32, 64, 8, 1>;
using K64x64 = KSplit<64, 64, 8, 1>;

enum Shape { S_K16x32, S_K32x32, S_K32x64, S_K64x64, S_R64x128, S_R128x128, S_256x256, S_COUNT };

// What a launch of each tile shape costs on MI355X, fitted to times at K =
// 512 .. 8192 and 64 to 3400 tiles: us once per launch, per round of tiles
// (their stores, and for the K-split kernel the start of a tile's loads, which
// nothing overlaps) and per K step of a round.  Below 256 x 256 the time per
// step is the tile's operand bytes at about 55 GB/s per compute unit, so a
// larger tile does more products per byte and a smaller one leaves fewer
// compute units idle.
//
// With few K steps a smaller tile's latency is not covered (a ring waits for
// the stores of the tile before, a K-split tile for its only step): many
// rounds take `few` + steps * `few_step` each at least.  At one K step, bf16,
// 128 x 128 tiles then take 2.3-2.5 us a round, not 1.4, and lose to 256 x
// 256: 9526 x 22336 129 against 106 us, 142102 x 1152 97 against 70.  Counted
// from the ninth round on for the rings (with fewer rounds 256 x 256 tiles do
// not reach their pace either: two K steps, 3 to 8 rounds, the rings are 1.05
// to 1.4 times as fast in the median of each output type), from the first if N leaves half of the
// 64 x 128 tile empty (63697 x 48 10.5 against 8.0), and for the K-split tiles
// beyond two rounds.  Over 1000 sizes of 1 to 4 steps and 1e6 to 2e8 outputs
// the choice was more than 3% slower than 256 x 256 tiles at 106, by up to 28%,
// and is now at 35, 32 of them of one step, by up to 16%; on average it is
// 1.15 times as fast as those.
//
// An estimate ranks the shapes; it does not predict the time.  It has no term
// for operands that come from HBM rather than L2, nor for the output's type:
// 61 x 28672 x 4096 is put at 17 us in E4M3 and takes 34, and at 10 in E2M1
// and takes 14.
struct Cost {
    int bm, bn;
    float once, round, step, few, few_step;
};
constexpr Cost kCost[S_COUNT] = {
    {16, 32, 1.3f, 1.0f, 0.14f, 1.6f, 0.0f},   {32, 32, 1.4f, 1.1f, 0.14f, 1.9f, 0.0f},
    {32, 64, 2.2f, 0.7f, 0.19f, 2.15f, 0.0f},  {64, 64, 0.4f, 2.6f, 0.275f, 2.9f, 0.2f},
    {64, 128, 3.1f, 0.4f, 0.425f, 1.1f, 0.3f}, {128, 128, 4.1f, 0.8f, 0.59f, 1.8f, 0.45f},
    {256, 256, 1.2f, 4.0f, 1.75f, 0.0f, 0.0f},
};

// us a launch over `cells` outputs of cm x cn takes on `cus` compute units
inline double launch_cost(int shape, int64_t cells, int64_t cm, int64_t cn, int steps, int cus)
{
    const Cost &c = kCost[shape];
    const int64_t tiles = cells * ((cm + c.bm - 1) / c.bm) * ((cn + c.bn - 1) / c.bn);
    const int64_t rounds = (tiles + cus - 1) / cus;
    const double per = c.round + (double)steps * c.step;
    const double few = std::max(per, (double)c.few + (double)steps * c.few_step);
    if (shape <= S_K64x64)
        return c.once + (double)rounds * (rounds > 2 ? few : per);
    double us = (double)rounds * per + (double)std::max<int64_t>(0, rounds - 8) * (few - per);
    if (shape == S_R64x128 && cn <= 64 && rounds > 2)
        us = std::max(us, (double)rounds * (1.3 + 0.3 * (double)steps));
    return c.once + us;
}

// How one product is computed: the whole output in tiles of `shape`; or, where
// that is at least 5% cheaper, its first `whole` cells of 256 x 256 (whole
// rounds of them) in one launch and the cells left in tiles of `tail` in a
// second.
struct Plan {
    int shape;
    int whole, tail; // whole = 0: one launch
    double us;
};

inline Plan plan_product(int64_t M, int64_t N, int steps, int cus)
{
    Plan P{S_256x256, 0, 0, launch_cost(S_256x256, 1, M, N, steps, cus)};
    for (int s = 0; s < S_256x256; ++s) {
        const double c = launch_cost(s, 1, M, N, steps, cus);
        if (c < P.us) {
            P.us = c;
            P.shape = s;
        }
    }
    const int64_t cells = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    const int64_t whole = cells / cus * cus, left = cells - whole;
    if (whole && left) {
        int tail = 0;
        double tcost = launch_cost(0, left, BM, BN, steps, cus);
        for (int s = 1; s < S_256x256; ++s) {
            const double c = launch_cost(s, left, BM, BN, steps, cus);
            if (c < tcost) {
                tcost = c;
                tail = s;
            }
        }
        const double two = launch_cost(S_256x256, whole, BM, BN, steps, cus) + tcost;
        if (two < 0.95 * P.us)
            P = Plan{S_256x256, (int)whole, tail, two};
    }
    return P;
}

template <int ELEM, int OUT> hipError_t launch_shape(int shape, const Args &A, hipStream_t stream)
{
    switch (shape) {
    case S_K16x32: return launch_ksplit<ELEM, OUT, K16x32>(A, stream);
    case S_K32x32: return launch_ksplit<ELEM, OUT, K32x32>(A, stream);
    case S_K32x64: return launch_ksplit<ELEM, OUT, K32x64>(A, stream);
    case S_K64x64: return launch_ksplit<ELEM, OUT, K64x64>(A, stream);
    case S_R64x128: return launch_ring<ELEM, OUT, R64x128>(A, stream);
    case S_R128x128: return launch_ring<ELEM, OUT, R128x128>(A, stream);
    default: return launch<ELEM, OUT>(A, stream);
    }
}

template <int ELEM, int OUT>
hipError_t multiply_as(const Plan &P, Args A, hipStream_t stream)
{
    set_tiles(A, kCost[P.shape].bm, kCost[P.shape].bn, 1024);
    if (!P.whole)
        return launch_shape<ELEM, OUT>(P.shape, A, stream);
    const int left = A.cells - P.whole;
    A.cells = P.whole;
    const hipError_t e = launch<ELEM, OUT>(A, stream);
    if (e != hipSuccess)
        return e;
    A.pid0 = P.whole;
    A.cells = left;
    A.sub_m = BM / kCost[P.tail].bm;
    A.sub_n = BN / kCost[P.tail].bn;
    return launch_shape<ELEM, OUT>(P.tail, A, stream);
}

template <int ELEM, int OUT> hipError_t multiply(const Args &A, hipStream_t stream)
{
    return multiply_as<ELEM, OUT>(plan_product(A.M, A.N, A.steps, A.grid_max), A, stream);
}

// Shares of the two products' tiles for `cus` workgroups that make the
// fullest workgroup's load, in steps, as small as two classes of workgroups
// can: class 0 takes n0 tiles of product 0, class 1 takes n1 > n0, and both
// fill what the load leaves with tiles of product 1.  A tile costs its K
// steps and about two steps' time for its stores.  Returns the load, or 0 if
// the products have too many tiles to search.
inline int64_t pair_plan(PairArgs &W, int cus)
{
    constexpr int kTileSteps = 2;
    const int64_t g0 = W.p[0].cells, g1 = W.p[1].cells;
    const int64_t c0 = W.p[0].steps + kTileSteps, c1 = W.p[1].steps + kTileSteps;
    const int64_t q = g0 / cus;
    if (q > 16 || g1 / cus > 4096)
        return 0;
    const int64_t lower = (g0 * c0 + g1 * c1 + cus - 1) / cus;
    int64_t best = 0;
    // the load of some workgroup is a * c0 + b * c1: for each a and pair of
    // shares, the smallest such load that holds both products
    for (int64_t lo = 0; lo <= q; ++lo)
        for (int64_t hi = q + 1; hi <= q + 3; ++hi) {
            // workgroups of class 1: the fewest that take the rest of product
            // 0, in eights, so that a tile number keeps its workgroup's XCD
            const int64_t k =
                std::max<int64_t>(0, (g0 - lo * cus + (hi - lo) - 1) / (hi - lo) + 7) / 8 * 8;
            if (k > cus)
                continue;
            for (int side = 0; side < 2; ++side) {
                const int64_t a = side ? hi : lo;
                int64_t b = lower > a * c0 ? (lower - a * c0 + c1 - 1) / c1 : 0;
                for (int t = 0; t < 4; ++t, ++b) {
                    const int64_t load = a * c0 + b * c1;
                    if (load < (k ? hi : lo) * c0 || (best && load >= best))
                        continue;
                    const int64_t b0 = (load - lo * c0) / c1, b1 = k ? (load - hi * c0) / c1 : 0;
                    if ((cus - k) * b0 + k * b1 < g1)
                        continue;
                    best = load;
                    W.split = (int)(cus - k);
                    W.n[0][0] = (int)lo;
                    W.n[0][1] = (int)b0;
                    W.n[1][0] = (int)hi;
                    W.n[1][1] = (int)b1;
                }
            }
        }
    return best;
}

// How two products are computed: one launch each, or in one launch on 256 x
// 256 tiles shared out by load or on 64 x 128 tiles that are all resident at
// once, where that is 3% cheaper.
enum PairMode { PAIR_APART, PAIR_LARGE, PAIR_SMALL };
struct PairPlan {
    int mode;
    bool can_large;             // the shares of the large tiles were found
    double apart, large, small; // us; large or small = apart: not possible
    PairArgs W;
    RingPair Q;
};

inline void plan_pair(PairPlan &P, const Args &A0, const Args &A1)
{
    const int cus = A0.grid_max;
    P.apart = plan_product(A0.M, A0.N, A0.steps, cus).us + plan_product(A1.M, A1.N, A1.steps, cus).us;
    P.W.p[0] = A0;
    P.W.p[1] = A1;
    set_tiles(P.W.p[0], BM, BN, 1024);
    set_tiles(P.W.p[1], BM, BN, 1024);
    const int64_t load = pair_plan(P.W, cus);
    P.can_large = load != 0;
    P.large = load ? kCost[S_256x256].once + (double)load * kCost[S_256x256].step : P.apart;

    // two workgroups of 64 x 128 tiles per compute unit
    constexpr Cost c = kCost[S_R64x128];
    P.Q.p[0] = A0;
    P.Q.p[1] = A1;
    set_tiles(P.Q.p[0], c.bm, c.bn, 1024);
    set_tiles(P.Q.p[1], c.bm, c.bn, 1024);
    P.Q.n0 = P.Q.p[0].cells;
    P.Q.n1 = P.Q.p[1].cells;
    P.Q.second_first = A1.steps > A0.steps;
    P.small = P.apart;
    if ((int64_t)P.Q.n0 + P.Q.n1 <= 2 * (int64_t)cus) {
        const double steps = std::max((double)std::max(A0.steps, A1.steps),
                                      ((double)P.Q.n0 * A0.steps + (double)P.Q.n1 * A1.steps) / cus);
        P.small = c.once + c.round + 1.2 * steps * c.step; // two loads share the step
    }
    P.mode = P.small <= P.large && P.small < 0.97 * P.apart ? PAIR_SMALL
             : P.large < 0.97 * P.apart                     ? PAIR_LARGE
                                                            : PAIR_APART;
}

// Products 0 (float output) and 1 (bf16 output) on one stream.
template <int ELEM>
hipError_t multiply_pair_as(const PairPlan &P, const Args &A0, const Args &A1, hipStream_t stream)
{
    if (P.mode == PAIR_SMALL) {
        hipLaunchKernelGGL((mx_gemm_ring_pair_kernel<ELEM, R64x128>),
                           dim3((unsigned)(P.Q.n0 + P.Q.n1)), dim3(R64x128::NT), 0, stream, P.Q);
        return hipGetLastError();
    }
    if (P.mode == PAIR_LARGE) {
        hipLaunchKernelGGL((mx_gemm_pair_kernel<ELEM>), dim3((unsigned)A0.grid_max), dim3(NT), 0,
                           stream, P.W);
        return hipGetLastError();
    }
    const hipError_t e = multiply<ELEM, MX_OUT_BF16>(A1, stream);
    return e != hipSuccess ? e : multiply<ELEM, MX_OUT_F32>(A0, stream);
}

template <int ELEM> hipError_t multiply_pair(const Args &A0, const Args &A1, hipStream_t stream)
{
    PairPlan P;
    plan_pair(P, A0, A1);
    return multiply_pair_as<ELEM>(P, A0, A1, stream);
}

} // namespace mxg

// host side -------------------------------------------------------------------

namespace {

bool aligned(const void *p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

// Compute units of the device `stream` runs on (the current device for the
// null stream), looked up once per device; 0 if unknown.
int compute_units(hipStream_t stream)
{
    static std::atomic<int> cache[64];
    int dev = -1;
    if (stream) {
        hipDevice_t hd;
        if (hipStreamGetDevice(static_cast<hipStream_t>(stream), &hd) != hipSuccess)
            return 0;
        dev = (int)hd;
    } else if (hipGetDevice(&dev) != hipSuccess) {
        return 0;
    }
    if (dev < 0 || dev >= 64)
        return 0;
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            return 0;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

} // namespace

namespace mxg {

mx_status check_product(const Product &P, int block, int elem, int out_dtype)
{
    if (P.M < 0 || P.N < 0 || P.K <= 0)
        return mxk::fail(MX_EINVAL, "M and N must be >= 0 and K > 0");
    if (elem != MX_ELEM_E4M3 && elem != MX_ELEM_E2M1)
        return mxk::fail(MX_EINVAL, "elem must be MX_ELEM_E4M3 or MX_ELEM_E2M1");
    if (out_dtype != MX_OUT_F32 && out_dtype != MX_OUT_BF16)
        return mxk::fail(MX_EINVAL, "out_dtype must be MX_OUT_F32 or MX_OUT_BF16");
    if (block != 32)
        return mxk::fail(MX_EUNSUPPORTED, "the matrix cores apply one scale per 32 elements: block must be 32");
    const int64_t kstep = elem == MX_ELEM_E2M1 ? 256 : 128;
    if (P.K % kstep != 0)
        return mxk::fail(MX_EUNSUPPORTED, "K must be a multiple of 128 (E4M3) or 256 (E2M1)");
    if (P.N % 16 != 0)
        return mxk::fail(MX_EUNSUPPORTED, "N must be a multiple of 16");
    if (P.K > MX_MATMUL_MAX_K)
        return mxk::fail(MX_EUNSUPPORTED, "K exceeds %d", MX_MATMUL_MAX_K);
    if (P.M == 0 || P.N == 0)
        return MX_OK;
    if (!P.a || !P.as || !P.b || !P.bs || !P.out)
        return mxk::fail(MX_EINVAL, "NULL pointer");
    if (!aligned(P.a, 16) || !aligned(P.b, 16) || !aligned(P.as, 4) || !aligned(P.bs, 4) ||
        !aligned(P.out, 16) || (P.gain && !aligned(P.gain, 8)))
        return mxk::fail(MX_EINVAL, "codes and out must be 16-byte, scales 4-byte and b_gain "
                               "8-byte aligned");
    const int64_t tm = (P.M + BM - 1) / BM, tn = (P.N + BN - 1) / BN;
    if (tm * tn > INT32_MAX / 2 || P.M > INT32_MAX || P.N > MX_MATMUL_MAX_N)
        return mxk::fail(MX_EUNSUPPORTED, "problem too large (N at most %d)", MX_MATMUL_MAX_N);
    return MX_OK;
}

} // namespace mxg

namespace {

// A checked product's kernel arguments.
void product_args(mxg::Args &A, const mxg::Product &P, int elem, hipStream_t stream)
{
    A.a = P.a;
    A.as = P.as;
    A.b = P.b;
    A.bs = P.bs;
    A.bgain = static_cast<const uint16_t *>(P.gain);
    A.out = P.out;
    A.M = P.M;
    A.N = P.N;
    A.rb = elem == MX_ELEM_E2M1 ? P.K / 2 : P.K;
    A.rs = P.K / 32;
    A.steps = (int)(A.rb / mxg::KB);
    const int cus = compute_units(stream);
    A.grid_max = cus > 0 ? cus : 256;
}

} // namespace

extern "C" {

mx_status mx_matmul_fwd(const uint8_t *a_codes, const uint8_t *a_scales, const uint8_t *b_codes,
                        const uint8_t *b_scales, int64_t M, int64_t N, int64_t K, int block,
                        int elem, const void *b_gain, int out_dtype, void *out, hipStream_t stream)
{
    mxk::clear_error();
    const mxg::Product P{a_codes, a_scales, b_codes, b_scales, M, N, K, b_gain, out};
    const mx_status ok = mxg::check_product(P, block, elem, out_dtype);
    if (ok != MX_OK || M == 0 || N == 0)
        return ok;
    mxg::Args A;
    product_args(A, P, elem, stream);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (elem == MX_ELEM_E4M3)
        e = out_dtype == MX_OUT_F32 ? mxg::multiply<MX_ELEM_E4M3, MX_OUT_F32>(A, st)
                                         : mxg::multiply<MX_ELEM_E4M3, MX_OUT_BF16>(A, st);
    else
        e = out_dtype == MX_OUT_F32 ? mxg::multiply<MX_ELEM_E2M1, MX_OUT_F32>(A, st)
                                         : mxg::multiply<MX_ELEM_E2M1, MX_OUT_BF16>(A, st);
    if (e != hipSuccess)
        return mxk::fail(MX_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
    return MX_OK;
}

} // extern "C"

namespace mxg {

mx_status matmul_pair(const Product &f32, const Product &bf16, int elem, hipStream_t stream)
{
    Args A0, A1;
    product_args(A0, f32, elem, stream);
    product_args(A1, bf16, elem, stream);
    const hipError_t e = elem == MX_ELEM_E4M3 ? multiply_pair<MX_ELEM_E4M3>(A0, A1, stream)
                                              : multiply_pair<MX_ELEM_E2M1>(A0, A1, stream);
    return e == hipSuccess ? MX_OK
                           : mxk::fail(MX_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
}

} // namespace mxg

// ---------------------------------------------------- for the library's tests --

namespace {

bool known_shape(int s) { return s >= 0 && s < mxg::S_COUNT; }

template <int ELEM>
hipError_t multiply_as(const mxg::Plan &P, const mxg::Args &A, int out_dtype, hipStream_t stream)
{
    return out_dtype == MX_OUT_F32 ? mxg::multiply_as<ELEM, MX_OUT_F32>(P, A, stream)
                                   : mxg::multiply_as<ELEM, MX_OUT_BF16>(P, A, stream);
}

// M, N and the K steps alone: what the plans depend on.
bool plan_args(mxg::Args &A, int64_t M, int64_t N, int64_t K, int elem, int units)
{
    const int64_t rb = elem == MX_ELEM_E2M1 ? K / 2 : K;
    if (M <= 0 || N <= 0 || K <= 0 || rb % mxg::KB != 0 || units <= 0)
        return false;
    A = mxg::Args{};
    A.M = M;
    A.N = N;
    A.steps = (int)(rb / mxg::KB);
    A.grid_max = units;
    return true;
}

} // namespace

extern "C" {

int mxt_product_plan(int64_t M, int64_t N, int64_t K, int elem, int units, int *whole, int *tail,
                     double *us)
{
    mxg::Args A;
    if (!plan_args(A, M, N, K, elem, units))
        return -1;
    const mxg::Plan P = mxg::plan_product(M, N, A.steps, units);
    *whole = P.whole;
    *tail = P.tail;
    *us = P.us;
    return P.shape;
}

int mxt_pair_plan(int64_t M0, int64_t N0, int64_t K0, int64_t M1, int64_t N1, int64_t K1, int elem,
                  int units, double *us)
{
    mxg::Args A0, A1;
    if (!plan_args(A0, M0, N0, K0, elem, units) || !plan_args(A1, M1, N1, K1, elem, units))
        return -1;
    mxg::PairPlan P;
    mxg::plan_pair(P, A0, A1);
    us[0] = P.apart;
    us[1] = P.large;
    us[2] = P.small;
    return P.mode;
}

mx_status mxt_matmul(const uint8_t *a_codes, const uint8_t *a_scales, const uint8_t *b_codes,
                     const uint8_t *b_scales, int64_t M, int64_t N, int64_t K, int elem,
                     const void *b_gain, int out_dtype, void *out, int shape, int whole, int units,
                     hipStream_t stream)
{
    mxk::clear_error();
    const mxg::Product P0{a_codes, a_scales, b_codes, b_scales, M, N, K, b_gain, out};
    const mx_status ok = mxg::check_product(P0, 32, elem, out_dtype);
    if (ok != MX_OK || M == 0 || N == 0)
        return ok;
    mxg::Args A;
    product_args(A, P0, elem, stream);
    const int64_t cells = ((M + mxg::BM - 1) / mxg::BM) * ((N + mxg::BN - 1) / mxg::BN);
    if (!known_shape(shape) || whole < 0 || whole >= cells || units < 0 || units > A.grid_max)
        return mxk::fail(MX_EINVAL, "no such tile shape, first launch or number of units");
    if (units)
        A.grid_max = units;
    const mxg::Plan P{whole ? (int)mxg::S_256x256 : shape, whole, shape, 0.0};
    const hipError_t e = elem == MX_ELEM_E4M3 ? multiply_as<MX_ELEM_E4M3>(P, A, out_dtype, stream)
                                              : multiply_as<MX_ELEM_E2M1>(P, A, out_dtype, stream);
    return e == hipSuccess ? MX_OK
                           : mxk::fail(MX_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
}

mx_status mxt_matmul_pair(const MxtProduct *f32, const MxtProduct *bf16, int elem, int mode,
                          int units, hipStream_t stream)
{
    mxk::clear_error();
    const mxg::Product p0{f32->a, f32->as, f32->b, f32->bs, f32->M, f32->N, f32->K, f32->gain, f32->out};
    const mxg::Product p1{bf16->a, bf16->as, bf16->b, bf16->bs, bf16->M, bf16->N, bf16->K, bf16->gain,
                          bf16->out};
    mx_status ok = mxg::check_product(p0, 32, elem, MX_OUT_F32);
    if (ok == MX_OK)
        ok = mxg::check_product(p1, 32, elem, MX_OUT_BF16);
    if (ok != MX_OK)
        return ok;
    mxg::Args A0, A1;
    product_args(A0, p0, elem, stream);
    product_args(A1, p1, elem, stream);
    if (f32->M == 0 || f32->N == 0 || bf16->M == 0 || bf16->N == 0 || units < 0 ||
        units > A0.grid_max)
        return mxk::fail(MX_EINVAL, "empty product, or no such number of units");
    if (units)
        A0.grid_max = A1.grid_max = units;
    mxg::PairPlan P;
    mxg::plan_pair(P, A0, A1);
    if (mode < 0 || mode > mxg::PAIR_SMALL || (mode == mxg::PAIR_LARGE && !P.can_large))
        return mxk::fail(MX_EINVAL, "no such pair launch");
    P.mode = mode;
    const hipError_t e = elem == MX_ELEM_E4M3
                             ? mxg::multiply_pair_as<MX_ELEM_E4M3>(P, A0, A1, stream)
                             : mxg::multiply_pair_as<MX_ELEM_E2M1>(P, A0, A1, stream);
    return e == hipSuccess ? MX_OK
                           : mxk::fail(MX_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
}

} // extern "C"
