// mx_gemm.h -- what the MX product kernels share: argument block, tile order,
// LDS DMA, fragment reads, output stores.  mx_gemm.hip holds the entry point,
// the choice of kernel and the 256 x 256 kernel; mx_gemm_ring.h smaller tiles
// with a deeper ring of K steps; mx_gemm_ksplit.h few small tiles, their K
// steps dealt to the waves.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "mxnorm.h"

namespace mxg {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))

constexpr int KB = 128;    // bytes of each row per K step
constexpr int NXCD = 8;

// scale bytes per row and K step: 4 blocks of 32 (E4M3), 8 blocks (E2M1)
template <int ELEM> constexpr int kSB = ELEM == MX_ELEM_E2M1 ? 8 : 4;

struct Args {
    const uint8_t *a, *as, *b, *bs;
    const uint16_t *bgain; // bf16 [N] or NULL
    void *out;
    int64_t M, N;
    int64_t rb;   // code bytes per row
    int64_t rs;   // scale bytes per row
    int steps;    // K steps of KB bytes
    // The output is cut into cells of cell_m x cell_n elements, tiles_m x
    // tiles_n of them, numbered in groups of `group` cell rows that share
    // operand blocks.  A launch computes cells pid0 .. pid0 + cells - 1, each
    // as sub_m x sub_n tiles of the kernel's size.
    int tiles_m, tiles_n, group;
    int cell_m, cell_n, sub_m, sub_n;
    int pid0, cells;
    int grid_max;   // workgroups resident at once
};

// The whole output as bm x bn cells of one tile each, in groups of
// `group_rows` output rows.
inline void set_tiles(Args &A, int bm, int bn, int group_rows)
{
    A.tiles_m = (int)((A.M + bm - 1) / bm);
    A.tiles_n = (int)((A.N + bn - 1) / bn);
    A.group = group_rows / bm;
    A.cell_m = bm;
    A.cell_n = bn;
    A.sub_m = A.sub_n = 1;
    A.pid0 = 0;
    A.cells = A.tiles_m * A.tiles_n;
}

// Cell number t of the launch, counted in the launch's order: its row and
// column of cells.
__device__ __forceinline__ void cell_of(const Args &A, int t, int &cm, int &cn)
{
    const int pid = A.pid0 + t;
    const int in_group = A.group * A.tiles_n;
    const int first_m = (pid / in_group) * A.group;
    const int gsz = min(A.tiles_m - first_m, A.group);
    cm = first_m + (pid % in_group) % gsz;
    cn = (pid % in_group) / gsz;
}

// Dispatch is round robin over the XCDs (each with its own L2): tile v of G,
// renumbered so that each XCD runs a contiguous range (256 x 256 tiles, E4M3,
// against plain round robin: 32768 x 6144 x 4096 737 against 801 us, 16384 x
// 28672 x 4096 1583 against 1715).
__device__ __forceinline__ int xcd_range(int v, int G)
{
    const int xcd = v % NXCD, loc = v / NXCD;
    const int q = G / NXCD, rem = G % NXCD;
    return xcd < rem ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
}

// Tile v of a launch: its first row and column.
__device__ __forceinline__ void tile_of(const Args &A, int bm, int bn, int v, int64_t &m0,
                                        int64_t &n0)
{
    const int nsub = A.sub_m * A.sub_n;
    const int t = xcd_range(v, A.cells * nsub), sub = t % nsub;
    int cm, cn;
    cell_of(A, t / nsub, cm, cn);
    m0 = (int64_t)cm * A.cell_m + (sub % A.sub_m) * bm;
    n0 = (int64_t)cn * A.cell_n + (sub / A.sub_m) * bn;
}

// Global -> LDS DMA loads: lane i of the wave reads gbase + off_i (gbase
// wave-uniform, in SGPRs; off_i a 32-bit lane offset) and writes the bytes at
// LDS address lds_base + bytes * i (lds_base wave-uniform, passed in M0).
// Written as inline asm rather than with the compiler builtin: for the builtin
// the compiler cannot tell that the LDS reads of one stage do not alias the
// DMA into the other, and would wait for the prefetch before every read.  The
// waits are explicit (wait_vmcnt) instead.  An LDS DMA needs one wait state
// after the scalar write of M0 that the compiler places just before the asm:
// hence the s_nop.
__device__ __forceinline__ void lds_load16(const void *gbase, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(gbase),
                 "{m0}"(lds_base)
                 : "memory");
}

__device__ __forceinline__ void lds_load4(const void *gbase, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(gbase),
                 "{m0}"(lds_base)
                 : "memory");
}

// The same with a whole address per lane.
__device__ __forceinline__ void lds_load4(const void *p, uint32_t lds_base)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(p), "{m0}"(lds_base) : "memory");
}

// Wait until at most N_ of this wave's vector memory operations (loads and
// stores, which complete in issue order) are outstanding.
template <int N_> __device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N_) : "memory");
}

// Wait until at most `ahead` steps' loads (L each, ahead <= N) are
// outstanding.  Stores issued in between only make the wait stricter.
template <int L, int N> __device__ __forceinline__ void wait_steps(int ahead)
{
    if (ahead >= N)
        wait_vmcnt<N * L>();
    else if constexpr (N > 0)
        wait_steps<L, N - 1>(ahead);
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence
// would wait for every outstanding load, including the DMA of the next step.
// LDS written by the DMA is covered by the vmcnt wait each wave makes before
// arriving; the lgkmcnt(0) completes this wave's own LDS reads, so that a
// stage read before the barrier can be refilled after it.  The "memory"
// clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ v8i join(u32x4 lo, u32x4 hi)
{
    return __builtin_bit_cast(v8i, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// two floats to bf16 (round to nearest even, on gfx950's conversion unit),
// the first in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const __bf16 x = (__bf16)a, y = (__bf16)b;
    return (uint32_t)__builtin_bit_cast(uint16_t, x) |
           ((uint32_t)__builtin_bit_cast(uint16_t, y) << 16);
}

// One operand fragment for a 16-row group and one K step: lane (g, q) holds
// the 16-byte chunks g and 4+g of row r (E4M3: k = 16g..16g+15 and
// 64+16g..64+16g+15 of the step, the matrix core's own k order for this
// operand size; E2M1: chunk g is the 32-element block g of the first
// instruction, chunk 4+g block g of the second) and the E8M0 scale bytes of
// the blocks it supplies (E4M3: block g; E2M1: blocks g and 4+g).
struct Frag {
    v8i v;
    int s0, s1;
};

// Lane-relative LDS offsets of one operand's fragments within a stage: the
// lane reads row r0 + qd (+16 j for fragment j) at chunks g and 4 + g,
// swizzled by (r0 + qd) & 7 = qd & 7 (r0 is a multiple of 16), and the
// scale bytes g (and 4 + g) of that row.
struct FragBase {
    uint32_t lo, hi, sc;
};

template <int ELEM>
__device__ __forceinline__ FragBase frag_base(uint32_t codes_off, uint32_t scales_off, int r0,
                                              int qd, int g)
{
    constexpr int SB = kSB<ELEM>;
    FragBase b;
    b.lo = codes_off + (r0 + qd) * KB + 16 * (g ^ (qd & 7));
    b.hi = codes_off + (r0 + qd) * KB + 16 * ((4 + g) ^ (qd & 7));
    b.sc = scales_off + (r0 + qd) * SB + g;
    return b;
}

// fragment J of an operand from the stage at st; the row offset J*16 rows is
// a compile-time constant that the LDS reads take as their immediate offset
template <int ELEM, int J>
__device__ __forceinline__ Frag read_frag(const LDS_AS uint8_t *st, const FragBase &b)
{
    constexpr int SB = kSB<ELEM>;
    Frag f;
    const u32x4 lo = *reinterpret_cast<const LDS_AS u32x4 *>(st + b.lo + J * 16 * KB);
    const u32x4 hi = *reinterpret_cast<const LDS_AS u32x4 *>(st + b.hi + J * 16 * KB);
    f.v = join(lo, hi);
    f.s0 = st[b.sc + J * 16 * SB];
    f.s1 = ELEM == MX_ELEM_E2M1 ? (int)st[b.sc + J * 16 * SB + 4] : 0;
    return f;
}

template <int ELEM, int N, int... J>
__device__ __forceinline__ void read_frags(Frag (&f)[N], const LDS_AS uint8_t *st,
                                           const FragBase &b, std::integer_sequence<int, J...>)
{
    ((f[J] = read_frag<ELEM, J>(st, b)), ...);
}

// acc += B-fragment x A-fragment over one K step (B is the instruction's first
// operand: each lane's four results are then four consecutive columns of one
// row of H).  E4M3: one instruction.  E2M1: the fragments' low halves, then
// their high halves.
__device__ __forceinline__ void mma_e4m3(v4f &acc, const Frag &b, const Frag &a)
{
    acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b.v, a.v, acc, 0, 0, 0, b.s0, 0, a.s0);
}

__device__ __forceinline__ void mma_e2m1_lo(v4f &acc, const Frag &b, const Frag &a)
{
    const v8i z = {0, 0, 0, 0, 0, 0, 0, 0};
    const v8i b0 = __builtin_shufflevector(b.v, z, 0, 1, 2, 3, 8, 8, 8, 8);
    const v8i a0 = __builtin_shufflevector(a.v, z, 0, 1, 2, 3, 8, 8, 8, 8);
    acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b0, a0, acc, 4, 4, 0, b.s0, 0, a.s0);
}

__device__ __forceinline__ void mma_e2m1_hi(v4f &acc, const Frag &b, const Frag &a)
{
    const v8i z = {0, 0, 0, 0, 0, 0, 0, 0};
    const v8i b1 = __builtin_shufflevector(b.v, z, 4, 5, 6, 7, 8, 8, 8, 8);
    const v8i a1 = __builtin_shufflevector(a.v, z, 4, 5, 6, 7, 8, 8, 8, 8);
    acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b1, a1, acc, 4, 4, 0, b.s1, 0, a.s1);
}

// acc[i] += B-fragment i x A-fragment, one K step.  E2M1: the low halves of
// all tiles before the high ones, so that an accumulator's two instructions
// are not back to back.
template <int ELEM, int FN>
__device__ __forceinline__ void mma_column(v4f (&acc)[FN], const Frag (&b)[FN], const Frag &a)
{
    if constexpr (ELEM == MX_ELEM_E4M3) {
#pragma unroll
        for (int i = 0; i < FN; ++i)
            mma_e4m3(acc[i], b[i], a);
    } else {
#pragma unroll
        for (int i = 0; i < FN; ++i)
            mma_e2m1_lo(acc[i], b[i], a);
#pragma unroll
        for (int i = 0; i < FN; ++i)
            mma_e2m1_hi(acc[i], b[i], a);
    }
}

// Output stores bypass the caches' normal allocation (cache policy sc0 sc1
// nt: system scope, non-temporal): H is written once and read by a later
// kernel, and with the default policy the stores slow the operand stream
// more (QKV shape, E4M3 -> bf16: 720 -> 673 us).
constexpr int kStorePolicy = 0x13;

// stores per wave and tile of FM x FN matrix-core tiles
template <int OUT, int FM, int FN>
constexpr int kTileStores = OUT == MX_OUT_F32 ? FM * FN : FM * FN / 2;

// Store a wave's accumulators as H[m0 + wm .., n0 + wn ..] (f32 or bf16),
// times the column gain if there is one.  Every lane runs the same stores
// (exactly kTileStores of them when the tile lies inside H); lanes outside H
// are masked.
template <int OUT, int FM, int FN>
__device__ __forceinline__ void store_tile(const Args &A, const v4f (&acc)[FN][FM], int64_t m0,
                                           int64_t n0, int wm, int wn, int g, int qd)
{
    // lane (g, qd) of tile (i, j) holds H[m][n .. n+3] with
    // m = m0 + wm + 16 j + qd and n = n0 + wn + 16 i + 4 g.  N is a multiple
    // of 16, so a tile column base below N has its 16 columns inside H.
    // The gains of the lane's columns are loaded before any store.
    uint2 gw[FN];
    if (A.bgain) {
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int64_t n = n0 + wn + 16 * i + 4 * g;
            gw[i] = *reinterpret_cast<const uint2 *>(A.bgain + (n < A.N ? n : 0));
        }
    }
    auto gained = [&](int i, int j) {
        v4f v = acc[i][j];
        if (A.bgain) {
            v[0] = v[0] * __uint_as_float(gw[i].x << 16);
            v[1] = v[1] * __uint_as_float(gw[i].x & 0xFFFF0000u);
            v[2] = v[2] * __uint_as_float(gw[i].y << 16);
            v[3] = v[3] * __uint_as_float(gw[i].y & 0xFFFF0000u);
        }
        return v;
    };
    constexpr int ES = OUT == MX_OUT_F32 ? 4 : 2; // bytes per element
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        // buffer over the 16 rows of tile row j (byte offsets below 2^31:
        // the host limits N)
        const int64_t mr = m0 + wm + 16 * j;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            static_cast<uint8_t *>(A.out) + mr * A.N * ES, 0, 0x7FFFFFFF, 0x00020000);
        const int64_t m = mr + qd;
        const uint32_t row = (uint32_t)(qd * A.N) * ES;
        if constexpr (OUT == MX_OUT_F32) {
#pragma unroll
            for (int i = 0; i < FN; ++i) {
                const int64_t n = n0 + wn + 16 * i + 4 * g;
                const v4f v = gained(i, j);
                if (m < A.M && n < A.N)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs,
                                                           (int)(row + (uint32_t)n * 4), 0,
                                                           kStorePolicy);
            }
        } else {
            // bf16: tiles i and i+1 are stored together.  v_permlane16_swap
            // trades the odd lane rows (g = 1, 3) of tile i's values with the
            // even lane rows (g = 0, 2) of tile i+1's, after which lane row g
            // holds 8 adjacent columns, 16 bytes, of tile i + (g & 1) from
            // column 8 (g >> 1): one 16-byte store per lane and tile pair
            // instead of two 8-byte stores.  The swap runs on every lane; only
            // the stores are masked.
            static_assert(FN % 2 == 0, "tiles are stored in pairs");
#pragma unroll
            for (int i = 0; i < FN; i += 2) {
                uint32_t lo[2], hi[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const v4f v = gained(i + h, j);
                    lo[h] = pack_bf16(v[0], v[1]);
                    hi[h] = pack_bf16(v[2], v[3]);
                }
                const auto sl = __builtin_amdgcn_permlane16_swap(lo[0], lo[1], false, false);
                const auto sh = __builtin_amdgcn_permlane16_swap(hi[0], hi[1], false, false);
                const int64_t n = n0 + wn + 16 * (i + (g & 1)) + 8 * (g >> 1);
                if (m < A.M && n < A.N)
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{sl[0], sh[0], sl[1], sh[1]}, rs,
                                                           (int)(row + (uint32_t)n * 2), 0,
                                                           kStorePolicy);
            }
        }
    }
}

} // namespace mxg
