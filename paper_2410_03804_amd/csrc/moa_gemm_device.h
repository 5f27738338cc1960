// The product of a tile of activation rows and a tile of weight rows (bf16, MFMA 16x16x32), both staged through LDS by
// direct global -> LDS loads: the loop shared by the projections and the LM head.  What bounds it and why it looks like
// this is said in moa_gemm_bf16.hip.
#ifndef MOA_GEMM_DEVICE_H
#define MOA_GEMM_DEVICE_H
#include "moa_common.h"

namespace moa {

// 64 lanes x 16 bytes from base + off (each lane its own) to 1 KB of LDS at `lds`.  Written out because the compiler, which
// knows what the builtin writes, waits for every such load in flight in front of any LDS read that might alias it: the
// loads of later k tiles would be waited for with the current one's.  A vector memory instruction reads a scalar too early
// when a vector instruction wrote it less than five wait states before (one restored from a lane of a spill register, say),
// and nobody inserts wait states in here: the base goes through a scalar move, which waits for it in hardware and is at the
// same time the wait state between the write of m0 and its use.  (m0 is reserved and cannot be named as clobbered; nothing
// else in the kernels that use this touches it.)
__device__ __forceinline__ void lds_dma16(uint32_t lds, uint32_t off, const void *base)
{
    uint64_t at;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0" : "=&s"(at) : "s"(lds), "v"(off), "s"(base));
}
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// WR x WF wavefronts along rows x features, MR blocks of 16 rows x NF blocks of 32 features per wavefront, SX / SW stages of the activation / weight
// ring, WK groups of wavefronts that take every WK-th k tile each.
template <int WR, int WF, int MR, int NF, int SX, int SW, int WK>
struct GemmLoop {
    static constexpr int BM = 16 * MR * WR, BN = 32 * NF * WF, BK = 64, NWV = WR * WF;   // NWV: wavefronts of one K group
    static constexpr int NXI = BM / 8 / NWV, NWI = (BN / 8 + NWV - 1) / NWV;             // load instructions per wavefront and k tile
    static constexpr uint32_t XST = BM * BK * 2, WST = BN * BK * 2;                      // bytes per stage
    static constexpr size_t LDS_BYTES = (size_t)(SX * BM + SW * BN) * 2 * BK * WK;
    static constexpr int ALLOW = (SX - 2) * (NXI + NWI) + (SW > SX ? NWI : 0);           // loads in flight when a tile is needed
    static_assert(BM % (8 * NWV) == 0 && SW >= SX && SX >= 2 && LDS_BYTES <= 160 * 1024, "");

    int lane, wave, kgrp;
    uint32_t xoff[NXI], woff[NWI], xdst[NXI], wdst[NWI];
    const char *xbase, *wbase[NWI];
    // acc[i][j][b][v]: feature 32 i + 8 (lane / 16) + 4 b + v of the wavefront's, row 16 j + lane % 16
    f32x4 acc[NF][MR][2];

    __device__ __forceinline__ GemmLoop()
    {
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) % NWV);
        kgrp = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) / NWV);
    }
    __device__ __forceinline__ int wave_row() const { return (wave / WF) * (16 * MR); }
    __device__ __forceinline__ int wave_feature() const { return (wave % WF) * (32 * NF); }

    // This lane's 16-byte pieces as offsets from the bases, for the first k tile.  An instruction moves eight tile rows of
    // 128 bytes into 1 KB of LDS; piece c of row r lives at position c ^ (r / 2 & 7) of its row, which spreads the operand
    // reads of 16 rows over all banks.  W rows are permuted inside blocks of 32 so that the 8 results a lane gets for a
    // row from a block are 8 consecutive features.
    // x: first row of the tile, rows_left of them valid (the last one is repeated behind them)
    __device__ __forceinline__ void set_x(const void *x, int64_t ldx, int64_t rows_left)
    {
        xbase = (const char *)x;
#pragma unroll
        for (int i = 0; i < NXI; ++i) {
            const int g = wave + NWV * i, row = 8 * g + (lane >> 3);
            const int rr = row < rows_left ? row : (int)rows_left - 1;
            xoff[i] = (uint32_t)(rr * ldx * 2 + 16 * ((lane & 7) ^ ((row >> 1) & 7)));
            xdst[i] = (uint32_t)(g * 1024);
        }
    }
    // base_of(block, &first): the matrix that block of 32 weight rows comes from (its row `n0`, uniform) and the block's
    // first row counted from there; rows_left of the rows from n0 on are valid
    template <typename F>
    __device__ __forceinline__ void set_w(int K, int rows_left, F base_of)
    {
#pragma unroll
        for (int i = 0; i < NWI; ++i) {
            int g = wave + NWV * i;
            if (g > BN / 8 - 1) g = BN / 8 - 1;                  // the same rows once more into the same place
            const int row = 8 * g + (lane >> 3), p = row & 31;
            int first = 0;
            wbase[i] = (const char *)base_of(g >> 2, &first);
            int f = first + 8 * ((p >> 2) & 3) + 4 * (p >> 4) + (p & 3);
            if (f > rows_left - 1) f = rows_left - 1;
            woff[i] = (uint32_t)f * (uint32_t)K * 2u + (uint32_t)(16 * ((lane & 7) ^ ((row >> 1) & 7)));
            wdst[i] = SX * XST + (uint32_t)(g * 1024);
        }
    }

    // nk k tiles of this K group, from column 64 (kt0 WK + kgrp) on in steps of 64 WK; with WK > 1 only group 0 has the
    // sums afterwards (the others return false).  Ends behind a barrier when WK > 1, and with no load in flight.
    __device__ __forceinline__ bool run(char *smem, int kt0, int nk)
    {
        const int64_t kbyte0 = ((int64_t)kt0 * WK + kgrp) * (BK * 2);
        const uint32_t ring = (uint32_t)kgrp * (SX * XST + SW * WST);
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem + ring;
        const int l16 = lane & 15, quart = lane >> 4;
        uint32_t xfill = 0, wfill = 0;             // stage (byte offset) the next load goes to
        auto issue_x = [&](int kt) {               // tiles past the last repeat it (nobody reads them)
            const int64_t ko = kbyte0 + (int64_t)(kt < nk ? kt : nk - 1) * (WK * BK * 2);
#pragma unroll
            for (int i = 0; i < NXI; ++i) lds_dma16(lds0 + xdst[i] + xfill, xoff[i], xbase + ko);
            xfill = xfill + XST == SX * XST ? 0 : xfill + XST;
        };
        auto issue_w = [&](int kt) {
            const int64_t ko = kbyte0 + (int64_t)(kt < nk ? kt : nk - 1) * (WK * BK * 2);
#pragma unroll
            for (int i = 0; i < NWI; ++i) lds_dma16(lds0 + wdst[i] + wfill, woff[i], wbase[i] + ko);
            wfill = wfill + WST == SW * WST ? 0 : wfill + WST;
        };
#pragma unroll
        for (int i = 0; i < SW; ++i) {
            if (i >= SW - SX) issue_x(i - (SW - SX));
            issue_w(i);
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < MR; ++j) acc[i][j][0] = acc[i][j][1] = f32x4{0.f, 0.f, 0.f, 0.f};

        uint32_t koff[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) koff[s] = (uint32_t)(l16 * 128 + 16 * ((4 * s + quart) ^ ((l16 >> 1) & 7)));
        const uint32_t xrd = ring + (uint32_t)(wave_row() * 128), wrd = ring + (uint32_t)(SX * XST + wave_feature() * 128);
        uint32_t xcur = 0, wcur = 0;                   // stages being read
        // A tile is multiplied in quarters: columns 32 (p / 2) .. of one half of the wavefront's features.  Both quarters of
        // 32 columns take the same activation operands.
        bf16x8 af[2][NF], bf[2][MR];
        auto read = [&](int p) {
            const char *wp = smem + (wrd + wcur + koff[p >> 1]), *xp = smem + (xrd + xcur + koff[p >> 1]);
#pragma unroll
            for (int i = 0; i < NF; ++i) af[p & 1][i] = *(const bf16x8 *)(wp + 2048 * (i + NF * (p & 1)));
            if (!(p & 1))
#pragma unroll
                for (int j = 0; j < MR; ++j) bf[p >> 1][j] = *(const bf16x8 *)(xp + 2048 * j);
        };
        auto multiply = [&](int p) {
#pragma unroll
            for (int i = NF * (p & 1); i < NF * (p & 1) + NF; ++i)
#pragma unroll
                for (int j = 0; j < MR; ++j) {
                    f32x4 &c = acc[i >> 1][j][i & 1];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[p & 1][i - NF * (p & 1)], bf[p >> 1][j], c, 0, 0, 0);
                }
        };
        auto advance = [&] {
            xcur = xcur + XST == SX * XST ? 0 : xcur + XST;
            wcur = wcur + WST == SW * WST ? 0 : wcur + WST;
        };
        wait_loads_and_barrier<ALLOW>();
        read(0);
        int kt = 0;
        for (; kt < nk - SX; ++kt) {
            read(1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(0);
            read(2);
            __builtin_amdgcn_sched_barrier(0);
            multiply(1);
            read(3);
            __builtin_amdgcn_sched_barrier(0);
            multiply(2);
            if (NF * MR >= 16) __builtin_amdgcn_sched_barrier(0);
            wait_loads_and_barrier<ALLOW>();           // tile kt + 1 is in LDS for everybody, nobody reads tile kt any more
            advance();
            read(0);
            __builtin_amdgcn_sched_barrier(0);
            multiply(3);
            issue_x(kt + SX);
            issue_w(kt + SW);
        }
        for (; kt < nk; ++kt) {
            read(1);
            multiply(0);
            read(2);
            multiply(1);
            read(3);
            multiply(2);
            if (kt + 1 < nk) {
                wait_loads_and_barrier<0>();
                advance();
                read(0);
            }
            multiply(3);
        }

        if (WK > 1) {                                  // the K groups' sums, added up in group order
            constexpr int PER = NF * MR * 8 * 64;
            float *red = (float *)smem;
            wait_loads_and_barrier<0>();
            if (kgrp > 0) {
#pragma unroll
                for (int i = 0; i < NF; ++i)
#pragma unroll
                    for (int j = 0; j < MR; ++j)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            red[((kgrp - 1) * NWV + wave) * PER + ((i * MR + j) * 8 + e) * 64 + lane] = acc[i][j][e >> 2][e & 3];
            }
            __syncthreads();
            if (kgrp > 0) return false;
#pragma unroll
            for (int g = 0; g < WK - 1; ++g)
#pragma unroll
                for (int i = 0; i < NF; ++i)
#pragma unroll
                    for (int j = 0; j < MR; ++j)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            acc[i][j][e >> 2][e & 3] += red[(g * NWV + wave) * PER + ((i * MR + j) * 8 + e) * 64 + lane];
        }
        return true;
    }
};

}  // namespace moa
#endif
