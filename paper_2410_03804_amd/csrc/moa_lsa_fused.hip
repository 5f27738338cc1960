// Layer Self-Attention with mean aggregation in ONE kernel (paper Sec. 3.1.1; Alg. 1, LSA_layer_with_mean):
// Q/K/V projection of a token's L layer rows, attention over the layer axis, and the mean over the layers, with the
// projected Q, K, V never leaving the compute unit.  Every token is independent of the others (Sec. 3.1.1), so a
// workgroup that owns whole tokens needs nothing from any other workgroup.
//
// A workgroup of eight wavefronts owns TT tokens (all their layer rows: RB = 32 NB TT rows, NB = ceil(L/32)) and the
// features of one KV head's group that one attention needs: two query heads, the key head and the value head, 4 dh
// features.  (A group of more than two query heads is cut into parts of two; each part recomputes K and V.)
//
//  projection  [RB x d_in] x [4 dh x d_in]^T on MFMA 16x16x32, walked along d_in in tiles of 64.  Wavefront w owns
//              the features w dh/2 .. and ALL rows, so its slice of the weight tile is its own: it fetches it itself
//              (global memory straight into LDS, 128-byte rows, XOR-swizzled against bank conflicts) into a private
//              two-stage ring and needs no barrier for it, only its own load counter.  As soon as a wavefront has
//              read its fragments of tile kt it requests tile kt+2 into the same place, so one whole tile and most of
//              another are in flight per compute unit while a tile is being multiplied.  The activation tile (RB rows,
//              shared by all wavefronts, an eighth of the weight tile) goes through a small ring of its own with one
//              barrier per tile.
//              (16x16x32 instructions: they give the bits of 32x32x16 ones chained along d_in -- one takes the place of two --
//              from the same operand bytes, and at the clock that the power budget leaves they make 2.03 PFLOP/s from
//              registers against 1.78.  From packed weights 60 tokens of 32 layers 40.9 -> 38.1 us with the output projection,
//              480 213 -> 194, 1024 443 -> 411, 240 of 80 layers 288 -> 262; from plain ones 1024 tokens 528 -> 475.)
//              Three things cost about the same per tile -- the weight tile's way from the L2 into LDS (64 KB per
//              64 of d_in, all workgroups of an XCD asking for the same lines at once), the operand reads from LDS
//              and the matrix work -- and they overlap only in part; the lever that is left is rows per workgroup
//              (2, 3 or 4 tokens at one 32-layer block each, from packed weights 5), chosen from the token count on the host.
//  attention   the accumulators are rounded to the storage type and parked in LDS as a [RB x 4 dh] tile (the ring
//              memory is reused); one wavefront per (token, query head): S^T = K Q^T by MFMA, fp32 softmax in
//              registers, column means of P summed over the 32 query lanes (DPP moves, one shuffle), then
//              abar = sum_j pbar_j V_j  (mean_i(P V) = (1^T P / L) V, exact in real arithmetic).  The output
//              projection follows in another launch on one row per token.
//
// Two kernels share that second half: k_lsa_fused (plain weights, as above) and k_lsa_fused_pk (weights packed once
// into MFMA-operand order and read straight into registers; the form a step runs when it is given the packed copy).
//
// Arithmetic is that of the three-kernel form (same MFMA order along d_in, Q/K/V rounded once to the storage type,
// the same order of additions in the column sums), so all give the same bits.
#include "moa_common.h"
#include "moa_lsa_plan.h"
#include "moa_tree_device.h"

#include <math.h>
#include <type_traits>
#include <utility>

namespace moa {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void global_void_t;

struct LsaFusedArgs {
    const bf16_t *hs;              // [T, L, d_in]
    const bf16_t *wq, *wk, *wv;    // [Hq*dh, d_in], [Hkv*dh, d_in] x 2
    const bf16_t *wpk;             // the same weights in MFMA-operand order (k_lsa_pack_weights), or NULL
    bf16_t *abar;                  // [T, Hq*dh]
    int64_t T;
    int L, d_in, Hq, Hkv;
    int parts;                     // Hq / Hkv / 2: workgroups per KV head
    int units;                     // Hkv * parts
    int units_per_xcd;
    int64_t wide_tiles;            // k_lsa_fused_pk_wide: tiles of five tokens in front of the others
    int lead_blocks;                           // workgroups in front of the kernel's own: integer work of a step
    int pf_lead;                               // the last of them (a multiple of the XCD count) only read ahead: see lsa_warm_block
    int rider_units;
    StepSmallArgs rider;
};

// DENSE: the rows of a tile's tokens follow one another (TT L <= RB) instead of each token starting a block of 32
template <int DH, int NB, int TT, bool DENSE = false>
struct LsaFusedGeom {
    static constexpr int NF = 4 * DH;            // features per workgroup
    static constexpr int FW = NF / 8;            // per wavefront
    static constexpr int RB = DENSE ? 160 : 32 * NB * TT;    // rows per workgroup
    static constexpr bool FULL = RB == 160;      // the parked tile fills the LDS to the last byte
    static constexpr int BK = 64;
    static constexpr int XS = RB <= 64 ? 3 : 2;  // stages of the activation ring
    static constexpr size_t w_bytes = (size_t)8 * 2 * FW * BK * sizeof(bf16_t);
    static constexpr size_t x_bytes = (size_t)XS * RB * BK * sizeof(bf16_t);
    // row of the parked Q/K/V tile: 16-byte reads of 8 rows hit all banks.  Where it fills the LDS its rows are not padded,
    // piece c of row r lies at c ^ (r & 15), and the column means go where the wavefront's Q was
    static constexpr int TLD = FULL ? NF : NF + 8;
    static constexpr size_t tile_bytes = (size_t)RB * TLD * sizeof(bf16_t);
    static constexpr size_t pbar_bytes = FULL ? 0 : (size_t)8 * 32 * NB * sizeof(float);
    static constexpr size_t loop_bytes = w_bytes + x_bytes;
    static constexpr size_t epi_bytes = tile_bytes + pbar_bytes;
    static constexpr size_t bytes = loop_bytes > epi_bytes ? loop_bytes : epi_bytes;
    // the form that takes packed weights keeps them in registers: only a two-stage activation ring is left in LDS
    // weight tiles held in registers per wavefront: with the requests spread between the MFMAs two do as well as four; beside
    // the accumulators of 128 rows and more there is room for one, and half of a tile's MFMAs hide a request (1024 tokens 411 us;
    // with two, twelve registers spilled, 443)
    static constexpr int WS = RB >= 128 ? 1 : 2;
    static constexpr int UN = 8;                 // tile steps per trip of the tile loop (a multiple of WS)
    static constexpr size_t pk_loop_bytes = (size_t)2 * RB * BK * sizeof(bf16_t);
    static constexpr size_t pk_bytes = pk_loop_bytes > epi_bytes ? pk_loop_bytes : epi_bytes;
};

// Second half of both kernels below: the accumulators of a workgroup's [RB x 4 dh] projection tile are rounded to the
// storage type and parked in LDS (`park` hands them over, four features of a row at a time), then one wavefront per (token of the tile, query head) runs the attention over the layer axis and the
// mean.  Called by all 512 threads; `sm` is the workgroup's whole LDS, free to reuse after the barrier in here.
template <int DH, int NB, int TT, bool DENSE, typename Park>
__device__ __forceinline__ void lsa_fused_epilogue(Park park, const LsaFusedArgs &a, bf16_t *sm, int64_t tok0, int g, int part)
{
    using Gm = LsaFusedGeom<DH, NB, TT, DENSE>;
    constexpr int TLD = Gm::TLD;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int G = a.Hq / a.Hkv, L = a.L;

    // park Q | Q' | K | V of the RB rows in LDS, rounded to the storage type
    __syncthreads();                             // every wavefront is done with the rings
    bf16_t *tile_s = sm;
    auto at = [&](int row, int col) {            // column `col` of a row, and what follows it in its piece of eight
        return Gm::FULL ? tile_s + row * TLD + 8 * ((col >> 3) ^ (row & 15)) + (col & 7) : tile_s + row * TLD + col;
    };
    // four features from `col` on of a row, rounded
    park([&](int row, int col, float x0, float x1, float x2, float x3) {
        u32x2 pk;
        pk[0] = pack_bf16x2(x0, x1);
        pk[1] = pack_bf16x2(x2, x3);
        *(u32x2 *)at(row, col) = pk;
    });
    __syncthreads();

    // attention over the layer axis: one wavefront per (token of the tile, query head); spare wavefronts redo a
    // unit and store nothing, so that the barriers below are reached by all.  In a dense tile four units have two wavefronts
    // each: the second takes the last block of query rows and hands its weights over (49 rows of 64; a token has more than 64).
    // Of ten units two wavefronts do two, one after another.
    constexpr int NU = 2 * TT;
    constexpr int NKS = DH / 16;
    static_assert(!DENSE || NU == 4, "two wavefronts per unit");
    const bool live_wave = wave < NU;
    const int ib0 = DENSE && !live_wave ? NB - 1 : 0, ib1 = DENSE && live_wave ? NB - 1 : NB;
    int u = NU > 8 ? __builtin_amdgcn_readfirstlane(wave) : wave % NU;
    do {
        const int tt = u >> 1, hq = u & 1;
        const int64_t tok = tok0 + tt;
        const int row0 = tt * (DENSE ? L : 32 * NB);                  // the token's first row
        const bf16_t *trow = tile_s + (size_t)row0 * TLD;
        auto tok_at = [&](int row, int col) {                         // rows past L are masked, or weighted 0
            return DENSE ? (const bf16_t *)at(row0 + min(row, L - 1), col) : Gm::FULL ? (const bf16_t *)at(row0 + row, col) : trow + row * TLD + col;
        };
        float *pbar_s = (float *)((char *)sm + Gm::tile_bytes) + wave * 32 * NB;
        auto pbar = [&](int j) -> float & { return Gm::FULL ? ((float *)(tile_s + (row0 + (j >> 6)) * TLD + hq * DH))[j & 63] : pbar_s[j]; };
        const float sc = 1.4426950408889634f / sqrtf((float)DH);      // log2 domain

        float hand_inv = 0.f;
        // column sums of P in the S^T register layout: csum[jb][v] belongs to key 32 jb + 8 (v/4) + 4 half + v%4
        float csum[NB][16];
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) csum[jb][e] = 0.f;
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {
            if (DENSE && (ib < ib0 || ib >= ib1)) continue;
            const bool qvalid = 32 * ib + l32 < L;
            bf16x8 qf[NKS];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)tok_at(32 * ib + l32, hq * DH + 16 * ks + 8 * half);
            f32x16 s[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
#pragma unroll
                for (int e = 0; e < 16; ++e) s[jb][e] = 0.f;
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {        // key fragments straight from the parked tile: nothing to keep across blocks
                    const bf16x8 kf = *(const bf16x8 *)tok_at(32 * jb + l32, 2 * DH + 16 * ks + 8 * half);
                    s[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[jb], 0, 0, 0);
                }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = 32 * jb + 8 * (e >> 2) + 4 * half + (e & 3);
                    const float x = key < L ? s[jb][e] * sc : -INFINITY;
                    s[jb][e] = x;
                    mx = fmaxf(mx, x);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            float sum = 0.f;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e) { const float p = exp2f(s[jb][e] - mx); s[jb][e] = p; sum += p; }
            sum += __shfl_xor(sum, 32);
            const float inv = qvalid ? 1.0f / sum : 0.f;              // padded query columns contribute nothing
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    if (DENSE && !live_wave) csum[jb][e] = s[jb][e];             // scaled where it is added: the same rounding
                    else csum[jb][e] += s[jb][e] * inv;
                }
            hand_inv = inv;
        }
        if (DENSE) {                                 // through the rows of the unit's Q, which nobody reads any more
            __syncthreads();
            auto place = [&](int jb, int e) -> float & { return ((float *)(tile_s + (row0 + 16 * jb + e) * TLD + hq * DH))[lane]; };
            if (!live_wave) {
#pragma unroll
                for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) place(jb, e) = csum[jb][e];
                place(NB, 0) = hand_inv;
            }
            __syncthreads();
            if (live_wave) {
                const float inv = place(NB, 0);
#pragma unroll
                for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) csum[jb][e] += place(jb, e) * inv;
            }
        }
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                csum[jb][e] = sum_over_lanes32(csum[jb][e]);
            }
        if (l32 == 0 && (!DENSE || live_wave)) {     // (a dense tile has one place per unit, which its own wavefront is done with)
            const float invL = 1.0f / (float)L;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e) pbar(32 * jb + 8 * (e >> 2) + 4 * half + (e & 3)) = csum[jb][e] * invL;
        }
        if (NU <= 8) __syncthreads();
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the wavefront's own

        // abar[c] = sum_j pbar[j] V[j][c]: a lane weights 8 components of its rows, then the row groups are added up
        constexpr int CPR = DH / 8;                  // 16-byte pieces per V row
        constexpr int RPI = 64 / CPR;                // rows per instruction
        constexpr int NVI = 32 / RPI;
        const int vrow0 = lane / CPR, vpiece = lane % CPR;
        float o[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = 0.f;
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int i = 0; i < NVI; ++i) {
                const int row = 32 * jb + RPI * i + vrow0;
                const float pj = row < L ? pbar(row) : 0.f;
                const u32x4 vv = *(const u32x4 *)tok_at(row, 3 * DH + 8 * vpiece);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    o[2 * w] = fmaf(pj, __uint_as_float(vv[w] << 16), o[2 * w]);
                    o[2 * w + 1] = fmaf(pj, __uint_as_float(vv[w] & 0xffff0000u), o[2 * w + 1]);
                }
            }
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int off = CPR; off < 64; off <<= 1) o[c] += __shfl_xor(o[c], off);
        if ((NU > 8 || live_wave) && tok < a.T && lane < CPR) {
            u32x4 pk;
#pragma unroll
            for (int w = 0; w < 4; ++w) pk[w] = pack_bf16x2(o[2 * w], o[2 * w + 1]);
            *(u32x4 *)(a.abar + tok * (int64_t)a.Hq * DH + (int64_t)(g * G + 2 * part + hq) * DH + 8 * lane) = pk;
        }
    } while (NU > 8 && (u += 8) < NU);
}

template <int DH, int NB, int TT>
__global__ __launch_bounds__(512) void k_lsa_fused(LsaFusedArgs a)
{
    using Gm = LsaFusedGeom<DH, NB, TT>;
    constexpr int FW = Gm::FW, RB = Gm::RB, BK = Gm::BK, XS = Gm::XS;
    constexpr int WFB = FW / 16;                 // 16-feature blocks per wavefront
    constexpr int NRB = RB / 16;                 // 16-row blocks
    constexpr int HRB = NRB / 2;                 // those of which a quarter of a tile takes the fragments
    constexpr int NWI = FW / 8;                  // weight-tile load instructions per wavefront (8 rows of 128 B each)
    constexpr int NXI = (RB / 8 + 7) / 8;        // activation-tile load instructions per wavefront
    constexpr int XD = XS - 1;                   // activation tiles requested ahead
    extern __shared__ __attribute__((aligned(16))) bf16_t sm[];

    if ((int)blockIdx.x < a.lead_blocks) {       // the first workgroups of the grid carry the step's integer work
        if ((int)blockIdx.x < a.rider_units && threadIdx.x < 64)
            step_small_unit(a.rider, (int)blockIdx.x, (int32_t *)sm, (int32_t *)sm + MOA_MAX_TREE);
        return;
    }
    // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: an XCD keeps the weight slices of its
    // units (2 MB each at the Llama-3-8B shape) and every token tile's activations pass through it once.
    const int bx = (int)blockIdx.x - a.lead_blocks;
    const int xcd = bx & 7, slot = bx >> 3;
    const int unit = xcd * a.units_per_xcd + slot % a.units_per_xcd;
    const int64_t tile = slot / a.units_per_xcd;
    if (unit >= a.units) return;                 // the whole workgroup leaves before any barrier
    const int g = unit / a.parts, part = unit - g * a.parts;
    const int G = a.Hq / a.Hkv, L = a.L, K = a.d_in;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, quart = lane >> 4;
    const int lrow = lane >> 3, lpos = lane & 7;

    f32x4 acc[WFB][NRB];
#pragma unroll
    for (int i = 0; i < WFB; ++i)
#pragma unroll
        for (int j = 0; j < NRB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nk = K / BK;                       // >= 2 (checked on the host)

    // this wavefront's FW feature rows of the weight tile: inside one of Wq (two heads), Wk, Wv
    const int which = wave * FW / DH;
    const bf16_t *wm = which < 2 ? a.wq + (int64_t)((g * G + 2 * part + which) * DH + wave * FW % DH) * K
                                 : (which == 2 ? a.wk : a.wv) + (int64_t)(g * DH + wave * FW % DH) * K;
    const bf16_t *wsrc[NWI];
#pragma unroll
    for (int i = 0; i < NWI; ++i) {
        const int row = 8 * i + lrow;
        wsrc[i] = wm + (int64_t)row * K + 8 * (lpos ^ ((row >> 1) & 7));
    }
    // its share of the activation tile: instruction xi covers tile rows 8 xi .. 8 xi + 7 (a row past the tokens or the
    // layers repeats a valid one; such rows are masked as keys and dropped as queries)
    const bf16_t *xsrc[NXI];
    int xrow0[NXI];
#pragma unroll
    for (int n = 0; n < NXI; ++n) {
        int xi = wave + 8 * n;
        if (xi > RB / 8 - 1) xi = RB / 8 - 1;    // a spare instruction repeats the last one (same bytes to the same place)
        xrow0[n] = 8 * xi;
        const int s = 8 * xi + lrow;
        int64_t tok = tile * TT + s / (32 * NB);
        int lay = s % (32 * NB);
        if (tok > a.T - 1) tok = a.T - 1;
        if (lay > L - 1) lay = L - 1;
        xsrc[n] = a.hs + (tok * L + lay) * (int64_t)K + 8 * (lpos ^ ((s >> 1) & 7));
    }
    bf16_t *wl = sm + (size_t)wave * 2 * FW * BK;                 // this wavefront's ring: [2][FW][BK]
    bf16_t *xl = sm + (size_t)8 * 2 * FW * BK;                    // [XS][RB][BK]
    auto issue_w = [&](int kt) {
        bf16_t *dst = wl + (kt & 1) * FW * BK;
#pragma unroll
        for (int i = 0; i < NWI; ++i)
            __builtin_amdgcn_global_load_lds((global_void_t *)(wsrc[i] + (int64_t)kt * BK), (lds_void_t *)(dst + 8 * i * BK), 16, 0, 0);
    };
    auto issue_x = [&](int kt) {
        bf16_t *dst = xl + (kt % XS) * RB * BK;
#pragma unroll
        for (int n = 0; n < NXI; ++n)
            __builtin_amdgcn_global_load_lds((global_void_t *)(xsrc[n] + (int64_t)kt * BK), (lds_void_t *)(dst + xrow0[n] * BK), 16, 0, 0);
    };

    // Requests are issued in the order X(0) W(0) X(1) W(1) (W(0) X(0) W(1) with a two-stage activation ring), then per
    // tile kt: X(kt+XD) W(kt+2), and complete in that order (all of them go straight to LDS).  At the top of tile kt,
    // X(kt) and W(kt) must have landed; what was requested after the later of the two is X(kt+1) W(kt+1) (only
    // W(kt+1) with the two-stage ring), and nothing in the last round.
    if (XD >= 2) issue_x(0);
    issue_w(0);
    issue_x(XD >= 2 ? 1 : 0);
    issue_w(1);
    constexpr int PENDING = XD >= 2 ? NXI + NWI : NWI;
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PENDING) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        const bf16_t *wb = wl + (kt & 1) * FW * BK;
        const bf16_t *xb = xl + (kt % XS) * RB * BK;
        // The quarters of a tile -- 32 columns (step p / 2) of one half of the rows -- are software-pipelined: the fragments of
        // the next one are requested from LDS before the MFMAs of this one are issued, so LDS reads and matrix work of one
        // wavefront overlap.  Once the last quarter's fragments have been read, the ring places this tile occupied are free and
        // are refilled.
        bf16x8 af[2][WFB], bfr[2][HRB];
        auto read_frags = [&](int p) {
            const int piece = 4 * (p >> 1) + quart;
#pragma unroll
            for (int i = 0; i < WFB; ++i) {
                if (p & 1) continue;                 // both halves of the rows take the same weights
                const int row = 16 * i + l16;
                af[p >> 1][i] = *(const bf16x8 *)&wb[row * BK + 8 * (piece ^ ((row >> 1) & 7))];
            }
#pragma unroll
            for (int j = 0; j < HRB; ++j) {
                const int row = 16 * ((p & 1) * HRB + j) + l16;
                bfr[p & 1][j] = *(const bf16x8 *)&xb[row * BK + 8 * (piece ^ ((row >> 1) & 7))];
            }
        };
        read_frags(0);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p < 3) read_frags(p + 1);
            if (p == 3) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (kt + XD < nk) issue_x(kt + XD);
                if (kt + 2 < nk) issue_w(kt + 2);
            }
#pragma unroll
            for (int i = 0; i < WFB; ++i)
#pragma unroll
                for (int j = 0; j < HRB; ++j) {
                    f32x4 &c = acc[i][(p & 1) * HRB + j];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[p >> 1][i], bfr[p & 1][j], c, 0, 0, 0);
                }
        }
    }

    // acc[i][j][v]: feature wave FW + 16 i + 4 quart + v, row 16 j + l16
    lsa_fused_epilogue<DH, NB, TT, false>([&](auto put) {
#pragma unroll
        for (int i = 0; i < WFB; ++i)
#pragma unroll
            for (int j = 0; j < NRB; ++j)
                put(16 * j + l16, wave * FW + 16 * i + 4 * quart, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    }, a, sm, tile * TT, g, part);
}

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{}): a loop whose index is a constant
// expression in the body (register arrays indexed by it stay in registers)
template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Helper workgroup `h` of `a.pf_lead` (packed form).  A cold weight tile is first touched by all of an XCD's
// workgroups at once (they walk the k tiles in step), so all of them wait for HBM together, tile after tile; from the
// L2 they do not.  At decode sizes the kernel's own workgroups leave sixteen compute units idle: two helpers per XCD
// read that XCD's units' packed weights once, tile by tile and in turn, ahead of the workgroups that multiply them,
// and throw them away.  (One compute unit pulls about 50 GB/s of misses however many requests it keeps in flight, so
// sixteen helpers move 0.8 TB/s: the 16 MiB of weights in the kernel's first half.  Reading further operands of the
// step's later launches ahead in the same way -- caches, output-projection weights, here or from the compute units
// the attention cores leave idle -- was measured too: what the later launches gained, the carrying launch lost.)
template <int DH, int NB, int TT>
__device__ __forceinline__ void lsa_warm_block(const LsaFusedArgs &a, int h, bf16_t *sm)
{
    constexpr int NWP = 4 * (LsaFusedGeom<DH, NB, TT>::FW / 32);
    static_assert(NWP * 64 == 512, "one piece per thread and (wavefront, k tile) block");
    const int tid = threadIdx.x, nk = a.d_in / 64;
    const int xcd = h & 7, turn = h >> 3, turns = a.pf_lead >> 3;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int uu = 0; uu < a.units_per_xcd; ++uu) {
        const int unit = xcd * a.units_per_xcd + uu;
        if (unit >= a.units) break;
        // [unit][wavefront][k tile] blocks of NWP * 64 pieces: one piece per thread and block
        const u32x4 *base = (const u32x4 *)a.wpk + (int64_t)unit * 8 * nk * (NWP * 64) + tid;
        for (int kt = 2 * turn; kt < nk; kt += 2 * turns) {          // two tiles per round: sixteen requests in flight
            const int kt1 = kt + 1 < nk ? kt + 1 : kt;
            u32x4 v[16];
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                v[w] = base[(int64_t)(w * nk + kt) * (NWP * 64)];
                v[8 + w] = base[(int64_t)(w * nk + kt1) * (NWP * 64)];
            }
#pragma unroll
            for (int w = 0; w < 16; ++w) acc ^= v[w];
        }
    }
    ((u32x4 *)sm)[tid] = acc;                    // into LDS nobody reads: what keeps the loads from being dropped
}

// The same kernel for weights that the caller has packed once into MFMA-operand order (k_lsa_pack_weights).  A
// wavefront's slice of the weight tile is used by that wavefront alone, so with the operands already in lane order it
// has no business in LDS: every 16-byte operand piece is loaded straight into the register that the MFMA reads, 1 KB
// contiguous per instruction.  That takes the weight tile (8/9 of the bytes) out of the LDS traffic -- reads and
// writes of the unpacked form add up to the LDS bandwidth of the whole tile time -- and lets WS - 1 whole tiles be in
// flight per wavefront in registers, which the 160 KB of LDS could not hold.  The activation tile goes through
// registers into a two-stage LDS ring (one bare barrier per tile); all loads are ordinary loads, so the waits are the
// compiler's.  Same MFMA order along d_in as the unpacked form: same bits.
//
// The tile of TT tokens from tok0 on, of one unit.
template <int DH, int NB, int TT, bool DENSE>
__device__ __forceinline__ void lsa_pk_tile(const LsaFusedArgs &a, int unit, int64_t tok0)
{
    using Gm = LsaFusedGeom<DH, NB, TT, DENSE>;
    constexpr int FW = Gm::FW, RB = Gm::RB, BK = Gm::BK, WS = Gm::WS;
    constexpr int WFB = FW / 16;                 // 16-feature blocks per wavefront
    constexpr int NRB = RB / 16;                 // 16-row blocks
    constexpr int HRB = NRB / 2;                 // those whose fragments are in registers at a time
    constexpr int NWP = 2 * WFB;                 // operand pieces per lane and weight tile
    constexpr int NXI = (RB / 8 + 7) / 8;        // activation-tile load instructions per wavefront
    extern __shared__ __attribute__((aligned(16))) bf16_t sm[];

    const int g = unit / a.parts, part = unit - g * a.parts;
    const int L = a.L, K = a.d_in;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, quart = lane >> 4;
    const int lrow = lane >> 3, lpos = lane & 7;

    f32x4 acc[WFB][NRB];
#pragma unroll
    for (int i = 0; i < WFB; ++i)
#pragma unroll
        for (int j = 0; j < NRB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nk = K / BK;

    // packed weights: [unit][wavefront][k tile][k step of 16][block of 32 features][feature + 32 (k half)] pieces of 8 elements
    const bf16x8 *wp = (const bf16x8 *)a.wpk + ((int64_t)(unit * 8 + wave) * nk) * (NWP * 64) + (quart >> 1) * 128 + (quart & 1) * 32 + l16;
    auto wpiece = [](int b) { return b / WFB * 256 + (b % WFB >> 1) * 64 + (b & 1) * 16; };     // piece b: step b / WFB, block b % WFB
    // activation rows as in the unpacked form: instruction n covers tile rows xrow0[n] .. + 7, the piece a lane fetches
    // is the one whose swizzled place in LDS is the lane's own
    const bf16_t *xsrc[NXI];
    int xrow0[NXI];
#pragma unroll
    for (int n = 0; n < NXI; ++n) {
        int xi = wave + 8 * n;
        if (xi > RB / 8 - 1) xi = RB / 8 - 1;
        xrow0[n] = 8 * xi;
        const int s = 8 * xi + lrow;
        const int in = DENSE ? min(s / L, TT - 1) : s / (32 * NB);
        int64_t tok = tok0 + in;
        int lay = DENSE ? s - in * L : s % (32 * NB);
        if (tok > a.T - 1) tok = a.T - 1;
        if (lay > L - 1) lay = L - 1;
        xsrc[n] = a.hs + (tok * L + lay) * (int64_t)K + 8 * (lpos ^ ((s >> 1) & 7));
    }
    bf16_t *xl = sm;                             // [2][RB][BK]

    // weights are requested WS tiles ahead into a register ring (a k-step's registers are refilled as soon as it has been
    // multiplied), activations one tile ahead
    bf16x8 wr[WS][NWP];
    bf16x8 xr[WS][NXI];
    auto load_w = [&](int kt, bf16x8 (&dst)[NWP]) {
#pragma unroll
        for (int b = 0; b < NWP; ++b) dst[b] = wp[(int64_t)kt * NWP * 64 + wpiece(b)];
    };
    auto load_x = [&](int kt, bf16x8 (&dst)[NXI]) {
#pragma unroll
        for (int n = 0; n < NXI; ++n) dst[n] = *(const bf16x8 *)(xsrc[n] + (int64_t)kt * BK);
    };
#pragma unroll
    for (int s = 0; s < WS; ++s) {               // a tile past the last repeats the last (nk >= 2)
        if (s == 0) load_x(s < nk ? s : nk - 1, xr[s]);
        load_w(s < nk ? s : nk - 1, wr[s]);
    }

    // One tile step on register stage S.  The activation tile of this step goes to LDS (the place was last read two
    // tiles ago, before the previous barrier) and the next one is requested into the registers it leaves.
    // Inside the step the weight requests are spread between the MFMAs: as soon as a k-step's MFMAs have been issued
    // its weight registers are refilled with the same k-step of the tile WS ahead.  Issued in one burst at the top of
    // a step, the requests of all eight wavefronts queue up at the compute unit's one address unit while the matrix
    // cores wait (measured on a cut-down loop: 0.99 us per tile in a burst, 0.78 us spread out).  The scheduling
    // barriers keep the compiler from regrouping them.  No branch surrounds a load: the compiler's load counter then
    // stays exact (partial waits), where a conditional request makes it wait for everything in flight; requests past
    // the last tile repeat the last tile.  GUARDED steps (the few behind the last whole trip) may lie past the last
    // tile and then skip their arithmetic; they refill in one go behind it.
    auto tile_step = [&](auto stage_c, auto guarded_c, int kt) {
        constexpr int S = decltype(stage_c)::value;
        constexpr bool GUARDED = decltype(guarded_c)::value;
        const bf16_t *xb = xl + (kt & 1) * RB * BK;
        {
            bf16_t *xw = xl + (kt & 1) * RB * BK;
#pragma unroll
            for (int n = 0; n < NXI; ++n) *(bf16x8 *)&xw[xrow0[n] * BK + 8 * lane] = xr[S][n];
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        load_x(kt + 1 < nk ? kt + 1 : nk - 1, xr[(S + 1) % WS]);
        const int kw = kt + WS < nk ? kt + WS : nk - 1;
        const bf16x8 *wnext = wp + (int64_t)kw * NWP * 64;
        // quarter p of a tile: 32 columns (step p / 2) of one half of the rows
        auto read_frags = [&](int p, bf16x8 (&fb)[HRB]) {
#pragma unroll
            for (int j = 0; j < HRB; ++j) {
                const int row = 16 * ((p & 1) * HRB + j) + l16;
                fb[j] = *(const bf16x8 *)&xb[row * BK + 8 * ((4 * (p >> 1) + quart) ^ ((row >> 1) & 7))];
            }
        };
        auto multiply = [&](int p, const bf16x8 (&fb)[HRB]) {
#pragma unroll
            for (int i = 0; i < WFB; ++i)
#pragma unroll
                for (int j = 0; j < HRB; ++j) {
                    f32x4 &c = acc[i][(p & 1) * HRB + j];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[S][(p >> 1) * WFB + i], fb[j], c, 0, 0, 0);
                }
        };
        if constexpr (GUARDED) {
            if (kt < nk) {
                bf16x8 bfr[2][HRB];
                read_frags(0, bfr[0]);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    if (p < 3) read_frags(p + 1, bfr[(p + 1) & 1]);
                    multiply(p, bfr[p & 1]);
                }
            }
            load_w(kw, wr[S]);
        } else {
            // operand fragments of the next quarter are read ahead where the registers allow (64-row tiles)
            constexpr int NBUF = HRB <= 2 ? 2 : 1;
            bf16x8 bfr[NBUF][HRB];
            read_frags(0, bfr[0]);
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if (NBUF == 2 && p < 3) read_frags(p + 1, bfr[(p + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(p, bfr[p % NBUF]);
                // (the compiler's mixture of MFMAs, fragment reads and requests is as good as any order tried; 64-row tiles with the
                // refill strictly behind the MFMAs: 60 tokens of 32 layers 42.3 us either way, 40 tokens 35.7 -> 36.2, 20 32.1 -> 32.5)
                if (NBUF == 1 && p < 3) read_frags(p + 1, bfr[0]);
                if (p & 1)
#pragma unroll
                    for (int i = 0; i < WFB; ++i) wr[S][(p >> 1) * WFB + i] = wnext[wpiece((p >> 1) * WFB + i)];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // whole trips of UN steps (at the top of a trip the compiler's wait is a conservative one, so trips are long), then
    // the remaining steps in rounds of WS
    constexpr int UN = Gm::UN;
    static_assert(UN % WS == 0, "a trip of the tile loop is a whole number of register-ring rounds");
    const int nk_main = nk / UN * UN;
#pragma unroll 1
    for (int kt0 = 0; kt0 < nk_main; kt0 += UN)
        static_for<UN>([&](auto u) { tile_step(std::integral_constant<int, decltype(u)::value % WS>{}, std::false_type{}, kt0 + decltype(u)::value); });
    const int nk_end = nk_main + (nk - nk_main + WS - 1) / WS * WS;
#pragma unroll 1
    for (int kt0 = nk_main; kt0 < nk_end; kt0 += WS)
        static_for<WS>([&](auto u) { tile_step(u, std::true_type{}, kt0 + decltype(u)::value); });
    // acc[i][j][v]: feature wave FW + 16 i + 4 quart + v, row 16 j + l16
    lsa_fused_epilogue<DH, NB, TT, DENSE>([&](auto put) {
#pragma unroll
        for (int i = 0; i < WFB; ++i)
#pragma unroll
            for (int j = 0; j < NRB; ++j)
                put(16 * j + l16, wave * FW + 16 * i + 4 * quart, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    }, a, sm, tok0, g, part);
}

// The workgroups in front of the kernel's own do the step's integer work or read ahead (NB, TT: the tile that asks for it).
// (Not one function that also says whether a workgroup is the kernel's own: with that the 96-row form spilled two registers,
// 10 tokens x 80 layers 49.5 -> 50.3 us.)
template <int DH, int NB, int TT>
__device__ __forceinline__ void lsa_pk_lead(const LsaFusedArgs &a)
{
    extern __shared__ __attribute__((aligned(16))) bf16_t sm[];
    if ((int)blockIdx.x >= a.lead_blocks - a.pf_lead)
        lsa_warm_block<DH, NB, TT>(a, (int)blockIdx.x - (a.lead_blocks - a.pf_lead), sm);
    else if ((int)blockIdx.x < a.rider_units && threadIdx.x < 64)
        step_small_unit(a.rider, (int)blockIdx.x, (int32_t *)sm, (int32_t *)sm + MOA_MAX_TREE);
}

// the unit and the tile of one of the kernel's own workgroups; units past the last have nothing to do
struct LsaPkPlace {
    int unit;
    int64_t tile;
    __device__ __forceinline__ LsaPkPlace(const LsaFusedArgs &a)
    {
        const int bx = (int)blockIdx.x - a.lead_blocks;
        const int xcd = bx & 7, slot = bx >> 3;
        unit = xcd * a.units_per_xcd + slot % a.units_per_xcd;
        tile = slot / a.units_per_xcd;
    }
};

template <int DH, int NB, int TT>
__global__ __launch_bounds__(512) void k_lsa_fused_pk(LsaFusedArgs a)
{
    if ((int)blockIdx.x < a.lead_blocks) {
        lsa_pk_lead<DH, NB, TT>(a);
        return;
    }
    const LsaPkPlace at(a);
    if (at.unit >= a.units) return;              // the whole workgroup leaves before any barrier
    lsa_pk_tile<DH, NB, TT, false>(a, at.unit, at.tile * TT);
}
// The first `wide_tiles` tiles take five tokens (160 rows), those behind them TT (where the line lies: lsa_fused_plan).  160
// rows bring a weight tile to more of them (63 us a round against 51 for 128), and their parked tile fills the LDS
// like a dense one's; ten (token, head) units on eight wavefronts cost the second pass.
template <int DH, int TT>
__global__ __launch_bounds__(512) void k_lsa_fused_pk_wide(LsaFusedArgs a)
{
    if ((int)blockIdx.x < a.lead_blocks) {
        lsa_pk_lead<DH, 1, TT>(a);
        return;
    }
    const LsaPkPlace at(a);
    if (at.unit >= a.units) return;
    if (at.tile < a.wide_tiles) lsa_pk_tile<DH, 1, 5, false>(a, at.unit, at.tile * 5);
    else lsa_pk_tile<DH, 1, TT, false>(a, at.unit, a.wide_tiles * 5 + (at.tile - a.wide_tiles) * TT);
}
// The same with the rows of TT tokens one behind another in 160 (five blocks of 32), for layer counts that leave much of
// their last block empty: 80 layers in 96 rows waste a sixth of the matrix work, two tokens in 160 nothing, and a weight
// tile serves 160 rows.  The accumulators take 160 registers, so one weight tile is in registers instead of two, and the parked tile
// fills the LDS to the last byte.  240 tokens x 80 layers (d_in 2048): 253 - 257 us; a token per workgroup takes 370 - 375,
// projection and attention as kernels of their own 257 + 55.  That is four rounds of 64 us: 1.7 per k tile at 160 rows, with the MFMA
// pipe busy for 65 % of the SIMDs' time, and 10 in front and behind (one round, 64 tokens: 39, 66 and 120 us at d_in 1024, 2048, 4096),
// from which giving a unit's query blocks to two wavefronts had taken 6.
template <int DH, int NB, int TT>
__global__ __launch_bounds__(512) void k_lsa_fused_pk_dense(LsaFusedArgs a)
{
    if ((int)blockIdx.x < a.lead_blocks) {
        lsa_pk_lead<DH, NB, TT>(a);
        return;
    }
    const LsaPkPlace at(a);
    if (at.unit >= a.units) return;
    lsa_pk_tile<DH, NB, TT, true>(a, at.unit, at.tile * TT);
}

// Packs Wq / Wk / Wv for k_lsa_fused_pk: piece (unit, wavefront, k tile, k step, feature block, lane) holds the 8
// elements that lane supplies as the A operand of that MFMA, i.e. row  f(unit, wavefront) + 32 block + lane % 32  of
// the wavefront's matrix at columns  64 tile + 16 step + 8 (lane / 32) ..  One thread per piece.
template <int DH>
__global__ __launch_bounds__(256) void k_lsa_pack_weights(const bf16_t *wq, const bf16_t *wk, const bf16_t *wv, bf16_t *out,
                                                          int d_in, int Hq, int Hkv, int64_t pieces)
{
    constexpr int FW = 4 * DH / 8, WFB = FW / 32;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= pieces) return;
    const int nk = d_in / 64, G = Hq / Hkv, parts = G / 2;
    int64_t r = p;
    const int lane = (int)(r % 64); r /= 64;
    const int i = (int)(r % WFB); r /= WFB;
    const int ks = (int)(r % 4); r /= 4;
    const int kt = (int)(r % nk); r /= nk;
    const int wave = (int)(r % 8); r /= 8;
    const int unit = (int)r;
    const int g = unit / parts, part = unit - g * parts;
    const int which = wave * FW / DH;
    const int frow = wave * FW % DH + 32 * i + (lane & 31);
    const bf16_t *src = which < 2 ? wq + (int64_t)((g * G + 2 * part + which) * DH + frow) * d_in
                                  : (which == 2 ? wk : wv) + (int64_t)(g * DH + frow) * d_in;
    *(u32x4 *)(out + p * 8) = *(const u32x4 *)(src + 64 * kt + 16 * ks + 8 * (lane >> 5));
}

// ------------------------------------------------------------------ host side
bool lsa_fused_ok(int dtype, int L, int d_in, int Hq, int Hkv, int dh, const void *hs, const void *wq, const void *wk,
                  const void *wv, const void *abar)
{
    auto al = [](const void *p) { return p && (((uintptr_t)p) & 15) == 0; };
    if (!lsa_fused_shape_ok(dtype, L, d_in, Hq, Hkv, dh)) return false;
    return al(hs) && al(wq) && al(wk) && al(wv) && al(abar);
}

bool lsa_fused_shape_ok(int dtype, int L, int d_in, int Hq, int Hkv, int dh)
{
    if (dtype != DT_BF16 || dh != 128) return false;
    if (L < 1 || L > 96 || d_in < 128 || d_in % 64) return false;
    if (Hkv < 1 || Hq % Hkv || (Hq / Hkv) % 2) return false;
    return true;
}

// LDS a workgroup may ask for on the current device (looked up once per device; 0 if the query fails)
static size_t lds_limit()
{
    static size_t limit[16] = {};
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 0;
    if (!limit[dev]) {
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0) return 0;
        limit[dev] = (size_t)v;
    }
    return limit[dev];
}

bool lsa_dense_ok(int L) { return lsa_dense_layers(L) && lds_limit() >= LSA_BIG_LDS; }
static_assert(LsaFusedGeom<128, 1, 4>::bytes == LSA_BIG_LDS && LsaFusedGeom<128, 2, 2>::bytes == LSA_BIG_LDS &&
                  LsaFusedGeom<128, 1, 5>::pk_bytes == LSA_BIG_LDS && LsaFusedGeom<128, 3, 2, true>::pk_bytes == LSA_BIG_LDS &&
                  LsaFusedGeom<128, 1, 3>::bytes < LSA_BIG_LDS && LsaFusedGeom<128, 3, 1>::bytes < LSA_BIG_LDS,
              "the forms the plan takes for those that fill the LDS");

template <int NB, int TT, bool DENSE = false>
static hipError_t launch_lsa_fused_as(LsaFusedArgs &fa, hipStream_t stream)
{
    using Gm = LsaFusedGeom<128, NB, TT, DENSE>;
    const int64_t rest = fa.T - 5 * fa.wide_tiles, tiles = fa.wide_tiles + (rest > 0 ? (rest + TT - 1) / TT : 0);
    // Two helper workgroups per XCD (lsa_warm_block), where they cost nothing and can do their job: the kernel's own
    // workgroups leave that many compute units idle (decode sizes), and an XCD's share of the weights fits its L2
    // beside the activations streaming through.  Otherwise they take compute units and L2 from the workgroups they
    // are meant to help (measured: first cycle 536 -> 559 us, d_in 4096 191 -> 197 us with helpers everywhere).
    if (fa.pf_lead) {
        static int cus = 0;
        if (!cus) {
            int dev = 0, n = 0;
            if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
            cus = n;
        }
        const int64_t own = 8 * (int64_t)fa.units_per_xcd * tiles;
        const size_t w_per_xcd = (size_t)fa.units_per_xcd * (size_t)(fa.d_in / 64) * 65536;
        if (own + fa.pf_lead > cus || w_per_xcd > ((size_t)3 << 20)) fa.pf_lead = 0;
        fa.lead_blocks += fa.pf_lead;
    }
    const int64_t grid = fa.lead_blocks + 8 * (int64_t)fa.units_per_xcd * tiles;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    if constexpr (DENSE) {
        static bool raised[16] = {};
        hipError_t e = raise_lds_limit_once(raised, (const void *)k_lsa_fused_pk_dense<128, NB, TT>, Gm::pk_bytes);
        if (e != hipSuccess) return e;
        prof_begin(K_LSA_FUSED_PK + 64 * (64 + NB * 8 + TT), stream);
        MOA_KLAUNCH((k_lsa_fused_pk_dense<128, NB, TT>), dim3((unsigned)grid), dim3(512), Gm::pk_bytes, stream, fa);
    } else if (fa.wide_tiles) {
        if constexpr (NB == 1) {
            using Wide = LsaFusedGeom<128, 1, 5>;
            constexpr size_t lds = Wide::pk_bytes > Gm::pk_bytes ? Wide::pk_bytes : Gm::pk_bytes;
            static bool raised[16] = {};
            hipError_t e = raise_lds_limit_once(raised, (const void *)k_lsa_fused_pk_wide<128, TT>, lds);
            if (e != hipSuccess) return e;
            prof_begin(K_LSA_FUSED_PK + 64 * (32 + TT), stream);
            MOA_KLAUNCH((k_lsa_fused_pk_wide<128, TT>), dim3((unsigned)grid), dim3(512), lds, stream, fa);
        }
    } else if (fa.wpk) {
        static bool raised[16] = {};
        hipError_t e = raise_lds_limit_once(raised, (const void *)k_lsa_fused_pk<128, NB, TT>, Gm::pk_bytes);
        if (e != hipSuccess) return e;
        prof_begin(K_LSA_FUSED_PK + 64 * (NB * 8 + TT), stream);
        MOA_KLAUNCH((k_lsa_fused_pk<128, NB, TT>), dim3((unsigned)grid), dim3(512), Gm::pk_bytes, stream, fa);
    } else {
        static bool raised[16] = {};
        hipError_t e = raise_lds_limit_once(raised, (const void *)k_lsa_fused<128, NB, TT>, Gm::bytes);
        if (e != hipSuccess) return e;
        prof_begin(K_LSA_FUSED + 64 * (NB * 8 + TT), stream);
        MOA_KLAUNCH((k_lsa_fused<128, NB, TT>), dim3((unsigned)grid), dim3(512), Gm::bytes, stream, fa);
    }
    prof_end(stream);
    return hipGetLastError();
}

size_t lsa_packed_weight_bytes(int d_in, int Hq, int Hkv, int dh)
{
    // a workgroup's unit is two query heads with their key and value head: 4 dh rows; a group of more than two query
    // heads repeats its K and V rows in each of its units
    return (size_t)(Hq / 2) * 4 * dh * d_in * sizeof(bf16_t);
}

hipError_t launch_lsa_pack_weights(const void *wq, const void *wk, const void *wv, void *out, int d_in, int Hq, int Hkv,
                                   hipStream_t stream)
{
    const int64_t pieces = (int64_t)(Hq / 2) * 4 * 128 * d_in / 8;
    const int64_t grid = (pieces + 255) / 256;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    prof_begin(K_LSA_PACK, stream);
    MOA_KLAUNCH((k_lsa_pack_weights<128>), dim3((unsigned)grid), dim3(256), 0, stream, (const bf16_t *)wq, (const bf16_t *)wk,
                (const bf16_t *)wv, (bf16_t *)out, d_in, Hq, Hkv, pieces);
    prof_end(stream);
    return hipGetLastError();
}

hipError_t launch_lsa_fused(const LsaFusedCall &c, hipStream_t stream)
{
    if (c.T <= 0) return hipSuccess;
    LsaFusedArgs fa = {};
    fa.hs = (const bf16_t *)c.hs;
    fa.wq = (const bf16_t *)c.wq;
    fa.wk = (const bf16_t *)c.wk;
    fa.wv = (const bf16_t *)c.wv;
    fa.wpk = (const bf16_t *)c.w_packed;
    fa.abar = (bf16_t *)c.abar;
    fa.T = c.T;
    fa.L = c.L;
    fa.d_in = c.d_in;
    fa.Hq = c.Hq;
    fa.Hkv = c.Hkv;
    fa.parts = c.Hq / c.Hkv / 2;
    fa.units = c.Hkv * fa.parts;
    fa.units_per_xcd = (fa.units + 7) / 8;
    fa.rider_units = c.rider_units;
    if (c.rider_units > 0) fa.rider = c.rider;
    fa.lead_blocks = (c.rider_units + 7) & ~7;   // multiples of the XCD count: the unit mapping keeps its phase
    fa.pf_lead = c.w_packed ? 16 : 0;     // wanted; launch_lsa_fused_as decides when it knows the grid
    const LsaFusedPlan plan = lsa_fused_plan(fa.wpk != nullptr, c.T, c.L, c.d_in, fa.units, lds_limit());
    fa.wide_tiles = plan.wide_tiles;
    const int nb = (c.L + 31) / 32;
    if (nb == 1 && plan.tokens == 4) return launch_lsa_fused_as<1, 4>(fa, stream);
    if (nb == 1 && plan.tokens == 3) return launch_lsa_fused_as<1, 3>(fa, stream);
    if (nb == 1) return launch_lsa_fused_as<1, 2>(fa, stream);
    if (nb == 2 && plan.tokens == 2) return launch_lsa_fused_as<2, 2>(fa, stream);
    if (nb == 2) return launch_lsa_fused_as<2, 1>(fa, stream);
    if (plan.dense) return launch_lsa_fused_as<3, 2, true>(fa, stream);
    return launch_lsa_fused_as<3, 1>(fa, stream);
}

}  // namespace moa
