// The attention core over a split key range (see moa_attn.hip) in tiles of 256 query rows per workgroup.
// head_dim 128 and more than 128 rows per (sequence, KV head).  Four wavefronts, one per SIMD, 64 query rows each (two blocks
// of 32), so that an operand read from LDS serves two MFMAs: with 32 rows per wavefront the reads of K and V alone keep LDS
// busy for three quarters of the matrix time.  Per 32 keys a wavefront has 32 MFMAs (1024 clocks) and about 900 clocks of
// other instructions, and nobody else on its SIMD to overlap them with, so the loop is laid out as phases of 16 MFMAs with
// one score element's arithmetic behind each:
//   phase 0 of 32 keys j:  S(j+1) of block 0 and P V(j-1) of block 1, between them the softmax of S(j) of block 0
//   phase 1:               S(j+1) of block 1 and P V(j)   of block 0, between them the softmax of S(j) of block 1
// The operands of a phase were read from LDS one phase earlier, each into the place of one just used.
// With one wavefront per SIMD every instruction costs its four clocks, one that needs the result of the instruction before it
// eight, so what is not arithmetic was taken out of the loop and the rest put in an order (measured, 8 x 32768 keys x 128
// nodes, both cores, clocks per 32 keys x 64 rows, by the wavefronts' counters: 2480 before, 1860 now, of which 1240 issue and
// 210 wait for the matrix pipe):
//   - three sets of scores change roles from phase to phase and the loop body is three tiles, so no score is moved;
//   - the queries are pinned to the accumulation registers, which an MFMA reads directly (left alone the compiler keeps
//     them there and copies four registers in front of each MFMA);
//   - an element's scaled score, its exponential and the use of the weight stand in three successive MFMA slots, and
//     the last weights of a phase are packed in the next one;
//   - LDS addresses are one base per operand with the piece XORed in; the loads of the tile three ahead are two to a phase;
//   - the masks stand only in the loop behind the full tiles.
// (Sums of the rounded weights by dot instructions: each costs 28 clocks between MFMAs, since it uses their pipe.)
// K and V come in tiles of 64 keys straight into an LDS ring of four (a piece of row r lies at position c ^ f(r), f a
// permutation of 0 .. 15 on 16 neighbouring rows: operand reads of K touch 16 rows of one column, the transposing reads of V
// eight rows of 64 bytes); one barrier per tile, two tiles in flight behind the current one.
// The reference of the exponent is the running maximum, exactly: the heaviest weights then sit at the top of a binade, where
// their rounding to bf16 is smallest (a reference that lags behind it by up to 2^8 gives 1.04 to 1.24 times the error against
// 64 bits, and would save 7 % of the time).  A rescale is 64 multiplications, so the accumulators are kept in vector
// registers and the operands that come from LDS in the accumulation registers, the other way round than the compiler's
// default (-amdgpu-mfma-vgpr-form for this file; in accumulation registers a rescale takes four times as long).
// What bounds it is instruction issue beside the matrix pipe, at the 1.9 GHz that the clock falls to under it.  8 x 32768 keys
// x 128 tree tokens, both cores, on one card: 1340 us with copies and everything in dependence order, 1150 now (0.96 PFLOP/s);
// 128 rows per workgroup take 1464 where the former took 1352.
#include "moa_attn_device.h"
#include "moa_gemm_device.h"

#include <math.h>

#include <type_traits>

namespace moa {

constexpr int LRING = 4;

template <int DH, int CALLS>
__global__ __launch_bounds__(256, 1) void k_attn_long(AttnGroup<CALLS> grp, SplitGeom geo)
{
    static_assert(DH == 128, "a row is 16 pieces of 16 bytes");
    constexpr int NKS = DH / 16, NDB = DH / 32;
    constexpr uint32_t ROWB = DH * 2, HALFT = LK * ROWB, TILEB = 2 * HALFT;    // bytes of a row, of a tile's K or V, of a tile
    extern __shared__ __attribute__((aligned(1024))) char smem[];      // operand addresses are made by XOR of low bits

    // Workgroups are dealt to the 8 XCDs round-robin: the row tiles of one key range are neighbours on one XCD, whose L2
    // then serves all but the first.
    const int xcd = (int)blockIdx.x & 7, slot0 = (int)blockIdx.x >> 3;
    const int unit = 8 * (slot0 / geo.rowtiles) + xcd, rowtile = slot0 % geo.rowtiles;
    if (unit >= geo.nsplit * grp.nbg * grp.ncalls) return;       // the whole workgroup, before any barrier
    const int split = unit % geo.nsplit, cbg = unit / geo.nsplit;
    const int call = cbg / grp.nbg, bg = cbg - call * grp.nbg;
    const AttnArgs &a = grp.a[call];
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.H / a.Hkv, RG = G * a.Mq, W = (a.mask_rows + 63) >> 6;
    const float sc = 1.4426950408889634f / sqrtf((float)DH);   // scores are kept in the log2 domain

    const int len = clamp_len(a.len[b], a.P_cap, tid == 0 ? a.dev_status : nullptr);
    const int nt = (len + LK - 1) / LK;
    const int per = (nt + geo.nsplit - 1) / geo.nsplit;
    const int t0 = min(split * per, nt), nc = min(t0 + per, nt) - t0;          // this slice's tiles of the cache
    const int Mt = a.mask ? a.Mt : 0;
    const int ntiles = __builtin_amdgcn_readfirstlane(nc + (split == geo.nsplit - 1 ? (Mt + LK - 1) / LK : 0));

    const char *kc = (const char *)a.kcache + (int64_t)bg * a.P_cap * ROWB, *vc = (const char *)a.vcache + (int64_t)bg * a.P_cap * ROWB;
    const char *ktp = (const char *)a.ktree + (int64_t)bg * a.tree_cap * ROWB, *vtp = (const char *)a.vtree + (int64_t)bg * a.tree_cap * ROWB;

    const int rowbase = rowtile * 256 + wave * 64;
    bf16x8 qf[2][NKS];
    int mrow[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const int rho = min(rowbase + 32 * blk + l32, RG - 1);
        mrow[blk] = rho / G;
        const bf16_t *qrow = (const bf16_t *)a.q + (((int64_t)b * a.Mq + mrow[blk]) * a.H + g * G + (rho - mrow[blk] * G)) * DH;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[blk][ks] = *(const bf16x8 *)(qrow + 16 * ks + 8 * half);
    }

    // tile i of this workgroup: cache tile t0 + i, then the tree's; past the last one it is the last one again (nobody reads
    // that).  Wavefront w moves rows 16 w .. 16 w + 15 of K and of V, four rows an instruction.
    auto first_row = [&](int i) { return i < nc ? (t0 + i) * LK : (i - nc) * LK; };
    auto rows_valid = [&](int i) { return (i < nc ? len : Mt) - first_row(i); };             // >= 1
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    // one wavefront's part of a tile is eight such loads, two to a phase: all at once they queue up at the compute unit's one
    // address unit and the wavefronts wait there
    struct Src { const char *k, *v; uint32_t dst; int last; };
    auto source = [&](int i_) {
        const int i = min(i_, ntiles - 1);
        const int64_t at = (int64_t)first_row(i) * ROWB;
        return Src{(i < nc ? kc : ktp) + at, (i < nc ? vc : vtp) + at,
                   lds0 + (uint32_t)(i_ & (LRING - 1)) * TILEB + (uint32_t)wave * 16 * ROWB, min(rows_valid(i), LK) - 1};
    };
    auto load_off = [&](const Src &s, int j) {
        const int row = 16 * wave + 4 * j + (lane >> 4);
        return (uint32_t)min(row, s.last) * ROWB + 16 * ((lane & 15) ^ (4 * (lane >> 4) + j));
    };
    auto issue = [&](int i) {
        const Src s = source(i);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lds_dma16(s.dst + 4 * j * ROWB, load_off(s, j), s.k);
            lds_dma16(s.dst + HALFT + 4 * j * ROWB, load_off(s, j), s.v);
        }
    };

    f32x16 acc[2][NDB];
    float mref[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};     // exponent's reference (log2 domain); this lane's part of the sum
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[blk][d][e] = 0.f;

    if (ntiles > 0) {
        // Operand reads, from the first tile's place on: piece 2 ks + half of K row l32 lies kbase ^ 32 ks, and of the V rows
        // the pieces of d at vbase ^ 64 d (and ^ 32, eight rows on, for the second half of an operand).
        // transpose read: lane j of a 16-lane group addresses key (j >> 2), head_dim 4 (j & 3) of the group's 16
        const int vkey = (lane & 15) >> 2;
        uint32_t kbase = lds0 + l32 * ROWB + 16 * (half ^ (4 * (l32 & 3) + ((l32 >> 2) & 3)));
        uint32_t vbase = lds0 + HALFT + (4 * half + vkey) * ROWB + 8 * (lane & 1) +
                         16 * ((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ (4 * vkey + half));

        bf16x8 kf[NKS], vf[2 * NDB];
        u32x4 pf[2][2];
        f32x16 s0, s1, s2;                        // scores: those being turned into weights, those waiting, those being made
        float tmax[2], neg[2] = {0.f, 0.f};       // maximum of the scores that the next softmax of either block takes; minus mref
        float late[2] = {0.f, 0.f};               // the last two weights of the phase before
        bool moved = true;                        // a score of the next softmax is above mref
        auto read_k = [&](int ks, int sub) { kf[ks] = *(const __attribute__((address_space(3))) bf16x8 *)(uintptr_t)((kbase ^ (32 * ks)) + sub * 32 * ROWB); };
        auto read_v = [&](int x, int sub) {               // x = 4 st2 + d: keys 16 st2 .., head_dim 32 d ..
            union { i16x4 h[2]; bf16x8 v; } u;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                u.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(uintptr_t)(
                    (vbase ^ (64 * (x % NDB) + 32 * h)) + (sub * 32 + (x / NDB) * 16 + 8 * h) * ROWB));
            vf[x] = u.v;
        };
        // keys that do not count (tree rows outside the ancestor set, rows past the end) get -inf
        auto mask_scores = [&](f32x16 &s, int blk, int i, int sub) {
            if (i >= ntiles) return;
            const int base = 32 * sub, nvalid = rows_valid(i) - base;
            if (i < nc && nvalid >= 32) return;                  // the same decision in the whole workgroup
            uint32_t vis = nvalid >= 32 ? 0xffffffffu : nvalid <= 0 ? 0u : (1u << nvalid) - 1u;
            if (i >= nc && nvalid > 0)
                vis &= (uint32_t)(a.mask[((int64_t)b * a.mask_rows + a.mask_row0 + mrow[blk]) * W + (i - nc)] >> base);
            vis >>= 4 * half;
            float tm = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (!(vis & (1u << (8 * (v >> 2) + (v & 3))))) s[v] = -INFINITY;
                tm = fmaxf(tm, s[v]);
            }
            tmax[blk] = tm;
            moved = __ballot(tm * sc > mref[blk]) != 0;
        };
        // BLK: the block whose softmax this phase does, of the scores `scur`; `swait` are the other block's, of which the
        // maximum is taken; `snew` takes this block's next ones.  Phase 0 reads V rows of 32-key half SUB of the current
        // tile, phase 1 K rows of the next tile's.  The scheduling barriers keep each step's arithmetic between its MFMAs, and no
        // instruction next to the one it depends on; the last weights of a phase are dealt with in the next one.
        auto phase = [&](auto blk_c, auto sub_c, const Src &src, f32x16 &scur, f32x16 &swait, f32x16 &snew) {
            constexpr int BLK = decltype(blk_c)::value, OB = 1 - BLK, SUB = decltype(sub_c)::value;
            if (__builtin_expect(moved, 0)) {
                // the other half's maximum by a lane swap in the vector unit: a shuffle would wait for the operand reads in flight
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax[BLK]), __float_as_uint(tmax[BLK]), false, false);
                const float tm = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
                const float mnew = fmaxf(mref[BLK], tm * sc);    // sc > 0: scaling keeps the order (and -inf)
                const float msafe = mnew == -INFINITY ? 0.f : mnew, corr = fast_exp2(mref[BLK] - msafe);
                mref[BLK] = mnew;
                neg[BLK] = -msafe;
                lsum[BLK] *= corr;
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[BLK][d][e] *= corr;
            }
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+a"(qf[BLK][ks]));
            asm volatile("" : "+v"(kbase), "+v"(vbase));      // the addresses made from them are not kept for the next phase
            float p[16], tm = -INFINITY, top = 0.f;
            uint32_t off = 0;
            float arg = fmaf(scur[0], sc, neg[BLK]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int x = e / 2;
                if (e == 0) {
                    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    snew = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[BLK][x], zero, 0, 0, 0);
                } else if (e % 2 == 0) snew = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[BLK][x], snew, 0, 0, 0);
                else acc[OB][x % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[x], __builtin_bit_cast(bf16x8, pf[OB][x / NDB]), acc[OB][x % NDB], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (BLK == 0 && e % 2 == 1) read_v(x, SUB);
                if (BLK == 1 && e % 2 == 0) read_k(x, SUB);
                if (e == 2 + BLK) off = load_off(src, 2 * SUB + BLK);
                if (e == 4 + BLK) lds_dma16(src.dst + 4 * (2 * SUB + BLK) * ROWB, off, src.k);
                if (e == 10 + BLK) lds_dma16(src.dst + HALFT + 4 * (2 * SUB + BLK) * ROWB, off, src.v);
                __builtin_amdgcn_sched_barrier(0);
                p[e] = fast_exp2(arg);
                asm volatile("" : "+v"(p[e]));
                __builtin_amdgcn_sched_barrier(0);
                if (e % 2 == 0) {                               // P^T slot t of step st2 is key 16 st2 + 8 (t >> 2) + 4 half + (t & 3)
                    uint32_t pk = e == 0 ? pack_bf16x2(late[0], late[1]) : pack_bf16x2(p[e - 2], p[e - 1]);
                    asm volatile("" : "+v"(pk));
                    if (e == 0) pf[OB][1][3] = pk;
                    else pf[BLK][(e - 2) / 8][(e - 2) % 8 / 2] = pk;
                } else if (e < 15) {                            // maxima 0, 1 | 2, 3 | .. of the other block's scores: done before the end
                    tm = fmaxf(fmaxf(tm, swait[e - 1]), swait[e]);
                    asm volatile("" : "+v"(tm));
                    if (e == 13) {
                        tm = fmaxf(fmaxf(tm, swait[14]), swait[15]);
                        asm volatile("" : "+v"(tm));
                    }
                } else {
                    top = tm * sc;
                    asm volatile("" : "+v"(top));
                }
                __builtin_amdgcn_sched_barrier(0);
                if (e == 0) {
                    lsum[OB] += late[1];
                    asm volatile("" : "+v"(lsum[OB]));
                } else {
                    lsum[BLK] += p[e - 1];
                    asm volatile("" : "+v"(lsum[BLK]));
                }
                __builtin_amdgcn_sched_barrier(0);
                if (e < 15) {
                    arg = fmaf(scur[e + 1], sc, neg[BLK]);
                    asm volatile("" : "+v"(arg));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            late[0] = p[14];
            late[1] = p[15];
            tmax[OB] = tm;
            moved = __ballot(top > mref[OB]) != 0;
        };
        typedef std::integral_constant<int, 0> C0;
        typedef std::integral_constant<int, 1> C1;

        issue(0);
        issue(1);
        wait_loads_and_barrier<8>();
        issue(2);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) read_k(ks, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) s0[e] = s1[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[0][ks], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[1][ks], s1, 0, 0, 0);
        }
        tmax[0] = s0[0];
#pragma unroll
        for (int e = 0; e < 16; ++e) tmax[0] = fmaxf(tmax[0], s0[e]);
        mask_scores(s0, 0, 0, 0);
        moved = true;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) read_k(ks, 1);
        kbase += TILEB;                            // of the tile after the current one from here on
#pragma unroll
        for (int x = 0; x < 2 * NDB; ++x)
#pragma unroll
            for (int t = 0; t < 8; ++t) vf[x][t] = (__bf16)0.f;
#pragma unroll
        for (int st2 = 0; st2 < 2; ++st2)
#pragma unroll
            for (int t = 0; t < 4; ++t) pf[1][st2][t] = 0u;

        auto tile = [&](auto mask_c, int t, f32x16 &a0, f32x16 &a1, f32x16 &a2) {
            constexpr bool MASK = decltype(mask_c)::value;
            // tile t + 1 is in LDS for everybody, nobody reads tile t - 1 any more (the eight reads of K that may be in
            // flight are the last phase's)
            asm volatile("s_waitcnt vmcnt(8) lgkmcnt(8)\n\ts_barrier" ::: "memory");
            const Src src = source(t + 3);
            phase(C0{}, C0{}, src, a0, a1, a2);
            if (MASK) mask_scores(a1, 1, t, 0);
            phase(C1{}, C0{}, src, a1, a2, a0);
            if (MASK) mask_scores(a2, 0, t, 1);
            phase(C0{}, C1{}, src, a2, a0, a1);
            if (MASK) mask_scores(a0, 1, t, 1);
            phase(C1{}, C1{}, src, a0, a1, a2);
            if (MASK) mask_scores(a1, 0, t + 1, 0);
            kbase += (t & (LRING - 1)) == LRING - 2 ? (uint32_t)-(LRING - 1) * TILEB : TILEB;
            vbase += (t & (LRING - 1)) == LRING - 1 ? (uint32_t)-(LRING - 1) * TILEB : TILEB;
        };
        // three sets of scores change places from phase to phase, so that three tiles make a round without moving any
        const int nfull = min(nc, (len - t0 * LK) / LK);           // tiles of the cache without rows past the end
        int t = 0;
        for (; t + 3 < nfull; t += 3) {
            tile(std::false_type{}, t, s0, s1, s2);
            tile(std::false_type{}, t + 1, s1, s2, s0);
            tile(std::false_type{}, t + 2, s2, s0, s1);
        }
        for (; t < ntiles; ++t) {
            tile(std::true_type{}, t, s0, s1, s2);
            const f32x16 s = s0;
            s0 = s1;
            s1 = s2;
            s2 = s;
        }
        pf[1][1][3] = pack_bf16x2(late[0], late[1]);
        lsum[1] += late[1];
#pragma unroll
        for (int x = 0; x < 2 * NDB; ++x)
            acc[1][x % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[x], __builtin_bit_cast(bf16x8, pf[1][x / NDB]), acc[1][x % NDB], 0, 0, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }

    // One slice: the result.  Several: the slice's own normalised output (a convex combination of V rows, so it fits fp16
    // with 2^-12 relative rounding, eight times finer than the bf16 result), reference and sum in fp32.
    f16_t *__restrict__ part_o = (f16_t *)a.ws;
    float *__restrict__ part_ml = (float *)(part_o + (size_t)grp.nbg * geo.nsplit * geo.rows_pad * DH);
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const float l = lsum[blk] + __shfl_xor(lsum[blk], 32);
        const int rho = rowbase + 32 * blk + l32;
        if (rho >= RG) continue;
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        if (geo.nsplit == 1) {
            bf16_t *o = (bf16_t *)a.out + (((int64_t)b * a.Mq + mrow[blk]) * a.H + g * G + (rho - mrow[blk] * G)) * DH + 4 * half;
#pragma unroll
            for (int d = 0; d < NDB; ++d)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    u32x2 pk;
                    pk[0] = pack_bf16x2(acc[blk][d][4 * q4] * inv, acc[blk][d][4 * q4 + 1] * inv);
                    pk[1] = pack_bf16x2(acc[blk][d][4 * q4 + 2] * inv, acc[blk][d][4 * q4 + 3] * inv);
                    *(u32x2 *)(o + 32 * d + 8 * q4) = pk;
                }
            if (l == 0.f && a.empty_is_error && half == 0 && a.dev_status) atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
            continue;
        }
        const int64_t prow = ((int64_t)bg * geo.nsplit + split) * geo.rows_pad + rho;
        if (half == 0) {
            part_ml[prow * 2 + 0] = mref[blk];
            part_ml[prow * 2 + 1] = l;
        }
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f16x4 v = {(f16_t)(acc[blk][d][4 * q4] * inv), (f16_t)(acc[blk][d][4 * q4 + 1] * inv),
                           (f16_t)(acc[blk][d][4 * q4 + 2] * inv), (f16_t)(acc[blk][d][4 * q4 + 3] * inv)};
                *(f16x4 *)(part_o + prow * DH + 32 * d + 8 * q4 + 4 * half) = v;
            }
    }
}

template <int CALLS>
hipError_t launch_attn_long(const AttnGroup<CALLS> &grp, const SplitGeom &g, hipStream_t stream)
{
    constexpr size_t lds = (size_t)LRING * LK * 128 * 2 * 2;
    static bool raised[16] = {};
    hipError_t e = raise_lds_limit_once(raised, (const void *)k_attn_long<128, CALLS>, lds);
    if (e != hipSuccess) return e;
    const int64_t units8 = ((int64_t)g.nsplit * grp.ncalls * grp.nbg + 7) / 8, grid = 8 * units8 * g.rowtiles;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    prof_begin(K_ATTN_LONG, stream);
    MOA_KLAUNCH((k_attn_long<128, CALLS>), dim3((unsigned)grid), dim3(256), lds, stream, grp, g);
    prof_end(stream);
    return hipGetLastError();
}

template hipError_t launch_attn_long(const AttnGroup<ATTN_FEW> &, const SplitGeom &, hipStream_t);
template hipError_t launch_attn_long(const AttnGroup<ATTN_CALLS> &, const SplitGeom &, hipStream_t);

}  // namespace moa
