// Which tile the one-kernel Layer Self-Attention (moa_lsa_fused.hip) takes.  Host arithmetic only, so that a test on a machine
// without a GPU can go through it.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace moa {

// Tokens per workgroup; `dense`: their rows one behind another in 160; `wide_tiles` tiles of five tokens stand in front.
struct LsaFusedPlan { int tokens; bool dense; int64_t wide_tiles; };

// LDS of a workgroup with 128 or 160 rows: all that a compute unit has, to the last byte
constexpr size_t LSA_BIG_LDS = (size_t)160 * 512 * 2;

// layer counts of which two tokens' rows fit 160 where one token's need a third block of 32 (from packed weights)
inline bool lsa_dense_layers(int L) { return L > 64 && L <= 80; }

// Rows per workgroup.  Measured at the Llama-3-8B shape (d_in 2048), a workgroup takes about 31 + 9 (rows / 32)
// microseconds from plain weights and 10 + 11.7 (rows / 32) from packed ones (or, in proportion, a twelfth less: the clock of
// a full chip follows its power), whatever else runs (it is bound by
// its own chain of tile fetches from the L2 and its matrix work), and the chip runs 256 of them at a time: few
// tokens want small tiles (every compute unit busy), many tokens large ones (fewer passes over the weights).  Pick
// the tile that minimises rounds x time per round.  units: workgroups per tile of tokens; lds: what a workgroup may ask for.
inline LsaFusedPlan lsa_fused_plan(bool packed, int64_t T, int L, int d_in, int units, size_t lds)
{
    const int nb = (L + 31) / 32, units_per_xcd = (units + 7) / 8;
    const bool big_ok = lds >= LSA_BIG_LDS;
    const double fixed = packed ? 10.0 : 31.0, per_block = packed ? 11.7 * d_in / 2048 : 9.0;
    // One workgroup per compute unit, all equally long: whole rounds, of the XCD that has the most units (each has 32
    // compute units, and four units leave half of the XCDs idle).
    auto us = [&](int64_t tokens, int tt, double blocks) {
        return (double)(((tokens + tt - 1) / tt * units_per_xcd + 31) / 32) * (fixed + per_block * blocks);
    };
    if (nb == 1) {
        int best = 2;
        if (us(T, 3, 3) < us(T, best, best)) best = 3;
        if (big_ok && us(T, 4, 4) < us(T, best, best)) best = 4;
        LsaFusedPlan plan = {best, false, 0};
        // Packed: whole rounds of 160-row tiles and what is left in smaller ones.  A row costs as much in 160 as in 128 (69 us a
        // round against 55), so this is about rounds that are nearly empty, and has to promise 4 % since a
        // round with idle compute units also clocks higher (with the output projection, d_in 2048: 140 tokens 93 -> 78 us, 300
        // 175 -> 153, 400 229 -> 199, 960 478 -> 448; 1024, where it promises 2 %, 472 -> 478).
        const int64_t round = 32 / units_per_xcd;          // tiles of one unit in a round of an XCD's 32 compute units
        if (!packed || !big_ok || round == 0) return plan;
        double least = 0.96 * us(T, best, best);
        const int64_t full = T / (5 * round);
        for (int64_t w = full > 3 ? full - 3 : 0; w <= full; ++w)
            for (int tt = 2; tt <= 5; ++tt) {
                if (w == 0 && tt < 5) continue;
                const double t = (double)w * (fixed + per_block * 5) + us(T - 5 * round * w, tt, tt);
                if (t >= least) continue;
                least = t;
                plan = tt < 5 ? LsaFusedPlan{tt, false, round * w} : LsaFusedPlan{4, false, (T + 4) / 5};
            }
        return plan;
    }
    if (nb == 2) return {big_ok && us(T, 2, 4) < us(T, 1, 2) ? 2 : 1, false, 0};
    // two tokens in 160 rows take 66 us a round where one in 96 takes 48, as much as 3.4 blocks: as soon as that saves a round
    // (6 or 8 units: 78 tokens in two rounds 136 us with the output projection, in three 151)
    const bool dense = packed && big_ok && lsa_dense_layers(L) && us(T, 2, 5) < us(T, 1, 3.4);
    return {dense ? 2 : 1, dense, 0};
}

}  // namespace moa
