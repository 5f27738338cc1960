// Which kernels the attention cores of a launch take and what scratch they need.  Host arithmetic only, so that a test on a
// machine without a GPU can go through it.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/moa.h"

namespace moa {

constexpr int KT = 32;        // keys per tile of the kernels with 128-row tiles and over the whole key range
constexpr int LK = 64;        // of the one with 256-row tiles

// 32-row blocks per wave of the split-KV kernel: one block per wave keeps two workgroups per CU, which measured
// 25 % faster than two blocks per wave at RG = 512 even though K/V are then read by twice as many row tiles
constexpr int ATTN_NBLK = 1;

struct SplitGeom {
    int nsplit;     // key-range slices
    int rowtiles;   // workgroups along the G*Mq rows of one (sequence, KV head)
    int rows_pad;   // rowtiles * rows per workgroup
    bool wide;      // 256 rows per workgroup (k_attn_long) instead of 128
};

// ncalls: 1, or 2 of this shape in one launch (the number of key slices of either form does not depend on it)
inline SplitGeom split_geometry(int form, int B, int Mq, int H, int Hkv, int dh, int P_cap, int ncalls)
{
    const int RG = (H / Hkv) * Mq;
    const int rows = 128 * ATTN_NBLK, tiles_cap = (P_cap + KT - 1) / KT;
    SplitGeom g;
    g.rowtiles = (RG + rows - 1) / rows;
    g.rows_pad = g.rowtiles * rows;
    int want = 512 / (B * Hkv * g.rowtiles);        // about two workgroups per compute unit
    int most = tiles_cap / 2;                        // at least two tiles per slice
    if (want > most) want = most;
    if (want > 64) want = 64;
    if (want < 1) want = 1;
    g.nsplit = want;
    g.wide = false;
    if (dh != 128 || RG <= 128) return g;
    // 256-row tiles, one workgroup per compute unit; never more scratch than the 128-row tiles' slices would take
    SplitGeom w;
    w.wide = true;
    w.rowtiles = (RG + 255) / 256;
    w.rows_pad = w.rowtiles * 256;
    want = 256 / (B * Hkv * w.rowtiles);
    most = ((P_cap + LK - 1) / LK) / 2;
    if (want > most) want = most;
    if (want > 64) want = 64;
    while (want > 1 && (int64_t)want * w.rows_pad > (int64_t)g.nsplit * g.rows_pad) --want;
    if (want < 1) want = 1;
    w.nsplit = want;
    // Which one, by an estimate in microseconds.  A round of 128-row workgroups takes 1.5 per tile of 32 keys with two per
    // compute unit and 1.2 with one; one of 256-row workgroups 1.05, 0.15 for each time its accumulators follow a new maximum
    // (nearly always on the first 32 tiles of a slice, then ever more rarely), and 4 more in front and behind.  It
    // decides where the rows fill their last tile badly (8 sequences x 32768 keys x 8 KV heads: 260 .. 384 rows in three tiles
    // of 128 against two of 256, which leave half of the chip idle), where the rows of an XCD's units need one workgroup
    // more than it has compute units, and where a slice is a few tiles.  Two calls in one launch can fill what one leaves idle.
    // Over 456 measured calls (512 .. 32768 keys, 1 .. 16 sequences, 132 .. 1024 rows) it is 0.5 % behind the better form.
    const int64_t units = (int64_t)ncalls * B * Hkv;
    const int64_t per128 = (tiles_cap + g.nsplit - 1) / g.nsplit, wgs128 = units * g.nsplit * g.rowtiles;
    const int64_t per256 = (tiles_cap + w.nsplit - 1) / w.nsplit, rounds256 = ((units * w.nsplit + 7) / 8 * 8 * w.rowtiles + 255) / 256;
    const int64_t rest = wgs128 % 512;
    const float us128 = (float)per128 * (1.5f * (float)(wgs128 / 512) + (rest == 0 ? 0.f : rest <= 256 ? 1.2f : 1.5f));
    const float tiles = (float)per256, follows = tiles <= 32.f ? tiles : 32.f + 32.f * logf(tiles / 32.f);
    const bool wide = form == MOA_ATTN_KERNEL_SPLIT_WIDE || 4.f + (float)rounds256 * (1.05f * tiles + 0.15f * follows) < us128;
    return wide ? w : g;
}

// scratch of one of `ncalls` calls in a launch
inline size_t split_bytes(const SplitGeom &g, int B, int Hkv, int dh)
{
    const size_t rows = g.nsplit > 1 || !g.wide ? (size_t)B * Hkv * g.nsplit * g.rows_pad : 0;
    return rows * ((size_t)dh * 2 + 2 * sizeof(float)) + 256;
}

// scratch with which a call may take the split form, alone or as one of two
inline size_t split_room(int form, int B, int Mq, int H, int Hkv, int dh, int P_cap)
{
    size_t bytes = 0;
    for (int ncalls : {1, 2}) bytes = std::max(bytes, split_bytes(split_geometry(form, B, Mq, H, Hkv, dh, P_cap, ncalls), B, Hkv, dh));
    return bytes;
}

// Which MFMA kernel.  The whole-key-range form needs one launch, writes no partial results and has the shorter
// fixed part, but re-reads K/V once per 32 query rows and runs one workgroup per CU: it wins while the call is
// latency-bound, i.e. while its workgroups fit the chip in one round and the key range is short (C1: 14.5 us
// against 17.8 + 6.8 us).  With more work the split form (128 rows per workgroup and two workgroups per CU, or 256
// rows and one, see split_geometry; then the merge) is ahead (B = 16, prefixes up to 2048: 122 against 166 us).  moa_debug_force_attn_kernel overrides the
// choice (the parity tests run every case through both forms).
constexpr int FUSED_MAX_KEYS = 8192;
constexpr int FUSED_MAX_WORKGROUPS = 256;
inline bool want_whole(int form, int B, int Mq, int Mt, int H, int Hkv, int P_cap)
{
    if (form == MOA_ATTN_KERNEL_SPLIT || form == MOA_ATTN_KERNEL_SPLIT_WIDE) return false;
    if (form == MOA_ATTN_KERNEL_WHOLE) return true;
    const int64_t wgs = (int64_t)B * Hkv * (((H / Hkv) * Mq + 31) / 32);
    return P_cap + Mt <= FUSED_MAX_KEYS && wgs <= FUSED_MAX_WORKGROUPS;
}

// One of several cores of the same shape (B, Mq, H, Hkv, dh): `mfma`, its operands are what the bf16 matrix kernels read;
// `room`, its scratch in bytes (0: none, or not aligned).
struct AttnCore { int P_cap, Mt; bool mfma; size_t room; };
// other: none of the bf16 matrix kernels
struct AttnChoice {
    enum { WHOLE, SPLIT, OTHER } kind;
    SplitGeom geo;
    bool shares_with(const AttnChoice &o) const
    {
        return kind == o.kind && (kind != SPLIT || (geo.nsplit == o.geo.nsplit && geo.rows_pad == o.geo.rows_pad && geo.wide == o.geo.wide));
    }
};

// What each of n cores that may share launches takes; those with the same choice can share one.  A core takes what it would
// take alone, so that its result does not depend on who else there is room for in a launch -- but `pair`: the first two, a step's
// cross-attention and first verification layer, have row tiles as two calls take them, at the larger P_cap.  (Tiles by the number
// of calls that are in the launch gain nothing that shows: a step of 32768 keys x 100 nodes x 4 layers 585 - 589 us so, 588 - 592 this
// way, 8 x 2048 x 60 x 4 443 - 444 and 445 - 448.)
// A geometry is one that the core's own scratch holds: geometries at a smaller P_cap can need more than at a larger one (4
// sequences x 1408 rows: 135 KB more at 8065 keys than at 8192), so scratch is compared at the P_cap that the geometry is for.
inline void choose_attn(int form, int B, int Mq, int H, int Hkv, int dh, const AttnCore *core, int n, bool pair, AttnChoice *out)
{
    auto split = [&](int i, int cap, int ncalls) {
        if (core[i].room < split_room(form, B, Mq, H, Hkv, dh, cap)) return false;
        out[i].geo = split_geometry(form, B, Mq, H, Hkv, dh, cap, ncalls);
        return true;
    };
    for (int i = 0; i < n; ++i)
        out[i].kind = !core[i].mfma ? AttnChoice::OTHER : want_whole(form, B, Mq, core[i].Mt, H, Hkv, core[i].P_cap) ? AttnChoice::WHOLE : AttnChoice::SPLIT;
    int i = 0;
    if (pair && n > 1 && out[0].kind == AttnChoice::SPLIT && out[1].kind == AttnChoice::SPLIT) {
        const int cap = std::max(core[0].P_cap, core[1].P_cap);
        if (split(0, cap, 2) && split(1, cap, 2)) i = 2;
    }
    for (; i < n; ++i)
        if (out[i].kind == AttnChoice::SPLIT && !split(i, core[i].P_cap, 1)) out[i].kind = AttnChoice::OTHER;
}

}  // namespace moa
