// Projections Y = X W^T of bf16 tensors on the matrix cores (MFMA 16x16x32), for any number of rows: one kernel,
// instantiated for the tiles that the path's row counts and widths ask for, and the rule that picks one.
//
// A workgroup owns a tile of rows x features and, as a rule, all of K: no partial sums, no second launch.  It walks K in
// tiles of 64; both operands come from global memory straight into LDS (128-byte row pieces, no registers, no LDS store
// instructions) through rings of several stages, so that loads of the next SX - 1 and SW - 1 k tiles are in flight
// behind the current one.  One barrier per k tile: it stands three quarters into the tile's MFMAs, when the last operands
// of the tile have been read, so that the first operands of the next one arrive behind the last quarter.  With WK > 1 the
// wavefronts form groups that take every WK-th k tile each, with rings of their own, and add up through LDS at the end:
// for few rows, where one group's chain of barrier, operand read and MFMA is longer than the memory needs.
//
// The matrix instruction is 16x16x32: the bits of two 32x32x16 ones chained along K from the same operand bytes, at 2.03 PFLOP/s
// from registers where the power budget leaves the larger one 1.78 (2048 x 4096 x 28672: 434 -> 421 us, 1024 x 14336 x 4096 140 ->
// 132), and a tile may have 16 rows: up to 16 rows a workgroup then brings half as many of the activations past its weights
// (8 x 4096 x 4096: 10.6 -> 8.8 us, 8 x 8192 x 8192 29.2 -> 28.0).
//
// What bounds it: for few rows the weights (60 x 4096 x 8192: 17.9 us = 3.7 TB/s and no summing pass, where K slices with
// fp32 partial sums took 21.0 + 4.0; 8 x 4096 x 128256: 162 us = 6.5 TB/s against 196 + 5), for many the way from L2 to
// LDS, which one compute unit fills at 50 - 60 GB/s here (loads alone 61 us, MFMAs alone 58, both 79 at 1024 x 4096 x
// 10240, where 128 x 128 tiles with everything waited for at each barrier took 135; 19200 x 2048 x 4096: 302 against 388).
#include "moa_common.h"
#include "moa_gemm_device.h"
#include "moa_tree_device.h"

#include <math.h>

namespace moa {

template <int WR, int WF, int MR, int NF, int SX, int SW, int WK, int SEGS>
__global__ __launch_bounds__(64 * WR * WF * WK) void k_linear_bf16(LinDev<SEGS> a)
{
    using Loop = GemmLoop<WR, WF, MR, NF, SX, SW, WK>;
    constexpr int BM = Loop::BM, BN = Loop::BN;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < a.lead_blocks) {
        if ((int)blockIdx.x < a.rider_units && tid < 64)
            step_small_unit(a.rider, (int)blockIdx.x, (int32_t *)smem, (int32_t *)smem + MOA_MAX_TREE);
        return;
    }
    // Workgroups are dealt to the 8 XCDs round-robin, and each XCD has its own L2: an XCD gets a contiguous group of
    // feature tiles for all row tiles, so that its slice of W is fetched into its L2 once.
    const int bx = (int)blockIdx.x - a.lead_blocks, xcd = bx & 7, j = bx >> 3;
    const int ftile = xcd * a.tiles_per_xcd + j % a.tiles_per_xcd;
    if (ftile >= a.tile_begin[SEGS]) return;
    const int rest = j / a.tiles_per_xcd, rt = rest % a.row_tiles, split = rest / a.row_tiles;
    const int s = a.segment(ftile);
    const int n0 = (ftile - a.tile_begin[s]) * (a.gated ? BN / 2 : BN), N = a.seg[s].N, K = a.K;
    const int64_t r0 = (int64_t)rt * BM;
    const int64_t ldx = a.seg[s].ldx;
    const int nk = K / (Loop::BK * WK * a.splits);
    Loop g;
    g.set_x((const char *)a.seg[s].X + r0 * ldx * 2, ldx, a.R - r0);
    const char *const w0 = (const char *)a.seg[s].W + (int64_t)n0 * K * 2, *const w1 = a.gated ? (const char *)a.seg[1].W + (int64_t)n0 * K * 2 : w0;
    g.set_w(K, N - n0, [&](int blk, int *first) {
        *first = 32 * (a.gated ? blk >> 1 : blk);
        return blk & 1 ? w1 : w0;
    });
    if (!g.run(smem, split * nk, nk)) return;
    const StoreSpec st = a.store(s);
    const int l16 = g.lane & 15, quart = g.lane >> 4, wfi = g.wave % WF;
    auto store8 = [](bf16_t *d, const float (&v)[8]) {
        u32x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
        *(u32x4 *)d = pk;
    };

    // values(i, v): features 32 i + 8 quart .. of the wavefront's, row 16 j + l16
#pragma unroll
    for (int j = 0; j < MR; ++j) {
        const int64_t r = r0 + g.wave_row() + 16 * j + l16;
        if (r >= a.R) continue;
        auto values = [&](int i, float (&v)[8]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = g.acc[i][j][e >> 2][e & 3];
        };
        if (a.splits > 1) {
            float *p = a.part + (((r >> 6) * a.splits + split) * 64 + (r & 63)) * a.ntot;
            int col = 0;
            for (int q = 0; q < s; ++q) col += a.seg[q].N;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int n = n0 + wfi * (32 * NF) + 32 * i + 8 * quart;
                if (n >= N) continue;
#pragma unroll
                for (int q = 0; q < 2; ++q) *(f32x4 *)(p + col + n + 4 * q) = g.acc[i][j][q];
            }
            continue;
        }
        if (NF % 2 == 0 && a.gated) {             // silu(gate) * up, both through the storage type first
#pragma unroll
            for (int i = 0; i + 1 < NF; i += 2) {
                const int n = n0 + wfi * (16 * NF) + 16 * i + 8 * quart;
                if (n >= N) continue;
                float v[8], u[8];
                values(i, v);
                values(i + (NF > 1), u);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float t = bf2f(f2bf(v[e]));
                    v[e] = t / (1.0f + __expf(-t)) * bf2f(f2bf(u[e]));
                }
                store8((bf16_t *)a.epi_out + r * N + n, v);
            }
            continue;
        }
        const int64_t rp = store_row_part(st, r);
        if (rp < 0) continue;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int n = n0 + wfi * (32 * NF) + 32 * i + 8 * quart;
            if (n >= N) continue;
            float v[8];
            values(i, v);
            if (a.epi == LinArgs::EPI_ADD_F32) {
                const float *h = a.epi_res + r * N + n;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = h[e] + bf2f(f2bf(v[e]));
                store8((bf16_t *)a.epi_out + r * N + n, v);
            } else {                               // eight features never straddle a head
                store8((bf16_t *)st.dst + rp + store_feat_part(st, n), v);
            }
        }
    }
}

// The instantiated tiles: wavefronts along rows and features, blocks of 16 rows and of 32 features per wavefront, stages
// of the activation and the weight ring, K groups; then microseconds per k tile of the workgroup's (64 WK columns) with
// one workgroup on a compute unit, with a second one on up to half of them, and with two on all (0: its LDS holds one),
// measured over 1 .. 4096 rows, K 2048 .. 14336 and 4096 .. 128256 features.  The 16-row tiles 14, 15, 16 are 0, 1, 2 in every
// number but the rows, and have those tiles' times: up to 32 rows the K groups are then the same, and without slices of K a row's
// sums do not depend on how many rows are beside it.
#define MOA_GEMM_TILES(T)                           \
    T(0, 2, 1, 1, 1, 5, 5, 2, 0.25f, 0.34f, 0.34f)  \
    T(1, 1, 1, 2, 1, 2, 3, 4, 0.55f, 0.66f, 0.66f)  \
    T(2, 2, 1, 1, 2, 3, 3, 2, 0.45f, 0.74f, 0.74f)  \
    T(3, 2, 1, 2, 1, 3, 4, 2, 0.44f, 0.75f, 0.75f)  \
    T(4, 2, 2, 2, 1, 4, 6, 1, 0.27f, 0.33f, 0.46f)  \
    T(5, 2, 2, 2, 2, 3, 3, 2, 0.88f, 0.f, 0.f)      \
    T(6, 4, 2, 2, 2, 4, 4, 1, 0.57f, 0.f, 0.f)      \
    T(7, 4, 1, 2, 5, 4, 4, 1, 0.72f, 0.f, 0.f)      \
    T(8, 4, 2, 4, 2, 3, 4, 1, 0.90f, 0.f, 0.f)      \
    T(9, 8, 1, 2, 5, 3, 3, 1, 1.12f, 0.f, 0.f)      \
    T(10, 4, 2, 4, 4, 2, 2, 1, 1.55f, 0.f, 0.f)     \
    T(11, 4, 2, 2, 1, 3, 4, 2, 0.82f, 0.f, 0.f)     \
    T(12, 4, 2, 4, 3, 2, 3, 1, 1.25f, 0.f, 0.f)     \
    T(13, 2, 2, 2, 1, 4, 5, 2, 0.66f, 0.f, 0.f)     \
    T(14, 1, 1, 1, 1, 5, 5, 2, 0.25f, 0.34f, 0.34f) \
    T(15, 1, 1, 1, 1, 2, 3, 4, 0.55f, 0.66f, 0.66f) \
    T(16, 1, 1, 1, 2, 3, 3, 2, 0.45f, 0.74f, 0.74f)

struct GemmTile {
    int bm, bn, threads, wk;
    size_t lds;
    bool gated;          // pairs of feature blocks in one wavefront: can apply a gated activation
    float us1, us_mid, us2;
};
#define MOA_GEMM_INFO(id, WR, WF, MR, NF, SX, SW, WK, US1, USM, US2)                                                            \
    {16 * MR * WR, 32 * NF * WF, 64 * WR * WF * WK, WK, (size_t)(SX * 16 * MR * WR + SW * 32 * NF * WF) * 128 * WK, NF % 2 == 0, US1, USM, US2},
static const GemmTile kTiles[] = {MOA_GEMM_TILES(MOA_GEMM_INFO)};

struct GemmPlan { int tile, splits; };

// The tile, and into how many slices K is cut, by an estimate of the time: rounds of workgroups over 256 compute units at
// the measured time per k tile, or the weights at 5.8 TB/s, whichever is longer; slices cost a pass over their sums.  An XCD
// gets whole feature tiles, so a round is full when its share of them fills its 32 compute units (1600 x 8192 x 9216 in
// 256 x 256: 252 workgroups, 35 of them on seven XCDs each, 355 us against 232 in 256 x 128).  Against the best tile and slices
// of each of 689 measured calls (33 shapes, 1 .. 4096 rows, weights from memory) the choice is 1.7 % slower on average, 0.7 % above 192
// rows, 4.9 % at 17 to 32 and 29 % at worst (180 x 10240 x 8192); the times of the 64-row tiles and larger were measured with
// 32x32x16 instructions, those of the others are kept for their order of sums.  What it comes to: up to 16
// rows the 16-row tiles, up to 32 the 32-row ones; up to some hundred the 64-row ones; with more, the largest tile that still gives every compute
// unit one (1024 x 4096: 256 x 160 for 10240 features, 77.6 us against 98 - 108 with the tiles next to it, 256 x 128 for
// 8192); slices only for a long K with few features (60 x 14336 x 4096: four, 30 us against 52).  A pass of its own behind
// an unsplit projection counts against not splitting, since the sum over slices does that work on the way.
//
// same_sums: pairs of K groups or one chain, no slices, whatever the features (see LinArgs).
static GemmPlan plan_gemm(int64_t R, int K, const int *n_seg, int nseg, int epi, bool in_order, int same_sums, int most_splits = 8)
{
    if (same_sums && R > LinArgs::pair_rows(same_sums, K)) in_order = true;
    GemmPlan best = {0, 1};
    int ntot = 0;
    for (int s = 0; s < nseg; ++s) {
        ntot += n_seg[s];
        if (n_seg[s] % 64) most_splits = 1;        // the pass over the sums takes features in 64s
    }
    if (nseg > LIN_FEW) most_splits = 1;           // and four matrices
    if (in_order || same_sums || R > 192) most_splits = 1;
    else if (R > 64 && most_splits > 4) most_splits = 4;       // eight pay off where the sums are few (64 x 4096 x 1024: 9.7 against 10.5 us)
    float best_us = 3.4e38f;
    const float stream_us = 6.f + 2.f * (float)K * (float)ntot / 5.8e6f;
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const GemmTile &t = kTiles[i];
        if (in_order ? t.wk > 1 : ((R <= 16 ? t.bm != 16 : R <= 32 ? t.bm != 32 : t.bm < 64) || K % (64 * t.wk) != 0 || (same_sums && t.wk != 2) || (nseg > LIN_FEW && t.wk > 2))) continue;
        const int64_t row_tiles = (R + t.bm - 1) / t.bm;
        int64_t tiles = 0;
        for (int s = 0; s < nseg; ++s) tiles += (n_seg[s] + t.bn - 1) / t.bn;
        tiles = (tiles + 7) / 8 * 8 * row_tiles;
        // two 64 x 64 workgroups of one row tile share nothing, and take as long as one after the other (60 x 8192 x 18432:
        // 0.63 us per k tile where two row tiles of the same weights take 0.38)
        const bool apart = t.bm == 64 && t.bn == 64 && row_tiles == 1;
        const float us_mid = apart ? 0.60f : t.us_mid, us2 = apart ? 0.65f : t.us2;
        for (int splits = 1; splits <= most_splits; splits *= 2) {
            if (splits > 1 && (K % (64 * t.wk * splits) || K / (64 * t.wk * splits) < 4)) break;
            const int64_t n = tiles * splits;
            float per;                             // k-tile times of one compute unit
            if (t.us2 > 0.f) {
                const int64_t rest = n % 512;
                per = (float)(n / 512) * us2;
                if (rest) per += rest <= 256 ? t.us1 : rest <= 384 ? us_mid : us2;
            } else {
                per = (float)((n + 255) / 256) * t.us1;
            }
            const float busy_us = 5.f + per * (float)(K / (64 * t.wk * splits));
            float us = busy_us > stream_us ? busy_us + 0.1f * stream_us : stream_us + 0.1f * busy_us;
            if (splits > 1) us += (epi == LinArgs::EPI_ROPE ? 8.f : 5.f) + (float)R * (float)ntot * (float)splits * 8.f / 3.5e6f;
            else if (epi == LinArgs::EPI_ROPE || epi == LinArgs::EPI_ADD_NORM || (epi == LinArgs::EPI_SWIGLU && !t.gated)) us += 5.f;
            if (us < best_us) {
                best_us = us;
                best = {i, splits};
            }
        }
    }
    return best;
}

static size_t partial_bytes(int64_t R, int ntot, int splits)
{
    return splits > 1 ? (size_t)((R + 63) / 64) * splits * 64 * (size_t)ntot * sizeof(float) : 0;
}

size_t linear_workspace_bytes(int dtype, int64_t R, int K, std::initializer_list<int> n_seg, bool upto)
{
    if (dtype != DT_BF16 || R < 1 || K % 128) return 0;
    int ntot = 0;
    for (int n : n_seg) ntot += n;
    size_t most = 0;
    auto ask = [&](int64_t r) {
        if (r > 192 || r > R) return;
        // (of all epilogues EPI_ADD_NORM counts most against not splitting, and none changes which split is the best one)
        const size_t n = partial_bytes(r, ntot, plan_gemm(r, K, n_seg.begin(), (int)n_seg.size(), LinArgs::EPI_ADD_NORM, false, 0).splits);
        if (n > most) most = n;
    };
    ask(R);
    // Between the row counts where some tile needs one more of itself, all that grows with the rows is the price of a
    // slice, so the fewest rows are cut into the most slices, and all have as many 64-row tiles of sums (those of 129 rows
    // or more: three).
    if (upto)
        for (int64_t r : {1, 33, 65, 129}) ask(r);
    return most;
}

template <int SEGS>
static hipError_t launch_tile(const LinArgs &a, const GemmPlan &p, hipStream_t stream, bool *fused, int *splits)
{
    const GemmTile &t = kTiles[p.tile];
    LinDev<SEGS> ga(a);
    ga.splits = *splits = p.splits;
    ga.part = (float *)a.ws;
    ga.gated = a.epi == LinArgs::EPI_SWIGLU && t.gated && p.splits == 1;
    *fused = ga.gated || (a.epi == LinArgs::EPI_ADD_F32 && p.splits == 1);
    int ft = 0;
    for (int s = 0; s < a.nseg; ++s) {
        ga.tile_begin[s] = ft;
        if (!ga.gated) ft += (a.seg[s].N + t.bn - 1) / t.bn;
        else if (s == 0) ft = (2 * a.seg[0].N + t.bn - 1) / t.bn;
    }
    for (int s = a.nseg; s <= SEGS; ++s) ga.tile_begin[s] = ft;
    ga.tiles_per_xcd = (ft + 7) / 8;
    ga.row_tiles = (int)((a.R + t.bm - 1) / t.bm);
    ga.lead_blocks = (a.rider_units + 7) & ~7;      // a multiple of the XCD count: the tile mapping keeps its phase
    const int64_t blocks = ga.lead_blocks + (int64_t)8 * ga.tiles_per_xcd * ga.row_tiles * ga.splits;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    static bool raised[sizeof(kTiles) / sizeof(kTiles[0])][16] = {};
    switch (p.tile) {
#define MOA_GEMM_LAUNCH(id, WR, WF, MR, NF, SX, SW, WK, US1, USM, US2)                                                               \
    case id:                                                                                                                             \
        if constexpr (SEGS == LIN_FEW || WK <= 2) {                                                                                      \
            e = raise_lds_limit_once(raised[id], (const void *)k_linear_bf16<WR, WF, MR, NF, SX, SW, WK, SEGS>, t.lds);                  \
            if (e != hipSuccess) return e;                                                                                               \
            prof_begin(K_LIN_BF16 + 64 * (id + 1), stream);                                                                              \
            MOA_KLAUNCH((k_linear_bf16<WR, WF, MR, NF, SX, SW, WK, SEGS>), dim3((unsigned)blocks), dim3(t.threads), t.lds, stream, ga);  \
        } else {                                                                                                                         \
            return hipErrorInvalidValue;         /* the plan gives more than LIN_FEW matrices no such tile */                            \
        }                                                                                                                                \
        break;
        MOA_GEMM_TILES(MOA_GEMM_LAUNCH)
    }
    prof_end(stream);
    return hipGetLastError();
}

static GemmPlan plan_of(const LinArgs &a)
{
    int ntot = 0, n_seg[LIN_SEGS] = {};
    for (int s = 0; s < a.nseg; ++s) {
        n_seg[s] = a.seg[s].N;
        ntot += a.seg[s].N;
    }
    GemmPlan p = plan_gemm(a.R, a.K, n_seg, a.nseg, a.epi, a.in_order, a.same_sums);
    // without room for the sums of slices another tile may be the best one (64 x 14336 x 4096: 52 us in 64 x 32 against
    // 71 in the 64 x 64 of four slices)
    if (p.splits > 1 && !(a.ws && a.ws_bytes >= partial_bytes(a.R, ntot, p.splits) && (((uintptr_t)a.ws) & 15) == 0))
        p = plan_gemm(a.R, a.K, n_seg, a.nseg, a.epi, a.in_order, a.same_sums, 1);
    return p;
}

int linear_bf16_order(const LinArgs &a)
{
    const GemmPlan p = plan_of(a);
    return kTiles[p.tile].wk * 16 + p.splits;
}

// One launch.  *fused: it applied a.epi; *splits > 1: the sums of that many K slices are in a.ws, to be added up.
hipError_t launch_linear_bf16(const LinArgs &a, hipStream_t stream, bool *fused, int *splits)
{
    const GemmPlan p = plan_of(a);
    return a.nseg <= LIN_FEW ? launch_tile<LIN_FEW>(a, p, stream, fused, splits) : launch_tile<LIN_SEGS>(a, p, stream, fused, splits);
}

// the kernel's name as a profiler prints it, without SEGS
const char *linear_bf16_name(int variant)
{
    static const char *const names[] = {
#define MOA_GEMM_NAME(id, WR, WF, MR, NF, SX, SW, WK, US1, USM, US2) "k_linear_bf16<" #WR ", " #WF ", " #MR ", " #NF ", " #SX ", " #SW ", " #WK ">",
        MOA_GEMM_TILES(MOA_GEMM_NAME)};
    return variant >= 1 && variant <= (int)(sizeof(names) / sizeof(names[0])) ? names[variant - 1] : "k_linear_bf16";
}

}  // namespace moa
