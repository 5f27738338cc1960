// Projections Y = X W^T whose products are formed in single precision: fp32 tensors, and bf16 ones that the bf16 matrix
// kernels do not take (a K or a feature count outside their tiles).  Both kernels run on the fp32 matrix instructions
// (v_mfma_f32_*: fp32 products, fp32 sums), read their operands with vector loads, take several weight matrices per
// launch, each with its own activations if it has any, and carry the step's integer work in workgroups of their own at
// the front of the grid.
//
//   k_linear_f32_latency  few output tiles: 16 features x 16 rows per workgroup, the four wavefronts split K and add up
//                         through LDS.  Bound by one memory round trip: at K = 256 every load of a wavefront is in
//                         flight before the first one is used.
//   k_linear_f32_tile     many: 64 x 64 tiles through LDS, 32 x 32 per wavefront.  Bound by the matrix pipe (256 flop per
//                         clock and compute unit).
//
// What they replaced was one 64 x 64 kernel of scalar loads and vector-unit FMAs with two barriers per 16 columns of K,
// one launch per weight matrix: 31 us for any projection of the tiny instance (8 rows, K = 256), twelve of them per step.
#include "moa_common.h"
#include "moa_tree_device.h"

namespace moa {

__device__ __forceinline__ f32x4 ld4(const float *p) { return *(const f32x4 *)p; }
__device__ __forceinline__ f32x4 ld4(const bf16_t *p)
{
    const u32x2 v = *(const u32x2 *)p;
    return f32x4{__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xffff0000u), __uint_as_float(v[1] << 16),
                 __uint_as_float(v[1] & 0xffff0000u)};
}
__device__ __forceinline__ void st4(float *p, const f32x4 &v) { *(f32x4 *)p = v; }
__device__ __forceinline__ void st4(bf16_t *p, const f32x4 &v)
{
    u32x2 o;
    o[0] = pack_bf16x2(v[0], v[1]);
    o[1] = pack_bf16x2(v[2], v[3]);
    *(u32x2 *)p = o;
}

// the integer work in the first workgroups of the grid; true when this workgroup was one of them
template <int SEGS>
__device__ __forceinline__ bool f32_lead_block(const LinDev<SEGS> &a, int32_t *lds)
{
    if ((int)blockIdx.x >= a.lead_blocks) return false;
    if ((int)blockIdx.x < a.rider_units && threadIdx.x < 64)
        step_small_unit(a.rider, (int)blockIdx.x, lds, lds + MOA_MAX_TREE);
    return true;
}

template <typename T, int SEGS>
__global__ __launch_bounds__(256) void k_linear_f32_latency(LinDev<SEGS> a)
{
    constexpr int UN = 4;                         // 16-column steps of K a wavefront has in flight
    __shared__ float red[4][16][20];              // 20: rows of four-float stores land on different banks
    if (f32_lead_block(a, (int32_t *)red)) return;
    const int ntiles = a.tile_begin[SEGS];
    const int bx = (int)blockIdx.x - a.lead_blocks, tile = bx % ntiles;
    const int64_t r0 = (int64_t)(bx / ntiles) * 16;
    const int s = a.segment(tile);
    const int N = a.seg[s].N, K = a.K, n0 = (tile - a.tile_begin[s]) * 16;
    const T *X = (const T *)a.seg[s].X;
    const int64_t ldx = a.seg[s].ldx;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, kg = lane >> 4;

    // operands of v_mfma_f32_16x16x4: lane (li, kg) loads k = 16 step + 4 kg .. + 3 of its row in one piece, and MFMA j
    // of a step takes element j of both pieces -- a permutation of K that both operands share
    const int64_t r = r0 + li < a.R ? r0 + li : a.R - 1;      // rows and features past the end repeat the last one
    const int n = n0 + li < N ? n0 + li : N - 1;
    const T *xp = X + r * ldx, *wp = (const T *)a.seg[s].W + (int64_t)n * K;
    const int steps = (K + 15) >> 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    f32x4 wf[2][UN], xf[2][UN];
    auto load = [&](int set, int first) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = 16 * (first + 4 * u) + 4 * kg;
            const int kc = k < K ? k : 0;         // K is a multiple of four: a piece is inside or outside as a whole
            wf[set][u] = ld4(wp + kc);
            xf[set][u] = ld4(xp + kc);
            if (k >= K) wf[set][u] = xf[set][u] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[set][u][j], xf[set][u][j], acc, 0, 0, 0);
    };
    load(0, wave);
    for (int st0 = wave; st0 < steps; st0 += 8 * UN) {        // wavefront w takes steps w, w + 4, ...; two batches a trip
        if (st0 + 4 * UN < steps) load(1, st0 + 4 * UN);
        multiply(0);
        if (st0 + 4 * UN >= steps) break;
        if (st0 + 8 * UN < steps) load(0, st0 + 8 * UN);
        multiply(1);
    }
    // lane holds features 4 kg .. 4 kg + 3 of row li
    *(f32x4 *)&red[wave][li][4 * kg] = acc;
    __syncthreads();
    const int row = threadIdx.x >> 4, f = threadIdx.x & 15;
    if (r0 + row >= a.R || n0 + f >= N) return;
    const float v = (red[0][row][f] + red[1][row][f]) + (red[2][row][f] + red[3][row][f]);
    const StoreSpec sp = a.store(s);
    const int64_t off = store_offset(sp, r0 + row, n0 + f);
    if (off >= 0) st<T>((T *)sp.dst + off, v);
}

template <typename T, int SEGS>
__global__ __launch_bounds__(256) void k_linear_f32_tile(LinDev<SEGS> a)
{
    constexpr int BK = 32, LD = BK + 4;           // 36-float rows: the 32 rows of an operand read hit 64 different banks
    __shared__ __attribute__((aligned(16))) float Ws[2][64 * LD];
    __shared__ __attribute__((aligned(16))) float Xs[2][64 * LD];
    if (f32_lead_block(a, (int32_t *)Ws)) return;
    const int ntiles = a.tile_begin[SEGS];
    const int bx = (int)blockIdx.x - a.lead_blocks, tile = bx % ntiles;
    const int64_t r0 = (int64_t)(bx / ntiles) * 64;
    const int s = a.segment(tile);
    const int N = a.seg[s].N, K = a.K, n0 = (tile - a.tile_begin[s]) * 64;
    const T *X = (const T *)a.seg[s].X;
    const int64_t ldx = a.seg[s].ldx;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wf0 = (wave & 1) * 32, wr0 = (wave >> 1) * 32;

    // thread t moves columns 4 (t & 7) .. + 3 of tile rows t / 8 and t / 8 + 32: eight lanes cover a row's 128 bytes
    const int lrow = tid >> 3, lcol = 4 * (tid & 7);
    const T *wp[2], *xp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = n0 + lrow + 32 * i;
        const int64_t r = r0 + lrow + 32 * i;
        wp[i] = (const T *)a.seg[s].W + (int64_t)(n < N ? n : N - 1) * K;
        xp[i] = X + (r < a.R ? r : a.R - 1) * ldx;
    }
    f32x4 wr[2], xr[2];
    auto fetch = [&](int k0) {
        const int k = k0 + lcol, kc = k < K ? k : 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            wr[i] = ld4(wp[i] + kc);
            xr[i] = ld4(xp[i] + kc);
            if (k >= K) wr[i] = xr[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *(f32x4 *)&Ws[buf][(lrow + 32 * i) * LD + lcol] = wr[i];
            *(f32x4 *)&Xs[buf][(lrow + 32 * i) * LD + lcol] = xr[i];
        }
    };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const int nk = (K + BK - 1) / BK;
    fetch(0);
    stage(0);
    if (nk > 1) fetch(BK);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
#pragma unroll
        for (int ks = 0; ks < BK / 8; ++ks) {
            const f32x4 wv = *(const f32x4 *)&Ws[buf][(wf0 + l32) * LD + 8 * ks + 4 * half];
            const f32x4 xv = *(const f32x4 *)&Xs[buf][(wr0 + l32) * LD + 8 * ks + 4 * half];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[j], xv[j], acc, 0, 0, 0);
        }
        if (kt + 1 < nk) stage(buf ^ 1);          // read last at tile kt - 1, a barrier ago
        if (kt + 2 < nk) fetch((kt + 2) * BK);
        __syncthreads();
    }
    // acc[v]: feature wf0 + 8 (v / 4) + 4 half + v % 4 of row wr0 + l32
    const int64_t r = r0 + wr0 + l32;
    if (r >= a.R) return;
    const StoreSpec sp = a.store(s);
    const int64_t rp = store_row_part(sp, r);
    if (rp < 0) return;
    T *dst = (T *)sp.dst;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = n0 + wf0 + 8 * q + 4 * half;
        if ((a.vec >> s & 1) && n + 4 <= N) {
            st4(dst + rp + store_feat_part(sp, n), f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]});
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) st<T>(dst + rp + store_feat_part(sp, n + e), acc[4 * q + e]);
        }
    }
}

static bool aligned_to(const void *p, size_t bytes) { return (((uintptr_t)p) & (bytes - 1)) == 0; }

// operands that vector loads of four elements can read
bool linear_f32_ok(int dtype, const LinArgs &a)
{
    const size_t piece = dtype == DT_BF16 ? 8 : 16;
    if (a.K % 4 || a.K < 4) return false;
    for (int s = 0; s < a.nseg; ++s) {
        const void *x = a.seg[s].X ? a.seg[s].X : a.X;
        const int64_t ldx = a.seg[s].X ? a.seg[s].ldx : a.ldx;
        if (ldx % 4 || !aligned_to(x, piece) || !aligned_to(a.seg[s].W, piece)) return false;
    }
    return true;
}

// 64 x 64 tiles once there are enough of them to keep the chip's matrix pipes busy; below that a workgroup's own chain
// of k tiles is what a launch costs, and 16 x 16 tiles spread it over sixteen times as many workgroups.  Launches that a
// step groups in one way or another (LinArgs::same_sums) count twice their widest segment: a layer's Q/K/V.
constexpr int64_t F32_TILE_MIN_WORKGROUPS = 128;

bool linear_f32_big(const LinArgs &a)
{
    int64_t t64 = 0, widest = 0;
    for (int s = 0; s < a.nseg; ++s) {
        const int64_t n = (a.seg[s].N + 63) / 64;
        t64 += n;
        if (n > widest) widest = n;
    }
    if (a.same_sums) t64 = 2 * widest;
    return t64 * ((a.R + 63) / 64) >= F32_TILE_MIN_WORKGROUPS;
}

template <int SEGS>
static hipError_t launch_f32_as(int dtype, const LinArgs &a, hipStream_t stream)
{
    LinDev<SEGS> fa(a);
    const size_t piece = dtype == DT_BF16 ? 8 : 16;
    for (int s = 0; s < a.nseg; ++s) {
        const StoreSpec &st = a.seg[s].st;
        fa.vec |= (uint32_t)(aligned_to(st.dst, piece) && (st.mode == StoreSpec::ROW ? st.ld % 4 == 0 : st.dh % 4 == 0)) << s;
    }
    const bool big = linear_f32_big(a);
    const int edge = big ? 64 : 16;
    int t = 0;
    for (int s = 0; s < a.nseg; ++s) { fa.tile_begin[s] = t; t += (a.seg[s].N + edge - 1) / edge; }
    for (int s = a.nseg; s <= SEGS; ++s) fa.tile_begin[s] = t;
    fa.lead_blocks = a.rider_units;
    const int64_t blocks = fa.lead_blocks + (int64_t)t * ((a.R + edge - 1) / edge);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    prof_begin(big ? K_LIN_F32_TILE : K_LIN_F32_LATENCY, stream);
    if (dtype == DT_BF16) {
        if (big) MOA_KLAUNCH((k_linear_f32_tile<bf16_t, SEGS>), grid, dim3(256), 0, stream, fa);
        else MOA_KLAUNCH((k_linear_f32_latency<bf16_t, SEGS>), grid, dim3(256), 0, stream, fa);
    } else {
        if (big) MOA_KLAUNCH((k_linear_f32_tile<float, SEGS>), grid, dim3(256), 0, stream, fa);
        else MOA_KLAUNCH((k_linear_f32_latency<float, SEGS>), grid, dim3(256), 0, stream, fa);
    }
    prof_end(stream);
    return hipGetLastError();
}

hipError_t launch_linear_f32(int dtype, const LinArgs &a, hipStream_t stream)
{
    return a.nseg <= LIN_FEW ? launch_f32_as<LIN_FEW>(dtype, a, stream) : launch_f32_as<LIN_SEGS>(dtype, a, stream);
}

}  // namespace moa
