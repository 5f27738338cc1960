// Projections Y = X W^T (W row-major [N, K]) for the Q/K/V/O projections of LSA, CA and tree verification: which kernel a
// call gets (moa_gemm_bf16.hip, moa_gemm_f32.hip, or the one here that takes whatever those two cannot read), the pass
// that adds up K slices, and the row-wise steps behind a projection.
#include "moa_common.h"
#include "moa_tree_device.h"
#include "moa_sum_device.h"

namespace moa {

// ------------------------------------------------------------------ generic
template <typename T>
__global__ __launch_bounds__(256) void k_linear_generic(const T *__restrict__ X, int64_t R, int K, int64_t ldx,
                                                        const T *__restrict__ W, int N, StoreSpec stp)
{
    __shared__ float Xs[16][65];
    __shared__ float Ws[16][65];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int64_t r0 = (int64_t)blockIdx.y * 64;
    const int n0 = blockIdx.x * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
        for (int i = 0; i < 4; ++i) {
            const int idx = tid + 256 * i, rr = idx >> 4, kk = idx & 15;
            const int64_t r = r0 + rr;
            const int n = n0 + rr, k = k0 + kk;
            Xs[kk][rr] = (r < R && k < K) ? ld<T>(X + r * ldx + k) : 0.f;
            Ws[kk][rr] = (n < N && k < K) ? ld<T>(W + (int64_t)n * K + k) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = Xs[kk][ty * 4 + i]; b[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    T *dst = (T *)stp.dst;
    for (int i = 0; i < 4; ++i) {
        const int64_t r = r0 + ty * 4 + i;
        if (r >= R) continue;
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n >= N) continue;
            const int64_t off = store_offset(stp, r, n);
            if (off >= 0) st<T>(dst + off, acc[i][j]);
        }
    }
}

// ------------------------------------------------------------------ the pass over K slices
__global__ __launch_bounds__(256) void k_linear_splitk_reduce(SumArgs sa) { splitk_reduce_block(sa, (int)blockIdx.x, (int)threadIdx.x); }

// The pass with the residual and the RMS norm behind it (LinArgs::EPI_ADD_NORM): one workgroup per row, every lane
// its 16-byte pieces of the row in registers for both halves (the sum of squares, then the scaled row).  The arithmetic
// is launch_rmsnorm's on x and the projection rounded to the storage type: the same bits as the two launches.
template <int NCH>
__global__ __launch_bounds__(256) void k_linear_splitk_reduce_norm(SumArgs sa)
{
    __shared__ float part[4];
    const int64_t r = blockIdx.x;
    const int d = sa.ntot, nch = d >> 3;
    const float *prow = sa.part + (((r >> 6) * sa.splits) * 64 + (r & 63)) * (int64_t)sa.ntot;
    const bf16_t *x = (const bf16_t *)sa.norm.x + r * d, *g = (const bf16_t *)sa.norm.g;
    float v[NCH][8];
    u32x4 gv[NCH];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = threadIdx.x + 256 * i;
        const bool live = c < nch;
        const int cc = live ? c : 0;
        f32x4 lo, hi;
        splitk_sum8(sa, prow + 8 * cc, lo, hi);
        const u32x4 yv = pack8(lo, hi);                      // the projection as it would be stored
        const u32x4 xv = *(const u32x4 *)(x + 8 * cc);
        gv[i] = *(const u32x4 *)(g + 8 * cc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float l = __uint_as_float(xv[e] << 16) + __uint_as_float(yv[e] << 16);
            const float h = __uint_as_float(xv[e] & 0xffff0000u) + __uint_as_float(yv[e] & 0xffff0000u);
            v[i][2 * e] = l;
            v[i][2 * e + 1] = h;
            if (live) ss += l * l + h * h;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float tot = (part[0] + part[1]) + (part[2] + part[3]);
    const float inv = 1.0f / sqrtf(tot / (float)d + sa.norm.eps);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c >= nch) continue;
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float glo = __uint_as_float(gv[i][e] << 16), ghi = __uint_as_float(gv[i][e] & 0xffff0000u);
            o[e] = pack_bf16x2(v[i][2 * e] * inv * glo, v[i][2 * e + 1] * inv * ghi);
        }
        *(u32x4 *)((bf16_t *)sa.norm.n + r * d + 8 * c) = o;
        *(f32x4 *)(sa.norm.h + r * d + 8 * c) = f32x4{v[i][0], v[i][1], v[i][2], v[i][3]};
        *(f32x4 *)(sa.norm.h + r * d + 8 * c + 4) = f32x4{v[i][4], v[i][5], v[i][6], v[i][7]};
    }
}

hipError_t launch_splitk_sum(const SumArgs &sa, hipStream_t stream)
{
    if (sa.blocks <= 0) return hipSuccess;
    prof_begin(K_LIN_REDUCE, stream);
    if (sa.epi == LinArgs::EPI_ADD_NORM) {
        if (sa.ntot <= 256 * 8 * 2) MOA_KLAUNCH(k_linear_splitk_reduce_norm<2>, dim3((unsigned)sa.R), dim3(256), 0, stream, sa);
        else MOA_KLAUNCH(k_linear_splitk_reduce_norm<4>, dim3((unsigned)sa.R), dim3(256), 0, stream, sa);
        prof_end(stream);
        return hipGetLastError();
    }
    MOA_KLAUNCH(k_linear_splitk_reduce, dim3((unsigned)sa.blocks), dim3(256), 0, stream, sa);
    prof_end(stream);
    return hipGetLastError();
}

// ------------------------------------------------------------------ dispatch
static bool aligned16(const void *p) { return (((uintptr_t)p) & 15) == 0; }

// which kernel a call gets, from types, shapes and alignment alone
enum LinPath { P_BF16, P_F32, P_EACH, P_GENERIC };

static LinPath linear_path(int dtype, const LinArgs &a)
{
    bool own_x = false;
    for (int s = 0; s < a.nseg; ++s) own_x = own_x || a.seg[s].X != nullptr;
    bool fast = dtype == DT_BF16 && a.K % 128 == 0 && a.ldx % 8 == 0 && aligned16(a.X);
    for (int s = 0; s < a.nseg && fast; ++s)
        if (a.seg[s].X) fast = a.seg[s].ldx % 8 == 0 && aligned16(a.seg[s].X);
    for (int s = 0; s < a.nseg && fast; ++s) {
        const StoreSpec &st = a.seg[s].st;
        fast = a.seg[s].N % 32 == 0 && aligned16(a.seg[s].W) && aligned16(st.dst) &&
               (st.mode == StoreSpec::ROW ? st.ld % 8 == 0 : st.dh % 8 == 0);
    }
    if (fast) return P_BF16;
    return linear_f32_ok(dtype, a) ? P_F32 : own_x ? P_EACH : P_GENERIC;
}

int linear_order(int dtype, const LinArgs &a)
{
    switch (linear_path(dtype, a)) {
    case P_BF16: return 2 + linear_bf16_order(a);
    case P_F32: return linear_f32_big(a) ? 2 : 1;
    default: return 0;
    }
}

static hipError_t launch_linear_impl(int dtype, const LinArgs &a, hipStream_t stream, bool *rode, bool *fused);

// the pass that adds up the K slices launch_linear_bf16 has left in a.ws
static hipError_t finish_splits(const LinArgs &a, int splits, hipStream_t stream, bool *fused)
{
    SumArgs sum = {};
    for (int s = 0; s < a.nseg; ++s) {
        sum.st[s] = a.seg[s].st;
        sum.tile_begin[s] = sum.ntot / 64;
        sum.ntot += a.seg[s].N;
    }
    sum.tile_begin[a.nseg] = sum.ntot / 64;
    // the residual + norm pass takes rows of at most 8192 values with 16-byte aligned operands
    const bool norm_ok = a.epi != LinArgs::EPI_ADD_NORM ||
                         (sum.ntot <= 256 * 8 * 4 && a.norm.x && a.norm.g && a.norm.h && a.norm.n &&
                          ((((uintptr_t)a.norm.x) | ((uintptr_t)a.norm.g) | ((uintptr_t)a.norm.h) | ((uintptr_t)a.norm.n)) & 15) == 0);
    *fused = a.epi != LinArgs::EPI_NONE && norm_ok;
    const int64_t items = a.R * ((a.epi == LinArgs::EPI_SWIGLU ? sum.ntot / 2 : sum.ntot) / 8);
    sum.blocks = (int)((items + 255) / 256);
    sum.R = a.R;
    sum.nseg = a.nseg;
    sum.splits = splits;
    sum.part = (const float *)a.ws;
    sum.epi = norm_ok ? a.epi : (int)LinArgs::EPI_NONE;
    sum.epi_res = a.epi_res;
    sum.epi_out = a.epi_out;
    sum.norm = a.norm;
    if (a.epi == LinArgs::EPI_ROPE) {
        sum.rope = a.rope;
        sum.rope_log_theta = log(a.rope.theta);
    }
    return launch_splitk_sum(sum, stream);
}

// kernels without per-segment activation support get one call per segment
static hipError_t launch_linear_each(int dtype, const LinArgs &a, hipStream_t stream)
{
    for (int s = 0; s < a.nseg; ++s) {
        LinArgs one = a;
        one.rider_units = 0;
        one.nseg = 1;
        one.seg[0] = a.seg[s];
        if (a.seg[s].X) { one.X = a.seg[s].X; one.ldx = a.seg[s].ldx; }
        one.seg[0].X = nullptr;
        one.epi = LinArgs::EPI_NONE;
        bool rode = false, fused = false;
        hipError_t e = launch_linear_impl(dtype, one, stream, &rode, &fused);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// *rode is set when the launch carried a.rider in its grid, *fused when it applied a.epi
static hipError_t launch_linear_impl(int dtype, const LinArgs &a, hipStream_t stream, bool *rode, bool *fused)
{
    *rode = false;
    *fused = false;
    if (a.R <= 0) return hipSuccess;
    const LinPath path = linear_path(dtype, a);
    if (path == P_BF16) {
        *rode = a.rider_units > 0;
        int splits = 1;
        // these epilogues store 16 bytes at a time; elsewhere the projection is stored and finished element by element
        if (!aligned16(a.epi_out)) {
            LinArgs b = a;
            b.epi = LinArgs::EPI_NONE;
            hipError_t e = launch_linear_bf16(b, stream, fused, &splits);
            return e != hipSuccess || splits == 1 ? e : finish_splits(b, splits, stream, fused);
        }
        hipError_t e = launch_linear_bf16(a, stream, fused, &splits);
        if (e != hipSuccess || splits == 1) return e;
        return finish_splits(a, splits, stream, fused);
    }
    if (path == P_F32) {
        *rode = a.rider_units > 0;
        return launch_linear_f32(dtype, a, stream);
    }
    if (path == P_EACH) return launch_linear_each(dtype, a, stream);
    for (int s = 0; s < a.nseg; ++s) {
        dim3 grid((a.seg[s].N + 63) / 64, (unsigned)((a.R + 63) / 64));
        if (dtype == DT_BF16)
            { prof_begin(K_LIN_GENERIC, stream); MOA_KLAUNCH(k_linear_generic<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t *)a.X, a.R, a.K,
                               a.ldx, (const bf16_t *)a.seg[s].W, a.seg[s].N, a.seg[s].st); prof_end(stream); }
        else
            { prof_begin(K_LIN_GENERIC, stream); MOA_KLAUNCH(k_linear_generic<float>, grid, dim3(256), 0, stream, (const float *)a.X, a.R, a.K,
                               a.ldx, (const float *)a.seg[s].W, a.seg[s].N, a.seg[s].st); prof_end(stream); }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_linear(int dtype, const LinArgs &a, hipStream_t stream)
{
    if (a.epi == LinArgs::EPI_ADD_F32 && a.nseg != 1) return hipErrorInvalidValue;
    if (a.epi == LinArgs::EPI_SWIGLU && (a.nseg != 2 || a.seg[0].N != a.seg[1].N)) return hipErrorInvalidValue;
    if (a.epi == LinArgs::EPI_ADD_NORM && a.nseg != 1) return hipErrorInvalidValue;
    if (a.epi == LinArgs::EPI_ROPE && (a.nseg != 3 || a.rope.dh % 16 || a.seg[0].N != a.rope.H * a.rope.dh || a.seg[1].N != a.rope.Hkv * a.rope.dh))
        return hipErrorInvalidValue;
    bool rode = false, fused = false;
    hipError_t e = launch_linear_impl(dtype, a, stream, &rode, &fused);
    if (e != hipSuccess) return e;
    if (a.epi != LinArgs::EPI_NONE && !fused) {     // the projection was stored as its segments say: finish row-wise
        const RopeArgs &ro = a.rope;
        if (a.epi == LinArgs::EPI_SWIGLU) e = launch_swiglu(dtype, a.seg[0].st.dst, a.R, a.seg[0].N, a.epi_out, stream);
        else if (a.epi == LinArgs::EPI_ROPE)
            e = launch_rope(dtype, ro.q, ro.k_draft, ro.prefix_len, ro.depth, ro.B, ro.Mn, ro.M, ro.node0, ro.H, ro.Hkv, ro.dh, ro.theta,
                            ro.P_cap, stream);
        else if (a.epi == LinArgs::EPI_ADD_NORM)
            e = launch_rmsnorm(dtype, a.norm.x, a.seg[0].st.dst, a.R, a.seg[0].N, a.norm.g, a.norm.eps, a.norm.h, a.norm.n, stream);
        else e = launch_add_out(dtype, a.epi_res, a.seg[0].st.dst, a.R * a.seg[0].N, a.epi_out, stream);
        if (e != hipSuccess) return e;
    }
    if (a.rider_units <= 0 || rode) return hipSuccess;
    return launch_step_small(a.rider, stream);      // the kernel that ran has no spare workgroups for it
}

}  // namespace moa

// ------------------------------------------------------------------ identity "projection"
// A NULL weight means the input is already projected; rows still have to reach the layout the
// store spec describes (e.g. [B, Hkv, M, dh] slabs).
namespace moa {

template <typename T>
__global__ void k_scatter_copy(const T *__restrict__ X, int64_t R, int N, int64_t ldx, StoreSpec stp)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= R * N) return;
    const int64_t r = idx / N;
    const int n = (int)(idx - r * N);
    const int64_t off = store_offset(stp, r, n);
    if (off >= 0) ((T *)stp.dst)[off] = X[r * ldx + n];
}

hipError_t launch_scatter_copy(int dtype, const void *X, int64_t R, int N, int64_t ldx, const StoreSpec &st,
                               hipStream_t stream)
{
    if (R <= 0) return hipSuccess;
    const int64_t total = R * N;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (dtype == DT_BF16)
        { prof_begin(K_SCATTER, stream); MOA_KLAUNCH(k_scatter_copy<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t *)X, R, N, ldx, st); prof_end(stream); }
    else
        { prof_begin(K_SCATTER, stream); MOA_KLAUNCH(k_scatter_copy<float>, grid, dim3(256), 0, stream, (const float *)X, R, N, ldx, st); prof_end(stream); }
    return hipGetLastError();
}

}  // namespace moa
