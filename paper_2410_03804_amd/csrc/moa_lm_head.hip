// Greedy token of the LLM at every tree node: tgt[r] = argmax_v x[r] . W[v] over the vocabulary (Sec. 2.1,
// y ~ Softmax(LM_head(o)); greedy verification takes the arg max).  The logits are never stored: the head is one
// pass over its weights ([V, d], 1 GiB at the Llama-3 shape, the largest single read of a decoding cycle), each
// workgroup reduces its tile of tokens to one (logit, id) pair per row and a second small kernel reduces the pairs.
// The product is the projections' (GemmLoop): HBM-bound up to about 128 rows, by the matrix cores and the way from L2
// to LDS above.  128256 tokens x 4096: 8 rows 173 us (6.1 TB/s), 60 rows 184 (5.7 TB/s; 204 with weights in registers and
// the activation chunk staged behind two barriers), 256 rows in one pass 256 us where passes of 64 rows took 4 x 204.
// That an XCD walks a contiguous range of the head is worth a tenth (tiles dealt round-robin: 211 us at 60 rows).
#include "moa_common.h"
#include "moa_gemm_device.h"
#include "../../include/moa.h"

namespace moa {

struct LmHeadArgs {
    const bf16_t *X;      // [R, K]
    const bf16_t *W;      // [V, K]
    int R, K, V;
    int tiles, tiles_per_xcd;
    float *pval;          // [R, tiles]
    int32_t *pid;         // [R, tiles]
};

__device__ __forceinline__ bool better(float a, int ia, float b, int ib) { return a > b || (a == b && ia < ib); }

template <int WR, int WF, int MR, int NF, int SX, int SW, int WK>
__global__ __launch_bounds__(64 * WR * WF * WK) void k_lm_head_argmax(LmHeadArgs a)
{
    using Loop = GemmLoop<WR, WF, MR, NF, SX, SW, WK>;
    constexpr int BM = Loop::BM, BN = Loop::BN;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // an XCD's workgroups (every eighth) walk a contiguous range of the head
    const int tile = (int)(blockIdx.x & 7) * a.tiles_per_xcd + (int)(blockIdx.x >> 3), n0 = tile * BN;
    if (tile >= a.tiles) return;
    Loop g;
    g.set_x(a.X, a.K, a.R);
    g.set_w(a.K, a.V - n0, [&](int blk, int *first) {          // tokens past the end repeat the last one; masked below
        *first = 32 * blk;
        return (const char *)a.W + (int64_t)n0 * a.K * 2;
    });
    const bool mine = g.run(smem, 0, a.K / (Loop::BK * WK));
    // best of the wavefront's tokens per row, then of the wavefronts along the tokens
    wait_loads_and_barrier<0>();                               // the rings are dead; their memory is reused
    float *wv = (float *)smem;                                 // [WF][BM]
    int32_t *wi = (int32_t *)(wv + WF * BM);
    const int l16 = g.lane & 15, quart = g.lane >> 4;
    if (mine) {
#pragma unroll
        for (int j = 0; j < MR; ++j) {
            float bv = -INFINITY;
            int bi = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int id = n0 + g.wave_feature() + 32 * i + 8 * quart + e;
                    const float v = g.acc[i][j][e >> 2][e & 3];
                    if (id < a.V && better(v, id, bv, bi)) { bv = v; bi = id; }
                }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
            }
            if (quart == 0) {
                const int at = (g.wave % WF) * BM + g.wave_row() + 16 * j + l16;
                wv[at] = bv;
                wi[at] = bi;
            }
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < BM && r < a.R; r += 64 * WR * WF * WK) {
        float bv = wv[r];
        int bi = wi[r];
#pragma unroll
        for (int w = 1; w < WF; ++w)
            if (better(wv[w * BM + r], wi[w * BM + r], bv, bi)) { bv = wv[w * BM + r]; bi = wi[w * BM + r]; }
        a.pval[(int64_t)r * a.tiles + tile] = bv;
        a.pid[(int64_t)r * a.tiles + tile] = bi;
    }
}

// one workgroup per row: the best of the tiles' pairs
__global__ __launch_bounds__(256) void k_lm_head_reduce(const float *__restrict__ pval, const int32_t *__restrict__ pid, int tiles,
                                                        int32_t *__restrict__ tgt, float *__restrict__ best)
{
    __shared__ float sv[4];
    __shared__ int si[4];
    const int r = blockIdx.x, t = threadIdx.x;
    const float *pv = pval + (int64_t)r * tiles;
    const int32_t *pi = pid + (int64_t)r * tiles;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int k = t; k < tiles; k += 256)
        if (better(pv[k], pi[k], bv, bi)) { bv = pv[k]; bi = pi[k]; }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(bv, o);
        const int oi = __shfl_xor(bi, o);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if ((t & 63) == 0) { sv[t >> 6] = bv; si[t >> 6] = bi; }
    __syncthreads();
    if (t == 0) {
#pragma unroll
        for (int w = 1; w < 4; ++w)
            if (better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
        tgt[r] = bi;
        if (best) best[r] = bv;
    }
}

// one pass: the most rows (at most pa->R on entry) whose pairs fit `pairs`
template <int WR, int WF, int MR, int NF, int SX, int SW, int WK>
static hipError_t launch_head(LmHeadArgs *pa, int64_t pairs, hipStream_t st)
{
    using Loop = GemmLoop<WR, WF, MR, NF, SX, SW, WK>;
    static_assert(Loop::BN >= Loop::BM, "");        // so that a pass takes (nearly) all the rows its tile has
    LmHeadArgs &a = *pa;
    a.tiles = (a.V + Loop::BN - 1) / Loop::BN;
    a.tiles_per_xcd = (a.tiles + 7) / 8;
    if (a.R > pairs / a.tiles) a.R = (int)(pairs / a.tiles);
    a.pid = (int32_t *)(a.pval + (size_t)a.tiles * a.R);
    static bool raised[16] = {};
    hipError_t e = raise_lds_limit_once(raised, (const void *)k_lm_head_argmax<WR, WF, MR, NF, SX, SW, WK>, Loop::LDS_BYTES);
    if (e != hipSuccess) return e;
    prof_begin(K_LM_HEAD, st);
    MOA_KLAUNCH((k_lm_head_argmax<WR, WF, MR, NF, SX, SW, WK>), dim3(8 * a.tiles_per_xcd), dim3(64 * WR * WF * WK), Loop::LDS_BYTES, st, a);
    prof_end(st);
    return hipGetLastError();
}

}  // namespace moa

using namespace moa;

extern "C" {

int32_t moa_lm_head_workspace_bytes(int32_t V, size_t *bytes_host)
{
    if (!bytes_host) return api_fail(MOA_ERR_NULL, "lm_head_workspace_bytes: bytes_host is NULL");
    if (V < 1) return api_fail(MOA_ERR_SHAPE, "lm_head_workspace_bytes: V < 1");
    *bytes_host = (size_t)((V + 63) / 64) * 64 * (sizeof(float) + sizeof(int32_t));
    return MOA_OK;
}

int32_t moa_lm_head_argmax(int32_t dtype, const void *x, int32_t R, int32_t d, const void *w, int32_t V, int32_t *tgt,
                           float *best, void *ws, size_t ws_bytes, void *stream)
{
    if (!x || !w || !tgt) return api_fail(MOA_ERR_NULL, "lm_head_argmax: NULL pointer");
    if (dtype != MOA_BF16) return api_fail(MOA_ERR_DTYPE, "lm_head_argmax: bf16 only");
    if (R < 1 || V < 1 || d < 128 || d % 128) return api_fail(MOA_ERR_SHAPE, "lm_head_argmax: R >= 1, V >= 1, d a multiple of 128");
    if ((((uintptr_t)x) | ((uintptr_t)w)) & 15) return api_fail(MOA_ERR_SHAPE, "lm_head_argmax: x and w must be 16-byte aligned");
    size_t need = 0;
    (void)moa_lm_head_workspace_bytes(V, &need);
    if (!ws || (((uintptr_t)ws) & 255) || ws_bytes < need) return api_fail(MOA_ERR_WORKSPACE, "lm_head_argmax: workspace NULL, misaligned or smaller than moa_lm_head_workspace_bytes");
    hipStream_t st = (hipStream_t)stream;
    // Up to 256 rows per pass over the weights, in the tile that the row count calls for.
    const int64_t pairs = (int64_t)(need / (sizeof(float) + sizeof(int32_t)));     // a pair per token in 64s
    LmHeadArgs a = {};
    for (int r0 = 0; r0 < R; r0 += a.R) {
        a.X = (const bf16_t *)x + (int64_t)r0 * d;
        a.W = (const bf16_t *)w;
        a.R = R - r0 < 256 ? R - r0 : 256;
        a.K = d;
        a.V = V;
        a.pval = (float *)ws;
        prof_set_site(S_LM_HEAD);
        // Wide tiles keep the activations' share of what goes through a compute unit small; with fewer of them than two
        // per compute unit the narrow ones fill the chip better (40 x 4096 x 32000: 50 against 58 us).
        // 17 to 32 rows: three stages of activations, 18 x 4096 x 128256 174 us, 30 rows 178; two of them up to 4 us more on some cards.
        const bool wide = V >= 2 * 256 * 128;
        hipError_t e;
        if (a.R <= 16) e = launch_head<1, 1, 1, 2, 3, 3, 2>(&a, pairs, st);
        else if (a.R <= 32) e = launch_head<2, 1, 1, 2, 3, 3, 2>(&a, pairs, st);
        else if (a.R <= 64) e = wide ? launch_head<2, 2, 2, 2, 3, 3, 1>(&a, pairs, st) : launch_head<2, 2, 2, 1, 4, 6, 1>(&a, pairs, st);
        else if (a.R <= 128) e = wide ? launch_head<2, 2, 4, 2, 2, 3, 1>(&a, pairs, st) : launch_head<4, 2, 2, 2, 4, 4, 1>(&a, pairs, st);
        else e = launch_head<4, 2, 4, 4, 2, 2, 1>(&a, pairs, st);
        if (e != hipSuccess) return api_fail(MOA_ERR_HIP, "lm_head_argmax: launch failed");
        prof_begin(K_LM_HEAD_REDUCE, st);
        MOA_KLAUNCH(k_lm_head_reduce, dim3(a.R), dim3(256), 0, st, a.pval, a.pid, a.tiles, tgt + r0, best ? best + r0 : nullptr);
        prof_end(st);
        if (hipGetLastError() != hipSuccess) return api_fail(MOA_ERR_HIP, "lm_head_argmax: launch failed");
    }
    return MOA_OK;
}

}  // extern "C"
