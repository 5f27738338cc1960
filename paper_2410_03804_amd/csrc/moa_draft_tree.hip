// Draft-tree construction on the device (Sec. 2.2, tree drafting as in EAGLE-2): per level, the joint
// log-probabilities of the Bw*Bw expansions and the best Bw of them; at the end the m best of all candidates,
// relabelled so that parents come first; and the Bw most probable tokens of a row of logits.
// Every ranking decision is taken on single-precision numbers formed by one addition, ties to the lower index,
// so results are a pure function of the inputs.  These are latency-sized kernels: one workgroup per sequence
// (or per row of logits), everything in LDS / registers.
#include "moa_common.h"
#include "../../include/moa.h"

namespace moa {

constexpr int TREE_MAX_BREADTH = 16;      // Bw*Bw expansions fit one 256-thread workgroup
constexpr int TREE_MAX_CAND = 4096;       // candidates ranked in LDS by moa_tree_finalize

__device__ __forceinline__ bool ranks_before(float a, int ia, float b, int ib) { return a > b || (a == b && ia < ib); }

// a float as an unsigned integer of the same order (-inf lowest)
__device__ __forceinline__ uint32_t orderable(float v)
{
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_orderable(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// (value, index) as one 64-bit key whose unsigned order is "ranks before": larger value first, then smaller index.
// -0 and +0 are one value.  NaN never gets here (callers map it to -inf first).
__device__ __forceinline__ uint64_t rank_key(float v, int idx)
{
    return ((uint64_t)orderable(v + 0.0f) << 32) | (uint64_t)(0xffffffffu - (uint32_t)idx);
}
__device__ __forceinline__ float key_value(uint64_t k) { return from_orderable((uint32_t)(k >> 32)); }
__device__ __forceinline__ int key_index(uint64_t k) { return (int)(0xffffffffu - (uint32_t)k); }

// how many of keys[0..n) rank before `mine`; keys is a 16-byte aligned LDS array, read two keys at a time (every
// lane reads the same address: a broadcast)
typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
__device__ __forceinline__ int rank_among(const uint64_t *keys, int n, uint64_t mine)
{
    int rank = 0;
    const int n2 = n & ~1;
#pragma unroll 4
    for (int u = 0; u < n2; u += 2) {
        const u64x2 a = *(const u64x2 *)&keys[u];
        rank += (a[0] > mine ? 1 : 0) + (a[1] > mine ? 1 : 0);
    }
    if (n2 < n) rank += keys[n2] > mine ? 1 : 0;
    return rank;
}

__global__ __launch_bounds__(256) void k_tree_expand(int level, int Bw, int n_max, const float *__restrict__ child_logp,
                                                     const int32_t *__restrict__ child_tok, float *__restrict__ cand_logp,
                                                     int32_t *__restrict__ cand_tok, int32_t *__restrict__ cand_parent,
                                                     int32_t *__restrict__ frontier)
{
    __shared__ __attribute__((aligned(16))) uint64_t lp[256];
    const int b = blockIdx.x, t = threadIdx.x;
    const int F = level == 1 ? 1 : Bw, n = F * Bw;
    const int base = level == 1 ? 0 : Bw + (level - 2) * Bw * Bw;
    float *clp = cand_logp + (int64_t)b * n_max;
    int32_t *ctk = cand_tok + (int64_t)b * n_max, *cpr = cand_parent + (int64_t)b * n_max, *fr = frontier + (int64_t)b * Bw;
    uint64_t mine = 0;
    if (t < n) {
        const int f = t / Bw;
        float v = child_logp[(int64_t)b * n + t];
        v = v == v ? fminf(v, 0.0f) : -INFINITY;          // a child is never more likely than its parent
        int par = -1;
        if (level > 1) {
            par = fr[f];
            par = par < 0 ? 0 : (par >= base ? base - 1 : par);      // a corrupt frontier cannot leave the array
            v = clp[par] + v;                                        // one single-precision addition
        }
        clp[base + t] = v;
        ctk[base + t] = child_tok[(int64_t)b * n + t];
        cpr[base + t] = par;
        mine = rank_key(v, t);
        lp[t] = mine;
    }
    __syncthreads();                                       // every read of the old frontier is done
    if (t < n) {
        const int rank = rank_among(lp, n, mine);
        if (rank < Bw) fr[rank] = base + t;
    }
}

// One thread per candidate (several where there are more than 1024).  Bound by the n^2 comparisons of one compute unit, so
// the keys are 32-bit values: which of two equal ones is ahead follows from the index alone, and for every candidate
// outside the wavefront's own 64 that is decided by >= against >.  328 candidates: 8.4 us against 12.3 with 64-bit keys and
// runs of candidates per thread.
__global__ __launch_bounds__(1024) void k_tree_finalize(int n, int n_max, int keep, int ld_out, const int32_t *__restrict__ root_tok,
                                                        const float *__restrict__ cand_logp, const int32_t *__restrict__ cand_tok,
                                                        const int32_t *__restrict__ cand_parent, int32_t *__restrict__ parent,
                                                        int32_t *__restrict__ tok, int32_t *__restrict__ node_cand,
                                                        int32_t *dev_status)
{
    __shared__ __attribute__((aligned(16))) uint32_t lp[TREE_MAX_CAND];     // 0 (below every value) behind the last
    __shared__ int32_t node_of[TREE_MAX_CAND];
    __shared__ int32_t cnt[TREE_MAX_CAND / 64];
    const int b = blockIdx.x, t = threadIdx.x, nt = blockDim.x, lane = t & 63;
    const float *clp = cand_logp + (int64_t)b * n_max;
    const int32_t *ctk = cand_tok + (int64_t)b * n_max, *cpr = cand_parent + (int64_t)b * n_max;
    int32_t *po = parent + (int64_t)b * ld_out, *to = tok + (int64_t)b * ld_out, *no = node_cand + (int64_t)b * ld_out;
    const int n64 = (n + 63) & ~63;
    for (int c = t; c < n64; c += nt) {
        const float v = c < n ? clp[c] : 0.f;
        lp[c] = c < n ? orderable((v == v ? v : -INFINITY) + 0.0f) : 0u;
    }
    if (t == 0) {
        po[0] = -1;
        to[0] = root_tok[b];
        no[0] = -1;
    }
    __syncthreads();
    // rank = candidates of a larger value + candidates of the same value in front.  n64 and nt are multiples of 64: a
    // wavefront holds 64 consecutive candidates or none
    for (int c = t; c < n64; c += nt) {
        const uint32_t mine = lp[c];
        const int own = c & ~63;
        int rank = 0;
#pragma unroll 4
        for (int u = 0; u < own; u += 4) {
            const u32x4 k = *(const u32x4 *)&lp[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += k[e] >= mine ? 1 : 0;
        }
#pragma unroll 4
        for (int u = own; u < own + 64; u += 4) {
            const u32x4 k = *(const u32x4 *)&lp[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += k[e] > mine || (k[e] == mine && u + e < c) ? 1 : 0;
        }
#pragma unroll 4
        for (int u = own + 64; u < n64; u += 4) {
            const u32x4 k = *(const u32x4 *)&lp[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += k[e] > mine ? 1 : 0;
        }
        const bool kept = c < n && rank < keep;
        const uint64_t who = __ballot(kept);
        node_of[c] = kept ? __popcll(who & ((1ull << lane) - 1)) : -1;      // its place among the wavefront's
        if (lane == 0) cnt[c >> 6] = __popcll(who);
    }
    __syncthreads();
    // node numbers in candidate order behind the root
    for (int c = t; c < n64; c += nt) {
        int before = 0;
        for (int w = lane; w < (c >> 6); w += 64) before += cnt[w];          // at most one: there are at most 64 groups
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o);
        if (node_of[c] >= 0) node_of[c] += 1 + before;
    }
    __syncthreads();
    for (int c = t; c < n; c += nt) {
        const int i = node_of[c];
        if (i < 0) continue;
        const int p = cpr[c];
        int pn = 0;
        if (p >= 0) {
            pn = (p < c) ? node_of[p] : -1;
            if (pn < 0) {                                  // cannot happen with arrays written by k_tree_expand
                pn = 0;
                if (dev_status) atomicOr(dev_status, MOA_DEV_BAD_PARENT);
            }
        }
        po[i] = pn;
        to[i] = ctk[c];
        no[i] = c;
    }
}

// ---- the Bw most probable tokens of a row of logits, with log-probabilities
// A row of the vocabulary is cut into S slices, one workgroup each, so that a handful of rows still fills the chip.  A
// thread holds its (at most 32) values in registers.  A wavefront ranks its 64 threads' best values; the Bw-th of them is a
// bound that Bw of its own values reach, so nothing below the largest of the four wavefronts' bounds can be among the
// slice's Bw best, and what reaches it (a few times Bw values, all of them in at most 4 Bw threads) is ranked in LDS.  A
// second kernel ranks the S*Bw survivors of a row and merges the slices' (max, sum of exponentials).
// Latency bound: two barriers per slice.  8 rows of 128256 bf16 logits: 6.4 + 3.9 us against 14.1 + 6.3 with every thread's
// values sorted, Bw rounds of two barriers over the heads of the 256 lists, and 2-byte loads.

// Wavefront-wide maximum of an unsigned value by data-parallel-primitive moves inside the vector ALU (four shifts within
// the rows of 16 lanes, then two row broadcasts), read from lane 63: a dozen ALU instructions where the shuffle form makes
// six trips through the LDS crossbar.  Lanes a move does not reach keep their own value, which is harmless for a maximum.
__device__ __forceinline__ uint32_t wave_reduce_max(uint32_t x)
{
#define MOA_DPP_STEP(ctrl)                                                                                   \
    {                                                                                                        \
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, 0xf, 0xf, false);     \
        x = o > x ? o : x;                                                                                   \
    }
    MOA_DPP_STEP(0x111)   // row_shr:1
    MOA_DPP_STEP(0x112)   // row_shr:2
    MOA_DPP_STEP(0x114)   // row_shr:4
    MOA_DPP_STEP(0x118)   // row_shr:8   -> lane 15 of a row holds the row's result
    MOA_DPP_STEP(0x142)   // row_bcast:15 -> lane 31: rows 0-1, lane 63: rows 2-3
    MOA_DPP_STEP(0x143)   // row_bcast:31 -> lane 63: all four rows
#undef MOA_DPP_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

constexpr int TOPK_EPT = 32;              // values a thread keeps
constexpr int TOPK_MIN_SLICES = 32;

static int topk_slices(int V)
{
    const int need = (V + 256 * TOPK_EPT - 1) / (256 * TOPK_EPT);
    return need > TOPK_MIN_SLICES ? need : TOPK_MIN_SLICES;
}

// scratch per (row, slice): Bw order keys (best first; the lowest value with id INT_MAX where the slice ran out), max, sum.
// VEC: rows are 16-byte aligned and whole 16-byte pieces.  A thread's values are runs of eight, so their ids ascend.
template <int EPT, bool VEC>
__global__ __launch_bounds__(256) void k_topk_slices(int is_bf16, const void *__restrict__ logits, int V, int Vs, int Bw, int S,
                                                     uint64_t *__restrict__ skey, float *__restrict__ smax, float *__restrict__ ssum)
{
    __shared__ __attribute__((aligned(16))) uint64_t heads[4][64];
    __shared__ __attribute__((aligned(16))) uint64_t ck[4 * TREE_MAX_BREADTH * EPT];
    __shared__ uint64_t bound[4];
    __shared__ float wm[4], wsum[4];
    __shared__ int count;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int s = blockIdx.x % S;
    const int64_t r = blockIdx.x / S;
    const int v0 = min(s * Vs, V), v1 = min(v0 + Vs, V);
    const float *rf = (const float *)logits + r * V;
    const bf16_t *rb = (const bf16_t *)logits + r * V;
    float x[EPT];
#pragma unroll
    for (int p = 0; p < EPT / 8; ++p) {
        const int v = v0 + 8 * (t + 256 * p);
        if (VEC) {
            u32x4 a = {}, b = {};
            if (v < v1) {
                a = is_bf16 ? *(const u32x4 *)(rb + v) : *(const u32x4 *)(rf + v);
                if (!is_bf16) b = *(const u32x4 *)(rf + v + 4);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float f0 = is_bf16 ? __uint_as_float((e & 1 ? a[e / 2] & 0xffff0000u : a[e / 2] << 16)) : __uint_as_float(a[e]);
                const float f1 = is_bf16 ? __uint_as_float((e & 1 ? a[2 + e / 2] & 0xffff0000u : a[2 + e / 2] << 16)) : __uint_as_float(b[e]);
                x[8 * p + e] = v < v1 ? f0 : -INFINITY;
                x[8 * p + 4 + e] = v < v1 ? f1 : -INFINITY;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[8 * p + e] = v + e < v1 ? (is_bf16 ? bf2f(rb[v + e]) : rf[v + e]) : -INFINITY;
        }
    }
    auto id_of = [&](int i) { return v0 + 8 * (t + 256 * (i >> 3)) + (i & 7); };
    float m = -INFINITY;
    uint32_t best = 0;
    int best_id = v0 + 8 * t;                              // the first of the thread's values that reach its best
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        m = fmaxf(m, x[i]);
        const uint32_t k = orderable(x[i] + 0.0f);         // -0 and +0 are the same value, as in every comparison here
        if (k > best) { best = k; best_id = id_of(i); }
    }
    const uint64_t head = best_id < v1 ? ((uint64_t)best << 32) | (uint64_t)(0xffffffffu - (uint32_t)best_id) : 0;
    const uint32_t mk = wave_reduce_max(orderable(m));
    heads[wave][lane] = head;
    if (lane == 0) { bound[wave] = 0; wm[wave] = from_orderable(mk); }
    if (t == 0) count = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a wavefront's LDS traffic is processed in order
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (rank_among(heads[wave], 64, head) == Bw - 1 && head) bound[wave] = head;   // no thread: every value counts
    __syncthreads();
    m = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
    uint64_t lo = bound[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) lo = bound[w] > lo ? bound[w] : lo;
    if (head && head >= lo) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const uint64_t k = rank_key(x[i], id_of(i));
            if (k >= lo && id_of(i) < v1) ck[atomicAdd(&count, 1)] = k;
        }
    }
    float sum = 0.f;
    if (m > -INFINITY) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) sum += __expf(x[i] - m);      // exp(-inf) = 0 for the padding
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0) wsum[wave] = sum;
    __syncthreads();
    const int64_t slot = r * S + s;
    if (t == 0) { smax[slot] = m; ssum[slot] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]); }
    const int n = count;
    for (int c = t; c < n; c += 256) {
        const uint64_t mine = ck[c];
        const int rank = rank_among(ck, n, mine);
        if (rank < Bw) skey[slot * Bw + rank] = mine;
    }
    if (t >= n && t < Bw) skey[slot * Bw + t] = rank_key(-INFINITY, 0x7fffffff);
}

// One workgroup per row: rank the S*Bw survivors, merge the log-sum-exp (every wavefront for itself: no barriers).  Four lanes
// share a candidate and count a quarter of the keys each: the chain of LDS reads behind one another is what the ranking costs
// (256 survivors, a thread per candidate: 6.1 us, of which that chain was a third; 3.9 now).
__global__ __launch_bounds__(1024) void k_topk_merge(int Bw, int S, const uint64_t *__restrict__ skey, const float *__restrict__ smax,
                                                     const float *__restrict__ ssum, int32_t *__restrict__ tok, float *__restrict__ logp)
{
    extern __shared__ __attribute__((aligned(16))) uint64_t ck[];   // order keys, 0 (behind every one) up to a multiple of eight
    const int t = threadIdx.x, lane = t & 63, nt = blockDim.x;
    const int64_t r = blockIdx.x;
    const int n = S * Bw, n8 = (n + 7) & ~7;
    // everything the row needs is requested at once: one trip to memory instead of three
    float m = -INFINITY, mk = -INFINITY, sk = 0.f;
    if (lane < S) { mk = smax[r * S + lane]; sk = ssum[r * S + lane]; }
    for (int c = t; c < n8; c += nt) ck[c] = c < n ? skey[r * n + c] : 0;
    m = mk;
    for (int k = lane + 64; k < S; k += 64) m = fmaxf(m, smax[r * S + k]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float sum = mk > -INFINITY ? sk * __expf(mk - m) : 0.f;
    for (int k = lane + 64; k < S; k += 64) {
        const float mm = smax[r * S + k];
        if (mm > -INFINITY) sum += ssum[r * S + k] * __expf(mm - m);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
    const float lse = m + __logf(sum);
    __syncthreads();
    const int part = t & 3;
    for (int c = t >> 2; c < n; c += nt >> 2) {            // the four lanes of a candidate stay together
        const uint64_t mine = ck[c];
        int rank = 0;
#pragma unroll 8
        for (int u = 2 * part; u < n8; u += 8) {
            const u64x2 a = *(const u64x2 *)&ck[u];
            rank += (a[0] > mine ? 1 : 0) + (a[1] > mine ? 1 : 0);
        }
        rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xf, 0xf, false);     // quad_perm [1, 0, 3, 2]
        rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xf, 0xf, false);     // quad_perm [2, 3, 0, 1]
        const int id = key_index(mine);
        if (part == 0 && id != 0x7fffffff && rank < Bw) {  // (an exhausted slice's filler)
            tok[r * Bw + rank] = id;
            logp[r * Bw + rank] = key_value(mine) - lse;
        }
    }
}

}  // namespace moa

using namespace moa;

extern "C" {

static int32_t tree_fail(int32_t code, const char *msg) { return moa::api_fail(code, msg); }

int32_t moa_tree_expand_level(int32_t level, int32_t B, int32_t Bw, int32_t n_max, const float *child_logp,
                              const int32_t *child_tok, float *cand_logp, int32_t *cand_tok, int32_t *cand_parent,
                              int32_t *frontier, void *stream)
{
    if (!child_logp || !child_tok || !cand_logp || !cand_tok || !cand_parent || !frontier) return tree_fail(MOA_ERR_NULL, "tree_expand_level: NULL pointer");
    if (level < 1 || B < 1 || Bw < 1 || Bw > TREE_MAX_BREADTH) return tree_fail(MOA_ERR_SHAPE, "tree_expand_level: level >= 1, B >= 1, 1 <= breadth <= 16");
    const int64_t end = level == 1 ? Bw : (int64_t)Bw + (int64_t)(level - 1) * Bw * Bw;
    if (end > n_max) return tree_fail(MOA_ERR_RANGE, "tree_expand_level: the level's candidates do not fit n_max");
    prof_set_site(S_TREE_EXPAND);
    prof_begin(K_TREE_EXPAND, (hipStream_t)stream);
    MOA_KLAUNCH(k_tree_expand, dim3(B), dim3(256), 0, (hipStream_t)stream, level, Bw, n_max, child_logp, child_tok, cand_logp,
                cand_tok, cand_parent, frontier);
    prof_end((hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? MOA_OK : tree_fail(MOA_ERR_HIP, "tree_expand_level: launch failed");
}

int32_t moa_tree_finalize(int32_t B, int32_t n_cand, int32_t n_max, int32_t m, const int32_t *root_tok,
                          const float *cand_logp, const int32_t *cand_tok, const int32_t *cand_parent, int32_t *parent,
                          int32_t *tok, int32_t *node_cand, int32_t *dev_status, void *stream)
{
    if (!root_tok || !cand_logp || !cand_tok || !cand_parent || !parent || !tok || !node_cand) return tree_fail(MOA_ERR_NULL, "tree_finalize: NULL pointer");
    if (B < 1 || n_cand < 0 || n_cand > n_max || n_cand > TREE_MAX_CAND || m < 0 || 1 + m > MOA_MAX_TREE)
        return tree_fail(MOA_ERR_SHAPE, "tree_finalize: 0 <= n_cand <= min(n_max, 4096), 1 + m <= 256");
    const int keep = m < n_cand ? m : n_cand;
    prof_set_site(S_TREE_FINALIZE);
    prof_begin(K_TREE_FINALIZE, (hipStream_t)stream);
    MOA_KLAUNCH(k_tree_finalize, dim3(B), dim3(n_cand < 64 ? 64 : n_cand > 960 ? 1024 : (n_cand + 63) & ~63), 0, (hipStream_t)stream, n_cand, n_max, keep, 1 + m, root_tok, cand_logp,
                cand_tok, cand_parent, parent, tok, node_cand, dev_status);
    prof_end((hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? MOA_OK : tree_fail(MOA_ERR_HIP, "tree_finalize: launch failed");
}

int32_t moa_topk_workspace_bytes(int32_t F, int32_t V, int32_t Bw, size_t *bytes_host)
{
    if (!bytes_host) return tree_fail(MOA_ERR_NULL, "topk_workspace_bytes: bytes_host is NULL");
    if (F < 1 || V < 1 || Bw < 1 || Bw > TREE_MAX_BREADTH) return tree_fail(MOA_ERR_SHAPE, "topk_workspace_bytes: F >= 1, V >= 1, 1 <= breadth <= 16");
    const size_t S = (size_t)topk_slices(V);
    *bytes_host = (size_t)F * S * ((size_t)Bw * 8 + 8);
    return MOA_OK;
}

int32_t moa_topk_logprob(int32_t dtype, const void *logits, int32_t F, int32_t V, int32_t Bw, int32_t *tok, float *logp,
                         void *ws, size_t ws_bytes, void *stream)
{
    if (!logits || !tok || !logp) return tree_fail(MOA_ERR_NULL, "topk_logprob: NULL pointer");
    if (dtype != MOA_F32 && dtype != MOA_BF16) return tree_fail(MOA_ERR_DTYPE, "topk_logprob: dtype");
    if (F < 1 || V < 1 || Bw < 1 || Bw > TREE_MAX_BREADTH || Bw > V) return tree_fail(MOA_ERR_SHAPE, "topk_logprob: F >= 1, 1 <= breadth <= min(16, V)");
    const int S = topk_slices(V);
    const size_t n = (size_t)F * S;
    if ((int64_t)F * S > 0x7fffffff) return tree_fail(MOA_ERR_SHAPE, "topk_logprob: too many rows");
    const size_t need = n * ((size_t)Bw * 8 + 8);
    if (!ws || (((uintptr_t)ws) & 255) || ws_bytes < need) return tree_fail(MOA_ERR_WORKSPACE, "topk_logprob: workspace NULL, misaligned or smaller than moa_topk_workspace_bytes");
    uint64_t *skey = (uint64_t *)ws;
    float *smax = (float *)(skey + n * Bw);
    float *ssum = smax + n;
    hipStream_t st = (hipStream_t)stream;
    prof_set_site(S_TOPK_LOGPROB);
    prof_begin(K_TOPK_LOGPROB, st);
    const int Vs = ((V + S - 1) / S + 7) & ~7;         // whole runs of eight
    const bool vec = V % 8 == 0 && (((uintptr_t)logits) & 15) == 0;
    auto *kernel = Vs <= 256 * 16 ? (vec ? k_topk_slices<16, true> : k_topk_slices<16, false>)     // half-filled slices: half the registers
                                  : (vec ? k_topk_slices<TOPK_EPT, true> : k_topk_slices<TOPK_EPT, false>);
    MOA_KLAUNCH(kernel, dim3((unsigned)n), dim3(256), 0, st, dtype == MOA_BF16 ? 1 : 0, logits, V, Vs, Bw, S, skey, smax, ssum);
    prof_end(st);
    if (hipGetLastError() != hipSuccess) return tree_fail(MOA_ERR_HIP, "topk_logprob: launch failed");
    const size_t lds = ((size_t)S * Bw + 7) / 8 * 8 * 8;
    if ((size_t)S * Bw * 8 + (size_t)S * 8 > 60 * 1024) return tree_fail(MOA_ERR_SHAPE, "topk_logprob: vocabulary too large for the merge");
    prof_begin(K_TOPK_MERGE, st);
    MOA_KLAUNCH(k_topk_merge, dim3(F), dim3(S * Bw <= 64 ? 256 : S * Bw <= 128 ? 512 : 1024), lds, st, Bw, S, skey, smax, ssum, tok, logp);
    prof_end(st);
    return hipGetLastError() == hipSuccess ? MOA_OK : tree_fail(MOA_ERR_HIP, "topk_logprob: launch failed");
}

}  // extern "C"
