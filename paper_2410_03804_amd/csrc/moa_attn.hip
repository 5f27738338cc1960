// Attention core shared by the draft model's cross-attention (no mask, cache rows only) and the
// tree-masked verification attention (cache rows, then the tree rows filtered by the ancestor
// bitset).  Input Q is already projected; the output is the concatenated heads before W_o.
//
//   k_attn_generic   any dtype / head_dim <= 256: one wavefront per (sequence, query, head),
//                    64 keys per step, exact online softmax with wavefront shuffles.
//   k_attn_f32       fp32, head_dim 64 / 128: 16 query rows per workgroup on the fp32 matrix instructions.
//   k_attn_fused     bf16, head_dim 64 / 128, short key ranges: a workgroup owns 32 query rows and the
//                    whole key range (its waves split the keys and are combined through LDS), so there
//                    are no partial results and no second launch.  Described at the kernel.
//   k_attn_mfma      bf16, head_dim 64 / 128, long key ranges: split-KV.  A workgroup owns one
//                    (sequence, KV head), one slice of the key range and up to 128*NBLK query rows (the
//                    GQA group's heads times the tree tokens are folded into the row dimension, so K/V
//                    are read once for all of them).  K/V tiles of 32 keys are staged row-major in LDS by
//                    row-contiguous 16-byte loads; scores are computed transposed (S^T = K Q^T) so that a
//                    lane owns one query column and the softmax max/sum need a single cross-lane
//                    exchange; P^T feeds the second MFMA straight from registers and V^T comes out of
//                    the LDS transpose read.
//   k_attn_long      the same split with 256 query rows per workgroup at head_dim 128, where that is faster (see
//                    split_geometry).  In moa_attn_long.hip.
//   k_attn_merge     combines the per-slice (max, sum, accumulator) triples.
#include "moa_attn_device.h"

#include <math.h>

#include <algorithm>
#include <atomic>

namespace moa {

// which MFMA form the attention core takes: 0 = chosen from the call's shape, 1 = whole key range per workgroup,
// 2 = split-KV + merge, 3 = that in 256-row tiles (moa_debug_force_attn_kernel; process-wide, read once per launch)
static std::atomic<int> g_attn_form{0};

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// ------------------------------------------------------------------ generic
template <typename T>
__global__ __launch_bounds__(64) void k_attn_generic(AttnArgs a)
{
    __shared__ float qs[256];
    const int lane = threadIdx.x;
    const int h = blockIdx.x % a.H;
    const int m = (blockIdx.x / a.H) % a.Mq;
    const int b = blockIdx.x / (a.H * a.Mq);
    const int g = h / (a.H / a.Hkv);
    const int dh = a.dh, W = (a.mask_rows + 63) >> 6;
    const float scale = 1.0f / sqrtf((float)dh);

    const T *q = (const T *)a.q + (((int64_t)b * a.Mq + m) * a.H + h) * dh;
    for (int c = lane; c < dh; c += 64) qs[c] = ld<T>(q + c);
    __syncthreads();

    const int len = clamp_len(a.len[b], a.P_cap, lane == 0 ? a.dev_status : nullptr);
    const int Mt = a.mask ? a.Mt : 0;
    const int total = len + Mt;
    const T *kc = (const T *)a.kcache + ((int64_t)b * a.Hkv + g) * (int64_t)a.P_cap * dh;
    const T *vc = (const T *)a.vcache + ((int64_t)b * a.Hkv + g) * (int64_t)a.P_cap * dh;
    const T *kt = (const T *)a.ktree + ((int64_t)b * a.Hkv + g) * (int64_t)a.tree_cap * dh;
    const T *vt = (const T *)a.vtree + ((int64_t)b * a.Hkv + g) * (int64_t)a.tree_cap * dh;
    const uint64_t *mrow = a.mask ? a.mask + ((int64_t)b * a.mask_rows + a.mask_row0 + m) * W : nullptr;

    float mrun = -INFINITY, lrun = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int base = 0; base < total; base += 64) {
        const int kidx = base + lane;
        float s = -INFINITY;
        if (kidx < total) {
            const T *krow = nullptr;
            if (kidx < len) {
                krow = kc + (int64_t)kidx * dh;
            } else {
                const int j = kidx - len;
                if ((mrow[j >> 6] >> (j & 63)) & 1) krow = kt + (int64_t)j * dh;
            }
            if (krow) {
                float d = 0.f;
                for (int c = 0; c < dh; ++c) d = fmaf(qs[c], ld<T>(krow + c), d);
                s = d * scale;
            }
        }
        const float mnew = fmaxf(mrun, wave_max(s));
        if (mnew == -INFINITY) continue;   // nothing visible yet (same decision in every lane)
        const float p = (s == -INFINITY) ? 0.f : expf(s - mnew);
        const float corr = expf(mrun - mnew);
        lrun = lrun * corr + wave_sum(p);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] *= corr;
        const int nk = min(64, total - base);
        for (int kk = 0; kk < nk; ++kk) {
            const float pk = __shfl(p, kk);
            if (pk == 0.f) continue;
            const int ki = base + kk;
            const T *vrow = ki < len ? vc + (int64_t)ki * dh : vt + (int64_t)(ki - len) * dh;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (lane + 64 * c < dh) acc[c] = fmaf(pk, ld<T>(vrow + lane + 64 * c), acc[c]);
        }
        mrun = mnew;
    }
    T *o = (T *)a.out + (((int64_t)b * a.Mq + m) * a.H + h) * dh;
    const float inv = lrun > 0.f ? 1.0f / lrun : 0.f;
    for (int c = 0; c < 4; ++c)
        if (lane + 64 * c < dh) st<T>(o + lane + 64 * c, acc[c] * inv);
    if (lrun == 0.f && a.empty_is_error && lane == 0 && a.dev_status) atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
}

// ------------------------------------------------------------------ MFMA split-KV
template <int DH, int NBLK, int CALLS>
__global__ __launch_bounds__(256, NBLK == 1 ? 2 : 1) void k_attn_mfma(AttnGroup<CALLS> grp, SplitGeom geo)
{
    const int call = blockIdx.z / grp.nbg;
    const AttnArgs &a = grp.a[call];
    f16_t *__restrict__ part_o = (f16_t *)a.ws;
    float *__restrict__ part_ml = (float *)(part_o + (size_t)grp.nbg * geo.nsplit * geo.rows_pad * DH);
    constexpr int KLD = DH + 8;           // padded K row (bf16): 16-byte operand reads of 16 rows hit 64 different banks
    constexpr int VSLD = DH + 32;         // padded V row: the 4 rows x 2 column groups of a transpose read hit different banks
    constexpr int NKS = DH / 16;          // MFMA steps along head_dim
    constexpr int NDB = DH / 32;          // 32-wide blocks of head_dim in the output
    constexpr int CPK = DH / 8;           // 16-byte chunks per key row
    constexpr int NLD = (KT * CPK) / 256; // chunks per thread per tile (1 for DH 64, 2 for DH 128)
    __shared__ __attribute__((aligned(16))) bf16_t Ks2[2][KT * KLD];    // two stages: one barrier per tile
    __shared__ __attribute__((aligned(16))) bf16_t Vs2[2][KT * VSLD];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int split = blockIdx.x, rowtile = blockIdx.y;
    const int bg = blockIdx.z - call * grp.nbg, b = bg / a.Hkv, g = bg % a.Hkv;
    const int G = a.H / a.Hkv, RG = G * a.Mq, W = (a.mask_rows + 63) >> 6;
    const float sc = 1.4426950408889634f / sqrtf((float)DH);   // scores are kept in the log2 domain

    const int len = clamp_len(a.len[b], a.P_cap, tid == 0 ? a.dev_status : nullptr);
    const int nt = (len + KT - 1) / KT;
    const int per = (nt + geo.nsplit - 1) / geo.nsplit;
    const int t0 = min(split * per, nt), t1 = min(t0 + per, nt);
    const int Mt = a.mask ? a.Mt : 0;
    const int ntree = (split == geo.nsplit - 1) ? (Mt + KT - 1) / KT : 0;
    const int ntiles = (t1 - t0) + ntree;

    const bf16_t *kc = (const bf16_t *)a.kcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *vc = (const bf16_t *)a.vcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *ktp = (const bf16_t *)a.ktree + (int64_t)bg * a.tree_cap * DH;
    const bf16_t *vtp = (const bf16_t *)a.vtree + (int64_t)bg * a.tree_cap * DH;

    // query fragments (B operand of S^T = K Q^T): lane = query column l32, 8 head_dim values
    const int rowbase = rowtile * (128 * NBLK) + wave * (32 * NBLK);
    bf16x8 qf[NBLK][NKS];
    int mrow_of[NBLK];
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
        int rho = rowbase + 32 * blk + l32;
        if (rho > RG - 1) rho = RG - 1;
        const int m = rho / G, hh = rho - m * G;
        mrow_of[blk] = m;
        const bf16_t *qrow = (const bf16_t *)a.q + (((int64_t)b * a.Mq + m) * a.H + g * G + hh) * DH;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[blk][ks] = *(const bf16x8 *)(qrow + 16 * ks + 8 * half);
    }

    f32x16 acc[NBLK][NDB];
    float mrun[NBLK], lrun[NBLK];
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
        mrun[blk] = -INFINITY;
        lrun[blk] = 0.f;
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[blk][d][e] = 0.f;
    }

    // tile i of this workgroup: cache tile t0+i, or tree tile i-(t1-t0).  K and V rows are fetched row-contiguously
    // (16 lanes cover a 256-byte row), staged row-major in LDS; V comes back transposed by the LDS transpose read.
    // A ring of RD register stages: the loads of tile i+RD are issued when tile i has been computed, so a tile has
    // RD-1 whole iterations to arrive (memory latency under load is longer than one iteration).
    constexpr int RD = 3;
    u32x4 kreg[RD][NLD], vreg[RD][NLD];
    auto full_tile = [&](int i) { return i < (t1 - t0) && (t0 + i + 1) * KT <= len; };
    auto fetch = [&](int i, u32x4 (&kr)[NLD], u32x4 (&vr)[NLD]) {
        if (full_tile(i)) {
            const int64_t off0 = (int64_t)(t0 + i) * KT * DH;
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                const int c = tid + 256 * j;
                kr[j] = *(const u32x4 *)(kc + off0 + (c / CPK) * DH + (c % CPK) * 8);
                vr[j] = *(const u32x4 *)(vc + off0 + (c / CPK) * DH + (c % CPK) * 8);
            }
            return;
        }
        const bool tree = i >= (t1 - t0);
        const int base = tree ? (i - (t1 - t0)) * KT : (t0 + i) * KT;
        const int limit = tree ? Mt : len;
        const bf16_t *ksrc = tree ? ktp : kc;
        const bf16_t *vsrc = tree ? vtp : vc;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int c = tid + 256 * j;
            int row = base + c / CPK;
            if (row > limit - 1) row = limit - 1;          // rows past the end repeat the last valid row
            kr[j] = *(const u32x4 *)(ksrc + (int64_t)row * DH + (c % CPK) * 8);
            vr[j] = *(const u32x4 *)(vsrc + (int64_t)row * DH + (c % CPK) * 8);
        }
    };
    auto stage = [&](int buf, const u32x4 (&kr)[NLD], const u32x4 (&vr)[NLD]) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int c = tid + 256 * j;
            *(u32x4 *)&Ks2[buf][(c / CPK) * KLD + (c % CPK) * 8] = kr[j];
            *(u32x4 *)&Vs2[buf][(c / CPK) * VSLD + (c % CPK) * 8] = vr[j];
        }
    };
    // transpose read: lane j of a 16-lane group addresses key (j >> 2), head_dim 4 (j & 3) of the group's 16
    const int tr_off = ((lane & 15) >> 2) * VSLD + 16 * ((lane >> 4) & 1) + 4 * (lane & 3) + 4 * half * VSLD;

    // Tile i+1 is staged into the other LDS buffer after tile i has been computed; the barrier at the end of an
    // iteration publishes it and retires the reads of tile i.  Three iterations per trip so that the register
    // stages are addressed statically.
#pragma unroll
    for (int d = 0; d < RD; ++d)
        if (d < ntiles) fetch(d, kreg[d], vreg[d]);
    if (ntiles > 0) stage(0, kreg[0], vreg[0]);
    __syncthreads();
    for (int i0 = 0; i0 < ntiles; i0 += RD) {
#pragma unroll
    for (int d = 0; d < RD; ++d) {
        const int i = i0 + d;
        if (i >= ntiles) continue;                             // same decision in the whole workgroup
        const bf16_t *Ks = Ks2[i & 1], *Vs = Vs2[i & 1];

        // S^T tile: keys x queries
        f32x16 s[NBLK];
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
            for (int e = 0; e < 16; ++e) s[blk][e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const bf16x8 kf = *(const bf16x8 *)&Ks[l32 * KLD + 16 * ks + 8 * half];
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk)
                s[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[blk][ks], s[blk], 0, 0, 0);
        }

        // keys that do not count (tree rows outside the ancestor set, rows past the end) get -inf; a cache tile
        // wholly below the length has none (the decision is the same for the whole workgroup)
        if (!full_tile(i)) {
            const bool tree = i >= (t1 - t0);
            const int base = tree ? (i - (t1 - t0)) * KT : (t0 + i) * KT;
            const int nvalid = (tree ? Mt : len) - base;       // >= 1
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk) {
                uint32_t vis = 0xffffffffu;
                if (tree) vis = (uint32_t)(a.mask[((int64_t)b * a.mask_rows + a.mask_row0 + mrow_of[blk]) * W + (base >> 6)] >> (base & 63));
                if (nvalid < 32) vis &= (1u << nvalid) - 1u;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = 8 * (v >> 2) + 4 * half + (v & 3);
                    if (!((vis >> key) & 1u)) s[blk][v] = -INFINITY;
                }
            }
        }

        bf16x8 pf[NBLK][2];
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk) {
            float tmax = s[blk][0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[blk][v]);
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            const float mnew = fmaxf(mrun[blk], tmax * sc);    // sc > 0: scaling keeps the order (and -inf)
            const float msafe = (mnew == -INFINITY) ? 0.f : mnew;
            const float corr = fast_exp2(mrun[blk] - msafe);
            float psum = 0.f;
            float p[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) { p[v] = fast_exp2(fmaf(s[blk][v], sc, -msafe)); psum += p[v]; }
            psum += __shfl_xor(psum, 32);
            lrun[blk] = lrun[blk] * corr + psum;
            mrun[blk] = mnew;
            if (__any(corr != 1.0f)) {                          // the running max moved in some column
                asm volatile("" ::: "memory");                  // keep this a real branch: the multiplies are skipped
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[blk][d][e] *= corr;
            }
#pragma unroll
            for (int st2 = 0; st2 < 2; ++st2)
#pragma unroll
                for (int t = 0; t < 8; ++t) pf[blk][st2][t] = (__bf16)p[8 * st2 + t];
        }

        // O^T += V^T P^T; P^T slot t of step st2 is key 16 st2 + 8 (t >> 2) + 4 half + (t & 3)
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int st2 = 0; st2 < 2; ++st2) {
                const bf16_t *vp = Vs + tr_off + 16 * st2 * VSLD + 32 * d;
                union { i16x4 h[2]; bf16x8 v; } vf;
                vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)vp);
                vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(vp + 8 * VSLD));
#pragma unroll
                for (int blk = 0; blk < NBLK; ++blk)
                    acc[blk][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pf[blk][st2], acc[blk][d], 0, 0, 0);
            }
        if (i + 1 < ntiles) stage((i + 1) & 1, kreg[(d + 1) % RD], vreg[(d + 1) % RD]);
        if (i + RD < ntiles) fetch(i + RD, kreg[d], vreg[d]);
        __syncthreads();
    }
    }

    // partial results of this slice: the slice's own normalised output (a convex combination of V rows, so it
    // fits fp16 with 2^-12 relative rounding, eight times finer than the bf16 result), running max (log2 domain)
    // and running sum in fp32
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
        const int rho = rowbase + 32 * blk + l32;
        if (rho >= RG) continue;
        const int64_t prow = ((int64_t)bg * geo.nsplit + split) * geo.rows_pad + rho;
        if (half == 0) {
            part_ml[prow * 2 + 0] = mrun[blk];
            part_ml[prow * 2 + 1] = lrun[blk];
        }
        const float inv = lrun[blk] > 0.f ? 1.0f / lrun[blk] : 0.f;
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

// ------------------------------------------------------------------ MFMA, whole key range in one workgroup
// One workgroup owns 32 query rows of one (sequence, KV head) and ALL of its keys: wave w takes the key tiles
// w, w + NW, ... with its own running (max, sum, accumulator), and the NW triples are combined through LDS at
// the end, in wave order, so no partial results go through HBM and no merge kernel follows.  The key loop has
// no workgroup barrier: each wave stages its tiles in a private LDS buffer.
//  - Global loads are row-contiguous (16 lanes cover 256 B): the memory pipeline handles one cache line per
//    lane group per clock, so loads in which every lane touches its own line run at a quarter of the rate.
//  - K goes to LDS row-major and comes back as MFMA operands (lane = key, 8 head_dim values).
//  - V goes to LDS row-major too and comes back TRANSPOSED by the LDS transpose read (within 16 lanes, lane i
//    receives element i%4 of the 8-byte datum addressed by lane i/4 + 4t, t = 0..3): the 16 lanes address 4
//    keys x 16 head_dim values, and lane i ends up with head_dim i for the 4 keys, which is the operand layout
//    of O^T += V^T P^T.  Two such reads (keys +0..3 and +8..11 of the lane's half) give the 8 keys that match
//    the key order of P^T in the score registers.
// Every row block re-reads the (sequence, KV head)'s K/V, which is why this form is used for short key ranges
// only; the blocks that share K/V are placed on the same XCD so that the re-reads hit its L2.
__device__ __forceinline__ void wave_lds_sync()
{
    // LDS traffic of one wavefront is processed in order; this only keeps the compiler from moving a read of
    // another lane's data above the write that produced it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int DH, int NW>
struct FusedLds {
    static constexpr int KLD = DH + 8;    // K / Q row (bf16): 16-byte operand reads of 16 rows hit 64 different banks
    static constexpr int VSLD = DH + 32;  // V row: the 4 rows x 2 column groups of a transpose read hit different banks
    static constexpr int NV = (DH / 32) * 16;
    static constexpr size_t q_bytes = (size_t)32 * KLD * sizeof(bf16_t);
    static constexpr size_t stage_bytes = (size_t)32 * VSLD * sizeof(bf16_t);
    static constexpr size_t loop_bytes = q_bytes + NW * stage_bytes;
    static constexpr size_t merge_bytes = ((size_t)NW * NV * 64 + 2 * NW * 32) * sizeof(float);
    static constexpr size_t bytes = loop_bytes > merge_bytes ? loop_bytes : merge_bytes;
};

template <int DH, int NW, int CALLS>
__global__ __launch_bounds__(64 * NW) void k_attn_fused(AttnGroup<CALLS> grp)
{
    const int nrb = grp.nrb;
    using L = FusedLds<DH, NW>;
    constexpr int KLD = L::KLD, VSLD = L::VSLD;
    constexpr int NKS = DH / 16;          // MFMA steps along head_dim
    constexpr int NDB = DH / 32;          // 32-wide blocks of head_dim in the output
    constexpr int CPK = DH / 8;           // 16-byte pieces per row
    constexpr int RPI = 64 / CPK;         // rows covered by one load instruction of the wave
    constexpr int NLD = KT / RPI;         // load instructions per tile
    constexpr int NV = L::NV;             // accumulator values per lane
    constexpr int VPW = NV / NW;          // accumulator values each wave finalises
    static_assert(VPW % 4 == 0, "finalisation stores four head_dim values at a time");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    // workgroup -> (unit, row block): the hardware deals consecutive workgroups round-robin to the 8 XCDs
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int u = xcd + 8 * (slot / nrb), rb = slot - (slot / nrb) * nrb;
    if (u >= grp.ncalls * grp.nbg) return;          // the whole workgroup leaves before any barrier
    const int call = u / grp.nbg, bg = u - call * grp.nbg;
    const AttnArgs &a = grp.a[call];
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    const int G = a.H / a.Hkv, RG = G * a.Mq, W = (a.mask_rows + 63) >> 6;
    const float sc = 1.4426950408889634f / sqrtf((float)DH);   // scores are kept in the log2 domain

    // the block's 32 query rows: requested first (they do not depend on the sequence length), row-contiguous
    constexpr int QPT = (32 * CPK + 64 * NW - 1) / (64 * NW);
    u32x4 qreg[QPT];
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int c = min(tid + 64 * NW * i, 32 * CPK - 1);
        int rq = rb * 32 + c / CPK;
        if (rq > RG - 1) rq = RG - 1;
        const int m = rq / G, hq = rq - m * G;
        const bf16_t *qrow = (const bf16_t *)a.q + (((int64_t)b * a.Mq + m) * a.H + g * G + hq) * DH;
        qreg[i] = *(const u32x4 *)(qrow + 8 * (c % CPK));
    }

    const int len = clamp_len(a.len[b], a.P_cap, tid == 0 ? a.dev_status : nullptr);
    const int Mt = a.mask ? a.Mt : 0;
    const int ntc = (len + KT - 1) / KT, nt = ntc + (Mt + KT - 1) / KT;

    const bf16_t *kc = (const bf16_t *)a.kcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *vc = (const bf16_t *)a.vcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *ktp = (const bf16_t *)a.ktree + (int64_t)bg * a.tree_cap * DH;
    const bf16_t *vtp = (const bf16_t *)a.vtree + (int64_t)bg * a.tree_cap * DH;

    // the K/V tile as the wave loads it: instruction j covers rows RPI j .. RPI j + RPI - 1, 16 bytes per lane.
    // A cache tile that lies wholly below the length needs no row clamp: one base address, constant offsets.
    const int ld_row = lane / CPK, ld_piece = lane % CPK;
    const int ld_off = ld_row * DH + 8 * ld_piece;
    u32x4 kreg[NLD], vreg[NLD];
    auto fetch = [&](int i) {
        if (i < ntc && (i + 1) * KT <= len) {
            const bf16_t *kp = kc + (int64_t)i * KT * DH + ld_off, *vp = vc + (int64_t)i * KT * DH + ld_off;
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                kreg[j] = *(const u32x4 *)(kp + j * RPI * DH);
                vreg[j] = *(const u32x4 *)(vp + j * RPI * DH);
            }
            return;
        }
        const bool tree = i >= ntc;
        const int base = tree ? (i - ntc) * KT : i * KT;
        const int limit = tree ? Mt : len;
        const bf16_t *ksrc = tree ? ktp : kc;
        const bf16_t *vsrc = tree ? vtp : vc;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            int row = base + RPI * j + ld_row;
            if (row > limit - 1) row = limit - 1;              // rows past the end repeat the last valid row
            const int64_t off = (int64_t)row * DH + 8 * ld_piece;
            kreg[j] = *(const u32x4 *)(ksrc + off);
            vreg[j] = *(const u32x4 *)(vsrc + off);
        }
    };
    if (wave < nt) fetch(wave);

    bf16_t *Qs = (bf16_t *)smem;
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int c = tid + 64 * NW * i;
        if (c < 32 * CPK) *(u32x4 *)&Qs[(c / CPK) * KLD + 8 * (c % CPK)] = qreg[i];
    }
    __syncthreads();
    bf16x8 qf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)&Qs[l32 * KLD + 16 * ks + 8 * half];

    int rho = rb * 32 + l32;                        // this lane's query column
    const bool row_ok = rho < RG;
    if (!row_ok) rho = RG - 1;
    const int mrow = rho / G, hh = rho - mrow * G;

    f32x16 acc[NDB];
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[d][e] = 0.f;
    float mrun = -INFINITY, lrun = 0.f;              // running max (scaled, log2 domain) and sum

    bf16_t *stg = (bf16_t *)(smem + L::q_bytes + wave * L::stage_bytes);   // this wave's tile buffer
    // transpose read: lane j of a 16-lane group addresses key (j >> 2), head_dim 4 (j & 3) of the group's 16
    const int tr_off = ((lane & 15) >> 2) * VSLD + 16 * ((lane >> 4) & 1) + 4 * (lane & 3) + 4 * half * VSLD;

    if (wave < nt) {
        const int last = wave + ((nt - 1 - wave) / NW) * NW;
        for (int i = wave; i <= last; i += NW) {
            // K tile -> LDS -> S^T = K Q^T (keys x queries)
#pragma unroll
            for (int j = 0; j < NLD; ++j) *(u32x4 *)&stg[(RPI * j + ld_row) * KLD + 8 * ld_piece] = kreg[j];
            wave_lds_sync();
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const bf16x8 kf = *(const bf16x8 *)&stg[l32 * KLD + 16 * ks + 8 * half];
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s, 0, 0, 0);
            }
            wave_lds_sync();
            // V tile into the same buffer, then the next tile's loads (clamped to the wave's last tile: a
            // repeated load of valid memory whose result is not used) fly during the softmax and the second MFMA
#pragma unroll
            for (int j = 0; j < NLD; ++j) *(u32x4 *)&stg[(RPI * j + ld_row) * VSLD + 8 * ld_piece] = vreg[j];
            wave_lds_sync();
            fetch(min(i + NW, last));

            // keys that do not count (tree rows outside the ancestor set, rows past the end) get -inf; a cache
            // tile wholly below the length has none (the decision is the same for the whole wavefront)
            if (!(i < ntc && (i + 1) * KT <= len)) {
                const bool tree = i >= ntc;
                const int base = tree ? (i - ntc) * KT : i * KT;
                const int nvalid = (tree ? Mt : len) - base;   // >= 1
                uint32_t vis = 0xffffffffu;
                if (tree) vis = (uint32_t)(a.mask[((int64_t)b * a.mask_rows + a.mask_row0 + mrow) * W + (base >> 6)] >> (base & 63));
                if (nvalid < 32) vis &= (1u << nvalid) - 1u;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = 8 * (v >> 2) + 4 * half + (v & 3);
                    if (!((vis >> key) & 1u)) s[v] = -INFINITY;
                }
            }
            float tmax = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            const float mnew = fmaxf(mrun, tmax * sc);         // sc > 0: scaling keeps the order (and -inf)
            const float msafe = (mnew == -INFINITY) ? 0.f : mnew;
            const float corr = fast_exp2(mrun - msafe);
            float psum = 0.f;
            float p[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) { p[v] = fast_exp2(fmaf(s[v], sc, -msafe)); psum += p[v]; }
            psum += __shfl_xor(psum, 32);
            lrun = lrun * corr + psum;
            mrun = mnew;
            if (__any(corr != 1.0f)) {                          // the running max moved in some column
                asm volatile("" ::: "memory");                  // keep this a real branch: 64 multiplies skipped
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[d][e] *= corr;
            }
            // O^T += V^T P^T; P^T slot t of step st2 is key 16 st2 + 8 (t >> 2) + 4 half + (t & 3)
#pragma unroll
            for (int st2 = 0; st2 < 2; ++st2) {
                bf16x8 pf;
#pragma unroll
                for (int t = 0; t < 8; ++t) pf[t] = (__bf16)p[8 * st2 + t];
#pragma unroll
                for (int d = 0; d < NDB; ++d) {
                    const bf16_t *vp = stg + tr_off + 16 * st2 * VSLD + 32 * d;
                    union { i16x4 h[2]; bf16x8 v; } vf;
                    vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)vp);
                    vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(vp + 8 * VSLD));
                    acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pf, acc[d], 0, 0, 0);
                }
            }
            wave_lds_sync();
        }
    }

    // combine the waves' triples: out = sum_w 2^(m_w - m*) acc_w / sum_w 2^(m_w - m*) l_w, waves in order
    __syncthreads();                                            // the tile buffers are dead; their memory is reused
    float *red = (float *)smem;                                 // [NW][NV][64]
    float *msh = red + NW * NV * 64;                            // [NW][32]
    float *lsh = msh + NW * 32;
    if (half == 0) {
        msh[wave * 32 + l32] = mrun;
        lsh[wave * 32 + l32] = lrun;
    }
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) red[((wave * NDB + d) * 16 + e) * 64 + lane] = acc[d][e];
    __syncthreads();

    float wgt[NW], mstar = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { wgt[w] = msh[w * 32 + l32]; mstar = fmaxf(mstar, wgt[w]); }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wgt[w] = (wgt[w] == -INFINITY) ? 0.f : exp2f(wgt[w] - mstar);
        lsum += wgt[w] * lsh[w * 32 + l32];
    }
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    bf16_t *orow = (bf16_t *)a.out + (((int64_t)b * a.Mq + mrow) * a.H + g * G + hh) * DH;
#pragma unroll
    for (int t4 = 0; t4 < VPW / 4; ++t4) {
        const int v0 = wave * VPW + 4 * t4;                     // accumulator values v0 .. v0+3: four consecutive head_dim
        float o[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += wgt[w] * red[(w * NV + v0 + t) * 64 + lane];
            o[t] = sum * inv;
        }
        const int dcol = 32 * (v0 >> 4) + 8 * ((v0 & 15) >> 2) + 4 * half;
        if (row_ok) {
            u32x2 pk;
            pk[0] = pack_bf16x2(o[0], o[1]);
            pk[1] = pack_bf16x2(o[2], o[3]);
            *(u32x2 *)(orow + dcol) = pk;
        }
    }
    if (wave == 0 && half == 0 && row_ok && lsum == 0.f && a.empty_is_error && a.dev_status)
        atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
}

// The same in blocks of 16 query rows, for calls that would leave much of the chip idle in blocks of 32: twice the workgroups, each
// with half the arithmetic per key (it reads as many keys).  One MFMA 16x16x32 takes the place of two 32x32x16 along the same
// products, a lane has the same keys' scores in the same slots, and sums are made in the same order, so the two forms give the
// same bits and a call may take either.  (Score slots of lane quarter q: keys 16 (q / 2) + 8 b + 4 (q % 2) + v of a tile, b = 0, 1.  The K
// rows are put into LDS so that the 16 that an operand read touches follow one another, and V rows are 16 longer than head_dim: the
// four quarters' transpose reads hit different banks.)  One sequence of 60 nodes x 1024 keys, 8 KV heads:
// 11.9 -> 11.0 us; 8 nodes 11.4 -> 10.4; 8 x 16 x 3000 35.6 -> 32.5.
template <int DH, int NW>
struct Fused16Lds {
    static constexpr int KLD = DH + 8, VSLD = DH + 16, NV = DH / 4;
    static constexpr size_t q_bytes = (size_t)16 * KLD * sizeof(bf16_t);
    static constexpr size_t stage_bytes = (size_t)32 * VSLD * sizeof(bf16_t);
    static constexpr size_t loop_bytes = q_bytes + NW * stage_bytes;
    static constexpr size_t merge_bytes = ((size_t)NW * NV * 64 + 2 * NW * 16) * sizeof(float);
    static constexpr size_t bytes = loop_bytes > merge_bytes ? loop_bytes : merge_bytes;
};

template <int DH, int NW, int CALLS>
__global__ __launch_bounds__(64 * NW) void k_attn_fused16(AttnGroup<CALLS> grp)
{
    const int nrb = grp.nrb;
    using L = Fused16Lds<DH, NW>;
    constexpr int KLD = L::KLD, VSLD = L::VSLD;
    constexpr int NKS = DH / 32;          // MFMA steps along head_dim
    constexpr int NDB = DH / 16;          // 16-wide blocks of head_dim in the output
    constexpr int CPK = DH / 8;           // 16-byte pieces per row
    constexpr int RPI = 64 / CPK;         // rows covered by one load instruction of the wave
    constexpr int NLD = KT / RPI;         // load instructions per tile
    constexpr int NV = L::NV;             // accumulator values per lane
    static_assert(RPI == 4 && NV == 4 * NW, "K rows are placed by fours; each wave finalises one block of head_dim");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, quart = lane >> 4;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int u = xcd + 8 * (slot / nrb), rb = slot - (slot / nrb) * nrb;
    if (u >= grp.ncalls * grp.nbg) return;          // the whole workgroup leaves before any barrier
    const int call = u / grp.nbg, bg = u - call * grp.nbg;
    const AttnArgs &a = grp.a[call];
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    const int G = a.H / a.Hkv, RG = G * a.Mq, W = (a.mask_rows + 63) >> 6;
    const float sc = 1.4426950408889634f / sqrtf((float)DH);   // scores are kept in the log2 domain

    u32x4 qreg;
    {
        const int c = min(tid, 16 * CPK - 1);
        const int rq = min(rb * 16 + c / CPK, RG - 1), m = rq / G, hq = rq - m * G;
        qreg = *(const u32x4 *)((const bf16_t *)a.q + (((int64_t)b * a.Mq + m) * a.H + g * G + hq) * DH + 8 * (c % CPK));
    }

    const int len = clamp_len(a.len[b], a.P_cap, tid == 0 ? a.dev_status : nullptr);
    const int Mt = a.mask ? a.Mt : 0;
    const int ntc = (len + KT - 1) / KT, nt = ntc + (Mt + KT - 1) / KT;

    const bf16_t *kc = (const bf16_t *)a.kcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *vc = (const bf16_t *)a.vcache + (int64_t)bg * a.P_cap * DH;
    const bf16_t *ktp = (const bf16_t *)a.ktree + (int64_t)bg * a.tree_cap * DH;
    const bf16_t *vtp = (const bf16_t *)a.vtree + (int64_t)bg * a.tree_cap * DH;

    const int ld_row = lane / CPK, ld_piece = lane % CPK;
    const int ld_off = ld_row * DH + 8 * ld_piece;
    u32x4 kreg[NLD], vreg[NLD];
    auto fetch = [&](int i) {
        if (i < ntc && (i + 1) * KT <= len) {
            const bf16_t *kp = kc + (int64_t)i * KT * DH + ld_off, *vp = vc + (int64_t)i * KT * DH + ld_off;
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                kreg[j] = *(const u32x4 *)(kp + j * RPI * DH);
                vreg[j] = *(const u32x4 *)(vp + j * RPI * DH);
            }
            return;
        }
        const bool tree = i >= ntc;
        const int base = tree ? (i - ntc) * KT : i * KT;
        const int limit = tree ? Mt : len;
        const bf16_t *ksrc = tree ? ktp : kc;
        const bf16_t *vsrc = tree ? vtp : vc;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            int row = base + RPI * j + ld_row;
            if (row > limit - 1) row = limit - 1;              // rows past the end repeat the last valid row
            const int64_t off = (int64_t)row * DH + 8 * ld_piece;
            kreg[j] = *(const u32x4 *)(ksrc + off);
            vreg[j] = *(const u32x4 *)(vsrc + off);
        }
    };
    if (wave < nt) fetch(wave);

    bf16_t *Qs = (bf16_t *)smem;
    if (tid < 16 * CPK) *(u32x4 *)&Qs[(tid / CPK) * KLD + 8 * (tid % CPK)] = qreg;
    __syncthreads();
    bf16x8 qf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)&Qs[l16 * KLD + 32 * ks + 8 * quart];

    int rho = rb * 16 + l16;                        // this lane's query column
    const bool row_ok = rho < RG;
    if (!row_ok) rho = RG - 1;
    const int mrow = rho / G, hh = rho - mrow * G;

    f32x4 acc[NDB];
#pragma unroll
    for (int d = 0; d < NDB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f;              // running max (scaled, log2 domain) and sum

    bf16_t *stg = (bf16_t *)(smem + L::q_bytes + wave * L::stage_bytes);   // this wave's tile buffer
    // transpose read: lane j of a 16-lane group addresses key (j >> 2) of the quarter's four, head_dim 4 (j & 3) of the block's 16
    const int key0 = 16 * (quart >> 1) + 4 * (quart & 1);              // the quarter's keys: key0 .. + 3 and eight further on
    const int tr_off = (key0 + (l16 >> 2)) * VSLD + 4 * (l16 & 3);

    if (wave < nt) {
        const int last = wave + ((nt - 1 - wave) / NW) * NW;
        for (int i = wave; i <= last; i += NW) {
            // K tile -> LDS (row bits 3 and 4 change places) -> S^T = K Q^T (keys x queries)
#pragma unroll
            for (int j = 0; j < NLD; ++j) *(u32x4 *)&stg[(RPI * ((j & 1) | (j & 2) << 1 | (j & 4) >> 1) + ld_row) * KLD + 8 * ld_piece] = kreg[j];
            wave_lds_sync();
            f32x4 s[2];
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                s[blk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    const bf16x8 kf = *(const bf16x8 *)&stg[(16 * blk + l16) * KLD + 32 * ks + 8 * quart];
                    s[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[ks], s[blk], 0, 0, 0);
                }
            }
            wave_lds_sync();
            // V tile into the same buffer, then the next tile's loads (clamped to the wave's last tile: a
            // repeated load of valid memory whose result is not used) fly during the softmax and the second MFMA
#pragma unroll
            for (int j = 0; j < NLD; ++j) *(u32x4 *)&stg[(RPI * j + ld_row) * VSLD + 8 * ld_piece] = vreg[j];
            wave_lds_sync();
            fetch(min(i + NW, last));

            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = s[e >> 2][e & 3];
            // keys that do not count (tree rows outside the ancestor set, rows past the end) get -inf; a cache
            // tile wholly below the length has none (the decision is the same for the whole wavefront)
            if (!(i < ntc && (i + 1) * KT <= len)) {
                const bool tree = i >= ntc;
                const int base = tree ? (i - ntc) * KT : i * KT;
                const int nvalid = (tree ? Mt : len) - base;   // >= 1
                uint32_t vis = 0xffffffffu;
                if (tree) vis = (uint32_t)(a.mask[((int64_t)b * a.mask_rows + a.mask_row0 + mrow) * W + (base >> 6)] >> (base & 63));
                if (nvalid < 32) vis &= (1u << nvalid) - 1u;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!((vis >> (key0 + 8 * (e >> 2) + (e & 3))) & 1u)) p[e] = -INFINITY;
            }
            float tmax = p[0];
#pragma unroll
            for (int e = 1; e < 8; ++e) tmax = fmaxf(tmax, p[e]);
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            const float mnew = fmaxf(mrun, tmax * sc);         // sc > 0: scaling keeps the order (and -inf)
            const float msafe = (mnew == -INFINITY) ? 0.f : mnew;
            const float corr = fast_exp2(mrun - msafe);
            float lower = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) { p[e] = fast_exp2(fmaf(p[e], sc, -msafe)); lower += p[e]; }
            // one chain over keys 0 .. 3, 8 .. 11, 16 .. 19, 24 .. 27 (and one over the others): the upper quarters go on where the lower ones ended
            float psum = __shfl_xor(lower, 32);
#pragma unroll
            for (int e = 0; e < 8; ++e) psum += p[e];
            const float upper = __shfl_xor(psum, 32);
            if (quart < 2) psum = upper;
            psum += __shfl_xor(psum, 16);
            lrun = lrun * corr + psum;
            mrun = mnew;
            if (__any(corr != 1.0f)) {                          // the running max moved in some column
                asm volatile("" ::: "memory");                  // keep this a real branch: the multiplies are skipped
#pragma unroll
                for (int d = 0; d < NDB; ++d) acc[d] *= corr;
            }
            // O^T += V^T P^T; P^T slot t of the quarter is key key0 + 8 (t >> 2) + (t & 3)
            bf16x8 pf;
#pragma unroll
            for (int t = 0; t < 8; ++t) pf[t] = (__bf16)p[t];
#pragma unroll
            for (int d = 0; d < NDB; ++d) {
                const bf16_t *vp = stg + tr_off + 16 * d;
                union { i16x4 h[2]; bf16x8 v; } vf;
                vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)vp);
                vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(vp + 8 * VSLD));
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf, acc[d], 0, 0, 0);
            }
            wave_lds_sync();
        }
    }

    // combine the waves' triples: out = sum_w 2^(m_w - m*) acc_w / sum_w 2^(m_w - m*) l_w, waves in order
    __syncthreads();                                            // the tile buffers are dead; their memory is reused
    float *red = (float *)smem;                                 // [NW][NV][64]
    float *msh = red + NW * NV * 64;                            // [NW][16]
    float *lsh = msh + NW * 16;
    if (quart == 0) {
        msh[wave * 16 + l16] = mrun;
        lsh[wave * 16 + l16] = lrun;
    }
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(wave * NV + 4 * d + v) * 64 + lane] = acc[d][v];
    __syncthreads();

    float wgt[NW], mstar = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { wgt[w] = msh[w * 16 + l16]; mstar = fmaxf(mstar, wgt[w]); }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wgt[w] = (wgt[w] == -INFINITY) ? 0.f : exp2f(wgt[w] - mstar);
        lsum += wgt[w] * lsh[w * 16 + l16];
    }
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    float o[4];                                                 // head_dim 16 wave + 4 quart ..
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += wgt[w] * red[(w * NV + 4 * wave + t) * 64 + lane];
        o[t] = sum * inv;
    }
    if (row_ok) {
        u32x2 pk;
        pk[0] = pack_bf16x2(o[0], o[1]);
        pk[1] = pack_bf16x2(o[2], o[3]);
        *(u32x2 *)((bf16_t *)a.out + (((int64_t)b * a.Mq + mrow) * a.H + g * G + hh) * DH + 16 * wave + 4 * quart) = pk;
    }
    if (wave == 0 && quart == 0 && row_ok && lsum == 0.f && a.empty_is_error && a.dev_status)
        atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
}

// ------------------------------------------------------------------ fp32, whole key range in one workgroup
// One workgroup owns 16 query rows of one (sequence, KV head) -- heads of the group times tree tokens, as above -- and
// all of its keys; wavefront w takes the 16-key tiles w, w + 8, ... and the eight (max, sum, accumulator) triples are
// combined through LDS in wavefront order.  Everything is v_mfma_f32_16x16x4 (fp32 products and sums): S^T = K Q^T puts a
// query in each lane column, and its result layout (lane (li, kg) holds keys 4 kg .. 4 kg + 3 of query li) is the operand
// layout of O^T += V^T P^T with key 4 kg + j in slot j, so the probabilities never leave their registers.  K and V come
// straight from global memory, the next tile's behind this tile's arithmetic.  At the sizes fp32 is used at it is bound by
// latency: one workgroup's chain is the launch.  It replaced k_attn_generic there (a serial dot product per lane and a
// shuffle per key: 20 us per core at 16 rows x 72 keys x 64).
constexpr int F32_NW = 8;

template <int DH>
constexpr size_t attn_f32_lds() { return ((size_t)F32_NW * (DH / 4) * 64 + 2 * F32_NW * 16) * sizeof(float); }

template <int DH, int CALLS>
__global__ __launch_bounds__(64 * F32_NW) void k_attn_f32(AttnGroup<CALLS> grp)
{
    const int nrb = grp.nrb;
    constexpr int NW = F32_NW, NKS = DH / 16, NDB = DH / 16, NV = 4 * NDB, VPW = NV / NW;
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, kg = lane >> 4;
    const int u = (int)blockIdx.x / nrb, rb = (int)blockIdx.x - u * nrb;
    const int call = u / grp.nbg, bg = u - call * grp.nbg;
    const AttnArgs &a = grp.a[call];
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    const int G = a.H / a.Hkv, RG = G * a.Mq, W = (a.mask_rows + 63) >> 6;
    const float scale = 1.0f / sqrtf((float)DH);

    int rho = rb * 16 + li;                          // this lane's query column
    const bool row_ok = rho < RG;
    if (!row_ok) rho = RG - 1;
    const int mrow = rho / G, hh = rho - mrow * G;
    const int64_t qoff = (((int64_t)b * a.Mq + mrow) * a.H + g * G + hh) * DH;
    f32x4 qf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const f32x4 *)((const float *)a.q + qoff + 16 * ks + 4 * kg);

    const int len = clamp_len(a.len[b], a.P_cap, tid == 0 ? a.dev_status : nullptr);
    const int Mt = a.mask ? a.Mt : 0;
    const int ntc = (len + 15) / 16, nt = ntc + (Mt + 15) / 16;
    const float *kc = (const float *)a.kcache + (int64_t)bg * a.P_cap * DH, *vc = (const float *)a.vcache + (int64_t)bg * a.P_cap * DH;
    const float *ktp = (const float *)a.ktree + (int64_t)bg * a.tree_cap * DH, *vtp = (const float *)a.vtree + (int64_t)bg * a.tree_cap * DH;
    const uint64_t *mbits = a.mask ? a.mask + ((int64_t)b * a.mask_rows + a.mask_row0 + mrow) * W : nullptr;

    f32x4 kf[2][NKS];
    float vf[2][NDB][4];
    auto fetch = [&](int set, int i) {
        const bool tree = i >= ntc;
        const int base = 16 * (tree ? i - ntc : i), last = (tree ? Mt : len) - 1;
        const float *ks_ = tree ? ktp : kc, *vs_ = tree ? vtp : vc;
        const float *kp = ks_ + (int64_t)min(base + li, last) * DH + 4 * kg;      // rows past the end repeat the last one
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) kf[set][ks] = *(const f32x4 *)(kp + 16 * ks);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float *vp = vs_ + (int64_t)min(base + 4 * kg + j, last) * DH + li;
#pragma unroll
            for (int d = 0; d < NDB; ++d) vf[set][d][j] = vp[16 * d];
        }
    };
    f32x4 acc[NDB];
#pragma unroll
    for (int d = 0; d < NDB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f;
    auto tile = [&](int set, int i) {
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[set][ks][j], qf[ks][j], s, 0, 0, 0);
        const bool tree = i >= ntc;
        const int base = 16 * (tree ? i - ntc : i), nvalid = (tree ? Mt : len) - base;     // >= 1
        uint32_t vis = 0xffffu;
        if (tree) vis &= (uint32_t)(mbits[base >> 6] >> (base & 63));
        if (nvalid < 16) vis &= (1u << nvalid) - 1u;
        float tmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            s[v] = ((vis >> (4 * kg + v)) & 1u) ? s[v] * scale : -INFINITY;
            tmax = fmaxf(tmax, s[v]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        const float mnew = fmaxf(mrun, tmax), msafe = (mnew == -INFINITY) ? 0.f : mnew;
        const float corr = expf(mrun - msafe);
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) { s[v] = expf(s[v] - msafe); psum += s[v]; }
        psum += __shfl_xor(psum, 16);
        psum += __shfl_xor(psum, 32);
        lrun = lrun * corr + psum;
        mrun = mnew;
#pragma unroll
        for (int d = 0; d < NDB; ++d) {
            acc[d] *= corr;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[set][d][j], s[j], acc[d], 0, 0, 0);
        }
    };
    if (wave < nt) {
        fetch(0, wave);
        for (int i = wave; i < nt; i += 2 * NW) {
            if (i + NW < nt) fetch(1, i + NW);
            tile(0, i);
            if (i + NW >= nt) break;
            if (i + 2 * NW < nt) fetch(0, i + 2 * NW);
            tile(1, i + NW);
        }
    }

    float *red = fsm, *msh = red + NW * NV * 64, *lsh = msh + NW * 16;       // [NW][NV][64], [NW][16] twice
    if (kg == 0) {
        msh[wave * 16 + li] = mrun;
        lsh[wave * 16 + li] = lrun;
    }
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(wave * NV + 4 * d + v) * 64 + lane] = acc[d][v];
    __syncthreads();
    float wgt[NW], mstar = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { wgt[w] = msh[w * 16 + li]; mstar = fmaxf(mstar, wgt[w]); }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wgt[w] = (wgt[w] == -INFINITY) ? 0.f : expf(wgt[w] - mstar);
        lsum += wgt[w] * lsh[w * 16 + li];
    }
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    float *orow = (float *)a.out + qoff;
#pragma unroll
    for (int t = 0; t < VPW; ++t) {
        const int v = wave * VPW + t;               // accumulator value v: head_dim 16 (v / 4) + 4 kg + v % 4
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += wgt[w] * red[(w * NV + v) * 64 + lane];
        if (row_ok) orow[16 * (v >> 2) + 4 * kg + (v & 3)] = sum * inv;
    }
    if (wave == 0 && kg == 0 && row_ok && lsum == 0.f && a.empty_is_error && a.dev_status)
        atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
}

// DH/8 lanes per (sequence, query, head) row, 8 head_dim values (one 16-byte load per slice) per lane; a
// workgroup of 256 threads folds 2048/DH rows
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

template <int DH, int CALLS>
__global__ __launch_bounds__(256) void k_attn_merge(AttnGroup<CALLS> grp, SplitGeom geo)
{
    constexpr int LPR = DH / 8;            // lanes per row
    constexpr int RPB = 256 / LPR;         // rows per workgroup
    const int per_call = grp.a[0].B * grp.a[0].Mq * grp.a[0].H;
    const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
    if (row >= (int64_t)grp.ncalls * per_call) return;
    const int call = (int)(row / per_call), blk = (int)(row - (int64_t)call * per_call);
    const int piece = threadIdx.x % LPR;
    const AttnArgs &a = grp.a[call];
    const f16_t *__restrict__ part_o = (const f16_t *)a.ws;
    const float *__restrict__ part_ml = (const float *)(part_o + (size_t)grp.nbg * geo.nsplit * geo.rows_pad * DH);
    const int h = blk % a.H;
    const int m = (blk / a.H) % a.Mq;
    const int b = blk / (a.H * a.Mq);
    const int G = a.H / a.Hkv, g = h / G, rho = m * G + (h - g * G);
    const int64_t bg = (int64_t)b * a.Hkv + g;

    // slices in groups of four: all (max, sum) pairs and accumulator pieces of a group are requested before any
    // is used; groups are folded with the usual running-max rescale
    const int64_t stride = geo.rows_pad;
    const int64_t prow0 = bg * geo.nsplit * stride + rho;
    float mstar = -INFINITY, lsum = 0.f, o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = 0.f;
    for (int s0 = 0; s0 < geo.nsplit; s0 += 4) {
        float ms[4], ls[4];
        f16x8 ov[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int sidx = min(s0 + u, geo.nsplit - 1);
            const int64_t prow = prow0 + sidx * stride;
            ms[u] = (s0 + u < geo.nsplit) ? part_ml[prow * 2] : -INFINITY;
            ls[u] = part_ml[prow * 2 + 1];
            ov[u] = *(const f16x8 *)(part_o + prow * DH + 8 * piece);
        }
        float gmax = mstar;
#pragma unroll
        for (int u = 0; u < 4; ++u) gmax = fmaxf(gmax, ms[u]);
        if (gmax == -INFINITY) continue;
        const float keep = exp2f(mstar - gmax);      // 0 on the first non-empty group
        lsum *= keep;
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] *= keep;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float w = (ms[u] == -INFINITY) ? 0.f : exp2f(ms[u] - gmax) * ls[u];   // slice weight
            lsum += w;
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] += w * (float)ov[u][c];
        }
        mstar = gmax;
    }
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    u32x4 pk;
#pragma unroll
    for (int w = 0; w < 4; ++w) pk[w] = pack_bf16x2(o[2 * w] * inv, o[2 * w + 1] * inv);
    *(u32x4 *)((bf16_t *)a.out + (((int64_t)b * a.Mq + m) * a.H + h) * DH + 8 * piece) = pk;
    if (lsum == 0.f && a.empty_is_error && piece == 0 && a.dev_status) atomicOr(a.dev_status, MOA_DEV_EMPTY_KEYS);
}

// ------------------------------------------------------------------ host side (which kernel: moa_attn_plan.h)
static int attn_form() { return g_attn_form.load(std::memory_order_relaxed); }

static bool mfma_ok(int dtype, int dh, const AttnArgs *a)
{
    if (dtype != DT_BF16 || (dh != 64 && dh != 128)) return false;
    if (!a) return true;
    auto al = [](const void *p) { return (((uintptr_t)p) & 15) == 0; };
    return al(a->q) && al(a->kcache) && al(a->vcache) && al(a->ktree) && al(a->vtree) && al(a->out);
}

size_t attn_workspace_bytes(int dtype, int B, int Mq, int H, int Hkv, int dh, int P_cap, bool upto)
{
    if (!mfma_ok(dtype, dh, nullptr)) return 0;
    if (upto) {
        const size_t row_bytes = (size_t)dh * sizeof(f16_t) + 2 * sizeof(float);
        // Neither fewer rows nor fewer sequences always need less (they leave room for more key slices), so this is a bound
        // that grows with every size.  `units` row tiles of 128 take at most max(units, min(512, units * most)) slices, and
        // the 256-row form never takes more rows than those.
        const int64_t units = (int64_t)B * Hkv * (((int64_t)(H / Hkv) * Mq + 127) / 128);
        int64_t most = ((P_cap + KT - 1) / KT) / 2;
        most = most < 1 ? 1 : most > 64 ? 64 : most;
        int64_t slices = units * most < 512 ? units * most : 512;
        if (slices < units) slices = units;
        return (size_t)slices * 128 * ATTN_NBLK * row_bytes + 256;
    }
    return split_room(attn_form(), B, Mq, H, Hkv, dh, P_cap);
}

bool attn_takes_whole_range(int dtype, int B, int Mq, int Mt, int H, int Hkv, int dh, int P_cap)
{
    return dtype != DT_BF16 || (mfma_ok(dtype, dh, nullptr) && want_whole(attn_form(), B, Mq, Mt, H, Hkv, P_cap));
}

static hipError_t launch_attn_generic(const AttnArgs &a, hipStream_t stream)
{
    const int nblocks = a.B * a.Mq * a.H;
    if (a.dh > 256) return hipErrorInvalidValue;
    if (a.dtype == DT_BF16) { prof_begin(K_ATTN_GENERIC, stream); MOA_KLAUNCH(k_attn_generic<bf16_t>, dim3(nblocks), dim3(64), 0, stream, a); prof_end(stream); }
    else { prof_begin(K_ATTN_GENERIC, stream); MOA_KLAUNCH(k_attn_generic<float>, dim3(nblocks), dim3(64), 0, stream, a); prof_end(stream); }
    return hipGetLastError();
}

static bool attn_f32_ok(const AttnArgs &a)
{
    auto al = [](const void *p) { return (((uintptr_t)p) & 15) == 0; };
    return a.dtype == DT_F32 && (a.dh == 64 || a.dh == 128) && al(a.q) && al(a.kcache) && al(a.ktree);
}

template <int CALLS>
static AttnGroup<CALLS> group_of(const AttnArgs *calls, int n)
{
    AttnGroup<CALLS> grp;
    grp.nrb = 0;
    for (int i = 0; i < CALLS; ++i) grp.a[i] = calls[i < n ? i : n - 1];
    grp.nbg = calls[0].B * calls[0].Hkv;
    grp.ncalls = n;
    return grp;
}

template <int DH, int CALLS>
static hipError_t launch_f32_as(const AttnGroup<CALLS> &grp, unsigned grid, hipStream_t stream)
{
    constexpr size_t lds = attn_f32_lds<DH>();
    static bool raised[16] = {};
    hipError_t e = raise_lds_limit_once(raised, (const void *)k_attn_f32<DH, CALLS>, lds);
    if (e != hipSuccess) return e;
    prof_begin(K_ATTN_F32, stream);
    MOA_KLAUNCH((k_attn_f32<DH, CALLS>), dim3(grid), dim3(64 * F32_NW), lds, stream, grp);
    prof_end(stream);
    return hipGetLastError();
}

// calls of identical shape (B, Mq, H, Hkv, dh)
template <int CALLS>
static hipError_t launch_attn_f32_as(const AttnArgs *calls, int n, hipStream_t stream)
{
    const AttnArgs &a = calls[0];
    AttnGroup<CALLS> grp = group_of<CALLS>(calls, n);
    const int nrb = grp.nrb = ((a.H / a.Hkv) * a.Mq + 15) / 16;
    const int64_t grid = (int64_t)n * grp.nbg * nrb;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    return a.dh == 128 ? launch_f32_as<128, CALLS>(grp, (unsigned)grid, stream) : launch_f32_as<64, CALLS>(grp, (unsigned)grid, stream);
}

// calls of identical shape (B, Mq, H, Hkv, dh)
template <int DH, int NW, int CALLS>
static hipError_t launch_fused_as(const AttnGroup<CALLS> &grp, unsigned grid, hipStream_t stream)
{
    constexpr size_t lds = FusedLds<DH, NW>::bytes;
    static bool raised[16] = {};
    hipError_t e = raise_lds_limit_once(raised, (const void *)k_attn_fused<DH, NW, CALLS>, lds);
    if (e != hipSuccess) return e;
    prof_begin(K_ATTN_FUSED + 64 * (DH * 8 + NW / 4), stream);
    MOA_KLAUNCH((k_attn_fused<DH, NW, CALLS>), dim3(grid), dim3(64 * NW), lds, stream, grp);
    prof_end(stream);
    return hipGetLastError();
}

template <int CALLS>
static hipError_t launch_attn_fused_as(const AttnArgs *calls, int n, hipStream_t stream)
{
    const AttnArgs &a = calls[0];
    AttnGroup<CALLS> grp = group_of<CALLS>(calls, n);
    const int RG = (a.H / a.Hkv) * a.Mq;
    const int64_t units8 = ((int64_t)n * grp.nbg + 7) / 8;
    // blocks of 16 rows while all of their workgroups run at once, unless another stream's launches want the compute units that this
    // takes (8B step with the Self-Attention layer on two streams: 159 us with them, 151 without; the results are the same bits)
    if (a.dh == 128 && !a.beside && 8 * units8 * ((RG + 15) / 16) <= 256) {
        constexpr size_t lds = Fused16Lds<128, 8>::bytes;
        static bool raised[16] = {};
        hipError_t e = raise_lds_limit_once(raised, (const void *)k_attn_fused16<128, 8, CALLS>, lds);
        if (e != hipSuccess) return e;
        grp.nrb = (RG + 15) / 16;
        prof_begin(K_ATTN_FUSED16, stream);
        MOA_KLAUNCH((k_attn_fused16<128, 8, CALLS>), dim3((unsigned)(8 * units8 * grp.nrb)), dim3(512), lds, stream, grp);
        prof_end(stream);
        return hipGetLastError();
    }
    const int nrb = grp.nrb = (RG + 31) / 32;
    const int64_t grid = 8 * units8 * nrb;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    if (a.dh == 128) return launch_fused_as<128, 8, CALLS>(grp, (unsigned)grid, stream);
    return launch_fused_as<64, 8, CALLS>(grp, (unsigned)grid, stream);
}

template <int CALLS>
static hipError_t launch_attn_split_as(const AttnArgs *calls, int n, const SplitGeom &g, hipStream_t stream)
{
    const AttnArgs &a = calls[0];
    AttnGroup<CALLS> grp = group_of<CALLS>(calls, n);
    const int nblocks = n * a.B * a.Mq * a.H;
    hipError_t e;
    if (g.wide) {
        e = launch_attn_long(grp, g, stream);
        if (e != hipSuccess || g.nsplit == 1) return e;
    } else {
        const dim3 grid(g.nsplit, g.rowtiles, n * grp.nbg);
        prof_begin(K_ATTN_MFMA + 64 * (a.dh * 8 + ATTN_NBLK), stream);
        if (a.dh == 128) MOA_KLAUNCH((k_attn_mfma<128, ATTN_NBLK, CALLS>), grid, dim3(256), 0, stream, grp, g);
        else MOA_KLAUNCH((k_attn_mfma<64, ATTN_NBLK, CALLS>), grid, dim3(256), 0, stream, grp, g);
        prof_end(stream);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    prof_begin(K_ATTN_MERGE + 64 * (a.dh * 8), stream);
    const int rpb = 2048 / a.dh;                      // rows per merge workgroup
    const unsigned mblocks = (unsigned)(((int64_t)nblocks + rpb - 1) / rpb);
    if (a.dh == 128) MOA_KLAUNCH((k_attn_merge<128, CALLS>), dim3(mblocks), dim3(256), 0, stream, grp, g);
    else MOA_KLAUNCH((k_attn_merge<64, CALLS>), dim3(mblocks), dim3(256), 0, stream, grp, g);
    prof_end(stream);
    return hipGetLastError();
}

static hipError_t launch_attn_f32(const AttnArgs *calls, int n, hipStream_t stream)
{
    return n <= ATTN_FEW ? launch_attn_f32_as<ATTN_FEW>(calls, n, stream) : launch_attn_f32_as<ATTN_CALLS>(calls, n, stream);
}
static hipError_t launch_attn_fused(const AttnArgs *calls, int n, hipStream_t stream)
{
    return n <= ATTN_FEW ? launch_attn_fused_as<ATTN_FEW>(calls, n, stream) : launch_attn_fused_as<ATTN_CALLS>(calls, n, stream);
}
static hipError_t launch_attn_split(const AttnArgs *calls, int n, const SplitGeom &g, hipStream_t stream)
{
    return n <= ATTN_FEW ? launch_attn_split_as<ATTN_FEW>(calls, n, g, stream) : launch_attn_split_as<ATTN_CALLS>(calls, n, g, stream);
}

// whole-tree defaults of the tree window; false when the window does not fit its tree
static bool tree_window(AttnArgs &a)
{
    if (!a.tree_cap) a.tree_cap = a.Mt;
    if (!a.mask_rows) a.mask_rows = a.Mq;
    return a.mask_row0 >= 0 && a.mask_row0 + a.Mq <= a.mask_rows && a.Mt <= a.tree_cap;
}

hipError_t launch_attn(const AttnArgs &a, hipStream_t stream) { return launch_attn_group(&a, 1, false, stream); }

hipError_t launch_attn_group(const AttnArgs *calls, int n, bool pair, hipStream_t stream)
{
    if (n < 1 || n > ATTN_CALLS) return hipErrorInvalidValue;
    AttnArgs a[ATTN_CALLS], part[ATTN_CALLS];
    AttnCore core[ATTN_CALLS];
    bool same = true, f32 = true;
    for (int i = 0; i < n; ++i) {
        a[i] = calls[i];
        if (!tree_window(a[i])) return hipErrorInvalidValue;
        same = same && a[i].dtype == a[0].dtype && a[i].B == a[0].B && a[i].Mq == a[0].Mq && a[i].H == a[0].H && a[i].Hkv == a[0].Hkv && a[i].dh == a[0].dh;
        f32 = f32 && attn_f32_ok(a[i]);
        core[i] = {a[i].P_cap, a[i].Mt, mfma_ok(a[i].dtype, a[i].dh, &a[i]), a[i].ws && ((uintptr_t)a[i].ws & 15) == 0 ? a[i].ws_bytes : 0};
    }
    hipError_t e = hipSuccess;
    if (!same) {
        for (int i = 0; i < n && e == hipSuccess; ++i) e = launch_attn_group(calls + i, 1, false, stream);
        return e;
    }
    if (f32) return launch_attn_f32(a, n, stream);
    AttnChoice choice[ATTN_CALLS];
    choose_attn(attn_form(), a[0].B, a[0].Mq, a[0].H, a[0].Hkv, a[0].dh, core, n, pair, choice);
    bool done[ATTN_CALLS] = {};
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        if (done[i]) continue;
        int m = 0;
        for (int k = i; k < n; ++k) {
            if (done[k] || !choice[i].shares_with(choice[k])) continue;
            part[m++] = a[k];
            done[k] = true;
        }
        if (choice[i].kind == AttnChoice::WHOLE) e = launch_attn_fused(part, m, stream);
        else if (choice[i].kind == AttnChoice::SPLIT) e = launch_attn_split(part, m, choice[i].geo, stream);
        else for (int k = 0; k < m && e == hipSuccess; ++k) e = attn_f32_ok(part[k]) ? launch_attn_f32(part + k, 1, stream) : launch_attn_generic(part[k], stream);
    }
    return e;
}

}  // namespace moa

extern "C" int32_t moa_debug_force_attn_kernel(int32_t form)
{
    if (form < MOA_ATTN_KERNEL_AUTO || form > MOA_ATTN_KERNEL_SPLIT_WIDE)
        return moa::api_fail(MOA_ERR_SHAPE, "debug_force_attn_kernel: form must be MOA_ATTN_KERNEL_AUTO / _WHOLE / _SPLIT / _SPLIT_WIDE");
    moa::g_attn_form.store(form, std::memory_order_relaxed);
    return MOA_OK;
}
