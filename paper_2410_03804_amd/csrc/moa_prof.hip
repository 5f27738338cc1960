// Optional per-kernel timing for the benchmark: when enabled, a pair of hipEvents is recorded on the
// caller's stream around every kernel launch (or around the launches of one chosen kernel only).
// Off by default; nothing here runs on the hot path unless the caller switches it on.
#include "../../include/moa.h"
#include "moa_common.h"

#include <stdio.h>
#include <stdlib.h>

#include <mutex>
#include <vector>

namespace moa {

namespace {
struct Rec { int site, kernel; hipEvent_t e0, e1; };
std::mutex g_mu;
bool g_on = false;
int g_only_kernel = -1;
int g_every = 1, g_seen = 0;
std::vector<Rec> g_recs;
std::vector<hipEvent_t> g_pool;
thread_local int t_site = S_NONE;
thread_local bool t_open = false;
thread_local hipEvent_t t_e0 = nullptr, t_e1 = nullptr;

hipEvent_t take_event()
{
    if (!g_pool.empty()) { hipEvent_t e = g_pool.back(); g_pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

const char *const kKernelNames[K_COUNT] = {
    "k_tree_build", "k_tree_accept", "k_append_lengths", "k_linear_generic",
    "k_linear_splitk_reduce", "k_scatter_copy", "k_attn_generic", "k_attn_mfma", "k_attn_merge", "k_lsa_attn", "k_lsa_attn_mfma", "k_step_small", "k_attn_fused", "k_probe_read", "k_probe_mfma",
    "k_rmsnorm", "k_rope", "k_swiglu", "k_add_out", "k_tree_expand", "k_tree_finalize", "k_topk_slices", "k_lm_head_argmax", "k_lm_head_reduce", "k_topk_merge", "k_msg_tree", "k_msg_accept", "k_lsa_fused", "k_lsa_fused_pk", "k_lsa_pack_weights", "k_linear_f32_latency", "k_linear_f32_tile", "k_attn_f32", "k_linear_bf16", "k_attn_long<128>", "k_attn_fused16<128, 8>"};
const char *const kSiteNames[S_COUNT] = {
    "none", "tree_build", "lsa.qkv_proj", "lsa.layer_attn", "lsa.o_proj", "ca_append.kv_proj", "ca_append.lengths",
    "ca.q_proj", "ca.core", "ca.o_proj", "verify.qkv_proj", "verify.core", "verify.o_proj", "tree_accept",
    "tree_build+accept+lengths", "ca.q_proj+verify.qkv_proj", "ca.core+verify.core", "ca.o_proj+verify.o_proj", "probe",
    "sa.qkv_proj", "sa.core", "sa.o_proj", "tli.qkv_proj", "tli.core", "tli.o_proj", "tli.rmsnorm", "tli.rope",
    "tli.gate_up_proj", "tli.swiglu", "tli.down_proj", "tli.residual", "tree_expand", "tree_finalize", "topk_logprob", "lm_head", "message", "linear", "mlp.rmsnorm", "mlp.gate_up_proj", "mlp.down_proj", "lsa.fused"};
}  // namespace

void prof_set_site(int site) { t_site = site; }

void prof_begin(int kernel, hipStream_t stream)
{
    if (!g_on) return;
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_on || (g_only_kernel >= 0 && kernel != g_only_kernel)) return;
    if (g_seen++ % g_every) return;
    Rec r = {t_site, kernel, take_event(), take_event()};
    if (!r.e0 || !r.e1) return;
    g_recs.push_back(r);
    t_e0 = r.e0;
    t_e1 = r.e1;
    t_open = true;
    (void)stream;
}

void prof_end(hipStream_t)
{
    t_open = false;
    t_e0 = t_e1 = nullptr;
}

hipEvent_t prof_start_event() { return t_open ? t_e0 : nullptr; }
hipEvent_t prof_stop_event() { return t_open ? t_e1 : nullptr; }

// ---- two probes of what this device delivers in practice, to put beside the published peaks
// plain streaming read: every lane 16 bytes, consecutive lanes consecutive addresses, eight loads in flight
__global__ __launch_bounds__(256) void k_probe_read(const u32x4 *__restrict__ p, size_t n16, uint32_t *sink)
{
    u32x4 acc = {0u, 0u, 0u, 0u};
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    for (; i + 7 * stride < n16; i += 8 * stride) {
        u32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[i + u * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= v[u];
    }
    for (; i < n16; i += stride) acc ^= p[i];
    if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9e3779b9u) *sink = acc[0];   // keeps the loads alive
}

// register-resident bf16 MFMA 32x32x16, four independent accumulators per wavefront, 16 wavefronts per CU
__global__ __launch_bounds__(256) void k_probe_mfma(int iters, float *sink)
{
    bf16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) { a[e] = (__bf16)(0.001f * (float)(threadIdx.x + e)); b[e] = (__bf16)(0.002f * (float)(threadIdx.x - e)); }
    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    for (int it = 0; it < iters; ++it)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[q], 0, 0, 0);
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += acc[q][0] + acc[q][15];
    if (s == 123456.789f) *sink = s;
}

}  // namespace moa

using namespace moa;

extern "C" {

int32_t moa_profile_enable(int32_t on, int32_t only_kernel)
{
    std::lock_guard<std::mutex> lk(g_mu);
    for (const Rec &r : g_recs) { g_pool.push_back(r.e0); g_pool.push_back(r.e1); }
    g_recs.clear();
    g_on = on != 0;
    g_only_kernel = only_kernel >= 0 ? only_kernel : -1;
    g_seen = 0;
    return MOA_OK;
}

int32_t moa_profile_sample_every(int32_t n)
{
    if (n < 1) return MOA_ERR_SHAPE;
    std::lock_guard<std::mutex> lk(g_mu);
    g_every = n;
    g_seen = 0;
    return MOA_OK;
}

int32_t moa_profile_collect(moa_profile_row_t *rows_host, int32_t max_rows, int32_t *n_rows_host)
{
    if (!rows_host || !n_rows_host || max_rows < 1) return MOA_ERR_NULL;
    std::lock_guard<std::mutex> lk(g_mu);
    int n = 0;
    int32_t rc = MOA_OK;
    for (const Rec &r : g_recs) {
        float ms = 0.f;
        if (hipEventSynchronize(r.e1) != hipSuccess || hipEventElapsedTime(&ms, r.e0, r.e1) != hipSuccess) {
            rc = MOA_ERR_HIP;
        } else {
            int i = 0;
            while (i < n && !(rows_host[i].site == r.site && rows_host[i].kernel == r.kernel)) ++i;
            if (i == n && n < max_rows) { rows_host[n] = {r.site, r.kernel, 0, 0.0}; ++n; }
            if (i < n) { rows_host[i].launches += 1; rows_host[i].total_ms += ms; }
        }
        g_pool.push_back(r.e0);
        g_pool.push_back(r.e1);
    }
    g_recs.clear();
    *n_rows_host = n;
    return rc;
}

int32_t moa_probe_read(const void *buf, size_t bytes, void *scratch4, void *stream)
{
    if (!buf || !scratch4 || bytes < 16 || (((uintptr_t)buf) & 15)) return MOA_ERR_NULL;
    prof_set_site(S_PROBE);
    prof_begin(K_PROBE_READ, (hipStream_t)stream);
    // one long-lived workgroup per compute unit streams fastest here (6.5 TB/s; 5.1 TB/s with eight per unit)
    int dev = 0, pg = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&pg, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || pg < 1) pg = 256;
    MOA_KLAUNCH(k_probe_read, dim3(pg), dim3(256), 0, (hipStream_t)stream, (const u32x4 *)buf, bytes / 16, (uint32_t *)scratch4);
    prof_end((hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? MOA_OK : MOA_ERR_HIP;
}

int32_t moa_probe_mfma(int32_t iters, void *scratch4, int64_t *flops_host, void *stream)
{
    if (!scratch4 || !flops_host || iters < 1) return MOA_ERR_NULL;
    const int blocks = 256 * 4;                       // four workgroups of four wavefronts per compute unit
    *flops_host = (int64_t)blocks * 4 * iters * 4 * (2LL * 32 * 32 * 16);
    prof_set_site(S_PROBE);
    prof_begin(K_PROBE_MFMA, (hipStream_t)stream);
    MOA_KLAUNCH(k_probe_mfma, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (int)iters, (float *)scratch4);
    prof_end((hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? MOA_OK : MOA_ERR_HIP;
}

// ids are base + 64 * variant; the variant spells the template arguments the way a profiler prints them (but not the room for segments or
// calls, LinDev and AttnGroup)
const char *moa_profile_kernel_name(int32_t kernel)
{
    static thread_local char buf[96];
    const int base = kernel & 63, var = kernel >> 6;
    if (kernel < 0 || base >= K_COUNT) return "?";
    if (var == 0) return kKernelNames[base];
    if (base == K_LIN_BF16) return linear_bf16_name(var);
    if (base == K_ATTN_FUSED) snprintf(buf, sizeof(buf), "%s<%d, %d>", kKernelNames[base], var >> 3, 4 * (var & 7));
    else if (base == K_LSA_FUSED_PK && var >> 3 == 4) snprintf(buf, sizeof(buf), "%s_wide<128, %d>", kKernelNames[base], var & 7);
    else if (base == K_LSA_FUSED || base == K_LSA_FUSED_PK) snprintf(buf, sizeof(buf), "%s%s<128, %d, %d>", kKernelNames[base], var & 64 ? "_dense" : "", (var >> 3) & 7, var & 7);
    else if (base == K_ATTN_MERGE) snprintf(buf, sizeof(buf), "%s<%d>", kKernelNames[base], var >> 3);
    else snprintf(buf, sizeof(buf), "%s<%d, %d>", kKernelNames[base], var >> 3, var & 7);
    return buf;
}
const char *moa_profile_site_name(int32_t site) { return (site >= 0 && site < S_COUNT) ? kSiteNames[site] : "?"; }

}  // extern "C"
