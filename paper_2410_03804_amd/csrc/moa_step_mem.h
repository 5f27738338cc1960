// Which verification layers of a step may share launches: a question of what memory they read and write, and of where their
// intermediate results go.  Host arithmetic only.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "../../include/moa.h"

namespace moa {

// ---- verification layers in common launches.
// A step is given every layer's input, so as a rule no layer needs another's output, and what a decoding program keeps in
// separate launches because one layer feeds the next can share them here: 3 sequences x 37 nodes x 3 layers of the 8B shape
// 261 -> 192 us.  But nothing keeps a caller from letting one layer read what another wrote (that order has always
// been kept), so memory decides.  A layer joins the launches of those before it, and the first layers the
// CA's, if what it writes is neither read nor written by them and what they write is not read by it.
inline size_t elem_bytes(const moa_shape_t *s) { return s->dtype == MOA_BF16 ? 2 : 4; }

struct MemRange {
    const char *lo = nullptr, *hi = nullptr;
    MemRange() {}
    MemRange(const void *p, size_t n) : lo((const char *)p), hi((const char *)p + (p ? n : 0)) {}
    bool meets(const MemRange &o) const { return lo < o.hi && o.lo < hi; }
};

template <size_t NA, size_t NB>
inline bool any_meet(const MemRange (&a)[NA], const MemRange (&b)[NB])
{
    for (const MemRange &x : a)
        for (const MemRange &y : b)
            if (x.meets(y)) return true;
    return false;
}

struct LayerMem {
    MemRange reads[7], writes[3];
    bool aligned;
    LayerMem(const moa_step_args_t *a, int l)
    {
        const moa_shape_t *s = a->shape;
        const size_t es = elem_bytes(s), d = s->d_model, e = (size_t)s->n_q_heads * s->head_dim, ekv = (size_t)s->n_kv_heads * s->head_dim;
        const size_t rows = (size_t)a->B * a->M, cache = (size_t)a->B * a->P_cap;
        reads[0] = {a->v_x_host[l], rows * d * es};
        reads[1] = {a->v_wq_host[l], e * d * es};
        reads[2] = {a->v_wk_host[l], ekv * d * es};
        reads[3] = {a->v_wv_host[l], ekv * d * es};
        reads[4] = {a->v_wo_host[l], d * e * es};
        reads[5] = {a->v_kcache_host[l], cache * ekv * es};
        reads[6] = {a->v_vcache_host[l], cache * ekv * es};
        writes[0] = {a->v_out_host[l], rows * d * es};
        writes[1] = {a->v_ktree_host[l], rows * ekv * es};
        writes[2] = {a->v_vtree_host[l], rows * ekv * es};
        uintptr_t all = 0;
        for (const MemRange &r : reads) all |= (uintptr_t)r.lo;
        for (const MemRange &r : writes) all |= (uintptr_t)r.lo;
        aligned = (all & 15) == 0;
    }
    bool apart(const LayerMem &o) const { return !any_meet(writes, o.reads) && !any_meet(o.writes, reads) && !any_meet(writes, o.writes); }
};

// the Self-Attention layer in front of the cross-attention
struct SaMem {
    MemRange reads[7], writes[3];
    bool aligned;
    explicit SaMem(const moa_step_args_t *a)
    {
        const moa_shape_t *s = a->sa_shape;
        const size_t es = elem_bytes(s), d = s->d_model, e = (size_t)s->n_q_heads * s->head_dim, ekv = (size_t)s->n_kv_heads * s->head_dim;
        const size_t rows = (size_t)a->B * a->M, cache = (size_t)a->B * a->sa_P_cap;
        reads[0] = {a->sa_emb, rows * d * es};
        reads[1] = {a->sa_wq, e * d * es};
        reads[2] = {a->sa_wk, ekv * d * es};
        reads[3] = {a->sa_wv, ekv * d * es};
        reads[4] = {a->sa_wo, d * e * es};
        reads[5] = {a->sa_kcache, cache * ekv * es};
        reads[6] = {a->sa_vcache, cache * ekv * es};
        writes[0] = {a->sa_out, rows * d * es};
        writes[1] = {a->sa_k_draft, rows * ekv * es};
        writes[2] = {a->sa_v_draft, rows * ekv * es};
        uintptr_t all = 0;
        for (const MemRange &r : reads) all |= (uintptr_t)r.lo;
        for (const MemRange &r : writes) all |= (uintptr_t)r.lo;
        aligned = (all & 15) == 0;
    }
};

// what the step's integer work reads and writes (the masks, which the layer is meant to read, aside)
inline bool apart_from_integers(const moa_step_args_t *a, const SaMem &m)
{
    const size_t ints = (size_t)a->B * a->M * sizeof(int32_t), seqs = a->B * sizeof(int32_t);
    const MemRange reads[] = {{a->parent, ints}, {a->tok, ints}, {a->tgt, ints}, {a->tok_off, seqs + sizeof(int32_t)}};
    const MemRange writes[] = {{a->depth, ints}, {a->path, ints}, {a->n_path, seqs}, {a->bonus, seqs}, {a->ca_len, seqs}, {a->dev_status, sizeof(int32_t)}};
    const MemRange mask[] = {{a->mask, (size_t)a->B * a->M * ((a->M + 63) / 64) * sizeof(uint64_t)}};
    return !any_meet(m.writes, reads) && !any_meet(m.writes, writes) && !any_meet(m.reads, writes) && !any_meet(m.writes, mask) && !any_meet(m.reads, mask);
}

// whether the layer's projections can go into a launch with the integer work and those of the first `layers` verification layers
inline bool sa_apart(const moa_step_args_t *a, int layers)
{
    const SaMem m(a);
    if (!m.aligned || !apart_from_integers(a, m)) return false;
    for (int l = 0; l < layers; ++l) {
        const LayerMem v(a, l);
        if (!v.aligned || any_meet(v.writes, m.reads) || any_meet(v.writes, m.writes) || any_meet(v.reads, m.writes)) return false;
    }
    return true;
}

// what the rest of a step -- the LSA, the memory, the cross-attention, the integer work -- reads and writes
inline bool apart_from_rest(const moa_step_args_t *a, const LayerMem &m)
{
    const moa_shape_t *s = a->shape;
    const size_t es = elem_bytes(s), R = (size_t)a->B * a->M, T = (size_t)a->T_lsa, d = s->d_model, ints = R * sizeof(int32_t);
    const size_t e = (size_t)s->n_q_heads * s->head_dim, ekv = (size_t)s->n_kv_heads * s->head_dim;
    const size_t eq = (size_t)s->lsa_q_heads * s->head_dim, el = (size_t)s->lsa_kv_heads * s->head_dim, din = s->d_lsa_in;
    const MemRange reads[] = {{a->parent, ints}, {a->tok, ints}, {a->tgt, ints}, {a->tok_off, (a->B + 1) * sizeof(int32_t)}, {a->prefix_len, a->B * sizeof(int32_t)},
                              {a->lsa_hs, T * s->n_layers * din * es}, {a->lsa_wq, eq * din * es}, {a->lsa_wk, el * din * es}, {a->lsa_wv, el * din * es},
                              {a->lsa_wo, eq * eq * es}, {a->lsa_w_packed, 2 * eq * din * es},
                              {a->ca_wk, ekv * eq * es}, {a->ca_wv, ekv * eq * es}, {a->ca_wk_lsa_wo, ekv * eq * es}, {a->ca_wv_lsa_wo, ekv * eq * es},
                              {a->ca_xq, R * d * es}, {a->ca_wq, e * d * es}, {a->ca_wo, e * d * es}};
    const MemRange writes[] = {{a->mask, R * ((a->M + 63) / 64) * sizeof(uint64_t)}, {a->depth, ints}, {a->path, ints}, {a->n_path, a->B * sizeof(int32_t)},
                               {a->bonus, a->B * sizeof(int32_t)}, {a->lsa_out, T * eq * es}, {a->ca_len, a->B * sizeof(int32_t)},
                               {a->ca_k, (size_t)a->B * a->ca_P_cap * ekv * es}, {a->ca_v, (size_t)a->B * a->ca_P_cap * ekv * es}, {a->ca_out, R * d * es},
                               {a->dev_status, sizeof(int32_t)}};
    return !any_meet(m.writes, reads) && !any_meet(m.writes, writes) && !any_meet(m.reads, writes);
}

// How many verification layers from l0 on go into common launches, `most` at most (at least one); with_rest: beside the
// CA's, where layer 0 has always been.  Layers with other alignments would take everybody to kernels that can read them.
inline int verify_run(const moa_step_args_t *a, int l0, int most, bool with_rest)
{
    if (most > a->n_verify_layers - l0) most = a->n_verify_layers - l0;
    if (most <= 1) return 1;
    auto whole = [&](int l) { return a->v_wq_host[l] && a->v_wk_host[l] && a->v_wv_host[l] && a->v_wo_host[l]; };
    const uintptr_t ca = (uintptr_t)a->ca_xq | (uintptr_t)a->ca_wq | (uintptr_t)a->ca_wo | (uintptr_t)a->ca_k | (uintptr_t)a->ca_v | (uintptr_t)a->ca_out;
    if (!whole(l0) || !LayerMem(a, l0).aligned || (with_rest && (ca & 15))) return 1;
    int n = 1;
    for (; n < most; ++n) {
        const LayerMem m(a, l0 + n);
        bool joins = whole(l0 + n) && m.aligned && (!with_rest || apart_from_rest(a, m));
        for (int i = 0; joins && i < n; ++i) joins = m.apart(LayerMem(a, l0 + i));
        if (!joins) break;
    }
    return n;
}

// A verification layer's buffers in common launches: queries and heads, and scratch of its core -- none where cores of this
// shape run over the whole key range (whatever they are made to do after all, nothing says that there is any).
struct VerifyMem {
    char *q, *h, *core;
    size_t core_bytes;
};

// Those of the layers after the first (mem[0] is there), up to `most` in all: queries and heads of qa bytes each in `spare`, memory that
// the step's layout leaves, and scratch of `core` bytes in `idle`, memory that is not in use while the cores run, and then in `spare` too.
// How many layers there are buffers for.
inline int carve_verify(VerifyMem *mem, int most, size_t qa, size_t core, char *spare, size_t spare_bytes, char *idle, size_t idle_bytes)
{
    int n = 1;
    for (; n < most; ++n) {
        const bool in_idle = core <= idle_bytes;
        const size_t take = 2 * qa + (in_idle ? 0 : core);
        if (spare_bytes < take) break;
        mem[n] = {spare, spare + qa, core == 0 ? nullptr : in_idle ? idle : spare + 2 * qa, core};
        if (core && in_idle) idle += core, idle_bytes -= core;
        spare += take;
        spare_bytes -= take;
    }
    return n;
}

}  // namespace moa
