// What comes before and after the fused adjoint walk, per particle: the upstream gradients and the zeros that the
// walk adds to, and the downward pass that collects a particle's gradients.  Each is a kernel of its own
// (adjoint.hip) and, in the MD step of small systems, part of a neighbouring kernel (md.hip).
#pragma once
#include "ffbh_internal.h"

namespace ffbh {

struct AdjSetup {
    const double *gH, *gE, *smom;
    const uint32_t *perm;
    int64_t n, ntot;
    double *hbar, *g_rm, *node_adj, *node_adjq;  // node_adjq: null without order-2 cells
    const uint32_t *nn;                          // nodes of the last build
    int64_t max_nodes;
    const int32_t *per_system;  // nodes below the root of each system where it was built by one workgroup, else null
};

inline AdjSetup adj_setup_args(const Handle &h, const double *gH, const double *gE)
{
    const Workspace &w = h.w;
    return {gH, gE, w.smom, w.perm, h.L.n, h.L.ntot, w.hbar, w.g_rm, w.node_adj,
            h.L.expansion == 2 ? w.node_adjq : nullptr, w.status + 2, h.L.max_nodes,
            h.L.n <= kSmallMax ? w.top_nodes : nullptr};
}

// Before the fused walk: the upstream field gradient in sorted order, Hbar = gH - 1/2 gE m, and zeros in the
// adjoint records of the particles (g_rm) and of the nodes the last build made (their counts are on the device).
// Bound by the writes, 104 B a particle and 64 B a node (2^20 particles: about 25 us); as three launches small
// systems paid 9 us more.
__device__ inline void adj_setup(const AdjSetup &a, int64_t t, int64_t stride)
{
    const int64_t n = a.n, ntot = a.ntot;
    for (int64_t s = t; s < ntot; s += stride) {
        const int64_t o = a.perm[s], b = o / n, i = o - b * n;
        if (o >= ntot) continue;
        const double ge = a.gE ? a.gE[b] : 0.0;
        for (int k = 0; k < 3; ++k) {
            double v = a.gH ? a.gH[b * 3 * n + k * n + i] : 0.0;
            v += -0.5 * ge * a.smom[k * ntot + s];
            a.hbar[k * ntot + s] = v;
        }
    }
    for (int64_t i = t; i < 8 * ntot; i += stride) a.g_rm[i] = 0.0;
    if (a.per_system) {
        // small systems: the roots, then 2 n node places per system of which the first per_system[b] are used
        const int64_t B = ntot / n;
        for (int64_t i = t; i < 8 * (B + 2 * ntot); i += stride) {
            const int64_t k = i / 8 - B, b = k / (2 * n);
            if (k >= 0 && k - 2 * n * b >= (int64_t)a.per_system[b]) continue;
            a.node_adj[i] = 0.0;
            if (a.node_adjq) a.node_adjq[i] = 0.0;
        }
        return;
    }
    const int64_t len = 8 * ((int64_t)*a.nn < a.max_nodes ? (int64_t)*a.nn : a.max_nodes);
    for (int64_t i = t; i < len; i += stride) a.node_adj[i] = 0.0;
    if (a.node_adjq)
        for (int64_t i = t; i < len; i += stride) a.node_adjq[i] = 0.0;
}

struct Downward {
    const NodeRec *nodes;
    const int32_t *leaf_of;
    const double *node_adj, *g_gather, *g_rm, *Hs, *part_buf;
    int parts;  // of a walk divided over the root's children (1: undivided, sums in g_gather and Hs)
    const double *hext, *gE;
    const uint32_t *perm;
    int64_t n, ntot, max_nodes;
    const double *node_adjq, *node_m64, *spos, *smom;  // node_adjq: null without order-2 cells
};

inline Downward downward_args(const Handle &h, const double *hext, const double *gE)
{
    const Workspace &w = h.w;
    return {w.nodes, w.leaf_of, w.node_adj, w.g_gather, w.g_rm, w.Hs, w.part_buf, h.adj_parts, hext, gE, w.perm,
            h.L.n, h.L.ntot, h.L.max_nodes, h.L.expansion == 2 ? w.node_adjq : nullptr, w.node_m64, w.spos, w.smom};
}

// What the walk summed for sorted particle s: gathered dL/dr and forward field (v), dL/dr and dL/dm as a source (q).
// The parts of a divided walk are summed here, in part order, so that the result does not depend on scheduling (a
// launch of their own cost small systems 5 us).
struct Sums {
    double v[6], q[6];
};

__device__ inline Sums load_sums(const Downward &a, int64_t s)
{
    const int64_t ntot = a.ntot;
    Sums u{};
    if (a.parts > 1) {
#pragma unroll 4
        for (int p = 0; p < a.parts; ++p)
#pragma unroll
            for (int c = 0; c < 6; ++c) u.v[c] += a.part_buf[((int64_t)p * 6 + c) * ntot + s];
    } else {
        for (int k = 0; k < 3; ++k) {
            u.v[k] = a.g_gather[k * ntot + s];
            u.v[3 + k] = a.Hs[k * ntot + s];
        }
    }
    for (int c = 0; c < 6; ++c) u.q[c] = a.g_rm[8 * s + c];
    return u;
}

// Downward pass of sorted particle s: it collects its cells' adjoints along the leaf-to-root path; the explicit
// derivative of E in m (-1/2 H - H_ext, times dL/dE) is added.  b: its system.
// FIRST: the sums are loaded beside the path (latency, small systems), else after it (fewer registers held, five
// instead of four waves per SIMD).
// With order-2 cells a member j of cell C also receives, through D_C = sum (r_j - c_C) m_j^T and c_C = the
// members' mean, dL/dr_j += E_C m_j - E_C M_C / n_C and dL/dm_j += E_C (r_j - c_C) (E_C symmetric, stored as xx,
// yy, zz, xy, xz, yz).
template <bool FIRST>
__device__ inline void downward(const Downward &a, int64_t s, int64_t b, double dr[3], double dm[3])
{
    const int64_t ntot = a.ntot;
    Sums u;
    if (FIRST) u = load_sums(a, s);
    double A[3] = {0.0, 0.0, 0.0}, B[3] = {0.0, 0.0, 0.0};
    double qr[3] = {0.0, 0.0, 0.0}, qm[3] = {0.0, 0.0, 0.0};
    double rj[3] = {0.0, 0.0, 0.0}, mj[3] = {0.0, 0.0, 0.0};
    if (a.node_adjq) {
        for (int k = 0; k < 3; ++k) {
            rj[k] = a.spos[k * ntot + s];
            mj[k] = a.smom[k * ntot + s];
        }
    }
    int node = a.leaf_of[s];
    for (int depth = 0; node >= 0 && node < a.max_nodes && depth < 2 * kMaxLevel + 2; ++depth) {
        const double *g = a.node_adj + 8 * (int64_t)node;
        const NodeRec nd = a.nodes[node];
        const double inv = 1.0 / (double)nd.count;
        for (int k = 0; k < 3; ++k) {
            A[k] += g[k];
            B[k] += g[3 + k] * inv;
        }
        if (a.node_adjq) {
            const double *e = a.node_adjq + 8 * (int64_t)node;
            const double E[3][3] = {{e[0], e[3], e[4]}, {e[3], e[1], e[5]}, {e[4], e[5], e[2]}};
            const double *M = a.node_m64 + 4 * (int64_t)node;
            const double d[3] = {rj[0] - nd.cx, rj[1] - nd.cy, rj[2] - nd.cz};
            for (int k = 0; k < 3; ++k) {
                qr[k] += E[k][0] * (mj[0] - M[0] * inv) + E[k][1] * (mj[1] - M[1] * inv) +
                         E[k][2] * (mj[2] - M[2] * inv);
                qm[k] += E[k][0] * d[0] + E[k][1] * d[1] + E[k][2] * d[2];
            }
        }
        node = nd.parent;
    }
    if (!FIRST) u = load_sums(a, s);
    const double ge = a.gE ? a.gE[b] : 0.0;
    const double *he = a.hext ? a.hext + 3 * b : nullptr;
    for (int k = 0; k < 3; ++k) {
        double ex = -0.5 * u.v[3 + k];
        if (he) ex -= he[k];
        dr[k] = u.v[k] - u.q[k] - B[k] + qr[k];
        dm[k] = u.q[3 + k] + A[k] + ge * ex + qm[k];
    }
}

}  // namespace ffbh
