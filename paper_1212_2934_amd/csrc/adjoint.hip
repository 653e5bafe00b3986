// Adjoint of the Barnes-Hut field: dL/dr and dL/dm for L = sum_i Hbar_i . H_i (+ the explicit
// dependence of E on m), with the tree, memberships and acceptance decisions of the forward pass held
// fixed.  The traversal is recomputed (nothing is stored from the forward pass): the same per-lane
// decisions are taken in the same order, and for every interaction
//   far (i, C):  dL/dr_i += g(x; Hbar_i, M_C);  B_C -= g;  A_C += T(x) Hbar_i      (x = r_i - c_C)
//   near (i, k): dL/dr_i += g(x; Hbar_i, m_k);  dL/dr_k -= g;  dL/dm_k += T(x) Hbar_i
// where g is the summand of the reduced dipolar force f_dip (Sec. 2) and T the dipole-field tensor of
// Eq. (H_dip).  Cell adjoints reach the members in a downward pass: every member k of C receives
// A_C in dL/dm_k and B_C / n_C in dL/dr_k (c_C is the mean of the members, Eq. magCenter).
// Scatters are reduced across the wave before one FP64 atomic per value.  The records hold the sums of
// +g (S_C = -B_C for a cell, the sum of g over a source's partners for a particle), and the downward pass
// subtracts them, so the scattered values need no negation.
#include "downward.h"
#include "traverse.h"

namespace ffbh {

__device__ inline void atomic_add_d(double *p, double v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Six scatter values of one wave added to six consecutive doubles at p (a 64-byte aligned record): the
// values are summed over the wave (lanes that do not contribute pass zeros) and the six lanes holding the
// totals add them with one atomic instruction, so the memory system sees one request per record.
// wcomp = total6_comp(lane).  Uniform control flow.
template <typename T>
__device__ inline void scatter6(uint64_t who, int lane, int wcomp, double *p, T v0, T v1, T v2, T v3, T v4, T v5)
{
    // reduced whatever `who` holds (no branch around the reduction, so the inputs need no copies); only
    // the atomic is skipped for an empty mask
    const T t = wave_total6<T>(lane, v0, v1, v2, v3, v4, v5);
    if (who != 0ull && wcomp >= 0) atomic_add_d(p + wcomp, (double)t);
}

// One pair of the fused traversal for a target with upstream field gradient a: adds the gathered dL/dr
// (g) and the field of b to the target's sums (FP32 partials since the last flush in MIXED mode, FP64
// otherwise) and returns g and T(x) a for the scatter.  Lanes with `use` false add and return zeros.
template <bool MIXED, typename T>
__device__ inline void fused_pair(bool use, T r2, T x, T y, T z, T ax, T ay, T az, T bx, T by, T bz, T &gx, T &gy,
                                  T &gz, T &tx, T &ty, T &tz, T &pgx, T &pgy, T &pgz, T &phx, T &phy, T &phz,
                                  double &grx, double &gry, double &grz, double &hx, double &hy, double &hz)
{
    if constexpr (MIXED) {
        T ug[3] = {pgx, pgy, pgz};
        adj_field_r2<T, true>(use, r2, x, y, z, ax, ay, az, bx, by, bz, gx, gy, gz, tx, ty, tz, phx, phy, phz, ug);
        pgx = ug[0]; pgy = ug[1]; pgz = ug[2];
    } else {
        adj_field_r2<T>(use, r2, x, y, z, ax, ay, az, bx, by, bz, gx, gy, gz, tx, ty, tz, hx, hy, hz);
        grx += gx; gry += gy; grz += gz;
    }
}

// Contact pairs of the FP32-mixed walk.  A chain bead's two neighbours pull it with forces of about 5 (in
// reduced units) in opposite directions, and its net force can be a thousand times smaller, so the FP32
// rounding of those two pairs (offset and arithmetic, about 1e-6 each) would dominate its error.  Direct
// pairs closer than 1.25 d (measured on the FP32 offset) are therefore listed per target during the walk
// and evaluated in FP64 after it, at most kCloseMax per target and wave (any further ones stay FP32).
constexpr int kCloseMax = 6;
constexpr float kClose2 = 1.5625f;  // (1.25 d)^2
template <bool ON>
struct CloseList {
};
template <>
struct CloseList<true> {
    uint32_t n[kWave];             // listed partners per target lane
    int32_t k[kWave][kCloseMax];   // their sorted indices
};

// LDS of the fused traversal (dynamic shared memory).  The targets: one record per wave of the block, or one
// for the block where its waves share their targets (split walks).
template <typename T>
struct AdjTargets {
    LdsTarget tgt[kWave];  // the wave's targets
    T hb[kWave][4];        // their upstream field gradients
};
// The rest: one record per wave.  A split walk lists lanes in bytes; sixteen records and the targets then take 62 KB in
// the FP32-mixed walk and 65 KB in FP64, so that two workgroups share a CU's 160 KB.
template <typename T, bool SPLIT>
struct AdjLds {
    T acc[kWave][6];  // direct-sum g (0..2) and field (3..5) of the current leaf, by owner lane
    T sbuf[16][6];    // member totals of the current chunk: sum g (0..2), sum T(x) a (3..5)
    typename std::conditional<SPLIT, uint8_t, int>::type list[kWave];  // lanes that opened the current leaf
    CloseList<std::is_same<T, float>::value> cl;  // contact pairs deferred to FP64 (FP32-mixed walk)
};
constexpr int kSplitMaxWaves = 16;
// A split walk's record also holds the wave's six FP64 sums per target at the end.
static_assert(sizeof(AdjLds<float, true>) >= 6 * kWave * sizeof(double) &&
                  sizeof(AdjLds<double, true>) >= 6 * kWave * sizeof(double),
              "the sums fit the record");
template <typename T, bool SPLIT>
constexpr size_t adj_lds_bytes(int waves)
{
    return (SPLIT ? 1 : waves) * sizeof(AdjTargets<T>) + waves * sizeof(AdjLds<T, SPLIT>);
}
static_assert(2 * adj_lds_bytes<float, true>(kSplitMaxWaves) <= kLdsPerCu &&
                  2 * adj_lds_bytes<double, true>(kSplitMaxWaves) <= kLdsPerCu,
              "two workgroups of a split walk share a CU's LDS");

// Direct sums of one leaf (first, count) for the c listed lanes, in groups of G lanes (see the compacted
// direct sums in traverse.h).  Lane b of group g pairs member b with listed target t0 + g: the group's
// totals of g and of the field go to the target's LDS slot; the member's totals over all listed targets
// are summed across the groups and added to its record with one atomic per component.
template <int G, typename T, bool SPLIT, typename Src>
__device__ inline void adj_leaf(AdjLds<T, SPLIT> &W, const AdjTargets<T> &A, int lane, const Src *__restrict__ sr, double *__restrict__ g_rm,
                                int first, int count, int c, bool &coincident)
{
    const int grp = lane / G, b = lane % G;
    for (int c0 = 0; c0 < count; c0 += G) {
        const int cn = min(G, count - c0);
        const bool sok = b < cn;
        const int k = first + c0 + (sok ? b : 0);
        const Src sk = sr[k];
        const T mx = (T)sk.mx, my = (T)sk.my, mz = (T)sk.mz;
        T s0 = 0, s1 = 0, s2 = 0, s3 = 0, s4 = 0, s5 = 0;
        for (int t0 = 0; t0 < c; t0 += kWave / G) {
            const int a = t0 + grp;
            const bool tok = a < c;
            const int tl = W.list[tok ? a : 0];
            const LdsTarget tg = A.tgt[tl];
            const T ax = A.hb[tl][0], ay = A.hb[tl][1], az = A.hb[tl][2];
            const T x = (T)(tg.rx - sk.x), y = (T)(tg.ry - sk.y), z = (T)(tg.rz - sk.z);
            const T r2 = norm2<T>(x, y, z);
            const bool other = tok && sok && k != tg.si;
            bool deferred = false;
            if constexpr (std::is_same<T, float>::value) {
                // a contact pair goes to the target's list (evaluated in FP64 after the walk) while it has room
                if (other && r2 > (T)0 && r2 < kClose2) {
                    const uint32_t q = __hip_atomic_fetch_add(&W.cl.n[tl], 1u, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_WAVEFRONT);
                    if (q < (uint32_t)kCloseMax) {
                        W.cl.k[tl][q] = k;
                        deferred = true;
                    }
                }
            }
            const bool use = other && r2 > (T)0 && !deferred;
            coincident |= other && !(r2 > (T)0);
            T qx, qy, qz, ux, uy, uz, hx = 0, hy = 0, hz = 0;
            adj_field_r2<T>(use, r2, x, y, z, ax, ay, az, mx, my, mz, qx, qy, qz, ux, uy, uz, hx, hy, hz);
            s0 += qx; s1 += qy; s2 += qz;
            s3 += ux; s4 += uy; s5 += uz;
            T o0, o1;
            group_sum6<G>(lane, qx, qy, qz, hx, hy, hz, o0, o1);
            if constexpr (G == 4) {
                const int j = lane & 3;  // holds slots 2j, 2j + 1
                if (tok && j < 3) {
                    lds_add(&W.acc[tl][2 * j], o0);
                    lds_add(&W.acc[tl][2 * j + 1], o1);
                }
            } else {
                if (tok && b < 6) lds_add(&W.acc[tl][b], o0);  // lane b < 6 holds slot b
            }
        }
        // sum g (subtracted from dL/dr_k downstream), dL/dm_k += sum T(x) a over the listed targets: the row
        // swaps move two of the six values each (rows 0..3 of x0 carry components 0, 2, 1, 3 and rows 0, 1 /
        // 2, 3 of x1 carry 4 / 5),
        // then lanes of equal member index inside a row are added
        const T w0 = swap32_pair(s0, s1), w1 = swap32_pair(s2, s3), w2 = swap32_pair(s4, s5);
        const T x0 = row_stride_sum<G>(swap16_pair(w0, w1)), x1 = row_stride_sum<G>(swap16_sum(w2));
        const int row = lane >> 4, p = lane & 15;
        if (p < cn) {
            W.sbuf[p][row == 0 ? 0 : row == 1 ? 2 : row == 2 ? 1 : 3] = x0;
            if ((row & 1) == 0) W.sbuf[p][4 + (row >> 1)] = x1;
        }
        wave_lds_sync();
        for (int base = 0; base < 6 * cn; base += kWave) {
            const int idx = base + lane;
            if (idx < 6 * cn) {
                const int m = idx / 6, comp = idx - 6 * m;
                const T v = W.sbuf[m][comp];
                if (v != (T)0) atomic_add_d(g_rm + 8 * (int64_t)(first + c0 + m) + comp, (double)v);
            }
        }
        wave_lds_sync();
    }
}

// The deferred contact pairs of one target lane, in FP64: offset from the FP64 positions, pair arithmetic
// with the FP64 upstream gradient and source moment; g and the field go to the lane's FP64 sums, the
// member's share (g and T(x) a) to its record with FP64 atomics.  Lanes walk their own lists together.
template <bool SPLIT>
__device__ inline void close_pairs(AdjLds<float, SPLIT> &W, int lane, bool valid, int si, double rx, double ry, double rz,
                                   const double *__restrict__ spos, const double *__restrict__ smom,
                                   const double *__restrict__ hbar, int64_t ntot, double *__restrict__ g_rm,
                                   double &grx, double &gry, double &grz, double &hx, double &hy, double &hz)
{
    wave_lds_sync();
    const uint32_t listed = valid ? W.cl.n[lane] : 0u;
    const int cnt = listed < (uint32_t)kCloseMax ? (int)listed : kCloseMax;
    const double ax = valid ? hbar[si] : 0.0, ay = valid ? hbar[ntot + si] : 0.0,
                 az = valid ? hbar[2 * ntot + si] : 0.0;
    for (int q = 0; q < kCloseMax; ++q) {
        const bool on = q < cnt;
        if (ballot(on) == 0ull) break;
        const int k = on ? W.cl.k[lane][q] : si;
        const double x = rx - spos[k], y = ry - spos[ntot + k], z = rz - spos[2 * ntot + k];
        const double bx = smom[k], by = smom[ntot + k], bz = smom[2 * ntot + k];
        double gx, gy, gz, tx, ty, tz;
        adj_field_r2<double>(on, norm2<double>(x, y, z), x, y, z, ax, ay, az, bx, by, bz, gx, gy, gz, tx, ty, tz,
                             hx, hy, hz);
        grx += gx; gry += gy; grz += gz;
        if (on) {
            double *r = g_rm + 8 * (int64_t)k;
            atomic_add_d(r, gx); atomic_add_d(r + 1, gy); atomic_add_d(r + 2, gz);
            atomic_add_d(r + 3, tx); atomic_add_d(r + 4, ty); atomic_add_d(r + 5, tz);
        }
    }
}

// The order of the arguments decides which of them the compiler keeps in scalar registers through the walk: with
// status between Hs and n the FP32-mixed walk read four back from vector lanes at every leaf, 0.4 % of an MD step.
#define FFBH_ADJ_PARAMS                                                                                         \
    const NodeRec *__restrict__ nodes, const double *__restrict__ node_m64, const double *__restrict__ spos,    \
        const double *__restrict__ smom, const void *__restrict__ src, const double *__restrict__ hbar,         \
        double *__restrict__ g_gather, double *__restrict__ g_rm, double *__restrict__ node_adj, int64_t n,     \
        int64_t ntot, double *__restrict__ Hs, uint32_t *__restrict__ status, int waves_per_seg,                \
        int num_waves, double theta2, int max_nodes, int tpw, int parts, double *__restrict__ part_buf,         \
        uint32_t *__restrict__ wave_cost, const void *__restrict__ node_q, double *__restrict__ node_adjq,      \
        const uint32_t *__restrict__ tgt_order, int inside_test
#define FFBH_ADJ_ARGS                                                                                           \
    nodes, node_m64, spos, smom, src, hbar, g_gather, g_rm, node_adj, n, ntot, Hs, status, waves_per_seg,       \
        num_waves, theta2, max_nodes, tpw, parts, part_buf, wave_cost, node_q, node_adjq, tgt_order, inside_test

// The fused walk of wave item gw.  If wave_cost is not null, lane 0 stores there a deterministic measure of
// the item's work (node visits plus leaf pair rounds), which orders the next launch.  QUAD: order-2 cells
// (node_q holds each node's first moment D, stride 16); an accepted cell adds its first-moment field, its
// gradient to the target and (negated) to the cell centre, and d/dD to node_adjq (six values, stride 8).
// SCALED: the node records hold s^2 / theta^2 and the acceptance test is s2 < d^2 (kMacScaled).  SPLIT: the
// block's waves (a power of two) share the item's targets and divide the tree by sorted positions, as in the
// forward walk (k_field): interval q of 2^split_shift positions belongs to wave q mod W; in the FP64 walk with a
// negative split_shift node i belongs to wave i mod W instead, and all waves descend.  Every far cell and
// every leaf is summed and scattered by one wave, an FP32-mixed wave sums whole segments between two leaf
// visits, and the FP64 sums of the targets meet in LDS, in wave order.
template <bool MIXED, bool QUAD, bool SCALED, bool SPLIT>
__device__ __forceinline__ void adjoint_wave(int gw, int split_shift, FFBH_ADJ_PARAMS)
{
    using T = typename std::conditional<MIXED, float, double>::type;
    using Src = typename std::conditional<MIXED, Src32, Src64>::type;
    const Src *__restrict__ sr = (const Src *)src;
    const int lane = threadIdx.x & (kWave - 1);
    const int wcomp = total6_comp(lane);
    // a wave owns tpw consecutive targets (lanes at and above tpw stay idle) and, with parts > 1, walks
    // the subtree of one child of the root (part p: child p); the parts' sums meet in downward()
    const int per_seg = waves_per_seg * parts;
    const int seg = gw / per_seg;
    const int grp = (gw - seg * per_seg) / parts, part = gw - seg * per_seg - grp * parts;
    const int local = grp * tpw + lane;
    const bool valid = lane < tpw && local < n;
    const int si = target_of(tgt_order, seg, n, local, valid);
    const double rx = spos[si], ry = spos[ntot + si], rz = spos[2 * ntot + si];
    const T ax = valid ? (T)hbar[si] : (T)0, ay = valid ? (T)hbar[ntot + si] : (T)0,
            az = valid ? (T)hbar[2 * ntot + si] : (T)0;

    double grx = 0.0, gry = 0.0, grz = 0.0;  // gathered dL/dr of the target (FP64)
    double hx = 0.0, hy = 0.0, hz = 0.0;     // forward field of the target (FP64)
    T pgx = 0, pgy = 0, pgz = 0, phx = 0, phy = 0, phz = 0;  // partial sums since the last flush
    bool coincident = false;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), waves = (int)(blockDim.x / kWave);
    // the waves of a split walk write the same targets to one record (each reads what it has written itself)
    unsigned char *rec = SPLIT ? ffbh_dyn_lds + sizeof(AdjTargets<T>) + (threadIdx.x / kWave) * sizeof(AdjLds<T, SPLIT>)
                               : ffbh_dyn_lds + (threadIdx.x / kWave) * adj_lds_bytes<T, SPLIT>(1) +
                                     sizeof(AdjTargets<T>);
    AdjTargets<T> &A = *(AdjTargets<T> *)(SPLIT ? ffbh_dyn_lds : rec - sizeof(AdjTargets<T>));
    AdjLds<T, SPLIT> &W = *(AdjLds<T, SPLIT> *)rec;
    A.tgt[lane] = LdsTarget{rx, ry, rz, si, 0};
    A.hb[lane][0] = ax; A.hb[lane][1] = ay; A.hb[lane][2] = az;
#pragma unroll
    for (int j = 0; j < 6; ++j) W.acc[lane][j] = (T)0;
    if constexpr (MIXED) W.cl.n[lane] = 0u;

    LaneStack st;
    if (parts == 1) {
        st.init(seg, 1, ballot(valid));
    } else {
        // the root holds every target of the system, so it is always opened: start at child `part` (a leaf
        // root is walked by part 0 alone)
        const NodeRec r = nodes[seg];
        const bool leaf_root = r.nchild == 0;
        const int first = leaf_root ? seg : r.child + part;
        int cnt = leaf_root ? (part == 0 ? 1 : 0) : (part < r.nchild ? 1 : 0);
        if (cnt > 0 && (unsigned)first >= (unsigned)max_nodes) {
            if (lane == 0) set_flag(status, BH_FLAG_TREE);
            cnt = 0;
        }
        st.init(first, cnt, ballot(valid));
    }
    // Node indices are checked where they enter the stack (the root above, child ranges at the push), so
    // every visited node is in [0, max_nodes); a wave pushes each internal node's children at most once,
    // so at most max_nodes pushes keep the walk finite whatever the tree holds.
    int guard = max_nodes;
    uint32_t work = 0;      // node visits plus leaf pair rounds (wave-uniform)
    const int seg0 = (int)(seg * n);
    bool live = !SPLIT || (MIXED && wave == 0);  // whether what is visited now is this wave's to sum
    while (st.more_any()) {
        uint64_t mask;
        const int cur = st.pop(mask);
        const NodeRec nd = nodes[cur];
        ++work;
        bool own = true;
        if (SPLIT && !MIXED && split_shift < 0) {
            // by node: the waves take turns at the children of a cell, and all descend
            own = live = (cur & (waves - 1)) == wave;
            if (!live && nd.nchild == 0) continue;
        } else if constexpr (SPLIT) {
            const int q0 = (nd.first - seg0) >> split_shift, q1 = (nd.first - seg0 + nd.count - 1) >> split_shift;
            own = ((q0 ^ wave) & (waves - 1)) == 0;
            if constexpr (!MIXED) live = own;
            // none of this wave's positions in the cell
            if (!live && ((wave - q0) & (waves - 1)) > q1 - q0) continue;
        }
        // masks of the lanes that take part, of the targets inside the node (opened whatever the test
        // says; below kSelfRejectTheta2 the test rejects them itself) and of the acceptance test
        uint64_t insm = 0ull;
        if (inside_test) insm = ballot((unsigned)(si - nd.first) < (unsigned)nd.count);
        const double dx = rx - nd.cx, dy = ry - nd.cy, dz = rz - nd.cz;
        const double d2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
        const uint64_t accm = mask & ~insm & ballot(SCALED ? nd.s2 < d2 : nd.s2 < theta2 * d2);
        const bool acc = lane_in(accm);
        if (accm != 0ull && live) {
            // the whole wave evaluates the pair (lanes that do not accept add zeros)
            T bx, by, bz;
            if (MIXED) {
                bx = (T)nd.mx; by = (T)nd.my; bz = (T)nd.mz;
            } else {
                const double *m = node_m64 + 4 * (int64_t)cur;
                bx = (T)m[0]; by = (T)m[1]; bz = (T)m[2];
            }
            T gx, gy, gz, tx, ty, tz;
            fused_pair<MIXED, T>(acc, (T)d2, (T)dx, (T)dy, (T)dz, ax, ay, az, bx, by, bz, gx, gy, gz, tx, ty, tz,
                                 pgx, pgy, pgz, phx, phy, phz, grx, gry, grz, hx, hy, hz);
            T e0 = 0, e1 = 0, e2 = 0, e3 = 0, e4 = 0, e5 = 0;
            if constexpr (QUAD) {
                const T *qd = (const T *)node_q + 16 * (int64_t)cur;
                T Gx, Gy, Gz;
                first_moment_adj_r2<T>(acc, (T)d2, (T)dx, (T)dy, (T)dz, qd, ax, ay, az, Gx, Gy, Gz, e0, e1, e2, e3, e4,
                                       e5);
                if constexpr (MIXED) {
                    first_moment_acc_r2<T>(acc, (T)d2, (T)dx, (T)dy, (T)dz, qd, phx, phy, phz);
                    pgx += Gx; pgy += Gy; pgz += Gz;
                } else {
                    first_moment_acc_r2<T>(acc, (T)d2, (T)dx, (T)dy, (T)dz, qd, hx, hy, hz);
                    grx += Gx; gry += Gy; grz += Gz;
                }
                gx += Gx; gy += Gy; gz += Gz;
            }
            // A_C += sum T(x) Hbar over the accepting lanes, S_C += sum g (B_C = -S_C)
            scatter6<T>(accm, lane, wcomp, node_adj + 8 * (int64_t)cur, tx, ty, tz, gx, gy, gz);
            if constexpr (QUAD) scatter6<T>(accm, lane, wcomp, node_adjq + 8 * (int64_t)cur, e0, e1, e2, e3, e4, e5);
        }
        // One loop exit and one back edge: error exits clear the stack instead of breaking, so that the
        // accumulators stay in the same registers on every path (no copies at the merges).
        const uint64_t open = mask & ~accm;
        if (open != 0ull) {
            if (nd.nchild != 0) {
                if (--guard < 0 || nd.child < 0 || nd.nchild > 8 || nd.child + nd.nchild > max_nodes) {
                    if (lane == 0) set_flag(status, BH_FLAG_TREE);
                    st.clear();
                } else if (st.sp >= kStackMax) {
                    if (lane == 0) set_flag(status, BH_FLAG_STACK);
                    st.clear();
                } else {
                    st.push(lane, nd.child, nd.nchild, open);
                }
            } else if (nd.first < 0 || nd.count < 1 || (uint32_t)nd.first + (uint32_t)nd.count > (uint32_t)ntot) {
                // the member range is checked here, where it is first used to index memory
                if (lane == 0) set_flag(status, BH_FLAG_TREE);
                st.clear();
            } else if (!live) {
                live = own;
            } else {
                // leaf: direct sums over its members, packed over the lanes that opened it
                if constexpr (SPLIT) live = own;
                if (lane_in(open)) W.list[lanes_below(open)] = lane;
                const int c = __builtin_popcountll(open);
                wave_lds_sync();
                if (nd.count <= 4) adj_leaf<4>(W, A, lane, sr, g_rm, nd.first, nd.count, c, coincident);
                else if (nd.count <= 8) adj_leaf<8>(W, A, lane, sr, g_rm, nd.first, nd.count, c, coincident);
                else adj_leaf<16>(W, A, lane, sr, g_rm, nd.first, nd.count, c, coincident);
                {
                    const int G = nd.count <= 4 ? 4 : nd.count <= 8 ? 8 : 16;
                    work += (uint32_t)(((nd.count + G - 1) / G) * ((c * G + kWave - 1) / kWave + 1));
                }
                T d[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    d[j] = W.acc[lane][j];
                    W.acc[lane][j] = (T)0;
                }
                if (MIXED) {
                    grx += (double)(pgx + d[0]); gry += (double)(pgy + d[1]); grz += (double)(pgz + d[2]);
                    hx += (double)(phx + d[3]); hy += (double)(phy + d[4]); hz += (double)(phz + d[5]);
                    pgx = pgy = pgz = phx = phy = phz = (T)0;
                } else {
                    grx += (double)d[0]; gry += (double)d[1]; grz += (double)d[2];
                    hx += (double)d[3]; hy += (double)d[4]; hz += (double)d[5];
                }
            }
        }
    }
    if constexpr (MIXED) {
        grx += (double)pgx; gry += (double)pgy; grz += (double)pgz;
        hx += (double)phx; hy += (double)phy; hz += (double)phz;
        close_pairs(W, lane, valid, si, rx, ry, rz, spos, smom, hbar, ntot, g_rm, grx, gry, grz, hx, hy, hz);
    }
    if (ballot(coincident) != 0ull && lane == 0) set_flag(status, BH_FLAG_COINCIDENT);
    if constexpr (SPLIT) {
        wave_lds_sync();
        double *sums = (double *)rec;
        const double mine[6] = {grx, gry, grz, hx, hy, hz};
#pragma unroll
        for (int c = 0; c < 6; ++c) sums[c * kWave + lane] = mine[c];
        __syncthreads();
        if (wave != 0) return;
        for (int w = 1; w < waves; ++w) {
            const double *o = (const double *)(rec + w * sizeof(AdjLds<T, SPLIT>)) + lane;
            grx += o[0]; gry += o[kWave]; grz += o[2 * kWave];
            hx += o[3 * kWave]; hy += o[4 * kWave]; hz += o[5 * kWave];
        }
    }
    if (wave_cost && lane == 0) wave_cost[gw] = work;
    if (parts > 1) {
        if (valid) {
            double *q = part_buf + (int64_t)part * 6 * ntot;
            q[si] = grx; q[ntot + si] = gry; q[2 * ntot + si] = grz;
            q[3 * ntot + si] = hx; q[4 * ntot + si] = hy; q[5 * ntot + si] = hz;
        }
        return;
    }

    if (valid) {
        g_gather[si] = grx;
        g_gather[ntot + si] = gry;
        g_gather[2 * ntot + si] = grz;
        Hs[si] = hx;
        Hs[ntot + si] = hy;
        Hs[2 * ntot + si] = hz;
    }
}

// Independent-wave fused traversal.  Without work counters every wave takes one item: its global wave
// index, or with `order` the item at that place of the order (light items of the previous launch last,
// so the launch does not end on a long item).  With work counters the launch is persistent: each wave
// takes item after item in the order given, until the items run out.  Every wave reaches the exit: the
// counters only grow.
// Waves per SIMD: five for the FP32-mixed walk with the paper's cells (96 VGPRs, a few spilled bytes;
// 3 % faster MD step than at four), four for the others (the FP64 walk fits 128 VGPRs and runs 7 % faster
// than at three, but spills heavily at five).
// Segments of the persistent launch's item order: segment x holds the items i with i * kXcds / nw == x,
// which start at ceil(x nw / kXcds).
constexpr int kXcds = 8;
__host__ __device__ inline uint32_t order_segment_start(int x, int nw)
{
    return (uint32_t)(((int64_t)x * nw + kXcds - 1) / kXcds);
}

template <bool MIXED, bool QUAD, bool SCALED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MIXED && !QUAD ? 5 : 4))) void k_adjoint(
    FFBH_ADJ_PARAMS, const uint32_t *__restrict__ order, uint32_t *__restrict__ work_ctr)
{
    if (!work_ctr) {
        // one wave per item; with an order, wave lin takes item order[lin] (heavy items of the previous
        // launch first within each XCD's range, light ones last)
        const int wpb = blockDim.x / kWave;
        const int lin = xcd_block(blockIdx.x, gridDim.x) * wpb + (int)(threadIdx.x / kWave);
        if (lin >= num_waves) return;
        int gw = lin;
        if (order) {
            const uint32_t o = order[lin];
            if (o < (uint32_t)num_waves) gw = (int)o;
        }
        adjoint_wave<MIXED, QUAD, SCALED, false>(gw, 0, FFBH_ADJ_ARGS);
        return;
    }
    // The items are split into kXcds contiguous segments (neighbouring items share tree data).  Workgroups
    // are dispatched to the XCDs round-robin, so workgroup b runs on XCD b mod kXcds: its waves take items
    // of that XCD's segment first, keeping its L2 on one part of the tree, and then help the other
    // segments.  Each segment has its own work counter, which only grows, so every wave reaches the exit.
    const int lane = threadIdx.x & (kWave - 1);
    const int home = (int)(blockIdx.x % kXcds);
    for (int k = 0; k < kXcds; ++k) {
        const int sg = (home + k) % kXcds;
        const uint32_t s0 = order_segment_start(sg, num_waves), len = order_segment_start(sg + 1, num_waves) - s0;
        for (;;) {
            uint32_t v = 0u;
            if (lane == 0) v = atomicAdd(work_ctr + sg, 1u);
            const uint32_t item = __builtin_amdgcn_readfirstlane(v);
            if (item >= len) break;
            const uint32_t gw = order[s0 + item];
            if (gw >= (uint32_t)num_waves) {
                if (lane == 0) set_flag(status, BH_FLAG_TREE);
                return;
            }
            adjoint_wave<MIXED, QUAD, SCALED, false>((int)gw, 0, FFBH_ADJ_ARGS);
        }
    }
}

// The split walk: one block per item, its waves share the item's 64 targets.  The FP64 walk and the order-2
// walks take up to 128 VGPRs (four waves per SIMD), the FP32-mixed walk with the paper's cells 96.
template <bool MIXED, bool QUAD, bool SCALED>
__global__ __launch_bounds__(kSplitMaxWaves *kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_adjoint_split(
    FFBH_ADJ_PARAMS, int split_shift)
{
    adjoint_wave<MIXED, QUAD, SCALED, true>(xcd_block(blockIdx.x, gridDim.x), split_shift, FFBH_ADJ_ARGS);
}

// Order of the wave items of the next persistent launch, from the previous launch's costs, within each of
// the kXcds segments of consecutive items: the items outside the lightest ~45 % (of the whole launch)
// first, in index order (neighbouring items share tree data, so the launch keeps its cache locality), then
// the light items, heaviest first (64 buckets of the cost range), so each segment ends on short items.  One
// workgroup per segment: each finds the cost range and the light buckets from all items, then sorts its own
// segment by a stable counting sort and resets its work counter.  Costs all zero (first launch) give the
// index order.  (One workgroup for all segments, with serial scans over 512 keys, took 62 us at 16384 items.)
constexpr int kOrderThreads = 1024;
constexpr int kOrderBins = 64;
// Share of the items moved to the end of their segment (measured at 2^20: 15 % and 30 % slower, 60 % and
// 75 % slower again; 45 % the fastest in both precisions).
constexpr uint32_t kLightPercent = 45u;

__global__ __launch_bounds__(kOrderThreads) void k_order_waves(const uint32_t *__restrict__ cost, int nw,
                                                               uint32_t *__restrict__ order,
                                                               uint32_t *__restrict__ work_ctr)
{
    constexpr int kWaves = kOrderThreads / kWave;
    static_assert(kOrderBins == kWave, "one lane per bucket");
    __shared__ uint32_t red[kWaves];
    __shared__ uint32_t fine[kOrderBins];  // items per cost bucket, lightest bucket first
    __shared__ uint32_t hist[kOrderBins];  // items of the segment per class, then the start of each class
    __shared__ uint32_t wcnt[kWaves][kOrderBins];
    __shared__ int split;                  // buckets below it are the light items
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave, seg = blockIdx.x;
    uint32_t mx = 0u;
    for (int i = t; i < nw; i += kOrderThreads) mx = max(mx, cost[i]);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, kWave));
    if (lane == 0) red[wave] = mx;
    if (t < kOrderBins) fine[t] = hist[t] = 0u;
    __syncthreads();
    uint32_t cmax = 0u;
    for (int w = 0; w < kWaves; ++w) cmax = max(cmax, red[w]);
    auto bucket = [cmax](uint32_t c) -> int { return (int)((uint64_t)c * kOrderBins / ((uint64_t)cmax + 1u)); };
    for (int i = t; i < nw; i += kOrderThreads) atomicAdd(&fine[bucket(cost[i])], 1u);
    __syncthreads();
    auto wave_scan = [lane](uint32_t v) {  // inclusive
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t x = (uint32_t)__shfl_up((int)v, off, kWave);
            if (lane >= off) v += x;
        }
        return v;
    };
    if (wave == 0) {
        // the light items: the lowest buckets holding at most kLightPercent % of the items (bucket 63 holds the
        // heaviest item and all items are more than that, so split <= 63)
        const uint32_t acc = wave_scan(fine[lane]);
        const uint64_t light = ballot((uint64_t)acc * 100u <= (uint64_t)nw * kLightPercent);
        if (lane == 0) split = __builtin_popcountll(light);
    }
    __syncthreads();
    const int sp = split;
    const int s0 = (int)order_segment_start(seg, nw), s1 = (int)order_segment_start(seg + 1, nw);
    // class 0: heavy items; class k = 1..split: light bucket split - k (heaviest light bucket first)
    auto class_of = [&](uint32_t c) -> int {
        const int q = bucket(c);
        return q >= sp ? 0 : sp - q;
    };
    for (int i = s0 + t; i < s1; i += kOrderThreads) atomicAdd(&hist[class_of(cost[i])], 1u);
    __syncthreads();
    if (wave == 0) {
        const uint32_t h = hist[lane];
        hist[lane] = (uint32_t)s0 + wave_scan(h) - h;
    }
    __syncthreads();
    for (int c0 = s0; c0 < s1; c0 += kOrderThreads) {
        wcnt[wave][lane] = 0u;
        const int i = c0 + t;
        const bool ok = i < s1;
        const int b = ok ? class_of(cost[i]) : 0;
        // lanes of this wave with the same class, and this lane's rank among them
        uint64_t m = ballot(ok);
#pragma unroll
        for (int bit = 0; bit < 6; ++bit) {
            const bool set = (b >> bit) & 1;
            const uint64_t v = ballot(set);
            m &= set ? v : ~v;
        }
        const int before = lanes_below(m);
        if (ok && before == 0) wcnt[wave][b] = (uint32_t)__builtin_popcountll(m);
        __syncthreads();
        if (t < kOrderBins) {
            uint32_t acc = hist[t];
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = wcnt[w][t];
                wcnt[w][t] = acc;
                acc += c;
            }
            hist[t] = acc;
        }
        __syncthreads();
        if (ok) {
            const uint32_t at = wcnt[wave][b] + (uint32_t)before;
            if (at < (uint32_t)nw) order[at] = (uint32_t)i;
        }
        __syncthreads();
    }
    if (t == 0) work_ctr[seg] = 0u;
}

__global__ __launch_bounds__(256) void k_adj_setup(AdjSetup a)
{
    adj_setup(a, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256);
}

// Gradients of the sorted particles, to caller order: one thread each, five waves per SIMD to hide the path's loads.
// Bound by the six scattered stores of a particle: 71 to 80 us at 2^20 from run to run, 205 us at 32 x 65536; one path
// per distinct leaf of a workgroup instead took 73 and 205.
__global__ __launch_bounds__(256, 5) void k_downward(Downward a, double *__restrict__ dpos, double *__restrict__ dmom)
{
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= a.ntot) return;
    const int64_t o = a.perm[s], b = o / a.n, i = o - b * a.n;
    if (o >= a.ntot) return;
    double dr[3], dm[3];
    downward<false>(a, s, b, dr, dm);
    for (int k = 0; k < 3; ++k) dpos[b * 3 * a.n + k * a.n + i] = dr[k];
    for (int k = 0; k < 3; ++k) dmom[b * 3 * a.n + k * a.n + i] = dm[k];
}

// dL/dH_ext = -dL/dE * sum_i m_i: partial sums of a system's moments over nb workgroups, then one wave per
// system folds them in order.  (One workgroup per system read 2^18 moments in 84 us.)
__global__ __launch_bounds__(256) void k_dhext_part(const double *__restrict__ mom, int64_t n,
                                                    double *__restrict__ part)
{
    __shared__ double red[3][256];
    const int b = blockIdx.y;
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        for (int a = 0; a < 3; ++a) s[a] += mom[(int64_t)b * 3 * n + a * n + i];
    for (int a = 0; a < 3; ++a) red[a][threadIdx.x] = s[a];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int a = 0; a < 3; ++a) red[a][threadIdx.x] += red[a][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) part[((int64_t)b * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = red[threadIdx.x][0];
}

__global__ __launch_bounds__(64) void k_dhext(const double *__restrict__ part, const double *__restrict__ gE, int nb,
                                              double *__restrict__ dhext)
{
    const int b = blockIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < nb; k += kWave)
        for (int a = 0; a < 3; ++a) s[a] += part[((int64_t)b * nb + k) * 3 + a];
    for (int a = 0; a < 3; ++a) s[a] = wave_sum(s[a]);
    if (threadIdx.x < 3) dhext[3 * b + threadIdx.x] = gE ? -gE[b] * (threadIdx.x == 0 ? s[0] : threadIdx.x == 1 ? s[1] : s[2]) : 0.0;
}

// Whether one wave (or, divided, one group) takes each 64 targets in index order: no part, no order of items.
static bool adjoint_plain(const Handle &h) { return h.adj_parts == 1 && h.adj_sched == 0 && h.adj_tpw == kWave; }
// Targets per item.
static int adjoint_targets(const Handle &h) { return adjoint_plain(h) ? walk_targets(h) : h.adj_tpw; }

// Items of the independent-wave fused traversal: (system, target wave, part).
static int adjoint_items(const Handle &h)
{
    const int tpw = adjoint_targets(h), wps = (int)((h.L.n + tpw - 1) / tpw);
    return (int)(h.L.B * wps * h.adj_parts);
}

// Waves that share a fused walk: the forward walk's rule, for the shapes of one wave per item in index order (the
// others have their own way to order the work).  Measured on the kernel,
// FP64 / FP32-mixed, undivided -> divided: 1000 particles 282 / 285 -> 60 / 62 us, 4096 451 / 459 -> 105 / 118 us,
// 20000 818 / 804 -> 271 / 300 us, 50000 838 / 759 -> 474 / 424 us, 64 systems of 1000 294 / 309 -> 187 / 168 us;
// at 131072 particles four waves take 1545 / 1529 us against 1301 / 1203.
// Above that the FP64 walk still gains from two waves that take turns at the nodes (shift -1): the work is dealt
// out evenly and only the opened cells are tested twice, where intervals long enough to be skipped leave most of a
// group's near cells to one wave (131072 particles: 1281 us undivided, 1436 with intervals, 1193 by node; with four waves
// and more intervals are ahead).  Up to 2560 groups: two waves of 2048 groups are one round of the chip at four waves a
// SIMD, and the gain of the shorter walks ends soon after.  bh_build and gradient, undivided over by node: 2344 to 2560
// groups 1.03 (13000 x 12) to 1.14 (30000 x 5), alone 160000 0.99; 2626 to 2700 0.93 (1000 x 168) to 1.05 (5000 x 34),
// alone 0.98; 3060 13000 x 15 0.93, 3130 20000 x 10 0.92; alone 185600 0.91, 198400 1.01.
// Shapes of fewer targets or of a part of the tree per item follow the same rule by their items, with sixteen waves
// up to 256 (256 items of 16 targets: 101 us with eight, 88 with sixteen; 500: 152 and 194); a walk of a part
// sees an eighth of the positions, so its intervals are a twelfth of that, and no shorter than deals a group's near
// cells to all waves.  FP32-mixed, undivided -> divided: 1000 particles 171 -> 47 us (16 targets), 92 -> 33 (parts),
// 62 -> 27 (16 targets and parts); 4096 275 -> 88 (16 targets), 159 -> 61 (parts), 20000 526 -> 436 (16 targets,
// 1250 items, four waves); 8000 (16 targets and parts, 4000 items) 217 -> 243 with four.
static int adjoint_split(const Handle &h, int &shift)
{
    if (h.adj_sched != 0) return 1;
    const bool plain = adjoint_plain(h);
    const int64_t items = plain ? h.L.num_waves : adjoint_items(h);
    const int W = !plain && items <= 256 ? kSplitMaxWaves : walk_split(items);
    if (h.adj_parts > 1) {
        const int64_t want = h.L.n / (12 * h.adj_parts), least = 128 / W, len = want > least ? want : least;
        for (shift = 0; ((int64_t)2 << shift) <= len;) ++shift;
        return W;
    }
    shift = split_shift(h.L.n, W);
    if (W == 1 && plain && h.p.precision == BH_FP64 && items <= 2560) {
        shift = -1;
        return 2;
    }
    return W;
}

bool uses_wave_order(const Handle &h) { return h.adj_sched && h.adj_parts == 1; }

void launch_order_items(const uint32_t *cost, int nw, uint32_t *order, uint32_t *work_ctr, hipStream_t s)
{
    hipLaunchKernelGGL(k_order_waves, dim3(kXcds), dim3(kOrderThreads), 0, s, cost, nw, order, work_ctr);
}

void launch_order_waves(Handle &h, hipStream_t s)
{
    launch_order_items(h.w.wave_cost, adjoint_items(h), h.w.wave_order, h.w.sched_ctr, s);
}

hipError_t launch_backward(Handle &h, const double *d_mom, const double *d_hext, const double *d_gH,
                           const double *d_gE, double *d_dpos, double *d_dmom, double *d_dhext, hipStream_t s,
                           bool moments_done, bool order_done, bool setup_done, bool enter)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    if (!moments_done) {
        hipError_t e = launch_upward_moments(h, d_mom, s, enter);  // pseudo-particle moments
        if (e != hipSuccess) return e;
    }
    const bool quad = L.expansion == 2;
    if (!setup_done)
        hipLaunchKernelGGL(k_adj_setup, dim3(grid_for(L.ntot, 256, 4096)), dim3(256), 0, s, adj_setup_args(h, d_gH, d_gE));
    const int wpb = h.waves_per_block;
    const double theta2 = h.p.theta * h.p.theta;
    if (h.ev[2]) (void)hipEventRecord(h.ev[2], s);
    const bool mixed = h.p.precision == BH_FP32_MIXED;
    {
        const int tpw = adjoint_targets(h), parts = h.adj_parts;
        const int wps = (int)((L.n + tpw - 1) / tpw);
        const int nwv = adjoint_items(h);
        const unsigned blk = (unsigned)((nwv + wpb - 1) / wpb);
        // cost-ordered launches: persistent (adj_sched 1: as many workgroups as can be resident at once,
        // items from per-XCD work counters) or one wave per item in that order (adj_sched 2)
        const bool sched = uses_wave_order(h);
        if (sched && !order_done) launch_order_waves(h, s);
        const bool persistent = sched && h.adj_sched == 1;
        const unsigned grid = persistent && (unsigned)h.adj_resident < blk ? (unsigned)h.adj_resident : blk;
        const uint32_t *ord = sched ? w.wave_order : nullptr;
        uint32_t *ctr = persistent ? w.sched_ctr : nullptr;
        uint32_t *cost = parts == 1 ? w.wave_cost : nullptr;
        const void *nq = mixed ? (const void *)w.node_q32 : (const void *)w.node_q64;
        const uint32_t *tgt = uses_target_order(L) ? w.tgt_order : nullptr;
        const int mac = mac_form(theta2);
        const int inside = mac == kMacInside ? 1 : 0;
        const bool scaled = mac == kMacScaled;
#define FFBH_ADJ(MX, QD, SC, T)                                                                                 \
    hipLaunchKernelGGL((k_adjoint<MX, QD, SC>), dim3(grid), dim3(wpb * kWave), (adj_lds_bytes<T, false>(wpb)), s, \
                       w.nodes, w.node_m64, w.spos, w.smom, MX ? w.src32 : w.src64, w.hbar, w.g_gather, w.g_rm, \
                       w.node_adj, L.n, L.ntot, w.Hs, w.status, wps, nwv, theta2, (int)L.max_nodes, tpw, parts, \
                       w.part_buf, cost, nq, w.node_adjq, tgt, inside, ord, ctr)
        int shift = 0;
        const int W = adjoint_split(h, shift);
#define FFBH_ADJ_SPLIT(MX, QD, SC, T)                                                                           \
    hipLaunchKernelGGL((k_adjoint_split<MX, QD, SC>), dim3((unsigned)nwv), dim3(W * kWave),                     \
                       (adj_lds_bytes<T, true>(W)), s, w.nodes, w.node_m64, w.spos, w.smom,                     \
                       MX ? w.src32 : w.src64, w.hbar, w.g_gather, w.g_rm, w.node_adj, L.n, L.ntot, w.Hs, w.status, \
                       wps, nwv, theta2, (int)L.max_nodes, tpw, parts, w.part_buf, nullptr, nq, w.node_adjq, tgt, \
                       inside, shift)
        if (W > 1) {
            if (scaled) {
                if (mixed && quad) FFBH_ADJ_SPLIT(true, true, true, float);
                else if (mixed) FFBH_ADJ_SPLIT(true, false, true, float);
                else if (quad) FFBH_ADJ_SPLIT(false, true, true, double);
                else FFBH_ADJ_SPLIT(false, false, true, double);
            } else {
                if (mixed && quad) FFBH_ADJ_SPLIT(true, true, false, float);
                else if (mixed) FFBH_ADJ_SPLIT(true, false, false, float);
                else if (quad) FFBH_ADJ_SPLIT(false, true, false, double);
                else FFBH_ADJ_SPLIT(false, false, false, double);
            }
        } else if (scaled) {
            if (mixed && quad) FFBH_ADJ(true, true, true, float);
            else if (mixed) FFBH_ADJ(true, false, true, float);
            else if (quad) FFBH_ADJ(false, true, true, double);
            else FFBH_ADJ(false, false, true, double);
        } else {
            if (mixed && quad) FFBH_ADJ(true, true, false, float);
            else if (mixed) FFBH_ADJ(true, false, false, float);
            else if (quad) FFBH_ADJ(false, true, false, double);
            else FFBH_ADJ(false, false, false, double);
        }
#undef FFBH_ADJ
#undef FFBH_ADJ_SPLIT
    }
    if (h.ev[3]) (void)hipEventRecord(h.ev[3], s);
    if (d_dpos)
        hipLaunchKernelGGL(k_downward, dim3(grid_for(L.ntot, 256)), dim3(256), 0, s, downward_args(h, d_hext, d_gE),
                           d_dpos, d_dmom);
    if (d_dhext) {
        // the build's partial boxes are free here
        const int nb = (int)(L.n < 256 * kBboxBlocks ? (L.n + 255) / 256 : kBboxBlocks);
        hipLaunchKernelGGL(k_dhext_part, dim3((unsigned)nb, (unsigned)L.B), dim3(256), 0, s, d_mom, L.n, w.bbox_part);
        hipLaunchKernelGGL(k_dhext, dim3((unsigned)L.B), dim3(64), 0, s, w.bbox_part, d_gE, nb, d_dhext);
    }
    return hipGetLastError();
}

// Workgroups of the independent-wave fused traversal that fit on the device at once (for the persistent
// launch), with this handle's precision and waves per workgroup.
hipError_t adjoint_resident_blocks(Handle &h, int &blocks)
{
    const int wpb = h.waves_per_block;
    int per_cu = 0, cus = 0;
    hipError_t e;
    const bool quad = h.L.expansion == 2;
    const bool sc = mac_form(h.p.theta * h.p.theta) == kMacScaled;
    // the instantiation the handle launches (the occupancy depends on its registers)
    if (h.p.precision == BH_FP32_MIXED) {
        auto k = quad ? (sc ? k_adjoint<true, true, true> : k_adjoint<true, true, false>)
                      : (sc ? k_adjoint<true, false, true> : k_adjoint<true, false, false>);
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, wpb * kWave, adj_lds_bytes<float, false>(wpb));
    } else {
        auto k = quad ? (sc ? k_adjoint<false, true, true> : k_adjoint<false, true, false>)
                      : (sc ? k_adjoint<false, false, true> : k_adjoint<false, false, false>);
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, wpb * kWave, adj_lds_bytes<double, false>(wpb));
    }
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h.device);
    if (e != hipSuccess) return e;
    blocks = per_cu * cus;
    return blocks > 0 ? hipSuccess : hipErrorInvalidValue;
}

}  // namespace ffbh
