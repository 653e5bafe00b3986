// All-pairs dipolar field and force (the paper's all-pairs GPU step, Sec. 3.1 / Alg. 1): for every particle
// i of a system, H_i = sum_{j != i} T(r_i - r_j) m_j (Eq. H_dip) and, optionally, the all-pairs energy
// gradient dE/dr_i = -sum_{j != i} f_dip(r_i - r_j; m_i, m_j) (the f_dip summand of Sec. 2), with
// E = -1/2 sum m.H - sum m.H_ext.  It is the exact reference the Barnes-Hut path approximates, and the
// paper's AP column of Table 1.
//
// Layout: a workgroup of W waves owns G = 64 / S targets and shares out the sources.  Lane l of a wave takes
// target l mod G, and the S lane groups of the W waves are S W workers: worker k sums source units k, k + S W,
// ...  A unit is 256 sources in the FP32-mixed mode (the span whose partial sums stay FP32 before they are added
// to the FP64 sums) and G in FP64.  Each wave stages its workers' sources through its own LDS slice, G records
// of 48 bytes (FP64 position, moment in T) per worker at a time, read by all lanes of a worker from the same
// address (broadcast), so no barrier separates the waves until their sums meet in LDS, in worker order.
// Offsets are formed in FP64 and rounded to T, as in the tree path.
//
// Bound by vector issue once the chip is full (28 vector instructions a pair in FP64, 23 in FP32-mixed; 300000
// particles: 0.97e12 and 1.73e12 pairs/s), by the latency of one worker's chain of pairs below about 10^4
// particles.  Against one workgroup for 512 targets and all sources: 1000 particles 186 -> 10 us (FP64 field)
// and 169 -> 23 us (FP32-mixed field), 20011 particles with the gradient, FP32-mixed, 4.84 -> 0.54 ms, 300000
// particles 136 -> 92 ms (FP64 field) and 136 -> 93 ms (FP32-mixed with the gradient).
#include "traverse.h"

namespace ffbh {

template <typename T>
struct ApSrc;
template <>
struct ApSrc<float> {
    double x, y, z;
    float mx, my, mz, pad0;
    double pad1;
};
template <>
struct ApSrc<double> {
    double x, y, z, mx, my, mz;
};
static_assert(sizeof(ApSrc<float>) == 48 && sizeof(ApSrc<double>) == 48, "48-byte LDS source records");

constexpr int kApMaxWaves = 16;
constexpr int ap_unit(bool mixed, int S) { return mixed ? 256 : kWave / S; }
// LDS bytes of one wave: the workers' records, each worker's run 16 bytes apart from a multiple of the banks, and
// later the 64 x 6 sums
constexpr int kApSlice = kWave * 48 + 64;

template <bool MIXED, bool FORCE, int S>
__global__ __launch_bounds__(kApMaxWaves *kWave) void k_ap(const double *__restrict__ pos,
                                                           const double *__restrict__ mom, int64_t n,
                                                           double *__restrict__ H, double *__restrict__ dEdr)
{
    using T = typename std::conditional<MIXED, float, double>::type;
    constexpr int C = FORCE ? 6 : 3;  // sums per target: the field, then the gradient's pair sums
    constexpr int G = kWave / S;
    constexpr int kUnit = ap_unit(MIXED, S);
    static_assert(kUnit % G == 0, "a unit is staged in whole runs of G sources");
    const int lane = threadIdx.x & (kWave - 1), W = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: scalar loop counters
    const int g = lane % G, sub = lane / G;
    // this worker's run of records
    ApSrc<T> *tile = (ApSrc<T> *)(ffbh_dyn_lds + (size_t)wave * kApSlice + (size_t)sub * (G * 48 + 16));
    const int64_t b = blockIdx.y;
    const double *p = pos + b * 3 * n;
    const double *m = mom + b * 3 * n;
    const int64_t ti = (int64_t)blockIdx.x * G + g, i = ti < n ? ti : 0;
    const double rx = p[i], ry = p[n + i], rz = p[2 * n + i];
    const T ax = FORCE ? (T)m[i] : (T)0, ay = FORCE ? (T)m[n + i] : (T)0, az = FORCE ? (T)m[2 * n + i] : (T)0;
    double sum[C];  // FP64 accumulation
#pragma unroll
    for (int c = 0; c < C; ++c) sum[c] = 0.0;
    auto load = [&](int64_t j) {
        const int64_t k = j < n ? j : 0;
        ApSrc<T> r{};
        r.x = p[k]; r.y = p[n + k]; r.z = p[2 * n + k];
        r.mx = (T)m[k]; r.my = (T)m[n + k]; r.mz = (T)m[2 * n + k];
        return r;
    };
    // all workers of a wave step together; a worker past its last source sums none
    const int64_t stride = (int64_t)W * S * kUnit;
    for (int64_t w0 = (int64_t)wave * S * kUnit; w0 < n; w0 += stride) {
        const int64_t u0 = w0 + sub * kUnit;
        T part[C];  // FP32 partial sums of the unit (mixed mode)
#pragma unroll
        for (int c = 0; c < C; ++c) part[c] = MIXED ? (T)0 : (T)sum[c];
        ApSrc<T> next = load(u0 + g);
#pragma unroll 1
        for (int c0 = 0; c0 < kUnit && w0 + c0 < n; c0 += G) {
            wave_lds_sync();  // the records of the last run have been read
            tile[g] = next;
            wave_lds_sync();
            if (c0 + G < kUnit) next = load(u0 + c0 + G + g);
            const int64_t left = n - (u0 + c0);
            const int cnt = left < 0 ? 0 : left < G ? (int)left : G;      // this worker's sources
            const int wcnt = n - (w0 + c0) < G ? (int)(n - (w0 + c0)) : G;  // the first worker's, the most
#pragma unroll 4
            for (int k = 0; k < wcnt; ++k) {
                const ApSrc<T> s = tile[k];
                // the target itself and any particle at its position are at distance zero and add zeros
                const T x = (T)(rx - s.x), y = (T)(ry - s.y), z = (T)(rz - s.z);
                const T r2 = norm2<T>(x, y, z);
                const bool use = r2 > (T)0 && (S == 1 || k < cnt);
                if constexpr (FORCE) {
                    T gx, gy, gz, tx, ty, tz;
                    adj_field_r2<T>(use, r2, x, y, z, ax, ay, az, s.mx, s.my, s.mz, gx, gy, gz, tx, ty, tz, part[0],
                                    part[1], part[2]);
                    part[3] += gx; part[4] += gy; part[5] += gz;
                } else {
                    dip_acc_r2<T>(use, r2, x, y, z, s.mx, s.my, s.mz, part[0], part[1], part[2]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) sum[c] = MIXED ? sum[c] + (double)part[c] : (double)part[c];
    }
    // the workers' sums meet in LDS and are added in worker order
    double *red = (double *)ffbh_dyn_lds;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) red[((wave * S + sub) * C + c) * G + g] = sum[c];
    __syncthreads();
    for (int e = threadIdx.x; e < C * G; e += blockDim.x) {
        const int64_t o = (int64_t)blockIdx.x * G + e % G;
        const int c = e / G;
        double v = 0.0;
        for (int w = 0; w < W * S; ++w) v += red[w * C * G + e];
        if (o < n) {
            if (c < 3) H[(b * 3 + c) * n + o] = v;
            else if (dEdr) dEdr[(b * 3 + c - 3) * n + o] = -v;
        }
    }
}

// E_b = -1/2 sum_i m_i.H_i - sum_i m_i.H_ext,b, one workgroup per system, in a fixed order.
__global__ __launch_bounds__(1024) void k_ap_energy(const double *__restrict__ mom, const double *__restrict__ H,
                                                    const double *__restrict__ hext, int64_t n,
                                                    double *__restrict__ E)
{
    __shared__ double red[1024];
    const int64_t b = blockIdx.x;
    const double *m = mom + b * 3 * n, *h = H + b * 3 * n;
    const double *he = hext ? hext + 3 * b : nullptr;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
        double e = -0.5 * (m[i] * h[i] + m[n + i] * h[n + i] + m[2 * n + i] * h[2 * n + i]);
        if (he) e -= m[i] * he[0] + m[n + i] * he[1] + m[2 * n + i] * he[2];
        s += e;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) E[b] = red[0];
}

template <bool MIXED, bool FORCE>
static void launch_k_ap(int64_t n, int32_t batch, const double *pos, const double *mom, double *H, double *dEdr,
                        hipStream_t s)
{
    const int64_t groups = ((n + kWave - 1) / kWave) * batch;  // of 64 targets
    // Narrower target groups where 64 targets a workgroup leave compute units idle or with one workgroup more
    // than others: from 1024 workgroups on the last round no longer counts (20011 particles, FP64 field: 680 us
    // with 64 targets, 566 with 32, 458 with 16; 100000: no difference).  The FP32-mixed units of 256 sources
    // are the limit of small systems, which gain nothing from more workers than units (1000 particles: 23 us
    // with 64 targets, 29 with 16).
    int S = groups >= 1024 ? 1 : 2 * groups >= 1024 ? 2 : 4;
    if (MIXED && n < 32 * ap_unit(true, 1)) S = 1;
    const int64_t units = (n + ap_unit(MIXED, S) - 1) / ap_unit(MIXED, S);
    int64_t W = units / S < kApMaxWaves ? units / S : kApMaxWaves;
    if (W < 1) W = 1;
    // as many rounds as W waves need, over as few waves as give as many rounds
    const int64_t rounds = (units + W * S - 1) / (W * S);
    W = (units + rounds * S - 1) / (rounds * S);
    const size_t lds = (size_t)W * kApSlice;
    const int G = kWave / S;
    const dim3 grid((unsigned)((n + G - 1) / G), (unsigned)batch), block((unsigned)(W * kWave));
    if (S == 1) hipLaunchKernelGGL((k_ap<MIXED, FORCE, 1>), grid, block, lds, s, pos, mom, n, H, dEdr);
    else if (S == 2) hipLaunchKernelGGL((k_ap<MIXED, FORCE, 2>), grid, block, lds, s, pos, mom, n, H, dEdr);
    else hipLaunchKernelGGL((k_ap<MIXED, FORCE, 4>), grid, block, lds, s, pos, mom, n, H, dEdr);
}

hipError_t launch_ap(int64_t n, int32_t batch, int32_t precision, const double *pos, const double *mom,
                     const double *hext, double *H, double *dEdr, double *E, hipStream_t s)
{
    const bool mixed = precision == BH_FP32_MIXED;
    if (mixed && dEdr) launch_k_ap<true, true>(n, batch, pos, mom, H, dEdr, s);
    else if (mixed) launch_k_ap<true, false>(n, batch, pos, mom, H, dEdr, s);
    else if (dEdr) launch_k_ap<false, true>(n, batch, pos, mom, H, dEdr, s);
    else launch_k_ap<false, false>(n, batch, pos, mom, H, dEdr, s);
    if (E) hipLaunchKernelGGL(k_ap_energy, dim3((unsigned)batch), dim3(1024), 0, s, mom, H, hext, n, E);
    return hipGetLastError();
}

}  // namespace ffbh
