// Tree construction on gfx950: bounding cube, Morton codes, LDS radix sort, octree, and the upward pass that forms the
// pseudo-particles.
//
// Paper: Sec. 3.2 (kernels 1-4 of the GPU Barnes-Hut scheme: bounding box, octree, cell centres and
// moments, sort by location) and Eq. (magCenter) (pseudo-particle = moment sum at the geometric
// centre of the members).  The lock-based insertion of the paper is replaced by a construction of all cells
// from the sorted codes at once, the spin-waiting moment kernel by an upward pass over chunks of the sorted
// particles.
#include "ffbh_internal.h"

namespace ffbh {

// ------------------------------------------------------------------------------------------------
// Bounding cube: lo = componentwise minimum, side = largest extent, scale = 2^21 / side.
// ------------------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_bbox_partial(const double *__restrict__ pos, int64_t n,
                                                      double *__restrict__ part,
                                                      uint32_t *__restrict__ status, int enter)
{
    if (enter && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) call_enter(status);
    __shared__ double red[6][256];
    const int b = blockIdx.y;
    const double *p = pos + (int64_t)b * 3 * n;
    double mn[3], mx[3];
    bool bad = false;
    for (int a = 0; a < 3; ++a) { mn[a] = __builtin_inf(); mx[a] = -__builtin_inf(); }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        for (int a = 0; a < 3; ++a) {
            double v = p[a * n + i];
            bad |= !__builtin_isfinite(v);
            if (v < mn[a]) mn[a] = v;
            if (v > mx[a]) mx[a] = v;
        }
    }
    if (bad) set_flag(status, BH_FLAG_NONFINITE);
    for (int a = 0; a < 3; ++a) { red[a][threadIdx.x] = mn[a]; red[3 + a][threadIdx.x] = mx[a]; }
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            for (int a = 0; a < 3; ++a) {
                double o = red[a][threadIdx.x + s];
                if (o < red[a][threadIdx.x]) red[a][threadIdx.x] = o;
                o = red[3 + a][threadIdx.x + s];
                if (o > red[3 + a][threadIdx.x]) red[3 + a][threadIdx.x] = o;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[((int64_t)b * kBboxBlocks + blockIdx.x) * 6 + threadIdx.x] = red[threadIdx.x][0];
}

// One workgroup of 256 per system folds the nb partial boxes (min and max are exact in any order).
// It also clears the count of the system's list of cells for k_upward_top, which the build fills.
__global__ __launch_bounds__(256) void k_bbox_final(const double *__restrict__ part, int nb,
                                                    double *__restrict__ bbox, int32_t *__restrict__ top,
                                                    double s2_scale)
{
    __shared__ double red[6][256];
    const int b = blockIdx.x;
    if (threadIdx.x == 0) top[b] = 0;
    double v[6];
    for (int a = 0; a < 3; ++a) {
        v[a] = __builtin_inf();
        v[3 + a] = -__builtin_inf();
    }
    for (int k = threadIdx.x; k < nb; k += 256) {
        const double *q = part + ((int64_t)b * kBboxBlocks + k) * 6;
        for (int a = 0; a < 3; ++a) {
            v[a] = fmin(v[a], q[a]);
            v[3 + a] = fmax(v[3 + a], q[3 + a]);
        }
    }
    for (int a = 0; a < 6; ++a) red[a][threadIdx.x] = v[a];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fmin(red[a][threadIdx.x], red[a][threadIdx.x + s]);
                red[3 + a][threadIdx.x] = fmax(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    double side = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double e = red[3 + a][0] - red[a][0];
        if (e > side) side = e;
    }
    double *o = bbox + 8 * b;
    o[0] = red[0][0]; o[1] = red[1][0]; o[2] = red[2][0];
    o[3] = side;
    o[4] = side > 0.0 ? 2097152.0 / side : 0.0;
    o[5] = s2_scale;  // factor of the squared cell sides in the node records (node_s2_scale)
}

// ------------------------------------------------------------------------------------------------
// Morton codes: q = min(2^21-1, floor((r - lo) * scale)) per axis, interleaved x-major.
// ------------------------------------------------------------------------------------------------

__device__ inline uint32_t quantise(double r, double lo, double scale)
{
    double t = (r - lo) * scale;
    double f = __builtin_floor(t);
    if (f >= (double)kQMax) return kQMax;
    if (f <= 0.0) return 0u;
    return (uint32_t)f;
}

__global__ __launch_bounds__(256) void k_morton(const double *__restrict__ pos, int64_t n, int64_t ntot,
                                                const double *__restrict__ bbox,
                                                uint64_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                uint32_t *__restrict__ mask)
{
    int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= ntot) return;
    int64_t b = o / n, i = o - b * n;
    const double *p = pos + b * 3 * n;
    const double *bb = bbox + 8 * b;
    uint32_t qx = quantise(p[i], bb[0], bb[4]);
    uint32_t qy = quantise(p[n + i], bb[1], bb[4]);
    uint32_t qz = quantise(p[2 * n + i], bb[2], bb[4]);
    keys[o] = morton(qx, qy, qz);
    vals[o] = (uint32_t)o;
    mask[o] = 0u;  // filled by k_oct_mark
}

// ------------------------------------------------------------------------------------------------
// LSD radix sort, 8-bit digits, stable, segmented by system: a tile never straddles two systems, and
// histograms are laid out (system, digit, tile) so one exclusive scan yields every output offset.
// ------------------------------------------------------------------------------------------------

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t *__restrict__ keys, int64_t n,
                                                             int tiles, int items, int shift,
                                                             uint32_t *__restrict__ hist)
{
    __shared__ uint32_t cnt[kRadixBins];
    const int b = blockIdx.x / tiles, t = blockIdx.x - b * tiles;
    const int64_t tile = (int64_t)kSortThreads * items;
    const int64_t lo = (int64_t)b * n + (int64_t)t * tile;
    const int64_t hi = min(lo + tile, (int64_t)(b + 1) * n);
    cnt[threadIdx.x] = 0;
    // all of this thread's keys are loaded before the first count, so their latencies overlap
    uint32_t d[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t i = lo + (int64_t)r * kSortThreads + threadIdx.x;
        d[r] = r < items && i < hi ? (uint32_t)(keys[i] >> shift) & (kRadixBins - 1) : kRadixBins;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if (d[r] < kRadixBins) atomicAdd(&cnt[d[r]], 1u);
    __syncthreads();
    hist[((int64_t)b * kRadixBins + threadIdx.x) * tiles + t] = cnt[threadIdx.x];
}

// Device-wide exclusive scan of a uint32 array (BITS: of its entries' bit counts) into another or in place, in
// three launches: per-tile sums, a scan of the tile sums (one workgroup), and the per-tile scan with its offset.
// Tiles are kScanTile entries, read and written through LDS so that global accesses are coalesced.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    // inclusive Hillis-Steele over 256 threads in LDS, then shift
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        uint32_t x = t >= off ? sh[t - off] : 0u;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    total = sh[kScanThreads - 1];
    uint32_t r = t ? sh[t - 1] : 0u;
    __syncthreads();
    return r;
}

template <bool BITS>
__device__ inline uint32_t scan_value(uint32_t v) { return BITS ? (uint32_t)__popc(v) : v; }

template <bool BITS>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const uint32_t *a, int64_t len,
                                                             uint32_t *__restrict__ tile_sum)
{
    __shared__ uint32_t sh[kScanThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
        if (i < len) s += scan_value<BITS>(a[i]);
    }
    uint32_t total;
    block_excl_scan(s, sh, total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_sums(uint32_t *__restrict__ tile_sum, int ntiles,
                                                            uint32_t *__restrict__ total_out)
{
    __shared__ uint32_t sh[kScanThreads];
    uint32_t carry = 0;
    for (int base = 0; base < ntiles; base += kScanThreads) {
        const int i = base + (int)threadIdx.x;
        uint32_t v = i < ntiles ? tile_sum[i] : 0u;
        uint32_t tot;
        uint32_t ex = block_excl_scan(v, sh, tot);
        if (i < ntiles) tile_sum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total_out) *total_out = carry;
}

template <bool BITS>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t *a, uint32_t *out, int64_t len,
                                                             const uint32_t *__restrict__ tile_off)
{
    __shared__ uint32_t tile[kScanTile];
    __shared__ uint32_t sh[kScanThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int k = 0; k < kScanItems; ++k) {
        const int j = k * kScanThreads + threadIdx.x;
        tile[j] = base + j < len ? scan_value<BITS>(a[base + j]) : 0u;
    }
    __syncthreads();
    // each thread scans its own run of kScanItems consecutive entries
    uint32_t run = 0;
    for (int k = 0; k < kScanItems; ++k) run += tile[threadIdx.x * kScanItems + k];
    uint32_t total;
    uint32_t off = block_excl_scan(run, sh, total) + tile_off[blockIdx.x];
    for (int k = 0; k < kScanItems; ++k) {
        const int j = threadIdx.x * kScanItems + k;
        const uint32_t v = tile[j];
        tile[j] = off;
        off += v;
    }
    __syncthreads();
    for (int k = 0; k < kScanItems; ++k) {
        const int j = k * kScanThreads + threadIdx.x;
        if (base + j < len) out[base + j] = tile[j];
    }
}

// Inclusive scan over the 64 lanes of a wave.
__device__ inline uint32_t wave_incl_scan_u32(uint32_t v, int lane)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t x = __shfl_up(v, off, kWave);
        if (lane >= off) v += x;
    }
    return v;
}

// Exclusive scan of a short array (len <= kScanSmallMax) in one launch of one workgroup: chunks of
// 8192 entries pass through LDS (coalesced loads and stores); each thread scans a run of 8 consecutive
// entries, offset by a wave scan and the wave totals.  LDS index j is padded to j + j/32 against bank
// conflicts of the strided run accesses.
constexpr int kScanSmallThreads = 1024;
constexpr int kScanSmallItems = 8;
constexpr int kScanSmallChunk = kScanSmallThreads * kScanSmallItems;
constexpr int64_t kScanSmallMax = 4 * (int64_t)kScanSmallChunk;

__device__ inline int scan_pad(int j) { return j + (j >> 5); }

template <bool BITS>
__global__ __launch_bounds__(kScanSmallThreads) void k_scan_small(const uint32_t *a, uint32_t *out, int64_t len,
                                                                  uint32_t *__restrict__ total_out)
{
    constexpr int kWaves = kScanSmallThreads / kWave;
    __shared__ uint32_t tile[kScanSmallChunk + kScanSmallChunk / 32];
    __shared__ uint32_t wsum[kWaves];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    uint32_t carry = 0;
    for (int64_t base = 0; base < len; base += kScanSmallChunk) {
#pragma unroll
        for (int k = 0; k < kScanSmallItems; ++k) {
            const int j = k * kScanSmallThreads + t;
            tile[scan_pad(j)] = base + j < len ? scan_value<BITS>(a[base + j]) : 0u;
        }
        __syncthreads();
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kScanSmallItems; ++k) run += tile[scan_pad(t * kScanSmallItems + k)];
        const uint32_t incl = wave_incl_scan_u32(run, lane);
        if (lane == kWave - 1) wsum[wave] = incl;
        __syncthreads();
        uint32_t woff = 0, ctot = 0;
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t x = wsum[w];
            woff += w < wave ? x : 0u;
            ctot += x;
        }
        uint32_t off = carry + woff + incl - run;
#pragma unroll
        for (int k = 0; k < kScanSmallItems; ++k) {
            const int j = scan_pad(t * kScanSmallItems + k);
            const uint32_t v = tile[j];
            tile[j] = off;
            off += v;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kScanSmallItems; ++k) {
            const int j = k * kScanSmallThreads + t;
            if (base + j < len) out[base + j] = tile[scan_pad(j)];
        }
        carry += ctot;
        __syncthreads();  // tile and wsum are rewritten by the next chunk
    }
    if (t == 0 && total_out) *total_out = carry;
}

// Exclusive scan of a into out (which may be a); writes the total to *total if not null.  scratch: one uint32
// per tile.
template <bool BITS>
static void scan_excl(const uint32_t *a, uint32_t *out, int64_t len, uint32_t *scratch, uint32_t *total, hipStream_t s)
{
    if (len <= kScanSmallMax) {
        hipLaunchKernelGGL(k_scan_small<BITS>, dim3(1), dim3(kScanSmallThreads), 0, s, a, out, len, total);
        return;
    }
    const int ntiles = (int)((len + kScanTile - 1) / kScanTile);
    hipLaunchKernelGGL(k_scan_tiles<BITS>, dim3(ntiles), dim3(kScanThreads), 0, s, a, len, scratch);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanThreads), 0, s, scratch, ntiles, total);
    hipLaunchKernelGGL(k_scan_apply<BITS>, dim3(ntiles), dim3(kScanThreads), 0, s, a, out, len, scratch);
}

constexpr int kFusedTiles = 256;

// One pass of the stable LSD sort over one tile of up to kSortThreads * items keys.  Each wave ranks a
// contiguous run of 64 * ceil(items / 4) keys (the keys of equal digit before it in the run: match masks from
// ballots plus running per-wave digit counts in LDS); the runs' counts give every key its position in
// the tile sorted by digit, where the keys are staged in LDS; then each digit's run of the tile is
// written out to consecutive addresses.  Four times as many threads as a count pass (a tile's keys are the
// same): the ranking is a chain of rounds, so more waves with fewer rounds each end sooner (bh_build of 2^20
// particles, seven passes of which four on the main stream, 419 -> 358 us together with k_order_waves' split).
constexpr int kScatterThreads = 4 * kSortThreads;
constexpr int kScatterItems = kSortItems / 4;  // most keys per thread per tile
__global__ __launch_bounds__(kScatterThreads) void k_radix_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout,
    uint32_t *__restrict__ vout, const uint32_t *__restrict__ hist, int64_t n, int tiles, int items, int shift,
    int64_t ntot, int fused)
{
    constexpr int kWaves = kScatterThreads / kWave;
    constexpr int kTileMax = kSortThreads * kSortItems;
    static_assert(kScatterThreads == 4 * kRadixBins && kWaves == 16, "four threads per digit, sixteen waves");
    __shared__ uint32_t gbase[kRadixBins];        // output offset of the tile's first key of digit d
    __shared__ uint32_t lstart[kRadixBins];       // position of that key in the digit-sorted tile
    __shared__ uint16_t wcnt[kWaves][kRadixBins]; // per-wave digit counts, then per-wave digit offsets
    __shared__ uint32_t dsum[kWaves], dtot[kWaves];
    __shared__ uint64_t skey[kTileMax];
    __shared__ uint32_t sval[kTileMax];
    const int b = blockIdx.x / tiles, t = blockIdx.x - b * tiles;
    const int64_t tile = (int64_t)kSortThreads * items;
    const int64_t lo = (int64_t)b * n + (int64_t)t * tile;
    const int64_t hi = min(lo + tile, (int64_t)(b + 1) * n);
    const int count = (int)(hi - lo);
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const uint32_t dmask = kRadixBins - 1;
    for (int k = tid; k < kWaves * kRadixBins / 2; k += kScatterThreads) ((uint32_t *)wcnt)[k] = 0u;

    // this wave's run of keys, loaded up front (coalesced, all loads in flight together)
    const int rounds = (items + 3) / 4;
    const int c0 = wave * kWave * rounds;
    uint64_t key[kScatterItems];
    uint32_t val[kScatterItems], rank[kScatterItems];
#pragma unroll
    for (int r = 0; r < kScatterItems; ++r) {
        const int p = c0 + r * kWave + lane;
        const bool valid = r < rounds && p < count;
        key[r] = valid ? kin[lo + p] : 0ull;
        val[r] = valid ? vin[lo + p] : 0u;
    }
    // the output offset of (digit, tile): four threads per digit, each a quarter of the digit's row of counts.
    // fused: hist holds raw counts, and the offset is the system's start, plus the keys of smaller digits, plus
    // this digit's keys in earlier tiles
    const int d4 = tid >> 2, q4 = tid & 3;
    uint32_t pre = 0, tot = 0;
    if (fused) {
        const uint32_t *hd = hist + ((int64_t)b * kRadixBins + d4) * tiles;
        if ((tiles & 3) == 0) {
            // rows of a multiple of four counts start 16-byte aligned: read them four at a time, sixteen
            // loads in flight (one at a time, the row's L2 latencies add up to most of the kernel)
            const uint4 *h4 = (const uint4 *)hd;
#pragma unroll 16
            for (int u4 = q4; u4 < tiles / 4; u4 += 4) {
                const uint4 c = h4[u4];
                const int u = 4 * u4;
                tot += c.x + c.y + c.z + c.w;
                pre += (u < t ? c.x : 0u) + (u + 1 < t ? c.y : 0u) + (u + 2 < t ? c.z : 0u) + (u + 3 < t ? c.w : 0u);
            }
        } else {
#pragma unroll 16
            for (int u = q4; u < tiles; u += 4) {
                const uint32_t c = hd[u];
                tot += c;
                pre += u < t ? c : 0u;
            }
        }
    }
    __syncthreads();  // wcnt cleared
#pragma unroll
    for (int r = 0; r < kScatterItems; ++r) {
        if (r < rounds) {
            const bool valid = c0 + r * kWave + lane < count;
            const uint32_t d = (uint32_t)(key[r] >> shift) & dmask;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int bit = 0; bit < kRadixBits; ++bit) {
                const bool set = (d >> bit) & 1u;
                const uint64_t v = __ballot(set);
                m &= set ? v : ~v;
            }
            const uint32_t before = (uint32_t)__popcll(m & lt);
            // one wave's LDS accesses complete in order: this read sees the previous round's update
            const uint32_t cur = valid ? wcnt[wave][d] : 0u;
            rank[r] = cur + before;
            if (valid && before == 0) wcnt[wave][d] = (uint16_t)(cur + (uint32_t)__popcll(m));
        }
    }
    __syncthreads();

    // the waves' offsets in the digit and the digits' starts in the tile and in the output
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = wcnt[4 * q4 + k][d4];
        sum += c[k];
    }
    const uint32_t incl = wave_incl_scan_u32(sum, lane), gincl = wave_incl_scan_u32(tot, lane);
    const uint32_t digit0 = (uint32_t)__shfl((int)(incl - sum), lane & ~3, kWave);
    uint32_t off = incl - sum - digit0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        wcnt[4 * q4 + k][d4] = (uint16_t)off;
        off += c[k];
    }
    pre += __shfl_xor(pre, 1, kWave);
    pre += __shfl_xor(pre, 2, kWave);
    if (lane == kWave - 1) {
        dsum[wave] = incl;
        dtot[wave] = gincl;
    }
    __syncthreads();
    uint32_t woff = 0, goff = 0;
    for (int w = 0; w < kWaves; ++w) {
        woff += w < wave ? dsum[w] : 0u;
        goff += w < wave ? dtot[w] : 0u;
    }
    if (q4 == 0) {
        lstart[d4] = woff + digit0;
        gbase[d4] = fused ? (uint32_t)((int64_t)b * n) + goff + gincl - tot + pre
                          : hist[((int64_t)b * kRadixBins + d4) * tiles + t];
    }
    __syncthreads();

    // stage the tile in digit order
#pragma unroll
    for (int r = 0; r < kScatterItems; ++r) {
        if (r < rounds && c0 + r * kWave + lane < count) {
            const uint32_t d = (uint32_t)(key[r] >> shift) & dmask;
            const uint32_t at = lstart[d] + wcnt[wave][d] + rank[r];
            if (at < (uint32_t)kTileMax) {  // always true for a consistent count
                skey[at] = key[r];
                sval[at] = val[r];
            }
        }
    }
    __syncthreads();
    // each digit's run goes to consecutive output addresses
    for (int j = tid; j < count; j += kScatterThreads) {
        const uint64_t k = skey[j];
        const uint32_t d = (uint32_t)(k >> shift) & dmask;
        const int64_t at = (int64_t)gbase[d] + (j - (int64_t)lstart[d]);
        if (at >= 0 && at < ntot) {  // always true for a consistent histogram
            kout[at] = k;
            vout[at] = sval[j];
        }
    }
}

// The tiled sort orders the codes by their bits above the low kTieBits only, stably, so particles whose
// codes agree above those bits are left in index order.  With 32 low bits left out the upper bits are the
// cell 2^-10 of the cube wide (and one bit of the next level): at 2^20 particles in the chain workload's
// cube that is 0.17 diameters, a cell no two particles that exclude each other share.  The thread at the
// start of each run of equal upper bits orders the run by the low bits, stably, which gives the order of
// the full codes (ties in index order).  Short runs by insertion; longer ones by a bottom-up merge through
// the second key buffer (free at this point), so any run, even all particles at one point, takes
// O(L log L).
constexpr int kTieInsertMax = 32;

__device__ inline bool low_less(uint64_t a, uint64_t b)
{
    constexpr uint64_t m = (1ull << kTieBits) - 1ull;
    return (a & m) < (b & m);
}

__global__ __launch_bounds__(256) void k_fix_ties(uint64_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                  uint64_t *__restrict__ tkeys, uint32_t *__restrict__ tvals,
                                                  int64_t n, int64_t ntot)
{
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= ntot) return;
    const int64_t b = o / n, end = (b + 1) * n;
    const uint64_t h = keys[o] >> kTieBits;
    if (o > b * n && (keys[o - 1] >> kTieBits) == h) return;  // not the start of a run
    if (o + 1 >= end || (keys[o + 1] >> kTieBits) != h) return;  // a run of one
    int64_t e = o + 2;
    while (e < end && (keys[e] >> kTieBits) == h) ++e;
    const int64_t len = e - o;
    if (len <= kTieInsertMax) {
        for (int64_t i = o + 1; i < e; ++i) {
            const uint64_t k = keys[i];
            const uint32_t v = vals[i];
            int64_t j = i;
            while (j > o && low_less(k, keys[j - 1])) {
                keys[j] = keys[j - 1];
                vals[j] = vals[j - 1];
                --j;
            }
            keys[j] = k;
            vals[j] = v;
        }
        return;
    }
    // bottom-up merge sort of [o, e), stable, ping-ponging between the buffers
    uint64_t *ka = keys, *kb = tkeys;
    uint32_t *va = vals, *vb = tvals;
    for (int64_t w = 1; w < len; w <<= 1) {
        for (int64_t lo = o; lo < e; lo += 2 * w) {
            const int64_t mid = min(lo + w, e), hi = min(lo + 2 * w, e);
            int64_t i = lo, j = mid, k = lo;
            while (i < mid && j < hi) {
                if (low_less(ka[j], ka[i])) { kb[k] = ka[j]; vb[k] = va[j]; ++j; }
                else { kb[k] = ka[i]; vb[k] = va[i]; ++i; }
                ++k;
            }
            while (i < mid) { kb[k] = ka[i]; vb[k] = va[i]; ++i; ++k; }
            while (j < hi) { kb[k] = ka[j]; vb[k] = va[j]; ++j; ++k; }
        }
        uint64_t *kt = ka; ka = kb; kb = kt;
        uint32_t *vt = va; va = vb; vb = vt;
    }
    if (ka != keys)
        for (int64_t i = o; i < e; ++i) {
            keys[i] = ka[i];
            vals[i] = va[i];
        }
}

// Sorted positions (SoA, global over systems).
__global__ __launch_bounds__(256) void k_gather3(const double *__restrict__ src, const uint32_t *__restrict__ perm,
                                                 int64_t n, int64_t ntot, double *__restrict__ dst,
                                                 float *__restrict__ dst32, uint32_t *__restrict__ status)
{
    int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= ntot) return;
    const int64_t o = perm[s];
    if (o >= ntot) {
        set_flag(status, BH_FLAG_TREE);
        return;
    }
    const int64_t b = o / n, i = o - b * n;
    const double *p = src + b * 3 * n;
    bool bad = false;
    for (int a = 0; a < 3; ++a) {
        double v = p[a * n + i];
        bad |= !__builtin_isfinite(v);
        dst[a * ntot + s] = v;
        if (dst32) dst32[a * ntot + s] = (float)v;
    }
    if (bad) set_flag(status, BH_FLAG_NONFINITE);
}

// ------------------------------------------------------------------------------------------------
// Octree from the sorted codes.  Call digits(a, c) the number of leading octal digits (of 21) that codes a and
// c share: the level of the deepest cell holding both.  A system's sorted codes then give its octree without
// a binary tree:
//   - A cell of level l around particle i holds more than `leaf` particles iff some window of leaf + 1
//     consecutive particles around i shares l digits, so the deepest such cell has level
//       W_i = max of digits(code_s, code_{s + leaf}) over the windows s .. s + leaf that hold i.
//   - Particles j - 1 and j lie in different children of the cell of level L = digits(code_{j-1}, code_j) that
//     holds both; the cell is split, and j starts a child, iff L <= W_j and L < 21.
//   - A stored cell is one that is split into at least two children (a run of unary cells is stored once, at its
//     deepest level, which leaves every pseudo-particle and every acceptance decision unchanged: same members,
//     smaller side), so each has exactly one first such j, the end of its first child: its key.  The octants of
//     its children are collected in mask[key], the exclusive scan of the masks' bit counts allocates the
//     children (contiguous, octant order), and a child's place is the number of lower octants in the mask.
//   - Leaves are the children of at most `leaf` particles (stored at the first level of their run) and, flagged,
//     the cells of level 21 with more.
// Cell ends and starts are found by galloping from the particle at hand, since most cells are small: a few
// dependent loads.
// (A binary radix tree over all particles with the octree cut from it took ten launches and 285 us at 2^20,
// where 2 % of its nodes were of use; this takes five launches.)
// ------------------------------------------------------------------------------------------------

__device__ inline int digits(uint64_t a, uint64_t c)
{
    return a == c ? kMaxLevel : (__clzll((long long)(a ^ c)) - 1) / 3;
}
// First and last code of the cell of level l that holds code x, and x's octant in its parent cell of level l - 1.
__device__ inline uint64_t cell_low(uint64_t x, int l) { return x & ~((1ull << (3 * (kMaxLevel - l))) - 1ull); }
__device__ inline uint64_t cell_high(uint64_t x, int l) { return x | ((1ull << (3 * (kMaxLevel - l))) - 1ull); }
__device__ inline uint32_t octant(uint64_t x, int l) { return (uint32_t)(x >> (3 * (kMaxLevel - l))) & 7u; }

// Smallest k in [0, j] with code_k >= low, for code_j >= low.
__device__ inline int gallop_left(const uint64_t *code, int j, uint64_t low)
{
    int hi = j, step = 1;
    while (hi - step >= 0 && code[hi - step] >= low) {
        hi -= step;
        step <<= 1;
    }
    int lo = hi - step < 0 ? -1 : hi - step;  // code_lo < low (or before the first)
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (code[m] >= low) hi = m; else lo = m;
    }
    return hi;
}
// Smallest k in (j, end] with code_k > high (end itself if none), for code_j <= high.
__device__ inline int gallop_right(const uint64_t *code, int j, int end, uint64_t high)
{
    int lo = j, step = 1;
    while (lo + step < end && code[lo + step] <= high) {
        lo += step;
        step <<= 1;
    }
    int hi = lo + step > end ? end : lo + step;  // code_hi > high (or past the last)
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (code[m] <= high) lo = m; else hi = m;
    }
    return hi;
}

// Particle j (1 <= j < n) of a system with W_j = wj: if it starts a child of a split cell, that cell's key (which
// gets the octants of this child and, at the key, of the first one), else -1.
template <typename Or>
__device__ inline int oct_mark(const uint64_t *code, int n, int j, int wj, const Or &or_mask)
{
    const uint64_t cj = code[j];
    const int L = digits(code[j - 1], cj);
    if (L > wj || L >= kMaxLevel) return -1;
    const int p = gallop_left(code, j, cell_low(cj, L));
    const uint64_t cp = code[p];
    const int key = gallop_right(code, p, j, cell_high(cp, L + 1));
    or_mask(key, (1u << octant(cj, L + 1)) | (key == j ? 1u << octant(cp, L + 1) : 0u));
    return key;
}

// What the node records and the leaf index are written to; ids of the system's children start at `base`.
struct OctOut {
    NodeRec *nodes;
    int32_t *node_level, *leaf_of, *cell_id;
    uint32_t *status;
    int64_t base, first, max_nodes;  // first: sorted position of the system's first particle
    int leaf;
};

// The record of cell [f, e) as node id; `level` is that of the first cell of its run.  A split cell also
// writes its id into its children's records (the one field they do not write themselves).
template <typename Mask, typename Scan>
__device__ inline void oct_cell(const OctOut &o, const uint64_t *code, int f, int e, int level, int64_t id,
                                const Mask &mask, const Scan &scan)
{
    if (id < 0 || id >= o.max_nodes) {
        set_flag(o.status, BH_FLAG_TREE);
        return;
    }
    const int count = e - f;
    int child = -1, nchild = 0;
    if (count > o.leaf) {
        level = digits(code[f], code[e - 1]);
        if (level >= kMaxLevel) {
            set_flag(o.status, BH_FLAG_DEEP_LEAF);
        } else {
            const int key = gallop_right(code, f, e, cell_high(code[f], level + 1));
            const uint32_t m = key < e ? mask(key) : 0u;
            const int64_t c = o.base + scan(key < e ? key : f);
            nchild = __popc(m);
            if (nchild < 2 || c + nchild > o.max_nodes) {
                set_flag(o.status, BH_FLAG_TREE);
                nchild = 0;
            } else {
                child = (int)c;
                if (o.cell_id) o.cell_id[o.first + key] = (int32_t)id;
                for (int q = 0; q < nchild; ++q) o.nodes[c + q].parent = (int32_t)id;
            }
        }
    }
    NodeRec *r = o.nodes + id;
    r->first = (int32_t)(o.first + f);
    r->count = count;
    r->child = child;
    r->nchild = nchild;
    o.node_level[id] = level;
    if (nchild == 0)
        for (int k = f; k < e; ++k) o.leaf_of[o.first + k] = (int32_t)id;
}

// The children that start at particle j, whose cell has key `key`: j's own cell and, at the key, the first child.
template <typename Mask, typename Scan>
__device__ inline void oct_children(const OctOut &o, const uint64_t *code, int n, int j, int key, const Mask &mask,
                                    const Scan &scan)
{
    const uint64_t cj = code[j];
    const int L = digits(code[j - 1], cj);
    const uint32_t m = mask(key);
    const int64_t c = o.base + scan(key);
    const uint32_t below = m & ((1u << octant(cj, L + 1)) - 1u);
    oct_cell(o, code, j, gallop_right(code, j, n, cell_high(cj, L + 1)), L + 1, c + __popc(below), mask, scan);
    if (key == j) oct_cell(o, code, gallop_left(code, j - 1, cell_low(code[j - 1], L + 1)), j, L + 1, c, mask, scan);
}

// The root of a system of n particles (node id): one leaf up to leaf_size particles.
template <typename Mask, typename Scan>
__device__ inline void oct_root(const OctOut &o, const uint64_t *code, int n, int64_t id, const Mask &mask,
                                const Scan &scan)
{
    o.nodes[id].parent = -1;
    oct_cell(o, code, 0, n, 0, id, mask, scan);
}

constexpr int kOctThreads = 256;
constexpr int kMaxLeaf = 64;  // largest leaf_size

// Keys and masks of all systems: one thread per particle, blockIdx.y the system.  The block's codes and a
// window of them on either side are staged in LDS for the windows' digits.
__global__ __launch_bounds__(kOctThreads) void k_oct_mark(const uint64_t *__restrict__ codes, int n, int leaf,
                                                          int32_t *__restrict__ keys, uint32_t *__restrict__ mask,
                                                          int64_t blocks_per_sys)
{
    __shared__ uint64_t sc[kOctThreads + 2 * kMaxLeaf];
    __shared__ int8_t win[kOctThreads + kMaxLeaf];  // digits of window s at s - (i0 - leaf); -1: not a window
    const int64_t b = blockIdx.x / blocks_per_sys;
    const int i0 = (int)(blockIdx.x - b * blocks_per_sys) * kOctThreads, t = threadIdx.x;
    const uint64_t *code = codes + b * n;
    for (int k = t; k < kOctThreads + 2 * leaf; k += kOctThreads) {
        const int i = i0 - leaf + k;
        sc[k] = i >= 0 && i < n ? code[i] : 0ull;
    }
    __syncthreads();
    for (int k = t; k < kOctThreads + leaf; k += kOctThreads) {
        const int i = i0 - leaf + k;
        win[k] = i >= 0 && i + leaf < n ? (int8_t)digits(sc[k], sc[k + leaf]) : (int8_t)-1;
    }
    __syncthreads();
    const int j = i0 + t;
    if (j >= n) return;
    int w = -1;
    for (int k = 0; k <= leaf; ++k) w = max(w, (int)win[t + k]);
    int key = -1;
    if (j > 0)
        key = oct_mark(code, n, j, w, [&](int k, uint32_t m) { atomicOr(&mask[b * n + k], m); });
    keys[b * n + j] = key;
}

__global__ __launch_bounds__(kOctThreads) void k_oct_emit(const uint64_t *__restrict__ codes, int64_t n, int64_t ntot,
                                                          int64_t B, int leaf, const int32_t *__restrict__ keys,
                                                          const uint32_t *__restrict__ mask,
                                                          const uint32_t *__restrict__ scan,
                                                          NodeRec *__restrict__ nodes, int32_t *__restrict__ node_level,
                                                          int32_t *__restrict__ leaf_of, int32_t *__restrict__ cell_id,
                                                          uint32_t *__restrict__ status, int64_t max_nodes)
{
    const int64_t g = (int64_t)blockIdx.x * kOctThreads + threadIdx.x;
    if (g >= ntot) return;
    if (g == 0) status[2] = (uint32_t)B + status[1];  // number of nodes
    const int64_t b = g / n, first = b * n;
    const int j = (int)(g - first);
    const OctOut o{nodes, node_level, leaf_of, cell_id, status, B, first, max_nodes, leaf};
    auto mask_of = [&](int k) { return mask[first + k]; };
    auto scan_of = [&](int k) { return (int64_t)scan[first + k]; };
    if (j == 0) oct_root(o, codes + first, (int)n, b, mask_of, scan_of);
    const int key = keys[g];
    if (key > 0 && key <= j) oct_children(o, codes + first, (int)n, j, key, mask_of, scan_of);
}

// ------------------------------------------------------------------------------------------------
// Upward pass: every leaf sums its members in sorted order starting from +0.0, every internal node its
// children's sums in octant order (the order they are stored in), children before parents.
//   MODE 0: positions -> centroid S / count and squared side into the node record.
//   MODE 1: moments   -> FP64 moment sum into node_m64 and its FP32 rounding into the record.
//
// One workgroup per chunk of consecutive sorted positions of a system (k_upward_sub) sums the leaves among the
// children that the chunk's keys allocated (consecutive ids), then, level by level with a barrier between
// levels, the cells inside the chunk: a cell's key lies inside it, so the chunk's keys list them all, and their
// children are leaves of the chunk's or cells inside the chunk.  Cells that reach beyond their chunk (the
// ancestors of the chunk boundaries, about seven a boundary) are listed per system when the tree is built and
// follow in a second launch of one workgroup per system (k_upward_top).
//
// A launch costs about 4.5 us in a stream, so what the pass cost before, one launch per level (twelve of them
// above 2^16 nodes, 50-60 us for a few us of work), is now two.
// ------------------------------------------------------------------------------------------------

// A node's centroid and s^2 from its position sums (bb: its system's cube), and its moments.
__device__ inline void up_centre(NodeRec &nd, int level, const double *bb, double sx, double sy, double sz)
{
    const double cnt = (double)nd.count;
    const double side = __builtin_ldexp(bb[3], -level);
    nd.cx = sx / cnt;
    nd.cy = sy / cnt;
    nd.cz = sz / cnt;
    nd.s2 = side * side * bb[5];  // bb[5]: 1, or 1 / theta^2 for the scaled acceptance test
}
__device__ inline void up_moment(NodeRec &nd, double *m64, double mx, double my, double mz)
{
    m64[0] = mx; m64[1] = my; m64[2] = mz;
    nd.mx = (float)mx; nd.my = (float)my; nd.mz = (float)mz;
}

// MODE 0: member positions -> centroids and s^2; MODE 1: member moments -> FP64 and FP32 moment sums;
// MODE 2: both in one pass (vals = positions, vals2 = moments).  Child sums are read from `sums` (8 doubles
// per node: position sums at 0..2, moment sums at 4..6).
// MODE 0: position sums and centres; 1: moment sums; 2: both; 3: moment sums and first moments
// D = sum_j (r_j - c) m_j^T about the centre c (vals = moments, vals2 = positions; centres from MODE 0/2):
// a leaf sums its members in sorted order, a parent adds its children's D shifted to its own centre,
// D_child + (c_child - c) M_child^T, in octant order.
template <int MODE>
__device__ inline void upward_node(int id, const NodeRec &nd, const double *__restrict__ vals,
                                   const double *__restrict__ vals2, int64_t ntot, int64_t n,
                                   NodeRec *__restrict__ nodes, double *__restrict__ sums,
                                   double *__restrict__ node_m64, const int32_t *__restrict__ node_level,
                                   const double *__restrict__ bbox, int64_t max_nodes, double *__restrict__ q64,
                                   float *__restrict__ q32)
{
    if (nd.first < 0 || nd.count < 1 || (int64_t)nd.first + nd.count > ntot ||
        (nd.nchild != 0 && (nd.child < 0 || (int64_t)nd.child + nd.nchild > max_nodes)))
        return;
    const int o = MODE == 1 || MODE == 3 ? 4 : 0;  // slot of the (first) sum
    double sx = 0.0, sy = 0.0, sz = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
    double D[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (MODE == 3) {
        const double c[3] = {nd.cx, nd.cy, nd.cz};
        if (nd.nchild == 0) {
            for (int k = nd.first; k < nd.first + nd.count; ++k) {
                const double d[3] = {vals2[k] - c[0], vals2[ntot + k] - c[1], vals2[2 * ntot + k] - c[2]};
                const double m[3] = {vals[k], vals[ntot + k], vals[2 * ntot + k]};
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) D[3 * a + b] = D[3 * a + b] + d[a] * m[b];
            }
        } else {
            for (int ch = nd.child; ch < nd.child + nd.nchild; ++ch) {
                const NodeRec cn = nodes[ch];
                const double d[3] = {cn.cx - c[0], cn.cy - c[1], cn.cz - c[2]};
                const double m[3] = {sums[8 * ch + 4], sums[8 * ch + 5], sums[8 * ch + 6]};
                const double *dc = q64 + 16 * (int64_t)ch;
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) D[3 * a + b] = D[3 * a + b] + (dc[3 * a + b] + d[a] * m[b]);
            }
        }
    }
    // sums in member (child) order, as the definition's; unrolled so that several members' loads are in
    // flight at once (the additions stay in order: no reassociation without fast-math)
    if (nd.nchild == 0) {
#pragma unroll 4
        for (int k = nd.first; k < nd.first + nd.count; ++k) {
            sx = sx + vals[k];
            sy = sy + vals[ntot + k];
            sz = sz + vals[2 * ntot + k];
            if (MODE == 2) {
                mx = mx + vals2[k];
                my = my + vals2[ntot + k];
                mz = mz + vals2[2 * ntot + k];
            }
        }
    } else {
#pragma unroll 4
        for (int c = nd.child; c < nd.child + nd.nchild; ++c) {
            sx = sx + sums[8 * c + o];
            sy = sy + sums[8 * c + o + 1];
            sz = sz + sums[8 * c + o + 2];
            if (MODE == 2) {
                mx = mx + sums[8 * c + 4];
                my = my + sums[8 * c + 5];
                mz = mz + sums[8 * c + 6];
            }
        }
    }
    if (MODE == 1 || MODE == 3) {
        mx = sx; my = sy; mz = sz;
    }
    if (MODE == 3) {
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            q64[16 * (int64_t)id + k] = D[k];
            q32[16 * (int64_t)id + k] = (float)D[k];
        }
    }
    sums[8 * id + o] = sx;
    sums[8 * id + o + 1] = sy;
    sums[8 * id + o + 2] = sz;
    if (MODE == 2) {
        sums[8 * id + 4] = mx;
        sums[8 * id + 5] = my;
        sums[8 * id + 6] = mz;
    }
    if (MODE == 0 || MODE == 2) up_centre(nodes[id], node_level[id], bbox + 8 * (nd.first / n), sx, sy, sz);
    if (MODE != 0) up_moment(nodes[id], node_m64 + 4 * (int64_t)id, mx, my, mz);
}

constexpr int kUpThreads = 1024;
constexpr int kUpChunkMax = 8192;  // positions per chunk, at most: as many cells as the LDS list holds
constexpr uint8_t kUpSkip = 255;

// Positions per chunk: 256 chunks a system (one a CU), of 2048 to 8192 positions.  Short chunks give more workgroups,
// long ones leave fewer cells to the one workgroup of the second launch.  bh_build and bh_field together at 2^20, with
// chunks of 2048 / 4096 / 8192: 2211 / 2174 / 2186 us; 2^19 1241 / 1239 / 1266; 2^18 804 / 808 / 835; 100003 725 / 738
// / 770 (1024: 720); 32 x 65536 1970 / 1953 / 1948.
static int64_t up_chunk_size(const Layout &L)
{
    return L.n / 256 < 2048 ? 2048 : L.n / 256 > kUpChunkMax ? kUpChunkMax : L.n / 256;
}

// The per-system lists of k_upward_top live in one array: entry b counts system b's list, which starts at
// entry B + 2 n b (a system has fewer than 2 n nodes).
__device__ inline int64_t up_list(int64_t B, int64_t n, int64_t b) { return B + 2 * n * b; }

#define FFBH_UP_PARAMS                                                                                          \
    const double *__restrict__ vals, const double *__restrict__ vals2, int64_t ntot, int64_t n,                  \
        NodeRec *__restrict__ nodes, double *__restrict__ sums, double *__restrict__ node_m64,                   \
        const int32_t *__restrict__ node_level, const double *__restrict__ bbox, int64_t max_nodes,              \
        double *__restrict__ q64, float *__restrict__ q32
#define FFBH_UP_ARGS vals, vals2, ntot, n, nodes, sums, node_m64, node_level, bbox, max_nodes, q64, q32

// The cells of a workgroup, at most CAP, in LDS, and the range of their levels.
template <int CAP>
struct UpList {
    static constexpr int cap = CAP;
    int32_t id[CAP];
    uint8_t lev[CAP];
    int count, lmin, lmax;
};

template <typename List>
__device__ inline void up_reset(List &S)
{
    if (threadIdx.x == 0) {
        S.count = 0;
        S.lmin = kMaxLevel + 1;
        S.lmax = -1;
    }
    __syncthreads();
}
template <int CAP>
__device__ inline void up_add(UpList<CAP> &S, int id, int level)
{
    if ((unsigned)level > (unsigned)kMaxLevel) return;
    const int k = atomicAdd(&S.count, 1);
    if (k >= CAP) return;  // never: a chunk holds fewer split cells than positions
    S.id[k] = id;
    S.lev[k] = (uint8_t)level;
    atomicMin(&S.lmin, level);
    atomicMax(&S.lmax, level);
}
// Sum the listed cells, deepest level first.
template <int MODE, typename List>
__device__ inline void up_levels(const List &S, FFBH_UP_PARAMS)
{
    __syncthreads();
    const int lmin = S.lmin, lmax = S.lmax, count = min(S.count, List::cap);
    for (int l = lmax; l >= lmin; --l) {
        for (int k = threadIdx.x; k < count; k += blockDim.x) {
            if (S.lev[k] != l) continue;
            const int id = S.id[k];
            const NodeRec nd = nodes[id];
            upward_node<MODE>(id, nd, FFBH_UP_ARGS);
        }
        __syncthreads();
    }
}
// Sum the leaves among the nodes [i0, i1) and, with `root`, that of system b; with `all`, list the other nodes.
template <int MODE, typename List>
__device__ inline void up_leaves(List &S, int64_t b, int64_t i0, int64_t i1, bool root, bool all, FFBH_UP_PARAMS)
{
    const int count = (int)(i1 > i0 ? i1 - i0 : 0) + (root ? 1 : 0);
    for (int k = threadIdx.x; k < count; k += blockDim.x) {
        const int id = root && k == 0 ? (int)b : (int)(i0 + k - (root ? 1 : 0));
        const NodeRec nd = nodes[id];
        if (nd.nchild == 0) upward_node<MODE>(id, nd, FFBH_UP_ARGS);
        else if (all) up_add(S, id, node_level[id]);
    }
}

// append: list the cells left to k_upward_top (the build's pass).
template <int MODE>
__global__ __launch_bounds__(kUpThreads) void k_upward_sub(FFBH_UP_PARAMS, const uint32_t *__restrict__ mask,
                                                           const uint32_t *__restrict__ scan,
                                                           const int32_t *__restrict__ cell_id,
                                                           const uint32_t *__restrict__ status, int64_t B,
                                                           int64_t chunk, int chunks, int32_t *__restrict__ top,
                                                           int append)
{
    __shared__ UpList<kUpChunkMax> S;
    const int64_t b = blockIdx.x / chunks;
    const int c = (int)(blockIdx.x - b * chunks);
    const int64_t first = b * n, c0 = c * chunk, c1 = min(c0 + chunk, n);
    up_reset(S);
    // the cells of the chunk's keys: inside the chunk, or left to the second launch
    for (int64_t j = c0 + threadIdx.x; j < c1; j += blockDim.x) {
        if (mask[first + j] == 0u) continue;
        const int id = cell_id[first + j];
        if ((unsigned)id >= (unsigned)max_nodes) continue;
        const int64_t f = nodes[id].first - first, e = f + nodes[id].count;
        if (f >= c0 && e <= c1) {
            up_add(S, id, node_level[id]);
        } else if (append) {
            const uint32_t at = atomicAdd((uint32_t *)&top[b], 1u);
            if ((int64_t)at < 2 * n) top[up_list(B, n, b) + at] = id;
        }
    }
    auto start = [&](int64_t i) { return B + (int64_t)(first + i < ntot ? scan[first + i] : status[1]); };
    up_leaves<MODE>(S, b, start(c0), min(start(c1), max_nodes), c == 0, false, FFBH_UP_ARGS);
    up_levels<MODE>(S, FFBH_UP_ARGS);
}

template <int MODE>
__global__ __launch_bounds__(kUpThreads) void k_upward_top(FFBH_UP_PARAMS, int64_t B, const int32_t *__restrict__ top)
{
    __shared__ uint8_t lev[kUpChunkMax];  // levels of the first entries; of the others they are read again
    __shared__ int lmin, lmax;
    const int64_t b = blockIdx.x;
    const int32_t *list = top + up_list(B, n, b);
    const int64_t listed = (uint32_t)top[b];
    const int count = (int)(listed < 2 * n ? listed : 2 * n);
    auto level_of = [&](int k) -> uint8_t {
        const int id = list[k];
        if ((unsigned)id >= (unsigned)max_nodes) return kUpSkip;
        const int l = node_level[id];
        return (unsigned)l > (unsigned)kMaxLevel ? kUpSkip : (uint8_t)l;
    };
    if (threadIdx.x == 0) {
        lmin = kMaxLevel + 1;
        lmax = -1;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < count; k += blockDim.x) {
        const uint8_t l = level_of(k);
        if (k < kUpChunkMax) lev[k] = l;
        if (l == kUpSkip) continue;
        atomicMin(&lmin, (int)l);
        atomicMax(&lmax, (int)l);
    }
    __syncthreads();
    for (int l = lmax; l >= lmin; --l) {
        for (int k = threadIdx.x; k < count; k += blockDim.x) {
            if ((k < kUpChunkMax ? lev[k] : level_of(k)) != l) continue;
            const int id = list[k];
            const NodeRec nd = nodes[id];
            upward_node<MODE>(id, nd, FFBH_UP_ARGS);
        }
        __syncthreads();
    }
}

// append: the build's pass lists the cells that reach beyond their chunk.
template <int MODE>
static void upward(Handle &h, const double *vals, const double *vals2, hipStream_t s, bool append)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    const int64_t chunk = up_chunk_size(L);
    const int chunks = (int)((L.n + chunk - 1) / chunk);
    hipLaunchKernelGGL(k_upward_sub<MODE>, dim3((unsigned)(L.B * chunks)), dim3(kUpThreads), 0, s, vals, vals2, L.ntot,
                       L.n, w.nodes, w.node_adj, w.node_m64, w.node_level, w.bbox, L.max_nodes, w.node_q64, w.node_q32,
                       w.cell_mask, w.cell_scan, w.cell_id, w.status, L.B, chunk, chunks, w.top_nodes, append ? 1 : 0);
    hipLaunchKernelGGL(k_upward_top<MODE>, dim3((unsigned)L.B), dim3(kUpThreads), 0, s, vals, vals2, L.ntot, L.n,
                       w.nodes, w.node_adj, w.node_m64, w.node_level, w.bbox, L.max_nodes, w.node_q64, w.node_q32, L.B,
                       w.top_nodes);
}

// Hilbert index of the cell (x, y, z) of a 2^b grid per axis: Skilling's transform of the axes to the
// transposed index (J. Skilling, "Programming the Hilbert curve", AIP Conf. Proc. 707, 381 (2004)),
// whose bits, interleaved from the most significant down with x first, are the index.
template <int b>
__device__ inline uint32_t hilbert_index(uint32_t x, uint32_t y, uint32_t z)
{
    uint32_t X[3] = {x, y, z};
    // undo the excess work of the curve's reflections and rotations, from the coarsest bit down
#pragma unroll
    for (uint32_t Q = 1u << (b - 1); Q > 1u; Q >>= 1) {
        const uint32_t P = Q - 1u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const bool invert = (X[i] & Q) != 0u;
            const uint32_t t = invert ? 0u : ((X[0] ^ X[i]) & P);  // exchange the low bits of X[0], X[i]
            X[0] ^= invert ? P : t;
            X[i] ^= t;
        }
    }
    // Gray encode
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t t = 0u;
#pragma unroll
    for (uint32_t Q = 1u << (b - 1); Q > 1u; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1u;
    X[0] ^= t; X[1] ^= t; X[2] ^= t;
    return (uint32_t)morton(X[0], X[1], X[2]);
}

// The Hilbert index of a code's cell at kHilbertBits bits per axis, read off the top bits of the code.
__device__ inline uint32_t hilbert_key(uint64_t code)
{
    const uint64_t c = code >> (3 * (kBits - kHilbertBits));
    return hilbert_index<kHilbertBits>(compact3(c >> 2), compact3(c >> 1), compact3(c));
}

// The packed source record of a sorted particle: FP64 position and the moment in the handle's precision.
__device__ inline void pack_source(double *r, bool mixed, double x, double y, double z, double mx, double my, double mz)
{
    r[0] = x; r[1] = y; r[2] = z;
    if (mixed) {
        float *f = (float *)(r + 3);
        f[0] = (float)mx; f[1] = (float)my; f[2] = (float)mz; f[3] = 0.0f;
    } else {
        r[3] = mx; r[4] = my; r[5] = mz;
    }
}

// ------------------------------------------------------------------------------------------------
// Systems of at most kSmallMax particles: the whole build of a system in one workgroup (k_build_small), with its
// keys, codes and cell masks in LDS, and the moments' upward pass of a later call in another
// (k_moments_small).  A launch costs about 4.5 us in a stream and a small system's kernels little more than
// that: 300 particles took twelve launches and 58 us for bh_build, this takes one of 20.  Against the launches over the
// whole batch that larger systems take (bh_build, us): one system of 513 28 / 77, 1000 35 / 84, 2049 70 / 123, 4096 97 /
// 122; 64 x 1000 39 / 127, 1048 x 1000 206 / 354, 64 x 4096 109 / 167, 256 x 4096 131 / 287.  The limit is LDS: above 4096
// two workgroups no longer share a CU.
// The children's ids of system b start at B + 2 n b (a system has fewer than 2 n nodes), so the ids of a batch
// have gaps; entry b of the list array counts the system's nodes below its root.
// ------------------------------------------------------------------------------------------------

// The workgroup of a system: its threads, the most particles and the most nodes whose sums stay in LDS.  Both kernels
// give the same bits with any.  One thread per particle as far as that goes: of 1024 threads a system of 32 leaves 992
// idle, two such workgroups fill a CU, and a batch is bound by their rounds, where 64 threads leave room for 32.
// bh_build and bh_field (FP64) with 1024 threads -> with the shape of the size: 4 particles x 262144 systems 14663 ->
// 1479 us, 32 x 32768 2409 -> 306, 64 x 16384 1304 -> 261, 100 x 10485 1168 -> 421, 256 x 4096 765 -> 441, 512 x 2048
// 626 -> 471.  One system gains from the cheaper barriers: 32 particles 29.0 -> 24.5 us, 65 32.0 -> 26.3, 256 44.3 ->
// 39.4, 512 49.0 -> 44.7.
template <int THREADS, int MAX, int SUM_NODES>
struct SmallShape {
    static constexpr int threads = THREADS, waves = THREADS / kWave, max = MAX, items = MAX / THREADS, sum_nodes = SUM_NODES;
    static constexpr bool passes = MAX > 2048;  // also sorts by counting passes
};
using ShapeWide = SmallShape<1024, kSmallMax, 1024>;
using ShapeHalf = SmallShape<512, 512, 256>;
using ShapeMid = SmallShape<256, 256, 128>;
using ShapeNarrow = SmallShape<64, 64, 64>;

// LDS of k_build_small: the sort's keys and values (ping-pong in the counting passes), then the codes in the keys'
// place and, in the values', the list of cell starts and their cells' keys; the cell masks and their scan.
template <typename SH>
struct SmallSort {
    static constexpr int bins = SH::passes ? kRadixBins : 1;
    union {
        uint32_t key[2][SH::max];  // 31 or 32 bits of the codes
        uint64_t code[SH::max];
    };
    uint16_t val[2][SH::max];  // index in the system
    union {
        uint16_t wcnt[SH::waves][bins];
        uint16_t scan[SH::max];
    };
    uint32_t mask[SH::max];
    uint32_t lstart[bins];
    uint32_t dsum[SH::waves];
    double box[SH::waves][6];
    int starts, flag;
};
// Sums and split cells of a system of at most NODES nodes, for its upward pass.
template <int NODES>
struct SumList {
    double sum[NODES][6];  // position sums, moment sums
    uint16_t from[NODES], len[NODES];  // leaf: first member and count; else first child and children
    uint16_t cell[NODES];              // the split cells
    uint8_t lev[NODES], leaf[NODES];
    int count, lmin, lmax;
};
template <typename SH>
union SmallUp {
    UpList<SH::max> list;
    SumList<SH::sum_nodes> sums;
};
template <typename SH>
union SmallLds {
    SmallSort<SH> s;
    SmallUp<SH> up;  // the upward pass, once the tree is written
};
static_assert(2 * sizeof(SmallLds<ShapeWide>) <= kLdsPerCu, "two workgroups of k_build_small share a CU's LDS");
static_assert(ShapeWide::threads == 4 * kRadixBins && ShapeWide::waves == 16, "four threads per digit, sixteen waves");

// One stable pass over 8 bits of the keys from buffer src to the other one: every wave ranks a contiguous run of
// keys (match masks from ballots, running per-wave digit counts), the counts give every key its place.
template <typename SH>
__device__ inline void small_pass(SmallSort<SH> &S, int n, int src, int shift)
{
    constexpr int kWaves = SH::waves, kSmallThreads = SH::threads, kSmallItems = SH::items;
    const int t = threadIdx.x, wave = t / kWave, lane = t & (kWave - 1);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const int chunk = ((n + kWaves * kWave - 1) / (kWaves * kWave)) * kWave, c0 = wave * chunk;
    for (int k = t; k < kWaves * kRadixBins / 2; k += kSmallThreads) ((uint32_t *)S.wcnt)[k] = 0u;
    __syncthreads();
    uint32_t rank[kSmallItems], dig[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        if (r * kWave >= chunk) break;
        const int p = c0 + r * kWave + lane;
        const bool valid = p < n;
        const uint32_t d = valid ? (S.key[src][p] >> shift) & (kRadixBins - 1) : 0u;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < kRadixBits; ++bit) {
            const bool set = (d >> bit) & 1u;
            const uint64_t v = __ballot(set);
            m &= set ? v : ~v;
        }
        const uint32_t before = (uint32_t)__popcll(m & lt);
        // one wave's LDS accesses complete in order: this read sees the previous round's update
        const uint32_t cur = valid ? S.wcnt[wave][d] : 0u;
        rank[r] = cur + before;
        dig[r] = d;
        if (valid && before == 0) S.wcnt[wave][d] = (uint16_t)(cur + (uint32_t)__popcll(m));
    }
    __syncthreads();
    // four threads per digit, each four waves' counts: the waves' offsets in the digit and the digits' starts
    {
        const int d = t >> 2, w0 = 4 * (t & 3);
        uint32_t c[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = S.wcnt[w0 + k][d];
            sum += c[k];
        }
        const uint32_t incl = wave_incl_scan_u32(sum, lane);
        // sums of the digit's threads before this one: the inclusive scan less that of the digit before
        const uint32_t digit0 = (uint32_t)__shfl((int)(incl - sum), lane & ~3, kWave);
        uint32_t at = incl - sum - digit0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            S.wcnt[w0 + k][d] = (uint16_t)at;
            at += c[k];
        }
        if (lane == kWave - 1) S.dsum[wave] = incl;
        __syncthreads();
        uint32_t woff = 0;
        for (int w = 0; w < kWaves; ++w) woff += w < wave ? S.dsum[w] : 0u;
        if ((t & 3) == 0) S.lstart[d] = woff + digit0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        if (r * kWave >= chunk) break;
        const int p = c0 + r * kWave + lane;
        if (p >= n) continue;
        const uint32_t at = S.lstart[dig[r]] + S.wcnt[wave][dig[r]] + rank[r];
        if (at < (uint32_t)SH::max) {  // always true for consistent counts
            S.key[src ^ 1][at] = S.key[src][p];
            S.val[src ^ 1][at] = S.val[src][p];
        }
    }
    __syncthreads();
}

// The value of lane l ^ M, by row and half-row moves where there is one.
template <int M>
__device__ inline uint32_t lane_xor(uint32_t v)
{
    if constexpr (M == 1) return __builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false);        // quad
    else if constexpr (M == 2) return __builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, false);   // quad
    else if constexpr (M == 3) return __builtin_amdgcn_update_dpp(0, (int)v, 0x1b, 0xf, 0xf, false);   // quad
    else if constexpr (M == 7) return __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);  // half-row mirror
    else if constexpr (M == 15) return __builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false); // row mirror
    else if constexpr (M == 8) return __builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);  // row rotate by 8
    else if constexpr (M == 4) return lane_xor<3>(lane_xor<7>(v));
    else return (uint32_t)__shfl_xor((int)v, M, kWave);
}

// One compare-exchange of a bitonic network between lanes l and l ^ M, by key, then index.
template <int M>
__device__ inline void sort_step(uint64_t &k, uint32_t &v, int lane)
{
    constexpr int top = M >= 32 ? 32 : M >= 16 ? 16 : M >= 8 ? 8 : M >= 4 ? 4 : M >= 2 ? 2 : 1;
    const uint64_t ok = (uint64_t)lane_xor<M>((uint32_t)(k >> 32)) << 32 | lane_xor<M>((uint32_t)k);
    const uint32_t ov = lane_xor<M>(v);
    const bool less = ok < k || (ok == k && ov < v);
    if (less == ((lane & top) == 0)) {
        k = ok;
        v = ov;
    }
}

// Stable ascending sort of a system of at most kMergeMax particles, S.code and the indices S.val[0]: runs of 64 in
// registers (a bitonic network of 21 steps), then rounds in which every key finds its place in the merged run of twice
// the length by a binary search in the other one.  300 / 1000 particles: 5 / 8 us, where the counting passes with
// their ties take 13 / 14.  It is bound by issue on the one CU, log(n)^2 a key against a fixed number of passes:
// 4096 take 32 us, where the passes take 31 (and the Hilbert keys' three passes 20).
constexpr int kMergeMax = 2048;
template <typename SH, typename KeyOf>
__device__ inline void small_merge_sort(SmallSort<SH> &S, int n, const KeyOf &key_of)
{
    constexpr int kSmallThreads = SH::threads, kItems = (SH::max < kMergeMax ? SH::max : kMergeMax) / kSmallThreads;
    const int t = threadIdx.x, lane = t & (kWave - 1);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int p = t + r * kSmallThreads;
        if (p - lane >= n) continue;  // for the whole wave
        uint64_t k = p < n ? key_of(p) : ~0ull;
        uint32_t v = (uint32_t)p;
        sort_step<1>(k, v, lane);
        sort_step<3>(k, v, lane); sort_step<1>(k, v, lane);
        sort_step<7>(k, v, lane); sort_step<2>(k, v, lane); sort_step<1>(k, v, lane);
        sort_step<15>(k, v, lane); sort_step<4>(k, v, lane); sort_step<2>(k, v, lane); sort_step<1>(k, v, lane);
        sort_step<31>(k, v, lane); sort_step<8>(k, v, lane); sort_step<4>(k, v, lane); sort_step<2>(k, v, lane);
        sort_step<1>(k, v, lane);
        sort_step<63>(k, v, lane); sort_step<16>(k, v, lane); sort_step<8>(k, v, lane); sort_step<4>(k, v, lane);
        sort_step<2>(k, v, lane); sort_step<1>(k, v, lane);
        if (p < n) {
            S.code[p] = k;
            S.val[0][p] = (uint16_t)v;
        }
    }
    __syncthreads();
    for (int width = kWave; width < n; width *= 2) {
        uint64_t k[kItems];
        uint16_t v[kItems];
        int start[kItems], len[kItems], at[kItems];
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const int p = t + r * kSmallThreads;
            at[r] = len[r] = start[r] = 0;
            k[r] = 0ull;
            v[r] = 0;
            if (p >= n) continue;
            k[r] = S.code[p];
            v[r] = S.val[0][p];
            start[r] = (p & ~(2 * width - 1)) + ((p & width) != 0 ? 0 : width);  // the other run
            len[r] = min(width, max(n - start[r], 0));
            if ((p & width) != 0) k[r] += 1ull;  // of equal keys those of the first run come first
        }
        // keys of the other run below k
        for (int step = width; step > 0; step >>= 1)
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                if (r * kSmallThreads >= n) break;
                const int next = at[r] + step;
                if (next <= len[r] && S.code[start[r] + next - 1] < k[r]) at[r] = next;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const int p = t + r * kSmallThreads;
            if (p >= n) continue;
            const bool second = (p & width) != 0;
            const int to = (second ? p - width : p) + at[r];
            S.code[to] = second ? k[r] - 1ull : k[r];
            S.val[0][to] = v[r];
        }
        __syncthreads();
    }
}

// The same by counting passes: the codes' upper 31 bits, then runs of equal upper bits by the low 32 (as k_fix_ties);
// where a run is longer than an insertion sort should take, all 63 bits from the start.
template <typename SH, typename KeyOf>
__device__ inline void small_count_sort(SmallSort<SH> &S, int n, const KeyOf &code_of)
{
    constexpr int kSmallThreads = SH::threads, kSmallItems = SH::items;
    const int t = threadIdx.x;
    if (t == 0) S.flag = 0;  // read behind the passes' barriers
    for (int i = t; i < n; i += kSmallThreads) {
        S.key[0][i] = (uint32_t)(code_of(i) >> kTieBits);
        S.val[0][i] = (uint16_t)i;
    }
    for (int q = 0; q < 4; ++q) small_pass(S, n, q & 1, 8 * q);
    for (int i = t; i + kTieInsertMax < n; i += kSmallThreads)
        if (S.key[0][i] == S.key[0][i + kTieInsertMax]) S.flag = 1;
    __syncthreads();
    const bool long_run = S.flag != 0;
    if (long_run) {
        for (int i = t; i < n; i += kSmallThreads) {
            S.key[0][i] = (uint32_t)code_of(i);
            S.val[0][i] = (uint16_t)i;
        }
        for (int q = 0; q < 4; ++q) small_pass(S, n, q & 1, 8 * q);
        for (int i = t; i < n; i += kSmallThreads) S.key[0][i] = (uint32_t)(code_of(S.val[0][i]) >> kTieBits);
        for (int q = 0; q < 4; ++q) small_pass(S, n, q & 1, 8 * q);
    }
    // the full codes, in the keys' place
    uint64_t c[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) c[r] = t + r * kSmallThreads < n ? code_of(S.val[0][t + r * kSmallThreads]) : 0ull;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r)
        if (t + r * kSmallThreads < n) S.code[t + r * kSmallThreads] = c[r];
    __syncthreads();
    if (!long_run) {
        for (int i = t; i < n; i += kSmallThreads) {
            const uint64_t h = S.code[i] >> kTieBits;
            if (i > 0 && (S.code[i - 1] >> kTieBits) == h) continue;  // not the start of a run
            for (int e = i + 1; e < n && (S.code[e] >> kTieBits) == h; ++e) {
                const uint64_t k = S.code[e];
                const uint16_t v = S.val[0][e];
                int j = e;
                while (j > i && low_less(k, S.code[j - 1])) {
                    S.code[j] = S.code[j - 1];
                    S.val[0][j] = S.val[0][j - 1];
                    --j;
                }
                S.code[j] = k;
                S.val[0][j] = v;
            }
        }
        __syncthreads();
    }
}

struct SmallArgs {
    const double *pos, *mom;
    int n, leaf, enter, leave, hilbert, mixed;
    int64_t ntot, B, max_nodes;
    double s2_scale;
    double *bbox, *spos, *smom, *src, *sums, *node_m64;
    uint64_t *codes;
    uint32_t *perm, *tgt_order, *status;
    NodeRec *nodes;
    int32_t *node_level, *leaf_of, *top;
};

template <int NODES>
__device__ inline void up_add(SumList<NODES> &S, int cell, int level)
{
    if ((unsigned)level > (unsigned)kMaxLevel) return;
    const int k = atomicAdd(&S.count, 1);
    if (k >= NODES) return;  // never: each node is listed once
    S.cell[k] = (uint16_t)cell;
    S.lev[k] = (uint8_t)level;
    atomicMin(&S.lmin, level);
    atomicMax(&S.lmax, level);
}

// Sum of src[0], src[stride], ... in order, FLIGHT loads at a time.
template <int FLIGHT>
__device__ inline double add_in_order(const double *src, int len, int stride)
{
    double acc = 0.0;
    for (int k = 0; k < len; k += FLIGHT) {
        double v[FLIGHT];
#pragma unroll
        for (int q = 0; q < FLIGHT; ++q) v[q] = src[min(k + q, len - 1) * stride];
#pragma unroll
        for (int q = 0; q < FLIGHT; ++q) acc = k + q < len ? acc + v[q] : acc;
    }
    return acc;
}

// Upward pass of one system whose `total` nodes below the root start at id base.  Where its nodes fit, their sums
// stay in LDS: a lane sums one component of a node (c = 0..2 positions, 4..6 moments; eight children or sixteen
// members in flight, added in order), and the records, which no sum needs, are written at the end.  Bound by latency:
// through memory a level was a chain of four or five loads, 3.7 us; one system of 1000 took 16 us in all and takes 7.
// First moments (MODE 3) go to memory, one lane for each of a node's nine.
template <int MODE, typename SH>
__device__ inline void small_upward(SmallUp<SH> &U, int64_t b, int64_t base, int64_t total, const double *vals,
                                    const double *vals2, const SmallArgs &a, double *q64, float *q32)
{
    constexpr int kSumNodes = SH::sum_nodes;
    // first moments: nine lanes a node leave the wide shape's 350 nodes of 4096 particles more rounds than a thread a
    // node has (bh_field 73 us, 97 with lanes); the narrower shapes gain (512 x 100 with order-2 cells 63.6 -> 52.2)
    if ((MODE == 3 && SH::max > ShapeHalf::max) || total >= kSumNodes || base + total > a.max_nodes) {
        up_reset(U.list);
        up_leaves<MODE>(U.list, b, base, min(base + total, a.max_nodes), true, true, vals, vals2, a.ntot, a.n, a.nodes,
                        a.sums, a.node_m64, a.node_level, a.bbox, a.max_nodes, q64, q32);
        up_levels<MODE>(U.list, vals, vals2, a.ntot, a.n, a.nodes, a.sums, a.node_m64, a.node_level, a.bbox,
                        a.max_nodes, q64, q32);
        return;
    }
    SumList<kSumNodes> &S = U.sums;
    constexpr int kLanes = MODE == 2 ? 8 : 4;
    const int nodes = (int)total + 1, t = threadIdx.x, group = t / kLanes, groups = (int)blockDim.x / kLanes;
    const int c = (t & (kLanes - 1)) + (MODE == 1 || MODE == 3 ? 4 : 0);
    const bool sums = (c & 3) != 3;
    const int comp = c < 4 ? c : c - 1;
    auto id_of = [&](int k) { return k == 0 ? (int)b : (int)base + k - 1; };
    up_reset(S);
    const int64_t first = (int64_t)b * a.n;
    for (int k = t; k < nodes; k += (int)blockDim.x) {
        const NodeRec &nd = a.nodes[id_of(k)];
        const int nchild = nd.nchild, slot = nd.child - (int)base + 1, at = (int)(nd.first - first), count = nd.count;
        const bool in = at >= 0 && count > 0 && at + count <= a.n;  // always, and a cell's children too
        const bool leaf = nchild == 0, ok = leaf ? in : in && nchild > 0 && slot > 0 && slot + nchild <= nodes;
        S.leaf[k] = leaf ? 1 : 0;
        S.from[k] = (uint16_t)(ok ? leaf ? at : slot : 0);
        S.len[k] = (uint16_t)(ok ? leaf ? count : nchild : 0);
        if (ok && !leaf) up_add(S, k, a.node_level[id_of(k)]);
    }
    __syncthreads();
    if (sums) {
        const double *src = (MODE == 2 && c >= 4 ? vals2 : vals) + (c & 3) * a.ntot + first;
        for (int k = group; k < nodes; k += groups)
            if (S.leaf[k]) S.sum[k][comp] = add_in_order<16>(src + S.from[k], S.len[k], 1);
    }
    __syncthreads();
    const int count = min(S.count, kSumNodes), lmin = S.lmin;
    for (int l = S.lmax; l >= lmin; --l) {
        for (int k = group; k < count; k += groups)
            if (sums && S.lev[k] == l) {
                const int cell = S.cell[k];
                S.sum[cell][comp] = add_in_order<8>(&S.sum[S.from[cell]][comp], S.len[cell], 6);
            }
        __syncthreads();
    }
    if constexpr (MODE == 3) {
        // the first moments as in upward_node, a lane for each of the nine components
        const int e = t & 15, ra = min(e / 3, 2), rb = e % 3, team = t >> 4, teams = (int)blockDim.x >> 4;
        auto centre = [&](int k) { return (&a.nodes[id_of(k)].cx)[ra]; };
        auto store = [&](int k, double D) {
            q64[16 * (int64_t)id_of(k) + e] = D;
            q32[16 * (int64_t)id_of(k) + e] = (float)D;
        };
        constexpr int kFlight = 8;
        for (int k = team; k < nodes; k += teams) {
            const int len = S.len[k];
            if (e >= 9 || !S.leaf[k] || len == 0) continue;
            const double *r = vals2 + ra * a.ntot + first + S.from[k], *m = vals + rb * a.ntot + first + S.from[k];
            const double x = centre(k);
            double D = 0.0;
            for (int j = 0; j < len; j += kFlight) {
                double rv[kFlight], mv[kFlight];
#pragma unroll
                for (int q = 0; q < kFlight; ++q) {
                    rv[q] = r[min(j + q, len - 1)];
                    mv[q] = m[min(j + q, len - 1)];
                }
#pragma unroll
                for (int q = 0; q < kFlight; ++q) D = j + q < len ? D + (rv[q] - x) * mv[q] : D;
            }
            store(k, D);
        }
        __syncthreads();
        for (int l = S.lmax; l >= lmin; --l) {
            for (int k = team; k < count; k += teams) {
                if (e >= 9 || S.lev[k] != l) continue;
                const int cell = S.cell[k], from = S.from[cell], len = S.len[cell];
                const double x = centre(cell);
                double cv[8], dv[8], D = 0.0;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int ch = from + min(q, len - 1);
                    cv[q] = centre(ch);
                    dv[q] = q64[16 * (int64_t)id_of(ch) + e];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) D = q < len ? D + (dv[q] + (cv[q] - x) * S.sum[from + q][3 + rb]) : D;
                store(cell, D);
            }
            __syncthreads();
        }
    }
    for (int k = t; k < nodes; k += (int)blockDim.x) {
        const int id = id_of(k);
        if (S.len[k] == 0) continue;
        NodeRec &nd = a.nodes[id];
        const double *v = S.sum[k];
        if (MODE == 0 || MODE == 2) up_centre(nd, a.node_level[id], a.bbox + 8 * b, v[0], v[1], v[2]);
        if (MODE != 0) up_moment(nd, a.node_m64 + 4 * (int64_t)id, v[3], v[4], v[5]);
    }
}

// Positions (POS) and moments (MOM) of system b in sorted order, and the packed source records: particle i comes from
// place from(i) of the caller's order, out-of-range places are flagged.  A thread loads all of its particles before
// it stores any: one after the other they were four round trips at 4096.
template <typename SH, bool MOM, bool POS, typename From, typename Also>
__device__ inline void small_gather(const SmallArgs &a, int64_t b, const double *p, const double *m, const From &from,
                                    const Also &also)
{
    constexpr int kSmallThreads = SH::threads, kSmallItems = SH::items;
    const int n = a.n, t = threadIdx.x;
    const int64_t first = b * n;
    int o[kSmallItems];
    double r[kSmallItems][3], v[kSmallItems][3];
#pragma unroll
    for (int q = 0; q < kSmallItems; ++q) o[q] = t + q * kSmallThreads < n ? from(t + q * kSmallThreads) : 0;
#pragma unroll
    for (int q = 0; q < kSmallItems; ++q) {
        const int i = t + q * kSmallThreads;
        if (i < n && (o[q] < 0 || o[q] >= n)) {
            set_flag(a.status, BH_FLAG_TREE);
            o[q] = -1;
        }
        if (i >= n || o[q] < 0) continue;
        for (int k = 0; k < 3; ++k) {
            r[q][k] = POS ? p[k * n + o[q]] : p[k * a.ntot + first + i];
            if (MOM) v[q][k] = m[k * n + o[q]];
        }
    }
    bool bad = false;
#pragma unroll
    for (int q = 0; q < kSmallItems; ++q) {
        const int i = t + q * kSmallThreads;
        if (i >= n || o[q] < 0) continue;
        const int64_t g = first + i;
        also(g, i);
        for (int k = 0; k < 3; ++k) {
            if (POS) a.spos[k * a.ntot + g] = r[q][k];
            if (MOM) a.smom[k * a.ntot + g] = v[q][k];
            if (MOM) bad |= !__builtin_isfinite(v[q][k]);
        }
        if (MOM) pack_source(a.src + 6 * g, a.mixed != 0, r[q][0], r[q][1], r[q][2], v[q][0], v[q][1], v[q][2]);
    }
    if (bad) set_flag(a.status, BH_FLAG_NONFINITE);
}

// Whether the deepest cell that holds particles j - 1 and j has more than `leaf` members: the first of them at most
// `leaf` before j (by halving steps), and the particle `leaf` after that one.
__device__ inline bool small_starts(const uint64_t *code, int n, int leaf, int j)
{
    const uint64_t cj = code[j];
    const int L = digits(code[j - 1], cj);
    if (L >= kMaxLevel) return false;
    const uint64_t low = cell_low(cj, L);
    int back = 1;  // j - 1 is inside
    for (int step = kMaxLeaf; step > 0; step >>= 1) {
        const int b = back + step;
        const uint64_t c = code[max(j - b, 0)];
        back = b <= leaf && b <= j && c >= low ? b : back;
    }
    const int e = j - back + leaf;
    return e < n && code[e] <= cell_high(cj, L);
}

template <bool MOM, typename SH>
__global__ __launch_bounds__(SH::threads) void k_build_small(SmallArgs a)
{
    constexpr int kSmallThreads = SH::threads, kSmallItems = SH::items, kWaves = SH::waves;
    __shared__ SmallLds<SH> lds;
    SmallSort<SH> &S = lds.s;
    const int t = threadIdx.x, wave = t / kWave, lane = t & (kWave - 1), n = a.n;
    const int64_t b = blockIdx.x, first = b * n;
    const double *p = a.pos + 3 * first;
    if (a.enter && b == 0 && t == 0) call_enter(a.status);

    // bounding cube (as k_bbox_partial and k_bbox_final)
    double lo[3], hi[3];
    bool bad = false;
    for (int c = 0; c < 3; ++c) { lo[c] = __builtin_inf(); hi[c] = -__builtin_inf(); }
    for (int i = t; i < n; i += kSmallThreads)
        for (int c = 0; c < 3; ++c) {
            const double v = p[c * n + i];
            bad |= !__builtin_isfinite(v);
            if (v < lo[c]) lo[c] = v;
            if (v > hi[c]) hi[c] = v;
        }
    if (bad) set_flag(a.status, BH_FLAG_NONFINITE);
    for (int c = 0; c < 3; ++c)
        for (int off = 1; off < kWave; off <<= 1) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], off, kWave));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], off, kWave));
        }
    if (lane == 0)
        for (int c = 0; c < 3; ++c) {
            S.box[wave][c] = lo[c];
            S.box[wave][3 + c] = hi[c];
        }
    if (t == 0) S.starts = 0;
    __syncthreads();
    double side = 0.0;
    for (int c = 0; c < 3; ++c) {
        lo[c] = S.box[lane & (kWaves - 1)][c];
        hi[c] = S.box[lane & (kWaves - 1)][3 + c];
        for (int off = 1; off < kWaves; off <<= 1) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], off, kWave));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], off, kWave));
        }
        if (hi[c] - lo[c] > side) side = hi[c] - lo[c];
    }
    const double scale = side > 0.0 ? 2097152.0 / side : 0.0;
    if (t == 0) {
        double *o = a.bbox + 8 * b;
        o[0] = lo[0]; o[1] = lo[1]; o[2] = lo[2];
        o[3] = side;
        o[4] = scale;
        o[5] = a.s2_scale;
    }
    auto code_of = [&](int i) {
        return morton(quantise(p[i], lo[0], scale), quantise(p[n + i], lo[1], scale), quantise(p[2 * n + i], lo[2], scale));
    };

    if (!SH::passes || n <= kMergeMax) {
        small_merge_sort(S, n, code_of);
    } else {
        if constexpr (SH::passes) small_count_sort(S, n, code_of);
    }

    // the particles in sorted order (as k_gather3 and k_gather_pack): all of a thread's loads before its stores
    small_gather<SH, MOM, true>(a, b, p, MOM ? a.mom + 3 * first : nullptr, [&](int i) { return (int)S.val[0][i]; },
                                [&](int64_t g, int i) {
                                    a.codes[g] = S.code[i];
                                    a.perm[g] = (uint32_t)(first + S.val[0][i]);
                                });
    // cell starts, keys and masks (as k_oct_mark): a particle starts a child of the deepest cell that holds it and
    // the one before it iff that cell has more than `leaf` members.  About a quarter do; they are listed first (in
    // any order), so that the searches below run with full waves.
    for (int i = t; i < n; i += kSmallThreads) S.mask[i] = 0u;
    __syncthreads();  // the values are read, their place takes the list
    for (int j0 = t - lane; j0 < n; j0 += kSmallThreads) {
        const int j = j0 + lane;
        const bool starts = j > 0 && j < n && small_starts(S.code, n, a.leaf, j);
        const uint64_t m = __ballot(starts);
        int at = 0;
        if (lane == 0 && m != 0ull) at = atomicAdd(&S.starts, (int)__popcll(m));
        at = __shfl(at, 0, kWave) + (int)__popcll(m & ((1ull << lane) - 1ull));
        if (starts) S.val[0][at] = (uint16_t)j;
    }
    __syncthreads();
    const int starts = S.starts;
    for (int k = t; k < starts; k += kSmallThreads) {
        const int j = S.val[0][k];
        S.val[1][k] = (uint16_t)max(oct_mark(S.code, n, j, kMaxLevel, [&](int q, uint32_t m) { atomicOr(&S.mask[q], m); }), 0);
    }
    __syncthreads();
    // scan of the masks' bit counts, each thread its run of kSmallItems positions
    uint32_t run = 0;
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int i = t * kSmallItems + r;
        run += i < n ? (uint32_t)__popc(S.mask[i]) : 0u;
    }
    const uint32_t incl = wave_incl_scan_u32(run, lane);
    if (lane == kWave - 1) S.dsum[wave] = incl;
    __syncthreads();
    uint32_t off = incl - run, total = 0;
    for (int w = 0; w < kWaves; ++w) {
        off += w < wave ? S.dsum[w] : 0u;
        total += S.dsum[w];
    }
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int i = t * kSmallItems + r;
        if (i >= n) break;
        S.scan[i] = (uint16_t)off;
        off += (uint32_t)__popc(S.mask[i]);
    }
    if (t == 0) {
        a.top[b] = (int32_t)total;
        // number of nodes; a batch's (at least its roots) is summed when it is asked for (k_small_total)
        if (b == 0) a.status[2] = a.B == 1 ? 1u + total : (uint32_t)a.B;
    }
    __syncthreads();
    const int64_t base = a.B + 2 * first;
    {
        const OctOut o{a.nodes, a.node_level, a.leaf_of, nullptr, a.status, base, first, a.max_nodes, a.leaf};
        auto mask_of = [&](int k) { return S.mask[k]; };
        auto scan_of = [&](int k) { return (int64_t)S.scan[k]; };
        if (t == kSmallThreads - 1) oct_root(o, S.code, n, b, mask_of, scan_of);
        for (int k = t; k < starts; k += kSmallThreads)
            if (S.val[1][k] > 0) oct_children(o, S.code, n, S.val[0][k], S.val[1][k], mask_of, scan_of);
    }
    __syncthreads();
    small_upward<MOM ? 2 : 0>(lds.up, b, base, total, a.spos, a.smom, a, nullptr, nullptr);
    if constexpr (SH::passes) {
        if (a.hilbert) {
            // target order (as launch_target_order)
            __syncthreads();
            for (int i = t; i < n; i += kSmallThreads) {
                S.key[0][i] = hilbert_key(a.codes[first + i]);
                S.val[0][i] = (uint16_t)i;
            }
            for (int q = 0; q < 3; ++q) small_pass(S, n, q & 1, 8 * q);
            for (int i = t; i < n; i += kSmallThreads) a.tgt_order[first + i] = (uint32_t)(first + S.val[1][i]);
        }
    }
    if (a.leave) {
        __syncthreads();
        if (t == 0) call_leave(a.status);
    }
}

// Moments of a small system: gathered into sorted order with the packed source records, then summed upward.
template <int MODE, typename SH>
__global__ __launch_bounds__(SH::threads) void k_moments_small(SmallArgs a, double *q64, float *q32)
{
    __shared__ SmallUp<SH> U;
    const int n = a.n;
    const int64_t b = blockIdx.x, first = b * n;
    if (a.enter && b == 0 && threadIdx.x == 0) call_enter(a.status);
    if (a.mom) {  // else they are there
        small_gather<SH, true, false>(a, b, a.spos, a.mom + 3 * first,
                                      [&](int i) {
                                          const int64_t o = (int64_t)a.perm[first + i] - first;
                                          return o < 0 || o >= n ? -1 : (int)o;
                                      },
                                      [](int64_t, int) {});
    }
    __syncthreads();
    const int64_t base = a.B + 2 * first, total = min((int64_t)(uint32_t)a.top[b], (int64_t)2 * n);
    small_upward<MODE>(U, b, base, total, a.smom, a.spos, a, q64, q32);
}

// Number of nodes from the scan's total; zero before the first build.
__global__ void k_small_total(uint32_t *status, int64_t B)
{
    if (threadIdx.x == 0 && status[2] != 0u) status[2] = (uint32_t)B + status[1];
}

static SmallArgs small_args(Handle &h, const double *d_pos, const double *d_mom, bool enter)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    SmallArgs a{};
    a.pos = d_pos;
    a.mom = d_mom;
    a.n = (int)L.n;
    a.leaf = h.p.leaf_size;
    a.enter = enter ? 1 : 0;
    a.hilbert = uses_target_order(L) ? 1 : 0;
    a.mixed = h.p.precision == BH_FP32_MIXED ? 1 : 0;
    a.ntot = L.ntot;
    a.B = L.B;
    a.max_nodes = L.max_nodes;
    a.s2_scale = node_s2_scale(h.p.theta * h.p.theta);
    a.bbox = w.bbox;
    a.spos = w.spos;
    a.smom = w.smom;
    a.src = (double *)w.src64;
    a.sums = w.node_adj;
    a.node_m64 = w.node_m64;
    a.codes = w.codes;
    a.perm = w.perm;
    a.tgt_order = w.tgt_order;
    a.status = w.status;
    a.nodes = w.nodes;
    a.node_level = w.node_level;
    a.leaf_of = w.leaf_of;
    a.top = w.top_nodes;
    return a;
}

// ------------------------------------------------------------------------------------------------
// Host launch sequences
// ------------------------------------------------------------------------------------------------

// f(shape) with the workgroup shape of systems of n particles: the narrowest with a thread for each.
template <typename F>
static void with_small_shape(int64_t n, const F &f)
{
    if (n <= ShapeNarrow::max) f(ShapeNarrow{});
    else if (n <= ShapeMid::max) f(ShapeMid{});
    else if (n <= ShapeHalf::max) f(ShapeHalf{});
    else f(ShapeWide{});
}

#define FFBH_TRY(x)                         \
    do {                                    \
        hipError_t e_ = (x);                \
        if (e_ != hipSuccess) return e_;    \
    } while (0)

static void gather_moments(Handle &h, const double *d_mom, hipStream_t s, bool enter);

hipError_t launch_build(Handle &h, const double *d_pos, hipStream_t s, const double *d_mom, hipStream_t side,
                        bool join, bool enter, const SortedWork &after_sort, bool *leave)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    const int64_t n = L.n, B = L.B, ntot = L.ntot;
    if (L.n <= kSmallMax) {
        SmallArgs a = small_args(h, d_pos, d_mom, enter);
        if (leave) a.leave = *leave = B == 1 && !after_sort;
        with_small_shape(n, [&](auto shape) {
            using SH = decltype(shape);
            if (d_mom) hipLaunchKernelGGL((k_build_small<true, SH>), dim3((unsigned)B), dim3(SH::threads), 0, s, a);
            else hipLaunchKernelGGL((k_build_small<false, SH>), dim3((unsigned)B), dim3(SH::threads), 0, s, a);
        });
        // the sort ends with the build: nothing of it is left to run beside after_sort's work
        if (after_sort) FFBH_TRY(after_sort(s));
        return hipGetLastError();
    }
    // partial boxes: at most kBboxBlocks per system, no more than one workgroup per 256 particles
    const int nb = (int)((n + 255) / 256 < kBboxBlocks ? (n + 255) / 256 : kBboxBlocks);
    hipLaunchKernelGGL(k_bbox_partial, dim3((unsigned)nb, (unsigned)B), dim3(256), 0, s, d_pos, n,
                       w.bbox_part, w.status, enter ? 1 : 0);
    hipLaunchKernelGGL(k_bbox_final, dim3((unsigned)B), dim3(256), 0, s, w.bbox_part, nb, w.bbox, w.top_nodes,
                       node_s2_scale(h.p.theta * h.p.theta));
    hipLaunchKernelGGL(k_morton, dim3(grid_for(ntot, 256)), dim3(256), 0, s, d_pos, n, ntot, w.bbox,
                       w.keys[0], w.vals[0], w.cell_mask);
    const int tiles = (int)L.tiles;
    const unsigned sblocks = (unsigned)(B * tiles);
    // the digits above the low kTieBits bits; k_fix_ties then orders the rare runs of equal upper bits
    for (int pass = kTieBits / kRadixBits; pass < kRadixPasses; ++pass) {
        const int src = pass & 1, dst = src ^ 1;
        const int shift = pass * kRadixBits;
        hipLaunchKernelGGL(k_radix_hist, dim3(sblocks), dim3(kSortThreads), 0, s, w.keys[src], n, tiles,
                           L.sort_items, shift, w.hist);
        // up to kFusedTiles tiles per system the scatter derives its offsets from the raw counts
        const int fused = tiles <= kFusedTiles;
        if (!fused) scan_excl<false>(w.hist, w.hist, (int64_t)L.hist_len, w.scan_tmp, nullptr, s);
        hipLaunchKernelGGL(k_radix_scatter, dim3(sblocks), dim3(kScatterThreads), 0, s, w.keys[src],
                           w.vals[src], w.keys[dst], w.vals[dst], w.hist, n, tiles, L.sort_items, shift, ntot,
                           fused);
    }
    hipLaunchKernelGGL(k_fix_ties, dim3(grid_for(ntot, 256)), dim3(256), 0, s, w.keys[0], w.vals[0], w.keys[1],
                       w.vals[1], n, ntot);
    static_assert((kRadixPasses - kTieBits / kRadixBits) % 2 == 0 && kTieBits % kRadixBits == 0,
                  "an even number of tiled passes leaves the sorted data in buffer 0");
    // the sorted data is back in buffer 0
    hipLaunchKernelGGL(k_gather3, dim3(grid_for(ntot, 256)), dim3(256), 0, s, d_pos, w.perm, n, ntot,
                       w.spos, (float *)nullptr, w.status);
    // the sorted codes, permutation and positions and the bounding cube are final from here on
    if (side) {
        hipError_t e = hipEventRecord(h.sorted_ev, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(side, h.sorted_ev, 0);
        if (e != hipSuccess) return e;
    }
    // Replayed graphs submit the kernels in the order they were captured, so the order of the enqueues
    // below matters: the first octree kernel goes first, the side stream's work next (before the rest of
    // the octree, which it runs beside).
    const int64_t sysblocks = (n + kOctThreads - 1) / kOctThreads;
    hipLaunchKernelGGL(k_oct_mark, dim3((unsigned)(B * sysblocks)), dim3(kOctThreads), 0, s, w.codes, (int)n,
                       (int)h.p.leaf_size, w.cell_key, w.cell_mask, sysblocks);
    if (uses_target_order(L)) launch_target_order(h, side ? side : s);
    if (after_sort) {
        const hipError_t e = after_sort(side ? side : s);
        if (e != hipSuccess) return e;
    }
    scan_excl<true>(w.cell_mask, w.cell_scan, ntot, w.scan_tmp, w.status + 1, s);
    hipLaunchKernelGGL(k_oct_emit, dim3(grid_for(ntot, kOctThreads)), dim3(kOctThreads), 0, s, w.codes, n, ntot, B,
                       (int)h.p.leaf_size, w.cell_key, w.cell_mask, w.cell_scan, w.nodes, w.node_level, w.leaf_of,
                       w.cell_id, w.status, L.max_nodes);
    if (d_mom) {
        // positions and moments summed in one upward pass
        gather_moments(h, d_mom, s, false);
        upward<2>(h, w.spos, w.smom, s, true);
    } else {
        upward<0>(h, w.spos, nullptr, s, true);
    }
    if (side && join) {
        hipError_t e = hipEventRecord(h.join_ev, side);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, h.join_ev, 0);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Target order: the traversal takes each wave's targets from a run of consecutive entries of this order.
// Sorted (Morton) order jumps between distant cells at every boundary of the Z curve, and a wave whose
// targets straddle such a jump walks the union of two far-apart neighbourhoods.  The Hilbert curve has no
// jumps (consecutive cells share a face), so waves of targets taken in Hilbert order span smaller regions
// and their union walks visit fewer nodes.  Results depend on the grouping only through the order of
// FP32-mixed partial sums and of the adjoint's reductions.
// ------------------------------------------------------------------------------------------------

// Key of sorted particle o: the Hilbert index of its cell at kHilbertBits bits per axis, read off the top
// bits of its Morton code (the same cube); the value is o itself.
__global__ __launch_bounds__(256) void k_hilbert_keys(const uint64_t *__restrict__ codes, int64_t ntot,
                                                      uint64_t *__restrict__ keys, uint32_t *__restrict__ vals)
{
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= ntot) return;
    keys[o] = hilbert_key(codes[o]);
    vals[o] = (uint32_t)o;
}

void launch_target_order(Handle &h, hipStream_t s)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    hipLaunchKernelGGL(k_hilbert_keys, dim3(grid_for(L.ntot, 256)), dim3(256), 0, s, w.codes, L.ntot, w.keys[1],
                       w.vals[1]);
    // three stable 8-bit passes over the 24-bit keys, per system: (keys[1], vals[1]) -> (hkeys, tgt_order)
    // -> (keys[1], vals[1]) -> (hkeys, tgt_order); within a cell the sorted order is kept
    static_assert(kHilbertBits <= kRadixBits, "three radix passes cover the Hilbert keys");
    uint64_t *kb[2] = {w.keys[1], w.hkeys};
    uint32_t *vb[2] = {w.vals[1], w.tgt_order};
    const int tiles = (int)L.tiles;
    const unsigned sblocks = (unsigned)(L.B * tiles);
    const int fused = tiles <= kFusedTiles;
    for (int pass = 0; pass < 3; ++pass) {
        const int src = pass & 1, dst = src ^ 1;
        const int shift = pass * kRadixBits;
        hipLaunchKernelGGL(k_radix_hist, dim3(sblocks), dim3(kSortThreads), 0, s, kb[src], L.n, tiles,
                           L.sort_items, shift, w.hist);
        if (!fused) scan_excl<false>(w.hist, w.hist, (int64_t)L.hist_len, w.hscan_tmp, nullptr, s);
        hipLaunchKernelGGL(k_radix_scatter, dim3(sblocks), dim3(kScatterThreads), 0, s, kb[src], vb[src], kb[dst],
                           vb[dst], w.hist, L.n, tiles, L.sort_items, shift, L.ntot, fused);
    }
}

}  // namespace ffbh

namespace ffbh {

// Moments gathered into sorted order (non-finite values flagged) and, in the same pass, the packed source
// record of every sorted particle in the handle's precision (FP64 moment or FP32 moment after the FP64
// position).
__global__ __launch_bounds__(256) void k_gather_pack(const double *__restrict__ mom, const uint32_t *__restrict__ perm,
                                                     const double *__restrict__ spos, int64_t n, int64_t ntot,
                                                     double *__restrict__ smom, double *__restrict__ src, int mixed,
                                                     uint32_t *__restrict__ status, int enter)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (enter && k == 0) call_enter(status);
    if (k >= ntot) return;
    const int64_t o = perm[k];
    if (o >= ntot) {
        set_flag(status, BH_FLAG_TREE);
        return;
    }
    const int64_t b = o / n, i = o - b * n;
    const double *p = mom + b * 3 * n;
    const double mx = p[i], my = p[n + i], mz = p[2 * n + i];
    if (!__builtin_isfinite(mx) || !__builtin_isfinite(my) || !__builtin_isfinite(mz))
        set_flag(status, BH_FLAG_NONFINITE);
    smom[k] = mx;
    smom[ntot + k] = my;
    smom[2 * ntot + k] = mz;
    pack_source(src + 6 * k, mixed != 0, spos[k], spos[ntot + k], spos[2 * ntot + k], mx, my, mz);
}

// Moments in sorted order and the packed source records of the handle's precision.  enter: the first kernel of
// the call.
static void gather_moments(Handle &h, const double *d_mom, hipStream_t s, bool enter)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    hipLaunchKernelGGL(k_gather_pack, dim3(grid_for(L.ntot, 256)), dim3(256), 0, s, d_mom, w.perm, w.spos, L.n,
                       L.ntot, w.smom, (double *)w.src64, h.p.precision == BH_FP32_MIXED ? 1 : 0, w.status,
                       enter ? 1 : 0);
}

// Moments of a small system summed upward (with the first moments for order-2 cells).
static void launch_moments_small(Handle &h, const SmallArgs &a, hipStream_t s)
{
    const unsigned B = (unsigned)h.L.B;
    with_small_shape(h.L.n, [&](auto shape) {
        using SH = decltype(shape);
        if (h.L.expansion == 2)
            hipLaunchKernelGGL((k_moments_small<3, SH>), dim3(B), dim3(SH::threads), 0, s, a, h.w.node_q64, h.w.node_q32);
        else
            hipLaunchKernelGGL((k_moments_small<1, SH>), dim3(B), dim3(SH::threads), 0, s, a, (double *)nullptr,
                               (float *)nullptr);
    });
}

// The same for systems of one leaf, whose moments are in sorted order: a thread sums a system.
constexpr int64_t kLeavesMin = 8192;
template <int MODE>
__global__ __launch_bounds__(256) void k_moments_leaf(FFBH_UP_PARAMS, int64_t B)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    const NodeRec nd = nodes[b];
    if (nd.nchild == 0) upward_node<MODE>((int)b, nd, FFBH_UP_ARGS);
}
static void launch_moments_leaf(Handle &h, hipStream_t s)
{
    const Layout &L = h.L;
    Workspace &w = h.w;
    if (L.expansion == 2)
        hipLaunchKernelGGL(k_moments_leaf<3>, dim3(grid_for(L.B, 256)), dim3(256), 0, s, w.smom, w.spos, L.ntot, L.n,
                           w.nodes, w.node_adj, w.node_m64, w.node_level, w.bbox, L.max_nodes, w.node_q64, w.node_q32,
                           L.B);
    else
        hipLaunchKernelGGL(k_moments_leaf<1>, dim3(grid_for(L.B, 256)), dim3(256), 0, s, w.smom, (double *)nullptr,
                           L.ntot, L.n, w.nodes, w.node_adj, w.node_m64, w.node_level, w.bbox, L.max_nodes,
                           (double *)nullptr, (float *)nullptr, L.B);
}

// First moments of every node from the moments and positions of a build with moments: the order-2 cells of an MD
// step.
hipError_t launch_upward_first_moments(Handle &h, const double *d_mom, hipStream_t s)
{
    if (h.L.n <= kSmallMax)
        launch_moments_small(h, small_args(h, nullptr, d_mom, false), s);
    else
        upward<3>(h, h.w.smom, h.w.spos, s, false);
    return hipGetLastError();
}

hipError_t launch_upward_moments(Handle &h, const double *d_mom, hipStream_t s, bool enter)
{
    if (h.L.n <= kSmallMax) {
        // one CU gathers 4096 moments in 13 us; a launch over many costs 4.5 us and pays above 2048
        // one leaf a system: a workgroup each pays up to the 8192 that the chip holds at once, above a thread does
        // (bh_field of 13107 systems of 10 particles 39 -> 33 us, with order-2 cells 63 -> 38; 100000 of 4 173 -> 98)
        const bool leaves = h.L.n <= h.p.leaf_size && h.L.B > kLeavesMin, apart = h.L.n > kMergeMax || leaves;
        if (apart) gather_moments(h, d_mom, s, enter);
        if (leaves) {
            launch_moments_leaf(h, s);
            return hipGetLastError();
        }
        const SmallArgs a = small_args(h, nullptr, apart ? nullptr : d_mom, enter && !apart);
        launch_moments_small(h, a, s);
        return hipGetLastError();
    }
    gather_moments(h, d_mom, s, enter);
    if (h.L.expansion == 2)
        upward<3>(h, h.w.smom, h.w.spos, s, false);
    else
        upward<1>(h, h.w.smom, nullptr, s, false);
    return hipGetLastError();
}

// Node counts of small systems, whose ids have gaps: the number of nodes of the batch into *total, and with off
// (B entries) the exclusive scan of the systems' counts.
void launch_small_counts(Handle &h, uint32_t *off, hipStream_t s)
{
    Workspace &w = h.w;
    scan_excl<false>((const uint32_t *)w.top_nodes, off, h.L.B, w.scan_tmp, w.status + 1, s);
    hipLaunchKernelGGL(k_small_total, dim3(1), dim3(64), 0, s, w.status, h.L.B);
}

}  // namespace ffbh
