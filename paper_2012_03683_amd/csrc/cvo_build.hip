// cvo_build.hip -- device-side preparation of point clouds for the pair pass.
//
// The paper's double sum (eq. (7)) is sparse (Sec. III-B): a point only
// interacts with points within the cutoff.  These kernels bin clouds so the
// pair pass scans neighbourhoods instead of all N*M pairs, and plan its work.
// Both sides of all pairs go through the same launches:
//   box_kernel        partial bounding boxes and the non-finite check
//   params_kernel     grids, cluster parameters and key widths from the boxes
//   key_kernel        cell index (reference side) / Hilbert index (query side)
//                     of every point, and the first pass's digit counts
//   sort_pass         one 8-bit pass of a stable LSD radix sort per launch
//   (radix_hist, scan_*, radix_scatter: the passes of large sorts)
//   view_kernel       sorted float4 copies, padded and pre-scaled feature
//                     rows, and the dense first-index-per-cell table
//   cluster_kernel    query clusters, their candidate counts at the current pose
//   plan_kernel       their pieces and output slots, the query map
//   record_kernel     the pieces in dispatch order, heaviest bucket first
// What bounds them is latency, not bytes (30,000 + 30,000 points with 24
// feature columns move under 20 MB in all), so the chain is made short: both
// sides share each launch, nothing is launched only to scan or to clear, and
// the host reads nothing before the piece and slot counts.  One evaluation of
// 14,873 x 15,000 points: 81 launches and 4 host waits (467-487 us) became 18
// launches and 2 waits (167 us).
// Every result is deterministic: orderings come from the stable sort; the
// atomics only place slots and records, whose position changes no sum.
#include "cvo_device.hpp"
#include "cvo_launch.hpp"

#include <algorithm>

namespace cvo {

// ---------------------------------------------------------------- boxes
// Partial box of one cloud (blockIdx.y = 2 pair + side), 8 floats per block:
// minimum, maximum, non-finite count.  A block takes the points of its grid
// stride; the partial boxes are joined in params_kernel.
__global__ __launch_bounds__(256) void box_kernel(const ViewArgs a)
{
    const PairIn &p = a.in[blockIdx.y >> 1];
    const bool q = blockIdx.y & 1;
    const float *xyz = q ? p.zx : p.xx;
    const long long n = q ? p.nz : p.nx;
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float v = xyz[3 * i + k];
            if (!isfinite(v)) { bad = 1; continue; }
            mn[k] = fminf(mn[k], v);
            mx[k] = fmaxf(mx[k], v);
        }
    }
    __shared__ float s_box[4][7];
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            mn[k] = fminf(mn[k], __shfl_xor(mn[k], off));
            mx[k] = fmaxf(mx[k], __shfl_xor(mx[k], off));
        }
        bad |= __shfl_xor(bad, off);
    }
    if ((threadIdx.x & 63) == 0) {
        float *o = s_box[threadIdx.x >> 6];
        for (int k = 0; k < 3; ++k) { o[k] = mn[k]; o[3 + k] = mx[k]; }
        o[6] = (float)bad;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        float v = s_box[0][threadIdx.x];
        for (int w = 1; w < 4; ++w) {
            const float o = s_box[w][threadIdx.x];
            v = threadIdx.x < 3 ? fminf(v, o) : fmaxf(v, o);
        }
        a.box[((long long)blockIdx.y * kBoxBlocks + blockIdx.x) * 8 + threadIdx.x] = v;
    }
}

__device__ inline int bits_for(unsigned long long v)  // bits that hold v
{
    return v ? 64 - __clzll(v) : 0;
}

// One workgroup: a wave joins a cloud's partial boxes and its first lane
// derives the cloud's grid (reference side) or cluster parameters (query
// side); then the cell tables' bases and the key widths of all pairs.
constexpr int kParamPairs = 512;  // pairs per round
__global__ __launch_bounds__(1024) void params_kernel(const ViewArgs a)
{
    __shared__ long long s_nc[kParamPairs];
    __shared__ int s_bad, s_mbits, s_max;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int cbits = bits_for((unsigned long long)(a.B - 1));
    const int maxbits = min(kCurveBits, (kKeyBits - cbits) / 3);
    if (threadIdx.x == 0) { s_bad = 0; s_mbits = 1; s_max = 1; }
    for (int i = threadIdx.x; i < kCostBuckets; i += 1024) a.info->hist[i] = 0;
    long long base = 0;  // (thread 0)
    for (int p0 = 0; p0 < a.B; p0 += kParamPairs) {
        const int np = min(kParamPairs, a.B - p0);
        __syncthreads();
        for (int c = wv; c < 2 * np; c += 16) {
            const int b = p0 + (c >> 1), side = c & 1;
            float v[7];
#pragma unroll
            for (int k = 0; k < 7; ++k)
                v[k] = lane < a.boxblocks ? a.box[((2LL * b + side) * kBoxBlocks + lane) * 8 + k]
                                          : (k < 3 ? INFINITY : k < 6 ? -INFINITY : 0.0f);
            for (int off = 32; off > 0; off >>= 1)
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    const float o = __shfl_xor(v[k], off);
                    v[k] = k < 3 ? fminf(v[k], o) : fmaxf(v[k], o);
                }
            if (lane != 0) continue;
            const PairIn &in = a.in[b];
            const long long n = side ? in.nz : in.nx;
            // (a cloud without any finite point on an axis gets an empty box;
            // the call ends with an error before its views are used)
            const bool none = n == 0 || !(v[0] <= v[3]) || !(v[1] <= v[4]) || !(v[2] <= v[5]);
            double lo[3], hi[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) { lo[k] = none ? 0.0 : (double)v[k]; hi[k] = none ? 0.0 : (double)v[3 + k]; }
            if (v[6] != 0.0f) s_bad = 1;
            const double ext = fmax(fmax(hi[0] - lo[0], hi[1] - lo[1]), fmax(hi[2] - lo[2], 1e-6));
            if (side == 0) {
                GridDesc g;
                double h = isfinite(in.rc) ? in.cell_factor * in.rc : ext * 1.01;
                h = fmax(h, ext * 1e-6);
                double nn[3], inv;
                for (;;) {
                    inv = 1.0 / h;
                    // same expression as the binning: floor((p - o) * inv_h)
#pragma unroll
                    for (int k = 0; k < 3; ++k) nn[k] = floor((hi[k] - lo[k]) * inv) + 1.0;
                    if (nn[0] * nn[1] * nn[2] <= (double)kCellCap) break;
                    h *= 1.25;
                }
                if (none) { h = inv = 1.0; nn[0] = nn[1] = nn[2] = 1.0; }
                g.ox = lo[0]; g.oy = lo[1]; g.oz = lo[2];
                g.h = h;
                g.inv_h = inv;
                g.nx = (int)nn[0]; g.ny = (int)nn[1]; g.nz = (int)nn[2];
                g.cell_base = 0;
                g.pt_base = in.xb;
                g.n = n;
                a.grid[b] = g;
                const long long nc = (long long)g.nx * g.ny * g.nz;
                s_nc[b - p0] = nc;
                atomicMax(&s_max, (int)nc);
            } else {
                // octree blocks need 16 quanta per cap; chunks only use the
                // order along the curve, which a finer quantum makes more local
                const double cap = isfinite(in.rc) ? in.cluster_factor * in.rc : ext * 2.0;
                int L = in.octree ? 4 : 5;
                double q = cap / (double)(1 << L);
                // quanta needed to cover the box must fit in maxbits per axis
                if (!(ext / q + 1.0 <= (double)(1 << maxbits))) {
                    q = ext / ((double)(1 << maxbits) - 2.0);
                    const double r = cap / q;
                    L = r < 2.0 ? 0 : (r >= 1048576.0 ? 20 : 31 - __clz((int)r));
                }
                L = min(L, maxbits);
                ClusterParam cp;
                cp.ox = lo[0]; cp.oy = lo[1]; cp.oz = lo[2];
                cp.iq = 1.0 / q;
                cp.cap = cap;
                cp.level = L;
                // quanta along the widest axis (+1 for rounding at the far face)
                cp.bits = min(max(max(L, 1), bits_for((unsigned long long)floor(ext / q) + 1)), maxbits);
                a.cand[b] = 0;
                a.cp[b] = cp;
                atomicMax(&s_mbits, cp.bits);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < np; ++i) {
                const long long nc = s_nc[i];
                s_nc[i] = base;
                base += nc + 1;
            }
        __syncthreads();
        for (int i = threadIdx.x; i < np; i += 1024) a.grid[p0 + i].cell_base = (int)min(s_nc[i], 0x7fffffffLL);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        BuildInfo &f = *a.info;
        f.pieces = 0;
        f.slots = 0;
        f.cells = base;
        f.bad = s_bad;
        f.overflow = base > a.cell_cap;
        f.nclus = 0;
        f.kbits = bits_for((unsigned long long)s_max);  // the cell count itself must fit
        f.mbits = s_mbits;
        f.sbits[0] = f.kbits + cbits;
        f.sbits[1] = 3 * f.mbits + cbits;
        f.passes = max(a.n[0] > 1 ? (f.sbits[0] + 7) / 8 : 0, a.n[1] > 1 ? (f.sbits[1] + 7) / 8 : 0);
    }
}

// ---------------------------------------------------------------- keys
// Cell index along one axis: floor((p - o) * s) in FP64, clamped, with s the
// same 1/h (or 1/q) the range computations use.  Subtraction and
// multiplication by a positive constant are monotone under rounding, so a
// point inside [lo, hi] lands in a cell between those of lo and hi.
__device__ inline int cell_of(float p, double o, double s, int n)
{
    double f = floor(((double)p - o) * s);
    f = fmin(fmax(f, 0.0), (double)(n - 1));
    return (int)f;
}

__device__ inline unsigned long long spread3(unsigned long long v)
{
    // spread the low 21 bits of v so bit k lands at bit 3k
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x1f00000000ffffULL;
    v = (v | (v << 16)) & 0x1f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

// Index of a quantised point along a Hilbert curve of `bits` bits per axis (the
// transpose method of J. Skilling, "Programming the Hilbert curve", 2004).  Like
// a Morton code its leading 3 k bits name an octree block, but consecutive blocks
// always touch, so runs of points are more compact: the pairs within the cutoff
// among those a cluster's cull lets through rise from 0.58 to 0.62 (RGB-D 40,000,
// ell 0.1), 0.40 to 0.45 (ell 0.05), 0.50 to 0.55 (stereo 30,000, ell 0.1).
__device__ inline unsigned long long hilbert3(unsigned x, unsigned y, unsigned z, int bits)
{
    unsigned X[3] = {x, y, z};
    for (unsigned q = 1u << (bits - 1); q > 1; q >>= 1) {
        const unsigned p = q - 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (X[i] & q) {
                X[0] ^= p;
            } else {
                const unsigned t = (X[0] ^ X[i]) & p;
                X[0] ^= t;
                X[i] ^= t;
            }
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    unsigned t = 0;
    for (unsigned q = 1u << (bits - 1); q > 1; q >>= 1)
        if (X[2] & q) t ^= q - 1;
    X[0] ^= t;
    X[1] ^= t;
    X[2] ^= t;
    return spread3(X[2]) | (spread3(X[1]) << 1) | (spread3(X[0]) << 2);
}

// The pair of global point i of a side (xb / zb ascend; empty clouds skipped).
__device__ inline int pair_of(const ViewArgs &a, int side, long long i)
{
    int lo = 0, hi = a.B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((side ? a.in[mid].zb : a.in[mid].xb) <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__host__ __device__ inline int tiles_of(long long n) { return (int)((n + kRadixTile - 1) / kRadixTile); }

// Digit table of pass `pass` of a side: 256 counts per tile of the keys as
// they stand before that pass.
__device__ inline int *digit_table(const ViewArgs &a, int side, int pass)
{
    const long long t0 = tiles_of(a.n[0]), t1 = tiles_of(a.n[1]);
    return a.table + 256 * (side ? kMaxPasses * t0 + pass * t1 : pass * t0);
}

// Keys of one tile.  TABLE: also the tile's digit counts of the first pass,
// and the zeros that the passes count the later digits into.
template <bool TABLE>
__global__ __launch_bounds__(1024) void key_kernel(const ViewArgs a)
{
    const int side = blockIdx.y;
    const long long n = a.n[side];
    const long long i = (long long)blockIdx.x * kRadixTile + threadIdx.x;
    if ((long long)blockIdx.x * kRadixTile >= n || a.info->overflow) return;
    __shared__ int h[256];
    if (TABLE) {
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        for (int p = 1 + (threadIdx.x >> 8); p < kMaxPasses; p += 4)
            digit_table(a, side, p)[256 * blockIdx.x + (threadIdx.x & 255)] = 0;
        __syncthreads();
    }
    if (i < n) {
        const int b = pair_of(a, side, i);
        const PairIn &in = a.in[b];
        const float *xyz = (side ? in.zx : in.xx) + 3 * (i - (side ? in.zb : in.xb));
        unsigned long long key;
        if (side == 0) {
            const GridDesc &g = a.grid[b];
            const int ix = cell_of(xyz[0], g.ox, g.inv_h, g.nx);
            const int iy = cell_of(xyz[1], g.oy, g.inv_h, g.ny);
            const int iz = cell_of(xyz[2], g.oz, g.inv_h, g.nz);
            key = (unsigned long long)ix +
                  (unsigned long long)g.nx * ((unsigned long long)iy + (unsigned long long)g.ny * iz);
            key |= (unsigned long long)b << a.info->kbits;
        } else {
            // (the curve of the pair's own bits: another number of them turns it)
            const ClusterParam &g = a.cp[b];
            const int lim = 1 << g.bits;
            key = hilbert3(cell_of(xyz[0], g.ox, g.iq, lim), cell_of(xyz[1], g.oy, g.iq, lim),
                           cell_of(xyz[2], g.oz, g.iq, lim), g.bits);
            key |= (unsigned long long)b << (3 * a.info->mbits);
        }
        const long long o = (side ? a.n[0] : 0) + i;
        a.key[0][o] = key;
        a.val[0][o] = (int)i;
        if (TABLE) atomicAdd(&h[key & 255], 1);
    }
    if (TABLE) {
        __syncthreads();
        if (threadIdx.x < 256) digit_table(a, side, 0)[256 * blockIdx.x + threadIdx.x] = h[threadIdx.x];
    }
}

// ---------------------------------------------------------------- scan
// Exclusive prefix sum of n ints in three launches: per-block scans of 2048
// elements, a single-block scan of the block sums, then the add-back.  (Summed
// as SortPlace: the points of both sides may pass 2^31.)
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ inline SortPlace block_exclusive_scan(SortPlace v, SortPlace *total)
{
    __shared__ SortPlace sh[kScanThreads];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        SortPlace t = (threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    SortPlace incl = sh[threadIdx.x];
    *total = sh[kScanThreads - 1];
    __syncthreads();
    return incl - v;
}

__device__ __forceinline__ bool scan_skips(const int *passes, int pass) { return passes && pass >= *passes; }

__global__ __launch_bounds__(kScanThreads) void scan_tiles(const int *in, int *out, int *bsum, long long n,
                                                           const int *passes, int pass)
{
    if (scan_skips(passes, pass)) return;
    const long long base = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanItems;
    SortPlace v[kScanItems];
    SortPlace s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        s += v[k];
    }
    SortPlace tot;
    SortPlace ex = block_exclusive_scan(s, &tot);
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = (int)ex;
        ex += v[k];
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = (int)tot;
}

__global__ __launch_bounds__(kScanThreads) void scan_sums(int *bsum, int nb, int *total, const int *passes, int pass)
{
    if (scan_skips(passes, pass)) return;
    // nb <= kScanTile * kScanTile is guaranteed by the launcher (chunks of 2048)
    SortPlace carry = 0;
    for (int base = 0; base < nb; base += kScanTile) {
        const int b0 = base + threadIdx.x * kScanItems;
        SortPlace v[kScanItems];
        SortPlace s = 0;
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = (b0 + k < nb) ? bsum[b0 + k] : 0;
            s += v[k];
        }
        SortPlace tot;
        SortPlace ex = block_exclusive_scan(s, &tot) + carry;
        for (int k = 0; k < kScanItems; ++k) {
            if (b0 + k < nb) bsum[b0 + k] = (int)ex;
            ex += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0 && total) *total = (int)carry;
}

__global__ __launch_bounds__(kScanThreads) void scan_add(int *out, const int *bsum, long long n, const int *passes,
                                                         int pass)
{
    if (scan_skips(passes, pass)) return;
    const long long base = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanItems;
    const SortPlace add = bsum[blockIdx.x];
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) out[base + k] = (int)(out[base + k] + add);
}

void launch_exclusive_scan(const int *in, int *out, int *bsum, long long n, int *total, hipStream_t s,
                           const int *passes, int pass)
{
    const int nb = (int)((n + kScanTile - 1) / kScanTile);
    if (nb == 0) {
        if (total) hipMemsetAsync(total, 0, sizeof(int), s);
        return;
    }
    hipLaunchKernelGGL(scan_tiles, dim3(nb), dim3(kScanThreads), 0, s, in, out, bsum, n, passes, pass);
    hipLaunchKernelGGL(scan_sums, dim3(1), dim3(kScanThreads), 0, s, bsum, nb, total, passes, pass);
    hipLaunchKernelGGL(scan_add, dim3(nb), dim3(kScanThreads), 0, s, out, bsum, n, passes, pass);
}

// ---------------------------------------------------------------- radix sort
// Passes alternate between the two buffers; after the last one the sorted
// keys are in buffer (passes & 1).
__device__ inline int passes_of(const ViewArgs &a, int side) { return a.n[side] > 1 ? (a.info->sbits[side] + 7) / 8 : 0; }

// The lanes of the wave with the same value of `bits` bits as this one.
template <int BITS> __device__ __forceinline__ unsigned long long wave_match(int v)
{
    unsigned long long peers = ~0ULL;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const unsigned long long bal = __ballot((v >> b) & 1);
        peers &= ((v >> b) & 1) ? bal : ~bal;
    }
    return peers;
}

// Rank of this lane's digit among the earlier lanes of its wave with the same
// digit, and the number of lanes that hold it (invalid lanes: digit 256).
__device__ __forceinline__ void wave_rank(int d, int lane, int &rank, int &count)
{
    const unsigned long long peers = wave_match<9>(d);
    rank = __popcll(peers & ((1ULL << lane) - 1ULL));
    count = __popcll(peers);
}

// One pass in one launch, both sides (blockIdx.y).  A tile finds where its
// digits go from the pass's digit table: the counts of all tiles (each
// thread adds a quarter of them for one digit), an exclusive scan over the
// digits, and the counts of the tiles before it.  Its 1,024 keys are ranked
// stably (earlier lanes of the wave, earlier waves) and written, and counted
// into the next pass's table at the tile they land in (one atomic per wave for
// the keys that share tile and digit: the high digits of neighbours agree,
// and one atomic per key on the same counter took 12.7 us at 15 tiles).
// Latency bound: 4.1 us per launch at 2 tiles a side, 6.1 us at 15, 7.4 us at
// 40, for both sides, against about 19 us for one side's histogram, three scan
// launches and scatter.  Every tile reads the whole table, so beyond
// kTableTiles tiles (128 KB read per tile) the separate launches win.
__global__ __launch_bounds__(1024) void sort_pass(const ViewArgs a, int pass)
{
    const int side = blockIdx.y;
    const long long n = a.n[side];
    const int ntiles = tiles_of(n);
    const int tile = blockIdx.x;
    if (tile >= ntiles || pass >= passes_of(a, side) || a.info->overflow) return;
    __shared__ int s_tot[4][256], s_bef[4][256], s_base[256], s_w[4];
    __shared__ int s_cnt[16][256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int part = tid >> 8, d0 = tid & 255;
    const long long o = side ? a.n[0] : 0;
    const int e = tile * kRadixTile + tid;
    const bool valid = e < n;
    const unsigned long long key = valid ? a.key[pass & 1][o + e] : 0ULL;
    const int val = valid ? a.val[pass & 1][o + e] : 0;
    {
        const int *tb = digit_table(a, side, pass);
        int tot = 0, bef = 0;
        for (int t = part; t < ntiles; t += 4) {
            const int c = tb[256 * t + d0];
            tot += c;
            bef += t < tile ? c : 0;
        }
        s_tot[part][d0] = tot;
        s_bef[part][d0] = bef;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) s_cnt[4 * part + k][d0] = 0;
    const int d = valid ? (int)((key >> (8 * pass)) & 255) : 256;
    int rank, count;
    wave_rank(d, lane, rank, count);
    __syncthreads();
    if (valid && rank == 0) s_cnt[wv][d] = count;
    int tot = 0, incl = 0;
    if (tid < 256) {
        tot = s_tot[0][tid] + s_tot[1][tid] + s_tot[2][tid] + s_tot[3][tid];
        incl = wave_scan_add(tot);
        if (lane == 63) s_w[wv] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        int acc = incl - tot + s_bef[0][tid] + s_bef[1][tid] + s_bef[2][tid] + s_bef[3][tid];
        for (int w = 0; w < wv; ++w) acc += s_w[w];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int c = s_cnt[w][tid];
            s_cnt[w][tid] = acc;
            acc += c;
        }
    }
    __syncthreads();
    int place = -1;  // counter of the next pass: destination tile and next digit
    if (valid) {
        const int pos = s_cnt[wv][d] + rank;
        a.key[(pass + 1) & 1][o + pos] = key;
        a.val[(pass + 1) & 1][o + pos] = val;
        place = 256 * (pos / kRadixTile) + (int)((key >> (8 * pass + 8)) & 255);
    }
    if (pass + 1 < passes_of(a, side)) {
        static_assert(kTableTiles <= 256, "a counter's number takes 16 bits");
        const unsigned long long same = wave_match<17>(place);  // (bit 16: invalid lanes)
        if (valid && (same & ((1ULL << lane) - 1ULL)) == 0)
            atomicAdd(&digit_table(a, side, pass + 1)[place], __popcll(same));
    }
}

// The passes of a large sort, both sides in the same launches: a histogram
// per tile (digit-major, the query side's after the reference side's), the
// scan of all of them, and the scatter.  The scan runs on from one side to
// the next as their keys do, so its values are places in the joint buffers.
// (A side that needs no more passes still counts, so that holds for the other;
// beyond the last pass of both nothing is counted or moved.)
__global__ __launch_bounds__(1024) void radix_hist(const ViewArgs a, int pass, int *hist)
{
    const int side = blockIdx.y, ntiles = tiles_of(a.n[side]);
    if (blockIdx.x >= ntiles || a.info->overflow || pass >= a.info->passes) return;
    __shared__ int h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const long long e = (long long)blockIdx.x * kRadixTile + threadIdx.x;
    const int buf = min(pass, passes_of(a, side)) & 1;
    if (e < a.n[side]) atomicAdd(&h[(a.key[buf][(side ? a.n[0] : 0) + e] >> (8 * pass)) & 255], 1);
    __syncthreads();
    const long long t0 = side ? tiles_of(a.n[0]) : 0;
    if (threadIdx.x < 256) hist[256 * t0 + (long long)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(1024) void radix_scatter(const ViewArgs a, int pass, const int *hist)
{
    const int side = blockIdx.y, ntiles = tiles_of(a.n[side]);
    if (blockIdx.x >= ntiles || pass >= passes_of(a, side) || a.info->overflow) return;
    __shared__ SortPlace s_cnt[16][256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const long long o = side ? a.n[0] : 0;
    const long long e = (long long)blockIdx.x * kRadixTile + tid;
    const bool valid = e < a.n[side];
    const unsigned long long key = valid ? a.key[pass & 1][o + e] : 0ULL;
    const int val = valid ? a.val[pass & 1][o + e] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) s_cnt[4 * (tid >> 8) + k][tid & 255] = 0;
    const int d = valid ? (int)((key >> (8 * pass)) & 255) : 256;
    int rank, count;
    wave_rank(d, lane, rank, count);
    __syncthreads();
    if (valid && rank == 0) s_cnt[wv][d] = count;
    __syncthreads();
    if (tid < 256) {
        const long long t0 = side ? tiles_of(a.n[0]) : 0;
        SortPlace acc = hist[256 * t0 + (long long)tid * ntiles + blockIdx.x];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const SortPlace c = s_cnt[w][tid];
            s_cnt[w][tid] = acc;
            acc += c;
        }
    }
    __syncthreads();
    if (valid) {
        const SortPlace pos = s_cnt[wv][d] + rank;
        a.key[(pass + 1) & 1][pos] = key;
        a.val[(pass + 1) & 1][pos] = val;
    }
}

// ---------------------------------------------------------------- views
__device__ inline long long lower_bound_u64(const unsigned long long *a, long long n, unsigned long long x)
{
    long long lo = 0, hi = n;
    while (lo < hi) {
        long long mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The key that entry k of the joint cell tables counts up to: the entry is
// the number of keys below it.
__device__ __forceinline__ unsigned long long entry_key(const ViewArgs &a, int kbits, long long k)
{
    int lo = 0, hi = a.B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.grid[mid].cell_base <= k) lo = mid; else hi = mid - 1;
    }
    return ((unsigned long long)lo << kbits) | (unsigned long long)(k - a.grid[lo].cell_base);
}

// Number of sorted keys below x, found by one wave: each round the lanes probe
// 64 evenly spaced keys (three rounds up to 262,144 keys, where a bisection
// takes 18 dependent loads).
__device__ __forceinline__ int wave_lower_bound(const unsigned long long *keys, long long n, unsigned long long x)
{
    const int lane = threadIdx.x & 63;
    long long lo = 0, len = n;  // the answer is in [lo, lo + len]
    while (len > 0) {
        const long long step = (len + 63) / 64;
        const long long i = lo + (lane + 1LL) * step - 1;
        const bool less = i < lo + len && keys[min(i, n - 1)] < x;
        const int c = __popcll(__ballot(less));  // the first c probes are below x
        const long long end = lo + len;
        lo += c * step;
        len = max(0LL, min(step - 1, end - lo));
    }
    return (int)lo;
}

// The cell tables, 256 consecutive entries per wave and turn: two searches
// find the run of keys that falls in them.  Most of a grid of surfaces is
// empty and is filled with one value; elsewhere each lane bisects the run for
// its four entries at once (their loads overlap).  One bisection per entry
// over all keys costs 15 dependent loads for each of up to 8 million entries:
// 40 us at 14,873 points and half-radius cells of 0.15 m, now 7.
__device__ void cell_entries(const ViewArgs &a)
{
    const unsigned long long *keys = a.key[passes_of(a, 0) & 1];
    const int kbits = a.info->kbits;
    const long long total = a.info->cells, n = a.n[0];
    const int lane = threadIdx.x & 63;
    for (long long k0 = 256LL * (blockIdx.x * 4LL + (threadIdx.x >> 6)); k0 < total; k0 += 1024LL * gridDim.x) {
        const long long last = min(k0 + 255, total - 1);
        const int lo = wave_lower_bound(keys, n, entry_key(a, kbits, k0));
        const int hi = wave_lower_bound(keys, n, entry_key(a, kbits, last));
        const long long k = k0 + 4 * lane;
        int e[4] = {lo, lo, lo, lo};
        if (lo < hi) {
            unsigned long long x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = entry_key(a, kbits, min(k + q, last));
            int len = hi - lo;
            while (len > 1) {
                const int half = len >> 1;
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] += keys[e[q] + half - 1] < x[q] ? half : 0;
                len -= half;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] += keys[e[q]] < x[q] ? 1 : 0;
        }
        if (k + 3 <= last) {
            *reinterpret_cast<int4 *>(a.cell_start + k) = make_int4(e[0], e[1], e[2], e[3]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + q <= last) a.cell_start[k + q] = e[q];
        }
    }
}

// blockIdx.y 0 and 1: sorted copies of a side -- the float4 coordinates and
// the padded feature row, one float4 per thread, so a row is read and written
// by consecutive threads (destination column k = source column col[k] times
// scale[k]).  blockIdx.y 2: the cell tables.
__global__ __launch_bounds__(256) void view_kernel(const ViewArgs a, const FeatLayout lay)
{
    if (a.info->overflow) return;
    const int side = blockIdx.y;
    if (side == 2) {
        cell_entries(a);
        return;
    }
    __shared__ int s_col[64];
    __shared__ float s_scale[64];
    if (threadIdx.x < 64) {
        s_col[threadIdx.x] = lay.col[threadIdx.x];
        s_scale[threadIdx.x] = lay.scale[threadIdx.x];
    }
    __syncthreads();
    const int buf = passes_of(a, side) & 1;
    const long long o = side ? a.n[0] : 0;
    const int shift = side ? 3 * a.info->mbits : a.info->kbits;
    const int f4 = lay.d4 / 4, items = f4 + 1;
    const long long total = a.n[side] * items;
    for (long long w = (long long)blockIdx.x * 256 + threadIdx.x; w < total; w += (long long)gridDim.x * 256) {
        const long long p = total < (1LL << 31) ? (long long)((unsigned)w / (unsigned)items) : w / items;
        const int f = (int)(w - p * items);
        const int b = (int)(a.key[buf][o + p] >> shift);
        const PairIn &in = a.in[b];
        const long long i = a.val[buf][o + p] - (side ? in.zb : in.xb);
        if (f == f4) {
            const float *xyz = (side ? in.zx : in.xx) + 3 * i;
            a.pts[side][p] = make_float4(xyz[0], xyz[1], xyz[2], 0.0f);
            if (side) a.perm[p] = (int)i;
            continue;
        }
        const float *row = (side ? in.zf : in.xf) + i * lay.src_dim;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * f + q, col = s_col[k];
            v[q] = 0.0f;
            if (col >= 0) {
                v[q] = row[col] * s_scale[k];
            } else if (col == -2) {
                // tensor-product column of the folded LIN blocks (eq. (6))
                int cc = k - lay.sed;
                v[q] = 1.0f;
                for (int l = lay.nlin - 1; l >= 0; --l) {
                    v[q] *= row[lay.lin_src[l] + cc % lay.lin_dim[l]];
                    cc /= lay.lin_dim[l];
                }
            }
        }
        reinterpret_cast<float4 *>(a.feat[side])[p * f4 + f] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// ---------------------------------------------------------------- clusters and plan
constexpr int kHalo = 64;         // points beside a block that a cluster may reach
constexpr int kClusThreads = 256;
constexpr int kClusBlocks = 256;  // blocks up to which a block takes fewer points

// A block takes PTS points.  One thread per point finds the point's cluster; the first
// point of a cluster is its head.
//   octree rule: the largest aligned octree block (level <= ClusterParam.level)
//     holding at most cluster_max points.  Block counts grow with the level, so
//     every point of a block makes the same choice, and a block of at most 64
//     points lies within the staged neighbours: its ends are found by walking
//     outward while the keys agree.  A level-0 block with more points is cut
//     into ceil(count / cluster_max) near-equal runs.
//   chunk rule: chunks of cluster_max consecutive points of the cloud, halved
//     until the part's bounding box edge is within ClusterParam.cap or the part
//     is one point.
// Then 2 to 64 lanes per head count the candidates of its neighbourhood at
// the current pose (one grid row per lane and turn).
// The kernel is a chain of dependent loads, so fewer points per block (more
// blocks, more lanes per head) are faster until the blocks' atomics become
// the bound: blocks of 64 / 256 points take 14.2 / 25.0 us at 15,000 points
// and 20.5 / 13.3 us at 30,000, so a block takes as few as keep their number
// within 256.
template <int PTS>
__global__ __launch_bounds__(kClusThreads) void cluster_kernel(const ViewArgs a, double kappa)
{
    constexpr int kClusSpan = PTS + 2 * kHalo;
    if (a.info->overflow) return;
    __shared__ float4 s_pt[kClusSpan];
    __shared__ unsigned long long s_key[kClusSpan];
    __shared__ Geo s_geo[PTS];
    __shared__ int s_first[PTS], s_n[PTS], s_b[PTS], s_C[PTS];
    __shared__ int s_w[4], s_heads, s_cbase;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const long long N = a.n[1];
    const long long p0 = (long long)blockIdx.x * PTS;
    const int buf = passes_of(a, 1) & 1;
    const unsigned long long *keys = a.key[buf] + a.n[0];
    for (int k = tid; k < kClusSpan; k += kClusThreads) {
        const long long p = p0 - kHalo + k;
        const bool in = p >= 0 && p < N;
        s_pt[k] = in ? a.pts[1][p] : make_float4(0.f, 0.f, 0.f, 0.f);
        s_key[k] = in ? keys[p] : ~0ULL;
    }
    __syncthreads();
    const long long p = p0 + tid;
    const int shift = 3 * a.info->mbits;
    bool head = false;
    int cnt = 0, b = 0;
    if (tid < PTS && p < N) {
        const int me = tid + kHalo;
        const unsigned long long key = s_key[me];
        b = (int)(key >> shift);
        const PairIn &in = a.in[b];
        const ClusterParam &cp = a.cp[b];
        const int tpw = in.cluster_max;
        long long start = p;
        if (!in.octree) {
            const long long rel = p - in.zb;
            const long long c0 = in.zb + rel / tpw * tpw;
            const int len = (int)min((long long)tpw, in.zb + in.nz - c0);
            const int l = (int)(p - c0);
            for (int sz = tpw;; sz >>= 1) {
                const int first = l & ~(sz - 1);
                const int plen = min(sz, len - first);
                const float4 *q = &s_pt[me - l + first];
                float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
                for (int k = 0; k < plen; ++k) {
                    const float4 v = q[k];
                    lo[0] = fminf(lo[0], v.x); hi[0] = fmaxf(hi[0], v.x);
                    lo[1] = fminf(lo[1], v.y); hi[1] = fmaxf(hi[1], v.y);
                    lo[2] = fminf(lo[2], v.z); hi[2] = fmaxf(hi[2], v.z);
                }
                const double edge = fmax((double)hi[0] - lo[0], fmax((double)hi[1] - lo[1], (double)hi[2] - lo[2]));
                if (edge <= cp.cap || plen <= 1) {
                    start = c0 + first;
                    cnt = plen;
                    break;
                }
            }
        } else {
            int lo = me, hi = me + 1;  // staged indices of the block at level L
            for (int L = 0; L <= cp.level; ++L) {
                const unsigned long long blk = key >> (3 * L);
                while (hi - lo <= tpw && lo > 0 && s_key[lo - 1] >> (3 * L) == blk) --lo;
                while (hi - lo <= tpw && hi < kClusSpan && s_key[hi] >> (3 * L) == blk) ++hi;
                if (hi - lo > tpw) {
                    if (L == 0) {
                        const long long lo0 = lower_bound_u64(keys, N, key), hi0 = lower_bound_u64(keys, N, key + 1);
                        const long long all = hi0 - lo0, nch = (all + tpw - 1) / tpw, sz = (all + nch - 1) / nch;
                        start = lo0 + (p - lo0) / sz * sz;
                        cnt = (int)(min(start + sz, hi0) - start);
                    }
                    break;
                }
                start = p0 - kHalo + lo;
                cnt = hi - lo;
            }
        }
        head = p == start;
    }
    // the block's heads, compacted in order, with their geometry
    {
        const unsigned long long m = __ballot(head);
        if (lane == 0) s_w[wv] = __popcll(m);
        __syncthreads();
        int k = __popcll(m & ((1ULL << lane) - 1ULL));
        for (int w = 0; w < wv; ++w) k += s_w[w];
        if (tid == 0) s_heads = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        if (head) {
            const float4 *q = &s_pt[tid + kHalo];
            double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
            for (int i = 0; i < cnt; ++i) {
                const double v[3] = {(double)q[i].x, (double)q[i].y, (double)q[i].z};
                for (int c = 0; c < 3; ++c) { lo[c] = fmin(lo[c], v[c]); hi[c] = fmax(hi[c], v[c]); }
            }
            double cc[3], r2 = 0.0, mag = 0.0;
            for (int c = 0; c < 3; ++c) { cc[c] = 0.5 * (lo[c] + hi[c]); mag = fmax(mag, fabs(cc[c])); }
            for (int i = 0; i < cnt; ++i) {
                const double dx = (double)q[i].x - cc[0], dy = (double)q[i].y - cc[1], dz = (double)q[i].z - cc[2];
                r2 = fmax(r2, dx * dx + dy * dy + dz * dz);
            }
            // inflate so FP64 rounding of the transformed centre and points can
            // never place a member outside the sphere
            const double r = sqrt(r2) * (1.0 + 1e-12) + 1e-12 * (mag + 1.0);
            s_geo[k] = Geo{cc[0], cc[1], cc[2], r};
            s_first[k] = (int)p;
            s_n[k] = cnt;
            s_b[k] = b;
        }
        __syncthreads();
    }
    const int nh = s_heads;
    const bool cut = isfinite(kappa);
    // lanes per head: as many as leave at most two turns (nh <= 256 / 2)
    const int lg = nh > 128 ? 1 : (nh > 64 ? 2 : (nh > 32 ? 3 : (nh > 16 ? 4 : (nh > 8 ? 5 : 6))));
    const int G = 1 << lg, lg_ = tid & (G - 1);
    for (int k0 = 0; k0 < nh; k0 += kClusThreads >> lg) {
        const int k = k0 + (tid >> lg);
        int C = 0;
        if (k < nh) {
            const int kb = s_b[k];
            double Pm[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) Pm[i] = a.in[kb].pose[i];
            const GridDesc gd = a.grid[kb];
            const Neighbourhood nb = neighbourhood(Pm, s_geo[k], a.in[kb].rc, cut, gd);
            if (nb.any) {
                const int nyr = nb.iy1 - nb.iy0 + 1, nrows = nyr * (nb.iz1 - nb.iz0 + 1);
                const BallRows br = ball_rows(nb, gd, cut);
#pragma unroll 4
                for (int r = lg_; r < nrows; r += G) {
                    const int iy = nb.iy0 + r % nyr, iz = nb.iz0 + r / nyr;
                    int i0, i1;
                    if (!row_cells(nb, br, iy, iz, i0, i1)) continue;
                    const long long c0 = (long long)gd.cell_base + (long long)gd.nx * (iy + (long long)gd.ny * iz);
                    C += a.cell_start[c0 + i1 + 1] - a.cell_start[c0 + i0];
                }
            }
        }
        for (int off = G >> 1; off > 0; off >>= 1) C += __shfl_xor(C, off);
        if (lg_ == 0 && k < nh) s_C[k] = C;
    }
    __syncthreads();
    const int C = tid < nh ? s_C[tid] : 0;
    if (tid == 0 && nh > 0) s_cbase = atomicAdd(&a.info->nclus, nh);
    // the candidates, by pair: one add a wave where it has clusters of one pair
    if (wv * 64 < nh) {
        const int mine = s_b[min(tid, nh - 1)], first = wave_uniform(mine);
        if (__all(mine == first)) {
            unsigned long long sum = C;
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == 0) atomicAdd(&a.cand[first], sum);
        } else if (tid < nh) {
            atomicAdd(&a.cand[mine], (unsigned long long)C);
        }
    }
    __syncthreads();
    if (tid < nh) {
        ClusterRec r;
        r.geo = s_geo[tid];
        r.first = s_first[tid];
        r.n = s_n[tid];
        r.cand = C;
        r.np = r.slot = r.code = r.place = 0;
        r.b = s_b[tid];
        r.inverse = a.in[r.b].inverse;
        r.pad[0] = r.pad[1] = r.pad[2] = 0;
        a.clus[s_cbase + tid] = r;
    }
}

// The pieces of every cluster, c_max = max(floor, work / n) candidates each (the
// floor from the candidates of the pair's clusters, see kPieceTarget), their output
// slots, their places in the dispatch order's cost buckets and the query map.
// A block reserves slots and bucket places for its 256 clusters with one
// atomic each (an atomic per cluster serialises on the few buckets that most
// clusters of a sparse cloud share: 22 us for 1,900 of them).
__global__ __launch_bounds__(256) void plan_kernel(const ViewArgs a)
{
    if (a.info->overflow) return;
    const int nclus = a.info->nclus;
    const int c0 = blockIdx.x * 256;
    if (c0 >= nclus) return;
    __shared__ int s_first[256], s_n[256], s_np[256], s_slot[256];
    __shared__ int s_hist[kCostBuckets];
    __shared__ int s_w[4], s_w2[4];
    __shared__ unsigned long long s_base;  // first slot of the block's clusters
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int k = tid; k < kCostBuckets; k += 256) s_hist[k] = 0;
    ClusterRec *rec = a.clus + c0 + tid;
    const bool in = c0 + tid < nclus;
    int n = 0, np = 0, C = 0, first = 0;
    if (in) {
        n = rec->n;
        C = rec->cand;
        first = rec->first;
        const unsigned long long even = (a.cand[rec->b] / kPieceTarget + 63) & ~63ULL;
        const int floor_ = (int)min(max(even, (unsigned long long)kPieceFew), (unsigned long long)kPieceMany);
        const int cm = max(floor_, a.work / n);
        np = C > 0 ? min((C + cm - 1) / cm, 4096) : 1;
    }
    const int ns = np * n;
    const int ip = wave_scan_add(np), is = wave_scan_add(ns);
    if (lane == 63) { s_w[wv] = ip; s_w2[wv] = is; }
    __syncthreads();
    int code = 0, place = 0;
    if (in) {
        const int cand = (C + np - 1) / np;  // candidates per piece
        code = kCostBuckets - 1 - cost_bucket((unsigned long long)n * (unsigned long long)(cand + 64));
        place = atomicAdd(&s_hist[code], np);
    }
    __syncthreads();
    for (int k = tid; k < kCostBuckets; k += 256)
        if (s_hist[k] > 0) s_hist[k] = atomicAdd(&a.info->hist[k], s_hist[k]);
    if (tid == 0) s_base = atomicAdd(&a.info->slots, (unsigned long long)(s_w2[0] + s_w2[1] + s_w2[2] + s_w2[3]));
    if (tid == 64) atomicAdd(&a.info->pieces, (unsigned long long)(s_w[0] + s_w[1] + s_w[2] + s_w[3]));
    __syncthreads();
    int slot = (int)s_base + is - ns;  // (of no use, and not used, in a plan that does not fit)
    for (int w = 0; w < wv; ++w) slot += s_w2[w];
    s_first[tid] = first;
    s_n[tid] = n;
    s_np[tid] = np;
    s_slot[tid] = slot;
    if (in) {
        rec->np = np;
        rec->slot = slot;
        rec->code = code;
        rec->place = s_hist[code] + place;
    }
    __syncthreads();
    for (int k = tid >> 4; k < 256; k += 16)
        for (int t = tid & 15; t < s_n[k]; t += 16) a.qmap[s_first[k] + t] = make_int4(t, s_n[k], s_np[k], s_slot[k] + t);
}

// The pieces' records, bucket by bucket (heaviest first; a cluster's pieces
// together): 16 lanes per cluster write them.  Nothing is written when there
// is no room for all of them, or the plan does not fit.  The build's counts are posted to the host first.
__global__ __launch_bounds__(256) void record_kernel(const ViewArgs a)
{
    static_assert(kCostBuckets == 512, "two buckets per thread");
    __shared__ int s_base[kCostBuckets];
    __shared__ int s_w[4];
    const BuildInfo *f = a.info;
    if (a.mail && blockIdx.x == 0 && threadIdx.x == 0) {
        HostMail *m = a.mail;
        __hip_atomic_store(&m->pieces, f->pieces, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m->slots, f->slots, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m->cells, f->cells, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m->bad, f->bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m->overflow, f->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m->build, a.build, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (f->overflow || !plan_fits(f->pieces, f->slots) || f->pieces > (unsigned long long)a.rec_cap) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l16 = tid & 15;
    const int h0 = f->hist[2 * tid], h1 = f->hist[2 * tid + 1];
    const int incl = wave_scan_add(h0 + h1);
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    int ex = incl - h0 - h1;
    for (int w = 0; w < wv; ++w) ex += s_w[w];
    s_base[2 * tid] = ex;
    s_base[2 * tid + 1] = ex + h0;
    __syncthreads();
    const int nclus = f->nclus;
    for (int c = blockIdx.x * 16 + (tid >> 4); c < nclus; c += gridDim.x * 16) {
        const ClusterRec r = a.clus[c];
        const int pos = s_base[r.code] + r.place;
        for (int k = l16; k < r.np; k += 16) {
            PieceRec o;
            o.pc = make_int4(r.first, k, r.np, r.slot + k * r.n);
            o.b = r.b;
            o.first = r.first;
            o.n = r.n;
            o.inverse = r.inverse;
            o.geo = r.geo;
            a.recs[pos + k] = o;
        }
    }
}

// ---------------------------------------------------------------- launchers
static int blocks_for(long long n, int threads, int cap = 65535)
{
    return (int)std::min<long long>(std::max<long long>((n + threads - 1) / threads, 1), cap);
}

static bool table_sort(const ViewArgs &a) { return std::max(tiles_of(a.n[0]), tiles_of(a.n[1])) <= kTableTiles; }

long long view_table_ints(long long n0, long long n1)
{
    const long long t0 = tiles_of(n0), t1 = tiles_of(n1);
    const bool table = std::max(t0, t1) <= kTableTiles;
    return 256 * std::max(1LL, (table ? kMaxPasses : 1) * (t0 + t1));
}

long long view_bsum_ints(long long n0, long long n1)
{
    return (256 * ((long long)tiles_of(n0) + tiles_of(n1)) + kScanTile - 1) / kScanTile + 1;
}

void launch_boxes(const ViewArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(box_kernel, dim3(a.boxblocks, 2 * a.B), dim3(256), 0, s, a);
}

void launch_params(const ViewArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(params_kernel, dim3(1), dim3(1024), 0, s, a);
}

void launch_views(const ViewArgs &a, const FeatLayout &lay, double kappa, hipStream_t s)
{
    int cbits = 0;
    while ((1LL << cbits) < a.B) ++cbits;
    // key bits of each side, at most (the device knows the exact number and
    // skips passes beyond it)
    const int most[2] = {24 + cbits, 3 * std::min(kCurveBits, (kKeyBits - cbits) / 3) + cbits};
    const int passes = (std::max(most[0], most[1]) + 7) / 8;
    const int tiles = std::max(tiles_of(a.n[0]), tiles_of(a.n[1]));
    if (tiles > 0) {
        if (table_sort(a)) {
            hipLaunchKernelGGL(key_kernel<true>, dim3(tiles, 2), dim3(kRadixTile), 0, s, a);
            for (int p = 0; p < passes; ++p) hipLaunchKernelGGL(sort_pass, dim3(tiles, 2), dim3(kRadixTile), 0, s, a, p);
        } else {
            hipLaunchKernelGGL(key_kernel<false>, dim3(tiles, 2), dim3(kRadixTile), 0, s, a);
            const long long ints = 256LL * (tiles_of(a.n[0]) + tiles_of(a.n[1]));
            for (int p = 0; p < passes; ++p) {
                hipLaunchKernelGGL(radix_hist, dim3(tiles, 2), dim3(kRadixTile), 0, s, a, p, a.table);
                launch_exclusive_scan(a.table, a.table, a.bsum, ints, nullptr, s, &a.info->passes, p);
                hipLaunchKernelGGL(radix_scatter, dim3(tiles, 2), dim3(kRadixTile), 0, s, a, p, a.table);
            }
        }
    }
    const long long items = std::max(a.n[0], a.n[1]) * (lay.d4 / 4 + 1);
    hipLaunchKernelGGL(view_kernel, dim3(std::max(2048, blocks_for(items, 256, 16384)), 3), dim3(256), 0, s, a, lay);
    if (a.n[1] > 0) {
        if (a.n[1] <= 64 * kClusBlocks)
            hipLaunchKernelGGL(cluster_kernel<64>, dim3(blocks_for(a.n[1], 64)), dim3(kClusThreads), 0, s, a, kappa);
        else if (a.n[1] <= 128 * kClusBlocks)
            hipLaunchKernelGGL(cluster_kernel<128>, dim3(blocks_for(a.n[1], 128)), dim3(kClusThreads), 0, s, a, kappa);
        else
            hipLaunchKernelGGL(cluster_kernel<256>, dim3(blocks_for(a.n[1], 256, 1 << 30)), dim3(kClusThreads), 0, s, a,
                               kappa);
        hipLaunchKernelGGL(plan_kernel, dim3(blocks_for(a.n[1], 256, 1 << 30)), dim3(256), 0, s, a);
    }
}

void launch_records(const ViewArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(record_kernel, dim3(blocks_for(a.n[1], 32, 2048)), dim3(256), 0, s, a);
}

}  // namespace cvo
