// cvo_select.hip -- point selection before registration (the paper's
// performance considerations, Sec. IV): pixels passing the FAST 9-of-16
// segment test, no non-maximum suppression, with the intensity threshold
// chosen so that the number of selected pixels with depth stays within a cap;
// the selection is compacted in raster order and back-projected.
//
//   score(p) = the largest integer t at which p is a corner: an arc A of 9
//              contiguous pixels of the radius-3 circle is all brighter than
//              I_p + t for t <= min_A I - I_p - 1 and all darker than I_p - t
//              for t <= I_p - max_A I - 1, so score(p) is the maximum of
//              these bounds over the 16 arcs (-1: a corner at no threshold,
//              or within 3 pixels of the border).
//   count(t) = #{p with depth : score(p) >= t} is non-increasing in t, so one
//              256-bin histogram of the scores gives every count; the
//              threshold is the smallest t with count(t) <= cap.
//
// Kernels: score + histogram (64 x 16 pixel tiles staged in LDS with a 3-pixel
// halo), threshold and per-block selected counts, and the emit pass (wave
// ballots give each selected pixel its rank).  All integer work, so the
// selection is exact.
//
// An image of 1241 x 376 is 3 MB, a few microseconds; what it takes is launches
// and atomics: with three launches after the clear of the histogram instead of
// seven, 108 -> 81 us a call.
#include "cvo_device.hpp"
#include "cvo_launch.hpp"

namespace cvo {

namespace {
constexpr int kTX = 64, kTY = 4, kTRows = 16;  // score tile: 64 x 16 pixels, 4 per thread
constexpr int kHalo = 3;
constexpr int kSelThreads = 256, kSelPix = 1024;  // pixels per workgroup of the count and emit passes
// Copies of the histogram, by workgroup: adds to one address take about 11 ns
// each, one after the other (1,880 tiles of 64 x 4 adding to one copy: 20 us).
constexpr int kHistCopies = 16;
// Images of at most this many count blocks (2 megapixels): every emit block adds
// up the counts before it by itself, at most 8 per thread, which is cheaper
// than the three launches of a scan; larger ones scan.
constexpr int kDirectBlocks = 2048;
}  // namespace

__global__ __launch_bounds__(kTX *kTY) void fast_score_kernel(const uint8_t *gray, const float *depth, int W, int H,
                                                               float dmin, float dmax, short *key, short *score_out,
                                                               int *hist)
{
    // int cells: byte cells would put four neighbours in one LDS bank
    __shared__ int tile[kTRows + 2 * kHalo][kTX + 2 * kHalo];
    __shared__ int lh[256];
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * kTX + tx;
    const int u0 = blockIdx.x * kTX, v0 = blockIdx.y * kTRows;
    lh[tid] = 0;
    for (int i = tid; i < (kTRows + 2 * kHalo) * (kTX + 2 * kHalo); i += kTX * kTY) {
        const int r = i / (kTX + 2 * kHalo), c = i % (kTX + 2 * kHalo);
        const int u = u0 + c - kHalo, v = v0 + r - kHalo;
        tile[r][c] = (u >= 0 && u < W && v >= 0 && v < H) ? (int)gray[(long long)v * W + u] : 0;
    }
    __syncthreads();
    const int u = u0 + tx;
    for (int row = ty; row < kTRows; row += kTY) {
        const int v = v0 + row;
        if (u >= W || v >= H) break;
        int s = -1;
        if (u >= kHalo && v >= kHalo && u < W - kHalo && v < H - kHalo) {
            // the radius-3 circle, (du, dv) in circular order
            constexpr int du[16] = {0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3, -3, -3, -2, -1};
            constexpr int dv[16] = {-3, -3, -2, -1, 0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3};
            const int c = tile[row + kHalo][tx + kHalo];
            int r[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) r[k] = tile[row + kHalo + dv[k]][tx + kHalo + du[k]];
            // min and max of every circular window of 9: windows of 2, 4, 8, then 9
            int a2[16], b2[16], a4[16], b4[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a2[k] = min(r[k], r[(k + 1) & 15]);
                b2[k] = max(r[k], r[(k + 1) & 15]);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a4[k] = min(a2[k], a2[(k + 2) & 15]);
                b4[k] = max(b2[k], b2[(k + 2) & 15]);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int mn = min(min(a4[k], a4[(k + 4) & 15]), r[(k + 8) & 15]);
                const int mx = max(max(b4[k], b4[(k + 4) & 15]), r[(k + 8) & 15]);
                s = max(s, max(mn - c - 1, c - mx - 1));
            }
        }
        const long long p = (long long)v * W + u;
        const float d = depth[p];
        const bool valid = (d >= dmin) && (d <= dmax);  // false for NaN and +-inf (finite bounds)
        if (score_out) score_out[p] = (short)s;
        key[p] = valid ? (short)s : (short)-1;
        if (valid && s >= 0) atomicAdd(&lh[s], 1);
    }
    __syncthreads();
    if (lh[tid]) atomicAdd(&hist[(blockIdx.y * gridDim.x + blockIdx.x) % kHistCopies * 256 + tid], lh[tid]);
}

// res = (threshold, count): count(t) = sum of hist[s >= t]; the threshold is
// the smallest t with count(t) <= cap (hist[255] is always 0, as scores never
// exceed 254, so t = 255 always qualifies).  Every workgroup finds it for
// itself (thread i holds count(255 - i), which grows with i) and counts its
// selected pixels.
__global__ __launch_bounds__(kSelThreads) void select_count_kernel(const short *key, long long npix, const int *hist,
                                                                   int cap, int *res, int *bcount)
{
    __shared__ int s_w[4], s_cnt[256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int k[kSelPix / kSelThreads];
#pragma unroll
    for (int j = 0; j < kSelPix / kSelThreads; ++j) {
        const long long p = (long long)blockIdx.x * kSelPix + j * kSelThreads + tid;
        k[j] = p < npix ? (int)key[p] : -1;
    }
    int h = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) h += hist[c * 256 + 255 - tid];
    h = wave_scan_add(h);
    if (lane == 63) s_w[wv] = h;
    __syncthreads();
    for (int w = 0; w < wv; ++w) h += s_w[w];
    s_cnt[tid] = h;
    const int ok = __syncthreads_count(h <= cap);
    const int t = 256 - ok;
    int n = 0;
#pragma unroll
    for (int j = 0; j < kSelPix / kSelThreads; ++j) n += __syncthreads_count(k[j] >= t);
    if (tid == 0) {
        bcount[blockIdx.x] = n;
        if (blockIdx.x == 0) {
            res[0] = t;
            res[1] = s_cnt[ok - 1];
        }
    }
}

// Row r of the output takes the r-th selected pixel in raster order:
// z = depth, x = (u - cx) z / fx, y = (v - cy) z / fy, each operation a
// rounded IEEE double (no contraction), then rounded to FP32; the feature row
// is copied unchanged.
// A block's selected pixels are contiguous rows of the output: the features are
// copied by all threads, value by value.
template <bool DIRECT>
__global__ __launch_bounds__(kSelThreads) void select_emit_kernel(const short *key, const float *depth,
                                                                  const float *feat, long long npix, int W, int D,
                                                                  double fx, double fy, double cx, double cy,
                                                                  const int *res, const int *before, float *xyz,
                                                                  float *fout)
{
#pragma clang fp contract(off)
    constexpr int kRows = kSelPix / kSelThreads;
    __shared__ int s_cnt[kRows][kSelThreads / 64], s_w[kSelThreads / 64];
    __shared__ int s_pix[kSelPix];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const long long base = (long long)blockIdx.x * kSelPix;
    const int t = res[0];
    bool sel[kRows];
    unsigned long long m[kRows];
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const long long p = base + j * kSelThreads + tid;
        sel[j] = p < npix && key[p] >= t;
        m[j] = __ballot(sel[j]);
        if (lane == 0) s_cnt[j][wv] = __popcll(m[j]);
    }
    long long r0 = 0;  // rows of the blocks before this one
    if (DIRECT) {
        int c = 0;
        for (int i = tid; i < (int)blockIdx.x; i += kSelThreads) c += before[i];
        c = wave_scan_add(c);
        if (lane == 63) s_w[wv] = c;
    } else {
        r0 = before[blockIdx.x];
    }
    __syncthreads();
    if (DIRECT)
        for (int w = 0; w < kSelThreads / 64; ++w) r0 += s_w[w];
    int n = 0;
#pragma unroll
    for (int j = 0; j < kRows; ++j)
        for (int w = 0; w < kSelThreads / 64; ++w) {
            if (w == wv && sel[j]) {
                const int r = n + __popcll(m[j] & ((1ULL << lane) - 1ULL));
                const long long p = base + j * kSelThreads + tid;
                s_pix[r] = j * kSelThreads + tid;
                const int u = (int)(p % W), v = (int)(p / W);
                const float zf = depth[p];
                const double z = (double)zf;
                float *o = xyz + 3 * (r0 + r);
                o[0] = (float)((((double)u - cx) * z) / fx);
                o[1] = (float)((((double)v - cy) * z) / fy);
                o[2] = zf;
            }
            n += s_cnt[j][w];
        }
    if (D == 0) return;
    __syncthreads();
    for (int e = tid; e < n * D; e += kSelThreads) {
        const int r = e / D;
        fout[r0 * D + e] = feat[(base + s_pix[r]) * D + (e - r * D)];
    }
}

int select_blocks(long long npix) { return (int)((npix + kSelPix - 1) / kSelPix); }
int select_hist_ints() { return 256 * kHistCopies; }

void launch_select(const SelectArgs &a, hipStream_t s)
{
    const long long npix = (long long)a.W * a.H;
    hipLaunchKernelGGL(fast_score_kernel, dim3((a.W + kTX - 1) / kTX, (a.H + kTRows - 1) / kTRows), dim3(kTX, kTY), 0,
                       s, a.gray, a.depth, a.W, a.H, a.dmin, a.dmax, a.key, a.score, a.hist);
    const int nb = select_blocks(npix);
    hipLaunchKernelGGL(select_count_kernel, dim3(nb), dim3(kSelThreads), 0, s, a.key, npix, a.hist, a.cap, a.res,
                       a.bcount);
    if (nb <= kDirectBlocks) {
        hipLaunchKernelGGL(select_emit_kernel<true>, dim3(nb), dim3(kSelThreads), 0, s, a.key, a.depth, a.feat, npix,
                           a.W, a.D, a.fx, a.fy, a.cx, a.cy, a.res, a.bcount, a.xyz, a.fout);
        return;
    }
    launch_exclusive_scan(a.bcount, a.boff, a.bsum, nb, nullptr, s);
    hipLaunchKernelGGL(select_emit_kernel<false>, dim3(nb), dim3(kSelThreads), 0, s, a.key, a.depth, a.feat, npix, a.W,
                       a.D, a.fx, a.fy, a.cx, a.cy, a.res, a.boff, a.xyz, a.fout);
}

}  // namespace cvo
