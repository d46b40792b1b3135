// cvo_internal.hpp -- shared host/device definitions of the gfx950 CVO library.
//
// Data layout in HBM (all arrays live in the handle's arena):
//   A cloud is prepared in one of two views, both holding sorted float4 copies
//   of the raw float32 coordinates (w unused) and sorted, padded feature rows
//   (stride D4 floats; SE columns pre-multiplied by sqrt(log2(e) / (2 ell_b^2))
//   so one exp2 of a plain sum of squares gives every SE factor, LIN columns
//   unscaled; padding columns are zero):
//     grid view    (reference side of a pair pass): points sorted by the
//                  row-major index of a uniform cell grid; a dense table
//                  cell_start[k] = first sorted index with cell >= k, so a
//                  run of cells along x is one contiguous index range.
//     cluster view (query side): points sorted along a Hilbert curve; a cluster is
//                  a run of at most cluster_max consecutive points (an aligned
//                  octree block, or part of a fixed-size chunk), with its
//                  centre and radius in the cloud's own frame.  A
//                  rigid motion keeps clusters compact, so they are built once
//                  per lengthscale band, never per iteration.
//   The views of several pairs are prepared together, both sides in the same
//   launches, by prefixing every sort key with the pair index; the plain path
//   is the batch of one.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cvo_limits.hpp"

namespace cvo {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 1;  // pair pass: one wave per workgroup, so a finished piece frees its slot at once
constexpr int kQueueCap = 80;    // LDS candidate queue per wave
constexpr int kQueueFlush = 16;  // process the queue once it holds this many (cap >= flush + 64)
constexpr int kTraceLen = 8;
constexpr int kRadixTile = 1024;  // keys per workgroup and pass of the radix sort
constexpr int kTableTiles = 128;  // sorts of at most this many tiles keep a digit table per pass (one launch a pass)
constexpr int kMaxPasses = 8;     // 8-bit passes over a 64-bit key
constexpr long long kCellCap = 1LL << 23;  // cells of one cloud's grid
// Bits per axis of the query order's curve.  The smallest octree block is within
// cluster_factor * r_c while the cloud's extent is within 2^19 of those edges, and
// the order resolves 16 parts of an edge within 2^15 of them.  With 16 bits (two sort
// launches a build fewer, 2 us) both ended at an eighth of that extent: 20,000 points
// and one 10^5 m off, ell 0.15: an evaluation 1,358 us, with 19 bits 520 us.
constexpr int kCurveBits = 19;
// Bits of a sort key: the curve's, and the pair above them (all 19 per axis up to 64
// pairs; the top bit stays clear, so no key is the all-ones mark of no point).
constexpr int kKeyBits = 63;
constexpr int kBoxBlocks = 64;    // partial bounding boxes per cloud
// Candidates of a piece, at least: as many as leave its pair about kPieceTarget
// pieces, within [kPieceFew, kPieceMany].  (Of the pair alone, so that its sums
// are the same bits whatever else is in the call.)  The chip holds 4,096-5,120 waves of the pair
// pass at once.  With fewer pieces than that the longest piece is the pass, so
// short pieces win; with many more, a piece's fixed cost and its partials do.
// Pair pass + reduction, us, at least 512 / 256 / 128 candidates / this rule:
// stereo 15,000 at ell 0.1 37.9 / 27.0 / 22.6 / 22.3, 30,000 at 0.1 41.6 / 31.5 /
// 34.2 / 31.3, 30,000 at 0.95 208 / 233 / 266 / 212, RGB-D 10,000 at 0.1 33.6 /
// 25.0 / 22.3 / 21.8, 40,000 at 0.1 75 / 81 / 99 / 75.  kPieceTarget 8,000 / 6,000
// / 5,000: stereo 8,000 at 0.95 41.6 / 37.5 / 37.2 against 37.2 here.
constexpr int kPieceFew = 128, kPieceMany = 512, kPieceTarget = 4000;
constexpr int kRedVals = 48;     // values reduced per pair by the reduction kernel
constexpr int kRedThreads = 256;

enum Status { ST_RUNNING = 0, ST_CONVERGED = 1, ST_MAX_ITER = 2, ST_NO_OVERLAP = 3, ST_STATIONARY = 4 };

// Holds a wave-uniform value in scalar registers at this point, so its load
// is issued here (with the others of its round) and not sunk past a branch.
__device__ __forceinline__ void in_sgpr(int v) { asm volatile("" ::"s"(v)); }
__device__ __forceinline__ void in_sgpr(double v) { asm volatile("" ::"s"(v)); }
__device__ __forceinline__ void in_sgpr(float v) { asm volatile("" ::"s"(v)); }
__device__ __forceinline__ void in_sgpr(long long v) { asm volatile("" ::"s"(v)); }

// Per-pair registration state, resident on the device for the whole ascent.
struct alignas(16) PairState {
    double T[12];        // current pose [R|t], maps the Z frame into the X frame
    double Tinv[12];     // inverse of the pose the state starts with (for the source-side backward
                         // pass; an ascent does not update it)
    double ell;          // current lengthscale
    double i_prev;       // indicator at the previous iteration (NaN: none)
    double F, i_theta, curv, r_max, dF_dell;
    double grad[6];
    double n_pairs;      // |P| of the last evaluation (exact integer in a double)
    double total_pairs;  // sum of |P| over the registration
    double rc_build;     // cutoff radius the current views were built for
    // lengthscale objective at the last evaluation (when it was asked for):
    // J = sum_{W_j > 0} log W_j - 3 |Z+| log ell, dJ/dell, its maximiser, |Z+|
    double J, dJ_dell, ell_ml, zplus;
    long long it;        // steps taken
    int status;          // Status
    int done;            // nonzero: later launches skip this pair
    int cls_built;       // pair-density class of the current views (-1: not chosen by density)
    int pause;           // nonzero: views must be rebuilt; launches skip the pair until then
};

// Density class of an evaluation from its in-cutoff pairs per query point
// (-1: unknown): 2 from t[0], 1 from t[1], else 0.
__host__ __device__ inline int density_class(double ppq, const double t[2])
{
    return !(ppq >= 0.0) ? -1 : (ppq >= t[0] ? 2 : (ppq >= t[1] ? 1 : 0));
}

// Per-pair constants of the ascent.
struct alignas(16) AlignConst {
    double ell_min, decay, ind_rel_tol, eps_rot, eps_trans, step_lambda;
    double sqrt_nm;      // sqrt(|X| |Z|)
    double inv_m;        // 1 / |Z|
    double kappa;        // cutoff radius / ell (infinite: no cutoff, views never rebuilt)
    double rebuild_ratio; // pause for new views once kappa ell < rebuild_ratio * rc_build
    long long max_iter;
    int fixed_iters;
    int metric;          // 0: kinetic-energy metric of the moving cloud, 1: identity
    int ell_mode;        // 0: annealing (Sec. IV), 1: adaptive (maximiser of the lengthscale objective)
    double ell_init;     // adaptive mode: upper clamp of ell
    int adaptive;        // nonzero: also pause when the density class drops below cls_built
    double cls_t[2];     // pairs per query where density classes 2 and 1 begin
    const double *ell_sched;  // replay: lengthscale of every iteration (device; null: annealing)
    long long n_sched;        // replay: iterations to run
};

// Uniform grid of one cloud (reference role).
struct alignas(16) GridDesc {
    double ox, oy, oz;   // origin (cell (0,0,0) starts here)
    double h;            // cell edge (m)
    double inv_h;        // 1 / h; a coordinate p lies in cell floor((p - o) * inv_h)
    int nx, ny, nz;
    int cell_base;       // offset of this cloud's table in cell_start
    long long pt_base;   // sorted points of this cloud: [pt_base, pt_base + n)
    long long n;
};

// Sorted query points of one pair: [pt_base, pt_base + n).
struct alignas(8) ClusterDesc {
    int pt_base, n;
};

// What a view build needs to know of one pair (uploaded; everything else is
// derived on the device).
struct alignas(16) PairIn {
    const float *xx, *xf;  // reference cloud: coordinates, features
    const float *zx, *zf;  // query cloud
    long long nx, nz;
    long long xb, zb;      // first sorted index of each cloud among its side's clouds
    double rc;             // cutoff radius (infinite: none)
    double pose[12];       // the pose of the queries to plan at
    double cell_factor, cluster_factor;
    int cluster_max;
    int octree;            // cluster rule: 1 octree blocks, 0 halved chunks
    int inverse;           // 0: queries are Z (pose T), 1: queries are X (pose T^-1)
    int pad;
};

// Cluster parameters of one pair, derived from its query cloud's box.
struct alignas(16) ClusterParam {
    double ox, oy, oz;     // origin of the curve's cube
    double iq;             // 1 / quantum (edge of a level-0 block)
    double cap;            // largest cluster bounding-box edge (chunk rule)
    int level;             // largest octree level of a cluster (octree rule)
    int bits;              // curve bits per axis of this pair
};

// State of one view build, on the device.
struct BuildInfo {
    unsigned long long slots;  // output slots planned
    long long cells;           // cell-table entries of all pairs
    int bad;                   // a cloud has a non-finite coordinate
    int overflow;              // the cell tables do not fit: nothing after the boxes was done
    int nclus;                 // clusters of all pairs
    int kbits, mbits;          // cell-index bits, curve bits per axis, the most of any pair (the pair index sits above)
    int sbits[2];              // key bits to sort: reference side, query side
    int passes;                // passes of the sort, the most of either side
    int hist[kCostBuckets];    // pieces per cost bucket
    // pieces planned (each block of the planner adds to this and to the slots: apart,
    // the two do not wait for each other)
    alignas(128) unsigned long long pieces;
};

// What kernels tell a waiting host without a copy: pinned host memory, written
// with system-scope stores.
constexpr int kMailStates = 4;
struct alignas(64) HostMail {
    // the counts of BuildInfo, then the number of the build they belong to
    unsigned long long pieces, slots;
    long long cells;
    int bad, overflow;
    unsigned long long build;
    unsigned long long pad[3];
    // one registration's progress: steps taken << 2 | paused << 1 | done
    unsigned long long progress;
    unsigned long long pad2[7];
    // evaluations of up to kMailStates pairs (the evaluation's fields only)
    PairState state[kMailStates];
};

// Geometry of a cluster in its own frame: the centre of its bounding box and
// the radius of its points about it.
struct Geo {
    double x, y, z, w;
};

// One cluster as planned: its geometry, its points, its pieces and slots.
struct alignas(16) ClusterRec {
    Geo geo;
    int first, n;              // sorted points [first, first + n)
    int cand;                  // candidates at the planning pose
    int np, slot;              // pieces, first output slot
    int b, inverse;            // pair, pose orientation
    int code, place;           // cost bucket of its pieces, their place in it
    int pad[3];
};

// Feature layout after combining the spec's blocks: all SE columns first
// (pre-scaled), then at most one LIN block.
struct FeatLayout {
    int sed, lind;     // SE columns, LIN columns of the kernel variant (padded)
    int d4;            // row stride (multiple of 4, >= sed + lind)
    int src_dim;       // D of the caller's rows
    // Several LIN blocks are folded into one by the tensor-product identity
    // of eq. (6), <u1 (x) u2, v1 (x) v2> = <u1, v1> <u2, v2>: destination LIN
    // column sed + c (c < prod lin_dim) holds prod_b u_b[digit_b(c)], the
    // digits of c in the mixed radix (lin_dim[0], ..., lin_dim[nlin - 1])
    // with block 0 most significant.  nlin = 0: at most one LIN block, mapped
    // column by column through col[].
    int nlin;
    int lin_src[8];    // first source column of each LIN block
    int lin_dim[8];    // its width
    int col[64];       // destination column -> source column (-1: zero padding; -2: tensor-product column)
    float scale[64];   // destination column scale (SE: sqrt(log2(e) / (2 ell_b^2)))
    double gscale[64]; // accumulated feature gradient -> dF/d(feature) (SE: 1/(scale ell_b^2))
    float sig2;        // sigma^2 * prod_b sigma_b^2 over SE blocks
};

// Arguments of the pair pass.  The unit of work is a piece: piece p of np
// takes every np-th 64-candidate chunk of one cluster's candidate list (the
// concatenation of its neighbourhood rows), so heavy clusters are split into
// pieces of similar work.  One wave per piece, pieces ordered heaviest first.
// One piece in dispatch order with what its wave needs first, gathered at
// planning time so the wave's prologue is one load: the piece (cluster's
// first point, p, np, first output slot), its pair, its cluster's points and
// geometry.
struct alignas(16) PieceRec {
    int4 pc;
    int b, first, n;
    int inverse;  // nonzero: queries are X points (pose T^-1)
    Geo geo;
};

struct PairPassArgs {
    // query side (cluster view)
    const float4 *qpts;
    const float *qfeat;
    const PieceRec *recs; // the pieces in processing order (heaviest first), with their cluster data
    int npieces;
    // reference side (grid view)
    const float4 *rpts;
    const float *rfeat;
    const int *cell_start;
    const GridDesc *grids;  // per pair
    // per-pair poses: T applied to query points, or T^-1 for pieces marked
    // inverse (the pair set itself is always decided with T)
    const PairState *state;
    float sig2;
    double kappa;           // +inf: no cutoff
    // Outputs.  A piece of a cluster of n queries owns n slots from its first
    // slot f, and in each array a block of (values per slot) n entries in which
    // the values follow one another over the queries: value v of query t is at
    // (values per slot) f + v n + t.
    double *oWD;    // forward: W, Dx, Dy, Dz
    float *oS;      // forward: S00, S01, S02, S11, S12, S22
    int *oCnt;      // forward: in-cutoff pairs
    // backward: D (3 values), sum w s', then d4 feature gradients
    double *oB;
};

}  // namespace cvo
