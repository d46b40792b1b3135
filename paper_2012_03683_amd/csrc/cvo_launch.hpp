// cvo_launch.hpp -- host-side launchers of the device kernels (internal).
#pragma once
#include "cvo_internal.hpp"

namespace cvo {

// Caller's buffers of one cloud.
struct CloudPtrs {
    const float *xyz;
    const float *feat;
    long long n;
};

// Arguments of the view build.  Side 0: reference clouds (grid view), side 1:
// query clouds (cluster view); their keys and sorted arrays hold all pairs'
// points one after another.
struct ViewArgs {
    const PairIn *in;
    int B;
    long long n[2];               // points per side
    float *box;                   // 2 B * kBoxBlocks partial boxes of 8 floats
    int boxblocks;                // partial boxes per cloud
    GridDesc *grid;               // B
    ClusterParam *cp;             // B
    // B: candidates of each pair's clusters.  Added to by every block of the cluster
    // kernel, so apart from what all of them read (beside the parameters, 8 million
    // points took 2.0 instead of 0.8 ms).
    unsigned long long *cand;
    BuildInfo *info;
    long long cell_cap;           // entries the cell table has room for
    // keys and values of both sides, [0, n[0]) and [n[0], n[0] + n[1]), and
    // the buffers the odd passes write
    unsigned long long *key[2];
    int *val[2];
    int *table;                   // digit tables of both sides, or the histogram of a large sort
    int *bsum;                    // scan scratch of a large sort
    int *cell_start;
    float4 *pts[2];
    float *feat[2];
    int *perm;                    // query side: sorted -> own cloud's index
    const PairState *state;       // of the pairs (for the callers; a plan's poses are in `in`)
    ClusterRec *clus;
    int4 *qmap;
    int work;                     // query x candidate products per piece
    PieceRec *recs;
    long long rec_cap;            // records there is room for
    HostMail *mail;               // record_kernel posts the build's counts here (may be null)
    unsigned long long build;     // its number
};
void launch_boxes(const ViewArgs &a, hipStream_t s);
void launch_params(const ViewArgs &a, hipStream_t s);
// keys, sort, sorted copies, cell tables, clusters and their plan
void launch_views(const ViewArgs &a, const FeatLayout &lay, double kappa, hipStream_t s);
void launch_records(const ViewArgs &a, hipStream_t s);
long long view_table_ints(long long n0, long long n1);  // entries of ViewArgs.table
long long view_bsum_ints(long long n0, long long n1);   // entries of ViewArgs.bsum

// (passes, on the device, may be null: nothing is done if pass is not below it)
void launch_exclusive_scan(const int *in, int *out, int *bsum, long long n, int *total, hipStream_t s,
                           const int *passes = nullptr, int pass = 0);

// pair pass: mode 0 = forward moments, 1 = backward (feature gradients), 2 = W and the
// pair count alone, its terms in FP64 (LIN columns without SE columns; other layouts take
// mode 0)
// returns false when no kernel exists for the feature layout
bool launch_pair_pass(const PairPassArgs &a, const FeatLayout &lay, int mode, hipStream_t s);

// Where a query's partial moments live: qmap[j] = (t, n, np, s0) for query j
// at position t of a cluster of n queries cut into np pieces; the cluster's
// pieces own consecutive blocks of n output slots from s0 - t on (see
// PairPassArgs for the values' places).  Partials are combined in piece order.
struct SlotMap {
    const int4 *qmap;
};

struct ReduceArgs {
    const float4 *qpts;
    const ClusterDesc *cdesc;  // per pair: query points [pt_base, pt_base + n)
    SlotMap map;
    const double *WD;          // per-piece partial moments (PairPassArgs.oWD, oS, oCnt)
    const float *S;
    const int *cnt;
    PairState *state;
    const AlignConst *ac;
    double *partials;          // B * kRedVals * nblk (per pair value-major: value v of block k at v * nblk + k)
    double *trace;             // B * trace_rows * kTraceLen, may be null
    long long trace_rows;
    HostMail *mail;            // progress (steps of one pair) or evaluations (B <= kMailStates); may be null
    int nblk;
    int mode;                  // 0: evaluate only, 1: evaluate and take an ascent step
    int ellobj;                // nonzero: also reduce the lengthscale objective's sums
    int one_query;             // nonzero: nblk * kRedThreads >= every cloud's query count (one query per thread)
};
void launch_reduce(const ReduceArgs &a, int B, hipStream_t s);

// backward post-processing: one or two sides, each the queries of one cloud
struct BackwardSide {
    const int4 *qmap;         // of the side's queries
    const int *qperm;         // sorted query index -> original index within its cloud
    int pose_is_inverse;
    long long n;
    float *dxyz;              // original-order output, n x 3 (may be null)
    float *dfeat;             // original-order output, n x src_dim (may be null)
    const float *src_feat;    // the query cloud's own feature rows (original order, n x src_dim), read
                              // for the chain rule through folded LIN blocks
    double *lsum;             // per block: the sum of its queries' L (may be null)
};
struct BackwardArgs {
    BackwardSide side[2];
    int nsides;
    const double *B;          // per-piece partial values (PairPassArgs.oB)
    const PairState *state;
    FeatLayout lay;
    double gF;
};
int backward_blocks(long long n);
void launch_backward_finish(const BackwardArgs &a, hipStream_t s);

// point selection (FAST scores, threshold, raster-order compaction)
struct SelectArgs {
    const uint8_t *gray;   // H x W
    const float *depth;    // H x W
    const float *feat;     // H x W x D (may be null if D == 0)
    int W, H, D;
    float dmin, dmax;      // valid depth range, compared in FP32
    double fx, fy, cx, cy;
    int cap;               // largest selection allowed
    short *key;            // H x W scratch: score if the pixel has depth, else -1
    short *score;          // H x W scores for the caller (may be null)
    int *hist;             // select_hist_ints(), zero on entry
    int *res;              // (threshold, count)
    int *bcount, *boff, *bsum;  // counts per select_blocks() block, their exclusive scan, scan scratch
    float *xyz;            // cap x 3
    float *fout;           // cap x D
};
void launch_select(const SelectArgs &a, hipStream_t s);
int select_blocks(long long npix);
int select_hist_ints();
void launch_sum_doubles(const double *in, long long n, double *out, hipStream_t s);

}  // namespace cvo
