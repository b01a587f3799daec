// fl_internal.h - types shared by the engine (fl_engine.hip) and the gfx950
// kernels (fl_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fl {

constexpr int kMaxParams = 32;
constexpr int kMaxSlots = 256;                    // candidate slots a node record can hold
constexpr int kMaxWords = 5;                      // 64-bit words per node record
constexpr int kBlock = 256;                       // threads per workgroup (4 waves of 64)
constexpr int kCompactItems = 8;                  // raw configurations per thread in compaction
constexpr int kCompactTile = kBlock * kCompactItems;
// single-pass compaction of one space: 16 per thread, 4096 per tile (about
// 1 100 tiles at 4.7 M configurations, all resident at once with 32 KB of
// LDS staging each)
constexpr int kSingleItems = 16;
constexpr int kSingleTile = kBlock * kSingleItems;
constexpr int kXcds = 8;                          // MI355X: 8 XCDs, workgroups dealt round-robin
constexpr int kBatch = 16;                        // candidate slots whose loads are issued together
constexpr int kMaxFinishGrid = 1024;              // workgroups of the batched step kernel (grid-stride)
constexpr int kFinishBlock = 1024;                // threads of a step kernel workgroup (1 mod 3)
// Workgroups of the slot sweep per CU.  At the large workload (W = 2) a sweep
// with its step kernel takes 32.6, 29.1, 28.8, 27.4 and 31.2 us with 4 to 8
// of them, one with the lagged step 27.9, 25.2, 25.3 and 24.5 us with 4 to 7
// (its registers allow no more): the eighth costs more in L1 lines than its
// loads in flight gain.
constexpr int kSlotWorkgroups = 7;
constexpr int kListQuads = 4;                     // quads of a wave's in-edge lists read at once (16 steps)
// List sweeps of at most this many waves run one per workgroup, over as many
// CUs as there are (7.9 k nodes, 171 k edges: 4.6 us against 5.7 with four per
// workgroup; 125 k nodes 6.2 : 6.6).
constexpr int kLoneWaves = 2048;
// Slot spaces of at most this many edges are swept by in-edge lists.  Per
// sweep, lists against slots: 18 k nodes, 44 k edges 3.9 : 5.1 us; 124 k, 1.2 M
// 6.8 : 7.4; 215 k, 3.7 M 14.3 : 9.6; 886 k, 15 M 38.6 : 19.7.  Of 63 spaces of
// 0.2 to 1.8 M edges that the rule takes, lists are 0.93 to 2.1 times as fast;
// they lose where nodes are many and edges few (adjacent neighbours: 302 k
// nodes, 1.5 M edges 8.4 : 7.9 us).  From there to 3.2 M edges adjacent spaces
// lose up to a third (653 k, 3.1 M 15.3 : 10.0), Hamming spaces run from 0.89
// (111 k, 2.4 M 8.4 : 7.5) to 1.7 (228 k, 2.2 M 9.6 : 16.0).
constexpr int64_t kListEdges = 7 << 18;
constexpr int kPanelBlock = 512;                  // threads of a workgroup of the lagged binned sweep (8 waves)
constexpr int kFillStage = 6144;                  // col_idx entries of a tile assembled in LDS by the fill
constexpr int kSmallTiles = 16;                   // batch members of at most this many tiles iterate in one workgroup

// Mixed-radix description of a search space X = S_1 x ... x S_n, parameter 0
// most significant: stride[i] = prod_{j>i} radix[j].
struct SpaceDesc {
    int32_t n;
    int32_t n_raw;
    int32_t radix[kMaxParams];
    int32_t stride[kMaxParams];
};

// Candidate neighbour slots, numbered independently of the node: slot s moves
// one parameter by delta list positions, i.e. to raw index i + off[s] with
// off[s] = delta * stride of the parameter.  Hamming (eq. 2) gives parameter k
// the 2(radix_k - 1) deltas +-1 .. +-(radix_k - 1); adjacent gives +-1.  A
// slot exists for a node iff 0 <= x_k + delta < radix_k.  Slots are sorted by
// off, so ascending slot order is ascending neighbour raw index (= node id).
//
// Node record (words x 64 bits): bits [0, k) flag the slots that are in-edges
// of the node; in the last word, bits 24..31 hold out_deg and bits 32..63 the
// raw index.  words = 0 when k + 40 > 64 * kMaxWords (then only the generic
// kernels and the CSR sweep are used).
//
// A parameter's slots form two contiguous runs in slot order (every offset of
// a less significant parameter is below the stride of a more significant
// one): deltas -len..-1 at [neg, neg + len) and +1..+len at [pos, pos + len).
// par holds them with the parameter's divisor, in whole words of one scalar
// load, for the parameters of more than one value, least significant first:
// q / radix = mulhi(q, magic) >> shift for every q < 2^31 (magic =
// ceil(2^(31 + l) / radix) with 2^(l - 1) < radix <= 2^l, so magic < 2^32 and
// magic * radix - 2^(31 + l) < radix <= 2^l; Granlund and Montgomery 1994).
struct SlotParam {
    uint32_t magic, shift;
    int32_t radix;
    int32_t neg, pos, len;
};
struct SlotTable {
    int32_t k;
    int32_t words;
    int32_t n_par;
    int32_t off[kMaxSlots];
    SlotParam par[kMaxParams];
};

// Sizes produced on the device by the build scans, copied to the host once.
struct BuildSizes {
    int32_t n_valid;
    int32_t n_bad;       // fitness <= 0 or -inf
    float f_opt;         // minimum valid fitness
    int32_t n_minima;
    int64_t n_edges;
    int32_t n_plateau;   // minima with a neighbour of equal fitness
    uint32_t stamp;      // host copy: the stage's stamp, stored after everything else
};

// Where a build stage reports its sizes besides device memory: a pinned copy
// (or null) and the stamp the host waits for there.
struct HostSizes {
    BuildSizes *sizes;
    uint32_t stamp;
};

// In-edge lists per wave of 64 consecutive nodes: wave w's quad u of lane l is
// quad[(w * stride + u) * 64 + l], four byte offsets into x; quads[w] of them
// are used, a positive multiple of kListQuads.
struct WaveLists {
    uint4 *quad;
    int32_t *quads;
    int32_t stride;
};

// One space of a segmented build: every space of a batch runs each build
// stage in the same launch (the node-tile stages once per record width and
// buffer form), each workgroup finding its space and tile in a tile list.
// Fields are filled stage by stage as the sizes become known on the host.
struct SegBuild {
    SpaceDesc sp;
    SlotTable sl;
    const float *fit;
    // compaction (sizes known from n_raw)
    int32_t *tile_cnt, *tile_bad, *tile_off;
    float *tile_min;
    int32_t *remap, *valid_raw;
    float *fit_c;
    BuildSizes *sizes;
    // degree pass (after the compaction: N)
    int32_t *in_deg, *out_deg;
    uint64_t *rec, *presence;
    int32_t *off_table;
    int64_t *tile_e, *tile_eoff;
    int32_t *tile_m, *tile_moff;
    // CSR fill (after the degree pass: E)
    int32_t *row_ptr, *col_idx, *minima;
    WaveLists lists;
    int32_t c_tiles, n_tiles, n, n_edges, k_pad, fit_bytes, remap_bytes, pad;
};
struct SegTile {
    int32_t seg, tile;
};


// Power-iteration state, device resident.  The stored iterate y_k is the
// normalised rank vector up to the factor s = 1/sum(y_k).
struct PrState {
    int32_t k;           // iterations completed
    int32_t done;        // 0 running, 1 converged, 2 iteration cap reached
    uint32_t ticket;     // last-workgroup election, reset by the elected one
    int32_t worked;      // iteration launches that did work
    double s;            // 1 / sum(y_k)
    double c;            // d*(sink mass)/N + (1-d)/N for the next iteration
    double sigma;        // sum(y_k)
    double resid;        // ||r_k - r_{k-1}||_1
    double resid_prev;
    double sink;         // sum of y_k over sinks
    double score_num;    // sum of ranks over L_p
    double score_den;    // sum of ranks over L
    // Lagged step (PrArgs::lag): sweep j adds the teleport-and-sink term of
    // r_{j-1}, gam[j & 1][0], and the residual of r_j against r_{j-1} uses
    // gam[j & 1][1] as well (the term of r_{j-2}); gam[j & 1][2] is
    // gam[j & 1][0] over the initial iterate 1/N; the result is the iterate
    // r = w + out_gamma in y buffer out_buf, whose entries sum to out_sigma.
    double gam[2][3];
    double out_gamma;
    double out_sigma;
    int32_t out_buf;
    int32_t lag_pad;
};

// Row formats of the PageRank sweep.
enum SweepKind : int32_t {
    kSweepCsr = 0,    // pull over the CSR, L lanes per row, x indexed by node id
    kSweepSlots = 1,  // pull over the records' in-edge slot bits, x indexed by raw index
    kSweepBinned = 2, // pull over the CSR with rows binned by in-degree, each bin its own lanes per row
    kSweepLists = 3,  // pull over the waves' in-edge lists, x indexed by node id (n + 1 entries, the last 0)
    kSweepPanels = 4  // as kSweepBinned, by panels of rows (lagged step only)
};

// Rows binned by in-degree: bucket 0 holds in-degree 0, bucket b >= 1 the
// in-degrees [2^(b-1), 2^b), the last bucket everything above.  A mapping
// gives every bucket its lanes per row L and rows blocks per tile T; buckets
// with the same (L, T) form one class, whose rows (node ids, ascending) are
// contiguous in the plan's bin_rows array.  A tile of a class is T blocks of
// kBlock / L rows and writes one partial-sum triple.
constexpr int kBuckets = 8;
struct BinClass {
    int32_t row_begin;   // first entry of the class in bin_rows
    int32_t rows;
    int32_t tile_begin;  // index of its first tile (and partial triple)
    int16_t lanes;       // L
    int16_t blocks;      // T
};
struct BinTable {
    int32_t n_classes;
    int32_t tiles;       // total tiles = partial triples of a sweep
    BinClass c[kBuckets];
};
__host__ __device__ inline int bucket_of(int32_t deg) {
    if (deg <= 0) return 0;
    int b = 1;
    while (b < kBuckets - 1 && deg >= (1 << b)) ++b;
    return b;
}

// Buffers of one sweep of the lagged step: sweep j reads w_j, w_{j-1} and the
// partial sums of sweep j - 1, and writes w_{j+1}.
struct LagBuffers {
    const float *y_in, *y_prev, *x_in;
    float *y_out, *x_out;
    const double *part_in;
    double *part_out;
};

struct PrArgs {
    LagBuffers cur;         // set for every launch of a lagged sweep
    const int32_t *row_ptr;
    const int32_t *col_idx;
    const int32_t *out_deg;
    const int32_t *valid_raw;
    const uint64_t *rec;    // node records (SlotTable), slot sweep only
    const uint64_t *presence;  // per wave of 64 nodes: OR of their in-edge slot bits
    const int32_t *off;     // 2 k_pad entries: slot raw-index offsets (SlotTable.off, 0 past k_slots),
                            // then the byte offsets 4 (off[s] - off[0]) of the buffer-load sweep
    int32_t k_slots;
    int32_t k_pad;          // stride of off's two halves: k_slots rounded up to 64, plus 64
    float *y[3];            // iterate (node ids): y[k & 1] holds y_k; lagged step: y[j % 3] holds w_j
    float *x[2];            // y / out_deg (0 at sinks): node ids (CSR) or raw indices (slots)
    double *partials;       // 3 doubles per tile (slot sweep) or per workgroup (CSR sweep)
    PrState *st;
    int32_t n;              // N
    int32_t kind;           // SweepKind
    double d;               // damping
    double tol;
    int32_t max_iter;
    int32_t adjacent;
    int32_t x_bytes;        // slot sweep: bytes its buffer loads span (x from the most negative slot
                            // offset to the end plus the largest), when < 2^31; else 0 (plain loads)
    int32_t exact;          // 1: Jacobi sweeps u <- 1 + d P u to an exact fixed point (s = c = 1)
    WaveLists lists;          // list sweep
    const int32_t *bin_rows;  // binned sweep: node ids grouped by class
    BinTable bins;            // binned sweep: classes and tiles
    // Lagged step (lag != 0): the sweeps run back to back with no step
    // kernel.  Sweep j (the host passes j in `sweep`) writes one partial
    // triple per workgroup, as three arrays of part_stride doubles, to
    // buffer j & 1 of `partials`; its workgroup 0 first reduces the n_parts
    // triples sweep j - 1 wrote into the state that sweep j + 1 reads.
    // The stored iterate w_j leaves out the constant teleport-and-sink term
    // gamma_{j-1} of r_j = w_j + gamma_{j-1}, which only the next step
    // knows; g (node ids) holds the in-edge sums of the first sweep, whose
    // x is r_0 / out_deg with r_0 = y0 = 1/N everywhere, so g / y0 is
    // P^T D^-1 1 and gamma_{j-1} g / y0 is what the constant contributes to
    // the next edge sums.
    int32_t lag;
    int32_t sweep;
    int32_t n_parts;
    int32_t part_stride;
    int32_t block;     // threads per workgroup of the sweep (list sweep: 64 or kBlock; panels: kPanelBlock;
                       // else kBlock)
    int32_t reducer;   // 1: the step has a workgroup of its own (the first of grid + 1)
    int64_t n_sinks;
    uint64_t *progress;   // pinned host word the step reports to (may be null)
    float *g;
};

// One member of a batch: an FFG with its own power iteration, run together
// with the other members in segmented launches.  Device resident.
struct BatchMember {
    const uint64_t *rec;       // node records
    const uint64_t *presence;  // per-wave slot presence
    const int32_t *off;        // 2 k_pad entries, as in PrArgs
    const int32_t *valid_raw;
    const int32_t *out_deg;
    const int32_t *minima;
    const float *fit_c;
    float *y[2];
    float *x[2];               // raw-index space
    double *partials;          // 3 per tile: sum y, residual, sink sum
    PrState *st;
    double *out_pagerank;      // caller's outputs
    int32_t *out_minima;
    double d, tol, threshold;
    int32_t n, m, k_slots, k_pad, words, x_bytes, n_tiles, max_iter;
    // binned members (words == 0 in the batch's lists): CSR, bin rows and
    // classes; x indexed by node id; a sweep writes bins.tiles partial
    // triples (the initial iterate n_tiles, one per kBlock nodes)
    const int32_t *row_ptr, *col_idx, *bin_rows;
    const int32_t *xmap;       // node -> x index for the initial iterate (valid_raw, or null for node ids)
    int32_t n_parts;           // partial triples a sweep writes
    int32_t pad;
    BinTable bins;
};

struct TileRef {
    int32_t member;  // index into the member table
    int32_t tile;    // tile of that member (kBlock nodes)
};

// ---- launchers (fl_kernels.hip); all enqueue on `stream` ----
// Compaction of one space (two passes, no scan kernel): tile_cnt,
// tile_min and tile_bad hold ceil(n_raw / kSingleTile) entries.
hipError_t launch_compact_single(const float *fit, int32_t n_raw, int32_t *tile_cnt, float *tile_min,
                                 int32_t *tile_bad, int32_t *remap, int32_t *valid_raw, float *fit_c,
                                 BuildSizes *sizes, const HostSizes &host, hipStream_t stream);
// Segmented build stages (see SegBuild): `tiles` lists (space, tile) pairs,
// `ids` the spaces of the one-workgroup-per-space scans.
hipError_t launch_seg_compact(const SegBuild *segs, const SegTile *tiles, int32_t n_tiles, const int32_t *ids,
                              int32_t n_ids, hipStream_t stream);
hipError_t launch_seg_degree(const SegBuild *segs, const SegTile *tiles, int32_t n_tiles, int words, bool buf,
                             hipStream_t stream);
hipError_t launch_seg_degree_scan(const SegBuild *segs, const int32_t *ids, int32_t n_ids, hipStream_t stream);
hipError_t launch_seg_fill(const SegBuild *segs, const SegTile *tiles, int32_t n_tiles, int words, bool buf,
                           hipStream_t stream);
hipError_t launch_degree(const SpaceDesc &sp, const SlotTable &sl, int adjacent, const float *fit,
                         const int32_t *valid_raw, int32_t n, int32_t *in_deg, int32_t *out_deg,
                         uint64_t *rec, uint64_t *presence, int32_t *off_table, int32_t k_pad,
                         int64_t *tile_e, int32_t *tile_m, int64_t *tile_eoff, int32_t *tile_moff,
                         BuildSizes *sizes, const HostSizes &host, hipStream_t stream);
hipError_t launch_fill(const SpaceDesc &sp, const SlotTable &sl, int adjacent, const float *fit,
                       const int32_t *valid_raw, const int32_t *remap, const uint64_t *rec,
                       const uint64_t *presence, int32_t n, int32_t n_edges, const int32_t *in_deg,
                       const int32_t *out_deg, const int64_t *tile_eoff, const int32_t *tile_moff,
                       int32_t *row_ptr, int32_t *col_idx, int32_t *minima, const WaveLists *lists,
                       hipStream_t stream);
// What a slot space's fill leaves when its CSR is not wanted: with `lists` the
// lists instead of the CSR, with launch_fill_minima the minima alone.
hipError_t launch_fill_minima(const int32_t *out_deg, int32_t n, const int32_t *tile_moff, int32_t *minima,
                              hipStream_t stream);
hipError_t launch_seg_minima(const SegBuild *segs, const SegTile *tiles, int32_t n_tiles, hipStream_t stream);
hipError_t launch_pr_init(const PrArgs &a, int grid, hipStream_t stream);
hipError_t launch_pr_iter(const PrArgs &a, const SpaceDesc &sp, const SlotTable &sl, int lanes,
                          int grid, hipStream_t stream);
// The two halves of launch_pr_iter: the sweep kernel, then the step kernel.
hipError_t launch_pr_sweep(const PrArgs &a, const SlotTable &sl, int lanes, int grid, hipStream_t stream);
hipError_t launch_pr_step(const PrArgs &a, int grid, hipStream_t stream);
// Workgroups of the sweep kernel for this layout that fit on one CU at once.
hipError_t pr_iter_blocks_per_cu(const PrArgs &a, const SpaceDesc &sp, const SlotTable &sl, int lanes,
                                 int *blocks);
hipError_t launch_make_lists(const int32_t *row_ptr, const int32_t *col_idx, int32_t n, const WaveLists &wl,
                             hipStream_t stream);
hipError_t launch_pr_output(const PrArgs &a, double *pagerank, const int32_t *minima, int32_t m, int32_t *out_minima,
                            int32_t *out_valid, hipStream_t stream);
// Binning of the rows by in-degree class: class_of[b] is the class of bucket
// b.  Count per (class, node tile) into cnt (kBuckets x n_tiles, class-major),
// scan it into off and totals (kBuckets entries), write bin_rows.
hipError_t launch_bin_rows(const int32_t *row_ptr, int32_t n, const int8_t *class_of_dev, int32_t *cnt,
                           int32_t *off, int32_t *totals, int32_t *bin_rows, hipStream_t stream);
// One binned sweep restricted to the given table (the autotuner times one
// class at a time this way), without the step kernel.
hipError_t launch_pr_sweep_binned(const PrArgs &a, const BinTable &t, int grid, hipStream_t stream);
// Panels (one workgroup at a time each) of a lagged binned sweep.
int32_t bin_panels(const BinTable &t);
hipError_t launch_batch_sweep_binned(const BatchMember *members, const TileRef *tiles, const int32_t *range_dev,
                                     int grid, hipStream_t stream);
hipError_t batch_sweep_binned_blocks_per_cu(int *blocks);
hipError_t launch_score(const double *pagerank, const int32_t *minima, int32_t m,
                        const float *fit_c, double threshold, PrState *st, hipStream_t stream);
// C_p for n thresholds: num[j], den[j] = rank sums over minima below
// thresholds[j] and over all minima (one workgroup per threshold).
hipError_t launch_score_curve(const double *pagerank, const int32_t *minima, int32_t m, const float *fit_c,
                              const double *thresholds, int32_t n, double *num_den, hipStream_t stream);
// f_opt / f(m) for every minimum, and a histogram of it over n_bins equal
// bins of [0, 1] (hist zeroed here).
hipError_t launch_naive(const int32_t *minima, int32_t m, const float *fit_c, float f_opt, double *ratio,
                        int32_t n_bins, uint32_t *hist, hipStream_t stream);

// Batched power iteration.  `tiles` lists the tiles to work on; `members`
// lists member indices for the per-member kernels.  The sweep kernel reads
// its list's start and length (range_dev[0], range_dev[1]) and the step
// kernel its list length from device memory, so launches captured in a
// graph stay valid while the lists change between replays.
hipError_t launch_batch_init(const BatchMember *members, const TileRef *tiles, int32_t n_tiles,
                             const int32_t *member_ids, int32_t n_members, const int32_t *n_members_dev,
                             hipStream_t stream);
hipError_t launch_batch_sweep(const BatchMember *members, const TileRef *tiles, const int32_t *ranges_dev, int grid,
                              hipStream_t stream);
hipError_t batch_sweep_blocks_per_cu(int *blocks);
hipError_t launch_batch_finish(const BatchMember *members, const int32_t *member_ids, const int32_t *n_members_dev,
                               int grid, hipStream_t stream);
// Small members, one workgroup each (grid-stride):
// up to max_sweeps sweeps and steps per member, back to back in the
// workgroup, until it stops.
hipError_t launch_batch_small(const BatchMember *members, const int32_t *member_ids, int32_t n_members,
                              int32_t max_sweeps, int grid, hipStream_t stream);
hipError_t launch_batch_output(const BatchMember *members, const TileRef *tiles, int32_t n_tiles,
                               const int32_t *member_ids, int32_t n_members, PrState *states_out,
                               hipStream_t stream);
hipError_t launch_batch_states(const BatchMember *members, const int32_t *member_ids, int32_t n_members,
                               PrState *states_out, hipStream_t stream);

}  // namespace fl
