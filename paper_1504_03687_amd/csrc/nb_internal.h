// Internal declarations shared by the HIP translation units of libnbreg.
// Not part of the public ABI (that is include/nbreg.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace nb {

// Work-group shape of every force kernel: 256 lanes = 4 wave64s.
constexpr int kBlock = 256;
constexpr int kWave = 64;
// j bodies staged per LDS tile by the row-per-lane kernel.
constexpr int kTile = 256;
// Mixed precision: FP32 partial sums run over this many j before they are
// folded into the FP64 running sums.
constexpr int kFold = 32;
// j-ranges of less than this many bodies run the passes that settle rare pairs
// (neighbours) once per kFold bodies, larger ones those that do it at once.
constexpr int64_t kRunMaxBodies = 65536;
// Capacity of one split's neighbour segment in scratch.  A segment that
// overflows is rebuilt by the merge kernel from its j-range.
constexpr int kSegCap = 96;

// Position used for padding bodies in a partial LDS tile / past the end of a
// j-range: far away (finite in FP32 after the FP64 difference), mass 0, so the
// pair adds exactly zero and never passes the neighbour test.
constexpr double kFar = 1.0e18;

// Status bits (mirrors include/nbreg.h).
constexpr uint32_t kStOverflow = 1u, kStBadIndex = 2u, kStNonFinite = 4u;

// One body of the packed j-set that the scalar-operand row pass streams: one
// 64-byte line, read by scalar loads.
struct alignas(64) JRec {
    double x, y, z, vx, vy, vz, m;
    float m32;
    int32_t pad;
};
// Padding records behind a packed j-range: the last run of kFold bodies is
// completed with bodies that add nothing, and the pass loads two bodies ahead.
constexpr int64_t kRecPad = kFold + 2;

// A contiguous range of j-set bodies [j_begin, j_end) and the rows that see it.
struct ForceArgs {
    int64_t n;            // bodies in the whole concatenated arrays (plane stride)
    const double *xp;     // [3][n]
    const double *vp;     // [3][n]
    const double *m;      // [n]
    int32_t n_i;          // rows (plane stride of per-row arrays)
    const int32_t *i_block;
    const double *rs2;
    int32_t cap;          // caller's nb_cap
    // final outputs (used directly when splits == 1)
    double *acc, *jerk;   // [3][n_i]
    int32_t *nb_count, *nb_list;
    int32_t *overflow;
    uint32_t *status;
    // words the call's first kernel zeroes as it starts (null: none): the pack
    // kernel, or the force kernel of a split launch, which writes neither the
    // overflow word nor the refinement counter (the merge does), so no
    // separate clearing launch is needed.
    int32_t *clear0, *clear1;
    // packed j-set [n + kRecPad] (null: the pass streams the SoA planes
    // through LDS)
    JRec *packed;
    // split layout: split s covers j in [s * split_len, min(n, (s+1) * split_len))
    int32_t splits;
    int64_t split_len;
    // scratch (splits > 1): one slot per (row, split), slot = b * splits + split;
    // part [total_slots][kSlotComp], seg_cnt [total_slots],
    // seg_list [total_slots][kSegCap]
    int64_t total_slots;
    double *part;
    int32_t *seg_cnt;
    int32_t *seg_list;
    // mixed precision: rows whose estimated error is too large are appended
    // (row, j-range) to the redo list and recomputed in FP64 afterwards
    double redo_k;        // 2^-24 * safety / tolerance; 0 disables
    int32_t *redo_count;  // device counter, zeroed before the force kernel
    int32_t *redo_arrive; // work-groups done with the first refinement pass;
                          // zero between calls (the last arrival resets it)
    int32_t *redo_rows;   // [n_i]
    int32_t *redo_j0, *redo_j1;
    float near_factor;    // mixed: FP64 near field below near_factor * rs2
    int32_t redo_groups;  // work-groups of the refinement kernel
    int32_t redo_chunks;  // chunks per refined row (j-range / kRedoChunk, rounded up)
    int32_t redo_rcap;    // rows refined through the chunk-partials buffer
    double *redo_part;    // [redo_rcap][redo_chunks][6] chunk partials
};

// Refinement works on fixed chunks of kRedoChunk bodies so that a refined
// row's FP64 sum does not depend on how many rows were refined in the call.
constexpr int64_t kRedoChunk = 2048;
constexpr int kRedoRows = 2;   // refined rows of one j-range summed together
constexpr int64_t kRedoPartItems = int64_t(1) << 20;   // chunk partials held at most

// Components per slot: acc x,y,z, jerk x,y,z, and the two error-scale sums.
constexpr int kSlotComp = 8;
// Extra scratch for the redo list of n_i rows (row / j-range arrays and the
// chunk partials); the counter is a separate word owned by the caller, so
// that it outlives later reuse of the scratch.
int32_t redo_groups_for(int cu_count);
// max_len: longest j-range of any row of the launch.  rcap_limit > 0 bounds
// the rows summed through chunk partials (the others are summed one
// work-group per row, to the same bits), and with it the partials' bytes.
size_t redo_scratch_bytes(int32_t n_i, int64_t max_len, int32_t rcap_limit = 0);
void bind_redo_scratch(ForceArgs &a, void *base, int32_t *counter, int32_t groups,
                       int64_t max_len, int32_t rcap_limit = 0);
int32_t redo_grid(const ForceArgs &a, int rows_per_item);
// one_range: every row of the launch has the same j-range (single-block calls).
hipError_t launch_redo(const ForceArgs &a, bool one_range, hipStream_t s);

struct Plan {
    int mapping;        // 1 = row per lane (LDS j-tiles), 2 = row group per wave
    int rows_per_lane;  // mapping 1: 1, 2, 4;  mapping 2: rows per wave 1, 2, 4
    int splits;         // j-ranges (mapping 1: per work-group; mapping 2: per wave)
    int f64;            // 1: a mixed-precision request runs the FP64 kernels
    int step;           // row-per-lane mappings: splits in steps of this many bodies
                        // (0: kTile in mapping 1, kWave in mapping 3)
};

// Scratch bytes needed for a plan (0 when splits == 1).
size_t force_scratch_bytes(const Plan &p, int32_t n_i);
// Scratch bytes for 'slots' split slots, and binding of the slot arrays.
size_t slot_scratch_bytes(int64_t slots);
void bind_slot_scratch(ForceArgs &a, int64_t slots, void *base);
// Carves the scratch pointers of 'a' out of 'base'.
void force_bind_scratch(ForceArgs &a, void *base);

// Packed j-set of n bodies: scratch bytes, and the launch that fills it from
// the SoA planes (and zeroes the call's words).
size_t packed_bytes(int64_t n);
hipError_t launch_pack(const ForceArgs &a, hipStream_t s);

// Launchers (return hipError_t of the launch).
hipError_t launch_force(const Plan &p, bool mixed, const ForceArgs &a, hipStream_t s);
hipError_t launch_merge(bool mixed, const ForceArgs &a, hipStream_t s);
hipError_t launch_predict(int64_t n, double t, const double *x, const double *v,
                          const double *a, const double *jrk, const double *t0,
                          const double *m, double *xp, double *vp, float *m32,
                          hipStream_t s);
hipError_t launch_fill_i32(int32_t *p, int32_t value, int64_t count, hipStream_t s);
// Zeroes *a and, if b is not null, *b in one launch.
hipError_t launch_clear_words(int32_t *a, int32_t *b, hipStream_t s);

// Adjoint: one recompute pass over (row block, body block) items.
struct AdjointArgs {
    int64_t n;
    const double *xp, *vp, *m;
    int32_t n_i;
    const int32_t *i_block;
    const double *rs2;
    const double *w_a, *w_j;  // [3][n_i]
    double *gx, *gv, *gm;     // [3][n], [n]
    uint32_t *status;
    double *row_part;         // scratch [6][n_i]: per-row "-" terms (set by the launcher)
};
struct AdjointShape {
    int32_t row_block;       // rows per row block: 256 or 512
    int32_t tile;            // 64 or 128: bodies per LDS tile of 256-row blocks (512: 128)
    int64_t body_len;        // bodies per body block
    int64_t panel_blocks;    // row blocks per launch (their body sums are kept apart)
    bool index_in_gm;        // the bodies' row index lives in the gm output
};
// Most scratch an adjoint call asks for by itself (next to the 6 n_i row sums),
// and most rows of a panel (the threads of its row reduction fit 32 bits).
constexpr size_t kAdjointBytes = size_t(1) << 30;
constexpr int64_t kAdjointPanelRows = int64_t(1) << 25;
// budget: bytes of scratch there may be (SIZE_MAX: any)
AdjointShape adjoint_shape(int64_t n, int32_t n_i, int cus, size_t budget);
size_t adjoint_scratch_bytes(int64_t n, int32_t n_i, const AdjointShape &sh);
hipError_t launch_adjoint(const AdjointArgs &a, const AdjointShape &sh, void *scratch,
                          hipStream_t s);

// Batched ensemble: clusters of the concatenated arrays.
struct BCluster {
    int64_t j_begin, j_end;   // bodies of the cluster
    int64_t split_len;        // j per split
    int64_t slot_base;        // first slot of the cluster (splits > 1 only)
    int64_t rec_base;         // packed ensembles: record of body j_begin
    int32_t row_begin;        // rows of the cluster
    int32_t n_rows;
    int32_t splits;
    float near;               // mixed: near-field factor of this cluster
};
struct BItem {
    int32_t cluster;
    int32_t row0;             // first row of the item's row tile
    int32_t split;
    int32_t pad;
};
struct BatchArgs {
    ForceArgs f;              // n, arrays, outputs, total_slots/part/seg_*
    const BCluster *clusters;
    const BItem *items;
    int32_t n_items;
    int32_t n_clusters;
    int32_t *queue;           // work counter, zeroed before each launch
    const int32_t *merge_rows;   // rows of clusters with splits > 1
    const int32_t *row_cluster;  // cluster of each merge row
    int32_t n_merge_rows;
    int32_t max_splits;          // largest split count of any cluster
};
// Shapes the batched kernel is built for: LDS tile length (j bodies per
// tile), work-group lanes, and rows per lane (a row tile is lanes x rows).
struct BShape {
    int tile;
    int lanes;
    int rows_per_lane;
};
constexpr int kBatchedShapes = 6;
constexpr BShape kBatchedShape[kBatchedShapes] = {
    {256, 256, 1}, {256, 256, 2}, {128, 128, 1}, {64, 64, 1}, {512, 512, 1}, {256, 512, 1}};
// j-splits of the batched ensemble are multiples of this many bodies (or of
// the ensemble's split length, where that is shorter), for every shape, so a
// cluster's split boundaries (and so its sums) depend only on its split count.
constexpr int kSplitUnit = 256;
// Index of a shape in kBatchedShape, or -1.
int batched_shape_index(int tile, int lanes, int rows_per_lane);
// packed: the scalar-operand kernel (items of one wave, kWave rows) instead of
// the LDS kernel of the shape; run: the one that settles rare pairs by runs.
hipError_t launch_batched(bool mixed, int shape, bool packed, bool run, int grid,
                          const BatchArgs &a, hipStream_t s);
hipError_t launch_batched_pack(const BatchArgs &a, hipStream_t s);
hipError_t launch_batched_merge(const BatchArgs &a, hipStream_t s);
int batched_max_blocks_per_cu(bool mixed, int shape, bool packed, bool run);

}  // namespace nb
