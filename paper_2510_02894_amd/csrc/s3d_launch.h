// s3d_launch.h -- host-side launchers of the kernels (one per pipeline step).
#pragma once
#include <hip/hip_runtime.h>

#include "s3d_internal.h"

namespace s3d {

// Per-ROI result record written by the finalisation kernel.
struct RoiResult {
  double out[6];
  double shape[11];  // the other Shape-class members (when moments were summed), order of SHAPE3D_CLASS_*
  long long n_in;    // inside voxels (when moments were summed)
  double vol_signed;
  long long V, T;
  long long ids[4][2];
  long long rows[4][2];
  long long cand[4];
  long long pairs2d;
  int status;
  int pad_;
};

// The small-mesh path (single ROIs): the four maximum squared distances
// (FP64 bits), the smallest id pair at each (id_lo * 2^32 + id_hi), the
// in-plane pair count and the ticket that finds the pair kernels' last
// workgroup.
struct SmallAcc {
  unsigned long long gmax[4];
  unsigned long long key[4];
  unsigned long long pairs2d;
  unsigned int ticket;
  unsigned int pad_;
};
constexpr long long kSmallMaxV = 16384;         // largest mesh the small path evaluates
// Larger ROIs go straight to the block-pair pass.  Whole call on one ellipsoid,
// small path against block-pair pass (us): uint8 28^3 60 / 75, 40^3 70 / 75, 48^3
// 82 / 72, 64^3 140 / 75, 100^3 (more than kSmallMaxV vertices) 124 / 83; soft (whose
// few thick bricks take as long in either) 32^3 87 / 102, 64^3 101 / 106, 80^3 267 / 154.
constexpr long long kSmallMaxVoxels = 1ll << 16, kSmallMaxSoftVoxels = 1ll << 18;
constexpr int kSmallOverflow = -100;             // status: more vertices than kSmallMaxV

// mesh.hip
// Dynamic LDS of the mesh kernels for ROIs with at most max_G row-groups per row.
size_t mesh_lds_bytes(int max_G);
// The small path's head (ROI record, cleared counts, case areas) and the
// mesh pass alone (no clearing, no case areas).
hipError_t launch_small_head(int dtype, const Roi& R, Roi* rois, long long* totals, SmallAcc* acc,
                             double* case_area, hipStream_t st);
hipError_t launch_mesh_core(int dtype, const Roi* rois, int n_rois, long long nbricks, int max_G,
                            double* case_area, BrickPart* part, unsigned long long* tmpkey, double* tmpt,
                            long long tmp_cap, long long* totals, int moments, hipStream_t st);
// small.hip: every pair of the staged vertices exactly (vmax at most, at
// most kSmallMaxV), in two persistent kernels of n_groups workgroups, then
// the ROI's result in res[0].  acc: small_acc_bytes() of device memory (the
// accumulators, then per-tile maxima).
size_t small_acc_bytes();
hipError_t launch_small_pairs(int dtype, const Roi* rois, const BrickPart* part, long long nbricks,
                              const double* case_area, const unsigned long long* tmpkey, const double* tmpt,
                              const long long* totals, long long vmax, SmallAcc* acc, int n_groups,
                              RoiResult* res, hipStream_t st);

// The bit pass over the volumes of a table of dense ROIs without labels
// (Roi::bits_begin, bitblk_begin): workgroups of rounds (1 or kBitRounds) times
// kBitRound elements; map: [n_blocks] scratch for the ROI of each.
constexpr int kBitRound = 4096, kBitRounds = 4;
struct VolumeBits {
  uint32_t* bits;
  int* map;
  long long n_blocks;
  int rounds;
};

// The mesh pass (one read of the volume): clears counters[0, n_counters),
// then per brick its BrickPart and its vertices' keys (and soft t) in the
// staging list (rows below tmp_cap are written; totals[8] counts all).
// case_area: [n_rois * 512] scratch for the binary masks' per-case areas and
// active-cube counts (case_hist);
// moments: also the inside-voxel moments;
// bmap: [nbricks] scratch for the brick -> ROI map of a batch (unused, and may
// be null, for one ROI).
// vb: the bit pass to run first, from whose strings the mesh pass then cuts its
// tiles, or null (the bricks read the volumes themselves).
// one: host ROI record of a call with one ROI, which the launch then stores in
// rois[0] (null: rois is already there).
hipError_t launch_mesh_pass(int dtype, Roi* rois, int n_rois, long long nbricks, int max_G,
                            double* case_area, BrickPart* part, unsigned int* counters, int n_counters,
                            unsigned long long* tmpkey, double* tmpt, long long tmp_cap, long long* totals,
                            int moments, int* bmap, float4* pbox, const VolumeBits* vb, const Roi* one, hipStream_t st);
// Per-ROI totals and each brick's first row within its ROI (brick_voff);
// prune_min_v: ROIs with at least this many vertices get the pruning pass's column-pair offsets.
hipError_t launch_mesh_totals(const Roi* rois, int n_rois, int dtype, const double* case_area, const BrickPart* part,
                              long long* brick_voff, RoiMeta* meta, long long* totals, int moments, int prune_min_v,
                              hipStream_t st);
// The capacity check (rows0_cap rows; *overflow raised and every ROI emptied
// beyond it), the 3D segments, and layout 0 from the staging list (tmp_cap
// rows): keys, soft t, pair-pass operands (pos, or posh when set), orig and
// block tags.
hipError_t launch_mesh_rows(const Roi* rois, int n_rois, long long nbricks, const BrickPart* part,
                            const long long* brick_voff, RoiMeta* meta, long long* totals, long long rows0_cap,
                            const unsigned long long* tmpkey, const double* tmpt, long long tmp_cap,
                            unsigned long long* key, double* tsoft, float* pos, uint4* posh, int* orig, int* blkseg,
                            Seg* segs, unsigned int* overflow, const int* bmap, hipStream_t st);

// The mesh pass's vertices in blocks of 32 staged rows, and the block-pair
// pass over them (blocks.hip).
struct BlockBufs {
  const Roi* rois;
  int n_rois;
  const RoiMeta* meta;
  const long long* totals;  // [8] staged rows, [9] blocks in ROI order (each ROI's padded to a superblock)
  const unsigned long long* key;  // [rows_cap] staged keys
  const double* t;                // [rows_cap] soft masks' interpolation parameters, else null
  long long rows_cap;
  const float4* pbox;  // [2 * rows_cap / 32] box of each staged block: lo x 3, hi x 3 (half voxels)
  const int* lphys;    // [lblk_cap] staged block of each block in ROI order, -1: padding
  long long lblk_cap;
  float4* lbox;        // [2 * lblk_cap] boxes in ROI order, then the staged block's index
  const int* sbroi;    // [lblk_cap / kSuper] ROI of each superblock
  float4* sbox;        // [2 * lblk_cap / kSuper] superblock boxes, then the ROI and its superblocks from here on
  float4* prad;        // [rows_cap / 32] largest squared distance of a staged block's vertices from the centre of the ROI's
                       // box: over all axes, and without axis 0, 1, 2 (units of 2^(2 RoiMeta::ex))
  float4* srad;        // [lblk_cap / kSuper] the same of the superblocks
  int4* list;          // [list_cap] block pairs: staged blocks, ROI, bound and families
  unsigned long long* list_n;
  long long list_cap;
  GroupRes* gres;      // [4 * n_rois]
  int cu_count;
  bool ids32;          // every canonical vertex id of the call is below 2^32
};
// again: also the kernels that serve a list that was too short (*list_n tells;
// without them the results of such a call are not valid); ev: optional events
// after the boxes, the listing and the exact maxima.
hipError_t launch_blocks(const BlockBufs& B, bool again, hipStream_t st, hipEvent_t* ev);

// What the totals pass writes for the block-pair pass (all null / 0 when the
// general pipeline follows).
struct BlockIndex {
  int* lphys;
  int* sbroi;
  GroupRes* gres;
  unsigned int* overflow;  // raised when more rows were staged than rows_cap
  long long rows_cap;
};

hipError_t launch_block_totals(const Roi* rois, int n_rois, int dtype, const double* case_area, const BrickPart* part,
                               RoiMeta* meta, long long* totals, int moments, const BlockIndex& X, hipStream_t st);

// labels.hip: the ROI table of labels 1..max_label of a dense uint8 label map
// (crop to each label's box, select the label), the voxel counts (counts,
// may be null) and the largest crop (max_dims, may be null).  The table's
// entries also hold the boxes while they are built.
hipError_t launch_label_rois(const unsigned char* lab, const long long dims[3], const double spacing[3],
                             int max_label, RoiDesc* rois, long long* counts, long long* max_dims, int cu_count,
                             hipStream_t st);

// ROI tables on the device: a caller's descriptors planned and validated in
// one workgroup (plan[0] = bricks, plan[1] = buckets), or one ROI by value.
hipError_t launch_plan_rois(const RoiDesc* in, int n, int dtype, const long long max_dims[3], const void* base,
                            long long alloc_elems, Roi* out, long long* plan, hipStream_t st);
hipError_t launch_set_roi(const Roi& R, Roi* out, hipStream_t st);

// scan.hip: exclusive scan of n int64 (n known on the host); total -> *total.
// With n_dev set, only the first min(n, *n_dev) elements are scanned (a count
// known on the device only): later tiles cost an early exit and their outputs
// are left unwritten.  tmp must hold scan_tmp_elems(n) int64.
long long scan_tmp_elems(long long n);
hipError_t launch_scan(const long long* in, long long* out, long long n, long long* total, long long* tmp,
                       hipStream_t st, const unsigned int* n_dev = nullptr);

// Tile sizes of the pair pass (chosen by the autotuner; results do not depend on them).
struct Tuning {
  int itile;          // 16-row blocks per wave: 2, 4 or 8 (kernel 1: 4 or 8)
  int jchunk;         // 16-row column blocks per work item: 64, 128, 256 or 512
  int blocks_per_cu;  // persistent workgroups per CU (0: as many as fit)
  int kernel;         // 0: FP32 16x16x4 MFMA; 1: split-f16 32x32x16 MFMA
  int prune;          // 1, 2: only block pairs that can reach a diameter (kernel 1); 0: all pairs
  int small_path;     // 1: small single ROIs take the exact all-pairs kernel after the mesh pass
};

// Buffers of the diameter passes.
// What a per-brick kernel needs to find a brick's vertices in layout 0.
struct BrickArgs {
  const Roi* rois;
  int n_rois;
  const RoiMeta* meta;
  const BrickPart* part;       // [nbricks] the mesh pass's per-brick records
  const long long* brick_voff;  // [nbricks] each brick's first vertex within its ROI
  const int* bmap;             // [nbricks] brick -> ROI map, or null (then the ROI table is searched)
  long long nbricks;
};

struct PairBufs {
  const Roi* rois;
  int n_rois;
  long long nbricks;            // bricks of the mesh pass (its grid)
  const BrickPart* part;        // [nbricks]
  const long long* brick_voff;  // [nbricks]
  const int* bmap;              // [nbricks] or null
  int brick_win;                // LDS plane-key windows of the per-brick bucket kernels (at most 2,048)
  const RoiMeta* meta;
  const unsigned long long* key;
  const double* tsoft;  // null for binary masks
  float* pos;
  uint4* posh;          // split-f16 B operands, 32 B per row (kernel 1)
  int* orig;
  float* rowmax;
  int* blkseg;
  Seg* segs;
  long long rows0;      // layout-0 rows (host copy)
  long long n_buckets;  // plane buckets of all ROIs
  unsigned int* bcnt;   // [n_buckets]
  unsigned int* bcur;   // [n_buckets]
  long long* bsz;       // [n_buckets]
  long long* bflag;     // [n_buckets]
  long long* brow;      // [n_buckets]
  long long* bseg;      // [n_buckets]
  int4* bbox;           // [n_buckets] key-coordinate boxes of the plane buckets (pruning)
  int* bgroup;          // [n_buckets] group roi * 4 + 1 + axis of each plane bucket
  long long seg_cap;    // n_rois + n_buckets
  long long* ncol;      // [seg_cap]
  long long* colbase;   // [seg_cap]
  long long col_cap;
  Col* cols;            // [col_cap]
  long long* nitem;     // [col_cap]
  long long* itembase;  // [col_cap]
  long long* totals;    // device scalars: see pairs.hip
  long long* scan_tmp;
  unsigned int* counters;  // [1] candidates, [2] overflow flag; pair-pass work counters from word kWorkStride
  GroupRes* gres;          // [4 * n_rois]
  long long cand_cap;      // candidate capacity: every row could be one
  int* cand;               // [cand_cap]
  long long* cand_nch;     // [cand_cap] chunks of each candidate's segment
  long long* cand_chbase;  // [cand_cap] prefix sum of cand_nch
  long long max_rows_seg;  // bound on rows of one segment
  long long rows_bound;    // bound on rows of all layouts (allocation)
  Tuning tune;
  RoiResult* res;          // [n_rois]
  long long* pairs2d;      // [n_rois] in-plane pairs n*(n-1)/2 summed over buckets
  int cu_count;
  bool moments;            // RoiMeta holds inside-voxel moments: finalise the whole Shape class
  bool ids32;              // every canonical vertex id of the call is below 2^32 (packed tie-break)
  // 3D pruning (prune.hip), kernel 1 only: when `prune` is set the 3D
  // segments run from the pruned item list instead of the work list
  bool prune;
  int prune_min_v;         // ROIs with at least this many vertices are pruned, the others run all pairs
  BlkRec* blkrec;          // [rows0 / 32] per 32-row block of layout 0
  RoiSeed* rseed;          // [n_rois]
  PItem* pitems;           // [pitem_cap]
  long long pitem_cap;
};

// soft.hip: adjoint of the soft-mask forward pass, for a table of ROIs.
// Cubes u in [-1, d-1]^3 have the flat index cube(u) = ((u0 + 1) (d1 + 1) +
// u1 + 1) (d2 + 1) + u2 + 1, below 2^31 (checked on the host).
struct SoftBwdRoi {
  const float* p;             // the ROI's probabilities (d0, d1, d2)
  float* grad;                // dL/dp, same layout
  int d[3];
  int G;                      // row-groups (32 cubes) per cube row
  int nrg;                    // row-groups of a cube plane: (d1 + 1) G
  int nzc;                    // z-chunks of tz cube planes
  int tz;                     // cube planes per workgroup of the scan
  int shG;                    // floor(n / G) = (n * mG) >> shG for 0 <= n < 2^31
  unsigned int mG;
  double s[3];
  double o[3];                // origin of the signed volume sum (array centre)
  double g_area;              // dL/dSurfaceArea
  double g_vol_signed;        // dL/dMeshVolume * sign(signed volume)
  double gdiam[4];            // dL/dD_f / D_f (0 if the feature has no pair)
  long long pair_ids[4][2];   // canonical ids of the maximising pairs, -1 if none
  long long cube_begin;       // first entry of the ROI in the cube index
  long long brick_begin;      // first workgroup of the scan
  long long bitblk_begin;     // ... and of the bit pass
  long long bits_begin;       // first word of its bit string
};

struct SoftBwdBufs {
  const SoftBwdRoi* rois;     // [n_rois], DEVICE
  int n_rois;
  long long n_bricks;         // workgroups of the scan
  size_t scan_lds;            // its dynamic LDS
  long long n_bitblks;        // workgroups of the bit pass
  int bit_rounds;             // their size, 4,096 elements times 1 or kBitRounds
  uint32_t* bits;             // the ROIs' bit strings
  // room for the active cubes and the voxels at crossing edges of a mask with
  // the forward pass's V vertices (an edge lies in four cubes and a cube has at
  // least three crossing edges; an edge has two ends)
  long long cap_cubes, cap_vox;
  unsigned long long* cubes;  // [cap_cubes] min corner (pack_key with axis 0) and ROI
  int* croi;
  double* cgrad;              // [12][cap_cubes] per cube edge, the gradient's component along it
  float* egrad;               // [3][cap_cubes] the summed gradient of the edges from its min corner
  unsigned long long* vox;    // [cap_vox]
  int* vroi;
  unsigned int* index;        // per cube of every ROI: its place in the list (active cubes only)
  long long* counters;        // [4] crossing edges, listed cubes, listed voxels; packed: both in the fourth
  bool packed;                // neither list can pass 2^32 - 1 entries
  int cu_count;
  int* blk_roi;               // [n_bricks + n_bitblks] ROI of each workgroup of the scan, then of the bit
                              // pass, or null (then searched)
};
hipError_t launch_soft_backward(const SoftBwdBufs& B, hipStream_t st);

// pairs.hip
uint4* split_rows(const PairBufs& B);  // split-f16 operand rows (kernel 1), else null
hipError_t launch_buckets(const PairBufs& B, hipStream_t st);       // plane buckets, segments, work list
// prune.hip: boxes, lower bound and the pruned 3D work items (B.prune set)
hipError_t launch_prune(const PairBufs& B, hipStream_t st);
hipError_t launch_pair_maxima(const PairBufs& B, hipStream_t st);   // MFMA pass over the work list
hipError_t launch_init_groups(const PairBufs& B, hipStream_t st);   // reset group results, pair-pass counters, row maxima
hipError_t launch_refine(const PairBufs& B, hipStream_t st);        // candidates + exact FP64 passes
hipError_t launch_plane_counts(const PairBufs& B, hipStream_t st);  // in-plane pair counts from the staged keys
// per-ROI results; status SHAPE3D_ECAPACITY when the ROIs' rows (totals[0]) exceed rows0_cap
// and kListShort when more than list_cap block pairs were listed (totals[10])
constexpr int kListShort = -101;
hipError_t launch_finalize(const PairBufs& B, long long rows0_cap, long long list_cap, hipStream_t st);
// res -> out[nf * n_rois] (nf = 6, or 17 for the whole Shape class; not written for a negative
// status) and status[n_rois] (may be null), on the device
hipError_t launch_results_out(const RoiResult* res, int n_rois, double* out, int* status, int nf, hipStream_t st);
hipError_t launch_export_vertices(const unsigned long long* key, const double* tsoft, const RoiMeta* meta,
                                  const Roi* rois, long long* ids, double* pos, long long V, hipStream_t st);

}  // namespace s3d
