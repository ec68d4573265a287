// The row-tile path of an update step (rows.hip): networks narrow enough that one
// workgroup holds a tile of batch rows with their activations in LDS.
#pragma once

#include "kernels.h"

namespace spz {

// Everything between the replay gather and the weight gradients is local to a batch row,
// so a workgroup takes a tile of 32 or 64 rows through a list of operations (RowOp): the
// layers of the target action, the target and online critics, the losses and the backward
// chains. Weights come from packed images, activations and output gradients leave as
// packed images for the weight-gradient product. One 1 KB fragment of a packed image is
// what one wave feeds to one matrix instruction group: 64 lanes of 16 bytes, lane l = 32 h
// + r holding
//   weights        (row r of a 32-row block, k = KS s + KS/2 h + j)   KS = 8 (fp32), 16 (bf16)
//   batch tensors  (column r of a 32-column block; batch rows 4 h + j (+ 8: bf16's j >= 4)
//                  of an 8-row (fp32) or 16-row (bf16) group)
// Fragments of a weight block are consecutive over s; those of a batch tensor consecutive
// over its column blocks. A batch fragment is four (eight) accumulator registers of the
// lane that computed them, so producing and consuming it needs no data movement.
constexpr int ROW_THREADS = 512, ROW_WAVES = ROW_THREADS / 64;
constexpr int ROW_MAX_BLOCKS = 4;   // 32-column blocks per wave of one operation

enum RowOpKind : int32_t {
  ROW_LOAD,      // batch operand tile -> X (flags 1: xsa, 0: xs2); pack[0]: packed image
  ROW_OBS,       // sampler observations -> X
  ROW_HIDDEN,    // H = relu(A W^T + b); ReLU mask bits at `mask`; pack: packed image of H
  ROW_Z,         // Z = A W^T + b (actor output)
  ROW_DGRAD,     // H = (H W) masked by the bits at `mask`; pack; part: column sums
  ROW_DACT,      // Z[net] = H W (gradient to the action)
  ROW_DOT,       // critic output layer: q[net] = H w + b
  ROW_TARGET,    // TD target
  ROW_CLOSS,     // critic loss and dq; part: sums of dq
  ROW_ALOSS,     // actor loss and dq
  ROW_DZ,        // H = dq w masked by the bits at `mask`; pack; part; wpart: sums of dq h
  ROW_HEAD,      // policy head on Z -> action columns of X (flags 1: policy side, 0: target)
  ROW_HEAD_BWD,  // Z (action gradients) -> actor output gradient in H; pack; part
  ROW_ACT        // sampler actions from Z
};

// Operand of two nets where an operation covers both critics (nets = 2: waves 0-3 take net0,
// waves 4-7 net0 + 1), else of one.
struct RowOp {
  int32_t kind, net0, nets;
  int32_t nblk;     // 32-column blocks of the result (ROW_DOT, ROW_DZ: of H)
  int32_t steps;    // KS-deep steps of the product
  int32_t from_h;   // A operand: H (else X)
  int32_t mask;     // u16 index into the mask area, -1: none
  int32_t flags;
  const void* w[2];          // packed weights (ROW_DOT, ROW_DZ: float32 row)
  const float* bias[2];
  void* pack[2];
  float* part[2];            // [tiles, 32 nblk] (ROW_CLOSS: [tiles])
  float* wpart[2];           // ROW_DZ: [tiles, 32 nblk]
  const void* hpack[2];      // ROW_DZ with wpart: packed image of H before it
};
static_assert(sizeof(RowOp) % 8 == 0, "read as 8-byte words");

struct RowArgs {
  const RowOp* ops;
  int op0[2], nops[2];   // operations of the two halves of the grid (critic part, actor part)
  int tiles, parts, B;
  int tm;                // 32-row blocks per tile
  // LDS: byte offsets, strides in elements (ldx, ldh: operand type; zp: floats)
  int oX, ldx, oH, ldh, hnet, oZ, zp, oV, oM;
  int A, Ka, Ap, Kc, pa, O, sac;
  uint64_t seed; const int64_t* step;
  const void *xsa, *xs2;
  const float *r, *d, *log_alpha;
  float gamma, lmin, lmax, noise, clip;
  float *y, *q1, *q2, *qp1, *qp2, *logp, *th, *se, *lm, *da;
  double *cpart, *apart;
  // sampler actions
  const float* obs; float* act; int stochastic; uint32_t counter; int64_t row0;
};

// max_blocks: the most blocks one wave takes in any operation (1 .. ROW_MAX_BLOCKS).
hipError_t launch_rows(bool bf16, const RowArgs& g, int max_blocks, size_t lds, hipStream_t s);

// Weight gradients from packed images: job j gives part[slice][m block][n block][1024]
// float32 sums over the slice's row groups, each 32 x 32 block in accumulator order.
struct RowWJob {
  const void *a, *b;   // packed dz (mblk column blocks) and packed layer input (bcb, of which nblk are used)
  float* part;
  int mblk, nblk, bcb, slices, task0;
};
constexpr int MAX_ROW_WJOBS = 24;
struct RowWArgs { RowWJob j[MAX_ROW_WJOBS]; int n, tasks, groups; int has_fin; FinishArgs fin; };
inline int row_wjob_tiles(int mblk, int nblk) { return ((mblk + 1) / 2) * ((nblk + 1) / 2); }
// Sets the jobs' task0 and the task count.
hipError_t launch_row_wgrad(bool bf16, RowWArgs& w, hipStream_t s);

// One workgroup of the reduction + Adam launch.
struct RowPBlk {
  int32_t kind;      // 0: a 32 x 32 weight block, 1: 16 columns of a vector, 2: a scalar, 3: log(alpha)
  int32_t net;       // 0 actor, 1 and 2 critics
  int64_t off;       // arena offset of element (0, 0)
  int32_t ld;        // row stride of the weight; kind 1: columns of the partials
  int32_t job;       // kind 0: index into RowPArgs::j
  int32_t blk;       // kind 0: block index in the job's partials
  int32_t fsteps, tsteps;
  int32_t pad_;
  int64_t fwd, tr;   // element offsets of the block's fragments in the packed images (tr < 0: none)
  const float* part; // kind 1, 2
};
struct RowPJob { const float* part; int64_t zstride; int slices; };
struct RowPArgs {
  AdamArgs a;
  const RowPBlk* blk; int first, count;
  RowPJob j[MAX_ROW_WJOBS];
  int vslices;
  void *PF, *PT, *TF;   // packed images: online, online transposed, target
  int update;           // 0: only rebuild the packed images from P and T
};
hipError_t launch_row_adam(bool bf16, const RowPArgs& p, hipStream_t s);

}  // namespace spz
