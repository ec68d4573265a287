// The row-tile path of an update step (rows.hip): networks narrow enough that one
// workgroup holds a tile of batch rows with their activations in LDS.
#pragma once

#include "kernels.h"

namespace spz {

// Everything from the replay sampling to the weight gradients is local to a batch row,
// so a workgroup takes a tile of 32 (bf16: or 64) rows through a list of operations (RowOp): the
// layers of the target action, the target and online critics, the losses and the backward
// chains. Weights come from packed images, activations and output gradients leave as
// packed images for the weight-gradient product. One 1 KB fragment of a packed image is
// what one wave feeds to one matrix instruction group: 64 lanes of 16 bytes, lane l = 32 h
// + r holding
//   weights        (row r of a 32-row block, k = KS s + KS/2 h + j)   KS = 8 (fp32), 16 (bf16)
//   batch tensors  (column r of a 32-column block, batch row KS g + KS/2 h + j)
// Fragments of a weight block are consecutive over the steps s; those of a batch tensor
// consecutive over its column blocks, then over the row groups g.
constexpr int ROW_MIN_TILE = 32;
constexpr int ROW_THREADS = 512, ROW_WAVES = ROW_THREADS / 64;
constexpr int ROW_MAX_BLOCKS = 4;   // 32-column blocks per wave of one operation

enum RowOpKind : int32_t {
  ROW_LOAD,      // sampled rows of the replay ring -> X (flags: RowLoadWhat)
  ROW_OBS,       // sampler observations -> X
  ROW_HIDDEN,    // H = relu(A W^T + b); ReLU mask bits at `mask`; pack: packed image of H
  ROW_Z,         // Z = A W^T + b (actor output)
  ROW_DGRAD,     // H = (H W) masked by the bits at `mask`; pack, part: column sums
  ROW_DACT,      // Z[net] = H W (gradient to the action)
  ROW_PACK,      // X or H (from_h) -> packed image; part: column sums
  ROW_DOT,       // critic output layer: q[net] = H w + b; then by flags: nothing, the TD
                 // target, the critic loss and dq (part: sums of dq), the actor loss and dq
  ROW_DZ,        // H = dq w masked by the bits at `mask`; pack, part; before: packed image
                 // hpack of H (flags 1: there already) and its sums weighted by dq (wpart)
  ROW_HEAD,      // policy head on Z -> action columns of X (flags 1: policy side, 0: target)
  ROW_HEAD_BWD,  // Z (action gradients) -> actor output gradient in H
  ROW_ACT        // sampler actions from Z
};
enum RowLoadWhat : int32_t { ROW_LOAD_NEXT, ROW_LOAD_SA, ROW_LOAD_S };
enum RowDotThen : int32_t { ROW_DOT_ONLY, ROW_DOT_TARGET, ROW_DOT_CLOSS, ROW_DOT_ALOSS };

// Operand of two nets where an operation covers both critics (nets = 2: waves 0-3 take net0,
// waves 4-7 net0 + 1), else of one.
struct RowOp {
  int32_t kind, net0, nets;
  int32_t nblk;     // 32-column blocks of the result (ROW_DOT, ROW_DZ: of H)
  int32_t steps;    // KS-deep steps of the product
  int32_t from_h;   // A operand: H (else X)
  int32_t mask;     // u16 index into the mask area, -1: none
  int32_t flags;
  int32_t split;    // products: waves per block, each with a range of the steps (a power of two)
  const void* w[2];          // packed weights (ROW_DOT, ROW_DZ: one row, operand type)
  const float* bias[2];
  void* pack[2];
  float* part[2];            // [tiles, 32 nblk] (ROW_DOT: [tiles, ROW_WAVES])
  float* wpart[2];           // [tiles, 32 nblk]
  void* hpack[2];
};

struct RowArgs {
  const RowOp* ops;
  int op0[2], nops[2];   // operations of the two halves of the grid (critic part, actor part)
  int tiles, parts, B;
  int tm;                // 32-row blocks per tile
  // LDS: byte offsets, strides in elements (ldx, ldh: operand type; zp, dp: floats, of the
  // actor output and of the action gradients in the Z area)
  int oX, ldx, oH, ldh, hnet, oZ, zp, dp, oV, oM, oS;
  int A, Ka, Ap, Kc, pa, O, sac;
  uint64_t seed; const int64_t* step;
  // replay ring, and the gathered batch in global memory (debug reads): [Bp, Kc] operands
  // (s | a) and (s' | 0), rewards, ends and ring rows
  const uint8_t* ring; int64_t row_bytes; int off_a, off_s2, off_r, off_d; uint32_t size;
  void *xsa, *xs2; float *r, *d; int32_t* idx;
  const uint8_t* warm[3]; int warm_lines;   // packed images to bring into L2: 128-byte lines of each
  const float* log_alpha;
  float gamma, lmin, lmax, noise, clip;
  float *y, *q1, *q2, *qp1, *qp2, *logp, *th, *se, *lm, *da;
  double *cpart, *apart;   // [tiles, ROW_WAVES] loss partials
  // sampler actions
  const float* obs; float* act; int stochastic; uint32_t counter; int64_t row0;
};

// Lets launch_rows use the whole LDS of a CU on the current device: once for each context, as
// the attribute is the device's and a first launch may be one that is being captured.
hipError_t prepare_rows(bool bf16);
// The caller's operations give no wave more than ROW_MAX_BLOCKS blocks. Sampler actions where
// obs is set, else halves of a step.
hipError_t launch_rows(bool bf16, const RowArgs& g, size_t lds, hipStream_t s);

// Weight gradients from packed images: job j gives part[slice][m block][n block][1024]
// float32 sums over the slice's row groups, each 32 x 32 block in accumulator order.
struct RowWJob {
  const void *a, *b;   // packed dz (mblk column blocks) and packed layer input (bcb, of which nblk are used)
  float* part;
  int mblk, nblk, bcb, slices, task0;
};
constexpr int MAX_ROW_WJOBS = 24;
// split (float32): the products run on bfloat16 parts of their operands, from ROW_SPLIT_ROWS
// batch rows on. Of a few rows each product's own rounding counts, and the float32 instructions
// are the nearer ones (one row: 1.03 times their distance from 64 bits, the largest element 1.4
// times), while a tile that is mostly padding takes the same time either way (2 x 64: 15 us).
constexpr int ROW_SPLIT_ROWS = 32;
struct RowWArgs { RowWJob j[MAX_ROW_WJOBS]; int n, tasks, groups; int split; int has_fin; FinishArgs fin; };
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
  int64_t fwd, tr;   // element offsets of the block's fragments in the packed images (tr < 0: none);
                     // kind 1: of the columns' operand image (fwd < 0: none)
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
