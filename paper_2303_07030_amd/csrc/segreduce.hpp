// Internal interface of the gather-reduce and SDDMM kernels.
#pragma once

#include "nsd_internal.hpp"

namespace nsd {

struct SgrParams {
    int32_t nseg = 0, nnz = 0, k = 0;
    nsd_plan plan{};                  // work items over the segments
    const int32_t *segptr = nullptr;  // [nseg+1]
    const int32_t *segidx = nullptr;  // [nnz] segment of each entry, sorted
    const int32_t *idx = nullptr;     // [nnz] row of X gathered by each entry
    const float *w = nullptr;         // weights (NULL: 1)
    const int32_t *wperm = nullptr;   // weight of entry p is w[wperm[p]]
    const float *X = nullptr;         // gathered dense operand (NULL: ones)
    float alpha = 1.f;
    float *out = nullptr;             // [nseg x k]
    float *part = nullptr;            // chunk partials (sgr_part_bytes)
    // Rows of `part` that hold a long segment's partials: its first chunk's
    // and, past it, those of the chunks at item indexes divisible by
    // chunk_stride (1: every chunk's; chunk_group<G>(): one per group of
    // slots, the group's chunks of a segment added together first, see
    // store_chunk_partial)
    int32_t chunk_stride = 1;
    int32_t item_blocks = 0;          // set by the launcher
};

struct SddmmParams {
    int32_t nnz = 0, k = 0, L = 0, nslots = 0;
    const int32_t *rowidx = nullptr;
    const int32_t *colind = nullptr;
    const float *X = nullptr;  // [nrows x k] (NULL: ones)
    const float *Y = nullptr;  // [ncols x k]
    float alpha = 1.f;
    float *out = nullptr;      // [nnz]
    const int32_t *operm = nullptr;  // entry p goes to out[operm[p]] (NULL: out[p])
    const float *w = nullptr;  // fused loss weights (NULL: no loss)
    double beta = 1.0;         // loss += beta * sum_p w_p * <X_i, Y_j>
    double *part = nullptr;    // [nblocks] block partials of the loss
};

struct SddmmShape {
    WidthPlan wp;
    int L;
    int64_t nslots, nblocks;
};

int choose_slot_len(int64_t nnz, int slots_per_wave);

// Entries per thread of the width-1 sampled product.
constexpr int kVec1SddmmEntries = 8;
size_t sgr_part_bytes(const nsd_plan &plan, int64_t nnz, int k);
nsd_status segreduce(SgrParams a, hipStream_t st);

// The loss total, run by one extra block of the last kernel of a call:
// *loss = sum of p1[0, n1) + sum of p2[0, n2) in a fixed order.
struct LossJob {
    const double *p1 = nullptr;
    int64_t n1 = 0;
    const double *p2 = nullptr;
    int64_t n2 = 0;
    double *loss = nullptr;  // NULL: no job
};

// A pass over a segmented sparse operand that also uses each segment's own
// dense row `own` (see dual.hip):
//   d_p = <own[seg_p], X[idx_p]>,  out[seg] = alpha * sum_p c_p X[idx_p],
// with c_p = w_p (kDualLin; then sdd[pos_p] = sdd_alpha * d_p when sdd is
// set, and loss += w_p d_p when count_loss) or c_p = w_p - d_p (kDualMf;
// loss += c_p^2 when count_loss).  pos_p = wperm[p] when the weights are
// permuted, else p.
// kDualSlice is kDualLin over k of the columns of wider rows, which lie `ld`
// floats apart in X, out and own; kDualSliceAdd the same where sdd[pos_p] holds
// the product over the columns before, which d_p then includes.  They are
// kinds of their own: with the rows' distance a value of every kernel (read
// from its arguments for the zeroed rows alone) the order-3 CP pass lost 1.4 to
// 2.7 % (10M entries, rank 48: 917 -> 927 us) and every small call 0.2 us.
constexpr int kDualLin = 0;
constexpr int kDualMf = 1;
constexpr int kDualSlice = 2;
constexpr int kDualSliceAdd = 3;
constexpr bool dual_sliced(int kind) { return kind == kDualSlice || kind == kDualSliceAdd; }

struct DualPass {
    SgrParams s;
    const float *own = nullptr;  // [nseg x k]
    float *sdd = nullptr;        // [nnz] sampled products at pos_p (kDualLin)
    float sdd_alpha = 1.f;
    int32_t count_loss = 0;
    int32_t item_blocks = 0, empty_blocks = 0;  // set by the launcher
    int32_t ld = 0;                             // kDualSlice, kDualSliceAdd
};

struct DualParams {
    DualPass pass[2];
    int32_t npass = 1;
    double *loss_part = nullptr;  // [dual_blocks] block partials (NULL: no loss)
    double loss_beta = 1.0;       // scale of every block partial
    LossJob early;                // a loss total over partials of earlier launches,
                                  // run by one extra block (when early.loss is set)
};

int64_t dual_blocks(const nsd_plan *const *plans, int npass, int64_t nnz, int k);
// The widths that a slot of one wave holds.
constexpr int kMaxFusedWidth = 256;
// Launches the passes and their long-segment combines, the last of which
// also runs `job` (when job.loss is set); a job without p1 sums the block
// partials of the dual kernel itself (f.loss_part).
nsd_status dual_fused(int kind, DualParams f, int probe_id, LossJob job, hipStream_t st);

// Fused SpMM-gradient passes (L = 1/2 ||A B||^2): rows = C = A B over the
// row plan with the loss; cols = a linear dual pass over the column plan
// (own = B, X = C): dB = seed A^T C and dA = seed <C_i, B_j>.
struct FrobParams {
    SgrParams rows;
    DualPass cols;
    double *loss_part = nullptr;  // [frob_row_blocks] row-pass block partials
    double *seg_loss = nullptr;   // [rows.plan.nlong] long-row partials
    double *loss = nullptr;
};

// One mode pass of the CP gradient: s is the gather-reduce over the mode's
// plan (segidx = mode coordinate, idx = coordinate of mode n+1, w = values,
// out = dF_n, alpha = -seed, k = rank); own = F_n, fa / fb = the factors of
// modes n+1 / n+2.  The first pass also writes the residual through perm.
struct CpMode {
    SgrParams s;
    const int32_t *idx_b = nullptr;
    const float *own = nullptr, *fa = nullptr, *fb = nullptr;
    const int32_t *perm = nullptr;
    float *resid = nullptr;
    float seed = 1.f;
    int32_t item_blocks = 0, empty_blocks = 0;  // set by the launcher
};

struct CpParams {
    CpMode m[3];
    double *loss_part = nullptr;
};

constexpr int kCpScalarWidth = 32;

// The lane layout of a fused CP pass over rows of `whole` quads or not, with
// plans of items of L entries.  Its items are short and its arithmetic long, so
// the quads win down to the narrowest ranks where there is work for them; one
// column per lane wins where a wave's items are few (cp3 of 20K entries, rank 7,
// us: 8.4 against 10.9; rank 13 9.2 / 9.7; rank 25 of 3K 8.6 / 9.0) or long (10M
// entries, rank 5, items of 12: 534 / 601; rank 10 of 24: 688 / 897), and at
// ranks 4 and 8, off 16-byte addresses here, where it leaves no lane idle (1M
// entries 43 / 48 and 53 / 56; cp4 of 10M, rank 8, 775 / 848).
inline WidthPlan cp_plan(int rank, bool whole, int64_t nnz, int L) {
    const bool scalar = rank <= 8    ? rank % 4 == 0 || L > 8 || nnz < (1 << 18)
                        : rank <= 16 ? L > 16 || nnz < (1 << 15)
                                     : nnz < (1 << 13);
    return narrow_plan(rank, whole || !scalar, kCpScalarWidth);
}
int64_t cp_blocks(const nsd_plan *plans, int rank);
nsd_status cp_fused(CpParams f, double *loss, hipStream_t st);

int64_t frob_row_blocks(const nsd_plan &rows, int64_t nnz, int k);
nsd_status frob_fused(FrobParams f, hipStream_t st);

SddmmShape sddmm_shape(int64_t nnz, int k, bool whole);
bool sddmm_whole(const SddmmParams &a);
nsd_status sddmm(SddmmParams a, hipStream_t st);

// Width-1 passes (vec1.hip): the gather-reduce (with a loss total of earlier
// partials on its combine launch), the linear dual pass (a job without p1
// sums the pass's own loss; `entries`: the operand's rows, columns and values
// in its own order with the dense operands, from which a small pass forms it)
// and the sampled product in `nblocks` blocks.
// vec1_max_tiles bounds the tiles of passes over up to nnz entries, one loss
// partial and two floats each.
nsd_status vec1_reduce(const SgrParams &a, LossJob job, hipStream_t st);
nsd_status vec1_dual(const DualPass &m, const SddmmParams &entries, double *loss_part,
                     int probe_id, LossJob job, hipStream_t st);
nsd_status vec1_sddmm(const SddmmParams &a, int64_t nblocks, hipStream_t st);
int64_t vec1_max_tiles(int64_t nnz);

nsd_status loss_finalize(const double *part, int64_t n, double *loss, hipStream_t st);

// *out = alpha * sum x_i y_i (y NULL: ones) in fp64, fixed order, plus the
// old *out when accumulating; part holds dot_blocks(n) doubles.
int64_t dot_blocks(int64_t n);
nsd_status dot(int64_t n, const float *x, const float *y, double alpha, bool accumulate,
               double *part, double *out, hipStream_t st);

// y = alpha x + beta y elementwise (x NULL: ones; beta 0: y is not read).
nsd_status axpby(int64_t n, float alpha, const float *x, float beta, float *y, hipStream_t st);
// out[p] = alpha where entry p's row equals its column, else 0.
nsd_status diag_keys(int64_t n, const int32_t *rowidx, const int32_t *colind, float alpha,
                     float *out, hipStream_t st);

}  // namespace nsd
